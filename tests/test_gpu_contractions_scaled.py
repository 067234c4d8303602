"""The float32 contractions with a float64 B at 64 and 129 active orbitals, whose energies (hundreds of Hartree and
more) exceed what an absolute bar allows for: rounding B to float32 changes each element by up to 6e-8, the energy by
a random sum of such terms.  Bars: 2e-9 of |E|; lambda, J and K 2e-6 of their largest element (129 products of two
float32 factors summed in float32: 11 x 6e-8 expected, thrice that)."""
import numpy as np
import pytest
import torch

import synth
from oracle import pnof, stream

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("nbf,naux,npairs,ncwo,tuning", [(64, 20, 32, 1, {"nsplit_b": 3, "nsplit_y": 7}), (64, 20, 32, 1, {}),
                                                         (131, 24, 43, 2, {"nsplit_b": 1, "nsplit_y": 1}), (131, 24, 43, 2, {})])
def test_float32_from_float64_integrals(nbf, naux, npairs, ncwo, tuning):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context(0)
    inst = synth.make(synth.Workload("edge", nbf, naux, npairs, ncwo, "f64"), 23)
    n = pnof.on_sigmoid(inst.gamma, npairs, ncwo)
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, P.FP32, P.INTS_DF_F64)
    ctx.set_tuning(**tuning)
    a = ctx.lagrangian(prob, t(inst.C), t(n), t(inst.H), t(inst.B), jk=True)
    torch.cuda.synchronize()
    orc = stream.lagrangian(inst.C, n, inst.H, inst.B, npairs, ncwo, pnof.PNOF7)
    assert abs(a["E"].item() - orc["E"]) < 2e-9 * abs(orc["E"])
    for k in ("lam", "J", "K"):
        assert np.max(np.abs(a[k].cpu().numpy() - orc[k])) < 2e-6 * np.max(np.abs(orc[k])), k
