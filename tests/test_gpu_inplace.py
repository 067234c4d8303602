"""pnof_lagrangian with the gradient written over the orbitals (dE/dC in C's buffer, which every part of the step
has read before): bit for bit the outputs of separate buffers, in each precision and form of the integrals."""
import numpy as np
import pytest
import torch

import synth
from oracle import pnof

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0)


@pytest.mark.parametrize("prec,ints", [(P.FP64, "f64"), (P.FP32, "bf16"), (P.BF16_SPLIT, "bf16"), (P.BF16_SPLIT, "f64"), (P.FP64, "eri4")])
@pytest.mark.parametrize("nbf,npairs,ncwo", [(24, 5, 1), (24, 6, 3), (61, 7, 4)])
def test_gradient_in_place_of_the_orbitals(ctx, nbf, npairs, ncwo, prec, ints):
    inst = synth.make(synth.Workload("inplace", nbf, 4 * nbf, npairs, ncwo, "f64"), 7)
    n = t(pnof.on_sigmoid(inst.gamma, npairs, ncwo))
    flat = inst.B.reshape(4 * nbf, -1)
    B = inst.B if ints != "eri4" else flat.T @ flat
    B = t(B).to(torch.bfloat16) if ints == "bf16" else t(B)
    kind = {"f64": P.INTS_DF_F64, "bf16": P.INTS_DF_BF16, "eri4": P.INTS_ERI4_F64}[ints]
    prob = P.problem(nbf, 0 if ints == "eri4" else 4 * nbf, npairs, ncwo, P.PNOF7, prec, kind)
    C, H = t(inst.C), t(inst.H)
    ref = ctx.lagrangian(prob, C, n, H, B, jk=True)
    out = {k: torch.empty_like(v) for k, v in ref.items() if k != "dEdC"}
    P.pnof_lagrangian(ctx, prob, C, n, H, B, out["lam"], out["E"], C, out["dEdn"], out["max_asym"], out["J"], out["K"])
    torch.cuda.synchronize()
    for k in out:
        assert torch.equal(out[k], ref[k]), k
    assert torch.equal(C, ref["dEdC"])
