"""The float64 and float32 three-index contractions at the edges of their tiles: active orbitals at, below and
past one 64-wide tile (and, with several tiles, both orientations of the stored half of W), stacked rows of B
that end inside a tile and inside a 16-long slab, B in both storage types, and chunks and splits that do not
divide the rows.  Bars: the precisions' own against the float64 oracle (float64 1e-8 Ha and 1e-10 on lambda;
float32 1e-6 Ha and 2e-5)."""
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


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0)


# nbf, naux, npairs, ncwo (active: npairs (1 + ncwo)), tuning
SHAPES = [(3, 5, 1, 1, {}), (17, 40, 3, 2, {"pchunk": 7}), (63, 33, 21, 2, {}), (64, 20, 32, 1, {"nsplit_b": 3, "nsplit_y": 7}),
          (65, 21, 13, 4, {"pchunk": 8}), (131, 24, 43, 2, {"nsplit_b": 1, "nsplit_y": 1}), (145, 18, 24, 5, {"pchunk": 5, "nsplit_y": 2})]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("bdt", ["bf16", "f64"])
@pytest.mark.parametrize("nbf,naux,npairs,ncwo,tuning", SHAPES)
def test_contractions(ctx, nbf, naux, npairs, ncwo, tuning, bdt, prec):
    if prec == "fp32" and bdt == "f64" and npairs in (32, 43):
        # B rounded to float32 (6e-8 of each element) is already 1.6e-6 of these 940 and 1270 Ha, and was with the
        # element-wise kernels before, to the last bit; the bar is absolute
        pytest.xfail("the energies are too large for the float32 bar")
    inst = synth.make(synth.Workload("edge", nbf, naux, npairs, ncwo, bdt), 23)
    n = pnof.on_sigmoid(inst.gamma, npairs, ncwo)
    B = t(inst.B) if bdt == "f64" else t(inst.B).to(torch.bfloat16)
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, P.FP64 if prec == "fp64" else P.FP32,
                     P.INTS_DF_F64 if bdt == "f64" else P.INTS_DF_BF16)
    ctx.set_tuning(**tuning)
    a = ctx.lagrangian(prob, t(inst.C), t(n), t(inst.H), B, jk=True)
    torch.cuda.synchronize()
    ctx.set_tuning(None)
    orc = stream.lagrangian(inst.C, n, inst.H, inst.B, npairs, ncwo, pnof.PNOF7)
    de, dl = (1e-8, 1e-10) if prec == "fp64" else (1e-6, 2e-5)
    assert abs(a["E"].item() - orc["E"]) < de
    assert np.max(np.abs(a["lam"].cpu().numpy() - orc["lam"])) < dl
