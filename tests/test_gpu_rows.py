"""The mixed precision over rows of B of every alignment: X reads a copy of B with 16-byte aligned rows
(formed with the chunk's bounds, or with the split of a float64 B), and its tiles run over the stacked
rows of all P.  Sizes below, at and past the pieces and lane groups of the copy (8 elements; 64, 128,
256 and 512 elements of bf16) and the 128-row tile, the rows of one P ending inside a tile.  Bars: the
mixed precision's own against the float64 oracle (1e-6 Ha, 2e-5 on lambda); bit-identity between the
bound and the unbound call, whose bounds come from different kernels."""
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


# nbf, naux, npairs, ncwo, rows of B per chunk (0: automatic; 7: several chunks, the last one short)
SHAPES = [(5, 9, 2, 1, 0), (7, 40, 2, 1, 7), (8, 30, 3, 1, 0), (33, 66, 5, 2, 7), (65, 70, 8, 3, 0), (127, 60, 11, 4, 7),
          (129, 61, 20, 5, 0), (257, 40, 20, 3, 7), (515, 24, 30, 4, 7)]


@pytest.mark.parametrize("bdt", ["bf16", "f64"])
@pytest.mark.parametrize("nbf,naux,npairs,ncwo,pchunk", SHAPES)
def test_split_rows(ctx, nbf, naux, npairs, ncwo, pchunk, bdt):
    inst = synth.make(synth.Workload("rows", nbf, naux, npairs, ncwo, bdt), 21)
    n = pnof.on_sigmoid(inst.gamma, npairs, ncwo)
    B = t(inst.B) if bdt == "f64" else t(inst.B).to(torch.bfloat16)
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, P.BF16_SPLIT, P.INTS_DF_F64 if bdt == "f64" else P.INTS_DF_BF16)
    ctx.set_tuning(pchunk=pchunk)
    ctx.bind_integrals()
    a = ctx.lagrangian(prob, t(inst.C), t(n), t(inst.H), B, jk=True)
    ctx.bind_integrals(prob, B)
    b = ctx.lagrangian(prob, t(inst.C), t(n), t(inst.H), B, jk=True)
    torch.cuda.synchronize()
    ctx.bind_integrals()
    ctx.set_tuning(None)
    orc = stream.lagrangian(inst.C, n, inst.H, inst.B, npairs, ncwo, pnof.PNOF7)
    assert abs(a["E"].item() - orc["E"]) < 1e-6
    assert np.max(np.abs(a["lam"].cpu().numpy() - orc["lam"])) < 2e-5
    for k in a:
        assert torch.equal(a[k], b[k]), k
