"""Active spaces of more than one 128-wide tile in a batch, at every pair of tile widths of b and Y: W is stored
once per pair of b's tiles, and a tile of Y reads whole or half blocks of it.  Active orbitals at and past 64, 128
and 192 (a last block of one row, of one interleaved run of eight and of a part of one), rows of B of every
remainder modulo 8.  Bars: lambda 2e-5, the mixed precision's own; E 5e-7 of its size (two factors of 22 bits)."""
import numpy as np
import pytest
import torch

import synth
from oracle import pnof, stream

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
SIZES = [(66, 20, 13, 4), (129, 12, 43, 2), (140, 14, 17, 7), (195, 10, 39, 4), (71, 31, 16, 3), (12, 7, 1, 3)]   # nbf, naux, npairs, ncwo


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def case():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context(0)
    insts = [synth.make(synth.Workload("tiles", *s, "bf16"), 25 + i) for i, s in enumerate(SIZES)]
    ns = [pnof.on_sigmoid(i.gamma, i.wl.npairs, i.wl.ncwo) for i in insts]
    refs = [stream.lagrangian(i.C, n, i.H, i.B, i.wl.npairs, i.wl.ncwo, pnof.PNOF7) for i, n in zip(insts, ns)]
    return ctx, insts, ns, refs


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("btile", [64, 128])
@pytest.mark.parametrize("ytile", [64, 128])
def test_batch_tiles(case, btile, ytile, persistent):
    ctx, insts, ns, refs = case
    probs = [P.problem(i.wl.nbf, i.wl.naux, i.wl.npairs, i.wl.ncwo, P.PNOF7, P.BF16_SPLIT, P.INTS_DF_BF16) for i in insts]
    batch = P.Batch(ctx, probs)
    outs = batch.bind([{"C": t(i.C), "H": t(i.H), "n": t(n), "B": t(i.B).to(torch.bfloat16)} for i, n in zip(insts, ns)])
    batch.set_tiles(128, btile, ytile)
    batch.run(graph=False, persistent=persistent)
    torch.cuda.synchronize()
    for inst, o, r in zip(insts, outs, refs):
        assert abs(o["E"].item() - r["E"]) < 5e-7 * abs(r["E"]), (inst.wl.nbf, o["E"].item(), r["E"])
        assert np.max(np.abs(o["lam"].cpu().numpy() - r["lam"])) < 2e-5, inst.wl.nbf
    batch.close()
