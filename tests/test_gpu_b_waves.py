"""The two wave grids of b's 128 tile, on either side of the number of blocks where the choice changes (256).  An
element's sum runs in the same order in both: a problem's results in a batch do not depend, to the last bit, on how
many others are beside it (13 blocks against 312); D and J = D^T D of a single problem do not on the splits."""
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


@pytest.mark.parametrize("prec", [P.BF16_SPLIT, P.BF16])
@pytest.mark.parametrize("npairs,ncwo", [(4, 3), (8, 7), (13, 3)])
def test_batch_of_one_and_of_many(ctx, npairs, ncwo, prec):
    nbf, naux = 64, 400
    inst = synth.make(synth.Workload("waves", nbf, naux, npairs, ncwo, "bf16"), 11)
    x = {"C": t(inst.C), "H": t(inst.H), "n": t(pnof.on_sigmoid(inst.gamma, npairs, ncwo)), "B": t(inst.B).to(torch.bfloat16)}
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, prec, P.INTS_DF_BF16)
    got = []
    for ninst in (1, 24):
        b = P.Batch(ctx, [prob] * ninst)
        b.set_tiles(0, 128, 0)
        b.bind([x] * ninst)
        outs = b.run(graph=False)
        torch.cuda.synchronize()
        got += [{k: v.clone() for k, v in o.items()} for o in outs]
        b.close()
    for o in got[1:]:
        for k in o:
            assert torch.equal(o[k], got[0][k]), k


@pytest.mark.parametrize("prec", [P.BF16_SPLIT, P.BF16])
@pytest.mark.parametrize("nbf,npairs,ncwo", [(61, 10, 3), (150, 30, 3)])
def test_single(ctx, nbf, npairs, ncwo, prec):
    inst = synth.make(synth.Workload("waves", nbf, 300, npairs, ncwo, "bf16"), 12)
    prob = P.problem(nbf, 300, npairs, ncwo, P.PNOF7, prec, P.INTS_DF_BF16)
    C, B = t(inst.C), t(inst.B).to(torch.bfloat16)
    J, K = [], []
    for nsplit in (1, 256, 257, 300):
        ctx.set_tuning(nsplit_b=nsplit)
        j, k = ctx.jk(prob, C, B)
        J.append(j)
        K.append(k)
    ctx.set_tuning(None)
    for j, k in zip(J, K):
        assert torch.equal(j, J[0])
        assert torch.max(torch.abs(k - K[0])) < 2e-6 * torch.max(K[0])   # float32 sums of 8 rows and of one
