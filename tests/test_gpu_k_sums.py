"""K of the mixed precision where its partial sums are formed in more than one way: float32 sums that end inside a
split and are added to (splits of more rows than one such sum, several chunks), splits of one row, and the
automatic ones.  Bar: 2e-5, the mixed precision's own on lambda; K's entries here are of order 1 at most."""
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
def case():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    inst = synth.make(synth.Workload("ksums", 135, 45, 26, 4, "bf16"), 31)
    n = pnof.on_sigmoid(inst.gamma, 26, 4)
    return P.Context(0), inst, n, stream.lagrangian(inst.C, n, inst.H, inst.B, 26, 4, pnof.PNOF7)


@pytest.mark.parametrize("prec", ["split", "bf16"])
@pytest.mark.parametrize("pchunk,nsplit", [(0, 0), (0, 1), (0, 2), (0, 45), (20, 1), (20, 20), (8, 3), (17, 2)])
def test_k_sums(case, pchunk, nsplit, prec):
    ctx, inst, n, orc = case
    prob = P.problem(135, 45, 26, 4, P.PNOF7, P.BF16_SPLIT if prec == "split" else P.BF16, P.INTS_DF_BF16)
    ctx.set_tuning(pchunk=pchunk, nsplit_b=nsplit)
    B = t(inst.B).to(torch.bfloat16)
    a = ctx.lagrangian(prob, t(inst.C), t(n), t(inst.H), B, jk=True)
    K = a["K"].cpu().numpy()
    ctx.set_tuning(None)
    b = ctx.lagrangian(prob, t(inst.C), t(n), t(inst.H), B, jk=True)
    assert np.array_equal(K, K.T)
    assert np.max(np.abs(K - b["K"].cpu().numpy())) < 2e-6 * np.max(np.abs(K))   # 8 rows of float32 sums
    if prec == "split":
        assert np.max(np.abs(K - orc["K"])) < 2e-5
