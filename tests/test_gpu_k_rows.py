"""How many rows of P one float32 sum of b^2 covers in the mixed precision (the sums of those are float64), where
B_P = a_P 1 and C = 1 make every b exactly a_P: a_P = 2^-13 disappears beside a_P = 1 within a sum, so that K tells
the rows per sum.  The bound is the even share of a chunk's rows among 1024 blocks, or among the splits that were set, and 8 (500 functions: chunks of 342 rows, 6 tiles).  Exact apart from that:
all factors are powers of two."""
import pytest
import torch

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


# nbf, naux, npairs, ncwo, tuning, rows per sum at most
SHAPES = [(200, 800, 20, 4, {}, 1), (300, 1200, 24, 4, {}, 1), (500, 1000, 50, 5, {}, 2), (200, 800, 20, 4, {"nsplit_b": 3}, 8),
          (500, 1000, 50, 5, {"pchunk": 1000}, 5), (520, 1600, 60, 7, {"pchunk": 1600, "nsplit_b": 2}, 8)]


@pytest.mark.parametrize("nbf,naux,npairs,ncwo,tuning,rows", SHAPES)
def test_rows_per_float32_sum(nbf, naux, npairs, ncwo, tuning, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context(0)
    ctx.set_tuning(**tuning)
    every = rows + 3   # a large row among `every`: a sum of r rows loses at most r - 1 small ones beside it
    big = torch.arange(naux, device=DEV) % every == 0
    a = torch.where(big, 1.0, 2.0 ** -13).to(torch.bfloat16)
    eye = torch.eye(nbf, device=DEV, dtype=torch.bfloat16)
    B = (a[:, None, None] * eye[None]).contiguous()
    C = torch.eye(nbf, device=DEV, dtype=torch.float64)
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, P.BF16_SPLIT, P.INTS_DF_BF16)
    J, K = ctx.jk(prob, C, B)
    torch.cuda.synchronize()
    nbig = int(big.sum())
    exact = nbig + (naux - nbig) * 2.0 ** -26
    lost = (exact - torch.diagonal(K)) * 2.0 ** 26
    assert 0 <= lost.min().item() and lost.max().item() <= (rows - 1) * nbig
    assert torch.count_nonzero(K - torch.diag(torch.diagonal(K))).item() == 0
