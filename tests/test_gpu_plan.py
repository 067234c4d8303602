"""Launch plans: rows of B per chunk."""
import pytest
import torch

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0)


@pytest.mark.parametrize("nbf,naux,npairs,ncwo,pchunk", [(64, 12000, 8, 3, 4000), (10, 20000, 3, 2, 4000), (64, 300, 8, 3, 300),
                                                         (500, 2000, 50, 5, 500)])
def test_float64_chunk_fills_the_chip(ctx, nbf, naux, npairs, ncwo, pchunk):
    """Blocks of 64 active orbitals and 64 functions: 4096 of them, or 512 rows, in chunks of equal length."""
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, P.FP64, P.INTS_DF_F64)
    assert ctx.plan(prob)["pchunk"] == pchunk
