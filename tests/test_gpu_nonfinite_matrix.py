"""An orbital step whose matrix is not finite ends with PNOF_E_EIG, in every form of the reduction and with the zeta
scaling, and the context goes on working; a matrix of subnormal numbers is solved."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("nbf", [8, 17, 40, 300, 1030])
def test_not_finite(ctx, nbf, bad):
    rng = np.random.default_rng(nbf)
    lam, C = rng.standard_normal((nbf, nbf)), np.eye(nbf)
    diag = np.sort(rng.standard_normal(nbf))
    good = ctx.orbital_step(t(lam), t(C), t(diag), 0.5)
    broken, bdiag = lam.copy(), diag.copy()
    broken[nbf // 2, nbf // 3] = bad
    bdiag[nbf // 2] = bad
    for args in ((t(broken), t(C)), (t(broken), t(C), t(diag), 0.5), (t(lam), t(C), t(bdiag), 0.5)):
        with pytest.raises(P.PnofError) as e:
            ctx.orbital_step(*args)
        assert e.value.status == 8
    again = ctx.orbital_step(t(lam), t(C), t(diag), 0.5)
    assert torch.equal(good[0], again[0]) and torch.equal(good[1], again[1])


def test_subnormal(ctx):
    nbf = 40
    lam = np.random.default_rng(1).standard_normal((nbf, nbf)) * 1e-310
    Cn, eps = ctx.orbital_step(t(lam), t(np.eye(nbf)))
    U = Cn.cpu().numpy()
    assert np.max(np.abs(U.T @ U - np.eye(nbf))) < 1e-12
    assert np.max(np.abs(eps.cpu().numpy())) < 1e-308
