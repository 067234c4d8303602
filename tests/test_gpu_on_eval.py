"""One evaluation of the occupation optimisation, E(n(gamma)) and dE/dgamma: rows shared between few and many blocks,
singly occupied orbitals, both maps, more variables than are read from host memory (256), and more than a block's LDS
holds.  After one iteration without history the step is along -dE/dgamma, and E is the energy at the returned gamma.
Bars: E 1e-11 of the sum of its terms' sizes (float64 sums of up to 1.5e7 terms), the direction 1e-9."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("npairs,ncwo,nsingle,trig", [(1, 1, 0, False), (2, 2, 1, False), (3, 4, 2, True), (13, 4, 0, False), (52, 4, 0, True),
                                                      (64, 3, 0, False), (65, 4, 3, True), (90, 2, 1, False), (1300, 2, 0, False)])
def test_evaluation(ctx, npairs, ncwo, nsingle, trig):
    rng = np.random.default_rng(npairs + ncwo)
    nact = npairs * (1 + ncwo) + nsingle
    hpp = rng.standard_normal(nact)
    J, K = rng.standard_normal((2, nact, nact)) * 0.1
    J, K = J + J.T, K + K.T
    ngam = npairs * ncwo if trig else nact
    gam = rng.uniform(0.3, 1.2, ngam) if trig else rng.standard_normal(ngam)
    prob = P.problem(nact, 1, npairs, ncwo, P.PNOF7, P.FP64, P.INTS_DF_F64, nsingle=nsingle)
    g, E, _ = ctx.optimize_on(prob, torch.eye(nact, dtype=torch.float64, device=DEV), torch.diag(t(hpp)), t(J), t(K), t(gam),
                              kind=P.ON_TRIG if trig else P.ON_SIGMOID, maxiter=1)
    g = g.cpu().numpy()
    on = (lambda x: pnof.on_trig(x, npairs, ncwo, nsingle)) if trig else (lambda x: pnof.on_sigmoid(x, npairs, ncwo, nsingle))
    n0, n1 = on(gam), on(g)
    scale = np.abs(hpp).sum() * 2 + (np.abs(J) * 2 + np.abs(K)).sum()
    assert abs(E - pnof.energy_from_jk(n1, hpp, J, K, npairs, ncwo, pnof.PNOF7, nsingle)) < 1e-11 * scale
    dn = pnof.grad_n(n0, hpp, J, K, npairs, ncwo, pnof.PNOF7, nsingle)
    jac = (pnof.on_trig_jac if trig else pnof.on_sigmoid_jac)(gam, npairs, ncwo, nsingle)
    ref = -(jac.T @ dn)
    step = g - gam
    assert np.linalg.norm(step) > 0
    assert np.max(np.abs(step / np.linalg.norm(step) - ref / np.linalg.norm(ref))) < 1e-9
