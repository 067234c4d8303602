"""The orbital step's reduction to tridiagonal form at the edges of its forms (one workgroup to 128, the
workgroups of one die to 1024, a launch per column before that), its leaves and blocks of reflectors, and
beside other work on the device: with few of its workgroups running at once it declines and the step
takes a launch per column instead, with the same bars.  Bars: eigenvalues and residual 1e-9, vectors
orthonormal to 1e-12, as for every size of the orbital step."""
import threading

import numpy as np
import pytest
import torch

from oracle import pnof

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _case(nbf, seed=0):
    rng = np.random.default_rng([nbf, seed])
    lam = rng.standard_normal((nbf, nbf))
    C, _ = np.linalg.qr(rng.standard_normal((nbf, nbf)))
    return lam, C


def _check(lam, C, Cn, eps):
    _, eps_r, S = pnof.orbital_step(lam, C)
    U = C.T @ Cn.cpu().numpy()
    e = eps.cpu().numpy()
    assert np.max(np.abs(e - eps_r)) < 1e-9
    assert np.max(np.abs(U.T @ U - np.eye(len(e)))) < 1e-12
    assert np.max(np.abs(S @ U - U * e[None, :])) < 1e-9


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0)


@pytest.mark.parametrize("nbf", [3, 4, 16, 17, 31, 32, 34, 63, 65, 113, 127, 145, 255, 256, 257, 511, 512, 513, 767, 768, 769,
                                 1023, 1024, 1026])
def test_reduction_sizes(ctx, nbf):
    lam, C = _case(nbf)
    Cn, eps = ctx.orbital_step(t(lam), t(C))
    _check(lam, C, Cn, eps)


def test_reduction_repeats_bit_for_bit(ctx):
    lam, C = _case(333)
    a = ctx.orbital_step(t(lam), t(C))
    for _ in range(3):
        b = ctx.orbital_step(t(lam), t(C))
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_reduction_beside_other_work(ctx):
    """Two threads with a context and stream each, and products on a third stream meanwhile."""
    cases = [_case(n, 1) for n in (140, 300, 300, 520)]
    dev = [(t(l), t(c)) for l, c in cases]
    got, errors = {}, []
    torch.cuda.synchronize()

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                c = P.Context(0)
                for i, (l, o) in enumerate(dev):
                    got[k, i] = c.orbital_step(l, o)
                s.synchronize()
                c.close()
        except Exception as e:   # reported by the main thread
            errors.append(e)

    side = torch.cuda.Stream()
    a = torch.randn(4096, 4096, device=DEV)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    with torch.cuda.stream(side):
        for _ in range(40):
            a = (a @ a) * 1e-4
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for (k, i), (Cn, eps) in got.items():
        _check(*cases[i], Cn, eps)
