"""Per-orbital AO matrices at the edges of their kernels.  Explicit integrals without any symmetry at sizes below, at
and past the 32-function form, the 128-pair tile and the largest size; density-fitted ones for odd and even sizes
around the 64-wide tile and the 128-element run, more requested orbitals than one pass takes, repeated and unordered
ones, several chunks, every storage of the half-transformed integrals.  Bars relative to the largest element:
1e-12 sqrt(terms)-like growth of float64 sums bounded by 1e-11; the split and float32 modes 2e-5, bf16 products
2e-2 (their operands' roundings, 2^-17 and 2^-8, through three factors)."""
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


def close(a, b, tol):
    a = a.cpu().numpy() if torch.is_tensor(a) else a
    return np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0)


@pytest.mark.parametrize("nbf,npairs,ncwo", [(2, 1, 1), (5, 1, 2), (11, 1, 10), (24, 6, 3), (31, 5, 2), (32, 16, 1), (33, 3, 3),
                                             (45, 9, 4), (64, 16, 3)])
def test_explicit_integrals(ctx, nbf, npairs, ncwo):
    rng = np.random.default_rng(nbf)
    ERI, C, H = rng.standard_normal((nbf,) * 4), rng.standard_normal((nbf, nbf)), rng.standard_normal((nbf, nbf))
    H = H + H.T
    nact = npairs * (1 + ncwo)
    n = pnof.on_sigmoid(rng.standard_normal(nact) * 0.1, npairs, ncwo)
    prob = P.problem(nbf, 0, npairs, ncwo, P.PNOF7, P.FP64, P.INTS_ERI4_F64)
    q = [nact - 1, 0]
    J, K, Jq, Kq = ctx.jk(prob, t(C), t(ERI), q_idx=q)
    Y, _ = ctx.fock(prob, t(C), t(n), t(H), t(ERI), q_idx=q)
    torch.cuda.synchronize()
    a, b = pnof.coefficients(n, npairs, ncwo, pnof.PNOF7)[:2]
    Jr, Kr = np.empty((nact, nbf, nbf)), np.empty((nact, nbf, nbf))
    for r in range(nact):
        T = ERI @ C[:, r]                        # (ma|b.)
        Jr[r], Kr[r] = T @ C[:, r], np.einsum("mln,l->mn", T, C[:, r])
    CA = C[:, :nact]
    for i, k in enumerate(q):
        assert close(Jq[i], Jr[k], 1e-11) and close(Kq[i], Kr[k], 1e-11)
    assert close(J, np.einsum("mp,qmn,np->pq", CA, Jr, CA, optimize=True), 1e-11)
    assert close(K, np.einsum("mp,qmn,np->pq", CA, Kr, CA, optimize=True), 1e-11)
    Yr = n[:nact] * (H @ CA) + np.einsum("qr,rmn,nq->mq", a, Jr, CA, optimize=True) + np.einsum("qr,rmn,nq->mq", b, Kr, CA, optimize=True)
    assert close(Y, Yr, 1e-11)


TOL = {"FP64": 1e-11, "FP32": 2e-5, "BF16_SPLIT": 2e-5, "BF16": 2e-2}


@pytest.mark.parametrize("prec", list(TOL))
@pytest.mark.parametrize("bdt", ["bf16", "f64"])
@pytest.mark.parametrize("nbf,naux,npairs,ncwo,pchunk,q", [
    (3, 4, 1, 1, 0, [1, 0, 1]), (11, 131, 2, 2, 0, [5]), (16, 9, 3, 1, 4, list(range(6))), (63, 30, 4, 2, 7, list(range(9))),
    (64, 20, 4, 3, 0, [15, 3]), (65, 140, 3, 2, 129, list(range(8))), (129, 25, 5, 2, 0, [14, 0, 7])])
def test_density_fitted(ctx, nbf, naux, npairs, ncwo, pchunk, q, bdt, prec):
    inst = synth.make(synth.Workload("ao", nbf, naux, npairs, ncwo, bdt), 17)
    n = pnof.on_sigmoid(inst.gamma, npairs, ncwo)
    B = t(inst.B) if bdt == "f64" else t(inst.B).to(torch.bfloat16)
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, getattr(P, prec), P.INTS_DF_F64 if bdt == "f64" else P.INTS_DF_BF16)
    ctx.set_tuning(pchunk=pchunk)
    _, _, Jq, Kq = ctx.jk(prob, t(inst.C), B, q_idx=q)
    _, Fq = ctx.fock(prob, t(inst.C), t(n), t(inst.H), B, q_idx=q)
    torch.cuda.synchronize()
    ctx.set_tuning(None)
    F = pnof.fock_ao(inst.C, n, inst.H, inst.B, npairs, ncwo, pnof.PNOF7)
    for i, k in enumerate(q):
        Jr, Kr = pnof.jk_ao_df(inst.B, inst.C, k)
        assert close(Jq[i], Jr, TOL[prec]) and close(Kq[i], Kr, TOL[prec]) and close(Fq[i], F[k], TOL[prec]), (i, k)
