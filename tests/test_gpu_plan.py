"""Launch plans: rows of B per chunk, workspaces that were lent at the size of an earlier layout (more partial sums,
no copy of B's rows, shorter float64 chunks), and problems that just fit the static array of
pnof_lagrangian_noalloc.  Bars between two plans of one problem, which differ in the order of sums: 1e-11 of the
largest element in float64; 2e-6 in the split and float32 modes (8 ulp of float32)."""
import ctypes
import math

import pytest
import torch

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return P.Context(0)


def _inputs(nbf, naux, npairs, ncwo, prec, b):
    g = torch.Generator(device=DEV).manual_seed(nbf)
    r = lambda *s: torch.randn(*s, generator=g, device=DEV, dtype=torch.float64)
    B = r(naux, nbf, nbf) / math.sqrt(naux * nbf)
    B = (B + B.transpose(1, 2)).contiguous()
    H = r(nbf, nbf)
    C = torch.linalg.qr(r(nbf, nbf).cpu())[0].to(DEV).contiguous()
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, prec, P.INTS_DF_F64 if b == "f64" else P.INTS_DF_BF16)
    n = torch.rand(prob.nact, generator=g, device=DEV, dtype=torch.float64)
    return prob, C, n, (H + H.T).contiguous(), B if b == "f64" else B.to(torch.bfloat16)


def _same(a, b, prec):
    bar = 1e-11 if prec == P.FP64 else 2e-6
    for k in ("E", "lam", "dEdC", "J", "K"):
        assert torch.max(torch.abs(a[k] - b[k])) <= bar * torch.max(torch.abs(b[k])), k


@pytest.mark.parametrize("nbf,naux,npairs,ncwo,pchunk", [(64, 12000, 8, 3, 4000), (10, 20000, 3, 2, 4000), (64, 300, 8, 3, 300),
                                                         (500, 2000, 50, 5, 500)])
def test_float64_chunk_fills_the_chip(ctx, nbf, naux, npairs, ncwo, pchunk):
    """Blocks of 64 active orbitals and 64 functions: 4096 of them, or 512 rows, in chunks of equal length."""
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, P.FP64, P.INTS_DF_F64)
    assert ctx.plan(prob)["pchunk"] == pchunk


LENT = [(300, 1200, 50, 5, P.FP64, "f64", 340554368), (300, 1200, 50, 5, P.FP64, "bf16", 458634368),
        (70, 5000, 9, 3, P.FP32, "bf16", 65120768), (213, 900, 25, 4, P.BF16_SPLIT, "bf16", 408425984),
        (300, 1200, 50, 5, P.BF16_SPLIT, "bf16", 713820160), (213, 900, 25, 4, P.BF16, "bf16", 275598592)]


@pytest.mark.parametrize("nbf,naux,npairs,ncwo,prec,b,lent", LENT)
def test_workspace_lent_at_an_earlier_size(nbf, naux, npairs, ncwo, prec, b, lent):
    prob, C, n, H, B = _inputs(nbf, naux, npairs, ncwo, prec, b)
    ref = P.Context(0).lagrangian(prob, C, n, H, B, jk=True)
    ctx = P.Context(0)
    ws = torch.empty(lent + 256, dtype=torch.uint8, device=DEV)
    base = (ws.data_ptr() + 255) // 256 * 256
    assert P.lib().pnof_set_workspace(ctx.handle, ctypes.c_void_p(base), lent) == 0
    small = _inputs(24, 96, 3, 3, prec, b)
    ctx.lagrangian(*small)   # streams and handles of the context
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    out = ctx.lagrangian(prob, C, n, H, B, jk=True)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 32 << 20
    _same(out, ref, prec)


EDGE = [(1655, 151, 3, P.FP64, "f64"), (1784, 172, 3, P.FP32, "bf16"), (2128, 137, 3, P.BF16_SPLIT, "bf16"),
        (2195, 102, 3, P.BF16_SPLIT, "f64"), (2129, 158, 3, P.BF16, "bf16")]


@pytest.mark.parametrize("nbf,npairs,ncwo,prec,b", EDGE)
def test_noalloc_at_the_edge_of_the_static_array(ctx, nbf, npairs, ncwo, prec, b):
    """One row of B per chunk, and no room for padding beta within 64 MiB beside two buffers of XT."""
    prob, C, n, H, B = _inputs(nbf, 4, npairs, ncwo, prec, b)
    ref = ctx.lagrangian(prob, C, n, H, B, jk=True)
    out = {k: torch.empty_like(v) for k, v in ref.items()}
    p = lambda k: ctypes.c_void_p(out[k].data_ptr())
    q = lambda t: ctypes.c_void_p(t.data_ptr())
    st = P.lib().pnof_lagrangian_noalloc(ctx.handle, ctypes.byref(prob), q(C), q(n), q(H), q(B), p("lam"), p("E"), p("dEdC"),
                                         p("dEdn"), p("max_asym"), p("J"), p("K"))
    assert st == 0, P.lib().pnof_last_error(ctx.handle)
    torch.cuda.synchronize()
    _same(out, ref, prec)
