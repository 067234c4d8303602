"""The forms of a plan: every one that a lent workspace of some size leads to (rows of B copied or read as they are, one
or two buffers of XT) gives the results of the full plan bit for bit, the chunks and splits being set alike.  X of rows
that are not 16-byte aligned (nbf not a multiple of 8 without the copy, or B itself at an odd address) runs its
register-staged form, whose sums run in the order of the direct one."""
import ctypes

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


def _inputs(nbf, naux, npairs, ncwo, prec, b):
    inst = synth.make(synth.Workload("forms", nbf, naux, npairs, ncwo, b), 17)
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, prec, P.INTS_DF_F64 if b == "f64" else P.INTS_DF_BF16)
    B = t(inst.B) if b == "f64" else t(inst.B).to(torch.bfloat16)
    return prob, t(inst.C), t(pnof.on_sigmoid(inst.gamma, npairs, ncwo)), t(inst.H), B


def _all(ctx, prob, C, n, H, B):
    out = ctx.lagrangian(prob, C, n, H, B, jk=True)
    out["Y"], out["Fq"] = ctx.fock(prob, C, n, H, B, [0, prob.nact - 1])
    _, _, out["Jq"], out["Kq"] = ctx.jk(prob, C, B, [1, 0])
    torch.cuda.synchronize()
    return out


CASES = [(P.BF16_SPLIT, "bf16"), (P.BF16_SPLIT, "f64"), (P.BF16, "bf16"), (P.FP32, "bf16"), (P.FP64, "f64")]


@pytest.mark.parametrize("prec,b", CASES)
@pytest.mark.parametrize("nbf,naux,npairs,ncwo,pchunk", [(77, 51, 7, 3, 8), (130, 40, 20, 4, 40), (5, 30, 2, 1, 7)])
def test_lent_workspaces_of_any_size(nbf, naux, npairs, ncwo, pchunk, prec, b):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    args = _inputs(nbf, naux, npairs, ncwo, prec, b)
    ctx = P.Context(0)
    ctx.set_tuning(pchunk=pchunk, nsplit_b=3, nsplit_y=2)
    full = ctx.reserve(args[0])
    ref = _all(ctx, *args)
    base = (ctx._ws.data_ptr() + 255) // 256 * 256
    for lent in (full - 256, full * 31 // 32, full * 15 // 16, full * 7 // 8, full * 3 // 4, full * 5 // 8, full // 4):
        assert P.lib().pnof_set_workspace(ctx.handle, ctypes.c_void_p(base), lent) == 0
        got = _all(ctx, *args)
        for k in ref:
            assert torch.equal(got[k], ref[k]), (k, lent, full)


@pytest.mark.parametrize("prec", [P.BF16_SPLIT, P.BF16, P.FP32, P.FP64])
@pytest.mark.parametrize("nbf,naux,npairs,ncwo", [(8, 30, 3, 1), (64, 21, 8, 3), (136, 18, 20, 5), (200, 30, 33, 3)])
def test_integrals_at_odd_addresses(nbf, naux, npairs, ncwo, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context(0)
    prob, C, n, H, B = _inputs(nbf, naux, npairs, ncwo, prec, "bf16")
    ref = _all(ctx, prob, C, n, H, B)
    for off in (1, 2, 4):
        flat = torch.empty(B.numel() + 8, dtype=B.dtype, device=DEV)
        odd = flat[off:off + B.numel()].reshape(B.shape)
        odd.copy_(B)
        for bind in (False, True):
            ctx.bind_integrals(*((prob, odd) if bind else ()))
            got = _all(ctx, prob, C, n, H, odd)
            ctx.bind_integrals()
            for k in ref:
                assert torch.equal(got[k], ref[k]), (k, off, bind)
