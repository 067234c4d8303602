"""X from a float64 B on either side of the choice between its tiles of 64 and 128 stacked rows (132 active orbitals,
520 functions: 41 and 42 rows of B per launch are 501 and 513 of the wider ones), float64 and float32.  An element's
sum runs in the same order in both, so that D and J = D^T D agree bit for bit; J against torch in float64 to 1e-12
(float64) and 1e-6 (float32) of its largest element."""
import pytest
import torch

P = pytest.importorskip("paper_2004_06142_amd")
pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("prec,bar", [(P.FP64, 1e-12), (P.FP32, 1e-6)])
def test_x_tiles(prec, bar):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = P.Context(0)
    nbf, naux, npairs, ncwo = 520, 84, 33, 3
    g = torch.Generator(device=DEV).manual_seed(3)
    r = lambda *s: torch.randn(*s, generator=g, device=DEV, dtype=torch.float64)
    B = r(naux, nbf, nbf) / nbf
    B = (B + B.transpose(1, 2)).contiguous()
    C = torch.linalg.qr(r(nbf, nbf).cpu())[0].to(DEV).contiguous()
    prob = P.problem(nbf, naux, npairs, ncwo, P.PNOF7, prec, P.INTS_DF_F64)
    J = []
    for pchunk in (41, 42, 84, 7):
        ctx.set_tuning(pchunk=pchunk)
        J.append(ctx.jk(prob, C, B)[0])
    ctx.set_tuning(None)
    CA = C[:, :prob.nact].contiguous()
    D = torch.stack([(CA * (B[p] @ CA)).sum(0) for p in range(naux)])
    ref = D.T @ D
    for x in J:
        assert torch.equal(x, J[0])
    assert torch.max(torch.abs(J[0] - ref)) <= bar * torch.max(torch.abs(ref))
