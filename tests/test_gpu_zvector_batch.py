"""Batches of Z-vector solves at the edges of the product's tiles (64 rows, 32
columns, 16 right-hand sides): the residual against the stopping rule, and a
right-hand side's solution the same in every batch it is in."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

RTOL = 1e-12


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_05222_amd import vmc
    vmc.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("d", [1, 2, 31, 32, 33, 63, 64, 65, 95, 97, 129, 1025])
@pytest.mark.parametrize("n", [2, 15, 16, 17, 33, 49, 64, 65])
def test_batch(dev, d, n):
    from paper_2511_05222_amd import vmc
    g = torch.Generator()
    g.manual_seed(97 * d + n)
    G = torch.randn((d, 64), dtype=torch.float64, generator=g)
    H = torch.mm(G, G.t()) / 64.0
    H = 0.5 * (H + H.t()) + torch.diag(0.5 * 10.0 ** torch.rand(d, dtype=torch.float64, generator=g))
    b = torch.randn((n, d), dtype=torch.float64, generator=g)
    tH, tb = H.contiguous().to(dev), b.to(dev)
    z, its = vmc.zvector_solve(tH, tb, rtol=RTOL, maxit=4000, jacobi=True)
    # (the recurrence's residual meets the rule; the true one differs by the
    # rounding of |H| |z|, eps d |H| |z| at most)
    r = (z.cpu() @ H + b).norm(dim=1)
    slack = 2.3e-16 * d * H.norm() * z.cpu().norm(dim=1)
    assert bool((r <= 1.01 * RTOL * b.norm(dim=1) + slack).all())
    k = max(2, n // 3)
    part, pits = vmc.zvector_solve(tH, tb[:k].contiguous(), rtol=RTOL, maxit=4000, jacobi=True)
    assert torch.equal(part, z[:k]) and pits == its[:k]
