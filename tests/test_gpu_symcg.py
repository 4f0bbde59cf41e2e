"""zvector_solve where it reads the lower triangle of H only (large symmetric H,
up to 32 right-hand sides): sizes around the tile and block edges and the
thresholds, against a direct FP64 solve and the stopping rule; an H that is not
symmetric to the last bit, or holds a NaN above the diagonal alone, is solved
or refused as by reading all of it."""
import numpy as np
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


def problem(dev, d, n, seed):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    G = torch.randn((d, 64), dtype=torch.float64, device=dev, generator=g)
    H = torch.mm(G, G.t().contiguous()) / 64.0
    H = 0.5 * (H + H.t())
    u = torch.rand(d, dtype=torch.float64, device=dev, generator=g)
    H += torch.diag(0.5 * 10.0 ** u)
    return H.contiguous(), torch.randn((n, d), dtype=torch.float64, device=dev, generator=g)


def check(H, b, z, rtol=RTOL):
    # (the CG residual is the recurrence's: the true one agrees to its rounding)
    r = torch.mm(z, H) + b
    assert (r.norm(dim=1) <= 1.01 * rtol * b.norm(dim=1)).all()
    ref = torch.linalg.solve(H, -b.t().contiguous()).t()
    assert ((z - ref).norm(dim=1) <= 1e-10 * ref.norm(dim=1)).all()


@pytest.mark.parametrize("d,n", [(3999, 1), (4000, 1), (4001, 1), (4097, 1), (4416, 1), (2400, 2), (2433, 2), (4159, 2),
                                 (2399, 5), (2400, 5), (2431, 3), (2497, 16), (2560, 17), (2623, 32), (2500, 33),
                                 (5601, 20), (8192, 4), (8257, 13)])
@pytest.mark.parametrize("jacobi", [False, True])
def test_solve(dev, d, n, jacobi):
    from paper_2511_05222_amd import vmc
    H, b = problem(dev, d, n, d + n)
    z, its = vmc.zvector_solve(H, b if n > 1 else b[0].contiguous(), rtol=RTOL, maxit=2000, jacobi=jacobi)
    check(H, b, z.view(n, d))
    # one at a time, in the library's own scratch: the single solve's bits
    x = torch.full_like(b[0], float("nan"))
    one = vmc.zvector_solve_noalloc(H, b[n - 1].contiguous(), x, rtol=RTOL, maxit=2000, jacobi=jacobi)
    zs, it1 = vmc.zvector_solve(H, b[n - 1].contiguous(), rtol=RTOL, maxit=2000, jacobi=jacobi)
    assert one == it1 and torch.equal(x, zs)


@pytest.mark.parametrize("n", [1, 2, 6])
def test_ends(dev, n):
    """A zero right-hand side among others, maxit, repeatability."""
    from paper_2511_05222_amd import vmc
    H, b = problem(dev, 4100, n, 3)
    solve = lambda x, **k: vmc.zvector_solve(H, x if n > 1 else x[0].contiguous(), jacobi=True, **k)
    z, its = solve(b)
    again, _ = solve(b)
    assert torch.equal(z, again)
    zero = b.clone()
    zero[0] = 0.0
    z0, it0 = solve(zero)
    assert (it0 if n == 1 else it0[0]) == 0 and float(z0.view(n, -1)[0].abs().max()) == 0.0
    if n > 1:
        assert torch.equal(z0[1:], z[1:]) and it0[1:] == its[1:]
    with pytest.raises(vmc.VmcError) as ei:
        solve(b, maxit=3)
    assert ei.value.code == vmc.VMC_ENOTCONV


@pytest.mark.parametrize("n", [1, 2, 6])
def test_not_symmetric(dev, n):
    from paper_2511_05222_amd import vmc
    H, b = problem(dev, 4100, n, 4)
    solve = lambda A: vmc.zvector_solve(A, b if n > 1 else b[0].contiguous(), jacobi=True)
    # (what reading all of H gives: rows of H, so that the residual is H z + b)
    A = H.clone()
    A[7, 4000] *= 1.0 + 2.0 ** -50
    z, _ = solve(A)
    r = torch.mm(A, z.view(n, -1).t().contiguous()).t() + b
    assert (r.norm(dim=1) <= 1.01 * RTOL * b.norm(dim=1)).all()
    A = H.clone()
    A[5, 4099] = float("nan")
    with pytest.raises(vmc.VmcError) as ei:
        solve(A)
    assert ei.value.code == vmc.VMC_ENONFINITE
