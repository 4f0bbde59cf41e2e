"""The row kernels (AO values times C) where their paths divide: shells of one,
two, three and five primitives in one basis (the first three primitives come
from the shells' records, the rest from the tables), and the two kernels of
the sweep's FP32 rows, chosen by the number of rows, which give the same bits.
"""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2511_05222_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_05222_amd import vmc
    vmc.lib()
    return torch.device("cuda:0")


def contractions(nprims):
    """The 9-atom molecule with nprims[s % len] primitives in shell s."""
    m = inputs.make_config(1).molecule
    rng = np.random.default_rng(31)
    n = np.array([nprims[s % len(nprims)] for s in range(m.basis.n_shells)], np.int32)
    exps = np.concatenate([np.sort(np.exp(rng.uniform(np.log(0.1), np.log(50.0), k)))[::-1] for k in n])
    basis = inputs.Basis(m.basis.shell_atom, m.basis.shell_l, n, exps, rng.uniform(0.2, 1.0, n.sum()))
    C = inputs.s_orthonormal_coefficients(inputs.overlap_matrix(m.xyz, basis), 33)
    return dataclasses.replace(m, basis=basis, C_full=C)


@pytest.mark.parametrize("nprims", [(1,), (2,), (5,), (1, 2, 3, 5)])
def test_contraction_lengths(dev, nprims):
    """FP64 measurement against the oracle (the parity suite's bound), mixed
    within FP32 round-off of it: the derivative bound of the mixed suite."""
    from oracle import derivatives as dv, wavefunction as wf
    from paper_2511_05222_amd import vmc
    m = contractions(nprims)
    r = inputs.initial_walkers(m, 5, 3)
    ref = dv.measure(wf.System(m), m.xyz, r)
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-3)):
        ctx = vmc.Context(m, max_walkers=5, precision=prec, promote_fraction=0.0)
        out = ctx.measure(torch.tensor(r, device=dev))
        for a, b in (("EL", "E_L"), ("dEL_dR", "H"), ("O", "O"), ("G", "G")):
            err = np.abs(out[a].cpu().numpy() - ref[b]).max() / np.abs(ref[b]).max()
            assert err <= tol, (prec, a, err)


@pytest.mark.parametrize("extra", [0, 1, 77])
def test_many_rows(dev, extra):
    """2^20 rows and more (the wavefront-per-64-rows kernel, ragged ends)
    against the first walkers alone (the block kernel): identical chains."""
    from paper_2511_05222_amd import vmc
    m = inputs.make_config(1).molecule
    W, few = -(-(1 << 20) // m.n_elec) + extra, 501
    w0 = torch.tensor(inputs.initial_walkers(m, 1, 9), device=dev).expand(W, -1, -1)
    g = torch.Generator(device=dev)
    g.manual_seed(4)
    w = (w0 + 0.1 * torch.randn(w0.shape, dtype=torch.float64, device=dev, generator=g)).contiguous()
    part = w[:few].clone()
    vmc.Context(m, max_walkers=W, precision="mixed").sweep(w, 2, 5, measure=False)
    vmc.Context(m, max_walkers=W, precision="mixed").sweep(part, 2, 5, measure=False)
    assert torch.equal(w[:few], part)


@pytest.mark.parametrize("n", [17, 32, 33, 48, 49, 64])
def test_many_rows_orbital_classes(dev, n):
    """The same at the edges of the other classes of 16 orbitals (each its own
    instance of both kernels): just over 2^20 rows, identical chains."""
    from paper_2511_05222_amd import vmc
    m = dataclasses.replace(inputs.family_member(6).molecule, n_up=n, n_dn=n)
    N, few = 2 * n, 501
    W = -(-(1 << 20) // N) + 1
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    at = torch.tensor(m.xyz[np.arange(N) % m.n_atoms], device=dev)
    w = (at + 0.5 * torch.randn((W, N, 3), dtype=torch.float64, device=dev, generator=g)).contiguous()
    assert few * N < (1 << 20) <= W * N
    start, part = w[:few].clone(), w[:few].clone()
    ctx = vmc.Context(m, max_walkers=W, precision="mixed")
    ctx.sweep(w, 1, 5, measure=False)
    ctx.sweep(part, 1, 5, measure=False)
    assert not torch.equal(part, start)
    assert torch.equal(w[:few], part)
