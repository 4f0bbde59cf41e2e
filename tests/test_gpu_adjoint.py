"""The adjoint kernel where its paths divide: orbitals at the edges of its
column tiles and electrons at those of its row tiles, with and (FP64, 114
electrons and more) without radial sums shared by a sub-tile's AOs, and
sub-tiles of 4 to 16 shells (7 are handled at a time)."""
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


def molecule(n, ls=None):
    """2 n electrons on the 15-atom family member; ls: momenta of its shells in turn."""
    m = inputs.family_member(3).molecule
    A, b = m.n_atoms, m.basis
    Z = np.full(A, (2 * n) // A, dtype=np.float64)
    Z[: 2 * n - int(Z.sum())] += 1.0
    if ls is not None:
        l = np.array([ls[s % len(ls)] for s in range(b.n_shells)], np.int32)
        b = inputs.Basis(b.shell_atom, l, b.shell_nprim, b.prim_exp, b.prim_coef)
        m = dataclasses.replace(m, basis=b,
                                C_full=inputs.s_orthonormal_coefficients(inputs.overlap_matrix(m.xyz, b), 5))
    return dataclasses.replace(m, Z=Z, n_up=n, n_dn=n)


@pytest.mark.parametrize("n,ls", [(1, None), (8, None), (9, None), (16, None), (17, None), (32, None), (33, None),
                                  (48, None), (49, None), (56, None), (57, None), (60, None), (64, None),
                                  (20, (0,)), (20, (0, 0, 0, 1)), (20, (0, 0, 1)), (57, (2,)), (33, (1, 2))])
def test_against_oracle(dev, n, ls):
    """FP64 to the parity suite's bound, mixed within the mixed suite's."""
    from oracle import derivatives as dv, wavefunction as wf
    from paper_2511_05222_amd import vmc
    m = molecule(n, ls)
    r = inputs.initial_walkers(m, 3, 3)
    ref = dv.measure(wf.System(m), m.xyz, r)
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-3)):
        ctx = vmc.Context(m, max_walkers=3, precision=prec, promote_fraction=0.0)
        out = ctx.measure(torch.tensor(r, device=dev))
        for a, b in (("dEL_dR", "H"), ("O", "O"), ("G", "G")):
            err = np.abs(out[a].cpu().numpy() - ref[b]).max() / np.abs(ref[b]).max()
            assert err <= tol, (prec, a, err)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [1, 13, 40, 58])
def test_many_walkers(dev, n, prec):
    """A walker's results do not depend on the launch it is in."""
    from paper_2511_05222_amd import vmc
    m = molecule(n)
    W = 513
    w = torch.tensor(inputs.initial_walkers(m, W, 8), device=dev)
    ctx = vmc.Context(m, max_walkers=W, precision=prec, promote_fraction=0.0, staging_walkers=W)
    many, parts = ctx.measure(w), [ctx.measure(x.contiguous()) for x in (w[:500], w[500:512], w[512:])]
    for k in many:
        assert torch.equal(many[k], torch.cat([p[k] for p in parts])), k


@pytest.mark.parametrize("n,ls", [(32, (0,)), (33, (0,)), (48, (0,)), (49, (0,)), (56, (0,)), (40, (0, 0, 0, 1)),
                                  (50, (0,) * 13 + (1,)), (56, (0, 0, 1))])
def test_subtiles_of_many_shells(dev, n, ls):
    """FP64 takes 7 shells at a time, from 33 orbitals on 14: sub-tiles of 16,
    14 and fewer.  (FP64 only: FP32 shares no sums, and some of these bases
    give Slater blocks of condition 2e5.)"""
    from oracle import derivatives as dv, wavefunction as wf
    from paper_2511_05222_amd import vmc
    m = molecule(n, ls)
    r = inputs.initial_walkers(m, 3, 3)
    ref = dv.measure(wf.System(m), m.xyz, r)
    out = vmc.Context(m, max_walkers=3).measure(torch.tensor(r, device=dev))
    for a, b in (("dEL_dR", "H"), ("O", "O"), ("G", "G")):
        err = np.abs(out[a].cpu().numpy() - ref[b]).max() / np.abs(ref[b]).max()
        assert err <= 1e-10, (a, err)
