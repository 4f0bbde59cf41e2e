"""The per-walker dense kernel at the edges of its orbital classes (16, 32, 48
and 64) and of its groups of lanes over electron pairs (32, 64 and 128): the
estimators of a measured sweep, from the sweep's inverses (the blocks that the
sweep leaves stale inverted anew), against the same walkers measured from
their MO rows alone.  FP64 agrees to the parity suite's bound; in mixed
precision the FP32 inverse is corrected by one FP64 step, which leaves the
mixed suite's bound on derivatives."""
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


def molecule(n):
    m = inputs.family_member(3).molecule
    A = m.n_atoms
    Z = np.full(A, (2 * n) // A, dtype=np.float64)
    Z[: 2 * n - int(Z.sum())] += 1.0
    return dataclasses.replace(m, Z=Z, n_up=n, n_dn=n)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-3)])
@pytest.mark.parametrize("refresh", [32, 1])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
def test_state_against_rows(dev, n, refresh, prec, tol):
    """refresh 32: inverses carried over; 1: every block stale at the sweep's end."""
    from paper_2511_05222_amd import vmc
    m = molecule(n)
    W = 7
    ctx = vmc.Context(m, max_walkers=W, precision=prec, refresh_period=refresh, promote_fraction=0.0)
    w = torch.tensor(inputs.initial_walkers(m, W, 6), device=dev)
    ctx.sweep(w, 2, 9, measure=False)
    ctx.sweep(w, 1, 9, sweep_offset=2, measure=True)
    a = ctx.accumulate()
    ctx.accumulate_walkers(w)
    b = ctx.accumulate()
    for k in ("E", "F_bare", "dE_dC", "dEL_dC_mean"):
        x, y = np.asarray(a[k]), np.asarray(b[k])
        assert np.abs(x - y).max() <= tol * max(np.abs(y).max(), 1e-300), k


@pytest.mark.parametrize("n", [15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
def test_newton_step_corrects_the_sweep_inverse(dev, n):
    """The energy from the sweep's FP32 inverses against that from the MO rows
    alone.  Both take the same FP32 orbital values and sum in FP64, so what is
    left is the inverse: R = I - A K is 2e-5 .. 2e-3 after a sweep of FP32
    updates and shifts the energy by 9e-9 .. 1e-5 of itself; one FP64 step
    leaves R^2, at most 7e-11 (all from an emulation of such a sweep on the
    host)."""
    from paper_2511_05222_amd import vmc
    m = molecule(n)
    ctx = vmc.Context(m, max_walkers=7, precision="mixed", refresh_period=4 * n + 1, promote_fraction=0.0)
    w = torch.tensor(inputs.initial_walkers(m, 7, 6), device=dev)
    ctx.sweep(w, 2, 9, measure=False)
    ctx.sweep(w, 1, 9, sweep_offset=2, measure=True)
    a = ctx.accumulate()["E"]
    ctx.accumulate_walkers(w)
    b = ctx.accumulate()["E"]
    assert abs(a - b) <= 1e-9 * max(abs(b), 10.0), (a, b)
