"""The in-register inverse rebuild at the edges of its register classes (16,
32, 48 and 64 orbitals) and of its 16-row groups: FP64 accept bits, positions
and the per-walker measurement against the oracle, and the mixed sweep's and
measurement's own rebuilds.  The molecule is the 15-atom family member's
geometry and basis with charges spread so that 2 n electrons are neutral."""
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


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 47, 48, 49, 63, 64])
def test_register_classes(dev, n):
    """Rebuilds every 5th move (at odd places of the blocks), four sweeps."""
    from oracle import derivatives as dv, sampler, wavefunction as wf
    from paper_2511_05222_amd import vmc
    m = molecule(n)
    W, sweeps, seed = 3, 4, 77
    w0 = inputs.initial_walkers(m, W, seed)
    s = wf.System(m)
    ref, bits = sampler.run(s, w0, sweeps, seed, refresh_period=5)
    ctx = vmc.Context(m, max_walkers=W, refresh_period=5)
    w = torch.tensor(w0, device=dev)
    acc = torch.zeros((sweeps, m.n_elec, W), dtype=torch.uint8, device=dev)
    ctx.sweep(w, sweeps, seed, measure=False, accept=acc)
    assert np.array_equal(acc.cpu().numpy().astype(bool), bits)
    assert np.abs(w.cpu().numpy() - ref.r).max() < 1e-12
    out = ctx.measure(w)
    r = dv.measure(s, s.xyz, ref.r)
    for a, b in (("EL", "E_L"), ("lnpsi", "lnpsi"), ("dEL_dR", "H"), ("O", "O"), ("G", "G")):
        x, y = out[a].cpu().numpy(), r[b]
        assert np.abs(x - y).max() <= 1e-10 * np.abs(y).max(), a
    # mixed: the sweep's inverses (FP32 rows, FP64 rebuild) decide as FP64's
    mix = vmc.Context(m, max_walkers=W, refresh_period=5, precision="mixed")
    wm = torch.tensor(w0, device=dev)
    am = torch.zeros_like(acc)
    mix.sweep(wm, 1, seed, measure=False, accept=am[:1])
    assert (am[0] != acc[0]).float().mean().item() <= 0.02
