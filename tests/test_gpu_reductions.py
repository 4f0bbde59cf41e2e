"""The reductions over walkers (estimators, vector-Jacobian product) and the
choice of the walkers measured again in FP64, at the edges of their turns of
8, 16 and 32 walkers, of 256 segments and of 1024 threads.  The sums are
compared with numpy's over the per-walker FP64 measurement: every partial sum
is FP64, so 1e-12 of the sum of magnitudes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2511_05222_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 8, 9, 15, 16, 17, 33, 511, 513, 4095, 4096, 4097, 8200]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_05222_amd import vmc
    vmc.lib()
    return torch.device("cuda:0")


def mean(x, wt):
    """Weighted mean over walkers and the same of magnitudes."""
    w = wt.reshape((-1,) + (1,) * (x.ndim - 1))
    return (w * x).sum(0) / wt.sum(), (w * np.abs(x)).sum(0) / wt.sum()


@pytest.mark.parametrize("W", SIZES)
def test_estimators(dev, W):
    from paper_2511_05222_amd import vmc
    m = inputs.make_config(0).molecule
    ctx = vmc.Context(m, max_walkers=W, staging_walkers=W)
    w = torch.tensor(inputs.initial_walkers(m, W, 3), device=dev)
    wt = torch.tensor(np.random.default_rng(W).uniform(0.2, 2.0, W), device=dev)
    one = {k: v.cpu().numpy() for k, v in ctx.measure(w).items()}
    for weights in (None, wt):
        v = np.ones(W) if weights is None else wt.cpu().numpy()
        ctx.accumulate_walkers(w, weights)
        r = ctx.accumulate()
        e, P = one["EL"], one["dlnpsi_dR"] + 0.5 * one["dlnjac_dR"]
        E, aE = mean(e, v)
        assert abs(r["E"] - E) <= 1e-12 * aE
        d = e - E
        H, aH = mean(one["dEL_dR"], v)
        eP, aeP = mean(d[:, None, None] * P, v)
        scale = aH + 2 * aeP + 2 * aE * mean(np.abs(P), v)[0]
        assert (np.abs(r["F_bare"] + H + 2 * eP) <= 1e-12 * scale.max()).all()
        G, aG = mean(one["G"], v)
        eO, aeO = mean(d[:, None, None] * one["O"], v)
        assert (np.abs(r["dEL_dC_mean"] - G) <= 1e-12 * aG.max()).all()
        scale = 2 * aeO + 2 * aE * mean(np.abs(one["O"]), v)[0]
        assert (np.abs(r["dE_dC"] - 2 * eO) <= 1e-12 * scale.max()).all()


@pytest.mark.parametrize("W", SIZES)
def test_vjp(dev, W):
    from paper_2511_05222_amd import vmc
    m = inputs.make_config(0).molecule
    ctx = vmc.Context(m, max_walkers=W, staging_walkers=W)
    w = torch.tensor(inputs.initial_walkers(m, W, 4), device=dev)
    C = torch.tensor(np.ascontiguousarray(m.C), device=dev)
    R0 = torch.tensor(np.ascontiguousarray(m.xyz), device=dev)
    R = R0 + 0.01
    one = {k: v.cpu().numpy() for k, v in ctx.measure(w, C, R, R0).items()}
    g = np.random.default_rng(W).standard_normal((3, W))
    dC, dR = ctx.adjoint(w, C, R, R0, *[torch.tensor(x, device=dev) for x in g])
    q = g[:, :, None, None]
    for got, terms in ((dC, (q[0] * one["G"], q[1] * one["O"])),
                       (dR, (q[0] * one["dEL_dR"], q[1] * one["dlnpsi_dR"], q[2] * one["dlnjac_dR"]))):
        ref = sum(t.sum(0) for t in terms)
        scale = sum(np.abs(t).sum(0) for t in terms).max()
        assert (np.abs(got.cpu().numpy() - ref) <= 1e-12 * scale).all()


@pytest.mark.parametrize("W", [1, 2, 63, 64, 65, 130, 1022, 1024, 1026, 2500, 8190, 8194])
@pytest.mark.parametrize("frac", [1e-4, 0.02, 0.3, 0.75])
def test_promoted(dev, W, frac):
    """ceil(frac W) walkers carry FP64 results; of two walkers at the same
    place (equal keys) the lower index is taken first, and a batch of copies
    of one walker is taken from its start."""
    from paper_2511_05222_amd import vmc
    m = inputs.make_config(1).molecule
    outs = ("EL", "lnpsi", "dEL_dR", "O")
    h = (W + 1) // 2
    half = torch.tensor(inputs.initial_walkers(m, h, 5), device=dev)
    k = int(np.ceil(frac * W))
    c64 = vmc.Context(m, max_walkers=W, staging_walkers=W)
    c32 = vmc.Context(m, max_walkers=W, precision="mixed", promote_fraction=frac, staging_walkers=W)
    for w in (torch.cat([half, half])[:W].contiguous(), half[:1].expand(W, -1, -1).contiguous()):
        ref = {x: v.cpu().numpy() for x, v in c64.measure(w, outputs=outs).items()}
        got = {x: v.cpu().numpy() for x, v in c32.measure(w, outputs=outs).items()}
        same = np.all([np.all((got[x] == ref[x]).reshape(W, -1), axis=1) for x in outs], axis=0)
        assert same.sum() == k
        if W > 1:
            assert not (same[h:] & ~same[:W - h]).any()
    assert same[:k].all()
