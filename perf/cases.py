"""Performance cases of the VMC force path: what a program that uses the
package has it do, through its public entry points (`vmc.Context`,
`vmc.vmc_energy`, `vmc.zvector_*`, `vmc.jackknife_stats`).

Kinds of case
  chain       a production step: sweeps with measurement, then the estimators
              (E, bare force, dE/dC) are read and reset;
  equilibrate sweeps without measurement;
  measure     per-walker E_L, ln|Psi| and derivatives at given walkers;
  reweight    given walkers with weights added to the estimators, then read;
  gradient    forward and backward of the differentiable fixed-sample energy;
  solve       the Z-vector step: right-hand sides from dE/dC, CG, back-map,
              and with several replicas their jackknife mean and error.

Molecules: "h2", "9" and "21" (the 9- and 21-atom molecules of
inputs.make_config), "family:<g>" (member g of the 64-geometry mixed-size
family, 9 to 21 atoms).  Jastrow: "pade", "exp" (two-body forms) or "body"
(with the one- and three/four-body terms).  `ecp`: the valence-only molecule
with the seeded pseudopotential.
"""
import dataclasses
import math
from functools import lru_cache

import numpy as np
import torch

from paper_2511_05222_amd import inputs, vmc

RTOL = 1e-12


def _case(name, kind, mol, walkers, precision="mixed", steps=1, jastrow="pade", ecp=False, **more):
    return dict(name=name, kind=kind, mol=mol, walkers=walkers, precision=precision, steps=steps, jastrow=jastrow,
                ecp=ecp, **more)


def listed():
    return [
        # the smallest molecule, as a new user's first run and the test of a
        # set-up: every kernel is over in microseconds, so launches count
        _case("h2_chain_fp64", "chain", "h2", 1024, "fp64", steps=8),
        # a trial run on a few walkers: latency of every kernel of the step
        _case("atom9_few_mixed", "chain", "9", 64, steps=4),
        # the 9-atom molecule in full precision at its configured walker count
        _case("atom9_step_fp64", "chain", "9", 16384, "fp64", steps=2),
        # the headline production step: 21 atoms, 65536 walkers
        _case("atom21_step_mixed", "chain", "21", 65536),
        # the same in full precision, a quarter of the walkers
        _case("atom21_step_fp64", "chain", "21", 16384, "fp64"),
        # a member of the mixed-size family (18 atoms, 37 orbitals: no
        # multiple of a tile), an odd number of walkers
        _case("family_step_mixed", "chain", "family:0", 8191),
        # production with the one- and three/four-body Jastrow
        _case("body_step_mixed", "chain", "21", 8192, jastrow="body"),
        # production with a pseudopotential (the paper's own setting)
        _case("ecp_step_mixed", "chain", "9", 16384, ecp=True),
        # the differentiable energy at the 256 walkers of the differentiation
        # workload, away from the sampling geometry: forward and backward
        _case("gradient_fp64", "gradient", "21", 256, "fp64"),
        # reweighted estimators of given walkers
        _case("reweight_mixed", "reweight", "21", 8192),
        # the Z-vector step for one right-hand side, 47 x 188 rotations
        _case("zvector_one", "solve", "21", 0, "fp64", n_rhs=1, jacobi=True),
        # its error bar: 12 jackknife replicas through the same solve
        _case("zvector_jackknife", "solve", "21", 0, "fp64", n_rhs=12, jacobi=True),
    ]


def draw(rng):
    def upto(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["chain", "chain", "chain", "equilibrate", "measure", "reweight", "gradient", "solve"])
    sizes = inputs.family_sizes()
    g = rng.randrange(len(sizes))
    mol = rng.choice(["h2", "9", "21"] + 4 * ["family:%d" % g])
    precision = rng.choice(["mixed", "fp64"])
    if kind == "solve":
        return _drop(_case("", kind, mol if mol != "h2" else "9", 0, "fp64", n_rhs=rng.randint(1, 16),
                           jacobi=rng.random() < 0.75))
    jastrow = rng.choice(["pade", "pade", "exp", "body"])
    ecp = rng.random() < 0.25
    if mol == "h2":
        jastrow, ecp = ("pade" if jastrow == "body" else jastrow), False
    if ecp and mol != "9" and sizes[g] > 12:
        mol = "9"
    if kind in ("measure", "reweight", "gradient"):
        # (the plain reference of these covers the two-body forms)
        jastrow, ecp = ("pade" if jastrow == "body" else jastrow), False
        walkers = upto(16, 2048 if kind == "measure" else 4096)
    else:
        walkers = upto(16, 6000 if jastrow == "body" else 16000)
    steps = rng.randint(1, 4) if walkers < 2000 else 1
    return _drop(_case("", kind, mol, walkers, precision, steps=steps, jastrow=jastrow, ecp=ecp))


def _drop(case):
    return {k: v for k, v in case.items() if k != "name"}


@lru_cache(maxsize=None)
def _molecule(name, jastrow, ecp):
    if name.startswith("family:"):
        m = inputs.family_member(int(name.split(":")[1])).molecule
    else:
        m = inputs.make_config({"h2": 0, "9": 1, "21": 2}[name]).molecule
    if ecp:
        m = inputs.with_ecp(m, 5)
    if jastrow == "body":
        m = inputs.with_body_jastrow(m, 7)
    elif jastrow == "exp":
        m = dataclasses.replace(m, jastrow=inputs.Jastrow(ee_a=0.5, ee_F=1.3, ee_form=1))
    return m


def _mol(case):
    return _molecule(case["mol"], case["jastrow"], case["ecp"])


def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _walkers(m, W, seed):
    """Start positions: every electron at its atom plus N(0, 0.5^2)."""
    base = torch.tensor(m.xyz[inputs.init_atom_of_electron(m.Z, m.n_up, m.n_dn)], device="cuda")
    z = torch.randn((W,) + tuple(base.shape), dtype=torch.float64, device="cuda", generator=_gen(seed, "cuda"))
    return (base[None] + 0.5 * z).contiguous()


def _geometry(m, seed):
    """Sampling nuclei and nuclei displaced by about 0.02 bohr."""
    R0 = torch.tensor(m.xyz, device="cuda")
    return R0, R0 + 0.02 * torch.randn(R0.shape, dtype=torch.float64, device="cuda", generator=_gen(seed + 1, "cuda"))


def _weights(W, seed):
    z = torch.randn(W, dtype=torch.float64, device="cuda", generator=_gen(seed + 2, "cuda"))
    return torch.exp(0.5 * z)


def _solve_inputs(m, n_rhs, seed):
    """Virtual orbitals, replicas of dE/dC and the orbital Hessian
    diag(log-uniform in [0.5, 5]) + G G^T / 64."""
    n = m.n_occ
    Cv = torch.tensor(np.ascontiguousarray(m.C_full[:, n:]), device="cuda")
    M, nv = Cv.shape
    g = _gen(seed, "cuda")
    rnd = lambda *s: torch.randn(s, dtype=torch.float64, device="cuda", generator=g)
    dEdC = rnd(M, n) + 0.05 * rnd(n_rhs, M, n)
    d = nv * n
    G = rnd(d, 64)
    H = torch.mm(G, G.t().contiguous()) / 64.0
    H = 0.5 * (H + H.t())
    u = torch.rand(d, dtype=torch.float64, device="cuda", generator=g)
    H += torch.diag(torch.exp(math.log(0.5) + u * math.log(10.0)))
    return Cv, dEdC.contiguous(), H.contiguous()


def prepare(case, seed):
    m, kind = _mol(case), case["kind"]
    if kind == "solve":
        Cv, dEdC, H = _solve_inputs(m, case["n_rhs"], seed)
        return dict(case=case, Cv=Cv, dEdC=dEdC, H=H)
    W = case["walkers"]
    ctx = vmc.Context(m, max_walkers=W, precision=case["precision"], refresh_period=32)
    w = _walkers(m, W, seed)
    s = dict(case=case, ctx=ctx, w=w, seed=int(seed), at=0)
    if kind in ("chain", "equilibrate"):
        # the chains leave their starting positions
        ctx.sweep(w, 4, int(seed), sweep_offset=0, measure=False)
        s["at"] = 4
    if kind == "reweight":
        s["wt"] = _weights(W, seed)
    if kind in ("measure", "gradient"):
        s["C"] = torch.tensor(m.C, device="cuda")
        s["R0"], s["R"] = _geometry(m, seed)
    if kind == "gradient":
        s["lnpsi0"] = ctx.measure(w, s["C"], s["R0"], s["R0"], outputs=("lnpsi",))["lnpsi"]
        s["C"].requires_grad_(True)
        s["R"].requires_grad_(True)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "solve":
        b = vmc.zvector_rhs(s["Cv"], s["dEdC"])
        k = case["n_rhs"]
        z, its = vmc.zvector_solve(s["H"], b.view(k, -1), rtol=RTOL, maxit=2000, jacobi=case["jacobi"])
        Z = vmc.zvector_backmap(s["Cv"], z.view(b.shape))
        out = dict(b=b, z=z, Z=Z, iterations=its)
        if k > 1:
            out["mean"], out["sigma"] = vmc.jackknife_stats(Z)
        return out
    ctx, w = s["ctx"], s["w"]
    if kind in ("chain", "equilibrate"):
        ctx.sweep(w, case["steps"], s["seed"], sweep_offset=s["at"], measure=kind == "chain")
        s["at"] += case["steps"]
        return (w, ctx.accumulate(reset=True)) if kind == "chain" else w
    if kind == "reweight":
        ctx.accumulate_walkers(w, s["wt"])
        return ctx.accumulate(reset=True)
    if kind == "measure":
        return ctx.measure(w, s["C"], s["R"], s["R0"])
    E = vmc.vmc_energy(s["C"], s["R"], ctx, w, s["R0"], s["lnpsi0"])
    dC, dR = torch.autograd.grad(E, (s["C"], s["R"]))
    return E, dC, dR


def work(case):
    """Counts of the method: positions read (and written by a sweep), C read,
    the returned values written; MO products on both sides, AO values and
    derivatives, ratios, updates and inverses, pair terms."""
    m = _mol(case)
    b, N, n, M, A = m.basis, m.n_elec, m.n_occ, m.basis.n_ao, m.n_atoms
    P, S = b.n_prim, b.n_shells
    if case["kind"] == "solve":
        d, k = n * (M - n), case["n_rhs"]
        its = 75   # of this Hessian to 1e-12
        return {"bytes": 8.0 * its * d * (d + 1) / 2, "flops": 2.0 * its * k * d * d}
    moves = N * (2 * M * n + 3 * P + 6 * S + 3 * M) + N * (2 * n + 24 * (N - 1) + 0.5 * 2 * n * n) + (N / 32) * 2 * n ** 3
    forward = 10 * N * M * n + N * (10 * P + 6 * S + 15 * M) + 8 * n ** 3 + 20 * N * (N - 1) + 8 * N * n
    adjoint = 10 * N * M * n + N * (60 * M + 12 * P) + 8 * n ** 3
    MJ = m.jastrow.jas_basis.n_ao if m.jastrow.jas_basis is not None else 0
    if MJ:
        moves += 2 * N * MJ * MJ
        forward += 2 * N * MJ * MJ + 8 * N * MJ
        adjoint += 2 * N * MJ * MJ + 60 * N * MJ
    if m.ecp is not None:
        q = 12 * 16
        forward += q * (2 * M * n + 30 * N)
        adjoint += q * (8 * M * n + 30 * M)
    kind, W, steps = case["kind"], case["walkers"], case["steps"]
    pos, coef, res = 24.0 * N * W, 8.0 * M * n, 8.0 * (2 * M * n + 3 * A)
    if kind == "chain":
        return {"bytes": steps * 2 * pos + coef + res, "flops": float(W * steps * (moves + forward + adjoint))}
    if kind == "equilibrate":
        return {"bytes": steps * 2 * pos + coef, "flops": float(W * steps * moves)}
    if kind == "measure":
        return {"bytes": pos + coef + 8.0 * W * (3 + 9 * A + 2 * M * n), "flops": float(W * (forward + adjoint))}
    if kind == "reweight":
        return {"bytes": pos + coef + res, "flops": float(W * (forward + adjoint))}
    return {"bytes": pos + coef + res, "flops": float(W * (2 * forward + adjoint))}


# ---------------------------------------------------------------------------
# The same results from plain torch in 64 bits.
# ---------------------------------------------------------------------------

def _ao_tables(m):
    """Per AO: shell, monomial powers, component factor; per primitive the
    coefficient that makes the contracted shell normalised."""
    b = m.basis
    off = b.prim_offsets()
    npr = int(b.shell_nprim.max())
    al, cp = np.ones((b.n_shells, npr)), np.zeros((b.n_shells, npr))
    comps = {0: [(0, 0, 0)], 1: [(1, 0, 0), (0, 1, 0), (0, 0, 1)],
             2: [(2, 0, 0), (1, 1, 0), (1, 0, 1), (0, 2, 0), (0, 1, 1), (0, 0, 2)]}
    shell, pw, eta = [], [], []
    for s in range(b.n_shells):
        l, k = int(b.shell_l[s]), int(b.shell_nprim[s])
        a = b.prim_exp[off[s]:off[s] + k]
        c = b.prim_coef[off[s]:off[s] + k] * (2 * a / np.pi) ** 0.75 * (4 * a) ** (0.5 * l)
        p = a[:, None] + a[None, :]
        c = c / np.sqrt((c[:, None] * c[None, :] * (np.pi / p) ** 1.5 / (2 * p) ** l).sum())
        al[s, :k], cp[s, :k] = a, c
        for q in comps[l]:
            shell.append(s)
            pw.append(q)
            eta.append(1.0 / math.sqrt(math.prod({0: 1, 1: 1, 2: 3}[x] for x in q)))
    t = lambda x: torch.tensor(np.array(x), device="cuda")
    pw = np.array(pw)
    return dict(al=t(al), cp=t(cp), atom=t(b.shell_atom.astype(np.int64)), shell=t(shell), eta=t(eta),
                hot=[t((pw == k).astype(np.float64)) for k in range(3)], l=t(pw.sum(1).astype(np.float64)))


def _ao(t, d, rho):
    """AO values, gradients and Laplacians [.., 5, M] from the displacements
    d [.., S, 3] to the shells' atoms and rho = |d|^2."""
    e = t["cp"] * torch.exp(-t["al"] * rho[..., None])
    R = [((-t["al"]) ** k * e).sum(-1)[..., t["shell"]] for k in range(3)]
    d, rho = d[..., t["shell"], :], rho[..., t["shell"]]
    h0, h1, h2 = t["hot"]
    f, f1, f2 = h0 + h1 * d + h2 * d * d, h1 + 2 * h2 * d, 2 * h2
    x, y, z = 0, 1, 2
    P = t["eta"] * f[..., x] * f[..., y] * f[..., z]
    g = [t["eta"] * f1[..., a] * f[..., b] * f[..., c] for a, b, c in ((x, y, z), (y, x, z), (z, x, y))]
    lap = t["eta"] * (f2[..., x] * f[..., y] * f[..., z] + f2[..., y] * f[..., x] * f[..., z] +
                      f2[..., z] * f[..., x] * f[..., y])
    out = [P * R[0]] + [g[k] * R[0] + 2 * d[..., k] * P * R[1] for k in range(3)]
    out.append(lap * R[0] + (4 * t["l"] + 6) * P * R[1] + 4 * rho * P * R[2])
    return torch.stack(out, dim=-2)


def _warp(r, R, R0):
    """Space-warped positions and ln Jac (weights d^-4 at R0)."""
    d = r[:, :, None, :] - R0                                     # [W, N, A, 3]
    d2 = (d * d).sum(-1)
    k = d2 ** -2
    om = k / k.sum(-1, keepdim=True)
    gk = -4 * d / d2[..., None]
    gom = om[..., None] * (gk - (om[..., None] * gk).sum(2, keepdim=True))
    disp = (R - R0)[:, None]                                      # [W, 1, A, 3]
    J = torch.eye(3, dtype=r.dtype, device=r.device) + (disp[..., :, None] * gom[..., None, :]).sum(2)
    return r + (om[..., None] * disp).sum(2), torch.linalg.det(J).log().sum(-1)


def _forward(m, t, r0, C, R, R0):
    """E_L, ln|Psi|, ln Jac of walkers r0 with per-walker C [W, M, n], R [W, A, 3]."""
    r, lnjac = _warp(r0, R, R0)
    W, N, n, nu = r.shape[0], m.n_elec, m.n_occ, m.n_up
    d = r[:, :, None, :] - R[:, t["atom"]][:, None]               # [W, N, S, 3]
    ao = _ao(t, d, (d * d).sum(-1))                               # [W, N, 5, M]
    phi = torch.bmm(ao.reshape(W, N * 5, -1), C).reshape(W, N, 5, n)
    lnpsi, b, lp = 0.0, [], []
    for s in (slice(0, nu), slice(nu, N)):
        K = torch.linalg.inv(phi[:, s, 0])                        # [W, i, e]
        lnpsi = lnpsi + torch.linalg.slogdet(phi[:, s, 0])[1]
        q = (phi[:, s, 1:] * K.transpose(1, 2)[:, :, None, :]).sum(-1)
        b.append(q[..., :3])
        lp.append(q[..., 3])
    b, lp = torch.cat(b, 1), torch.cat(lp, 1)
    a, F = m.jastrow.ee_a, m.jastrow.ee_F
    i, j = torch.triu_indices(N, N, 1, device=r.device)
    v = r[:, i] - r[:, j]
    s = (v * v).sum(-1).sqrt()
    if m.jastrow.ee_form == 1:
        u, u1, u2 = a * (1 - torch.exp(-F * s)) / F, a * torch.exp(-F * s), -a * F * torch.exp(-F * s)
    else:
        u, u1, u2 = a * s / (1 + F * s), a / (1 + F * s) ** 2, -2 * a * F / (1 + F * s) ** 3
    f = (u1 / s)[..., None] * v
    g = torch.zeros_like(r).index_add(1, i, f).index_add(1, j, -f)
    lapJ = 2 * (u2 + 2 * u1 / s).sum(-1)
    Z = torch.tensor(m.Z, device=r.device)
    ne = (r[:, :, None, :] - R[:, None]).pow(2).sum(-1).sqrt()
    E = -0.5 * ((lp + 2 * (b * g).sum(-1) + (g * g).sum(-1)).sum(-1) + lapJ) + (1 / s).sum(-1) - (Z / ne).sum((1, 2))
    p, q = torch.triu_indices(m.n_atoms, m.n_atoms, 1, device=r.device)
    E = E + (Z[p] * Z[q] / (R[:, p] - R[:, q]).pow(2).sum(-1).sqrt()).sum(-1)
    return E, lnpsi + u.sum(-1), lnjac


def _plain(m, r, R, R0, grads=True, each=None):
    """Per-walker results at C of the molecule, in chunks; `each` reduces a chunk's."""
    t = _ao_tables(m)
    C0 = torch.tensor(m.C, device="cuda")
    step = max(1, int(1.5e9 / (m.n_elec * m.basis.n_ao * 8 * 40)))
    got = []
    for k in range(0, r.shape[0], step):
        w = r[k:k + step]
        C = C0.expand(w.shape[0], -1, -1).clone().requires_grad_(grads)
        Rw = R.expand(w.shape[0], -1, -1).clone().requires_grad_(grads)
        E, lp, lj = _forward(m, t, w, C, Rw, R0)
        o = dict(EL=E.detach(), lnpsi=lp.detach(), lnjac=lj.detach())
        if grads:
            o["G"], o["dEL_dR"] = torch.autograd.grad(E.sum(), (C, Rw), retain_graph=True)
            o["O"], o["dlnpsi_dR"] = torch.autograd.grad(lp.sum(), (C, Rw), retain_graph=True)
            o["dlnjac_dR"], = torch.autograd.grad(lj.sum(), (Rw,))
        got.append(each(o, k) if each else o)
    return got


def exact(case, seed):
    m, kind = _mol(case), case["kind"]
    if kind in ("chain", "equilibrate"):
        return None   # Markov chains: what follows an accept decision has no value of its own
    if kind == "solve":
        Cv, dEdC, H = _solve_inputs(m, case["n_rhs"], seed)
        b = torch.matmul(Cv.t().contiguous(), dEdC)
        k = case["n_rhs"]
        z = -torch.linalg.solve(H, b.reshape(k, -1).t().contiguous()).t().contiguous()
        Z = torch.matmul(Cv, z.view(b.shape))
        out = dict(b=b, z=z, Z=Z, iterations=None)
        if k > 1:
            mean = Z.mean(0)
            out["mean"], out["sigma"] = mean, ((k - 1) / k * ((Z - mean) ** 2).sum(0)).sqrt()
        return out
    W = case["walkers"]
    r = _walkers(m, W, seed)
    R0, R = _geometry(m, seed)
    if kind == "measure":
        got = _plain(m, r, R, R0)
        return {k: torch.cat([o[k] for o in got]) for k in got[0]}
    if kind == "reweight":
        wt = _weights(W, seed)
        n_atoms = m.n_atoms

        def sums(o, k):
            q = wt[k:k + o["EL"].shape[0]]
            P = o["dlnpsi_dR"] + 0.5 * o["dlnjac_dR"]
            mean = lambda x: (q.view([-1] + [1] * (x.dim() - 1)) * x).sum(0)
            eP, eO = o["EL"][:, None, None] * P, o["EL"][:, None, None] * o["O"]
            return [mean(x) for x in (o["EL"], o["dEL_dR"], P, eP, o["O"], eO, o["G"])]

        E, H, P, eP, O, eO, G = (sum(x) / wt.sum() for x in zip(*_plain(m, r, R0, R0, each=sums)))
        return dict(E=E, E_sigma=None, F_bare=-H - 2 * (eP - E * P), dE_dC=2 * (eO - E * O), dEL_dC_mean=G,
                    n_samples=None)
    ln0 = torch.cat([o["lnpsi"] for o in _plain(m, r, R0, R0, grads=False)])
    got = _plain(m, r, R, R0)
    o = {k: torch.cat([x[k] for x in got]) for k in got[0]}
    w = torch.softmax(2 * (o["lnpsi"] - ln0) + o["lnjac"], 0)
    E = (w * o["EL"]).sum()
    c = (w * (o["EL"] - E))[:, None, None]
    dC = (w[:, None, None] * o["G"] + 2 * c * o["O"]).sum(0)
    dR = (w[:, None, None] * o["dEL_dR"] + c * (2 * o["dlnpsi_dR"] + o["dlnjac_dR"])).sum(0)
    return E, dC, dR
