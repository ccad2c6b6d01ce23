"""Performance cases: what a user of this framework has it do, through its public
entry points, from single small propagations to paper-size products.

A case is a dict of plain values.  `kind` names the work:

  rk4      fixed-step RK4 mean-field propagation of a batch (`Context.run`)
  dp5      adaptive Dormand-Prince propagation of a batch (`Context.run`)
  columns  decoupled (AT) dynamics of many initial states per path on a
           truncated coupling matrix (`Context.load_system_coo` + `Context.run`)
  adjoint  forward and backward of the differentiable propagation (`propagate`)
  build    coupling matrices of a top + linear rotor (`Context.build_couplings`)
  xsec     cross sections of a propagated batch (`Context.cross_sections`)
  rates    rate coefficients from cross sections (`mqct_rate_coefficients`)

The collision systems are seeded synthetic ones of the forms the framework's own
workloads have: a rigid rotor + atom, two rigid rotors, a random smooth Hermitian
coupling with an asymmetric top's or a dense spectrum, truncated m-block couplings.
Every potential is written M(R_k) = sum_t V_t(R_k) G_t, which `prepare` turns into
the tables the framework takes and `exact` propagates directly in 64 bits.

The outputs of a propagation are its final probabilities, amplitudes, classical
states, times, counts and status.  The conservation diagnostics (norm_err,
energy_err, angmom_err) are left out: at these windows they are rounding residues.
"""
import functools
import math

import numpy as np
import torch

import paper_2312_02322_amd as mq

CM = 1.0 / 219474.6313705          # hartree per cm^-1
ANG = 1.0 / 0.529177210903         # bohr per angstrom
AMU = 1822.888486209               # electron masses per atomic mass unit
DEV = "cuda"
ITEM = {"R64": 8, "C128": 16, "R32": 4, "C64": 8}


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # one trajectory of a small system: a script's single call, all latency
        dict(name="single_rotor", kind="rk4", system="rotor_atom", jmax=4, K=200, storage="R64",
             layout="dense", schedule="auto", B=1, steps=100, dt=40.0),
        # 64 trajectories of rotor + atom, N = 49, FP64: the small workload through collisions
        dict(name="rotor_atom_64", kind="rk4", system="rotor_atom", jmax=6, K=200, storage="R64",
             layout="dense", schedule="auto", B=64, steps=500, dt=47.8),
        # adaptive steps on truncated tables, two rotors, N = 256: the work list
        dict(name="two_rotor_dp5", kind="dp5", system="rotor_rotor", jmax=3, K=200, storage="R64",
             layout="sparse", schedule="auto", B=192),
        # a Monte-Carlo batch on the default schedule with FP64 complex tables, N = 969
        dict(name="top_atom_fp64", kind="rk4", system="random", top=8, K=200, storage="C128",
             layout="dense", schedule="auto", B=1024, steps=2, dt=12.0),
        # the mid-collision window of N = 969 with FP32 tables on the matrix cores
        dict(name="top_atom_binned", kind="rk4", system="random", top=8, K=200, storage="C64",
             layout="dense", schedule="binned", B=4096, steps=3, dt=12.0),
        # N = 4096, 512 trajectories scattered over the grid: the headline's mid-collision stages
        dict(name="random4096_binned", kind="rk4", system="random", n=4096, K=128, storage="C64",
             layout="dense", schedule="binned", B=512, steps=1, dt=10.0),
        # the paper's form: 206 k states, 13 M kept couplings, 100 initial states on one path
        dict(name="columns_paper", kind="columns", levels=5300, jtop=38, partners=92, K=63,
             storage="R32", paths=1, cols=100, steps=8),
        # a middle-sized truncated basis, FP64 tables, an odd number of columns on two paths
        dict(name="columns_fp64", kind="columns", levels=1501, jtop=19, partners=60, K=63,
             storage="R64", paths=2, cols=37, steps=12),
        # gradient with respect to 96 potential coefficients, N = 256
        dict(name="two_rotor_gradient", kind="adjoint", jmax=3, K=200, layout="sparse", B=1024,
             steps=64, dt=23.0),
        # coupling matrices of a top (j1 <= 5) + para-H2 on the radial grid
        dict(name="coupling_tables", kind="build", j1max=5, j2max=4, terms=83, K=63),
        # cross sections of a finished batch
        dict(name="cross_sections", kind="xsec", B=4096, top=8),
        # rate coefficients between the paper's number of levels
        dict(name="rates_1032", kind="rates", L=1032, nE=10, nT=20),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["small", "small", "dp5", "window", "window", "columns", "adjoint", "build",
                       "xsec", "rates"])
    if kind == "small":
        system = rng.choice(["rotor_atom", "rotor_atom", "rotor_rotor"])
        return dict(kind="rk4", system=system,
                    jmax=rng.randint(2, 9 if system == "rotor_atom" else 3),
                    K=rng.randint(120, 260), storage=rng.choice(["R64", "R64", "R32"]),
                    layout=rng.choice(["dense", "sparse"]), schedule="auto",
                    B=_logint(rng, 1, 200), steps=_logint(rng, 5, 60), dt=rng.uniform(20.0, 45.0))
    if kind == "dp5":
        return dict(kind="dp5", system=rng.choice(["rotor_atom", "rotor_rotor"]),
                    jmax=rng.randint(2, 3), K=rng.randint(150, 220), storage="R64",
                    layout=rng.choice(["dense", "sparse"]), schedule="auto",
                    B=_logint(rng, 8, 200))
    if kind == "window":
        storage = rng.choice(["C64", "C128"])
        return dict(kind="rk4", system="random", n=_logint(rng, 150, 1200), K=rng.randint(60, 200),
                    storage=storage, layout="dense",
                    schedule="binned" if storage == "C64" else rng.choice(["auto", "binned"]),
                    B=_logint(rng, 64, 3000), steps=rng.randint(1, 3), dt=rng.uniform(5.0, 12.0))
    if kind == "columns":
        return dict(kind="columns", levels=_logint(rng, 200, 3000), jtop=rng.randint(6, 24),
                    partners=rng.randint(10, 60), K=rng.randint(20, 63),
                    storage=rng.choice(["R32", "R64"]), paths=rng.randint(1, 3),
                    cols=_logint(rng, 1, 128), steps=rng.randint(2, 12))
    if kind == "adjoint":
        return dict(kind="adjoint", jmax=rng.randint(1, 3), K=rng.randint(100, 200),
                    layout=rng.choice(["dense", "sparse"]), B=_logint(rng, 16, 700),
                    steps=_logint(rng, 4, 40), dt=rng.uniform(10.0, 25.0))
    if kind == "build":
        return dict(kind="build", j1max=rng.randint(2, 4), j2max=rng.choice([0, 2, 4]),
                    terms=rng.randint(5, 83), K=rng.randint(7, 63))
    if kind == "xsec":
        return dict(kind="xsec", B=_logint(rng, 50, 8000), top=rng.randint(2, 8))
    return dict(kind="rates", L=_logint(rng, 20, 900), nE=rng.randint(3, 14), nT=rng.randint(1, 20))


# ---------------------------------------------------------------- angular factors

def _plm(lmax, x):
    """Normalised associated Legendre functions P[l][m](x), m >= 0, such that
    Y_lm = P[l][m](cos theta) e^{i m phi} with the Condon-Shortley phase."""
    s = np.sqrt(1.0 - x * x)
    P = [[None] * (lmax + 1) for _ in range(lmax + 1)]
    P[0][0] = np.full_like(x, math.sqrt(1.0 / (4.0 * math.pi)))
    for m in range(1, lmax + 1):
        P[m][m] = -math.sqrt((2 * m + 1) / (2.0 * m)) * s * P[m - 1][m - 1]
    for m in range(lmax):
        P[m + 1][m] = math.sqrt(2 * m + 3) * x * P[m][m]
    for m in range(lmax + 1):
        for l in range(m + 2, lmax + 1):
            a = math.sqrt((4.0 * l * l - 1) / (l * l - m * m))
            b = math.sqrt(((l - 1.0) ** 2 - m * m) / (4.0 * (l - 1) ** 2 - 1))
            P[l][m] = a * (x * P[l - 1][m] - b * P[l - 2][m])
    return P


@functools.lru_cache(None)
def _ylm_matrix(jmax, l, mu):
    """<j'' m''| Y_{l mu} |j' m'> over |j m>, j <= jmax (Gauss-Legendre quadrature, exact)."""
    x, w = np.polynomial.legendre.leggauss(jmax + l + 2)
    P = _plm(max(jmax, l), x)
    f = lambda a, m: P[a][m] if m >= 0 else (-1.0) ** (-m) * P[a][-m]
    st = [(j, m) for j in range(jmax + 1) for m in range(-j, j + 1)]
    A = np.zeros((len(st), len(st)))
    for a, (jb, mb) in enumerate(st):
        for b, (ja, ma) in enumerate(st):
            if mb == ma + mu:
                A[a, b] = 2.0 * math.pi * float(np.sum(w * f(jb, mb) * f(l, mu) * f(ja, ma)))
    A[np.abs(A) < 1e-13] = 0.0
    return A


def _cg(j1, m1, j2, m2, J):
    """<j1 m1 j2 m2 | J m1 + m2> (Racah's sum)."""
    M, f = m1 + m2, math.factorial
    if abs(m1) > j1 or abs(m2) > j2 or abs(M) > J or not abs(j1 - j2) <= J <= j1 + j2:
        return 0.0
    pre = math.sqrt((2 * J + 1) * f(J + j1 - j2) * f(J - j1 + j2) * f(j1 + j2 - J)
                    / f(j1 + j2 + J + 1))
    pre *= math.sqrt(f(J + M) * f(J - M) * f(j1 - m1) * f(j1 + m1) * f(j2 - m2) * f(j2 + m2))
    s = 0.0
    for k in range(max(0, j2 - J - m1, j1 - J + m2), min(j1 + j2 - J, j1 - m1, j2 + m2) + 1):
        s += (-1) ** k / (f(k) * f(j1 + j2 - J - k) * f(j1 - m1 - k) * f(j2 + m2 - k)
                          * f(J - j2 + m1 + k) * f(J - j1 - m2 + k))
    return pre * s


def _jx_blocks(js):
    """J_x over consecutive blocks of |j m>, m = -j..j: coordinate list."""
    r, c, v, o = [], [], [], 0
    for j in js:
        for m in range(-j, j):
            e = 0.5 * math.sqrt(j * (j + 1) - m * (m + 1))
            r += [o + m + j, o + m + 1 + j]
            c += [o + m + 1 + j, o + m + j]
            v += [e, e]
        o += 2 * j + 1
    return np.array(r, np.int32), np.array(c, np.int32), np.array(v, np.float64)


BIPOLAR = [(0, 0, 0), (1, 0, 1), (0, 1, 1), (1, 1, 0), (1, 1, 2), (2, 0, 2),
           (0, 2, 2), (2, 1, 1), (2, 1, 3), (1, 2, 1), (1, 2, 3), (2, 2, 0)]


@functools.lru_cache(None)
def _rotor_rotor_G(jmax):
    G = []
    for l1, l2, lam in BIPOLAR:
        s = 0.0
        for mu in range(-min(l1, l2), min(l1, l2) + 1):
            cg = _cg(l1, mu, l2, -mu, lam)
            if cg:
                s = s + 4.0 * math.pi * cg * np.kron(_ylm_matrix(jmax, l1, mu),
                                                     _ylm_matrix(jmax, l2, -mu))
        G.append(0.5 * (s + s.T))
    return np.stack(G)


# ---------------------------------------------------------------- collision systems

def _gen(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 16 + salt)


def _wall(rng):
    """A repulsive exponential with a dispersion tail, cm^-1 over angstrom."""
    a = rng.uniform(2.8, 3.4)
    return 1000.0 * math.exp(3.0 * a) * rng.uniform(0.8, 1.25), a, rng.uniform(5e4, 2e5)


def _system(case, seed):
    """R [K], E [N], V [T, K] and G [T, N, N] of M = sum_t V_t G_t, J_x, mu, channel sets."""
    rng = np.random.default_rng([int(seed), 77])
    R_ang = np.linspace(2.0, 20.0, case["K"])
    kind, s = case.get("system", "rotor_rotor"), {}
    if kind == "rotor_atom":
        jm = case["jmax"]
        A, a, C = _wall(rng)
        V, G = [], []
        for lam in range(5):
            fa, fe, fc = (1.0, 1.0, 1.0) if lam == 0 else (rng.uniform(-0.2, 0.2),
                                                           rng.uniform(1.0, 1.2),
                                                           rng.uniform(-0.3, 0.3))
            V.append(A * fa * np.exp(-a * fe * R_ang) - C * fc / R_ang ** 6)
            G.append(math.sqrt(4.0 * math.pi / (2 * lam + 1)) * _ylm_matrix(jm, lam, 0))
        j = np.array([x for x in range(jm + 1) for _ in range(2 * x + 1)])
        s.update(E=2.0 * j * (j + 1.0), V=np.array(V), G=np.stack(G), mu=4.0,
                 jx=_jx_blocks(range(jm + 1)), init=np.where(j <= 2)[0])
    elif kind == "rotor_rotor":
        jm = case["jmax"]
        th = rng.standard_normal((len(BIPOLAR), 8))
        th[0, 6] = 5.0
        g = np.stack([np.exp(-(1.25 ** c) * (R_ang - 3.0)) for c in range(7)]
                     + [-(3.0 / R_ang) ** 6])
        scale = np.array([100.0] + [30.0] * (len(BIPOLAR) - 1))
        rad = scale[:, None, None] * g[None]                                    # [12, 8, K]
        st = [(j, m) for j in range(jm + 1) for m in range(-j, j + 1)]
        j1 = np.array([a[0] for a in st for _ in st])
        j2 = np.array([b[0] for _ in st for b in st])
        r, c, v = _jx_blocks(range(jm + 1))
        J = np.zeros((len(st), len(st)))
        J[r, c] = v
        J = np.kron(J, np.eye(len(st))) + np.kron(np.eye(len(st)), J)
        r, c = np.nonzero(J)
        s.update(E=2.0 * j1 * (j1 + 1.0) + 1.5 * j2 * (j2 + 1.0),
                 V=(th[:, :, None] * rad).sum(1), G=_rotor_rotor_G(jm), mu=8.0,
                 jx=(r.astype(np.int32), c.astype(np.int32), J[r, c]),
                 init=np.where((j1 <= 1) & (j2 <= 1))[0], theta=th.reshape(-1),
                 radial=rad.reshape(-1, R_ang.size) * CM,
                 gidx=np.repeat(np.arange(len(BIPOLAR)), 8).astype(np.int32))
    else:
        # a random smooth Hermitian coupling (random Fourier features, decaying e^{-R})
        Q = 8
        if "top" in case:
            js = [j for j in range(case["top"] + 1) for _ in range(2 * j + 1)]
            E = np.concatenate([np.full(2 * j + 1, 11.9 * j * (j + 1.0) + 15.1 * rng.uniform(0, j * j + 1e-9))
                                for j in js])
            s.update(E=E, jx=_jx_blocks(js), mu=3.275, init=np.arange(35))
        else:
            E = np.sort(rng.uniform(0.0, 2000.0, case["n"]))
            s.update(E=E, jx=None, mu=9.0, init=np.arange(16))
        N = E.size
        A, a, C = _wall(rng)
        om, ph = rng.standard_normal(Q), rng.uniform(0.0, 2.0 * math.pi, Q)
        sc = 5.0 if "top" in case else 2.0
        V = np.sqrt(2.0 / Q) * np.cos(om[:, None] * R_ang + ph[:, None]) * sc * np.exp(3.0 - R_ang)
        gen = _gen(seed, 1)
        H = torch.empty((Q, N, N), dtype=torch.complex128, device=DEV)
        for q in range(Q):
            X = torch.view_as_complex(torch.randn((N, N, 2), generator=gen, dtype=torch.float64,
                                                  device=DEV))
            H[q] = (X + X.conj().T) * 0.5
        s.update(V=V, G=H, iso=(A * np.exp(-a * R_ang) - C / R_ang ** 6) * CM)
    s.update(R=R_ang * ANG, E=s["E"] * CM, V=s["V"] * CM, mu=s["mu"] * AMU)
    if not torch.is_tensor(s["G"]):
        s["G"] = torch.as_tensor(s["G"], device=DEV)
    return s


def _tables(s):
    """M [K, N, N] = sum_t V_t G_t (+ iso 1)."""
    G, N, K = s["G"], s["G"].shape[1], s["R"].size
    V = torch.as_tensor(s["V"].T.copy(), device=DEV)                            # [K, T]
    cx = G.is_complex()
    flat = (torch.view_as_real(G) if cx else G).reshape(G.shape[0], -1)
    M = torch.empty((K, flat.shape[1]), dtype=torch.float64, device=DEV)
    for k in range(0, K, 16):
        torch.matmul(V[k:k + 16], flat, out=M[k:k + 16])
    M = torch.view_as_complex(M.view(K, N, N, 2)) if cx else M.view(K, N, N)
    if "iso" in s:
        M.diagonal(dim1=1, dim2=2).real.add_(torch.as_tensor(s["iso"], device=DEV)[:, None])
    return M


def _batch(case, s, seed):
    """Start conditions: a mid-collision population (rk4, adjoint), or whole collisions
    from the grid's end (dp5)."""
    rng = np.random.default_rng([int(seed), 78])
    B = case["B"]
    full = case["kind"] == "dp5"
    if full:
        E = np.exp(rng.uniform(math.log(150.0), math.log(2000.0), B))
        R0 = np.full(B, s["R"][-1])
        b = rng.uniform(0.0, 10.0 * ANG, B)
    else:
        E = rng.uniform(100.0, 2000.0, B)
        R0 = rng.uniform(4.0, 12.0 if "jmax" in case else 19.5, B) * ANG
        b = rng.uniform(0.0, 1.0, B) * np.minimum(12.0 * ANG, 0.9 * R0)
    ch = s["init"][rng.integers(0, s["init"].size, B)].astype(np.int32)
    return dict(init_channel=ch, E_coll=E * CM, b=b, R0=R0)


KEEP = ("P", "a_final", "classical", "t_final", "steps", "rejects", "status")


# ---------------------------------------------------------------- prepare / run

def prepare(case, seed):
    k = case["kind"]
    return {"rk4": _prep_traj, "dp5": _prep_traj, "columns": _prep_columns, "adjoint": _prep_adjoint,
            "build": _prep_build, "xsec": _prep_xsec, "rates": _prep_rates}[k](case, seed)


def run(state):
    return state["run"]()


def _prep_traj(case, seed):
    s = _system(case, seed)
    ctx = mq.Context(0)
    sid = ctx.load_system(R_grid=s["R"], E=s["E"], M=_tables(s), jx=s["jx"], mu=s["mu"],
                          storage=case["storage"], layout=case["layout"])
    torch.cuda.empty_cache()                     # the FP64 input tables are not kept
    bt, B, N = _batch(case, s, seed), case["B"], s["E"].size
    kw = dict(schedule=case["schedule"])
    if case["kind"] == "rk4":
        kw.update(dt=case["dt"], n_steps=case["steps"])
    else:
        kw.update(integrator="dp5", rtol=1e-8, atol=1e-8, max_steps=5000)
    sids, Ns = np.full(B, sid, np.int32), np.full(B, N)

    def go():
        out = ctx.run(sids, Ns, **bt, **kw)
        return {n: out[n] for n in KEEP}
    return {"run": go, "ctx": ctx}


def _columns_inputs(case, seed):
    """A truncated coupling matrix in m-blocks, as sum_t V_t(R_k) g_t(e) over its kept
    elements e: levels of j = 0..jtop ordered by m then level, about
    `partners` coupled levels per level, J_x within a level."""
    rng = np.random.default_rng([int(seed), 79])
    L, P = case["levels"], case["partners"]
    j = rng.permutation(np.arange(L) % (case["jtop"] + 1))
    E = (11.9 * j * (j + 1.0) + rng.uniform(0.0, 400.0, L)) * CM
    a = rng.integers(0, L, L * P // 2)
    c = rng.integers(0, L, L * P // 2)
    lo, hi = np.minimum(a, c), np.maximum(a, c)
    key = np.unique(np.concatenate([lo * L + hi, np.arange(L) * (L + 1)]))
    pa, pb = torch.as_tensor(key // L, device=DEV), torch.as_tensor(key % L, device=DEV)
    jt = torch.as_tensor(j, device=DEV)
    jm = int(j.max())
    idx, n = [], 0
    lev = []
    for m in range(-jm, jm + 1):
        on = np.where(j >= abs(m))[0]
        full = np.full(L, -1, np.int64)
        full[on] = n + np.arange(on.size)
        n += on.size
        idx.append(full)
        lev.append(on)
    pos = torch.as_tensor(np.stack(idx), device=DEV)                            # [2 jm + 1, L]
    rows, cols, src = [], [], []
    pair = torch.arange(pa.numel(), device=DEV)
    for m in range(-jm, jm + 1):
        ok = torch.minimum(jt[pa], jt[pb]) >= abs(m)
        r, q = pos[m + jm][pa[ok]], pos[m + jm][pb[ok]]
        rows.append(r), cols.append(q), src.append(pair[ok])
    r, q, e = torch.cat(rows), torch.cat(cols), torch.cat(src)
    gen = _gen(seed, 2)
    g = torch.randn((2, r.numel()), generator=gen, dtype=torch.float64, device=DEV)
    g = g * (0.5 + 0.5 * torch.rand(pa.numel(), generator=gen, dtype=torch.float64,
                                    device=DEV)[e])
    off = r != q
    rr, qq = torch.cat([r, q[off]]), torch.cat([q, r[off]])
    g = torch.cat([g, g[:, off]], 1).contiguous()
    R = np.exp(np.linspace(math.log(3.0), math.log(30.0), case["K"]))
    V = np.stack([4.0 * np.exp(-1.3 * (R - 5.0)), -2.0 * (5.0 / R) ** 6]) * CM
    U = (200.0 * np.exp(-1.6 * (R - 5.0)) - 100.0 * (5.0 / R) ** 6) * CM
    lv = np.concatenate(lev)
    mm = np.concatenate([np.full(x.size, m - jm) for m, x in enumerate(lev)])
    ph = np.stack(idx)
    jr, jc, jv = [], [], []
    for m in range(-jm, jm):
        both = lev[m + jm] if m < 0 else lev[m + 1 + jm]       # levels with |m|, |m + 1| <= j
        both = both[(j[both] >= abs(m)) & (j[both] >= abs(m + 1))]
        x, y = ph[m + jm][both], ph[m + 1 + jm][both]
        v = 0.5 * np.sqrt(j[both] * (j[both] + 1.0) - m * (m + 1.0))
        jr += [x, y]
        jc += [y, x]
        jv += [v, v]
    cat = lambda z, t: np.concatenate(z).astype(t) if z else np.zeros(0, t)
    C, W = case["cols"], case["paths"]
    path = np.repeat(np.arange(W), C)
    bt = dict(E_coll=rng.uniform(200.0, 900.0, W)[path] * CM, b=rng.uniform(0.0, 3.0, W)[path],
              R0=rng.uniform(7.0, 9.0, W)[path],
              init_channel=(np.argsort(np.abs(mm), kind="stable")[:128][np.tile(np.arange(C), W) % n]
                            ).astype(np.int32))
    return dict(R=R, E=E[lv], V=V, U=U, g=g, rows=rr, cols=qq, N=n, mu=1.8 * AMU, batch=bt,
                jx=(cat(jr, np.int32), cat(jc, np.int32), cat(jv, np.float64)), B=C * W)


def _prep_columns(case, seed):
    s = _columns_inputs(case, seed)
    V = torch.as_tensor(s["V"], device=DEV)
    ctx = mq.Context(0)
    sid = ctx.load_system_coo(R_grid=s["R"], E=s["E"], rows=s["rows"].int(), cols=s["cols"].int(),
                              values=V.T.contiguous() @ s["g"], mu=s["mu"], jx=s["jx"],
                              storage=case["storage"])
    ctx.set_driver(sid, s["U"])
    B, N, bt = s["B"], s["N"], s["batch"]
    del s
    torch.cuda.empty_cache()
    sids, Ns, steps = np.full(B, sid, np.int32), np.full(B, N), case["steps"]

    def go():
        out = ctx.run(sids, Ns, dynamics="at", dt=10.0, n_steps=steps, **bt)
        return {n: out[n] for n in KEEP}
    return {"run": go, "ctx": ctx}


def _adjoint_weights(case, seed, B, N):
    return torch.rand((B, N), generator=_gen(seed, 3), dtype=torch.float64, device=DEV)


def _prep_adjoint(case, seed):
    s = _system(case, seed)
    ctx = mq.Context(0)
    sid = ctx.load_system(R_grid=s["R"], E=s["E"], M=_tables(s), jx=s["jx"], mu=s["mu"],
                          storage="R64", layout=case["layout"])
    ctx.set_params(sid, s["radial"], s["gidx"], s["G"].cpu().numpy())
    bt, N = _batch(case, s, seed), s["E"].size
    bt.update(dt=case["dt"], n_steps=np.full(case["B"], case["steps"]))
    w = _adjoint_weights(case, seed, case["B"], N)
    th0 = torch.as_tensor(s["theta"], device=DEV)

    def go():
        theta = th0.clone().requires_grad_(True)
        P = mq.propagate(theta, ctx, sid, N, bt)
        (P * w).sum().backward()
        return {"P": P.detach(), "grad": theta.grad}
    return {"run": go, "ctx": ctx}


class _NS:
    pass


def _top_states(j):
    """Asymmetric-top states of one j over k = -j..j (rigid rotor, H2O constants)."""
    A, B, C = 27.88, 14.51, 9.28
    k = np.arange(-j, j + 1)
    H = np.diag(0.5 * (B + C) * (j * (j + 1) - k * k) + A * k * k).astype(float)
    for i in range(2 * j - 1):
        x = 0.25 * (B - C) * math.sqrt((j * (j + 1) - k[i] * (k[i] + 1))
                                       * (j * (j + 1) - (k[i] + 1) * (k[i] + 2)))
        H[i, i + 2] = H[i + 2, i] = x
    return np.linalg.eigh(H)[1].T


def _build_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 80])
    jm = case["j1max"]
    b, rj = [], []
    for j in range(jm + 1):
        v = _top_states(j)
        for q in range(2 * j + 1):
            row = np.zeros(2 * jm + 1)
            row[:2 * j + 1] = v[q]
            b.append(row)
            rj.append(j)
    lv = [(r, j2, j) for r in range(len(rj)) for j2 in range(0, case["j2max"] + 1, 2)
          for j in range(abs(rj[r] - j2), rj[r] + j2 + 1)]
    jt = max(x[2] for x in lv)
    ch = [(m, *x) for m in range(-jt, jt + 1) for x in lv if x[2] >= abs(m)]
    basis, exp = _NS(), _NS()
    col = lambda i: np.array([c[i] for c in ch], np.int32)
    basis.m, basis.rot1, basis.j2, basis.j = col(0), col(1), col(2), col(3)
    basis.rot1_j, basis.b = np.array(rj, np.int32), np.array(b)
    terms = [(l1, mu, l2, l) for l1 in range(10) for mu in range(0, min(l1, 6) + 1, 2)
             for l2 in range(0, 7, 2) for l in range(abs(l1 - l2), min(l1 + l2, 11) + 1)
             if mu or (l1 + l2 + l) % 2 == 0]
    pick = np.sort(np.concatenate([[0], 1 + rng.permutation(len(terms) - 1)[:case["terms"] - 1]]))
    t = np.array([terms[i] for i in pick], np.int32)
    exp.lam1, exp.mu1, exp.lam2, exp.lam = (np.ascontiguousarray(t[:, i]) for i in range(4))
    R = np.exp(np.linspace(math.log(3.0), math.log(30.0), case["K"]))
    sc = 1.0 / (1.0 + t[:, 0] + t[:, 2])
    exp.v = CM * ((60.0 * sc * rng.standard_normal(len(t)))[:, None]
                  * np.exp(-(1.2 + 0.6 * rng.random(len(t)))[:, None] * (R - 5.0))
                  - (20.0 * sc * rng.standard_normal(len(t)))[:, None] * (5.0 / R) ** 6)
    return basis, exp


def _prep_build(case, seed):
    basis, exp = _build_inputs(case, seed)
    ctx = mq.Context(0)
    return {"run": lambda: ctx.build_couplings(basis, exp), "ctx": ctx}


def _xsec_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 81])
    js = [j for j in range(case["top"] + 1) for _ in range(2 * j + 1)]
    lev = np.concatenate([np.full(2 * j + 1, i) for i, j in enumerate(js)]).astype(np.int32)
    N, B = lev.size, case["B"]
    P = torch.rand((B, N), generator=_gen(seed, 4), dtype=torch.float64, device=DEV) ** 8
    P /= P.sum(1, keepdim=True)
    init = rng.integers(0, N, B)
    return P, rng.uniform(0.0, 22.0, B), lev[init], lev, len(js)


def _prep_xsec(case, seed):
    P, b, il, lev, nl = _xsec_inputs(case, seed)
    ctx = mq.Context(0)
    return {"run": lambda: ctx.cross_sections(P, b, il, lev, nl, 22.0), "ctx": ctx}


def _rates_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 82])
    L, nE, nT = case["L"], case["nE"], case["nT"]
    U = np.exp(np.linspace(math.log(20.0), math.log(12000.0), nE)) * rng.uniform(0.9, 1.1, nE) * CM
    E = np.sort(rng.uniform(0.0, 4000.0, L)) * CM
    g = (2.0 * rng.integers(0, 20, L) + 1.0) * (2.0 * rng.integers(0, 8, L) + 1.0)
    beta = np.linspace(10.0, 2000.0, nT) * 0.695034800 * CM
    x = torch.rand((nE, L, L), generator=_gen(seed, 5), dtype=torch.float64, device=DEV)
    sym = (x + x.transpose(1, 2)) * 10.0
    d = lambda a: torch.as_tensor(a, device=DEV)
    return d(np.sort(U)), d(E), d(g), sym, 1.8 * AMU, d(beta)


def _prep_rates(case, seed):
    U, E, g, sym, mu, beta = _rates_inputs(case, seed)
    ctx = mq.Context(0)
    nE, L, nT = case["nE"], case["L"], case["nT"]

    def go():
        k = torch.empty((nT, L, L), dtype=torch.float64, device=DEV)
        code = mq.lib().mqct_rate_coefficients(ctx.h, mq.MEM_DEVICE, nE, L, U.data_ptr(),
                                               E.data_ptr(), g.data_ptr(), sym.data_ptr(), mu, nT,
                                               beta.data_ptr(), k.data_ptr())
        if code != mq.OK:
            raise mq.MQCTError(code, mq.lib().mqct_last_error(ctx.h).decode())
        return k
    return {"run": go, "ctx": ctx}


# ---------------------------------------------------------------- what a pass cannot do without

def _nchan(case):
    if "jmax" in case:
        n = (case["jmax"] + 1) ** 2
        return n * n if case.get("system", "rotor_rotor") == "rotor_rotor" else n
    return sum((2 * j + 1) ** 2 for j in range(case["top"] + 1)) if "top" in case else case["n"]


def work(case):
    k = case["kind"]
    if k in ("rk4", "dp5", "adjoint"):
        N, B, K = _nchan(case), case["B"], case["K"]
        cx = case.get("storage", "R64") in ("C64", "C128")
        item = ITEM[case.get("storage", "R64")]
        el = N * N * (1.0 if cx else 0.1)        # the real systems' selection rules leave ~10 %
        if k == "rk4":
            evals, knots = 4 * case["steps"], min(K, 2 * B)
        else:
            evals, knots = (600, K) if k == "dp5" else (4 * case["steps"], min(K, int(0.5 * K)))
        flops = B * evals * el * (32.0 if cx else 16.0) * (3.5 if k == "adjoint" else 1.0)
        out = B * N * 24.0 if k != "adjoint" else B * N * 16.0
        return {"bytes": 2.0 * knots * el * item + out, "flops": flops}
    if k == "columns":
        N = case["levels"] * (case["jtop"] + 1)
        cols = case["cols"] * case["paths"]
        nnz = case["levels"] * case["partners"] * (case["jtop"] / 1.5 + 1.0) + N
        item = ITEM[case["storage"]]
        return {"bytes": 4.0 * nnz * item + N * cols * 24.0,
                "flops": nnz * cols * 4.0 * 4 * case["steps"]}
    if k == "build":
        b, e = _build_inputs(case, 0)
        N = b.m.size
        nz = sum(float(np.sum(b.m == m)) ** 2 for m in np.unique(b.m))
        return {"bytes": 8.0 * case["K"] * N * N, "flops": 2.0 * nz * case["terms"] * (case["K"] + 1)}
    if k == "xsec":
        N = sum((2 * j + 1) ** 2 for j in range(case["top"] + 1))
        return {"bytes": 8.0 * case["B"] * N, "flops": 2.0 * case["B"] * N}
    LL = float(case["L"]) ** 2
    return {"bytes": 8.0 * LL * (case["nE"] + case["nT"]), "flops": LL * case["nT"] * case["nE"] * 40.0}


# ---------------------------------------------------------------- the same in 64 bits

def exact(case, seed):
    k = case["kind"]
    return {"rk4": _exact_rk4, "dp5": _exact_dp5, "columns": _exact_columns,
            "adjoint": _exact_adjoint, "build": _exact_build, "xsec": _exact_xsec,
            "rates": _exact_rates}[k](case, seed)


def _curv(R, y):
    """Natural-spline second derivatives of y [T, K]."""
    K = R.size
    h = np.diff(R)
    A = np.eye(K)
    D = np.zeros((K, K))
    for k in range(1, K - 1):
        A[k, k - 1:k + 2] = [h[k - 1] / 6.0, (h[k - 1] + h[k]) / 3.0, h[k] / 6.0]
        D[k, k - 1:k + 2] = [1.0 / h[k - 1], -1.0 / h[k - 1] - 1.0 / h[k], 1.0 / h[k]]
    return np.linalg.solve(A, D @ np.asarray(y).T).T


class _Spline:
    """Value and slope of the functions y [T, K] at R [B] (held past the last knot,
    continued linearly below the first)."""

    def __init__(self, R, y):
        d = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=DEV)
        self.x, self.y, self.c = d(R), d(np.asarray(y).T), d(_curv(R, y).T)      # [K, T]

    def __call__(self, R):
        x = self.x
        K = x.numel()
        k = (torch.searchsorted(x, R.detach().contiguous(), right=True) - 1).clamp(0, K - 2)
        h = x[k + 1] - x[k]
        below, above = R < x[0], R > x[K - 1]
        Rc = torch.where(below, x[0], torch.where(above, x[K - 1], R))
        A = (x[k + 1] - Rc) / h
        Bq = 1.0 - A
        w = [A, Bq, (A ** 3 - A) * h * h / 6.0, (Bq ** 3 - Bq) * h * h / 6.0]
        d = [-1.0 / h, 1.0 / h, -(3.0 * A * A - 1.0) * h / 6.0, (3.0 * Bq * Bq - 1.0) * h / 6.0]
        y = [self.y[k], self.y[k + 1], self.c[k], self.c[k + 1]]
        v = sum(a[:, None] * b for a, b in zip(w, y))
        s = sum(a[:, None] * b for a, b in zip(d, y))
        s = torch.where(above[:, None], torch.zeros_like(s), s)
        v = torch.where(below[:, None], v + (R - x[0])[:, None] * s, v)
        return v, s


def _rhs(s):
    """da/dt and d(R, Phi, P_R, P_Phi)/dt of a batch, a [B, N] complex, y [B, 4]."""
    G, mu = s["G"], s["mu"]
    T, N = G.shape[0], G.shape[1]
    E = torch.as_tensor(s["E"], device=DEV)
    iso = "iso" in s
    sp = _Spline(s["R"], np.concatenate([s["V"], s["iso"][None]]) if iso else s["V"])
    Gt = G.transpose(1, 2).permute(1, 0, 2).reshape(N, T * N).contiguous()      # [m, (t, n)]
    J = None
    if s["jx"] is not None and len(s["jx"][0]):
        J = torch.zeros((N, N), dtype=torch.float64, device=DEV)
        J[torch.as_tensor(s["jx"][0]).long(), torch.as_tensor(s["jx"][1]).long()] = \
            torch.as_tensor(s["jx"][2], device=DEV)
    if not Gt.is_complex() and J is not None:
        Gt, J = torch.cat([Gt, J], 1), None
    real = not Gt.is_complex()

    def mm(c, A):
        if A.is_complex():
            return c @ A
        return torch.complex(c.real @ A, c.imag @ A)

    def f(t, a, y):
        V, D = sp(y[:, 0])
        e = torch.exp(1j * E[None] * t[:, None])
        c = e.conj() * a
        Y = mm(c, Gt)
        x = Y[:, T * N:] if real and Y.shape[1] > T * N else (mm(c, J) if J is not None else torch.zeros_like(c))
        Y = Y[:, :T * N].reshape(-1, T, N)
        u, v = (V[:, :T, None] * Y).sum(1), (D[:, :T, None] * Y).sum(1)
        if iso:
            u, v = u + V[:, T:] * c, v + D[:, T:] * c
        R, P, L = y[:, 0], y[:, 2], y[:, 3]
        om = L / (mu * R * R)
        force = (c.conj() * v).sum(1).real
        torque = (x.conj() * u).sum(1).imag
        da = -1j * e * (u + om[:, None] * x)
        return da, torch.stack([P / mu, om, -force + L * L / (mu * R ** 3), 2.0 * torque], 1)
    return f


def _start(s, bt):
    d = lambda a: torch.as_tensor(a, device=DEV, dtype=torch.float64)
    E, b, R0 = d(bt["E_coll"]), d(bt["b"]), d(bt["R0"])
    L = b * torch.sqrt(2.0 * s["mu"] * E)
    P = -torch.sqrt(2.0 * s["mu"] * E - L * L / (R0 * R0))
    y = torch.stack([R0, torch.zeros_like(R0), P, L], 1)
    a = torch.zeros((R0.numel(), s["E"].size), dtype=torch.complex128, device=DEV)
    a[torch.arange(R0.numel()), torch.as_tensor(bt["init_channel"]).long()] = 1.0
    return a, y


def _rk4_step(f, t, h, a, y):
    ka, ky = f(t, a, y)
    sa, sy = ka, ky
    for c, w in ((0.5, 2.0), (0.5, 2.0), (1.0, 1.0)):
        ka, ky = f(t + c * h, a + c * h * ka, y + c * h * ky)
        sa, sy = sa + w * ka, sy + w * ky
    return a + h / 6.0 * sa, y + h / 6.0 * sy


def _result(a, y, t):
    half = torch.full_like(t, 0.5 * math.pi)
    cl = torch.stack([y[:, 0], half, y[:, 1], y[:, 2], torch.zeros_like(t), y[:, 3]], 1)
    return {"P": (a.abs() ** 2).reshape(-1), "a_final": a.reshape(-1), "classical": cl, "t_final": t,
            "steps": None, "rejects": None, "status": None}


def _exact_rk4(case, seed):
    s = _system(case, seed)
    bt = _batch(case, s, seed)
    f, (a, y), h = _rhs(s), _start(s, bt), case["dt"]
    t = torch.zeros(case["B"], dtype=torch.float64, device=DEV)
    for j in range(case["steps"]):
        a, y = _rk4_step(f, t + j * h, h, a, y)
    return _result(a, y, t + case["steps"] * h)


DP_C = [0.0, 1 / 5, 3 / 10, 4 / 5, 8 / 9, 1.0, 1.0]
DP_A = [[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
        [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
        [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
        [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]]
DP_E = [71 / 57600, 0.0, -71 / 16695, 71 / 1920, -17253 / 339200, 22 / 525, -1 / 40]


def _exact_dp5(case, seed):
    """Dormand & Prince 5(4) with the framework's documented norm, controller and
    starting step (Hairer, Norsett & Wanner), every trajectory with its own step."""
    s = _system(case, seed)
    f, (a, y) = _rhs(s), _start(s, _batch(case, s, seed))
    tol = 1e-8
    B, N = a.shape
    nc = 2.0 * N + 6.0
    const = torch.tensor([0.5 * math.pi, 0.0], device=DEV, dtype=torch.float64).expand(B, 2)
    flat = lambda p, q: torch.cat([torch.view_as_real(p.contiguous()).reshape(B, -1), q], 1)
    norm = lambda v, sc, extra=0.0: torch.sqrt((((v / sc) ** 2).sum(1) + extra) / nc)
    t = torch.zeros(B, dtype=torch.float64, device=DEV)
    fa, fy = f(t, a, y)
    sc = tol + tol * flat(a, y).abs()
    d0 = norm(flat(a, y), sc, ((const / (tol + tol * const)) ** 2).sum(1))
    d1 = norm(flat(fa, fy), sc)
    h0 = torch.where((d0 < 1e-5) | (d1 < 1e-5), torch.full_like(d0, 1e-6), 0.01 * d0 / d1)
    ga, gy = f(t + h0, a + h0[:, None] * fa, y + h0[:, None] * fy)
    dm = torch.maximum(d1, norm(flat(ga - fa, gy - fy), sc) / h0)
    h = torch.minimum(100.0 * h0, torch.where(dm <= 1e-15, torch.clamp(h0 * 1e-3, min=1e-6),
                                              (0.01 / dm) ** 0.2))
    R_exit = y[:, 0].clone()
    live = torch.ones(B, dtype=torch.bool, device=DEV)
    rej = torch.zeros_like(live)
    for _ in range(4000):
        ka, ky = [fa], [fy]
        for q in range(1, 7):
            sa = a + sum(h[:, None] * c * k for c, k in zip(DP_A[q], ka))
            sy = y + sum(h[:, None] * c * k for c, k in zip(DP_A[q], ky))
            p, r = f(t + DP_C[q] * h, sa, sy)
            ka.append(p), ky.append(r)
        ea = sum(c * k for c, k in zip(DP_E, ka)) * h[:, None]
        ey = sum(c * k for c, k in zip(DP_E, ky)) * h[:, None]
        en = norm(flat(ea, ey), tol + tol * torch.maximum(flat(a, y).abs(), flat(sa, sy).abs()))
        ok = live & (en <= 1.0)
        t = torch.where(ok, t + h, t)
        a, y = torch.where(ok[:, None], sa, a), torch.where(ok[:, None], sy, y)
        fa, fy = torch.where(ok[:, None], ka[6], fa), torch.where(ok[:, None], ky[6], fy)
        out = ok & (y[:, 0] >= R_exit) & (y[:, 2] > 0.0)
        fac = torch.clamp(0.9 * en ** -0.2, 0.2, 5.0)
        fac = torch.where(en <= 1.0, torch.where(rej, fac.clamp(max=1.0), fac), fac)
        rej = torch.where(live, en > 1.0, rej)
        live = live & ~out
        h = torch.where(live, h * fac, h)
        if not bool(live.any()):
            break
    return _result(a, y, t)


def _exact_columns(case, seed):
    s = _columns_inputs(case, seed)
    bt, N, C, W = s["batch"], s["N"], case["cols"], case["paths"]
    dev = lambda a: torch.as_tensor(a, device=DEV)
    order = torch.argsort(s["rows"].long() * N + s["cols"].long())
    rows, cols, g = s["rows"][order], s["cols"][order], s["g"][:, order]
    crow = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    crow[1:] = torch.bincount(rows, minlength=N).cumsum(0)
    jr, jc, jv = (dev(x) for x in s["jx"])
    E = dev(s["E"])[:, None]
    spV, spU, mu, h = _Spline(s["R"], s["V"]), _Spline(s["R"], s["U"][None]), s["mu"], 10.0
    outs = []
    for w in range(W):
        sel = {k: v[w * C:(w + 1) * C] for k, v in bt.items()}
        y = _start(dict(mu=mu, E=np.zeros(1)), {**{k: v[:1] for k, v in sel.items()},
                                                "init_channel": np.zeros(1, np.int64)})[1]
        a = torch.zeros((N, C), dtype=torch.complex128, device=DEV)
        a[dev(sel["init_channel"]).long(), torch.arange(C, device=DEV)] = 1.0

        def f(t, a, y):
            R, P, L = y[0, 0], y[0, 2], y[0, 3]
            val = (spV(y[:, 0])[0].T * g).sum(0)
            A = torch.sparse_csr_tensor(crow, cols, val, (N, N))
            e = torch.exp(1j * E * t)
            c = torch.view_as_real((e.conj() * a).contiguous()).reshape(N, 2 * C)
            u = torch.view_as_complex((A @ c).reshape(N, C, 2))
            x = torch.zeros_like(a)
            if jr.numel():
                x.index_add_(0, jr, jv[:, None] * a[jc.long()])
            om = L / (mu * R * R)
            dU = spU(y[:, 0])[1][0, 0]
            ky = torch.stack([P / mu, om, -dU + L * L / (mu * R ** 3), 0.0 * P])[None]
            return -1j * (e * u + om * x), ky
        for j in range(case["steps"]):
            a, y = _rk4_step(f, j * h, h, a, y)
        outs.append(_result(a.T.contiguous(), y.expand(C, 4).contiguous(),
                            torch.full((C,), case["steps"] * h, dtype=torch.float64, device=DEV)))
    return {k: (None if outs[0][k] is None else torch.cat([o[k] for o in outs])) for k in outs[0]}


def _exact_adjoint(case, seed):
    """The gradient of the same RK4 map by automatic differentiation, step by step."""
    s = _system(case, seed)
    bt, N, h = _batch(case, s, seed), s["E"].size, case["dt"]
    w = _adjoint_weights(case, seed, case["B"], N)
    T = s["G"].shape[0]
    rad = torch.as_tensor(s["radial"], device=DEV).reshape(T, 8, -1)
    cur = torch.as_tensor(_curv(s["R"], s["radial"]), device=DEV).reshape(T, 8, -1)
    f = _rhs(s)
    sp = next(c.cell_contents for c in f.__closure__ if isinstance(c.cell_contents, _Spline))
    t0 = torch.zeros(case["B"], dtype=torch.float64, device=DEV)
    a, y = _start(s, bt)
    states = []
    with torch.no_grad():
        for j in range(case["steps"]):
            states.append((a, y))
            a, y = _rk4_step(f, t0 + j * h, h, a, y)
    P = (a.abs() ** 2).reshape(case["B"], N)
    ga, gy = 2.0 * w * a, torch.zeros_like(y)
    grad = torch.zeros(s["theta"].size, dtype=torch.float64, device=DEV)
    for j in reversed(range(case["steps"])):
        a, y = (v.clone().requires_grad_(True) for v in states[j])
        th = torch.as_tensor(s["theta"], device=DEV).requires_grad_(True)
        sp.y = (th.reshape(T, 8, 1) * rad).sum(1).T
        sp.c = (th.reshape(T, 8, 1) * cur).sum(1).T
        a1, y1 = _rk4_step(f, t0 + j * h, h, a, y)
        ga, gy, gt = torch.autograd.grad([a1, y1], [a, y, th], [ga, gy])
        grad += gt
    return {"P": P, "grad": grad}


def _cg_table(jmax, l, mu, m):
    """<ja m l mu | jb m + mu> for ja, jb <= jmax as a [ja, jb] array."""
    out = np.zeros((jmax + 1, jmax + 1))
    for ja in range(abs(m), jmax + 1):
        for jb in range(max(abs(ja - l), abs(m + mu)), min(jmax, ja + l) + 1):
            out[ja, jb] = _cg(ja, m, l, mu, jb)
    return out


@functools.lru_cache(None)
def _cg1(j1, m1, j2, m2, J):
    return _cg(j1, m1, j2, m2, J)


def _exact_build(case, seed):
    """Eq. 17 by its Clebsch-Gordan sums: the reduced factor of every (j1, j2, j) pair
    from one projection that does not vanish, then the Wigner-Eckart theorem in m."""
    basis, exp = _build_inputs(case, seed)
    T, N = len(exp.lam1), basis.m.size
    j1 = basis.rot1_j[basis.rot1]
    lv, inv = np.unique(np.stack([j1, basis.j2, basis.j], 1), axis=0, return_inverse=True)
    inv = inv.reshape(-1)
    nJ, n1 = len(lv), basis.rot1_j.size
    jt = int(basis.j.max())
    dev = lambda a: torch.as_tensor(a, device=DEV)
    M = torch.zeros((exp.v.shape[1], N, N), dtype=torch.float64, device=DEV)
    F = np.zeros((T, nJ, nJ))
    for (l1, l2, l) in {(int(exp.lam1[t]), int(exp.lam2[t]), int(exp.lam[t])) for t in range(T)}:
        ninej = np.zeros((nJ, nJ))
        for A in range(nJ):
            for B in range(nJ):
                a, b, c = (int(x) for x in lv[A])
                g, h, i = (int(x) for x in lv[B])
                if not (abs(a - l1) <= g <= a + l1 and abs(b - l2) <= h <= b + l2
                        and abs(c - l) <= i <= c + l) or (b + l2 + h) % 2:
                    continue
                ninej[B, A] = _reduced(a, b, c, l1, l2, l, g, h, i)
        for t in range(T):
            if (exp.lam1[t], exp.lam2[t], exp.lam[t]) == (l1, l2, l):
                F[t] = ninej
    Kr = np.zeros((T, n1, n1))
    for t in range(T):
        l1, mu = int(exp.lam1[t]), int(exp.mu1[t])
        sg = (-1.0) ** (l1 + mu + int(exp.lam2[t]) + int(exp.lam[t]))
        for ra in range(n1):
            ja = int(basis.rot1_j[ra])
            for rb in range(n1):
                jb = int(basis.rot1_j[rb])
                x = 0.0
                for ka in range(-ja, ja + 1):
                    for kb, q, fct in ((ka + mu, mu, 1.0), (ka - mu, -mu, sg)):
                        if abs(kb) <= jb:
                            x += fct * basis.b[rb, kb + jb] * basis.b[ra, ka + ja] * \
                                _cg1(ja, ka, l1, q, jb)
                Kr[t, rb, ra] = x
    v, Fd, Kd = dev(exp.v), dev(F), dev(Kr)
    J, r, jd = dev(inv), dev(basis.rot1).long(), dev(basis.j).long()
    for m in range(-jt, jt + 1):
        idx = dev(np.where(basis.m == m)[0])
        C = {l: dev(_cg_table(jt, l, 0, m)) for l in set(int(x) for x in exp.lam)}
        acc = torch.zeros((exp.v.shape[1], idx.numel(), idx.numel()), dtype=torch.float64, device=DEV)
        for t in range(T):
            Gt = Fd[t][J[idx]][:, J[idx]] * Kd[t][r[idx]][:, r[idx]] * \
                C[int(exp.lam[t])].T[jd[idx]][:, jd[idx]]
            acc += v[t][:, None, None] * Gt
        M[:, idx[:, None], idx[None, :]] = acc
    return {"M": M}


@functools.lru_cache(None)
def _reduced(a, b, c, l1, l2, l, g, h, i):
    """sqrt factors x C(b 0 l2 0|h 0) x 9j{a b c; l1 l2 l; g h i}, the 9j from the
    recoupling sum of five Clebsch-Gordan coefficients at a projection m with
    C(c m l 0 | i m) not zero."""
    best = max(range(0, min(c, i) + 1), key=lambda m: abs(_cg1(c, m, l, 0, i)))
    den = _cg1(c, best, l, 0, i)
    if abs(den) < 1e-12:
        return 0.0
    s = 0.0
    for m1 in range(-a, a + 1):
        m2 = best - m1
        if abs(m2) > b:
            continue
        x = _cg1(a, m1, b, m2, c)
        for eta in range(-min(l1, l2), min(l1, l2) + 1):
            if abs(m1 + eta) <= g and abs(m2 - eta) <= h:
                s += x * _cg1(l1, eta, l2, -eta, l) * _cg1(a, m1, l1, eta, g) * \
                    _cg1(b, m2, l2, -eta, h) * _cg1(g, m1 + eta, h, m2 - eta, i)
    # s = sqrt((2c+1)(2l+1)(2g+1)(2h+1)) 9j C(c m l 0|i m)
    root = math.sqrt((2 * a + 1) * (2 * b + 1) * (2 * l1 + 1) * (2 * l2 + 1)
                     / ((2.0 * g + 1) * (2 * h + 1)))
    return root / (4.0 * math.pi) * _cg1(b, 0, l2, 0, h) * s / den


def _exact_xsec(case, seed):
    P, b, il, lev, nl = _xsec_inputs(case, seed)
    A = torch.zeros((P.shape[1], nl), dtype=torch.float64, device=DEV)
    A[torch.arange(P.shape[1]), torch.as_tensor(lev).long()] = 1.0
    on = torch.nn.functional.one_hot(torch.as_tensor(il, device=DEV).long(), nl).double()
    cnt = on.sum(0)
    s = (on * torch.as_tensor(b, device=DEV)[:, None]).T @ (P @ A)
    return torch.where(cnt[:, None] > 0, 2.0 * math.pi * 22.0 / cnt.clamp(min=1.0)[:, None] * s,
                       torch.zeros_like(s))


def _exact_rates(case, seed):
    """16-point Gauss-Legendre on pieces of 2 beta, from the threshold to 60 beta past it."""
    U, E, g, sym, mu, beta = _rates_inputs(case, seed)
    nE, L, nT = case["nE"], case["L"], case["nT"]
    Un = U.cpu().numpy()
    S = torch.as_tensor(_curv(Un, np.eye(nE)).T.copy(), device=DEV)              # [K, basis]
    y = sym.reshape(nE, -1)
    c = S @ y
    i, f = torch.meshgrid(torch.arange(L, device=DEV), torch.arange(L, device=DEV), indexing="ij")
    i, f = i.reshape(-1), f.reshape(-1)
    dE = E[f] - E[i]
    th = dE.abs() * 0.5
    gx, gw = np.polynomial.legendre.leggauss(16)
    out = torch.empty((nT, L * L), dtype=torch.float64, device=DEV)
    for t in range(nT):
        b = float(beta[t])
        tot = torch.zeros_like(th)
        for e in range(nE + 1):
            lo = th if e == 0 else torch.clamp(th, min=float(Un[e - 1]))
            hi = torch.clamp(th, min=float(Un[e])) if e < nE else lo + 60.0 * b
            hi = torch.minimum(hi, torch.maximum(lo, th + 60.0 * b))
            n = max(1, int(math.ceil(0.5 * float((hi - lo).max()) / b)))
            w = (hi - lo) / n
            for q in range(n):
                for x, wt in zip(gx, gw):
                    u = lo + (q + 0.5 + 0.5 * x) * w
                    if e == 0:
                        s = y[0] * (u - th) / torch.where(Un[0] - th > 0, Un[0] - th,
                                                          torch.ones_like(th))
                    elif e == nE:
                        s = y[nE - 1]
                    else:
                        h = Un[e] - Un[e - 1]
                        A = (Un[e] - u) / h
                        Bq = 1.0 - A
                        s = A * y[e - 1] + Bq * y[e] + ((A ** 3 - A) * c[e - 1]
                                                        + (Bq ** 3 - Bq) * c[e]) * h * h / 6.0
                    tot += 0.5 * wt * w * s * u * torch.exp(-(u - th) / b)
        out[t] = math.sqrt(8.0 / (math.pi * mu)) * b ** -1.5 * torch.exp(-(th + 0.5 * dE) / b) * tot / g[i]
    return out.reshape(nT, L, L)
