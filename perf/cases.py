"""Performance cases: the work that programs built on this library have it do.

Four kinds of program, each through the package's public entry points:

  expmv    exp(-i H dt) applied to a vector on a set the program holds in
           device memory (Model.expmv, Model.expmv_static)
  run      a trajectory: a Sim from its initial state, n time steps, the
           observation records (Sim, Sim.step, Sim.series), where the case
           asks for it also the final state (Sim.state)
  rerun    the same on a Sim that the program keeps and sets back to the
           initial state (Sim.set_state): one trajectory per disorder draw or
           excitation on one handle
  adjoint  the autocorrelation of a trajectory and the gradient of a loss of
           it with respect to the model parameters (AutocorrFn, backward)

Shapes, thresholds and step counts are those of `workloads` and the bench
(shorter runs of them).  The seed draws the site energies (static disorder)
and the amplitudes given to expmv.

A trajectory's results are its records: norm, energy, autocorrelation,
discarded weight, spectral bounds, populations and set sizes of every step.
The set lives in an order that differs between runs, so final states are
returned sorted by key, and only where reading and sorting them is small
beside the run (a program reads them for a checkpoint, not per pass).
"""
import math

import numpy as np
import torch

import paper_2603_07341_amd as P
import workloads as WL

STATE = "norm2 energy mass_step E_min E_max".split()


# ---- cases -------------------------------------------------------------------
def _lat(dims, periodic, cutoff, omega, g, J):
    return {"dims": dims, "periodic": periodic, "cutoff": cutoff,
            "omega": omega, "g": g, "J": J}


RING4 = _lat("4", True, "4", "1", "1", -0.5)
RING16 = _lat("16", True, "12", "1", "1.2", -1.0)
RING12 = _lat("12", True, "10", "1", "1", -1.0)
SQ6X6 = _lat("6x6", True, "15", "1", "1", -0.8)
CUBE4 = _lat("4x4x4", True, "15,31", "1,0.2", "1,0.5", -0.5)


def _run(kind, lat, **over):
    c = dict(lat, kind=kind, sigma=0.1, n_real=1, init="bloch", dt=0.01, k=4,
             k_init=4, theta=1e-8, precision=64, max_states=0, q_nom=0,
             krylov=0, taylor=0, state=False)
    c.update(over)
    return c


def listed():
    return [
        # the smallest call: the whole space of the 4-site ring, where only
        # latency and launches count
        dict(RING4, name="expmv_ring4", kind="expmv", sigma=0.1, dt=0.01,
             n_max=16, keep=1.0, static=False),
        # a serving loop that may not allocate, at a set near the static work
        # memory's usual fill; rows missing at random leave ragged columns
        dict(RING16, name="expmv_static_ring16", kind="expmv", sigma=0.1,
             dt=0.01, n_max=4, keep=0.93, static=True),
        # an ordinary large set given by the caller
        dict(RING16, name="expmv_ring16", kind="expmv", sigma=0.1, dt=0.01,
             n_max=6, keep=0.97, static=False),
        # the smallest trajectory at its own length; its final state is read
        _run("run", RING4, name="ring4", init="local", theta=1e-10, steps=500,
             state=True),
        # the first part of an absorption run: sets of 10^2 to 4 10^5 states
        _run("run", RING16, name="ring16_start", steps=60),
        # the benchmark's growth to its timed window (10^7 states), on a
        # handle that is kept
        _run("rerun", RING16, name="ring16_grown", steps=160),
        # the same in complex64
        _run("rerun", RING16, name="ring16_c64", precision=32, steps=140),
        # disorder average: 64 realizations in one set, complex64
        _run("rerun", SQ6X6, name="sq6x6_batch64", sigma=0.2, n_real=64,
             dt=0.02, k=2, k_init=2, theta=1e-7, precision=32, steps=20),
        # two modes per site on a 3D lattice under a state cap, ten-word keys,
        # complex64; the cap binds from about step 30 on
        _run("run", CUBE4, name="cube4_capped", sigma=0.05, init="local", k=2,
             k_init=2, theta=1e-7, precision=32, max_states=500_000,
             steps=48),
        # the paper's 1D run at g = 4 with fixed-size truncation (long series
        # of 20 terms, three-word keys, sets past the last-level cache)
        _run("rerun", _lat("25", False, "63", "1", "4", 1.0),
             name="chain25_qnom", sigma=0.05, init="local", dt=0.05, k=2,
             k_init=10, theta=0.0, q_nom=4_000_000, steps=24),
        # the paper's 3D aggregate with its own propagator, the truncated
        # Taylor series
        _run("rerun", _lat("3x3x3", False, "15", "1", "0.71", 0.55),
             name="aggregate_taylor", sigma=0.05, dt=0.05, k=2, k_init=6,
             theta=0.0, q_nom=500_000, taylor=-1, steps=20),
        # fitting a spectrum: gradient through 100 steps of the 12-site ring
        _run("adjoint", RING12, name="adjoint_ring12", steps=100, ckpt=50),
    ]


def draw(rng):
    """One more case of the listed ranges."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def lattice(small=False):
        nd = rng.choice([1, 1, 2, 3])
        if small:
            nd = 1
            ext = [rng.randint(3, 5)]
        elif nd == 1:
            ext = [rng.randint(5, 25)]
        elif nd == 2:
            ext = [rng.randint(2, 6), rng.randint(2, 6)]
        else:
            ext = [rng.randint(2, 4) for _ in range(3)]
        two = not small and rng.random() < 0.3
        cut = [rng.randint(3, 5 if small else 20)] + ([rng.randint(3, 31)] if two else [])
        om = [1.0] + ([round(rng.uniform(0.1, 0.6), 3)] if two else [])
        g = [round(rng.uniform(0.5, 1.5), 3)] + ([round(rng.uniform(0.2, 0.7), 3)] if two else [])
        txt = lambda v: ",".join(repr(x) for x in v)  # noqa: E731
        return _lat("x".join(map(str, ext)), min(ext) >= 3 and rng.random() < 0.6,
                    txt(cut), txt(om), txt(g), round(rng.uniform(-1.2, -0.3), 3))

    def usual(c):
        c["sigma"] = round(rng.uniform(0.02, 0.2), 3)
        c["dt"] = rng.choice([0.01, 0.01, 0.02])
        c["precision"] = rng.choice([64, 64, 32])
        c["init"] = rng.choice(["bloch", "local"])
        c["k"] = c["k_init"] = rng.choice([2, 2, 3, 4])
        c["theta"] = round(10.0 ** rng.uniform(-9, -6), 12)
        return c

    kind = rng.choice(["expmv", "expmv", "small", "capped", "qnom", "batch",
                       "propagator", "adjoint"])
    if kind == "expmv":
        lat = _lat(str(rng.randint(3, 24)), rng.random() < 0.7,
                   str(rng.randint(3, 15)), "1", "1.1", -0.9)
        n, top = int(lat["dims"]), logint(50, 1_200_000)
        ph = 1
        while ph < 30 and n * math.comb(n + ph + 1, ph + 1) <= top:
            ph += 1
        rows = n * math.comb(n + ph, ph)
        return dict(lat, kind="expmv", sigma=0.1, dt=rng.choice([0.01, 0.02, 0.05]),
                    n_max=ph, keep=round(rng.uniform(0.6, 1.0), 3),
                    static=rows <= 300_000 and rng.random() < 0.5)
    if kind == "small":
        c = usual(_run("run", lattice(small=True)))
        return dict(c, precision=64, steps=rng.randint(20, 300), state=True)
    if kind == "capped":
        c = usual(_run(rng.choice(["run", "rerun"]), lattice()))
        return dict(c, k=2, k_init=2, max_states=logint(2_000, 60_000),
                    steps=rng.randint(10, 40))
    if kind == "qnom":
        c = usual(_run("run", lattice()))
        return dict(c, k=2, k_init=rng.randint(2, 4), theta=0.0,
                    q_nom=logint(1_000, 200_000), dt=rng.choice([0.02, 0.05]),
                    steps=rng.randint(10, 40))
    if kind == "batch":
        c = usual(_run("rerun", lattice()))
        return dict(c, k=2, k_init=2, theta=round(10.0 ** rng.uniform(-7, -6), 10),
                    n_real=rng.randint(2, 48), steps=rng.randint(4, 9))
    if kind == "propagator":
        c = usual(_run("run", lattice()))
        p = rng.choice([rng.randint(2, 12), -1, 0])
        return dict(c, k=2, k_init=2, steps=rng.randint(6, 14),
                    krylov=max(p, 0), taylor=min(p, 0))
    c = usual(_run("adjoint", lattice(small=True)))
    return dict(c, precision=64, steps=rng.randint(5, 60), ckpt=rng.randint(4, 50))


# ---- inputs ------------------------------------------------------------------
def _nums(text, kind=float):
    return [kind(x) for x in text.split(",")]


def _config(case):
    ext = [int(x) for x in case["dims"].split("x")]
    per = [1 if case["periodic"] else 0] * len(ext)
    pad = [1] * (3 - len(ext))
    return {"ndim": len(ext), "extent": ext + pad, "periodic": per + [0] * (3 - len(ext)),
            "n_modes": len(case["cutoff"].split(",")), "cutoff": _nums(case["cutoff"], int),
            "omega": _nums(case["omega"]), "g": _nums(case["g"]),
            "J": [case["J"]] * len(ext), "eps_sigma": case["sigma"], "eps_seed": None}


def _params(case, seed):
    cfg = _config(case)
    n, R = WL.n_sites(cfg), case.get("n_real", 1)
    rng = np.random.default_rng([int(seed), 1])
    eps = rng.normal(0.0, case["sigma"], R * n).tolist()
    p = WL.model_params(cfg, eps=eps[:n])
    p["eps"] = eps
    p["n_real"] = R
    return cfg, p


def _run_params(case):
    return {"dt": case["dt"], "k": case["k"], "k_init": case["k_init"],
            "theta": case["theta"], "precision": case["precision"],
            "max_states": case["max_states"], "q_nom": case["q_nom"],
            "krylov_order": case["krylov"], "taylor_order": case["taylor"]}


def _initial(case, cfg):
    return WL.initial_state(cfg, case["init"], site=WL.n_sites(cfg) // 2)


def _rows(case, cfg, seed):
    """Rows of an expmv case: the phonon ball of at most n_max quanta, a
    random part of it left out, and random amplitudes."""
    exc, occ, _ = WL.phonon_ball_state(cfg, case["n_max"])
    rng = np.random.default_rng([int(seed), 2])
    if case["keep"] < 1.0:
        on = np.sort(rng.permutation(len(exc))[:max(1, int(case["keep"] * len(exc)))])
        exc, occ = exc[on], occ[on]
    n = len(exc)
    amp = 10.0 ** (-6.0 * rng.random(n)) * np.exp(2j * np.pi * rng.random(n))
    return exc, occ, amp / np.linalg.norm(amp)


def _target(case, seed):
    """Target a(t) of the adjoint loss."""
    rng = np.random.default_rng([int(seed), 3])
    t = case["dt"] * np.arange(case["steps"] + 1)
    return np.exp(-0.3 * t * t - 1j * rng.uniform(-1.0, 1.0) * t)


def prepare(case, seed):
    cfg, params = _params(case, seed)
    st = {"case": case}
    if case["kind"] == "expmv":
        st["model"] = P.Model(params)
        exc, occ, amp = _rows(case, cfg, seed)
        st["keys"] = torch.from_numpy(st["model"].pack(exc, occ).view(np.int64)).cuda()
        st["phi"] = torch.from_numpy(amp).cuda()
        st["out"] = torch.empty_like(st["phi"])
        return st
    st["run"], st["init"] = _run_params(case), _initial(case, cfg)
    if case["kind"] == "adjoint":
        st["params"] = params
        st["theta"] = torch.tensor(P.theta_of(params), dtype=torch.float64)
        st["target"] = torch.from_numpy(_target(case, seed)).cuda()
        return st
    st["model"] = P.Model(params)
    if case["kind"] == "rerun":
        st["sim"] = P.Sim(st["model"], st["run"], *st["init"])
        st["start"] = st["sim"].state(with_real=True)
    return st


# ---- one pass ----------------------------------------------------------------
def _records(case, rec):
    rec = np.asarray(rec)
    f = {name: rec[..., i] for i, name in enumerate(P.OBS_FIELDS)}
    out = {name: np.ascontiguousarray(f[name]) for name in STATE}
    out["a"] = f["a_re"] + 1j * f["a_im"]
    out["pop"] = np.ascontiguousarray(rec[..., 12:])
    if not case["krylov"]:
        # the Krylov propagator's inner products sum in row order: a state
        # within rounding of the threshold may fall on either side of it
        out["n"] = np.stack([f["n_S"], f["n_M"], f["K"]], -1).astype(np.int64)
    else:
        del out["mass_step"]
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "expmv":
        m = state["model"]
        fn = m.expmv_static if case["static"] else m.expmv
        return fn(state["keys"], state["phi"], case["dt"], out=state["out"])
    if kind == "adjoint":
        theta = state["theta"].clone().requires_grad_(True)
        a = P.AutocorrFn.apply(theta, state["params"], state["run"], state["init"],
                               case["steps"], case["ckpt"])
        loss = (a - state["target"]).abs().square().sum()
        loss.backward()
        return {"a": a.detach(), "grad": theta.grad}
    if kind == "rerun":
        sim = state["sim"]
        keys, amps, real = state["start"]
        sim.set_state(keys, amps, 0.0, real=real)
        first = sim.num_records()
        sim.step(case["steps"])
        return _records(case, sim.series(first))
    sim = P.Sim(state["model"], state["run"], *state["init"])
    sim.step(case["steps"])
    out = _records(case, sim.series())
    if case["state"]:
        keys, amps = sim.state()
        order = np.lexsort(keys.T[::-1])
        out["keys"], out["amps"] = keys[order].view(np.int64), amps[order]
    sim.close()
    return out


# ---- necessary work ----------------------------------------------------------
def work(case):
    """Bytes and operations of one pass.  Per state and series term: the
    input, the term before it, the start vector and the result (A bytes
    each), D columns of 4 and 8 of row data; a complex multiply-add per
    nonzero.  Besides, per step and state: the amplitude read by the
    truncation and by the observables and the key, row data and columns of
    a state written once.  Row and term counts come from a run."""
    cfg, params = _params(case, 0)
    m = P.Model(params)
    D, W = m.D, m.W
    if case["kind"] == "expmv":
        n = int(len(_rows(case, cfg, 0)[0]))
        K = 10
        return {"bytes": float(n * (8 * W + 2 * 16 + (K - 1) * (64 + 4 * D + 8))),
                "flops": float(n * (K - 1) * 8 * (D + 1))}
    sim = P.Sim(m, _run_params(case), *_initial(case, cfg))
    sim.step(case["steps"])
    rec = sim.series().reshape(-1, m.rec_doubles)
    sim.close()
    A = case["precision"] // 4
    rows, K = rec[:, 7], rec[:, 9]
    new = float(np.maximum(rows[1:] - rows[:-1], 0).sum() + rows[0]) if m.R == 1 else float(rows.max())
    term = float((rows * np.maximum(K - 1, 1)).sum())
    by = term * (4 * A + 4 * D + 8) + float(rows.sum()) * 2 * A + new * (8 * W + 8 + 4 * D)
    fl = term * 8 * (D + 1)
    if case["kind"] == "adjoint":
        # the backward sweep: the adjoint vector back, both vectors to the
        # quadrature nodes, the node vectors contracted
        by, fl = by * 4, fl * 4
    return {"bytes": by, "flops": fl}


# ---- 64-bit results in plain torch -------------------------------------------
def _lattice_table(cfg):
    """Neighbour sites [N][2 ndim], -1 where a hop leaves the lattice."""
    ext, per, nd = cfg["extent"], cfg["periodic"], cfg["ndim"]
    N = WL.n_sites(cfg)
    out = np.full((N, 2 * nd), -1, dtype=np.int64)
    for i in range(N):
        c = [i % ext[0], (i // ext[0]) % ext[1], i // (ext[0] * ext[1])]
        for a in range(nd):
            for q, s in enumerate((1, -1)):
                d = list(c)
                d[a] += s
                if not 0 <= d[a] < ext[a]:
                    if not per[a]:
                        continue
                    d[a] %= ext[a]
                out[i, 2 * a + q] = d[0] + ext[0] * (d[1] + ext[1] * d[2])
    return out


class _Graph:
    """H on the given rows (one realization): neighbour rows by a 64-bit
    sum hash and searchsorted, values from the parameters."""

    def __init__(self, cfg, exc, occ):
        N, V, nd = WL.n_sites(cfg), cfg["n_modes"], cfg["ndim"]
        rng = np.random.default_rng(12345)
        r = rng.integers(1, 2 ** 63, size=N * V, dtype=np.uint64)
        rj = rng.integers(1, 2 ** 63, size=N, dtype=np.uint64)
        exc = np.asarray(exc, dtype=np.int64)
        occ = np.asarray(occ).reshape(len(exc), N * V)
        h = rj[exc].copy()
        for i in range(N * V):
            h += occ[:, i].astype(np.uint64) * r[i]
        order = np.argsort(h)
        hs = h[order]

        def find(key, ok):
            at = np.minimum(np.searchsorted(hs, key), len(hs) - 1)
            return np.where(ok & (hs[at] == key), order[at], -1)

        nbr = _lattice_table(cfg)
        self.col, self.val = [], []
        rows = np.arange(len(exc))
        for s in range(2 * nd):
            jn = nbr[exc, s]
            self.col.append(find(h - rj[exc] + rj[np.maximum(jn, 0)], jn >= 0))
            self.val.append(("J", s // 2, None))
        for nu in range(V):
            at = exc * V + nu
            n = occ[rows, at].astype(np.int64)
            self.col.append(find(h - r[at], n > 0))
            self.val.append(("g", nu, torch.from_numpy(np.sqrt(n.astype(np.float64)))))
            self.col.append(find(h + r[at], n < cfg["cutoff"][nu]))
            self.val.append(("g", nu, torch.from_numpy(np.sqrt(n + 1.0))))
        self.col = [torch.from_numpy(c) for c in self.col]
        self.tot = [torch.from_numpy(occ.reshape(-1, N, V)[:, :, nu].sum(1).astype(np.float64))
                    for nu in range(V)]
        self.exc = torch.from_numpy(exc)

    def to(self, dev):
        self.col = [c.to(dev) for c in self.col]
        self.val = [(a, b, v if v is None else v.to(dev)) for a, b, v in self.val]
        self.tot, self.exc = [t.to(dev) for t in self.tot], self.exc.to(dev)
        return self

    def matrix(self, th, nd, V, on=None):
        """Diagonal and (column, value) lists for parameters th (J, g,
        omega, eps), restricted to the rows of mask `on`."""
        J, g, om, eps = th[:nd], th[nd:nd + V], th[nd + V:nd + 2 * V], th[nd + 2 * V:]
        d = eps[self.exc]
        for nu in range(V):
            d = d + om[nu] * self.tot[nu]
        off = []
        for c, (what, q, v) in zip(self.col, self.val):
            ok = c >= 0
            if on is not None:
                ok = ok & on & on[c.clamp(min=0)]
            w = J[q].expand(len(c)) if what == "J" else g[q] * v
            off.append((c.clamp(min=0), w * ok))
        return d, off


def _apply(mat, x):
    d, off = mat
    y = d * x
    for c, w in off:
        y = y + w * x[c]
    return y


def _bounds(mat, on=None):
    d, off = mat
    rad = sum(w.abs() for _, w in off)
    lo, hi = d - rad, d + rad
    if on is not None:
        lo, hi = lo[on], hi[on]
    lo, hi = float(lo.min()), float(hi.max())
    pad = 1e-12 * (abs(lo) + abs(hi))
    return lo - pad, hi + pad


def _expm(mat, x, dt, lo, hi):
    """exp(-i H dt) x by the Taylor series about the interval's centre."""
    b, a = 0.5 * (lo + hi), 0.5 * (hi - lo)
    parts = max(1, math.ceil(a * dt))
    for _ in range(parts):
        term = acc = x
        for k in range(1, 40):
            term = (_apply(mat, term) - b * term) * (-1j * dt / parts / k)
            acc = acc + term
        x = acc
    return x * complex(math.cos(b * dt), -math.sin(b * dt))


def _full_space(cfg):
    """Every state of a small lattice, or None."""
    N, V = WL.n_sites(cfg), cfg["n_modes"]
    dims = [c + 1 for _ in range(N) for c in cfg["cutoff"]]
    if N * math.prod(dims) > 12_000:
        return None
    occ = np.indices(dims).reshape(N * V, -1).T
    return np.repeat(np.arange(N), len(occ)), np.tile(occ, (N, 1))


def exact(case, seed):
    cfg, params = _params(case, seed)
    nd, V, N = cfg["ndim"], cfg["n_modes"], WL.n_sites(cfg)
    if case["kind"] == "expmv":
        exc, occ, amp = _rows(case, cfg, seed)
        g = _Graph(cfg, exc, occ).to("cuda")
        th = torch.tensor(P.theta_of(params), dtype=torch.float64, device="cuda")
        mat = g.matrix(th, nd, V)
        return _expm(mat, torch.from_numpy(amp).cuda(), case["dt"], *_bounds(mat))
    space = None
    if case.get("n_real", 1) == 1 and case["precision"] == 64 and not (
            case["max_states"] or case["q_nom"] or case["krylov"] or case["taylor"]):
        space = _full_space(cfg)
    if space is None or case["steps"] * len(space[0]) > 1_500_000:
        return None
    exc, occ = space
    g = _Graph(cfg, exc, occ)
    adjoint = case["kind"] == "adjoint"
    th = torch.tensor(P.theta_of(params), dtype=torch.float64, requires_grad=adjoint)
    ie, io, ic = _initial(case, cfg)
    io = np.asarray(io).reshape(len(ie), N * V)
    psi0 = torch.zeros(len(exc), dtype=torch.complex128)
    for q, j in enumerate(ie):
        at = int(np.nonzero((exc == j) & (occ == io[q]).all(1))[0][0])
        psi0[at] = complex(ic[2 * q], ic[2 * q + 1])
    psi, inside = psi0, psi0 != 0
    out = {"norm2": [], "energy": [], "mass_step": [], "E_min": [], "E_max": [],
           "a": [], "pop": []}
    a = [(psi0.conj() * psi0).sum()]
    for step in range(case["steps"]):
        c = psi.detach()
        w = c.real ** 2 + c.imag ** 2
        M = inside if step == 0 and case["kind"] != "rerun" else inside & (w >= case["theta"] ** 2)
        S = M.clone()
        for _ in range(case["k_init"] if step == 0 and case["kind"] != "rerun" else case["k"]):
            grown = S.clone()
            for col in g.col:
                ok = S & (col >= 0)
                grown[col[ok]] = True
            S = grown
        mat = g.matrix(th, nd, V, S)
        phi = psi * S
        lo, hi = _bounds((mat[0].detach(), [(x, y.detach()) for x, y in mat[1]]), S)
        out["mass_step"].append(float(w[inside & ~S].sum()))
        out["E_min"].append(lo)
        out["E_max"].append(hi)
        out["energy"].append(float((phi.conj() * _apply(mat, phi)).sum().detach().real))
        psi, inside = _expm(mat, phi, case["dt"], lo, hi) * S, S
        a.append((psi0.conj() * psi).sum())
        v = psi.detach()
        w = v.real ** 2 + v.imag ** 2
        out["norm2"].append(float(w.sum()))
        out["pop"].append(torch.bincount(g.exc, w, N).numpy())
    if adjoint:
        a = torch.stack(a)
        (a - torch.from_numpy(_target(case, seed))).abs().square().sum().backward()
        return {"a": a.detach(), "grad": th.grad}
    out = {k: np.asarray(v) for k, v in out.items()}
    out["a"] = torch.stack(a[1:]).detach().numpy()
    out["n"] = None
    if case["state"]:
        m = P.Model(params)
        on = inside.numpy()
        keys = m.pack(exc[on], occ[on])
        order = np.lexsort(keys.T[::-1])
        out["keys"], out["amps"] = None, psi.detach().numpy()[on][order]
    return out
