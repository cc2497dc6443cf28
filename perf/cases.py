"""Timed cases of the library's public entry points.

A case names an entry point (`kind`), a mechanism size, a number of states and
the options of the call.  Mechanisms and states are the seeded synthetic ones
of `synth`: the four benchmark workloads (13, 53, 111 and 360 species) and, in
drawn cases, a few sizes between them.

  kind       call timed                                       result
  jacobian   Mechanism.eval_jacobian                          J
  rates      Mechanism.eval_rates, every output               R_f, R_r, c, wdot, dphi
  rhs        Mechanism.eval_rates, the RHS alone              dphi
  conc       Mechanism.eval_jacobian_conc                     the sparse concentration form
  newton     Mechanism.newton_solve on a Jacobian in hand     x and the status
  step       eval_jacobian, then newton_solve                 J, x and the status
  sdirk3     Mechanism.sdirk3_step                            the next state
  serve      Server.submit of a burst, then Server.wait       every request's x and status

`exact` evaluates the same quantities with plain torch in 64 bits: the rates
from their textbook formulas, derivatives by the complex step.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1605_03262_amd import NEWTON_FP64, NEWTON_MIXED, Mechanism, Server
from synth import NEWTON_GAMMA, WORKLOADS, config_mechanism, draw_states, make_mechanism

# (reactions, composition bounds) of the generic sizes between the workloads
GENERIC = {28: (100, dict(C=1, H=3, O=2, N=1)), 40: (100, dict(C=1, H=3, O=2, N=1)),
           62: (400, dict(C=2, H=6, O=3, N=1)), 80: (560, dict(C=2, H=6, O=3, N=1)),
           200: (1200, dict(C=5, H=12, O=3, N=1))}
WORKLOAD_OF = {w["n_species"]: c for c, w in WORKLOADS.items()}
SIZES = sorted(list(WORKLOAD_OF) + list(GENERIC))
SDIRK_GAMMA = 0.43586652150845899942
SDIRK_ITERS = 4
R_GAS, ATM, LN10 = 8314.462618, 101325.0, math.log(10.0)


# ------------------------------------------------------------------- cases
def _case(kind, species, n, pad=0, mode="fp64", tuned=False):
    return {"kind": kind, "species": species, "n": n, "pad": pad, "mode": mode, "tuned": tuned}


def listed():
    def named(name, *a, **k):
        return dict(_case(*a, **k), name=name)
    return [
        # a single reactor's cell or a handful of particles: launch latency
        named("jacobian_13sp_48", "jacobian", 13, 48),
        # one PaSR ensemble of 1,000 particles, the handle as loaded
        named("jacobian_53sp_1000", "jacobian", 53, 1000),
        # the benchmark step: tuned Jacobian and mixed Newton solve of a full batch
        named("step_53sp_100000_mixed", "step", 53, 100_000, mode="mixed", tuned=True),
        # the larger mechanisms, batches cut by a domain decomposition (odd, padded rows)
        named("jacobian_111sp_20001", "jacobian", 111, 20_001, pad=15, tuned=True),
        named("jacobian_360sp_2051", "jacobian", 360, 2051, tuned=True),
        # an explicit integrator's call, and a sensitivity study's, with every output
        named("rhs_111sp_30000", "rhs", 111, 30_000),
        named("rates_53sp_100000", "rates", 53, 100_000),
        # constant-volume reactors
        named("conc_53sp_30011", "conc", 53, 30_011, tuned=True),
        # an implicit integrator's own Newton solves, FP64 and mixed
        named("newton_53sp_100000_fp64", "newton", 53, 100_000),
        named("newton_360sp_4099_fp64", "newton", 360, 4099),
        # one implicit step per cell, as the particle driver takes it
        named("sdirk3_111sp_4003", "sdirk3", 111, 4003),
        # the server under a closed burst of mixed requests
        named("serve_burst_24", "serve", 0, 24, mode="mixed"),
    ]


# most N^2 n of a drawn case, so that none takes longer than the longest listed one
MOST = {"jacobian": 2.8e8, "rates": 2.8e8, "rhs": 3.7e8, "conc": 2.8e8, "newton": 2.6e8, "step": 2.6e8,
        "sdirk3": 4.9e7}


def draw(rng):
    kind = rng.choice(["jacobian", "jacobian", "rates", "rhs", "conc", "newton", "newton", "newton", "step", "step",
                       "sdirk3", "sdirk3"] + ["serve"] * (rng.random() < 0.3))
    mode = rng.choice(["fp64", "mixed"])
    if kind == "serve":
        return _case("serve", 0, rng.randint(6, 24), mode=mode)
    species = rng.choice(SIZES)
    top = min(100_000, int(MOST[kind] / species ** 2))
    if kind == "sdirk3" and species > 111:      # thirteen passes over every factor
        top //= 3
    n = int(round(math.exp(rng.uniform(math.log(8), math.log(top)))))
    if rng.random() < 0.5:
        n = min(top, n | 1)
    return _case(kind, species, n, pad=rng.choice([0, 0, 0, 1, 7, 32]), mode=mode,
                 tuned=kind in ("jacobian", "conc", "step") and rng.random() < 0.5)


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def _mech(species):
    """The synthetic mechanism of that size (the input data, not a handle)."""
    if species in WORKLOAD_OF:
        m = config_mechanism(WORKLOAD_OF[species])
    else:
        nr, bounds = GENERIC[species]
        el, tb, fo, sri = round(0.7 * nr), round(0.1 * nr), round(0.05 * nr), round(0.03 * nr)
        mix = {"elementary": el, "thirdbody": tb, "falloff_lindemann": fo, "falloff_sri": sri,
               "falloff_troe": nr - el - tb - fo - sri}
        m = make_mechanism(1605 + species, species, nr, ["C", "H", "O", "N", "Ar"], bounds, mix)
    return m, m.to_text()


def _states(species, n, ld, seed):
    """phi [N, ld] and p [ld] on the host; columns past n hold states as well."""
    w = WORKLOADS[WORKLOAD_OF.get(species, 1)]
    return draw_states(seed, species, ld, w["T"], w["P_atm"], w["dirichlet"])


def _factors(seed, n, lo, hi):
    return np.exp(np.random.default_rng([seed, 1]).uniform(math.log(lo), math.log(hi), n))


def _rhs(seed, N, ld):
    return np.random.default_rng([seed, 2]).standard_normal((N, ld))


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _step_sizes(J, N, c, gamma):
    """h = c / (gamma ||J||_inf) per state, as an integrator's step control keeps it."""
    return c / (gamma * J.view(N, N, -1).abs().sum(1).max(0).values)


def _requests(count, seed):
    """(species, states, seed) of a burst: the serving mix's weights and
    log-uniform sizes, the same for every seed; the seed draws the states."""
    rng, weights = np.random.default_rng(count), [0.4, 0.3, 0.2, 0.1]
    return [(sorted(WORKLOAD_OF)[int(rng.choice(4, p=weights))], int(math.exp(rng.uniform(0.0, math.log(513.0)))),
             seed + 1000 * i) for i in range(count)]


_MODE = {"fp64": NEWTON_FP64, "mixed": NEWTON_MIXED}


def _prepare_serve(case, seed):
    mechs = {s: Mechanism(text=_mech(s)[1]) for s in sorted(WORKLOAD_OF)}
    srv = Server(hbm_budget_bytes=16 << 30, max_batch_states=1024, n_streams=4)
    reqs = []
    for s, n, sd in _requests(case["n"], seed):
        phi, p = _states(s, n, n, sd)
        h = _step_sizes(mechs[s].eval_jacobian(_gpu(phi), _gpu(p)), s, _gpu(_factors(sd, n, 1.0, 3.0e3)), NEWTON_GAMMA)
        reqs.append((mechs[s], phi, p, h.cpu().numpy(), _rhs(sd, s, n)))
    # a running server has its pools: one request of every mechanism beforehand
    for s, m in mechs.items():
        phi, p = _states(s, 1, 1, 5)
        srv.wait(srv.submit(m, phi, p, np.full(1, 1e-12), np.ones((s, 1)), NEWTON_GAMMA, _MODE[case["mode"]])[0])
    return {"case": case, "srv": srv, "reqs": reqs, "mechs": mechs}


def prepare(case, seed):
    kind, N, n = case["kind"], case["species"], case["n"]
    if kind == "serve":
        return _prepare_serve(case, seed)
    M = Mechanism(text=_mech(N)[1])
    ld = n + case["pad"]
    phi_h, p_h = _states(N, n, ld, seed)
    if kind == "conc":
        phi_h = _concentrations(_mech(N)[0], phi_h, p_h)
    phi, p = _gpu(phi_h), _gpu(p_h)
    st = {"case": case, "M": M, "phi": phi[:, :n], "p": p}
    new = lambda rows: torch.empty((rows, ld), dtype=torch.float64, device="cuda")  # noqa: E731
    if case["tuned"]:
        M.autotune(2 if kind == "conc" else 1, st["phi"], p)
    if kind in ("jacobian", "newton", "step"):
        st["out"] = new(N * N)[:, :n]
    elif kind == "conc":
        st["out"] = new(3 * N + 1 + len(M.conc_pattern()[1]))[:, :n]
    elif kind == "rates":
        NR = M.n_reactions
        st["outs"] = {k: new(r) for k, r in (("rop_f", NR), ("rop_r", NR), ("pres_mod", NR), ("wdot", N), ("dphi", N))}
    elif kind == "rhs":
        st["outs"] = {"rop_f": False, "rop_r": False, "pres_mod": False, "wdot": False, "dphi": new(N)}
    if kind in ("newton", "step", "sdirk3"):
        small, gamma = kind == "sdirk3", SDIRK_GAMMA if kind == "sdirk3" else NEWTON_GAMMA
        J = M.eval_jacobian(phi, p)             # the padding columns are states too
        c = _gpu(_factors(seed, ld, 0.1, 10.0) if small else _factors(seed, ld, 1.0, 3.0e3))
        st["h"] = _step_sizes(J, N, c, gamma)
        if small:
            st["next"] = new(N)[:, :n]
            st["ws"] = torch.empty((_sdirk_bytes(M, n, ld, case["mode"]),), dtype=torch.uint8, device="cuda")
        else:
            st["rhs"] = _gpu(_rhs(seed, N, ld))[:, :n]
            if kind == "newton":
                st["out"] = J[:, :n]
            need = M.newton_workspace_bytes(n, _MODE[case["mode"]])
            st["ws"] = torch.empty((need,), dtype=torch.uint8, device="cuda") if need else None
    return st


def _sdirk_bytes(M, n, ld, mode):
    from paper_1605_03262_amd import _lib
    return max(1, _lib.pyjac_sdirk3_workspace_bytes(M.handle, n, ld, _MODE[mode]))


def run(st):
    case = st["case"]
    kind, n, mode = case["kind"], case["n"], _MODE[case["mode"]]
    if kind == "serve":
        got = [st["srv"].submit(m, phi, p, h, b, NEWTON_GAMMA, mode) for m, phi, p, h, b in st["reqs"]]
        for rid, _, _ in got:
            st["srv"].wait(rid)
        return [{"x": x, "failed": info < 0} for _, x, info in got]
    M = st["M"]
    if kind == "jacobian":
        return M.eval_jacobian(st["phi"], st["p"], out=st["out"])
    if kind == "conc":
        return M.eval_jacobian_conc(st["phi"], out=st["out"])
    if kind in ("rates", "rhs"):
        return {k: v[:, :n] for k, v in M.eval_rates(st["phi"], st["p"], **st["outs"]).items()}
    if kind == "sdirk3":
        # (the second result, each stage's last increment, is at the level of rounding)
        y, _ = M.sdirk3_step(st["phi"], st["p"], st["h"], newton_iters=SDIRK_ITERS, mode=mode, out=st["next"],
                             workspace=st["ws"])
        return y
    if kind == "step":
        M.eval_jacobian(st["phi"], st["p"], out=st["out"])
    x, info = M.newton_solve(st["out"], st["h"], st["rhs"], NEWTON_GAMMA, mode=mode, workspace=st["ws"])
    # an integrator looks at whether a state was solved; the sweep count of
    # the mixed mode (info >= 1) is a diagnostic
    res = {"x": x[:, :n], "failed": info[:n] < 0}
    if kind == "step":
        res["jac"] = st["out"]
    return res


def work(case):
    """Least traffic and arithmetic of one pass: inputs read once, outputs
    written once, an LU and its solves; 80 operations per reaction (two
    exponentials, the products), and two per Jacobian element."""
    if case["kind"] == "serve":
        by = fl = 0.0
        for s, n, _ in _requests(case["n"], 0):
            by += n * 8.0 * (3 * s + 2)
            fl += n * (2.0 / 3.0 * s ** 3 + 2.0 * s ** 2 + 80.0 * len(_mech(s)[0].reactions))
        return {"bytes": by, "flops": fl}
    kind, N, n = case["kind"], case["species"], case["n"]
    NR = len(_mech(N)[0].reactions)
    react, lu = 80.0 * NR, 2.0 / 3.0 * N ** 3 + 2.0 * N ** 2
    by, fl = {
        "jacobian": (8.0 * (N + 1 + N * N), react + 2.0 * N * N),
        "rates": (8.0 * (N + 1 + 3 * NR + 2 * N), react),
        "rhs": (8.0 * (N + 1 + N), react),
        "conc": (8.0 * (N + 1 + 3 * N + 1 + len(_pattern(N)[1])), react + 2.0 * N * N),
        "newton": (8.0 * (N * N + 2 * N + 1) + 4.0, lu),
        "step": (8.0 * (N * N + 3 * N + 2) + 4.0, lu + react + 2.0 * N * N),
        "sdirk3": (8.0 * (2 * N + 2), lu + react * (3 * SDIRK_ITERS + 3) + 2.0 * N * N * 3 * SDIRK_ITERS),
    }[kind]
    return {"bytes": n * by, "flops": n * fl}


# ------------------------------------------------- the same in plain torch
def _concentrations(m, phi, p):
    """{T, [X_1 .. X_N]} of the constant-pressure states (numpy)."""
    W = np.array([s.W for s in m.species])
    Y = np.vstack([phi[1:], 1.0 - phi[1:].sum(0)])
    rho = p / (R_GAS * phi[0] * (Y / W[:, None]).sum(0))
    return np.vstack([phi[:1], rho * np.maximum(Y, 0.0) / W[:, None]])


@functools.lru_cache(maxsize=None)
def _pattern(species):
    """Compressed columns of the concentration form's sparse part."""
    m = _mech(species)[0]
    cols = [set() for _ in range(species)]
    for r in m.reactions:
        net = {}
        for side, sign in ((r.reac, -1), (r.prod, 1)):
            for k, v in side:
                net[k] = net.get(k, 0) + sign * v
        who = {k for k, _ in r.reac} | ({k for k, _ in r.prod} if r.rev != "irrev" else set())
        if r.collider == "mix":
            who |= {k for k, a in r.eff.items() if a != 1.0}
        elif r.collider == "species":
            who.add(r.collider_species)
        for j in who:
            cols[j] |= {k for k, v in net.items() if v}
    ptr, rows = [0], []
    for c in cols:
        rows += sorted(c)
        ptr.append(len(rows))
    return ptr, rows


class _Plain:
    """The kinetics of one mechanism as torch tensors, reactions by states.
    Every quantity may be complex: the imaginary part carries a derivative."""

    def __init__(self, m):
        g = lambda a, t=torch.float64: torch.tensor(np.asarray(a), dtype=t, device="cuda")  # noqa: E731
        self.N, self.NR = N, NR = m.n_species, m.n_reactions
        self.W = g([s.W for s in m.species])[:, None]
        self.tmid = g([s.tmid for s in m.species])[:, None]
        self.lo, self.hi = g([s.low for s in m.species]), g([s.high for s in m.species])
        nu = np.zeros((N, NR))
        mol = np.full((6, NR), N)
        am1 = np.zeros((NR, N))
        base = np.zeros(NR)
        arr = np.ones((NR, 3))
        for i, r in enumerate(m.reactions):
            for side, sign, at in ((r.reac, -1, 0), (r.prod, 1, 3)):
                for k, v in side:
                    nu[k, i] += sign * v
                    mol[at:at + v, i] = k
                    at += v
            if r.collider == "mix":
                base[i] = 1.0
                for k, a in r.eff.items():
                    am1[i, k] = a - 1.0
            elif r.collider == "species":
                am1[i, r.collider_species] = 1.0
            src = r.arr or (r.high if r.kind.startswith("falloff") else r.low)
            if src is not None:
                arr[i] = src
        assert all(r.rev == "kc" for r in m.reactions)
        kinds = [r.kind for r in m.reactions]
        at = lambda f: g([i for i, k in enumerate(kinds) if f(k)], torch.int64)  # noqa: E731
        self.nu, self.mol, self.arr = g(nu), g(mol, torch.int64), g(arr)
        self.thd = at(lambda k: k == "thirdbody")
        self.blend = at(lambda k: k.startswith(("falloff", "chemact")))
        self.coll = torch.cat([self.thd, self.blend])
        self.am1, self.base = g(am1)[self.coll], g(base)[self.coll][:, None]
        b = [m.reactions[i] for i in self.blend.tolist()]
        self.ratio = [g([f(r) for r in b])[:, None] for f in (lambda r: r.low[0] / r.high[0],
                                                             lambda r: r.low[1] - r.high[1],
                                                             lambda r: r.low[2] - r.high[2])]
        self.act = g([r.kind.startswith("chemact") for r in b], torch.bool)[:, None]
        self.troe = g([i for i, r in enumerate(b) if r.troe is not None], torch.int64)
        self.sri = g([i for i, r in enumerate(b) if r.sri is not None], torch.int64)
        tr = [list(r.troe) + [math.inf] * (4 - len(r.troe)) for r in b if r.troe is not None]
        sr = [list(r.sri) + [1.0, 0.0][len(r.sri) - 3:] for r in b if r.sri is not None]
        self.tp = g(np.array(tr).reshape(-1, 4)).T[:, :, None]
        self.sp = g(np.array(sr).reshape(-1, 5)).T[:, :, None]
        self.plog = [(i, sorted(r.plog)) for i, r in enumerate(m.reactions) if r.plog is not None]
        self.cheb = [(i, r.cheb) for i, r in enumerate(m.reactions) if r.cheb is not None]

    def thermo(self, T):
        """C_p/R, H/RT, S/R per species."""
        a = torch.where((T.real if T.is_complex() else T)[None] <= self.tmid, self.lo.T[:, :, None], self.hi.T[:, :, None])
        cp = a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4])))
        h = a[0] + T * (a[1] / 2 + T * (a[2] / 3 + T * (a[3] / 4 + T * a[4] / 5))) + a[5] / T
        s = a[0] * torch.log(T) + T * (a[1] + T * (a[2] / 2 + T * (a[3] / 3 + T * a[4] / 4))) + a[6]
        return cp, h, s

    def constants(self, T, p):
        """What depends on temperature and pressure only."""
        lT, iT = torch.log(T), 1.0 / T
        re = lambda v: v.real if v.is_complex() else v  # noqa: E731
        kf = self.arr[:, :1] * torch.exp(self.arr[:, 1:2] * lT - self.arr[:, 2:3] * iT)
        if p.is_complex() and not kf.is_complex():
            kf = kf.to(p.dtype)
        lp = torch.log(p)
        for i, pts in self.plog:
            ln = lambda q: math.log(q[1]) + q[2] * lT - q[3] * iT  # noqa: E731
            v = ln(pts[0])
            v = v.to(kf.dtype)
            for q, (u, w) in enumerate(zip(pts, pts[1:])):
                l0, l1 = math.log(u[0]), math.log(w[0])
                f = (lp - l0) / (l1 - l0)
                v = torch.where(re(lp) >= l0, ln(u) + (ln(w) - ln(u)) * f, v)
                if q == len(pts) - 2:
                    v = torch.where(re(lp) >= l1, ln(w).to(v.dtype), v)
            kf[i] = torch.exp(v)
        for i, c in self.cheb:
            x = (2 * iT - 1 / c["Tmin"] - 1 / c["Tmax"]) / (1 / c["Tmax"] - 1 / c["Tmin"])
            y = (2 * lp / LN10 - math.log10(c["Pmin"]) - math.log10(c["Pmax"])) / math.log10(c["Pmax"] / c["Pmin"])
            ch = lambda t, k: [1.0, t] + [0.0] * max(0, k - 2)  # noqa: E731
            tx, ty = ch(x, c["nT"]), ch(y, c["nP"])
            for t, v in ((tx, x), (ty, y)):
                for k in range(2, len(t)):
                    t[k] = 2 * v * t[k - 1] - t[k - 2]
            eta = np.asarray(c["coef"], float).reshape(c["nT"], c["nP"])
            kf[i] = torch.exp(LN10 * sum(eta[a, b] * tx[a] * ty[b] for a in range(c["nT"]) for b in range(c["nP"])))
        _, h, s = self.thermo(T)
        lnK = self.nu.to(h.dtype).T @ (s - h) + self.nu.sum(0)[:, None] * torch.log(ATM / (R_GAS * T))
        ratio = self.ratio[0] * torch.exp(self.ratio[1] * lT - self.ratio[2] * iT)
        t, q = self.tp, self.sp
        Fc = (1 - t[0]) * torch.exp(-T / t[1]) + t[0] * torch.exp(-T / t[2]) + torch.exp(-t[3] * iT)
        sri = q[0] * torch.exp(-q[1] * iT) + torch.exp(-T / q[2])
        return kf, kf * torch.exp(-lnK), ratio, torch.log(Fc), torch.log(sri), torch.log(q[3]) + q[4] * lT

    def progress(self, const, X, M):
        """R_f, R_r and c from the concentrations; M: the sum of them that an
        all-species collider starts from."""
        kf, kr, ratio, lF, lS, lD = const
        Xp = torch.cat([X, torch.ones_like(X[:1])])
        pf = Xp[self.mol[0]] * Xp[self.mol[1]] * Xp[self.mol[2]]
        pr = Xp[self.mol[3]] * Xp[self.mol[4]] * Xp[self.mol[5]]
        Rf, Rr = kf * pf, kr * pr
        c = torch.ones_like(Rf)
        if M.is_complex() and not c.is_complex():
            c = c.to(M.dtype)
        E = self.base * M + self.am1.to(X.dtype) @ X
        nt = len(self.thd)
        c[self.thd] = E[:nt].to(c.dtype)
        if len(self.blend):
            Pr = ratio * E[nt:]
            pos = (Pr.real if Pr.is_complex() else Pr) > 0
            lP = torch.log10(torch.where(pos, Pr, torch.ones_like(Pr)))
            lnF = torch.zeros_like(Pr)
            if len(self.troe):
                a, l = lP[self.troe], lF / LN10
                A, B = a - 0.67 * l - 0.4, 0.806 - 1.1762 * l - 0.14 * a
                lnF[self.troe] = torch.where(pos[self.troe], lF / (1 + (A / B) ** 2), lF / (1 + 1 / 0.14 ** 2)).to(lnF.dtype)
            if len(self.sri):
                a = lP[self.sri]
                lnF[self.sri] = (lD + torch.where(pos[self.sri], lS / (1 + a * a), torch.zeros_like(a))).to(lnF.dtype)
            c[self.blend] = (torch.exp(lnF) * torch.where(self.act, 1 / (1 + Pr), Pr / (1 + Pr))).to(c.dtype)
        return Rf, Rr, c

    def wdot(self, const, X, M):
        Rf, Rr, c = self.progress(const, X, M)
        q = c * (Rf - Rr)
        return self.nu.to(q.dtype) @ q

    def gas(self, phi, p):
        T, Y = phi[0], torch.cat([phi[1:], 1.0 - phi[1:].sum(0, keepdim=True)])
        rho = p / (R_GAS * T * (Y / self.W).sum(0))
        return T, Y, rho, rho * Y / self.W

    def rhs(self, phi, p, const=None):
        T, Y, rho, X = self.gas(phi, p)
        wd = self.wdot(const or self.constants(T, p), X, p / (R_GAS * T))
        cp, h, _ = self.thermo(T)
        cp = (Y * cp * R_GAS / self.W).sum(0)
        dT = -(h * R_GAS * T * wd).sum(0) / (rho * cp)
        return torch.cat([dT[None], (self.W * wd / rho)[:-1]])

    def chunks(self, n):
        m = max(1, int(2.4e7 / self.NR))
        return [slice(a, min(n, a + m)) for a in range(0, n, m)]

    def jacobian(self, phi, p):
        """[N*N, n], column by column by the complex step."""
        N, n, eps = self.N, phi.shape[1], 1e-30
        J = torch.empty((N, N, n), dtype=torch.float64, device=phi.device)
        for sl in self.chunks(n):
            f, pc = phi[:, sl], p[sl]
            real = self.constants(f[0], pc)
            for j in range(N):
                z = f.to(torch.complex128)
                z[j] += 1j * eps
                J[:, j, sl] = self.rhs(z, pc, real if j else None).imag / eps
        return J.view(N * N, n)

    def conc(self, phi, ptr, rows):
        """The concentration form's outputs, in its order."""
        N, n, eps = self.N, phi.shape[1], 1e-30
        out = torch.empty((3 * N + 1 + len(rows), n), dtype=torch.float64, device=phi.device)
        for sl in self.chunks(n):
            T, X = phi[0, sl], phi[1:, sl]
            M = X.sum(0)
            z = torch.complex(torch.zeros_like(T), torch.full_like(T, eps))

            def energy(T, X, wd):
                cp, h, _ = self.thermo(T)
                return -((h - 1) * R_GAS * T * wd).sum(0) / (X * (cp - 1) * R_GAS).sum(0)

            real = self.constants(T, R_GAS * T * M)
            Tz = T + z
            wd = self.wdot(self.constants(Tz, R_GAS * Tz * M), X.to(z.dtype), M)
            out[0, sl] = energy(Tz, X, wd).imag / eps
            out[1:N + 1, sl] = wd.imag / eps
            u = self.wdot(self.constants(T, R_GAS * T * (M + z)), X.to(z.dtype), M + z).imag
            out[2 * N + 1:3 * N + 1, sl] = u / eps
            for j in range(N):
                Xz = X.to(z.dtype)
                Xz[j] += z
                wd = self.wdot(real, Xz, M)
                out[3 * N + 1 + ptr[j]:3 * N + 1 + ptr[j + 1], sl] = wd.imag[rows[ptr[j]:ptr[j + 1]]] / eps
                out[N + 1 + j, sl] = energy(T, Xz, wd + 1j * u).imag / eps
        return out


def _solve(J, N, h, gamma, rhs):
    """x [N, n] of (I - h gamma J) x = rhs."""
    n = rhs.shape[1]
    x = torch.empty_like(rhs)
    step = max(1, int(2.0e8 / N ** 2))
    on = "cuda" if N <= 128 else "cpu"          # large systems one by one
    for a in range(0, n, step):
        sl = slice(a, min(n, a + step))
        A = -(h[sl] * gamma)[:, None, None] * J.view(N, N, n)[:, :, sl].permute(2, 0, 1)
        A = (A + torch.eye(N, dtype=torch.float64, device=J.device)).contiguous().to(on)
        x[:, sl] = torch.linalg.solve(A, rhs[:, sl].T.contiguous()[:, :, None].to(on))[:, :, 0].T.to(x.device)
    return x


def _sdirk(P, phi, p, h, iters):
    """Alexander's three-stage SDIRK method, simplified Newton from z = 0."""
    g, N, n = SDIRK_GAMMA, P.N, phi.shape[1]
    a = [[], [(1 - g) / 2], [-(6 * g * g - 16 * g + 1) / 4, (6 * g * g - 20 * g + 5) / 4]]
    J = P.jacobian(phi, p).view(N, N, n).permute(2, 0, 1)
    A = torch.eye(N, dtype=torch.float64, device=phi.device) - (h * g)[:, None, None] * J
    on = "cuda" if N <= 128 else "cpu"
    lu = torch.linalg.lu_factor(A.contiguous().to(on))
    F = []
    for ai in a:
        z = torch.zeros_like(phi)
        for _ in range(iters):
            r = h * (sum(c * f for c, f in zip(ai, F)) + g * P.rhs(phi + z, p)) - z
            z = z + torch.linalg.lu_solve(*lu, r.T.contiguous()[:, :, None].to(on))[:, :, 0].T.to(z.device)
        F.append(P.rhs(phi + z, p))
    return phi + z


def exact(case, seed):
    kind, N, n = case["kind"], case["species"], case["n"]
    if kind == "serve":
        got = []
        for s, m, sd in _requests(n, seed):
            P = _Plain(_mech(s)[0])
            phi, p = (_gpu(v) for v in _states(s, m, m, sd))
            J = P.jacobian(phi, p)
            h = _step_sizes(J, s, _gpu(_factors(sd, m, 1.0, 3.0e3)), NEWTON_GAMMA)
            got.append({"x": _solve(J, s, h, NEWTON_GAMMA, _gpu(_rhs(sd, s, m))).cpu().numpy(), "failed": None})
        return got
    P = _Plain(_mech(N)[0])
    ld = n + case["pad"]
    phi_h, p_h = _states(N, n, ld, seed)
    if kind == "conc":
        return P.conc(_gpu(_concentrations(_mech(N)[0], phi_h, p_h))[:, :n], *_pattern(N))
    phi, p = _gpu(phi_h)[:, :n].contiguous(), _gpu(p_h)[:n]
    if kind == "jacobian":
        return P.jacobian(phi, p)
    if kind in ("rates", "rhs"):
        T, Y, rho, X = P.gas(phi, p)
        const = P.constants(T, p)
        dphi = P.rhs(phi, p, const)
        if kind == "rhs":
            return {"dphi": dphi}
        Rf, Rr, c = P.progress(const, X, p / (R_GAS * T))
        return {"rop_f": Rf, "rop_r": Rr, "pres_mod": c, "wdot": P.nu @ (c * (Rf - Rr)), "dphi": dphi}
    J = P.jacobian(phi, p)
    if kind == "sdirk3":
        return _sdirk(P, phi, p, _step_sizes(J, N, _gpu(_factors(seed, ld, 0.1, 10.0))[:n], SDIRK_GAMMA), SDIRK_ITERS)
    h = _step_sizes(J, N, _gpu(_factors(seed, ld, 1.0, 3.0e3))[:n], NEWTON_GAMMA)
    x = _solve(J, N, h, NEWTON_GAMMA, _gpu(_rhs(seed, N, ld))[:, :n].contiguous())
    return {"x": x, "failed": None, "jac": J} if kind == "step" else {"x": x, "failed": None}
