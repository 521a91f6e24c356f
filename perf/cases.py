"""What a user of this package has it do, as cases to be timed.

The kinds follow the path of a fit: targets of a relaxation model, one
generation of a global search over many materials (move, then the cost of
every candidate), whole small fits, cost and gradient of given candidates, the
gradient through a material model, the polish of each material's best, and
the report (weights, error, model curves).  Sizes are those of the package's
benchmark workloads and tests (a shard of the largest), and ragged ones.

Materials, spectra and candidates are drawn here from the seed alone, with
plain torch; candidates of a search are uniform in their box, those of a
gradient, a polish or a report are spread over it, one to each N-th of the
box, as fitted ones are.
"""
import math

import numpy as np
import torch

import paper_2109_01928_amd as D

DEV = "cuda"
DAMPING = 1e-8


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the paper's example: one HN material, a whole particle-swarm fit;
        # latency and launches
        dict(name="fit one material", kind="fit", M=1, F=50, N=5, P=40, iters=50, decades=5),
        # a gprMax input file's materials, fitted together from start to end
        dict(name="fit an input file", kind="fit", M=24, F=100, N=6, P=64, iters=100, decades=4),
        # one swarm iteration over mixed materials, the benchmark's middle workload
        dict(name="iteration mixed N8", kind="search", opt="pso", M=1024, F=1000, N=8, P=256, decades=4, ragged=False),
        # one swarm iteration over user tables (a shard of 65,536): the benchmark's default, its largest work
        dict(name="iteration tables N20", kind="search", opt="pso", M=2048, F=4096, N=20, P=128, decades=6,
             ragged=False),
        # uneven batch: spectra, pole counts and swarm sizes differ by material, odd sizes among them
        dict(name="iteration ragged", kind="search", opt="pso", M=512, F=5000, N=20, P=512, decades=4, ragged=True),
        # one generation of differential evolution, the paper's alternative, at twelve poles
        dict(name="generation de N12", kind="search", opt="de", M=256, F=2000, N=12, P=256, decades=6, ragged=False),
        # cost and gradient of several starts per material
        dict(name="gradient N12", kind="grad", M=1024, F=2000, N=12, P=8, decades=6),
        # material parameters learned through the fit: forward and backward of
        # HN targets and the fit's cost
        dict(name="train HN parameters", kind="train", M=64, F=501, N=6, P=16, decades=5),
        # the first steps of the L-BFGS polish of every material's best
        dict(name="polish N12", kind="polish", M=1024, F=2000, N=12, steps=2, decades=6),
        # targets of sums of HN terms with noise: the tables' synthesis
        dict(name="targets tables", kind="targets", M=2048, F=4096, decades=6),
        # after a fit: weights, eps_inf, cost and error of one candidate per material
        dict(name="report N12", kind="report", M=4096, F=1000, N=12, decades=6),
        # Debye basis of a batch of fitted candidates, for the models' curves
        dict(name="curves N8", kind="curves", M=1024, F=1000, N=8, decades=4),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    # gradients, polish and report: up to two poles a decade, as the listed
    # twelve on six decades (denser poles are resolved by no table's noise)
    kind = rng.choice(["fit", "search", "search", "search", "grad", "train", "polish", "targets", "report", "curves"])
    dec = rng.choice([3, 4, 5, 6])
    if kind == "fit":
        return dict(kind=kind, M=_log_int(rng, 1, 48), F=_log_int(rng, 30, 200), N=rng.randint(1, 12),
                    P=_log_int(rng, 20, 64), iters=_log_int(rng, 20, 100), decades=dec)
    if kind == "search":
        c = dict(kind=kind, opt=rng.choice(["pso", "pso", "de", "da"]), M=_log_int(rng, 1, 2048),
                 F=_log_int(rng, 50, 5000), N=rng.randint(1, 24), P=_log_int(rng, 32, 512), decades=dec,
                 ragged=rng.random() < 0.3)
        while _search_flops(c) > 5e11:
            c["M"] = max(1, c["M"] // 2)
        return c
    if kind == "grad":
        c = dict(kind=kind, M=_log_int(rng, 1, 1024), F=_log_int(rng, 50, 5000), N=rng.randint(1, 2 * dec),
                 P=_log_int(rng, 1, 64), decades=dec)
        while c["M"] * c["P"] * _eval_flops(c["F"], c["N"]) > 1e11:
            c["M"] = max(1, c["M"] // 2)
        return c
    if kind == "train":
        return dict(kind=kind, M=_log_int(rng, 1, 256), F=_log_int(rng, 50, 1001), N=rng.randint(2, 2 * dec),
                    P=_log_int(rng, 1, 32), decades=dec)
    if kind == "polish":
        return dict(kind=kind, M=_log_int(rng, 16, 1024), F=_log_int(rng, 100, 4096), N=rng.randint(2, 2 * dec),
                    steps=rng.randint(1, 2), decades=dec)
    if kind == "targets":
        return dict(kind=kind, M=_log_int(rng, 1, 4096), F=_log_int(rng, 50, 4096), decades=dec)
    if kind == "report":
        return dict(kind=kind, M=_log_int(rng, 1, 8192), F=_log_int(rng, 50, 4096), N=rng.randint(1, 2 * dec),
                    decades=dec)
    return dict(kind=kind, M=_log_int(rng, 1, 1024), F=_log_int(rng, 50, 4096), N=rng.randint(1, 20), decades=dec)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    return np.random.Generator(np.random.Philox(key=[int(seed), int(stream)]))


def _band(case):
    f_lo = {3: 1e7, 4: 1e6, 5: 1e5, 6: 1e5}[case["decades"]]
    return f_lo, f_lo * 10.0 ** case["decades"]


def _box(case):
    f_lo, f_hi = _band(case)
    return math.floor(-math.log10(2 * math.pi * f_hi)) - 1.0, float(math.floor(-math.log10(2 * math.pi * f_lo)))


def _grid(case, F):
    f_lo, f_hi = _band(case)
    return 2 * math.pi * np.logspace(math.log10(f_lo), math.log10(f_hi), F)


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(np.asarray(sizes, np.int64))])


def _shape(case):
    """Spectrum length, pole count and candidates of each material."""
    M, P = case["M"], case.get("P", 1)
    if not case.get("ragged"):
        return np.full(M, case["F"]), np.full(M, case.get("N", 1)), np.full(M, P)
    # the same sizes for every seed, as one user's batch has
    g = np.random.Generator(np.random.Philox(key=[M, case["F"]]))
    F = g.integers(max(1, case["F"] // 50), case["F"] + 1, size=M)
    N = g.integers(min(2, case["N"]), case["N"] + 1, size=M)
    N[0] = case["N"]
    return F, N, np.maximum(1, P >> g.integers(0, 4, size=M))


def _hn_draw(M, g):
    """[M][3 terms][d_eps, tau0, alpha, beta], eps_inf [M], terms used [M]."""
    u = g.random((M, 3, 4))
    p = np.stack([5 + 75 * u[..., 0], 10 ** (-11 + 4 * u[..., 1]), 0.3 + 0.7 * u[..., 2], 0.3 + 0.7 * u[..., 3]], -1)
    return p, 2 + 6 * g.random(M), g.integers(1, 4, size=M)


def _hn_sum(omega, mat, p, einf, terms):
    """eps of each point (complex128) from its material's HN terms."""
    eps = einf[mat].to(torch.complex128)
    for t in range(3):
        q = p[:, t][mat]
        jw = torch.complex(torch.zeros_like(omega), omega * q[:, 1])
        v = q[:, 0] * (1 + jw ** q[:, 2]) ** (-q[:, 3])
        eps = eps + torch.where(terms[mat] > t, v, torch.zeros_like(v))
    return eps


def _spectra(case, seed):
    """Offsets, omega and targets (eps', eps''; 1 % noise, as measured tables have) of the case's materials."""
    F, _, _ = _shape(case)
    f_off = _offsets(F)
    if case.get("ragged"):
        omega = np.concatenate([_grid(case, int(f)) for f in F])
    else:
        omega = np.tile(_grid(case, case["F"]), case["M"])
    om = torch.tensor(omega, device=DEV)
    mat = torch.repeat_interleave(torch.arange(case["M"], device=DEV), torch.tensor(F, device=DEV))
    p, einf, terms = (torch.tensor(a, device=DEV) for a in _hn_draw(case["M"], _gen(seed, 1)))
    er, ei = torch.empty_like(om), torch.empty_like(om)
    for a in range(0, len(omega), 1 << 22):
        s = slice(a, a + (1 << 22))
        e = _hn_sum(om[s], mat[s], p, einf, terms)
        er[s], ei[s] = e.real, -e.imag
    noise = torch.Generator(device=DEV).manual_seed(int(seed) * 7 + 1)
    er *= 1 + 0.01 * torch.randn(len(omega), generator=noise, dtype=torch.float64, device=DEV)
    ei *= 1 + 0.01 * torch.randn(len(omega), generator=noise, dtype=torch.float64, device=DEV)
    return f_off, om, er, ei


def _batch(case, seed):
    _, N, P = _shape(case)
    f_off, om, er, ei = _spectra(case, seed)
    return D.Batch(f_off, _offsets(P), N, om, er, ei, DEV)


def _box_tensors(case):
    lo, hi = _box(case)
    return (torch.full((case["M"],), lo, dtype=torch.float64, device=DEV),
            torch.full((case["M"],), hi, dtype=torch.float64, device=DEV))


def _uniform_theta(case, b, seed):
    lo, hi = _box(case)
    return torch.tensor(lo + (hi - lo) * _gen(seed, 3).random((b.P, b.max_poles)), device=DEV)


def _spread_theta(case, rows, seed):
    """One relaxation time in each N-th of the box (its middle half)."""
    lo, hi = _box(case)
    N = case["N"]
    return torch.tensor(lo + (hi - lo) * (np.arange(N) + 0.25 + 0.5 * _gen(seed, 3).random((rows, N))) / N, device=DEV)


def _hn_params(M, seed):
    p, einf, _ = _hn_draw(M, _gen(seed, 2))
    prm = np.zeros((M, D.PARAM_STRIDE))
    prm[:, 0], prm[:, 1:5] = einf, p[:, 0]
    return torch.tensor(prm, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, seed=int(seed) % (1 << 31))
    if kind == "targets":
        p, einf, terms = _hn_draw(case["M"], _gen(seed, 1))
        prm = np.zeros((case["M"], D.PARAM_STRIDE))
        prm[:, 0], prm[:, 1], prm[:, 2:14], prm[:, 14] = einf, terms, p.reshape(-1, 12), 0.01
        f_off = _offsets(np.full(case["M"], case["F"]))
        om = torch.tensor(np.tile(_grid(case, case["F"]), case["M"]), device=DEV)
        s["batch"] = D.Batch(f_off, np.arange(case["M"] + 1), np.ones(case["M"]), om, om, om, DEV)
        s["materials"] = torch.full((case["M"],), 6, dtype=torch.int8, device=DEV)
        s["params"] = torch.tensor(prm, device=DEV)
        return s
    if kind == "curves":
        s["omega"] = torch.tensor(_grid(case, case["F"]), device=DEV)
        s["theta"] = _spread_theta(case, case["M"], seed)
        return s
    if kind == "train":
        M = case["M"]
        f_off, om, er, ei = _spectra(case, seed)
        s["batch"] = b = D.Batch(f_off, _offsets(np.full(M, case["P"])), np.full(M, case["N"]), om, er, ei, DEV)
        s["plan"] = D.Plan(b, target_grads=True)
        s["params"] = _hn_params(M, seed)
        s["materials"] = torch.full((M,), 1, dtype=torch.int8, device=DEV)
        s["theta"] = _spread_theta(case, b.P, seed)
        return s
    s["batch"] = b = _batch(case, seed)
    s["lb"], s["ub"] = _box_tensors(case)
    if kind == "polish":
        s["theta"] = _spread_theta(case, b.P, seed)
        s["polish"] = D.Polish(b, case["N"], steps=case["steps"])
        return s
    s["plan"] = D.Plan(b)
    if kind == "fit":
        s["swarm"] = D.Swarm.empty(b.P, b.M, b.max_poles, case["iters"] + 1, DEV)
    elif kind == "search":
        x = _uniform_theta(case, b, seed)
        cost = torch.tensor(1.0 + _gen(seed, 4).random(b.P), device=DEV) * (b.eps_re.square().mean() * case["F"] * 1e-2)
        if case["opt"] == "pso":
            s["swarm"] = sw = D.Swarm.empty(b.P, b.M, b.max_poles, 8, DEV)
            sw.x.copy_(x)
            sw.v.copy_(_uniform_theta(case, b, seed + 1) - x)
            sw.pbest_x.copy_(x)
            sw.pbest_cost.fill_(math.inf)
            sw.gbest_cost.fill_(math.inf)
            sw.gbest_idx.fill_(-1)
        else:
            s["pop"] = pop = D.Population.empty(b.P, b.M, b.max_poles, 8, DEV)
            pop.x.copy_(x)
            pop.fit.copy_(cost)
            pop.best_cost.fill_(math.inf)
            pop.best_idx.fill_(-1)
        s["cost"] = cost
        s["out"] = (torch.empty_like(cost), None, None, torch.empty(b.P, dtype=torch.int8, device=DEV))
    else:
        s["theta"] = _spread_theta(case, b.P, seed)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case, kind, seed = s["case"], s["case"]["kind"], s["seed"]
    if kind == "targets":
        return D.material_eval(s["materials"], s["params"], s["batch"], noise_seed=seed)
    if kind == "curves":
        return D.basis(s["omega"], s["theta"], case["N"])
    b = s["batch"]
    if kind == "fit":
        sw = s["swarm"]
        cost = D.pso_run(s["plan"], b, s["lb"], s["ub"], sw, case["iters"], seed=seed)
        return sw.gbest_x, sw.gbest_cost, sw.gbest_idx, sw.history, cost
    if kind == "search":
        lb, ub, out = s["lb"], s["ub"], s["out"]
        if case["opt"] == "pso":
            sw = s["swarm"]
            D.pso_step(b, lb, ub, sw, 3, True, s["cost"], seed=seed)
            D.fit_eval(s["plan"], b, sw.x, want_weights=False, out=out)
            return sw.x, sw.v, sw.gbest_cost, out[0], out[3]
        pop = s["pop"]
        if case["opt"] == "de":
            D.de_trial(b, lb, ub, pop, 3, seed=seed)
            D.fit_eval(s["plan"], b, pop.u, want_weights=False, out=out)
            D.de_select(b, pop, 3, pop.u, out[0])
        else:
            D.da_visit(b, lb, ub, pop, 3, seed=seed)
            D.fit_eval(s["plan"], b, pop.u, want_weights=False, out=out)
            D.da_accept(b, pop, 3, pop.u, out[0], seed=seed)
        return pop.x, pop.fit, pop.best_cost, out[0], out[3]
    if kind == "grad":
        cost, g, _, _, st = D.fit_eval_grad(s["plan"], b, s["theta"])
        return cost, g, st
    if kind == "train":
        prm, th = s["params"].clone().requires_grad_(True), s["theta"].clone().requires_grad_(True)
        er, ei = D.HNTarget.apply(prm, s["materials"], b)
        cost = D.DebyeCost.apply(th, er, ei, s["plan"], b)
        cost.sum().backward()
        return cost.detach(), th.grad, prm.grad
    if kind == "polish":
        theta = s["theta"].clone()
        hist = torch.empty((b.M, case["steps"] + 1), dtype=torch.float64, device=DEV)
        s["polish"].run(b, theta, s["lb"], s["ub"], cost_hist=hist)
        return theta, hist
    cost, w, einf, st = D.fit_eval(s["plan"], b, s["theta"])
    return cost, w, einf, st, D.afe(b, s["theta"], w, einf)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _eval_flops(F, N):
    """One cost evaluation, basis counted once."""
    return F * (N * N + 13 * N + 5) + N ** 3 / 3 + 2 * N * N


def _search_flops(case):
    F, N, P = (a.astype(float) for a in _shape(case))
    return float(np.sum(P * _eval_flops(F, N)))


def work(case):
    kind, M, F = case["kind"], case["M"], case["F"]
    N, P = case.get("N", 1), case.get("P", 1)
    ev = _eval_flops(F, N)
    if kind == "fit":
        return dict(flops=M * P * (case["iters"] + 1) * ev, bytes=24.0 * M * F + 8.0 * M * (P + N + case["iters"] + 1))
    if kind == "search":
        Fm, Nm, Pm = (a.astype(float) for a in _shape(case))
        # spectra; positions (and velocities, personal bests) in and out; cost
        return dict(flops=_search_flops(case), bytes=24 * float(Fm.sum()) + float((Pm * (40 * Nm + 25)).sum()))
    if kind == "grad":
        # the adjoint's further terms: 18 N + 8 a point
        return dict(flops=M * P * (ev + F * (18 * N + 8)), bytes=24.0 * M * F + M * P * (16.0 * N + 9))
    if kind == "train":
        # targets and Jacobian 300 a point; forward, adjoint and target sums
        return dict(flops=M * P * (ev + F * (26 * N + 16)) + 320.0 * M * F,
                    bytes=8.0 * M * F + M * P * (16.0 * N + 8) + 256.0 * M)
    if kind == "polish":
        # the starting gradient, then a full step and a gradient each
        return dict(flops=M * (2 * case["steps"] + 1) * (ev + F * (9 * N + 4)),
                    bytes=24.0 * M * F + M * (16.0 * N + 8 * (case["steps"] + 1)))
    if kind == "targets":
        # about 100 operations an HN term (two of three on average), 100 the noise
        return dict(flops=300.0 * M * F, bytes=24.0 * M * F + 128.0 * M)
    if kind == "report":
        return dict(flops=M * (ev + F * (9 * N + 8)), bytes=24.0 * M * F + M * (16.0 * N + 25))
    return dict(flops=8.0 * M * N * F, bytes=16.0 * M * N * F + 8 * F + 8.0 * M * N)


# ---------------------------------------------------------------------------
# the same in plain 64-bit arithmetic
# ---------------------------------------------------------------------------
def _fit64(omega, er, ei, tau):
    """Weights, eps_inf and cost of tau [C][N] on spectra [C][F] (damped least
    squares on eps'' by QR, signs flipped, eps_inf the mean)."""
    x = omega[:, :, None] * tau[:, None, :]
    R = 1 / (1 + x * x)
    I = x * R
    A = torch.cat([I, math.sqrt(DAMPING) * torch.diag_embed(I.square().sum(1).sqrt())], 1)
    y = torch.cat([ei, torch.zeros_like(tau)], 1)
    q, r = torch.linalg.qr(A)
    z = torch.linalg.solve_triangular(r, q.mT @ y[:, :, None], upper=True)
    w = z.abs()
    model = (R @ w)[:, :, 0]
    einf = (er - model).mean(1)
    cost = (er - einf[:, None] - model).square().sum(1) + (ei - (I @ w)[:, :, 0]).square().sum(1)
    return w[:, :, 0], einf, cost, R, I


def _philox(k, mat, seed):
    """The first two words of Philox4x64-10 (Salmon et al. 2011) at counter (k, 0, 0, 2), key (seed, mat)."""
    lo32 = 0xFFFFFFFF

    def signed(v):
        return v - (1 << 64) if v >= 1 << 63 else v

    def mul(a, v):
        al, ah, bl, bh = a & lo32, (a >> 32) & lo32, v & lo32, (v >> 32) & lo32
        m0, m1, m2 = al * bl, ah * bl, al * bh
        c = ((m0 >> 32) & lo32) + (m1 & lo32) + (m2 & lo32)
        return ah * bh + ((m1 >> 32) & lo32) + ((m2 >> 32) & lo32) + (c >> 32), a * signed(v)

    c = [k, torch.zeros_like(k), torch.zeros_like(k), torch.full_like(k, 2)]
    k0, k1 = torch.full_like(k, seed), mat.clone()
    for _ in range(10):
        ha, la = mul(c[0], 0xD2E7470EE14C6C93)
        hb, lb = mul(c[2], 0xCA5A826395121157)
        c = [hb ^ c[1] ^ k0, lb, ha ^ c[3] ^ k1, la]
        k0, k1 = k0 + signed(0x9E3779B97F4A7C15), k1 + signed(0xBB67AE8584CAA73B)
    return [((v >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53 for v in c[:2]]


def exact(case, seed):
    kind, M, F = case["kind"], case["M"], case["F"]
    if kind == "curves":
        x = torch.tensor(_grid(case, F), device=DEV) * (10.0 ** _spread_theta(case, M, seed))[:, :, None]
        return 1 / (1 + x * x), x / (1 + x * x)
    if kind == "targets":
        p, einf, terms = (torch.tensor(a, device=DEV) for a in _hn_draw(M, _gen(seed, 1)))
        om = torch.tensor(_grid(case, F), device=DEV)
        er, ei = torch.empty(M * F, dtype=torch.float64, device=DEV), torch.empty(M * F, dtype=torch.float64, device=DEV)
        for a in range(0, M * F, 1 << 21):
            g = torch.arange(a, min(M * F, a + (1 << 21)), device=DEV)
            m, k = g // F, g % F
            e = _hn_sum(om[k], m, p, einf, terms)
            u1, u2 = _philox(k, m, int(seed) % (1 << 31))
            rad = (-2 * torch.log(1 - u1)).sqrt()
            er[g] = e.real * (1 + 0.01 * rad * torch.cos(2 * math.pi * u2))
            ei[g] = -e.imag * (1 + 0.01 * rad * torch.sin(2 * math.pi * u2))
        return er, ei
    if kind in ("fit", "search", "polish"):
        return None   # a search's state depends on comparisons of costs, a polish on its line searches
    C = M * case.get("P", 1)
    N = case["N"]
    if C * F * N * N > 1.2e9 or (kind == "train" and C * F * N * N > 6e8):
        return None
    th = _spread_theta(case, C, seed).cpu()
    om = torch.tensor(_grid(case, F))
    per = case.get("P", 1)
    if kind != "train":
        er, ei = (e.cpu().view(M, F) for e in _spectra(case, seed)[2:])
    if kind == "report":
        cost, w, einf, afe = [], [], [], []
        for m in range(0, M, 64):
            t = slice(m, m + 64)
            wi, e, c, R, I = _fit64(om[None].expand(len(th[t]), F), er[t], ei[t], 10.0 ** th[t])
            mr, mi = e[:, None] + (R @ wi[:, :, None])[:, :, 0], (I @ wi[:, :, None])[:, :, 0]
            cost.append(c)
            w.append(wi)
            einf.append(e)
            afe.append(100 * (((er[t] - mr).abs() / er[t].abs()).mean(1) + ((ei[t] - mi).abs() / ei[t].abs()).mean(1)))
        return torch.cat(cost), torch.cat(w), torch.cat(einf), None, torch.cat(afe)
    cost, g_th = [], []
    if kind == "grad":
        for a in range(0, C, 64):
            t = th[a:a + 64].clone().requires_grad_(True)
            m = torch.arange(a, a + len(t)) // per
            c = _fit64(om[None].expand(len(t), F), er[m], ei[m], 10.0 ** t)[2]
            c.sum().backward()
            cost.append(c.detach())
            g_th.append(t.grad)
        return torch.cat(cost), torch.cat(g_th), None
    prm = _hn_params(M, seed).cpu().requires_grad_(True)
    for m in range(M):
        t = th[m * per:(m + 1) * per].clone().requires_grad_(True)
        q = prm[m]
        e = q[0] + q[1] * (1 + torch.complex(torch.zeros_like(om), om * q[2]) ** q[3]) ** (-q[4])
        c = _fit64(om[None].expand(per, F), e.real[None].expand(per, F), -e.imag[None].expand(per, F), 10.0 ** t)[2]
        c.sum().backward()
        cost.append(c.detach())
        g_th.append(t.grad)
    return torch.cat(cost), torch.cat(g_th), prm.grad
