"""Workloads of the solver at the sizes and options it is used with, each one
a whole call from a user's program: create a handle from the LP, run a fixed
budget of iterations (tolerance 0, so that the work does not depend on the
rounding of a stopping test), fetch the solution, destroy the handle.

listed() names the workloads, draw() gives others of the same ranges,
prepare() makes an LP's arrays (and a server's handle), run() is one pass,
work() its unavoidable bytes and operations, exact() the same iterates by
plain torch in FP64.
"""
import math

import numpy as np
import torch

import paper_2407_16144_amd as halp

METHODS = {"r2hpdhg": halp.LP_METHOD_R2HPDHG, "rhpdhg": halp.LP_METHOD_RHPDHG, "rapdhg": halp.LP_METHOD_RAPDHG}
CHECK = 64          # iterations between checks (the library's default)
LONGEST_ROW = 5000  # of the power-law row lengths


def _single(name, m, n, per_col, budget, method="r2hpdhg", precision="fp64", how="device", fixed_order=False):
    return {"name": name, "kind": "single", "m": m, "n": n, "per_col": per_col, "budget": budget, "method": method,
            "precision": precision, "how": how, "fixed_order": fixed_order}


def _many(name, kind, count, m_lo, m_hi, budget, precision="fp64"):
    return {"name": name, "kind": kind, "count": count, "m_lo": m_lo, "m_hi": m_hi, "per_col": 8.0, "budget": budget,
            "method": "r2hpdhg", "precision": precision}


def listed():
    return [
        # the smallest calls, from host arrays: a modelling layer that solves a tiny LP after another
        _single("tiny-60x120-host", 60, 120, 6.0, 1000, how="host"),
        # the allocation-free entry point of serving loops and harnesses, at a small LP
        _single("static-2kx7k", 2000, 7000, 8.0, 1000, how="static"),
        # one LP of the batched sizes alone, Algorithm 1
        _single("one-2.4kx8k-rhpdhg", 2400, 8000, 8.0, 1000, method="rhpdhg"),
        # the largest of the batched sizes alone
        _single("one-20kx70k", 20000, 70000, 8.0, 1000),
        # the large requests of the serving mix, given with 64-bit row pointers
        _single("one-100kx400k-int64", 100_000, 400_000, 10.0, 1000, how="device64"),
        # the same in the bit-reproducible layouts (fixed-order sums)
        _single("fixed-order-100kx400k", 100_000, 400_000, 10.0, 640, fixed_order=True),
        # the large LP: its matrices just about fill the last-level cache
        _single("large-200kx1M", 200_000, 1_000_000, 9.77, 1500),
        # the mixed-size LP of the default benchmark, far beyond the caches
        _single("mixed-500kx2M", 500_000, 2_000_000, 14.8, 1300),
        # the same in mixed precision: a tenth of the budget in FP32, the rest in FP64
        _single("mixed-500kx2M-polish", 500_000, 2_000_000, 14.8, 640, precision="polish"),
        # many uneven LPs at once
        _many("batch-128", "batch", 128, 500, 20000, 1000),
        # the same in mixed precision
        _many("batch-48-polish", "batch", 48, 500, 20000, 700, precision="polish"),
        # requests from host arrays through the continuous-batching server
        _many("server-24", "server", 24, 500, 20000, 640),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "single", "single", "batch", "server"])
    if kind == "single":
        # single precision alone (a first answer of a few digits) for one check
        # only: two roundings of it agree to those digits no longer than that
        precision = rng.choice(["fp64", "fp64", "fp64", "polish", "fp32"])
        m = _log(rng, 60, 400_000)
        n = int(m * rng.uniform(2.0, 5.0)) | 1
        how = rng.choice(["device", "device", "device64", "host"] if m > 4000 else ["device", "static", "host"])
        if how == "host" and m > 50_000:
            how = "device"
        if how == "static":
            precision = "fp64"
        c = _single("", m, n, round(rng.uniform(6.0, 14.0), 2),
                    CHECK if precision == "fp32" else rng.choice([400, 640, 1000]),
                    method=rng.choice(["r2hpdhg", "r2hpdhg", "rhpdhg", "rapdhg"]) if precision == "fp64" else "r2hpdhg",
                    precision=precision, how=how, fixed_order=rng.random() < 0.15)
    elif kind == "batch":
        c = _many("", "batch", _log(rng, 3, 100), _log(rng, 100, 1000), _log(rng, 4000, 20000), rng.choice([400, 640]),
                  precision=rng.choice(["fp64", "polish"]))
    else:
        c = _many("", "server", _log(rng, 2, 24), _log(rng, 100, 1000), _log(rng, 4000, 20000), rng.choice([320, 640]))
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs


class LP:
    """One LP: K = [A; G] in CSR, min c.x, A x = b, G x >= h, lb <= x <= ub."""

    def __init__(self, n, m_eq, m_ineq, rowptr, col, val, c, rhs, lb, ub):
        self.n, self.m_eq, self.m_ineq, self.m = n, m_eq, m_ineq, m_eq + m_ineq
        self.rowptr, self.col, self.val, self.c, self.rhs, self.lb, self.ub = rowptr, col, val, c, rhs, lb, ub

    def arrays(self):
        return self.rowptr, self.col, self.val, self.c, self.rhs, self.lb, self.ub

    def host(self):
        return LP(self.n, self.m_eq, self.m_ineq, *(a.cpu().numpy() for a in self.arrays()))


def _shortest(mean, longest):
    """Lower end a of the row lengths' law L^-2 on [a, longest] with this mean."""
    lo, hi = 1e-6, float(longest)
    if mean >= hi:
        return hi
    for _ in range(100):
        a = 0.5 * (lo + hi)
        if math.log(longest / a) / (1.0 / a - 1.0 / longest) < mean:
            lo = a
        else:
            hi = a
    return 0.5 * (lo + hi)


def _powerlaw(m, n, per_col, seed):
    """Power-law row lengths, uniform columns, values N(0, 1) scaled by
    10^U(-3, 3) per row, 80% of the variables boxed and 20% free, a feasible
    point and a dual one planted: the synthetic LPs of the benchmark."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rand = lambda k, lo=0.0, hi=1.0: torch.rand(k, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo
    normal = lambda k: torch.randn(k, generator=g, device="cuda", dtype=torch.float64)
    longest = min(LONGEST_ROW, n)
    a = _shortest(min(per_col * n / m, 0.5 * longest), longest)
    length = (1.0 / (1.0 / a - rand(m) * (1.0 / a - 1.0 / longest))).round().clamp(1, longest).long()
    rows = torch.repeat_interleave(torch.arange(m, device="cuda"), length)
    cols = torch.randint(0, n, (rows.numel(),), generator=g, device="cuda")
    empty = (torch.bincount(cols, minlength=n) == 0).nonzero().flatten()
    key = torch.cat([rows * n + cols, torch.randint(0, m, (empty.numel(),), generator=g, device="cuda") * n + empty])
    key = torch.unique(key)
    rows, cols = key // n, key % n
    del key
    per_row = torch.bincount(rows, minlength=m)
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(per_row, 0)
    scale = 10.0 ** rand(m, -3.0, 3.0)
    val = normal(rows.numel()) * scale[rows]
    free = rand(n) < 0.2
    ub = rand(n, 1.0, 100.0)
    xs = torch.where(free, rand(n, -50.0, 50.0), rand(n) * ub)
    lb = torch.where(free, -math.inf, 0.0).double()
    ub = torch.where(free, math.inf, ub)
    m_eq = (3 * m) // 4
    rhs = torch.segment_reduce(val * xs[cols], "sum", lengths=per_row)
    rhs[m_eq:] -= scale[m_eq:] * rand(m - m_eq)
    ys = normal(m)
    ys[m_eq:] = ys[m_eq:].abs()
    by_col = torch.argsort(cols, stable=True)
    c = torch.segment_reduce(val[by_col] * ys[rows[by_col]], "sum", lengths=torch.bincount(cols, minlength=n))
    c += torch.where(free, 0.0, normal(n))
    return LP(n, m_eq, m - m_eq, rowptr, cols.int(), val, c, rhs, lb, ub)


def _lps(case, seed):
    if case["kind"] == "single":
        return [_powerlaw(case["m"], case["n"], case["per_col"], seed)]
    rng = np.random.default_rng([case["count"], case["m_lo"], case["m_hi"]])  # the sizes are the case's own
    ms = np.exp(rng.uniform(math.log(case["m_lo"]), math.log(case["m_hi"]), case["count"]))
    ns = ms * rng.uniform(2.0, 5.0, case["count"])
    return [_powerlaw(int(m), int(n), case["per_col"], seed * 1000 + i) for i, (m, n) in enumerate(zip(ms, ns))]


def _options(case):
    o = {"method": METHODS[case["method"]]}
    if case["precision"] != "fp64":
        o["precision"] = halp.LP_PREC_FP32
    if case["precision"] == "fp32":
        o["polish_tol"] = 0.0
    if case.get("fixed_order"):
        o.update(plain_sort=0, slice_sort=0)
    return halp.lp_default_options(**o)


class State:
    """The inputs of a pass, and the server that takes them."""

    def __init__(self, case, lps):
        self.case, self.opt, self.server = case, _options(case), None
        how = case.get("how", case["kind"])
        self.lps = [lp.host() for lp in lps] if how in ("host", "server") else lps
        if how == "device64":
            lps[0].rowptr = lps[0].rowptr.long()
        elif how == "static":
            self.x = torch.empty(lps[0].n, dtype=torch.float64, device="cuda")
            self.y = torch.empty(lps[0].m, dtype=torch.float64, device="cuda")
        elif how == "batch":
            self.problems = (halp.lp_problem * len(lps))()
            for p, lp in zip(self.problems, lps):
                p.n, p.m_eq, p.m_ineq = lp.n, lp.m_eq, lp.m_ineq
                p.row_ptr, p.col_idx, p.val, p.c, p.rhs, p.lb, p.ub = (a.data_ptr() for a in lp.arrays())
        elif how == "server":
            self.server = halp.lp_server_create(2 << 30, 64, opt=self.opt)

    def __del__(self):
        if getattr(self, "server", None) is not None:
            halp.lp_server_destroy(self.server)


def prepare(case, seed):
    return State(case, _lps(case, seed))


# ------------------------------------------------------------------ one pass


def _answer(case, x, y, results):
    """x and y as the solver computed them: the iterates of a solve with a
    single-precision phase hold single-precision numbers."""
    if case["precision"] != "fp64":
        x, y = x.astype(np.float32), y.astype(np.float32)
    return {"x": x, "y": y, "iters": np.array([r.iters for r in results]),
            "restarts": np.array([r.restarts for r in results]), "status": np.array([r.status for r in results])}


def run(s):
    case = s.case
    budget = case["budget"]
    if case["kind"] == "batch":
        h = halp.lp_batch_create_from(s.problems, len(s.lps), True, opt=s.opt)
        try:
            halp.lp_batch_solve(h, 0.0, budget)
            results = [halp.lp_batch_status(h, i) for i in range(len(s.lps))]
            points = [halp.lp_batch_get_solution(h, i, lp.n, lp.m) for i, lp in enumerate(s.lps)]
        finally:
            halp.lp_batch_destroy(h)
        return _answer(case, np.concatenate([p[0] for p in points]), np.concatenate([p[1] for p in points]), results)
    if case["kind"] == "server":
        h = s.server
        tickets = [halp.lp_server_submit(h, lp, 0.0, budget, halp.lp_server_clock(h)) for lp in s.lps]
        done = {}
        while len(done) < len(tickets):
            halp.lp_server_step(h, 1)
            for t, lp in zip(tickets, s.lps):
                if t not in done:
                    r, _ = halp.lp_server_poll(h, t)
                    if r is not None:
                        done[t] = (r, *halp.lp_server_get_solution(h, t, lp.n, lp.m))
                        halp.lp_server_release(h, t)
        got = [done[t] for t in tickets]
        return _answer(case, np.concatenate([g[1] for g in got]), np.concatenate([g[2] for g in got]),
                       [g[0] for g in got])
    lp = s.lps[0]
    if case["how"] == "static":
        r = halp.lp_solve_static(lp.n, lp.m_eq, lp.m_ineq, *lp.arrays(), 0.0, budget, x=s.x, y=s.y, opt=s.opt)
        return {"x": s.x, "y": s.y, "iters": r.iters, "restarts": r.restarts, "status": r.status}
    create = halp.lp_create64 if case["how"] == "device64" else halp.lp_create
    h = create(lp.n, lp.m_eq, lp.m_ineq, *lp.arrays(), inputs_on_device=int(case["how"] != "host"), opt=s.opt)
    try:
        halp.lp_solve(h, 0.0, budget)
        r = halp.lp_status(h)
        x, y = halp.lp_get_solution(h, lp.n, lp.m)
    finally:
        halp.lp_destroy(h)
    return _answer(case, x, y, [r])


def work(case):
    """Per iteration: the values and indices of K and of its transpose once,
    c, l, u, x, x0 read and x and the extrapolated point written, the latter
    read by the second product; q, y and y0 read and y written and read; four
    operations per matrix entry."""
    if case["kind"] == "single":
        m, n, nnz = case["m"], case["n"], case["per_col"] * case["n"]
    else:
        lo, hi = case["m_lo"], case["m_hi"]
        m = case["count"] * (hi - lo) / math.log(hi / lo)
        n = 3.5 * m
        nnz = case["per_col"] * n
    s = 4 if case["precision"] == "fp32" else 8
    return {"bytes": case["budget"] * (2 * nnz * (s + 4) + s * (8 * n + 5 * m)), "flops": case["budget"] * 4 * nnz}


# ------------------------------------------------------------------ the same in plain torch


def _start_vector(n):
    """SplitMix64 outputs of stream 0 on [-1, 1): the published start of the power iteration."""
    with np.errstate(over="ignore"):
        z = np.arange(1, n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return torch.from_numpy((z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 * 2.0 - 1.0).cuda()


class Scaled:
    """Ten Ruiz passes, one Pock-Chambolle pass, the step size by power iteration."""

    def __init__(self, lp):
        m, n = lp.m, lp.n
        col = lp.col.long()
        row = torch.repeat_interleave(torch.arange(m, device="cuda"), (lp.rowptr[1:] - lp.rowptr[:-1]).long())
        v = lp.val.clone()
        self.dr, self.dc = torch.ones(m, device="cuda").double(), torch.ones(n, device="cuda").double()
        for k in range(11):
            a = v.abs()
            how = "amax" if k < 10 else "sum"
            r = torch.zeros_like(self.dr).scatter_reduce_(0, row, a, how).sqrt()
            c = torch.zeros_like(self.dc).scatter_reduce_(0, col, a, how).sqrt()
            r[r == 0], c[c == 0] = 1.0, 1.0
            v = v / r[row] / c[col]
            self.dr, self.dc = self.dr / r, self.dc / c
        order = torch.argsort(col, stable=True)
        ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
        ptr[1:] = torch.cumsum(torch.bincount(col, minlength=n), 0)
        self.A = torch.sparse_csr_tensor(lp.rowptr.int(), lp.col, v, (m, n))
        self.AT = torch.sparse_csr_tensor(ptr, row[order].int(), v[order], (n, m))
        self.c, self.q = self.dc * lp.c, self.dr * lp.rhs
        self.l, self.u = lp.lb / self.dc, lp.ub / self.dc
        self.m_eq = lp.m_eq
        w = _start_vector(n)
        w, last = w / w.norm(), None
        for t in range(1, 1001):
            w = self.KT(self.K(w))
            norm = float(w.norm())
            sigma, w = math.sqrt(norm), w / norm
            if last is not None and t >= 20 and abs(sigma - last) <= 1e-4 * sigma:
                break
            last = sigma
        self.eta = 0.9 / sigma

    # added to a zero vector: the plain product leaves now and then a NaN that
    # its uninitialised result held
    def K(self, x):
        return torch.addmv(torch.zeros_like(self.q), self.A, x)

    def KT(self, y):
        return torch.addmv(torch.zeros_like(self.c), self.AT, y)

    def iterate(self, x, y, omega, budget, reflect):
        """Restarted (reflected) Halpern PDHG from (x, y) to the first check
        at or past `budget` evaluations: T(z) there and the last weight."""
        tau, sigma = self.eta / omega, self.eta * omega
        x0, y0, k, t, epoch, r0 = x, y, 0, 0, 0, None
        while True:
            xp = torch.clamp(x - tau * (self.c - self.KT(y)), self.l, self.u)
            yp = y + sigma * (self.q - self.K(2.0 * xp - x))
            yp[self.m_eq:].clamp_(min=0.0)
            t += 1
            if k % CHECK == 0:
                dx, dy = x - xp, y - yp
                res = float(((dx @ dx) / tau + (dy @ dy) / sigma + 2.0 * (dy @ self.K(dx))).clamp(min=0.0).sqrt())
                if k == 0:
                    r0 = res
                else:
                    if t >= budget:
                        return xp, yp, omega, t
                    if epoch == 0 or res <= math.exp(-1.0) * r0 or k >= 0.36 * t:
                        far_x, far_y = float((xp - x0).norm()), float((yp - y0).norm())
                        if far_x > 1e-10 and far_y > 1e-10:
                            omega = math.exp(0.5 * math.log(far_y / far_x) + 0.5 * math.log(omega))
                        tau, sigma = self.eta / omega, self.eta * omega
                        x, y, x0, y0, k = xp, yp, xp, yp, 0
                        epoch += 1
                        continue
            w = (k + 1.0) / (k + 2.0)
            x = w * (2.0 * xp - x if reflect else xp) + (1.0 - w) * x0
            y = w * (2.0 * yp - y if reflect else yp) + (1.0 - w) * y0
            k += 1


def exact(case, seed):
    if case["method"] == "rapdhg" or case.get("count", 1) * case["budget"] > 36_000:  # no such loop here; too slow
        return None
    xs, ys = [], []
    for lp in _lps(case, seed):
        p = Scaled(lp)
        reflect = case["method"] == "r2hpdhg"
        nc, nq = float(p.c.norm()), float(p.q.norm())
        omega = nc / nq if nc > 1e-10 and nq > 1e-10 else 1.0
        x, y = torch.clamp(torch.zeros_like(p.c), p.l, p.u), torch.zeros_like(p.q)
        budget = case["budget"]
        if case["precision"] == "polish":  # the first phase may take a tenth of the budget
            x, y, omega, t = p.iterate(x, y, omega, budget // 10, reflect)
            budget -= t
        x, y, *_ = p.iterate(x, y, omega, budget, reflect)
        xs.append(p.dc * x)
        ys.append(p.dr * y)
    return {"x": torch.cat(xs), "y": torch.cat(ys), "iters": None, "restarts": None, "status": None}
