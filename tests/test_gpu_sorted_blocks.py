"""Column-sorted blocks at the sizes where their kernel can go wrong: a block
of one row, rows at the limits of the replicated row sums (a row of 256
entries or more that dominates its block) and of the sorted blocks (2^15
entries), blocks whose first entry is not aligned to the kernel's 32-entry
lines, empty rows and columns, blocks large enough for 512 threads.  Each
trajectory agrees with the oracle's at the same step size to 1e-10, the bound
of the other FP64 trajectory tests (both sides round the same sums in another
order)."""
import numpy as np
import pytest
import scipy.sparse as sp

import lpgen
import oracle
from oracle import core

pytestmark = pytest.mark.gpu

halp = pytest.importorskip("paper_2407_16144_amd")
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _lp(lens, n, seed, m_eq=None):
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(n, L, replace=False)) for L in lens]
    col = np.concatenate(cols).astype(np.int32)
    val = rng.standard_normal(col.size)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    m = len(lens)
    m_eq = (3 * m) // 4 if m_eq is None else m_eq
    xs = rng.uniform(1.0, 9.0, n)
    kx = sp.csr_matrix((val, col, rp), shape=(m, n)) @ xs
    rhs = np.concatenate([kx[:m_eq], kx[m_eq:] - rng.uniform(0.0, 1.0, m - m_eq)])
    return lpgen.LP(n, m_eq, m - m_eq, rp, col, val, rng.standard_normal(n), rhs, np.zeros(n), np.full(n, 10.0))


CASES = {
    "one row": lambda: _lp([300], 301, 1, m_eq=1),
    "one entry per row": lambda: _lp([1] * 33, 40, 2),
    "copies 255": lambda: _lp([255] + [3] * 30, 600, 3),
    "copies 256": lambda: _lp([256] + [3] * 30, 600, 4),
    "copies in a wide block": lambda: _lp([3] * 500 + [2000] + [2] * 700, 2500, 5),
    "row of 2^15": lambda: _lp([7] * 100 + [1 << 15] + [5] * 50, 40000, 6),
    "row of 2^15 + 1": lambda: _lp([7] * 100 + [(1 << 15) + 1] + [5] * 50, 40000, 7),
    "empty rows and columns": lambda: _lp([0, 0, 31, 0, 1, 33, 0] * 12 + [0], 500, 8),
    "512 threads": lambda: _lp(list(np.random.default_rng(9).integers(200, 420, 8000)), 60000, 9),
}


@pytest.mark.parametrize("name", list(CASES))
def test_sorted_block_trajectory(name):
    lp = CASES[name]()
    print(f"case sorted block {name} m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
    P = core.scaled_problem(lp)
    s, _ = oracle.power_iteration(P.K, 0, max_iters=30)
    eta = 0.9 / s
    opt = halp.lp_default_options(eta=eta)
    res, x, y, _ = halp.solve_lp(lp, tol=0.0, max_iter=130, opt=opt)
    ref = oracle.solve(lp, oracle.Options(tol=0.0, max_iter=130, eta=eta))
    assert res["iters"] == ref.iters and res["restarts"] == ref.restarts
    for a, b in ((x, ref.x), (y, ref.y)):
        floor = max(1e-2 * float(np.max(np.abs(b))), 1e-300)
        assert float(np.max(np.abs(a - b) / np.maximum(np.abs(b), floor))) <= 1e-10


@pytest.mark.parametrize("blocks", ["from the start", "cut again while running"])
def test_batch_sorted_together(blocks):
    """The blocks of a whole batch are sorted together: LPs of unequal column
    counts (another number of row bits and column bits each), one without
    entries, one of a single entry, one whose long row stays out of the sort.
    With LPs that finish early the rest are cut into smaller blocks, again
    together.  Every LP agrees with its solve alone to 1e-10 (the same sums in
    another order)."""
    rng = np.random.default_rng(21)
    lps = [_lp(list(rng.integers(0, 30, 700)), 90, 10), _lp([0, 0, 0], 5, 11), _lp([1], 1, 12, m_eq=1),
           _lp([7] * 100 + [(1 << 15) + 1] + [5] * 50, 40000, 13), _lp(list(rng.integers(1, 9, 2500)), 70000, 14)]
    n = len(lps)
    group = list(lps)
    if blocks != "from the start":
        one = dict(n=1, m_eq=1, m_ineq=0, rowptr=np.array([0, 1], np.int32), col=np.array([0], np.int32),
                   val=np.array([1.0]), c=np.array([1.0]), rhs=np.array([1.0]), lb=np.zeros(1), ub=np.full(1, 10.0))
        group += [lpgen.LP(**one) for _ in range(40)]
    opt = halp.lp_default_options(eta=1e-2)
    print(f"case batch sorted together, {blocks}", flush=True)
    h = halp.lp_batch_create(group, opt=opt)
    try:
        halp.lp_batch_solve(h, 1e-13, 400)
        got = [(halp.lp_batch_status(h, i).as_dict(), *halp.lp_batch_get_solution(h, i, group[i].n, group[i].m))
               for i in range(n)]
    finally:
        halp.lp_batch_destroy(h)
    for lp, (res, x, y) in zip(lps, got):
        ref, xr, yr, _ = halp.solve_lp(lp, tol=1e-13, max_iter=400, opt=opt)
        assert res["status"] == ref["status"] and res["iters"] == ref["iters"] and res["restarts"] == ref["restarts"]
        for a, b in ((x, xr), (y, yr)):
            floor = max(1e-2 * float(np.max(np.abs(b))), 1e-300)
            assert float(np.max(np.abs(a - b) / np.maximum(np.abs(b), floor))) <= 1e-10


RESIDENT = {
    "one entry": lambda: _lp([1], 1, 30, m_eq=1),
    "256 rows, 2048 entries": lambda: _lp([8] * 256, 256, 31),
    "2049 entries": lambda: _lp([8] * 255 + [9], 256, 32),
    "257 rows": lambda: _lp([3] * 257, 200, 33),
    "one dominant row": lambda: _lp([900] + [1] * 50, 1000, 34),
    "1024 rows, 8192 entries": lambda: _lp([8] * 1024, 1024, 35),
    "8193 entries": lambda: _lp([8] * 1023 + [9], 1024, 36),
    "1025 columns": lambda: _lp([4] * 300, 1025, 37),
    "empty rows and columns": lambda: _lp([0, 0, 31, 0, 1, 33, 0] * 12 + [0], 500, 38),
}


@pytest.mark.parametrize("method", ["r2hpdhg", "rhpdhg", "rapdhg"])
@pytest.mark.parametrize("name", list(RESIDENT))
def test_small_lp_on_one_cu(name, method):
    """LPs at the limits of the kernel that steps a small LP on one CU (rows and
    entries per workgroup size, one past each), and the same LPs in the kernels
    per product (a timed engine keeps to them): each agrees with the oracle's
    trajectory to 1e-10."""
    if method != "r2hpdhg" and name not in ("257 rows", "one dominant row"):
        pytest.skip("methods differ in the row functions, which all sizes share")
    lp = RESIDENT[name]()
    print(f"case small LP {name} {method} m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
    P = core.scaled_problem(lp)
    s, _ = oracle.power_iteration(P.K, 0, max_iters=30)
    eta = 0.9 / s
    code = {"rhpdhg": 0, "r2hpdhg": 1, "rapdhg": 2}[method]
    ref = oracle.solve(lp, oracle.Options(tol=0.0, max_iter=330, eta=eta, method=method))
    for profile in (0, 1):
        opt = halp.lp_default_options(eta=eta, method=code, profile=profile)
        res, x, y, _ = halp.solve_lp(lp, tol=0.0, max_iter=330, opt=opt)
        assert res["iters"] == ref.iters and res["restarts"] == ref.restarts
        for a, b in ((x, ref.x), (y, ref.y)):
            floor = max(1e-2 * float(np.max(np.abs(b))), 1e-300)
            assert float(np.max(np.abs(a - b) / np.maximum(np.abs(b), floor))) <= 1e-10


def test_small_lps_joined_by_a_large_one():
    """A server steps small LPs on one CU each until a larger LP joins them
    (their blocks are then cut for shared launches) and again once it has
    retired: every LP ends as it does alone, and the optimal ones meet their
    tolerance as the oracle measures it."""
    small = [lpgen.scaled_powerlaw(40 + i, 150 + 60 * i, 400 + 100 * i) for i in range(5)]
    big = lpgen.scaled_powerlaw(50, 4000, 12000)
    print("case small LPs joined by a large one", flush=True)
    lps = small[:3] + [big] + small[3:]
    h = halp.lp_server_create(1 << 30, 8)
    try:
        tickets = [halp.lp_server_submit(h, lp, 1e-6, 200_000, 0.0) for lp in lps[:3]]
        halp.lp_server_step(h, 1)
        tickets += [halp.lp_server_submit(h, lp, 1e-6, 200_000, 1.0) for lp in lps[3:]]
        open_ = set(range(len(lps)))
        for _ in range(10_000):
            halp.lp_server_step(h, 4)
            for k in sorted(open_):
                r, _t = halp.lp_server_poll(h, tickets[k])
                if r is None:
                    continue
                x, y = halp.lp_server_get_solution(h, tickets[k], lps[k].n, lps[k].m)
                halp.lp_server_release(h, tickets[k])
                open_.discard(k)
                kkt, parts = oracle.rel_kkt(lps[k], x, y)
                alone, *_ = halp.solve_lp(lps[k], tol=1e-6, max_iter=200_000)
                assert r.status == alone["status"], k
                assert r.status != halp.LP_OPTIMAL or kkt <= 1e-6 * (1 + 1e-6), (k, parts)
            if not open_:
                break
        assert not open_
    finally:
        halp.lp_server_destroy(h)
