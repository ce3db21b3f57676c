"""Layouts of the step kernels that depend on how a matrix's entries are
spread: sorted groups split because their entries crowd into few column
slices, and blocks cut by the entries of few long rows; column-sorted blocks
of small LPs in the kernels per product; the power iteration over either
layout.  Each trajectory
agrees with the oracle's at the same step size to 1e-10, the bound of the
other FP64 trajectory tests (both sides round the same sums in another
order)."""
import numpy as np
import pytest
import scipy.sparse as sp

import lpgen
import oracle
from oracle import core

from test_gpu_sorted_blocks import CASES as BLOCKS

pytestmark = pytest.mark.gpu

halp = pytest.importorskip("paper_2407_16144_amd")
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _lp(rows, cols, m, n, seed):
    rng = np.random.default_rng(seed)
    a = sp.csr_matrix((rng.standard_normal(rows.size), (rows, cols)), shape=(m, n))
    a.sum_duplicates()
    a.sort_indices()
    m_eq = (3 * m) // 4
    kx = a @ rng.uniform(1.0, 9.0, n)
    rhs = np.concatenate([kx[:m_eq], kx[m_eq:] - rng.uniform(0.0, 1.0, m - m_eq)])
    return lpgen.LP(n, m_eq, m - m_eq, a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data,
                    rng.standard_normal(n), rhs, np.zeros(n), np.full(n, 10.0))


def _band(m, n, per_row, width, seed):
    """Columns within `width` of the diagonal."""
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(m), per_row)
    cols = np.clip(rows * n // m + rng.integers(-width // 2, width // 2, rows.size), 0, n - 1)
    return _lp(rows, cols, m, n, seed + 1)


def _uniform(lens, n, seed):
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(len(lens)), lens)
    return _lp(rows, rng.integers(0, n, rows.size), len(lens), n, seed + 1)


CASES = {
    # 8 slices whatever the width: a group's entries lie in one or two of them
    "banded groups": (lambda: _band(20000, 40000, 40, 400, 1), dict(slice_min_bytes=0)),
    "banded groups in one pair of slices": (lambda: _band(40000, 20000, 30, 16000, 2), dict(slice_min_bytes=0)),
    "few long rows": (lambda: _uniform([1500] * 150 + [5000, 30000], 60000, 3), {}),
    "few long columns": (lambda: _uniform([12] * 20000, 150, 4), {}),
    # more than 512 blocks of at most 128 rows: the 128-thread kernel; one row
    # more, or 512 blocks, the other one
    "many small blocks": (lambda: _uniform([7] * 20000 + [3000] * 3, 70000, 5), dict(sort_rows=128)),
    "many blocks of 129 rows": (lambda: _uniform([7] * 20000, 70000, 6), dict(sort_rows=129)),
    "512 blocks": (lambda: _uniform([4] * 512, 512, 7), dict(sort_rows=1)),
    "513 blocks": (lambda: _uniform([4] * 513, 513, 8), dict(sort_rows=1)),
    # more than 32 groups per CU of less than a batch of entries
    "many small groups": (lambda: _uniform([5] * 33000, 34000, 9), dict(sort_rows=32, slice_min_bytes=0)),
}


def _agrees(got, ref):
    for a, b in zip(got, ref):
        floor = max(1e-2 * float(np.max(np.abs(b))), 1e-300)
        assert float(np.max(np.abs(a - b) / np.maximum(np.abs(b), floor))) <= 1e-10


@pytest.mark.parametrize("name", list(CASES))
def test_trajectory(name):
    make, options = CASES[name]
    lp = make()
    print(f"case layout {name} m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
    P = core.scaled_problem(lp)
    s, _ = oracle.power_iteration(P.K, 0, max_iters=30)
    eta = 0.9 / s
    res, x, y, _ = halp.solve_lp(lp, tol=0.0, max_iter=130, opt=halp.lp_default_options(eta=eta, **options))
    ref = oracle.solve(lp, oracle.Options(tol=0.0, max_iter=130, eta=eta))
    assert res["iters"] == ref.iters and res["restarts"] == ref.restarts
    _agrees((x, y), (ref.x, ref.y))


@pytest.mark.parametrize("name", list(BLOCKS))
def test_sorted_blocks_of_a_timed_engine(name):
    """The blocks of test_gpu_sorted_blocks in the kernels per product: a timed
    engine keeps its small LPs in them, which otherwise step on one CU."""
    lp = BLOCKS[name]()
    print(f"case timed sorted block {name} m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
    P = core.scaled_problem(lp)
    s, _ = oracle.power_iteration(P.K, 0, max_iters=30)
    eta = 0.9 / s
    res, x, y, _ = halp.solve_lp(lp, tol=0.0, max_iter=130, opt=halp.lp_default_options(eta=eta, profile=1))
    ref = oracle.solve(lp, oracle.Options(tol=0.0, max_iter=130, eta=eta))
    assert res["iters"] == ref.iters and res["restarts"] == ref.restarts
    _agrees((x, y), (ref.x, ref.y))


def _holes(m, n, per_row, long_row, seed):
    """Empty rows and columns, and one row of `long_row` entries."""
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(1, m, 3), per_row)
    cols = rng.integers(0, n // 2, rows.size) * 2
    extra = rng.choice(n // 2, long_row, replace=False) * 2
    return _lp(np.concatenate([rows, np.full(long_row, 2)]), np.concatenate([cols, extra]), m, n, seed + 1)


POWER = {
    # (LPs of one add, options): K^T of more than 512 tiles in all, so that the
    # power iteration runs on the layouts of the steps
    "sorted blocks, copies, holes": (lambda: [_holes(6000, 150000, 60, 20000, 11)], {}),
    "a row of its own beside sorted blocks": (lambda: [_holes(6000, 150000, 60, 40000, 12)], {}),
    "more than 512 blocks": (lambda: [_uniform([20] * (1500 + 40 * i), 6000 + 100 * i, 20 + i) for i in range(40)], {}),
    "groups of few rows": (lambda: [_uniform([12] * 20000, 140000, 13)], dict(slice_min_bytes=65536)),
    "groups, split": (lambda: [_band(20000, 140000, 60, 2000, 14)], dict(slice_min_bytes=65536)),
    "groups beside blocks and tiles": (lambda: [_holes(6000, 90000, 60, 40000, 15), _uniform([12] * 20000, 90000, 16),
                                               _uniform([3] * 50, 100, 17)], dict(slice_min_bytes=65536)),
    "groups and blocks, more than 512": (lambda: [_uniform([12] * 20000, 90000, 30)] +
                                         [_uniform([20] * 1500, 6000, 31 + i) for i in range(40)],
                                         dict(slice_min_bytes=65536)),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(POWER))
def test_power_iteration(name, precision):
    """sigma_hat of every LP of an add to 1e-10 of the oracle's (the same
    iterates; the row sums are added in another order), after as many
    iterations; the FP32 engine computes it in FP64 too."""
    make, options = POWER[name]
    lps = make()
    print(f"case power {name} precision={precision} nnz={[lp.nnz for lp in lps][:4]}", flush=True)
    h = halp.lp_batch_create(lps, opt=halp.lp_default_options(precision=precision, **options))
    try:
        got = [halp.lp_batch_status(h, i) for i in range(len(lps))]
    finally:
        halp.lp_batch_destroy(h)
    for lp, r in zip(lps, got):
        s, iters = oracle.power_iteration(core.scaled_problem(lp).K, 0)
        assert r.sigma_hat == pytest.approx(s, rel=1e-10)
        assert r.power_iters == iters
