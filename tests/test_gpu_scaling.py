"""The stored K~ is rounded as the oracle's: every pass divides each entry by
its row's factor and then by its column's.  Ruiz passes take only largest
entries, roots and quotients, all correctly rounded on both sides, so K~ equals
the oracle's bit for bit, and its transpose too.  The Pock-Chambolle pass sums
rows of N entries in another order than the oracle: either sum is within N
rounding errors of the true one, so their roots are within N of each other; the
powers of alpha = 0.5 (one unit each) add 2 per root, roots and quotients 8 in
all, and K~ is within N_row + N_col + 16 rounding errors of the oracle's.  Cases: tiles of one row and of 256,
full and just overfull tiles of 1024 entries, rows with a block of their own,
empty rows and columns, a single entry, both precisions."""
import numpy as np
import pytest
import scipy.sparse as sp

import lpgen
import oracle

pytestmark = pytest.mark.gpu

halp = pytest.importorskip("paper_2407_16144_amd")
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

ROW_ORDER = dict(plain_sort=0, slice_sort=0, slice_min_bytes=-1)


def _lp(seed, n, counts):
    """Row i holds counts[i] entries over six decades in random columns."""
    rng = np.random.default_rng(seed)
    m = len(counts)
    col = np.concatenate([np.sort(rng.choice(n, c, replace=False)) for c in counts]).astype(np.int32)
    val = rng.choice([-1.0, 1.0], col.size) * 10.0 ** rng.uniform(-3, 3, col.size)
    return lpgen.LP(n=n, m_eq=m // 2, m_ineq=m - m // 2,
                    rowptr=np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), col=col, val=val,
                    c=rng.normal(size=n), rhs=rng.normal(size=m), lb=np.zeros(n), ub=np.full(n, 10.0))


def _ragged():
    return _lp(21, 3000, [0, 1, 1023, 1, 1024, 0, 1025, 3000, 2, 4] + [4] * 600 + [0] * 300 + [1] * 257)


CASES = {"single entry": lambda: _lp(22, 3, [1]), "ragged": _ragged,
         "powerlaw 3k x 9k": lambda: lpgen.scaled_powerlaw(11, 3000, 9000)}


def _stored(lp, **kw):
    h = halp.lp_create(lp.n, lp.m_eq, lp.m_ineq, lp.rowptr, lp.col, lp.val, lp.c, lp.rhs, lp.lb, lp.ub,
                       opt=halp.lp_default_options(**ROW_ORDER, **kw))
    try:
        return halp.lp_get_scaled_matrix(h, 0, lp.m, lp.nnz)[2], halp.lp_get_scaled_matrix(h, 1, lp.n, lp.nnz)[2]
    finally:
        halp.lp_destroy(h)


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("passes,alpha", [(0, 0.0), (1, 0.0), (2, 0.0), (10, 0.0), (0, 1.0), (10, 1.0), (3, 0.5)])
@pytest.mark.parametrize("name", list(CASES))
def test_scaled_values_equal_oracle(name, passes, alpha, fp32):
    lp = CASES[name]()
    print(f"case scaling {name} passes {passes} alpha {alpha} fp32 {fp32}", flush=True)
    k = sp.csr_matrix((lp.val, lp.col, lp.rowptr), shape=(lp.m, lp.n))
    ref, _, _ = oracle.scale(k, passes, alpha if alpha > 0 else None)
    v, vt = _stored(lp, ruiz_iters=passes, pc_alpha=alpha,
                    precision=halp.LP_PREC_FP32 if fp32 else halp.LP_PREC_FP64)
    kt = ref.T.tocsr()
    kt.sort_indices()
    if alpha == 0.0:
        assert np.array_equal(v, ref.data) and np.array_equal(vt, kt.data)
        return
    per_row, per_col = np.diff(lp.rowptr), np.bincount(lp.col, minlength=lp.n)
    bound = np.repeat(per_row, per_row) + per_col[lp.col] + 16
    assert np.all(np.abs(v - ref.data) <= bound * 2.0 ** -53 * np.abs(ref.data))
    assert np.array_equal(vt, sp.csr_matrix((v, lp.col, lp.rowptr), shape=k.shape).T.tocsr().data)
