"""Device-resident batches are validated together: the first LP at fault
decides the error, wherever it stands, and the batch that is in order solves
like its LPs alone."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu

halp = pytest.importorskip("paper_2407_16144_amd")
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _lps():
    return [lpgen.scaled_powerlaw(60 + i, m, 3 * m) for i, m in enumerate([30, 700, 5, 1500])]


def _spoil(lp, what):
    lp.val, lp.col, lp.rowptr, lp.lb, lp.rhs = (np.array(a) for a in (lp.val, lp.col, lp.rowptr, lp.lb, lp.rhs))
    if what == "value":
        lp.val[-1] = np.inf
    elif what == "column":
        lp.col[-1] = lp.n
    elif what == "order":
        r = int(np.argmax(np.diff(lp.rowptr)))
        lp.col[lp.rowptr[r] + 1] = lp.col[lp.rowptr[r]]
    elif what == "rows":
        lp.rowptr[1] = lp.rowptr[-1] + 1
    elif what == "ends":
        lp.rowptr[-1] = -1
    elif what == "rhs":
        lp.rhs[0] = np.nan
    elif what == "bounds":
        lp.lb[-1] = np.inf


MESSAGE = {"value": "non-finite matrix value", "column": "in-range", "order": "strictly increasing",
           "rows": "non-decreasing", "ends": "row_ptr[m] must be >= 0", "rhs": "right-hand side", "bounds": "invalid bounds"}


def _create(lps):
    arr, keep = halp.make_problems(lps, on_device=True)
    torch.cuda.synchronize()
    return halp.lp_batch_create_from(arr, len(lps), True), keep


@pytest.mark.parametrize("what", list(MESSAGE))
@pytest.mark.parametrize("at,later", [(0, "ends"), (1, "ends"), (0, "bounds"), (1, "value"), (3, None)])
def test_first_faulty_lp_decides(what, at, later):
    """(The entry count of every LP is read before any is looked at closer, so
    a bad one decides wherever it stands.)"""
    print(f"case faulty LP {at}: {what}, later {later}", flush=True)
    lps = _lps()
    _spoil(lps[at], what)
    if later:
        _spoil(lps[3], later)
    with pytest.raises(halp.HalpError) as ei:
        _create(lps)
    assert ei.value.code == halp.LP_ERR_INVALID
    assert (MESSAGE["ends"] if "ends" in (what, later) else MESSAGE[what]) in str(ei.value)


def test_batch_in_order_is_accepted():
    print("case batch in order", flush=True)
    lps = _lps()
    h, keep = _create(lps)
    del keep
    try:
        halp.lp_batch_solve(h, 1e-6, 200_000)
        for i, lp in enumerate(lps):
            assert halp.lp_batch_status(h, i).status == halp.solve_lp(lp, tol=1e-6, max_iter=200_000)[0]["status"]
    finally:
        halp.lp_batch_destroy(h)
