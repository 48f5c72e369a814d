"""GPU tests of the pivoted FP64 LU with entries that are not finite: one rule for
every height of a panel (one work-group up to 8192 rows, the whole device above) --
the largest magnitude, a NaN counting as zero, the first among equals -- so that
every ipiv names a row on or below its pivot, and the first pivot that is zero or
not finite is reported."""
import numpy as np
import pytest
import torch

import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu
NAN, INF = float("nan"), float("inf")


def _factor(n, fill):
    prob = mxp.mxp_generate(n, 1, n, store="f64", kind=mxp.GEN_UNIFORM)
    fill(mxp.as_matrix(prob.A, n))
    A = mxp.as_matrix(prob.A, n).cpu().numpy().copy() if n <= 300 else None
    fac = mxp.mxp_lu64_factor(prob.A, n, prob.lda, True)
    ipiv = fac.ipiv.cpu().numpy()
    assert np.all(ipiv >= np.arange(n)) and np.all(ipiv < n)
    return A, fac, ipiv


def _pivots(A):
    """the rule, column by column"""
    A = A.copy()
    n = len(A)
    out = []
    with np.errstate(all="ignore"):
        for k in range(n):
            p = k + int(np.argmax(np.fmax(np.abs(A[k:, k]), 0.0)))
            out.append(p)
            A[[k, p]] = A[[p, k]]
            if A[k, k] == 0.0 or not np.isfinite(A[k, k]):
                return out, k + 1
            A[k + 1:, k] /= A[k, k]
            A[k + 1:, k + 1:] -= np.outer(A[k + 1:, k], A[k, k + 1:])
    return out, 0


# heights of the panel's forms: 16 columns at a time to 2048 rows, 8 to 4096, 4 to
# 8192, the device-wide one above (rows of its work-groups: 64, their first lanes
# at multiples of it)
@pytest.mark.parametrize("n", [12, 300, 2049, 4100, 8200, 8300])
@pytest.mark.parametrize("what", ["entry", "rows", "column", "all", "infinity"])
def test_nonfinite_entries(n, what):
    print("lu64 nonfinite", n, what, flush=True)
    col = n // 3

    def fill(A):
        if what == "entry":                 # the first row: its NaN is never a pivot before the last column
            A[0, 0] = NAN
        elif what == "rows":                # every 64th row, all of them first lanes
            A[::64, 0] = NAN
        elif what == "column":
            A[:, col] = NAN
        elif what == "all":
            A.fill_(NAN)
        else:
            A[n // 2, col] = INF

    A, fac, ipiv = _factor(n, fill)
    want = {"entry": n, "rows": n - (n + 63) // 64 + 1, "column": col + 1, "all": 1}.get(what)
    assert fac.status == mxp.ESINGULAR
    if want is not None:
        assert fac.info == want
    if A is not None:
        piv, info = _pivots(A)
        assert fac.info == info
        assert ipiv[:info].tolist() == piv[:info]
