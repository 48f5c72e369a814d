"""GPU tests of the FP64 LU on matrices that give its unpivoted form badly
conditioned diagonal blocks (entries uniform in [-1, 1), the pivoting study) and
values at the ends of the range."""
import pytest
import torch

import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def _split(fac, n):
    LU = mxp.as_matrix(fac.LU, n)
    L = torch.tril(LU, -1) + torch.eye(n, dtype=torch.float64, device="cuda")
    return L, torch.triu(LU)


# Without pivoting, substitution keeps |L U - A| a small multiple of eps |L| |U|
# elementwise whatever the conditioning of a block: an entry's sum is rounded once
# per product (n eps |L| |U| at the very most; the errors being of random sign and
# the largest products few, a true substitution has been seen at 2.7 eps over these
# orders and seeds).  Explicit inverses of the 16 x 16 diagonal blocks lose what
# the block's conditioning takes: 6 to 363 eps from n = 100 on.  8: three times the
# substitution's, the product that checks it being FP64 too.
@pytest.mark.parametrize("n", [16, 100, 128, 300, 1000, 2000, 4600])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_unpivoted_uniform_is_backward_stable(n, seed):
    print("lu64 unpivoted uniform", n, seed, flush=True)
    prob = mxp.mxp_generate(n, 1, seed, store="f64", kind=mxp.GEN_UNIFORM)
    A = mxp.as_matrix(prob.A, n).clone()
    fac = mxp.mxp_lu64_factor(prob.A, n, prob.lda, False)
    assert fac.info == 0
    L, U = _split(fac, n)
    ratio = float(((L @ U - A).abs() / (L.abs() @ U.abs())).max()) / EPS
    print("  |LU - A| / (eps |L||U|): %.2f" % ratio, flush=True)
    assert ratio <= 8


# blocks of 64 (orders above 32768), on a sample of the rows
def test_unpivoted_uniform_with_blocks_of_64():
    n = 32900
    print("lu64 unpivoted uniform", n, flush=True)
    prob = mxp.mxp_generate(n, 1, 2, store="f64", kind=mxp.GEN_UNIFORM)
    rows = torch.cat([torch.arange(r, r + 70, device="cuda") for r in (0, 60, 5000, 20000, n - 70)])
    A = mxp.as_matrix(prob.A, n)[rows].clone()
    fac = mxp.mxp_lu64_factor(prob.A, n, prob.lda, False)
    assert fac.info == 0
    LU = mxp.as_matrix(fac.LU, n)
    L = torch.where(torch.arange(n, device="cuda")[None, :] < rows[:, None], LU[rows], 0.0)
    L[torch.arange(len(rows), device="cuda"), rows] = 1.0
    U = torch.triu(LU)
    ratio = float(((L @ U - A).abs() / (L.abs() @ U.abs_())).max()) / EPS
    print("  |LU - A| / (eps |L||U|): %.2f" % ratio, flush=True)
    assert ratio <= 8


# Diagonal blocks with 2^100 beside the diagonal: the inverse of such a 16 x 16
# block overflows, the substitution for the right-hand sides here is exact.  In
# the block's own 128 rows and in the strips beyond.
@pytest.mark.parametrize("lower", [False, True])
def test_blocks_whose_inverses_overflow(lower):
    n = 200
    print("lu64 overflowing inverse", lower, flush=True)
    i = torch.arange(n)
    D = torch.eye(n, dtype=torch.float64)
    k = i[:-1][i[:-1] % 16 != 15]
    D[k + 1, k] = 2.0 ** 100                       # lower bidiagonal inside each 16
    E = torch.zeros((n, n), dtype=torch.float64)
    r = i[(i > 16) & (i % 16 != 0)]
    E[r, 15] = (1 + r).double()                    # past the first 16 rows; rows from 128 on in a strip
    L, U = (D, torch.eye(n, dtype=torch.float64) + E.t()) if lower else (torch.eye(n, dtype=torch.float64) + E, D.t())
    prob = mxp.mxp_generate(n, 1, 1, store="f64")
    mxp.as_matrix(prob.A, n).copy_(L @ U)
    fac = mxp.mxp_lu64_factor(prob.A, n, prob.lda, False)
    assert fac.info == 0
    Lg, Ug = _split(fac, n)
    assert torch.equal(Lg.cpu(), L) and torch.equal(Ug.cpu(), U)


def _substitution(LU, B):
    """L y = b, U x = y row by row and with true quotients, on the CPU"""
    n = LU.shape[0]
    x = B.clone()
    for s in range(n):
        x[:, s + 1:] -= LU[s + 1:, s] * x[:, s:s + 1]
    for s in range(n - 1, -1, -1):
        x[:, s] /= LU[s, s]
        x[:, :s] -= LU[:s, s] * x[:, s:s + 1]
    return x


# diagonal entries whose reciprocal overflows, is zero or subnormal, a singular
# factor, infinite entries of a right-hand side: finite, infinite or NaN as a
# substitution with true quotients has it (row by row 2 n eps of the sums, entries
# of one sign)
@pytest.mark.parametrize("what", ["subnormal", "zero", "infinite", "huge", "rhs_first", "rhs_last", "overflow"])
@pytest.mark.parametrize("n,nrhs", [(40, 1), (130, 2), (300, 7)])
def test_solve_at_the_ends_of_the_range(what, n, nrhs):
    print("lu64 solve range", what, n, nrhs, flush=True)
    gen = torch.Generator().manual_seed(n)
    LU = -torch.rand((n, n), generator=gen, dtype=torch.float64) / n
    LU.diagonal().copy_(1 + torch.rand(n, generator=gen, dtype=torch.float64))
    B = 1 + torch.rand((nrhs, n), generator=gen, dtype=torch.float64)
    for s in (n // 3, n - 2):
        if what == "subnormal":                       # a row that stands alone, as small as its pivot
            LU[s, :], LU[:, s], LU[s, s] = 0.0, 0.0, 2.0 ** -1070
            B[:, s] = 3 * 2.0 ** -1071
        elif what == "huge":
            LU[s, :], LU[:, s], LU[s, s] = 0.0, 0.0, 1.5 * 2.0 ** 1023
            B[:, s] = 1.25 * 2.0 ** 1023
        elif what == "overflow":
            LU[s, s] = 2.0 ** -1000
            B[:, s] = 2.0 ** 1000
        elif what in ("zero", "infinite"):
            LU[s, s] = 0.0 if what == "zero" else float("inf")
    if what.startswith("rhs"):
        B[0, 1 if what == "rhs_first" else n - 1] = float("inf")
    want = _substitution(LU, B)
    got = mxp.mxp_lu64_solve(mxp.Factor64(n, LU.t().contiguous().cuda(), n, None, 0, 0), B.cuda()).cpu()
    for r in range(nrhs):                             # whatever stands beside it
        one = mxp.mxp_lu64_solve(mxp.Factor64(n, LU.t().contiguous().cuda(), n, None, 0, 0), B[r:r + 1].cuda()).cpu()
        assert torch.equal(one[0].nan_to_num(nan=7.0), got[r].nan_to_num(nan=7.0))
    fin = want.isfinite()
    assert torch.equal(got.isfinite(), fin) and torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got[~fin & ~want.isnan()], want[~fin & ~want.isnan()])
    assert bool(((got - want)[fin].abs() <= 2 * n * EPS * want[fin].abs()).all())


# groups of one, two and four right-hand sides, the last one with one to four: each
# solution as if alone
@pytest.mark.parametrize("n", [16, 129, 700])
@pytest.mark.parametrize("nrhs", [2, 3, 4, 5, 63, 64])
def test_right_hand_sides_are_independent(n, nrhs):
    print("lu64 right-hand sides", n, nrhs, flush=True)
    prob = mxp.mxp_generate(n, nrhs, 9, store="f64", kind=mxp.GEN_UNIFORM)
    fac = mxp.mxp_lu64_factor(prob.A, n, prob.lda, True)
    X = mxp.mxp_lu64_solve(fac, prob.B)
    for r in {0, nrhs // 2, nrhs - 1}:
        assert torch.equal(mxp.mxp_lu64_solve(fac, prob.B[r:r + 1].contiguous())[0], X[r])
