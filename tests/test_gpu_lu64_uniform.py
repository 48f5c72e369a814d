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
