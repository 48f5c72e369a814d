"""GPU tests of the strip solves of a block step, L21 = A21 U11^-1 and U12 = L11^-1
A12, against FP64 from the FP32 factor of the diagonal block: of the first block
step, whose panels receive no update before and none after, so that the stored
panels are the solves' results rounded once (L21 under its strips' powers of two)."""
import pytest
import torch

import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu


def _first_step(n, nb, update, store, seed=6, kind=mxp.GEN_DOMINANT):
    """(stored, exact) of both sides, lines of the solve as rows, in the stored scale"""
    prob = mxp.mxp_generate(n, 1, seed, store=store, kind=kind, gamma=1.0)
    A = mxp.as_matrix(prob.A, n)
    A21, A12 = A[nb:, :nb].double(), A[:nb, nb:].double()
    fac = mxp.mxp_factor(prob, nb, update)
    assert fac.info == 0
    lay = mxp.factor_layout(n, nb, update)
    T = fac.aux[lay.T:lay.T + 4 * nb * nb].view(torch.float32).view(nb, nb).t().double()
    lsc = fac.aux[lay.lsc:lay.lsc + 4 * lay.strips].view(torch.float32).double()
    s = lsc[torch.arange(nb, n, device="cuda") // 32][:, None]
    F = mxp.as_matrix(fac.LU, n)
    U = torch.triu(T)
    L = torch.tril(T, -1) + torch.eye(nb, dtype=torch.float64, device="cuda")
    l = torch.linalg.solve_triangular(U, A21, upper=True, left=False)
    u = torch.linalg.solve_triangular(L, A12, upper=False, unitriangular=True).t()
    return (F[nb:, :nb], l * s), (F[:nb, nb:].t(), u)


# The strips next to the diagonal block are solved by FP32 substitution.  Where
# the others are too -- more than 4096 rows left but less than 16 blocks -- they
# must be as close to the exact solution: the share of entries that are not its
# rounding to FP16 is the mean error over the spacing, so twice the first
# strips' share and five deviations of its count leave no room for a solve of
# fewer bits (products with two FP16 parts of the inverse: 12 to 35 times the
# first strips' share).
@pytest.mark.parametrize("n,nb,update", [(5300, 512, "f16"), (6100, 1024, "f16"), (7000, 512, "f8")])
@pytest.mark.parametrize("kind", [mxp.GEN_DOMINANT, mxp.GEN_SQRTN])
def test_every_strip_is_as_accurate_as_the_first(n, nb, update, kind):
    print("strips", n, nb, update, kind, flush=True)
    assert 4096 < n - nb < 16 * nb
    for got, want in _first_step(n, nb, update, "f16", kind=kind):
        off = got != want.to(torch.float16)
        first, rest = off[:nb], off[nb:]
        a, b = int(first.sum()), int(rest.sum())
        expect = rest.numel() / first.numel()
        print("  not the exact rounding: first %d of %d, others %d of %d" % (a, first.numel(), b, rest.numel()),
              flush=True)
        assert b <= expect * (2 * a + 5 * max(a, 1) ** 0.5)
