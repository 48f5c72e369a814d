"""GPU tests of the block kernels at the sizes where their tilings change.

* The FP32 diagonal-block LU (one block, n <= nb): L U against the stored
  matrix in FP64, elementwise within the error of an FP32 elimination
  (2 (kb + 32) 2^-24 |L||U|: kb sums and the reciprocal's two roundings per
  element), the row-major copy and the stored block equal to it, and the
  64 x 64 sub-block inverses within the same relative error.
* The FP64 LU and solve: L U against P A within 8 n eps |L||U|, |L| <= 1 with
  pivoting, the solution's HPL scaled residual below 16.
"""
import pytest
import torch

import paper_2509_19618_amd as mxp
from test_gpu_factor import _dense_prec
from test_gpu_factor import test_factor_backward_and_forward_error as _factor_error

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


# one tile, a tile and a row, whole 64s, tiles at every distance from the
# diagonal (from 4 tiles on), ragged ends, the largest block; then a zero pivot
@pytest.mark.parametrize("n,nb,store", [(1, 64, "f32"), (33, 64, "f16"), (64, 64, "bf16"), (96, 128, "f32"),
                                        (128, 128, "f16"), (161, 256, "bf16"), (512, 512, "f32"),
                                        (501, 512, "f16"), (1000, 1024, "bf16"), (1024, 1024, "f32")])
def test_diagonal_block(n, nb, store):
    print("diag", n, nb, store, flush=True)
    prob = mxp.mxp_generate(n, 1, 11 + n, store=store, kind=mxp.GEN_SQRTN, gamma=1.0)
    A = mxp.as_matrix(prob.A, n).double().clone()
    fac = mxp.mxp_factor(prob, nb, store)
    assert fac.info == 0
    lay = mxp.factor_layout(n, nb, store)

    def f32(off, shape):
        cnt = shape[0] * shape[1]
        return fac.aux[off:off + 4 * cnt].view(torch.float32).view(shape)

    T = f32(lay.T, (nb, nb)).t()[:n, :n]
    assert torch.equal(T, f32(lay.Trm, (nb, nb))[:n, :n])
    stored = mxp.as_matrix(fac.LU, n)
    assert torch.equal(stored, T.to(stored.dtype))
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    L, U = torch.tril(T.double(), -1) + eye, torch.triu(T.double())
    bound = 2 * (n + 32) * 2.0 ** -24
    assert bool(((L @ U - A).abs() <= bound * (L.abs() @ U.abs())).all())
    for b in range(n // 64):
        s = slice(64 * b, 64 * b + 64)
        Li = f32(lay.linv + b * 16384, (64, 64)).t().double()
        Ui = f32(lay.uinv + b * 16384, (64, 64)).double()
        e = eye[s, s]
        assert bool(((Li @ L[s, s] - e).abs() <= bound * (Li.abs() @ L[s, s].abs())).all())
        assert bool(((Ui @ U[s, s] - e).abs() <= bound * (Ui.abs() @ U[s, s].abs())).all())


@pytest.mark.parametrize("n,nb,col", [(64, 64, 0), (130, 256, 37), (600, 512, 290), (600, 128, 599)])
def test_first_zero_pivot_is_reported(n, nb, col):
    print("zero pivot", n, nb, col, flush=True)
    prob = mxp.mxp_generate(n, 1, 5, store="f32")
    A = mxp.as_matrix(prob.A, n)
    A.copy_(torch.eye(n, device="cuda"))
    A[col, col] = 0.0
    assert mxp.mxp_factor(prob, nb, "f32").info == col + 1


# unpivoted: 16-wide tiles, the 128 block; pivoted also the widths of the
# one-work-group panel (16 columns to 2048 rows, 8 to 4096, 4 to 8192) and the
# device-wide one beyond
@pytest.mark.parametrize("n,pivot,nrhs", [(1, False, 1), (15, False, 3), (17, True, 1), (128, False, 4),
                                          (129, True, 5), (257, False, 7), (300, True, 2), (2049, True, 1),
                                          (4100, True, 1), (8200, True, 1)])
def test_lu64_and_solve(n, pivot, nrhs):
    print("lu64", n, pivot, nrhs, flush=True)
    prob = mxp.mxp_generate(n, nrhs, 3 + n, store="f64", kind=mxp.GEN_UNIFORM if pivot else mxp.GEN_DOMINANT)
    A = mxp.as_matrix(prob.A, n).clone()
    fac = mxp.mxp_lu64_factor(prob.A, n, prob.lda, pivot)
    assert fac.info == 0
    X = mxp.mxp_lu64_solve(fac, prob.B)
    r = prob.B - X @ A.t()
    den = (A.abs().sum(1).max() * X.abs().amax(1) + prob.B.abs().amax(1)) * n * EPS
    assert bool((r.abs().amax(1) / den < 16).all())
    LU = mxp.as_matrix(fac.LU, n)
    L, U = torch.tril(LU, -1), torch.triu(LU)
    if pivot:
        assert float(L.abs().max()) <= 1.0 + 2 * EPS
        perm = list(range(n))
        for k, p in enumerate(fac.ipiv.tolist()):
            assert k <= p < n
            perm[k], perm[p] = perm[p], perm[k]
        A = A[torch.tensor(perm, device="cuda")]
    L = L + torch.eye(n, dtype=torch.float64, device="cuda")
    assert bool(((L @ U - A).abs() <= 8 * n * EPS * (L.abs() @ U.abs())).all())


# a last strip of 1 to 63 rows, lda ending inside it or past it: the 16-byte
# loads (padding rows filled with NaN) against the element loads of an odd lda
@pytest.mark.parametrize("n,nb,store,lda", [(321, 64, "f16", 384), (600, 128, "bf16", 640), (1000, 128, "f16", 1000),
                                            (1087, 256, "f32", 1088)])
def test_ragged_last_strip_of_the_substitution(n, nb, store, lda):
    print("ragged strip", n, nb, store, lda, flush=True)
    out = []
    for ld in (lda, n + 1 - n % 2):
        prob = mxp.mxp_generate(n, 3, 21, store=store, lda=ld)
        fac = mxp.mxp_factor(prob, nb, store)
        fac.LU[:, n:] = float("nan")
        out.append(mxp.mxp_apply_prec(fac, prob.B))
    assert torch.equal(out[0], out[1])


# shares of eight waves that are empty, of one column, ragged or whole; one
# block, a block of one column behind it, several; FP32 storage (a panel in two
# groups of loads): against L and U in FP64 within the FP32 error of the inverses
# (as the apply's own test: 32 D 2^-24, D the substitution's block), the same bits
# from each right-hand side alone and again
@pytest.mark.parametrize("n,nb,store", [(1, 64, "f16"), (65, 64, "f32"), (130, 64, "bf16"), (1025, 512, "f32"),
                                        (1100, 1024, "f16"), (2100, 512, "bf16")])
def test_substitution_shares(n, nb, store):
    print("substitution", n, nb, store, flush=True)
    prob = mxp.mxp_generate(n, 3, 51, store=store)
    fac = mxp.mxp_factor(prob, nb, store)
    Z = mxp.mxp_apply_prec(fac, prob.B)
    L, U = (torch.from_numpy(M) for M in _dense_prec(prob, fac))
    D = 2 * nb if nb <= 512 else nb
    for r in range(3):
        y = torch.linalg.solve_triangular(L, prob.B[r:r + 1, :n].cpu().T, upper=False, unitriangular=True)
        z = torch.linalg.solve_triangular(U, y, upper=True)[:, 0]
        assert float((Z[r, :n].cpu() - z).abs().max()) <= 32 * D * 2.0 ** -24 * float(z.abs().max())
        assert torch.equal(mxp.mxp_apply_prec(fac, prob.B[r:r + 1].contiguous())[0], Z[r])
    assert torch.equal(mxp.mxp_apply_prec(fac, prob.B), Z)


# rows in groups of four per thread: whole, ragged, and columns that are not
# aligned for the group's store give the same entries, row norms and diagonal
@pytest.mark.parametrize("n", [1, 3, 130, 1027])
@pytest.mark.parametrize("store", ["f16", "bf16", "f32", "f64"])
def test_generator_does_not_depend_on_the_leading_dimension(n, store):
    print("generate", n, store, flush=True)
    a = mxp.mxp_generate(n, 1, 77, store=store, kind=mxp.GEN_UNIFORM)
    b = mxp.mxp_generate(n, 1, 77, store=store, kind=mxp.GEN_UNIFORM, lda=n + 1 - n % 2)
    assert torch.equal(mxp.as_matrix(a.A, n), mxp.as_matrix(b.A, n))
    assert torch.equal(a.diag, b.diag) and torch.equal(a.row_l1, b.row_l1)
    assert float(a.a_inf) == float(a.row_l1.max())


# more right-hand sides than one pass takes (16 and 4), at a size whose sums
# are one block's and one where they are not; each solution as if alone
@pytest.mark.parametrize("n", [700, 4100])
def test_many_right_hand_sides(n):
    print("rhs batches", n, flush=True)
    prob = mxp.mxp_generate(n, 20, 31, store="bf16")
    fac = mxp.mxp_factor(prob, 128, "bf16")
    res = mxp.mxp_solve_ir(prob, fac)
    assert res.code == 0 and all(e < 16 for e in res.eta)
    for r in (0, 15, 16, 19):
        one = mxp.mxp_solve_ir(prob, fac, B=prob.B[r:r + 1].contiguous())
        assert float((res.X[r] - one.X[0]).abs().max()) <= 1e-12 * float(one.X[0].abs().max())


# more strips than CUs (a trailing part of more than 4096): the first strips of a
# step on their own, the others by substitution (FP32 storage) or through the
# block inverses, against the definition; then in a group bit for bit
@pytest.mark.parametrize("n,nb,update,store", [(4300, 64, "bf16", "bf16"), (4500, 128, "f8", "f16"),
                                               (4900, 512, "f32", "f32"), (4400, 256, "f16", "f16"),
                                               (5400, 1024, "bf16", "bf16")])
def test_factor_of_more_strips_than_cus(n, nb, update, store):
    _factor_error(n, nb, update, store)
    probs = [mxp.mxp_generate(n - 100 * i, 1, 6 + i, store=store) for i in range(2)]
    facs = mxp.mxp_factor_group(probs, [nb, nb], update)
    for i, fac in enumerate(facs):
        one = mxp.mxp_factor(mxp.mxp_generate(n - 100 * i, 1, 6 + i, store=store), nb, update)
        m = n - 100 * i                              # (the columns' padding is nobody's)
        assert fac.info == 0 and torch.equal(fac.LU[:, :m], one.LU[:, :m])


# the swaps alone (identity factor), in order: chunks of 64 whole and ragged, rows
# named by several swaps, and a vector past what LDS holds
@pytest.mark.parametrize("n", [1, 64, 65, 1087, 2500, 18400])
def test_lu64_solve_applies_the_swaps_in_order(n):
    print("swaps", n, flush=True)
    gen = torch.Generator().manual_seed(n)
    k = torch.arange(n)
    piv = k + (torch.rand(n, generator=gen) * torch.minimum(n - k, torch.tensor(n if n % 2 else 70))).long()
    want = torch.arange(2.0 * n, dtype=torch.float64).reshape(2, n)
    B = want.clone().cuda()
    order = list(range(n))
    for i, p in enumerate(piv.tolist()):
        order[i], order[p] = order[p], order[i]
    fac = mxp.Factor64(n, torch.eye(n, dtype=torch.float64, device="cuda"), n, piv.cuda(), 0, 0)
    assert torch.equal(mxp.mxp_lu64_solve(fac, B).cpu(), want[:, order])


# four blocks per update: one group and a ragged rest, a rest of one row, a group
# whose successor is taken block by block
@pytest.mark.parametrize("n", [4097, 4224, 4609, 5000])
def test_lu64_in_groups_of_blocks(n):
    test_lu64_and_solve(n, False, 1)
