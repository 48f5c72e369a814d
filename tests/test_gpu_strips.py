"""GPU tests of the strip solves of a block step, L21 = A21 U11^-1 and U12 = L11^-1
A12, against FP64 from the FP32 factor of the diagonal block: of the first block
step, whose panels receive no update before and none after, so that the stored
panels are the solves' results rounded once (L21 under its strips' powers of two)."""
import pytest
import torch

import paper_2509_19618_amd as mxp
from test_gpu_factor import test_factor_backward_and_forward_error as _factor_error

pytestmark = pytest.mark.gpu


def _first_step(n, nb, update, store, seed=6, kind=mxp.GEN_DOMINANT):
    """Of both sides, lines of the solve as rows: the stored panel, the exact one in
    its scale, the scale, the right-hand sides and the triangle's inverse."""
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
    eye = torch.eye(nb, dtype=torch.float64, device="cuda")
    Ui = torch.linalg.solve_triangular(U, eye, upper=True)
    Li = torch.linalg.solve_triangular(L, eye, upper=False, unitriangular=True)
    return (F[nb:, :nb], l * s, s, A21, Ui), (F[:nb, nb:].t(), u, torch.ones_like(s), A12.t(), Li.t())


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
    for got, want, *_ in _first_step(n, nb, update, "f16", kind=kind):
        off = got != want.to(torch.float16)
        first, rest = off[:nb], off[nb:]
        a, b = int(first.sum()), int(rest.sum())
        expect = rest.numel() / first.numel()
        print("  not the exact rounding: first %d of %d, others %d of %d" % (a, first.numel(), b, rest.numel()),
              flush=True)
        assert b <= expect * (2 * a + 5 * max(a, 1) ** 0.5)


def _on_inverse_path(n, nb):
    # more strips than one launch takes, at least 16 blocks left
    return n - nb > 4096 and n - nb >= 16 * nb


INVERSE = [(4300, 64, "f16", "f16"), (4500, 128, "f8", "bf16"), (4700, 256, "f8", "f16"), (4700, 256, "bf16", "bf16"),
           (8800, 512, "f16", "f16"), (17500, 1024, "f16", "f16"), (17500, 1024, "bf16", "bf16")]


# The strips through the block's inverses: 64-row tiles (FP16, nb <= 512; waves
# without a column block at nb = 64), 32-row tiles, every number of parts and
# operand format.  Within the rounding to storage, FP32 products (4 nb 2^-24 |A|
# |U^-1|: the inverse and the sum) and the parts' last place (2^-24 of a line's
# largest, doubled).
@pytest.mark.parametrize("n,nb,update,store", INVERSE)
def test_strips_through_the_inverses(n, nb, update, store):
    print("inverse strips", n, nb, update, store, flush=True)
    assert _on_inverse_path(n, nb)
    for side, (got, want, s, rhs, inv) in enumerate(_first_step(n, nb, update, store)):
        rhs, inv = rhs.abs(), inv.abs()
        err = 4 * nb * 2.0 ** -24 * (rhs @ inv) + 2.0 ** -23 * rhs.sum(1)[:, None] * inv.amax(0)[None, :]
        u = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[store]
        bound = u * want.abs() + (1 + u) * s * err + (2.0 ** -25 if store == "f16" else 0.0)
        ratio = float(((got.double() - want).abs() / bound).max())
        print("  side %d error / bound %.3g" % (side, ratio), flush=True)
        assert ratio <= 1.0


@pytest.mark.parametrize("n,nb,update,store", [(4300, 64, "f16", "f16"), (4500, 128, "f8", "bf16")])
def test_whole_factor_with_inverse_strips(n, nb, update, store):
    assert _on_inverse_path(n, nb)
    _factor_error(n, nb, update, store)


# members on and off the inverse path, of different block sizes on it (the launch's
# tiles follow its largest), in one group: bit for bit the single factorisations
@pytest.mark.parametrize("store,group", [("f16", [(4400, 64), (8800, 512), (700, 128), (4500, 256), (4700, 512)]),
                                         ("bf16", [(4400, 64), (8800, 512), (700, 128), (4500, 256)]),
                                         ("f16", [(17500, 1024), (4400, 64), (4500, 256)])])
def test_group_of_members_on_and_off_the_inverse_path(store, group):
    print("group", store, group, flush=True)
    on = {nb for n, nb in group if _on_inverse_path(n, nb)}
    assert len(on) >= 3 and (len(on) < len(group) or 1024 in on)
    probs = [mxp.mxp_generate(n, 1, 60 + i, store=store) for i, (n, _) in enumerate(group)]
    facs = mxp.mxp_factor_group(probs, [nb for _, nb in group], store)
    for i, ((n, nb), fac) in enumerate(zip(group, facs)):
        one = mxp.mxp_factor(mxp.mxp_generate(n, 1, 60 + i, store=store), nb, store)
        assert fac.info == 0 and torch.equal(fac.LU[:, :n], one.LU[:, :n]), (n, nb)


# FP32 storage shows the solves' own roundings.  An entry of the size of the largest
# is rounded in the right-hand side's last sum and in the result, L21 also in the
# reciprocal of its pivot; entries spread evenly below the largest, a rounding is
# 0.22 units of 2^-24 of it, rms: two of them 0.31 (U12: 0.36), with a reciprocal to
# 1 ulp and the product's binade anywhere at most 0.5 (L21).  Terms added after the
# diagonal one, by far the largest, each add such a rounding: 0.46 and 0.60.  The
# sums themselves: j products of size p in two accumulators, each partial sum of
# about p sqrt(k) rounded to 0.42 units of its own size, come to 0.21 p j, over the
# columns j < nb 0.12 p nb (dominant: below 0.01; sqrt(n) kind: 0.42 at nb = 1024).
@pytest.mark.parametrize("n,nb", [(3000, 512), (3000, 128), (2500, 1024)])
@pytest.mark.parametrize("kind", [mxp.GEN_DOMINANT, mxp.GEN_SQRTN])
def test_rounding_of_the_substitution(n, nb, kind):
    print("fp32 strips", n, nb, kind, flush=True)
    for side, (got, want, _, rhs, inv) in enumerate(_first_step(n, nb, "f32", "f32", kind=kind)):
        top = want.abs().amax(0) if side == 0 else want.abs().max()
        rms = float((((got.double() - want) / top) ** 2).mean() ** 0.5) * 2.0 ** 24
        # a product: of a solution's entry and one beside the diagonal, about as large as
        # one of the right-hand side over the pivot is; relative to the right-hand side
        p = float(want.square().mean().sqrt() * (rhs.square().mean().sqrt() if side == 0 else
                                                 inv.triu(1).square().sum().div(nb * (nb - 1) / 2).sqrt())) / \
            float(rhs.abs().max())
        bound = ((0.5, 0.36)[side] ** 2 + (0.12 * p * nb) ** 2) ** 0.5
        print("  side %d rms %.3f (bound %.3f)" % (side, rms, bound), flush=True)
        assert rms <= bound


# the 64 x 64 inverses, |M Y - I| / |M| |Y|: their lower left quarter as a product
# (0.51, the right one 0.56) and not as a solve, whose 32 terms per entry are each
# rounded at the result's size (0.61, 0.66)
@pytest.mark.parametrize("nb", [512, 1024])
def test_rounding_of_the_sub_block_inverses(nb):
    print("64 x 64 inverses", nb, flush=True)
    rms = [[], []]
    eye = torch.eye(64, dtype=torch.float64, device="cuda")
    for seed in range(1, 7):
        fac = mxp.mxp_factor(mxp.mxp_generate(nb, 1, seed, store="f32"), nb, "f32")
        lay = mxp.factor_layout(nb, nb, "f32")
        T = fac.aux[lay.T:lay.T + 4 * nb * nb].view(torch.float32).view(nb, nb).t().double()[:64, :64]
        for side, off in enumerate((lay.linv, lay.uinv)):
            Y = fac.aux[off:off + 4 * 4096].view(torch.float32).view(64, 64).double()
            M, Y = (torch.tril(T, -1) + eye, Y.t()) if side == 0 else (torch.triu(T), Y)
            E = (M @ Y - eye).abs() / (M.abs() @ Y.abs()).clamp_min(1e-30)
            rms[side].append(float((E ** 2).mean() ** 0.5) * 2.0 ** 24)
    mean = [sum(r) / len(r) for r in rms]
    print("  rms L %.3f U %.3f" % tuple(mean), flush=True)
    assert mean[0] <= 0.55 and mean[1] <= 0.6
