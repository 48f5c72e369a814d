"""GPU test of the generator at the edges of its work-groups' rows (128 in FP64, 256 in
the other formats) and of their waves' column quads: bit for bit the oracle's matrix,
diagonal and row norms."""
import numpy as np
import pytest

import oracle
import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 31, 32, 33, 127, 128, 129, 255, 256, 257, 1025])
@pytest.mark.parametrize("kind", [mxp.GEN_DOMINANT, mxp.GEN_UNIFORM])
def test_generator_edges(n, kind):
    print("generate edges", n, kind, flush=True)
    A, _ = oracle.generate(n, 5, kind)
    norms = []
    # (rounded once from FP64 by the oracle: torch's conversion to bfloat16 goes through
    # FP32 and rounds some entries twice)
    for store, want in (("f64", A), ("f32", oracle.round_array(oracle.FMT_F32, A)),
                        ("bf16", oracle.round_array(oracle.FMT_BF16, A))):
        p = mxp.mxp_generate(n, 1, 5, store=store, kind=kind)
        assert np.array_equal(mxp.as_matrix(p.A, n).double().cpu().numpy(), want)
        assert np.array_equal(p.diag.cpu().numpy(), np.diag(A))
        norms.append(p.row_l1.cpu().numpy())
    assert np.abs(norms[0] - np.abs(A).sum(axis=1)).max() <= n * 2.0 ** -52 * norms[0].max()
    assert np.array_equal(norms[0], norms[1]) and np.array_equal(norms[0], norms[2])
