"""GPU test of leading dimensions whose columns lie so far apart that a block of the
substitution's loads leaves 32-bit offsets."""
import pytest
import torch

import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu


# 127 columns of 33 MB and more span 4 GB: the same bits as with dense columns (38 GB
# of matrix, n rows of each column touched)
@pytest.mark.parametrize("nb", [512, 1024])
def test_substitution_with_columns_far_apart(nb):
    n, lda = 1100, (1 << 24) + (1 << 19)
    print("far columns", nb, lda, flush=True)
    assert 127 * lda * 2 > 1 << 32
    out = []
    for ld in (1152, lda):
        prob = mxp.mxp_generate(n, 2, 41, store="bf16", lda=ld)
        fac = mxp.mxp_factor(prob, nb, "bf16")
        assert fac.info == 0
        out.append(mxp.mxp_apply_prec(fac, prob.B))
    assert torch.equal(out[0], out[1])
