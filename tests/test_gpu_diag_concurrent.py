"""GPU test of diagonal-block LUs of many work-groups on several streams at once."""
import threading

import pytest
import torch

import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu


# Groups of eight with 22 and 10 work-groups per block (a tile column each: the
# blocks' first indices fall on different XCDs), the first of them more from
# three host threads together than the device holds: every factorisation completes
# (an expired wait raises) and equals the same one run alone, bit for bit.
@pytest.mark.parametrize("nb,n", [(704, 1500), (320, 1000)])
def test_grouped_diagonal_blocks_from_several_threads(nb, n):
    print("concurrent groups", nb, n, flush=True)
    want = []
    for i in range(8):
        one = mxp.mxp_factor(mxp.mxp_generate(n - 8 * i, 1, 90 + i, store="bf16"), nb, "bf16")
        assert one.info == 0
        want.append(one.LU[:, :n - 8 * i].clone())
    torch.cuda.synchronize()
    bad = []

    def run():
        s = torch.cuda.Stream()
        try:
            with torch.cuda.stream(s):
                for _ in range(6):
                    probs = [mxp.mxp_generate(n - 8 * i, 1, 90 + i, store="bf16", stream=s) for i in range(8)]
                    facs = mxp.mxp_factor_group(probs, [nb] * 8, "bf16", stream=s)
                    s.synchronize()
                    for i, f in enumerate(facs):
                        if f.info != 0 or not torch.equal(f.LU[:, :n - 8 * i], want[i]):
                            bad.append((i, f.info))
        except Exception as e:          # an expired wait raises MxpError
            bad.append(repr(e))

    ths = [threading.Thread(target=run) for _ in range(3)]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    assert not bad, bad
