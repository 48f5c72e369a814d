"""GPU tests of calls under stream capture: the captured call gives the eager call's
result on every replay, with eager work between them."""
import pytest
import torch

import paper_2509_19618_amd as mxp

pytestmark = pytest.mark.gpu


def _replays_equal_eager(run, outputs):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        run()
    s.synchronize()
    want = [o.clone() for o in outputs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        run()
    for _ in range(3):
        for o in outputs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, w) for o, w in zip(outputs, want))
        with torch.cuda.stream(s):
            run()                                    # eager work between the replays
        s.synchronize()
        assert all(torch.equal(o, w) for o, w in zip(outputs, want))


# one block; every strip of a step in one launch; more of them than CUs, through the
# inverses and by substitution
@pytest.mark.parametrize("n,nb,store", [(500, 512, "f16"), (2000, 256, "f16"), (5000, 128, "bf16"),
                                        (5200, 512, "f32")])
def test_factorisation_under_capture(n, nb, store):
    print("capture", n, nb, store, flush=True)
    L = mxp.lib()
    prob = mxp.mxp_generate(n, 1, 3, store=store)
    A0 = prob.A.clone()
    aux = torch.empty(L.mxp_factor_aux_bytes(n, nb), dtype=torch.uint8, device="cuda")
    work = torch.empty(L.mxp_factor_work_bytes(n, nb, mxp.dtype_code(store)), dtype=torch.uint8, device="cuda")

    def run():
        prob.A.copy_(A0)
        mxp.mxp_factor(prob, nb, store, work=work, aux=aux, sync_info=False)

    _replays_equal_eager(run, [prob.A[:, :n]])
