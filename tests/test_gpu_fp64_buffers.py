"""FP64 calls of many targets in capture-safe mode, where the pipeline's buffers
are those an earlier call has grown: the sets of a multi call take the kernels
of their own calls, bit for bit, whatever buffers there are."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import dev, flush, require_gpu

pytestmark = pytest.mark.gpu

N = 12288 + 15


@pytest.mark.parametrize("order", [2, 3])
@pytest.mark.parametrize("grown", ["none", "scalar", "divfree", "both"])
def test_multi_equals_separate_calls_with_the_buffers_there_are(order, grown):
    G = require_gpu()
    k = 30 if order == 2 else 50
    x = dev(W.jittered_grid(N, 3, 51))
    sets = [(G.BASIS_SCALAR, G.F_LAPLACIAN), (G.BASIS_DIVFREE, G.F_VALUE | G.F_LAPLACIAN)]
    c = G.Context(0)
    rp, col, eps = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=k, eps_mult=1.5)
    flush(f"buffers: order={order} grown={grown}")
    call = lambda b, m: G.gmls_stencils(c, x, x, order, b, m, 4, eps, rp, col)[0]
    # the buffers of every kernel but the pipeline, by calls with forced QR
    c.set_option(G.OPT_QR_SHAPE, 0)
    qr = [call(b, m) for b, m in sets]
    G.gmls_stencils_multi(c, x, x, order, 4, eps, rp, col, sets)
    c.set_option(G.OPT_QR_SHAPE, -1)
    # then the pipeline's
    for i, name in enumerate(("scalar", "divfree")):
        if grown in (name, "both"):
            call(*sets[i])
    c.set_option(G.OPT_CAPTURE_SAFE, 1)
    outs, _ = G.gmls_stencils_multi(c, x, x, order, 4, eps, rp, col, sets)
    sep = [call(b, m) for b, m in sets]
    torch.cuda.synchronize()
    for i, ((w, _), r) in enumerate(zip(outs, sep)):
        assert torch.equal(w, r), i
    # and those that had to be QR's are
    assert torch.equal(sep[0], qr[0]) == (grown == "none" or (grown == "divfree" and order == 3))
    assert torch.equal(sep[1], qr[1]) == (grown in ("none", "scalar") and order == 2)
    c.close()
