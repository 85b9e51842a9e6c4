"""Windows of the FP64 pipeline: from 4096 targets a window (GMLS_OPT_PIPE_CHUNK)
the same weights bit for bit, below that, where the launches of its windows
would take longer than the QR kernel, those of the QR kernel."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import dev, flush, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("basis", ["scalar", "divfree"])
def test_windows(basis):
    G = require_gpu()
    c = G.Context(0)
    n = 12288 + 15
    x = dev(W.jittered_grid(n, 3, 41))
    rp, col, eps = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=24, eps_mult=1.5)
    b = G.BASIS_SCALAR if basis == "scalar" else G.BASIS_DIVFREE
    out = {}
    for chunk in (0, 4096, 4095, 64):
        c.set_option(G.OPT_PIPE_CHUNK, chunk)
        out[chunk] = G.gmls_stencils(c, x, x, 2, b, G.F_VALUE, 4, eps, rp, col)[0]
    c.set_option(G.OPT_QR_SHAPE, 0)
    qr = G.gmls_stencils(c, x, x, 2, b, G.F_VALUE, 4, eps, rp, col)[0]
    flush(f"windows: {basis}")
    assert torch.equal(out[4096], out[0]) and not torch.equal(out[0], qr)
    assert torch.equal(out[4095], qr) and torch.equal(out[64], qr)
    c.close()
