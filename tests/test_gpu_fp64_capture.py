"""FP64 calls of many targets in capture-safe mode and in a replayed graph: the
grids, windows and queues are sized without the bin table on the host, and the
results are those of the ordinary calls bit for bit.  Rows of every bin, some
too short and some over 256, and flat neighbourhoods left to the QR kernel."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import dev, flush, host, require_gpu

pytestmark = pytest.mark.gpu

N = 12288 + 70


def rows(dim, order):
    """A cloud whose first targets lie in a thin sheet, and rows of 4 to 300."""
    import numpy as np

    x = W.jittered_grid(N, dim, 71)
    x[:512, -1] = 0.5 + 1e-9 * (x[:512, -1] - 0.5)
    k = {(2, 2): 14, (2, 4): 32, (3, 2): 24, (3, 3): 44, (3, 4): 72}[dim, order]
    lens = np.full(N, k, np.int64)
    lens[5::97] = 4
    lens[9::53] = k + 64
    lens[11::1009] = 300
    return x, lens


def calls(G, c, x, eps, rp, col, dim, order, kind, nrm):
    sv = G.F_VALUE | G.F_LAPLACIAN
    if kind == "multi":
        (a, sa), (b, sb) = G.gmls_stencils_multi(c, x, x, order, 4, eps, rp, col,
                                                 [(G.BASIS_SCALAR, G.F_LAPLACIAN), (G.BASIS_DIVFREE, sv)])[0]
        return a, sa, b, sb
    if kind == "divfree":
        return G.gmls_stencils(c, x, x, order, G.BASIS_DIVFREE, sv, 4, eps, rp, col)[:2]
    if kind == "constrained":
        return G.gmls_stencils_constrained(c, x, x, order, G.F_LAPLACIAN, 4, eps, rp, col, nrm)[:3]
    return G.gmls_stencils_staggered(c, x, x, order - 1, G.F_GRAD | G.F_LAPLACIAN, 4, eps, rp, col)[:3]


@pytest.mark.parametrize("kind,dim,order", [("multi", 2, 4), ("multi", 3, 2), ("multi", 3, 3), ("multi", 3, 4),
                                            ("divfree", 2, 2), ("divfree", 3, 3), ("constrained", 3, 3),
                                            ("staggered", 3, 3)])
def test_replays_equal_ordinary_calls(kind, dim, order):
    import numpy as np

    G = require_gpu()
    s = torch.cuda.Stream()
    c = G.Context(0, stream=s)
    with torch.cuda.stream(s):
        xh, lens = rows(dim, order)
        x = dev(xh)
        kmax = int(lens.max())
        _, colk, _ = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=kmax, eps_mult=1.5)
        colk = host(colk).reshape(N, kmax)
        rp_h = np.zeros(N + 1, np.int64)
        rp_h[1:] = np.cumsum(lens)
        # rows of the kNN call are sets: order them by distance and cut
        d = ((xh[colk] - xh[:, None, :]) ** 2).sum(2)
        o = np.argsort(d, axis=1, kind="stable")
        colk, d = np.take_along_axis(colk, o, 1), np.take_along_axis(d, o, 1)
        keep = np.arange(kmax)[None, :] < lens[:, None]
        rp, col = dev(rp_h), dev(colk[keep].astype(np.int32))
        eps = dev(1.5 * np.sqrt(d[np.arange(N), lens - 1]))
        nrm = torch.nn.functional.normalize(dev(W.jittered_grid(N, dim, 72)) - 0.5, dim=1)
        flush(f"capture, many targets: {kind} dim={dim} order={order}")
        ref = calls(G, c, x, eps, rp, col, dim, order, kind, nrm)
        s.synchronize()
        ref = [r.clone() for r in ref]
        bits = lambda t: t if t.dtype == torch.uint8 else t.view(torch.int64)
        c.set_option(G.OPT_CAPTURE_SAFE, 1)

        def compare(tag, got):
            s.synchronize()
            for i, (a, b) in enumerate(zip(got, ref)):
                assert torch.equal(bits(a), bits(b)), (tag, i)
            c.check()

        compare("capture-safe", calls(G, c, x, eps, rp, col, dim, order, kind, nrm))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            got = calls(G, c, x, eps, rp, col, dim, order, kind, nrm)
        for rep in range(3):
            for t in got:
                t.fill_(7)
            s.synchronize()
            g.replay()
            compare(f"replay {rep}", got)
        # not the QR kernel's by another route
        c.set_option(G.OPT_CAPTURE_SAFE, 0)
        c.set_option(G.OPT_QR_SHAPE, 0)
        qr = calls(G, c, x, eps, rp, col, dim, order, kind, nrm)
        s.synchronize()
        assert not torch.equal(bits(qr[0]), bits(ref[0]))
    c.close()
