"""FP64 calls of many targets: what their kernels leave to the QR kernel (ill-
conditioned targets, rows over 256 of the wavefront kernel's bases) is computed
by it in the shape of the target's own bin, so that the weights are those of a
call with forced QR bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_helpers import dev, flush, require_gpu

pytestmark = pytest.mark.gpu

N = 12288 + 15


def sheet(n, seed):
    """Points within 1e-7 of a paraboloid: the monomials of degree 2 and less
    are dependent to that distance, which the Cholesky factor of the Gram sees
    squared and Householder QR does not."""
    g = W.rng(seed)
    x = g.uniform(-1, 1, size=(n, 3))
    x[:, 2] = (x[:, 0] ** 2 + x[:, 1] ** 2) / 2 + 1e-7 * x[:, 2]
    return x


def both(G, call):
    fast, qr = G.Context(0), G.Context(0)
    qr.set_option(G.OPT_QR_SHAPE, 0)
    out = [call(c) for c in (fast, qr)]
    fast.close()
    qr.close()
    return out


@pytest.mark.parametrize("basis,order,k", [("scalar", 2, 30), ("scalar", 3, 60), ("scalar", 3, 150), ("scalar", 4, 100),
                                           ("divfree", 2, 30), ("divfree", 3, 70), ("staggered", 3, 40),
                                           ("constrained", 2, 30)])
def test_ill_conditioned_targets_equal_qr(basis, order, k):
    G = require_gpu()
    c = G.Context(0)
    x = dev(sheet(N, 21))
    rp, col, eps = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=k, eps_mult=1.5)
    nrm = torch.stack([x[:, 0], x[:, 1], -torch.ones_like(x[:, 0])], 1).contiguous()
    c.close()
    flush(f"left targets: {basis} order={order} k={k}")

    def call(c):
        if basis == "staggered":
            w, t, st, _ = G.gmls_stencils_staggered(c, x, x, order - 1, G.F_GRAD | G.F_LAPLACIAN, 4, eps, rp, col)
            return w, t, st
        if basis == "constrained":
            return G.gmls_stencils_constrained(c, x, x, order, G.F_LAPLACIAN, 4, eps, rp, col, nrm)[:3]
        b = G.BASIS_SCALAR if basis == "scalar" else G.BASIS_DIVFREE
        w, st, _ = G.gmls_stencils(c, x, x, order, b, G.F_LAPLACIAN, 4, eps, rp, col)
        return w, st, st

    a, b = both(G, call)
    for u, v in zip(a, b):
        assert torch.equal(u.nan_to_num(), v.nan_to_num())


@pytest.mark.parametrize("basis,order", [("scalar", 4), ("divfree", 3), ("divfree", 4)])
def test_long_rows_equal_qr(basis, order):
    G = require_gpu()
    c = G.Context(0)
    x = dev(W.jittered_grid(N, 3, 22))
    rp, col, eps = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=270, eps_mult=1.5)
    c.close()
    b = G.BASIS_SCALAR if basis == "scalar" else G.BASIS_DIVFREE
    flush(f"long rows: {basis} order={order}")
    u, v = both(G, lambda c: G.gmls_stencils(c, x, x, order, b, G.F_LAPLACIAN, 4, eps, rp, col)[:2])
    assert torch.equal(u[0], v[0]) and torch.equal(u[1], v[1])


@pytest.mark.parametrize("order", [3, 4])
def test_multi_of_left_targets_equals_separate_calls(order):
    G = require_gpu()
    c = G.Context(0)
    g = W.rng(23)
    x = dev(np.concatenate([sheet(N - 600, 24), g.normal(0.0, 0.02, size=(600, 3))]))
    rp, col, eps = G.gmls_neighbors(c, x, x, G.SEARCH_RADIUS, radius=0.05, k_min=60)
    n = rp[1:] - rp[:-1]
    assert int(n.max()) > 256 and int(n.min()) <= 64
    sets = [(G.BASIS_SCALAR, G.F_GRAD), (G.BASIS_DIVFREE, G.F_LAPLACIAN)]
    flush(f"multi, left targets: order={order}")
    outs, _ = G.gmls_stencils_multi(c, x, x, order, 4, eps, rp, col, sets)
    for (w, st), (b, m) in zip(outs, sets):
        rw, rs, _ = G.gmls_stencils(c, x, x, order, b, m, 4, eps, rp, col)
        assert torch.equal(st, rs) and torch.equal(w.nan_to_num(), rw.nan_to_num())
    c.close()
