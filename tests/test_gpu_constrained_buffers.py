"""Constrained calls of many targets keep one more right-hand side a target (the
constraint's solution) than their functionals.  With a single functional that
doubles the coefficient buffer: a fresh context's first call leaves its inputs
and the tensors around them as they were, and gives the QR kernel's weights."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import dev, flush, require_gpu

pytestmark = pytest.mark.gpu

N = 12288 + 15
TOL = 1e-10
Q = {(2, 2): 6, (2, 3): 10, (2, 4): 15, (3, 2): 10, (3, 3): 20}


@pytest.mark.parametrize("dim,order", sorted(Q))
def test_one_functional_fits_its_buffer(dim, order):
    G = require_gpu()
    k = 3 * Q[dim, order]
    x = dev(W.jittered_grid(N, dim, 61))
    nrm = torch.nn.functional.normalize(dev(W.jittered_grid(N, dim, 62)) - 0.5, dim=1)
    qr, c = G.Context(0), G.Context(0)
    qr.set_option(G.OPT_QR_SHAPE, 0)
    rp, col, eps = G.gmls_neighbors(qr, x, x, G.SEARCH_KNN, k=k, eps_mult=1.5)
    b = G.gmls_stencils_constrained(qr, x, x, order, G.F_LAPLACIAN, 4, eps, rp, col, nrm)
    ins = [x, nrm, rp, col, eps, *b[:3]]
    before = [t.clone() for t in ins]
    flush(f"constrained, one functional, many targets: dim={dim} order={order}")
    a = G.gmls_stencils_constrained(c, x, x, order, G.F_LAPLACIAN, 4, eps, rp, col, nrm)
    torch.cuda.synchronize()
    for t, u in zip(ins, before):
        assert torch.equal(t, u)
    assert torch.equal(a[2], b[2]) and int(a[2].max()) == 0
    scale = torch.hypot(b[0].reshape(N, k).norm(dim=1), b[1].reshape(N))
    ea = float(((a[0] - b[0]).reshape(N, k).norm(dim=1) / scale).max())
    eb = float(((a[1] - b[1]).reshape(N).abs() / scale).max())
    flush(f"  max rel err alpha {ea:.3e} beta {eb:.3e}")
    assert ea <= TOL and eb <= TOL
    assert not torch.equal(a[0], b[0])  # the pipeline's own
    c.close()
    qr.close()
