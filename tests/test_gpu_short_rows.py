"""Targets of at most 32 rows, whose weights leave from registers: several
functional rows of several targets per wavefront, in every row shape, against
the FP64 QR kernel within the mixed gate (each functional row's coefficients
pass through the same LDS buffer)."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import dev, flush, require_gpu
from tests.test_gpu_stencils import MIXED_TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("basis,k", [("scalar", 13), ("scalar", 32), ("staggered", 13), ("staggered", 32)])
def test_short_rows_of_every_shape(basis, k):
    G = require_gpu()
    c = G.Context(0)
    n = 4099
    x = dev(W.jittered_grid(n, 3, 9))
    rp, col, eps = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=k, eps_mult=1.5)

    def call(prec):
        if basis == "staggered":
            w, t, st, _ = G.gmls_stencils_staggered(c, x, x, 1, G.F_GRAD | G.F_LAPLACIAN, 4, eps, rp, col, prec=prec)
            return torch.cat([w.reshape(n, 4, k), t.reshape(n, 4, 1)], 2), st
        w, st, _ = G.gmls_stencils(c, x, x, 2, G.BASIS_SCALAR, G.F_VALUE | G.F_GRAD | G.F_LAPLACIAN, 4, eps, rp, col,
                                   prec=prec)
        return w.reshape(n, 5, k), st

    ref, rs = call(G.PREC_FP64)
    for cand in (0, 1, 2):
        c.set_option(G.OPT_PIPE_SHAPE, cand)
        w, st = call(G.PREC_MIXED)
        assert torch.equal(st == 1, rs == 1)
        e = float(((w - ref).norm(dim=2) / ref.norm(dim=2))[rs != 1].max())
        flush(f"short rows: {basis} k={k} candidate {cand}: {e:.2e}")
        assert e <= MIXED_TOL
    c.close()
