"""The assembly's first allocation bounds the operator from above; where the
device has no room for the bound, the exact size is asked for and allocated."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import ctx, dev, flush, require_gpu

pytestmark = pytest.mark.gpu


def test_no_room_for_the_bound(monkeypatch):
    G = require_gpu()
    pts, bnd, nrm = W.stokes_cloud(6, 2, 1)
    c = ctx()
    x = dev(pts)
    rp, col, _ = G.gmls_neighbors(c, x, x, G.SEARCH_KNN, k=12, eps_mult=1.5)
    n, m = len(pts), col.numel()
    g = torch.Generator(device="cuda").manual_seed(3)
    z = lambda q: torch.rand(q, generator=g, dtype=torch.float64, device="cuda")
    args = (c, rp, col, dev(bnd), dev(nrm), z(4 * m), z(2 * m), z(m), z(n), z(m), z(n))
    flush("stokes memory: with room")
    ref = G.gmls_assemble_stokes(*args)
    limit, empty = ref[1].numel(), torch.empty

    def bounded(size, *a, **kw):
        if isinstance(size, int) and size > limit and kw.get("dtype") in (torch.int32, torch.float64):
            raise torch.OutOfMemoryError("no room")
        return empty(size, *a, **kw)

    monkeypatch.setattr(torch, "empty", bounded)
    flush("stokes memory: without")
    got = G.gmls_assemble_stokes(*args)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
