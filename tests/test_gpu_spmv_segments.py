"""gmls_spmv with long rows cut into 64, 32, 16, 8, 4 and 2 segments (1 to 128
of them) and whole (more), empty segments' lengths among them, against a long
double product.  Bound: a lane's chain is at most 20000 / 64 / 4 entries (a
whole row, 64 lanes of a wavefront, four sums, four wavefronts) plus 14
additions, each 2^-53 of the row's sum of absolute products; 128 * 2^-53
covers it."""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import ctx, dev, flush, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_long", [1, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65, 127, 128, 129, 300])
def test_numbers_of_long_rows(n_long):
    G = require_gpu()
    g = np.random.default_rng(n_long)
    lens = np.concatenate([g.integers(0, 90, size=150), g.integers(8193, 20000, size=n_long)]).astype(np.int64)
    lens = lens[g.permutation(len(lens))]
    rp = np.zeros(len(lens) + 1, dtype=np.int64)
    np.cumsum(lens, out=rp[1:])
    n_cols = 5000
    col = g.integers(0, n_cols, size=int(rp[-1])).astype(np.int32)
    val, x = g.standard_normal(int(rp[-1])), g.standard_normal(n_cols)
    flush(f"spmv segments: {n_long} long rows")
    d = [dev(a) for a in (rp, col, val, x)]
    y = host(G.gmls_spmv(ctx(), *d))
    out = torch.full((len(lens),), float("nan"), dtype=torch.float64, device="cuda")
    for _ in range(3):
        assert np.array_equal(y, host(G.gmls_spmv(ctx(), *d)))
        assert np.array_equal(y, host(G.gmls_spmv_noalloc(ctx(), *d, out)))
    prod = val.astype(np.longdouble) * x.astype(np.longdouble)[col]
    ref = np.array([prod[rp[i]:rp[i + 1]].sum() for i in range(len(lens))])
    scale = np.array([np.abs(prod[rp[i]:rp[i + 1]]).sum() for i in range(len(lens))])
    assert (np.abs(y - ref) <= 128 * 2.0 ** -53 * scale).all()
