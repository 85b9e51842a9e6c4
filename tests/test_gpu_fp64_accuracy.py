"""FP64 calls of many targets on rows with little or no surplus over the basis,
one-sided ones among them, where condition numbers are large: their error
against extended precision.

Per target: what the kernels keep for themselves meets the gate of one-sided
FP64 stencils, max(1e-10, 4 cond 2^-53) with the condition number of the
weighted sample matrix (for eps = 1.5 times the farthest neighbour; where the
farthest one's weight all but vanishes QR does not meet it either).  Over the
targets: the root mean square of the errors is that of a call by Householder QR
(the residual's rounding reaches the weights through a projection, so the
corrected step adds no more than QR's own solves do), compared with room for
the chance that single targets dominate both: factor 1.5, the largest 2."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import extended
from tests.gpu_helpers import dev, flush, host, require_gpu

pytestmark = pytest.mark.gpu

N_TGT = 12288 + 15
SAMPLE = 1200
Q = {(2, 2): 6, (2, 4): 15, (3, 2): 10, (3, 3): 20, (3, 4): 35}


def own_rows(dim, n, side, mult, seed):
    """Every target with n sources of its own, uniform in a ball around it (or
    the half of it with x > 0), eps = mult times the farthest."""
    g = W.rng(seed)
    s = g.normal(size=(N_TGT, n, dim))
    s *= g.uniform(size=(N_TGT, n, 1)) ** (1 / dim) / np.linalg.norm(s, axis=2, keepdims=True)
    if side == "half":
        s[..., 0] = np.abs(s[..., 0])
    tgt = g.uniform(size=(N_TGT, dim))
    src = tgt[:, None] + 0.05 * s
    return src, tgt, mult * np.linalg.norm(src - tgt[:, None], axis=2).max(1)


CASES = [(b, d, o, n, side, mult) for b, d, o, n in
         [("scalar", 2, 2, 6), ("scalar", 2, 4, 15), ("scalar", 2, 4, 20), ("scalar", 3, 2, 12), ("scalar", 3, 3, 20),
          ("scalar", 3, 3, 24), ("scalar", 3, 3, 36), ("scalar", 3, 4, 37), ("scalar", 3, 4, 60), ("divfree", 3, 2, 13),
          ("divfree", 3, 3, 26), ("staggered", 3, 3, 24), ("constrained", 3, 3, 24), ("constrained", 2, 4, 18)]
         for side, mult in [("full", 1.5), ("half", 1.5), ("half", 1.05)]]


@pytest.mark.parametrize("basis,dim,order,n,side,mult", CASES)
def test_error_is_that_of_qr(basis, dim, order, n, side, mult):
    G = require_gpu()
    src, tgt, eps = own_rows(dim, n, side, mult, 31)
    nrm = None
    if basis == "constrained":
        nrm = W.rng(32).normal(size=tgt.shape)
    x, t, e = dev(src.reshape(-1, dim)), dev(tgt), dev(eps)
    rp = torch.arange(N_TGT + 1, dtype=torch.int64, device="cuda") * n
    col = torch.arange(N_TGT * n, dtype=torch.int32, device="cuda")
    flush(f"accuracy: {basis} dim={dim} order={order} n={n} {side} {mult}")

    def call(force):
        c = G.Context(0)
        if force:
            c.set_option(G.OPT_QR_SHAPE, 0)
        beta = None
        if basis == "staggered":
            w, _, st, _ = G.gmls_stencils_staggered(c, x, t, order - 1, G.F_GRAD | G.F_LAPLACIAN, 4, e, rp, col)
        elif basis == "constrained":
            w, beta, st, _ = G.gmls_stencils_constrained(c, x, t, order, G.F_GRAD | G.F_LAPLACIAN, 4, e, rp, col, dev(nrm))
        else:
            b, m = (G.BASIS_SCALAR, G.F_VALUE | G.F_GRAD | G.F_LAPLACIAN) if basis == "scalar" else \
                (G.BASIS_DIVFREE, G.F_VALUE | G.F_LAPLACIAN)
            w, st, _ = G.gmls_stencils(c, x, t, order, b, m, 4, e, rp, col)
        c.close()
        assert not st.any()
        C = dim if basis == "divfree" else 1
        return host(w).reshape(N_TGT, -1, n * C), None if beta is None else host(beta)

    (wf, bf), (wq, bq) = call(False), call(True)
    # a sample, and the targets where the two differ most
    pick = np.linspace(0, N_TGT - 1, SAMPLE).astype(int)
    diff = np.sqrt(((wf - wq) ** 2).sum(2) / (wq ** 2).sum(2)).max(1)
    pick = np.concatenate([pick, np.argsort(diff)[-300:]])
    kinds = {"scalar": ["value", "grad", "lap"], "divfree": ["value", "lap"]}.get(basis, ["grad", "lap"])
    cond = extended.condition(src[pick], tgt[pick], eps[pick], order, 4, basis)
    ref = extended.weights(src[pick], tgt[pick], eps[pick], order, 4, kinds, basis, None if nrm is None else nrm[pick])
    if nrm is not None:
        ref, rb = ref
        ref = np.concatenate([ref, rb[..., None]], 2)
        wf, wq = (np.concatenate([w, b[..., None]], 2) for w, b in ((wf, bf), (wq, bq)))
    norm = np.sqrt((ref * ref).sum(2).astype(float))
    ef, eq = (np.sqrt(((w[pick] - ref) ** 2).sum(2).astype(float)) / norm for w in (wf, wq))
    rms = lambda v: float(np.sqrt((v[:SAMPLE] ** 2).mean()))
    own = (wf != wq).any((1, 2))[pick]
    flush(f"  kept {own[:SAMPLE].mean():.3f}, to {ef[own].max():.2e}; rms {rms(ef):.2e} (QR {rms(eq):.2e}), "
          f"max {ef[:SAMPLE].max():.2e} ({eq[:SAMPLE].max():.2e})")
    if mult == 1.5:
        assert (ef.max(1) <= np.maximum(1e-10, 4 * 2.0 ** -53 * cond))[own].all()
    assert rms(ef) <= 1.5 * rms(eq)
    assert ef[:SAMPLE].max() <= 2.0 * eq[:SAMPLE].max()
