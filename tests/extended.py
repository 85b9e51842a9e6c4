"""Stencil weights in x87 extended precision, batched over targets whose rows
have the same length: Householder QR of the weighted sample matrix,
alpha = W^(1/2) Q R^-T lambda.  The divergence-free fit takes the sample matrix
of an explicit basis of the space, the staggered one drops the constant, the
constraint n . grad = h is eliminated by its multiplier.  With 64 bits of
significand and no Gram matrix the error is cond * 2^-64."""
import math

import numpy as np

from oracle.constrained import exponents
from oracle.divfree import explicit_basis

LD = np.longdouble


def _qr(A):
    """(R, apply): apply(y) is Q [y; 0] for y [T, Q]."""
    A = A.copy()
    T, N, Q = A.shape
    refl = []
    for k in range(Q):
        v = A[:, k:, k].copy()
        beta = np.sqrt((v * v).sum(1))
        v[:, 0] += np.where(v[:, 0] >= 0, beta, -beta)
        vv = (v * v).sum(1)
        tau = np.where(vv > 0, 2 / np.where(vv > 0, vv, 1), 0)
        A[:, k:, k:] -= v[:, :, None] * (np.einsum("tn,tnq->tq", v, A[:, k:, k:]) * tau[:, None])[:, None, :]
        refl.append((v, tau))

    def apply(y):
        z = np.zeros((T, N), LD)
        z[:, :Q] = y
        for k in range(Q - 1, -1, -1):
            v, tau = refl[k]
            z[:, k:] -= v * ((v * z[:, k:]).sum(1) * tau)[:, None]
        return z

    return A[:, :Q], apply


def _rt_solve(R, lam):
    y = np.zeros((R.shape[0], R.shape[1]), LD)
    for j in range(R.shape[1]):
        y[:, j] = (lam[:, j] - (R[:, :j, j] * y[:, :j]).sum(1)) / R[:, j, j]
    return y


def _functionals(dim, ex, kinds, eps):
    """lambda of each of `kinds` ("value", "grad", "lap") on the monomials s^a,
    [rows][T, Q]."""
    one = {tuple(e): i for i, e in enumerate(ex.tolist())}
    unit = lambda d, n: one[tuple(n if c == d else 0 for c in range(3))]
    out = []
    for kind in kinds:
        cols = {"value": [[0]], "grad": [[unit(d, 1)] for d in range(dim)], "lap": [[unit(d, 2) for d in range(dim)]]}[kind]
        scale = {"value": np.ones_like(eps), "grad": 1 / eps, "lap": 2 / eps ** 2}[kind]
        for c in cols:
            v = np.zeros((len(eps), len(ex)), LD)
            v[:, c] = scale[:, None]
            out.append(v)
    return out


def _sample(src, tgt, eps, order, p, basis):
    """Square-rooted row weights [T, rows] and sample matrix [T, rows, Q], and
    the columns' exponents and divergence-free coefficients."""
    T, N, dim = src.shape
    s = (src.astype(LD) - tgt.astype(LD)[:, None]) / eps[:, None, None]
    r = np.sqrt((s * s).sum(-1))
    sw = np.sqrt(np.where(r < 1, 1 - r, 0) ** p)
    ex = exponents(dim, order)
    P = np.stack([np.prod([s[..., d] ** int(e[d]) for d in range(dim)], axis=0) for e in ex], -1)
    if basis == "staggered":
        return sw, P[..., 1:], ex, None
    if basis != "divfree":
        return sw, P, ex, None
    # explicit_basis: rows over (scaled monomial s^a / a!, component)
    B = explicit_basis(dim, order).astype(LD)
    fact = np.array([math.prod(math.factorial(int(q)) for q in e) for e in ex], LD)
    Bc = [B[c::dim] / fact[:, None] for c in range(dim)]
    P = np.stack([P @ b for b in Bc], 2).reshape(T, N * dim, B.shape[1])
    return np.repeat(sw, dim, axis=1), P, ex, Bc


def condition(src, tgt, eps, order, p, basis="scalar"):
    """2-norm condition number of the weighted sample matrix [T]."""
    sw, P, _, _ = _sample(src, tgt, eps.astype(LD), order, p, basis)
    sv = np.linalg.svd((sw[..., None] * P).astype(float), compute_uv=False)
    return sv[:, 0] / sv[:, -1]


def weights(src, tgt, eps, order, p, kinds, basis="scalar", normals=None):
    """src [T, N, dim], tgt [T, dim], eps [T] (FP64).  Returns alpha
    [T, rows, N * components] and, for normals [T, dim], beta [T, rows]."""
    dim = src.shape[2]
    eps = eps.astype(LD)
    rows, P, ex, Bc = _sample(src, tgt, eps, order, p, basis)
    lam = _functionals(dim, ex, kinds, eps)
    if basis == "staggered":
        lam = [v[:, 1:] for v in lam]
    if basis == "divfree":
        lam = [v @ b for v in lam for b in Bc]
    R, apply = _qr(rows[..., None] * P)
    ys = [_rt_solve(R, v) for v in lam]
    alpha = [rows * apply(y) for y in ys]
    if normals is None:
        return np.stack(alpha, 1)
    f = sum(normals[:, d, None].astype(LD) * g for d, g in enumerate(_functionals(dim, ex, ["grad"], eps)))
    z = _rt_solve(R, f)
    az = rows * apply(z)
    beta = [(z * y).sum(1) / (z * z).sum(1) for y in ys]
    return np.stack([a - b[:, None] * az for a, b in zip(alpha, beta)], 1), np.stack(beta, 1)
