"""The error bound behind the subregions found from 8-bit rows, checked on the CPU with numpy's fp32.

A neighbour's row is s' = step q + d (s' = s - centre, q whole and at most 127), a point x' = u w + dx with w in 15 bits.  With
everything a region's neighbours have in common left out (|x'|^2 - 2 <dx, x'> and the share of the region's centroid) a neighbour's
score is a times
    |s'|^2            - 2 step u <w, q>   to within 2 (|dx| |x' - step q| + |x'| |d|)             or
    |s'|^2 - 2 <step q, d> - 2 step u <w, q>   to within 2 (|dx| |x' - step q| + |x' - step q| |d|),
of which the kernel takes what leaves less out, minus a (1 - a) cs.  Here that is formed as the kernels form it
(csrc/encode.hpp: pack_byte_rows_kernel, subregion_kernel) and compared with the fp32 score that decides (encode_kernel's).
"""
import numpy as np
import pytest

F = np.float32


def _fma(a, b, c):
    return (np.asarray(a, np.float64) * b + c).astype(F)


def _sum2(v):
    s = np.zeros(v.shape[:-1], F)
    for t in range(v.shape[-1]):
        s = _fma(v[..., t], v[..., t], s)
    return s


def _pack(C, centre):
    """q, step, |s'|^2, |d| and 2 <step q, d>, lengths rounded up."""
    v = (C - centre).astype(F)
    big = np.abs(v).max(1)
    step = big * F(1 / 127)
    q = np.clip(np.rint(v * np.where(big > 0, F(127) / np.where(big > 0, big, 1), 0).astype(F)[:, None]), -127, 127).astype(F)
    d = _fma(-q, step[:, None], v)
    qd = np.zeros(len(C), F)
    for t in range(C.shape[1]):
        qd = _fma(q[:, t] * step, d[:, t], qd)
    return q, step, _sum2(v), np.sqrt(_sum2(d)) * F(1 + 2.0 ** -10), F(2) * qd


def _chain(X, S):
    """Squared distances as encode_kernel sums them: lanes of four components, then a tree of sixteen."""
    D = X.shape[-1]
    lanes = []
    for c in range(16):
        acc = np.zeros(np.broadcast_shapes(X.shape, S.shape)[:-1], F)
        for t in [4 * (c + 16 * h) + k for h in range(2) for k in range(4)]:
            if t < D:
                u = (X[..., t] - S[..., t]).astype(F)
                acc = _fma(u, u, acc)
        lanes.append(acc)
    for o in (8, 4, 2, 1):
        lanes = [lanes[c] + lanes[c ^ o] for c in range(16)]
    return lanes[0]


def _scores(X, S, c, alpha, centre=None, near=True, ds=True, dx=True, qd=True, roundings=True):
    """(the fp32 score of every point and neighbour without what they have in common, h, err): X [n][D], S [L][D], c [D], alpha [n]."""
    D, Dp = X.shape[1], (X.shape[1] + 31) // 32 * 32
    centre = np.zeros(D, F) if centre is None else centre
    a = alpha.astype(F)[:, None]
    cs = _chain(c[None], S)[None]
    q, step, s2, dl, g = _pack(S, centre)
    _, _, c2, _, _ = _pack(c[None], centre)
    xc = (X - centre).astype(F)
    big = np.abs(xc).max(1)
    u = big * F(1 / 16256)
    w = np.clip(np.rint(xc * (F(16256) / big)[:, None]), -16256, 16256)
    rest = _fma(-w, u[:, None], xc)
    x2, xl, rl = (v[:, None] for v in (_sum2(xc), np.sqrt(_sum2(xc) + F(2.0 ** -100)) * F(1 + 2.0 ** -10), np.sqrt(_sum2(rest) + F(2.0 ** -100)) * F(1 + 2.0 ** -10)))
    if not ds:
        dl = dl * 0
    if not dx:
        rl = rl * 0
    if not qd:
        g = g * 0
    dot = (w.astype(np.int64) @ q.T.astype(np.int64)).astype(F) * (u[:, None] * step[None])
    both, ln = x2 + s2, np.sqrt(s2) * F(1 + 2.0 ** -10)
    far2 = _fma(-2, dot, both - g) + _fma(2 * rl, ln + dl, F(2.0 ** -18) * both)
    far = np.sqrt(np.maximum(far2, 0)) * F(1 + 2.0 ** -10)
    closer = (far < xl) & near
    h = _fma(a, _fma(-2, dot, np.where(closer, s2 - g, s2)), -a * (1 - a) * cs)
    k = F(Dp + 32) * F(2.0 ** -24) if roundings else F(0)
    e = _fma(rl, far, _fma(np.where(closer, far, xl), dl, k * xl * ln))
    aa, ac = np.abs(a), np.abs(1 - a)
    size = _fma(aa, both, _fma(ac, x2 + c2, aa * ac * np.abs(cs)))
    err = _fma(2 * aa, e, (_fma(aa * F(D // 16 + 12) * F(2.0 ** -23), both, F(2.0 ** -20) * size) if roundings else 0) + F(2.0 ** -120))
    dxc = _chain(X, c[None])[:, None]
    sc = _fma(a, _chain(X[:, None], S[None]), _fma(1 - a, dxc, -a * (1 - a) * cs))
    x64, a64 = xc.astype(np.float64), a.astype(np.float64)
    shared = (1 - a64) * dxc + a64 * ((x64 ** 2).sum(1) - 2 * (rest.astype(np.float64) * x64).sum(1))[:, None]
    return sc, sc.astype(np.float64) - shared, h.astype(np.float64), err.astype(np.float64)


KINDS = ("unit", "sift", "decay", "groups", "offset", "narrow", "near")


def _rows(kind, rng, n=200, L=64):
    D = {"sift": 128, "narrow": 20, "near": 64}.get(kind, 96)
    S = rng.standard_normal((L + 1, D))
    if kind == "sift":
        S = np.clip(np.round(10 * S ** 2), 0, 255)
    else:
        S /= np.linalg.norm(S, axis=1, keepdims=True)
    if kind == "decay":
        S *= np.arange(1, D + 1) ** -0.5
    if kind == "groups":                                      # a group of centroids a few times its width from the table's middle
        m = rng.standard_normal(D)
        S += 4 * m / np.linalg.norm(m)
    if kind == "near":                                        # neighbours at a tenth of their length
        S = S[:1] + 0.1 * S
    noise = 6.0 if kind == "sift" else 0.02 if kind == "near" else 0.065
    X = S[L] + noise * rng.standard_normal((n, D))
    centre = np.zeros(D)
    if kind == "offset":
        S, X, centre = S + 1000, X + 1000, centre + 1000
    return X.astype(F), S[:L].astype(F), S[L].astype(F), centre.astype(F)


@pytest.mark.parametrize("alpha", [None, 1.0, -3.0, 7.0])
@pytest.mark.parametrize("kind", KINDS)
def test_bound_holds_and_keeps_the_answer(kind, alpha):
    rng = np.random.default_rng(3)
    X, S, c, centre = _rows(kind, rng)
    a = rng.uniform(0.05, 0.17, len(X)) if alpha is None else np.full(len(X), alpha)
    sc, true, h, err = _scores(X, S, c, a, centre)
    assert (np.abs(h - true) <= err).all()
    listed = ~(h - err > (h + err).min(1, keepdims=True))
    assert listed[sc == sc.min(1, keepdims=True)].all()
    if alpha is None and kind in ("unit", "decay", "offset", "narrow"):   # ... and few are left to the fp32 scores
        assert listed.sum(1).mean() < 4


def test_distance_to_the_row_takes_the_place_of_the_points_length():
    """Far from the table's middle the bound follows the distances of the neighbours, not the length of the point."""
    X, S, c, centre = _rows("groups", np.random.default_rng(4))
    a = np.full(len(X), 0.1)
    few, many = ((lambda t: (~(t[2] - t[3] > (t[2] + t[3]).min(1, keepdims=True))).sum(1).mean())(_scores(X, S, c, a, centre, near=b)) for b in (True, False))
    assert 2 * few < many


def test_bound_needs_each_of_its_terms():
    """Rows and points whose roundings all point the same way fill it; without a term they break it, and so do sums without
    any allowance for their own roundings where rows and points are packed without an error."""
    rng = np.random.default_rng(5)
    D, L, n = 96, 64, 50
    holds = lambda X, S, c, **off: (lambda t: (np.abs(t[2] - t[1]) <= t[3]).all())(_scores(X, S, c, np.ones(len(X)), **off))
    c = rng.standard_normal(D).astype(F)
    X = rng.standard_normal((n, D)).astype(F)
    S = np.rint(40 * rng.standard_normal((L, D))) + 0.49 * np.sign(rng.standard_normal((L, D)))   # (steps of 1 below)
    S[:, 0] = 127
    for scale in (30, 300):                                    # both forms
        Y = (scale * np.sign(S[:n] - np.rint(S[:n]))).astype(F)
        assert holds(Y, S.astype(F), c) and not holds(Y, S.astype(F), c, ds=False)
    Y = (np.rint(S[:n]) + 50 * np.sign(S[:n] - np.rint(S[:n])) + 100 * np.sign(S[:n])).astype(F)
    T = (np.rint(S) + 0.49 * np.sign(S)).astype(F)             # the errors all along the row
    Y = T[:n] + F(0.2) * X
    assert holds(Y, T, c) and not holds(Y, T, c, qd=False)
    Q = np.rint(40 * rng.standard_normal((L, D))).astype(F)    # rows without an error
    Q[:, 0] = 127
    W = np.rint(5000 * rng.standard_normal((n, D)))
    W = W + 0.49 * np.sign(W - Q[:n])
    W[:, 0] = 16256
    assert holds(W.astype(F), Q, c) and not holds(W.astype(F), Q, c, dx=False)
    W = np.rint(W).astype(F)
    assert holds(W, Q, c) and not holds(W, Q, c, roundings=False)
