"""The error bound that the nearest-centroid shortlist relies on, checked on the CPU with numpy's fp16 and fp32.

The device pass forms g = <hq, hc> - |c|^2 / 2 from rows rounded to fp16 (one power-of-two scale for all rows of a chunk, one
for the table) and accumulated in fp32 from a start value s = (-1/2 + k) |c|^2, k = (Dp + 32) 2^-24.  With the lengths of the rows
and of their rounding errors (rounded up, at least 2^-50 in scaled units), and with the largest of a tile of 128 centroids,
    e = |dq| cm + (|q| + |dq|) dcm + k |q| cm,
the exact G = <q,c> - |c|^2 / 2 lies in [acc + back s_min - e, acc + e], back = 2 k / (1/2 - k); a centroid whose upper end is below
the largest lower end of a row is not its nearest.  The same with a centroid's own lengths decides which pairs are looked at.
Here all of this is formed as the kernels form it (csrc/coarse.hpp: pack_hi_rows_kernel, shortlist_tiles_kernel, shortlist_eps,
shortlist_lower), in fp32, the products one after the other.
"""
import numpy as np
import pytest

F = np.float32


def _scale(X):
    """hi_scale of the largest finite magnitude: the exponent that takes it into [2^14, 2^15)."""
    m = np.abs(X[np.isfinite(X)]).max(initial=F(0))
    e = int(F(m).view(np.uint32) >> 23) - 127
    return 14 - min(max(e, -62), 62)


def _pack(X, sh):
    """(fp16 rows as fp32, lengths, lengths of the rounding errors) of scaled rows."""
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        f = np.ldexp(X, sh).astype(F)
        h = f.astype(np.float16).astype(F)
        d = f - h
        up = F(1 + 2.0 ** -10)
        s2, d2 = np.zeros(len(X), F), np.zeros(len(X), F)
        for t in range(X.shape[1]):
            s2 += f[:, t] * f[:, t]
            d2 += d[:, t] * d[:, t]
        fits = (s2 < np.inf) & (d2 < np.inf)
        ln, dl = np.sqrt(s2 + F(2.0 ** -100)) * up, np.sqrt(d2 + F(2.0 ** -100)) * up
    h[~fits] = 0
    ln[~fits] = dl[~fits] = np.inf
    return h, ln, dl


def _bounds(Q, C, k_factor=1.0, start_factor=1.0, lengths=True):
    """(G in fp64, lower and upper ends with a tile's lengths, the same with a centroid's own), all in units of the product."""
    Dp = (Q.shape[1] + 31) // 32 * 32
    k = F(k_factor * (Dp + 32) * 2.0 ** -24)
    back = F(2) * k / (F(0.5) - k)
    sq, sc = _scale(Q), _scale(C)
    hq, ql, dq = _pack(Q, sq)
    hc, cl, dc = _pack(C, sc)
    if not lengths:
        dq, dc = dq * 0, dc * 0
    len0 = cl * F(1 / (1 + 2.0 ** -10))
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        start = F(start_factor) * (F(-0.5) + k) * np.ldexp(len0 * len0, sq - sc).astype(F)
        good = np.isfinite(cl)
        start[~good] = -np.inf
        acc = np.tile(start, (len(Q), 1))
        for t in range(Q.shape[1]):
            acc += hq[:, t, None] * hc[None, :, t]                # each product exact in fp32

        def eps(c, d):
            return dq[:, None] * c + ((ql + dq)[:, None] * d + k * ql[:, None] * c)

        T = (len(C) + 127) // 128
        pad = lambda a, v: np.concatenate([np.where(good, a, v), np.full(T * 128 - len(C), v, F)]).reshape(T, 128)
        wide = lambda a: np.repeat(a, 128)[:len(C)]
        e = eps(wide(pad(cl, 0).max(1)), wide(pad(dc, 0).max(1)))
        low, up = back * wide(pad(start, np.inf).min(1)) + acc - e, acc + e
        own = eps(np.where(good, cl, 0), np.where(good, dc, 0))
        low1, up1 = back * np.where(good, start, 0) + acc - own, acc + own
    q64, c64 = np.ldexp(Q.astype(np.float64), sq), np.ldexp(C.astype(np.float64), sc)
    G = q64 @ c64.T - 0.5 * np.ldexp((c64 ** 2).sum(1), sq - sc)
    return G, low, up, low1, up1


def _holds(G, low, up):
    return (G >= low) & (G <= up)


def _rows(kind, rng):
    D = {"unit": 96, "sift": 128, "scales": 64, "midpoints": 32, "wide": 260, "narrow": 20, "huge row": 40}[kind]
    C = rng.standard_normal((500, D))
    if kind == "unit":
        C /= np.linalg.norm(C, axis=1, keepdims=True)
    if kind == "sift":
        C = np.clip(np.round(10 * C ** 2), 0, 255)
    if kind == "scales":
        C *= np.exp2(rng.integers(-30, 1, (500, 1)))
    if kind == "midpoints":                                   # halfway between two fp16 numbers: the errors are as large as they get
        C = np.tile((1 + 2.0 ** -11) * np.exp2(np.arange(D) % 3), (500, 1)) * rng.choice([-1, 1], (500, D))
    if kind == "huge row":
        C *= 2.0 ** -30
    Q = C[rng.integers(0, 500, 300)] + 0.05 * np.linalg.norm(C, axis=1).mean() / np.sqrt(D) * rng.standard_normal((300, D))
    if kind == "huge row":                                    # nothing is left of the others under its scale
        Q[7] = 0
        Q[7, 3] = 2.0 ** 62
    return Q.astype(F), C.astype(F)


@pytest.mark.parametrize("kind", ["unit", "sift", "scales", "midpoints", "wide", "narrow", "huge row"])
def test_bound_holds_and_its_list_holds_the_nearest(kind):
    Q, C = _rows(kind, np.random.default_rng(5))
    G, low, up, low1, up1 = _bounds(Q, C)
    assert _holds(G, low, up).all() and _holds(G, low1, up1).all()
    best = G == G.max(1, keepdims=True)
    L = np.maximum(low, low1).max(1, keepdims=True)
    assert (up >= L)[best].all() and (up1 >= L)[best].all()
    if kind in ("unit", "sift"):                               # ... and stays short on such data
        assert (up1 >= L).sum(1).max() < 60


def test_bound_needs_the_lengths_of_the_rounding_errors():
    """On rounding midpoints the errors of a row and of its centroid have the same sign: without the lengths the bound is broken
    by far more than the roundings, with them it is filled to a good part."""
    Q, C = _rows("midpoints", np.random.default_rng(6))
    Q = C[:300]
    G, low, up, low1, up1 = _bounds(Q, C)
    assert _holds(G, low1, up1).all()
    assert not _holds(*[_bounds(Q, C, lengths=False)[i] for i in (0, 3, 4)]).all()
    mid, half = (low1 + up1) / 2, (up1 - low1) / 2
    assert (np.abs(G - mid) / half).max() > 0.5


def test_bound_needs_its_rounding_terms():
    """Whole numbers that fp16 holds: the rows are packed without an error, and what is left is the rounding of the sums and
    of the norms.  Without k (in the bound and in the start value) and with a start value off by 2^-12 of itself,
    2^-13 |c|^2 where the bound has room for k (|c|^2 + |q| |c|), about 2^-14.9 |c|^2, the bound is broken."""
    rng = np.random.default_rng(7)
    C = rng.integers(1000, 2048, (300, 256)).astype(F)
    Q = rng.integers(1000, 2048, (200, 256)).astype(F)
    assert _pack(C, _scale(C))[2].max() < 2.0 ** -49
    G, low, up, low1, up1 = _bounds(Q, C)
    assert _holds(G, low, up).all() and _holds(G, low1, up1).all()
    for off in ({"k_factor": 0.0}, {"start_factor": 1 + 2.0 ** -12}, {"start_factor": 1 - 2.0 ** -12}):
        G, low, up, low1, up1 = _bounds(Q, C, **off)
        assert not _holds(G, low1, up1).all(), off


def test_rows_that_are_not_finite_leave_the_others_alone():
    """The scale is that of the finite values, a row that has no length packs to zeros, and a centroid without one is out of
    the tile's bounds."""
    Q, C = _rows("unit", np.random.default_rng(8))
    Q, C = Q * F(1e6), C * F(1e6)
    ref = _bounds(Q, C)
    Q2, C2 = Q.copy(), C.copy()
    Q2[3], Q2[9, 5] = np.nan, np.inf
    C2[130], C2[200, 0] = np.nan, -np.inf
    with np.errstate(invalid="ignore"):
        got = _bounds(Q2, C2)
    q, c = np.setdiff1d(np.arange(len(Q)), [3, 9]), np.setdiff1d(np.arange(len(C)), [130, 200])
    for a, b in zip(ref[3:], got[3:]):
        assert np.array_equal(a[np.ix_(q, c)], b[np.ix_(q, c)])
    assert _holds(*[a[np.ix_(q, c)] for a in (got[0], got[1], got[2])]).all()
    assert (got[2][np.ix_(q, [130, 200])] == -np.inf).all()
