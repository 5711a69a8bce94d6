"""The bound by which the search without the distance matrix lists blocks of 64 centroids, checked on the CPU with numpy's fp16 and fp32.

The sweep leaves x = the largest of <hq, hc> - (1/2 - k) |c|^2 over a block, from fp16 rows (the table's at its scale, the queries'
at the same, 2^-10 of it).  As a distance in units of the product, |q|^2 - 2 G, the block's smallest one lies between two
ends that are widened by the rounding of the exact distances too; the P-th smallest upper end of the pieces (of every TP
tiles) bounds the P-th smallest distance, blocks whose lower end does not exceed it are listed, and thr is the bound as a
distance.  Where that lists more than cap blocks, bins of equal width over the upper ends of all blocks give a closer bound.  All of
this is formed as the kernels form it (csrc/sparse.hpp: minima_tiles_kernel, sparse_queries_kernel, flag_blocks_kernel), in fp32.
"""
import numpy as np
import pytest

from test_shortlist_bound import F, _pack, _scale

HEAD = 10                                                     # the queries' rows are 2^-10 of the table's scale


def _ends(Q, C, lengths=1.0, start_factor=1.0):
    """(fp64 smallest distances of the blocks, upper ends, gaps to the lower ends, |q|^2 as the kernel has it) in units of the product."""
    K, Dp = len(C), (Q.shape[1] + 31) // 32 * 32
    k = F((Dp + 32) * 2.0 ** -24)
    back = F(2) * k / (F(0.5) - k)
    sc = _scale(C)
    sq = sc - HEAD
    hq, ql, dq = _pack(Q, sq)
    hc, cl, dc = _pack(C, sc)
    good = np.isfinite(cl)
    len0 = cl * F(1 / (1 + 2.0 ** -10))
    T = (K + 127) // 128
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        start = F(start_factor) * (F(-0.5) + k) * np.ldexp(len0 * len0, -HEAD).astype(F)
        start = np.where(good, start, -np.inf).astype(F)
        acc = np.tile(start, (len(Q), 1))
        for t in range(Q.shape[1]):
            acc += hq[:, t, None] * hc[None, :, t]            # each product exact in fp32
        x = np.full((len(Q), 2 * T * 64), -np.inf, F)
        x[:, :K] = acc
        x = x.reshape(len(Q), 2 * T, 64).max(2)
        pad = lambda a, v: np.concatenate([a, np.full(T * 128 - K, v, F)]).reshape(T, 128)
        wide = lambda a: np.repeat(a.astype(F), 2)[None, :]   # of a tile, for its two blocks
        c, d = wide(pad(cl, 0).max(1)), wide(pad(dc, 0).max(1)) * F(lengths)
        low = back * wide(pad(np.where(good, start, 0), 0).min(1))
        q2 = (F(2.0 ** HEAD) * ql * ql)[:, None]
        eps_q = F(2.0 ** -18) * q2 + F(2.0 ** -20) * ql[:, None]
        eps_c = k * ql[:, None] + dq[:, None] * F(lengths)
        eps_d = (ql + dq)[:, None]
        eps = eps_c * c + (eps_d * d + (F(2.0 ** (-18 - HEAD)) * c * c + eps_q))
        known = eps < np.inf
        far = np.where(known, np.maximum(F(-2) * x + (F(2) * (eps - low) + q2), 0), np.inf).astype(F)
        gap = np.where(known, F(2) * (F(2) * eps - low), np.inf).astype(F)
    nb = (K + 63) // 64
    q64, c64 = np.ldexp(Q.astype(np.float64), sq), np.ldexp(C.astype(np.float64), sc)
    with np.errstate(invalid="ignore", over="ignore"):
        # (the kernel's |q|^2 is that of a length rounded up, the same in all ends of a query and taken off again in thr)
        D = q2.astype(np.float64) + np.ldexp((c64 ** 2).sum(1), -HEAD) - 2 * (q64 @ c64.T)
        room = 16 * 2.0 ** -24 * (np.ldexp((q64 ** 2).sum(1), HEAD)[:, None] + np.ldexp((c64 ** 2).sum(1), -HEAD))   # what the exact distances may be off by
    return D, room, far[:, :nb], gap[:, :nb], q2[:, 0], sc


def _list(far, gap, P, TP, cap):
    """flag_blocks_kernel's decision for one query: (listed, bound)."""
    nb = len(far)
    piece = np.arange(nb) // (2 * TP)
    n = piece[-1] + 1
    least = np.array([far[piece == p].min() for p in range(n)])
    wide = np.array([gap[piece == p].max() for p in range(n)])[piece]
    limit = np.sort(least)[P - 1] if P <= n else F(np.inf)
    with np.errstate(invalid="ignore"):
        listed = (far - wide <= limit) | np.isinf(far)
        if listed.sum() > cap and 0 < limit < np.inf:
            per = F(1024) / F(limit)
            f = far[far <= limit]
            bins = np.minimum(f * per, F(1023)).astype(int)
            bin_ = np.searchsorted(np.cumsum(np.bincount(bins, minlength=1024)), P)
            limit = min(limit, F(bin_ + 1) / per * F(1 + 2.0 ** -20))
            listed = (far - wide <= limit) | np.isinf(far)
    return listed, F(limit)


def _rows(kind, rng):
    D = {"unit": 96, "sift": 128, "scales": 64, "midpoints": 32, "far": 96, "narrow": 20, "same": 32}[kind]
    K = 3333
    C = rng.standard_normal((K, D))
    if kind == "unit":
        C /= np.linalg.norm(C, axis=1, keepdims=True)
    if kind == "sift":
        C = np.clip(np.round(10 * C ** 2), 0, 255)
    if kind == "scales":
        C *= np.exp2(rng.integers(-30, 1, (K, 1)))
    if kind == "midpoints":                                   # halfway between two fp16 numbers: the errors are as large as they get
        C = np.tile((1 + 2.0 ** -11) * np.exp2(np.arange(D) % 3), (K, 1)) * rng.choice([-1, 1], (K, D))
    if kind == "far":
        C = C / np.sqrt(D) + 0.3
    if kind == "same":                                        # several blocks of equal centroids
        C[700:1100] = C[700]
    at = rng.integers(0, K, 60)
    Q = C[at] + 0.3 * np.linalg.norm(C - C.mean(0), axis=1).mean() / np.sqrt(D) * rng.standard_normal((60, D))
    Q[:8] = C[at[:8]]
    Q[8] = 0
    Q[9:12] *= 1.5 * 2 ** HEAD * np.abs(C).max() / np.abs(Q[9:12]).max()   # nearly as large as fp16 rows of that scale hold
    Q[12:15] *= 2.0 ** -np.arange(4, 25, 8)[:, None]
    if kind == "same":
        Q[20:28] = C[700] + 1e-3 * rng.standard_normal((8, D))
    return Q.astype(F), C.astype(F)


KINDS = ["unit", "sift", "scales", "midpoints", "far", "narrow", "same"]


def _block_min(D):
    pad = np.full((len(D), -D.shape[1] % 64), np.inf)
    return np.concatenate([D, pad], 1).reshape(len(D), -1, 64).min(2)


@pytest.mark.parametrize("kind", KINDS)
def test_ends_hold_the_smallest_distance_of_a_block(kind):
    Q, C = _rows(kind, np.random.default_rng(5))
    D, room, far, gap, q2, _ = _ends(Q, C)
    assert (_block_min(D + room) <= far).all() and (_block_min(D - room) >= far.astype(np.float64) - gap).all()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("P,TP", [(1, 1), (5, 1), (16, 2), (12, 4), (40, 1)])
def test_listed_blocks_hold_the_closest(kind, P, TP):
    """Whatever the exact distances are within their rounding: the blocks of all that can be among the P closest are listed, or the query
    is one whose blocks are decided by exact minima; no distance of the P closest is above thr."""
    Q, C = _rows(kind, np.random.default_rng(6))
    D, room, far, gap, q2, sc = _ends(Q, C)
    cap = max(4, 1 << (2 * P - 1).bit_length())
    hard = 0
    for q in range(len(Q)):
        listed, limit = _list(far[q], gap[q], P, TP, cap)
        if listed.sum() > cap:
            hard += 1
            continue
        kth = np.sort(D[q] + room[q])[P - 1]
        dist = kth - q2[q].astype(np.float64) + np.ldexp((Q[q].astype(np.float64) ** 2).sum(), 2 * sc - HEAD)
        can = D[q] - room[q] <= kth
        assert listed[np.unique(np.nonzero(can)[0] // 64)].all(), q
        n = F((Q[q].astype(F) ** 2).sum(dtype=F))
        two_g = np.ldexp(F(limit - q2[q]), HEAD - 2 * sc).astype(F)
        thr = max(n + two_g + F(2.0 ** -21) * (n + abs(two_g)), F(0)) if limit < np.inf else np.inf
        assert thr >= np.ldexp(dist, HEAD - 2 * sc), q
    if kind in ("unit", "sift", "narrow") and P <= 5:          # (53 blocks: more probes than that ask for most of them)
        assert hard < len(Q) // 4


def test_ends_need_the_rounding_errors_of_the_rows_and_the_norms():
    """Planted in the oracle: without the lengths of the rounding errors, and with a start value off by 2^-9 of itself, the ends do not
    hold."""
    Q, C = _rows("midpoints", np.random.default_rng(7))
    Q[:] = C[:60]
    for off in ({"lengths": 0.0}, {"start_factor": 1 + 2.0 ** -9}, {"start_factor": 1 - 2.0 ** -9}):
        D, room, far, gap, q2, _ = _ends(Q, C, **off)
        assert not ((_block_min(D + room) <= far).all() and (_block_min(D - room) >= far.astype(np.float64) - gap).all()), off
    D, room, far, gap, q2, _ = _ends(Q, C)
    assert (_block_min(D + room) <= far).all() and (_block_min(D - room) >= far.astype(np.float64) - gap).all()


def test_far_queries_have_a_bound():
    """A hundred times as far as the table is large: the list stays short."""
    Q, C = _rows("unit", np.random.default_rng(9))
    D, room, far, gap, q2, _ = _ends(Q[20:] * F(100), C)
    assert np.isfinite(far).all()
    assert max(_list(f, g, 5, 1, 16)[0].sum() for f, g in zip(far, gap)) <= 16


def test_centroids_that_are_not_finite_are_always_looked_at():
    Q, C = _rows("unit", np.random.default_rng(8))
    C[130], C[1000, 0] = np.nan, np.inf
    D, room, far, gap, q2, _ = _ends(Q, C)
    for q in range(len(Q)):
        listed, _ = _list(far[q], gap[q], 8, 1, 32)
        assert listed[[2, 3, 14, 15]].all()                   # both blocks of their tiles
    ok = np.setdiff1d(np.arange(far.shape[1]), [2, 3, 14, 15])
    good = _block_min(D + room)[:, ok]
    assert (good <= far[:, ok]).all()
