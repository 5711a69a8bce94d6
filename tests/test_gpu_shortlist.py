"""Nearest-centroid assignment through the certified shortlist (reduced-precision pass with an error
bound, exact decision among the listed pairs) against fp64 brute force: the returned centroid must be
the exact nearest one, whatever the magnitudes, however many ties there are, and also where the list
overflows and the one-pass kernel takes over."""
import os

import numpy as np
import pytest
import torch

import paper_1802_02422_amd as ivf

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _exact(C, Q):
    c64, q64 = C.astype(np.float64), Q.astype(np.float64)
    d = (q64 ** 2).sum(1)[:, None] + (c64 ** 2).sum(1)[None, :] - 2.0 * q64 @ c64.T
    return np.maximum(d, 0.0)


def _assign(C, Q):
    gid, gd = ivf.ivf_coarse_topk(torch.from_numpy(C).cuda(), torch.from_numpy(Q).cuda(), 1)
    return gid.cpu().numpy()[:, 0].astype(np.int64), gd.cpu().numpy()[:, 0].astype(np.float64)


def _check(C, Q, gid, gd):
    """ids: the fp64 nearest, or within the fp32 rounding of the exact pass of it; distances within that rounding."""
    d = _exact(C, Q)
    best = d.min(1)
    tol = 16 * U * ((Q.astype(np.float64) ** 2).sum(1) + (C.astype(np.float64) ** 2).sum(1).max())
    got = d[np.arange(len(Q)), gid]
    assert (got <= best + tol).all(), float(((got - best) / tol).max())
    assert (np.abs(gd - got) <= tol).all()
    # clear winners must be returned exactly, and among exact duplicates of the winner the smallest id
    first = d.argmin(1)                                   # numpy: the first minimum = the smallest id
    second = np.partition(d, 1, axis=1)[:, 1] if d.shape[1] > 1 else np.full(len(Q), np.inf)
    clear = second - best > 2 * tol
    assert (gid[clear] == first[clear]).all()
    return int((~clear).sum())


@pytest.mark.parametrize("D,K,nq", [(96, 4096, 3000), (128, 1000, 700), (20, 300, 1), (100, 2500, 129), (64, 64, 50),
                                    (96, 1000, 300), (96, 50, 40), (96, 20000, 500), (128, 128, 128)])
def test_shortlist_assignment_is_the_exact_nearest(D, K, nq):
    """Widths of 1 to 4 stages of the swept kernel (20 -> 32, 64, 96, 100 -> 128; wider rows take the tile kernel, below); whole
    and partial last centroid tiles, fewer centroids than a tile, more tiles than one workgroup sweeps, one row."""
    print("case: shortlist", D, K, nq, flush=True)
    rng = np.random.default_rng(7 * D + K + nq)
    # clustered points around the centroids, rows of very different magnitude, a point that is a centroid
    C = rng.standard_normal((K, D)) * np.exp2(rng.integers(-12, 1, size=(K, 1)))
    own = rng.integers(0, K, size=nq)
    Q = C[own] + 0.3 * rng.standard_normal((nq, D)) * np.linalg.norm(C[own], axis=1, keepdims=True) / np.sqrt(D)
    Q[0] = C[K // 2]
    C, Q = C.astype(np.float32), Q.astype(np.float32)
    before = ivf.ivf_assign_stats()
    gid, gd = _assign(C, Q)
    after = ivf.ivf_assign_stats()
    assert after[0] == before[0] + 1 and after[1] == before[1]      # decided by the shortlist, no fallback
    _check(C, Q, gid, gd)
    assert gid[0] == K // 2 and gd[0] <= 16 * U * 2 * float((Q[0].astype(np.float64) ** 2).sum())


def test_shortlist_with_many_near_ties_and_duplicates():
    """Unit vectors in few dimensions: thousands of centroids at almost the same distance from every
    query, a quarter of them exact duplicates.  Still the exact nearest, the smallest id among duplicates."""
    print("case: shortlist near-ties", flush=True)
    rng = np.random.default_rng(11)
    D, K, nq = 8, 4096, 600
    C = rng.standard_normal((K, D))
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    C[K // 4 * 3:] = C[:K // 4]                                      # duplicates with larger ids
    Q = rng.standard_normal((nq, D))
    Q /= np.linalg.norm(Q, axis=1, keepdims=True)
    C, Q = C.astype(np.float32), Q.astype(np.float32)
    gid, gd = _assign(C, Q)
    _check(C, Q, gid, gd)
    assert (gid < K // 4 * 3).all()                                  # never the larger id of a duplicate pair


def test_list_overflow_falls_back_to_the_one_pass_kernel():
    """Every centroid the same vector: every pair is a candidate, the list overflows, the exact kernel decides
    and returns id 0 for every row."""
    print("case: shortlist overflow", flush=True)
    rng = np.random.default_rng(12)
    D, K, nq = 32, 2048, 4096
    C = np.tile(rng.standard_normal((1, D)), (K, 1)).astype(np.float32)
    Q = rng.standard_normal((nq, D)).astype(np.float32)
    before = ivf.ivf_assign_stats()
    gid, gd = _assign(C, Q)
    after = ivf.ivf_assign_stats()
    assert after[1] == before[1] + 1 and after[0] == before[0]      # the fallback ran
    assert (gid == 0).all()
    d = _exact(C, Q)[:, 0]
    assert (np.abs(gd - d) <= 16 * U * ((Q.astype(np.float64) ** 2).sum(1) + float((C[0].astype(np.float64) ** 2).sum()))).all()


def test_shortlist_and_one_pass_kernel_agree(small):
    """The two ways of deciding a chunk on a real workload: the same region for every point that has a
    clear nearest centroid, and both within rounding of the fp64 minimum everywhere."""
    spec, ix, Q, X = small
    print("case: shortlist vs one-pass on the small workload", flush=True)
    C = ix.centroids
    P = X[:20000]
    a_id, a_d = _assign(C, P)
    os.environ["IVF_GP_EXACT_ASSIGN"] = "1"
    try:
        b_id, b_d = _assign(C, P)
    finally:
        del os.environ["IVF_GP_EXACT_ASSIGN"]
    unclear = _check(C, P, a_id, a_d)
    _check(C, P, b_id, b_d)
    assert (a_id != b_id).sum() <= unclear


def _mixed_chunk(D, K, nq):
    """Rows and centroids of sizes 1 and 10^6, where fp16 without a scale would overflow."""
    rng = np.random.default_rng(D + K + nq)
    C = rng.standard_normal((K, D)) * np.where(rng.random((K, 1)) < 0.5, 1.0, 1e6)
    own = rng.integers(0, K, nq)
    Q = C[own] + 0.3 * rng.standard_normal((nq, D)) * np.linalg.norm(C[own], axis=1, keepdims=True) / np.sqrt(D)
    return C.astype(np.float32), Q.astype(np.float32)


@pytest.mark.parametrize("D,K,nq", [(96, 1000, 700), (136, 300, 257), (24, 70, 1000)])
@pytest.mark.parametrize("bad", ["nan", "inf", "both"])
def test_rows_that_are_not_finite_harm_only_themselves(D, K, nq, bad):
    """Rows with an infinity or not a number in them have no nearest centroid; all the others of their chunk do."""
    print("case: shortlist, rows not finite", D, K, nq, bad, flush=True)
    C, Q = _mixed_chunk(D, K, nq)
    lost = np.zeros(nq, bool)
    if bad != "inf":
        Q[5, D - 1], Q[nq - 1] = np.nan, np.nan
        lost[[5, nq - 1]] = True
    if bad != "nan":
        Q[130, 3], Q[131, 0] = np.inf, -np.inf
        lost[[130, 131]] = True
    before = ivf.ivf_assign_stats()
    gid, gd = _assign(C, Q)
    after = ivf.ivf_assign_stats()
    assert after[0] == before[0] + 1 and after[1] == before[1]
    assert (gid[lost] == -1).all()
    _check(C, Q[~lost], gid[~lost], gd[~lost])


@pytest.mark.parametrize("D,K,nq", [(96, 1000, 700), (132, 300, 257)])
def test_centroids_that_are_not_finite_are_nobodys_nearest(D, K, nq):
    print("case: shortlist, centroids not finite", D, K, nq, flush=True)
    C, Q = _mixed_chunk(D, K, nq)
    bad = np.array([3, 130, K - 1])
    Q = Q[:nq]
    C[3], C[130, 1], C[K - 1, D - 1] = np.nan, np.inf, -np.inf
    gid, gd = _assign(C, Q)
    assert not np.isin(gid, bad).any() and (gid >= 0).all()
    good = np.setdiff1d(np.arange(K), bad)
    place = np.full(K, -1)
    place[good] = np.arange(len(good))
    _check(C[good], Q, place[gid], gd)


def test_centroid_that_is_not_a_number_leaves_the_tables_scale_alone():
    """The distances of the other centroids keep their accuracy (in the distance tile, P > 1)."""
    print("case: distance tile, centroid not a number", flush=True)
    rng = np.random.default_rng(3)
    C = (1e6 * rng.standard_normal((300, 96))).astype(np.float32)
    Q = (C[rng.integers(0, 299, 50)] + 1e5 * rng.standard_normal((50, 96))).astype(np.float32)
    C[299] = np.nan
    ids, d = (v.cpu().numpy() for v in ivf.ivf_coarse_topk(torch.from_numpy(C).cuda(), torch.from_numpy(Q).cuda(), 4))
    full = _exact(C[:299], Q)
    tol = 16 * U * ((Q.astype(np.float64) ** 2).sum(1) + (C[:299].astype(np.float64) ** 2).sum(1).max())
    for q in range(50):
        m = ids[q] != 299
        assert (np.abs(d[q][m] - full[q][ids[q][m]]) <= tol[q]).all()
        assert (full[q][ids[q][m]] <= np.sort(full[q])[3] + 2 * tol[q]).all()


@pytest.mark.parametrize("D", [96, 132])
def test_one_huge_row_does_not_hide_the_others(D):
    """A row 2^92 times the size of the others of its chunk: what is left of those under the chunk's scale is nothing, and
    the bound has to know."""
    print("case: shortlist, one huge row", D, flush=True)
    rng = np.random.default_rng(9)
    K, nq = 500, 300
    C = (2.0 ** -30 * rng.standard_normal((K, D))).astype(np.float32)
    Q = (C[rng.integers(0, K, nq)] + 2.0 ** -33 * rng.standard_normal((nq, D))).astype(np.float32)
    Q[77] = 0
    Q[77, 5] = 2.0 ** 62
    gid, gd = _assign(C, Q)
    assert gid[77] >= 0
    keep = np.arange(nq) != 77
    _check(C, Q[keep], gid[keep], gd[keep])


@pytest.mark.parametrize("D,M,codes", [(96, 8, True), (96, 8, False), (136, 8, False), (40, 8, True)])
def test_encoder_takes_rows_that_are_not_finite(D, M, codes):
    """They go to region 0, subregion 0 and, where the displacement is not a number, word 0; the other rows to their own.
    Both subregion kernels and both code kernels (D = 136; D / M = 5)."""
    print("case: encoder, rows not finite", D, M, codes, flush=True)
    K, nq = 50, 257
    assert nq * 2 >= 10 * K                                    # points enough for the table of 8-bit rows, where D takes it
    C, Q = _mixed_chunk(D, K, nq)
    lost = np.array([5, 130, 256])
    Q[5], Q[130, 3], Q[256, D - 1] = np.nan, np.inf, np.nan
    rest = np.setdiff1d(np.arange(nq), lost)
    nbr = np.stack([(np.arange(K) + 1) % K, (np.arange(K) + 2) % K], 1).astype(np.int32)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cb = np.random.default_rng(1).standard_normal((M, 256, D // M)).astype(np.float32)
    d = ivf.IndexDesc(up(C), up(nbr), up(np.zeros(K, np.float32)), up(np.zeros((K, 2), np.float32)), up(cb) if codes else None,
                      M=M, const_table=up(np.linspace(-1, 1, 256, dtype=np.float32)) if codes else None)
    region, sub, code, byte, _ = ivf.ivf_encode(d, up(Q))
    region, sub = region.cpu().numpy(), sub.cpu().numpy()
    gid, gd = _assign(C, Q)
    assert (region[lost] == 0).all() and (region[rest] == gid[rest]).all() and (sub == 0).all()
    if codes:
        assert (code.cpu().numpy()[5] == 0).all()
        alone = ivf.ivf_encode(d, up(Q[rest]))
        assert (alone[2].cpu().numpy() == code.cpu().numpy()[rest]).all() and (alone[3].cpu().numpy() == byte.cpu().numpy()[rest]).all()


@pytest.mark.parametrize("D,K,nq", [(132, 700, 300), (160, 128, 129), (256, 2000, 500), (1024, 300, 130)])
def test_wide_rows_take_the_tile_kernel(D, K, nq):
    """More than 128 dimensions: one tile of rows and centroids a workgroup, partial ones of either, rows of different size;
    decided by the shortlist, and by the one-pass kernel where every centroid is the same."""
    print("case: shortlist, wide rows", D, K, nq, flush=True)
    rng = np.random.default_rng(D + K)
    C = rng.standard_normal((K, D)) * np.exp2(rng.integers(-6, 1, size=(K, 1)))
    own = rng.integers(0, K, size=nq)
    Q = C[own] + 0.3 * rng.standard_normal((nq, D)) * np.linalg.norm(C[own], axis=1, keepdims=True) / np.sqrt(D)
    C, Q = C.astype(np.float32), Q.astype(np.float32)
    before = ivf.ivf_assign_stats()
    gid, gd = _assign(C, Q)
    after = ivf.ivf_assign_stats()
    assert after[0] == before[0] + 1 and after[1] == before[1]
    _check(C, Q, gid, gd)
    big = np.tile(Q, (20000 // nq + 1, 1))
    gid, gd = _assign(np.tile(C[:1], (2048, 1)), big)
    last = ivf.ivf_assign_stats()
    assert last[1] == after[1] + 1 and last[0] == after[0]
    assert (gid == 0).all()


@pytest.mark.parametrize("D,K,nq", [(96, 8191, 16_640), (96, 300, 350_000), (20, 40_001, 3400), (64, 16_385, 8193), (128, 8320, 16_129),
                                    (96, 140_001, 1000), (32, 66_000, 3000)])
def test_rows_enough_for_a_wavefront_to_64(D, K, nq):
    """The sweep whose workgroups take 256 rows (from 8192 tiles of 128 x 128 on): partial last tiles of rows and centroids, a last
    workgroup with rows for one wavefront, sweeps of odd and even numbers of tiles.  The last two have tiles enough and stay with 128 rows
    a workgroup, since 256 would leave some of the XCDs without."""
    print("case: wide sweep", D, K, nq, flush=True)
    assert -(-nq // 128) * -(-K // 128) >= 8192
    g = torch.Generator(device="cuda").manual_seed(D + K + nq)
    C = torch.randn(K, D, generator=g, device="cuda")
    own = torch.randint(0, K, (nq,), generator=g, device="cuda")
    Q = C[own] + 0.4 * torch.randn(nq, D, generator=g, device="cuda")
    before = ivf.ivf_assign_stats()
    gid, gd = ivf.ivf_coarse_topk(C, Q, 1)
    assert ivf.ivf_assign_stats()[0] > before[0]
    c64 = C.double()
    cn = (c64 ** 2).sum(1)
    for a in range(0, nq, 4096):
        q = Q[a:a + 4096].double()
        qn = (q ** 2).sum(1)
        d = (qn[:, None] + cn[None]).addmm_(q, c64.t(), alpha=-2.0).clamp_(min=0.0)
        best, first = d.min(1)
        tol = 16 * U * (qn + cn.max())
        at = gid[a:a + 4096, 0].long()
        got = d.gather(1, at[:, None])[:, 0]
        assert bool((got <= best + tol).all()) and bool(((gd[a:a + 4096, 0].double() - got).abs() <= tol).all())
        d.scatter_(1, first[:, None], float("inf"))
        clear = d.min(1)[0] - best > 2 * tol
        assert bool((at[clear] == first[clear]).all())
