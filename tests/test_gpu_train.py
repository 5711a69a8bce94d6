"""The device-side index construction routines against the oracle's (needs an MI355X)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import synthdata as sd
import paper_1802_02422_amd as ivf
from oracle import ivf_oracle as orc
import parity


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n,nb", [(1, 1), (4097, 3), (100_000, 70_000), (300_001, 1 << 21), (50_000, 2)])
def test_group_is_a_stable_counting_sort(n, nb):
    print("case: group", n, nb, flush=True)
    rng = np.random.default_rng(n + nb)
    bucket = rng.integers(0, nb, n).astype(np.int32)
    if n > 1000:
        bucket[rng.integers(0, n, n // 3)] = nb - 1        # one crowded bucket, many empty ones
    perm, off = ivf.ivf_group(dev(bucket), nb)
    perm, off = perm.cpu().numpy(), off.cpu().numpy().view(np.uint32).astype(np.int64)
    ref = np.lexsort((np.arange(n), bucket))
    assert (perm == ref).all()
    sizes = np.bincount(bucket, minlength=nb)
    assert off[0] == 0 and (np.diff(off) == sizes).all()
    # the rows in grouped order
    rows = rng.integers(0, 255, (n, 16)).astype(np.uint8)
    got = ivf.ivf_gather_rows(dev(rows), dev(perm.astype(np.int32))).cpu().numpy()
    assert (got == rows[ref]).all()
    b1 = rng.integers(0, 255, n).astype(np.uint8)
    assert (ivf.ivf_gather_rows(dev(b1), dev(perm.astype(np.int32))).cpu().numpy() == b1[ref]).all()
    r, s = rng.integers(0, 1000, n).astype(np.int32), rng.integers(0, 7, n).astype(np.int32)
    assert (ivf.ivf_bucket_ids(dev(r), dev(s), 7).cpu().numpy() == r * 7 + s).all()


def test_cluster_means_and_kmeans_match_oracle(small):
    spec, ix, Q, X = small
    print("case: kmeans small", flush=True)
    mix = sd.make_mixture(spec.kind, spec.n_mix, spec.D)
    Xt = sd.draw_points(mix, spec.n_train, 0, "train")[0].numpy()
    init = sd.draw_indices(spec.n_train, spec.K, "kmeans-init").numpy()
    Xd = dev(Xt)
    # zero rounds: the initial points
    c0 = ivf.ivf_kmeans(Xd, spec.K, 0, dev(init)).cpu().numpy()
    assert (c0 == Xt[init]).all()
    # update step alone, from the oracle's assignment: means in fp64 rounded to fp32
    lab, _ = orc.assign(Xt, c0)
    got = ivf.ivf_cluster_means(Xd, dev(lab), dev(c0)).cpu().numpy()
    sums = np.zeros((spec.K, spec.D))
    np.add.at(sums, lab, Xt.astype(np.float64))
    cnt = np.bincount(lab, minlength=spec.K)
    ref = np.where(cnt[:, None] > 0, sums / np.maximum(cnt, 1)[:, None], c0).astype(np.float32)
    assert np.abs(got - ref).max() <= 1e-7
    assert (got[cnt == 0] == c0[cnt == 0]).all()
    # whole Lloyd runs from the same start
    for iters in (1, 3):
        c_g, obj = ivf.ivf_kmeans(Xd, spec.K, iters, dev(init), want_objective=True)
        c_g, obj = c_g.cpu().numpy(), obj.cpu().numpy()
        c_o, obj_o = orc.kmeans(Xt, spec.K, iters, init)
        close = np.abs(c_g - c_o).max(1) <= 1e-5
        print("  iters", iters, "centroids equal within 1e-5:", close.mean(), "objective", obj, obj_o, flush=True)
        assert close.mean() >= 0.99
        np.testing.assert_allclose(obj, obj_o, rtol=1e-5)
        assert (np.diff(obj) <= 1e-6 * obj[0]).all()
    again = ivf.ivf_kmeans(Xd, spec.K, 3, dev(init)).cpu().numpy()
    assert (again == c_g).all(), "two runs must give the same bits"


def test_neighbours_match_oracle_with_duplicate_centroids(tiny):
    spec, ix, Q, X = tiny
    print("case: neighbours", flush=True)
    C = ix.centroids.copy()
    C[10:20] = C[5]                                  # eleven identical centroids (ids 5, 10..19)
    for L in (8, 3):
        nbr, cs = ivf.ivf_neighbours(dev(C), L)
        nbr, cs = nbr.cpu().numpy(), cs.cpu().numpy()
        o_nbr, o_cs = orc.neighbours(C, L)
        same = (nbr == o_nbr)
        print("  L", L, "agreement", same.mean(), flush=True)
        assert same.mean() >= 0.999
        # rows of the duplicated centroids: the lowest other ids among the copies, at distance 0
        for r in (5, 10, 19):
            assert (nbr[r] == o_nbr[r]).all() and (cs[r][: min(L, 10)] <= 1e-6).all()
        np.testing.assert_allclose(cs[same], o_cs[same], rtol=1e-4, atol=1e-6)
        assert (np.diff(cs, axis=1) >= 0).all() and (nbr != np.arange(spec.K)[:, None]).all()


def test_learn_alpha_matches_oracle(tiny):
    spec, ix, Q, X = tiny
    print("case: alpha", flush=True)
    n = 20000
    x = X[:n]
    reg, _ = orc.assign(x, ix.centroids)
    a = ivf.ivf_learn_alpha(dev(ix.centroids), dev(ix.nbr), dev(x), dev(reg)).cpu().numpy()
    ref = orc.learn_alpha(x, reg, ix.centroids, ix.nbr)
    np.testing.assert_allclose(a, ref, rtol=0, atol=2e-6)        # pooled value of regions without points included
    assert (np.bincount(reg, minlength=spec.K) == 0).any(), "the case should contain regions without training points"
    b = ivf.ivf_learn_alpha(dev(ix.centroids), dev(ix.nbr), dev(x), dev(reg)).cpu().numpy()
    assert (a == b).all(), "two runs must give the same bits"


def test_pq_train_and_scalar_table_match_oracle(tiny):
    spec, ix, Q, X = tiny
    print("case: pq_train", flush=True)
    n = 30000
    x = X[:n]
    reg, _ = orc.assign(x, ix.centroids)
    sub, mu, res = orc.sub_assign(x, reg, ix.centroids, ix.nbr, ix.alpha)
    E = res.astype(np.float32)
    init = sd.draw_indices(n, 256, "pq-init-test").numpy()
    for iters in (0, 1, 4):
        cb = ivf.ivf_pq_train(dev(E), spec.M, iters, dev(init)).cpu().numpy()
        cb_o, _ = orc.pq_train(E, spec.M, iters, init)
        close = np.abs(cb - cb_o).max(2) <= 1e-6
        print("  iters", iters, "codewords equal within 1e-6:", close.mean(), flush=True)
        assert close.mean() >= (1.0 if iters == 0 else 0.97)
        # as good a codebook: quantisation error of the training rows within 0.1 %
        err = lambda c: float(((E.astype(np.float64) - orc.pq_decode(orc.pq_encode(E.astype(np.float64), c), c)) ** 2).sum())
        if iters:
            assert abs(err(cb) - err(cb_o)) <= 1e-3 * err(cb_o)
    # the 256-level table on the per-point terms
    codes = orc.pq_encode(res, cb_o)
    t = orc.const_term(mu, codes, cb_o).astype(np.float32)
    for iters in (0, 1, 20):
        tab = ivf.ivf_lloyd_1d(dev(t), iters).cpu().numpy()
        tab_o = orc.lloyd_1d(t.astype(np.float64), iters)
        assert (np.diff(tab) >= 0).all()
        print("  table iters", iters, "max abs diff", np.abs(tab - tab_o).max(), flush=True)
        np.testing.assert_allclose(tab, tab_o, rtol=1e-6, atol=1e-7)
    # few values, many equal: levels without values keep their entries
    t2 = np.repeat(np.array([0.5, -1.0, 2.0], np.float32), 40)
    np.testing.assert_allclose(ivf.ivf_lloyd_1d(dev(t2), 5).cpu().numpy(), orc.lloyd_1d(t2.astype(np.float64), 5), rtol=1e-6)


def test_whole_construction_from_the_oracles_start(small):
    """The construction pipeline step by step through the C ABI, from the training sample and the
    initial indices the oracle used for the cached `small` index: the product must be that index up
    to near-ties (k-means amplifies a rounding-level difference in one assignment into slightly
    different centroids, so later arrays are compared where the earlier ones agree)."""
    spec, ix, Q, X = small
    print("case: construction small", flush=True)
    mix = sd.make_mixture(spec.kind, spec.n_mix, spec.D)
    Xt = sd.draw_points(mix, spec.n_train, 0, "train")[0].numpy()
    ci = sd.draw_indices(spec.n_train, spec.K, "kmeans-init").numpy()
    pi = sd.draw_indices(spec.n_train, 256, "pq-init").numpy()
    Xd, Xb = dev(Xt), dev(X)
    cent = ivf.ivf_kmeans(Xd, spec.K, 10, dev(ci))
    c_same = (np.abs(cent.cpu().numpy() - ix.centroids).max(1) <= 1e-5)
    print("  centroids equal:", c_same.mean(), flush=True)
    assert c_same.mean() >= 0.98
    # from here on with the oracle's centroids, so that each later step is compared on equal inputs
    cent = dev(ix.centroids)
    nbr, cs = ivf.ivf_neighbours(cent, spec.L)
    assert (nbr.cpu().numpy() == ix.nbr).mean() >= 0.999
    reg_t = ivf.ivf_coarse_topk(cent, Xd, 1)[0].view(-1).contiguous()
    nbr = dev(ix.nbr)
    alpha = ivf.ivf_learn_alpha(cent, nbr, Xd, reg_t)
    a_same = np.abs(alpha.cpu().numpy() - ix.alpha) <= 1e-5
    print("  alpha equal:", a_same.mean(), flush=True)
    assert a_same.mean() >= 0.99
    desc = ivf.IndexDesc(cent, nbr, dev(ix.alpha), dev(ix.cs_dist2), None, spec.M)
    _, _, _, _, _, res = ivf.ivf_encode(desc, Xd, region_in=reg_t, want_residual=True)
    cb = ivf.ivf_pq_train(res, spec.M, 20, dev(pi))
    cb_same = np.abs(cb.cpu().numpy() - ix.pq_codebook).max(2) <= 1e-5
    print("  codewords equal:", cb_same.mean(), flush=True)
    assert cb_same.mean() >= 0.9
    desc.pq_codebook = dev(ix.pq_codebook)
    _, _, _, _, t = ivf.ivf_encode(desc, Xd, region_in=reg_t, want_t=True)
    tab = ivf.ivf_lloyd_1d(t, 20).cpu().numpy()
    print("  table max diff:", np.abs(tab - ix.const_table).max(), flush=True)
    np.testing.assert_allclose(tab, ix.const_table, rtol=2e-3, atol=2e-5)
    desc.const_table = dev(ix.const_table)
    # encode the base set and group it: the oracle's grouped index, near-ties aside
    r, s_, cd, by, _ = ivf.ivf_encode(desc, Xb)
    bucket = ivf.ivf_bucket_ids(r, s_, spec.L)
    perm, off = ivf.ivf_group(bucket, spec.K * spec.L)
    codes = ivf.ivf_gather_rows(cd, perm).cpu().numpy()
    byte = ivf.ivf_gather_rows(by, perm).cpu().numpy()
    perm, off = perm.cpu().numpy(), off.cpu().numpy().view(np.uint32)
    o_bucket = np.repeat(np.arange(spec.K * spec.L), np.diff(ix.sub_offsets.astype(np.int64)))
    o_bucket_of_id = np.empty(spec.N, np.int64)
    o_bucket_of_id[ix.ids] = o_bucket
    same_bucket = bucket.cpu().numpy() == o_bucket_of_id
    print("  points in the oracle's subregion:", same_bucket.mean(), flush=True)
    assert same_bucket.mean() >= 0.995
    if same_bucket.all():
        assert (perm == ix.ids).all() and (off == ix.sub_offsets).all()
        assert (codes == ix.codes).mean() >= 0.999 and (byte == ix.const_byte).mean() >= 0.99
    # and it searches like the oracle says it should
    d2 = ivf.IndexDesc(cent, nbr, dev(ix.alpha), dev(ix.cs_dist2), dev(ix.pq_codebook), const_table=dev(ix.const_table),
                       sub_offsets=dev(off.view(np.int32)), codes=dev(codes), const_byte=dev(byte), ids=dev(perm))
    ix2 = orc.Index(spec.D, spec.M, spec.L, spec.K, spec.N, ix.centroids, ix.nbr, ix.alpha, ix.cs_dist2, ix.pq_codebook,
                    ix.const_table, off, codes, byte, perm)
    handle = ivf.ivf_load_index(d2)
    out = parity.run_gpu_search(handle, Q[:100], spec.nprobe, spec.prune_frac, spec.k)
    rep = parity.check_search(ix2, Q[:100], spec.nprobe, spec.prune_frac, spec.k, out)
    print(rep, flush=True)
    rep.assert_ok()


@pytest.mark.parametrize("M,ds,n", [(16, 6, 64 * 256 * 16 + 33), (16, 8, 1), (8, 16, 4097), (8, 12, 63), (16, 4, 65), (8, 6, 1000)])
@pytest.mark.parametrize("kind", ["gauss", "grid", "scales"])
def test_codes_are_the_nearest_codewords(M, ds, n, kind):
    """Codes of displacements against fp64 distances.  "grid": small whole numbers, where every distance is exact, so
    that the lowest index of the many exact ties has to come out; else a code may be off the nearest by what the fp32
    chain of differences can round, 2 (ds + 2) u (|x|^2 + |c|^2)."""
    print("case: codes", M, ds, n, kind, flush=True)
    rng = np.random.default_rng(M * ds + n)
    D = M * ds
    x = rng.standard_normal((n, D)).astype(np.float32)
    cb = rng.standard_normal((M, 256, ds)).astype(np.float32)
    if kind == "grid":
        x, cb = np.round(x), np.round(cb)
    if kind == "scales":   # points far smaller and far larger than the codewords, zeros, one block at another scale
        x *= np.exp2(rng.integers(-30, 25, (n, 1))).astype(np.float32)
        x[::5] = 0
        cb[1] *= 1e-20
    z = lambda *s, dt=np.float32: dev(np.zeros(s, dt))
    desc = ivf.IndexDesc(z(2, D), dev(np.array([[1], [0]], np.int32)), z(2), z(2, 1), dev(cb), const_table=dev(np.linspace(-1, 1, 256, dtype=np.float32)))
    _, _, codes, byte, t = ivf.ivf_encode(desc, dev(x), region_in=z(n, dt=np.int32), want_t=True)
    codes, byte, t = codes.cpu().numpy(), byte.cpu().numpy(), t.cpu().numpy()
    take = np.unique(np.linspace(0, n - 1, min(n, 5000)).astype(np.int64))
    xs = x[take].astype(np.float64).reshape(-1, M, ds)
    c64 = cb.astype(np.float64)
    rec = np.zeros((len(take), M, ds))
    for m in range(M):
        d = ((xs[:, m, None] - c64[m][None]) ** 2).sum(-1)
        got = codes[take, m]
        if kind == "grid":
            assert (got == d.argmin(1)).all()
        room = 2 * (ds + 2) * parity.U * ((xs[:, m] ** 2).sum(-1) + (c64[m] ** 2).sum(-1).max())
        assert (d[np.arange(len(take)), got] <= d.min(1) + room).all()
        rec[:, m] = c64[m][got]
    ref = (rec ** 2).sum((1, 2))                                # mu = 0
    assert np.abs(t[take] - ref).max() <= 2 * D * parity.U * ref.max()
    tab = np.linspace(-1, 1, 256, dtype=np.float32)
    assert (byte[take] == np.abs(t[take][:, None] - tab[None]).argmin(1)).all()


@pytest.mark.parametrize("M,ds,n,small", [(8, 6, 256, 0), (16, 6, 8192 + 2049, 0), (3, 8, 20_000, 0), (8, 16, 5000, 0), (5, 12, 3000, 0),
                                          (16, 4, 70_000, 20), (8, 6, 5000, 45), (8, 8, 5000, 100)])
def test_codeword_means_of_one_round(M, ds, n, small):
    """One round from well separated rows: every mean is the fp64 mean rounded once, also where half of the components are
    2^-small of the others (below the exact range of the fixed-point sums the segment sums take over)."""
    print("case: codeword means", M, ds, n, small, flush=True)
    rng = np.random.default_rng(n + small)
    D = M * ds
    code = np.stack([np.concatenate([rng.permutation(256), rng.integers(0, 256, n - 256)]) for _ in range(M)], 1)
    code[:256] = np.arange(256)[:, None]
    centre = rng.permutation(2048)[:256].astype(np.float64)
    E = np.zeros((n, M, ds))
    E[:, :, 0] = centre[code]                              # apart by 1 at least
    E += rng.uniform(-0.1, 0.1, E.shape)
    E[:, :, 1::2] *= 2.0 ** -small
    E = E.astype(np.float32).reshape(n, D)
    got = ivf.ivf_pq_train(dev(E), M, 1, dev(np.arange(256, dtype=np.int64))).cpu().numpy()
    for m in range(M):
        x = E.reshape(n, M, ds)[:, m].astype(np.float64)
        s, a, c = np.zeros((256, ds)), np.zeros((256, ds)), np.bincount(code[:, m], minlength=256)[:, None]
        np.add.at(s, code[:, m], x)
        np.add.at(a, code[:, m], np.abs(x))
        # one rounding to fp32; n additions in fp64 on either side; what the flag lets pass, 2^-29 of the mean
        assert (np.abs(got[m] - s / c) <= (2.0 ** -24 + 2.0 ** -28) * np.abs(s / c) + 2 * n * 2.0 ** -53 * a / c).all()


@pytest.mark.parametrize("M,ds", [(1, 4), (3, 4), (5, 4), (9, 4), (1, 6), (3, 6), (2, 8), (1, 12), (3, 16)])
def test_one_round_of_few_quantisers_with_equal_codewords(M, ds):
    """Fewer quantisers than are loaded together, numbers that leave some over, rows at an address of four bytes, codewords that
    start equal (the lowest index has all points, the others keep their value): whole numbers, every distance exact."""
    print("case: few quantisers", M, ds, flush=True)
    rng = np.random.default_rng(M * 100 + ds)
    n, D = 3000, M * ds
    E = rng.integers(-3, 4, (n, D)).astype(np.float32)
    E[1:256:3] = E[0:255:3]                                   # every third codeword equal to the one before it
    flat = dev(np.concatenate([np.zeros(1, np.float32), E.ravel()]))
    got = ivf.ivf_pq_train(flat[1:].view(n, D), M, 1, dev(np.arange(256, dtype=np.int64))).cpu().numpy()
    for m in range(M):
        x = E[:, m * ds:(m + 1) * ds].astype(np.float64)
        code = ((x[:, None] - x[None, :256]) ** 2).sum(-1).argmin(1)
        s, c = np.zeros((256, ds)), np.bincount(code, minlength=256)[:, None]
        np.add.at(s, code, x)
        want = np.where(c > 0, s / np.maximum(c, 1), x[:256])
        assert (np.abs(got[m] - want) <= 2.0 ** -24 * np.abs(want)).all()   # exact sums, one rounding


@pytest.mark.parametrize("D,L,n,order", [(32, 64, 1000, "sorted"), (64, 5, 1601, "mixed"), (96, 63, 1000, "sorted"), (104, 64, 999, "mixed"),
                                         (128, 17, 65, "sorted"), (96, 1, 4000, "mixed"), (96, 64, 3, "mixed")])
@pytest.mark.parametrize("kind", ["plain", "tight", "flat"])
def test_subregions_and_displacements(D, L, n, order, kind):
    """Subregion of every point against fp64 scores of Eq. (7): the lowest within what fp32 can tell, the lowest index among
    exact ties.  "tight": neighbours that differ by little more than fp16 resolves, where the fp32 scores have to decide;
    "flat": half of the scaling factors are 0, every score of such a region ties.  With codebooks (codes and constants
    follow) and without (displacements only)."""
    print("case: subregions", D, L, n, order, kind, flush=True)
    rng = np.random.default_rng(D + L + n)
    K, M = max(L + 1, 70), 8 if D % 16 else 16
    M = M if D // M in (4, 6, 8, 12, 16) else 8
    C = rng.standard_normal((K, D))
    if kind == "tight":
        C = C[:1] + 2.0 ** -9 * C
    C = C.astype(np.float32)
    reg = rng.integers(0, K, n).astype(np.int32)
    if order == "sorted":
        reg.sort()
    x = (C[reg] + 0.3 * (2.0 ** -9 if kind == "tight" else 1) * rng.standard_normal((n, D))).astype(np.float32)
    nbr = np.stack([rng.permutation(np.delete(np.arange(K), r))[:L] for r in range(K)]).astype(np.int32)
    cs = ((C[:, None].astype(np.float64) - C[nbr]) ** 2).sum(-1).astype(np.float32)
    alpha = rng.uniform(0, 1, K).astype(np.float32)
    if kind == "flat":
        alpha[::2] = 0
    cb = (0.3 * rng.standard_normal((M, 256, D // M))).astype(np.float32)
    d = ivf.IndexDesc(dev(C), dev(nbr), dev(alpha), dev(cs), dev(cb) if D % M == 0 and D // M in (4, 6, 8, 12, 16) else None, M=M)
    _, sub, codes, _, t, res = ivf.ivf_encode(d, dev(x), region_in=dev(reg), want_t=True, want_residual=True)
    d.pq_codebook = None
    _, sub2, _, _, _, res2 = ivf.ivf_encode(d, dev(x), region_in=dev(reg), want_residual=True)
    sub, res = sub.cpu().numpy(), res.cpu().numpy()
    assert (sub == sub2.cpu().numpy()).all() and (res == res2.cpu().numpy()).all()
    x64, c64, a = x.astype(np.float64), C.astype(np.float64), alpha[reg].astype(np.float64)[:, None]
    dxc = ((x64 - c64[reg]) ** 2).sum(-1)[:, None]
    dxs = ((x64[:, None] - c64[nbr[reg]]) ** 2).sum(-1)
    sc = a * dxs + (1 - a) * dxc - a * (1 - a) * cs[reg]
    u = 2.0 ** -24
    room = 2 * (a * (D / 16 + 12) * u * dxs.max(1, keepdims=True) + 8 * u * (dxc + a * dxs.max(1, keepdims=True) + cs[reg].max(1, keepdims=True)))
    got = sc[np.arange(n), sub]
    assert (got <= sc.min(1) + room[:, 0]).all()
    flat = a[:, 0] == 0
    assert (sub[flat] == 0).all()
    s = c64[nbr[reg, sub]]
    mu = c64[reg] + a * (s - c64[reg])
    assert np.abs(res - (x64 - mu)).max() <= 8 * u * (np.abs(x64).max() + np.abs(c64).max())


@pytest.mark.parametrize("D,L,K,n,offset", [(96, 64, 700, 3000, 0.0), (96, 64, 700, 3000, 100.0), (128, 64, 66, 2000, 30.0), (32, 33, 600, 1000, -7.0),
                                            (64, 64, 5000, 6000, 1000.0)])
def test_subregions_of_points_with_an_offset(D, L, K, n, offset):
    """Subregions by 8-bit rows, of unit vectors and of such with an offset that all have in common (the table's centre takes it
    out), with a point and two centroids that are not finite: the lowest fp64 score of Eq. (7) within what fp32 can tell.  The two
    centroids are nobody's region, but neighbours of many, and of the rows from which the centre is formed."""
    print("case: subregions with an offset", D, L, K, n, offset, flush=True)
    rng = np.random.default_rng(D + K)
    C = rng.standard_normal((K, D))
    C = (C / np.linalg.norm(C, axis=1, keepdims=True) + offset).astype(np.float32)
    bad = np.array([0, K // 16])
    reg = np.sort(rng.choice(np.setdiff1d(np.arange(K), bad), n)).astype(np.int32)
    x = (C[reg] + 0.065 * rng.standard_normal((n, D))).astype(np.float32)
    nbr = np.stack([rng.permutation(np.delete(np.arange(K), r))[:L] for r in range(K)]).astype(np.int32)
    cs = ((C[:, None].astype(np.float64) - C[nbr]) ** 2).sum(-1).astype(np.float32)
    alpha = rng.uniform(0.05, 0.17, K).astype(np.float32)
    C[0, 1], C[K // 16, D - 1] = np.nan, np.inf
    lost = np.isin(nbr[reg], bad)
    assert lost.any(1).sum() > n * L // K and not lost.all(1).any()   # (2 n L / K points have one of the two, within a tenth)
    x[n // 2] = np.nan
    d = ivf.IndexDesc(dev(C), dev(nbr), dev(alpha), dev(cs), None, M=8)
    assert n * L >= 10 * K                                     # packed rows
    _, sub, _, _, _, res = ivf.ivf_encode(d, dev(x), region_in=dev(reg), want_residual=True)
    sub = sub.cpu().numpy()
    x64, c64, a = x.astype(np.float64), C.astype(np.float64), alpha[reg].astype(np.float64)[:, None]
    dxc = ((x64 - c64[reg]) ** 2).sum(-1)[:, None]
    dxs = np.where(lost, 0, ((x64[:, None] - c64[nbr[reg]]) ** 2).sum(-1))
    sc = np.where(lost, np.inf, a * dxs + (1 - a) * dxc - a * (1 - a) * cs[reg])
    # encode_kernel's sums: (D / 16 + 12) u of a neighbour's distance, a few u of the score's terms
    u = 2.0 ** -24
    room = 2 * (a * (D / 16 + 12) * u * dxs.max(1, keepdims=True) + 8 * u * (dxc + a * dxs.max(1, keepdims=True) + cs[reg].max(1, keepdims=True)))
    ok = np.arange(n) != n // 2
    got = sc[np.arange(n), sub]
    assert (got <= sc.min(1) + room[:, 0])[ok].all() and 0 <= sub[n // 2] < L


@pytest.mark.parametrize("D,L,kind", [(96, 64, "unit"), (96, 64, "groups"), (128, 64, "groups"), (32, 33, "equal"), (64, 64, "near"), (24, 8, "lost"),
                                      (96, 64, "lost"), (104, 17, "whole")])
@pytest.mark.parametrize("codes", [False, True])
def test_subregions_are_those_of_the_fp32_rows(D, L, kind, codes):
    """A call with points enough for the table of 8-bit rows against calls with fewer, which read the fp32 rows: the same
    subregions, displacements and codes, bit for bit.  Groups of centroids far from the table's middle, neighbours that are equal or nearly
    so, whole numbers with many equal scores, rows and points that are not finite."""
    print("case: subregions against the fp32 rows", D, L, kind, codes, flush=True)
    rng = np.random.default_rng(D + L)
    K, n, M = 640, 5003, 8 if D < 64 else 16
    if D // M not in (4, 6, 8) or D % M:
        M, codes = 8, False
    C = rng.standard_normal((K, D))
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    if kind == "groups":
        m = rng.standard_normal((8, D))
        C += 5 * (m / np.linalg.norm(m, axis=1, keepdims=True))[np.arange(K) % 8]
    if kind == "equal":
        C = C[np.arange(K) // 8]
    if kind == "near":
        C = C[:1] + 2.0 ** -7 * C
    if kind == "whole":
        C = rng.integers(-2, 3, (K, D))
    nbr = np.stack([8 * rng.permutation(K // 8)[:L] + r % 8 if kind == "groups" else rng.permutation(K)[:L] for r in range(K)]).astype(np.int32)
    cs = ((C[:, None] - C[nbr]) ** 2).sum(-1).astype(np.float32)
    alpha = np.full(K, 0.25) if kind == "whole" else rng.uniform(-0.2, 1.2, K)
    reg = rng.integers(0, K, n).astype(np.int32)
    x = C[reg] + (rng.integers(-1, 2, (n, D)) if kind == "whole" else (2.0 ** -7 if kind == "near" else 1) * 0.065 * rng.standard_normal((n, D)))
    C, x = C.astype(np.float32), x.astype(np.float32)
    if kind == "lost":
        C[0, 0], C[40, 1], C[99] = np.nan, np.inf, -np.inf
        x[5], x[17, 3], x[18, D - 1] = np.nan, np.inf, -np.inf
        C[7], x[40] = 3e19, -3e19                               # squares that leave the range of fp32
    cb = (0.05 * rng.standard_normal((M, 256, D // M))).astype(np.float32)
    d = ivf.IndexDesc(dev(C), dev(nbr), dev(alpha.astype(np.float32)), dev(cs), dev(cb) if codes else None, M=M)
    few = (10 * K - 1) // L
    assert n * L >= 10 * K > few * L
    words = lambda a, b: [v if v.dtype != torch.float32 else v.view(torch.int32)
                          for v in ivf.ivf_encode(d, dev(x[a:b]), region_in=dev(reg[a:b]), want_t=codes, want_residual=True) if v is not None]
    got, parts = words(0, n), [words(a, min(n, a + few)) for a in range(0, n, few)]
    for v, *w in zip(got, *parts):
        assert torch.equal(v, torch.cat(w))


@pytest.mark.parametrize("given,codes", [(True, False), (False, False), (False, True)])
def test_no_memory_for_the_packed_table(given, codes):
    """The table of 8-bit rows is given up where it finds no room beside what a call cannot do without; the results stay."""
    from test_gpu_sparse import fill_memory, make
    print("case: encoder, no memory for the packed table", given, codes, flush=True)
    K, D, L, M = 1 << 18, 96, 64, 16
    n = 10 * K // L + 9
    table = K * 128                                           # bytes of the 8-bit rows
    g = torch.Generator(device="cuda").manual_seed(5)
    C = torch.randn(K, D, generator=g, device="cuda")
    nbr = torch.randint(0, K, (K, L), generator=g, device="cuda", dtype=torch.int32)
    cs = torch.rand(K, L, generator=g, device="cuda") * 2 * D
    reg = torch.randint(0, K, (n,), generator=g, device="cuda", dtype=torch.int32)
    x = C[reg.long()] + 0.3 * torch.randn(n, D, generator=g, device="cuda")
    d = ivf.IndexDesc(C, nbr, torch.rand(K, generator=g, device="cuda"), cs, 0.3 * torch.randn(M, 256, D // M, generator=g, device="cuda") if codes else None, M=M,
                      const_table=torch.linspace(-100, 100, 256, device="cuda") if codes else None)
    give_back = lambda: ivf.ivf_free_index(make(1000, 32, 8, 8, 1, 1.0, 0.0)[0])   # what the library keeps for index-time calls
    call = lambda: [v for v in ivf.ivf_encode(d, x, region_in=reg if given else None) if v is not None]
    give_back()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    ref = call()
    need = free - torch.cuda.mem_get_info()[0]
    assert need >= table
    give_back()
    held = fill_memory(need - table // 2)
    try:
        got = call()
    finally:
        del held
        torch.cuda.empty_cache()
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


@pytest.mark.parametrize("n,D,K,iters,kind", [(20_000, 96, 700, 5, "groups"), (20_000, 96, 700, 4, "tight"), (6000, 160, 300, 4, "lost"), (1500, 64, 1500, 3, "plain"),
                                              ((1 << 20) + 3001, 8, 63, 3, "lost")])
def test_rounds_that_start_from_the_round_before(n, D, K, iters, kind):
    """Rounds of k-means, whose bounds start from the last round's nearest centroids and which leave a row's only candidate
    undecided, against the nearest centroids with their distances and the means, called one after the other: the same centroids, bit
    for bit.  Both sweeps (D = 160: wide rows), several chunks of rows, rows with many candidates ("tight"), rows that are not finite and have
    no centroid, centroids that start equal."""
    print("case: k-means from bounds", n, D, K, iters, kind, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + D)
    m = torch.randn(K, D, generator=g, device="cuda")
    if kind == "tight":
        m = m[:1] + 2.0 ** -9 * m
    x = m[torch.randint(0, K, (n,), generator=g, device="cuda")] + (2.0 ** -10 if kind == "tight" else 0.7) * torch.randn(n, D, generator=g, device="cuda")
    init = torch.randperm(n, generator=g, device="cuda")[:K].contiguous()
    if kind == "lost":
        rows = torch.tensor([0, 77, n // 2, n - 1], device="cuda")
        rows = rows[~torch.isin(rows, init)]
        x[rows[:2], 1], x[rows[2:], D - 1] = float("nan"), float("inf")
    elif kind != "tight":
        x[init[1]] = x[init[0]]
    c = x[init].contiguous()
    for _ in range(iters):
        near, d = ivf.ivf_coarse_topk(c, x, 1)
        c = ivf.ivf_cluster_means(x, near[:, 0].contiguous(), c.clone())
    before = ivf.ivf_assign_stats()
    plain = ivf.ivf_kmeans(x, K, iters, init)
    after = ivf.ivf_assign_stats()
    if kind != "tight":                                        # (whose lists may overflow)
        assert after[0] - before[0] == iters * (2 if n > 1 << 20 else 1) and after[1] == before[1]
    with_sums, _ = ivf.ivf_kmeans(x, K, iters, init, want_objective=True)
    assert torch.isfinite(c).all()
    assert torch.equal(plain, c) and torch.equal(with_sums, c)


@pytest.mark.parametrize("n,D,K", [(1, 1, 1), (2560, 64, 10), (2561, 64, 10), (5000, 65, 700), (999, 130, 1500), (300, 1024, 40), (4097, 96, 3)])
def test_cluster_means_of_short_and_long_clusters(n, D, K):
    """Both kernels and the line between them (256 rows a cluster on average), clusters of none, one and many rows, columns
    past a wavefront's 64: the fp64 mean rounded once."""
    print("case: cluster means", n, D, K, flush=True)
    rng = np.random.default_rng(n + D)
    x = (rng.standard_normal((n, D)) * 10 + 3).astype(np.float32)
    lab = (rng.random(n) ** 3 * K).astype(np.int32)
    c0 = rng.standard_normal((K, D)).astype(np.float32)
    got = ivf.ivf_cluster_means(dev(x), dev(lab), dev(c0)).cpu().numpy()
    s, a = np.zeros((K, D)), np.zeros((K, D))
    np.add.at(s, lab, x.astype(np.float64))
    np.add.at(a, lab, np.abs(x).astype(np.float64))
    cnt = np.bincount(lab, minlength=K)[:, None]
    ref = s / np.maximum(cnt, 1)
    assert (got[cnt[:, 0] == 0] == c0[cnt[:, 0] == 0]).all()
    full = cnt[:, 0] > 0
    assert (np.abs(got - ref)[full] <= (2.0 ** -24 * np.abs(ref) + 2 * n * 2.0 ** -53 * a / np.maximum(cnt, 1))[full]).all()


@pytest.mark.parametrize("a", [-0.5, -0.01, 1.5, 4.0, 1e4, -1e4])
@pytest.mark.parametrize("D,L,n", [(96, 64, 1000), (128, 7, 333)])
def test_subregions_with_scaling_factors_outside_0_1(D, L, n, a):
    """The scaling factor of a region may be any number: subregions against fp64 scores of Eq. (7), within what the fp32
    score rounds, its terms being |a| |x - s|^2, |1 - a| |x - c|^2 and |a (1 - a)| |c - s|^2."""
    print("case: subregions, scaling factor", D, L, n, a, flush=True)
    rng = np.random.default_rng(D + L)
    K = 80
    C = rng.standard_normal((K, D))
    C = (C / np.linalg.norm(C, axis=1, keepdims=True)).astype(np.float32)
    reg = rng.integers(0, K, n).astype(np.int32)
    x = (C[reg] + 0.05 * rng.standard_normal((n, D))).astype(np.float32)
    nbr = np.stack([rng.permutation(np.delete(np.arange(K), r))[:L] for r in range(K)]).astype(np.int32)
    cs = ((C[:, None].astype(np.float64) - C[nbr]) ** 2).sum(-1).astype(np.float32)
    alpha = np.full(K, a, np.float32)
    alpha[::7] = 0.1
    d = ivf.IndexDesc(dev(C), dev(nbr), dev(alpha), dev(cs), None, M=8)
    _, sub, _, _, _, res = ivf.ivf_encode(d, dev(x), region_in=dev(reg), want_residual=True)
    sub, res = sub.cpu().numpy(), res.cpu().numpy()
    x64, c64, al = x.astype(np.float64), C.astype(np.float64), alpha[reg].astype(np.float64)[:, None]
    dxc = ((x64 - c64[reg]) ** 2).sum(-1)[:, None]
    dxs = ((x64[:, None] - c64[nbr[reg]]) ** 2).sum(-1)
    sc = al * dxs + (1 - al) * dxc - al * (1 - al) * cs[reg]
    u = 2.0 ** -24
    terms = np.abs(al) * dxs.max(1, keepdims=True) + np.abs(1 - al) * dxc + np.abs(al * (1 - al)) * cs[reg].max(1, keepdims=True)
    room = 2 * (np.abs(al) * (D / 16 + 12) * u * dxs.max(1, keepdims=True) + 8 * u * terms)
    assert (sc[np.arange(n), sub] <= sc.min(1) + room[:, 0]).all()
    clear = np.sort(sc, 1)[:, 1] - sc.min(1) > 2 * room[:, 0]
    assert (sub[clear] == sc.argmin(1)[clear]).all()
    s = c64[nbr[reg, sub]]
    mu = c64[reg] + al * (s - c64[reg])
    assert (np.abs(res - (x64 - mu)) <= 8 * u * (np.abs(x64) + np.abs(mu) + (1 + np.abs(al)) * (np.abs(s) + np.abs(c64[reg])))).all()


@pytest.mark.parametrize("M,ds,n", [(8, 4, 256 * 3), (16, 8, 70_001)])
def test_codeword_means_keep_every_bit_of_an_fp64_sum(M, ds, n):
    """Two rows a codeword, a component of them a + b with b a little above half a unit in the last place of a and nearly all
    of its bits far below 2^-49 of the matrix's largest magnitude: the mean is the exact one rounded once, which goes up."""
    print("case: codeword means, last bits", M, ds, n, flush=True)
    rng = np.random.default_rng(n)
    E = np.zeros((n, M, ds))
    code = rng.permutation(np.arange(n) % 255)
    first, second = np.full(255, -1), np.full(255, -1)
    for i, j in enumerate(code):                            # (the rows beyond two a codeword are left out)
        if first[j] < 0: first[j] = i
        elif second[j] < 0: second[j] = i
    E[:, :, 0] = (code[:, None] + 1) / 256.0
    k = rng.integers(0, 1 << 21, (255, M)) * 2              # an even last place: a tie would go down
    E[:, :, 2:] = 2.0 ** -10
    E[first, :, 1] = 2.0 ** -19 * (1 + k * 2.0 ** -23)
    E[second, :, 1] = 2.0 ** -43 * (1 + rng.integers(1, 1 << 9, k.shape) * 2.0 ** -20)
    keep = (np.arange(n) == first[code]) | (np.arange(n) == second[code])
    E = E[keep]                                             # two rows of each codeword ...
    E = np.concatenate([E, np.full((2, M, ds), 1.0)])       # ... and the largest magnitude, 1, a codeword of its own
    order = rng.permutation(len(E))
    E, code = E[order], np.concatenate([code[keep], [255, 255]])[order]
    start = np.array([np.flatnonzero(code == j)[0] for j in range(256)])
    E32 = E.astype(np.float32)
    assert (E32.astype(np.float64) == E).all()
    reps = max(1, n // len(E))
    E32, code = np.tile(E32.reshape(len(E), M * ds), (reps, 1)), np.tile(code, reps)
    got = ivf.ivf_pq_train(dev(E32), M, 1, dev(start.astype(np.int64))).cpu().numpy()
    s = np.zeros((256, M, ds))
    np.add.at(s, code, E32.reshape(-1, M, ds).astype(np.float64))      # exact: multiples of 2^-63, sums below 2^-10 but for component 0
    ref = (s / np.bincount(code, minlength=256)[:, None, None]).astype(np.float32)
    assert (got[:, :, 1] == ref.transpose(1, 0, 2)[:, :, 1]).all()
    assert np.abs(got - ref.transpose(1, 0, 2)).max() <= 2.0 ** -24


@pytest.mark.parametrize("n,D,K,crowd", [(9000, 96, 300, [512, 513, 640, 641]), (40_000, 130, 5000, [20_000]), (3000, 64, 3, [2487, 513]),
                                         (5000, 20, 2, [5000])])
def test_cluster_means_where_a_cluster_is_crowded(n, D, K, crowd):
    """Clusters on both sides of the length from which a workgroup takes them, beside short and empty ones: the fp64 mean
    rounded once, n additions in fp64 on either side."""
    print("case: crowded clusters", n, D, K, crowd, flush=True)
    rng = np.random.default_rng(n + D)
    x = (rng.standard_normal((n, D)) * 10 + 3).astype(np.float32)
    lab = np.concatenate([np.full(c, i) for i, c in enumerate(crowd)] + [rng.integers(len(crowd), K, n - sum(crowd)) if n > sum(crowd) else np.empty(0, int)])
    lab = rng.permutation(lab).astype(np.int32)
    c0 = rng.standard_normal((K, D)).astype(np.float32)
    got = ivf.ivf_cluster_means(dev(x), dev(lab), dev(c0)).cpu().numpy()
    s, a = np.zeros((K, D)), np.zeros((K, D))
    np.add.at(s, lab, x.astype(np.float64))
    np.add.at(a, lab, np.abs(x).astype(np.float64))
    cnt = np.bincount(lab, minlength=K)[:, None]
    assert (got[cnt[:, 0] == 0] == c0[cnt[:, 0] == 0]).all()
    full = cnt[:, 0] > 0
    ref = s / np.maximum(cnt, 1)
    assert (np.abs(got - ref)[full] <= (2.0 ** -24 * np.abs(ref) + 2 * n * 2.0 ** -53 * a / np.maximum(cnt, 1))[full]).all()
    assert (got == ivf.ivf_cluster_means(dev(x), dev(lab), dev(c0)).cpu().numpy()).all()


@pytest.mark.parametrize("M,ds,n", [(16, 6, 5000), (16, 8, 333), (8, 16, 1000), (8, 12, 64), (16, 4, 5000)])
@pytest.mark.parametrize("kinds", [1, 3, 40, 200])
def test_codes_where_codewords_are_equal(M, ds, n, kinds):
    """Codebooks of few distinct codewords (one block of each quantiser with -0 for 0, one with a codeword of its own behind its
    copies): the first of the nearest ones."""
    print("case: equal codewords", M, ds, n, kinds, flush=True)
    rng = np.random.default_rng(M * ds + n + kinds)
    D = M * ds
    base = rng.integers(-20, 21, (M, kinds, ds)).astype(np.float32)
    cb = np.stack([base[m][rng.integers(0, kinds, 256)] for m in range(M)])
    cb[:, 255] = 50.0 + np.arange(M)[:, None]
    cb[:, 100:120] = np.where(cb[:, 100:120] == 0, -0.0, cb[:, 100:120])
    x = rng.integers(-25, 60, (n, D)).astype(np.float32)
    x[::3] = cb[:, rng.integers(0, 256, len(x[::3]))].transpose(1, 0, 2).reshape(-1, D)
    z = lambda *s, dt=np.float32: dev(np.zeros(s, dt))
    desc = ivf.IndexDesc(z(2, D), dev(np.array([[1], [0]], np.int32)), z(2), z(2, 1), dev(cb), const_table=dev(np.linspace(-1, 1, 256, dtype=np.float32)))
    codes = ivf.ivf_encode(desc, dev(x), region_in=z(n, dt=np.int32))[2].cpu().numpy()
    for m in range(M):                                      # whole numbers: exact
        d = ((x.reshape(n, M, ds)[:, m, None].astype(np.int64) - cb[m][None].astype(np.int64)) ** 2).sum(-1)
        assert (codes[:, m] == d.argmin(1)).all()
