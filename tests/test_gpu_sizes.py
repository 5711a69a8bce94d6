"""Parity at sizes that span many kernel tiles with ragged tails, on the SIFT-like data,
and at the full benchmark sizes on sampled queries (needs an MI355X)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import synthdata as sd
import paper_1802_02422_amd as ivf
from paper_1802_02422_amd import index_builder
from oracle import ivf_oracle as orc
import parity
from bench import download_index


def run_and_check(ix, Q, spec, sample=None, nprobe=None, tau=None, k=None, max_near_frac=0.05):
    nprobe, tau, k = nprobe or spec.nprobe, tau or spec.prune_frac, k or spec.k
    handle = ivf.ivf_load_index(parity.to_device(ix))
    out = parity.run_gpu_search(handle, Q, nprobe, tau, k)
    ivf.ivf_free_index(handle)
    if sample is not None:
        out = {n: v[sample] for n, v in out.items()}
        Q = Q[sample]
    rep = parity.check_search(ix, Q, nprobe, tau, k, out)
    print(rep, flush=True)
    rep.assert_ok(max_near_frac=max_near_frac)
    return rep


def test_small_deep_many_tiles(small):
    spec, ix, Q, X = small          # K = 2000 (not a multiple of 128), nq = 333, M = 16, L = 24
    print("case: small", spec, flush=True)
    run_and_check(ix, Q, spec)
    run_and_check(ix, Q[:130], spec, nprobe=7, tau=1.0, k=1)
    run_and_check(ix, Q[:9], spec, nprobe=300, tau=0.05, k=300)
    # nprobe * L > 4096: scoring by 1024 threads from the whole row of distances; rows of probe ids that do not start on
    # cache-line boundaries (190 x 4 bytes), a whole batch and a handful of queries
    run_and_check(ix, Q, spec, nprobe=190, tau=0.3, k=50)
    run_and_check(ix, Q[:5], spec, nprobe=190, tau=0.3, k=50)
    run_and_check(ix, Q[:70], spec, nprobe=256, tau=0.1, k=10)


def test_small_sift_like(small_sift):
    spec, ix, Q, X = small_sift     # D = 128, uint8-valued components, K = 1000
    print("case: small_sift", spec, flush=True)
    run_and_check(ix, Q, spec)


def test_k_not_multiple_of_four_and_tiny_lists():
    """K = 509: scalar store path of the distance tile, partial last block of 64, L close to K."""
    mix = sd.make_mixture("deep", 100, 32)
    X = sd.draw_points(mix, 6000, 0, "odd-base")[0].numpy()
    Xt = sd.draw_points(mix, 4000, 0, "odd-train")[0].numpy()
    Q = sd.draw_queries(mix, 70, "odd-query").numpy()
    ix = orc.build_index(Xt, X, 509, 5, 8, sd.draw_indices(4000, 509, "odd-k").numpy(),
                         sd.draw_indices(4000, 256, "odd-pq").numpy(), kmeans_iters=3, pq_iters=3)
    spec = sd.WorkloadSpec("odd", "deep", 6000, 32, 100, 509, 5, 8, 70, 33, 0.4, 20, 4000)
    print("case: odd K", flush=True)
    run_and_check(ix, Q, spec, max_near_frac=0.1)
    run_and_check(ix, Q, spec, nprobe=509, tau=1.0, k=64, max_near_frac=0.1)     # exhaustive


def test_long_lists_duplicates_and_empty_regions():
    """Few regions (lists of thousands of records, many chunks per descriptor), exact duplicate
    points (exact distance ties) and regions that stay empty."""
    mix = sd.make_mixture("deep", 6, 32, name="degenerate")
    X = sd.draw_points(mix, 30000, 0, "deg-base")[0].numpy()
    X[5000:7000] = X[4999]                      # 2001 identical points
    X[20000:20300] = X[123]
    Xt = sd.draw_points(mix, 5000, 0, "deg-train")[0].numpy()
    Q = sd.draw_queries(mix, 40, "deg-query").numpy()
    Q[0] = X[4999]
    Q[1] = X[123]
    ix = orc.build_index(Xt, X, 12, 3, 16, sd.draw_indices(5000, 12, "deg-k").numpy(),
                         sd.draw_indices(5000, 256, "deg-pq").numpy(), kmeans_iters=3, pq_iters=3)
    sizes = np.diff(ix.sub_offsets.astype(np.int64))
    print("case: degenerate; list sizes", sizes.tolist(), flush=True)
    assert sizes.max() > 2000
    spec = sd.WorkloadSpec("deg", "deep", 30000, 32, 6, 12, 3, 16, 40, 5, 0.5, 50, 5000)
    run_and_check(ix, Q, spec, max_near_frac=1.0)
    run_and_check(ix, Q, spec, nprobe=12, tau=1.0, k=1024, max_near_frac=1.0)
    run_and_check(ix, Q[:3], spec, nprobe=1, tau=0.3, k=7, max_near_frac=1.0)


def check_stored_points_against_oracle_encoder(spec, mix, mode, desc, ix, n_check=2048):
    """A sample of the points of the first generated chunk, encoded by the oracle from the raw
    vectors (region given where the builder was given it), against what the device-built index
    stores for them: subregion, PQ code and constant byte, near-ties of the oracle's fp64
    decisions aside."""
    n0 = min(10_000_000, spec.N)
    X, lab = sd.draw_points(mix, n0, 0, "base", sorted_labels=(mode == "mixture"))
    pick = torch.from_numpy(np.random.default_rng(7).choice(n0, n_check, replace=False)).to(X.device)
    x = X[pick].cpu().numpy()
    region = lab[pick].int().cpu().numpy() if mode == "mixture" else None
    del X, lab
    inv = torch.empty(spec.N, dtype=torch.int32, device=desc.ids.device)
    inv[desc.ids.long()] = torch.arange(spec.N, dtype=torch.int32, device=desc.ids.device)
    pos = inv[pick].long().cpu().numpy()
    del inv
    enc = orc.encode(x, ix.centroids, ix.nbr, ix.alpha, ix.pq_codebook, ix.const_table, region=region)
    off = ix.sub_offsets.astype(np.int64)
    b = enc.region.astype(np.int64) * spec.L + enc.sub
    inside = (off[b] <= pos) & (pos < off[b + 1])
    codes_same = inside & (ix.codes[pos] == enc.codes).all(1)
    byte_same = codes_same & (ix.const_byte[pos] == enc.const_byte)
    print(f"  stored vs oracle encoder on {n_check} points: subregion {inside.mean():.4f}, "
          f"code {codes_same.mean():.4f}, byte {byte_same.mean():.4f}", flush=True)
    assert inside.mean() >= 0.995 and codes_same.mean() >= 0.99 and byte_same.mean() >= 0.98
    # every point the oracle places elsewhere is a near-tie of its own fp64 choice
    c64 = ix.centroids.astype(np.float64)
    stored_bucket = np.searchsorted(off, pos, side="right") - 1
    for i in np.flatnonzero(~inside):
        r_st, l_st = divmod(int(stored_bucket[i]), spec.L)
        def sub_dist(r, l):
            mu = c64[r] + float(ix.alpha[r]) * (c64[ix.nbr[r, l]] - c64[r])
            return float(((x[i].astype(np.float64) - mu) ** 2).sum())
        d_st, d_or = sub_dist(r_st, l_st), sub_dist(int(enc.region[i]), int(enc.sub[i]))
        assert abs(d_st - d_or) <= 1e-5 * max(d_or, 1.0), (i, d_st, d_or)


def full_size_case(name, n_sample, extra_batches=(), budget=0, n_budget=32):
    spec = sd.WORKLOADS[name]
    dev = torch.device("cuda:0")
    mix = sd.make_mixture(spec.kind, spec.n_mix, spec.D, dev)
    mode = "mixture" if spec.K >= (1 << 18) else "kmeans"
    desc, stats = index_builder.build(spec, mix, mode=mode)
    print("built", name, stats, flush=True)
    Q = sd.draw_queries(mix, spec.nq).contiguous()
    ix = download_index(desc, spec)
    check_stored_points_against_oracle_encoder(spec, mix, mode, desc, ix)
    handle = ivf.ivf_load_index(desc)
    desc.codes = desc.const_byte = desc.ids = None
    torch.cuda.empty_cache()
    ivf.ivf_set_scratch_limit(handle, 48 << 30)              # the launch configuration bench.py times
    out = ivf.ivf_search_stages(handle, Q, spec.nprobe, spec.prune_frac, spec.k)
    torch.cuda.synchronize()
    # every query, not only the sampled ones: a second run of the whole batch returns the same bits
    # (the kernels' hand-counted waits on asynchronous copies would show up here as run-to-run noise)
    again = ivf.ivf_search_stages(handle, Q, spec.nprobe, spec.prune_frac, spec.k)
    torch.cuda.synchronize()
    for n in ("probe_id", "probe_d", "kept_sub", "ids", "dists"):
        assert torch.equal(out[n], again[n]), (name, n)
    del again
    sample = np.linspace(0, spec.nq - 1, n_sample).astype(np.int64)
    out = {n: v[torch.from_numpy(sample).to(dev)].cpu().numpy() for n, v in out.items()}
    rep = parity.check_search(ix, Q.cpu().numpy()[sample], spec.nprobe, spec.prune_frac, spec.k, out)
    print(name, rep, flush=True)
    rep.assert_ok(max_near_frac=0.1)
    if budget:                                               # the candidate-budget entry point at full size
        sq = torch.from_numpy(sample[:n_budget]).to(dev)
        Qs = Q[sq].contiguous()
        so = ivf.ivf_search_stages(handle, Qs, spec.nprobe, spec.prune_frac, spec.k)
        bo = ivf.ivf_search_budget(handle, Qs, spec.nprobe, spec.prune_frac, budget, spec.k)
        torch.cuda.synchronize()
        so = {n: v.cpu().numpy() for n, v in so.items()}
        bo = {n: v.cpu().numpy() for n, v in bo.items()}
        rep = parity.check_search_budget(ix, Qs.cpu().numpy(), spec.nprobe, spec.prune_frac, budget, spec.k, so, bo)
        print(name, "budget", budget, rep, flush=True)
        rep.assert_ok(max_near_frac=0.1)
        assert (bo["n_scanned"] >= np.minimum(budget, so["n_scanned"])).all()
    for nb in extra_batches:                                 # other batch sizes of the same workload
        o2 = ivf.ivf_search_stages(handle, Q[:nb].contiguous(), spec.nprobe, spec.prune_frac, spec.k)
        torch.cuda.synchronize()
        o2 = {n: v.cpu().numpy() for n, v in o2.items()}
        rep = parity.check_search(ix, Q[:nb].cpu().numpy(), spec.nprobe, spec.prune_frac, spec.k, o2)
        print(name, "batch", nb, rep, flush=True)
        rep.assert_ok(max_near_frac=0.1)
    ivf.ivf_free_index(handle)


def test_full_size_deep10m_sampled_queries():
    print("case: deep10m full size", flush=True)
    full_size_case("deep10m", 128, budget=1000)


def test_full_size_sift10m_sampled_queries():
    print("case: sift10m full size", flush=True)
    full_size_case("sift10m", 128)


def test_full_size_deep100m_latency_batches():
    print("case: deep100m full size, nq = 64 and nq = 1", flush=True)
    full_size_case("deep100m", 64, extra_batches=(1,))


def test_full_size_deep1b_sampled_queries():
    print("case: deep1b full size", flush=True)
    full_size_case("deep1b", 256, budget=30000)


@pytest.mark.parametrize("mode", ["zero", "one", "mixed"])
def test_degenerate_scaling_factors(tiny, mode):
    """alpha = 0 puts every subcentroid of a region on its centroid (all L scores of a region tie
    exactly and all points fall into subregion 0: the variant without grouping), alpha = 1 puts
    them on the neighbouring centroids; 'mixed' alternates 0, 1 and 1/2 between regions."""
    spec, ix, Q, X = tiny
    K, N = spec.K, spec.N
    r3 = np.arange(K) % 3
    alpha = {"zero": np.zeros(K), "one": np.ones(K),
             "mixed": np.where(r3 == 0, 0.0, np.where(r3 == 1, 1.0, 0.5))}[mode].astype(np.float32)
    enc = orc.encode(X, ix.centroids, ix.nbr, alpha, ix.pq_codebook, ix.const_table)
    perm, off = orc.group(enc.region, enc.sub, spec.L, K)
    ix2 = orc.Index(spec.D, spec.M, spec.L, K, N, ix.centroids, ix.nbr, alpha, ix.cs_dist2, ix.pq_codebook,
                    ix.const_table, off, np.ascontiguousarray(enc.codes[perm]),
                    np.ascontiguousarray(enc.const_byte[perm]), np.arange(N, dtype=np.int32)[perm].copy())
    if mode == "zero":
        assert (enc.sub == 0).all()
    print("case: degenerate alpha", mode, flush=True)
    run_and_check(ix2, Q, spec, max_near_frac=0.1)
    run_and_check(ix2, Q, spec, nprobe=spec.K, tau=1.0, k=50, max_near_frac=0.1)
    # the library's encoder on the same trained index
    n = 4000
    desc = parity.to_device(ix2, with_codes=False)
    region, sub, codes, byte, _ = ivf.ivf_encode(desc, torch.from_numpy(X[:n]).cuda())
    region, sub, codes = region.cpu().numpy(), sub.cpu().numpy(), codes.cpu().numpy()
    same = (region == enc.region[:n]) & (sub == enc.sub[:n])
    assert same.mean() >= 0.99, same.mean()
    assert (codes[same] == enc.codes[:n][same]).mean() >= 0.999
    if mode == "zero":
        assert (sub == 0).all()


@pytest.mark.parametrize("nq,K,D", [(129, 128 * 1025, 96), (65, 128 * 2049, 100), (1100, 128 * 228, 128), (700, 128 * 340, 96), (70, 4224, 96), (200, 1000, 64)])
def test_distance_gemm_over_few_query_tiles(nq, K, D):
    """Few query tiles: the swept kernel in sweeps of 8 to 64 tiles whose last group is partial, and one tile a workgroup
    below its threshold.  The three nearest centroids against fp64: ids where fp32 can tell, distances within the bound
    that stage 1 is held to, 16 u (|q|^2 + max |c|^2)."""
    print("case: few query tiles", nq, K, D, flush=True)
    g = torch.Generator(device="cuda").manual_seed(nq)
    C = torch.randn(K, D, generator=g, device="cuda")
    Q = torch.randn(nq, D, generator=g, device="cuda")
    ids, d = ivf.ivf_coarse_topk(C, Q, 3)
    c64, q64 = C.double(), Q.double()
    cn, qn = (c64 * c64).sum(1), (q64 * q64).sum(1)
    tol = 16 * 2.0 ** -24 * (qn + cn.max())
    for a in range(0, nq, 64):
        full = (cn[None] - 2 * q64[a:a + 64] @ c64.t() + qn[a:a + 64, None])
        ref, at = full.topk(4, dim=1, largest=False)
        got = torch.gather(full, 1, ids[a:a + 64].long())
        t = tol[a:a + 64, None]
        assert ((d[a:a + 64].double() - got).abs() <= t).all()
        assert (got.sort(1)[0] <= ref[:, :3] + 2 * t).all()
        clear = ref[:, 3] - ref[:, 2] > 2 * t[:, 0]
        assert (ids[a:a + 64][clear].long() == at[clear, :3].sort(1)[0]).all()


@pytest.mark.parametrize("nq,K,P", [(1, 1, 1), (5, 63, 63), (7, 64, 16), (300, 1024, 16), (3, 2048, 256), (66, 2000, 1500), (130, 2049, 33),
                                    (70, 65536, 64), (5, 65473, 1), (9, 20000, 256), (33, 30000, 64)])
@pytest.mark.parametrize("kind", ["plain", "ties"])
def test_selection_of_the_nearest_by_distance_and_id(nq, K, P, kind):
    """Whole-number vectors, so that every distance is exact: the P nearest by (distance, id), whatever the kernel, also
    where thousands of centroids tie with the P-th (more than a wavefront's survivors, all of them equal)."""
    print("case: selection", nq, K, P, kind, flush=True)
    rng = np.random.default_rng(nq + K + P)
    C = rng.integers(-9, 10, (K, 32)).astype(np.float32)
    if kind == "ties":
        C[rng.random(K) < 0.7] = C[0]
    Q = rng.integers(-9, 10, (nq, 32)).astype(np.float32)
    Q[0] = C[0]
    if P == 1 and K > 1:                                             # (P = 1 is the assignment: another kernel)
        P = 2
    ids, d = ivf.ivf_coarse_topk(torch.from_numpy(C).cuda(), torch.from_numpy(Q).cuda(), P)
    ids, d = ids.cpu().numpy(), d.cpu().numpy()
    full = ((Q[:, None, :].astype(np.int64) - C[None].astype(np.int64)) ** 2).sum(-1) if nq * K < 3e6 else None
    for q in range(nq):
        row = full[q] if full is not None else ((Q[q].astype(np.int64) - C.astype(np.int64)) ** 2).sum(-1)
        ref = np.sort(np.lexsort((np.arange(K), row))[:P])
        assert (ids[q] == ref).all(), q
        assert (d[q] == row[ref]).all()


@pytest.mark.parametrize("K,L,nprobe,nq", [(512, 31, 20, 40), (8192, 16, 40, 33), (9001, 40, 70, 9), (12000, 64, 64, 17), (16385, 64, 100, 5), (3000, 63, 250, 70)])
def test_scoring_from_whole_rows(K, L, nprobe, nq):
    """Scoring that reads the whole row of distances through LDS: one and several parts, partial and unaligned last ones,
    both workgroup sizes."""
    print("case: scoring from rows", K, L, nprobe, nq, flush=True)
    rng = np.random.default_rng(K + L)
    D, M, N = 32, 8, 20000
    X = rng.standard_normal((N, D)).astype(np.float32)
    Xt = rng.standard_normal((max(K, 4000), D)).astype(np.float32)
    ix = orc.build_index(Xt, X, K, L, M, np.arange(K), np.arange(256), kmeans_iters=0, pq_iters=1)
    h = ivf.ivf_load_index(parity.to_device(ix))
    Q = rng.standard_normal((nq, D)).astype(np.float32)
    out = parity.run_gpu_search(h, Q, nprobe, 0.3, 20)
    parity.check_search(ix, Q, nprobe, 0.3, 20, out).assert_ok()


@pytest.mark.parametrize("nq,K,P", [(1024, 4096, 64), (1031, 4161, 64), (1023, 4096, 64), (960, 20000, 40), (1025, 65536, 64), (5, 4096, 16),
                                    (384, 2049, 16), (49, 8192, 2)])
@pytest.mark.parametrize("kind", ["line", "pairs", "ties"])
def test_selection_where_near_centroids_have_near_ids(nq, K, P, kind):
    """Numbers that follow the places: a block of 64 centroids is near or far as a whole, so that thousands of distances lie
    at or below the P-th smallest block minimum ("pairs": and most of them tie with another).  Whole numbers: exact."""
    print("case: selection, sorted centroids", nq, K, P, kind, flush=True)
    rng = np.random.default_rng(nq + K + P)
    C = rng.integers(-2, 3, (K, 32)).astype(np.float32)
    C[:, 0] = np.arange(K) // (2048 if kind == "pairs" else 64)
    if kind == "pairs":
        C[1::2] = C[0:-1:2][:len(C[1::2])]
    if kind == "ties":
        C[rng.random(K) < 0.7] = C[K // 2]
    Q = np.concatenate([C[rng.integers(0, K, nq, dtype=np.int64)][:, :1], rng.integers(-2, 3, (nq, 31))], 1).astype(np.float32)
    ids, d = ivf.ivf_coarse_topk(torch.from_numpy(C).cuda(), torch.from_numpy(Q).cuda(), P)
    ids, d = ids.cpu().numpy(), d.cpu().numpy()
    c64 = C.astype(np.float64)
    for a in range(0, nq, 128):
        q64 = Q[a:a + 128].astype(np.float64)
        full = ((q64 ** 2).sum(1)[:, None] + (c64 ** 2).sum(1)[None] - 2 * q64 @ c64.T).astype(np.int64) * K + np.arange(K)
        ref = np.sort(np.partition(full, P - 1, axis=1)[:, :P] % K, axis=1)
        assert (ids[a:a + 128] == ref).all()
        assert (d[a:a + 128] == np.take_along_axis(full, ref, 1) // K).all()


def _random_index(K, L, D, M, N, seed):
    """An index of random parts (neighbours included): what the query path does with it does not depend on how it was made."""
    rng = np.random.default_rng(seed)
    C = rng.standard_normal((K, D)).astype(np.float32)
    nbr = ((np.arange(K)[:, None] + 1 + rng.integers(0, K - 1, (K, L))) % K).astype(np.int32)
    cs = np.concatenate([((C[a:a + 4096, None] - C[nbr[a:a + 4096]]) ** 2).sum(-1) for a in range(0, K, 4096)]).astype(np.float32)
    sizes = rng.multinomial(N, np.full(K * L, 1.0 / (K * L)))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)
    return orc.Index(D, M, L, K, N, C, nbr, rng.uniform(0.05, 0.2, K).astype(np.float32), cs,
                     (0.3 * rng.standard_normal((M, 256, D // M))).astype(np.float32), np.sort(rng.standard_normal(256)).astype(np.float32),
                     off, rng.integers(0, 256, (N, M)).astype(np.uint8), rng.integers(0, 256, N).astype(np.uint8),
                     rng.permutation(N).astype(np.int32))


@pytest.mark.parametrize("K,L,nprobe,few,many", [(1024, 24, 40, 512, 513), (16384, 16, 64, 512, 513), (49160, 64, 65, 255, 256), (70000, 64, 65, 3, 300),
                                                 (20001, 8, 100, 5, 600), (1024, 8, 16, 5, 700), (3000, 30, 300, 2, 520), (40001, 16, 300, 9, 257)])
def test_scoring_does_not_depend_on_the_batch(K, L, nprobe, few, many):
    """Both sides of the rules by which rows, gathers or the launch with the selection in it do the scoring (and a
    workgroup or a wavefront the selection): the same bits for a query in a small and in a large batch, and what the oracle says."""
    print("case: scoring by batch", K, L, nprobe, few, many, flush=True)
    ix = _random_index(K, L, 32, 8, 200_000, K + L)
    h = ivf.ivf_load_index(parity.to_device(ix))
    Q = np.random.default_rng(K).standard_normal((many, 32)).astype(np.float32)
    big = parity.run_gpu_search(h, Q, nprobe, 0.3, 20)
    small = parity.run_gpu_search(h, Q[:few], nprobe, 0.3, 20)
    for n in big:
        assert np.array_equal(big[n][:few], small[n]), n
    take = np.linspace(0, many - 1, 12).astype(np.int64)
    parity.check_search(ix, Q[take], nprobe, 0.3, 20, {n: v[take] for n, v in big.items()}).assert_ok()


@pytest.mark.parametrize("nq,K,D", [(4100, 100, 64), (1300, 1100, 96), (33_000, 9 * 128, 96), (66_000, 19 * 128, 128), (1000, 73 * 128, 96),
                                     (2900, 1100, 96), (2950, 130, 200), (3400, 2001, 32)])
def test_distance_gemm_over_few_groups(nq, K, D):
    """The same where the groups of centroids that are dealt to the XCDs are fewer than 8, or no multiple of 8, and on both
    sides of the 24 query tiles from which these are dealt."""
    test_distance_gemm_over_few_query_tiles(nq, K, D)


def test_noalloc_takes_a_batch_that_fits_with_fewer_workgroups_a_query():
    """298 queries x 52 001 centroids fill the 64 MiB array: 66.7 MB with one scan workgroup a query, 67.7 with two (the array
    holds 67.1), which the lists of 20 points would have otherwise.  The results do not depend on it."""
    print("case: noalloc at its limit", flush=True)
    ix = _random_index(52_001, 4, 32, 8, 4_300_000, 3)
    h = ivf.ivf_load_index(parity.to_device(ix))
    Q = torch.from_numpy(np.random.default_rng(4).standard_normal((301, 32)).astype(np.float32)).cuda()
    ids = torch.full((301, 100), -7, dtype=torch.int32, device="cuda")
    d = torch.full((301, 100), -7.0, dtype=torch.float32, device="cuda")
    ivf.ivf_search_noalloc(h, Q[:298], 16, 1.0, 100, ids[:298], d[:298])
    ref_ids, ref_d = ivf.ivf_search(h, Q[:298], 16, 1.0, 100)
    assert torch.equal(ids[:298], ref_ids) and torch.equal(d[:298], ref_d)
    with pytest.raises(ivf.IvfError):
        ivf.ivf_search_noalloc(h, Q, 16, 1.0, 100, ids, d)
    ivf.ivf_free_index(h)
