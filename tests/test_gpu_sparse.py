"""Large batches go without the distance matrix: the same bits as the same queries in batches that go with it."""
import pytest

pytestmark = pytest.mark.gpu


def make_desc(K, D, L, M, seed, spread, offset, kind=""):
    import torch
    import paper_1802_02422_amd as ivf
    g = torch.Generator(device="cuda").manual_seed(seed)
    cent = torch.randn(K, D, generator=g, device="cuda") * spread + offset
    if kind == "copies":                                      # 47 blocks and a bit of equal centroids
        cent[1000:4030] = cent[1000]
    nbr = torch.randint(0, K, (K, L), generator=g, device="cuda", dtype=torch.int32)
    cs = torch.stack([((cent - cent[nbr[:, l].long()]) ** 2).sum(1) for l in range(L)], 1).contiguous()
    if kind == "holes":                                       # distance 0 from everywhere, as with the matrix
        cent[5000], cent[9000, 3] = float("nan"), float("inf")
    alpha = torch.rand(K, generator=g, device="cuda") * 0.3
    cb = torch.randn(M, 256, D // M, generator=g, device="cuda") * 0.1 * spread
    n = 2 * K * L
    off = torch.sort(torch.randint(0, n + 1, (K * L + 1,), generator=g, device="cuda"))[0].int()
    off[0], off[-1] = 0, n
    desc = ivf.IndexDesc(cent, nbr, alpha, cs, cb, const_table=torch.sort(torch.randn(256, generator=g, device="cuda"))[0].contiguous(),
                         sub_offsets=off, codes=torch.randint(0, 256, (n, M), generator=g, device="cuda", dtype=torch.uint8),
                         const_byte=torch.randint(0, 256, (n,), generator=g, device="cuda", dtype=torch.uint8),
                         ids=torch.randperm(n, generator=g, device="cuda").int())
    return desc, cent, g


def make(*args):
    import paper_1802_02422_amd as ivf
    desc, cent, g = make_desc(*args)
    return ivf.ivf_load_index(desc), cent, g


def ways(call, *args):
    """(what the call returns, passes it took without the matrix, passes with it)"""
    import paper_1802_02422_amd as ivf
    before = ivf.ivf_search_stats()
    got = call(*args)
    after = ivf.ivf_search_stats()
    return got, after[0] - before[0], after[1] - before[1]


def same(got, ref):
    import torch
    for name in ref:
        assert torch.equal(got[name].view(torch.uint8), ref[name].view(torch.uint8)), name


# partial last tiles and blocks, every packed width, L below, at and above a group of 64 neighbours and of odd length; "hard": queries
# too large for the table's scale, all without a bound; "far": far from the table; "tiny": the queries' fp16 components are subnormal;
# "some": queries too large for the table's scale, far, without a finite length, zero, and equal to centroids;
# "copies": more centroids at the same distance than the selection holds in LDS; "holes": centroids that are not finite
@pytest.mark.parametrize("K,D,L,M,P,nq,kind", [
    (16_400, 96, 64, 16, 16, 9000, "plain"), (16_385, 32, 7, 8, 13, 8500, "plain"), (20_033, 64, 65, 16, 16, 7001, "plain"), (16_500, 32, 128, 8, 12, 8200, "plain"),
    (17_000, 128, 33, 16, 8, 9000, "plain"), (70_001, 48, 64, 8, 60, 4200, "plain"), (16_400, 96, 32, 16, 16, 8300, "hard"), (16_400, 96, 32, 16, 16, 8300, "far"),
    (16_400, 96, 32, 16, 16, 8300, "tiny"),
    (16_640, 96, 16, 16, 16, 8300, "some"), (16_400, 96, 16, 16, 16, 8300, "equal"), (66_000, 32, 16, 8, 64, 4200, "copies"),
    (16_600, 96, 16, 16, 16, 8300, "holes")])
def test_same_bits_as_with_the_distance_matrix(K, D, L, M, P, nq, kind):
    import torch
    import paper_1802_02422_amd as ivf
    h, cent, g = make(K, D, L, M, K + D, 1.0, 0.0, kind)
    q = cent[torch.randint(0, K, (nq,), generator=g, device="cuda")].nan_to_num(0.0, 0.0, 0.0)
    if kind == "copies":
        q[::3] = cent[1000]
    q = (q + 0.5 * torch.randn(nq, D, generator=g, device="cuda") + {"hard": 1e5, "far": 50.0}.get(kind, 0.0)).contiguous()
    if kind == "tiny":
        q *= 2.0 ** -19
    if kind == "some":
        q[::7] *= 1e5
        q[1::7] *= 300.0
        q[3::11] = 0.0
        q[5::13] = cent[:q[5::13].shape[0]]
        q[1, 0], q[2, 3], q[400, 5] = float("nan"), float("inf"), -float("inf")
    if kind == "equal":                                       # every query the same: one block and one region have all pairs
        q[:] = q[0]
    ivf.ivf_set_scratch_limit(h, 16 << 30)
    whole, without, matrix = ways(ivf.ivf_search_stages, h, q, P, 0.3, 20)
    assert (without, matrix) == (1, 0)
    parts, without, matrix = ways(lambda: [ivf.ivf_search_stages(h, q[a:a + 500].contiguous(), P, 0.3, 20) for a in range(0, nq, 500)])
    assert (without, matrix) == (0, len(parts))
    same(whole, {name: torch.cat([p[name] for p in parts]) for name in whole})
    # a scratch limit that cuts three times the batch into passes
    q, whole = q.repeat(3, 1), {name: torch.cat([v] * 3) for name, v in whole.items()}
    for mb in range(700, 50, -25):
        ivf.ivf_set_scratch_limit(h, mb << 20)
        again, without, matrix = ways(ivf.ivf_search_stages, h, q, P, 0.3, 20)
        if without != 1 or matrix:
            break
    assert without > 1 and matrix == 0
    same(again, whole)
    ivf.ivf_free_index(h)


# batches whose pairs are not grouped: one query, odd numbers, the largest; no bound for every query or for some, far queries, tiny ones.  Tables of more than
# 4096 blocks, whose queries without a bound take another kernel: such a batch, and one whose pairs are grouped
@pytest.mark.parametrize("K,D,L,M,P,nq,kind", [
    (300_000, 32, 8, 8, 16, 100, "plain"), (262_144, 96, 64, 16, 64, 1, "plain"), (270_001, 64, 33, 16, 20, 33, "plain"),
    (262_144, 128, 65, 8, 16, 129, "plain"), (262_144, 96, 16, 16, 16, 70, "hard"), (262_144, 96, 16, 16, 16, 256, "some"),
    (300_000, 32, 8, 8, 16, 40, "hard"), (300_000, 32, 8, 8, 16, 40, "far"), (262_144, 96, 16, 16, 16, 70, "tiny"), (300_001, 32, 8, 8, 16, 700, "some")])
def test_small_batches_same_bits(K, D, L, M, P, nq, kind):
    import torch
    import paper_1802_02422_amd as ivf
    h, cent, g = make(K, D, L, M, K + D, 1.0, 0.0)
    q = cent[torch.randint(0, K, (nq,), generator=g, device="cuda")]
    q = (q + 0.5 * torch.randn(nq, D, generator=g, device="cuda") + {"hard": 1e5, "far": 50.0}.get(kind, 0.0)).contiguous()
    if kind == "tiny":
        q *= 2.0 ** -19
    if kind == "some":
        q[::7] *= 1e5
        q[1::7] *= 300.0
        q[3::11] = 0.0
        q[1, 0], q[2, 3] = float("nan"), float("inf")
    got, without, matrix = ways(ivf.ivf_search_stages, h, q, P, 0.3, 20)
    assert (without, matrix) == (1, 0)
    ivf.ivf_set_scratch_limit(h, 4 << 20)                     # less than such a pass takes: the distance matrix, a few queries at a time
    ref, without, matrix = ways(ivf.ivf_search_stages, h, q, P, 0.3, 20)
    assert without == 0 and matrix >= 1
    same(got, ref)
    if nq <= 33:                                              # what fits the static array, always with the matrix
        ids, d = torch.empty_like(ref["ids"]), torch.empty_like(ref["dists"])
        ivf.ivf_search_noalloc(h, q, P, 0.3, 20, ids, d)
        same({"ids": ids, "dists": d}, {"ids": ref["ids"], "dists": ref["dists"]})
    ivf.ivf_free_index(h)


def test_last_pass_of_a_large_batch_is_a_small_one():
    """Scratch limits that cut 2100 queries into passes, the last of which may be small enough for pairs that are not grouped."""
    import torch
    import paper_1802_02422_amd as ivf
    h, cent, g = make(262_144, 32, 8, 8, 5, 1.0, 0.0)
    q = (cent[torch.randint(0, 262_144, (2100,), generator=g, device="cuda")] + 0.5 * torch.randn(2100, 32, generator=g, device="cuda")).contiguous()
    ivf.ivf_set_scratch_limit(h, 16 << 30)
    ref, without, matrix = ways(ivf.ivf_search_stages, h, q, 16, 0.3, 20)
    assert (without, matrix) == (1, 0)
    for mb, passes in ((45, (4, 0)), (60, (2, 0)), (20, (0, 105))):   # (640 a pass and 180 left; 1152 and 948; 20 with the matrix)
        ivf.ivf_set_scratch_limit(h, mb << 20)
        got, without, matrix = ways(ivf.ivf_search_stages, h, q, 16, 0.3, 20)
        assert (without, matrix) == passes, mb
        same(got, ref)
    ivf.ivf_free_index(h)


# more than 64 neighbours a region: each further 64 are rows of their own to read, for every pair
@pytest.mark.parametrize("L,nq,ways", [(64, 2048, (1, 0)), (128, 2048, (1, 0)), (256, 2048, (0, 1)), (256, 8192, (1, 0))])
def test_way_by_the_number_of_neighbours(L, nq, ways):
    import torch
    import paper_1802_02422_amd as ivf
    h, cent, g = make(65_536, 32, L, 8, 3, 1.0, 0.0)
    q = cent[torch.randint(0, 65_536, (nq,), generator=g, device="cuda")].contiguous()
    before = ivf.ivf_search_stats()
    ivf.ivf_search(h, q, 16, 0.1, 10)
    assert tuple(a - b for a, b in zip(ivf.ivf_search_stats(), before)) == ways
    ivf.ivf_free_index(h)


def test_scratch_keeps_to_the_limit():
    """Passes without the distance matrix are of more queries than passes with it: descriptors, tables and lists of all of
    them count.  A handle that has seen both kinds holds one buffer for both."""
    import torch
    import paper_1802_02422_amd as ivf
    K, nq, limit = 65_536, 40_000, 1 << 30
    h, cent, g = make(K, 32, 32, 16, 9, 1.0, 0.0)
    q = (cent[torch.randint(0, K, (nq,), generator=g, device="cuda")] + 0.5 * torch.randn(nq, 32, generator=g, device="cuda")).contiguous()
    ids, dists = (torch.empty(nq, 1000, dtype=t, device="cuda") for t in (torch.int32, torch.float32))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    before = ivf.ivf_search_stats()
    ivf.ivf_set_scratch_limit(h, limit)
    ivf.ivf_search(h, q, 16, 1.0, 1000, ids, dists)
    without, matrix = (a - b for a, b in zip(ivf.ivf_search_stats(), before))
    assert without >= 2 and matrix == 0
    ivf.ivf_search(h, q[:1024], 16, 1.0, 1000, ids[:1024], dists[:1024])
    assert ivf.ivf_search_stats()[1] == before[1] + 1
    torch.cuda.synchronize()
    held = free - torch.cuda.mem_get_info()[0]
    assert held <= limit, held
    again = torch.empty_like(ids), torch.empty_like(dists)
    ivf.ivf_set_scratch_limit(h, 16 << 30)
    ivf.ivf_search(h, q, 16, 1.0, 1000, *again)
    assert torch.equal(ids, again[0]) and torch.equal(dists, again[1])
    ivf.ivf_free_index(h)


def fill_memory(leave):
    """Takes all of the GPU's memory but `leave` bytes."""
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while torch.cuda.mem_get_info()[0] > leave + (8 << 20):
        held.append(torch.empty(min(8 << 30, torch.cuda.mem_get_info()[0] - leave), dtype=torch.uint8, device="cuda"))
    return held


def test_no_memory_for_a_whole_batch():
    """Less memory than the batch's pass asks for, and the limit allows: it goes in smaller ones, and so do the next."""
    import torch
    import paper_1802_02422_amd as ivf
    K, nq = 65_536, 40_000
    h, cent, g = make(K, 32, 32, 16, 9, 1.0, 0.0)
    q = (cent[torch.randint(0, K, (nq,), generator=g, device="cuda")] + 0.5 * torch.randn(nq, 32, generator=g, device="cuda")).contiguous()
    ids, dists = (torch.empty(nq, 1000, dtype=t, device="cuda") for t in (torch.int32, torch.float32))
    again = torch.empty_like(ids), torch.empty_like(dists)
    ivf.ivf_set_scratch_limit(h, 1 << 30)
    ivf.ivf_search(h, q, 16, 1.0, 1000, ids, dists)
    ivf.ivf_free_index(h)
    h, cent, g = make(K, 32, 32, 16, 9, 1.0, 0.0)
    ivf.ivf_set_scratch_limit(h, 16 << 30)
    held = fill_memory(2 << 30)                               # (a pass of all of them takes 2.9 GB)
    try:
        passes = []
        for _ in range(2):
            before = ivf.ivf_search_stats()
            ivf.ivf_search(h, q, 16, 1.0, 1000, *again)
            torch.cuda.synchronize()
            passes.append(tuple(a - b for a, b in zip(ivf.ivf_search_stats(), before)) + torch.cuda.mem_get_info())
    finally:
        del held
        torch.cuda.empty_cache()
    assert passes[0][0] >= 2 and passes[0][1] == 0 and passes[0] == passes[1]
    assert torch.equal(ids, again[0]) and torch.equal(dists, again[1])
    ivf.ivf_free_index(h)


def test_no_memory_beside_the_tables():
    """A batch that goes with the matrix, and has no room for it beside the tables of the other way."""
    import torch
    import paper_1802_02422_amd as ivf
    K = 1 << 20
    h, cent, g = make(K, 96, 64, 8, 9, 1.0, 0.0)
    q = cent[torch.randint(0, K, (256,), generator=g, device="cuda")].contiguous()
    few = q[:16].contiguous()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ref = ivf.ivf_search(h, q, 300, 0.2, 10)
    before = ivf.ivf_search_stats()
    small = ivf.ivf_search(h, few, 16, 0.2, 10)
    assert ivf.ivf_search_stats()[0] == before[0] + 1
    torch.cuda.synchronize()
    need = free - torch.cuda.mem_get_info()[0]
    ivf.ivf_free_index(h)
    h = make(K, 96, 64, 8, 9, 1.0, 0.0)[0]
    ivf.ivf_free_index(make(1000, 32, 8, 8, 1, 1.0, 0.0)[0])    # (gives back what the library keeps for index-time calls)
    held = fill_memory(need - (200 << 20))
    try:
        got = ivf.ivf_search(h, q, 300, 0.2, 10)
        before = ivf.ivf_search_stats()
        less = ivf.ivf_search(h, few, 16, 0.2, 10)
        assert ivf.ivf_search_stats()[1] == before[1] + 1
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert all(torch.equal(a, b) for a, b in zip(got + less, ref + small))
    ivf.ivf_free_index(h)


def test_no_memory_for_the_tables():
    """An index that can be loaded, but not with the tables of the search without the matrix: it goes with the matrix."""
    import torch
    import paper_1802_02422_amd as ivf
    K = 1 << 20
    desc, cent, g = make_desc(K, 128, 8, 8, 9, 1.0, 0.0)      # (312 bytes a region; sizes and offsets on the way 64)
    q = cent[torch.randint(0, K, (16,), generator=g, device="cuda")].contiguous()
    small = [make_desc(1000, 32, 8, 8, 1, 1.0, 0.0)[0] for _ in range(2)]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    h = ivf.ivf_load_index(desc)
    ivf.ivf_free_index(ivf.ivf_load_index(small[0]))          # (gives back what the library keeps for index-time calls)
    need = free - torch.cuda.mem_get_info()[0]
    ref = ivf.ivf_search(h, q, 16, 0.2, 10)
    ivf.ivf_free_index(h)
    held = fill_memory(need - (200 << 20))
    try:
        h = ivf.ivf_load_index(desc)
    finally:
        del held
        torch.cuda.empty_cache()
    ivf.ivf_free_index(ivf.ivf_load_index(small[1]))
    before = ivf.ivf_search_stats()
    got = ivf.ivf_search(h, q, 16, 0.2, 10)
    torch.cuda.synchronize()
    assert ivf.ivf_search_stats()[1] == before[1] + 1
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    ivf.ivf_free_index(h)


# a table far from the origin compared with its spread: bounds too wide for all its queries
@pytest.mark.parametrize("K,P,nq,offset,way", [(65_536, 16, 4096, 0.0, 0), (65_536, 16, 4096, 50.0, 1), (262_144, 16, 64, 0.0, 0), (262_144, 16, 64, 50.0, 1)])
def test_tables_with_wide_bounds_go_with_the_matrix(K, P, nq, offset, way):
    import torch
    import paper_1802_02422_amd as ivf
    h, cent, g = make(K, 32, 8, 8, 6, 1.0, offset)
    q = (cent[torch.randint(0, K, (nq,), generator=g, device="cuda")] + 0.5 * torch.randn(nq, 32, generator=g, device="cuda")).contiguous()
    before = ivf.ivf_search_stats()
    ivf.ivf_search(h, q, P, 0.3, 20)
    assert ivf.ivf_search_stats()[way] == before[way] + 1
    ivf.ivf_free_index(h)


@pytest.mark.parametrize("nq", [64, 1024])
def test_replays_from_a_captured_graph(nq):
    """Every replay, on other queries and with eager searches of both kinds of batches in between, returns the bits of the eager call."""
    import torch
    import paper_1802_02422_amd as ivf
    K = 262_144
    h, cent, g = make(K, 32, 8, 8, 4, 1.0, 0.0)
    draw = lambda: (cent[torch.randint(0, K, (nq,), generator=g, device="cuda")] + 0.5 * torch.randn(nq, 32, generator=g, device="cuda")).contiguous()
    q = draw()
    eager, without, matrix = ways(ivf.ivf_search, h, q, 16, 0.3, 20)     # sizes the scratch buffers
    assert (without, matrix) == (1, 0)
    ivf.ivf_search(h, draw()[:50].contiguous(), 300, 0.3, 20)
    ids, d = torch.empty_like(eager[0]), torch.empty_like(eager[1])
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ivf.ivf_search(h, q, 16, 0.3, 20, ids, d)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ivf.ivf_search(h, q, 16, 0.3, 20, ids, d)
    for rep in range(4):
        q.copy_(draw())
        ids.fill_(-7)
        d.fill_(-7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = ids.clone(), d.clone()
        ivf.ivf_search(h, draw()[:50].contiguous(), 300 if rep % 2 else 16, 0.3, 20)
        ref = ivf.ivf_search(h, q, 16, 0.3, 20)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), rep
    del graph
    ivf.ivf_free_index(h)
