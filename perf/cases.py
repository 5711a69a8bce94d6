"""The calls whose time is measured: the query path (single queries, small batches, whole batches, the
candidate budget) and the construction of an index (encoding, k-means, product-quantiser training).

Inputs are drawn on the GPU with plain torch from a seed.  A search gets a synthetic trained index: region
centroids are the means of a Gaussian mixture (unit vectors for "deep", heavy-tailed non-negative ones for
"sift"), neighbours are the nearest of a random thousand of the other centroids, sizes of the subregions are
Poisson around a skewed rate (many subregions of a sparse index are empty), codes are uniform bytes.
"""
from __future__ import annotations

import math

import torch

import paper_1802_02422_amd as ivf

DEV = "cuda"


# ------------------------------------------------------------------------------------------ the cases

def _search(name, data, N, D, K, L, M, nq, nprobe, frac, k, budget=0):
    return {"name": name, "kind": "search", "data": data, "N": N, "D": D, "K": K, "L": L, "M": M, "nq": nq,
            "nprobe": nprobe, "frac": frac, "k": k, "budget": budget}


def listed():
    return [
        # the smallest index of the benchmark: a hundred queries, where launches are the cost
        _search("search_tiny", "deep", 100_000, 96, 1024, 8, 8, 100, 16, 0.5, 10),
        # odd numbers of queries and regions, a middle-sized index
        _search("search_small", "deep", 300_000, 96, 2000, 24, 16, 333, 40, 0.3, 100),
        # serving: one query at a time, and a small batch, against 10^8 points
        _search("search_one", "deep", 100_000_000, 96, 1 << 20, 64, 8, 1, 128, 0.2, 10),
        _search("search_64", "deep", 100_000_000, 96, 1 << 20, 64, 8, 64, 128, 0.2, 10),
        # throughput: whole batches of 10 000 against 10^7 points of both kinds and 10^9 points
        _search("search_deep10m", "deep", 10_000_000, 96, 65_536, 64, 16, 10_000, 64, 0.25, 100),
        _search("search_sift10m", "sift", 10_000_000, 128, 65_536, 64, 16, 10_000, 64, 0.25, 100),
        _search("search_deep1b", "deep", 1_000_000_000, 96, 1 << 20, 64, 16, 10_000, 256, 0.2, 100),
        # evaluation at a fixed candidate-list length
        _search("budget_deep10m", "deep", 10_000_000, 96, 65_536, 64, 16, 2_000, 256, 0.5, 100, 10_000),
        # building: base points whose region has to be found, and asked for their constant too
        {"name": "encode_base", "kind": "encode", "data": "deep", "n": 500_000, "D": 96, "K": 65_536, "L": 64, "M": 16,
         "given": False, "want_t": True},
        # building: a chunk of a very large base set, in the order of the regions it was assigned to
        {"name": "encode_chunk", "kind": "encode", "data": "deep", "n": 2_000_000, "D": 96, "K": 1 << 20, "L": 64, "M": 16,
         "given": True, "want_t": False},
        # building: the region codebook and the product quantiser from their training samples
        {"name": "kmeans", "kind": "kmeans", "data": "deep", "n": 500_000, "D": 96, "K": 16_384, "iters": 5},
        {"name": "pq_train", "kind": "pq", "data": "deep", "n": 1_000_000, "D": 96, "M": 16, "iters": 20},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "search", "budget", "encode", "encode", "kmeans", "pq"])
    data = rng.choice(["deep", "deep", "sift"])
    M = rng.choice([8, 16])
    if kind in ("search", "budget"):
        ds = rng.choice([4, 5, 6, 7, 8, 12, 16] if M == 8 else [4, 5, 6, 7, 8])
        K = 1 << rng.randint(10, 20) if rng.random() < 0.5 else _log(rng, 1000, 1 << 20)
        L = rng.randint(8, 64)
        nprobe = rng.randint(16, min(256, 32_000 // L))
        N = min(1_000_000_000, K * _log(rng, 30, 1000))
        # (the 10^9-point batch of the list is the largest amount of work in each respect)
        nq = min(_log(rng, 1, 10_000), max(1, int(10_000 * (1 << 20) * 96 / (K * max(96, M * ds)))))
        frac = round(rng.uniform(0.1, 0.5), 3)
        scanned = min(N, N / (K * L) * nprobe * L * frac)
        nq = max(1, min(nq, int(5e8 / max(scanned, 1))))
        return {"kind": "search", "data": data, "N": N, "D": M * ds, "K": K, "L": L, "M": M, "nq": nq, "nprobe": nprobe,
                "frac": frac, "k": _log(rng, 1, 100),
                "budget": _log(rng, 100, 30_000) if kind == "budget" else 0}
    if kind == "encode":
        given = rng.random() < 0.5
        return {"kind": "encode", "data": data, "n": _log(rng, 1000, 2_000_000 if given else 500_000),
                "D": M * rng.choice([4, 6, 8, 12] if M == 8 else [4, 6, 8]),
                "K": _log(rng, 1000, 1 << 20 if given else 65_536), "L": rng.randint(8, 64), "M": M, "given": given,
                "want_t": rng.random() < 0.5}
    if kind == "kmeans":
        K = _log(rng, 256, 16_384)
        return {"kind": "kmeans", "data": data, "n": K * rng.randint(25, 50), "D": rng.choice([64, 96, 104, 128]), "K": K,
                "iters": rng.randint(1, 5)}
    return {"kind": "pq", "data": data, "n": _log(rng, 20_000, 1_000_000), "D": M * rng.choice([4, 6, 8]), "M": M,
            "iters": rng.randint(5, 20)}


# ------------------------------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1_000_003 + 17)


def _means(data, n, D, g):
    m = torch.randn(n, D, generator=g, device=DEV)
    return m / m.norm(dim=1, keepdim=True) if data == "deep" else 10.0 * m * m


def _points(data, means, labels, g):
    """Mixture points: component mean plus noise, then unit length ("deep") or whole values in 0..255 ("sift")."""
    x = torch.randn(labels.shape[0], means.shape[1], generator=g, device=DEV)
    x.mul_(0.065 if data == "deep" else 6.0).add_(means[labels])
    return x / x.norm(dim=1, keepdim=True) if data == "deep" else x.round_().clamp_(0.0, 255.0)


def _neighbours(cent, L, g, block=1024):
    """(nbr [K, L] int32, squared distances [K, L]): the nearest among a random block of the other centroids."""
    K = cent.shape[0]
    block = min(block, K)
    perm = torch.randperm(K, generator=g, device=DEV)
    nbr = torch.empty(K, L, dtype=torch.int32, device=DEV)
    cs = torch.empty(K, L, device=DEV)

    def some(ids):                                         # ids [b, block]
        c = cent[ids]
        n2 = (c * c).sum(2)
        d = n2[:, :, None] + n2[:, None, :] - 2.0 * torch.bmm(c, c.transpose(1, 2).contiguous())
        d.clamp_(min=0.0).diagonal(dim1=1, dim2=2).fill_(math.inf)
        v, at = d.topk(L, dim=2, largest=False)
        return torch.gather(ids[:, None, :].expand(-1, block, -1), 2, at).int(), v

    full = K // block
    for b0 in range(0, full, 128):
        ids = perm[b0 * block:min(b0 + 128, full) * block].view(-1, block)
        nbr[ids], cs[ids] = some(ids)
    left = K - full * block
    if left:                                               # the last ones: a block that reaches back
        ids = perm[K - block:].view(1, block)
        a, b = some(ids)
        nbr[ids[0, -left:]], cs[ids[0, -left:]] = a[0, -left:], b[0, -left:]
    return nbr, cs


def _trained(c, g):
    """The trained part of an index as plain tensors."""
    cent = _means(c["data"], c["K"], c["D"], g)
    nbr, cs = _neighbours(cent, c["L"], g)
    noise = 0.065 if c["data"] == "deep" else 6.0
    t = {"cent": cent, "nbr": nbr, "cs": cs, "alpha": 0.05 + 0.12 * torch.rand(c["K"], generator=g, device=DEV)}
    t["cb"] = noise * torch.randn(c["M"], 256, c["D"] // c["M"], generator=g, device=DEV)
    # the constant of a point is 2<mu, r> + ||r||^2 with ||r||^2 about D noise^2
    size = float(cent[:1000].norm(dim=1).mean())
    t["table"] = (c["D"] * noise * noise + 2.0 * size * noise * torch.randn(256, generator=g, device=DEV)).sort()[0].contiguous()
    return t


def _encoded(c, t, g):
    """The encoded part: sizes of the subregions, codes, constants, ids."""
    nsub = c["K"] * c["L"]
    rate = torch.empty(nsub, device=DEV).exponential_(generator=g).mul_(c["N"] / nsub)
    off = torch.zeros(nsub + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.poisson(rate, generator=g).to(torch.int64)
    off = off.cumsum(0)
    n = int(off[-1])
    t["off"] = off.to(torch.int32)                         # (n is below 2^31)
    t["codes"] = torch.randint(0, 256, (n, c["M"]), generator=g, device=DEV, dtype=torch.uint8)
    t["byte"] = torch.randint(0, 256, (n,), generator=g, device=DEV, dtype=torch.uint8)
    t["ids"] = torch.empty(n, dtype=torch.int32, device=DEV)
    for a in range(0, n, 1 << 26):                         # position -> id: a fixed permutation of 0 .. n-1
        b = min(n, a + (1 << 26))
        t["ids"][a:b] = (torch.arange(a, b, device=DEV) * 2_654_435_761 % n).int()
    return t


def _queries(c, t, g):
    return _points(c["data"], t["cent"], torch.randint(0, c["K"], (c["nq"],), generator=g, device=DEV), g).contiguous()


def _desc(t, encoded=True):
    d = ivf.IndexDesc(t["cent"], t["nbr"], t["alpha"], t["cs"], t["cb"], const_table=t["table"])
    if encoded:
        d.sub_offsets, d.codes, d.const_byte, d.ids = t["off"], t["codes"], t["byte"], t["ids"]
    return d


def _inputs(c, seed):
    g = _gen(seed)
    if c["kind"] == "search":
        t = _encoded(c, _trained(c, g), g)
        return t, _queries(c, t, g)
    if c["kind"] == "encode":
        t = _trained(c, g)
        lab = torch.randint(0, c["K"], (c["n"],), generator=g, device=DEV)
        if c["given"]:
            lab = lab.sort()[0]
        return t, _points(c["data"], t["cent"], lab, g).contiguous(), lab.int() if c["given"] else None
    if c["kind"] == "kmeans":
        m = _means(c["data"], c["K"], c["D"], g)
        x = _points(c["data"], m, torch.randint(0, c["K"], (c["n"],), generator=g, device=DEV), g).contiguous()
        return x, torch.randperm(c["n"], generator=g, device=DEV)[:c["K"]].contiguous()
    # displacements: noise of a size that differs from dimension to dimension
    s = 0.02 + 0.08 * torch.rand(c["D"], generator=g, device=DEV)
    x = torch.randn(c["n"], c["D"], generator=g, device=DEV).mul_(s * (1.0 if c["data"] == "deep" else 100.0)).contiguous()
    return x, torch.randperm(c["n"], generator=g, device=DEV)[:256].contiguous()


# ------------------------------------------------------------------------------------------ the passes

def prepare(case, seed):
    c, got = case, _inputs(case, seed)
    if c["kind"] != "search":
        return (c, _desc(got[0], False), got[1], got[2]) if c["kind"] == "encode" else (c, *got)
    h = ivf.ivf_load_index(_desc(got[0]))
    ivf.ivf_set_scratch_limit(h, 48 << 30)                 # as the benchmark does: a batch is one pass
    return c, h, got[1]


def run(state):
    c = state[0]
    if c["kind"] == "search":
        _, h, q = state
        if not c["budget"]:
            return ivf.ivf_search(h, q, c["nprobe"], c["frac"], c["k"])
        r = ivf.ivf_search_budget(h, q, c["nprobe"], c["frac"], c["budget"], c["k"])
        return r["ids"], r["dists"]                        # the rest lists what was visited, for evaluations
    if c["kind"] == "encode":
        _, d, x, region = state
        r = ivf.ivf_encode(d, x, region_in=region, want_t=c["want_t"])
        return r if c["want_t"] else r[:4]
    if c["kind"] == "kmeans":
        return ivf.ivf_kmeans(state[1], c["K"], c["iters"], state[2])
    return ivf.ivf_pq_train(state[1], c["M"], c["iters"], state[2])


def work(case):
    c = case
    D = c["D"]
    if c["kind"] == "search":
        K, L, P, nq = c["K"], c["L"], c["nprobe"], c["nq"]
        S = nq * math.ceil(c["frac"] * P * L)
        recs = S * c["N"] / (K * L)
        if c["budget"]:
            recs = min(recs, nq * c["budget"])
        # centroids once, neighbours and constants of the probed regions, sizes of the kept subregions, records, results
        b = 4 * D * (K + nq) + 8 * L * min(K, nq * P) + 8 * min(K * L, S) + min(recs, c["N"]) * (c["M"] + 1) + 12 * nq * c["k"]
        return {"bytes": b, "flops": 2 * nq * K * D + 4 * nq * P * L + 2 * nq * 256 * D + recs * (c["M"] + 1)}
    n = c["n"]
    if c["kind"] == "encode":
        K, L = c["K"], c["L"]
        b = n * (4 * D + c["M"] + 9 + 4 * c["given"] + 4 * c["want_t"]) + 4 * D * K + 8 * L * min(K, n)
        return {"bytes": b, "flops": (0 if c["given"] else 2 * n * K * D) + 2 * n * L * D + 2 * n * 256 * D}
    if c["kind"] == "kmeans":
        return {"bytes": c["iters"] * (n * 4 * D + 8 * c["K"] * D), "flops": c["iters"] * (2 * n * c["K"] * D + n * D)}
    return {"bytes": c["iters"] * n * 4 * D, "flops": c["iters"] * (2 * n * 256 * D + n * D)}


def tolerance(case):
    """About four times what the results differ by from 64-bit arithmetic over the ranges of draw()."""
    k = case["kind"]
    if k == "search":
        # 32-bit sums, seen 5e-6 and 2e-5 ("sift" cancels most), 6e-5 of the ids; "max" leaves room for a subregion at
        # the edge of what is kept that changes places with its neighbour, and its points with it
        return {"rel": 2e-5, "max": 5e-3, "differ": 3e-4}
    if k == "encode":
        # whole values (seen 2e-4: a constant between two levels) but for the constant, which moves with the code of a
        # point between two words or two regions: seen 1e-3 over all points, of one point as large as the constants are
        return {"rel": 4e-3, "max": 0.99, "differ": 1e-3}
    # Lloyd rounds: a point between two centres goes to either and moves them, and so for the points after it
    return {"rel": 1e-3, "max": 0.3} if k == "kmeans" else {"rel": 3e-3, "max": 0.06}


# ------------------------------------------------------------------------------------------ in 64 bits

def _exact_search(c, t, Q):
    K, L, P, M, k = c["K"], c["L"], c["nprobe"], c["M"], c["k"]
    S = min(P * L, max(1, math.ceil(float(torch.tensor(c["frac"], dtype=torch.float32)) * P * L)))
    cent = t["cent"].double()
    cn = (cent * cent).sum(1)
    alpha, cs, table, cb = t["alpha"].double(), t["cs"], t["table"].double(), t["cb"].double()
    off = t["off"].long()
    out_i = torch.full((c["nq"], k), -1, dtype=torch.int32, device=DEV)
    out_d = torch.full((c["nq"], k), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, min(256, int(2e8 / K), int(6e6 / max(1.0, S * c["N"] / (K * L)))))
    for a in range(0, c["nq"], step):
        q = Q[a:a + step].double()
        b = q.shape[0]
        d = ((q * q).sum(1)[:, None] + cn[None]).addmm_(q, cent.t(), alpha=-2.0).clamp_(min=0.0)
        dp, pid = d.topk(P, dim=1, largest=False, sorted=False)
        nb = t["nbr"][pid].long()                                              # [b, P, L]
        al = alpha[pid][:, :, None]
        sc = (1 - al) * dp[:, :, None] + al * torch.gather(d, 1, nb.view(b, -1)).view(b, P, L) - al * (1 - al) * cs[pid].double()
        del d
        base, at = sc.view(b, -1).topk(S, dim=1, largest=False)                # ascending
        sub = torch.gather(pid, 1, at // L) * L + at % L
        start = off[sub]
        ln = off[sub + 1] - start
        if c["budget"]:
            ln = torch.where(ln.cumsum(1) - ln < c["budget"], ln, 0)
        flat = ln.reshape(-1)
        n = int(flat.sum())
        if not n:
            continue
        run_ = torch.repeat_interleave(torch.arange(flat.shape[0], device=DEV), flat, output_size=n)
        pos = torch.arange(n, device=DEV) - (flat.cumsum(0) - flat)[run_] + start.reshape(-1)[run_]
        who = run_ // S
        T = -2.0 * torch.bmm(cb, q.view(b, M, -1).permute(1, 2, 0).contiguous())  # [M, 256, b]
        est = base.reshape(-1)[run_] + table[t["byte"][pos].long()]
        codes = t["codes"][pos]
        for m in range(M):
            est += T[m].t().reshape(-1)[who * 256 + codes[:, m].long()]
        per = ln.sum(1)
        wide = int(per.max())
        full = torch.full((b, max(wide, k)), math.inf, dtype=torch.float64, device=DEV)
        col = torch.arange(n, device=DEV) - (per.cumsum(0) - per)[who]
        full[who, col] = est
        held = torch.full((b, max(wide, k)), -1, dtype=torch.int32, device=DEV)
        held[who, col] = t["ids"][pos]
        v, at = full.topk(k, dim=1, largest=False)
        out_d[a:a + b], out_i[a:a + b] = v, torch.gather(held, 1, at)
    return out_i, out_d


def _nearest(x, cent, step=None):
    """Index of the nearest row of cent for each row of x, in 64 bits."""
    cent = cent.double()
    cn = (cent * cent).sum(1)
    step = step or max(1, int(4e8 / cent.shape[0]))
    return torch.cat([(cn[None] + 0.0).expand(x[a:a + step].shape[0], -1).addmm(x[a:a + step].double(), cent.t(), alpha=-2.0).argmin(1)
                      for a in range(0, x.shape[0], step)])


def _means_of(x, lab, cent):
    """Mean of each label's rows (rounded to 32 bits, as a codebook is kept); a label without rows keeps its row."""
    K = cent.shape[0]
    s = torch.zeros(K, x.shape[1], dtype=torch.float64, device=DEV).index_add_(0, lab, x.double())
    n = torch.bincount(lab, minlength=K)
    return torch.where((n > 0)[:, None], (s / n.clamp(min=1)[:, None]).float(), cent)


def _exact_encode(c, t, x, region):
    D, M = c["D"], c["M"]
    cent = t["cent"]
    reg = region.long() if region is not None else _nearest(x, cent)
    sub, codes, byte, const = [], [], [], []
    cb, table = t["cb"].double(), t["table"].double()
    step = max(1, min(40_000, int(3e8 / (c["L"] * D))))
    for a in range(0, x.shape[0], step):
        xs, r = x[a:a + step].double(), reg[a:a + step]
        cr, al = cent[r].double(), t["alpha"][r].double()
        s = cent[t["nbr"][r].long()].double()                                  # [b, L, D]
        mu = cr[:, None] + al[:, None, None] * (s - cr[:, None])
        l = (xs[:, None] - mu).square().sum(2).argmin(1)
        mu = mu[torch.arange(mu.shape[0], device=DEV), l]
        e = (xs - mu).view(-1, M, D // M)
        dec = torch.empty_like(e)
        cd = torch.empty(e.shape[0], M, dtype=torch.uint8, device=DEV)
        for m in range(M):
            at = (e[:, m, None] - cb[m]).square().sum(2).argmin(1)
            cd[:, m], dec[:, m] = at.to(torch.uint8), cb[m][at]
        dec = dec.reshape(-1, D)
        v = (2 * mu * dec + dec * dec).sum(1)
        sub.append(l.int()), codes.append(cd), const.append(v)
        hi = torch.searchsorted(table, v).clamp(1, 255)
        byte.append(torch.where(v - table[hi - 1] <= table[hi] - v, hi - 1, hi).to(torch.uint8))
    r = reg.int(), torch.cat(sub), torch.cat(codes), torch.cat(byte)
    return (*r, torch.cat(const)) if c["want_t"] else r


def exact(case, seed):
    c, got = case, _inputs(case, seed)
    if c["kind"] == "search":
        return _exact_search(c, *got)
    if c["kind"] == "encode":
        return _exact_encode(c, *got)
    x, init = got
    if c["kind"] == "kmeans":
        cent = x[init]
        for _ in range(c["iters"]):
            cent = _means_of(x, _nearest(x, cent), cent)
        return cent.double()
    M, ds = c["M"], c["D"] // c["M"]
    book = []
    for m in range(M):
        xm = x[:, m * ds:(m + 1) * ds].contiguous()
        cb = xm[init]
        for _ in range(c["iters"]):
            cb = _means_of(xm, _nearest(xm, cb), cb)
        book.append(cb.double())
    return torch.stack(book)
