// C ABI of the library (see include/ivf_gp.h): argument checks, scratch
// management and the launch sequence of the query path.  gfx950 only.
#include "../../include/ivf_gp.h"

#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include <hip/hip_runtime.h>
#include <rocprim/device/device_scan.hpp>

#include "budget.hpp"
#include "coarse.hpp"
#include "encode.hpp"
#include "latency.hpp"
#include "layout.hpp"
#include "order.hpp"
#include "pool.hpp"
#include "pq.hpp"
#include "query.hpp"
#include "scan.hpp"
#include "sparse.hpp"
#include "train.hpp"

using namespace ivf;

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIPCHK(expr)                                                                         \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(e_ == hipErrorOutOfMemory ? IVF_ENOMEM : IVF_EHIP, "%s: %s", #expr,  \
                        hipGetErrorString(e_));                                              \
    } while (0)

#define LAUNCHCHK(name)                                                                      \
    do {                                                                                     \
        hipError_t e_ = hipGetLastError();                                                   \
        if (e_ != hipSuccess) return fail(IVF_EHIP, "launch %s: %s", name, hipGetErrorString(e_)); \
    } while (0)

struct Buf {
    void *p = nullptr;
    size_t bytes = 0;
};

DevPool g_pool;

// Scratch from the pool, given back when the scope ends, error returns included: the owner has waited for the stream by then.
struct DevTmp {
    void *p = nullptr;
    size_t bytes = 0;
    int dev = 0;
    DevTmp() = default;
    DevTmp(const DevTmp &) = delete;
    DevTmp &operator=(const DevTmp &) = delete;
    hipError_t alloc(size_t n) { return g_pool.take(&p, &bytes, &dev, n); }
    ~DevTmp() { if (p) g_pool.give(p, bytes, dev); }
};

// Waits for the stream when the scope ends: declared behind the DevTmps of a function that may return in the middle.
struct StreamWait {
    hipStream_t st;
    explicit StreamWait(hipStream_t s) : st(s) {}
    ~StreamWait() { (void)hipStreamSynchronize(st); }
};

int ensure(Buf &b, size_t bytes)
{
    if (bytes <= b.bytes) return IVF_OK;
    if (b.p) {
        HIPCHK(hipDeviceSynchronize());
        HIPCHK(hipFree(b.p));
        b.p = nullptr;
        b.bytes = 0;
    }
    HIPCHK(g_pool.fresh(&b.p, bytes));
    b.bytes = bytes;
    return IVF_OK;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int next_pow2(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

int check_trained(const ivf_index_desc *d)
{
    if (!d) return fail(IVF_EINVAL, "index descriptor is NULL");
    if (d->D < 4 || d->D > IVF_MAX_D || d->D % 4) return fail(IVF_EINVAL, "D=%d must be a multiple of 4 in [4, %d]", d->D, IVF_MAX_D);
    if (d->M != 8 && d->M != 16) return fail(IVF_EINVAL, "M=%d must be 8 or 16", d->M);
    if (d->D % d->M) return fail(IVF_EINVAL, "D=%d is not a multiple of M=%d", d->D, d->M);
    if (d->L < 1 || d->K < 1) return fail(IVF_EINVAL, "K=%lld and L=%d must be positive", (long long)d->K, d->L);
    if ((int64_t)d->L >= d->K && d->K > 1) return fail(IVF_EINVAL, "L=%d needs at least L+1 centroids", d->L);
    if (d->K * (int64_t)d->L >= (1ll << 31)) return fail(IVF_EINVAL, "K*L must be below 2^31");
    if (!d->centroids || !d->nbr || !d->alpha || !d->cs_dist2)
        return fail(IVF_EINVAL, "a trained array (centroids, nbr, alpha, cs_dist2) is NULL");
    if (!aligned16(d->centroids)) return fail(IVF_EINVAL, "centroids must be 16-byte aligned");
    return IVF_OK;
}

// ------------------------------------------------------------ stage 1 driver
template <bool FINITE>
int launch_absmax(const float *X, int64_t count, uint32_t *gmax, hipStream_t st)
{
    HIPCHK(hipMemsetAsync(gmax, 0, sizeof(uint32_t), st));
    int64_t grid = (count + 1023) / 1024;
    if (grid > 1024) grid = 1024;
    absmax_kernel<FINITE><<<dim3((unsigned)grid), dim3(256), 0, st>>>(X, count, gmax);
    LAUNCHCHK("absmax_kernel");
    return IVF_OK;
}

// Packs the rows of X for the GEMM (hi/lo fp16 stages, see split_rows_kernel) and writes their
// squared norms and inverse scales.  gmax != NULL: one scale for the whole matrix (gmax is a
// device word used for the reduction, inv receives one float); else one scale per row.
int pack_rows(const float *X, int64_t n, int D, uint32_t *gmax, _Float16 *P, float *norm, float *inv,
              hipStream_t st)
{
    if (n <= 0) return IVF_OK;
    if (gmax) {
        int rc = launch_absmax<true>(X, n * D, gmax, st);
        if (rc) return rc;
    }
    split_rows_kernel<<<dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st>>>(X, n, D, gmax, P, norm, inv);
    LAUNCHCHK("split_rows_kernel");
    return IVF_OK;
}

// Tiles from which the swept GEMM is taken: below, one tile a workgroup spreads them over more of the chip (100 queries x
// 1024 centroids: 40 us as one workgroup's sweep, 16 as eight).
constexpr int64_t SWEEP_MIN_TILES = 2048;

// Centroid tiles that a workgroup of the swept GEMM takes: as many as leave 1024 workgroups, but no more than 64 and no
// fewer than 8, unless the last round is the better filled with another number.  Two workgroups fit a compute unit, 64 an
// XCD; the XCD with most work goes through its sweeps, each with a tile's time for loading its query tile, in rounds, and half
// a sweep more where they drift apart.  By sweep length 64, 32, 16, 8 (us; in brackets the one taken, a * for 1024 workgroups):
// 10 000 queries x 65 536 844, 748*, [695], 666; x 131 072 1412*, 1300, [1232], 1271; x 100 096 1150*, 1062, [974], 981;
// 7000 x 65 536 510, 496, [459]*, 469; 4000 259, 231, [248]*, 252; 100 000 x 2432 (19 tiles) 315, 315, 371*, [271]; x 1152
// (9 tiles: all but 8 take it whole) [181], 181, 181, 217*.
int sweep_length(int64_t tiles_q, int64_t tiles_c)
{
    auto estimate = [&](int p) {
        const int64_t groups = (tiles_c + p - 1) / p, rounds = (group_grid(tiles_q, groups) / N_XCD + 63) / 64;
        return (double)rounds * ((double)tiles_c / (double)groups + 1.0) + 0.5 * (double)(p < tiles_c ? p : tiles_c);
    };
    int best = 64;
    while (best > SWEEP_BMC && tiles_q * ((tiles_c + best - 1) / best) < 1024) best /= 2;
    double least = 0.95 * estimate(best);
    for (int p = 64; p >= SWEEP_BMC; p /= 2) {
        const double e = estimate(p);
        if (e < least) {
            best = p;
            least = e;
        }
    }
    return best;
}

int launch_coarse(const _Float16 *xp, const float *xn, const float *xsi, int64_t nq, const _Float16 *Cp,
                  const float *cn, const float *csi, int64_t K, int Dp, float *Dt, float *bm, hipStream_t st)
{
    const int64_t ldt = dt_stride(K);
    const int nb = (int)((K + BMW - 1) / BMW);
    if (nq <= 2 * SKQ) {   // small batch: one tile of 32 or 64 queries, the centroid table streamed once
        const int64_t cblocks = (K + SKC - 1) / SKC;
        const int64_t grid = (cblocks + N_XCD - 1) / N_XCD * N_XCD;
        if (nq <= SKQ)
            coarse_gemm_skinny_kernel<1><<<dim3((unsigned)grid), dim3(256), 0, st>>>(xp, xn, xsi, nq, Cp, cn, csi, K, Dp, Dt, ldt, bm, nb, 1);
        else
            coarse_gemm_skinny_kernel<2><<<dim3((unsigned)grid), dim3(256), 0, st>>>(xp, xn, xsi, nq, Cp, cn, csi, K, Dp, Dt, ldt, bm, nb, 1);
        LAUNCHCHK("coarse_gemm_skinny_kernel");
        return IVF_OK;
    }
    const int tiles_q = (int)((nq + GT - 1) / GT);
    const int64_t tiles_c = (K + GT - 1) / GT;
    const int stages = Dp / DK;
    if ((stages == 6 || stages == 8) && K % GT == 0 && (int64_t)tiles_q * tiles_c >= SWEEP_MIN_TILES) {
        // Query tile held in registers, centroid tiles swept.  The kernel works on whole tiles: the
        // rows of a partial last query tile are computed too, into the padding every per-query
        // buffer of the coarse stage carries up to a multiple of the tile height.
        const int per_wg = sweep_length(tiles_q, tiles_c);
        static_assert(64 % SWEEP_BMC == 0, "a workgroup's first tile starts a 64-byte piece of the block minima");
        const int64_t g2 = group_grid(tiles_q, (tiles_c + per_wg - 1) / per_wg);
        if (g2 >= (1ll << 24)) return fail(IVF_EINVAL, "coarse tile grid too large (more than 2^32 threads)");
        if (stages == 6)
            coarse_gemm_sweep_kernel<6><<<dim3((unsigned)g2), dim3(256), 0, st>>>(xp, xn, xsi, (int64_t)tiles_q * GT, Cp, cn, csi, K, Dt, ldt, bm, nb, tiles_q, (int)tiles_c, per_wg);
        else
            coarse_gemm_sweep_kernel<8><<<dim3((unsigned)g2), dim3(256), 0, st>>>(xp, xn, xsi, (int64_t)tiles_q * GT, Cp, cn, csi, K, Dt, ldt, bm, nb, tiles_q, (int)tiles_c, per_wg);
        LAUNCHCHK("coarse_gemm_sweep_kernel");
        return IVF_OK;
    }
    const int64_t grid = tile_grid(tiles_q, tiles_c);
    if (grid >= (1ll << 24)) return fail(IVF_EINVAL, "coarse tile grid too large (more than 2^32 threads)");
    coarse_gemm_kernel<<<dim3((unsigned)grid), dim3(256), 0, st>>>(xp, xn, xsi, nq, Cp, cn, csi, K, Dp, Dt, ldt, bm, nb, tiles_q);
    LAUNCHCHK("coarse_gemm_kernel");
    return IVF_OK;
}

// Whether probe_select_wave_kernel takes the selection of P of K for nq queries.  Up to PW_K_DIRECT distances always (1000:
// 17 us for 300 queries, 38 for 10 000; a workgroup a query 26 and 405).  Above, a wavefront has P flagged blocks to read,
// 16 at a time, and takes 20 us (P = 16), 33 (40) or 50 (64) however few the queries are, where the 512 workgroups
// that run at a time take 24: 500 queries 29, 1000 51, 2000 94, P = 64 with a wavefront each 51, 52, 54.  Where more
// distances survive than a wavefront holds (centroids whose numbers follow their places) it takes twice that.  From 16 P
// queries on it is the faster one, or equal, and then at most 1.4 times as slow up to 24 P.
bool wave_select_fits(int64_t K, int P, int64_t nq)
{
    if (K <= PW_K_DIRECT) return true;
    const int64_t nb = (K + BMW - 1) / BMW;
    return nb <= PW_NB_MAX && P <= nb && P <= PW_P_MAX && nq >= 16 * P;
}

int launch_probe_select(const float *Dt, const float *bm, int64_t nq, int64_t K, int P, int32_t *pid,
                        float *pd, hipStream_t st)
{
    const int nb = (int)((K + BMW - 1) / BMW);
    const size_t lds = (size_t)2 * P * sizeof(int);
    if (wave_select_fits(K, P, nq)) {            // a wavefront per query, keys in registers
        const dim3 grid((unsigned)((nq + 3) / 4));
        if (K <= PW_K_DIRECT / 2) probe_select_wave_kernel<PW_K_DIRECT / 2><<<grid, dim3(256), 0, st>>>(Dt, dt_stride(K), bm, K, nb, P, nq, pid, pd);
        else if (K <= PW_K_DIRECT) probe_select_wave_kernel<PW_K_DIRECT><<<grid, dim3(256), 0, st>>>(Dt, dt_stride(K), bm, K, nb, P, nq, pid, pd);
        else probe_select_wave_kernel<0><<<grid, dim3(256), 0, st>>>(Dt, dt_stride(K), bm, K, nb, P, nq, pid, pd);
        LAUNCHCHK("probe_select_wave_kernel");
        return IVF_OK;
    }
    if (P <= PS_P_MAX && nb <= PS_NB_MAX) {   // a workgroup per query, keys in registers
        const size_t lds2 = ps_lds_bytes(P);
        if (lds2 > 48 * 1024)
            HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&probe_select_lds_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds2));
        probe_select_lds_kernel<<<dim3((unsigned)nq), dim3(1024), lds2, st>>>(Dt, dt_stride(K), bm, K, nb, P, pid, pd);
        LAUNCHCHK("probe_select_lds_kernel");
        return IVF_OK;
    }
    if (P >= 1024)
        probe_select_kernel<1024><<<dim3((unsigned)nq), dim3(1024), lds, st>>>(Dt, dt_stride(K), bm, K, nb, P, pid, pd);
    else
        probe_select_kernel<256><<<dim3((unsigned)nq), dim3(256), lds, st>>>(Dt, dt_stride(K), bm, K, nb, P, pid, pd);
    LAUNCHCHK("probe_select_kernel");
    return IVF_OK;
}

// Device scratch of one pass over a tile of queries, and the launch shape that goes with it.
struct SearchWs {
    float *dt = nullptr, *bm = nullptr, *qn = nullptr, *qsi = nullptr;
    _Float16 *qpk = nullptr;
    int32_t *probe_id = nullptr;
    float *probe_d = nullptr;
    SubDesc *desc = nullptr;
    float *lut = nullptr;
    uint64_t *partial = nullptr;
    float *qrot = nullptr;       // rotated queries (indexes with a rotation in front of the PQ)
    unsigned char *sparse() const { return reinterpret_cast<unsigned char *>(dt); }   // a pass has either
};

enum { WS_DT, WS_BM, WS_QN, WS_QSI, WS_QPK, WS_PID, WS_PD, WS_DESC, WS_LUT, WS_PARTIAL, WS_QROT, WS_COUNT };

// Scratch of a pass of the search without the distance matrix: pieces of one buffer.
enum { SP_QH, SP_QLEN, SP_BEST, SP_FLAG, SP_LIST, SP_RANK, SP_THR, SP_COUNT, SP_OFFSET, SP_HARD, SP_HROWS, SP_HN, SP_HSI, SP_PAIRS, SP_ITEMS,
       SP_HEAD, SP_BIG, SP_PIECES };   // SP_BIG: the distances of the flagged blocks, then the scores
struct SparsePlan {
    bool direct = false;         // a pair is a work item
    int cap = 0, shift = 0;
    int64_t block_items = 0, region_items = 0, count_words = 0;
    size_t off[SP_PIECES], total = 0;
};

// Queries up to which a pair is a work item of its own, instead of being grouped with the other queries' pairs of its block or region:
// grouping takes four launches and counters for all regions.  A search in us grouped / so (the matrix where that is the faster), L = 64,
// D = 96: K = 2^20, P = 16, 128 queries 188 / 132, 256 231 / 176, 512 317 / 269, 1024 496 / 468; P = 64, 256 323 / 279, 512 454 / 460;
// P = 128, 256 445 / 409, 512 579 / 715; K = 262 144, P = 16, 256 140 / 115, 512 165 / 170.
constexpr int64_t SPARSE_DIRECT = 256;

// Whether an index gets the tables for it.
bool sparse_table(int64_t K, int D) { return K >= SPARSE_MIN_K && (K + BMW - 1) / BMW <= PS_NB_MAX && packed_dim(D) <= 128; }

SparsePlan plan_sparse(int64_t K, int D, int P, int L, int64_t n)
{
    SparsePlan sp;
    const int Dp = packed_dim(D);
    const int64_t nb = (K + BMW - 1) / BMW, pad = packed_rows(n);
    while ((1 << sp.shift) < 2 * P || sp.shift < 2) ++sp.shift;
    sp.cap = 1 << sp.shift;
    const int64_t bp = n * (sp.cap < nb ? sp.cap : nb), rp = n * P;
    sp.direct = n <= SPARSE_DIRECT;
    sp.block_items = sp.direct ? bp : bp / PAIR_Q + (bp < nb ? bp : nb);
    sp.region_items = sp.direct ? rp : rp / PAIR_Q + (rp < K ? rp : K);
    sp.count_words = ((sp.direct ? 0 : N_XCD * (nb + K)) + 8) / 2;   // 64-bit words: counts of blocks and regions, totals
    size_t bytes[SP_PIECES];
    bytes[SP_QH] = (size_t)pad * Dp * sizeof(_Float16);
    bytes[SP_QLEN] = (size_t)pad * sizeof(float2);
    bytes[SP_BEST] = (size_t)pad * 2 * minima_half(K) * sizeof(float);
    bytes[SP_FLAG] = bytes[SP_THR] = bytes[SP_HARD] = (size_t)n * 4;
    bytes[SP_LIST] = bytes[SP_RANK] = (size_t)n * sp.cap * 4;
    bytes[SP_COUNT] = (size_t)sp.count_words * 8;
    bytes[SP_OFFSET] = sp.direct ? 0 : (size_t)N_XCD * K * 4;
    bytes[SP_HROWS] = (size_t)pad * Dp * 2 * sizeof(_Float16);
    bytes[SP_HN] = bytes[SP_HSI] = (size_t)pad * sizeof(float);
    bytes[SP_PAIRS] = (size_t)n * sp.cap * 4;
    bytes[SP_ITEMS] = (size_t)(sp.block_items > sp.region_items ? sp.block_items : sp.region_items) * sizeof(uint4);
    bytes[SP_HEAD] = (size_t)n * sp.cap * sizeof(uint4);
    const size_t cand = (size_t)n * sp.cap * BMW * 4, keys = (size_t)n * P * L * 4;
    bytes[SP_BIG] = cand > keys ? cand : keys;
    for (int i = 0; i < SP_PIECES; ++i) {
        sp.off[i] = sp.total;
        sp.total += (bytes[i] + 255) / 256 * 256;
    }
    return sp;
}

// ... of a batch taken n at a time: the last pass may be a small one, of the other kind
size_t sparse_bytes(int64_t K, int D, int P, int L, int64_t n)
{
    const size_t whole = plan_sparse(K, D, P, L, n).total, last = n > SPARSE_DIRECT ? plan_sparse(K, D, P, L, SPARSE_DIRECT).total : 0;
    return whole > last ? whole : last;
}

struct SearchPlan {
    bool sparse = false;         // without the distance matrix
    int64_t tile = 0;            // queries per pass
    int S = 0, nsplit = 1, n_lists = 0, merge_n = 0, merge_pow2 = 0;
    size_t bytes[WS_COUNT] = {};
    size_t total() const
    {
        size_t sum = 0;
        for (size_t b : bytes) sum += b;
        return sum;
    }
};

// Rows of the distance tile (and of the block minima) a pass over n queries may write: the sweep
// kernel works on whole tiles of GT query rows, the other two check every row.
int64_t dt_rows(int64_t n, int64_t K, int Dp)
{
    const int stages = Dp / DK;
    const bool sweep = n > 2 * SKQ && (stages == 6 || stages == 8) && K % GT == 0;   // (with enough tiles)
    return sweep ? (n + GT - 1) / GT * GT : n;
}

// per: points of a subregion on average; shared: whether several workgroups may divide what one wavefront would do (scratch for
// more partial lists; the results are the same); sparse: sparse_bytes() of such a pass where it goes without the distance matrix, in whose
// place that scratch is
SearchPlan plan_search(int64_t K, int D, int M, int P, int S, double per, int k, int64_t tile, bool rotated, bool shared = true, size_t sparse = 0)
{
    SearchPlan pl;
    pl.sparse = sparse > 0;
    pl.tile = tile;
    pl.S = S;
    // Workgroups per query in the scan: fill the chip when the batch is small, but with at most 8 per
    // query: every workgroup hands 4 k candidates to the final k-select, whose time grows with them
    // faster than the scan's shrinks (one query on the 100M-point workload, scan + k-select in us:
    // 17 + 9 with 2 workgroups, 12 + 9 with 4, 10.5 + 10 with 8, 10 + 12 / 14 / 20 with 16 / 32 / 64).
    // A wavefront takes up to 64 descriptors at a time, so that more than S / 256 workgroups divide what one wavefront would
    // do, each of them loading the table again.  That pays while the chip has wavefronts to spare, and the longer the
    // longer the lists are (scan + k-select in us with one for 16 descriptors against one for 256; 64 descriptors of 30
    // points, 64 queries 27 against 34, 333 40 against 36; of 120 points, 333 63 against 85, 1000 114 against 93; 256 of 30
    // points, 64 queries 33 against 37, 200 52 against 41; of 120, 64 61 against 81, 200 98 against 88; of 6, 200 35 against
    // 24), and where there are points for them, more where four wavefronts share them anyway and the k-select has more to do
    // (288 descriptors of 6, k = 100, one query 32 against 28; 520 of 3, k = 89, a search 63 against 58; 530 of 23, k = 94, five
    // queries 158 against 151).
    int nsplit = (int)((2048 + tile - 1) / tile);
    if (nsplit > 8) nsplit = 8;
    const int whole = (S + SCAN_WAVES * WAVE - 1) / (SCAN_WAVES * WAVE);
    int most = whole;
    if (shared && (double)tile * (S < WAVE ? WAVE : S) < 16384.0 + 200.0 * (per < 190.0 ? per : 190.0)) {
        const double by_points = (double)S * per / (640.0 * (whole > 1 ? 1.0 + k / 32.0 : 1.0));
        most = (S + 15) / 16;
        if (by_points < (double)most) most = by_points > (double)whole ? (int)by_points : whole;
    }
    if (nsplit > most) nsplit = most;
    while (nsplit > 1 && (int64_t)nsplit * SCAN_WAVES * k > 8192) --nsplit;
    if (nsplit < 1) nsplit = 1;
    pl.nsplit = nsplit;
    pl.n_lists = nsplit * SCAN_WAVES;
    pl.merge_n = pl.n_lists * k;
    pl.merge_pow2 = next_pow2(pl.merge_n);
    const int Dp = packed_dim(D);
    const size_t rows = (size_t)dt_rows(tile, K, Dp);
    const size_t tile_pad = (size_t)packed_rows(tile);   // the GEMM tiles copy whole tiles of packed rows
    const int64_t nb = (K + BMW - 1) / BMW;
    pl.bytes[WS_DT] = sparse ? sparse : rows * dt_stride(K) * sizeof(float);
    pl.bytes[WS_BM] = sparse ? 0 : rows * nb * sizeof(float);
    pl.bytes[WS_QN] = tile_pad * sizeof(float);
    pl.bytes[WS_QSI] = tile_pad * sizeof(float);
    pl.bytes[WS_QPK] = tile_pad * Dp * 2 * sizeof(_Float16);
    pl.bytes[WS_PID] = (size_t)tile * P * sizeof(int32_t);
    pl.bytes[WS_PD] = (size_t)tile * P * sizeof(float);
    pl.bytes[WS_DESC] = (size_t)tile * S * sizeof(SubDesc);
    pl.bytes[WS_LUT] = (size_t)tile * M * 256 * sizeof(float);
    pl.bytes[WS_PARTIAL] = (size_t)tile * pl.merge_n * sizeof(uint64_t);
    pl.bytes[WS_QROT] = rotated ? (size_t)tile * D * sizeof(float) : 0;
    return pl;
}

}  // namespace

struct ivf_index {
    int dev = 0;                 // the GPU it lies on
    int D = 0, M = 0, L = 0;
    int64_t K = 0, N = 0;
    float *centroids = nullptr, *cnorm = nullptr, *alpha = nullptr, *cst = nullptr;
    _Float16 *cpk = nullptr;     // centroids packed for the GEMM
    // for the search without the distance matrix (NULL: not built): fp16 rows and their lengths, start values and bounds of the
    // tiles, squared norms of the neighbours, the order of the regions, in one allocation
    _Float16 *chi = nullptr;
    float2 *clen = nullptr;
    float *mstart = nullptr, *nbr_norm = nullptr;
    float4 *mtile = nullptr;
    uint32_t *order = nullptr, *order_inv = nullptr;   // regions with common neighbours side by side (order.hpp)
    float *csi = nullptr;        // csi[0] inverse scale of the packed centroids; csi[1] reduction word
    float *codebook = nullptr, *const_table = nullptr;
    float *rot_t = nullptr;      // transposed rotation in front of the PQ, or NULL
    int32_t *nbr = nullptr, *ids = nullptr;
    uint4 *sub_info = nullptr;   // per subregion: block offset, first position, length
    uint8_t *blocks = nullptr;
    size_t chi_bytes = 0;        // of that allocation
    uint32_t hard = 0;           // of SPARSE_DIRECT centroids
    int64_t scratch_limit = 8ll << 30;
    size_t no_room = SIZE_MAX;   // scratch of the smallest pass without the distance matrix that there was no memory for
    Buf dt, bm, qn, qpk, qsi, probe_id, probe_d, desc, lut, partial, qrot;
    // optional per-stage timing with HIP events on the caller's stream
    bool profile = false;
    std::vector<hipEvent_t> ev[IVF_N_STAGES + 1];   // ev[s][i], ev[s+1][i] bracket stage s of pass i
    int64_t launches = 0;
};

extern "C" const char *ivf_last_error(void) { return g_err.c_str(); }

extern "C" int64_t ivf_num_kept(int nprobe, int L, float prune_frac)
{
    int64_t total = (int64_t)nprobe * L;
    int64_t S = (int64_t)std::ceil((double)prune_frac * (double)nprobe * (double)L);
    if (S < 1) S = 1;
    if (S > total) S = total;
    return S;
}

extern "C" void ivf_free_index(ivf_index *ix)
{
    if (!ix) return;
    (void)hipDeviceSynchronize();
    void *owned[] = {ix->centroids, ix->cnorm, ix->alpha, ix->cst, ix->codebook, ix->const_table,
                     ix->nbr, ix->ids, ix->sub_info, ix->blocks, ix->dt.p, ix->bm.p, ix->qn.p,
                     ix->cpk, ix->csi, ix->qpk.p, ix->qsi.p,
                     ix->probe_id.p, ix->probe_d.p, ix->desc.p, ix->lut.p, ix->partial.p, ix->qrot.p, ix->rot_t,
                     ix->chi};
    for (void *p : owned)
        if (p) (void)hipFree(p);
    for (auto &v : ix->ev)
        for (hipEvent_t e : v) (void)hipEventDestroy(e);
    g_pool.trim(ix->dev);
    delete ix;
}

extern "C" int ivf_set_scratch_limit(ivf_index *ix, int64_t bytes)
{
    if (!ix || bytes < 4096) return fail(IVF_EINVAL, "scratch limit must be at least 4096 bytes");
    ix->scratch_limit = bytes;
    ix->no_room = SIZE_MAX;
    return IVF_OK;
}

namespace {

inline unsigned grid_for(int64_t n, int block = 256) { return (unsigned)((n + block - 1) / block); }

// Stable sort of n (key, value) pairs by the low `bits` bits of the key, ascending: one
// least-significant-digit pass per 8 bits.  vals_in == NULL: the values are the positions 0..n-1.
// The sorted pairs end up in *keys_sorted / *vals_sorted, which point into the caller's two pairs
// of buffers (a: first, b: second; keys_in may be the a buffer).  hist: 256 * nblocks words,
// scan_tmp: temporary of rocprim's scan (scan_bytes).
struct RadixBufs {
    DevTmp ka, kb, va, vb, hist, base, scan;
    size_t scan_bytes = 0;
    int64_t nblocks = 0, cap = 0;
    int init(int64_t n)
    {
        cap = n;
        nblocks = (n + RS_TILE - 1) / RS_TILE;
        if (nblocks < 1) nblocks = 1;
        const size_t nb = (size_t)(n > 0 ? n : 1) * sizeof(uint32_t);
        HIPCHK(ka.alloc(nb));
        HIPCHK(kb.alloc(nb));
        HIPCHK(va.alloc(nb));
        HIPCHK(vb.alloc(nb));
        HIPCHK(hist.alloc((size_t)256 * nblocks * sizeof(uint32_t)));
        HIPCHK(base.alloc((size_t)256 * nblocks * sizeof(uint32_t)));
        HIPCHK(rocprim::exclusive_scan(nullptr, scan_bytes, static_cast<uint32_t *>(hist.p), static_cast<uint32_t *>(base.p),
                                       0u, (size_t)256 * nblocks, rocprim::plus<uint32_t>(), nullptr));
        HIPCHK(scan.alloc(scan_bytes ? scan_bytes : 16));
        return IVF_OK;
    }
    uint32_t *keys_a() { return static_cast<uint32_t *>(ka.p); }
    // Sorts the n keys held in the a buffer (values: positions, or the a value buffer when
    // have_vals).  Returns the buffers that hold the result.
    int sort(int64_t n, int bits, bool have_vals, uint32_t **keys_sorted, uint32_t **vals_sorted, hipStream_t st)
    {
        if (n > cap) return fail(IVF_EINVAL, "radix sort buffers too small");
        uint32_t *kin = static_cast<uint32_t *>(ka.p), *kout = static_cast<uint32_t *>(kb.p);
        uint32_t *vin = static_cast<uint32_t *>(va.p), *vout = static_cast<uint32_t *>(vb.p);
        const int64_t nbk = (n + RS_TILE - 1) / RS_TILE > 0 ? (n + RS_TILE - 1) / RS_TILE : 1;
        bool first = !have_vals;
        if (bits < 1) bits = 1;
        for (int shift = 0; shift < bits; shift += 8) {
            radix_hist_kernel<<<dim3((unsigned)nbk), dim3(RS_BLOCK), 0, st>>>(kin, n, shift, static_cast<uint32_t *>(hist.p), nbk);
            LAUNCHCHK("radix_hist_kernel");
            size_t sb = scan_bytes;
            HIPCHK(rocprim::exclusive_scan(scan.p, sb, static_cast<uint32_t *>(hist.p), static_cast<uint32_t *>(base.p), 0u,
                                           (size_t)256 * nbk, rocprim::plus<uint32_t>(), st));
            radix_scatter_kernel<<<dim3((unsigned)nbk), dim3(RS_BLOCK), 0, st>>>(
                kin, first ? nullptr : vin, n, shift, static_cast<uint32_t *>(base.p), nbk, kout, vout);
            LAUNCHCHK("radix_scatter_kernel");
            first = false;
            std::swap(kin, kout);
            std::swap(vin, vout);
        }
        *keys_sorted = kin;
        *vals_sorted = vin;
        return IVF_OK;
    }
};

int bits_for(int64_t nbuckets)
{
    int b = 1;
    while (b < 32 && (1ll << b) < nbuckets) ++b;
    return b;
}

// keys[r]: by which regions are sorted into the order of order.hpp; first: K words of scratch
int launch_region_keys(const int32_t *nbr, int64_t K, int L, uint32_t *first, uint32_t *keys, hipStream_t st)
{
    const dim3 grid((unsigned)((K * 16 + 255) / 256));
    shingle_kernel<true><<<grid, dim3(256), 0, st>>>(nbr, K, L, L, nullptr, first);
    LAUNCHCHK("shingle_kernel");
    shingle_kernel<false><<<grid, dim3(256), 0, st>>>(nbr, K, L, L < 16 ? L : 16, first, keys);
    LAUNCHCHK("shingle_kernel");
    return IVF_OK;
}

template <class T>
int dev_copy(T *&dst, const T *src, size_t count, hipStream_t st)
{
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&dst), count * sizeof(T) ? count * sizeof(T) : 16));
    if (count) HIPCHK(hipMemcpyAsync(dst, src, count * sizeof(T), hipMemcpyDeviceToDevice, st));
    return IVF_OK;
}

// Of SPARSE_DIRECT centroids of the index, as queries, those whose bound leaves too many blocks: with any of them small batches go with
// the matrix, with more than SPARSE_HARD all do.  A hard query costs exact block minima of a tile of queries over the whole table (one of
// them alone, K = 2^20, P = 16 254 us, with the matrix 133; in a batch of 64 272 and 207), in a large batch its share of the distance GEMM:
// 10 000, K = 2^20, P = 16, with 160 of the 256 7.57 ms, 210 11.4 - 11.8, all 14.6, with the matrix 10.7; none of them 3.1.
// Centroids as far from the origin as four times their spread are such, up to twice it they are not.
constexpr uint32_t SPARSE_HARD = 160;
int count_hard(const ivf_index *ix, hipStream_t st, uint32_t *hard);

// The tables of the search without the distance matrix, from the index's copies of centroids and neighbours
int load_sparse_tables(ivf_index *ix, hipStream_t st)
{
    const int64_t K = ix->K, nsub = K * ix->L, tiles = (K + GT - 1) / GT, pad = packed_rows(K);
    const int D = ix->D, L = ix->L, Dp = packed_dim(D);
    int rc;
    size_t total = 0;
    auto place = [&](auto *&p, size_t count) {                   // pieces of one allocation, which starts with chi
        p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(reinterpret_cast<unsigned char *>(ix->chi) + total);
        total += (count * sizeof(*p) + 255) / 256 * 256;
    };
    auto all = [&]() {
        total = ((size_t)pad * Dp * sizeof(_Float16) + 255) / 256 * 256;
        place(ix->clen, (size_t)pad);
        place(ix->mstart, (size_t)tiles * GT);
        place(ix->mtile, (size_t)tiles);
        place(ix->nbr_norm, (size_t)nsub);
        place(ix->order, (size_t)K);
        place(ix->order_inv, (size_t)K);
        return total;
    };
    ix->chi_bytes = all();
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->chi), ix->chi_bytes));
    (void)all();
    pack_hi_rows_kernel<<<dim3((unsigned)((pad + 15) / 16)), dim3(256), 0, st>>>(ix->centroids, K, pad, D, Dp,
                                                                                 reinterpret_cast<uint32_t *>(ix->csi + 1), ix->chi, ix->clen);
    LAUNCHCHK("pack_hi_rows_kernel");
    minima_tiles_kernel<<<dim3((unsigned)tiles), dim3(128), 0, st>>>(ix->clen, K, Dp, ix->mstart, ix->mtile);
    LAUNCHCHK("minima_tiles_kernel");
    neighbour_norm_kernel<<<dim3((unsigned)((nsub + 255) / 256)), dim3(256), 0, st>>>(ix->nbr, nsub, ix->cnorm, ix->nbr_norm);
    LAUNCHCHK("neighbour_norm_kernel");
    RadixBufs rb;
    StreamWait before_they_go(st);
    if ((rc = rb.init(K))) return rc;
    uint32_t *keys, *order;
    if ((rc = launch_region_keys(ix->nbr, K, L, ix->order_inv, rb.keys_a(), st))) return rc;
    if ((rc = rb.sort(K, SHINGLE_BITS, false, &keys, &order, st))) return rc;
    HIPCHK(hipMemcpyAsync(ix->order, order, (size_t)K * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
    inverse_kernel<<<dim3(grid_for(K)), dim3(256), 0, st>>>(ix->order, K, ix->order_inv);
    LAUNCHCHK("inverse_kernel");
    if ((rc = count_hard(ix, st, &ix->hard))) return rc;
    if (ix->hard <= SPARSE_HARD) return IVF_OK;
    HIPCHK(hipFree(ix->chi));
    ix->chi = nullptr;
    return IVF_OK;
}

int load_impl(const ivf_index_desc *d, hipStream_t st, ivf_index *ix)
{
    const int64_t K = d->K, N = d->N, nsub = K * d->L;
    const int D = d->D, M = d->M, L = d->L;
    ix->D = D; ix->M = M; ix->L = L; ix->K = K; ix->N = N;
    HIPCHK(hipGetDevice(&ix->dev));
    int rc;
    if ((rc = dev_copy(ix->centroids, d->centroids, (size_t)K * D, st))) return rc;
    if ((rc = dev_copy(ix->nbr, d->nbr, (size_t)nsub, st))) return rc;
    if ((rc = dev_copy(ix->alpha, d->alpha, (size_t)K, st))) return rc;
    if ((rc = dev_copy(ix->codebook, d->pq_codebook, (size_t)256 * D, st))) return rc;
    if ((rc = dev_copy(ix->const_table, d->const_table, (size_t)256, st))) return rc;
    if ((rc = dev_copy(ix->ids, d->ids, (size_t)N, st))) return rc;

    if (d->rotation) {
        HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->rot_t), (size_t)D * D * sizeof(float)));
        transpose_square_kernel<<<dim3((unsigned)((D * D + 255) / 256)), dim3(256), 0, st>>>(d->rotation, D, ix->rot_t);
        LAUNCHCHK("transpose_square_kernel");
    }
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->cnorm), (size_t)K * sizeof(float)));
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->cpk), (size_t)packed_rows(K) * packed_dim(D) * 2 * sizeof(_Float16)));
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->csi), 2 * sizeof(float)));
    if ((rc = pack_rows(ix->centroids, K, D, reinterpret_cast<uint32_t *>(ix->csi + 1), ix->cpk, ix->cnorm, ix->csi, st)))
        return rc;
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->cst), (size_t)nsub * sizeof(float)));
    cst_kernel<<<dim3((unsigned)((nsub + 255) / 256)), dim3(256), 0, st>>>(ix->alpha, d->cs_dist2, L, nsub, ix->cst);
    LAUNCHCHK("cst_kernel");

    // 64-bit check of the 32-bit block offsets: N*(M+1) bytes plus at most one block of padding each
    if (((uint64_t)N * (M + 1)) / BLK_ALIGN + (uint64_t)nsub >= (1ull << 32))
        return fail(IVF_EINVAL, "index too large for 32-bit block offsets");
    // block offsets: exclusive prefix sum of the block sizes
    DevTmp sz_mem, off_mem, scan_mem;
    StreamWait before_they_go(st);
    HIPCHK(sz_mem.alloc((size_t)nsub * sizeof(uint32_t)));
    HIPCHK(off_mem.alloc((size_t)nsub * sizeof(uint32_t)));
    uint32_t *sz = static_cast<uint32_t *>(sz_mem.p), *blk_off = static_cast<uint32_t *>(off_mem.p);
    blk_size_kernel<<<dim3((unsigned)((nsub + 255) / 256)), dim3(256), 0, st>>>(d->sub_offsets, nsub, M, sz);
    LAUNCHCHK("blk_size_kernel");
    size_t tmp_bytes = 0;
    HIPCHK(rocprim::exclusive_scan(nullptr, tmp_bytes, sz, blk_off, 0u, (size_t)nsub,
                                   rocprim::plus<uint32_t>(), st));
    HIPCHK(scan_mem.alloc(tmp_bytes ? tmp_bytes : 16));
    HIPCHK(rocprim::exclusive_scan(scan_mem.p, tmp_bytes, sz, blk_off, 0u, (size_t)nsub,
                                   rocprim::plus<uint32_t>(), st));
    uint32_t last_off = 0, last_sz = 0;
    HIPCHK(hipMemcpyAsync(&last_off, blk_off + nsub - 1, 4, hipMemcpyDeviceToHost, st));
    HIPCHK(hipMemcpyAsync(&last_sz, sz + nsub - 1, 4, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    const uint64_t total_blk = (uint64_t)last_off + last_sz;
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->blocks), (size_t)(total_blk ? total_blk : 1) * BLK_ALIGN));
    repack_kernel<<<dim3((unsigned)((nsub * 16 + 255) / 256)), dim3(256), 0, st>>>(
        d->sub_offsets, blk_off, nsub, M, d->codes, d->const_byte, ix->blocks);
    LAUNCHCHK("repack_kernel");
    HIPCHK(g_pool.fresh(reinterpret_cast<void **>(&ix->sub_info), (size_t)nsub * sizeof(uint4)));
    sub_info_kernel<<<dim3((unsigned)((nsub + 255) / 256)), dim3(256), 0, st>>>(d->sub_offsets, blk_off, nsub, ix->sub_info);
    LAUNCHCHK("sub_info_kernel");
    HIPCHK(hipStreamSynchronize(st));   // the temporaries are released on return
    return IVF_OK;
}

}  // namespace

extern "C" int ivf_load_index(const ivf_index_desc *d, void *hip_stream, ivf_index **out)
{
    int rc = check_trained(d);
    if (rc) return rc;
    if (!out) return fail(IVF_EINVAL, "out is NULL");
    if (!d->pq_codebook || !d->const_table || !d->sub_offsets || !d->codes || !d->const_byte || !d->ids)
        return fail(IVF_EINVAL, "pq_codebook or an encoded array (const_table, sub_offsets, codes, const_byte, ids) is NULL");
    if (d->N < 0 || d->N >= (1ll << 32)) return fail(IVF_EINVAL, "N=%lld out of range", (long long)d->N);
    if (!aligned16(d->codes)) return fail(IVF_EINVAL, "codes must be 16-byte aligned");
    ivf_index *ix = new (std::nothrow) ivf_index;
    if (!ix) return fail(IVF_ENOMEM, "host allocation failed");
    rc = load_impl(d, static_cast<hipStream_t>(hip_stream), ix);
    // last, and without the scratch of the rest: where there is no room for them searches go with the distance matrix
    if (!rc && sparse_table(ix->K, ix->D) && (rc = load_sparse_tables(ix, static_cast<hipStream_t>(hip_stream))) == IVF_ENOMEM) {
        if (ix->chi) (void)hipFree(ix->chi);
        ix->chi = nullptr;
        rc = IVF_OK;
    }
    if (rc) {
        std::string keep = g_err;
        ivf_free_index(ix);
        g_err = keep;
        return rc;
    }
    *out = ix;
    return IVF_OK;
}

namespace {

double mean_length(const ivf_index *ix) { return (double)ix->N / ((double)ix->K * ix->L); }

struct SearchArgs {
    const float *queries;
    int64_t nq;
    int P, k, S;
    int32_t *out_ids;
    float *out_dists;
    int32_t *probe_id_out;
    float *probe_d_out;
    int64_t *kept_sub_out;
    int64_t *n_scanned_out;
    int64_t budget;          // candidate budget R, 0 = none
    uint8_t *visited_out;    // [nq][S] flags of the budget mode (may be NULL)
};

int check_search_args(const ivf_index *ix, const float *queries, int64_t nq, int nprobe, float prune_frac, int k,
                      const int32_t *out_ids, const float *out_dists)
{
    if (!ix) return fail(IVF_EINVAL, "index is NULL");
    if (nq < 0 || nq >= (1ll << 31)) return fail(IVF_EINVAL, "nq=%lld out of range", (long long)nq);
    if (nq == 0) return IVF_OK;
    if (!queries || !out_ids || !out_dists) return fail(IVF_EINVAL, "queries / out_ids / out_dists is NULL");
    if (!aligned16(queries)) return fail(IVF_EINVAL, "queries must be 16-byte aligned");
    if (nprobe < 1 || nprobe > ix->K || nprobe > 4096)
        return fail(IVF_EINVAL, "nprobe=%d must be in [1, min(K, 4096)]", nprobe);
    if (!(prune_frac > 0.f) || prune_frac > 1.f) return fail(IVF_EINVAL, "prune_frac must be in (0, 1]");
    if (k < 1 || k > IVF_MAX_K_RESULTS) return fail(IVF_EINVAL, "k=%d must be in [1, %d]", k, IVF_MAX_K_RESULTS);
    const int64_t PL = (int64_t)nprobe * ix->L;
    if (PL > IVF_MAX_SCORES) return fail(IVF_EINVAL, "nprobe*L=%lld exceeds %d", (long long)PL, IVF_MAX_SCORES);
    return IVF_OK;
}

// Dynamic LDS sizes of the stage kernels; raises the kernels' limits where they exceed the default window.
struct LdsPlan { size_t scan, merge, sp, ssp; };   // ssp: the fused selection + scoring launch

// How the scoring of a search runs.  SCORE_STREAM_*: the whole row of distances through LDS, STREAM_512 / STREAM_1024 at a
// time; SCORE_GIVEN_*: the scores are there (search without the distance matrix); SCORE_FUSED: selection and scoring in one launch of 1024 threads a query (where the selection needs a workgroup
// of its own too); SCORE_GATHER: the rest.
enum ScoreMode { SCORE_GATHER, SCORE_FUSED, SCORE_STREAM_512, SCORE_STREAM_1024, SCORE_GIVEN_512, SCORE_GIVEN_1024 };
constexpr int STREAM_512 = 8192, STREAM_1024 = 16384;   // distances in LDS at a time (512 / 1024 threads)

// Rows are read where they are at most as many bytes as half the 128-byte lines that P L gathers touch, K <= 16 P L, with these
// exceptions (selection + scoring in us, rows against the rest):
//  - a batch that leaves compute units idle waits for one workgroup's parts, a longer chain than the gathers where the row is
//    long: K = 65 536, P L = 4096, 1 to 128 queries 67 - 92 against 64 - 87, 500 equal, 2000 220 against 251; K = 131 072,
//    P L = 12 800, 64 queries 84 against 81, 256 93 against 106; K = 262 144, P L = 16 384, 64 queries 116 against 95, 256 equal,
//    500 185 against 220; K = 32 768, P L = 4096, any number of queries: rows.
//  - a short row stays in the caches under its gathers, which 256 threads do with more queries at a time: 10 000 queries,
//    P L = 2048 and K = 1024 326 against 293, 4096 688 against 662, 8192 431 against 455; P L = 1024, K = 8192 396 against 369;
//    K = 4096, P L = 3072 745 against 726, 4096 772 against 790 (M = 16; with M = 8, K = 3324, P L = 3840, 2202 queries a search
//    takes 268 against 274).  Up to 500 queries rows are equal or 2 us better there.
ScoreMode score_mode(int64_t K, int P, int L, const SearchPlan &pl)
{
    const int64_t PL = (int64_t)P * L, nb = (K + BMW - 1) / BMW, nq = pl.tile;
    if (pl.sparse) return PL <= 4096 ? SCORE_GIVEN_512 : SCORE_GIVEN_1024;
    if (PL <= 4096 && K <= 16 * PL && (nq <= 512 ? K <= 12 * PL : K * PL >= (3ll << 22))) return SCORE_STREAM_512;
    if (PL > 4096 && PL <= 16384 && K <= 16 * PL && (K <= 8 * PL || nq >= 256)) return SCORE_STREAM_1024;
    if (P <= PS_P_MAX && nb <= PS_NB_MAX && PL > 4096) return SCORE_FUSED;
    return SCORE_GATHER;
}

int plan_lds(const ivf_index *ix, int P, int k, const SearchPlan &pl, LdsPlan &l)
{
    const int64_t PL = (int64_t)P * ix->L;
    const ScoreMode mode = score_mode(ix->K, P, ix->L, pl);
    l.scan = (size_t)SCAN_WAVES * pool_capacity(k) * sizeof(uint64_t);   // dynamic part: the pools
    l.merge = (size_t)pl.merge_pow2 * sizeof(uint64_t);
    l.sp = (size_t)((pl.sparse ? 2 * (int64_t)pl.S : PL) + 3 * P) * sizeof(uint32_t);
    if (l.sp < (size_t)ix->D * sizeof(float)) l.sp = (size_t)ix->D * sizeof(float);   // the table workgroups hold a query
    if (l.sp > 154 * 1024)   // one workgroup holds a query's scores in the 160 KB of LDS, beside 5 KB of static data
        return fail(IVF_EINVAL, "nprobe*L + 3*nprobe = %lld words exceed the LDS of one workgroup", (long long)(PL + 3 * P));
    if (mode == SCORE_STREAM_512 || mode == SCORE_STREAM_1024) {
        const int64_t part = mode == SCORE_STREAM_512 ? STREAM_512 : STREAM_1024;
        const size_t need = (size_t)((PL > part + 4 ? PL : part + 4) + 3 * P) * sizeof(uint32_t);
        if (l.sp < need) l.sp = need;
    }
    if (l.sp > 48 * 1024) {
        const void *fn = mode == SCORE_GIVEN_1024 ? reinterpret_cast<const void *>(&score_prune_kernel<1024, 4, -1>)
                         : mode == SCORE_STREAM_512 ? reinterpret_cast<const void *>(&score_prune_kernel<512, 2, STREAM_512>)
                         : mode == SCORE_STREAM_1024 ? reinterpret_cast<const void *>(&score_prune_kernel<1024, 4, STREAM_1024>)
                         : PL > 16384 ? reinterpret_cast<const void *>(&score_prune_kernel<1024, 8>)
                         : PL > 4096 ? reinterpret_cast<const void *>(&score_prune_kernel<1024, 4>)
                                     : reinterpret_cast<const void *>(&score_prune_kernel<256, 4>);
        HIPCHK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)l.sp));
    }
    {   // the fused launch needs what either half needs (see launch_probe_select for the selection's share)
        const size_t sel = ps_lds_bytes(P);
        l.ssp = sel > l.sp ? sel : l.sp;
        if (mode == SCORE_FUSED && l.ssp > 48 * 1024) {
            const void *fn = PL > 16384 ? reinterpret_cast<const void *>(&select_score_prune_kernel<8>)
                                        : reinterpret_cast<const void *>(&select_score_prune_kernel<4>);
            HIPCHK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)l.ssp));
        }
    }
    if (l.merge > 40 * 1024)
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&merge_kernel<256, 32>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)l.merge));
    if (l.scan > 32 * 1024) {   // dynamic + static LDS above the default 64 KB window
        const void *fn = ix->M == 16 ? reinterpret_cast<const void *>(&scan_kernel<16>)
                                     : reinterpret_cast<const void *>(&scan_kernel<8>);
        HIPCHK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)l.scan));
    }
    return IVF_OK;
}

// The first half of launch_sparse: the blocks that can hold one of a query's P closest, and the hard queries (a.total[0] of them).
int launch_flags(const ivf_index *ix, const float *Q, int64_t n, int P, const SearchWs &ws, const SparsePlan &sp, SparseArgs &a, hipStream_t st)
{
    const int64_t K = ix->K;
    const int D = ix->D, L = ix->L, Dp = packed_dim(D), nb = (int)((K + BMW - 1) / BMW);
    auto piece = [&](auto *&p, int i) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(ws.sparse() + sp.off[i]); };
    _Float16 *qh;
    float2 *qlen;
    piece(qh, SP_QH);
    piece(qlen, SP_QLEN);
    piece(a.best, SP_BEST);
    piece(a.n_flag, SP_FLAG);
    piece(a.blist, SP_LIST);
    piece(a.rank, SP_RANK);
    piece(a.thr, SP_THR);
    piece(a.count, SP_COUNT);
    piece(a.offset, SP_OFFSET);
    piece(a.hard, SP_HARD);
    piece(a.hard_rows, SP_HROWS);
    piece(a.hard_n, SP_HN);
    piece(a.hard_si, SP_HSI);
    piece(a.pairs, SP_PAIRS);
    piece(a.items, SP_ITEMS);
    piece(a.head, SP_HEAD);
    piece(a.cand, SP_BIG);
    piece(a.keys, SP_BIG);
    a.direct = sp.direct;
    a.region_count = sp.direct ? nullptr : a.count + N_XCD * nb;
    a.total = sp.direct ? a.count : a.region_count + N_XCD * K;
    a.K = K;
    a.half_ld = minima_half(K);
    a.nb = nb;
    a.P = P;
    a.L = L;
    a.cap = sp.cap;
    a.shift = sp.shift;
    a.Dp = Dp;
    a.tile = ix->mtile;
    a.qlen = qlen;
    a.qn = ws.qn;
    a.qsi = ws.qsi;
    a.cmax = reinterpret_cast<const uint32_t *>(ix->csi + 1);
    a.Qp = ws.qpk;
    a.Cp = ix->cpk;
    a.cnorm = ix->cnorm;
    a.csi = ix->csi;
    a.probe_id = nullptr;
    a.probe_d = nullptr;
    a.nbr = ix->nbr;
    a.nbr_norm = ix->nbr_norm;
    a.cst = ix->cst;
    a.alpha = ix->alpha;
    a.order_inv = ix->order_inv;

    const int64_t pad = packed_rows(n);
    const unsigned rows_grid = (unsigned)(pad / 4), zero_grid = (unsigned)((sp.count_words + 2047) / 2048);
    sparse_queries_kernel<<<dim3(rows_grid + zero_grid), dim3(256), 0, st>>>(Q, n, pad, D, Dp, a.cmax, ws.qpk, ws.qn, ws.qsi, qh, qlen, rows_grid,
                                                                            reinterpret_cast<unsigned long long *>(a.count), sp.count_words);
    LAUNCHCHK("sparse_queries_kernel");
    const bool wide = sweep_wide(n, K);
    const int per_q = wide ? 2 * GT : GT, tiles_q = (int)((n + per_q - 1) / per_q), tiles_c = (int)((K + GT - 1) / GT);
    int per_wg = 64;
    while (per_wg > 4 && group_grid(tiles_q, (tiles_c + per_wg - 1) / per_wg) < 1536) per_wg /= 2;
    const int64_t grid = group_grid(tiles_q, (tiles_c + per_wg - 1) / per_wg);
    if (grid >= (1ll << 24)) return fail(IVF_EINVAL, "coarse tile grid too large (more than 2^32 threads)");
    auto sweep = [&](auto few_kernel, auto wide_kernel) {
        (wide ? wide_kernel : few_kernel)<<<dim3((unsigned)grid), dim3(256), 0, st>>>(qh, ix->chi, ix->mstart, a.best, a.half_ld, tiles_q, tiles_c, per_wg);
    };
    if (Dp == 32) sweep(&coarse_minima_few_kernel<1>, &coarse_minima_kernel<1>);
    else if (Dp == 64) sweep(&coarse_minima_few_kernel<2>, &coarse_minima_kernel<2>);
    else if (Dp == 96) sweep(&coarse_minima_few_kernel<3>, &coarse_minima_kernel<3>);
    else sweep(&coarse_minima_few_kernel<4>, &coarse_minima_kernel<4>);
    LAUNCHCHK("coarse_minima_kernel");
    // pieces: at least 8 P of them (sparse_pays: the table has at least 8 P tiles), or 2048
    const dim3 gq((unsigned)n);
    static_assert(PS_NB_MAX <= 2 * 4 * 4 * 512, "four pieces of four tiles a thread, 512 threads");
    if (tiles_c <= 512) flag_blocks_kernel<256, 1, 2><<<gq, dim3(256), 0, st>>>(a);
    else if (tiles_c <= 2048) flag_blocks_kernel<256, 1, 8><<<gq, dim3(256), 0, st>>>(a);
    else if (tiles_c <= 4096) flag_blocks_kernel<512, 2, 4><<<gq, dim3(512), 0, st>>>(a);
    else flag_blocks_kernel<512, 4, 4><<<gq, dim3(512), 0, st>>>(a);
    LAUNCHCHK("flag_blocks_kernel");
    return IVF_OK;
}

// Stages 1 and 2 without the distance matrix: probes to pid and pd, the keys of the scores to ws.sparse() (SP_BIG).
template <class Mark>
int launch_sparse(ivf_index *ix, const float *Q, int64_t n, int P, const SearchWs &ws, int32_t *pid, float *pd, Mark mark, hipStream_t st)
{
    const int64_t K = ix->K;
    const int L = ix->L, Dp = packed_dim(ix->D), nb = (int)((K + BMW - 1) / BMW);
    const SparsePlan sp = plan_sparse(K, ix->D, P, L, n);
    SparseArgs a;
    int rc;
    if ((rc = launch_flags(ix, Q, n, P, ws, sp, a, st))) return rc;
    a.probe_id = pid;
    a.probe_d = pd;
    const bool wide = nb > 4096;                                // (16 blocks a thread at most)
    hard_minima_kernel<<<dim3(1024), dim3(256), 0, st>>>(a);
    LAUNCHCHK("hard_minima_kernel");
    if (wide) hard_flag_kernel<1024><<<dim3(512), dim3(1024), 0, st>>>(a);
    else hard_flag_kernel<256><<<dim3(1024), dim3(256), 0, st>>>(a);
    LAUNCHCHK("hard_flag_kernel");
    auto grouped = [&](uint32_t *count, int64_t buckets, uint32_t *total, const int32_t *bucket, int width, const uint32_t *n_flag,
                       const uint32_t *order, const uint32_t *inv) -> int {
        bucket_items_kernel<<<dim3((unsigned)((buckets + 1023) / 1024)), dim3(1024), 0, st>>>(count, buckets, total, a.offset, order, a.items);
        LAUNCHCHK("bucket_items_kernel");
        place_pairs_kernel<<<dim3((unsigned)((n * width + 255) / 256)), dim3(256), 0, st>>>(bucket, a.rank, n, width, buckets, sp.cap, sp.shift, n_flag, inv, a.offset, a.pairs);
        LAUNCHCHK("place_pairs_kernel");
        return IVF_OK;
    };
    if (!sp.direct && (rc = grouped(a.count, nb, a.total + 1, a.blist, sp.cap, a.n_flag, nullptr, nullptr))) return rc;
    const int chunks = (L + BMW - 1) / BMW;
    auto pairs = [&](auto region, int64_t items, const uint32_t *total) -> int {
        constexpr bool REGION = decltype(region)::value;
        const int c = REGION ? chunks : 1;
        const int64_t each = items * c / 3072;                   // (1536 workgroups run at a time)
        const int run = each < 1 ? 1 : each < PAIR_RUN ? (int)each : PAIR_RUN;
        auto kernel = [&](auto whole) {
            constexpr bool W = decltype(whole)::value;
            return Dp == 32 ? &pair_distance_kernel<2, REGION, W> : Dp == 64 ? &pair_distance_kernel<4, REGION, W> : Dp == 96 ? &pair_distance_kernel<6, REGION, W> : &pair_distance_kernel<8, REGION, W>;
        };
        (!REGION || L % BMW == 0 ? kernel(std::true_type()) : kernel(std::bool_constant<!REGION>()))<<<dim3(pair_grid(items, c, run)), dim3(64), 0, st>>>(a, total, c, run);
        LAUNCHCHK("pair_distance_kernel");
        return IVF_OK;
    };
    if ((rc = pairs(std::false_type(), sp.block_items, a.total + 2))) return rc;
    if ((rc = mark(1))) return rc;
    static_assert(2 * PICK_BLOCK >= 2 * PS_P_MAX, "two of a query's blocks a thread");
    probe_pick_kernel<<<dim3((unsigned)n), dim3(PICK_BLOCK), 2 * PICK_CAP * sizeof(uint32_t), st>>>(a);
    LAUNCHCHK("probe_pick_kernel");
    if ((rc = mark(2))) return rc;
    if (!sp.direct && (rc = grouped(a.region_count, K, a.total + 3, pid, P, nullptr, ix->order, ix->order_inv))) return rc;
    if ((rc = pairs(std::true_type(), sp.region_items, a.total + 4))) return rc;
    return IVF_OK;
}

// Of SPARSE_DIRECT centroids of the index, as queries for 16 regions: those whose bound leaves too many blocks
int count_hard(const ivf_index *ix, hipStream_t st, uint32_t *hard)
{
    const int64_t n = SPARSE_DIRECT, pad = packed_rows(n);
    const int D = ix->D, P = 16;
    const SparsePlan sp = plan_sparse(ix->K, D, P, ix->L, n);
    DevTmp rows, packed, norm, scale, mem;
    StreamWait before_they_go(st);
    HIPCHK(rows.alloc((size_t)n * D * sizeof(float)));
    HIPCHK(packed.alloc((size_t)pad * packed_dim(D) * 2 * sizeof(_Float16)));
    HIPCHK(norm.alloc((size_t)pad * sizeof(float)));
    HIPCHK(scale.alloc((size_t)pad * sizeof(float)));
    HIPCHK(mem.alloc(sp.total));
    SearchWs ws;
    ws.dt = static_cast<float *>(mem.p);
    ws.qn = static_cast<float *>(norm.p);
    ws.qsi = static_cast<float *>(scale.p);
    ws.qpk = static_cast<_Float16 *>(packed.p);
    const size_t row = (size_t)D * sizeof(float);
    HIPCHK(hipMemcpy2DAsync(rows.p, row, ix->centroids, (size_t)(ix->K / n) * row, row, (size_t)n, hipMemcpyDeviceToDevice, st));
    SparseArgs a;
    int rc;
    if ((rc = launch_flags(ix, static_cast<const float *>(rows.p), n, P, ws, sp, a, st))) return rc;
    HIPCHK(hipMemcpyAsync(hard, a.total, sizeof(*hard), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    return IVF_OK;
}

std::atomic<int64_t> g_passes_sparse{0}, g_passes_matrix{0};

// The launch sequence of the query path over the batch, `pl.tile` queries per pass, on scratch the
// caller provides.  Allocates nothing (stage timing, which creates events, is the allocating
// entry points' option: `timed`).
int run_search(ivf_index *ix, const SearchArgs &a, const SearchPlan &pl, const LdsPlan &lds, const SearchWs &ws,
               bool timed, hipStream_t st)
{
    const int P = a.P, L = ix->L, M = ix->M, D = ix->D, S = a.S, k = a.k;
    const int64_t K = ix->K, PL = (int64_t)P * L;
    const int Dp = packed_dim(D);
    int rc;
    for (int64_t q0 = 0; q0 < a.nq; q0 += pl.tile) {
        const int64_t n = (a.nq - q0 < pl.tile) ? a.nq - q0 : pl.tile;
        const float *Q = a.queries + q0 * D;
        int32_t *pid = a.probe_id_out ? a.probe_id_out + q0 * P : ws.probe_id;
        float *pd = a.probe_d_out ? a.probe_d_out + q0 * P : ws.probe_d;

        auto mark = [&](int stage) -> int {
            if (!timed) return IVF_OK;
            hipEvent_t e;
            HIPCHK(hipEventCreate(&e));
            HIPCHK(hipEventRecord(e, st));
            ix->ev[stage].push_back(e);
            return IVF_OK;
        };
        if ((rc = mark(0))) return rc;
        (pl.sparse ? g_passes_sparse : g_passes_matrix)++;
        if (pl.sparse) {
            if ((rc = launch_sparse(ix, Q, n, P, ws, pid, pd, mark, st))) return rc;
        } else if ((rc = pack_rows(Q, n, D, nullptr, ws.qpk, ws.qn, ws.qsi, st))) {
            return rc;
        } else if ((rc = launch_coarse(ws.qpk, ws.qn, ws.qsi, n, ix->cpk, ix->cnorm, ix->csi, K, Dp, ws.dt, ws.bm, st))) return rc;
        if (!pl.sparse && (rc = mark(1))) return rc;
        // Where both are workgroups of 1024 threads with their keys in LDS, the selection runs inside the
        // scoring launch (one workgroup per query does both): one kernel boundary less, and the selection
        // of one query (LDS and ALU work) runs while the other workgroup of the CU waits for its gathers.
        const int nb = (int)((K + BMW - 1) / BMW);
        const ScoreMode mode = score_mode(K, P, L, pl);
        const bool fused = mode == SCORE_FUSED;
        if (!fused && !pl.sparse && (rc = launch_probe_select(ws.dt, ws.bm, n, K, P, pid, pd, st))) return rc;
        if (!pl.sparse && (rc = mark(2))) return rc;

        int64_t *ks = a.kept_sub_out ? a.kept_sub_out + q0 * S : nullptr;
        int64_t *ns = a.n_scanned_out ? a.n_scanned_out + q0 : nullptr;
        const float *Qt = Q;                                   // what the lookup tables are built from
        if (ix->rot_t) {
            rotate_rows_kernel<<<dim3((unsigned)((n + ROT_ROWS - 1) / ROT_ROWS)), dim3(256), (size_t)ROT_ROWS * D * sizeof(float), st>>>(
                Q, n, D, ix->rot_t, ws.qrot);
            LAUNCHCHK("rotate_rows_kernel");
            Qt = ws.qrot;
        }
        // stages 2-3 (one workgroup per query) and stage 4 (one more for every lut_per queries) in one launch
#define IVF_SP_LAUNCH(BLK, ...)                                                                                    \
    score_prune_kernel<BLK, __VA_ARGS__><<<dim3(lut_grid(n, lut_per)), dim3(BLK), lds.sp, st>>>(                                \
        ws.dt, dt_stride(K), K, pid, pd, P, L, ix->nbr, ix->cst, ix->alpha, S, ix->sub_info, ws.desc, ks, ns, n, Qt, \
        D, M, ix->codebook, ws.lut, lut_per)
#define IVF_SSP_LAUNCH(MV)                                                                                          \
    select_score_prune_kernel<MV><<<dim3(lut_grid(n, lut_per)), dim3(1024), lds.ssp, st>>>(                             \
        ws.dt, dt_stride(K), ws.bm, K, nb, pid, pd, P, L, ix->nbr, ix->cst, ix->alpha, S, ix->sub_info, ws.desc, ks, ns, \
        n, Qt, D, M, ix->codebook, ws.lut, lut_per)
        const int lut_per = lut_queries(n, D, lds.sp);
        if (pl.sparse) {
            const uint32_t *given = reinterpret_cast<const uint32_t *>(ws.sparse() + plan_sparse(K, D, P, L, n).off[SP_BIG]);
            auto prune = [&](auto kernel, int block) {
                kernel<<<dim3(lut_grid(n, lut_per)), dim3(block), lds.sp, st>>>(reinterpret_cast<const float *>(given), PL, K, pid, pd, P, L, ix->nbr,
                    ix->cst, ix->alpha, S, ix->sub_info, ws.desc, ks, ns, n, Qt, D, M, ix->codebook, ws.lut, lut_per);
            };
            if (mode == SCORE_GIVEN_512) prune(&score_prune_kernel<512, 2, -1>, 512);
            else prune(&score_prune_kernel<1024, 4, -1>, 1024);
        } else if (fused && PL > 16384) IVF_SSP_LAUNCH(8);
        else if (fused) IVF_SSP_LAUNCH(4);
        else if (mode == SCORE_STREAM_512) IVF_SP_LAUNCH(512, 2, STREAM_512);
        else if (mode == SCORE_STREAM_1024) IVF_SP_LAUNCH(1024, 4, STREAM_1024);
        else if (PL > 16384) IVF_SP_LAUNCH(1024, 8);
        else if (PL > 4096) IVF_SP_LAUNCH(1024, 4);
        else IVF_SP_LAUNCH(256, 4);
#undef IVF_SP_LAUNCH
#undef IVF_SSP_LAUNCH
        LAUNCHCHK("score_prune_kernel");
        if (a.budget > 0) {
            const uint32_t R = a.budget > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)a.budget;
            auto cut = [&](auto kernel) {
                kernel<<<dim3((unsigned)n), dim3(BUDGET_BLOCK), 0, st>>>(ws.desc, S, R, a.visited_out ? a.visited_out + q0 * S : nullptr, ns);
            };
            static_assert(IVF_MAX_SCORES <= 32 * BUDGET_BLOCK, "items of a thread");
            if (S <= 4 * BUDGET_BLOCK) cut(&budget_cut_kernel<4>);
            else if (S <= 8 * BUDGET_BLOCK) cut(&budget_cut_kernel<8>);
            else if (S <= 16 * BUDGET_BLOCK) cut(&budget_cut_kernel<16>);
            else cut(&budget_cut_kernel<32>);
            LAUNCHCHK("budget_cut_kernel");
        }
        if ((rc = mark(3))) return rc;
        if ((rc = mark(4))) return rc;   // (the lookup tables are built inside the launch above)

        if (M == 16)
            scan_kernel<16><<<dim3((unsigned)(n * pl.nsplit)), dim3(SCAN_BLOCK), lds.scan, st>>>(
                ix->blocks, ix->const_table, ws.desc, S, ws.lut, k, pl.nsplit, ws.partial);
        else
            scan_kernel<8><<<dim3((unsigned)(n * pl.nsplit)), dim3(SCAN_BLOCK), lds.scan, st>>>(
                ix->blocks, ix->const_table, ws.desc, S, ws.lut, k, pl.nsplit, ws.partial);
        LAUNCHCHK("scan_kernel");
        if ((rc = mark(5))) return rc;

        auto merge = [&](auto kernel) {
            kernel<<<dim3((unsigned)n), dim3(256), lds.merge, st>>>(ws.partial, ix->ids, pl.merge_n, k, a.out_ids + q0 * k, a.out_dists + q0 * k);
        };
        if (pl.merge_n <= 4 * 256) merge(&merge_kernel<256, 4>);
        else if (pl.merge_n <= 16 * 256) merge(&merge_kernel<256, 16>);
        else merge(&merge_kernel<256, 32>);
        LAUNCHCHK("merge_kernel");
        if ((rc = mark(6))) return rc;
        if (timed) ix->launches++;
    }
    return IVF_OK;
}

// Scratch for callers that must not allocate: one array per GPU, part of the loaded code object,
// so it exists from the moment the library is loaded until the process ends.  Host code never uses
// the array's name as an address; it asks the runtime for the array's device address once per
// device and keeps that.
static __device__ __align__(256) unsigned char scratch[IVF_NOALLOC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_ptr[MAX_DEVICES] = {};

// Device address of this GPU's copy of `scratch` (the current device).
int scratch_of_current_device(unsigned char **out)
{
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(IVF_EINVAL, "device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(IVF_EHIP, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[dev] = static_cast<unsigned char *>(p);
    }
    *out = g_scratch_ptr[dev];
    return IVF_OK;
}

// Whether a pass of nq queries goes without the distance matrix (sparse.hpp).  What it saves grows with nq K, what it costs with
// nq P, with the 64 neighbours at a time of every region and with the launches.  A search in us, with / without, L = 64, D = 96: K = 2^20, P = 256,
// 2048 queries 3390 / 2040, 10 000 14 490 / 6500; P = 16, 10 000 11 260 / 3530; K = 262 144, P = 256, 512 409 / 437, 1024 738 / 669, 10 000 6290 / 3000;
// P = 64, 512 318 / 247, 4096 1890 / 855; K = 65 536, P = 64, 512 153 / 169, 1024 241 / 228, 4096 726 / 502; P = 16, 512 96 / 109, 1024 158 / 148,
// 2048 295 / 232; K = 32 768, P = 16, 1024 137 / 182, 4096 454 / 424; D = 128, where the sweep has two wavefronts a SIMD, K = 65 536, P = 16, 2048 331 / 265,
// P = 64, 10 000 1703 / 1095 (neighbours that regions of a group of 1024 have in common; neighbours anywhere in the table cost the way
// without the matrix up to a fifth more).
// With more than 64 neighbours the difference grows: a group of 2 L regions / neighbours anywhere, without over with: K = 65 536, P = 16,
// L = 128 2048 queries .72 / .91; L = 256 2048 .90 / 1.20, 4096 .81 / 1.09, 10 000 .68 / .87; L = 512 4096 1.13 / 1.57, 10 000 .91 / 1.21; L = 1024 2048
// 1.68 / 2.43, 10 000 1.16 / 1.57; K = 262 144, P = 64, L = 128 2048 .67 / .99, L = 256 2048 .85 / 1.41, 4096 .73 / 1.17, 10 000 .57 / .84; P = 128,
// L = 128 2048 .79 / 1.22, 4096 .63 / .93; P = 16, L = 512 2048 .71 / 1.10, 4096 .67 / 1.03.  The line lies where neighbours anywhere lose nothing.
// Up to SPARSE_DIRECT queries, in us: half the table's bytes instead of all of them, the matrix (0.9 10^-6 a distance written and read)
// and one workgroup's selection (less of it for few probes) are saved, the launches of seven small kernels and 24 KB for every 64 rows of a pair are spent.  With /
// without: K = 2^20, P = 16, 1 query 134 / 93, 64 199 / 111, 128 308 / 130, 256 387 / 176; P = 128, 1 151 / 102, 64 224 / 193, 256 445 / 410 (L = 128 472 / 544);
// P = 250, 1 170 / 110, 32 213 / 198, 64 252 / 260, 256 498 / 655; K = 262 144, P = 2, 1 58 / 60, 64 70 / 64, 256 120 / 78; P = 16, 1 70 / 69, 64 88 / 79, 256 140 / 114
// (L = 256 176 / 159, L = 512 208 / 226); P = 64, 1 81 / 73, 64 104 / 104, 128 119 / 139; P = 250, 1 98 / 83, 32 123 / 146; K = 65 536, P = 2,
// 256 55 / 64; P = 16, 1 50 / 55, 64 63 / 68, 256 69 / 96; P = 64, 1 63 / 60, 32 76 / 78.
bool sparse_pays(int64_t K, int D, int P, int L, int64_t nq)
{
    if (K < 1024 * (int64_t)P) return false;
    const int64_t chunks = (L + BMW - 1) / BMW;
    if (nq <= SPARSE_DIRECT) {
        const double wide = packed_dim(D) / 96.0, fixed = 17.0 - 5.0 / 16.0 * (P < 16 ? P : 16);
        return (0.9 * (double)nq + 50.0 * wide) * 1e-6 * (double)K + 0.05 * P > fixed + (0.0055 + 0.0023 * (double)chunks) * wide * (double)nq * P;
    }
    const int64_t pairs = (int64_t)P * (chunks > 2 ? chunks * chunks / 2 : chunks) << (packed_dim(D) <= 96 ? 22 : 23);
    return nq * K >= (pairs > (1ll << 27) ? pairs : 1ll << 27);
}

// Plan of a pass of n queries without the distance matrix
SearchPlan plan_without_matrix(const ivf_index *ix, int P, int S, int k, int64_t n)
{
    return plan_search(ix->K, ix->D, ix->M, P, S, mean_length(ix), k, n, ix->rot_t != nullptr, true, sparse_bytes(ix->K, ix->D, P, ix->L, n));
}

// Queries of a pass without the distance matrix; 0: with it, `tile` of them.  Its own scratch keeps to the limit that the matrix would
// keep to, and a pass of more queries than that keeps to it with everything that grows with them (descriptors, tables, lists).
int64_t sparse_tile(const ivf_index *ix, int P, int S, int k, int64_t nq, int64_t tile)
{
    if (!ix->chi || P > PS_P_MAX || (int64_t)P * ix->L > 16384) return 0;
    auto fits = [&](int64_t n) {
        const SearchPlan pl = plan_without_matrix(ix, P, S, k, n);
        return (n <= tile ? pl.bytes[WS_DT] : pl.total()) <= (size_t)ix->scratch_limit && pl.total() < ix->no_room;
    };
    auto pays = [&](int64_t n) { return (n > SPARSE_DIRECT || ix->hard == 0) && sparse_pays(ix->K, ix->D, P, ix->L, n); };
    int64_t n = nq < (1 << 20) ? nq : (1 << 20);
    while (pays(n) && !fits(n)) {
        if (n <= 128) return 0;
        n = (n / 2 + 127) & ~127ll;
    }
    return pays(n) ? n : 0;
}

// Whether `bytes` of scratch find room once the tables of the search without the distance matrix have gone
bool room_without_tables(const ivf_index *ix, size_t bytes)
{
    size_t left = 0, all = 0;
    return ix->chi && hipMemGetInfo(&left, &all) == hipSuccess && left + ix->chi_bytes >= bytes;
}

// The query path on the handle's own growable scratch (allocates when a call needs more than any before).
int search_alloc(ivf_index *ix, const float *queries, int64_t nq, int nprobe, float prune_frac, int k,
                 int32_t *out_ids, float *out_dists, int32_t *probe_id_out, float *probe_d_out,
                 int64_t *kept_sub_out, int64_t *n_scanned_out, int64_t budget, uint8_t *visited_out,
                 void *hip_stream)
{
    int rc = check_search_args(ix, queries, nq, nprobe, prune_frac, k, out_ids, out_dists);
    if (rc || nq == 0) return rc;
    const int64_t K = ix->K;
    const int S = (int)ivf_num_kept(nprobe, ix->L, prune_frac);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);

    // queries per pass: bounded by the distance tile
    int64_t tile = ix->scratch_limit / (K * (int64_t)sizeof(float));
    if (tile < 1) tile = 1;
    if (tile >= nq) tile = nq;
    else if (tile >= 256) tile -= tile % 256;   // whole blocks of the padded row count
    else if (tile >= GT) tile -= tile % GT;

    // Where memory is short, smaller passes without the matrix, then with it, then with it and without the tables of the other way
    SearchPlan pl;
    Buf *bufs[WS_COUNT] = {&ix->dt, &ix->bm, &ix->qn, &ix->qsi, &ix->qpk, &ix->probe_id, &ix->probe_d,
                           &ix->desc, &ix->lut, &ix->partial, &ix->qrot};
    while (true) {
        const int64_t n = sparse_tile(ix, nprobe, S, k, nq, tile);
        pl = n > 0 ? plan_without_matrix(ix, nprobe, S, k, n) : plan_search(K, ix->D, ix->M, nprobe, S, mean_length(ix), k, tile, ix->rot_t != nullptr);
        for (int i = 0; i < WS_COUNT && !rc; ++i) rc = ensure(*bufs[i], pl.bytes[i]);
        if (rc != IVF_ENOMEM) break;
        HIPCHK(hipDeviceSynchronize());
        for (Buf *b : bufs) {
            if (b->p) HIPCHK(hipFree(b->p));
            *b = Buf();
        }
        if (n > 0) {
            ix->no_room = pl.total();
        } else if (room_without_tables(ix, pl.total())) {
            HIPCHK(hipFree(ix->chi));
            ix->chi = nullptr;
        } else {
            break;
        }
        rc = IVF_OK;
    }
    if (rc) return rc;
    SearchWs ws;
    ws.dt = static_cast<float *>(ix->dt.p);
    ws.bm = static_cast<float *>(ix->bm.p);
    ws.qn = static_cast<float *>(ix->qn.p);
    ws.qsi = static_cast<float *>(ix->qsi.p);
    ws.qpk = static_cast<_Float16 *>(ix->qpk.p);
    ws.probe_id = static_cast<int32_t *>(ix->probe_id.p);
    ws.probe_d = static_cast<float *>(ix->probe_d.p);
    ws.desc = static_cast<SubDesc *>(ix->desc.p);
    ws.lut = static_cast<float *>(ix->lut.p);
    ws.partial = static_cast<uint64_t *>(ix->partial.p);
    ws.qrot = static_cast<float *>(ix->qrot.p);
    LdsPlan lds;
    if ((rc = plan_lds(ix, nprobe, k, pl, lds))) return rc;
    const SearchArgs a = {queries, nq, nprobe, k, S, out_ids, out_dists, probe_id_out, probe_d_out, kept_sub_out,
                          n_scanned_out, budget, visited_out};
    return run_search(ix, a, pl, lds, ws, ix->profile, st);
}

}  // namespace

extern "C" int ivf_search_stages(ivf_index *ix, const float *queries, int64_t nq, int nprobe,
                                 float prune_frac, int k, int32_t *out_ids, float *out_dists,
                                 int32_t *probe_id_out, float *probe_d_out, int64_t *kept_sub_out,
                                 int64_t *n_scanned_out, void *hip_stream)
{
    return search_alloc(ix, queries, nq, nprobe, prune_frac, k, out_ids, out_dists, probe_id_out, probe_d_out,
                        kept_sub_out, n_scanned_out, 0, nullptr, hip_stream);
}

extern "C" void ivf_search_stats(int64_t *out)
{
    out[0] = g_passes_sparse;
    out[1] = g_passes_matrix;
}

extern "C" int ivf_search_budget(ivf_index *ix, const float *queries, int64_t nq, int nprobe, float prune_frac,
                                 int64_t max_candidates, int k, int32_t *out_ids, float *out_dists,
                                 int64_t *kept_sub_out, uint8_t *visited_out, int64_t *n_scanned_out,
                                 void *hip_stream)
{
    if (max_candidates < 1) return fail(IVF_EINVAL, "max_candidates=%lld must be positive", (long long)max_candidates);
    return search_alloc(ix, queries, nq, nprobe, prune_frac, k, out_ids, out_dists, nullptr, nullptr,
                        kept_sub_out, n_scanned_out, max_candidates, visited_out, hip_stream);
}

extern "C" int ivf_search_noalloc(ivf_index *ix, const float *queries, int64_t nq, int nprobe, float prune_frac,
                                  int k, int32_t *out_ids, float *out_dists, void *hip_stream)
{
    int rc = check_search_args(ix, queries, nq, nprobe, prune_frac, k, out_ids, out_dists);
    if (rc || nq == 0) return rc;
    const int S = (int)ivf_num_kept(nprobe, ix->L, prune_frac);
    // the whole batch in one pass: the scratch is carved out of the static array, 256-byte aligned pieces
    SearchPlan pl;
    size_t off[WS_COUNT], total = 0;
    for (bool shared : {true, false}) {
        pl = plan_search(ix->K, ix->D, ix->M, nprobe, S, mean_length(ix), k, nq, ix->rot_t != nullptr, shared);
        total = 0;
        for (int i = 0; i < WS_COUNT; ++i) {
            off[i] = total;
            total += (pl.bytes[i] + 255) / 256 * 256;
        }
        if (total <= (size_t)IVF_NOALLOC_SCRATCH_BYTES) break;
    }
    if (total > (size_t)IVF_NOALLOC_SCRATCH_BYTES)
        return fail(IVF_EINVAL, "ivf_search_noalloc: this batch needs %zu bytes of scratch, the static array holds %zu "
                    "(nq=%lld, K=%lld); use fewer queries per call or ivf_search",
                    total, (size_t)IVF_NOALLOC_SCRATCH_BYTES, (long long)nq, (long long)ix->K);
    unsigned char *base = nullptr;
    if ((rc = scratch_of_current_device(&base))) return rc;
    SearchWs ws;
    ws.dt = reinterpret_cast<float *>(base + off[WS_DT]);
    ws.bm = reinterpret_cast<float *>(base + off[WS_BM]);
    ws.qn = reinterpret_cast<float *>(base + off[WS_QN]);
    ws.qsi = reinterpret_cast<float *>(base + off[WS_QSI]);
    ws.qpk = reinterpret_cast<_Float16 *>(base + off[WS_QPK]);
    ws.probe_id = reinterpret_cast<int32_t *>(base + off[WS_PID]);
    ws.probe_d = reinterpret_cast<float *>(base + off[WS_PD]);
    ws.desc = reinterpret_cast<SubDesc *>(base + off[WS_DESC]);
    ws.lut = reinterpret_cast<float *>(base + off[WS_LUT]);
    ws.partial = reinterpret_cast<uint64_t *>(base + off[WS_PARTIAL]);
    ws.qrot = reinterpret_cast<float *>(base + off[WS_QROT]);
    LdsPlan lds;
    if ((rc = plan_lds(ix, nprobe, k, pl, lds))) return rc;
    const SearchArgs a = {queries, nq, nprobe, k, S, out_ids, out_dists, nullptr, nullptr, nullptr, nullptr, 0, nullptr};
    return run_search(ix, a, pl, lds, ws, false, static_cast<hipStream_t>(hip_stream));
}

extern "C" int ivf_profile_enable(ivf_index *ix, int on)
{
    if (!ix) return fail(IVF_EINVAL, "index is NULL");
    ix->profile = on != 0;
    return IVF_OK;
}

extern "C" int ivf_profile_read(ivf_index *ix, double *stage_ms, int64_t *launches)
{
    if (!ix || !stage_ms || !launches) return fail(IVF_EINVAL, "NULL argument");
    HIPCHK(hipDeviceSynchronize());
    for (int s = 0; s < IVF_N_STAGES; ++s) {
        double tot = 0.0;
        for (size_t i = 0; i < ix->ev[s].size() && i < ix->ev[s + 1].size(); ++i) {
            float ms = 0.f;
            HIPCHK(hipEventElapsedTime(&ms, ix->ev[s][i], ix->ev[s + 1][i]));
            tot += ms;
        }
        stage_ms[s] = tot;
    }
    *launches = ix->launches;
    for (int s = 0; s <= IVF_N_STAGES; ++s) {
        for (hipEvent_t e : ix->ev[s]) (void)hipEventDestroy(e);
        ix->ev[s].clear();
    }
    ix->launches = 0;
    return IVF_OK;
}

extern "C" int ivf_search(ivf_index *ix, const float *queries, int64_t nq, int nprobe, float prune_frac,
                          int k, int32_t *out_ids, float *out_dists, void *hip_stream)
{
    return ivf_search_stages(ix, queries, nq, nprobe, prune_frac, k, out_ids, out_dists, nullptr,
                             nullptr, nullptr, nullptr, hip_stream);
}

namespace {

std::atomic<int64_t> g_assign_short{0}, g_assign_exact{0};

// Rows as fp16 with their lengths, for packed_rows(n) rows (see pack_hi_rows_kernel).
int launch_pack_hi(const float *X, int64_t n, int D, uint32_t *gmax, _Float16 *H, float2 *len, hipStream_t st)
{
    int rc = launch_absmax<true>(X, n * D, gmax, st);
    if (rc) return rc;
    const int64_t pad = packed_rows(n);
    pack_hi_rows_kernel<<<dim3((unsigned)((pad + 15) / 16)), dim3(256), 0, st>>>(X, n, pad, D, packed_dim(D), gmax, H, len);
    LAUNCHCHK("pack_hi_rows_kernel");
    return IVF_OK;
}

// Nearest-centroid assignment (P = 1) with buffers that live across calls: the packed centroid
// table and the per-chunk query scratch.  No distance tile: the minimum is fused into the GEMM.
//
// Two passes: the hi halves of the operands alone (a third of the MFMA work) give every row a short
// list of centroids that may be its nearest, with a proven error bound (coarse_shortlist_kernel), and
// the exact distances of the listed pairs decide (rerank_kernel).  A chunk whose list overflows (rows
// with very many centroids at nearly the same distance) is redone by the exact kernel, whose operands
// are packed only then.
struct ArgminCtx {
    int64_t K = 0, chunk = 0;
    int D = 0, Dp = 0;
    DevTmp cn, csi, cpk, xn, xsi, xpk;                       // operands of the exact kernel
    static constexpr int N_COUNTS = 2 * SHORTLIST_SEGS * 16;   // counters of the entries, then of the pairs
    DevTmp mem;                                               // what follows lies in it
    _Float16 *chk = nullptr, *xhk = nullptr;
    float2 *clen = nullptr, *xlen = nullptr;
    uint32_t *words = nullptr;                                // largest magnitudes, of the table and of each chunk of rows
    float *start = nullptr;
    float4 *tile = nullptr;
    unsigned long long *best = nullptr, *counts = nullptr;
    uint32_t *L = nullptr, *n_pairs = nullptr;                // side by side
    ShortEntry *list = nullptr;
    ShortPair *pairs = nullptr;
    unsigned long long seg_cap = 0, pair_cap = 0;
    const float *centroids = nullptr;          // the caller's table, as of the last set_centroids
    bool exact_packed = false;                 // ... is packed for the exact kernel
    bool shortlist = true;
    bool keep_rows = false;                    // the packed rows of every chunk stay (the same x in every run())
    bool rows_packed = false;
    ArgminCtx() = default;
    ArgminCtx(const ArgminCtx &) = delete;
    ArgminCtx &operator=(const ArgminCtx &) = delete;
    template <class T> static T *ptr(const DevTmp &m) { return static_cast<T *>(m.p); }
    // many_runs: run() will be called with the same rows again and again
    int init(int64_t K_, int D_, int64_t max_rows, bool many_runs = false)
    {
        K = K_; D = D_; Dp = packed_dim(D);
        // rows per launch: at most 2^20, and few enough that the grid (one workgroup of 256 threads per
        // tile of 128 rows x 128 centroids) stays below the 2^32 threads a launch may have
        const int64_t tiles_c = (K + GT - 1) / GT;
        int64_t max_tq = ((1ll << 24) - 1) / tiles_c / N_XCD * N_XCD;
        if (max_tq < N_XCD) return fail(IVF_EINVAL, "K=%lld: too many centroid tiles for one launch", (long long)K);
        chunk = max_tq * GT < (1ll << 20) ? max_tq * GT : (1ll << 20);
        if (max_rows < chunk) chunk = max_rows > 0 ? max_rows : 1;
        const char *off = getenv("IVF_GP_EXACT_ASSIGN");   // (for measurements: the one-pass exact kernel only)
        shortlist = !(off && off[0] == '1');
        if (!shortlist) {
            HIPCHK(mem.alloc((size_t)chunk * sizeof(unsigned long long)));
            best = static_cast<unsigned long long *>(mem.p);
            return IVF_OK;
        }
        // room for 24 entries per row on average (10 are usual at K = 2^16, growing with log K) and for 8 pairs (one is
        // usual), and for at least 2^16 of either in a segment
        seg_cap = (unsigned long long)(24 * chunk + SHORTLIST_SEGS - 1) / SHORTLIST_SEGS;
        pair_cap = (unsigned long long)(8 * chunk + SHORTLIST_SEGS - 1) / SHORTLIST_SEGS;
        if (seg_cap < (1ull << 16)) seg_cap = 1ull << 16;
        if (pair_cap < (1ull << 16)) pair_cap = 1ull << 16;
        keep_rows = many_runs && packed_rows(max_rows) * Dp * (int64_t)sizeof(_Float16) <= (8ll << 30);
        // one allocation for everything, 256-byte aligned pieces
        size_t total = 0;
        auto place = [&](auto *&p, size_t count) {
            p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(total);
            total += (count * sizeof(*p) + 255) / 256 * 256;
        };
        auto all = [&](size_t base) {
            const int64_t rows = keep_rows ? max_rows : chunk, n_words = 1 + (keep_rows ? (max_rows + chunk - 1) / chunk : 1);
            total = base;
            place(best, (size_t)chunk);
            place(chk, (size_t)packed_rows(K) * Dp);
            place(clen, (size_t)packed_rows(K));
            place(words, (size_t)n_words);
            place(start, (size_t)tiles_c * GT);
            place(tile, (size_t)tiles_c);
            place(xhk, (size_t)packed_rows(rows) * Dp);
            place(xlen, (size_t)packed_rows(rows));
            place(L, (size_t)(2 * (chunk + 2)));                // filled in 64-bit words
            place(list, (size_t)seg_cap * SHORTLIST_SEGS);
            place(pairs, (size_t)pair_cap * SHORTLIST_SEGS);
            place(counts, (size_t)N_COUNTS);
            return total;
        };
        hipError_t e = mem.alloc(all(0));
        if (e == hipErrorOutOfMemory && keep_rows) {            // packed a chunk at a time then, again in every run
            keep_rows = false;
            e = mem.alloc(all(0));
        }
        HIPCHK(e);
        all(reinterpret_cast<size_t>(mem.p));
        return IVF_OK;
    }
    int set_centroids(const float *centroids_, hipStream_t st)
    {
        centroids = centroids_;
        exact_packed = false;
        return shortlist ? launch_pack_hi(centroids, K, D, words, chk, clen, st) : IVF_OK;
    }
    // the exact one-pass kernel on m rows
    int run_exact(const float *x, int64_t m, hipStream_t st)
    {
        const int tiles_q = (int)((m + GT - 1) / GT);
        const int64_t grid = (int64_t)((tiles_q + N_XCD - 1) / N_XCD) * N_XCD * ((K + GT - 1) / GT);
        if (grid >= (1ll << 24)) return fail(IVF_EINVAL, "coarse tile grid too large");
        if (!cn.p) {
            HIPCHK(cn.alloc((size_t)K * sizeof(float)));
            HIPCHK(cpk.alloc((size_t)packed_rows(K) * Dp * 2 * sizeof(_Float16)));
            HIPCHK(csi.alloc(2 * sizeof(float)));
            HIPCHK(xn.alloc((size_t)chunk * sizeof(float)));
            HIPCHK(xsi.alloc((size_t)chunk * sizeof(float)));
            HIPCHK(xpk.alloc((size_t)packed_rows(chunk) * Dp * 2 * sizeof(_Float16)));
        }
        int rc;
        if (!exact_packed) {
            if ((rc = pack_rows(centroids, K, D, ptr<uint32_t>(csi) + 1, ptr<_Float16>(cpk), ptr<float>(cn), ptr<float>(csi), st))) return rc;
            exact_packed = true;
        }
        if ((rc = pack_rows(x, m, D, nullptr, ptr<_Float16>(xpk), ptr<float>(xn), ptr<float>(xsi), st))) return rc;
        fill_u64_kernel<<<dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st>>>(best, m, ~0ull);
        LAUNCHCHK("fill_u64_kernel");
        coarse_argmin_kernel<<<dim3((unsigned)grid), dim3(256), 0, st>>>(ptr<_Float16>(xpk), ptr<float>(xn), ptr<float>(xsi), m, ptr<_Float16>(cpk),
                                                                         ptr<float>(cn), ptr<float>(csi), K, Dp, best, tiles_q);
        LAUNCHCHK("coarse_argmin_kernel");
        ++g_assign_exact;
        return IVF_OK;
    }
    // shortlist + exact decision for the rows q0 .. q0 + m of x; *overflow = the list did not hold every candidate
    // (best[] is then incomplete); near (may be NULL): a centroid of every row, likely a near one; want_d: distances too, not
    // only the centroids
    int run_shortlist(const float *x, int64_t q0, int64_t m, const int32_t *near, bool want_d, bool *overflow, hipStream_t st)
    {
        const int64_t tiles_c = (K + GT - 1) / GT;
        const float *xm = x + q0 * D;
        uint32_t *xw = words + 1 + (keep_rows ? q0 / chunk : 0);
        _Float16 *xh = xhk + (keep_rows ? q0 : 0) * (int64_t)Dp;
        float2 *xl = xlen + (keep_rows ? q0 : 0);
        int rc;
        if (!(keep_rows && rows_packed) && (rc = launch_pack_hi(xm, m, D, xw, xh, xl, st))) return rc;
        shortlist_tiles_kernel<<<dim3((unsigned)tiles_c), dim3(128), 0, st>>>(clen, K, Dp, words, xw,
                                                                              start, tile);
        LAUNCHCHK("shortlist_tiles_kernel");
        // L and the numbers of pairs: 32-bit words, cleared two at a time
        n_pairs = L + (m + 1) / 2 * 2;
        static_assert(N_COUNTS % 2 == 0, "whole words");
        shortlist_clear_kernel<<<dim3((unsigned)((m + 1 + 255) / 256 + (N_COUNTS + 255) / 256)), dim3(256), 0, st>>>(
            best, m, reinterpret_cast<unsigned long long *>(L), (m + 1) / 2 * 2, counts, N_COUNTS);
        LAUNCHCHK("shortlist_clear_kernel");
        ShortlistArgs a;
        a.Qh = xh;
        a.qlen = xl;
        a.nq = m;
        a.K = K;
        a.Ch = chk;
        a.start = start;
        a.tile = tile;
        a.clen = clen;
        a.Dp = Dp;
        a.L = L;
        a.n_pairs = n_pairs;
        a.list = list;
        a.pairs = pairs;
        a.count = counts;
        a.pair_count = a.count + N_COUNTS / 2;
        a.seg_cap = seg_cap;
        a.pair_cap = pair_cap;
        a.tiles_c = (int)tiles_c;
        if (near) {
            seed_bounds_kernel<<<dim3((unsigned)((m + 63) / 64)), dim3(256), 0, st>>>(a, near + q0);
            LAUNCHCHK("seed_bounds_kernel");
        }
        const bool wide = Dp <= 128 && shortlist_wide(m, K);
        const int per_q = wide ? 2 * GT : GT;
        a.tiles_q = (int)((m + per_q - 1) / per_q);
        const int64_t tq8 = (int64_t)((a.tiles_q + N_XCD - 1) / N_XCD) * N_XCD;
        if (Dp <= 128) {   // query tile in registers, centroid tiles swept: long sweeps unless the chip would stand empty
            int per_wg = 64;
            while (per_wg > 4 && tq8 * ((tiles_c + per_wg - 1) / per_wg) < 1536) per_wg /= 2;
            const dim3 grid((unsigned)(tq8 * ((tiles_c + per_wg - 1) / per_wg)));
            auto sweep = [&](auto narrow_kernel, auto wide_kernel) { (wide ? wide_kernel : narrow_kernel)<<<grid, dim3(256), 0, st>>>(a, per_wg); };
            if (Dp == 32) sweep(&coarse_shortlist_sweep_kernel<1, 2>, &coarse_shortlist_sweep_kernel<1, 4>);
            else if (Dp == 64) sweep(&coarse_shortlist_sweep_kernel<2, 2>, &coarse_shortlist_sweep_kernel<2, 4>);
            else if (Dp == 96) sweep(&coarse_shortlist_sweep_kernel<3, 2>, &coarse_shortlist_sweep_kernel<3, 4>);
            else sweep(&coarse_shortlist_sweep_kernel<4, 2>, &coarse_shortlist_sweep_kernel<4, 4>);
            LAUNCHCHK("coarse_shortlist_sweep_kernel");
        } else {
            if (tq8 * tiles_c >= (1ll << 24)) return fail(IVF_EINVAL, "coarse tile grid too large");
            coarse_shortlist_kernel<<<dim3((unsigned)(tq8 * tiles_c)), dim3(256), 0, st>>>(a);
            LAUNCHCHK("coarse_shortlist_kernel");
        }
        // (loops over the lists: a grid that fills the chip, whatever their length)
        shortlist_pairs_kernel<<<dim3(64, SHORTLIST_SEGS), dim3(256), 0, st>>>(a);
        LAUNCHCHK("shortlist_pairs_kernel");
        (want_d ? &rerank_kernel<true> : &rerank_kernel<false>)<<<dim3(32, SHORTLIST_SEGS), dim3(256), 0, st>>>(xm, centroids, D, a, best);
        LAUNCHCHK("rerank_kernel");
        unsigned long long n[N_COUNTS];
        HIPCHK(hipMemcpyAsync(n, counts, sizeof(n), hipMemcpyDeviceToHost, st));
        HIPCHK(hipStreamSynchronize(st));
        unsigned long long longest = 0, most = 0;
        for (int sgm = 0; sgm < SHORTLIST_SEGS; ++sgm) {
            longest = n[sgm * 16] > longest ? n[sgm * 16] : longest;
            most = n[N_COUNTS / 2 + sgm * 16] > most ? n[N_COUNTS / 2 + sgm * 16] : most;
        }
        *overflow = longest > seg_cap || most > pair_cap || longest == 0;
        if (*overflow) return IVF_OK;
        ++g_assign_short;
        return IVF_OK;
    }
    // out_id[i] = nearest centroid of x[i] by (distance, id), out_d[i] (may be NULL) its squared distance; near: may be out_id
    int run(const float *x, int64_t n, int32_t *out_id, float *out_d, hipStream_t st, int32_t missing = -1, const int32_t *near = nullptr)
    {
        int rc;
        for (int64_t q0 = 0; q0 < n; q0 += chunk) {
            const int64_t m = (n - q0 < chunk) ? n - q0 : chunk;
            bool overflow = true;
            if (shortlist && (rc = run_shortlist(x, q0, m, near, out_d != nullptr, &overflow, st))) return rc;
            if (overflow && (rc = run_exact(x + q0 * D, m, st))) return rc;
            argmin_unpack_kernel<<<dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st>>>(best, m, missing, out_id + q0, out_d ? out_d + q0 : nullptr);
            LAUNCHCHK("argmin_unpack_kernel");
        }
        rows_packed = true;
        return IVF_OK;
    }
};

int check_coarse_args(const float *centroids, int64_t K, int D, const float *x, int64_t nq)
{
    if (!centroids || !x) return fail(IVF_EINVAL, "NULL argument");
    if (D < 4 || D % 4 || D > IVF_MAX_D) return fail(IVF_EINVAL, "D=%d must be a multiple of 4 in [4, %d]", D, IVF_MAX_D);
    if (K < 1 || K >= (1ll << 31)) return fail(IVF_EINVAL, "K=%lld out of range", (long long)K);
    if (nq < 0 || nq >= (1ll << 31)) return fail(IVF_EINVAL, "row count out of range");
    if (!aligned16(centroids) || !aligned16(x)) return fail(IVF_EINVAL, "centroids and x must be 16-byte aligned");
    return IVF_OK;
}

// The P nearest centroids of every row of x through the distance tile (P > 1), on scratch of its own.
int coarse_topk_tiled(const float *centroids, int64_t K, int D, const float *x, int64_t nq, int P,
                      int32_t *out_id, float *out_d, hipStream_t st)
{
    int64_t tile = (4ll << 30) / (K * (int64_t)sizeof(float));
    if (tile < 1) tile = 1;
    if (tile >= nq) tile = nq;
    else if (tile >= 256) tile -= tile % 256;   // whole blocks of the padded row count
    else if (tile >= GT) tile -= tile % GT;
    const int64_t nb = (K + BMW - 1) / BMW;
    const int Dp = packed_dim(D);
    DevTmp cn, csi, cpk, xn, xsi, xpk, Dt, bm;
    HIPCHK(cn.alloc((size_t)K * sizeof(float)));
    HIPCHK(cpk.alloc((size_t)packed_rows(K) * Dp * 2 * sizeof(_Float16)));
    HIPCHK(csi.alloc(2 * sizeof(float)));
    const size_t tile_pad = (size_t)packed_rows(tile);   // the GEMM may write whole tiles of rows
    HIPCHK(xn.alloc(tile_pad * sizeof(float)));
    HIPCHK(xsi.alloc(tile_pad * sizeof(float)));
    HIPCHK(xpk.alloc(tile_pad * Dp * 2 * sizeof(_Float16)));
    HIPCHK(Dt.alloc(tile_pad * dt_stride(K) * sizeof(float)));
    HIPCHK(bm.alloc(tile_pad * nb * sizeof(float)));
    float *csi_f = static_cast<float *>(csi.p);
    int rc = pack_rows(centroids, K, D, reinterpret_cast<uint32_t *>(csi_f + 1), static_cast<_Float16 *>(cpk.p),
                       static_cast<float *>(cn.p), csi_f, st);
    for (int64_t q0 = 0; q0 < nq && !rc; q0 += tile) {
        const int64_t n = (nq - q0 < tile) ? nq - q0 : tile;
        if ((rc = pack_rows(x + q0 * D, n, D, nullptr, static_cast<_Float16 *>(xpk.p), static_cast<float *>(xn.p),
                            static_cast<float *>(xsi.p), st))) break;
        if ((rc = launch_coarse(static_cast<_Float16 *>(xpk.p), static_cast<float *>(xn.p), static_cast<float *>(xsi.p), n,
                                static_cast<_Float16 *>(cpk.p), static_cast<float *>(cn.p), csi_f, K, Dp,
                                static_cast<float *>(Dt.p), static_cast<float *>(bm.p), st))) break;
        rc = launch_probe_select(static_cast<float *>(Dt.p), static_cast<float *>(bm.p), n, K, P, out_id + q0 * P,
                                 out_d + q0 * P, st);
    }
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);   // the temporaries are released on return
    g_err = keep;
    return rc;
}

}  // namespace

namespace {

bool pq_width(int ds) { return ds == 4 || ds == 6 || ds == 8 || ds == 12 || ds == 16; }

// Codes of n displacements (and, with MU, constants), for the block widths pq_width() names.
template <int DS>
int launch_pq_encode_ds(const float *E, const float *MU, int64_t n, int M, const float *codebook, const float *const_table,
                        uint8_t *out_codes, uint8_t *out_byte, float *out_t, hipStream_t st)
{
    const int Mg = pq_per_group(M, PqRow<DS>::bytes), groups = (M + Mg - 1) / Mg;
    if (MU && groups > 1) return fail(IVF_EINVAL, "the constants need all quantisers in one workgroup");
    const int lds = Mg * PqRow<DS>::bytes;
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&pq_encode_kernel<DS>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    int64_t grid = (n + WAVE - 1) / WAVE;   // one workgroup of 16 wavefronts fits a compute unit
    if (grid > 256) grid = 256;
    pq_encode_kernel<DS><<<dim3((unsigned)grid, (unsigned)groups), dim3(1024), lds, st>>>(E, MU, n, M, Mg, codebook, const_table, out_codes, out_byte, out_t);
    LAUNCHCHK("pq_encode_kernel");
    return IVF_OK;
}

int launch_pq_encode(int ds, const float *E, const float *MU, int64_t n, int M, const float *codebook, const float *const_table,
                     uint8_t *out_codes, uint8_t *out_byte, float *out_t, hipStream_t st)
{
    auto fn = ds == 4 ? &launch_pq_encode_ds<4> : ds == 6 ? &launch_pq_encode_ds<6> : ds == 8 ? &launch_pq_encode_ds<8>
            : ds == 12 ? &launch_pq_encode_ds<12> : &launch_pq_encode_ds<16>;
    return fn(E, MU, n, M, codebook, const_table, out_codes, out_byte, out_t, st);
}

// The codebook update from the codes: slices of sums and counts (scratch of pq_sum_slices(n) of them), then the means.
// state: the largest magnitude of E and the flag of pq_means_kernel (32 bits each), [M][256] counts and [M][256][DS] rests
// (64 bits each), which start at 0.
int64_t pq_sum_slices(int64_t n) { return n >= 2048 * PQ_SUM_MAX_G ? PQ_SUM_MAX_G : (n + 2047) / 2048; }

template <int DS>
int launch_pq_means_ds(const float *E, int64_t n, int M, const uint8_t *codes, uint32_t *state, double *psum, uint32_t *pcnt,
                       float *codebook, hipStream_t st)
{
    unsigned long long *small = reinterpret_cast<unsigned long long *>(state + 2), *rest = small + (size_t)M * 256;
    const int64_t G = pq_sum_slices(n), per = (n + G - 1) / G;
    const int groups = (M + PqSums<DS>::MG - 1) / PqSums<DS>::MG;
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&pq_sums_kernel<DS>), hipFuncAttributeMaxDynamicSharedMemorySize, PqSums<DS>::lds));
    pq_sums_kernel<DS><<<dim3(pq_sums_grid(G, groups)), dim3(PQ_SUM_BLOCK), PqSums<DS>::lds, st>>>(E, n, M, codes, state, (int)G, per, psum, pcnt, rest, small);
    LAUNCHCHK("pq_sums_kernel");
    pq_means_kernel<DS><<<dim3((unsigned)(M * 256 * DS / 64)), dim3(64 * PQ_MEAN_PARTS), 0, st>>>(psum, pcnt, M, (int)G, state, rest, small, state + 1, codebook);
    LAUNCHCHK("pq_means_kernel");
    return IVF_OK;
}

int launch_pq_means(int ds, const float *E, int64_t n, int M, const uint8_t *codes, uint32_t *state, double *psum, uint32_t *pcnt,
                    float *codebook, hipStream_t st)
{
    auto fn = ds == 4 ? &launch_pq_means_ds<4> : ds == 6 ? &launch_pq_means_ds<6> : ds == 8 ? &launch_pq_means_ds<8>
            : ds == 12 ? &launch_pq_means_ds<12> : &launch_pq_means_ds<16>;
    return fn(E, n, M, codes, state, psum, pcnt, codebook, st);
}

}  // namespace

extern "C" void ivf_assign_stats(int64_t *out)
{
    out[0] = g_assign_short.load();
    out[1] = g_assign_exact.load();
}

extern "C" int ivf_coarse_topk(const float *centroids, int64_t K, int D, const float *x, int64_t nq, int P,
                               int32_t *out_id, float *out_d, void *hip_stream)
{
    int rc = check_coarse_args(centroids, K, D, x, nq);
    if (rc) return rc;
    if (!out_id || !out_d) return fail(IVF_EINVAL, "NULL argument");
    if (P < 1 || P > K || P > 4096) return fail(IVF_EINVAL, "need 1 <= P <= min(K, 4096)");
    if (nq == 0) return IVF_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (P > 1) return coarse_topk_tiled(centroids, K, D, x, nq, P, out_id, out_d, st);
    ArgminCtx ctx;   // fused per-row minimum, no distance tile
    if ((rc = ctx.init(K, D, nq))) return rc;
    if (!(rc = ctx.set_centroids(centroids, st))) rc = ctx.run(x, nq, out_id, out_d, st);
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

namespace {

// The centroid table as 8-bit rows (rows NULL: not packed).
struct SubregionTable {
    const uint8_t *rows = nullptr, *tails = nullptr;
    const float *centre = nullptr;
};

template <int DP>
int pack_subregion_table(const ivf_index_desc *t, uint8_t *mem, SubregionTable &table, hipStream_t st)
{
    typedef ByteRow<DP> R;
    constexpr int per = 256 / (R::BYTES / 16);               // rows of a workgroup
    float *centre = reinterpret_cast<float *>(mem);
    mem += 128 * sizeof(float);
    uint8_t *tails = R::INSIDE ? mem + DP : mem + (size_t)t->K * R::BYTES;
    const int64_t grid = (t->K + per - 1) / per;
    pack_byte_rows_kernel<DP><<<dim3((unsigned)(grid < BYTE_ROWS_GRID ? grid : BYTE_ROWS_GRID)), dim3(256), 0, st>>>(t->centroids, t->K, t->D, centre, mem, tails);
    LAUNCHCHK("pack_byte_rows_kernel");
    table.rows = mem;
    table.tails = tails;
    table.centre = centre;
    return IVF_OK;
}

int launch_subregions(const ivf_index_desc *t, const float *x, int64_t n, const int32_t *region, const int32_t *perm,
                      const SubregionTable &table, int32_t *out_sub, float *out_res, float *out_mu, hipStream_t st)
{
    const int dp = packed_dim(t->D);
    auto kernel = dp == 32 ? &subregion_kernel<32> : dp == 64 ? &subregion_kernel<64> : dp == 96 ? &subregion_kernel<96> : &subregion_kernel<128>;
    kernel<<<dim3((unsigned)((n + 4 * SUB_RUN - 1) / (4 * SUB_RUN))), dim3(256), 0, st>>>(
        x, n, t->D, t->L, region, perm, t->centroids, table.centre, table.rows, table.tails, t->nbr, t->alpha, t->cs_dist2, out_sub, out_res, out_mu);
    LAUNCHCHK("subregion_kernel");
    return IVF_OK;
}

}  // namespace

extern "C" int ivf_encode(const ivf_index_desc *t, const float *x, int64_t n, const int32_t *region_in,
                          int32_t *out_region, int32_t *out_sub, uint8_t *out_codes,
                          uint8_t *out_const_byte, float *out_const_t, float *out_residual,
                          void *hip_stream)
{
    int rc = check_trained(t);
    if (rc) return rc;
    if (!x || !out_region || !out_sub) return fail(IVF_EINVAL, "NULL argument");
    if (t->pq_codebook && !out_codes) return fail(IVF_EINVAL, "out_codes is NULL");
    if (t->pq_codebook && !aligned16(t->pq_codebook)) return fail(IVF_EINVAL, "pq_codebook must be 16-byte aligned");
    if (t->pq_codebook && t->const_table && !out_const_byte) return fail(IVF_EINVAL, "out_const_byte is NULL");
    if (!aligned16(x)) return fail(IVF_EINVAL, "x must be 16-byte aligned");
    if (n < 0 || n >= (1ll << 31)) return fail(IVF_EINVAL, "n out of range");
    if (n == 0) return IVF_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ArgminCtx ctx;                               // the assignment's, with the packed centroid table
    DevTmp byte_mem;
    StreamWait before_they_go(st);               // (every return below: the pool takes their blocks back when nothing uses them)
    SubregionTable table;
    if (region_in) {
        if (region_in != out_region)
            HIPCHK(hipMemcpyAsync(out_region, region_in, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
    } else {
        rc = ctx.init(t->K, t->D, n);
        if (!rc) rc = ctx.set_centroids(t->centroids, st);
        if (!rc) rc = ctx.run(x, n, out_region, nullptr, st, 0);   // (rows that are not numbers: a region that can be read)
        if (rc) {
            std::string keep = g_err;
            (void)hipStreamSynchronize(st);   // the temporaries are released on return
            g_err = keep;
            return rc;
        }
    }
    // PQ codes on the matrix units when the codebook fits LDS and D / M is one of the compiled
    // block widths; else by the wavefront-per-point kernel, which does everything.
    const int ds = t->D / t->M;
    const size_t cb_bytes = (size_t)256 * t->D * sizeof(float);
    const bool fast = t->pq_codebook && cb_bytes <= 140 * 1024 && pq_width(ds);
    if (t->rotation && t->pq_codebook && !fast)
        return fail(IVF_EINVAL, "a rotation in front of the PQ needs D/M in {4, 6, 8, 12, 16} and a codebook that fits LDS");
    // Subregions by 8-bit rows with a bound where the rows fit registers and there are points enough to pay for packing the table.  Whole calls
    // with given regions, 96 dimensions, us by fp32 / 8-bit rows: K = 2^20, L = 64, n L = 4 K 319 / 344, 6 K 444 / 419, 9 K 640 / 513; L = 16, 6 K 720 / 783,
    // 9 K 1087 / 1053; L = 8, 6 K 1274 / 1278, 9 K 1904 / 1813.  On small tables the chain of 16 points that a wavefront takes one after the
    // other is longer than the fp32 rows of so few: K = 65 536, L = 64, 9 K 108 / 130, L = 8, 9 K 155 / 172; K = 4096 80 / 110 at any of these.  The table is
    // allocated behind everything else: where there is no room for it, encode_kernel reads the fp32 rows.
    const bool packs = packed_dim(t->D) <= 128 && t->L <= 64 && n * t->L >= 10 * t->K;
    auto prepare_table = [&]() -> int {
        if (!packs) return IVF_OK;
        const int dp = packed_dim(t->D);
        const hipError_t no_room = byte_mem.alloc(128 * sizeof(float) + (size_t)t->K * byte_row_bytes(dp));
        if (no_room == hipErrorOutOfMemory) return IVF_OK;
        HIPCHK(no_room);
        auto pack = dp == 32 ? &pack_subregion_table<32> : dp == 64 ? &pack_subregion_table<64> : dp == 96 ? &pack_subregion_table<96> : &pack_subregion_table<128>;
        return pack(t, static_cast<uint8_t *>(byte_mem.p), table, st);
    };
    if (!fast && !t->pq_codebook) {
        rc = prepare_table();
        if (!rc && table.rows) rc = launch_subregions(t, x, n, out_region, nullptr, table, out_sub, out_residual, nullptr, st);
        if (rc || table.rows) {
            std::string keep = g_err;
            const hipError_t e = hipStreamSynchronize(st);
            g_err = keep;
            return rc ? rc : e == hipSuccess ? IVF_OK : fail(IVF_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
        }
    }
    if (!fast) {
        encode_kernel<<<dim3((unsigned)n), dim3(64), (size_t)4 * t->D * sizeof(float), st>>>(
            x, n, t->D, t->M, t->L, out_region, t->centroids, t->nbr, t->alpha, t->cs_dist2, t->pq_codebook,
            t->const_table, out_sub, out_codes, out_const_byte, out_const_t, out_residual, nullptr);
        LAUNCHCHK("encode_kernel");
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    }
    const int64_t chunk = n < (1ll << 20) ? n : (1ll << 20);
    const int D = t->D;
    DevTmp e, mu, erot, rt;
    RadixBufs rb;
    auto body = [&]() -> int {
        // regions found here come in the order of the points: sorted, the points of a region share its rows
        const bool order = packs && !region_in && n >= 4 * t->K;
        int r3 = order ? rb.init(chunk) : IVF_OK;
        if (r3) return r3;
        if (!out_residual) HIPCHK(e.alloc((size_t)chunk * D * sizeof(float)));
        HIPCHK(mu.alloc((size_t)chunk * D * sizeof(float)));
        if (t->rotation) {   // the PQ sees R (x - mu), the per-point constant is taken with R mu
            HIPCHK(erot.alloc((size_t)chunk * D * sizeof(float)));
            HIPCHK(rt.alloc((size_t)D * D * sizeof(float)));
            transpose_square_kernel<<<dim3((unsigned)((D * D + 255) / 256)), dim3(256), 0, st>>>(t->rotation, D, static_cast<float *>(rt.p));
            LAUNCHCHK("transpose_square_kernel");
        }
        if ((r3 = prepare_table())) return r3;
        float *muc = static_cast<float *>(mu.p);
        for (int64_t i0 = 0; i0 < n; i0 += chunk) {
            const int64_t m = n - i0 < chunk ? n - i0 : chunk;
            float *ec = out_residual ? out_residual + i0 * D : static_cast<float *>(e.p);
            if (table.rows) {
                const int32_t *perm = nullptr;
                if (order) {
                    HIPCHK(hipMemcpyAsync(rb.keys_a(), out_region + i0, (size_t)m * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
                    uint32_t *ks, *vs;
                    if ((r3 = rb.sort(m, bits_for(t->K), false, &ks, &vs, st))) return r3;
                    perm = reinterpret_cast<const int32_t *>(vs);
                }
                if ((r3 = launch_subregions(t, x + i0 * D, m, out_region + i0, perm, table, out_sub + i0, ec, muc, st))) return r3;
            } else {
                encode_kernel<<<dim3((unsigned)m), dim3(64), (size_t)4 * D * sizeof(float), st>>>(
                    x + i0 * D, m, D, t->M, t->L, out_region + i0, t->centroids, t->nbr, t->alpha, t->cs_dist2,
                    nullptr, nullptr, out_sub + i0, nullptr, nullptr, nullptr, ec, muc);
                LAUNCHCHK("encode_kernel");
            }
            const float *pe = ec;
            if (t->rotation) {
                const unsigned rg = (unsigned)((m + ROT_ROWS - 1) / ROT_ROWS);
                const size_t rl = (size_t)ROT_ROWS * D * sizeof(float);
                rotate_rows_kernel<<<dim3(rg), dim3(256), rl, st>>>(ec, m, D, static_cast<float *>(rt.p), static_cast<float *>(erot.p));
                LAUNCHCHK("rotate_rows_kernel");
                rotate_rows_kernel<<<dim3(rg), dim3(256), rl, st>>>(muc, m, D, static_cast<float *>(rt.p), muc);
                LAUNCHCHK("rotate_rows_kernel");
                pe = static_cast<float *>(erot.p);
            }
            uint8_t *oc = out_codes + i0 * t->M;
            uint8_t *ob = out_const_byte ? out_const_byte + i0 : nullptr;
            float *ot = out_const_t ? out_const_t + i0 : nullptr;
            int r2 = launch_pq_encode(ds, pe, muc, m, t->M, t->pq_codebook, t->const_table, oc, ob, ot, st);
            if (r2) return r2;
        }
        HIPCHK(hipStreamSynchronize(st));
        return IVF_OK;
    };
    rc = body();
    {
        std::string keep = g_err;
        (void)hipStreamSynchronize(st);   // the temporaries are released on return
        g_err = keep;
    }
    return rc;
}

extern "C" int ivf_rotate(const float *x, int64_t n, int D, const float *rotation, float *out, void *hip_stream)
{
    if (!x || !rotation || !out) return fail(IVF_EINVAL, "NULL argument");
    if (D < 1 || D > IVF_MAX_D || n < 0 || n >= (1ll << 31)) return fail(IVF_EINVAL, "bad sizes");
    if (n == 0) return IVF_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    DevTmp rt;
    HIPCHK(rt.alloc((size_t)D * D * sizeof(float)));
    transpose_square_kernel<<<dim3((unsigned)((D * D + 255) / 256)), dim3(256), 0, st>>>(rotation, D, static_cast<float *>(rt.p));
    int rc = IVF_OK;
    hipError_t e1 = hipGetLastError();
    if (e1 != hipSuccess) rc = fail(IVF_EHIP, "launch transpose_square_kernel: %s", hipGetErrorString(e1));
    if (!rc) {
        rotate_rows_kernel<<<dim3((unsigned)((n + ROT_ROWS - 1) / ROT_ROWS)), dim3(256), (size_t)ROT_ROWS * D * sizeof(float), st>>>(
            x, n, D, static_cast<float *>(rt.p), out);
        e1 = hipGetLastError();
        if (e1 != hipSuccess) rc = fail(IVF_EHIP, "launch rotate_rows_kernel: %s", hipGetErrorString(e1));
    }
    std::string keep = g_err;
    (void)hipStreamSynchronize(st);
    g_err = keep;
    return rc;
}

extern "C" int ivf_copy_bytes(void *dst, const void *src, int64_t nbytes, void *hip_stream)
{
    if (!dst || !src || nbytes < 0 || nbytes % 16 || !aligned16(dst) || !aligned16(src))
        return fail(IVF_EINVAL, "ivf_copy_bytes needs 16-byte aligned pointers and a multiple of 16 bytes");
    if (nbytes == 0) return IVF_OK;
    const int64_t n16 = nbytes / 16;
    int64_t grid = (n16 + 255) / 256;
    if (grid > 256 * 32) grid = 256 * 32;
    copy_bytes_kernel<<<dim3((unsigned)grid), dim3(256), 0, static_cast<hipStream_t>(hip_stream)>>>(
        static_cast<const uint4 *>(src), static_cast<uint4 *>(dst), n16);
    LAUNCHCHK("copy_bytes_kernel");
    return IVF_OK;
}

#include "train_api.hpp"
