// Stages 1 to 2 of the query path without the distance matrix, for large batches and for small ones on large tables
// (sparse_pays).  Of the nq x K distances a search needs
// some hundred blocks of 64 per query (the nprobe closest regions lie in them) and the L neighbours of its nprobe
// regions: 2 % of them at K = 2^20.  Writing all of them, and reading 4 bytes from a 128-byte line each, took 14.3 of the
// 16.3 ms of 10 000 queries there.  Here:
//   1. coarse_minima_kernel: <q, c> - |c|^2 / 2 with operands rounded to fp16, a third of the matrix work, and only the largest
//      value of every 64 centroids is written.  It is known within a bound (coarse_shortlist_sweep_kernel has the same).
//   2. flag_blocks_kernel: the blocks of 64 that can hold one of the P closest, a few more than P.
//   3. pair_distance_kernel<false>: the exact distances of the flagged blocks, grouped by block, so that the rows of a block are
//      read once for the up to 32 queries a wavefront takes.
//   4. probe_pick_kernel: the P closest regions among them.
//   5. pair_distance_kernel<true>: the scores of Eq. (7), grouped by region: the neighbours' rows are read once for the
//      queries that probe the region, regions with common neighbours side by side (order.hpp).
// Up to SPARSE_DIRECT queries the pairs of 3. and 5. are not grouped.
// The distances are formed by the same products in the same order as in coarse_gemm_kernel, so a query's results do
// not depend on which way its batch goes.  A query whose bound is too wide to leave at most 2 P blocks (vectors far from the
// origin compared with their spread, rows that are not finite) gets exact block minima first (hard_* kernels, which end at
// once when there is none): for a tile of 128 such queries or less a pass over the whole table.  One query that is not finite alone, K = 2^20,
// P = 16 254 us (90 with a bound, 129 with the matrix), P = 256 331 (104, 193); one among 64 266 (105, 208), among 256 324 (172, 389),
// among 10 000 3530 (3360, 11 500).  Tables that have such queries themselves do not go this way (count_hard).
#pragma once
#include "coarse.hpp"
#include "query.hpp"

namespace ivf {

// The queries' fp16 rows have the centroid table's scale, 2^10 times smaller: room for components 2000 times the table's
// largest (a query with a larger one is a hard one), and 2^18 times smaller than it before they lose bits.
constexpr int SPARSE_HEADROOM = 10;
constexpr int64_t SPARSE_MIN_K = 16384;   // (sparse_pays: below, no batch of less than 8192 queries takes it)

// |x| and |dx| of a row (see pack_hi_rows_kernel) with infinite lengths where a centroid of the tile is not finite: such a
// block is always looked at.  start[c] = (-1/2 + k) |c|^2 in units of the product, -inf past K; tile[t] = (largest |c|,
// largest |dc|, smallest start value, 0).
__global__ __launch_bounds__(128) void minima_tiles_kernel(const float2 *__restrict__ clen, int64_t K, int Dp, float *__restrict__ start,
                                                           float4 *__restrict__ tile)
{
    __shared__ float4 part[2];
    const int64_t c = (int64_t)blockIdx.x * 128 + threadIdx.x;
    float2 l = make_float2(0.f, 0.f);
    float v = -INFINITY, low = 0.f;
    if (c < K) {
        l = clen[c];
        if (l.x < INFINITY) {
            const float len0 = l.x * (1.f / (1.f + 0x1p-10f));     // (the length was rounded up by 2^-10)
            v = low = (-0.5f + (float)(Dp + 32) * 0x1p-24f) * __builtin_amdgcn_ldexpf(len0 * len0, -SPARSE_HEADROOM);
        }
    }
    start[c] = v;
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        l.x = fmaxf(l.x, __shfl_xor(l.x, o, WAVE));
        l.y = fmaxf(l.y, __shfl_xor(l.y, o, WAVE));
        low = fminf(low, __shfl_xor(low, o, WAVE));
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = make_float4(l.x, l.y, low, 0.f);
    __syncthreads();
    if (threadIdx.x == 0)
        tile[blockIdx.x] = make_float4(fmaxf(part[0].x, part[1].x), fmaxf(part[0].y, part[1].y), fminf(part[0].z, part[1].z), 0.f);
}

// nbr_norm[r][l] = |s_l|^2: read as one piece where the neighbours' own norms would be a line each
__global__ __launch_bounds__(256) void neighbour_norm_kernel(const int32_t *__restrict__ nbr, int64_t total, const float *__restrict__ cnorm,
                                                             float *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < total) out[i] = cnorm[nbr[i]];
}

// The queries as hi/lo rows (split_rows_kernel) and as fp16 rows in pack_hi_rows_kernel's layout, at the table's scale; a wavefront a row.  Rows past n (up to n_pad)
// are zeros.  Workgroups from rows_grid on clear `words` 64-bit words of counters.
__global__ __launch_bounds__(256) void sparse_queries_kernel(const float *__restrict__ X, int64_t n, int64_t n_pad, int D, int Dp,
                                                             const uint32_t *__restrict__ cmax, _Float16 *__restrict__ P, float *__restrict__ norm,
                                                             float *__restrict__ inv_scale, _Float16 *__restrict__ H, float2 *__restrict__ len,
                                                             unsigned rows_grid, unsigned long long *__restrict__ zero, int64_t words)
{
    if (blockIdx.x >= rows_grid) {
        for (int64_t i = (int64_t)(blockIdx.x - rows_grid) * 256 + threadIdx.x; i < words; i += (int64_t)(gridDim.x - rows_grid) * 256) zero[i] = 0;
        return;
    }
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= n_pad) return;
    if (row < n) split_row(X, row, D, nullptr, P, norm, inv_scale);
    const int sh = hi_scale(*cmax) - SPARSE_HEADROOM;
    float s2 = 0.f, d2 = 0.f;
    _Float16 hi[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + u * WAVE;
        const float f = row < n && i < D ? __builtin_amdgcn_ldexpf(X[row * D + i], sh) : 0.f;
        hi[u] = (_Float16)f;
        const float d = f - (float)hi[u];
        s2 = fmaf(f, f, s2);
        d2 = fmaf(d, d, d2);
    }
    s2 = wave_sum(s2);
    d2 = wave_sum(d2);
    const bool fits = s2 < INFINITY && d2 < INFINITY;              // (a component that fp16 cannot hold leaves an infinite rest)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + u * WAVE, k8 = (i >> 3) & 3;
        if (i < Dp) H[row * Dp + (i & ~31) + 8 * ((k8 & 1) * 2 + (k8 >> 1)) + (i & 7)] = fits ? hi[u] : (_Float16)0.f;
    }
    if (lane == 0)
        len[row] = fits ? make_float2(sqrtf(s2 + 0x1p-100f) * (1.f + 0x1p-10f), sqrtf(d2 + 0x1p-100f) * (1.f + 0x1p-10f)) : make_float2(INFINITY, INFINITY);
}

// Row q of the block maxima: the even blocks of 64 (first halves of the tiles), then the odd ones, each padded to a
// multiple of four.
__host__ __device__ inline int64_t minima_half(int64_t K) { return ((K + GT - 1) / GT + 3) / 4 * 4; }

// best[q][half][t] = the largest of <q, c> - (1/2 - k) |c|^2 over the 64 centroids of the half of tile t, for a sweep of
// `tiles_per_wg` (a multiple of four) centroid tiles by a workgroup, 64 queries a wavefront (sweep_tile).  A lane ends up with the maxima of
// one query, four tiles in a row, and stores them as 16 bytes.  10 000 x 2^20, 96 dimensions: 1.62 ms (1.24 PFLOP/s), 2.03 with two
// wavefronts to 64 queries and the fragments waited for where they are read; 10 000 x 65 536 0.115 and 0.131, 128 dimensions 0.156 and 0.191.
template <int SH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void coarse_minima_kernel(
    const _Float16 *__restrict__ Qh, const _Float16 *__restrict__ Ch, const float *__restrict__ start, float *__restrict__ best, int64_t half_ld,
    int tiles_q, int tiles_c, int tiles_per_wg)
{
    __shared__ __attribute__((aligned(16))) SweepTile<SH> buf0;
    __shared__ __attribute__((aligned(16))) SweepTile<SH> buf1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    int64_t tq, group;
    if (!group_of_block(blockIdx.x, tiles_q, (tiles_c + tiles_per_wg - 1) / tiles_per_wg, tq, group)) return;
    const int tb = (int)(group * tiles_per_wg);
    int t_end = tb < tiles_c ? tiles_c - tb : 0;
    if (t_end > tiles_per_wg) t_end = tiles_per_wg;
    if (t_end <= 0) return;
    const int64_t q0 = tq * (2 * GT) + wave * 64;
    const TileTwists<SH> twists(wave, lane);
    auto issue = [&](int t, SweepTile<SH> &buf) { sweep_copy(Ch, start, tb + t, buf, twists, wave, lane); };
    issue(0, buf0);
    gu32x4 afr[SH][2][2];
    sweep_rows(afr, Qh, q0, l32, h);
    float *out = best + (q0 + lane) * (2 * half_ld) + tb;
    floatx4 four[2];                                       // of the halves of the tiles
#pragma unroll
    for (int o = 0; o < 2; ++o) four[o] = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    auto step = [&](int t, const SweepTile<SH> &buf) {
        float top[2];
        sweep_tile<SH, 4>(buf, afr, 0, l32, h, [&](int j, const floatx16 (&acc)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float m = j & 1 ? top[i] : acc[i][15];
#pragma unroll
                for (int v = 0; v < (j & 1 ? 16 : 15); ++v) m = __builtin_elementwise_maximum(m, acc[i][v]);
                top[i] = m;
            }
            if (j & 1) {
                // lane half 0 gets query block 0's maximum over both halves' centroids, lane half 1 block 1's
                const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(top[0]), __float_as_uint(top[1]), false, false);
                floatx4 &f = four[j >> 1];
                f = floatx4{f[1], f[2], f[3], __builtin_elementwise_maximum(__uint_as_float(s[0]), __uint_as_float(s[1]))};
                if ((t & 3) == 3) *reinterpret_cast<floatx4 *>(out + (j >> 1) * half_ld + t - 3) = f;
            }
        });
    };
    for (int t = 0; t < t_end;) {
        sweep_barrier();
        if (t + 1 < t_end) issue(t + 1, buf1);
        step(t, buf0);
        if (++t == t_end) break;
        sweep_barrier();
        if (t + 1 < t_end) issue(t + 1, buf0);
        step(t, buf1);
        ++t;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no copy into LDS may outlive the workgroup
    if (t_end & 3) {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            for (int t = t_end; t & 3; ++t) four[o] = floatx4{four[o][1], four[o][2], four[o][3], -INFINITY};
            *reinterpret_cast<floatx4 *>(out + o * half_ld + (t_end & ~3)) = four[o];
        }
    }
}

// The same for up to 256 queries and below 8192 tiles (sweep_wide), where the table's bytes are what it takes: 128 queries a workgroup, a wavefront with 64 of them and half a
// tile, every fragment waited for where it is read.  One query on 2^20, 96 dimensions: 36 us (5.6 TB/s), 64 queries 46; with sweep_tile 38 and
// 48.5, whichever number of tiles a workgroup takes.
template <int SH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void coarse_minima_few_kernel(
    const _Float16 *__restrict__ Qh, const _Float16 *__restrict__ Ch, const float *__restrict__ start, float *__restrict__ best, int64_t half_ld,
    int tiles_q, int tiles_c, int tiles_per_wg)
{
    typedef const __attribute__((address_space(1))) void *gptr_t;
    typedef __attribute__((address_space(3))) void *lptr_t;
    constexpr int Dpf = SH * DK;                           // floats per row of the hi-only tables
    constexpr int SLOT = GT * ROWF;
    __shared__ __attribute__((aligned(16))) float ring[2][SH * SLOT];
    __shared__ __attribute__((aligned(16))) float cns[2][GT];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64;
    int64_t tq, group;
    if (!group_of_block(blockIdx.x, tiles_q, (tiles_c + tiles_per_wg - 1) / tiles_per_wg, tq, group)) return;
    const int tb = (int)(group * tiles_per_wg);
    int t_end = tb < tiles_c ? tiles_c - tb : 0;
    if (t_end > tiles_per_wg) t_end = tiles_per_wg;
    if (t_end <= 0) return;
    const int64_t q0 = tq * GT;

    const TileTwists<SH> twists(wave, lane);
    const float *cbase = reinterpret_cast<const float *>(Ch);
    auto issue_tile = [&](int t) {
        if (wave < 2)
            __builtin_amdgcn_global_load_lds((gptr_t)(start + (int64_t)(tb + t) * GT + wave * 64 + lane), (lptr_t)(&cns[t & 1][wave * 64]), 4, 0, 0);
        const float *src = cbase + (int64_t)(tb + t) * GT * Dpf;
        float *dst = &ring[t & 1][0];
#pragma nounroll
        for (int n = wave; n < 8 * SH; n += 4)
            __builtin_amdgcn_global_load_lds((gptr_t)(src + n * 256 + 4 * (lane ^ (int)twists.of(n))), (lptr_t)(dst + n * 256), 16, 0, 0);
    };
    issue_tile(0);
    gu32x4 afr[SH][2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const gu32x4 *row = reinterpret_cast<const gu32x4 *>(reinterpret_cast<const float *>(Qh) + (q0 + wq + i * 32 + l32) * Dpf) + 2 * h;
#pragma unroll
        for (int s = 0; s < SH; ++s) {
            afr[s][i][0] = row[s * 4 + 0];
            afr[s][i][1] = row[s * 4 + 1];
        }
    }
    float *out = best + (q0 + wq + lane) * (2 * half_ld) + (wave & 1) * half_ld + tb;
    floatx4 four = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int t = 0; t < t_end; ++t) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // this wavefront's copies of tile t (issued a tile ago) are in
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // ... and everyone's; tile t - 1's buffer is free
        if (t + 1 < t_end) issue_tile(t + 1);
        float top[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            floatx16 acc[2];
            union { floatx16 all; floatx4 part[4]; } init;
            const int rb = wc + j * 32 + l32;
            const uint32_t cb = (uint32_t)reinterpret_cast<uintptr_t>(&cns[t & 1][wc + j * 32 + 4 * h]);
            const uint32_t rsw = 4u * (uint32_t)(rb * Dpf), k0 = 16u * ((uint32_t)(2 * h) ^ tile_twist<SH>(rb)), k1 = 16u * ((uint32_t)(2 * h + 1) ^ tile_twist<SH>(rb));
#pragma unroll
            for (int s = 0; s < SH; ++s) {
                const uint32_t bs = (uint32_t)reinterpret_cast<uintptr_t>(&ring[t & 1][0]) + rsw;
                const uint32_t b0 = bs + (SH & 1 ? k0 + 64u * s : k0 ^ 64u * s), b1 = bs + (SH & 1 ? k1 + 64u * s : k1 ^ 64u * s);
                gu32x4 b[2];
                if (s == 0)
                    asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %6 offset:32\n\tds_read_b128 %2, %6 offset:64\n\tds_read_b128 %3, %6 offset:96\n\t"
                                 "ds_read_b128 %4, %7\n\tds_read_b128 %5, %8\n\ts_waitcnt lgkmcnt(0)"
                                 : "=&v"(init.part[0]), "=&v"(init.part[1]), "=&v"(init.part[2]), "=&v"(init.part[3]), "=&v"(b[0]), "=&v"(b[1])
                                 : "v"(cb), "v"(b0), "v"(b1));
                else
                    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(b[0]), "=&v"(b[1]) : "v"(b0), "v"(b1));
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, b[p]), __builtin_bit_cast(halfx8, afr[s][i][p]),
                                                                        s == 0 && p == 0 ? init.all : acc[i], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float m = acc[i][0];
#pragma unroll
                for (int v = 1; v < 16; ++v) m = __builtin_elementwise_maximum(m, acc[i][v]);
                top[i] = j == 0 ? m : __builtin_elementwise_maximum(top[i], m);
            }
            __builtin_amdgcn_sched_barrier(0);   // the next half's products start with this half's registers free
        }
        // lane half 0 gets query block 0's maximum over both halves' centroids, lane half 1 block 1's
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(top[0]), __float_as_uint(top[1]), false, false);
        four = floatx4{four[1], four[2], four[3], __builtin_elementwise_maximum(__uint_as_float(s[0]), __uint_as_float(s[1]))};
        if ((t & 3) == 3) *reinterpret_cast<floatx4 *>(out + t - 3) = four;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no copy into LDS may outlive the workgroup
    if (t_end & 3) {
        for (int t = t_end; t & 3; ++t) four = floatx4{four[1], four[2], four[3], -INFINITY};
        *reinterpret_cast<floatx4 *>(out + (t_end & ~3)) = four;
    }
}

// What the kernels after the sweep share.
struct SparseArgs {
    int64_t K, half_ld;
    int nb, P, L, cap, shift, Dp;              // cap >= 2 P: blocks a query may list; a pair is query << shift | slot
    bool direct;                               // small batches: a pair is a work item, listed by the workgroup that finds it
    const float4 *tile;
    const float2 *qlen;
    const float *qn, *qsi;                     // |q|^2, inverse scales
    const uint32_t *cmax;
    const _Float16 *Qp, *Cp;                   // hi/lo rows
    const float *cnorm, *csi;
    float *best;                               // [rows][2 half_ld] block maxima (of hard queries: smallest distances)
    uint32_t *n_flag;                          // [nq]
    int32_t *blist;                            // [nq][cap] flagged blocks, ascending
    uint32_t *rank;                            // [nq][cap] place of a pair among those of its bucket
    float *thr;                                // [nq] no distance of the P closest is larger
    uint32_t *count, *region_count;            // [N_XCD][nb], [N_XCD][K] pairs of a bucket, by query % N_XCD
    uint32_t *offset;                          // the same for the first pair of each
    uint32_t *total;                           // [0]: hard queries; [1], [2]: pairs, work items of the blocks; [3], [4]: of the regions
    uint32_t *hard;                            // [nq] the hard queries
    _Float16 *hard_rows;
    float *hard_n, *hard_si;
    uint32_t *pairs;
    uint4 *items;                              // bucket, first pair, pairs
    uint4 *head;                               // [nq][cap] of a flagged block: distances up to thr, the first one's key and centroid
    uint32_t *cand;                            // [nq][cap][64] the keys of all 64, where it is more than one
    uint32_t *keys;                            // [nq][P L] scores
    int32_t *probe_id;
    float *probe_d;
    const int32_t *nbr;
    const float *nbr_norm, *cst, *alpha;
    const uint32_t *order_inv;                 // [K] a region's bucket: its place in the order of order.hpp
};

// Takes a query's flagged blocks: counted by block, to be grouped (bucket_items_kernel), or as the work items themselves, of one pair
// each, in room for `total` of them.  Built by the whole workgroup (a barrier); word: a word of LDS.
struct PairList {
    const SparseArgs &a;
    int64_t q;
    uint32_t first = 0;
    __device__ __forceinline__ PairList(const SparseArgs &args, int64_t query, uint32_t total, uint32_t *word) : a(args), q(query)
    {
        if (!a.direct) return;
        if (threadIdx.x == 0) *word = atomicAdd(&a.total[2], total);
        __syncthreads();
        first = *word;
    }
    __device__ __forceinline__ void operator()(uint32_t at, int b) const
    {
        a.blist[q * a.cap + at] = b;
        if (a.direct) {
            a.pairs[first + at] = (uint32_t)q << a.shift | at;
            a.items[first + at] = make_uint4((uint32_t)b, first + at, 1u, 0u);
        } else {
            a.rank[q * a.cap + at] = atomicAdd(&a.count[(q % N_XCD) * a.nb + b], 1u);
        }
    }
};

// Lists the blocks of 64 that can hold one of a query's P closest centroids: a block's smallest distance lies between two ends,
// and the block is listed if its lower end does not exceed an upper bound of the P-th smallest upper end.  The ends are widened by the
// rounding of the exact distances too, by whose computed values everything that follows decides.  They are taken as distances in
// units of the product, |q|^2 - 2 G: not negative, so that their bits order like them (and not -G, whose sign changes from block to
// block: bins of equal width would be wasted on the exponents around zero).
// A thread takes NP pieces of TP tiles (2 TP blocks) of every 256 in a row, all in registers.  The bound is the P-th smallest of
// the pieces' smallest upper ends: where near blocks lie anywhere it lists 7 % more than need be, for an eighth of the keys to select
// from.  Where it lists too many (near blocks side by side) a histogram of all blocks gives a closer one; what is over cap then
// is a hard query.  Few threads a query: the selection's steps cost every wavefront the same instructions, few keys or many
// (10 000 queries x 16 384 blocks: 340 us, 425 with 1024 threads, 750 with 256 and more blocks than registers).
template <int BLOCK, int TP, int NP>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4, 8))) void flag_blocks_kernel(SparseArgs a)
{
    constexpr int NB = 2 * TP, NW = BLOCK / WAVE;
    __shared__ SelectRegs<1024> sh;
    __shared__ uint32_t base[NW * NP];
    static_assert(NP * NW <= WAVE, "a lane for a piece and wavefront");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t q = blockIdx.x;
    const float *row = a.best + q * 2 * a.half_ld;
    const int tiles = (a.nb + 1) / 2, pieces = (tiles + TP - 1) / TP;
    const float k = (float)(a.Dp + 32) * 0x1p-24f, back = 2.f * k / (0.5f - k);
    const float2 ql = a.qlen[q];
    // half a distance's rounding error, 64 u (|q|^2 + |c|^2), in units of the product (four times the measured bound of the
    // parity checks), and the low halves below fp16's range
    const float up2 = 1.f * (1 << SPARSE_HEADROOM), down2 = 1.f / (1 << SPARSE_HEADROOM), q2 = up2 * ql.x * ql.x;
    const float eps_q = fmaf(0x1p-18f, q2, 0x1p-20f * ql.x), eps_c = fmaf(k, ql.x, ql.y), eps_d = ql.x + ql.y;
    uint32_t far[NP][NB];                                        // upper ends
    float gap[NP];                                               // ... to the lower ones, the largest of a piece
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int pc = tid + u * BLOCK, t0 = pc < pieces ? pc * TP : (pieces - 1) * TP;   // (every thread loads)
        float x[2][TP];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const float *src = row + o * a.half_ld + t0;
            if constexpr (TP == 4) {
                const float4 w = *reinterpret_cast<const float4 *>(src);
                x[o][0] = w.x; x[o][1] = w.y; x[o][2] = w.z; x[o][3] = w.w;
            } else if constexpr (TP == 2) {
                const float2 w = *reinterpret_cast<const float2 *>(src);
                x[o][0] = w.x; x[o][1] = w.y;
            } else {
                x[o][0] = src[0];
            }
        }
        gap[u] = 0.f;
#pragma unroll
        for (int i = 0; i < TP; ++i) {
            const float4 tl = a.tile[t0 + i < tiles ? t0 + i : tiles - 1];
            const float eps = fmaf(eps_c, tl.x, fmaf(eps_d, tl.y, fmaf(0x1p-18f * down2 * tl.x, tl.x, eps_q))), low = back * tl.z;
            const bool known = eps < INFINITY;
            gap[u] = fmaxf(gap[u], known ? 2.f * (2.f * eps - low) : INFINITY);
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const float d = known ? fmaxf(fmaf(-2.f, x[o][i], fmaf(2.f, eps - low, q2)), 0.f) : INFINITY;
                far[u][2 * i + o] = pc < pieces && 2 * (t0 + i) + o < a.nb ? __float_as_uint(d) : NO_KEY;
            }
        }
    }
    uint32_t least[NP], pivot, need;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        least[u] = far[u][0];
#pragma unroll
        for (int i = 1; i < NB; ++i) least[u] = far[u][i] < least[u] ? far[u][i] : least[u];
    }
    // (fewer pieces than P: everything is listed that is not over cap)
    float limit = INFINITY;
    if (a.P <= pieces) {
        block_select_runs<BLOCK>(least, NP, (uint32_t)a.P, sh, pivot, need);
        limit = __uint_as_float(pivot);
    }
    uint32_t flags[NP], total;
    auto flag = [&]() {                                           // which blocks, and the places of this thread's first in every piece
        uint32_t word[3] = {0, 0, 0};
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            flags[u] = 0;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const float f = __uint_as_float(far[u][i]);      // (a block without an end: listed; a NaN is no block)
                if (f - gap[u] <= limit || f == INFINITY) flags[u] |= 1u << i;
            }
            word[u / 3] |= (uint32_t)__popc(flags[u]) << (10 * (u % 3));
        }
        uint32_t inc[3];
#pragma unroll
        for (int w = 0; w < 3; ++w) inc[w] = wave_inclusive_scan(word[w]);   // (at most 64 * 8 of a piece: 10 bits)
        if (lane == WAVE - 1) {
#pragma unroll
            for (int u = 0; u < NP; ++u) base[u * NW + wave] = inc[u / 3] >> (10 * (u % 3)) & 1023u;
        }
        __syncthreads();
        const uint32_t in = lane < NW * NP ? base[lane] : 0u, all = wave_inclusive_scan(in);
        total = (uint32_t)__builtin_amdgcn_readlane((int)all, WAVE - 1);
        uint32_t at[NP];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int from = u * NW + wave;                       // pieces are in order of u, then of the threads
            at[u] = (uint32_t)__builtin_amdgcn_readlane((int)(all - in), from) + ((inc[u / 3] - word[u / 3]) >> (10 * (u % 3)) & 1023u);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NP; ++u) least[u] = at[u];
    };
    flag();
    if (total > (uint32_t)a.cap && limit < INFINITY && limit > 0.f) {          // uniform
        // bins of equal width up to the bound; its new value is the end of the bin that the P-th smallest falls into
        const float per = 1024.f / limit;
        for (int i = tid; i < 1024; i += BLOCK) sh.hist[i] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NP; ++u)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const float f = __uint_as_float(far[u][i]);
                const int bin = (int)fminf(f * per, 1023.f);
                if (f <= limit) atomicAdd(&sh.hist[bin], 1u);
            }
        __syncthreads();
        constexpr int PER = 1024 / BLOCK;
        uint32_t c[PER], s = 0, all;
#pragma unroll
        for (int j = 0; j < PER; ++j) { c[j] = sh.hist[PER * tid + j]; s += c[j]; }
        uint32_t cum = block_exclusive_scan<BLOCK>(s, sh.scan, all);
        if (cum < (uint32_t)a.P && cum + s >= (uint32_t)a.P) {
            int bin = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                if (cum < (uint32_t)a.P) bin = PER * tid + j;
                cum += c[j];
            }
            sh.pick[0] = (uint32_t)bin;
        }
        __syncthreads();
        limit = fminf(limit, (float)(sh.pick[0] + 1u) / per * (1.f + 0x1p-20f));
        flag();
    }
    if (total > (uint32_t)a.cap || !(ql.x < INFINITY)) {                       // uniform
        if (tid == 0) {
            const uint32_t r = atomicAdd(&a.total[0], 1u);
            a.n_flag[q] = 0;
            a.hard[r] = (uint32_t)q;
            a.hard_n[r] = a.qn[q];
            a.hard_si[r] = a.qsi[q];
            sh.pick[0] = r;
        }
        __syncthreads();
        const int64_t r = sh.pick[0], chunks = a.Dp / 4;                     // 16-byte pieces of a row
        for (int c = tid; c < chunks; c += BLOCK) reinterpret_cast<gu32x4 *>(a.hard_rows)[r * chunks + c] = reinterpret_cast<const gu32x4 *>(a.Qp)[q * chunks + c];
        return;
    }
    const PairList put(a, q, total, &sh.pick[0]);
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        uint32_t at = least[u];
        while (flags[u]) {
            const int b = 2 * TP * (tid + u * BLOCK) + __builtin_ctz(flags[u]);
            put(at++, b);
            flags[u] &= flags[u] - 1;
        }
    }
    if (tid == 0) {
        a.n_flag[q] = total;
        const int shc = hi_scale(*a.cmax);
        const float two_g = __builtin_amdgcn_ldexpf(limit - q2, SPARSE_HEADROOM - 2 * shc), n = a.qn[q];
        const float d = n + two_g + 0x1p-21f * (n + fabsf(two_g));
        a.thr[q] = limit < INFINITY ? fmaxf(d, 0.f) : INFINITY;
    }
}

// ---- hard queries: block minima of their exact distances.  Loops over what there is, nearly always nothing ----
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void hard_minima_kernel(SparseArgs a)
{
    __shared__ __attribute__((aligned(16))) float ops0[DBUF];
    __shared__ __attribute__((aligned(16))) float ops1[DBUF];
    __shared__ __attribute__((aligned(16))) float cns[GT];
    const int64_t n = a.total[0], tiles_h = (n + GT - 1) / GT, tiles_c = (a.K + GT - 1) / GT;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64, l32 = lane & 31, h = lane >> 5;
    for (int64_t item = blockIdx.x; item < tiles_h * tiles_c; item += gridDim.x) {
        const int64_t q0 = item % tiles_h * GT, t = item / tiles_h, c0 = t * GT;
        __syncthreads();                                                   // everyone has read the norms of the last tile
        if (threadIdx.x < GT) cns[threadIdx.x] = c0 + threadIdx.x < a.K ? a.cnorm[c0 + threadIdx.x] : 0.f;
        floatx16 acc[2][2];
        gemm_tile(a.hard_rows, n, q0, a.Cp, a.K, c0, a.Dp, ops0, ops1, acc);
        const float m2c = -2.f * a.csi[0];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t r = q0 + wq + i * 32 + l32;
            const float qr = r < n ? a.hard_n[r] : 0.f, m2 = r < n ? m2c * a.hard_si[r] : 0.f;
            float m = INFINITY;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int cl = wc + j * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (c0 + cl < a.K) m = fminf(m, fmaxf(fmaf(m2, acc[i][j][v], qr + cns[cl]), 0.f));
                }
            m = fminf(m, __shfl_xor(m, 32, WAVE));
            if (h == 0 && r < n) a.best[a.hard[r] * 2 * a.half_ld + (wave & 1) * a.half_ld + t] = m;
        }
    }
}

// flag_blocks_kernel for what hard_minima_kernel wrote: by the rule of probe_select_kernel, at most 2 P - 1 blocks
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void hard_flag_kernel(SparseArgs a)
{
    __shared__ SelectRegs<1024> sh;
    constexpr int N = 16;
    const uint32_t n = a.total[0];
    const int ipt = run_length<BLOCK>(a.nb), i0 = threadIdx.x * ipt;
    for (uint32_t at = blockIdx.x; at < n; at += gridDim.x) {
        __syncthreads();
        const int64_t q = a.hard[at];
        const float *row = a.best + q * 2 * a.half_ld;
        uint32_t kv[N], pivot, need;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int b = j < ipt && i0 + j < a.nb ? i0 + j : 0;
            const uint32_t key = float_key(row[(b & 1) * a.half_ld + (b >> 1)]);
            kv[j] = j < ipt && i0 + j < a.nb ? key : NO_KEY;
        }
        block_select_runs<BLOCK>(kv, ipt, a.P < a.nb ? (uint32_t)a.P : (uint32_t)a.nb, sh, pivot, need);
        // (at most P below the pivot and P more, or all blocks: counted first)
        const uint32_t total = block_emit_runs<BLOCK>(kv, ipt, pivot, (uint32_t)a.P, sh.scan, [](uint32_t, int, uint32_t) {});
        const PairList put(a, q, total, &sh.pick[0]);
        block_emit_runs<BLOCK>(kv, ipt, pivot, (uint32_t)a.P, sh.scan, [&](uint32_t pos, int b, uint32_t) { put(pos, b); });
        if (threadIdx.x == 0) {
            a.n_flag[q] = total;
            a.thr[q] = a.nb < a.P ? INFINITY : key_float(pivot);
        }
    }
}

// ---- pairs in the order of their buckets (blocks or regions) ----
constexpr int PAIR_Q = 32;   // queries of a work item

// A bucket's pairs are counted as N_XCD parts: workgroup q counts in part q % N_XCD, so that the counters that an XCD adds to stay
// in its L2 (one part for all: 10 000 queries, 1024 blocks, 66 listed: 154 us for flag_blocks_kernel, 62 so).
// First pair of every part of every bucket and the work items.  The order of the buckets among each other does not matter: a
// workgroup adds up its 1024 and takes room for them with one atomic.
__global__ __launch_bounds__(1024) void bucket_items_kernel(const uint32_t *__restrict__ count, int64_t n, uint32_t *__restrict__ total,
                                                            uint32_t *__restrict__ offset, const uint32_t *__restrict__ order, uint4 *__restrict__ items)
{
    __shared__ uint32_t scan[16], base[2];
    const int64_t b = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    uint32_t part[N_XCD], c = 0;
#pragma unroll
    for (int x = 0; x < N_XCD; ++x) {
        part[x] = b < n ? count[x * n + b] : 0u;
        c += part[x];
    }
    const uint32_t m = (c + PAIR_Q - 1) / PAIR_Q;
    uint32_t pairs, work;
    const uint32_t at = block_exclusive_scan<1024>(c, scan, pairs), it = block_exclusive_scan<1024>(m, scan, work);
    if (threadIdx.x == 0) {
        base[0] = pairs ? atomicAdd(&total[0], pairs) : 0u;
        base[1] = work ? atomicAdd(&total[1], work) : 0u;
    }
    __syncthreads();
    if (b >= n) return;
    uint32_t first = base[0] + at;
#pragma unroll
    for (int x = 0; x < N_XCD; ++x) {
        offset[x * n + b] = first;
        first += part[x];
    }
    const uint32_t name = order && c ? order[b] : (uint32_t)b;
    for (uint32_t u = 0; u < m; ++u) {
        const uint32_t left = c - u * PAIR_Q;
        items[base[1] + it + u] = make_uint4(name, base[0] + at + u * PAIR_Q, left < PAIR_Q ? left : PAIR_Q, 0u);
    }
}

// slot s of query q (n_flag[q] of them, or P where there is none) to its place
__global__ __launch_bounds__(256) void place_pairs_kernel(const int32_t *__restrict__ bucket, const uint32_t *__restrict__ rank, int64_t nq, int width,
                                                          int64_t buckets, int rank_ld, int shift, const uint32_t *__restrict__ n_flag,
                                                          const uint32_t *__restrict__ inv, const uint32_t *__restrict__ offset, uint32_t *__restrict__ pairs)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nq * width) return;
    const int64_t q = i / width;
    const int s = (int)(i - q * width);
    if (n_flag && (uint32_t)s >= n_flag[q]) return;
    const int64_t b = inv ? (int64_t)inv[bucket[i]] : (int64_t)bucket[i];
    pairs[offset[(q % N_XCD) * buckets + b] + rank[q * rank_ld + s]] = (uint32_t)q << shift | (uint32_t)s;
}

// The exact distances of up to 32 queries (a work item) to 64 rows of the table, a step.  REGION: the rows are neighbours of
// region `bucket` and the result is the score of Eq. (7) as an ordered key; else they are the 64 centroids of a block.
// Products and their order are those of gemm_tile.  A wavefront takes `run` = PAIR_RUN steps in a row; rows are copied to LDS
// directly, six such workgroups a compute unit (fewer steps where there are not enough for all).  While a step's results are written the rows of the next are on their way, and
// before them the next one's pairs and neighbours, and before those the item after that: each depends on the one before, and
// one step a workgroup waited 2 of its 4.7 us for them.  The results pass through LDS as they come, PAIR_OUT queries at a
// time, and a lane a row makes distances of them for the queries there are (three of 32 for the regions of 10 000 queries on
// 2^20).
constexpr int PAIR_RUN = 8, PAIR_OUT = 8;

inline unsigned pair_grid(int64_t items, int chunks, int run)
{
    const int64_t share = (items + N_XCD - 1) / N_XCD * chunks;
    return (unsigned)((share + run - 1) / run * N_XCD);
}

// WHOLE: every step has 64 rows (L a multiple of 64).
template <int STAGES, bool REGION, bool WHOLE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void pair_distance_kernel(SparseArgs a, const uint32_t *__restrict__ n_items, int chunks, int run)
{
    typedef const __attribute__((address_space(1))) void *gptr_t;
    typedef __attribute__((address_space(3))) void *lptr_t;
    static_assert(STAGES % 2 == 0, "two stages at a time");
    constexpr int Dp = STAGES * DK;                                        // floats per row
    constexpr int OLD = BMW + 4;                                           // row stride of the results in LDS
    __shared__ __attribute__((aligned(16))) float rows[STAGES * BMW * ROWF];
    __shared__ __attribute__((aligned(16))) float out[PAIR_OUT * OLD];
    // workgroup b runs on XCD b % N_XCD: an XCD takes items in a row, whose rows (those of a block; the neighbours that regions
    // side by side have in common) it then finds in its L2
    const uint32_t items = *n_items, share = (items + N_XCD - 1) / N_XCD;
    const uint32_t i_end = (blockIdx.x % N_XCD + 1) * share < items ? (blockIdx.x % N_XCD + 1) * share : items;
    const uint32_t begin = blockIdx.x % N_XCD * share * chunks + blockIdx.x / N_XCD * run;
    uint32_t end = i_end * chunks;
    if (begin >= end) return;                                              // (also where blockIdx.x % N_XCD * share > items)
    if (end - begin > (uint32_t)run) end = begin + run;
    const int lane = threadIdx.x, l32 = lane & 31, h = lane >> 5, mask = (1 << a.shift) - 1;
    const int width = REGION ? a.L : BMW;
    const float m2c = -2.f * a.csi[0];
    struct Ids { uint32_t bucket; int n, l0, nl; uint32_t pair; int32_t row; };   // a step: all but pair and row uniform
    struct Ops { float cn, cs, al, qr, si, pd; };                          // of row `lane`, of the region, of query l32
    // (an index that the compiler does not know to be uniform: it would read the item into scalar registers, and wait for it, where it is
    // asked for, and not where it is used)
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));
    auto item_of = [&](uint32_t t) { return a.items[(t < end ? t : end - 1) / (uint32_t)chunks + zero]; };
    auto ids_of = [&](uint32_t t, uint4 item) {
        Ids s;
        s.bucket = (uint32_t)__builtin_amdgcn_readfirstlane((int)item.x);
        s.n = __builtin_amdgcn_readfirstlane((int)item.z);
        s.l0 = (int)((t < end ? t : end - 1) % (uint32_t)chunks) * BMW;
        s.nl = WHOLE || width - s.l0 > BMW ? BMW : width - s.l0;
        s.pair = a.pairs[(uint32_t)__builtin_amdgcn_readfirstlane((int)item.y) + (l32 < s.n ? l32 : 0)];   // (columns past n: the first query again)
        s.row = REGION ? a.nbr[(int64_t)s.bucket * a.L + s.l0 + (lane < s.nl ? lane : 0)] : (int32_t)(s.bucket * BMW) + lane;   // (the packed table has whole tiles of rows)
        return s;
    };
    gu32x4 qf[STAGES][2];
    const int f = (lane & 7) ^ (lane >> 3);                                // chunk of two stages that this lane copies
    const float *src[8];                                                   // its rows of the step whose rows are copied, their query's row
    const gu32x4 *qrow;
    auto aim = [&](const Ids &s) {
#pragma unroll
        for (int g = 0; g < 8; ++g)
            src[g] = reinterpret_cast<const float *>(a.Cp) + (int64_t)__shfl(s.row, 8 * g + (lane >> 3), WAVE) * Dp + f * 4;
        qrow = reinterpret_cast<const gu32x4 *>(reinterpret_cast<const float *>(a.Qp) + (int64_t)(s.pair >> a.shift) * Dp) + 2 * h;
    };
    // two stages, whole 128-byte lines of 8 rows a load: with a stage at a time (16 rows, half a line of each) the loads of the other
    // halves waited for the lines, 2.41 ms for 10 000 queries on 2^20, P = 256, and 2.02 so
    auto copy_stages = [&](const Ids &s, int c) {
#pragma unroll
        for (int g = 0; g < 8; ++g)
            if (WHOLE || 8 * g < s.nl) __builtin_amdgcn_global_load_lds((gptr_t)(src[g] + c * DK), (lptr_t)(rows + c * (BMW * ROWF) + g * 256), 16, 0, 0);
    };
    auto query_stage = [&](const Ids &s, int c) {
        if (l32 < s.n) {                                                   // (columns past n: whatever is there, not stored)
            qf[c][0] = qrow[c * 4 + 0];
            qf[c][1] = qrow[c * 4 + 1];
        }
    };
    auto operands = [&](const Ids &s) {
        Ops o;
        const int64_t q = s.pair >> a.shift;
        o.qr = a.qn[q];
        o.si = a.qsi[q];                                                   // (no arithmetic on them here: it would wait)
        if (REGION) {
            const int64_t at = (int64_t)s.bucket * a.L + s.l0 + (lane < s.nl ? lane : 0);
            o.cn = a.nbr_norm[at];
            o.cs = a.cst[at];
            o.al = a.alpha[s.bucket + zero];
            o.pd = a.probe_d[q * a.P + (s.pair & (uint32_t)mask)];
        } else {
            const int64_t c = (int64_t)s.bucket * BMW + lane;
            o.cn = a.cnorm[c < a.K ? c : a.K - 1];
            o.cs = o.al = 0.f;
            o.pd = a.thr[q];
        }
        return o;
    };
    uint32_t t = begin;
    Ids now = ids_of(t, item_of(t));
    aim(now);
#pragma unroll
    for (int c = 0; c < STAGES; ++c) {
        if (!(c & 1)) copy_stages(now, c);
        qf[c][0] = qf[c][1] = gu32x4{0, 0, 0, 0};
        query_stage(now, c);
    }
    Ops ops = operands(now);
    Ids next = ids_of(t + 1, item_of(t + 1));
    uint4 item = item_of(t + 2);
    while (true) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        wave_sync();
        const bool more = t + 1 < end;                                     // (uniform)
        gu32x4 b[2][2][2];                                                 // of two stages
        auto read_stage = [&](int c) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = j * 32 + l32;
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    b[c & 1][j][p] = *reinterpret_cast<const gu32x4 *>(&rows[(c >> 1) * (2 * BMW * ROWF) + r * (2 * ROWF) + (((4 * (c & 1) + 2 * h + p) ^ (r & 7)) << 2)]);
            }
        };
        read_stage(0);
        floatx16 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
        const bool both = WHOLE || now.nl > 32;                                     // (uniform)
        const Ids is = now;
        const Ops o = ops;
        if (more) {
            aim(next);
            ops = operands(next);
        }
#pragma unroll
        for (int c = 0; c < STAGES; ++c) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // two stages' rows have been read: the next step's may come
            if (more && (c & 1)) copy_stages(next, c - 1);
            if (c + 1 < STAGES) read_stage(c + 1);
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                acc[0] = mfma3(b[c & 1][0], qf[c], acc[0], e);
                if (both) acc[1] = mfma3(b[c & 1][1], qf[c], acc[1], e);
            }
            if (more) query_stage(next, c);
        }
        if (more) {
            now = next;
            next = ids_of(t + 2, item);
            item = item_of(t + 3);
        }
        uint4 head = make_uint4(0u, 0u, 0u, 0u);                           // of query `lane`
        for (int i0 = 0; i0 < is.n; i0 += PAIR_OUT) {
            if ((l32 & ~(PAIR_OUT - 1)) == i0) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *reinterpret_cast<float4 *>(&out[(l32 & (PAIR_OUT - 1)) * OLD + j * 32 + 8 * g + 4 * h]) =
                            make_float4(acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]);
            }
            wave_sync();
            float v[PAIR_OUT];
#pragma unroll
            for (int u = 0; u < PAIR_OUT; ++u) v[u] = out[u * OLD + lane];
#pragma unroll
            for (int u = 0; u < PAIR_OUT; ++u) {
                const int i = i0 + u;
                if (i >= is.n) break;                                      // (uniform)
                auto of = [&](float v) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), i)); };
                const uint32_t pr = (uint32_t)__builtin_amdgcn_readlane((int)is.pair, i);
                const int64_t qi = pr >> a.shift, s = pr & (uint32_t)mask;
                const float d = fmaxf(fmaf(m2c * of(o.si), v[u], of(o.qr) + o.cn), 0.f), pd = of(o.pd);
                if (REGION) {
                    const uint32_t key = float_key(fmaf(o.al, d, fmaf(1.f - o.al, pd, o.cs)));
                    if (lane < is.nl) a.keys[(qi * a.P + s) * a.L + is.l0 + lane] = key;
                } else {
                    const uint32_t key = (int64_t)is.bucket * BMW + lane < a.K ? float_key(d) : NO_KEY;
                    const uint64_t m = __ballot(key <= float_key(pd));
                    const int first = m ? __builtin_ctzll(m) : 0;
                    const uint32_t kf = (uint32_t)__builtin_amdgcn_readlane((int)key, first);
                    if (lane == i) head = make_uint4((uint32_t)__popcll(m), kf, is.bucket * BMW + (uint32_t)first, 0u);
                    if (m & (m - 1)) a.cand[(qi * a.cap + s) * BMW + lane] = key;   // (uniform; one is usual)
                }
            }
            wave_sync();                                                   // (read: the next queries' results may come)
        }
        if (!REGION && lane < is.n) a.head[(int64_t)(is.pair >> a.shift) * a.cap + (is.pair & (uint32_t)mask)] = head;
        if (!more) break;
        ++t;
    }
}

// The P closest of the distances of a query's flagged blocks by (distance, id), ascending in id.  A thread takes two blocks,
// nearly all of which have one distance that matters; the others' rows are read by a wavefront each.  (All rows read and filtered
// here, 16 a wavefront at a time: 440 us for 10 000 queries and P = 256, 130 so.)  Dynamic LDS: 2 PICK_CAP words.
constexpr int PICK_CAP = 2048, PICK_BLOCK = 256;

__global__ __launch_bounds__(PICK_BLOCK) void probe_pick_kernel(SparseArgs a)
{
    constexpr int BLOCK = PICK_BLOCK;
    __shared__ SelectRegs<1024> sh;
    __shared__ uint2 more[2 * BLOCK];                                       // blocks with several: slot, first place
    __shared__ uint32_t n_more;
    SelectShared &sh_mem = *reinterpret_cast<SelectShared *>(&sh);          // (only where more survive than fit)
    static_assert(sizeof(SelectShared) <= sizeof(sh), "the same place");
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    uint32_t *sk = dyn;
    int32_t *si = reinterpret_cast<int32_t *>(dyn + PICK_CAP);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, P = a.P;
    const int64_t q = blockIdx.x;
    const int n = (int)a.n_flag[q];
    const uint4 *head = a.head + q * a.cap;
    const uint32_t *cand = a.cand + q * a.cap * BMW;
    const uint32_t tf = float_key(a.thr[q]);
    auto put = [&](uint32_t pos, int32_t id, uint32_t key) {
        a.probe_id[q * P + pos] = id;
        a.probe_d[q * P + pos] = key_float(key);
        if (a.direct) {
            a.pairs[q * P + pos] = (uint32_t)q << a.shift | pos;
            a.items[q * P + pos] = make_uint4((uint32_t)id, (uint32_t)(q * P + pos), 1u, 0u);
        } else {
            a.rank[q * a.cap + pos] = atomicAdd(&a.region_count[(q % N_XCD) * a.K + a.order_inv[id]], 1u);
        }
    };
    if (a.direct && tid == 0) atomicAdd(&a.total[4], (uint32_t)P);
    uint4 h[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) h[u] = head[2 * tid + u < n ? 2 * tid + u : 0];
    if (tid == 0) n_more = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) h[u].x = 2 * tid + u < n ? h[u].x : 0u;
    uint32_t total;
    uint32_t at = block_exclusive_scan<BLOCK>(h[0].x + h[1].x, sh.scan, total);
    uint32_t pivot, need;
    if (total > (uint32_t)PICK_CAP || total < (uint32_t)P) {                // uniform; the second cannot happen
        const int64_t nc = (int64_t)n * BMW;
        __syncthreads();
        auto key = [&](int64_t v) {
            const uint4 w = head[v >> 6];
            return w.x == 0 ? NO_KEY : w.x > 1 ? cand[v] : (w.z & 63u) == (uint32_t)(v & 63) ? w.y : NO_KEY;
        };
        block_radix_select<BLOCK>(key, nc, (uint32_t)P, sh_mem, pivot, need);
        block_emit_selected<BLOCK>(key, nc, (uint32_t)P, pivot, need, sh_mem,
                                   [&](uint32_t pos, int64_t v, uint32_t k) { put(pos, a.blist[q * a.cap + (v >> 6)] * BMW + (int)(v & 63), k); });
        return;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (h[u].x == 1) {
            sk[at] = h[u].y;
            si[at] = (int32_t)h[u].z;
        } else if (h[u].x > 1) {
            more[atomicAdd(&n_more, 1u)] = make_uint2((uint32_t)(2 * tid + u), at);
        }
        at += h[u].x;
    }
    __syncthreads();
    const int nm = (int)n_more;
    for (int m0 = wave * 4; m0 < nm; m0 += BLOCK / WAVE * 4) {              // four rows on their way at a time
        uint2 w[4];
        uint32_t key[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            w[u] = more[m0 + u < nm ? m0 + u : m0];
            key[u] = cand[(int64_t)w[u].x * BMW + lane];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint64_t m = m0 + u < nm ? __ballot(key[u] <= tf) : 0ull;
            if (m >> lane & 1u) {
                const uint32_t o = w[u].y + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                sk[o] = key[u];
                si[o] = a.blist[q * a.cap + w[u].x] * BMW + lane;
            }
        }
    }
    __syncthreads();
    static_assert(PICK_CAP <= 8 * BLOCK, "items of a thread");
    uint32_t kv[8];
    const int ipt = run_length<BLOCK>((int)total);
    load_run<BLOCK>(sk, (int)total, kv, [](uint32_t w) { return w; });
    block_select_runs<BLOCK>(kv, ipt, (uint32_t)P, sh, pivot, need);
    block_emit_runs<BLOCK>(kv, ipt, pivot, need, sh.scan, [&](uint32_t pos, int i, uint32_t k) { put(pos, si[i], k); });
}

}  // namespace ivf
