// Nearest codeword of every block of a displacement (Section 2: product quantiser), the per-point constant of
// Eq. (6), and the sums of the codebook training.
//
// The nearest codeword is decided on the matrix units, with a proof per decision.  <x, c> - |c|^2 / 2 is formed for
// all 256 codewords as fp16 products of operands split into a high and a low half (22 bits, accumulated in fp32); a
// point whose best value leads the others by more than twice the error bound has its answer, the others (about
// one in a thousand) are decided by the whole wavefront with the chain of fused multiply-adds over the differences
// that defines the result.  The codes are therefore those of that chain, the lowest index on ties.  A codeword equal to
// one before it (a codebook that starts from rows may hold hundreds) can never be the answer and is left out, or every point
// near it would be one of the others: 300 000 x 96 rows of 100 kinds, 16 quantisers, one training round 0.72 ms, 2.24
// with the copies (2.08 with a thread a point).
#pragma once
#include "coarse.hpp"

namespace ivf {

// A codeword of DS components in LDS: CH pieces of 8 fp16 (high halves) and CH of 8 (low halves).  -|c|^2 / 2 takes
// two more slots (high and low): those the last piece has left over, or a word of its own.
template <int DS>
struct PqRow {
    static constexpr int CH = (DS + 7) / 8;
    static constexpr int LAST = DS - 8 * (CH - 1);        // components in the last piece
    static constexpr bool ROOM = LAST <= 6;
    static constexpr int GROUP = DS == 4 ? 4 : DS == 6 ? 2 : 1;   // quantisers whose components are loaded together
    static constexpr int bytes = 256 * (32 * CH + (ROOM ? 0 : 4));   // of a quantiser in LDS
};

constexpr int PQ_LDS_MAX = 150 * 1024;

typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at any float's address
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));

// (two of them in a row are one instruction; of a number and what is no number, the latter)
__device__ __forceinline__ float larger(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// quantisers of one workgroup (their codewords stay in LDS): all of them, or a multiple of 4
inline int pq_per_group(int M, int quantiser_bytes)
{
    const int g = PQ_LDS_MAX / quantiser_bytes;
    return M <= g ? M : g & ~3;
}

// E and MU are [n][M * DS] fp32 (MU == NULL: codes only); grid (workgroups, groups of Mg quantisers; one group when MU
// is given).  Also t = 2<mu, r> + ||r||^2 of Eq. (6), a chain over the components in order, and its nearest entry
// of const_table, the lowest index on ties.
//
// A wavefront takes 64 points as two blocks of 32: v_mfma_f32_32x32x16_f16 with 32 codewords as the rows and 32 points
// as the columns.  Lane half 0 feeds the high halves of its point's 8 components and half 1 the low halves, against
// the codeword's high halves in both lane halves, then against its low halves: two products a piece of 8
// components, and the points' operands are built once for all 256 codewords, each lane those of its own point (a swap of lane
// halves brings them where they belong).  The vector units look for the four codewords in a row (a lane's quarter of 16) with
// the largest value and for the second largest of such fours: five instructions a four, where the largest and the second largest
// value with their numbers took three a value.  Which of the four it is is decided by dot products of the same halves, from
// LDS, a point a lane, and within the same bound.  10^6 points x 96 components, 16 quantisers: 0.375 ms, 0.575 with three
// instructions a value and every point packed by two lanes from words loaded one by one (1.48 ms with a thread a point
// that walks all codewords in LDS).  Bound by the vector and matrix instructions, which overlap only in part here: 40 of the former
// and 4 of the latter take 97 ns on a SIMD with four wavefronts, 72 and 62 alone; a tile takes 119.  Eights instead of fours (13
// instructions a block and tile instead of 20, twice the dot products) 0.385 ms; the codewords of a tile read ahead 0.38; two
// tiles at a time 0.41.
template <int DS>
__global__ __launch_bounds__(1024) void pq_encode_kernel(
    const float *__restrict__ E, const float *__restrict__ MU, int64_t n, int M, int Mg,
    const float *__restrict__ codebook, const float *__restrict__ const_table,
    uint8_t *__restrict__ out_codes, uint8_t *__restrict__ out_byte, float *__restrict__ out_t)
{
    typedef PqRow<DS> R;
    constexpr int CH = R::CH, G = R::GROUP;
    extern __shared__ __attribute__((aligned(16))) unsigned char pq_lds[];
    __shared__ float tab[256];
    __shared__ float cmax_s[64];                           // largest |c'|^2 of a quantiser (scaled), NaN: decide by the chain
    __shared__ float scale_s[64];                           // power of two that takes its largest component to below 1
    __shared__ float xmax_s[64];                            // |x'|^2 from which on the chain may overflow
    __shared__ uint32_t copy_s[64][8];                      // its codewords that are equal to one before them, a word a tile
    __shared__ uint32_t copies_s[64];                       // whether there are any
    __shared__ int tab_sorted;
    gu32x4 *rows = reinterpret_cast<gu32x4 *>(pq_lds);      // [Mg][CH][high, low][256]
    uint32_t *norms = reinterpret_cast<uint32_t *>(rows + (size_t)Mg * CH * 512);   // [Mg][256], only without ROOM
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int D = M * DS;
    const int m0 = blockIdx.y * Mg, mn = M - m0 < Mg ? M - m0 : Mg;

    if (tid == 0) tab_sorted = 1;
    if (tid < 256) tab[tid] = const_table ? const_table[tid] : 0.f;
    __syncthreads();
    if (const_table && tid < 255 && !(tab[tid] <= tab[tid + 1])) tab_sorted = 0;
    for (int m = wave; m < mn; m += 16) {                   // a wavefront packs a quantiser, four codewords a lane
        const float *cb = codebook + (int64_t)(m0 + m) * 256 * DS;
        float cw[4][DS];                                    // codewords lane, lane + 64, ...
        float big = 0.f;
        bool odd = false;                                   // an infinity or not a number among them
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int t = 0; t < DS; ++t) {
                cw[k][t] = cb[(lane + k * WAVE) * DS + t];
                big = fmaxf(big, fabsf(cw[k][t]));
                odd = odd || !(fabsf(cw[k][t]) < INFINITY);
            }
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) big = fmaxf(big, __shfl_xor(big, o, WAVE));
        const int ec = __builtin_amdgcn_frexp_expf(big);    // components scaled to below 1
        // The first codeword of every hash value, in the place of the rows that are packed below, and whether the others
        // with that value are equal to it (one that is equal to a codeword which is not the first stays in: no harm).
        uint32_t *first = reinterpret_cast<uint32_t *>(rows + (size_t)m * CH * 512), hash[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) first[lane + k * WAVE] = 0xFFFFFFFFu;
        wave_sync();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            hash[k] = 0;
#pragma unroll
            for (int t = 0; t < DS; ++t) hash[k] = (hash[k] << 7 | hash[k] >> 25) ^ __float_as_uint(cw[k][t] + 0.f);   // (-0 is 0)
            hash[k] = hash[k] * 0x9E3779B1u >> 24;
            atomicMin(&first[hash[k]], (uint32_t)(lane + k * WAVE));
        }
        wave_sync();
        uint64_t any = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int f = (int)first[hash[k]];
            bool same = f < lane + k * WAVE;
            if (same) {
#pragma unroll
                for (int t = 0; t < DS; ++t) same = same && cw[k][t] == cb[f * DS + t];
            }
            const uint64_t w = __ballot(same);
            any |= w;
            if (lane == 0) {
                copy_s[m][2 * k] = (uint32_t)w;
                copy_s[m][2 * k + 1] = (uint32_t)(w >> 32);
            }
        }
        if (lane == 0) copies_s[m] = any != 0;
        wave_sync();
        float cm = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = lane + k * WAVE;
            float n2 = 0.f;
            _Float16 hi[CH * 8], lo[CH * 8];
#pragma unroll
            for (int t = 0; t < CH * 8; ++t) {
                const float v = t < DS ? __builtin_amdgcn_ldexpf(cw[k][t < DS ? t : 0], -ec) : 0.f;
                n2 = fmaf(v, v, n2);
                hi[t] = (_Float16)v;
                lo[t] = (_Float16)(v - (float)hi[t]);
            }
            cm = fmaxf(cm, n2);
            const float nh = -0.5f * n2;                     // (|c'|^2 / 2 <= 8)
            const _Float16 nhi = (_Float16)nh, nlo = (_Float16)(nh - (float)nhi);
            if (R::ROOM) {
                hi[CH * 8 - 2] = nhi;
                hi[CH * 8 - 1] = nlo;
            } else {
                const halfx2 p = {nhi, nlo};
                norms[m * 256 + j] = __builtin_bit_cast(uint32_t, p);
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                halfx8 a, b;
#pragma unroll
                for (int t = 0; t < 8; ++t) { a[t] = hi[8 * q + t]; b[t] = lo[8 * q + t]; }
                rows[((m * CH + q) * 2 + 0) * 256 + j] = __builtin_bit_cast(gu32x4, a);
                rows[((m * CH + q) * 2 + 1) * 256 + j] = __builtin_bit_cast(gu32x4, b);
            }
        }
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) cm = fmaxf(cm, __shfl_xor(cm, o, WAVE));
        if (__any(odd) || ec < -40 || ec > 55) cm = NAN;     // the chain's own under- and overflows decide there
        if (lane == 0) {
            cmax_s[m] = cm;
            scale_s[m] = __builtin_amdgcn_ldexpf(1.f, ec < -40 ? 40 : ec > 55 ? -55 : -ec);
            xmax_s[m] = __builtin_amdgcn_ldexpf(1.f, 2 * (55 - ec));
        }
    }
    __syncthreads();
    uint32_t keep = ~31u, keep4 = ~3u;                       // (in registers, so that masking and index are one instruction)
    asm volatile("" : "+v"(keep), "+v"(keep4));
    const bool sorted = tab_sorted != 0;
    const bool words = (M & 3) == 0 && (Mg & 3) == 0 && (reinterpret_cast<uintptr_t>(out_codes) & 3) == 0;

    // a wavefront's batches of 64 points, dealt so that few points spread over the workgroups
    for (int64_t b0 = ((int64_t)wave * gridDim.x + blockIdx.x) * WAVE; b0 < n; b0 += (int64_t)16 * gridDim.x * WAVE) {
        const int64_t own = b0 + lane, i0 = own < n ? own : n - 1;   // this lane's point: column l32 of block h
        float tval = 0.f;
        uint32_t word = 0;
        // a group's components are requested while the one before is worked on
        float x[G * DS], xn[G * DS];
        auto place = [&](int mg) { return mg + G <= mn ? mg : mn - G; };   // (the last group may reach back)
        auto fetch = [&](int ml) {
            const float *src = E + i0 * D + (int64_t)(m0 + ml) * DS;
            if (m0 + ml >= 0) {                               // (uniform)
#pragma unroll
                for (int t = 0; t + 4 <= G * DS; t += 4) {
                    const float4u w = *reinterpret_cast<const float4u *>(src + t);
                    xn[t] = w.x; xn[t + 1] = w.y; xn[t + 2] = w.z; xn[t + 3] = w.w;
                }
            } else {                                          // fewer than G quantisers
#pragma unroll
                for (int t = 0; t < G * DS; ++t) xn[t] = (m0 + ml) * DS + t >= 0 ? src[t] : 0.f;
            }
        };
        static_assert(G * DS % 4 == 0, "whole loads");
        // codeword and subcentroid of the quantiser before: the constant follows a quantiser behind, where there are registers for it, so that
        // the loads' way is covered (10^6 points with constants, 6 components: 0.497 ms, 0.468 so)
        constexpr bool LAG = DS <= 8;
        float rv[DS], mv[DS];
        auto add_constant = [&]() {
#pragma unroll
            for (int t = 0; t < DS; ++t) tval = fmaf(2.f * mv[t], rv[t], fmaf(rv[t], rv[t], tval));
        };
        fetch(place(0));
        for (int mg = 0; mg < mn; mg += G) {
            const int ml = place(mg);
#pragma unroll
            for (int t = 0; t < G * DS; ++t) x[t] = xn[t];
            if (mg + G < mn) fetch(place(mg + G));
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int m = ml + g;
                if (m < mg || m >= mn) continue;             // (uniform)
                const float *xv = &x[g * DS];
                const float cm = cmax_s[m], scale = scale_s[m];
                const bool copies = __builtin_amdgcn_readfirstlane((int)copies_s[m]) != 0;
                // at the codewords' scale: a component that fp16 does not hold there, 2^16 times the largest of theirs, makes every
                // value no number
                float x2 = 0.f;
                union { halfx8 all[CH]; uint32_t word[4 * CH]; } high, low, B[2];
                union { halfx8 all; uint32_t word[4]; } last[2];
                const halfx2 one = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
                for (int i = 0; i < 4 * CH; ++i) {
                    high.word[i] = low.word[i] = 0;
                    if (2 * i >= DS) continue;
                    const float u = xv[2 * i] * scale, v = xv[2 * i + 1] * scale;
                    x2 = fmaf(v, v, fmaf(u, u, x2));
                    const halfx2 hi = {(_Float16)u, (_Float16)v};
                    high.word[i] = __builtin_bit_cast(uint32_t, hi);
                    float du, dv;                             // u - hi[0], v - hi[1]
                    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(du) : "v"(high.word[i]), "v"(u));
                    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(dv) : "v"(high.word[i]), "v"(v));
                    const halfx2 lo = {(_Float16)du, (_Float16)dv};
                    low.word[i] = __builtin_bit_cast(uint32_t, lo);
                }
                if (R::ROOM) high.word[4 * CH - 1] = __builtin_bit_cast(uint32_t, one);
                auto swap = [](uint32_t a, uint32_t b, uint32_t &lo, uint32_t &hi) {
                    const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
                    lo = s[0];
                    hi = s[1];
                };
#pragma unroll
                for (int i = 0; i < 4 * CH; ++i) swap(high.word[i], low.word[i], B[0].word[i], B[1].word[i]);
                if (!R::ROOM) {   // last product: half 0 high halves against low ones, half 1 the norm
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        swap(high.word[4 * CH - 4 + i], i == 0 ? __builtin_bit_cast(uint32_t, one) : 0u, last[0].word[i], last[1].word[i]);
                }
                // Bound, in units of the products: halves of 22 bits on either side 2^-22 (X + C), what fp16 leaves of their ends
                // 1.5 * 2^-22 (X + C) (C is at least 1/4), the norm 2^-21 C, fp32 accumulation 2^-21 (X + C) on the matrix
                // units and 2^-19 (X + C) of the dot products below, the chain's own roundings 18 * 2^-24 (X + C), the 5 bits an index
                // replaces 2^-18 (X + C), 2 bits in a four: together below 2^-17 (X + C) either way, X = |x|^2, C = the largest
                // |c|^2; a leads b truly if it leads by twice that here
                const float band = 0x1p-16f * (x2 + cm);
                float v1[2] = {-INFINITY, -INFINITY}, v2[2] = {-INFINITY, -INFINITY};
                const gu32x4 *mrow = rows + (size_t)m * CH * 512;
#pragma unroll 1
                for (int tile = 0; tile < 8; ++tile) {
                    floatx16 acc[2];
                    gu32x4 a[CH][2];
#pragma unroll
                    for (int q = 0; q < CH; ++q) {
                        a[q][0] = mrow[(q * 2 + 0) * 256 + tile * 32 + l32];
                        a[q][1] = mrow[(q * 2 + 1) * 256 + tile * 32 + l32];
                    }
                    if (!R::ROOM) {
                        const uint32_t nw = norms[m * 256 + tile * 32 + l32];
                        a[CH - 1][1] = h ? gu32x4{nw, 0u, 0u, 0u} : a[CH - 1][1];
                    }
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
#pragma unroll
                    for (int q = 0; q < CH; ++q)
#pragma unroll
                        for (int p = 0; p < 2; ++p)
#pragma unroll
                            for (int b = 0; b < 2; ++b)
                                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                    __builtin_bit_cast(halfx8, a[q][p]), (!R::ROOM && q == CH - 1 && p == 1) ? last[b].all : B[b].all[q], acc[b], 0, 0, 0);
                    if (copies) {                            // (uniform; far below every value that a codeword can have)
                        const uint32_t out = copy_s[m][tile] >> (4 * h);
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            if (out >> (8 * (v >> 2) + (v & 3)) & 1u) acc[0][v] = acc[1][v] = -0x1p127f;
                    }
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        float s[4];                          // largest of four codewords in a row, its number in the low bits
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float w = larger(larger(larger(acc[b][4 * k], acc[b][4 * k + 1]), acc[b][4 * k + 2]), acc[b][4 * k + 3]);
                            s[k] = __uint_as_float((__float_as_uint(w) & keep) | (uint32_t)(4 * tile + k));
                        }
                        // largest and second largest of them all, two at a time
                        const float t1 = __builtin_amdgcn_fmed3f(v1[b], s[0], s[1]);
                        v1[b] = larger(larger(v1[b], s[0]), s[1]);
                        const float t2 = __builtin_amdgcn_fmed3f(v1[b], s[2], s[3]);
                        v1[b] = larger(larger(v1[b], s[2]), s[3]);
                        v2[b] = larger(larger(v2[b], t1), t2);
                    }
                }
                // the halves of the lanes hold the even and odd groups of four codewords: lane p < 32 takes point p
                // of block 0, lane 32 + p point p of block 1
                uint32_t u1, w1, u2, w2;
                swap(__float_as_uint(v1[0]), __float_as_uint(v1[1]), u1, w1);
                swap(__float_as_uint(v2[0]), __float_as_uint(v2[1]), u2, w2);
                const float a1 = __uint_as_float(u1), b1 = __uint_as_float(w1);
                const bool upper = b1 > a1;
                const float best = upper ? b1 : a1;
                const float next = larger(fminf(a1, b1), larger(__uint_as_float(u2), __uint_as_float(w2)));
                const uint32_t four = (upper ? w1 : u1) & 31u;
                const int j0 = (int)(8u * four + (upper ? 4u : 0u));   // first codeword of the four
                // Which of the four: their values again, by dot products (the lanes start with another one each, or their reads would
                // all go to a quarter of the banks)
                float f[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    f[k] = 0.f;
                    if (!R::ROOM) f[k] = __builtin_amdgcn_fdot2(one, __builtin_bit_cast(halfx2, norms[m * 256 + j0 + ((lane + k) & 3)]), f[k], false);
                }
#pragma unroll
                for (int q = 0; q < CH; ++q) {
                    gu32x4 ch[4], cl[4];                      // (all on their way together)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        ch[k] = mrow[(q * 2 + 0) * 256 + j0 + ((lane + k) & 3)];
                        cl[k] = mrow[(q * 2 + 1) * 256 + j0 + ((lane + k) & 3)];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const halfx2 xh = __builtin_bit_cast(halfx2, high.word[4 * q + i]), xl = __builtin_bit_cast(halfx2, low.word[4 * q + i]);
                        const bool used = q < CH - 1 || 2 * i < R::LAST;   // (behind the components: zeros, or the norm's slots in `high`)
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (used) f[k] = __builtin_amdgcn_fdot2(xh, __builtin_bit_cast(halfx2, (uint32_t)cl[k][i]), f[k], false);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (used) f[k] = __builtin_amdgcn_fdot2(xl, __builtin_bit_cast(halfx2, (uint32_t)ch[k][i]), f[k], false);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (used || (R::ROOM && i == 3)) f[k] = __builtin_amdgcn_fdot2(xh, __builtin_bit_cast(halfx2, (uint32_t)ch[k][i]), f[k], false);
                    }
                    if (q + 1 < CH) __builtin_amdgcn_sched_barrier(0);   // (room for one piece's words)
                }
                if (copies) {
                    const uint32_t out = copy_s[m][four >> 2] >> (j0 & 31);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (out >> ((lane + k) & 3) & 1u) f[k] = -0x1p127f;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = __uint_as_float((__float_as_uint(f[k]) & keep4) | (uint32_t)((lane + k) & 3));
                const float f01 = larger(f[0], f[1]), first = larger(larger(f01, f[2]), f[3]);
                const float second = larger(fminf(f[0], f[1]), __builtin_amdgcn_fmed3f(f01, f[2], f[3]));
                int code = j0 + (int)(__float_as_uint(first) & 3u);
                const bool sure = best - next > band && first - second > band && best < INFINITY && x2 < xmax_s[m];
                uint64_t open = __ballot(!sure && own < n);
                while (open) {
                    const int s = __builtin_ctzll(open);
                    open &= open - 1;
                    float xs[DS];
#pragma unroll
                    for (int t = 0; t < DS; ++t) xs[t] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(xv[t]), s));
                    float bd = INFINITY;
                    uint32_t bj = 0xFFFFFFFFu;
                    float cw[4][DS];                          // (all on their way together)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int t = 0; t < DS; t += 2) {
                            const float2u w = *reinterpret_cast<const float2u *>(codebook + ((int64_t)(m0 + m) * 256 + lane + k * WAVE) * DS + t);
                            cw[k][t] = w.x; cw[k][t + 1] = w.y;
                        }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        float dd = 0.f;
#pragma unroll
                        for (int t = 0; t < DS; ++t) {
                            const float u = xs[t] - cw[k][t];
                            dd = fmaf(u, u, dd);
                        }
                        if (dd < bd) { bd = dd; bj = (uint32_t)(lane + k * WAVE); }
                    }
                    const float least = wave_smallest(bd);
                    bj = wave_extreme<false>(bd == least ? bj : 0xFFFFFFFFu);
                    if (lane == s) code = bj == 0xFFFFFFFFu ? 0 : (int)bj;
                }
                if (words) {                                  // four codes at a time
                    word |= (uint32_t)code << (8 * (m & 3));
                    if ((m & 3) == 3) {
                        if (own < n) *reinterpret_cast<uint32_t *>(out_codes + own * M + m0 + m - 3) = word;
                        word = 0;
                    }
                } else if (own < n) {
                    out_codes[own * M + m0 + m] = (uint8_t)code;
                }
                if (MU) {                                     // (uniform)
                    if (LAG && m > 0) add_constant();
                    const float *cw = codebook + ((int64_t)(m0 + m) * 256 + code) * DS, *mu = MU + i0 * D + (m0 + m) * DS;
#pragma unroll
                    for (int t = 0; t + 2 <= DS; t += 2) {
                        const float2u a = *reinterpret_cast<const float2u *>(cw + t), b = *reinterpret_cast<const float2u *>(mu + t);
                        rv[t] = a.x; rv[t + 1] = a.y;
                        mv[t] = b.x; mv[t + 1] = b.y;
                    }
                    if (!LAG) add_constant();
                }
            }
        }
        if (LAG && MU) add_constant();
        if (own >= n) continue;
        if (out_t) out_t[own] = tval;
        if (const_table) {
            int bj = 0;
            if (sorted && tval == tval) {
                // differences grow to both sides of the value's place: the nearest is one of its two neighbours, and
                // the lowest index among equals lies at or before the left one
                int lo = 0, hi = 256;                          // first entry >= tval
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (tab[mid] < tval) lo = mid + 1;
                    else hi = mid;
                }
                const float dl = lo > 0 ? fabsf(tval - tab[lo - 1]) : INFINITY, dr = lo < 256 ? fabsf(tval - tab[lo]) : INFINITY;
                bj = lo < 256 ? lo : 255;
                if (lo > 0 && dl <= dr) {
                    bj = lo - 1;
                    while (bj > 0 && fabsf(tval - tab[bj - 1]) <= dl) --bj;
                }
                if (!(fminf(dl, dr) < INFINITY)) bj = 0;
            } else {
                float bd = INFINITY;
                for (int j = 0; j < 256; ++j) {
                    const float dd = fabsf(tval - tab[j]);
                    if (dd < bd) { bd = dd; bj = j; }
                }
            }
            out_byte[own] = (uint8_t)bj;
        }
    }
}

// ------------------------------------------------------------------ codeword sums of the training
// Sums of the rows of each codeword in fixed point, so that the order of the additions does not matter: every value
// is taken to a multiple of q = 2^-49 of the largest magnitude of E and added as a 64-bit whole number in LDS.  Values
// of at least 2^-26 of that magnitude are whole multiples; what is left of a smaller one (a few in 10^8 of normally
// distributed values are so small) is added in memory, as a multiple of 2^-31 q.  Values below 2^-57 of the largest
// magnitude may lose 2^-32 q each there, and are counted: where that could reach 2^-53 of a sum, the last place of an
// fp64 sum, a flag is raised and the training is done again with fp64 segment sums (data whose rows lie many
// powers of two apart).
// This takes the place of a sort by code, a segment sum with one workgroup a codeword and five more launches per
// quantiser: 10^6 x 96, 16 quantisers, one round: 1.55 -> 0.12 ms.  Bound by the LDS additions and by reading E.
template <int DS>
struct PqSums {
    static constexpr int MG = DS <= 8 ? 4 : 2;              // quantisers of a workgroup
    static constexpr int lds = MG * 256 * (DS * 8 + 8);
};
inline unsigned pq_sums_grid(int64_t G, int groups) { return (unsigned)((G + N_XCD - 1) / N_XCD * N_XCD * groups); }
constexpr int PQ_SUM_PART = 8192;                           // points between two write-outs: 2^13 * 2^49 stays below 2^63
constexpr int PQ_SUM_MAX_G = 256;
constexpr int PQ_SUM_BLOCK = 1024;                           // two workgroups a compute unit: all the wavefronts it holds (half of them: 152 us, 108 so)

// Slice g's points [g * per, (g + 1) * per) and a group of quantisers a workgroup; the groups of a slice side by side on one XCD, whose L2 then has
// the lines that their parts of a row share.  Grid: pq_sums_grid.  psum [G][M][256][DS] fp64 and pcnt [G][M][256]
// receive its sums and counts (each slice is written by one workgroup, part by part in order); rest [M][256][DS] receives
// the multiples of 2^-31 q, small [M][256] counts the values below their exact range.
template <int DS>
__global__ __launch_bounds__(PQ_SUM_BLOCK) __attribute__((amdgpu_waves_per_eu(8, 8))) void pq_sums_kernel(const float *__restrict__ E, int64_t n, int M,
                                                      const uint8_t *__restrict__ codes, const uint32_t *__restrict__ gmax,
                                                      int G, int64_t per, double *__restrict__ psum, uint32_t *__restrict__ pcnt,
                                                      unsigned long long *__restrict__ rest, unsigned long long *__restrict__ small)
{
    constexpr int MG = PqSums<DS>::MG, W = MG * DS / 2;      // pairs of components a point has in this group
    extern __shared__ __attribute__((aligned(16))) unsigned char pq_lds[];
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(pq_lds);   // [MG][256][DS]
    uint32_t *cnt = reinterpret_cast<uint32_t *>(acc + MG * 256 * DS);           // [MG][256]
    uint32_t *cut = cnt + MG * 256;                                              // [MG][256]
    const int tid = threadIdx.x;
    const int groups = (M + MG - 1) / MG, local = blockIdx.x / N_XCD;
    const int m0 = local % groups * MG, mn = M - m0 < MG ? M - m0 : MG;
    const int64_t D = (int64_t)M * DS, g = (int64_t)(local / groups) * N_XCD + blockIdx.x % N_XCD;
    if (g >= G) return;
    // v + 1.5 * 2^(52 - k) holds round(v * 2^k) in the low bits of its mantissa (|v| 2^k < 2^49): the bit patterns are
    // added, and the pattern of the constant comes off again count times at the end
    const int ex = __builtin_amdgcn_frexp_expf(__uint_as_float(*gmax));
    const double scale = __builtin_amdgcn_ldexp(1.0, 49 - ex), back = __builtin_amdgcn_ldexp(1.0, ex - 49);
    const double magic = 6755399441055744.0;                 // 1.5 * 2^52
    // first magnitude whose last bit is q, or 2^-31 q, or more (as a bit pattern; 1: all of them)
    const uint32_t whole_from = ex - 26 > -126 ? (uint32_t)(ex - 26 + 127) << 23 : 1u;
    const uint32_t rest_from = ex - 57 > -126 ? (uint32_t)(ex - 57 + 127) << 23 : 1u;
    const unsigned long long mbits = __builtin_bit_cast(unsigned long long, magic);
    const int64_t lo = g * per, hi = lo + per < n ? lo + per : n;
    for (int64_t p0 = lo; p0 < hi || p0 == lo; p0 += PQ_SUM_PART) {
        const int64_t pn = hi - p0 < PQ_SUM_PART ? hi - p0 : PQ_SUM_PART;
        for (int i = tid; i < MG * 256 * DS; i += PQ_SUM_BLOCK) acc[i] = 0;
        for (int i = tid; i < 2 * MG * 256; i += PQ_SUM_BLOCK) cnt[i] = 0;
        __syncthreads();
        const int work = (int)pn * W;
#pragma unroll 4
        for (int i = tid; i < work; i += PQ_SUM_BLOCK) {
            const int p = i / W, c = (i - p * W) * 2;        // point of the part, component of the group
            const int m = c / DS, t = c - m * DS;
            if (m < mn) {
                const int64_t row = p0 + p;
                const int code = codes[row * M + m0 + m];
                const float *src = E + row * D + m0 * DS + c;
                const float va = src[0], vb = src[1];
                const double a = fma((double)va, scale, magic), b = fma((double)vb, scale, magic);
                unsigned long long *to = acc + (m * 256 + code) * DS + t;
                atomicAdd(to, __builtin_bit_cast(unsigned long long, a));
                atomicAdd(to + 1, __builtin_bit_cast(unsigned long long, b));
                if (t == 0) atomicAdd(&cnt[m * 256 + code], 1u);
                const uint32_t ua = (__float_as_uint(va) & 0x7FFFFFFFu) - 1u, ub = (__float_as_uint(vb) & 0x7FFFFFFFu) - 1u;
                if (ua < whole_from - 1u || ub < whole_from - 1u) {
                    // (magic - a is a whole number, and what the fma leaves of the value at most 1/2: both exact)
                    unsigned long long *over = rest + (((int64_t)m0 + m) * 256 + code) * DS + t;
                    const double ra = fma((double)va, scale, magic - a) * 0x1p31, rb = fma((double)vb, scale, magic - b) * 0x1p31;
                    if (ua < whole_from - 1u) atomicAdd(over, (unsigned long long)(long long)rint(ra));
                    if (ub < whole_from - 1u) atomicAdd(over + 1, (unsigned long long)(long long)rint(rb));
                    const uint32_t lost = (ua < rest_from - 1u ? 1u : 0u) + (ub < rest_from - 1u ? 1u : 0u);
                    if (lost) atomicAdd(&cut[m * 256 + code], lost);
                }
            }
        }
        __syncthreads();
        double *ps = psum + (g * M + m0) * 256 * DS;
        for (int i = tid; i < mn * 256 * DS; i += PQ_SUM_BLOCK) {
            const unsigned long long whole = acc[i] - mbits * (unsigned long long)cnt[i / DS];
            const double v = (double)(long long)whole * back;
            ps[i] = p0 == lo ? v : ps[i] + v;
        }
        uint32_t *pc = pcnt + (g * M + m0) * 256;
        for (int i = tid; i < mn * 256; i += PQ_SUM_BLOCK) {
            pc[i] = p0 == lo ? cnt[i] : pc[i] + cnt[i];
            if (cut[i]) atomicAdd(&small[m0 * 256 + i], (unsigned long long)cut[i]);
        }
        __syncthreads();
    }
}

// codebook[m][j][t] = sum over the G slices and rest / count, rounded to fp32; a codeword without points keeps its value.
// A workgroup takes 64 components; PARTS threads a component add a part of the slices each, in order (10^6 x 96, 256 slices: four parts 31 us,
// 13 with 16).  rest is left at
// 0 for the next round.  *inexact is set where values that were not added exactly (counted over all rounds) could show.
constexpr int PQ_MEAN_PARTS = 16;

template <int DS>
__global__ __launch_bounds__(64 * PQ_MEAN_PARTS) void pq_means_kernel(const double *__restrict__ psum, const uint32_t *__restrict__ pcnt,
                                                       int M, int G, const uint32_t *__restrict__ gmax,
                                                       unsigned long long *__restrict__ rest, const unsigned long long *__restrict__ small,
                                                       uint32_t *__restrict__ inexact, float *__restrict__ codebook)
{
    __shared__ double part[PQ_MEAN_PARTS][64];
    __shared__ uint32_t part_n[PQ_MEAN_PARTS][64];
    const int c = threadIdx.x & 63, u = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + c, words = (int64_t)M * 256;   // (M * 256 * DS is a multiple of 64)
    const int g0 = (int)((int64_t)G * u / PQ_MEAN_PARTS), g1 = (int)((int64_t)G * (u + 1) / PQ_MEAN_PARTS);
    double s = 0.0;
    uint32_t k = 0;
#pragma unroll 8
    for (int g = g0; g < g1; ++g) {
        s += psum[g * words * DS + i];
        k += pcnt[g * words + i / DS];
    }
    part[u][c] = s;
    part_n[u][c] = k;
    __syncthreads();
    if (u) return;
    for (int v = 1; v < PQ_MEAN_PARTS; ++v) {
        s += part[v][c];
        k += part_n[v][c];
    }
    if (!k) return;
    const int ex = __builtin_amdgcn_frexp_expf(__uint_as_float(*gmax));
    s += (double)(long long)rest[i] * __builtin_amdgcn_ldexp(1.0, ex - 80);
    rest[i] = 0;
    codebook[i] = (float)(s / (double)k);
    if ((double)small[i / DS] * __builtin_amdgcn_ldexp(1.0, ex - 81) > 0x1p-53 * fabs(s)) *inexact = 1u;
}

}  // namespace ivf
