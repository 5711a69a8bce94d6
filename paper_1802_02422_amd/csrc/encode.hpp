// Index-time kernels: subregion assignment (Eq. (3)), displacement (Eq. (4)),
// PQ encoding, the per-point constant of Eq. (6), and the statistics for
// learning alpha (Eqs. (11)-(12)).  One wavefront per point.
#pragma once
#include "coarse.hpp"

namespace ivf {

// LDS per workgroup (one wavefront): x, c and e/mu, each D floats.  With codebook == NULL the
// kernel stops after the displacement (written to out_res, the subcentroid to out_mu).
__global__ __launch_bounds__(64) void encode_kernel(
    const float *__restrict__ X, int64_t n, int D, int M, int L, const int32_t *__restrict__ region,
    const float *__restrict__ C, const int32_t *__restrict__ nbr, const float *__restrict__ alpha,
    const float *__restrict__ cs_dist2, const float *__restrict__ codebook,
    const float *__restrict__ const_table, int32_t *__restrict__ out_sub,
    uint8_t *__restrict__ out_codes, uint8_t *__restrict__ out_byte, float *__restrict__ out_t,
    float *__restrict__ out_res, float *__restrict__ out_mu)
{
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float *xs = sm, *cs = sm + D, *es = sm + 2 * D, *mus = sm + 3 * D;   // D is a multiple of 4: all 16-byte aligned
    const int lane = threadIdx.x;
    const int64_t i = blockIdx.x;
    if (i >= n) return;
    const int64_t r = region[i];
    const float a = alpha[r];
    for (int t = lane; t < D; t += WAVE) {
        xs[t] = X[i * D + t];
        cs[t] = C[r * D + t];
    }
    wave_sync();

    // Eq. (3) through the closed form of the subcentroid distance:
    // ||x - mu_l||^2 = (1-a)||x-c||^2 + a||x-s_l||^2 - a(1-a)||c-s_l||^2
    // Four neighbour rows at a time, 16 lanes per row, a lane taking every 16th group of four
    // components: a load instruction then reads four rows of up to 256 contiguous bytes (with a
    // lane per neighbour it touched 64 different rows, and the kernel was bounded by the number
    // of cache lines its loads addressed).
    const int D4 = D >> 2;
    const int g = lane >> 4, c16 = lane & 15;
    float dxc = 0.f;
    for (int cc = lane; cc < D4; cc += WAVE) {
        const float4 xv = *reinterpret_cast<const float4 *>(xs + 4 * cc);
        const float4 cv = *reinterpret_cast<const float4 *>(cs + 4 * cc);
        const float u0 = xv.x - cv.x, u1 = xv.y - cv.y, u2 = xv.z - cv.z, u3 = xv.w - cv.w;
        dxc = fmaf(u0, u0, dxc);
        dxc = fmaf(u1, u1, dxc);
        dxc = fmaf(u2, u2, dxc);
        dxc = fmaf(u3, u3, dxc);
    }
    dxc = wave_sum(dxc);
    float best = INFINITY;
    int best_l = 0x7fffffff;
    for (int lb = 0; lb < L; lb += WAVE) {            // 64 neighbours at a time: their ids in one load
        const int my_nbr = lb + lane < L ? nbr[r * L + lb + lane] : 0;
        const float my_cs = lb + lane < L ? cs_dist2[r * L + lb + lane] : 0.f;
        const int nl = L - lb < WAVE ? L - lb : WAVE;
        for (int l0 = 0; l0 < nl; l0 += 16) {         // four steps of four rows, their loads issued together
            float4 sv[4][2];
            const float4 *s4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t row = __shfl(my_nbr, (l0 + 4 * u + g) & (WAVE - 1), WAVE);
                s4[u] = reinterpret_cast<const float4 *>(C + row * D);
                const bool live = l0 + 4 * u + g < nl;
                sv[u][0] = live && c16 < D4 ? s4[u][c16] : make_float4(0.f, 0.f, 0.f, 0.f);
                sv[u][1] = live && c16 + 16 < D4 ? s4[u][c16 + 16] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int lw = l0 + 4 * u + g;          // neighbour within this batch of 64
                const bool live = lw < nl;
                const float csl = __shfl(my_cs, lw & (WAVE - 1), WAVE);
                float dxs = 0.f;
                if (live) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (c16 + 16 * h < D4) {
                            const float4 xv = *reinterpret_cast<const float4 *>(xs + 4 * (c16 + 16 * h));
                            const float u0 = xv.x - sv[u][h].x, u1 = xv.y - sv[u][h].y, u2 = xv.z - sv[u][h].z,
                                        u3 = xv.w - sv[u][h].w;
                            dxs = fmaf(u0, u0, dxs);
                            dxs = fmaf(u1, u1, dxs);
                            dxs = fmaf(u2, u2, dxs);
                            dxs = fmaf(u3, u3, dxs);
                        }
                    for (int cc = c16 + 32; cc < D4; cc += 16) {   // D > 128
                        const float4 sw = s4[u][cc];
                        const float4 xv = *reinterpret_cast<const float4 *>(xs + 4 * cc);
                        const float u0 = xv.x - sw.x, u1 = xv.y - sw.y, u2 = xv.z - sw.z, u3 = xv.w - sw.w;
                        dxs = fmaf(u0, u0, dxs);
                        dxs = fmaf(u1, u1, dxs);
                        dxs = fmaf(u2, u2, dxs);
                        dxs = fmaf(u3, u3, dxs);
                    }
                }
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) dxs += __shfl_xor(dxs, o, WAVE);   // over the 16 lanes of the row
                if (live && c16 == 0) {
                    const float sc = fmaf(a, dxs, fmaf(1.f - a, dxc, -a * (1.f - a) * csl));
                    if (sc < best) { best = sc; best_l = lb + lw; }
                }
            }
        }
    }
    wave_argmin(best, best_l);
    if (best_l == 0x7fffffff) best_l = 0;              // (no score is a number)
    if (lane == 0) out_sub[i] = best_l;

    // Eq. (4): displacement from the chosen subcentroid
    const float *s = C + (int64_t)nbr[r * L + best_l] * D;
    for (int t = lane; t < D; t += WAVE) {
        float mu = fmaf(a, s[t] - cs[t], cs[t]);
        mus[t] = mu;
        es[t] = xs[t] - mu;
        if (out_res) out_res[i * D + t] = xs[t] - mu;
        if (out_mu) out_mu[i * D + t] = mu;
    }
    wave_sync();
    if (!codebook) return;   // trained up to alpha only, or the codes are left to pq_encode_kernel

    // PQ: nearest of the 256 codewords per block of D/M dims, lowest index on ties
    const int ds = D / M;
    float tpart = 0.f;   // lane-partial of 2<mu, r> + ||r||^2
    for (int m = 0; m < M; ++m) {
        float bd = INFINITY;
        int bj = 0x7fffffff;
        for (int j = lane; j < 256; j += WAVE) {
            const float *cw = codebook + ((int64_t)m * 256 + j) * ds;
            float dd = 0.f;
            for (int t = 0; t < ds; ++t) {
                float u = es[m * ds + t] - cw[t];
                dd = fmaf(u, u, dd);
            }
            if (dd < bd) { bd = dd; bj = j; }
        }
        wave_argmin(bd, bj);
        if (bj == 0x7fffffff) bj = 0;
        if (lane == 0) out_codes[i * M + m] = (uint8_t)bj;
        const float *cw = codebook + ((int64_t)m * 256 + bj) * ds;
        for (int t = lane; t < ds; t += WAVE) {
            float rv = cw[t];
            tpart = fmaf(2.f * mus[m * ds + t], rv, fmaf(rv, rv, tpart));
        }
    }
    float tval = wave_sum(tpart);
    if (lane == 0 && out_t) out_t[i] = tval;

    if (const_table) {
        float bd = INFINITY;
        int bj = 0x7fffffff;
        for (int j = lane; j < 256; j += WAVE) {
            float dd = fabsf(tval - const_table[j]);
            if (dd < bd) { bd = dd; bj = j; }
        }
        wave_argmin(bd, bj);
        if (lane == 0) out_byte[i] = (uint8_t)bj;
    }
}

// Subregion, displacement and subcentroid (Eqs. (3), (4)) for packed dimensions up to 128 and L <= 64, one wavefront for
// SUB_RUN consecutive points.  Bound by the neighbours' rows: encode_kernel reads L fp32 rows a point.  Here the
// wavefront holds the neighbours' rows as fp16 (pack_hi_rows_kernel) in registers, half the bytes, and keeps them while
// the region stays the same: points in the order of their regions share the read.  Four lanes hold a row, 64 bytes of it
// each load (a row a lane: 64 rows for 16 bytes each, 0.54 against 0.50 ms for 500 000 points on 65 536 regions);
// neighbour 16 p + g is looked after by lane 4 g + p.  The score of Eq. (7) is then known to within
//   err_l = 2 |a| e_l + roundings,  e_l = |dx| |s_l| + (|x| + |dx|) |ds_l| + k |x| |s_l|
// (see the nearest-centroid shortlist), and only neighbours whose lower end does not exceed the smallest upper end, 1.1
// of 64 on unit vectors, are decided by the fp32 differences, with encode_kernel's arithmetic: the same subregion.
// 2 * 10^6 points in region order (two a region), K = 2^20, L = 64, D = 96: 3.8 ms against 7.3, and 5.7 TB/s of the
// 128-byte lines that rows, points and displacements touch.
// perm (may be NULL): the order in which the points are taken.
constexpr int SUB_RUN = 16;

template <int NCH>   // 16-byte chunks of a packed row
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NCH <= 12 ? 4 : 3, NCH <= 12 ? 4 : 3))) void subregion_kernel(
    const float *__restrict__ X, int64_t n, int D, int L, const int32_t *__restrict__ region, const int32_t *__restrict__ perm,
    const float *__restrict__ C, const _Float16 *__restrict__ Ch, const float2 *__restrict__ clen, const uint32_t *__restrict__ cmax,
    const int32_t *__restrict__ nbr, const float *__restrict__ alpha, const float *__restrict__ cs_dist2,
    int32_t *__restrict__ out_sub, float *__restrict__ out_res, float *__restrict__ out_mu)
{
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
    constexpr int Dp = NCH * 8;
    __shared__ __attribute__((aligned(16))) float xs_all[4][Dp];
    __shared__ __attribute__((aligned(16))) _Float16 xh_all[4][Dp];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float *xs = xs_all[wave];
    _Float16 *xh = xh_all[wave];
    const int sh = hi_scale(*cmax);
    const float inv_round = 1.f / (1.f + 0x1p-10f);            // (lengths are rounded up by it)
    const int64_t first = ((int64_t)blockIdx.x * 4 + wave) * SUB_RUN;
    if (first >= n) return;
    const int cnt = n - first < SUB_RUN ? (int)(n - first) : SUB_RUN;
    // lane j: point and region of the run's j-th point, later its subregion.  The points, and the neighbour ids of the next
    // region, are requested a step ahead: what is left to wait for is the rows.
    const int64_t i_of = lane < cnt ? (perm ? (int64_t)perm[first + lane] : first + lane) : 0;
    const int32_t r_of = lane < cnt ? region[i_of] : 0;
    int32_t l_of = 0;
    auto point = [&](int j) { return ((int64_t)__builtin_amdgcn_readlane((int)(i_of >> 32), j) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)i_of, j); };
    constexpr int XP = (Dp + WAVE - 1) / WAVE;
    float xn[XP];
    auto fetch_x = [&](int j) {
        const int64_t i = point(j);
#pragma unroll
        for (int u = 0; u < XP; ++u) xn[u] = lane + u * WAVE < D ? X[i * D + lane + u * WAVE] : 0.f;
    };
    const int part = lane & 3, my_l = 16 * part + (lane >> 2);
    int32_t nbr_n = 0;
    float cs_n = 0.f, a_n = 0.f;
    auto fetch_nbr = [&](int64_t r) {
        nbr_n = my_l < L ? nbr[r * L + my_l] : 0;
        cs_n = my_l < L ? cs_dist2[r * L + my_l] : 0.f;
        a_n = alpha[r];
    };
    fetch_x(0);
    fetch_nbr(__builtin_amdgcn_readlane(r_of, 0));
    int64_t held = -1;                                          // region whose rows the lanes hold
    gu32x4 row[4][NCH / 4];                                      // [t]: of neighbour 16 t + lane / 4, chunks part, part + 4, ..
    float a = 0.f, cs = 0.f, s2 = 0.f, c2 = 0.f;
    float2 sl = make_float2(0.f, 0.f);
    int32_t my_nbr = 0;
    for (int j = 0; j < cnt; ++j) {                             // (uniform)
        const int64_t r = __builtin_amdgcn_readlane(r_of, j);
        if (r != held) {
            held = r;
            a = a_n;
            my_nbr = nbr_n;
            cs = cs_n;
            sl = clen[my_nbr];
            const int of_t[4] = {__builtin_amdgcn_update_dpp(0, my_nbr, 0x00, 0xf, 0xf, false), __builtin_amdgcn_update_dpp(0, my_nbr, 0x55, 0xf, 0xf, false),
                                 __builtin_amdgcn_update_dpp(0, my_nbr, 0xAA, 0xf, 0xf, false), __builtin_amdgcn_update_dpp(0, my_nbr, 0xFF, 0xf, 0xf, false)};   // lane t of the quad
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int k = 0; k < NCH / 4; ++k)
                    row[t][k] = *reinterpret_cast<const gu32x4 *>(Ch + (int64_t)of_t[t] * Dp + 8 * (4 * k + part));
            const float cl = clen[r].x;
            const uint64_t later = __ballot(lane > j && lane < cnt && r_of != (int32_t)r);
            if (later) fetch_nbr(__builtin_amdgcn_readlane(r_of, __builtin_ctzll(later)));
            s2 = sl.x * inv_round * (sl.x * inv_round);
            c2 = cl * cl;
        }
        // the point: fp32 and, in the order of the packed rows, fp16
        float x2 = 0.f, d2 = 0.f;
        wave_sync();
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            const int t = lane + u * WAVE;
            if (t >= Dp) break;
            const float v = xn[u], f = __builtin_amdgcn_ldexpf(v, sh);
            const _Float16 hi = (_Float16)f;
            const float d = f - (float)hi;
            x2 = fmaf(f, f, x2);
            d2 = fmaf(d, d, d2);
            xs[t] = v;
            const int k8 = (t >> 3) & 3;                       // 8 dimensions k8 of 32 lie in chunk 0, 2, 1, 3
            xh[(t & ~31) + 8 * ((k8 & 1) * 2 + (k8 >> 1)) + (t & 7)] = hi;
        }
        if (j + 1 < cnt) fetch_x(j + 1);
        x2 = wave_total(x2);
        d2 = wave_total(d2);
        wave_sync();
        float d4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NCH / 4; ++k) {
            const gu32x4 w = *reinterpret_cast<const gu32x4 *>(&xh[8 * (4 * k + part)]);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    d4[t] = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2, (uint32_t)w[u]), __builtin_bit_cast(halfx2, (uint32_t)row[t][k][u]), d4[t], false);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {                             // over the four lanes of the row
            d4[t] += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(d4[t]), 0xB1, 0xf, 0xf, false));
            d4[t] += __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(d4[t]), 0x4E, 0xf, 0xf, false));
        }
        const float dot = part & 2 ? (part & 1 ? d4[3] : d4[2]) : (part & 1 ? d4[1] : d4[0]);
        // in units of the scaled rows; what all neighbours have in common is left out
        const float2 ql = make_float2(sqrtf(x2) * (1.f + 0x1p-10f), sqrtf(d2) * (1.f + 0x1p-10f));
        const float css = __builtin_amdgcn_ldexpf(cs, 2 * sh);
        const float h = fmaf(a, fmaf(-2.f, dot, s2), -a * (1.f - a) * css);
        // roundings: of the fp32 sum of differences, (D/16 + 12) 2^-24 of at most 2 (x2 + s2), and of the three-term score,
        // 2^-20 of the size of its terms (the scaling factor may be any number: none of them has to be small)
        const float aa = fabsf(a), ac = fabsf(1.f - a);
        const float size = fmaf(aa, x2 + s2, fmaf(ac, x2 + c2, aa * ac * fabsf(css)));
        const float err = fmaf(2.f * aa, shortlist_eps(ql, sl.x, sl.y, Dp), fmaf(aa * (float)(D / 16 + 12) * 0x1p-23f, x2 + s2, 0x1p-20f * size));
        float up = my_l < L ? h + err : INFINITY;
        up = wave_smallest(up);
        uint64_t todo = __ballot(my_l < L && !(h - err > up));
        auto l_at = [](int s) { return 16 * (s & 3) + (s >> 2); };
        int best_l = todo ? l_at(__builtin_ctzll(todo)) : 0;
        if (todo & (todo - 1)) {                               // more than one: the fp32 scores decide
            const int D4 = D >> 2, g = lane >> 4, c16 = lane & 15;
            float dxc = 0.f;
            for (int cc = lane; cc < D4; cc += WAVE) {
                const float4 xv = *reinterpret_cast<const float4 *>(xs + 4 * cc);
                const float4 cv = *reinterpret_cast<const float4 *>(C + r * D + 4 * cc);
                const float u0 = xv.x - cv.x, u1 = xv.y - cv.y, u2 = xv.z - cv.z, u3 = xv.w - cv.w;
                dxc = fmaf(u0, u0, dxc);
                dxc = fmaf(u1, u1, dxc);
                dxc = fmaf(u2, u2, dxc);
                dxc = fmaf(u3, u3, dxc);
            }
            dxc = wave_sum(dxc);
            float best = INFINITY;
            best_l = 0x7fffffff;
            while (todo) {                                      // four at a time, 16 lanes each
                int from = -1;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (todo) {
                        if (g == u) from = __builtin_ctzll(todo);
                        todo &= todo - 1;
                    }
                const int l = from < 0 ? -1 : l_at(from);
                const int64_t srow = __shfl(my_nbr, from < 0 ? 0 : from, WAVE);
                const float csl = __shfl(cs, from < 0 ? 0 : from, WAVE);
                float dxs = 0.f;
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
                    if (l >= 0 && c16 + 16 * hh < D4) {
                        const float4 sv = *reinterpret_cast<const float4 *>(C + srow * D + 4 * (c16 + 16 * hh));
                        const float4 xv = *reinterpret_cast<const float4 *>(xs + 4 * (c16 + 16 * hh));
                        const float u0 = xv.x - sv.x, u1 = xv.y - sv.y, u2 = xv.z - sv.z, u3 = xv.w - sv.w;
                        dxs = fmaf(u0, u0, dxs);
                        dxs = fmaf(u1, u1, dxs);
                        dxs = fmaf(u2, u2, dxs);
                        dxs = fmaf(u3, u3, dxs);
                    }
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) dxs += __shfl_xor(dxs, o, WAVE);
                if (l >= 0 && c16 == 0) {
                    const float sc = fmaf(a, dxs, fmaf(1.f - a, dxc, -a * (1.f - a) * csl));
                    if (sc < best || (sc == best && l < best_l)) { best = sc; best_l = l; }
                }
            }
            wave_argmin(best, best_l);
            if (best_l == 0x7fffffff) best_l = 0;               // (no score is a number)
        }
        if (lane == j) {
            out_sub[i_of] = best_l;
            l_of = best_l;
        }
    }
    // displacements: independent of each other, so that several points' rows are on their way together
#pragma unroll 4
    for (int j = 0; j < cnt; ++j) {
        const int64_t i = point(j), r = __builtin_amdgcn_readlane(r_of, j);
        const float aj = alpha[r];
        const float *s = C + (int64_t)nbr[r * L + __builtin_amdgcn_readlane(l_of, j)] * D, *c = C + r * D;
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            const int t = lane + u * WAVE;
            if (t < D) {
                const float x = X[i * D + t], mu = fmaf(aj, s[t] - c[t], c[t]);
                if (out_res) out_res[i * D + t] = x - mu;
                if (out_mu) out_mu[i * D + t] = mu;
            }
        }
    }
}

}  // namespace ivf
