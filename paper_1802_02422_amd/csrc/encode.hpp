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

// The centroid table in 8 bits for subregion_kernel: row c is s - centre ~ step * q, q in -127 .. 127, step the 127th part of its largest
// component, with its step, |s|^2, |ds| and 2 <step q, ds> (ds: what the rounding left out) behind the components where a row of 128
// bytes has room for them, so that one line holds it all, and in an array of their own where 128 components fill it.  A row that is not
// finite: zeros with infinite lengths.
template <int DP>   // packed dimension
struct ByteRow {
    static constexpr bool INSIDE = DP < 128;
    static constexpr int BYTES = DP == 32 ? 64 : 128, TAIL_STRIDE = INSIDE ? BYTES : 16;
    static constexpr int CHUNKS = BYTES / 64;                // 16-byte pieces of a row that a lane of four holds
};
inline size_t byte_row_bytes(int Dp) { return Dp == 32 ? 64 : Dp == 128 ? 144 : 128; }   // of a row and what belongs to it

// The rows are taken as differences to a point near the middle of the table, like the points later: distances between them are the same, and
// an offset that all have in common does not cost the 8 bits anything.  It is the mean of up to 16 rows (any point is right), which every
// workgroup forms for itself, from the same numbers in the same order; the first writes it to `centre` (0 behind D).
constexpr int CENTRE_ROWS = 16;
constexpr int64_t BYTE_ROWS_GRID = 2048;

template <int DP>
__global__ __launch_bounds__(256) void pack_byte_rows_kernel(const float *__restrict__ X, int64_t n, int D, float *__restrict__ centre,
                                                             uint8_t *__restrict__ rows, uint8_t *__restrict__ tails)
{
    typedef ByteRow<DP> R;
    constexpr int PER = R::BYTES / 16, LIVE = DP / 16;        // 16 bytes a lane
    __shared__ __attribute__((aligned(16))) float mid[2][128];
    {
        const int c = threadIdx.x & 127, g = threadIdx.x >> 7, many = n < CENTRE_ROWS ? (int)n : CENTRE_ROWS;
        const int64_t stride = n / many;
        float w[CENTRE_ROWS / 2], s = 0.f;
#pragma unroll
        for (int u = 0; u < CENTRE_ROWS / 2; ++u)             // (every thread loads: all are on their way together)
            w[u] = X[(int64_t)(2 * u + g < many ? 2 * u + g : 0) * stride * D + (c < D ? c : 0)];
#pragma unroll
        for (int u = 0; u < CENTRE_ROWS / 2; ++u) {
            const float t = c < D && 2 * u + g < many ? w[u] * (1.f / CENTRE_ROWS) : 0.f;
            s += fabsf(t) < INFINITY ? t : 0.f;
        }
        mid[g][c] = s;
        __syncthreads();
        s = (mid[0][c] + mid[1][c]) * ((float)CENTRE_ROWS / (float)many);
        s = fabsf(s) < INFINITY ? s : 0.f;
        __syncthreads();
        if (g == 0) {
            mid[0][c] = s;
            if (blockIdx.x == 0) centre[c] = s;
        }
        __syncthreads();
    }
    const int lane = threadIdx.x % PER;
    for (int64_t row0 = (int64_t)blockIdx.x * (256 / PER); row0 < n; row0 += (int64_t)gridDim.x * (256 / PER)) {   // (uniform)
        const int64_t row = row0 + threadIdx.x / PER;
        float v[16], big = 0.f, s2 = 0.f, d2 = 0.f, qd = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < n && lane < LIVE && 16 * lane + 4 * u < D) w = *reinterpret_cast<const float4 *>(X + row * D + 16 * lane + 4 * u);   // (D is a multiple of 4)
            const float4 m = lane < LIVE ? *reinterpret_cast<const float4 *>(&mid[0][16 * lane + 4 * u]) : make_float4(0.f, 0.f, 0.f, 0.f);   // (0 behind D)
            v[4 * u] = w.x - m.x; v[4 * u + 1] = w.y - m.y; v[4 * u + 2] = w.z - m.z; v[4 * u + 3] = w.w - m.w;
            if (row >= n) v[4 * u] = v[4 * u + 1] = v[4 * u + 2] = v[4 * u + 3] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            big = fmaxf(big, fabsf(v[i]));
            s2 = fmaf(v[i], v[i], s2);
        }
#pragma unroll
        for (int o = PER / 2; o > 0; o >>= 1) {
            big = fmaxf(big, __shfl_xor(big, o, WAVE));
            s2 += __shfl_xor(s2, o, WAVE);
        }
        const bool finite = s2 < INFINITY;
        const float step = big * (1.f / 127.f), per = big > 0x1p-100f && finite ? 127.f / big : 0.f;
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float q = fminf(fmaxf(rintf((finite ? v[i] : 0.f) * per), -127.f), 127.f), d = fmaf(-q, step, v[i]);
            d2 = fmaf(d, d, d2);
            qd = fmaf(q * step, d, qd);
            w[i >> 2] |= ((uint32_t)(int)q & 255u) << (8 * (i & 3));
        }
#pragma unroll
        for (int o = PER / 2; o > 0; o >>= 1) {
            d2 += __shfl_xor(d2, o, WAVE);
            qd += __shfl_xor(qd, o, WAVE);
        }
        if (row >= n) continue;
        if (lane < LIVE) *reinterpret_cast<uint4 *>(rows + row * R::BYTES + 16 * lane) = make_uint4(w[0], w[1], w[2], w[3]);
        if (lane == 0)
            *reinterpret_cast<float4 *>(tails + row * R::TAIL_STRIDE) =
                finite ? make_float4(step, s2, sqrtf(d2) * (1.f + 0x1p-10f), 2.f * qd) : make_float4(0.f, INFINITY, INFINITY, INFINITY);
    }
}

// Subregion, displacement and subcentroid (Eqs. (3), (4)) for packed dimensions up to 128 and L <= 64, one wavefront for
// SUB_RUN consecutive points.  Bound by the neighbours' rows: encode_kernel reads L fp32 rows a point.  Here the
// wavefront holds the neighbours' rows in 8 bits (pack_byte_rows_kernel) in registers, a 128-byte line each, and keeps them while
// the region stays the same: points in the order of their regions share the read.  Four lanes hold a row, 64 bytes of it
// each load (a row a lane: 64 rows for 16 bytes each, 0.54 against 0.50 ms for 500 000 points on 65 536 regions);
// neighbour 16 p + g is looked after by lane 4 g + p.  The point is taken in 15 bits, as two 8-bit halves, so that products are whole numbers
// (v_dot4).  With what all neighbours of a region share left out, the score of Eq. (7) is then known to within 2 |a| e_l and the
// roundings of sums, |x - s_l|^2 being |s_l|^2 - 2 <x, q_l> with
//   e_l = |dx| |x - q_l| + |x| |ds_l| + k |x| |s_l|,   or |s_l|^2 - 2 <q_l, ds_l> - 2 <x, q_l> with   e_l = (|dx| + |ds_l|) |x - q_l| + k |x| |s_l|
// (q_l: the row as packed), whichever is smaller: the second where a point is nearer to its neighbours than to the table's middle, as in tables of
// several groups far apart.  (500 000 points, 65 536 regions in 16 groups of width 1 with means of length 2, 4, 8, 16, us a call: 781, 913, 1452, 2123,
// with the first alone 872, 1840, 2123, 2130, with fp16 rows 911, 982, 1199, 2704; of one group 755 either way.)
// Only neighbours whose lower end does not exceed the smallest upper end are decided by the
// fp32 differences, with encode_kernel's arithmetic: the same subregion.  A third of the points of unit vectors have several such; they
// are put by and decided when the wavefront has been through its points, eight neighbours on their way at a time whatever point
// they belong to (decided where they come up, with the loads and sums of one point behind those of another: 0.56 ms for
// 500 000 points on 65 536 regions, 0.50 so, 0.445 with five wavefronts a SIMD).
// With vectors that share an offset of 1 (10) in every component such a call takes 0.73 (0.73) ms, without the centre 0.96 (2.16), with fp16
// rows 1.46 (3.0); encode_kernel 1.63 whatever the vectors.
// 2 * 10^6 points in region order (two a region), K = 2^20, L = 64, D = 96: 2.27 ms; with fp16 rows, two lines each, whose bound leaves
// 1.1 of 64, 3.8; encode_kernel 7.3.
// perm (may be NULL): the order in which the points are taken.
constexpr int SUB_RUN = 16;

template <int DP>   // packed dimension
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 5))) void subregion_kernel(
    const float *__restrict__ X, int64_t n, int D, int L, const int32_t *__restrict__ region, const int32_t *__restrict__ perm,
    const float *__restrict__ C, const float *__restrict__ centre, const uint8_t *__restrict__ rows, const uint8_t *__restrict__ tails,
    const int32_t *__restrict__ nbr, const float *__restrict__ alpha, const float *__restrict__ cs_dist2,
    int32_t *__restrict__ out_sub, float *__restrict__ out_res, float *__restrict__ out_mu)
{
    typedef ByteRow<DP> R;
    constexpr int CH = R::CHUNKS;
    __shared__ float mid_all[4][(DP + WAVE - 1) / WAVE * WAVE];   // the centre, 0 behind D
    __shared__ __attribute__((aligned(16))) int8_t xh_all[4][2][R::BYTES];   // high and low halves; zeros behind the components
    __shared__ uint16_t pairs_all[4][SUB_RUN * WAVE];
    __shared__ unsigned long long best_all[4][SUB_RUN];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int8_t *xh = xh_all[wave][0], *xl = xh_all[wave][1];
    uint16_t *pairs = pairs_all[wave];
    unsigned long long *best = best_all[wave];
    const int64_t first = ((int64_t)blockIdx.x * 4 + wave) * SUB_RUN;
    if (first >= n) return;
    for (int t = lane; t < 2 * R::BYTES / 4; t += WAVE) reinterpret_cast<uint32_t *>(xh)[t] = 0;
    float *mid = mid_all[wave];
    for (int t = lane; t < (DP + WAVE - 1) / WAVE * WAVE; t += WAVE) mid[t] = centre[t];
    const int cnt = n - first < SUB_RUN ? (int)(n - first) : SUB_RUN;
    // lane j: point and region of the run's j-th point, later its subregion.  The points, and the neighbour ids of the next
    // region, are requested a step ahead: what is left to wait for is the rows.
    const int64_t i_of = lane < cnt ? (perm ? (int64_t)perm[first + lane] : first + lane) : 0;
    const int32_t r_of = lane < cnt ? region[i_of] : 0;
    int32_t l_of = 0;
    unsigned long long best_of = 0;                             // ~0: undecided
    int n_pairs = 0;                                            // (uniform) point << 6 | neighbour in `pairs`
    auto point = [&](int j) { return ((int64_t)__builtin_amdgcn_readlane((int)(i_of >> 32), j) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)i_of, j); };
    constexpr int XP = (DP + WAVE - 1) / WAVE;
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
    auto tail = [&](int64_t r) { return *reinterpret_cast<const float4 *>(tails + r * R::TAIL_STRIDE); };
    fetch_x(0);
    fetch_nbr(__builtin_amdgcn_readlane(r_of, 0));
    int64_t held = -1;                                          // region whose rows the lanes hold
    gu32x4 row[4][CH];                                           // [t]: of neighbour 16 t + lane / 4, chunks part, part + 4, ..
    float a = 0.f, cs = 0.f, c2 = 0.f;
    float4 sl = make_float4(0.f, 0.f, 0.f, 0.f);                 // step, |s|^2, |ds|, 2 <q, ds>
    int32_t my_nbr = 0;
    for (int j = 0; j < cnt; ++j) {                             // (uniform)
        const int64_t r = __builtin_amdgcn_readlane(r_of, j);
        if (r != held) {
            held = r;
            a = a_n;
            my_nbr = nbr_n;
            cs = cs_n;
            const int of_t[4] = {__builtin_amdgcn_update_dpp(0, my_nbr, 0x00, 0xf, 0xf, false), __builtin_amdgcn_update_dpp(0, my_nbr, 0x55, 0xf, 0xf, false),
                                 __builtin_amdgcn_update_dpp(0, my_nbr, 0xAA, 0xf, 0xf, false), __builtin_amdgcn_update_dpp(0, my_nbr, 0xFF, 0xf, 0xf, false)};   // lane t of the quad
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int k = 0; k < CH; ++k)
                    row[t][k] = *reinterpret_cast<const gu32x4 *>(rows + (int64_t)of_t[t] * R::BYTES + 16 * (4 * k + part));
            sl = tail(my_nbr);
            c2 = tail(r).y;
            const uint64_t later = __ballot(lane > j && lane < cnt && r_of != (int32_t)r);
            if (later) fetch_nbr(__builtin_amdgcn_readlane(r_of, __builtin_ctzll(later)));
        }
        // the point as two bytes a component.  (What the subtraction of the centre rounds, 2^-24 of the difference, is a part of the bound's last
        // term: the products are exact.)
        float x2 = 0.f, d2 = 0.f, big = 0.f, xc[XP];
        wave_sync();
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            xc[u] = xn[u] - mid[lane + u * WAVE];
            big = fmaxf(big, fabsf(xc[u]));
        }
        big = __uint_as_float(wave_extreme<true>(__float_as_uint(big)));   // (not negative: the bits order like it)
        const float step = big * (1.f / 16256.f), per = big > 0x1p-100f && big < INFINITY ? 16256.f / big : 0.f;
        wave_sync();
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            const int t = lane + u * WAVE;
            const float v = xc[u], q = fminf(fmaxf(rintf(v * per), -16256.f), 16256.f), d = fmaf(-q, step, v);
            x2 = fmaf(v, v, x2);
            d2 = fmaf(d, d, d2);
            if (t < DP) {
                const int w = (int)q, hi = (w + 64) >> 7;
                xh[t] = (int8_t)hi;
                xl[t] = (int8_t)(w - 128 * hi);
            }
        }
        if (j + 1 < cnt) fetch_x(j + 1);
        x2 = wave_total(x2);
        d2 = wave_total(d2);
        wave_sync();
        int ih[4] = {0, 0, 0, 0}, il[4] = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const gu32x4 wh = *reinterpret_cast<const gu32x4 *>(&xh[16 * (4 * k + part)]), wl = *reinterpret_cast<const gu32x4 *>(&xl[16 * (4 * k + part)]);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    ih[t] = __builtin_amdgcn_sdot4((int)wh[u], (int)row[t][k][u], ih[t], false);
                    il[t] = __builtin_amdgcn_sdot4((int)wl[u], (int)row[t][k][u], il[t], false);
                }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {                             // over the four lanes of the row (below 2^28)
            ih[t] = 128 * ih[t] + il[t];
            ih[t] += __builtin_amdgcn_update_dpp(0, ih[t], 0xB1, 0xf, 0xf, false);
            ih[t] += __builtin_amdgcn_update_dpp(0, ih[t], 0x4E, 0xf, 0xf, false);
        }
        const float dot = (float)(part & 2 ? (part & 1 ? ih[3] : ih[2]) : (part & 1 ? ih[1] : ih[0])) * (step * sl.x);
        // what all neighbours have in common is left out
        // (the instruction alone: what it may be off, and for what is subnormal, is made room for)
        const float2 ql = make_float2(__builtin_amdgcn_sqrtf(x2 + 0x1p-100f) * (1.f + 0x1p-10f), __builtin_amdgcn_sqrtf(d2 + 0x1p-100f) * (1.f + 0x1p-10f));
        const float s2 = sl.y, both = x2 + s2, len = __builtin_amdgcn_sqrtf(s2) * (1.f + 0x1p-10f);
        // |x - q| or more, and which of the two forms has less left out
        const float far2 = fmaf(-2.f, dot, both - sl.w) + fmaf(2.f * ql.y, len + sl.z, fmaf(0x1p-18f, both, 0x1p-120f));
        const float far = __builtin_amdgcn_sqrtf(fmaxf(far2, 0.f)) * (1.f + 0x1p-10f);
        const bool near = far < ql.x;
        const float h = fmaf(a, fmaf(-2.f, dot, near ? s2 - sl.w : s2), -a * (1.f - a) * cs);
        const float e = fmaf(ql.y, far, fmaf(near ? far : ql.x, sl.z, (float)(DP + 32) * 0x1p-24f * ql.x * len));
        // roundings: of the fp32 sum of differences, (D/16 + 12) 2^-24 of at most 2 (x2 + s2), and of the three-term score,
        // 2^-20 of the size of its terms (the scaling factor may be any number: none of them has to be small)
        const float aa = fabsf(a), ac = fabsf(1.f - a);
        // (and 2^-120 for values whose squares leave the range of fp32)
        const float size = fmaf(aa, both, fmaf(ac, x2 + c2, aa * ac * fabsf(cs)));
        const float err = fmaf(2.f * aa, e, fmaf(aa * (float)(D / 16 + 12) * 0x1p-23f, both, fmaf(0x1p-20f, size, 0x1p-120f)));
        float up = my_l < L ? h + err : INFINITY;
        up = wave_smallest(up);
        uint64_t todo = __ballot(my_l < L && !(h - err > up));
        auto l_at = [](int s) { return 16 * (s & 3) + (s >> 2); };
        int best_l = todo ? l_at(__builtin_ctzll(todo)) : 0;
        if (todo & (todo - 1)) {                               // more than one: the fp32 scores decide, below
            if (todo >> lane & 1u) pairs[n_pairs + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(todo >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)todo, 0u))] = (uint16_t)(j << 6 | my_l);
            n_pairs += __popcll(todo);
            if (lane == j) best_of = ~0ull;
        } else if (lane == j) {
            l_of = best_l;
        }
    }
    // The fp32 scores of what is left, whatever point it belongs to: 16 lanes a neighbour, eight of them on their way at a time
    if (n_pairs) {                                              // (uniform)
        if (lane < SUB_RUN) best[lane] = best_of;
        wave_sync();
        const int D4 = D >> 2, g = lane >> 4, c16 = lane & 15;
        for (int p0 = 0; p0 < n_pairs; p0 += 8) {
            int who[2];
            float4 sv[2][2], cv[2][2], xv[2][2];
            float csl[2], aj[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int p = p0 + 4 * u + g;
                who[u] = pairs[p < n_pairs ? p : p0];
                const int j = who[u] >> 6, l = who[u] & 63;
                const int64_t r = __shfl(r_of, j, WAVE), i = (int64_t)((uint64_t)(uint32_t)__shfl((int)(i_of >> 32), j, WAVE) << 32 | (uint32_t)__shfl((int)i_of, j, WAVE));
                const int64_t sr = nbr[r * L + l];
                csl[u] = cs_dist2[r * L + l];
                aj[u] = alpha[r];
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int c4 = 4 * (c16 + 16 * hh < D4 ? c16 + 16 * hh : 0);
                    xv[u][hh] = *reinterpret_cast<const float4 *>(X + i * D + c4);
                    cv[u][hh] = *reinterpret_cast<const float4 *>(C + r * D + c4);
                    sv[u][hh] = *reinterpret_cast<const float4 *>(C + sr * D + c4);
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // encode_kernel's sums: a lane of four components each against the region's centroid, in pairs of lanes 16 apart first; against the
                // neighbour a lane goes on with the components 64 behind
                float dxc = 0.f, dxs = 0.f;
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const float4 x = xv[u][hh], c = cv[u][hh], s = sv[u][hh];
                    const bool live = c16 + 16 * hh < D4;
                    const float c0 = x.x - c.x, c1 = x.y - c.y, c2 = x.z - c.z, c3 = x.w - c.w;
                    const float part_c = fmaf(c3, c3, fmaf(c2, c2, fmaf(c1, c1, c0 * c0)));
                    dxc += live ? part_c : 0.f;
                    const float s0 = x.x - s.x, s1 = x.y - s.y, s2 = x.z - s.z, s3 = x.w - s.w;
                    const float next = fmaf(s3, s3, fmaf(s2, s2, fmaf(s1, s1, fmaf(s0, s0, dxs))));
                    dxs = live ? next : dxs;
                }
                dxc = sum_of_16(dxc);
                dxs = sum_of_16(dxs);
                const float sc = fmaf(aj[u], dxs, fmaf(1.f - aj[u], dxc, -aj[u] * (1.f - aj[u]) * csl[u])) + 0.f;   // (-0 is 0)
                if (c16 == 0 && p0 + 4 * u + g < n_pairs && sc < INFINITY)
                    atomicMin(&best[who[u] >> 6], (unsigned long long)float_key(sc) << 32 | (uint32_t)(who[u] & 63));
            }
        }
        wave_sync();
        if (lane < SUB_RUN && best_of == ~0ull) l_of = best[lane] == ~0ull ? 0 : (int32_t)(uint32_t)best[lane];   // (no score is a number: 0)
    }
    if (lane < cnt) out_sub[i_of] = l_of;
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
