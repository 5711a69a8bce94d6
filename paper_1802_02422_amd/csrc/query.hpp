// Stages 2-4 of the query path: subcentroid scoring by the closed form of
// Eq. (7), pruning to the S closest subregions, and the per-query table of
// -2<q_m, r^m_j> of Eq. (6).
#pragma once
#include "select.hpp"

namespace ivf {

constexpr int SCORE_BINS = 1024;
template <int BLOCK, int STREAM> constexpr int score_bins() { return STREAM < 0 ? 4 * BLOCK : SCORE_BINS; }

// One kept subregion of one query, as the scan consumes it.
struct SubDesc {
    uint32_t blk;    // start of the subregion's record block, in BLK_ALIGN-byte units
    uint32_t pos0;   // grouped position of its first point (indexes ids[])
    uint32_t len;    // number of points
    float base;      // distance from the query to the subcentroid
};

// T[q][m][j] = -2 <q_m, r^m_j> (Eq. (6)) for nl <= LUT_Q queries in a row by one workgroup of BLOCK threads: the queries in LDS
// (qs, [D][LUT_Q] floats; [D] for one), every thread one (sub-quantiser, codeword) pair at a time, each entry one chain of fused
// multiply-adds over the block's dimensions.  Bound by the reads of the codewords, so that where there are queries enough a
// workgroup takes LUT_Q of them.
constexpr int LUT_Q = 8;

template <int BLOCK>
__device__ __forceinline__ void lut_body(const float *__restrict__ Q, int nl, int D, int M, const float *__restrict__ codebook,
                                         float *__restrict__ T, float *qs)
{
    const int ds = D / M;
    if (nl == 1) {
        for (int i = threadIdx.x; i < D; i += BLOCK) qs[i] = Q[i];
        __syncthreads();
        for (int e = threadIdx.x; e < M * 256; e += BLOCK) {
            const float *cw = codebook + (int64_t)e * ds, *qm = qs + (e >> 8) * ds;
            float s = 0.f;
            for (int i = 0; i < ds; ++i) s = fmaf(qm[i], cw[i], s);
            T[e] = -2.f * s;
        }
        return;
    }
    for (int i = threadIdx.x; i < nl * D; i += BLOCK) qs[(i % D) * LUT_Q + i / D] = Q[i];
    __syncthreads();
    for (int e = threadIdx.x; e < M * 256; e += BLOCK) {
        const float *cw = codebook + (int64_t)e * ds, *qm = qs + (e >> 8) * ds * LUT_Q;
        float s[LUT_Q];
#pragma unroll
        for (int j = 0; j < LUT_Q; ++j) s[j] = 0.f;
        for (int i = 0; i < ds; ++i) {
            const float c = cw[i];
#pragma unroll
            for (int j = 0; j < LUT_Q; j += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(&qm[i * LUT_Q + j]);   // (past nl: whatever is there, not stored)
                s[j] = fmaf(v.x, c, s[j]);
                s[j + 1] = fmaf(v.y, c, s[j + 1]);
                s[j + 2] = fmaf(v.z, c, s[j + 2]);
                s[j + 3] = fmaf(v.w, c, s[j + 3]);
            }
        }
#pragma unroll
        for (int j = 0; j < LUT_Q; ++j)
            if (j < nl) T[(int64_t)j * M * 256 + e] = -2.f * s[j];
    }
}

// Queries of a table workgroup: LUT_Q where that leaves a workgroup for every compute unit and their rows fit the launch's LDS.
inline int lut_queries(int64_t n, int D, size_t lds) { return n >= 256 * LUT_Q && (size_t)LUT_Q * D * sizeof(float) <= lds ? LUT_Q : 1; }
inline unsigned lut_grid(int64_t n, int per) { return (unsigned)(n + (n + per - 1) / per); }   // scoring workgroups, then table ones

// Stages 2 and 3 fused, one workgroup per query.
// Stage 2 (Eq. (7)): score[p][l] = (1-a) D[q][r] + a D[q][nbr[r][l]] + cst[r][l], r = probe_id[q][p],
// cst[r][l] = -a(1-a)||c_r - s_l||^2 tabulated at load time.  The neighbour distances are gathered from
// the stage-1 distance tile, not recomputed; every thread has PL/BLOCK independent gathers in flight.
// The scores formed here never leave the chip: they are kept in LDS as order-preserving keys.
// Stage 3: keep the S smallest of the P*L scores by (score, r*L + l).  probe_id is ascending in r, so
// position order in the score row is subregion-id order and the descriptors come out sorted by address.
// The selection leaves the kept score indices, in order, in LDS (over the keys, which every thread
// holds in registers by then) and their scores in the descriptors; the rest of a descriptor is
// then filled position by position, consecutive lanes writing consecutive descriptors, with the
// reads of the subregion table of four positions in flight per thread (filled item by item as
// they were selected, every read of that table was waited for before the next was issued).
// Dynamic LDS: P*L keys + P probe ids + P probe distances + P alphas.  P*L <= 4 * MAXV * BLOCK.
// Stage 4 rides along: behind the nq workgroups there is one for every lut_per queries' lookup
// tables (lut_body, from Qt = the queries, rotated if the index has a rotation) while the first nq
// gather and select; the two halves share nothing, and the table work hides under the gathers.
// Dynamic LDS must also hold D floats.
// STREAM > 0: the query's whole row of the tile is read, STREAM distances at a time, into LDS (over the place of the keys,
// which come after it), and the neighbours' distances are picked there: a gather costs a 128-byte line of the row for
// each 4 bytes, so that with 16 P L >= K the row is the smaller number of bytes, and whole lines in order (where that
// pays: score_mode).  Dynamic LDS:
// max(P*L, STREAM + 4) + 3 P words.
// STREAM < 0: the keys of the scores are given (pair_distance_kernel), ldt = P*L of them a query in the place of Dt, and go to
// registers; dynamic LDS: 2 S + 3 P words.
// (the body of a scoring workgroup, for query q of the batch: also the second half of select_score_prune_kernel)
template <int BLOCK, int MAXV, int STREAM = 0>
__device__ __forceinline__ void score_prune_body(
    const float *__restrict__ Dt, int64_t ldt, int64_t K, const int32_t *__restrict__ probe_id,
    const float *__restrict__ probe_d, int P, int L, const int32_t *__restrict__ nbr,
    const float *__restrict__ cst, const float *__restrict__ alpha, int S,
    const uint4 *__restrict__ sub_info,
    SubDesc *__restrict__ desc, int64_t *__restrict__ kept_sub, int64_t *__restrict__ n_scanned,
    int64_t q, uint32_t *dyn, SelectRegs<score_bins<BLOCK, STREAM>()> &sh)
{
    __shared__ unsigned long long codes_total;
    const int PL = P * L;
    uint32_t *keys = dyn;
    const int front = STREAM < 0 ? 2 * S : STREAM > 0 && PL < STREAM + 4 ? STREAM + 4 : PL;
    int32_t *pid = reinterpret_cast<int32_t *>(dyn + front);
    float *pd = reinterpret_cast<float *>(dyn + front + P);
    float *pa = reinterpret_cast<float *>(dyn + front + 2 * P);
    const float *row = Dt + q * ldt;
    uint32_t kv[4 * MAXV], pivot, need;
    const int ipt = run_length<BLOCK>(PL);
    auto same = [](uint32_t w) { return w; };
    const int32_t first = probe_id[q * P + ((int)threadIdx.x < P ? (int)threadIdx.x : P - 1)];
    if constexpr (STREAM < 0) {                           // (the keys requested with the probes: 10 000 queries of 16 384 547 -> 513 us)
        if ((PL & 3) == 0) load_run<BLOCK>(reinterpret_cast<const uint32_t *>(row), PL, kv, same);
        else load_run<BLOCK, false>(reinterpret_cast<const uint32_t *>(row), PL, kv, same);
    }
    for (int p = threadIdx.x; p < P; p += BLOCK) {
        const int32_t r = p < BLOCK ? first : probe_id[q * P + p];
        pid[p] = r;
        if constexpr (STREAM >= 0) {
            pd[p] = probe_d[q * P + p];
            pa[p] = alpha[r];
        }
    }
    if (threadIdx.x == 0) codes_total = 0;
    __syncthreads();
    if constexpr (STREAM > 0) {
        constexpr int U = 4 * MAXV;                      // items of a thread: threadIdx.x + u * BLOCK
        uint32_t word[U];                                 // neighbour id, then the distance (found: bit u)
        uint32_t found = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * BLOCK;
            word[u] = 0xFFFFFFFFu;
            if (i < PL) {
                const int p = i / L;
                word[u] = (uint32_t)nbr[(int64_t)pid[p] * L + (i - p * L)];
            }
        }
        float *part = reinterpret_cast<float *>(keys);
        const int skew = (int)((reinterpret_cast<uintptr_t>(row) >> 2) & 3);
        for (int64_t c0 = 0; c0 < K; c0 += STREAM) {
            const int n = K - c0 < STREAM ? (int)(K - c0) : STREAM;
            if (c0) __syncthreads();                      // the previous part has been picked from
            // 16-byte loads from the boundary at or before the part, `skew` floats of the row before (or of the part before)
            // with it; what is left at the end one by one
            const int whole = (n + skew) / 4;
            const float4 *src = reinterpret_cast<const float4 *>(row + c0 - skew);
            // (a register array that has all loads on their way before the first store took 0.45 ms more)
#pragma unroll
            for (int v = 0; v <= STREAM / 4 / BLOCK; ++v)
                if ((int)threadIdx.x + v * BLOCK < whole) reinterpret_cast<float4 *>(part)[threadIdx.x + v * BLOCK] = src[threadIdx.x + v * BLOCK];
            if ((int)threadIdx.x < n + skew - 4 * whole) part[4 * whole + threadIdx.x] = row[c0 - skew + 4 * whole + threadIdx.x];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t at = word[u] - (uint32_t)c0;
                if (!(found >> u & 1u) && at < (uint32_t)n) {
                    word[u] = __float_as_uint(part[at + skew]);
                    found |= 1u << u;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = threadIdx.x + u * BLOCK;
            if (i < PL) {
                const int p = i / L;
                const float a = pa[p];
                keys[i] = float_key(fmaf(a, __uint_as_float(word[u]), fmaf(1.f - a, pd[p], cst[(int64_t)pid[p] * L + (i - p * L)])));
            }
        }
    } else if constexpr (STREAM == 0) {
#pragma unroll 4
        for (int i = threadIdx.x; i < PL; i += BLOCK) {
            const int p = i / L, l = i - p * L;
            const int64_t r = pid[p];
            const float a = pa[p];
            const float ds = row[nbr[r * L + l]];
            keys[i] = float_key(fmaf(a, ds, fmaf(1.f - a, pd[p], cst[r * L + l])));
        }
    }
    if constexpr (STREAM >= 0) {
        __syncthreads();
        load_run<BLOCK>(keys, PL, kv, same);
    }
    block_select_runs<BLOCK>(kv, ipt, (uint32_t)S, sh, pivot, need);   // (every key is in registers behind its first barrier)
    float *base_of = &desc[q * S].base;                  // stride of one descriptor: 4 floats
    block_emit_runs<BLOCK>(kv, ipt, pivot, need, sh.scan, [&](uint32_t pos, int i, uint32_t k) {
        keys[pos] = (uint32_t)i;
        if (STREAM < 0) keys[S + pos] = __float_as_uint(key_float(k));
        else base_of[4 * pos] = key_float(k);
    });
    __syncthreads();
    const float per_l = 1.f / (float)L;                  // (i + 1/2) / L is at least 1/(2 L) from a whole number, and i below 2^15
    unsigned long long mine = 0;
    for (int p0 = 0; p0 < S; p0 += 4 * BLOCK) {
        uint4 info[4];
        int64_t sub[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int pos = p0 + u * BLOCK + (int)threadIdx.x;
            if (pos < S) {
                const int i = (int)keys[pos], p = (int)(((float)i + 0.5f) * per_l);
                sub[u] = (int64_t)pid[p] * L + (i - p * L);
                info[u] = sub_info[sub[u]];                // one 16-byte read per kept subregion
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int pos = p0 + u * BLOCK + (int)threadIdx.x;
            if (pos < S) {
                if (STREAM < 0) {
                    *reinterpret_cast<uint4 *>(&desc[q * S + pos]) = make_uint4(info[u].x, info[u].y, info[u].z, keys[S + pos]);
                } else {
                    uint32_t *d = &desc[q * S + pos].blk;  // blk, pos0, len: the first 12 bytes
                    d[0] = info[u].x;
                    d[1] = info[u].y;
                    d[2] = info[u].z;
                }
                if (kept_sub) kept_sub[q * S + pos] = sub[u];
                mine += info[u].z;
            }
        }
    }
    if (mine) atomicAdd(&codes_total, mine);
    __syncthreads();
    if (threadIdx.x == 0 && n_scanned) n_scanned[q] = (int64_t)codes_total;
}

template <int BLOCK, int MAXV, int STREAM = 0>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(STREAM ? 8 : 1, 8))) void score_prune_kernel(
    const float *__restrict__ Dt, int64_t ldt, int64_t K, const int32_t *__restrict__ probe_id,
    const float *__restrict__ probe_d, int P, int L, const int32_t *__restrict__ nbr,
    const float *__restrict__ cst, const float *__restrict__ alpha, int S,
    const uint4 *__restrict__ sub_info,
    SubDesc *__restrict__ desc, int64_t *__restrict__ kept_sub, int64_t *__restrict__ n_scanned,
    int64_t nq, const float *__restrict__ Qt, int D, int M, const float *__restrict__ codebook,
    float *__restrict__ lut, int lut_per)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    if ((int64_t)blockIdx.x >= nq) {   // (uniform) a table workgroup
        const int64_t ql = ((int64_t)blockIdx.x - nq) * lut_per;
        lut_body<BLOCK>(Qt + ql * D, nq - ql < lut_per ? (int)(nq - ql) : lut_per, D, M, codebook, lut + ql * (int64_t)M * 256, reinterpret_cast<float *>(dyn));
        return;
    }
    __shared__ SelectRegs<score_bins<BLOCK, STREAM>()> sh;
    score_prune_body<BLOCK, MAXV, STREAM>(Dt, ldt, K, probe_id, probe_d, P, L, nbr, cst, alpha, S, sub_info, desc, kept_sub, n_scanned,
                                          blockIdx.x, dyn, sh);
}

// Rotation in front of the product quantiser (Section 4: OPQ-compressed displacements, one global
// rotation): Y[i] = R X[i] for n rows of D floats, with Rt = R transposed ([b][a] = R[a][b]) so
// that consecutive lanes read consecutive words.  A workgroup takes ROT_ROWS rows into LDS and
// every thread owns output components a = tid, tid + 256, ...; each component is one chain of
// fused multiply-adds in the order b = 0 .. D-1.  X and Y may be the same array (a workgroup reads
// its rows before it writes them).  Dynamic LDS: ROT_ROWS * D floats.
constexpr int ROT_ROWS = 16;

__global__ __launch_bounds__(256) void rotate_rows_kernel(const float *__restrict__ X, int64_t n, int D,
                                                          const float *__restrict__ Rt, float *__restrict__ Y)
{
    extern __shared__ float xs[];                       // [ROT_ROWS][D]
    const int64_t r0 = (int64_t)blockIdx.x * ROT_ROWS;
    const int rows = n - r0 < ROT_ROWS ? (int)(n - r0) : ROT_ROWS;
    for (int i = threadIdx.x; i < rows * D; i += 256) xs[i] = X[r0 * D + i];
    __syncthreads();
    for (int a = threadIdx.x; a < D; a += 256) {
        float acc[ROT_ROWS];
#pragma unroll
        for (int r = 0; r < ROT_ROWS; ++r) acc[r] = 0.f;
        for (int b = 0; b < D; ++b) {
            const float w = Rt[(int64_t)b * D + a];
#pragma unroll
            for (int r = 0; r < ROT_ROWS; ++r) acc[r] = fmaf(w, xs[r * D + b], acc[r]);   // rows past `rows` hold stale data, never stored
        }
        for (int r = 0; r < rows; ++r) Y[(r0 + r) * D + a] = acc[r];
    }
}

// out[b][a] = in[a][b] for a D x D matrix
__global__ __launch_bounds__(256) void transpose_square_kernel(const float *__restrict__ in, int D, float *__restrict__ out)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= D * D) return;
    const int a = i / D, b = i - a * D;
    out[b * D + a] = in[i];
}

}  // namespace ivf
