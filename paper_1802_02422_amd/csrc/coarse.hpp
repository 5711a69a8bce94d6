// Stage 1: squared distances from a tile of queries to all K centroids as an
// MFMA GEMM (||q||^2 - 2<q,c> + ||c||^2), and the exact per-query selection of
// the nprobe closest regions (exhaustive assignment, Section 3.1).
//
// The inner products run on the fp16 matrix cores at fp32 accuracy: every
// operand row is scaled by a power of two so that its largest magnitude lies in
// [2^14, 2^15) and split into hi = fp16(x) and lo = fp16(x - hi), which
// together carry 22 significant bits; <q,c> is accumulated in fp32 from the
// three products lo*hi + hi*lo + hi*hi per 16 dimensions (each fp16 product is
// exact in fp32; the dropped lo*lo term is below 2^-24 of |q_i c_i|), and the
// scales, being powers of two, are undone exactly in the epilogue.  The
// rounding error of a distance is that of an fp32 dot product with 18 instead
// of 96 accumulation steps.
#pragma once
#include <type_traits>

#include "select.hpp"

namespace ivf {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef uint32_t gu32x4 __attribute__((ext_vector_type(4)));

// Largest magnitude of count floats, as the bit pattern of a non-negative float (those order like unsigned integers);
// out must start at 0.  FINITE: infinities and values that are not numbers are left out, so that the scale taken from it
// is the others' own; else they count, one that is not a number as larger than infinity.  One atomic a workgroup: with
// one a wavefront and 2^16 of them the reduction of a 25 MB table took 0.75 ms, all of it spent at that one address.
template <bool FINITE>
__global__ __launch_bounds__(256) void absmax_kernel(const float *__restrict__ X, int64_t count,
                                                     uint32_t *__restrict__ out)
{
    __shared__ uint32_t best[4];
    uint32_t m = 0;
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
        const uint32_t v = __float_as_uint(X[i]) & 0x7FFFFFFFu;
        m = v > m && (!FINITE || v < 0x7F800000u) ? v : m;
    }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        const uint32_t v = __shfl_xor(m, o, WAVE);
        m = v > m ? v : m;
    }
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) m = best[w] > m ? best[w] : m;
        atomicMax(out, m);
    }
}

constexpr int DK = 16;                       // dimensions per operand stage
// packed width of a row: whole stages, and an even number of them (the GEMM loops are unrolled by two)
__host__ __device__ inline int packed_dim(int D) { return (D + 2 * DK - 1) / (2 * DK) * (2 * DK); }
// Rows a packed matrix of n rows must be allocated for: the GEMM tiles copy whole tiles of up
// to 256 rows without clamping (rows past n are read, their products are never stored).
__host__ __device__ inline int64_t packed_rows(int64_t n) { return (n + 255) / 256 * 256; }

// Operand packing for the GEMM: row r of X ([n][D] fp32) becomes packed_dim(D)/16
// (an even number of) stages of 64 bytes, stage t = [hi k0..7 | lo k0..7 | hi k8..15 | lo k8..15] of
// dimensions 16t + k (fp16, zero beyond D), scaled by s = 2^(14 - floor(log2 m)):
// m is the row's largest magnitude, or the whole matrix's when gmax (the result
// of absmax_kernel) is given.  Also writes ||row||^2 and 1/s (per row, or
// inv_scale[0] for a matrix-wide scale).  One wavefront per row.
__device__ __forceinline__ void split_row(const float *__restrict__ X, int64_t row, int D, const uint32_t *__restrict__ gmax,
                                          _Float16 *__restrict__ P, float *__restrict__ norm, float *__restrict__ inv_scale)
{
    const int lane = threadIdx.x & 63;
    const int Dp = packed_dim(D);
    float s2 = 0.f, m = 0.f;
    for (int i = lane; i < D; i += WAVE) {
        const float v = X[row * D + i];
        s2 = fmaf(v, v, s2);
        m = fmaxf(m, fabsf(v));
    }
    s2 = wave_sum(s2);
    if (gmax) {
        m = __uint_as_float(*gmax);
    } else {
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, WAVE));
    }
    int e = (m > 0.f && m < INFINITY) ? ilogbf(m) : 14;
    e = e < -100 ? -100 : e > 100 ? 100 : e;
    const float s = ldexpf(1.f, 14 - e);
    _Float16 *out = P + row * (int64_t)Dp * 2;
    for (int i = lane; i < Dp; i += WAVE) {
        const float v = i < D ? X[row * D + i] * s : 0.f;
        const _Float16 hi = (_Float16)v;
        const _Float16 lo = (_Float16)(v - (float)hi);
        const int at = (i >> 4) * 32 + ((i >> 3) & 1) * 16 + (i & 7);
        out[at] = hi;
        out[at + 8] = lo;
    }
    if (lane == 0) {
        norm[row] = s2;
        if (!gmax) inv_scale[row] = ldexpf(1.f, e - 14);
        else if (row == 0) inv_scale[0] = ldexpf(1.f, e - 14);
    }
}

__global__ __launch_bounds__(256) void split_rows_kernel(const float *__restrict__ X, int64_t n, int D,
                                                         const uint32_t *__restrict__ gmax,
                                                         _Float16 *__restrict__ P, float *__restrict__ norm,
                                                         float *__restrict__ inv_scale)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row < n) split_row(X, row, D, gmax, P, norm, inv_scale);
}

constexpr int GT = 128;        // tile: GT queries x GT centroids per workgroup
constexpr int DBUF = 2 * GT * DK;            // floats per operand buffer (A rows then B rows)
constexpr int ROWF = DK;                     // floats (4-byte units) per packed row stage: 64 bytes

// acc += <A row, B row> over one staged 16 dimensions for this lane's fragments:
// a[0]/b[0] hold hi, a[1]/b[1] lo of the lane half's 8 dimensions.  The small
// cross terms go first.  The centroids are the MFMA's row operand.
__device__ __forceinline__ floatx16 mfma3(const gu32x4 (&bfrag)[2], const gu32x4 (&afrag)[2], floatx16 acc, int which)
{
    const halfx8 bh = __builtin_bit_cast(halfx8, bfrag[0]), bl = __builtin_bit_cast(halfx8, bfrag[1]);
    const halfx8 ah = __builtin_bit_cast(halfx8, afrag[0]), al = __builtin_bit_cast(halfx8, afrag[1]);
    if (which == 0) return __builtin_amdgcn_mfma_f32_32x32x16_f16(bl, ah, acc, 0, 0, 0);
    if (which == 1) return __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, al, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, ah, acc, 0, 0, 0);
}

// One 128x128 tile of <Q[q], C[j]> per workgroup of 4 wavefronts; each
// wavefront owns a 64x64 quadrant as 2x2 v_mfma_f32_32x32x16_f16 accumulators.
// Operands are the packed rows above, copied global -> LDS by
// global_load_lds_dwordx4 (no registers, no ds_write) in stages of 16
// dimensions, two LDS buffers so that the copy of stage s+1 runs under the MFMA
// block of stage s with one barrier per stage.  A direct-to-LDS load puts lane
// i's 16 bytes at base + 16 i, so the layout is unpadded rows of four 16-byte
// chunks; bank conflicts of the operand reads are avoided by storing chunk f of
// row r in slot f ^ ((r >> 2) & 3) (each lane simply fetches the chunk that
// belongs to its slot).  Lane half h feeds dimensions [8h, 8h+8) of the stage:
// chunks 2h (hi) and 2h+1 (lo).  All variants of the kernel use this k order,
// so a query's distances do not depend on the batch it arrives in.
// In acc[i][j], lane l holds query (column) wq + 32i + l%32 and element v is
// centroid (row) wc + 32j + 8*(v/4) + 4*(l/32) + v%4, i.e. four groups of four
// consecutive centroids, which the epilogues store as 128-bit words and reduce
// without leaving the lane.  buf0 and buf1 each hold (128 + 128) rows x 64 bytes.
//
// HI = true: the operands are the hi-only tables of pack_hi_rows_kernel (a row stage of 64 bytes holds 32
// dimensions: for lane half h the chunks 2h and 2h+1 are its 8 dimensions of the stage's first and
// second 16), Dp is that table's row length in 4-byte units, and a stage is two products hi*hi: a
// third of the MFMA work and half the bytes for an approximation of <q,c> whose error the caller bounds.
template <bool HI = false>
__device__ __forceinline__ void gemm_tile(const _Float16 *__restrict__ Qp, int64_t nq, int64_t q0,
                                          const _Float16 *__restrict__ Cp, int64_t K, int64_t c0, int Dp,
                                          float *buf0, float *buf1, floatx16 (&acc)[2][2])
{
    typedef const __attribute__((address_space(1))) void *gptr_t;
    typedef __attribute__((address_space(3))) void *lptr_t;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64;
    const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // This wave's four copies per stage: 16-row blocks 4 wave .. 4 wave + 3 of the buffer, i.e. 64
    // consecutive rows of one operand (waves 0-1 the query rows, 2-3 the centroid rows).  Both
    // packed matrices are allocated up to a multiple of the tile height, so no row is clamped
    // (products of rows past the end are never stored), and the copies are one instruction in a
    // rolled loop: the compiler tracks only a handful of distinct LDS copies exactly.
    const int r0 = (wave & 1) * 64 + (lane >> 2);                      // first row inside the operand tile
    const int f = (lane & 3) ^ ((r0 >> 2) & 3);                        // chunk this slot holds (same for all four rows)
    const float *src0 = wave < 2 ? reinterpret_cast<const float *>(Qp) + (q0 + r0) * Dp + f * 4
                                 : reinterpret_cast<const float *>(Cp) + (c0 + r0) * Dp + f * 4;
    auto issue = [&](int k0, float *dst) {
#pragma nounroll
        for (int n = 0; n < 4; ++n)
            __builtin_amdgcn_global_load_lds((gptr_t)(src0 + (int64_t)n * 16 * Dp + k0),
                                             (lptr_t)(dst + (wave * 4 + n) * 256), 16, 0, 0);
    };
    auto compute = [&](const float *As) {
        const float *Bs = As + GT * ROWF;
        gu32x4 a[2][2], b[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ra = wq + i * 32 + l32, rb = wc + i * 32 + l32;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                a[i][p] = *reinterpret_cast<const gu32x4 *>(&As[ra * ROWF + (((2 * h + p) ^ ((ra >> 2) & 3)) << 2)]);
                b[i][p] = *reinterpret_cast<const gu32x4 *>(&Bs[rb * ROWF + (((2 * h + p) ^ ((rb >> 2) & 3)) << 2)]);
            }
        }
        // the four accumulators are independent: cycle through them so that no MFMA
        // waits for the one issued just before it
        if (HI) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, b[j][p]),
                                                                           __builtin_bit_cast(halfx8, a[i][p]), acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = mfma3(b[j], a[i], acc[i][j], e);
        }
    };
    // The two buffers are separate LDS objects and every step names them statically (the loop
    // is unrolled by two): the compiler can then tell that the operand reads of one buffer do
    // not depend on the copy in flight into the other, and leaves that copy running under the
    // MFMA block.
    const int stages = Dp / DK;               // (even for the hi/lo tables, any number for the hi-only ones)
    issue(0, buf0);
    for (int s = 0; s < stages; s += 2) {
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's copies of stage s have landed
        __syncthreads();                      // ... and everyone's; all waves are done with the other buffer
        if (s + 1 < stages) issue((s + 1) * DK, buf1);
        compute(buf0);
        if (s + 1 < stages) {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if (s + 2 < stages) issue((s + 2) * DK, buf0);
            compute(buf1);
        }
    }
    __syncthreads();   // operands are dead: the buffers may be reused
}

constexpr int BMW = 64;   // centroids per block minimum
constexpr int N_XCD = 8;  // workgroups are dealt round-robin to the 8 XCDs, each with its own L2

// Tile of workgroup b: XCD x = b % 8 owns the query tiles x, x+8, ... (a few hundred KB that
// stay in its L2) and sweeps the centroid tiles in order, so every XCD streams the centroid
// matrix once and the eight of them work on the same centroid tile at about the same time.
__device__ __forceinline__ bool tile_of_block(int64_t b, int tiles_q, int64_t &q0, int64_t &c0)
{
    const int tq_per = (tiles_q + N_XCD - 1) / N_XCD;
    const int xcd = (int)(b % N_XCD);
    const int64_t local = b / N_XCD;
    const int tq = (int)(local % tq_per) * N_XCD + xcd;
    q0 = (int64_t)tq * GT;
    c0 = (local / tq_per) * GT;
    return tq < tiles_q;
}

// The distance GEMMs deal the other way round: XCD x = b % 8 owns the centroid groups (of whatever many tiles) x, x + 8,
// ... and takes each of them through all query tiles, which are few: a group comes from memory once for the whole chip,
// and all XCDs have work however few the query tiles are.  Where the groups are no multiple of 8, which would leave some
// XCDs a group more than others, each takes an eighth of the tiles in a row; with fewer than 8 groups, where most XCDs would
// have none, a row goes through the groups of a query tile, so that a last group of few centroids is dealt evenly too
// (100 000 queries x 100, 1152, 2432: 143, 639, 1159 us with the groups dealt one by one, 69, 181, 271).
__device__ __forceinline__ bool group_of_block(int64_t b, int64_t tiles_q, int64_t groups, int64_t &tq, int64_t &group)
{
    const int64_t local = b / N_XCD, x = b % N_XCD;
    if (groups % N_XCD == 0) {
        tq = local % tiles_q;
        group = local / tiles_q * N_XCD + x;
        return true;
    }
    const int64_t at = x * ((groups * tiles_q + N_XCD - 1) / N_XCD) + local;
    if (groups < N_XCD) {
        tq = at / groups;
        group = at % groups;
    } else {
        tq = at % tiles_q;
        group = at / tiles_q;
    }
    return at < groups * tiles_q;
}

// workgroups of a launch that deals this way
inline int64_t group_grid(int64_t tiles_q, int64_t groups) { return (groups * tiles_q + N_XCD - 1) / N_XCD * N_XCD; }

constexpr int SLD = 64 + 4;   // row stride (floats) of a wavefront's 32x64 output staging area in LDS

// Epilogue of one 32-query x 64-centroid block held by a wavefront as two accumulators
// (acc[j]: centroids 32j .. 32j+31 of the block): distances max(0, qr + cn + m2 * acc), the
// block minimum per query into bm (BM_LDS: into the LDS word bm_lds[query of the block * bm_lds_stride]),
// and the distances out through the wavefront's LDS staging
// area, [query][centroid], so that 16 lanes cover one query row and every store instruction
// writes four rows of 256 contiguous bytes, as streaming (non-temporal) stores: the matrix is
// far larger than the caches and is read back by other kernels only after this one has ended,
// and on the MI355X the sweep kernel runs 10 % faster with them than with ordinary stores.
// qb / cb: first query / centroid of the block;
// cnw: the 64 centroid norms of the block (LDS).  EDGE = false skips all bounds checks (the
// block lies inside Dt and K is a multiple of 4).
template <bool EDGE, int SROWS = 32, bool BM_LDS = false>
__device__ __forceinline__ void emit_block(const floatx16 (&acc)[2], float qr, float m2, const float *cnw,
                                           float *stage, int64_t qb, int64_t nq, int64_t cb, int64_t K,
                                           float *__restrict__ Dt, int64_t ldt, float *__restrict__ bm, int nb,
                                           float *bm_lds = nullptr, int bm_lds_stride = 0)
{
    static_assert(SROWS == 32 || SROWS == 16, "the staging area holds 32 or 16 query rows");
    const int lane = threadIdx.x & 63;
    const int l32 = lane & 31, h = lane >> 5;
    const int sr = lane >> 4, sc = (lane & 15) * 4;
    float4 d[2][4];
    float m = INFINITY;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int cl = j * 32 + 8 * g + 4 * h;          // centroid of element 4g inside the block
            const float4 cv = *reinterpret_cast<const float4 *>(&cnw[cl]);
            float4 &e = d[j][g];
            e.x = fmaxf(fmaf(m2, acc[j][4 * g + 0], qr + cv.x), 0.f);
            e.y = fmaxf(fmaf(m2, acc[j][4 * g + 1], qr + cv.y), 0.f);
            e.z = fmaxf(fmaf(m2, acc[j][4 * g + 2], qr + cv.z), 0.f);
            e.w = fmaxf(fmaf(m2, acc[j][4 * g + 3], qr + cv.w), 0.f);
            if (EDGE) {
                const int64_t c = cb + cl;
                m = fminf(m, c + 0 < K ? e.x : INFINITY);
                m = fminf(m, c + 1 < K ? e.y : INFINITY);
                m = fminf(m, c + 2 < K ? e.z : INFINITY);
                m = fminf(m, c + 3 < K ? e.w : INFINITY);
            } else {
                m = fminf(fminf(m, e.x), fminf(e.y, fminf(e.z, e.w)));
            }
        }
    m = fminf(m, __shfl_xor(m, 32, WAVE));   // the other half holds the other 32 centroids
    const int64_t q = qb + l32, blk = cb / BMW;
    if (BM_LDS) {   // the caller collects the minima of several blocks and writes them out as whole sectors
        // (an explicit instruction: before an ordinary LDS write the compiler may wait for every
        // outstanding vector-memory operation when direct-to-LDS copies are in flight)
        const uint32_t at = (uint32_t)reinterpret_cast<uintptr_t>(bm_lds + l32 * bm_lds_stride);   // LDS byte address
        if (h == 0) asm volatile("ds_write_b32 %0, %1" ::"v"(at), "v"(m) : "memory");
    } else if (h == 0 && (!EDGE || (q < nq && blk < nb))) {
        bm[q * nb + blk] = m;
    }
    // through the staging area, SROWS query rows at a time (the lanes of the other rows sit a pass out).
    // The interior path issues exactly (32 / SROWS) * (SROWS / 4) store instructions: the sweep kernel's
    // hand-counted waits depend on that number.
#pragma unroll
    for (int pass = 0; pass < 32 / SROWS; ++pass) {
        if (SROWS == 32 || (l32 / SROWS) == pass) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<float4 *>(&stage[(l32 % SROWS) * SLD + j * 32 + 8 * g + 4 * h]) = d[j][g];
        }
        wave_sync();
        const int64_t qp = qb + pass * SROWS;
        if (EDGE) {
            const bool vec = (K & 3) == 0;
#pragma unroll
            for (int it = 0; it < SROWS / 4; ++it) {
                const int r = it * 4 + sr;
                const int64_t qq = qp + r, c = cb + sc;
                const float4 v = *reinterpret_cast<const float4 *>(&stage[r * SLD + sc]);
                if (qq < nq) {
                    float *rowp = Dt + qq * ldt;
                    if (vec && c + 3 < K) {
                        *reinterpret_cast<float4 *>(rowp + c) = v;
                    } else {
                        const float dv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (c + e < K) rowp[c + e] = dv[e];
                    }
                }
            }
        } else {
            float *p = Dt + (qp + sr) * ldt + cb + sc;
#pragma unroll
            for (int it = 0; it < SROWS / 4; ++it) {
                __builtin_nontemporal_store(*reinterpret_cast<const floatx4 *>(&stage[(it * 4 + sr) * SLD + sc]),
                                            reinterpret_cast<floatx4 *>(p));
                p += 4 * ldt;
            }
        }
        wave_sync();
    }
}

// Row stride of the distance matrix Dt in floats.  Unpadded: padding the rows (by 128 bytes up
// to 16 KB) made the tile stores slower on the MI355X, not faster.
__host__ __device__ inline int64_t dt_stride(int64_t K) { return K; }

// From this many query tiles on coarse_gemm_kernel deals query tiles to the XCDs (tile_of_block) instead of centroid tiles: an
// XCD then has three or more of them for every centroid tile that it reads (10 000 queries x 142 306, 96 dimensions 3553 us
// with centroid tiles dealt, 3100 so; x 20 001 435 and 388; 3072 142 and 130, 3404 157 and 157; 2500 111 and 123, 700 45 and 54).
constexpr int DEAL_QUERY_TILES = 24;

inline int64_t tile_grid(int64_t tiles_q, int64_t tiles_c)
{
    return tiles_q >= DEAL_QUERY_TILES ? (tiles_q + N_XCD - 1) / N_XCD * N_XCD * tiles_c : group_grid(tiles_q, tiles_c);
}

// Dt[q][j] = max(0, qn[q] + cn[j] - 2 <Q[q], C[j]>), and bm[q][b] = the minimum
// of Dt[q][64b .. 64b+63] (each wavefront's 64-centroid quadrant gives one block
// minimum per query).  qsi[q] and csi[0] are the inverse operand scales.  The
// grid has tile_grid(tiles_q, tiles_c) workgroups.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void coarse_gemm_kernel(
    const _Float16 *__restrict__ Qp, const float *__restrict__ qn, const float *__restrict__ qsi, int64_t nq,
    const _Float16 *__restrict__ Cp, const float *__restrict__ cn, const float *__restrict__ csi, int64_t K,
    int Dp, float *__restrict__ Dt, int64_t ldt, float *__restrict__ bm, int nb, int tiles_q)
{
    // two operand buffers of 256 rows x 64 bytes, each reused as the output staging of two wavefronts
    __shared__ __attribute__((aligned(16))) float ops0[2 * 32 * SLD];
    __shared__ __attribute__((aligned(16))) float ops1[2 * 32 * SLD];
    static_assert(DBUF <= 2 * 32 * SLD, "an operand buffer must fit the staging area of two wavefronts");
    __shared__ __attribute__((aligned(16))) float cns[GT];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int64_t q0, c0;
    if (tiles_q >= DEAL_QUERY_TILES) {
        if (!tile_of_block(blockIdx.x, tiles_q, q0, c0)) return;
    } else {
        if (!group_of_block(blockIdx.x, tiles_q, (K + GT - 1) / GT, q0, c0)) return;
        q0 *= GT;
        c0 *= GT;
    }
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64;
    const int l32 = lane & 31, h = lane >> 5;
    if (threadIdx.x < GT) cns[threadIdx.x] = c0 + threadIdx.x < K ? cn[c0 + threadIdx.x] : 0.f;
    floatx16 acc[2][2];
    gemm_tile(Qp, nq, q0, Cp, K, c0, Dp, ops0, ops1, acc);   // ends with a barrier: cns is visible, operands are dead
    const float m2c = -2.f * csi[0];
    float *stage = (wave < 2 ? ops0 : ops1) + (wave & 1) * (32 * SLD);
    const bool interior = q0 + GT <= nq && c0 + GT <= K && (K & 3) == 0;   // uniform over the workgroup
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t qb = q0 + wq + i * 32, q = qb + l32;
        const float qr = q < nq ? qn[q] : 0.f;
        const float m2 = q < nq ? m2c * qsi[q] : 0.f;
        if (interior) emit_block<false>(acc[i], qr, m2, cns + wc, stage, qb, nq, c0 + wc, K, Dt, ldt, bm, nb);
        else emit_block<true>(acc[i], qr, m2, cns + wc, stage, qb, nq, c0 + wc, K, Dt, ldt, bm, nb);
    }
}

// s_waitcnt immediate that waits until at most n vector-memory operations of the wavefront are
// outstanding (they complete in issue order) and leaves the other counters alone.
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// Large batches, STAGES = packed_dim / 16 known at compile time: a workgroup keeps ONE query
// tile and sweeps `tiles_per_wg` consecutive centroid tiles.  Its query operand never passes
// through LDS: every lane holds the fragments of its query rows for all stages in registers
// (16 STAGES of them), so per centroid tile only the 128 centroid rows are copied
// (global -> LDS, 8 KB a stage) into a ring of RING buffers, PD = RING - 1 stages ahead (a copy
// takes a few microseconds to land, several steps' worth of MFMA work), and
// the ring keeps running across tiles: the copies of the next tile's first stages are in
// flight during the epilogue of the current one.  The distance stores of a workgroup walk
// along its 128 rows of Dt, tile after tile.  STAGES is a multiple of RING, so stage s of
// every tile uses buffer s % RING and each step names its buffer statically (separate LDS
// objects, see gemm_tile).  Same k order and products as gemm_tile: identical results.
//
// Waiting for a copy with operations issued after it still in flight relies on in-order
// completion; the counts below are the vector-memory operations a wavefront issues between a
// copy and the step that consumes it, or a lower bound of them (2 copies a step, at least 16
// stores an epilogue).  With six stages the ring holds a whole tile and every copy is issued
// ahead of the stores of the tile before the one it belongs to: a wavefront never has to wait
// for its stores to drain before it can go on, it runs up to one tile ahead of them.  Only whole
// tiles are handled (K a multiple of 128; the rows of a partial last query tile are computed
// too, into the padding of the per-query buffers).  The workgroup barrier of a step orders LDS
// traffic only (operands arrive by copies that each wavefront has waited for, nothing else is
// shared), so it is issued without the global-memory fence of __syncthreads, which would drain
// the queue at every step.
//
// Block minima: a tile gives every query two of them (one per 64-centroid half), 4 bytes each in
// 128 different rows of bm.  Written directly, those scattered words took a third of the
// kernel's store-path cycles; they are collected in LDS for SWEEP_BMC consecutive tiles instead
// and written as 64-byte pieces (16 consecutive blocks of a row).
constexpr int SWEEP_BMC = 8;   // tiles per write-out of the block minima

template <int STAGES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void coarse_gemm_sweep_kernel(
    const _Float16 *__restrict__ Qp, const float *__restrict__ qn, const float *__restrict__ qsi, int64_t nq,
    const _Float16 *__restrict__ Cp, const float *__restrict__ cn, const float *__restrict__ csi, int64_t K,
    float *__restrict__ Dt, int64_t ldt, float *__restrict__ bm, int nb, int tiles_q, int tiles_c, int tiles_per_wg)
{
    typedef const __attribute__((address_space(1))) void *gptr_t;
    typedef __attribute__((address_space(3))) void *lptr_t;
    constexpr int RING = STAGES <= 6 ? STAGES : 4;        // 6 stages: the ring holds a whole tile
    static_assert(STAGES % RING == 0 && STAGES >= RING && RING <= 6, "stage s of every tile must use buffer s % RING");
    constexpr int PD = RING - 1;
    constexpr int Dp = STAGES * DK;
    constexpr int SLOT = GT * ROWF;                        // floats per ring buffer: 128 rows x 64 bytes
    // Distance stores of one tile's interior epilogue per wavefront: two emit_block<false, SROWS = 16, true>
    // calls, each 32 / SROWS passes of SROWS / 4 store instructions for its two 32-centroid halves' 64
    // columns (one instruction covers 4 rows x 256 bytes).  The waits below count on exactly this number
    // of vector-memory operations between a copy and its consumer: emit_block's store count is part of
    // this kernel's contract.
    constexpr int EPI_SROWS = 16;
    constexpr int EPI_STORES = 2 * (32 / EPI_SROWS) * (EPI_SROWS / 4);
    static_assert(EPI_STORES == 16, "the vmcnt immediates of the sweep loop assume 16 epilogue stores per tile");
    __shared__ __attribute__((aligned(16))) float ring0[SLOT];
    __shared__ __attribute__((aligned(16))) float ring1[SLOT];
    __shared__ __attribute__((aligned(16))) float ring2[SLOT];
    __shared__ __attribute__((aligned(16))) float ring3[RING > 3 ? SLOT : 4];
    __shared__ __attribute__((aligned(16))) float ring4[RING > 4 ? SLOT : 4];
    __shared__ __attribute__((aligned(16))) float ring5[RING > 5 ? SLOT : 4];
    __shared__ __attribute__((aligned(16))) float stage_all[4 * 16 * SLD];   // 16 query rows per wavefront at a time
    __shared__ __attribute__((aligned(16))) float cns[2][GT];
    constexpr int BMC = SWEEP_BMC, BMLD = 2 * BMC + 4;     // row stride of the collected minima (floats)
    __shared__ __attribute__((aligned(16))) float bmbuf[GT * BMLD];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64;

    // workgroup -> (query tile, range of centroid tiles); step t of the workgroup is centroid tile tb + t
    int64_t tq, group;
    if (!group_of_block(blockIdx.x, tiles_q, (tiles_c + tiles_per_wg - 1) / tiles_per_wg, tq, group)) return;
    const int tb = (int)(group * tiles_per_wg);             // a multiple of SWEEP_BMC (the host's tiles_per_wg is)
    const int t_begin = 0;
    int t_end = tb < tiles_c ? tiles_c - tb : 0;            // steps inside the matrix
    if (t_end > tiles_per_wg) t_end = tiles_per_wg;
    if (t_begin >= t_end) return;
    const int64_t q0 = tq * GT;

    // this wave's two copies per stage: rows 32 wave + 16 n + lane / 4 of the centroid tile
    const int rl = wave * 32 + (lane >> 2);
    const int fl = (lane & 3) ^ ((lane >> 4) & 3);         // ((row >> 2) & 3 is the same for both rows)
    const float *cbase = reinterpret_cast<const float *>(Cp) + (int64_t)rl * Dp + fl * 4;
    auto slot_of = [&](int s) -> float * {
        const int r = s % RING;
        return r == 0 ? ring0 : r == 1 ? ring1 : r == 2 ? ring2 : r == 3 ? ring3 : r == 4 ? ring4 : ring5;
    };
    // copy stage s (may be >= STAGES: a stage of the following tile) of tile t; past the range the
    // last tile is copied again (never read), so that the number of copies per step is fixed
    auto issue = [&](int t, int s) {
        if (s >= STAGES) { s -= STAGES; ++t; }
        if (t >= t_end) t = t_end - 1;
        const float *src = cbase + (int64_t)(tb + t) * GT * Dp + s * DK;
        float *dst = slot_of(s) + wave * 512;
#pragma nounroll
        for (int n = 0; n < 2; ++n)
            __builtin_amdgcn_global_load_lds((gptr_t)(src + (int64_t)n * 16 * Dp), (lptr_t)(dst + n * 256), 16, 0, 0);
    };

    // RING == STAGES: the ring holds one whole tile; the copy of a stage of the next tile is issued
    // one step after that stage was consumed, and the last one right after the tile's MFMA work,
    // ahead of the epilogue's stores, so that no copy ever queues behind a store it is needed before.
    constexpr bool WHOLE = RING == STAGES;
#pragma unroll
    for (int s = 0; s < (WHOLE ? STAGES : PD); ++s) issue(t_begin, s);

    // query fragments: for stage s and block i the 32 bytes [hi | lo] of row wq + 32 i + l32, half h
    gu32x4 afr[STAGES][2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const gu32x4 *row = reinterpret_cast<const gu32x4 *>(reinterpret_cast<const float *>(Qp) + (q0 + wq + i * 32 + l32) * Dp) + 2 * h;
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            afr[s][i][0] = row[s * 4 + 0];
            afr[s][i][1] = row[s * 4 + 1];
        }
    }
    float qr[2], m2[2];
    {
        const float m2c = -2.f * csi[0];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t q = q0 + wq + i * 32 + l32;
            qr[i] = qn[q];
            m2[i] = m2c * qsi[q];
        }
    }
    cns[t_begin & 1][tid & (GT - 1)] = cn[(int64_t)tb * GT + (tid & (GT - 1))];
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // fragments and the first copies are in: the counts below start from an empty queue
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    float *stage = stage_all + wave * (16 * SLD);

    // Writes out the minima collected for steps [t0, t1) (t1 - t0 <= BMC, t0 a multiple of BMC): for each
    // of the tile's 128 queries the 2 (t1 - t0) consecutive blocks starting at block 2 (tb + t0).  Four
    // lanes cover a row's 64 bytes, one store instruction 16 rows.  Every wavefront's minima of these
    // steps must be in LDS (a workgroup barrier lies between their epilogues and this call).
    const bool bm_vec = (nb & 3) == 0;                    // rows of bm start on 16-byte boundaries
    auto flush_bm = [&](int t0, int t1) {
        const int ncol = 2 * (t1 - t0);
        const int cq = (tid & 3) * 4;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            const int row = pass * 64 + (tid >> 2);
            if (cq < ncol) {
                const float4 v = *reinterpret_cast<const float4 *>(&bmbuf[row * BMLD + cq]);
                float *dst = bm + (q0 + row) * (int64_t)nb + (int64_t)(tb + t0) * (GT / BMW) + cq;
                if (bm_vec && cq + 3 < ncol) {
                    *reinterpret_cast<float4 *>(dst) = v;
                } else {
                    const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (cq + u < ncol) dst[u] = e[u];
                }
            }
        }
    };

    float cn_next = 0.f;
    for (int t = t_begin; t < t_end; ++t) {
        const int64_t c0 = (int64_t)(tb + t) * GT;
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            // operations issued after the copy of this stage: the copies of the PD - 1 stages after it,
            // the norm load when it was issued in between, the epilogue stores when it lies in between
            // (the tile's one norm load is left out of the count: wherever the compiler places it,
            // waiting for one operation more than needed is harmless)
            constexpr int COPIES = 2 * (PD - 1);
            if (WHOLE) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * STAGES - 2 + EPI_STORES));   // the same count at every step
            else if (s < PD) __builtin_amdgcn_s_waitcnt(vmcnt_imm(COPIES + EPI_STORES));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(COPIES));
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (!WHOLE) issue(t, s + PD);
            else if (s >= 1) issue(t, STAGES + s - 1);
            // the minima of the last BMC tiles are complete (every wavefront is past their epilogues)
            if (s == 0 && t > t_begin && (t - t_begin) % BMC == 0) flush_bm(t - t_begin - BMC, t - t_begin);
            // this tile's centroid norms, requested at the end of the previous tile (below), go to LDS
            // in the middle of this one: the stores of the previous epilogue and the copies of the
            // steps since were issued after that load
            if (s == STAGES / 2 && t > t_begin) {
                asm volatile("s_waitcnt vmcnt(%1)" : "+v"(cn_next) : "n"(EPI_STORES + 2 * (STAGES / 2)));
                cns[t & 1][tid & (GT - 1)] = cn_next;
            }
            // The centroid fragments are read with explicit instructions: for an ordinary LDS read of a
            // buffer that copies write, the compiler waits for every outstanding vector-memory
            // operation (the stores of the previous epilogue included).  The waits above and the
            // barrier already order these reads after the copy they need.
            const uint32_t bs = (uint32_t)reinterpret_cast<uintptr_t>(slot_of(s));   // LDS byte address
            gu32x4 b[2][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int rb = wc + j * 32 + l32;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const uint32_t at = bs + 4u * (uint32_t)(rb * ROWF + (((2 * h + p) ^ ((rb >> 2) & 3)) << 2));
                    asm volatile("ds_read_b128 %0, %1" : "=v"(b[j][p]) : "v"(at));
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(b[0][0]), "+v"(b[0][1]), "+v"(b[1][0]), "+v"(b[1][1]));
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = mfma3(b[j], afr[s][i], acc[i][j], e);
        }
        if (WHOLE) {   // everyone is done with the last buffer: refill it before the stores go out
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            issue(t, 2 * STAGES - 1);
        }
        {   // norms of the next tile (index clamped past the end).  The load is hidden from the compiler,
            // which would otherwise drain the whole queue, stores included, where the value is used.
            // (cn_next's register is written when the load returns: nothing may read or move it before the
            // explicit wait at its use; the parity tests of this kernel are what checks a new build.)
            const int64_t cnx = c0 + GT + (tid & (GT - 1));
            const float *pn = cn + (cnx < K ? cnx : K - 1);
            asm volatile("global_load_dword %0, %1, off" : "=v"(cn_next) : "v"(pn) : "memory");
        }
        const float *cnw = cns[t & 1] + wc;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            emit_block<false, EPI_SROWS, true>(acc[i], qr[i], m2[i], cnw, stage, q0 + wq + i * 32, nq, c0 + wc, K, Dt, ldt, bm, nb,
                                        &bmbuf[(wq + i * 32) * BMLD + ((t - t_begin) % BMC) * 2 + (wave & 1)], BMLD);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no copy into LDS may outlive the workgroup
    __syncthreads();                              // the last epilogues' minima are in LDS
    flush_bm((t_end - t_begin - 1) / BMC * BMC, t_end - t_begin);
}

// The same for small batches (latency mode): a workgroup takes 32 QT queries x 256 centroids (QT = 1
// or 2), all four wavefronts share the queries and each owns 64 of the centroids (2 QT
// accumulators), so a batch of up to 32 queries costs a quarter of the MFMA work of the
// 128-query tile and the kernel is bounded by streaming the centroid matrix once per batch of
// up to 64 queries.  Operand rows in LDS: the query rows, then 256 centroid rows per buffer,
// staged like the large tile.
constexpr int SKQ = 32, SKC = 256;

template <int QT>
__global__ __launch_bounds__(256) void coarse_gemm_skinny_kernel(
    const _Float16 *__restrict__ Qp, const float *__restrict__ qn, const float *__restrict__ qsi, int64_t nq,
    const _Float16 *__restrict__ Cp, const float *__restrict__ cn, const float *__restrict__ csi, int64_t K,
    int Dp, float *__restrict__ Dt, int64_t ldt, float *__restrict__ bm, int nb, int tiles_q)
{
    typedef const __attribute__((address_space(1))) void *gptr_t;
    typedef __attribute__((address_space(3))) void *lptr_t;
    static_assert(QT == 1 || QT == 2, "one or two blocks of 32 queries");
    constexpr int QROWS = QT * SKQ;
    constexpr int SKBUF = (QROWS + SKC) * ROWF;   // floats per operand buffer
    // two operand buffers, each reused as the output staging of two wavefronts
    constexpr int OPS = SKBUF > 2 * 32 * SLD ? SKBUF : 2 * 32 * SLD;
    __shared__ __attribute__((aligned(16))) float ops0[OPS];
    __shared__ __attribute__((aligned(16))) float ops1[OPS];
    __shared__ __attribute__((aligned(16))) float cns[SKC];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // The query tiles of one block of 256 centroids go to the same XCD (workgroup b runs on XCD b % 8),
    // one after the other: the centroid rows are fetched from HBM once and found in that XCD's L2 by
    // the other tiles.  Grid: 8 * ceil(blocks / 8) * tiles_q workgroups.
    const int64_t local = blockIdx.x / N_XCD;
    const int64_t cblk = (local / tiles_q) * N_XCD + blockIdx.x % N_XCD;
    const int64_t q0 = (local % tiles_q) * QROWS, c0 = cblk * SKC;
    if (c0 >= K) return;                                           // (before any barrier; uniform)
    const int wc = wave * 64;
    const int l32 = lane & 31, h = lane >> 5;
    cns[tid] = c0 + tid < K ? cn[c0 + tid] : 0.f;
    floatx16 acc[QT][2];
#pragma unroll
    for (int i = 0; i < QT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    // Copies per stage: wave w takes the centroid blocks (16 rows each) w, w+4, w+8, w+12 with one
    // instruction in a rolled loop, the first 2 QT waves also one block of query rows (see gemm_tile).
    const int rl = lane >> 2;
    const int fq = (lane & 3) ^ ((rl >> 2) & 3);                       // (r >> 2) & 3 depends on the row inside the block only
    const float *srcc = reinterpret_cast<const float *>(Cp) + (c0 + wave * 16 + rl) * Dp + fq * 4;
    const float *srcq = reinterpret_cast<const float *>(Qp) + (q0 + (wave & (2 * QT - 1)) * 16 + rl) * Dp + fq * 4;
    auto issue = [&](int k0, float *dst) {
#pragma nounroll
        for (int n = 0; n < 4; ++n)
            __builtin_amdgcn_global_load_lds((gptr_t)(srcc + (int64_t)n * 64 * Dp + k0),
                                             (lptr_t)(dst + (2 * QT + wave + 4 * n) * 256), 16, 0, 0);
        if (wave < 2 * QT)
            __builtin_amdgcn_global_load_lds((gptr_t)(srcq + k0), (lptr_t)(dst + wave * 256), 16, 0, 0);
    };
    auto compute = [&](const float *As) {
        const float *Bs = As + QROWS * ROWF;
        gu32x4 a[QT][2], b[2][2];
#pragma unroll
        for (int i = 0; i < QT; ++i)
#pragma unroll
            for (int p = 0; p < 2; ++p)
                a[i][p] = *reinterpret_cast<const gu32x4 *>(&As[(i * 32 + l32) * ROWF + (((2 * h + p) ^ ((l32 >> 2) & 3)) << 2)]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int rb = wc + j * 32 + l32;
#pragma unroll
            for (int p = 0; p < 2; ++p)
                b[j][p] = *reinterpret_cast<const gu32x4 *>(&Bs[rb * ROWF + (((2 * h + p) ^ ((rb >> 2) & 3)) << 2)]);
        }
#pragma unroll
        for (int e = 0; e < 3; ++e)
#pragma unroll
            for (int i = 0; i < QT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma3(b[j], a[i], acc[i][j], e);
    };
    const int stages = Dp / DK;
    issue(0, ops0);
    for (int s = 0; s < stages; s += 2) {     // unrolled by two, see gemm_tile
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        issue((s + 1) * DK, ops1);
        compute(ops0);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        if (s + 2 < stages) issue((s + 2) * DK, ops0);
        compute(ops1);
    }
    __syncthreads();
    const float m2c = -2.f * csi[0];
    float *stage = (wave < 2 ? ops0 : ops1) + (wave & 1) * (32 * SLD);
    const bool interior = q0 + QROWS <= nq && c0 + SKC <= K && (K & 3) == 0;
#pragma unroll
    for (int i = 0; i < QT; ++i) {
        const int64_t qb = q0 + i * 32, q = qb + l32;
        const float qr = q < nq ? qn[q] : 0.f;
        const float m2 = q < nq ? m2c * qsi[q] : 0.f;
        if (interior) emit_block<false>(acc[i], qr, m2, cns + wc, stage, qb, nq, c0 + wc, K, Dt, ldt, bm, nb);
        else emit_block<true>(acc[i], qr, m2, cns + wc, stage, qb, nq, c0 + wc, K, Dt, ldt, bm, nb);
    }
}

// Nearest centroid only (P = 1): the same tile product, reduced on the fly to
// the per-query minimum of (distance, centroid id), merged across centroid
// tiles with a 64-bit atomic minimum; no distance tile is written.  best[]
// must be pre-filled with all ones.
__global__ __launch_bounds__(256) void coarse_argmin_kernel(
    const _Float16 *__restrict__ Qp, const float *__restrict__ qn, const float *__restrict__ qsi, int64_t nq,
    const _Float16 *__restrict__ Cp, const float *__restrict__ cn, const float *__restrict__ csi, int64_t K,
    int Dp, unsigned long long *__restrict__ best, int tiles_q)
{
    __shared__ __attribute__((aligned(16))) float ops0[DBUF];
    __shared__ __attribute__((aligned(16))) float ops1[DBUF];
    __shared__ __attribute__((aligned(16))) float cns[GT];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int64_t q0, c0;
    if (!tile_of_block(blockIdx.x, tiles_q, q0, c0)) return;
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64;
    const int l32 = lane & 31, h = lane >> 5;
    if (threadIdx.x < GT) cns[threadIdx.x] = c0 + threadIdx.x < K ? cn[c0 + threadIdx.x] : 0.f;
    floatx16 acc[2][2];
    gemm_tile(Qp, nq, q0, Cp, K, c0, Dp, ops0, ops1, acc);
    const float m2c = -2.f * csi[0];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t q = q0 + wq + i * 32 + l32;
        const float qr = q < nq ? qn[q] : 0.f;
        const float m2 = q < nq ? m2c * qsi[q] : 0.f;
        unsigned long long key = ~0ull;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int cl = wc + j * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                const int64_t c = c0 + cl;
                if (c < K) {
                    float d = fmaxf(fmaf(m2, acc[i][j][v], qr + cns[cl]), 0.f);
                    unsigned long long kc = ((unsigned long long)float_key(d) << 32) | (uint32_t)c;
                    key = kc < key ? kc : key;
                }
            }
        unsigned long long other = __shfl_xor(key, 32, WAVE);
        key = other < key ? other : key;
        if (h == 0 && q < nq) atomicMin(&best[q], key);
    }
}

__global__ __launch_bounds__(256) void argmin_unpack_kernel(const unsigned long long *__restrict__ best,
                                                            int64_t n, int32_t missing, int32_t *__restrict__ out_id,
                                                            float *__restrict__ out_d)
{   // missing: the id of a row without any distance that is a number
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    unsigned long long k = best[i];
    out_id[i] = k == ~0ull ? missing : (int32_t)(uint32_t)k;
    if (out_d) out_d[i] = key_float((uint32_t)(k >> 32));
}

// ---- Nearest centroid through a certified shortlist ----
// The nearest centroid of q is the one with the largest G = <q,c> - |c|^2 / 2.  The hi halves alone, one product
// per 16 dimensions instead of three, give it as g = <hq, hc> - |c|^2 / 2 with hq, hc the operands rounded to fp16
// (one power-of-two scale for all rows, one for the table).  With dq = q - hq and dc = c - hc, whose lengths are
// computed when the rows are packed,
//   <q,c> - <hq,hc> = <dq, c> + <hq, dc>,  so  |g - G| <= |dq| |c| + (|q| + |dq|) |dc| + roundings,
// the roundings of the accumulation and of the norms being below k (|q| |c| + |c|^2), k = (Dp + 32) 2^-24.  A tile of 128
// centroids has the largest |c| and |dc| in it: e(q, tile) = |dq| cm + (|q| + |dq|) dcm + k |q| cm.  The |c|^2 part of
// the bound goes into the product's start value: acc starts at -|c|^2 / 2 + k |c|^2, so that acc + e is an upper end
// of G and acc - 2 k |c|^2 - e a lower end.  L[q], the largest lower end seen so far, never exceeds the true maximum:
// every centroid that attains it has acc + e >= L[q] when it is looked at.  The kernel looks at the 16 centroids of a lane
// together: if their largest acc + e reaches L[q] it appends (q, those of the 16 that do, that upper end) to a list.  When all
// tiles have been seen, shortlist_pairs_kernel drops the entries whose upper end lies below L[q] by then (nearly all:
// entries made before the bound was tight), looks at the centroids of the others one by one with the lengths of their
// own instead of the tile's largest (rows of a table may lie many powers of two apart), which tightens L further, and
// lists the pairs that are left; rerank_kernel decides among those with exact arithmetic.  Stale reads of L only lengthen
// the lists.

// Rows of X ([n][D] fp32) as fp16 in the layout of gemm_tile<true>: per 32 dimensions the 16-byte chunks [k 0-7 | k
// 16-23 | k 8-15 | k 24-31], so that lane half h finds its dimensions of the two 16-wide products in chunks 2h and
// 2h+1; zero beyond D and in the rows n .. n_pad-1.  Scaled by 2^(14 - floor(log2 m)), m the largest magnitude *gmax.
// len[r] = (|row|, |row - packed row|) in scaled units (n_pad of them), both rounded up and at least 2^-50: what a square
// loses below fp32's range (a row 2^-89 the size of the largest) cannot make a length too short.  A row whose length is
// not a number or beyond fp32 is packed as zeros, its lengths infinite: it has no nearest centroid, and as a centroid it
// is nobody's.  16 lanes per row, a chunk of 8 dimensions a lane: whole 16-byte stores, 32-byte reads.
__host__ __device__ inline int hi_scale(uint32_t gmax_bits)
{
    const int e = (int)(gmax_bits >> 23) - 127;             // (a subnormal or zero maximum: the clamp)
    return 14 - (e < -62 ? -62 : e > 62 ? 62 : e);
}

__global__ __launch_bounds__(256) void pack_hi_rows_kernel(const float *__restrict__ X, int64_t n, int64_t n_pad, int D, int Dp,
                                                           const uint32_t *__restrict__ gmax, _Float16 *__restrict__ H,
                                                           float2 *__restrict__ len)
{
    const int64_t row = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const int lane = threadIdx.x & 15;
    if (row >= n_pad) return;
    const int sh = hi_scale(*gmax);
    float s2 = 0.f, d2 = 0.f;
    for (int ch = lane; ch < Dp / 8; ch += 16) {
        const int dim = 32 * (ch >> 2) + 8 * ((ch & 1) * 2 + ((ch & 3) >> 1));   // chunks 0,1,2,3 hold k 0, 16, 8, 24
        halfx8 w;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (row < n && dim + 4 * u < D) v = *reinterpret_cast<const float4 *>(X + row * D + dim + 4 * u);   // (D is a multiple of 4)
            const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float f = __builtin_amdgcn_ldexpf(e[t], sh);
                const _Float16 hi = (_Float16)f;
                const float d = f - (float)hi;
                w[4 * u + t] = hi;
                s2 = fmaf(f, f, s2);
                d2 = fmaf(d, d, d2);
            }
        }
        *reinterpret_cast<halfx8 *>(H + row * (int64_t)Dp + ch * 8) = w;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        s2 += __shfl_xor(s2, o, WAVE);
        d2 += __shfl_xor(d2, o, WAVE);
    }
    const bool fits = s2 < INFINITY && d2 < INFINITY;
    if (!fits)
        for (int ch = lane; ch < Dp / 8; ch += 16) *reinterpret_cast<gu32x4 *>(H + row * (int64_t)Dp + ch * 8) = gu32x4{0u, 0u, 0u, 0u};
    if (lane == 0)
        len[row] = fits ? make_float2(sqrtf(s2 + 0x1p-100f) * (1.f + 0x1p-10f), sqrtf(d2 + 0x1p-100f) * (1.f + 0x1p-10f)) : make_float2(INFINITY, INFINITY);
}

// Start values and bounds of the centroids for rows of scale *xmax: start[c] = (-1/2 + k) |c|^2 in units of the product,
// -inf for c in [K, tiles * 128) and for centroids without a length; tile[t] = (largest |c|, largest |dc|, smallest start
// value) of tile t, the lengths in the table's units.
__global__ __launch_bounds__(128) void shortlist_tiles_kernel(const float2 *__restrict__ clen, int64_t K, int Dp, const uint32_t *__restrict__ cmax,
                                                              const uint32_t *__restrict__ xmax, float *__restrict__ start,
                                                              float4 *__restrict__ tile)
{
    __shared__ float4 part[2];
    const int64_t c = (int64_t)blockIdx.x * 128 + threadIdx.x;
    float2 l = make_float2(0.f, 0.f);
    float v = -INFINITY, low = INFINITY;
    if (c < K) l = clen[c];
    if (!(l.x < INFINITY)) {
        l = make_float2(0.f, 0.f);
    } else if (c < K) {
        // (the length was rounded up by 2^-10: not into the start value, which has to be |c|^2 to k)
        const float len0 = l.x * (1.f / (1.f + 0x1p-10f));
        v = low = (-0.5f + (float)(Dp + 32) * 0x1p-24f) * __builtin_amdgcn_ldexpf(len0 * len0, hi_scale(*xmax) - hi_scale(*cmax));
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

constexpr int SHORTLIST_SEGS = 64;

// One entry of the list: query, first of the lane's 16 centroids, which of them (bit v: centroid c + 8 (v / 4) + v % 4),
// the largest upper end.  A pair has a whole centroid.  The segments have a counter each (128 bytes apart), so that the
// appends of different workgroups do not all queue at one address.  Entries beyond a segment's capacity are dropped (the
// caller compares the counters with the capacity and falls back to the exact kernel).
struct ShortEntry { int q, c; uint32_t which; float up; };
struct ShortPair { int q, c; float up; };

struct ShortlistArgs {
    const _Float16 *Qh;          // packed rows
    const float2 *qlen;          // their lengths
    int64_t nq, K;
    const _Float16 *Ch;          // packed centroids
    const float *start;          // start values, whole tiles
    const float4 *tile;          // per tile bounds
    const float2 *clen;          // lengths of the centroids, whole tiles
    int Dp;
    uint32_t *L;                 // [nq] float_key of the largest lower end seen (starts at 0: below every key)
    uint32_t *n_pairs;           // [nq] pairs of a row (starts at 0)
    ShortEntry *list;
    ShortPair *pairs;
    unsigned long long *count, *pair_count;
    unsigned long long seg_cap, pair_cap;
    int tiles_q, tiles_c;
};

// (c: |c|, d: |dc|)
__device__ __forceinline__ float shortlist_eps(float2 ql, float c, float d, int Dp)
{
    return fmaf(ql.y, c, fmaf(ql.x + ql.y, d, (float)(Dp + 32) * 0x1p-24f * ql.x * c));
}

// The larger of a lane's value and that of the other lane half (the same query, the other 16 centroids).
__device__ __forceinline__ float max_of_halves(float v)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}

// Bit v: acc[v] reaches thr.
__device__ __forceinline__ uint32_t reaching(const floatx16 &acc, float thr)
{
    uint32_t w = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) w |= (acc[v] >= thr ? 1u : 0u) << v;
    return w;
}

// Lower end of G of the value top of a tile whose smallest start value is low (acc - 2 k |c|^2 - eps, and a start
// value is (-1/2 + k) |c|^2).
__device__ __forceinline__ float shortlist_lower(float top, float low, float eps, int Dp)
{
    const float k = (float)(Dp + 32) * 0x1p-24f, back = 2.f * k / (0.5f - k);
    return fmaf(back, low, top) - eps;
}

// Any packed dimension: the tile loop of gemm_tile, one tile of 128 x 128 a workgroup.
__global__ __launch_bounds__(256) void coarse_shortlist_kernel(ShortlistArgs a)
{
    ShortEntry *list = a.list + (blockIdx.x % SHORTLIST_SEGS) * a.seg_cap;
    unsigned long long *count = a.count + (blockIdx.x % SHORTLIST_SEGS) * 16;
    __shared__ __attribute__((aligned(16))) float ops0[DBUF];
    __shared__ __attribute__((aligned(16))) float ops1[DBUF];
    __shared__ __attribute__((aligned(16))) float cns[GT];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int64_t q0, c0;
    if (!tile_of_block(blockIdx.x, a.tiles_q, q0, c0)) return;
    const int wq = (wave >> 1) * 64, wc = (wave & 1) * 64;
    const int l32 = lane & 31, h = lane >> 5;
    if (threadIdx.x < GT) cns[threadIdx.x] = a.start[c0 + threadIdx.x];
    // the bounds as they stand now, requested before the product so that their latency is hidden under it
    // (an older bound is a weaker one, never a wrong one)
    uint32_t seen[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t q = q0 + wq + i * 32 + l32;
        seen[i] = q < a.nq ? __hip_atomic_load(&a.L[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    }
    floatx16 acc[2][2];
    gemm_tile<true>(a.Qh, a.nq, q0, a.Ch, 0, c0, a.Dp / 2, ops0, ops1, acc);
    const float4 tl = a.tile[c0 / GT];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t q = q0 + wq + i * 32 + l32;
        float2 ql = q < a.nq ? a.qlen[q] : make_float2(INFINITY, INFINITY);
        const bool qok = ql.x < INFINITY;
        if (!qok) ql = make_float2(0.f, 0.f);
        const float eps = shortlist_eps(ql, tl.x, tl.y, a.Dp);
        const float before = !qok ? INFINITY : seen[i] ? key_float(seen[i]) : -INFINITY;   // (a row past the end, or without a length, reports nothing)
        float bound = before;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float top = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][j][v] += cns[wc + j * 32 + 8 * (v >> 2) + 4 * h + (v & 3)];
                top = fmaxf(top, acc[i][j][v]);
            }
            bound = max_of_halves(fmaxf(bound, shortlist_lower(top, tl.z, eps, a.Dp)));
            if (top + eps >= bound && top > -INFINITY) {
                const unsigned long long at = atomicAdd(count, 1ull);
                if (at < a.seg_cap) list[at] = ShortEntry{(int)q, (int)c0 + wc + j * 32 + 4 * h, reaching(acc[i][j], bound - eps), top + eps};
            }
        }
        if (qok && h == 0 && bound > before) atomicMax(&a.L[q], float_key(bound));
    }
}

// A tile of GT fp16 rows of SH 64-byte stages in LDS: the rows as they lie in memory, so that each load of 1 KB takes whole
// 128-byte lines (16 rows' 64 bytes of a stage a load: the loads of the other halves of the lines waited for them: 500 000 rows x 65 536 6.2 - 6.4 ms,
// 6.0 so; 10 000 x 2^20 block maxima 2.28 and 2.05), with
// the 16-byte chunks of row r at their number ^ tile_twist(r): 16 rows' reads of a chunk then go to all banks.
template <int SH>
__device__ __forceinline__ uint32_t tile_twist(int r) { return SH == 4 ? r & 15 : SH == 2 ? (r >> 1) & 7 : (r >> 2) & 3; }

// ... of the row that lane `lane` copies a chunk of in piece n = wave, wave + 4, ..: the same for all of them but for three stages
template <int SH>
struct TileTwists {
    uint32_t word = 0;
    __device__ __forceinline__ TileTwists(int wave, int lane)
    {
#pragma unroll
        for (int k = 0; k < (SH == 3 ? 2 * SH : 1); ++k) word |= tile_twist<SH>((64 * (wave + 4 * k) + lane) / (4 * SH)) << (2 * k);
    }
    __device__ __forceinline__ uint32_t of(int n) const { return SH == 3 ? word >> (2 * (n >> 2)) & 3u : word; }
};

// ---- sweeps: a workgroup of four wavefronts keeps the fragments of its rows (queries, points) in registers, 64 a wavefront, and goes
// through tiles of 128 centroids in two LDS buffers, one barrier a tile: the copies of tile t + 1 are issued right behind the
// barrier of tile t and waited for at the barrier of tile t + 1.  The buffers are objects of their own, so that the compiler knows
// that reads of one do not have to wait for copies into the other (only direct-to-LDS copies write them).
// Rows a workgroup takes: 64 for each of its wavefronts where there are products enough to fill the chip that way (three workgroups
// a compute unit), or 64 for two of them, which leaves more workgroups and shorter steps.  By rows x centroids, us
// with two wavefronts to 64 rows / with one: 600 x 65 536 39 / 43, 2000 x 65 536 56 / 47, 5000 x 65 536 88 / 89, 20 000 x 2000 23 / 27,
// 20 000 x 16 384 90 / 79, 100 000 x 1000 46 / 49, 100 000 x 16 384 407 / 340.
inline bool sweep_wide(int64_t rows, int64_t K) { return rows > 2 * GT && (rows + GT - 1) / GT * ((K + GT - 1) / GT) >= 8192; }

// ... of the nearest-centroid sweep, which deals its blocks of rows to the XCDs: an XCD gets up to ceil(rows / 2048) blocks of 256 or ceil(rows / 1024) of 128,
// and where the latter is odd the former are half a block more.  That is more than the wide sweep gains while an XCD has few blocks and they have many
// tiles to go through.  Whole calls of 96 dimensions, rows x centroids, us with two wavefronts to 64 rows / with one: 1000 x 2^20 527 / 634, 2000 x 2^20
// 684 / 641, 2560 x 2^20 852 / 941, 1000 x 200 000 209 / 222, 3000 x 200 000 270 / 292, 3584 x 200 000 308 / 294, 5000 x 200 000 345 / 352, 7000 x 200 000 411 / 425,
// 9000 x 200 000 498 / 483, 5000 x 131 072 274 / 280, 7000 x 131 072 327 / 323, 5000 x 100 000 257 / 256, 3000 x 65 536 176 / 178, 7000 x 65 536 230 / 224.
inline bool shortlist_wide(int64_t rows, int64_t K)
{
    const int64_t each = (rows + N_XCD * GT - 1) / (N_XCD * GT);
    return sweep_wide(rows, K) && !(each % 2 && each <= 7 && K >= 21000 * each);
}

template <int SH>
struct SweepTile {
    float rows[SH * GT * ROWF];
    float start[GT];                                       // start values of the products' accumulators
};

// Tile `tile` of the table into buf: 8 SH pieces of 1 KB, dealt to the wavefronts (tile_twist), and from two of them 64 of the start values each
template <int SH>
__device__ __forceinline__ void sweep_copy(const _Float16 *Ch, const float *start, int64_t tile, SweepTile<SH> &buf, const TileTwists<SH> &twists, int wave, int lane)
{
    typedef const __attribute__((address_space(1))) void *gptr_t;
    typedef __attribute__((address_space(3))) void *lptr_t;
    if (wave < 2) __builtin_amdgcn_global_load_lds((gptr_t)(start + tile * GT + wave * 64 + lane), (lptr_t)(buf.start + wave * 64), 4, 0, 0);
    const float *src = reinterpret_cast<const float *>(Ch) + tile * (GT * SH * DK);
    // (one instruction in a rolled loop: the compiler tracks only a handful of distinct LDS copies exactly)
#pragma nounroll
    for (int n = wave; n < 8 * SH; n += 4)
        __builtin_amdgcn_global_load_lds((gptr_t)(src + n * 256 + 4 * (lane ^ (int)twists.of(n))), (lptr_t)(buf.rows + n * 256), 16, 0, 0);
}

// This wavefront's copies are in, then everyone's, and everyone is through with the other buffer.
__device__ __forceinline__ void sweep_barrier()
{
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int SH>
__device__ __forceinline__ void sweep_rows(gu32x4 (&afr)[SH][2][2], const _Float16 *rows, int64_t first, int l32, int h)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const gu32x4 *row = reinterpret_cast<const gu32x4 *>(reinterpret_cast<const float *>(rows) + (first + i * 32 + l32) * (SH * DK)) + 2 * h;
#pragma unroll
        for (int s = 0; s < SH; ++s) {
            afr[s][i][0] = row[s * 4 + 0];
            afr[s][i][1] = row[s * 4 + 1];
        }
    }
}

// The products of a wavefront's 64 rows with JN blocks of 32 centroids from row wc of the tile on; each(j, acc) looks at a
// block's: acc[i][v] is that of row 32 i + lane % 32 and centroid wc + 32 j + 8 (v / 4) + 4 (lane / 32) + v % 4.  A block's first fragments
// are on their way while the one before is looked at, the others under the first products.
template <int SH, int JN, class Each>
__device__ __forceinline__ void sweep_tile(const SweepTile<SH> &buf, const gu32x4 (&afr)[SH][2][2], int wc, int l32, int h, Each each)
{
    union Start { floatx16 all; floatx4 part[4]; };
    gu32x4 b[SH][2];
    Start start;
    const uint32_t tw = tile_twist<SH>(l32);               // (the same for all blocks of 32)
    auto load_start = [&](int j) {
        const float *c = buf.start + wc + j * 32 + 4 * h;
#pragma unroll
        for (int k = 0; k < 4; ++k) start.part[k] = *reinterpret_cast<const floatx4 *>(c + 8 * k);
    };
    auto load = [&](int j, int s) {
        const float *r = buf.rows + (wc + j * 32 + l32) * (SH * DK);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t chunk = SH & 1 ? 4u * s + ((uint32_t)(2 * h + p) ^ tw) : (uint32_t)(4 * s + 2 * h + p) ^ tw;
            b[s][p] = *reinterpret_cast<const gu32x4 *>(r + 4 * chunk);
        }
    };
    load(0, 0);
    load_start(0);
#pragma unroll
    for (int j = 0; j < JN; ++j) {
        floatx16 acc[2];
#pragma unroll
        for (int s = 1; s < SH; ++s) load(j, s);
#pragma unroll
        for (int s = 0; s < SH; ++s)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, b[s][p]), __builtin_bit_cast(halfx8, afr[s][i][p]),
                                                                    s == 0 && p == 0 ? start.all : acc[i], 0, 0, 0);
        if (j + 1 < JN) {
            load(j + 1, 0);
            load_start(j + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        each(j, acc);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The same pass for SH = 1 .. 4 stages of 32 dimensions (packed dimension up to 128) as a sweep over `tiles_per_wg` centroid tiles.
// JN = 4: a wavefront has 64 rows of its own and takes all of a tile with them, JN = 2: two wavefronts share 64 rows and take half
// a tile each (shortlist_wide).  The bound stays in registers over the sweep and reaches L[q] once.
// The start values arrive in the accumulators' layout as the C operand of the first product, so that nothing but the
// largest value of a lane is left to the vector units (8 instructions a block of 32 x 32 against 2 SH products of
// 32 cycles); three wavefronts a SIMD cover the LDS and barrier latencies.  A report is kept short, since the other three
// wavefronts wait for it at the tile's barrier: no look at single centroids, no LDS round trip, no atomic; the entries
// are held in LDS, 64 at a time, and those that the bounds have not overtaken meanwhile go out with one atomic.
// 500 000 rows x 16 384 (65 536) centroids, 96 dimensions: 1.38 (4.92) ms, 1.14 (1.28) PFLOP/s, where the library's product
// reaches 1.37.  With two wavefronts to 64 rows and every fragment waited for where it is read 1.58 - 1.67 (5.86): a tile was copied for half
// as many products and a wavefront had half as many between barriers.  All of a block's fragments ahead of the block before instead
// of the first: spills, 1.44 (5.13).  What is left is power: the matrix units are busy 0.53 (0.7) of the time, at 1.9 (1.6) GHz of 2.4.
template <int SH, int JN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void coarse_shortlist_sweep_kernel(
    ShortlistArgs a, int tiles_per_wg)
{
    __shared__ __attribute__((aligned(16))) SweepTile<SH> buf0;
    __shared__ __attribute__((aligned(16))) SweepTile<SH> buf1;
    __shared__ __attribute__((aligned(16))) uint2 held_all[4][WAVE];
    ShortEntry *list = a.list + (blockIdx.x % SHORTLIST_SEGS) * a.seg_cap;
    unsigned long long *count = a.count + (blockIdx.x % SHORTLIST_SEGS) * 16;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, h = lane >> 5;
    const int wq = (JN == 4 ? wave : wave >> 1) * 64, wc = JN == 4 ? 0 : (wave & 1) * 64;
    const int tq_per = (a.tiles_q + N_XCD - 1) / N_XCD;
    const int xcd = (int)(blockIdx.x % N_XCD);
    const int64_t local = blockIdx.x / N_XCD;
    const int tq = (int)(local % tq_per) * N_XCD + xcd;
    if (tq >= a.tiles_q) return;
    const int tb = (int)(local / tq_per) * tiles_per_wg;
    int t_end = tb < a.tiles_c ? a.tiles_c - tb : 0;
    if (t_end > tiles_per_wg) t_end = tiles_per_wg;
    if (t_end <= 0) return;
    const int64_t q0 = (int64_t)tq * (GT / 2 * JN) + wq;      // this wavefront's first row

    const TileTwists<SH> twists(wave, lane);
    float4 tl, tl_next;                                      // bounds of the tile, requested with its rows
    auto issue = [&](int t, SweepTile<SH> &buf) {
        const int tc = tb + (t < t_end ? t : t_end - 1);     // (past the range: never read)
        sweep_copy(a.Ch, a.start, tc, buf, twists, wave, lane);
        tl_next = a.tile[tc];
    };
    issue(0, buf0);

    gu32x4 afr[SH][2][2];
    float2 ql[2];
    float bound[2], before[2];
    bool qok[2];
    sweep_rows(afr, a.Qh, q0, l32, h);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t q = q0 + i * 32 + l32;
        ql[i] = q < a.nq ? a.qlen[q] : make_float2(INFINITY, INFINITY);
        qok[i] = ql[i].x < INFINITY;
        if (!qok[i]) ql[i] = make_float2(0.f, 0.f);
        // the bound as it stands now (an older bound is a weaker one, never a wrong one); a row past the end, or without a length,
        // has nothing to report
        const uint32_t seen = qok[i] ? __hip_atomic_load(&a.L[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        before[i] = bound[i] = !qok[i] ? INFINITY : seen ? key_float(seen) : -INFINITY;
    }

    // the wavefront's entries: row (6 bits), lane half, block (2 bits), tile (6 bits), which of the 16; upper end
    const uint32_t held = (uint32_t)reinterpret_cast<uintptr_t>(&held_all[wave][0]);
    int n_held = 0;                                           // (uniform)
    auto flush = [&]() {
        uint2 e;
        asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(e) : "v"(held + 8u * (uint32_t)lane));
        const int qi = (int)(e.x & 63u);
        const float b0 = __shfl(bound[0], qi & 31, WAVE), b1 = __shfl(bound[1], qi & 31, WAVE);
        const float up = __uint_as_float(e.y);
        const bool live = lane < n_held && up >= (qi & 32 ? b1 : b0);
        const uint64_t m = __ballot(live);
        if (m) {
            unsigned long long at = 0;
            if (lane == 0) at = atomicAdd(count, (unsigned long long)__popcll(m));
            at = __shfl(at, 0, WAVE) + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (live && at < a.seg_cap)
                list[at] = ShortEntry{(int)q0 + qi, (tb + (int)(e.x >> 9 & 63u)) * GT + wc + (int)(e.x >> 7 & 3u) * 32 + (int)(e.x >> 6 & 1u) * 4, e.x >> 16, up};
        }
        n_held = 0;
    };

    auto step = [&](int t, const SweepTile<SH> &buf) {
        float eps[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) eps[i] = shortlist_eps(ql[i], tl.x, tl.y, a.Dp);
        sweep_tile<SH, JN>(buf, afr, wc, l32, h, [&](int j, const floatx16 (&acc)[2]) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float top = acc[i][0];
#pragma unroll
                for (int v = 1; v < 16; ++v) top = __builtin_elementwise_maximum(top, acc[i][v]);
                if (__any(!(top + eps[i] < bound[i]))) {
                    if (!(top == top)) {                       // (largest of the values that are numbers)
                        top = -INFINITY;
#pragma unroll
                        for (int v = 0; v < 16; ++v) top = fmaxf(top, acc[i][v]);
                    }
                    bound[i] = max_of_halves(fmaxf(bound[i], shortlist_lower(top, tl.z, eps[i], a.Dp)));
                    const bool pass = top + eps[i] >= bound[i] && top > -INFINITY;
                    const uint64_t m = __ballot(pass);
                    const int n = __popcll(m);
                    if (n_held + n > WAVE) flush();
                    const uint32_t at = held + 8u * ((uint32_t)n_held + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)));
                    const uint2 e = make_uint2((uint32_t)(i * 32 + l32) | (uint32_t)h << 6 | (uint32_t)j << 7 | (uint32_t)t << 9 | reaching(acc[i], bound[i] - eps[i]) << 16,
                                               __float_as_uint(top + eps[i]));
                    if (pass) asm volatile("ds_write_b64 %0, %1" ::"v"(at), "v"(e) : "memory");
                    n_held += n;
                }
            }
        });
    };
    for (int t = 0; t < t_end;) {
        sweep_barrier();
        tl = tl_next;
        issue(t + 1, buf1);
        step(t, buf0);
        if (++t == t_end) break;
        sweep_barrier();
        tl = tl_next;
        issue(t + 1, buf0);
        step(t, buf1);
        ++t;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // no copy into LDS may outlive the workgroup
    flush();
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (qok[i] && h == 0 && bound[i] > before[i]) atomicMax(&a.L[q0 + i * 32 + l32], float_key(bound[i]));
}

// What the passes of a chunk start from, in one launch: best[0 .. m-1] all ones, zero[0 .. n_zero-1] and count[0 .. n_count-1] zeros
__global__ __launch_bounds__(256) void shortlist_clear_kernel(unsigned long long *__restrict__ best, int64_t m, unsigned long long *__restrict__ zero, int64_t n_zero,
                                                              unsigned long long *__restrict__ count, int64_t n_count)
{
    const int64_t step = (int64_t)gridDim.x * 256, t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t i = t; i < m; i += step) best[i] = ~0ull;
    for (int64_t i = t; i < n_zero; i += step) zero[i] = 0ull;
    for (int64_t i = t; i < n_count; i += step) count[i] = 0ull;
}

// Bounds to start with where a centroid of every row is known that is likely near it (the nearest one of the last round of
// k-means): L[q] = the lower end of its value, with its own lengths, as in shortlist_pairs_kernel.  A sweep that starts without
// reports a row whenever a centroid is nearer than all before it, ln K times, and with 32 rows to a block nearly half of the blocks:
// 500 000 rows x 16 384 1.38 ms, 1.32 with the bounds, which take 0.033, and shortlist_pairs_kernel 0.086 and 0.057.  Four lanes a row.
__global__ __launch_bounds__(256) void seed_bounds_kernel(ShortlistArgs a, const int32_t *__restrict__ near)
{
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
    const int64_t q = (int64_t)blockIdx.x * 64 + (threadIdx.x >> 2);
    const int part = threadIdx.x & 3;
    if (q >= a.nq) return;
    const int64_t c = near[q];
    if (c < 0 || c >= a.K) return;                           // (a row that is not finite has none)
    const gu32x4 *qr = reinterpret_cast<const gu32x4 *>(a.Qh + q * a.Dp), *cr = reinterpret_cast<const gu32x4 *>(a.Ch + c * a.Dp);
    float g = 0.f;
#pragma unroll 4
    for (int d = part; d < a.Dp / 8; d += 4) {
        const gu32x4 u = qr[d], w = cr[d];
#pragma unroll
        for (int t = 0; t < 4; ++t) g = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2, (uint32_t)u[t]), __builtin_bit_cast(halfx2, (uint32_t)w[t]), g, false);
    }
    g += __shfl_xor(g, 1, WAVE);
    g += __shfl_xor(g, 2, WAVE);
    const float2 ql = a.qlen[q], cl = a.clen[c];
    const float k = (float)(a.Dp + 32) * 0x1p-24f, back = 2.f * k / (0.5f - k), st = a.start[c];
    const float low = fmaf(back, st, g + st) - shortlist_eps(ql, cl.x, cl.y, a.Dp);
    if (part == 0 && low > -INFINITY) a.L[q] = float_key(low);
}

// Entries -> pairs.  A wavefront looks at 64 entries at a time; a lane whose entry L leaves forms the products of its
// centroids from the packed rows again, one after the other (one is usual).  Grid: (any, SHORTLIST_SEGS); a segment whose
// list overflowed is left alone.
__global__ __launch_bounds__(256) void shortlist_pairs_kernel(ShortlistArgs a)
{
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
    __shared__ ShortPair held_all[4][WAVE];                  // a wavefront's pairs: one atomic for 64 of them
    const int lane = threadIdx.x & 63;
    ShortPair *held = held_all[threadIdx.x >> 6];
    int n_held = 0;
    auto flush = [&]() {
        unsigned long long at = 0;
        if (lane == 0) at = atomicAdd(&a.pair_count[blockIdx.y * 16], (unsigned long long)n_held);
        at = __shfl(at, 0, WAVE) + lane;
        wave_sync();
        if (lane < n_held && at < a.pair_cap) a.pairs[blockIdx.y * a.pair_cap + at] = held[lane];
        wave_sync();
        n_held = 0;
    };
    const unsigned long long n = a.count[blockIdx.y * 16];
    if (n > a.seg_cap) return;
    const float k = (float)(a.Dp + 32) * 0x1p-24f, back = 2.f * k / (0.5f - k);
    for (unsigned long long i0 = (blockIdx.x * 4ull + (threadIdx.x >> 6)) * WAVE; i0 < n; i0 += (unsigned long long)gridDim.x * 4 * WAVE) {
        ShortEntry e = {0, 0, 0, 0.f};
        uint32_t seen = 0;
        if (i0 + lane < n) {
            e = a.list[blockIdx.y * a.seg_cap + i0 + lane];
            seen = __hip_atomic_load(&a.L[e.q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (float_key(e.up) < seen) e.which = 0;
        }
        while (__any(e.which != 0)) {
            const int v = e.which ? __builtin_ctz(e.which) : 0, c = e.c + 8 * (v >> 2) + (v & 3);
            bool pass = e.which != 0 && c < a.K;
            e.which &= e.which - 1;
            float up = 0.f;
            if (pass) {
                const gu32x4 *qr = reinterpret_cast<const gu32x4 *>(a.Qh + (int64_t)e.q * a.Dp), *cr = reinterpret_cast<const gu32x4 *>(a.Ch + (int64_t)c * a.Dp);
                float g = 0.f;
#pragma unroll 4
                for (int d = 0; d < a.Dp / 8; ++d) {
                    const gu32x4 u = qr[d], w = cr[d];
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        g = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2, (uint32_t)u[t]), __builtin_bit_cast(halfx2, (uint32_t)w[t]), g, false);
                }
                const float2 cl = a.clen[c];
                const float st = a.start[c], eps = shortlist_eps(a.qlen[e.q], cl.x, cl.y, a.Dp);
                g += st;
                up = g + eps;
                pass = float_key(up) >= seen;
                const uint32_t low = float_key(fmaf(back, st, g) - eps);
                if (pass && low > seen) {
                    atomicMax(&a.L[e.q], low);
                    seen = low;
                }
            }
            const uint64_t m = __ballot(pass);
            if (n_held + __popcll(m) > WAVE) flush();
            if (pass) atomicAdd(&a.n_pairs[e.q], 1u);
            if (pass) held[n_held + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = ShortPair{e.q, c, up};
            n_held += __popcll(m);
        }
    }
    if (n_held) flush();
}

// Exact decision among the pairs that the final bounds leave: a wavefront per pair computes |x - c|^2 from the fp32
// rows (differences squared, summed in a tree over the lanes: a few ulps) and merges (distance, id) into best[q] with a
// 64-bit atomic minimum.  best must be pre-filled with all ones.  A wavefront looks at up to 64 pairs at a time, fewer
// where the list is short, so that all wavefronts have some (11 575 rows: 69 us with 64 always).  Where the distances are not asked
// for (DIST = false), a row's only pair needs none: 500 000 rows, nearly all of which have one, 100 us, 13 so.
template <bool DIST>
__global__ __launch_bounds__(256) void rerank_kernel(const float *__restrict__ X, const float *__restrict__ C, int D, ShortlistArgs a,
                                                     unsigned long long *__restrict__ best)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long n = a.pair_count[blockIdx.y * 16];
    if (n > a.pair_cap) return;
    const unsigned long long waves = gridDim.x * 4ull, share = (n + waves - 1) / waves;
    const int step = share < 2 ? 2 : share > WAVE ? WAVE : (int)share;
    for (unsigned long long i0 = (blockIdx.x * 4ull + (threadIdx.x >> 6)) * step; i0 < n; i0 += waves * step) {
        ShortPair e = {0, 0, 0.f};
        bool live = lane < step && i0 + lane < n;
        if (live) {
            e = a.pairs[blockIdx.y * a.pair_cap + i0 + lane];
            live = float_key(e.up) >= a.L[e.q];
            if (!DIST && a.n_pairs[e.q] == 1u) {
                best[e.q] = (uint32_t)e.c;
                live = false;
            }
        }
        for (uint64_t todo = __ballot(live); todo; todo &= todo - 1) {
            const int s = __builtin_ctzll(todo);
            const int q = __builtin_amdgcn_readlane(e.q, s), cc = __builtin_amdgcn_readlane(e.c, s);
            const float *x = X + (int64_t)q * D, *c = C + (int64_t)cc * D;
            float d = 0.f;
            for (int k = lane; k < D; k += WAVE) {
                const float u = x[k] - c[k];
                d = fmaf(u, u, d);
            }
            d = wave_sum(d);
            if (lane == 0) atomicMin(&best[q], ((unsigned long long)float_key(d) << 32) | (uint32_t)cc);
        }
    }
}

// The P closest centroids of each query row of Dt by (distance, id), written
// in ascending centroid id.  One workgroup per query, in three steps:
//   1. t = the min(P, nb)-th smallest block minimum.  The P smallest block
//      minima are P distinct distances <= t, so every one of the P closest
//      centroids has distance <= t and lies in a block whose minimum is <= t.
//   2. list, in ascending order, every block with minimum < t (fewer than P)
//      and the first P blocks with minimum == t (a later such block is
//      preceded by at least P distances equal to t, so it cannot contribute).
//   3. exact radix select of the P smallest (distance, id) among the
//      elements of the listed blocks (at most 2P*64), read from Dt.
// blist is dynamic LDS of 2*P ints.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void probe_select_kernel(const float *__restrict__ Dt, int64_t ldt,
                                                             const float *__restrict__ bm, int64_t K,
                                                             int nb, int P,
                                                             int32_t *__restrict__ probe_id,
                                                             float *__restrict__ probe_d)
{
    __shared__ SelectShared sh;
    __shared__ uint32_t nflag_s;
    extern __shared__ int blist[];
    const int64_t q = blockIdx.x;
    const float *row = Dt + q * ldt;
    const float *bmr = bm + q * nb;
    auto keyb = [bmr](int64_t b) { return float_key(bmr[b]); };
    const uint32_t nselb = P < nb ? (uint32_t)P : (uint32_t)nb;
    uint32_t t, needb;
    block_radix_select<BLOCK>(keyb, nb, nselb, sh, t, needb);
    uint32_t nflag = block_emit_selected<BLOCK>(keyb, nb, 0xFFFFFFFFu, t, (uint32_t)P, sh,
                                                [&](uint32_t pos, int64_t b, uint32_t) { blist[pos] = (int)b; });
    if (threadIdx.x == 0) nflag_s = nflag;
    __syncthreads();
    nflag = nflag_s;
    auto keyv = [row, K](int64_t v, const int *bl) {
        int64_t c = (int64_t)bl[v >> 6] * BMW + (v & 63);
        return c < K ? float_key(row[c]) : 0xFFFFFFFFu;
    };
    auto key = [&](int64_t v) { return keyv(v, blist); };
    uint32_t pivot, need;
    block_radix_select<BLOCK>(key, (int64_t)nflag * BMW, (uint32_t)P, sh, pivot, need);
    block_emit_selected<BLOCK>(key, (int64_t)nflag * BMW, (uint32_t)P, pivot, need, sh,
                               [&](uint32_t pos, int64_t v, uint32_t k) {
                                   probe_id[q * P + pos] = blist[v >> 6] * BMW + (int)(v & 63);
                                   probe_d[q * P + pos] = key_float(k);
                               });
}

// The same selection with the keys held in registers, for nb <= PS_NB_MAX block minima and
// P <= PS_P_MAX: the block minima are read once (not once per radix pass), and of the flagged
// blocks' elements only those at or below the block threshold t are kept (t is the P-th
// smallest block minimum, so the P closest centroids are among them; with randomly numbered
// centroids little more than P survive), compacted in ascending centroid id, and selected
// from LDS.  A query with more than PS_CAP survivors (duplicated centroids) takes the
// global-memory path of probe_select_kernel.  Dynamic LDS: ps_lds_bytes(P).
constexpr int PS_NB_MAX = 16384, PS_P_MAX = 256, PS_CAP = 4096;
inline size_t ps_lds_bytes(int P) { return ((size_t)2 * P + 3 + 2 * PS_CAP) * sizeof(int); }

// (the body, for query q of the batch: also the first half of select_score_prune_kernel)
__device__ __forceinline__ void probe_select_lds_body(const float *__restrict__ Dt, int64_t ldt,
                                                      const float *__restrict__ bm, int64_t K, int nb, int P,
                                                      int32_t *__restrict__ probe_id, float *__restrict__ probe_d,
                                                      int64_t q, int *ps_dyn, SelectRegs<1024> &sh)
{
    constexpr int BLOCK = 1024;
    SelectShared &sh_mem = *reinterpret_cast<SelectShared *>(&sh);  // (only where more survive than fit)
    static_assert(sizeof(SelectShared) <= sizeof(sh), "the same place");
    __shared__ uint32_t nflag_s;
    int *blist = ps_dyn;                                           // 2P flagged blocks
    uint32_t *keys = reinterpret_cast<uint32_t *>(ps_dyn + ((2 * P + 3) & ~3));   // (16-byte aligned) the survivors
    const int tid = threadIdx.x;
    const float *row = Dt + q * ldt;
    const uint32_t *bmr = reinterpret_cast<const uint32_t *>(bm + q * nb);
    static_assert(PS_NB_MAX <= 16 * BLOCK && PS_CAP <= 4 * BLOCK, "items of a thread");
    uint32_t t, needb, nflag;
    {
        uint32_t kv[16];
        auto as_key = [](uint32_t w) { return float_key(__uint_as_float(w)); };
        if ((nb & 3) == 0) load_run<BLOCK>(bmr, nb, kv, as_key);
        else load_run<BLOCK, false>(bmr, nb, kv, as_key);
        block_select_runs<BLOCK>(kv, run_length<BLOCK>(nb), P < nb ? (uint32_t)P : (uint32_t)nb, sh, t, needb);
        nflag = block_emit_runs<BLOCK>(kv, run_length<BLOCK>(nb), t, (uint32_t)P, sh.scan,
                                       [&](uint32_t pos, int b, uint32_t) { blist[pos] = b; });
    }
    if (tid == 0) nflag_s = nflag;
    __syncthreads();                                               // blist complete
    nflag = nflag_s;
    const uint32_t tf = nb >= P ? t : 0xFFFFFFFFu;                 // fewer blocks than P: no filter
    // Candidates: the 64 distances of every flagged block, a block per wavefront and step (one
    // 256-byte row piece per load instruction), 16 blocks in flight per wavefront.  Survivors (at or
    // below the block threshold) are compacted in ascending centroid id: inside a wavefront by
    // ballots, across wavefronts by one workgroup scan of the wavefronts' counts per round.
    constexpr int CB = 16;                                         // blocks per wavefront and round
    const int wave = tid >> 6, lane = tid & 63;
    uint32_t *sk = keys;
    int *si = reinterpret_cast<int *>(keys + PS_CAP);
    uint32_t total = 0;                                            // survivors so far
    bool overflow = false;
    for (int b0 = 0; b0 < (int)nflag; b0 += CB * (BLOCK / WAVE)) { // uniform
        uint32_t kv[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            // (every lane loads, or each load would be waited for inside its branch)
            const int bi = b0 + wave * CB + j;
            const int64_t c = (int64_t)blist[bi < (int)nflag ? bi : 0] * BMW + lane;
            const uint32_t key = float_key(row[c < K ? c : K - 1]);
            kv[j] = bi < (int)nflag && c < K ? key : 0xFFFFFFFFu;
        }
        uint32_t wcnt = 0;
#pragma unroll
        for (int j = 0; j < CB; ++j) wcnt += (uint32_t)__popcll(__ballot(kv[j] <= tf && kv[j] != 0xFFFFFFFFu));
        uint32_t round_total;
        const uint32_t exc = block_exclusive_scan<BLOCK>(lane == 0 ? wcnt : 0u, sh.scan, round_total);
        if (total + round_total > (uint32_t)PS_CAP) { overflow = true; break; }   // uniform
        uint32_t at = total + (uint32_t)__builtin_amdgcn_readfirstlane((int)exc);   // the wavefront's next output slot
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const bool sel = kv[j] <= tf && kv[j] != 0xFFFFFFFFu;
            const uint64_t m = __ballot(sel);
            if (sel) {
                const uint32_t o = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                sk[o] = kv[j];
                si[o] = blist[b0 + wave * CB + j] * BMW + lane;
            }
            at += (uint32_t)__popcll(m);
        }
        total += round_total;
    }
    if (overflow || total < (uint32_t)P) {                          // uniform; the second cannot happen for nb >= P
        const int n_c = (int)nflag * BMW;
        __syncthreads();
        auto key = [&](int64_t v) {
            const int64_t c = (int64_t)blist[v >> 6] * BMW + (v & 63);
            return c < K ? float_key(row[c]) : 0xFFFFFFFFu;
        };
        uint32_t pivot, need;
        block_radix_select<BLOCK>(key, (int64_t)n_c, (uint32_t)P, sh_mem, pivot, need);
        block_emit_selected<BLOCK>(key, (int64_t)n_c, (uint32_t)P, pivot, need, sh_mem,
                                   [&](uint32_t pos, int64_t v, uint32_t k) {
                                       probe_id[q * P + pos] = blist[v >> 6] * BMW + (int)(v & 63);
                                       probe_d[q * P + pos] = key_float(k);
                                   });
        return;
    }
    __syncthreads();
    uint32_t kv[4], pivot, need;
    load_run<BLOCK>(sk, (int)total, kv, [](uint32_t w) { return w; });
    block_select_runs<BLOCK>(kv, 4, (uint32_t)P, sh, pivot, need);
    block_emit_runs<BLOCK>(kv, run_length<BLOCK>((int)total), pivot, need, sh.scan, [&](uint32_t pos, int i, uint32_t k) {
        probe_id[q * P + pos] = si[i];
        probe_d[q * P + pos] = key_float(k);
    });
}

__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8, 8))) void probe_select_lds_kernel(const float *__restrict__ Dt, int64_t ldt,
                                                                const float *__restrict__ bm, int64_t K,
                                                                int nb, int P,
                                                                int32_t *__restrict__ probe_id,
                                                                float *__restrict__ probe_d)
{
    extern __shared__ __attribute__((aligned(16))) int ps_dyn[];
    __shared__ SelectRegs<1024> sh;
    probe_select_lds_body(Dt, ldt, bm, K, nb, P, probe_id, probe_d, blockIdx.x, ps_dyn, sh);
}

// ---- The selection by one wavefront per query, for small tables ----
// The workgroup selection above spends its time in barriers when there are few keys for its 1024 threads (10 000 queries x
// 65 536 centroids, P = 64: 0.44 ms, 0.11 here).  With the keys of a query in the registers of one wavefront the nsel-th
// smallest is found by a binary search over the key's bits, a comparison and a population count a register and bit.

// pivot and need such that the nsel smallest keys are those below pivot and `need` of those equal to it (the first ones in
// order).  Keys of 0xFFFFFFFF are no keys; nsel is at most the number of keys.
template <int R>
__device__ __forceinline__ void wave_select(const uint32_t (&k)[R], uint32_t nsel, uint32_t &pivot, uint32_t &need)
{
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        lo = k[r] < lo ? k[r] : lo;
        hi = k[r] != 0xFFFFFFFFu && k[r] > hi ? k[r] : hi;
    }
    lo = wave_extreme<false>(lo);
    hi = wave_extreme<true>(hi);
    const int top = lo < hi ? 31 - __builtin_clz(lo ^ hi) : -1;   // highest bit in which keys differ
    uint32_t t = top >= 0 ? hi & ~((2u << top) - 1u) : lo;
    uint32_t below = 0;                                        // keys < t
    for (int bit = top; bit >= 0; --bit) {
        const uint32_t trial = t | 1u << bit;
        // counted per lane and added over the lanes: a population count per register goes through the scalar unit, whose
        // waits a lone wavefront has nothing to cover with (333 queries x 2000: 29 us, 26 so, 15 with all loads ahead of their use)
        uint32_t mine = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) mine += k[r] < trial ? 1u : 0u;
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(mine), WAVE - 1);
        if (c <= nsel) {
            t = trial;
            below = c;
            if (c == nsel) break;
        }
    }
    pivot = t;
    need = nsel - below;
}

// Calls emit(position among the selected, r, key) for the selected keys in the order r * 64 + lane.
template <int R, class EmitFn>
__device__ __forceinline__ void wave_emit(const uint32_t (&k)[R], uint32_t pivot, uint32_t need, EmitFn emit)
{
    uint32_t out = 0, eq_seen = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t eqm = __ballot(k[r] == pivot && need > 0);
        const uint32_t eq_rank = eq_seen + __builtin_amdgcn_mbcnt_hi((uint32_t)(eqm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eqm, 0u));
        const bool sel = k[r] < pivot || (k[r] == pivot && eq_rank < need);
        const uint64_t m = __ballot(sel);
        if (sel) emit(out + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)), r, k[r]);
        out += (uint32_t)__popcll(m);
        eq_seen += (uint32_t)__popcll(eqm);
    }
}

constexpr int PW_K_DIRECT = 2048;   // up to here the whole row of distances goes into registers
constexpr int PW_NB_MAX = 1024;     // up to here the block minima do (and P <= nb, P <= PW_P_MAX)
constexpr int PW_P_MAX = 64;
constexpr int PW_CAP = 512;         // survivors held in LDS; where there are more, the bound is taken from these and lowered

// Four queries a workgroup.  Same three steps and the same result as probe_select_kernel.  KMAX > 0: the whole row, of
// at most KMAX distances, goes into registers (and LDS, from where a short loop writes the selected ones out).  A small
// batch waits for one wavefront's chain of steps, which grows with the registers it holds: 100 queries x 1024 19 us with
// KMAX = 2048, 13 with 1024 (9.1 with all loads ahead of their use, 8.4 with the words that are written out read four at a time; 333 x 2000
// 15.2 and 13.9).
template <int KMAX>
__global__ __launch_bounds__(256) void probe_select_wave_kernel(const float *__restrict__ Dt, int64_t ldt, const float *__restrict__ bm,
                                                                int64_t K, int nb, int P, int64_t nq, int32_t *__restrict__ probe_id,
                                                                float *__restrict__ probe_d)
{
    constexpr bool DIRECT = KMAX > 0;
    constexpr int R = DIRECT ? KMAX / WAVE : PW_NB_MAX / WAVE;
    __shared__ uint32_t row_all[DIRECT ? 4 : 1][DIRECT ? KMAX : 1];
    __shared__ int blist_all[DIRECT ? 1 : 4][DIRECT ? 1 : 2 * PW_P_MAX];
    __shared__ uint32_t sk_all[DIRECT ? 1 : 4][DIRECT ? 1 : PW_CAP];
    __shared__ int si_all[DIRECT ? 1 : 4][DIRECT ? 1 : PW_CAP];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= nq) return;                                       // (whole wavefronts; no barrier follows)
    const float *row = Dt + q * ldt;
    int32_t *oid = probe_id + q * P;
    float *od = probe_d + q * P;
    uint32_t k[R], pivot, need;
    const int n = DIRECT ? (int)K : nb;
    const float *src = DIRECT ? row : bm + q * nb;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * WAVE + lane;
        const uint32_t key = float_key(src[i < n ? i : n - 1]);   // (every lane loads: all are on their way together)
        k[r] = i < n ? key : 0xFFFFFFFFu;
    }
    if (DIRECT) {
        uint32_t *held = row_all[DIRECT ? wave : 0];
#pragma unroll
        for (int r = 0; r < R; ++r) held[DIRECT ? r * WAVE + lane : 0] = k[r];
        wave_select<R>(k, (uint32_t)P, pivot, need);
        wave_sync();
        uint32_t out = 0, eq_seen = 0;
        // (four words on their way at a time; behind the row, none)
        static_assert(!DIRECT || KMAX % (4 * WAVE) == 0, "whole steps");
#pragma nounroll
        for (int c4 = 0; c4 < n; c4 += 4 * WAVE) {
            uint32_t word[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) word[u] = held[DIRECT ? c4 + u * WAVE + lane : 0];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t key = word[u];
                const int c = c4 + u * WAVE + lane;
                const uint64_t eqm = __ballot(key == pivot && need > 0 && c < n);
                const uint32_t eq_rank = eq_seen + __builtin_amdgcn_mbcnt_hi((uint32_t)(eqm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eqm, 0u));
                const bool sel = key < pivot || (key == pivot && eq_rank < need && c < n);
                const uint64_t m = __ballot(sel);
                if (sel) {
                    const uint32_t o = out + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    oid[o] = c;
                    od[o] = key_float(key);
                }
                out += (uint32_t)__popcll(m);
                eq_seen += (uint32_t)__popcll(eqm);
            }
        }
        return;
    }
    wave_select<R>(k, (uint32_t)P, pivot, need);
    // blocks that may hold one of the P closest: minimum below pivot, or (first P of them) equal to it; with need == 0
    // the P-th smallest minimum itself lies below pivot, and so do the P closest distances
    int *blist = blist_all[wave];
    uint32_t *sk = sk_all[wave];
    int *si = si_all[wave];
    uint32_t nflag = 0;
    wave_emit<R>(k, pivot, need > 0 ? (uint32_t)P : 0u, [&](uint32_t pos, int r, uint32_t) { blist[pos] = r * WAVE + lane; });
#pragma unroll
    for (int r = 0; r < R; ++r) nflag += (uint32_t)__popcll(__ballot(k[r] < pivot));
    if (need > 0) {
        uint32_t eq = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) eq += (uint32_t)__popcll(__ballot(k[r] == pivot));
        nflag += eq < (uint32_t)P ? eq : (uint32_t)P;
    }
    wave_sync();
    uint32_t lim = need > 0 ? pivot : pivot - 1u;              // the P closest have keys of at most lim
    auto fetch = [&](uint32_t f0, uint32_t (&kv)[16]) {        // the lane's column of 16 flagged blocks
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int64_t c = (int64_t)blist[f0 + j < nflag ? f0 + j : 0] * BMW + lane;
            const uint32_t key = float_key(row[c < K ? c : K - 1]);   // (every lane loads: all 16 are on their way together)
            kv[j] = f0 + j < nflag && c < K ? key : 0xFFFFFFFFu;
        }
    };
    // the survivors, in order, up to PW_CAP of them; AGAIN: of those equal to lim only the first P, which alone can be among
    // the P closest
    auto collect = [&](auto again) {
        uint32_t total = 0, eq_seen = 0;
        for (uint32_t f0 = 0; f0 < nflag; f0 += 16) {
            uint32_t kv[16];
            fetch(f0, kv);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                bool sel = kv[j] <= lim && kv[j] != 0xFFFFFFFFu;
                if constexpr (decltype(again)::value) {
                    const uint64_t eqm = __ballot(sel && kv[j] == lim);
                    if (kv[j] == lim) sel = sel && eq_seen + __builtin_amdgcn_mbcnt_hi((uint32_t)(eqm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eqm, 0u)) < (uint32_t)P;
                    eq_seen += (uint32_t)__popcll(eqm);
                }
                const uint64_t m = __ballot(sel);
                const uint32_t o = total + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (sel && o < (uint32_t)PW_CAP) {
                    sk[o] = kv[j];
                    si[o] = blist[f0 + j] * BMW + lane;
                }
                total += (uint32_t)__popcll(m);
            }
        }
        wave_sync();
        return total;
    };
    uint32_t s[PW_CAP / WAVE];
    auto select_kept = [&](uint32_t total) {
#pragma unroll
        for (int r = 0; r < PW_CAP / WAVE; ++r) s[r] = r * WAVE + lane < (int)total ? sk[r * WAVE + lane] : 0xFFFFFFFFu;
        wave_select<PW_CAP / WAVE>(s, (uint32_t)P, pivot, need);
    };
    uint32_t total = collect(std::false_type());
    if (total > (uint32_t)PW_CAP) {
        // The P closest of any PW_CAP distances bound the P closest of all: first of the 512 smallest, one of each lane's column
        // of every eighth block, which are near ones wherever those lie (of the first survivors in order, centroids whose
        // numbers follow their places took six rounds, 0.2 ms); should that not be enough, of those kept.  At most P of
        // these equal lim then, the others lie below it, and at least PW_CAP - P distances fall above the new bound every time.
#pragma unroll
        for (int r = 0; r < PW_CAP / WAVE; ++r) s[r] = 0xFFFFFFFFu;
        for (uint32_t f0 = 0; f0 < nflag; f0 += 16) {
            uint32_t kv[16];
            fetch(f0, kv);
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j % (PW_CAP / WAVE)] = kv[j] < s[j % (PW_CAP / WAVE)] ? kv[j] : s[j % (PW_CAP / WAVE)];
        }
        wave_select<PW_CAP / WAVE>(s, (uint32_t)P, pivot, need);
        while (true) {
            const uint32_t lower = need > 0 ? pivot : pivot - 1u;
            lim = lower < lim ? lower : lim;
            wave_sync();                                       // the kept ones have been read
            total = collect(std::true_type());
            if (total <= (uint32_t)PW_CAP) break;
            select_kept(total);
        }
    }
    select_kept(total);
    wave_emit<PW_CAP / WAVE>(s, pivot, need, [&](uint32_t pos, int r, uint32_t key) {
        oid[pos] = si[r * WAVE + lane];
        od[pos] = key_float(key);
    });
}

}  // namespace ivf
