// Small device helpers shared by the kernels: order-preserving float keys,
// wavefront (64 lanes) and workgroup scans / reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ivf {

constexpr int WAVE = 64;
constexpr uint64_t EMPTY_KEY = ~0ull;

// fp32 -> uint32 such that a < b  <=>  key(a) < key(b) (for non-NaN values)
__device__ __forceinline__ uint32_t float_key(float f)
{
    uint32_t u = __float_as_uint(f);
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k)
{
    uint32_t u = k ^ ((k >> 31) ? 0x80000000u : 0xFFFFFFFFu);
    return __uint_as_float(u);
}

// LDS traffic between lanes of one wavefront: keep the compiler from moving
// LDS accesses across this point (the hardware executes a wave's LDS
// instructions in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// DPP move with 0 for lanes that have no source (shifted out of their row of 16,
// or in a row excluded by ROW_MASK).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive prefix sum over the 64 lanes in 6 DPP steps, no LDS: row_shr 1/2/4/8 scan each row
// of 16, row_bcast15 carries rows 0,2 into rows 1,3, row_bcast31 carries lane 31 into rows 2,3.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xf>(v);
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    return v;
}

// Sum and smallest value over the wave in 6 DPP steps each (see wave_inclusive_scan), no LDS: for values that
// only enter a bound, where the order of the additions does not matter.
__device__ __forceinline__ float wave_total(float v)
{
    v += __uint_as_float(dpp_or_zero<0x111, 0xf>(__float_as_uint(v)));
    v += __uint_as_float(dpp_or_zero<0x112, 0xf>(__float_as_uint(v)));
    v += __uint_as_float(dpp_or_zero<0x114, 0xf>(__float_as_uint(v)));
    v += __uint_as_float(dpp_or_zero<0x118, 0xf>(__float_as_uint(v)));
    v += __uint_as_float(dpp_or_zero<0x142, 0xa>(__float_as_uint(v)));
    v += __uint_as_float(dpp_or_zero<0x143, 0xc>(__float_as_uint(v)));
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), WAVE - 1));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_or_self(float v)
{
    const int u = (int)__float_as_uint(v);
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(u, u, CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float wave_smallest(float v)
{
    v = fminf(v, dpp_or_self<0x111, 0xf>(v));
    v = fminf(v, dpp_or_self<0x112, 0xf>(v));
    v = fminf(v, dpp_or_self<0x114, 0xf>(v));
    v = fminf(v, dpp_or_self<0x118, 0xf>(v));
    v = fminf(v, dpp_or_self<0x142, 0xa>(v));
    v = fminf(v, dpp_or_self<0x143, 0xc>(v));
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), WAVE - 1));
}

// Smallest and largest word over the wave, for every lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_word_or_self(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROW_MASK, 0xf, false);
}

template <bool LARGEST>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v)
{
    auto of = [](uint32_t a, uint32_t b) { return (LARGEST ? a > b : a < b) ? a : b; };
    v = of(v, dpp_word_or_self<0x111, 0xf>(v));
    v = of(v, dpp_word_or_self<0x112, 0xf>(v));
    v = of(v, dpp_word_or_self<0x114, 0xf>(v));
    v = of(v, dpp_word_or_self<0x118, 0xf>(v));
    v = of(v, dpp_word_or_self<0x142, 0xa>(v));
    v = of(v, dpp_word_or_self<0x143, 0xc>(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, WAVE - 1);
}

// Sum over the 16 lanes of a row, with the additions and the order of wave_sum's last four steps (lane ^ 8, ^ 4, ^ 2, ^ 1) but without LDS: after
// the first the values repeat every 8 lanes, so that a rotation by 4 brings lane ^ 4's.
__device__ __forceinline__ float sum_of_16(float v)
{
    v += dpp_or_self<0x128, 0xf>(v);                       // row_ror:8
    v += dpp_or_self<0x124, 0xf>(v);                       // row_ror:4
    v += dpp_or_self<0x4E, 0xf>(v);                        // quad_perm: lane ^ 2
    v += dpp_or_self<0xB1, 0xf>(v);                        // quad_perm: lane ^ 1
    return v;
}

// argmin over the wave of (value, index) pairs, lowest index on equal values;
// every lane receives the winner.
__device__ __forceinline__ void wave_argmin(float &v, int &idx)
{
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        float ov = __shfl_xor(v, o, WAVE);
        int oi = __shfl_xor(idx, o, WAVE);
        if (ov < v || (ov == v && oi < idx)) { v = ov; idx = oi; }
    }
}

__device__ __forceinline__ void wave_argmin(double &v, int &idx)
{
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        double ov = __shfl_xor(v, o, WAVE);
        int oi = __shfl_xor(idx, o, WAVE);
        if (ov < v || (ov == v && oi < idx)) { v = ov; idx = oi; }
    }
}

// Exclusive scan of one uint32 per thread over a workgroup of BLOCK threads
// (BLOCK a multiple of 64).  sh must hold BLOCK/64 words of LDS.  Returns the
// exclusive prefix; total receives the workgroup sum.  Contains barriers.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t &total)
{
    constexpr int NW = BLOCK / WAVE;
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    uint32_t inc = wave_inclusive_scan(v);
    if (lane == WAVE - 1) sh[w] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        uint32_t s = sh[i];
        if (i < w) before += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return before + inc - v;
}

}  // namespace ivf
