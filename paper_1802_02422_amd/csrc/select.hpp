// Exact selection of the nsel smallest of n items by (key, position) inside
// one workgroup: an MSB-first radix select on order-preserving uint32 keys
// followed by an ordered compaction, so the winners come out in ascending
// position and ties on the key resolve to the lowest positions.
#pragma once
#include "util.hpp"

namespace ivf {

struct SelectShared {
    uint32_t hist[4][256];   // one histogram per radix pass
    uint32_t scan[16];
    uint32_t pick[4][2];
};

// hist[bin] += 1 for the calling lanes.  Keys that share their leading bytes (distances of one
// query) put whole wavefronts into one bin of the first passes; 64 atomics on one LDS word are
// executed one after the other, so a wavefront whose lanes all agree adds its population count once.
__device__ __forceinline__ void hist_add(uint32_t *hist, uint32_t bin)
{
    const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    const uint64_t active = __ballot(true), same = __ballot(bin == b0);
    if (same == active) {
        if (__builtin_amdgcn_mbcnt_hi((uint32_t)(active >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)active, 0u)) == 0)
            atomicAdd(&hist[b0], (uint32_t)__popcll(active));
    } else {
        atomicAdd(&hist[bin], 1u);
    }
}

// Finds the key value `pivot` of the nsel-th smallest item and the number
// `need` of items equal to pivot that belong to the selection (those at the
// lowest positions).  key(i) must be pure.  1 <= nsel <= n.
template <int BLOCK, class KeyFn>
__device__ void block_radix_select(KeyFn key, int64_t n, uint32_t nsel, SelectShared &sh,
                                   uint32_t &pivot, uint32_t &need)
{
    const int tid = threadIdx.x;
    uint32_t prefix = 0, mask = 0, remaining = nsel;
    __syncthreads();                              // the previous user of sh is done
    for (int i = tid; i < 4 * 256; i += BLOCK) (&sh.hist[0][0])[i] = 0;
    __syncthreads();
    for (int pass = 0; pass < 4; ++pass) {        // two barriers per pass
        const int shift = 24 - 8 * pass;
        uint32_t *hist = sh.hist[pass];
        // several independent key reads in flight per thread before their histogram updates
        int64_t i = tid;
        for (; i + 3 * BLOCK < n; i += 4 * BLOCK) {
            uint32_t k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) k[u] = key(i + u * BLOCK);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if ((k[u] & mask) == prefix) hist_add(hist, (k[u] >> shift) & 255u);
        }
        for (; i < n; i += BLOCK) {
            uint32_t k = key(i);
            if ((k & mask) == prefix) hist_add(hist, (k >> shift) & 255u);
        }
        __syncthreads();
        if (tid < WAVE) {
            uint32_t c[4], s = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { c[j] = hist[4 * tid + j]; s += c[j]; }
            uint32_t inc = wave_inclusive_scan(s);
            uint32_t exc = inc - s;
            if (exc < remaining && inc >= remaining) {   // exactly one lane
                uint32_t cum = exc;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (cum < remaining && cum + c[j] >= remaining) {
                        sh.pick[pass][0] = 4 * tid + j;
                        sh.pick[pass][1] = remaining - cum;
                    }
                    cum += c[j];
                }
            }
        }
        __syncthreads();
        prefix |= sh.pick[pass][0] << shift;
        mask |= 0xFFu << shift;
        remaining = sh.pick[pass][1];
    }
    pivot = prefix;
    need = remaining;
}

// Calls emit(out_pos, i, key) for every item with key < pivot and for the
// `need` lowest-positioned items with key == pivot, where out_pos is the item's
// rank among the emitted ones in ascending i.  Stops early once nsel items
// have been emitted.  Returns the number emitted.
template <int BLOCK, class KeyFn, class EmitFn>
__device__ uint32_t block_emit_selected(KeyFn key, int64_t n, uint32_t nsel, uint32_t pivot,
                                        uint32_t need, SelectShared &sh, EmitFn emit)
{
    const int tid = threadIdx.x;
    uint32_t run_lt = 0, run_eq = 0;
    for (int64_t base = 0; base < n; base += BLOCK) {
        int64_t i = base + tid;
        bool valid = i < n;
        uint32_t k = valid ? key(i) : 0u;
        bool lt = valid && k < pivot, eq = valid && k == pivot;
        uint32_t packed = (lt ? 1u : 0u) | (eq ? 0x10000u : 0u), total;
        uint32_t exc = block_exclusive_scan<BLOCK>(packed, sh.scan, total);
        uint32_t lt_ex = exc & 0xFFFFu, eq_ex = run_eq + (exc >> 16);
        if (lt) {
            emit(run_lt + lt_ex + (eq_ex < need ? eq_ex : need), i, k);
        } else if (eq && eq_ex < need) {
            emit(run_lt + lt_ex + eq_ex, i, k);
        }
        run_lt += total & 0xFFFFu;
        run_eq += total >> 16;
        if (run_lt + (run_eq < need ? run_eq : need) >= nsel) break;   // uniform
    }
    return run_lt + (run_eq < need ? run_eq : need);
}

// ---- The same selection with the keys in registers ----
// Thread t holds items [t ipt, (t + 1) ipt) of n in k[0 .. N-1], ipt = run_length(n) <= N; NO_KEY where there is none.
// Bins of equal width between the smallest and the largest key spread the keys that one byte of them would put into one or
// two bins, so that one pass over the registers, without a branch, leaves a few around the nsel-th for one wavefront to decide:
// seven barriers, where block_radix_select has ten and reads the keys four times, most of its additions to the same few
// words.
constexpr uint32_t NO_KEY = 0xFFFFFFFFu;         // (the key of no number; a NaN of that pattern becomes the next one)

template <int NB>                                // bins: 4 a thread at most
struct SelectRegs {
    uint32_t hist[NB + WAVE];                    // ... and a word a lane for what is no key
    uint32_t lo[16], hi[16], sum[16], scan[16];
    uint32_t pick[3];                            // bin, rank inside it, items in it; then pivot and need
    uint32_t list[WAVE], n_list;
};

template <int BLOCK>
__device__ __forceinline__ int run_length(int n) { return ((n + BLOCK - 1) / BLOCK + 3) & ~3; }

// k[0 .. N-1] from an array that is 16-byte aligned and readable up to the next multiple of four past n (ALIGNED = false: from any);
// as_key turns a word into its key
template <int BLOCK, bool ALIGNED = true, int N, class KeyFn>
__device__ __forceinline__ void load_run(const uint32_t *words, int n, uint32_t (&k)[N], KeyFn as_key)
{
    const int ipt = run_length<BLOCK>(n), i0 = threadIdx.x * ipt;
    // (every thread loads, from the last items where it has none: a load in a branch is waited for before the next one)
    uint32_t w[N];
#pragma unroll
    for (int v = 0; v < N; v += 4) {
        if (v >= ipt) break;                                      // (uniform)
        if (ALIGNED) {
            const int i = i0 + v < n ? i0 + v : (n - 1) & ~3;
            const uint4 u = *reinterpret_cast<const uint4 *>(&words[i]);
            w[v] = u.x; w[v + 1] = u.y; w[v + 2] = u.z; w[v + 3] = u.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) w[v + j] = words[i0 + v + j < n ? i0 + v + j : n - 1];
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (j < ipt) {
            const uint32_t key = as_key(w[j]);
            k[j] = i0 + j < n ? (key < NO_KEY ? key : NO_KEY - 1u) : NO_KEY;
        } else {
            k[j] = NO_KEY;
        }
    }
}

// pivot and need as in block_radix_select; used: all keys lie in k[0 .. used-1] (uniform); 1 <= nsel <= number of keys
template <int BLOCK, int NB, int N>
__device__ __forceinline__ void block_select_runs(const uint32_t (&k)[N], int used, uint32_t nsel, SelectRegs<NB> &sh, uint32_t &pivot, uint32_t &need)
{
    constexpr int NW = BLOCK / WAVE, PER = NB / BLOCK, BITS = NB == 1024 ? 10 : NB == 2048 ? 11 : 12;   // bins of a thread in the search
    static_assert(NB == 1 << BITS && PER >= 1 && PER * BLOCK == NB, "whole bins a thread");
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    uint32_t lo = NO_KEY, hi = 0;                                 // (hi: one more than the largest key)
#pragma unroll
    for (int v = 0; v < N; v += 4)
        if (v < used) {
#pragma unroll
            for (int j = v; j < v + 4 && j < N; ++j) {
                lo = k[j] < lo ? k[j] : lo;
                hi = k[j] + 1u > hi ? k[j] + 1u : hi;
            }
        }
    lo = wave_extreme<false>(lo);
    hi = wave_extreme<true>(hi);
#pragma unroll
    for (int i = 0; i < PER; ++i) sh.hist[tid + i * BLOCK] = 0;
    if (lane == 0) {
        sh.lo[wave] = lo;
        sh.hi[wave] = hi;
    }
    if (tid == 0) sh.n_list = 0;
    __syncthreads();
    {
        const int at = lane < NW ? lane : 0;
        lo = wave_extreme<false>(sh.lo[at]);
        hi = wave_extreme<true>(sh.hi[at]);
    }
    uint32_t range = hi - 1u - lo, remaining = nsel, cnt;
    int shift = range >= (uint32_t)NB ? 32 - BITS - __builtin_clz(range) : 0;   // (uniform, like all that follows)
#pragma unroll
    for (int v = 0; v < N; v += 4)
        if (v < used) {
#pragma unroll
            for (int j = v; j < v + 4 && j < N; ++j) atomicAdd(&sh.hist[k[j] != NO_KEY ? (k[j] - lo) >> shift : (uint32_t)(NB + lane)], 1u);
        }
    while (true) {
        __syncthreads();
        uint32_t c[PER], s = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            c[j] = sh.hist[tid * PER + j];
            s += c[j];
        }
        const uint32_t inc = wave_inclusive_scan(s);
        if (lane == WAVE - 1) sh.sum[wave] = inc;
        __syncthreads();
        // sums of the wavefronts before this one
        const uint32_t sums = wave_inclusive_scan(lane < NW ? sh.sum[lane < NW ? lane : 0] : 0u);
        uint32_t cum = inc - s + (wave ? (uint32_t)__builtin_amdgcn_readlane((int)sums, wave ? wave - 1 : 0) : 0u);
        if (cum < remaining && cum + s >= remaining) {            // exactly one lane
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                if (cum < remaining && cum + c[j] >= remaining) {
                    sh.pick[0] = tid * PER + j;
                    sh.pick[1] = remaining - cum;
                    sh.pick[2] = c[j];
                }
                cum += c[j];
            }
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) sh.hist[tid * PER + j] = 0;
        __syncthreads();
        lo += sh.pick[0] << shift;
        remaining = sh.pick[1];
        cnt = sh.pick[2];
        range = (1u << shift) - 1u;
        if (shift == 0) {
            pivot = lo;
            need = remaining;
            return;
        }
        if (cnt <= (uint32_t)WAVE) break;
        shift = shift > BITS ? shift - BITS : 0;
#pragma unroll
        for (int j = 0; j < N; ++j)                               // (no key is not in the range: it is above every key)
            if (k[j] - lo <= range && k[j] != NO_KEY) atomicAdd(&sh.hist[(k[j] - lo) >> shift], 1u);
    }
#pragma unroll
    for (int v = 0; v < N; v += 4)
        if (v < used) {
#pragma unroll
            for (int j = v; j < v + 4 && j < N; ++j)
                if (k[j] - lo <= range && k[j] != NO_KEY) sh.list[atomicAdd(&sh.n_list, 1u)] = k[j] - lo;
        }
    __syncthreads();
    if (wave == 0) {
        const uint32_t mine = lane < (int)cnt ? sh.list[lane] : NO_KEY;
        uint32_t t = 0;
        for (int bit = shift - 1; bit >= 0; --bit) {
            const uint32_t trial = t | 1u << bit;
            if ((uint32_t)__popcll(__ballot(mine < trial)) < remaining) t = trial;
        }
        const uint32_t below = (uint32_t)__popcll(__ballot(mine < t));
        if (lane == 0) {
            sh.pick[0] = lo + t;
            sh.pick[1] = remaining - below;
        }
    }
    __syncthreads();
    pivot = sh.pick[0];
    need = sh.pick[1];
}

// emit(position among the selected, item, key) for the selected ones, in ascending order of the items; returns their number
template <int BLOCK, int N, class EmitFn>
__device__ __forceinline__ uint32_t block_emit_runs(const uint32_t (&k)[N], int ipt, uint32_t pivot, uint32_t need, uint32_t *scan, EmitFn emit)
{
    uint32_t lt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        lt += k[j] < pivot ? 1u : 0u;
        eq += k[j] == pivot ? 1u : 0u;
    }
    uint32_t total;
    const uint32_t exc = block_exclusive_scan<BLOCK>(lt | (eq << 16), scan, total);
    uint32_t lt_seen = exc & 0xFFFFu, eq_seen = exc >> 16;
    const int i0 = threadIdx.x * ipt;
    if (lt | eq) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if (k[j] < pivot) {
                emit(lt_seen + (eq_seen < need ? eq_seen : need), i0 + j, k[j]);
                ++lt_seen;
            } else if (k[j] == pivot) {
                if (eq_seen < need) emit(lt_seen + eq_seen, i0 + j, k[j]);
                ++eq_seen;
            }
        }
    }
    const uint32_t tl = total & 0xFFFFu, te = total >> 16;
    return tl + (te < need ? te : need);
}

// In-place ascending bitonic sort of n (a power of two) uint64 keys in LDS by
// the whole workgroup.
template <int BLOCK>
__device__ void block_bitonic_sort(uint64_t *a, int n)
{
    for (int size = 2; size <= n; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < n / 2; t += BLOCK) {
                int i = 2 * t - (t & (stride - 1)), j = i + stride;
                bool up = (i & size) == 0;
                uint64_t x = a[i], y = a[j];
                if ((x > y) == up) { a[i] = y; a[j] = x; }
            }
        }
    __syncthreads();
}

// The same for one wavefront on its private LDS array.
__device__ __forceinline__ void wave_bitonic_sort(uint64_t *a, int n)
{
    const int lane = threadIdx.x & (WAVE - 1);
    for (int size = 2; size <= n; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            wave_sync();
            for (int t = lane; t < n / 2; t += WAVE) {
                int i = 2 * t - (t & (stride - 1)), j = i + stride;
                bool up = (i & size) == 0;
                uint64_t x = a[i], y = a[j];
                if ((x > y) == up) { a[i] = y; a[j] = x; }
            }
        }
    wave_sync();
}

}  // namespace ivf
