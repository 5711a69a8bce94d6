// Candidate budget (Section 4 evaluates candidate lists of a given length R): of the subregions
// that survived the pruning, only a prefix in ascending order of (Eq. (7) distance, subregion id)
// is scanned, up to and including the subregion with which the points collected reach R.
#pragma once
#include "query.hpp"

namespace ivf {

// One workgroup per query, after score_prune_kernel has written the query's S <= N * BUDGET_BLOCK descriptors (in
// ascending subregion id).  A subregion is visited iff the subregions before it in (score,
// id) order hold fewer than R points together.  Scores (as order-preserving keys) and lengths are read once, into registers.  The score
// of the crossing subregion is found as block_select_runs finds the n-th smallest key, with bins that weigh the
// points of their subregions; among subregions that tie with it the order is position order (= id
// order), resolved by ordered scans where there are several.  The length of every subregion that is not visited is
// set to 0 (the scan skips empty descriptors), visited[q][i] (may be NULL) receives the flags and
// n_scanned[q] (may be NULL) the number of points of the visited subregions.
// Bound by the steps of one workgroup, two of them a compute unit: 2000 queries, S = 8192 103 us (a radix search by bytes of the
// descriptors in memory 246: most additions of its first passes went to the same few words).
constexpr int BUDGET_BLOCK = 1024;

template <int N>
__global__ __launch_bounds__(BUDGET_BLOCK) __attribute__((amdgpu_waves_per_eu(N <= 8 ? 8 : 4, 8))) void budget_cut_kernel(SubDesc *__restrict__ desc, int S, uint32_t R,
                                                                  uint8_t *__restrict__ visited, int64_t *__restrict__ n_scanned)
{
    constexpr int BLOCK = BUDGET_BLOCK, BITS = 10, NW = BLOCK / WAVE;
    static_assert(BLOCK == 1 << BITS, "a bin a thread");
    __shared__ uint32_t hist[BLOCK + WAVE];                       // ... and a word a lane for what is out of the range
    __shared__ uint32_t scan_s[NW], lo_s[NW], hi_s[NW], pick[4];
    __shared__ unsigned long long total_s;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int64_t q = blockIdx.x;
    SubDesc *d = desc + q * S;
    unsigned char *bytes = reinterpret_cast<unsigned char *>(d), *flags = visited ? visited + q * S : nullptr;   // (at 32-bit offsets: fewer registers)
    static_assert(sizeof(SubDesc) == 16 && offsetof(SubDesc, len) == 8 && offsetof(SubDesc, base) == 12, "length and score side by side");
    uint32_t key[N], len[N], sum = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {                                 // (every thread loads: all are on their way together)
        const uint32_t i = tid + u * BLOCK, at = i < (uint32_t)S ? i : S - 1;
        const uint2 w = *reinterpret_cast<const uint2 *>(bytes + (at * 16u + 8u));
        len[u] = i < (uint32_t)S ? w.x : 0u;
        sum += len[u];
        key[u] = float_key(__uint_as_float(w.y));
    }
    uint32_t lo = 0xFFFFFFFFu, hi = 0, all_points;
#pragma unroll
    for (int u = 0; u < N; ++u) {                                 // (an empty subregion has no weight, wherever its score lies)
        lo = key[u] < lo ? key[u] : lo;
        hi = key[u] > hi ? key[u] : hi;
    }
    lo = wave_extreme<false>(lo);
    hi = wave_extreme<true>(hi);
    if (lane == 0) {
        lo_s[wave] = lo;
        hi_s[wave] = hi;
    }
    if (tid == 0) {
        total_s = 0;
        pick[2] = 0;
    }
    hist[tid] = 0;
    block_exclusive_scan<BLOCK>(sum, scan_s, all_points);          // (barriers: what was written above is there)
    lo = wave_extreme<false>(lo_s[lane < NW ? lane : 0]);
    hi = wave_extreme<true>(hi_s[lane < NW ? lane : 0]);
    auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    const bool all = uniform(all_points) < R;                     // visit everything
    uint32_t remaining = R, place = 0;
    // the value in [low, high] with which the points of smaller and equal values reach `remaining`, which becomes the points still
    // wanted from the subregions with that value
    auto crossing = [&](auto value, uint32_t low, uint32_t high) {
        uint32_t range = high - low;
        int shift = range >= (uint32_t)BLOCK ? 32 - BITS - __builtin_clz(range) : 0;
#pragma nounroll
        while (true) {
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const uint32_t v = value(u) - low;
                atomicAdd(&hist[v <= range ? v >> shift : (uint32_t)(BLOCK + lane)], len[u]);
                if (N > 8 && u % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (fewer registers)
            }
            __syncthreads();
            const uint32_t c = hist[tid];
            hist[tid] = 0;
            uint32_t tot;
            const uint32_t cum = block_exclusive_scan<BLOCK>(c, scan_s, tot);
            if (cum < remaining && cum + c >= remaining) {        // exactly one thread
                pick[0] = (uint32_t)tid;
                pick[1] = remaining - cum;
            }
            __syncthreads();
            low += uniform(pick[0]) << shift;
            remaining = uniform(pick[1]);
            range = (1u << shift) - 1u;
            if (shift == 0) return low;
            shift = shift > BITS ? shift - BITS : 0;
        }
    };
    if (!all) {
        lo = crossing([&](int u) { return key[u]; }, lo, hi);
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (key[u] == lo && len[u]) {
                atomicAdd(&pick[2], 1u);
                pick[3] = (uint32_t)(tid + u * BLOCK);            // (its place, where there is one)
            }
        __syncthreads();
        place = uniform(pick[3]);
        if (uniform(pick[2]) > 1) place = crossing([&](int u) { return key[u] == lo ? (uint32_t)(tid + u * BLOCK) : NO_KEY; }, 0u, (uint32_t)(N * BLOCK - 1));
    }
    unsigned long long mine = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const uint32_t i = tid + u * BLOCK;
        const bool vis = all || key[u] < lo || (key[u] == lo && i <= place);
        if (!vis && len[u]) *reinterpret_cast<uint32_t *>(bytes + (i * 16u + 8u)) = 0u;   // (past S: no points)
        if (vis) mine += len[u];
        if (flags && i < (uint32_t)S) flags[i] = vis ? 1 : 0;
        if (N > 8 && u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (n_scanned) {
        if (mine) atomicAdd(&total_s, mine);
        __syncthreads();
        if (tid == 0) n_scanned[q] = (int64_t)total_s;
    }
}

}  // namespace ivf
