// An order of the regions that puts regions with common neighbours side by side, so that whoever goes through regions with
// all their neighbours' rows finds most of the rows in an XCD's L2 (4 MB; 64 rows of 96 dimensions are 24 KB, and each row is
// a neighbour of 64 regions).  The places that regions have in the table say nothing about it.
// Two rounds of min-wise hashing over the neighbour lists: a region takes the smallest hash among itself and its neighbours, then
// the smallest of what its neighbours took.  Two regions take the same with the probability that the sets within two steps of
// them agree, and a group is of the size of such a set (a thousand regions for 64 neighbours); inside a group the first
// round's value puts those with a neighbour in common together.
// It pays where neighbourhoods are shared and costs nothing elsewhere.  10 000 queries, L = 64, D = 96, a search in us in the table's order /
// in this one: K = 262 144, P = 128, neighbours within groups of 1024 2780 / 2260; the nearest of data of 10 intrinsic dimensions 2757 / 2428, of
// 20 2766 / 2609, of 96 2733 / 2717; anywhere 2776 / 2797; K = 65 536, P = 64 1084 / 983, 1080 / 999, 1082 / 1044, 1090 / 1089, 1092 / 1092; the
// nearest of 2^20 means that are all equally far apart, P = 256 9606 / 9737.
#pragma once
#include "util.hpp"

namespace ivf {

constexpr int SHINGLE_BITS = 24;   // 16 of the group, 8 inside it: three passes of the radix sort

__device__ __forceinline__ uint32_t scatter_bits(uint32_t v) { return v * 0x9E3779B1u; }   // one to one; the upper bits depend on all

// 16 lanes a region.  FIRST: out[r] = the smallest hash of r and its neighbours; else the key to sort by, from the first round's
// in[], of the first `use` neighbours (bound by these gathers: K = 2^20, all 64 382 us, 16 of them 112, and the same times
// of what goes by the order).
template <bool FIRST>
__global__ __launch_bounds__(256) void shingle_kernel(const int32_t *__restrict__ nbr, int64_t K, int L, int use, const uint32_t *__restrict__ in,
                                                      uint32_t *__restrict__ out)
{
    const int64_t r = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
    const int c = threadIdx.x & 15;
    if (r >= K) return;
    const uint32_t own = FIRST ? scatter_bits((uint32_t)r) : in[r];
    uint32_t v = own;
    for (int l = c; l < use; l += 16) {
        const uint32_t s = (uint32_t)nbr[r * L + l], o = FIRST ? scatter_bits(s) : in[s];
        v = o < v ? o : v;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        const uint32_t w = (uint32_t)__shfl_xor((int)v, o, 16);
        v = w < v ? w : v;
    }
    // (the smallest of many hashes are small numbers: spread again before their upper bits are taken)
    if (c == 0) out[r] = FIRST ? v : (scatter_bits(v) >> 16) << 8 | scatter_bits(own) >> 24;
}

__global__ __launch_bounds__(256) void inverse_kernel(const uint32_t *__restrict__ order, int64_t n, uint32_t *__restrict__ inv)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) inv[order[i]] = (uint32_t)i;
}

}  // namespace ivf
