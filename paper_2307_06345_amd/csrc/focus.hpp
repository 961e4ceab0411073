// The minimum-distance MAC of octree nodes against a focus range F of the curve
// (Sec. 7.1), for device code.
#pragma once

#include "common.hpp"
#include "hilbert.hpp"

namespace cs {

// F = [fa, fb), the curve and theta^2.
struct FocusSpec {
    uint64_t fa, fb;
    int curve;
    double theta2;
};

constexpr uint32_t kMaxFocusBlocks = 320;  // 2 x 7 x 21 = 294 at most

// F cut into its maximal aligned key blocks, each as its grid box {corner x, y,
// z, edge}, and the table that decodes Hilbert keys; in LDS.
struct FocusSmem {
    uint4 blocks[kMaxFocusBlocks];
    uint16_t dec[kStates * 8];
    uint32_t count;
    uint32_t lo[3], hi[3];  // around all of them
};

// Fills sm, all threads of the block (which then needs a barrier, as it does
// before). With a_e (b_e) the range's start rounded up (end rounded down) to a
// multiple of 8^e, and E the largest e with a_e < b_e, the blocks are those of
// span 8^e between a_e and a_{e + 1} and between b_{e + 1} and b_e for e < E,
// and those of span 8^E between a_E and b_E: slot d of (side, e) is the d-th,
// so every block is found by its own thread (a copy from the host took longer
// than the launches it preceded); then the blocks found, a few dozen, are taken
// by the first threads together for the 21 dependent steps to their corners.
__device__ __forceinline__ void focus_fill(const FocusSpec& f, FocusSmem& sm) {
    for (uint32_t e = threadIdx.x; e < kStates * 8; e += blockDim.x) sm.dec[e] = kHilbertDecode.dec[e];
    if (threadIdx.x == 0) sm.count = 0;
    if (threadIdx.x < 3) {
        sm.lo[threadIdx.x] = 1u << kL;
        sm.hi[threadIdx.x] = 0;
    }
    __syncthreads();
    auto up = [&](int e) { return (f.fa + ((1ull << (3 * e)) - 1)) >> (3 * e) << (3 * e); };
    auto down = [&](int e) { return f.fb >> (3 * e) << (3 * e); };
    int top = -1;
    for (int e = 0; e <= kL; ++e)
        if (up(e) < down(e)) top = e;
    for (uint32_t t = threadIdx.x; t < 16u * (kL + 1) * 2u; t += blockDim.x) {
        const int e = static_cast<int>(t >> 5);
        const uint32_t d = t & 15u;
        const bool right = (t >> 4) & 1u;
        if (e > top || (e == top && right)) continue;
        const uint64_t from = right ? down(e + 1) : up(e);
        const uint64_t to = right ? down(e) : (e == top ? down(e) : up(e + 1));
        if (from >= to || d >= (to - from) >> (3 * e)) continue;  // (from + d 8^e alone could pass 2^64)
        const uint64_t k = from + (static_cast<uint64_t>(d) << (3 * e));
        const uint32_t at = atomicAdd(&sm.count, 1u);
        if (at < kMaxFocusBlocks)
            sm.blocks[at] = make_uint4(static_cast<uint32_t>(k), static_cast<uint32_t>(k >> 32), static_cast<uint32_t>(e), 0);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < min(sm.count, kMaxFocusBlocks); b += blockDim.x) {
        const uint4 v = sm.blocks[b];
        uint32_t c[3];
        node_corner((static_cast<uint64_t>(v.y) << 32) | v.x, kL - static_cast<int>(v.z), f.curve, sm.dec, c);
        const uint32_t edge = 1u << v.z;
        sm.blocks[b] = make_uint4(c[0], c[1], c[2], edge);
        for (int d = 0; d < 3; ++d) {
            atomicMin(&sm.lo[d], c[d]);
            atomicMax(&sm.hi[d], c[d] + edge);
        }
    }
}

// Squared distance of two grid boxes, exact: gaps are below 2^22, so the sum of
// their squares is below 2^53.
__device__ __forceinline__ double box_distance2(const uint32_t c[3], uint32_t edge, const uint32_t lo[3], const uint32_t hi[3]) {
    double r2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int a0 = static_cast<int>(c[d]), a1 = static_cast<int>(c[d] + edge);
        const int b0 = static_cast<int>(lo[d]), b1 = static_cast<int>(hi[d]);
        const double gap = static_cast<double>(max(max(b0 - a1, a0 - b1), 0));
        r2 = fma(gap, gap, r2);
    }
    return r2;
}

// MAC of the node (corner, edge): fails iff some block lies within l / theta,
// tested as r^2 theta^2 <= l^2 with one rounding in the product. It passes for
// all blocks if it does for the box around them, which settles most far nodes.
// (4 M Plummer particles, N_crit 32, one of 64 ranges: the launch that tests a
// node or two per 50 particles took 77 us with 64-bit integers and without that
// box, 45 with both.)
__device__ __forceinline__ bool mac_fails_dev(const uint32_t c[3], uint32_t edge, const FocusSmem& sm, double theta2) {
    const uint32_t nblocks = min(sm.count, kMaxFocusBlocks);
    if (nblocks == 0) return false;
    const double l2 = static_cast<double>(edge) * static_cast<double>(edge);
    if (box_distance2(c, edge, sm.lo, sm.hi) * theta2 > l2) return false;
    for (uint32_t b = 0; b < nblocks; ++b) {
        const uint4 f = sm.blocks[b];
        const uint32_t lo[3] = {f.x, f.y, f.z}, hi[3] = {f.x + f.w, f.y + f.w, f.z + f.w};
        if (!(box_distance2(c, edge, lo, hi) * theta2 > l2)) return true;
    }
    return false;
}

// The same for the node of `level` that holds (or starts at) a key.
__device__ __forceinline__ bool node_fails(uint64_t key, uint32_t level, const FocusSpec& f, const FocusSmem& sm) {
    uint32_t c[3];
    node_corner(key, static_cast<int>(level), f.curve, sm.dec, c);
    return mac_fails_dev(c, 1u << (kL - level), sm, f.theta2);
}

}  // namespace cs
