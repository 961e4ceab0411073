// Node properties of the linked octree and particles in curve order.
//
// Node counts (Sec. 5: properties of all n nodes in separate arrays, here the
// particle count an upward pass gives every node). The count of a node is the
// sum of its leaves' counts, and a node's leaves are a contiguous run of K:
// with S the exclusive prefix sum of the leaf counts, a node covering the key
// range [a, b) holds S[lb(K, b)] - S[lb(K, a)] particles. So one scan of the
// leaf counts and one pass over the nodes (two searches of K each, adjacent
// threads searching adjacent keys, so their paths share cache lines) replace
// the level-by-level pass, with the same exact integers.
//
// Gather (Sec. 4, the permutation that sorts the keys applied to the particle
// arrays): dst[i] = src[perm[i]]. The writes and the reads of perm stream; the
// source reads follow the curve, scattered for unsorted input. One array per
// pass keeps the array being gathered (8 B per particle) resident in the
// 256 MB last-level cache for inputs up to 2^25 particles. Every scattered read
// of 8 B moves a whole line all the same, so with room for 24 B per particle the
// three coordinates are first put side by side and read together (see
// gather_packed_kernel).
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace cs {
namespace {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr uint32_t kScanTile = kScanBlock * kScanItems;
constexpr int kNodeBlock = 256;
constexpr int kGatherBlock = 256;
constexpr int kGatherItems = 8;

// Exclusive prefix sum in two launches: the tiles' sums, then every tile its
// part, after the sums of the tiles before it, which its block adds up itself
// (one read per 256 tiles, all in flight). Above kSumTiles tiles a launch between
// the two scans the sums. Tiles wait for nobody: a decoupled look-back, at 33 ns
// per tile of polling across the XCDs, took 20 us for 1.1 M counts, now 13.
constexpr uint32_t kSumTiles = 2048;

__device__ __forceinline__ uint32_t scan_tile_load(const uint32_t* __restrict__ counts, uint32_t n, uint64_t base,
                                                   uint32_t v[kScanItems]) {
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {  // blocked: each thread a run of items
        v[i] = base + i < n ? counts[base + i] : 0u;
        mine += v[i];
    }
    return mine;
}

__global__ __launch_bounds__(kScanBlock) void scan_sums_kernel(const uint32_t* __restrict__ counts, uint32_t n,
                                                               uint32_t* __restrict__ sums) {
    __shared__ uint32_t tmp[kScanBlock / kWave];
    uint32_t v[kScanItems], total;
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
    (void)block_exclusive_sum<uint32_t, kScanBlock>(scan_tile_load(counts, n, base, v), tmp, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// sums: the tiles' sums, or scanned, the sums of all tiles before each.
__global__ __launch_bounds__(kScanBlock) void exclusive_scan_kernel(const uint32_t* __restrict__ counts, uint32_t n,
                                                                    const uint32_t* __restrict__ sums, bool scanned,
                                                                    uint32_t* __restrict__ S) {
    __shared__ uint32_t tmp[kScanBlock / kWave];
    uint32_t v[kScanItems], total, prefix = 0;
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
    if (scanned) {
        prefix = sums[blockIdx.x];
    } else {
        uint32_t before = 0;
#pragma unroll
        for (uint32_t k = 0; k < kSumTiles / kScanBlock; ++k) {
            const uint32_t t = k * kScanBlock + threadIdx.x;
            before += t < blockIdx.x ? sums[t] : 0u;
        }
        (void)block_exclusive_sum<uint32_t, kScanBlock>(before, tmp, &prefix);
    }
    uint32_t run = prefix + block_exclusive_sum<uint32_t, kScanBlock>(scan_tile_load(counts, n, base, v), tmp, &total);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i <= n) S[base + i] = run;  // the entry at n is the total
        run += v[i];
    }
}

// Particle count of every node: the leaf run of its key range, by two
// searches of K. A node that does not start at a leaf boundary (node keys of
// another tree) gets 0xffffffff.
__global__ __launch_bounds__(kNodeBlock) void node_counts_tree_kernel(const uint64_t* __restrict__ K, uint32_t nl,
                                                                      const uint32_t* __restrict__ S,
                                                                      const uint64_t* __restrict__ NK, uint32_t n,
                                                                      uint32_t* __restrict__ out) {
    const uint32_t p = blockIdx.x * kNodeBlock + threadIdx.x;
    if (p >= n) return;
    const uint64_t key = NK[p];
    const int level = (63 - clz64(key)) / 3;  // the placeholder bit sits at 3 * level
    const int shift = 3 * (kL - level);
    const uint64_t start = (key ^ (1ull << (3 * level))) << shift;
    const uint64_t end = start + (1ull << shift);
    const uint32_t i0 = static_cast<uint32_t>(lower_bound_u64(K, 0, nl, start));
    if (i0 >= nl || K[i0] != start) {  // never for a node of this tree: it starts at a leaf boundary
        out[p] = 0xffffffffu;
        return;
    }
    // the run's end: the next leaf (a leaf node), else a galloping search forward
    uint32_t i1 = i0 + 1;
    if (K[i1] < end) {
        uint32_t step = 1, lo = i1;
        while (true) {
            const uint32_t probe = static_cast<uint32_t>(std::min<uint64_t>(static_cast<uint64_t>(lo) + step, nl));
            if (K[probe] >= end) {
                i1 = static_cast<uint32_t>(lower_bound_u64(K, lo + 1, probe, end));
                break;
            }
            lo = probe;
            step <<= 1;
        }
    }
    out[p] = S[i1] - S[i0];
}

template <int ARRAYS>
__global__ __launch_bounds__(kGatherBlock) void gather_kernel(const double* __restrict__ a0,
                                                              const double* __restrict__ a1,
                                                              const double* __restrict__ a2,
                                                              const uint32_t* __restrict__ perm, uint32_t n,
                                                              double* __restrict__ o0, double* __restrict__ o1,
                                                              double* __restrict__ o2) {
    const size_t base = static_cast<size_t>(blockIdx.x) * (kGatherBlock * kGatherItems) + threadIdx.x;
    uint32_t src[kGatherItems];
#pragma unroll
    for (int i = 0; i < kGatherItems; ++i) {
        const size_t j = base + i * kGatherBlock;
        src[i] = j < n ? perm[j] : 0u;
    }
    double v[kGatherItems];
#pragma unroll
    for (int i = 0; i < kGatherItems; ++i) v[i] = base + i * kGatherBlock < n ? a0[src[i]] : 0.0;
#pragma unroll
    for (int i = 0; i < kGatherItems; ++i)
        if (base + i * kGatherBlock < n) o0[base + i * kGatherBlock] = v[i];
    if constexpr (ARRAYS > 1) {
#pragma unroll
        for (int i = 0; i < kGatherItems; ++i) v[i] = base + i * kGatherBlock < n ? a1[src[i]] : 0.0;
#pragma unroll
        for (int i = 0; i < kGatherItems; ++i)
            if (base + i * kGatherBlock < n) o1[base + i * kGatherBlock] = v[i];
    }
    if constexpr (ARRAYS > 2) {
#pragma unroll
        for (int i = 0; i < kGatherItems; ++i) v[i] = base + i * kGatherBlock < n ? a2[src[i]] : 0.0;
#pragma unroll
        for (int i = 0; i < kGatherItems; ++i)
            if (base + i * kGatherBlock < n) o2[base + i * kGatherBlock] = v[i];
    }
}

constexpr int kPackBlock = 256;
constexpr uint32_t kPackTile = 1024;  // particles a block packs at a time
constexpr uint32_t kPackNear = 1u << 15;

// Whether perm scatters: more than two fifths of 64 pairs of neighbours spread over
// it lie kPackNear (256 KB of an array, which L2 holds many times) or more apart.
// Random input has nearly all of them apart, input in the order of an earlier step
// next to none. The same for every wave. In between, 2^24 particles by the arrays /
// by records, us, with the share of pairs apart: places off by up to 8000 (0.00) 367
// / 435, 16,000 (0.00) 486 / 469, 65,000 (0.24) 508 / 474, 130,000 (0.55) 517 / 480; a
// tenth of them anywhere (0.19) 254 / 342, a fifth (0.36) 342 / 363, 0.3 (0.51) 431 /
// 394, half (0.75) 608 / 458.
__device__ __forceinline__ bool perm_scatters(const uint32_t* __restrict__ perm, uint32_t n) {
    const uint32_t i = lane_id() * (n / kWave);  // i + 1 < n
    const uint32_t a = perm[i], b = perm[i + 1];
    return __popcll(__ballot((a > b ? a - b : b - a) >= kPackNear)) * 5 > kWave * 2;
}

// rec[i] = {x[i], y[i], z[i]}, through LDS so that both sides are whole lines,
// if perm scatters; *packed says so. Bound: 48 B a particle (2^24: 145 us, 5.5 TB/s).
__global__ __launch_bounds__(kPackBlock) void gather_pack_kernel(const double* __restrict__ x, const double* __restrict__ y,
                                                                 const double* __restrict__ z,
                                                                 const uint32_t* __restrict__ perm, uint32_t n,
                                                                 double* __restrict__ rec, uint32_t* packed) {
    __shared__ double t[3 * kPackTile];
    const bool scatters = perm_scatters(perm, n);
    if (blockIdx.x == 0 && threadIdx.x == 0) *packed = scatters;
    if (!scatters) return;
    const uint32_t tiles = (n - 1) / kPackTile + 1;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const size_t base = static_cast<size_t>(tile) * kPackTile;
        const uint32_t m = static_cast<uint32_t>(min<size_t>(kPackTile, n - base));
#pragma unroll
        for (uint32_t k = 0; k < kPackTile / kPackBlock; ++k) {
            const uint32_t l = k * kPackBlock + threadIdx.x;
            if (l < m) {
                t[3 * l] = x[base + l];
                t[3 * l + 1] = y[base + l];
                t[3 * l + 2] = z[base + l];
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < 3 * kPackTile / kPackBlock; ++k) {
            const uint32_t l = k * kPackBlock + threadIdx.x;
            if (l < 3 * m) rec[3 * base + l] = t[l];
        }
        __syncthreads();
    }
}

// The gather itself. From the records, the first third of the blocks takes all;
// where perm does not scatter, the three thirds each take one array, one after
// another: a pass over one array has a smaller window to keep in the L1 (all
// three at once were 10% slower for 2^24 particles in order up to 2000 places).
// Bound: scattered reads, one or two lines per record. 2^24 particles in random
// order: three passes over the arrays 990 us, records 145 + 385 (32-byte records
// 175 + 345), 2^22: 226 against 134 us, 2^21: 98 against 67, 2^20: 44 against 34.
// Particles in order: 2^24 178 against 170 us, 2^22 38 against 39, 2^21 23 against
// 21, but 2^20 14 against 17 with what the call does on the host, so from 2^21 on.
// The records' stores go past the caches (2^25: 919 -> 838 us).
constexpr uint32_t kPackedTile = kGatherBlock * kGatherItems;
__global__ __launch_bounds__(kGatherBlock) void gather_packed_kernel(const double* __restrict__ x, const double* __restrict__ y,
                                                                     const double* __restrict__ z,
                                                                     const double* __restrict__ rec,
                                                                     const uint32_t* __restrict__ packed,
                                                                     const uint32_t* __restrict__ perm, uint32_t n,
                                                                     uint32_t tiles, double* __restrict__ ox,
                                                                     double* __restrict__ oy, double* __restrict__ oz) {
    const uint32_t third = blockIdx.x / tiles, tile = blockIdx.x - third * tiles;
    const bool records = *packed;  // uniform
    if (records && third) return;
    const size_t base = static_cast<size_t>(tile) * kPackedTile + threadIdx.x;
    size_t src[kGatherItems];
#pragma unroll
    for (int i = 0; i < kGatherItems; ++i) src[i] = base + i * kGatherBlock < n ? perm[base + i * kGatherBlock] : 0u;
    if (records) {
        double a[kGatherItems], b[kGatherItems], c[kGatherItems];
#pragma unroll
        for (int i = 0; i < kGatherItems; ++i) {
            a[i] = rec[3 * src[i]];
            b[i] = rec[3 * src[i] + 1];
            c[i] = rec[3 * src[i] + 2];
        }
#pragma unroll
        for (int i = 0; i < kGatherItems; ++i) {
            const size_t j = base + i * kGatherBlock;
            if (j < n) {
                __builtin_nontemporal_store(a[i], ox + j);
                __builtin_nontemporal_store(b[i], oy + j);
                __builtin_nontemporal_store(c[i], oz + j);
            }
        }
        return;
    }
    const double* from = third == 0 ? x : (third == 1 ? y : z);
    double* to = third == 0 ? ox : (third == 1 ? oy : oz);
    double v[kGatherItems];
#pragma unroll
    for (int i = 0; i < kGatherItems; ++i) v[i] = from[src[i]];
#pragma unroll
    for (int i = 0; i < kGatherItems; ++i)
        if (base + i * kGatherBlock < n) to[base + i * kGatherBlock] = v[i];
}

struct PackWs {
    double* rec;
    uint32_t* packed;
    size_t bytes;
};

PackWs carve_pack(void* ws, size_t n) {
    Carve c(ws);
    PackWs w{};
    w.rec = c.take<double>(3 * n);
    w.packed = c.take<uint32_t>(1);
    w.bytes = c.off;
    return w;
}

constexpr size_t kPackMin = size_t{1} << 21;

struct ScanWs {
    uint32_t *sums, *total;
    size_t tiles, bytes;
};

ScanWs carve_scan(void* ws, size_t n) {
    Carve c(ws);
    ScanWs w{};
    w.tiles = (n + 1 + kScanTile - 1) / kScanTile;
    w.sums = c.take<uint32_t>(w.tiles);
    w.total = c.take<uint32_t>(1);
    w.bytes = c.off;
    return w;
}

}  // namespace

size_t scan_u32_workspace_bytes(size_t n) { return carve_scan(nullptr, n).bytes; }

cstone_status launch_scan_u32(const uint32_t* in, size_t n, uint32_t* out, void* ws, size_t ws_bytes,
                              hipStream_t stream) {
    ScanWs w = carve_scan(ws, n);
    if (ws_bytes < w.bytes || n >= 0xffffffffull) return CSTONE_ERR_INVALID_ARG;
    const uint32_t un = static_cast<uint32_t>(n), tiles = static_cast<uint32_t>(w.tiles);
    const bool scanned = tiles > kSumTiles;
    if (tiles > 1)
        hipLaunchKernelGGL(scan_sums_kernel, dim3(tiles), dim3(kScanBlock), 0, stream, in, un, w.sums);
    if (scanned) launch_row_scan(w.sums, 1, tiles, w.total, stream);
    hipLaunchKernelGGL(exclusive_scan_kernel, dim3(tiles), dim3(kScanBlock), 0, stream, in, un, w.sums, scanned, out);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

size_t node_props_workspace_bytes(size_t n_leaves) {
    Carve c(nullptr);
    c.take<uint32_t>(n_leaves + 1);
    return c.off + scan_u32_workspace_bytes(n_leaves);
}

cstone_status launch_octree_node_counts(const uint64_t* leaves, const uint32_t* counts, size_t nl,
                                        const uint64_t* node_keys, size_t n_nodes, uint32_t* node_counts, void* ws,
                                        size_t ws_bytes, hipStream_t stream) {
    if (ws_bytes < node_props_workspace_bytes(nl)) return CSTONE_ERR_INVALID_ARG;
    Carve c(ws);
    uint32_t* S = c.take<uint32_t>(nl + 1);
    cstone_status st = launch_scan_u32(counts, nl, S, static_cast<char*>(ws) + c.off, ws_bytes - c.off, stream);
    if (st != CSTONE_OK) return st;
    if (n_nodes)
        hipLaunchKernelGGL(node_counts_tree_kernel, dim3(static_cast<uint32_t>((n_nodes + kNodeBlock - 1) / kNodeBlock)),
                           dim3(kNodeBlock), 0, stream, leaves, static_cast<uint32_t>(nl), S, node_keys,
                           static_cast<uint32_t>(n_nodes), node_counts);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

cstone_status launch_gather(const double* const* src, const uint32_t* perm, size_t n, double* const* dst, int arrays,
                            bool fused, hipStream_t stream) {
    if (n == 0) return CSTONE_OK;
    const uint32_t un = static_cast<uint32_t>(n);
    const dim3 grid(static_cast<uint32_t>((n + kGatherBlock * kGatherItems - 1) / (kGatherBlock * kGatherItems)));
    if (fused && arrays == 3) {
        hipLaunchKernelGGL(gather_kernel<3>, grid, dim3(kGatherBlock), 0, stream, src[0], src[1], src[2], perm, un,
                           dst[0], dst[1], dst[2]);
    } else {
        for (int a = 0; a < arrays; ++a)
            hipLaunchKernelGGL(gather_kernel<1>, grid, dim3(kGatherBlock), 0, stream, src[a],
                               static_cast<const double*>(nullptr), static_cast<const double*>(nullptr), perm, un,
                               dst[a], static_cast<double*>(nullptr), static_cast<double*>(nullptr));
    }
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

size_t gather_packed_workspace_bytes(size_t n) { return n < kPackMin ? 0 : carve_pack(nullptr, n).bytes; }

cstone_status launch_gather_packed(const double* const* src, const uint32_t* perm, size_t n, double* const* dst, void* ws,
                                   size_t ws_bytes, hipStream_t stream) {
    if (n < kPackMin) return launch_gather(src, perm, n, dst, 3, false, stream);
    const PackWs w = carve_pack(ws, n);
    if (!ws || ws_bytes < w.bytes) return CSTONE_ERR_INVALID_ARG;
    const uint32_t un = static_cast<uint32_t>(n), tiles = static_cast<uint32_t>((n - 1) / kPackedTile + 1);
    hipLaunchKernelGGL(gather_pack_kernel, dim3(1024), dim3(kPackBlock), 0, stream, src[0], src[1], src[2], perm, un,
                       w.rec, w.packed);
    hipLaunchKernelGGL(gather_packed_kernel, dim3(3 * tiles), dim3(kGatherBlock), 0, stream, src[0], src[1], src[2],
                       w.rec, w.packed, perm, un, tiles, dst[0], dst[1], dst[2]);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

}  // namespace cs
