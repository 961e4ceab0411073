// The replicated tree of particles spread over several ranks (Sec. 6),
// emulated on one GPU, and the partition of its leaves into rank domains.
//
// The particles are split into G shards (contiguous ranges of the input), as
// ranks would hold them; each shard's keys are sorted. A round
// then applies f to every shard (Eq. histogram against the shard's own sorted
// keys), sums the G count arrays element by element (f_r, the reduction that
// a collective over the ranks performs; here one kernel), and applies
// g = g3 . g2 . g1 to the summed counts, which every rank would do
// identically. Rounds repeat until no leaf changes. Since the counts of the
// union are the sums of the shards' counts, the result is the tree of all
// particles, bit for bit.
//
// The same rounds build the tree focused on a range F of the curve (Sec. 7):
// with one shard, and g1 replaced by g^LE_1, which splits a leaf over N_crit
// only if it fails the minimum-distance MAC against F and also merges a group
// of 8 sibling leaves whose parent passes it. The MAC of a node is evaluated
// against F cut into maximal aligned key blocks (at most 2 x 7 per level),
// whose grid boxes every block finds by itself and holds in LDS.
//
// The partition (Sec. 6) groups the leaves into n_ranks bins of consecutive
// leaves with about N / n_ranks particles each: bin r starts at the first
// leaf boundary whose particle prefix reaches r N / n_ranks.
#include <algorithm>
#include <cmath>

#include <type_traits>

#include "common.hpp"
#include "focus.hpp"
#include "internal.hpp"

namespace cs {
namespace {

constexpr int kGBlock = 256;

// f on every shard: Ng[g * nl + i] = particles of shard g in leaf i.
__global__ __launch_bounds__(kGBlock) void shard_counts_kernel(const uint64_t* __restrict__ P,
                                                               const uint64_t* __restrict__ shard_off, uint32_t G,
                                                               const uint64_t* __restrict__ K, uint32_t nl,
                                                               uint32_t* __restrict__ Ng) {
    const size_t t = static_cast<size_t>(blockIdx.x) * kGBlock + threadIdx.x;
    if (t >= static_cast<size_t>(G) * nl) return;
    const uint32_t g = static_cast<uint32_t>(t / nl), i = static_cast<uint32_t>(t % nl);
    const uint64_t a = shard_off[g], b = shard_off[g + 1];
    const uint64_t lo = lower_bound_u64(P, a, b, K[i]);
    const uint64_t hi = lower_bound_u64(P, lo, b, K[i + 1]);
    Ng[t] = static_cast<uint32_t>(hi - lo);
}

// f_r: N[i] = sum over the shards of Ng[g * nl + i].
__global__ __launch_bounds__(kGBlock) void shard_reduce_kernel(const uint32_t* __restrict__ Ng, uint32_t G,
                                                               uint32_t nl, uint32_t* __restrict__ N) {
    const uint32_t i = blockIdx.x * kGBlock + threadIdx.x;
    if (i >= nl) return;
    uint32_t sum = 0;
    for (uint32_t g = 0; g < G; ++g) sum += Ng[static_cast<size_t>(g) * nl + i];
    N[i] = sum;
}

__device__ __forceinline__ uint32_t level_of_delta(uint64_t delta) {  // delta = 8^(L - level)
    return kL - (63 - clz64(delta)) / 3;
}

// g1 (Eq. g1 with a leaf of span 1 never split, the root never merged and a
// merge iff the 8 siblings' counts sum to at most n_crit), or with FOCUS
// g^LE_1: a split also needs the leaf to fail the MAC, and a complete sibling
// group also merges if its parent passes it. O[i] in {8, 0, 1}, O[nl] = 0;
// *changed set if some O[i] != 1.
template <bool FOCUS>
__global__ __launch_bounds__(kGBlock) void global_decide_kernel(const uint64_t* __restrict__ K,
                                                                const uint32_t* __restrict__ N, uint32_t nl,
                                                                uint32_t n_crit, uint32_t* __restrict__ O,
                                                                uint32_t* changed, FocusSpec focus) {
    __shared__ std::conditional_t<FOCUS, FocusSmem, uint32_t> fsm;
    if constexpr (FOCUS) {
        focus_fill(focus, fsm);
        __syncthreads();
    }
    const uint32_t i = blockIdx.x * kGBlock + threadIdx.x;
    if (i > nl) return;
    if (i == nl) {
        O[nl] = 0;
        return;
    }
    const uint64_t k = K[i], delta = K[i + 1] - k;
    uint32_t op = 1;
    bool split = N[i] > n_crit && delta > 1;
    if constexpr (FOCUS) {
        if (split) split = node_fails(k, level_of_delta(delta), focus, fsm);
    }
    if (split) {
        op = 8;
    } else if (delta < kKeyEnd) {
        const uint64_t j = (k % (8 * delta)) / delta;  // place among the siblings
        if (j >= 1 && i >= j && i - j + 8 <= nl && K[i - j] + 8 * delta == K[i - j + 8]) {
            uint64_t group = 0;
            for (uint32_t m = 0; m < 8; ++m) group += N[i - j + m];
            bool merge = group <= n_crit;
            if constexpr (FOCUS) {
                // the parent passes the MAC
                if (!merge) merge = !node_fails(K[i - j], level_of_delta(delta) - 1, focus, fsm);
            }
            if (merge) op = 0;
        }
    }
    O[i] = op;
    if (__ballot(op != 1) && lane_id() == 0) atomicOr(changed, 1u);
}

// f^LE_2: the MAC of every node of a linked octree (placeholder keys), 1 if
// it fails against the focus range.
__global__ __launch_bounds__(kGBlock) void focus_mac_kernel(const uint64_t* __restrict__ NK, uint32_t n,
                                                            FocusSpec focus, uint8_t* __restrict__ fails) {
    __shared__ FocusSmem fsm;
    focus_fill(focus, fsm);
    __syncthreads();
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * kGBlock;
    for (uint64_t p = blockIdx.x * kGBlock + threadIdx.x; p < n; p += stride) {
        const uint64_t key = NK[p];
        const int level = (63 - clz64(key)) / 3;
        const uint64_t start = (key ^ (1ull << (3 * level))) << (3 * (kL - level));
        fails[p] = node_fails(start, level, focus, fsm) ? 1 : 0;
    }
}

// g3 (Eqs. rebalancecopy, rebalancesplit) into K_out, unless the new array
// (Op[nl] + 1 keys) exceeds the capacity.
__global__ __launch_bounds__(kGBlock) void global_write_kernel(const uint64_t* __restrict__ K,
                                                               const uint32_t* __restrict__ O,
                                                               const uint32_t* __restrict__ Op, uint32_t nl,
                                                               uint64_t cap, uint64_t* __restrict__ K_out) {
    const uint32_t i = blockIdx.x * kGBlock + threadIdx.x;
    if (i > nl || Op[nl] > cap) return;
    if (i == nl) {
        K_out[Op[nl]] = kKeyEnd;
        return;
    }
    const uint64_t k = K[i];
    if (O[i] == 1) {
        K_out[Op[i]] = k;
    } else if (O[i] == 8) {
        const uint64_t step = (K[i + 1] - k) / 8;
        for (uint32_t j = 0; j < 8; ++j) K_out[Op[i] + j] = k + j * step;
    }
}

// bounds[r] = min { i <= nl : S[i] * R >= r * S[nl] } for r < R, bounds[R] = nl;
// a wave per bound, 64 probes a step (a thread each: 20 dependent reads of 1.1 M
// sums, 7 us; now 4).
__global__ __launch_bounds__(kGBlock) void partition_kernel(const uint32_t* __restrict__ S, uint32_t nl, uint32_t R,
                                                            uint32_t* __restrict__ bounds) {
    const uint32_t lane = lane_id();
    const uint32_t r = blockIdx.x * (kGBlock / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (r > R) return;
    const uint64_t target = static_cast<uint64_t>(r) * S[nl];
    uint32_t lo = 0, hi = r == R ? 0u : nl;  // the answer lies in [lo, hi]
    while (lo < hi) {
        // probes lo, lo + step, ...: those below the target come first
        const uint32_t step = (hi - lo - 1) / kWave + 1;
        const uint64_t i = lo + static_cast<uint64_t>(step) * lane;
        const bool below = i < hi && static_cast<uint64_t>(S[i]) * R < target;
        const uint32_t c = static_cast<uint32_t>(__popcll(__ballot(below)));
        if (c == 0) break;  // lo itself
        hi = static_cast<uint32_t>(min<uint64_t>(hi, lo + static_cast<uint64_t>(step) * c));
        lo += step * (c - 1) + 1;
    }
    if (lane == 0) bounds[r] = r == R ? nl : lo;
}

// The same, a thread per bound: for many ranks, which fill the chip that way.
__global__ __launch_bounds__(kGBlock) void partition_many_kernel(const uint32_t* __restrict__ S, uint32_t nl, uint32_t R,
                                                                 uint32_t* __restrict__ bounds) {
    const uint64_t r = static_cast<uint64_t>(blockIdx.x) * kGBlock + threadIdx.x;
    if (r > R) return;
    const uint64_t target = r * S[nl];
    uint32_t lo = 0, hi = r == R ? 0u : nl;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (static_cast<uint64_t>(S[mid]) * R >= target)
            hi = mid;
        else
            lo = mid + 1;
    }
    bounds[r] = r == R ? nl : lo;
}

struct GlobalWs {
    uint64_t* K_alt;
    uint32_t *Ng, *N, *O, *Op, *flags;
    void* scan;
    size_t scan_bytes, bytes;
};

GlobalWs carve_global(void* ws, size_t cap, uint32_t G) {
    Carve c(ws);
    GlobalWs w{};
    w.K_alt = c.take<uint64_t>(cap + 1);
    w.Ng = c.take<uint32_t>(static_cast<size_t>(G) * cap);
    w.N = c.take<uint32_t>(cap);
    w.O = c.take<uint32_t>(cap + 1);
    w.Op = c.take<uint32_t>(cap + 1);
    w.flags = c.take<uint32_t>(2);
    w.scan_bytes = scan_u32_workspace_bytes(cap + 1);
    w.scan = c.take<char>(w.scan_bytes);
    w.bytes = c.off;
    return w;
}

uint32_t grid_of(size_t items) { return static_cast<uint32_t>(std::max<size_t>(1, (items + kGBlock - 1) / kGBlock)); }

}  // namespace

__global__ void clear_flags_kernel(uint32_t* f) { f[0] = 0; }

size_t global_rebalance_workspace_bytes(size_t leaf_capacity, uint32_t G) {
    return carve_global(nullptr, leaf_capacity, G).bytes;
}

namespace {

cstone_status run_rounds(const uint64_t* P, const uint64_t* shard_off_dev, uint32_t G, uint32_t n_crit,
                         uint64_t* leaves, size_t* n_leaves, size_t cap, uint32_t* counts, uint32_t max_iters,
                         uint32_t* iters_done, void* ws, size_t ws_bytes, const FocusSpec* focus,
                         hipStream_t stream) {
    GlobalWs w = carve_global(ws, cap, G);
    if (ws_bytes < w.bytes) return CSTONE_ERR_INVALID_ARG;
    if (max_iters == 0) max_iters = kL + 1;
    uint64_t* buf[2] = {leaves, w.K_alt};
    int cur = 0;
    size_t nl = *n_leaves;
    uint32_t rounds = 0;
    cstone_status status = CSTONE_ERR_NOT_CONVERGED;
    while (rounds < max_iters) {
        const uint32_t unl = static_cast<uint32_t>(nl);
        hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(1), 0, stream, w.flags);
        hipLaunchKernelGGL(shard_counts_kernel, dim3(grid_of(static_cast<size_t>(G) * nl)), dim3(kGBlock), 0, stream,
                           P, shard_off_dev, G, buf[cur], unl, w.Ng);
        hipLaunchKernelGGL(shard_reduce_kernel, dim3(grid_of(nl)), dim3(kGBlock), 0, stream, w.Ng, G, unl, w.N);
        if (focus)
            hipLaunchKernelGGL(global_decide_kernel<true>, dim3(grid_of(nl + 1)), dim3(kGBlock), 0, stream, buf[cur],
                               w.N, unl, n_crit, w.O, w.flags, *focus);
        else
            hipLaunchKernelGGL(global_decide_kernel<false>, dim3(grid_of(nl + 1)), dim3(kGBlock), 0, stream, buf[cur],
                               w.N, unl, n_crit, w.O, w.flags, FocusSpec{});
        cstone_status st = launch_scan_u32(w.O, nl, w.Op, w.scan, w.scan_bytes, stream);
        if (st != CSTONE_OK) return st;
        hipLaunchKernelGGL(global_write_kernel, dim3(grid_of(nl + 1)), dim3(kGBlock), 0, stream, buf[cur], w.O, w.Op,
                           unl, static_cast<uint64_t>(cap), buf[cur ^ 1]);
        CS_HIP(hipGetLastError());
        uint32_t host[2] = {0, 0};  // changed, new leaf count
        CS_HIP(hipMemcpyAsync(&host[0], w.flags, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
        CS_HIP(hipMemcpyAsync(&host[1], w.Op + nl, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
        CS_HIP(hipStreamSynchronize(stream));
        ++rounds;
        if (!host[0]) {  // converged: the summed counts belong to the final array
            status = CSTONE_OK;
            break;
        }
        if (host[1] > cap) {
            status = CSTONE_ERR_CAPACITY;
            *n_leaves = host[1];
            break;
        }
        cur ^= 1;
        nl = host[1];
    }
    if (status == CSTONE_ERR_NOT_CONVERGED) {  // counts of the last array
        const uint32_t unl = static_cast<uint32_t>(nl);
        hipLaunchKernelGGL(shard_counts_kernel, dim3(grid_of(static_cast<size_t>(G) * nl)), dim3(kGBlock), 0, stream,
                           P, shard_off_dev, G, buf[cur], unl, w.Ng);
        hipLaunchKernelGGL(shard_reduce_kernel, dim3(grid_of(nl)), dim3(kGBlock), 0, stream, w.Ng, G, unl, w.N);
    }
    if (status != CSTONE_ERR_CAPACITY) {
        if (cur == 1) CS_HIP(hipMemcpyAsync(leaves, w.K_alt, (nl + 1) * sizeof(uint64_t), hipMemcpyDeviceToDevice, stream));
        if (counts) CS_HIP(hipMemcpyAsync(counts, w.N, nl * sizeof(uint32_t), hipMemcpyDeviceToDevice, stream));
        CS_HIP(hipStreamSynchronize(stream));
        *n_leaves = nl;
    } else if (cur == 1) {  // leave the last valid array in `leaves`
        CS_HIP(hipMemcpyAsync(leaves, w.K_alt, (nl + 1) * sizeof(uint64_t), hipMemcpyDeviceToDevice, stream));
        CS_HIP(hipStreamSynchronize(stream));
    }
    if (iters_done) *iters_done = rounds;
    return status;
}

}  // namespace

cstone_status run_global_rebalance(const uint64_t* P, const uint64_t* shard_off_dev, uint32_t G, uint32_t n_crit,
                                   uint64_t* leaves, size_t* n_leaves, size_t cap, uint32_t* counts,
                                   uint32_t max_iters, uint32_t* iters_done, void* ws, size_t ws_bytes,
                                   hipStream_t stream) {
    return run_rounds(P, shard_off_dev, G, n_crit, leaves, n_leaves, cap, counts, max_iters, iters_done, ws, ws_bytes,
                      nullptr, stream);
}

// The focused tree comes from the sorted keys directly (tree.hip), if so many
// rounds are allowed: one pass over the keys replaces the rounds' searches,
// launches and waits for the host. 4 M Plummer particles, N_crit 32, one of 64
// ranges, with links and the nodes' MAC: 1000 -> 200 us. From the root (5 to 15
// rounds) it is the faster one at least to 2^26 keys (Plummer, N_crit 16: 936
// against 1784 us). From another tree it takes a round to see that nothing has
// changed and two for a little, whatever n; direct against rounds in us, unchanged
// / changed: 2^18 Plummer keys, N_crit 16: 216 / 217 against 169 / 307, 2^20 232 /
// 233 against 165 / 295, 2^22 272 / 275 against 176 / 314, 2^24 472 / 472 against
// 188 / 336; N_crit 1000: 2^20 168 / 171 against 158 / 273, 2^24 336 / 332 against
// 175 / 313.
constexpr size_t kFocusDirect = size_t{1} << 21, kFocusDirectRoot = size_t{1} << 27;

size_t focus_rounds_bytes(size_t leaf_capacity) {
    Carve c(nullptr);
    c.take<uint64_t>(2);
    return c.off + global_rebalance_workspace_bytes(leaf_capacity, 1);
}

size_t focus_workspace_bytes(size_t leaf_capacity) {
    return std::max(focus_rounds_bytes(leaf_capacity),
                    leaf_capacity ? focus_tree_workspace_bytes(kFocusDirectRoot, leaf_capacity) : 0);
}

cstone_status run_focus_rebalance(const uint64_t* P, size_t n, uint32_t n_crit, int curve, uint64_t fa, uint64_t fb,
                                  double theta, uint64_t* leaves, size_t* n_leaves, size_t cap, uint32_t* counts,
                                  uint32_t max_iters, uint32_t* iters_done, void* ws, size_t ws_bytes,
                                  hipStream_t stream) {
    if (ws_bytes < focus_rounds_bytes(cap)) return CSTONE_ERR_INVALID_ARG;
    const FocusSpec f{fa, fb, curve, theta * theta};
    if (tree_possible(n, max_iters) && n <= (*n_leaves > 1 ? kFocusDirect : kFocusDirectRoot)) {
        TreePass tree;
        if (tree.run(P, n, n_crit, leaves, *n_leaves, cap, counts, nullptr, nullptr, nullptr, ws, ws_bytes, nullptr,
                     nullptr, nullptr, stream, &f)) {
            bool fits = false;
            const cstone_status s = tree.wait(&fits);
            if (s != CSTONE_OK) return s;
            if (fits) {
                *n_leaves = tree.n_leaves;
                if (iters_done) *iters_done = tree.rounds;
                return CSTONE_OK;
            }
        }
    }
    Carve c(ws);
    uint64_t* off = c.take<uint64_t>(2);
    const uint64_t host_off[2] = {0, n};
    CS_HIP(hipMemcpyAsync(off, host_off, sizeof host_off, hipMemcpyHostToDevice, stream));
    return run_rounds(P, off, 1, n_crit, leaves, n_leaves, cap, counts, max_iters, iters_done,
                      static_cast<char*>(ws) + c.off, ws_bytes - c.off, &f, stream);
}

// At most so many blocks (four on a CU), since each first finds the range's key
// blocks. By a block per 256 nodes and now: 2.5 M nodes, a range of one key block
// 27 -> 18 us, a ragged one 116 -> 35; 1.3 M 16 -> 13 and 65 -> 34.
constexpr uint32_t kMacBlocks = 1024;

// What callers have to pass, as they always had; nothing is kept in it.
size_t focus_mac_workspace_bytes() { return kMaxFocusBlocks * sizeof(uint4); }

cstone_status launch_focus_mac(const uint64_t* node_keys, size_t n_nodes, int curve, uint64_t fa, uint64_t fb,
                               double theta, uint8_t* fails, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (!ws || ws_bytes < focus_mac_workspace_bytes()) return CSTONE_ERR_INVALID_ARG;
    const FocusSpec f{fa, fb, curve, theta * theta};
    if (n_nodes)
        hipLaunchKernelGGL(focus_mac_kernel, dim3(std::min(grid_of(n_nodes), kMacBlocks)), dim3(kGBlock), 0, stream, node_keys,
                           static_cast<uint32_t>(n_nodes), f, fails);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

size_t sfc_partition_workspace_bytes(size_t n_leaves) {
    Carve c(nullptr);
    c.take<uint32_t>(n_leaves + 1);
    return c.off + scan_u32_workspace_bytes(n_leaves);
}

// From so many ranks on a thread per bound. Whole calls by a wave per bound against
// a thread: 1.1 M leaves, 16,384 ranks 20 / 19 us, 65,536 35 / 19, 200,000 68 / 20; 7
// M leaves, 8192 59 / 59, 16,384 62 / 59, 200,000 121 / 64.
constexpr uint32_t kManyRanks = 1u << 14;

cstone_status launch_sfc_partition(const uint32_t* counts, size_t nl, uint32_t n_ranks, uint32_t* bounds, void* ws,
                                   size_t ws_bytes, hipStream_t stream) {
    if (ws_bytes < sfc_partition_workspace_bytes(nl)) return CSTONE_ERR_INVALID_ARG;
    Carve c(ws);
    uint32_t* S = c.take<uint32_t>(nl + 1);
    cstone_status st = launch_scan_u32(counts, nl, S, static_cast<char*>(ws) + c.off, ws_bytes - c.off, stream);
    if (st != CSTONE_OK) return st;
    const size_t bounds_n = static_cast<size_t>(n_ranks) + 1;
    if (n_ranks < kManyRanks)
        hipLaunchKernelGGL(partition_kernel, dim3(grid_of(bounds_n * kWave)), dim3(kGBlock), 0, stream, S,
                           static_cast<uint32_t>(nl), n_ranks, bounds);
    else
        hipLaunchKernelGGL(partition_many_kernel, dim3(grid_of(bounds_n)), dim3(kGBlock), 0, stream, S,
                           static_cast<uint32_t>(nl), n_ranks, bounds);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}


namespace {

// ---- shards out of the order of all keys ---------------------------------------
//
// Every shard's sorted keys are a stable selection from the sorted keys of all
// shards (the sort keeps input order among equal keys, and a shard is a range of
// the input). So one sort of all keys serves the tree and, parted by the shard
// that each key's particle lies in, every shard: 12 B a particle read and
// written once more instead of a sort per shard one after another, and no search
// of all shards in every round. 2^24 uniform particles in 8 shards: the sorts and
// rounds took 2350 us of 2480, now 750 of 880.

constexpr int kShardBlock = 512;
constexpr int kShardItems = 8;
constexpr uint32_t kShardTile = kShardBlock * kShardItems;
constexpr int kShardWaves = kShardBlock / kWave;
constexpr uint32_t kMaxPartShards = 64;  // one thread per wave and shard; runs of 64 keys per tile and shard

// This thread's items of the tile (places wave * 512 + it * 64 + lane, so that a
// wave's items are in order): shard of each (kMaxPartShards: none) and its rank
// among the wave's items of that shard; counts[shard][wave].
__device__ __forceinline__ void shard_ranks(const uint32_t idx[kShardItems], uint32_t first, uint32_t lane, uint64_t left,
                                            const uint64_t* off, uint32_t G, uint32_t bits, uint32_t* counts,
                                            uint32_t wave, uint32_t shard[kShardItems], uint32_t rank[kShardItems]) {
#pragma unroll
    for (int it = 0; it < kShardItems; ++it) {
        const bool in = first + it * kWave + lane < left;
        uint32_t lo = 0, hi = G;  // the last shard that starts at or before idx
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (off[mid] <= idx[it])
                lo = mid;
            else
                hi = mid;
        }
        uint64_t same = __ballot(in);
        for (uint32_t b = 0; b < bits; ++b) {
            const bool bit = (lo >> b) & 1u;
            const uint64_t m = __ballot(bit);
            same &= bit ? m : ~m;
        }
        shard[it] = in ? lo : kMaxPartShards;
        const uint32_t below = lanes_below(same);
        uint32_t* count = counts + lo * kShardWaves + wave;
        const uint32_t base = in ? *count : 0u;
        rank[it] = base + below;
        __builtin_amdgcn_wave_barrier();
        if (in && below == 0) *count = base + static_cast<uint32_t>(__popcll(same));
        __builtin_amdgcn_wave_barrier();
    }
}

struct ShardSmem {
    uint64_t off[kMaxPartShards + 1];
    uint32_t counts[kMaxPartShards * kShardWaves];
};

__device__ __forceinline__ void shard_smem_fill(const uint64_t* off, uint32_t G, ShardSmem& sm) {
    for (uint32_t g = threadIdx.x; g <= G; g += kShardBlock) sm.off[g] = off[g];
    for (uint32_t i = threadIdx.x; i < G * kShardWaves; i += kShardBlock) sm.counts[i] = 0;
    __syncthreads();
}

// rows[g][tile]: particles of shard g among the tile's. Bound: the chain of
// search, ballots and counts per item (33 us for 2^24; reading perm alone is 13).
__global__ __launch_bounds__(kShardBlock) void shard_tile_counts_kernel(const uint32_t* __restrict__ perm, uint64_t n,
                                                                        const uint64_t* __restrict__ off, uint32_t G,
                                                                        uint32_t bits, uint32_t* __restrict__ rows) {
    __shared__ ShardSmem sm;
    shard_smem_fill(off, G, sm);
    const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kShardTile, left = n - base;
    const uint32_t first = wave * kShardItems * kWave;
    uint32_t idx[kShardItems], shard[kShardItems], rank[kShardItems];
#pragma unroll
    for (int it = 0; it < kShardItems; ++it) {
        const uint32_t i = first + it * kWave + lane;
        idx[it] = i < left ? perm[base + i] : 0u;
    }
    shard_ranks(idx, first, lane, left, sm.off, G, bits, sm.counts, wave, shard, rank);
    __syncthreads();
    if (threadIdx.x < G) {
        uint32_t sum = 0;
        for (int w = 0; w < kShardWaves; ++w) sum += sm.counts[threadIdx.x * kShardWaves + w];
        rows[static_cast<size_t>(threadIdx.x) * gridDim.x + blockIdx.x] = sum;
    }
}

// The tile's keys and particles to their shards, in order; rows scanned. They
// are put in the shards' order in LDS first, so that every shard's run is
// written whole. Bound: 12 B a particle read and 12 written (90 us for 2^24, 4.5
// TB/s).
__global__ __launch_bounds__(kShardBlock) void shard_write_kernel(const uint64_t* __restrict__ P,
                                                                  const uint32_t* __restrict__ perm, uint64_t n,
                                                                  const uint64_t* __restrict__ off, uint32_t G,
                                                                  uint32_t bits, const uint32_t* __restrict__ rows,
                                                                  uint64_t* __restrict__ out_keys,
                                                                  uint32_t* __restrict__ out_perm) {
    __shared__ ShardSmem sm;
    __shared__ uint64_t keys[kShardTile];
    __shared__ uint32_t vals[kShardTile];
    __shared__ uint8_t of[kShardTile];
    __shared__ uint64_t to[kMaxPartShards];  // where the shard's run of the tile goes, less its place in the tile
    __shared__ uint32_t tmp[kShardWaves];
    shard_smem_fill(off, G, sm);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kShardTile, left = n - base;
    const uint32_t first = wave * kShardItems * kWave;
    uint64_t k[kShardItems];
    uint32_t idx[kShardItems], shard[kShardItems], rank[kShardItems];
#pragma unroll
    for (int it = 0; it < kShardItems; ++it) {
        const uint32_t i = first + it * kWave + lane;
        idx[it] = i < left ? perm[base + i] : 0u;
        k[it] = i < left ? P[base + i] : 0ull;
    }
    shard_ranks(idx, first, lane, left, sm.off, G, bits, sm.counts, wave, shard, rank);
    __syncthreads();
    const uint32_t mine = tid < G * kShardWaves ? sm.counts[tid] : 0u;  // shard tid / waves, wave tid % waves
    uint32_t total;
    const uint32_t at = block_exclusive_sum<uint32_t, kShardBlock>(mine, tmp, &total);
    if (tid < G * kShardWaves) {
        sm.counts[tid] = at;
        const uint32_t g = tid / kShardWaves;
        if (tid % kShardWaves == 0) to[g] = sm.off[g] + rows[static_cast<size_t>(g) * gridDim.x + blockIdx.x] - at;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kShardItems; ++it) {
        if (shard[it] < kMaxPartShards) {
            const uint32_t p = sm.counts[shard[it] * kShardWaves + wave] + rank[it];
            keys[p] = k[it];
            vals[p] = idx[it] - static_cast<uint32_t>(sm.off[shard[it]]);
            of[p] = static_cast<uint8_t>(shard[it]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kShardItems; ++it) {
        const uint32_t p = it * kShardBlock + tid;
        if (p < total) {
            const uint64_t d = to[of[p]] + p;
            if (d < n) {  // (always; guards memory should the sort have failed)
                out_keys[d] = keys[p];
                out_perm[d] = vals[p];
            }
        }
    }
}

// Workspace of the sharded build: unsorted keys and the shard offsets on the
// device; then the sorts (one shard at a time) or the rounds; or all keys
// sorted, the rows of the tiles' counts, and the sort or the tree of all.
struct ShardedWs {
    uint64_t* keys;
    uint64_t* off;
    void* stage;
    size_t stage_bytes, bytes;  // sort per shard, rounds
    uint32_t* flag;
    uint64_t* all_keys;
    uint32_t *all_perm, *rows, *totals;
    void* all_stage;
    size_t all_stage_bytes, all_bytes;  // one sort
};

ShardedWs carve_sharded(void* ws, size_t n, size_t max_shard, size_t cap, uint32_t G) {
    Carve c(ws);
    ShardedWs w{};
    w.keys = c.take<uint64_t>(n);
    w.off = c.take<uint64_t>(G + 1);
    Carve one = c;
    w.stage_bytes = std::max(sort_workspace_bytes(max_shard, true), cs::global_rebalance_workspace_bytes(cap, G));
    w.stage = c.take<char>(w.stage_bytes);
    w.bytes = c.off;
    w.flag = one.take<uint32_t>(1);
    w.all_keys = one.take<uint64_t>(n);
    w.all_perm = one.take<uint32_t>(n);
    w.rows = one.take<uint32_t>(static_cast<size_t>(G) * ((n + kShardTile - 1) / kShardTile));
    w.totals = one.take<uint32_t>(G);
    w.all_stage_bytes = std::max(prepared_sort_workspace_bytes(n), n && cap ? tree_workspace_bytes(n, 1, cap, true) : 0);
    w.all_stage = one.take<char>(w.all_stage_bytes);
    w.all_bytes = one.off;
    return w;
}

bool offsets_ok(const uint64_t* off, uint32_t G, size_t n, size_t* max_shard) {
    if (!off || G == 0 || off[0] != 0 || off[G] != n) return false;
    size_t mx = 0;
    for (uint32_t g = 0; g < G; ++g) {
        if (off[g + 1] < off[g]) return false;
        mx = std::max<size_t>(mx, off[g + 1] - off[g]);
    }
    if (max_shard) *max_shard = mx;
    return true;
}

constexpr size_t kMaxN = 0xffffffffull;

// Keys, shards and tree by one sort. *done false: shards are sorted, but the
// rounds have to say how far the capacity lets them come.
cstone_status build_shards_at_once(const double* x, const double* y, const double* z, size_t n,
                                   const uint64_t* shard_offsets, uint32_t G, const cstone_box& box, cstone_curve curve,
                                   uint32_t n_crit, uint64_t* sorted_keys, uint32_t* perm, uint64_t* leaves,
                                   size_t* n_leaves, size_t cap, uint32_t* counts, uint32_t* iters_done,
                                   const ShardedWs& w, bool* done, hipStream_t stream) {
    const int variant = sort_resolve_variant(n);
    uint32_t *hist_parts = nullptr, *bad_parts = nullptr, hist_mask = 0, hist_shift = 0, parts = 0, hist_digits = 1;
    sort_key_parts(w.all_stage, n, true, 63, variant, &hist_parts, &bad_parts, &hist_mask, &hist_shift, &hist_digits);
    cstone_status st = launch_keys(x, y, z, n, box, curve, w.keys, nullptr, stream, hist_parts, hist_mask, hist_shift,
                                   bad_parts, &parts, hist_digits);
    if (st != CSTONE_OK) return st;
    st = sort_setup_from_keys(w.all_stage, n, true, variant, parts, w.keys, w.flag, nullptr, 0, stream);
    if (st != CSTONE_OK) return st;
    uint32_t host_flag = 0;
    CS_HIP(hipMemcpyAsync(&host_flag, w.flag, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    CS_HIP(hipMemcpyAsync(w.off, shard_offsets, (static_cast<size_t>(G) + 1) * sizeof(uint64_t), hipMemcpyHostToDevice,
                          stream));
    CS_HIP(hipStreamSynchronize(stream));
    if (host_flag & CSTONE_FLAG_NONFINITE) return CSTONE_ERR_NONFINITE;
    uint64_t* all_keys = G > 1 ? w.all_keys : sorted_keys;
    uint32_t* all_perm = G > 1 ? w.all_perm : perm;
    st = launch_sort(w.keys, all_keys, all_perm, n, 63, w.all_stage, w.all_stage_bytes, stream, nullptr,
                     /*prepared=*/true, variant, w.flag);
    if (st != CSTONE_OK) return st;
    if (G > 1) {
        const uint32_t tiles = static_cast<uint32_t>((n + kShardTile - 1) / kShardTile);
        uint32_t bits = 0;
        while ((1u << bits) < G) ++bits;
        const uint64_t un = n;
        hipLaunchKernelGGL(shard_tile_counts_kernel, dim3(tiles), dim3(kShardBlock), 0, stream, all_perm, un, w.off, G,
                           bits, w.rows);
        launch_row_scan(w.rows, G, tiles, w.totals, stream);
        hipLaunchKernelGGL(shard_write_kernel, dim3(tiles), dim3(kShardBlock), 0, stream, all_keys, all_perm, un, w.off,
                           G, bits, w.rows, sorted_keys, perm);
    }
    TreePass tree;
    if (!tree.run(all_keys, n, n_crit, leaves, *n_leaves, cap, counts, nullptr, nullptr, nullptr, w.all_stage,
                  w.all_stage_bytes, nullptr, w.flag, nullptr, stream))
        return CSTONE_ERR_INVALID_ARG;  // (the workspace covers it)
    st = tree.wait(done);
    if (st != CSTONE_OK) return st;
    if (tree.input_flags) return CSTONE_ERR_DEVICE;  // the sort gave up a wait
    if (*done) {
        *n_leaves = tree.n_leaves;
        if (iters_done) *iters_done = tree.rounds;
    }
    return CSTONE_OK;
}

}  // namespace
}  // namespace cs

extern "C" {

CSTONE_API size_t cstone_global_rebalance_workspace_bytes(size_t leaf_capacity, uint32_t n_shards) {
    cs::Carve c(nullptr);
    c.take<uint64_t>(static_cast<size_t>(n_shards) + 1);
    return c.off + cs::global_rebalance_workspace_bytes(leaf_capacity, n_shards);
}

CSTONE_API cstone_status cstone_global_rebalance(const uint64_t* sorted_keys, const uint64_t* shard_offsets,
                                                 uint32_t n_shards, uint32_t n_crit, uint64_t* leaves,
                                                 size_t* n_leaves, size_t leaf_capacity, uint32_t* counts,
                                                 uint32_t max_iters, uint32_t* iters_done, void* ws, size_t ws_bytes,
                                                 hipStream_t stream) {
    if (n_crit == 0 || !leaves || !n_leaves || !ws || n_shards == 0 || !shard_offsets) return CSTONE_ERR_INVALID_ARG;
    const size_t n = shard_offsets[n_shards];
    if (n > cs::kMaxN || !cs::offsets_ok(shard_offsets, n_shards, n, nullptr) || (n && !sorted_keys))
        return CSTONE_ERR_INVALID_ARG;
    if (*n_leaves < 1 || *n_leaves > leaf_capacity || leaf_capacity >= cs::kMaxN) return CSTONE_ERR_INVALID_ARG;
    if (ws_bytes < cstone_global_rebalance_workspace_bytes(leaf_capacity, n_shards)) return CSTONE_ERR_INVALID_ARG;
    cs::Carve c(ws);
    uint64_t* off = c.take<uint64_t>(static_cast<size_t>(n_shards) + 1);
    CS_HIP(hipMemcpyAsync(off, shard_offsets, (static_cast<size_t>(n_shards) + 1) * sizeof(uint64_t),
                          hipMemcpyHostToDevice, stream));
    return cs::run_global_rebalance(sorted_keys, off, n_shards, n_crit, leaves, n_leaves, leaf_capacity, counts,
                                    max_iters, iters_done, static_cast<char*>(ws) + c.off, ws_bytes - c.off, stream);
}

CSTONE_API size_t cstone_build_sharded_workspace_bytes(const uint64_t* shard_offsets, uint32_t n_shards,
                                                       size_t leaf_capacity) {
    size_t mx = 0;
    if (!shard_offsets || !cs::offsets_ok(shard_offsets, n_shards, shard_offsets[n_shards], &mx)) return 0;
    const cs::ShardedWs w = cs::carve_sharded(nullptr, shard_offsets[n_shards], mx, leaf_capacity, n_shards);
    return n_shards <= cs::kMaxPartShards ? std::max(w.bytes, w.all_bytes) : w.bytes;
}

CSTONE_API size_t cstone_build_sharded_least_workspace_bytes(const uint64_t* shard_offsets, uint32_t n_shards,
                                                             size_t leaf_capacity) {
    size_t mx = 0;
    if (!shard_offsets || !cs::offsets_ok(shard_offsets, n_shards, shard_offsets[n_shards], &mx)) return 0;
    return cs::carve_sharded(nullptr, shard_offsets[n_shards], mx, leaf_capacity, n_shards).bytes;
}

CSTONE_API cstone_status cstone_build_sharded(const double* x, const double* y, const double* z,
                                              const uint64_t* shard_offsets, uint32_t n_shards,
                                              const cstone_box* box, cstone_curve curve, uint32_t n_crit,
                                              uint64_t* sorted_keys, uint32_t* perm, uint64_t* leaves,
                                              size_t* n_leaves, size_t leaf_capacity, uint32_t* counts,
                                              uint32_t max_iters, uint32_t* iters_done, void* ws, size_t ws_bytes,
                                              hipStream_t stream) {
    size_t mx = 0;
    if (!shard_offsets || n_shards == 0) return CSTONE_ERR_INVALID_ARG;
    const size_t n = shard_offsets[n_shards];
    if (n > cs::kMaxN || !cs::offsets_ok(shard_offsets, n_shards, n, &mx) || n_crit == 0 || !box || !leaves ||
        !n_leaves || !ws)
        return CSTONE_ERR_INVALID_ARG;
    if (n && (!x || !y || !z || !sorted_keys || !perm)) return CSTONE_ERR_INVALID_ARG;
    if (curve != CSTONE_MORTON && curve != CSTONE_HILBERT) return CSTONE_ERR_INVALID_ARG;
    if (*n_leaves < 1 || *n_leaves > leaf_capacity || leaf_capacity >= cs::kMaxN) return CSTONE_ERR_INVALID_ARG;
    for (int d = 0; d < 3; ++d)
        if (!std::isfinite(box->lo[d]) || !std::isfinite(box->hi[d]) || !(box->lo[d] < box->hi[d]))
            return CSTONE_ERR_INVALID_ARG;
    cs::ShardedWs w = cs::carve_sharded(ws, n, mx, leaf_capacity, n_shards);
    if (ws_bytes < w.bytes) return CSTONE_ERR_INVALID_ARG;
    if (n_shards <= cs::kMaxPartShards && ws_bytes >= w.all_bytes && cs::tree_possible(n, max_iters)) {
        bool done = false;
        const cstone_status st = cs::build_shards_at_once(x, y, z, n, shard_offsets, n_shards, *box, curve, n_crit,
                                                          sorted_keys, perm, leaves, n_leaves, leaf_capacity, counts,
                                                          iters_done, w, &done, stream);
        if (st != CSTONE_OK || done) return st;
        return cs::run_global_rebalance(sorted_keys, w.off, n_shards, n_crit, leaves, n_leaves, leaf_capacity, counts,
                                        max_iters, iters_done, w.stage, w.stage_bytes, stream);
    }
    // keys of every particle (a rank's keys depend only on its own particles),
    // with the non-finite flag in the first word of the offsets' slot, read
    // back before the offsets are copied in
    uint32_t* flag = reinterpret_cast<uint32_t*>(w.off);
    hipLaunchKernelGGL(cs::clear_flags_kernel, dim3(1), dim3(1), 0, stream, flag);
    cstone_status st = cs::launch_keys(x, y, z, n, *box, curve, w.keys, flag, stream);
    if (st != CSTONE_OK) return st;
    uint32_t host_flag = 0;
    CS_HIP(hipMemcpyAsync(&host_flag, flag, sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    CS_HIP(hipStreamSynchronize(stream));
    if (host_flag & CSTONE_FLAG_NONFINITE) return CSTONE_ERR_NONFINITE;
    // every shard's keys sorted on their own (perm relative to the shard's first particle)
    for (uint32_t g = 0; g < n_shards; ++g) {
        const size_t a = shard_offsets[g], m = shard_offsets[g + 1] - a;
        if (m == 0) continue;
        st = cs::launch_sort(w.keys + a, sorted_keys + a, perm + a, m, 63, w.stage, w.stage_bytes, stream);
        if (st != CSTONE_OK) return st;
    }
    CS_HIP(hipMemcpyAsync(w.off, shard_offsets, (static_cast<size_t>(n_shards) + 1) * sizeof(uint64_t),
                          hipMemcpyHostToDevice, stream));
    return cs::run_global_rebalance(sorted_keys, w.off, n_shards, n_crit, leaves, n_leaves, leaf_capacity, counts,
                                    max_iters, iters_done, w.stage, w.stage_bytes, stream);
}

CSTONE_API size_t cstone_focus_rebalance_workspace_bytes(size_t leaf_capacity) {
    return cs::focus_workspace_bytes(leaf_capacity);
}

CSTONE_API size_t cstone_focus_rebalance_least_workspace_bytes(size_t leaf_capacity) {
    return cs::focus_rounds_bytes(leaf_capacity);
}

CSTONE_API cstone_status cstone_focus_rebalance(const uint64_t* sorted_keys, size_t n, uint32_t n_crit,
                                                cstone_curve curve, uint64_t focus_start, uint64_t focus_end,
                                                double theta, uint64_t* leaves, size_t* n_leaves,
                                                size_t leaf_capacity, uint32_t* counts, uint32_t max_iters,
                                                uint32_t* iters_done, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n > cs::kMaxN || n_crit == 0 || !leaves || !n_leaves || !ws || (n && !sorted_keys)) return CSTONE_ERR_INVALID_ARG;
    if (curve != CSTONE_MORTON && curve != CSTONE_HILBERT) return CSTONE_ERR_INVALID_ARG;
    if (!(focus_start <= focus_end && focus_end <= cs::kKeyEnd) || !(theta >= 0.0) || !std::isfinite(theta))
        return CSTONE_ERR_INVALID_ARG;
    if (*n_leaves < 1 || *n_leaves > leaf_capacity || leaf_capacity >= cs::kMaxN) return CSTONE_ERR_INVALID_ARG;
    return cs::run_focus_rebalance(sorted_keys, n, n_crit, curve, focus_start, focus_end, theta, leaves, n_leaves,
                                   leaf_capacity, counts, max_iters, iters_done, ws, ws_bytes, stream);
}

CSTONE_API size_t cstone_focus_mac_workspace_bytes(void) { return cs::focus_mac_workspace_bytes(); }

CSTONE_API cstone_status cstone_focus_mac(const uint64_t* node_keys, size_t n_nodes, cstone_curve curve,
                                          uint64_t focus_start, uint64_t focus_end, double theta, uint8_t* fails,
                                          void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n_nodes > cs::kMaxN || (n_nodes && (!node_keys || !fails)) || !ws) return CSTONE_ERR_INVALID_ARG;
    if (curve != CSTONE_MORTON && curve != CSTONE_HILBERT) return CSTONE_ERR_INVALID_ARG;
    if (!(focus_start <= focus_end && focus_end <= cs::kKeyEnd) || !(theta >= 0.0) || !std::isfinite(theta))
        return CSTONE_ERR_INVALID_ARG;
    return cs::launch_focus_mac(node_keys, n_nodes, curve, focus_start, focus_end, theta, fails, ws, ws_bytes, stream);
}

CSTONE_API size_t cstone_sfc_partition_workspace_bytes(size_t n_leaves) {
    return cs::sfc_partition_workspace_bytes(n_leaves);
}

CSTONE_API cstone_status cstone_sfc_partition(const uint32_t* counts, size_t n_leaves, uint32_t n_ranks,
                                              uint32_t* bounds, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n_leaves < 1 || n_leaves >= cs::kMaxN || n_ranks == 0 || !counts || !bounds || !ws)
        return CSTONE_ERR_INVALID_ARG;
    return cs::launch_sfc_partition(counts, n_leaves, n_ranks, bounds, ws, ws_bytes, stream);
}

}  // extern "C"
