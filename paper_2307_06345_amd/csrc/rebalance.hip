// Leaf counts f (Eq. histogram) and the rebalance loop g = g3.g2.g1 (Sec. 4).
//
// The loop runs to a tree that the sorted keys alone determine, and tree.hip
// writes that tree at once, with the number of rounds. The rounds below run
// where their steps show: for fewer than L + 1 rounds (max_iters), where an
// array on the way exceeds the capacity (the last one that fitted is the
// result), and for an empty set.
//
// The loop keeps, next to the cornerstone array K, the position of every key
// of K in the sorted particle keys P (the lower bound that f computes). A
// leaf's count is the difference of two adjacent positions, and the combined
// count of 8 sibling leaves is the difference of the positions around them.
// Each round is two kernels:
//   round_kernel   g1 (decision), g2 (exclusive scan of O in one pass with a
//                  wave-wide decoupled look-back) and g3 (writing K'); copied
//                  leaves and the first child of a split keep their position,
//                  and every split leaf is appended to a list;
//   split_search   f for the next round: the 7 inner boundaries of every split
//                  leaf, searched inside that leaf's own range of P, spread
//                  over the whole GPU (one lane per search, or one wave with
//                  63 probes per step when the range is long).
// Rounds are enqueued ahead of the host's convergence check; a round that
// starts after convergence (or after a capacity overflow) exits at once, and a
// finalize kernel leaves the last complete round's array in place with its
// counts and its leaf count in device memory.
#include <algorithm>
#include <cstddef>
#include <cstring>
#include <memory>

#include "common.hpp"
#include "internal.hpp"

namespace cs {
namespace {

constexpr int kCountBlock = 256;
constexpr int kRBlock = 256;
constexpr int kRItems = 8;
constexpr int kRTile = kRBlock * kRItems;
constexpr uint32_t kMaxGrid = 2048;
constexpr uint32_t kSearchBlock = 256;


// ---- f as a standalone operation -----------------------------------------

__global__ __launch_bounds__(kCountBlock) void node_counts_kernel(const uint64_t* __restrict__ P, size_t n,
                                                                   const uint64_t* __restrict__ K, size_t nl,
                                                                   uint32_t* __restrict__ counts) {
    __shared__ uint32_t pos[kCountBlock + 1];
    const size_t base = static_cast<size_t>(blockIdx.x) * kCountBlock;
    const size_t i = base + threadIdx.x;
    if (i <= nl) pos[threadIdx.x] = static_cast<uint32_t>(lower_bound_u64(P, 0, n, K[i]));
    if (threadIdx.x == 0) {
        const size_t e = base + kCountBlock;
        if (e <= nl) pos[kCountBlock] = static_cast<uint32_t>(lower_bound_u64(P, 0, n, K[e]));
    }
    __syncthreads();
    if (i < nl) counts[i] = pos[threadIdx.x + 1] - pos[threadIdx.x];
}

// Positions of every key of K in P (start of the loop from a given array).
__global__ __launch_bounds__(kCountBlock) void positions_kernel(const uint64_t* __restrict__ P, size_t n,
                                                                 const uint64_t* __restrict__ K, size_t nl,
                                                                 uint32_t* __restrict__ pos) {
    const size_t i = static_cast<size_t>(blockIdx.x) * kCountBlock + threadIdx.x;
    if (i <= nl) pos[i] = static_cast<uint32_t>(lower_bound_u64(P, 0, n, K[i]));
}

__global__ __launch_bounds__(256) void loop_init_kernel(LoopState* st, uint64_t nl0, uint64_t* lb, size_t lb_words,
                                                        uint32_t* pos, uint32_t n, int root, uint64_t* K,
                                                        const uint32_t* input_flags) {
    const size_t t = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = t; i < lb_words; i += stride) lb[i] = 0;
    if (t < kMaxRounds) {
        st->changed[t] = 0;
        st->merged[t] = 0;
        st->over[t] = 0;
        st->counters[t][0] = 0;
        st->nsplit[t] = 0;
    }
    if (t <= kMaxRounds) st->nl[t] = t == 0 ? nl0 : 0;
    if (t == 0) {
        st->err = 0;
        st->input_flags = input_flags ? *input_flags : 0u;
        if (root) {  // the only one-leaf cornerstone array
            K[0] = 0;
            K[1] = kKeyEnd;
            pos[0] = 0;
            pos[1] = n;
        }
    }
}

// ---- one round: g1 + g2 + g3 -------------------------------------------------
//
// A tile is kRTile consecutive leaves. Their keys and positions, with kRHalo
// entries on either side (K_{i+1} and the 8-sibling checks reach up to 8
// entries away), are first read into LDS with coalesced loads; each thread
// then decides its kRItems consecutive leaves from LDS. When the tile's new
// entries fit in the same LDS (no split-heavy tile), they are assembled there
// and stored with coalesced writes; otherwise every thread writes its own.

constexpr int kRHalo = 8;
constexpr int kRSpan = kRTile + 2 * kRHalo;

__global__ __launch_bounds__(kRBlock, 4) void round_kernel(uint32_t n, uint32_t n_crit, const uint64_t* __restrict__ K,
                                                         const uint32_t* __restrict__ pos,
                                                         uint64_t* __restrict__ K_out, uint32_t* __restrict__ pos_out,
                                                         uint64_t* __restrict__ splits, uint32_t split_capacity,
                                                         LoopState* st, int round, uint64_t capacity, uint64_t* lb) {
    __shared__ uint32_t slot;
    __shared__ uint64_t scan_tmp[kRBlock / kWave];
    __shared__ uint64_t tile_prefix;
    __shared__ uint32_t split_base;
    __shared__ uint32_t any_change;
    __shared__ uint32_t any_merge;
    __shared__ uint64_t sK[kRSpan];  // K[base - kRHalo ...], then the tile's new entries
    __shared__ uint32_t sP[kRSpan];

    // Converged in an earlier round; or the last round only split, and no new
    // child can split (this round would copy every leaf: merges need 8 leaves
    // whose sum is at most n_crit, and no such group was made or changed)
    if (round > 0 && (st->changed[round - 1] == 0 || (st->merged[round - 1] == 0 && st->over[round - 1] == 0)))
        return;
    const uint64_t nl = st->nl[round];
    if (nl == 0 || nl > capacity) return;  // an earlier round overflowed
    const uint32_t tiles = static_cast<uint32_t>((nl + kRTile - 1) / kRTile);
    if (blockIdx.x >= tiles) return;  // more blocks than tiles: the rest stay off the counter
    const uint32_t tid = threadIdx.x;
    const uint32_t epoch = static_cast<uint32_t>(round + 1);
    if (tid == 0) {
        any_change = 0;
        any_merge = 0;
    }

    for (;;) {
        const uint32_t tile = take_tile(st->counters[round], &slot);
        if (tile >= tiles) break;
        const int64_t base = static_cast<int64_t>(tile) * kRTile;
        {  // K and positions of entries base-8 .. base+kRTile+7: all loads in flight at once (an index
           // outside 0 .. nl reads entry 0 or nl instead, and is not stored)
            constexpr int kLoads = (kRSpan + kRBlock - 1) / kRBlock;
            constexpr int kHalf = (kLoads + 1) / 2;  // two batches of loads keep the registers in budget
#pragma unroll
            for (int h = 0; h < kLoads; h += kHalf) {
                uint64_t lk[kHalf];
                uint32_t lp[kHalf];
#pragma unroll
                for (int q = 0; q < kHalf; ++q) {
                    const int64_t g = base - kRHalo + static_cast<int64_t>(tid) + (h + q) * kRBlock;
                    const int64_t c = min(max(g, int64_t{0}), static_cast<int64_t>(nl));
                    lk[q] = K[c];
                    lp[q] = pos[c];
                }
#pragma unroll
                for (int q = 0; q < kHalf; ++q) {
                    const int j = static_cast<int>(tid) + (h + q) * kRBlock;
                    const int64_t g = base - kRHalo + j;
                    if (h + q < kLoads && j < kRSpan && g >= 0 && g <= static_cast<int64_t>(nl)) {
                        sK[j] = lk[q];
                        sP[j] = lp[q];
                    }
                }
            }
        }
        __syncthreads();
        const uint32_t lfirst = tid * kRItems;  // first leaf of this thread, relative to base
        const uint64_t first = static_cast<uint64_t>(base) + lfirst;

        // g1: decision O_i for this thread's leaves
        uint32_t op[kRItems];
        uint64_t kk[kRItems + 1];
        uint32_t pp[kRItems];
        uint32_t osum = 0, nsplit = 0;
        bool changed = false, merged = false;
#pragma unroll
        for (int j = 0; j <= kRItems; ++j) kk[j] = sK[kRHalo + lfirst + j];
#pragma unroll
        for (int j = 0; j < kRItems; ++j) {
            const uint64_t i = first + j;
            const int li = kRHalo + static_cast<int>(lfirst) + j;
            uint32_t o = 0;
            pp[j] = sP[li];
            if (i < nl) {
                const uint64_t ki = kk[j];
                const uint64_t delta = kk[j + 1] - ki;
                const uint32_t cnt = sP[li + 1] - pp[j];
                o = 1;
                if (cnt > n_crit && delta > 1) {
                    o = 8;  // subdivide
                } else if (delta < kKeyEnd) {  // the root never merges
                    // place among its siblings, (K_i mod 8 delta) / delta; delta is a power of 8
                    const uint64_t js = (ki >> (63 - clz64(delta))) & 7u;
                    if (js >= 1 && i >= js && i - js + 8 <= nl && sK[li - js] + 8 * delta == sK[li - js + 8] &&
                        sP[li - js + 8] - sP[li - js] <= n_crit)
                        o = 0;  // 8 sibling leaves with at most n_crit particles: merge
                }
                changed |= (o != 1);
                merged |= (o == 0);
            }
            op[j] = o;
            osum += o;
            nsplit += o == 8;
        }
        if (merged) any_merge = 1;

        // g2: exclusive scan of O (low word) and of the split count (high word)
        uint64_t block_total;
        const uint64_t excl = block_exclusive_sum<uint64_t, kRBlock>(
            (static_cast<uint64_t>(nsplit) << 32) | osum, scan_tmp, &block_total);
        if (tid < kWave) {
            uint64_t prefix = 0;
            uint64_t* w = lb + tile;
            const uint64_t agg = block_total & 0xffffffffull;
            if (tile == 0) {
                if (tid == 0) st_agent(w, lb_word(kFlagInc, epoch, agg));
            } else {
                if (tid == 0) st_agent(w, lb_word(kFlagAgg, epoch, agg));
                prefix = lookback_wave<4>(lb, tile, epoch, &st->err);
                if (tid == 0) st_agent(w, lb_word(kFlagInc, epoch, prefix + agg));
            }
            if (tid == 0) {
                tile_prefix = prefix;
                const uint32_t sc = static_cast<uint32_t>(block_total >> 32);
                split_base = sc ? atomicAdd(&st->nsplit[round], sc) : 0u;
            }
        }
        if (changed) any_change = 1;
        __syncthreads();
        const uint64_t tp = tile_prefix;
        const uint32_t out_total = static_cast<uint32_t>(block_total);  // new entries of this tile
        const bool staged = out_total <= static_cast<uint32_t>(kRSpan);  // block-uniform

        // g3: K' (Eqs. rebalancecopy / rebalancesplit) and the known positions of K'
        uint32_t lo = static_cast<uint32_t>(excl);  // this thread's first new entry, relative to tp
        uint32_t s_at = split_base + static_cast<uint32_t>(excl >> 32);
#pragma unroll
        for (int j = 0; j < kRItems; ++j) {
            const uint64_t i = first + j;
            if (i < nl) {
                const uint64_t ki = kk[j];
                const uint64_t o_prime = tp + lo;
                if (op[j] == 1) {
                    if (staged) {
                        sK[lo] = ki;
                        sP[lo] = pp[j];
                    } else if (o_prime <= capacity) {
                        K_out[o_prime] = ki;
                        pos_out[o_prime] = pp[j];
                    }
                } else if (op[j] == 8) {
                    const uint64_t child = (kk[j + 1] - ki) >> 3;
                    if (staged) {
#pragma unroll
                        for (int c = 0; c < 8; ++c) sK[lo + c] = ki + c * child;
                        sP[lo] = pp[j];  // the other 7 come from the split search
                    } else if (o_prime + 7 <= capacity) {
#pragma unroll
                        for (int c = 0; c < 8; ++c) K_out[o_prime + c] = ki + c * child;
                        pos_out[o_prime] = pp[j];
                    }
                    if (o_prime + 7 <= capacity && s_at < split_capacity) splits[s_at] = i | (o_prime << 32);
                    ++s_at;
                }
            }
            lo += op[j];
        }
        if (staged) {  // the g3 writes above went to LDS (sK / sP were free after g1)
            __syncthreads();
            for (uint32_t j = tid; j < out_total; j += kRBlock) {
                if (tp + j <= capacity) {
                    K_out[tp + j] = sK[j];
                    pos_out[tp + j] = sP[j];  // split children 1..7 are overwritten by the split search
                }
            }
        }
        // the owner of the last leaf closes K' with 8^L
        if (first < nl && nl <= first + kRItems) {
            const uint64_t o_prime = tp + lo;
            st->nl[round + 1] = o_prime;
            if (o_prime <= capacity) {
                K_out[o_prime] = kKeyEnd;
                pos_out[o_prime] = n;
            }
        }
        __syncthreads();
    }
    if (tid == 0 && any_change) atomicOr(&st->changed[round], 1u);
    if (tid == 0 && any_merge) atomicOr(&st->merged[round], 1u);
}

// ---- f for the next round: positions of the inner child boundaries ----------

// Child boundaries of the listed splits: positions in P of the 7 inner
// boundaries of each split leaf. With at most one search per wave (early
// rounds: few splits, long ranges) every search gets a whole wave (63 probes
// per step). Otherwise a wave takes 8 splits, 8 lanes each: a range of at most
// kSmallRange keys is read by its 8 lanes at once (16 keys each, independent
// loads) and every boundary is the count of the range's keys below it; a
// longer range is searched by lanes 1..7, one binary search each, in parallel.
constexpr uint32_t kSmallRange = 128;

__global__ __launch_bounds__(kSearchBlock) void split_search_kernel(const uint64_t* __restrict__ P, uint32_t n,
                                                                     const uint64_t* __restrict__ K,
                                                                     const uint32_t* __restrict__ pos,
                                                                     uint32_t* __restrict__ pos_out,
                                                                     const uint64_t* __restrict__ splits,
                                                                     uint32_t split_capacity, LoopState* st,
                                                                     int round, uint64_t capacity, uint32_t n_crit) {
    const uint64_t nl = st->nl[round];
    if (st->nl[round + 1] > capacity || nl > capacity) return;  // overflowed round: K' is discarded
    const uint32_t listed = min(st->nsplit[round], split_capacity);
    const uint32_t lane = lane_id();
    const uint32_t t = lane & 7u;  // child boundary t (1..7) of the group's split
    const uint32_t waves = gridDim.x * (kSearchBlock / kWave);
    const uint32_t wave = blockIdx.x * (kSearchBlock / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (static_cast<uint64_t>(listed) * 7u <= waves) {  // one search per wave (wave-uniform branch)
        for (uint32_t w = wave; w < listed * 7u; w += waves) {
            const uint64_t e = splits[w / 7u];
            const uint32_t c = w % 7u + 1u;
            const uint64_t i = e & 0xffffffffull;
            const uint64_t ki = K[i];
            const uint64_t key = ki + c * ((K[i + 1] - ki) >> 3);
            const uint32_t hi = min(pos[i + 1], n);
            const uint32_t lo = min(pos[i], hi);
            const uint32_t dst = static_cast<uint32_t>(e >> 32) + c;
            const uint32_t at = wave_lower_bound(P, lo, hi, key);
            if (lane == 0 && dst <= capacity) pos_out[dst] = at;
        }
        // the children's counts are not gathered here: let the next round run
        if (listed != 0 && wave == 0 && lane == 0) atomicOr(&st->over[round], 1u);
        return;
    }
    bool wave_over = false;  // one flag write per wave, not per group of splits
    for (uint32_t base = wave * 8u; base < listed; base += waves * 8u) {
        const uint32_t sidx = base + (lane >> 3);
        bool valid = sidx < listed;
        uint32_t lo = 0, hi = 0, dst0 = 0;
        uint64_t ki = 0, step = 0;
        if (valid) {
            const uint64_t e = splits[sidx];
            const uint64_t i = e & 0xffffffffull;
            ki = K[i];
            step = (K[i + 1] - ki) >> 3;
            hi = min(pos[i + 1], n);  // positions never exceed n; the clamps guard memory all the same
            lo = min(pos[i], hi);
            dst0 = static_cast<uint32_t>(e >> 32);
        }
        valid = valid && static_cast<uint64_t>(dst0) + 7u <= capacity;  // always true for a listed split
        const uint64_t key = ki + t * step;
        const bool small = valid && hi - lo <= kSmallRange;
        // short ranges: every lane of the group counts its 16 keys below each boundary
        uint32_t cnt[7] = {0, 0, 0, 0, 0, 0, 0};
        if (small) {
            uint64_t kq[kSmallRange / 8];
#pragma unroll
            for (uint32_t m = 0; m < kSmallRange / 8; ++m) {
                const uint32_t q = lo + t + 8u * m;
                kq[m] = q < hi ? P[q] : ~0ull;
            }
#pragma unroll
            for (uint32_t m = 0; m < kSmallRange / 8; ++m)
#pragma unroll
                for (uint32_t c = 0; c < 7; ++c) cnt[c] += kq[m] < ki + (c + 1) * step ? 1u : 0u;
        }
#pragma unroll
        for (uint32_t c = 0; c < 7; ++c) {  // sums over the group's 8 lanes (all lanes take part)
            cnt[c] += __shfl_xor(cnt[c], 1, kWave);
            cnt[c] += __shfl_xor(cnt[c], 2, kWave);
            cnt[c] += __shfl_xor(cnt[c], 4, kWave);
        }
        uint32_t b = lo;  // this lane's boundary (lane 0 of a group: the range's start)
        if (small && t != 0) {
            uint32_t below = 0;
#pragma unroll
            for (uint32_t c = 0; c < 7; ++c) below = c + 1 == t ? cnt[c] : below;
            b = lo + below;
            pos_out[dst0 + t] = b;
        }
        if (valid && !small && t != 0) {
            b = static_cast<uint32_t>(lower_bound_u64(P, lo, hi, key));
            pos_out[dst0 + t] = b;
        }
        // does a new child hold more than n_crit (and could split: span above 1)?
        const uint32_t before = __shfl(b, static_cast<int>(lane) - 1, kWave);  // lane 0's value is not used
        const bool over = valid && t != 0 && step > 1 && (b - before > n_crit || (t == 7 && hi - b > n_crit));
        wave_over = wave_over || __ballot(over) != 0ull;
    }
    if (wave_over && lane == 0) atomicOr(&st->over[round], 1u);
}

// ---- pick the array of the last complete round --------------------------------

struct Outcome {
    uint32_t last;     // rounds completed (the array after them is the result)
    uint32_t code;     // 0 running, 1 converged, 2 capacity exceeded
    uint64_t nl;       // leaves of that array
    uint32_t buf;      // which of the two arrays holds it (the parity of the rounds that ran)
};

// settle_last: the last enqueued round may settle too; its check round is then
// counted without having been enqueued (the caller allows one more round).
__device__ __forceinline__ Outcome loop_outcome(const LoopState* st, uint32_t enqueued, uint64_t capacity,
                                                bool settle = true, bool settle_last = false) {
    for (uint32_t q = 0; q < enqueued; ++q) {
        if (st->nl[q + 1] > capacity) return {q, 2u, st->nl[q], q & 1u};
        if (st->changed[q] == 0) return {q + 1, 1u, st->nl[q + 1], (q + 1) & 1u};  // round q copied every leaf
        // round q + 1 would copy every leaf: it does not run, and counts
        if (settle && (q + 1 < enqueued || settle_last) && st->merged[q] == 0 && st->over[q] == 0)
            return {q + 2, 1u, st->nl[q + 1], (q + 1) & 1u};
    }
    return {enqueued, 0u, st->nl[enqueued], enqueued & 1u};
}

// Leaves the result array in K[0] (copied from K[1] when an odd number of
// rounds completed), writes its counts, and publishes its leaf count.
__global__ __launch_bounds__(256) void finalize_kernel(LoopState* st, uint32_t enqueued, uint64_t capacity,
                                                       uint64_t* __restrict__ K0, const uint64_t* __restrict__ K1,
                                                       const uint32_t* __restrict__ pos0,
                                                       const uint32_t* __restrict__ pos1,
                                                       uint32_t* __restrict__ counts, uint32_t settle_last) {
    const Outcome o = loop_outcome(st, enqueued, capacity, true, settle_last != 0);
    const uint64_t nl = o.nl <= capacity ? o.nl : 0;
    const bool odd = o.buf != 0;
    const uint32_t* pos = odd ? pos1 : pos0;
    const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i <= nl; i += stride) {
        if (odd) K0[i] = K1[i];
        if (counts && i < nl) counts[i] = pos[i + 1] - pos[i];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->final_nl = nl;
        st->final_last = o.last;
        st->final_code = o.code;
    }
}

struct RebalanceWs {
    uint64_t* K_alt;
    uint32_t* pos[2];
    uint64_t* splits;
    uint32_t split_capacity;
    LoopState* st;
    uint64_t* lb;
    size_t lb_words;
    size_t bytes;
};

RebalanceWs carve_rebalance(void* ws, size_t n, uint32_t n_crit, size_t cap) {
    Carve c(ws);
    RebalanceWs r{};
    r.K_alt = c.take<uint64_t>(cap + 1);
    r.pos[0] = c.take<uint32_t>(cap + 1);
    r.pos[1] = c.take<uint32_t>(cap + 1);
    // leaves that split in one round hold > n_crit particles each and are disjoint
    const size_t max_splits = std::min<size_t>(cap, n / (static_cast<size_t>(n_crit) + 1)) + 1;
    r.split_capacity = static_cast<uint32_t>(max_splits);
    r.splits = c.take<uint64_t>(max_splits);
    r.st = c.take<LoopState>(1);
    r.lb_words = (cap + kRTile - 1) / kRTile + 1;
    r.lb = c.take<uint64_t>(r.lb_words);
    r.bytes = c.off;
    return r;
}

uint32_t grid_1d(size_t items, int block) { return static_cast<uint32_t>((items + block - 1) / block); }

uint32_t clamp_grid(size_t blocks) {
    return static_cast<uint32_t>(std::max<size_t>(1, std::min<size_t>(blocks, kMaxGrid)));
}

// one wave per search while searches are few
uint32_t search_grid(size_t splits) { return clamp_grid(grid_1d((splits + 7) / 8, kSearchBlock / kWave)); }  // 8 splits a wave

}  // namespace

cstone_status launch_node_counts(const uint64_t* sorted_keys, size_t n, const uint64_t* leaves, size_t n_leaves,
                                 uint32_t* counts, hipStream_t stream) {
    if (n_leaves == 0) return CSTONE_OK;
    hipLaunchKernelGGL(node_counts_kernel, dim3(grid_1d(n_leaves, kCountBlock)), dim3(kCountBlock), 0, stream,
                       sorted_keys, n, leaves, n_leaves, counts);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

size_t rebalance_rounds_bytes(size_t n, uint32_t n_crit, size_t leaf_capacity) {
    return carve_rebalance(nullptr, n, n_crit ? n_crit : 1, leaf_capacity).bytes;
}

size_t rebalance_workspace_bytes(size_t n, uint32_t n_crit, size_t leaf_capacity) {
    return std::max(rebalance_rounds_bytes(n, n_crit, leaf_capacity),
                    leaf_capacity ? tree_workspace_bytes(n, n_crit ? n_crit : 1, leaf_capacity) : 0);
}

cstone_status RebalanceLoop::begin(const uint64_t* P, size_t n, uint32_t n_crit, uint64_t* leaves, size_t nl0,
                                   size_t cap, uint32_t* counts, uint32_t max_iters, void* ws, size_t ws_bytes,
                                   hipStream_t stream, const uint32_t* input_flags) {
    RebalanceWs w = carve_rebalance(ws, n, n_crit, cap);
    if (ws_bytes < w.bytes) return CSTONE_ERR_INVALID_ARG;
    if (nl0 < 1 || nl0 > cap || cap >= 0xffffffffull) return CSTONE_ERR_INVALID_ARG;
    P_ = P;
    n_ = n;
    n_crit_ = n_crit;
    leaves_ = leaves;
    nl0_ = nl0;
    cap_ = cap;
    counts_ = counts;
    max_iters_ = std::min<uint32_t>(max_iters ? max_iters : kL + 1, kMaxRounds);
    enqueued_ = 0;
    stream_ = stream;
    ws_ = ws;
    st_ = w.st;
    root_ = nl0 == 1;
    const size_t init_items = std::max<size_t>(w.lb_words, kMaxRounds + 1);
    hipLaunchKernelGGL(loop_init_kernel, dim3(clamp_grid(grid_1d(init_items, 256))), dim3(256), 0, stream, w.st,
                       static_cast<uint64_t>(nl0), w.lb, w.lb_words, w.pos[0], static_cast<uint32_t>(n),
                       root_ ? 1 : 0, leaves, input_flags);
    if (!root_)
        hipLaunchKernelGGL(positions_kernel, dim3(grid_1d(nl0 + 1, kCountBlock)), dim3(kCountBlock), 0, stream, P, n,
                           leaves, nl0, w.pos[0]);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

cstone_status RebalanceLoop::enqueue(uint32_t rounds) {
    RebalanceWs w = carve_rebalance(ws_, n_, n_crit_, cap_);
    if (rounds == 0) {
        rounds = 2;
        if (root_) {  // from the root: about log8(n / (n_crit + 1)) + 2 rounds
            double ratio = static_cast<double>(n_) / (static_cast<double>(n_crit_) + 1.0);
            while (ratio > 1.0) {
                ratio /= 8.0;
                ++rounds;
            }
        }
    }
    rounds = std::min(rounds, max_iters_ - enqueued_);
    uint64_t* bufK[2] = {leaves_, w.K_alt};
    for (uint32_t q = enqueued_; q < enqueued_ + rounds; ++q) {
        // leaves entering round q: at most nl0 * 8^q and the capacity
        double bound = static_cast<double>(nl0_);
        for (uint32_t e = 0; e < q && bound < static_cast<double>(cap_); ++e) bound *= 8.0;
        const size_t rows = static_cast<size_t>(std::min<double>(bound, static_cast<double>(cap_)));
        hipLaunchKernelGGL(round_kernel, dim3(clamp_grid(grid_1d(rows, kRTile))), dim3(kRBlock), 0, stream_,
                           static_cast<uint32_t>(n_), n_crit_, bufK[q & 1], w.pos[q & 1], bufK[(q + 1) & 1],
                           w.pos[(q + 1) & 1], w.splits, w.split_capacity, w.st, static_cast<int>(q),
                           static_cast<uint64_t>(cap_), w.lb);
        const size_t max_splits = std::min<size_t>(rows, w.split_capacity);
        hipLaunchKernelGGL(split_search_kernel, dim3(search_grid(max_splits)),
                           dim3(kSearchBlock), 0, stream_, P_, static_cast<uint32_t>(n_), bufK[q & 1], w.pos[q & 1],
                           w.pos[(q + 1) & 1], w.splits, w.split_capacity, w.st, static_cast<int>(q),
                           static_cast<uint64_t>(cap_), n_crit_);
    }
    enqueued_ += rounds;
    hipLaunchKernelGGL(finalize_kernel, dim3(clamp_grid(grid_1d(cap_ + 1, 256))), dim3(256), 0, stream_, w.st,
                       enqueued_, static_cast<uint64_t>(cap_), leaves_, w.K_alt, w.pos[0], w.pos[1], counts_,
                       enqueued_ < max_iters_ ? 1u : 0u);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

const uint64_t* RebalanceLoop::device_leaf_count() const { return &st_->final_nl; }

cstone_status RebalanceLoop::wait(bool* finished) {
    LoopHeader host;  // the loop state without its tile counters
    CS_HIP(hipMemcpyAsync(&host, static_cast<const LoopHeader*>(st_), sizeof(LoopHeader), hipMemcpyDeviceToHost,
                          stream_));
    CS_HIP(hipStreamSynchronize(stream_));
    input_flags = host.input_flags;
    rounds = host.final_last;
    *finished = true;
    if (host.err) {
        status = CSTONE_ERR_DEVICE;
        return status;
    }
    if (host.final_code == 2) {
        n_leaves = host.nl[host.final_last + 1];  // what the failing round needed
        status = CSTONE_ERR_CAPACITY;
        return status;
    }
    n_leaves = host.final_nl;
    if (host.final_code == 1) {
        status = CSTONE_OK;
    } else if (enqueued_ >= max_iters_) {
        status = CSTONE_ERR_NOT_CONVERGED;
    } else {
        status = CSTONE_OK;
        *finished = false;
    }
    return status;
}

namespace {

// Whether the tree straight from the keys is the faster one: it reads all keys
// and compares the arrays, whatever there is to change, while a round goes by the
// leaves alone. From the root it always is (2^17 .. 2^27 keys, N_crit 16 .. 1 M:
// 0.2 to 1 of the rounds' time, but 1.5 for uniform ones at 2^27 and N_crit from
// 1000 on). From another array, direct against rounds in us, for a tree that stays
// as it is / changes a little / is far off: 2^18 keys, N_crit 16: 79 / 87 / 86
// against 96 / 106 / 110; 2^20: 113 / 115 / 116 against 87 / 100 / 102; 2^24, N_crit
// 256: 138 / 139 / 139 against 111 / 110 / 112; 2^27: 596 / 597 / 602 against 326 /
// 325 / 364, and N_crit 10^5 218 against 87. With many leaves the rounds' searches
// cost as much: 2^27, N_crit 16, a leaf per 8 keys: 1013 / 1023 / 1072 against 934 /
// 1157 / 4311.
constexpr size_t kDirectKeys = size_t{1} << 18;
constexpr size_t kDirectManyKeys = size_t{1} << 24;
bool direct_pays(size_t n, size_t nl0) {
    return nl0 == 1 || n <= kDirectKeys || (n >= kDirectManyKeys && nl0 >= n / 8);
}

}  // namespace

cstone_status run_rebalance(const uint64_t* P, size_t n, uint32_t n_crit, uint64_t* leaves, size_t* n_leaves,
                            size_t cap, uint32_t* counts, uint32_t max_iters, uint32_t* iters_done, void* ws,
                            size_t ws_bytes, hipStream_t stream) {
    cstone_status s;
    if (ws_bytes < rebalance_rounds_bytes(n, n_crit, cap)) return CSTONE_ERR_INVALID_ARG;  // what both ways need
    if (tree_possible(n, max_iters) && direct_pays(n, *n_leaves)) {
        TreePass tree;
        if (tree.run(P, n, n_crit, leaves, *n_leaves, cap, counts, nullptr, nullptr, nullptr, ws, ws_bytes, nullptr,
                     nullptr, nullptr, stream)) {
            bool fits = false;
            if ((s = tree.wait(&fits)) != CSTONE_OK) return s;
            if (fits) {
                *n_leaves = tree.n_leaves;
                if (iters_done) *iters_done = tree.rounds;
                return CSTONE_OK;
            }
        }
    }
    RebalanceLoop loop;
    s = loop.begin(P, n, n_crit, leaves, *n_leaves, cap, counts, max_iters, ws, ws_bytes, stream, nullptr);
    if (s != CSTONE_OK) return s;
    bool finished = false;
    uint32_t batch = 0;
    while (!finished) {
        if ((s = loop.enqueue(batch)) != CSTONE_OK) return s;
        loop.wait(&finished);
        batch = 4;
    }
    if (loop.status == CSTONE_ERR_DEVICE) return loop.status;
    *n_leaves = loop.n_leaves;
    if (iters_done) *iters_done = loop.rounds;
    return loop.status;
}

}  // namespace cs
