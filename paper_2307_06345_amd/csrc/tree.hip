// The balanced tree straight from the sorted keys, and its links.
//
// The fixed point of f and g (Sec. 4) is the tree whose internal nodes are the
// octants that hold more than N = N_crit particles (above level L), whatever
// array the rounds start from. In the sorted keys P an octant is a run, so it
// holds more than N particles exactly if some P[j] and P[j + N] both lie in it.
// With common(a, b) the number of leading octal digits two keys share, the
// internal nodes whose first particle is j have the levels
//   common(P[j - 1], P[j]) + 1 .. min(L - 1, common(P[j], P[j + N]))
// (from level 0 for j = 0, none if j + N >= n). So three launches replace the
// rounds, which read and wrote the array once per level, and the link:
//   mark   one pass over P lists the internal nodes in preorder (by first
//          particle, then level), tile by tile, and counts them per level;
//   scan   of the tiles' counts, per level and over all levels;
//   write  every internal node finds where its 8 children start in P. Children
//          with at most N particles are leaves. Internal node r (in preorder)
//          of level l has its children at LO[l + 1] + 8 r .. + 7 of NK and CO;
//          a leaf is preceded in K by 7 leaves for every internal node that
//          lies wholly before it and by as many as its path digits add up to.
// The work after the first pass goes with the internal nodes, a seventh of the
// leaves. Tiles are independent in every launch: a decoupled look-back instead
// of the scan (one pass over P writing K) took 208 us against 32 + 7 + 48 us
// for 2^24 keys, at 33-80 ns per tile of polling between the XCDs.
//
// The rounds' count is known too: every round moves a leaf by one level at
// most, and from the root it takes depth rounds and the check round; from
// another array, 1 + the largest level difference between two overlapping
// leaves of the two arrays.
//
// The tree focused on a range of the curve (Sec. 7) is the same with fewer
// internal nodes, those that fail the MAC too. A node that fails has only
// ancestors that fail (they are larger and no farther), so the mark launch ends
// each particle's levels before the first that passes, and the write launch
// looks for their children in the list too. With few internal nodes the
// particles' bytes are neither kept nor read.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "focus.hpp"
#include "internal.hpp"
#include "overlap.hpp"

namespace cs {
namespace {

constexpr int kMarkBlock = 512;
constexpr int kMarkItems = 8;
constexpr uint32_t kTreeTile = kMarkBlock * kMarkItems;  // particles per tile of all three launches
constexpr int kMarkWaves = kMarkBlock / kWave;
// N_crit up to which the write launch goes by the particles' bytes; above it the
// bytes of 8 N particles are too many round trips, and all nodes are searched.
// Builds of 2^24 Plummer particles by bytes / by searches: N_crit 200 742 / 733 us,
// 256 741 / 730, 500 750 / 727, 1000 751 / 717; uniform 2^20, 256 169 / 161. (Both
// take the same at 100.)
constexpr uint32_t kByteMaxCrit = 128;
constexpr size_t kBytesPad = 192;  // a byte after the last particle's, and what the last groups read past it

// Leading octal digits two keys share, 0 .. 21. Keys are below 2^63, so the bits
// they share are one less than the leading zeros of their difference; / 3 as
// * 43 / 128 is exact below 64.
__device__ __forceinline__ uint32_t common_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    const uint32_t z = x ? static_cast<uint32_t>(__builtin_clzll(x)) : 64u;
    return (z * 43u - 43u) >> 7;
}

// Sum of the octal digits of a placeholder-bit key (without the placeholder).
__device__ __forceinline__ uint32_t digit_sum(uint64_t node) {
    const uint64_t k = node ^ (1ull << (63 - clz64(node)));
    return static_cast<uint32_t>(__popcll(k & 0x1249249249249249ull) + 2 * __popcll(k & 0x2492492492492492ull) +
                                 4 * __popcll(k & 0x4924924924924924ull));
}

// Slots for the internal nodes of a tile, by what balanced trees hold (0.5 to
// 0.6 of T / (N + 1)); a tile with more of them takes a run of shared slots. (A
// run reserved by every tile, one atomic each on one word and the wait for it,
// took 160 of 420 us for 2^27 keys.)
__host__ __device__ inline uint32_t tile_slots(uint32_t n_crit) {
    return kTreeTile / (n_crit < kTreeTile ? n_crit + 1u : kTreeTile) + 16u;
}
__host__ __device__ inline uint64_t tree_tiles_of(uint64_t n) { return (n + kTreeTile - 1) / kTreeTile; }

// Data-parallel moves within and across the rows of 16 lanes (no LDS round trips).
__device__ __forceinline__ uint32_t wave_add_up(uint32_t v) {  // inclusive sum over the lanes up to this one
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x111, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x112, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x114, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x118, 0xf, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));
    return v;
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, false));
}
// Over the 8 lanes of a group: lanes 1 apart, 2 apart, then mirrored.
__device__ __forceinline__ uint32_t group_min(uint32_t v) {
    v = min(v, dpp<0xb1>(v));   // quad_perm 1, 0, 3, 2
    v = min(v, dpp<0x4e>(v));   // quad_perm 2, 3, 0, 1
    return min(v, dpp<0x141>(v));  // row_half_mirror
}
__device__ __forceinline__ uint32_t group_or(uint32_t v) {
    v |= dpp<0xb1>(v);
    v |= dpp<0x4e>(v);
    return v | dpp<0x141>(v);
}
__device__ __forceinline__ uint32_t group_add_up(uint32_t v, uint32_t c) {  // inclusive sum; c: place in the group
    uint32_t o = dpp<0x111>(v);  // row_shr 1, 2, 4
    v += c >= 1 ? o : 0u;
    o = dpp<0x112>(v);
    v += c >= 2 ? o : 0u;
    o = dpp<0x114>(v);
    return v + (c >= 4 ? o : 0u);
}
__device__ __forceinline__ uint64_t from_lane_before(uint64_t v) {  // lane 0 gets 0
    const uint32_t lo = static_cast<uint32_t>(v), hi = static_cast<uint32_t>(v >> 32);
    return (static_cast<uint64_t>(static_cast<uint32_t>(
                __builtin_amdgcn_update_dpp(0, static_cast<int>(hi), 0x138, 0xf, 0xf, false)))
            << 32) |
           static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), 0x138, 0xf, 0xf, false));
}

struct NoFocus {};
template <bool FOCUS>
using FocusPart = std::conditional_t<FOCUS, FocusSmem, NoFocus>;

struct MarkSmem {
    uint32_t list[kTreeTile];     // per wave: its particles that start internal nodes: place | u << 12 | e << 17
    uint32_t level[kTreeLevels];  // internal nodes of the tile per level
    uint32_t sum[kMarkWaves];
    uint32_t slot;
};

// ---- mark --------------------------------------------------------------------
//
// Besides the list, a byte per particle is kept for the write launch: u_j =
// common(P[j - 1], P[j]) + 1, the level below which j starts a node of its own;
// 0 for a set's first particle and after the last one of all.
//
// Bound: reading P, 8 B a particle (P[j + N] and P[j - 1] are the tile's own
// cache lines, or the next one's, for N_crit in the hundreds), about 40
// instructions a key. A wave takes 512 consecutive particles, so that their
// starts (one particle in 100 at N_crit 64) are gathered in order by ballots
// without a barrier; only they are expanded. From N_crit 512 on most waves look
// at three keys instead (2^27 keys: 305 us for any N_crit before, 160 at 2000 and
// 64 at 10^6).
// One wave's 512 particles from place wbase of the tile on: their bytes, and
// the list of those that start internal nodes (in order; returns how many).
// FULL: every key that is read exists; otherwise keys past the end read the
// last key and are masked. BYTES: the particles' bytes are kept. Where they are
// not, and N spans the wave's particles, most waves need not read them: with g
// the digits that all keys from the one before the first to the last share, and h
// those of the last and P[first + N], every particle j of the wave has
// common(P[j - 1], P[j]) >= g and common(P[j], P[j + N]) <= h, so none starts an
// internal node unless h > g.
template <bool FULL, bool BYTES>
__device__ __forceinline__ uint32_t mark_wave(const uint64_t* __restrict__ Ps, uint32_t base, uint32_t wbase, uint32_t n,
                                              uint32_t N, uint32_t max_level, uint8_t* __restrict__ below,
                                              uint32_t* mylist) {
    const uint32_t lane = lane_id();
    const uint32_t first = base + wbase;  // wave-uniform
    if (!FULL && first >= n) return 0;
    const uint64_t last = n - 1;
    if constexpr (!BYTES) {
        if (static_cast<uint64_t>(first) + N >= n) return 0;
        if (first && N >= kMarkItems * kWave) {
            const uint64_t end = Ps[first + kMarkItems * kWave - 1];
            if (min(common_digits(end, Ps[first + N]), max_level) <= common_digits(Ps[first - 1], end)) return 0;
        }
    }
    uint64_t edge = Ps[first ? first - 1 : 0];
    uint64_t a[kMarkItems], b[kMarkItems];
    const uint64_t* pa = Ps + first + lane;
    const uint64_t* pb = pa + N;
#pragma unroll
    for (int it = 0; it < kMarkItems; ++it) {
        if constexpr (FULL) {
            a[it] = pa[it * kWave];
            b[it] = pb[it * kWave];
        } else {
            const uint64_t j = static_cast<uint64_t>(first) + it * kWave + lane;
            a[it] = Ps[min(j, last)];
            b[it] = Ps[min(j + N, last)];
        }
    }
    uint8_t* out = below + first + lane;
    uint32_t starts = 0;  // wave-uniform
#pragma unroll
    for (int it = 0; it < kMarkItems; ++it) {
        // the key before this lane's: the lane before holds it, lane 0 takes the run's edge
        const uint64_t shifted = from_lane_before(a[it]);
        const uint64_t before = lane ? shifted : edge;
        edge = (static_cast<uint64_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(a[it] >> 32), kWave - 1)) << 32) |
               static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(a[it]), kWave - 1));
        uint32_t u = common_digits(before, a[it]) + 1u;
        if (it == 0 && first == 0 && lane == 0) u = 0;
        const uint32_t e = min(common_digits(a[it], b[it]), max_level) + 1u;
        bool start = e > u;
        if constexpr (FULL) {
            if constexpr (BYTES) out[it * kWave] = static_cast<uint8_t>(u);
        } else {
            const uint64_t j = static_cast<uint64_t>(first) + it * kWave + lane;
            if (BYTES && j < n) out[it * kWave] = static_cast<uint8_t>(u);
            start = start && j + N < n;
        }
        const uint64_t m = __ballot(start);
        if (m) {  // wave-uniform
            if (start) mylist[starts + lanes_below(m)] = (wbase + it * kWave + lane) | (u << 12) | (e << 17);
            starts += static_cast<uint32_t>(__popcll(m));
        }
    }
    return starts;
}

// FOCUS (one set): a tile has no slots of its own, since most hold none of the
// few internal nodes; those that do take a run of the shared ones. KEEP: whether
// the bytes are kept (a batch's sets may differ in it; the branch costs 1 us in 33
// for 2^24 particles).
enum class Keep { kNone, kBytes, kByCrit };
template <bool BATCH, bool FOCUS, Keep KEEP>
__global__ __launch_bounds__(kMarkBlock) void tree_mark_kernel(const uint64_t* __restrict__ P, TreeOne one,
                                                               const BatchSet* __restrict__ sets,
                                                               const uint32_t* __restrict__ tile_set, uint32_t n_tiles,
                                                               uint32_t max_level, uint8_t* __restrict__ below,
                                                               uint64_t* __restrict__ inodes,
                                                               uint32_t* __restrict__ ipos,
                                                               uint64_t* __restrict__ tile_off,
                                                               uint32_t* __restrict__ rows, uint32_t* reserved,
                                                               FocusSpec focus) {
    __shared__ MarkSmem sm;
    __shared__ FocusPart<FOCUS> fsm;
    const uint32_t tid = threadIdx.x, lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t gtile = blockIdx.x;
    uint32_t tile = gtile;
    TreeOne o = one;
    if constexpr (BATCH) {
        const uint32_t s = tile_set[gtile];
        const BatchSet& S = sets[s];
        tile = gtile - S.tree_tile0;
        o = {S.part_off, S.n, S.n_crit, S.leaf_off, S.cap, S.inode_off};
        reserved += s;
        below += S.part_off;
    }
    const uint32_t N = o.n_crit, n = o.n;
    const uint64_t* Ps = P + o.first;
    const uint32_t base = tile * kTreeTile;
    const uint32_t wbase = wave * kMarkItems * kWave;  // the wave's first place
    if (tid < kTreeLevels) sm.level[tid] = 0;
    if (KEEP != Keep::kNone && tid == 0) {  // where a set ends, for those that go by their bytes
        if (tile == 0) below[0] = 0;
        if (gtile + 1 == n_tiles) below[n] = 0;
    }
    const bool full = static_cast<uint64_t>(base) + kTreeTile + N <= n;  // block-uniform: every key exists
    uint32_t* mylist = sm.list + wbase;
    const auto wave_starts = [&](auto bytes) {
        return full ? mark_wave<true, bytes.value>(Ps, base, wbase, n, N, max_level, below, mylist)
                    : mark_wave<false, bytes.value>(Ps, base, wbase, n, N, max_level, below, mylist);
    };
    uint32_t starts;
    if constexpr (KEEP != Keep::kByCrit)
        starts = wave_starts(std::bool_constant<KEEP == Keep::kBytes>{});
    else
        starts = N <= kByteMaxCrit ? wave_starts(std::true_type{}) : wave_starts(std::false_type{});
    if constexpr (FOCUS) {
        if (__syncthreads_or(static_cast<int>(starts))) {  // block-uniform; sm.level is cleared
            focus_fill(focus, fsm);
            __syncthreads();
            for (uint32_t r = lane; r < starts; r += kWave) {  // (the wave's own places)
                const uint32_t x = mylist[r], u = (x >> 12) & 31u, e = x >> 17;
                const uint64_t key = Ps[base + (x & 0xfffu)];
                uint32_t l = u;
                while (l < e && node_fails(key, l, focus, fsm)) ++l;
                mylist[r] = (x & 0x1ffffu) | (l << 17);
            }
        }
    } else {
        __syncthreads();  // sm.level is cleared
    }
    // internal nodes of the wave, per level and in all
    uint32_t mine = 0;
    for (uint32_t r = lane; r < starts; r += kWave) {
        const uint32_t x = mylist[r], u = (x >> 12) & 31u, e = x >> 17;
        mine += e - u;
        for (uint32_t l = u; l < e; ++l) atomicAdd(&sm.level[l], 1u);
    }
    mine = wave_add_up(mine);
    if (lane == kWave - 1) sm.sum[wave] = mine;
    __syncthreads();
    uint32_t total = 0, ahead = 0;
#pragma unroll
    for (int v = 0; v < kMarkWaves; ++v) {
        const uint32_t c = sm.sum[v];
        if (v < static_cast<int>(wave)) ahead += c;
        total += c;
    }
    if (tid < kTreeRows) rows[static_cast<size_t>(tid) * n_tiles + gtile] = tid < kTreeLevels ? sm.level[tid] : total;
    if (total == 0) return;  // block-uniform
    // the tile's own slots, or a run of the set's shared ones after them
    const uint32_t own = FOCUS ? 0u : tile_slots(N);
    const uint64_t shared = static_cast<uint64_t>(own) * tree_tiles_of(n);
    const uint64_t slots = shared + (o.cap - 1) / 7 + 1;
    uint64_t at = static_cast<uint64_t>(tile) * own;
    if (total > own) {  // block-uniform
        if (tid == 0) sm.slot = atomicAdd(reserved, total);
        __syncthreads();
        at = shared + sm.slot;
    }
    if (tid == 0) tile_off[gtile] = at;
    at += ahead;
    for (uint32_t r0 = 0; r0 < starts; r0 += kWave) {
        const uint32_t r = r0 + lane;
        const bool in = r < starts;
        const uint32_t x = in ? mylist[r] : 0u, u = (x >> 12) & 31u, e = x >> 17;
        const uint32_t m = e - u;
        const uint32_t inc = wave_add_up(m);
        uint64_t p = at + (inc - m);
        at += __builtin_amdgcn_readlane(inc, kWave - 1);
        if (in) {
            const uint32_t j = base + (x & 0xfffu);
            const uint64_t key = Ps[j];
            for (uint32_t l = u; l < e; ++l, ++p) {
                if (p < slots) {  // always, if the tree is within the capacity; others are not written at all
                    inodes[o.inode_off + p] = (1ull << (3 * l)) | (key >> (3 * (kL - l)));
                    ipos[o.inode_off + p] = j;
                }
            }
        }
    }
}

// ---- scan --------------------------------------------------------------------

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
// Sets of at most this many tiles are summed by the write blocks themselves, which
// spares small builds a launch (builds of 2^15 .. 2^20 particles by 16, 64 and 128:
// within 2 us of each other, by turns).
constexpr uint32_t kDirectTiles = 64;

// Block (row, set): exclusive scan of one row of counts over the set's tiles, in place, and its total.
template <bool BATCH>
__global__ __launch_bounds__(kScanBlock) void tree_scan_kernel(const BatchSet* __restrict__ sets, uint32_t n_tiles,
                                                               uint32_t* __restrict__ rows,
                                                               uint32_t* __restrict__ totals) {
    __shared__ uint32_t tmp[kScanBlock / kWave];
    const uint32_t tid = threadIdx.x, s = blockIdx.y, l = blockIdx.x;
    uint32_t first = 0, tiles = n_tiles;
    if constexpr (BATCH) {
        first = sets[s].tree_tile0;
        tiles = sets[s].tree_tiles;
    }
    uint32_t* row = rows + static_cast<size_t>(l) * n_tiles + first;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < tiles; base += kScanBlock * kScanItems) {
        uint32_t v[kScanItems];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t t = base + tid * kScanItems + k;
            v[k] = t < tiles ? row[t] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) sum += v[k];
        uint32_t all;
        uint32_t ex = carry + block_exclusive_sum<uint32_t, kScanBlock>(sum, tmp, &all);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t t = base + tid * kScanItems + k;
            if (t < tiles) row[t] = ex;
            ex += v[k];
        }
        carry += all;
    }
    if (tid == 0) totals[s * kTreeRows + l] = carry;
}

// ---- write -------------------------------------------------------------------

// What a batch writes besides the trees.
struct TreeResults {
    uint32_t rounds;  // rounds allowed: leaf levels are cut at it
    const uint32_t* set_flags;
    const uint32_t* sort_err;
    BatchResult* results;
};

// Result of set s. After r rounds from the root the leaves are the tree's down
// to level r, and the set has converged if a round was left to see no change:
// if its leaves end above level r.
__device__ __forceinline__ void write_set_result(const BatchSet& S, uint32_t s, uint64_t nl, uint32_t depth,
                                                 const TreeResults& r) {
    uint32_t status = CSTONE_OK;
    if (r.sort_err && *r.sort_err != 0)  // a device-side wait gave up: every array is unreliable
        status = CSTONE_ERR_DEVICE;
    else if (r.set_flags[s] & CSTONE_FLAG_NONFINITE)
        status = CSTONE_ERR_NONFINITE;
    else if (nl > S.cap)
        status = CSTONE_ERR_CAPACITY;
    else if (depth >= r.rounds)
        status = CSTONE_ERR_NOT_CONVERGED;
    r.results[s] = {static_cast<uint32_t>(nl), static_cast<uint32_t>(nl + (nl - 1) / 7), min(depth + 1, r.rounds),
                    status};
}

// First index in [lo, hi) of a sorted array that is >= k (hi if none): three
// probes a step, all in flight (the empty asm keeps the compiler from reading
// them one by one as they are compared), so that 512 keys take five round
// trips, not nine. (Seven probes a step were slower: the lines they touch cost
// more than the round trips they save.)
template <class T>
__device__ __forceinline__ uint32_t lower_bound_4(const T* __restrict__ a, uint32_t lo, uint32_t hi, T k) {
    while (hi > lo) {
        const uint32_t len = hi - lo, q = len >> 2;
        const uint32_t i0 = lo + q, i1 = lo + (len >> 1), i2 = lo + (len >> 1) + ((len + 1) >> 2);
        T k0 = a[i0], k1 = a[i1], k2 = a[min(i2, hi - 1)];
        asm volatile("" : "+v"(k0), "+v"(k1), "+v"(k2));
        const bool b0 = k0 < k, b1 = k1 < k, b2 = k2 < k;
        const uint32_t j2 = min(i2, hi - 1);
        lo = b2 ? j2 + 1 : (b1 ? i1 + 1 : (b0 ? i0 + 1 : lo));
        hi = b2 ? hi : (b1 ? j2 : (b0 ? i1 : i0));
        hi = max(hi, lo);
    }
    return lo;
}

constexpr int kWriteBlock = 128;
constexpr int kWriteWaves = kWriteBlock / kWave;

// One block per tile, or (small sets of very small leaves, where a tile holds a
// thousand internal nodes and few blocks are there) several that take its chunks
// of 64 in turn. Every wave takes the tile's internal nodes 64 at a time
// to find their ranks among the nodes of their level (ballots, and the running
// count of level l in lane l); then 8 lanes work for each node, the block's
// waves on 8 nodes each. A node without internal children holds at most 8 N
// particles, and the bytes u of its particles say everything: it ends before
// the first particle after its own with u <= l, and its children start at its
// first particle and where u = l + 1 (which child, the key's digit says). Its
// lanes read 64 of the bytes at a time. A node with internal children is
// searched in P, lane c for the start of child c (lane 0: for its end); these
// nodes (one in 8) are taken together, after the others, so that the others'
// waves do not wait for their searches.
//
// Bound: instructions (about 40 per node for the bytes, its lanes together),
// and three dependent reads (list, bytes, keys of the children's starts); 26 B
// of K, counts, NK and CO are written per leaf.
template <bool BATCH, bool FOCUS>
__global__ __launch_bounds__(kWriteBlock) void tree_write_kernel(const uint64_t* __restrict__ P, TreeOne one,
                                                                 const BatchSet* __restrict__ sets,
                                                                 const uint32_t* __restrict__ tile_set,
                                                                 uint32_t n_tiles, uint32_t max_level,
                                                                 const uint64_t* __restrict__ inodes,
                                                                 const uint32_t* __restrict__ ipos,
                                                                 const uint64_t* __restrict__ tile_off,
                                                                 const uint8_t* __restrict__ below,
                                                                 const uint32_t* __restrict__ rows, bool scanned,
                                                                 const uint32_t* __restrict__ totals_all,
                                                                 uint64_t* __restrict__ K, uint32_t* __restrict__ counts,
                                                                 uint64_t* __restrict__ nk, uint32_t* __restrict__ co,
                                                                 uint32_t* __restrict__ lo_out, TreeState* st,
                                                                 const uint32_t* input_flags, const uint32_t* listed,
                                                                 TreeResults res, FocusSpec focus) {
    __shared__ FocusPart<FOCUS> fsm;
    __shared__ uint32_t before[kTreeRows], after[kTreeRows], totals[kTreeRows];
    __shared__ uint32_t found[kWriteWaves][kWave];  // per wave and group: particles that start children
    __shared__ uint64_t first_key[kWriteWaves][kWave];  // per wave: the chunk's nodes' first keys and particles
    __shared__ uint32_t first_at[kWriteWaves][kWave];
    const uint32_t tid = threadIdx.x, lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t gtile = blockIdx.x, part = blockIdx.y, parts = gridDim.y;
    // Of keys that the sort has not finished only the state is written, to say so:
    // the tree would be thrown away, and what it leaves out is not there to read.
    const uint32_t unsorted = listed ? *listed : 0u;
    uint32_t s = 0, tile = gtile, tiles = n_tiles;
    TreeOne o = one;
    uint64_t node_off = 0;
    if constexpr (BATCH) {
        s = tile_set[gtile];
        const BatchSet& S = sets[s];
        tile = gtile - S.tree_tile0;
        tiles = S.tree_tiles;
        o = {S.part_off, S.n, S.n_crit, S.leaf_off, S.cap, S.inode_off};
        node_off = S.node_off;
        below += S.part_off;
    }
    if (scanned) {
        if (tid < kTreeRows) {
            const uint32_t* row = rows + static_cast<size_t>(tid) * n_tiles + gtile;
            const uint32_t t = totals_all[s * kTreeRows + tid];
            before[tid] = row[0];
            after[tid] = tile + 1 < tiles ? row[1] : t;
            totals[tid] = t;
        }
    } else {  // few tiles: 8 lanes add up a row
      for (uint32_t r = tid / 8; r < static_cast<uint32_t>(kTreeRows); r += kWriteBlock / 8) {
        const uint32_t g = tid % 8;
        const uint32_t* row = rows + static_cast<size_t>(r) * n_tiles + (gtile - tile);
        uint32_t v[kDirectTiles / 8];
#pragma unroll
        for (uint32_t k = 0; k < kDirectTiles / 8; ++k) v[k] = g + 8 * k < tiles ? row[g + 8 * k] : 0u;
        uint32_t b = 0, a = 0, t = 0;
#pragma unroll
        for (uint32_t k = 0; k < kDirectTiles / 8; ++k) {
            const uint32_t at = g + 8 * k;
            b += at < tile ? v[k] : 0u;
            a += at <= tile ? v[k] : 0u;
            t += v[k];
        }
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            b += __shfl_xor(b, d, kWave);
            a += __shfl_xor(a, d, kWave);
            t += __shfl_xor(t, d, kWave);
        }
        if (g == 0) {
            before[r] = b;
            after[r] = a;
            totals[r] = t;
        }
      }
    }
    __syncthreads();
    // leaves of the set; its level offsets: level l + 1 holds 8 nodes per internal node of level l
    const uint32_t tot = lane < kTreeLevels ? totals[lane] : 0u;
    const uint64_t ni = wave_sum<uint64_t>(tot);
    const uint64_t nl = 7 * ni + 1;
    const uint32_t depth = static_cast<uint32_t>(64 - clz64(__ballot(tot != 0)));
    uint32_t lo;
    {
        const uint32_t above = __shfl_up(tot, 1, kWave);
        const uint32_t v = lane == 0 ? 1u : (lane <= kTreeLevels ? 8u * above : 0u);
        lo = wave_inclusive_sum(v) - v;  // lane l: LO[l]; lane L + 1: the number of nodes
    }
    uint64_t* Ko = K + o.leaf_off;
    uint32_t* Co = counts ? counts + o.leaf_off : nullptr;
    const bool fits = nl <= o.cap;
    if (tile == 0 && part == 0) {
        if constexpr (BATCH) {
            if (tid == 0) write_set_result(sets[s], s, nl, depth, res);
        } else {
            if (tid == 0) {
                st->nl = fits ? nl : 0;
                st->n_leaves = nl;
                st->depth = depth;
                st->input_flags = input_flags ? *input_flags : 0u;
                st->listed = unsorted;
            }
        }
        if (fits && !unsorted) {
            if (tid == 0) {
                Ko[nl] = kKeyEnd;
                if (ni == 0) {  // the root alone
                    Ko[0] = 0;
                    if (Co) Co[0] = o.n;
                }
                if (nk) {
                    nk[node_off] = 1;
                    if (ni == 0) co[node_off] = 0;
                }
            }
            if (nk && tid <= static_cast<uint32_t>(kL + 1)) lo_out[static_cast<size_t>(s) * (kL + 2) + tid] = lo;
        }
    }
    if (!fits || unsorted) return;
    const uint32_t N = o.n_crit, n = o.n;
    const uint64_t* Ps = P + o.first;
    const uint32_t p0 = before[kTreeLevels];
    const uint32_t here = after[kTreeLevels] - before[kTreeLevels];  // internal nodes of this tile
    if (here == 0) return;  // block-uniform
    if constexpr (FOCUS) {
        focus_fill(focus, fsm);
        __syncthreads();
    }
    const uint64_t* In = inodes + o.inode_off;
    const uint32_t* Ip = ipos + o.inode_off;
    const uint64_t list = tile_off[gtile];
    const uint32_t nodes = static_cast<uint32_t>(nl + ni);
    uint64_t* Nk = nk ? nk + node_off : nullptr;
    uint32_t* Cn = nk ? co + node_off : nullptr;
    uint32_t run = lane < kTreeLevels ? before[lane] : 0u;
    const uint32_t c = lane & 7u, group = lane & ~7u;
    const uint32_t ua = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(below) & 7u);
    const uint64_t* words = reinterpret_cast<const uint64_t*>(below - ua);  // the bytes by aligned words
    uint32_t next_base = part * kWave;
    for (uint32_t base = 0; base < here; base += kWave) {
        const bool in = base + lane < here;
        const uint64_t key = in ? In[list + base + lane] : 1ull;
        const uint32_t pos = in ? Ip[list + base + lane] : 0u;
        const uint32_t level = in ? static_cast<uint32_t>(63 - clz64(key)) * 43u >> 7 : 31u;
        // rank among the nodes of its level, and the parent's: the last node of
        // the level above at or before this one
        const uint32_t lq = in ? level : 0u;
        uint32_t rank = __shfl(run, lq, kWave);
        uint32_t prank = __shfl(run, lq ? lq - 1 : 0u, kWave) - 1u;
        for (uint64_t left = __ballot(in); left;) {  // the levels present, a few
            const uint32_t q = __builtin_amdgcn_readlane(level, __builtin_ctzll(left));
            const uint64_t m = __ballot(level == q);
            const uint32_t k = lanes_below(m);
            rank += level == q ? k : 0u;
            prank += level == q + 1 ? k : 0u;
            if (lane == q) run += static_cast<uint32_t>(__popcll(m));
            left &= ~m;
        }
        if (base != next_base) continue;  // another block's chunk
        next_base += parts * kWave;
        // index of the first child, and the node's own
        const uint32_t child = __shfl(lo, lq + 1, kWave) + 8u * rank;
        const uint32_t lo_own = __shfl(lo, lq, kWave);
        const uint32_t self = lq ? lo_own + 8u * prank + static_cast<uint32_t>(key & 7u) : 0u;
        // index in K of a leaf child 0 with no internal node below this one before it
        const uint32_t leaf0 = 7u * (p0 + base + lane - lq) + digit_sum(key);
        if (Nk && in && self < nodes) Cn[self] = child;
        __builtin_amdgcn_wave_barrier();
        first_key[wave][lane] = in ? (key ^ (1ull << (3 * lq))) << (3 * (kL - lq)) : ~0ull;
        first_at[wave][lane] = pos;
        __builtin_amdgcn_wave_barrier();
        // nodes without internal children first: the next node of the list is
        // not one level down (at the end of the tile it is not known: searched)
        bool leafy = false;
        {
            const uint32_t next = __shfl_down(level, 1, kWave);
            if (!FOCUS && N <= kByteMaxCrit && base + lane + 1 < here) {
                const uint32_t nlv = lane + 1 < kWave
                                         ? next
                                         : static_cast<uint32_t>(63 - clz64(In[list + base + kWave])) / 3u;
                leafy = nlv != level + 1 && level < max_level;  // (a child on the last level may hold any number)
            }
        }
        const uint64_t m_leafy = __ballot(leafy), m_rest = __ballot(in && !leafy);
        const uint32_t n_leafy = static_cast<uint32_t>(__popcll(m_leafy)), n_rest = static_cast<uint32_t>(__popcll(m_rest));
        // place t holds the lane of the t-th leafy node, then of the others (and of no node)
        const uint32_t place = leafy ? lanes_below(m_leafy)
                                     : (in ? n_leafy + lanes_below(m_rest) : lane);  // (lanes past the list stay last)
        const uint32_t order = static_cast<uint32_t>(__builtin_amdgcn_ds_permute(static_cast<int>(place * 4), static_cast<int>(lane)));
        const uint32_t leafy_steps = (n_leafy + 7) / 8, steps = leafy_steps + (n_rest + 7) / 8;
        for (uint32_t step_i = wave; step_i < steps; step_i += kWriteWaves) {
            const bool bytes = step_i < leafy_steps;  // wave-uniform
            const uint32_t t = bytes ? step_i * 8 + lane / 8 : n_leafy + (step_i - leafy_steps) * 8 + lane / 8;
            const bool on = t < (bytes ? n_leafy : n_leafy + n_rest);
            const uint32_t x = __shfl(order, on ? t : 0, kWave);  // this lane's node of the chunk
            const uint64_t kx = (static_cast<uint64_t>(__shfl(static_cast<uint32_t>(key >> 32), x, kWave)) << 32) |
                                static_cast<uint32_t>(__shfl(static_cast<uint32_t>(key), x, kWave));
            const uint32_t px = __shfl(pos, x, kWave), l = __shfl(level, x, kWave);
            const uint32_t cx = __shfl(child, x, kWave);
            uint32_t at = __shfl(leaf0, x, kWave) + c;
            const uint32_t shift = 3 * (kL - 1 - l);  // of the children's digit
            const uint64_t ck = (kx << 3) | c;        // this lane's child
            uint32_t b;  // lane c: the first particle of child c or after it; lane 0: the node's end
            bool inner = false;
            uint32_t next_q = 0;  // place in the chunk of the first node in or after this child
            uint32_t ahead = 0;  // internal nodes below this one that start before this child, if the chunk says so
            if (bytes) {
                const uint32_t le_l = (l * 0x01010101u) | 0x80808080u, le_n = le_l + 0x01010101u;
                uint32_t kids = 1, stop = n;
                bool more = on;
                if (on && c == 0) found[wave][group] = px;
                const uint64_t first = static_cast<uint64_t>(px) + 1 + ua;  // of the bytes that are looked at
                uint32_t piece = static_cast<uint32_t>(first >> 3) + c;
                uint64_t skip = c ? ~0ull : ~0ull << (8 * (first & 7u));
                uint32_t turns = N / 8 + 3;  // 8 N particles hold the node's end; always fewer, bounds the loop
                uint64_t w_next = on ? words[piece] : 0ull;
                while (__ballot(more) && turns--) {
                    uint32_t le0 = 0, le1 = 0, eq0 = 0, eq1 = 0;
                    const uint64_t w = w_next;
                    if (more) {
                        w_next = words[piece + 8];  // (of the next turn, in flight during this one)
                        const uint32_t w0 = static_cast<uint32_t>(w), w1 = static_cast<uint32_t>(w >> 32);
                        const uint32_t s0 = static_cast<uint32_t>(skip) & 0x80808080u, s1 = static_cast<uint32_t>(skip >> 32) & 0x80808080u;
                        le0 = (le_l - w0) & s0;  // the high bit of each byte that is at most l
                        le1 = (le_l - w1) & s1;
                        eq0 = (le_n - w0) & s0 & ~le0;
                        eq1 = (le_n - w1) & s1 & ~le1;
                    }
                    const uint32_t at0 = piece * 8 - ua;  // particle of the word's first byte (mod 2^32 for places before 0)
                    // the first place at or above the node's level, over the 8 lanes
                    const uint32_t mine = le0 ? static_cast<uint32_t>(__builtin_ctz(le0)) >> 3
                                              : 4u + (static_cast<uint32_t>(__builtin_ctz(le1 | 0x80000000u)) >> 3);
                    const uint32_t e = group_min((le0 | le1) ? 8 * c + mine : 64u);  // place among the group's 64
                    const uint32_t mybit = 64u * c;  // bit of this lane's first place
                    if (8 * e < mybit + 64u) {  // places from the end on do not count
                        const uint64_t keep = 8 * e <= mybit ? 0ull : (1ull << (8 * e - mybit)) - 1ull;
                        eq0 &= static_cast<uint32_t>(keep);
                        eq1 &= static_cast<uint32_t>(keep >> 32);
                    }
                    const uint32_t own = static_cast<uint32_t>(__popc(eq0) + __popc(eq1));
                    const uint32_t inc = group_add_up(own, c);
                    uint64_t eq = (static_cast<uint64_t>(eq1) << 32) | eq0;
                    uint32_t k = kids + inc - own;
                    while (eq) {
                        if (k < 8) found[wave][group + k] = at0 + (static_cast<uint32_t>(__builtin_ctzll(eq)) >> 3);
                        ++k;
                        eq &= eq - 1;
                    }
                    kids += __shfl(inc, static_cast<int>(group + 7), kWave);
                    if (more && e < 64u) {
                        stop = at0 - 8 * c + e;
                        more = false;
                    }
                    piece += 8;
                    skip = ~0ull;
                }
                __builtin_amdgcn_wave_barrier();
                uint32_t j = stop, bit = 0;
                if (on && c < kids) {
                    j = min(found[wave][lane], n - 1);  // (below n always; guards memory)
                    bit = 1u << (static_cast<uint32_t>(Ps[j] >> shift) & 7u);
                }
                __builtin_amdgcn_wave_barrier();
                const uint32_t digits = group_or(bit);  // which children have particles
                const uint32_t nth = static_cast<uint32_t>(__popc(digits & ((1u << c) - 1u)));
                const uint32_t at_c = __shfl(j, static_cast<int>(group + min(nth, 7u)), kWave);
                b = c == 0 ? stop : ((digits >> c) ? at_c : stop);
            } else {
                b = 0;
                const uint64_t start = (ck ^ (1ull << (3 * (l + 1)))) << shift;  // child c's first key
                const uint64_t first = c ? start : start + (8ull << shift);      // lane 0: the node's end
                // the chunk's first node at or after this key, and the last one before it
                const uint32_t chunk = min(here - base, static_cast<uint32_t>(kWave));
                uint32_t q = x + 1, q_hi = chunk;
                while (q < q_hi) {
                    const uint32_t mid = (q + q_hi) >> 1;
                    if (first_key[wave][mid] < first)
                        q = mid + 1;
                    else
                        q_hi = mid;
                }
                ahead = q < chunk ? q - x - 1 : 0xffffffffu;
                next_q = c ? q : x + 1;
                uint32_t lo_at = on ? first_at[wave][q - 1] : 0u, hi_at = lo_at;
                if (on && q < chunk) {
                    hi_at = first_at[wave][q];
                    if (first_key[wave][q] == first) lo_at = hi_at;  // that child itself (or what follows the node)
                }
                // past the chunk's nodes: a place at or past the node's end; the
                // lanes try 8 N, 16 N, ... from the last one's first particle
                const bool beyond = on && q == chunk;
                if (__ballot(beyond)) {
                    const uint64_t end = start + (static_cast<uint64_t>(8 - c) << shift);
                    const uint32_t from_at = first_at[wave][chunk - 1];
                    uint64_t far = 0;
                    bool open = ((__ballot(beyond) >> group) & 0xffull) != 0;
                    for (uint64_t step = 8ull * N; __ballot(open); step <<= 8) {
                        const uint64_t mine = from_at + (step << c);
                        const bool past = !open || mine >= n || Ps[mine] >= end;
                        const uint32_t which = static_cast<uint32_t>((__ballot(past) >> group) & 0xffull);
                        if (open && which) {
                            far = from_at + (step << __builtin_ctz(which));
                            open = false;
                        }
                    }
                    if (beyond) hi_at = static_cast<uint32_t>(min<uint64_t>(far, n));
                }
                if (on) b = lower_bound_4(Ps, lo_at, hi_at, first);
            }
            const uint32_t next = __shfl(b, static_cast<int>(c == 7 ? group : lane + 1), kWave);
            const uint32_t from = c ? b : px;
            const uint32_t cnt = next - from;
            if (!bytes) {
                inner = on && l + 1 <= max_level && cnt > N;
                if constexpr (FOCUS) {
                    // the child is internal if nodes of the list lie in it; past
                    // the chunk the MAC has to say (the MAC for all: 78 us, now 38)
                    if (inner) {
                        const uint64_t start = (ck ^ (1ull << (3 * (l + 1)))) << shift;
                        inner = next_q < min(here - base, static_cast<uint32_t>(kWave))
                                    ? first_key[wave][next_q] < start + (1ull << shift)
                                    : node_fails(start, l + 1, focus, fsm);
                    }
                }
                const bool family = ((__ballot(inner) >> group) & 0xffull) != 0;
                if (on && !inner && c && ahead != 0xffffffffu) {
                    at += 7u * ahead;
                } else if (on && !inner && family && from > px) {  // counted over the tiles
                    uint32_t upto = static_cast<uint32_t>(ni);
                    if (from < n) {
                        const uint32_t tl = from / kTreeTile, gt = gtile - tile + tl;
                        uint32_t b0 = 0, b1 = 0;  // internal nodes before tile tl and up to its end
                        if (scanned) {
                            const uint32_t* row = rows + static_cast<size_t>(kTreeLevels) * n_tiles + gt;
                            b0 = row[0];
                            b1 = tl + 1 < tiles ? row[1] : totals[kTreeLevels];
                        } else {
                            const uint32_t* row = rows + static_cast<size_t>(kTreeLevels) * n_tiles + (gtile - tile);
                            for (uint32_t k = 0; k <= tl; ++k) {
                                b0 = b1;
                                b1 += row[k];
                            }
                        }
                        upto = b0;
                        if (b1 > b0) {
                            const uint32_t* q = Ip + tile_off[gt];
                            upto += lower_bound_4(q, 0u, b1 - b0, from);
                        }
                    }
                    const uint32_t p1 = p0 + base + x + 1;  // nodes up to and with this one
                    if (upto > p1) at += 7u * (upto - p1);
                }
            }
            if (on && !inner && at < nl) {  // (at < nl always; guards memory)
                Ko[at] = (ck ^ (1ull << (3 * (l + 1)))) << shift;
                if (Co) Co[at] = cnt;
            }
            if (on && Nk && cx + c < nodes) {  // (always)
                Nk[cx + c] = ck;
                if (!inner) Cn[cx + c] = 0;
            }
        }
    }
}

// Sets without particles: the root leaf.
__global__ __launch_bounds__(64) void tree_empty_sets_kernel(const BatchSet* __restrict__ sets, uint32_t n_sets,
                                                             uint64_t* __restrict__ K, uint32_t* __restrict__ counts,
                                                             uint64_t* __restrict__ nk, uint32_t* __restrict__ co,
                                                             uint32_t* __restrict__ lo_out, TreeResults res) {
    const uint32_t s = blockIdx.x * 64 + threadIdx.x;
    if (s >= n_sets || sets[s].n != 0) return;
    const BatchSet& S = sets[s];
    K[S.leaf_off] = 0;
    K[S.leaf_off + 1] = kKeyEnd;
    counts[S.leaf_off] = 0;
    nk[S.node_off] = 1;
    co[S.node_off] = 0;
    for (int l = 0; l <= kL + 1; ++l) lo_out[static_cast<size_t>(s) * (kL + 2) + l] = l ? 1u : 0u;
    write_set_result(S, s, 1, 0, res);
}

// ---- rounds from another array ----------------------------------------------------
//
// From an array K_old the rounds reach the same tree; their number is 1 + the
// largest level difference between two overlapping leaves (a leaf over N_crit
// splits one level a round, a subtree under a leaf of the tree merges one
// level a round), and no round's array is longer than the leaves of the two
// arrays that lie on their finer side together (`inter`).
//
// Bound: the chain of reads and searches of a tile, one after another, so as
// many blocks as fit: two arrays of 28 M leaves 397 us with four on a CU, 308
// with six (reading both is 90). Starting each search where the block's tile
// before ended gains 9 us more, not worth its code.

constexpr int kCmpBlock = 256;
constexpr uint32_t kCmpTile = 1024;
constexpr uint32_t kCmpOld = 2048;
constexpr size_t kCmpBlocks = 6 * 256;  // as many as the LDS of all CUs holds at once

__device__ __forceinline__ int delta_level(uint64_t delta) { return kL - (63 - clz64(delta)) / 3; }

__global__ __launch_bounds__(kCmpBlock) void tree_compare_kernel(const uint64_t* __restrict__ K_old, uint32_t nl_old,
                                                                 const uint64_t* __restrict__ K, uint64_t cap,
                                                                 TreeState* st) {
    __shared__ uint64_t a[kCmpTile + 1];
    __shared__ uint64_t b[kCmpOld + 2];
    __shared__ uint32_t range[2];
    __shared__ uint32_t red_n[kCmpBlock / kWave], red_d[kCmpBlock / kWave];
    const uint64_t nl = st->n_leaves;
    if (nl > cap || st->listed) return;  // (nothing was written)
    const uint32_t tiles = static_cast<uint32_t>((nl + kCmpTile - 1) / kCmpTile);
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint64_t inter = 0;
    int diff = 0;
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t base = tile * kCmpTile;
        const uint32_t m = static_cast<uint32_t>(min<uint64_t>(kCmpTile, nl - base));
        for (uint32_t i = tid; i <= m; i += kCmpBlock) a[i] = K[base + i];
        __syncthreads();
        if (wave < 2) {  // the old leaves that start in this tile's keys
            const uint32_t at = wave_lower_bound(K_old, 0, nl_old, wave ? a[m] : a[0]);
            if (lane_id() == 0) range[wave] = at;
        }
        __syncthreads();
        const uint32_t p0 = range[0], p1 = range[1];
        const OldKeys old = old_keys(p0, p1);  // (at most nl_old: K_old has a closing key)
        const uint32_t q0 = old.first, q1 = old.last;
        const uint32_t held = q1 - q0 + 1;
        const bool staged = held <= kCmpOld + 2;
        if (staged) {
            for (uint32_t i = tid; i < held; i += kCmpBlock) b[i] = K_old[q0 + i];
            __syncthreads();
        }
        for (uint32_t j = tid; j < m; j += kCmpBlock) {  // leaves as fine as the old one around them, or finer
            const uint32_t p = staged ? at_or_before(b, 0u, q1 - q0, a[j]) : at_or_before(K_old, q0, q1, a[j]);
            const uint64_t d_old = staged ? b[p + 1] - b[p] : K_old[p + 1] - K_old[p];
            const int d = delta_level(a[j + 1] - a[j]) - delta_level(d_old);
            if (d >= 0) {
                ++inter;
                diff = max(diff, d);
            }
        }
        for (uint32_t i = p0 + tid; i < p1; i += kCmpBlock) {  // old leaves finer than the new one around them
            const uint64_t k = staged ? b[i - q0] : K_old[i];
            const uint64_t d_old = (staged ? b[i - q0 + 1] : K_old[i + 1]) - k;
            const uint32_t j = at_or_before(a, 0u, m, k);
            const int d = delta_level(d_old) - delta_level(a[j + 1] - a[j]);
            if (d > 0) {
                ++inter;
                diff = max(diff, d);
            }
        }
        __syncthreads();
    }
    const uint64_t n_wave = wave_sum<uint64_t>(inter);
    for (int d = 1; d < kWave; d <<= 1) diff = max(diff, __shfl_xor(diff, d, kWave));
    if (lane_id() == 0) {
        red_n[wave] = static_cast<uint32_t>(n_wave);
        red_d[wave] = static_cast<uint32_t>(diff);
    }
    __syncthreads();
    if (tid == 0) {
        uint64_t sum = 0;
        uint32_t most = 0;
        for (int v = 0; v < kCmpBlock / kWave; ++v) {
            sum += red_n[v];
            most = max(most, red_d[v]);
        }
        if (sum) atomicAdd(reinterpret_cast<unsigned long long*>(&st->inter), static_cast<unsigned long long>(sum));
        if (most) atomicMax(&st->max_diff, most);
    }
}

// The new array into `leaves`, if the rounds would have reached it within the capacity.
__global__ __launch_bounds__(256) void tree_commit_kernel(const uint64_t* __restrict__ K, uint64_t* __restrict__ leaves,
                                                          uint64_t cap, TreeState* st) {
    const uint64_t nl = st->n_leaves;
    if (st->listed) return;
    const bool fits = nl <= cap && st->inter <= cap;
    const size_t t = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (!fits) {
        if (t == 0) st->nl = 0;
        return;
    }
    for (size_t i = t; i <= nl; i += static_cast<size_t>(gridDim.x) * 256) leaves[i] = K[i];
}

struct TreeWs {
    uint64_t* K_new;  // the new array while the old one is still needed
    uint64_t* inodes;
    uint32_t *ipos, *rows, *totals;
    uint64_t* tile_off;
    uint8_t* below;
    TreeState* st;
    size_t bytes;
};

TreeWs carve_tree(void* ws, size_t n, uint32_t n_crit, size_t cap, bool incremental, bool focus) {
    Carve c(ws);
    TreeWs w{};
    const size_t tiles = tree_tiles(n), slots = focus ? (cap - 1) / 7 + 1 : tree_slots(n, n_crit, cap);
    w.st = c.take<TreeState>(1);
    w.K_new = incremental ? c.take<uint64_t>(cap + 1) : nullptr;
    w.inodes = c.take<uint64_t>(slots);
    w.ipos = c.take<uint32_t>(slots);
    w.tile_off = c.take<uint64_t>(tiles);
    w.rows = c.take<uint32_t>(kTreeRows * tiles);
    w.totals = c.take<uint32_t>(kTreeRows);
    w.below = focus ? nullptr : c.take<uint8_t>(n + kBytesPad);
    w.bytes = c.off;
    return w;
}

// Blocks per tile of the write launch: one for every four chunks that a tile of
// such leaves holds, as long as that leaves two tiles' blocks on a CU. N_crit 1,
// whole builds of uniform particles by one block a tile and by eight: 5000 346 ->
// 158 us, 65,536 389 -> 166.
uint32_t write_parts(uint32_t n_crit, uint32_t tiles) {
    constexpr uint32_t kMaxParts = 8, kMaxBlocks = 512;
    return std::max(1u, std::min({kMaxParts, tile_slots(n_crit) / (4 * kWave), kMaxBlocks / tiles}));
}

__global__ void tree_clear_kernel(TreeState* st) { *st = TreeState{}; }

}  // namespace

size_t tree_workspace_bytes(size_t n, uint32_t n_crit, size_t cap, bool incremental) {
    return carve_tree(nullptr, n, n_crit, cap, incremental, false).bytes;
}

size_t focus_tree_workspace_bytes(size_t n, size_t cap) { return carve_tree(nullptr, n, 1, cap, true, true).bytes; }

size_t tree_tiles(size_t n) { return tree_tiles_of(n); }

size_t tree_slots(size_t n, uint32_t n_crit, size_t cap) { return tree_tiles(n) * tile_slots(n_crit) + (cap - 1) / 7 + 1; }

bool tree_possible(size_t n, uint32_t max_iters) {
    return n > 0 && (max_iters == 0 || max_iters >= static_cast<uint32_t>(kL + 1));
}

bool TreePass::run(const uint64_t* P, size_t n, uint32_t n_crit, uint64_t* leaves, size_t nl0, size_t cap,
                   uint32_t* counts, uint64_t* node_keys, uint32_t* child, uint32_t* level_offsets, void* ws,
                   size_t ws_bytes, TreeState* cleared, const uint32_t* input_flags, const uint32_t* listed,
                   hipStream_t stream, const FocusSpec* focus) {
    incremental_ = nl0 > 1;
    const TreeWs w = carve_tree(ws, n, n_crit, cap, incremental_, focus != nullptr);
    if (ws_bytes < w.bytes || cap >= 0xffffffffull) return false;
    stream_ = stream;
    st_ = cleared ? cleared : w.st;
    if (!cleared) hipLaunchKernelGGL(tree_clear_kernel, dim3(1), dim3(1), 0, stream, st_);
    const uint32_t tiles = static_cast<uint32_t>(tree_tiles(n));
    const bool scanned = tiles > kDirectTiles;
    const TreeOne one{0, static_cast<uint32_t>(n), n_crit, 0, cap, 0};
    const BatchSet* no_sets = nullptr;
    const uint32_t* no_table = nullptr;
    constexpr uint32_t max_level = kL - 1;
    uint64_t* K = incremental_ ? w.K_new : leaves;
    const auto mark = focus ? tree_mark_kernel<false, true, Keep::kNone>
                            : (n_crit <= kByteMaxCrit ? tree_mark_kernel<false, false, Keep::kBytes>
                                                      : tree_mark_kernel<false, false, Keep::kNone>);
    const auto write = focus ? tree_write_kernel<false, true> : tree_write_kernel<false, false>;
    const FocusSpec spec = focus ? *focus : FocusSpec{};
    hipLaunchKernelGGL(mark, dim3(tiles), dim3(kMarkBlock), 0, stream, P, one, no_sets, no_table, tiles, max_level,
                       w.below, w.inodes, w.ipos, w.tile_off, w.rows, &st_->reserved, spec);
    if (scanned) launch_row_scan(w.rows, kTreeRows, tiles, w.totals, stream);
    hipLaunchKernelGGL(write, dim3(tiles, write_parts(n_crit, tiles)), dim3(kWriteBlock), 0, stream, P, one, no_sets, no_table, tiles, max_level,
                       w.inodes, w.ipos, w.tile_off, w.below, w.rows, scanned, w.totals, K, counts, node_keys, child,
                       level_offsets, st_, input_flags, listed, TreeResults{}, spec);
    if (incremental_) {
        const uint32_t grid = static_cast<uint32_t>(std::min<size_t>((cap + kCmpTile - 1) / kCmpTile, kCmpBlocks));
        hipLaunchKernelGGL(tree_compare_kernel, dim3(grid), dim3(kCmpBlock), 0, stream, leaves,
                           static_cast<uint32_t>(nl0), w.K_new, static_cast<uint64_t>(cap), st_);
        hipLaunchKernelGGL(tree_commit_kernel, dim3(static_cast<uint32_t>(std::min<size_t>((cap + 256) / 256, 2048))),
                           dim3(256), 0, stream, w.K_new, leaves, static_cast<uint64_t>(cap), st_);
    }
    return true;
}

cstone_status TreePass::wait(bool* fits) {
    *fits = false;
    CS_HIP(hipGetLastError());
    TreeState host;
    CS_HIP(hipMemcpyAsync(&host, st_, sizeof host, hipMemcpyDeviceToHost, stream_));
    CS_HIP(hipStreamSynchronize(stream_));
    input_flags = host.input_flags;
    listed = host.listed;
    n_leaves = host.nl;
    rounds = 1 + (incremental_ ? host.max_diff : host.depth);
    *fits = host.nl != 0;
    return CSTONE_OK;
}

void launch_row_scan(uint32_t* rows, uint32_t n_rows, uint32_t row_length, uint32_t* totals, hipStream_t stream) {
    const BatchSet* no_sets = nullptr;
    hipLaunchKernelGGL(tree_scan_kernel<false>, dim3(n_rows), dim3(kScanBlock), 0, stream, no_sets, row_length, rows, totals);
}

// ---- batched trees -------------------------------------------------------------------

namespace {

struct BatchTreeWs {
    uint64_t* inodes;
    uint32_t *ipos, *rows, *totals;
    uint64_t* tile_off;
    uint8_t* below;
    size_t bytes;
};

BatchTreeWs carve_batch_tree(void* ws, size_t n_total, uint32_t n_sets, size_t tiles, size_t inode_slots) {
    Carve c(ws);
    BatchTreeWs w{};
    w.inodes = c.take<uint64_t>(inode_slots);
    w.ipos = c.take<uint32_t>(inode_slots);
    w.tile_off = c.take<uint64_t>(tiles);
    w.rows = c.take<uint32_t>(kTreeRows * tiles);
    w.totals = c.take<uint32_t>(kTreeRows * static_cast<size_t>(n_sets));
    w.below = c.take<uint8_t>(n_total + kBytesPad);
    w.bytes = c.off;
    return w;
}

}  // namespace

size_t batch_tree_workspace_bytes(size_t n_total, uint32_t n_sets, size_t tiles, size_t inode_slots) {
    return carve_batch_tree(nullptr, n_total, n_sets, tiles, inode_slots).bytes;
}

cstone_status launch_batch_tree(const uint64_t* P, size_t n_total, const BatchSet* sets, uint32_t n_sets, const uint32_t* tile_set,
                                size_t n_tiles, size_t max_tiles, bool empty_sets, uint32_t most_crit, size_t inode_slots, uint32_t rounds,
                                const uint32_t* set_flags, const uint32_t* sort_err, uint32_t* reserved,
                                uint64_t* leaves, uint32_t* counts, uint64_t* node_keys, uint32_t* child,
                                uint32_t* level_offsets, BatchResult* results, void* ws, size_t ws_bytes,
                                hipStream_t stream) {
    const BatchTreeWs w = carve_batch_tree(ws, n_total, n_sets, n_tiles, inode_slots);
    if (ws_bytes < w.bytes || n_tiles >= 0xffffffffull || rounds < 1) return CSTONE_ERR_INVALID_ARG;
    const uint32_t tiles = static_cast<uint32_t>(n_tiles);
    const TreeOne one{};
    const uint32_t max_level = std::min<uint32_t>(rounds - 1, kL - 1);  // r rounds from the root split levels 0 .. r - 1
    const TreeResults res{rounds, set_flags, sort_err, results};
    if (tiles) {
        const bool scanned = max_tiles > kDirectTiles;
        const auto mark = most_crit <= kByteMaxCrit ? tree_mark_kernel<true, false, Keep::kBytes>
                                                    : tree_mark_kernel<true, false, Keep::kByCrit>;
        hipLaunchKernelGGL(mark, dim3(tiles), dim3(kMarkBlock), 0, stream, P, one, sets,
                           tile_set, tiles, max_level, w.below, w.inodes, w.ipos, w.tile_off, w.rows, reserved,
                           FocusSpec{});
        if (scanned)
            hipLaunchKernelGGL(tree_scan_kernel<true>, dim3(kTreeRows, n_sets), dim3(kScanBlock), 0, stream, sets, tiles,
                               w.rows, w.totals);
        hipLaunchKernelGGL((tree_write_kernel<true, false>), dim3(tiles), dim3(kWriteBlock), 0, stream, P, one, sets,
                           tile_set, tiles, max_level, w.inodes, w.ipos, w.tile_off, w.below, w.rows, scanned, w.totals, leaves,
                           counts, node_keys, child, level_offsets, static_cast<TreeState*>(nullptr),
                           static_cast<const uint32_t*>(nullptr), static_cast<const uint32_t*>(nullptr), res, FocusSpec{});
    }
    if (empty_sets)
        hipLaunchKernelGGL(tree_empty_sets_kernel, dim3((n_sets + 63) / 64), dim3(64), 0, stream, sets, n_sets, leaves,
                           counts, node_keys, child, level_offsets, res);
    CS_HIP(hipGetLastError());
    return CSTONE_OK;
}

}  // namespace cs
