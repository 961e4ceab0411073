// C ABI entry points of libcstone (declared and documented in cstone.h):
// argument checks, workspace layout and the order of the stages on a stream.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "internal.hpp"

using namespace cs;

namespace {

bool box_ok(const cstone_box* b) {
    if (!b) return false;
    for (int d = 0; d < 3; ++d)
        if (!std::isfinite(b->lo[d]) || !std::isfinite(b->hi[d]) || !(b->lo[d] < b->hi[d])) return false;
    return true;
}

constexpr size_t kMaxN = 0xffffffffull;  // counts, perm, CO and LO are uint32

// Builds below this size run the sort's low passes only when a bucket was listed
// (see cstone_build). Always enqueued / on demand, uniform particles: 65,536 127 / 116
// us, 2^20 173 / 165, 2^24 650 / 642, 2^25 1189 / 1178, 2^26 2256 / 2246. Above it less
// than a hundredth is gained, and a build that lists a bucket writes its tree twice.
constexpr size_t kListMaxKeys = size_t{1} << 25;

// Whether a build takes its tree from the sorted keys directly, where it may. Only
// large builds from an array of few leaves are faster by rounds, which go by the
// leaves and not by the keys. Builds from the last step's tree, direct against
// rounds in us, uniform keys: 2^26, N_crit 64 (a leaf per 32 keys) 2321 / 2277,
// N_crit 256 2318 / 2232, 1000 2202 / 2117; 2^25 1246 / 1265, 1182 / 1128, 1161 /
// 1148; Plummer 2^27, N_crit 64 (a leaf per 18) 5323 / 5336, 256 5147 / 4906; 2^24 is a
// tie from N_crit 256 on.
constexpr size_t kRoundsKeys = size_t{1} << 25;
bool direct_pays(size_t n, size_t nl0) { return nl0 <= 1 || n < kRoundsKeys || nl0 >= n / 32; }

// What a build's stages hand on besides their arrays.
struct BuildWords {
    TreeState tree;  // cleared by the sort's set-up
    uint32_t flag;   // non-finite coordinates; the sort's errors
};

size_t nodes_of(size_t nl) { return nl + (nl ? (nl - 1) / 7 : 0); }

__global__ void clear_word_kernel(uint32_t* w) { *w = 0; }

}  // namespace

extern "C" {

const char* cstone_status_string(cstone_status s) {
    switch (s) {
        case CSTONE_OK: return "ok";
        case CSTONE_ERR_INVALID_ARG: return "invalid argument";
        case CSTONE_ERR_NONFINITE: return "non-finite coordinate";
        case CSTONE_ERR_CAPACITY: return "leaf capacity exceeded";
        case CSTONE_ERR_NOT_CONVERGED: return "rebalance did not converge within max_iters";
        case CSTONE_ERR_DEVICE: return "device error";
    }
    return "unknown status";
}

cstone_status cstone_compute_keys(const double* x, const double* y, const double* z, size_t n, const cstone_box* box,
                                  cstone_curve curve, uint64_t* keys, uint32_t* flags, hipStream_t stream) {
    if (n > kMaxN || !box_ok(box) || (curve != CSTONE_MORTON && curve != CSTONE_HILBERT)) return CSTONE_ERR_INVALID_ARG;
    if (n && (!x || !y || !z || !keys)) return CSTONE_ERR_INVALID_ARG;
    return launch_keys(x, y, z, n, *box, curve, keys, flags, stream);
}

size_t cstone_sort_workspace_bytes(size_t n) { return sort_workspace_bytes(n, true); }

cstone_status cstone_sort(const uint64_t* keys_in, uint64_t* keys_out, uint32_t* perm_out, size_t n, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
    if (n > kMaxN) return CSTONE_ERR_INVALID_ARG;
    if (n && (!keys_in || !keys_out || !perm_out || !ws)) return CSTONE_ERR_INVALID_ARG;
    return launch_sort(keys_in, keys_out, perm_out, n, 63, ws, ws_bytes, stream);
}

cstone_status cstone_node_counts(const uint64_t* sorted_keys, size_t n, const uint64_t* leaves, size_t n_leaves,
                                 uint32_t* counts, hipStream_t stream) {
    if (n > kMaxN || n_leaves < 1 || !leaves || !counts || (n && !sorted_keys)) return CSTONE_ERR_INVALID_ARG;
    return launch_node_counts(sorted_keys, n, leaves, n_leaves, counts, stream);
}

size_t cstone_rebalance_workspace_bytes(size_t n, uint32_t n_crit, size_t leaf_capacity) {
    return rebalance_workspace_bytes(n, n_crit, leaf_capacity);
}

size_t cstone_rebalance_least_workspace_bytes(size_t n, uint32_t n_crit, size_t leaf_capacity) {
    return rebalance_rounds_bytes(n, n_crit, leaf_capacity);
}

size_t cstone_leaf_capacity_bound(size_t n, uint32_t n_crit, size_t n_leaves_start) {
    const size_t full = n / (static_cast<size_t>(n_crit) + 1);
    size_t bound = 7 * static_cast<size_t>(kL) * full + 1;
    if (n_leaves_start > 1) bound = std::max(bound, n_leaves_start + 7 * full);
    return bound;
}

cstone_status cstone_rebalance(const uint64_t* sorted_keys, size_t n, uint32_t n_crit, uint64_t* leaves,
                               size_t* n_leaves, size_t leaf_capacity, uint32_t* counts, uint32_t max_iters,
                               uint32_t* iters_done, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n > kMaxN || n_crit == 0 || !leaves || !n_leaves || !ws || (n && !sorted_keys)) return CSTONE_ERR_INVALID_ARG;
    if (*n_leaves < 1 || *n_leaves > leaf_capacity) return CSTONE_ERR_INVALID_ARG;
    return run_rebalance(sorted_keys, n, n_crit, leaves, n_leaves, leaf_capacity, counts, max_iters, iters_done, ws,
                         ws_bytes, stream);
}

size_t cstone_node_count(size_t n_leaves) { return nodes_of(n_leaves); }

size_t cstone_link_workspace_bytes(size_t n_leaves) { return link_workspace_bytes(n_leaves); }

cstone_status cstone_link_octree(const uint64_t* leaves, size_t n_leaves, uint64_t* node_keys, uint32_t* child,
                                 uint32_t* level_offsets, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n_leaves < 1 || n_leaves > kMaxN || (n_leaves - 1) % 7 != 0) return CSTONE_ERR_INVALID_ARG;
    if (!leaves || !node_keys || !child || !level_offsets || !ws) return CSTONE_ERR_INVALID_ARG;
    return launch_link(leaves, n_leaves, nullptr, node_keys, child, level_offsets, ws, ws_bytes, stream);
}

cstone_status cstone_link_octree_by_sort(const uint64_t* leaves, size_t n_leaves, uint64_t* node_keys, uint32_t* child,
                                         uint32_t* level_offsets, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n_leaves < 1 || n_leaves > kMaxN || (n_leaves - 1) % 7 != 0) return CSTONE_ERR_INVALID_ARG;
    if (!leaves || !node_keys || !child || !level_offsets || !ws) return CSTONE_ERR_INVALID_ARG;
    return launch_link_by_sort(leaves, n_leaves, node_keys, child, level_offsets, ws, ws_bytes, stream);
}

cstone_status cstone_radix_tree(const uint64_t* keys, size_t m, uint32_t* first, uint32_t* last, uint32_t* split,
                                uint32_t* prefix_len, hipStream_t stream) {
    if (m > kMaxN || (m >= 2 && (!keys || !prefix_len))) return CSTONE_ERR_INVALID_ARG;
    return launch_radix_tree(keys, m, first, last, split, prefix_len, stream);
}

size_t cstone_link_octree_radix_workspace_bytes(size_t n_leaves) { return radix_link_workspace_bytes(n_leaves); }

cstone_status cstone_link_octree_radix(const uint64_t* leaves, size_t n_leaves, uint64_t* node_keys, uint32_t* child,
                                       uint32_t* level_offsets, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n_leaves < 1 || n_leaves > kMaxN || (n_leaves - 1) % 7 != 0) return CSTONE_ERR_INVALID_ARG;
    if (!leaves || !node_keys || !child || !level_offsets || !ws) return CSTONE_ERR_INVALID_ARG;
    return launch_link_radix(leaves, n_leaves, node_keys, child, level_offsets, ws, ws_bytes, stream);
}

size_t cstone_compact_octree_workspace_bytes(size_t n_leaves) { return compact_octree_workspace_bytes(n_leaves); }

cstone_status cstone_compact_octree(const uint64_t* leaves, const uint32_t* counts, size_t n_leaves,
                                    uint64_t* node_keys, uint32_t* parent, uint32_t* level_offsets, size_t* n_nodes,
                                    void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n_leaves < 1 || n_leaves >= kMaxN / 2) return CSTONE_ERR_INVALID_ARG;
    if (!leaves || !counts || !node_keys || !parent || !level_offsets || !n_nodes || !ws) return CSTONE_ERR_INVALID_ARG;
    return launch_compact_octree(leaves, counts, n_leaves, node_keys, parent, level_offsets, n_nodes, ws, ws_bytes,
                                 stream);
}

size_t cstone_octree_node_counts_workspace_bytes(size_t n_leaves) { return node_props_workspace_bytes(n_leaves); }

cstone_status cstone_octree_node_counts(const uint64_t* leaves, const uint32_t* counts, size_t n_leaves,
                                        const uint64_t* node_keys, size_t n_nodes, uint32_t* node_counts, void* ws,
                                        size_t ws_bytes, hipStream_t stream) {
    if (n_leaves < 1 || n_leaves > kMaxN || n_nodes > kMaxN) return CSTONE_ERR_INVALID_ARG;
    if (!leaves || !counts || !ws || (n_nodes && (!node_keys || !node_counts))) return CSTONE_ERR_INVALID_ARG;
    return launch_octree_node_counts(leaves, counts, n_leaves, node_keys, n_nodes, node_counts, ws, ws_bytes, stream);
}

cstone_status cstone_gather(const double* src, const uint32_t* perm, size_t n, double* dst, hipStream_t stream) {
    if (n > kMaxN || (n && (!src || !perm || !dst))) return CSTONE_ERR_INVALID_ARG;
    return launch_gather(&src, perm, n, &dst, 1, false, stream);
}

cstone_status cstone_gather_xyz(const double* x, const double* y, const double* z, const uint32_t* perm, size_t n,
                                double* ox, double* oy, double* oz, int fused, hipStream_t stream) {
    if (n > kMaxN || (n && (!x || !y || !z || !perm || !ox || !oy || !oz))) return CSTONE_ERR_INVALID_ARG;
    const double* src[3] = {x, y, z};
    double* dst[3] = {ox, oy, oz};
    return launch_gather(src, perm, n, dst, 3, fused != 0, stream);
}

size_t cstone_gather_xyz_workspace_bytes(size_t n) { return n > kMaxN ? 0 : gather_packed_workspace_bytes(n); }

cstone_status cstone_gather_xyz_packed(const double* x, const double* y, const double* z, const uint32_t* perm, size_t n,
                                       double* ox, double* oy, double* oz, void* ws, size_t ws_bytes,
                                       hipStream_t stream) {
    if (n > kMaxN || (n && (!x || !y || !z || !perm || !ox || !oy || !oz))) return CSTONE_ERR_INVALID_ARG;
    const double* src[3] = {x, y, z};
    double* dst[3] = {ox, oy, oz};
    return launch_gather_packed(src, perm, n, dst, ws, ws_bytes, stream);
}

size_t cstone_build_workspace_bytes(size_t n, size_t leaf_capacity) {
    Carve c(nullptr);
    c.take<uint64_t>(n);  // unsorted keys
    c.take<BuildWords>(1);
    // the sort runs before the loop; the loop and the link share the stream
    // without a host check in between, so they get separate parts (the split
    // list of the loop is largest for n_crit = 1)
    size_t stage = std::max(prepared_sort_workspace_bytes(n),
                            rebalance_workspace_bytes(n, 1, leaf_capacity) + link_workspace_bytes(leaf_capacity));
    return c.off + stage;
}

cstone_status cstone_build(const double* x, const double* y, const double* z, size_t n, const cstone_box* box,
                           cstone_curve curve, uint32_t n_crit, uint64_t* sorted_keys, uint32_t* perm,
                           uint64_t* leaves, size_t* n_leaves, size_t leaf_capacity, uint32_t* counts,
                           uint64_t* node_keys, uint32_t* child, uint32_t* level_offsets, uint32_t max_iters,
                           uint32_t* iters_done, void* ws, size_t ws_bytes, cstone_timings* timings,
                           hipStream_t stream) {
    if (n > kMaxN || n_crit == 0 || !box_ok(box) || !leaves || !n_leaves || !ws) return CSTONE_ERR_INVALID_ARG;
    if (curve != CSTONE_MORTON && curve != CSTONE_HILBERT) return CSTONE_ERR_INVALID_ARG;
    if (n && (!x || !y || !z || !sorted_keys || !perm)) return CSTONE_ERR_INVALID_ARG;
    if ((node_keys == nullptr) != (child == nullptr) || (node_keys && !level_offsets)) return CSTONE_ERR_INVALID_ARG;
    if (leaf_capacity < 1 || *n_leaves > leaf_capacity) return CSTONE_ERR_INVALID_ARG;
    if (ws_bytes < cstone_build_workspace_bytes(n, leaf_capacity)) return CSTONE_ERR_INVALID_ARG;

    Carve c(ws);
    uint64_t* keys = c.take<uint64_t>(n);
    BuildWords* words = c.take<BuildWords>(1);
    uint32_t* flag = &words->flag;
    TreeState* tree_state = &words->tree;
    // the sort shape is looked up once: the key kernel's digit counts, the
    // sort's set-up and its passes must all use the same one
    const int variant = sort_resolve_variant(n);
    void* stage_ws = static_cast<char*>(ws) + c.off;
    const size_t stage_bytes = ws_bytes - c.off;

    hipEvent_t ev[5] = {};
    hipEvent_t pass_ev[9] = {};
    hipEvent_t low_ev = nullptr;  // low passes run after the first look: from here to ev[2]
    bool again = false;           // they did
    float first_ms[2] = {};       // then: the sort before them, and the tree that was of no use
    const int passes = sort_passes(n, 63, true, variant);
    const bool timed = timings != nullptr;
    auto cleanup = [&]() {
        for (auto& e : ev)
            if (e) (void)hipEventDestroy(e);
        for (auto& e : pass_ev)
            if (e) (void)hipEventDestroy(e);
        if (low_ev) (void)hipEventDestroy(low_ev);
    };
    if (timed) {
        if (hipEventCreate(&low_ev) != hipSuccess) return CSTONE_ERR_DEVICE;
        for (auto& e : ev)
            if (hipEventCreate(&e) != hipSuccess) { cleanup(); return CSTONE_ERR_DEVICE; }
        for (int i = 0; i <= passes; ++i)
            if (hipEventCreate(&pass_ev[i]) != hipSuccess) { cleanup(); return CSTONE_ERR_DEVICE; }
    }
    auto mark = [&](int i) -> hipError_t { return timed ? hipEventRecord(ev[i], stream) : hipSuccess; };
    cstone_status s = CSTONE_OK;
    uint32_t host_flag = 0;
    size_t nl = *n_leaves;
    do {
        if (mark(0) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
        // The key kernel goes first (a long launch, so the host's later
        // launches overlap it) and stores per-block counts of the sort's first
        // digit (of all three top digits for the split sort) and per-block
        // non-finite flags; the sort's set-up launch sums them, writes the
        // flag word and clears what the passes need cleared.
        if (n) {
            uint32_t *hist_parts = nullptr, *bad_parts = nullptr, hist_mask = 0, hist_shift = 0, parts = 0,
                     hist_digits = 1;
            sort_key_parts(stage_ws, n, true, 63, variant, &hist_parts, &bad_parts, &hist_mask, &hist_shift,
                           &hist_digits);
            s = launch_keys(x, y, z, n, *box, curve, keys, nullptr, stream, hist_parts, hist_mask, hist_shift,
                            bad_parts, &parts, hist_digits);
            if (s != CSTONE_OK) break;
            if (mark(1) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
            if ((s = sort_setup_from_keys(stage_ws, n, true, variant, parts, keys, flag,
                                          reinterpret_cast<uint64_t*>(tree_state), sizeof(TreeState) / 8, stream)) !=
                CSTONE_OK)
                break;
        } else {
            hipLaunchKernelGGL(clear_word_kernel, dim3(1), dim3(1), 0, stream, flag);
            if (mark(1) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
        }
        // The sort's low passes (five launches) rarely find a bucket to sort.
        // Where the host looks at the build's end anyway, they are only run if
        // it then sees one listed, and the tree once more; from kListMaxKeys on,
        // and where the tree's workspace would overwrite the list, they are always
        // enqueued.
        const bool direct = tree_possible(n, max_iters) && direct_pays(n, nl);
        const uint32_t* listed = nullptr;
        if (n && n < kListMaxKeys && direct &&
            tree_workspace_bytes(n, n_crit, leaf_capacity, nl > 1) <= sort_scratch_bytes(n))
            listed = sort_listed_word(stage_ws, n, variant);
        // the sort reports a failed device-side wait into the same flag word
        s = launch_sort(keys, sorted_keys, perm, n, 63, stage_ws, stage_bytes, stream,
                        timed && n ? pass_ev : nullptr, /*prepared=*/true, variant, flag, /*low_passes=*/!listed);
        if (s != CSTONE_OK) break;
        if (mark(2) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
        if (nl == 0) nl = 1;  // start from the root leaf {0, 8^L}
        bool done = false;
        if (direct) {  // tree and links are enqueued together, and the host looks once
            TreePass tree;
            if (tree.run(sorted_keys, n, n_crit, leaves, nl, leaf_capacity, counts, node_keys, child, level_offsets,
                         stage_ws, stage_bytes, tree_state, flag, listed, stream)) {
                if (mark(3) != hipSuccess || mark(4) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
                if ((s = tree.wait(&done)) != CSTONE_OK) break;
                if (tree.listed) {  // some buckets are not sorted yet: sort them, and the tree again
                    again = true;
                    if (timed && (hipEventElapsedTime(&first_ms[0], ev[1], ev[2]) != hipSuccess ||
                                  hipEventElapsedTime(&first_ms[1], ev[2], ev[3]) != hipSuccess ||
                                  hipEventRecord(low_ev, stream) != hipSuccess)) {
                        s = CSTONE_ERR_DEVICE;
                        break;
                    }
                    s = launch_sort_low(sorted_keys, perm, n, stage_ws, variant, flag, stream);
                    if (s != CSTONE_OK) break;
                    if (mark(2) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
                    tree.run(sorted_keys, n, n_crit, leaves, nl, leaf_capacity, counts, node_keys, child, level_offsets,
                             stage_ws, stage_bytes, nullptr, flag, nullptr, stream);
                    if (mark(3) != hipSuccess || mark(4) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
                    if ((s = tree.wait(&done)) != CSTONE_OK) break;
                }
                if (done) {
                    *n_leaves = tree.n_leaves;
                    if (iters_done) *iters_done = tree.rounds;
                    host_flag = tree.input_flags;
                }
            }
        }
        if (!done) {
            // The rounds and the link are enqueued together; the host looks
            // once, after the link, and only goes round again if the loop
            // needs more rounds.
            const size_t reb_bytes = rebalance_workspace_bytes(n, n_crit, leaf_capacity);
            void* link_ws = static_cast<char*>(stage_ws) + reb_bytes;
            const size_t link_bytes = stage_bytes - reb_bytes;
            RebalanceLoop loop;
            s = loop.begin(sorted_keys, n, n_crit, leaves, nl, leaf_capacity, counts, max_iters, stage_ws, reb_bytes,
                           stream, flag);
            if (s != CSTONE_OK) break;
            // The link is enqueued behind the first batch of rounds (usually the
            // last one), so one synchronisation serves both; if more rounds are
            // needed, it runs again once, after the last batch.
            bool finished = false, linked = false;
            for (uint32_t batch = 0; !finished; batch = 4) {
                if ((s = loop.enqueue(batch)) != CSTONE_OK) break;
                if (mark(3) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
                if (node_keys && batch == 0) {
                    s = launch_link(leaves, leaf_capacity, loop.device_leaf_count(), node_keys, child, level_offsets,
                                    link_ws, link_bytes, stream);
                    if (s != CSTONE_OK) break;
                    linked = true;
                }
                if (mark(4) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
                loop.wait(&finished);
                if (!finished) linked = false;
            }
            if (s != CSTONE_OK) break;
            if (node_keys && !linked && loop.status == CSTONE_OK) {  // the tree the first link saw was not the last
                if (mark(3) != hipSuccess) { s = CSTONE_ERR_DEVICE; break; }
                s = launch_link(leaves, leaf_capacity, loop.device_leaf_count(), node_keys, child, level_offsets,
                                link_ws, link_bytes, stream);
                if (s != CSTONE_OK) break;
                if (mark(4) != hipSuccess || hipStreamSynchronize(stream) != hipSuccess) {
                    s = CSTONE_ERR_DEVICE;
                    break;
                }
            }
            *n_leaves = loop.n_leaves;
            if (iters_done) *iters_done = loop.rounds;
            host_flag = loop.input_flags;
            s = loop.status;
        }
        if (host_flag & ~CSTONE_FLAG_NONFINITE) { s = CSTONE_ERR_DEVICE; break; }  // the sort gave up a wait
        if (host_flag & CSTONE_FLAG_NONFINITE) { s = CSTONE_ERR_NONFINITE; break; }
        if (s != CSTONE_OK) break;
        if (timed) {
            for (int i = 0; i < 4; ++i)
                if (hipEventElapsedTime(&timings->stage_ms[i], ev[i], ev[i + 1]) != hipSuccess) s = CSTONE_ERR_DEVICE;
            timings->sort_passes = n ? static_cast<uint32_t>(passes) : 0u;
            for (int p = 0; p < 8; ++p) timings->sort_pass_ms[p] = 0.f;
            for (int p = 0; n && p < passes; ++p)
                if (hipEventElapsedTime(&timings->sort_pass_ms[p], pass_ev[p], pass_ev[p + 1]) != hipSuccess)
                    s = CSTONE_ERR_DEVICE;
            if (again) {  // a split sort: its last entry is the low passes
                float low = 0.f;
                if (hipEventElapsedTime(&low, low_ev, ev[2]) != hipSuccess) s = CSTONE_ERR_DEVICE;
                timings->sort_pass_ms[passes - 1] = low;
                timings->stage_ms[1] = first_ms[0] + low;
                timings->stage_ms[2] += first_ms[1];
            }
        }
    } while (false);
    cleanup();
    return s;
}

}  // extern "C"
