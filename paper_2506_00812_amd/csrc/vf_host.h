// Host-side state of the library: the index object behind the C ABI of include/vecflow.h, its
// per-stream workspaces, the tuning switches, and the functions the host source files share.
// Nothing here is part of the C ABI.
#pragma once

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/vecflow.h"
#include "vf_internal.h"

namespace vf {

#define VF_HIP(expr)                                                                                   \
    do {                                                                                               \
        hipError_t e_ = (expr);                                                                        \
        if (e_ != hipSuccess) {                                                                        \
            ::vf::set_error(std::string(#expr) + ": " + hipGetErrorString(e_));                        \
            return e_ == hipErrorOutOfMemory ? VF_ENOMEM : VF_EHIP;                                    \
        }                                                                                              \
    } while (0)

#define VF_REQUIRE(cond, msg)                 \
    do {                                      \
        if (!(cond)) {                        \
            ::vf::set_error(msg);             \
            return VF_EINVAL;                 \
        }                                     \
    } while (0)

// Runs the body of an extern "C" entry point: no exception crosses the ABI.
template <class F> int guarded(F &&body) noexcept
{
    try {
        return body();
    } catch (const std::bad_alloc &) {
        set_error("out of host memory");
        return VF_ENOMEM;
    } catch (const std::exception &e) {
        set_error(std::string("internal error: ") + e.what());
        return VF_EINTERNAL;
    } catch (...) {
        set_error("internal error (unknown exception)");
        return VF_EINTERNAL;
    }
}

// Where the index's device memory comes from: the allocator the caller gave to vf_build_index, or
// hipMalloc / hipFree.
struct DeviceAllocator {
    vf_allocator user{};   // user.alloc == nullptr: hipMalloc / hipFree
    int64_t live_bytes = 0, peak_bytes = 0;
    int alloc(void **p, size_t bytes);
    void release(void *p, size_t bytes);
};

struct DevBuf {
    void *p = nullptr;
    size_t cap = 0;
    DeviceAllocator *al = nullptr;   // nullptr: hipMalloc / hipFree
    DevBuf() = default;
    explicit DevBuf(DeviceAllocator *a) : al(a) {}
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    // Grows the buffer to at least `bytes` (contents are not kept); never shrinks.
    int reserve(size_t bytes);
    void release();
    template <class T> T *as() const { return (T *)p; }
};

// Releases temporaries on every exit path of a function.
struct DevBufGuard {
    std::vector<DevBuf *> bufs;
    DevBufGuard(std::initializer_list<DevBuf *> b) : bufs(b) {}
    ~DevBufGuard() { for (DevBuf *b : bufs) b->release(); }
};

// Switches and sizes that experiments and tests may change (vf_tune); the defaults are the measured optima.
// An index copies the process-wide defaults when it is built; afterwards it has its own.
struct Tuning {
    int seg_groups = 16;          // 32-vector groups per scan-list segment
    int seg_groups_heavy = 16;    // the same for tiles of >= heavy_rows queries
    int heavy_rows = 9;
    int tile_rows = 16;           // queries per scan tile
    // a per-call routing blob up to this size is read in place from pinned host memory: a call of 1,000 queries saves the
    // copy, its event and a wait, 105 -> 80 us; at 10,000 queries the reads cost more than that (216 -> 222 us)
    int zero_copy_bytes = 32768;
    int scan_valu = 1;            // float32 FMA scan kernel: 0 never, 1 for batches of <= 256 scan queries, 2 always
    int scan16 = 1;               // 0: float32 search tiles keep the 32-row matrix-core kernel
    int scan_bf16 = 1;            // float32 lists of large batches: filter from the bfloat16 copy, re-rank exactly (0: off)
    int scan_bf16_margin = 22;    // approximations kept beyond k per query and segment by that filter
    int scan_bf16_slots = 1;      // list groups a wave of that filter keeps in flight (1 or 2)
    int scan_bf16_seg_groups = 24;   // 32-vector groups per list segment when that filter runs (half the bytes per group)
    int beam_lat_waves = 1024;    // beam launches of up to this many graph queries (float32 without predicates: twice as many) use the latency instantiation; 0: never
    int overlap = 1;              // 0: the scan path runs on the caller's stream, before the graph path
    int seed_exact = 0;           // 1: seeds are scored by the ordered-distance kernel, never on the matrix cores
    double seed_slack = 1.0;      // scales the rounding-error bound of the float32 seed proofs
    int seed_margin = 8;          // approximations kept beyond itopk for re-ranking (float32 copy of the seeds)
    int seed_margin_bf16 = 24;    // the same from the 16-bit (binary16) copy
    int seed_cache = 1;           // 0: no interleaved copy of the seeds, the seed kernel gathers rows
    int seed_bf16 = 1;            // 0: float32 data keep only the float32 copy of the seeds, not the 16-bit one
    // Calls with fewer graph queries use the float32 copy when it is resident.  Without predicates neither is the better one by much (a batch
    // of 64, 6,144 seeds: binary16 1 - 4 % faster); predicates' proofs re-score 16 seeds fewer from the float32 copy, which
    // a few queries notice (one pair 66 against 72 us), and from some 256 pairs on binary16 is ahead.
    int seed_bf16_min_batch = 512;
    int seed_fb_window = 131072;  // graph queries between two looks at the failed-proof counter
    int seed_select = 0;          // 1: the seed kernel also selects (runs of keys instead of every distance; itopk <= 64)
    int seed_seg_seeds = 0;       // seeds per wave of the selecting seed kernel; 0: chosen per call (512 .. 16384)
    int build16 = 1;              // 0: float32 kNN self-joins on the 32-row scan kernel, list by list, not on the join kernel
    int build_panel_kb = 4096;    // 16-row self-joins of long lists (tables the join's proofs do not cover) go panel by panel, this much of the list per launch
    int build_progress = 0;       // 1: a line on stderr every ten seconds while graphs are built
    // returns false for an unknown name or a value out of range
    bool set(const char *name, double value);
};
Tuning &default_tuning();
std::mutex &default_tuning_mutex();

struct Staging {  // pinned host blob + the event that says its last upload has finished
    void *p = nullptr;
    size_t cap = 0;
    hipEvent_t done = nullptr;
    bool pending = false;
};

// Result of routing one batch (host side) and the scratch it reuses between calls.
struct Routed {
    std::vector<int32_t> gq_query, gq_label;          // graph queries, grouped by label (ascending), stable in query order
    std::vector<int32_t> others_off, others;          // [nq+1], AND partner labels per query
    std::vector<uint64_t> scan_pairs;                 // (label << 32 | query) of scan queries, ascending
    std::vector<int32_t> xq_query, xq_label;          // AND queries on short graph lists that are answered exactly
    bool any_and = false;
    // scratch kept between calls
    std::vector<int32_t> q_best;                      // searched label of each query, -1: empty result
    std::vector<int32_t> empty_q;                     // queries with q_best == -1
    std::vector<int32_t> cnt;                         // [n_labels] queries per searched label (zero between calls)
    std::vector<int32_t> touched;                     // [n_labels + 1] labels with cnt > 0, first
    std::vector<uint64_t> label_bits;                 // ... while they are put in order
    std::vector<int32_t> order;                       // queries grouped by label
};

// What routing needs to know of an index (a view, so that routing can be exercised without a device).
struct RouteView {
    const int32_t *S;     // [n_labels] posting-list sizes
    int32_t n_labels, T;
};

// ClassifyQueries (Alg. 2) + smallest-list choice (Section 4.3.2).  all_scan: every list is scanned (exact
// mode); first_is_searched: a query searches the list of its first label, the others are the predicate.
int route_queries(const RouteView &ix, int64_t nq, const int64_t *qoff, const int32_t *qids, bool all_scan,
                  bool first_is_searched, Routed &r);

// Work list of the scan path: the (label, query) pairs of one label are cut into tiles of <= tile_rows
// queries; a long list is cut into segments of whole 32-vector groups so that many waves share it, and a
// merge item per query then combines the segments.
constexpr int kMaxSegs = 64;
struct ItemBuilder {
    std::vector<int32_t> qrow;
    std::vector<ScanItem> items;
    std::vector<MergeItem> merges;
    int64_t part_rows = 0;
    int32_t max_nseg = 1;
    int32_t tile_rows = 16, seg_groups = 16, seg_groups_heavy = 16, heavy_rows = 9;
    bool all_partial = false;   // every item writes partial rows and every query gets a merge item (one-segment lists too)
    explicit ItemBuilder(const Tuning &t)
        : tile_rows(t.tile_rows), seg_groups(t.seg_groups), seg_groups_heavy(t.seg_groups_heavy), heavy_rows(t.heavy_rows) {}
    // pairs[lo, hi) all carry the same label, whose list is (group0, map_off, n)
    void add_label(const std::vector<uint64_t> &pairs, size_t lo, size_t hi, int64_t group0, int64_t map_off, int32_t n);
};

// Everything a call writes besides its outputs.  An index has kWorkspaces of them and hands one to each
// stream that calls it, so that calls on different streams can overlap on the GPU (small batches leave most
// of the chip idle); calls on one stream share one workspace and run in order.
// The work lists of a call's plan, kept for the next call's (what they hold is not; new ones are half a megabyte of page faults)
struct PlanStore {
    std::vector<int32_t> qrow;
    std::vector<ScanItem> items;
    std::vector<MergeItem> merges;
    std::vector<SeedTile> tiles;
    template <class Plan> void swap_with(Plan &P)
    {
        qrow.swap(P.ib.qrow); items.swap(P.ib.items); merges.swap(P.ib.merges); tiles.swap(P.tiles);
    }
    void clear() { qrow.clear(); items.clear(); merges.clear(); tiles.clear(); }
};

struct Workspace {
    PlanStore plan;
    DevBuf ws_blob, ws_blob_b;
    DevBuf dseed;   // seed distances, then partial result rows
    // vf_search_multi: gathered query rows, results of the sub-searches
    DevBuf multi_q, multi_ids, multi_dists;
    std::vector<int32_t> multi_host;      // [n_sub parents | nq + 1 first sub-search of each query]
    std::vector<int32_t> multi_first;
    std::vector<int64_t> multi_qoff;
    std::vector<int32_t> multi_qids;
    // the scan path runs beside the graph path on a second stream of the same (default) priority
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    bool prev_forked = false;   // the previous call on this workspace ran its scan path on the side stream
    int blob_next = 0;   // the device blob alternates between two buffers
    Staging stage[2];
    int stage_next = 0;
    Routed routed;
    bool ready = false;          // stream and events exist
    bool owned = false;
    hipStream_t owner = nullptr; // the stream whose calls use this workspace
    std::vector<DevBuf *> bufs()
    {
        return {&ws_blob, &ws_blob_b, &dseed, &multi_q, &multi_ids, &multi_dists};
    }
};

// The seeds of every graph list for one n_seeds (local ids floor(j n / ns)), interleaved like a scan list, so
// that the matrix-core seed kernel reads its B operand with coalesced loads.  Derived from the index and
// n_seeds alone.  An index keeps a few of them (calls on different streams may use different seed counts at
// the same time); a copy is only rebuilt or dropped after the whole device has drained, which dimensions without a kernel
// instantiation of their own never ask for: they keep the first ones and score any further seed count without a copy.
struct SeedCopy {
    int32_t n_seeds = -1;        // -1: slot unused
    bool ok = false;             // false: the copy did not fit, the kernel gathers rows from the vector table
    bool has_f32 = false;        // blk is valid
    bool has_f16 = false;        // blk16 is valid (float32 data only)
    float f16_delta = 0.f;       // upper bound of the rounding errors |x - x^| of the seeds of the copy
    uint64_t last_use = 0;
    DevBuf blk, blk16, norm;
    DevBuf goff;                 // first group of each graph list, and behind them the tables that the copy was made from
    DevBuf map;                  // [group * 32 + v] global id of the seed (AND predicate inside the seed kernel)
    std::vector<DevBuf *> bufs() { return {&blk, &blk16, &norm, &goff, &map}; }
};

}  // namespace vf

struct vf_index {
    vf::DeviceAllocator alloc;
    vf::Tuning tune;
    int dtype = 0;
    int64_t n = 0;
    int32_t dim = 0, n_labels = 0, T = 0, R = 0, ncp = 0;
    int32_t graph_kind = 0, knn_degree = 0;
    const void *X = nullptr;
    // host metadata
    std::vector<int32_t> S, hs_slot;
    std::vector<int64_t> O_HS, O_LS, GO_LS;
    std::vector<int32_t> graph_labels;
    int64_t n_HS = 0, n_LS = 0, n_groups_LS = 0, bitset_words = 0;
    int32_t n_scan_labels = 0;
    // device
    vf::DevBuf d_S, d_O_HS, d_O_LS, d_hs_slot, d_M_HS, d_M_LS, d_G, d_X_LS, d_xnorm_LS, d_bitsets;
    // float32 data: the scan lists once more in bfloat16 (16-byte chunks of 8 components, half the bytes), which the
    // filtering scan kernel streams; ls_bf16_delta = max |x - bf16(x)| over the lists' vectors (its error bound)
    vf::DevBuf d_X_LS16, d_scan_fb;    // d_scan_fb: [0] failed proofs, [1] refused queries of the ground-truth call that runs
    bool refused_unread = false;       // [1] may not be zero (a call failed between)
    bool has_ls16 = false;
    float ls_bf16_delta = 0.f, ls_xn_max = 0.f;   // ... and the largest squared norm of a list vector
    uint32_t scan_fb_seen = 0;   // failed proofs already reported (d_scan_fb counts them on the device)
    vf::DevBuf d_Gg;   // [n_HS][R] the graph rows once more with global ids: saves the search one dependent load per expansion
    // indexes with graph labels: squared norm of every row of X and the largest of them, for the matrix-core
    // seed scoring (its error bound needs the largest norm)
    vf::DevBuf d_xnorm_all;
    float xn_max = 0.f;
    // float32: the join kernel's origin (a vector near the mean of X), the squared norms of all rows measured from it and the
    // largest of them (0: the table's norms are outside the proofs' range, nothing is joined)
    vf::DevBuf d_centre, d_xnorm_c;
    // float32 self-joins on binary16 operands; off from the batch of lists on where a look at 256 rows left 1 in 16 without a proof,
    // or the join 1 in 64
    bool join_single = true;
    // ... and ground truth, of at most so many results: set by a build that kept to binary16 and whose rows would nearly all have
    // been proven as queries, whose own rounding is not known (0: two parts).  No call changes it.
    int32_t exact_single_k = 0;
    float xc_max = 0.f, xc_rho = 0.f;   // (... and the largest relative error of a centred row rounded to 11 bits)
    bool seed_mfma_ok = false;   // the norms exist and are finite: seeds may be scored on the matrix cores
    // search workspaces (see Workspace); profiled calls and vf_search_exact must not overlap with other calls
    static constexpr int kWorkspaces = 8;
    vf::Workspace ws[kWorkspaces];
    int ws_steal = 0;
    std::recursive_mutex mu;     // host side of every call
    vf::Routed noalloc_routed;   // host-side scratch of vf_search_noalloc (kept between calls)
    std::vector<char> noalloc_blob;
    vf::DevBuf tmp_blk, tmp_norm, counters;
    static constexpr int kSeedCopies = 4;
    vf::SeedCopy seed_copies[kSeedCopies];
    uint64_t seed_tick = 0;
    // Watch on the 16-bit form of the seed copies: queries whose proof failed are counted on the device; the
    // count is fetched every tune.seed_fb_window graph queries, the first time after kFirstLook, and read at a later call.
    // More than 1/64 failures (a failed proof costs its query a gather of every seed): calls that have ordered distances to go
    // back to -- dimensions without a kernel instantiation of their own, lists of more than 48 entries -- do so, and after a
    // whole window the others' copies are rebuilt in float32.
    bool seed_proofs_off = false;
    bool seed_bf16_off = false;
    vf::DevBuf d_fb_count;
    uint32_t *h_fb = nullptr;    // pinned
    hipEvent_t ev_fb = nullptr;
    bool fb_pending = false, fb_looked = false, fb_first = false;   // a count is on its way; one was; it is the first
    uint32_t fb_last = 0;
    int64_t fb_window_q = 0, fb_sent_q = 0;
    // profiling
    bool profiling = false, prof_valid = false;
    // a ring of event sets (scan begin/end, graph begin, seeds end, beam end), one set per profiled call:
    // a call never waits for an earlier one unless kProfRing calls are still unread
    static constexpr int kProfRing = 64;
    hipEvent_t prof_ring[kProfRing][5] = {};
    hipEvent_t *prof_ev = prof_ring[0];   // the set of the call being issued
    int prof_next = 0, prof_unfolded = 0; // next ring slot; recorded sets whose durations are not in the sums yet
    bool prof_serial = false;  // vf_profile_enable(index, 2): every launch on the caller's stream
    bool prof_exact_counts = false;   // ... | 4: count the seeds that pass each AND query's predicate before every call
    vf_profile prof{};
    std::vector<int32_t> prof_graph_queries;   // graph-routed queries of the last profiled call
    double prof_scan_sum = 0, prof_seed_sum = 0, prof_beam_sum = 0;
    double prof_host_plan = 0, prof_host_blob = 0, prof_host_launch = 0, prof_host_wait = 0;   // host milliseconds inside profiled calls
    int64_t prof_calls = 0;

    vf_index();
    std::vector<vf::DevBuf *> bufs()
    {
        return {&d_S, &d_O_HS, &d_O_LS, &d_hs_slot, &d_M_HS, &d_M_LS, &d_G, &d_Gg, &d_X_LS, &d_xnorm_LS, &d_bitsets,
                &d_xnorm_all, &d_centre, &d_xnorm_c, &tmp_blk, &tmp_norm, &counters, &d_fb_count, &d_X_LS16, &d_scan_fb};
    }
    vf::LabelMeta meta() const
    {
        vf::LabelMeta m;
        m.S = d_S.as<int32_t>(); m.O_HS = d_O_HS.as<int64_t>(); m.O_LS = d_O_LS.as<int64_t>();
        m.hs_slot = d_hs_slot.as<int32_t>(); m.M_HS = d_M_HS.as<int32_t>(); m.M_LS = d_M_LS.as<int32_t>();
        m.bitsets = d_bitsets.as<uint32_t>(); m.bitset_words = bitset_words;
        return m;
    }
    vf::RouteView route_view() const { return vf::RouteView{S.data(), n_labels, T}; }
    size_t elem() const { return dtype == VF_U8 ? 1 : 4; }
    size_t group_bytes() const { return (size_t)2 * ncp * 32 * 16; }
    // float32 seed proofs: |approximation - ordered distance| <= seed_err_bound() (|q|^2 + xn_max)
    float seed_err_bound() const { return (float)(tune.seed_slack * 3.0517578125e-05); }
    // the power of two that brings the largest norm into [32, 64): binary16 operands
    static float half_scale(float norm2)
    {
        int e;
        (void)std::frexp(std::sqrt(norm2), &e);
        return std::ldexp(1.f, 6 - e);
    }
    float seed_scale() const { return xn_max > 0.f ? half_scale(xn_max) : 1.f; }
    // Whether the proofs of approximate seeds can be expected to hold: their bound is relative to the norms, and on a table far from
    // the origin it lets most seeds through, while ordered distances take the same time wherever the table is.  Clusters of 100
    // components shifted by 3 / 5 / 8 / 12 / 20 times their width (norms, squared, over those from the mean: 2.8, 6, 14, 30, 81): 64
    // queries x 4,096 seeds 49 / 49 / 50 / 52 / 66 us, ordered 81, AND pairs 78 / 76 / 76 / 77 / 259 and 99, 1,200 x 1,000 61 / 62 / 63 / 63 /
    // 118 and 104; lists of 64 58 / 60 / 72 / 251 / 245 and 86, 4,000 x 2,500 125 / 124 / 384 / - / - and 276.  Clusters that are
    // up to 100 times further apart than they are wide, or of 200 copies each, take as long as near ones.
    bool seeds_provable(int32_t itopk) const { return dtype == VF_U8 || xn_max <= (itopk > 48 ? 5.0f : 20.0f) * xc_max; }
    // squared norms the join kernel takes for its lists
    const uint32_t *join_norms() const { return dtype == VF_U8 ? d_xnorm_all.as<uint32_t>() : d_xnorm_c.as<uint32_t>(); }
    // the operands of a self-join, and of a join of queries
    int join_kind() const { return dtype == VF_U8 ? vf::kJoinU8 : join_single ? vf::kJoinSingle : vf::kJoinSplit; }
    int exact_kind(int32_t k) const { return dtype == VF_U8 ? vf::kJoinU8 : k <= exact_single_k ? vf::kJoinSingle : vf::kJoinSplit; }
    // ... and those that the packed lists' buffer is sized for
    int join_kind_max() const { return dtype == VF_U8 ? vf::kJoinU8 : vf::kJoinSplit; }
    // the same for the approximations of the join kernel (norms from its origin, see vf_join.hip); what it decides is
    // stored or is the ground truth: "seed_slack" below 1 does not make its proofs weaker
    float join_err_bound(int kind) const
    {
        return (float)(std::max(1.0, tune.seed_slack) * ((512 + 4 * dim) * 5.9604644775390625e-08 + (kind == vf::kJoinSingle ? 1.220703125e-04 : 0.0)));
    }
    // ... and what is proportional to |q|: the rounding of both operands to 11 bits, the table's rows by at most xc_rho of
    // their length, any vector by 2^-11 (own: the rows are the table's)
    float join_err_q(int kind, bool own) const
    {
        return kind == vf::kJoinSingle ? 2.01f * (xc_rho + (own ? xc_rho : 4.8828125e-04f)) * std::sqrt(xc_max) : 0.f;
    }
    // its scale is that of the centred norms
    float join_scale(int kind) const { return kind == vf::kJoinSingle && xc_max > 0.f ? half_scale(xc_max) : 1.f; }
};

namespace vf {

template <class T> int upload(DevBuf &b, const std::vector<T> &v, hipStream_t s)
{
    int rc = b.reserve(std::max<size_t>(v.size() * sizeof(T), 16));
    if (rc != VF_OK) return rc;
    if (!v.empty()) VF_HIP(hipMemcpyAsync(b.p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s));
    return VF_OK;
}

// vf_search.hip: the pieces of one search call
struct BlobLayout {
    size_t off_gq_query, off_gq_label, off_xq_query, off_xq_label, off_others_off, off_others, off_qrow, off_items, off_merges, off_tiles, off_empty, off_jlists, off_multi, total;
};

// Everything the host decides about a call before anything is launched.
struct HsRun { int32_t label; size_t item_lo, item_hi; };   // exact mode: the scan items of one graph list
// exact mode on the join kernel: graph lists packed together, their positions in CallPlan::jlists and their items
struct JoinBatch { size_t list_lo, list_hi, item_lo, item_hi; int64_t groups; };
struct CallPlan {
    int64_t nq = 0;
    int32_t k = 0, itopk = 0, width = 0, iters = 0, n_seeds = 0;
    bool exact = false;
    bool tight = false;                   // temporaries live in a fixed array: nothing is spent on more segments or minima
    int32_t beam_LP = 128, beam_hb = 9;   // beam kernel geometry: list slots and visited-table size
    int32_t ns_top = 0;                   // seeds a list may have
    int32_t ns_stride = 0;                // row length of the seed distance matrix
    int32_t nb_stride = 0;                // > 0: the seed kernel leaves the minima of its 32-seed blocks too, rows of this length
    ItemBuilder ib;
    size_t n_ls_items = 0, n_ls_merges = 0;
    std::vector<HsRun> hs_runs;
    int32_t max_hs_list = 0;
    // ... the same on the join kernel (vf_join.hip): join_keep candidates per partial row, whose rows follow ls_part_words
    std::vector<JoinList> jlists;
    size_t join_bytes = (size_t)1 << 30;  // packed lists of a batch (a list that is larger goes by itself); 0: nothing is joined
    std::vector<JoinBatch> jbatches;
    int64_t join_groups = 0;              // of the largest batch
    int32_t join_keep = 0, join_max_nseg = 1;
    int join_kind = kJoinU8, join_tile = kJoinRows;
    size_t join_bound_at = 0, join_first_row = 0, join_rows = 0;   // the rows' shared bounds, among the partial rows' bits
    size_t ls_part_words = 0;
    std::vector<SeedTile> tiles;          // dense seed scoring: tiles of <= 64 (32) graph queries of one label
    size_t n_gq = 0;
    size_t n_xq = 0;                      // AND queries answered by the exact predicate scan of a short graph list
    bool dense_seeds = false, seeds_mfma = false;
    // seeds_mfma with the selection fused into the seed kernel: runs of sel_K keys per (query, segment)
    bool seed_select = false, sel_f16 = false, seeds_f16 = false;
    int32_t sel_K = 0, seg_seeds = 0, max_segs = 0;
    BlobLayout L{};
    size_t dseed_words = 0;               // seed distance matrix
    size_t part_words = 0;                // partial result rows x k (x scan_keep with the bfloat16 filter)
    // float32 scan lists filtered from their bfloat16 copy and re-ranked
    bool scan_bf16 = false;
    int32_t scan_keep = 0;                // approximations kept per (query, segment)
    explicit CallPlan(const Tuning &t) : ib(t) {}
};

// Where a call's device-side temporaries live (a workspace's buffers, or the static scratch array of the entry
// point that allocates nothing).
struct CallMem {
    char *blob = nullptr;          // device address of the routing blob
    uint32_t *dseed = nullptr;
    int32_t *part_idx = nullptr;
    uint32_t *part_bits = nullptr;
    int32_t *refused = nullptr;    // ground truth: see RerankParams::refused
    uint32_t *refused_any = nullptr;
};

int check_search_args(const vf_index *ix, const void *queries, int64_t nq, int32_t k, const int64_t *out_ids,
                      const float *out_dists);
int check_search_params(const vf_index *ix, bool exact, int32_t k, int32_t &itopk, int32_t width, int32_t iters,
                        int32_t &n_seeds);
// How many words a call's seed distances may take.  words: what is allocated or fixed; beyond that, where the buffer may
// grow (cap: its bytes), into at most half of the free memory -- the driver is only asked by a call that needs it, the
// query is slow.
struct SeedBudget {
    uint64_t words = 0;
    bool grows = false;
    size_t cap = 0;
    bool fits(uint64_t need)
    {
        if (need <= words || !grows) return need <= words;
        grows = false;
        size_t free_b = 0, total_b = 0;
        if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) { (void)hipGetLastError(); return false; }
        words = std::max<uint64_t>(words, (uint64_t)((free_b + cap) / 2) / 5);   // / 4 bytes, / 1.25 growth
        return need <= words;
    }
};
// Who may make a copy of the seeds (see seed_copy_for), and on which stream.
struct SeedCopyMaker {
    vf_index *ix;
    hipStream_t stream;
};
// sc: the resident copy of the seeds for n_seeds, if there is one; where there is none and the call would score from it, it is made
// (make == nullptr: nothing is).
int plan_call(const vf_index *ix, Routed &r, int64_t nq, const int64_t *qoff, const int32_t *qids, bool exact,
              bool first_is_searched, int32_t k, int32_t itopk, int32_t width, int32_t iters, int32_t n_seeds,
              int32_t and_scan_limit, SeedBudget budget, const SeedCopyMaker *make, SeedCopy *&sc, CallPlan &P);
// May this call's seeds be scored on the matrix cores (so that an interleaved seed copy is worth having)?
bool wants_seed_copy(const vf_index *ix, bool exact, int32_t itopk, int32_t n_seeds);
// The resident copy for n_seeds, or (build = true) a new one; *out stays null when there is none.
int seed_copy_for(vf_index *ix, int32_t n_seeds, hipStream_t s, bool build, SeedCopy **out);
int build_seed_copy(vf_index *ix, int32_t n_seeds, hipStream_t s, bool want_f16, bool keep_f32, SeedCopy *c);
void half_bound(const vf_index *ix, float delta, BeamParams &b);
void fill_blob(const CallPlan &P, const Routed &r, char *hp);
int launch_call(vf_index *ix, const CallPlan &P, const Routed &r, const CallMem &M, const SeedCopy *sc, const void *queries,
                int64_t *out_ids, float *out_dists, hipStream_t s, hipStream_t side, hipEvent_t ev_fork,
                hipEvent_t ev_join, bool may_allocate);

// vf_index_build.hip
int build_index_impl(const void *vectors, int dtype, int64_t n, int32_t dim, const int64_t *label_offsets,
                     const int32_t *label_ids, int32_t n_labels, int32_t T, int32_t graph_degree, int32_t graph_kind,
                     int32_t knn_degree, const vf_allocator *allocator, void *hip_stream, vf_index **out);
void free_index(vf_index *ix);

// vf_search.hip
// What vf_search_multi adds to the batch of its sub-searches: their queries are gathered from `rows` before it, their
// results merged into out_* after it.
struct MultiCall {
    const std::vector<int32_t> *host;   // [n_sub parents | nq + 1 first sub-search of each query]
    const void *rows;
    int64_t nq;
    int64_t *out_ids;
    float *out_dists;
};
int search_impl(vf_index *ix, const void *queries, int64_t nq, const int64_t *qoff, const int32_t *qids, int32_t k,
                int32_t itopk, int32_t width, int32_t iters, int32_t n_seeds, bool exact, int64_t *out_ids,
                float *out_dists, hipStream_t s, bool first_is_searched = false, int32_t and_scan_limit = 0,
                const MultiCall *multi = nullptr);
int search_multi_impl(vf_index *ix, const void *queries, int64_t nq, const int64_t *qoff, const int32_t *qids,
                      int32_t mode, int32_t k, int32_t itopk, int32_t width, int32_t iters, int32_t n_seeds,
                      int64_t *out_ids, float *out_dists, hipStream_t s);
int fold_profile(vf_index *ix, int count);
// Drops every interleaved seed copy (after the device has drained): they are rebuilt on demand.
int drop_seed_copies(vf_index *ix);

// LDS bytes of the scan kernels for a tile (host-side check before a launch)
size_t scan_lds_bytes(int32_t ncp, int32_t tile_rows, int32_t K);

}  // namespace vf
