// Index construction (Alg. 1): posting lists, the HS / LS split at threshold T, the compacted S / O / M arrays
// of each partition, the interleaved scan lists of Section 4.2.2, membership bitsets for the AND predicate of
// Section 4.3.2, and one proximity graph per graph list (Section 4.2.1).  Also the index's memory management.
#include <ctime>

#include "vf_host.h"

namespace vf {

int DeviceAllocator::alloc(void **p, size_t bytes)
{
    *p = nullptr;
    if (user.alloc != nullptr) {
        void *q = user.alloc(bytes, user.ctx);
        if (q == nullptr) {
            set_error("the caller's device allocator returned NULL for " + std::to_string(bytes) + " bytes");
            return VF_ENOMEM;
        }
        if (((uintptr_t)q & 255) != 0) {
            user.free(q, user.ctx);
            set_error("the caller's device allocator returned memory that is not 256-byte aligned");
            return VF_EINVAL;
        }
        *p = q;
    } else {
        VF_HIP(hipMalloc(p, bytes));
    }
    live_bytes += (int64_t)bytes;
    peak_bytes = std::max(peak_bytes, live_bytes);
    return VF_OK;
}

void DeviceAllocator::release(void *p, size_t bytes)
{
    if (p == nullptr) return;
    if (user.alloc != nullptr) {
        // the allocator may hand the block to someone else at once: everything that used it must have completed
        // (hipFree waits for the device by itself)
        (void)hipDeviceSynchronize();
        user.free(p, user.ctx);
    } else {
        (void)hipFree(p);
    }
    live_bytes -= (int64_t)bytes;
}

int DevBuf::reserve(size_t bytes)
{
    if (bytes <= cap) return VF_OK;
    // a first allocation is exact (index arrays are sized once); a buffer that grows takes a quarter more than
    // asked, so that a workspace settles after a few calls
    const bool grows = p != nullptr;
    release();
    const size_t want = grows ? bytes + bytes / 4 + 256 : ((bytes + 255) & ~(size_t)255);
    if (al != nullptr) {
        int rc = al->alloc(&p, want);
        if (rc != VF_OK) return rc;
    } else {
        VF_HIP(hipMalloc(&p, want));
    }
    cap = want;
    return VF_OK;
}

void DevBuf::release()
{
    if (p != nullptr) {
        if (al != nullptr) al->release(p, cap);
        else (void)hipFree(p);
    }
    p = nullptr;
    cap = 0;
}

}  // namespace vf

using namespace vf;

vf_index::vf_index()
{
    for (DevBuf *b : bufs()) b->al = &alloc;
    for (Workspace &w : ws)
        for (DevBuf *b : w.bufs()) b->al = &alloc;
    for (SeedCopy &c : seed_copies)
        for (DevBuf *b : c.bufs()) b->al = &alloc;
}

namespace vf {

void free_index(vf_index *ix)
{
    if (!ix) return;
    // memory goes back to the allocator only after everything that used it has completed
    (void)hipDeviceSynchronize();
    for (DevBuf *b : ix->bufs()) b->release();
    for (SeedCopy &c : ix->seed_copies)
        for (DevBuf *b : c.bufs()) b->release();
    for (auto &set : ix->prof_ring)
        for (hipEvent_t e : set)
            if (e) (void)hipEventDestroy(e);
    if (ix->ev_fb) (void)hipEventDestroy(ix->ev_fb);
    if (ix->h_fb) (void)hipHostFree(ix->h_fb);
    for (Workspace &w : ix->ws) {
        for (DevBuf *b : w.bufs()) b->release();
        if (w.ev_fork) (void)hipEventDestroy(w.ev_fork);
        if (w.ev_join) (void)hipEventDestroy(w.ev_join);
        if (w.side) (void)hipStreamDestroy(w.side);
        for (Staging &s : w.stage) {
            if (s.done) (void)hipEventDestroy(s.done);
            if (s.p) (void)hipHostFree(s.p);
        }
    }
    delete ix;
}

constexpr int kLookRows = 256;   // rows that tell which operands a batch of self-joins takes, 32 of each of the eight longest lists

// Exact kNN rows of the graph lists graph_labels[lo, hi), which lie one after the other in M_HS: pack them, contract every
// list against itself in one launch (vf_join.hip; a list of a few thousand vectors alone would leave most of the chip
// idle), keep K candidates per vertex and order `deg` of them into rows_out (per list [|C_l|][deg] local ids).
// rows_out: row of the first vertex; global_ids as in build_graph_for_label.  for_queries: stays true while binary16 operands have
// proven nearly all rows, and would have with a query's bound.
static int build_graphs_joined(vf_index *ix, size_t lo, size_t hi, int32_t K, int32_t deg, int32_t *rows_out, bool global_ids,
                               DevBuf &cand_idx, DevBuf &cand_dist, DevBuf &d_items, bool &for_queries, hipStream_t s)
{
    const int64_t base0 = ix->O_HS[(size_t)ix->graph_labels[lo]];
    std::vector<JoinList> lists;
    std::vector<ScanItem> items;
    int64_t n_groups = 0;
    for (size_t i = lo; i < hi; ++i) {
        const int32_t l = ix->graph_labels[i], nl = ix->S[(size_t)l];
        const int64_t base = ix->O_HS[(size_t)l], group0 = n_groups;
        lists.push_back(JoinList{base, (int32_t)group0, nl});
        n_groups += (nl + 31) / 32;
        for (int32_t e = 0; e < nl; e += kJoinRowsShared) {
            ScanItem it{};
            it.group0 = group0; it.n = nl;
            it.q_begin = (int32_t)(base - base0 + e); it.q_count = std::min(kJoinRowsShared, nl - e);
            it.self_base = e; it.part_row = it.q_begin;
            items.push_back(it);
        }
    }
    // the tiles of the longest lists first: they take the longest
    std::stable_sort(items.begin(), items.end(), [](const ScanItem &a, const ScanItem &b) { return a.n > b.n; });
    int rc;
    DevBuf d_lists(&ix->alloc), d_unproven(&ix->alloc);
    DevBufGuard rel{&d_lists, &d_unproven};
    if ((rc = upload(d_lists, lists, s)) != VF_OK) return rc;
    const int32_t *map = ix->d_M_HS.as<int32_t>();
    const int64_t n_rows = ix->O_HS[(size_t)ix->graph_labels[hi - 1]] + ix->S[(size_t)ix->graph_labels[hi - 1]] - base0;
    int kind = ix->join_kind();
    // d_unproven: how many rows (of a few) would have no proof as queries, how many have none, which, and those that are joined again
    const int64_t sel_at = 2 + n_rows;
    if (kind == kJoinSingle && (rc = d_unproven.reserve((size_t)(sel_at + std::max<int64_t>(n_rows, kLookRows)) * 4)) != VF_OK) {
        if (rc != VF_ENOMEM) return rc;
        (void)hipGetLastError();
        kind = kJoinSplit;
    }
    auto pack = [&](int kd) {
        launch_join_pack(kd, ix->X, ix->dim, map, d_lists.as<JoinList>(), (int)lists.size(), n_groups, ix->join_norms(),
                         ix->d_centre.as<float>(), ix->join_scale(kd), ix->tmp_blk.as<uint4>(), ix->tmp_norm.p, nullptr, 0, s);
    };
    auto join = [&](int kd, const int32_t *sel, int tile_rows, int n_items) {
        JoinParams p{};
        p.xblk = ix->tmp_blk.as<uint4>(); p.xnorm = ix->tmp_norm.p;
        p.qsrc = ix->X; p.qrow = map + base0; p.sel = sel; p.items = d_items.as<ScanItem>();
        p.dim = ix->dim; p.K = K; p.centre = ix->d_centre.as<float>(); p.scale = ix->join_scale(kd);
        p.res_idx = cand_idx.as<int32_t>(); p.res_bits = cand_dist.as<uint32_t>();
        p.meta = ix->meta();
        launch_join(kd, p, tile_rows, n_items, s);
    };
    // n rows of list i (sel null: all of them) from their candidates, which begin at row cand_at
    int32_t *const loose = d_unproven.as<int32_t>(), *const unproven_rows = loose + 1;
    auto rows = [&](int kd, size_t i, int64_t cand_at, const int32_t *sel, int64_t n, int32_t nseg, int64_t seg_stride, int32_t *unproven,
                    int32_t *loose = nullptr) {
        const int32_t l = ix->graph_labels[i];
        const int64_t base = ix->O_HS[(size_t)l];
        GraphRowsParams g{};
        g.X = ix->X; g.dim = ix->dim; g.map = map + base; g.n_list = ix->S[(size_t)l]; g.n = n;
        g.sel = sel; g.row_base = (int32_t)(base - base0); g.nseg = nseg; g.seg_stride = seg_stride;
        g.cand_idx = cand_idx.as<int32_t>() + cand_at * K; g.cand_bits = cand_dist.as<uint32_t>() + cand_at * K; g.K = K; g.R = deg;
        g.G_rows = rows_out + (base - base0) * deg;
        g.err_bound = ix->join_err_bound(kd); g.err_q = ix->join_err_q(kd, true); g.xn_max = ix->xc_max;
        g.approx_unit = 1.0f / (ix->join_scale(kd) * ix->join_scale(kd)); g.centre = ix->d_centre.as<float>();
        g.unproven = unproven;
        g.loose = loose; g.err_q_query = ix->join_err_q(kd, false);
        launch_graph_rows(ix->dtype, g, s);
    };
    auto fetch_counts = [&](int32_t (&count)[2]) -> int {   // as a query, as a row
        VF_HIP(hipMemcpyAsync(count, d_unproven.p, 8, hipMemcpyDeviceToHost, s));
        VF_HIP(hipStreamSynchronize(s));
        return VF_OK;
    };
    // The rows of sel (ascending, of any lists).  Few rows do not fill the chip with whole lists: as many segments as do,
    // and as the candidates' buffer has room for (about 1,024 items; builds of 200,000 x 128 with some of the rows joined again:
    // with 256 3 to 8 % longer, with 4,096 2 to 6).  VF_ENOMEM (for the items): nothing was launched.
    auto selected = [&](int kd, const std::vector<int32_t> &sel, int32_t *unproven) -> int {
        int rc;
        int32_t *d_sel = d_unproven.as<int32_t>() + sel_at;
        // (few rows are a matter of latency, most of it a wave's selection: 32 rows of a list of 60,000 x 128, K = 48, by 64 items
        // of 32 rows 351 us, by 256 of 8 118)
        const int waves = join_tile_rows(kd, ix->dim), tile = sel.size() <= kLookRows ? 8 : waves;
        const int64_t most = std::min<int64_t>(n_rows / (int64_t)sel.size(), 1024 / (int64_t)(sel.size() / tile + 1));
        const int32_t nseg = (int32_t)std::max<int64_t>(1, std::min<int64_t>(64, most));
        std::vector<ScanItem> part;
        std::vector<size_t> first;   // of list lo + i in sel
        size_t at = 0;
        for (size_t i = lo; i < hi; ++i) {
            const int32_t l = ix->graph_labels[i], nl = ix->S[(size_t)l], ng = (nl + 31) / 32, per = (ng + nseg - 1) / nseg;
            const int64_t row0 = ix->O_HS[(size_t)l] - base0;
            first.push_back(at);
            size_t e = at;
            while (e < sel.size() && sel[e] < row0 + nl) ++e;
            for (size_t count; at < e; at += count) {
                count = std::min<size_t>((size_t)tile, e - at);
                for (int32_t sg = 0; sg < nseg; ++sg) {   // (an empty segment still writes its rows)
                    const int32_t g0 = std::min(sg * per, ng - 1);
                    ScanItem it{};
                    it.group0 = lists[i - lo].group0 + g0; it.entry0 = g0 * 32;
                    it.n = sg * per < ng ? std::min(per * 32, nl - g0 * 32) : 0;
                    it.q_begin = (int32_t)at; it.q_count = (int32_t)count;
                    it.self_base = (int32_t)row0; it.part_row = (int32_t)(at + (size_t)sg * sel.size());
                    part.push_back(it);
                }
            }
        }
        first.push_back(at);
        std::stable_sort(part.begin(), part.end(), [](const ScanItem &a, const ScanItem &b) { return a.n > b.n; });
        if ((rc = upload(d_items, part, s)) != VF_OK) return rc;
        VF_HIP(hipMemcpyAsync(d_sel, sel.data(), sel.size() * 4, hipMemcpyHostToDevice, s));
        join(kd, d_sel, waves, (int)part.size());
        for (size_t i = lo; i < hi; ++i)
            rows(kd, i, (int64_t)first[i - lo], d_sel + first[i - lo], (int64_t)(first[i - lo + 1] - first[i - lo]), nseg,
                 (int64_t)sel.size(), unproven);
        VF_HIP(hipStreamSynchronize(s));
        return VF_OK;
    };
    pack(kind);
    // Where a batch takes milliseconds: would binary16 prove its rows?  32 rows of each of the eight longest lists, whose
    // neighbours are closest together, tell.  The look takes 0.2 ms; not looking costs tables of far clusters a join that
    // proves little and then the one that does: 60,000 x 128, clusters twelve times as far apart as they are wide, build
    // 9.6 ms without, 5.4 with it (near clusters 4.5 and 4.7); 300,000, ten times as far: 64 and 52 ms.  At 30,000 (9e8 pairs)
    // the table of far clusters still does as well without.
    double pairs = 0;
    for (const JoinList &l : lists) pairs += (double)l.n * l.n;
    if (kind == kJoinSingle && pairs > 1.5e9) {
        std::vector<size_t> by_size(lists.size());
        for (size_t i = 0; i < by_size.size(); ++i) by_size[i] = i;
        std::stable_sort(by_size.begin(), by_size.end(), [&](size_t a, size_t b) { return lists[a].n > lists[b].n; });
        std::vector<int32_t> sel;
        for (size_t u = 0; u < std::min<size_t>(8, by_size.size()); ++u)
            for (int32_t r = 0; r < kLookRows / 8; ++r)
                sel.push_back((int32_t)(lists[by_size[u]].src - base0 + (int64_t)lists[by_size[u]].n * r / (kLookRows / 8)));
        std::sort(sel.begin(), sel.end());
        VF_HIP(hipMemsetAsync(d_unproven.p, 0, 8, s));
        int32_t count[2] = {0, 0};
        rc = selected(kind, sel, unproven_rows);
        if (rc == VF_OK) rc = fetch_counts(count);
        if (rc != VF_OK && rc != VF_ENOMEM) return rc;
        if (rc == VF_ENOMEM) (void)hipGetLastError();   // (no look then)
        if ((size_t)count[1] > sel.size() / 16) {
            ix->join_single = false;
            pack(kind = kJoinSplit);
        }
    }
    if ((rc = upload(d_items, items, s)) != VF_OK) return rc;
    if (kind == kJoinSingle) VF_HIP(hipMemsetAsync(d_unproven.p, 0, 8, s));
    join(kind, nullptr, kJoinRowsShared, (int)items.size());
    for (size_t i = lo; i < hi; ++i)
        rows(kind, i, ix->O_HS[(size_t)ix->graph_labels[i]] - base0, nullptr, ix->S[(size_t)ix->graph_labels[i]], 1, 0,
             kind == kJoinSingle ? unproven_rows : nullptr, kind == kJoinSingle ? loose : nullptr);
    if (kind == kJoinSingle) {
        int32_t counts[2] = {0, 0};
        if ((rc = fetch_counts(counts)) != VF_OK) return rc;
        const int32_t count = counts[1];
        int64_t n_looked = 0;
        for (const JoinList &l : lists) n_looked += (l.n + kLooseStep - 1) / kLooseStep;
        if ((int64_t)counts[0] > n_looked / 64) for_queries = false;
        if ((int64_t)count > n_rows / 2) {   // all once more, with operands that keep twice the bits: most have to be, and need not be listed
            pack(kJoinSplit);
            join(kJoinSplit, nullptr, kJoinRowsShared, (int)items.size());
            for (size_t i = lo; i < hi; ++i)
                rows(kJoinSplit, i, ix->O_HS[(size_t)ix->graph_labels[i]] - base0, nullptr, ix->S[(size_t)ix->graph_labels[i]], 1, 0, nullptr);
            ix->join_single = false;
        } else if (count > 0) {   // those once more
            std::vector<int32_t> sel((size_t)count);
            VF_HIP(hipMemcpy(sel.data(), unproven_rows + 1, sel.size() * 4, hipMemcpyDeviceToHost));
            std::sort(sel.begin(), sel.end());
            pack(kJoinSplit);
            rc = selected(kJoinSplit, sel, nullptr);
            if (rc == VF_ENOMEM) {   // each by its wave, from every entry of its list
                (void)hipGetLastError();
                for (size_t i = lo; i < hi; ++i)
                    rows(kJoinSingle, i, ix->O_HS[(size_t)ix->graph_labels[i]] - base0, nullptr, ix->S[(size_t)ix->graph_labels[i]], 1, 0, nullptr);
            } else if (rc != VF_OK) {
                return rc;
            }
            if ((int64_t)count > n_rows / 64) ix->join_single = false;
        }
    }
    if (kind != kJoinSingle || !ix->join_single) for_queries = false;
    if (global_ids)
        for (size_t i = lo; i < hi; ++i) {
            const int32_t l = ix->graph_labels[i];
            const int64_t base = ix->O_HS[(size_t)l];
            launch_graph_global_ids(rows_out + (base - base0) * deg, map + base, (int64_t)ix->S[(size_t)l] * deg, ix->d_Gg.as<int32_t>() + base * ix->R, s);
        }
    VF_HIP(hipGetLastError());
    VF_HIP(hipStreamSynchronize(s));   // the tables above are pageable host memory and temporaries
    return VF_OK;
}

// The same for one list on the scan kernels: float32 tables whose norms the join's proofs do not cover (NaN, overflow,
// norms outside [1e-24, 1e30]), and "build16" = 0.  Interleave the list, contract it against itself, keep K candidates per
// vertex, order `deg` of them into rows_out ([|C_l|][deg] local ids); with global_ids the same rows also go
// to the index's global-id table (deg == R).
static int build_graph_for_label(vf_index *ix, int32_t l, int32_t K, int32_t deg, int32_t *rows_out, bool global_ids,
                                 DevBuf &cand_idx, DevBuf &cand_dist, DevBuf &d_items, hipStream_t s)
{
    const int64_t base = ix->O_HS[l];
    const int32_t nl = ix->S[l];
    const int64_t n_groups = (nl + 31) / 32;
    const int32_t *map = ix->d_M_HS.as<int32_t>() + base;
    launch_interleave(ix->dtype, ix->X, ix->dim, map, nullptr, nullptr, nl, n_groups, ix->ncp, ix->tmp_blk.as<uint4>(),
                      ix->tmp_norm.p, s);
    // dim 96 / 128: 16-row tiles on the 16x16x4 MFMA (their smaller LDS footprint more than doubles the resident waves)
    const int32_t TR = (ix->tune.build16 && scan16_supported(ix->dtype, ix->dim, 16)) ? 16 : 32;
    const int64_t n_tiles = (nl + TR - 1) / TR;
    std::vector<ScanItem> items((size_t)n_tiles);
    for (int64_t t = 0; t < n_tiles; ++t) {
        ScanItem &it = items[(size_t)t];
        it.group0 = 0; it.map_off = 0; it.entry0 = 0; it.n = nl;
        it.q_begin = (int32_t)(t * TR);
        it.q_count = (int32_t)std::min<int64_t>(TR, nl - t * TR);
        it.self_base = it.q_begin;
        it.part_row = it.q_begin;
    }
    int rc = upload(d_items, items, s);
    if (rc != VF_OK) return rc;
    VF_HIP(hipStreamSynchronize(s));  // `items` is pageable host memory
    ScanParams p{};
    p.xblk = ix->tmp_blk.as<uint4>(); p.xnorm = ix->tmp_norm.p; p.map = map;
    p.qsrc = ix->X; p.qrow = map; p.items = d_items.as<ScanItem>();
    p.dim = ix->dim; p.ncp = ix->ncp; p.K = K; p.tile_rows = TR;
    p.res_idx = cand_idx.as<int32_t>(); p.res_bits = cand_dist.as<uint32_t>();
    p.others_off = nullptr; p.others = nullptr; p.meta = ix->meta();
    if (TR == 16) {
        // long lists go panel by panel so that the resident waves share L2 (4 MiB of list per launch by
        // default -- the measured optimum, one XCD's L2; lists of up to 4 panels are not cut)
        const int64_t panel_bytes = (int64_t)std::max(1, ix->tune.build_panel_kb) << 10;
        const int64_t list_bytes = n_groups * (int64_t)ix->group_bytes();
        if (list_bytes <= 4 * panel_bytes) {
            launch_scan16(p, (int)n_tiles, s);
        } else {
            const int32_t panel = (int32_t)std::max<int64_t>(32, panel_bytes / ((int64_t)ix->group_bytes() / 32) / 32 * 32);
            for (int64_t e0 = 0; e0 < nl; e0 += panel) {
                p.panel_entry0 = (int32_t)e0; p.panel_n = panel; p.carry = e0 > 0;
                launch_scan16(p, (int)n_tiles, s);
            }
        }
    } else {
        launch_scan(ix->dtype, p, (int)n_tiles, s);
    }
    // float32 rows are accepted only with a proof that the self-join's K candidates contain them (the bound of the
    // float32 matrix-core approximations, relative to the largest squared norm of the table)
    const bool checked = ix->dtype == VF_F32 && ix->xn_max > 0.f;
    GraphRowsParams g{};
    g.X = ix->X; g.dim = ix->dim; g.map = map; g.n_list = nl; g.n = nl;
    g.cand_idx = cand_idx.as<int32_t>(); g.cand_bits = cand_dist.as<uint32_t>(); g.K = K; g.R = deg; g.G_rows = rows_out; g.nseg = 1;
    g.err_bound = checked ? ix->seed_err_bound() : -1.f; g.xn_max = ix->xn_max; g.approx_unit = 1.f;
    launch_graph_rows(ix->dtype, g, s);
    if (global_ids)
        launch_graph_global_ids(rows_out, map, (int64_t)nl * deg, ix->d_Gg.as<int32_t>() + base * ix->R, s);
    VF_HIP(hipGetLastError());
    return VF_OK;
}

// Reduces the degree-D rows of all lists (knn, [n_HS][D]) to the index's degree-R rows: rank-based pruning,
// reverse edges, merge (vf_graphopt.hip).  d_Gg serves as the forward rows' storage until the end.
static int optimize_graphs(vf_index *ix, const int32_t *d_knn, int32_t D, hipStream_t s)
{
    const int64_t nn = ix->n_HS;
    const int32_t R = ix->R;
    int rc;
    DevBuf d_base(&ix->alloc), d_deg(&ix->alloc), d_off(&ix->alloc), d_seg(&ix->alloc);
    DevBufGuard rel{&d_base, &d_deg, &d_off, &d_seg};
    std::vector<int32_t> base((size_t)nn);
    for (int32_t l : ix->graph_labels)
        std::fill(base.begin() + ix->O_HS[(size_t)l], base.begin() + ix->O_HS[(size_t)l] + ix->S[(size_t)l],
                  (int32_t)ix->O_HS[(size_t)l]);
    if ((rc = upload(d_base, base, s)) != VF_OK) return rc;
    if ((rc = d_deg.reserve((size_t)nn * 4)) != VF_OK) return rc;
    if ((rc = d_off.reserve((size_t)(nn + 1) * 8)) != VF_OK) return rc;
    int32_t *F = ix->d_Gg.as<int32_t>();
    launch_graph_prune(d_knn, d_base.as<int32_t>(), nn, D, R, F, s);
    VF_HIP(hipMemsetAsync(d_deg.p, 0, (size_t)nn * 4, s));
    launch_graph_indegree(F, d_base.as<int32_t>(), nn, R, d_deg.as<int32_t>(), s);
    std::vector<int32_t> deg((size_t)nn);
    VF_HIP(hipMemcpyAsync(deg.data(), d_deg.p, (size_t)nn * 4, hipMemcpyDeviceToHost, s));
    VF_HIP(hipStreamSynchronize(s));   // also: `base` is pageable host memory
    std::vector<int64_t> off((size_t)nn + 1);
    off[0] = 0;
    for (int64_t g = 0; g < nn; ++g) off[(size_t)g + 1] = off[(size_t)g] + deg[(size_t)g];
    VF_REQUIRE(off[(size_t)nn] <= nn * (int64_t)R, "internal: more proposals than forward edges");
    if ((rc = upload(d_off, off, s)) != VF_OK) return rc;
    if ((rc = d_seg.reserve((size_t)std::max<int64_t>(1, off[(size_t)nn]) * 8)) != VF_OK) return rc;
    VF_HIP(hipMemsetAsync(d_deg.p, 0, (size_t)nn * 4, s));   // now the per-target cursors
    launch_graph_reverse_fill(F, d_base.as<int32_t>(), nn, R, d_off.as<int64_t>(), d_deg.as<int32_t>(),
                              d_seg.as<uint64_t>(), s);
    launch_graph_reverse_merge(F, d_off.as<int64_t>(), d_seg.as<uint64_t>(), nn, R, ix->d_G.as<int32_t>(), s);
    launch_graph_global_ids_based(ix->d_G.as<int32_t>(), d_base.as<int32_t>(), ix->d_M_HS.as<int32_t>(), nn, R,
                                  ix->d_Gg.as<int32_t>(), s);
    VF_HIP(hipGetLastError());
    VF_HIP(hipStreamSynchronize(s));   // `off` is pageable host memory; the temporaries are freed on return
    return VF_OK;
}

int build_index_impl(const void *vectors, int dtype, int64_t n, int32_t dim, const int64_t *label_offsets,
                     const int32_t *label_ids, int32_t n_labels, int32_t T, int32_t graph_degree, int32_t graph_kind,
                     int32_t knn_degree, const vf_allocator *allocator, void *hip_stream, vf_index **out)
{
    VF_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    VF_REQUIRE(vectors && label_offsets && label_ids, "NULL input pointer");
    VF_REQUIRE(dtype == VF_U8 || dtype == VF_F32, "dtype must be VF_U8 or VF_F32");
    VF_REQUIRE(n > 0 && n < ((int64_t)1 << 31), "n must be in [1, 2^31)");
    const int64_t row_bytes = (int64_t)dim * (dtype == VF_U8 ? 1 : 4);
    VF_REQUIRE(dim > 0 && row_bytes % 16 == 0 && row_bytes >= 16 && row_bytes <= 2048,
               "dim: uint8 needs dim % 16 == 0, float32 dim % 4 == 0, 16 <= bytes per vector <= 992");
    // a 32-row tile of the contraction kernel with the 64 candidates per row of a graph build must fit in LDS
    VF_REQUIRE(scan_lds_bytes((int32_t)((row_bytes / 16 + 1) / 2), 32, 64) <= 64 * 1024,
               "dim: vectors of more than 992 bytes are not supported (LDS of the contraction kernel)");
    VF_REQUIRE(allocator == nullptr || (allocator->alloc != nullptr && allocator->free != nullptr),
               "allocator: both functions must be given");
    VF_REQUIRE(((uintptr_t)vectors & 15) == 0, "vectors must be 16-byte aligned");
    VF_REQUIRE(n_labels > 0, "n_labels must be positive");
    VF_REQUIRE(graph_degree >= 1 && graph_degree <= 64, "graph_degree must be in [1, 64]");
    VF_REQUIRE(T >= graph_degree + 1, "T must be at least graph_degree + 1");
    VF_REQUIRE(graph_kind == VF_GRAPH_KNN || graph_kind == VF_GRAPH_PRUNED, "graph_kind must be VF_GRAPH_KNN or VF_GRAPH_PRUNED");
    // degree of the kNN graph a pruned graph starts from: 2 R, as far as the self-join's 64 candidates per
    // row reach (float32 rows are re-ranked out of 16 candidates more than they keep)
    const int32_t knn_max = dtype == VF_U8 ? 64 : 48;
    int32_t D = graph_degree;
    if (graph_kind == VF_GRAPH_PRUNED) {
        D = knn_degree > 0 ? knn_degree : std::min(2 * graph_degree, knn_max);
        VF_REQUIRE(D >= graph_degree && D <= knn_max,
                   "knn_degree must lie in [graph_degree, 64] (uint8) or [graph_degree, 48] (float32)");
        VF_REQUIRE(T >= D + 1, "T must be at least knn_degree + 1");
    } else {
        VF_REQUIRE(knn_degree == 0, "knn_degree is only used with VF_GRAPH_PRUNED");
    }
    VF_REQUIRE(label_offsets[0] == 0, "label_offsets[0] must be 0");
    for (int64_t i = 0; i < n; ++i) VF_REQUIRE(label_offsets[i + 1] >= label_offsets[i], "label_offsets must not decrease");
    const int64_t n_raw = label_offsets[n];
    for (int64_t p = 0; p < n_raw; ++p)
        VF_REQUIRE(label_ids[p] >= 0 && label_ids[p] < n_labels, "label id outside [0, n_labels)");

    hipStream_t s = (hipStream_t)hip_stream;
    vf_index *ix = new (std::nothrow) vf_index();
    if (!ix) { set_error("out of host memory"); return VF_ENOMEM; }
    struct Guard { vf_index *ix; ~Guard() { if (ix) free_index(ix); } } guard{ix};
    ix->dtype = dtype; ix->n = n; ix->dim = dim; ix->n_labels = n_labels; ix->T = T; ix->R = graph_degree;
    ix->X = vectors;
    ix->ncp = (int32_t)((row_bytes / 16 + 1) / 2);
    if (allocator != nullptr) ix->alloc.user = *allocator;
    {
        std::lock_guard<std::mutex> lock(default_tuning_mutex());
        ix->tune = default_tuning();
    }

    {
        // ---- pass 1 (Alg. 1): posting-list sizes over sorted, duplicate-free label sets
        std::vector<int32_t> uniq((size_t)n_raw);
        std::vector<int64_t> uoff((size_t)n + 1, 0);
        int64_t w = 0;
        for (int64_t i = 0; i < n; ++i) {
            const int64_t b = label_offsets[i], e = label_offsets[i + 1], start = w;
            for (int64_t p = b; p < e; ++p) uniq[(size_t)w++] = label_ids[p];
            std::sort(uniq.begin() + start, uniq.begin() + w);
            w = std::unique(uniq.begin() + start, uniq.begin() + w) - uniq.begin();
            uoff[(size_t)i + 1] = w;
        }
        ix->S.assign((size_t)n_labels, 0);
        for (int64_t p = 0; p < w; ++p) ix->S[(size_t)uniq[(size_t)p]]++;

        // ---- split by T; S/O/M per partition, compacted in ascending label id
        ix->O_HS.assign((size_t)n_labels, -1); ix->O_LS.assign((size_t)n_labels, -1);
        ix->GO_LS.assign((size_t)n_labels, -1); ix->hs_slot.assign((size_t)n_labels, -1);
        for (int32_t l = 0; l < n_labels; ++l) {
            const int32_t sz = ix->S[(size_t)l];
            if (sz >= T) {
                ix->O_HS[(size_t)l] = ix->n_HS; ix->n_HS += sz;
                ix->hs_slot[(size_t)l] = (int32_t)ix->graph_labels.size();
                ix->graph_labels.push_back(l);
            } else if (sz > 0) {
                ix->O_LS[(size_t)l] = ix->n_LS; ix->n_LS += sz;
                ix->GO_LS[(size_t)l] = ix->n_groups_LS; ix->n_groups_LS += (sz + 31) / 32;
                ix->n_scan_labels++;
            }
        }
        std::vector<int32_t> M_HS((size_t)ix->n_HS), M_LS((size_t)ix->n_LS);
        {
            std::vector<int32_t> fill((size_t)n_labels, 0);
            for (int64_t i = 0; i < n; ++i)
                for (int64_t p = uoff[(size_t)i]; p < uoff[(size_t)i + 1]; ++p) {
                    const int32_t l = uniq[(size_t)p];
                    if (ix->O_HS[(size_t)l] >= 0) M_HS[(size_t)(ix->O_HS[(size_t)l] + fill[(size_t)l]++)] = (int32_t)i;
                    else M_LS[(size_t)(ix->O_LS[(size_t)l] + fill[(size_t)l]++)] = (int32_t)i;
                }
        }
        std::vector<int32_t>().swap(uniq);
        std::vector<int64_t>().swap(uoff);

        int rc;
        if ((rc = upload(ix->d_S, ix->S, s)) != VF_OK) return rc;
        if ((rc = upload(ix->d_O_HS, ix->O_HS, s)) != VF_OK) return rc;
        if ((rc = upload(ix->d_O_LS, ix->O_LS, s)) != VF_OK) return rc;
        if ((rc = upload(ix->d_hs_slot, ix->hs_slot, s)) != VF_OK) return rc;
        if ((rc = upload(ix->d_M_HS, M_HS, s)) != VF_OK) return rc;
        if ((rc = upload(ix->d_M_LS, M_LS, s)) != VF_OK) return rc;
        VF_HIP(hipStreamSynchronize(s));

        if (dtype == VF_F32) {   // failed proofs of the filtering scans
            if ((rc = ix->d_scan_fb.reserve(8)) != VF_OK) return rc;
            VF_HIP(hipMemsetAsync(ix->d_scan_fb.p, 0, 8, s));
        }
        // ---- scan partition: StoreInterleaved over every scan list (Section 4.2.2)
        if (ix->n_groups_LS > 0) {
            std::vector<int64_t> grp_src((size_t)ix->n_groups_LS);
            std::vector<int32_t> grp_cnt((size_t)ix->n_groups_LS);
            for (int32_t l = 0; l < n_labels; ++l) {
                if (ix->GO_LS[(size_t)l] < 0) continue;
                const int32_t sz = ix->S[(size_t)l];
                for (int32_t g = 0; g < (sz + 31) / 32; ++g) {
                    grp_src[(size_t)(ix->GO_LS[(size_t)l] + g)] = ix->O_LS[(size_t)l] + (int64_t)g * 32;
                    grp_cnt[(size_t)(ix->GO_LS[(size_t)l] + g)] = std::min(32, sz - g * 32);
                }
            }
            DevBuf d_src(&ix->alloc), d_cnt(&ix->alloc);
            DevBufGuard r2{&d_src, &d_cnt};
            if ((rc = upload(d_src, grp_src, s)) != VF_OK) return rc;
            if ((rc = upload(d_cnt, grp_cnt, s)) != VF_OK) return rc;
            if ((rc = ix->d_X_LS.reserve((size_t)ix->n_groups_LS * ix->group_bytes())) != VF_OK) return rc;
            if ((rc = ix->d_xnorm_LS.reserve((size_t)ix->n_groups_LS * 32 * 4)) != VF_OK) return rc;
            launch_interleave(dtype, vectors, dim, ix->d_M_LS.as<int32_t>(), d_src.as<int64_t>(), d_cnt.as<int32_t>(),
                              ix->n_LS, ix->n_groups_LS, ix->ncp, ix->d_X_LS.as<uint4>(), ix->d_xnorm_LS.p, s);
            VF_HIP(hipGetLastError());
            VF_HIP(hipStreamSynchronize(s));
            // float32 lists once more in bfloat16, for the filtering scan kernel.  Its proofs need the largest
            // rounding error |x - bf16(x)| and the largest squared norm of a list vector; a table with NaN or
            // overflowing values, or norms outside [1e-24, 1e30] (the bound is relative to the norm and assumes
            // that what the matrix cores flush is negligible beside it), keeps the exact kernels only.
            if (dtype == VF_F32 && ix->tune.scan_bf16 && scan_bf16_supported(dtype, dim, 16, 32)) {
                const size_t n_slots = (size_t)ix->n_groups_LS * 32;
                DevBuf d_err2(&ix->alloc);
                DevBufGuard r4{&d_err2};
                if ((rc = ix->d_X_LS16.reserve((size_t)ix->n_groups_LS * ix->group_bytes() / 2)) != VF_OK) return rc;
                if ((rc = d_err2.reserve(n_slots * 4)) != VF_OK) return rc;
                launch_seed_pack_bf16(ix->d_X_LS.as<uint4>(), ix->n_groups_LS, ix->ncp, ix->d_X_LS16.as<uint4>(),
                                      d_err2.as<float>(), s);
                std::vector<float> e2(n_slots), nr(n_slots);
                VF_HIP(hipMemcpyAsync(e2.data(), d_err2.p, n_slots * 4, hipMemcpyDeviceToHost, s));
                VF_HIP(hipMemcpyAsync(nr.data(), ix->d_xnorm_LS.p, n_slots * 4, hipMemcpyDeviceToHost, s));
                VF_HIP(hipStreamSynchronize(s));
                double mx_e = 0.0;
                float mx_n = 0.f;
                bool finite = true;
                for (size_t i = 0; i < n_slots; ++i) {
                    finite = finite && e2[i] == e2[i] && e2[i] <= 3.0e38f && nr[i] == nr[i] && nr[i] <= 3.0e38f;
                    mx_e = e2[i] > mx_e ? e2[i] : mx_e;
                    mx_n = nr[i] > mx_n ? nr[i] : mx_n;
                }
                if (finite && mx_n >= 1e-24f && mx_n <= 1e30f) {
                    ix->has_ls16 = true;
                    ix->ls_bf16_delta = (float)(std::sqrt(mx_e) * 1.001);
                    ix->ls_xn_max = mx_n;
                } else {
                    ix->d_X_LS16.release();
                }
            }
        }

        // ---- graph partition: membership bitsets and one exact kNN graph per list
        const int32_t n_gl = (int32_t)ix->graph_labels.size();
        ix->bitset_words = (n + 31) / 32;
        if (n_gl > 0) {
            const size_t bs_bytes = (size_t)n_gl * ix->bitset_words * 4;
            if ((rc = ix->d_bitsets.reserve(bs_bytes)) != VF_OK) return rc;
            VF_HIP(hipMemsetAsync(ix->d_bitsets.p, 0, bs_bytes, s));
            if ((rc = ix->d_G.reserve((size_t)ix->n_HS * ix->R * 4)) != VF_OK) return rc;
            if ((rc = ix->d_Gg.reserve((size_t)ix->n_HS * ix->R * 4)) != VF_OK) return rc;
            int32_t max_list = 0;
            for (int32_t l : ix->graph_labels) max_list = std::max(max_list, ix->S[(size_t)l]);
            const bool pruned = graph_kind == VF_GRAPH_PRUNED;
            const int32_t K = dtype == VF_U8 ? D : std::min(64, D + 16);
            DevBuf d_knn(&ix->alloc);
            DevBufGuard rk{&d_knn};
            if (pruned && (rc = d_knn.reserve((size_t)ix->n_HS * D * 4)) != VF_OK) return rc;
            DevBuf cand_idx(&ix->alloc), cand_dist(&ix->alloc), d_items(&ix->alloc);
            DevBufGuard r3{&cand_idx, &cand_dist, &d_items};
            // squared norm of every row of X and the largest of them: the joins and the matrix-core seed scoring read the
            // norms, the proofs of both need the largest (float32 joins: those of the centred rows)
            if ((rc = ix->d_xnorm_all.reserve((size_t)n * 4)) != VF_OK) return rc;
            if (ix->dtype == VF_F32) {
                DevBuf parts(&ix->alloc);
                DevBufGuard rp{&parts};
                if ((rc = parts.reserve(((size_t)kCentreParts * dim + 3) * 4)) != VF_OK) return rc;
                if ((rc = ix->d_centre.reserve((size_t)dim * 4)) != VF_OK) return rc;
                if ((rc = ix->d_xnorm_c.reserve((size_t)n * 4)) != VF_OK) return rc;
                uint32_t *max_bits = parts.as<uint32_t>() + (size_t)kCentreParts * dim;
                launch_centre(ix->X, dim, n, parts.as<float>(), ix->d_centre.as<float>(), s);
                VF_HIP(hipMemsetAsync(max_bits, 0, 12, s));
                launch_row_norms_f32(ix->X, dim, n, ix->d_centre.as<float>(), ix->d_xnorm_all.as<uint32_t>(), ix->d_xnorm_c.as<uint32_t>(),
                                     max_bits, s);
                VF_HIP(hipGetLastError());
                float mx[3] = {0.f, 0.f, 0.f};
                VF_HIP(hipMemcpyAsync(mx, max_bits, 12, hipMemcpyDeviceToHost, s));
                VF_HIP(hipStreamSynchronize(s));
                // a table with NaN or overflowing norms keeps the exact kernel, and so does one whose largest
                // squared norm is outside [1e-24, 1e30]: the proofs' bound is relative to that norm and assumes
                // that what the matrix cores flush (products under 1.2e-38) is negligible beside it.
                // The bound itself: |approximation - ordered distance| <= 300 u (|q|^2 + |x|^2), u = 2^-24 (dot
                // product of <= 512 terms in any order, two norms, the final additions, the ordered sum's own
                // error); 512 u = 2^-15 is used (vf_index::seed_err_bound).
                auto in_range = [](float m) { return m >= 1e-24f && m <= 1e30f; };
                if (in_range(mx[0])) {
                    ix->xn_max = mx[0];
                    ix->seed_mfma_ok = seed_mfma_supported(ix->dtype, ix->dim);
                }
                if (!ix->seed_mfma_ok) ix->d_xnorm_all.release();
                if (in_range(mx[0]) && in_range(mx[1])) {
                    ix->xc_max = mx[1];
                    ix->xc_rho = std::min(std::sqrt(mx[2]) * 1.001f, 4.8828125e-04f);
                }
                else ix->d_xnorm_c.release();
            } else {
                launch_row_norms_u8(ix->X, ix->dim, n, ix->d_xnorm_all.as<uint32_t>(), s);
                ix->seed_mfma_ok = seed_mfma_supported(ix->dtype, ix->dim);
            }
            bool joined = ix->dtype == VF_U8 || (ix->xc_max > 0.f && ix->tune.build16);
            // Lists are joined many to a launch: as many as fit, packed and with their candidates, into a GiB (or one list
            // that is larger than that).  The scan kernels take one list at a time.  Where there is no memory for that:
            // smaller batches, down to single lists, and then the scan kernels, whose copies of a list are smaller.
            int64_t batch_rows = joined ? (int64_t)(((size_t)1 << 30) / (join_group_bytes(ix->join_kind_max(), ix->dim) / 32 + (size_t)K * 8)) : 0;
            std::vector<size_t> batch_end;   // positions in graph_labels
            while (true) {
                int64_t tmp_groups = 0, tmp_rows = 0;
                batch_end.clear();
                for (size_t i = 0; i < ix->graph_labels.size();) {
                    int64_t rows_in = 0, groups_in = 0;
                    size_t e = i;
                    while (e < ix->graph_labels.size() && (e == i || (joined && rows_in + ix->S[(size_t)ix->graph_labels[e]] <= batch_rows))) {
                        rows_in += ix->S[(size_t)ix->graph_labels[e]];
                        groups_in += (ix->S[(size_t)ix->graph_labels[e]] + 31) / 32;
                        ++e;
                    }
                    tmp_groups = std::max(tmp_groups, groups_in);
                    tmp_rows = std::max(tmp_rows, rows_in);
                    batch_end.push_back(e);
                    i = e;
                }
                const size_t cand_bytes = (size_t)(tmp_rows + 31) / 32 * 32 * K * 4;
                if ((rc = ix->tmp_blk.reserve((size_t)tmp_groups * (joined ? join_group_bytes(ix->join_kind_max(), ix->dim) : ix->group_bytes()))) == VF_OK &&
                    (rc = ix->tmp_norm.reserve((size_t)tmp_groups * 32 * 4)) == VF_OK && (rc = cand_idx.reserve(cand_bytes)) == VF_OK &&
                    (rc = cand_dist.reserve(cand_bytes)) == VF_OK)
                    break;
                if (rc != VF_ENOMEM || !joined) return rc;
                (void)hipGetLastError();
                for (DevBuf *t : {&ix->tmp_blk, &ix->tmp_norm, &cand_idx, &cand_dist}) t->release();
                if (batch_rows <= max_list) joined = false;
                batch_rows = std::max<int64_t>(batch_rows / 4, max_list);
            }
            // optionally a line on stderr every few seconds (index builds of 10^7 vectors take minutes)
            const bool progress = ix->tune.build_progress != 0;
            time_t last_print = time(nullptr);
            size_t done = 0;
            bool for_queries = joined && ix->dtype == VF_F32;
            for (const size_t end : batch_end) {
                if (progress && time(nullptr) - last_print >= 10) {
                    fprintf(stderr, "[vf_build_index] %zu of %zu label graphs built, next list holds %d vectors\n", done,
                            ix->graph_labels.size(), ix->S[(size_t)ix->graph_labels[done]]);
                    fflush(stderr);
                    last_print = time(nullptr);
                }
                for (size_t i = done; i < end; ++i) {
                    const int32_t l = ix->graph_labels[i];
                    launch_bitset_fill(ix->d_M_HS.as<int32_t>() + ix->O_HS[(size_t)l], ix->S[(size_t)l],
                                       ix->d_bitsets.as<uint32_t>() + (int64_t)ix->hs_slot[(size_t)l] * ix->bitset_words, s);
                }
                const int32_t first = ix->graph_labels[done];
                const int64_t base = ix->O_HS[(size_t)first];
                int32_t *rows = pruned ? d_knn.as<int32_t>() + base * D : ix->d_G.as<int32_t>() + base * ix->R;
                if (joined)
                    rc = build_graphs_joined(ix, done, end, K, D, rows, !pruned, cand_idx, cand_dist, d_items, for_queries, s);
                else
                    rc = build_graph_for_label(ix, first, K, D, rows, !pruned, cand_idx, cand_dist, d_items, s);
                if (rc != VF_OK) return rc;
                done = end;
            }
            // (distances spread out towards the nearest: k of a query and 22 to spare are as far apart as D of a row and K - D, or
            // further, up to k = D)
            if (for_queries) ix->exact_single_k = D;
            VF_HIP(hipStreamSynchronize(s));
            if (pruned) {
                cand_idx.release(); cand_dist.release();
                if ((rc = optimize_graphs(ix, d_knn.as<int32_t>(), D, s)) != VF_OK) return rc;
            }
            ix->graph_kind = graph_kind; ix->knn_degree = pruned ? D : 0;
            ix->tmp_blk.release();
            ix->tmp_norm.release();
        }
        VF_HIP(hipGetLastError());
    }
    guard.ix = nullptr;
    *out = ix;
    return VF_OK;
}

}  // namespace vf
