// Search calls (Alg. 2): per-stream workspaces, the interleaved seed copies, and the launch schedule of one
// batch -- route on the host, IVF-BFS scan beside IVF-Graph seed scoring and beam search, finalise.
#include <chrono>

#include "vf_host.h"

namespace vf {

// Adds the durations of the oldest `count` unread profiled calls to the sums (waits for them).
int fold_profile(vf_index *ix, int count)
{
    for (; count > 0 && ix->prof_unfolded > 0; --count, --ix->prof_unfolded) {
        const int slot = (ix->prof_next - ix->prof_unfolded + 2 * vf_index::kProfRing) % vf_index::kProfRing;
        hipEvent_t *ev = ix->prof_ring[slot];
        VF_HIP(hipEventSynchronize(ev[4]));
        VF_HIP(hipEventSynchronize(ev[1]));
        VF_HIP(hipEventElapsedTime(&ix->prof.scan_ms, ev[0], ev[1]));
        VF_HIP(hipEventElapsedTime(&ix->prof.seed_ms, ev[2], ev[3]));
        VF_HIP(hipEventElapsedTime(&ix->prof.beam_ms, ev[3], ev[4]));
        ix->prof_scan_sum += ix->prof.scan_ms;
        ix->prof_seed_sum += ix->prof.seed_ms;
        ix->prof_beam_sum += ix->prof.beam_ms;
        ix->prof_calls++;
    }
    return VF_OK;
}

static size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }


// The workspace of the calls on stream s: the one the stream has used before, else a free one, else one taken
// from another stream once that stream has drained.
static int workspace_for(vf_index *ix, hipStream_t s, Workspace **out)
{
    Workspace *w = nullptr;
    for (Workspace &c : ix->ws)
        if (c.owned && c.owner == s) { w = &c; break; }
    if (!w)
        for (Workspace &c : ix->ws)
            if (!c.owned) { w = &c; break; }
    if (!w) {
        // every workspace has an owner: take one whose streams are idle, else the next in turn once its streams
        // have drained (a stream its owner has destroyed meanwhile has drained; the error that reports it is dropped)
        for (Workspace &c : ix->ws) {
            const hipError_t qo = hipStreamQuery(c.owner), qs = hipStreamQuery(c.side);
            if (qo != hipSuccess || qs != hipSuccess) (void)hipGetLastError();
            if (qo != hipErrorNotReady && qs == hipSuccess) { w = &c; break; }
        }
        if (!w) {
            w = &ix->ws[ix->ws_steal];
            ix->ws_steal = (ix->ws_steal + 1) % vf_index::kWorkspaces;
            if (hipStreamSynchronize(w->owner) != hipSuccess) (void)hipGetLastError();
            VF_HIP(hipStreamSynchronize(w->side));
        }
    }
    if (!w->owned || w->owner != s) w->prev_forked = false;
    w->owned = true;
    w->owner = s;
    if (!w->ready) {
        VF_HIP(hipStreamCreateWithFlags(&w->side, hipStreamNonBlocking));
        VF_HIP(hipEventCreateWithFlags(&w->ev_fork, hipEventDisableTiming));
        VF_HIP(hipEventCreateWithFlags(&w->ev_join, hipEventDisableTiming));
        w->ready = true;
    }
    *out = w;
    return VF_OK;
}

static int get_staging(Workspace *W, size_t bytes, Staging **out)
{
    Staging &st = W->stage[W->stage_next];
    W->stage_next ^= 1;
    if (st.pending) { VF_HIP(hipEventSynchronize(st.done)); st.pending = false; }
    if (!st.done) VF_HIP(hipEventCreateWithFlags(&st.done, hipEventDisableTiming));
    if (bytes > st.cap) {
        if (st.p) { (void)hipHostFree(st.p); st.p = nullptr; st.cap = 0; }
        const size_t want = bytes + bytes / 2 + 4096;
        VF_HIP(hipHostMalloc(&st.p, want, hipHostMallocDefault));
        st.cap = want;
    }
    *out = &st;
    return VF_OK;
}

int check_search_args(const vf_index *ix, const void *queries, int64_t nq, int32_t k, const int64_t *out_ids,
                             const float *out_dists)
{
    VF_REQUIRE(ix != nullptr, "index is NULL");
    VF_REQUIRE(nq >= 0 && nq < ((int64_t)1 << 31), "nq out of range");
    VF_REQUIRE(nq == 0 || (queries && out_ids && out_dists), "NULL query or output pointer");
    VF_REQUIRE(((uintptr_t)queries & 15) == 0, "queries must be 16-byte aligned");
    VF_REQUIRE(k >= 1 && k <= 64, "k must be in [1, 64]");
    return VF_OK;
}

constexpr int kFirstLook = 4096;   // graph queries before the first look at the failed proofs

// Drops every interleaved seed copy.  Other streams may still be reading them: the device drains first.
int drop_seed_copies(vf_index *ix)
{
    VF_HIP(hipDeviceSynchronize());
    for (SeedCopy &c : ix->seed_copies) {
        for (DevBuf *b : c.bufs()) b->release();
        c.n_seeds = -1;
        c.ok = c.has_f32 = c.has_f16 = false;
    }
    return VF_OK;
}

bool wants_seed_copy(const vf_index *ix, bool exact, int32_t itopk, int32_t n_seeds)
{
    if (exact || ix->graph_labels.empty() || !ix->seed_mfma_ok || ix->tune.seed_exact) return false;
    const bool own = seed_mfma_own(ix->dtype, ix->dim);
    if (n_seeds < (own ? 65 : kSeedMfmaLeast)) return false;
    if (ix->dtype == VF_U8) return true;
    if (itopk > 64) return false;
    // (the ordered kernel would score the others' seeds, whatever the vectors are)
    return (own && itopk <= 48) || ((own || ix->tune.seed_bf16) && !ix->seed_proofs_off && ix->seeds_provable(itopk));
}

// The interleaved copy of the seeds of every graph list for n_seeds (see SeedCopy): the resident one, or a new
// one built on the caller's stream (the call returns after it is complete, so later calls on any stream may
// read it).  The index keeps kSeedCopies of them; the least recently used one makes room, after the device
// has drained, since calls on other streams may still be reading it (dimensions without a kernel instantiation of their own keep
// the first ones).  (*out)->ok is false when a copy would need
// more than half of the free device memory: the seed kernel then gathers rows from the vector table.
int seed_copy_for(vf_index *ix, int32_t n_seeds, hipStream_t s, bool build, SeedCopy **out)
{
    SeedCopy *c = nullptr;
    *out = nullptr;
    for (SeedCopy &x : ix->seed_copies)
        if (x.n_seeds == n_seeds) c = &x;
    if (c != nullptr) {
        c->last_use = ++ix->seed_tick;
        *out = c;
        return VF_OK;
    }
    if (!build) return VF_OK;
    for (SeedCopy &x : ix->seed_copies)
        if (x.n_seeds < 0) { c = &x; break; }
    if (c == nullptr) {
        // (dimensions without a kernel instantiation of their own score any further seed count without a copy, and wait for nothing)
        if (!seed_mfma_own(ix->dtype, ix->dim)) return VF_OK;
        c = &ix->seed_copies[0];
        for (SeedCopy &x : ix->seed_copies)
            if (x.last_use < c->last_use) c = &x;
        VF_HIP(hipDeviceSynchronize());
        for (DevBuf *b : c->bufs()) b->release();
    }
    c->last_use = ++ix->seed_tick;
    *out = c;
    return build_seed_copy(ix, n_seeds, s, ix->dtype == VF_F32 && ix->tune.seed_bf16 && !ix->seed_bf16_off, false, c);
}

// The watch on failed proofs of the binary16 form: its counter, and where the host reads it.
static int reserve_failed_proofs(vf_index *ix, hipStream_t s)
{
    if (ix->h_fb) return VF_OK;
    int rc = ix->d_fb_count.reserve(4);
    if (rc != VF_OK) return rc;
    VF_HIP(hipMemsetAsync(ix->d_fb_count.p, 0, 4, s));
    VF_HIP(hipStreamSynchronize(s));
    if (!ix->ev_fb) VF_HIP(hipEventCreateWithFlags(&ix->ev_fb, hipEventDisableTiming));
    VF_HIP(hipHostMalloc((void **)&ix->h_fb, 4, hipHostMallocDefault));
    *ix->h_fb = 0;
    return VF_OK;
}

// Fills *c for n_seeds on stream s (complete when the call returns).  want_f16: float32 data also get the
// binary16 form (and have the float32 one only up to 128 MiB, unless it is to be kept).
int build_seed_copy(vf_index *ix, int32_t n_seeds, hipStream_t s, bool want_f16, bool keep_f32, SeedCopy *c)
{
    c->n_seeds = n_seeds;
    c->ok = c->has_f32 = c->has_f16 = false;
    c->f16_delta = 0.f;
    if (!ix->tune.seed_cache) return VF_OK;
    const size_t n_gl = ix->graph_labels.size();
    int64_t n_groups = 0;
    for (const int32_t l : ix->graph_labels) n_groups += ((int64_t)std::min(n_seeds, ix->S[(size_t)l]) + 31) / 32;
    if (n_groups == 0) return VF_OK;
    {
        const size_t need = (size_t)n_groups * (ix->group_bytes() * 3 / 2 + 32 * 4 + 32 * 4 + 32 * 4 + 32 * 4 + 32);
        size_t free_b = 0, total_b = 0;
        VF_HIP(hipMemGetInfo(&free_b, &total_b));
        if (need + need / 4 > free_b / 2) return VF_OK;
    }
    // What the copy is made from, in one buffer that stays with it.  (Nothing is given back here: that waits for the whole device,
    // and beside a serving session until the session ends.)
    const size_t ng = (size_t)n_groups;
    std::vector<int64_t> tables(2 * n_gl + ng + (n_gl + 3 * ng + 2) / 2, 0);
    int64_t *goff = tables.data(), *slot_base = goff + n_gl, *grp_src = slot_base + n_gl;
    int32_t *slot_n = (int32_t *)(grp_src + ng), *grp_slot = slot_n + n_gl, *grp_j0 = grp_slot + ng, *grp_cnt = grp_j0 + ng, *err2 = grp_cnt + ng;
    size_t g = 0;
    for (size_t t = 0; t < n_gl; ++t) {
        const int32_t l = ix->graph_labels[t];
        const int32_t n = ix->S[(size_t)l], ns = std::min(n_seeds, n);
        goff[t] = (int64_t)g; slot_base[t] = ix->O_HS[(size_t)l]; slot_n[t] = n;
        for (int32_t j0 = 0; j0 < ns; j0 += 32, ++g) {
            grp_slot[g] = (int32_t)t; grp_j0[g] = j0;
            grp_src[g] = (int64_t)g * 32; grp_cnt[g] = std::min(32, ns - j0);
        }
    }
    int rc;
    // small batches are served from the float32 copy, so one of up to 128 MiB stays (dimensions that have a kernel for it)
    const bool want_own = !want_f16 || keep_f32 || (seed_mfma_own(ix->dtype, ix->dim) && ng * ix->group_bytes() <= ((size_t)128 << 20));
    // No memory for it: no copy, as where the device is known to be short of it.  No memory for the binary16 form beside one that is
    // made anyway: that one alone.  (The largest first: nothing to give back where that fails.)
    auto without = [&](int why) {
        if (why != VF_ENOMEM) return why;
        (void)hipGetLastError();
        for (DevBuf *b : c->bufs()) b->release();
        return (int)VF_OK;
    };
    if (want_own && (rc = c->blk.reserve(ng * ix->group_bytes())) != VF_OK) return without(rc);
    if (want_f16 && ((rc = c->blk16.reserve(ng * ix->group_bytes() / 2)) != VF_OK || (rc = reserve_failed_proofs(ix, s)) != VF_OK)) {
        if (rc != VF_ENOMEM || !want_own) return without(rc);
        (void)hipGetLastError();
        c->blk16.release();
        want_f16 = false;
    }
    if ((rc = c->norm.reserve(ng * 32 * 4)) != VF_OK) return without(rc);
    if ((rc = c->map.reserve(ng * 32 * 4)) != VF_OK) return without(rc);
    if ((rc = upload(c->goff, tables, s)) != VF_OK) return without(rc);
    auto on_device = [&](const void *host) { return (void *)(c->goff.as<char>() + ((const char *)host - (const char *)tables.data())); };
    const int32_t *d_cnt = (const int32_t *)on_device(grp_cnt);
    launch_seed_map(ix->d_M_HS.as<int32_t>(), (const int64_t *)on_device(slot_base), (const int32_t *)on_device(slot_n), n_seeds,
                    (const int32_t *)on_device(grp_slot), (const int32_t *)on_device(grp_j0), n_groups, c->map.as<int32_t>(), s);
    if (want_own)
        launch_interleave(ix->dtype, ix->X, ix->dim, c->map.as<int32_t>(), (const int64_t *)on_device(grp_src), d_cnt, n_groups * 32, n_groups,
                          ix->ncp, c->blk.as<uint4>(), c->norm.p, s);
    float mx = 0.f;
    if (want_f16) {
        // float32 data: the copy in binary16; the largest rounding error of a seed goes into the beam kernel's proof (zero for
        // integer-valued data of up to 11 bits, SIFT's kind)
        uint32_t *d_err2 = (uint32_t *)on_device(err2);
        if (want_own) launch_seed_pack_f16(c->blk.as<uint4>(), n_groups, ix->ncp, ix->seed_scale(), c->blk16.as<uint4>(), d_err2, s);
        else launch_seed_rows_f16(ix->X, ix->dim, c->map.as<int32_t>(), d_cnt, n_groups, ix->ncp, ix->seed_scale(), c->blk16.as<uint4>(), c->norm.as<float>(), d_err2, s);
        VF_HIP(hipMemcpyAsync(&mx, d_err2, 4, hipMemcpyDeviceToHost, s));
    }
    VF_HIP(hipGetLastError());
    VF_HIP(hipStreamSynchronize(s));   // (the tables are pageable host memory)
    c->has_f32 = want_own;
    if (want_f16) {
        if (mx >= 0.f && mx <= 3.0e38f) {
            c->has_f16 = true;
            c->f16_delta = (float)(std::sqrt((double)mx) * 1.001);
        }
    }
    c->ok = c->has_f32 || c->has_f16;
    return VF_OK;
}

// ---------------------------------------------------------------- one search call: plan, blob, launches

int check_search_params(const vf_index *ix, bool exact, int32_t k, int32_t &itopk, int32_t width, int32_t iters,
                               int32_t &n_seeds)
{
    if (exact) return VF_OK;
    VF_REQUIRE(itopk >= k && itopk >= 1 && itopk <= 256, "itopk must be in [k, 256]");
    VF_REQUIRE(width >= 1 && width <= 8 && width * ix->R <= 128, "width must be >= 1 with width * R <= 128");
    VF_REQUIRE(iters >= 0, "iters must be >= 0");
    VF_REQUIRE(n_seeds >= 0, "n_seeds must be >= 0");
    if (n_seeds == 0) n_seeds = itopk;
    return VF_OK;
}

// How joined lists are cut into work items.
struct JoinTiles {
    int kernel;       // rows a workgroup of the kernel can take (kJoinRows, kJoinRowsShared)
    int rows;         // ... and is given
    int seg_groups;   // groups of a segment
};

// lists: groups and rows of each.  A row's thresholds start over in each segment, so no more of them than keep the chip busy: two
// workgroups of four waves per CU at a time, eight of one wave; three rounds of them level out the last one (with a third of
// that, 4,250 queries over 51 lists 8 % less to 8 % more).  Where tiles of 32
// rows leave most SIMDs without a wave, smaller ones: a wave's selection takes longer than reading the list, and is a matter of
// its rows and of what is kept of each (lists of 20,000 / 133,000 x 128 float32, 32 queries: k = 10 336 -> 196 and 471 -> 307 us,
// k = 48 599 -> 265 and 716 -> 426; a shared reading of the list by four waves, as before there were tiles of one, took 413, 505, 538
// and 632).
static JoinTiles join_tiles(int kind, int32_t dim, const std::vector<std::pair<int64_t, int64_t>> &lists)
{
    constexpr int64_t kShort = 64;
    auto count = [&](int64_t rows, int64_t seg) {
        int64_t c = 0;
        for (const auto &l : lists) c += ((l.second + rows - 1) / rows) * (seg > 0 ? (l.first + seg - 1) / seg : l.first);
        return c;
    };
    JoinTiles t;
    t.kernel = t.rows = join_tile_rows(kind, dim);
    if (t.kernel == kJoinRows)
        while (t.rows > 8 && count(t.rows, kShort) < 1024) t.rows /= 2;
    t.seg_groups = (int)std::max<int64_t>(kShort, count(t.rows, 0) / (t.kernel == kJoinRows ? 6144 : 1536));
    return t;
}

// Routing, work lists, blob layout.  budget: how large a seed distance matrix may be (beyond it the
// beam kernel gathers the seeds itself).
int plan_call(const vf_index *ix, Routed &r, int64_t nq, const int64_t *qoff, const int32_t *qids, bool exact,
                     bool first_is_searched, int32_t k, int32_t itopk, int32_t width, int32_t iters, int32_t n_seeds,
                     int32_t and_scan_limit, SeedBudget budget, const SeedCopyMaker *make, SeedCopy *&sc, CallPlan &P)
{
    int rc;
    P.nq = nq; P.k = k; P.itopk = itopk; P.width = width; P.iters = iters; P.n_seeds = n_seeds; P.exact = exact;
    if (!exact) {
        while (P.beam_LP < itopk + std::max(64, width * ix->R)) P.beam_LP <<= 1;
        const int64_t visits = (int64_t)iters * width * ix->R;
        while (P.beam_hb < 13 && ((int64_t)1 << P.beam_hb) < 2 * visits) ++P.beam_hb;
        BeamParams chk{};
        chk.dim = ix->dim; chk.LP = P.beam_LP; chk.hash_bits = P.beam_hb;
        VF_REQUIRE(beam_lds_bytes(chk, ix->dtype) <= 64 * 1024, "search parameters need more than 64 KiB of LDS");
        // The visited table is most of a wave's LDS, and no result depends on its size.  A batch of more queries than can be
        // resident with it gets half of it, as long as a CU then still holds fewer than 24 waves and the table half of the
        // edges that are looked at (of those one to four in ten are met for the first time): 50,000 uint8 queries at 32
        // iterations, 9.9 KiB and 16 waves -> 5.9 KiB and 27, 2.08 -> 1.80 ms.  Batches that are resident anyway keep it
        // (1,777 queries of 48 edges x 24 iterations: 193 us with 16 KiB, 199 with 4).
        auto crowded = [&]() {
            chk.hash_bits = P.beam_hb;
            const int64_t waves = 160 * 1024 / (int64_t)beam_lds_bytes(chk, ix->dtype);
            return waves < 24 && nq > 256 * waves;
        };
        while (P.beam_hb > 9 && ((int64_t)1 << P.beam_hb) >= visits && crowded()) --P.beam_hb;
    }
    VF_REQUIRE(scan_lds_bytes(ix->ncp, exact ? 32 : std::max(P.ib.tile_rows, 16), k) <= 64 * 1024,
               "the scan tile of this dim and k needs more than 64 KiB of LDS");
    if ((rc = route_queries(ix->route_view(), nq, qoff, qids, exact, first_is_searched, r)) != VF_OK) return rc;

    // scan items over the stored interleaved lists (scan labels); in exact mode graph labels follow
    ItemBuilder &ib = P.ib;
    size_t first_hs = r.scan_pairs.size();
    // float32 lists of large batches are filtered from their bfloat16 copy and re-ranked (every item then leaves
    // partial rows of scan_keep candidates and every scan query gets a merge item); small batches keep the FMA kernel
    {
        const Tuning &tn = ix->tune;
        const int32_t keep = std::min(64, k + tn.scan_bf16_margin);
        const bool small_batch = tn.scan_valu == 2 || (tn.scan_valu == 1 && r.scan_pairs.size() <= 256);
        if (ix->has_ls16 && tn.scan_bf16 && tn.scan16 && !small_batch && keep > k &&
            !r.scan_pairs.empty() && scan_bf16_supported(ix->dtype, ix->dim, ib.tile_rows, keep) &&
            scan_bf16_lds_bytes(std::max(ib.tile_rows, 16), keep) <= 64 * 1024) {
            P.scan_bf16 = true;
            P.scan_keep = keep;
            ib.all_partial = true;
            ib.seg_groups = ib.seg_groups_heavy = tn.scan_bf16_seg_groups;
        }
    }
    if (exact) {
        // scan labels first, graph labels after them (both still ordered by label)
        std::stable_partition(r.scan_pairs.begin(), r.scan_pairs.end(), [&](uint64_t pr) {
            return ix->O_LS[(size_t)(pr >> 32)] >= 0;
        });
        first_hs = 0;
        while (first_hs < r.scan_pairs.size() && ix->O_LS[(size_t)(r.scan_pairs[first_hs] >> 32)] >= 0) ++first_hs;
    }
    ib.qrow.reserve(r.scan_pairs.size());     // (no regrowth while the work lists are built)
    ib.items.reserve(r.scan_pairs.size());
    ib.merges.reserve(r.scan_pairs.size());
    // A launch with fewer work items than SIMDs lasts as long as its longest item, and an item is one wave's serial chain:
    // short lists are then cut into up to eight segments (1,000 queries on lists of up to 500 uint8 vectors, 60 items of
    // 16 groups: 63 us, in segments of two groups 28 us and 7 us for the merge).
    const bool cut_short = !P.scan_bf16 && !P.tight;
    int64_t tile_groups = 0;
    if (cut_short)
        for (size_t i = 0; i < first_hs;) {
            const uint64_t l = r.scan_pairs[i] >> 32;
            size_t e = i;
            while (e < first_hs && r.scan_pairs[e] >> 32 == l) ++e;
            tile_groups += (int64_t)((e - i + ib.tile_rows - 1) / ib.tile_rows) * ((ix->S[(size_t)l] + 31) / 32);
            i = e;
        }
    const int seg_default = ib.seg_groups, seg_heavy = ib.seg_groups_heavy;
    for (size_t i = 0; i < first_hs;) {
        const int32_t l = (int32_t)(r.scan_pairs[i] >> 32);
        size_t e = i;
        while (e < first_hs && (int32_t)(r.scan_pairs[e] >> 32) == l) ++e;
        if (cut_short) {
            const int least = (int)std::max<int64_t>(2, std::max<int64_t>(tile_groups / 1024, (ix->S[(size_t)l] + 255) / 256));
            ib.seg_groups = std::min(seg_default, least);
            ib.seg_groups_heavy = std::min(seg_heavy, least);
        }
        ib.add_label(r.scan_pairs, i, e, ix->GO_LS[(size_t)l], ix->O_LS[(size_t)l], ix->S[(size_t)l]);
        i = e;
    }
    // (graph lists of exact mode: what the scan lists' kernels and sizes have asked for is not theirs)
    ib.seg_groups = ix->tune.seg_groups; ib.seg_groups_heavy = ix->tune.seg_groups_heavy;
    P.n_ls_items = ib.items.size(); P.n_ls_merges = ib.merges.size();
    const size_t ls_qrows = ib.qrow.size();
    VF_REQUIRE(ib.part_rows < ((int64_t)1 << 31), "too many partial result rows in one call");
    P.ls_part_words = P.part_words = (size_t)ib.part_rows * (P.scan_bf16 ? P.scan_keep : k);
    // Exact mode, graph lists: packed copies of all of them (as many as fit into a GiB, or one that is larger) and one join
    // over their queries.  float32 keeps spare candidates and proves the re-ranked result, which needs the norms to be
    // within the proofs' range and room for enough spare ones.
    const int32_t join_keep = ix->dtype == VF_U8 ? k : std::min(64, k + 22);
    const bool joined = exact && P.join_bytes > 0 && first_hs < r.scan_pairs.size() && ix->join_norms() != nullptr &&
                        (ix->dtype == VF_U8 || (ix->xc_max > 0.f && ix->tune.scan_bf16 && join_keep >= k + 16));
    if (joined) {
        P.join_keep = join_keep;
        P.join_kind = ix->exact_kind(k);
        ItemBuilder jb(ix->tune);
        jb.all_partial = true;
        std::vector<std::pair<int64_t, int64_t>> list_rows;
        for (size_t i = first_hs, e; i < r.scan_pairs.size(); i = e) {
            const uint64_t l = r.scan_pairs[i] >> 32;
            for (e = i; e < r.scan_pairs.size() && r.scan_pairs[e] >> 32 == l;) ++e;
            list_rows.emplace_back((ix->S[(size_t)l] + 31) / 32, (int64_t)(e - i));
        }
        const JoinTiles tiles = join_tiles(P.join_kind, ix->dim, list_rows);
        P.join_tile = tiles.kernel;
        jb.tile_rows = tiles.rows;
        jb.seg_groups = jb.seg_groups_heavy = tiles.seg_groups;
        const int64_t batch_groups = (int64_t)(P.join_bytes / join_group_bytes(ix->join_kind_max(), ix->dim));
        int64_t groups = 0;
        JoinBatch b{0, 0, 0, 0, 0};
        auto close = [&]() {
            b.list_hi = P.jlists.size(); b.item_hi = jb.items.size(); b.groups = groups;
            // every tile's first segment before any second one: what the first find bounds the others
            std::stable_sort(jb.items.begin() + (std::ptrdiff_t)b.item_lo, jb.items.end(), [](const ScanItem &x, const ScanItem &y) { return x.entry0 < y.entry0; });
            P.jbatches.push_back(b);
            P.join_groups = std::max(P.join_groups, groups);
            b.list_lo = b.list_hi; b.item_lo = b.item_hi; groups = 0;
        };
        for (size_t i = first_hs, e; i < r.scan_pairs.size(); i = e) {
            const int32_t l = (int32_t)(r.scan_pairs[i] >> 32), n = ix->S[(size_t)l];
            for (e = i; e < r.scan_pairs.size() && (int32_t)(r.scan_pairs[e] >> 32) == l;) ++e;
            const int64_t ng = (n + 31) / 32;
            if (groups > 0 && groups + ng > batch_groups) close();
            P.jlists.push_back(JoinList{ix->O_HS[(size_t)l], (int32_t)groups, n});
            jb.add_label(r.scan_pairs, i, e, groups, ix->O_HS[(size_t)l], n);
            groups += ng;
        }
        close();
        for (ScanItem &it : jb.items) it.q_begin += (int32_t)ls_qrows;
        VF_REQUIRE(jb.part_rows < ((int64_t)1 << 31), "too many partial result rows in one call");
        P.part_words += (size_t)jb.part_rows * join_keep;
        P.join_bound_at = P.part_words;
        P.join_first_row = ls_qrows;
        P.join_rows = jb.qrow.size();
        P.part_words += P.join_rows;
        P.join_max_nseg = jb.max_nseg;
        ib.qrow.insert(ib.qrow.end(), jb.qrow.begin(), jb.qrow.end());
        ib.items.insert(ib.items.end(), jb.items.begin(), jb.items.end());
        ib.merges.insert(ib.merges.end(), jb.merges.begin(), jb.merges.end());
    } else
    // ... or one temporary interleaved copy per graph label, used right after it is made
    for (size_t i = first_hs; i < r.scan_pairs.size();) {
        const int32_t l = (int32_t)(r.scan_pairs[i] >> 32);
        size_t e = i;
        while (e < r.scan_pairs.size() && (int32_t)(r.scan_pairs[e] >> 32) == l) ++e;
        const size_t lo = ib.items.size();
        ib.add_label(r.scan_pairs, i, e, 0, ix->O_HS[(size_t)l], ix->S[(size_t)l]);
        P.hs_runs.push_back({l, lo, ib.items.size()});
        P.max_hs_list = std::max(P.max_hs_list, ix->S[(size_t)l]);
        i = e;
    }
    if (!joined) {
        VF_REQUIRE(ib.part_rows < ((int64_t)1 << 31), "too many partial result rows in one call");
        P.part_words = (size_t)ib.part_rows * (P.scan_bf16 ? P.scan_keep : k);
    }

    // selectivity-aware routing: AND queries whose (smallest) graph list is short leave the graph path
    r.xq_query.clear(); r.xq_label.clear();
    if (!exact && and_scan_limit > 0 && r.any_and) {
        size_t w = 0;
        for (size_t i = 0; i < r.gq_query.size(); ++i) {
            const int32_t q = r.gq_query[i], l = r.gq_label[i];
            if (r.others_off[(size_t)q + 1] > r.others_off[(size_t)q] && ix->S[(size_t)l] <= and_scan_limit) {
                r.xq_query.push_back(q); r.xq_label.push_back(l);
            } else {
                r.gq_query[w] = q; r.gq_label[w] = l; ++w;
            }
        }
        r.gq_query.resize(w); r.gq_label.resize(w);
    }
    P.n_xq = r.xq_query.size();
    P.n_gq = r.gq_query.size();
    // (a list has no more seeds than entries: with seed counts beyond any list's length, "every entry", the rows of the matrix and the
    // grids of its kernels are as long as the longest list)
    P.ns_top = n_seeds;
    if (n_seeds > 1 << 23) {
        int32_t longest = 1;
        for (const int32_t l : ix->graph_labels) longest = std::max(longest, ix->S[(size_t)l]);
        P.ns_top = std::min(n_seeds, longest);
    }
    const int32_t ns_blocks = (int32_t)(((int64_t)P.ns_top + 31) / 32);
    P.ns_stride = (int32_t)((int64_t)ns_blocks * 32 <= INT32_MAX ? ns_blocks * 32 : INT32_MAX & ~31);
    auto and_queries = [&] {   // graph queries with a predicate
        int64_t n = 0;
        if (r.any_and)
            for (size_t i = 0; i < P.n_gq; ++i) n += r.others_off[(size_t)r.gq_query[i] + 1] > r.others_off[(size_t)r.gq_query[i]] ? 1 : 0;
        return n;
    };
    // every distance goes through the seed distance matrix, which must fit
    const uint64_t matrix = (uint64_t)P.n_gq * (uint64_t)P.ns_stride;
    // Seeds on the matrix cores.  uint8: they give the exact integer distances, nothing else changes.
    // float32: approximations, re-ranked by the beam kernel (its proof under a predicate needs a list of at most 48 entries).
    // (a tile's rows are addressed by 32-bit offsets)
    const bool own_dim = seed_mfma_own(ix->dtype, ix->dim);
    bool mfma_ok = wants_seed_copy(ix, exact, itopk, n_seeds) && P.n_gq > 0 && P.ns_stride <= 1 << 23 && (ix->dtype == VF_U8 || itopk <= 48 || !r.any_and);
    auto dist_pays = [&] { return seed_dist_pays(ix->dtype, ix->dim, P.ns_top, (int64_t)P.n_gq, seed_dist_own(ix->dtype, ix->dim) ? 0 : and_queries()); };
    // float32 vectors of more than 32 chunks in batches of mostly predicates: a wave that gathers tests the predicate first and scores
    // what passes, so the launch pays from about 80 passing seeds a query on, taking the labels as independent.  One query, gathering
    // -> on the matrix cores, at 20 / 60 / 90 / 150 passing seeds: 160 components 25 / 37 / 38 / 64 -> 36 / 39 / 39 / 48 us, 232
    // 27 / 40 / 39 / 68 -> 38 / 41 / 40 / 49.
    auto few_pass = [&] {
        if (ix->dtype != VF_F32 || ix->dim <= 128 || 2 * and_queries() <= (int64_t)P.n_gq) return false;
        double passing = 0.0;
        int64_t n_and = 0;
        for (size_t i = 0; i < P.n_gq; ++i) {
            const int32_t b = r.others_off[(size_t)r.gq_query[i]], e = r.others_off[(size_t)r.gq_query[i] + 1];
            if (e == b) continue;
            double pass = std::min(n_seeds, ix->S[(size_t)r.gq_label[i]]);
            for (int32_t o = b; o < e; ++o) pass *= (double)ix->S[(size_t)r.others[(size_t)o]] / (double)ix->n;
            passing += pass;
            ++n_and;
        }
        return passing < 80.0 * (double)n_and;
    };
    auto mfma_pays = [&] { return seed_mfma_pays(ix->dtype, ix->dim, itopk, P.ns_top, (int64_t)P.n_gq) && !few_pass(); };
    // A copy of the seeds is made by the first call that scores from it.  Dimensions without an instantiation of their own are
    // scored from the copy only.
    if (mfma_ok && make != nullptr && sc == nullptr &&
        (own_dim || ((mfma_pays() || dist_pays()) && budget.fits(matrix))) &&
        (rc = seed_copy_for(make->ix, n_seeds, make->stream, true, &sc)) != VF_OK)
        return rc;
    if (!own_dim && (P.tight || sc == nullptr || !sc->ok || (ix->dtype == VF_F32 && !sc->has_f16))) mfma_ok = false;
    // With an interleaved seed copy the seed kernel also selects (itopk <= 64: the beam kernel's one-register
    // list): it leaves sel_K keys per (query, seed segment) instead of every distance.  float32 data: from the
    // binary16 copy; calls with few graph queries keep the float32 copy and the unfused kernel (see
    // seed_bf16_min_batch).
    const Tuning &tune = ix->tune;
    if (mfma_ok && sc != nullptr && sc->ok && tune.seed_select && itopk <= 64 &&
        seed_select_supported(ix->dtype, ix->dim, sc->has_f16) &&
        (ix->dtype == VF_U8 || !sc->has_f32 || (int64_t)P.n_gq >= tune.seed_bf16_min_batch)) {
        P.sel_f16 = ix->dtype == VF_F32;
        P.sel_K = ix->dtype == VF_U8 ? itopk : std::min(64, itopk + std::max(tune.seed_margin_bf16, tune.seed_margin));
        int32_t longest = 0;
        size_t n_tiles = 0;
        for (size_t i = 0; i < P.n_gq;) {
            size_t e = i;
            while (e < P.n_gq && r.gq_label[e] == r.gq_label[i]) ++e;
            longest = std::max(longest, std::min(n_seeds, ix->S[(size_t)r.gq_label[i]]));
            n_tiles += (e - i + 31) / 32;
            i = e;
        }
        // seeds per wave: long segments select better (a row's threshold tightens as the segment streams by) but
        // the launch needs a few thousand waves
        int32_t seg = tune.seed_seg_seeds;
        if (seg <= 0) {
            const int64_t want_segs = std::max<int64_t>(1, (2048 + (int64_t)n_tiles - 1) / (int64_t)n_tiles);
            seg = (int32_t)std::min<int64_t>(16384, std::max<int64_t>(512, (longest / want_segs) / 32 * 32));
        }
        seg = std::max(32, seg / 32 * 32);
        P.seg_seeds = seg;
        P.max_segs = (longest + seg - 1) / seg;
        const uint64_t need = (uint64_t)P.n_gq * (uint64_t)P.max_segs * (uint64_t)P.sel_K * 2;   // 8-byte keys
        if (budget.fits(need)) {
            P.seed_select = true;
            P.dense_seeds = P.seeds_mfma = true;
            P.dseed_words = (size_t)need;
        }
    }
    if (!P.seed_select) {
        // (the driver is asked last: 12 us of a call that gathers its seeds)
        P.dense_seeds = !exact && P.n_gq > 0 && ((mfma_ok && mfma_pays()) || dist_pays()) &&
                        budget.fits(matrix);
        P.seeds_mfma = P.dense_seeds && mfma_ok;
        if (P.dense_seeds) P.dseed_words = (size_t)matrix;
    }
    if (P.dense_seeds) {
        // (without the watch on failed proofs, which needs a pinned counter, the binary16 form is used only where it is the only one)
        P.seeds_f16 = P.seeds_mfma && ix->dtype == VF_F32 && sc != nullptr && sc->ok && sc->has_f16 &&
                      (!sc->has_f32 || !own_dim || (!P.tight && (int64_t)P.n_gq >= tune.seed_bf16_min_batch));
        size_t tile_q = P.seed_select ? 32 : P.seeds_mfma ? (size_t)seed_mfma_tile_of(ix->dtype, ix->dim, P.seeds_f16) : 64;
        // (launches that would leave SIMDs without a wave even at 128 seeds a wave: smaller tiles)
        if (P.seeds_mfma && (int64_t)(P.n_gq / 64) * ((P.ns_top + kSeedMfmaChunk - 1) / kSeedMfmaChunk) < 1024) tile_q = 32;
        for (size_t i = 0; i < P.n_gq;) {
            size_t e = i;
            while (e < P.n_gq && r.gq_label[e] == r.gq_label[i]) ++e;
            for (size_t t = i; t < e; t += tile_q)
                P.tiles.push_back(SeedTile{r.gq_label[i], (int32_t)t, (int32_t)std::min<size_t>(tile_q, e - t)});
            i = e;
        }
    }
    // The minima of the seeds' blocks, where the seeds come from their copy and enough queries can use them: no predicate, and
    // three blocks per list entry or more (fewer: most blocks would be read anyway), float32 two.  50,000 uint8 queries with 16,384 seeds:
    // seed kernel 805 -> 825 us, beam kernel 1,561 -> 1,260; 10,000 float32 queries with 6,144 seeds: 107 -> 115 and 269 ->
    // 221 us; a lone query, whose wave otherwise goes through
    // the whole row by itself, 74 -> 65 us, 64 queries 109 -> 103.
    if (P.seeds_mfma && !P.seed_select && !P.tight && sc != nullptr && sc->ok && (ix->dtype == VF_U8 || !r.any_and)) {
        const int32_t stride = (ns_blocks + 15) & ~15;
        if (ns_blocks >= (ix->dtype == VF_U8 ? 3 : kSeedMinimaF32) * itopk && 2 * and_queries() <= (int64_t)P.n_gq && budget.fits((uint64_t)P.dseed_words + (uint64_t)P.n_gq * (uint64_t)stride)) {
            P.nb_stride = stride;
            P.dseed_words += P.n_gq * (size_t)stride;
        }
    }
    BlobLayout &L = P.L;
    size_t o = 0;
    L.off_gq_query = o; o = align_up(o + P.n_gq * 4);
    L.off_gq_label = o; o = align_up(o + P.n_gq * 4);
    L.off_xq_query = o; o = align_up(o + P.n_xq * 4);
    L.off_xq_label = o; o = align_up(o + P.n_xq * 4);
    L.off_others_off = o; o = align_up(o + (r.any_and ? r.others_off.size() : 1) * 4);   // (not sent when no query has partners)
    L.off_others = o; o = align_up(o + std::max<size_t>(r.others.size(), 1) * 4);
    L.off_qrow = o; o = align_up(o + std::max<size_t>(ib.qrow.size(), 1) * 4);
    L.off_items = o; o = align_up(o + std::max<size_t>(ib.items.size(), 1) * sizeof(ScanItem));
    L.off_merges = o; o = align_up(o + std::max<size_t>(ib.merges.size(), 1) * sizeof(MergeItem));
    L.off_tiles = o; o = align_up(o + std::max<size_t>(P.tiles.size(), 1) * sizeof(SeedTile));
    L.off_empty = o; o = align_up(o + std::max<size_t>(r.empty_q.size(), 1) * 4);
    L.off_jlists = o; o = align_up(o + P.jlists.size() * sizeof(JoinList));
    L.total = o;
    return VF_OK;
}

// The routing blob in host memory (hp holds P.L.total bytes).
void fill_blob(const CallPlan &P, const Routed &r, char *hp)
{
    const BlobLayout &L = P.L;
    const ItemBuilder &ib = P.ib;
    if (P.n_gq) {
        memcpy(hp + L.off_gq_query, r.gq_query.data(), P.n_gq * 4);
        memcpy(hp + L.off_gq_label, r.gq_label.data(), P.n_gq * 4);
    }
    if (P.n_xq) {
        memcpy(hp + L.off_xq_query, r.xq_query.data(), P.n_xq * 4);
        memcpy(hp + L.off_xq_label, r.xq_label.data(), P.n_xq * 4);
    }
    if (r.any_and) memcpy(hp + L.off_others_off, r.others_off.data(), r.others_off.size() * 4);
    if (!r.others.empty()) memcpy(hp + L.off_others, r.others.data(), r.others.size() * 4);
    if (!ib.qrow.empty()) memcpy(hp + L.off_qrow, ib.qrow.data(), ib.qrow.size() * 4);
    if (!ib.items.empty()) memcpy(hp + L.off_items, ib.items.data(), ib.items.size() * sizeof(ScanItem));
    if (!ib.merges.empty()) memcpy(hp + L.off_merges, ib.merges.data(), ib.merges.size() * sizeof(MergeItem));
    if (!P.tiles.empty()) memcpy(hp + L.off_tiles, P.tiles.data(), P.tiles.size() * sizeof(SeedTile));
    if (!P.jlists.empty()) memcpy(hp + L.off_jlists, P.jlists.data(), P.jlists.size() * sizeof(JoinList));
    if (!r.empty_q.empty()) memcpy(hp + L.off_empty, r.empty_q.data(), r.empty_q.size() * 4);
}

// The bounds of approximations from the binary16 copy (see vf_seed.hip): 2048 u, and dx; |q^| <= |q| (1 + 2^-11) and a little.
void half_bound(const vf_index *ix, float delta, BeamParams &b)
{
    b.err_bound = ix->seed_err_bound() * 4.0f;
    b.err_q = 2.002f * delta;
    b.scale = ix->seed_scale();
    b.q_max = 1.07374182e9f / (b.scale * b.scale);   // 2^30: the scaled length is below 2^15
}

// The launches of one call.  s: the caller's stream; side: the stream the scan path runs on beside the graph path
// (ev_fork / ev_join tie it to s), or nullptr: everything on s.  may_allocate = false (the entry point that
// allocates nothing): no seed copy is built, no profiling, no failed-proof watch.
int launch_call(vf_index *ix, const CallPlan &P, const Routed &r, const CallMem &M, const SeedCopy *sc, const void *queries,
                int64_t *out_ids, float *out_dists, hipStream_t s, hipStream_t side, hipEvent_t ev_fork, hipEvent_t ev_join,
                bool may_allocate)
{
    int rc;
    const Tuning &tune = ix->tune;
    const BlobLayout &L = P.L;
    const ItemBuilder &ib = P.ib;
    char *dp = M.blob;
    const int32_t k = P.k;
    const size_t n_gq = P.n_gq;
    const bool forked = side != nullptr;
    const bool exact = P.exact;

    // every routed query's kernel writes all k entries of its row; only queries without any match are padded here
    launch_fill_rows(out_ids, out_dists, (const int32_t *)(dp + L.off_empty), (int64_t)r.empty_q.size(), k, s);

    const bool prof = may_allocate && ix->profiling;
    if (prof) {
        if (ix->prof_unfolded == vf_index::kProfRing && (rc = fold_profile(ix, 1)) != VF_OK) return rc;
        ix->prof_ev = ix->prof_ring[ix->prof_next];
        // [nq][4] counters, then [nq] gathered; written by the beam kernel for graph queries only (no clearing
        // pass: the rows of the other queries are never read)
        if ((rc = ix->counters.reserve((size_t)P.nq * 24)) != VF_OK) return rc;
        ix->prof_graph_queries = r.gq_query;
        ix->prof_graph_queries.insert(ix->prof_graph_queries.end(), r.xq_query.begin(), r.xq_query.end());
        vf_profile &pf = ix->prof;
        pf = vf_profile{};
        pf.nq = P.nq; pf.n_graph_queries = (int64_t)r.gq_query.size(); pf.n_scan_queries = (int64_t)ib.qrow.size();
        pf.n_scan_items = (int64_t)ib.items.size();
        for (const ScanItem &it : ib.items) { pf.scan_list_entries += it.n; pf.scan_pairs += (int64_t)it.n * it.q_count; }
        pf.n_seed_tiles = (int64_t)P.tiles.size();
        pf.seeds_on_matrix_cores = P.seeds_mfma ? 1 : 0;
        for (const SeedTile &t : P.tiles) {
            const int64_t ns_l = std::min<int64_t>(P.n_seeds, ix->S[(size_t)t.label]);
            pf.seed_pairs += ns_l * t.q_count;
            pf.seed_tile_seeds += ns_l;
        }
    }
    hipStream_t ss = s;
    const int32_t *d_others_off = r.any_and ? (const int32_t *)(dp + L.off_others_off) : nullptr;
    const int32_t *d_others = (const int32_t *)(dp + L.off_others);

    BeamParams bp{};
    if (n_gq || P.n_xq) {
        bp.X = ix->X; bp.Q = queries; bp.G = ix->d_G.as<int32_t>(); bp.Gg = ix->d_Gg.as<int32_t>();
        bp.gq_query = (const int32_t *)(dp + L.off_gq_query);
        bp.gq_label = (const int32_t *)(dp + L.off_gq_label);
        bp.others_off = d_others_off; bp.others = d_others; bp.meta = ix->meta();
        bp.dim = ix->dim; bp.R = ix->R; bp.k = k; bp.itopk = P.itopk; bp.width = P.width; bp.iters = P.iters;
        bp.n_seeds = P.n_seeds;
        bp.lat_waves = ix->tune.beam_lat_waves;
        bp.LP = P.beam_LP;
        bp.hash_bits = P.beam_hb;
        bp.out_ids = out_ids; bp.out_dists = out_dists;
        bp.counters = prof ? ix->counters.as<int32_t>() : nullptr;
        bp.gathered = prof ? ix->counters.as<int32_t>() + (size_t)P.nq * 4 : nullptr;
        bp.dseed = nullptr; bp.ns_stride = P.ns_stride;
    }
    // While profiling, the beam kernel's launch takes the two events that bracket it (end of seed scoring = its begin,
    // and its end) as the kernel's own begin and end times: events recorded around it would each put a barrier packet
    // on the stream, and the timed kernels a few microseconds apart.
    const bool attach = prof && n_gq > 0 && P.n_xq == 0;
    auto count_passing_seeds = [&]() {
        if (prof && ix->prof_exact_counts && n_gq && (P.seed_select || P.dense_seeds) && r.any_and) {
            // profiling only, outside the timed interval: the counters report the seeds that pass the predicate as
            // distances computed, and neither the selecting seed kernel nor the beam kernel's selection from a
            // row of seed distances tests the seeds that cannot enter a full list
            launch_seed_pass_count(bp.gq_query, bp.gq_label, bp.meta, P.n_seeds, d_others_off, d_others,
                                   ix->counters.as<int32_t>() + (size_t)P.nq * 5, (int)n_gq, s);
        }
    };
    auto run_seeds = [&]() -> int {
        // (a profiled call that forks has recorded this event already: it is its fork event)
        if (prof && !forked) VF_HIP(hipEventRecord(ix->prof_ev[2], s));
        if (n_gq && P.seed_select) {
            // scoring and selection in one kernel: runs of sel_K keys per (query, seed segment)
            SeedSelParams sl{};
            sl.Q = queries; sl.gq_query = bp.gq_query;
            sl.tiles = (const SeedTile *)(dp + L.off_tiles); sl.meta = bp.meta;
            sl.dim = ix->dim; sl.n_seeds = P.n_seeds; sl.K = P.sel_K; sl.seg_seeds = P.seg_seeds; sl.max_segs = P.max_segs;
            sl.seed_blk = P.sel_f16 ? sc->blk16.as<uint4>() : sc->blk.as<uint4>();
            sl.seed_norm = sc->norm.as<uint32_t>();
            sl.seed_goff = sc->goff.as<int64_t>();
            sl.seed_map = sc->map.as<int32_t>();
            sl.others_off = d_others_off; sl.others = d_others;
            sl.runs = (uint64_t *)M.dseed;
            sl.scale = ix->seed_scale(); sl.minus_two_unscaled = -2.0f / (sl.scale * sl.scale);
            launch_seed_select(ix->dtype, sl, (int)P.tiles.size(), s);
            bp.seed_runs = sl.runs; bp.run_K = P.sel_K; bp.run_segs = P.max_segs; bp.seg_seeds = P.seg_seeds;
            if (prof) {
                ix->prof.seeds_on_matrix_cores = P.sel_f16 ? 2 : 1;
                ix->prof.seed_selected = 1;
                for (const SeedTile &t : P.tiles) {
                    const int64_t ns_l = std::min<int64_t>(P.n_seeds, ix->S[(size_t)t.label]);
                    ix->prof.seed_run_keys += (int64_t)t.q_count * ((ns_l + P.seg_seeds - 1) / P.seg_seeds) * P.sel_K;
                }
                if (ix->prof_exact_counts && r.any_and) bp.seed_pass = ix->counters.as<int32_t>() + (size_t)P.nq * 5;   // filled before the timed interval
            }
            if (ix->dtype == VF_F32) {
                bp.seed_approx = 1; bp.xn_max = ix->xn_max;
                half_bound(ix, sc->f16_delta, bp);
                bp.seed_keep = P.sel_K;
                if (may_allocate) bp.fallback_count = ix->d_fb_count.as<uint32_t>();
            }
        } else if (n_gq && P.dense_seeds) {
            SeedParams sd{};
            sd.X = ix->X; sd.Q = queries; sd.gq_query = bp.gq_query;
            sd.tiles = (const SeedTile *)(dp + L.off_tiles); sd.meta = bp.meta;
            sd.dim = ix->dim; sd.n_seeds = P.n_seeds; sd.ns_stride = P.ns_stride;
            sd.dseed = M.dseed;
            sd.scale = ix->seed_scale(); sd.minus_two_unscaled = -2.0f / (sd.scale * sd.scale);
            if (P.seeds_mfma) {
                sd.chunk_seeds = kSeedMfmaChunk;
                sd.max_chunks = (P.ns_top + kSeedMfmaChunk - 1) / kSeedMfmaChunk;
                sd.xnorm_all = ix->d_xnorm_all.as<uint32_t>();
                float seed_delta = 0.f;
                if (sc != nullptr && sc->ok) {
                    const bool use16 = P.seeds_f16;
                    sd.blk_chunks = use16 ? ix->ncp : 2 * ix->ncp;
                    sd.seed_blk = use16 ? sc->blk16.as<uint4>() : sc->blk.as<uint4>();
                    sd.seed_norm = sc->norm.as<uint32_t>();
                    sd.seed_goff = sc->goff.as<int64_t>();
                    sd.seed_f16 = use16 ? 1 : 0;
                    seed_delta = sc->f16_delta;
                    if (prof && sd.seed_f16) ix->prof.seeds_on_matrix_cores = 2;
                    // seeds per wave: few long waves share the chip better with the scan (512 seeds:
                    // step 0.374 -> 0.340 ms on 10,000-query batches), small batches need many short ones
                    sd.chunk_seeds = 4 * kSeedMfmaChunk;
                    if ((int64_t)P.tiles.size() * ((P.ns_top + sd.chunk_seeds - 1) / sd.chunk_seeds) < 512)
                        sd.chunk_seeds = kSeedMfmaChunk;
                    // a launch that leaves most SIMDs without a wave even so (a handful of queries): a wave per group of
                    // 32 seeds, its four groups' serial chain of MFMAs cut to one
                    if ((int64_t)P.tiles.size() * ((P.ns_top + kSeedMfmaChunk - 1) / kSeedMfmaChunk) < 256) sd.chunk_seeds = 32;
                    sd.max_chunks = (P.ns_top + sd.chunk_seeds - 1) / sd.chunk_seeds;
                    if (P.nb_stride > 0) {
                        sd.dmin = M.dseed + (P.dseed_words - n_gq * (size_t)P.nb_stride);   // (behind the matrix)
                        sd.nb_stride = P.nb_stride;
                        bp.dmin = sd.dmin; bp.nb_stride = sd.nb_stride;
                    }
                }
                launch_seed_mfma(ix->dtype, sd, (int)P.tiles.size(), s);
                if (ix->dtype == VF_F32) {
                    bp.seed_approx = 1; bp.err_bound = ix->seed_err_bound(); bp.xn_max = ix->xn_max; bp.q_max = 3.0e38f;
                    bp.seed_keep = std::min(64, P.itopk + tune.seed_margin);
                    if (sd.seed_f16) {
                        // its wider margin: more approximations are kept for re-ranking under a predicate (a failed proof
                        // costs the query a gather of every seed)
                        half_bound(ix, seed_delta, bp);
                        if (may_allocate) bp.fallback_count = ix->d_fb_count.as<uint32_t>();
                        bp.seed_keep = std::min(64, P.itopk + std::max(tune.seed_margin_bf16, tune.seed_margin));
                    }
                }
            } else {
                // (an even number of them: with 63 chunks a tile instead of 64 the tiles of a label meet another XCD's L2 at each chunk;
                // 1,200 queries x 1,000 seeds x 128 float32 27.8 instead of 26.1 us, AND pairs 27.8 instead of 25.0)
                sd.max_chunks = P.ns_stride / kSeedChunk;
                launch_seed_dist(ix->dtype, sd, (int)P.tiles.size(), s);
            }
            bp.dseed = sd.dseed;
            if (r.any_and && sc != nullptr && sc->ok) { bp.seed_map = sc->map.as<int32_t>(); bp.seed_goff = sc->goff.as<int64_t>(); }
            if (prof && ix->prof_exact_counts && r.any_and) bp.seed_pass = ix->counters.as<int32_t>() + (size_t)P.nq * 5;   // filled before the timed interval
        }
        if (prof && !attach) VF_HIP(hipEventRecord(ix->prof_ev[3], s));
        return VF_OK;
    };
    auto run_scan = [&]() -> int {
        if (forked) {
            // (while profiling the event that marks the start of the graph path serves as the fork event: every
            // event recorded on the caller's stream delays the kernel behind it by a few microseconds)
            hipEvent_t fork = prof ? ix->prof_ev[2] : ev_fork;
            VF_HIP(hipEventRecord(fork, s));
            VF_HIP(hipStreamWaitEvent(side, fork, 0));
            ss = side;
        }
        if (prof) VF_HIP(hipEventRecord(ix->prof_ev[0], ss));

        ScanParams sp{};
        sp.qsrc = queries; sp.qrow = (const int32_t *)(dp + L.off_qrow);
        sp.dim = ix->dim; sp.ncp = ix->ncp; sp.K = k; sp.tile_rows = ib.tile_rows;
        sp.out_ids = out_ids; sp.out_dists = out_dists;
        sp.res_idx = M.part_idx; sp.res_bits = M.part_bits;
        const MergeItem *d_merges = (const MergeItem *)(dp + L.off_merges);
        sp.others_off = d_others_off; sp.others = d_others; sp.meta = ix->meta();
        if (P.n_ls_items) {
            sp.xblk = ix->d_X_LS.as<uint4>(); sp.xnorm = ix->d_xnorm_LS.p; sp.map = ix->d_M_LS.as<int32_t>();
            sp.items = (const ScanItem *)(dp + L.off_items);
            // small batches are latency-bound: the FMA kernel finishes a one-query tile three times sooner;
            // large batches keep the matrix-core kernel, which leaves the vector ALU to the beam search
            const bool small_batch = tune.scan_valu == 2 || (tune.scan_valu == 1 && ib.qrow.size() <= 256);
            if (P.scan_bf16) {
                // filter from the bfloat16 copy, then re-rank (a query whose result is not proven complete is
                // scanned exactly by its re-ranking wave)
                ScanParams sb = sp;
                sb.xblk = ix->d_X_LS16.as<uint4>(); sb.K = P.scan_keep;
                launch_scan_bf16(sb, (int)P.n_ls_items, tune.scan_bf16_slots, ss);
                if (prof) ix->prof.scan_kernel = 3;
                if (prof && !exact) VF_HIP(hipEventRecord(ix->prof_ev[1], ss));
                RerankParams rp{};
                rp.items = d_merges; rp.res_idx = sp.res_idx; rp.res_bits = sp.res_bits; rp.map = sp.map;
                rp.X = ix->X; rp.Q = queries; rp.dim = ix->dim; rp.Kc = P.scan_keep; rp.K = k;
                // two bfloat16 products per component into a float32 accumulator, norms of the unrounded vectors, the lists'
                // own largest norm and rounding error
                rp.err_bound = ix->seed_err_bound() * 8.0f; rp.xn_max = ix->ls_xn_max; rp.err_q = 2.0f * ix->ls_bf16_delta;
                rp.approx_unit = 1.f; rp.q_max = 3.0e38f;
                rp.fail_count = ix->d_scan_fb.as<uint32_t>();
                rp.others_off = sp.others_off; rp.others = sp.others; rp.meta = sp.meta;
                rp.refused = M.refused; rp.refused_any = M.refused_any; rp.refused_count = ix->d_scan_fb.as<int32_t>() + 1;
                rp.out_ids = out_ids; rp.out_dists = out_dists;
                launch_scan_rerank(rp, (int)P.n_ls_merges, ss);
            } else if (small_batch && scan_valu_supported(ix->dtype, ix->dim, sp.tile_rows)) {
                launch_scan_valu(sp, (int)P.n_ls_items, ss);
                if (prof) ix->prof.scan_kernel = 2;
            } else if (tune.scan16 && scan16_supported(ix->dtype, ix->dim, sp.tile_rows)) {
                launch_scan16(sp, (int)P.n_ls_items, ss);
                if (prof) ix->prof.scan_kernel = 1;
            } else {
                launch_scan(ix->dtype, sp, (int)P.n_ls_items, ss);
            }
            // a search times its scan kernel by itself (the merge of the segments' candidates follows it)
            if (!P.scan_bf16) {
                if (prof && !exact) VF_HIP(hipEventRecord(ix->prof_ev[1], ss));
                launch_scan_merge(ix->dtype, d_merges, (int)P.n_ls_merges, sp.res_idx, sp.res_bits, k, ib.max_nseg * k,
                                  ix->d_M_LS.as<int32_t>(), out_ids, out_dists, ss);
            }
        }
        if (!P.jbatches.empty()) {
            JoinParams jp{};   // (ix->tmp_blk, tmp_norm: reserved with the plan)
            const int kind = P.join_kind;
            const float scale = ix->join_scale(kind);
            jp.xblk = ix->tmp_blk.as<uint4>(); jp.xnorm = ix->tmp_norm.p; jp.map = ix->d_M_HS.as<int32_t>();
            jp.qsrc = queries; jp.qrow = sp.qrow; jp.dim = ix->dim; jp.K = P.join_keep; jp.centre = ix->d_centre.as<float>(); jp.scale = scale;
            jp.res_idx = M.part_idx + P.ls_part_words; jp.res_bits = M.part_bits + P.ls_part_words;
            uint32_t *bound = M.part_bits + P.join_bound_at;
            jp.bound = bound; jp.bound_row0 = (int32_t)P.join_first_row;
            jp.others_off = d_others_off; jp.others = d_others; jp.meta = sp.meta;
            for (const JoinBatch &b : P.jbatches) {
                launch_join_pack(kind, ix->X, ix->dim, jp.map, (const JoinList *)(dp + L.off_jlists) + b.list_lo,
                                 (int)(b.list_hi - b.list_lo), b.groups, ix->join_norms(), ix->d_centre.as<float>(), scale, ix->tmp_blk.as<uint4>(),
                                 ix->tmp_norm.p, bound, (int64_t)P.join_rows, s);
                jp.items = (const ScanItem *)(dp + L.off_items) + P.n_ls_items + b.item_lo;
                launch_join(kind, jp, P.join_tile, (int)(b.item_hi - b.item_lo), s);
            }
            const int n_merges = (int)(ib.merges.size() - P.n_ls_merges);
            if (ix->dtype == VF_U8) {
                launch_scan_merge(ix->dtype, d_merges + P.n_ls_merges, n_merges, jp.res_idx, jp.res_bits, k, P.join_max_nseg * k,
                                  jp.map, out_ids, out_dists, s);
            } else {
                RerankParams rp{};
                rp.items = d_merges + P.n_ls_merges; rp.res_idx = jp.res_idx; rp.res_bits = jp.res_bits; rp.map = jp.map;
                rp.X = ix->X; rp.Q = queries; rp.dim = ix->dim; rp.Kc = P.join_keep; rp.K = k;
                rp.err_bound = ix->join_err_bound(kind); rp.xn_max = ix->xc_max; rp.err_q = ix->join_err_q(kind, false); rp.centre = jp.centre;
                // (a component beyond binary16 is infinite, and a query with one has no candidates)
                rp.approx_unit = 1.0f / (scale * scale); rp.q_max = kind == kJoinSingle ? 1.0e9f * rp.approx_unit : 3.0e38f;
                rp.fail_count = ix->d_scan_fb.as<uint32_t>();
                rp.others_off = sp.others_off; rp.others = sp.others; rp.meta = sp.meta;
                rp.refused = M.refused; rp.refused_any = M.refused_any; rp.refused_count = ix->d_scan_fb.as<int32_t>() + 1;
                rp.refused_first = (int32_t)P.n_ls_merges;
                rp.out_ids = out_ids; rp.out_dists = out_dists;
                launch_scan_rerank(rp, n_merges, s);
            }
        }
        if (!P.hs_runs.empty()) {
            const int64_t max_groups = (P.max_hs_list + 31) / 32;
            if ((rc = ix->tmp_blk.reserve((size_t)max_groups * ix->group_bytes())) != VF_OK) return rc;
            if ((rc = ix->tmp_norm.reserve((size_t)max_groups * 32 * 4)) != VF_OK) return rc;
            for (const HsRun &run : P.hs_runs) {
                const int32_t nl = ix->S[(size_t)run.label];
                launch_interleave(ix->dtype, ix->X, ix->dim, ix->d_M_HS.as<int32_t>() + ix->O_HS[(size_t)run.label], nullptr,
                                  nullptr, nl, (nl + 31) / 32, ix->ncp, ix->tmp_blk.as<uint4>(), ix->tmp_norm.p, s);
                sp.xblk = ix->tmp_blk.as<uint4>(); sp.xnorm = ix->tmp_norm.p; sp.map = ix->d_M_HS.as<int32_t>();
                sp.items = (const ScanItem *)(dp + L.off_items) + run.item_lo;
                launch_scan(ix->dtype, sp, (int)(run.item_hi - run.item_lo), s);
            }
            launch_scan_merge(ix->dtype, d_merges + P.n_ls_merges, (int)(ib.merges.size() - P.n_ls_merges), sp.res_idx,
                              sp.res_bits, k, ib.max_nseg * k, ix->d_M_HS.as<int32_t>(), out_ids, out_dists, s);
        }
        if (prof && (exact || !P.n_ls_items)) VF_HIP(hipEventRecord(ix->prof_ev[1], ss));
        if (forked) VF_HIP(hipEventRecord(ev_join, ss));
        return VF_OK;
    };
    // the scan goes first: its longest work items decide when it ends (measured: forking it
    // after the seed kernel costs 6 to 20 % of the step)
    count_passing_seeds();
    if ((rc = run_scan()) != VF_OK) return rc;
    if ((rc = run_seeds()) != VF_OK) return rc;
    if (n_gq) launch_beam(ix->dtype, bp, (int)n_gq, s, attach ? ix->prof_ev[3] : nullptr, attach ? ix->prof_ev[4] : nullptr);
    if (P.n_xq) {
        // the exact route of short AND queries: the beam kernel with every member of the list as a seed, no
        // iteration and a list of k entries -- each member is tested with the predicate, the members that pass
        // are gathered and scored, the k best stay
        BeamParams bx = bp;
        bx.gq_query = (const int32_t *)(dp + L.off_xq_query);
        bx.gq_label = (const int32_t *)(dp + L.off_xq_label);
        bx.n_seeds = 0x7FFFFFFF; bx.iters = 0; bx.itopk = k; bx.LP = 128; bx.hash_bits = 9;
        bx.dseed = nullptr; bx.dmin = nullptr; bx.seed_runs = nullptr; bx.seed_pass = nullptr; bx.seed_approx = 0; bx.fallback_count = nullptr;
        launch_beam(ix->dtype, bx, (int)P.n_xq, s);
    }
    if (bp.fallback_count != nullptr) {
        ix->fb_window_q += (int64_t)n_gq;
        // (a first look after 4,096 queries, for the calls that have another way: a failed proof is 1 to 10 times such a query's time)
        const bool first = !ix->fb_looked && tune.seed_fb_window > kFirstLook;
        if (!ix->fb_pending && ix->fb_window_q >= (first ? kFirstLook : tune.seed_fb_window)) {
            ix->fb_looked = true;
            ix->fb_first = first;
            VF_HIP(hipMemcpyAsync(ix->h_fb, bp.fallback_count, 4, hipMemcpyDeviceToHost, s));
            VF_HIP(hipEventRecord(ix->ev_fb, s));
            ix->fb_pending = true;
            ix->fb_sent_q = ix->fb_window_q;
            ix->fb_window_q = 0;
        }
    }
    if (prof) {
        if (!attach) VF_HIP(hipEventRecord(ix->prof_ev[4], s));
        ix->prof_valid = true;
        ix->prof_next = (ix->prof_next + 1) % vf_index::kProfRing;
        ++ix->prof_unfolded;
    }
    if (forked) VF_HIP(hipStreamWaitEvent(s, ev_join, 0));
    return VF_OK;
}

// Ground truth of the queries whose filtered result was refused a proof (RerankParams::refused): by the ordered distance,
// kOrderedRows of a list at a time, every list cut into as many segments as keep the chip busy.  (One wave per query, in
// the re-ranking kernel, takes as long as the longest list: 400,000 x 128 float32, one query with a NaN made a batch of
// 4,000 take 21.6 instead of 2.2 ms, now 2.5; a table whose clusters lie so far apart that 2,245 of them are refused 21.0,
// now 6.5.)  The stream is idle; waits for the results.
static int answer_refused(vf_index *ix, const CallPlan &P, const Routed &r, const CallMem &M, const void *queries, int64_t *out_ids,
                          float *out_dists, hipStream_t s)
{
    int32_t n_refused = 0;
    VF_HIP(hipMemcpy(&n_refused, ix->d_scan_fb.as<int32_t>() + 1, 4, hipMemcpyDeviceToHost));
    std::vector<int32_t> which((size_t)n_refused);
    VF_HIP(hipMemcpy(which.data(), M.refused, which.size() * 4, hipMemcpyDeviceToHost));
    std::sort(which.begin(), which.end());   // queries of a list become neighbours, scan lists come first
    const std::vector<MergeItem> &merges = P.ib.merges;
    constexpr size_t kBatch = 4096;          // bounds the partial rows: 64 segments of 64 results each
    DevBuf d_items(&ix->alloc), d_merges(&ix->alloc), d_qrow(&ix->alloc), parts(&ix->alloc);
    DevBufGuard guard{&d_items, &d_merges, &d_qrow, &parts};
    int rc;
    for (size_t lo = 0; lo < which.size();) {
        const bool ls = (size_t)which[lo] < P.n_ls_merges;
        size_t hi = lo;
        while (hi < which.size() && hi - lo < kBatch && ((size_t)which[hi] < P.n_ls_merges) == ls) ++hi;
        ItemBuilder ib(ix->tune);
        ib.tile_rows = kOrderedRows;
        ib.all_partial = true;
        std::vector<uint64_t> rows;          // (queries of one list)
        auto list_end = [&](size_t i) {
            size_t e = i;
            while (e < hi && merges[(size_t)which[e]].map_off == merges[(size_t)which[i]].map_off) ++e;
            return e;
        };
        int64_t tile_groups = 0;
        for (size_t i = lo, e; i < hi; i = e) {
            e = list_end(i);
            tile_groups += (int64_t)((e - i + kOrderedRows - 1) / kOrderedRows) * ((merges[(size_t)which[i]].n + 31) / 32);
        }
        ib.seg_groups = ib.seg_groups_heavy = (int)std::max<int64_t>(8, tile_groups / 4096);
        for (size_t i = lo, e; i < hi; i = e) {
            e = list_end(i);
            rows.clear();
            for (size_t u = i; u < e; ++u) rows.push_back((uint64_t)(uint32_t)merges[(size_t)which[u]].qrow);
            ib.add_label(rows, 0, rows.size(), 0, merges[(size_t)which[i]].map_off, merges[(size_t)which[i]].n);
        }
        const size_t words = (size_t)ib.part_rows * P.k;
        if ((rc = parts.reserve(words * 8)) != VF_OK) return rc;
        if ((rc = upload(d_items, ib.items, s)) != VF_OK || (rc = upload(d_merges, ib.merges, s)) != VF_OK ||
            (rc = upload(d_qrow, ib.qrow, s)) != VF_OK)
            return rc;
        OrderedScanParams p{};
        p.X = ix->X; p.Q = queries; p.map = ls ? ix->d_M_LS.as<int32_t>() : ix->d_M_HS.as<int32_t>();
        p.items = d_items.as<ScanItem>(); p.qrow = d_qrow.as<int32_t>();
        p.dim = ix->dim; p.K = P.k;
        p.res_idx = parts.as<int32_t>(); p.res_bits = parts.as<uint32_t>() + words;
        if (r.any_and) {
            p.others_off = (const int32_t *)(M.blob + P.L.off_others_off);
            p.others = (const int32_t *)(M.blob + P.L.off_others);
        }
        p.meta = ix->meta();
        launch_ordered_scan(p, (int)ib.items.size(), s);
        launch_scan_merge(ix->dtype, d_merges.as<MergeItem>(), (int)ib.merges.size(), p.res_idx, p.res_bits, P.k, ib.max_nseg * P.k,
                          p.map, out_ids, out_dists, s);
        VF_HIP(hipGetLastError());
        VF_HIP(hipStreamSynchronize(s));     // the tables are pageable host memory, the next batch takes the same buffers
        lo = hi;
    }
    return VF_OK;
}

// first_is_searched: every query searches the list of its first label (the others are the
// predicate) instead of its smallest list -- the sub-searches of vf_search_multi.
int search_impl(vf_index *ix, const void *queries, int64_t nq, const int64_t *qoff, const int32_t *qids, int32_t k,
                int32_t itopk, int32_t width, int32_t iters, int32_t n_seeds, bool exact, int64_t *out_ids,
                float *out_dists, hipStream_t s, bool first_is_searched, int32_t and_scan_limit, const MultiCall *multi)
{
    int rc = check_search_args(ix, queries, nq, k, out_ids, out_dists);
    if (rc != VF_OK) return rc;
    std::lock_guard<std::recursive_mutex> lock(ix->mu);
    const auto t_enter = std::chrono::steady_clock::now();
    if ((rc = check_search_params(ix, exact, k, itopk, width, iters, n_seeds)) != VF_OK) return rc;
    Workspace *W = nullptr;
    if ((rc = workspace_for(ix, s, &W)) != VF_OK) return rc;
    if (nq == 0) return VF_OK;
    const Tuning &tune = ix->tune;
    // the seed distance matrix reuses what is allocated, or grows into at most half of the free memory
    SeedBudget budget;
    budget.words = W->dseed.cap / 4;
    budget.grows = true;
    budget.cap = W->dseed.cap;
    // the interleaved copy of the seeds for this seed count (made by the plan of the first call that uses it), after a look
    // at the watch on failed float32 proofs
    SeedCopy *sc = nullptr;
    if (wants_seed_copy(ix, exact, itopk, n_seeds)) {
        if (ix->fb_pending && hipEventQuery(ix->ev_fb) == hipSuccess) {
            const uint32_t now = *ix->h_fb, failed = now - ix->fb_last;
            ix->fb_last = now;
            ix->fb_pending = false;
            if ((int64_t)failed * 64 > ix->fb_sent_q) {
                ix->seed_proofs_off = true;
                if (!ix->fb_first && seed_mfma_own(ix->dtype, ix->dim)) {
                    ix->seed_bf16_off = true;   // the copies are rebuilt in float32
                    if ((rc = drop_seed_copies(ix)) != VF_OK) return rc;
                }
            }
        } else if (ix->fb_pending) {
            (void)hipGetLastError();      // "not ready" is no error
        }
        if ((rc = seed_copy_for(ix, n_seeds, s, false, &sc)) != VF_OK) return rc;
    }
    CallPlan P(tune);
    struct Lend {
        CallPlan &P;
        PlanStore &store;
        Lend(CallPlan &p, PlanStore &s) : P(p), store(s) { store.clear(); store.swap_with(P); }
        ~Lend() { store.swap_with(P); }
    } lend(P, W->plan);
    Routed &r = W->routed;
    VF_REQUIRE(and_scan_limit >= 0, "and_scan_limit must be >= 0");
    const SeedCopyMaker make{ix, s};
    auto plan = [&] {
        return plan_call(ix, r, nq, qoff, qids, exact, first_is_searched, k, itopk, width, iters, n_seeds, and_scan_limit, budget, &make, sc, P);
    };
    if ((rc = plan()) != VF_OK) return rc;
    auto words_up = [](size_t v) { return (v + 63) & ~(size_t)63; };
    // Ground truth over joined lists: the packed lists and partial rows before anything is sent.  Where there is no memory
    // for them: smaller batches of lists, down to single ones, and then the scan kernels, whose copies of a list are smaller.
    while (!P.jbatches.empty()) {
        if ((rc = ix->tmp_blk.reserve((size_t)P.join_groups * join_group_bytes(ix->join_kind_max(), ix->dim))) == VF_OK &&
            (rc = ix->tmp_norm.reserve((size_t)P.join_groups * 32 * 4)) == VF_OK &&
            (rc = W->dseed.reserve((2 * words_up(P.part_words) + words_up(P.ib.merges.size())) * 4)) == VF_OK)
            break;
        if (rc != VF_ENOMEM) return rc;
        (void)hipGetLastError();
        ix->tmp_blk.release();
        ix->tmp_norm.release();
        const bool one_each = P.jbatches.size() == P.jlists.size();
        const size_t bytes = one_each ? 0 : P.join_bytes / 4;
        P = CallPlan(tune);
        P.join_bytes = bytes;
        if ((rc = plan()) != VF_OK) return rc;
    }
    if (multi != nullptr) {   // (a copy of its own would wait for the caller's stream: the vectors are pageable memory)
        P.L.off_multi = P.L.total;
        P.L.total = align_up(P.L.total + multi->host->size() * 4);
    }
    const BlobLayout &L = P.L;
    const auto t_planned = std::chrono::steady_clock::now();
    Staging *st = nullptr;
    // (ground truth: behind the blob is the word that says whether there are refused queries)
    const size_t flag_at = (L.total + 63) & ~(size_t)63;
    if ((rc = get_staging(W, flag_at + 64, &st)) != VF_OK) return rc;
    const auto t_staged = std::chrono::steady_clock::now();   // (waiting for the staging buffer is the GPU's time, not the host's)
    char *hp = (char *)st->p;
    fill_blob(P, r, hp);
    if (multi != nullptr) memcpy(hp + L.off_multi, multi->host->data(), multi->host->size() * 4);
    const auto t_blob = std::chrono::steady_clock::now();
    // seed distances and partial rows in one buffer: one allocation where a workspace meets its first call
    const size_t dseed_words = P.dense_seeds ? words_up(P.dseed_words) : 0, part_words = words_up(P.part_words);
    const size_t refused_words = exact && (P.scan_bf16 || (!P.jbatches.empty() && ix->dtype == VF_F32)) ? words_up(P.ib.merges.size()) : 0;
    if (dseed_words + part_words > 0 && (rc = W->dseed.reserve((dseed_words + 2 * part_words + refused_words) * 4)) != VF_OK) return rc;
    // The scan path runs on the side stream beside the graph path on the caller's stream.
    const bool forked = tune.overlap && !ix->prof_serial && !exact && P.n_gq > 0 && !P.ib.items.empty();
    // Two device blobs alternate.  When the call forks, its blob is uploaded on the side stream: there it
    // follows the previous call's scan, not the previous call's beam search, so the upload is off the
    // critical path.  The buffer was last read two calls ago, by kernels on the side stream (which precede the
    // upload there) and on the caller's stream: those precede the fork event of the previous call, which the
    // side stream has waited for -- if that call forked; if not, and where the buffer is new, the upload first waits for
    // the caller's stream.
    // A small blob (small batches) is not copied at all: the kernels read the few hundred bytes they need
    // straight from the pinned staging buffer, which saves the copy's submission and its latency; the
    // staging buffer then stays untouched until the call's last kernel has ended.
    const bool zero_copy = tune.zero_copy_bytes > 0 && L.total <= (size_t)tune.zero_copy_bytes;
    const int bsel = W->blob_next;
    DevBuf &blob = bsel ? W->ws_blob_b : W->ws_blob;
    CallMem M;
    if (zero_copy) {
        void *dev_view = nullptr;
        VF_HIP(hipHostGetDevicePointer(&dev_view, st->p, 0));
        M.blob = (char *)dev_view;
    } else {
        W->blob_next ^= 1;
        // (a buffer that is allocated now may, with an allocator that works in stream order, still be in use by work that
        // the caller has queued on its stream: another index's outputs, say)
        const bool fresh = L.total > blob.cap;
        if ((rc = blob.reserve(L.total)) != VF_OK) return rc;
        M.blob = blob.as<char>();
        hipStream_t cs = forked ? W->side : s;
        if (forked && (!W->prev_forked || fresh)) {
            VF_HIP(hipEventRecord(W->ev_fork, s));
            VF_HIP(hipStreamWaitEvent(cs, W->ev_fork, 0));
        }
        VF_HIP(hipMemcpyAsync(M.blob, hp, L.total, hipMemcpyHostToDevice, cs));
        VF_HIP(hipEventRecord(st->done, cs));
        st->pending = true;
        if (forked) VF_HIP(hipStreamWaitEvent(s, st->done, 0));
    }
    W->prev_forked = forked;
    M.dseed = W->dseed.as<uint32_t>();
    M.part_idx = W->dseed.as<int32_t>() + dseed_words;
    M.part_bits = W->dseed.as<uint32_t>() + dseed_words + part_words;
    if (refused_words > 0) {
        M.refused = W->dseed.as<int32_t>() + dseed_words + 2 * part_words;
        void *dev_view = nullptr;
        VF_HIP(hipHostGetDevicePointer(&dev_view, st->p, 0));
        M.refused_any = (uint32_t *)((char *)dev_view + flag_at);
        memset(hp + flag_at, 0, 4);
        if (ix->refused_unread) VF_HIP(hipMemsetAsync(ix->d_scan_fb.as<uint32_t>() + 1, 0, 4, s));
        ix->refused_unread = true;
    }
    if (multi != nullptr)
        launch_gather_rows(multi->rows, (int32_t)((size_t)ix->dim * ix->elem()), (const int32_t *)(M.blob + L.off_multi), nq, W->multi_q.p, s);
    if ((rc = launch_call(ix, P, r, M, sc, queries, out_ids, out_dists, s, forked ? W->side : nullptr, W->ev_fork,
                          W->ev_join, true)) != VF_OK)
        return rc;
    auto merge_multi = [&] {
        launch_multi_merge((const int32_t *)(M.blob + L.off_multi) + nq, multi->nq, out_ids, out_dists, k, multi->out_ids, multi->out_dists, s);
    };
    if (multi != nullptr && !exact) merge_multi();
    // (nothing reads the blob after this; ground truth still does)
    if (zero_copy && !exact) {
        VF_HIP(hipEventRecord(st->done, s));
        st->pending = true;
    }
    VF_HIP(hipGetLastError());
    if (ix->profiling) {
        const auto t_end = std::chrono::steady_clock::now();
        auto ms = [](auto a, auto b) { return std::chrono::duration<double, std::milli>(b - a).count(); };
        ix->prof_host_plan += ms(t_enter, t_planned);
        ix->prof_host_wait += ms(t_planned, t_staged);
        ix->prof_host_blob += ms(t_staged, t_blob);
        ix->prof_host_launch += ms(t_blob, t_end);
    }
    if (exact) {
        VF_HIP(hipStreamSynchronize(s));
        ix->tmp_blk.release();
        ix->tmp_norm.release();
        uint32_t any = 0;
        if (M.refused != nullptr) memcpy(&any, hp + flag_at, 4);
        if (any != 0 && (rc = answer_refused(ix, P, r, M, queries, out_ids, out_dists, s)) != VF_OK) return rc;
        if (any == 0) ix->refused_unread = false;
        if (multi != nullptr) {
            merge_multi();
            VF_HIP(hipGetLastError());
            if (zero_copy) {
                VF_HIP(hipEventRecord(st->done, s));
                st->pending = true;
            }
        }
    }
    return VF_OK;
}

// OR queries (Section 4.3.1) and the parallel AND policy (end of Section 4.3.2): every query becomes
// one search per label, the searches run as one ordinary batch, and a merge kernel combines them.
int search_multi_impl(vf_index *ix, const void *queries, int64_t nq, const int64_t *qoff, const int32_t *qids, int32_t mode,
                      int32_t k, int32_t itopk, int32_t width, int32_t iters, int32_t n_seeds, int64_t *out_ids,
                      float *out_dists, hipStream_t s)
{
    const bool exact = (mode & VF_MULTI_EXACT) != 0;
    mode &= ~VF_MULTI_EXACT;
    VF_REQUIRE(mode == VF_AND_GREEDY || mode == VF_AND_PARALLEL || mode == VF_OR, "mode must be VF_AND_GREEDY, VF_AND_PARALLEL or VF_OR");
    if (mode == VF_AND_GREEDY)
        return search_impl(ix, queries, nq, qoff, qids, k, itopk, width, iters, n_seeds, exact, out_ids, out_dists, s, false);
    int rc = check_search_args(ix, queries, nq, k, out_ids, out_dists);
    if (rc != VF_OK) return rc;
    VF_REQUIRE(qoff && qids, "NULL query label arrays");
    if (nq == 0) return VF_OK;
    std::lock_guard<std::recursive_mutex> lock(ix->mu);
    Workspace *W = nullptr;
    if ((rc = workspace_for(ix, s, &W)) != VF_OK) return rc;
    {
        std::vector<int32_t> &host = W->multi_host;
        std::vector<int64_t> &sqoff = W->multi_qoff;
        std::vector<int32_t> &sqids = W->multi_qids;
        std::vector<int32_t> &first = W->multi_first;
        host.clear(); sqoff.assign(1, 0); sqids.clear();
        first.resize((size_t)nq + 1);
        first[0] = 0;
        int32_t labs[kMaxOthers + 1];
        for (int64_t j = 0; j < nq; ++j) {
            const int64_t b = qoff[j], e = qoff[j + 1];
            VF_REQUIRE(e > b, "every query needs at least one label");
            if (mode == VF_OR && e - b <= 2) {   // the common case as a straight line: a search for every label with a list
                const int32_t l0 = qids[b], l1 = qids[e - 1];
                VF_REQUIRE((uint32_t)l0 < (uint32_t)ix->n_labels && (uint32_t)l1 < (uint32_t)ix->n_labels, "query label outside [0, n_labels)");
                const size_t at = host.size(), one = ix->S[(size_t)l0] > 0, two = (l0 != l1) & (ix->S[(size_t)l1] > 0);
                host.resize(at + one + two, (int32_t)j);
                sqids.resize(at + one + two, l1);
                if (one) sqids[at] = l0;
                first[(size_t)j + 1] = (int32_t)host.size();
                continue;
            }
            int32_t nl = 0;
            for (int64_t p = b; p < e; ++p) {
                const int32_t l = qids[p];
                VF_REQUIRE(l >= 0 && l < ix->n_labels, "query label outside [0, n_labels)");
                bool seen = false;
                for (int32_t i = 0; i < nl; ++i) seen = seen || labs[i] == l;
                if (seen) continue;
                VF_REQUIRE(nl <= kMaxOthers, "more than 8 distinct labels in one query");
                labs[nl++] = l;
            }
            auto add = [&](int32_t searched, bool with_others) {
                host.push_back((int32_t)j);
                sqids.push_back(searched);
                if (with_others)
                    for (int32_t i = 0; i < nl; ++i)
                        if (labs[i] != searched) sqids.push_back(labs[i]);
                if (mode != VF_OR) sqoff.push_back((int64_t)sqids.size());
            };
            if (mode == VF_OR) {
                for (int32_t i = 0; i < nl; ++i)
                    if (ix->S[(size_t)labs[i]] > 0) add(labs[i], false);
            } else {
                int32_t best = labs[0];
                bool empty = false;
                for (int32_t i = 0; i < nl; ++i) {
                    const int32_t sl = ix->S[(size_t)labs[i]], sb = ix->S[(size_t)best];
                    if (sl == 0) empty = true;
                    if (sl < sb || (sl == sb && labs[i] < best)) best = labs[i];
                }
                if (!empty) {
                    if (ix->S[(size_t)best] < ix->T) add(best, true);   // the filtered scan of the smallest list is exact
                    else for (int32_t i = 0; i < nl; ++i) add(labs[i], true);
                }
            }
            first[(size_t)j + 1] = (int32_t)host.size();
        }
        const int64_t n_sub = (int64_t)host.size();
        if (mode == VF_OR) {   // (one label each)
            sqoff.resize((size_t)n_sub + 1);
            std::iota(sqoff.begin(), sqoff.end(), (int64_t)0);
        }
        if (n_sub == 0) {
            launch_fill_out(out_ids, out_dists, nq * (int64_t)k, s);
            VF_HIP(hipGetLastError());
            return VF_OK;
        }
        host.insert(host.end(), first.begin(), first.end());
        const size_t row_bytes = (size_t)ix->dim * ix->elem();
        if ((rc = W->multi_q.reserve((size_t)n_sub * row_bytes)) != VF_OK) return rc;
        if ((rc = W->multi_ids.reserve((size_t)n_sub * k * 8)) != VF_OK) return rc;
        if ((rc = W->multi_dists.reserve((size_t)n_sub * k * 4)) != VF_OK) return rc;
        const MultiCall multi{&host, queries, nq, out_ids, out_dists};
        return search_impl(ix, W->multi_q.p, n_sub, sqoff.data(), sqids.data(), k, itopk, width, iters, n_seeds, exact,
                           W->multi_ids.as<int64_t>(), W->multi_dists.as<float>(), s, true, 0, &multi);
    }
}

}  // namespace vf
