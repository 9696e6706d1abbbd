// Queue-driven serving of small batches (Section 4.2.3): one kernel stays resident for a whole session and pulls
// single queries from a job queue, so a query costs neither a kernel launch nor a host-side synchronisation.
//
// Shape on this machine.  The host writes a job (query vector + labels) into a ring in pinned host memory and
// bumps a counter.  Workgroup 0 of the resident kernel is the DISPATCHER: it alone polls that counter across
// PCIe and publishes a job by writing its number into the ready word of the job's slot in device memory.  The
// other workgroups are WORKERS (one query at a time, as in the paper's one block per query; NW waves each: all of
// them score a share of the query's seeds, or scan a share of its list, then the first wave searches or merges while
// the others wait at the workgroup's barrier): a free worker draws the next job number with one atomic addition --
// the atomic ring buffer of the paper's figure -- and waits for that job's ready word; it copies the job from the
// host's ring itself, routes it (smallest list, graph or scan by T, Section 4.1.2 / 4.3.2), runs the same beam search
// or list scan the batched kernels run (the device functions are shared), writes the k results straight into the
// result ring in host memory and releases a per-job done flag there.
//
// What bounds a session is the latency of one search, times what the places in flight allow.  While free workers compared
// and swapped one common head word and the dispatcher copied one job after the other (a PCIe round trip each, two more
// for the counter and the stop word), a job cost about 5 us however many workers there were.  Now free workers wait at as
// many words as there are slots, the dispatcher's poll is one round trip for any number of jobs, and the copies of different jobs
// overlap.  300,000 x 128 float32, 6,144 seeds, width 2, 12 iterations, queries/s with 1 / 8 / 64 / 240 in flight: 8.7 k /
// 56 k / 185 k / 191 k before, 12.9 k / 100 k / 757 k / 2.24 M now; p50 of a query 146 / 174 / 311 / 1,192 us before, 103 /
// 104 / 108 / 127 now.  Of the 102 us of such a search 63 went by with the seeds and 38 with the search; with the seeds filtered
// in binary16 on the matrix cores and the search in the form for a wave that has its SIMD to itself, and what is derived from
// the lane's number kept out of the registers between jobs (464 -> 48 bytes spilled), 26 and 42, which the scoring of the
// filter's survivors is part of: 1 / 64 in flight 13.1 k / 788 k -> 19.2 k / 1.08 M queries/s.
//
// Every wave exits on its own.  The dispatcher leaves when the host asks it to, when max_jobs jobs have been
// published, or after idle_polls consecutive polls without a new job; leaving, it raises the device-side stop
// flag.  A worker leaves when it sees that flag and the job it has drawn is not among those published, and in any
// case once the dispatcher's heartbeat has stood still for a bounded number of its looks.  So a session that is
// never ended ends by itself, and vf_serve_end always returns.
#include <atomic>
#include <chrono>

#include "vf_beam.h"
#include "vf_host.h"
#include "vf_scan_item.h"

namespace vf {

constexpr int kServeHdr = 64;    // bytes of a job slot before the query vector
constexpr int kReadyBytes = 64;  // behind a device slot: its ready word, whose 128-byte line ends with the query or begins the next slot
constexpr int kServeQuickPolls = 64;   // the dispatcher's, after a job, with a short sleep between them
constexpr int kServeSleep = 16;  // s_sleep between a waiting worker's polls, 64 cycles each

struct ServeJobHdr {            // first kServeHdr bytes of a job slot (host ring and device ring)
    int32_t n_labels;
    int32_t labels[kMaxOthers + 1];
    int32_t pad[7];
};
static_assert(sizeof(ServeJobHdr) == kServeHdr, "job header size");

struct ServeResult {            // one slot of the result ring (pinned host memory)
    uint64_t done;              // job id + 1 once ids / dists of that job are complete
    int64_t ids[64];
    float dists[64];
};

struct ServeHostCtrl {          // pinned host memory, both sides read and write
    uint64_t tail;              // host: jobs submitted so far
    uint32_t stop;              // host: 1 = end the session (the dispatcher reads tail and stop with one instruction)
    uint32_t pad0;
    uint64_t jobs_done;         // device: jobs completed (written at exit)
    uint32_t exit_reason;       // device: 0 while running; 1 host asked, 2 max_jobs reached, 3 idle bound
    uint32_t pad1;
};

struct ServeDevCtrl {           // device memory; the workers' words and the dispatcher's apart
    uint64_t head;              // next job to draw
    uint64_t jobs_done;
    uint64_t pad0[14];
    uint64_t tail;              // jobs published
    uint64_t beat;              // the dispatcher's heartbeat
    uint32_t stop;
    uint32_t pad1;
};

struct ServeParams {
    BeamParams bp;              // static part: tables, dim, R, k, itopk, width, iters, n_seeds, LP, hash_bits
    ScanParams sp;              // static part: scan lists, norms, map, dim, ncp, K, tile_rows, meta
    const int64_t *GO_LS;       // [n_labels] first 32-vector group of a scan list
    int32_t T, n_labels;
    int32_t ring_slots, slot_stride, row_bytes;
    const char *host_ring;      // device view of the pinned job ring, slots of slot_stride bytes
    char *dev_ring;             // slots of slot_stride + kReadyBytes: the job, then its ready word (job + 1 once published)
    ServeResult *results;       // device view of the pinned result ring
    ServeHostCtrl *hctrl;       // device view
    ServeDevCtrl *dctrl;
    int64_t max_jobs, idle_polls;
    int32_t lds_kernels;        // bytes of LDS the search functions use; the worker's own words follow (lds_own bytes)
    int32_t lds_own;
    int32_t lds_scan;           // bytes of LDS the scan of one wave uses
    const uint4 *sblk16;        // optional: the seeds in binary16 (bp.scale), the filter of jobs without a predicate
    const float *snorm;         // with it: norms of the unrounded seeds
    int32_t s16_chunks;         // 16-byte chunks of a seed in it
    uint32_t *rows;             // a row of row_words words per worker: approximations, then the minima of their blocks of 32
    int32_t ns_stride, row_words;
    float minus_two_unscaled;
};

template <class T> __device__ __forceinline__ T load_sys(const T *p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM); }
template <class T> __device__ __forceinline__ T load_dev(const T *p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT); }
template <class T> __device__ __forceinline__ T look_dev(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ char *serve_slot(const ServeParams &p, uint64_t job)
{
    return p.dev_ring + (size_t)(job % (uint64_t)p.ring_slots) * (size_t)(p.slot_stride + kReadyBytes);
}
__device__ __forceinline__ uint64_t *serve_ready(const ServeParams &p, uint64_t job) { return (uint64_t *)(serve_slot(p, job) + p.slot_stride); }

// One lane: draws the next job and waits for it; -1: the session is over.  A worker that waits reads the ready word of its
// job's slot, which it shares with others only where there are fewer slots than workers, and every 16th time the dispatcher's
// words.
__device__ __forceinline__ int64_t serve_next_job(const ServeParams &p)
{
    const uint64_t job = __hip_atomic_fetch_add(&p.dctrl->head, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t *ready = serve_ready(p, job);
    // looks at an unchanged heartbeat (one in 16 polls, some 30 us) before a worker gives the dispatcher up; the
    // dispatcher beats at least once in 16 of its polls, so this is longer than its own idle bound, and never short
    const int64_t bound = 16 * p.idle_polls > 65536 ? 16 * p.idle_polls : 65536;
    uint64_t beat = 0;
    int64_t still = 0;
    for (uint32_t poll = 0;; ++poll) {
        if (look_dev(ready) == job + 1) return (int64_t)job;
        if ((poll & 15u) == 15u) {
            const uint32_t stop = load_dev(&p.dctrl->stop);
            if (stop != 0) {
                if (job >= look_dev(&p.dctrl->tail)) return -1;   // drained
                continue;                                         // published before the flag was raised: its word is there
            }
            const uint64_t b = look_dev(&p.dctrl->beat);
            still = b == beat ? still + 1 : 0;
            beat = b;
            if (still > bound) return -1;   // the dispatcher must be gone
        }
        __builtin_amdgcn_s_sleep(kServeSleep);
    }
}

// Approximate distances of seeds [j_lo, j_hi) (whole groups of 32 but for the list's end) from their binary16 copy, on the matrix
// cores, as seed_mfma_kernel computes them: the seeds are the rows of a 32x32 product, and every column is the one query.  STEPS:
// contraction steps (FIT = false: at most).  A worker's seeds come from far memory at the rate that what it keeps in flight
// allows, so the copy of half the bytes is read, AHEAD groups a wave in flight, and nothing waits for a group but its own product;
// groups past the last one are that one once more, so that no request or store is conditional.
// (One query, 6,144 seeds x 128, eight waves: 63 us scored in float32, 64 seeds a step, 26 us so, with 64 queries in flight.)
template <int STEPS, bool FIT>
__device__ __forceinline__ void seed_filter_segment(const ServeParams &p, int label, const uint4 *q16, float qn, int ns, int j_lo, int j_hi,
                                                    uint32_t *norms, uint32_t *row, uint32_t *mins, int lane)
{
    constexpr int AHEAD = STEPS <= 8 ? 4 : 1;
    const int n32 = lane & 31, h = lane >> 5;
    const int chunks = FIT ? 2 * STEPS : p.s16_chunks, steps = FIT ? STEPS : (chunks + 1) / 2;
    const int last = (j_hi - j_lo + 31) / 32 - 1;
    const int64_t g0 = p.bp.sgoff[p.bp.meta.hs_slot[label]] + j_lo / 32;
    const uint4 *const blk = p.sblk16 + g0 * (int64_t)(chunks * 32) + n32;
    const float *const xn_at = p.snorm + g0 * 32 + n32;
    uint4 q[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const bool in = 2 * s + h < chunks;
        q[s] = q16[in ? 2 * s + h : 0];
        if (!in) q[s] = make_uint4(0, 0, 0, 0);
    }
    uint4 b[AHEAD][STEPS];
    float xn[AHEAD];
    auto fetch = [&](int u, int g) {
        g = g < last ? g : last;
        const uint4 *src = blk + (int64_t)g * (chunks * 32);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) b[u][s] = src[(FIT || 2 * s + h < chunks ? 2 * s + h : chunks - 1) * 32];
        xn[u] = xn_at[(int64_t)g * 32];
    };
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) fetch(u, u);
    for (int base = 0; base <= last; base += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int g = base + u < last ? base + u : last, j0 = j_lo + g * 32;
            v16f_seed acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                if (FIT || s < steps)   // (wave-uniform)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h_seed, b[u][s]), __builtin_bit_cast(v8h_seed, q[s]), acc, 0, 0, 0);
            wave_sync<true>();          // (the last group's norms have been read)
            norms[n32] = j0 + n32 < ns ? __float_as_uint(xn[u]) : 0x7F800000u;
            fetch(u, base + u + AHEAD);
            wave_sync<true>();
            uint32_t m = 0xFFFFFFFFu;
            uint4 mine = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // seeds 8 i + 4 h + 0..3 of the group, in every lane of that half
                const uint4 n4 = *(const uint4 *)&norms[8 * i + 4 * h];
                const uint32_t nx[4] = {n4.x, n4.y, n4.z, n4.w};
                uint32_t bits[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    bits[w] = __float_as_uint(fmaxf(__builtin_fmaf(p.minus_two_unscaled, acc[4 * i + w], qn + __uint_as_float(nx[w])), 0.0f));
                    m = bits[w] < m ? bits[w] : m;
                }
                if (n32 == i) mine = make_uint4(bits[0], bits[1], bits[2], bits[3]);
            }
            const auto r = __builtin_amdgcn_permlane32_swap(m, m, false, false);
            if (n32 < 4) *(uint4 *)&row[j0 + 8 * n32 + 4 * h] = mine;
            if (lane == 0) mins[j0 / 32] = r[0] < r[1] ? r[0] : r[1];
        }
    }
}

// DT: 0 uint8, 1 float32.  NC: compile-time chunk count of the scan function (chunk pairs for scan_topk_item,
// chunks for scan_valu_item), 0 = generic.
template <int DT, int NC, int NW>
__global__ __launch_bounds__(64 * NW) void serve_kernel(ServeParams p)
{
    extern __shared__ uint4 smem[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;

    if (blockIdx.x == 0) {
        // ---------------- dispatcher (the first wave; it never meets a workgroup barrier)
        if (wv != 0) return;
        uint64_t published = 0, beat = 0;
        int64_t idle = -kServeQuickPolls;
        uint32_t reason = 0;
        while (reason == 0) {
            // lane 0 reads the counter, lane 1 the stop word: one trip across PCIe
            const uint64_t word = load_sys((const uint64_t *)p.hctrl + (lane & 1));
            const uint64_t t = readlane64(word, 0);
            const uint32_t stop = (uint32_t)readlane64(word, 1);
            const uint64_t upto = t < (uint64_t)p.max_jobs ? t : (uint64_t)p.max_jobs;
            if (upto > published) {   // at most ring_slots jobs: a slot is written again when its job is done
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                for (uint64_t j = published + lane; j < upto; j += 64)
                    __hip_atomic_store(serve_ready(p, j), j + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                published = upto;
                idle = -kServeQuickPolls;
            } else {
                // (quick polls are not counted: one that is counted takes about 4 us, whatever the bound)
                if (++idle > 0) __builtin_amdgcn_s_sleep(100);
                else __builtin_amdgcn_s_sleep(4);
            }
            if ((++beat & 15u) == 0 && lane == 0) __hip_atomic_store(&p.dctrl->beat, beat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (stop != 0) reason = 1;
            else if ((int64_t)published >= p.max_jobs) reason = 2;
            else if (idle > p.idle_polls) reason = 3;
        }
        if (lane == 0) __hip_atomic_store(&p.dctrl->tail, published, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();   // the ready words and the tail before the flag
        if (lane == 0) __hip_atomic_store(&p.dctrl->stop, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        // the session's exit record is complete once every published job is done: bounded wait for the workers
        // (counted from the last of them that was done: one worker may have a queue of jobs before it)
        uint64_t done = load_dev(&p.dctrl->jobs_done);
        for (int64_t spins = 0; done < published && spins < 16 * p.idle_polls + 1024; ++spins) {
            __builtin_amdgcn_s_sleep(32);
            const uint64_t now = load_dev(&p.dctrl->jobs_done);
            if (now != done) spins = 0;
            done = now;
        }
        if (lane == 0) {
            p.hctrl->jobs_done = load_dev(&p.dctrl->jobs_done);
            __hip_atomic_store(&p.hctrl->exit_reason, reason, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return;
    }

    // ---------------- worker
    // Every wave of the workgroup passes the same four barriers per job.  LDS: the search functions' area (first
    // wave; a scan: a part for each), then [0..7] others, [8..9] others_off, [10] qrow, [11..12] job, then per wave a
    // copy of the query and a run of 64 seed keys (a scan: 64 entries and 64 distances); until the job is routed its header
    // lies where the runs will be.
    int32_t *own = (int32_t *)((char *)smem + p.lds_kernels);
    char *share = (char *)smem + p.lds_kernels + p.lds_own;
    const int q_bytes = (p.row_bytes + 15) & ~15;
    uint4 *hq = (uint4 *)(share + (size_t)wv * q_bytes);                         // this wave's copy of the query
    uint64_t *runs = (uint64_t *)(share + (size_t)NW * q_bytes);                 // [NW][64]
    // own[16]: whether the seeds' binary16 copy is used; [20..23] the last search's counters.  A query whose proof fails (more than
    // 128 seeds within the bound) has its seeds scored by one wave: a worker that meets more than one in 16 does without.
    int met = 0, failed = 0;
    if (threadIdx.x == 0) own[16] = p.sblk16 != nullptr ? 1 : 0;
    while (true) {
        const int lane = wave_lane<true, DT == 1>();
        if (wv == 0) {
            int64_t drawn = lane == 0 ? serve_next_job(p) : 0;
            drawn = (int64_t)readlane64((uint64_t)drawn, 0);
            if (lane == 0) {
                own[11] = (int32_t)(drawn & 0xFFFFFFFFll);
                own[12] = (int32_t)(drawn >> 32);
            }
            if (drawn >= 0) {   // wave-uniform: the job from the host's ring, its header to LDS, the query to the device slot
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
                const uint4 *src = (const uint4 *)(p.host_ring + (size_t)((uint64_t)drawn % (uint64_t)p.ring_slots) * (size_t)p.slot_stride);
                uint4 *dst = (uint4 *)serve_slot(p, (uint64_t)drawn);
                const int n16 = p.slot_stride / 16;
                for (int i = lane; i < n16; i += 128) {   // (a slot has at most 68 pieces: one trip across PCIe)
                    const uint4 a = src[i];
                    const bool two = i + 64 < n16;
                    const uint4 b = two ? src[i + 64] : make_uint4(0, 0, 0, 0);
                    if (i < kServeHdr / 16) ((uint4 *)runs)[i] = a;
                    else dst[i] = a;
                    if (two) dst[i + 64] = b;
                }
            }
        }
        __syncthreads();
        const int64_t job = ((int64_t)own[12] << 32) | (uint32_t)own[11];
        if (job < 0) return;   // (the whole workgroup: every wave reads the same word)
        const size_t soff = (size_t)((uint64_t)job % (uint64_t)p.ring_slots);
        const void *qvec = serve_slot(p, (uint64_t)job) + kServeHdr;
        ServeResult *res = p.results + soff;

        // route (ClassifyQueries of Alg. 2, smallest list of Section 4.3.2): every lane computes the same
        const ServeJobHdr *hdr = (const ServeJobHdr *)runs;
        int nl = 0;
        int32_t labs[kMaxOthers + 1];
        const int n_hdr = hdr->n_labels;
        const int n_in = n_hdr < kMaxOthers + 1 ? n_hdr : kMaxOthers + 1;
        for (int i = 0; i < n_in; ++i) {
            const int32_t l = hdr->labels[i];
            bool seen = l < 0 || l >= p.n_labels;   // (the host has checked the range; never trust a ring)
            for (int u = 0; u < nl; ++u) seen = seen || labs[u] == l;
            if (!seen) labs[nl++] = l;
        }
        int32_t best = nl > 0 ? labs[0] : -1;
        bool empty = nl == 0;
        for (int i = 0; i < nl; ++i) {
            const int32_t sl = p.bp.meta.S[labs[i]], sb = p.bp.meta.S[best];
            if (sl == 0) empty = true;
            if (sl < sb || (sl == sb && labs[i] < best)) best = labs[i];
        }
        int o_cnt = 0;
        if (wv == 0 && lane == 0) {
            for (int i = 0; i < nl; ++i)
                if (labs[i] != best) own[o_cnt++] = labs[i];
            own[8] = 0; own[9] = o_cnt; own[10] = 0;
        }
        o_cnt = nl > 0 ? nl - 1 : 0;
        __syncthreads();

        const int k = p.bp.k;
        const bool graph = !empty && p.bp.meta.S[best] >= p.T;
        // the seeds of a graph job are shared out over the workgroup's waves: each scores its share from the
        // interleaved seed copy into a list of its own and leaves that list as a sorted run of keys
        const bool shared_seeds = graph && p.bp.sblk != nullptr;
        int seg = 64;
        const int ns = graph ? (p.bp.n_seeds < p.bp.meta.S[best] ? p.bp.n_seeds : p.bp.meta.S[best]) : 0;
        const bool filtered = DT == 1 && shared_seeds && o_cnt == 0 && own[16] != 0 && ns >= kSeedMfmaLeast;
        uint32_t *const seed_row = filtered ? p.rows + (int64_t)(blockIdx.x - 1) * p.row_words : nullptr;
        if (filtered) {
            if constexpr (DT == 1) {
                seg = (((ns + NW - 1) / NW) + 31) & ~31;
                const int j_lo = wv * seg, j_hi = j_lo + seg < ns ? j_lo + seg : ns;
                // the query in binary16, and its norm
                const int nchunks = p.row_bytes / kChunkBytes;
                uint4 v0 = make_uint4(0, 0, 0, 0), v1 = v0;
                if (2 * lane < nchunks) v0 = ((const uint4 *)qvec)[2 * lane];
                if (2 * lane + 1 < nchunks) v1 = ((const uint4 *)qvec)[2 * lane + 1];
                const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
                float qn = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) qn += __uint_as_float(w[i]) * __uint_as_float(w[i]);
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) qn += __shfl_xor(qn, o);
                if (lane < p.s16_chunks) hq[lane] = scaled_half8(v0, v1, p.bp.scale);
                wave_sync<true>();
                constexpr int STEPS = NC == 32 ? 8 : NC == 24 ? 6 : 16;
                if (j_lo < j_hi)
                    seed_filter_segment<STEPS, NC != 0>(p, best, hq, qn, ns, j_lo, j_hi, (uint32_t *)(runs + wv * 64), seed_row, seed_row + p.ns_stride, lane);
            }
        } else if (shared_seeds) {
            const int nchunks = p.row_bytes / kChunkBytes;
            seg = (((ns + NW - 1) / NW) + 63) & ~63;
            const int j_lo = wv * seg, j_hi = j_lo + seg < ns ? j_lo + seg : ns;
            for (int i = lane; i < nchunks; i += 64) hq[i] = ((const uint4 *)qvec)[i];
            wave_sync<true>();
            TopM<1> part;
            part.init(p.bp.itopk);
            if (j_lo < j_hi) stream_seed_segment<DT>(p.bp, best, own, o_cnt, hq, nchunks, j_lo, j_hi, true, part, lane);
            const uint64_t key = part.cur[0];   // (distance bits << 32 | seed index << 1 | 1), ascending
            runs[wv * 64 + lane] = key == KEY_MAX ? KEY_MAX : (key & 0xFFFFFFFF00000000ull) | ((key >> 1) & 0x7FFFFFFFull);
        }
        // a scan list is shared out the same way, in whole groups: each wave leaves the k best of its share (one wave
        // scanning a list of a few thousand vectors was the longest job of a session)
        int32_t *part_idx = (int32_t *)(runs + wv * 64);
        uint32_t *part_bits = (uint32_t *)part_idx + 64;
        if (!empty && !graph) {
            const int n = p.bp.meta.S[best], per = ((n + kGroup * NW - 1) / (kGroup * NW)) * kGroup;
            ScanParams sp = p.sp;
            sp.qsrc = qvec; sp.qrow = own + 10;
            sp.others_off = o_cnt > 0 ? own + 8 : nullptr; sp.others = own;
            sp.res_idx = part_idx; sp.res_bits = part_bits;
            ScanItem it;
            it.group0 = p.GO_LS[best] + wv * (per / kGroup); it.map_off = p.bp.meta.O_LS[best]; it.entry0 = wv * per;
            it.n = n - wv * per < per ? n - wv * per : per;
            it.q_begin = 0; it.q_count = 1; it.self_base = -1; it.part_row = 0;
            uint4 *scan_smem = (uint4 *)((char *)smem + (size_t)wv * p.lds_scan);
            if (it.n <= 0) {
                part_idx[lane] = -1;
            } else if constexpr (DT == 1 && (NC == 24 || NC == 32)) {
                // the FMA scan takes its query as a wave-uniform operand: from LDS here (see scan_valu_item)
                for (int i = lane; i < NC; i += 64) hq[i] = ((const uint4 *)qvec)[i];
                wave_sync<true>();
                scan_valu_item<NC, true>(sp, it, scan_smem, (const float *)hq);
            } else {
                scan_topk_item<DT, NC, true>(sp, it, scan_smem);
            }
        }
        __syncthreads();

        if (wv == 0) {
            if (empty) {
                if (lane < k) { res->ids[lane] = -1; res->dists[lane] = __builtin_inff(); }
            } else if (graph) {
                BeamQuery bq;
                bq.q = qvec; bq.label = best; bq.others = own; bq.o_cnt = o_cnt;
                bq.out_ids = res->ids; bq.out_dists = res->dists;
                bq.counters = nullptr; bq.gathered = nullptr; bq.dseed_row = nullptr; bq.runs = nullptr; bq.seed_pass = -1;
                BeamParams bp = p.bp;
                bp.seed_approx = filtered ? 1 : 0;
                if (filtered) {
                    bq.dseed_row = seed_row;
                    bq.dmin_row = seed_row + p.ns_stride;
                    bq.counters = own + 20;
                } else if (shared_seeds) {   // the waves' runs, merged by the search as the runs of a selecting seed kernel would be
                    bq.runs = runs;
                    bp.run_K = 64; bp.run_segs = NW; bp.seg_seeds = seg;
                }
                // (uint8 workers leave registers for other kernels on their compute unit)
                if constexpr (DT == 0) beam_search_wave<DT, 1, true>(bp, bq, smem);
                else if (o_cnt == 0) beam_search_wave<DT, 1, true, false, true>(bp, bq, smem);
                else beam_search_wave<DT, 1, true, true, true>(bp, bq, smem);
                if (filtered) {
                    wave_sync<true>();
                    ++met;
                    failed += __builtin_amdgcn_readfirstlane(own[23]) & 1;
                    if (lane == 0 && 16 * failed > met + 64) own[16] = 0;
                }
            } else {
                TopM<1> list;   // the waves' runs, ascending by (distance, entry)
                list.init(k);
                for (int w = 0; w < NW; ++w) {
                    const int32_t *ri = (const int32_t *)(runs + w * 64);
                    const int32_t idx = lane < k ? ri[lane] : -1;
                    merge_sorted_run(list, idx >= 0 ? ((uint64_t)(uint32_t)ri[64 + lane] << 32) | (uint32_t)idx : KEY_MAX, lane);
                }
                if (lane < k) {
                    const uint64_t key = list.cur[0];
                    const uint32_t hi = (uint32_t)(key >> 32);
                    res->ids[lane] = key == KEY_MAX ? -1 : (int64_t)p.sp.map[p.bp.meta.O_LS[best] + (uint32_t)key];
                    res->dists[lane] = key == KEY_MAX ? __builtin_inff() : DT == 0 ? (float)(int)hi : __uint_as_float(hi);
                }
            }
            wave_sync<true>();
            __threadfence_system();
            if (lane == 0) {
                __hip_atomic_store(&res->done, (uint64_t)job + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_fetch_add(&p.dctrl->jobs_done, (uint64_t)1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
    }
}

}  // namespace vf

using namespace vf;

struct vf_server {
    vf_index *ix = nullptr;
    hipStream_t stream = nullptr;
    char *h_ring = nullptr;               // pinned
    ServeResult *h_results = nullptr;     // pinned
    ServeHostCtrl *h_ctrl = nullptr;      // pinned
    DevBuf d_ring, d_ctrl, d_GO_LS, d_rows;
    SeedCopy seeds;                       // the session's own interleaved copy of the seeds (workers score from it)
    int32_t ring_slots = 0, slot_stride = 0, row_bytes = 0, k = 0;
    int64_t max_jobs = 0;
    uint64_t next_job = 0;
    bool launched = false;
    std::mutex mu;
};

static void free_server(vf_server *sv)
{
    if (!sv) return;
    if (sv->stream) { (void)hipStreamSynchronize(sv->stream); (void)hipStreamDestroy(sv->stream); }
    sv->d_ring.release(); sv->d_ctrl.release(); sv->d_GO_LS.release(); sv->d_rows.release();
    for (DevBuf *b : sv->seeds.bufs()) b->release();
    if (sv->h_ring) (void)hipHostFree(sv->h_ring);
    if (sv->h_results) (void)hipHostFree(sv->h_results);
    if (sv->h_ctrl) (void)hipHostFree(sv->h_ctrl);
    delete sv;
}

// No more workers than are resident on all compute units but kServeFreeCus.  A session that fills the chip lets nothing else
// run until it ends: workers of 256 registers (float32) take a compute unit's whole register file, and a caller who then waits
// for a copy of up to 16 KiB, which is a kernel (12 KiB beside 255 workers: until the idle bound; beside 240 0.2 ms), submits
// nothing more until the session has ended by itself.  A worker that is not resident does nothing for the session either: job
// numbers are drawn by running workers only.
constexpr int kServeFreeCus = 16;

template <int DT, int NC, int NW> static int launch_serve_nw(const ServeParams &p, int n_workers, size_t lds, hipStream_t s)
{
    int per_cu = 0, dev = 0, cus = 0;
    VF_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, serve_kernel<DT, NC, NW>, 64 * NW, lds));
    VF_HIP(hipGetDevice(&dev));
    VF_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int most = std::max(1, per_cu * std::max(1, cus - kServeFreeCus));
    hipLaunchKernelGGL((serve_kernel<DT, NC, NW>), dim3(1 + std::min(n_workers, most)), dim3(64 * NW), lds, s, p);
    VF_HIP(hipGetLastError());
    return VF_OK;
}

template <int DT, int NC> static int launch_serve(const ServeParams &p, int n_workers, int waves, size_t lds, hipStream_t s)
{
    if (waves == 1) return launch_serve_nw<DT, NC, 1>(p, n_workers, lds, s);
    if (waves == 4) return launch_serve_nw<DT, NC, 4>(p, n_workers, lds, s);
    return launch_serve_nw<DT, NC, 8>(p, n_workers, lds, s);
}

static int serve_begin_impl(vf_index *ix, const vf_serve_params *prm, vf_server **out)
{
    VF_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    VF_REQUIRE(ix != nullptr && prm != nullptr, "NULL argument");
    int32_t k = prm->k, itopk = prm->itopk, width = prm->width, iters = prm->iters, n_seeds = prm->n_seeds;
    VF_REQUIRE(k >= 1 && k <= 64, "k must be in [1, 64]");
    int rc = check_search_params(ix, false, k, itopk, width, iters, n_seeds);
    if (rc != VF_OK) return rc;
    VF_REQUIRE(itopk <= 64, "vf_serve_begin: itopk must be at most 64");
    const int32_t n_workers = prm->n_workers > 0 ? prm->n_workers : 240;
    const int32_t waves = prm->waves_per_worker > 0 ? prm->waves_per_worker : 8;
    VF_REQUIRE(waves == 1 || waves == 4 || waves == 8, "waves_per_worker must be 1, 4 or 8 (0 = 8)");
    const int32_t ring_slots = prm->ring_slots > 0 ? prm->ring_slots : 1024;
    VF_REQUIRE(n_workers >= 1 && n_workers <= 1023, "n_workers must be in [1, 1023]");
    VF_REQUIRE(ring_slots >= 1 && ring_slots <= (1 << 20), "ring_slots must be in [1, 2^20]");
    const int64_t max_jobs = prm->max_jobs > 0 ? prm->max_jobs : ((int64_t)1 << 62);
    const int64_t idle_polls = prm->idle_polls > 0 ? prm->idle_polls : 2000000;
    VF_REQUIRE(idle_polls <= ((int64_t)1 << 32), "idle_polls must be at most 2^32");

    std::lock_guard<std::recursive_mutex> lock(ix->mu);
    vf_server *sv = new vf_server();
    struct Guard { vf_server *sv; ~Guard() { if (sv) free_server(sv); } } guard{sv};
    sv->ix = ix; sv->k = k; sv->ring_slots = ring_slots; sv->max_jobs = max_jobs;
    sv->row_bytes = (int32_t)((size_t)ix->dim * ix->elem());
    sv->slot_stride = kServeHdr + ((sv->row_bytes + 63) & ~63);
    sv->d_ring.al = sv->d_ctrl.al = sv->d_GO_LS.al = sv->d_rows.al = &ix->alloc;
    for (DevBuf *b : sv->seeds.bufs()) b->al = &ix->alloc;
    const size_t ring_bytes = (size_t)ring_slots * sv->slot_stride, dev_ring_bytes = ring_bytes + (size_t)ring_slots * kReadyBytes;
    const unsigned flags = hipHostMallocMapped | hipHostMallocCoherent;
    VF_HIP(hipHostMalloc((void **)&sv->h_ring, ring_bytes, flags));
    VF_HIP(hipHostMalloc((void **)&sv->h_results, (size_t)ring_slots * sizeof(ServeResult), flags));
    VF_HIP(hipHostMalloc((void **)&sv->h_ctrl, sizeof(ServeHostCtrl), flags));
    memset(sv->h_ring, 0, ring_bytes);
    memset(sv->h_results, 0, (size_t)ring_slots * sizeof(ServeResult));
    memset(sv->h_ctrl, 0, sizeof(ServeHostCtrl));
    VF_HIP(hipStreamCreateWithFlags(&sv->stream, hipStreamNonBlocking));
    if ((rc = sv->d_ring.reserve(dev_ring_bytes)) != VF_OK) return rc;
    if ((rc = sv->d_ctrl.reserve(sizeof(ServeDevCtrl))) != VF_OK) return rc;
    if ((rc = upload(sv->d_GO_LS, ix->GO_LS, sv->stream)) != VF_OK) return rc;
    VF_HIP(hipMemsetAsync(sv->d_ctrl.p, 0, sizeof(ServeDevCtrl), sv->stream));
    VF_HIP(hipMemsetAsync(sv->d_ring.p, 0, dev_ring_bytes, sv->stream));
    VF_HIP(hipStreamSynchronize(sv->stream));
    // the seeds of every graph list, interleaved, in the data's own type (exact distances): a worker streams its
    // query's seeds from it, one seed per lane.  The session owns the copy (the index's copies may be dropped
    // while the kernel runs).  When it does not fit, workers gather the seeds' rows from the vector table.
    // float32 data: beside it the copy in binary16 (see seed_filter_segment).
    int32_t longest = 0;
    for (int32_t l : ix->graph_labels) longest = std::max(longest, std::min(n_seeds, ix->S[(size_t)l]));
    const int32_t ns_stride = (longest + 31) & ~31, row_words = ns_stride + (((ns_stride / 32) + 63) & ~63);
    const bool want_f16 = ix->dtype == VF_F32 && ix->dim <= 256 && wants_seed_copy(ix, false, itopk, n_seeds) && ix->seeds_provable(itopk) && n_seeds >= kSeedMfmaLeast && ix->tune.seed_bf16 && !ix->seed_bf16_off &&
                          longest >= kSeedMfmaLeast && (int64_t)n_workers * row_words <= ((int64_t)64 << 20);
    if (!ix->graph_labels.empty() && (rc = build_seed_copy(ix, n_seeds, sv->stream, want_f16, true, &sv->seeds)) != VF_OK) return rc;

    ServeParams p{};
    // beam search: geometry as vf_search computes it
    int32_t LP = 128, hb = 9;
    while (LP < itopk + std::max(64, width * ix->R)) LP <<= 1;
    const int64_t visits = (int64_t)iters * width * ix->R;
    while (hb < 13 && ((int64_t)1 << hb) < 2 * visits) ++hb;
    p.bp.X = ix->X; p.bp.G = ix->d_G.as<int32_t>(); p.bp.Gg = ix->d_Gg.as<int32_t>(); p.bp.meta = ix->meta();
    p.bp.dim = ix->dim; p.bp.R = ix->R; p.bp.k = k; p.bp.itopk = itopk; p.bp.width = width; p.bp.iters = iters;
    p.bp.n_seeds = n_seeds; p.bp.LP = LP; p.bp.hash_bits = hb;
    if (sv->seeds.ok && sv->seeds.has_f32) {
        p.bp.sblk = sv->seeds.blk.as<uint4>(); p.bp.sgoff = sv->seeds.goff.as<int64_t>(); p.bp.sblk_chunks = 2 * ix->ncp;
    }
    bool filter = p.bp.sblk != nullptr && sv->seeds.has_f16;
    if (filter && (rc = sv->d_rows.reserve((size_t)n_workers * row_words * 4)) != VF_OK) {   // (no memory for them: the float32 copy serves)
        if (rc != VF_ENOMEM) return rc;
        (void)hipGetLastError();
        filter = false;
    }
    if (filter) {
        p.sblk16 = sv->seeds.blk16.as<uint4>(); p.snorm = sv->seeds.norm.as<float>(); p.s16_chunks = ix->ncp;
        p.rows = sv->d_rows.as<uint32_t>(); p.ns_stride = ns_stride; p.row_words = row_words;
        half_bound(ix, sv->seeds.f16_delta, p.bp);
        p.bp.xn_max = ix->xn_max; p.bp.seed_keep = 64;
        p.minus_two_unscaled = -2.0f / (p.bp.scale * p.bp.scale);
    }
    const size_t beam_lds = beam_lds_bytes(p.bp, ix->dtype);
    // scan: one query against a whole list
    p.sp.xblk = ix->d_X_LS.as<uint4>(); p.sp.xnorm = ix->d_xnorm_LS.p; p.sp.map = ix->d_M_LS.as<int32_t>();
    p.sp.dim = ix->dim; p.sp.ncp = ix->ncp; p.sp.K = k; p.sp.tile_rows = 1; p.sp.meta = ix->meta();
    const bool valu = scan_valu_supported(ix->dtype, ix->dim, 16);
    const size_t scan_lds = ((valu ? (size_t)(96 + (k | 1)) * 8 + 2 * 32 * 4 : scan_lds_bytes(ix->ncp, 1, k)) + 63) & ~(size_t)63;   // of one wave
    const size_t lds_kernels = (std::max(beam_lds, waves * scan_lds) + 63) & ~(size_t)63;
    const size_t lds_own = 128;
    // per wave a copy of the query and a run of 64 seed keys
    const size_t lds_share = (size_t)waves * ((((size_t)sv->row_bytes + 15) & ~(size_t)15) + 64 * 8);
    VF_REQUIRE(lds_kernels + lds_own + lds_share <= 64 * 1024, "search parameters need more than 64 KiB of LDS");
    p.GO_LS = sv->d_GO_LS.as<int64_t>(); p.T = ix->T; p.n_labels = ix->n_labels;
    p.ring_slots = ring_slots; p.slot_stride = sv->slot_stride; p.row_bytes = sv->row_bytes;
    void *dv = nullptr;
    VF_HIP(hipHostGetDevicePointer(&dv, sv->h_ring, 0)); p.host_ring = (const char *)dv;
    VF_HIP(hipHostGetDevicePointer(&dv, sv->h_results, 0)); p.results = (ServeResult *)dv;
    VF_HIP(hipHostGetDevicePointer(&dv, sv->h_ctrl, 0)); p.hctrl = (ServeHostCtrl *)dv;
    p.dev_ring = sv->d_ring.as<char>(); p.dctrl = sv->d_ctrl.as<ServeDevCtrl>();
    p.max_jobs = max_jobs; p.idle_polls = idle_polls; p.lds_kernels = (int32_t)lds_kernels; p.lds_own = (int32_t)lds_own; p.lds_scan = (int32_t)scan_lds;
    const size_t lds = lds_kernels + lds_own + lds_share;
    if (ix->dtype == VF_U8) {
        if (ix->dim == 128) rc = launch_serve<0, 4>(p, n_workers, waves, lds, sv->stream);
        else if (ix->dim == 192) rc = launch_serve<0, 6>(p, n_workers, waves, lds, sv->stream);
        else rc = launch_serve<0, 0>(p, n_workers, waves, lds, sv->stream);
    } else {
        if (ix->dim == 128) rc = launch_serve<1, 32>(p, n_workers, waves, lds, sv->stream);
        else if (ix->dim == 96) rc = launch_serve<1, 24>(p, n_workers, waves, lds, sv->stream);
        else rc = launch_serve<1, 0>(p, n_workers, waves, lds, sv->stream);
    }
    if (rc != VF_OK) return rc;
    sv->launched = true;
    guard.sv = nullptr;
    *out = sv;
    return VF_OK;
}

static int serve_submit_impl(vf_server *sv, const void *query, const int32_t *labels, int32_t n_labels, int64_t *job)
{
    VF_REQUIRE(sv && query && labels && job, "NULL argument");
    VF_REQUIRE(n_labels >= 1 && n_labels <= kMaxOthers + 1, "a query needs 1 to 8 labels");
    for (int32_t i = 0; i < n_labels; ++i)
        VF_REQUIRE(labels[i] >= 0 && labels[i] < sv->ix->n_labels, "query label outside [0, n_labels)");
    std::lock_guard<std::mutex> lock(sv->mu);
    std::atomic_thread_fence(std::memory_order_acquire);
    VF_REQUIRE(__atomic_load_n(&sv->h_ctrl->exit_reason, __ATOMIC_ACQUIRE) == 0,
               "the serving kernel has ended (stop requested, max_jobs reached, or idle for too long): begin a new session");
    VF_REQUIRE((int64_t)sv->next_job < sv->max_jobs, "max_jobs of this session have been submitted");
    const uint64_t j = sv->next_job;
    if (j >= (uint64_t)sv->ring_slots) {
        // the slot's previous job must be done: its worker copies it from the host ring, after it was published, and its
        // result slot is about to be reused
        const uint64_t prev = j - (uint64_t)sv->ring_slots;
        const uint64_t done = __atomic_load_n(&sv->h_results[prev % (uint64_t)sv->ring_slots].done, __ATOMIC_ACQUIRE);
        if (done < prev + 1) {
            set_error("the job ring is full");
            return VF_EBUSY;
        }
    }
    char *slot = sv->h_ring + (size_t)(j % (uint64_t)sv->ring_slots) * sv->slot_stride;
    ServeJobHdr hdr{};
    hdr.n_labels = n_labels;
    for (int32_t i = 0; i < n_labels; ++i) hdr.labels[i] = labels[i];
    memcpy(slot, &hdr, sizeof(hdr));
    memcpy(slot + kServeHdr, query, (size_t)sv->row_bytes);
    __atomic_store_n(&sv->h_ctrl->tail, j + 1, __ATOMIC_RELEASE);
    sv->next_job = j + 1;
    *job = (int64_t)j;
    return VF_OK;
}

static int serve_poll_impl(vf_server *sv, int64_t job, int64_t *out_ids, float *out_dists, int32_t *done)
{
    VF_REQUIRE(sv && done, "NULL argument");
    *done = 0;
    VF_REQUIRE(job >= 0 && (uint64_t)job < sv->next_job, "no such job");
    const ServeResult *res = sv->h_results + (size_t)((uint64_t)job % (uint64_t)sv->ring_slots);
    const uint64_t d = __atomic_load_n(&res->done, __ATOMIC_ACQUIRE);
    VF_REQUIRE(d <= (uint64_t)job + 1, "the job's result has been overwritten by a later job (the result ring wrapped)");
    if (d < (uint64_t)job + 1) {
        // not done: say so, unless the kernel has ended and never will be
        if (__atomic_load_n(&sv->h_ctrl->exit_reason, __ATOMIC_ACQUIRE) != 0 &&
            __atomic_load_n(&res->done, __ATOMIC_ACQUIRE) < (uint64_t)job + 1) {
            set_error("the serving kernel ended before this job was processed");
            return VF_EINVAL;
        }
        return VF_OK;
    }
    if (out_ids) memcpy(out_ids, res->ids, (size_t)sv->k * 8);
    if (out_dists) memcpy(out_dists, res->dists, (size_t)sv->k * 4);
    *done = 1;
    return VF_OK;
}

static int serve_end_impl(vf_server *sv, int64_t *jobs_done, int32_t *exit_reason)
{
    VF_REQUIRE(sv != nullptr, "server is NULL");
    {
        std::lock_guard<std::mutex> lock(sv->mu);
        __atomic_store_n(&sv->h_ctrl->stop, 1u, __ATOMIC_RELEASE);
    }
    VF_HIP(hipStreamSynchronize(sv->stream));   // every wave of the kernel exits by itself
    if (jobs_done) *jobs_done = (int64_t)__atomic_load_n(&sv->h_ctrl->jobs_done, __ATOMIC_ACQUIRE);
    if (exit_reason) *exit_reason = (int32_t)__atomic_load_n(&sv->h_ctrl->exit_reason, __ATOMIC_ACQUIRE);
    free_server(sv);
    return VF_OK;
}

// A host batch through the session: submit in order with at most in_flight jobs outstanding, collect as they finish.
static int serve_run_impl(vf_server *sv, const void *queries, int64_t nq, const int64_t *qoff, const int32_t *qids,
                          int32_t in_flight, int64_t *out_ids, float *out_dists, float *latency_us)
{
    VF_REQUIRE(sv && queries && qoff && qids && out_ids && out_dists, "NULL argument");
    VF_REQUIRE(nq >= 0 && in_flight >= 1 && in_flight <= sv->ring_slots, "in_flight must be in [1, ring_slots]");
    using clock = std::chrono::steady_clock;
    std::vector<clock::time_point> t_sub((size_t)nq);
    std::vector<int64_t> job_of((size_t)nq);
    // Jobs finish out of order (a scan of a short list long before a graph search): each is collected when it is done and
    // its place in flight goes to the next query at once.  Waiting for the oldest first left most of the places idle.
    std::vector<int64_t> open;    // submitted, not collected; ascending
    open.reserve((size_t)in_flight);
    int64_t next = 0;
    const auto deadline = clock::now() + std::chrono::seconds(120);
    while (next < nq || !open.empty()) {
        bool moved = false;
        // (a result must be read before ring_slots further jobs are submitted)
        while (next < nq && (int64_t)open.size() < in_flight && (open.empty() || next - open[0] < sv->ring_slots)) {
            const int64_t b = qoff[next], e = qoff[next + 1];
            VF_REQUIRE(e > b && e - b <= kMaxOthers + 1, "a query needs 1 to 8 labels");
            int64_t job = -1;
            const int rc = serve_submit_impl(sv, (const char *)queries + (size_t)next * sv->row_bytes, qids + b, (int32_t)(e - b), &job);
            if (rc == VF_EBUSY) break;
            if (rc != VF_OK) return rc;
            t_sub[(size_t)next] = clock::now();
            job_of[(size_t)next] = job;
            open.push_back(next);
            ++next;
            moved = true;
        }
        size_t left = 0;
        for (const int64_t q : open) {
            int32_t done = 0;
            const int rc = serve_poll_impl(sv, job_of[(size_t)q], out_ids + q * sv->k, out_dists + q * sv->k, &done);
            if (rc != VF_OK) return rc;
            if (done) {
                if (latency_us) latency_us[q] = std::chrono::duration<float, std::micro>(clock::now() - t_sub[(size_t)q]).count();
                moved = true;
            } else {
                open[left++] = q;
            }
        }
        open.resize(left);
        if (!moved && clock::now() > deadline) {
            set_error("vf_serve_run: no progress for two minutes");
            return VF_EHIP;
        }
    }
    return VF_OK;
}

extern "C" int vf_serve_run(vf_server *server, const void *queries, int64_t nq, const int64_t *qlabel_offsets,
                            const int32_t *qlabel_ids, int32_t in_flight, int64_t *out_ids, float *out_dists,
                            float *latency_us)
{
    return guarded([&] { return serve_run_impl(server, queries, nq, qlabel_offsets, qlabel_ids, in_flight, out_ids, out_dists, latency_us); });
}

extern "C" int vf_serve_begin(vf_index *index, const vf_serve_params *params, vf_server **out)
{
    return guarded([&] { return serve_begin_impl(index, params, out); });
}

extern "C" int vf_serve_submit(vf_server *server, const void *query, const int32_t *labels, int32_t n_labels, int64_t *job)
{
    return guarded([&] { return serve_submit_impl(server, query, labels, n_labels, job); });
}

extern "C" int vf_serve_poll(vf_server *server, int64_t job, int64_t *out_ids, float *out_dists, int32_t *done)
{
    return guarded([&] { return serve_poll_impl(server, job, out_ids, out_dists, done); });
}

extern "C" int vf_serve_end(vf_server *server, int64_t *jobs_done, int32_t *exit_reason)
{
    return guarded([&] { return serve_end_impl(server, jobs_done, exit_reason); });
}
