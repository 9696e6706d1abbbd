// Contraction of many rows against whole lists with the exact top-K selection fused in: the kNN self-joins of the index
// build (Alg. 1) and the scans of graph lists for the exact ground truth.  Where the scan kernels serve a handful of
// queries per list and are bound by the list's bytes, a join has as many rows as it has and is bound by the matrix cores
// and by the selection, so everything here is arranged around those two.
//
// Tile.  A wave takes 32 rows, their operand in registers.  Where rows are many a workgroup of four waves streams a
// segment of the list through LDS, one group of 32 entries per step, two buffers: a group is fetched from L2 once per 128
// rows (every wave by itself: the self-joins below are bound by the memory behind L2, 45 ms instead of 30).  A list of queries
// (ground truth; rows that are joined again) is read by one wave by itself, up to 8 steps (kJoinAloneSteps).  Lists come packed
// (join_pack_kernel): per group the 16-byte chunks chunk-major, which is the B operand of the 32-column MFMAs, lane
// (n32, h) reading chunk 2 s + h of entry n32.
//
// Operands.  float32 data is centred (a vector near the table's mean is subtracted while it is packed and split): distances
// stay what they are, and what norms and products lose is relative to the spread of the data instead of to its distance
// from the origin.  With u = 2^-24:
//   one part (kJoinSingle): x rounded to binary16 after multiplication by a power of two that brings the table's largest
//   norm into [32, 64): a relative error of 2^-11 of any vector, of the table's own rows measured when the index is built
//   (about 2^-12.3), so 2 (rho_q + rho_x) |q||x| in the distance; components that fall below binary16's range lose at
//   most 2^-15 of the largest norm in all, 2^-13 (|q|^2 + |x|^2) in the distance.  One product on
//   v_mfma_f32_32x32x16_f16.  The gap between the R-th and the 48th neighbour is ten times that on the repository's
//   workloads; whatever row is not proven (clusters several times further apart than they are wide) is joined again on
//   two parts, and an index of such rows takes two parts from the start.  Queries have the larger bound and a k of their own:
//   they take one part where the build's rows would have been proven as queries, and for k up to the rows' length (5,000
//   queries over 500,000: 1.18 ms, on two parts 1.38; where they would not, a lone query over 200,000 x 128 at k = 48 took
//   828 us on one part, answered by the ordered scan, and takes 302 on two).
//   two parts (kJoinSplit): x = hi + lo with hi = bf16(x), lo = bf16(x - hi); lo.hi and hi.lo into an accumulator of their
//   own (their partial sums stay small), hi.hi into another, added at the end.  They leave out: |x - hi - lo| <= 2^-18 |x|
//   twice and the product of the low parts 2^-18, together 192 u |q||x| in q.x, 193 u (|q|^2 + |x|^2) in the distance.
//   both: the sums 2 u per term; norms, summed one after the other, u per term; the subtraction of the centre, u per
//   component, 4 u (|q|^2 + |x|^2) in the distance; final additions, the thresholds' and the ordered distance's own
//   rounding < 100 u: 300 u + 3 u per component in all.  The bound used is 512 u + 4 u per component = join_err_bound().
// Callers re-rank what the join keeps with the ordered distance and prove with these bounds that nothing else belongs to
// the result, so results do not depend on the operands.
// uint8 data: v_mfma_i32_32x32x32_i8 on the bytes shifted by -128: exact.
//
// Selection.  With v = q.x - |x|^2 / 2 (uint8: 2 q.x - |x|^2) a distance is below a row's threshold where v is at least
// a per-row constant t, or q.x - t at least |x|^2 / 2: the right side is the lane's entry's alone, so one subtraction per pair
// and the maxima of four rows each decide, and only quarters with a candidate are looked at by element.  (In float32 the two forms
// round differently: the second one holds for every entry whose unrounded v is at least t, and thresholds allow for what v's own
// rounding adds.)  Candidates are
// appended to one list of the wave in LDS, without a look at its end; a group that overruns it (before thresholds exist) is
// gone through again, delivering in between; when it is half full they are delivered to the rows' queues (16 slots, LDS
// atomics over 64 candidates at a time), and rows with ten or more merge their queue into their sorted K best: four rows
// share a 64-lane sort network, then one merge network per row.  The K best live in the partial result rows in global
// memory, the next four rows' requested while four are merged.  The waves of a workgroup deliver together: a wave that
// merges lets the others wait at the next group's barrier, so merges at different times cost the workgroup their sum.
// First thresholds come from a sample of up to 64 groups (the largest values of two groups' lanes, K of which are at or
// above the K-th largest of them); without it a third of all candidates fall into a row's first thousand entries.  The
// segments of a ground truth list share the rows' bounds.
//
// Measured: self-joins of 36 lists of 4,000 to 170,000 float32 vectors, dim 128 (4.7e10 pairs) 29.4 -> 22.9 ms, uint8 of 128
// and 192 components 4.26 -> 3.60 and 5.47 -> 5.05 (before: a compare and a mask in scalar registers per pair, sixteen of them
// kept, spilled and branched on in every group with a candidate; 156 registers, three waves per SIMD); ground truth of 5,000
// queries over 500,000 0.67 -> 0.63 ms.  Per 32 x 32 pairs a SIMD takes 1,180 cycles: 113 vector instructions (450), 8 MFMAs (260),
// and what four waves leave uncovered of a wave's chain of LDS reads, products, branches and the workgroup's barrier (3,200
// cycles, a quarter each).  Made no difference: list groups that are always in cache, half the LDS reads, groups touched four
// ahead, more rows of the sample, wave priorities, two groups per barrier with two chains of products (three waves: 25 ms).
#include "vf_select.h"

namespace vf {

typedef __bf16 v8bf_join __attribute__((ext_vector_type(8)));
typedef _Float16 v8h_join __attribute__((ext_vector_type(8)));
typedef float v16f_join __attribute__((ext_vector_type(16)));
typedef int v16i_join __attribute__((ext_vector_type(16)));
typedef int v4i_join __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_join __attribute__((ext_vector_type(4)));

// four components of a row (chunk c) less those of the centre
__device__ __forceinline__ float4 centred(float4 v, const float *centre, int c)
{
    const float4 m = ((const float4 *)centre)[c];
    return make_float4(v.x - m.x, v.y - m.y, v.z - m.z, v.w - m.w);
}

// bfloat16 high parts of eight floats, and the bfloat16 rounding of what they leave
__device__ __forceinline__ void split_bf16x8(const float (&f)[8], uint4 &hi, uint4 &lo)
{
    uint32_t a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = bf16_rn_bits(f[i]);
        b[i] = bf16_rn_bits(f[i] - __uint_as_float(a[i] << 16));
    }
    hi = make_uint4(a[0] | (a[1] << 16), a[2] | (a[3] << 16), a[4] | (a[5] << 16), a[6] | (a[7] << 16));
    lo = make_uint4(b[0] | (b[1] << 16), b[2] | (b[3] << 16), b[4] | (b[5] << 16), b[6] | (b[7] << 16));
}

// eight floats rounded to binary16
__device__ __forceinline__ uint4 half8(const float (&f)[8])
{
    v8h_join x;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (_Float16)f[i];
    return __builtin_bit_cast(uint4, x);
}

// ---------------------------------------------------------------- sorting networks over the lanes of a wave
//
// Bitonic networks over 64-bit keys held one per lane, every cross-lane move on the vector ALU: lane ^ 1, 2, 4, 8 are
// DPP moves (xor 4 = the mirror of 8 lanes, then the mirror of 4), lane ^ 16 and ^ 32 the row swaps of gfx950, which
// leave both partners' keys in both lanes.  Which lanes keep the smaller key of a stage is a constant, so a stage is two
// moves, one compare, one scalar xor of its result with that constant, and two selects.  Several sets run at a time here,
// which hides the trip through the scalar unit; a lone chain (lane_exchange_lone in vf_device.h) selects twice instead.

// One compare-exchange stage: the lanes of MIN keep the smaller key of the pair (lane, lane ^ J), the others the larger.
template <int J, uint64_t MIN> __device__ __forceinline__ uint64_t lane_exchange(uint64_t v)
{
    uint32_t al, bl, ah, bh;
    lane_pair<J>((uint32_t)v, al, bl);
    lane_pair<J>((uint32_t)(v >> 32), ah, bh);
    const uint64_t a = ((uint64_t)ah << 32) | al, b = ((uint64_t)bh << 32) | bl;
    return __builtin_amdgcn_inverse_ballot_w64(__builtin_amdgcn_ballot_w64(a < b) ^ ~MIN) ? a : b;
}

// ... and of 32-bit values
template <int J, uint64_t MIN> __device__ __forceinline__ float lane_exchange(float v) { return lane_exchange_32<J, MIN>(v); }
template <int J, uint64_t MIN> __device__ __forceinline__ int lane_exchange(int v) { return lane_exchange_32<J, MIN>(v); }

// The stages J, J / 2, .. 1 that make a bitonic sequence of each aligned block of K lanes ascending (DESC: descending);
// LAST: every block, else blocks alternate.  NR independent sets: their dependent chains interleave.
template <int K, int J, bool LAST, bool DESC, class T, int NR> __device__ __forceinline__ void lane_merge_stages(T (&v)[NR])
{
#pragma unroll
    for (int u = 0; u < NR; ++u) v[u] = lane_exchange<J, keep_min_lanes<K, J, LAST, DESC>()>(v[u]);
    if constexpr (J > 1) lane_merge_stages<K, J / 2, LAST, DESC>(v);
}
template <int K, int SEG, bool DESC, class T, int NR> __device__ __forceinline__ void lane_sort_stages(T (&v)[NR])
{
    lane_merge_stages<K, K / 2, K == SEG, DESC>(v);
    if constexpr (K < SEG) lane_sort_stages<K * 2, SEG, DESC>(v);
}

// Sort of the values held one per lane, inside every aligned segment of SEG lanes.
template <int SEG, bool DESC, class T, int NR> __device__ __forceinline__ void lane_sort(T (&v)[NR])
{
    lane_sort_stages<2, SEG, DESC>(v);
}
// Ascending sort of a sequence that is bitonic inside every aligned segment of SEG lanes.
template <int SEG, class T, int NR> __device__ __forceinline__ void lane_merge(T (&v)[NR])
{
    lane_merge_stages<SEG, SEG / 2, true, false>(v);
}

__device__ __forceinline__ float larger(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ int larger(int a, int b) { return a > b ? a : b; }

constexpr int kJoinQueue = 16;   // pending keys per row
constexpr int kJoinMerge = 10;   // a row with as many of them is merged when its wave delivers
// candidates on their way to the rows' queues (two rows of a group add up to 64); one wave by itself has the LDS for twice as many: before
// thresholds tighten, rows that keep 60 entries and more have over 128 in a group
__host__ __device__ constexpr int join_flat(int w) { return w == 1 ? 256 : 128; }
constexpr int kJoinFull = 64;    // as many of them make the waves of a workgroup deliver together
__host__ __device__ constexpr int join_wave_lds(int w) { return 32 * kJoinQueue * 8 + join_flat(w) * 8 + 32 * 4 + 32 * 4 + join_flat(w); }   // bytes of a wave
// Groups that are looked at first, for a row's first threshold; a quarter of them where the rows and what is kept of each
// are so few (kJoinFew keys in all) that reading 64 groups twice costs more than the candidates it saves (a lone query over a
// list of 300,000 x 128, segments of 147 groups, split operands: 371 -> 341 us).
constexpr int kJoinSample = 64, kJoinSampleFew = 16, kJoinFew = 128;

template <int DT> struct JoinAcc { using type = v16f_join; using scalar = float; };
template <> struct JoinAcc<0> { using type = v16i_join; using scalar = int; };

// 16-byte chunks of a packed vector: DT 0 uint8, 1 float32 in two bfloat16 parts, 2 float32 in one binary16 part
template <int DT> __host__ __device__ constexpr int join_chunks(int nk) { return DT == 1 ? 4 * nk : 2 * nk; }

// lanes below this one whose bit is set in m
__device__ __forceinline__ int lanes_before(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Waves per SIMD that the registers are shared out for: as many as the row operand leaves registers for, without scratch memory but for
// uint8 of 4 steps with predicates where one wave reads the list (20 bytes a lane), of 6 steps where four do (16 bytes) and split
// operands of 16 steps (116 bytes, at two waves).
__host__ __device__ constexpr int join_waves(int dt, int nk, int w)
{
    return dt == 1 || nk > 8 ? 2 : (w == 1 ? nk > (dt == 0 ? 4 : 6) : nk > (dt == 0 ? 6 : 8)) ? 3 : 4;
}

// Operand chunks in flight: the steps of a group that are requested together.  A wave that reads split operands by itself has
// the registers for a whole group.
__host__ __device__ constexpr int join_prefetch(int dt, int nk, int w) { return nk <= 4 || (w == 1 && dt == 1) ? nk : nk == 6 ? 3 : 4; }

// Steps whose row operand lies in LDS: 32 steps leave no registers for the last ones, and a reload from scratch memory in the
// loop over the groups waits for the next group's loads as well (a lone query over 300,000 x 960 uint8: 515 -> 415 us).
__host__ __device__ constexpr int join_lds_steps(int nk) { return nk == 32 ? 2 : 0; }

// LDS buffers of one group of nc chunks: two where they leave room for other workgroups on the CU
__host__ __device__ constexpr int join_buffers(int nc) { return nc <= 32 ? 2 : 1; }

template <int DT, int NK, int W> constexpr size_t join_lds_bytes()
{
    constexpr int NC = join_chunks<DT>(NK);
    return (size_t)(W > 1 ? join_buffers(NC) * NC * 512 + 16 : 0) + (size_t)W * (join_wave_lds(W) + join_lds_steps(NK) * 1024);
}

// NK: contraction steps (16 components of float32, 32 of uint8), the vectors zero padded to them.  W: waves of a workgroup,
// 32 rows each.  Four share the list's groups through LDS; one reads them by itself.
template <int DT, int NK, bool AND, int W>
__global__ __launch_bounds__(64 * W, join_waves(DT, NK, W)) void join_kernel(JoinParams p)
{
    extern __shared__ uint4 smem[];
    using acc_t = typename JoinAcc<DT>::type;
    using val_t = typename JoinAcc<DT>::scalar;
    typedef val_t val4_t __attribute__((ext_vector_type(4)));
    constexpr int NC = join_chunks<DT>(NK), NPRE = join_prefetch(DT, NK, W), STAGE = NC * 32;
    static_assert(NK % NPRE == 0, "whole requests");
    constexpr int NBUF = W > 1 ? join_buffers(NC) : 0, NL = (STAGE + 64 * W - 1) / (64 * W);
    const ScanItem it = p.items[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, n32 = lane & 31, h = lane >> 5;
    const int wave = W > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int K = p.K, row_base = wave * 32;
    const int rows = it.q_count - row_base < 32 ? it.q_count - row_base : 32;   // rows of this wave (<= 0: none)
    constexpr int kJoinFlat = join_flat(W), kJoinWaveLds = join_wave_lds(W);
    static_assert(kJoinWaveLds % 16 == 0, "alignment");
    uint64_t *pend = (uint64_t *)((char *)(smem + NBUF * STAGE) + wave * kJoinWaveLds);   // [32 rows][kJoinQueue]
    uint64_t *flat = pend + 32 * kJoinQueue;                   // (v << 32 | entry) of a candidate
    int *pending = (int *)(flat + kJoinFlat);                  // [32] keys in the rows' queues (may count past their ends)
    val_t *tvs = (val_t *)(pending + 32);                      // [32] the rows' thresholds: read per group, they would be 16 registers
    uint8_t *flat_row = (uint8_t *)(tvs + 32);                 // a candidate's row; kTaken: gone to the row's queue, or not wanted
    int *want = (int *)((char *)(smem + NBUF * STAGE) + W * kJoinWaveLds);   // [3], the groups' in turn: a wave wants to deliver
    constexpr int NR = NK - join_lds_steps(NK);                // steps whose row operand is in registers
    uint4 *late = (uint4 *)((char *)(smem + NBUF * STAGE) + W * kJoinWaveLds + 16) + wave * (NK - NR) * 64;   // [NK - NR][64 lanes]
    constexpr uint32_t kTaken = 255;
    int flat_n = 0;

    // ---- the rows' operand (lane (n32, h): chunk 2 s + h of row n32) and squared norms
    int qr = -1, self = -1;   // row n32's vector, and the entry of the list that is the row itself
    if (n32 < rows) {
        int at = it.q_begin + row_base + n32;
        if (p.sel != nullptr) at = p.sel[at];
        qr = p.qrow[at];
        if (it.self_base >= 0) self = p.sel != nullptr ? at - it.self_base : it.self_base + row_base + n32;
    }
    uint4 a[NR], alo[DT == 1 ? NK : 1];
    val_t qnorm = 0;
    {
        const char *qp = (const char *)p.qsrc + (int64_t)(qr >= 0 ? qr : 0) * (p.dim * (DT == 0 ? 1 : 4));
#pragma unroll
        for (int s = 0; s < NK; ++s) {
            const int c = 2 * s + h;
            if constexpr (DT == 0) {
                uint4 v = make_uint4(0, 0, 0, 0);
                if (qr >= 0 && c * 16 < p.dim) {
                    v = *(const uint4 *)(qp + c * 16);
                    v.x ^= 0x80808080u; v.y ^= 0x80808080u; v.z ^= 0x80808080u; v.w ^= 0x80808080u;
                }
                if (s < NR) a[s < NR ? s : 0] = v;
                else late[(s - NR) * 64 + lane] = v;   // (each lane reads its own)
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) qnorm = __builtin_amdgcn_sdot4((int)w[i], (int)w[i], qnorm, false);
            } else {
                float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
                if (qr >= 0 && c * 8 < p.dim) x = centred(*(const float4 *)(qp + c * 32), p.centre, 2 * c);
                if (qr >= 0 && c * 8 + 4 < p.dim) y = centred(*(const float4 *)(qp + c * 32 + 16), p.centre, 2 * c + 1);
                float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
                if constexpr (DT == 1) {
                    split_bf16x8(f, a[s], alo[s]);
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] *= p.scale;
                    a[s] = half8(f);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) qnorm += f[i] * f[i];
            }
        }
        qnorm += __shfl_xor(qnorm, 32);
    }

    // ---- state of row r, held by lane r < 32: keys waiting, K-th best key, threshold on v (rows that do not exist: never)
    const val_t never = DT == 0 ? (val_t)0x7FFFFFFF : (val_t)__builtin_inff();
    val_t tv = n32 < rows ? (DT == 0 ? (val_t)(-0x20000000) : (val_t)(-3.0e38f)) : never;
    int pcv = 0;
    uint64_t row_kth = KEY_MAX;
    uint32_t touched = 0;            // rows whose partial result row has been written
    // threshold of a row whose K-th distance (of any segment of its list) has the bits kd
    auto threshold = [&](uint32_t kd) -> val_t {
        if constexpr (DT == 0) return qnorm - (int)kd;
        // (lowered by a few units in the last place: a pair that is left out has an approximation of at least the K-th best)
        else return 0.5f * (qnorm - __uint_as_float(kd)) - 2.4e-7f * (qnorm + __uint_as_float(kd));
    };
    uint32_t *bound = p.bound != nullptr ? p.bound + (it.q_begin - p.bound_row0) + row_base : nullptr;
    const val_t first = DT == 0 ? (val_t)(-0x20000000) : (val_t)(-3.0e38f);   // every entry passes
    val_t start = first;
    const bool filtered = AND && qr >= 0 && p.others_off[qr + 1] > p.others_off[qr];   // (its sample says nothing about those that pass)
    if (bound != nullptr && n32 < rows) {
        const uint32_t kd = __hip_atomic_load(bound + n32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (kd != 0xFFFFFFFFu) tv = threshold(kd);
    }
    const int64_t part0 = (int64_t)it.part_row + row_base;
    if (h == 0) tvs[n32] = tv;
    if (h == 0) pending[n32] = 0;
    wave_lds_sync();
    // Merge the queues of the rows in `todo` into their K best, four rows at a time, and empty them.
    auto drain = [&](uint32_t todo) {
        wave_lds_sync();
        const uint32_t done = todo;
        int r_next[4];
        bool on_next[4];
        uint64_t best_next[4];
        auto pick = [&]() {   // the next four rows, their K best requested while the last four are merged
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                on_next[u] = todo != 0;
                r_next[u] = on_next[u] ? __builtin_ctz(todo) : 0;
                todo &= todo - 1;
                best_next[u] = KEY_MAX;
                if (on_next[u] && ((touched >> r_next[u]) & 1u) && lane < K) {
                    const int64_t o = (part0 + r_next[u]) * K + lane;
                    const int32_t idx = p.res_idx[o];
                    if (idx >= 0) best_next[u] = ((uint64_t)p.res_bits[o] << 32) | (uint32_t)idx;
                }
            }
        };
        pick();
        while (on_next[0]) {
            int r[4];
            bool on[4];
            uint64_t best[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { r[u] = r_next[u]; on[u] = on_next[u]; best[u] = best_next[u]; }
            pick();
            // the four queues in the wave's quarters, each sorted descending, then in the last quarter behind KEY_MAX:
            // against the ascending best, that makes the smallest 64 of both a bitonic sequence
            static_assert(kJoinQueue == 16, "a quarter of the lanes");
            const int quarter = lane >> 4, ls = lane & 15;
            const int rq = quarter < 2 ? (quarter == 0 ? r[0] : r[1]) : (quarter == 2 ? r[2] : r[3]);
            const int pc_q = __shfl(pcv, rq);
            const uint64_t kth_q = shfl64(row_kth, rq);
            const val_t qn_q = __shfl(qnorm, rq);
            uint64_t x[1] = {KEY_MAX};
            if (ls < pc_q) {   // v -> distance of the row
                const uint64_t key = pend[rq * kJoinQueue + ls];
                const uint32_t vb = (uint32_t)(key >> 32);
                const uint32_t bits = DT == 0 ? (uint32_t)((int)qn_q - (int)vb)
                                              : __float_as_uint(fmaxf((float)qn_q - 2.0f * __uint_as_float(vb), 0.0f));
                const uint64_t k = ((uint64_t)bits << 32) | (uint32_t)key;
                x[0] = k < kth_q ? k : KEY_MAX;
            }
            lane_sort<16, true>(x);
            uint64_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint64_t y = shfl64(x[0], 16 * u + ls), z = quarter == 3 ? y : KEY_MAX;
                v[u] = best[u] < z ? best[u] : z;
            }
            lane_merge<64>(v);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (on[u]) {   // wave-uniform
                    if (lane < K) {
                        const int64_t o = (part0 + r[u]) * K + lane;
                        p.res_idx[o] = v[u] == KEY_MAX ? -1 : (int32_t)(uint32_t)v[u];
                        p.res_bits[o] = (uint32_t)(v[u] >> 32);
                    }
                    const uint64_t nk = readlane64(v[u], K - 1);
                    if (lane == r[u]) row_kth = nk;
                }
            }
        }
        touched |= done;
        if ((done >> n32) & 1u) {
            if (h == 0) pending[n32] = 0;
            uint32_t kd = (uint32_t)(row_kth >> 32);
            if (bound != nullptr) {
                // what the other segments' workgroups know of the row: no segment needs what is above any one's K-th best
                if (row_kth != KEY_MAX && h == 0) atomicMin(bound + n32, kd);
                const uint32_t b = __hip_atomic_load(bound + n32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                kd = row_kth != KEY_MAX && kd < b ? kd : b;
                if (kd != 0xFFFFFFFFu) tv = threshold(kd);
            } else if (row_kth != KEY_MAX) tv = threshold(kd);
        }
        if (h == 0) tvs[n32] = tv;
        wave_lds_sync();
    };
    // The collected candidates to their rows' queues, 64 at a time, less those that are the row itself or fail the
    // predicate; then the queues that are half full (last: all) are merged.  Where a queue is too short for what it is
    // sent (before thresholds exist), the rest follows after the merge.
    auto deliver = [&](bool last) {
        while (true) {
            wave_lds_sync();
            bool over = false;
            for (int i0 = 0; i0 < flat_n; i0 += 64) {
                const int i = i0 + lane;
                const uint32_t row = i < flat_n ? flat_row[i] : kTaken;
                const uint64_t key = i < flat_n ? flat[i] : 0;
                const int entry = (int)(uint32_t)key;
                const int row_self = __shfl(self, (int)row & 31);   // (outside any condition: the source lane has to be active)
                bool ok = row != kTaken && entry != row_self;
                if constexpr (AND) {
                    const int q = __shfl(qr, (int)row & 31);
                    if (ok) {
                        const int o_begin = p.others_off[q], o_end = p.others_off[q + 1];
                        if (o_begin < o_end) {
                            const int gid = p.map[it.map_off + entry];
                            for (int o = o_begin; o < o_end && ok; ++o) ok = has_label(p.meta, p.others[o], gid);
                        }
                    }
                }
                const int slot = ok ? atomicAdd(&pending[row], 1) : 0;
                const bool fits = slot < kJoinQueue;
                if (ok && fits) pend[row * kJoinQueue + slot] = key;
                if (row != kTaken && fits) flat_row[i] = (uint8_t)kTaken;
                over = over || !fits;
            }
            wave_lds_sync();
            const int n = pending[n32];
            pcv = n < kJoinQueue ? n : kJoinQueue;
            const bool again = __any(over);
            const uint32_t todo = (uint32_t)__ballot(lane < 32 && pcv >= (last && !again ? 1 : kJoinMerge));
            if (todo != 0) drain(todo);
            if (!again) break;
        }
        flat_n = 0;
    };

    // ---- the list's groups: the next one is on its way while one is worked on
    const int n_groups = (it.n + kGroup - 1) / kGroup;
    const v4u_join *blk = (const v4u_join *)p.xblk + it.group0 * (int64_t)STAGE;
    const val_t *xnorm = (const val_t *)p.xnorm + it.group0 * kGroup + n32;
    v4u_join b[NPRE * (DT == 1 ? 2 : 1)];   // (split operands: high parts, then low parts)
    v4u_join pre[W > 1 ? NL : 1];           // (the native vector type: an array of uint4 ends up in scratch memory here)
    val_t xn_next;
    auto load_b = [&](const v4u_join *src) {   // chunks of NPRE steps, lane (n32, h): chunk 2 s + h of entry n32
#pragma unroll
        for (int u = 0; u < NPRE; ++u) {
            b[u] = src[u * 64 + h * 32 + n32];
            if constexpr (DT == 1) b[NPRE + u] = src[(NK + u) * 64 + h * 32 + n32];
        }
    };
    auto fetch = [&](int g) {   // W > 1: this thread's part of a group
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (STAGE % (64 * W) == 0 || tid + i * 64 * W < STAGE) pre[W > 1 ? i : 0] = blk[(int64_t)g * STAGE + tid + i * 64 * W];
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (STAGE % (64 * W) == 0 || tid + i * 64 * W < STAGE) ((v4u_join *)smem)[buf * STAGE + tid + i * 64 * W] = pre[W > 1 ? i : 0];
    };
    auto begin = [&]() {
        if constexpr (W > 1) {
            fetch(0);
            put(0);
            __syncthreads();
        } else {
            load_b(blk);
        }
        xn_next = xnorm[0];
    };
    // the contraction of group g, and what comes after it set on its way
    acc_t qx;   // q.x of the lane's 16 pairs
    val_t xn;   // |x|^2 / 2 of its entry (uint8: |x|^2)
    auto contract = [&](int g) {
        const int gn = g + 1 < n_groups ? g + 1 : g;   // (the last one is read twice)
        xn = xn_next;
        if constexpr (W > 1) fetch(gn);
        xn_next = xnorm[gn * kGroup];
        if (W > 1 && rows <= 0) return;
        const v4u_join *B = (const v4u_join *)smem + (NBUF == 2 ? (g & 1) : 0) * STAGE;
        acc_t acc, acc_lo;   // (split operands: the products with a low part by themselves, so that their sums stay small)
#pragma unroll
        for (int j = 0; j < 16; ++j) { acc[j] = 0; acc_lo[j] = 0; }
#pragma unroll
        for (int s0 = 0; s0 < NK; s0 += NPRE) {
            if constexpr (W > 1) {
                load_b(B + s0 * 64);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (DT == 0) {
#pragma unroll
                for (int u = 0; u < NPRE; ++u) {
                    const uint4 ar = s0 + u < NR ? a[s0 + u < NR ? s0 + u : 0] : late[(s0 + u - NR) * 64 + lane];
                    const v4i_join av = {(int)ar.x, (int)ar.y, (int)ar.z, (int)ar.w};
                    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, __builtin_bit_cast(v4i_join, b[u]), acc, 0, 0, 0);
                }
            } else if constexpr (DT == 2) {
#pragma unroll
                for (int u = 0; u < NPRE; ++u)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h_join, a[s0 + u]), __builtin_bit_cast(v8h_join, b[u]), acc, 0, 0, 0);
            } else {
#pragma unroll
                for (int u = 0; u < NPRE; ++u) {
                    const v8bf_join bh = __builtin_bit_cast(v8bf_join, b[u]), bl = __builtin_bit_cast(v8bf_join, b[NPRE + u]);
                    acc_lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, alo[s0 + u]), bh, acc_lo, 0, 0, 0);
                    acc_lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, a[s0 + u]), bl, acc_lo, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, a[s0 + u]), bh, acc, 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (W == 1) {   // the chunks that follow, as soon as the matrix cores have taken these
                if (s0 + NPRE < NK) load_b(blk + (int64_t)g * STAGE + (s0 + NPRE) * 64);
                else load_b(blk + (int64_t)gn * STAGE);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) qx[j] = DT == 1 ? acc_lo[j] + acc[j] : acc[j];
    };
    auto value = [&](int j) -> val_t { return DT == 0 ? qx[j] * 2 - xn : qx[j] - xn; };
    auto advance = [&](int g) {   // W > 1: the group after g into LDS
        if constexpr (W > 1) {
            if (NBUF == 1) __syncthreads();
            put(NBUF == 2 ? (g + 1) & 1 : 0);
            __syncthreads();
        }
    };

    // ---- first thresholds: every lane's largest v of the even and of the odd groups of a sample; a row's K-th largest of
    // those 64 (K + 1 where the row itself may be among them) has K entries at or above it.  Without this a row's first
    // thousand entries make a queue's worth of candidates every few groups.  The sample's values are q.x - |x|^2 / 2 rounded, and the
    // groups are compared as q.x - t rounded, which never leaves out an entry whose unrounded value is at least t: so a
    // float32 threshold is the sample's value less a few units in its last place, and all K entries pass (copies of one
    // vector, that is, all of them or none).
    const int rank = K - (it.self_base >= 0 ? 0 : 1);
    const int most = it.q_count * K < kJoinFew ? kJoinSampleFew : kJoinSample;
    const int sample = n_groups / 2 < most ? n_groups / 2 : most;
    if (sample >= 8 && rank < 64 && (W > 1 || __any(n32 < rows && !filtered && !(tv > first)))) {
        val_t top[2][16];
#pragma unroll
        for (int j = 0; j < 16; ++j) top[0][j] = top[1][j] = first;
        begin();
        for (int g = 0; g < sample; g += 2) {
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                contract(g + o);
                if (W == 1 || rows > 0)
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const val_t v = value(j);
                        top[o][j] = v > top[o][j] ? v : top[o][j];
                    }
                advance(g + o);
            }
        }
        if (W == 1 || rows > 0) {
#pragma unroll
            for (int j0 = 0; j0 < 16; j0 += 4) {
                val_t up[4], down[4], kth[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) { up[u] = top[0][j0 + u]; down[u] = top[1][j0 + u]; }
                lane_sort<32, false>(up);
                lane_sort<32, true>(down);
                // (ascending against descending: the larger ones of the pairs are the 32 largest)
#pragma unroll
                for (int u = 0; u < 4; ++u) kth[u] = (rank < 32) == (up[u] > down[u]) ? up[u] : down[u];
                lane_merge<32>(kth);
                // ascending within a half: the r-th largest of 32 is at lane 31 - r
                const int at = rank < 32 ? 31 - rank : 63 - rank;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u, r0 = 8 * (j >> 2) + (j & 3);
                    const val_t k0 = __shfl(kth[u], at), k1 = __shfl(kth[u], 32 + at);
                    if (n32 == r0) start = k0;
                    if (n32 == r0 + 4) start = k1;
                }
            }
            if constexpr (DT != 0) start -= 2.4e-7f * __builtin_fabsf(start);   // (four halves of a unit; differences below the normal range are exact)
            if (n32 < rows && !filtered && start > tv) tv = start;
            if (h == 0) tvs[n32] = tv;
            wave_lds_sync();
        }
    }

    // ---- the groups against the thresholds
    if (W > 1 && tid < 3) want[tid] = 0;
    begin();
    for (int g = 0, turn = 0; g < n_groups; ++g, turn = turn < 2 ? turn + 1 : 0) {
        contract(g);
        if (W > 1 && rows <= 0) {
            advance(g);
            continue;
        }
        val_t t[16];   // element j: row 8 (j / 4) + 4 h + j % 4
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const val4_t t4 = ((const val4_t *)tvs)[2 * q + h];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[4 * q + u] = t4[u];
        }
        auto over = [&](int j) -> val_t { return DT == 0 ? qx[j] * 2 - t[j] : qx[j] - t[j]; };
        val_t most[4];   // of rows 8 q .. 8 q + 7
#pragma unroll
        for (int q = 0; q < 4; ++q) most[q] = larger(larger(larger(over(4 * q), over(4 * q + 1)), over(4 * q + 2)), over(4 * q + 3));
        const int entry = it.entry0 + g * kGroup + n32;   // list-relative
        auto append = [&](int j, uint64_t m) {
            const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)flat_n));
            if (__builtin_amdgcn_inverse_ballot_w64(m) && at < kJoinFlat) {   // (v for now: the drain makes a distance of it)
                const val_t v = value(j);
                flat[at] = ((uint64_t)(DT == 0 ? (uint32_t)v : __float_as_uint((float)v)) << 32) | (uint32_t)entry;
                int row = 4 * h;
                asm("" : "+v"(row));   // (else the sixteen rows' numbers are kept in as many registers)
                flat_row[at] = (uint8_t)(row + 8 * (j >> 2) + (j & 3));
            }
            flat_n += __builtin_popcountll(m);
        };
        int left = 16;   // elements from here on have not been looked at
        if (__builtin_amdgcn_ballot_w64(larger(larger(larger(most[0], most[1]), most[2]), most[3]) >= xn) != 0) {
            const int before = flat_n;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (__builtin_amdgcn_ballot_w64(most[q] >= xn) == 0) continue;   // (wave-uniform, as all that follows but the stores)
#pragma unroll
                for (int j = 4 * q; j < 4 * q + 4; ++j) {
                    const uint64_t m = __builtin_amdgcn_ballot_w64(over(j) >= xn);
                    if (m != 0) append(j, m);
                }
            }
            if (__builtin_expect(flat_n > kJoinFlat, 0)) {   // more than there is room for (before thresholds exist)
                flat_n = before;
                left = 0;
            }
        }
        bool now = flat_n >= kJoinFull || left < 16;
        if constexpr (W > 1) {
            // a wave that merges lets the others wait at the barrier: they merge together
            // (the next group's word was last read two barriers ago, and is not written before the one to come)
            if (now && lane == 0) want[turn] = 1;
            if (tid == 0) want[turn < 2 ? turn + 1 : 0] = 0;
            advance(g);
            now = want[turn] != 0;
        }
        if (now) {
            while (true) {
                deliver(false);
                if (__builtin_expect(left == 16, 1)) break;
#pragma unroll 1
                for (; left < 16; ++left) {
                    const val_t tj = tvs[8 * (left >> 2) + 4 * h + (left & 3)];
                    const uint64_t m = __builtin_amdgcn_ballot_w64((DT == 0 ? qx[left] * 2 - tj : qx[left] - tj) >= xn);
                    if (flat_n + __builtin_popcountll(m) > kJoinFlat) break;
                    if (m != 0) append(left, m);
                }
                if (left == 16 && flat_n < kJoinFull) break;
            }
        }
    }
    deliver(true);
    for (int r = 0; r < rows; ++r)   // rows without a candidate
        if (((touched >> r) & 1u) == 0 && lane < K) {
            p.res_idx[(part0 + r) * K + lane] = -1;
            p.res_bits[(part0 + r) * K + lane] = 0xFFFFFFFFu;
        }
}

// One thread per (group, chunk, entry): the lists' vectors gathered through `map` in the layout the join reads (float32:
// 2 NK chunks of high parts, then 2 NK of low parts, of the centred vector), and per entry half its squared norm (uint8:
// the squared norm of the shifted bytes); an entry past the end of its list never passes a threshold.
template <int DT>
__global__ void join_pack_kernel(const char *X, int32_t dim, const int32_t *map, const JoinList *lists, int32_t n_lists,
                                 int64_t n_groups, int32_t nk, const uint32_t *norm_all, const float *centre, float scale, uint4 *xblk, uint32_t *xnorm,
                                 uint32_t *bound, int64_t n_bound)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t; i < n_bound; i += (int64_t)gridDim.x * blockDim.x) bound[i] = 0xFFFFFFFFu;   // of the join that follows
    const int nch = 2 * nk;
    if (t >= n_groups * nch * 32) return;
    const int v = (int)(t & 31);
    const int64_t gc = t >> 5;
    const int c = (int)(gc % nch);
    const int64_t g = gc / nch;
    int lo = 0, hi = n_lists - 1;   // the list of group g
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (lists[mid].group0 <= g) lo = mid; else hi = mid - 1;
    }
    const int64_t e = (g - lists[lo].group0) * 32 + v;
    const bool valid = e < lists[lo].n;
    const int64_t row = valid ? map[lists[lo].src + e] : 0;
    if (DT == 0) {
        uint4 w = make_uint4(0, 0, 0, 0);
        if (valid && c * 16 < dim) {
            w = *(const uint4 *)(X + row * dim + c * 16);
            w.x ^= 0x80808080u; w.y ^= 0x80808080u; w.z ^= 0x80808080u; w.w ^= 0x80808080u;
        }
        xblk[(g * nch + c) * 32 + v] = w;
        if (c == 0) xnorm[g * 32 + v] = valid ? norm_all[row] : 0x3FFFFFFFu;
    } else {
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
        if (valid && c * 8 < dim) x = centred(*(const float4 *)(X + row * dim * 4 + c * 32), centre, 2 * c);
        if (valid && c * 8 + 4 < dim) y = centred(*(const float4 *)(X + row * dim * 4 + c * 32 + 16), centre, 2 * c + 1);
        float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        if (DT == 1) {
            uint4 hi, lo;
            split_bf16x8(f, hi, lo);
            xblk[(g * 2 * nch + c) * 32 + v] = hi;
            xblk[(g * 2 * nch + nch + c) * 32 + v] = lo;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] *= scale;
            xblk[(g * nch + c) * 32 + v] = half8(f);
        }
        if (c == 0) xnorm[g * 32 + v] = valid ? __float_as_uint(0.5f * __uint_as_float(norm_all[row]) * (scale * scale)) : 0x7F800000u;
    }
}

// The centre: the mean of up to 4,096 rows spread over the table.  Any fixed vector would do, so a sample is enough; one
// pass over 2 MiB at dim 128 (16,384 rows took 23 us, which a build of 2.5 ms notices).  Block b takes every
// kCentreParts-th row of the sample, a thread four components of every rows_at_a_time-th of them.
constexpr int64_t kCentreRows = 4096;

__global__ __launch_bounds__(256) void centre_part_kernel(const float *X, int32_t dim, int64_t n, float *parts)
{
    __shared__ float4 sum[256];
    const int nch = dim / 4, rows_at_a_time = 256 / nch;   // (at most 62 chunks)
    const int c = threadIdx.x % nch, r = threadIdx.x / nch;
    const int64_t sample = n < kCentreRows ? n : kCentreRows;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < rows_at_a_time)
        for (int64_t i = blockIdx.x + (int64_t)r * kCentreParts; i < sample; i += (int64_t)rows_at_a_time * kCentreParts) {
            const float4 v = ((const float4 *)(X + i * n / sample * dim))[c];
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
        }
    sum[threadIdx.x] = a;
    __syncthreads();
    if (r == 0) {
        for (int o = 1; o < rows_at_a_time; ++o) {
            const float4 v = sum[o * nch + c];
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
        }
        ((float4 *)(parts + (int64_t)blockIdx.x * dim))[c] = a;
    }
}

__global__ __launch_bounds__(256) void centre_mean_kernel(const float *parts, int32_t dim, int64_t n, float *centre)
{
    const int e = threadIdx.x;
    if (e >= dim) return;
    float a = 0.f;
    for (int b = 0; b < kCentreParts; ++b) a += parts[b * dim + e];
    centre[e] = a / (float)(n < kCentreRows ? n : kCentreRows);
}

// x rounded to 11 significant bits, as binary16 does within its range
__device__ __forceinline__ float round_11_bits(float x)
{
    const uint32_t u = __float_as_uint(x);
    return __uint_as_float((u + 0xFFFu + ((u >> 13) & 1u)) & ~0x1FFFu);
}

// One thread per row, elements in ascending order (400,000 x 128: 0.32 ms).
__global__ __launch_bounds__(256) void row_norm_f32_kernel(const float *X, int32_t dim, int64_t n, const float *centre, uint32_t *out,
                                                           uint32_t *out_c, uint32_t *max_bits)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float acc = 0.f, acc_c = 0.f, acc_e = 0.f;
    if (i < n) {
        const float4 *x = (const float4 *)(X + i * dim);
        for (int c = 0; c < dim / 4; ++c) {
            const float4 v = x[c], w = centred(v, centre, c);
            acc += v.x * v.x; acc += v.y * v.y; acc += v.z * v.z; acc += v.w * v.w;
            acc_c += w.x * w.x; acc_c += w.y * w.y; acc_c += w.z * w.z; acc_c += w.w * w.w;
            const float4 e = make_float4(w.x - round_11_bits(w.x), w.y - round_11_bits(w.y), w.z - round_11_bits(w.z), w.w - round_11_bits(w.w));
            acc_e += e.x * e.x; acc_e += e.y * e.y; acc_e += e.z * e.z; acc_e += e.w * e.w;
        }
        out[i] = __float_as_uint(acc);
        out_c[i] = __float_as_uint(acc_c);
    }
    // (no norm is negative: their bits are ordered as they are, with NaN of either sign above infinity)
    uint32_t m = __float_as_uint(acc), m_c = __float_as_uint(acc_c), m_e = acc_c > 0.f ? __float_as_uint(acc_e / acc_c) : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t v = (uint32_t)__shfl_xor((int)m, o), w = (uint32_t)__shfl_xor((int)m_c, o), e = (uint32_t)__shfl_xor((int)m_e, o);
        m = v > m ? v : m;
        m_c = w > m_c ? w : m_c;
        m_e = e > m_e ? e : m_e;
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(max_bits, m);
        atomicMax(max_bits + 1, m_c);
        atomicMax(max_bits + 2, m_e);
    }
}

void launch_centre(const void *X, int32_t dim, int64_t n, float *tmp, float *centre, hipStream_t s)
{
    hipLaunchKernelGGL(centre_part_kernel, dim3(kCentreParts), dim3(256), 0, s, (const float *)X, dim, n, tmp);
    hipLaunchKernelGGL(centre_mean_kernel, dim3(1), dim3(256), 0, s, (const float *)tmp, dim, n, centre);
}

void launch_row_norms_f32(const void *X, int32_t dim, int64_t n, const float *centre, uint32_t *out, uint32_t *out_c, uint32_t *max_bits,
                          hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(row_norm_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const float *)X, dim, n, centre, out,
                       out_c, max_bits);
}

// Contraction steps the kernel is compiled for: the smallest that holds the vector.
static int32_t join_steps(int kind, int32_t dim)
{
    const int32_t need = kind == kJoinU8 ? (dim + 31) / 32 : (dim + 15) / 16;
    for (const int32_t nk : {2, 4, 6, 8, 16}) if (need <= nk) return nk;
    return kind == kJoinU8 && need <= 32 ? 32 : 0;
}

// Steps up to which queries' lists are read by one wave each, however many rows there are: 5,000 / 50,000 queries of a list of
// 150,000 x 128 float32 1.03 / 4.86 ms, by workgroups of four waves 1.20 / 5.82 (20,000 entries 0.34 / 1.44 and 0.48 / 1.62; uint8
// x 256, 30,000 queries 2.39 and 2.85).  Beyond them a group is 16 KB and more, and four waves that load a quarter each are ahead
// for any number of rows, a single one included (a lone query and 100 over a list of 300,000: uint8 of 512 components 400 / 425 us
// by one wave, 288 / 356 by four; float32 of 248, split 866 / 1,017 and 705 / 1,001).
constexpr int32_t kJoinAloneSteps = 8;

int join_tile_rows(int kind, int32_t dim) { return join_steps(kind, dim) > kJoinAloneSteps ? kJoinRowsShared : kJoinRows; }

size_t join_group_bytes(int kind, int32_t dim)
{
    const int32_t nk = join_steps(kind, dim);
    return (size_t)(kind == kJoinSplit ? join_chunks<1>(nk) : join_chunks<0>(nk)) * 512;
}

void launch_join_pack(int kind, const void *X, int32_t dim, const int32_t *map, const JoinList *lists, int n_lists,
                      int64_t n_groups, const uint32_t *norm_all, const float *centre, float scale, uint4 *xblk, void *xnorm,
                      uint32_t *bound, int64_t n_bound, hipStream_t s)
{
    if (n_groups <= 0) return;
    const int32_t nk = join_steps(kind, dim);
    const dim3 blocks((unsigned)((n_groups * 2 * nk * 32 + 255) / 256)), threads(256);
#define VF_LAUNCH_PACK(DT_) \
    hipLaunchKernelGGL(join_pack_kernel<DT_>, blocks, threads, 0, s, (const char *)X, dim, map, lists, n_lists, n_groups, nk, norm_all, \
                       centre, scale, xblk, (uint32_t *)xnorm, bound, n_bound)
    if (kind == kJoinU8) VF_LAUNCH_PACK(0);
    else if (kind == kJoinSplit) VF_LAUNCH_PACK(1);
    else VF_LAUNCH_PACK(2);
#undef VF_LAUNCH_PACK
}

template <int DT, int NK, int W> static void launch_join_w(const JoinParams &p, int n_items, hipStream_t s)
{
    constexpr size_t lds = join_lds_bytes<DT, NK, W>();
    if constexpr (W == 1 || NK > kJoinAloneSteps) {   // (only queries have predicates)
        if (p.others_off != nullptr) {
            hipLaunchKernelGGL((join_kernel<DT, NK, true, W>), dim3(n_items), dim3(64 * W), lds, s, p);
            return;
        }
    }
    hipLaunchKernelGGL((join_kernel<DT, NK, false, W>), dim3(n_items), dim3(64 * W), lds, s, p);
}

template <int DT, int NK> static void launch_join_nk(const JoinParams &p, int rows, int n_items, hipStream_t s)
{
    if constexpr (NK <= kJoinAloneSteps) {
        if (rows <= kJoinRows) return launch_join_w<DT, NK, 1>(p, n_items, s);
    }
    launch_join_w<DT, NK, kJoinRowsShared / kJoinRows>(p, n_items, s);
}

template <int DT> static void launch_join_f32(const JoinParams &p, int32_t nk, int rows, int n_items, hipStream_t s)
{
    switch (nk) {
    case 2: launch_join_nk<DT, 2>(p, rows, n_items, s); break;
    case 4: launch_join_nk<DT, 4>(p, rows, n_items, s); break;
    case 6: launch_join_nk<DT, 6>(p, rows, n_items, s); break;
    case 8: launch_join_nk<DT, 8>(p, rows, n_items, s); break;
    default: launch_join_nk<DT, 16>(p, rows, n_items, s); break;
    }
}

void launch_join(int kind, const JoinParams &p, int rows, int n_items, hipStream_t s)
{
    if (n_items <= 0) return;
    const int32_t nk = join_steps(kind, p.dim);
    if (kind == kJoinSplit) return launch_join_f32<1>(p, nk, rows, n_items, s);
    if (kind == kJoinSingle) return launch_join_f32<2>(p, nk, rows, n_items, s);
    switch (nk) {
    case 2: launch_join_nk<0, 2>(p, rows, n_items, s); break;
    case 4: launch_join_nk<0, 4>(p, rows, n_items, s); break;
    case 6: launch_join_nk<0, 6>(p, rows, n_items, s); break;
    case 8: launch_join_nk<0, 8>(p, rows, n_items, s); break;
    case 16: launch_join_nk<0, 16>(p, rows, n_items, s); break;
    default: launch_join_nk<0, 32>(p, rows, n_items, s); break;
    }
}

}  // namespace vf
