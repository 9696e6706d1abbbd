// Contraction of many rows against whole lists with the exact top-K selection fused in: the kNN self-joins of the index
// build (Alg. 1) and the scans of graph lists for the exact ground truth.  Where the scan kernels serve a handful of
// queries per list and are bound by the list's bytes, a join has as many rows as it has and is bound by the matrix cores
// and by the selection, so everything here is arranged around those two.
//
// Tile.  A workgroup of four waves takes 128 rows (32 per wave) and streams a segment of a list through LDS, one group
// of 32 entries per step, shared by its waves: a group is fetched from L2 once per 128 rows instead of once per 16 (the
// 16-row kernel's 16 KiB per group and 16 rows would need more L2 bandwidth than there is at this rate).  The rows'
// operand stays in registers; where those do not suffice a part of it is in scratch memory (float32 of more than 128
// components 82 registers' worth, with the predicate 118, and 24 from 100 components on; uint8 of more than 512 25 and 69):
// 100,000 x 236 float32 vectors still build in 25 ms, on the 32-row scan kernel in 115.  Lists come packed
// (join_pack_kernel): per group the 16-byte chunks chunk-major, which is the B operand of the 32-column MFMAs, lane
// (n32, h) reading chunk 2 s + h of entry n32.
//
// float32 data: v_mfma_f32_32x32x16_bf16 on two-part splits of both operands, x = hi + lo with hi = bf16(x), lo =
// bf16(x - hi), after subtraction of a vector near the table's mean: distances stay what they are, and what the norms
// and products lose is relative to the spread of the data instead of to its distance from the origin (100,000 x 128,
// unit noise, shifted by 20 per coordinate: without it most rows are refused a proof, build 77 ms, 3,000 queries' ground
// truth 5.5 ms; with it 12.5 ms and 1.25 ms, as without the shift).  The products lo.hi and hi.lo first, then hi.hi, into one float32 accumulator (in this order the small
// terms are summed while the partial sums are small).  Three products at 16 times the rate of the float32 MFMA.  What
// they leave out, with u = 2^-24: |x - hi - lo| <= 2^-18 |x| twice and the product of the low parts 2^-18, together
// 192 u |q||x| in q.x, 193 u (|q|^2 + |x|^2) in the distance; the sums of the high parts 2 u per term; norms, summed one
// after the other, u per term; the subtraction of the centre, u per component, 4 u (|q|^2 + |x|^2) in the distance; final
// additions, the thresholds' and the ordered distance's own rounding < 100 u: 300 u + 3 u per component in all.  The
// bound used is 512 u + 4 u per component = join_err_bound(); callers re-rank what the join keeps with the ordered
// distance and prove with that bound that nothing else belongs to the result.
// uint8 data: v_mfma_i32_32x32x32_i8 on the bytes shifted by -128: exact.
//
// Selection.  With v = q.x - |x|^2 / 2 (uint8: 2 q.x - |x|^2) a distance is below a row's threshold where v is at least
// a per-row constant, one subtraction and one compare per pair; the compares' lane masks are or-ed on the scalar unit,
// and a group without a candidate (most, once the thresholds have tightened) is done.  Otherwise candidates go to the
// rows' queues in LDS (32 slots; positions by population counts of the masks, no atomics), and full queues are merged
// into the rows' sorted K best: two rows share a 64-lane sort network, then one merge network per row.  The K best live
// in the partial result rows in global memory: a row is drained about 15 times, so LDS is better spent on a second
// workgroup per CU.
//
// Measured, self-joins of 36 lists of 4,000 to 170,000 float32 vectors, dim 128 (4.7e10 pairs): 59 ms; the 16-row kernel
// on the float32 MFMA, one launch per list and 4 MiB panel, 167 ms.  The matrix cores are busy for 15 ms of it; the
// streaming alone (no candidates) takes 32 ms, whether the lists come from L2 or from memory: two waves per SIMD and a
// barrier per group; the rest is the selection.
#include "vf_select.h"

namespace vf {

typedef __bf16 v8bf_join __attribute__((ext_vector_type(8)));
typedef float v16f_join __attribute__((ext_vector_type(16)));
typedef int v16i_join __attribute__((ext_vector_type(16)));
typedef int v4i_join __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_join __attribute__((ext_vector_type(4)));

// LDS buffers of one group of nc chunks: two where both fit beside the queues in 64 KiB
__host__ __device__ constexpr int join_buffers(int nc) { return nc <= 32 ? 2 : 1; }

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

// ---------------------------------------------------------------- sorting networks over the lanes of a wave
//
// Bitonic networks over 64-bit keys held one per lane, every cross-lane move on the vector ALU: lane ^ 1, 2, 4, 8 are
// DPP moves (xor 4 = the mirror of 8 lanes, then the mirror of 4), lane ^ 16 and ^ 32 the row swaps of gfx950, which
// leave both partners' keys in both lanes.  Which lanes keep the smaller key of a stage is a constant, so a stage is two
// moves, one compare, one scalar xor of its result with that constant, and two selects; through ds_bpermute (the usual
// shuffle) it is two LDS accesses and twice the selects.  They pay where several sets run at a time, as here; a lone
// chain waits for every stage's trip through the scalar unit (in the beam search: a lone query 92 -> 97 us), so the
// search kernels keep the shuffles.

// Lanes that keep the smaller key when keys at distance J are compared inside ascending (descending: DESC) blocks of K.
template <int K, int J, bool LAST, bool DESC> __host__ __device__ constexpr uint64_t keep_min_lanes()
{
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l) {
        const bool up = (LAST || (l & K) == 0) != DESC;
        if (((l & J) == 0) == up) m |= 1ull << l;
    }
    return m;
}

// a, b: the keys of a lane and of its partner at lane ^ J (J = 1, 2, 4, 8: a is the lane's own key; J = 16, 32: a is
// the key of the partner whose bit J is clear, in both lanes)
template <int J> __device__ __forceinline__ void lane_pair(uint32_t v, uint32_t &a, uint32_t &b)
{
    static_assert(J == 1 || J == 2 || J == 4 || J == 8 || J == 16 || J == 32, "J is a power of two below 64");
    if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = r[0]; b = r[1];
    } else if constexpr (J == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = r[0]; b = r[1];
    } else {
        a = v;
        if constexpr (J == 1) b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);        // quad_perm [1,0,3,2]
        else if constexpr (J == 2) b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
        else if constexpr (J == 8) b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);  // row_ror:8
        else {
            const int m = __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);                         // row_half_mirror
            b = (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xF, 0xF, true);                               // quad_perm [3,2,1,0]
        }
    }
}

// One compare-exchange stage: the lanes of MIN keep the smaller key of the pair (lane, lane ^ J), the others the larger.
template <int J, uint64_t MIN> __device__ __forceinline__ uint64_t lane_exchange(uint64_t v)
{
    uint32_t al, bl, ah, bh;
    lane_pair<J>((uint32_t)v, al, bl);
    lane_pair<J>((uint32_t)(v >> 32), ah, bh);
    const uint64_t a = ((uint64_t)ah << 32) | al, b = ((uint64_t)bh << 32) | bl;
    return __builtin_amdgcn_inverse_ballot_w64(__builtin_amdgcn_ballot_w64(a < b) ^ ~MIN) ? a : b;
}

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

constexpr int kJoinQueue = 32;   // pending keys per row: what one group can add

template <int DT> struct JoinAcc { using type = v16f_join; using scalar = float; };
template <> struct JoinAcc<0> { using type = v16i_join; using scalar = int; };

template <int DT> __host__ __device__ constexpr int join_chunks(int nk) { return DT == 0 ? 2 * nk : 4 * nk; }

// v of lane `lane` (a constant) := x (wave-uniform)
__device__ __forceinline__ void set_lane(int &v, int x, int lane)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(x), "n"(lane));
}

// NK: contraction steps (16 components of float32, 32 of uint8), the vectors zero padded to them.
template <int DT, int NK, bool AND>
__global__ __launch_bounds__(256, 2) void join_kernel(JoinParams p)
{
    extern __shared__ uint4 smem[];
    using acc_t = typename JoinAcc<DT>::type;
    using val_t = typename JoinAcc<DT>::scalar;
    constexpr int NC = join_chunks<DT>(NK), STAGE = NC * 32, NL = (STAGE + 255) / 256;
    constexpr int NBUF = join_buffers(NC);
    const ScanItem it = p.items[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, n32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = p.K, row_base = wave * 32;
    const int rows = it.q_count - row_base < 32 ? it.q_count - row_base : 32;   // rows of this wave (<= 0: none)
    uint64_t *pend = (uint64_t *)(smem + NBUF * STAGE) + row_base * kJoinQueue;   // [32 rows][32]

    // ---- the rows' operand (lane (n32, h): chunk 2 s + h of row n32) and squared norms
    const int qr = n32 < rows ? p.qrow[it.q_begin + row_base + n32] : -1;
    uint4 a[NK], alo[DT == 0 ? 1 : NK];
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
                a[s] = v;
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) qnorm = __builtin_amdgcn_sdot4((int)w[i], (int)w[i], qnorm, false);
            } else {
                float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
                if (qr >= 0 && c * 8 < p.dim) x = centred(*(const float4 *)(qp + c * 32), p.centre, 2 * c);
                if (qr >= 0 && c * 8 + 4 < p.dim) y = centred(*(const float4 *)(qp + c * 32 + 16), p.centre, 2 * c + 1);
                const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
                split_bf16x8(f, a[s], alo[s]);
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
    const int64_t part0 = (int64_t)it.part_row + row_base;
    // per accumulator element: row 8 (j / 4) + 4 h + j % 4
    val_t t[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) t[j] = __shfl(tv, 8 * (j >> 2) + 4 * h + (j & 3));
    uint32_t and_rows = 0;
    int qr_of[AND ? 16 : 1];
    if constexpr (AND) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int r = 8 * (j >> 2) + 4 * h + (j & 3);
            qr_of[j] = __shfl(qr, r);
            if (qr_of[j] >= 0 && p.others_off[qr_of[j] + 1] > p.others_off[qr_of[j]]) and_rows |= 1u << j;
        }
    }

    auto qnorm_of = [&](int r) -> val_t {   // (wave-uniform r)
        if constexpr (DT == 0) return __builtin_amdgcn_readlane(qnorm, r);
        else return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(qnorm), r));
    };
    // Merge the queues of the rows in `todo` into their K best, four rows at a time, and empty them.
    auto drain = [&](uint32_t todo) {
        wave_lds_sync();
        const uint32_t done = todo;
        while (todo != 0) {
            int r[4];
            bool on[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                on[u] = todo != 0;
                r[u] = on[u] ? __builtin_ctz(todo) : r[0];
                todo &= todo - 1;
            }
            uint64_t best[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                best[u] = KEY_MAX;
                if (((touched >> r[u]) & 1u) && lane < K) {
                    const int64_t o = (part0 + r[u]) * K + lane;
                    const int32_t idx = p.res_idx[o];
                    if (idx >= 0) best[u] = ((uint64_t)p.res_bits[o] << 32) | (uint32_t)idx;
                }
            }
            uint64_t x[2];   // rows r[2u] and r[2u + 1] in the wave's halves
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int c0 = __builtin_amdgcn_readlane(pcv, r[2 * u]), c1 = __builtin_amdgcn_readlane(pcv, r[2 * u + 1]);
                const uint64_t k0 = readlane64(row_kth, r[2 * u]), k1 = readlane64(row_kth, r[2 * u + 1]);
                uint64_t key = n32 < (h ? c1 : c0) ? pend[(h ? r[2 * u + 1] : r[2 * u]) * kJoinQueue + n32] : KEY_MAX;
                if (key != KEY_MAX) {   // v -> distance of the row
                    const val_t q0 = qnorm_of(r[2 * u]), q1 = qnorm_of(r[2 * u + 1]), q = h ? q1 : q0;
                    const uint32_t vb = (uint32_t)(key >> 32);
                    const uint32_t bits = DT == 0 ? (uint32_t)((int)q - (int)vb)
                                                  : __float_as_uint(fmaxf((float)q - 2.0f * __uint_as_float(vb), 0.0f));
                    key = ((uint64_t)bits << 32) | (uint32_t)key;
                }
                x[u] = key < (h ? k1 : k0) ? key : KEY_MAX;
            }
            lane_sort<32, true>(x);
            uint64_t v[4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                // both halves' sorted keys in the upper lanes: descending behind KEY_MAX, against the ascending best
                uint32_t l0, l1, h0, h1;
                lane_pair<32>((uint32_t)x[u], l0, l1);
                lane_pair<32>((uint32_t)(x[u] >> 32), h0, h1);
                const uint64_t x0 = h ? ((uint64_t)h0 << 32) | l0 : KEY_MAX, x1 = h ? ((uint64_t)h1 << 32) | l1 : KEY_MAX;
                v[2 * u] = best[2 * u] < x0 ? best[2 * u] : x0;
                v[2 * u + 1] = best[2 * u + 1] < x1 ? best[2 * u + 1] : x1;
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
            if (h == 0) pcv = 0;
            if (row_kth != KEY_MAX) {
                const uint32_t kd = (uint32_t)(row_kth >> 32);
                if constexpr (DT == 0) tv = qnorm - (int)kd;
                // (lowered by a few units in the last place: a pair that is left out has an approximation of at least
                // the K-th best)
                else tv = 0.5f * (qnorm - __uint_as_float(kd)) - 2.4e-7f * (qnorm + __uint_as_float(kd));
            }
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) t[j] = __shfl(tv, 8 * (j >> 2) + 4 * h + (j & 3));
        wave_lds_sync();
    };

    // ---- stream the segment
    const int n_groups = (it.n + kGroup - 1) / kGroup;
    v4u_join pre[NL];   // (the native vector type: an array of uint4 ends up in scratch memory here)
    auto fetch = [&](int g) {
        const v4u_join *blk = (const v4u_join *)p.xblk + (it.group0 + g) * (int64_t)STAGE;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (STAGE % 256 == 0 || tid + i * 256 < STAGE) pre[i] = blk[tid + i * 256];
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            if (STAGE % 256 == 0 || tid + i * 256 < STAGE) ((v4u_join *)smem)[buf * STAGE + tid + i * 256] = pre[i];
    };
    const val_t *xnorm = (const val_t *)p.xnorm;
    fetch(0);
    val_t xn_next = xnorm[it.group0 * kGroup + n32];
    put(0);
    __syncthreads();
    for (int g = 0; g < n_groups; ++g) {
        const bool more = g + 1 < n_groups;
        const val_t xn = xn_next;
        if (more) {
            fetch(g + 1);
            xn_next = xnorm[(it.group0 + g + 1) * kGroup + n32];
        }
        if (rows > 0) {   // wave-uniform
            const uint4 *B = smem + (NBUF == 2 ? (g & 1) : 0) * STAGE;
            acc_t acc;
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = 0;
            // NPRE steps of the B operand at a time, requested before the first of them is used: left to itself the
            // compiler requests each chunk right before its MFMA and waits for the LDS every time
            constexpr int NPRE = NK < 8 ? NK : 8;
            if constexpr (DT == 0) {
#pragma unroll
                for (int s0 = 0; s0 < NK; s0 += NPRE) {
                    v4i_join b[NPRE];
#pragma unroll
                    for (int u = 0; u < NPRE; ++u) b[u] = ((const v4i_join *)B)[(2 * (s0 + u) + h) * 32 + n32];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < NPRE; ++u) {
                        const v4i_join av = {(int)a[s0 + u].x, (int)a[s0 + u].y, (int)a[s0 + u].z, (int)a[s0 + u].w};
                        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, b[u], acc, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int s0 = 0; s0 < NK; s0 += NPRE) {
                    v8bf_join bh[NPRE], bl[NPRE];
#pragma unroll
                    for (int u = 0; u < NPRE; ++u) {
                        bh[u] = ((const v8bf_join *)B)[(2 * (s0 + u) + h) * 32 + n32];
                        bl[u] = ((const v8bf_join *)B)[(2 * NK + 2 * (s0 + u) + h) * 32 + n32];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < NPRE; ++u) {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, alo[s0 + u]), bh[u], acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, a[s0 + u]), bl[u], acc, 0, 0, 0);
                    }
                    if (NK <= NPRE) {   // (all of it is still in registers)
#pragma unroll
                        for (int u = 0; u < NPRE; ++u)
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, a[s0 + u]), bh[u], acc, 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (NK > NPRE) {
#pragma unroll
                    for (int s0 = 0; s0 < NK; s0 += NPRE) {
                        v8bf_join bh[NPRE];
#pragma unroll
                        for (int u = 0; u < NPRE; ++u) bh[u] = ((const v8bf_join *)B)[(2 * (s0 + u) + h) * 32 + n32];
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < NPRE; ++u)
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_join, a[s0 + u]), bh[u], acc, 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            uint64_t m[16], any = 0;
            val_t v[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                v[j] = DT == 0 ? acc[j] * 2 - xn : acc[j] - xn;   // (float32: xn holds |x|^2 / 2)
                m[j] = __builtin_amdgcn_ballot_w64(v[j] >= t[j]);
                any |= m[j];
            }
            if (any != 0) {
                const int entry = it.entry0 + g * kGroup + n32;   // list-relative
                // graph build: the entry that is the row itself (self_base + row) is no candidate
                const int self = it.self_base >= 0 ? it.self_base + row_base : -0x40000000;
                if (self + 31 >= it.entry0 + g * kGroup && self <= it.entry0 + g * kGroup + 31) {
                    const int rel = entry - self - 4 * h;
#pragma unroll
                    for (int j = 0; j < 16; ++j) m[j] &= __builtin_amdgcn_ballot_w64(rel != 8 * (j >> 2) + (j & 3));
                }
                if constexpr (AND) {
                    const int gid = p.map[it.map_off + (g * kGroup + n32 < it.n ? entry : it.entry0)];
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        if (m[j] == 0) continue;
                        bool ok = (m[j] >> lane) & 1u;
                        if (ok && ((and_rows >> j) & 1u)) {
                            const int o_begin = p.others_off[qr_of[j]], o_end = p.others_off[qr_of[j] + 1];
                            for (int o = o_begin; o < o_end && ok; ++o) ok = has_label(p.meta, p.others[o], gid);
                        }
                        m[j] = __builtin_amdgcn_ballot_w64(ok);
                    }
                }
                int inc = 0;   // keys that row r receives from this group, in lane r
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int row0 = 8 * (j >> 2) + (j & 3);
                    set_lane(inc, __builtin_popcount((uint32_t)m[j]), row0);
                    set_lane(inc, __builtin_popcount((uint32_t)(m[j] >> 32)), row0 + 4);
                }
                // (rows that are half full go along: their next drain would come soon)
                if (__any(pcv + inc > kJoinQueue))
                    drain((uint32_t)__ballot(lane < 32 && pcv > 0 && (pcv + inc > kJoinQueue || pcv >= kJoinQueue / 2)));
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    if (m[j] == 0) continue;
                    const int row = 8 * (j >> 2) + (j & 3) + 4 * h;
                    const uint32_t mine = h ? (uint32_t)(m[j] >> 32) : (uint32_t)m[j];
                    const int at = __shfl(pcv, row);
                    if ((mine >> n32) & 1u) {
                        const int slot = at + __builtin_popcount(mine & ((1u << n32) - 1u));
                        // (v for now: the drain makes a distance of it)
                        pend[row * kJoinQueue + slot] = ((uint64_t)(DT == 0 ? (uint32_t)v[j] : __float_as_uint((float)v[j])) << 32) | (uint32_t)entry;
                    }
                }
                pcv += inc;
            }
        }
        if (more) {
            if (NBUF == 1) __syncthreads();
            put(NBUF == 2 ? (g + 1) & 1 : 0);
            __syncthreads();
        }
    }
    drain((uint32_t)__ballot(lane < 32 && pcv > 0));
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
                                 int64_t n_groups, int32_t nk, const uint32_t *norm_all, const float *centre, uint4 *xblk, uint32_t *xnorm)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
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
        const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        uint4 hi, lo;
        split_bf16x8(f, hi, lo);
        xblk[(g * 2 * nch + c) * 32 + v] = hi;
        xblk[(g * 2 * nch + nch + c) * 32 + v] = lo;
        if (c == 0) xnorm[g * 32 + v] = valid ? __float_as_uint(0.5f * __uint_as_float(norm_all[row])) : 0x7F800000u;
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

// One thread per row, elements in ascending order (400,000 x 128: 0.32 ms).
__global__ __launch_bounds__(256) void row_norm_f32_kernel(const float *X, int32_t dim, int64_t n, const float *centre, uint32_t *out,
                                                           uint32_t *out_c, uint32_t *max_bits)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float acc = 0.f, acc_c = 0.f;
    if (i < n) {
        const float4 *x = (const float4 *)(X + i * dim);
        for (int c = 0; c < dim / 4; ++c) {
            const float4 v = x[c], w = centred(v, centre, c);
            acc += v.x * v.x; acc += v.y * v.y; acc += v.z * v.z; acc += v.w * v.w;
            acc_c += w.x * w.x; acc_c += w.y * w.y; acc_c += w.z * w.z; acc_c += w.w * w.w;
        }
        out[i] = __float_as_uint(acc);
        out_c[i] = __float_as_uint(acc_c);
    }
    // (no norm is negative: their bits are ordered as they are, with NaN of either sign above infinity)
    uint32_t m = __float_as_uint(acc), m_c = __float_as_uint(acc_c);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t v = (uint32_t)__shfl_xor((int)m, o), w = (uint32_t)__shfl_xor((int)m_c, o);
        m = v > m ? v : m;
        m_c = w > m_c ? w : m_c;
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(max_bits, m);
        atomicMax(max_bits + 1, m_c);
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
int32_t join_steps(int dtype, int32_t dim)
{
    const int32_t need = dtype == 0 ? (dim + 31) / 32 : (dim + 15) / 16;
    for (const int32_t nk : {2, 4, 6, 8, 16}) if (need <= nk) return nk;
    return dtype == 0 && need <= 32 ? 32 : 0;
}

size_t join_group_bytes(int dtype, int32_t dim)
{
    const int32_t nk = join_steps(dtype, dim);
    return (size_t)(dtype == 0 ? join_chunks<0>(nk) : join_chunks<1>(nk)) * 512;
}

void launch_join_pack(int dtype, const void *X, int32_t dim, const int32_t *map, const JoinList *lists, int n_lists,
                      int64_t n_groups, const uint32_t *norm_all, const float *centre, uint4 *xblk, void *xnorm, hipStream_t s)
{
    if (n_groups <= 0) return;
    const int32_t nk = join_steps(dtype, dim);
    const unsigned blocks = (unsigned)((n_groups * 2 * nk * 32 + 255) / 256);
    if (dtype == 0)
        hipLaunchKernelGGL(join_pack_kernel<0>, dim3(blocks), dim3(256), 0, s, (const char *)X, dim, map, lists, n_lists,
                           n_groups, nk, norm_all, centre, xblk, (uint32_t *)xnorm);
    else
        hipLaunchKernelGGL(join_pack_kernel<1>, dim3(blocks), dim3(256), 0, s, (const char *)X, dim, map, lists, n_lists,
                           n_groups, nk, norm_all, centre, xblk, (uint32_t *)xnorm);
}

template <int DT, int NK> static void launch_join_nk(const JoinParams &p, int n_items, hipStream_t s)
{
    constexpr int NC = join_chunks<DT>(NK);
    const size_t lds = (size_t)join_buffers(NC) * NC * 512 + kJoinRows * kJoinQueue * 8;
    if (p.others_off != nullptr) hipLaunchKernelGGL((join_kernel<DT, NK, true>), dim3(n_items), dim3(256), lds, s, p);
    else hipLaunchKernelGGL((join_kernel<DT, NK, false>), dim3(n_items), dim3(256), lds, s, p);
}

void launch_join(int dtype, const JoinParams &p, int n_items, hipStream_t s)
{
    if (n_items <= 0) return;
    const int32_t nk = join_steps(dtype, p.dim);
    if (dtype == 0) {
        switch (nk) {
        case 2: launch_join_nk<0, 2>(p, n_items, s); break;
        case 4: launch_join_nk<0, 4>(p, n_items, s); break;
        case 6: launch_join_nk<0, 6>(p, n_items, s); break;
        case 8: launch_join_nk<0, 8>(p, n_items, s); break;
        case 16: launch_join_nk<0, 16>(p, n_items, s); break;
        default: launch_join_nk<0, 32>(p, n_items, s); break;
        }
    } else {
        switch (nk) {
        case 2: launch_join_nk<1, 2>(p, n_items, s); break;
        case 4: launch_join_nk<1, 4>(p, n_items, s); break;
        case 6: launch_join_nk<1, 6>(p, n_items, s); break;
        case 8: launch_join_nk<1, 8>(p, n_items, s); break;
        default: launch_join_nk<1, 16>(p, n_items, s); break;
        }
    }
}

}  // namespace vf
