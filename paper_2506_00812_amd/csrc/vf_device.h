// Device-side helpers shared by the gfx950 kernels.
#pragma once

#include "vf_internal.h"

#pragma clang fp contract(off)

namespace vf {

// Membership test "global id g carries label l" (the predicate of Section 4.3.2).
// Graph labels answer from their bitset; scan labels by binary search in their
// ascending posting list.
__device__ __forceinline__ bool has_label(const LabelMeta &m, int32_t l, int32_t g)
{
    const int32_t slot = m.hs_slot[l];
    if (slot >= 0) return (m.bitsets[(int64_t)slot * m.bitset_words + (g >> 5)] >> (g & 31)) & 1u;
    const int64_t off = m.O_LS[l];
    if (off < 0) return false;
    int32_t lo = 0, hi = m.S[l] - 1;
    while (lo <= hi) {
        const int32_t mid = (lo + hi) >> 1;
        const int32_t v = m.M_LS[off + mid];
        if (v == g) return true;
        if (v < g) lo = mid + 1; else hi = mid - 1;
    }
    return false;
}

// The barrier of a one-wave workgroup; or (WAVE_ONLY), for a wave that works by itself inside a larger workgroup
// (the serving kernel's workers), only what a one-wave barrier is needed for: the ordering of the wave's own LDS
// traffic -- without the workgroup barrier the other waves would have to join.
template <bool WAVE_ONLY> __device__ __forceinline__ void wave_sync()
{
    if constexpr (WAVE_ONLY) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}
// (OPAQUE: so that a kernel that works job after job does not keep what it derives from the lane in registers
// across all of them)
template <bool WAVE_ONLY, bool OPAQUE = false> __device__ __forceinline__ int wave_lane()
{
    int lane = WAVE_ONLY ? (int)(threadIdx.x & 63u) : (int)threadIdx.x;
    if constexpr (OPAQUE) asm volatile("" : "+v"(lane));
    return lane;
}

// float -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint32_t bf16_rn_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// ---------------------------------------------------------------- 8-lane teams

// Sum over the 8 lanes of a team in the fixed tree ((a0+a1)+(a2+a3)) + ((a4+a5)+(a6+a7));
// every lane of the team receives the result.
__device__ __forceinline__ float team_sum_f(float v)
{
    v = v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));  // quad_perm [1,0,3,2]
    v = v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));  // quad_perm [2,3,0,1]
    v = v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true)); // row_half_mirror
    return v;
}
__device__ __forceinline__ int team_sum_i(int v)
{
    v = v + __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
    v = v + __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
    v = v + __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);
    return v;
}

// Squared L2 distance between the query (16-byte chunks in qv) and the row at xrow,
// computed by one 8-lane team; tl = lane within the team.  Lane tl handles chunks
// tl, tl+8, ... .  fp32: lane-sequential acc = fma(d, d, acc) with d = q-x rounded, then
// team_sum_f -- an order that a CPU evaluation (C fmaf) reproduces bit for bit.
// No lane takes a branch: those without a chunk in the last step read an existing one and leave its terms out (a load or
// an LDS read under a lane's condition is a branch of its own, and its wait stands in front of the next: 6,400 queries of
// 24 rows of 32 edges 141 -> 137 us).  LANES: with those branches and a register or two less, which is the better form everywhere
// else: lists of more than one register (1,200 queries x 200, lists of 128: 319 us, 330 without), predicates (3,000 pairs x 200
// that gather 260 and 270), the latency form where vectors have more than 32 chunks (1,000 pairs x 200 597 and 617), and such
// vectors without predicates (2,500 queries x 200, 40 x 2 rows, 163.5 and 170).
__device__ __forceinline__ float team_acc_f32(float acc, const uint4 &q, const uint4 &x, bool in)
{
    float d, a = acc;
    d = __uint_as_float(q.x) - __uint_as_float(x.x); a = __builtin_fmaf(d, d, a);
    d = __uint_as_float(q.y) - __uint_as_float(x.y); a = __builtin_fmaf(d, d, a);
    d = __uint_as_float(q.z) - __uint_as_float(x.z); a = __builtin_fmaf(d, d, a);
    d = __uint_as_float(q.w) - __uint_as_float(x.w); a = __builtin_fmaf(d, d, a);
    return in ? a : acc;
}
template <bool LANES = false>
__device__ __forceinline__ uint32_t team_dist_bits_f32(const uint4 *qv, const char *xrow, int nchunks, int tl)
{
    const int steps = (nchunks + 7) >> 3;
    float acc = 0.0f;
    for (int st0 = 0; st0 < steps; st0 += 4) {
        uint4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {   // all loads of the batch are issued before the first use
            if (!LANES && u > 0 && st0 + u >= steps) break;   // (wave-uniform)
            const int ci = (st0 + u) * 8 + tl;
            if constexpr (LANES) {
                x[u] = make_uint4(0, 0, 0, 0);
                if (ci < nchunks) x[u] = *(const uint4 *)(xrow + ci * kChunkBytes);
            } else {
                x[u] = *(const uint4 *)(xrow + (ci < nchunks ? ci : 0) * kChunkBytes);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!LANES && u > 0 && st0 + u >= steps) break;
            const int ci = (st0 + u) * 8 + tl;
            if constexpr (LANES) {
                if (ci < nchunks) acc = team_acc_f32(acc, qv[ci], x[u], true);
            } else {
                acc = team_acc_f32(acc, qv[ci < nchunks ? ci : 0], x[u], ci < nchunks);
            }
        }
    }
    return __float_as_uint(team_sum_f(acc));
}

// uint8: exact integer sum of (q-x)^2 = q.q + x.x - 2 q.x on the packed dot-product unit.
// qq_lane = sum of q^2 over the bytes this lane handles.
__device__ __forceinline__ int lane_qq_u8(const uint4 *qv, int nchunks, int tl)
{
    uint32_t qq = 0;
    for (int ci = tl; ci < nchunks; ci += 8) {
        const uint4 q = qv[ci];
        qq = __builtin_amdgcn_udot4(q.x, q.x, qq, false);
        qq = __builtin_amdgcn_udot4(q.y, q.y, qq, false);
        qq = __builtin_amdgcn_udot4(q.z, q.z, qq, false);
        qq = __builtin_amdgcn_udot4(q.w, q.w, qq, false);
    }
    return (int)qq;
}
// One team of four lanes (t4 = lane within it), without |q|^2: whole numbers, so neither the split nor the order matters, and
// a wave takes sixteen rows at a time.
__device__ __forceinline__ uint32_t quad_dist_u8(const uint4 *qv, const char *xrow, int nchunks, int t4)
{
    const int steps = (nchunks + 3) >> 2;
    uint32_t xx = 0, qx = 0;
    for (int st0 = 0; st0 < steps; st0 += 4) {
        uint4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u > 0 && st0 + u >= steps) break;   // (wave-uniform)
            const int ci = (st0 + u) * 4 + t4;
            x[u] = *(const uint4 *)(xrow + (ci < nchunks ? ci : 0) * kChunkBytes);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u > 0 && st0 + u >= steps) break;
            const int ci = (st0 + u) * 4 + t4;
            const uint4 q = qv[ci < nchunks ? ci : 0];
            uint32_t a = xx, b = qx;
            a = __builtin_amdgcn_udot4(x[u].x, x[u].x, a, false); b = __builtin_amdgcn_udot4(q.x, x[u].x, b, false);
            a = __builtin_amdgcn_udot4(x[u].y, x[u].y, a, false); b = __builtin_amdgcn_udot4(q.y, x[u].y, b, false);
            a = __builtin_amdgcn_udot4(x[u].z, x[u].z, a, false); b = __builtin_amdgcn_udot4(q.z, x[u].z, b, false);
            a = __builtin_amdgcn_udot4(x[u].w, x[u].w, a, false); b = __builtin_amdgcn_udot4(q.w, x[u].w, b, false);
            xx = ci < nchunks ? a : xx; qx = ci < nchunks ? b : qx;
        }
    }
    int v = (int)xx - 2 * (int)qx;
    v = v + __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    v = v + __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    return (uint32_t)v;
}

typedef _Float16 v8h_seed __attribute__((ext_vector_type(8)));

// eight components (two 16-byte chunks) scaled and rounded to binary16
__device__ __forceinline__ uint4 scaled_half8(const uint4 &a, const uint4 &b, float scale)
{
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    v8h_seed x;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (_Float16)(__uint_as_float(w[i]) * scale);
    return __builtin_bit_cast(uint4, x);
}
typedef float v16f_seed __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src)
{
    const uint32_t lo = __shfl((uint32_t)v, src), hi = __shfl((uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_up64(uint64_t v)
{
    const uint32_t lo = __shfl_up((uint32_t)v, 1), hi = __shfl_up((uint32_t)(v >> 32), 1);
    return ((uint64_t)hi << 32) | lo;
}

// value of lane `src` (wave-uniform index) in every lane
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int src)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, src), hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}
// lane i receives the value of lane i - 1 (lane 0 keeps its own): DPP wave_shr:1
__device__ __forceinline__ uint64_t wave_shr1_64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)v, (int)(uint32_t)v, 0x138, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(v >> 32), (int)(uint32_t)(v >> 32), 0x138, 0xF, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}

// ---------------------------------------------------------------- sorting networks over the lanes of a wave

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

// One compare-exchange stage of 32-bit values (a float is no NaN): the lanes of MIN keep the smaller value of the pair
// (lane, lane ^ J), the others the larger.
template <int J, uint64_t MIN, class V> __device__ __forceinline__ V lane_exchange_32(V v)
{
    uint32_t ab, bb;
    lane_pair<J>(__builtin_bit_cast(uint32_t, v), ab, bb);
    const V a = __builtin_bit_cast(V, ab), b = __builtin_bit_cast(V, bb);
    const V lo = a < b ? a : b, hi = a < b ? b : a;
    return __builtin_amdgcn_inverse_ballot_w64(MIN) ? lo : hi;
}

// ... of 64-bit keys, one set by itself: both results of the comparison are selected by it and the wanted one by a constant,
// so that no stage waits for the scalar unit.
template <int J, uint64_t MIN> __device__ __forceinline__ uint64_t lane_exchange_lone(uint64_t v)
{
    uint32_t al, bl, ah, bh;
    lane_pair<J>((uint32_t)v, al, bl);
    lane_pair<J>((uint32_t)(v >> 32), ah, bh);
    const uint64_t a = ((uint64_t)ah << 32) | al, b = ((uint64_t)bh << 32) | bl;
    const bool less = a < b;
    const uint64_t lo = less ? a : b, hi = less ? b : a;
    return __builtin_amdgcn_inverse_ballot_w64(MIN) ? lo : hi;
}

template <int K, int J> __device__ __forceinline__ uint32_t wave_stages(uint32_t v)
{
    v = lane_exchange_32<J, keep_min_lanes<K, J, K == 64, false>()>(v);
    if constexpr (J > 1) return wave_stages<K, J / 2>(v);
    else return v;
}
template <int K, int J> __device__ __forceinline__ uint64_t wave_stages(uint64_t v)
{
    v = lane_exchange_lone<J, keep_min_lanes<K, J, K == 64, false>()>(v);
    if constexpr (J > 1) return wave_stages<K, J / 2>(v);
    else return v;
}
template <int K, class T> __device__ __forceinline__ T wave_sort_from(T v)
{
    v = wave_stages<K, K / 2>(v);
    if constexpr (K < 64) return wave_sort_from<2 * K>(v);
    else return v;
}

// Ascending bitonic sort of the 64 values held one per lane, and ascending sort of a bitonic sequence of them; every move on
// the vector ALU: through ds_bpermute each of the 21 (6) stages waits for an LDS access.
__device__ __forceinline__ uint32_t wave_sort_u32(uint32_t v, int) { return wave_sort_from<2>(v); }
__device__ __forceinline__ uint32_t wave_merge_u32(uint32_t v, int) { return wave_stages<64, 32>(v); }
__device__ __forceinline__ uint64_t wave_sort64(uint64_t v, int) { return wave_sort_from<2>(v); }
__device__ __forceinline__ uint64_t wave_merge64(uint64_t v, int) { return wave_stages<64, 32>(v); }

// Bitonic sort of keys[0..n) ascending in LDS by one wave; n a power of two.
__device__ __forceinline__ void wave_bitonic_sort(uint64_t *keys, int n, int lane)
{
    for (int k = 2; k <= n; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = lane; i < n / 2; i += 64) {
                const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1)), b = a | j;
                const bool up = (a & k) == 0;
                const uint64_t x = keys[a], y = keys[b];
                if ((x > y) == up) { keys[a] = y; keys[b] = x; }
            }
            __syncthreads();
        }
}

}  // namespace vf
