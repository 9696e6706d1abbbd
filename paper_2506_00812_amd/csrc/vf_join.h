// The join kernel (vf_join.hip): many rows against whole lists with the top-K selection fused in.
#pragma once

#include "vf_device.h"

namespace vf {

struct JoinParams {
    const uint4 *xblk;      // packed lists (launch_join_pack)
    const void *xnorm;      // per slot: half the squared norm (float32), the squared norm of the shifted bytes (uint8)
    const int32_t *map;     // local -> global id (AND predicate)
    const void *qsrc;       // row-major [*][dim]
    const int32_t *qrow;    // row of qsrc for each tile row
    const ScanItem *items;  // <= kJoinRows rows each; every item writes partial rows
    int32_t dim, K;         // K <= 64
    int32_t *res_idx;       // [*][K] list-relative entry index, ascending by (distance, index), -1 = none
    uint32_t *res_bits;     //        distance bits: exact (uint8), approximations (float32)
    const int32_t *others_off, *others;   // AND partner labels per query row value, may be null
    LabelMeta meta;
};

constexpr int kJoinRows = 128;

// LDS buffers of one group of nc chunks: two where both fit beside the queues in 64 KiB
__host__ __device__ constexpr int join_buffers(int nc) { return nc <= 32 ? 2 : 1; }

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

// ---------------------------------------------------------------- host side

size_t join_group_bytes(int dtype, int32_t dim);   // packed bytes of a group of 32 vectors
void launch_join_pack(int dtype, const void *X, int32_t dim, const int32_t *map, const int64_t *grp_src, const int32_t *grp_cnt,
                      int64_t n_groups, const uint32_t *norm_all, uint4 *xblk, void *xnorm, hipStream_t s);
void launch_join(int dtype, const JoinParams &p, int n_items, hipStream_t s);

}  // namespace vf
