// Graph-search initialisation (Section 4.2.1: the initial candidates are sampled
// inside the label's list): distances from every graph query to the seeds of its
// label, computed densely.
//
// The seeds of a label -- local ids floor(j * n / ns) -- do not depend on the query,
// so all queries of a label score the same vectors: a dense queries x seeds block per label
// instead of every query gathering its seeds from HBM.  Three kernels fill that block:
//
//   seed_mfma_kernel    the default wherever it has an instantiation.  The block is a contraction,
//                       |q|^2 + |x|^2 - 2 q.x on the matrix cores: exact for uint8, an approximation
//                       for float32 that the beam kernel re-ranks under a proof (see below).
//   seed_select_kernel  the same scoring with the selection fused in: per (query, seed segment) only a
//                       run of the K smallest keys leaves the kernel (off by default: slower than the
//                       unfused pair except on long uint8 seed lists).
//   seed_dist_kernel    the ordered distance itself on the vector ALU, for dimensions and list sizes the
//                       matrix-core kernels do not cover and as the reference route of the tests: one wave
//                       takes up to 64 queries of one label (one query per lane, the query vector held in
//                       registers) and a chunk of kSeedChunk seeds; a seed vector is the same for all lanes,
//                       so it is fetched with scalar loads and used as a scalar operand -- no LDS or
//                       cross-lane traffic in the inner loop.  A lane evaluates the distance in exactly the
//                       order the 8-lane teams of the beam kernel use (partial sum t takes the 16-byte
//                       chunks 8s + t, fused multiply-add, fixed tree), so the bits are identical to a
//                       gathered evaluation and to the CPU evaluation.
//
// Output of the unfused kernels: dseed[gq][j] = distance bits of graph query gq to seed j, consumed by the
// beam kernel, which keeps the best itopk.
#include <type_traits>
#include <utility>

#include "vf_select.h"

namespace vf {

// NCH: 16-byte chunks per vector; FIT = false: an upper bound of them (dimensions without an instantiation of their own),
// the chunks that do not exist are zero on both sides, which leaves every partial sum as it is.
template <int DT, int NCH, bool FIT>
__global__ __launch_bounds__(64) void seed_dist_kernel(SeedParams p)
{
    constexpr int SC = kSeedChunk;
    __shared__ uint32_t outb[64 * (SC + 1)];
    const int lane = threadIdx.x;
    const int tile = blockIdx.x / p.max_chunks, chunk = blockIdx.x % p.max_chunks;
    const SeedTile t = p.tiles[tile];
    const int n = p.meta.S[t.label];
    const int64_t base = p.meta.O_HS[t.label];
    const int ns = p.n_seeds < n ? p.n_seeds : n;
    const int j0 = chunk * SC;
    if (j0 >= ns) return;
    const int cnt = ns - j0 < SC ? ns - j0 : SC;
    const int nch = FIT ? NCH : p.dim * (DT == 0 ? 1 : 4) / kChunkBytes;
    const int row_bytes = nch * kChunkBytes;

    // seeds of this chunk -> global ids (lane i holds seed j0 + i)
    int g = 0;
    if (lane < cnt) g = p.meta.M_HS[base + (int64_t)(((uint64_t)(j0 + lane) * (uint64_t)n) / (uint64_t)ns)];

    // this lane's query
    uint32_t q[NCH * 4];
    {
        const int qi = p.gq_query[t.gq_begin + (lane < t.q_count ? lane : 0)];
        const uint4 *qrow = (const uint4 *)((const char *)p.Q + (int64_t)qi * row_bytes);
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (FIT || ch < nch) v = qrow[ch];
            q[ch * 4] = v.x; q[ch * 4 + 1] = v.y; q[ch * 4 + 2] = v.z; q[ch * 4 + 3] = v.w;
        }
    }
    uint32_t qq = 0;
    if (DT == 0) {
#pragma unroll
        for (int w = 0; w < NCH * 4; ++w) qq = __builtin_amdgcn_udot4(q[w], q[w], qq, false);
    }

    for (int i = 0; i < cnt; ++i) {
        // the seed vector is wave uniform: it comes in through scalar loads and feeds the VALU
        // as a scalar operand -- no LDS staging, no cross-lane traffic
        const int gi = __builtin_amdgcn_readlane(g, i);
        const uint32_t *__restrict__ xp = (const uint32_t *)((const char *)p.X + (int64_t)gi * row_bytes);
        // chunk ch of the seed (every load is a whole chunk, unconditional and in bounds, so that all of a vector's can be
        // in flight)
        auto chunk_of = [&](int ch, uint32_t (&x)[4]) {
            const uint32_t *c = xp + 4 * (FIT || ch < nch ? ch : nch - 1);
#pragma unroll
            for (int w = 0; w < 4; ++w) x[w] = c[w];
            if (!FIT && ch >= nch) x[0] = x[1] = x[2] = x[3] = 0u;
        };
        uint32_t bits;
        if (DT == 0) {
            uint32_t xx = 0, qx = 0;
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                uint32_t x[4];
                chunk_of(ch, x);
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    xx = __builtin_amdgcn_udot4(x[w], x[w], xx, false);
                    qx = __builtin_amdgcn_udot4(q[ch * 4 + w], x[w], qx, false);
                }
            }
            bits = (uint32_t)((int)qq + (int)xx - 2 * (int)qx);
        } else {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = 0.0f;
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                uint32_t x[4];
                chunk_of(ch, x);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float d = __uint_as_float(q[ch * 4 + c]) - __uint_as_float(x[c]);
                    a[ch & 7] = __builtin_fmaf(d, d, a[ch & 7]);
                }
            }
            const float b0 = a[0] + a[1], b1 = a[2] + a[3], b2 = a[4] + a[5], b3 = a[6] + a[7];
            const float c0 = b0 + b1, c1 = b2 + b3;
            bits = __float_as_uint(c0 + c1);
        }
        outb[lane * (SC + 1) + i] = bits;
    }
    __syncthreads();

    // rows of dseed: SC consecutive seeds per query
    for (int r0 = 0; r0 < t.q_count; r0 += 64 / SC) {
        const int r = r0 + lane / SC, col = lane % SC;
        if (r < t.q_count && col < cnt)
            p.dseed[(int64_t)(t.gq_begin + r) * p.ns_stride + j0 + col] = outb[r * (SC + 1) + col];
    }
}

// ---------------------------------------------------------------------------------------------
// Matrix cores.  queries x seeds of one label is a dense contraction, |q|^2 + |x|^2 - 2 q.x.  One wave: a tile of <= 64 or 32
// queries (seed_mfma_tile; in registers) against NG groups of 32 seeds; lane (v, h) holds the 16-byte chunks 2 s + h of query v, and of seed v.
// uint8 data: v_mfma_i32_32x32x32_i8 on the vectors shifted by -128 (the shift cancels in q - x): the int32 result is the
// exact distance, so nothing is approximate there and the rows of dseed are used as they are.
// float32 data: v_mfma_f32_32x32x2_f32 on the rows or a float32 copy of the seeds (small batches, tables without a copy), or,
// from a copy of the seeds in binary16, v_mfma_f32_32x32x16_f16 (a sixteenth of the matrix-core time): both operands
// rounded to binary16 after multiplication by a power of two that brings the table's largest norm into [32, 64), norms
// those of the unrounded vectors.  The values are a filter only: the beam kernel scores the seeds that may belong to its list
// with the ordered distance, under a bound of the difference.  With u = 2^-24, q^ and x^ the rounded vectors (unscaled), and dx
// the largest |x - x^|, measured when the copy is built:
//   |2 q.x - 2 q^.x^| <= 2 |q - q^| |x|max + 2 |q^| dx    (|q - q^|: measured by the beam kernel)
//   the sum of <= 256 products, 2 u each, norms and final additions < 1024 u (|q|^2 + |x|max^2); 2048 u are used
// (a query whose scaled length is beyond 2^15 has no usable approximations: the beam kernel scores its seeds itself).
// float32 products: <= 512 terms in any order, norms, final additions: 300 u, 512 u used.  (Bfloat16 seeds and queries in two
// bfloat16 parts, as before, take twice the products, and their bound on 1,000,000 x 128 is 3.6 instead of 0.8.)
typedef int v16i_seed __attribute__((ext_vector_type(16)));
typedef int v4i_seed __attribute__((ext_vector_type(4)));
// Queries of a tile: 64 where the registers allow it: every seed is then read from L2 half as often (6,500 x 6,144 x 128: 52 us
// instead of 59; 10,700 AND pairs x 96: 180 instead of 210; uint8 x 192: the same).
static constexpr __host__ __device__ int seed_mfma_tile(int dt, int steps) { return dt != 1 && steps <= 8 ? 64 : 32; }

template <class F, int... G> __device__ __forceinline__ void while_each(F &&f, std::integer_sequence<int, G...>)
{
    (void)(f(std::integral_constant<int, G>()) && ...);
}

// DT: 0 uint8, 1 float32, 2 float32 data from the copy in binary16.
// CACHED: the seeds come from their interleaved copy (coalesced 1-KiB loads); otherwise every lane gathers its seed's row
// from X.  NCP: contraction steps.  FIT = false: vectors of fewer steps than NCP (dimensions without an instantiation of
// their own; from the copy only); the steps that do not exist have a zero query operand and read the copy's last chunk once
// more.  NG: groups of a wave, unrolled.
// The seeds are the rows of the product and the queries its columns, so a lane has 16 seeds of one query: the minimum of a
// group's 32 is eight instructions and one swap.  The result goes through LDS to be stored as whole rows, 1 KB an
// instruction.  Bound by the stores, and by what is in flight: loads and stores are counted by one counter in order, so a
// wave that waits for its next group's chunks waits for every store issued before their request, too (requests two groups
// ahead, where the registers allow it, leave the stores of the last two groups in flight).  39,000 queries x 16,384 seeds x 192 uint8 (2.4 GB)
// 807 -> 655 us (nothing but the stores: 400), 10,700 AND pairs x up to 16,384 seeds x 96 220 -> 180 us, 6,500 queries x 6,144
// seeds x 128 79 -> 52 us; before: queries as rows, their operand read from LDS, two products a step, 16 addresses by 64-bit
// multiplication and 45 instructions of minima per group.
// Queries a tile does not have repeat its last one, and seeds past the end of a list are stored within its row, so that every
// store is unconditional.
template <int DT, int NCP, bool CACHED, int NG, bool FIT = true>
__global__ __launch_bounds__(64, NCP <= (FIT ? 8 : 6) ? 3 : 2) void seed_mfma_kernel(SeedParams p)
{
    static_assert((DT != 2 && FIT) || CACHED, "binary16 seeds and other dimensions only from the interleaved copy");
    constexpr int QT = seed_mfma_tile(DT, NCP) / 32;               // sets of 32 queries
    constexpr int PITCH = 36, MINS = NG + 1, AHEAD = NG > 1 && NCP <= 4 ? 2 : 1;   // words of a row in LDS; groups requested ahead
    __shared__ uint32_t rows[32 * PITCH];
    __shared__ uint32_t mins[CACHED ? QT * 32 * MINS : 1];         // the groups' minima of each query
    __shared__ uint32_t norms[32];
    const int blk_chunks = FIT ? 2 * NCP : p.blk_chunks;            // 16-byte chunks of a seed in the copy
    const int row_bytes = p.dim * (DT == 0 ? 1 : 4);                // of a query
    const int lane = threadIdx.x, n32 = lane & 31, h = lane >> 5;
    const int tile = blockIdx.x / p.max_chunks, chunk = blockIdx.x % p.max_chunks;
    const SeedTile t = p.tiles[tile];
    const int n = p.meta.S[t.label];
    const int64_t base = p.meta.O_HS[t.label];
    const int ns = p.n_seeds < n ? p.n_seeds : n;
    const int j0 = chunk * (NG * 32);
    if (j0 >= ns) return;
    const bool second = QT > 1 && t.q_count > 32;

    const int64_t grp0 = CACHED ? p.seed_goff[p.meta.hs_slot[t.label]] + j0 / 32 : 0;
    int gid[CACHED ? 1 : NG];   // without a copy: global id of this lane's seed in each group
    if constexpr (!CACHED) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int j = j0 + g * 32 + n32;
            gid[g] = p.meta.M_HS[base + (j < ns ? (int)(((uint64_t)j * (uint64_t)n) / (uint64_t)ns) : 0)];
        }
    }

    // the tile's operand: lane (n32, h) holds the chunks 2 s + h of query n32 of each set
    uint4 q[QT][NCP];
    uint32_t qn[QT];
#pragma unroll
    for (int o = 0; o < QT; ++o) {
        const int at = 32 * o + n32;
        const int qr = p.gq_query[t.gq_begin + (at < t.q_count ? at : t.q_count - 1)];
        const char *qp = (const char *)p.Q + (int64_t)qr * row_bytes;
        auto chunk_of = [&](int c) -> uint4 {   // (those that do not exist: the first one is read, and zeros are in its place)
            const bool in = FIT || c * kChunkBytes < row_bytes;
            uint4 v = *(const uint4 *)(qp + (in ? c * kChunkBytes : 0));
            if (!in) v = make_uint4(0, 0, 0, 0);
            return v;
        };
        if constexpr (DT == 0) {
            int acc = 0;
#pragma unroll
            for (int s = 0; s < NCP; ++s) {
                const int c = 2 * s + h;
                uint4 v = chunk_of(c);
                if (FIT || c * kChunkBytes < row_bytes) { v.x ^= 0x80808080u; v.y ^= 0x80808080u; v.z ^= 0x80808080u; v.w ^= 0x80808080u; }
                q[o][s] = v;
                acc = __builtin_amdgcn_sdot4((int)v.x, (int)v.x, acc, false); acc = __builtin_amdgcn_sdot4((int)v.y, (int)v.y, acc, false);
                acc = __builtin_amdgcn_sdot4((int)v.z, (int)v.z, acc, false); acc = __builtin_amdgcn_sdot4((int)v.w, (int)v.w, acc, false);
            }
            acc += __shfl_xor(acc, 32);
            qn[o] = (uint32_t)acc;
        } else {
            float acc = 0.f;
#pragma unroll
            for (int s = 0; s < NCP; ++s) {
                if constexpr (DT == 1) {
                    const uint4 v = chunk_of(2 * s + h);
                    q[o][s] = v;
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc += __uint_as_float(w[i]) * __uint_as_float(w[i]);
                } else {   // components 8 (2 s + h) and the next seven
                    const uint4 v0 = chunk_of(4 * s + 2 * h), v1 = chunk_of(4 * s + 2 * h + 1);
                    const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc += __uint_as_float(w[i]) * __uint_as_float(w[i]);
                    q[o][s] = scaled_half8(v0, v1, p.scale);
                }
            }
            acc += __shfl_xor(acc, 32);
            qn[o] = __float_as_uint(acc);
        }
    }
    // where rows 8 i + lane / 8 of a set's result go, as bytes from the tile's first row (64 rows: less than 4 GiB)
    uint32_t at[QT][4];
#pragma unroll
    for (int o = 0; o < QT; ++o)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 32 * o + 8 * i + (lane >> 3);
            at[o][i] = ((uint32_t)(row < t.q_count ? row : t.q_count - 1) * (uint32_t)p.ns_stride + 4u * (lane & 7)) * 4u;
        }
    char *const out = (char *)(p.dseed + (int64_t)t.gq_begin * p.ns_stride + j0);

    constexpr uint32_t kNever = DT == 0 ? 0x3FFFFFFFu : 0x7F800000u;   // norm of a seed that does not exist: larger than any
    uint4 b[AHEAD][NCP];
    uint32_t xn[AHEAD];               // norm of seed n32
    const int last = (ns - j0 + 31) / 32 - 1;
    auto fetch_group = [&](int gg) {  // group gg of this wave's seeds (past the last one that exists: that one again, so that every
        uint4 (&to)[NCP] = b[gg % AHEAD];   // request is unconditional and the waits can be counted)
        uint32_t &xn_to = xn[gg % AHEAD];
        if constexpr (CACHED) {
            const int g = gg < last ? gg : last;
            const uint4 *blk = p.seed_blk + (grp0 + g) * (int64_t)(blk_chunks * 32);
#pragma unroll
            for (int s = 0; s < NCP; ++s) to[s] = blk[(FIT || 2 * s + h < blk_chunks ? 2 * s + h : blk_chunks - 1) * 32 + n32];
            xn_to = p.seed_norm[(grp0 + g) * 32 + n32];
        } else {
            const int id = gid[gg];   // (every one of them is a seed)
            const char *xrow = (const char *)p.X + (int64_t)id * row_bytes;
#pragma unroll
            for (int s = 0; s < NCP; ++s) to[s] = *(const uint4 *)(xrow + (2 * s + h) * kChunkBytes);
            xn_to = p.xnorm_all[id];
        }
    };
#pragma unroll
    for (int g = 0; g < AHEAD; ++g) fetch_group(g);
    auto group = [&](auto number) -> bool {
        constexpr int g = decltype(number)::value;
        if (g > last) return false;    // (wave-uniform)
        uint4 (&x)[NCP] = b[g % AHEAD];
        wave_lds_sync();               // (the last group's rows have been read)
        norms[n32] = j0 + g * 32 + n32 < ns ? xn[g % AHEAD] : kNever;
        using acc_t = typename std::conditional<DT == 0, v16i_seed, v16f_seed>::type;
        acc_t acc[QT];
#pragma unroll
        for (int o = 0; o < QT; ++o)
#pragma unroll
            for (int jj = 0; jj < 16; ++jj) acc[o][jj] = 0;
        if constexpr (DT == 0) {
#pragma unroll
            for (int s = 0; s < NCP; ++s) { x[s].x ^= 0x80808080u; x[s].y ^= 0x80808080u; x[s].z ^= 0x80808080u; x[s].w ^= 0x80808080u; }
        }
#pragma unroll
        for (int o = 0; o < QT; ++o) {
            if (o > 0 && !second) break;   // (wave-uniform)
#pragma unroll
            for (int s = 0; s < NCP; ++s) {
                if constexpr (DT == 0) {
                    acc[o] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i_seed, x[s]), __builtin_bit_cast(v4i_seed, q[o][s]), acc[o], 0, 0, 0);
                } else if constexpr (DT == 2) {
                    acc[o] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h_seed, x[s]), __builtin_bit_cast(v8h_seed, q[o][s]), acc[o], 0, 0, 0);
                } else {
                    acc[o] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x[s].x), __uint_as_float(q[o][s].x), acc[o], 0, 0, 0);
                    acc[o] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x[s].y), __uint_as_float(q[o][s].y), acc[o], 0, 0, 0);
                    acc[o] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x[s].z), __uint_as_float(q[o][s].z), acc[o], 0, 0, 0);
                    acc[o] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x[s].w), __uint_as_float(q[o][s].w), acc[o], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (g + AHEAD < NG) fetch_group(g + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < QT; ++o) {
            if (o > 0 && !second) break;   // (wave-uniform)
            wave_lds_sync();
            uint32_t m = 0xFFFFFFFFu;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 n4 = *(const uint4 *)&norms[8 * i + 4 * h];
                const uint32_t nx[4] = {n4.x, n4.y, n4.z, n4.w};
                uint32_t bits[4];          // seeds 8 i + 4 h + u of query n32
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int jj = 4 * i + u;
                    if constexpr (DT == 0) bits[u] = qn[o] + nx[u] - ((uint32_t)acc[o][jj] << 1);
                    else bits[u] = __float_as_uint(fmaxf(__builtin_fmaf(DT == 1 ? -2.0f : p.minus_two_unscaled, acc[o][jj], __uint_as_float(qn[o]) + __uint_as_float(nx[u])), 0.0f));
                    m = bits[u] < m ? bits[u] : m;
                }
                *(uint4 *)&rows[n32 * PITCH + 8 * i + 4 * h] = make_uint4(bits[0], bits[1], bits[2], bits[3]);
            }
            if constexpr (CACHED) {
                const auto r = __builtin_amdgcn_permlane32_swap(m, m, false, false);
                mins[(32 * o + n32) * MINS + g] = r[0] < r[1] ? r[0] : r[1];
            }
            wave_lds_sync();
#pragma unroll
            for (int i = 0; i < 4; ++i) *(uint4 *)(out + at[o][i] + g * 128) = *(const uint4 *)&rows[(8 * i + (lane >> 3)) * PITCH + 4 * (lane & 7)];
        }
        return true;
    };
    while_each(group, std::make_integer_sequence<int, NG>());   // (a loop that is left early is not unrolled)
    if constexpr (CACHED) {
        wave_lds_sync();
        if (p.dmin != nullptr && lane < t.q_count && lane < QT * 32) {   // (the minima of groups that do not exist are not read)
            uint32_t *dst = p.dmin + (int64_t)(t.gq_begin + lane) * p.nb_stride + j0 / 32;
            const uint32_t *m = &mins[lane * MINS];
            if constexpr (NG % 4 == 0) {   // (rows of minima are multiples of 16 words)
#pragma unroll
                for (int g = 0; g < NG; g += 4) *(uint4 *)(dst + g) = make_uint4(m[g], m[g + 1], m[g + 2], m[g + 3]);
            } else {
#pragma unroll
                for (int g = 0; g < NG; ++g) dst[g] = m[g];
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Seed scoring with the selection fused in.  The beam search starts from the best `itopk` of a query's
// seeds, a few dozen out of thousands, so nothing but those needs to leave the kernel that scores them.
// One wave takes a tile of <= 32 same-label queries and a SEGMENT of the label's seeds (seg_seeds of them,
// whole 32-seed groups of the interleaved copy), contracts them on the matrix cores group by group like
// seed_mfma_kernel, and keeps per query row the K smallest (value, seed index) pairs with the queue-and-merge
// selection of the scan kernels: a row's threshold tightens as the segment streams by, so after the first
// groups only a few values per group reach a queue.  Output: one sorted run of K keys
// (value bits << 32 | seed index) per (query, segment); the beam kernel merges a query's runs.
// Why that is enough.  uint8 values are the exact distances, and the order of keys is the order of
// (distance, local id) since the local id floor(j n / ns) grows with j: the K best of the union of the runs are
// the K best seeds.  float32 values are approximations: the beam kernel keeps the K best of the union, re-scores
// them with the ordered distance and needs a lower bound T on the approximation of every seed it did NOT keep.
// A seed missing from the union was rejected in its segment by K values that all are in the union, so its
// approximation is at least the union's K-th smallest value, which is T as before.
// A operand (queries) in registers for the whole segment; LDS holds only the queues and the lists.
// DT = 0: uint8 data (v_mfma_i32_32x32x32_i8 on the -128 shifted bytes).  DT = 2: float32 data, seeds from the binary16 copy.
template <int DT, int NCP>
__global__ __launch_bounds__(64, 2) void seed_select_kernel(SeedSelParams p)
{
    static_assert(DT == 0 || DT == 2, "uint8, or float32 data with a binary16 seed copy");
    extern __shared__ uint4 smem[];
    constexpr int NCH = 2 * NCP, PC = 64;
    constexpr int row_bytes = (DT == 2 ? 2 : 1) * NCH * kChunkBytes;   // of a query
    const int K = p.K, KS = K | 1;
    uint64_t *pend = (uint64_t *)smem;               // [32][PC] candidates not yet merged
    uint64_t *best = pend + 32 * PC;                 // [32][KS] K best so far, ascending, KEY_MAX padded
    uint32_t *qnorm_s = (uint32_t *)(best + 32 * KS); // [32] float bits / int
    uint32_t *pcnt = qnorm_s + 32;                   // [32] keys waiting in pend[r]
    int32_t *qrow_s = (int32_t *)(pcnt + 32);        // [32] query index of the row, -1: none
    int32_t *pslot_s = qrow_s + 32;                  // [32] bitset row of the row's AND partner, see below

    const int lane = threadIdx.x, n32 = lane & 31, h = lane >> 5;
    const int tile = blockIdx.x / p.max_segs, seg = blockIdx.x % p.max_segs;
    const SeedTile t = p.tiles[tile];
    const int n = p.meta.S[t.label];
    const int ns = p.n_seeds < n ? p.n_seeds : n;
    const int j0 = seg * p.seg_seeds;
    if (j0 >= ns) return;   // the label has fewer segments than the grid allows for (the whole workgroup leaves)
    const int nj = ns - j0 < p.seg_seeds ? ns - j0 : p.seg_seeds;
    const int n_groups = (nj + 31) >> 5;
    const int64_t grp0 = p.seed_goff[p.meta.hs_slot[t.label]] + (j0 >> 5);

    if (lane < 32) {
        const int qr = lane < t.q_count ? p.gq_query[t.gq_begin + lane] : -1;
        qrow_s[lane] = qr;
        pcnt[lane] = 0;
        // the common AND query has one partner label, a graph label: its predicate is one bit of that label's
        // bitset, which can be fetched for all of a lane's rows at once (pslot_s >= 0); other rows evaluate the
        // general predicate pair by pair
        int ps = -1;
        if (qr >= 0 && p.others_off != nullptr && p.others_off[qr + 1] - p.others_off[qr] == 1)
            ps = p.meta.hs_slot[p.others[p.others_off[qr]]];
        pslot_s[lane] = ps;
    }
    for (int i = lane; i < 32 * KS; i += 64) best[i] = KEY_MAX;
    __syncthreads();

    // ---- A operand: lane (n32, h) holds chunks 2 cp + h of query row n32 (zeros for a row without a query)
    uint4 areg[NCP];
    {
        const int qr = qrow_s[n32];
        const char *qp = (const char *)p.Q + (int64_t)(qr >= 0 ? qr : 0) * row_bytes;
        float facc = 0.f;
        int iacc = 0;
#pragma unroll
        for (int cp = 0; cp < NCP; ++cp) {
            const int c = 2 * cp + h;
            if constexpr (DT == 2) {   // components 8 c .. 8 c + 7
                uint4 v0 = make_uint4(0, 0, 0, 0), v1 = v0;
                if (qr >= 0) {
                    v0 = *(const uint4 *)(qp + (2 * c) * kChunkBytes);
                    v1 = *(const uint4 *)(qp + (2 * c + 1) * kChunkBytes);
                }
                const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
                for (int i = 0; i < 8; ++i) facc += __uint_as_float(w[i]) * __uint_as_float(w[i]);
                areg[cp] = scaled_half8(v0, v1, p.scale);
            } else {
                uint4 v = make_uint4(0, 0, 0, 0);
                if (qr >= 0) {
                    v = *(const uint4 *)(qp + c * kChunkBytes);
                    v.x ^= 0x80808080u; v.y ^= 0x80808080u; v.z ^= 0x80808080u; v.w ^= 0x80808080u;
                }
                areg[cp] = v;
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int bb = 0; bb < 4; ++bb) {
                        const int e = (int)(int8_t)(w[i] >> (8 * bb));
                        iacc += e * e;
                    }
            }
        }
        if (DT == 0) {
            iacc += __shfl_xor(iacc, 32);
            if (h == 0) qnorm_s[n32] = (uint32_t)iacc;
        } else {
            facc += __shfl_xor(facc, 32);
            if (h == 0) qnorm_s[n32] = __float_as_uint(facc);
        }
    }
    __syncthreads();

    // per-lane constants for its 16 accumulator rows: row(j) = 8 * (j / 4) + 4 * h + (j % 4)
    uint32_t qn[16], thr[16];
    uint32_t live_rows = 0, and_rows = 0, fast_rows = 0;   // and_rows: general predicate; fast_rows: one bitset bit
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int row = 8 * (j >> 2) + 4 * h + (j & 3);
        qn[j] = qnorm_s[row];
        thr[j] = 0xFFFFFFFFu;
        if (row < t.q_count) {
            live_rows |= 1u << j;
            if (p.others_off != nullptr) {
                const int qr = qrow_s[row];
                if (pslot_s[row] >= 0) fast_rows |= 1u << j;
                else if (p.others_off[qr + 1] > p.others_off[qr]) and_rows |= 1u << j;
            }
        }
    }
    const bool any_and = __any((and_rows | fast_rows) != 0);
    int pcv = 0;                  // state of tile row r, held by lane r (r < 32)
    uint64_t row_kth = KEY_MAX;

    // Merge queues into lists: only the rows whose queue could overflow on the next group (more than PC - 32
    // keys), or every row with a key at the end of the segment.  A drain costs a sort and a merge per row
    // whatever the queue holds, so a row is left alone until its queue is worth it.
    auto drain = [&](bool all) {
        wave_lds_sync();
        const bool mine = lane < 32 && pcv > (all ? 0 : PC - 32);
        int pcv_sel = mine ? pcv : 0;
        if (K <= 32) wave_drain_rows_packed<32>(pend, PC, best, KS, K, pcv_sel, row_kth, lane);
        wave_drain_rows<4>(pend, PC, best, KS, K, pcv_sel, row_kth, lane);
        if (mine) { pcnt[lane] = 0; pcv = 0; }
        wave_lds_sync();
        const uint32_t tk = (uint32_t)(row_kth >> 32);
#pragma unroll
        for (int j = 0; j < 16; ++j) thr[j] = __shfl(tk, 8 * (j >> 2) + 4 * h + (j & 3));
    };

    // B operand: the whole group in registers, each half refilled with the next group's chunks right after its
    // own MFMAs have been issued
    constexpr int H0 = (NCP + 1) / 2;
    uint4 breg[NCP];
    {
        const uint4 *blk0 = p.seed_blk + grp0 * (int64_t)(NCH * 32);
#pragma unroll
        for (int cp = 0; cp < NCP; ++cp) breg[cp] = blk0[(2 * cp + h) * 32 + n32];
    }
    uint32_t xn_next = p.seed_norm[grp0 * 32 + n32];
    int32_t gid_next = -1;
    if (any_and) gid_next = p.seed_map[grp0 * 32 + n32];
    for (int grp = 0; grp < n_groups; ++grp) {
        const uint4 *nblk = p.seed_blk + (grp0 + grp + 1) * (int64_t)(NCH * 32);
        const bool more = grp + 1 < n_groups;
        const uint32_t xn = xn_next;
        const int32_t gid = gid_next;
        if (more) {
            xn_next = p.seed_norm[(grp0 + grp + 1) * 32 + n32];
            if (any_and) gid_next = p.seed_map[(grp0 + grp + 1) * 32 + n32];
        }
        uint32_t bitsv[16];
        if constexpr (DT == 0) {
            v16i_seed acc;
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = 0;
            auto contract = [&](int cp) {
                uint4 b = breg[cp];
                b.x ^= 0x80808080u; b.y ^= 0x80808080u; b.z ^= 0x80808080u; b.w ^= 0x80808080u;
                const uint4 a = areg[cp];
                const v4i_seed av = {(int)a.x, (int)a.y, (int)a.z, (int)a.w};
                const v4i_seed bv = {(int)b.x, (int)b.y, (int)b.z, (int)b.w};
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, acc, 0, 0, 0);
            };
#pragma unroll
            for (int cp = 0; cp < H0; ++cp) contract(cp);
            if (more) {
#pragma unroll
                for (int cp = 0; cp < H0; ++cp) breg[cp] = nblk[(2 * cp + h) * 32 + n32];
            }
#pragma unroll
            for (int cp = H0; cp < NCP; ++cp) contract(cp);
            if (more) {
#pragma unroll
                for (int cp = H0; cp < NCP; ++cp) breg[cp] = nblk[(2 * cp + h) * 32 + n32];
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) bitsv[j] = (uint32_t)((int)qn[j] + (int)xn - 2 * acc[j]);
        } else {
            v16f_seed acc;
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[j] = 0.f;
            auto contract = [&](int cp) {
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h_seed, areg[cp]), __builtin_bit_cast(v8h_seed, breg[cp]), acc, 0, 0, 0);
            };
#pragma unroll
            for (int cp = 0; cp < H0; ++cp) contract(cp);
            if (more) {
#pragma unroll
                for (int cp = 0; cp < H0; ++cp) breg[cp] = nblk[(2 * cp + h) * 32 + n32];
            }
#pragma unroll
            for (int cp = H0; cp < NCP; ++cp) contract(cp);
            if (more) {
#pragma unroll
                for (int cp = H0; cp < NCP; ++cp) breg[cp] = nblk[(2 * cp + h) * 32 + n32];
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float d = __builtin_fmaf(p.minus_two_unscaled, acc[j], __uint_as_float(qn[j]) + __uint_as_float(xn));
                bitsv[j] = __float_as_uint(fmaxf(d, 0.0f));
            }
        }
        // phase 1 (branch-free): threshold tests of this lane's 16 rows against its seed of the group
        const int jrel = grp * 32 + n32;
        uint32_t pm = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) pm |= (bitsv[j] <= thr[j] ? 1u : 0u) << j;
        pm &= jrel < nj ? live_rows : 0u;
        if (any_and && __any((pm & fast_rows) != 0)) {
            // one bitset word per candidate pair, all requested before the first is looked at (pairs that are
            // no candidates read the table's first word: one cached address for the whole wave)
            const uint32_t *bs = p.meta.bitsets;
            const int64_t wi = gid >> 5;
#pragma unroll
            for (int j0 = 0; j0 < 16; j0 += 8) {
                uint32_t wv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = j0 + u;
                    const bool c = ((pm & fast_rows) >> j) & 1u;
                    const int ps = pslot_s[8 * (j >> 2) + 4 * h + (j & 3)];
                    wv[u] = bs[c ? (int64_t)ps * p.meta.bitset_words + wi : 0];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = j0 + u;
                    if ((((pm & fast_rows) >> j) & 1u) && !((wv[u] >> (gid & 31)) & 1u)) pm &= ~(1u << j);
                }
            }
        }
        if (any_and && (pm & and_rows) != 0) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if (((pm & and_rows) >> j) & 1u) {
                    const int qr = qrow_s[8 * (j >> 2) + 4 * h + (j & 3)];
                    const int o_begin = p.others_off[qr], o_end = p.others_off[qr + 1];
                    bool ok = true;
                    for (int o = o_begin; o < o_end && ok; ++o) ok = has_label(p.meta, p.others[o], gid);
                    if (!ok) pm &= ~(1u << j);
                }
            }
        }
        // phase 2: queue the candidates (slot from the row's LDS counter)
        if (pm != 0) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if ((pm >> j) & 1u) {
                    const int row = 8 * (j >> 2) + 4 * h + (j & 3);
                    const uint32_t slot = atomicAdd(&pcnt[row], 1u);
                    pend[row * PC + slot] = ((uint64_t)bitsv[j] << 32) | (uint32_t)(j0 + jrel);
                }
            }
        }
        if (__any(pm != 0)) {
            wave_lds_sync();
            pcv = lane < 32 ? (int)pcnt[lane] : 0;
        }
        const bool last = grp + 1 == n_groups;
        if (__any(pcv > PC - 32) || (last && __any(pcv != 0))) drain(last);
    }
    __syncthreads();

    // ---- one sorted run of K keys per (query, segment)
    for (int r = 0; r < t.q_count; ++r)
        if (lane < K) p.runs[((int64_t)(t.gq_begin + r) * p.max_segs + seg) * K + lane] = best[r * KS + lane];
}

bool seed_select_supported(int dtype, int dim, bool f16_copy)
{
    return dtype == 0 ? (dim == 128 || dim == 192) : (f16_copy && (dim == 96 || dim == 128));
}

size_t seed_select_lds_bytes(int32_t K) { return (size_t)32 * 64 * 8 + (size_t)32 * (K | 1) * 8 + 4 * 32 * 4; }

void launch_seed_select(int dtype, const SeedSelParams &p, int n_tiles, hipStream_t s)
{
    if (n_tiles <= 0) return;
    const dim3 grid((unsigned)n_tiles * (unsigned)p.max_segs), block(64);
    const size_t lds = seed_select_lds_bytes(p.K);
    if (dtype == 0 && p.dim == 128) hipLaunchKernelGGL((seed_select_kernel<0, 4>), grid, block, lds, s, p);
    else if (dtype == 0 && p.dim == 192) hipLaunchKernelGGL((seed_select_kernel<0, 6>), grid, block, lds, s, p);
    else if (dtype == 1 && p.dim == 128) hipLaunchKernelGGL((seed_select_kernel<2, 8>), grid, block, lds, s, p);
    else if (dtype == 1 && p.dim == 96) hipLaunchKernelGGL((seed_select_kernel<2, 6>), grid, block, lds, s, p);
}

// Profiling only: how many of a graph query's seeds pass its AND predicate (the "distances computed" figure the
// search is accounted with counts them; the selection kernel tests only the seeds that reach a queue).
__global__ __launch_bounds__(64) void seed_pass_count_kernel(const int32_t *gq_query, const int32_t *gq_label, LabelMeta meta,
                                                             int32_t n_seeds, const int32_t *others_off,
                                                             const int32_t *others, int32_t *pass_count)
{
    const int gq = blockIdx.x, lane = threadIdx.x;
    const int qi = gq_query[gq], label = gq_label[gq];
    const int n = meta.S[label];
    const int ns = n_seeds < n ? n_seeds : n;
    const int64_t base = meta.O_HS[label];
    const int o_begin = others_off[qi], o_end = others_off[qi + 1];
    int cnt = 0;
    for (int j = lane; j < ns; j += 64) {
        const int g = meta.M_HS[base + (int64_t)(((uint64_t)j * (uint64_t)n) / (uint64_t)ns)];
        bool ok = true;
        for (int o = o_begin; o < o_end && ok; ++o) ok = has_label(meta, others[o], g);
        cnt += ok ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0) pass_count[gq] = cnt;
}

void launch_seed_pass_count(const int32_t *gq_query, const int32_t *gq_label, const LabelMeta &meta, int32_t n_seeds,
                            const int32_t *others_off, const int32_t *others, int32_t *pass_count, int n_gq, hipStream_t s)
{
    if (n_gq <= 0) return;
    hipLaunchKernelGGL(seed_pass_count_kernel, dim3(n_gq), dim3(64), 0, s, gq_query, gq_label, meta, n_seeds, others_off,
                       others, pass_count);
}

int seed_mfma_tile_of(int dtype, int dim, bool f16)
{
    if (dtype == 1 && !f16) return 32;
    const int steps = dtype == 1 ? (dim + 15) / 16 : (dim + 31) / 32;
    return seed_mfma_tile(dtype == 0 ? 0 : 2, steps);
}

bool seed_mfma_own(int dtype, int dim)
{
    return dtype == 1 ? (dim == 96 || dim == 128) : (dim == 128 || dim == 192);
}

// (the bound of the float32 proofs is that of 512 products)
bool seed_mfma_supported(int dtype, int dim) { return dim <= (dtype == 1 ? 256 : 512); }

// Dimensions without an instantiation of their own score on the matrix cores wherever the ordered kernel would score them, and
// beyond its lines (seed_dist_pays) from 192 seeds on.  Whole calls among others, before (gathered or ordered) -> on the matrix
// cores, at 192 / 384 / 1,024 / 4,096 seeds:
//   float32 dim 100    1 query      48 65 65 72 -> 42 43 44 47 us,   3,000 queries   91 115 123 263 -> 77 78 73 92
//   float32 dim 200   64 queries    72 99 109 124 -> 60 61 61 65,    3,000 queries   114 142 238 719 -> 99 100 97 120
//   float32 dim 200   64 AND pairs  71 95 176 649 -> 68 70 71 88,    3,000 AND pairs 119 147 231 659 -> 110 113 117 161
//   uint8 dim 112      1 query      46 47 47 55 -> 39 40 41 42,      3,000 AND pairs 84 98 98 150 -> 75 81 85 120
//   uint8 dim 400      1 query      52 83 82 89 -> 44 44 43 43,      3,000 queries   121 145 193 372 -> 89 92 95 108
// Lists of more than 48 entries re-score more, and ordered distances, where they are given, need none of that: from four
// million pairs on (dim 200, 3,000 queries x 4,096 seeds 743 -> 150 us).
bool seed_mfma_pays(int dtype, int dim, int32_t itopk, int n_seeds, int64_t n_gq)
{
    if (!seed_mfma_supported(dtype, dim)) return false;
    if (itopk > 48) return (int64_t)n_seeds * n_gq >= (int64_t)1 << 22;
    return n_seeds >= kSeedMfmaLeast;
}

// Dimensions without an instantiation of their own: the next larger one, from the copy of the seeds.
template <int DT, int NCP> static void launch_seed_mfma_nofit(const SeedParams &p, dim3 grid, hipStream_t s)
{
    if (p.chunk_seeds == 4 * kSeedMfmaChunk) hipLaunchKernelGGL((seed_mfma_kernel<DT, NCP, true, 16, false>), grid, dim3(64), 0, s, p);
    else if (p.chunk_seeds == 32) hipLaunchKernelGGL((seed_mfma_kernel<DT, NCP, true, 1, false>), grid, dim3(64), 0, s, p);
    else hipLaunchKernelGGL((seed_mfma_kernel<DT, NCP, true, 4, false>), grid, dim3(64), 0, s, p);
}
template <int DT> static void launch_seed_mfma_any(const SeedParams &p, dim3 grid, hipStream_t s)
{
    const int steps = (p.blk_chunks + 1) / 2;
    if (steps <= 2) launch_seed_mfma_nofit<DT, 2>(p, grid, s);
    else if (steps <= 4) launch_seed_mfma_nofit<DT, 4>(p, grid, s);
    else if (steps <= 8) launch_seed_mfma_nofit<DT, 8>(p, grid, s);
    else if (steps <= 12) launch_seed_mfma_nofit<DT, 12>(p, grid, s);
    else launch_seed_mfma_nofit<DT, 16>(p, grid, s);
}

void launch_seed_mfma(int dtype, const SeedParams &p, int n_tiles, hipStream_t s)
{
    if (n_tiles <= 0) return;
    const dim3 grid((unsigned)n_tiles * (unsigned)p.max_chunks), block(64);
    // instantiations for the operand sources and for the seeds per wave (p.chunk_seeds: 128, or 32 or 512 with the copy)
    const bool cached = p.seed_blk != nullptr;
    if (!seed_mfma_own(dtype, p.dim)) {
        if (dtype == 0) launch_seed_mfma_any<0>(p, grid, s);
        else launch_seed_mfma_any<2>(p, grid, s);
        return;
    }
#define VF_LAUNCH_SEED(DT_, NCP_) \
    do { \
        if (cached && p.chunk_seeds == 4 * kSeedMfmaChunk) hipLaunchKernelGGL((seed_mfma_kernel<DT_, NCP_, true, 16>), grid, block, 0, s, p); \
        else if (cached && p.chunk_seeds == 32) hipLaunchKernelGGL((seed_mfma_kernel<DT_, NCP_, true, 1>), grid, block, 0, s, p); \
        else if (cached) hipLaunchKernelGGL((seed_mfma_kernel<DT_, NCP_, true, 4>), grid, block, 0, s, p); \
        else if constexpr (DT_ != 2) hipLaunchKernelGGL((seed_mfma_kernel<DT_, NCP_, false, 4>), grid, block, 0, s, p); \
    } while (0)
    if (dtype == 0 && p.dim == 128) VF_LAUNCH_SEED(0, 4);
    else if (dtype == 0) VF_LAUNCH_SEED(0, 6);
    else if (p.seed_f16 && p.dim == 128) VF_LAUNCH_SEED(2, 8);
    else if (p.seed_f16) VF_LAUNCH_SEED(2, 6);
    else if (p.dim == 128) VF_LAUNCH_SEED(1, 16);
    else VF_LAUNCH_SEED(1, 12);
#undef VF_LAUNCH_SEED
}

// The float32 copy of the seeds as binary16 (nch16 chunks of 8 components), times scale; *err2_max = the largest |x - x^|^2 of the
// unscaled vectors (its bits; a NaN's are above all others), which the proofs allow for.  One thread per seed.
__global__ void seed_pack_f16_kernel(const uint4 *blk32, int64_t n_vec, int32_t nch16, float scale, uint4 *blk16, uint32_t *err2_max)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_vec) return;
    const int64_t g = t >> 5;
    const int v = (int)(t & 31);
    const float unscale = 1.0f / scale;   // (a power of two)
    float e2 = 0.f;
    for (int c = 0; c < nch16; ++c) {
        const uint4 a = blk32[(g * (2 * nch16) + 2 * c) * 32 + v], b = blk32[(g * (2 * nch16) + 2 * c + 1) * 32 + v];
        const uint4 r = scaled_half8(a, b, scale);
        const v8h_seed x = __builtin_bit_cast(v8h_seed, r);
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float d = __uint_as_float(w[i]) - (float)x[i] * unscale;
            e2 += d * d;
        }
        blk16[(g * nch16 + c) * 32 + v] = r;
    }
    uint32_t most = __float_as_uint(e2);   // (whole halves of a wave: groups have 32 seeds)
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) { const uint32_t other = (uint32_t)__shfl_xor((int)most, o, 32); most = other > most ? other : most; }
    if (v == 0) atomicMax(err2_max, most);
}

void launch_seed_pack_f16(const uint4 *blk32, int64_t n_groups, int32_t nch16, float scale, uint4 *blk16, uint32_t *err2_max, hipStream_t s)
{
    if (n_groups <= 0) return;
    hipLaunchKernelGGL(seed_pack_f16_kernel, dim3((unsigned)((n_groups * 32 + 255) / 256)), dim3(256), 0, s, blk32,
                       n_groups * 32, nch16, scale, blk16, err2_max);
}

// The same from the vector table where no float32 copy is kept, with the norms of the unrounded vectors (0 for a seed that does not
// exist): map[g * 32 + v] is the seed's row, grp_cnt[g] the seeds of group g.  One thread per seed; a lane's next 32 bytes are in the
// line it has just read.
__global__ void seed_rows_f16_kernel(const float *X, int32_t dim, const int32_t *map, const int32_t *grp_cnt, int64_t n_vec, int32_t nch16,
                                     float scale, uint4 *blk16, float *norm, uint32_t *err2_max)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_vec) return;
    const int64_t g = t >> 5;
    const int v = (int)(t & 31);
    const bool valid = v < grp_cnt[g];
    const float *row = X + (int64_t)(valid ? map[t] : 0) * dim;
    const float unscale = 1.0f / scale;
    float e2 = 0.f, acc = 0.f;
    for (int c = 0; c < nch16; ++c) {
        uint4 a = make_uint4(0, 0, 0, 0), b = a;
        if (valid && 8 * c < dim) a = *(const uint4 *)(row + 8 * c);
        if (valid && 8 * c + 4 < dim) b = *(const uint4 *)(row + 8 * c + 4);
        const uint4 r = scaled_half8(a, b, scale);
        const v8h_seed x = __builtin_bit_cast(v8h_seed, r);
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float f = __uint_as_float(w[i]), d = f - (float)x[i] * unscale;
            acc += f * f;
            e2 += d * d;
        }
        blk16[(g * nch16 + c) * 32 + v] = r;
    }
    norm[t] = acc;
    uint32_t most = __float_as_uint(e2);
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) { const uint32_t other = (uint32_t)__shfl_xor((int)most, o, 32); most = other > most ? other : most; }
    if (v == 0) atomicMax(err2_max, most);
}

void launch_seed_rows_f16(const void *X, int32_t dim, const int32_t *map, const int32_t *grp_cnt, int64_t n_groups, int32_t nch16, float scale,
                          uint4 *blk16, float *norm, uint32_t *err2_max, hipStream_t s)
{
    if (n_groups <= 0) return;
    hipLaunchKernelGGL(seed_rows_f16_kernel, dim3((unsigned)((n_groups * 32 + 255) / 256)), dim3(256), 0, s, (const float *)X, dim, map, grp_cnt,
                       n_groups * 32, nch16, scale, blk16, norm, err2_max);
}

// An interleaved float32 copy (of the scan lists; groups of 32, 2 * nch16 chunks of 4 components) rounded to
// bfloat16 (nch16 chunks of 8 components); err2[group * 32 + v] = |x - bf16(x)|^2.  One thread per vector.
__global__ void seed_pack_bf16_kernel(const uint4 *blk32, int64_t n_vec, int32_t nch16, uint4 *blk16, float *err2)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_vec) return;
    const int64_t g = t >> 5;
    const int v = (int)(t & 31);
    float e2 = 0.f;
    for (int c = 0; c < nch16; ++c) {
        const uint4 a = blk32[(g * (2 * nch16) + 2 * c) * 32 + v], b = blk32[(g * (2 * nch16) + 2 * c + 1) * 32 + v];
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint32_t r[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float f = __uint_as_float(w[i]);
            r[i] = bf16_rn_bits(f);
            const float d = f - __uint_as_float(r[i] << 16);
            e2 += d * d;
        }
        blk16[(g * nch16 + c) * 32 + v] = make_uint4(r[0] | (r[1] << 16), r[2] | (r[3] << 16), r[4] | (r[5] << 16), r[6] | (r[7] << 16));
    }
    err2[t] = e2;
}

void launch_seed_pack_bf16(const uint4 *blk32, int64_t n_groups, int32_t nch16, uint4 *blk16, float *err2, hipStream_t s)
{
    if (n_groups <= 0) return;
    hipLaunchKernelGGL(seed_pack_bf16_kernel, dim3((unsigned)((n_groups * 32 + 255) / 256)), dim3(256), 0, s, blk32,
                       n_groups * 32, nch16, blk16, err2);
}

__global__ void seed_map_kernel(const int32_t *M_HS, const int64_t *slot_base, const int32_t *slot_n, int32_t n_seeds,
                                const int32_t *grp_slot, const int32_t *grp_j0, int64_t n_groups, int32_t *seed_map)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_groups * 32) return;
    const int64_t g = t >> 5;
    const int slot = grp_slot[g];
    const int n = slot_n[slot];
    const int ns = n_seeds < n ? n_seeds : n;
    const int j = grp_j0[g] + (int)(t & 31);
    seed_map[t] = j < ns ? M_HS[slot_base[slot] + (int64_t)(((uint64_t)j * (uint64_t)n) / (uint64_t)ns)] : 0;
}

void launch_seed_map(const int32_t *M_HS, const int64_t *slot_base, const int32_t *slot_n, int32_t n_seeds,
                     const int32_t *grp_slot, const int32_t *grp_j0, int64_t n_groups, int32_t *seed_map, hipStream_t s)
{
    if (n_groups <= 0) return;
    hipLaunchKernelGGL(seed_map_kernel, dim3((unsigned)((n_groups * 32 + 255) / 256)), dim3(256), 0, s, M_HS, slot_base,
                       slot_n, n_seeds, grp_slot, grp_j0, n_groups, seed_map);
}

// One thread per row: sum of (x - 128)^2 over the bytes.
__global__ void row_norm_u8_kernel(const uint8_t *X, int32_t dim, int64_t n, uint32_t *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint4 *x = (const uint4 *)(X + i * dim);
    int acc = 0;
    for (int e = 0; e < dim / 16; ++e) {
        const uint4 v = x[e];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int d = (int)((w[a] >> (8 * b)) & 0xFFu) - 128;
                acc += d * d;
            }
    }
    out[i] = (uint32_t)acc;
}

void launch_row_norms_u8(const void *X, int32_t dim, int64_t n, uint32_t *out, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(row_norm_u8_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const uint8_t *)X, dim, n, out);
}

bool seed_dist_own(int dtype, int dim)
{
    const int nch = dim * (dtype == 0 ? 1 : 4) / kChunkBytes;
    return nch == 8 || nch == 12 || nch == 16 || nch == 24 || nch == 32;
}

// Whether a launch of the dense kernel pays.  Dimensions with an instantiation of their own: always.  Others (an index has
// vectors of at most 62 chunks) score n_gq queries with the chunks of the next larger one, and leave the distances where
// the beam kernel, which would gather its seeds itself in the same launch, has to read them: that needs enough seeds per
// query, and beyond 32 chunks, where a query no longer fits into registers beside the sums, few enough queries.  Whole
// calls among others, gathering -> dense (at the lines for up to 32 chunks a call that is waited for is 10 us faster):
//   float32 dim 36     512 queries x   128 seeds   53 ->  59 us, x   192  57 ->  58, x   512  76 ->  59
//   float32 dim 100     64 queries x   256 seeds   62 ->  72 us, x   384  70 ->  73, x 1,024 109 ->  72
//   float32 dim 200      1 query   x   512 seeds  102 -> 100 us, x 1,024 158 ->  99
//                      512 queries x 1,024 seeds  217 -> 239 us, x 4,096 685 -> 536
//                    3,000 queries x 1,024 seeds  248 -> 433 us, x 4,096 721 -> 1,105
//   uint8 dim 528       64 queries x   256 seeds   80 -> 110 us, x   512 113 -> 109
//   uint8 dim 992    3,000 queries x 1,024 seeds  491 -> 519 us, x 4,096 1,578 -> 1,266
// Queries with a predicate test it first when they gather, and score only the seeds that pass: batches of mostly such
// queries take more seeds (AND pairs, gathering -> dense):
//   float32 dim 36     512 queries x   384 seeds   81 ->  91 us, x 1,024 118 -> 103
//   float32 dim 100    512 queries x   384 seeds   83 ->  98 us, x 2,048 199 -> 166
//   float32 dim 200    512 queries x 4,096 seeds  425 -> 583 us, x 8,192 762 -> 686
//   uint8 dim 528       64 queries x   384 seeds   85 -> 127 us, x 2,048 214 -> 215, x 4,096 484 -> 280
bool seed_dist_pays(int dtype, int dim, int n_seeds, int64_t n_gq, int64_t n_and)
{
    const int nch = dim * (dtype == 0 ? 1 : 4) / kChunkBytes;
    if (seed_dist_own(dtype, dim)) return true;
    if (nch < 1 || nch > 64) return false;
    if (2 * n_and > n_gq) return n_seeds >= (nch <= 16 ? 1024 : nch <= 32 || dtype == 0 ? 2048 : 8192);
    if (nch <= 16) return n_seeds >= 192;
    if (nch <= 32) return n_seeds >= 384;
    if (dtype == 1) return n_gq <= 512 && n_seeds >= std::max<int64_t>(1024, 8 * n_gq);
    return n_seeds >= 512 && (nch <= 48 || n_gq <= 1024 || n_seeds >= 2048);
}

// Dimensions without an instantiation of their own take the next larger one with the missing chunks zeroed: a few
// scalar selects per seed (1,200 graph queries x 777 seeds, dim 100: the beam kernel gathering its seeds instead
// took 214 us, both together 176 us).
template <int DT> static void launch_seed_dt(const SeedParams &p, int nch, unsigned grid, hipStream_t s)
{
#define VF_SEED_DIST(NCH_, FIT_) hipLaunchKernelGGL((seed_dist_kernel<DT, NCH_, FIT_>), dim3(grid), dim3(64), 0, s, p)
    if (nch == 8) VF_SEED_DIST(8, true);
    else if (nch == 12) VF_SEED_DIST(12, true);
    else if (nch == 16) VF_SEED_DIST(16, true);
    else if (nch == 24) VF_SEED_DIST(24, true);
    else if (nch == 32) VF_SEED_DIST(32, true);
    else if (nch < 8) VF_SEED_DIST(8, false);
    else if (nch < 16) VF_SEED_DIST(16, false);
    else if (nch < 24) VF_SEED_DIST(24, false);
    else if (nch < 32) VF_SEED_DIST(32, false);
    else if (nch <= 48) VF_SEED_DIST(48, false);
    else VF_SEED_DIST(64, false);
#undef VF_SEED_DIST
}

void launch_seed_dist(int dtype, const SeedParams &p, int n_tiles, hipStream_t s)
{
    if (n_tiles <= 0) return;
    const int nch = p.dim * (dtype == 0 ? 1 : 4) / kChunkBytes;
    const unsigned grid = (unsigned)n_tiles * (unsigned)p.max_chunks;
    if (dtype == 0) launch_seed_dt<0>(p, nch, grid, s);
    else launch_seed_dt<1>(p, nch, grid, s);
}

}  // namespace vf
