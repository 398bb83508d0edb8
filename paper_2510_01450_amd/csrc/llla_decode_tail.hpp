// What the matrix-core decode kernels have in common after (and before) their pass over the cache: how a cache is cut into the
// shares of workgroups, the merge of the waves of a workgroup, the record a workgroup leaves, the merge of a head's records, and the
// solve and output of a head.
//
// Moments of a head: omega, mu~, sum w v, and 16x16 tiles in the MFMA accumulator layout -- Sigma~ (upper triangle, row by row), then
// G~ = sum w k v^T row-major -- all relative to 2^m.  PERM: element n of feature block I is feature NB n + I instead of 16 I + n (the
// order in which the fp32 kernels load their operands).
#pragma once

#include "llla_dual.hpp"
#include "llla_mfma_common.hpp"
#include "llla_mfma_solve128.hpp"
#include <algorithm>
#include <type_traits>

namespace llla {
namespace mfma {

constexpr int DEC_NT = 256;                               // threads of every decode workgroup

template <int D>
struct DecShape {
    static constexpr int NB = D / 16;                     // 16-wide feature blocks
    static constexpr int NSIG = NB * (NB + 1) / 2;
    static constexpr int NTILES = NSIG + NB * NB;
    static constexpr int HDR = 64 + 2 * D;                // record: [m, omega, ..], mu~ at 64, sum w v at 64 + D, tiles at HDR
    static constexpr int REC_F = HDR + NTILES * 256;
};

// ---- shares ----------------------------------------------------------------------------------------------------------
// Even (slots == 0): every (batch, head) gets nsplit workgroups, grid (nsplit, B H); a sequence's own length is divided evenly
// over them.  With nsplit == 1 a workgroup solves its head and writes the output itself.
// Flat (slots > 0), grid (slots, H): the keys of all sequences of a head index, one sequence behind the other, are cut into slots
// equal shares; a workgroup walks through the one or more sequences that its share touches and leaves a record for each.
// Lengths that differ, or a number of heads that does not divide the GPU's slots, then leave no workgroup idle: with even
// parts a batch with lengths uniform in [L/8, L] takes as long as if all had length L (1.8 times its keys' worth).
// Positions are counted in units of `unit` keys, sequences padded to whole units, so that no piece is smaller than a unit.
struct DecSplit {
    const int32_t *seqlens;
    int B, H, L_max;
    int nsplit;            // even: workgroups per head
    int slots;             // flat: workgroups per head index
    int unit;              // flat: keys per unit
    int units_min;         // flat: fewest units worth a workgroup
    int max_split;         // flat: most pieces of a sequence (about)
};

constexpr int FLAT_MAX_B = 256;                           // more sequences with lengths of their own: the even cut

struct DecPiece {
    int b, h, bh, L;       // sequence, head, length
    int k0, k1;            // keys [k0, k1) of it
    int rec;               // index of the record
};

// Start of sequence b (in units), the sum of all and the share of a workgroup
struct FlatPlan { int start, total, share; };

__device__ inline int seq_len(const DecSplit &s, int b) { return s.seqlens ? min(max(s.seqlens[b], 1), s.L_max) : s.L_max; }
__device__ inline int seq_units(const DecSplit &s, int b) { return (seq_len(s, b) + s.unit - 1) / s.unit; }

__device__ inline int flat_share(const DecSplit &s, int total, int longest)
{
    const int even = (total + s.slots - 1) / s.slots, cap = (longest + s.max_split - 1) / s.max_split;
    return max(max(even, cap), s.units_min);
}

// `b_of`: the sequence whose start is asked for, or -1 for the one that holds position pos(share)
template <class Pos>
__device__ inline FlatPlan flat_plan(const DecSplit &s, int &b_of, Pos pos)
{
    FlatPlan r;
    if (s.seqlens == nullptr) {
        const int u = (s.L_max + s.unit - 1) / s.unit;
        r.total = u * s.B;
        r.share = flat_share(s, r.total, u);
        if (b_of < 0) b_of = min(pos(r.share) / u, s.B - 1);
        r.start = b_of * u;
        return r;
    }
    const int lane = threadIdx.x % 64;
    int u[FLAT_MAX_B / 64], incl[FLAT_MAX_B / 64], total = 0, longest = 0;
#pragma unroll
    for (int c = 0; c < FLAT_MAX_B / 64; ++c) {
        u[c] = incl[c] = 0;
        if (64 * c < s.B) {                               // wave-uniform
            const int b = 64 * c + lane;
            u[c] = b < s.B ? seq_units(s, b) : 0;
            int x = u[c];
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(x, off);
                if (lane >= off) x += y;
            }
            incl[c] = total + x;
            longest = max(longest, u[c]);
            total = __builtin_amdgcn_readlane(incl[c], 63);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off));
    r.total = total;
    r.share = __builtin_amdgcn_readfirstlane(flat_share(s, total, longest));
    if (b_of < 0) {                                       // the first sequence that ends beyond the position
        const int at = pos(r.share);
        int b = 0;
#pragma unroll
        for (int c = 0; c < FLAT_MAX_B / 64; ++c)
            if (64 * c < s.B) b += __builtin_popcountll(__builtin_amdgcn_ballot_w64(64 * c + lane < s.B && incl[c] <= at));
        b_of = min(b, s.B - 1);
    }
    r.start = 0;
#pragma unroll
    for (int c = 0; c < FLAT_MAX_B / 64; ++c)
        if ((b_of >> 6) == c) r.start = __builtin_amdgcn_readlane(incl[c] - u[c], b_of & 63);
    return r;
}

// Calls body(piece) for every piece of this workgroup's share, with a barrier between two of them (the body owns the workgroup's
// LDS).  Everything that decides the control flow is wave-uniform and the same in all waves.  ONE: even cut, one piece.  heads_first: flat, in a grid
// (H, slots) instead of (slots, H).
template <bool ONE, class Body>
__device__ __forceinline__ void for_pieces(const DecSplit &s, Body body, bool heads_first = false)
{
    DecPiece pc;
    const bool flat = !ONE && s.slots != 0;
    int start = 0, stop = 0, end = 0;
    if (!flat) {
        pc.bh = blockIdx.y;
        pc.b = pc.bh / s.H;
        pc.h = pc.bh % s.H;
        pc.L = __builtin_amdgcn_readfirstlane(seq_len(s, pc.b));
        const int part = (pc.L + s.nsplit - 1) / s.nsplit;
        pc.k0 = min((int)blockIdx.x * part, pc.L);
        pc.k1 = min(pc.k0 + part, pc.L);
        pc.rec = pc.bh * s.nsplit + blockIdx.x;
    } else {
        const int x = (int)(heads_first ? blockIdx.y : blockIdx.x), y = (int)(heads_first ? blockIdx.x : blockIdx.y);
        int b = -1;
        const FlatPlan plan = flat_plan(s, b, [x](int share) { return x * share; });
        pc.b = __builtin_amdgcn_readfirstlane(b);
        pc.h = y;
        const int share = __builtin_amdgcn_readfirstlane(plan.share), at = x * share;
        end = min(at + share, __builtin_amdgcn_readfirstlane(plan.total));
        if (at >= end) return;
        start = __builtin_amdgcn_readfirstlane(plan.start);
        pc.L = __builtin_amdgcn_readfirstlane(seq_len(s, pc.b));
        stop = min(end, start + (pc.L + s.unit - 1) / s.unit);
        pc.k0 = (at - start) * s.unit;
        pc.k1 = min((stop - start) * s.unit, pc.L);
        pc.bh = pc.b * s.H + pc.h;
        pc.rec = y * (s.slots + s.B) + x + pc.b;
    }
    for (;;) {
        body(pc);
        if (ONE || stop == end) break;
        __syncthreads();
        start = stop;
        ++pc.b;
        ++pc.rec;
        pc.bh += s.H;
        pc.L = __builtin_amdgcn_readfirstlane(seq_len(s, pc.b));
        stop = min(end, start + (pc.L + s.unit - 1) / s.unit);
        pc.k0 = 0;
        pc.k1 = min((stop - start) * s.unit, pc.L);
    }
}

// The lane index as a value of its own for every piece: what a body derives from it would otherwise be kept in registers across
// the pieces (the d = 128 kernel spilled 64 registers that way).
__device__ inline int piece_lane()
{
    int lane = threadIdx.x % 64;
    asm volatile("" : "+v"(lane));
    return lane;
}

constexpr int MAX_RECORDS = 64;                           // of a head: a lane each in the merge
struct DecRecords { int first, count; };
__device__ inline DecRecords dec_records(const DecSplit &s, int bh)
{
    if (s.slots == 0) return DecRecords{bh * s.nsplit, s.nsplit};
    int b = bh / s.H;
    const int h = bh % s.H;
    const FlatPlan plan = flat_plan(s, b, [](int) { return 0; });
    const int x0 = plan.start / plan.share, x1 = (plan.start + seq_units(s, b) - 1) / plan.share;
    return DecRecords{__builtin_amdgcn_readfirstlane(h * (s.slots + s.B) + x0 + b), __builtin_amdgcn_readfirstlane(x1 - x0 + 1)};
}

// Host side.  Which cut a call takes: room = records that the scratch holds; gpu_slots = workgroups the GPU holds at once.
// Flat where the lengths differ, or where the even cut's last round would leave more than a fifth of the slots idle.
inline DecSplit choose_split(const Problem &p, int nsplit, size_t room, int gpu_slots, int unit, int keys_min, int max_split)
{
    const int bh = p.B * p.H;
    DecSplit s{p.seqlens, p.B, p.H, p.n, nsplit, 0, unit, std::max(keys_min / unit, 1), max_split};
    const int slots = std::max(gpu_slots / p.H, 1);
    const bool fits = p.B >= 2 && (size_t)(slots + p.B) * p.H <= room && (long long)p.B * (p.n / keys_min) > 1;
    const long long wgs = (long long)bh * nsplit, rounds = (wgs + gpu_slots - 1) / gpu_slots;
    const bool uneven = wgs > gpu_slots && 5 * wgs < 4 * rounds * gpu_slots;
    if (fits && (p.seqlens ? p.B <= FLAT_MAX_B : uneven)) s.slots = slots;
    return s;
}
inline size_t flat_records(int B, int H, int gpu_slots) { return (size_t)(std::max(gpu_slots / H, 1) + B) * H; }

// ---- exchanges inside a wave ------------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

__device__ __forceinline__ float wave_max_dpp(float x)    // maximum over the wave, in every lane
{
    x = fmaxf(x, dpp_f<0xB1>(x));
    x = fmaxf(x, dpp_f<0x4E>(x));
    x = fmaxf(x, dpp_f<0x124>(x));
    x = fmaxf(x, dpp_f<0x128>(x));
    x = fmaxf(x, rows_1_3_from_rows_0_2(x));
    x = fmaxf(x, rows_2_3_from_row_1(x));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}

// ---- merge, solve, output ----------------------------------------------------------------------------------------------
struct HeadOut {
    const void *q;
    void *o;
    int out_bf16;
    float lambda;
};

// LDS of one head: NBUF copies of the tiles (the merge of a workgroup's waves), NW copies of the vectors, the solve's scratch
template <int D, int NBUF, int NW>
struct HeadLds {
    float tiles[NBUF][DecShape<D>::NTILES * 256];
    float mu[NW][D], yv[NW][D];
    float mw[4], om[4];
    float sc[D == 128 ? 16 * SC_PITCH + D + 4 : 4];
};

// The ridge of attempt a at a solve: lambda + eta S~_ii.  The centred matrix carries the rounding of moments of the size of |k|^2: some
// 2^-24 of them, or 2^-11 where the weighted keys are 16-bit floats.  Where that exceeds lambda a pivot comes out below lambda / 2,
// and a factorisation that only raises such pivots amplifies the noise of their columns block by block until it overflows (a common
// offset of 100 in 64 features: 23 of 48 outputs not finite).  The solve is then repeated with a ridge of the size of that noise, feature by
// feature; the last one dominates any.  All arithmetic before the first such pivot is that of lambda alone.
constexpr int SOLVE_TRIES = 5;
__device__ inline float noise_ridge(int attempt) { return attempt == 0 ? 0.f : __builtin_ldexpf(1.f, 6 * attempt - 28); }

// Second moments of 2^-102 and less have terms that matrix cores read as zero where they are taken in three bf16.  That matters where the ridge is
// no larger: then keys and query are taken 2^r times, which brings the largest second moment to about one and leaves the output as it is.
// (32 fp32 features of size 2^-60, 100 keys: 2.7e-5 off without it, 1e-7 with it and on fp32 MFMA.)  In LDS, in front of the solve: a choice between the
// loads and the factorisation held up every call by 0.2 us, here it is 0.1 (16 heads x 4096 bf16 keys).
constexpr float RIDGE_SMALL = 0x1p-80f;
template <int D, class Lds>
__device__ __forceinline__ int enlarge_keys(Lds &lds, int wave, int lane)      // (all four waves)
{
    using S = DecShape<D>;
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < 4 * S::NB; ++i) top = fmaxf(top, fabsf(lds.tiles[0][upper_tile<S::NB>(i / 4, i / 4) * 256 + lane * 4 + i % 4]));
    const int r = max(-__builtin_amdgcn_frexp_expf(wave_max_dpp(top)) / 2, 0), tid = wave * 64 + lane;
    __syncthreads();
    for (int i = tid; i < S::NTILES * 256; i += DEC_NT) lds.tiles[0][i] = __builtin_ldexpf(lds.tiles[0][i], i < S::NSIG * 256 ? 2 * r : r);
    if (tid < D) lds.mu[0][tid] = __builtin_ldexpf(lds.mu[0][tid], r);
    __syncthreads();
    return r;
}

// What a lane needs of the head's query (features 16 P + 4 g + t; at d = 128 16 P + n), requested by the caller long before the solve: a trip to memory is a tenth of it.
template <int D>
struct QueryPart { static constexpr int PER = D == 128 ? 1 : 4; float v[D / 16][PER]; };
template <int D, typename TI, bool PERM>
__device__ __forceinline__ QueryPart<D> load_query(const HeadOut &out, int bh, int lane)
{
    constexpr int NB = D / 16;
    const TI *qp = static_cast<const TI *>(out.q) + (size_t)bh * D;
    constexpr int PER = QueryPart<D>::PER;
    QueryPart<D> q;
#pragma unroll
    for (int i = 0; i < PER * NB; ++i) {
        const int P = i / PER, n = PER == 1 ? lane % 16 : 4 * (lane / 16) + i % PER;
        const TI v = qp[PERM ? NB * n + P : 16 * P + n];
        if constexpr (sizeof(TI) == 2) q.v[P][i % PER] = bf16_to_f32(v);
        else q.v[P][i % PER] = v;
    }
    return q;
}

// Solve and output of one head whose merged moments lie in lds.tiles[0], lds.mu[0], lds.yv[0], lds.om[0].  Called by all four
// waves after a barrier.
// The intercept is eliminated first: with the centred Sigma_c = Sigma~ - mu~ mu~^T / omega, q_c = q - mu~ / omega, G_c = G~ -
// mu~ (sum w v)^T / omega and Sigma_c + lambda I = U^T U the output is sum w v / omega + (U^{-T} G_c)^T U^{-T} q_c: every pivot is
// lambda or more however few keys the head sees.  Eliminated last it leaves omega - mu~^T (Sigma~ + lambda I)^{-1} mu~, which cancels
// to zero in fp32 where one key far from the origin holds nearly all the weight (a common offset of 100 in the 32 features of 1000
// fp32 keys, ridge 10^-2: 14 of 48 outputs were not finite).
// q_c and the columns of G_c are further block columns of the factorisation, so there is no back substitution; wave W
// carries column W of G_c and repeats the factorisation itself (every wave has a SIMD of its own, and an exchange
// of tiles would cost the barriers that this saves).  What bounds it is the serial chain of the diagonal tiles.  One wave with both
// substitutions on the vector ALU: 64 heads of 1024 to 8192 fp32 keys, d = 64, 86.7 instead of 81.2 us; 256 heads x 4096 bf16
// keys, d = 32, 53.7 instead of 51.5.
// Of 15 500 cycles at d = 64 the diagonal tiles were 2300 each (on the way through LDS and back 500, elimination 1420, inverse 320), the products 4700,
// loading and the query's trip to memory 1200.  Now tiles are symmetric as loaded and become rows by lane exchanges (230), products run on
// 16-bit MFMA from operands in three bf16, and the query is on its way while the records are merged: us, 16 heads x 4096 bf16 keys 23.7 -> 23.4,
// 16 x 512 (one workgroup per head) 17.4 -> 16.3, 512 x 700 30.4 -> 28.7; fp32 16 x 4096 29.8 -> 28.7; errors 0.6 to 1.0 times those before.
// (The columns dealt over the four waves, tiles handed on through LDS with two barriers per step: 23.9, 17.2, 28.5, 29.2; d = 128 53.7 -> 56.3.)
template <int D, typename TI, bool PERM, class Lds>
__device__ __forceinline__ void solve_and_store(Lds &lds, const HeadOut &out, QueryPart<D> q, int bh, int wave, int lane)
{
    using S = DecShape<D>;
    constexpr int NB = S::NB;
    static_assert(NB <= 4, "a column of G_c per wave");
    const int g = lane / 16, nn = lane % 16;
    float lambda = out.lambda;
    if (lambda < RIDGE_SMALL) {                           // (a scalar branch)
        const int r = enlarge_keys<D>(lds, wave, lane);
        lambda = __builtin_ldexpf(lambda, 2 * r);
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i) q.v[i / 4][i % 4] = __builtin_ldexpf(q.v[i / 4][i % 4], r);
    }
    if (wave >= NB) return;                               // (scalar branches: what follows contains MFMAs)
    const float oinv = 1.f / lds.om[0], yc = lds.yv[0][16 * wave + nn], floor = 0.5f * lambda;
    float o = 0.f;
    for (int attempt = 0; attempt < SOLVE_TRIES; ++attempt) {
        asm volatile("" ::: "memory");                    // (the moments are read again: not kept in registers for a second attempt)
        const float eta = noise_ridge(attempt);
        f32x4 acc[S::NSIG], x[2][NB];                     // x: the wave's column of G_c; q_c in column 0
        float mc[NB];
#pragma unroll
        for (int J = 0; J < NB; ++J) mc[J] = lds.mu[0][16 * J + nn];
#pragma unroll
        for (int P = 0; P < NB; ++P) {
            const f32x4 mr = oinv * *reinterpret_cast<const f32x4 *>(&lds.mu[0][16 * P + 4 * g]);
            const f32x4 gt = *reinterpret_cast<const f32x4 *>(&lds.tiles[0][(S::NSIG + NB * P + wave) * 256 + lane * 4]);
#pragma unroll
            for (int J = P; J < NB; ++J) {
                const float *tile = &lds.tiles[0][upper_tile<NB>(P, J) * 256];
                const f32x4 st = *reinterpret_cast<const f32x4 *>(tile + lane * 4);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    float v = fmaf(mr[t], mc[J], -st[t]);
                    if (J == P) {                         // symmetrised: element [nn][4 g + t] beside [4 g + t][nn]
                        const float other = fmaf(oinv * mc[J], lds.mu[0][16 * P + 4 * g + t], -tile[(16 * (nn >> 2) + 4 * g + t) * 4 + (nn & 3)]);
                        v = 0.5f * (v + other);
                        v -= (nn == 4 * g + t) ? fmaf(eta, st[t], lambda) : 0.f;
                    }
                    acc[upper_tile<NB>(P, J)][t] = v;
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                x[0][P][t] = fmaf(mr[t], yc, -gt[t]);
                x[1][P][t] = nn == 0 ? mr[t] - q.v[P][t] : 0.f;
            }
        }
        // Every column of G_c, and q_c, times a power of two of its own, which takes it out of the way of three bf16 at both ends of the range (the
        // third term of a value below 2^-110 is subnormal, which matrix cores read as zero; the first of one above 2^127.99 infinite): as on
        // fp32 MFMA, what one value feature holds is nothing to the others.
        auto column_exponent = [&](const f32x4 (&c)[NB]) {
            float top = 0.f;
#pragma unroll
            for (int i = 0; i < 4 * NB; ++i) top = fmaxf(top, fabsf(c[i / 4][i % 4]));
            return max(min(__builtin_amdgcn_frexp_expf(rows_allmax(top)), 120), -120);      // (0 for 0 and infinity)
        };
        const int eg = column_exponent(x[0]), eq = column_exponent(x[1]);
        const float sg = __builtin_ldexpf(1.f, -eg), sq = __builtin_ldexpf(1.f, -eq);
#pragma unroll
        for (int I = 0; I < NB; ++I) { x[0][I] *= sg; x[1][I] *= sq; }
        const float low = factorise_columns<NB, 2>(acc, g, nn, floor, x);
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i) s = fmaf(x[0][i / 4][i % 4], row_bcast<0>(x[1][i / 4][i % 4]), s);
        s = __builtin_ldexpf(rows_allsum(s), eg + __builtin_amdgcn_update_dpp(0, eq, 0x150, 0xf, 0xf, true));      // (eq of lane 0 of the row)
        o = fmaf(oinv, yc, s);
        if (__builtin_amdgcn_ballot_w64(low < floor) == 0) break;      // (at the end: nothing but o outlives an attempt)
    }
    if (g == 0) {
        const size_t at = (size_t)bh * D + (PERM ? NB * nn + wave : 16 * wave + nn);
        if (out.out_bf16) static_cast<bf16_t *>(out.o)[at] = f32_to_bf16(o);
        else static_cast<float *>(out.o)[at] = o;
    }
}

// The same at d = 128, where the further block columns would be 108 of 220 tile products per wave (merge kernel 56 us instead of
// 49): one wave factorises and substitutes on the vector ALU, all waves form the output as y0 sum w v + G~^T y1, y0 = (1 - mu~ . y1) /
// omega.
template <int D, typename TI, bool PERM, class Lds>
__device__ __forceinline__ void solve_and_store_128(Lds &lds, const HeadOut &out, const QueryPart<D> &q, int bh, int wave, int lane)
{
    using S = DecShape<D>;
    constexpr int NB = S::NB;
    const int g = lane / 16, nn = lane % 16;
    float *scratch = lds.sc, *ys = scratch + 16 * SC_PITCH;
    if (wave == 0) {                                      // scalar branch: the block contains MFMAs
        const float oinv = 1.f / lds.om[0], floor = 0.5f * out.lambda;
        for (int attempt = 0; attempt < SOLVE_TRIES; ++attempt) {
            int lane_e = lane;                            // an attempt keeps nothing for the next: neither the moments nor what follows
            asm volatile("" : "+v"(lane_e) :: "memory");  // from the lane index (registers for both cost 0.5 us)
            const int g = lane_e / 16, nn = lane_e % 16;
            const float eta = noise_ridge(attempt);
            f32x4 acc[S::NSIG], rhs[NB];
            float mc[NB];
#pragma unroll
            for (int J = 0; J < NB; ++J) mc[J] = lds.mu[0][16 * J + nn];
#pragma unroll
            for (int P = 0; P < NB; ++P) {                // -(Sigma_c + ridge)
                const f32x4 mr = oinv * *reinterpret_cast<const f32x4 *>(&lds.mu[0][16 * P + 4 * g]);
#pragma unroll
                for (int J = P; J < NB; ++J) {
                    const float *tile = &lds.tiles[0][upper_tile<NB>(P, J) * 256];
                    const f32x4 st = *reinterpret_cast<const f32x4 *>(tile + lane_e * 4);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        float v = fmaf(mr[t], mc[J], -st[t]);
                        if (J == P) {                     // symmetrised, as above
                            const float other = fmaf(oinv * mc[J], lds.mu[0][16 * P + 4 * g + t], -tile[(16 * (nn >> 2) + 4 * g + t) * 4 + (nn & 3)]);
                            v = 0.5f * (v + other);
                            v -= (nn == 4 * g + t) ? fmaf(eta, st[t], out.lambda) : 0.f;
                        }
                        acc[upper_tile<NB>(P, J)][t] = v;
                    }
                }
            }
            float low = INFINITY;
            factorise_one<NB, true, false, false, true>(acc, scratch, g, nn, floor, &low);
            float tv[1][NB];                                  // -q_c, U^{-T} q_c, its negative
#pragma unroll
            for (int P = 0; P < NB; ++P) {
                tv[0][P] = fmaf(lds.mu[0][16 * P + nn], oinv, -q.v[P][0]);
            }
            substitute_forward<NB, 1>(acc, tv, scratch, g, nn);
#pragma unroll
            for (int P = 0; P < NB; ++P) tv[0][P] = -tv[0][P];
            substitute_back<NB, 1>(acc, tv, rhs, scratch, g, nn);
            float my = 0.f;
#pragma unroll
            for (int P = 0; P < NB; ++P) {
                const f32x4 m = *reinterpret_cast<const f32x4 *>(&lds.mu[0][16 * P + 4 * g]);
#pragma unroll
                for (int t = 0; t < 4; ++t) my = fmaf(m[t], rhs[P][t], my);
            }
            const float y0 = (1.f - rows_allsum(my)) * oinv;
            if (nn == 0) {
#pragma unroll
                for (int P = 0; P < NB; ++P) *reinterpret_cast<f32x4 *>(&ys[16 * P + 4 * g]) = rhs[P];
                if (g == 0) ys[D] = y0;
            }
            if (__builtin_amdgcn_ballot_w64(low < floor) == 0) break;
        }
    }
    __syncthreads();
    const float y0 = ys[D];
    for (int J = wave; J < NB; J += 4) {
        float s = 0.f;
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            const f32x4 gv = *reinterpret_cast<const f32x4 *>(&lds.tiles[0][(S::NSIG + NB * I + J) * 256 + lane * 4]);
            const f32x4 y1 = *reinterpret_cast<const f32x4 *>(&ys[16 * I + 4 * g]);
#pragma unroll
            for (int t = 0; t < 4; ++t) s = fmaf(gv[t], y1[t], s);        // G~[16I+4g+t][16J+nn] y1[16I+4g+t]
        }
        s = rows_allsum(s);
        const float o = fmaf(y0, lds.yv[0][16 * J + nn], s);
        if (g == 0) {
            const size_t at = (size_t)bh * D + (PERM ? NB * nn + J : 16 * J + nn);
            if (out.out_bf16) static_cast<bf16_t *>(out.o)[at] = f32_to_bf16(o);
            else static_cast<float *>(out.o)[at] = o;
        }
    }
}

template <int D, typename TI, bool PERM, class Lds>
__device__ __forceinline__ void solve_head(Lds &lds, const HeadOut &out, const QueryPart<D> &q, int bh, int wave, int lane)
{
    if constexpr (D == 128) solve_and_store_128<D, TI, PERM>(lds, out, q, bh, wave, lane);
    else solve_and_store<D, TI, PERM>(lds, out, q, bh, wave, lane);
}

// The four waves of a workgroup, each with moments of its own share of the keys, become one set of moments: in the workgroup's
// record R, or (FUSED: one workgroup per head) in LDS, from where the head is solved and its output written.  Summed in a fixed
// order through NBUF LDS copies of the tiles.  A record per wave instead cost four times the traffic (27 KB each at d = 64).
//   mref: the exponent the wave's moments refer to; mtrue: the largest logit of its keys (both wave-uniform, -inf without keys)
//   om: sum of the wave's weights; mu[J], yv[J]: element n of block J, in the lanes of group 0 at least
template <int D, typename TI, bool PERM, bool FUSED, int NBUF, class Lds>
__device__ __forceinline__ void finish_workgroup(Lds &lds, f32x4 (&acc)[DecShape<D>::NTILES], float (&mu)[DecShape<D>::NB],
                                                 float (&yv)[DecShape<D>::NB], float om, float mref, float mtrue, float *R,
                                                 const HeadOut &out, int bh, int wave, int lane)
{
    using S = DecShape<D>;
    constexpr int NB = S::NB, NTILES = S::NTILES;
    static_assert(NBUF == 2 || NBUF == 4, "two or four copies of the tiles");
    const int nn = lane % 16, tid = wave * 64 + lane;
    if (lane == 0) lds.mw[wave] = mtrue;
    __syncthreads();
    const float mall = fmaxf(fmaxf(lds.mw[0], lds.mw[1]), fmaxf(lds.mw[2], lds.mw[3]));
    const float f = mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - mall);
    auto put = [&](float *dst, bool add) {
#pragma unroll
        for (int t = 0; t < NTILES; ++t) {
            f32x4 *p = reinterpret_cast<f32x4 *>(dst + t * 256 + lane * 4);
            *p = add ? *p + f * acc[t] : f * acc[t];
        }
    };
    if (lane < 16) {
#pragma unroll
        for (int J = 0; J < NB; ++J) { lds.mu[wave][16 * J + nn] = f * mu[J]; lds.yv[wave][16 * J + nn] = f * yv[J]; }
    }
    if (lane == 0) lds.om[wave] = f * om;
    if (wave < NBUF) put(lds.tiles[wave & (NBUF - 1)], false);
    __syncthreads();
    if constexpr (NBUF == 2) {
        if (wave >= 2) put(lds.tiles[wave - 2], true);
        __syncthreads();
    }
    for (int i = tid; i < NTILES * 64; i += DEC_NT) {
        f32x4 v = reinterpret_cast<const f32x4 *>(lds.tiles[0])[i];
#pragma unroll
        for (int bf = 1; bf < NBUF; ++bf) v += reinterpret_cast<const f32x4 *>(lds.tiles[bf])[i];
        if constexpr (FUSED) reinterpret_cast<f32x4 *>(lds.tiles[0])[i] = v;
        else *reinterpret_cast<f32x4 *>(R + S::HDR + 4 * i) = v;
    }
    if (tid < 2 * D) {
        float *src = tid < D ? &lds.mu[0][tid] : &lds.yv[0][tid - D];
        const float v = (src[0] + src[D]) + (src[2 * D] + src[3 * D]);
        if constexpr (FUSED) src[0] = v;
        else R[64 + tid] = v;
    }
    QueryPart<D> q;
    if constexpr (FUSED) q = load_query<D, TI, PERM>(out, bh, lane);
    const float oall = (lds.om[0] + lds.om[1]) + (lds.om[2] + lds.om[3]);
    if constexpr (FUSED) {
        __syncthreads();
        if (tid == 0) lds.om[0] = oall;
        __syncthreads();
        solve_head<D, TI, PERM>(lds, out, q, bh, wave, lane);
    } else if (tid == 0) {
        R[0] = mall;
        R[1] = oall;
    }
}

// Merge of a head's records (max-rescaled sum), solve, output: one head per workgroup.  Every thread owns the same 16 bytes of each tile
// of every record.  What bounds it is the number of round trips to memory in front of the solve: lane l fetches maximum and weight sum of
// record l, one trip for all of them; header vectors and tiles come in groups of records, unconditionally and all in flight together
// (a load under a condition, or behind the scalar load of its record's maximum, was waited for by itself: 16 trips per eight records),
// and only records that there are (three of 100 KB cost eight).  Four records at a time; one at d = 128, where it is 25 loads per
// thread and a compute unit takes 1 us for it however many are requested together.  Eight (at d = 64) take more registers than two workgroups on
// a compute unit have: 512 heads x 8192 170 instead of 164 us.  us of a call, eight at a time and so: d = 128, 8 heads x 1000 keys 48.7 / 44.1,
// 16 x 4096 69.5 / 63.9; d = 64, 16 x 4096 28.4 / 26.1; fp32, 16 x 4096 40.0 / 35.6; d = 16, fp32, 64 heads of 512 .. 4096 24.9 / 20.5.
// DUAL: a call whose sequences of at most 64 keys are served in key space has one more workgroup per head for that, in the same
// launch; which of the two writes the head follows from its length.
template <int D, typename TI, bool PERM, bool DUAL = false>
__global__ __launch_bounds__(DEC_NT, D == 128 ? 1 : 2) void decode_merge_kernel(DecSplit split, HeadOut out, const float *__restrict__ parts,
                                                                 dual::DualArgs da = {}, int heads = 0)
{
    using S = DecShape<D>;
    using Dual = dual::DualShared<D, DUAL_MAX_KEYS>;
    constexpr size_t LDS_B = sizeof(HeadLds<D, 1, 1>) > sizeof(Dual) || !DUAL ? sizeof(HeadLds<D, 1, 1>) : sizeof(Dual);
    __shared__ __align__(16) unsigned char raw[LDS_B];
    if constexpr (DUAL) {
        if ((int)blockIdx.x >= heads) {
            if (out.out_bf16) dual::dual_decode_head<D, TI, bf16_t>(*reinterpret_cast<Dual *>(raw), da, split.seqlens, blockIdx.x - heads);
            else dual::dual_decode_head<D, TI, float>(*reinterpret_cast<Dual *>(raw), da, split.seqlens, blockIdx.x - heads);
            return;
        }
        if (seq_len(split, blockIdx.x / split.H) <= DUAL_MAX_KEYS) return;
    }
    HeadLds<D, 1, 1> &lds = *reinterpret_cast<HeadLds<D, 1, 1> *>(raw);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, bh = blockIdx.x;
    const QueryPart<D> q = load_query<D, TI, PERM>(out, bh, lane);
    const DecRecords rec = dec_records(split, bh);
    const int np = rec.count;
    const float *P0 = parts + (size_t)rec.first * S::REC_F;
    float f, om;                                          // factor and weights of record `lane`
    {
        const float *P = P0 + (size_t)min(lane, np - 1) * S::REC_F;
        const float mp = P[0], o = P[1], m = lane < np ? mp : -INFINITY;
        const float top = wave_max_dpp(m);                // (all lanes take part)
        f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - top);
        om = rows_allsum(row_allsum(f * o));
    }
    constexpr int N4 = (S::NTILES * 64 + DEC_NT - 1) / DEC_NT;
    f32x4 acc[N4];
#pragma unroll
    for (int i = 0; i < N4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float hv = 0.f;
    struct Part { float h; f32x4 v[N4]; };                // what a thread owns of a record
    constexpr int LAST = S::NTILES * 64 - DEC_NT * (N4 - 1);          // threads that own a piece of the last round
    // (scalar base and unsigned byte offset per lane: one address register for all loads)
    const unsigned hoff = 4u * (unsigned)min(tid, 2 * D - 1), toff = 16u * (unsigned)tid, tlast = 16u * (unsigned)min(tid, LAST - 1);
    auto fetch = [&](Part &r, int p) {
        const char *P = reinterpret_cast<const char *>(P0 + (size_t)min(p, np - 1) * S::REC_F);
        r.h = *reinterpret_cast<const float *>(P + 256 + hoff);
#pragma unroll
        for (int i = 0; i < N4; ++i) r.v[i] = *reinterpret_cast<const f32x4 *>(P + 4 * S::HDR + 16 * DEC_NT * i + (i + 1 < N4 ? toff : tlast));
    };
    auto add = [&](const Part &r, int p) {
        const float fp = p < np ? __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f), p)) : 0.f;
        hv = fmaf(fp, r.h, hv);
#pragma unroll
        for (int i = 0; i < N4; ++i) acc[i] += fp * r.v[i];
    };
    auto group = [&](int pb, auto size) {                 // records pb .. pb + N - 1, those there are
        constexpr int N = decltype(size)::value;
        Part r[N];
#pragma unroll
        for (int k = 0; k < N; ++k) fetch(r[k], pb + k);
        __builtin_amdgcn_sched_barrier(0);                // all loads first: the scheduler put the first sum, and its wait, between them
#pragma unroll
        for (int k = 0; k < N; ++k) add(r[k], pb + k);
    };
    // (all branches on np are scalar)
    if constexpr (D == 128) {
#pragma unroll 1
        for (int p = 0; p < np; ++p) group(p, std::integral_constant<int, 1>{});
    } else {
        for (int pb = 0; pb < np; pb += 4) {
            if (np - pb > 2) group(pb, std::integral_constant<int, 4>{});
            else if (np - pb > 1) group(pb, std::integral_constant<int, 2>{});
            else group(pb, std::integral_constant<int, 1>{});
        }
    }
#pragma unroll
    for (int i = 0; i < N4; ++i)
        if (tid + DEC_NT * i < S::NTILES * 64) reinterpret_cast<f32x4 *>(lds.tiles[0])[tid + DEC_NT * i] = acc[i];
    if (tid < 2 * D) (tid < D ? lds.mu[0] : lds.yv[0])[tid & (D - 1)] = hv;
    if (tid == 0) lds.om[0] = om;
    __syncthreads();
    solve_head<D, TI, PERM>(lds, out, q, bh, wave, lane);
}

}  // namespace mfma
}  // namespace llla
