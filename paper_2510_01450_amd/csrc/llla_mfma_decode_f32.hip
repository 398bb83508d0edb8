// fp32 matrix-core decode for gfx950: fp32 caches at every d, bf16 caches at d = 16 / 32 and at any d below the capacity from
// which the 16-bit kernels serve.  The precision of fp32 (bf16 is widened exactly), as in the vector kernels: on v_mfma_f32_16x16x4_f32, or, fp32
// caches at d = 64 and bf16 ones at d = 16 / 32, on 16-bit matrix instructions with operands in three bf16 (below).  One pass over the cache, the method of llla_mfma_decode.hip: each wave accumulates, relative to a
// running reference exponent, omega, mu~, Sigma~ and the value moments sum w v and G~ = sum w k v^T, and the solved system gives
// o = y0 * sum w v + G~^T y1.
//
// No LDS and no data movement in the loop, but for fp32 rows at d = 64.  An MFMA with the key as contraction index wants lane (g, n) to hold element n of
// key g; the features may be numbered in any order, so lane (g, n) owns features NB n .. NB n + NB - 1 (NB = d / 16) of key g: one
// vector load per lane and four keys, fully coalesced (the wave reads four whole rows), and register I is directly the A operand
// (times w) of row block I and the B operand of column block I of every tile product.  Feature NB n + I is element n of block I in
// all tiles and vectors below; only the query at the solve and the output at the end translate.
// The logits of 4 keys x 4 chunks are reduced over the 16 lanes of a row by two exchange stages that leave chunk (n & 3) in
// lane n, so a lane forms ONE exponential per 16 keys; the weights go back to the row as DPP broadcasts.
//
// bf16 caches at d = 16 / 32 leave the fp32 MFMA rate behind: slot (g, t) of a 16x16x32 MFMA stands for key 4 t + g, so the registers
// of eight chunks are its operands as they are; k and v are bf16 already, and w k is split into three (24 significant bits), three
// products instead of eight fp32 ones of twice the cycles.
//
// fp32 caches at d = 64 do likewise (compute_roots): 26 tiles of 16x16x4 per four keys were 832 matrix-core cycles for 2 KB of cache, 6 TB/s
// at 2.4 GHz and 2.7 reached; both operands in three bf16, as sqrt(w) k and sqrt(w) v, take 296.  Their rows pass through LDS stages of the wave's own.
//
// What bounds it: HBM at d = 16 / 32; at d = 64 in fp32 nearly HBM (194 us = 5.5 TB/s of 6.6 at 256 heads x 8192) and nearly the two waves of a SIMD, matrix cores 36 % and
// vector port 45 % busy, and in short calls latency (64 heads of 1024 to 8192 keys, six steps a wave: 3.6 TB/s, 19 and 28 %); at d = 128
// 100 tiles of 16x16x4 per four keys, 3 TB/s: the matrix cores.  There the accumulators of a stream (400 registers) are dealt over the four waves of a workgroup:
// wave W owns row blocks W and 7 - W, 25 tiles whatever W; every wave loads the whole rows (the first-level cache serves three
// of the four) and forms the weights for itself, so there is no exchange at all.
#include "llla_decode_tail.hpp"

namespace llla {
namespace {

using namespace mfma;

constexpr int NT = DEC_NT;
constexpr int ROOT_STAGE_B = 16384;     // by roots: a wave's LDS stage, 32 keys and 32 values of 64 floats
constexpr float VALUE_SCALE = 0x1p64f, VALUE_SMALL = 0x1p-16f;      // see compute_roots
constexpr float REF_SLACK = 8.f;        // the reference exponent moves when a logit exceeds it by more than 2^8 (weights stay <= 256)

template <int D>
struct F32Shape : DecShape<D> {
    static constexpr bool TEAM = D == 128;                // four waves share one key stream
    static constexpr int NC = TEAM ? 2 : 4;               // chunks of four keys whose logits are reduced together
    static constexpr int NG = D == 16 ? 2 : 1;            // such groups per step
    static constexpr int STEP = 4 * NC * NG;              // keys per step
    static constexpr int NR = TEAM ? 2 : D / 16;          // row blocks of a wave
    static constexpr int NBUF = D <= 32 ? 4 : TEAM ? 1 : 2;   // LDS copies of the tiles in the merge of a workgroup's waves
    static constexpr int KEYS_MIN = TEAM ? 128 : 256;     // fewest keys worth a workgroup (its record is read back by the merge)
    static constexpr int SLOTS = D <= 16 ? 1024 : 512;    // workgroups worth having at once
    static constexpr int MAX_SPLIT = 32;
    static_assert(MAX_SPLIT < MAX_RECORDS, "the flat cut can leave one piece more");
};

template <typename TI, int NB>
struct RowFrag {                                          // the NB features of one key that a lane owns, as loaded
    static constexpr int BYTES = NB * (int)sizeof(TI);
    static constexpr int WORDS = BYTES < 4 ? 1 : BYTES / 4;
    unsigned u[WORDS];
};

typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

template <typename TI, int NB, bool NT_HINT>
__device__ __forceinline__ RowFrag<TI, NB> load_frag(const char *p)
{
    RowFrag<TI, NB> f;
    constexpr int BYTES = RowFrag<TI, NB>::BYTES;
    if constexpr (BYTES == 2) {
        f.u[0] = *reinterpret_cast<const uint16_t *>(p);
    } else if constexpr (BYTES == 4) {
        f.u[0] = NT_HINT ? __builtin_nontemporal_load(reinterpret_cast<const unsigned *>(p)) : *reinterpret_cast<const unsigned *>(p);
    } else if constexpr (BYTES == 8) {
        const uint2v v = NT_HINT ? __builtin_nontemporal_load(reinterpret_cast<const uint2v *>(p)) : *reinterpret_cast<const uint2v *>(p);
        f.u[0] = v[0]; f.u[1] = v[1];
    } else {
#pragma unroll
        for (int i = 0; i < BYTES / 16; ++i) {
            const uint4v v = NT_HINT ? __builtin_nontemporal_load(reinterpret_cast<const uint4v *>(p) + i)
                                     : reinterpret_cast<const uint4v *>(p)[i];
#pragma unroll
            for (int t = 0; t < 4; ++t) f.u[4 * i + t] = v[t];
        }
    }
    return f;
}

template <typename TI, int NB>
__device__ __forceinline__ float frag_f32(const RowFrag<TI, NB> &f, int i)
{
    if constexpr (sizeof(TI) == 4) return __uint_as_float(f.u[i]);
    else return __uint_as_float((i & 1) ? f.u[i >> 1] & 0xffff0000u : f.u[i >> 1] << 16);
}

// sums of p[0..NC-1] over the 16 lanes of a row; lane n receives the sum of p[n & (NC - 1)]
template <int NC>
__device__ __forceinline__ float reduce_chunks(const float (&p)[NC], int nn)
{
    const bool b0 = (nn & 1) != 0, b1 = (nn & 2) != 0;
    float s;
    if constexpr (NC == 4) {
        const float s0 = (b0 ? p[1] : p[0]) + dpp_f<0xB1>(b0 ? p[0] : p[1]);
        const float s1 = (b0 ? p[3] : p[2]) + dpp_f<0xB1>(b0 ? p[2] : p[3]);
        s = (b1 ? s1 : s0) + dpp_f<0x4E>(b1 ? s0 : s1);
    } else {
        s = (b0 ? p[1] : p[0]) + dpp_f<0xB1>(b0 ? p[0] : p[1]);
        s += dpp_f<0x4E>(s);
    }
    s += dpp_f<0x124>(s);                                 // row_ror:4
    s += dpp_f<0x128>(s);                                 // row_ror:8
    return s;
}

struct F32Args {
    const void *K, *V;
    llla_strides sk, sv;
    DecSplit split;
    HeadOut out;
    float cscale;
    float *parts;
    int heads_first;       // flat cut by roots: grid (H, slots)
};

// The stream of one wave and what becomes of its moments.  W: the wave's share of the tiles (TEAM), else 0.
// FUSED: one workgroup per head; it solves and writes the output itself.
// stages (ROOTS): the LDS stages of the four waves and, behind them, a kilobyte per wave for the query; the merge reuses them.
template <int D, typename TI, bool FUSED, bool ROOTS, int W, class Lds>
__device__ __forceinline__ void decode_f32_body(const F32Args &a, const DecPiece &pc, Lds &lds, unsigned char *stages, int wave, int lane)
{
    using S = F32Shape<D>;
    constexpr bool SPLIT = sizeof(TI) == 2 && D <= 32;    // w k in three bf16 on 16-bit MFMA, eight chunks at a time
    constexpr int NB = S::NB, NC = S::NC, NG = SPLIT || ROOTS ? 2 : S::NG, NR = S::NR, CH = NC * NG, STEP = 4 * CH;
    constexpr int row[4] = {S::TEAM ? W : 0, S::TEAM ? 7 - W : 1, 2, 3};      // row blocks of this wave: row[0..NR-1]
    const int g = lane / 16, nn = lane % 16;
    // the piece is divided over the four waves (TEAM: walked by all four together); rows at and beyond L are never read
    const int L = pc.L, b = pc.b, h = pc.h, bh = pc.bh;
    const int share = S::TEAM ? pc.k1 - pc.k0 : ((pc.k1 - pc.k0 + 3) / 4 + STEP - 1) / STEP * STEP;
    const int r0 = __builtin_amdgcn_readfirstlane(min(pc.k0 + (S::TEAM ? 0 : wave * share), pc.k1));
    const int r1 = __builtin_amdgcn_readfirstlane(min(r0 + share, pc.k1));
    const int nsteps = (r1 - r0 + STEP - 1) / STEP;
    const char *Kh = reinterpret_cast<const char *>(static_cast<const TI *>(a.K) + b * a.sk.batch + h * a.sk.head);
    const char *Vh = reinterpret_cast<const char *>(static_cast<const TI *>(a.V) + b * a.sv.batch + h * a.sv.head);
    const int64_t krow = a.sk.seq * (int64_t)sizeof(TI), vrow = a.sv.seq * (int64_t)sizeof(TI);
    const unsigned koff = (unsigned)(g * (int)krow + NB * nn * (int)sizeof(TI)), voff = (unsigned)(g * (int)vrow + NB * nn * (int)sizeof(TI));

    float q[NB];
    if constexpr (!ROOTS) {
        const TI *qp = static_cast<const TI *>(a.out.q) + (size_t)bh * D + NB * nn;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            if constexpr (sizeof(TI) == 2) q[i] = bf16_to_f32(qp[i]) * a.cscale;
            else q[i] = qp[i] * a.cscale;
        }
    }

    f32x4 acc[S::NTILES];                                 // (TEAM: the tiles of row blocks row[0] and row[1] only)
    float mu[NR], yv[NR];
#pragma unroll
    for (int t = 0; t < S::NTILES; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NR; ++i) { mu[i] = 0.f; yv[i] = 0.f; }
    auto for_tiles = [&](auto fn) {                       // the tiles of this wave
#pragma unroll
        for (int i = 0; i < NR; ++i) {
#pragma unroll
            for (int J = row[i]; J < NB; ++J) fn(upper_tile<NB>(row[i], J));
#pragma unroll
            for (int J = 0; J < NB; ++J) fn(S::NSIG + NB * row[i] + J);
        }
    };
    float om = 0.f, mref = -INFINITY, mtrue = -INFINITY;

    // by roots, value features taken VALUE_SCALE times (all to begin with): bit 16 i + n is feature NB n + i
    unsigned long long small = ~0ull;
    auto value_scale = [&](unsigned long long which, int i, float s) {       // s for the lane's feature i if it is among them, else 1
        return ((unsigned)(which >> (i & 2) * 16) >> (16 * (i & 1) + nn)) & 1 ? s : 1.f;
    };
    auto unscale_values = [&](unsigned long long which) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const float f = value_scale(which, i, 1.f / VALUE_SCALE);
            yv[i] *= f;
#pragma unroll
            for (int I = 0; I < NB; ++I) acc[S::NSIG + NB * I + i] *= f;
        }
    };
    typedef RowFrag<TI, NB> Frag;
    struct Step { Frag k[CH], v[CH]; };
    auto load_rows = [&](Frag (&f)[CH], const char *base, int64_t pitch, unsigned off, int s) {
        const int j0 = r0 + (s < nsteps ? s : 0) * STEP;              // past the end: the first step again, never used
        if (j0 + STEP <= L) {
            const char *p = base + j0 * pitch;
#pragma unroll
            for (int c = 0; c < CH; ++c) f[c] = load_frag<TI, NB, !S::TEAM>(p + 4 * c * pitch + off);
        } else {                                          // rows beyond the sequence: its last row (their weights are 0)
#pragma unroll
            for (int c = 0; c < CH; ++c) f[c] = load_frag<TI, NB, !S::TEAM>(base + min(j0 + 4 * c + g, L - 1) * pitch + NB * nn * (int)sizeof(TI));
        }
    };
    // fp32 at d = 32: keys and values alternate, and the last rows are a choice of addresses instead of a branch (us, as the others / this: 256 heads
    // x 4096 66.8 / 58.0, 16 x 8192 21.2 / 18.6; bf16 at d = 32, 256 x 4096, 32.7 / 35.3).
    auto load = [&](Step &st, int s) {
        if constexpr (D != 32 || sizeof(TI) == 2) {
            load_rows(st.k, Kh, krow, koff, s);
            load_rows(st.v, Vh, vrow, voff, s);
        } else {
            const int j0 = r0 + (s < nsteps ? s : 0) * STEP;
            const bool whole = j0 + STEP <= L;
            const char *kb = Kh + j0 * krow + koff, *vb = Vh + j0 * vrow + voff;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int j = min(j0 + 4 * c + g, L - 1), lane_off = NB * nn * (int)sizeof(TI);
                st.k[c] = load_frag<TI, NB, true>(whole ? kb + 4 * c * krow : Kh + j * krow + lane_off);
                st.v[c] = load_frag<TI, NB, true>(whole ? vb + 4 * c * vrow : Vh + j * vrow + lane_off);
            }
        }
    };
    // logits of a step's 32 keys, the reference exponent, and the exponents of the weights (log2, ROOTS too, which halves them itself): e[grp]
    // belongs to key 4 (n % 4) + g of group grp
    auto step_exponents = [&](const auto &k, int s, float (&e)[2]) {
        const int j0 = r0 + s * STEP;
        float t[2];
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
            float p[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                p[c] = 0.f;
#pragma unroll
                for (int i = 0; i < NB; ++i) p[c] = fmaf(q[i], frag_f32<TI, NB>(k[grp * NC + c], i), p[c]);
            }
            t[grp] = reduce_chunks<NC>(p, nn);                        // logit (log2 units) of key 4 (n % NC) + g of the group
            t[grp] = j0 + grp * 4 * NC + 4 * (nn & (NC - 1)) + g < r1 ? t[grp] : -INFINITY;
        }
        const float top = fmaxf(t[0], t[1]);
        if (__builtin_amdgcn_ballot_w64(top > mref + REF_SLACK) != 0) {
            const float mnew = wave_max_dpp(top);
            const float alpha = mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - mnew);
            mref = mnew;
            om *= alpha;
#pragma unroll
            for (int i = 0; i < NR; ++i) { mu[i] *= alpha; yv[i] *= alpha; }
            for_tiles([&](int t) { acc[t] *= alpha; });
        }
        mtrue = fmaxf(mtrue, top);
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) e[grp] = t[grp] - mref;
    };
    auto compute_split = [&](const auto &st, int s) {
        float e[2], w[2];
        step_exponents(st.k, s, e);
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
            w[grp] = __builtin_amdgcn_exp2f(e[grp]);                  // exp2(-inf) = 0 masks the tail
            om += w[grp];
        }
        const float wc[8] = {row_bcast<0>(w[0]), row_bcast<1>(w[0]), row_bcast<2>(w[0]), row_bcast<3>(w[0]),
                             row_bcast<0>(w[1]), row_bcast<1>(w[1]), row_bcast<2>(w[1]), row_bcast<3>(w[1])};
        // element I of eight chunks as an MFMA operand: bf16 bits as loaded
        auto operand = [](const auto &f, int I) {
            uint4v u;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const unsigned a = f[2 * c].u[I >> 1], b = f[2 * c + 1].u[I >> 1];
                u[c] = (I & 1) ? __builtin_amdgcn_perm(b, a, 0x07060302u) : __builtin_amdgcn_perm(b, a, 0x05040100u);
            }
            return __builtin_bit_cast(bf16x8, u);
        };
        bf16x8 kb[NB], vb[NB];
#pragma unroll
        for (int J = 0; J < NB; ++J) { kb[J] = operand(st.k, J); vb[J] = operand(st.v, J); }
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            float x[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                x[c] = wc[c] * frag_f32<TI, NB>(st.k[c], I);
                mu[I] += x[c];
                yv[I] = fmaf(wc[c], frag_f32<TI, NB>(st.v[c], I), yv[I]);
            }
            bf16x8 h, m, l;
            split3_bf16(x, h, m, l);
            auto product = [&](f32x4 &t, bf16x8 b) { t = mfma_bf16(h, b, mfma_bf16(m, b, mfma_bf16(l, b, t))); };
#pragma unroll
            for (int J = I; J < NB; ++J) product(acc[upper_tile<NB>(I, J)], kb[J]);
#pragma unroll
            for (int J = 0; J < NB; ++J) product(acc[S::NSIG + NB * I + J], vb[J]);
        }
    };
    // sqrt(w) k and sqrt(w) v split into three bf16 each, six products per tile of the nine (the rest is below 2^-24), as in the moments
    // kernel of the forward: 96 matrix-core cycles per tile and 32 keys instead of 256 (64 in a diagonal tile).  The products of a step
    // start from zero and are then added to the tile: one rounding of the sum per step, 0.29 ulp rms, instead of six times the 0.58 of an
    // MFMA.  (Chained onto the sum, errors against fp64 grew with the keys per wave: 32 heads x 32768 unit keys 8.0e-7, 3.5e-7
    // now, 4.9e-7 on fp32 MFMA; 32 x 8192 3.5e-7, 2.7e-7, 3.2e-7.  64 heads x 1024 to 8192 61.3 -> 61.8 us a call, 256 x 8192 220 -> 241.)
    // Two waves per SIMD.  The rows come by DMA into LDS, and a conversion reads the two feature blocks it needs; kept in registers, with sums put off
    // by the compiler until after the next branch (their terms kept until then), a wave took 430 registers, was alone on its SIMD and
    // waited for its values.  246 to 249 now; the conversion of the next block is pinned to alternate with the products of this one.  us, one wave with
    // rows in registers / one with two LDS stages / two waves: 256 heads x 8192 234 / 215 / 212, 512 x 1000 79 / 74 / 66, 1024 x 2000 260 / 243 / 220.  On fp32 MFMA, also two waves: 512 x 100 25.7 (22.1 here), 512 x 512
    // 51.4 (42.3), 384 x 300 38.0 (30.9), 320 x 777 74.0 (60.0), 1024 x 800 137 (108).
    // The third term of a value below 2^-110 would be subnormal, which matrix cores read as zero.  So a stream starts with its values taken
    // VALUE_SCALE times and goes over to the values as they are, feature by feature, at the first one above VALUE_SMALL, ordinarily in its first
    // step (64 heads x 1024 to 8192 62.6 -> 63.3 us, 16 x 32768 77.9 -> 79.0; values of size 2^-110 3e-7, 2^-124 1.4e-3 off without it, rounding
    // with it).  A feature that stays below, of zeros for instance, costs its stream the choice in every step: 256 heads x 8192 with a quarter of the
    // features zero 208 -> 214 us, as long as with none (213).
    // Rows of a step by DMA, a wave's own stages: lane l's 16 bytes of a chunk land at 16 l of its kilobyte, which is where the lane reads
    // them, so there is no swizzle and no barrier, and the 16-byte reads have no bank conflicts; those of a half, 8 bytes at a distance of 16, have
    // (43 % of LDS cycles, which are 18 % of all).  tile: 0 keys, 1 values.
    unsigned char *const mine = stages + wave * ROOT_STAGE_B;
    auto fetch_rows = [&](int tile, int s) {
        const char *base = tile ? Vh : Kh;
        const int64_t pitch = tile ? vrow : krow;
        const unsigned dst = lds_offset(mine) + (unsigned)(tile * (ROOT_STAGE_B / 2));
        const int j0 = r0 + s * STEP;
        if (j0 + STEP <= L) {
            const char *p = base + j0 * pitch;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                dma16_base_nt_off(p, tile ? voff : koff, dst + 1024u * c);
                p += 4 * pitch;
                asm volatile("" : "+s"(p));               // (kept as sixteen hoisted bases: 44 spilled scalar registers)
            }
        } else {                                          // rows beyond the sequence: its last row (their weights are 0)
#pragma unroll
            for (int c = 0; c < CH; ++c) dma16_nt_off(base + min(j0 + 4 * c + g, L - 1) * pitch + 16 * nn, dst + 1024u * c);
        }
    };
    // features 2 half and 2 half + 1 of the lane's rows
    auto read_half = [&](float (&f)[2][CH], int tile, int half) {
        const float2v *p = reinterpret_cast<const float2v *>(mine + tile * (ROOT_STAGE_B / 2)) + 2 * lane + half;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const float2v v = p[128 * c];
            f[0][c] = v[0];
            f[1][c] = v[1];
        }
    };
    auto compute_roots = [&](auto s) {               // (generic: instantiated only where it is called)
        const bool more = s + 1 < nsteps;
        dma_wait_but<CH>();                               // all but the values of this step
        float e[2], rt[2];
        {
            Frag k[CH];
            const uint4v *p = reinterpret_cast<const uint4v *>(mine) + lane;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const uint4v v = p[64 * c];
#pragma unroll
                for (int t = 0; t < 4; ++t) k[c].u[t] = v[t];
            }
            step_exponents(k, s, e);
        }
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
            rt[grp] = __builtin_amdgcn_exp2f(0.5f * e[grp]);          // exp2(-inf) = 0 masks the tail
            om = fmaf(rt[grp], rt[grp], om);
        }
        asm volatile("" : "+v"(om), "+v"(mtrue));
        const float rc[8] = {row_bcast<0>(rt[0]), row_bcast<1>(rt[0]), row_bcast<2>(rt[0]), row_bcast<3>(rt[0]),
                             row_bcast<0>(rt[1]), row_bcast<1>(rt[1]), row_bcast<2>(rt[1]), row_bcast<3>(rt[1])};
        struct Split3 { bf16x8 h, m, l; };
        auto scaled = [&](const float (&f)[CH], float &sum) {
            float x[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                x[c] = rc[c] * f[c];
                sum = fmaf(rc[c], x[c], sum);
            }
            asm volatile("" : "+v"(sum));                 // (summed here: not put off, with the terms kept in registers)
            Split3 r;
            split3_bf16(x, r.h, r.m, r.l);
            return r;
        };
        // a vector instruction of the next conversion behind every product
        auto alternate = [](auto n, auto each) {
#pragma unroll
            for (int i = 0; i < decltype(n)::value; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, decltype(each)::value, 0);
            }
        };
        // tiles z[0..N-1] x b from zero, added to the sums; the chains of the tiles alternate
        auto products = [&](auto n, auto keys, auto jtag, const Split3 (&z)[NB], const Split3 &b) {
            constexpr int N = decltype(n)::value, J = decltype(jtag)::value;
            f32x4 t[N > 0 ? N : 1];
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = mfma_bf16(z[I].l, b.h, t[I]);
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = mfma_bf16(z[I].h, b.l, t[I]);
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = mfma_bf16(z[I].m, b.m, t[I]);
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = mfma_bf16(z[I].m, b.h, t[I]);
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = mfma_bf16(z[I].h, b.m, t[I]);
#pragma unroll
            for (int I = 0; I < N; ++I) t[I] = mfma_bf16(z[I].h, b.h, t[I]);
#pragma unroll
            for (int I = 0; I < N; ++I) acc[decltype(keys)::value ? upper_tile<NB>(I, J) : S::NSIG + NB * I + J] += t[I];
#pragma unroll
            for (int I = 0; I < N; ++I) asm volatile("" : "+v"(acc[decltype(keys)::value ? upper_tile<NB>(I, J) : S::NSIG + NB * I + J]));
        };
        asm volatile("" ::: "memory");                    // the rows are read again, not kept
        Split3 z[NB], v;
        float raw[2][CH];
        read_half(raw, 0, 0);
        z[0] = scaled(raw[0], mu[0]);
        auto key_block = [&](auto jtag) {
            constexpr int J = decltype(jtag)::value;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (J + 1 < NB) z[J + 1] = scaled(raw[(J + 1) & 1], mu[J + 1]);
            else v = scaled(raw[0], yv[0]);
            products(jtag, std::true_type{}, jtag, z, z[J]);
            // diagonal: h^T m and m^T h are each other's transposes, and the solve takes (T + T^T) / 2
            const bf16x8 h2 = twice_bf16(z[J].h);
            f32x4 t = {0.f, 0.f, 0.f, 0.f};
            t = mfma_bf16(h2, z[J].l, t);
            t = mfma_bf16(z[J].m, z[J].m, t);
            t = mfma_bf16(h2, z[J].m, t);
            t = mfma_bf16(z[J].h, z[J].h, t);
            acc[upper_tile<NB>(J, J)] += t;
            asm volatile("" : "+v"(acc[upper_tile<NB>(J, J)]));
            alternate(std::integral_constant<int, 6 * J + 4>{}, std::integral_constant<int, J == 0 ? 8 : J == 1 ? 6 : J == 2 ? 5 : 4>{});
            __builtin_amdgcn_sched_barrier(0);
        };
        key_block(std::integral_constant<int, 0>{});
        read_half(raw, 0, 1);
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");        // read before the transfer that overwrites them is requested
            fetch_rows(0, s + 1);
        }
        key_block(std::integral_constant<int, 1>{});
        key_block(std::integral_constant<int, 2>{});
        if (more) dma_wait_but<CH>();                     // all but the next step's keys
        else dma_wait_but<0>();
        auto read_values = [&](int half) {
            read_half(raw, 1, half);
            if (half && more) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                fetch_rows(1, s + 1);
            }
            if (small != 0) {                             // (a scalar branch)
                unsigned long long large = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float top = 0.f;
#pragma unroll
                    for (int c = 0; c < CH; ++c) top = fmaxf(top, fabsf(raw[i][c]));
                    unsigned long long m = __builtin_amdgcn_ballot_w64(top > VALUE_SMALL);
                    m |= m >> 32;
                    m |= m >> 16;
                    large |= (m & 0xffff) << (32 * half + 16 * i);
                }
                if ((large & small) != 0) {
                    unscale_values(large & small);
                    small &= ~large;
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const float f = value_scale(small, 2 * half + i, VALUE_SCALE);
#pragma unroll
                    for (int c = 0; c < CH; ++c) raw[i][c] *= f;
                }
            }
        };
        asm volatile("" ::: "memory");
        read_values(0);
        key_block(std::integral_constant<int, 3>{});
        auto value_block = [&](auto jtag) {
            constexpr int J = decltype(jtag)::value;
            __builtin_amdgcn_sched_barrier(0);
            Split3 next = v;
            if constexpr (J + 1 < NB) next = scaled(raw[(J + 1) & 1], yv[J + 1]);
            products(std::integral_constant<int, NB>{}, std::false_type{}, jtag, z, v);
            v = next;
            alternate(std::integral_constant<int, 6 * NB>{}, std::integral_constant<int, 4>{});
            __builtin_amdgcn_sched_barrier(0);
        };
        value_block(std::integral_constant<int, 0>{});
        read_values(1);
        value_block(std::integral_constant<int, 1>{});
        value_block(std::integral_constant<int, 2>{});
        value_block(std::integral_constant<int, 3>{});
    };
    auto compute_f32 = [&](const Step &st, int s) {
        const int j0 = r0 + s * STEP;
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            float p[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                p[c] = 0.f;
#pragma unroll
                for (int i = 0; i < NB; ++i) p[c] = fmaf(q[i], frag_f32<TI, NB>(st.k[grp * NC + c], i), p[c]);
            }
            float t = reduce_chunks<NC>(p, nn);                       // logit (log2 units) of key 4 (n % NC) + g of the group
            const int key = j0 + grp * 4 * NC + 4 * (nn & (NC - 1)) + g;
            t = key < r1 ? t : -INFINITY;
            if (__builtin_amdgcn_ballot_w64(t > mref + REF_SLACK) != 0) {
                const float mnew = wave_max_dpp(t);
                const float alpha = mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - mnew);
                mref = mnew;
                om *= alpha;
#pragma unroll
                for (int i = 0; i < NR; ++i) { mu[i] *= alpha; yv[i] *= alpha; }
                for_tiles([&](int t) { acc[t] *= alpha; });
            }
            mtrue = fmaxf(mtrue, t);
            const float w = __builtin_amdgcn_exp2f(t - mref);         // exp2(-inf) = 0 masks the tail
            om += w;
            auto chunk = [&](auto ctag) {
                constexpr int c = decltype(ctag)::value;
                const Frag &kf = st.k[grp * NC + c], &vf = st.v[grp * NC + c];
                const float wc = row_bcast<c>(w);
                float kx[NB], vx[NB];
#pragma unroll
                for (int J = 0; J < NB; ++J) { kx[J] = frag_f32<TI, NB>(kf, J); vx[J] = frag_f32<TI, NB>(vf, J); }
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    const float wk = wc * kx[row[i]];
                    mu[i] += wk;
                    yv[i] = fmaf(wc, vx[row[i]], yv[i]);
#pragma unroll
                    for (int J = row[i]; J < NB; ++J) {
                        f32x4 &t = acc[upper_tile<NB>(row[i], J)];
                        t = __builtin_amdgcn_mfma_f32_16x16x4f32(wk, kx[J], t, 0, 0, 0);
                    }
#pragma unroll
                    for (int J = 0; J < NB; ++J) {
                        f32x4 &t = acc[S::NSIG + NB * row[i] + J];
                        t = __builtin_amdgcn_mfma_f32_16x16x4f32(wk, vx[J], t, 0, 0, 0);
                    }
                }
            };
            chunk(std::integral_constant<int, 0>{});
            chunk(std::integral_constant<int, 1>{});
            if constexpr (NC == 4) {
                chunk(std::integral_constant<int, 2>{});
                chunk(std::integral_constant<int, 3>{});
            }
        }
    };
    auto compute = [&](const Step &st, int s) {
        if constexpr (SPLIT) compute_split(st, s);
        else compute_f32(st, s);
    };
    if constexpr (ROOTS) {
        static_assert(CH * 1024 == ROOT_STAGE_B / 2, "a transfer of one kilobyte per chunk");
        // the query comes the same way, in front of the rows: a load of its own would be waited for with all transfers behind it
        unsigned char *const qs = stages + 4 * ROOT_STAGE_B + 1024 * wave;
        if (nsteps > 0) {
            dma16(static_cast<const char *>(a.out.q) + ((size_t)bh * D + NB * nn) * sizeof(TI), qs);
            fetch_rows(0, 0);
            fetch_rows(1, 0);
            dma_wait_but<2 * CH>();
            const f32x4 v = reinterpret_cast<const f32x4 *>(qs)[lane];
#pragma unroll
            for (int i = 0; i < NB; ++i) q[i] = v[i] * a.cscale;
        }
#pragma unroll 1
        for (int s = 0; s < nsteps; ++s) compute_roots(s);
        if (small != 0) unscale_values(small);            // (nothing, where there was no step)
        __syncthreads();                                  // the stages of all waves are dead
    } else if (nsteps > 0) {
        Step sa, sb;
        load(sa, 0);
        for (int s = 0; s < nsteps; s += 2) {
            load(sb, s + 1);
            compute(sa, s);
            load(sa, s + 2);
            if (s + 1 < nsteps) compute(sb, s + 1);
        }
    }

    mtrue = wave_max_dpp(mtrue);
    om += dpp_f<0xB1>(om);
    if constexpr (NC == 4) om += dpp_f<0x4E>(om);
    om = rows_allsum(om);
#pragma unroll
    for (int i = 0; i < NR; ++i) { mu[i] = rows_allsum(mu[i]); yv[i] = rows_allsum(yv[i]); }
    float *R = a.parts + (size_t)pc.rec * S::REC_F;       // this workgroup's record (not FUSED)
    if constexpr (!S::TEAM) {
        finish_workgroup<D, TI, true, FUSED, S::NBUF>(lds, acc, mu, yv, om, mref, mtrue, R, a.out, bh, wave, lane);
    } else {                                              // every wave's own tiles, relative to the true maximum
        const float f = mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - mtrue);
        float *tiles, *mud, *yvd;
        if constexpr (FUSED) { tiles = lds.tiles[0]; mud = lds.mu[0]; yvd = lds.yv[0]; }
        else { tiles = R + S::HDR; mud = R + 64; yvd = R + 64 + D; }
        for_tiles([&](int t) { *reinterpret_cast<f32x4 *>(tiles + t * 256 + lane * 4) = f * acc[t]; });
        if (g == 0) {
#pragma unroll
            for (int i = 0; i < NR; ++i) { mud[16 * row[i] + nn] = f * mu[i]; yvd[16 * row[i] + nn] = f * yv[i]; }
        }
        if (W == 0 && lane == 0) {
            if constexpr (FUSED) lds.om[0] = f * om;
            else { R[0] = mtrue; R[1] = f * om; }
        }
        if constexpr (FUSED) {
            const QueryPart<D> query = load_query<D, TI, true>(a.out, bh, lane);
            __syncthreads();
            solve_head<D, TI, true>(lds, a.out, query, bh, wave, lane);
        }
    }
}

// Two waves per SIMD for the split form at d = 32: four leave 128 registers, 24 too few, and three are still slower (256 heads x 4096
// keys: 53.9, 38.4 and 35.9 us with 1024, 768 and 512 workgroups; on fp32 MFMA 52.6; 512 x 16384: 254, 201, 191 and 303).
template <int D, typename TI, bool FUSED, bool ROOTS>
__global__ __launch_bounds__(NT, D == 32 && sizeof(TI) == 2 ? 2 : D <= 32 ? 4 : (D == 128 && FUSED) ? 1 : 2) void decode_f32_kernel(F32Args a)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    using S = F32Shape<D>;
    if constexpr (S::TEAM) {                              // scalar branches; all four waves meet at the same barriers
        // (the waves of a team write their own parts of the record: only the solve needs the tiles in LDS)
        __shared__ __align__(16) unsigned char raw[FUSED ? sizeof(HeadLds<D, 1, 1>) : 16];
        HeadLds<D, 1, 1> &lds = *reinterpret_cast<HeadLds<D, 1, 1> *>(raw);
        for_pieces<FUSED>(a.split, [&](const DecPiece &pc) {
            if (wave == 0) decode_f32_body<D, TI, FUSED, ROOTS, 0>(a, pc, lds, nullptr, wave, piece_lane());
            else if (wave == 1) decode_f32_body<D, TI, FUSED, ROOTS, 1>(a, pc, lds, nullptr, wave, piece_lane());
            else if (wave == 2) decode_f32_body<D, TI, FUSED, ROOTS, 2>(a, pc, lds, nullptr, wave, piece_lane());
            else decode_f32_body<D, TI, FUSED, ROOTS, 3>(a, pc, lds, nullptr, wave, piece_lane());
        });
    } else {
        using Lds = HeadLds<D, S::NBUF, 4>;
        constexpr size_t STAGES_B = ROOTS ? 4 * (ROOT_STAGE_B + 1024) : 0;
        __shared__ __align__(16) unsigned char raw[STAGES_B > sizeof(Lds) ? STAGES_B : sizeof(Lds)];
        Lds &lds = *reinterpret_cast<Lds *>(raw);
        for_pieces<FUSED>(a.split, [&](const DecPiece &pc) { decode_f32_body<D, TI, FUSED, ROOTS, 0>(a, pc, lds, raw, wave, piece_lane()); },
                          ROOTS && a.heads_first != 0);
    }
}

constexpr size_t MAX_RECORD_BYTES = (size_t)64 << 20;     // what llla_decode_static can hold

// Workgroups per head.  Rounds of the GPU's slots times the keys of a workgroup is the time of the pass; a further workgroup per
// head only pays where it shortens that by more than its record costs (about KEYS_MIN / 4 keys' worth of time).
template <int D>
int f32_nsplit(int bh, int L, size_t ws_bytes, int slots = F32Shape<D>::SLOTS)
{
    using S = F32Shape<D>;
    int best = 1;
    double best_cost = 1e300;
    for (int ns = 1; ns <= S::MAX_SPLIT; ++ns) {
        if (ns > 1 && ((L + ns - 1) / ns < S::KEYS_MIN || (size_t)bh * ns * S::REC_F * sizeof(float) > ws_bytes)) break;
        const double rounds = (double)(((long long)bh * ns + slots - 1) / slots);
        const double cost = rounds * ((double)L / ns + S::KEYS_MIN / 4) + (ns > 1 ? S::KEYS_MIN / 8 * ns : 0);
        if (cost < best_cost) { best_cost = cost; best = ns; }
    }
    return best;
}

// Records that the scratch has room for: the even cut's or the flat one's, whichever is more, where that is useful and fits
template <int D>
size_t f32_records(int B, int H, int L)
{
    using S = F32Shape<D>;
    const int ns = f32_nsplit<D>(B * H, L, MAX_RECORD_BYTES);
    size_t n = ns > 1 ? (size_t)B * H * ns : 0;
    const size_t flat = flat_records(B, H, S::SLOTS);
    if (B >= 2 && L > S::KEYS_MIN && flat * S::REC_F * sizeof(float) <= MAX_RECORD_BYTES) n = std::max(n, flat);
    return n;
}

template <int D>
size_t f32_workspace(int B, int H, int L) { return round_up(f32_records<D>(B, H, L) * F32Shape<D>::REC_F * sizeof(float), 256); }

template <int D, typename TI, bool ROOTS>
hipError_t f32_launch(const Problem &p)
{
    using S = F32Shape<D>;
    const int bh = p.B * p.H;
    F32Args a;
    a.K = p.K; a.V = p.V;
    a.sk = p.sk; a.sv = p.sv;
    // a caller without the scratch that the records need gets one workgroup per head
    const size_t records = f32_records<D>(p.B, p.H, p.n);
    const bool scratch = p.ws != nullptr && (reinterpret_cast<uintptr_t>(p.ws) & 255u) == 0 && p.ws_bytes >= records * S::REC_F * sizeof(float);
    // By roots the even cut counts one workgroup per compute unit, although two fit: on one each they run almost twice as fast, and half the records
    // are left to merge; two from 4096 keys per workgroup on (us with 256 / 512 counted: 256 heads x 512 26 / 34, x 1024 38 / 45, x 8192 231 / 220;
    // 64 x 4096 43.5 / 45.9, 16 x 32768 72 / 74).  The flat cut counts both, in units of 256 keys (128: 64 heads of 1024 to 8192 63.7 instead of
    // 61.7, 32 of 3750 to 30 000 97.0 instead of 94.2, 256 of 256 to 2048 53.4 instead of 55.4).
    const size_t room = ROOTS ? records * S::REC_F * sizeof(float) : MAX_RECORD_BYTES;
    int ns = scratch ? f32_nsplit<D>(bh, p.n, room, ROOTS ? 256 : S::SLOTS) : 1;
    if (ROOTS && scratch && p.n >= 4096 * ns && 2 * bh * ns <= S::SLOTS && 2 * ns <= S::MAX_SPLIT && (size_t)bh * 2 * ns <= records) ns *= 2;
    a.split = choose_split(p, ns, scratch ? records : 0, S::SLOTS, ROOTS ? 256 : 4 * S::STEP, S::KEYS_MIN, S::MAX_SPLIT);
    // Two workgroups of a flat cut share a compute unit only where there are more than compute units: neighbours in the grid go round them, so shares
    // that hold keys come first, all heads' first ones, where a part of the slots stays empty (at most two units of keys per slot, were all sequences
    // as long as the cache).  us, a head's shares together / this: 2 sequences x 16 heads of up to 500 keys 27.3 / 22.4, of up to 5000 36.8 / 33.5, 16 x 16 of up
    // to 900 43.9 / 40.3; with fuller slots it changes little (4 x 16 of up to 8192 59.9 / 60.8, 8 x 16 of up to 8192 89.3 / 87.9).
    a.heads_first = ROOTS && a.split.slots != 0 && (long long)bh * ((p.n + 255) / 256) <= 2 * S::SLOTS ? 1 : 0;
    a.out = HeadOut{p.Q, p.O, p.out == LLLA_BF16 ? 1 : 0, p.lambda};
    a.cscale = p.scale * LOG2E;
    a.parts = static_cast<float *>(p.ws);
    if (a.split.nsplit == 1 && a.split.slots == 0) {
        stage_mark(p.stream, "decode_f32");
        hipLaunchKernelGGL((decode_f32_kernel<D, TI, true, ROOTS>), dim3(1, bh), dim3(NT), 0, p.stream, a);
        // without lengths every sequence is long; with them, those of at most 64 keys are served in key space
        const hipError_t e = hipGetLastError();
        return e != hipSuccess || p.seqlens == nullptr ? e : dual_decode(p);
    } else {
        stage_mark(p.stream, "decode_partial");
        hipLaunchKernelGGL((decode_f32_kernel<D, TI, false, ROOTS>), !a.split.slots ? dim3(a.split.nsplit, bh) : a.heads_first ? dim3(p.H, a.split.slots) : dim3(a.split.slots, p.H),
                           dim3(NT), 0, p.stream, a);
        stage_mark(p.stream, "decode_merge");
        if (p.seqlens == nullptr)
            hipLaunchKernelGGL((decode_merge_kernel<D, TI, true>), dim3(bh), dim3(NT), 0, p.stream, a.split, a.out, (const float *)a.parts,
                               dual::DualArgs{}, 0);
        else
            hipLaunchKernelGGL((decode_merge_kernel<D, TI, true, true>), dim3(2 * bh), dim3(NT), 0, p.stream, a.split, a.out,
                               (const float *)a.parts, dual::dual_args(p), bh);
    }
    return hipGetLastError();
}

template <int D>
hipError_t f32_by_dtype(const Problem &p)
{
    if constexpr (D == 64) {
        if (p.in == LLLA_F32) return f32_launch<D, float, true>(p);
    } else {
        if (p.in == LLLA_F32) return f32_launch<D, float, false>(p);
    }
    return f32_launch<D, bf16_t, false>(p);
}

}  // namespace

size_t mfma_decode_f32_workspace_bytes(int B, int H, int L_max, int d)
{
    switch (d) {
        case 16: return f32_workspace<16>(B, H, L_max);
        case 32: return f32_workspace<32>(B, H, L_max);
        case 64: return f32_workspace<64>(B, H, L_max);
        case 128: return f32_workspace<128>(B, H, L_max);
        default: return 0;
    }
}

bool mfma_decode_f32_takes(const Problem &p)
{
    // per-lane byte offsets inside a chunk of four keys are kept in 32 bits; (batch, head) is the y dimension of the grid
    const int64_t reach = 4 * 4 * (p.sk.seq > p.sv.seq ? p.sk.seq : p.sv.seq);
    return p.n > dual_max_keys(p.d) && reach < (int64_t(1) << 31) && (int64_t)p.B * p.H <= 65535;
}

hipError_t mfma_decode_f32(const Problem &p)
{
    switch (p.d) {
        case 16: return f32_by_dtype<16>(p);
        case 32: return f32_by_dtype<32>(p);
        case 64: return f32_by_dtype<64>(p);
        case 128: return f32_by_dtype<128>(p);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace llla
