// Device helpers shared by the matrix-core (MFMA) kernels of the gfx950 LLA library: vector types,
// MFMA wrappers, DPP broadcasts, LDS DMA, and the on-chip exact solve of the per-query system.
#pragma once

#include <type_traits>

#include "llla_common.hpp"

namespace llla {
namespace mfma {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KB = 32;         // keys per workspace tile / MFMA step
constexpr float LOG2E = 1.4426950408889634f;

// Shape of the matrix-core kernels for head dimension DD (64 or 128).  The second moment of one
// query is NTILE upper-triangular 16x16 fp32 tiles = 4*NTILE accumulator registers per lane, which
// fixes how many queries a wave can carry: 4 at d = 64 (160 registers), 1 at d = 128 (144).
template <int DD>
struct Shape {
    static constexpr int D = DD;
    static constexpr int NB = DD / 16;                 // 16-wide feature blocks
    static constexpr int NTILE = NB * (NB + 1) / 2;    // upper-triangular tiles
    static constexpr int NF = DD / 32;                 // 32-feature steps of a logits MFMA chain
    static constexpr int QW = (DD == 64) ? 4 : 1;      // queries per wave (moments kernel)
    static constexpr int NW = NB;                      // waves per workgroup (moments kernel): one mu~ block each
    static constexpr int QB = QW * NW;                 // queries per workgroup (moments kernel)
    static constexpr int NT = 64 * NW;                 // threads per workgroup (moments kernel)
    static constexpr int YP = DD + 16;                 // pitch of a y row in the workspace: y1[0..D), y0 at [D]; rows start on 64-byte boundaries
    static constexpr int EARLY_ROWS = 2 * DD;          // rows served by the precise variant
    __host__ __device__ static constexpr int tix(int I, int J) { return I * NB - I * (I - 1) / 2 + (J - I); }
};

// Which (batch-head, block) a workgroup serves in a grid (blocks, heads).  Workgroups are handed to the 8 XCDs (each
// with an L2 of its own) round-robin in dispatch order, blockIdx.x fastest.  With the plain mapping the neighbouring
// blocks of one head land on all 8 XCDs and every L2 fetches that head's tiles for itself.  Here a group of 8 heads
// is spread over the 8 XCDs, one head per XCD, and an XCD walks through the blocks of its head in the order given
// (callers put the longest first) before the next group of heads starts: each head's tiles are fetched by one L2
// only.  Heads beyond the last full group of 8 keep the plain mapping.  Used by the moments kernels (16 or 8 rows per
// workgroup, hundreds of workgroups per head).  The 64-row sweeps do not use it: all blocks of a head fit an XCD at
// once, they would start together and the XCD would wait for the longest; those kernels put the head on blockIdx.x.
struct BlockMap { int bh, blk; };
// (32 bits: a call has fewer than 2^31 rows, and a division of 64 costs a workgroup some hundred instructions)
__device__ inline int linear_block() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }
// workgroup `lin` (in dispatch order) of nblk blocks of nbh heads
__device__ inline BlockMap xcd_block_map(int lin, int nblk, int nbh)
{
    const unsigned l = (unsigned)lin, nb = (unsigned)nblk;
    if (l >= (unsigned)(nbh & ~7) * nb) return BlockMap{(int)(l / nb), (int)(l % nb)};
    const unsigned k = l >> 3;
    return BlockMap{(int)(k / nb * 8 + (l & 7)), (int)(k % nb)};
}
__device__ inline BlockMap xcd_block_map() { return xcd_block_map(linear_block(), (int)gridDim.x, (int)gridDim.y); }

// Row broadcasts across the 16-lane rows of a wave: rows 1 and 3 receive lane 15 of rows 0 and 2 (the other rows
// keep x); rows 2 and 3 receive lane 31, the last lane of row 1 (rows 0 and 1 keep x).
__device__ inline float rows_1_3_from_rows_0_2(float x)
{
    const int v = __builtin_bit_cast(int, x);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
}
__device__ inline float rows_2_3_from_row_1(float x)
{
    const int v = __builtin_bit_cast(int, x);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
}

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int C>
__device__ inline float row_bcast(float x)   // value of lane C of the caller's 16-lane row
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x150 + C, 0xf, 0xf, true));
}
template <int J>
__device__ inline float quad_bcast(float x)   // value of lane (lane & ~3) + J
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), J * 0x55, 0xf, 0xf, true));
}
__device__ inline float lane_xor1(float x)   // value of lane ^ 1
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, true));
}

// x = hi + lo with both halves f16 (about 20 significant bits).  hi is x rounded toward zero by a conversion
// builtin on purpose: a plain (_Float16) cast of a product may be fused with the multiply at one use (one
// rounding of the exact product) and not at another (product rounded to fp32 first), the two results can differ
// by one f16 ulp, and a lo computed against the one would then be added to the other.
__device__ inline void split_f16(const float (&x)[8], half8 &hi, half8 &lo)
{
    typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 half2v __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const half2v h = __builtin_bit_cast(half2v, (fp16x2)__builtin_amdgcn_cvt_pkrtz(x[2 * p], x[2 * p + 1]));
        const half2v l = __builtin_bit_cast(
            half2v, (fp16x2)__builtin_amdgcn_cvt_pkrtz(x[2 * p] - (float)h[0], x[2 * p + 1] - (float)h[1]));
        hi[2 * p] = h[0]; hi[2 * p + 1] = h[1];
        lo[2 * p] = l[0]; lo[2 * p + 1] = l[1];
    }
}

typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

// x = h + m + l, three bf16 (24 significant bits; bf16 has the exponents of fp32, so this holds over its whole range).  The
// remainders x - h are v_dot2_f32_bf16 with (-1, 0) and (0, -1), exact like the subtractions they stand for: one instruction per value
// instead of an unpacking and a subtraction.  (The two constants come in scalar registers: as a literal the compiler encodes (-1, 0)
// as the inline constant -1.0, which this instruction reads as the fp32 bit pattern, i.e. (0, -1); seen with ROCm 7.2.)
// The stages of the eight values are kept apart (the empty statements): a vector instruction that reads the result of v_dot2_f32_bf16 less than three
// instructions later is held up, and the scheduler, left to itself, put the two next to each other.
__device__ inline void tie8(float (&x)[8])
{
    asm("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
}
__device__ inline void split3_bf16(const float (&x)[8], bf16x8 &h, bf16x8 &m, bf16x8 &l)
{
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    asm("" : "+s"(lo), "+s"(hi));
    const bf16x2v first = __builtin_bit_cast(bf16x2v, lo), second = __builtin_bit_cast(bf16x2v, hi);
    float r[8];
    auto terms = [&](const float (&v)[8], bf16x8 &o) {
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            const bf16x2v a = __builtin_convertvector(float2v{v[t], v[t + 1]}, bf16x2v);
            o[t] = a[0]; o[t + 1] = a[1];
        }
    };
    auto remainders = [&](const bf16x8 &o, const float (&v)[8]) {
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            const bf16x2v a = {o[t], o[t + 1]};
            r[t] = __builtin_amdgcn_fdot2_f32_bf16(a, first, v[t], false);
            r[t + 1] = __builtin_amdgcn_fdot2_f32_bf16(a, second, v[t + 1], false);
        }
        tie8(r);
    };
    terms(x, h);
    remainders(h, x);
    terms(r, m);
    remainders(m, r);
    terms(r, l);
}

// 2 x for finite x of at least 2^-126 in absolute value, by the exponent field (a smaller x becomes x +- 2^-126; infinities are not kept)
__device__ inline bf16x8 twice_bf16(bf16x8 x)
{
    typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (u16x8)(__builtin_bit_cast(u16x8, x) + (unsigned short)0x80));
}

__device__ inline f32x4 mfma_f16(half8 a, half8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
__device__ inline f32x4 mfma_bf16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// C += A^T B for 16x16 fp32 tiles held in the MFMA accumulator layout (lane (g,n), reg t = X[4g+t][n]).
// The contraction slot (chunk kc, lane group g) is mapped to index 4g+kc, which is exactly where
// register kc of both tiles sits, so no data moves.
__device__ inline f32x4 tile_atb(f32x4 c, f32x4 a, f32x4 b)
{
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kc], b[kc], c, 0, 0, 0);
    return c;
}

// The same on 16-bit MFMA from operands in three bf16 (see split3_bf16): a tile's terms m, h, l lie side by side, so (m, h) and (h, l)
// are operands whose two halves are the same sixteen rows in two terms, and three MFMAs are the six products that count --
// hm + lh, mh + hl, mm + hh; what is left out is below 2^-24 of the result.  48 cycles of the matrix cores instead of 128, for 14
// vector instructions per operand tile.
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x6 __attribute__((ext_vector_type(6)));
__device__ inline u32x6 split_tile(f32x4 x)
{
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    asm("" : "+s"(lo), "+s"(hi));
    const bf16x2v first = __builtin_bit_cast(bf16x2v, lo), second = __builtin_bit_cast(bf16x2v, hi);
    u32x6 r;
    float v[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
    for (int term = 0; term < 3; ++term) {                // h, m, l; the stages kept apart as in split3_bf16
        const int at = term == 0 ? 2 : term == 1 ? 0 : 4;
        const bf16x2v a = __builtin_convertvector(float2v{v[0], v[1]}, bf16x2v), b = __builtin_convertvector(float2v{v[2], v[3]}, bf16x2v);
        r[at] = __builtin_bit_cast(unsigned, a);
        r[at + 1] = __builtin_bit_cast(unsigned, b);
        if (term == 2) break;
        v[0] = __builtin_amdgcn_fdot2_f32_bf16(a, first, v[0], false);
        v[1] = __builtin_amdgcn_fdot2_f32_bf16(a, second, v[1], false);
        v[2] = __builtin_amdgcn_fdot2_f32_bf16(b, first, v[2], false);
        v[3] = __builtin_amdgcn_fdot2_f32_bf16(b, second, v[3], false);
        asm("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    }
    return r;
}
__device__ inline f32x4 split_atb(f32x4 c, const u32x6 &a, const u32x6 &b)
{
    const bf16x8 amh = __builtin_bit_cast(bf16x8, (u32x4v)__builtin_shufflevector(a, a, 0, 1, 2, 3));
    const bf16x8 ahl = __builtin_bit_cast(bf16x8, (u32x4v)__builtin_shufflevector(a, a, 2, 3, 4, 5));
    const bf16x8 bmh = __builtin_bit_cast(bf16x8, (u32x4v)__builtin_shufflevector(b, b, 0, 1, 2, 3));
    const bf16x8 bhl = __builtin_bit_cast(bf16x8, (u32x4v)__builtin_shufflevector(b, b, 2, 3, 4, 5));
    c = mfma_bf16(ahl, bmh, c);
    c = mfma_bf16(amh, bhl, c);
    return mfma_bf16(amh, bmh, c);
}

constexpr int SC_PITCH = 20;         // floats per row of a 16x16 scratch tile

// ---- diagonal tiles -----------------------------------------------------------------------------------------------------------
// Their factorisation is most of the vector work of every solve in the library and is bound by instruction issue (two waves share a
// SIMD and the matrix cores add nothing to it), so what counts is the number of instructions.  Row-broadcast multiply-adds are VOP2 DPP
// instructions; the compiler does not fuse a DPP move into an FMA by itself.  A DPP read needs two wait states after a vector-ALU
// write of the register it reads, and the compiler's hazard handling does not look inside inline assembly: every statement
// starts with its own s_nop 1, all registers it reads through DPP are operands of the statement (whatever wrote them lies before that
// s_nop), and what a statement both writes and reads through DPP lies two instructions apart or has an s_nop between.
#define LLLA_FROM(M, K) LLLA_FROM_##K(M)
#define LLLA_FROM_15(M) M(15)
#define LLLA_FROM_14(M) M(14) LLLA_FROM_15(M)
#define LLLA_FROM_13(M) M(13) LLLA_FROM_14(M)
#define LLLA_FROM_12(M) M(12) LLLA_FROM_13(M)
#define LLLA_FROM_11(M) M(11) LLLA_FROM_12(M)
#define LLLA_FROM_10(M) M(10) LLLA_FROM_11(M)
#define LLLA_FROM_9(M) M(9) LLLA_FROM_10(M)
#define LLLA_FROM_8(M) M(8) LLLA_FROM_9(M)
#define LLLA_FROM_7(M) M(7) LLLA_FROM_8(M)
#define LLLA_FROM_6(M) M(6) LLLA_FROM_7(M)
#define LLLA_FROM_5(M) M(5) LLLA_FROM_6(M)
#define LLLA_FROM_4(M) M(4) LLLA_FROM_5(M)
#define LLLA_FROM_3(M) M(3) LLLA_FROM_4(M)
#define LLLA_FROM_2(M) M(2) LLLA_FROM_3(M)
#define LLLA_FROM_1(M) M(1) LLLA_FROM_2(M)
#define LLLA_DPP(C) " row_newbcast:" #C " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"

// max(x of lane K of the caller's 16-lane row, lo); a NaN gives lo
template <int K>
__device__ inline float bcast_max(float x, float lo)
{
    float d;
    asm volatile("s_nop 1\n\tv_max_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1" : "=v"(d) : "v"(x), "v"(lo), "n"(K));
    return d;
}
template <int K>
__device__ inline float bcast_settled(float src)     // row broadcast of a value that inline assembly may have written
{
    float d;
    asm volatile("s_nop 1\n\tv_mov_b32_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf bound_ctrl:1" : "=v"(d) : "v"(src), "n"(K));
    return d;
}
// a[c] -= (v of lane c of the row) * v for c = K+1 .. 15
template <int K>
__device__ inline void rank1_row(float (&a)[16], float v)
{
#define F(C) "v_fmac_f32_dpp %[a" #C "], %[v], -%[v]" LLLA_DPP(C)
#define O(C) , [a##C] "+v"(a[C])
#define LLLA_RANK1(K, C) \
    if constexpr (K == C - 1) asm volatile("s_nop 1\n\t" LLLA_FROM(F, C) : [v] "+v"(v) LLLA_FROM(O, C));
    LLLA_RANK1(K, 1) LLLA_RANK1(K, 2) LLLA_RANK1(K, 3) LLLA_RANK1(K, 4) LLLA_RANK1(K, 5) LLLA_RANK1(K, 6) LLLA_RANK1(K, 7) LLLA_RANK1(K, 8)
    LLLA_RANK1(K, 9) LLLA_RANK1(K, 10) LLLA_RANK1(K, 11) LLLA_RANK1(K, 12) LLLA_RANK1(K, 13) LLLA_RANK1(K, 14) LLLA_RANK1(K, 15)
#undef LLLA_RANK1
#undef O
#undef F
}

// Cholesky factorisation S = L D L^T (L unit lower triangular) of the symmetric tiles of the wave's systems: lane 16 q + r owns row r of
// system q's tile, a[c] = S[r][c].  On return (a destroyed)
//   nl[k] = -L[r][k] for r > k, else 0  (k = 0..14);   ndinv = -D[r]^(-1/2).
// What is subtracted are columns v = D^(1/2) L, the same rounded values on both sides of the product and D^(-1/2) the one that ndinv
// returns: the rounding errors of L and D then cancel in the products of the tiles.  With L[r][k] on one side and a[k] on the other (no
// roots on the way, three instructions less per step) the errors of fp32 rows were 0.5-1 % larger, and rows of sharp weights missed their bound.
// Per tile, inverse included, 520 instructions (690 with a statement and its wait states per 8, 4, 2 and 1 columns and the inverse started
// from the identity): 96 heads x 1000 rows of the bf16 forward at d = 64 500 -> 482 us, 64 x 4096 2880 -> 2845, decode of 16 x 4096 keys
// 26.2 -> 24.5.  The root is the hardware's estimate, which is within one unit in the last place: a Newton step, whose own roundings are as
// large, changed the errors of no call (forward, backward, decode, d = 32 to 128, both types: 0.98 to 1.02 times, without a trend) and is a sixth
// of the instructions (16 x 2048, d = 128, 1088 -> 1057 us; 160 x 376, d = 64, 225 -> 219, 96 x 1000 436 -> 428, 64 x 4096 2758 -> 2737).
// pivot_floor: every pivot D of (a positive semi-definite matrix + lambda I) is at least lambda in exact arithmetic; a computed
// pivot below the floor (half of lambda) is a rounding artefact of an ill-conditioned row and is raised to it, which keeps the
// factorisation finite.  LOW: *low becomes the smallest pivot before that, if smaller (NaN pivots are passed over).
// DROP: such a pivot is not raised but made infinite, which takes its column and its unknown out of the system.  Where the pivot is
// noise its column is too, of the size of the matrix's rounding: divided by the root of a raised pivot a few such columns in a row
// overflow.
template <bool LOW, bool DROP>
__device__ inline void eliminate16(float (&a)[16], float (&nl)[16], float &ndinv, int r, float pivot_floor, float *low)
{
    float own = 0.f;
    auto step = [&](auto ktag) {
        constexpr int K = decltype(ktag)::value;
        const float ak = a[K];
        float d;
        if constexpr (LOW || DROP) d = bcast_settled<K>(ak);
        if constexpr (LOW) *low = fminf(*low, d);
        if constexpr (LOW && !DROP) d = fmaxf(d, pivot_floor);
        if constexpr (!LOW && !DROP) d = bcast_max<K>(ak, pivot_floor);
        float rinv = __builtin_amdgcn_rsqf(d);
        if constexpr (DROP) rinv = d < pivot_floor ? 0.f : rinv;
        own = (r == K) ? rinv : own;
        if constexpr (K < 15) {
            const float v = ak * rinv;                       // in rows r >= K; the others are finished and never read again
            nl[K] = (r > K) ? -v * rinv : 0.f;
            rank1_row<K>(a, v);                              // a[c] -= v[r] v[c], c > K
        }
    };
#define STEP(K) step(std::integral_constant<int, K>{});
    STEP(0) LLLA_FROM(STEP, 1)
#undef STEP
    ndinv = -own;
}

// The inverse of what eliminate16 found: li[c] = -(D^(-1/2) L^-1)[r][c], zero above the diagonal (with S = U^T U that is
// -(U^-T)[r][c]).  M = L^-1: M[r][c] = [r == c] - sum_{c<=p<r} L[r][p] M[p][c]; column p starts as the first term that it takes.
__device__ inline void invert16(const float (&nl)[16], float ndinv, int r, float (&li)[16])
{
#pragma unroll
    for (int c = 0; c < 15; ++c) li[c] = (r == c) ? 1.f : nl[c];
    li[15] = (r == 15) ? 1.f : 0.f;
#define G(C, P) "v_fmac_f32_dpp %[l" #C "], %[l" #C "], %[n" #P "]" LLLA_DPP(P)
#define R1(P) G(0, P)
#define R2(P) R1(P) G(1, P)
#define R3(P) R2(P) G(2, P)
#define R4(P) R3(P) G(3, P)
#define R5(P) R4(P) G(4, P)
#define R6(P) R5(P) G(5, P)
#define R7(P) R6(P) G(6, P)
#define R8(P) R7(P) G(7, P)
#define R9(P) R8(P) G(8, P)
#define R10(P) R9(P) G(9, P)
#define R11(P) R10(P) G(10, P)
#define R12(P) R11(P) G(11, P)
#define R13(P) R12(P) G(12, P)
#define R14(P) R13(P) G(13, P)
#define L(C) [l##C] "+v"(li[C])
#define N(C) [n##C] "v"(nl[C])
    asm volatile("s_nop 1\n\t" R1(1) "s_nop 1\n\t" R2(2) "s_nop 0\n\t" R3(3) R4(4) R5(5) R6(6) R7(7)
                 : L(0), L(1), L(2), L(3), L(4), L(5), L(6)
                 : N(1), N(2), N(3), N(4), N(5), N(6), N(7));
    asm volatile("s_nop 1\n\t" R8(8) R9(9) R10(10) R11(11) R12(12) R13(13) R14(14)
                 : L(0), L(1), L(2), L(3), L(4), L(5), L(6), L(7), L(8), L(9), L(10), L(11), L(12), L(13)
                 : N(8), N(9), N(10), N(11), N(12), N(13), N(14));
#undef N
#undef L
#undef R14
#undef R13
#undef R12
#undef R11
#undef R10
#undef R9
#undef R8
#undef R7
#undef R6
#undef R5
#undef R4
#undef R3
#undef R2
#undef R1
#undef G
#pragma unroll
    for (int c = 0; c < 16; ++c) li[c] *= ndinv;
}

// The same for ONE system, whose tile the four 16-lane rows of the wave hold four copies of: lane (g, r) forms columns 4g..4g+3 of
// its row only, li[t] = -(D^(-1/2) L^-1)[r][4g+t].  That is 60 multiply-adds instead of 105, and what a lane then holds is the
// fragment of N = -U^-1 in the accumulator layout (register t = N[4g+t][r]): no exchange through LDS.
__device__ inline f32x4 invert16_quarter(const float (&nl)[16], float ndinv, int r, int g)
{
    float l0 = (r == 4 * g) ? 1.f : 0.f, l1 = (r == 4 * g + 1) ? 1.f : 0.f, l2 = (r == 4 * g + 2) ? 1.f : 0.f, l3 = (r == 4 * g + 3) ? 1.f : 0.f;
#define G(C, P) "v_fmac_f32_dpp %[l" #C "], %[l" #C "], %[n" #P "]" LLLA_DPP(P)
#define Q(P) G(0, P) G(1, P) G(2, P) G(3, P)
#define N(C) [n##C] "v"(nl[C])
    asm volatile("s_nop 1\n\t" Q(0) Q(1) Q(2) Q(3) Q(4) Q(5) Q(6) Q(7) Q(8) Q(9) Q(10) Q(11) Q(12) Q(13) Q(14)
                 : [l0] "+v"(l0), [l1] "+v"(l1), [l2] "+v"(l2), [l3] "+v"(l3)
                 : N(0), N(1), N(2), N(3), N(4), N(5), N(6), N(7), N(8), N(9), N(10), N(11), N(12), N(13), N(14));
#undef N
#undef Q
#undef G
    return f32x4{l0 * ndinv, l1 * ndinv, l2 * ndinv, l3 * ndinv};
}

typedef __attribute__((address_space(3))) void *lds_void_ptr;
typedef const __attribute__((address_space(1))) void *glb_void_ptr;

// 16 bytes per lane straight from global memory into LDS (no registers): lane l's data lands at
// lds_base + 16 l, the global address is per lane.  Written as inline assembly on purpose: the
// compiler makes every later LDS read wait for a DMA it knows about (it cannot tell the two
// buffers apart), which would serialise the prefetch; here the waits are placed by hand with
// dma_wait() before the data is read.  The s_nop is the wait state gfx9 needs between a scalar
// write of M0 and an LDS-DMA instruction that reads it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void dma16(const void *gsrc, void *lds_base)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_ptr)lds_base);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gsrc), "s"(lds) : "memory", "m0");
}
// The same with a wave-uniform base address in scalar registers plus a 32-bit per-lane byte offset: no vector-ALU
// address arithmetic per transfer.
__device__ inline void dma16_base(const void *sbase, unsigned voff, void *lds_base)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_ptr)lds_base);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds) : "memory", "m0");
}
// The same with the LDS destination given as a byte offset into the workgroup's LDS (lds_offset of the array plus
// plain integer arithmetic): a pointer that went through pointer arithmetic in the generic address space costs four
// scalar instructions per transfer to turn back into an LDS address.
__device__ inline unsigned lds_offset(const void *lds_object) { return (unsigned)(uintptr_t)(lds_void_ptr)lds_object; }
__device__ inline void dma16_base_off(const void *sbase, unsigned voff, unsigned lds_byte_off)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane(lds_byte_off);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds) : "memory", "m0");
}
// The same two transfers with the non-temporal hint, for data that is read exactly once (the decode kernel's cache
// stream): without it the stream stays about 10 % below what plain streaming loads reach on this part.
__device__ inline void dma16_nt(const void *gsrc, void *lds_base)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_ptr)lds_base);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(gsrc), "s"(lds) : "memory", "m0");
}
__device__ inline void dma16_base_nt(const void *sbase, unsigned voff, void *lds_base)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_void_ptr)lds_base);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(sbase), "s"(lds) : "memory", "m0");
}
// (and with the LDS destination as a byte offset, see dma16_base_off)
__device__ inline void dma16_nt_off(const void *gsrc, unsigned lds_byte_off)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane(lds_byte_off);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(gsrc), "s"(lds) : "memory", "m0");
}
__device__ inline void dma16_base_nt_off(const void *sbase, unsigned voff, unsigned lds_byte_off)
{
    const unsigned lds = __builtin_amdgcn_readfirstlane(lds_byte_off);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(sbase), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ inline void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// all but this wave's N youngest transfers (and loads and stores) have landed
template <int N>
__device__ inline void dma_wait_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// index of tile (I, J), I <= J, among the upper-triangular 16x16 tiles of a matrix of NB 16-wide blocks (row by row)
template <int NB>
__host__ __device__ constexpr int upper_tile(int I, int J) { return I * NB - I * (I - 1) / 2 + (J - I); }

// A symmetric tile from the accumulator layout to one row per lane: a[c] = X[n][c] in lane (g, n), four copies.  Column n is what the four lanes
// (g, n) hold between them, so the four 16-lane rows exchange their registers (inline assembly and its s_nop: see rows_transpose4); through
// LDS, a write and a read in a chain, it took three times as long.
__device__ __forceinline__ void symmetric_rows(const f32x4 &x, float (&a)[16])
{
    float e0 = x[0], e1 = x[1], e2 = x[2], e3 = x[3], f0 = e0, f1 = e1, f2 = e2, f3 = e3;
    asm volatile("s_nop 1\n\t"
                 "v_permlane16_swap_b32 %0, %4\n\t"
                 "v_permlane16_swap_b32 %1, %5\n\t"
                 "v_permlane16_swap_b32 %2, %6\n\t"
                 "v_permlane16_swap_b32 %3, %7"
                 : "+v"(e0), "+v"(e1), "+v"(e2), "+v"(e3), "+v"(f0), "+v"(f1), "+v"(f2), "+v"(f3));      // rows 0 0 2 2 and 1 1 3 3
    float g0 = e0, g1 = e1, g2 = e2, g3 = e3, h0 = f0, h1 = f1, h2 = f2, h3 = f3;
    asm volatile("s_nop 1\n\t"
                 "v_permlane32_swap_b32 %0, %8\n\t"
                 "v_permlane32_swap_b32 %1, %9\n\t"
                 "v_permlane32_swap_b32 %2, %10\n\t"
                 "v_permlane32_swap_b32 %3, %11\n\t"
                 "v_permlane32_swap_b32 %4, %12\n\t"
                 "v_permlane32_swap_b32 %5, %13\n\t"
                 "v_permlane32_swap_b32 %6, %14\n\t"
                 "v_permlane32_swap_b32 %7, %15"
                 : "+v"(e0), "+v"(e1), "+v"(e2), "+v"(e3), "+v"(f0), "+v"(f1), "+v"(f2), "+v"(f3), "+v"(g0), "+v"(g1), "+v"(g2), "+v"(g3),
                   "+v"(h0), "+v"(h1), "+v"(h2), "+v"(h3));
    a[0] = e0; a[1] = e1; a[2] = e2; a[3] = e3;
    a[4] = f0; a[5] = f1; a[6] = f2; a[7] = f3;
    a[8] = g0; a[9] = g1; a[10] = g2; a[11] = g3;
    a[12] = h0; a[13] = h1; a[14] = h2; a[15] = h3;
}

// Blocked factorisation of ONE system per wave, all in registers / wave-private LDS scratch (the first half of solve_one;
// solve_wave_q4 has its own for four systems at d = 64):
//   in : acc[upper_tile(I,J)]  upper-triangular 16x16 tiles of T = -(Sigma~ + lambda I) (MFMA accumulator layout)
//        scw                   >= 16*SC_PITCH floats of LDS owned by this wave
//        pivot_floor           half the ridge of the row (see eliminate16)
//   out: acc(P,J), P < J, holds U(P,J) and acc(P,P) holds N_P = -U(P,P)^{-1}, with Sigma~ + lambda I = U^T U.
// 16-blocked upper Cholesky whose block products are C += A^T B on fp32 MFMA; the diagonal tile is factorised with one
// row per lane and DPP row broadcasts (the four lane groups of the wave hold four copies).  The matrix cores only add
// products, so everything that the textbook recursion subtracts is carried negated instead: the trailing matrix (T), the
// inverse diagonal factors (N_P), and, in the substitutions, the partial right-hand sides; no tile is ever negated on
// the vector ALU.
// LOW: low as in eliminate16, over all pivots.
// SPLIT: the block products on 16-bit MFMA from operands in three bf16.  fp32 MFMA and vector instructions of the two waves of a SIMD do not
// overlap, and 112 tile products at d = 128 are a third of the solve.  Each product starts from zero and is added to its tile on the vector
// ALU: chained onto the tile its three MFMAs left errors of up to 1.09 times those of fp32 MFMA, which rounds at each of a product's sixteen
// rows; so they are 0.80 to 0.99 times those (O, dQ, dK, dV; 140 to 400 rows, bf16 and fp32).  us a call, fp32 MFMA and split: 16 heads x
// 2048 1049 and 1012, 16 x 8192 9674 and 9613, 8 x 44 46.7 and 43.8, backward 8 x 961 402 and 386; fp32 64 x 700 2413 and 2357.  Decode at
// d = 128, one solve per compute unit, gains nothing (224 heads of up to 589 keys 54.7 and 55.6), nor do four systems per wave at d = 64 (64 x 4096 bf16
// 2829 and 2916, 16 x 1024 fp32 346 and 352).
// SYMMETRIC: the diagonal tiles come in symmetric to the last bit and stay so under their updates (fp32 products u^T u, with SPLIT = false), and the
// factorisation takes one triangle of them (symmetric_rows); otherwise it takes the mean of the two.
template <int NB, bool LOW = false, bool DROP = false, bool SPLIT = true, bool SYMMETRIC = false>
__device__ __forceinline__ void factorise_one(f32x4 (&acc)[NB * (NB + 1) / 2], float *scw, int g, int nn, float pivot_floor, float *low = nullptr)
{
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        float a[16], nl[16], ndinv;
        if constexpr (SYMMETRIC) {
            symmetric_rows(-acc[upper_tile<NB>(P, P)], a);
        } else {                                          // one row per lane, symmetrised
#pragma unroll
            for (int t = 0; t < 4; ++t) scw[(4 * g + t) * SC_PITCH + nn] = acc[upper_tile<NB>(P, P)][t];
            wave_sync();
#pragma unroll
            for (int c4 = 0; c4 < 4; ++c4) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(scw + nn * SC_PITCH + 4 * c4);
#pragma unroll
                for (int t = 0; t < 4; ++t) a[4 * c4 + t] = v[t];
            }
#pragma unroll
            for (int c = 0; c < 16; ++c) a[c] = -0.5f * (a[c] + scw[c * SC_PITCH + nn]);    // -T, symmetrised
            wave_sync();
        }
        eliminate16<LOW, DROP>(a, nl, ndinv, nn, pivot_floor, low);
        // N_P replaces the consumed diagonal tile; U(P,J) = N_P^T T(P,J), and the trailing tiles take T(I,J) += U(P,I)^T U(P,J)
        const f32x4 ui = invert16_quarter(nl, ndinv, nn, g);
        acc[upper_tile<NB>(P, P)] = ui;
        if constexpr (!SPLIT) {
#pragma unroll
            for (int J = P + 1; J < NB; ++J) acc[upper_tile<NB>(P, J)] = tile_atb(zero, ui, acc[upper_tile<NB>(P, J)]);
#pragma unroll
            for (int I = P + 1; I < NB; ++I)
#pragma unroll
                for (int J = I; J < NB; ++J)
                    acc[upper_tile<NB>(I, J)] = tile_atb(acc[upper_tile<NB>(I, J)], acc[upper_tile<NB>(P, I)], acc[upper_tile<NB>(P, J)]);
        } else if (P + 1 < NB) {
            const u32x6 us = split_tile(ui);
            u32x6 row[NB];
#pragma unroll
            for (int J = P + 1; J < NB; ++J) {
                f32x4 &u = acc[upper_tile<NB>(P, J)];
                u = split_atb(zero, us, split_tile(u));
                row[J] = split_tile(u);
            }
#pragma unroll
            for (int I = P + 1; I < NB; ++I)
#pragma unroll
                for (int J = I; J < NB; ++J) acc[upper_tile<NB>(I, J)] += split_atb(zero, row[I], row[J]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The same with further block columns (the decode tail's solve at d <= 64):
//   in : x[v][P]               NX further block columns, negated right-hand sides -B in the same layout
//   out: x = U^{-T} B; returns the smallest pivot before it was raised to the floor
// Diagonal tiles come in symmetric; their updates in three bf16 add the mixed terms [i][j] and [j][i] in another order each and leave them up to a rounding
// apart, and the elimination takes one triangle, the lower.  What bounds it is one chain per head: per diagonal tile rows, 1400
// cycles of elimination, 300 of inversion, products.  Rows by lane exchanges and products in three bf16, against a way through LDS and fp32 MFMA, with the
// query's early request: us a call, 16 heads x 4096 23.7 -> 23.4, 16 x 512 (solved by the pass) 17.4 -> 16.3; errors 0.6 to 1.0 times the former.
template <int NB, int NX>
__device__ __forceinline__ float factorise_columns(f32x4 (&acc)[NB * (NB + 1) / 2], int g, int nn, float pivot_floor, f32x4 (&x)[NX][NB])
{
    float low = INFINITY;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        float a[16], nl[16], ndinv;
        symmetric_rows(-acc[upper_tile<NB>(P, P)], a);
        eliminate16<true, false>(a, nl, ndinv, nn, pivot_floor, &low);
        // N_P replaces the consumed diagonal tile; U(P,J) = N_P^T T(P,J), and the trailing tiles take T(I,J) += U(P,I)^T U(P,J)
        const f32x4 ui = invert16_quarter(nl, ndinv, nn, g);
        const u32x6 us = split_tile(ui);
        u32x6 row[NB], xs[NX];
#pragma unroll
        for (int J = P + 1; J < NB; ++J) {
            f32x4 &u = acc[upper_tile<NB>(P, J)];
            u = split_atb(zero, us, split_tile(u));
            row[J] = split_tile(u);
        }
#pragma unroll
        for (int v = 0; v < NX; ++v) {
            x[v][P] = split_atb(zero, us, split_tile(x[v][P]));
            if (P + 1 < NB) xs[v] = split_tile(x[v][P]);
        }
#pragma unroll
        for (int I = P + 1; I < NB; ++I) {
#pragma unroll
            for (int J = I; J < NB; ++J) acc[upper_tile<NB>(I, J)] += split_atb(zero, row[I], row[J]);
#pragma unroll
            for (int v = 0; v < NX; ++v) x[v][I] += split_atb(zero, row[I], xs[v]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    return low;
}

}  // namespace mfma
}  // namespace llla
