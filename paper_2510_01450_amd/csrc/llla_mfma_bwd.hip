// Matrix-core sweeps of the LLA backward pass (bf16 inputs, d = 64 / 128).  Key sweep: dK_j and dV_j of a block of keys,
// summed over the query rows at and after the block (Appendix D: Delta_V = S^T G and the key-side sums of the
// w- and z-paths, here in the un-centred form described at the top of llla_bwd.hip).
//
// A wave owns 16 keys and walks over the query rows in steps of 32.  Per step, with C = A B on 16x16x32 bf16 MFMA:
//   * four products of a [16 queries x d] row tile with the wave's key (or value) fragments give, in the accumulator
//     layout (lane (g, nn): queries 4g..4g+3, key nn), the logits q_i.k_j, the linear forms y1_i.k_j and u1_i.k_j
//     (y1, u1 as bf16 hi + lo) and gamma_ij = dO_i.v_j; y0 and -u0 are the accumulators' starting values, and gamma joins
//     the chain of -u1.k, so that w a and w (gamma - b) are one product each;
//   * the vector ALU turns them into the three coefficient tiles s_ij, e_ij, scale p^_ij and splits each into
//     bf16 hi + lo;
//   * those registers are already the A operand of the second product family, whose contraction index is the query
//     (slot 4s+r of lane group g <-> query 16s+4g+r): dV += S^T dO,  dK += E^T Y1 - S^T U1 + scale P^T Q.  The B operands
//     are the same row tiles read transposed by ds_read_tr16_b64 (lane nn gets four consecutive queries of feature
//     16J+nn), so no tile is stored twice.
// Accumulators stay in registers for the whole sweep; every output element is written once (no atomics).
//
// What bounds it: 64 MFMAs (1024 cycles) and some 160 vector instructions per step and 16 keys, in a chain products -> coefficients ->
// products; the two kinds of work hardly overlap between waves, so the rest has to stay out of the way.  The dQ sweep leaves y1 and -u1
// of every row split into bf16 hi and lo, in the place of the fp32 rows (one split per row instead of one per row and block of 64
// keys), which lets all six tiles of a step arrive by DMA, at d = 64 one step ahead into a second buffer with one barrier per step,
// scalar bases and constant offsets.  Mask and correction of the maximum are one scalar branch each per step.
// NK = 2 (d = 64): two blocks of 16 keys per wave share every operand fragment (a wave reads 48 KB of LDS per step, with one block
// 1.5 times what LDS delivers while its products run).  It pays from TWO_KEY_BLOCKS_FROM workgroups of 128 keys on: 64 heads x 4096 rows
// 1063 -> 942 us (one block 1036), 96 x 1000 130 -> 124; below, the longest workgroup decides: 16 x 4096 318 -> 390, 16 x 1000 57 -> 83.
#include "llla_mfma_common.hpp"

namespace llla {
namespace {

using namespace mfma;

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v *lds_short4_ptr;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int QS = 32;        // query rows per step

// transposed fragment of a natural [32 rows][pitch P halves] tile: for feature 16J + nn the rows 4g..4g+3 and
// 16+4g..16+4g+3 -- addr is the lane's own address (row 4g + nn/4, features 16J + 4(nn%4)..) in halves
__device__ inline bf16x8 tr_frag(const bf16_t *tile, int addr, int pitch)
{
    const short4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(tile + addr));
    const short4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(tile + 16 * pitch + addr));
    const uint2 au = __builtin_bit_cast(uint2, a), bu = __builtin_bit_cast(uint2, b);
    return __builtin_bit_cast(bf16x8, make_uint4(au.x, au.y, bu.x, bu.y));
}

// x = hi + lo with both halves bf16, two values per conversion instruction and one per remainder (see split3_bf16)
__device__ inline void split_bf16(const float (&x)[8], bf16x8 &hi, bf16x8 &lo)
{
    unsigned c0 = 0x0000bf80u, c1 = 0xbf800000u;
    asm("" : "+s"(c0), "+s"(c1));
    const bf16x2v first = __builtin_bit_cast(bf16x2v, c0), second = __builtin_bit_cast(bf16x2v, c1);
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
        const bf16x2v h = __builtin_convertvector(float2v{x[t], x[t + 1]}, bf16x2v);
        const bf16x2v l = __builtin_convertvector(float2v{__builtin_amdgcn_fdot2_f32_bf16(h, first, x[t], false),
                                                          __builtin_amdgcn_fdot2_f32_bf16(h, second, x[t + 1], false)}, bf16x2v);
        hi[t] = h[0]; hi[t + 1] = h[1];
        lo[t] = l[0]; lo[t + 1] = l[1];
    }
}

// The tiles of the key sweep: rows of DD halves without padding (the DMA writes whole 1 KB wave rows), 16-byte chunk c of row r at
// c ^ row_swizzle(r).  Sixteen rows read at one chunk land on 16 different chunk positions of the 64 banks (d = 64: two rows per
// 256 bytes, so 8 positions for the rows of one parity), and the chunk pairs that a half-wave of a transposing read takes from 8
// rows are disjoint.  Rows 16 apart share their swizzle.
template <int DD>
__device__ inline int row_swizzle(int r)
{
    if (DD == 64) { const int k = (r >> 1) & 7; return ((k & 3) << 1) | (k >> 2); }
    return ((r & 7) << 1) | ((r >> 3) & 1);
}

// LIVE < NB (a d = 16 / 32 call on zero-padded copies): features and value columns from 16 LIVE on are zero; the contractions stop after
// the chunks that hold live ones, and only live columns are formed and stored, in rows of 16 LIVE.  The same in the row sweeps below.
template <int DD, int NK, int LIVE = Shape<DD>::NB>
__global__ __launch_bounds__(256, DD == 64 && NK == 1 ? 3 : 2) void bwd_keys_mfma_kernel(
    const bf16_t *__restrict__ Qg, const bf16_t *__restrict__ Kg, const bf16_t *__restrict__ Vg,
    const bf16_t *__restrict__ Gg, llla_strides sq, llla_strides sk, llla_strides sv, llla_strides sg, int H, int n,
    float scale, const float *__restrict__ Yg, const float *__restrict__ Ug, const float *__restrict__ Sc,
    float *__restrict__ dK, float *__restrict__ dV)
{
    using S = Shape<DD>;
    constexpr int NF = (16 * LIVE + 31) / 32, NB = LIVE, YP = S::YP;
    constexpr int CH = DD / 8;                           // 16-byte chunks per row
    constexpr int TILE = QS * DD;                        // halves
    constexpr int NBUF = DD == 64 ? 2 : 1;               // 50 KB per workgroup
    constexpr int RPT = 64 / CH, NTR = QS / RPT / 4;     // rows and number of a wave's transfers per tile
    enum { TQ, TG, TYH, TYL, TUH, TUL, NTILE };          // u: -u1, both uses subtract it
    __shared__ __align__(16) bf16_t tiles[NBUF][NTILE][TILE];
    __shared__ __align__(16) float rs[NBUF][QS * 8];     // y0, u0, m (log2 units), correction, argmax of the step's rows

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    // A low key block sees the most rows (up to n/32 steps), the last one two steps.  Workgroups are dispatched
    // with blockIdx.x running fastest, so the head is put there: all heads' longest blocks start first and the
    // shortest ones fill the tail, instead of the last head's longest block running alone at the end.
    const int bh = blockIdx.x, b = bh / H, h = bh % H;
    const int j0 = (int)blockIdx.y * (64 * NK), jw = j0 + 16 * NK * wave;       // first key of the workgroup, of the wave
    const char *Qh = reinterpret_cast<const char *>(Qg + b * sq.batch + h * sq.head);
    const char *Gh = reinterpret_cast<const char *>(Gg + b * sg.batch + h * sg.head);
    const char *Yh = reinterpret_cast<const char *>(Yg + (size_t)bh * n * YP), *Uh = reinterpret_cast<const char *>(Ug + (size_t)bh * n * YP);
    const float *Sh = Sc + (size_t)bh * n * 8;
    const float cscale = scale * LOG2E;

    bf16x8 kf[NK][NF], vf[NK][NF];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int jkc = min(jw + 16 * k + nn, n - 1);
        const bf16_t *krow = Kg + b * sk.batch + h * sk.head + (int64_t)jkc * sk.seq;
        const bf16_t *vrow = Vg + b * sv.batch + h * sv.head + (int64_t)jkc * sv.seq;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            kf[k][f] = *reinterpret_cast<const bf16x8 *>(krow + 32 * f + 8 * g);
            vf[k][f] = *reinterpret_cast<const bf16x8 *>(vrow + 32 * f + 8 * g);
        }
    }
    f32x4 dv[NK][NB], dk[NK][NB];
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int J = 0; J < NB; ++J) dv[k][J] = dk[k][J] = f32x4{0.f, 0.f, 0.f, 0.f};
    int row_addr[NF], tr_addr[NB];                       // operand reads: rows (+ 16 s DD), columns
#pragma unroll
    for (int f = 0; f < NF; ++f) row_addr[f] = nn * DD + (((g + 4 * f) ^ row_swizzle<DD>(nn)) * 8);
    {
        const int r = 4 * g + (nn >> 2);
#pragma unroll
        for (int J = 0; J < NB; ++J) tr_addr[J] = r * DD + (((2 * J + ((nn & 3) >> 1)) ^ row_swizzle<DD>(r)) * 8) + (nn & 1) * 4;
    }

    // Transfer t of wave w fills rows RPT (NTR w + t) ...  Steps inside the sequence take a scalar base and offsets that never change (no
    // address arithmetic on the vector ALU); in the last one rows past the end repeat the last row (their coefficients are zero).
    unsigned q_off[NTR], g_off[NTR], y_off[NTR];
    const bool small_pitch = sq.seq < (int64_t(1) << 24) && sg.seq < (int64_t(1) << 24);       // the offsets fit 32 bits
    const int n_whole = small_pitch ? n : 0;
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
        const int r = RPT * (NTR * wave + t) + lane / CH, col = ((lane % CH) ^ row_swizzle<DD>(r)) * 16;
        q_off[t] = 2u * (unsigned)(r * (int)sq.seq) + col;
        g_off[t] = 2u * (unsigned)(r * (int)sg.seq) + col;
        y_off[t] = (unsigned)(r * (YP * 4) + col);
    }
    const unsigned tiles_lds = lds_offset(&tiles[0][0][0]), rs_lds = lds_offset(&rs[0][0]);
    auto issue = [&](int buf, int it0) {
        const bool whole = it0 + QS <= n_whole;
        const char *qb = Qh + (int64_t)it0 * sq.seq * 2, *gb = Gh + (int64_t)it0 * sg.seq * 2;
        const char *yb = Yh + (int64_t)it0 * (YP * 4), *ub = Uh + (int64_t)it0 * (YP * 4);
#pragma unroll
        for (int t = 0; t < NTR; ++t) {
            const int r0 = RPT * (NTR * wave + t);
            const unsigned dst = tiles_lds + 2u * (unsigned)(buf * NTILE * TILE + r0 * DD);
            if (whole) {
                dma16_base_off(qb, q_off[t], dst + 2u * (TQ * TILE));
                dma16_base_off(gb, g_off[t], dst + 2u * (TG * TILE));
                dma16_base_off(yb, y_off[t], dst + 2u * (TYH * TILE));
                dma16_base_off(yb + 2 * DD, y_off[t], dst + 2u * (TYL * TILE));
                dma16_base_off(ub, y_off[t], dst + 2u * (TUH * TILE));
                dma16_base_off(ub + 2 * DD, y_off[t], dst + 2u * (TUL * TILE));
            } else {
                const int r = r0 + lane / CH;
                const int64_t i = min(it0 + r, n - 1);
                const int col = ((lane % CH) ^ row_swizzle<DD>(r)) * 16;
                const char *y = Yh + i * (YP * 4) + col, *u = Uh + i * (YP * 4) + col;
                dma16(Qh + i * sq.seq * 2 + col, &tiles[buf][TQ][r0 * DD]);
                dma16(Gh + i * sg.seq * 2 + col, &tiles[buf][TG][r0 * DD]);
                dma16(y, &tiles[buf][TYH][r0 * DD]);
                dma16(y + 2 * DD, &tiles[buf][TYL][r0 * DD]);
                dma16(u, &tiles[buf][TUH][r0 * DD]);
                dma16(u + 2 * DD, &tiles[buf][TUL][r0 * DD]);
            }
        }
        if (wave == 0) {
            if (whole) dma16_base_off(Sh + (size_t)it0 * 8, 16u * lane, rs_lds + 4u * (unsigned)(buf * QS * 8));
            else dma16(Sh + (size_t)min(it0 + (lane >> 1), n - 1) * 8 + 4 * (lane & 1), rs[buf]);
        }
    };

    // one step (buf: with two key blocks a run-time value, since two copies of the loop spill; else a constant, so that the operand
    // addresses are registers plus immediates)
    auto step = [&](auto buf, int it0) {
        if (NBUF == 1) {
            __syncthreads();                             // the previous step's tiles are consumed
            issue(0, it0);
        }
        dma_wait();
        __syncthreads();                                 // this step has arrived (NBUF 2: and the previous one is consumed)
        const bool more = NBUF == 2 && it0 + QS < n;
        if (NK > 1 && more) issue(buf ^ 1, it0 + QS);
        if (NK > 1 && it0 + QS <= jw) return;            // every row of the step lies before the wave's first key
        const bf16_t *qt = tiles[buf][TQ], *gt = tiles[buf][TG], *yh = tiles[buf][TYH], *yl = tiles[buf][TYL];
        const bf16_t *uh = tiles[buf][TUH], *ul = tiles[buf][TUL];

        // ---- coefficients: lane (g, nn) holds the pairs (query it0 + 16s + 4g + r, key jw + 16k + nn) ----------
        float sv_[NK][8], ev_[NK][8], pv_[NK][8];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            f32x4 st[NK], at[NK], et[NK];
            float m[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const f32x4 s4 = *reinterpret_cast<const f32x4 *>(&rs[buf][(16 * s + 4 * g + r) * 8]);
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    st[k][r] = 0.f;
                    at[k][r] = s4[0];
                    et[k][r] = -s4[1];
                }
                m[r] = s4[2];
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int ar = row_addr[f] + 16 * s * DD;
                const bf16x8 qf = *reinterpret_cast<const bf16x8 *>(qt + ar);
                const bf16x8 gf = *reinterpret_cast<const bf16x8 *>(gt + ar);
                const bf16x8 yhf = *reinterpret_cast<const bf16x8 *>(yh + ar);
                const bf16x8 ylf = *reinterpret_cast<const bf16x8 *>(yl + ar);
                const bf16x8 uhf = *reinterpret_cast<const bf16x8 *>(uh + ar);
                const bf16x8 ulf = *reinterpret_cast<const bf16x8 *>(ul + ar);
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    st[k] = mfma_bf16(qf, kf[k][f], st[k]);
                    at[k] = mfma_bf16(ylf, kf[k][f], at[k]);
                    et[k] = mfma_bf16(ulf, kf[k][f], et[k]);
                    at[k] = mfma_bf16(yhf, kf[k][f], at[k]);
                    et[k] = mfma_bf16(uhf, kf[k][f], et[k]);
                    et[k] = mfma_bf16(gf, vf[k][f], et[k]);          // gamma - u0 - u1.k
                }
            }
            // (with one key block behind the first products, so that the reads above do not wait for its scalar work: few heads 3 % faster;
            // with two 3 % slower)
            if (NK == 1 && s == 0 && more) issue(buf ^ 1, it0 + QS);
#pragma unroll
            for (int k = 0; k < NK; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float w = __builtin_amdgcn_exp2f(fmaf(st[k][r], cscale, -m[r]));
                    sv_[k][4 * s + r] = w * at[k][r];
                    ev_[k][4 * s + r] = w * et[k][r];
                    pv_[k][4 * s + r] = sv_[k][4 * s + r] * et[k][r];
                }
        }
        // the correction of the maximum, where a row of the step attains it at one of the wave's keys (lane l looks at row l % 32)
        if (__any((unsigned)(__float_as_int(rs[buf][(lane & 31) * 8 + 4]) - jw) < 16u * NK)) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float *row = &rs[buf][(16 * (t >> 2) + 4 * g + (t & 3)) * 8];
#pragma unroll
                for (int k = 0; k < NK; ++k) pv_[k][t] += jw + 16 * k + nn == __float_as_int(row[4]) ? row[3] : 0.f;
            }
        }
        if (it0 < jw + 16 * NK - 1 || it0 + QS > n) {
#pragma unroll
            for (int k = 0; k < NK; ++k)
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int i = it0 + 16 * (t >> 2) + 4 * g + (t & 3);
                    const bool valid = jw + 16 * k + nn <= i && i < n;
                    sv_[k][t] = valid ? sv_[k][t] : 0.f;
                    ev_[k][t] = valid ? ev_[k][t] : 0.f;
                    pv_[k][t] = valid ? pv_[k][t] : 0.f;
                }
        }

#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
            for (int t = 0; t < 8; ++t) pv_[k][t] *= scale;

        // ---- accumulate over the step's 32 queries ----------------------------------------------------------------
        if constexpr (NK == 1) {
            bf16x8 s_hi, s_lo, e_hi, e_lo, p_hi, p_lo;
            split_bf16(sv_[0], s_hi, s_lo);
            split_bf16(ev_[0], e_hi, e_lo);
            split_bf16(pv_[0], p_hi, p_lo);
#pragma unroll
            for (int J = 0; J < NB; ++J) {
                f32x4 &dvj = dv[0][J], &dkj = dk[0][J];
                const bf16x8 gT = tr_frag(gt, tr_addr[J], DD);
                dvj = mfma_bf16(s_lo, gT, dvj);
                const bf16x8 yhT = tr_frag(yh, tr_addr[J], DD), ylT = tr_frag(yl, tr_addr[J], DD);
                dkj = mfma_bf16(e_lo, yhT, dkj);
                dvj = mfma_bf16(s_hi, gT, dvj);
                dkj = mfma_bf16(e_hi, ylT, dkj);
                dkj = mfma_bf16(e_hi, yhT, dkj);
                const bf16x8 uhT = tr_frag(uh, tr_addr[J], DD), ulT = tr_frag(ul, tr_addr[J], DD);
                dkj = mfma_bf16(s_lo, uhT, dkj);
                dkj = mfma_bf16(s_hi, ulT, dkj);
                dkj = mfma_bf16(s_hi, uhT, dkj);
                const bf16x8 qT = tr_frag(qt, tr_addr[J], DD);
                dkj = mfma_bf16(p_lo, qT, dkj);
                dkj = mfma_bf16(p_hi, qT, dkj);
            }
        } else {
            // one coefficient after the other: the next one is split beside the products of this one
            bf16x8 c_hi[NK], c_lo[NK];
#pragma unroll
            for (int k = 0; k < NK; ++k) split_bf16(sv_[k], c_hi[k], c_lo[k]);
#pragma unroll
            for (int J = 0; J < NB; ++J) {
                const bf16x8 gT = tr_frag(gt, tr_addr[J], DD), uhT = tr_frag(uh, tr_addr[J], DD), ulT = tr_frag(ul, tr_addr[J], DD);
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    dv[k][J] = mfma_bf16(c_lo[k], gT, dv[k][J]);
                    dk[k][J] = mfma_bf16(c_lo[k], uhT, dk[k][J]);
                }
#pragma unroll
                for (int k = 0; k < NK; ++k) {
                    dv[k][J] = mfma_bf16(c_hi[k], gT, dv[k][J]);
                    dk[k][J] = mfma_bf16(c_hi[k], ulT, dk[k][J]);
                }
#pragma unroll
                for (int k = 0; k < NK; ++k) dk[k][J] = mfma_bf16(c_hi[k], uhT, dk[k][J]);
            }
#pragma unroll
            for (int k = 0; k < NK; ++k) split_bf16(ev_[k], c_hi[k], c_lo[k]);
#pragma unroll
            for (int J = 0; J < NB; ++J) {
                const bf16x8 yhT = tr_frag(yh, tr_addr[J], DD), ylT = tr_frag(yl, tr_addr[J], DD);
#pragma unroll
                for (int k = 0; k < NK; ++k) dk[k][J] = mfma_bf16(c_lo[k], yhT, dk[k][J]);
#pragma unroll
                for (int k = 0; k < NK; ++k) dk[k][J] = mfma_bf16(c_hi[k], ylT, dk[k][J]);
#pragma unroll
                for (int k = 0; k < NK; ++k) dk[k][J] = mfma_bf16(c_hi[k], yhT, dk[k][J]);
            }
#pragma unroll
            for (int k = 0; k < NK; ++k) split_bf16(pv_[k], c_hi[k], c_lo[k]);
#pragma unroll
            for (int J = 0; J < NB; ++J) {
                const bf16x8 qT = tr_frag(qt, tr_addr[J], DD);
#pragma unroll
                for (int k = 0; k < NK; ++k) dk[k][J] = mfma_bf16(c_lo[k], qT, dk[k][J]);
#pragma unroll
                for (int k = 0; k < NK; ++k) dk[k][J] = mfma_bf16(c_hi[k], qT, dk[k][J]);
            }
        }
    };
    if (NBUF == 2) issue(0, j0);
    if constexpr (NK == 1) {
        for (int it0 = j0; it0 < n; it0 += NBUF * QS) {
            step(std::integral_constant<int, 0>{}, it0);
            if (NBUF == 2 && it0 + QS < n) step(std::integral_constant<int, NBUF - 1>{}, it0 + QS);
        }
    } else {
        for (int it0 = j0, c = 0; it0 < n; it0 += QS, ++c) step(c & 1, it0);
    }

    // dv[k][J], dk[k][J]: lane (g, nn) reg r = gradient of key jw + 16k + 4g + r, feature 16J + nn
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int key = jw + 16 * k + 4 * g + r;
            if (key < n) {
                const size_t off = ((size_t)bh * n + key) * (16 * LIVE) + nn;
#pragma unroll
                for (int J = 0; J < NB; ++J) {
                    dK[off + 16 * J] = dk[k][J][r];
                    dV[off + 16 * J] = dv[k][J][r];
                }
            }
        }
}


// ---- row sweeps ---------------------------------------------------------------------------------------------
// The mirror image of the key sweep: a wave owns 16 query rows (their fragments stay in registers) and walks over
// the keys in steps of 32; the coefficient tiles come out as [key][query] (lane (g, nn): keys 4g..4g+3, query nn),
// which is the A operand of a product that contracts over keys, with the K tile read transposed as B.
//   MODE 0 (before the solve): c_ij = w_ij gamma_ij;  r1_i = sum_j c_ij k_j, r0_i = sum_j c_ij, and the first key that
//                              attains the row maximum (the logits are produced exactly as in the row-maximum sweep);
//   MODE 1 (after it):         dL/dlambda_i = -u1_i.y1_i, c_ij = p^_ij;  dQ_i = u1_i + scale sum_j c_ij k_j, and what the key
//                              sweep reads: the row scalars (y0, u0, m in log2 units, correction, argmax) and, in the place of the
//                              fp32 rows, y1 and -u1 as bf16 hi (DD halves) and lo.
// Rows [first_row, n).  The first 2d rows of a sequence, a launch of their own, have the worst conditioned systems: u_i and the
// coefficients are large and cancel (dQ_0 is exactly 0 as the difference of two large terms), and two terms are not enough there.  They
// take TERMS = 3: y1, u1 and the coefficients in three bf16, i.e. fp32 accuracy, since q, k, v and dO are bf16 already.  (In fp32 on the
// vector ALU the two modes took 23 + 29 us at 16 heads x 1000 rows, 25 + 33 at 64 x 4096; the calls went from 259 to 223 and from 4420 to 4342, errors of those
// rows 0.7-1 times the former.)
// The K and V tiles come by DMA into NST stages as in the key sweep, one barrier per block.  A block is so short (16 and 32 MFMAs) that the
// transfers' latency shows where they are one block ahead: MODE 1 keeps three on their way (64 heads x 4096: through registers and two
// barriers 493 us, one block ahead 480, three 434).  MODE 0, bound by its vector work, has two stages and the loop unrolled
// over them (341 -> 307; three blocks ahead 319), and NQ = 2 blocks of 16 queries per wave from TWO_QUERY_BLOCKS_FROM workgroups of 128
// rows on (328 -> 310; 64 x 2048 102 -> 106, 96 x 1000 47 -> 55).
template <int DD, int MODE>
struct RowTiles {
    static constexpr int NST = MODE == 0 ? 2 : 4;        // blocks in LDS: the one in use and NST - 1 on their way
    bf16_t kt[NST][KB * DD], vt[NST][KB * DD];
};

// (row block yblk of ny, from first_row on)
template <int DD, int MODE, int NQ, int TERMS, int LIVE>
__device__ __forceinline__ void bwd_rows_body(
    RowTiles<DD, MODE> &tiles, const bf16_t *__restrict__ Qg, const bf16_t *__restrict__ Kg, const bf16_t *__restrict__ Vg,
    const bf16_t *__restrict__ Gg, llla_strides sq, llla_strides sk, llla_strides sv, llla_strides sg, int H, int n,
    int first_row, int yblk, int ny, int mpitch, float scale, float lambda, const float *__restrict__ LamRows, const float *__restrict__ Mg,
    float *Yg, float *Ug, float *__restrict__ Rv, float *__restrict__ Sc, float *__restrict__ dQ, float *__restrict__ dLam)
{
    using S = Shape<DD>;
    constexpr int NF = (16 * LIVE + 31) / 32, NB = LIVE, YP = S::YP;
    constexpr int CH = DD / 8, TILE = KB * DD, RPT = 64 / CH, NTR = KB / RPT / 4;     // as in the key sweep
    constexpr int NST = RowTiles<DD, MODE>::NST;
    auto &kt = tiles.kt;
    auto &vt = tiles.vt;

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    // head on blockIdx.x (dispatched fastest), row block on y, longest rows first: see bwd_keys_mfma_kernel
    const int bh = blockIdx.x, b = bh / H, h = bh % H;
    const int i0 = first_row + (ny - 1 - yblk) * (64 * NQ), iw = i0 + 16 * NQ * wave;   // first row of the workgroup, of the wave
    const char *Kh = reinterpret_cast<const char *>(Kg + b * sk.batch + h * sk.head);
    const char *Vh = reinterpret_cast<const char *>(Vg + b * sv.batch + h * sv.head);
    // MODE 0 compares raw products with the maximum, so the sign of the scale goes into the query operand
    const float cscale = MODE == 0 ? fabsf(scale * LOG2E) : scale * LOG2E;
    const unsigned flip = MODE == 0 && scale < 0.f ? 0x80008000u : 0u;

    bf16x8 qf[NQ][NF], gf[NQ][NF], yhf[NQ][NF], ylf[NQ][NF], uhf[NQ][NF], ulf[NQ][NF], y3f[NQ][NF], u3f[NQ][NF];
    float mrow[NQ], near[NQ], y0[NQ], u0[NQ], corr[NQ];
    int jstar[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int iq = iw + 16 * q + nn, iqc = min(iq, n - 1);
        const size_t row = (size_t)bh * n + iqc;
        const bf16_t *qrow = Qg + b * sq.batch + h * sq.head + (int64_t)iqc * sq.seq;
        const bf16_t *grow = Gg + b * sg.batch + h * sg.head + (int64_t)iqc * sg.seq;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            u32x4 u = *reinterpret_cast<const u32x4 *>(qrow + 32 * f + 8 * g);
            if (MODE == 0) u ^= flip;
            qf[q][f] = __builtin_bit_cast(bf16x8, u);
            gf[q][f] = *reinterpret_cast<const bf16x8 *>(grow + 32 * f + 8 * g);
        }
        mrow[q] = Mg[(size_t)bh * mpitch + iqc];                          // log2 units
        // a product from here on can be the row's maximum (a zero scale: every one)
        near[q] = (mrow[q] - (1e-4f * fabsf(mrow[q]) + 1e-30f)) / cscale;
        y0[q] = u0[q] = corr[q] = 0.f;
        jstar[q] = 0;
        if (MODE == 1) {
            const float *yr = Yg + row * YP, *ur = Ug + row * YP;
            y0[q] = yr[DD];
            u0[q] = ur[DD];
            jstar[q] = __float_as_int(Rv[row * YP + DD + 1]);
            float dl = 0.f;
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                float yv[8], uv[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    yv[t] = yr[32 * f + 8 * g + t];
                    const float u = ur[32 * f + 8 * g + t];
                    dl = fmaf(-u, yv[t], dl);
                    uv[t] = -u;
                }
                if constexpr (TERMS == 3) {
                    split3_bf16(yv, yhf[q][f], ylf[q][f], y3f[q][f]);
                    split3_bf16(uv, uhf[q][f], ulf[q][f], u3f[q][f]);
                } else {
                    split_bf16(yv, yhf[q][f], ylf[q][f]);
                    split_bf16(uv, uhf[q][f], ulf[q][f]);
                }
            }
            dl += __shfl_xor(dl, 16);
            dl += __shfl_xor(dl, 32);
            corr[q] = (LamRows ? LamRows[row] : lambda) * dl;
            if (g == 0 && iq < n) {
                float *sc = Sc + row * 8;
                sc[0] = y0[q]; sc[1] = u0[q]; sc[2] = mrow[q]; sc[3] = corr[q]; sc[4] = __int_as_float(jstar[q]);
                if (dLam) dLam[row] = dl;
            }
        }
    }
    f32x4 acc[NQ][NB];
    float csum[NQ], best[NQ];
    int arg[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int J = 0; J < NB; ++J) acc[q][J] = f32x4{0.f, 0.f, 0.f, 0.f};
        csum[q] = 0.f;
        best[q] = -INFINITY;
        arg[q] = 0;
    }
    int row_addr[NF], tr_addr[NB];                       // operand reads: rows (+ 16 s DD), columns
#pragma unroll
    for (int f = 0; f < NF; ++f) row_addr[f] = nn * DD + (((g + 4 * f) ^ row_swizzle<DD>(nn)) * 8);
    {
        const int r = 4 * g + (nn >> 2);
#pragma unroll
        for (int J = 0; J < NB; ++J) tr_addr[J] = r * DD + (((2 * J + ((nn & 3) >> 1)) ^ row_swizzle<DD>(r)) * 8) + (nn & 1) * 4;
    }
    // as in the key sweep; keys past the end repeat the last one: no row that is stored sees them
    unsigned k_off[NTR], v_off[NTR];
    const int n_whole = sk.seq < (int64_t(1) << 24) && sv.seq < (int64_t(1) << 24) ? n : 0;
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
        const int r = RPT * (NTR * wave + t) + lane / CH, col = ((lane % CH) ^ row_swizzle<DD>(r)) * 16;
        k_off[t] = 2u * (unsigned)(r * (int)sk.seq) + col;
        v_off[t] = 2u * (unsigned)(r * (int)sv.seq) + col;
    }
    const unsigned kt_lds = lds_offset(&kt[0][0]), vt_lds = lds_offset(&vt[0][0]);
    auto issue = [&](int buf, int c) {
        const bool whole = c * KB + KB <= n_whole;
        const char *kb = Kh + (int64_t)(c * KB) * sk.seq * 2, *vb = Vh + (int64_t)(c * KB) * sv.seq * 2;
#pragma unroll
        for (int t = 0; t < NTR; ++t) {
            const int r0 = RPT * (NTR * wave + t);
            if (whole) {
                dma16_base_off(kb, k_off[t], kt_lds + 2u * (unsigned)(buf * TILE + r0 * DD));
                dma16_base_off(vb, v_off[t], vt_lds + 2u * (unsigned)(buf * TILE + r0 * DD));
            } else {
                const int r = r0 + lane / CH;
                const int64_t j = min(c * KB + r, n - 1);
                const int col = ((lane % CH) ^ row_swizzle<DD>(r)) * 16;
                dma16(Kh + j * sk.seq * 2 + col, &kt[buf][r0 * DD]);
                dma16(Vh + j * sv.seq * 2 + col, &vt[buf][r0 * DD]);
            }
        }
    };

    const int nblk = min(i0 + 64 * NQ - 1, n - 1) / KB + 1;
    auto step = [&](auto buf, int c) {
        dma_wait_but<2 * NTR * (NST - 2)>();
        __syncthreads();                                 // this block has arrived, the previous one is consumed
        const int next = min(c + NST - 1, nblk - 1);     // (past the end: the last block again, so that the count above holds)
        if (MODE == 1) issue((buf + NST - 1) & (NST - 1), next);
        if (c * KB > iw + 16 * NQ - 1) {                 // every key of the block lies behind the wave's last row
            if (MODE == 0) issue((buf + NST - 1) & (NST - 1), next);
            return;
        }
        float cv[NQ][8], lg[NQ][8];                      // coefficients; MODE 0: raw products
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            f32x4 st[NQ], et[NQ], at[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                st[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                et[q] = f32x4{-u0[q], -u0[q], -u0[q], -u0[q]};            // MODE 0: y0 = u0 = 0
                at[q] = f32x4{y0[q], y0[q], y0[q], y0[q]};
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const bf16x8 kfr = *reinterpret_cast<const bf16x8 *>(&kt[buf][row_addr[f] + 16 * s * DD]);
                const bf16x8 vfr = *reinterpret_cast<const bf16x8 *>(&vt[buf][row_addr[f] + 16 * s * DD]);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    st[q] = mfma_bf16(kfr, qf[q][f], st[q]);
                    if (MODE == 1 && TERMS == 3) {
                        at[q] = mfma_bf16(kfr, y3f[q][f], at[q]);
                        et[q] = mfma_bf16(kfr, u3f[q][f], et[q]);
                    }
                    if (MODE == 1) {
                        at[q] = mfma_bf16(kfr, ylf[q][f], at[q]);
                        et[q] = mfma_bf16(kfr, ulf[q][f], et[q]);
                        at[q] = mfma_bf16(kfr, yhf[q][f], at[q]);
                        et[q] = mfma_bf16(kfr, uhf[q][f], et[q]);
                    }
                    et[q] = mfma_bf16(vfr, gf[q][f], et[q]);
                }
            }
            // (MODE 0: behind the first products, so that the reads above do not wait for its scalar work: few heads 8 % faster; MODE 1 7 % slower)
            if (MODE == 0 && s == 0) issue((buf + NST - 1) & (NST - 1), next);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float w = __builtin_amdgcn_exp2f(fmaf(st[q][r], cscale, -mrow[q]));
                    cv[q][4 * s + r] = MODE == 0 ? w * et[q][r] : w * at[q][r] * et[q][r];
                    lg[q][4 * s + r] = st[q][r];
                }
        }
        // lane (g, nn): cv[q][4s + r] belongs to key 32c + 16s + 4g + r and query iw + 16q + nn
        const int j0 = c * KB + 4 * g;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (MODE == 0) {
                // the first key at the row maximum: only a block that comes near the maximum is looked at
                float top = fmaxf(lg[q][0], lg[q][1]);
#pragma unroll
                for (int t = 2; t < 8; t += 2) top = fmaxf(fmaxf(top, lg[q][t]), lg[q][t + 1]);
                if (__any(!(top < near[q]))) {
                    const int iq = iw + 16 * q + nn;
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int j = j0 + 16 * (t >> 2) + (t & 3);
                        const float l = lg[q][t] * cscale;
                        if (j <= iq && iq < n && l > best[q]) {
                            best[q] = l;
                            arg[q] = j;
                        }
                    }
                }
            } else if (__any((unsigned)(jstar[q] - c * KB) < (unsigned)KB)) {
#pragma unroll
                for (int t = 0; t < 8; ++t) cv[q][t] += j0 + 16 * (t >> 2) + (t & 3) == jstar[q] ? corr[q] : 0.f;
            }
        }
        if (c * KB + KB - 1 > iw) {                      // only the blocks that reach past the wave's first query need the causal mask
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 8; ++t) cv[q][t] = j0 + 16 * (t >> 2) + (t & 3) <= iw + 16 * q + nn ? cv[q][t] : 0.f;
        }
        bf16x8 c_hi[NQ], c_lo[NQ], c_3[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (MODE == 0) {
#pragma unroll
                for (int t = 0; t < 8; ++t) csum[q] += cv[q][t];
            }
            if constexpr (TERMS == 3) split3_bf16(cv[q], c_hi[q], c_lo[q], c_3[q]);
            else split_bf16(cv[q], c_hi[q], c_lo[q]);
        }
#pragma unroll
        for (int J = 0; J < NB; ++J) {
            const bf16x8 kT = tr_frag(kt[buf], tr_addr[J], DD);
            if constexpr (TERMS == 3) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) acc[q][J] = mfma_bf16(c_3[q], kT, acc[q][J]);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q][J] = mfma_bf16(c_lo[q], kT, acc[q][J]);
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q][J] = mfma_bf16(c_hi[q], kT, acc[q][J]);
        }
    };
#pragma unroll
    for (int c = 0; c < NST - 1; ++c) issue(c, min(c, nblk - 1));
    if constexpr (MODE == 0) {
        for (int c = 0; c < nblk; c += NST) {
            step(std::integral_constant<int, 0>{}, c);
            if (c + 1 < nblk) step(std::integral_constant<int, 1>{}, c + 1);
        }
    } else {
        for (int c = 0; c < nblk; ++c) step(c & (NST - 1), c);
    }
    dma_wait();                                          // no transfer is left when the workgroup's LDS goes to the next one

#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int iq = iw + 16 * q + nn;
        const size_t row = (size_t)bh * n + min(iq, n - 1);
        if (MODE == 0) {
            // lanes (g, nn), g = 0..3, hold query nn's partial sums and maxima over disjoint keys
            csum[q] += __shfl_xor(csum[q], 16);
            csum[q] += __shfl_xor(csum[q], 32);
#pragma unroll
            for (int sft = 16; sft <= 32; sft <<= 1) {
                const float ob = __shfl_xor(best[q], sft);
                const int oa = __shfl_xor(arg[q], sft);
                const bool take = (ob > best[q]) || (ob == best[q] && oa < arg[q]);
                best[q] = take ? ob : best[q];
                arg[q] = take ? oa : arg[q];
            }
            if (g == 0 && iq < n) {
                Rv[row * YP + DD] = csum[q];
                Rv[row * YP + DD + 1] = __int_as_float(arg[q]);
            }
        }
        // acc[q][J]: lane (g, nn) reg r = sum for query iw + 16 q + 4g + r, feature 16J + nn
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = iw + 16 * q + 4 * g + r;
            if (i < n) {
                const size_t ro = (size_t)bh * n + i;
#pragma unroll
                for (int J = 0; J < NB; ++J) {
                    if (MODE == 0) Rv[ro * YP + 16 * J + nn] = acc[q][J][r];
                    else dQ[ro * (16 * LIVE) + 16 * J + nn] = fmaf(scale, acc[q][J][r], Ug[ro * YP + 16 * J + nn]);
                }
            }
        }
    }
    if (MODE == 1) {
        __syncthreads();                                 // the fp32 rows have been read for the last time
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int iq = iw + 16 * q + nn;
            const size_t row = (size_t)bh * n + iq;
            if (iq < n) {
                bf16_t *yr = reinterpret_cast<bf16_t *>(Yg + row * YP), *ur = reinterpret_cast<bf16_t *>(Ug + row * YP);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    *reinterpret_cast<bf16x8 *>(yr + 32 * f + 8 * g) = yhf[q][f];
                    *reinterpret_cast<bf16x8 *>(yr + DD + 32 * f + 8 * g) = ylf[q][f];
                    *reinterpret_cast<bf16x8 *>(ur + 32 * f + 8 * g) = uhf[q][f];
                    *reinterpret_cast<bf16x8 *>(ur + DD + 32 * f + 8 * g) = ulf[q][f];
                }
            }
        }
    }
}

// TERMS = 0: rows [0, early) with three terms and those behind them with two, in one launch (the last early / 64 row blocks).
template <int DD, int MODE, int NQ, int TERMS, int LIVE = Shape<DD>::NB>
__global__ __launch_bounds__(256, TERMS == 3 ? 1 : 2) void bwd_rows_mfma_kernel(
    const bf16_t *__restrict__ Qg, const bf16_t *__restrict__ Kg, const bf16_t *__restrict__ Vg,
    const bf16_t *__restrict__ Gg, llla_strides sq, llla_strides sk, llla_strides sv, llla_strides sg, int H, int n, int early,
    int first_row, int mpitch, float scale, float lambda, const float *__restrict__ LamRows, const float *__restrict__ Mg,
    float *Yg, float *Ug, float *__restrict__ Rv, float *__restrict__ Sc, float *__restrict__ dQ, float *__restrict__ dLam)
{
    __shared__ __align__(16) RowTiles<DD, MODE> tiles;
    const int yblk = blockIdx.y, ny = gridDim.y;
    if constexpr (TERMS == 0) {
        const int late = ny - early / 64;
        if (yblk < late)
            bwd_rows_body<DD, MODE, NQ, 2, LIVE>(tiles, Qg, Kg, Vg, Gg, sq, sk, sv, sg, H, n, early, yblk, late, mpitch, scale, lambda, LamRows, Mg,
                                                 Yg, Ug, Rv, Sc, dQ, dLam);
        else
            bwd_rows_body<DD, MODE, NQ, 3, LIVE>(tiles, Qg, Kg, Vg, Gg, sq, sk, sv, sg, H, n, 0, yblk - late, ny - late, mpitch, scale, lambda,
                                                 LamRows, Mg, Yg, Ug, Rv, Sc, dQ, dLam);
    } else {
        bwd_rows_body<DD, MODE, NQ, TERMS, LIVE>(tiles, Qg, Kg, Vg, Gg, sq, sk, sv, sg, H, n, first_row, yblk, ny, mpitch, scale, lambda, LamRows, Mg,
                                                 Yg, Ug, Rv, Sc, dQ, dLam);
    }
}

// ---- output sweep of the forward ---------------------------------------------------------------------------------
// O_i = sum_j w_ij (y0_i + k_j . y1_i) v_j for the rows [first_row, n): the row sweeps' loop with other products, 20 MFMAs and some 50
// vector instructions per wave, block of 32 keys and 16 queries at d = 64, which hardly overlap.  What bounded sweep_kernel beyond
// that was the staging through registers with two barriers per block; here the tiles come by DMA one block ahead, one barrier per
// block, and V is read transposed from its natural tile, so no V^T is made either.  us a call: 64 heads x 4096 at d = 64 2822 -> 2771, 96 x 1000
// with statistics 456 -> 438, 16 x 8192 at d = 128 10003 -> 9721.  (Three blocks ahead 2779, 441, 9747; two blocks of 16 queries per
// wave 2758, 443.)
// LIVE < NB (a d = 16 / 32 call on zero-padded copies): features and value columns from 16 LIVE on are zero and left out.
// (us a call: 64 heads x 4096 at d = 32 1422 -> 1378, d = 16 1079 -> 1039, 32 x 300 at d = 32 53.9 -> 50.5.)
// TERMS = 3 (the first rows, whose coefficients cancel to a few digits): y1 and the coefficients in three bf16, as in the sweeps above.
template <int DD, int LIVE, int TERMS>
__device__ __forceinline__ void out_rows_body(
    RowTiles<DD, 0> &tiles, const bf16_t *__restrict__ Qg, const bf16_t *__restrict__ Kg, const bf16_t *__restrict__ Vg, llla_strides sq,
    llla_strides sk, llla_strides sv, int H, int n, int first_row, int yblk, int ny, int mpitch, float cscale, const float *__restrict__ Mg,
    const float *__restrict__ Yg, void *__restrict__ Og, llla_strides so, int out_bf16, int causal)
{
    using S = Shape<DD>;
    constexpr int NF = (16 * LIVE + 31) / 32, NB = LIVE, YP = S::YP;      // feature chunks of 32 and output tiles that are live
    constexpr int CH = DD / 8, TILE = KB * DD, RPT = 64 / CH, NTR = KB / RPT / 4;     // as in the key sweep
    auto &kt = tiles.kt;                                 // two blocks: the one in use and the next, on its way
    auto &vt = tiles.vt;

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    const int bh = blockIdx.x, b = bh / H, h = bh % H;
    const int i0 = first_row + (ny - 1 - yblk) * 64, iw = i0 + 16 * wave;   // first row of the workgroup, of the wave
    const char *Kh = reinterpret_cast<const char *>(Kg + b * sk.batch + h * sk.head);
    const char *Vh = reinterpret_cast<const char *>(Vg + b * sv.batch + h * sv.head);

    const int iq = iw + nn, iqc = min(iq, n - 1), last = causal ? iq : n - 1;         // this lane's query, the last key it sees
    const bf16_t *qrow = Qg + b * sq.batch + h * sq.head + (int64_t)iqc * sq.seq;
    const float *yr = Yg + ((size_t)bh * n + iqc) * YP;
    const float mrow = Mg[(size_t)bh * mpitch + iqc], y0 = yr[DD];                   // (mrow in log2 units)
    bf16x8 qf[NF], yh[NF], ym[NF], yl[NF];
    f32x4 acc[NB];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        qf[f] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * f + 8 * g);
        float yv[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) yv[t] = yr[32 * f + 8 * g + t];
        if constexpr (TERMS == 3) split3_bf16(yv, yh[f], ym[f], yl[f]);
        else split_bf16(yv, yh[f], yl[f]);
    }
#pragma unroll
    for (int J = 0; J < NB; ++J) acc[J] = f32x4{0.f, 0.f, 0.f, 0.f};
    int row_addr[NF], tr_addr[NB];                       // operand reads: rows (+ 16 s DD), columns
#pragma unroll
    for (int f = 0; f < NF; ++f) row_addr[f] = nn * DD + (((g + 4 * f) ^ row_swizzle<DD>(nn)) * 8);
    {
        const int r = 4 * g + (nn >> 2);
#pragma unroll
        for (int J = 0; J < NB; ++J) tr_addr[J] = r * DD + (((2 * J + ((nn & 3) >> 1)) ^ row_swizzle<DD>(r)) * 8) + (nn & 1) * 4;
    }
    // as in the row sweeps of the backward; keys past the end repeat the last one and are masked
    unsigned k_off[NTR], v_off[NTR];
    const int n_whole = sk.seq < (int64_t(1) << 24) && sv.seq < (int64_t(1) << 24) ? n : 0;
#pragma unroll
    for (int t = 0; t < NTR; ++t) {
        const int r = RPT * (NTR * wave + t) + lane / CH, col = ((lane % CH) ^ row_swizzle<DD>(r)) * 16;
        k_off[t] = 2u * (unsigned)(r * (int)sk.seq) + col;
        v_off[t] = 2u * (unsigned)(r * (int)sv.seq) + col;
    }
    const unsigned kt_lds = lds_offset(&kt[0][0]), vt_lds = lds_offset(&vt[0][0]);
    auto issue = [&](int buf, int c) {
        const bool whole = c * KB + KB <= n_whole;
        const char *kb = Kh + (int64_t)(c * KB) * sk.seq * 2, *vb = Vh + (int64_t)(c * KB) * sv.seq * 2;
#pragma unroll
        for (int t = 0; t < NTR; ++t) {
            const int r0 = RPT * (NTR * wave + t);
            if (whole) {
                dma16_base_off(kb, k_off[t], kt_lds + 2u * (unsigned)(buf * TILE + r0 * DD));
                dma16_base_off(vb, v_off[t], vt_lds + 2u * (unsigned)(buf * TILE + r0 * DD));
            } else {
                const int r = r0 + lane / CH;
                const int64_t j = min(c * KB + r, n - 1);
                const int col = ((lane % CH) ^ row_swizzle<DD>(r)) * 16;
                dma16(Kh + j * sk.seq * 2 + col, &kt[buf][r0 * DD]);
                dma16(Vh + j * sv.seq * 2 + col, &vt[buf][r0 * DD]);
            }
        }
    };

    // coefficients of block c: lane (g, nn): cv[4s + r] belongs to key 32c + 16s + 4g + r and query iw + nn.  key_rows(f, s): the operand of
    // key 16s + nn, features 32f + 8g ..
    auto coefficients = [&](auto key_rows, int c, float (&cv)[8]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            f32x4 st = {0.f, 0.f, 0.f, 0.f}, ut = {y0, y0, y0, y0};
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const bf16x8 kfr = key_rows(f, s);
                st = mfma_bf16(kfr, qf[f], st);
                ut = mfma_bf16(kfr, yl[f], ut);
                if constexpr (TERMS == 3) ut = mfma_bf16(kfr, ym[f], ut);
                ut = mfma_bf16(kfr, yh[f], ut);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) cv[4 * s + r] = __builtin_amdgcn_exp2f(fmaf(st[r], cscale, -mrow)) * ut[r];
        }
        if (causal ? c * KB + KB - 1 > iw : c * KB + KB > n) {
            const int j0 = c * KB + 4 * g;
#pragma unroll
            for (int t = 0; t < 8; ++t) cv[t] = j0 + 16 * (t >> 2) + (t & 3) <= last ? cv[t] : 0.f;
        }
    };
    const int nblk = (causal ? min(i0 + 63, n - 1) : n - 1) / KB + 1;
    auto step = [&](auto buf, int c) {
        dma_wait();
        __syncthreads();                                 // this block has arrived, the previous one is consumed
        if (c + 1 < nblk) issue(buf ^ 1, c + 1);
        if (causal && c * KB > iw + 15) return;          // every key of the block lies behind the wave's last row
        float cv[8];
        coefficients([&](int f, int s) { return *reinterpret_cast<const bf16x8 *>(&kt[buf][row_addr[f] + 16 * s * DD]); }, c, cv);
        bf16x8 ch, cm, cl;
        if constexpr (TERMS == 3) split3_bf16(cv, ch, cm, cl);
        else split_bf16(cv, ch, cl);
#pragma unroll
        for (int J = 0; J < NB; ++J) {
            const bf16x8 vT = tr_frag(vt[buf], tr_addr[J], DD);
            acc[J] = mfma_bf16(cl, vT, acc[J]);
            if constexpr (TERMS == 3) acc[J] = mfma_bf16(cm, vT, acc[J]);
            acc[J] = mfma_bf16(ch, vT, acc[J]);
        }
    };
    issue(0, 0);
    for (int c = 0; c < nblk; c += 2) {
        step(std::integral_constant<int, 0>{}, c);
        if (c + 1 < nblk) step(std::integral_constant<int, 1>{}, c + 1);
    }

    // The first rows see no later value, one that is not finite included: where a sum has come out so, the wave's rows are summed again with
    // each key left out of the rows before it instead of multiplied by zero (a scalar branch; no barrier and no LDS in it).
    if constexpr (TERMS == 3) {
        bool odd = false;
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) odd = odd || !(fabsf(acc[J][r]) < INFINITY);
        if (__any(odd)) {
#pragma unroll
            for (int J = 0; J < NB; ++J) acc[J] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int nbw = (causal ? min(iw + 15, n - 1) : n - 1) / KB + 1;
            for (int c = 0; c < nbw; ++c) {
                float cv[8];
                coefficients([&](int f, int s) {
                    const int64_t j = min(c * KB + 16 * s + nn, n - 1);
                    return *reinterpret_cast<const bf16x8 *>(Kh + 2 * (j * sk.seq + 32 * f + 8 * g));
                }, c, cv);
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    for (int gk = 0; gk < 4; ++gk) {     // key j: cv[t] of lanes (gk, query)
                        const int j = c * KB + 16 * (t >> 2) + 4 * gk + (t & 3);
                        const bf16_t *vrow = reinterpret_cast<const bf16_t *>(Vh) + (int64_t)min(j, n - 1) * sv.seq + nn;
                        float w[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) w[r] = __shfl(cv[t], 16 * gk + 4 * g + r);
#pragma unroll
                        for (int J = 0; J < NB; ++J) {
                            const float v = bf16_to_f32(vrow[16 * J]);
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc[J][r] = j <= (causal ? min(iw + 4 * g + r, n - 1) : n - 1) ? fmaf(w[r], v, acc[J][r]) : acc[J][r];
                        }
                    }
            }
        }
    }

    // acc[J]: lane (g, nn) reg r = O[query iw + 4g + r][feature 16J + nn]
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = iw + 4 * g + r;
        if (i < n) {
            const int64_t off = b * so.batch + h * so.head + (int64_t)i * so.seq;
#pragma unroll
            for (int J = 0; J < NB; ++J) {
                if (out_bf16) ((bf16_t *)Og)[off + 16 * J + nn] = f32_to_bf16(acc[J][r]);
                else ((float *)Og)[off + 16 * J + nn] = acc[J][r];
            }
        }
    }
}

// TERMS = 0: as in the row sweeps
template <int DD, int LIVE, int TERMS>
__global__ __launch_bounds__(256, TERMS == 3 ? 1 : 2) void out_rows_kernel(
    const bf16_t *__restrict__ Qg, const bf16_t *__restrict__ Kg, const bf16_t *__restrict__ Vg, llla_strides sq, llla_strides sk,
    llla_strides sv, int H, int n, int early, int first_row, int mpitch, float cscale, const float *__restrict__ Mg, const float *__restrict__ Yg,
    void *__restrict__ Og, llla_strides so, int out_bf16, int causal)
{
    __shared__ __align__(16) RowTiles<DD, 0> tiles;
    const int yblk = blockIdx.y, ny = gridDim.y;
    if constexpr (TERMS == 0) {
        const int late = ny - early / 64;
        if (yblk < late)
            out_rows_body<DD, LIVE, 2>(tiles, Qg, Kg, Vg, sq, sk, sv, H, n, early, yblk, late, mpitch, cscale, Mg, Yg, Og, so, out_bf16, causal);
        else
            out_rows_body<DD, LIVE, 3>(tiles, Qg, Kg, Vg, sq, sk, sv, H, n, 0, yblk - late, ny - late, mpitch, cscale, Mg, Yg, Og, so, out_bf16, causal);
    } else {
        out_rows_body<DD, LIVE, TERMS>(tiles, Qg, Kg, Vg, sq, sk, sv, H, n, first_row, yblk, ny, mpitch, cscale, Mg, Yg, Og, so, out_bf16, causal);
    }
}

constexpr long long TWO_QUERY_BLOCKS_FROM = 1536, TWO_KEY_BLOCKS_FROM = 768;

// The first rows (three terms) and the others in one launch.  A launch of the first rows alone is a few workgroups' latency, 5 to 30 us; the
// price is the registers of three terms for all, i.e. fewer resident workgroups.  us a call, two launches and one: 4 heads x 400 41.2 and
// 35.1, backward 4 x 300 90.8 and 75.1, 96 x 157 with statistics 74.6 and 69.1, backward 8 x 961 at d = 128 435 and 403, 16 x 1000
// 108 and 102, 96 x 1000 (1344 workgroups) 445 and 438, backward 681 and 668, 64 x 2048 (1920) 840 and 829; but 64 x 3000 at d = 16 (2880)
// 583 and 592, backward 64 x 4096 (3968) 4275 and 4333.  At d = 128 the gain is larger and there is no loss up to the same line: 4 x 600 122 and
// 109, backward 242 and 212, 16 x 2048 (448) 1019 and 1007, backward 1439 and 1409, 64 x 2048 (1792) 3836 and 3831, backward 5100 and 5081, 16 x 8192
// (1984) 9525 and 9516.  Backward 64 x 2048 at d = 64 1285 and 1293, at d = 32 727 and 716, at d = 16 590 and 577.
constexpr long long ONE_LAUNCH_UP_TO = 2048;
bool one_launch(int heads, int n, int early)
{
    return early > 0 && early < n && early % 64 == 0 && (long long)heads * ((n - early + 63) / 64) <= ONE_LAUNCH_UP_TO;
}

template <int DD, int MODE, int LIVE = Shape<DD>::NB>
hipError_t launch_rows(const BackwardProblem &p, const BackwardLayout &L, int early)
{
    char *base = static_cast<char *>(p.ws);
    const float *M = reinterpret_cast<const float *>(base + L.fwd + L.m);
    float *Y = reinterpret_cast<float *>(base + L.fwd + L.y);
    float *U = reinterpret_cast<float *>(base + L.u);
    float *R = reinterpret_cast<float *>(base + L.r);
    float *Sc = reinterpret_cast<float *>(base + L.sc);
    auto launch = [&](auto kernel, int rows, int r0, int r1) {        // rows [r0, r1) in blocks of `rows`; r1 a multiple of 64 or n
        hipLaunchKernelGGL(kernel, dim3(p.B * p.H, (r1 - r0 + rows - 1) / rows), dim3(256), 0, p.stream,
                           static_cast<const bf16_t *>(p.Q), static_cast<const bf16_t *>(p.K), static_cast<const bf16_t *>(p.V),
                           static_cast<const bf16_t *>(p.dO), p.sq, p.sk, p.sv, p.sdo, p.H, p.n, early, r0, L.npad, p.scale,
                           p.lambda, p.lambda_rows, M, Y, U, R, Sc, p.dQ, p.dlambda);
        return hipGetLastError();
    };
    if (one_launch(p.B * p.H, p.n, early)) return launch(bwd_rows_mfma_kernel<DD, MODE, 1, 0, LIVE>, 64, 0, p.n);
    const hipError_t e = launch(bwd_rows_mfma_kernel<DD, MODE, 1, 3, LIVE>, 64, 0, early);
    if (e != hipSuccess || early >= p.n) return e;
    if constexpr (DD == 64 && MODE == 0) {
        if ((long long)p.B * p.H * ((p.n - early + 127) / 128) >= TWO_QUERY_BLOCKS_FROM)
            return launch(bwd_rows_mfma_kernel<64, 0, 2, 2, LIVE>, 128, early, p.n);
    }
    return launch(bwd_rows_mfma_kernel<DD, MODE, 1, 2, LIVE>, 64, early, p.n);
}

// 16-feature blocks that can be non-zero (fewer than d / 16 on the zero-padded copies of a d = 16 / 32 call)
int live_blocks(int d, int live_d) { return d == 64 && live_d > 0 ? (live_d + 15) / 16 : d / 16; }

template <int MODE>
hipError_t rows(const BackwardProblem &p, const BackwardLayout &L, int early)
{
    if (p.d != 64) return launch_rows<128, MODE>(p, L, early);
    const int live = live_blocks(p.d, p.live_d);
    return live == 1 ? launch_rows<64, MODE, 1>(p, L, early) : live == 2 ? launch_rows<64, MODE, 2>(p, L, early) : launch_rows<64, MODE>(p, L, early);
}

}  // namespace

// early: the rows at the beginning that take three-term operands, a multiple of 64 or all
hipError_t mfma_backward_r(const BackwardProblem &p, const BackwardLayout &L, int early)
{
    return rows<0>(p, L, early);
}

hipError_t mfma_backward_dq(const BackwardProblem &p, const BackwardLayout &L, int early)
{
    return rows<1>(p, L, early);
}

hipError_t mfma_backward_keys(const BackwardProblem &p, const BackwardLayout &L)
{
    char *base = static_cast<char *>(p.ws);
    const float *Y = reinterpret_cast<const float *>(base + L.fwd + L.y);
    const float *U = reinterpret_cast<const float *>(base + L.u);
    const float *Sc = reinterpret_cast<const float *>(base + L.sc);
    const bf16_t *Q = static_cast<const bf16_t *>(p.Q), *K = static_cast<const bf16_t *>(p.K),
                 *V = static_cast<const bf16_t *>(p.V), *G = static_cast<const bf16_t *>(p.dO);
    auto launch = [&](auto kernel, int keys) {
        hipLaunchKernelGGL(kernel, dim3(p.B * p.H, (p.n + keys - 1) / keys), dim3(256), 0, p.stream, Q, K, V, G, p.sq, p.sk, p.sv, p.sdo,
                           p.H, p.n, p.scale, Y, U, Sc, p.dK, p.dV);
    };
    const bool two = (long long)p.B * p.H * ((p.n + 127) / 128) >= TWO_KEY_BLOCKS_FROM;
    const int live = live_blocks(p.d, p.live_d);
    if (p.d != 64) launch(bwd_keys_mfma_kernel<128, 1>, 64);
    else if (live == 1) two ? launch(bwd_keys_mfma_kernel<64, 2, 1>, 128) : launch(bwd_keys_mfma_kernel<64, 1, 1>, 64);
    else if (live == 2) two ? launch(bwd_keys_mfma_kernel<64, 2, 2>, 128) : launch(bwd_keys_mfma_kernel<64, 1, 2>, 64);
    else two ? launch(bwd_keys_mfma_kernel<64, 2>, 128) : launch(bwd_keys_mfma_kernel<64, 1>, 64);
    return hipGetLastError();
}

// output of a bf16 forward; rows [0, early), whose coefficients cancel, with three-term operands: a multiple of 64, or all
hipError_t mfma_output_rows(const Problem &p, const float *M, int mpitch, const float *Y, int early)
{
    auto launch = [&](auto kernel, int r0, int r1) {
        hipLaunchKernelGGL(kernel, dim3(p.B * p.H, (r1 - r0 + 63) / 64), dim3(256), 0, p.stream, static_cast<const bf16_t *>(p.Q),
                           static_cast<const bf16_t *>(p.K), static_cast<const bf16_t *>(p.V), p.sq, p.sk, p.sv, p.H, p.n, early, r0, mpitch,
                           p.scale * LOG2E, M, Y, p.O, p.so, p.out == LLLA_BF16 ? 1 : 0, p.causal);
    };
    auto sweep = [&](auto dtag, auto livetag) {
        constexpr int DD = decltype(dtag)::value, LIVE = decltype(livetag)::value;
        if (one_launch(p.B * p.H, p.n, early)) {
            stage_mark(p.stream, "output");
            launch(out_rows_kernel<DD, LIVE, 0>, 0, p.n);
            return;
        }
        if (early > 0) {
            stage_mark(p.stream, "output_early_rows");
            launch(out_rows_kernel<DD, LIVE, 3>, 0, early);
        }
        if (early < p.n) {
            stage_mark(p.stream, "output");
            launch(out_rows_kernel<DD, LIVE, 2>, early, p.n);
        }
    };
    using std::integral_constant;
    const int live = live_blocks(p.d, p.live_d);
    if (p.d != 64) sweep(integral_constant<int, 128>{}, integral_constant<int, 8>{});
    else if (live == 1) sweep(integral_constant<int, 64>{}, integral_constant<int, 1>{});
    else if (live == 2) sweep(integral_constant<int, 64>{}, integral_constant<int, 2>{});
    else sweep(integral_constant<int, 64>{}, integral_constant<int, 4>{});
    return hipGetLastError();
}

}  // namespace llla
