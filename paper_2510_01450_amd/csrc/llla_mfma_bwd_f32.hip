// Matrix-core backward pass for fp32 inputs, d = 16, 32, 64 and 128, and the output sweep of the fp32 forward.  The sweeps form every contraction on
// v_mfma_f32_16x16x4_f32 at the head's own dimension, fp32 operands and fp32 accumulation; the second moment comes from operands split into three
// bf16 (24 significant bits) on 16-bit MFMA, at d = 16 / 32 from copies of Q and K in rows of 64 features.
//
// Errors against fp64 times those of the vector kernels of llla_bwd.hip (whose notation is used here), which serve these calls on request; dQ, dK,
// dV and dlambda, geometric means of 48 to 160 heads at two to seven lengths each:
//   unit keys, ridge 10^-2      d = 16 0.83-0.98   d = 32 0.78-0.88   d = 128 0.66-0.69
//   normal keys, 10^-2 and 10^-3       0.76-1.06          0.73-0.98           0.71-0.78
//   normal keys, 10^-4                 0.80-1.22          0.74-1.10           0.65-0.78     (|k|^2 / ridge 10^5 and more)
//   normal keys times 10, 10^-2        0.97-1.14          0.86-1.13           0.70-0.91     (10^5 to 10^6: dlambda has one digit on either)
//   normal keys plus 3, 10^-2          0.65-0.83          0.56-0.66           0.35-0.38
// Large logits, dK at d = 128 (normal keys, ridge 0.05, 40 to 300 rows, logits of standard deviation 8 / 16 / 32 / 64): 0.66-0.96 / 1.0-1.2 / 1.3-1.4 / 1.6-1.9;
// where moments and sweeps sum the logits in different orders 1.8-3.3 / 3.1-4.1 / 4.5-5.0 / 5.9-7.4.
// (d = 16: six, eight or nine partial products, pivots dropped or raised, a Newton step on their roots, r from final weights or from fused
// multiply-adds make no difference; fp32 MFMA for the second moment 1.1 times more.)
//
//   r sweep   r_i = sum_j w_ij gamma_ij [1; k_j], the row maximum m_i and the first key that attains it;
//   moments   the forward's fp32 moments kernel with m_i given and a second right-hand side in its solve: y_i and u_i;
//   dQ sweep  p^_ij, dQ_i, dlambda_i and the scalars of row i that the key sweep reads;
//   key sweep dK_j, dV_j.
//
// What bounds it: the sweeps the fp32 matrix rate (1/16 of the 16-bit one; a tile of 16 queries x 16 keys costs 48 + 80 + 128 MFMAs (d = 64) of
// 32 cycles in the three of them), the moments see llla_mfma_fwd_f32.hip.  The vector kernels spend d^2 multiply-adds per pair on
// the vector ALU, out of LDS, and eliminate a (d+1)^2 system with one barrier per pivot.  16 heads x 1024 rows at d = 64: 2811 us on the
// vector kernels, 494 here; 2 x 128: 207 and 82; other dimensions beside takes_backward_f32 and in llla_mfma_fwd_f32_128.hip.
//
// The sweeps (and the output sweep of the fp32 forward, a fourth) share one shape: 32 rows per workgroup, four waves = 2 groups of 16 rows x 2 halves of every 32-row step
// of the other side, the halves' sums added through LDS at the end.  (64 rows per workgroup without the split leave a
// 1024-row head with 16 workgroups whose longest is twice the mean; with it and balanced_block the r, dQ and key sweeps of 16 heads x
// 1024 rows at d = 64 take 55, 64 and 110 us, in plain longest-first order 62, 79 and 131; the output sweep 53, before the split 64.)  Tiles arrive by DMA one step ahead, two buffers, one
// barrier per step; 16-byte chunks are XOR-swizzled with the row, so that rows are read 16 bytes per lane (operand with the
// features as contraction index) and columns 4 bytes per lane (operand with the rows as contraction index) from one copy.
#include "llla_mfma_common.hpp"

namespace llla {
namespace {

using namespace mfma;

constexpr int RT = 32;                 // rows per workgroup and rows per step
constexpr float LAZY_BITS = 64.f;      // as in the forward: the reference exponent moves when a tile exceeds it by more

// position of the scalar behind a y, u or r row, and the pitch of the rows: those of the moments kernel, which at d = 16 / 32 runs on
// copies padded to 64 features
template <int DD>
constexpr int SP = DD < 64 ? 64 : DD;

// where 16-byte chunk c of tile row r sits: c ^ swz(r)
template <int DD>
__device__ inline int swz(int r) { return DD >= 32 ? r & 7 : (r >> 1) & 3; }

// 32 rows of DD floats -> LDS, chunks swizzled; rows past `last` repeat it
template <int DD>
__device__ inline void dma_tile(const float *src, int64_t pitch, int row0, int last, float *dst, int wave, int lane)
{
    constexpr int CH = DD / 4, RPT = 64 / CH, NTR = RT / RPT;         // 16-byte chunks per row, rows of a transfer, transfers
    constexpr int NW = NTR < 4 ? 1 : NTR / 4;                         // transfers of a wave (d = 16: of the first two)
    if (NTR < 4 && wave >= NTR) return;
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        const int r0 = (wave * NW + t) * RPT, row = r0 + lane / CH;
        const int j = min(row0 + row, last);
        dma16(src + (int64_t)j * pitch + 4 * ((lane % CH) ^ swz<DD>(row)), dst + r0 * DD);
    }
}

// Which of ny blocks of a head workgroup y of the grid (heads, ny) serves, blocks numbered from the longest.  Where the whole grid
// is resident at once (up to four workgroups per compute unit), a compute unit that gets a long one in the first round
// must get a short one in the second: every second group of 256 workgroups takes its blocks in reverse.
__device__ inline int balanced_block(int y, int ny, int heads)
{
    const int group = max(256 / heads, 1), first = y / group * group;
    return ((y / group) & 1) != 0 && y < 4 * group && first + group <= ny ? 2 * first + group - 1 - y : y;
}

// The blocks of a head on y and z of a grid: y alone ends at 65535, and a forward call is accepted up to 64 times that many rows.
struct BlockGrid { unsigned y, z; };
constexpr BlockGrid block_grid(int blocks)
{
    const unsigned z = (unsigned)(blocks + 65534) / 65535u;
    return BlockGrid{((unsigned)blocks + z - 1) / z, z};
}
constexpr bool covered(int blocks)
{
    return block_grid(blocks).y <= 65535 && block_grid(blocks).y * block_grid(blocks).z >= (unsigned)blocks &&
           block_grid(blocks).y * (block_grid(blocks).z - 1) < (unsigned)blocks;
}
static_assert(covered(1) && covered(65535) && block_grid(65535).z == 1 && covered(65536) && covered(65537) && covered(131070),
              "row blocks of the longest forward call: 64 x 65535 rows");

// C += T R^T over the features: T = 16 rows of a tile (tile row nn of the lane), R = a row per lane in registers; contraction
// slot (s, g) stands for feature DD/4 g + s on both sides, at d = 128 for 64 (s / 16) + 16 g + s % 16: chunk v of lane group g.
// Logits are to have the bits that the moments kernels give them (see weight() below), so at d = 128 they are the sum of two
// halves of the features, as there.
template <int DD>
__device__ inline int chunk_of(int g, int v) { return DD == 128 ? 16 * (v >> 2) + 4 * g + (v & 3) : DD / 16 * g + v; }

template <int DD>
__device__ inline f32x4 row_chunk(const float *trow, int g, int v, int nn)
{
    return *reinterpret_cast<const f32x4 *>(trow + 4 * (chunk_of<DD>(g, v) ^ swz<DD>(nn)));
}

// 2^x as the square of its root: the moments kernel works with the roots of the weights, and the sweeps use the same weights to
// the last bit (logits of some sixty bits amplify the difference of two roundings to the size of the result's error).
__device__ inline float weight(float x)
{
    const float root = __builtin_amdgcn_exp2f(0.5f * x);
    return root * root;
}

template <int DD>
__device__ inline void load_row(const float *row, int g, float (&x)[DD / 4])
{
#pragma unroll
    for (int v = 0; v < DD / 16; ++v) {
        const f32x4 a = *reinterpret_cast<const f32x4 *>(row + 4 * chunk_of<DD>(g, v));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * v + e] = a[e];
    }
}

// ---- row sweeps ---------------------------------------------------------------------------------------------
// MODE 0: the r sweep; MODE 1: the dQ sweep; MODE 2: the output sweep of a forward call, O_i = sum_j w_ij (y0_i + k_j . y1_i) v_j
// (third loop of Algorithm 1), rows from `skip` on (a multiple of RT, or all).  S^T = K Q^T and the like come out as (lane (g, nn): keys 4g + r, query nn),
// which is the A operand of the product that contracts over keys when slot g of step r stands for key 4g + r.
template <int DD, int MODE>
__global__ __launch_bounds__(256, 2) void bwd_rows_f32_kernel(
    const float *__restrict__ Qg, const float *__restrict__ Kg, const float *__restrict__ Vg, const float *__restrict__ Gg,
    llla_strides sq, llla_strides sk, llla_strides sv, llla_strides sg, int H, int n, int npad, float scale, float lambda,
    const float *__restrict__ LamRows, float *__restrict__ Mg, const float *__restrict__ Yg, const float *Ug, float *Rv,
    float *__restrict__ Sc, float *__restrict__ dQ, float *__restrict__ dLam, int causal = 1, int skip = 0, void *Og = nullptr,
    llla_strides so = {}, int out_bf16 = 0)
{
    constexpr int NS = DD / 4, NV = DD / 16, NB = DD / 16, YP = SP<DD> + 16, RP = DD + 4;
    __shared__ __align__(16) float tiles[2][2][RT * DD];
    __shared__ float rbest[4][16], rref[4][16], rsum[4][16];
    __shared__ int rarg[4][16];
    static_assert(4 * 16 * RP <= 4 * RT * DD, "the final sums reuse the tiles");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    const int rg = wave & 1, ks = wave >> 1;
    // head on blockIdx.x (dispatched fastest), row block on y (and z, see block_grid), longest rows first
    const int bh = blockIdx.x, b = bh / H, h = bh % H;
    const int ny = (n - skip + RT - 1) / RT, yb = (int)(blockIdx.z * gridDim.y + blockIdx.y);
    if (yb >= ny) return;
    const int i0 = skip + (ny - 1 - balanced_block(yb, ny, gridDim.x)) * RT;
    const int iq = min(i0 + 16 * rg + nn, n - 1);           // rows past the end repeat the last one and are not stored
    const int jlim = MODE == 2 && !causal ? n - 1 : iq;     // the last key the lane's query sees, and the wave's queries
    const int wlast = MODE == 2 && !causal ? n - 1 : min(i0 + 16 * rg + 15, n - 1);
    const size_t row = (size_t)bh * n + iq;
    const float *Kh = Kg + b * sk.batch + h * sk.head;
    const float *Vh = Vg + b * sv.batch + h * sv.head;
    const float cscale = scale * LOG2E;

    float qr[NS], gr[MODE < 2 ? NS : 1], yr[MODE ? NS : 1], ur[MODE == 1 ? NS : 1];
    load_row<DD>(Qg + b * sq.batch + h * sq.head + (int64_t)iq * sq.seq, g, qr);
    if constexpr (MODE < 2) load_row<DD>(Gg + b * sg.batch + h * sg.head + (int64_t)iq * sg.seq, g, gr);
    float mh = -INFINITY, y0 = 0.f, u0 = 0.f, corr = 0.f;
    int jstar = 0;
    if constexpr (MODE == 1) {
        load_row<DD>(Yg + row * YP, g, yr);
        load_row<DD>(Ug + row * YP, g, ur);
        y0 = Yg[row * YP + SP<DD>];
        u0 = Ug[row * YP + SP<DD>];
        jstar = __float_as_int(Ug[row * YP + SP<DD> + 1]);
        mh = Mg[(size_t)bh * npad + iq];
        float dl = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s) dl = fmaf(-ur[s], yr[s], dl);
        dl += __shfl_xor(dl, 16);
        dl += __shfl_xor(dl, 32);
        corr = (LamRows ? LamRows[row] : lambda) * dl;
        if (ks == 0 && g == 0 && i0 + 16 * rg + nn < n) {
            float *sc = Sc + row * 8;
            *reinterpret_cast<f32x4 *>(sc) = f32x4{y0, u0, mh, corr};
            sc[4] = __int_as_float(jstar);
            if (dLam) dLam[row] = dl;
        }
    }
    if constexpr (MODE == 2) {
        load_row<DD>(Yg + row * YP, g, yr);
        y0 = Yg[row * YP + SP<DD>];
        mh = Mg[(size_t)bh * npad + iq];
    }
    f32x4 acc[NB];
#pragma unroll
    for (int J = 0; J < NB; ++J) acc[J] = f32x4{0.f, 0.f, 0.f, 0.f};
    float csum = 0.f, best = -INFINITY, cf[4] = {0.f, 0.f, 0.f, 0.f};
    int arg = 0;
    // Where not every query of the wave sees every key of a tile, the products multiply what a row does not see by zero.  If one of the
    // tile's keys (MODE 2: values) is not finite they are left out instead, as on the vector kernels, and formed after the loop, where
    // nothing else is in registers: rows before such a key keep their results.
    bool odd = false;

    const int nblk = (MODE == 2 && !causal ? n - 1 : min(i0 + RT - 1, n - 1)) / RT + 1;
    auto issue = [&](int c) {
        dma_tile<DD>(Kh, sk.seq, c * RT, n - 1, tiles[c & 1][0], wave, lane);
        dma_tile<DD>(Vh, sv.seq, c * RT, n - 1, tiles[c & 1][1], wave, lane);
    };
    issue(0);
    for (int c = 0; c < nblk; ++c) {
        dma_wait();
        __syncthreads();                                     // step c has arrived, step c - 1 is consumed
        if (c + 1 < nblk) issue(c + 1);
        const int jb = c * RT + 16 * ks;
        if (jb > wlast) continue;                            // no query of this wave sees these keys
        const float *kt = &tiles[c & 1][0][16 * ks * DD], *vt = &tiles[c & 1][1][16 * ks * DD];
        f32x4 z = {0.f, 0.f, 0.f, 0.f}, zb = z, gm = z, at = {y0, y0, y0, y0}, bt = {u0, u0, u0, u0};
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const f32x4 kv = row_chunk<DD>(kt + nn * DD, g, v, nn);
            f32x4 vv = kv;
            if constexpr (MODE < 2) vv = row_chunk<DD>(vt + nn * DD, g, v, nn);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f32x4 &zv = DD == 128 && v >= 4 ? zb : z;
                zv = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], qr[4 * v + e], zv, 0, 0, 0);
                if constexpr (MODE < 2) gm = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[e], gr[4 * v + e], gm, 0, 0, 0);
                if constexpr (MODE >= 1) at = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], yr[4 * v + e], at, 0, 0, 0);
                if constexpr (MODE == 1) {
                    bt = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], ur[4 * v + e], bt, 0, 0, 0);
                }
            }
        }
        if constexpr (DD == 128) z += zb;
        float zs[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) zs[r] = z[r] * cscale;
        if constexpr (MODE == 0) {
            float pm = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = jb + 4 * g + r;
                if (j <= iq) {
                    pm = fmaxf(pm, zs[r]);
                    if (zs[r] > best) { best = zs[r]; arg = j; }
                }
            }
            pm = fmaxf(pm, __shfl_xor(pm, 16));
            pm = fmaxf(pm, __shfl_xor(pm, 32));
            const bool moves = pm > mh + LAZY_BITS || (mh == -INFINITY && pm > -INFINITY);
            if (__any(moves)) {
                const float rsc = !moves ? 1.f : mh == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mh - pm);
                if (moves) mh = pm;
                csum *= rsc;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float f = __shfl(rsc, 4 * g + r);
#pragma unroll
                    for (int J = 0; J < NB; ++J) acc[J][r] *= f;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = jb + 4 * g + r;
            const float w = weight(zs[r] - mh);
            if constexpr (MODE == 0) {
                cf[r] = j <= iq ? w * gm[r] : 0.f;
                csum += cf[r];
            } else if constexpr (MODE == 2) {
                cf[r] = j <= jlim ? w * at[r] : 0.f;
            } else {
                const float pv = w * at[r] * (gm[r] - bt[r]);
                cf[r] = j <= iq ? (j == jstar ? pv + corr : pv) : 0.f;
            }
        }
        const float *tile = MODE == 2 ? vt : kt;             // what the coefficients multiply: keys or values, key row kr, feature 16 J + nn
        auto value = [&](int kr, int J) { return tile[kr * DD + (nn & 3) + 4 * ((4 * J + (nn >> 2)) ^ swz<DD>(kr))]; };
        if (jb + 15 > (causal ? min(i0 + 16 * rg, n - 1) : n - 1)) {        // (a scalar branch, in the last step)
            float zero = 0.f;                                // 0 times every element
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int J = 0; J < NB; ++J) zero = fmaf(value(4 * g + r, J), 0.f, zero);
            odd = __any(!(zero == 0.f));
            asm volatile("" ::: "memory");                   // (read again for the products: kept, they cost registers in every step)
            if (odd) continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int J = 0; J < NB; ++J) acc[J] = __builtin_amdgcn_mfma_f32_16x16x4f32(cf[r], value(4 * g + r, J), acc[J], 0, 0, 0);
    }
    if (odd) {                                               // the wave's share of the last step, which is still in LDS, without what a row does not see
        const int c = nblk - 1, jb = c * RT + 16 * ks;
        const float *tile = &tiles[c & 1][MODE == 2 ? 1 : 0][16 * ks * DD];
#pragma unroll 1
        for (int gk = 0; gk < 4; ++gk)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {                // key 4 gk + r, query 4 g + e
                    const int kr = 4 * gk + r;
                    const float w = __shfl(cf[r], 16 * gk + 4 * g + e);
                    const bool seen = jb + kr <= (causal ? min(i0 + 16 * rg + 4 * g + e, n - 1) : n - 1);
#pragma unroll
                    for (int J = 0; J < NB; ++J) {
                        const float v = tile[kr * DD + (nn & 3) + 4 * ((4 * J + (nn >> 2)) ^ swz<DD>(kr))];
                        acc[J][e] = seen ? fmaf(w, v, acc[J][e]) : acc[J][e];
                    }
                }
    }

    // ---- the two halves of a row's keys meet in LDS ---------------------------------------------------------------
    float fac[4] = {1.f, 1.f, 1.f, 1.f};
    if constexpr (MODE == 0) {
        csum += __shfl_xor(csum, 16);
        csum += __shfl_xor(csum, 32);
#pragma unroll
        for (int sft = 16; sft <= 32; sft <<= 1) {
            const float ob = __shfl_xor(best, sft);
            const int oa = __shfl_xor(arg, sft);
            const bool take = ob > best || (ob == best && oa < arg);
            best = take ? ob : best;
            arg = take ? oa : arg;
        }
        if (g == 0) {
            rbest[wave][nn] = best;
            rarg[wave][nn] = arg;
            rref[wave][nn] = mh;
            rsum[wave][nn] = csum;
        }
    }
    __syncthreads();                                         // (also: every wave is done with the tiles)
    if constexpr (MODE == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {                        // from the reference exponent to the row maximum; a half
            const int q = 4 * g + r;                         // that saw no key holds zeros
            const float ref = rref[wave][q], m = fmaxf(rbest[rg][q], rbest[rg + 2][q]);
            fac[r] = ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ref - m);
        }
    }
    float *red = &tiles[0][0][0];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int J = 0; J < NB; ++J) red[(wave * 16 + 4 * g + r) * RP + 16 * J + nn] = acc[J][r] * fac[r];
    __syncthreads();
    for (int idx = tid; idx < RT * (DD / 4); idx += 256) {
        const int rw = idx / (DD / 4), c = 4 * (idx % (DD / 4));
        if (i0 + rw >= n) continue;
        const size_t ro = (size_t)bh * n + i0 + rw;
        const f32x4 s = *reinterpret_cast<const f32x4 *>(red + rw * RP + c) + *reinterpret_cast<const f32x4 *>(red + (RT + rw) * RP + c);
        if constexpr (MODE == 0) {
            *reinterpret_cast<f32x4 *>(Rv + ro * YP + c) = s;
        } else if constexpr (MODE == 2) {
            const int64_t off = b * so.batch + h * so.head + (int64_t)(i0 + rw) * so.seq + c;
            if (out_bf16) {
                typedef bf16_t bf16_4 __attribute__((ext_vector_type(4)));
                *reinterpret_cast<bf16_4 *>((bf16_t *)Og + off) = bf16_4{f32_to_bf16(s[0]), f32_to_bf16(s[1]), f32_to_bf16(s[2]), f32_to_bf16(s[3])};
            } else {
                *reinterpret_cast<f32x4 *>((float *)Og + off) = s;
            }
        } else {
            const f32x4 u = *reinterpret_cast<const f32x4 *>(Ug + ro * YP + c);
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(scale, s[e], u[e]);
            *reinterpret_cast<f32x4 *>(dQ + ro * DD + c) = o;
        }
    }
    if (MODE == 0 && tid < RT && i0 + tid < n) {
        const int w0 = tid / 16, q = tid % 16, w1 = w0 + 2;
        const size_t ro = (size_t)bh * n + i0 + tid;
        const float b0 = rbest[w0][q], b1 = rbest[w1][q], m = fmaxf(b0, b1);
        float r0 = rref[w0][q] == -INFINITY ? 0.f : rsum[w0][q] * __builtin_amdgcn_exp2f(rref[w0][q] - m);
        r0 += rref[w1][q] == -INFINITY ? 0.f : rsum[w1][q] * __builtin_amdgcn_exp2f(rref[w1][q] - m);
        const int a = b1 > b0 || (b1 == b0 && rarg[w1][q] < rarg[w0][q]) ? rarg[w1][q] : rarg[w0][q];
        Rv[ro * YP + SP<DD>] = r0;
        Rv[ro * YP + SP<DD> + 1] = __int_as_float(a);
        Mg[(size_t)bh * npad + i0 + tid] = m;
    }
}

// ---- key sweep ------------------------------------------------------------------------------------------------
// Mirror image: rows of Q, dO, y1, u1 pass through LDS, the keys' rows of K and V stay in registers; the coefficient tiles
// (lane (g, nn): queries 4g + r, key nn) are the A operands of the products that contract over the queries.
template <int DD>
__global__ __launch_bounds__(256, DD <= 64 ? 2 : 1) void bwd_keys_f32_kernel(
    const float *__restrict__ Qg, const float *__restrict__ Kg, const float *__restrict__ Vg, const float *__restrict__ Gg,
    llla_strides sq, llla_strides sk, llla_strides sv, llla_strides sg, int H, int n, float scale, const float *__restrict__ Yg,
    const float *__restrict__ Ug, const float *__restrict__ Sc, float *__restrict__ dK, float *__restrict__ dV)
{
    constexpr int NS = DD / 4, NV = DD / 16, NB = DD / 16, YP = SP<DD> + 16, RP = DD + 4;
    __shared__ __align__(16) float tiles[2][4][RT * DD];
    __shared__ __align__(16) float scal[2][RT * 8];
    static_assert(2 * 4 * 16 * RP <= 8 * RT * DD, "the final sums reuse the tiles");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    const int kg = wave & 1, qs = wave >> 1;
    // head on blockIdx.x (dispatched fastest); low key blocks see the most rows: they go first for every head
    const int bh = blockIdx.x, b = bh / H, h = bh % H;
    const int j0 = balanced_block(blockIdx.y, gridDim.y, gridDim.x) * RT;
    const int jk = min(j0 + 16 * kg + nn, n - 1);            // keys past the end repeat the last one and are not stored
    const float *Qh = Qg + b * sq.batch + h * sq.head;
    const float *Gh = Gg + b * sg.batch + h * sg.head;
    const float *Yh = Yg + (size_t)bh * n * YP, *Uh = Ug + (size_t)bh * n * YP, *Sh = Sc + (size_t)bh * n * 8;
    const float cscale = scale * LOG2E;

    float kr[NS], vr[NS];
    load_row<DD>(Kg + b * sk.batch + h * sk.head + (int64_t)jk * sk.seq, g, kr);
    load_row<DD>(Vg + b * sv.batch + h * sv.head + (int64_t)jk * sv.seq, g, vr);
    f32x4 dk[NB], dv[NB];
#pragma unroll
    for (int J = 0; J < NB; ++J) dk[J] = dv[J] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto issue = [&](int buf, int it0) {
        dma_tile<DD>(Qh, sq.seq, it0, n - 1, tiles[buf][0], wave, lane);
        dma_tile<DD>(Gh, sg.seq, it0, n - 1, tiles[buf][1], wave, lane);
        dma_tile<DD>(Yh, YP, it0, n - 1, tiles[buf][2], wave, lane);
        dma_tile<DD>(Uh, YP, it0, n - 1, tiles[buf][3], wave, lane);
        if (wave == 0) dma16(Sh + (size_t)min(it0 + (lane >> 1), n - 1) * 8 + 4 * (lane & 1), scal[buf]);
    };
    issue(0, j0);
    for (int it0 = j0, c = 0; it0 < n; it0 += RT, ++c) {
        dma_wait();
        __syncthreads();                                     // step c has arrived, step c - 1 is consumed
        if (it0 + RT < n) issue((c + 1) & 1, it0 + RT);
        const int ib = it0 + 16 * qs;
        if (ib >= n || ib + 15 < j0 + 16 * kg) continue;     // no pair of this wave in the step
        const float *qt = &tiles[c & 1][0][16 * qs * DD], *gt = &tiles[c & 1][1][16 * qs * DD];
        const float *yt = &tiles[c & 1][2][16 * qs * DD], *ut = &tiles[c & 1][3][16 * qs * DD];
        const float *st = &scal[c & 1][16 * qs * 8];
        f32x4 z = {0.f, 0.f, 0.f, 0.f}, zb = z, gm = z, at = z, bt = z;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const f32x4 qv = row_chunk<DD>(qt + nn * DD, g, v, nn), gv = row_chunk<DD>(gt + nn * DD, g, v, nn);
            const f32x4 yv = row_chunk<DD>(yt + nn * DD, g, v, nn), uv = row_chunk<DD>(ut + nn * DD, g, v, nn);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f32x4 &zv = DD == 128 && v >= 4 ? zb : z;
                zv = __builtin_amdgcn_mfma_f32_16x16x4f32(qv[e], kr[4 * v + e], zv, 0, 0, 0);
                gm = __builtin_amdgcn_mfma_f32_16x16x4f32(gv[e], vr[4 * v + e], gm, 0, 0, 0);
                at = __builtin_amdgcn_mfma_f32_16x16x4f32(yv[e], kr[4 * v + e], at, 0, 0, 0);
                bt = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[e], kr[4 * v + e], bt, 0, 0, 0);
            }
        }
        if constexpr (DD == 128) z += zb;
        float cs[4], ce[4], cp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int qrow = 4 * g + r, i = ib + qrow;
            const f32x4 s4 = *reinterpret_cast<const f32x4 *>(st + qrow * 8);      // y0, u0, m, correction
            const int jstar = __float_as_int(st[qrow * 8 + 4]);
            const bool valid = jk <= i && i < n;
            const float w = weight(z[r] * cscale - s4[2]);
            const float a = s4[0] + at[r];
            const float ev = w * (gm[r] - (s4[1] + bt[r]));
            const float pv = jk == jstar ? fmaf(a, ev, s4[3]) : a * ev;
            cs[r] = valid ? w * a : 0.f;
            ce[r] = valid ? ev : 0.f;
            cp[r] = valid ? scale * pv : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int qrow = 4 * g + r;
            int off[NB];
#pragma unroll
            for (int J = 0; J < NB; ++J) off[J] = qrow * DD + (nn & 3) + 4 * ((4 * J + (nn >> 2)) ^ swz<DD>(qrow));
#pragma unroll
            for (int J = 0; J < NB; ++J) dv[J] = __builtin_amdgcn_mfma_f32_16x16x4f32(cs[r], gt[off[J]], dv[J], 0, 0, 0);
#pragma unroll
            for (int J = 0; J < NB; ++J) dk[J] = __builtin_amdgcn_mfma_f32_16x16x4f32(ce[r], yt[off[J]], dk[J], 0, 0, 0);
#pragma unroll
            for (int J = 0; J < NB; ++J) dk[J] = __builtin_amdgcn_mfma_f32_16x16x4f32(-cs[r], ut[off[J]], dk[J], 0, 0, 0);
#pragma unroll
            for (int J = 0; J < NB; ++J) dk[J] = __builtin_amdgcn_mfma_f32_16x16x4f32(cp[r], qt[off[J]], dk[J], 0, 0, 0);
        }
    }
    __syncthreads();
    float *rk = &tiles[0][0][0], *rv = rk + 4 * 16 * RP;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int J = 0; J < NB; ++J) {
            const int o = (wave * 16 + 4 * g + r) * RP + 16 * J + nn;
            rk[o] = dk[J][r];
            rv[o] = dv[J][r];
        }
    __syncthreads();
    for (int idx = tid; idx < RT * (DD / 4); idx += 256) {
        const int rw = idx / (DD / 4), c = 4 * (idx % (DD / 4));
        if (j0 + rw >= n) continue;
        const size_t o = ((size_t)bh * n + j0 + rw) * DD + c;
        *reinterpret_cast<f32x4 *>(dK + o) =
            *reinterpret_cast<const f32x4 *>(rk + rw * RP + c) + *reinterpret_cast<const f32x4 *>(rk + (RT + rw) * RP + c);
        *reinterpret_cast<f32x4 *>(dV + o) =
            *reinterpret_cast<const f32x4 *>(rv + rw * RP + c) + *reinterpret_cast<const f32x4 *>(rv + (RT + rw) * RP + c);
    }
}

struct BwdF32Layout {
    size_t m, y, ru, sc, q, k, total;
    int npad;
};

// The rows of r are overwritten by those of u (the workgroup of the moments kernel that reads r_i writes u_i); the scalars
// of a row follow its vector: r0, later u0, and the key of the row maximum.  q, k: at d = 16 / 32 the copies of Q and K, padded to 64
// features, that the moments kernel works on (see llla_pad.hip); the sweeps read the tensors themselves.
BwdF32Layout make_bwd_f32_layout(int B, int H, int n, int d)
{
    BwdF32Layout L{};
    const size_t bh = (size_t)B * H;
    const int yp = (d < 64 ? 64 : d) + 16;
    L.npad = (n + 63) / 64 * 64;
    size_t off = 0;
    L.m = off;  off += round_up(bh * L.npad * 4, 256);
    L.y = off;  off += round_up(bh * (size_t)n * yp * 4, 256);
    L.ru = off; off += round_up(bh * (size_t)n * yp * 4, 256);
    L.sc = off; off += round_up(bh * (size_t)n * 8 * 4, 256);
    const size_t padded = d < 64 ? round_up(bh * (size_t)n * 64 * 4, 256) : 0;
    L.q = off;  off += padded;
    L.k = off;  off += padded;
    L.total = off;
    return L;
}

template <int DD, int MODE>
hipError_t launch_rows(const BackwardProblem &p, const BwdF32Layout &L)
{
    char *ws = static_cast<char *>(p.ws);
    float *M = reinterpret_cast<float *>(ws + L.m), *Y = reinterpret_cast<float *>(ws + L.y);
    float *RU = reinterpret_cast<float *>(ws + L.ru), *Sc = reinterpret_cast<float *>(ws + L.sc);
    hipLaunchKernelGGL((bwd_rows_f32_kernel<DD, MODE>), dim3(p.B * p.H, (p.n + RT - 1) / RT), dim3(256), 0, p.stream,
                       static_cast<const float *>(p.Q), static_cast<const float *>(p.K), static_cast<const float *>(p.V),
                       static_cast<const float *>(p.dO), p.sq, p.sk, p.sv, p.sdo, p.H, p.n, L.npad, p.scale, p.lambda,
                       p.lambda_rows, M, (const float *)Y, (const float *)RU, RU, Sc, p.dQ, p.dlambda);
    return hipGetLastError();
}

}  // namespace

hipError_t mfma_output_f32(const Problem &p, int npad, float *M, const float *Y, int skip)
{
    if (skip >= p.n) return hipSuccess;
    const float *Q = static_cast<const float *>(p.Q), *K = static_cast<const float *>(p.K), *V = static_cast<const float *>(p.V);
    const BlockGrid grid = block_grid((p.n - skip + RT - 1) / RT);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(p.B * p.H, grid.y, grid.z), dim3(256), 0, p.stream, Q, K, V, nullptr, p.sq, p.sk, p.sv,
                           llla_strides{}, p.H, p.n, npad, p.scale, 0.f, nullptr, M, Y, nullptr, nullptr, nullptr, nullptr, nullptr,
                           p.causal, skip, p.O, p.so, p.out == LLLA_BF16 ? 1 : 0);
    };
    if (p.d == 128) launch(bwd_rows_f32_kernel<128, 2>);
    else if (p.d == 64) launch(bwd_rows_f32_kernel<64, 2>);
    else if (p.d == 32) launch(bwd_rows_f32_kernel<32, 2>);
    else launch(bwd_rows_f32_kernel<16, 2>);
    return hipGetLastError();
}

bool mfma_backward_f32_supported(int n, int d, llla_dtype in)
{
    return in == LLLA_F32 && (d == 16 || d == 32 || d == 64 || d == 128) && (n + RT - 1) / RT <= 65535;
}

size_t mfma_backward_f32_workspace_bytes(int B, int H, int n, int d) { return make_bwd_f32_layout(B, H, n, d).total; }

namespace {

template <int DD>
hipError_t launch_backward_f32(const BackwardProblem &p)
{
    const BwdF32Layout L = make_bwd_f32_layout(p.B, p.H, p.n, DD);
    char *ws = static_cast<char *>(p.ws);
    const float *Y = reinterpret_cast<const float *>(ws + L.y), *U = reinterpret_cast<const float *>(ws + L.ru);
    const float *Sc = reinterpret_cast<const float *>(ws + L.sc);
    stage_mark(p.stream, "backward_r");
    hipError_t e = launch_rows<DD, 0>(p, L);
    if (e != hipSuccess) return e;
    stage_mark(p.stream, "moments");
    BackwardProblem pm = p;
    if constexpr (DD < 64) {
        e = pad_queries_keys(p, ws + L.q, ws + L.k);
        if (e != hipSuccess) return e;
        pm.Q = ws + L.q;
        pm.K = ws + L.k;
        pm.sq = pm.sk = llla_strides{(int64_t)p.H * p.n * 64, (int64_t)p.n * 64, 64};
        pm.live_d = DD;
    }
    float *M = reinterpret_cast<float *>(ws + L.m), *Yw = reinterpret_cast<float *>(ws + L.y), *RU = reinterpret_cast<float *>(ws + L.ru);
    e = DD == 128 ? mfma_moments_f32_wide_given(pm, L.npad, M, Yw, RU) : mfma_moments_f32_given(pm, L.npad, M, Yw, RU);
    if (e != hipSuccess) return e;
    stage_mark(p.stream, "backward_dq");
    e = launch_rows<DD, 1>(p, L);
    if (e != hipSuccess) return e;
    stage_mark(p.stream, "backward_keys");
    hipLaunchKernelGGL((bwd_keys_f32_kernel<DD>), dim3(p.B * p.H, (p.n + RT - 1) / RT), dim3(256), 0, p.stream,
                       static_cast<const float *>(p.Q), static_cast<const float *>(p.K), static_cast<const float *>(p.V),
                       static_cast<const float *>(p.dO), p.sq, p.sk, p.sv, p.sdo, p.H, p.n, p.scale, Y, U, Sc, p.dK, p.dV);
    return hipGetLastError();
}

}  // namespace

hipError_t mfma_backward_f32(const BackwardProblem &p)
{
    return p.d == 16 ? launch_backward_f32<16>(p) : p.d == 32 ? launch_backward_f32<32>(p)
           : p.d == 64 ? launch_backward_f32<64>(p) : launch_backward_f32<128>(p);
}

}  // namespace llla
