// Matrix-core forward path for fp32 inputs, d = 64 (and the moments at d = 16 / 32, on copies in rows of 64 features), with the accuracy of the vector kernels and no value-range condition: logits and
// first moment on v_mfma_f32_16x16x4_f32, the second moment Sigma~_i = Z^T Z with the rows z_j = sqrt(w_ij) k_j split into three bf16
// (24 significant bits, fp32's exponents) on 16-bit MFMA, six of the nine partial products, fp32 accumulation.
//
// What bounds it: on fp32 MFMA the second moment is 256 matrix-core cycles per 16x16 tile and 32 keys, and 80 % of the call.  Six
// products of 16-bit MFMA are 96.  Both operands being the same z, a query's keys are scaled and split once (36 vector
// instructions per 16 features and lane, 2.9 per MFMA; three fit beside one), and products and splitting are made to alternate.
// 16 heads x 1024: call 606 -> 419 us.  Errors against fp64 over normal, unit, peaked and badly scaled inputs, ridges 10^-2 and
// 10^-4: equal or smaller (unit, 10^-2: 1.7e-6 before and after; normal: 1.4e-5 and 1.2e-5).
//
//   moments  per block of 16 queries: weights, omega_i, mu~_i and Sigma~_i (Eq. (tilded_form)) on chip, the ten upper
//            16x16 tiles of Sigma~_i per query in MFMA accumulators, then the exact per-query solve (solve_wave_q4);
//   output   third loop of Algorithm 1 as a flash-style sweep, its three products on fp32 MFMA (llla_mfma_bwd_f32.hip);
//   rows that see at most 64 keys are served in fp64 and key space (llla_dual.hpp) by further workgroups of the moments kernel:
//            serial chains that share a compute unit with the matrix-core workgroups instead of running alone at the end.
//
// Running maximum.  There is no separate sweep for the row maxima.  fp32 weights have 2^127 of headroom, so the
// weights are taken relative to a reference exponent mh_i that only moves when a block's largest logit exceeds it by
// more than 2^64 (Algorithm 1's running maximum and rescale, applied lazily: for ordinary data mh_i is the first
// block's maximum and never moves), while the true maximum m_i is tracked beside it.  With F_i = 2^(m_i - mh_i) every
// moment is F_i times the max-normalised one, so the system solved is the max-normalised one times F_i:
// [omega' mu~'^T; mu~' Sigma~' + lambda F I] y' = [1; q], and the output weights w'_ij (y0' + k_j . y1') equal those of
// Eq. (lla).  mh_i and y'_i go to the output sweep; delta_i = delta'_i / F_i (rho_i needs no correction).
#include <algorithm>
#include "llla_dual.hpp"
#include "llla_mfma_common.hpp"
#include "llla_mfma_solve64.hpp"

namespace llla {
namespace {

using namespace mfma;

constexpr int FD = 64;                 // head dimension
constexpr int FKB = 64;                // keys per block
constexpr int FWP = 68;                // floats per query row of the weight tile
constexpr float LAZY_BITS = 64.f;      // the reference exponent moves when a block exceeds it by more than this

struct F32Layout {
    size_t m, lf, y, total;
    int npad;
};

F32Layout make_f32_layout(int B, int H, int n)
{
    F32Layout L;
    L.npad = (n + FKB - 1) / FKB * FKB;
    const size_t bh = (size_t)B * H;
    size_t off = 0;
    L.m = off;  off += round_up(bh * L.npad * 4, 256);                       // reference exponent mh (log2 units)
    L.lf = off; off += round_up(bh * L.npad * 4, 256);                       // log2 F = m - mh
    L.y = off;  off += round_up(bh * (size_t)n * Shape<FD>::YP * 4, 256);    // y' rows
    L.total = off;
    return L;
}

// The K tile of one block: 64 keys x 64 floats, unpadded (the DMA writes whole 1 KB wave rows), 16-byte chunks
// XOR-swizzled so that both operand reads are free of bank conflicts: chunk c of key row r sits at c ^ swz(r),
// swz(r) = ((r & 1) << 2) | ((r >> 1) & 3).  (b32 reads of rows 4s+g, g = 0..3, 16 consecutive floats each: rows of
// different parity land in different halves of the banks; b128 reads of 8 consecutive rows at one chunk: 8 distinct
// chunk positions.)
__device__ inline int swz(int r) { return ((r & 1) << 2) | ((r >> 1) & 3); }

struct F32Shared {
    float kt[2][FKB * FD];
    float wt[16 * FWP];                // roots of the weights of the current block: [query][g * 16 + s], key = 4 s + g
    float pm[4][16];                   // block maximum of every query, per weight wave
    float rs[16];                      // rescale factor of every query for this block (1 unless its reference moved)
    float mus[16][FD + 4];
    float oms[16];
    float fsc[16];                     // F of every query
    float sc[4][4][16 * SC_PITCH];
};

// schedule: N times one MFMA, then V vector instructions
template <int N, int V>
__device__ __forceinline__ void alternate()
{
    if constexpr (N > 0) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
        alternate<N - 1, V>();
    }
}

// LIVE: feature blocks of 16 that can be non-zero (4, except for calls at d = 16 / 32 that run here on zero-padded
// copies: the tiles, scaled operands and solve blocks of padded feature blocks are skipped, see moments_body).
// BWD (the backward pass, llla_mfma_bwd_f32.hip): Mg holds the row maxima already, so nothing is ever rescaled and one of
// the three barriers per block goes; RUg holds r1 and r0 of every row (pitch YP, r0 at [FD]) and receives u1, u0 in their
// place -- the right-hand sides are read before the solve by the lanes that store its result.
template <int LIVE, bool BWD = false>
__global__ __launch_bounds__(256, 2) void moments_f32_kernel(const float *__restrict__ Qg, const float *__restrict__ Kg,
                                                            llla_strides sq, llla_strides sk, int H, int n, int npad,
                                                            float cscale, float lambda, const float *__restrict__ lam_rows,
                                                            float *__restrict__ Mg, float *__restrict__ LFg,
                                                            float *__restrict__ Yg, float *__restrict__ RUg, int causal, int nqb,
                                                            dual::DualArgs da, int rows_at, int mixed, int out_bf16)
{
    // nqb: blocks of 16 query rows the sequence has; rows [0, da.nrows), a multiple of 16 or all, are the key-space workgroups' (four each),
    // which start after rows_at others and work on the caller's own tensors (mixed: see block_order)
    using S = Shape<FD>;
    constexpr int NB = 4, QW = 4, QB = 16, YP = S::YP;
    // The backward at d = 16 / 32 sums mu~ and omega on the vector ALU, from the same rounded sqrt(w) k that Sigma~ is formed of, which leaves
    // the centred matrix of a row with few keys less noise than a product of rounded weights with the keys.  Errors against fp64, keys with a
    // common offset of 3 0.65 to 0.87 times what they were, unit keys with ridge 10^-4 0.84 to 1.0; 256 heads x 512, d = 16, 490 -> 467 us,
    // 256 x 256, d = 32, 301 -> 292.
    constexpr bool MU_VALU = BWD && LIVE < 4;
    __shared__ __align__(16) F32Shared sm;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    const int own = BWD ? nqb : nqb - (da.nrows + QB - 1) / QB;      // blocks of a head here
    const int lin = linear_block();
    BlockMap bm;
    if constexpr (BWD) {
        bm = xcd_block_map(lin, own, (int)gridDim.y);
    } else {
        const int heads = (int)gridDim.y, parts = ((int)gridDim.x - own) * heads, at = lin - rows_at;
        if (__builtin_expect((unsigned)at < (unsigned)parts, 0)) {
            const int bh = (int)((unsigned)at % (unsigned)heads), part = (int)((unsigned)at / (unsigned)heads);
            using DS = dual::DualSharedRows<16 * LIVE, 4>;
            static_assert(sizeof(DS) <= sizeof(F32Shared), "key-space rows fit the workgroup's LDS");
            auto &ds = *reinterpret_cast<DS *>(&sm);
            const int top = da.nrows - 1 - 4 * part;
            if (out_bf16) dual::dual_forward_rows<16 * LIVE, 4, bf16_t>(ds, da, bh, top);
            else dual::dual_forward_rows<16 * LIVE, 4, float>(ds, da, bh, top);
            return;
        }
        const int l = at < 0 ? lin : lin - parts;
        bm = mixed ? BlockMap{(int)((unsigned)l % (unsigned)heads), (int)((unsigned)l / (unsigned)heads)} : xcd_block_map(l, own, heads);
    }
    const int bh = bm.bh, b = bh / H, h = bh % H;
    const int i0 = (nqb - 1 - bm.blk) * QB;                           // long rows first
    const int ilast = min(i0 + QB - 1, n - 1);
    const int nblk = causal ? ilast / FKB + 1 : (n + FKB - 1) / FKB;
    const float *Kh = Kg + b * sk.batch + h * sk.head;
    const float *Qh = Qg + b * sq.batch + h * sq.head;

    // weight role: lane (g, nn) of wave w serves query i0 + nn and keys 16 w + 4 g + r of a block
    const int iq = i0 + nn;
    const int jlim = causal ? iq : n - 1;                              // last key the lane's query sees
    const bool q_live = iq < n;
    // the 16 query rows wait in LDS (in the rows that hold mu~ after the sweep) instead of in 16 registers per lane:
    // thread t brings floats 4 (t % 16) .. + 3 of query t / 16
    {
        const int qr = tid >> 4, qc = 4 * (tid & 15);
        *reinterpret_cast<f32x4 *>(&sm.mus[qr][qc]) =
            *reinterpret_cast<const f32x4 *>(Qh + (int64_t)min(i0 + qr, n - 1) * sq.seq + qc);
    }

    f32x4 acc[QW][10];
#pragma unroll
    for (int q = 0; q < QW; ++q)
#pragma unroll
        for (int t = 0; t < 10; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 mu_acc = {0.f, 0.f, 0.f, 0.f};
    float mu[QW][LIVE];                    // MU_VALU: this lane's share (keys of its lane group) of mu~'[16 I + nn]
#pragma unroll
    for (int q = 0; q < QW; ++q)
#pragma unroll
        for (int I = 0; I < LIVE; ++I) mu[q][I] = 0.f;
    float om_part = 0.f;                   // this lane's share of omega' of query nn (its keys: 4 g + r of every wave block)
    float mh = -INFINITY, mtrue = -INFINITY;   // reference exponent and true maximum of query nn (log2 units)
    if constexpr (BWD) mh = Mg[(size_t)bh * npad + min(iq, n - 1)];

    // DMA of one K block: 16 KB = 16 wave transfers of 1 KB, four per wave; transfer t of wave w fills key rows
    // 16 w + 4 t .. + 3; lane l of it writes row 16 w + 4 t + l / 16, stored chunk l % 16
    // Full blocks: a wave-uniform base address per block (scalar registers) plus one 32-bit byte offset per lane and
    // transfer, formed when needed from an opaque copy of the lane index (nothing address-like stays live over the
    // sweep); the last, ragged block clamps its rows to n - 1.
    auto issue_dma = [&](int blk) {
        float *dst = sm.kt[blk & 1];
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));
        if (blk * FKB + FKB <= n && sk.seq < (int64_t(1) << 23)) {       // whole block, byte offsets fit 32 bits
            const float *base = Kh + (int64_t)blk * FKB * sk.seq;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int row = 16 * wave + 4 * t + (lane_e >> 4);
                const int chunk = (lane_e & 15) ^ swz(row);
                dma16_base(base, (unsigned)(row * (int)sk.seq + 4 * chunk) * 4u, dst + (16 * wave + 4 * t) * FD);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int row = 16 * wave + 4 * t + (lane_e >> 4);
                const int j = min(blk * FKB + row, n - 1);
                const int chunk = (lane_e & 15) ^ swz(row);
                dma16(Kh + (int64_t)j * sk.seq + 4 * chunk, dst + (16 * wave + 4 * t) * FD);
            }
        }
    };

    issue_dma(0);
    __builtin_amdgcn_s_setprio(2);         // the loop before the solve of the other workgroup of the compute unit: 1-2 %
    for (int c = 0; c < nblk; ++c) {
        const float *kt = sm.kt[c & 1];
        dma_wait();
        __syncthreads();                   // tile c complete; everybody is done with block c-1

        // ---- weights of block c: S^T = K Q^T for this wave's 16 keys, contraction slot (s, g) <-> feature 4 LIVE g + s ----
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
        {
            const int row = 16 * wave + nn;
            const float *krow = kt + row * FD;
            const int sw = swz(row);
#pragma unroll
            for (int v = 0; v < LIVE; ++v) {
                const f32x4 kv = *reinterpret_cast<const f32x4 *>(krow + 4 * ((LIVE * g + v) ^ sw));
                const f32x4 qv = *reinterpret_cast<const f32x4 *>(&sm.mus[nn][4 * LIVE * g + 4 * v]);   // Q[query nn][4 (LIVE g + v) ..]
#pragma unroll
                for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], qv[e], z, 0, 0, 0);
            }
        }
        float zs[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) zs[r] = z[r] * cscale;
        if constexpr (!BWD) {
            float pmx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = c * FKB + 16 * wave + 4 * g + r;
                pmx = (q_live && j <= jlim) ? fmaxf(pmx, zs[r]) : pmx;
            }
            pmx = fmaxf(pmx, __shfl_xor(pmx, 16));
            pmx = fmaxf(pmx, __shfl_xor(pmx, 32));
            if (g == 0) sm.pm[wave][nn] = pmx;
            __syncthreads();
            const float bmx = fmaxf(fmaxf(sm.pm[0][nn], sm.pm[1][nn]), fmaxf(sm.pm[2][nn], sm.pm[3][nn]));
            mtrue = fmaxf(mtrue, bmx);
            float rsc = 1.f;
            if (bmx > mh + LAZY_BITS || (mh == -INFINITY && bmx > -INFINITY)) {       // the reference moves (first block: always)
                rsc = (mh == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mh - bmx);
                mh = bmx;
            }
            if (wave == 0 && g == 0) sm.rs[nn] = rsc;
            om_part *= rsc;
        }
        {
            float wf[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = c * FKB + 16 * wave + 4 * g + r;
                const float root = __builtin_amdgcn_exp2f(0.5f * (zs[r] - mh));
                const float sw = (q_live && j <= jlim) ? root : 0.f;
                sm.wt[nn * FWP + r * 16 + 4 * wave + g] = sw;
                if constexpr (MU_VALU) om_part = fmaf(sw, sw, om_part);
                else wf[r] = sw * sw;
            }
            if constexpr (!MU_VALU) om_part += (wf[0] + wf[1]) + (wf[2] + wf[3]);
        }
        // The last block holds keys behind the workgroup's first query, whose weight 0 must stay 0 in the products below: an element that is not
        // finite is cleared, now that its logits are formed (rows that see it have a weight that is not a number).  Each wave has read
        // only its own 16 rows so far.  (Once per workgroup; a select or a check in the products' loop cost 1 to 3 % of a d = 16 / 32 call.)
        if (c == nblk - 1) {
            float *krow = sm.kt[c & 1] + (16 * wave + nn) * FD;
#pragma unroll
            for (int v = 0; v < LIVE; ++v) {
                f32x4 *kv = reinterpret_cast<f32x4 *>(krow + 4 * ((LIVE * g + v) ^ swz(16 * wave + nn)));
                f32x4 x = *kv;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = fabsf(x[e]) < INFINITY ? x[e] : 0.f;
                *kv = x;
            }
        }
        __syncthreads();                   // weights and rescale factors of block c visible
        if (c + 1 < nblk) issue_dma(c + 1);

        // ---- rescale what has been accumulated (factors are 1 unless a reference exponent moved) -------------------
        if constexpr (!BWD) {
            const f32x4 r4 = *reinterpret_cast<const f32x4 *>(&sm.rs[4 * g]);        // rows 4 g + r of mu~
#pragma unroll
            for (int r = 0; r < 4; ++r) mu_acc[r] *= r4[r];
            const f32x4 mine = *reinterpret_cast<const f32x4 *>(&sm.rs[QW * wave]);  // this wave's four queries
#pragma unroll
            for (int q = 0; q < QW; ++q) {
                if (mine[q] != 1.f) {                                                  // wave-uniform
#pragma unroll
                    for (int t = 0; t < 10; ++t) acc[q][t] *= mine[q];
                }
            }
        }

        // ---- moments of block c, in halves of 32 keys, up to the last key a query of the workgroup sees -----------
        const int nhalf = causal ? min(2, (ilast - c * FKB) / 32 + 1) : 2;
#pragma unroll 1
        for (int hf = 0; hf < nhalf; ++hf) {
            // Key 4 (8 hf + t) + g is slot t of lane group g; its row starts at t * 4 FD from this lane's first.  The swizzle of row
            // 4 t + g is ((g & 1) << 2) | ((2 t + (g >> 1)) & 3), so four addresses per lane (parities of t and I) and immediates
            // serve all reads.  (They are formed from copies of the lane indices that the compiler cannot see through: it would
            // keep all 32 in registers over the whole sweep.)
            int g_e = g, nn_e = nn;
            asm volatile("" : "+v"(g_e), "+v"(nn_e));
            const int c4 = nn_e >> 2;
            const float *krow = kt + (32 * hf + g_e) * FD + (nn_e & 3);
            const float *ka[2][2];
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int ip = 0; ip < 2; ++ip) ka[tp][ip] = krow + 4 * (4 * (ip ^ (g_e & 1)) + (c4 ^ ((2 * tp + (g_e >> 1)) & 3)));
            // Work items (query q, feature block I): z = sqrt(w) k of block I in three bf16, then the products of block I with
            // blocks 0..I.  A wave's vector instructions and MFMAs overlap only where they alternate, so a region of the schedule
            // holds the products of one item and the z of the next.
            bf16x8 zh[QW + 1][NB], zm[QW + 1][NB], zl[QW + 1][NB];
            f32x4 w0, w1;
            auto make_z = [&](int q, int I) {
                if (I == 0) {
                    const float *wp = &sm.wt[(QW * wave + q) * FWP + g_e * 16 + 8 * hf];
                    w0 = *reinterpret_cast<const f32x4 *>(wp);
                    w1 = *reinterpret_cast<const f32x4 *>(wp + 4);
                }
                // read again for every query: 32 registers for the keys of a half would push accumulators into scratch memory (as it is,
                // 37 are spilled around this loop; nothing inside it touches scratch memory)
                asm volatile("" ::: "memory");
                float x[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float sw = t < 4 ? w0[t & 3] : w1[t & 3];
                    x[t] = sw * ka[t & 1][I & 1][4 * t * FD + 32 * (I >> 1)];
                    if constexpr (MU_VALU) mu[q][I] = fmaf(sw, x[t], mu[q][I]);
                }
                split3_bf16(x, zh[q][I], zm[q][I], zl[q][I]);
            };
            make_z(0, 0);
#pragma unroll
            for (int q = 0; q < QW; ++q)
#pragma unroll
                for (int I = 0; I < LIVE; ++I) {
                    if (I + 1 < LIVE) make_z(q, I + 1);
                    else if (q + 1 < QW) make_z(q + 1, 0);
                    // six products of the nine: what is left out is below 2^-24 of the result.  In a diagonal tile h^T m and m^T h (and
                    // h^T l and l^T h) are each other's transposes: (2 h)^T m and (2 h)^T l serve, and the solve's (T + T^T) / 2 does the rest.
#pragma unroll
                    for (int J = 0; J < I; ++J) {
                        f32x4 &t = acc[q][S::tix(J, I)];
                        t = mfma_bf16(zl[q][J], zh[q][I], t);
                        t = mfma_bf16(zh[q][J], zl[q][I], t);
                        t = mfma_bf16(zm[q][J], zm[q][I], t);
                        t = mfma_bf16(zm[q][J], zh[q][I], t);
                        t = mfma_bf16(zh[q][J], zm[q][I], t);
                        t = mfma_bf16(zh[q][J], zh[q][I], t);
                    }
                    {
                        f32x4 &t = acc[q][S::tix(I, I)];
                        const bf16x8 h2 = twice_bf16(zh[q][I]);
                        t = mfma_bf16(h2, zl[q][I], t);
                        t = mfma_bf16(zm[q][I], zm[q][I], t);
                        t = mfma_bf16(h2, zm[q][I], t);
                        t = mfma_bf16(zh[q][I], zh[q][I], t);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
                    if (I == 0) alternate<4, 11>();
                    else if (I == 1) alternate<10, 5>();
                    else if (I == 2) alternate<16, 3>();
                    else alternate<22, 2>();
                    __builtin_amdgcn_sched_barrier(0);
                }
            if constexpr (MU_VALU) continue;
            // mu~: fp32, four keys per MFMA, the weights of all 16 queries against this wave's feature block
            const float *wp = &sm.wt[nn_e * FWP + g_e * 16 + 8 * hf];
            w0 = *reinterpret_cast<const f32x4 *>(wp);
            w1 = *reinterpret_cast<const f32x4 *>(wp + 4);
            if (LIVE < 4 && wave >= LIVE) continue;       // a padded feature block (a scalar branch)
            // (this wave's two addresses as offsets: chosen among the four pointers they were loads through the generic address space, each waited for by
            // itself and for the transfers of the next block with it)
            const int row0 = (32 * hf + g_e) * FD + (nn_e & 3), blk = 4 * ((wave & 1) ^ (g_e & 1));
            const int at[2] = {row0 + 4 * (blk + (c4 ^ (g_e >> 1))) + 32 * (wave >> 1), row0 + 4 * (blk + (c4 ^ (2 + (g_e >> 1)))) + 32 * (wave >> 1)};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float sw = t < 4 ? w0[t & 3] : w1[t & 3];
                const float kmu = kt[at[t & 1] + 4 * t * FD];
                mu_acc = __builtin_amdgcn_mfma_f32_16x16x4f32(-sw * sw, kmu, mu_acc, 0, 0, 0);   // -mu~'[query 4g+r][16 wave + nn]
            }
        }
    }
#pragma unroll
    for (int q = 0; q < QW; ++q)                                      // the solve works on -Sigma~'
#pragma unroll
        for (int t = 0; t < 10; ++t) acc[q][t] = -acc[q][t];

    __builtin_amdgcn_s_setprio(0);
    // ---- hand mu~', omega' and F to the waves that own the queries -------------------------------------------------
    __syncthreads();
    if constexpr (!MU_VALU) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sm.mus[4 * g + r][16 * wave + nn] = mu_acc[r];
    } else {
#pragma unroll
        for (int q = 0; q < QW; ++q)
#pragma unroll
            for (int I = 0; I < NB; ++I) {
                float m = 0.f;                                          // (padded blocks)
                if (I < LIVE) {
                    m = mu[q][I < LIVE ? I : 0];
                    m += __shfl_xor(m, 16);
                    m += __shfl_xor(m, 32);
                }
                if (g == 0) sm.mus[QW * wave + q][16 * I + nn] = -m;
            }
    }
    om_part += __shfl_xor(om_part, 16);
    om_part += __shfl_xor(om_part, 32);
    if (g == 0) sm.pm[wave][nn] = om_part;
    const float lf = (q_live && !BWD) ? mtrue - mh : 0.f;                // log2 F
    if (wave == 0 && g == 0) {
        sm.fsc[nn] = __builtin_amdgcn_exp2f(lf);
        if (q_live && !BWD) {
            Mg[(size_t)bh * npad + iq] = mh;
            LFg[(size_t)bh * npad + iq] = lf;
        }
    }
    __syncthreads();
    if (tid < 16) sm.oms[tid] = ((sm.pm[0][tid] + sm.pm[1][tid]) + (sm.pm[2][tid] + sm.pm[3][tid]));
    __syncthreads();

    // ---- the ridge lambda F on the diagonal (the tiles hold -Sigma~'), the intercept eliminated, then the solve -----------
    // The intercept goes first, which leaves the centred Sigma~ - mu~ mu~^T / omega + lambda F I: at least lambda F however few keys
    // the row sees.  Eliminated last it leaves omega - mu~^T (Sigma~ + lambda F I)^-1 mu~, which few keys far apart cancel to zero in
    // fp32 (64 rows, features from 10^-3 to 10, ridge 10^-4: non-finite gradients).
    const int qi = QW * wave + g;                                       // solve role: lane (g, nn) = (query, element)
    const int row = min(i0 + qi, n - 1);
#pragma unroll
    for (int q = 0; q < QW; ++q) {
        const int rq = min(i0 + QW * wave + q, n - 1);
        const float lq = (lam_rows ? lam_rows[(size_t)bh * n + rq] : lambda) * sm.fsc[QW * wave + q];
        const float oinv = 1.f / sm.oms[QW * wave + q];
        const float *mq = sm.mus[QW * wave + q];
        float mc[NB];
#pragma unroll
        for (int J = 0; J < LIVE; ++J) mc[J] = mq[16 * J + nn];
#pragma unroll
        for (int I = 0; I < NB; ++I) {
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[q][S::tix(I, I)][t] -= (nn == 4 * g + t) ? lq : 0.f;
            if (I < LIVE) {
                const f32x4 mr = oinv * *reinterpret_cast<const f32x4 *>(mq + 16 * I + 4 * g);
#pragma unroll
                for (int J = I; J < LIVE; ++J)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[q][S::tix(I, J)][t] = fmaf(mr[t], mc[J], acc[q][S::tix(I, J)][t]);
            }
        }
    }
    const float pivot_floor = 0.5f * (lam_rows ? lam_rows[(size_t)bh * n + row] : lambda) * sm.fsc[qi];
    const float *qrow = Qh + (int64_t)row * sq.seq;
    const float oinv = 1.f / sm.oms[qi];
    float nm[4], tmu[4], tq[4], te[4], y1[4], u1[4], y0 = 0.f, u0 = 0.f;
    float r0 = 0.f;
    const float *rr = BWD ? RUg + ((size_t)bh * n + row) * YP : nullptr;
    if constexpr (BWD) r0 = rr[FD];
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        nm[P] = sm.mus[qi][16 * P + nn];                                 // -mu~'
        tmu[P] = 0.f;
        tq[P] = fmaf(-nm[P], oinv, -qrow[16 * P + nn]);                  // -(q - mu~ / omega)
        te[P] = BWD ? fmaf(-nm[P], r0 * oinv, -rr[16 * P + nn]) : 0.f;   // -(r1 - mu~ r0 / omega)
        y1[P] = 0.f; u1[P] = 0.f;
    }
    // (pivots below half the ridge are dropped, not raised: 500 rows with a common offset of 30 in all features, ridge 10^-2, had NaN in 832
    // rows of dK and in 18 of O)
    solve_wave_q4<BWD, LIVE, true, false>(acc, tmu, tq, te, r0, 1.f, &sm.sc[wave][0][0], g, nn, pivot_floor, y1, y0, u1, u0);
    {
        float my = 0.f, mu = 0.f;
#pragma unroll
        for (int P = 0; P < LIVE; ++P) {
            my = fmaf(nm[P], y1[P], my);
            if constexpr (BWD) mu = fmaf(nm[P], u1[P], mu);
        }
        y0 = (1.f + row_allsum(my)) * oinv;
        if constexpr (BWD) u0 = (r0 + row_allsum(mu)) * oinv;
    }
    if (i0 + qi < n) {
        float *yr = Yg + ((size_t)bh * n + row) * YP;
#pragma unroll
        for (int P = 0; P < NB; ++P) yr[16 * P + nn] = y1[P];
        if (nn == 0) yr[FD] = y0;
        if constexpr (BWD) {
            float *ur = RUg + ((size_t)bh * n + row) * YP;
#pragma unroll
            for (int P = 0; P < NB; ++P) ur[16 * P + nn] = u1[P];
            if (nn == 0) ur[FD] = u0;
        }
    }
}

// The order in which the workgroups of a launch start: `rows_at` blocks of query rows, then all key-space workgroups, then the other blocks; mixed: the
// longest block of every head, then the second longest ..., else head by head, a head's blocks on one XCD (xcd_block_map).
// A launch of some 500 workgroups, what the GPU holds at once, is as long as its worst compute unit, and which two workgroups share one follows from the
// order: neighbours go round the XCDs, and on an XCD the 33rd joins the first.  Head by head, the longest block of a head joins one of the next head
// that is nearly as long, and a further workgroup waits for the shader engine whose turn it is.  Mixed, the first 256 are the longest of the call, each
// on a compute unit of its own; then come the short key-space workgroups (all else at d = 64 is longer), and short blocks at the end fill what is left.
// us a call, head by head with the key-space workgroups behind their own head's blocks / behind all blocks / this, d = 64: 4 x 1500 325 / 366 / 268,
// 12 x 500 138 / 145 / 107, 16 x 500 139 / 140 / 112, 16 x 600 160 / 172 / 144, 16 x 1000 332 / 324 / 314, 64 x 1000 1224 / 1115 / 1089.
// Where a head has fewer than 24 blocks for its 16 key-space workgroups they are no small part of the call any more and go last (mixed, 48 x 300 153 ->
// 161, 16 x 350 93 -> 96); with more than 16 heads the same holds up to 28 blocks (40 x 480 221 -> 229).
// At d = 16 / 32 a block is hardly longer than a key-space workgroup.  In front of all else, where they meet the longest blocks, they pay while they are few, three for
// eight compute units, or while all start at once (d = 16, 4 x 1100 86 -> 75, behind 256 blocks 88; d = 32, 10 x 500 82 -> 76; d = 16, 10 x 600, 500 workgroups,
// 69 -> 72), behind 256 blocks where the blocks alone fill the GPU nearly twice (d = 16, 16 x 600 92 -> 73; 8 x 900, 424 blocks, 76 -> 83).
struct BlockOrder { int rows_at, mixed; };
inline BlockOrder block_order(int live, int heads, int own, int parts)
{
    const int blocks = own * heads;
    if (parts == 0) return BlockOrder{blocks, 0};
    if (live == 4) return own >= (heads <= 16 ? 24 : 28) ? BlockOrder{std::min(blocks, 256), 1} : BlockOrder{blocks, 0};
    if (blocks > 256 && (parts * heads <= 96 || blocks + parts * heads <= 480)) return BlockOrder{0, 1};
    return blocks >= 480 ? BlockOrder{256, 1} : BlockOrder{blocks, 0};
}

// Statistics of Eq. (lla) from y' and F: 1/delta' = y0' + q . y1', delta = delta' / F, rho = -delta' y1'.  One wave per row.
__global__ __launch_bounds__(256) void stats_f32_kernel(const float *__restrict__ Qg, llla_strides sq, int H, int n, int npad,
                                                        const float *__restrict__ Yg, const float *__restrict__ LFg,
                                                        float *__restrict__ rho, float *__restrict__ delta, int d, int skip)
{
    constexpr int YP = Shape<FD>::YP;
    const int lane = threadIdx.x % 64, i = blockIdx.x * 4 + threadIdx.x / 64, bh = blockIdx.y;
    if (i >= n || i < skip) return;
    const float *qrow = Qg + (bh / H) * sq.batch + (bh % H) * sq.head + (int64_t)i * sq.seq;
    const float *yr = Yg + ((size_t)bh * n + i) * YP;
    const float y1 = yr[lane];
    float qy = lane < d ? qrow[lane] * y1 : 0.f;
#pragma unroll
    for (int sft = 32; sft >= 1; sft >>= 1) qy += __shfl_xor(qy, sft);
    const float dl = 1.f / (yr[FD] + qy);                                 // delta'
    const size_t row = (size_t)bh * n + i;
    if (delta != nullptr && lane == 0) delta[row] = dl * __builtin_amdgcn_exp2f(-LFg[(size_t)bh * npad + i]);
    if (rho != nullptr && lane < d) rho[row * d + lane] = -dl * y1;
}

}  // namespace

bool mfma_forward_f32_supported(int d, bool causal) { (void)causal; return d == FD; }

size_t mfma_forward_f32_workspace_bytes(int B, int H, int n) { return make_f32_layout(B, H, n).total; }

// call: the caller's own tensors, at d = 16 / 32 with p's Q and K copies of them in rows of 64 features (see llla_pad.hip)
hipError_t mfma_forward_f32(const Problem &p, const Problem &call)
{
    using S = Shape<FD>;
    const F32Layout L = make_f32_layout(p.B, p.H, p.n);
    char *ws = static_cast<char *>(p.ws);
    float *M = reinterpret_cast<float *>(ws + L.m), *LF = reinterpret_cast<float *>(ws + L.lf);
    float *Y = reinterpret_cast<float *>(ws + L.y);
    const int bh = p.B * p.H;
    const float *Q = static_cast<const float *>(p.Q), *K = static_cast<const float *>(p.K);
    stage_mark(p.stream, "moments");
    const int live = p.live_d > 0 ? (p.live_d + 15) / 16 : 4;      // a d = 16 / 32 call on zero-padded copies: 1 or 2
    dual::DualArgs da = dual::dual_args(call);
    da.nrows = dual_forward_rows(p);                               // up to 64 keys at every head dimension
    const int nqb = (p.n + S::QB - 1) / S::QB, obf = p.out == LLLA_BF16 ? 1 : 0;
    const int own = nqb - (da.nrows + S::QB - 1) / S::QB, parts = (da.nrows + 3) / 4;
    const dim3 grid(own + parts, bh);
    const BlockOrder order = block_order(live, bh, own, parts);
    if (live == 1)
        hipLaunchKernelGGL(moments_f32_kernel<1>, grid, dim3(256), 0, p.stream, Q, K, p.sq, p.sk, p.H, p.n, L.npad,
                           p.scale * LOG2E, p.lambda, p.lambda_rows, M, LF, Y, nullptr, p.causal, nqb, da, order.rows_at, order.mixed, obf);
    else if (live == 2)
        hipLaunchKernelGGL(moments_f32_kernel<2>, grid, dim3(256), 0, p.stream, Q, K, p.sq, p.sk, p.H, p.n, L.npad,
                           p.scale * LOG2E, p.lambda, p.lambda_rows, M, LF, Y, nullptr, p.causal, nqb, da, order.rows_at, order.mixed, obf);
    else
        hipLaunchKernelGGL(moments_f32_kernel<4>, grid, dim3(256), 0, p.stream, Q, K, p.sq, p.sk, p.H, p.n, L.npad,
                           p.scale * LOG2E, p.lambda, p.lambda_rows, M, LF, Y, nullptr, p.causal, nqb, da, order.rows_at, order.mixed, obf);
    if (p.rho != nullptr || p.delta != nullptr) {
        stage_mark(p.stream, "statistics");
        hipLaunchKernelGGL(stats_f32_kernel, dim3((p.n + 3) / 4, bh), dim3(256), 0, p.stream, Q, p.sq, p.H, p.n, L.npad,
                           (const float *)Y, (const float *)LF, p.rho, p.delta, call.d, da.nrows);
    }
    stage_mark(p.stream, "output");
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : mfma_output_f32(call, L.npad, M, Y, da.nrows);
}

hipError_t mfma_moments_f32_given(const BackwardProblem &p, int npad, float *M, float *Y, float *RU)
{
    const float *Q = static_cast<const float *>(p.Q), *K = static_cast<const float *>(p.K);
    const int nqb = (p.n + Shape<FD>::QB - 1) / Shape<FD>::QB;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nqb, p.B * p.H), dim3(256), 0, p.stream, Q, K, p.sq, p.sk, p.H, p.n, npad, p.scale * LOG2E,
                           p.lambda, p.lambda_rows, M, nullptr, Y, RU, 1, nqb, dual::DualArgs{}, 0, 0, 0);
    };
    if (p.live_d == 16) launch(moments_f32_kernel<1, true>);
    else if (p.live_d == 32) launch(moments_f32_kernel<2, true>);
    else launch(moments_f32_kernel<4, true>);
    return hipGetLastError();
}

}  // namespace llla
