// Matrix-core forward path for fp32 inputs, d = 128, and the moments of its backward pass: the method of llla_mfma_fwd_f32.hip (logits on
// fp32 MFMA, the second moment from z_j = sqrt(w_ij) k_j in three bf16 on 16-bit MFMA, a reference exponent that moves lazily, the
// intercept eliminated first, pivots that are noise dropped), in the shape of the bf16 kernel for d = 128: one query per wave, 36 tiles
// = 144 accumulator registers, eight waves per workgroup.
//
// Split.  z of all eight 16-feature blocks would be 96 registers beside the tiles.  Blocks 0..3 stay while 4..7 pass by one at a time, then
// blocks 4..7 stay: eleven blocks are scaled and split per 32 keys instead of eight, 36 vector instructions each beside 200 MFMAs.  A wave
// needs the weights of its own query only: lane j of it is key j of the block, so the maximum, the reference exponent and the weights
// never leave the wave.  The logits of the eight queries are one 16-column tile product, its contraction split over the two halves
// of the workgroup.  mu~ is summed on the vector ALU from the same sqrt(w) k.
//
// What bounds it: MFMA and splitting as at d = 64, and for short sequences the per-row solve and the chain of the key-space rows (74 us).
// us a call, vector kernels (which served d = 128 before) and these.  Forward: 8 heads x 65 rows 349 and 84, 8 x 250 1190 and 98, 64 x 700
// 37900 and 2345; backward: 1 x 64 396 and 83, 8 x 250 3256 and 189, 32 x 700 43800 and 1510.  Errors of O against fp64, 140 and 300 rows, times
// those of the vector kernels: unit keys 0.67-0.68, normal keys 0.72-0.75 with ridges from 10^-2 to 10^-4, 0.70 times 10, 0.37 plus 3.
#include "llla_dual.hpp"
#include "llla_mfma_common.hpp"
#include "llla_mfma_solve128.hpp"

namespace llla {
namespace {

using namespace mfma;

constexpr int WD = 128;                // head dimension
constexpr int WKB = 64;                // keys per block
constexpr int WNB = WD / 16;           // feature blocks
constexpr int WNT = 512;               // threads: eight waves, one query each
constexpr int WQB = 8;
constexpr int WYP = WD + 16;           // pitch of a y row
constexpr float LAZY_BITS = 64.f;      // the reference exponent moves when a block exceeds it by more than this

struct WideLayout {
    size_t m, lf, y, total;
    int npad;
};

WideLayout make_wide_layout(int B, int H, int n)
{
    WideLayout L;
    L.npad = (n + WKB - 1) / WKB * WKB;
    const size_t bh = (size_t)B * H;
    size_t off = 0;
    L.m = off;  off += round_up(bh * L.npad * 4, 256);               // reference exponent mh (log2 units)
    L.lf = off; off += round_up(bh * L.npad * 4, 256);               // log2 F = m - mh
    L.y = off;  off += round_up(bh * (size_t)n * WYP * 4, 256);      // y' rows
    L.total = off;
    return L;
}

// 16-byte chunk c of key row r sits at c ^ swz(r): both operand reads are free of bank conflicts (see llla_mfma_fwd_f32.hip)
__device__ inline int swz(int r) { return ((r & 1) << 2) | ((r >> 1) & 3); }

struct WideShared {
    float kt[2][WKB * WD];
    float pz[2][WQB][WKB + 4];         // partial logits: [half of the features][query][key]
    float qs[WQB][WD + 4];
    float wt[WQB][WKB];                // roots of the weights, each row its wave's own: [(key % 4) * 16 + key / 4]
    float sc[WQB][16 * SC_PITCH];
    float mus[WQB][WD];
};

template <int N, int V>
__device__ __forceinline__ void alternate()      // schedule: N times one MFMA, then V vector instructions
{
    if constexpr (N > 0) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
        alternate<N - 1, V>();
    }
}

struct Split3 {
    bf16x8 h, m, l;
};

// six products of the nine (the rest is below 2^-24 of the result); in a diagonal tile h^T m and m^T h (h^T l and l^T h) are each other's
// transposes and the solve symmetrises: (2 h)^T m and (2 h)^T l serve
__device__ __forceinline__ void tile_product(f32x4 &t, const Split3 &a, const Split3 &b)
{
    t = mfma_bf16(a.l, b.h, t);
    t = mfma_bf16(a.h, b.l, t);
    t = mfma_bf16(a.m, b.m, t);
    t = mfma_bf16(a.m, b.h, t);
    t = mfma_bf16(a.h, b.m, t);
    t = mfma_bf16(a.h, b.h, t);
}
__device__ __forceinline__ void diagonal_product(f32x4 &t, const Split3 &a)
{
    const bf16x8 h2 = twice_bf16(a.h);
    t = mfma_bf16(h2, a.l, t);
    t = mfma_bf16(a.m, a.m, t);
    t = mfma_bf16(h2, a.m, t);
    t = mfma_bf16(a.h, a.h, t);
}

// BWD: Mg holds the row maxima already, RUg r1 and r0 of every row (pitch WYP, r0 at [WD]), which u1 and u0 replace; as in
// moments_f32_kernel.  Rows [0, da.nrows), a multiple of 8 or all, are the key-space workgroups', eight each.
template <bool BWD>
__global__ __launch_bounds__(WNT, 1) void moments_f32_wide_kernel(
    const float *__restrict__ Qg, const float *__restrict__ Kg, llla_strides sq, llla_strides sk, int H, int n, int npad, float cscale,
    float lambda, const float *__restrict__ lam_rows, float *__restrict__ Mg, float *__restrict__ LFg, float *__restrict__ Yg,
    float *__restrict__ RUg, int causal, int nqb, dual::DualArgs da, int out_bf16)
{
    __shared__ __align__(16) WideShared sm;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64, g = lane / 16, nn = lane % 16;
    const int own = BWD ? nqb : nqb - (da.nrows + WQB - 1) / WQB;      // blocks of a head here
    const int lin = linear_block();
    if constexpr (!BWD) {
        const int at = lin - own * (int)gridDim.y;         // behind the blocks of all heads (us so / behind their own head's: 16 x 500 364 / 375)
        if (at >= 0) {
            const int bh = (int)((unsigned)at % gridDim.y), part = (int)((unsigned)at / gridDim.y);
            using DS = dual::DualSharedRows<WD, WQB>;
            static_assert(sizeof(DS) <= sizeof(WideShared), "key-space rows fit the workgroup's LDS");
            auto &ds = *reinterpret_cast<DS *>(&sm);
            const int top = da.nrows - 1 - WQB * part;
            if (out_bf16) dual::dual_forward_rows<WD, WQB, bf16_t>(ds, da, bh, top);
            else dual::dual_forward_rows<WD, WQB, float>(ds, da, bh, top);
            return;
        }
    }
    const BlockMap bm = xcd_block_map(lin, own, (int)gridDim.y);
    const int bh = bm.bh, b = bh / H, h = bh % H;
    const int i0 = (nqb - 1 - bm.blk) * WQB;                           // long rows first
    const int ilast = min(i0 + WQB - 1, n - 1);
    const int nblk = causal ? ilast / WKB + 1 : (n + WKB - 1) / WKB;
    const float *Kh = Kg + b * sk.batch + h * sk.head;
    const float *Qh = Qg + b * sq.batch + h * sq.head;
    const int iq = min(i0 + wave, n - 1);                              // this wave's query; past the end the last one again, not stored
    const int jlim = causal ? iq : n - 1;                              // last key it sees
    {
        const int qr = tid >> 6, qc = 2 * (tid & 63);
        const float *qp = Qh + (int64_t)min(i0 + qr, n - 1) * sq.seq + qc;
        sm.qs[qr][qc] = qp[0];
        sm.qs[qr][qc + 1] = qp[1];
    }

    constexpr int NTILE = WNB * (WNB + 1) / 2;
    f32x4 acc[NTILE];
#pragma unroll
    for (int t = 0; t < NTILE; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mu[WNB];                             // this lane's share (keys of its lane group) of mu~'[16 I + nn]
#pragma unroll
    for (int I = 0; I < WNB; ++I) mu[I] = 0.f;
    float om = 0.f;                            // and of omega' (keys = lane mod 64)
    float mh = -INFINITY, mtrue = -INFINITY;   // reference exponent and true maximum (log2 units), uniform in the wave
    if constexpr (BWD) mh = Mg[(size_t)bh * npad + iq];

    // DMA of one K block: 32 wave transfers of 1 KB = two key rows, four per wave
    auto issue_dma = [&](int blk) {
        float *dst = sm.kt[blk & 1];
        int lane_e = lane;
        asm volatile("" : "+v"(lane_e));       // (nothing address-like stays live over the sweep)
        const bool whole = blk * WKB + WKB <= n && sk.seq < (int64_t(1) << 23);      // byte offsets fit 32 bits
        const float *base = Kh + (int64_t)blk * WKB * sk.seq;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int row = 8 * wave + 2 * t + (lane_e >> 5), chunk = (lane_e & 31) ^ swz(row);
            float *to = dst + (8 * wave + 2 * t) * WD;
            if (whole) dma16_base(base, (unsigned)(row * (int)sk.seq + 4 * chunk) * 4u, to);
            else dma16(Kh + (int64_t)min(blk * WKB + row, n - 1) * sk.seq + 4 * chunk, to);
        }
    };

    issue_dma(0);
    __builtin_amdgcn_s_setprio(2);
    for (int c = 0; c < nblk; ++c) {
        const float *kt = sm.kt[c & 1];
        dma_wait();
        __syncthreads();                       // tile c complete; everybody is done with block c - 1
        // ---- logits: 16 keys x 8 queries (columns 8..15 repeat them) over half of the features; slot (s, g) <-> feature 64 half + 16 g + s
        {
            const int half = wave >> 2, kw = 16 * (wave & 3), row = kw + nn, sw = swz(row);
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const f32x4 kv = *reinterpret_cast<const f32x4 *>(kt + row * WD + 4 * ((16 * half + 4 * g + v) ^ sw));
                const f32x4 qv = *reinterpret_cast<const f32x4 *>(&sm.qs[nn & 7][64 * half + 16 * g + 4 * v]);
#pragma unroll
                for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[e], qv[e], z, 0, 0, 0);
            }
            if (nn < 8) *reinterpret_cast<f32x4 *>(&sm.pz[half][nn][kw + 4 * g]) = z;
        }
        __syncthreads();                       // logits visible (and the other tile's buffer is free since the barrier before)
        if (c + 1 < nblk) issue_dma(c + 1);
        // ---- weights of this wave's query: lane = key ----
        {
            const float zs = (sm.pz[0][wave][lane] + sm.pz[1][wave][lane]) * cscale;
            const bool seen = c * WKB + lane <= jlim;
            if constexpr (!BWD) {
                float bmx = seen ? zs : -INFINITY;
#pragma unroll
                for (int off = 1; off <= 32; off <<= 1) bmx = fmaxf(bmx, __shfl_xor(bmx, off));
                bmx = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, bmx)));
                mtrue = fmaxf(mtrue, bmx);
                if (bmx > mh + LAZY_BITS || (mh == -INFINITY && bmx > -INFINITY)) {       // uniform: the reference moves (first block: always)
                    const float rsc = (mh == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mh - bmx);
                    mh = bmx;
                    om *= rsc;
#pragma unroll
                    for (int I = 0; I < WNB; ++I) mu[I] *= rsc;
#pragma unroll
                    for (int t = 0; t < NTILE; ++t) acc[t] *= rsc;
                }
            }
            const float root = __builtin_amdgcn_exp2f(0.5f * (zs - mh));
            const float sw = seen ? root : 0.f;
            sm.wt[wave][(lane & 3) * 16 + (lane >> 2)] = sw;
            om = fmaf(sw, sw, om);
        }
        wave_sync();

        // ---- moments, in halves of 32 keys, up to the last key a query of the workgroup sees ----
        const int nhalf = causal ? min(2, (ilast - c * WKB) / 32 + 1) : 2;
#pragma unroll 1
        for (int hf = 0; hf < nhalf; ++hf) {
            // key 4 (8 hf + t) + g is slot t of lane group g; four addresses per lane and immediates serve all reads (see moments_f32_kernel)
            int g_e = g, nn_e = nn;
            asm volatile("" : "+v"(g_e), "+v"(nn_e));
            const int c4 = nn_e >> 2;
            const float *krow = kt + (32 * hf + g_e) * WD + (nn_e & 3);
            const float *ka[2][2];
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int ip = 0; ip < 2; ++ip) ka[tp][ip] = krow + 4 * (4 * (ip ^ (g_e & 1)) + (c4 ^ ((2 * tp + (g_e >> 1)) & 3)));
            const float *wp = &sm.wt[wave][g_e * 16 + 8 * hf];
            const f32x4 w0 = *reinterpret_cast<const f32x4 *>(wp), w1 = *reinterpret_cast<const f32x4 *>(wp + 4);
            auto make = [&](int I, bool first) {
                asm volatile("" ::: "memory");         // (keys are read again rather than kept)
                float x[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float sw = t < 4 ? w0[t & 3] : w1[t & 3], v = sw * ka[t & 1][I & 1][4 * t * WD + 32 * (I >> 1)];
                    x[t] = sw == 0.f ? 0.f : v;        // a key that the row does not see need not be finite
                }
                if (first) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) mu[I] = fmaf(t < 4 ? w0[t & 3] : w1[t & 3], x[t], mu[I]);
                }
                Split3 s;
                split3_bf16(x, s.h, s.m, s.l);
                return s;
            };
            Split3 z[4], p, next;
            z[0] = make(0, true);
#pragma unroll
            for (int I = 0; I < 4; ++I) {              // the triangle of blocks 0..3
                next = make(I < 3 ? I + 1 : 7, true);
#pragma unroll
                for (int J = 0; J < I; ++J) tile_product(acc[upper_tile<WNB>(J, I)], z[J], z[I]);
                diagonal_product(acc[upper_tile<WNB>(I, I)], z[I]);
                __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
                if (I == 0) alternate<4, 12>();
                else if (I == 1) alternate<10, 5>();
                else if (I == 2) alternate<16, 3>();
                else alternate<22, 2>();
                __builtin_amdgcn_sched_barrier(0);
                if (I < 3) z[I + 1] = next;
            }
            p = next;
#pragma unroll
            for (int I = 7; I >= 4; --I) {             // blocks 7..4 against 0..3
                if (I > 4) next = make(I - 1, true);
#pragma unroll
                for (int J = 0; J < 4; ++J) tile_product(acc[upper_tile<WNB>(J, I)], z[J], p);
                __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
                alternate<24, 2>();
                __builtin_amdgcn_sched_barrier(0);
                if (I > 4) p = next;
            }
            z[0] = p;
#pragma unroll
            for (int I = 0; I < 4; ++I) {              // the triangle of blocks 4..7
                if (I < 3) next = make(I + 5, false);
#pragma unroll
                for (int J = 0; J < I; ++J) tile_product(acc[upper_tile<WNB>(J + 4, I + 4)], z[J], z[I]);
                diagonal_product(acc[upper_tile<WNB>(I + 4, I + 4)], z[I]);
                __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
                if (I == 0) alternate<4, 10>();
                else if (I == 1) alternate<10, 4>();
                else alternate<16, 3>();
                __builtin_amdgcn_sched_barrier(0);
                if (I < 3) z[I + 1] = next;
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);

    // ---- the ridge lambda F, the intercept, the solve: this wave's query alone ----
    int lane_f = lane;
    asm volatile("" : "+v"(lane_f));
    const int gf = lane_f >> 4, nf = lane_f & 15;
    float *mus = sm.mus[wave], *scw = sm.sc[wave];
#pragma unroll
    for (int off = 1; off <= 32; off <<= 1) om += __shfl_xor(om, off);
    const float oinv = 1.f / om, lf = BWD ? 0.f : mtrue - mh;
    const float lam = (lam_rows ? lam_rows[(size_t)bh * n + iq] : lambda) * __builtin_amdgcn_exp2f(lf);
#pragma unroll
    for (int I = 0; I < WNB; ++I) {
        mu[I] = rows_allsum(mu[I]);
        if (gf == 0) mus[16 * I + nf] = mu[I];
    }
    wave_sync();
#pragma unroll
    for (int I = 0; I < WNB; ++I) {                                    // T = -(Sigma~' - mu~ mu~^T / omega + lambda F I)
        const f32x4 mr = oinv * *reinterpret_cast<const f32x4 *>(mus + 16 * I + 4 * gf);
#pragma unroll
        for (int J = I; J < WNB; ++J) {
            f32x4 &t = acc[upper_tile<WNB>(I, J)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                t[r] = fmaf(mr[r], mu[J], -t[r]);
                if (I == J) t[r] -= (nf == 4 * gf + r) ? lam : 0.f;
            }
        }
    }
    factorise_one<WNB, false, true>(acc, scw, gf, nf, 0.5f * lam);
    constexpr int NV = BWD ? 2 : 1;
    float tv[NV][WNB], r0 = 0.f;
    const float *qrow = Qh + (int64_t)iq * sq.seq;
    const float *rr = BWD ? RUg + ((size_t)bh * n + iq) * WYP : nullptr;
    if constexpr (BWD) r0 = rr[WD];
#pragma unroll
    for (int P = 0; P < WNB; ++P) {
        const float m = mus[16 * P + nf];
        tv[0][P] = fmaf(m, oinv, -qrow[16 * P + nf]);                  // -(q - mu~ / omega)
        if constexpr (BWD) tv[1][P] = fmaf(m, r0 * oinv, -rr[16 * P + nf]);
    }
    substitute_forward<WNB, NV>(acc, tv, scw, gf, nf);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int P = 0; P < WNB; ++P) tv[v][P] = -tv[v][P];
    f32x4 rhs[WNB];
    substitute_back<WNB, NV>(acc, tv, rhs, scw, gf, nf);              // register t = y1[16 P + 4 g + t]; BWD, lanes n == 1: u1
    float dot = 0.f;
#pragma unroll
    for (int P = 0; P < WNB; ++P) {
        const f32x4 m = *reinterpret_cast<const f32x4 *>(mus + 16 * P + 4 * gf);
#pragma unroll
        for (int r = 0; r < 4; ++r) dot = fmaf(m[r], rhs[P][r], dot);
    }
    dot = rows_allsum(dot);
    if (i0 + wave < n) {
        const size_t row = (size_t)bh * n + iq;
        if (nf == 0) {
            float *yr = Yg + row * WYP;
#pragma unroll
            for (int P = 0; P < WNB; ++P) *reinterpret_cast<f32x4 *>(yr + 16 * P + 4 * gf) = rhs[P];
            if (gf == 0) {
                yr[WD] = (1.f - dot) * oinv;
                if (!BWD) {
                    Mg[(size_t)bh * npad + iq] = mh;
                    LFg[(size_t)bh * npad + iq] = lf;
                }
            }
        }
        if (BWD && nf == 1) {
            float *ur = RUg + row * WYP;
#pragma unroll
            for (int P = 0; P < WNB; ++P) *reinterpret_cast<f32x4 *>(ur + 16 * P + 4 * gf) = rhs[P];
            if (gf == 0) ur[WD] = (r0 - dot) * oinv;
        }
    }
}

// Statistics of Eq. (lla) from y' and F (see stats_f32_kernel).  One wave per row.
__global__ __launch_bounds__(256) void stats_f32_wide_kernel(const float *__restrict__ Qg, llla_strides sq, int H, int n, int npad,
                                                             const float *__restrict__ Yg, const float *__restrict__ LFg,
                                                             float *__restrict__ rho, float *__restrict__ delta, int skip)
{
    const int lane = threadIdx.x % 64, i = blockIdx.x * 4 + threadIdx.x / 64, bh = blockIdx.y;
    if (i >= n || i < skip) return;
    const float *qrow = Qg + (bh / H) * sq.batch + (bh % H) * sq.head + (int64_t)i * sq.seq;
    const float *yr = Yg + ((size_t)bh * n + i) * WYP;
    const float y0 = yr[lane], y1 = yr[lane + 64];
    float qy = fmaf(qrow[lane], y0, qrow[lane + 64] * y1);
#pragma unroll
    for (int sft = 32; sft >= 1; sft >>= 1) qy += __shfl_xor(qy, sft);
    const float dl = 1.f / (yr[WD] + qy);                                 // delta'
    const size_t row = (size_t)bh * n + i;
    if (delta != nullptr && lane == 0) delta[row] = dl * __builtin_amdgcn_exp2f(-LFg[(size_t)bh * npad + i]);
    if (rho != nullptr) {
        rho[row * WD + lane] = -dl * y0;
        rho[row * WD + lane + 64] = -dl * y1;
    }
}

}  // namespace

size_t mfma_forward_f32_wide_workspace_bytes(int B, int H, int n) { return make_wide_layout(B, H, n).total; }

hipError_t mfma_forward_f32_wide(const Problem &p)
{
    const WideLayout L = make_wide_layout(p.B, p.H, p.n);
    char *ws = static_cast<char *>(p.ws);
    float *M = reinterpret_cast<float *>(ws + L.m), *LF = reinterpret_cast<float *>(ws + L.lf), *Y = reinterpret_cast<float *>(ws + L.y);
    const int bh = p.B * p.H;
    const float *Q = static_cast<const float *>(p.Q), *K = static_cast<const float *>(p.K);
    const dual::DualArgs da = dual::dual_args(p);
    const int nqb = (p.n + WQB - 1) / WQB;          // (key-space rows: a workgroup serves as many as one of the others)
    stage_mark(p.stream, "moments");
    hipLaunchKernelGGL(moments_f32_wide_kernel<false>, dim3(nqb, bh), dim3(WNT), 0, p.stream, Q, K, p.sq, p.sk, p.H, p.n, L.npad,
                       p.scale * LOG2E, p.lambda, p.lambda_rows, M, LF, Y, nullptr, p.causal, nqb, da, p.out == LLLA_BF16 ? 1 : 0);
    if (p.rho != nullptr || p.delta != nullptr) {
        stage_mark(p.stream, "statistics");
        hipLaunchKernelGGL(stats_f32_wide_kernel, dim3((p.n + 3) / 4, bh), dim3(256), 0, p.stream, Q, p.sq, p.H, p.n, L.npad,
                           (const float *)Y, (const float *)LF, p.rho, p.delta, da.nrows);
    }
    stage_mark(p.stream, "output");
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : mfma_output_f32(p, L.npad, M, Y, da.nrows);
}

hipError_t mfma_moments_f32_wide_given(const BackwardProblem &p, int npad, float *M, float *Y, float *RU)
{
    const int nqb = (p.n + WQB - 1) / WQB;
    hipLaunchKernelGGL(moments_f32_wide_kernel<true>, dim3(nqb, p.B * p.H), dim3(WNT), 0, p.stream, static_cast<const float *>(p.Q),
                       static_cast<const float *>(p.K), p.sq, p.sk, p.H, p.n, npad, p.scale * LOG2E, p.lambda, p.lambda_rows, M, nullptr,
                       Y, RU, 1, nqb, dual::DualArgs{}, 0);
    return hipGetLastError();
}

}  // namespace llla
