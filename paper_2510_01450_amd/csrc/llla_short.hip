// Forward of short sequences with fp32 inputs at d = 16 / 32: one wave per query row, no barrier.
//
// What bounds such a call is latency: the vector kernels serve 16 rows and more per workgroup in chains of barriers over key tiles,
// twice, and eliminate in LDS; a row by itself is a few thousand cycles.  Here lane l owns keys l, l + 64, .. of the row (logits, weights
// and output weights); the moments go through v_mfma_f32_16x16x4_f32 with the key as contraction index, lane (g, n) holding feature n of
// key 4 c + g; the system is solved by the wave as in the fp32 matrix-core forward: the intercept eliminated first, pivots that are noise
// dropped (llla_mfma_fwd_f32.hip).  Rows that see at most d keys are served in key space by further workgroups (dual_row).
// 1 head x 128 rows at d = 16: 24 us (the vector kernel alone) -> 8.1 on the GPU, which is what such calls take one after the other.
#include "llla_decode_tail.hpp"

namespace llla {
namespace {

using namespace mfma;

constexpr int SHORT_ROWS = 256;                           // longest sequence: four keys per lane

template <int D>
struct ShortWave {
    float w[SHORT_ROWS];                                  // weights, then output weights
    float v[2 * D];                                       // mu~, then y1
    float sc[16 * SC_PITCH];
};

template <int D, typename TO>
__global__ __launch_bounds__(256, 2) void short_rows_kernel(dual::DualArgs a, int skip)
{
    constexpr int NB = D / 16, NT = NB * (NB + 1) / 2, KPL = SHORT_ROWS / 64;
    __shared__ __align__(16) union Shared {
        ShortWave<D> wave[4];
        dual::DualShared<D> row;
        __device__ Shared() {}
    } sm;
    const int bh = blockIdx.y;
    if ((int)blockIdx.x < skip) {                         // key-space rows, the longest first
        dual::dual_forward_row<D, float, TO>(sm.row, a, bh, skip - 1 - (int)blockIdx.x);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, g = lane / 16, nn = lane % 16;
    const int i = a.n - 1 - (4 * ((int)blockIdx.x - skip) + wave);      // long rows first
    if (i < skip) return;                                 // (no barrier below)
    const int m = a.causal ? i + 1 : a.n;                 // keys that the row sees
    const int b = bh / a.H, h = bh % a.H;
    const float *Kh = (const float *)a.K + b * a.sk.batch + h * a.sk.head, *Vh = (const float *)a.V + b * a.sv.batch + h * a.sv.head;
    const float *qrow = (const float *)a.Q + b * a.sq.batch + h * a.sq.head + (int64_t)i * a.sq.seq;
    auto &lw = sm.wave[wave].w;
    auto &lv = sm.wave[wave].v;
    const size_t row = (size_t)bh * a.n + i;
    const float lam = a.lam_rows ? a.lam_rows[row] : a.lambda;

    // ---- logits, weights: lane l, keys l + 64 t -------------------------------------------------------------------
    f32x4 q[D / 4], k[KPL][D / 4];
#pragma unroll
    for (int c = 0; c < D / 4; ++c) q[c] = *reinterpret_cast<const f32x4 *>(qrow + 4 * c);
#pragma unroll
    for (int t = 0; t < KPL; ++t)
        if (64 * t < m) {                                 // (scalar branches: m is uniform)
            const float *kr = Kh + (int64_t)min(lane + 64 * t, m - 1) * a.sk.seq;
#pragma unroll
            for (int c = 0; c < D / 4; ++c) k[t][c] = *reinterpret_cast<const f32x4 *>(kr + 4 * c);
        }
    float s[KPL], top = -INFINITY;
#pragma unroll
    for (int t = 0; t < KPL; ++t) {
        s[t] = -INFINITY;
        if (64 * t < m) {
            float p = 0.f;
#pragma unroll
            for (int c = 0; c < D / 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) p = fmaf(q[c][e], k[t][c][e], p);
            if (lane + 64 * t < m) s[t] = p * (a.scale * LOG2E);
        }
        top = fmaxf(top, s[t]);
    }
    top = wave_max_dpp(top);
    float om = 0.f;
#pragma unroll
    for (int t = 0; t < KPL; ++t)
        if (64 * t < m) {
            s[t] = __builtin_amdgcn_exp2f(s[t] - top);    // exp2(-inf) = 0 beyond the row
            om += s[t];
            lw[lane + 64 * t] = s[t];
        }
    om = rows_allsum(row_allsum(om));
    wave_sync();

    // ---- moments: T = -Sigma~ in tiles, mu~ ----------------------------------------------------------------------------
    // Four sums of every fourth chunk: this MFMA rounds at each of its four keys, and in one chain over the row the errors of rho and O were
    // up to 1.05 times the vector kernels' (rows of 17 to 256 unit and normal keys, d = 16 / 32); of four sums they are 0.76 to 0.9 times,
    // and a row takes as long as before.
    constexpr int CB = 8, CA = 4;                         // chunks of four keys whose loads are in flight together; sums
    f32x4 part[CA][NT], acc[NT];
    float mu[NB];
#pragma unroll
    for (int c = 0; c < CA; ++c)
#pragma unroll
        for (int t = 0; t < NT; ++t) part[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int I = 0; I < NB; ++I) mu[I] = 0.f;
    for (int c0 = 0; c0 < m; c0 += 4 * CB) {
        float kx[CB][NB], wx[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int j = c0 + 4 * c + g, jc = min(j, m - 1);
            wx[c] = lw[jc];
            wx[c] = j < m ? -wx[c] : 0.f;
#pragma unroll
            for (int J = 0; J < NB; ++J) kx[c][J] = Kh[(int64_t)jc * a.sk.seq + 16 * J + nn];
        }
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int I = 0; I < NB; ++I) {
                const float wk = wx[c] * kx[c][I];
                mu[I] -= wk;
#pragma unroll
                for (int J = I; J < NB; ++J)
                    part[c % CA][upper_tile<NB>(I, J)] =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(wk, kx[c][J], part[c % CA][upper_tile<NB>(I, J)], 0, 0, 0);
            }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]);
    // ---- the intercept eliminated, the ridge, the solve -----------------------------------------------------------------
    const float oinv = 1.f / om;
#pragma unroll
    for (int I = 0; I < NB; ++I) {
        mu[I] = rows_allsum(mu[I]);
        if (g == 0) lv[16 * I + nn] = mu[I];
    }
    wave_sync();
    f32x4 mr[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) mr[I] = *reinterpret_cast<const f32x4 *>(&lv[16 * I + 4 * g]);
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = I; J < NB; ++J)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float x = fmaf(oinv * mr[I][t], mu[J], acc[upper_tile<NB>(I, J)][t]);
                if (I == J) x -= (nn == 4 * g + t) ? lam : 0.f;
                acc[upper_tile<NB>(I, J)][t] = x;
            }
    float qn[NB];
#pragma unroll
    for (int P = 0; P < NB; ++P) qn[P] = qrow[16 * P + nn];
    f32x4 y1[NB];
    float one;
    solve_one<NB, false, true>(acc, y1, one, 1.f, sm.wave[wave].sc, g, nn, 0.5f * lam, [&](int P, float &mm, float &qq, float &) {
        mm = 0.f;
        qq = fmaf(mu[P], oinv, -qn[P]);                   // -(q - mu~ / omega)
    });
    if (nn == 0) {
#pragma unroll
        for (int P = 0; P < NB; ++P) *reinterpret_cast<f32x4 *>(&lv[D + 16 * P + 4 * g]) = y1[P];
    }
    wave_sync();

    // ---- output weights w (1 / omega + (k - mu~ / omega) . y1), the same as w (y0 + k . y1) ---------------------------------
    f32x4 y[D / 4];
    float my = 0.f, qy = 0.f;
#pragma unroll
    for (int c = 0; c < D / 4; ++c) {
        y[c] = *reinterpret_cast<const f32x4 *>(&lv[D + 4 * c]);
        const f32x4 mc = *reinterpret_cast<const f32x4 *>(&lv[4 * c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            my = fmaf(mc[e], y[c][e], my);
            qy = fmaf(q[c][e], y[c][e], qy);
        }
    }
    const float y0 = (1.f - my) * oinv;
#pragma unroll
    for (int t = 0; t < KPL; ++t)
        if (64 * t < m) {
            float p = y0;
#pragma unroll
            for (int c = 0; c < D / 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) p = fmaf(k[t][c][e], y[c][e], p);
            lw[lane + 64 * t] = s[t] * p;
        }
    wave_sync();
    float o[NB];
#pragma unroll
    for (int J = 0; J < NB; ++J) o[J] = 0.f;
    for (int c0 = 0; c0 < m; c0 += 4 * CB) {
        float vx[CB][NB], wx[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int j = c0 + 4 * c + g, jc = min(j, m - 1);
            wx[c] = lw[jc];
            wx[c] = j < m ? wx[c] : 0.f;
#pragma unroll
            for (int J = 0; J < NB; ++J) vx[c][J] = Vh[(int64_t)jc * a.sv.seq + 16 * J + nn];
        }
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int J = 0; J < NB; ++J) o[J] = fmaf(wx[c], vx[c][J], o[J]);
    }
    TO *orow = (TO *)a.O + b * a.so.batch + h * a.so.head + (int64_t)i * a.so.seq;
#pragma unroll
    for (int J = 0; J < NB; ++J) {
        o[J] = rows_allsum(o[J]);
        if (g == 0) dual::st_out(orow + 16 * J + nn, (double)o[J]);
    }
    if (a.Rho != nullptr || a.Delta != nullptr) {
        const float dl = 1.f / (y0 + qy);                 // y0 = (1 + q.rho) / delta, y1 = -rho / delta
        if (a.Delta != nullptr && lane == 0) a.Delta[row] = dl;
        if (a.Rho != nullptr && lane < D) a.Rho[row * D + lane] = -dl * lv[D + lane];
    }
}

template <int D>
hipError_t launch(const Problem &p)
{
    const dual::DualArgs a = dual::dual_args(p);
    const int skip = a.nrows;
    const dim3 grid(skip + (p.n - skip + 3) / 4, p.B * p.H);
    if (p.out == LLLA_F32) hipLaunchKernelGGL((short_rows_kernel<D, float>), grid, dim3(256), 0, p.stream, a, skip);
    else hipLaunchKernelGGL((short_rows_kernel<D, bf16_t>), grid, dim3(256), 0, p.stream, a, skip);
    return hipGetLastError();
}

}  // namespace

// A row per wave is the shorter chain, not the less work: it pays while the rows fit the GPU about once (us, vector kernels / here: d = 16,
// 1 head x 256 43 / 16, 16 x 256 44 / 24, 32 x 128 25 / 18, 64 x 64 16 / 18, 64 x 256 45 / 62; d = 32, 1 x 256 42 / 20, 8 x 128 26 / 18, 8 x 256
// 43 / 36, 16 x 64 18 / 24, 16 x 128 26 / 31, where the key-space rows' workgroups find only two places per compute unit).
bool short_forward_takes(int heads, int n, int d, llla_dtype in)
{
    if (in != LLLA_F32 || n > SHORT_ROWS) return false;
    return d == 16 ? heads <= 32 && heads * n <= 4096 : d == 32 && heads <= 8;
}

hipError_t short_forward(const Problem &p)
{
    if (dual_forward_rows(p) >= p.n) return dual_forward(p);
    return p.d == 16 ? launch<16>(p) : launch<32>(p);
}

}  // namespace llla
