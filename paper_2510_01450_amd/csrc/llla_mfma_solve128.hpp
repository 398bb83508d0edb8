// Exact solve of ONE augmented system per wave (the moments kernel at head dimension 128, one query per wave; the decode
// tail at d = 128): the 16-blocked Cholesky factorisation (factorise_one) on the matrix cores, forward and back substitutions on the
// vector ALU.
//
// Why.  With one query per wave a substitution step is a 16x16 tile times two or three right-hand-side columns; as a
// 16x16x16 fp32 tile product it occupies the matrix cores for 128 cycles and uses two or three of sixteen output
// columns.  At d = 128 that is 88 of the 200 tile products of a row's solve, and with the eight waves of a workgroup
// solving at the same time the phase is bound by exactly those matrix-core cycles.  On the vector ALU the same step
// is four multiply-adds per lane and column:
//   * a tile stays in the accumulator layout: lane (g, n) holds X[4g+t][n] in register t;
//   * a vector block lives in one of two layouts: C, lane (g, n) holds element n (the same in every g), or R, lane
//     (g, n) holds elements 4g..4g+3 in four registers (the same in every n);
//   * X^T v (forward substitution: U^T a = b) takes v in R, multiplies per lane and sums over g (the four 16-lane rows of
//     the wave), which gives C;  X v (back substitution: U x = z) takes v in C, multiplies per lane and sums over n (the
//     16 lanes of a row), which gives R;
//   * C <-> R goes through the wave's scratch tile in LDS (16 floats per vector).
// The sign conventions are factorise_one's: tiles hold T = -(Sigma~ + lambda I) factorised as U^T U with acc(P,P) = N_P =
// -U(P,P)^{-1}, right-hand sides come in negated.
#pragma once

#include "llla_mfma_common.hpp"
#include "llla_mfma_solve64.hpp"      // row_allsum

namespace llla {
namespace mfma {

// sum of x over the four 16-lane rows of the wave (same lane position), in every row.  Row swaps on the vector ALU: through __shfl_xor, i.e.
// LDS, the sums were six LDS round trips of a block step's chain (inline assembly and its s_nop: see rows_transpose4).
__device__ inline float rows_allsum(float x)
{
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));       // rows 0 0 2 2 and 1 1 3 3
    a += b;
    b = a;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return a + b;
}
// the largest instead of the sum (a NaN is passed over)
__device__ inline float rows_allmax(float x)
{
    float a = x, b = x;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    a = fmaxf(a, b);
    b = a;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return fmaxf(a, b);
}

// C -> R and R -> C for NV vectors at once through the scratch tile (vector v at scw + 16 v)
template <int NV>
__device__ __forceinline__ void c_to_r(const float (&c)[NV], f32x4 (&r)[NV], float *scw, int g, int nn)
{
    if (g == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) scw[16 * v + nn] = c[v];
    }
    wave_sync();
#pragma unroll
    for (int v = 0; v < NV; ++v) r[v] = *reinterpret_cast<const f32x4 *>(scw + 16 * v + 4 * g);
    wave_sync();
}
template <int NV>
__device__ __forceinline__ void r_to_c(const f32x4 (&r)[NV], float (&c)[NV], float *scw, int g, int nn)
{
    if (nn == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) *reinterpret_cast<f32x4 *>(scw + 16 * v + 4 * g) = r[v];
    }
    wave_sync();
#pragma unroll
    for (int v = 0; v < NV; ++v) c[v] = scw[16 * v + nn];
    wave_sync();
}

// Forward substitution of NV right-hand sides after factorise_one.  tv[v][P], C layout: in, element 16P + n of -b; out, of
// U^{-T} b:  t_P = -b_P + sum_{I<P} U(I,P)^T a_I,  a_P = N_P^T t_P
template <int NB, int NV>
__device__ __forceinline__ void substitute_forward(const f32x4 (&acc)[NB * (NB + 1) / 2], float (&tv)[NV][NB], float *scw, int g, int nn)
{
    auto dot4 = [](const f32x4 &x, const f32x4 &v) { return fmaf(x[3], v[3], fmaf(x[2], v[2], fmaf(x[1], v[1], x[0] * v[0]))); };
    float part[NV][NB];                    // partial sums over this lane's g
#pragma unroll
    for (int P = 0; P < NB; ++P)
#pragma unroll
        for (int v = 0; v < NV; ++v) part[v][P] = 0.f;
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        float tc[NV];
        f32x4 tr[NV], ar[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) tc[v] = P == 0 ? tv[v][P] : tv[v][P] + rows_allsum(part[v][P]);
        c_to_r<NV>(tc, tr, scw, g, nn);
        const f32x4 np = acc[upper_tile<NB>(P, P)];
        float ac[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            ac[v] = rows_allsum(dot4(np, tr[v]));
            tv[v][P] = ac[v];
        }
        if (P + 1 < NB) {
            c_to_r<NV>(ac, ar, scw, g, nn);
#pragma unroll
            for (int I = P + 1; I < NB; ++I) {
                const f32x4 u = acc[upper_tile<NB>(P, I)];
#pragma unroll
                for (int v = 0; v < NV; ++v) part[v][I] += dot4(u, ar[v]);
            }
        }
    }
}

// Back substitution, block rows NB-1..0:  x_P = N_P (z_P + sum_{J>P} U(P,J) x_J), i.e. x = -U^{-1} z.  zc: C layout; rhs: R layout (NV = 2:
// lanes n == 1 hold the second solution)
template <int NB, int NV>
__device__ __forceinline__ void substitute_back(const f32x4 (&acc)[NB * (NB + 1) / 2], const float (&zc)[NV][NB], f32x4 (&rhs)[NB], float *scw,
                                                int g, int nn)
{
    float xc[NV][NB];                      // C layout
#pragma unroll
    for (int P = NB - 1; P >= 0; --P) {
        f32x4 ir[NV], xr[NV];
        float ic[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            // per lane: rows 4g+t of U(P,J) x_J restricted to column n, plus z_P on the diagonal positions
            f32x4 p;
#pragma unroll
            for (int t = 0; t < 4; ++t) p[t] = (nn == 4 * g + t) ? zc[v][P] : 0.f;
#pragma unroll
            for (int J = P + 1; J < NB; ++J) {
                const f32x4 u = acc[upper_tile<NB>(P, J)];
#pragma unroll
                for (int t = 0; t < 4; ++t) p[t] = fmaf(u[t], xc[v][J], p[t]);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) ir[v][t] = row_allsum(p[t]);
        }
        r_to_c<NV>(ir, ic, scw, g, nn);
        const f32x4 np = acc[upper_tile<NB>(P, P)];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int t = 0; t < 4; ++t) xr[v][t] = row_allsum(np[t] * ic[v]);
        rhs[P] = xr[0];
        if constexpr (NV == 2) rhs[P] = (nn == 1) ? xr[1] : xr[0];
        if (P > 0) {
            float c[NV];
            r_to_c<NV>(xr, c, scw, g, nn);
#pragma unroll
            for (int v = 0; v < NV; ++v) xc[v][P] = c[v];
        }
    }
}

//   in : acc[upper_tile(I,J)]  upper-triangular 16x16 tiles of T = -(Sigma~ + lambda I), accumulator layout (destroyed)
//        load_rhs(P, m, q, e)  element 16P + n (n = the lane's position in its row) of -mu~, -q and, WITH_U, -r1
//        omega; scw: >= 16 * SC_PITCH floats of LDS owned by this wave; pivot_floor, DROP as in eliminate16
//        WITH_U: r0
//   out: rhs[P] register t = y1[16P + 4g + t] (every lane; WITH_U: lanes n == 1 hold u1 instead), y0, u0
// with [omega mu~^T; mu~ Sigma~ + lambda I] [y0; y1] = [1; q] and, WITH_U, the same matrix times [u0; u1] = [r0; r1].
template <int NB, bool WITH_U = false, bool DROP = false, class LoadRhs>
__device__ __forceinline__ void solve_one(f32x4 (&acc)[NB * (NB + 1) / 2], f32x4 (&rhs)[NB], float &y0, float omega, float *scw,
                                          int g, int nn, float pivot_floor, LoadRhs load_rhs, float r0 = 0.f, float *u0_out = nullptr)
{
    constexpr int NS = WITH_U ? 3 : 2;
    factorise_one<NB, false, DROP>(acc, scw, g, nn, pivot_floor);
    float tv[NS][NB];
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        float m = 0.f, q = 0.f, e = 0.f;
        load_rhs(P, m, q, e);
        tv[0][P] = m; tv[1][P] = q;
        if constexpr (WITH_U) tv[2][P] = e;
    }
    substitute_forward<NB, NS>(acc, tv, scw, g, nn);
    // tv[0] = a = U^{-T} mu~, tv[1] = c = U^{-T} q (tv[2] = e = U^{-T} r1).  Schur step on the intercept:
    // y0 = (1 - a.c) / (omega - a.a), then y1 = U^{-1} (c - a y0), started as z = a y0 - c (the factors N_P are negated)
    float saa = 0.f, sac = 0.f, sae = 0.f;
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        saa = fmaf(tv[0][P], tv[0][P], saa);
        sac = fmaf(tv[0][P], tv[1][P], sac);
        if constexpr (WITH_U) sae = fmaf(tv[0][P], tv[2][P], sae);
    }
    saa = row_allsum(saa);
    sac = row_allsum(sac);
    const float dinv = 1.f / (omega - saa);
    y0 = (1.f - sac) * dinv;
    float u0 = 0.f;
    if constexpr (WITH_U) {
        sae = row_allsum(sae);
        u0 = (r0 - sae) * dinv;
        *u0_out = u0;
    }
    constexpr int NZ = WITH_U ? 2 : 1;       // systems of the back substitution
    float zc[NZ][NB];                        // C layout
#pragma unroll
    for (int P = 0; P < NB; ++P) {
        zc[0][P] = tv[0][P] * y0 - tv[1][P];
        if constexpr (WITH_U) zc[1][P] = tv[0][P] * u0 - tv[2][P];
    }
    substitute_back<NB, NZ>(acc, zc, rhs, scw, g, nn);
}

}  // namespace mfma
}  // namespace llla
