// Queries that see few keys (at most min(d, 64)), in fp64 and in the dual (key-space) form of the local linear
// regression of Section 2.3.
//
// Why a kernel of their own.  With m <= d visible keys the d x d matrix Sigma_i of Eq. (query_specific) has rank
// <= m and is held up by the ridge alone in the other directions, so rho_i and delta_i of Eq. (lla) are of size
// ||z|| / lambda and lambda / ||z||^2, and the output weights w (1 - z . rho) / delta are differences of numbers
// ~ ||z||^2 / lambda (10^4 for unit-variance keys at d = 128): fp32 keeps three digits of them.  The same
// minimiser written over the keys instead of the features has none of that.  With u_j = sqrt(w_ij),
// z_j = k_j - q_i, Z' the m x d matrix of rows u_j z_j and G' = Z' Z'^T (m x m), the push-through identity
// (Z'^T Z' + lambda I)^{-1} Z'^T = Z'^T (G' + lambda I)^{-1} gives, with t = (G' + lambda I)^{-1} u,
//     rho_i = Z'^T t,   delta_i = lambda (u . t),   s_ij = w_ij (1 - z_j . rho_i) / delta_i = u_j t_j / (u . t),
// i.e. one m x m positive definite system (all eigenvalues >= lambda, and for m well below d nowhere near it) and
// output weights that are formed directly, without cancellation.  fp64 throughout: these rows are a vanishing part
// of the work (m^2 d / 2 + m^3 / 3 multiply-adds per row).
//
// One 256-thread workgroup per (batch, head, row).  Forward: rows [0, nrows) of a causal call, or every row of a
// non-causal call with n <= the limit.  Decode: one workgroup per (batch, head); a sequence longer than the limit
// exits at once and keeps the output the decode kernel proper has written.
//
// A row is a serial chain (16 steps of four columns at d = 64) that leaves the matrix cores and most of the vector ALU idle,
// so the forward kernels carry these workgroups in their own grids where they can: behind the moments kernel of an fp32 call
// with 16 heads x 1024 rows they took 84 us of 613.
#pragma once

#include "llla_common.hpp"

namespace llla {
namespace dual {

constexpr int DUAL_NT = 256;

template <typename T> __device__ inline float ld_f32(const T *p, int c);
template <> __device__ inline float ld_f32<float>(const float *p, int c) { return p[c]; }
template <> __device__ inline float ld_f32<bf16_t>(const bf16_t *p, int c) { return bf16_to_f32(p[c]); }
template <typename T> __device__ inline void st_out(T *p, double v);
template <> __device__ inline void st_out<float>(float *p, double v) { *p = (float)v; }
template <> __device__ inline void st_out<bf16_t>(bf16_t *p, double v) { *p = f32_to_bf16((float)v); }

__device__ inline int tri(int j, int l) { return j * (j + 1) / 2 + l; }      // l <= j

// 1 / sqrt(x) in fp64 from the hardware estimate and two Newton steps (relative error ~1e-16 for x well inside the range)
__device__ inline double rsqrt_f64(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    r = r * (1.5 - 0.5 * x * r * r);
    r = r * (1.5 - 0.5 * x * r * r);
    return r;
}

__device__ inline double lane_value(double x, int k)      // x of lane k (k wave-uniform)
{
    const long long v = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_readlane((int)v, k), hi = __builtin_amdgcn_readlane((int)(v >> 32), k);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// LDS of one row that sees at most MK keys (a forward row at most min(D, 64), a decoded sequence 64 at every d)
template <int D, int MAX_KEYS = (D < DUAL_MAX_KEYS ? D : DUAL_MAX_KEYS)>
struct DualShared {
    static constexpr int MK = MAX_KEYS;
    double G[MK * (MK + 1) / 2];                   // lower triangle of G' + lambda I, then its Cholesky factor
    double u[64], kq[MK + 1];
    double y[MK];                                  // u as one more row of the factorisation: L^{-1} u
    double rd[MK], ld[MK / 4][6];                  // diagonal blocks of L: reciprocal diagonal, entries 10, 20, 30, 21, 31, 32
    double ut;
    float ks[(MK + 1) * (D + 1)];                  // visible keys, pitch D + 1; the query as one more row
};

// Where the rows of a forward call come from and go to
struct DualArgs {
    const void *Q, *K, *V;
    void *O;
    llla_strides sq, sk, sv, so;
    int H, n, causal;
    float lambda, scale;
    const float *lam_rows;
    float *Rho, *Delta;
    int nrows;                                     // rows [0, nrows) are served here
};

// Row i of (batch, head) bh, which sees m <= MK keys: output row O, statistics rho, delta (either may be NULL)
template <int D, typename TI, typename TO, class Shared>
__device__ __forceinline__ void dual_row(Shared &sm, const TI *qrow, const TI *Kh, const TI *Vh, int64_t kseq, int64_t vseq,
                                         int m, double lam, float scale, TO *orow, float *rho, float *delta)
{
    constexpr int MK = Shared::MK, d = D;
    constexpr int CT = D < 32 ? 32 : D;            // threads along a row of K; the others walk further rows
    constexpr int RT = DUAL_NT / CT;
    auto &ks = sm.ks;
    auto &G = sm.G;
    auto &u = sm.u;
    auto &kq = sm.kq;
    auto &rd = sm.rd;
    auto &y = sm.y;
    const int tid = threadIdx.x;
    const int m4 = (m + 3) & ~3;                   // the system is padded with identity rows to a multiple of 4
    constexpr int pitch = d + 1;
    // the values this thread needs at the very end (thread c < d: column c of the visible rows of V), requested now
    // (every load below has a valid, clamped address and no condition around it, so that the loads of a thread are
    // all in flight together; a condition per load made the compiler wait for each in turn)
    float vcol[MK];
    {
        const int cc = tid < d ? tid : d - 1;
#pragma unroll
        for (int j = 0; j < MK; ++j) vcol[j] = ld_f32(Vh + (int64_t)(j < m ? j : m - 1) * vseq, cc);
    }
    float *qs = ks + m * pitch;                    // row m of the tile: the query
    {
        // thread (r, c) walks rows r, r + RT, ..: coalesced along c
        const int r = tid / CT, c = tid % CT, cc = c < d ? c : d - 1;
        constexpr int IT = (MK + RT - 1) / RT;
        float kv[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int j = RT * it + r;
            kv[it] = ld_f32(Kh + (int64_t)(j < m ? j : m - 1) * kseq, cc);
        }
        const float qv = ld_f32(qrow, cc);
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int j = RT * it + r;
            if (j < m && c < d) ks[j * pitch + c] = kv[it];
        }
        if (r == 0 && c < d) qs[c] = qv;
    }
    __syncthreads();

    // <k_j, q> for the m keys and <q, q> (row m): four threads per row (m + 1 <= 65 rows: the last one by threads 0..3
    // in a second round)
    for (int base = 0; base <= m; base += DUAL_NT / 4) {
        const int j = base + (tid >> 2), sub = tid & 3;
        double s = 0.0;
        if (j <= m)
            for (int c = sub; c < d; c += 4) s += (double)qs[c] * (double)ks[j * pitch + c];
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        if (j <= m && sub == 0) kq[j] = s;
    }
    __syncthreads();
    // logits, their maximum, u_j = sqrt(w_j) = exp((s_j - max) / 2): the first wave, one key per lane
    if (tid < 64) {
        const double lg = tid < m ? (double)scale * kq[tid] : -INFINITY;
        double mx = lg;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
        u[tid] = tid < m ? exp(0.5 * (lg - mx)) : 0.0;
    }
    __syncthreads();

    // G'_jl = u_j u_l <z_j, z_l>, lambda on the diagonal; <z_j, z_l> = <k_j, k_l> - <k_j, q> - <k_l, q> + <q, q>
    // (products of fp32 values are exact in fp64, so the four-term form loses nothing that matters beside lambda);
    // rows m .. m4 - 1 are identity
    const int ty = tid >> 4, tx = tid & 15;        // 16 x 16 threads tile the lower triangle
    const double qq = kq[m];
    for (int j = ty; j < m4; j += 16)
        for (int l = tx; l <= j; l += 16) {
            double g = (j == l) ? 1.0 : 0.0;
            if (j < m) {
                double s0 = 0.0, s1 = 0.0;
                const float *kj = ks + j * pitch, *kl = ks + l * pitch;
#pragma unroll 4
                for (int c = 0; c < d; c += 4) {                 // d is a multiple of 16
                    s0 += (double)kj[c] * (double)kl[c];
                    s1 += (double)kj[c + 1] * (double)kl[c + 1];
                    s0 += (double)kj[c + 2] * (double)kl[c + 2];
                    s1 += (double)kj[c + 3] * (double)kl[c + 3];
                }
                g = u[j] * u[l] * (((s0 + s1) - kq[j]) - kq[l] + qq) + (j == l ? lam : 0.0);
            }
            G[tri(j, l)] = g;
        }
    if (tid < MK) y[tid] = u[tid];                 // zero from m on
    __syncthreads();

    // Cholesky G' + lambda I = L L^T in place, four columns per step (two barriers per step): every thread factorises the 4 x 4
    // diagonal block in registers; one thread per row below solves the row's four entries of the panel; all threads share
    // the rank-4 update of what is left.  u rides along as one more row, which turns it into L^{-1} u.
    for (int k0 = 0; k0 < m4; k0 += 4) {
        double a00 = G[tri(k0, k0)], a10 = G[tri(k0 + 1, k0)], a11 = G[tri(k0 + 1, k0 + 1)], a20 = G[tri(k0 + 2, k0)],
               a21 = G[tri(k0 + 2, k0 + 1)], a22 = G[tri(k0 + 2, k0 + 2)], a30 = G[tri(k0 + 3, k0)],
               a31 = G[tri(k0 + 3, k0 + 1)], a32 = G[tri(k0 + 3, k0 + 2)], a33 = G[tri(k0 + 3, k0 + 3)];
        // L_d (lower, its diagonal kept as reciprocals r0..r3)
        const double r0 = rsqrt_f64(a00);
        const double l10 = a10 * r0, l20 = a20 * r0, l30 = a30 * r0;
        a11 -= l10 * l10; a21 -= l20 * l10; a31 -= l30 * l10; a22 -= l20 * l20; a32 -= l30 * l20; a33 -= l30 * l30;
        const double r1 = rsqrt_f64(a11);
        const double l21 = a21 * r1, l31 = a31 * r1;
        a22 -= l21 * l21; a32 -= l31 * l21; a33 -= l31 * l31;
        const double r2 = rsqrt_f64(a22);
        const double l32 = a32 * r2;
        a33 -= l32 * l32;
        const double r3 = rsqrt_f64(a33);
        if (tid == 0) {
            rd[k0] = r0; rd[k0 + 1] = r1; rd[k0 + 2] = r2; rd[k0 + 3] = r3;
            double *ld = sm.ld[k0 / 4];
            ld[0] = l10; ld[1] = l20; ld[2] = l30; ld[3] = l21; ld[4] = l31; ld[5] = l32;
        }
        // panel: row j of L in columns k0..k0+3 solves x L_d^T = G[j][k0..k0+3] (forward substitution along the row)
        const int j = k0 + 4 + tid;                // m4 - k0 - 4 <= 60 rows, and the row of u
        if (j < m4 || tid == DUAL_NT - 1) {
            const bool border = tid == DUAL_NT - 1;
            double *row = border ? &y[k0] : &G[tri(j, k0)];
            const double g0 = row[0], g1 = row[1], g2 = row[2], g3 = row[3];
            const double x0 = g0 * r0;
            const double x1 = (g1 - x0 * l10) * r1;
            const double x2 = (g2 - x0 * l20 - x1 * l21) * r2;
            const double x3 = (g3 - x0 * l30 - x1 * l31 - x2 * l32) * r3;
            row[0] = x0; row[1] = x1; row[2] = x2; row[3] = x3;
        }
        __syncthreads();
        for (int j = k0 + 4 + ty; j < m4; j += 16) {
            const double j0 = G[tri(j, k0)], j1 = G[tri(j, k0 + 1)], j2 = G[tri(j, k0 + 2)], j3 = G[tri(j, k0 + 3)];
            for (int l = k0 + 4 + tx; l <= j; l += 16)
                G[tri(j, l)] -= j0 * G[tri(l, k0)] + j1 * G[tri(l, k0 + 1)] + j2 * G[tri(l, k0 + 2)] + j3 * G[tri(l, k0 + 3)];
        }
        if (ty == 15) {
            for (int l = k0 + 4 + tx; l < m4; l += 16)
                y[l] -= y[k0] * G[tri(l, k0)] + y[k0 + 1] * G[tri(l, k0 + 1)] + y[k0 + 2] * G[tri(l, k0 + 2)] + y[k0 + 3] * G[tri(l, k0 + 3)];
        }
        __syncthreads();
    }

    // L^T t = y in the first wave, lane j owning element j (m4 <= 64), four elements per step: every lane solves the diagonal block
    // for the four values (scalar broadcasts), every earlier element takes its update.
    if (tid < 64) {
        const int j = tid;
        double s = (j < m4) ? y[j] : 0.0;
        for (int k0 = m4 - 4; k0 >= 0; k0 -= 4) {
            const double *ld = sm.ld[k0 / 4];
            const int jj = j < k0 ? j : 0;
            const double g0 = G[tri(k0, jj)], g1 = G[tri(k0 + 1, jj)], g2 = G[tri(k0 + 2, jj)], g3 = G[tri(k0 + 3, jj)];
            const double t3 = lane_value(s, k0 + 3) * rd[k0 + 3];
            const double t2 = (lane_value(s, k0 + 2) - ld[5] * t3) * rd[k0 + 2];
            const double t1 = (lane_value(s, k0 + 1) - ld[3] * t2 - ld[4] * t3) * rd[k0 + 1];
            const double t0 = (lane_value(s, k0) - ld[0] * t1 - ld[1] * t2 - ld[2] * t3) * rd[k0];
            if (j < k0) s -= g0 * t0 + g1 * t1 + g2 * t2 + g3 * t3;
            else if (j < k0 + 4) s = j == k0 ? t0 : j == k0 + 1 ? t1 : j == k0 + 2 ? t2 : t3;
        }
        const double ujt = (j < m) ? u[j] * s : 0.0;        // u_j t_j: output weight s_j = u_j t_j / (u . t)
        double ut = ujt;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) ut += __shfl_xor(ut, off);
        u[j] = ujt;
        if (j == 0) sm.ut = ut;
    }
    __syncthreads();
    const double ut = sm.ut;

    if (tid < d) {                                   // d <= 128 < DUAL_NT
        const int c = tid;
        double o = 0.0, r = 0.0;
#pragma unroll
        for (int j = 0; j < MK; ++j) {
            if (j < m) {
                o += u[j] * (double)vcol[j];
                r += u[j] * ((double)ks[j * pitch + c] - (double)qs[c]);
            }
        }
        st_out(orow + c, o / ut);
        if (rho != nullptr) rho[c] = (float)r;
    }
    if (delta != nullptr && tid == 0) *delta = (float)(lam * ut);
}

// Row i of a forward call
template <int D, typename TI, typename TO>
__device__ __forceinline__ void dual_forward_row(DualShared<D> &sm, const DualArgs &a, int bh, int i)
{
    const int b = bh / a.H, h = bh % a.H;
    const size_t row = (size_t)bh * a.n + i;
    dual_row<D, TI, TO>(sm, (const TI *)a.Q + b * a.sq.batch + h * a.sq.head + (int64_t)i * a.sq.seq,
                        (const TI *)a.K + b * a.sk.batch + h * a.sk.head, (const TI *)a.V + b * a.sv.batch + h * a.sv.head, a.sk.seq,
                        a.sv.seq, a.causal ? i + 1 : a.n, (double)(a.lam_rows ? a.lam_rows[row] : a.lambda), a.scale,
                        (TO *)a.O + b * a.so.batch + h * a.so.head + (int64_t)i * a.so.seq, a.Rho ? a.Rho + row * D : nullptr,
                        a.Delta ? a.Delta + row : nullptr);
}

// R consecutive rows of a forward call with fp32 inputs, R = 4 or, at d = 128, 8, one per wave: rows top - R + 1 .. top (those
// below 0 are absent).
//
// What bounds dual_row is its chain: two barriers per block step of the factorisation, four roots one after the other in each, a
// back substitution in one wave, and every row forms the inner products of the same first keys again: some 60 000 cycles of a
// workgroup per row.  Here the products of the keys are formed once for the four rows, on fp64 MFMA, and a wave solves its row by itself:
// lane j holds row j of G' + lambda I in registers, Gauss-Jordan without pivoting (the matrix is positive definite), the row of the
// pivot broadcast by v_readlane.  All lanes take part in every update anyway, so the elimination above the diagonal is free and
// there is no back substitution; the columns move down by one register per step, so that the loop over the pivots need not be unrolled.
// 16 heads x 1024 rows: moments kernel 415 -> 360 us, the call 418 -> 359.
template <int D, int R>
struct DualSharedRows {
    double gram[64][65];                           // <k_j, k_l>
    float ks[64][D + 1];                           // the keys that the rows see, zero beyond
    float qs[R][D];
};

typedef double f64x4 __attribute__((ext_vector_type(4)));

// 1 / x in fp64 from the hardware estimate and two Newton steps
__device__ inline double rcp_f64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

__device__ inline double wave_sum_f64(double x)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
    return x;
}

template <int D, int R, typename TO>
__device__ __forceinline__ void dual_forward_rows(DualSharedRows<D, R> &sm, const DualArgs &a, int bh, int top)
{
    constexpr int MK = 64, NC = D < 64 ? 1 : D / 64;       // keys at most, columns of a lane: col + 64 c
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int col = D < 64 ? lane % D : lane;      // d = 16 / 32: lanes from d on repeat the others and store nothing
    const bool own_col = D >= 64 || lane < D;
    const int b = bh / a.H, h = bh % a.H;
    const float *Kh = (const float *)a.K + b * a.sk.batch + h * a.sk.head, *Vh = (const float *)a.V + b * a.sv.batch + h * a.sv.head;
    const float *Qh = (const float *)a.Q + b * a.sq.batch + h * a.sq.head;
    const int mtop = a.causal ? top + 1 : a.n;     // keys that the last of the rows sees, at most 64
    const int i = top - wave, ic = i > 0 ? i : 0;  // this wave's row
    const int m = a.causal ? ic + 1 : a.n;
#pragma unroll
    for (int t = 0; t < MK / R; ++t) {
        const int j = R * t + wave;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const float v = Kh[(int64_t)(j < mtop ? j : mtop - 1) * a.sk.seq + col + 64 * c];
            sm.ks[j][col + 64 * c] = j < mtop ? v : 0.f;
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) sm.qs[wave][col + 64 * c] = Qh[(int64_t)ic * a.sq.seq + col + 64 * c];
    __syncthreads();

    // products of the keys: tiles (I, J), J <= I, of 16 x 16, dealt over the waves; slot g of a chunk of four is feature 4 kc + g
    {
        const int g = lane / 16, nn = lane % 16, nb = (mtop + 15) / 16;
        for (int tile = wave; tile < nb * (nb + 1) / 2; tile += R) {
            int I = 0;
            while ((I + 1) * (I + 2) / 2 <= tile) ++I;
            const int J = tile - I * (I + 1) / 2;
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kc = 0; kc < D / 4; ++kc)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)sm.ks[16 * I + nn][4 * kc + g], (double)sm.ks[16 * J + nn][4 * kc + g], acc, 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {          // register t of lane (g, n): element [4 t + g][n]
                sm.gram[16 * I + 4 * t + g][16 * J + nn] = acc[t];
                sm.gram[16 * J + nn][16 * I + 4 * t + g] = acc[t];
            }
        }
    }
    __syncthreads();
    if (i < 0) return;                             // (no barrier and no MFMA below)

    const size_t row = (size_t)bh * a.n + i;
    const double lam = (double)(a.lam_rows ? a.lam_rows[row] : a.lambda);
    // lane j: <k_j, q>, the root of its weight (zero from m on)
    double kq = 0.0;
#pragma unroll 8
    for (int c = 0; c < D; ++c) kq = __builtin_fma((double)sm.qs[wave][c], (double)sm.ks[lane][c], kq);
    double ql[NC], qs2 = 0.0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        ql[c] = (double)sm.qs[wave][col + 64 * c];
        if (own_col) qs2 = __builtin_fma(ql[c], ql[c], qs2);
    }
    const double qq = wave_sum_f64(qs2);
    const double lg = lane < m ? (double)a.scale * kq : -INFINITY;
    double mx = lg;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    const double u = lane < m ? exp(0.5 * (lg - mx)) : 0.0;

    // row j of G' + lambda I (see dual_row); rows and columns from m on are zero and never become pivots.  The rows are selected, not
    // multiplied by u = 0: lanes m .. mtop - 1 hold keys behind this row, which need not be finite, and what lanes from 16 nb on
    // find in gram nobody has written in this workgroup.  (With rows of zeros every f, y and u_j t_j from m on is an exact zero.)
    double x[MK];
#pragma unroll
    for (int l = 0; l < MK; ++l) {
        x[l] = 0.0;
        if (l < m) {                               // (m is uniform: a scalar branch)
            const double g = ((sm.gram[lane][l] - kq) - lane_value(kq, l)) + qq;
            const double v = u * lane_value(u, l) * g + (lane == l ? lam : 0.0);
            x[l] = lane < m ? v : 0.0;
        }
    }
    double y = u, own = 0.0;
    for (int k = 0; k < m; ++k) {
        const double r = rcp_f64(lane_value(x[0], k));
        own = lane == k ? r : own;
        const double f = lane == k ? 0.0 : -x[0] * r;
        y = __builtin_fma(f, lane_value(y, k), y);
#pragma unroll
        for (int c0 = 0; c0 < MK; c0 += 8) {
            if (k + (c0 > 0 ? c0 : 1) < m) {       // scalar branches
#pragma unroll
                for (int c = (c0 > 0 ? c0 : 1); c < c0 + 8; ++c) x[c - 1] = __builtin_fma(f, lane_value(x[c], k), x[c]);
            }
        }
    }
    const double ujt = u * (y * own), ut = wave_sum_f64(ujt), inv = 1.0 / ut;     // u_j t_j: output weight s_j = u_j t_j / (u . t)

    double o[NC], rh[NC];                          // columns lane + 64 c
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = rh[c] = 0.0;
    for (int j0 = 0; j0 < m; j0 += 16) {
        float v[16][NC];
#pragma unroll
        for (int t = 0; t < 16; ++t)
#pragma unroll
            for (int c = 0; c < NC; ++c) v[t][c] = Vh[(int64_t)(j0 + t < m ? j0 + t : m - 1) * a.sv.seq + col + 64 * c];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            if (j0 + t < m) {
                const double w = lane_value(ujt, j0 + t);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    o[c] = __builtin_fma(w, (double)v[t][c], o[c]);
                    rh[c] = __builtin_fma(w, (double)sm.ks[j0 + t][col + 64 * c] - ql[c], rh[c]);
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (own_col) st_out((TO *)a.O + b * a.so.batch + h * a.so.head + (int64_t)i * a.so.seq + col + 64 * c, o[c] * inv);
        if (a.Rho != nullptr && own_col) a.Rho[row * D + col + 64 * c] = (float)rh[c];
    }
    if (a.Delta != nullptr && lane == 0) a.Delta[row] = (float)(lam * ut);
}

// The sequence of (batch, head) bh of a decode call (q, o contiguous); returns at once if it is longer than 64 keys
template <int D, typename TI, typename TO>
__device__ __forceinline__ void dual_decode_head(DualShared<D, DUAL_MAX_KEYS> &sm, const DualArgs &a, const int32_t *seqlens, int bh)
{
    const int b = bh / a.H, h = bh % a.H;
    int m = seqlens ? seqlens[b] : a.n;
    m = m < 1 ? 1 : (m > a.n ? a.n : m);
    if (m > DUAL_MAX_KEYS) return;                            // the whole workgroup
    dual_row<D, TI, TO>(sm, (const TI *)a.Q + (int64_t)bh * D, (const TI *)a.K + b * a.sk.batch + h * a.sk.head,
                        (const TI *)a.V + b * a.sv.batch + h * a.sv.head, a.sk.seq, a.sv.seq, m, (double)a.lambda, a.scale,
                        (TO *)a.O + (int64_t)bh * D, nullptr, nullptr);
}

inline DualArgs dual_args(const Problem &p)
{
    return DualArgs{p.Q, p.K, p.V, p.O, p.sq, p.sk, p.sv, p.so, p.H, p.n, p.causal, p.lambda, p.scale, p.lambda_rows, p.rho, p.delta,
                    dual_forward_rows(p)};
}

}  // namespace dual
}  // namespace llla

