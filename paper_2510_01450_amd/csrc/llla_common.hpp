// Shared declarations of the gfx950 Local Linear Attention library (host + device).
// Nothing here is used by, or shared with, the CPU oracle.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "llla.h"

namespace llla {

// The tensors of a d = 16 / 32 call and their copies in rows of 64 features, zero from d on (llla_pad.hip)
struct PadSource {
    const char *src;           // [B,H,n,d], strides s in elements
    uint4 *dst;                // [B*H*n, 64] contiguous
    llla_strides s;
};
struct PadSources {
    PadSource t[4];            // Q, K, V, dO
    int count;
};

// One forward or decode problem, as validated by the C ABI layer.
struct Problem {
    const void *Q, *K, *V;     // forward: [B,H,n,d]; decode: Q = q [B,H,d], K/V = caches [B,H,n,d]
    void *O;                   // forward: [B,H,n,d]; decode: [B,H,d]
    llla_strides sq, sk, sv, so;
    const int32_t *seqlens;    // decode only (device, [B]) or nullptr
    int B, H, n, d;            // n = sequence length (forward) or L_max (decode)
    llla_dtype in, out;
    int causal;
    int live_d;                // forward on zero-padded copies: features [live_d, d) are zero in Q and K; 0 = none are
    const PadSources *pad;     // bf16: Q, K and V are copies that the call has yet to make from these; or nullptr
    float lambda, scale;
    const float *lambda_rows;  // forward only: [B,H,n] ridge per query row, or nullptr (then `lambda` for all rows)
    float *rho, *delta;        // forward only: optional outputs [B,H,n,d] and [B,H,n] (Eq. (lla)), or nullptr
    void *ws;
    size_t ws_bytes;
    hipStream_t stream;
};

// One backward problem (causal), as validated by the C ABI layer.  Gradients are fp32, contiguous.
struct BackwardProblem {
    const void *Q, *K, *V, *dO;  // [B,H,n,d] in dtype `in`
    llla_strides sq, sk, sv, sdo;
    float *dQ, *dK, *dV;         // [B,H,n,d]
    float *dlambda;              // [B,H,n] or nullptr
    int B, H, n, d;
    int live_d;                  // on zero-padded copies: features [live_d, d) of Q and K are zero; 0 = none are
    const PadSources *pad;       // bf16: Q, K, V and dO are copies that the call has yet to make from these; or nullptr
    llla_dtype in;
    float lambda, scale;
    const float *lambda_rows;    // [B,H,n] or nullptr
    void *ws;
    size_t ws_bytes;
    hipStream_t stream;
};

// Launchers return hipSuccess or the launch error.  Each lives in its own translation unit.
hipError_t valu_forward(const Problem &p);
// fp32 inputs, d = 16 / 32, short sequences: one wave per row (llla_short.hip)
bool short_forward_takes(int heads, int n, int d, llla_dtype in);
hipError_t short_forward(const Problem &p);
// sweep 3 only, for query rows [0, nrows): y (pitch ypitch floats: y1 then y0) and the row maxima (log2
// units) come from device memory
hipError_t valu_forward_given(const Problem &p, int nrows, const float *M, int mpitch, const float *Y, int ypitch);
hipError_t valu_decode(const Problem &p);

// Queries that see at most dual_max_keys(d) = min(d, DUAL_MAX_KEYS) keys: fp64, key-space form of the same minimiser
// (llla_dual.hpp).  dual_forward() serves rows [0, dual_forward_rows(p)) of a forward call (O, and rho / delta when
// asked for); dual_decode() serves the sequences of a decode call that are short enough and leaves the others alone.
constexpr int DUAL_MAX_KEYS = 64;
int dual_max_keys(int d);
int dual_forward_rows(const Problem &p);
hipError_t dual_forward(const Problem &p);
hipError_t dual_decode(const Problem &p);

size_t valu_backward_workspace_bytes(int B, int H, int n, int d);
hipError_t valu_backward(const BackwardProblem &p);
// backward with the matrix-core moments and solve (bf16, d = 64 / 128): workspace layout and the two MFMA stages
struct BackwardLayout {
    size_t fwd;        // the forward's workspace (re-tiled K, V; row maxima M; y rows)
    size_t u, r, sc;   // u rows and r rows (pitch ypitch floats: vector then scalar), row scalars (8 floats per row)
    size_t total;
    int npad;          // pitch of the row maxima (log2 units), in floats
    int ypitch;        // pitch of a y / u / r row, in floats
    size_t m, y;       // offsets of M and of the y rows inside the forward's workspace
};
BackwardLayout mfma_backward_layout(int B, int H, int n, int d);
hipError_t mfma_backward_rowmax(const BackwardProblem &p, const BackwardLayout &L);   // re-tiling and row maxima
hipError_t mfma_backward_solve(const BackwardProblem &p, const BackwardLayout &L);    // moments, y and u of every row
hipError_t mfma_backward_r(const BackwardProblem &p, const BackwardLayout &L, int early);   // r rows, argmax
hipError_t mfma_backward_dq(const BackwardProblem &p, const BackwardLayout &L, int early);  // dQ, dlambda, row scalars
// output of a bf16 forward from the row maxima (log2 units) and the solved rows (llla_mfma_bwd.hip); early: rows with three-term operands
hipError_t mfma_output_rows(const Problem &p, const float *M, int mpitch, const float *Y, int early);
hipError_t mfma_backward_keys(const BackwardProblem &p, const BackwardLayout &L);     // dK, dV from y, u and the row scalars
// the same for fp32 inputs: sweeps on the fp32 matrix cores (llla_mfma_bwd_f32.hip); its moments kernel is the
// forward's, with the row maxima M given and the rows r replaced by u
bool mfma_backward_f32_supported(int n, int d, llla_dtype in);
size_t mfma_backward_f32_workspace_bytes(int B, int H, int n, int d);
hipError_t mfma_backward_f32(const BackwardProblem &p);
hipError_t mfma_moments_f32_given(const BackwardProblem &p, int npad, float *M, float *Y, float *RU);
size_t backward_workspace_bytes(int B, int H, int n, int d, llla_dtype in, llla_path path);     // what a call must have
size_t backward_wanted_bytes(int B, int H, int n, int d, llla_dtype in);                        // and what it can make use of
hipError_t backward(const BackwardProblem &p, llla_path path);

// MFMA (matrix-core) paths; *_supported() says whether one exists for the shape and dtype.
bool mfma_forward_supported(int d, llla_dtype in, bool causal);
size_t mfma_forward_workspace_bytes(int B, int H, int n, int d, llla_dtype in);
hipError_t mfma_forward(const Problem &p);
// the same for fp32 inputs (d = 64): llla_mfma_fwd_f32.hip
bool mfma_forward_f32_supported(int d, bool causal);
size_t mfma_forward_f32_workspace_bytes(int B, int H, int n);
hipError_t mfma_forward_f32(const Problem &p, const Problem &call);
hipError_t mfma_output_f32(const Problem &p, int npad, float *M, const float *Y, int skip);      // its output sweep, rows from skip on
// and at d = 128: llla_mfma_fwd_f32_128.hip.  The workspace is optional: a call with less runs on the vector kernels.
size_t mfma_forward_f32_wide_workspace_bytes(int B, int H, int n);
hipError_t mfma_forward_f32_wide(const Problem &p);
hipError_t mfma_moments_f32_wide_given(const BackwardProblem &p, int npad, float *M, float *Y, float *RU);
// head dimensions 16 and 32 (bf16 or fp32): the d = 64 matrix-core forward on zero-padded copies (llla_pad.hip)
bool padded_forward_supported(int d, llla_dtype in);
size_t padded_forward_workspace_bytes(int B, int H, int n, int d, llla_dtype in);
hipError_t padded_forward(const Problem &p);
size_t padded_forward_cg_workspace_bytes(int B, int H, int n, int d, llla_dtype in);   // bf16 only, like the mode itself
hipError_t padded_forward_cg(const Problem &p, int T, float eps, int32_t *iters);
bool padded_backward_supported(int d, llla_dtype in);          // bf16 only, like the matrix-core backward itself
size_t padded_backward_workspace_bytes(int B, int H, int n, int d, llla_dtype in);
hipError_t padded_backward(const BackwardProblem &p);
hipError_t pad_queries_keys(const BackwardProblem &p, void *Q, void *K);      // Q and K in rows of 64 features, zero from p.d on
// approximate mode: T conjugate-gradient steps per row (bf16, d = 64 / 128, causal); iters: [B,H,n] steps done, or nullptr
size_t mfma_forward_cg_workspace_bytes(int B, int H, int n, int d, llla_dtype in);
hipError_t mfma_forward_cg(const Problem &p, int T, float eps, int32_t *iters);
bool mfma_decode_supported(int d, llla_dtype in);
size_t mfma_decode_workspace_bytes(int B, int H, int L_max, int d, llla_dtype in);      // what a call must have
size_t mfma_decode_wanted_bytes(int B, int H, int L_max, int d, llla_dtype in);         // and what it can make use of (at least that)
// whether the MFMA decode path serves this call (it needs the full cache length for every sequence)
bool mfma_decode_takes(const Problem &p);
hipError_t mfma_decode(const Problem &p);
// fp32 matrix-core decode (llla_mfma_decode_f32.hip): fp32 caches, and bf16 caches that the 16-bit kernels do not serve.  The
// workspace is optional: a call with less than the size asked for runs one workgroup per head.
size_t mfma_decode_f32_workspace_bytes(int B, int H, int L_max, int d);
bool mfma_decode_f32_takes(const Problem &p);
hipError_t mfma_decode_f32(const Problem &p);
// the d = 128 kernels behind mfma_decode (a translation unit of their own)
size_t mfma_decode128_workspace_bytes(int B, int H, int L_max);
size_t mfma_decode128_flat_bytes(int B, int H, int L_max);
hipError_t mfma_decode128(const Problem &p);

// ---- stage hooks ---------------------------------------------------------------------------------
// stage_mark(stream, name) labels the work enqueued AFTER it, up to the next mark; stage_begin() starts a new call,
// stage_end() closes the last stage.  In the production library they compile to nothing.  The measurement build
// (-DLLLA_MEASURE, a library of its own) records HIP events there so that a benchmark can time each kernel of a call.
#ifdef LLLA_MEASURE
void stage_begin(hipStream_t stream);
void stage_mark(hipStream_t stream, const char *name);
void stage_end(hipStream_t stream);
#else
inline void stage_begin(hipStream_t) {}
inline void stage_mark(hipStream_t, const char *) {}
inline void stage_end(hipStream_t) {}
#endif

// ---- storage types -----------------------------------------------------------------------------
// bf16 is handled as raw uint16_t bits; conversions are written out so that rounding is explicit.
typedef uint16_t bf16_t;

__host__ __device__ inline float bf16_to_f32(bf16_t x)
{
    union { uint32_t u; float f; } c;
    c.u = (uint32_t)x << 16;
    return c.f;
}

// round-to-nearest-even; NaN stays NaN (quiet)
__host__ __device__ inline bf16_t f32_to_bf16(float f)
{
    union { uint32_t u; float f; } c;
    c.f = f;
    if ((c.u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((c.u >> 16) | 0x40);
    c.u += 0x7fffu + ((c.u >> 16) & 1u);
    return (bf16_t)(c.u >> 16);
}

// 16-byte chunk `id` of a padded tensor: chunks inside the original row are copied, the others cleared.  ESZ = bytes per element.
template <int ESZ>
__device__ __forceinline__ void pad_chunk(const PadSource &t, size_t id, int H, int n, int d, size_t nchunks)
{
    constexpr int CPR = 64 * ESZ / 16;                      // chunks per padded row
    if (id >= nchunks) return;
    const size_t row = id / CPR;
    const int c = (int)(id % CPR);
    const int i = (int)(row % n);
    const size_t bh = row / n;
    const int h = (int)(bh % H);
    const int64_t b = (int64_t)(bh / H);
    uint4 v = {0u, 0u, 0u, 0u};
    if (c * 16 < d * ESZ) {
        const int64_t e = b * t.s.batch + (int64_t)h * t.s.head + (int64_t)i * t.s.seq;
        v = *reinterpret_cast<const uint4 *>(t.src + e * ESZ + c * 16);
    }
    t.dst[id] = v;
}

__host__ __device__ inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace llla
