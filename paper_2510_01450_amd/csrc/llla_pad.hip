// Head dimensions 16 and 32 on the matrix-core forward: the call is run at d = 64 on zero-padded copies.
//
// Why this is exact.  With the features d .. 63 of every query and key equal to zero the logits are unchanged, the
// padded entries of mu~ are zero, the padded rows and columns of Sigma~ are zero, and the ridge puts lambda on the
// padded diagonal: the system of Eq. (query_specific) splits into the original one and lambda * y_pad = 0.  The
// products that fill the padded tiles are products with exact zeros, so the factorisation sees an exactly
// block-diagonal matrix and the original block is solved as it would be alone (up to the order of rounding).  The
// padded columns of V give padded columns of O that are dropped.
//
// Why it pays.  The d x d moment of a query-key pair is a contraction only the matrix cores do fast; the vector
// kernels need d^2 fp32 multiply-adds per pair, the padded call 64^2 / 2 on 16-bit MFMA at sixteen times the rate
// (fp32 inputs: fp32 MFMA).  The copies are Theta(B H n 64), like the rest of the workspace.
//
// The bf16 kernels know the number of 16-feature blocks that are not padding: they skip the padded ones and write the caller's tensors
// themselves (outputs through padded rows and a copy out: 3 x 16 heads x 1606, d = 32, with statistics 259 us, 250 without; the
// backward's sweeps over all 64 features as well: 96 heads x 1882 1134 us, 974).  With fp32 inputs only the moments run on copies.  The approximate
// mode writes padded rows.
#include "llla_common.hpp"

namespace llla {
namespace {

constexpr int PD = 64;      // padded head dimension

struct PadLayout {
    size_t q, k, v, o, rho, inner, total;
};

PadLayout make_pad_layout(int B, int H, int n, llla_dtype in, bool cg = false)
{
    const size_t rows = (size_t)B * H * n;
    const size_t esz = in == LLLA_F32 ? 4 : 2;
    PadLayout L{};
    size_t off = 0;
    L.q = off; off += round_up(rows * PD * esz, 256);
    L.k = off; off += round_up(rows * PD * esz, 256);
    L.v = off; off += round_up(rows * PD * esz, 256);       // (not fp32)
    // rows of O and rho: the approximate mode alone writes them; the size that callers are told stays what it was
    L.o = off; off += round_up(rows * PD * 4, 256);
    L.rho = off; off += round_up(rows * PD * 4, 256);
    L.inner = off;
    off += round_up(cg ? mfma_forward_cg_workspace_bytes(B, H, n, PD, in)
                       : in == LLLA_F32 ? mfma_forward_f32_workspace_bytes(B, H, n) : mfma_forward_workspace_bytes(B, H, n, PD, in), 256);
    L.total = off;
    return L;
}

// One thread per 16-byte chunk of a padded row, blockIdx.y the tensor.
// All tensors of a call in one launch, on the way in and, in the approximate mode, on the way out: a copy of a small call takes 5 us, nearly all
// of it the launch.  (The exact bf16 calls make theirs in the launch that forms the row maxima.)
template <int ESZ>
__global__ __launch_bounds__(256) void pad_rows_kernel(PadSources a, int H, int n, int d, size_t nchunks)
{
    pad_chunk<ESZ>(a.t[blockIdx.y], (size_t)blockIdx.x * 256 + threadIdx.x, H, n, d, nchunks);
}

// The first d elements of every padded row back into a strided [B,H,n,d] tensor, one 16-byte chunk per thread.  A destination whose
// rows are 16-byte aligned takes it whole, the statistics, which need not be, in words of 4 bytes.
struct UnpadTarget {
    const uint4 *src;
    char *dst;
    llla_strides s;
    int elem;                                               // bytes per element of source and destination
    int words;                                              // stored in words of 4 bytes
};
struct UnpadTargets {
    UnpadTarget t[3];
};

__global__ __launch_bounds__(256) void unpad_rows_kernel(UnpadTargets a, int H, int n, int d, size_t nrows)
{
    const UnpadTarget &t = a.t[blockIdx.y];
    const int cpr = d * t.elem / 16;                        // chunks per original row
    const size_t id = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t row = id / cpr;
    if (row >= nrows) return;
    const int c = (int)(id % cpr);
    const int i = (int)(row % n);
    const size_t bh = row / n;
    const int h = (int)(bh % H);
    const int64_t b = (int64_t)(bh / H);
    const int64_t e = b * t.s.batch + (int64_t)h * t.s.head + (int64_t)i * t.s.seq;
    const uint4 v = t.src[row * (PD * t.elem / 16) + c];
    char *dst = t.dst + e * t.elem + c * 16;
    if (t.words) {
        uint32_t *w = reinterpret_cast<uint32_t *>(dst);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else {
        *reinterpret_cast<uint4 *>(dst) = v;
    }
}

struct Rows {
    int B, H, n, d;
    hipStream_t stream;
};

hipError_t pad_rows(const PadSources &a, const Rows &r, bool f32)
{
    const size_t rows = (size_t)r.B * r.H * r.n, nch = rows * (PD * (f32 ? 4 : 2) / 16);
    const dim3 grid((unsigned)((nch + 255) / 256), a.count);
    if (f32) pad_rows_kernel<4><<<grid, dim3(256), 0, r.stream>>>(a, r.H, r.n, r.d, nch);
    else pad_rows_kernel<2><<<grid, dim3(256), 0, r.stream>>>(a, r.H, r.n, r.d, nch);
    return hipGetLastError();
}

hipError_t unpad_rows(const UnpadTargets &a, int count, const Rows &r)
{
    const size_t rows = (size_t)r.B * r.H * r.n;
    int elem = 0;
    for (int i = 0; i < count; ++i) elem = a.t[i].elem > elem ? a.t[i].elem : elem;
    const size_t nch = rows * (r.d * elem / 16);
    unpad_rows_kernel<<<dim3((unsigned)((nch + 255) / 256), count), dim3(256), 0, r.stream>>>(a, r.H, r.n, r.d, rows);
    return hipGetLastError();
}

PadSource pad_source(const void *src, llla_strides s, void *dst) { return PadSource{static_cast<const char *>(src), static_cast<uint4 *>(dst), s}; }
UnpadTarget unpad_target(const void *src, void *dst, llla_strides s, int elem, bool words = false)
{
    return UnpadTarget{static_cast<const uint4 *>(src), static_cast<char *>(dst), s, elem, words ? 1 : 0};
}

// O, and with statistics rho, from the padded rows of a forward call
hipError_t unpad_forward(const Problem &p, char *ws, const PadLayout &L, const Rows &r)
{
    const llla_strides sr = {(int64_t)p.H * p.n * p.d, (int64_t)p.n * p.d, (int64_t)p.d};
    UnpadTargets a{};
    a.t[0] = unpad_target(ws + L.o, p.O, p.so, p.out == LLLA_F32 ? 4 : 2);
    if (p.rho) a.t[1] = unpad_target(ws + L.rho, p.rho, sr, 4, true);
    return unpad_rows(a, p.rho ? 2 : 1, r);
}

struct PadBackwardLayout {
    size_t q, k, v, g, inner, total;
};

PadBackwardLayout make_pad_backward_layout(int B, int H, int n)
{
    const size_t rows = (size_t)B * H * n;
    PadBackwardLayout L{};
    size_t off = 0;
    L.q = off; off += round_up(rows * PD * 2, 256);
    L.k = off; off += round_up(rows * PD * 2, 256);
    L.v = off; off += round_up(rows * PD * 2, 256);
    L.g = off; off += round_up(rows * PD * 2, 256);
    L.inner = off;
    off += round_up(backward_workspace_bytes(B, H, n, PD, LLLA_BF16, LLLA_PATH_MFMA), 256);
    L.total = off;
    return L;
}

}  // namespace

hipError_t pad_queries_keys(const BackwardProblem &p, void *Q, void *K)
{
    const PadSources in = {{pad_source(p.Q, p.sq, Q), pad_source(p.K, p.sk, K)}, 2};
    return pad_rows(in, Rows{p.B, p.H, p.n, p.d, p.stream}, p.in == LLLA_F32);
}

bool padded_forward_supported(int d, llla_dtype in)
{
    if (d != 16 && d != 32) return false;
    return in == LLLA_F32 ? mfma_forward_f32_supported(PD, true) : mfma_forward_supported(PD, in, true);
}

size_t padded_forward_workspace_bytes(int B, int H, int n, int d, llla_dtype in)
{
    if (!padded_forward_supported(d, in)) return 0;
    return make_pad_layout(B, H, n, in).total;
}

hipError_t padded_forward(const Problem &p)
{
    // every grid below is one-dimensional in 256-thread groups over 16-byte chunks: at most 2^31 rows * 16 chunks
    const PadLayout L = make_pad_layout(p.B, p.H, p.n, p.in);
    char *ws = static_cast<char *>(p.ws);
    const llla_strides sp = {(int64_t)p.H * p.n * PD, (int64_t)p.n * PD, (int64_t)PD};

    Problem q = p;
    q.Q = ws + L.q; q.K = ws + L.k;
    q.sq = q.sk = sp;
    q.d = PD;
    q.live_d = p.d;
    q.ws = ws + L.inner;
    q.ws_bytes = L.total - L.inner;
    if (p.in == LLLA_F32) {                                 // the moments alone run on copies; the rest reads and writes the tensors themselves
        stage_mark(p.stream, "pad");
        const PadSources in = {{pad_source(p.Q, p.sq, ws + L.q), pad_source(p.K, p.sk, ws + L.k)}, 2};
        const hipError_t e = pad_rows(in, Rows{p.B, p.H, p.n, p.d, p.stream}, true);
        return e != hipSuccess ? e : mfma_forward_f32(q, p);
    }
    const PadSources in = {{pad_source(p.Q, p.sq, ws + L.q), pad_source(p.K, p.sk, ws + L.k), pad_source(p.V, p.sv, ws + L.v)}, 3};
    q.V = ws + L.v;
    q.sv = sp;
    q.pad = &in;
    return mfma_forward(q);
}

// The approximate mode (conjugate gradients) at d = 16 / 32 (bf16): the same padding.  The padded entries of every
// iterate stay zero -- the residual there is mu_pad - (Sigma p)_pad = 0 - lambda * 0 -- so steps, residuals and the
// active mask are those of the original system.
size_t padded_forward_cg_workspace_bytes(int B, int H, int n, int d, llla_dtype in)
{
    if (in != LLLA_BF16 || !padded_forward_supported(d, in)) return 0;
    return make_pad_layout(B, H, n, in, true).total;
}

hipError_t padded_forward_cg(const Problem &p, int T, float eps, int32_t *iters)
{
    const PadLayout L = make_pad_layout(p.B, p.H, p.n, p.in, true);
    char *ws = static_cast<char *>(p.ws);
    const llla_strides sp = {(int64_t)p.H * p.n * PD, (int64_t)p.n * PD, (int64_t)PD};
    const Rows r{p.B, p.H, p.n, p.d, p.stream};
    const PadSources in = {{pad_source(p.Q, p.sq, ws + L.q), pad_source(p.K, p.sk, ws + L.k), pad_source(p.V, p.sv, ws + L.v)}, 3};
    hipError_t e = pad_rows(in, r, false);
    if (e != hipSuccess) return e;
    Problem q = p;
    q.Q = ws + L.q; q.K = ws + L.k; q.V = ws + L.v; q.O = ws + L.o;
    q.sq = q.sk = q.sv = q.so = sp;
    q.d = PD;
    q.rho = p.rho ? reinterpret_cast<float *>(ws + L.rho) : nullptr;
    q.ws = ws + L.inner;
    q.ws_bytes = L.total - L.inner;
    e = mfma_forward_cg(q, T, eps, iters);
    if (e != hipSuccess) return e;
    return unpad_forward(p, ws, L, r);
}

// The backward pass at d = 16 / 32 (bf16): the same padding.  The gradient with respect to a padded feature is zero to
// first order -- a padded key feature enters the output only through its product with the padded part of y, and both
// factors vanish -- so the padded columns of dQ, dK and dV are dropped; dlambda has no feature index.
bool padded_backward_supported(int d, llla_dtype in)
{
    return (d == 16 || d == 32) && in == LLLA_BF16 && mfma_forward_supported(PD, in, true);
}

size_t padded_backward_workspace_bytes(int B, int H, int n, int d, llla_dtype in)
{
    if (!padded_backward_supported(d, in)) return 0;
    return make_pad_backward_layout(B, H, n).total;
}

hipError_t padded_backward(const BackwardProblem &p)
{
    const PadBackwardLayout L = make_pad_backward_layout(p.B, p.H, p.n);
    char *ws = static_cast<char *>(p.ws);
    const llla_strides sp = {(int64_t)p.H * p.n * PD, (int64_t)p.n * PD, (int64_t)PD};
    const PadSources in = {{pad_source(p.Q, p.sq, ws + L.q), pad_source(p.K, p.sk, ws + L.k), pad_source(p.V, p.sv, ws + L.v),
                            pad_source(p.dO, p.sdo, ws + L.g)}, 4};

    BackwardProblem q = p;
    q.Q = ws + L.q; q.K = ws + L.k; q.V = ws + L.v; q.dO = ws + L.g;
    q.sq = q.sk = q.sv = q.sdo = sp;
    q.d = PD;
    q.live_d = p.d;
    q.pad = &in;
    q.ws = ws + L.inner;
    q.ws_bytes = L.total - L.inner;
    return backward(q, LLLA_PATH_MFMA);
}

}  // namespace llla
