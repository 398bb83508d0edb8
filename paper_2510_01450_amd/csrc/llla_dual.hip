// Launches of the key-space rows (llla_dual.hpp) on their own: decode, and the forward calls whose kernels do not carry them.
#include "llla_dual.hpp"

namespace llla {
namespace {

using namespace dual;

template <int D, typename TI, typename TO>
__global__ __launch_bounds__(DUAL_NT) void dual_rows_kernel(DualArgs a)
{
    __shared__ DualShared<D> sm;
    dual_forward_row<D, TI, TO>(sm, a, blockIdx.y, blockIdx.x);
}

// Decode: one workgroup per (batch, head); a longer sequence is served by the decode kernel proper
template <int D, typename TI, typename TO>
__global__ __launch_bounds__(DUAL_NT) void dual_decode_kernel(DualArgs a, const int32_t *__restrict__ seqlens)
{
    __shared__ DualShared<D, DUAL_MAX_KEYS> sm;
    dual_decode_head<D, TI, TO>(sm, a, seqlens, blockIdx.y);
}

template <int D, typename TI, typename TO>
hipError_t launch_dual(const Problem &p, bool decode)
{
    const DualArgs a = dual_args(p);
    if (decode)
        hipLaunchKernelGGL((dual_decode_kernel<D, TI, TO>), dim3(1, p.B * p.H), dim3(DUAL_NT), 0, p.stream, a, p.seqlens);
    else
        hipLaunchKernelGGL((dual_rows_kernel<D, TI, TO>), dim3(a.nrows, p.B * p.H), dim3(DUAL_NT), 0, p.stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t dual_by_dtype(const Problem &p, bool decode)
{
    if (p.in == LLLA_F32) return p.out == LLLA_F32 ? launch_dual<D, float, float>(p, decode) : launch_dual<D, float, bf16_t>(p, decode);
    return p.out == LLLA_F32 ? launch_dual<D, bf16_t, float>(p, decode) : launch_dual<D, bf16_t, bf16_t>(p, decode);
}

hipError_t dual_by_dim(const Problem &p, bool decode)
{
    switch (p.d) {
        case 16: return dual_by_dtype<16>(p, decode);
        case 32: return dual_by_dtype<32>(p, decode);
        case 64: return dual_by_dtype<64>(p, decode);
        case 128: return dual_by_dtype<128>(p, decode);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int dual_max_keys(int d) { return d < DUAL_MAX_KEYS ? d : DUAL_MAX_KEYS; }

int dual_forward_rows(const Problem &p)
{
    const int lim = dual_max_keys(p.d);
    if (p.causal) return p.n < lim ? p.n : lim;
    return p.n <= lim ? p.n : 0;
}

hipError_t dual_forward(const Problem &p)
{
    if (dual_forward_rows(p) == 0) return hipSuccess;
    return dual_by_dim(p, false);
}

hipError_t dual_decode(const Problem &p) { return dual_by_dim(p, true); }

}  // namespace llla
