// The head-shared step of caches of few slots: its two launches of swa_short_kernel.
#include "swa_short.hpp"

namespace swa {

template <typename T, int D, int NT, int U>
static int launch_shared_f(const DecodeArgs& a, int64_t pairs, hipStream_t stream)
{
    if constexpr (short_rows<T, D, NT, U>() > 0) {
        const dim3 grid((unsigned)pairs), block(NT);
        if (a.phase == 1) hipLaunchKernelGGL((swa_short_kernel<T, D, NT, U, false, 1>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((swa_short_kernel<T, D, NT, U, false, 2>), grid, block, 0, stream, a);
        return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
    }
    return SWA_ERR_BAD_SHAPE;          // (short_form names no such form)
}

template <typename T, int D>
static int launch_shared_t(const DecodeArgs& a, int64_t pairs, ShortForm f, hipStream_t stream)
{
    if (f.nt == 128) return launch_shared_f<T, D, 128, short_unroll<T, D>(8)>(a, pairs, stream);
    if (f.nt == 512) return launch_shared_f<T, D, 512, short_unroll<T, D>(8)>(a, pairs, stream);
    if (f.u == 12) return launch_shared_f<T, D, 256, short_unroll<T, D>(12)>(a, pairs, stream);
    return launch_shared_f<T, D, 256, short_unroll<T, D>(8)>(a, pairs, stream);
}

int launch_short_shared(const DecodeArgs& a, const swa_params& p, int64_t pairs, ShortForm f, hipStream_t stream)
{
    if (p.flags & SWA_KV_INT8)
        return p.d == 64 ? launch_shared_t<Q8, 64>(a, pairs, f, stream) : launch_shared_t<Q8, 128>(a, pairs, f, stream);
    if (p.dtype == SWA_F32)
        return p.d == 64 ? launch_shared_t<F32, 64>(a, pairs, f, stream) : launch_shared_t<F32, 128>(a, pairs, f, stream);
    if (p.dtype == SWA_F16)
        return p.d == 64 ? launch_shared_t<F16, 64>(a, pairs, f, stream) : launch_shared_t<F16, 128>(a, pairs, f, stream);
    return p.d == 64 ? launch_shared_t<BF16, 64>(a, pairs, f, stream) : launch_shared_t<BF16, 128>(a, pairs, f, stream);
}

}  // namespace swa
