// The head-shared step of caches of few slots: its two launches of swa_short_kernel.
#include "swa_short.hpp"

namespace swa {

namespace {
struct LaunchShared {
    const DecodeArgs& a;
    int64_t pairs;
    hipStream_t stream;

    template <typename T, int D, int NT, int U>
    int go() const
    {
        if constexpr (short_rows<T, D, NT, U>() > 0) {
            const dim3 grid((unsigned)pairs), block(NT);
            if (a.phase == 1) launch_kernel((swa_short_kernel<T, D, NT, U, false, 1>), grid, block, 0, stream, a);
            else launch_kernel((swa_short_kernel<T, D, NT, U, false, 2>), grid, block, 0, stream, a);
            return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
        }
        return SWA_ERR_BAD_SHAPE;          // (short_form names no such form)
    }
};
}  // namespace

int launch_short_shared(const DecodeArgs& a, const swa_params& p, int64_t pairs, ShortForm f, hipStream_t stream)
{
    return with_form(p, f, LaunchShared{a, pairs, stream});
}

}  // namespace swa
