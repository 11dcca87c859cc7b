// Which calls the kernel for caches of few slots serves, and its launches (swa_short.hpp; the head-shared step's two are in
// swa_short_shared.hip).
#include "swa_short.hpp"

namespace swa {

// The forms: threads per workgroup and rows per lane.
constexpr ShortForm kForms[] = {{128, 8}, {256, 8}, {256, 12}, {512, 8}};

template <typename T, int D>
static int short_rows(ShortForm f)
{
    if (f.nt == 128) return short_rows<T, D, 128, short_unroll<T, D>(8)>();
    if (f.nt == 512) return short_rows<T, D, 512, short_unroll<T, D>(8)>();
    return f.u == 12 ? short_rows<T, D, 256, short_unroll<T, D>(12)>() : short_rows<T, D, 256, short_unroll<T, D>(8)>();
}

static int short_rows(const swa_params& p, ShortForm f)
{
    if (p.flags & SWA_KV_INT8) return p.d == 64 ? short_rows<Q8, 64>(f) : short_rows<Q8, 128>(f);
    if (p.dtype == SWA_F32) return p.d == 64 ? short_rows<F32, 64>(f) : short_rows<F32, 128>(f);
    return p.d == 64 ? short_rows<F16, 64>(f) : short_rows<F16, 128>(f);
}

// Which calls: the two-call form and unordered compaction (in token order rows shift by way of LDS; the strict window together
// with head-shared selection is left to the streaming kernel), with a bound on the lengths that a form covers; the smallest
// form that does.
// Streaming kernel / this one, us a step, f16 unless stated, d = 128, one token evicted:
//      32 pairs   106 slots 7.0 / 5.0,  140  7.6 / 5.4,  206  8.4 / 6.2;  8-bit 206  8.6 / 7.2
//     512 pairs    64 slots 7.2 / 5.3,  106  7.9 / 6.5,  140  9.4 / 8.5,  206 12.3 / 12.0;  8-bit 106  8.5 / 7.3,  206 10.1 / 9.3
//    1024 pairs   106 slots 12.9 / 11.3,  140 16.0 / 15.1,  206 21.3 / 21.2;  8-bit 206 14.5 / 15.9
//    2560 pairs    32 slots 16.2 / 9.8,  106 26.6 / 23.9,  140 32.9 / 32.1,  206 46.6 / 47.1;  8-bit 106 20.2 / 17.9,  206 30.4 / 30.7
//    8192 pairs   106 slots 77 / 75,  160 112 / 110
// The forms that fill half a CU with one workgroup (512 threads, and 256 on the 8-bit cache, whose lanes hold
// 16 channels) pay while the chip is not full of workgroups; the strict window, rings of 16 rows: 512 pairs x 106 slots 10.5 / 7.9, 206
// 15.2 / 13.7, 2560 pairs x 106 35.4 / 30.1.
ShortForm short_form(const swa_params& p, int64_t pairs, int len_bound, bool ring)
{
    const bool fuse = (p.flags & SWA_FUSE_COMPACTION) != 0;
    if (fuse && !(p.flags & SWA_UNORDERED)) return {0, 0};
    if ((p.flags & SWA_HEAD_SHARED) && ring) return {0, 0};
    for (const ShortForm& f : kForms) {
        const int rows = short_rows(p, f);
        if (rows < len_bound) continue;
        const bool wide = f.nt == 512 || ((p.flags & SWA_KV_INT8) && f.nt == 256);
        return wide && pairs > 512 ? ShortForm{0, 0} : f;
    }
    return {0, 0};
}

template <typename T, int D, int NT, int U>
static int launch_short_f(const DecodeArgs& a, int64_t pairs, hipStream_t stream)
{
    if constexpr (short_rows<T, D, NT, U>() > 0) {
        if (a.ring) hipLaunchKernelGGL((swa_short_kernel<T, D, NT, U, true, 0>), dim3((unsigned)pairs), dim3(NT), 0, stream, a);
        else hipLaunchKernelGGL((swa_short_kernel<T, D, NT, U, false, 0>), dim3((unsigned)pairs), dim3(NT), 0, stream, a);
        return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
    }
    return SWA_ERR_BAD_SHAPE;          // (short_form names no such form)
}

template <typename T, int D>
static int launch_short_t(const DecodeArgs& a, int64_t pairs, ShortForm f, hipStream_t stream)
{
    if (f.nt == 128) return launch_short_f<T, D, 128, short_unroll<T, D>(8)>(a, pairs, stream);
    if (f.nt == 512) return launch_short_f<T, D, 512, short_unroll<T, D>(8)>(a, pairs, stream);
    if (f.u == 12) return launch_short_f<T, D, 256, short_unroll<T, D>(12)>(a, pairs, stream);
    return launch_short_f<T, D, 256, short_unroll<T, D>(8)>(a, pairs, stream);
}

int launch_short(const DecodeArgs& a, const swa_params& p, int64_t pairs, ShortForm f, hipStream_t stream)
{
    if (p.flags & SWA_KV_INT8)
        return p.d == 64 ? launch_short_t<Q8, 64>(a, pairs, f, stream) : launch_short_t<Q8, 128>(a, pairs, f, stream);
    if (p.dtype == SWA_F32)
        return p.d == 64 ? launch_short_t<F32, 64>(a, pairs, f, stream) : launch_short_t<F32, 128>(a, pairs, f, stream);
    if (p.dtype == SWA_F16)
        return p.d == 64 ? launch_short_t<F16, 64>(a, pairs, f, stream) : launch_short_t<F16, 128>(a, pairs, f, stream);
    return p.d == 64 ? launch_short_t<BF16, 64>(a, pairs, f, stream) : launch_short_t<BF16, 128>(a, pairs, f, stream);
}

}  // namespace swa
