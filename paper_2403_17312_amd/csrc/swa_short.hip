// Which calls the kernel for caches of few slots serves, and its launches (swa_short.hpp; the head-shared step's two are in
// swa_short_shared.hip).
#include "swa_short.hpp"

namespace swa {

// The forms: threads per workgroup and rows per lane.
constexpr ShortForm kForms[] = {{128, 8}, {256, 8}, {256, 12}, {512, 8}};

namespace {
struct Rows {
    template <typename T, int D, int NT, int U>
    int go() const { return short_rows<T, D, NT, U>(); }
};
}  // namespace

// Which calls: the two-call form and unordered compaction (in token order rows shift by way of LDS; the strict window together
// with head-shared selection is left to the streaming kernel), with a bound on the lengths that a form covers; the smallest
// form that does.
// Streaming kernel / this one, us a step, f16 unless stated, d = 128, one token evicted:
//      32 pairs   106 slots 7.0 / 5.0,  140  7.6 / 5.4,  206  8.4 / 6.2;  8-bit 206  8.6 / 7.2
//     512 pairs    64 slots 7.2 / 5.3,  106  7.9 / 6.5,  140  9.4 / 8.5,  206 12.3 / 12.0;  8-bit 106  8.5 / 7.3,  206 10.1 / 9.3
//    1024 pairs   106 slots 12.9 / 11.3,  140 16.0 / 15.1,  206 21.3 / 21.2;  8-bit 206 14.5 / 15.9
//    2560 pairs    32 slots 16.2 / 9.8,  106 26.6 / 23.9,  140 32.9 / 32.1,  206 46.6 / 47.1;  8-bit 106 20.2 / 17.9,  206 30.4 / 30.7
//    8192 pairs   106 slots 77 / 75,  160 112 / 110
// The narrower rows and fp32, streaming kernel / this one (fp32, d = 128 has no form beyond 128 slots):
//      32 pairs   64 slots f16, d = 64 6.0 / 4.4, fp32, d = 64 5.8 / 4.3, fp32, d = 128 6.8 / 5.4,  128  6.1 / 5.0, 6.8 / 5.6, 8.5 / 6.5,
//                256 7.2 / 6.2, 8.4 / 7.0;  8-bit, d = 64  64 7.3 / 5.2,  256 7.7 / 6.6;  strict window, f16, d = 64  64 8.0 / 6.4,  256 9.5 / 7.9
//     512 pairs   64 7.6 / 6.1, 8.0 / 6.8, 10.5 / 9.0,  128  8.7 / 7.4, 10.6 / 9.3, 15.3 / 13.8,  256 11.2 / 10.0, 15.4 / 14.1;
//                8-bit  64 9.3 / 7.0,  256 10.7 / 9.7
//    2560 pairs   64 18.1 / 12.9, 20.1 / 16.3, 32.3 / 30.6,  128  20.9 / 17.4, 30.8 / 29.6,  256 31.9 / 30.7 (f16);  8-bit  64 17.1 / 12.5
//    8192 pairs   64 45 / 29, 53 / 47, 96 / 96,  128  55 / 48, 93 / 91,  256 94 / 92 (f16);  8-bit  128 41 / 33;  strict window  256 124 / 120
// The forms that fill half a CU with one workgroup (512 threads, and 256 on the 8-bit cache, whose lanes hold
// 16 channels) pay while the chip is not full of workgroups; the strict window, rings of 16 rows: 512 pairs x 106 slots 10.5 / 7.9, 206
// 15.2 / 13.7, 2560 pairs x 106 35.4 / 30.1.
ShortForm short_form(const swa_params& p, int64_t pairs, int len_bound, bool ring)
{
    const bool fuse = (p.flags & SWA_FUSE_COMPACTION) != 0;
    if (fuse && !(p.flags & SWA_UNORDERED)) return {0, 0};
    if ((p.flags & SWA_HEAD_SHARED) && ring) return {0, 0};
    for (const ShortForm& f : kForms) {
        const int rows = with_form(p, f, Rows{});
        if (rows < len_bound) continue;
        const bool wide = f.nt == 512 || ((p.flags & SWA_KV_INT8) && f.nt == 256);
        return wide && pairs > 512 ? ShortForm{0, 0} : f;
    }
    return {0, 0};
}

namespace {
struct Launch {
    const DecodeArgs& a;
    int64_t pairs;
    hipStream_t stream;

    template <typename T, int D, int NT, int U>
    int go() const
    {
        if constexpr (short_rows<T, D, NT, U>() > 0) {
            if (a.ring) launch_kernel((swa_short_kernel<T, D, NT, U, true, 0>), dim3((unsigned)pairs), dim3(NT), 0, stream, a);
            else launch_kernel((swa_short_kernel<T, D, NT, U, false, 0>), dim3((unsigned)pairs), dim3(NT), 0, stream, a);
            return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
        }
        return SWA_ERR_BAD_SHAPE;          // (short_form names no such form)
    }
};
}  // namespace

int launch_short(const DecodeArgs& a, const swa_params& p, int64_t pairs, ShortForm f, hipStream_t stream)
{
    return with_form(p, f, Launch{a, pairs, stream});
}

}  // namespace swa
