// Channel-wise 8-bit compression of an fp16 KV cache (Section V-B): for every (sequence, head)
// pair and every channel, lambda = (max - min) / 255 over the cached tokens and the zero point
// z = nint(-min / lambda); then code = round(x / lambda + z) for every cached element.  Runs once, when
// the prompt's cache is handed over.  Two kernels: longer prompts are read once and kept in registers by large
// workgroups, short ones (where large workgroups would be mostly idle) are read twice by small ones.  The lengths are
// known on the device only, so both may be launched; each leaves the other's pairs alone.
#include "swa_kernels.hpp"

namespace swa {

struct QuantArgs {
    const char* src[2];   // fp16 K and V caches
    char* dst[2];         // code caches
    const int32_t* cache_len;
    float* qparams;       // lambda_K, z_K, lambda_V, z_V, each qstride values
    int64_t qstride;
    int64_t units;        // (pair, tensor): two per pair
    int64_t units_x;      // of them in one row of the grid
    int64_t items;        // 64-channel pieces of units, in the order that the longer prompts' kernel takes them
    int32_t b, h, cap;
    int32_t short_rows;   // prompts of up to this many rows are the short kernel's, longer ones the other's (-1: all)
};

constexpr float kMinRange = 0.0078125f;   // 2^-7: a flat channel still gets a non-zero scale

// x / lam correctly rounded, inv = 1 / lam correctly rounded: two steps of quotient += (x - quotient lam) inv, the
// remainder exact in an FMA.  The first makes the quotient faithful, the second rounds it correctly (Markstein's
// theorem; lam is at least 2^-7 / 255 and x comes from fp16, so nothing leaves the normal range).  Five
// operations instead of the eleven of a full division, which bounded the kernel.  Where lam is not finite
// the codes are 0 on either way.
__device__ __forceinline__ float divide_by(float x, float lam, float inv)
{
    float q = x * inv;
    q = __builtin_fmaf(__builtin_fmaf(-q, lam, x), inv, q);
    return __builtin_fmaf(__builtin_fmaf(-q, lam, x), inv, q);
}

// lambda, 1 / lambda and zero point of a channel with extrema l, u.
__device__ __forceinline__ void channel_params(float l, float u, int len, float& lam, float& inv, float& zero)
{
    if (len == 0) l = u = 0.f;
    float range = __fsub_rn(u, l);
    range = range < kMinRange ? kMinRange : range;
    lam = __fdiv_rn(range, 255.f);
    inv = __fdiv_rn(1.f, lam);
    zero = rintf(__fdiv_rn(-l, lam));
}

// Eight codes: quantise_one() with the division above, one rounding per operation, ties to even, saturated (NaN: 0).
__device__ __forceinline__ uint2 quantise_eight(const Vec16& v, const float (&lam)[8], const float (&inv)[8], const float (&zero)[8])
{
    float f[8];
    unpack<F16>(v, f);
    uint32_t w[2] = {0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float t = rintf(__fadd_rn(divide_by(f[e], lam[e], inv[e]), zero[e]));
        t = fminf(fmaxf(t, 0.f), 255.f);
        w[e >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(t, e & 3, w[e >> 2]);
    }
    return make_uint2(w[0], w[1]);
}

// Extrema of eight channels over the lanes of a wave that are a multiple of `first` apart.
__device__ __forceinline__ void wave_extrema(half8_t& lo, half8_t& hi, int first)
{
#pragma unroll
    for (int o = first; o < kWave; o <<= 1) {
        Vec16 x = __builtin_bit_cast(Vec16, lo), y = __builtin_bit_cast(Vec16, hi);
        x = Vec16{(uint32_t)__shfl_xor((int)x.x, o, kWave), (uint32_t)__shfl_xor((int)x.y, o, kWave),
                  (uint32_t)__shfl_xor((int)x.z, o, kWave), (uint32_t)__shfl_xor((int)x.w, o, kWave)};
        y = Vec16{(uint32_t)__shfl_xor((int)y.x, o, kWave), (uint32_t)__shfl_xor((int)y.y, o, kWave),
                  (uint32_t)__shfl_xor((int)y.z, o, kWave), (uint32_t)__shfl_xor((int)y.w, o, kWave)};
        lo = __builtin_elementwise_min(lo, __builtin_bit_cast(half8_t, x));
        hi = __builtin_elementwise_max(hi, __builtin_bit_cast(half8_t, y));
    }
}

// Short prompts: one small workgroup per (pair, tensor) with whole rows, read twice (the second time from the
// caches).  Bound: the latency of its few dependent phases, so what counts is how many workgroups a CU holds.
template <int D>
__global__ void __launch_bounds__(256) swa_quantize_short_kernel(QuantArgs a)
{
    constexpr int LPR = D / 8;        // lanes per row, 8 channels each
    constexpr int NG = 256 / LPR;     // row groups
    constexpr int NW = 256 / kWave;
    constexpr int ROWB = D * 2;
    __shared__ float s_lo[NW][D];
    __shared__ float s_hi[NW][D];
    __shared__ __align__(16) float s_lam[D];
    __shared__ __align__(16) float s_inv[D];
    __shared__ __align__(16) float s_zero[D];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int sub = tid % LPR;
    int grp = tid / LPR;
    const int64_t unit = (int64_t)blockIdx.y * a.units_x + blockIdx.x;
    if (unit >= a.units) return;
    const int64_t pair = unit >> 1;
    const int which = (int)(unit & 1);
    int len = a.cache_len[(int)(pair / a.h)];
    len = len < 0 ? 0 : (len > a.cap ? a.cap : len);
    if (len > a.short_rows) return;
    const char* src = a.src[which] + pair * (int64_t)a.cap * ROWB + sub * 16;
    char* dst = a.dst[which] + pair * (int64_t)a.cap * D + sub * 8;

    half8_t lo, hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lo[e] = (_Float16)INFINITY;
        hi[e] = (_Float16)-INFINITY;
    }
#pragma unroll 4
    for (int row = grp; row < len; row += NG) {
        const half8_t v = __builtin_bit_cast(half8_t, load16(src + (int64_t)row * ROWB));
        lo = __builtin_elementwise_min(lo, v);
        hi = __builtin_elementwise_max(hi, v);
    }
    wave_extrema(lo, hi, LPR);
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            s_lo[wave][sub * 8 + e] = (float)lo[e];
            s_hi[wave][sub * 8 + e] = (float)hi[e];
        }
    }
    __syncthreads();
    if (tid < D) {
        float l = INFINITY, u = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            l = fminf(l, s_lo[w][tid]);
            u = fmaxf(u, s_hi[w][tid]);
        }
        float lam, inv, z;
        channel_params(l, u, len, lam, inv, z);
        s_lam[tid] = lam;
        s_inv[tid] = inv;
        s_zero[tid] = z;
        a.qparams[(2 * which) * a.qstride + pair * D + tid] = lam;
        a.qparams[(2 * which + 1) * a.qstride + pair * D + tid] = z;
    }
    __syncthreads();
    float lam[8], inv[8], zero[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lam[e] = s_lam[sub * 8 + e];
        inv[e] = s_inv[sub * 8 + e];
        zero[e] = s_zero[sub * 8 + e];
    }
#pragma unroll 2
    for (int row = grp; row < len; row += NG)
        *reinterpret_cast<uint2*>(dst + (int64_t)row * D) = quantise_eight(load16(src + (int64_t)row * ROWB), lam, inv, zero);
}

// Longer prompts.  Bound: HBM (2 bytes read, 1 written per element).  A workgroup of NT threads keeps the first 16 * NT / 8
// rows of its 64 channels in registers between the two passes (64 of a thread's registers; 64 channels are one
// 128-byte line of every row, and halving the rows' width lets two workgroups of 1024 rows share a CU, so that one
// loads while the other stores); rows beyond those are read again.
// 2560 pairs x 1024 rows x 128 channels, K and V: 0.46 ms (0.69 with two reads of the cache and a division per element).
// NARROW: fewer workgroups than items, each taking several in turn, after a look at whether there is anything
// to do; up to 15 % slower on long prompts (0.52 ms), and 2 to 4 us instead of 10 to 20 where every prompt is short.
template <int D, int NT, bool NARROW>
__global__ void __launch_bounds__(NT) swa_quantize_kernel(QuantArgs a)
{
    constexpr int LPR = 8;            // lanes per 128-byte piece of a row, 8 channels each
    constexpr int NG = NT / LPR;      // row groups
    constexpr int NW = NT / kWave;
    constexpr int ROWB = D * 2;
    constexpr int PIECES = D / 64;
    constexpr int KEEP = 16;          // row pieces a thread keeps
    constexpr int kXcds = 8;
    __shared__ float s_lo[NW][64];
    __shared__ float s_hi[NW][64];
    __shared__ __align__(16) float s_lam[64];
    __shared__ __align__(16) float s_inv[64];
    __shared__ __align__(16) float s_zero[64];

    if constexpr (NARROW) {
        int any = 0;
        for (int i = threadIdx.x; i < a.b; i += NT) any |= a.cache_len[i] > a.short_rows ? 1 : 0;
        if (!__syncthreads_or(any)) return;
    }
    for (uint64_t item = blockIdx.x; item < (uint64_t)a.items; item += gridDim.x) {
    int tid = threadIdx.x;
    if constexpr (NARROW) asm volatile("" : "+v"(tid));       // addresses are computed in every round, not kept in registers
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int sub = tid % LPR;
    int grp = tid / LPR;
    // the pieces of one row go to the same XCD, next to each other: their codes share lines
    const uint64_t i = item / kXcds;
    const int piece = (int)(i % PIECES);
    const uint64_t unit = i / PIECES * kXcds + item % kXcds;
    if (unit >= (uint64_t)a.units) {
        if (NARROW) continue;
        return;
    }
    const int64_t pair = (int64_t)(unit >> 1);
    const int which = (int)(unit & 1);
    const int s = (int)((uint32_t)pair / (uint32_t)a.h);       // (2^32 pairs would not fit the memory)
    int len = a.cache_len[s];
    len = len < 0 ? 0 : (len > a.cap ? a.cap : len);
    if (len <= a.short_rows) {
        if (NARROW) continue;
        return;
    }
    const char* src = a.src[which] + pair * (int64_t)a.cap * ROWB + piece * 128 + sub * 16;
    char* dst = a.dst[which] + pair * (int64_t)a.cap * D + piece * 64 + sub * 8;

    Vec16 keep[KEEP];
    half8_t lo, hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lo[e] = (_Float16)INFINITY;
        hi[e] = (_Float16)-INFINITY;
    }
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        if (k * NG < len) {                       // uniform; a thread past the end repeats the last row
            const int row = grp + k * NG < len ? grp + k * NG : len - 1;
            keep[k] = load16_stream(src + (int64_t)row * ROWB);
        } else if constexpr (NARROW) {
            keep[k] = Vec16{0u, 0u, 0u, 0u};      // (so that nothing is carried from item to item)
        }
    }
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        if (k * NG < len) {
            lo = __builtin_elementwise_min(lo, __builtin_bit_cast(half8_t, keep[k]));
            hi = __builtin_elementwise_max(hi, __builtin_bit_cast(half8_t, keep[k]));
        }
    }
    for (int row = grp + KEEP * NG; row < len; row += NG) {
        const half8_t v = __builtin_bit_cast(half8_t, load16(src + (int64_t)row * ROWB));
        lo = __builtin_elementwise_min(lo, v);
        hi = __builtin_elementwise_max(hi, v);
    }
    wave_extrema(lo, hi, LPR);
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            s_lo[wave][sub * 8 + e] = (float)lo[e];
            s_hi[wave][sub * 8 + e] = (float)hi[e];
        }
    }
    __syncthreads();
    if (tid < 64) {
        float l = INFINITY, u = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            l = fminf(l, s_lo[w][tid]);
            u = fmaxf(u, s_hi[w][tid]);
        }
        float lam, inv, z;
        channel_params(l, u, len, lam, inv, z);
        s_lam[tid] = lam;
        s_inv[tid] = inv;
        s_zero[tid] = z;
        a.qparams[(2 * which) * a.qstride + pair * D + piece * 64 + tid] = lam;
        a.qparams[(2 * which + 1) * a.qstride + pair * D + piece * 64 + tid] = z;
    }
    __syncthreads();
    float lam[8], inv[8], zero[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lam[e] = s_lam[sub * 8 + e];
        inv[e] = s_inv[sub * 8 + e];
        zero[e] = s_zero[sub * 8 + e];
    }
    if constexpr (NARROW) asm volatile("" : "+v"(grp));
    auto put = [&](int row, const Vec16& v) {
        *reinterpret_cast<uint2*>(dst + (int64_t)row * D) = quantise_eight(v, lam, inv, zero);
    };
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
        if (grp + k * NG < len) put(grp + k * NG, keep[k]);
    for (int row = grp + KEEP * NG; row < len; row += NG) put(row, load16(src + (int64_t)row * ROWB));
    if (!NARROW) return;
    }
}

template <int D, int NT, int RESIDENT>
static void launch_longer(const QuantArgs& a, bool stated, hipStream_t stream)
{
    const dim3 one((unsigned)a.items);
    if constexpr (RESIDENT > 0) {
        if (!stated && a.items > RESIDENT) {
            launch_kernel((swa_quantize_kernel<D, NT, true>), dim3((unsigned)RESIDENT), dim3(NT), 0, stream, a);
            return;
        }
    }
    launch_kernel((swa_quantize_kernel<D, NT, false>), one, dim3(NT), 0, stream, a);
}

// `stated`: the caller's bound on the lengths, or 0.
//
// Threads: as many as it takes to keep every row in registers, up to 2048 rows (with a margin where only the capacity is
// known, which is often a little above the prompts).  The line between the two kernels, each measured alone, d = 128,
// short / longer in us:
//   NT = 256   512 pairs x 128 rows 13.5 / 16.2, 256 rows 27 / 27;    2560 pairs x 128 rows 65 / 62, 256 rows 134 / 98
//   NT = 512   512 pairs x 256 rows 27 / 32, 512 rows 50 / 51;        2560 pairs x 256 rows 136 / 131, 320 rows 172 / 152
//   NT = 1024  512 pairs x 512 rows 52 / 64, 1024 rows 121 / 105;     2560 pairs x 400 rows 222 / 248, 512 rows 301 / 280
// Where the chip holds all pieces at once (few pairs) latency decides and the longer prompts' kernel serves all lengths
// (64 pairs: 16 rows 3.7 / 4.7, 64 rows 4.7 / 5.0, 128 rows 6.2 / 5.4, 256 rows 9.3 / 6.5).
// A stated bound says that some prompt is about that long, so the longer prompts' kernel gets one workgroup per
// piece, and the other is left out up to eight rounds of the chip (2 us of 90 at 512 pairs x 1024 rows).  Without one the
// longer prompts' kernel may find nothing to do (every prompt short, in a large cache) and comes with a narrow grid,
// 4 rounds of the chip at NT = 512 and 1 at 1024 (in us, 2560 pairs: 16 rows in caches of 1088 17, of 2112 16, with one
// workgroup per piece 22 and 33, without this launch 13; 1024 rows in 1088 516, with one workgroup per piece 463).
template <int D>
static void launch_quantize_d(QuantArgs a, int stated, hipStream_t stream)
{
    const int nt = (a.cap <= 576 || (stated && stated <= 385)) ? 256 : ((a.cap <= 1280 || (stated && stated <= 1025)) ? 512 : 1024);
    const int line = nt == 256 ? 112 : (nt == 512 ? 256 : 448);
    const int bound = stated && stated < a.cap ? stated : a.cap;
    if (a.items * nt <= (stated ? 8 : 1) * 256 * 1024 && bound > 64) a.short_rows = -1;
    else if (bound <= 64 || (stated && bound <= line)) a.short_rows = a.cap;
    else a.short_rows = line;
    if (a.short_rows >= 0) {
        const dim3 grid((unsigned)a.units_x, (unsigned)((a.units + a.units_x - 1) / a.units_x));
        launch_kernel((swa_quantize_short_kernel<D>), grid, dim3(256), 0, stream, a);
        if (a.short_rows >= a.cap) return;
    }
    if (nt == 256) launch_longer<D, 256, 0>(a, stated > 0, stream);
    else if (nt == 512) launch_longer<D, 512, 4 * 512>(a, stated > 0, stream);
    else launch_longer<D, 1024, 256>(a, stated > 0, stream);
}

int launch_quantize(const swa_params& p, const void* k_cache, const void* v_cache, const int32_t* cache_len,
                    void* k_codes, void* v_codes, float* qparams, hipStream_t stream)
{
    QuantArgs a;
    a.src[0] = static_cast<const char*>(k_cache);
    a.src[1] = static_cast<const char*>(v_cache);
    a.dst[0] = static_cast<char*>(k_codes);
    a.dst[1] = static_cast<char*>(v_codes);
    a.cache_len = cache_len;
    a.qparams = qparams;
    a.qstride = (int64_t)p.b * p.h * p.d;
    a.b = p.b;
    a.h = p.h;
    a.cap = p.cap;
    a.units = (int64_t)p.b * p.h * 2;
    a.units_x = a.units < (1 << 20) ? a.units : (1 << 20);       // (a grid row holds fewer than 2^32 threads)
    a.items = (a.units + 7) / 8 * 8 * (p.d / 64);
    if (p.d == 64) launch_quantize_d<64>(a, p.len_bound, stream);
    else launch_quantize_d<128>(a, p.len_bound, stream);
    return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
}

}  // namespace swa
