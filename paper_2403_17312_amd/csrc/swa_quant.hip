// Channel-wise 8-bit compression of an fp16 KV cache (Section V-B): for every (sequence, head)
// pair and every channel, lambda = (max - min) / 255 over the cached tokens and the zero point
// z = nint(-min / lambda); then code = round(x / lambda + z) for every cached element.
// One workgroup per (pair, tensor, 64 channels): it reads its 128-byte row pieces once, finds the channel
// extrema, and quantises from registers.  Runs once, when the prompt's cache is handed over.
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
    int32_t h, cap;
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

// Bound: HBM (2 bytes read, 1 written per element).  A workgroup of NT threads keeps the first 16 * NT / 8 rows of its
// 64 channels in registers between the two passes (64 of a thread's registers; 64 channels are one 128-byte line of
// every row, and halving the rows' width lets two workgroups of 1024 rows share a CU, so that one loads while the other
// stores); rows beyond those are read again.
// 2560 pairs x 1024 rows x 128 channels, K and V: 0.68 -> 0.45 ms by the difference of whole passes (two reads of the cache and a division
// per element before).
template <int D, int NT>
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

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int sub = tid % LPR;
    const int grp = tid / LPR;
    // the pieces of one row go to the same XCD, next to each other: their codes share lines
    const int xcd = blockIdx.x % kXcds;
    const int i = blockIdx.x / kXcds;
    const int piece = i % PIECES;
    const int64_t in_row = (int64_t)(i / PIECES) * kXcds + xcd;
    const int64_t unit = (int64_t)blockIdx.y * a.units_x + in_row;
    if (in_row >= a.units_x || unit >= a.units) return;
    const int64_t pair = unit >> 1;
    const int which = (int)(unit & 1);
    const int s = (int)(pair / a.h);
    int len = a.cache_len[s];
    len = len < 0 ? 0 : (len > a.cap ? a.cap : len);
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
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) {
        Vec16 x = __builtin_bit_cast(Vec16, lo), y = __builtin_bit_cast(Vec16, hi);
        x = Vec16{(uint32_t)__shfl_xor((int)x.x, o, kWave), (uint32_t)__shfl_xor((int)x.y, o, kWave),
                  (uint32_t)__shfl_xor((int)x.z, o, kWave), (uint32_t)__shfl_xor((int)x.w, o, kWave)};
        y = Vec16{(uint32_t)__shfl_xor((int)y.x, o, kWave), (uint32_t)__shfl_xor((int)y.y, o, kWave),
                  (uint32_t)__shfl_xor((int)y.z, o, kWave), (uint32_t)__shfl_xor((int)y.w, o, kWave)};
        lo = __builtin_elementwise_min(lo, __builtin_bit_cast(half8_t, x));
        hi = __builtin_elementwise_max(hi, __builtin_bit_cast(half8_t, y));
    }
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
        if (len == 0) l = u = 0.f;
        float range = __fsub_rn(u, l);
        range = range < kMinRange ? kMinRange : range;
        const float lam = __fdiv_rn(range, 255.f);
        const float z = rintf(__fdiv_rn(-l, lam));
        s_lam[tid] = lam;
        s_inv[tid] = __fdiv_rn(1.f, lam);
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
    auto put = [&](int row, const Vec16& v) {
        float f[8];
        unpack<F16>(v, f);
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            // quantise_one() with the division above: one rounding per operation, ties to even, saturated (NaN: 0)
            float t = rintf(__fadd_rn(divide_by(f[e], lam[e], inv[e]), zero[e]));
            t = fminf(fmaxf(t, 0.f), 255.f);
            w[e >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(t, e & 3, w[e >> 2]);
        }
        *reinterpret_cast<uint2*>(dst + (int64_t)row * D) = make_uint2(w[0], w[1]);
    };
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
        if (grp + k * NG < len) put(grp + k * NG, keep[k]);
    for (int row = grp + KEEP * NG; row < len; row += NG) put(row, load16(src + (int64_t)row * ROWB));
}

template <int D>
static void launch_quantize_d(const QuantArgs& a, dim3 grid, hipStream_t stream)
{
    // as many threads as it takes to keep every row that fits the cache in registers, up to 2048 rows (a margin for
    // caches that are a little longer than their prompts)
    if (a.cap <= 576) hipLaunchKernelGGL((swa_quantize_kernel<D, 256>), grid, dim3(256), 0, stream, a);
    else if (a.cap <= 1280) hipLaunchKernelGGL((swa_quantize_kernel<D, 512>), grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL((swa_quantize_kernel<D, 1024>), grid, dim3(1024), 0, stream, a);
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
    a.h = p.h;
    a.cap = p.cap;
    a.units = (int64_t)p.b * p.h * 2;
    a.units_x = a.units < (1 << 20) ? a.units : (1 << 20);       // (a grid row holds fewer than 2^32 threads)
    const dim3 grid((unsigned)((a.units_x + 7) / 8 * 8 * (p.d / 64)), (unsigned)((a.units + a.units_x - 1) / a.units_x));
    if (p.d == 64) launch_quantize_d<64>(a, grid, stream);
    else launch_quantize_d<128>(a, grid, stream);
    return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
}

}  // namespace swa
