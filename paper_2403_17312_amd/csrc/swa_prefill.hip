// Prefill importance seed on MFMA: the local attention sum of Algorithm 1 line 2
// evaluated at the end of the prompt,
//   score[j] = sum_{r<R} softmax_causal(Q_tail K^T * scale)[r, j].
// One workgroup (4 waves) per (sequence, head) pair, or several, each with a slice of the keys, where there are few
// pairs.  The R x s logit tile is never stored: pass 1 computes every query row's max and normaliser, pass 2
// recomputes the logits and reduces exp(z - max_r) / sum_r over the rows.  After the prefill attention kernel, which
// knows those statistics, pass 2 runs alone: one read of the keys instead of two (64 x 32 pairs of 512..2048 keys,
// R = 32: 244 -> 163 us; 1792 pairs of 4096 keys, R = 64: 620 -> about 400 us, by the
// difference of whole calls).
//
// MFMA operand layout used here (32x32 tiles, wave64): lane l supplies row
// (l % 32) of its operand and the contiguous half-row (l / 32) of the head
// dimension; successive MFMA issues walk along that half-row.  Both operands
// use the same walk, so the contraction is over the whole head dimension
// whatever order the hardware sums in.  The 32x32 fp32 result gives lane l
// column (l % 32) and rows 8*(i/4) + 4*(l/32) + (i%4), i = 0..15.
//   pass 1: A = key tile,   B = query tile -> lane owns ONE query, 16 keys
//           (row statistics reduce inside the lane);
//   pass 2: A = query tile, B = key tile   -> lane owns ONE key, 16 queries
//           (column sums reduce inside the lane).
#include "swa_kernels.hpp"

namespace swa {

struct PrefillArgs {
    const char* q_tail;
    const char* k_cache;
    const int32_t* cache_len;
    float* score;   // column sums over the R rows, or NULL
    float* rows;    // [b,h,R,cap] the R rows themselves, or NULL
    int32_t h, cap, R;
    int32_t q_in_place;   // 0: q_tail is [b,h,R,d]; 1: it is the whole prompt's [b,h,cap,d] and the
                          //    R rows are the ones at positions cache_len-R .. cache_len-1
    float scale_log2e;
    // For the column sums the columns are cut into G slices of `cols` (a multiple of 32; the last one ends at cap), one
    // workgroup each.
    // A slice's first 2 R output columns (score, or row 0 of the ring) bring it the row statistics from the
    // launch before: maximum of row r at [r], normaliser at [R + r].
    int32_t G, cols;
    int32_t bound;        // on the lengths: where the slices are laid (host side)
    bool stated;          // the bound is the caller's, not the capacity (host side)
    int32_t row_tiles;    // statistics: workgroups per pair, one for every 32 query rows
};

// What one launch does.
constexpr int kSeedWhole = 0;   // both passes, one workgroup per pair
constexpr int kSeedStats = 1;   // row statistics of one pair, a copy for every slice
constexpr int kSeedSums = 2;    // column sums of one slice, from the statistics of whole rows

// Merge two (max, sum-of-exp2) pairs of disjoint key sets.
__device__ __forceinline__ void merge_stats(float& M, float& L, float M2, float L2)
{
    const float Mn = fmaxf(M, M2);
    if (Mn == -INFINITY) return;   // both empty
    const float a = (M == -INFINITY) ? 0.f : L * exp2f(M - Mn);
    const float b = (M2 == -INFINITY) ? 0.f : L2 * exp2f(M2 - Mn);
    M = Mn;
    L = a + b;
}

// WR: also write the R rows themselves (the ring of the strict local attention sum).
template <typename T, int D, int RT, bool WR, int MODE>
__global__ void __launch_bounds__(256) swa_prefill_kernel(PrefillArgs a)
{
    constexpr int NT = 256;
    constexpr int NW = NT / kWave;
    constexpr int ROWB = D * Elem<T>::kBytes;
    constexpr int NV = (ROWB / 2) / 16;   // 16-byte vectors per lane and tile row
    constexpr int RP = RT * 32;           // padded query rows

    __shared__ float s_m[NW][RP];
    __shared__ float s_l[NW][RP];
    __shared__ __align__(16) float s_M[RP];
    __shared__ __align__(16) float s_invL[RP];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int l32 = lane & 31;
    const int hb = lane >> 5;
    const int64_t pair = MODE == kSeedSums ? blockIdx.x / a.G : (MODE == kSeedStats ? blockIdx.x / a.row_tiles : blockIdx.x);
    const int rt0 = MODE == kSeedStats ? blockIdx.x % a.row_tiles : 0;     // first row tile of this workgroup
    const int g = MODE == kSeedSums ? blockIdx.x % a.G : 0;
    const int cap = a.cap;
    const int R = a.R;
    int s = a.cache_len[pair / a.h];
    s = s > cap ? cap : s;
    // the columns this workgroup owns; it reads the key tiles among them
    const int col0 = MODE == kSeedSums ? g * a.cols : 0;
    const int col1 = (MODE != kSeedSums || g == a.G - 1) ? cap : col0 + a.cols;
    float* Sp = a.score ? a.score + pair * (int64_t)cap : nullptr;
    float* Rp = WR ? a.rows + pair * (int64_t)R * cap : nullptr;

    if (s <= 0) {
        if (MODE == kSeedStats) return;
        if (Sp)
            for (int j = col0 + tid; j < col1; j += NT) Sp[j] = 0.f;
        if (Rp)
            for (int r = 0; r < R; ++r)
                for (int j = col0 + tid; j < col1; j += NT) Rp[(int64_t)r * cap + j] = 0.f;
        return;
    }
    float* St = MODE == kSeedWhole ? nullptr : (WR ? a.rows + pair * (int64_t)R * cap : a.score + pair * (int64_t)cap) + col0;

    const char* Kp = a.k_cache + pair * (int64_t)cap * ROWB;
    const int qbase = a.q_in_place ? s - R : 0;   // row index of query 0 (negative: rows before the prompt)
    const char* Qp = a.q_tail + pair * (int64_t)(a.q_in_place ? cap : R) * ROWB;

    // Lane (row, hb) supplies the 16-byte chunks 2v + hb, v = 0..NV-1, of its row: the two
    // half-wave lanes of a row read adjacent chunks, and query and key fragments use the same
    // walk, so every MFMA issue contracts matching slices of the head dimension.
    const int lane_off = hb * 16;

    // Query fragments stay in registers for both passes.  Rows >= R are zero.
    Vec16 qv[RT][NV];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int r = (rt0 + rt) * 32 + l32;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int qrow = qbase + r > 0 ? qbase + r : 0;          // rows before the prompt are masked below
            qv[rt][v] = (r < R) ? load16(Qp + (int64_t)qrow * ROWB + v * 32 + lane_off)
                                : Vec16{0u, 0u, 0u, 0u};
        }
    }

    const int tile0 = col0 / 32;
    const int tile1 = (s < col1 ? s : col1) > col0 ? ((s < col1 ? s : col1) + 31) / 32 : tile0;   // (col0 is a multiple of 32)
    const int t_off = s - R;   // query r sits at position t_off + r and sees keys 0..t_off+r

    // Unconditional tile load (rows past the end re-read the last row and are masked later), so
    // that the loads of the next tile can stay in flight while the current one is reduced.
    // Plain loads, not streaming ones: a lane takes 32 bytes of a line per instruction, so the line
    // has to survive in the cache between the instructions that consume it.
    auto load_tile = [&](int tile, Vec16(&kv)[NV]) {
        int krow = tile * 32 + l32;
        krow = krow < s ? krow : s - 1;
        krow = krow < 0 ? 0 : krow;
        const char* src = Kp + (int64_t)krow * ROWB + lane_off;
#pragma unroll
        for (int v = 0; v < NV; ++v) kv[v] = load16(src + v * 32);
    };

    if constexpr (MODE != kSeedSums) {
    // ------------------------------ pass 1: row statistics ------------------------------
    float M[RT], L[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        M[rt] = -INFINITY;
        L[rt] = 0.f;
    }
    auto stats_tile = [&](int tile, const Vec16(&kv)[NV]) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float16_t c;
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
            for (int v = 0; v < NV; ++v) c = Mfma<T>::run(kv[v], qv[rt][v], c);   // C[key][query]
            const int r = (rt0 + rt) * 32 + l32;
            const int tmax = (r < R) ? t_off + r : -1;   // last visible key of this lane's query
            float z[16];
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int key = tile * 32 + 8 * (i / 4) + 4 * hb + (i % 4);
                z[i] = (key <= tmax) ? c[i] * a.scale_log2e : -INFINITY;
                mx = fmaxf(mx, z[i]);
            }
            if (mx > -INFINITY) {
                const float Mn = fmaxf(M[rt], mx);
                float acc = L[rt] * __builtin_amdgcn_exp2f(M[rt] - Mn);   // 0 while M is -inf
#pragma unroll
                for (int i = 0; i < 16; ++i) acc += __builtin_amdgcn_exp2f(z[i] - Mn);
                M[rt] = Mn;
                L[rt] = acc;
            }
        }
    };
    if constexpr (MODE == kSeedStats) {
        // one workgroup has a CU to itself: three tiles per wave in flight while a fourth is reduced
        constexpr int AHEAD = 4;
        Vec16 kr[AHEAD][NV];
#pragma unroll
        for (int u = 0; u < AHEAD - 1; ++u) load_tile(tile0 + wave + u * NW, kr[u]);
        for (int tile = tile0 + wave; tile < tile1; tile += AHEAD * NW) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                load_tile(tile + (u + AHEAD - 1) * NW, kr[(u + AHEAD - 1) % AHEAD]);
                if (tile + u * NW < tile1) stats_tile(tile + u * NW, kr[u]);
            }
        }
    } else {
        Vec16 kA[NV], kB[NV];
        load_tile(tile0 + wave, kA);
        for (int tile = tile0 + wave; tile < tile1; tile += 2 * NW) {
            load_tile(tile + NW, kB);
            stats_tile(tile, kA);
            load_tile(tile + 2 * NW, kA);
            if (tile + NW < tile1) stats_tile(tile + NW, kB);
        }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const float M2 = __shfl_xor(M[rt], 32, kWave);
        const float L2 = __shfl_xor(L[rt], 32, kWave);
        merge_stats(M[rt], L[rt], M2, L2);
        if (hb == 0) {
            s_m[wave][rt * 32 + l32] = M[rt];
            s_l[wave][rt * 32 + l32] = L[rt];
        }
    }
    __syncthreads();
    if (tid < RP) {
        float Mt = s_m[0][tid], Lt = s_l[0][tid];
#pragma unroll
        for (int v = 1; v < NW; ++v) merge_stats(Mt, Lt, s_m[v][tid], s_l[v][tid]);
        if constexpr (MODE == kSeedStats) {
            const int r = rt0 * 32 + tid;
            if (r < R) {
                for (int g2 = 0; g2 < a.G; ++g2) {
                    St[g2 * a.cols + r] = Mt;
                    St[g2 * a.cols + R + r] = Lt;
                }
            }
        }
        const bool ok = Mt > -INFINITY && Lt > 0.f;
        s_M[tid] = ok ? Mt : 0.f;
        s_invL[tid] = ok ? 1.f / Lt : 0.f;
    }
    if constexpr (MODE == kSeedStats) return;
    __syncthreads();
    }
    if constexpr (MODE == kSeedSums) {
        if (tid < RP) {
            const bool row = tid < R && t_off + tid >= 0;
            const float Mt = row ? St[tid] : -INFINITY, Lt = row ? St[R + tid] : 0.f;
            const bool ok = Mt > -INFINITY && Lt > 0.f;
            s_M[tid] = ok ? Mt : 0.f;
            s_invL[tid] = ok ? 1.f / Lt : 0.f;
        }
        __syncthreads();          // read by everyone before the slice's columns are written
    }

    // ------------------------------ pass 2: column sums ---------------------------------
    auto colsum_tile = [&](int tile, const Vec16(&kv)[NV]) {
        const int key = tile * 32 + l32;
        float colsum = 0.f;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float16_t c;
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
            for (int v = 0; v < NV; ++v) c = Mfma<T>::run(qv[rt][v], kv[v], c);   // C[query][key]
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // the lane's rows 8g + 4hb .. +3 of this query tile: one 16-byte LDS read each
                const int r0 = rt * 32 + 8 * g + 4 * hb;
                const float4_t Mr = *reinterpret_cast<const float4_t*>(&s_M[r0]);
                const float4_t Ir = *reinterpret_cast<const float4_t*>(&s_invL[r0]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = r0 + j;
                    const bool vis = (r < R) && (key <= t_off + r);
                    const float p = __builtin_amdgcn_exp2f(c[4 * g + j] * a.scale_log2e - Mr[j]) * Ir[j];
                    colsum += vis ? p : 0.f;
                    if constexpr (WR) {
                        if (r < R && key < s) Rp[(int64_t)r * cap + key] = vis ? p : 0.f;
                    }
                }
            }
        }
        colsum += __shfl_xor(colsum, 32, kWave);
        if (Sp && hb == 0 && key < s) Sp[key] = colsum;
    };
    {
        Vec16 kA[NV], kB[NV];
        // the keys read last by pass 1 are read first here
        const int last = tile1 - 1 - wave;
        load_tile(last, kA);
        for (int tile = last; tile >= tile0; tile -= 2 * NW) {
            load_tile(tile - NW, kB);
            colsum_tile(tile, kA);
            load_tile(tile - 2 * NW, kA);
            if (tile - NW >= tile0) colsum_tile(tile - NW, kB);
        }
    }
    const int z0 = s > col0 ? s : col0;
    if (Sp)
        for (int j = z0 + tid; j < col1; j += NT) Sp[j] = 0.f;
    if (Rp)
        for (int r = 0; r < R; ++r)
            for (int j = z0 + tid; j < col1; j += NT) Rp[(int64_t)r * cap + j] = 0.f;
}

// Slices per pair for the column sums.  One workgroup per pair reads its keys twice at about 30 GB/s, and with few
// pairs most of the chip waits for it.  The statistics of 32 rows stay with one workgroup (their sum has an order, and the
// selection that follows can hang on its last bit), which then keeps twice as many loads in flight; the column
// sums are independent and get one workgroup per CU in all, over the columns up to the bound on the lengths (the last
// slice has the rest).  Every slice holds the row statistics and is about 256 keys long at least.
constexpr int kSeedGrid = 256;
static int seed_slices(int64_t pairs, int bound, int cap, int R, int& cols)
{
    const int least = 2 * R > 256 ? 2 * R : 256;
    int64_t G = (kSeedGrid + pairs - 1) / pairs;
    if (G > (bound + least - 1) / least) G = (bound + least - 1) / least;
    cols = (int)((bound + G - 1) / G + 31) / 32 * 32;
    if (cols < 2 * R) cols = (2 * R + 31) / 32 * 32;
    while (G > 1 && (G - 1) * cols + 2 * R > cap) --G;         // the last slice has room for the statistics as well
    return (int)G;
}

// Statistics and sliced sums in a launch each, or everything in one launch?  The statistics read the keys once per 32 rows, with
// one workgroup per 32 rows of a pair: two launches pay while those workgroups find a CU of their own and the keys
// are long enough for the second launch.  One / two launches in us, f16, d = 128, R = 64 (R = 16 and 128, the ring's
// rows, d = 64 and fp32 draw the line in the same places):
//    32 pairs   1024 keys 22 / 19, 2048 38 / 28, 4096 70 / 45, 8192 137 / 79
//    64 pairs   1024 keys 22 / 21, 2048 39 / 31, 8192 140 / 89
//   128 pairs   1024 keys 23 / 24, 2048 40 / 38, 4096 74 / 67, 8192 143 / 125
//   160 pairs   1024 keys 24 / 37, 4096 75 / 108, 8192 150 / 207
// With 65 to 128 pairs only under a stated bound: without one the slices are laid over the whole capacity, and prompts that fill
// a quarter of it lose more (128 pairs x 4096 keys in 16384 slots 77 / 87) than full ones gain.  Up to 64 pairs
// the gain is worth the risk: short prompts under a long bound lose 2 to 5 us (32 pairs x 32 keys 7 / 10).
bool seed_in_two(int64_t pairs, int bound, bool stated, int R)
{
    if (pairs <= 64) return bound >= 1024;
    return stated && pairs <= 128 && pairs * ((R + 31) / 32) <= 256 && bound >= 4096;
}

template <typename T, int D, int RT, bool WR>
static int launch_prefill_rt(PrefillArgs a, int64_t pairs, bool stats_ready, hipStream_t stream)
{
    const int G = seed_slices(pairs, a.bound, a.cap, a.R, a.cols);
    a.G = G;
    const dim3 one((unsigned)pairs), all((unsigned)(pairs * G));
    if (stats_ready) {
        hipLaunchKernelGGL((swa_prefill_kernel<T, D, RT, WR, kSeedSums>), all, dim3(256), 0, stream, a);
    } else if (G > 1 && seed_in_two(pairs, a.bound, a.stated, a.R)) {
        a.row_tiles = RT;
        hipLaunchKernelGGL((swa_prefill_kernel<T, D, 1, WR, kSeedStats>), dim3((unsigned)(pairs * RT)), dim3(256), 0, stream, a);
        if (hipGetLastError() != hipSuccess) return SWA_ERR_HIP;
        hipLaunchKernelGGL((swa_prefill_kernel<T, D, RT, WR, kSeedSums>), all, dim3(256), 0, stream, a);
    } else {
        hipLaunchKernelGGL((swa_prefill_kernel<T, D, RT, WR, kSeedWhole>), one, dim3(256), 0, stream, a);
    }
    return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
}

template <typename T, int D>
static int launch_prefill_t(const PrefillArgs& a, int64_t pairs, bool stats_ready, hipStream_t stream)
{
    const int rt = (a.R + 31) / 32;
    if (a.rows) {
        switch (rt) {
            case 1: return launch_prefill_rt<T, D, 1, true>(a, pairs, stats_ready, stream);
            case 2: return launch_prefill_rt<T, D, 2, true>(a, pairs, stats_ready, stream);
            default: return SWA_ERR_BAD_SHAPE;
        }
    }
    switch (rt) {
        case 1: return launch_prefill_rt<T, D, 1, false>(a, pairs, stats_ready, stream);
        case 2: return launch_prefill_rt<T, D, 2, false>(a, pairs, stats_ready, stream);
        case 3: return launch_prefill_rt<T, D, 3, false>(a, pairs, stats_ready, stream);
        case 4: return launch_prefill_rt<T, D, 4, false>(a, pairs, stats_ready, stream);
        default: return SWA_ERR_BAD_SHAPE;
    }
}

// Where swa_prefill_attention leaves the statistics of the prompt's last R rows for the sums: G copies, `cols` apart
// (G = 0: no room for them, the seed computes its own).
void seed_stats_place(int64_t pairs, int bound, int cap, int R, int& G, int& cols)
{
    cols = 0;
    G = (R > 0 && 2 * R <= cap) ? seed_slices(pairs, bound, cap, R, cols) : 0;
}

int launch_prefill(const swa_params& p, float scale, const void* q_tail, int32_t R, const void* k_cache,
                   const int32_t* cache_len, float* score, float* rows, bool q_in_place, bool stats_ready,
                   hipStream_t stream)
{
    PrefillArgs a;
    a.G = a.cols = a.row_tiles = 0;
    a.q_in_place = q_in_place ? 1 : 0;
    a.rows = rows;
    a.q_tail = static_cast<const char*>(q_tail);
    a.k_cache = static_cast<const char*>(k_cache);
    a.cache_len = cache_len;
    a.score = score;
    a.h = p.h;
    a.cap = p.cap;
    a.stated = p.len_bound > 0;
    a.bound = (p.len_bound > 0 && p.len_bound < p.cap) ? p.len_bound : p.cap;
    a.R = R;
    a.scale_log2e = scale * 1.44269504088896340736f;
    const int64_t pairs = (int64_t)p.b * p.h;
    if (p.dtype == SWA_F32) {
        return p.d == 64 ? launch_prefill_t<F32, 64>(a, pairs, stats_ready, stream) : launch_prefill_t<F32, 128>(a, pairs, stats_ready, stream);
    } else if (p.dtype == SWA_F16) {
        return p.d == 64 ? launch_prefill_t<F16, 64>(a, pairs, stats_ready, stream) : launch_prefill_t<F16, 128>(a, pairs, stats_ready, stream);
    } else {
        return p.d == 64 ? launch_prefill_t<BF16, 64>(a, pairs, stats_ready, stream) : launch_prefill_t<BF16, 128>(a, pairs, stats_ready, stream);
    }
}

}  // namespace swa
