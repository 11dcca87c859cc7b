// Decode step with one pair's rows split over several workgroups (SWA_SPLIT_ROWS): for few
// (sequence, head) pairs with long caches - small batches, long contexts, caches that are compacted
// rarely or never - one workgroup per pair cannot keep the memory system busy.  The step then runs
// as three launches:
//   1. swa_split_logits_kernel   G workgroups per pair: logits q . k_i * scale of a slice of the
//                                cached keys (Eq. 1 numerator), written to the workspace;
//   2. swa_split_select_kernel   one workgroup per pair: append, softmax over the stored logits,
//                                importance accumulation, budget and selection (Alg. 1 lines 1-5),
//                                kept list and the kept tokens' weights to memory;
//   3. swa_split_gather_kernel   one workgroup per pair and 64 bytes of a row: out = sum p_i v_i / sum p_i
//                                over the kept list (Alg. 1 lines 6-8), rounded once to the output type.
// The logits are formed exactly as the one-workgroup kernel forms them (same products, same
// reduction order), so weights, importance and the kept set are bit-identical to that form; only
// the order in which the output's partial sums are added differs.
#include "swa_kernels.hpp"
#include "swa_select.hpp"

namespace swa {

struct SplitArgs {
    const char* q;
    const char* k_new;
    const char* v_new;
    char* k_cache;
    char* v_cache;
    float* score;
    int32_t* pos;
    int32_t* cache_len;
    const int32_t* seq_len;
    int32_t* kept_idx;
    int32_t* kept_cnt;
    float* probs_dbg;
    int32_t* status;
    int32_t* arrive;
    float* ws_z;        // [pairs, cap] logits
    float* ws_p;        // [pairs, cap] weights of the kept tokens, in the order of the kept list
    int32_t* ws_ok;     // [pairs] 1 once launch 2 has finished the pair's step (0: skipped, cache full)
    char* out;
    int64_t pairs;
    int32_t h, cap, G;
    int32_t w, sparsity_bp, lds_slots;
    float scale;
};

constexpr int kSelThreads = 1024;    // launch 2: a whole CU's worth of one pair
constexpr int kGatherThreads = 1024;
constexpr int kPieceBytes = 128;     // of a value row, per workgroup of launch 3
constexpr int kXcds = 8;             // workgroups are dealt round-robin to the 8 XCDs, each with its own L2
constexpr int kSelPer = SWA_MAX_CAP / kSelThreads;   // slots per thread at most

// Launch 1.  cache_len is the length BEFORE the step's append; slot `len` is the new token, whose
// key comes from k_new (launch 2 writes it to the cache).
template <typename T, int D, int NT>
__global__ void __launch_bounds__(NT) swa_split_logits_kernel(SplitArgs a)
{
    constexpr int EPV = Elem<T>::kPerVec;
    constexpr int LPR = D / EPV;
    constexpr int NG = NT / LPR;
    constexpr int ROWB = D * Elem<T>::kBytes;
    constexpr int UK = 8;
    const int tid = threadIdx.x;
    const int sub = tid % LPR;
    const int grp = tid / LPR;
    const int64_t pair = blockIdx.x / a.G;
    const int g = blockIdx.x % a.G;
    const int s = (int)(pair / a.h);
    const int len = a.cache_len[s];
    const int m = len + 1;
    if (g == 0 && tid == 0) a.ws_ok[pair] = 0;         // launch 2 sets it when it completes the pair
    if (len < 0 || m > a.cap) return;                  // launch 2 reports the full cache
    const int per = (m + a.G - 1) / a.G;
    const int lo = g * per;
    const int hi = lo + per < m ? lo + per : m;
    const char* Kp = a.k_cache + pair * (int64_t)a.cap * ROWB;
    float* Zp = a.ws_z + pair * (int64_t)a.cap;
    QFrag<T> qf;
    qf.load(load16(a.q + pair * ROWB + sub * 16));
    const Vec16 nk = load16(a.k_new + pair * ROWB + sub * 16);
    for (int base = lo; base < hi; base += NG * UK) {
        Vec16 kv[UK];
#pragma unroll
        for (int u = 0; u < UK; ++u) {
            const int row = base + u * NG + grp;
            kv[u] = (row < len && row < hi) ? load16_stream(Kp + (int64_t)row * ROWB + sub * 16) : nk;
        }
#pragma unroll
        for (int u = 0; u < UK; ++u) {
            const int row = base + u * NG + grp;
            const float d = group_sum<LPR>(qf.dot(kv[u], 0.f)) * a.scale;
            if (sub == 0 && row < hi) Zp[row] = d;
        }
    }
}

// Launch 2.  Softmax over the stored logits, importance, budget and selection of one pair; append of the new token.
//
// Bound: the dependent chain of one workgroup (a few pairs on 256 CUs), so every load of the pair's logits and
// importance is requested at once, keys stay in registers between the phases, and 1024 threads share the work.
// Weights are bit-identical to the one-workgroup kernel's: its 512 threads' sums are added up in its order.
// 32 pairs x 8192 rows, f16, d = 128: 17 us (33 with the one-workgroup kernel in this place).
template <typename T, int D>
__global__ void __launch_bounds__(kSelThreads) swa_split_select_kernel(SplitArgs a)
{
    constexpr int NT = kSelThreads;
    constexpr int NW = NT / kWave;
    constexpr int SUMT = 512;               // threads of the one-workgroup kernel on such caches
    constexpr int EPV = Elem<T>::kPerVec;
    constexpr int LPR = D / EPV;
    constexpr int ROWB = D * Elem<T>::kBytes;
    extern __shared__ __align__(16) char smem[];
    float* s_p = reinterpret_cast<float*>(smem);                       // exponentials, then weights
    uint32_t* s_key = reinterpret_cast<uint32_t*>(s_p + a.lds_slots);
    uint16_t* s_kept = reinterpret_cast<uint16_t*>(s_key);             // over the keys, once all of them are read
    __shared__ SelectScratch<NT> s_sel;
    __shared__ float s_red[NW];
    __shared__ float s_sum[SUMT / kWave];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t pair = blockIdx.x;
    const int s = (int)(pair / a.h);
    const int cap = a.cap;
    const int len = a.cache_len[s];
    const int n = a.seq_len[s];
    const int m = len + 1;
    const bool overflow = (m > cap) || (m > a.lds_slots) || (len < 0);
    int keep = 0, n_local = 0, n_global = 0, w_eff = 0;

    if (!overflow) {
        const float* Zp = a.ws_z + pair * (int64_t)cap;
        float* Sp = a.score + pair * (int64_t)cap;
        float* Wp = a.ws_p + pair * (int64_t)cap;
        float z[kSelPer], sc[kSelPer];
#pragma unroll
        for (int k = 0; k < kSelPer; ++k) {
            const int i = tid + k * NT;
            z[k] = i < m ? Zp[i] : -INFINITY;
            sc[k] = i < len ? Sp[i] : 0.f;
        }
        // append: the new row's key, value and position
        if (tid < 2 * LPR) {
            const int at = (tid % LPR) * 16;
            const char* row = tid < LPR ? a.k_new : a.v_new;
            store16((tid < LPR ? a.k_cache : a.v_cache) + (pair * (int64_t)cap + len) * ROWB + at, load16(row + pair * ROWB + at));
        }
        if (tid == 0) a.pos[pair * (int64_t)cap + len] = n - 1;

        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < kSelPer; ++k) mx = fmaxf(mx, z[k]);
        mx = wave_max(mx);
        if (lane == 0) s_red[wave] = mx;
        __syncthreads();
        mx = s_red[0];
#pragma unroll
        for (int v = 1; v < NW; ++v) mx = fmaxf(mx, s_red[v]);
#pragma unroll
        for (int k = 0; k < kSelPer; ++k) {
            const int i = tid + k * NT;
            if (i < m) {
                z[k] = expf(z[k] - mx);
                s_p[i] = z[k];
            }
        }
        __syncthreads();
        if (tid < SUMT) {
            float sum = 0.f;
            for (int i = tid; i < m; i += SUMT) sum += s_p[i];
            sum = wave_sum(sum);
            if (lane == 0) s_sum[wave] = sum;
        }
        __syncthreads();
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < SUMT / kWave; ++v) sum += s_sum[v];

        budget(n, m, a.w, a.sparsity_bp, keep, n_local, n_global, w_eff);
        const int ncand = m - n_local;
        uint32_t key[kSelPer];
#pragma unroll
        for (int k = 0; k < kSelPer; ++k) {
            const int i = tid + k * NT;
            key[k] = 0u;
            if (i < m) {
                const float p = z[k] / sum;
                const float v = sc[k] + p;
                Sp[i] = v;
                s_p[i] = p;
                key[k] = order_key(v);
                s_key[i] = key[k];
            }
        }
        if (a.probs_dbg) {
            __syncthreads();
            float* dbg = a.probs_dbg + pair * (int64_t)cap;
            for (int i = tid; i < cap; i += NT) dbg[i] = (i < m) ? s_p[i] : 0.f;
        }

        int32_t* kout = a.kept_idx + pair * (int64_t)cap;
        if (keep == m) {                                    // everything stays
            __syncthreads();
            for (int i = tid; i < m; i += NT) {
                kout[i] = i;
                Wp[i] = s_p[i];
            }
        } else {
            uint32_t thr = 0u;
            int rem = 0, n_eq = 0;
            if (n_global > 0) {
                auto each = [&](auto f) {
#pragma unroll
                    for (int k = 0; k < kSelPer; ++k)
                        if (tid + k * NT < ncand) f(key[k]);
                };
                select_threshold<NT>(s_sel, n_global, each, thr, rem, n_eq);
            } else {
                __syncthreads();
            }
            // every thread owns a run of slots; ties go to the lowest slots
            const int per = (m + NT - 1) / NT;
            const int lo = tid * per;
            const int hi = lo + per < m ? lo + per : m;
            uint64_t surem = 0ull, eqm = 0ull;
            for (int k = 0; lo + k < hi; ++k) {
                const int i = lo + k;
                if (i >= ncand) {
                    surem |= 1ull << k;
                } else if (n_global > 0) {
                    const uint32_t q = s_key[i];
                    if (q > thr) surem |= 1ull << k;
                    else if (q == thr) eqm |= 1ull << k;
                }
            }
            const uint64_t kept = keep_mask<NT>(s_sel.cnt, surem, eqm, rem);
            int at = 0, total = 0;
            block_scan<NT>(s_sel.cnt, (int)__popcll(kept), at, total);
            for (int k = 0; lo + k < hi; ++k)
                if ((kept >> k) & 1ull) s_kept[at++] = (uint16_t)(lo + k);
            __syncthreads();
            for (int j = tid; j < keep; j += NT) {
                const int i = s_kept[j];
                kout[j] = i;
                Wp[j] = s_p[i];
            }
        }
    }

    // per-sequence arrival: the last head to finish publishes the new length (every workgroup read it before)
    if (tid == 0) {
        if (overflow) {
            atomicOr(a.status, kStatusCapacityBit);
        } else {
            a.kept_cnt[s] = keep;
            a.ws_ok[pair] = 1;
        }
        const int old = atomicAdd(&a.arrive[s], 1);
        if (old == a.h - 1) {
            atomicExch(&a.arrive[s], 0);
            if (!overflow) a.cache_len[s] = m;
        }
    }
}

// Launch 3.  Output of one pair from its kept list, 128 bytes of the row per workgroup.
//
// Bound: what a CU can load (about 100 GB/s with random rows) and the launch's own latency.  Whole rows in slices of the list, or inside
// launch 2, would need either a fourth launch that adds the slices up or a choice by the number of kept rows, which
// the host does not know: a compacted cache or a wide window keeps many times the share that the sparsity
// names.  Channels need no sum across workgroups, whatever is kept.  64-byte pieces are 1 to 5 us faster with few pairs and much
// kept, but slower from about 96 pairs on (128 pairs x 8192 kept rows, whole step 118 against 102 us).
// Whole step, f16, d = 128, this form / partial sums and a fourth launch / output in launch 2, in us: 32 pairs, 20 of 2048 rows
// kept 20.6 / 26.3 / 19.4; 410 of 2048 23.2 / 28.8 / 23.1; all of 2048 21.4 / 28.2 / 33.3; 1638 of 8192 40.1 / 45.3 / 46.5; all
// of 8192 52.8 / 59.2 / 98; 128 pairs, all of 8192 102 / 130 / 136.
template <typename T, int D>
__global__ void __launch_bounds__(kGatherThreads) swa_split_gather_kernel(SplitArgs a)
{
    constexpr int NT = kGatherThreads;
    constexpr int NW = NT / kWave;
    constexpr int EPV = Elem<T>::kPerVec;
    constexpr int ROWB = D * Elem<T>::kBytes;
    constexpr int LPR = kPieceBytes / 16;         // lanes per piece of a row
    constexpr int PIECES = ROWB / kPieceBytes;
    constexpr int CH = LPR * EPV;                 // channels of a piece
    constexpr int NG = NT / LPR;
    constexpr int UV = 8;
    __shared__ float s_acc[NW * CH];
    __shared__ float s_ps[NW];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int sub = tid % LPR;
    const int grp = tid / LPR;
    // the pieces of a pair go to the XCD that ran its selection, next to each other: they share lines, list and weights
    const int64_t b = blockIdx.x / kXcds;
    const int piece = (int)(b % PIECES);
    const int64_t pair = b / PIECES * kXcds + blockIdx.x % kXcds;
    if (pair >= a.pairs || a.ws_ok[pair] == 0) return;          // (a skipped pair: nothing is written for it)
    int keep = a.kept_cnt[(int)(pair / a.h)];
    keep = keep < 0 ? 0 : (keep > a.cap ? a.cap : keep);
    const char* Vp = a.v_cache + pair * (int64_t)a.cap * ROWB + piece * kPieceBytes + sub * 16;
    const float* Wp = a.ws_p + pair * (int64_t)a.cap;
    const int32_t* idx = a.kept_idx + pair * (int64_t)a.cap;
    float acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
    float ps = 0.f;
    for (int j0 = 0; j0 < keep; j0 += NG * UV) {
        int i[UV];
        float pw[UV];
        Vec16 vv[UV];
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            const int j = j0 + u * NG + grp;
            i[u] = j < keep ? idx[j] : 0;
            pw[u] = j < keep ? Wp[j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            i[u] = i[u] < 0 ? 0 : (i[u] >= a.cap ? a.cap - 1 : i[u]);
            vv[u] = Vec16{0u, 0u, 0u, 0u};
            if (j0 + u * NG + grp < keep) vv[u] = load16_stream(Vp + (int64_t)i[u] * ROWB);
        }
#pragma unroll
        for (int u = 0; u < UV; ++u) {
            float f[EPV];
            unpack<T>(vv[u], f);
#pragma unroll
            for (int e = 0; e < EPV; ++e) acc[e] = __builtin_fmaf(pw[u], f[e], acc[e]);
            ps += pw[u];
        }
    }
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) acc[e] += __shfl_xor(acc[e], o, kWave);
        ps += __shfl_xor(ps, o, kWave);
    }
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) s_acc[wave * CH + sub * EPV + e] = acc[e];
        if (lane == 0) s_ps[wave] = ps;
    }
    __syncthreads();
    if (tid < CH) {
        float t = 0.f, pst = 0.f;
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            t += s_acc[v * CH + tid];
            pst += s_ps[v];
        }
        store_elem<T>(a.out + pair * ROWB, piece * CH + tid, keep > 0 ? t / pst : 0.f);   // an empty budget: an empty sum
    }
}

template <typename T, int D>
static int launch_split_t(const SplitArgs& a, int64_t pairs, hipStream_t stream)
{
    constexpr int NT = 256;
    const dim3 grid((unsigned)(pairs * a.G));
    hipLaunchKernelGGL((swa_split_logits_kernel<T, D, NT>), grid, dim3(NT), 0, stream, a);
    if (hipGetLastError() != hipSuccess) return SWA_ERR_HIP;
    auto sel = swa_split_select_kernel<T, D>;
    const size_t lds = (size_t)a.lds_slots * 8;
    const int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(sel), lds);
    if (rc != SWA_OK) return rc;
    hipLaunchKernelGGL(sel, dim3((unsigned)pairs), dim3(kSelThreads), lds, stream, a);
    if (hipGetLastError() != hipSuccess) return SWA_ERR_HIP;
    const int64_t pieces = (pairs + kXcds - 1) / kXcds * kXcds * (D * Elem<T>::kBytes / kPieceBytes);
    hipLaunchKernelGGL((swa_split_gather_kernel<T, D>), dim3((unsigned)pieces), dim3(kGatherThreads), 0, stream, a);
    return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
}

int launch_split(const swa_params& p, float scale, int G, const void* q, const void* k_new, const void* v_new, void* k_cache,
                 void* v_cache, float* score, int32_t* pos, int32_t* cache_len, const int32_t* seq_len, int32_t* kept_idx,
                 int32_t* kept_cnt, void* out, float* probs_dbg, void* workspace, hipStream_t stream)
{
    const int64_t pairs = (int64_t)p.b * p.h;
    const int bound = (p.len_bound > 0 && p.len_bound < p.cap) ? p.len_bound : p.cap;
    char* ws = static_cast<char*>(workspace);
    char* base = ws + shared_workspace_offset(p);
    const size_t slab = (size_t)pairs * p.cap * sizeof(float);
    SplitArgs a;
    a.q = static_cast<const char*>(q);
    a.k_new = static_cast<const char*>(k_new);
    a.v_new = static_cast<const char*>(v_new);
    a.k_cache = static_cast<char*>(k_cache);
    a.v_cache = static_cast<char*>(v_cache);
    a.score = score;
    a.pos = pos;
    a.cache_len = cache_len;
    a.seq_len = seq_len;
    a.kept_idx = kept_idx;
    a.kept_cnt = kept_cnt;
    a.out = static_cast<char*>(out);
    a.probs_dbg = probs_dbg;
    a.status = reinterpret_cast<int32_t*>(ws + kWsStatusOffset);
    a.arrive = reinterpret_cast<int32_t*>(ws + kWsArriveOffset);
    a.ws_z = reinterpret_cast<float*>(base);
    a.ws_p = reinterpret_cast<float*>(base + slab);
    a.ws_ok = reinterpret_cast<int32_t*>(base + 2 * slab);
    a.pairs = pairs;
    a.h = p.h;
    a.cap = p.cap;
    a.G = G;
    a.w = p.w;
    a.sparsity_bp = p.sparsity_bp;
    a.lds_slots = (bound + 63) & ~63;
    a.scale = scale;
    if (p.dtype == SWA_F32) {
        return p.d == 64 ? launch_split_t<F32, 64>(a, pairs, stream) : launch_split_t<F32, 128>(a, pairs, stream);
    } else if (p.dtype == SWA_F16) {
        return p.d == 64 ? launch_split_t<F16, 64>(a, pairs, stream) : launch_split_t<F16, 128>(a, pairs, stream);
    }
    return p.d == 64 ? launch_split_t<BF16, 64>(a, pairs, stream) : launch_split_t<BF16, 128>(a, pairs, stream);
}

template <typename T>
static int prepare_split_t()
{
    int rc = raise_dynamic_lds(reinterpret_cast<const void*>(swa_split_select_kernel<T, 64>));
    if (rc == SWA_OK) rc = raise_dynamic_lds(reinterpret_cast<const void*>(swa_split_select_kernel<T, 128>));
    return rc;
}

int prepare_split()
{
    int rc = prepare_split_t<F32>();
    if (rc == SWA_OK) rc = prepare_split_t<F16>();
    if (rc == SWA_OK) rc = prepare_split_t<BF16>();
    return rc;
}

}  // namespace swa
