// Decode step with one pair's rows split over several workgroups (SWA_SPLIT_ROWS): for few
// (sequence, head) pairs with long caches - small batches, long contexts, caches that are compacted
// rarely or never - one workgroup per pair cannot keep the memory system busy.  The step then runs
// as three launches:
//   1. swa_split_logits_kernel   G workgroups per pair: logits q . k_i * scale of a slice of the
//                                cached keys (Eq. 1 numerator), written to the workspace;
//   2. swa_split_select_kernel   one workgroup per pair: append, softmax over the stored logits,
//                                importance accumulation, budget and selection (Alg. 1 lines 1-5),
//                                kept list and the kept tokens' weights to memory;
//   3. swa_split_gather_kernel   one workgroup per pair and 64 or 128 bytes of a row: out = sum p_i v_i / sum p_i
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
    int32_t w, sparsity_bp, lds_slots, row_bytes;
    float scale;
};

constexpr int kSelThreads = 1024;    // launch 2: a whole CU's worth of one pair
constexpr int kGatherThreads = 1024;
constexpr int kXcds = 8;             // workgroups are dealt round-robin to the 8 XCDs, each with its own L2
constexpr int kSelPer = SWA_MAX_CAP / kSelThreads;   // slots per thread of launch 2 at most

// Launch 1.  cache_len is the length BEFORE the step's append; slot `len` is the new token, whose
// key comes from k_new (launch 2 writes it to the cache).
//
// Bound: HBM, and the time until the first rows arrive.  A stage's rows are reduced while the next one's travel, and the new token
// does not lengthen a slice (32 pairs x 8192 rows, f16, d = 128: 15.8 -> 13.5 us, 5.0 TB/s).
template <typename T, int D, int NT>
__global__ void __launch_bounds__(NT) swa_split_logits_kernel(SplitArgs a)
{
    constexpr int EPV = Elem<T>::kPerVec;
    constexpr int LPR = D / EPV;
    constexpr int NG = NT / LPR;
    constexpr int ROWB = D * Elem<T>::kBytes;
    constexpr int UK = 8;                              // rows per lane and stage; two stages are in flight
    const int tid = threadIdx.x;
    const int sub = tid % LPR;
    const int grp = tid / LPR;
    const int64_t pair = blockIdx.x / a.G;
    const int g = blockIdx.x % a.G;
    const int s = (int)(pair / a.h);
    const int len = a.cache_len[s];
    if (g == 0 && tid == 0) a.ws_ok[pair] = 0;         // launch 2 sets it when it completes the pair
    if (len < 0 || len >= a.cap) return;                 // launch 2 reports the full cache
    const int per = (len + a.G - 1) / a.G;
    const int lo = g * per;
    const int hi = lo + per < len ? lo + per : len;
    const char* Kp = a.k_cache + pair * (int64_t)a.cap * ROWB;
    float* Zp = a.ws_z + pair * (int64_t)a.cap;
    QFrag<T> qf;
    qf.load(load16(a.q + pair * ROWB + sub * 16));
    // (rows past the end re-read the slice's last one)
    auto request = [&](int base, Vec16(&kv)[UK]) {
#pragma unroll
        for (int u = 0; u < UK; ++u) {
            const int row = base + u * NG + grp;
            kv[u] = load16_stream(Kp + (uint32_t)(row < hi ? row : hi - 1) * ROWB + sub * 16);
        }
    };
    auto reduce = [&](int base, const Vec16(&kv)[UK]) {
#pragma unroll
        for (int u = 0; u < UK; ++u) {
            const int row = base + u * NG + grp;
            const float d = group_sum<LPR>(qf.dot(kv[u], 0.f)) * a.scale;
            if (sub == 0 && row < hi) Zp[row] = d;
        }
    };
    constexpr int STEP = NG * UK;
    Vec16 kA[UK], kB[UK];
    if (lo < hi) request(lo, kA);
    for (int base = lo; base < hi; base += 2 * STEP) {
        if (base + STEP < hi) request(base + STEP, kB);
        reduce(base, kA);
        if (base + STEP >= hi) break;
        if (base + 2 * STEP < hi) request(base + 2 * STEP, kA);
        reduce(base + STEP, kB);
    }
    if (g == a.G - 1 && tid < kWave) {                 // the new token
        const float d = group_sum<LPR>(qf.dot(load16(a.k_new + pair * ROWB + sub * 16), 0.f)) * a.scale;
        if (tid == 0) Zp[len] = d;
    }
}

// Launch 2.  Softmax over the stored logits, importance, budget and selection of one pair; append of the new token.
//
// Bound: the dependent chain of one workgroup (a few pairs on 256 CUs), so every load of the pair's logits and
// importance is requested at once, before the length is known, weights and keys stay in registers between the phases, and 1024
// threads share the work.  PER: slots per thread.  Weights are bit-identical to the one-workgroup kernel's: its 512 threads'
// sums are added up in its order.
// 32 pairs x 8192 rows, f16, d = 128: 14.6 us (17 with weights and keys in LDS, two rounds of histograms and runs of
// slots per thread, 33 with the one-workgroup kernel in this place); then 32 400 -> 28 100 clocks with the range of the keys from the old
// importance (no pass over the new keys and no barrier for it), ranks counted by all waves, and the kept slots placed from lane masks (whole
// step, with the narrower pieces of launch 3, 8 pairs x 12000 36.8 -> 33.7 us, 32 x 8192 35.2 -> 33.1, 64 x 8192 48.7 -> 46.7).
template <int PER>
__global__ void __launch_bounds__(kSelThreads) swa_split_select_kernel(SplitArgs a)
{
    constexpr int NT = kSelThreads;
    constexpr int NW = NT / kWave;
    constexpr int SUMT = 512;               // threads of the one-workgroup kernel on such caches
    constexpr int CHUNKS = kSelPer * NW;    // runs of 64 slots: chunk k NW + w is wave w's register k
    static_assert(NT == 2 * SUMT && CHUNKS == 4 * kWave, "how the sum is shared out and the chunks are scanned");
    __shared__ float s_x[PER][SUMT];                               // exponentials of the upper half of the threads
    __shared__ SelectScratch<NT> s_sel;
    __shared__ float s_red[NW];
    __shared__ float s_sum[SUMT / kWave];
    __shared__ __align__(16) uint32_t s_chunk[CHUNKS];                 // kept for sure | equal to the threshold << 16

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t pair = blockIdx.x;
    const int s = (int)(pair / a.h);
    const int cap = a.cap;
    const float* Zp = a.ws_z + pair * (int64_t)cap;
    float* Sp = a.score + pair * (int64_t)cap;
    float* Wp = a.ws_p + pair * (int64_t)cap;
    // requested before the length is known: what lies at or beyond it is not used
    float z[PER], sc[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (k * NT >= a.lds_slots) continue;
        const int i = tid + k * NT < cap ? tid + k * NT : cap - 1;
        z[k] = Zp[i];
        sc[k] = Sp[i];
    }
    s_sel.hist[2 * tid] = 0;
    s_sel.hist[2 * tid + 1] = 0;
    if (tid == 0) s_sel.listed = 0;
    if (tid < kWave) s_sel.rank[tid] = 0;
    const int len = a.cache_len[s];
    const int n = a.seq_len[s];
    const int m = len + 1;
    const bool overflow = (m > cap) || (m > a.lds_slots) || (len < 0);
    int keep = 0, n_local = 0, n_global = 0, w_eff = 0;
    // A length to compare slots with, anew in every phase: PER lane masks carried from phase to phase take more scalar registers than
    // there are (43 and 120 of them spilled at 9 and 16 slots a thread; four fifths evicted, f16, d = 128, whole step, 32 pairs x 8192
    // 35.3 -> 34.4 us, x 12000 50.1 -> 47.7; 4 pairs x 12000, bf16, d = 64 32.3 -> 30.2).
    auto anew = [](int v) {
        asm volatile("" : "+s"(v));
        return v;
    };

    if (!overflow) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = tid + k * NT;
            z[k] = i < m ? z[k] : -INFINITY;
            sc[k] = i < len ? sc[k] : 0.f;
        }
        // append: the new row's key, value and position
        const int lpr = a.row_bytes / 16;
        if (tid < 2 * lpr) {
            const int at = (tid < lpr ? tid : tid - lpr) * 16;
            const char* row = tid < lpr ? a.k_new : a.v_new;
            store16((tid < lpr ? a.k_cache : a.v_cache) + (pair * (int64_t)cap + len) * a.row_bytes + at,
                    load16(row + pair * a.row_bytes + at));
        }
        if (tid == 0) a.pos[pair * (int64_t)cap + len] = n - 1;

        budget(n, m, a.w, a.sparsity_bp, keep, n_local, n_global, w_eff);
        const int ncand = m - n_local;
        float mx = -INFINITY;
        // the old importance of the candidates, as keys: with the largest weight it bounds the new
        uint32_t kmin = 0xffffffffu, kmax = 0u;
        const int n0 = anew(keep < m ? ncand : 0);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            mx = fmaxf(mx, z[k]);
            if (k * NT >= n0) continue;
            const uint32_t old = order_key(sc[k]);
            const bool cand = tid + k * NT < n0;
            kmin = cand && old < kmin ? old : kmin;
            kmax = cand && old > kmax ? old : kmax;
        }
        mx = wave_max(mx);
        wave_min_max(kmin, kmax);
        if (lane == 0) {
            s_red[wave] = mx;
            s_sel.lo[wave] = kmin;
            s_sel.hi[wave] = kmax;
        }
        __syncthreads();
        mx = s_red[0];
#pragma unroll
        for (int v = 1; v < NW; ++v) mx = fmaxf(mx, s_red[v]);
        const int m1 = anew(m);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (k * NT >= m1) continue;
            z[k] = tid + k * NT < m1 ? expf(z[k] - mx) : 0.f;
            if (tid >= SUMT) s_x[k][tid - SUMT] = z[k];
        }
        __syncthreads();
        if (tid < SUMT) {
            // thread t of the one-workgroup kernel adds up slots t, t + 512, t + 1024, ...  (a zero past the end changes nothing)
            float sum = 0.f;
            const int m2 = anew(m);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (k * NT >= m2) continue;
                sum += z[k];
                sum += s_x[k][tid];
            }
            sum = wave_sum(sum);
            if (lane == 0) s_sum[wave] = sum;
        }
        __syncthreads();
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < SUMT / kWave; ++v) sum += s_sum[v];

        uint32_t key[PER];
        const int m3 = anew(m);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            key[k] = 0u;
            if (k * NT >= m3) continue;
            const int i = tid + k * NT;
            if (i < m3) {
                z[k] = z[k] / sum;                          // the weight
                const float v = sc[k] + z[k];
                Sp[i] = v;
                key[k] = order_key(v);
            }
        }
        if (a.probs_dbg) {
            float* dbg = a.probs_dbg + pair * (int64_t)cap;
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if (tid + k * NT < m) dbg[tid + k * NT] = z[k];
            for (int i = m + tid; i < cap; i += NT) dbg[i] = 0.f;
        }

        int32_t* kout = a.kept_idx + pair * (int64_t)cap;
        if (keep == m) {                                    // everything stays
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int i = tid + k * NT;
                if (i < m) {
                    kout[i] = i;
                    Wp[i] = z[k];
                }
            }
        } else {
            // Kept: slots from ncand on, the candidates before it with keys above thr, and of those equal to it the `rem` lowest slots.
            uint32_t thr = 0xffffffffu;
            int rem = 0, n_eq = 0;
            if (n_global > 0) {
                auto each = [&](auto f) {
                    const int n = anew(ncand);
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        if (k * NT >= n) continue;
                        if (tid + k * NT < n) f(key[k]);
                    }
                };
                // Range of the keys: adding a weight, which is at most 1 / sum, to the old importance rounds monotonically, so the range of
                // the old values and that weight (a little more of it) enclose the new ones; what is not finite is looked at itself.
#pragma unroll
                for (int v = 0; v < NW; ++v) {
                    kmin = s_sel.lo[v] < kmin ? s_sel.lo[v] : kmin;
                    kmax = s_sel.hi[v] > kmax ? s_sel.hi[v] : kmax;
                }
                const float most = key_value(kmax) + 1.0001f / sum;
                if (kmin > order_key(-INFINITY) && kmax < order_key(INFINITY) && most < INFINITY && sum < INFINITY) kmax = order_key(most);
                else key_range<NT>(s_sel, each, kmin, kmax);
                select_threshold<NT>(s_sel, n_global, kmin, kmax, each, thr, rem, n_eq);
            }
            // The kept list: a wave's 64 slots of a register are one run, so ballots place them within it and a scan of the runs' counts
            // (every wave for itself) places the runs.
            auto below = [](uint64_t mask) __attribute__((always_inline)) {       // lanes of it before this one
                return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            };
            // which lanes' slots of register k are kept for sure, and which tie with the threshold
            auto lanes = [&](int k, int m, int n, uint32_t thr, uint64_t& in, uint64_t& eq) __attribute__((always_inline)) {
                in = __ballot(key[k] > thr);
                eq = __ballot(key[k] == thr);
                if ((k + 1) * NT > n) {                         // (not all of them candidates)
                    const int i = tid + k * NT;
                    const uint64_t cand = __ballot(i < n);
                    in = (in & cand) | (__ballot(i < m) & ~cand);
                    eq &= cand;
                }
            };
            const uint32_t thr_u = (uint32_t)__builtin_amdgcn_readfirstlane((int)thr);
            int counts = 0;                                     // lane k: register k
            const int m4 = anew(m), n4 = anew(ncand);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (k * NT >= m4) continue;
                uint64_t in, eq;
                lanes(k, m4, n4, thr_u, in, eq);
                counts = lane == k ? (int)__popcll(in) | ((int)__popcll(eq) << 16) : counts;
            }
            if (lane < kSelPer) s_chunk[lane * NW + wave] = (uint32_t)counts;
            __syncthreads();
            const uint4 c4 = *reinterpret_cast<const uint4*>(&s_chunk[4 * lane]);
            const uint32_t own = c4.x + c4.y + c4.z + c4.w;
            const uint32_t inc = (uint32_t)wave_scan((int)own);
            const int part = wave & 3;                          // chunk k NW + wave: lane (k NW + wave) / 4, its entry `part`
            const uint32_t first = inc - own + (part > 0 ? c4.x : 0u) + (part > 1 ? c4.y : 0u) + (part > 2 ? c4.z : 0u);
            const int m5 = anew(m), n5 = anew(ncand), thr5 = anew((int)thr_u);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                if (k * NT >= m5) continue;
                uint64_t mask, ties;
                lanes(k, m5, n5, (uint32_t)thr5, mask, ties);
                const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)first, k * (NW / 4) + wave / 4);
                const int eq = (int)(before >> 16);
                if (ties) {                                     // the lowest slots of what ties
                    const bool t = __builtin_amdgcn_inverse_ballot_w64(ties) && eq + below(ties) < rem;
                    mask |= __ballot(t);
                }
                if (__builtin_amdgcn_inverse_ballot_w64(mask)) {
                    const uint32_t at = (before & 0xffffu) + (uint32_t)(eq < rem ? eq : rem) + (uint32_t)below(mask);
                    kout[at] = tid + k * NT;
                    Wp[at] = z[k];
                }
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

// Launch 3.  Output of one pair from its kept list, PIECE bytes of the row per workgroup.
//
// Bound: what a CU can load (about 100 GB/s with random rows) and the launch's own latency.  Whole rows in slices of the list, or inside
// launch 2, would need either a fourth launch that adds the slices up or a choice by the number of kept rows, which
// the host does not know: a compacted cache or a wide window keeps many times the share that the sparsity
// names.  Channels need no sum across workgroups, whatever is kept.  Pieces of 64 bytes double the workgroups and halve the rounds that each
// makes over the list, which pays up to 64 pairs, where that leaves a CU to every workgroup; beyond, the halves of a line cost more.
// Whole step, f16, d = 128, pieces of 128 / 64 bytes, us: 8 pairs x 8192 rows, a fifth kept 28.9 / 27.3, all 43.2 / 37.0; 32 pairs 35.3 /
// 33.6, 52.6 / 49.0; 64 pairs 48.3 / 47.4, 70.3 / 66.3; 96 pairs 62.7 / 65.1, 85.8 / 107; 128 pairs 72.7 / 75.3, 104 / 123; 32 pairs, bf16, d =
// 64 31.3 / 28.8, fp32, d = 128 47.7 / 46.7.
// This form / partial sums and a fourth launch / output in launch 2, when it was chosen (launches 1 and 2 took 3 to 6 us more): 32 pairs, 20 of 2048
// rows kept 20.6 / 26.3 / 19.4; all of 2048 21.4 / 28.2 / 33.3; 1638 of 8192 40.1 / 45.3 / 46.5; all of 8192 52.8 / 59.2 / 98; 128
// pairs, all of 8192 102 / 130 / 136.  Reading the list a round ahead changed nothing, or cost 2 %.
template <typename T, int D, int PIECE>
__global__ void __launch_bounds__(kGatherThreads) swa_split_gather_kernel(SplitArgs a)
{
    constexpr int NT = kGatherThreads;
    constexpr int NW = NT / kWave;
    constexpr int EPV = Elem<T>::kPerVec;
    constexpr int ROWB = D * Elem<T>::kBytes;
    constexpr int LPR = PIECE / 16;         // lanes per piece of a row
    constexpr int PIECES = ROWB / PIECE;
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
    const char* Vp = a.v_cache + pair * (int64_t)a.cap * ROWB + piece * PIECE + sub * 16;
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
    // over the wave's row groups
    auto over_groups = [](float x) __attribute__((always_inline)) {
        x += dpp_move<0x128>(x);                  // row_ror 8
        if constexpr (LPR == 4) x += dpp_move<0x124>(x);
        const uint32_t u = f2u(x);
        const auto r16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        const uint32_t v = f2u(u2f(r16[0]) + u2f(r16[1]));
        const auto r32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return u2f(r32[0]) + u2f(r32[1]);
    };
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = over_groups(acc[e]);
    ps = over_groups(ps);
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

// Slots per thread: as many as the bound on the lengths asks for (the loops over them are unrolled, and code that no slot needs is
// still fetched), a little more than the powers of two for the answer behind a prompt.
static int launch_select(const SplitArgs& a, int64_t pairs, hipStream_t stream)
{
    const dim3 grid((unsigned)pairs), block(kSelThreads);
    const int per = (a.lds_slots + kSelThreads - 1) / kSelThreads;
    if (per <= 3) launch_kernel((swa_split_select_kernel<3>), grid, block, 0, stream, a);
    else if (per <= 5) launch_kernel((swa_split_select_kernel<5>), grid, block, 0, stream, a);
    else if (per <= 9) launch_kernel((swa_split_select_kernel<9>), grid, block, 0, stream, a);
    else launch_kernel((swa_split_select_kernel<kSelPer>), grid, block, 0, stream, a);
    return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
}

// Bytes of a row per workgroup of launch 3 (both sides of the line measured above).
int split_piece_bytes(int64_t pairs) { return pairs <= 64 ? 64 : 128; }

template <typename T, int D>
static int launch_split_t(const SplitArgs& a, int64_t pairs, hipStream_t stream)
{
    constexpr int NT = 256;
    const dim3 grid((unsigned)(pairs * a.G));
    launch_kernel((swa_split_logits_kernel<T, D, NT>), grid, dim3(NT), 0, stream, a);
    if (hipGetLastError() != hipSuccess) return SWA_ERR_HIP;
    if (launch_select(a, pairs, stream) != SWA_OK) return SWA_ERR_HIP;
    const int64_t at_most = (pairs + kXcds - 1) / kXcds * kXcds * D * Elem<T>::kBytes;      // bytes of all rows
    if (split_piece_bytes(pairs) == 64)
        launch_kernel((swa_split_gather_kernel<T, D, 64>), dim3((unsigned)(at_most / 64)), dim3(kGatherThreads), 0, stream, a);
    else
        launch_kernel((swa_split_gather_kernel<T, D, 128>), dim3((unsigned)(at_most / 128)), dim3(kGatherThreads), 0, stream, a);
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
    a.row_bytes = cache_row_bytes(p);
    a.scale = scale;
    if (p.dtype == SWA_F32) {
        return p.d == 64 ? launch_split_t<F32, 64>(a, pairs, stream) : launch_split_t<F32, 128>(a, pairs, stream);
    } else if (p.dtype == SWA_F16) {
        return p.d == 64 ? launch_split_t<F16, 64>(a, pairs, stream) : launch_split_t<F16, 128>(a, pairs, stream);
    }
    return p.d == 64 ? launch_split_t<BF16, 64>(a, pairs, stream) : launch_split_t<BF16, 128>(a, pairs, stream);
}

}  // namespace swa
