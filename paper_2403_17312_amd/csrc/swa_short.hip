// Decode step for caches of few slots: one workgroup per (sequence, head) pair, the pair's whole state in registers.
//
// What bounds the step there is latency, not bytes: 512 pairs of 106 rows are 28 MB, 4 us of reading, and the streaming
// kernel (swa_decode.hip) takes 6.8 us a workgroup, 4.0 for rows that arrive in four stages and 2.7 for the phases
// behind them (softmax, selection, the evicted row's second read, output, importance), with a barrier between each two.  Here
//   - every key and value row of the pair is requested at once, the first half before the length is known;
//   - the value rows stay in registers until the selection is known, so the output is the sum over the kept rows
//     alone and nothing is read twice;
//   - every wave holds all logits, importance values and positions (one to four slots per lane) and forms softmax,
//     importance and selection for itself: one barrier behind the logits, one before the output.
// Weights, importance and kept set are bit-identical to the streaming kernel's (same products, same order of additions).
#include <type_traits>

#include "swa_decode.hpp"
#include "swa_select.hpp"

namespace swa {

template <typename T, int D, int NT, int U>
struct ShortShape {
    static constexpr int LPR = D / Elem<T>::kPerVec;     // lanes per row
    static constexpr int NG = NT / LPR;                  // rows per workgroup and load
    static constexpr int ROWS = NG * U;                  // slots at most
};

// Waves per SIMD: what the registers of a lane's rows leave room for (none of the kernels in use spills).
template <typename T, int D, int NT, int U, bool RING>
constexpr int short_waves()
{
    return U > 8 || (RING && (Elem<T>::kBytes == 1 || ShortShape<T, D, NT, U>::ROWS == NT)) ? 3 : 4;
}

template <typename T, int D, int NT, int U, bool RING>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(short_waves<T, D, NT, U, RING>())))
swa_short_kernel(DecodeArgs a)
{
    constexpr int EPV = Elem<T>::kPerVec;
    constexpr int LPR = ShortShape<T, D, NT, U>::LPR;
    constexpr int NG = ShortShape<T, D, NT, U>::NG;
    constexpr int ROWS = ShortShape<T, D, NT, U>::ROWS;
    constexpr int NW = NT / kWave;
    constexpr int SL = ROWS / kWave;                     // slots per lane
    constexpr int UE = U / 4;                            // rows requested before the length is known
    constexpr int ROWB = D * Elem<T>::kBytes;
    typedef typename Act<T>::type AT;
    constexpr int XROWB = D * Elem<AT>::kBytes;
    constexpr bool kQ8 = Elem<T>::kBytes == 1;
    constexpr int PARTS = NW / SL;                       // strict window: waves that share the rows of a chunk's ring
    constexpr int kRingAhead = PARTS > 1 ? 16 : 32;      // ring entries per lane requested ahead
    static_assert(ROWS % kWave == 0 && kWave % NG == 0 && SL <= NW, "every wave has a chunk of 64 slots at most");

    __shared__ float s_z[ROWS];                          // logits
    __shared__ float s_sc[RING ? ROWS : 1];              // new importance
    __shared__ unsigned long long s_cand[ROWS];          // several evictions: (key, ~token) of the candidates
    __shared__ uint64_t s_mask[SL];                      // several evictions: kept slots
    __shared__ uint16_t s_hole[ROWS], s_dst[ROWS];       // several evictions, unordered: holes, and every slot's final slot
    __shared__ float s_acc[NW * D];
    __shared__ __align__(16) unsigned char s_newc[kQ8 ? 2 * D : 16];   // codes of the new K and V rows
    __shared__ __align__(16) float s_qs[kQ8 ? D : 4];
    __shared__ __align__(16) float s_qz[kQ8 ? D : 4];
    constexpr int kNowhere = 0xffff;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = lane % LPR;
    const int grp = tid / LPR;
    const int64_t pair = blockIdx.x;
    const int s = (int)(blockIdx.x / (uint32_t)a.h);
    const int head = (int)(blockIdx.x - (uint32_t)s * (uint32_t)a.h);
    const int cap = a.cap;
    const bool bag = a.unordered != 0;                   // else: the two-call form, nothing is compacted
    char* Kp = a.k_cache + pair * (int64_t)cap * ROWB;
    char* Vp = a.v_cache + pair * (int64_t)cap * ROWB;
    float* Sp = a.score + pair * (int64_t)cap;
    int32_t* Pp = a.pos + pair * (int64_t)cap;

    const int len = a.cache_len[s];
    const int n = a.seq_len[s];
    // rows, importance and positions whose place does not depend on the length (whatever lies at or beyond it is not used)
    // byte offset of this lane's piece of its row u, no further than row `last` (uniform base + 32-bit offset)
    auto at = [&](int u, int last) -> uint32_t {
        const int row = u * NG + grp;
        return (uint32_t)(row < last ? row : last) * ROWB + (uint32_t)sub * 16;
    };
    Vec16 kv[U], vv[U];
#pragma unroll
    for (int u = 0; u < UE; ++u) {
        kv[u] = load16_stream(Kp + at(u, cap - 1));
    }
    float sold[SL];
    int pold[SL];
#pragma unroll
    for (int k = 0; k < SL; ++k) {
        int i = lane + k * kWave;
        i = i < cap ? i : cap - 1;
        sold[k] = RING ? 0.f : Sp[i];
        pold[k] = bag ? Pp[i] : 0;
    }
    Vec16 nk, nv;
    QFrag<T> qf;
    float pq = 0.f, pl = 0.f, pz = 0.f, pkn = 0.f, pvn = 0.f, plv = 0.f, pzv = 0.f;
    const float* lamK = kQ8 ? a.qparams + pair * D : nullptr;
    if constexpr (kQ8) {
        if (tid < D) {
            pl = lamK[tid];
            pz = lamK[a.qstride + tid];
            plv = lamK[2 * a.qstride + tid];
            pzv = lamK[3 * a.qstride + tid];
            pq = (float)reinterpret_cast<const _Float16*>(a.q + pair * XROWB)[tid];
            pkn = (float)reinterpret_cast<const _Float16*>(a.k_new + pair * XROWB)[tid];
            pvn = (float)reinterpret_cast<const _Float16*>(a.v_new + pair * XROWB)[tid];
        }
    } else {
        qf.load(load16(a.q + pair * XROWB + sub * 16));
        nk = load16(a.k_new + pair * XROWB + sub * 16);
        nv = load16(a.v_new + pair * XROWB + sub * 16);
    }
#pragma unroll
    for (int u = 0; u < UE; ++u) {
        vv[u] = load16_stream(Vp + at(u, cap - 1));
    }

    const int m = len + 1;
    const bool overflow = (m > cap) || (m > a.lds_slots) || (len < 0);
    int keep = 0;
    if (!overflow) {
        // strict window: the ring entries of a chunk of 64 slots, in order shared out between PARTS waves
        const int chunk = wave % SL;
        const int mine = chunk * kWave + lane;           // this lane's slot in what is shared out between the waves
        const bool owner = wave < SL;
        float* Rg = RING ? a.ring + pair * (int64_t)a.ring_rows * cap : nullptr;
        const int rper = RING ? (a.ring_rows + PARTS - 1) / PARTS : 0;
        const int rlo = wave / SL * rper;
        const int rhi = rlo + rper < a.ring_rows ? rlo + rper : a.ring_rows;
        const bool ring_ahead = RING && rper <= kRingAhead;
        float rpre[RING ? kRingAhead : 1];
        if constexpr (RING) {
            if (ring_ahead) {
                const bool old = mine < len;
#pragma unroll
                for (int j = 0; j < kRingAhead; ++j)
                    rpre[j] = (old && rlo + j < rhi && rlo + j != a.ring_row) ? Rg[(int64_t)(rlo + j) * cap + mine] : 0.f;
            }
        }
        // the new token's rows and the query in the cache's format, once the first loads are in flight
        auto new_rows = [&]() __attribute__((always_inline)) {
            if constexpr (kQ8) {
                if (tid < D) {
                    s_newc[tid] = (unsigned char)quantise_one(pkn, pl, pz);
                    s_newc[D + tid] = (unsigned char)quantise_one(pvn, plv, pzv);
                    const float qs = pq * pl;
                    s_qs[tid] = qs;
                    s_qz[tid] = qs * pz;
                }
                __syncthreads();
                nk = *reinterpret_cast<const Vec16*>(s_newc + sub * 16);
                nv = *reinterpret_cast<const Vec16*>(s_newc + D + sub * 16);
                qf.load(s_qs + sub * 16, s_qz + sub * 16);
            }
        };
        int n_local = 0, n_global = 0, w_eff = 0;
        budget(n, m, a.w, a.sparsity_bp, keep, n_local, n_global, w_eff);
        const int ncand = m - n_local;
        const int wlo = n - w_eff;                       // unordered layout: the window is pos >= wlo
        const int E = m - keep;

        // ---- the other rows, logits -------------------------------------------------------------
        // As many rows per lane as the length needs, in steps of UE (the counts are written out so that the compiler knows
        // what is in flight when a key row is used).  Lanes past the end read slot `len`; what they find has no weight.
        float z[U];
        auto rows = [&](auto count) __attribute__((always_inline)) {
            constexpr int C = count.value;
#pragma unroll
            for (int u = UE; u < C; ++u) {
                kv[u] = load16_stream(Kp + at(u, len));
            }
#pragma unroll
            for (int u = UE; u < C; ++u) {
                vv[u] = load16_stream(Vp + at(u, len));
            }
#pragma unroll
            for (int u = C; u < U; ++u) vv[u] = Vec16{0u, 0u, 0u, 0u};
            new_rows();
#pragma unroll
            for (int u = 0; u < C; ++u) z[u] = group_sum<LPR>(qf.dot(kv[u], 0.f)) * a.scale;
#pragma unroll
            for (int u = C; u < U; ++u) z[u] = 0.f;
        };
        const int stages = (m + NG * UE - 1) / (NG * UE);
        if (stages <= 1) rows(std::integral_constant<int, UE>());
        else if (stages == 2) rows(std::integral_constant<int, 2 * UE>());
        else if (stages == 3) rows(std::integral_constant<int, 3 * UE>());
        else rows(std::integral_constant<int, U>());
        // every lane of a group has the group's logits: lane u of it stores row u's
        {
            float zs = z[0];
#pragma unroll
            for (int u = 1; u < U; ++u) zs = sub == u ? z[u] : zs;
            const float znew = group_sum<LPR>(qf.dot(nk, 0.f)) * a.scale;
            const int row = sub * NG + grp;
            if (sub < U && row < m) s_z[row] = row == len ? znew : zs;
        }
        // the old importance and positions have arrived before any wave may overwrite them
#pragma unroll
        for (int k = 0; k < SL; ++k) asm volatile("" ::"v"(sold[k]), "v"(pold[k]));
        __syncthreads();

        // ---- softmax, importance: every wave for all slots ------------------------------------
        float p[SL], sc[SL];
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            const int i = lane + k * kWave;
            p[k] = i < m ? s_z[i] : -INFINITY;
            mx = fmaxf(mx, p[k]);
        }
        mx = wave_max(mx);
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            p[k] = lane + k * kWave < m ? expf(p[k] - mx) : 0.f;
            sum += wave_sum(p[k]);
        }
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            p[k] = p[k] / sum;
            const int i = lane + k * kWave;
            if (i >= len) {
                sold[k] = 0.f;
                pold[k] = n - 1;
            }
            sc[k] = sold[k] + p[k];
        }
        if constexpr (RING) {
            // the rows of the ring in index order, the current weight standing in for the row this step replaces
            float pm = p[0];
#pragma unroll
            for (int k = 1; k < SL; ++k) pm = k == chunk ? p[k] : pm;
#pragma unroll
            for (int part = 0; part < PARTS; ++part) {
                if (wave / SL == part) {
                    float t = part ? s_sc[mine] : 0.f;
                    if (ring_ahead) {
#pragma unroll
                        for (int j = 0; j < kRingAhead; ++j)
                            if (rlo + j < rhi) t += (rlo + j == a.ring_row) ? pm : rpre[j];
                    } else {
                        const bool old = mine < len;
                        for (int j0 = rlo; j0 < rhi; j0 += 8) {
                            float v[8];
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                v[j] = (old && j0 + j < rhi && j0 + j != a.ring_row) ? Rg[(int64_t)(j0 + j) * cap + mine] : 0.f;
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                if (j0 + j < rhi) t += (j0 + j == a.ring_row) ? pm : v[j];
                        }
                    }
                    s_sc[mine] = t;
                }
                __syncthreads();
            }
#pragma unroll
            for (int k = 0; k < SL; ++k) sc[k] = s_sc[lane + k * kWave];
        }

        // ---- selection ------------------------------------------------------------------------
        // (key << 32 | ~t): min = lowest score, then the latest token; t is the slot, or the token position when slots
        // are unordered
        auto rank_key = [&](int k) -> unsigned long long {
            const uint32_t t = bag ? (uint32_t)pold[k] : (uint32_t)(lane + k * kWave);
            return ((unsigned long long)order_key(sc[k]) << 32) | (uint32_t)(~t);
        };
        auto candidate = [&](int k) -> bool {
            const int i = lane + k * kWave;
            return i < m && (bag ? pold[k] < wlo : i < ncand);
        };
        uint64_t kept[SL];                               // kept slots, the same in every lane
        int jstar = m;                                   // one eviction: the evicted slot (m = none)
        const bool listed = E > 1 || (E == 1 && n_global <= 0);
        if (!listed) {
            if (E == 1) {
                unsigned long long best = ~0ull;
                int bslot = m;
#pragma unroll
                for (int k = 0; k < SL; ++k) {
                    const unsigned long long c = rank_key(k);
                    if (candidate(k) && c < best) {
                        best = c;
                        bslot = lane + k * kWave;
                    }
                }
                wave_min64p(best, bslot);
                jstar = __builtin_amdgcn_readfirstlane(bslot);
                jstar = jstar < 0 ? 0 : (jstar > len ? len : jstar);
            }
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const int i = lane + k * kWave;
                kept[k] = __ballot(i < m && i != jstar);
            }
        } else {
            // A candidate is kept if fewer than n_global candidates go before it: larger importance, or the same and an
            // earlier token.  Rare (the step after a short prompt, a budget that was cut), so it is simply counted.
            if (bag) {
                int present = 0;
#pragma unroll
                for (int k = 0; k < SL; ++k) present += (int)__popcll(__ballot(lane + k * kWave < m && pold[k] >= wlo));
                n_global = keep - present;
            }
#pragma unroll
            for (int k = 0; k < SL; ++k)
                if (k == wave) s_cand[mine] = candidate(k) ? rank_key(k) : 0ull;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                if (k != wave) continue;
                const bool cand = candidate(k);
                const unsigned long long c = rank_key(k);
                int before = 0;
                for (int j = 0; j < m; ++j) before += s_cand[j] > c ? 1 : 0;
                const uint64_t b = __ballot(mine < m && (!cand || before < n_global));
                if (lane == 0) s_mask[k] = b;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < SL; ++k) kept[k] = s_mask[k];
            if (bag) {
                // holes below `keep` are filled by kept rows above it, in ascending order both
                auto below = [&](int limit, int k) -> uint64_t {           // slots of chunk k below limit
                    const int c = limit - k * kWave;
                    return c <= 0 ? 0ull : (c >= kWave ? ~0ull : ((1ull << c) - 1ull));
                };
                const uint64_t lower = (1ull << lane) - 1ull;
                int holes = 0, movers = 0, mr = 0;
                bool is_kept = false;
#pragma unroll
                for (int k = 0; k < SL; ++k) {
                    const uint64_t hm = ~kept[k] & below(keep, k), mm = kept[k] & ~below(keep, k);
                    if (k == wave) {
                        if ((hm >> lane) & 1ull) s_hole[holes + (int)__popcll(hm & lower)] = (uint16_t)mine;
                        mr = movers + (int)__popcll(mm & lower);
                        is_kept = (kept[k] >> lane) & 1ull;
                    }
                    holes += (int)__popcll(hm);
                    movers += (int)__popcll(mm);
                }
                __syncthreads();
                if (owner) s_dst[mine] = !is_kept ? kNowhere : (mine < keep ? mine : (mr < holes ? s_hole[mr] : kNowhere));
                __syncthreads();
            }
        }

        // ---- output: sum over the kept rows, in registers -------------------------------------
        float pk[SL];
        float ps = 0.f;
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            pk[k] = ((kept[k] >> lane) & 1ull) ? p[k] : 0.f;
            ps += pk[k];
        }
        ps = wave_sum(ps);
        // the new token's share, in one group of rows
        float wn = pk[0];
#pragma unroll
        for (int k = 1; k < SL; ++k) wn = k == len / kWave ? pk[k] : wn;
        wn = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wn), len & (kWave - 1)));
        float acc[EPV];
        {
            float f[EPV];
            unpack<T>(nv, f);
#pragma unroll
            for (int e = 0; e < EPV; ++e) acc[e] = (grp == 0 && wn != 0.f) ? wn * f[e] : 0.f;
        }
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = __shfl(pk[u * NG / kWave], u * NG % kWave + grp, kWave);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = u * NG + grp;
            float wr = w[u];
            Vec16 x = vv[u];
            if (row >= len || wr == 0.f) {                 // evicted, new or past the end: whatever the slot holds
                wr = 0.f;
                x = Vec16{0u, 0u, 0u, 0u};
            }
            // (widened here and not as soon as the row arrives, which would take twice the registers)
            asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
            float f[EPV];
            unpack<T>(x, f);
#pragma unroll
            for (int e = 0; e < EPV; ++e) acc[e] = __builtin_fmaf(wr, f[e], acc[e]);
        }
#pragma unroll
        for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
            for (int e = 0; e < EPV; ++e) acc[e] += __shfl_xor(acc[e], o, kWave);
        if (lane < LPR) {
#pragma unroll
            for (int e = 0; e < EPV; ++e) s_acc[wave * D + sub * EPV + e] = acc[e];
        }

        // ---- state ----------------------------------------------------------------------------
        int32_t* kout = a.kept_idx ? a.kept_idx + pair * (int64_t)cap : nullptr;
        const int hole = (E == 1 && jstar < keep) ? jstar : m;      // one eviction: where the new token goes
        int first = 0;                                              // kept slots in the chunks before
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            if (k == wave) {
                const bool in = (kept[k] >> lane) & 1ull;
                if (a.probs_dbg && mine < m) a.probs_dbg[pair * (int64_t)cap + mine] = p[k];
                if (!bag) {
                    if (mine < m) Sp[mine] = sc[k];
                    if (in) kout[first + (int)__popcll(kept[k] & ((1ull << lane) - 1ull))] = mine;
                } else {
                    int dst = kNowhere;
                    if (in) dst = listed ? (int)s_dst[mine] : (mine == len && hole < m ? hole : mine);
                    if (dst < keep) {
                        Sp[dst] = sc[k];
                        if (dst != mine || mine == len) Pp[dst] = pold[k];
                        if (kout) kout[dst] = mine;
                        if constexpr (RING) {
                            Rg[(int64_t)a.ring_row * cap + dst] = p[k];
                            // the other rows of the ring follow a token that moved; the new token has none
                            if (listed && (dst != mine || mine == len))
                                for (int j = 0; j < a.ring_rows; ++j)
                                    if (j != a.ring_row) Rg[(int64_t)j * cap + dst] = mine == len ? 0.f : Rg[(int64_t)j * cap + mine];
                        }
                    }
                }
            }
            first += (int)__popcll(kept[k]);
        }
        if (a.probs_dbg)
            for (int i = m + tid; i < cap; i += NT) a.probs_dbg[pair * (int64_t)cap + i] = 0.f;
        if (!listed || !bag) {
            // the new token's rows: into the hole or behind the others
            const int dst = !bag ? len : (hole < m ? hole : len);
            if (!bag || dst < keep) {
                if (tid < LPR) store16(Kp + dst * ROWB + sub * 16, nk);
                else if (tid < 2 * LPR) store16(Vp + dst * ROWB + sub * 16, nv);
                if (!bag && tid == 0) Pp[len] = n - 1;
                if constexpr (RING) {
                    for (int j = tid; j < a.ring_rows; j += NT)
                        if (j != a.ring_row) Rg[(int64_t)j * cap + dst] = 0.f;
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int row = u * NG + grp;
                const int dst = row < m ? (int)s_dst[row] : kNowhere;
                if (dst < keep && (dst != row || row == len)) {
                    Vec16 x = nk, y = nv;
                    if (row < len) {
                        x = load16(Kp + row * ROWB + sub * 16);
                        y = load16(Vp + row * ROWB + sub * 16);
                    }
                    store16(Kp + dst * ROWB + sub * 16, x);
                    store16(Vp + dst * ROWB + sub * 16, y);
                }
            }
        }

        __syncthreads();
        for (int e = tid; e < D; e += NT) {
            float t = 0.f;
#pragma unroll
            for (int v = 0; v < NW; ++v) t += s_acc[v * D + e];
            t /= ps;
            if constexpr (kQ8) t = lamK[2 * a.qstride + e] * (t - lamK[3 * a.qstride + e]);      // accumulated in code space
            store_elem<AT>(a.out + pair * XROWB, e, keep > 0 ? t : 0.f);      // an empty budget: an empty sum
        }
    }

    if (tid == 0) {
        if (overflow) atomicOr(a.status, kStatusCapacityBit);
        if (bag) {
            // every head of a sequence computes the same value: head 0 writes it; cache_len is only read
            if (head == 0) a.kept_cnt[s] = overflow ? len : keep;
        } else {
            // the last head to finish publishes the new length: every workgroup has read the old one by then
            if (!overflow) a.kept_cnt[s] = keep;
            const int old = atomicAdd(&a.arrive[s], 1);
            if (old == a.h - 1) {
                atomicExch(&a.arrive[s], 0);
                if (!overflow) a.cache_len[s] = m;
            }
        }
    }
}

// The forms: threads per workgroup and rows per lane.
constexpr ShortForm kForms[] = {{128, 8}, {256, 8}, {256, 12}, {512, 8}};

// Slots that a form serves, 0 where there is no such kernel (beyond 256 slots it gained little).  (64 channels of 8 bits are 4 lanes of a row: half the rows per
// lane give as many.)
template <typename T, int D, int NT, int U>
constexpr int short_rows()
{
    typedef ShortShape<T, D, NT, U> S;
    if (U == 12 && S::LPR != 16) return 0;
    return S::NG <= kWave && S::ROWS % kWave == 0 && S::ROWS <= NT && S::ROWS <= 256 ? S::ROWS : 0;
}
template <typename T, int D>
constexpr int short_unroll(int u) { return Elem<T>::kBytes == 1 && D == 64 ? u / 2 : u; }

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

// Which calls: the two-call form and unordered compaction (in token order rows shift by way of LDS, and the head-shared step
// has more than one launch), with a bound on the lengths that a form covers; the smallest form that does.
// Streaming kernel / this one, us a step, f16 unless stated, d = 128, one token evicted:
//      32 pairs   106 slots 7.0 / 5.0,  140  7.6 / 5.4,  206  8.4 / 6.2;  8-bit 206  8.6 / 7.2
//     512 pairs    64 slots 7.2 / 5.3,  106  7.9 / 6.5,  140  9.4 / 8.5,  206 12.3 / 12.0;  8-bit 106  8.5 / 7.3,  206 10.1 / 9.3
//    1024 pairs   106 slots 12.9 / 11.3,  140 16.0 / 15.1,  206 21.3 / 21.2;  8-bit 206 14.5 / 15.9
//    2560 pairs    32 slots 16.2 / 9.8,  106 26.6 / 23.9,  140 32.9 / 32.1,  206 46.6 / 47.1;  8-bit 106 20.2 / 17.9,  206 30.4 / 30.7
//    8192 pairs   106 slots 77 / 75,  160 112 / 110
// The forms that fill half a CU with one workgroup (512 threads, and 256 on the 8-bit cache, whose lanes hold
// 16 channels) pay while the chip is not full of workgroups; the strict window, rings of 16 rows: 512 pairs x 106 slots 10.5 / 7.9, 206
// 15.2 / 13.7, 2560 pairs x 106 35.4 / 30.1.
ShortForm short_form(const swa_params& p, int64_t pairs, int len_bound)
{
    const bool fuse = (p.flags & SWA_FUSE_COMPACTION) != 0;
    if ((p.flags & SWA_HEAD_SHARED) || (fuse && !(p.flags & SWA_UNORDERED))) return {0, 0};
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
        if (a.ring) hipLaunchKernelGGL((swa_short_kernel<T, D, NT, U, true>), dim3((unsigned)pairs), dim3(NT), 0, stream, a);
        else hipLaunchKernelGGL((swa_short_kernel<T, D, NT, U, false>), dim3((unsigned)pairs), dim3(NT), 0, stream, a);
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
