// Decode step for caches of few slots: one workgroup per (sequence, head) pair, the pair's whole state in registers.
//
// What bounds the step there is latency, not bytes: 512 pairs of 106 rows are 28 MB, 4 us of reading, and the streaming
// kernel (swa_decode.hip) takes 6.8 us a workgroup, 4.0 for rows that arrive in four stages and 2.7 for the phases
// behind them (softmax, selection, the evicted row's second read, output, importance), with a barrier between each two.  Here
//   - every key and value row of the pair is requested at once, the first quarter before the length is known;
//   - the value rows stay in registers until the selection is known, so the output is the sum over the kept rows
//     alone and nothing is read twice;
//   - where most rows go (the step after a short prompt) the values wait for the selection instead and only kept rows' are read,
//     candidates are ranked by 32-bit counts that all waves share, and rows and ring columns that change slot are moved many at
//     a time.  Streaming kernel / this one with all values read, 64-bit counts and moves one by one / as it is, us a step with four
//     fifths of the rows evicted: 512 pairs x 206, f16, d = 128 20.5 / 23.8 / 18.7; 4096 x 256, f16, d = 64 66.8 / 78.8 / 58.2, strict
//     window of 16 rows 86 / 126 / 74;
//   - every wave holds all logits, importance values and positions (one to four slots per lane) and forms softmax,
//     importance and selection for itself: one barrier behind the logits, one before the output.
// Weights, importance and kept set are bit-identical to the streaming kernel's (same products, same order of additions).
//
// The head-shared step takes two launches of it (PHASE 1 and 2): the first leaves every pair's weights, new importance and dense
// output in the workspace, the second sums the importance over the heads, selects, takes the evicted row out of
// the dense output and finishes the state.
#pragma once

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

template <typename T, int D, int NT, int U, bool RING, int PHASE>
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
    constexpr int PARTS = NW / SL;                       // waves that share what a chunk has to do
    constexpr int kRingAhead = PARTS > 1 ? 16 : 32;      // ring entries per lane requested ahead
    static_assert(ROWS % kWave == 0 && kWave % NG == 0 && SL <= NW, "every wave has a chunk of 64 slots at most");

    __shared__ float s_z[ROWS];                          // logits
    __shared__ float s_sc[RING ? ROWS : 1];              // new importance
    __shared__ __align__(16) uint32_t s_key[ROWS];       // several evictions: what the candidates are ranked by
    __shared__ uint16_t s_above[PARTS > 1 ? PARTS * ROWS : 1];         // ... their ranks, by parts of the keys
    __shared__ uint64_t s_mask[SL];                      // ... and which slots are kept
    __shared__ int32_t s_in[SL], s_top;
    __shared__ uint16_t s_hole[ROWS], s_mov[ROWS];       // several evictions, unordered: holes, and the slots that fill them
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
    if constexpr (PHASE != 2) {
#pragma unroll
        for (int u = 0; u < UE; ++u) kv[u] = load16_stream(Kp + at(u, cap - 1));
    }
    float sold[SL];          // (PHASE 2: the new importance)
    int pold[SL];
    float pw[SL];            // PHASE 2: weights
#pragma unroll
    for (int k = 0; k < SL; ++k) {
        int i = lane + k * kWave;
        i = i < cap ? i : cap - 1;
        if constexpr (PHASE == 2) {
            pw[k] = a.ws_p[pair * (int64_t)cap + i];
            sold[k] = a.ws_snew[pair * (int64_t)cap + i];
        } else {
            sold[k] = RING ? 0.f : Sp[i];
        }
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
    if constexpr (PHASE != 2) {
#pragma unroll
        for (int u = 0; u < UE; ++u) vv[u] = load16_stream(Vp + at(u, cap - 1));
    }
    float dense[EPV];        // PHASE 2: this lane's piece of the dense output
    if constexpr (PHASE == 2) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) dense[e] = a.ws_abar[pair * D + sub * EPV + e];
        // the selection key of slot tid: the new importance summed over the heads, fp32, head 0 first
        if (tid < ROWS) {
            const int i = tid < cap ? tid : cap - 1;
            float t = 0.f;
            if (a.ws_tot) {
                t = a.ws_tot[(int64_t)s * cap + i];
            } else {
                const float* Sh = a.ws_snew + (int64_t)s * a.h * cap + i;
                int hh = 0;
                for (; hh + 16 <= a.h; hh += 16) {
                    float v[16];
#pragma unroll
                    for (int k = 0; k < 16; ++k) v[k] = Sh[(int64_t)(hh + k) * cap];
#pragma unroll
                    for (int k = 0; k < 16; ++k) t += v[k];
                }
                if (hh < a.h) {
                    float v[16];
#pragma unroll
                    for (int k = 0; k < 16; ++k) v[k] = Sh[(int64_t)(hh + k < a.h ? hh + k : a.h - 1) * cap];
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        if (hh + k < a.h) t += v[k];
                }
            }
            s_z[tid] = t;
        }
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
            if (ring_ahead && PHASE != 2) {
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

        const bool listed = E > 1 || (E == 1 && n_global <= 0);
        // Where most rows go (the step after a prompt), the values wait until the selection is known, and only those of kept rows are
        // read.  The first launch of the head-shared step reads them all, though the second has no use for its output where several rows
        // go: without them 4096 pairs x 250 slots, f16, d = 64, four fifths evicted take 64 instead of 81 us, but the loads' second form made
        // every other step 0.1 us slower (84 pairs x 200, bf16, d = 64, one evicted 9.3 / 9.4).
        const bool late = PHASE == 0 && 2 * E > m;

        // ---- the other rows, logits -------------------------------------------------------------
        // As many rows per lane as the length needs, in steps of UE (the counts are written out so that the compiler knows
        // what is in flight when a key row is used).  Lanes past the end read slot `len`; what they find has no weight.
        float z[U];
        auto rows = [&](auto count, auto values) __attribute__((always_inline)) {
            constexpr int C = count.value;
            constexpr int CV = values.value ? C : UE;
#pragma unroll
            for (int u = UE; u < C; ++u) {
                kv[u] = load16_stream(Kp + at(u, len));
            }
#pragma unroll
            for (int u = UE; u < CV; ++u) {
                vv[u] = load16_stream(Vp + at(u, len));
            }
#pragma unroll
            for (int u = CV; u < U; ++u) vv[u] = Vec16{0u, 0u, 0u, 0u};
            new_rows();
#pragma unroll
            for (int u = 0; u < C; ++u) z[u] = group_sum<LPR>(qf.dot(kv[u], 0.f)) * a.scale;
#pragma unroll
            for (int u = C; u < U; ++u) z[u] = 0.f;
        };
        // the output is formed with the exponentials themselves, one rounding less than with the weights p
        float p[SL], ex[SL], sc[SL];
        if constexpr (PHASE != 2) {
        const int stages = (m + NG * UE - 1) / (NG * UE);
        if (late) rows(std::integral_constant<int, U>(), std::false_type());
        else if (stages <= 1) rows(std::integral_constant<int, UE>(), std::true_type());
        else if (stages == 2) rows(std::integral_constant<int, 2 * UE>(), std::true_type());
        else if (stages == 3) rows(std::integral_constant<int, 3 * UE>(), std::true_type());
        else rows(std::integral_constant<int, U>(), std::true_type());
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
            ex[k] = p[k];
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
        if (a.probs_dbg) {
#pragma unroll
            for (int k = 0; k < SL; ++k)
                if (k == wave && mine < m) a.probs_dbg[pair * (int64_t)cap + mine] = p[k];
            for (int i = m + tid; i < cap; i += NT) a.probs_dbg[pair * (int64_t)cap + i] = 0.f;
        }
        if constexpr (PHASE == 1) {
            // what the second launch needs; every slot by the wave that owns its chunk
#pragma unroll
            for (int k = 0; k < SL; ++k)
                if (k == wave && mine < m) {
                    a.ws_p[pair * (int64_t)cap + mine] = p[k];
                    a.ws_snew[pair * (int64_t)cap + mine] = sc[k];
                }
        }
        } else {
            new_rows();
            // (the old positions have arrived before any wave may overwrite them)
#pragma unroll
            for (int k = 0; k < SL; ++k) asm volatile("" ::"v"(pold[k]));
            __syncthreads();                             // the sums over the heads
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const int i = lane + k * kWave;
                ex[k] = p[k] = i < m ? pw[k] : 0.f;
                sc[k] = sold[k];
                if (i >= len) pold[k] = n - 1;
            }
        }

        // ---- selection ------------------------------------------------------------------------
        // (key << 32 | ~t): min = lowest score, then the latest token; t is the slot, or the token position when slots
        // are unordered
        auto rank_key = [&](int k) -> unsigned long long {
            const uint32_t t = bag ? (uint32_t)pold[k] : (uint32_t)(lane + k * kWave);
            const float v = PHASE == 2 ? s_z[lane + k * kWave] : sc[k];
            return ((unsigned long long)order_key(v) << 32) | (uint32_t)(~t);
        };
        auto candidate = [&](int k) -> bool {
            const int i = lane + k * kWave;
            return i < m && (bag ? pold[k] < wlo : i < ncand);
        };
        uint64_t kept[SL];                               // kept slots, the same in every lane
        int jstar = m;                                   // one eviction: the evicted slot (m = none)
        int moves = 0, final_slot = kNowhere;            // listed, unordered: rows that change slot; where this lane's slot goes
        if (!listed || PHASE == 1) {
            if (E == 1 && PHASE != 1) {
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
            // Kept: what is no candidate, and of the candidates the n_global that come first, by larger importance, then by earlier
            // token.  A candidate's rank is counted, over the keys first and, where equal ones lie across the line, over their
            // tokens; the waves of a chunk share the count.  (Looking for the last kept key bit by bit in registers took twice as long.)
            if (bag) {
                int present = 0;
#pragma unroll
                for (int k = 0; k < SL; ++k) present += (int)__popcll(__ballot(lane + k * kWave < m && pold[k] >= wlo));
                n_global = keep - present;
            }
            bool open = false, stays = false;            // this lane's slot of the chunk
            uint32_t key = 0u, token = 0u;
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const bool c = candidate(k);
                const unsigned long long r = rank_key(k);
                open = k == chunk ? c : open;
                key = k == chunk ? (uint32_t)(r >> 32) : key;
                token = k == chunk ? (uint32_t)r : token;
                kept[k] = __ballot(lane + k * kWave < m && !c);
            }
            stays = mine < m && !open;
            int left = n_global;                         // how many of the open ones stay
            for (int round = 0; round < 2 && left > 0; ++round) {
                const uint32_t own = open ? (round ? token : key) : 0u;
                if (owner) s_key[mine] = own;
                if (tid == 0) s_top = 0;
                __syncthreads();
                const int part = wave / SL;
                const int hi = (part + 1) * (ROWS / PARTS) < m ? (part + 1) * (ROWS / PARTS) : m;
                int above = 0;
                for (int j = part * (ROWS / PARTS); j < hi; j += 16) {
#pragma unroll
                    for (int u = 0; u < 16; u += 4) {
                        const uint4 v = *reinterpret_cast<const uint4*>(&s_key[j + u]);
                        above += (v.x > own ? 1 : 0) + (v.y > own ? 1 : 0) + (v.z > own ? 1 : 0) + (v.w > own ? 1 : 0);
                    }
                }
                if constexpr (PARTS > 1) {
                    if (part < PARTS) s_above[part * ROWS + mine] = (uint16_t)above;
                    __syncthreads();
                    above = 0;
#pragma unroll
                    for (int q = 0; q < PARTS; ++q) above += s_above[q * ROWS + mine];
                }
                const bool in = open && above < left;
                const uint64_t b = __ballot(in || stays), c = __ballot(in);
                if (owner && lane == 0) {
                    s_mask[wave] = b;
                    s_in[wave] = (int)__popcll(c);
                }
                __syncthreads();
                int got = 0;
#pragma unroll
                for (int k = 0; k < SL; ++k) {
                    kept[k] = s_mask[k];
                    got += s_in[k];
                }
                if (__builtin_amdgcn_readfirstlane(got) <= left) break;
                // equal keys across the line: those with the most keys above them
                if (owner && in) atomicMax(&s_top, above);
                __syncthreads();
                const int top = __builtin_amdgcn_readfirstlane(s_top);
                stays = stays || (in && above < top);
                open = in && above == top;
                left -= top;
                __syncthreads();
            }
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
                        if ((mm >> lane) & 1ull) s_mov[mr] = (uint16_t)mine;
                        is_kept = (kept[k] >> lane) & 1ull;
                    }
                    holes += (int)__popcll(hm);
                    movers += (int)__popcll(mm);
                }
                __syncthreads();
                if (is_kept) final_slot = mine < keep ? mine : (mr < holes ? (int)s_hole[mr] : kNowhere);
                moves = holes < movers ? holes : movers;
            }
        }

        // ---- output: sum over the kept rows, in registers -------------------------------------
        float pk[SL];                                    // (negative: not kept)
        float ps = 0.f;
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            const bool in = (kept[k] >> lane) & 1ull;
            pk[k] = in ? ex[k] : -1.f;
            ps += in ? ex[k] : 0.f;
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
            for (int e = 0; e < EPV; ++e) acc[e] = (grp == 0 && !(wn < 0.f)) ? wn * f[e] : 0.f;
        }
        bool subtract = PHASE == 1 && listed;            // (then the second launch sums the kept rows up)
        if constexpr (PHASE == 2) {
            // one row or none leaves the dense output; where little weight would be left the kept rows are added up instead
            float pj = p[0];
#pragma unroll
            for (int k = 1; k < SL; ++k) pj = k == jstar / kWave ? p[k] : pj;
            pj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, pj), jstar & (kWave - 1)));
            if (jstar >= m) pj = 0.f;
            subtract = !listed && 1.f - pj >= kMinKeptMass;
            if (subtract && tid < LPR) {
                float f[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) f[e] = 0.f;
                if (jstar < m) unpack<T>(jstar == len ? nv : load16(Vp + jstar * ROWB + sub * 16), f);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    float t = (dense[e] - pj * f[e]) / (1.f - pj);
                    if constexpr (kQ8) t = lamK[2 * a.qstride + sub * EPV + e] * (t - lamK[3 * a.qstride + sub * EPV + e]);
                    f[e] = t;
                }
                if constexpr (kQ8) {
                    store16(a.out + pair * XROWB + sub * 32, pack<F16>(f));
                    store16(a.out + pair * XROWB + sub * 32 + 16, pack<F16>(f + 8));
                } else {
                    store16(a.out + pair * XROWB + sub * 16, pack<T>(f));
                }
            }
        }
        if (!subtract) {
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = __shfl(pk[u * NG / kWave], u * NG % kWave + grp, kWave);
        if (PHASE == 2 || late) {
#pragma unroll
            for (int u = PHASE == 2 ? 0 : UE; u < U; ++u)
                if (u * NG + grp < len && !(w[u] < 0.f)) vv[u] = load16(Vp + at(u, len));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = u * NG + grp;
            float wr = w[u];
            Vec16 x = vv[u];
            if (row >= len || wr < 0.f) {                  // evicted, new or past the end: whatever the slot holds
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
        }

        // ---- state ----------------------------------------------------------------------------
        if constexpr (PHASE != 1) {
        int32_t* kout = a.kept_idx ? a.kept_idx + pair * (int64_t)cap : nullptr;
        const int hole = (E == 1 && jstar < keep) ? jstar : m;      // one eviction: where the new token goes
        int first = 0;                                              // kept slots in the chunks before
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            if (k == wave) {
                const bool in = (kept[k] >> lane) & 1ull;
                if (!bag) {
                    if (mine < m) Sp[mine] = sc[k];
                    if (in) kout[first + (int)__popcll(kept[k] & ((1ull << lane) - 1ull))] = mine;
                } else {
                    int dst = kNowhere;
                    if (in) dst = listed ? final_slot : (mine == len && hole < m ? hole : mine);
                    if (dst < keep) {
                        Sp[dst] = sc[k];
                        if (dst != mine || mine == len) Pp[dst] = pold[k];
                        if (kout) kout[dst] = mine;
                        if constexpr (RING) Rg[(int64_t)a.ring_row * cap + dst] = p[k];
                    }
                }
            }
            first += (int)__popcll(kept[k]);
        }
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
            // The rows that change slot, the new token's among them; nobody reads what lies in their final slots.
            for (int r0 = grp; r0 < moves; r0 += 2 * NG) {
                Vec16 x[2], y[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    x[u] = nk;
                    y[u] = nv;
                    const int src = r0 + u * NG < moves ? (int)s_mov[r0 + u * NG] : len;
                    if (src != len) {
                        x[u] = load16(Kp + src * ROWB + sub * 16);
                        y[u] = load16(Vp + src * ROWB + sub * 16);
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (r0 + u * NG < moves) {
                        const int dst = s_hole[r0 + u * NG];
                        store16(Kp + dst * ROWB + sub * 16, x[u]);
                        store16(Vp + dst * ROWB + sub * 16, y[u]);
                    }
                }
            }
            if constexpr (RING) {
                // the other rows of the ring follow them; the new token has none there
                for (int j0 = wave; j0 < a.ring_rows; j0 += 4 * NW) {
                    for (int r = lane; r < moves; r += kWave) {
                        const int src = s_mov[r], dst = s_hole[r];
                        float v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int j = j0 + u * NW;
                            v[u] = (src != len && j < a.ring_rows) ? Rg[(int64_t)j * cap + src] : 0.f;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int j = j0 + u * NW;
                            if (j < a.ring_rows && j != a.ring_row) Rg[(int64_t)j * cap + dst] = v[u];
                        }
                    }
                }
            }
        }

        }

        __syncthreads();
        if (!subtract)
        for (int e = tid; e < D; e += NT) {
            float t = 0.f;
#pragma unroll
            for (int v = 0; v < NW; ++v) t += s_acc[v * D + e];
            t /= ps;
            if constexpr (PHASE == 1) {
                a.ws_abar[pair * D + e] = t;
                continue;
            }
            if constexpr (kQ8) t = lamK[2 * a.qstride + e] * (t - lamK[3 * a.qstride + e]);      // accumulated in code space
            store_elem<AT>(a.out + pair * XROWB, e, keep > 0 ? t : 0.f);      // an empty budget: an empty sum
        }
    }

    if (PHASE != 1 && tid == 0) {
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

// go<T, D, NT, U>() for the form and the formats of a call.
template <typename T, int D, typename G>
int with_form(ShortForm f, const G& g)
{
    if (f.nt == 128) return g.template go<T, D, 128, short_unroll<T, D>(8)>();
    if (f.nt == 512) return g.template go<T, D, 512, short_unroll<T, D>(8)>();
    if (f.u == 12) return g.template go<T, D, 256, short_unroll<T, D>(12)>();
    return g.template go<T, D, 256, short_unroll<T, D>(8)>();
}

template <typename G>
int with_form(const swa_params& p, ShortForm f, const G& g)
{
    if (p.flags & SWA_KV_INT8) return p.d == 64 ? with_form<Q8, 64>(f, g) : with_form<Q8, 128>(f, g);
    if (p.dtype == SWA_F32) return p.d == 64 ? with_form<F32, 64>(f, g) : with_form<F32, 128>(f, g);
    if (p.dtype == SWA_F16) return p.d == 64 ? with_form<F16, 64>(f, g) : with_form<F16, 128>(f, g);
    return p.d == 64 ? with_form<BF16, 64>(f, g) : with_form<BF16, 128>(f, g);
}

}  // namespace swa
