// Workgroup-level piece of the selection (Algorithm 1 lines 3-5): the threshold of a top-k over 32-bit keys.
#pragma once

#include "swa_device.hpp"

namespace swa {

// Monotone map fp32 -> uint32 (larger float <=> larger key).
__device__ __forceinline__ uint32_t order_key(float f)
{
    uint32_t u = f2u(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ... and back.
__device__ __forceinline__ float key_value(uint32_t key) { return u2f((key & 0x80000000u) ? key ^ 0x80000000u : ~key); }

// Sum over the lanes up to and including this one.
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);      // row_shr 1, 2, 4, 8 within 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // lane 15 of a row into the next, odd rows
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // lane 31 into the upper half
    return v;
}

template <int CTRL>
__device__ __forceinline__ void min_max_dpp(uint32_t& lo, uint32_t& hi)
{
    const uint32_t a = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, CTRL, 0xf, 0xf, true);
    const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, 0xf, 0xf, true);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
}

// Largest of a wave's values, none of them negative, in every lane.
__device__ __forceinline__ int wave_max_int(int v)
{
    auto step = [&](int o) { v = o > v ? o : v; };
    step(__builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true));
    step(__builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true));
    step(__builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true));
    step(__builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true));
    step(__builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));     // lane 15 of a row into the next, odd rows
    step(__builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));     // lane 31 into the upper half
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

// Smallest and largest of a wave's values, in every lane.
__device__ __forceinline__ void wave_min_max(uint32_t& lo, uint32_t& hi)
{
    min_max_dpp<0xB1>(lo, hi);
    min_max_dpp<0x4E>(lo, hi);
    min_max_dpp<0x141>(lo, hi);
    min_max_dpp<0x140>(lo, hi);
#pragma unroll
    for (int o = 16; o < kWave; o <<= 1) {
        const uint32_t a = (uint32_t)__shfl_xor((int)lo, o, kWave), b = (uint32_t)__shfl_xor((int)hi, o, kWave);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
}

// LDS of one workgroup's selection.
template <int NT>
struct SelectScratch {
    int32_t hist[2 * NT];          // two bins per thread, zero before and after a selection
    uint32_t lo[NT / kWave], hi[NT / kWave];
    int32_t cnt[NT / kWave];
    int32_t sel[3];
    int32_t listed;                // keys of the bin that holds the threshold, once they are few; zero before a selection
    int32_t rank[kWave];           // ... and how many of them are larger; zero before a selection
    __align__(16) uint32_t list[kWave];
};

// Smallest and largest candidate key.  each(f) calls f(key) for every candidate key of the calling thread; every thread of the
// workgroup takes part.
template <int NT, typename Each>
__device__ __forceinline__ void key_range(SelectScratch<NT>& s, Each each, uint32_t& kmin, uint32_t& kmax)
{
    constexpr int NW = NT / kWave;
    kmin = 0xffffffffu;
    kmax = 0u;
    each([&](uint32_t key) {
        kmin = key < kmin ? key : kmin;
        kmax = key > kmax ? key : kmax;
    });
    wave_min_max(kmin, kmax);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s.lo[threadIdx.x >> 6] = kmin;
        s.hi[threadIdx.x >> 6] = kmax;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        kmin = s.lo[v] < kmin ? s.lo[v] : kmin;
        kmax = s.hi[v] > kmax ? s.hi[v] : kmax;
    }
}

// The `want`-th largest (want >= 1, at most the number of candidates) of the candidate keys, as a
// threshold: keys above thr are kept, and of the n_eq keys equal to thr the first rem (n_eq == rem: all).
// Every candidate key lies in kmin .. kmax; hist, listed and rank are zero, and a barrier has passed since they were cleared.
//
// Histogram select with 2 NT bins over kmin .. kmax (a radix select from the top of the word has its
// first digit, sign and exponent, shared by nearly all keys, and its counters serialise), refined inside the
// bin that holds the threshold until all of that bin is kept, its keys are equal or there are so few that
// they can be listed and ranked.  Importance values of a cache are spread enough that this takes one round and
// the list as a rule, and never more than four rounds.  A range that begins at zero (an importance that nothing has seeded) has 16 bins an octave
// and as a rule a second round, which costs what finding the keys' own range did: first step, f16, d = 128, seeded / not, 32 pairs x
// 8192 40.0 / 39.1 us (with the own range 40.9 / 40.6), 128 x 8192 79.0 / 79.6 (80.2 / 80.1).
//
// Bound: the instructions that 16 waves on one CU issue, and barriers: the ranks are counted by all waves together (32 pairs x 8192: 5400 ->
// 3900 clocks for list and ranks).
template <int NT, typename Each>
__device__ __forceinline__ void select_threshold(SelectScratch<NT>& s, int want, uint32_t kmin, uint32_t kmax, Each each, uint32_t& thr,
                                                 int& rem, int& n_eq)
{
    constexpr int NW = NT / kWave;
    constexpr int LB = NT == 1024 ? 11 : (NT == 512 ? 10 : (NT == 256 ? 9 : 8));
    static_assert(2 * NT == 1 << LB, "two bins per thread");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    uint32_t lo = kmin;
    uint32_t top = kmax >= kmin ? kmax - kmin : 0u;      // largest offset from lo that still belongs to the range
    int left = want;
    for (bool whole = true;; whole = false) {
        const int bits = top ? 32 - __builtin_clz(top) : 0;
        const int shift = bits > LB ? bits - LB : 0;
        if (whole) {
            each([&](uint32_t key) {
                const uint32_t bin = (key - lo) >> shift;
                atomicAdd(&s.hist[bin < 2 * NT ? bin : 2 * NT - 1], 1);
            });
        } else {
            each([&](uint32_t key) {
                const uint32_t off = key - lo;
                if (key >= lo && off <= top) atomicAdd(&s.hist[off >> shift], 1);
            });
        }
        if (tid == 0) {
            s.sel[0] = 0;
            s.sel[1] = s.sel[2] = left;
        }
        __syncthreads();
        const int c0 = s.hist[2 * tid], c1 = s.hist[2 * tid + 1];
        s.hist[2 * tid] = 0;
        s.hist[2 * tid + 1] = 0;
        const int upto = wave_scan(c0 + c1);
        const int total = __builtin_amdgcn_readlane(upto, kWave - 1);
        if (lane == 0) s.cnt[wave] = total;
        __syncthreads();
        int above = total - upto;                         // keys in higher bins
#pragma unroll
        for (int v = 0; v < NW; ++v)
            if (v > wave) above += s.cnt[v];
        if (above < left && left <= above + c1) {
            s.sel[0] = 2 * tid + 1;
            s.sel[1] = left - above;
            s.sel[2] = c1;
        } else if (above + c1 < left && left <= above + c1 + c0) {
            s.sel[0] = 2 * tid;
            s.sel[1] = left - above - c1;
            s.sel[2] = c0;
        }
        __syncthreads();
        lo += (uint32_t)s.sel[0] << shift;
        top = (1u << shift) - 1u;
        left = s.sel[1];
        n_eq = s.sel[2];
        if (shift == 0 || left == n_eq) break;            // equal keys, or the whole bin is kept
        if (n_eq <= kWave) {
            // a bin of few keys: listed, and their ranks counted by all waves, four keys to compare with each (NW = 16)
            each([&](uint32_t key) {
                if (key >= lo && key - lo <= top) s.list[atomicAdd(&s.listed, 1)] = key;
            });
            __syncthreads();
            const uint32_t mine = s.list[lane];
            for (int j = 4 * wave; j < n_eq; j += 4 * NW) {
                const uint4 o = *reinterpret_cast<const uint4*>(&s.list[j]);
                int larger = o.x > mine ? 1 : 0;
                larger += (j + 1 < n_eq && o.y > mine) ? 1 : 0;
                larger += (j + 2 < n_eq && o.z > mine) ? 1 : 0;
                larger += (j + 3 < n_eq && o.w > mine) ? 1 : 0;
                if (larger) atomicAdd(&s.rank[lane], larger);
            }
            __syncthreads();
            // the wanted key: of those with fewer than `left` larger ones the one with most
            const int larger = s.rank[lane];
            const bool in = lane < n_eq && larger < left;
            int most = in ? larger : 0;
            most = wave_max_int(most);
            const uint64_t at = __ballot(in && larger == most);
            lo = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)__builtin_ctzll(at));
            left -= most;
            n_eq = (int)__popcll(at);
            break;
        }
        __syncthreads();                                  // everyone has read the result of this round
    }
    thr = lo;
    rem = left;
}

}  // namespace swa
