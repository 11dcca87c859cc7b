// Workgroup-level pieces of the selection (Algorithm 1 lines 3-5): the threshold of a top-k over 32-bit keys, and the
// prefix sum that places what was kept.
#pragma once

#include "swa_device.hpp"

namespace swa {

// Monotone map fp32 -> uint32 (larger float <=> larger key).
__device__ __forceinline__ uint32_t order_key(float f)
{
    uint32_t u = f2u(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// LDS of one workgroup's selection.
template <int NT>
struct SelectScratch {
    int32_t hist[2 * NT];          // two bins per thread
    uint32_t lo[NT / kWave], hi[NT / kWave];
    int32_t cnt[NT / kWave];
    int32_t sel[3];
};

// The `want`-th largest (want >= 1, at most the number of candidates) of the candidate keys, as a
// threshold: keys above thr are kept, and of the n_eq keys equal to thr the first rem (n_eq == rem: all).
// each(f) calls f(key) for every candidate key of the calling thread; every thread of the workgroup takes part.
//
// Histogram select with 2 NT bins over the range the keys really span (a radix select from the top of the word has its
// first digit, sign and exponent, shared by nearly all keys, and its counters serialise), refined inside the
// bin that holds the threshold until all of that bin is kept or its keys are equal.  Importance values of
// a cache are spread enough that this takes two rounds as a rule, and never more than four.
template <int NT, typename Each>
__device__ __forceinline__ void select_threshold(SelectScratch<NT>& s, int want, Each each, uint32_t& thr, int& rem, int& n_eq)
{
    constexpr int NW = NT / kWave;
    constexpr int LB = NT == 1024 ? 11 : (NT == 512 ? 10 : (NT == 256 ? 9 : 8));
    static_assert(2 * NT == 1 << LB, "two bins per thread");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    uint32_t kmin = 0xffffffffu, kmax = 0u;
    each([&](uint32_t key) {
        kmin = key < kmin ? key : kmin;
        kmax = key > kmax ? key : kmax;
    });
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t a = (uint32_t)__shfl_xor((int)kmin, o, kWave), b = (uint32_t)__shfl_xor((int)kmax, o, kWave);
        kmin = a < kmin ? a : kmin;
        kmax = b > kmax ? b : kmax;
    }
    if (lane == 0) {
        s.lo[wave] = kmin;
        s.hi[wave] = kmax;
    }
    if (tid == 0) {
        s.sel[0] = 0;
        s.sel[1] = s.sel[2] = want;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        kmin = s.lo[v] < kmin ? s.lo[v] : kmin;
        kmax = s.hi[v] > kmax ? s.hi[v] : kmax;
    }
    uint32_t lo = kmin;
    uint32_t top = kmax >= kmin ? kmax - kmin : 0u;      // largest offset from lo that still belongs to the range
    int left = want;
    for (;;) {
        const int bits = top ? 32 - __builtin_clz(top) : 0;
        const int shift = bits > LB ? bits - LB : 0;
        s.hist[2 * tid] = 0;
        s.hist[2 * tid + 1] = 0;
        __syncthreads();
        each([&](uint32_t key) {
            const uint32_t off = key - lo;
            if (key >= lo && off <= top) atomicAdd(&s.hist[off >> shift], 1);
        });
        __syncthreads();
        const int c0 = s.hist[2 * tid], c1 = s.hist[2 * tid + 1];
        int suf = c0 + c1;                                // inclusive suffix sum over the wave's lanes
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int t = __shfl_down(suf, o, kWave);
            if (lane + o < kWave) suf += t;
        }
        if (lane == 0) s.cnt[wave] = suf;
        __syncthreads();
        int above = suf - c0 - c1;                        // keys in higher bins
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
        if (shift == 0 || left == s.sel[2]) break;        // equal keys, or the whole bin is kept
    }
    thr = lo;
    rem = left;
    n_eq = s.sel[2];
}

// Exclusive prefix sum of v over the threads of the workgroup, and the total.  s_cnt: NT / 64 words of LDS.
template <int NT>
__device__ __forceinline__ void block_scan(int32_t* s_cnt, int v, int& before, int& total)
{
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += t;
    }
    if (lane == kWave - 1) s_cnt[wave] = inc;
    __syncthreads();
    int wb = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int c = s_cnt[w];
        if (w < wave) wb += c;
        tot += c;
    }
    before = wb + inc - v;
    total = tot;
    __syncthreads();
}

// Ordered compaction of one thread's contiguous run of at most 64 slots: the slots to keep as a mask.  surem: kept for
// sure; eqm: equal to the threshold, of which the workgroup keeps the first rem.
template <int NT>
__device__ __forceinline__ uint64_t keep_mask(int32_t* s_cnt, uint64_t surem, uint64_t eqm, int rem)
{
    int eq_before = 0, eq_total = 0;
    block_scan<NT>(s_cnt, (int)__popcll(eqm), eq_before, eq_total);
    int take = rem - eq_before;
    while (take > 0 && eqm != 0ull) {
        const uint64_t low = eqm & (~eqm + 1ull);
        surem |= low;
        eqm ^= low;
        --take;
    }
    return surem;
}

}  // namespace swa
