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
#include <type_traits>

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
    // A slice's first 2 R `chains` output columns (score, or row 0 of the ring) bring it the row statistics from the
    // launch before: for every chain maximum of row r at [r], normaliser at [R + r], the next chain's 2 R columns further on.
    int32_t G, cols;
    int32_t bound;        // on the lengths: where the slices are laid (host side)
    bool stated;          // the bound is the caller's, not the capacity (host side)
    int32_t chains;       // statistics: parts of the keys whose sums are still to be merged, kChains or 1
};

// What one launch does.
constexpr int kSeedWhole = 0;   // both passes, one workgroup per pair
constexpr int kSeedStats = 1;   // row statistics of 32 rows of one pair, a copy for every slice
constexpr int kSeedSums = 2;    // column sums of one slice, from the row statistics of another launch
constexpr int kSeedSumsFar = 3; // the same, keys read past the caches (16-bit formats)
constexpr int kChains = 4;      // row statistics: key tile t belongs to chain t % 4, whose sums are merged in ascending order

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

// Row statistics of this lane's query after one more key tile: C[key][query] of the tile, its keys up to tmax (the
// last one that the query sees).
__device__ __forceinline__ void add_tile_stats(const float16_t& c, int tile, int hb, int tmax, float scale_log2e, float& M, float& L)
{
    float z[16];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int key = tile * 32 + 8 * (i / 4) + 4 * hb + (i % 4);
        z[i] = (key <= tmax) ? c[i] * scale_log2e : -INFINITY;
        mx = fmaxf(mx, z[i]);
    }
    if (mx > -INFINITY) {
        const float Mn = fmaxf(M, mx);
        float acc = L * __builtin_amdgcn_exp2f(M - Mn);   // 0 while M is -inf
#pragma unroll
        for (int i = 0; i < 16; ++i) acc += __builtin_amdgcn_exp2f(z[i] - Mn);
        M = Mn;
        L = acc;
    }
}

// The same without branches, for tiles that every row sees to their end (SEEN) or any.
template <bool SEEN>
__device__ __forceinline__ void add_tile_stats_flat(const float16_t& c, int tile, int hb, int tmax, float scale_log2e, float& M,
                                                    float& L)
{
#pragma clang fp contract(off)
    float z[16];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int key = tile * 32 + 8 * (i / 4) + 4 * hb + (i % 4);
        z[i] = c[i] * scale_log2e;
        if (!SEEN) z[i] = (key <= tmax) ? z[i] : -INFINITY;
        mx = fmaxf(mx, z[i]);
    }
    const float Mn = fmaxf(M, mx);
    float acc = __builtin_fmaf(L, __builtin_amdgcn_exp2f(M - Mn), __builtin_amdgcn_exp2f(z[0] - Mn));   // (0 + .. while M is -inf)
#pragma unroll
    for (int i = 1; i < 16; ++i) acc += __builtin_amdgcn_exp2f(z[i] - Mn);
    asm volatile("" : "+v"(acc));                         // (formed in any case: a branch here would end the overlap)
    L = mx > -INFINITY ? acc : L;
    M = mx > -INFINITY ? Mn : M;
}

// Row statistics of 32 query rows over one chain of key tiles (NW = 1) or over all four, merged (NW = 4): the same sums in the
// same order as in the kernel below, whose pass 1 this is where a pair's keys are long and pairs few.
//
// Bound: the chain of a tile's steps in the one wave that owns it, 0.6 us a tile (32 pairs x 8192 keys, f16, d = 128, R =
// 64: 37 us; 60 with the operands' own layout and 64 workgroups).  A tile's rows are loaded as they lie, whole lines by one
// instruction (an operand's own layout takes 32 bytes of a line at a time, and lines were lost between their
// uses), and reach that layout by way of LDS, in which a row's 16-byte chunks are permuted by the row
// so that the lanes of a read spread over the banks.  A chain cannot be cut (its sum has an order), so its one wave
// overlaps what a tile needs: loads, LDS, products and exponentials of different tiles.  Rows of 512 bytes (fp32, d = 128) leave no
// registers for that and are bound by their products; they keep the operands' own layout (kSeedStats below; whole seed, 32
// pairs x 4096 keys, R = 64: 111 us, 118 by way of LDS; 32 keys 17.6 / 21.9).
template <typename T, int D, bool WR, int NW>
__global__ void __launch_bounds__(NW * kWave) __attribute__((amdgpu_waves_per_eu(1, 1)))
swa_seed_stats_kernel(PrefillArgs a)
{
    constexpr int ROWB = D * Elem<T>::kBytes;
    constexpr int NV = (ROWB / 2) / 16;
    constexpr int CPR = ROWB / 16;                   // chunks of a row
    constexpr int RPI = kWave / CPR;                 // rows per load instruction
    constexpr int NL = 32 / RPI;                     // loads per lane and tile
    constexpr int AHEAD = 4;                         // tiles requested ahead (even: the two tiles of fragments alternate)
    static_assert(ROWB < 512, "no registers for wider rows");
    __shared__ __align__(16) char s_tile[NW][32 * ROWB];
    __shared__ float s_m[NW][32], s_l[NW][32];

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int l32 = lane & 31;
    const int hb = lane >> 5;
    // the row tiles of a pair read the same keys: their workgroups are a multiple of the number of XCDs apart
    // where the pairs are, and share an L2
    const uint32_t per = (uint32_t)(kChains / NW), all = gridDim.x / (uint32_t)((a.R + 31) / 32);
    const int rt0 = (int)(blockIdx.x / all);
    const int64_t pair = (blockIdx.x % all) / per;
    const int chain = NW == 1 ? (int)(blockIdx.x % per) : wave;
    const int cap = a.cap;
    const int R = a.R;
    int s = a.cache_len[pair / a.h];
    s = s > cap ? cap : s;
    if (s <= 0) return;
    const char* Kp = a.k_cache + pair * (int64_t)cap * ROWB;
    const int qbase = a.q_in_place ? s - R : 0;
    const char* Qp = a.q_tail + pair * (int64_t)(a.q_in_place ? cap : R) * ROWB;
    const int r = rt0 * 32 + l32;
    const int qrow = qbase + r > 0 ? qbase + r : 0;
    Vec16 qv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v)
        qv[v] = (r < R) ? load16(Qp + (int64_t)qrow * ROWB + v * 32 + hb * 16) : Vec16{0u, 0u, 0u, 0u};
    const int tmax = (r < R) ? s - R + r : -1;
    const int tiles = (s + 31) / 32;

    const int lrow = lane / CPR, lchunk = lane % CPR;
    const uint32_t lane_at = (uint32_t)lrow * ROWB + (uint32_t)lchunk * 16, last_at = (uint32_t)(s - 1) * ROWB + (uint32_t)lchunk * 16;
    // tile t of the chain (unconditional: rows past the end re-read the last one and are masked)
    auto request = [&](int t, Vec16(&kr)[NL]) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const uint32_t at = lane_at + (uint32_t)((chain + t * kChains) * 32 + j * RPI) * ROWB;
            kr[j] = load16(Kp + (at < last_at ? at : last_at));
        }
    };
    char* buf = s_tile[wave];
    // Rows pass between the lanes of one wave: its LDS accesses are carried out in order, the fences keep the compiler from changing it.
    auto wave_order = []() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    };
    auto stage = [&](const Vec16(&kr)[NL], Vec16(&f)[NV]) {
        wave_order();
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int row = j * RPI + lrow;
            *reinterpret_cast<Vec16*>(buf + row * ROWB + ((lchunk ^ (row & (CPR - 1))) * 16)) = kr[j];
        }
        wave_order();
#pragma unroll
        for (int v = 0; v < NV; ++v)
            f[v] = *reinterpret_cast<const Vec16*>(buf + l32 * ROWB + (((2 * v + hb) ^ (l32 & (CPR - 1))) * 16));
    };
    auto products = [&](const Vec16(&f)[NV]) -> float16_t {
        float16_t c;
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
        for (int v = 0; v < NV; ++v) c = Mfma<T>::run(f[v], qv[v], c);      // C[key][query]
        return c;
    };
    // While a tile's weights are summed, the next one's products run and the rows of the one behind it go through LDS.
    float M = -INFINITY, L = 0.f;
    const int nt = (tiles - chain + kChains - 1) / kChains;      // (0 or less: nothing to do)
    const int seen = (s - R + rt0 * 32 + 1) / 32;                // tiles below it: every row sees all keys
    Vec16 kr[AHEAD][NL], f[2][NV];
    float16_t c;
    if (nt > 0) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) request(u, kr[u]);
        stage(kr[0], f[0]);
        c = products(f[0]);
    }
    // A chain's last tiles from t on, fewer than a round or as many: nothing is formed or waited for behind its end.  (In the loop below a
    // prompt of 32 keys pays for eight tiles: whole seed, 32 pairs in 4096 slots, R = 64, fp32, d = 64 16.4 / 11.5 us, f16, d = 128 11.0 /
    // 9.5.)  In 16 bits for chains of no more than a round alone: behind the loop it cost 0.5 us from 1024 keys on, and 700 keys are
    // fast as they are (kernel before this one / now 20.7 / 18.3 us).  fp32 gains more than that: 700 keys 31.0 / 27.6.
    constexpr bool kRest = Elem<T>::kBytes == 4;
    auto rest = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (t + u >= nt) break;
            float16_t next = c;
            if (t + u + 2 < nt) stage(kr[(u + 2) % AHEAD], f[u % 2]);
            if (t + u + 1 < nt) next = products(f[(u + 1) % 2]);
            add_tile_stats_flat<false>(c, chain + (t + u) * kChains, hb, tmax, a.scale_log2e, M, L);
            c = next;
        }
    };
    if (nt > AHEAD) {
        stage(kr[1], f[1]);
        request(AHEAD, kr[0]);
        request(AHEAD + 1, kr[1]);
        int t = 0;
        for (; kRest ? t + AHEAD <= nt : t < nt; t += AHEAD) {
            auto some = [&](auto all_seen) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    stage(kr[(u + 2) % AHEAD], f[u % 2]);                       // tile t + u + 2
                    const float16_t next = products(f[(u + 1) % 2]);
                    add_tile_stats_flat<all_seen.value>(c, chain + (t + u) * kChains, hb, tmax, a.scale_log2e, M, L);
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 64 / NV + 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x400, 16 / NV, 0);
                    }
                    c = next;
                    request(t + u + AHEAD + 2, kr[(u + 2) % AHEAD]);
                }
            };
            if (chain + (t + AHEAD - 1) * kChains < seen) some(std::true_type());
            else some(std::false_type());
        }
        if constexpr (kRest) rest(t);
    } else {
        if (nt > 1) stage(kr[1], f[1]);
        rest(0);
    }
    const float M2 = __shfl_xor(M, 32, kWave);
    const float L2 = __shfl_xor(L, 32, kWave);
    merge_stats(M, L, M2, L2);
    if constexpr (NW > 1) {
        if (hb == 0) {
            s_m[wave][l32] = M;
            s_l[wave][l32] = L;
        }
        __syncthreads();
        if (wave != 0 || hb != 0) return;
#pragma unroll
        for (int v = 1; v < NW; ++v) merge_stats(M, L, s_m[v][l32], s_l[v][l32]);
    }
    if (hb == 0 && r < R) {
        float* St = (WR ? a.rows + pair * (int64_t)R * cap : a.score + pair * (int64_t)cap) + (NW == 1 ? chain * 2 * R : 0);
        for (int g = 0; g < a.G; ++g) {
            St[(int64_t)g * a.cols + r] = M;
            St[(int64_t)g * a.cols + R + r] = L;
        }
    }
}

// How key tiles reach the operands' layout.  By LDS (16-bit formats): every wave has room for one tile; its rows go there straight from
// memory as they lie, whole lines by one instruction, and are read back as operands, and the next tile is requested as soon as they
// are in registers.  Bound: HBM, two reads of the keys at 6.2 TB/s where they are many; before, tiles were loaded in the operands' layout, 32 bytes of
// a line at a time, and lines were fetched again between their uses.  Whole seed before / now, us: 1792 pairs x 4096 keys, bf16, d =
// 128, R = 64 640 / 609; 2560 x 1024 f16 219 / 196; 320 x 8000 299 / 234; 512 x 512 24.4 / 21.6; 8192 of 100..500, d = 64, R = 33
// 155 / 121; 6400 of 17..31 47 / 31; sums after the attention, 1792 x 4096 387 / 308 (differences of whole calls).  Room for two or four
// tiles leaves fewer workgroups on a CU: no gain, up to 1.6 times as slow.
// The sums behind the attention find their code cold, so what is fixed in a launch (whether the loads pass the caches, whether there is a
// score at all, whether a tile can be seen by all rows) is fixed in the code and not asked in the loop, which the compiler
// copied for every answer: attention and sums before LDS / with copies / without, us: 40 pairs of 69..279 keys, d = 64, R = 33 12.7 /
// 13.1 / 12.9, d = 128, R = 128 22.8 / 23.4 / 22.7; 128 of 200..256, d = 64, R = 33 14.3 / 14.7 / 14.4; rows, 32 x 1000, R = 16 20.5 / 18.5 /
// 16.8, R = 64 30.9 / 30.8 / 29.3.  Up to 64 keys with more than 96 rows at d = 128 are 2 to 4 % slower than before LDS (2048 of 17..31 74.5 / 77.1).
// fp32 is bound by its products and keeps the operands' layout (d = 64, R = 33 476 / 508 by LDS), and so do more than 32 rows that are written
// out, whose stores the wait for a tile would wait for as well (320 x 8000, R = 64 546 / 565; up to 32 rows 512 x 512 23.4 / 21.4).
template <typename T, int RT, bool WR, int MODE>
constexpr bool kSeedByLds = Elem<T>::kBytes == 2 && !(WR && RT > 1) && MODE != kSeedStats;

// Sum of a tile's column over the R rows, for the lane's key: logits again, weights from the rows' statistics.  For tiles loaded in the
// operands' layout; the kernel has it a second time, with a form that skips the mask, for tiles by way of LDS, in 16 bits (one body for both:
// fp32's sums of 97 to 128 rows spill 134 registers instead of 97, 512 pairs x 2048 keys 897 / 914 us; this function for both: 16 bits 1 to 3 %
// slower where prompts are short).
template <typename T, int RT, bool WR, int NV>
__device__ __forceinline__ float tile_colsum(const Vec16(&qv)[RT][NV], const Vec16(&kv)[NV], const float* s_M, const float* s_invL, int hb,
                                             int key, int R, int t_off, float scale_log2e, float* Rp, int cap, int s)
{
#pragma clang fp contract(off)
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
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(c[4 * g + j], scale_log2e, -Mr[j])) * Ir[j];
                colsum += vis ? p : 0.f;
                if constexpr (WR) {
                    if (r < R && key < s) Rp[(int64_t)r * cap + key] = vis ? p : 0.f;
                }
            }
        }
    }
    return colsum + __shfl_xor(colsum, 32, kWave);
}

// Tiles by way of LDS: chunk c of row r lies at c ^ swizzle(r), chosen by the lane's global address, so that the lanes of an
// operand's read spread over the banks.
template <int ROWB, int NW, bool FAR>
struct KeyTiles {
    static constexpr int TILE = 32 * ROWB;
    static constexpr int CPR = ROWB / 16;                // 16-byte chunks per row
    static constexpr int RPI = kWave / CPR;              // rows per load instruction
    static constexpr int NV = CPR / 2;
    const char* Kp;
    const char* mine;                                    // this wave's room
    int s, lane;

    __device__ __forceinline__ KeyTiles(const char* keys, int len, int wave, int lane_) : Kp(keys), s(len), lane(lane_)
    {
        __shared__ __align__(1024) char room[NW][TILE];
        mine = room[wave];
    }
    static __device__ __forceinline__ int swz(int r) { return ROWB == 256 ? (r & 15) : ((r >> 1) & 7); }
    __device__ __forceinline__ void request(int tile) const
    {
        const uint32_t at = lds_address(mine);
        const int r_last = s - 1 - tile * 32;            // (rows past the prompt re-read its last one and are masked)
        const char* base = Kp + (uint32_t)tile * TILE;
#pragma unroll
        for (int x = 0; x < TILE / 1024; ++x) {
            const int j = x * RPI + lane / CPR;
            const uint32_t off = (uint32_t)(j < r_last ? j : r_last) * ROWB + (uint32_t)(((lane % CPR) ^ swz(j)) * 16);
            load_to_lds<FAR>(base, off, at + x * 1024);
        }
    }
    __device__ __forceinline__ void receive(Vec16(&kv)[NV]) const
    {
        __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0): the tile is there
        asm volatile("" ::: "memory");
        const int l32 = lane & 31, hb = lane >> 5;
        const char* at = mine + l32 * ROWB;
#pragma unroll
        for (int v = 0; v < NV; ++v) kv[v] = load16(at + (((2 * v + hb) ^ swz(l32)) << 4));
        __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0): it may be overwritten
        asm volatile("" ::: "memory");
    }
};

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
    constexpr bool kByLds = kSeedByLds<T, RT, WR, MODE>;
    constexpr bool kStats = MODE == kSeedStats;
    constexpr bool kSums = MODE == kSeedSums || MODE == kSeedSumsFar;
    const int row_tiles = kStats ? (a.R + 31) / 32 : 1;
    const int64_t pair = kSums ? blockIdx.x / a.G : blockIdx.x / row_tiles;
    const int rt0 = kStats ? blockIdx.x % row_tiles : 0;        // first row tile of this workgroup
    const int g = kSums ? blockIdx.x % a.G : 0;
    const int cap = a.cap;
    const int R = a.R;
    int s = a.cache_len[pair / a.h];
    s = s > cap ? cap : s;
    // the columns this workgroup owns; it reads the key tiles among them
    const int col0 = kSums ? g * a.cols : 0;
    const int col1 = (!kSums || g == a.G - 1) ? cap : col0 + a.cols;
    float* Sp = WR ? nullptr : a.score + pair * (int64_t)cap;      // (either the sums or the rows)
    float* Rp = WR ? a.rows + pair * (int64_t)R * cap : nullptr;

    if (s <= 0) {
        if (kStats) return;
        if (!WR)
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
        const uint32_t at = (uint32_t)krow * ROWB + (uint32_t)lane_off;      // (cap <= SWA_MAX_CAP: below 8 MiB)
#pragma unroll
        for (int v = 0; v < NV; ++v) kv[v] = load16(Kp + at + v * 32);
    };

    if constexpr (!kSums) {
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
            const int r = (rt0 + rt) * 32 + l32;
            const int tmax = (r < R) ? t_off + r : -1;   // last visible key of this lane's query
            float16_t c;
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
            for (int v = 0; v < NV; ++v) c = Mfma<T>::run(kv[v], qv[rt][v], c);   // C[key][query]
            add_tile_stats(c, tile, hb, tmax, a.scale_log2e, M[rt], L[rt]);
        }
    };
    if constexpr (kStats) {
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
    } else if constexpr (kByLds) {
        const int wave_u = __builtin_amdgcn_readfirstlane(wave);
        const KeyTiles<ROWB, NW, MODE == kSeedSumsFar> tiles(Kp, s, wave_u, lane);
        auto logits = [](const Vec16(&rows)[NV], const Vec16(&cols)[NV]) __attribute__((always_inline)) {
            float16_t c;
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
            for (int v = 0; v < NV; ++v) c = Mfma<T>::run(rows[v], cols[v], c);
            return c;
        };
        const int seen = RT * 32 <= R ? (t_off + 1) / 32 : 0;     // tiles below it: every row sees all keys
        if (tile0 + wave_u < tile1) tiles.request(tile0 + wave_u);
        for (int tile = tile0 + wave_u; tile < tile1; tile += NW) {
            Vec16 kv[NV];
            tiles.receive(kv);
            if (tile + NW < tile1) tiles.request(tile + NW);
            auto stats = [&](auto all_seen) __attribute__((always_inline)) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const int r = rt * 32 + l32;
                    add_tile_stats_flat<all_seen.value>(logits(kv, qv[rt]), tile, hb, (r < R) ? t_off + r : -1, a.scale_log2e, M[rt], L[rt]);
                }
            };
            if (tile < seen) stats(std::true_type());
            else stats(std::false_type());
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
        if constexpr (kStats) {
            const int r = rt0 * 32 + tid;
            if (r < R) {
                for (int g2 = 0; g2 < a.G; ++g2) {
                    St[(int64_t)g2 * a.cols + r] = Mt;
                    St[(int64_t)g2 * a.cols + R + r] = Lt;
                }
            }
            return;
        }
        const bool ok = Mt > -INFINITY && Lt > 0.f;
        s_M[tid] = ok ? Mt : 0.f;
        s_invL[tid] = ok ? 1.f / Lt : 0.f;
    }
    if constexpr (kStats) return;
    __syncthreads();
    }
    if constexpr (kSums) {
        if (tid < RP) {
            const bool row = tid < R && t_off + tid >= 0;
            float Mt = row ? St[tid] : -INFINITY, Lt = row ? St[R + tid] : 0.f;
            if (ROWB < 512 && a.chains > 1) {          // (rows of 512 bytes come merged; their kernels have no register to spare)
                float M2[kChains], L2[kChains];
#pragma unroll
                for (int v = 1; v < kChains; ++v) {
                    M2[v] = row ? St[v * 2 * R + tid] : -INFINITY;
                    L2[v] = row ? St[v * 2 * R + R + tid] : 0.f;
                }
#pragma unroll
                for (int v = 1; v < kChains; ++v) merge_stats(Mt, Lt, M2[v], L2[v]);
            }
            const bool ok = Mt > -INFINITY && Lt > 0.f;
            s_M[tid] = ok ? Mt : 0.f;
            s_invL[tid] = ok ? 1.f / Lt : 0.f;
        }
        __syncthreads();          // read by everyone before the slice's columns are written
    }

    // ------------------------------ pass 2: column sums ---------------------------------
    if constexpr (kByLds) {
        const int wave_u = __builtin_amdgcn_readfirstlane(wave);
        const KeyTiles<ROWB, NW, MODE == kSeedSumsFar> tiles(Kp, s, wave_u, lane);
        auto colsum_tile = [&](auto all_seen, int tile, const Vec16(&kv)[NV], auto take) {
#pragma clang fp contract(off)
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
                        const bool vis = all_seen.value || ((r < R) && (key <= t_off + r));
                        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(c[4 * g + j], a.scale_log2e, -Mr[j])) * Ir[j];
                        colsum += vis ? p : 0.f;
                        if constexpr (WR) {
                            if (r < R && key < s) Rp[(int64_t)r * cap + key] = vis ? p : 0.f;
                        }
                    }
                }
            }
            colsum += __shfl_xor(colsum, 32, kWave);
            take(key, colsum);
        };
        auto put = [&](int key, float colsum) {
            if (!WR && hb == 0 && key < s) Sp[key] = colsum;
        };
        const int seen = RT * 32 <= R ? (t_off + 1) / 32 : 0;
        const int last = tile1 - 1 - wave_u;             // the keys read last by pass 1 are read first here
        float before = 0.f;                              // a tile's sums are stored ahead of the next request, which the wait is for
        int first = last;                                // (unknown to the compiler, which peels the first round off and doubles the code)
        asm("" : "+s"(first));
        if (last >= tile0) tiles.request(last);
        for (int tile = last; tile >= tile0; tile -= NW) {
            Vec16 kv[NV];
            tiles.receive(kv);
            if (tile != first) put((tile + NW) * 32 + l32, before);
            if (tile - NW >= tile0) tiles.request(tile - NW);
            auto keep = [&](int, float colsum) { before = colsum; };
            if (tile < seen) colsum_tile(std::true_type(), tile, kv, keep);
            else colsum_tile(std::false_type(), tile, kv, keep);
        }
        if (last >= tile0) put((tile0 + (last - tile0) % NW) * 32 + l32, before);
    } else {
        auto colsum_tile = [&](int tile, const Vec16(&kv)[NV]) {
            const int key = tile * 32 + l32;
            const float colsum = tile_colsum<T, RT, WR, NV>(qv, kv, s_M, s_invL, hb, key, R, t_off, a.scale_log2e, Rp, cap, s);
            if (!WR && hb == 0 && key < s) Sp[key] = colsum;
        };
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
    if (!WR)
        for (int j = z0 + tid; j < col1; j += NT) Sp[j] = 0.f;
    if (Rp)
        for (int r = 0; r < R; ++r)
            for (int j = z0 + tid; j < col1; j += NT) Rp[(int64_t)r * cap + j] = 0.f;
}

// Slices per pair for the column sums.  One workgroup per pair reads its keys twice at about 30 GB/s, and with few
// pairs most of the chip waits for it.  The statistics of 32 rows are four chains of key tiles, one wave each, merged in a fixed
// order (the selection that follows can hang on the sum's last bit): in one workgroup, or in four whose sums
// the column sums' launch merges.  The column sums are independent and get one workgroup per CU in all, over the columns up to the
// bound on the lengths (the last slice has the rest).  Every slice holds the row statistics and is about 256 keys long at least.
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
// one workgroup per 32 rows of a pair or four: two launches pay while those find a CU of their own and the keys
// are long enough for the second launch.  One / two launches in us, f16, d = 128, R = 64 (the ring's rows, d = 64
// and fp32 draw the line in the same places; in parentheses two launches with the statistics in the operands' own layout,
// one workgroup per 32 rows):
//     8 pairs   1024 keys 21 / 16, 2048 36 / 20, 4096 65 / 27, 8192 124 / 43
//    32 pairs    512 keys 14 / 14, 1024 21 / 16 (19), 2048 36 / 21 (28), 4096 66 / 29 (45), 8192 128 / 47 (79)
//    64 pairs    512 keys 14 / 14, 1024 21 / 17 (21), 2048 36 / 22 (31), 4096 67 / 34, 8192 129 / 58 (89)
//   128 pairs   1024 keys 22 / 22 (24), 2048 37 / 31 (38), 4096 68 / 49 (67), 8192 135 / 86 (125)
//   160 pairs   1024 keys 22 / 33, 4096 69 / 81, 8192 141 / 153
// R = 128, 64 pairs x 1024 keys 36 / 21; R = 16, fp32, d = 128, 12 pairs x 1024 keys 43 / 36.
// With 65 to 128 pairs only under a stated bound: without one the slices are laid over the whole capacity, and prompts that fill
// a quarter of it gain little (128 pairs x 4096 keys in 16384 slots 71 / 67); and from 4096 keys on, where the gain is
// more than a few microseconds.  Up to 64 pairs short prompts under a long bound lose 1 to 4 us (32 pairs x 32 keys 7 / 9).
bool seed_in_two(int64_t pairs, int bound, bool stated, int R)
{
    if (pairs <= 64) return bound >= 1024;
    return stated && pairs <= 128 && pairs * ((R + 31) / 32) <= 256 && bound >= 4096;
}

// Does every chain of the statistics get a workgroup of its own?  Where a slice has the room to bring all of them along.
bool seed_chains_apart(int G, int cols, int cap, int R)
{
    const int room = 2 * kChains * R;
    return cols >= room && (int64_t)(G - 1) * cols + room <= cap;
}

template <typename T, int D, int RT, bool WR>
static int launch_prefill_rt(PrefillArgs a, int64_t pairs, bool stats_ready, hipStream_t stream)
{
    const int G = seed_slices(pairs, a.bound, a.cap, a.R, a.cols);
    a.G = G;
    // Keys that the launch before has read are still in the 256 MB Infinity Cache where there are few; loads that pass it by are
    // faster where there are many: plain / streaming, us, attention and sums, R = 64, 1792 x 4096 bf16 7608 / 7555, 2048 x 1001 f16 899 / 881, 2048 x 513
    // 357 / 343, 2048 x 300 185 / 184; 128 x 1001 58.1 / 59.2, 128 x 300 19.3 / 20.1; seed in two launches, 32 x 8192 47.7 / 54.0.
    const bool far = pairs * a.bound * (D * Elem<T>::kBytes) > (128ll << 20);
    const dim3 one((unsigned)pairs), all((unsigned)(pairs * G));
    auto sums = [&]() {
        if constexpr (kSeedByLds<T, RT, WR, kSeedSums>) {
            if (far) {
                launch_kernel((swa_prefill_kernel<T, D, RT, WR, kSeedSumsFar>), all, dim3(256), 0, stream, a);
                return;
            }
        }
        launch_kernel((swa_prefill_kernel<T, D, RT, WR, kSeedSums>), all, dim3(256), 0, stream, a);
    };
    if (stats_ready) {
        sums();
    } else if (G > 1 && seed_in_two(pairs, a.bound, a.stated, a.R)) {
        if constexpr (D * Elem<T>::kBytes >= 512) {
            launch_kernel((swa_prefill_kernel<T, D, 1, WR, kSeedStats>), dim3((unsigned)(pairs * RT)), dim3(256), 0, stream, a);
        } else if (seed_chains_apart(G, a.cols, a.cap, a.R)) {
            a.chains = kChains;
            launch_kernel((swa_seed_stats_kernel<T, D, WR, 1>), dim3((unsigned)(pairs * RT * kChains)), dim3(kWave), 0, stream, a);
        } else {
            launch_kernel((swa_seed_stats_kernel<T, D, WR, kChains>), dim3((unsigned)(pairs * RT)), dim3(kChains * kWave), 0, stream, a);
        }
        if (hipGetLastError() != hipSuccess) return SWA_ERR_HIP;
        sums();
    } else {
        launch_kernel((swa_prefill_kernel<T, D, RT, WR, kSeedWhole>), one, dim3(256), 0, stream, a);
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
    a.G = a.cols = 0;
    a.chains = 1;
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
