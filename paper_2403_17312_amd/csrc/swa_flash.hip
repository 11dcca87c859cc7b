// Prefill attention on MFMA: Eq. 1-2 over the whole prompt with the causal mask,
//   out[t] = sum_{j<=t} softmax_{j<=t}(q_t . k_j * scale) v_j      for every prompt position t.
// One workgroup (4 waves) per (pair, block of 128 queries); a wave owns 32 queries.  The
// attention-weight matrix is never stored: key tiles of 32 stream through LDS and every wave keeps
// flash-style running (max, sum, output) state for its queries.
//
// Both contractions are arranged so that a lane owns ONE query throughout:
//   S^T = K Q^T     A = key tile (LDS, row-major), B = query fragments (registers)
//                   -> lane l holds, for query l%32, the logits of 16 of the tile's keys;
//   O^T = V^T P^T   A = value tile, transposed, B = the lane's own 16 weights, packed
//                   -> lane l holds, for query l%32, 16 channels of every 32-channel tile.
// So the row statistics, the rescaling of the running output and the weights that feed the
// second product never leave the lane (one exchange with the other half-wave for the maximum).
// The 16 keys a lane holds are keys 8*(i/4) + 4*(l/32) + (i%4) of the tile; the value fragments are
// read in that order, so the contraction pairs every weight with its own key.
//
// Two kernels: one for the 16-bit formats, and one for short prompts and for fp32 (which is there for completeness).
#include <type_traits>

#include "swa_kernels.hpp"

namespace swa {

struct FlashArgs {
    const char* q;
    const char* k;
    const char* v;
    char* out;
    const int32_t* cache_len;
    int32_t h, cap;
    int32_t pairs, nqb;    // (sequence, head) pairs and query blocks per pair in the grid
    int32_t front;         // query blocks are laid from the prompt's start (else from its end)
    int32_t per_xcd, tail; // pairs per XCD, and how many of them (the last ones) are dealt out block by block
    float scale_log2e;
    float* stat;           // [pairs, cap]: statistics of the last R rows, stat_G copies stat_cols apart, or NULL
    int32_t R, stat_G, stat_cols;
};

constexpr int kXcds = 8;   // workgroups are dealt round-robin to the 8 XCDs, each with its own L2

// Where the reference maximum of a row's running sum starts.  Finite, so that keys whose logit is -inf weigh nothing
// (exp2(-inf - reference) = 0) also when they come before the row's first finite logit.
constexpr float kNoReference = -3.0e38f;

constexpr int BQ = 128;             // queries per workgroup

// Which queries a workgroup serves: BQ of them from q0 on, of a prompt of s rows.  False: none.
//
// XCD-aware placement: the query blocks of one pair all read the same K and V, so they go to the same XCD, next to each other
// in launch order, and share the pair's rows through that XCD's L2; the XCDs work on different pairs.  Longest blocks of
// a pair first.  The last pairs of an XCD (a.tail of them, about 128 blocks, a little more than run at once, in the 16-bit formats) are
// dealt out block by block instead: their longest blocks start together and the short ones fill in behind, where pair by
// pair the last pair's longest block would run on alone.  32 pairs x 4096 rows, f16, d = 128: 177 -> 153 us; 128 of 300..1200
// 48 -> 42; dealt out like that as a whole, large batches lose what the L2 gave them (2048 of 512..2048: 1253 -> 1919).
// fp32 is bound by its products and gains from more of it: 512 blocks.  Pair by pair from the start / 128 / 512, us, d = 64: 2048
// pairs x 129 134 / 144 / 99, x 161 164 / 177 / 131, x 420 755 / 816 / 685, 256 x 2048 1421 / 1267 / 1178.
// The blocks are laid from the prompt's end (to a multiple of 32, so that a wave's queries meet one diagonal tile): what is
// left over is the first block, which has the fewest keys, and its idle waves cost least.  2048 pairs of 512..2048 rows 1253 -> 1196 us.
// While every block has a CU of its own (a.front) the longest one decides, and what is left over is better there, as its last block,
// whose few waves run alone: from the end / from the start, us, 32 pairs x 161 rows, f16, d = 128 9.2 / 8.2, bf16, d = 64 7.0 / 6.2, fp32, d
// = 64 17.8 / 16.7; 32 x 700 18.0 / 17.0, 13.6 / 12.4, 54.3 / 52.5; one block more than CUs and it is the other way round (64 x 513, f16,
// d = 128 15.8 / 18.9).
__device__ __forceinline__ bool query_block(const FlashArgs& a, int64_t& pair, int& s, int& q0)
{
    const int idx = blockIdx.x / kXcds;
    const int head = a.per_xcd - a.tail;
    int at, qb;
    if (idx < head * a.nqb) {
        at = idx / a.nqb;
        qb = a.nqb - 1 - (idx - at * a.nqb);
    } else {
        const int r = idx - head * a.nqb;
        qb = a.nqb - 1 - r / a.tail;
        at = head + r % a.tail;
    }
    pair = blockIdx.x % kXcds + (int64_t)kXcds * at;
    if (pair >= a.pairs) return false;
    s = a.cache_len[(uint32_t)pair / (uint32_t)a.h];
    s = s > a.cap ? a.cap : s;
    if (a.front) {
        q0 = qb * BQ;
        return q0 < s;
    }
    int q_end = (s + 31) & ~31;
    q_end = q_end < a.nqb * BQ ? q_end : a.nqb * BQ;     // (a prompt beyond the stated bound: its rows up to the bound)
    const int blocks = (q_end + BQ - 1) / BQ;
    q0 = q_end - (blocks - qb) * BQ;                     // (negative in a first block that is not full)
    return qb < blocks;
}

// Half-precision element e (0..7) of a 16-byte vector, in the low 16 bits.
__device__ __forceinline__ uint32_t half_of(const Vec16& v, int e)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    return (w[e >> 1] >> ((e & 1) * 16)) & 0xffffu;
}

// x of lane (l % 32) and x of lane (l % 32) + 32, in every lane: v_permlane32_swap exchanges the
// upper half of one register with the lower half of another, so two copies of x come back as
// (the lower half's x, the upper half's x) - no trip through LDS.
__device__ __forceinline__ void both_halves(float x, float& lo, float& hi)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    lo = __uint_as_float(r[0]);
    hi = __uint_as_float(r[1]);
}

// Two fp32 values rounded to T, packed into one dword.
template <typename T>
__device__ __forceinline__ uint32_t pack2(float f0, float f1);
template <>
__device__ __forceinline__ uint32_t pack2<F16>(float f0, float f1)
{
    return f32x2_to_f16x2_bits(f0, f1);
}
template <>
__device__ __forceinline__ uint32_t pack2<BF16>(float f0, float f1)
{
    return f32x2_to_bf16x2_bits(f0, f1);
}

// The 16 weights of one lane's query and key tile, exp2(c scale - m), their sum, and the rescaling that goes with them.
//
// The reference m only has to bound the exponents, not equal the maximum (out = o / l whatever it is).  So the weights are
// formed with the reference as it is, and only where a lane's sum shows that it is too low (a sum above 2^12, so some weight
// above 2^8, or not finite, as on the first tile) is the tile's maximum looked for, the running output o and sum l rescaled
// and the weights formed again: a few times per query.  With the maximum looked for on every tile, and fp16 weights rounded one
// by one: 1792 pairs x 4096, bf16 6.96 -> 6.82 ms; 2048 of 512..2048, f16 1179 -> 1139 us, d = 64 695 -> 628.
// A single weight may reach 2^12 that way, which fp16 holds and fp32 sums.
constexpr float kSlack = 8.f;           // how far (powers of two) all 16 logits may exceed the reference
constexpr float kTooMuch = 4096.f;      // sum of a lane's 16 weights beyond which one of them must exceed 2^kSlack
template <int CT>
__device__ __forceinline__ float tile_weights(const float16_t& c, float scale_log2e, float& m, float& l, float16_t (&o)[CT], float (&p)[16])
{
    float ps;
    auto weights = [&]() __attribute__((always_inline)) {
        ps = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(c[i], scale_log2e, -m));   // 0 for masked keys
            ps += p[i];
        }
    };
    weights();
    if (__any(ps > kTooMuch)) {
        float mx = c[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, c[i]);
        float mx_lo, mx_hi;
        both_halves(mx, mx_lo, mx_hi);
        mx = fmaxf(mx_lo, mx_hi) * scale_log2e;       // scale > 0: max commutes
        const float m_new = (mx > m + kSlack) ? mx : m;
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);     // 0 on the first tile
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[ct][i] *= alpha;
        weights();
    }
    return ps;
}

// Tiles staged through registers, double-buffered, the value tile transposed on its way into LDS: short prompts in
// the 16-bit formats (three workgroups per CU, 168 registers per lane, 38 KB of LDS each), and fp32.  fp32 (32x32x2
// MFMA, four issues per 16-byte fragment) is there for completeness, not speed: two waves per SIMD, and at d = 128 a
// single LDS buffer.
template <typename T, int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Elem<T>::kBytes == 2 ? 3 : 2)))
swa_flash_prefill_kernel(FlashArgs a)
{
    constexpr int NT = 256;
    constexpr int EB = Elem<T>::kBytes;     // 2 or 4
    constexpr int EPV = Elem<T>::kPerVec;   // elements per 16-byte fragment: 8 or 4
    constexpr int NP = 16 / EPV;            // fragments that hold a lane's 16 weights
    constexpr int ROWB = D * EB;
    constexpr int NV = ROWB / 32;       // 16-byte vectors a lane supplies for a 32-row operand
    constexpr int CT = D / 32;          // 32-channel tiles of the output
    constexpr int BK = 32;              // keys per tile
    constexpr int KSTR = ROWB + 16;     // LDS row of the key tile, padded against bank conflicts
    constexpr int VSTR = BK * EB + 16;  // LDS row (one channel, 32 keys) of the transposed value tile
    constexpr int CPR = ROWB / 16;      // 16-byte chunks per cache row
    constexpr int LD = BK * CPR / NT;   // chunks per thread, per tensor and tile
    constexpr bool kPaired = EB == 2 && LD == 2;
    constexpr int PF = 3;               // LDS fragment reads in flight ahead of the product that uses them
    constexpr int NBUF = (EB == 4 && D == 128) ? 1 : 2;   // LDS buffers (64 KB of static LDS at most)
    static_assert(LD >= 1 && BK * CPR % NT == 0, "tile must split evenly over the workgroup");

    __shared__ __align__(16) char s_k[NBUF][BK * KSTR];
    // Channel c's row of the transposed value tile starts at vt_row(c): 80 bytes per row keep the
    // 16-byte fragment reads of 16 consecutive channels on disjoint banks, and every group of 16
    // channels is skewed by another 16 bytes so that the transposing stores (16 lanes, channels 8
    // apart) spread over the banks as well.
    constexpr int VT_BYTES = D * VSTR + (D / 16) * 16;
    __shared__ __align__(16) char s_vt[NBUF][VT_BYTES];
    auto vt_row = [](int c) { return c * VSTR + (c >> 4) * 16; };

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int l32 = lane & 31;
    const int hb = lane >> 5;
    int64_t pair;
    int s, q0;
    if (!query_block(a, pair, s, q0)) return;

    const char* Qp = a.q + pair * (int64_t)a.cap * ROWB;
    const char* Kp = a.k + pair * (int64_t)a.cap * ROWB;
    const char* Vp = a.v + pair * (int64_t)a.cap * ROWB;
    char* Op = a.out + pair * (int64_t)a.cap * ROWB;

    const int t = q0 + wave * 32 + l32;          // this lane's query position
    const int tq = t < 0 ? 0 : (t < s ? t : s - 1);      // lanes outside the prompt shadow a query of it
    Vec16 qv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) qv[v] = load16(Qp + (int64_t)tq * ROWB + v * 32 + hb * 16);

    const int q_hi = (q0 + BQ < s ? q0 + BQ : s) - 1;    // last query of the workgroup
    const int nkt = q_hi / BK + 1;                        // key tiles 0..nkt-1 cover keys 0..q_hi
    const int w_lo = q0 + wave * 32;
    const int w_hi = (w_lo + 31 < s - 1) ? w_lo + 31 : s - 1;
    const int my_last = (w_lo >= 0 && w_lo < s) ? w_hi / BK : -1;      // last tile with a visible key for this wave

    // Which tile rows a thread stages.  With two chunks per thread (d = 128) they are an even key
    // and its successor, which sit next to each other in a lane's key order, so their values are
    // stored to the transposed tile as one dword; the four (even key) slots of a wave are chosen
    // so that, with the 16 channel groups, its 64 stores hit 64 different banks.
    auto tile_key = [&](int x) {
        if constexpr (kPaired) {
            const int q = tid / CPR;                 // 0..15
            const int pr = (q & 1) + 4 * ((q >> 1) & 1) + 2 * ((q >> 2) & 1) + 8 * (q >> 3);
            return 2 * pr + x;
        } else {
            return (tid + x * NT) / CPR;
        }
    };
    Vec16 gk[LD], gv[LD];
    auto gload = [&](int kt) {
#pragma unroll
        for (int x = 0; x < LD; ++x) {
            const int j = tile_key(x), cc = tid % CPR;
            int row = kt * BK + j;
            row = row < s ? row : s - 1;          // rows past the prompt are masked; keep them finite
            // uniform base + 32-bit offset (cap <= SWA_MAX_CAP keeps a pair's rows within 8 MiB)
            const uint32_t off = (uint32_t)row * ROWB + cc * 16;
            gk[x] = load16(Kp + off);
            gv[x] = load16(Vp + off);
        }
    };
    // key j is element i16 of half-wave hbk's 16 keys: its place (in elements) in a channel's
    // row.  16-bit: fragment v of half-wave hbk holds i16 = 8v..8v+7; fp32 fragments hold four
    // consecutive keys, so there the natural order is already the lanes' order.
    auto key_slot = [](int j) {
        if constexpr (EB == 4) return j;
        const int i16 = 4 * (j / 8) + (j % 4);
        const int hbk = (j / 4) % 2;
        return ((i16 / 8) * 2 + hbk) * 8 + (i16 % 8);
    };
    auto lstore = [&](int buf) {
        const int cc = tid % CPR;
#pragma unroll
        for (int x = 0; x < LD; ++x) store16(s_k[buf] + tile_key(x) * KSTR + cc * 16, gk[x]);
        if constexpr (kPaired) {
            const int posk = key_slot(tile_key(0));      // even, and key_slot(tile_key(1)) == posk + 1
            const uint32_t w0[4] = {gv[0].x, gv[0].y, gv[0].z, gv[0].w}, w1[4] = {gv[1].x, gv[1].y, gv[1].z, gv[1].w};
#pragma unroll
            for (int e = 0; e < 8; ++e)      // channel e of the even key below, of its successor above: one byte permute
                *reinterpret_cast<uint32_t*>(s_vt[buf] + vt_row(cc * 8 + e) + posk * 2) =
                    __builtin_amdgcn_perm(w1[e >> 1], w0[e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
        } else if constexpr (EB == 2) {
#pragma unroll
            for (int x = 0; x < LD; ++x) {
                const int posk = key_slot(tile_key(x));
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    *reinterpret_cast<uint16_t*>(s_vt[buf] + vt_row(cc * 8 + e) + posk * 2) = (uint16_t)half_of(gv[x], e);
            }
        } else {
#pragma unroll
            for (int x = 0; x < LD; ++x) {
                const int posk = key_slot(tile_key(x));
                const uint32_t w[4] = {gv[x].x, gv[x].y, gv[x].z, gv[x].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<uint32_t*>(s_vt[buf] + vt_row(cc * 4 + e) + posk * 4) = w[e];
            }
        }
    };

    float16_t o[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ct][i] = 0.f;
    float m = kNoReference, l = 0.f;

    gload(0);
    lstore(0);
    // Every load issued so far (the query fragments among them) is waited for HERE, once: the
    // memory counter is in-order, so a query fragment still in flight at the loop's entry would
    // make the compiler wait, inside every iteration's first product, for counts that on all
    // later iterations mean "the tile just requested has arrived" - the prefetch would be lost.
    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
    __syncthreads();
    for (int kt = 0; kt < nkt; ++kt) {
        const int buf = kt % NBUF;
        if (kt + 1 < nkt) gload(kt + 1);
        if (kt <= my_last) {
            float16_t c;
#pragma unroll
            for (int i = 0; i < 16; ++i) c[i] = 0.f;
            const char* kb = s_k[buf] + l32 * KSTR + hb * 16;
            // key fragments are read from LDS PF products ahead of their use, in this order
            Vec16 kf[NV];
#pragma unroll
            for (int v = 0; v < PF && v < NV; ++v) kf[v] = load16(kb + v * 32);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                if (v + PF < NV) kf[v + PF] = load16(kb + (v + PF) * 32);
                __builtin_amdgcn_sched_barrier(0);
                c = Mfma<T>::run(kf[v], qv[v], c);   // C[key][query]
                __builtin_amdgcn_sched_barrier(0);
            }
            // only the tiles that reach the wave's diagonal need the causal mask
            if (kt * BK + BK - 1 > w_lo) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = kt * BK + 8 * (i / 4) + 4 * hb + (i % 4);
                    c[i] = (key <= tq) ? c[i] : -INFINITY;
                }
            }
            float p[16];
            const float ps = tile_weights(c, a.scale_log2e, m, l, o, p);
            l += ps;
            Vec16 pv[NP];
#pragma unroll
            for (int v = 0; v < NP; ++v) pv[v] = pack<T>(p + v * EPV);
            // value fragments likewise: fragment f = ct * NP + v, read PF products ahead
            Vec16 vf[CT * NP];
            // vt_row(32 ct + l32) = vt_row(l32) + ct (32 VSTR + 32): one lane address, constant offsets
            const char* vb0 = s_vt[buf] + vt_row(l32) + hb * 16;
            // product f works on channel tile f % CT with weight fragment f / CT: consecutive products
            // accumulate into different tiles, so none waits for the one before it
            auto vfrag = [&](int f) { return load16(vb0 + (f % CT) * (32 * VSTR + 32) + (f / CT) * 32); };
#pragma unroll
            for (int f = 0; f < PF && f < CT * NP; ++f) vf[f] = vfrag(f);
#pragma unroll
            for (int f = 0; f < CT * NP; ++f) {
                if (f + PF < CT * NP) vf[f + PF] = vfrag(f + PF);
                __builtin_amdgcn_sched_barrier(0);
                o[f % CT] = Mfma<T>::run(vf[f], pv[f / CT], o[f % CT]);   // C[channel][query]
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (NBUF == 1) __syncthreads();      // every wave is done with the only buffer
        if (kt + 1 < nkt) lstore((kt + 1) % NBUF);
        __syncthreads();
    }

    float l_lo, l_hi;
    both_halves(l, l_lo, l_hi);
    l = l_lo + l_hi;
    // the seed's column sums need these rows' statistics: handing them over saves it one of two reads of the keys
    const int r = t - (s - a.R);
    if (a.stat && hb == 0 && t >= 0 && t < s && r >= 0) {
        float* St = a.stat + pair * (int64_t)a.cap;
        for (int g = 0; g < a.stat_G; ++g) {
            St[g * a.stat_cols + r] = m;
            St[g * a.stat_cols + a.R + r] = l;
        }
    }
    if (t >= 0 && t < s) {
        const float inv = 1.f / l;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // channels 32 ct + 8 g + 4 hb + 0..3 of query t
                char* dst = Op + (int64_t)t * ROWB + (32 * ct + 8 * g + 4 * hb) * EB;
                if constexpr (EB == 4) {
                    float f[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) f[r] = o[ct][4 * g + r] * inv;
                    store16(dst, pack<F32>(f));
                } else {
                    uint32_t w[2];
#pragma unroll
                    for (int r = 0; r < 2; ++r)
                        w[r] = pack2<T>(o[ct][4 * g + 2 * r] * inv, o[ct][4 * g + 2 * r + 1] * inv);
                    *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
                }
            }
        }
    }
}

// Two transposing LDS reads as one 16-byte fragment.  ds_read_b64_tr_b16, within 16 lanes: lane j supplies the
// address of row j/4, columns 4 (j%4) .. +3 of a 4x16 block and receives column j of its four rows.
typedef short short4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Vec16 lds_read_tr(const char* lo, const char* hi)
{
    typedef __attribute__((address_space(3))) short4_t* ptr_t;
    const uint2 x = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr_t)lo));
    const uint2 y = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr_t)hi));
    return Vec16{x.x, x.y, y.x, y.y};
}

// 16-bit formats, prompts of more than 256 rows.  Bound: the matrix cores at the clock the power limit leaves them
// (1.65-1.8 GHz under this kernel; busy 60 % of the cycles), next to as many clocks of vector work for the
// softmax.  What it took there, on 1792 pairs of 4096 rows, bf16, d = 128 (before: 8.3-8.4 ms, busy 51 %):
//   - Key and value tiles go from L2 straight to LDS (global_load_lds, 16 bytes per lane), with no registers in
//     between and no LDS store instructions.  Such a load writes 64 consecutive 16-byte chunks, so rows cannot
//     be padded; instead chunk c of row r holds the row's chunk c ^ swizzle(r), chosen by the lane's GLOBAL
//     address, and the readers apply the same permutation.  The value tile stays row-major:
//     ds_read_b64_tr_b16 hands a lane four consecutive keys of its channel, half of the fragment the
//     second product wants.  8.0 ms.
//   - Three buffers, two tiles ahead: 7.5 ms.
//   - The loads of a tile are issued between the products of another instead of all at once: 7.1 ms.
// Three waves per SIMD (168 registers, 48 KB of LDS per workgroup) at d = 128, four at d = 64.
template <typename T, int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 3)))
swa_flash16_kernel(FlashArgs a)
{
    constexpr int NW = 4;
    constexpr int ROWB = D * 2;
    constexpr int NV = ROWB / 32;       // 16-byte fragments a lane supplies for a 32-row operand
    constexpr int CT = D / 32;          // 32-channel tiles of the output
    constexpr int BK = 32;              // keys per tile
    constexpr int TILE = BK * ROWB;
    constexpr int CPR = ROWB / 16;      // 16-byte chunks per cache row
    constexpr int RPI = kWave / CPR;    // rows that one wave-wide load covers
    constexpr int LD = BK / RPI / NW;   // such loads per wave, per tensor and tile
    static_assert(2 * LD == NV / 2, "one of them behind every second product of the first contraction");
    constexpr int PF = 2;               // LDS fragment reads in flight ahead of the product that uses them

    // three buffers for a key and a value tile
    __shared__ __align__(1024) char s_k0[TILE], s_k1[TILE], s_v0[TILE], s_v1[TILE], s_k2[TILE], s_v2[TILE];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31;
    const int hb = lane >> 5;
    int64_t pair;
    int s, q0;
    if (!query_block(a, pair, s, q0)) return;

    const char* Qp = a.q + pair * (int64_t)a.cap * ROWB;
    const char* Kp = a.k + pair * (int64_t)a.cap * ROWB;
    const char* Vp = a.v + pair * (int64_t)a.cap * ROWB;
    char* Op = a.out + pair * (int64_t)a.cap * ROWB;

    const int t = q0 + wave * 32 + l32;          // this lane's query position
    const int tq = t < 0 ? 0 : (t < s ? t : s - 1);      // lanes outside the prompt shadow a query of it

    const int q_hi = (q0 + BQ < s ? q0 + BQ : s) - 1;    // last query of the workgroup
    const int nkt = q_hi / BK + 1;                        // key tiles 0..nkt-1 cover keys 0..q_hi
    const int w_lo = q0 + wave * 32;
    const int w_hi = (w_lo + 31 < s - 1) ? w_lo + 31 : s - 1;
    const int my_last = (w_lo >= 0 && w_lo < s) ? w_hi / BK : -1;      // last tile with a visible key for this wave

    // Load x of this wave covers tile rows (wave * LD + x) * RPI + lane / CPR; the lane's chunk of the LDS
    // row is lane % CPR.  The LDS serves 256 bytes a clock: 16 lanes of a fragment read (16 neighbouring rows
    // of the key tile), 32 lanes of a transposing read (4 rows, 64 bytes of each).  The swizzles put what
    // one clock serves on different banks (a row of 128 channels is as long as the banks are wide, of 64
    // channels half as long); with only 8 rows told apart the reads measured half as fast.
    auto swzK = [](int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
    auto swzV = [](int r) { return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); };
    uint32_t offK[LD], offV[LD];
    auto offsets = [&](int last) {     // rows past tile row `last` re-read that one (finite values, masked later)
        int ln = lane;
        asm volatile("" : "+v"(ln));   // computed where it is needed (twice), not kept in registers around the loop
        const int ldr = ln / CPR, ldc = ln % CPR;
#pragma unroll
        for (int x = 0; x < LD; ++x) {
            const int j = (wave * LD + x) * RPI + ldr;
            const int r = j < last ? j : last;
            offK[x] = (uint32_t)r * ROWB + (uint32_t)((ldc ^ swzK(j)) * 16);
            offV[x] = (uint32_t)r * ROWB + (uint32_t)((ldc ^ swzV(j)) * 16);
        }
    };
    // Load x = 0 .. 2 LD - 1 of the staging of tile kt (uniform base; cap <= SWA_MAX_CAP: below 8 MiB).  Before the
    // prompt's last tile, which no full one follows, edge() aims the lanes at rows that exist.
    auto edge = [&](int kt) {
        if (kt * BK + BK > s) offsets(s - 1 - kt * BK);
    };
    auto load = [&](int x, int kt, char* dk, char* dv) {
        const uint32_t at = (uint32_t)kt * (BK * ROWB);
        if (x < LD) load_to_lds(Kp + at, offK[x], lds_address(dk) + (wave * LD + x) * 1024);
        else load_to_lds(Vp + at, offV[x - LD], lds_address(dv) + (wave * LD + x - LD) * 1024);
    };
    auto stage = [&](int kt, char* dk, char* dv) {
        edge(kt);
#pragma unroll
        for (int x = 0; x < 2 * LD; ++x) load(x, kt, dk, dv);
    };
    offsets(BK);

    stage(0, s_k0, s_v0);
    Vec16 qv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) qv[v] = load16(Qp + (int64_t)tq * ROWB + v * 32 + hb * 16);

    // Fragment addresses.  Key fragment v: row l32, chunk 2v + hb.  Value fragment (ct, v): keys
    // 16v + 4hb + 0..3 and 16v + 8 + 4hb + 0..3 of channel 32 ct + l32, one transposing read each: within
    // 16 lanes, lane j supplies the address of key j/4, channels 4 (j%4) .. +3, and receives channel j.
    const uint32_t ka = (uint32_t)(l32 * ROWB + ((hb ^ swzK(l32)) << 4));
    const int j16 = lane & 15;
    const uint32_t va = (uint32_t)((4 * hb + (j16 >> 2)) * ROWB +
                                   (((2 * ((lane >> 4) & 1) + ((j16 & 3) >> 1)) ^ swzV(j16 >> 2)) << 4) + (j16 & 1) * 8);

    // The query fragments are waited for here, where the compiler sees it: it would otherwise wait for them at
    // their first use in every round of the loop, and with them for the tiles requested since.
    __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
    if (nkt > 1) stage(1, s_k1, s_v1);

    float16_t o[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ct][i] = 0.f;
    float m = kNoReference, l = 0.f;

    // all: two more tiles are to come for certain
    auto compute = [&](auto all, int kt, const char* sk, const char* sv, char* nk, char* nv) __attribute__((always_inline)) {
        const int st = kt + 2;
        const bool more = all.value || st < nkt;
        if (more) edge(st);
        float16_t c;
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = 0.f;
        // key fragments are read from LDS PF products ahead of their use, in this order
        auto kfrag = [&](int v) { return load16(sk + (ka ^ (v << 5))); };
        Vec16 kf[NV];
#pragma unroll
        for (int v = 0; v < PF && v < NV; ++v) kf[v] = kfrag(v);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (v + PF < NV) kf[v + PF] = kfrag(v + PF);
            __builtin_amdgcn_sched_barrier(0);
            c = Mfma<T>::run(kf[v], qv[v], c);   // C[key][query]
            __builtin_amdgcn_sched_barrier(0);
            // the loads of a later tile are issued between the products, which hide the time they wait to be
            // accepted: the four waves' sixteen 1 KiB loads together keep the CU's 64-byte path busy for 256 clocks
            if ((v & 1) && more) load(v >> 1, st, nk, nv);
        }
        // only the tiles that reach the wave's diagonal need the causal mask
        if (kt * BK + BK - 1 > w_lo) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int key = kt * BK + 8 * (i / 4) + 4 * hb + (i % 4);
                c[i] = (key <= tq) ? c[i] : -INFINITY;
            }
        }
        float p[16];
        const float ps = tile_weights(c, a.scale_log2e, m, l, o, p);
        l += ps;
        Vec16 pv[2];
        pv[0] = pack<T>(p);
        pv[1] = pack<T>(p + 8);
        // value fragments likewise; product f works on channel tile f % CT with weight fragment f / CT, so that
        // consecutive products accumulate into different tiles
        auto vfrag = [&](int f) {
            const int ct = f % CT, v = f / CT;
            const char* at = sv + ((va ^ (ct << 6)) + v * 16 * ROWB);
            return lds_read_tr(at, at + 8 * ROWB);
        };
        Vec16 vf[2 * CT];
#pragma unroll
        for (int f = 0; f < PF && f < 2 * CT; ++f) vf[f] = vfrag(f);
#pragma unroll
        for (int f = 0; f < 2 * CT; ++f) {
            if (f + PF < 2 * CT) vf[f + PF] = vfrag(f + PF);
            __builtin_amdgcn_sched_barrier(0);
            o[f % CT] = Mfma<T>::run(vf[f], pv[f / CT], o[f % CT]);   // C[channel][query]
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Tile kt is read while kt+1 and kt+2 are on their way (three buffers).  Loads return in order, so "all but
    // the newest tile's" is a count; behind the last tile nothing is requested, and the count is zero.  Every read of
    // the buffer that is about to be refilled has returned when its wave arrives at the barrier.
    auto ready = [&](bool newer) {
        if (newer) __builtin_amdgcn_s_waitcnt(0x0070 | (2 * LD));      // vmcnt(2 LD) lgkmcnt(0)
        else __builtin_amdgcn_s_waitcnt(0x0070);                       // vmcnt(0) lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto tile = [&](auto all, int kt, const char* sk, const char* sv, char* nk, char* nv) __attribute__((always_inline)) {
        ready(all.value || kt + 1 < nkt);
        compute(all, kt, sk, sv, nk, nv);
    };
    // The last tiles of a query block ask whether there is one more to request (asking in every round cost 2 to 9 % on
    // prompts of 1000 and more rows).
    int kt = 0;
    for (; kt + 2 <= my_last && kt + 4 < nkt; kt += 3) {
        tile(std::true_type(), kt, s_k0, s_v0, s_k2, s_v2);
        tile(std::true_type(), kt + 1, s_k1, s_v1, s_k0, s_v0);
        tile(std::true_type(), kt + 2, s_k2, s_v2, s_k1, s_v1);
    }
    // at most four are left: kt + 4 >= nkt, or kt + 2 > my_last
    if (kt <= my_last) tile(std::false_type(), kt, s_k0, s_v0, s_k2, s_v2);
    if (kt + 1 <= my_last) tile(std::false_type(), kt + 1, s_k1, s_v1, s_k0, s_v0);
    if (kt + 2 <= my_last) tile(std::false_type(), kt + 2, s_k2, s_v2, s_k1, s_v1);
    if (kt + 3 <= my_last) tile(std::false_type(), kt + 3, s_k0, s_v0, s_k2, s_v2);
    // the tiles behind this wave's last query: it still takes its part in staging them for the others
    for (kt = my_last + 1; kt < nkt; ++kt) {
        const int st = kt + 2;
        const int buf = kt % 3;
        ready(kt + 1 < nkt);
        if (st < nkt) {
            edge(st);
            stage(st, buf == 0 ? s_k2 : (buf == 1 ? s_k0 : s_k1), buf == 0 ? s_v2 : (buf == 1 ? s_v0 : s_v1));
        }
    }
    float l_lo, l_hi;
    both_halves(l, l_lo, l_hi);
    l = l_lo + l_hi;
    // the seed's column sums need these rows' statistics: handing them over saves it one of two reads of the keys
    const int r = t - (s - a.R);
    if (a.stat && hb == 0 && t >= 0 && t < s && r >= 0) {
        float* St = a.stat + pair * (int64_t)a.cap;
        for (int g = 0; g < a.stat_G; ++g) {
            St[g * a.stat_cols + r] = m;
            St[g * a.stat_cols + a.R + r] = l;
        }
    }
    if (t >= 0 && t < s) {
        const float inv = 1.f / l;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // channels 32 ct + 8 g + 4 hb + 0..3 of query t
                uint32_t w[2];
#pragma unroll
                for (int r = 0; r < 2; ++r) w[r] = pack2<T>(o[ct][4 * g + 2 * r] * inv, o[ct][4 * g + 2 * r + 1] * inv);
                *reinterpret_cast<uint2*>(Op + (int64_t)t * ROWB + (32 * ct + 8 * g + 4 * hb) * 2) = make_uint2(w[0], w[1]);
            }
        }
    }
}

// The grid for prompts of at most `bound` rows (false: more workgroups than a launch can have).
static bool flash_grid(FlashArgs& a, int bound, bool f32, int64_t& wgs)
{
    a.nqb = (bound + BQ - 1) / BQ;
    a.per_xcd = (a.pairs + kXcds - 1) / kXcds;
    a.tail = ((f32 ? 512 : 128) + a.nqb - 1) / a.nqb;
    if (a.tail > a.per_xcd) a.tail = a.per_xcd;
    a.front = (int64_t)a.pairs * a.nqb <= 256;
    wgs = (int64_t)a.per_xcd * kXcds * a.nqb;
    return wgs <= 0x7fffffffLL;
}

int launch_flash_prefill(const swa_params& p, float scale, const void* q, const void* k_cache, const void* v_cache,
                         const int32_t* cache_len, void* out, int32_t R, float* score, bool& stats_written,
                         hipStream_t stream)
{
    FlashArgs a;
    a.q = static_cast<const char*>(q);
    a.k = static_cast<const char*>(k_cache);
    a.v = static_cast<const char*>(v_cache);
    a.out = static_cast<char*>(out);
    a.cache_len = cache_len;
    a.h = p.h;
    a.cap = p.cap;
    a.scale_log2e = scale * 1.44269504088896340736f;
    const int bound = (p.len_bound > 0 && p.len_bound < p.cap) ? p.len_bound : p.cap;
    a.pairs = p.b * p.h;
    a.R = R;
    a.stat_G = a.stat_cols = 0;
    seed_stats_place(a.pairs, bound, p.cap, R, a.stat_G, a.stat_cols);
    a.stat = a.stat_G > 0 ? score : nullptr;
    stats_written = a.stat != nullptr;
    // The direct-to-LDS kernel has a longer start and end, which short prompts feel.  Staged through registers / direct in
    // us, f16 at d = 128, bf16 at d = 128, f16 at d = 64: 256 x 40 pairs of 32 rows 250 / 255, 232 / 242, 114 / 117; 256 x 32 of
    // 60..250 rows 523 / 535, 511 / 527, 281 / 286; 64 x 32 of 128..512 rows 167 / 160, 161 / 156, 95 / 87 (longer
    // ones: up to 1.25 times as fast).
    const bool direct = p.dtype != SWA_F32 && bound > 256;
    int64_t wgs = 0;
    if (!flash_grid(a, bound, p.dtype == SWA_F32, wgs)) return SWA_ERR_BAD_SHAPE;
    auto go = [&](auto small, auto large) {
        launch_kernel(p.d == 64 ? small : large, dim3((unsigned)wgs), dim3(256), 0, stream, a);
    };
    if (p.dtype == SWA_F32) go(swa_flash_prefill_kernel<F32, 64>, swa_flash_prefill_kernel<F32, 128>);
    else if (p.dtype == SWA_F16 && direct) go(swa_flash16_kernel<F16, 64>, swa_flash16_kernel<F16, 128>);
    else if (p.dtype == SWA_F16) go(swa_flash_prefill_kernel<F16, 64>, swa_flash_prefill_kernel<F16, 128>);
    else if (direct) go(swa_flash16_kernel<BF16, 64>, swa_flash16_kernel<BF16, 128>);
    else go(swa_flash_prefill_kernel<BF16, 64>, swa_flash_prefill_kernel<BF16, 128>);
    return hipGetLastError() == hipSuccess ? SWA_OK : SWA_ERR_HIP;
}

}  // namespace swa
