// What the decode kernels are handed: one launch of a step for every (sequence, head) pair.
#pragma once

#include "swa_kernels.hpp"

namespace swa {

constexpr float kMinKeptMass = 0.05f;      // below it the evicted rows are not subtracted: too little would be left

struct DecodeArgs {
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
    char* out;
    float* probs_dbg;
    int32_t* status;
    int32_t* arrive;
    int32_t h, cap, lds_slots, w, sparsity_bp;
    int32_t key_slots;    // selection keys in LDS: lds_slots, or 0 where they are formed from the new importance instead
    float scale;
    int32_t sum_threads;  // the softmax sum is formed as by so many threads (at most the workgroup's)
    int32_t fuse_compaction;
    int32_t unordered;    // fused compaction fills holes instead of shifting rows (order by pos only)
    // Head-shared selection runs as two or three launches: phase 1 streams the cache and publishes the
    // new importance, the attention weights and the dense output of every pair; a small kernel
    // sums the new importance over the heads of every sequence, where phase 2 does not do that itself (short caches,
    // ws_tot = NULL); phase 2 selects from that sum (every head of a sequence reaches the same decision) and finishes
    // output and compaction.
    int32_t phase;        // 0 = whole step in one launch; 1, 2 = the two halves of the head-shared
                          // step
    float* ws_p;          // [b,h,cap] attention weights of phase 1
    float* ws_snew;       // [b,h,cap] new importance of phase 1
    float* ws_abar;       // [b,h,d]   dense attention output of phase 1
    float* ws_tot;        // [b,cap]   new importance summed over the heads (NULL: phase 2 sums)
    int32_t stash_rows;   // fused compaction: newest rows kept in LDS during the streaming pass
    // Compressed cache (Section V-B): per (pair, channel) scale and zero point of keys and values,
    // four fp32 arrays of qstride = b*h*d values each (lambda_K, z_K, lambda_V, z_V).
    const float* qparams;
    int64_t qstride;
    // Strict local attention sum (Algorithm 1 line 2): the last ring_rows attention rows per pair,
    // [b,h,ring_rows,cap]; this step overwrites row ring_row and the importance is the sum of
    // the rows.  NULL: running sum in `score`.
    float* ring;
    int32_t ring_rows, ring_row;
};

// The step of caches of few slots (swa_short.hip): which form of that kernel serves a call (nt = 0: swa_decode_kernel does).
struct ShortForm {
    int nt, u;      // threads per workgroup, rows per lane
};
ShortForm short_form(const swa_params& p, int64_t pairs, int len_bound, bool ring);
int launch_short(const DecodeArgs& a, const swa_params& p, int64_t pairs, ShortForm f, hipStream_t stream);
int launch_short_shared(const DecodeArgs& a, const swa_params& p, int64_t pairs, ShortForm f, hipStream_t stream);   // a.phase

}  // namespace swa
