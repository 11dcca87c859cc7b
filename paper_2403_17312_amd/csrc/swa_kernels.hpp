// Host-side launch interface between the C-ABI entry points and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "swa.h"
#include "swa_device.hpp"

namespace swa {

// One launch; every launch of the library goes this way.  The error, if any, is the runtime's last one, as behind <<<>>>, whose compiled
// form puts the launch's shape on a stack of the runtime's and takes it off again: 2.45 us of host time to issue a launch that way, 2.23 this way.
template <typename T>
struct Given { typedef T type; };      // (the kernel's parameters say the types, the arguments are converted to them)
template <typename... A>
inline void launch_kernel(void (*kernel)(A...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, const typename Given<A>::type&... args)
{
    void* arg[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, arg, lds, stream);
}

// Raises the dynamic-LDS limit of a kernel when a launch needs more than the default.  The
// limits already granted are remembered per process (one mutex-guarded table): the only state
// the library keeps besides the address of the static scratch array.
int ensure_dynamic_lds(const void* kernel, size_t bytes);

// Raises that limit to what the current device allows next to the kernel's static LDS.
int raise_dynamic_lds(const void* kernel);

// Raises that limit for every instantiation of the decode kernel on the current device.
int prepare_decode();

// Threads per workgroup of the decode kernel for these params (form, cache format, whether the bound is stated), this many (sequence, head)
// pairs and this bound on the cached length (stated by the caller, or the capacity).
int decode_block_threads(const swa_params& p, int64_t pairs, int len_bound, bool ring);

// Byte offset, inside the caller's workspace, of the slabs the head-shared step passes from its
// first launch to its second (present only when SWA_HEAD_SHARED is set).
size_t shared_workspace_offset(const swa_params& p);

// Bytes of one cache row.
inline int cache_row_bytes(const swa_params& p)
{
    return (p.flags & SWA_KV_INT8) ? p.d : p.d * (p.dtype == SWA_F32 ? 4 : 2);
}

// Rows of K and V the fused-compaction decode parks in LDS (0 = none).
int decode_stash_rows(const swa_params& p);

int launch_workspace_init(const swa_params& p, void* workspace, hipStream_t stream);

int launch_decode(const swa_params& p, float scale, const void* q, const void* k_new, const void* v_new,
                  void* k_cache, void* v_cache, float* score, int32_t* pos, int32_t* cache_len,
                  const int32_t* seq_len, int32_t* kept_idx, int32_t* kept_cnt, void* out,
                  float* probs_dbg, void* workspace, const float* qparams, float* ring, int32_t ring_rows,
                  int32_t ring_row, hipStream_t stream);

// Channel-wise 8-bit compression of an fp16 cache (Section V-B): parameters from the cached rows,
// then the codes.  qparams: four fp32 arrays of b*h*d values (lambda_K, z_K, lambda_V, z_V).
int launch_quantize(const swa_params& p, const void* k_cache, const void* v_cache, const int32_t* cache_len,
                    void* k_codes, void* v_codes, float* qparams, hipStream_t stream);

int launch_compact(const swa_params& p, void* k_cache, void* v_cache, float* score, int32_t* pos,
                   const int32_t* kept_idx, const int32_t* kept_cnt, int32_t* cache_len,
                   hipStream_t stream);

int launch_prefill(const swa_params& p, float scale, const void* q_tail, int32_t R, const void* k_cache,
                   const int32_t* cache_len, float* score, float* rows, bool q_in_place, bool stats_ready,
                   hipStream_t stream);

// Row statistics of the prompt's last R rows, on their way from the attention kernel to the seed's column sums: G copies
// inside the pair's score row, `cols` floats apart, maximum of row r at [r] and normaliser at [R + r].  G = 0: none.
void seed_stats_place(int64_t pairs, int bound, int cap, int R, int& G, int& cols);

// Whether the seed on its own runs as two launches (bound on the lengths: stated by the caller, or the capacity).
bool seed_in_two(int64_t pairs, int bound, bool stated, int R);

// Whether its row statistics then come from four workgroups per 32 rows, whose sums the column sums merge, or from one.
bool seed_chains_apart(int G, int cols, int cap, int R);

// SWA_SPLIT_ROWS: workgroups per pair for this many pairs, this bound on the cached length (stated by the caller, or the capacity) and rows of so many bytes
// (1 = the one-workgroup kernel serves the call), and the launches of the step.
constexpr int kMaxSplit = 16;
int split_factor(int64_t pairs, int len_bound, bool stated, int row_bytes);
int split_piece_bytes(int64_t pairs);
int launch_split(const swa_params& p, float scale, int G, const void* q, const void* k_new, const void* v_new, void* k_cache,
                 void* v_cache, float* score, int32_t* pos, int32_t* cache_len, const int32_t* seq_len, int32_t* kept_idx,
                 int32_t* kept_cnt, void* out, float* probs_dbg, void* workspace, hipStream_t stream);

// Token-level offload tier (Section V-A, Algorithm 2): evicted rows to the host store, requested rows back.
int launch_offload(const swa_params& p, const void* k_cache, const void* v_cache, const float* score,
                   const int32_t* pos, const int32_t* kept_idx, const int32_t* kept_cnt, const int32_t* cache_len,
                   const swa_host_store& st, void* workspace, hipStream_t stream);
int launch_reload(const swa_params& p, const swa_host_store& st, const int32_t* req_idx, const int32_t* req_cnt,
                  int32_t max_req, void* k_cache, void* v_cache, float* score, int32_t* pos,
                  const int32_t* cache_len, int32_t* new_len, void* workspace, hipStream_t stream);

// Causal attention over the whole prompt (Eq. 1-2) on MFMA: out[t] for every prompt position.  Where it can, it leaves
// the statistics of the last R rows in score (seed_stats_place) and says so.
int launch_flash_prefill(const swa_params& p, float scale, const void* q, const void* k_cache, const void* v_cache,
                         const int32_t* cache_len, void* out, int32_t R, float* score, bool& stats_written,
                         hipStream_t stream);

}  // namespace swa
