// Internal declarations shared by the host entry points and the gfx950 kernels.
#ifndef LF_COMMON_H
#define LF_COMMON_H

#include <stddef.h>
#include <stdint.h>

#include "lf.h"

#define LF_MAX_CAND_BLOCKS 2048  // |B_r| the selection kernel can rank in LDS
#define LF_MAX_CAND_FRAMES 1024  // |M| the selection kernel can rank in LDS
#define LF_MAX_HIST_FRAMES 4096  // F_h bound (flag array in LDS)
#define LF_MAX_CHUNK_FRAMES 1024 // f bound: with the three above it keeps the selection kernel's
                                 // dynamic LDS below 64 KiB, so the size is known to fit
                                 // before anything is enqueued

// Size of the library-owned device scratch behind lf_select_mask_static (per GPU).
#define LF_STATIC_SCRATCH_BYTES ((size_t)16 << 20)

// Derived sizes of one call; filled by lf_derive() after validation.
struct lf_dims {
  int H, d, n, f, F, F_h, nb, n_q, n_k, m;
  int n_tf;     // selected history frames: n_sink + n_win + k_frames
  int n_cand;   // |B_r|
  size_t off_qt, off_kt, off_kh, ws_bytes;
};

// Validates shape (and budget when non-NULL); returns LF_OK or an lf_status.
int lf_derive(const lf_shape* s, const lf_budget* b, lf_dims* out);

// Whether the query-major attention kernels divide each list among the four pairs of wavefronts of
// a workgroup instead of giving every (head, query block) one pair.  A divided block takes a
// compute unit (256 of them) to itself at d = 128.  Measured, d = 128, forward call / backward call
// (dQ divided, the rest as it was), us before -> after:
//   <= 256 blocks: 192 blocks, lists of 8: 18.0 -> 14.3 / 53.5 -> 48.9; of 40: 51.1 -> 27.9 / 130 -> 97;
//     lists of 4 are one step a slice: 13.5 -> 13.3 / 41.1 -> 41.6, not divided;
//   two rounds: 320 blocks, lists of 16: 27.8 -> 31.2 / 90.3 -> 89.1; of 40: 54.8 -> 52.1 / 158 -> 149;
//     480 blocks, lists of 40: 63.1 -> 56.2 / 199 -> 188;
//   three: 560 blocks, lists of 40: 74.4 -> 80.4 / 217 -> 242.
// At d = 64 two divided blocks share a compute unit and the gain is larger (480 blocks, lists of 40:
// 47.3 -> 37.8 / 165 -> 153; of 8: 16.0 -> 18.3 / 57.4 -> 58.5); the same line serves.
inline bool lf_split_lists(int blocks, int list_len) {
  return (blocks <= 256 && list_len >= 6) || (blocks <= 512 && list_len >= 32);
}

// Kernel launchers (defined in the .hip files); return LF_OK or LF_ERR_HIP.
int lf_launch_select(const void* Q, const void* K, const lf_shape* s, const lf_budget* b,
                     const lf_dims* dm, int32_t* indices, void* workspace, void* stream);
int lf_launch_kcache_update(const void* K, const lf_shape* s, const lf_dims* dm, int frame0, int frame1,
                            int max_frames, void* kcache, void* stream);
int lf_launch_select_cached(const void* Q, const void* Kcur, void* kcache, int max_frames,
                            const lf_shape* s, const lf_budget* b, const lf_dims* dm, int32_t* indices,
                            void* workspace, void* stream);
int lf_launch_qk_norm_rope(const void* X, const float* g, const float* cosv, const float* sinv,
                           const lf_producer_shape* p, void* Y, void* stream);
// Device address of the library's static scratch on the current device (looked up on the first
// call per device); LF_OK or LF_ERR_HIP.
int lf_static_scratch(void** ptr);
int lf_launch_attn(const void* Q, const void* K, const void* V, const lf_shape* s,
                   const lf_dims* dm, const int32_t* indices, int32_t list_len, int32_t list_stride,
                   float scale, void* O, const float* state_o, const float* state_ml, float* lse2,
                   void* stream);
int lf_launch_attn_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                       const float* lse2, const lf_shape* s, const lf_dims* dm, const int32_t* indices,
                       int32_t list_len, float scale, void* dQ, void* dK, void* dV, float* ndelta,
                       int32_t* tlist, int32_t* tcnt, int32_t* order, void* stream);
int lf_launch_attn_dense(const void* Q, const void* K, const void* V, const lf_shape* s,
                         const lf_dims* dm, int kv0, int kv1, float scale, float* state_o,
                         float* state_ml, void* stream);

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
// Launches a kernel and returns this launch's own status (an error left behind by the caller's
// earlier work is neither reported nor cleared).
template <typename... KArgs, typename... Args>
inline hipError_t lf_launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds_bytes,
                            hipStream_t stream, Args... args) {
  void* argv[] = {(void*)&args...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, argv, lds_bytes, stream);
}
#endif

#endif
