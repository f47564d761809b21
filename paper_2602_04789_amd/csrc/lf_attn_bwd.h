// Shared by the backward kernels: their arguments, the LDS tile layout and small device helpers.
#ifndef LF_ATTN_BWD_H
#define LF_ATTN_BWD_H

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lf_common.h"

// Arguments of the backward kernels.
struct BwdArgs {
  const uint16_t* X;     // owner-side operand of the scores (Q for dQ, K for dK and dV)
  const uint16_t* Y;     // owner-side operand of dP (dO for dQ, V for dK)
  const uint16_t* A1;    // streamed operand of the scores (K for dQ, Q for dK and dV)
  const uint16_t* A2;    // streamed operand of dP (V for dQ, dO for dK and dV)
  uint16_t* out1;        // dQ or dK: scale * sum of A1^T dS'
  uint16_t* out2;        // dV: sum of A2^T P'
  const float* lse2;     // log-sum-exp per query row (exp2 domain), [H][q_len]
  const float* ndelta;   // -delta per query row, [H][q_len]
  const int32_t* idx;    // lists: [H][owners][list_stride]
  const int32_t* cnt;    // key-major: entries per transposed list
  int32_t* order;        // owner handled by workgroup slot w of the key-major launch (made beside the dQ launch)
  const int32_t* order_cnt;                      // dQ launch: entries per transposed list, for the order
  int order_total, order_per_xcd, order_n_k;
  uint32_t order_step, order_stride;             // step through a head; (threads of a workgroup x step) mod n_k
  int64_t x_tok, x_head, y_tok, y_head, a1_tok, a1_head, a2_tok, a2_head;
  int64_t o1_tok, o1_head, o2_tok, o2_head;
  int n, nb, owners, streams, list_len, list_stride, q_len;
  int total_wg, wg_per_xcd;
  float c, scale;
};

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int int32x4 __attribute__((ext_vector_type(4)));

union Frag {
  uint4 u;
  bf16x8 v;
};

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// One swizzle for both tiles of a step, since each is read both ways.  Row reads: 16 bytes per
// lane, 16 consecutive rows at one logical chunk per quarter wavefront, which must land in 16
// different chunks.  Transposing reads: half a wavefront takes four consecutive chunks from each
// of four consecutive rows (4 k .. 4 k + 3), which must land in four different quarters of the
// banks.  For 256-byte rows: the row's two low bits go to the chunk's two high bits (the four
// rows of a transposing read differ there), the next two row bits to the chunk's two low bits
// (constant within a transposing read, and together a bijection of the 16 rows of a row read).
template <int CH> __device__ __forceinline__ int swz(int row, int ch) {
  return CH == 16 ? ch ^ (((row & 3) << 2) | ((row >> 2) & 3)) : ch ^ ((row & 1) << 2);
}
// The transposing read of rows 8..15 of a 16-row group sees row bit 3, i.e. chunk bit 1, flipped:
// 16 elements aside.
template <int CH> constexpr int kTrHiFlip = CH == 16 ? 16 : 0;

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

}  // namespace

// dK and dV at head dimension 128 (lf_attn_bwd_wide.hip); `a` as for the other key-major kernel.
hipError_t lf_launch_attn_bwd_kv_wide(const BwdArgs& a, hipStream_t st);

#endif
