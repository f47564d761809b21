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

// Launch order of the key-major pass: its workgroups differ in work by the length of their
// transposed list (a sink or current-chunk block is kept by every query block, a block of the
// middle history by few).  Workgroup indices go round-robin to the eight XCDs, so every XCD works
// through a fixed set of blocks: `per_xcd` places of the sequence "head after head, and inside a
// head the KV blocks in steps of `step` blocks".  All heads carry the same number of tiles; where
// an XCD's share ends inside a head, the step (about 0.618 n_k, prime to n_k) spreads the share
// evenly over the head's blocks, heavy and light.  With the blocks in plain order the XCD that
// got the head's second half, current chunk included, had 27 % more tiles than the one with the
// first half, and a quarter of the launch's time was spent waiting for it (12 heads, 525 KV
// blocks: the forward and backward calls together 1780 us, now 1672 us).
// Inside an XCD workgroups are started in index order, so the long ones go first: one workgroup per
// XCD sorts its share by descending count with a counting sort.  These eight ride at the front of
// the dQ launch, which does not need the order (a launch of their own took 5 us).  The place of equal counts
// among each other is left to the order the atomics happen to take: any permutation is valid,
// and the gradients do not depend on which workgroup computes a block.
constexpr int kOrderBins = 1024;
__device__ __forceinline__ void order_share(const BwdArgs& a, int xcd, int* bins /* [kOrderBins] in LDS */) {
  const int threads = blockDim.x, tid = threadIdx.x;
  const int w0 = xcd * a.order_per_xcd, w1 = min(a.order_total, w0 + a.order_per_xcd);
  // Block at place i of the sequence: head i / n_k, and in it the block i step mod n_k (whole heads before it
  // drop out of the remainder), which moves on by a constant when i moves on by the number of threads.
  const uint32_t nk = (uint32_t)a.order_n_k;
  const uint32_t c0 = (uint32_t)((uint64_t)((uint32_t)(w0 + tid) % nk) * a.order_step % nk);
  // Every block of the share with its bin, U at a time: their loads (and LDS atomics) are in flight together.
  // A long history has thousands of blocks a share, and one at a time the loop outlasts the dQ launch.
  auto each_block = [&](auto put) __attribute__((always_inline)) {
    constexpr int U = 8;
    uint32_t c = c0;
    for (int i0 = w0 + tid; i0 < w1; i0 += U * threads) {
      int w[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * threads;
        w[u] = i < w1 ? (int)((uint32_t)i / nk * nk + c) : w[0];   // past the end: any block, loaded and dropped
        c += a.order_stride;
        c -= c >= nk ? nk : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) b[u] = min(a.order_cnt[w[u]], kOrderBins - 1);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + u * threads < w1) put(w[u], b[u]);
    }
  };
  for (int i = tid; i < kOrderBins; i += threads) bins[i] = 0;
  __syncthreads();
  each_block([&](int, int b) { atomicAdd(&bins[b], 1); });
  __syncthreads();
  // bins[b] <- number of places in bins above b (where bin b starts in the descending order); lane l
  // of the first wavefront takes the l-th sixteen bins from the top
  if (tid < 64) {
    constexpr int PER = kOrderBins / 64;
    int cnt[PER], sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      cnt[j] = bins[kOrderBins - 1 - (PER * tid + j)];
      sum += cnt[j];
    }
    int run = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(run, d);
      if (tid >= d) run += up;
    }
    run -= sum;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      bins[kOrderBins - 1 - (PER * tid + j)] = run;
      run += cnt[j];
    }
  }
  __syncthreads();
  each_block([&](int w, int b) { a.order[w0 + atomicAdd(&bins[b], 1)] = w; });
}

}  // namespace

// dQ at head dimension 128 with one wavefront per query block (lf_attn_bwd_q_wide.hip); `a` as for the other dQ kernel.
hipError_t lf_launch_attn_bwd_q_wide(const BwdArgs& a, hipStream_t st);
// dK and dV at head dimension 128 (lf_attn_bwd_wide.hip); `a` as for the other key-major kernel.
hipError_t lf_launch_attn_bwd_kv_wide(const BwdArgs& a, hipStream_t st);

#endif
