// Producer of Q and K next to the hot path: RMSNorm, then rotary position embedding, written
// head-major in the layout mask selection and attention read (the paper's "Efficient
// Deployment" section names fused RoPE and RMSNorm kernels; it defines neither, so these are
// the textbook operators, see lf.h).  HBM-bound: one read of the token-major activations, one
// write of the head-major result, plus the angle table.
//
// One wavefront per token.  A lane owns 16-byte chunks (8 channels) of the token, chunk
// 64 it + lane in iteration it; the CH = d/8 chunks of a head sit in CH neighbouring lanes, so
// the per-head mean of squares is a reduction over CH lanes and the rotation partner of the
// "half" pairing is CH/2 lanes away.  All arithmetic is float32; the result is rounded to
// bfloat16 once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lf_common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct ProducerArgs {
  const uint16_t* X;
  const float* g;
  const float* cosv;
  const float* sinv;
  uint16_t* Y;
  int64_t x_stride_tok, y_stride_tok, y_stride_head;
  int H, L, across_heads, pairing;
  float eps;
};

constexpr int kTokensPerWg = 4;

__device__ __forceinline__ void unpack8(const uint4& u, float (&x)[8]) {
  x[0] = __uint_as_float(u.x << 16); x[1] = __uint_as_float(u.x & 0xffff0000u);
  x[2] = __uint_as_float(u.y << 16); x[3] = __uint_as_float(u.y & 0xffff0000u);
  x[4] = __uint_as_float(u.z << 16); x[5] = __uint_as_float(u.z & 0xffff0000u);
  x[6] = __uint_as_float(u.w << 16); x[7] = __uint_as_float(u.w & 0xffff0000u);
}

// NI > 0: a token is at most 64 NI chunks, read once and held in registers (4 per chunk) between
// the mean of squares and the rotation.  NI = 0: any length; the second pass reads the token again.
// What bounds it: one wavefront per token is one round of wavefronts on the chip at the sizes of a
// chunk (4 680 tokens), so the time is one token's chain -- read, reduce over the lanes, scale,
// rotate, write -- on top of the bytes.  The angles, which depend on the lane only and not on the head, are
// requested together with the token; so are the norm weights of tokens up to 256 chunks (8 registers per
// chunk), and longer tokens ask for theirs after the reduction, from the L2.
// 12 heads x 128, 4 680 tokens: 9.3 us a call with the token read twice and the weights and angles requested where used,
// 8.6 us now (28.8 MB: 3.3 TB/s).
template <int D, int NI>
__global__ __launch_bounds__(64 * kTokensPerWg) void lf_qk_norm_rope_kernel(ProducerArgs a) {
  constexpr int CH = D / 8;
  constexpr bool kHeld = NI > 0;
  constexpr int NX = kHeld ? NI : 1;
  constexpr bool kEarlyG = kHeld && NI <= 4;    // norm weights in registers too (8 per chunk)
  constexpr int NG = kEarlyG ? NI : 1;
  const int lane = threadIdx.x & 63;
  const int tok = blockIdx.x * kTokensPerWg + (threadIdx.x >> 6);
  if (tok >= a.L) return;                       // whole wavefronts leave; no barrier below
  const int nc = a.H * CH;                      // chunks per token
  const uint16_t* xrow = a.X + (int64_t)tok * a.x_stride_tok;
  const int cih = lane % CH;                    // place inside the head: 64 is a multiple of CH

  uint4 xr[NX];
  float4 gr[NG][2];
  auto load_g = [&](int c, float4 (&g)[2]) __attribute__((always_inline)) {
    g[0] = *reinterpret_cast<const float4*>(a.g + 8 * c);
    g[1] = *reinterpret_cast<const float4*>(a.g + 8 * c + 4);
  };
  if constexpr (kHeld) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int c = 64 * i + lane;
      xr[i] = c < nc ? *reinterpret_cast<const uint4*>(xrow + 8 * c) : make_uint4(0, 0, 0, 0);
    }
  }
  // angles: pairs (2i, 2i+1): this chunk holds pairs 4 cih .. 4 cih + 3;
  // pairs (i, i + d/2): this chunk and its partner hold pairs 8 (cih mod CH/2) .. + 7
  float4 cs[2], sn[2];
  {
    const float* ct = a.cosv + (int64_t)tok * (D / 2);
    const float* st = a.sinv + (int64_t)tok * (D / 2);
    const int i0 = a.pairing == 0 ? 4 * cih : 8 * (cih % (CH / 2));
    cs[0] = *reinterpret_cast<const float4*>(ct + i0);
    sn[0] = *reinterpret_cast<const float4*>(st + i0);
    if (a.pairing != 0) {
      cs[1] = *reinterpret_cast<const float4*>(ct + i0 + 4);
      sn[1] = *reinterpret_cast<const float4*>(st + i0 + 4);
    } else {
      cs[1] = sn[1] = make_float4(0, 0, 0, 0);
    }
  }
  if constexpr (kEarlyG) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      if (64 * i + lane < nc) load_g(64 * i + lane, gr[i]);
      else gr[i][0] = gr[i][1] = make_float4(0, 0, 0, 0);
    }
  }

  float inv_all = 0.0f;
  if (a.across_heads) {
    float ss = 0.0f;
    auto add = [&](const uint4& u) __attribute__((always_inline)) {
      float x[8];
      unpack8(u, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
    };
    if constexpr (kHeld) {
#pragma unroll
      for (int i = 0; i < NX; ++i) add(xr[i]);
    } else {
      for (int c = lane; c < nc; c += 64) add(*reinterpret_cast<const uint4*>(xrow + 8 * c));
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) ss += __shfl_xor(ss, off);
    inv_all = 1.0f / sqrtf(ss / (float)(a.H * D) + a.eps);
  }

  // chunk c of this lane (past the last chunk a lane still takes part in the exchanges)
  auto chunk = [&](int c, const uint4& u, const float4 (&g)[2]) __attribute__((always_inline)) {
    float x[8];
    unpack8(u, x);
    float inv = inv_all;
    if (!a.across_heads) {
      float ss = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
#pragma unroll
      for (int off = 1; off < CH; off <<= 1) ss += __shfl_xor(ss, off);
      inv = 1.0f / sqrtf(ss / (float)D + a.eps);
    }
    const float gg[8] = {g[0].x, g[0].y, g[0].z, g[0].w, g[1].x, g[1].y, g[1].z, g[1].w};
    const float cc[8] = {cs[0].x, cs[0].y, cs[0].z, cs[0].w, cs[1].x, cs[1].y, cs[1].z, cs[1].w};
    const float sv[8] = {sn[0].x, sn[0].y, sn[0].z, sn[0].w, sn[1].x, sn[1].y, sn[1].z, sn[1].w};
    float y[8], r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = x[e] * inv * gg[e];
    if (a.pairing == 0) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        r[2 * p] = y[2 * p] * cc[p] - y[2 * p + 1] * sv[p];
        r[2 * p + 1] = y[2 * p] * sv[p] + y[2 * p + 1] * cc[p];
      }
    } else {
      // the partner chunk is CH/2 lanes away inside the head
      const bool first = cih < CH / 2;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float other = __shfl_xor(y[e], CH / 2);
        r[e] = first ? y[e] * cc[e] - other * sv[e] : other * sv[e] + y[e] * cc[e];
      }
    }
    if (c < nc) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (__bf16)r[e];
      *reinterpret_cast<bf16x8*>(a.Y + (int64_t)(c / CH) * a.y_stride_head + (int64_t)tok * a.y_stride_tok + 8 * cih) = o;
    }
  };
  if constexpr (kHeld) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      if (64 * i >= nc) break;
      const int c = 64 * i + lane;
      if constexpr (kEarlyG) {
        chunk(c, xr[i], gr[i]);
      } else {
        float4 g[2] = {make_float4(0, 0, 0, 0), make_float4(0, 0, 0, 0)};
        if (c < nc) load_g(c, g);
        chunk(c, xr[i], g);
      }
    }
  } else {
    for (int c0 = 0; c0 < nc; c0 += 64) {
      const int c = c0 + lane;
      uint4 u = make_uint4(0, 0, 0, 0);
      float4 g[2] = {make_float4(0, 0, 0, 0), make_float4(0, 0, 0, 0)};
      if (c < nc) {
        u = *reinterpret_cast<const uint4*>(xrow + 8 * c);
        load_g(c, g);
      }
      chunk(c, u, g);
    }
  }
}

template <int D>
hipError_t launch_producer(const ProducerArgs& a, dim3 grid, hipStream_t st) {
  const int nc = a.H * (D / 8);
  // registers: 4 x 12 for the wider form leave four wavefronts per SIMD; beyond it the token is read twice
  const dim3 block(64 * kTokensPerWg);
  if (nc <= 4 * 64) return lf_launch(lf_qk_norm_rope_kernel<D, 4>, grid, block, 0, st, a);
  if (nc <= 12 * 64) return lf_launch(lf_qk_norm_rope_kernel<D, 12>, grid, block, 0, st, a);
  return lf_launch(lf_qk_norm_rope_kernel<D, 0>, grid, block, 0, st, a);
}

}  // namespace

int lf_launch_qk_norm_rope(const void* X, const float* g, const float* cosv, const float* sinv,
                           const lf_producer_shape* p, void* Y, void* stream) {
  ProducerArgs a;
  a.X = (const uint16_t*)X;
  a.g = g;
  a.cosv = cosv;
  a.sinv = sinv;
  a.Y = (uint16_t*)Y;
  a.x_stride_tok = p->x_stride_tok;
  a.y_stride_tok = p->y_stride_tok;
  a.y_stride_head = p->y_stride_head;
  a.H = p->heads;
  a.L = p->tokens;
  a.across_heads = p->across_heads;
  a.pairing = p->pairing;
  a.eps = p->eps;
  const unsigned grid = (unsigned)((p->tokens + kTokensPerWg - 1) / kTokensPerWg);
  hipStream_t st = (hipStream_t)stream;
  const hipError_t rc = p->head_dim == 128 ? launch_producer<128>(a, dim3(grid), st) : launch_producer<64>(a, dim3(grid), st);
  return rc == hipSuccess ? LF_OK : LF_ERR_HIP;
}
