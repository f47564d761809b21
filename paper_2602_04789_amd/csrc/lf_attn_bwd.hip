// Backward pass of the blockwise sparse attention (Eq. 13) for gfx950: gradients with respect
// to Q, K and V for an upstream gradient dO, over exactly the tiles the index lists keep
// (the paper finetunes with the sparse mask in place, Sec. 5 "Experimental Details").
//
// With s_xy = scale q_x.k_y, p = softmax over the kept columns, o = p v:
//     dV_y = sum_x p_xy dO_x          dp_xy = dO_x . v_y      delta_x = dO_x . o_x
//     ds_xy = p_xy (dp_xy - delta_x)  dQ_x = scale sum_y ds_xy k_y    dK_y = scale sum_x ds_xy q_x
// p is rebuilt from the row's log-sum-exp, which the training forward call leaves (in the exp2
// domain: lse2_x = log2 sum_y exp2(s_xy log2 e)), so no row maximum or sum is needed here.
//
// No atomics and a fixed summation order: every launch owns its outputs.  The dQ launch is
// query-major (a workgroup owns a query block, walks its list of KV blocks, keeps dQ in
// registers); the dK/dV launch is key-major (a workgroup owns a KV block and walks the list of
// query blocks that keep it -- the transposed lists, made by a small kernel -- and keeps dK and dV
// in registers).  Both recompute the scores of a tile.  The products are arranged as in the
// forward kernel: the "score-like" products S' = A1 X^T and dP' = A2 Y^T take their A operand
// from a 32-row tile in LDS (row reads) and their B operand from registers that hold the owner
// block, which leaves a lane with one owner column and 16 stream rows; P' and dS' are then
// already in the B-operand layout of the accumulating product, whose A operand is the same tile
// read through the transposing LDS read.
//     dQ:      owner = query block (X = Q, Y = dO), stream = KV blocks (A1 = K, A2 = V),
//              dQ^T += K^T dS'
//     dK, dV:  owner = KV block (X = K, Y = V), stream = query blocks (A1 = Q, A2 = dO),
//              dK^T += Q^T dS'  and  dV^T += dO^T P', by two kinds of wavefront that share P'
#include "lf_attn_bwd.h"

namespace {

constexpr int kThreads = 128;    // two wavefronts of 32 owner rows each
constexpr int kPass = 256;       // list entries decoded per pass

// dQ: a workgroup of two wavefronts owns a query block (wavefront rh its rows [32 rh, +32)) and
// walks the block's list of KV blocks in half tiles of 32 KV rows.  SPLIT > 1 (two or four): the workgroup has
// SPLIT such pairs with a tile stage each, every pair walks a SPLIT-th of the list (the barriers are
// common, the slices equally long but for empty entries at the end), and their sums are added
// through LDS in a fixed order: for calls with too few query blocks to fill the chip.  HALF: for fewer still, the
// workgroup has one row half of a query block, and a slice is one wavefront with a stage of its own, without barriers in
// the loop (four slices at d = 128, where LDS holds no more stages, eight at d = 64).
template <int D, int SPLIT, bool HALF = false>
__global__ __launch_bounds__((HALF ? 64 : kThreads) * SPLIT, HALF ? 1 : D == 64 && SPLIT == 1 ? 3 : 2) void lf_attn_bwd_q_kernel(BwdArgs a) {
  constexpr int WPS = HALF ? 1 : 2;         // wavefronts that share a tile stage
  constexpr int kStageThreads = 64 * WPS;        // ... and their threads
  constexpr int CH = D / 8;
  constexpr int KS = D / 16;
  constexpr int MB = D / 32;
  constexpr int RPI = 64 / CH;
  constexpr int LPW = 32 / (RPI * WPS);
  constexpr int TILE = 32 * CH;             // uint4 per 32-row tile
  constexpr int NBUF = 2;

  __shared__ uint4 buf_all[SPLIT][NBUF][2 * TILE];     // [slice][step mod NBUF][A1 tile | A2 tile]
  __shared__ int2 ent_all[SPLIT][kPass];               // (first token, token count) per list entry of a pass

  if (blockIdx.x < 8) {
    static_assert(sizeof(buf_all) >= kOrderBins * sizeof(int), "the order's bins use the tile stage");
    order_share(a, blockIdx.x, reinterpret_cast<int*>(buf_all));
    return;
  }
  const int w = (blockIdx.x & 7) * a.wg_per_xcd + (blockIdx.x >> 3) - 1;
  if (w >= a.total_wg) return;
  const int h = (HALF ? w >> 1 : w) / a.owners, r = (HALF ? w >> 1 : w) % a.owners;
  const int slice = SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kStageThreads) : 0;
  uint4 (*const buf)[2 * TILE] = buf_all[slice];
  int2* const ent = ent_all[slice];
  const int tid = threadIdx.x % kStageThreads, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, kg = lane >> 5;

  // owner block: tokens [otok0, otok0 + o_cnt); this lane's owner row (a column of S')
  const int otok0 = (r / a.nb) * a.n + (r % a.nb) * 64;
  const int o_cnt = min(64, a.n - (r % a.nb) * 64);
  const int rh = HALF ? w & 1 : wave;       // row half
  const int orow = 32 * rh + ln;
  const bool o_ok = orow < o_cnt;
  if (HALF && 32 * rh >= o_cnt) return;     // the other half of a short query block

  // this pair's slice: entries [slice n_ent, +n_ent) of the list, of which my_ent exist
  const int n_ent = (a.list_len + SPLIT - 1) / SPLIT;
  const int my_ent = SPLIT > 1 ? min(max(a.list_len - slice * n_ent, 0), n_ent) : n_ent;
  const int32_t* list = a.idx + ((int64_t)h * a.owners + r) * a.list_stride + (SPLIT > 1 ? slice * n_ent : 0);

  // B operands: lane (column ln, k-group kg) holds 8 consecutive channels of its owner row
  Frag xf[KS], yf[KS];
  {
    const uint16_t* xp = a.X + (int64_t)h * a.x_head + (int64_t)(otok0 + orow) * a.x_tok;
    const uint16_t* yp = a.Y + (int64_t)h * a.y_head + (int64_t)(otok0 + orow) * a.y_tok;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      xf[s].u = o_ok ? *reinterpret_cast<const uint4*>(xp + s * 16 + kg * 8) : make_uint4(0, 0, 0, 0);
      yf[s].u = o_ok ? *reinterpret_cast<const uint4*>(yp + s * 16 + kg * 8) : make_uint4(0, 0, 0, 0);
    }
  }
  // dQ: the query row of this lane; its log-sum-exp and delta (a row outside the block gets
  // +inf, which makes all its probabilities zero)
  float my_lse = INFINITY, my_nd = 0.0f;
  if (o_ok) {
    my_lse = a.lse2[(int64_t)h * a.q_len + otok0 + orow];
    my_nd = a.ndelta[(int64_t)h * a.q_len + otok0 + orow];
  }

  const char* A1h = reinterpret_cast<const char*>(a.A1 + (int64_t)h * a.a1_head);
  const char* A2h = reinterpret_cast<const char*>(a.A2 + (int64_t)h * a.a2_head);
  const uint32_t a1_row_bytes = (uint32_t)(a.a1_tok * 2), a2_row_bytes = (uint32_t)(a.a2_tok * 2);

  // tile loads, global -> LDS (see the forward kernel): load i of wavefront `wave` fills rows
  // [RPI (LPW wave + i), +RPI); the buffer resource is the tile itself, so rows past the count
  // read as zeros and ids outside the tensor become empty tiles
  const int ld_r = lane / CH, ld_p = lane % CH;
  uint32_t off1[LPW], off2[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int row = RPI * (LPW * wave + i) + ld_r;
    off1[i] = (uint32_t)row * a1_row_bytes + (uint32_t)swz<CH>(row, ld_p) * 16u - 1024u * (i & 3);
    off2[i] = (uint32_t)row * a2_row_bytes + (uint32_t)swz<CH>(row, ld_p) * 16u - 1024u * (i & 3);
  }
  auto rsrc = [](const char* base, uint32_t row_bytes, int2 e) {
    int32x4 rs;
    const uint64_t b = (uint64_t)base + (uint64_t)(uint32_t)e.x * row_bytes;
    rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    rs[2] = __builtin_amdgcn_readfirstlane((int)((uint32_t)e.y * row_bytes));
    rs[3] = 0x00020000;
    return rs;
  };
  auto fetch = [&](int32x4 rs, uint4* dst, const uint32_t (&off)[LPW]) __attribute__((always_inline)) {
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)LDS_PTR(void, dst + RPI * LPW * wave * CH));
    if constexpr (LPW >= 4) {
#pragma unroll
      for (int i = 0; i < LPW; i += 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                     "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
                     :: "s"(lds0 + 1024u * i), "v"(off[i]), "v"(off[i + 1]), "v"(off[i + 2]), "v"(off[i + 3]), "s"(rs)
                     : "memory", "m0");
    } else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                   "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds"
                   :: "s"(lds0), "v"(off[0]), "v"(off[1]), "s"(rs) : "memory", "m0");
  };
  // half tile t of the pass: list entry t/2 (given as read from `ent`), rows [32 (t&1), +32) of its block
  auto half = [](int2 e, int t) {
    const int2 u = make_int2(__builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y));
    return (t & 1) ? make_int2(u.x + 32, max(u.y - 32, 0)) : make_int2(u.x, min(u.y, 32));
  };
  auto request = [&](int2 e, uint4* stage) __attribute__((always_inline)) {
    fetch(rsrc(A1h, a1_row_bytes, e), stage, off1);
    fetch(rsrc(A2h, a2_row_bytes, e), stage + TILE, off2);
  };

  // LDS addresses of this lane's fragments (loop invariants): row reads of row ln, chunk 2s+kg
  int raddr[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) raddr[s] = ln * CH + swz<CH>(ln, 2 * s + kg);
  // transposing reads (see the forward kernel), in bf16 elements
  int tbase[MB];
  {
    const int i16 = lane & 15;
    const int tr_row = 4 * kg + (i16 >> 2);
    const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int col = 32 * mb + tr_col;
      tbase[mb] = (tr_row * CH + swz<CH>(tr_row, col >> 3)) * 8 + (col & 7);
    }
  }
  auto tfrag = [&](const uint4* tile, int u, int mb) __attribute__((always_inline)) {
    const uint16_t* p16 = reinterpret_cast<const uint16_t*>(tile);
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p16 + tbase[mb] + (16 * u) * CH * 8));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        LDS_PTR(bf16x4, p16 + (tbase[mb] ^ kTrHiFlip<CH>) + (16 * u + 8) * CH * 8));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  f32x16 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[mb][i] = 0.0f;
  f32x16 zero16;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero16[i] = 0.0f;

  f32x16 nd16;
#pragma unroll
  for (int i = 0; i < 16; ++i) nd16[i] = my_nd;

  // S'[stream row, owner column] = A1 X^T and dP' = A2 Y^T of this wavefront's 32 x 32 tile.
  // The fragment reads are kept KS/2 k-steps ahead of the products that use them (the compiler,
  // left alone, issues each read right before its product and waits for it); the scheduling
  // barriers pin that order.
  auto scores = [&](const uint4* tile, f32x16& sacc, f32x16& pacc) __attribute__((always_inline)) {
    constexpr int HB = KS / 2;
    Frag f1[HB], f2[HB];
    sacc = zero16;
    pacc = nd16;
#pragma unroll
    for (int s = 0; s < HB; ++s) {
      f1[s].u = tile[raddr[s]];
      f2[s].u = tile[TILE + raddr[s]];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < HB; ++s) {
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[s].v, xf[s].v, sacc, 0, 0, 0);
      f1[s].u = tile[raddr[HB + s]];
      pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[s].v, yf[s].v, pacc, 0, 0, 0);
      f2[s].u = tile[TILE + raddr[HB + s]];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < HB; ++s) {
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[s].v, xf[HB + s].v, sacc, 0, 0, 0);
      pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[s].v, yf[HB + s].v, pacc, 0, 0, 0);
    }
  };
  // P' = exp2(s c - lse2), dS' = P' (dP' - delta), packed to bfloat16 in the B-operand layout of
  // the accumulating product; accumulator i is stream row 8 (i/4) + 4 kg + i%4
  auto probs = [&](f32x16& sacc, const f32x16& pacc, int cnt, bf16x8 (&dsf)[2]) __attribute__((always_inline)) {
    // stream rows past a short half tile's count were loaded as zeros: their scores become -inf
    // (P' = 0); a full half tile, the common case, skips this
    if (cnt < 32) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + 4 * kg + (i & 3) >= cnt) sacc[i] = -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p = __builtin_amdgcn_exp2f(fmaf(sacc[i], a.c, -my_lse));
      dsf[i >> 3][i & 7] = (__bf16)(p * pacc[i]);
    }
  };
  // acc += K^T dS'.  The transposed fragments of the first 16
  // stream rows are requested by `first_half` before the exp2 work, which covers their latency;
  // those of the second 16 rows are requested between the products of the first.
  auto first_half = [&](const uint4* tile, bf16x8 (&tf)[MB]) __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) tf[mb] = tfrag(tile, 0, mb);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto accumulate = [&](const uint4* tile, bf16x8 (&tf)[MB], const bf16x8 (&dsf)[2]) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[mb], dsf[0], acc[mb], 0, 0, 0);
      tf[mb] = tfrag(tile, 1, mb);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[mb], dsf[1], acc[mb], 0, 0, 0);
  };

  for (int l0 = 0; l0 < n_ent; l0 += kPass) {
    const int l1 = min(n_ent, l0 + kPass);
    const int n_local = l1 - l0, steps = 2 * n_local;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    for (int i = tid; i < n_local; i += kStageThreads) {
      const int cidx = l0 + i < my_ent ? list[l0 + i] : -1;
      const bool ok = (unsigned)cidx < (unsigned)a.streams;
      const int tau = ok ? cidx / a.nb : 0, j = ok ? cidx % a.nb : 0;
      ent[i] = make_int2(tau * a.n + j * 64, ok ? min(64, a.n - j * 64) : 0);
    }
    __syncthreads();

    // Step t uses buf[t & 1]; its tiles are requested one step ahead, and the list entry behind a
    // request is read a step before that.  The number of steps is even: two an iteration, so that the
    // stages are constants (with the entry read where used and the stage in a register the last-chunk
    // call took 1260 us, now 1227 us).
    int2 e_cur = half(ent[0], 0), e_nxt = half(ent[0], 1);
    request(e_cur, buf[0]);
    auto step = [&](int t, uint4* tile, uint4* other) __attribute__((always_inline)) {
      const int cnt = e_cur.y;
      const int2 e_raw = ent[min((t + 2) >> 1, n_local - 1)];
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      if constexpr (HALF) {                // the stage is this wavefront's own: only its own reads have to be done
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
      } else {
        lds_barrier();                     // (waits for e_raw too)
      }
      if (t + 1 < steps) request(e_nxt, other);
      e_cur = e_nxt;
      e_nxt = half(e_raw, t);              // (t + 2 is as even as t)
      f32x16 sacc, pacc;
      bf16x8 dsf[2];
      bf16x8 tf[MB];
      scores(tile, sacc, pacc);
      first_half(tile, tf);
      probs(sacc, pacc, cnt, dsf);
      // the accumulating products run at low priority, scores and exp2 at high priority: with
      // two wavefronts per SIMD this helps to keep them in different parts of the step
      __builtin_amdgcn_s_setprio(0);
      accumulate(tile, tf, dsf);
      __builtin_amdgcn_s_setprio(3);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < steps; t += 2) {
      step(t, buf[0], buf[1]);
      step(t + 1, buf[1], buf[0]);
    }
  }

  // accumulator i of acc[mb] is channel 32 mb + 8 (i/4) + 4 kg + i%4 of the owner row
  if constexpr (SPLIT > 1) {
    // every pair leaves its sums where its tiles were; wavefront (slice, row half) adds and stores a
    // SPLIT-th of the row half's channels
    constexpr int NGRP = MB * 4, PER = NGRP / SPLIT;
    static_assert(NGRP * 64 == 2 * TILE && NGRP % SPLIT == 0, "a row half fills one tile buffer");
    __syncthreads();                          // no request is in flight: the last step makes none
    float4* const mine = reinterpret_cast<float4*>(buf[wave]);   // (wave: the row half within the workgroup)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        mine[(mb * 4 + g) * 64 + lane] =
            make_float4(acc[mb][4 * g + 0], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]);
    __syncthreads();
    if (!o_ok) return;
    uint16_t* op = a.out1 + (int64_t)h * a.o1_head + (int64_t)(otok0 + orow) * a.o1_tok;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int grp = slice * PER + p;
      float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int q2 = 0; q2 < SPLIT; ++q2) {
        const float4 v = reinterpret_cast<const float4*>(buf_all[q2][wave])[grp * 64 + lane];
        o[0] += v.x; o[1] += v.y; o[2] += v.z; o[3] += v.w;
      }
      bf16x4 o4;
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(o[e] * a.scale);
      *reinterpret_cast<bf16x4*>(op + 32 * (grp >> 2) + 8 * (grp & 3) + 4 * kg) = o4;
    }
    return;
  }
  if (o_ok) {
    uint16_t* op = a.out1 + (int64_t)h * a.o1_head + (int64_t)(otok0 + orow) * a.o1_tok;
    const float factor = a.scale;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(acc[mb][4 * g + e] * factor);
        *reinterpret_cast<bf16x4*>(op + 32 * mb + 8 * g + 4 * kg) = o4;
      }
  }
}

// dK and dV in one launch without computing the scores twice: a workgroup of four wavefronts
// owns one KV block and walks the query blocks that keep it in half tiles of 32 query rows.
// Wavefront i = (rh, role): rh = owner row half; role 0 computes S' = Q K^T, P' and
// dV^T += dO^T P'; role 1 computes dP' = dO V^T, dS' = P' (dP' - delta) and dK^T += Q^T dS'.
// P' goes from the role-0 wavefront to its role-1 partner (same rh: the same lanes hold the same
// elements) through LDS, and the partner uses it one step later, so the one barrier per step is
// enough; a tile therefore lives for two steps and the stage is triple-buffered.  Each wavefront
// keeps one owner operand and one accumulator set, which fits two wavefronts per SIMD (two
// workgroups per CU, not in step with each other).
constexpr int kKvThreads = 256;
// SPLIT = 2: a workgroup holds two such groups of four wavefronts, each with a stage of its own and half of
// the block's query blocks, and the sums are added through LDS: for calls with few KV blocks.  HALF: the workgroup
// owns one row half of the block, and a group is its two wavefronts.
template <int D, int SPLIT, bool HALF = false>
__global__ __launch_bounds__((HALF ? 128 : kKvThreads) * SPLIT, HALF ? 1 : D == 64 && SPLIT == 1 ? 3 : 2) void lf_attn_bwd_kv_kernel(BwdArgs a) {
  constexpr int WPG = HALF ? 2 : 4;         // wavefronts of a group
  constexpr int kGroupThreads = 64 * WPG;      // ... and their threads
  constexpr int CH = D / 8;
  constexpr int KS = D / 16;
  constexpr int MB = D / 32;
  constexpr int RPI = 64 / CH;              // tile rows one wavefront load instruction covers
  constexpr int LPW = 32 / (RPI * WPG);     // load instructions per wavefront, per tensor, per half tile
  constexpr int T32 = 32 * CH;              // uint4 per half tile (32 rows)
  static_assert(LPW == 1 || LPW == 2 || LPW == 4, "a half tile splits over the wavefronts of a group");

  __shared__ uint4 buf_all[SPLIT][3][2 * T32];   // [half tile mod 3][Q | dO]
  __shared__ float4 st_all[SPLIT][3][WPG][16];     // lse2 (role 0) or -delta (role 1) of the 32 streamed rows, one copy per
                                            // wavefront; its upper half takes the zeros of the lanes past the 32 rows
  __shared__ uint4 ph_all[SPLIT][2][WPG / 2][2][64];   // P' handoff: [step parity][row half][k-step][lane]
  __shared__ int2 ent_all[SPLIT][kPass];

  const int slot = (blockIdx.x & 7) * a.wg_per_xcd + (blockIdx.x >> 3);
  if ((HALF ? slot >> 1 : slot) >= a.total_wg) return;
  const int w = a.order[HALF ? slot >> 1 : slot];
  const int h = w / a.owners, r = w % a.owners;
  const int slice = SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kGroupThreads) : 0;
  uint4 (*const buf)[2 * T32] = buf_all[slice];
  float4 (*const st)[WPG][16] = st_all[slice];
  uint4 (*const ph)[WPG / 2][2][64] = ph_all[slice];
  int2* const ent = ent_all[slice];
  const int tid = threadIdx.x % kGroupThreads, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rh = HALF ? slot & 1 : wave & 1, pair = HALF ? 0 : rh;
  const bool is_ds = wave >= WPG / 2;       // role 1: dP', dS', dK
  const int ln = lane & 31, kg = lane >> 5;

  const int otok0 = (r / a.nb) * a.n + (r % a.nb) * 64;
  const int o_cnt = min(64, a.n - (r % a.nb) * 64);
  const int orow = 32 * rh + ln;
  const bool o_ok = orow < o_cnt;
  if (HALF && 32 * rh >= o_cnt) return;     // the other half of a short KV block
  // this group's slice of the list: entries [slice n_ent, +n_ent), of which my_ent exist
  const int n_all = a.cnt[(int64_t)h * a.owners + r];
  const int n_ent = (n_all + SPLIT - 1) / SPLIT;
  const int my_ent = SPLIT > 1 ? min(n_all - slice * n_ent, n_ent) : n_ent;
  const int32_t* list = a.idx + ((int64_t)h * a.owners + r) * a.list_stride + (SPLIT > 1 ? slice * n_ent : 0);

  // owner operand: K rows for role 0 (scores), V rows for role 1 (dP')
  Frag of[KS];
  {
    const uint16_t* op = is_ds ? a.Y + (int64_t)h * a.y_head + (int64_t)(otok0 + orow) * a.y_tok
                               : a.X + (int64_t)h * a.x_head + (int64_t)(otok0 + orow) * a.x_tok;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      of[s].u = o_ok ? *reinterpret_cast<const uint4*>(op + s * 16 + kg * 8) : make_uint4(0, 0, 0, 0);
  }

  const char* A1h = reinterpret_cast<const char*>(a.A1 + (int64_t)h * a.a1_head);
  const char* A2h = reinterpret_cast<const char*>(a.A2 + (int64_t)h * a.a2_head);
  const char* STh = reinterpret_cast<const char*>((is_ds ? a.ndelta : a.lse2) + (int64_t)h * a.q_len);
  const uint32_t a1_row_bytes = (uint32_t)(a.a1_tok * 2), a2_row_bytes = (uint32_t)(a.a2_tok * 2);

  // tile loads: wavefront `wave` fills its share of a half tile's rows with LPW instructions
  const int ld_r = lane / CH, ld_p = lane % CH;
  uint32_t off1[LPW], off2[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int row = RPI * (LPW * wave + i) + ld_r;
    off1[i] = (uint32_t)row * a1_row_bytes + (uint32_t)swz<CH>(row, ld_p) * 16u - 1024u * i;
    off2[i] = (uint32_t)row * a2_row_bytes + (uint32_t)swz<CH>(row, ld_p) * 16u - 1024u * i;
  }
  const uint32_t st_off = (uint32_t)lane * 4u;
  auto rsrc = [](const char* base, uint32_t row_bytes, int first, int count) {
    int32x4 rs;
    const uint64_t b = (uint64_t)base + (uint64_t)(uint32_t)first * row_bytes;
    rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    rs[2] = __builtin_amdgcn_readfirstlane((int)((uint32_t)count * row_bytes));
    rs[3] = 0x00020000;
    return rs;
  };
  auto fetch = [&](int32x4 rs, uint4* dst, const uint32_t (&off)[LPW]) __attribute__((always_inline)) {
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)LDS_PTR(void, dst + RPI * LPW * wave * CH));
    if constexpr (LPW == 4)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                   "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
                   "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
                   "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
                   :: "s"(lds0), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(rs) : "memory", "m0");
    else if constexpr (LPW == 2)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                   "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds"
                   :: "s"(lds0), "v"(off[0]), "v"(off[1]), "s"(rs) : "memory", "m0");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(lds0), "v"(off[0]), "s"(rs) : "memory", "m0");
  };
  // half tile t of the pass: list entry t/2 (given as read from `ent`), rows [32 (t&1), +32) of its block
  auto half = [&](int2 e, int t) {
    const int2 u = make_int2(__builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y));
    return (t & 1) ? make_int2(u.x + 32, max(u.y - 32, 0)) : make_int2(u.x, min(u.y, 32));
  };
  // half tile e -> its stage: the Q and dO rows and the row statistic of this wavefront's role
  auto request = [&](int2 e, int stage) __attribute__((always_inline)) {
    fetch(rsrc(A1h, a1_row_bytes, e.x, e.y), buf[stage], off1);
    fetch(rsrc(A2h, a2_row_bytes, e.x, e.y), buf[stage] + T32, off2);
    const int32x4 rs = rsrc(STh, 4u, e.x, e.y);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(void, st[stage][wave]));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dword %1, %2, 0 offen lds"
                 :: "s"(lds0), "v"(st_off), "s"(rs) : "memory", "m0");
  };

  int raddr[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) raddr[s] = ln * CH + swz<CH>(ln, 2 * s + kg);
  int tbase[MB];
  {
    const int i16 = lane & 15;
    const int tr_row = 4 * kg + (i16 >> 2);
    const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int col = 32 * mb + tr_col;
      tbase[mb] = (tr_row * CH + swz<CH>(tr_row, col >> 3)) * 8 + (col & 7);
    }
  }
  auto tfrag = [&](const uint4* tile, int u, int mb) __attribute__((always_inline)) {
    const uint16_t* p16 = reinterpret_cast<const uint16_t*>(tile);
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p16 + tbase[mb] + (16 * u) * CH * 8));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        LDS_PTR(bf16x4, p16 + (tbase[mb] ^ kTrHiFlip<CH>) + (16 * u + 8) * CH * 8));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  f32x16 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[mb][i] = 0.0f;
  f32x16 zero16;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero16[i] = 0.0f;

  // The parts of a step.  All LDS reads of a part are requested before the first matrix instruction that
  // needs one of them (the scheduling barriers pin that order; left alone the compiler keeps two to
  // four in flight and every matrix instruction waits for its operand).
  // Fragments of a tile's rows, and the score-like product: `c` + rows of the tile times the owner operand.
  auto rows_of = [&](const uint4* tile, Frag (&f)[KS]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < KS; ++s) f[s].u = tile[raddr[s]];
  };
  auto product = [&](const Frag (&f)[KS], f32x16 c) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < KS; ++s) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s].v, of[s].v, c, 0, 0, 0);
    return c;
  };
  // acc += tile^T (transposing reads) times b[0], b[1]; tf holds the fragments of the first 16 rows
  auto first_half = [&](const uint4* tile, bf16x8 (&tf)[MB]) __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) tf[mb] = tfrag(tile, 0, mb);
  };
  auto accumulate = [&](const uint4* tile, bf16x8 (&tf)[MB], const bf16x8 (&b)[2]) __attribute__((always_inline)) {
    bf16x8 t2[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) t2[mb] = tfrag(tile, 1, mb);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[mb], b[0], acc[mb], 0, 0, 0);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t2[mb], b[1], acc[mb], 0, 0, 0);
  };
  // accumulator i of a score tile is streamed row 8 (i/4) + 4 kg + i%4: the row statistics in
  // that order are four 16-byte reads.  Role 1 starts its product from them (dP' - delta needs no
  // subtraction then); a role reads only its own statistic (pairs of both took twice the LDS reads).
  auto stats16 = [&](int stage) __attribute__((always_inline)) {
    f32x16 v;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 x = st[stage][wave][2 * g + kg];
      v[4 * g] = x.x; v[4 * g + 1] = x.y; v[4 * g + 2] = x.z; v[4 * g + 3] = x.w;
    }
    return v;
  };

  for (int l0 = 0; l0 < n_ent; l0 += kPass) {
    const int n_local = min(n_ent - l0, kPass);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    for (int i = tid; i < n_local; i += kGroupThreads) {
      const int cidx = l0 + i < my_ent ? list[l0 + i] : -1;
      const bool ok = (unsigned)cidx < (unsigned)a.streams;
      const int tau = ok ? cidx / a.nb : 0, j = ok ? cidx % a.nb : 0;
      ent[i] = make_int2(tau * a.n + j * 64, ok ? min(64, a.n - j * 64) : 0);
    }
    __syncthreads();

    // Step t: half tile t is in stage t mod 3 (requested a step ago), half tile t-1 still in its
    // stage.  Role 0 works on t; role 1 forms dP' of t and finishes t-1 with the P' its partner
    // left during step t-1.  The first step has nothing to finish and the last one only finishes,
    // so they are peeled off and the loop body has no condition but the role.
    const int steps = 2 * n_local;
    f32x16 dp_prev = zero16;
    // role 0 on half tile t (stage cur, cnt rows): S', P' (handed over), dV^T += dO^T P'
    auto p_step = [&](int t, int cur, int cnt) __attribute__((always_inline)) {
      Frag f[KS];
      rows_of(buf[cur], f);
      const f32x16 lse = stats16(cur);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 sacc = product(f, zero16);
      bf16x8 tf[MB];
      first_half(buf[cur] + T32, tf);
      __builtin_amdgcn_sched_barrier(0);
      // stream rows past a short half tile's count were loaded as zeros (scores and statistics
      // alike): their scores become -inf (P' = 0); a full half tile, the common case, skips this
      if (cnt < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + 4 * kg + (i & 3) >= cnt) sacc[i] = -INFINITY;
      }
      bf16x8 pf[2];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        pf[i >> 3][i & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sacc[i], a.c, -lse[i]));
      ph[t & 1][pair][0][lane] = __builtin_bit_cast(uint4, pf[0]);
      ph[t & 1][pair][1][lane] = __builtin_bit_cast(uint4, pf[1]);
      accumulate(buf[cur] + T32, tf, pf);
    };
    // role 1 finishing half tile t (stage prv): dS' = P' (dP' - delta), dK^T += Q^T dS'; dp_prev holds
    // dP' - delta, pu the P' its partner left, tf the first transposed fragments of Q
    auto ds_finish = [&](int prv, const uint4 (&pu)[2], bf16x8 (&tf)[MB]) __attribute__((always_inline)) {
      bf16x8 dsf[2];
      const bf16x8 pf[2] = {__builtin_bit_cast(bf16x8, pu[0]), __builtin_bit_cast(bf16x8, pu[1])};
#pragma unroll
      for (int i = 0; i < 16; ++i) dsf[i >> 3][i & 7] = (__bf16)((float)pf[i >> 3][i & 7] * dp_prev[i]);
      accumulate(buf[prv], tf, dsf);
    };
    auto take_p = [&](int t, uint4 (&pu)[2]) __attribute__((always_inline)) {
      pu[0] = ph[t & 1][pair][0][lane];
      pu[1] = ph[t & 1][pair][1][lane];
    };
    // e_cur, e_nxt: half tiles t and t + 1; that of t + 2 is looked up a step ahead
    int2 e_cur = half(ent[0], 0), e_nxt = half(ent[0], 1);
    request(e_cur, 0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    lds_barrier();
    request(e_nxt, 1);                     // steps >= 2: a list entry is two half tiles
    if (!is_ds) {
      p_step(0, 0, e_cur.y);
    } else {
      Frag f[KS];
      dp_prev = stats16(0);
      rows_of(buf[0] + T32, f);
      dp_prev = product(f, dp_prev);
    }
    // stages of step t: cur = t mod 3, nxt = t + 1 mod 3, prv = t + 2 mod 3, constants in a loop of three steps
    auto step = [&](int t, int cur, int nxt, int prv) __attribute__((always_inline)) {
      e_cur = e_nxt;
      const int2 e_raw = ent[min(t + 1, steps - 1) >> 1];
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      lds_barrier();                       // (waits for e_raw too)
      if (t + 1 < steps) {
        e_nxt = half(e_raw, t + 1);
        request(e_nxt, nxt);
      }
      if (!is_ds) {
        p_step(t, cur, e_cur.y);
      } else {
        Frag f[KS];
        uint4 pu[2];
        f32x16 dp_cur = stats16(cur);
        rows_of(buf[cur] + T32, f);
        take_p(t - 1, pu);
        __builtin_amdgcn_sched_barrier(0);
        dp_cur = product(f, dp_cur);       // dP' - delta of half tile t
        bf16x8 tf[MB];
        first_half(buf[prv], tf);
        __builtin_amdgcn_sched_barrier(0);
        ds_finish(prv, pu, tf);
        dp_prev = dp_cur;
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 1; t < steps; t += 3) {
      step(t, 1, 2, 0);
      if (t + 1 >= steps) break;
      step(t + 1, 2, 0, 1);
      if (t + 2 >= steps) break;
      step(t + 2, 0, 1, 2);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    lds_barrier();
    if (is_ds) {
      uint4 pu[2];
      bf16x8 tf[MB];
      const int prv = (steps - 1) % 3;
      take_p(steps - 1, pu);
      first_half(buf[prv], tf);
      ds_finish(prv, pu, tf);
    }
  }

  // accumulator i of acc[mb] is channel 32 mb + 8 (i/4) + 4 kg + i%4 of the owner row
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  if constexpr (SPLIT > 1) {
    // the second group leaves its sums where both groups' tiles were, the first adds them to its own
    constexpr int NGRP = MB * 4;
    static_assert(SPLIT == 2 && WPG * NGRP * 64 <= 2 * 3 * 2 * T32, "the sums of a group fit the stages");
    float4* const sums = reinterpret_cast<float4*>(buf_all) + wave * NGRP * 64;
    __syncthreads();
    if (slice == 1) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          sums[(mb * 4 + g) * 64 + lane] =
              make_float4(acc[mb][4 * g + 0], acc[mb][4 * g + 1], acc[mb][4 * g + 2], acc[mb][4 * g + 3]);
    }
    __syncthreads();
    if (slice == 1) return;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 v = sums[(mb * 4 + g) * 64 + lane];
        acc[mb][4 * g + 0] += v.x; acc[mb][4 * g + 1] += v.y;
        acc[mb][4 * g + 2] += v.z; acc[mb][4 * g + 3] += v.w;
      }
  }
  if (o_ok) {
    uint16_t* op = is_ds ? a.out1 + (int64_t)h * a.o1_head + (int64_t)(otok0 + orow) * a.o1_tok
                         : a.out2 + (int64_t)h * a.o2_head + (int64_t)(otok0 + orow) * a.o2_tok;
    const float factor = is_ds ? a.scale : 1.0f;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(acc[mb][4 * g + e] * factor);
        *reinterpret_cast<bf16x4*>(op + 32 * mb + 8 * g + 4 * kg) = o4;
      }
  }
}

// What the two gradient launches need beforehand, in one launch: the first workgroups make the transposed
// lists, the others delta.  The former wait for dependent loads, the latter stream O and dO (on the
// last-chunk call 10 and 7 us and a gap apart, 15 us together).  With the launch order beside the dQ
// launch a backward call is three launches instead of five: small ragged training step 79.7 -> 74.0 us.
struct PrepArgs {
  const int32_t* idx;
  int32_t* tlist;
  int32_t* tcnt;
  const uint16_t* O;
  const uint16_t* dO;
  float* ndelta;
  int64_t o_tok, o_head;
  int heads, n_q, n_k, list_len, q_len, rows, tr_blocks;
};

// Transposed lists: for every (head, KV block c) the query blocks whose list holds c, ascending.
// One wavefront per (head, c): lane i looks c up in the list of query block r0 + i by bisection
// (lists are ascending), and the hits of the 64 lanes are compacted in order through a ballot.
__device__ __forceinline__ void transpose_lists(const PrepArgs& a, int gid) {
  if (gid >= a.heads * a.n_k) return;
  const int lane = threadIdx.x & 63;
  const int h = gid / a.n_k, c = gid % a.n_k;
  int32_t* out = a.tlist + (int64_t)gid * a.n_q;
  int cnt = 0;
  for (int r0 = 0; r0 < a.n_q; r0 += 64) {
    const int r = r0 + lane;
    bool hit = false;
    if (r < a.n_q) {
      const int32_t* l = a.idx + ((int64_t)h * a.n_q + r) * a.list_len;
      int lo = 0, hi = a.list_len;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (l[mid] < c) lo = mid + 1; else hi = mid;
      }
      hit = lo < a.list_len && l[lo] == c;
    }
    const uint64_t m = __ballot(hit);
    if (hit) out[cnt + __popcll(m & ((1ull << lane) - 1))] = r;
    cnt += __popcll(m);
  }
  if (lane == 0) a.tcnt[gid] = cnt;
}

template <int D>
__global__ __launch_bounds__(256) void lf_attn_bwd_prep_kernel(PrepArgs a) {
  if ((int)blockIdx.x < a.tr_blocks) {
    transpose_lists(a, blockIdx.x * 4 + (threadIdx.x >> 6));
    return;
  }
  // -delta_x, delta_x = dO_x . O_x (float32), one group of d/8 lanes per row
  constexpr int LPR = D / 8;                  // lanes per row
  const int gid = (blockIdx.x - a.tr_blocks) * 256 + threadIdx.x;
  const int row = gid / LPR, ch = gid % LPR;
  float s = 0.0f;
  if (row < a.rows) {
    const int h = row / a.q_len, x = row % a.q_len;
    const int64_t off = (int64_t)h * a.o_head + (int64_t)x * a.o_tok + ch * 8;
    const uint4 u = *reinterpret_cast<const uint4*>(a.O + off), v = *reinterpret_cast<const uint4*>(a.dO + off);
    const uint32_t uu[4] = {u.x, u.y, u.z, u.w}, vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s = fmaf(__uint_as_float(uu[i] << 16), __uint_as_float(vv[i] << 16), s);
      s = fmaf(__uint_as_float(uu[i] & 0xffff0000u), __uint_as_float(vv[i] & 0xffff0000u), s);
    }
  }
#pragma unroll
  for (int o = 1; o < LPR; o <<= 1) s += __shfl_xor(s, o);
  if (row < a.rows && ch == 0) a.ndelta[row] = -s;
}

// The step of the launch order: the number nearest below 0.618 n that is prime to n (1 for n < 3).
uint32_t spread_step(uint32_t n) {
  uint32_t s = (uint32_t)(0.6180339887 * n);
  for (; s > 1; --s) {
    uint32_t a = n, b = s;
    while (b) { const uint32_t t = a % b; a = b; b = t; }
    if (a == 1) break;
  }
  return s > 1 ? s : 1;
}

}  // namespace

int lf_launch_attn_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                       const float* lse2, const lf_shape* s, const lf_dims* dm, const int32_t* indices,
                       int32_t list_len, float scale, void* dQ, void* dK, void* dV, float* ndelta,
                       int32_t* tlist, int32_t* tcnt, int32_t* order, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int q_len = dm->f * dm->n;
  {
    PrepArgs p;
    p.idx = indices;
    p.tlist = tlist;
    p.tcnt = tcnt;
    p.O = (const uint16_t*)O;
    p.dO = (const uint16_t*)dO;
    p.ndelta = ndelta;
    p.o_tok = s->o_stride_tok;
    p.o_head = s->o_stride_head;
    p.heads = dm->H;
    p.n_q = dm->n_q;
    p.n_k = dm->n_k;
    p.list_len = list_len;
    p.q_len = q_len;
    p.rows = dm->H * q_len;
    p.tr_blocks = (dm->H * dm->n_k + 3) / 4;
    const unsigned grid = (unsigned)(p.tr_blocks + (p.rows * (dm->d / 8) + 255) / 256);
    const hipError_t rc = dm->d == 128 ? lf_launch(lf_attn_bwd_prep_kernel<128>, dim3(grid), dim3(256), 0, st, p)
                                       : lf_launch(lf_attn_bwd_prep_kernel<64>, dim3(grid), dim3(256), 0, st, p);
    if (rc != hipSuccess) return LF_ERR_HIP;
  }
  BwdArgs a = {};
  a.lse2 = lse2;
  a.ndelta = ndelta;
  a.n = dm->n;
  a.nb = dm->nb;
  a.q_len = q_len;
  a.c = scale * 1.4426950408889634f;
  a.scale = scale;
  // dQ
  a.X = (const uint16_t*)Q;   a.x_tok = s->q_stride_tok;  a.x_head = s->q_stride_head;
  a.Y = (const uint16_t*)dO;  a.y_tok = s->o_stride_tok;  a.y_head = s->o_stride_head;
  a.A1 = (const uint16_t*)K;  a.a1_tok = s->k_stride_tok; a.a1_head = s->k_stride_head;
  a.A2 = (const uint16_t*)V;  a.a2_tok = s->v_stride_tok; a.a2_head = s->v_stride_head;
  a.out1 = (uint16_t*)dQ;     a.o1_tok = s->q_stride_tok; a.o1_head = s->q_stride_head;
  a.out2 = nullptr;
  a.idx = indices; a.cnt = nullptr; a.list_len = list_len; a.list_stride = list_len;
  a.owners = dm->n_q; a.streams = dm->n_k;
  a.total_wg = dm->H * dm->n_q;
  a.wg_per_xcd = (a.total_wg + 7) / 8;
  const lf_form dq_form = lf_dq_form(dm->d, a.total_wg, list_len);
  const bool halve = dq_form == LF_FORM_HALVES;
  const int parts = dq_form == LF_FORM_TWO ? 2 : dq_form == LF_FORM_FOUR ? 4 : 1;
  if (halve) {
    a.total_wg *= 2;
    a.wg_per_xcd = (a.total_wg + 7) / 8;
  }
  a.order = order;
  a.order_cnt = tcnt;
  a.order_n_k = dm->n_k;
  a.order_total = dm->H * dm->n_k;
  a.order_per_xcd = (a.order_total + 7) / 8;
  a.order_step = spread_step((uint32_t)dm->n_k);
  // eight workgroups in front for the order of the next launch
  hipError_t rc;
  if (dq_form == LF_FORM_WIDE) {
    a.order_stride = (uint32_t)((uint64_t)64 * a.order_step % (uint32_t)dm->n_k);
    rc = lf_launch_attn_bwd_q_wide(a, st);
  } else {
    const dim3 grid1((unsigned)(a.wg_per_xcd * 8 + 8)), block1((unsigned)(halve ? (dm->d == 128 ? 256 : 512) : parts * kThreads));
    a.order_stride = (uint32_t)((uint64_t)block1.x * a.order_step % (uint32_t)dm->n_k);
    rc = dm->d == 128
        ? lf_launch(halve ? lf_attn_bwd_q_kernel<128, 4, true> : parts == 4 ? lf_attn_bwd_q_kernel<128, 4>
                    : parts == 2 ? lf_attn_bwd_q_kernel<128, 2> : lf_attn_bwd_q_kernel<128, 1>, grid1, block1, 0, st, a)
        : lf_launch(halve ? lf_attn_bwd_q_kernel<64, 8, true> : parts == 4 ? lf_attn_bwd_q_kernel<64, 4>
                    : parts == 2 ? lf_attn_bwd_q_kernel<64, 2> : lf_attn_bwd_q_kernel<64, 1>, grid1, block1, 0, st, a);
  }
  if (rc != hipSuccess) return LF_ERR_HIP;
  // dK and dV
  a.X = (const uint16_t*)K;   a.x_tok = s->k_stride_tok;  a.x_head = s->k_stride_head;
  a.Y = (const uint16_t*)V;   a.y_tok = s->v_stride_tok;  a.y_head = s->v_stride_head;
  a.A1 = (const uint16_t*)Q;  a.a1_tok = s->q_stride_tok; a.a1_head = s->q_stride_head;
  a.A2 = (const uint16_t*)dO; a.a2_tok = s->o_stride_tok; a.a2_head = s->o_stride_head;
  a.out1 = (uint16_t*)dK;     a.o1_tok = s->k_stride_tok; a.o1_head = s->k_stride_head;
  a.out2 = (uint16_t*)dV;     a.o2_tok = s->v_stride_tok; a.o2_head = s->v_stride_head;
  a.idx = tlist; a.cnt = tcnt; a.list_len = dm->n_q; a.list_stride = dm->n_q;
  a.owners = dm->n_k; a.streams = dm->n_q;
  a.total_wg = dm->H * dm->n_k;
  a.wg_per_xcd = (a.total_wg + 7) / 8;
  const lf_kv_form form = lf_kv_form_of(dm->d, a.total_wg, list_len, dm->n_q, dm->n_k);
  if (form == LF_KV_HALVES) {
    a.wg_per_xcd *= 2;     // both halves of a block on the XCD its place in the order belongs to
    const dim3 grid((unsigned)(a.wg_per_xcd * 8));
    rc = dm->d == 128 ? lf_launch(lf_attn_bwd_kv_kernel<128, 2, true>, grid, dim3(2 * 128), 0, st, a)
                      : lf_launch(lf_attn_bwd_kv_kernel<64, 2, true>, grid, dim3(2 * 128), 0, st, a);
    return rc == hipSuccess ? LF_OK : LF_ERR_HIP;
  }
  const dim3 grid2((unsigned)(a.wg_per_xcd * 8));
  const bool groups = form == LF_KV_GROUPS;
  if (form == LF_KV_WIDE) return lf_launch_attn_bwd_kv_wide(a, st) == hipSuccess ? LF_OK : LF_ERR_HIP;
  const dim3 block2((unsigned)(groups ? 2 * kKvThreads : kKvThreads));
  rc = dm->d == 64 ? lf_launch(lf_attn_bwd_kv_kernel<64, 1>, grid2, block2, 0, st, a)
       : groups    ? lf_launch(lf_attn_bwd_kv_kernel<128, 2>, grid2, block2, 0, st, a)
                   : lf_launch(lf_attn_bwd_kv_kernel<128, 1>, grid2, block2, 0, st, a);
  return rc == hipSuccess ? LF_OK : LF_ERR_HIP;
}
