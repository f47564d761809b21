// dQ of the blockwise sparse attention at head dimension 128, one wavefront per query block.
#include "lf_attn_bwd.h"
#include "lf_slots.h"

namespace {

// What bounds it: instruction issue of the one wavefront that a SIMD holds, and with the chip full the LDS.  The kernel with two
// wavefronts per query block reads a tile's fragments once per 32 query rows, this one once per 64, and its tiles are its own, so
// no barrier stands in the loop.  A window (half tile) is 48 slots of one matrix instruction (32 cycles) each, in which the other
// instructions have to fit: they are inline assembly, which keeps its place, as are the products (as builtins they are moved
// together: window 2 180 cycles, 1 980 as written here; the products alone take 1 536).  An instruction costs its four cycles of
// issue whatever it does, so the loads go one to a slot behind a product, M0 is written once per four of them, and what the
// compiler would put at the loop's end (places, entries) is moved inside.  The fragments and Q, dO and dQ fill the
// register file (255 + 256, nothing spilled): the list's entries are in registers and LDS holds tiles only.
// The compiler does not see the latency of the products: results are read at least two products after the last one into them
// (scores: slots 21 and 22, read from slots 0 and 2 of the next phase on).
// 12 x 128, 4 680 queries, 32 760 keys, lists of 188: dQ and the launch before it 518 -> 491 us, of 45 (4 680 keys) 153 -> 142;
// by the loop without its loads 13 % of that would go, without its LDS reads 15 %, without both 27 %.
constexpr int kQWideEnt = 256;     // half tiles decoded per pass: four registers, one entry a lane
constexpr int lgkmcnt_imm(int n) { return 15 | (3 << 14) | (7 << 4) | (n << 8); }
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(64, 1) void lf_attn_bwd_q_wide_kernel(BwdArgs a) {
  constexpr int D = 128, CH = D / 8, KS = D / 16, MB = D / 32;
  constexpr int T32 = 32 * CH;              // uint4 per half tile: 8 KB
  constexpr uint32_t kTile = T32 * 16u;
  struct alignas(1024) Stage {
    uint4 k[3][T32], v[2][T32];             // half tile mod 3 and mod 2
  };
  __shared__ Stage st;                      // 40 KB: four workgroups share a compute unit

  if (blockIdx.x < 8) {
    static_assert(sizeof(st) >= kOrderBins * sizeof(int), "the order's bins use the tile stage");
    order_share(a, blockIdx.x, reinterpret_cast<int*>(&st));
    return;
  }
  const int w = (blockIdx.x & 7) * a.wg_per_xcd + (blockIdx.x >> 3) - 1;
  if (w >= a.total_wg) return;
  const int h = w / a.owners, r = w % a.owners;
  const int lane = threadIdx.x & 63, ln = lane & 31, kg = lane >> 5;
  const int otok0 = (r / a.nb) * a.n + (r % a.nb) * 64;
  const int o_cnt = min(64, a.n - (r % a.nb) * 64);
  const int32_t* list = a.idx + ((int64_t)h * a.owners + r) * a.list_stride;

  // Owner rows (B operands): Q and dO.  A row past a short block's end gets a log-sum-exp of +inf: its probabilities are zero.
  bf16x8 xf[2][KS], yf[2][KS];
  float lse[2], nd[2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int row = 32 * hh + ln;
    const uint16_t* xp = a.X + (int64_t)h * a.x_head + (int64_t)(otok0 + row) * a.x_tok;
    const uint16_t* yp = a.Y + (int64_t)h * a.y_head + (int64_t)(otok0 + row) * a.y_tok;
    lse[hh] = INFINITY;
    nd[hh] = 0.0f;
    if (row < o_cnt) {
      lse[hh] = a.lse2[(int64_t)h * a.q_len + otok0 + row];
      nd[hh] = a.ndelta[(int64_t)h * a.q_len + otok0 + row];
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      uint4 u = make_uint4(0, 0, 0, 0), v = make_uint4(0, 0, 0, 0);
      if (row < o_cnt) {
        u = *reinterpret_cast<const uint4*>(xp + s * 16 + kg * 8);
        v = *reinterpret_cast<const uint4*>(yp + s * 16 + kg * 8);
      }
      xf[hh][s] = __builtin_bit_cast(bf16x8, u);
      yf[hh][s] = __builtin_bit_cast(bf16x8, v);
    }
  }
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" : "+a"(xf[hh][s]), "+a"(yf[hh][s]));

  // Tile loads, global -> LDS, a quarter block (16 rows) at a time: load i fills rows [4 i, +4) of it; the buffer resource is the
  // quarter itself, so rows past the tile's count read as zeros, and both quarters of a half tile use the same four offsets.
  const char* Kh = reinterpret_cast<const char*>(a.A1 + (int64_t)h * a.a1_head);
  const char* Vh = reinterpret_cast<const char*>(a.A2 + (int64_t)h * a.a2_head);
  const uint32_t k_pitch = (uint32_t)(a.a1_tok * 2), v_pitch = (uint32_t)(a.a2_tok * 2);
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(void, &st));
  // quarter q of half tile e (entry); one head's K or V spans less than 2 GiB.  Made by scalar instructions alone: a load behind a
  // vector instruction that writes its resource would have to wait for it (five wait states, which nobody counts into assembly).
  auto rsrc = [](const char* base, uint32_t pitch, uint32_t e, int q) {
    int32x4 rs;
    const uint64_t b = (uint64_t)base + (uint64_t)(((e >> 6) + 16u * q) * pitch);
    uint32_t cnt = e & 63u;
    if (q) {
      asm("s_max_u32 %0, %1, 16" : "=s"(cnt) : "s"(cnt) : "scc");
      cnt -= 16u;
    }
    rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    rs[2] = __builtin_amdgcn_readfirstlane((int)(cnt * pitch));
    rs[3] = 0x00020000;
    return rs;
  };
  auto fetch4 = [&](int32x4 rs, uint32_t lds0, const uint32_t* o) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
                 :: "s"(lds0), "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]), "s"(rs) : "memory", "m0");
  };
  const uint32_t k_lds = lds_base, v_lds = lds_base + 3 * kTile;
  auto request = [&](const char* base, uint32_t pitch, uint32_t e, uint32_t lds0, const uint32_t* o) __attribute__((always_inline)) {
    fetch4(rsrc(base, pitch, e, 0), lds0, o);
    fetch4(rsrc(base, pitch, e, 1), lds0 + kTile / 2, o);
  };
  auto flipped = [](uint32_t base, uint32_t bits) __attribute__((always_inline)) {   // in the slot it is written in
    uint32_t at;
    asm volatile("v_xor_b32 %0, %1, %2" : "=v"(at) : "s"(bits), "v"(base));
    return at;
  };
  auto row_frag = [&](uint32_t base, int s) __attribute__((always_inline)) {
    const uint32_t at = s == 0 ? base : flipped(base, 32u * s);
    return __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4*)at);
  };
  auto tread = [&](uint32_t at, int u, int hf) __attribute__((always_inline)) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(at + (16u * u + 8u * hf) * CH * 16u));
  };
  auto moved = [](uint32_t& to, const uint32_t& from) __attribute__((always_inline)) { asm volatile("s_mov_b32 %0, %1" : "=s"(to) : "s"(from)); };
  auto join = [](const bf16x4& lo, const bf16x4& hi) { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7); };
  // c += x y, held in the accumulation registers
  auto accumulate = [](f32x16& c, const bf16x8& x, const bf16x8& y) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
  };
  // scores: c = x y from zero, from c0, and c += x y, in registers that vector instructions reach
  auto mfma_zero = [](f32x16& c, const bf16x8& x, const bf16x8& y) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(x), "a"(y));
  };
  auto mfma_from = [](f32x16& c, const bf16x8& x, const bf16x8& y, const f32x16& c0) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(c) : "v"(x), "a"(y), "v"(c0));
  };
  auto mfma = [](f32x16& c, const bf16x8& x, const bf16x8& y) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(x), "a"(y));
  };

  f32x16 acc[2][MB];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[hh][mb][i] = 0.0f;

  for (int l0 = 0; l0 < a.list_len; l0 += kQWideEnt / 2) {
    const int l1 = min(a.list_len, l0 + kQWideEnt / 2);
    // Decode: entries -> half tiles, back to back, through the tile stage (no load is in flight) into four registers.
    uint32_t* const ent = reinterpret_cast<uint32_t*>(&st);
    uint32_t er[kQWideEnt / 64];
#pragma unroll
    for (int j = 0; j < kQWideEnt / 64; ++j) ent[64 * j + lane] = 0;
    int nt = 0;
#pragma unroll
    for (int j = 0; j < kQWideEnt / 128; ++j) {
      const int i = l0 + 64 * j + lane;
      const int c = i < l1 ? list[i] : -1;
      const bool ok = (unsigned)c < (unsigned)a.streams;
      const int tau = ok ? c / a.nb : 0, b = ok ? c % a.nb : 0;
      const uint32_t tok = (uint32_t)(tau * a.n + b * 64);
      const int cnt = ok ? min(64, a.n - b * 64) : 0;
      const unsigned long long one = __ballot(cnt > 0), two = __ballot(cnt > 32);
      const unsigned long long below = (1ull << lane) - 1ull;
      const int pos = nt + __popcll(one & below) + __popcll(two & below);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      if (cnt > 0) ent[pos] = tok << 6 | (uint32_t)min(cnt, 32);
      if (cnt > 32) ent[pos + 1] = (tok + 32) << 6 | (uint32_t)(cnt - 32);
      nt += __popcll(one) + __popcll(two);
    }
    nt = __builtin_amdgcn_readfirstlane(nt);
    if (nt == 0) continue;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
#pragma unroll
    for (int j = 0; j < kQWideEnt / 64; ++j) er[j] = ent[64 * j + lane];
    __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(0));
    asm volatile("" : "+v"(er[0]), "+v"(er[1]), "+v"(er[2]), "+v"(er[3]) :: "memory");
    // What depends on the lane alone is made in every pass (at_lane hides that it does not change): kept over the whole kernel it
    // is spilled.  Load offsets; LDS addresses of this lane's fragments in a tile, one register each, flipped where read: rows (chunk
    // 2 s + kg of row ln; s flips address bits 5 to 7), and the transposing reads (mb flips bits 6 and 7, the upper eight rows bit 5).
    int at_lane = lane;
    asm volatile("" : "+v"(at_lane));
    uint32_t koff[4], voff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * i + (at_lane >> 4);
      const uint32_t at = (uint32_t)swz<CH>(row, at_lane & 15) * 16u - 1024u * i;
      koff[i] = (uint32_t)row * k_pitch + at;
      voff[i] = (uint32_t)row * v_pitch + at;
    }
    const uint32_t row_at = 16u * ((at_lane & 31) * CH + swz<CH>(at_lane & 31, at_lane >> 5));
    uint32_t tr_at;
    {
      const int i16 = at_lane & 15;
      const int tr_row = 4 * (at_lane >> 5) + (i16 >> 2);
      const int tr_col = 16 * ((at_lane >> 4) & 1) + 4 * (i16 & 3);
      tr_at = 2u * ((tr_row * CH + swz<CH>(tr_row, tr_col >> 3)) * 8 + (tr_col & 7));
    }
    // half tiles t .. t + 3 (empty ones past the end)
    uint32_t e0 = __builtin_amdgcn_readlane(er[0], 0), e1 = __builtin_amdgcn_readlane(er[0], 1);
    uint32_t e2 = __builtin_amdgcn_readlane(er[0], 2), e3 = __builtin_amdgcn_readlane(er[0], 3);

    bf16x8 rk[KS], rv[KS];             // row fragments of K and V
    bf16x4 tlo[2 * MB], thi[2 * MB];   // transposed fragments of K
    f32x16 sc[2], dp[2], nd16[2];      // S' and dP' - delta, what the latter starts from: [owner half]
#pragma unroll
    for (int i = 0; i < 16; ++i) { nd16[0][i] = nd[0]; nd16[1][i] = nd[1]; }
    u32x4 pk[2][2];                    // dS', packed: [owner half][k-step]
    float x[2], ee[2], m[2];
    // rows past a short half tile's count were loaded as zeros: their scores become -inf (P' = 0)
    auto mask = [&](int hh, int cnt) __attribute__((always_inline)) {
      if (cnt < 32) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + 4 * kg + (i & 3) >= cnt) sc[hh][i] = -INFINITY;
      }
    };
    // Slot i of a phase: value v of owner half hh is scaled in slot v, exp2 in slot v + 1, multiplied by dP' - delta in slot
    // v + 2.  The empty statements keep the vector instructions in their slots: they are only needed a phase later.
    auto soft = [&](int i, int hh) __attribute__((always_inline)) {
      // values start in slots 0, 1, 2, 4, 5, 7, ..., 21
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int at = v * 7 / 5;
        if (i == at + 2) {
          if (v & 1)
            asm volatile("v_mul_f32 %1, %2, %3\n\tv_cvt_pk_bf16_f32 %0, %4, %1"
                         : "=v"(pk[hh][v >> 3][(v & 7) >> 1]), "=&v"(m[1]) : "v"(ee[1]), "v"(dp[hh][v]), "v"(m[0]));
          else
            asm volatile("v_mul_f32 %0, %1, %2" : "=v"(m[0]) : "v"(ee[0]), "v"(dp[hh][v]));
        }
        if (i == at + 1) {
          asm volatile("v_exp_f32 %0, %1" : "=v"(ee[v & 1]) : "v"(x[v & 1]));
        }
        if (i == at) {
          asm volatile("v_fma_f32 %0, %1, %2, -%3" : "=v"(x[v & 1]) : "v"(sc[hh][v]), "s"(a.c), "v"(lse[hh]));
        }
      }
    };
    request(Kh, k_pitch, e0, k_lds + 0 * kTile, koff);
    request(Vh, v_pitch, e0, v_lds + 0 * kTile, voff);
    request(Kh, k_pitch, e1, k_lds + 1 * kTile, koff);
    request(Vh, v_pitch, e1, v_lds + 1 * kTile, voff);
    request(Kh, k_pitch, e2, k_lds + 2 * kTile, koff);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(24));       // half tile 0 has landed
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      rk[s] = row_frag(k_lds + row_at, s);
      rv[s] = row_frag(v_lds + row_at, s);
    }
    __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(0));
    __builtin_amdgcn_sched_barrier(0);
    request(Vh, v_pitch, e2, v_lds + 0 * kTile, voff);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s == 0) mfma_zero(sc[0], rk[s], xf[0][s]);
      else mfma(sc[0], rk[s], xf[0][s]);
      if (s == 0) mfma_from(dp[0], rv[s], yf[0][s], nd16[0]);
      else mfma(dp[0], rv[s], yf[0][s]);
    }
#pragma unroll
    for (int f = 0; f < 2 * MB; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) tlo[f][e] = thi[f][e] = (__bf16)0.0f;
    pk[1][0] = pk[1][1] = u32x4{0u, 0u, 0u, 0u};
    asm volatile("s_nop 15" : "+v"(sc[0]));
    mask(0, (int)(e0 & 63u));
    __builtin_amdgcn_sched_barrier(0);

    // Window t, two phases of 24 slots, one matrix instruction each, S', dP' and dQ in turn.  Phase 0: dS' of (t, half 0) beside the
    // scores of (t, half 1) and dQ of (t - 1, half 1), whose fragments are replaced as they are used; phase 1: dS' of (t, half 1)
    // beside the scores of (t + 1, half 0), dQ of (t, half 0) and the requests of half tile t + 3.
    // Places: K of t (taken over by t + 3), of t + 1, the third; V of t + 1 (taken over by t + 3), of t + 2.
    uint32_t kp = k_lds, kn = k_lds + kTile, kf = k_lds + 2 * kTile, vp = v_lds + kTile, vn = v_lds;
    constexpr int kEarly = 4;          // row fragments replaced in phase 0, the others in phase 1
    constexpr int kKeep = 4;           // ... of which this many reads are in flight when those of K's tile must be done
    for (int t = 0; t < nt; ++t) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(16));     // half tile t + 1 has landed
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      uint32_t tr[2 * MB];
      const uint32_t k_rows = kn + row_at, v_rows = vp + row_at, k_tr = kp + tr_at;
#pragma unroll
      for (int i = 0; i < 24; ++i) {
        const int k = i / 3;
        soft(i, 0);
        if (i % 3 == 0) {
          if (k == 0) mfma_zero(sc[1], rk[k], xf[1][k]);
          else mfma(sc[1], rk[k], xf[1][k]);
          if (k < kEarly) rk[k] = row_frag(k_rows, k);
        } else if (i % 3 == 1) {
          if (k == 0) mfma_from(dp[1], rv[k], yf[1][k], nd16[1]);
          else mfma(dp[1], rv[k], yf[1][k]);
          if (k < kEarly) rv[k] = row_frag(v_rows, k);
        } else {
          accumulate(acc[1][k % MB], join(tlo[k], thi[k]), __builtin_bit_cast(bf16x8, pk[1][k / MB]));
          if (k < MB) {
            tr[k] = k == 0 ? k_tr : flipped(k_tr, 64u * k);
            tr[MB + k] = flipped(k_tr, (64u * k) ^ (2u * kTrHiFlip<CH>));
          }
          tlo[k] = tread(tr[k % MB], k / MB, 0);
          thi[k] = tread(tr[MB + k % MB], k / MB, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      mask(1, (int)(e0 & 63u));
      int32x4 rs;
      uint32_t kt;
      if (((t + 4) & 63) == 0) {                     // the next 64 entries
        er[0] = er[1]; er[1] = er[2]; er[2] = er[3]; er[3] = 0;
        asm volatile("" : "+v"(er[0]));
      }
      const uint32_t e4 = __builtin_amdgcn_readlane(er[0], (t + 4) & 63);
      __builtin_amdgcn_sched_barrier(0);
      auto slot = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, k = i / 3;
        soft(i, 1);
        if constexpr (i < 2 * (KS - kEarly)) {
          if constexpr (i == kKeep) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(kKeep));   // all reads of this half tile of K are done
          if constexpr (i & 1) rv[kEarly + i / 2] = row_frag(v_rows, kEarly + i / 2);
          else rk[kEarly + i / 2] = row_frag(k_rows, kEarly + i / 2);
        }
        if constexpr (i == 12) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(0));            // ... and of the next of V
        if constexpr (i >= 5 && i < 21) {
          constexpr int l = i - 5, j = l & 3;
          if constexpr (j == 0) rs = l < 8 ? rsrc(Kh, k_pitch, e3, l >> 2) : rsrc(Vh, v_pitch, e3, (l >> 2) - 2);
          const uint32_t lds0 = (l < 8 ? kp : vp) + (l & 4 ? kTile / 2 : 0);
          const uint32_t o = l < 8 ? koff[j] : voff[j];
          if constexpr (i % 3 == 0) { LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+v", sc[0], rk[k], "a", xf[0][k], rs, lds0, o, j) }
          else if constexpr (i % 3 == 1) { LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+v", dp[0], rv[k], "a", yf[0][k], rs, lds0, o, j) }
          else { LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+a", acc[0][k % MB], join(tlo[k], thi[k]), "v",
                         __builtin_bit_cast(bf16x8, pk[0][k / MB]), rs, lds0, o, j) }
        } else {
          if constexpr (i == 0) mfma_zero(sc[0], rk[k], xf[0][k]);
          else if constexpr (i == 1) mfma_from(dp[0], rv[k], yf[0][k], nd16[0]);
          else if constexpr (i % 3 == 0) mfma(sc[0], rk[k], xf[0][k]);
          else if constexpr (i % 3 == 1) mfma(dp[0], rv[k], yf[0][k]);
          else accumulate(acc[0][k % MB], join(tlo[k], thi[k]), __builtin_bit_cast(bf16x8, pk[0][k / MB]));
        }
        // the places go round and the entries move up, here rather than at the loop's end where no product covers it
        if constexpr (i == 13) moved(kt, kp);
        if constexpr (i == 14) { moved(kp, kn); moved(kn, kf); }
        if constexpr (i == 15) moved(kf, kt);
        if constexpr (i == 21) { moved(kt, vp); moved(vp, vn); }
        if constexpr (i == 22) { moved(vn, kt); moved(e0, e1); moved(e1, e2); }
        if constexpr (i == 23) { moved(e2, e3); moved(e3, e4); }
        __builtin_amdgcn_sched_barrier(0);
      };
      each_slot(slot, std::make_integer_sequence<int, 24>{});
      mask(0, (int)(e0 & 63u));
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_nop 7" : "+v"(pk[1][1]) :: "memory");
#pragma unroll
    for (int k = 0; k < 2 * MB; ++k) accumulate(acc[1][k % MB], join(tlo[k], thi[k]), __builtin_bit_cast(bf16x8, pk[1][k / MB]));
    // the last products have been written (here: behind the loop the compiler first copies the sums, and sees no reason to wait)
    asm volatile("s_nop 15" : "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][2]), "+a"(acc[1][3]));
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // requests past the end (empty: they write zeros)
    asm volatile("" ::: "memory");
  }

  // Accumulator i of acc[hh][mb] is channel 32 mb + 8 (i/4) + 4 kg + i%4 of owner row 32 hh + ln.  The rows go through LDS
  // (16-byte chunks XORed with the row), so that four rows of 256 bytes leave with one store.
  char* const rows = reinterpret_cast<char*>(&st);
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(acc[hh][mb][4 * g + e] * a.scale);
        const int row = 32 * hh + ln;
        *reinterpret_cast<bf16x4*>(rows + row * 256 + (((4 * mb + g) ^ (row & 15)) * 16 + 8 * kg)) = o4;
      }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  uint16_t* const out = a.out1 + (int64_t)h * a.o1_head;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = 4 * i + (lane >> 4), ch = lane & 15;
    const uint4 v = *reinterpret_cast<const uint4*>(rows + row * 256 + ((ch ^ (row & 15)) * 16));
    if (row < o_cnt) *reinterpret_cast<uint4*>(out + (int64_t)(otok0 + row) * a.o1_tok + 8 * ch) = v;
  }
}

}  // namespace

hipError_t lf_launch_attn_bwd_q_wide(const BwdArgs& a, hipStream_t st) {
  return lf_launch(lf_attn_bwd_q_wide_kernel, dim3((unsigned)(a.wg_per_xcd * 8 + 8)), dim3(64), 0, st, a);
}
