// dK and dV of the blockwise sparse attention at head dimension 128, one wavefront per SIMD.
#include "lf_attn_bwd.h"
#include "lf_slots.h"

namespace {

// dK and dV at head dimension 128 for calls whose lists are long, one wavefront per SIMD.  A pair of wavefronts owns a KV block:
// role 0 computes S' = Q K^T, P' and dV^T += dO^T P', role 1 dP' = dO V^T, dS' = P' (dP' - delta) and dK^T += Q^T dS', both over
// all 64 owner rows.
//
// What bounds it: instruction issue of one wavefront.  The kernel with 32 owner rows per wavefront and two wavefronts per SIMD
// reads every tile from LDS twice as often per product (4.2e7 LDS instructions a call; here 2.3e7) and has its matrix cores
// busy for 0.44 of the time.  With 64 rows a wavefront has the register file of a SIMD: 128 accumulators, 64 registers
// of owner rows.  Role 0 and role 1 need about the same time, so the two SIMDs of a pair wait for each other only a little.
// The loop is a list of slots, each one matrix instruction (32 cycles) with the vector, LDS and load
// instructions of another part of the window that fit beside it; the accumulating and the score-like products take turns, since two
// products into the same accumulators would follow each other at once.  sched_barrier and inline assembly keep the slots as
// written; a slot has room for seven instructions beside its product.  Loads go one to a slot behind a product, and what they need
// (resource, addresses of the next places) is made in slots that have room: with loads four at a time, their resources at the
// window's top and packing where the compiler put it, role 1 had slots of 19 to 23 instructions beside empty ones, and role 0
// waited for it (training step of 12 x 128, 4 680 queries: 32 760 keys 1 465 -> 1 441 us, 4 680 keys 387.5 -> 379.6).
// The accumulators are named by inline assembly in the accumulation half of the register file; the scores stay in the other half,
// where vector instructions reach them (left to itself the compiler copies the accumulators around the loop or spills).
// The compiler does not see the latency of those instructions: `settle` waits for the last ones before their results are
// read, and vector results used by them are at least two instructions old (slot order; s_nop before the last products).
// Largest dK/dV launch of a 12 x 128 model (4 680 queries, 32 760 keys): 1.52 million cycles with that kernel, 1.40 with this one's first form, and
// the whole backward call 1 215 us and 1 150; with 4 680 keys 316 and 296.  Up to 52 registers a wavefront are spilled around the
// loop (none is touched in it).
constexpr int kWideEnt = 512;      // half tiles decoded per pass
// Up to this many (head, KV block) pairs a block takes two pairs of wavefronts, each with half of the list: a compute unit holds
// two workgroups of one pair, so fewer blocks leave SIMDs idle.  Backward call in us, one pair and two: 256 blocks with
// 24 query blocks each 83.7 and 69.8, with 64 each 169.8 and 138.6; 384 blocks with 24 each 114.1 and 114.8.
constexpr int kWideSplitBlocks = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int lgkmcnt_imm(int n) { return 15 | (3 << 14) | (7 << 4) | (n << 8); }

template <int SPLIT>
__global__ __launch_bounds__(128 * SPLIT, 1) void lf_attn_bwd_kv_wide_kernel(BwdArgs a) {
  constexpr int D = 128, CH = D / 8, KS = D / 16, MB = D / 32;
  constexpr int T32 = 32 * CH;              // uint4 per half tile: 8 KB
  constexpr uint32_t kTile = T32 * 16u;
  struct Stage {
    uint4 q[4][T32], o[4][T32];             // Q and dO, half tile mod 4
    uint4 p[2][2][2][64];                   // P' handed over: [half tile mod 2][owner half][k-step][lane]
    float4 lse[4][16], nd[4][16];           // row statistics, the upper halves take the zeros of the lanes past the 32 rows
    uint32_t ent[kWideEnt + 8];             // first token << 6 | token count per half tile of a pass; read up to 5 past it
  };
  __shared__ Stage stages[SPLIT];

  const int slot = (blockIdx.x & 7) * a.wg_per_xcd + (blockIdx.x >> 3);
  if (slot >= a.total_wg) return;
  const int w = a.order[slot];
  const int h = w / a.owners, r = w % a.owners;
  const int slice = SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / 128) : 0;
  Stage& st = stages[slice];
  const int lane = threadIdx.x & 63;
  const int role = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 1);
  const int ln = lane & 31, kg = lane >> 5;

  const int otok0 = (r / a.nb) * a.n + (r % a.nb) * 64;
  const int o_cnt = min(64, a.n - (r % a.nb) * 64);
  const int n_all = a.cnt[(int64_t)h * a.owners + r];
  const int n_ent = (n_all + SPLIT - 1) / SPLIT;
  const int my_ent = SPLIT > 1 ? max(min(n_all - slice * n_ent, n_ent), 0) : n_ent;
  const int32_t* list = a.idx + ((int64_t)h * a.owners + r) * a.list_stride + (SPLIT > 1 ? slice * n_ent : 0);

  // the first pass's list entries are asked for together with the owner rows (places past the count hold nothing yet)
  int pre[kWideEnt / 128];
#pragma unroll
  for (int j = 0; j < kWideEnt / 128; ++j) pre[j] = 64 * j + lane < a.list_stride - (SPLIT > 1 ? slice * n_ent : 0) ? list[64 * j + lane] : -1;

  // owner operand: K rows for role 0 (scores), V rows for role 1 (dP')
  bf16x8 of[2][KS];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int row = 32 * hh + ln;
    const uint16_t* op = role ? a.Y + (int64_t)h * a.y_head + (int64_t)(otok0 + row) * a.y_tok
                              : a.X + (int64_t)h * a.x_head + (int64_t)(otok0 + row) * a.x_tok;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      uint4 u = make_uint4(0, 0, 0, 0);
      if (row < o_cnt) u = *reinterpret_cast<const uint4*>(op + s * 16 + kg * 8);
      of[hh][s] = __builtin_bit_cast(bf16x8, u);
    }
  }

  // Tile loads, global -> LDS, 16 rows at a time: load i fills rows [4 i, +4) of them; the buffer resource is those rows, so rows
  // past the half tile's count read as zeros, and both parts of a half tile use the same four offsets.
  const char* Qh = reinterpret_cast<const char*>(a.A1 + (int64_t)h * a.a1_head);
  const char* Oh = reinterpret_cast<const char*>(a.A2 + (int64_t)h * a.a2_head);
  const char* Lh = reinterpret_cast<const char*>(a.lse2 + (int64_t)h * a.q_len);
  const char* Dh = reinterpret_cast<const char*>(a.ndelta + (int64_t)h * a.q_len);
  const uint32_t q_pitch = (uint32_t)(a.a1_tok * 2), o_pitch = (uint32_t)(a.a2_tok * 2);
  uint32_t qoff[4], ooff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 4 * i + (lane >> 4);
    const uint32_t at = (uint32_t)swz<CH>(row, lane & 15) * 16u - 1024u * i;
    qoff[i] = (uint32_t)row * q_pitch + at;
    ooff[i] = (uint32_t)row * o_pitch + at;
  }
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(void, &st));
  auto lds_at = [&](const void* p) { return lds_base + (uint32_t)(reinterpret_cast<const char*>(p) - reinterpret_cast<const char*>(&st)); };
  auto rsrc = [](const char* base, uint32_t pitch, uint32_t e) {
    int32x4 rs;
    const uint64_t b = (uint64_t)base + (uint64_t)(e >> 6) * pitch;
    rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    rs[2] = __builtin_amdgcn_readfirstlane((int)((e & 63u) * pitch));
    rs[3] = 0x00020000;
    return rs;
  };
  auto lower_rows = [](int32x4& rs, uint32_t pitch) __attribute__((always_inline)) {   // from the first 16 rows to the others
    const uint64_t b = ((uint64_t)(uint32_t)rs[1] << 32 | (uint32_t)rs[0]) + (uint64_t)16 * pitch;
    rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    uint32_t end;
    asm("s_max_u32 %0, %1, %2" : "=s"(end) : "s"(rs[2]), "s"(16u * pitch) : "scc");
    rs[2] = (int)(end - 16u * pitch);
  };
  auto fetch4 = [&](int32x4 rs, uint32_t lds0, const uint32_t* o) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
                 :: "s"(lds0), "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]), "s"(rs) : "memory", "m0");
  };
  const uint32_t st_off = (uint32_t)lane * 4u;
  auto fetch_stat = [&](int32x4 rs, uint32_t lds0) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :: "s"(lds0), "v"(st_off), "s"(rs) : "memory", "m0");
  };
  // half tile e (entry) -> a place: nine loads
  auto request_q = [&](uint32_t e, int j) __attribute__((always_inline)) {
    int32x4 rs = rsrc(Qh, q_pitch, e);
    fetch4(rs, lds_at(st.q[j]), qoff);
    lower_rows(rs, q_pitch);
    fetch4(rs, lds_at(st.q[j]) + kTile / 2, qoff);
    fetch_stat(rsrc(Lh, 4u, e), lds_at(st.lse[j]));
  };
  auto request_o = [&](uint32_t e, int j) __attribute__((always_inline)) {
    int32x4 rs = rsrc(Oh, o_pitch, e);
    fetch4(rs, lds_at(st.o[j]), ooff);
    lower_rows(rs, o_pitch);
    fetch4(rs, lds_at(st.o[j]) + kTile / 2, ooff);
    fetch_stat(rsrc(Dh, 4u, e), lds_at(st.nd[j]));
  };

  uint32_t raddr[KS], tbase[2 * MB];
  // row fragment s and half hf of the transposed fragment f = (k-step f / MB, channels f mod MB), `j` places (0 or 1) on
  auto row_frag = [&](int j, int s) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4*)(raddr[s] + (uint32_t)j * kTile));
  };
  auto tread = [&](int j, int f, int hf) __attribute__((always_inline)) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        (__attribute__((address_space(3))) bf16x4*)(tbase[hf * MB + f % MB] + (uint32_t)j * kTile + 16u * (f / MB) * CH * 16u));
  };
  auto join = [](const bf16x4& lo, const bf16x4& hi) { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7); };
  // c += x y, held in the accumulation registers
  auto accumulate = [](f32x16& c, const bf16x8& x, const u32x4& y) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
  };
  // scores: c = x y from zero, from c0, and c += x y, in registers that vector instructions reach
  auto mfma_zero = [](f32x16& c, const bf16x8& x, const bf16x8& y) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(x), "v"(y));
  };
  auto mfma_from = [](f32x16& c, const bf16x8& x, const bf16x8& y, const f32x16& c0) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(c) : "v"(x), "v"(y), "v"(c0));
  };
  auto mfma = [](f32x16& c, const bf16x8& x, const bf16x8& y) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(x), "v"(y));
  };

  f32x16 acc[2][MB];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[hh][mb][i] = 0.0f;

  // the last products into acc[1] have been written
  auto settle = [&]() __attribute__((always_inline)) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][2]), "+a"(acc[1][3]));
  };
  for (int l0 = 0; l0 < n_ent; l0 += kWideEnt / 2) {
    // Decode: entries -> half tiles, back to back; both wavefronts of the pair write the same values.
    if (l0 > 0) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kWideEnt / 128; ++j) pre[j] = l0 + 64 * j + lane < my_ent ? list[l0 + 64 * j + lane] : -1;
    }
    int nt = 0;
#pragma unroll
    for (int e = 0; e < kWideEnt / 128; ++e) {
      if (l0 + 64 * e >= n_ent) break;
      const int c = pre[e];
      const bool ok = l0 + 64 * e + lane < my_ent && (unsigned)c < (unsigned)a.streams;
      const int tau = ok ? c / a.nb : 0, j = ok ? c % a.nb : 0;
      const uint32_t tok = (uint32_t)(tau * a.n + j * 64);
      const int cnt = ok ? min(64, a.n - j * 64) : 0;
      const unsigned long long one = __ballot(cnt > 0), two = __ballot(cnt > 32);
      const unsigned long long below = (1ull << lane) - 1ull;
      const int pos = nt + __popcll(one & below) + __popcll(two & below);
      if (cnt > 0) st.ent[pos] = tok << 6 | (uint32_t)min(cnt, 32);
      if (cnt > 32) st.ent[pos + 1] = (tok + 32) << 6 | (uint32_t)(cnt - 32);
      nt += __popcll(one) + __popcll(two);
    }
    int longest = nt;      // the barriers below are common to the pairs of a workgroup
    if constexpr (SPLIT > 1) {
      int* const cnts = reinterpret_cast<int*>(stages[0].p);
      __syncthreads();
      if (lane == 0 && role == 0) cnts[slice] = nt;
      __syncthreads();
      longest = max(cnts[0], cnts[1]);
      __syncthreads();
    }
    nt = __builtin_amdgcn_readfirstlane(nt);
    longest = __builtin_amdgcn_readfirstlane((longest + 1) & ~1);   // windows go in pairs
    if (longest == 0) continue;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    auto ent_at = [&](int i) -> uint32_t {
      const uint32_t e = st.ent[i];
      return __builtin_amdgcn_readfirstlane(i < nt ? e : 0u);
    };
    auto entry = [&](int i, uint32_t raw) __attribute__((always_inline)) {      // what was read at i, without a branch
      uint32_t e;
      asm("s_cmp_lt_i32 %1, %2\n\ts_cselect_b32 %0, %3, 0" : "=s"(e) : "s"(i), "s"(nt), "s"(__builtin_amdgcn_readfirstlane(raw)) : "scc");
      return e;
    };
    uint32_t e0 = ent_at(0), e1 = ent_at(1), e2 = ent_at(2);   // half tiles t, t + 1, t + 2
    bf16x8 rf[KS];                     // row fragments
    bf16x4 tlo[2 * MB], thi[2 * MB];   // transposed fragments
    f32x16 sc[2];                      // S' or dP' - delta: [owner half]
    u32x4 pk[2][2];                    // P' or dS', packed: [owner half][k-step]
    // LDS addresses of this lane's fragments in place 0: rows of what this role loads, transposed reads of the other's.  Those of the
    // transposed reads are made here in every pass (at_lane hides that they do not change): kept over the whole kernel they are
    // spilled, and the wait for their reload stood in the loop, a vmcnt(0) in every second window that drained the tile loads
    // (backward call of a 12 x 128 chunk, 4 680 queries: 32 760 keys 1 172 -> 1 150 us, 4 680 keys 299.5 -> 295.5).
    int at_lane = lane;
    asm volatile("" : "+v"(at_lane));
#pragma unroll
    for (int s = 0; s < KS; ++s) raddr[s] = lds_at(role ? st.o[0] : st.q[0]) + 16u * (ln * CH + swz<CH>(ln, 2 * s + kg));
    {
      const int i16 = at_lane & 15;
      const int tr_row = 4 * (at_lane >> 5) + (i16 >> 2);
      const int tr_col = 16 * ((at_lane >> 4) & 1) + 4 * (i16 & 3);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int col = 32 * mb + tr_col;
        const uint32_t at = 2u * ((tr_row * CH + swz<CH>(tr_row, col >> 3)) * 8 + (col & 7));
        tbase[mb] = lds_at(role ? st.q[0] : st.o[0]) + at;
        tbase[MB + mb] = lds_at(role ? st.q[0] : st.o[0]) + (at ^ (2u * kTrHiFlip<CH>)) + 8u * CH * 16u;
      }
    }
    // A window is two phases of sixteen slots, one matrix instruction each, the accumulating and the score-like product in
    // turn: phase 0 takes half 1 of the half tile before and half 1 of this one, phase 1 half 0 of this one and half 0 of the
    // next.  Windows go in pairs, which share two of the four places; the addresses move to the other two by `hop`.
    uint32_t far = 2 * kTile;                       // the places that this pair does not use
    int hop = 2 * (int)kTile;
    uint32_t saddr = lds_at(role ? st.nd[0] : st.lse[0]) + 16u * kg;   // this lane's row statistics
    auto stat4 = [&](f32x16& v, int j, int g) __attribute__((always_inline)) {
      const f32x4 q = *(const __attribute__((address_space(3))) f32x4*)(saddr + 256u * j + 32u * g);
      v[4 * g] = q[0]; v[4 * g + 1] = q[1]; v[4 * g + 2] = q[2]; v[4 * g + 3] = q[3];
    };
    // in slots 8 to 15 of phase 1, one address each: rows behind the first window of a pair, transposed reads behind the second
    auto hop_one = [&](int b, int i) __attribute__((always_inline)) {
      uint32_t& at = b == 0 ? raddr[i] : tbase[i];
      asm volatile("v_add_u32 %0, %1, %0" : "+v"(at) : "s"(hop));
      if (b == 1 && i == 7) {
        far ^= 2 * kTile;
        hop = -hop;
      }
    };
    static_assert(KS == 8 && 2 * MB == 8, "one address a slot");
#pragma unroll
    for (int f = 0; f < 2 * MB; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) tlo[f][e] = thi[f][e] = (__bf16)0.0f;
    pk[1][0] = pk[1][1] = u32x4{0u, 0u, 0u, 0u};
    if (role == 0) {
      f32x16 lse;
      float x[2] = {-INFINITY, -INFINITY}, ee[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        sc[1][i] = -INFINITY;
        lse[i] = 0.0f;
      }
      auto fma_of = [&](int hh, int v) __attribute__((always_inline)) {
        asm volatile("v_fma_f32 %0, %1, %2, -%3" : "=v"(x[v & 1]) : "v"(sc[hh][v]), "s"(a.c), "v"(lse[v]));
      };
      auto exp_of = [&](int v) __attribute__((always_inline)) { asm volatile("v_exp_f32 %0, %1" : "=v"(ee[v & 3]) : "v"(x[v & 1])); };
      auto pack_of = [&](int hh, int v) __attribute__((always_inline)) {   // v odd
        asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(pk[hh][v >> 3][(v & 7) >> 1]) : "v"(ee[(v - 1) & 3]), "v"(ee[v & 3]));
      };
      // rows past a short half tile's count were loaded as zeros: their scores become -inf (P' = 0); the last of their products
      // stands right before
      auto mask = [&](int hh, int cnt) __attribute__((always_inline)) {
        if (cnt < 32) {
          asm volatile("s_nop 15" : "+v"(sc[hh]));
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (8 * (i >> 2) + 4 * kg + (i & 3) >= cnt) sc[hh][i] = -INFINITY;
        }
      };
      // slot i of a phase that works on half hh: value v is scaled in slot v + 2, exp2 in slot v + 3, packed (odd v) in slot
      // v + 4; the first slots finish the other half's last values
      auto soft = [&](int i, int hh) __attribute__((always_inline)) {
        exp_of((i + 13) & 15);
        fma_of(i < 2 ? hh ^ 1 : hh, (i + 14) & 15);
        if (i & 1) pack_of(i < 4 ? hh ^ 1 : hh, (i + 12) & 15);
      };
      auto window = [&](int t, int b) __attribute__((always_inline)) {
        uint32_t e_raw = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int k = i >> 1;
          soft(i, 0);
          if (i == 1) mfma_zero(sc[1], rf[k], of[1][k]);
          else if (i & 1) mfma(sc[1], rf[k], of[1][k]);
          else accumulate(acc[1][k % MB], join(tlo[k], thi[k]), pk[1][k / MB]);
          if (i == 3) stat4(lse, b, 3);
          if (i == 4 && b == 1) saddr += (uint32_t)(hop >> 5);
          if (i == 4) st.p[b ^ 1][1][1][lane] = __builtin_bit_cast(uint4, pk[1][1]);
          if (i == 6) lds_barrier();
          if (i >= 6) {
            const int f = (i - 6) >> 1;
            if (i & 1) thi[f] = tread(b, f, 1);
            else tlo[f] = tread(b, f, 0);
          }
          if (i >= 9 && (i & 1)) rf[(i - 9) >> 1] = row_frag(b ^ 1, (i - 9) >> 1);
          if (i == 12) st.p[b][0][0][lane] = __builtin_bit_cast(uint4, pk[0][0]);
          if (i == 14) e_raw = st.ent[t + 2];
          __builtin_amdgcn_sched_barrier(0);
        }
        mask(1, (int)(e0 & 63u));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int k = i >> 1;
          soft(i, 1);
          if (i == 1) mfma_zero(sc[0], rf[k], of[0][k]);
          else if (i & 1) mfma(sc[0], rf[k], of[0][k]);
          else accumulate(acc[0][k % MB], join(tlo[k], thi[k]), pk[0][k / MB]);
          if (i < 6) {
            const int f = 5 + (i >> 1);
            if (i & 1) thi[f] = tread(b, f, 1);
            else tlo[f] = tread(b, f, 0);
          }
          if (i < 8 && (i & 1)) rf[4 + (i >> 1)] = row_frag(b ^ 1, 4 + (i >> 1));
          if (i == 4) st.p[b][0][1][lane] = __builtin_bit_cast(uint4, pk[0][1]);
          if (i == 8) stat4(lse, b ^ 1, 0);
          if (i == 11) stat4(lse, b ^ 1, 1);
          if (i == 13) stat4(lse, b ^ 1, 2);
          if (i == 12) st.p[b][1][0][lane] = __builtin_bit_cast(uint4, pk[1][0]);
          if (i >= 8) hop_one(b, i - 8);
          __builtin_amdgcn_sched_barrier(0);
        }
        mask(0, (int)(e1 & 63u));
        e0 = e1;
        e1 = entry(t + 2, e_raw);
        __builtin_amdgcn_sched_barrier(0);
      };
      // the first four half tiles of Q; the others come from the other role
      request_q(e0, 0);
      request_q(e1, 1);
      request_q(e2, 2);
      request_q(ent_at(3), 3);
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      asm volatile("" ::: "memory");
#pragma unroll
      for (int s = 0; s < KS; ++s) rf[s] = row_frag(0, s);
#pragma unroll
      for (int g = 0; g < 4; ++g) stat4(lse, 0, g);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s == 0) mfma_zero(sc[0], rf[s], of[0][s]);
        else mfma(sc[0], rf[s], of[0][s]);
      }
      asm volatile("s_nop 15" : "+v"(sc[0]));
      mask(0, (int)(e0 & 63u));
      __builtin_amdgcn_sched_barrier(0);
      for (int t = 0; t < longest; t += 2) {
        window(t, 0);
        window(t + 1, 1);
      }
      // the last half tile's half 1
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        exp_of(13 + i);
        if (i < 2) fma_of(1, 14 + i);
        if (i == 1) pack_of(1, 13);
      }
      pack_of(1, 15);
      st.p[1][1][1][lane] = __builtin_bit_cast(uint4, pk[1][1]);
      asm volatile("s_nop 7" : "+v"(pk[1][1]) :: "memory");
#pragma unroll
      for (int k = 0; k < 2 * MB; ++k) accumulate(acc[1][k % MB], join(tlo[k], thi[k]), pk[1][k / MB]);
      settle();
      lds_barrier();
      lds_barrier();                  // the other role has read the last tile
    } else {
      uint32_t e3 = 0;                // half tile t + 4
      f32x16 nd;
      uint4 pu[2][2];                 // P' of role 0: [owner half][k-step]
      float m[2];
      pu[1][1] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[1][i] = 0.0f;
      auto mul_of = [&](int hh, int v) __attribute__((always_inline)) {
        const uint32_t p = reinterpret_cast<const uint32_t*>(&pu[hh][v >> 3])[(v & 7) >> 1];
        if (v & 1)
          asm volatile("v_and_b32 %1, 0xffff0000, %2\n\tv_mul_f32 %1, %1, %3\n\tv_cvt_pk_bf16_f32 %0, %4, %1"
                       : "=v"(pk[hh][v >> 3][(v & 7) >> 1]), "=&v"(m[1]) : "v"(p), "v"(sc[hh][v]), "v"(m[0]));
        else
          asm volatile("v_lshlrev_b32 %0, 16, %1\n\tv_mul_f32 %0, %0, %2" : "=&v"(m[0]) : "v"(p), "v"(sc[hh][v]));
      };
      // The pair meets in slot 10 of phase 1, behind the window's last load, after which P' of half tile t + 1 is there; value v of a half in slot v + 2.
      // This role loads for both: it has less vector work.
      auto meet = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(18));    // all but the last request of dO and of Q has landed
        lds_barrier();
      };
      // The product of slot i with a tile load behind it in slots 2 to 9.
      int32x4 rs, rl = rsrc(Lh, 4u, 0), rd = rsrc(Dh, 4u, 0);
      uint32_t e_raw = 0;
      auto tile_rsrc = [&](const char* base, uint32_t pitch, uint32_t e) __attribute__((always_inline)) {
        asm volatile("" : "+s"(e));
        const uint64_t at = (uint64_t)base + (uint64_t)(e >> 6) * pitch;
        rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)at);
        rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
        rs[3] = 0x00020000;
      };
      // row statistics: the resource ends behind the half tile's rows
      auto load_stat = [&](int32x4& r, uint32_t e, uint32_t lds0) __attribute__((always_inline)) {
        asm volatile("" : "+s"(e));      // made here, not at the loop's top
        const uint32_t first = (e >> 6) * 4u;
        r[2] = __builtin_amdgcn_readfirstlane((int)(first + (e & 63u) * 4u));
        uint32_t off;
        asm volatile("s_mov_b32 m0, %3\n\tv_add_u32 %0, %1, %2\n\tbuffer_load_dword %0, %4, 0 offen lds"
                     : "=&v"(off) : "s"(first), "v"(st_off), "s"(lds0), "s"(r) : "memory", "m0");
      };
      auto window = [&](int t, auto bc) __attribute__((always_inline)) {
        constexpr int b = decltype(bc)::value;
        const uint32_t here = far ^ (2 * kTile);
        const uint32_t to = b ? here : far + kTile;     // place of half tile t + 3 of dO; that of t + 4 of Q is this one's
        auto slot = [&](auto ic) __attribute__((always_inline)) {
          constexpr int ph = decltype(ic)::value >> 4, hh = 1 - ph, i = decltype(ic)::value & 15, k = i >> 1, j = (i - 2) & 3;
          mul_of(i < 2 ? hh : 1 - hh, (i + 14) & 15);
          if constexpr (ph == 1 && i == 2) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(10));   // rows 0 to 15 of Q have been read
          if constexpr (ph == 1 && i == 6) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(3));    // rows 16 to 31
          if constexpr (i == 6) lower_rows(rs, ph ? q_pitch : o_pitch);
          const uint32_t lds0 = (ph ? lds_at(st.q[b]) + here : lds_at(st.o[0]) + to) + (i >= 6 ? kTile / 2 : 0);
          const uint32_t o = i < 2 || i > 9 ? 0u : ph ? qoff[j] : ooff[j];
          if constexpr (i >= 2 && i < 10) {
            if constexpr (i & 1) { LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+v", sc[hh], rf[k], "v", of[hh][k], rs, lds0, o, j) }
            else { LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+a", acc[hh][k % MB], join(tlo[k], thi[k]), "v", pk[hh][k / MB], rs, lds0, o, j) }
          } else if constexpr (i == 1) {
            mfma_from(sc[hh], rf[k], of[hh][k], nd);
          } else if constexpr (i & 1) {
            mfma(sc[hh], rf[k], of[hh][k]);
          } else {
            accumulate(acc[hh][k % MB], join(tlo[k], thi[k]), pk[hh][k / MB]);
          }
          // The product of slot 1 reads nd for seven wait states: kept up to here, so that no vector instruction gets its place before.
          if constexpr (i == 2) asm volatile("" :: "v"(nd));
          if constexpr (ph == 0) {
            if constexpr (i == 12) tile_rsrc(Qh, q_pitch, e3);      // of the next phase's loads
            if constexpr (i == 13) rs[2] = __builtin_amdgcn_readfirstlane((int)((e3 & 63u) * q_pitch));
            if constexpr (i == 3) pu[1][1] = st.p[b][1][1][lane];
            if constexpr (i == 4 && b == 1) saddr += (uint32_t)(hop >> 5);
            if constexpr (i == 10) load_stat(rd, e2, lds_at(st.nd[0]) + (to >> 5));
            // a fragment of Q gives its place to the next one behind its last product
            if constexpr (i & 1) {
              tlo[k] = tread(b, k, 0);
              thi[k] = tread(b, k, 1);
            }
            if constexpr (i >= 8 && !(i & 1)) stat4(nd, b ^ 1, (i - 8) >> 1);
            if constexpr (i >= 9 && (i & 1)) rf[(i - 9) >> 1] = row_frag(b ^ 1, (i - 9) >> 1);
            if constexpr (i == 15) e_raw = st.ent[t + 5];
          } else {
            if constexpr (i < 8 && (i & 1)) rf[4 + (i >> 1)] = row_frag(b ^ 1, 4 + (i >> 1));
            if constexpr (i == 13) tile_rsrc(Oh, o_pitch, e3);
            if constexpr (i == 14) rs[2] = __builtin_amdgcn_readfirstlane((int)((e3 & 63u) * o_pitch));
            if constexpr (i == 10) {
              load_stat(rl, e3, lds_at(st.lse[b]) + (here >> 5));
              meet();
              pu[0][0] = st.p[b ^ 1][0][0][lane];
            }
            if constexpr (i == 11) pu[0][1] = st.p[b ^ 1][0][1][lane];
            if constexpr (i == 12) pu[1][0] = st.p[b ^ 1][1][0][lane];
            if constexpr (i >= 8) hop_one(b, i - 8);
            if constexpr (i == 15) {
              e2 = e3;
              e3 = entry(t + 5, e_raw);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        each_slot(slot, std::make_integer_sequence<int, 32>{});
      };
      request_o(e0, 0);
      request_o(e1, 1);
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(9));
      lds_barrier();
      request_o(e2, 2);
#pragma unroll
      for (int s = 0; s < KS; ++s) rf[s] = row_frag(0, s);
#pragma unroll
      for (int g = 0; g < 4; ++g) stat4(nd, 0, g);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s == 0) mfma_from(sc[0], rf[s], of[0][s], nd);
        else mfma(sc[0], rf[s], of[0][s]);
      }
      asm volatile("s_nop 15" : "+v"(sc[0]));
      e2 = ent_at(3);
      e3 = ent_at(4);
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(9));     // half tile 1 of dO has landed
      lds_barrier();
      pu[0][0] = st.p[0][0][0][lane];
      pu[0][1] = st.p[0][0][1][lane];
      pu[1][0] = st.p[0][1][0][lane];
      rs = rsrc(Oh, o_pitch, e2);
      __builtin_amdgcn_sched_barrier(0);
      for (int t = 0; t < longest; t += 2) {
        window(t, std::integral_constant<int, 0>{});
        window(t + 1, std::integral_constant<int, 1>{});
      }
#pragma unroll
      for (int v = 14; v < 16; ++v) mul_of(1, v);
      asm volatile("s_nop 7" : "+v"(pk[1][1]) :: "memory");
#pragma unroll
      for (int k = 0; k < 2 * MB; ++k) accumulate(acc[1][k % MB], join(tlo[k], thi[k]), pk[1][k / MB]);
      settle();
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // requests past the end (empty: they write zeros)
  }

  // Role 1 loads the tiles of both, and its requests past the end of the list write zeros: role 0 may put its sums where Q was
  // only when they have landed.  (Role 1's last meeting in the loop leaves those of the last window in flight.)
  __syncthreads();
  if constexpr (SPLIT > 1) {
    // the second pair leaves its sums where its tiles were, the first adds them to its own
    float4* const sums = reinterpret_cast<float4*>(role ? stages[1].o[0] : stages[1].q[0]);
    if (slice == 1) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            sums[((hh * MB + mb) * 4 + g) * 64 + lane] = make_float4(acc[hh][mb][4 * g + 0], acc[hh][mb][4 * g + 1],
                                                                     acc[hh][mb][4 * g + 2], acc[hh][mb][4 * g + 3]);
    }
    __syncthreads();
    if (slice == 1) return;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 v = sums[((hh * MB + mb) * 4 + g) * 64 + lane];
          acc[hh][mb][4 * g + 0] += v.x; acc[hh][mb][4 * g + 1] += v.y;
          acc[hh][mb][4 * g + 2] += v.z; acc[hh][mb][4 * g + 3] += v.w;
        }
  }
  // Accumulator i of acc[hh][mb] is channel 32 mb + 8 (i/4) + 4 kg + i%4 of owner row 32 hh + ln.  The rows go through LDS
  // (16-byte chunks XORed with the row, where this role's tiles were: the barrier above follows the other role's reads of them and
  // all loads into them), so that four rows of 256 bytes leave with one store.
  char* const rows = reinterpret_cast<char*>(role ? st.o[0] : st.q[0]);
  const float factor = role ? a.scale : 1.0f;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(acc[hh][mb][4 * g + e] * factor);
        const int row = 32 * hh + ln;
        *reinterpret_cast<bf16x4*>(rows + row * 256 + (((4 * mb + g) ^ (row & 15)) * 16 + 8 * kg)) = o4;
      }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  uint16_t* const out = role ? a.out1 + (int64_t)h * a.o1_head : a.out2 + (int64_t)h * a.o2_head;
  const int64_t out_tok = role ? a.o1_tok : a.o2_tok;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = 4 * i + (lane >> 4), ch = lane & 15;
    const uint4 v = *reinterpret_cast<const uint4*>(rows + row * 256 + ((ch ^ (row & 15)) * 16));
    if (row < o_cnt) *reinterpret_cast<uint4*>(out + (int64_t)(otok0 + row) * out_tok + 8 * ch) = v;
  }
}

}  // namespace

hipError_t lf_launch_attn_bwd_kv_wide(const BwdArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)(a.wg_per_xcd * 8));
  return a.total_wg <= kWideSplitBlocks ? lf_launch(lf_attn_bwd_kv_wide_kernel<2>, grid, dim3(256), 0, st, a)
                           : lf_launch(lf_attn_bwd_kv_wide_kernel<1>, grid, dim3(128), 0, st, a);
}
