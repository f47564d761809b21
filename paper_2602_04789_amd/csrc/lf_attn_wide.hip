// Blockwise sparse attention at head dimension 128, one wavefront per query block: undivided list-driven calls with enough query
// blocks (lf_launch_attn has the rule).
//
// What bounds it: instruction issue of the one wavefront that a SIMD holds.  The two-wavefront form reads a tile's K and V fragments
// once per 32 query rows, this one once per 64, and it has no barrier: K and V are private to the wavefront, two half tiles of each.
// A step works on half tile t in 32 slots of one matrix instruction (32 cycles) each, kept as written by sched_barrier: 16 of
// S of t + 1 and then 16 of O += V^T P of t - 1, with the exponentials of t, the LDS reads for what comes next and the loads of K
// of t + 3 and V of t + 1 beside them.  Products and exponentials are inline assembly: as builtins the compiler moves them
// together, which leaves slots too full beside empty ones.  A slot holds about one exponential (16 cycles of issue), one scaling,
// half a conversion and one or two LDS reads or loads; the loads go one to a slot, with M0 written once per four.  O is named by inline assembly in the accumulation half of the register file; scores stay
// in the other half, where vector instructions reach them (left to itself the compiler copies O around the loop).
// The compiler does not see those instructions' latency: `settle` waits before O is read or changed.
// A load goes to the place that the reads before it leave, so each is preceded by a wait that counts the LDS reads issued since.
// 12 x 128, 4 680 queries, lists of 188 blocks: 333 us with two wavefronts per query block, 323 with one, of these slots 319;
// 12 x 2 880, lists of 40: 70.5 us with the products as builtins and the loads four at a time, 68.9 now; 30 x 6 400, lists of 64:
// 385 and 381.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lf_common.h"
#include "lf_slots.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int int32x4 __attribute__((ext_vector_type(4)));

struct WideArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  uint16_t* O;
  const int32_t* idx;
  int64_t q_stride_tok, q_stride_head, k_stride_head, v_stride_head, o_stride_tok, o_stride_head;
  uint32_t k_row_bytes, v_row_bytes;
  int n, nb, n_q, n_k;
  uint32_t nb_inv;      // floor((2^32 - 1) / nb)
  int list_len, own_len, tail0;   // entries of a list; those of them that are read; entry i beyond is block tail0 + i
  int total, wg_per_xcd;
  float c;              // softmax_scale * log2(e)
  float* lse2;
  int q_len;
};

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

constexpr int lgkmcnt_imm(int n) { return 15 | (3 << 14) | (7 << 4) | (n << 8); }

constexpr int D = 128, CH = D / 8, KS = D / 16, MB = D / 32;
constexpr int TILE = 32 * CH;      // uint4 per tile (32 KV rows of K or V): 8 KB
constexpr int kEnt = 1024;         // tiles decoded per pass
constexpr int kLoads = 8;          // load instructions per tile: 1 KB, four rows each

__device__ __forceinline__ int k_swz(int row, int ch) { return ch ^ (row & (CH - 1)); }
__device__ __forceinline__ int v_swz(int row, int ch) { return ch ^ ((row & 3) << 2); }

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}
__device__ __forceinline__ void mfma_first(f32x16& s, const bf16x8& a, const bf16x8& b) {
  s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, zero16(), 0, 0, 0);
}
__device__ __forceinline__ void mfma_next(f32x16& s, const bf16x8& a, const bf16x8& b) {
  s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, s, 0, 0, 0);
}

// O += V^T P^T, held in the accumulation registers
__device__ __forceinline__ void accumulate(f32x16& c, const bf16x8& x, const bf16x8& y) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
}

struct Stage {
  uint4 k[2][TILE], v[2][TILE];   // half tile mod 2
  uint32_t ent[kEnt];             // first token << 6 | token count
};

__global__ __launch_bounds__(64, 1) void lf_attn_wide_kernel(WideArgs a) {
  __shared__ Stage st;
  const int w = (blockIdx.x & 7) * a.wg_per_xcd + (blockIdx.x >> 3);
  if (w >= a.total) return;
  const int h = w / a.n_q, r = w % a.n_q;
  const int lane = threadIdx.x & 63, ln = lane & 31, kg = lane >> 5;
  const int jb = r % a.nb, qtok0 = (r / a.nb) * a.n + jb * 64, q_cnt = min(64, a.n - jb * 64);
  const int32_t* list = a.idx + ((int64_t)h * a.n_q + r) * a.list_len;

  bf16x8 qf[2][KS];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int row = 32 * hh + ln;
    const uint16_t* qp = a.Q + (int64_t)h * a.q_stride_head + (int64_t)(qtok0 + row) * a.q_stride_tok;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      uint4 u = make_uint4(0, 0, 0, 0);
      if (row < q_cnt) u = *reinterpret_cast<const uint4*>(qp + s * 16 + kg * 8);
      qf[hh][s] = __builtin_bit_cast(bf16x8, u);
    }
  }
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" : "+a"(qf[hh][s]));
  const char* Kh = reinterpret_cast<const char*>(a.K + (int64_t)h * a.k_stride_head);
  const char* Vh = reinterpret_cast<const char*>(a.V + (int64_t)h * a.v_stride_head);

  uint32_t koff[kLoads], voff[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; ++i) {
    const int row = 4 * i + (lane >> 4), p = lane & 15;
    koff[i] = (uint32_t)row * a.k_row_bytes + (uint32_t)k_swz(row, p) * 16u - 1024u * (i & 3);
    voff[i] = (uint32_t)row * a.v_row_bytes + (uint32_t)v_swz(row, p) * 16u - 1024u * (i & 3);
  }
  auto rsrc = [](const char* base, uint32_t row_bytes, uint32_t e) {
    int32x4 rs;
    const uint64_t b = (uint64_t)base + (uint64_t)((e >> 6) * row_bytes);   // one head's K or V spans less than 2 GiB
    rs[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    rs[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    rs[2] = __builtin_amdgcn_readfirstlane((int)((e & 63u) * row_bytes));
    rs[3] = 0x00020000;
    return rs;
  };
  auto fetch4 = [&](int32x4 rs, uint4* dst, const uint32_t* off) __attribute__((always_inline)) {
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(void, &st)) +
                          (uint32_t)(reinterpret_cast<const char*>(dst) - reinterpret_cast<const char*>(&st));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
                 :: "s"(lds0), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(rs) : "memory", "m0");
  };
  auto fetch_k = [&](uint32_t e, uint4* dst) __attribute__((always_inline)) {
    const int32x4 rs = rsrc(Kh, a.k_row_bytes, e);
    fetch4(rs, dst, koff);
    fetch4(rs, dst + TILE / 2, koff + 4);
  };
  auto fetch_v = [&](uint32_t e, uint4* dst) __attribute__((always_inline)) {
    const int32x4 rs = rsrc(Vh, a.v_row_bytes, e);
    fetch4(rs, dst, voff);
    fetch4(rs, dst + TILE / 2, voff + 4);
  };

  int kaddr[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) kaddr[s] = ln * CH + k_swz(ln, 2 * s + kg);
  int vbase[MB];
  {
    const int i16 = lane & 15;
    const int tr_row = 4 * kg + (i16 >> 2);
    const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int col = 32 * mb + tr_col;
      vbase[mb] = (tr_row * CH + v_swz(tr_row, col >> 3)) * 8 + (col & 7);
    }
  }
  auto vread = [&](const uint4* tile, int u, int hf, int mb) __attribute__((always_inline)) {
    const uint16_t* p16 = reinterpret_cast<const uint16_t*>(tile);
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p16 + vbase[mb] + (16 * u + 8 * hf) * CH * 8));
  };

  f32x16 oacc[2][MB];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[hh][mb][i] = 0.0f;
  // waits for the products on their way into O (and, after O was changed, before the next ones read it)
  auto settle = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
      asm volatile("s_nop 15\n\ts_nop 3" : "+a"(oacc[hh][0]), "+a"(oacc[hh][1]), "+a"(oacc[hh][2]), "+a"(oacc[hh][3]));
  };
  constexpr float kSumMax = 1.0e30f;
  float m_run[2] = {-1.0e30f, -1.0e30f};
  // Row sums of P as rounded, by 4 x 4 x 4 products with ones: a lane's four results are all the sum of its own four values, so no
  // lane sees another row's.  The dot product that adds two values at a time does not overlap with the matrix cores: 332 us with it
  // for the largest call, 323 with these products (and 340 with the values taken apart and added in float32).
  f32x4 l_run[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
  u32x2 one4 = {0x3f803f80u, 0x3f803f80u};
  asm volatile("" : "+a"(one4));   // stays there: made anew in front of a product it would be read too early
  auto row_max = [](const f32x16& sc) __attribute__((always_inline)) {
    float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
#pragma unroll
    for (int i = 4; i < 16; i += 2) mx = fmaxf(mx, fmaxf(sc[i], sc[i + 1]));
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};   // where the reference moves, the sum is taken with dot products

  for (int l0 = 0; l0 < a.list_len; l0 += kEnt / 2) {
    const int l1 = min(a.list_len, l0 + kEnt / 2);
    int nt = 0;
    for (int i0 = l0; i0 < l1; i0 += 256) {
      int ids[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + 64 * j + lane;
        ids[j] = i < min(l1, a.own_len) ? list[i] : -1;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + 64 * j + lane;
        const uint32_t c = (uint32_t)(i >= a.own_len && i < l1 ? a.tail0 + i : ids[j]);
        uint32_t tau = __umulhi(c, a.nb_inv);
        uint32_t rem = c - tau * a.nb;
        if (rem >= (uint32_t)a.nb) { rem -= a.nb; ++tau; }
        const uint32_t tok = tau * a.n + rem * 64;
        const int cnt = c < (uint32_t)a.n_k ? min(64, a.n - (int)rem * 64) : 0;
        const unsigned long long one = __ballot(cnt > 0), two = __ballot(cnt > 32);
        const unsigned long long below = (1ull << lane) - 1ull;
        const int pos = nt + __popcll(one & below) + __popcll(two & below);
        if (cnt > 0) st.ent[pos] = tok << 6 | (uint32_t)min(cnt, 32);
        if (cnt > 32) st.ent[pos + 1] = (tok + 32) << 6 | (uint32_t)(cnt - 32);
        nt += __popcll(one) + __popcll(two);
      }
    }
    nt = __builtin_amdgcn_readfirstlane(nt);
    if (nt == 0) continue;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    auto ent_at = [&](int i) -> uint32_t {
      const uint32_t e = st.ent[i & (kEnt - 1)];
      return __builtin_amdgcn_readfirstlane(i < nt ? e : 0u);
    };

    uint32_t e0 = ent_at(0), e1 = ent_at(1), e2 = ent_at(2), e3 = ent_at(3);   // tiles t .. t + 3
    fetch_k(e0, st.k[0]);
    fetch_k(e1, st.k[1]);
    fetch_v(e0, st.v[0]);

    bf16x8 kf[KS], vf[2 * MB];
    f32x16 s0[2], s1[2];
    u32x4 p0[2][2], p1[2][2];
    auto read_k = [&](const uint4* tile) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < KS; ++s) kf[s] = __builtin_bit_cast(bf16x8, tile[kaddr[s]]);
    };
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(16));
    asm volatile("" ::: "memory");
    read_k(st.k[0]);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        if (s == 0) mfma_first(s0[hh], kf[s], qf[hh][s]);
        else mfma_next(s0[hh], kf[s], qf[hh][s]);
      }
    __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(0));   // tile 0 is in registers: its place takes tile 2
    __builtin_amdgcn_sched_barrier(0);
    fetch_k(e2, st.k[0]);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(16));
    asm volatile("" ::: "memory");
    read_k(st.k[1]);
    __builtin_amdgcn_sched_barrier(0);

    // Step t: sc = S of tile t, sn receives S of tile t + 1; pc receives P of tile t, pv = P of tile t - 1.
    // kt: tile t + 2's place (even steps 0); vt: tile t - 1's place.
    auto mask = [&](f32x16 (&sc)[2], int cnt) __attribute__((always_inline)) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i >> 2) + 4 * kg + (i & 3) >= cnt) sc[hh][i] = -INFINITY;
    };
    asm volatile("s_nop 15" : "+v"(s0[0]), "+v"(s0[1]));
    if ((e0 & 63u) < 32u) mask(s0, (int)(e0 & 63u));
    auto step = [&](int t, auto first_, auto last_, uint4* k_free, uint4* k_next, uint4* vt, f32x16 (&sc)[2], f32x16 (&sn)[2],
                    u32x4 (&pc)[2][2], const u32x4 (&pv)[2][2]) __attribute__((always_inline)) {
      constexpr bool first = decltype(first_)::value, last = decltype(last_)::value;
      uint32_t e_raw;
      // V of t - 1 has landed (K of t + 2 and V of t are in flight)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(16));
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      float x[4], ee[4];
      const u32x2 ones4 = one4;
      const float l_old[2] = {l_run[0][0], l_run[1][0]};
      int32x4 rs;
      bf16x4 vlo[2 * MB], vhi[2 * MB];
      // Value v of the softmax is scaled in slot at(v) = 0 .. 28, exp2 in the next one, packed (odd v) and, four at a time,
      // added to the row's sum in the one after.
      auto soft = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 32; ++v) {
          const int at = v * 28 / 31, hh = v >> 4, e = v & 15;
          if (i == at + 2 && (e & 1)) {
            asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(pc[hh][e >> 3][(e & 7) >> 1]) : "v"(ee[(v - 1) & 3]), "v"(ee[v & 3]));
          }
          if (i == at + 1) asm volatile("v_exp_f32 %0, %1" : "=v"(ee[v & 3]) : "v"(x[v & 3]));
          if (i == at) asm volatile("v_fma_f32 %0, %1, %2, -%3" : "=v"(x[v & 3]) : "v"(sc[hh][e]), "s"(a.c), "v"(m_run[hh]));
        }
      };
      // The sums come behind a slot's other instructions, a slot after their last value is packed: a product may read what a
      // vector instruction wrote two instructions before at the earliest.
      auto sums = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 3; v < 32; v += 4)
          if (i == v * 28 / 31 + 3) {
            const int hh = v >> 4, e = v & 15;
            const u32x2 p4 = {pc[hh][e >> 3][((e & 7) >> 1) - 1], pc[hh][e >> 3][(e & 7) >> 1]};
            if (v == 31) asm volatile("s_nop 1\n\tv_mfma_f32_4x4x4_16b_bf16 %0, %1, %2, %0" : "+v"(l_run[hh]) : "a"(ones4), "v"(p4));
            else asm volatile("v_mfma_f32_4x4x4_16b_bf16 %0, %1, %2, %0" : "+v"(l_run[hh]) : "a"(ones4), "v"(p4));
          }
      };
      auto place = [&](const uint4* dst) __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(void, &st)) +
               (uint32_t)(reinterpret_cast<const char*>(dst) - reinterpret_cast<const char*>(&st));
      };
      auto score_slot = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, s = i >> 1, hh = i & 1;
        if constexpr (i == 4) rs = rsrc(Kh, a.k_row_bytes, e3);
        if constexpr (i >= 5 && i < 13) {
          constexpr int l = i - 5;
          if constexpr (last) {
            if constexpr ((l & 3) == 0) fetch4(rs, k_free + (l >> 2) * (TILE / 2), koff + (l & 4));
          } else {
            LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+v", sn[hh], kf[s], "a", qf[hh][s], rs,
                                place(k_free + (l >> 2) * (TILE / 2)), koff[l], l & 3)
          }
        } else if constexpr (last) {   // no tile follows
        } else if constexpr (s == 0) {
          asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(sn[hh]) : "v"(kf[s]), "a"(qf[hh][s]));
        } else {
          asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(sn[hh]) : "v"(kf[s]), "a"(qf[hh][s]));
        }
        if constexpr (!first) {
          if constexpr (hh) vhi[i >> 1] = vread(vt, i >> 3, 1, (i >> 1) & 3);
          else vlo[i >> 1] = vread(vt, i >> 3, 0, (i >> 1) & 3);
        }
        if constexpr (i == 4) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(first ? 0 : 5));   // K of t + 1 is in registers
        soft(i);
        sums(i);
        __builtin_amdgcn_sched_barrier(0);
      };
      each_slot(score_slot, std::make_integer_sequence<int, 16>{});
#pragma unroll
      for (int i = 0; i < 2 * MB; ++i) vf[i] = __builtin_shufflevector(vlo[i], vhi[i], 0, 1, 2, 3, 4, 5, 6, 7);
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(first ? 8 : 16));   // K of t + 2
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      auto value_slot = [&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, u = i >> 3, mb = (i >> 1) & 3, hh = i & 1;
        if constexpr (i == 4) rs = rsrc(Vh, a.v_row_bytes, e1);
        if constexpr (i >= 5 && i < 13) {
          constexpr int l = i - 5;
          const uint32_t to = place(vt + (l >> 2) * (TILE / 2));
          if constexpr (first) {
            if constexpr ((l & 3) == 0) fetch4(rs, vt + (l >> 2) * (TILE / 2), voff + (l & 4));
          } else {
            LF_PRODUCT_AND_LOAD("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0", "+a", oacc[hh][mb], vf[u * MB + mb], "v",
                                __builtin_bit_cast(bf16x8, pv[hh][u]), rs, to, voff[l], l & 3)
          }
        } else if constexpr (!first) {
          accumulate(oacc[hh][mb], vf[u * MB + mb], __builtin_bit_cast(bf16x8, pv[hh][u]));
        }
        if constexpr (i < 12 && i % 3 != 2) kf[i - i / 3] = __builtin_bit_cast(bf16x8, k_next[kaddr[i - i / 3]]);
        if constexpr (i == 2) e_raw = st.ent[(t + 4) & (kEnt - 1)];
        // V of t - 1 is in registers (no reads of K follow in the last step: they are unused there)
        if constexpr (i == 4) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(last ? 0 : 5));
        soft(16 + i);
        sums(16 + i);
        __builtin_amdgcn_sched_barrier(0);
      };
      each_slot(value_slot, std::make_integer_sequence<int, 16>{});
      asm volatile("s_nop 4" : "+v"(l_run[0]), "+v"(l_run[1]));
      const unsigned long long far = __ballot(fmaxf(l_run[0][0], l_run[1][0]) > kSumMax);
      const int next_cnt = (int)(e1 & 63u);
      if (far != 0ull || next_cnt < 32) {
        if (far != 0ull) {
          settle();
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            if (__ballot(l_run[hh][0] > kSumMax) == 0ull) continue;
            const float m_new = fmaxf(m_run[hh], row_max(sc[hh]) * a.c);
            const float alpha = __builtin_amdgcn_exp2f(m_run[hh] - m_new);
            m_run[hh] = m_new;
            float l = l_old[hh] * alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
              for (int i = 0; i < 16; ++i) oacc[hh][mb][i] *= alpha;
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
              const float pa = __builtin_amdgcn_exp2f(fmaf(sc[hh][e], a.c, -m_new)), pb = __builtin_amdgcn_exp2f(fmaf(sc[hh][e + 1], a.c, -m_new));
              const bf16x2 pr = {(__bf16)pa, (__bf16)pb};
              pc[hh][e >> 3][(e & 7) >> 1] = __builtin_bit_cast(uint32_t, pr);
              l = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l, false);
            }
            l_run[hh][0] = l_run[hh][1] = l_run[hh][2] = l_run[hh][3] = l;
          }
          settle();
        }
        if (next_cnt < 32) mask(sn, next_cnt);
      }
      e0 = e1; e1 = e2; e2 = e3;
      e3 = __builtin_amdgcn_readfirstlane(t + 4 < nt ? e_raw : 0u);
      __builtin_amdgcn_sched_barrier(0);
    };
    const std::true_type yes{};
    const std::false_type no{};
    step(0, yes, no, st.k[1], st.k[0], st.v[1], s0, s1, p0, p1);
    int t = 1;
    for (; t + 1 < nt; t += 2) {
      step(t, no, no, st.k[0], st.k[1], st.v[0], s1, s0, p1, p0);
      step(t + 1, no, no, st.k[1], st.k[0], st.v[1], s0, s1, p0, p1);
    }
    if (t < nt) {
      step(t, no, yes, st.k[0], st.k[1], st.v[0], s1, s0, p1, p0);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) { p0[hh][0] = p1[hh][0]; p0[hh][1] = p1[hh][1]; }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    asm volatile("" ::: "memory");
    {
      const uint4* vt = st.v[(nt - 1) & 1];
#pragma unroll
      for (int i = 0; i < 2 * MB; ++i)
        vf[i] = __builtin_shufflevector(vread(vt, i >> 2, 0, i & 3), vread(vt, i >> 2, 1, i & 3), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int u = i >> 3, mb = (i >> 1) & 3, hh = i & 1;
        accumulate(oacc[hh][mb], vf[u * MB + mb], __builtin_bit_cast(bf16x8, p0[hh][u]));
      }
      settle();
    }
  }

#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    float l = l_run[hh][0];
    l += __shfl_xor(l, 32);
    const int row = 32 * hh + ln;
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    if (row < q_cnt) {
      if (a.lse2 != nullptr && kg == 0)
        a.lse2[(int64_t)h * a.q_len + qtok0 + row] = l > 0.0f ? m_run[hh] + __builtin_log2f(l) : INFINITY;
      uint16_t* op = a.O + (int64_t)h * a.o_stride_head + (int64_t)(qtok0 + row) * a.o_stride_tok;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 o4;
#pragma unroll
          for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(oacc[hh][mb][4 * g + e] * inv);
          *reinterpret_cast<bf16x4*>(op + 32 * mb + 8 * g + 4 * kg) = o4;
        }
    }
  }
}

}  // namespace

int lf_launch_attn_wide(const void* Q, const void* K, const void* V, const lf_shape* s, const lf_dims* dm,
                        const int32_t* indices, int32_t list_len, int32_t own_len, int blocks, float scale, void* O, float* lse2,
                        void* stream) {
  WideArgs a = {};
  a.Q = (const uint16_t*)Q;
  a.K = (const uint16_t*)K;
  a.V = (const uint16_t*)V;
  a.O = (uint16_t*)O;
  a.idx = indices;
  a.q_stride_tok = s->q_stride_tok;
  a.q_stride_head = s->q_stride_head;
  a.k_stride_head = s->k_stride_head;
  a.v_stride_head = s->v_stride_head;
  a.o_stride_tok = s->o_stride_tok;
  a.o_stride_head = s->o_stride_head;
  a.k_row_bytes = (uint32_t)(s->k_stride_tok * 2);
  a.v_row_bytes = (uint32_t)(s->v_stride_tok * 2);
  a.n = dm->n;
  a.nb = dm->nb;
  a.n_q = dm->n_q;
  a.n_k = dm->n_k;
  a.nb_inv = 0xffffffffu / (uint32_t)dm->nb;
  a.list_len = list_len;
  a.own_len = own_len;
  a.tail0 = dm->n_k - list_len;
  a.total = blocks;
  a.wg_per_xcd = (a.total + 7) / 8;
  a.c = scale * 1.4426950408889634f;
  a.lse2 = lse2;
  a.q_len = dm->f * dm->n;
  return lf_launch(lf_attn_wide_kernel, dim3((unsigned)(a.wg_per_xcd * 8)), dim3(64), 0, (hipStream_t)stream, a) == hipSuccess
             ? LF_OK : LF_ERR_HIP;
}
