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
  int k_blocks; // retrieved blocks per list (0 without a budget)
  size_t off_qt, off_kt, off_kh, ws_bytes;
};

// Validates shape (and budget when non-NULL); returns LF_OK or an lf_status.
int lf_derive(const lf_shape* s, const lf_budget* b, lf_dims* out);

// Whether a query-major attention kernel divides each list in two parts, one for each pair of wavefronts of a workgroup.
// Two such blocks share a compute unit at d = 128 (three at d = 64), so that a call in which the undivided form, two blocks to a
// workgroup, leaves one wavefront on a SIMD has two there; with at most 256 blocks there is less to merge than with four parts.
// Forward, us, undivided or in four parts (where lf_split_lists says so) -> in two (random lists):
//   129 to 256 blocks: 200 blocks, d = 128, lists of 3: 10.6 -> 9.7, of 4: 11.5 -> 9.4, of 8: 12.4 -> 11.4, of 14: 16.2 -> 14.6, of 20: 17.8 ->
//     18.1, of 120: 63.7 -> 74.7; lists of 1: 0.96 - 1.00.  d = 64, of 4: 9.1 -> 7.4, of 8: 9.0 both, of 10: 10.7 -> 9.7, of 12: 10.3 -> 10.5, of 120: 44.7 -> 55.2;
//   257 to 512: d = 128, 260 blocks, of 7: 15.2 -> 16.0, of 8: 16.6 -> 15.9, of 32: 42.3 -> 33.5, of 64: 76.9 -> 56.2; 510 blocks, of
//     8: 20.3 -> 19.4, of 32: 49.1 -> 43.4, of 120: 143 -> 132.  d = 64, 260 blocks, of 5: 9.9 -> 10.2, of 8: 12.3 -> 11.0, of 32: 30.2 -> 23.8;
//     (Lists of 8 to 15 in 449 to 512 blocks would gain 3 - 10 %, but stay undivided, with the bits of the calls of 513 to 1 024 blocks.)
//   more: d = 128, 520 blocks, of 16: 36.5 -> 38.4.  d = 64, 580 blocks, of 1: 0.89, of 2: 1.06, of 3: 0.98, of 4: 1.10, of 32: 41.6 -> 33.0; 760 blocks,
//     of 8: 1.02, of 120: 137 -> 112; 780 (a second round), of 32: 0.93.
inline bool lf_two_parts(int d, int blocks, int list_len) {
  if (blocks <= 256) return list_len >= 2 && list_len <= (d == 128 ? 14 : 10);
  if (d == 128) return blocks <= 512 && list_len >= (blocks <= 448 ? 8 : 16);
  return blocks <= 768 && list_len >= (blocks <= 512 ? 6 : 2);
}
// dQ and the launch before it, us, likewise: 200 blocks, d = 128, lists of 3: 12.9 -> 13.4, of 4: 14.4 -> 13.5, of 8: 17.9 -> 16.6, of 14: 23.1 -> 21.3, of
// 20: 25.1 -> 25.8; 256 blocks, of 14: 26.7 -> 22.8, of 20: 29.6 -> 28.6; d = 64, 200 blocks, of 4: 11.6 -> 10.8, of 14: 19.9 -> 18.1, of 20: 21.7 -> 22.5.
// d = 128, 260 blocks, of 8: 26.1 -> 22.6, of 32: 67.6 -> 45.8; 510 blocks, of 7: 29.6 -> 30.3, of 8: 31.1 -> 30.4, of 32: 75.3 -> 62.3, of 120: 190 -> 187;
// 520, of 32: 75.1 -> 84.1.  d = 64, 510 blocks, of 8: 21.1 -> 21.2, of 12: 26.0 -> 25.7, of 32: 53.0 -> 49.4; 260, of 64: 92.0 -> 84.1; 520, of 32: 65.9 -> 74.3.
inline bool lf_two_parts_dq(int d, int blocks, int list_len) {
  if (blocks <= 256) return list_len >= 4 && list_len <= 14;
  return blocks <= 512 && list_len >= (d == 128 ? 8 : 10);
}
// Whether a query-major attention kernel divides each list among the four pairs of wavefronts of a
// workgroup instead of giving every (head, query block) one pair.  `blocks` is the number of
// these pairs, list_len the entries walked, n_k the KV blocks of a head.  A divided block has a compute unit (of 256)
// to itself, so with more than 256 of them the second round starts when the first ends, and the
// undivided form keeps more loads of one list's tiles in flight per compute unit.  lf_attn_form and lf_dq_form ask for row halves and two
// parts first, which leave to these two rules lists of more than 14 (at d = 64 the forward's of more than 10) in calls of 129 to 256 blocks; beyond
// 256 they are as they were before lists were divided in two, and decide nothing.
// Forward, d = 128, us undivided -> divided (random lists):
//   <= 256 blocks (up to 128 lf_halve_blocks comes first): 192 blocks, lists of 6: 13.6 -> 12.4; of 195: 222 -> 109; lists of 4 are one step a slice;
// Forward, d = 64: 208 blocks, lists of 52: 48 -> 23.
inline bool lf_split_lists(int d, int blocks, int list_len, int n_k) {
  if (blocks <= 256) return list_len >= 6;
  if (blocks > 512) return false;
  return d == 64 ? list_len >= 32 : list_len >= 96 && 2 * (int64_t)list_len >= n_k;
}
// Whether the two row halves of each (head, query block) get a workgroup each, and with it a compute unit: as
// long as there are no more of them than compute units.  us, one workgroup a block -> two, in a row of calls: 128 blocks, d = 128,
// lists of 2: 8.6 -> 7.6, of 6: 12.3 -> 9.3, of 32: 20.8 -> 16.8; d = 64, of 2: 6.6 -> 6.8, of 3: 7.4 -> 6.9, of 32: 15.0 -> 11.8; but
// 135 blocks (two rounds), d = 128, of 16: 16.1 -> 21.9; d = 64: 10.3 -> 15.8.
inline bool lf_halve_blocks(int d, int blocks, int list_len) { return blocks <= 128 && list_len >= (d == 128 ? 2 : 3); }
// dQ (backward call, the rest the same), d = 128: 132 blocks, lists of 6: 33.5 -> 34.6, of 8: 38.7 -> 34.4 (80 blocks);
// d = 64: 125 blocks, lists of 6: 29.7 -> 30.6; 78, of 7: 25.9 -> 24.9; 120, of 138: 213 -> 160.
inline bool lf_split_lists_dq(int d, int blocks, int list_len) {
  return (blocks <= 256 && list_len >= 7) || (d == 128 && blocks <= 512 && list_len >= 48);
}
// As lf_halve_blocks.  Backward call, one workgroup a block -> two: d = 128, 24 blocks, lists of 2: 21.5 -> 21.0, of 4: 24.1 -> 21.2, of
// 16: 32.5 -> 26.7, of 64: 60.9 -> 43.9; 128 blocks, of 2: 25.2 -> 26.2, of 4: 29.0 -> 27.4, of 32: 57.5 -> 52.7; d = 64, 128 blocks, of 4:
// 21.3 -> 23.1, of 6: 23.7 -> 23.3, of 32: 52.3 -> 43.1; 56 blocks, of 28: 45.9 -> 36.4.
inline bool lf_halve_blocks_dq(int d, int blocks, int list_len) { return blocks <= 128 && list_len >= (d == 128 ? 4 : 6); }

// How a query-major kernel takes the (head, query block) pairs of a launch, asked in this order.
//   LF_FORM_HALVES  the two row halves of a block get a workgroup each
//   LF_FORM_TWO, LF_FORM_FOUR  a workgroup a block, its list divided among two or four pairs of wavefronts
//   LF_FORM_WIDE    one wavefront a block (d = 128)
//   LF_FORM_BLOCK   a pair of wavefronts a block, lists undivided
enum lf_form { LF_FORM_HALVES, LF_FORM_TWO, LF_FORM_FOUR, LF_FORM_WIDE, LF_FORM_BLOCK };
// One wavefront per query block (lf_attn_wide.hip; d = 128): a SIMD holds one of its wavefronts, so it is
// the faster one where the last round of 1 024 query blocks is more than half full (the kernel of lf_attn.hip has room for 2 048
// wavefronts of half a block: its last round takes as long for one block as for 1 024), and its start and end count where lists
// are short.  How much faster, least and mean of 6 calls each, lists as selected: 513 to 768 blocks, lists of 16 to 23 and 24 to 31:
// 1.07, 1.09 and 1.08, 1.10; 769 to 1 024: 1.01, 1.04 and 1.02, 1.03; 1 537 to 1 792, of 16 to 23 and 32 to 63: 1.02, 1.03 and 1.02, 1.04;
// 1 793 to 2 048, of 16 to 23: 1.00, 1.02; 2 561 to 2 816: 1.00, 1.01; 2 817 to 3 072: 1.01, 1.03; 3 000, of 128: 740 -> 709 us; but 320, of
// 32: 42 -> 51 us; 1 281 to 1 536, of 16 to 63: 0.94, 0.96; 2 305 to 2 560: 0.94, 0.95; 769 to 1 024, of 1 to 9: 0.95, 0.98.
inline lf_form lf_attn_form(int d, int blocks, int list_len, int n_k) {
  if (lf_halve_blocks(d, blocks, list_len)) return LF_FORM_HALVES;
  if (lf_two_parts(d, blocks, list_len)) return LF_FORM_TWO;
  if (lf_split_lists(d, blocks, list_len, n_k)) return LF_FORM_FOUR;
  return d == 128 && list_len >= 16 && (blocks - 1) % 1024 >= 512 ? LF_FORM_WIDE : LF_FORM_BLOCK;
}
// Whether the full rounds of 1 024 query blocks of a call go to the kernel with one wavefront per block and the blocks past
// them, few enough to divide their lists, to a launch of their own.  Otherwise the call takes as long as one with a full last round.
// How much faster, least and mean (random lists, one and two full rounds before the others):
//   1 to 256 blocks past them:    lists of 16 to 23: 1.02, 1.13;  24 to 31: 1.06, 1.16;  32 to 63: 1.06, 1.20;  64 to 160: 1.09, 1.22
//   257 to 448 blocks past them:  lists of 9 to 13: 0.90, 0.93;  19 to 31: 1.00, 1.03;  41 to 130: 1.08, 1.11
// (1 050 blocks, lists of 188: 544 us as one launch, 431 as two.)  Lists of 8 to 15 would gain up to 17 % with few blocks past the rounds, but
// stay one launch, with the bits of the calls of 512 to 1 024 blocks.
inline bool lf_full_rounds_apart(int d, int blocks, int list_len) {
  const int past = blocks % 1024;
  return d == 128 && blocks > 1024 && past > 0 && past <= 448 && list_len >= (past <= 256 ? 16 : 32);
}
// Whether the dQ launch takes the kernel with one wavefront per query block (lf_attn_bwd_q_wide.hip): a SIMD holds one of its
// wavefronts, so the last round of 1 024 query blocks has to be filled well enough.  dQ with the launch before it, the
// kernel of lf_attn_bwd.hip against that one, lists of 8 and 150: 520 blocks 1.02, 1.07; 768: 1.05, 1.06; 1 024: 1.05, 1.04; 1 040: 0.95, 0.91; 1 200: 0.96,
// 1.02; 1 300: 1.03, 1.05; 1 500: 1.08, 1.09; 2 040: 1.18, 1.26; 2 060, of 8 and 64: 1.00, 0.99; 2 100: 1.03, 1.01; 3 016, of 8 and 150: 1.11, 1.13;
// 3 090, of 8 and 64: 1.01, 1.01.  At most 512 blocks: 0.95 .. 1.01.  Lists of 2 and 4: 520 blocks 0.99, 1.00; 1 300: 0.96, 0.98; 3 090: 1.03, 0.92.
inline bool lf_q_wide(int d, int blocks, int list_len) {
  if (d != 128 || list_len < 8 || blocks <= 512) return false;
  return blocks <= 1024 || (blocks - 1) % 1024 >= (blocks <= 2048 ? 256 : 48);
}
inline lf_form lf_dq_form(int d, int blocks, int list_len) {
  if (lf_halve_blocks_dq(d, blocks, list_len)) return LF_FORM_HALVES;
  if (lf_two_parts_dq(d, blocks, list_len)) return LF_FORM_TWO;
  if (lf_split_lists_dq(d, blocks, list_len)) return LF_FORM_FOUR;
  return lf_q_wide(d, blocks, list_len) ? LF_FORM_WIDE : LF_FORM_BLOCK;
}

// Which kernel computes dK and dV.  `blocks` is the number of (head, KV block) pairs; a KV block's list holds list_len n_q / n_k query
// blocks on the mean.
//   LF_KV_HALVES  the two row halves of a KV block get a workgroup each, of two groups of two wavefronts
//   LF_KV_GROUPS  a workgroup of two groups of four wavefronts, half of the block's list each
//   LF_KV_BLOCK   a workgroup of four wavefronts
//   LF_KV_WIDE    one wavefront per SIMD (lf_attn_bwd_wide.hip)
// Halves, as long as they bring compute units to work: at d = 128 one such workgroup fills a unit's LDS, at d = 64 two fit.  Backward call in us,
// halves and the faster one of BLOCK and GROUPS, on lists of equal length / random / skewed (every query block draws from the same popular blocks):
//   d = 64:  150 blocks, mean 16: 42.6, 42.0 / 46.3, 53.2 / 121.5, 165.4;  225 blocks, mean 8: 28.7, 28.9 / 31.1, 35.1 / 65.0, 85.8, mean 64: 118.8,
//     118.0 / 120.4, 125.9 / 128.0, 130.1;  256 blocks, mean 200: 345, 344 / 347, 355 / 384, 397;  350 blocks, mean 8: 40.3, 40.5 / 41.9, 44.3 / 71.8,
//     92.4, mean 64: 193, 207 / 193, 208 / 199, 213;  384 blocks, mean 11: 47.9, 47.3.
//     Past 256 blocks some units have more than two, and where lists hold a few query blocks each and most of all there are (so that
//     they hardly differ), halves take longer than BLOCK: mean up to 4, at least half of all: 1.07 to 1.11 times;  5 to 8, three quarters and more: 1.02
//     to 1.08, half to three quarters: 0.92 to 1.00;  9: 1.01, 0.90 to 0.97.
//   d = 128, halves in how much of the time of WIDE:  64 blocks, mean 16: 0.88 / 0.93 / 1.02;  128 blocks, mean 16: 0.88 / 0.92 / 1.05, mean 32: 0.95 / 0.98 /
//     1.07, mean 48: 0.99 / 1.00 / 1.06, mean 64: 1.02 / 1.02 / 1.06, mean 128: 1.06 / 1.05 / 1.05;  168 blocks, mean 14, of GROUPS: 58.0, 47.6.
// GROUPS, d = 128: such a workgroup has a compute unit (of 256) to itself.  Mean 12: 256 blocks 52.9 -> 50.4; of 24: 76.6 -> 70.0; two rounds, of 12: 384
//   blocks 59.5 -> 66.8.
// WIDE, d = 128: it has the shorter loop, but nobody works on its SIMDs while a list starts and ends.  So the lists have to be long enough, and longer
// where few blocks share the chip and the longest list decides.  How much faster the backward call is with it, lists as the mask
// selection makes them, least and mean of 2 to 13 calls:
//   129 to 256 blocks:      mean 9 to 11: 0.95, 1.02;  12 to 14: 0.97, 1.04;  18 to 20: 1.01, 1.06;  24 to 26: 1.10, 1.12;  36 to 38: 1.07, 1.11
//   257 to 512 blocks:      mean 9 to 11: 0.97, 1.01;  12 to 14: 0.99, 1.01;  15 to 17: 0.99, 1.01;  18 to 20: 1.01, 1.06;  24 to 26: 1.04, 1.05
//   513 to 768 blocks:      mean 9 to 11: 1.01, 1.03;  12 to 14: 0.98, 1.02;  15 to 17: 1.04, 1.07;  18 to 20: 1.02, 1.04;  33 to 35: 1.05, 1.09
//   769 to 1 024 blocks:    mean 9 to 11: 0.97, 1.00;  12 to 14: 1.00, 1.02;  15 to 17: 1.01, 1.04;  18 to 20: 1.00, 1.05;  27 to 29: 1.07, 1.09
//   1 025 to 1 280 blocks:  mean 9 to 11: 0.98, 1.02;  12 to 14: 1.04, 1.05;  15 to 17: 1.04, 1.05;  24 to 26: 1.04, 1.08;  33 to 35: 1.05, 1.08
//   1 281 to 1 536 blocks:  mean 9 to 11: 0.98, 1.00;  12 to 14: 1.02, 1.02;  18 to 20: 1.03, 1.04;  27 to 29: 1.06, 1.08
//   1 537 blocks and more:  mean 9 to 11: 0.98, 1.03;  12 to 14: 1.05, 1.06;  18 to 20: 1.02, 1.05;  30 to 32: 1.06, 1.07
enum lf_kv_form { LF_KV_HALVES, LF_KV_GROUPS, LF_KV_BLOCK, LF_KV_WIDE };
inline lf_kv_form lf_kv_form_of(int d, int blocks, int list_len, int n_q, int n_k) {
  const int64_t entries = (int64_t)list_len * n_q;      // mean list times n_k
  if (d == 64) {
    const bool few_and_all = (entries <= (int64_t)4 * n_k && (int64_t)2 * list_len >= n_k) ||
                             (entries <= (int64_t)8 * n_k && (int64_t)4 * list_len >= (int64_t)3 * n_k);
    return blocks <= 256 || (blocks <= 352 && !few_and_all) ? LF_KV_HALVES : LF_KV_BLOCK;
  }
  if (blocks <= 128) return entries >= (int64_t)48 * n_k ? LF_KV_WIDE : LF_KV_HALVES;
  if (entries >= (int64_t)(blocks <= 512 ? 18 : 15) * n_k) return LF_KV_WIDE;
  return blocks <= 256 ? LF_KV_GROUPS : LF_KV_BLOCK;
}

// Whether lf_sparse_attn_split computes the current chunk's blocks, n_q of them in every list, in a dense phase of their own, whose
// state the list-driven kernel goes on from.  The dense phase takes the chunk's tokens as one row of tiles.  One pass takes every
// query block as 64 rows and every KV block as whole half tiles of 32, so short frames that do not fill their blocks cost it
// `padded / n^2` of the work there (frames of 97 tokens 1.7 times, of 200 1.4, of 1 560 1.03).  Against that, two
// phases carry the state of every row through memory (as long as some 8 blocks of a list take), have two last rounds to fill, cannot divide
// lists among wavefronts, and at d = 128 have the slower kernel for them, a share of the whole list that falls with the number of query blocks.
// The line: 17 500 random calls, both ways each (mean, and worst, of what the slower choice would cost where this one is wrong):
//   d = 128: 257 to 512 query blocks 0.0002, 0.05;  513 to 1 280: 0.003, 0.15;  more: 0.003, 0.10;  up to 256 one pass is always faster;
//   d = 64:  257 to 768: 0.0003, 0.10;  more: 0.002, 0.17.
// Time of one pass to that of two phases: frames of 97 tokens, chunk of 300 blocks, lists of 30 beside it, 1 500 query blocks: 1.27 (d = 64: 1.29);
//   frames of 200, calls of more than 2 048: up to 1.2 (1.3), of 513 to 640: 0.7 to 1.1;  of 33: up to 2.0 (2.3);
//   whole frames, d = 128: 75 blocks 0.75 to 0.95 (3 000 query blocks), 225: 1 125 query blocks 0.76, 1 800 0.93, 4 725 0.95, 300: 1 200
//   0.81, 2 100 0.85, 6 000 0.97, but 1 500 1.01;  d = 64: 225: 675 0.75, 900 0.97, 2 700 0.99, 4 725 1.00.
inline bool lf_two_phases(const lf_dims& m) {
  const int blocks = m.H * m.n_q;
  if (blocks <= 256) return false;
  const double padded = 64.0 * m.nb * 32.0 * ((m.n + 31) / 32);
  const double saved = m.n_q * (1.0 - (double)m.n * m.n / padded);      // blocks of the list
  const double slower = m.d == 128 ? (blocks <= 512 ? 0.4 : blocks <= 1280 ? 0.15 : 0.07) : blocks <= 768 ? 0.4 : 0.0;
  return saved > 8.0 + slower * (m.n_q + m.k_blocks);
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
// The first `blocks` query blocks of a call at d = 128 with one wavefront each; entries from own_len on are the cache's last blocks, unread.
int lf_launch_attn_wide(const void* Q, const void* K, const void* V, const lf_shape* s, const lf_dims* dm,
                        const int32_t* indices, int32_t list_len, int32_t own_len, int blocks, float scale, void* O, float* lse2,
                        void* stream);
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
