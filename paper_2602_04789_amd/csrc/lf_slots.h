// Helpers of the kernels that are inline assembly in part, first of all those whose loop is written as slots of one matrix
// instruction each.
//
// The products of the latter, and in part their vector instructions, are inline assembly, which keeps its place.  The compiler knows neither
// their latency nor the wait states between them: a product may read what a vector instruction wrote three instructions before at
// the earliest (two in between), and a vector instruction a product's result 11 wait states behind it (4 x 4 x 4: 5); other
// registers that a product starts from may be overwritten seven behind it.  The loops are written with more than that in between, and copies that the compiler puts in are what a test of the assembly looks for.
#ifndef LF_SLOTS_H
#define LF_SLOTS_H

#include <type_traits>
#include <utility>

// f(0), f(1), ... with the index a constant
template <typename F, int... I>
__device__ __forceinline__ void each_slot(const F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// A load's resource, old enough to be read in inline assembly: a memory instruction may read a scalar register five wait states behind
// the vector instruction (v_readfirstlane) that wrote it.  The compiler counts them ahead of its own loads, not into a block of
// assembly.  Three stand here, two at the head of the block (M0 and the wait behind it).
template <typename Resource>
__device__ __forceinline__ Resource aged(Resource rs) {
  asm volatile("s_nop 2" : "+s"(rs));
  return rs;
}

// The product `op` on c, x, y with load j (of four, 1 KB each) of a tile part behind it: resource rs, LDS base lds0, offset o.  The first
// load sets M0, the product standing between that and the load; nothing else in these loops writes M0.
#define LF_PRODUCT_AND_LOAD(op, cons, c, x, ycons, y, rs, lds0, o, j)                                                                 \
  if constexpr ((j) == 0)                                                                                                             \
    asm volatile("s_mov_b32 m0, %3\n\t" op "\n\tbuffer_load_dwordx4 %4, %5, 0 offen lds"                                                \
                 : cons(c) : "v"(x), ycons(y), "s"(lds0), "v"(o), "s"(rs) : "memory", "m0");                                            \
  else                                                                                                                                \
    asm volatile(op "\n\tbuffer_load_dwordx4 %3, %4, 0 offen offset:%5 lds"                                                             \
                 : cons(c) : "v"(x), ycons(y), "v"(o), "s"(rs), "n"((j) * 1024) : "memory");

#endif
