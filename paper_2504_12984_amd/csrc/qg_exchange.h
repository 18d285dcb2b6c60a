// Split-K of the streaming kernels: the slabs of a strip meet in a binary tree of exchanges.
//
// Workgroups meet pairwise, element by element: each swaps its partial sums into the pair's slot
// (device-scope atomics, which work on memory shared by the XCDs) and looks at what was there.  Nothing
// (zero): it came first and is done with that element.  The other one's sums: it came second, adds
// them -- lower slab first, so the result does not depend on who came when --, empties the slot for the next
// call and goes up one level; who wins the root stores the result.  Nobody waits, and a level is one trip
// to memory where storing partial sums, counting arrivals and reading back are three (M = 1,
// K = N = 4096, u4: 7.0 us -> 5.8; M = 16, K = 14336, N = 4096 in four slabs: 11.4 -> 10.2; with
// 32 rows 2 %, with 64 rows 4 to 9 % longer: too many sums for exchanges of 8 bytes, so up to two row tiles).
// Sums travel complemented, two to an exchange where a thread has two; the one NaN pattern
// that would read as nothing is replaced by another.
#pragma once
#include <type_traits>

#include "qg_common.h"

namespace qg {

__device__ __forceinline__ uint32_t exchange_code(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  return u == 0xffffffffu ? 0x80000000u : ~u;                   // never zero
}

// sum[mt][e]: column offset idx0 + e of row tile mt, lane l, strip nc; live[mt][e / PAIR]: rows to exchange on
// entry, sums that are complete and mine to store on return.  Returns whether any are.
// Slots: (splitk - 1) nodes of the tree x NCH strips x MT * 1024 sums.
template <int MT, int PER>
__device__ __forceinline__ bool tree_exchange(float (&sum)[MT][PER], bool (&live)[MT][PER >= 2 ? PER / 2 : 1], void* slots,
                                              int nc, int NCH, int slab, int splitk, int idx0, int l) {
  constexpr int PAIR = PER >= 2 ? 2 : 1, NP = PER / PAIR;
  typedef std::conditional_t<PAIR == 2, unsigned long long, uint32_t> slot_t;
  slot_t* level = reinterpret_cast<slot_t*>(slots) + (int64_t)nc * (MT * 1024 / PAIR) + (idx0 / PAIR) * 64 + l;
  const int64_t node = (int64_t)NCH * (MT * 1024 / PAIR);       // slots of one node of the tree, all strips
  bool any = true;
  for (int n = splitk, s = slab; n > 1; level += (n >> 1) * node, n = (n + 1) >> 1, s >>= 1) {
    if (s == n - 1 && (n & 1)) continue;                        // the odd one out has no partner on this level
    slot_t* slot = level + (s >> 1) * node;
    slot_t other[MT][NP];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        other[mt][q] = 0;
        if (live[mt][q]) {
          slot_t v = exchange_code(sum[mt][PAIR * q]);
          if constexpr (PAIR == 2) v |= (slot_t)exchange_code(sum[mt][PAIR * q + 1]) << 32;
          other[mt][q] = __hip_atomic_exchange(slot + (mt * (16 / PAIR) + q) * 64, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    any = false;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        live[mt][q] = other[mt][q] != 0;
        any |= live[mt][q];
        if (live[mt][q]) {
#pragma unroll
          for (int x = 0; x < PAIR; ++x) {
            const float o = __builtin_bit_cast(float, ~(uint32_t)(other[mt][q] >> (PAIR == 2 ? 32 * x : 0)));
            float& own = sum[mt][PAIR * q + x];
            own = (s & 1) ? o + own : own + o;
          }
          __hip_atomic_store(slot + (mt * (16 / PAIR) + q) * 64, (slot_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    if (!any) break;
  }
  return any;
}

}  // namespace qg
