// fill.h -- the -inf fill of one group of eight logits (grid_apply).
#pragma once
#include <cstdint>

#include "lexhash.h"

namespace grid {

template <typename T>
struct __attribute__((packed, aligned(sizeof(T)), may_alias)) Logits16 {  // 16 bytes of logits
  uint32_t w[4];
};

// Eight logits at p, n of them in the row; bit j of bits keeps logit j.  A whole
// group takes 16-byte stores, at whatever element it starts (the memory takes a
// 16-byte access at any element).  In aligned rows that includes a group with
// kept logits, which are read first and written back unchanged; in rows that are
// not aligned a kept logit is never written, so there such a group, like one at a
// ragged row end, is written logit by logit.
template <typename T>
GRID_HD void fill_group(T* p, uint32_t bits, int n, bool aligned, uint32_t neg_inf_bits) {
  if (n >= 8 && (aligned || bits == 0u)) {
    Logits16<T>* q = reinterpret_cast<Logits16<T>*>(p);
    if (sizeof(T) == 2) {
      Logits16<T> v = {{0, 0, 0, 0}};
      if (bits) v = q[0];
      for (int k = 0; k < 4; ++k) {
        const uint32_t lo = (bits >> (2 * k)) & 1u ? v.w[k] & 0xFFFFu : neg_inf_bits;
        const uint32_t hi = (bits >> (2 * k + 1)) & 1u ? v.w[k] & 0xFFFF0000u : neg_inf_bits << 16;
        v.w[k] = lo | hi;
      }
      q[0] = v;
    } else {
      Logits16<T> v0 = {{0, 0, 0, 0}}, v1 = v0;
      if (bits & 0x0Fu) v0 = q[0];
      if (bits & 0xF0u) v1 = q[1];
      for (int k = 0; k < 4; ++k) {
        v0.w[k] = (bits >> k) & 1u ? v0.w[k] : neg_inf_bits;
        v1.w[k] = (bits >> (4 + k)) & 1u ? v1.w[k] : neg_inf_bits;
      }
      q[0] = v0;
      q[1] = v1;
    }
    return;
  }
  for (int j = 0; j < 8 && j < n; ++j)
    if (!((bits >> j) & 1u)) p[j] = (T)neg_inf_bits;
}

}  // namespace grid
