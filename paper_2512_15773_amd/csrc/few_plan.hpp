// Host-side rules of the spread forward pass (few_rows.hpp); plain C++ without HIP.
#pragma once
#include <algorithm>
#include <cstddef>

namespace tsdp {

// Rows below this one a launch may start to read before it knows how many rows are live.  In the context's own row
// buffers any row up to their capacity exists, and every running environment has one: the loads of the first B rows travel
// together with the live row count.  A caller's buffers hold the live rows and no more -- finished environments own none,
// so not even the first B need exist -- and nothing of them is read before the count is known.
inline int few_safe_rows(bool own_rows, int B, int R_cap) { return own_rows ? std::min(B, R_cap) : 0; }

// Floats of the two residual and of the two partial-sum buffers, shared by both networks.  Which networks take the spread
// path can change with every tsdp_load_weights, so what a context holds is compared with what its networks need now, and
// replaced by a larger buffer where it is too small.
struct FewShape { bool few; size_t d, slices; };
struct FewSize { size_t h = 0, part = 0; };
inline FewSize few_size(size_t tokens, const FewShape& base, const FewShape& draft) {
  FewSize z;
  for (const FewShape* n : {&base, &draft})
    if (n->few) {
      z.h = std::max(z.h, tokens * n->d);
      z.part = std::max(z.part, tokens * n->d * n->slices);
    }
  return z;
}
inline bool few_fits(const FewSize& have, const FewSize& need) { return need.h <= have.h && need.part <= have.part; }

}  // namespace tsdp
