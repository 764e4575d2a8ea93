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

}  // namespace tsdp
