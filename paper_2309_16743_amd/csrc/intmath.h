// Integer helpers, free of HIP.
#pragma once

#include <cstdint>

namespace ot {

inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace ot
