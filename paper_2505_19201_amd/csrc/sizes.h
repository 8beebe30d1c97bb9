// Arithmetic on sizes, for the host.
#pragma once
#include <cstddef>
#include <cstdint>

namespace dream {

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

}  // namespace dream
