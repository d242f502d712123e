// Integer arithmetic of host code that also has to compile without the HIP headers.
#pragma once

#include <stdint.h>

namespace kvp {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace kvp
