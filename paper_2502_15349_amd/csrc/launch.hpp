// How many workgroups one launch may have.
#pragma once
#include <stdint.h>

namespace ae {
// The runtime counts the threads of a launch in 32 bits and, beyond them, launches the remainder without an error.
inline bool launch_fits(int64_t workgroups, int threads) { return workgroups > 0 && workgroups * threads <= 0xffffffffLL; }
}  // namespace ae
