// Scratch of the multichannel density (host side).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace msx {

constexpr int64_t kDensityScratch = (int64_t)1 << 28;  // doubles (2 GiB)

// Doubles that the density keeps for calls of n events, in a context whose
// channels have up to `dims` dimensions and whose processes have up to `run`
// consecutive channels that share a launch: those channels' uniforms and
// Jacobians, but not more than kDensityScratch unless one channel alone needs
// more.  It depends on the context and n only and never falls with n: after one
// call, every call of as many events or fewer, of any process, finds its scratch
// in place, so work that was captured into a graph keeps valid memory through
// them.
inline int64_t density_scratch(int dims, int run, int64_t n) {
    const int64_t one = (int64_t)(dims + 1) * n;
    const int64_t fit = std::max<int64_t>(1, kDensityScratch / std::max<int64_t>(one, 1));
    return fit >= run ? run * one : std::max(one, kDensityScratch);
}

}  // namespace msx
