// Positions in lists of fewer than 2^31 entries, free of HIP so that they are
// tested on the host.
#pragma once

namespace slg {

// Halfway between positions (their sum can pass 2^31).
constexpr int middle(int lo, int hi) { return (int)(((unsigned)lo + (unsigned)hi) >> 1); }

}  // namespace slg
