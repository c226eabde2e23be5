// Positions in lists of fewer than 2^31 entries, free of HIP so that they are
// tested on the host.
#pragma once

namespace slg {

// Halfway between positions (their sum can pass 2^31).
constexpr int middle(int lo, int hi) { return (int)(((unsigned)lo + (unsigned)hi) >> 1); }

// First position of the aligned block of eight that holds p, or of the one
// `ahead` blocks on (which can start at 2^31).
constexpr unsigned block_at(unsigned p, unsigned ahead = 0) { return (p & ~7u) + 8u * ahead; }

}  // namespace slg
