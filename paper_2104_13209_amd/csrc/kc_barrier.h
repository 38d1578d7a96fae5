// Arrival counts of a barrier (plain C++: also compiled by the host compiler alone).
#pragma once

namespace kc {

// Whether a barrier that waits for `want` arrivals since the launch still misses some, with
// both counts modulo 2^32: they differ by less than a grid's blocks, and a launch may have
// more than 2^31 arrivals (64 blocks: 33.5 million rounds, half the vertices of a path).
constexpr bool arrivals_missing(unsigned int arrived, unsigned int want) {
    return static_cast<int>(arrived - want) < 0;
}

}  // namespace kc
