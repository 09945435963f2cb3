// Rules that cut a call into launch sequences, free of HIP: a plain C++ program can run them over
// their whole range.
#pragma once
#include <algorithm>
#include <cstdint>

namespace vsp {

// Reads per launch sequence: at most 2^14 transformed selectors (2.4 GB of scratch) at a time. A ROM of one
// word has no address bits (v = 0).
inline uint64_t read_chunk(uint64_t R, uint32_t v) {
  return std::min<uint64_t>(R, std::max<uint64_t>(1, (1ull << 14) / std::max<uint32_t>(v, 1)));
}

}  // namespace vsp
