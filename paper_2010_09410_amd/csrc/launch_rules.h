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

// Copies of the bootstrapping key for gates that each read their own (vsp_gates_key_copies). A call is taken
// when 61.9 MB for every copy asked for (none for a single one, the context's key) and 1 GiB are free.
constexpr uint64_t kKeyCopyAsked = 630ull * 2 * 3 * 2 * 1024 * 8;
inline bool key_copies_accepted(uint64_t copies, uint64_t free_bytes) {
  return (copies > 1 ? copies * kKeyCopyAsked : 0) + (1ull << 30) <= free_bytes;
}
// How many are made, with `free_bytes` left for them: no form of the blind rotation holds more than `held` gates
// at once, so more add nothing; a copy takes more than it is asked for, so there may be room for fewer.
inline uint64_t key_copies_made(uint64_t copies, uint64_t held, uint64_t free_bytes, uint64_t key_bytes) {
  constexpr uint64_t tables = 32ull << 20;  // a pointer per copy and two bytes per gate
  const uint64_t room = free_bytes > tables ? (free_bytes - tables) / key_bytes : 0;
  return std::max<uint64_t>(1, std::min({copies, held, room}));
}

}  // namespace vsp
