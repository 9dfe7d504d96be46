// Cursor words of the deposit records (plain C++, no HIP types): segment << 32
// | count.  A deposit adds 1 to its bucket's cursor; a count below kLogSeg is
// its place in the segment, the one that finds kLogSeg installs the workgroup's
// next segment as (segment << 32 | 1), the others add again or, at the latest
// when the workgroup has no segment left, go to the tally.
//
// Counts past kLogSeg keep growing then, by one per deposit, and must not carry
// into the segment number: how many deposits a workgroup makes has no bound
// that the host could check (a history may scatter up to half a million times).
// So a deposit that goes to the tally and found the count at kCursorHigh or
// above replaces the word it left by cursor_full of it, with a compare and
// exchange: nothing happens where another deposit has moved the word meanwhile
// (a newly installed segment is never lost), and the last one to add succeeds.
#pragma once

#include <cstdint>

namespace ctd {

constexpr uint32_t kLogSeg = 256;            // records of a segment
constexpr uint32_t kCursorHigh = 1u << 31;

// The same segment, full and past the deposit that installs the next one.
constexpr unsigned long long cursor_full(unsigned long long w) {
  return (w >> 32) << 32 | (kLogSeg + 1u);
}

}  // namespace ctd
