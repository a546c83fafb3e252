// How one copy of optimizer state between pinned host memory and HBM is handed to the runtime (state_copy in model.hip).
// Host arithmetic only, so that every size can be checked without a GPU.
#pragma once
#include <stddef.h>

namespace hift {

// A part is at most this long and goes as a rectangle of two rows, so a row is at most 128 MiB: far below the widest pitch that
// a rectangle may have (2^31 - 1 bytes) and the 32-bit extents that it becomes further down, however much state a group has.
// Each part leaves the link idle for a few microseconds.  A sweep of two layers of width 4096 with their state on the host (21 GB
// over the link): 115.9 ms with rectangles of any size, 116.1 with these parts; with parts of 64 MiB 117.5 against 116.7.
constexpr size_t COPY_PART_MAX = size_t(256) << 20;
constexpr size_t COPY_RECT_MIN = size_t(64) << 10;  // shorter pieces: one plain copy

// fn(offset, row, n) for every part, in order: n bytes from `offset` on, as a rectangle of two rows of `row` bytes that follow
// each other, or as a plain copy where row is 0.  The first result other than 0 ends the walk and is returned.
template <class F>
int copy_parts(size_t bytes, F fn) {
  for (size_t at = 0; at < bytes;) {
    const size_t part = bytes - at < COPY_PART_MAX ? bytes - at : COPY_PART_MAX;
    const size_t row = part >= COPY_RECT_MIN ? part / 32 * 16 : 0;  // 16-byte rows; less than 32 bytes remain
    const size_t n = row ? 2 * row : part;
    if (const int e = fn(at, row, n)) return e;
    at += n;
  }
  return 0;
}

}  // namespace hift
