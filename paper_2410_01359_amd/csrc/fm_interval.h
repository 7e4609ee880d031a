// A masked row interval [start, end) of a key as the dK/dV loop's element mask tests it: one subtraction and one
// comparison per row, in unsigned arithmetic, because the distance between a row and a bound (any int32 value) may not
// fit an int.  Plain integer code: the host compiles it too.
#pragma once

#if defined(__HIP__)
#define FM_HOST_DEVICE __host__ __device__
#else
#define FM_HOST_DEVICE
#endif

// Rows of the interval, 0 for an empty one.
FM_HOST_DEVICE inline unsigned interval_length(int start, int end) {
  return end > start ? (unsigned)end - (unsigned)start : 0u;
}
// Where `row` lies from the interval's start (modulo 2^32).  A row `dr` further on lies at offset + dr.
FM_HOST_DEVICE inline unsigned interval_offset(int row, int start) { return (unsigned)row - (unsigned)start; }
// Whether the row at this offset lies in the interval.
FM_HOST_DEVICE inline bool in_interval(unsigned offset, unsigned length) { return offset < length; }
