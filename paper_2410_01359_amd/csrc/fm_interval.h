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
// The next 32 rows at once: bit p tells whether the row p further on than this offset lies in the interval.  (An interval
// that starts at or before the first row reaches past none of them or `length - offset` of them; one that starts later
// starts -offset rows on, modulo 2^32.  first_row + 31 and the bounds are int32 values, so neither sum wraps.)
FM_HOST_DEVICE inline unsigned interval_rows(unsigned offset, unsigned length) {
  const unsigned first = in_interval(offset, length) ? 0u : 0u - offset, end = length - offset;
  const unsigned from_first = (unsigned)(0xFFFFFFFFull << (first < 32 ? first : 32));
  const unsigned from_end = (unsigned)(0xFFFFFFFFull << (end < 32 ? end : 32));
  return from_first & ~from_end;
}
