// Arithmetic of the list builders' counts and prefix sums (plain C++, also
// compiled for the host by its test).
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define PSE_LIST_FN __host__ __device__ __forceinline__
#else
#define PSE_LIST_FN inline
#endif

namespace pse {

// Row starts are 32-bit.  Sums stay at LIST_MAX once they reach it instead of
// wrapping: N coincident spheres have N (N - 1) pairs, beyond 2^31 from N =
// 46342 on, and so have positions that are all non-finite (each is taken as
// 0).  Some room is left below 2^31 for the readers, which look up to a
// group's width past a row's start.  A list whose total is LIST_MAX is too
// long for any storage.
constexpr int LIST_MAX = 0x7fffff00;

// a + b for a and b in [0, LIST_MAX]; associative, so any order of a scan
// gives the same sums.
PSE_LIST_FN int list_add(int a, int b) {
  const uint32_t s = (uint32_t)a + (uint32_t)b;
  return s < (uint32_t)LIST_MAX ? (int)s : LIST_MAX;
}

// Entries that a list of capacity cap can hold.
PSE_LIST_FN int list_limit(int64_t cap) { return cap < LIST_MAX ? (int)cap : LIST_MAX; }

// Slot of a row's entry `rank`, or -1 where the list (limit entries) ends
// before it.
PSE_LIST_FN int list_slot(int start, int rank, int limit) {
  return rank < limit - start ? start + rank : -1;
}

// End of the row whose successor starts at `next`: no entry at or beyond the
// limit was written.
PSE_LIST_FN int list_row_end(int next, int limit) { return next < limit ? next : limit; }

}  // namespace pse
