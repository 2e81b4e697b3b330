// The parts of the kernels' requests to memory that a host program can run against a model (tests/schedule_driver.cpp):
// the order of requests and waits of the small-batch form whose activations are streamed through registers (sfmp_decode.hip,
// RS), and what a copy of an activation block asks for (sfmp_prefill.hip).
#pragma once

#include <stdint.h>

#if defined(__HIP__)
#define SFMP_SCHEDULE_FN __device__ __forceinline__
#else
#define SFMP_SCHEDULE_FN inline
#endif

namespace sfmp {

template <int V>
struct Const {
  static constexpr int value = V;
};

// Walks `count` >= 1 tile columns with three register sets for the activations and three ring slots for the slabs.
// Requests complete in the order in which they were made.
//   load(Const<set>, i)    requests the activations of column i (the caller substitutes the last column for i >= count)
//   copy(Const<slot>, i)   requests the slabs of column i
//   wait(columns)          returns once at most so many of the youngest requests are outstanding: the activations of
//                              one column and the slabs of `columns` columns (0 or 1)
//   use(Const<set>, i)     consumes column i: the activations of set i mod 3, the slabs of slot i mod 3
//   keep_loads()           consumes all three sets
// A(i) before D(i), in the order A(0) A(1) D(0) A(2) D(1) A(3) D(2) ...: the wait for D(i), counted here, is stricter than
// the one for A(i), which the compiler counts without knowing of the copies.  The loads past the last column are counted
// like the others, so they have to be made: their values are consumed at the end, as a compiler may leave out or move a load
// whose value nobody reads, and a wait that counts it would then return before the slabs have landed.
template <class Load, class Copy, class Wait, class Use, class Keep>
SFMP_SCHEDULE_FN void stream_columns(const int count, const Load& load, const Copy& copy, const Wait& wait, const Use& use,
                                     const Keep& keep_loads) {
  load(Const<0>(), 0);
  load(Const<1>(), 1);
  copy(Const<0>(), 0);
  load(Const<2>(), 2);
  if (count > 1) copy(Const<1>(), 1);
  auto column = [&](int i, auto set) __attribute__((always_inline)) {
    constexpr int s = decltype(set)::value;
    // D(i) has landed once only A(i+2) and D(i+1) (if there is one) are outstanding
    wait(i + 1 < count ? 1 : 0);
    use(set, i);
    load(set, i + 3);
    if (i + 2 < count) copy(Const<(s + 2) % 3>(), i + 2);
    return i + 1 < count;
  };
  for (int i = 0;; i += 3) {
    if (!column(i, Const<0>())) break;
    if (!column(i + 1, Const<1>())) break;
    if (!column(i + 2, Const<2>())) break;
  }
  keep_loads();
}

// Copy of the activation block of one tile column through a raw buffer descriptor: scalar offset and number of records
// (bytes).  Past the end (of a schedule that makes the same number of copies in every step) a request of nothing: no
// records and no scalar offset, out of range whether or not the scalar offset counts in the range check.
struct BlockRequest {
  uint32_t offset, records;
};
SFMP_SCHEDULE_FN BlockRequest block_request(const uint32_t column_offset, const uint32_t bytes, const bool wanted) {
  return BlockRequest{wanted ? column_offset : 0u, wanted ? bytes : 0u};
}

}  // namespace sfmp
