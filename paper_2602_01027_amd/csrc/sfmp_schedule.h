// The parts of the kernels' requests to memory that a host program can run against a model (tests/schedule_driver.cpp):
// the order of requests and waits of the small-batch form whose activations are streamed through registers (sfmp_decode.hip,
// RS), and what the copies of activation blocks ask for and which blocks a workgroup owns (sfmp_prefill.hip).
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

// Division by a number that the host knows: a few scalar instructions where the compiler's own goes through vector floats.
struct Divisor {
  uint32_t by, inverse;  // floor(2^32 / by), 2^32 - 1 for one: the estimate is right or one too small
};
inline Divisor divisor(const uint32_t by) { return Divisor{by, by == 1 ? 0xFFFFFFFFu : (uint32_t)(((uint64_t)1 << 32) / by)}; }
struct Quotient {
  uint32_t q, rest;
};
SFMP_SCHEDULE_FN Quotient divide(const uint32_t x, const Divisor d) {
  const uint32_t q = (uint32_t)(((uint64_t)x * d.inverse) >> 32), rest = x - q * d.by;
  return rest >= d.by ? Quotient{q + 1, rest - d.by} : Quotient{q, rest};
}

// The work items of a product of ntr tile rows and n_mtiles blocks of activation rows, in `ksplit` K ranges: the ranges innermost,
// then M blocks inside tile rows - all of them, or (grouped) kMGroup at a time, the last group being what is left.
constexpr uint32_t kMGroup = 8;
struct Place {
  int ks, mt, tr;
};
struct WorkItems {
  uint32_t whole;                  // M blocks in whole groups
  uint32_t by_ranges, by_group;    // inverses of the K ranges and of the items of a whole group
  Divisor last;                    // M blocks of the last (or only) group

  SFMP_SCHEDULE_FN Place place(const uint32_t block, const uint32_t ntr, const uint32_t ksplit) const {
    const Quotient k = divide(block, Divisor{ksplit, by_ranges});
    const uint32_t whole_items = whole * ntr;
    const bool in_whole = k.q < whole_items;
    const Quotient d = divide(k.q - (in_whole ? 0u : whole_items), in_whole ? Divisor{kMGroup * ntr, by_group} : last);
    return Place{(int)k.rest, (int)(in_whole ? d.q * kMGroup + d.rest % kMGroup : whole + d.rest), (int)(in_whole ? d.rest / kMGroup : d.q)};
  }
};
inline WorkItems work_items(const uint32_t ntr, const uint32_t n_mtiles, const uint32_t ksplit, const bool grouped) {
  const uint32_t whole = grouped ? n_mtiles / kMGroup * kMGroup : 0u, left = n_mtiles - whole;
  return WorkItems{whole, divisor(ksplit).inverse, divisor(kMGroup * ntr).inverse, divisor(left ? left : 1u)};
}

// What a workgroup with BM rows of the batch from row m0 on (a multiple of BM) copies of the staged activations, which lie in
// blocks of 128 rows (block_bytes = K * 256 each, 256 bytes per row and tile column): copies of 8 rows, no more row blocks than
// there are.
template <int BM>
struct StagedRows {
  static constexpr int kBlock = 128;
  static constexpr bool kInside = kBlock % BM == 0, kWhole = BM % kBlock == 0;  // the rows lie in one block; they start one
  int64_t base;  // first byte of the range in the staged activations
  int rows;      // rows of the row blocks that the workgroup's rows reach into, as far as they are there
  uint32_t bytes, block_bytes;
  int first;     // the workgroup's first row, counted from `base` (where the rows may cross from block to block)

  SFMP_SCHEDULE_FN StagedRows(const int M, const int m0, const uint32_t bytes_of_block) {
    block_bytes = bytes_of_block;
    const int sub = kInside ? m0 % kBlock : 0;
    first = kInside || kWhole ? 0 : m0 % kBlock;
    base = (int64_t)(m0 / kBlock) * block_bytes + sub * 256;
    // at most three blocks of 14.7 MB (all that are left, in bytes, pass 32 bits from M * K = 2^31 on)
    const int left = (M + kBlock - 1) / kBlock - m0 / kBlock, reached = kInside ? 1 : (first + BM + kBlock - 1) / kBlock;
    const int blocks = left < reached ? left : reached;
    rows = blocks * kBlock;
    bytes = (uint32_t)blocks * block_bytes - (uint32_t)sub * 256u;
  }
  // Rows `row` ... `row` + 7 of the workgroup in tile column 0: offset from `base` and records (none: rows that are not there)
  SFMP_SCHEDULE_FN BlockRequest copy(const int row) const {
    const int r = first + row;
    const bool there = r < rows;
    return BlockRequest{there ? (uint32_t)(r / kBlock) * block_bytes + (uint32_t)(r % kBlock) * 256u : 0u, there ? bytes : 0u};
  }
};

}  // namespace sfmp
