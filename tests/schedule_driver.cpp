// Host checks of csrc/sfmp_schedule.h.
//
// The schedule of the streamed-activation form against a model of a wavefront's memory queue: requests complete in order, a
// wait returns with as many outstanding as it allows.  A load whose value nothing reads may not be made at all (a compiler
// may leave it out), so every walk is checked with those loads and without them.
//
// Copies of activation blocks against the range check of a raw buffer, with the scalar offset counted in it and not: what is
// wanted is read from inside the row block, and nothing is read past the end.  And the copies of a workgroup's rows, which may
// lie in two or three row blocks of a batch of any length: the bytes that are meant, inside the staged activations.  And the
// numbering of the work items.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2602_01027_amd/csrc/sfmp_schedule.h"

struct Event {
  enum Kind { kLoad, kCopy, kWait, kUse, kKeep } kind;
  int place;   // set or slot (kWait: columns)
  int column;
  bool read;   // kLoad: something consumes the value
};

static void fail(const char* what, int count, int slabs, bool unread, int column) {
  std::printf("%s: %d columns, %d slabs, unread loads %s, column %d\n", what, count, slabs, unread ? "made" : "left out", column);
  std::exit(1);
}

static void check(const std::vector<Event>& events, int count, int slabs, bool unread) {
  std::vector<int> requests;  // the queue: one entry per instruction, +column + 1 for slabs, -(column + 1) for activations
  size_t complete = 0;        // how many of them are known to have completed
  int in_set[3] = {-1, -1, -1}, in_slot[3] = {-1, -1, -1}, next = 0;
  bool set_free[3] = {true, true, true}, slot_free[3] = {true, true, true};
  for (const Event& e : events) {
    switch (e.kind) {
      case Event::kLoad:
        if (!set_free[e.place]) fail("set overwritten before its use", count, slabs, unread, e.column);
        in_set[e.place] = e.column, set_free[e.place] = e.column >= count;
        if (e.read || unread) requests.insert(requests.end(), 4, -(e.column + 1));
        break;
      case Event::kCopy:
        if (!slot_free[e.place]) fail("slot overwritten before its use", count, slabs, unread, e.column);
        in_slot[e.place] = e.column, slot_free[e.place] = false;
        requests.insert(requests.end(), 2 * slabs, e.column + 1);
        break;
      case Event::kWait: {
        const size_t allowed = 4 + 2 * (size_t)slabs * e.place;
        if (requests.size() > allowed && requests.size() - allowed > complete) complete = requests.size() - allowed;
        break;
      }
      case Event::kUse:
        if (e.column != next++) fail("columns out of order", count, slabs, unread, e.column);
        if (in_set[e.place] != e.column || in_slot[e.place] != e.column) fail("another column's data", count, slabs, unread, e.column);
        for (size_t r = complete; r < requests.size(); ++r)
          if (requests[r] == e.column + 1) fail("slabs used before they have landed", count, slabs, unread, e.column);
        set_free[e.place] = slot_free[e.place] = true;
        break;
      case Event::kKeep:
        break;
    }
  }
  if (next != count) fail("columns left out", count, slabs, unread, next);
}

static void check_block_requests() {
  constexpr uint32_t kBlock = 32768;  // bytes of a tile column's block of 128 rows
  for (uint32_t ntc : {1u, 8u, 57u, 448u})
    for (uint32_t tc = 0; tc < ntc; ++tc)
      for (bool wanted : {true, false}) {
        const sfmp::BlockRequest x = sfmp::block_request(tc * kBlock, ntc * kBlock, wanted);
        for (uint32_t lane_offset = 0; lane_offset < kBlock; lane_offset += 16) {
          const bool read_with = lane_offset < x.records - x.offset;  // (unsigned, as the hardware's documents put it)
          const bool read_without = lane_offset < x.records;
          const bool inside = (uint64_t)x.offset + lane_offset + 16 <= (uint64_t)ntc * kBlock;
          if (wanted ? !(read_with && read_without && inside) : (read_with || read_without)) {
            std::printf("block request: column %u of %u, wanted %d, lane offset %u\n", tc, ntc, (int)wanted, lane_offset);
            std::exit(1);
          }
        }
      }
}

template <int BM>
static void check_staged_rows(const int M, const uint32_t ntc) {
  const int64_t block = (int64_t)ntc * 32768, blocks = (M + 127) / 128, end = blocks * block;
  const int groups = (M + BM - 1) / BM;
  for (int g = 0; g < groups; ++g) {
    const sfmp::StagedRows<BM> staged(M, g * BM, (uint32_t)block);
    for (int row = 0; row < BM; row += 8) {
      const sfmp::BlockRequest rows = staged.copy(row);
      const int64_t m = (int64_t)g * BM + row;  // (eight rows from a multiple of 8 on are in one block)
      const bool there = m / 128 < blocks;
      for (const uint32_t tc : {0u, ntc - 1})
        for (const uint32_t half : {0u, 128u}) {
          const sfmp::BlockRequest x = sfmp::block_request(tc * 32768u + half + rows.offset, rows.records, true);
          const int64_t meant = m / 128 * block + (int64_t)tc * 32768 + (m % 128) * 256 + half;
          const uint64_t last = 7 * 256 + 112;  // offset of the last 16 bytes of the copy within its 8 rows
          const bool read_with = x.records >= 16 && x.offset <= x.records && last + 16 <= x.records - x.offset;
          const bool read_without = last + 16 <= x.records;
          const bool right = there ? read_with && read_without && staged.base + x.offset == meant &&
                                         staged.base + (int64_t)x.records <= end && (uint64_t)x.offset + last + 16 <= x.records
                                   : x.records == 0;
          if (!right) {
            std::printf("staged rows: %d rows in workgroups of %d, %u tile columns: row %lld, column %u + %u: offset %u of %u records\n",
                        M, BM, ntc, (long long)m, tc, half, x.offset, x.records);
            std::exit(1);
          }
        }
    }
  }
}

static void check_staged_rows_of_all_forms(const int M, const uint32_t ntc) {
  check_staged_rows<64>(M, ntc);
  check_staged_rows<80>(M, ntc);
  check_staged_rows<96>(M, ntc);
  check_staged_rows<112>(M, ntc);
  check_staged_rows<128>(M, ntc);
  check_staged_rows<160>(M, ntc);
  check_staged_rows<192>(M, ntc);
  check_staged_rows<224>(M, ntc);
  check_staged_rows<256>(M, ntc);
}

// Every tile row, M block and K range is the place of one work item; without groups in the plain order.
static void check_work_items() {
  for (uint32_t ntr : {1u, 3u, 8u, 57u})
    for (uint32_t n_mtiles = 1; n_mtiles <= 70; ++n_mtiles)
      for (uint32_t ksplit : {1u, 2u, 7u, 8u})
        for (bool grouped : {false, true}) {
          const sfmp::WorkItems items = sfmp::work_items(ntr, n_mtiles, ksplit, grouped);
          std::vector<int> owners((size_t)ntr * n_mtiles * ksplit, 0);
          for (uint32_t block = 0; block < ntr * n_mtiles * ksplit; ++block) {
            const sfmp::Place w = items.place(block, ntr, ksplit);
            const bool inside = w.ks >= 0 && w.ks < (int)ksplit && w.tr >= 0 && w.tr < (int)ntr && w.mt >= 0 && w.mt < (int)n_mtiles;
            const bool plain = w.ks == (int)(block % ksplit) && w.mt == (int)(block / ksplit % n_mtiles) && w.tr == (int)(block / ksplit / n_mtiles);
            if (!inside || !(grouped || plain) || owners[((size_t)w.tr * n_mtiles + w.mt) * ksplit + w.ks]++ != 0) {
              std::printf("work item %u of %u x %u x %u: tile row %d, M block %d, range %d\n", block, ntr, n_mtiles, ksplit, w.tr, w.mt, w.ks);
              std::exit(1);
            }
          }
        }
  for (uint32_t by : {1u, 2u, 3u, 7u, 8u, 57u, 640u, 1792u, 65535u, 1u << 20, (1u << 31) - 1})
    for (uint64_t q : {0ull, 1ull, 2ull, 1000ull, 65536ull, 4000000ull})
      for (int64_t off = -2; off <= 2; ++off) {
        const int64_t x = (int64_t)(q * by) + off;
        if (x < 0 || x > 0xFFFFFFFFll) continue;
        const sfmp::Quotient r = sfmp::divide((uint32_t)x, sfmp::divisor(by));
        if (r.q != (uint32_t)x / by || r.rest != (uint32_t)x % by) {
          std::printf("%lld / %u: %u, rest %u\n", (long long)x, by, r.q, r.rest);
          std::exit(1);
        }
      }
}

int main() {
  check_block_requests();
  check_work_items();
  for (const uint32_t ntc : {1u, 2u, 31u, 128u, 224u, 448u}) {
    for (int M = 17; M < 800; M += 61) check_staged_rows_of_all_forms(M, ntc);
    if (ntc < 31) continue;
    // staged activations of a little less than 4 and 8 GiB, just that and a little more
    for (const int64_t bytes : {(int64_t)1 << 32, (int64_t)1 << 33}) {
      const int M = (int)(bytes / ((int64_t)ntc * 256));
      for (const int rows : {M - 200, M, M + 1, M + 700}) check_staged_rows_of_all_forms(rows, ntc);
    }
  }
  for (int count = 1; count <= 64; ++count) {
    std::vector<Event> events;
    auto load = [&](auto set, int i) { events.push_back({Event::kLoad, decltype(set)::value, i, false}); };
    auto copy = [&](auto slot, int i) { events.push_back({Event::kCopy, decltype(slot)::value, i, false}); };
    auto wait = [&](int columns) { events.push_back({Event::kWait, columns, 0, false}); };
    auto use = [&](auto set, int i) { events.push_back({Event::kUse, decltype(set)::value, i, false}); };
    auto keep = [&]() { events.push_back({Event::kKeep, 0, 0, false}); };
    sfmp::stream_columns(count, load, copy, wait, use, keep);
    for (size_t a = 0; a < events.size(); ++a) {
      if (events[a].kind != Event::kLoad) continue;
      for (size_t b = a + 1; b < events.size(); ++b) {
        const bool same = events[b].place == events[a].place;
        if (events[b].kind == Event::kKeep || (events[b].kind == Event::kUse && same)) events[a].read = true;
        if (events[b].kind == Event::kLoad && same) break;
      }
    }
    for (int slabs = 1; slabs <= 2; ++slabs)
      for (bool unread : {false, true}) check(events, count, slabs, unread);
  }
  std::puts("ok");
}
