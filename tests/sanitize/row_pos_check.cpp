// Walks rows at the end of the largest column array a CSR may have (2^31 - 1
// arcs) the way the kernels' waves do, with the functions they use, and counts
// which columns are read: every column of the row once (a covered row: a front
// part of it), none outside it. Built with the undefined-behaviour sanitizer by
// tests/test_row_pos.py; exits with status 0 only if all hold.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "row_pos.h"

using blest::row_pos;

static int failures = 0;

struct Row {
  int64_t begin, end;
  std::vector<int> reads;
  Row(int64_t b, int64_t e) : begin(b), end(e), reads(static_cast<size_t>(e - b), 0) {}
  void read(row_pos i) {
    if (static_cast<int64_t>(i) < begin || static_cast<int64_t>(i) >= end) {
      std::printf("column %u of row [%lld, %lld) read\n", i, static_cast<long long>(begin), static_cast<long long>(end));
      ++failures;
    } else {
      ++reads[i - static_cast<row_pos>(begin)];
    }
  }
  void check(const char* what) {
    for (int r : reads)
      if (r != 1) {
        std::printf("%s: a column of a row of %zu read %d times\n", what, reads.size(), r);
        ++failures;
        return;
      }
    for (int& r : reads) r = 0;
  }
};

// A wave's steps of 64 columns of each of M pieces, the next step's loaded ahead.
static void wave_scan(Row& row, row_pos p, row_pos e, int M) {
  auto load = [&](row_pos P, uint32_t ahead) {
    for (uint32_t lane = 0; lane < 64; ++lane)
      if (blest::row_has(P, ahead + lane, e)) row.read(P + (ahead + lane));
  };
  std::vector<row_pos> P(M);
  for (int m = 0; m < M; ++m) P[m] = p + 64 * m;
  for (int m = 0; m < M; ++m) load(P[m], 0);
  while (P[0] < e)
    for (int m = 0; m < M; ++m) {
      load(P[m], 64 * M);
      P[m] += 64 * M;
    }
}

int main() {
  const int64_t top = blest::kMaxArcs;
  const int64_t lengths[] = {1, 3, 4, 5, 31, 33, 63, 64, 65, 255, 256, 257, 511, 513, 4097, 4160, 20000};
  const int64_t ends[] = {top, top - 1, top - 3, top - 255, top - 510, top - 1100, 40000};
  for (int64_t end : ends)
    for (int64_t len : lengths) {
      Row row(end - len, end);
      const row_pos b = static_cast<row_pos>(row.begin), e = static_cast<row_pos>(row.end);
      // a lane's steps of four columns
      for (row_pos q = b; q < e; q += 4)
        for (uint32_t t = 0; t < 4; ++t)
          if (blest::row_has(q, t, e)) row.read(q + t);
      row.check("lane");
      // a lane group's steps of 8 columns, two steps ahead
      for (uint32_t G : {2u, 4u}) {
        const uint32_t L = G == 2 ? 4 : 1, step = G * L;
        auto columns = [&](row_pos q) {
          for (uint32_t sub = 0; sub < L; ++sub)
            for (uint32_t g = 0; g < G; ++g)
              if (blest::row_has(q + G * sub, g, e)) row.read(q + G * sub + g);
        };
        columns(b);
        columns(b + step);
        for (row_pos p = b;; p += step) {
          columns(p + 2 * step);
          if (p + step >= e) break;
        }
        row.check("group");
      }
      // one row a wave, and its chunks of 256
      for (row_pos p = b; p < e; p += 64)
        for (uint32_t lane = 0; lane < 64; ++lane)
          if (blest::row_has(p, lane, e)) row.read(p + lane);
      row.check("wave");
      for (int64_t c = 0; c < len; c += 256) {
        const row_pos cb = b + static_cast<uint32_t>(c), ce = blest::row_part_end(cb, 256, e);
        for (uint32_t lane = 0; lane < 64; ++lane)
          for (row_pos p = cb + lane; p < ce; p += 64) row.read(p);
      }
      row.check("chunks");
      for (int M : {2, 4}) {
        wave_scan(row, b, e, M);
        row.check("scan");
        for (uint32_t i = 0; i < 16; ++i) {
          const uint32_t n = blest::row_piece_len(b, e, 16);
          const row_pos p = b + i * n;
          wave_scan(row, p, blest::row_part_end(p, n, e), M);
        }
        row.check("pieces");
      }
    }
  std::printf("row_pos_check: %d failures\n", failures);
  return failures == 0 ? 0 : 1;
}
