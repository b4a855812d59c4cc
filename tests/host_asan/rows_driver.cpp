// Host check of long rows in a row program (csrc/closed.cpp), built by
// tests/test_rows_host.py: every entry of every row up to kMaxRowEntries is run
// once by the lanes of the row's group, and a longer row, whose quads a batch
// word could not hold, is refused.
#include <cstdio>
#include <cstdlib>

#include "closed.h"

using namespace emt;

static void require(bool ok, const char *what) {
  if (ok) return;
  std::printf("FAILED: %s\n", what);
  std::exit(1);
}

static void check(const std::vector<int> &sizes, int lanes) {
  std::vector<RowSum> rows(sizes.size());
  int id = 1;
  for (size_t r = 0; r < rows.size(); ++r) {
    rows[r].row = (int)r;
    for (int e = 0; e < sizes[r]; ++e, ++id) rows[r].e.push_back({id % 30000, id});
  }
  const RowProgram p = schedule_rows(rows, lanes, 0, 0);
  const int waves = lanes / 64;
  std::vector<char> seen(id, 0);
  std::vector<int> wrote(rows.size(), 0);
  for (int b = 0; b < p.batches; ++b) {
    const uint32_t m = (uint32_t)p.meta[waves + 1 + b];
    const int q0 = (int)(m & 0xFFFF), nq = (int)((m >> 16) & 0xFF), lg = (int)(m >> 24);
    require(lg <= 4 && nq >= 1 && q0 + nq <= p.quads, "batch word");
    for (int lane = 0; lane < 64; ++lane) {
      const int row = p.row[b * 64 + lane];
      if (row == 0xFFFF) continue;
      wrote[row]++;
      int cnt = 0;
      for (int l = lane - (1 << lg) + 1; l <= lane; ++l)
        for (int q = q0; q < q0 + nq; ++q)
          for (int k = 0; k < 4; ++k) {
            const int src = p.src[q * 256 + (k / 2) * 128 + l * 2 + (k & 1)];
            if (src == 0) continue;
            require(src < id && !seen[src], "an entry runs once");
            require(p.code[(q * 64 + l) * 4 + k] == src % 30000, "an entry's code");
            seen[src] = 1;
            ++cnt;
          }
      require(cnt == sizes[row], "a row's entries run in its group");
    }
  }
  for (int w : wrote) require(w == 1, "a row is written once");
}

int main() {
  for (int lanes : {64, 256, 512})
    for (int n : {1, 64, kMaxRowEntries - 1, kMaxRowEntries, kMaxRowEntries + 1, 2 * kMaxRowEntries, 65500}) {
      bool refused = false;
      try {
        check({n}, lanes);
        check({3, n, 0, 17, n / 2}, lanes);
      } catch (const Error &e) {
        refused = e.status == EMT_EINVAL;
      }
      require(refused == (n > kMaxRowEntries), "rows of up to kMaxRowEntries entries");
    }
  std::printf("ok\n");
  return 0;
}
