// Checks of the gridding cut (grid_cut.hpp) on the CPU: prints one line per case, exits 1 at the
// first that fails.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>

#include "grid_cut.hpp"

using namespace psara;

struct Tiles {
  std::vector<int> k0, beg, end;
  int start = 0;
  // a tile of windows with the given numbers of rows
  void add(const std::vector<int>& windows) {
    beg.push_back((int)k0.size());
    for (int rows : windows) {
      for (int i = 0; i < rows; ++i) k0.push_back(start);
      ++start;
    }
    end.push_back((int)k0.size());
  }
};

// chunks of every tile when cut with c, row by row and without the functions under test
static void count(const Tiles& t, int c, int* most, int* all) {
  *most = *all = 0;
  for (size_t i = 0; i < t.beg.size(); ++i) {
    int chunks = 0, rows = 0;
    for (int e = t.beg[i]; e < t.end[i];) {
      int len = 1;
      while (len < 32 && e + len < t.end[i] && t.k0[e + len] == t.k0[e]) ++len;
      if (chunks == 0 || rows + len > c) { ++chunks; rows = 0; }
      rows += len;
      e += len;
    }
    *all += chunks;
    if (chunks > *most) *most = chunks;
  }
}

static void check(bool ok, const std::string& what) {
  if (ok) return;
  std::printf("FAILED %s\n", what.c_str());
  std::exit(1);
}

static void run(const char* name, const Tiles& t) {
  const int got = grid_chunk_entries(t.k0, t.beg, t.end, 1024);
  int most, all;
  // the smallest of the sizes tried in falling order that all keep the bounds
  int want = 1024;
  for (int c = 512; c >= 64; c /= 2) {
    count(t, c, &most, &all);
    if (most > 4 || all > 512) break;
    want = c;
  }
  check(got == want, std::string(name) + ": size " + std::to_string(got) + ", expected " + std::to_string(want));
  count(t, got, &most, &all);
  if (got < 1024) check(most <= 4 && all <= 512, std::string(name) + ": " + std::to_string(most) + " of " + std::to_string(all));
  // what is cut is what was counted, every row once, whole runs, at most `got` rows a chunk
  int cut = 0;
  for (size_t i = 0; i < t.beg.size(); ++i) {
    const std::vector<Run> runs = tile_runs(t.k0, t.beg[i], t.end[i]);
    int at = t.beg[i];
    for (size_t r = 0; r < runs.size(); ++cut) {
      const size_t e = chunk_end(runs, r, got);
      check(e > r, std::string(name) + ": an empty chunk");
      int rows = 0;
      for (; r < e; ++r) {
        check(runs[r].first == at && runs[r].second >= 1 && runs[r].second <= kRunMax, std::string(name) + ": runs");
        at += runs[r].second;
        rows += runs[r].second;
      }
      check(rows <= got, std::string(name) + ": a chunk too large");
    }
    check(at == t.end[i], std::string(name) + ": rows lost");
  }
  check(cut == all, std::string(name) + ": cut " + std::to_string(cut) + ", counted " + std::to_string(all));
  for (int asked : {256, 512}) check(grid_chunk_entries(t.k0, t.beg, t.end, asked) == asked, std::string(name) + ": asked size");
  std::printf("%s: %d entries, %d chunks, %d of a tile\n", name, got, all, most);
}

int main() {
  Tiles none;
  run("no tiles", none);
  Tiles empty;
  for (int i = 0; i < 16; ++i) empty.add({});
  run("empty tiles", empty);
  Tiles one;
  one.add({1});
  run("one row", one);
  // windows of 33 rows are runs of 32 and 1: 33 rows to a chunk of 64, seven chunks of a tile that by
  // its rows has four
  Tiles w33;
  for (int i = 0; i < 128; ++i) w33.add(std::vector<int>(7, 33));
  run("windows of 33", w33);
  Tiles w33s;
  w33s.add(std::vector<int>(7, 33));
  w33s.add({5});
  run("windows of 33, one tile", w33s);
  Tiles full;                      // 512 chunks exactly, and one more
  for (int i = 0; i < 128; ++i) full.add(std::vector<int>(256, 1));
  run("at the bound", full);
  full.add({1});
  run("beyond the bound", full);
  std::mt19937 rng(7);
  for (int k = 0; k < 400; ++k) {
    Tiles t;
    const int tiles = 1 + rng() % (k % 10 == 0 ? 300 : 30), top = 1 + rng() % (k % 3 == 0 ? 1200 : 250);
    for (int i = 0; i < tiles; ++i) {
      std::vector<int> w;
      const int rows = rng() % top, wide = 1 + rng() % 70;
      for (int left = rows; left > 0;) {
        const int r = std::min<int>(left, 1 + rng() % wide);
        w.push_back(r);
        left -= r;
      }
      t.add(w);
    }
    run(("random " + std::to_string(k)).c_str(), t);
  }
  return 0;
}
