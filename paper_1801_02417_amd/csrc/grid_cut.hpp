// How a gridding tile's rows are cut into runs and chunks, and the chunk size that a problem is cut
// with (plain C++, no device code).
#pragma once

#include <algorithm>
#include <cstddef>
#include <utility>
#include <vector>

namespace psara {

constexpr int kRunMax = 32;         // longest run of same-window visibilities one lane group takes
constexpr int kChunkEntries = 1024; // largest gridding chunk (entries per workgroup, staged in LDS)
constexpr int kLeastChunk = 64;     // smallest chunk size
constexpr int kMaxTileChunks = 4, kMaxSmallChunks = 512;   // of a chunk size below the default
static_assert(kRunMax <= kLeastChunk, "a run fits a chunk");

// {first row, length}
using Run = std::pair<int, int>;

// The runs of rows beg .. end-1: consecutive rows with the same window start (their taps hit the
// same cells), split at kRunMax.
inline std::vector<Run> tile_runs(const std::vector<int>& k0, int beg, int end) {
  std::vector<Run> runs;
  for (int e = beg; e < end;) {
    int f = e + 1;
    while (f < end && f - e < kRunMax && k0[f] == k0[e]) ++f;
    runs.push_back({e, f - e});
    e = f;
  }
  return runs;
}

// The end of the chunk that begins at run r: whole runs with at most `entries` rows.
inline size_t chunk_end(const std::vector<Run>& runs, size_t r, int entries) {
  int rows = 0;
  const size_t r0 = r;
  while (r < runs.size() && (rows + runs[r].second <= entries || r == r0)) rows += runs[r++].second;
  return r;
}

// The entries the chunks are cut for (row_beg, row_end: the rows of every tile).  The default asks
// for the smallest size at which no tile has more than kMaxTileChunks chunks and all chunks together
// are at most kMaxSmallChunks (two workgroups per CU): a problem that does not fill the GPU is bound
// by its longest chunk, and the column inverse FFT, which adds a tile's slots one after the other, by
// the tile with the most.  256 and 512 are taken as asked for.
//   us per iteration at 1024, 512, 256, 128, 64 entries (most chunks of one tile):
//   32^2 FP64, 600 rows   46.5 46.4 46.4 42.5 39.6  (1 1 1 2 4)
//   64^2 FP32, 1511 rows  37.6 37.6 37.6 37.3 35.1  (1 1 1 2 3)
//   64^2 FP64, 3000 rows  70.0 67.4 56.2 55.6 60.5  (1 2 3 5 9)
//   128^2 FP32, 12000     47.8 44.4 42.3 43.7 48.0  (1 2 3 6 11)
//   128^2 FP32 with Mueller matrices, 20001   57.4 at 1024, 44.9 at 256 (1, 4)
//   64^2 FP32, 30000      52.7 48.7 54.0 74.0 115.7 (5 10 20 39 77)
//   256^2 FP32, 2e5       94.9 95.7 100  126  182   (4 8 16 31 61; 848 chunks at 1024)
inline int grid_chunk_entries(const std::vector<int>& k0, const std::vector<int>& row_beg,
                              const std::vector<int>& row_end, int asked) {
  const size_t tiles = row_beg.size();
  std::vector<std::vector<Run>> runs;
  int best = asked;
  for (int c = asked / 2; asked == kChunkEntries && c >= kLeastChunk; c /= 2) {
    // a tile has no fewer chunks than its rows ask for; that turns large problems away unread
    long long least = 0, all = 0;
    bool fits = true;
    for (size_t t = 0; t < tiles && fits; ++t) {
      const int k = (row_end[t] - row_beg[t] + c - 1) / c;
      least += k;
      fits = k <= kMaxTileChunks && least <= kMaxSmallChunks;
    }
    if (!fits) break;
    if (runs.empty())
      for (size_t t = 0; t < tiles; ++t) runs.push_back(tile_runs(k0, row_beg[t], row_end[t]));
    for (size_t t = 0; t < tiles && fits; ++t) {
      int k = 0;
      for (size_t r = 0; r < runs[t].size(); ++k) r = chunk_end(runs[t], r, c);
      all += k;
      fits = k <= kMaxTileChunks && all <= kMaxSmallChunks;
    }
    if (!fits) break;
    best = c;
  }
  return best;
}

}  // namespace psara
