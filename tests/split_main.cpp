// Checks of teno_split.h on the host: every split covers its lines, fits its
// workgroup, its staging array and one launch; prints "ok" at the end.
#include "teno_split.h"

#include <cstdio>
#include <ctime>

using namespace tenom;

static int bad = 0;
static volatile long check_thin = 0;  // keeps the timed choices

static void check_faces(int nfl, int across, long nlines, int K) {
  const int nc = 416;
  const FaceSplit s = face_split(nfl, across, nlines, K, nc);
  const long nch = (nfl + s.fj - 1) / s.fj, ncg = (s.width + s.tx - 1) / s.tx, blocks = nlines / s.width * ncg * nch;
  const bool fits = s.fj >= 1 && s.tx >= 1 && s.fj * s.tx <= 256 && (s.fj + K - 1) * s.tx <= nc;
  if (!fits || nlines % s.width || (nch - 1) * s.fj >= nfl || (ncg - 1) * s.tx >= s.width ||
      (nlines > 1 && blocks >= 1l << 24)) {
    std::printf("face_split(%d, %d, %ld, %d): %d x %d of %d, %ld blocks\n", nfl, across, nlines, K, s.fj, s.tx, s.width,
                blocks);
    ++bad;
  }
}

// tile_segment by trying every chunk count up to the whole line
static int segment_by_all(int axis, int n, int nx, int ny, int nz, int bc) {
  const double lines = (double)tile_count(axis, nx, ny, nz);
  int best = n;
  double best_t = 0.0;
  for (int c = 1;; ++c) {
    const int seg = 32 * c - 1;
    const bool whole = seg >= n || (bc == 0 && seg + 1 == n);
    const double t = tile_segment_time(lines, n, bc, c, whole);
    if (c == 1 || t < best_t) {
      best_t = t;
      best = whole ? n : seg;
    }
    if (whole) return best;
  }
}

static void check_segment(int axis, int n, int across, int others, int bc) {
  const int nx = axis == 0 ? n : across, ny = axis == 0 ? across : (axis == 1 ? n : others);
  const int nz = axis == 2 ? n : others;
  const int got = tile_segment(axis, n, nx, ny, nz, bc), want = segment_by_all(axis, n, nx, ny, nz, bc);
  if (got != want) {
    std::printf("tile_segment(%d, %d, %d x %d x %d, %d): %d, not %d\n", axis, n, nx, ny, nz, bc, got, want);
    ++bad;
  }
}

int main() {
  for (int axis = 0; axis < 3; ++axis)
    for (int bc = 0; bc < 2; ++bc)
      for (int across : {6, 9, 64, 500, 5000})
        for (int others : {1, 6, 100, 1000}) {
          if (axis == 2 && others == 1) continue;
          for (int n = 6; n <= 700; ++n) check_segment(axis, n, across, others, bc);
          for (int n : {1023, 1024, 1025, 9999, 10016, 65536, 200000, 1000000})
            if ((long)n * across * others < 0x7fffffffl) check_segment(axis, n, across, others, bc);
        }
  // x sweeps by the row sweep: few rows, or rows that fill its workgroups better
  struct { int nx, ny, nz, bc; bool row; } xs[] = {{256, 256, 1, 0, true},   {200000, 9, 1, 1, true},
      {20000, 17, 1, 0, true}, {500, 10, 100, 0, true},  {255, 255, 9, 1, true}, {20000, 90, 1, 0, true},
      {256, 256, 256, 0, false}, {256, 256, 256, 1, false}, {256, 41, 30, 1, false}, {256, 41, 30, 0, true}, {300, 1200, 1, 0, false},
      {1024, 1024, 1, 0, false}, {187, 93, 150, 0, false}, {64, 9, 9, 0, false}, {8, 100000, 1, 0, false}};
  for (const auto& x : xs)
    if (row_sweep_x(x.nx, x.ny, x.nz, x.bc) != x.row) {
      std::printf("row_sweep_x(%d, %d, %d, %d) is %d\n", x.nx, x.ny, x.nz, x.bc, !x.row);
      ++bad;
    }
  // faces straight from global memory: up to one wavefront per SIMD, and two where
  // the split's lines are few or its chunks all touch a transmissive end
  struct { int axis, n, bc; long nlines; int across, K; bool direct; } fs[] = {{0, 40, 0, 1600, 40, 6, true},
      {2, 39, 1, 1600, 40, 8, true},   {0, 50, 0, 2500, 50, 6, false},  {1, 50, 0, 2500, 50, 6, true},
      {1, 50, 0, 2500, 50, 8, false},  {2, 12, 1, 10000, 100, 6, true}, {2, 12, 1, 10000, 100, 8, true},
      {0, 12, 1, 10000, 100, 8, false}, {2, 45, 1, 1892, 44, 6, true},  {2, 45, 1, 1892, 44, 8, false},
      {1, 48, 0, 2304, 48, 6, false},  {1, 340, 1, 340, 340, 6, false}, {2, 64, 0, 4096, 64, 6, false},
      {0, 60000, 1, 1, 1, 6, false},   {1, 20, 1, 100000, 1000, 6, false}};
  for (const auto& x : fs) {
    const int nfl = x.bc ? x.n + 1 : x.n;
    const FaceSplit s = face_split(nfl, x.across, x.nlines, x.K, 416);
    if (faces_direct(x.axis, x.bc, nfl, x.nlines, x.K, true, s) != x.direct) {
      std::printf("faces_direct(%d, %d, %d, %ld, %d) is %d\n", x.axis, x.bc, nfl, x.nlines, x.K, !x.direct);
      ++bad;
    }
  }
  // a long thin grid: a thousand choices of 0.65 ms each by trying every count
  const std::clock_t t0 = std::clock();
  for (int i = 0; i < 1000; ++i) check_thin = check_thin + tile_segment(0, 4000000 + i, 4000000 + i, 9, 1, 1);
  const double ms = 1e3 * (double)(std::clock() - t0) / CLOCKS_PER_SEC;
  if (ms > 100.0) {
    std::printf("tile_segment of a line of 4,000,000 cells: %.1f us\n", ms);
    ++bad;
  }
  for (int K = 6; K <= 8; K += 2) {
    for (int n = K; n <= 3000; ++n)
      for (int open = 0; open < 2; ++open)
        for (int across : {6, 7, 8, 9, 37, 64, 1000, 4097})
          // one plane, some, and the most cells a grid may have
          for (long planes : {1l, 6l, 53l, 0x7fffffffl / n / across})
            if (planes > 0) check_faces(n + open, across, across * planes, K);
    check_faces(2000000000, 1, 1, K);
  }
  if (!bad) std::printf("ok\n");
  return bad != 0;
}
