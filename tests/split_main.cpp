// Checks of teno_split.h on the host: every split covers its lines, fits its
// workgroup, its staging array and one launch; prints "ok" at the end.
#include "teno_split.h"

#include <cstdio>

using namespace tenom;

static int bad = 0;

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

int main() {
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
