// How the tile kernels split a grid into workgroups: plain host arithmetic.
#pragma once

#include <initializer_list>

namespace tenom {

// Waves per SIMD the face, row and tile kernels are compiled for: at most 168
// VGPRs, and three tiles fit in a CU's LDS.  None of them spills at six points; at
// eight TVD5 and the adaptive cutoff do (12 to 44 bytes a lane; the 1D faces, most
// with flags, 12 to 92), which still beats two wavefronts (256^3 x 1573 us, 1394 so).
constexpr int kFaceWaves = 3;

// Workgroups of 256 threads the chip holds at kFaceWaves (256 CUs, one
// wavefront of a workgroup per SIMD).
constexpr double kFaceSlots = 256.0 * kFaceWaves;

// Lines side by side in a workgroup's tile, as a rule: a wavefront then holds 8 x
// 8 faces, which lie whole in smooth regions more often than strips.
constexpr int kTileColumns = 8;

// Whole-line workgroups of a tile sweep along `axis`: the lines of the other
// axis times the column groups (x columns for y and z, y rows for x).
inline long tile_count(int axis, int nx, int ny, int nz) {
  const long lines = (axis == 2) ? ny : nz;
  const int across = (axis == 0) ? ny : nx;
  return lines * ((across + kTileColumns - 1) / kTileColumns);
}

// Places a workgroup's chunk takes whose tile has f of 32 faces a line: half its
// place, and half its share of wavefronts (of 8 faces of 8 lines).
inline double chunk_cost(int f) { return 0.5 + 0.125 * ((f + 7) / 8); }

// Cells per segment of a tile sweep.  Segments of 32 c - 1 cells take c
// chunks (one redundant face each); a whole line hands its faces on instead.
// More segments fill the chip and shorten the last round, fewer save the
// redundant faces, halo rows and partly filled chunks.  The c with the smallest
// estimate of
//   workgroups (chunks + 0.05) / slots + 0.4 (chunks of one workgroup + 0.05),
// slots = workgroups the chip holds, is taken; it agrees within 3 % with the best
// of the measured sweeps (Euler, six points, y and z, smooth (rough) data, us; one
// chunk, two, three, whole periodic lines): 64^3 51, 47, -, 46 (75, 65, -, 63);
// 96^3 113, 114, -, 102 (179, 178, -, 162); 100^3 129, 129, 142, 144 (198, 199, 233,
// 236); 128^3 216, 225, 228, 200 (351, 373, 371, 320); 187x150x93 257, 260, 271, 272
// (411, 426, 433, 433); 1024^2 52, 53, 52, 162 (80, 83, 82, 225); 2048^2 166, 159,
// 161, 312 (261, 256, 255, 443).  The search ends where the second term alone
// exceeds the best, so that enqueuing a long thin grid's sweep does not take longer
// than the sweep (every c took 158 us for 10^6 cells).
inline double tile_segment_time(double lines, int n, int bc, int c, bool whole) {
  constexpr double start = 0.05;
  auto chunks = [](long faces) { return (double)(faces / 32) + (faces % 32 ? chunk_cost((int)(faces % 32)) : 0.0); };
  const long seg = whole ? n : 32l * c - 1, nseg = whole ? 1 : (n + seg - 1) / seg;
  const double one = chunks(whole && bc == 0 ? n : seg + 1) + start;
  const double last = chunks(whole && bc == 0 ? n : n - (nseg - 1) * seg + 1) + start;
  return lines * ((nseg - 1) * one + last) / kFaceSlots + 0.4 * one;
}

inline int tile_segment(int axis, int n, int nx, int ny, int nz, int bc) {
  const double lines = (double)tile_count(axis, nx, ny, nz);
  // chunks of the whole line: the first c whose segment holds it
  const int last = (bc == 0 && n % 32 == 0) ? n / 32 : n / 32 + 1;
  int best = n;
  double best_t = 0.0;
  for (int c = 1; c < last; ++c) {
    const double t = tile_segment_time(lines, n, bc, c, false);
    if (c == 1 || t < best_t) {
      best_t = t;
      best = 32 * c - 1;
    }
    if (0.4 * c > best_t) break;
  }
  return last == 1 || tile_segment_time(lines, n, bc, last, true) < best_t ? n : best;
}

// Whether the row sweep takes the x sweep of a 2D or 3D grid, instead of the tile
// sweep: its workgroups (256 faces of one row) are at most two per CU, or the rows
// fill them better than rows and columns fill the tiles.
inline bool row_sweep_x(int nx, int ny, int nz, int bc) {
  if ((long)((nx + 254) / 255) * ny * nz <= 512 && nx >= 128) return true;
  const int cells = (bc == 0 && nx <= 256) ? 256 : 255;
  const double row = (double)nx / ((double)cells * ((nx + cells - 1) / cells));
  const double tile = (double)nx / (32.0 * ((nx + 31) / 32)) * ny / (kTileColumns * (double)((ny + kTileColumns - 1) / kTileColumns));
  return row > tile;
}

// Split of the face kernel: a workgroup of 256 threads takes fj faces of tx lines;
// its lines are side by side in rows of `width` lines.
struct FaceSplit {
  int width, fj, tx;
};

// Estimated time of a split, in rounds of full workgroups: a workgroup whose
// threads are partly idle costs half its place and half its share of wavefronts;
// 0.7 is the last round; each staged cell costs a tenth of a face, and wavefronts
// that are not square skip the limiter less often.
inline double face_split_time(int nfl, long nlines, int K, const FaceSplit& s) {
  const int full = nfl / s.fj, rest = nfl - full * s.fj;
  auto cost = [&](int f) { return 0.5 + 0.125 * ((f * s.tx + 63) / 64); };  // as chunk_cost
  const double groups = (double)(nlines / s.width) * ((s.width + s.tx - 1) / s.tx);
  const double work = 1.0 + 0.1 * (s.fj + K - 1) * s.tx / 256.0 + 0.005 * (s.tx + 64.0 / s.tx - 16.0);
  return work * (groups * (full * cost(s.fj) + (rest ? cost(rest) : 0.0)) / kFaceSlots + 0.7);
}

// The split of nlines lines of nfl faces each, `across` of them in a plane, at K
// points and at most nc staged cells a workgroup.  A single line fills the
// workgroup.  Else 32 faces of 8 lines of a plane, unless they fill the chunks so
// badly that chunks of equal length, with as many of all lines side by side as
// fit, promise 8 %.  us, 32 x 8 and the other, Euler at eight points, smooth (rough)
// data: 72x72x33 along the transmissive z (34 faces: 17 x 15) 33 and 24 (43 and
// 34); 100x100x12 along z (12 x 21) 34 and 26 (39 and 30); 65x65x65 (22 x 11) 44 and
// 36 (55 and 45); 50x50x50 (50 x 5) 25 and 22 (29 and 26); where they promise less
// they lose up to 15 % (1394x130, 300x300, 1024x1024 transmissive).
// Fewer than 8 columns of x side by side (strided: faces along y and z) use less
// than a 64-byte sector of each row, which costs 7 % more: 57x153x133 along y 51 x 5
// 79 us, 32 x 8 74; 32x50x93 50 x 5 31.5, 28.6; 33x151x44 along z 39 x 6 40, 50.
inline FaceSplit face_split(int nfl, int across, long nlines, int K, int nc, bool strided = false) {
  if (nlines == 1) return FaceSplit{1, nfl < 256 ? nfl : 256, 1};
  FaceSplit best{across, 32, kTileColumns};
  double best_t = face_split_time(nfl, nlines, K, best) / 1.08;
  for (const int f : {6, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64}) {
    const int chunks = (nfl + f - 1) / f, fj = (nfl + chunks - 1) / chunks;
    int tx = 256 / fj;
    if (tx > nc / (fj + K - 1)) tx = nc / (fj + K - 1);
    if (tx > nlines) tx = (int)nlines;
    const FaceSplit s{(int)nlines, fj, tx};
    const double t = face_split_time(nfl, nlines, K, s) * (strided && tx < kTileColumns ? 1.07 : 1.0);
    if (t < best_t) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

// Faces of one wavefront for each of the 1024 SIMDs.
constexpr long kWaveFaces = 65536;

// Whether one thread per face straight from global memory takes the Euler faces of
// a 2D or 3D grid (which are too many for one wavefront per field) instead of the
// split s.  It fills one wavefront per SIMD with kWaveFaces and costs as much
// below; two with twice that.  us, that and the split, smooth (rough) data, with
// flags, six points unless stated: one wavefront, 40^3 periodic 8.5 and 9.7 (8.5
// and 14.7), at eight points 12.4 and 14.5 (12.1 and 21); 40x40x39 transmissive
// 11.5 and 19.  Two, well filled, along y and z, where the split's lines are few
// side by side and flags are stored: 50^3 13.8 and 14.1 (13.8 and 19.0), at eight
// points 22 and 17.6 (no), without flags 13.2 and 11.5 (no); or where every chunk
// has a face of a transmissive end, which is rough as soon as the state has a
// slope there: 50^3 13.8 and 18.3 (13.8 and 19.0), at eight points 22 and 23.4 (22
// and 24.1), 44x43x45 13.2 and 15.6 (13.1 and 16.0), at eight points 21.6 and 20.8
// (no).  Elsewhere it loses on smooth data what it gains on rough: 48^3 13.6 and
// 12.5 (13.6 and 19.2), 360x360 11.6 and 10.4 (11.6 and 16.0), 1394x130 along y
// 16.4 and 16.0 (16.4 and 22.9).
inline bool faces_direct(int axis, int bc, int nfl, long nlines, int K, bool flags, const FaceSplit& s) {
  const long faces = nlines * nfl;
  if (nlines == 1 || faces > 2 * kWaveFaces) return false;
  if (faces <= kWaveFaces) return true;
  if (axis == 0) return false;
  if (bc != 0 && nfl <= 2 * s.fj) return faces >= (K == 6 ? 1.25 : 1.5) * kWaveFaces;
  return K == 6 && flags && s.tx < kTileColumns && faces >= 1.5 * kWaveFaces;
}

}  // namespace tenom
