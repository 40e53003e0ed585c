// Kernels of the TENO-M path and their launchers.
//
//  k_faces         face fluxes (and optionally the smoothness flags) of one
//                  axis from staged tiles.  The unit the reconstruct_faces
//                  call exposes, with k_faces_direct (from global memory) and
//                  k_faces_fields (one wavefront per field) on smaller grids.
//  k_sweep_row     sweep along x (unit stride).  A 256-thread workgroup owns
//                  one row segment: the segment's cells are staged in LDS
//                  with their flux, signal speed and Roe inputs, each thread
//                  computes one face flux, the fluxes go back to LDS, then
//                  each thread forms one cell's divergence and applies the
//                  epilogue.  A periodic row of <= 256 cells is one segment,
//                  so every face and every cell is computed exactly once.
//  k_sweep_tile    sweep along any axis of a 2D or 3D grid: a workgroup takes
//                  TX adjacent lines (x columns for y and z, y rows for x)
//                  over a segment of the axis and walks it in chunks, each
//                  chunk a row sweep of a strided tile staged in LDS.
//  k_sweep_march   sweep along y or z (strided), the line kernel that
//                  tenom_set_sweep_kernel can ask for.  Each lane owns one x
//                  column (coalesced 512-byte rows per wave; the block's
//                  wavefronts take consecutive (line, segment) units) and marches
//                  along the axis over a segment of cells, keeping the face's
//                  K cells in an LDS ring and carrying the previous face
//                  flux in registers.  The next face's new cell and the
//                  epilogue operands of the cell being closed are loaded
//                  before the face is computed, so their latency hides
//                  behind it.  M cells cost M+1 faces.
//
// Sweep epilogues (divergence -dF/dx of the axis, then):
//  STORE  R = div                      ACCUM  R += div
//  RK     Uout = a U0 + b (Us + dt (R + div))      RK1   Uout = a U0 + b (Us + dt div)
// where Us is the stage state the stencils read (p.U); the kernels take it
// from their LDS copy of the cell instead of reading HBM again.
#pragma once

#include <type_traits>

#include "teno_device.h"
#include "teno_split.h"

namespace tenom {

enum : int { EPI_STORE = 0, EPI_ACCUM = 1, EPI_RK = 2, EPI_RK1 = 3 };

template <int NF>
struct SweepParams {
  const double* U;   // state the stencils read
  double* R;         // divergence accumulator (STORE/ACCUM write, RK reads)
  const double* U0;  // RK: U^n
  double* Uout;      // RK: output state
  double a, b, dt;   // RK coefficients
  const double* dtp; // if not NULL: dt is read from this device address instead
  int mode;
  int nx, ny, nz;    // grid extents (1 for unused axes)
  int n;             // cells along the sweep axis
  int bc;            // boundary rule of the sweep axis
  double inv_dx;     // 1 / dx of the sweep axis
  int seg;           // cells per segment
  int nseg;          // segments per line
  int fld[NF];       // rotated component -> storage field
  FaceParams fp;
};

// Operands the epilogue reads from HBM: R (ACCUM, RK) and U^n (RK with
// a != 0).  Loaded by epi_load so that a caller can issue them early.
template <int NF>
struct EpiIn {
  double r[NF], u0[NF];
};

template <int NF>
__device__ __forceinline__ void epi_load(const SweepParams<NF>& p, long N, long cell, EpiIn<NF>& in) {
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    const long o = (long)p.fld[q] * N + cell;
    in.r[q] = (p.mode == EPI_ACCUM || p.mode == EPI_RK) ? p.R[o] : 0.0;
    in.u0[q] = (p.mode >= EPI_RK && p.a != 0.0) ? p.U0[o] : 0.0;
  }
}

// The step size of the RK modes, read once per thread.
template <int NF>
__device__ __forceinline__ double epi_dt(const SweepParams<NF>& p) {
  return p.dtp ? *p.dtp : p.dt;
}

// us: the cell's stage state (rotated components), only used by RK modes
template <int NF>
__device__ __forceinline__ void epi_store(const SweepParams<NF>& p, long N, long cell, const double (&div)[NF],
                                          const EpiIn<NF>& in, const double (&us)[NF], double dt) {
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    const long o = (long)p.fld[q] * N + cell;
    if (p.mode == EPI_STORE) {
      p.R[o] = div[q];
    } else if (p.mode == EPI_ACCUM) {
      p.R[o] = in.r[q] + div[q];
    } else {
      const double rhs = (p.mode == EPI_RK) ? in.r[q] + div[q] : div[q];
      const double v = fma(dt, rhs, us[q]);
      p.Uout[o] = (p.a != 0.0) ? fma(p.a, in.u0[q], p.b * v) : p.b * v;
    }
  }
}

// ---------------------------------------------------------------------------
// Row sweep.  Cells of the segment (plus K-1 halo cells) are staged once in
// LDS together with their physical flux, signal speed and Roe inputs, so a
// face reads its K cells instead of recomputing them.
// ---------------------------------------------------------------------------
template <int NF>
struct RowStage {
  static constexpr int NE = (NF == 1) ? 1 : 3 * NF + 1;  // U, F, lambda, Roe input
};

// CS: staging-index step between consecutive cells of the sweep axis (1 in
// the row sweep, the tile width in the tile sweep; 0: known at run time, cs).
// REREAD: the Euler face
// projects its stencil group by group of fields from fresh reads of the
// cells and lets wavefronts whose candidates are all smooth skip the limiter
// (worth it where most wavefronts see only smooth data: the tile sweep's
// 8 x 8 patches of faces, which a discontinuity crosses far less often than
// the row sweep's strips of 64, and the batched 1D problems' constant
// states).  ONE: a 1D face at six points takes its fields as one group whatever
// the limiter (see euler_face).
template <int NF, int K, int CS = 1, bool REREAD = false, bool ONE = false>
struct StagedCells {
  static constexpr bool kReread = REREAD;  // the face reads the cells again per group of fields
  static constexpr bool kOneGroup = ONE;
  static constexpr bool kUniform = REREAD && NF == 3 && CS == 1;  // 1D: constant states skip the face
  const double* s;  // LDS: [NE][NC]
  int nc;           // row pitch of the staging array
  int c0;           // staging index of window cell 0
  int cs = CS;      // run-time step where CS is 0
  __device__ __forceinline__ int step() const { return CS ? CS : cs; }
  __device__ __forceinline__ double at(int e, int c) const { return s[e * nc + c]; }
  // the same provider, its position hidden from the compiler, so that reads
  // through it are not merged with earlier reads of the same cells
  __device__ __forceinline__ StagedCells fresh() const {
    int c = c0;
    asm volatile("" : "+v"(c));
    return StagedCells<NF, K, CS, REREAD, ONE>{s, nc, c, cs};
  }
  __device__ __forceinline__ void state_flux(int m, double (&X)[NF], double (&F)[NF]) const {
    const int c = c0 + m * step();
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      X[q] = at(q, c);
      F[q] = at(NF + q, c);
    }
  }
  // Whether all cells that the wavefront's faces read are equal, bit for bit.
  // The active lanes hold consecutive faces from lane 0 on: lane l compares the
  // pairs (l, l + 1) and (l + K - 2, l + K - 1) of the wavefront's cells, which
  // cover all of them when at least K - 2 lanes are active.
  __device__ __forceinline__ bool uniform() const {
    bool differ = false;
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      differ |= __double_as_longlong(at(q, c0)) != __double_as_longlong(at(q, c0 + CS));
      differ |= __double_as_longlong(at(q, c0 + (K - 2) * CS)) != __double_as_longlong(at(q, c0 + (K - 1) * CS));
    }
    return __builtin_amdgcn_ballot_w64(differ) == 0 && __popcll(__builtin_amdgcn_ballot_w64(true)) >= K - 2;
  }
  __device__ __forceinline__ double speed(int m) const { return at(2 * NF, c0 + m * step()); }
  __device__ __forceinline__ void cell(int m, double (&X)[NF], double (&F)[NF], double& lam) const {
    const int c = c0 + m * step();
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      X[q] = at(q, c);
      F[q] = at(NF + q, c);
    }
    lam = at(2 * NF, c);
  }
  __device__ __forceinline__ void roe(int sd, RoeIn<NF>& r) const {
    const int c = c0 + (K / 2 - 1 + sd) * step();
    r.rs = at(2 * NF + 1, c);
#pragma unroll
    for (int d = 0; d < NF - 2; ++d) r.u[d] = at(2 * NF + 2 + d, c);
    r.H = at(3 * NF, c);
  }
  __device__ __forceinline__ double value(int m) const { return at(0, c0 + m * step()); }
};

// Stage a cell of state X at staging index c: its state and, for the Euler
// equations, its flux, signal speed and Roe inputs.
template <int NF>
__device__ __forceinline__ void stage_put(double* stage, int nc, int c, const double (&X)[NF], double gamma) {
#pragma unroll
  for (int q = 0; q < NF; ++q) stage[q * nc + c] = X[q];
  if constexpr (NF > 1) {
    double F[NF], lam;
    RoeIn<NF> r;
    cell_physics<NF>(X, gamma, F, lam);
    roe_input<NF>(X, gamma, r);
#pragma unroll
    for (int q = 0; q < NF; ++q) stage[(NF + q) * nc + c] = F[q];
    stage[(2 * NF) * nc + c] = lam;
    stage[(2 * NF + 1) * nc + c] = r.rs;
#pragma unroll
    for (int d = 0; d < NF - 2; ++d) stage[(2 * NF + 2 + d) * nc + c] = r.u[d];
    stage[(3 * NF) * nc + c] = r.H;
  }
}

// Load cell `cell` of the grid and stage it.
template <int NF>
__device__ __forceinline__ void stage_cell(double* stage, int nc, int c, const double* __restrict__ U,
                                           const int (&fld)[NF], double gamma, long N, long cell) {
  double X[NF];
#pragma unroll
  for (int q = 0; q < NF; ++q) X[q] = U[fld[q] * N + cell];
  stage_put<NF>(stage, nc, c, X, gamma);
}

template <int NF, int K, int LIM, bool ADAPT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kFaceWaves)))
void k_sweep_row(SweepParams<NF> p) {
  constexpr int NC = 256 + K - 1;  // staged cells per segment
  constexpr int NE = RowStage<NF>::NE;
  __shared__ double stage[NE * NC];
  const int s = blockIdx.x % p.nseg;
  const long row = blockIdx.x / p.nseg;  // y + ny * z
  const int c_begin = s * p.seg;
  const int ncell = min(p.seg, p.n - c_begin);
  const bool wrap = (p.bc == 0) && (p.seg >= p.n);  // whole periodic row
  const int nface = wrap ? p.n : ncell + 1;
  const int nstage = nface + K - 1;
  const long N = (long)p.nx * p.ny * p.nz;
  const Line L{row * p.nx, 1, p.n, p.bc};
  const int t = threadIdx.x;
  // wave priority: high while the wave issues its global loads and stores
  // (staging, epilogue), normal while it computes faces, so that a block's
  // memory phase is not queued behind other blocks' arithmetic on the SIMD
  __builtin_amdgcn_s_setprio(3);

  // stage cells c_begin - K/2 .. c_begin + nface + K/2 - 2
  for (int c = t; c < nstage; c += 256) stage_cell<NF>(stage, NC, c, p.U, p.fld, p.fp.gamma, N, cell_at(L, c_begin - K / 2 + c));
  __syncthreads();

  double F[NF];
  __builtin_amdgcn_s_setprio(0);
  if (t < nface) {
    StagedCells<NF, K, 1, true, true> prov{stage, NC, t};
    uint32_t bits[2][NF];
    face_flux<NF, K, LIM, ADAPT, false>(prov, p.fp, F, bits);
  }
  // stage state of this thread's cell (staged at t + K/2), copied before the
  // staging array is reused
  double us[NF];
  if (t < ncell) {
#pragma unroll
    for (int q = 0; q < NF; ++q) us[q] = stage[q * NC + t + K / 2];
  }
  __syncthreads();  // every face has read the staged cells
  double* Fs = stage;  // reuse: [NF][257]
  if (t < nface) {
#pragma unroll
    for (int q = 0; q < NF; ++q) Fs[q * 257 + t] = F[q];
  }
  __syncthreads();
  __builtin_amdgcn_s_setprio(3);
  if (t < ncell) {
    const long cell = L.base + c_begin + t;
    EpiIn<NF> ein;
    epi_load<NF>(p, N, cell, ein);
    const int r = (wrap && t == p.n - 1) ? 0 : t + 1;
    double div[NF];
#pragma unroll
    for (int q = 0; q < NF; ++q) div[q] = (Fs[q * 257 + t] - Fs[q * 257 + r]) * p.inv_dx;
    epi_store<NF>(p, N, cell, div, ein, us, epi_dt(p));
  }
}

// ---------------------------------------------------------------------------
// Tile sweep (any axis).  A 256-thread workgroup owns a segment (or the
// whole, tile_segment) of TX adjacent lines along the axis (x columns for y
// and z, y rows for x) and walks it in chunks of FJ = 256 / TX faces per line.  Each chunk is a row sweep on a
// tile: its cells are staged in LDS (row r of the chunk at staging indices
// r TX .. r TX + TX - 1) with their flux, signal speed and Roe inputs, each
// thread computes one face, the fluxes go through LDS and each thread closes
// the cell left of its face.  The last face of a chunk is handed to the next
// chunk through LDS and face 0 of a whole periodic line is kept for its last
// cell, so M cells cost M faces (M + 1 for a segment or a transmissive line);
// only the K - 1 halo rows of each chunk are staged twice.  A wavefront's 64 faces
// form an 8 x 8 patch (8 lines by 8 faces), which a discontinuity crosses
// far less often than a strip of 64 faces along one line: most wavefronts
// then skip the limiter (StagedCells with REREAD).
// ---------------------------------------------------------------------------
template <int NF, int K>
struct SweepTile {
  static constexpr int TX = kTileColumns;
  static constexpr int FJ = 256 / TX;    // faces per column per chunk
  static constexpr int ROWS = FJ + K - 1;  // staged cells per column per chunk
};

template <int NF, int K, int LIM, bool ADAPT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kFaceWaves)))
void k_sweep_tile(SweepParams<NF> p, int axis) {
  using S = SweepTile<NF, K>;
  constexpr int TX = S::TX, FJ = S::FJ;
  constexpr int NC = S::ROWS * TX;
  constexpr int NE = RowStage<NF>::NE;
  static_assert(256 % TX == 0, "whole columns per workgroup");
  __shared__ double stage[NE * NC];
  __shared__ double Fb[NF * FJ * TX];  // face f of the chunk at row f
  __shared__ double Fc[2 * NF * TX];   // last face of chunk k at [k mod 2], for the next chunk
  __shared__ double Fw[NF * TX];       // face 0 of a periodic line, the right face of its last cell
  // tiles in XCD order: blocks b, b + 8, ... run on one XCD and take
  // consecutive tiles, so the column groups of a line share that XCD's L2
  const int nb = (int)gridDim.x, b = (int)blockIdx.x;
  const int xcd = b & 7, q8 = nb >> 3, r8 = nb & 7;
  const int tile = xcd * q8 + min(xcd, r8) + (b >> 3);
  // column groups: x columns for y and z, y rows for x
  const int ncg = ((axis == 0 ? p.ny : p.nx) + TX - 1) / TX;
  const int o = tile / ncg / p.nseg;  // z of an x or y line, y of a z line
  const int c0 = (tile / ncg % p.nseg) * p.seg;  // first cell of the segment
  const long N = (long)p.nx * p.ny * p.nz;
  const bool wrap = p.bc == 0 && p.nseg == 1;  // a whole periodic line
  const int nface = wrap ? p.n : min(p.seg, p.n - c0) + 1;  // face j lies between cells c0 + j - 1 and c0 + j
  const int nchunk = (nface + FJ - 1) / FJ;
  // A periodic x line is walked from its cell 1 (cell m of the walk is cell
  // m + 1 of the line, the last one cell 0): a chunk then closes 32
  // consecutive cells that start on a cache-line boundary, and writes them
  // whole.  On a ring every face has the same stencil either way, so the
  // fluxes and the results have the same bits.
  const int rot = (axis == 0 && wrap) ? 1 : 0;
  // Phases of a chunk, each ended by a barrier: staging; faces (their
  // fluxes into LDS); closing the cells, which reads the staged cells and
  // the fluxes from LDS.  No value is held in registers across a barrier.
  // The thread's column and line address are formed anew in each phase from
  // an opaque copy of the thread index: hoisted out of the loop they would
  // hold registers through the face computation.
  struct Where {
    int col, f;
    bool in;
    Line L;
  };
  auto where = [&]() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    Where w;
    w.col = t % TX;
    w.f = t / TX;
    const int c = (tile % ncg) * TX + w.col;
    const int nc = axis == 0 ? p.ny : p.nx;
    w.in = c < nc;
    const int cs = w.in ? c : nc - 1;  // columns beyond the grid stage a real line and store nothing
    if (axis == 0)
      w.L = Line{((long)cs + (long)p.ny * o) * p.nx, 1, p.nx, p.bc};
    else if (axis == 1)
      w.L = Line{cs + (long)p.nx * p.ny * o, p.nx, p.ny, p.bc};
    else
      w.L = Line{cs + (long)p.nx * o, (long)p.nx * p.ny, p.nz, p.bc};
    return w;
  };
  for (int k = 0; k < nchunk; ++k) {
    const int j0 = k * FJ;
    const int nfk = min(FJ, nface - j0);  // faces of this chunk per column
    __builtin_amdgcn_s_setprio(3);
    {
      const Where w = where();
      for (int r = w.f; r < nfk + K - 1; r += FJ)
        stage_cell<NF>(stage, NC, r * TX + w.col, p.U, p.fld, p.fp.gamma, N, cell_at(w.L, c0 + j0 - K / 2 + r + rot));
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(0);
    {
      const Where w = where();
      const int f = w.f, col = w.col, j = j0 + f;
      if (f < nfk) {
        double F[NF];
        StagedCells<NF, K, TX, true> prov{stage, NC, f * TX + col};
        uint32_t bits[2][NF];
        face_flux<NF, K, LIM, ADAPT, false>(prov, p.fp, F, bits);
#pragma unroll
        for (int q = 0; q < NF; ++q) Fb[(q * FJ + f) * TX + col] = F[q];
        if (f == FJ - 1) {
#pragma unroll
          for (int q = 0; q < NF; ++q) Fc[((k & 1) * NF + q) * TX + col] = F[q];
        }
        if (wrap && j == 0) {
#pragma unroll
          for (int q = 0; q < NF; ++q) Fw[q * TX + col] = F[q];
        }
      }
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(3);
    {
      // this thread closes cell c0 + j - 1 and, on a whole periodic line, the
      // last cell (right of the last face) with face 0 as its right face.  The
      // epilogue's parameters are read anew through an opaque pointer to the
      // argument: held from the kernel's start they would be spilled across
      // the face and read back lane by lane.
      long off = 0;
      asm volatile("" : "+s"(off));
      const SweepParams<NF>& pe = *(const SweepParams<NF>*)((const char*)&p + off);
      const Where w = where();
      const int f = w.f, col = w.col, j = j0 + f;
      const bool act = f < nfk && w.in;
      if (act && j >= 1) {
        const long cell = w.L.base + (long)(c0 + j - 1 + rot) * w.L.stride;
        EpiIn<NF> ein;
        epi_load<NF>(pe, N, cell, ein);
        double us[NF], div[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) {
          us[q] = stage[q * NC + (f + K / 2 - 1) * TX + col];
          const double fl = f > 0 ? Fb[(q * FJ + f - 1) * TX + col] : Fc[(((k - 1) & 1) * NF + q) * TX + col];
          div[q] = (fl - Fb[(q * FJ + f) * TX + col]) * pe.inv_dx;
        }
        epi_store<NF>(pe, N, cell, div, ein, us, epi_dt(pe));
      }
      if (wrap && act && j == nface - 1) {
        const long cell = w.L.base + (long)(rot ? 0 : j) * w.L.stride;
        EpiIn<NF> ein;
        epi_load<NF>(pe, N, cell, ein);
        double us[NF], div[NF];
#pragma unroll
        for (int q = 0; q < NF; ++q) {
          us[q] = stage[q * NC + (f + K / 2) * TX + col];
          div[q] = (Fb[(q * FJ + f) * TX + col] - Fw[q * TX + col]) * pe.inv_dx;
        }
        epi_store<NF>(pe, N, cell, div, ein, us, epi_dt(pe));
      }
    }
    __syncthreads();  // the next chunk's staging overwrites the cells read here
  }
}

// ---------------------------------------------------------------------------
// Face fluxes of one axis (and, with FLAGS, the smoothness bytes).  A
// 256-thread workgroup takes fj faces of tx lines (face_split), staged as one
// chunk of the tile sweep is: the cell physics once per cell instead of K times,
// and wavefronts whose faces are all smooth skip cutoff and limiter.  Thread t
// takes face t / tx of line t % tx and its window cell m sits at t + m tx: the
// stores of a strided axis join, and no two lanes meet in an LDS bank.  Bound by
// VALU issue like the sweeps.  1D (NF = 3) is one line, a step of one cell.
// 64^3 Euler with flags at eight points: 50 us from global memory, one thread per
// face, 25 staged.
// ---------------------------------------------------------------------------
template <int NF>
struct FacesParams {
  const double* U;
  double* Fhat;
  uint8_t* flags;
  int n, nfl, bc;  // cells and faces of a line; a periodic line's face n is its face 0
  int fj, tx;
  int width;  // lines of a row of workgroups (those of a plane, or all)
  int ncg;    // workgroups side by side in a row
  int nch;    // workgroups along a line
  int div;    // y lines in one row: the lines of a plane, else 0
  long step;          // between cells and between faces of a line
  long crow, cline;   // first cell of a line: per row, per line of the row
  long frow, fline;   // its face 0
  long cdiv, fdiv;    // per plane before the line (div)
  long N, nfaces;
  int fld[NF];
  FaceParams fp;
};

// Row, first line l0 of the row and chunk of workgroup b: side by side along a
// row, then its chunks, then the rows, so that workgroups that share cache lines
// and halo rows run close together (128^3 along y 100 us with the chunks first, 90
// so).
template <int NF>
__device__ __forceinline__ void faces_block(const FacesParams<NF>& p, int b, int tx, int& row, int& l0, int& chunk) {
  row = b / (p.ncg * p.nch);
  const int r = b - row * (p.ncg * p.nch);
  chunk = r / p.ncg;
  l0 = (r - chunk * p.ncg) * tx;
}

// Line l of row `row`, and the index of its face 0.
template <int NF>
__device__ __forceinline__ Line faces_line(const FacesParams<NF>& p, int row, int l, long& face) {
  long cell = row * p.crow + l * p.cline;
  face = row * p.frow + l * p.fline;
  if (p.div) {
    const int z = l / p.div;
    cell += z * p.cdiv;
    face += z * p.fdiv;
  }
  return Line{cell, p.step, p.n, p.bc};
}

// What the host forms of the grid for the kernels (set_lines: rows of `width`
// lines).
template <int NF>
void set_lines(FacesParams<NF>& p, int axis, int nx, int ny, int width) {
  const long plane = (long)nx * ny;
  p.width = width;
  p.step = axis == 0 ? 1 : (axis == 1 ? nx : plane);
  p.cline = axis == 0 ? nx : 1;
  p.fline = axis == 0 ? nx + 1 : 1;
  p.crow = width * p.cline;
  p.frow = width * p.fline;
  p.div = 0;
  p.cdiv = p.fdiv = 0;
  if (axis == 1 && width == nx) {
    p.crow = plane;
    p.frow = plane + nx;
  } else if (axis == 1) {
    p.div = nx;
    p.cdiv = plane - nx;
    p.fdiv = plane;
  }
}

// Staged cells of a workgroup of k_faces: three of the largest fit in a CU's LDS.
template <int NF, int K>
constexpr int kFacesCells = NF == 3 ? 256 + K - 1 : 416;

// CS: lines side by side, 0 where known at run time
template <int NF, int K, int LIM, bool ADAPT, bool FLAGS, int CS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kFaceWaves)))
void k_faces(FacesParams<NF> p) {
  constexpr int NC = kFacesCells<NF, K>;
  __shared__ double stage[RowStage<NF>::NE * NC];
  int row, l0, chunk;
  faces_block(p, (int)blockIdx.x, CS ? CS : p.tx, row, l0, chunk);
  const int j0 = chunk * p.fj;
  const int nfk = min(p.fj, p.nfl - j0);
  // This thread's place, formed anew before and after the face (an opaque copy
  // of the thread index): held across it would be spilled (a scalar face holds it).
  struct Where {
    int tx, t, f, col;
  };
  auto where = [&]() {
    Where w;
    int tt = threadIdx.x;
    if constexpr (NF > 1) asm volatile("" : "+v"(tt));
    w.tx = CS ? CS : p.tx;
    w.t = tt;
    w.f = tt / w.tx;
    w.col = tt - w.f * w.tx;
    return w;
  };
  long face;
  __builtin_amdgcn_s_setprio(3);  // high while loads and stores issue, as in the sweeps
  {
    const Where w = where();
    const Line L = faces_line<NF>(p, row, min(l0 + w.col, p.width - 1), face);  // beyond the row: its last line
    const int frows = 256 / w.tx;
    if (w.f < frows)
      for (int r = w.f; r < nfk + K - 1; r += frows)
        stage_cell<NF>(stage, NC, r * w.tx + w.col, p.U, p.fld, p.fp.gamma, p.N, cell_at(L, j0 - K / 2 + r));
  }
  __syncthreads();
  __builtin_amdgcn_s_setprio(0);
  double F[NF];
  uint32_t bits[2][NF];
  {
    const Where w = where();
    if (w.f >= nfk) return;
    StagedCells<NF, K, CS, true> prov{stage, NC, w.t, w.tx};
    face_flux<NF, K, LIM, ADAPT, FLAGS>(prov, p.fp, F, bits);
  }
  __builtin_amdgcn_s_setprio(3);
  const Where w = where();
  if (l0 + w.col >= p.width) return;
  faces_line<NF>(p, row, l0 + w.col, face);
  const long nfaces = p.nfaces;
  auto store = [&](int j) {
    const long at = face + j * p.step;
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      p.Fhat[(long)p.fld[q] * nfaces + at] = F[q];
      if constexpr (FLAGS) {
        p.flags[(long)q * nfaces + at] = (uint8_t)bits[0][q];
        p.flags[(long)(NF + q) * nfaces + at] = (uint8_t)bits[1][q];
      }
    }
  };
  store(j0 + w.f);
  if (j0 + w.f == 0 && p.nfl == p.n) store(p.n);
}

// The cells of face j of a line straight from global memory.
template <int NF, int K>
struct GridCells {
  static constexpr bool kReread = false;  // again from memory
  const double* __restrict__ U;
  long N;
  const int* fld;
  Line L;
  int j;
  double gamma;
  __device__ __forceinline__ void load(int pos, double (&X)[NF]) const {
    const long cell = cell_at(L, pos);
#pragma unroll
    for (int q = 0; q < NF; ++q) X[q] = U[fld[q] * N + cell];
  }
  __device__ __forceinline__ void cell(int m, double (&X)[NF], double (&F)[NF], double& lam) const {
    load(j - K / 2 + m, X);
    cell_physics<NF>(X, gamma, F, lam);
  }
  __device__ __forceinline__ void roe(int s, RoeIn<NF>& r) const {
    double X[NF];
    load(j - 1 + s, X);
    roe_input<NF>(X, gamma, r);
  }
};

// The same, one thread per face straight from global memory, for grids of at most
// two wavefronts per SIMD (faces_direct): no staging, no barrier and no branch, so
// that one wavefront's operations overlap, and the time does not depend on the
// data.  Threads run along x, or along the line on axis 0.  Bound by the latency
// of a face; at eight points compiled for one wavefront per SIMD where there is
// one (40x40x39 11.5 us, 13.4 by the 256 registers of two, which in 3D spill 12 to
// 60 bytes a lane, TVD5 with flags 216).  40x40x39, transmissive, us at six
// (eight) points: staged 12 to 16 (19 to 21), so 8.2 (11.5); 100x100x12 along z
// 17.4 to 19.9 (24.5 to 27) and 13.7 (21.3).
template <int NF, int K, int LIM, bool ADAPT, bool FLAGS, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_faces_direct(FacesParams<NF> p) {
  const int t = (int)(blockIdx.x * 256 + threadIdx.x);
  if (t >= p.nch) return;  // the faces of all lines
  const int r = t / p.width, row = r / p.nfl, j = r - row * p.nfl;
  long face;
  const Line L = faces_line<NF>(p, row, t - r * p.width, face);
  GridCells<NF, K> prov{p.U, p.N, p.fld, L, j, p.fp.gamma};
  double F[NF];
  uint32_t bits[2][NF];
  face_flux<NF, K, LIM, ADAPT, FLAGS>(prov, p.fp, F, bits);
  const long nfaces = p.nfaces;
  auto store = [&](int jj) {
    const long at = face + jj * p.step;
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      p.Fhat[(long)p.fld[q] * nfaces + at] = F[q];
      if constexpr (FLAGS) {
        p.flags[(long)q * nfaces + at] = (uint8_t)bits[0][q];
        p.flags[(long)(NF + q) * nfaces + at] = (uint8_t)bits[1][q];
      }
    }
  };
  store(j);
  if (j == 0 && p.nfl == p.n) store(p.n);
}

// The same for grids that leave the chip part empty, where the time is one
// workgroup's chain: one wavefront per characteristic field takes 64 faces (64 /
// TX of TX lines), wave q stores component q.  288 cells at eight points 11.8 ->
// 7.5 us, 128x128 14.7 -> 8.6, 20x20x20 16.0 -> 9.8.
template <int NF, int K, int LIM, bool ADAPT, bool FLAGS, int TX>
__global__ __launch_bounds__(64 * NF) void k_faces_fields(FacesParams<NF> p) {
  constexpr int FJ = 64 / TX, NC = (FJ + K - 1) * TX;
  __shared__ double stage[RowStage<NF>::NE * NC];
  __shared__ double fcs[NF * 64];
  int row, l0, chunk;
  faces_block(p, (int)blockIdx.x, TX, row, l0, chunk);
  const int j0 = chunk * FJ;
  const int nfk = min(FJ, p.nfl - j0);
  const int t = threadIdx.x, q = threadIdx.y, col = t % TX, f = t / TX;
  // every c of a thread is one column's: 64 NF is a multiple of TX
  long face;
  const Line L = faces_line<NF>(p, row, min(l0 + col, p.width - 1), face);
  for (int c = q * 64 + t; c < (nfk + K - 1) * TX; c += 64 * NF)
    stage_cell<NF>(stage, NC, c, p.U, p.fld, p.fp.gamma, p.N, cell_at(L, j0 - K / 2 + c / TX));
  __syncthreads();
  StagedCells<NF, K, TX, true> prov{stage, NC, min(f, nfk - 1) * TX + col};
  RoeFrame<NF> fr;
  uint32_t bits[2] = {0u, 0u};
  roe_frame<NF>(prov, p.fp.gamma, fr);
  fcs[q * 64 + t] = field_by_index<NF, K, LIM, FLAGS, ADAPT>(q, prov, fr, p.fp.tp, bits);
  __syncthreads();
  double fc[NF], Fh[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) fc[i] = fcs[i * 64 + t];
  fr.back_project(fc, Fh);
  double F = Fh[0];
#pragma unroll
  for (int i = 1; i < NF; ++i) F = q == i ? Fh[i] : F;
  if (f >= nfk || l0 + col >= p.width) return;
  const long nfaces = p.nfaces;
  auto store = [&](int j) {
    const long at = face + j * p.step;
    p.Fhat[(long)p.fld[q] * nfaces + at] = F;
    if constexpr (FLAGS) {
      p.flags[(long)q * nfaces + at] = (uint8_t)bits[0];
      p.flags[(long)(NF + q) * nfaces + at] = (uint8_t)bits[1];
    }
  };
  store(j0 + f);
  if (j0 + f == 0 && p.nfl == p.n) store(p.n);
}

// ---------------------------------------------------------------------------
// March sweep (axis 1 or 2).  blockDim = (64, LINES): x = lane, y = line.
// Each lane keeps the K cell states of its current face in an LDS ring
// (slot of window cell m: (slot0 + m) mod K) and fetches the one new cell of
// the next face while the current face is computed.
// ---------------------------------------------------------------------------
template <int NF>
struct RoeCarry {
  RoeIn<NF> r;
};
template <>
struct RoeCarry<1> {};

template <int NF, int K>
struct RingCells {
  static constexpr bool kReread = false;  // the cell flux is recomputed per read
  // values per ring slot: the cell's state and, for the Euler equations, its
  // signal speed (computed once, when the cell enters the window)
  static constexpr int NR = (NF > 1) ? NF + 1 : NF;
  const double* ring;  // LDS: [K][NR][T] with T threads per block
  int T, tid, slot0;
  double gamma;
  RoeCarry<NF>* carry;  // Roe input of the face's right cell, the next face's left
  __device__ __forceinline__ int slot(int m) const {
    const int sl = slot0 + m;
    return sl >= K ? sl - K : sl;
  }
  __device__ __forceinline__ void load(int m, double (&X)[NF]) const {
    const int sl = slot(m);
#pragma unroll
    for (int q = 0; q < NF; ++q) X[q] = ring[(sl * NR + q) * T + tid];
  }
  __device__ __forceinline__ void cell(int m, double (&X)[NF], double (&F)[NF], double& lam) const {
    load(m, X);
    cell_flux<NF>(X, cell_prim<NF>(X, gamma), gamma, F);
    lam = ring[(slot(m) * NR + NF) * T + tid];
  }
  __device__ __forceinline__ void roe(int s, RoeIn<NF>& r) const {
    if (s == 0) {
      r = carry->r;
    } else {
      double X[NF];
      load(K / 2, X);
      roe_input<NF>(X, gamma, r);
      carry->r = r;
    }
  }
  __device__ __forceinline__ double value(int m) const { return ring[slot(m) * NR * T + tid]; }
};

// Store a cell into ring slot sl (state, and the signal speed for Euler).
template <int NF, int K>
__device__ __forceinline__ void ring_put(double* ring, int T, int tid, int sl, const double (&X)[NF], double gamma) {
  constexpr int NR = RingCells<NF, K>::NR;
#pragma unroll
  for (int q = 0; q < NF; ++q) ring[(sl * NR + q) * T + tid] = X[q];
  if constexpr (NF > 1) ring[(sl * NR + NF) * T + tid] = cell_speed<NF>(cell_prim<NF>(X, gamma), gamma);
}

template <int NF, int K>
struct MarchShape {
  // lines per block: 4, or 2 when the ring of 4 lines would exceed 80 KiB
  // (two blocks per CU must fit in its 160 KiB of LDS)
  static constexpr int LINES = (K * RingCells<NF, K>::NR * 8 * 64 * 4 <= 81920) ? 4 : 2;
};

template <int NF, int K, int LIM, bool ADAPT>
__global__ __launch_bounds__((64 * MarchShape<NF, K>::LINES)) void k_sweep_march(SweepParams<NF> p, int axis) {
  constexpr int LINES = MarchShape<NF, K>::LINES;
  constexpr int T = 64 * LINES;
  __shared__ double ring[K * RingCells<NF, K>::NR * T];
  const int x = blockIdx.x * 64 + threadIdx.x;
  const int n_other = (axis == 1) ? p.nz : p.ny;
  // unit u = (line o of the other axis, segment s), o fastest: a 2D grid
  // (one other line) still fills every wavefront of the block
  const long u = ((long)blockIdx.z * gridDim.y + blockIdx.y) * LINES + threadIdx.y;
  if (x >= p.nx || u >= (long)n_other * p.nseg) return;  // no block-wide barrier follows
  const int o = (int)(u % n_other);
  const int s = (int)(u / n_other);
  const int tid = threadIdx.y * 64 + threadIdx.x;
  const long N = (long)p.nx * p.ny * p.nz;
  Line L;
  if (axis == 1)
    L = Line{x + (long)p.nx * p.ny * o, p.nx, p.ny, p.bc};
  else
    L = Line{x + (long)p.nx * o, (long)p.nx * p.ny, p.nz, p.bc};
  const int c_begin = s * p.seg;
  const int ncell = min(p.seg, p.n - c_begin);
  // faces c_begin .. c_begin + ncell; on a whole periodic line face n reads
  // the same wrapped cells as face 0, so its flux is recomputed bit for bit

  auto fetch = [&](int pos, double (&X)[NF]) {
    const long cell = cell_at(L, pos);
#pragma unroll
    for (int q = 0; q < NF; ++q) X[q] = p.U[p.fld[q] * N + cell];
  };
  // window of the first face
#pragma unroll
  for (int m = 0; m < K; ++m) {
    double X[NF];
    fetch(c_begin - K / 2 + m, X);
    ring_put<NF, K>(ring, T, tid, m, X, p.fp.gamma);
  }
  int slot0 = 0;
  RoeCarry<NF> carry;  // the first face's left cell; then handed on face to face
  if constexpr (NF > 1) {
    double X[NF];
    RingCells<NF, K>{ring, T, tid, 0, p.fp.gamma, nullptr}.load(K / 2 - 1, X);
    roe_input<NF>(X, p.fp.gamma, carry.r);
  }
  // six points: dt read once and held in a vector register.  The loop is
  // short of scalar registers, and a scalar copy spills into lanes that every
  // iteration reads back; the eight-point loop, short of vector registers
  // instead, reads it at each store.
  double dt = epi_dt(p);
  if constexpr (K == 6) asm volatile("" : "+v"(dt));
  double Fprev[NF];
  for (int t = 0; t <= ncell; ++t) {
    const int j = c_begin + t;
    const bool more = (t < ncell);
    double nxt[NF];
    __builtin_amdgcn_s_setprio(3);  // high while loads and stores issue, as in the row sweep
    if (more) fetch(j + K / 2, nxt);  // the new cell of face j + 1
    const long ecell = L.base + (long)(j - 1) * L.stride;  // cell closed by face j
    EpiIn<NF> ein;
    double us[NF];
    if (t > 0) epi_load<NF>(p, N, ecell, ein);
    double F[NF];
    __builtin_amdgcn_s_setprio(0);
    {
      RingCells<NF, K> prov{ring, T, tid, slot0, p.fp.gamma, &carry};
      prov.load(K / 2 - 1, us);  // cell j - 1 is window cell K/2 - 1 of face j
      uint32_t bits[2][NF];
      face_flux<NF, K, LIM, ADAPT, false>(prov, p.fp, F, bits);
    }
    __builtin_amdgcn_s_setprio(3);
    if (more) {
      ring_put<NF, K>(ring, T, tid, slot0, nxt, p.fp.gamma);
      slot0 = (slot0 + 1 == K) ? 0 : slot0 + 1;
    }
    if (t > 0) {
      double div[NF];
#pragma unroll
      for (int q = 0; q < NF; ++q) div[q] = (Fprev[q] - F[q]) * p.inv_dx;
      epi_store<NF>(p, N, ecell, div, ein, us, K == 6 ? dt : epi_dt(p));
    }
#pragma unroll
    for (int q = 0; q < NF; ++q) Fprev[q] = F[q];
  }
}

// ---------------------------------------------------------------------------
// Launch descriptors (host side)
// ---------------------------------------------------------------------------
struct FacesLaunch {
  const double* U;
  double* Fhat;
  uint8_t* flags;
  int axis, nx, ny, nz, bc;
  int fld[5];
  FaceParams fp;
  hipStream_t stream;
};

struct SweepLaunch {
  int axis;
  const double* U;
  double* R;
  const double* U0;
  double* Uout;
  double a, b, dt;
  const double* dtp;  // device dt (NULL: use dt)
  int mode;
  int nx, ny, nz, bc;
  double inv_dx;
  int seg;  // cells per segment along the axis (march sweeps)
  int fld[5];
  FaceParams fp;
  hipStream_t stream;
};

// Wavefronts up to which the faces run with one per field (four per SIMD).  us,
// one per field and all fields in one, at six (eight) points: 128x128, 1024
// wavefronts, 9.6 and 12.3 (8.6 and 14.7); 256x256, 4096, 11.7 and 11.7 (13.0 and
// 15.3); 36x31x37, 3600, 11.8 and 17.3 (17.0 and 23.2); 40x40x40, 5000, 15.9 and
// 16.7 (24.4 and 22.9); 50x50x50, 12250, 30 and 23 (46 and 31).
constexpr long kFieldsFaces = 4096;

template <int NF, int K, int LIM, bool ADAPT>
hipError_t launch_faces(const FacesLaunch& a) {
  FacesParams<NF> p;
  p.U = a.U;
  p.Fhat = a.Fhat;
  p.flags = a.flags;
  p.bc = a.bc;
  p.fp = a.fp;
  for (int q = 0; q < NF; ++q) p.fld[q] = a.fld[q];
  const int n = a.axis == 0 ? a.nx : (a.axis == 1 ? a.ny : a.nz);
  const int nfl = a.bc == 0 ? n : n + 1;
  const long nlines = (long)a.nx * a.ny * a.nz / n;
  p.n = n;
  p.nfl = nfl;
  p.N = nlines * n;
  p.nfaces = nlines * (n + 1);
  if (NF == 3 && nlines != 1) return hipErrorInvalidValue;
  const int across = a.axis == 0 ? a.ny : a.nx;
  auto take = [&](int width, int fj, int tx) {  // workgroups of fj faces of tx lines of a row
    set_lines(p, a.axis, a.nx, a.ny, width);
    p.fj = fj;
    p.tx = tx;
    p.ncg = (width + tx - 1) / tx;
    p.nch = (nfl + fj - 1) / fj;
    return nlines / width * p.ncg * p.nch;
  };
  if constexpr (NF > 1) {
    constexpr int TX = NF == 3 ? 1 : kTileColumns;
    // rows of all lines where a plane's leave more than 8 % of the columns empty
    const long rows = nlines / across * ((across + TX - 1) / TX) * TX;
    const long blocks = take(rows > 1.08 * nlines ? (int)nlines : across, 64 / TX, TX);
    if (blocks * NF <= kFieldsFaces) {
      const dim3 gr((unsigned)blocks), bl(64, NF);
      if (a.flags)
        hipLaunchKernelGGL((k_faces_fields<NF, K, LIM, ADAPT, true, TX>), gr, bl, 0, a.stream, p);
      else
        hipLaunchKernelGGL((k_faces_fields<NF, K, LIM, ADAPT, false, TX>), gr, bl, 0, a.stream, p);
      return hipGetLastError();
    }
  }
  if constexpr (NF > 3) {
    if (nlines * nfl <= 2 * kWaveFaces &&
        faces_direct(a.axis, a.bc, nfl, nlines, K, a.flags != nullptr,
                     face_split(nfl, across, nlines, K, kFacesCells<NF, K>))) {
      set_lines(p, a.axis, a.nx, a.ny, a.axis == 0 ? 1 : (a.axis == 1 ? a.nx : (int)nlines));
      p.nch = (int)(nlines * nfl);
      const dim3 gr((unsigned)((nlines * nfl + 255) / 256));
      auto go = [&](auto waves) {
        constexpr int WAVES = decltype(waves)::value;
        if (a.flags)
          hipLaunchKernelGGL((k_faces_direct<NF, K, LIM, ADAPT, true, WAVES>), gr, dim3(256), 0, a.stream, p);
        else
          hipLaunchKernelGGL((k_faces_direct<NF, K, LIM, ADAPT, false, WAVES>), gr, dim3(256), 0, a.stream, p);
      };
      if (K == 8 && nlines * nfl <= kWaveFaces)
        go(std::integral_constant<int, K == 8 ? 1 : 2>());
      else
        go(std::integral_constant<int, 2>());
      return hipGetLastError();
    }
  }
  FaceSplit sp = face_split(nfl, across, nlines, K, kFacesCells<NF, K>, a.axis != 0);
  if constexpr (NF == 1) {
    // a scalar face is a few loads and stores, which other widths only scatter
    // (80x70x60 along y 8.0 us, 6.6 by 32 x 8): the split only where the launch
    // would be too large
    const FaceSplit plain{across, 32, kTileColumns};
    if (nlines > 1 && take(plain.width, plain.fj, plain.tx) < 1l << 24) sp = plain;
  }
  const long blocks = take(sp.width, sp.fj, sp.tx);
  if (blocks >= 1l << 24) return hipErrorInvalidValue;  // 2^32 threads; the split keeps 2^31 cells below
  const dim3 gr((unsigned)blocks);
  auto go = [&](auto cs) {
    constexpr int CS = decltype(cs)::value;
    if (a.flags)
      hipLaunchKernelGGL((k_faces<NF, K, LIM, ADAPT, true, CS>), gr, dim3(256), 0, a.stream, p);
    else
      hipLaunchKernelGGL((k_faces<NF, K, LIM, ADAPT, false, CS>), gr, dim3(256), 0, a.stream, p);
  };
  if constexpr (NF == 3) {
    go(std::integral_constant<int, 1>());
  } else {
    if (p.tx == kTileColumns)
      go(std::integral_constant<int, kTileColumns>());
    else if (NF == 1 && nlines == 1)
      go(std::integral_constant<int, NF == 1 ? 1 : 0>());
    else
      go(std::integral_constant<int, 0>());
  }
  return hipGetLastError();
}

// what every sweep kernel takes over from the launch
template <int NF>
void fill_sweep(const SweepLaunch& a, SweepParams<NF>& p) {
  p.U = a.U;
  p.R = a.R;
  p.U0 = a.U0;
  p.Uout = a.Uout;
  p.a = a.a;
  p.b = a.b;
  p.dt = a.dt;
  p.dtp = a.dtp;
  p.mode = a.mode;
  p.nx = a.nx;
  p.ny = a.ny;
  p.nz = a.nz;
  p.bc = a.bc;
  p.inv_dx = a.inv_dx;
  p.fp = a.fp;
  for (int q = 0; q < NF; ++q) p.fld[q] = a.fld[q];
}

template <int NF, int K, int LIM, bool ADAPT>
hipError_t launch_sweep(const SweepLaunch& a) {
  SweepParams<NF> p;
  fill_sweep<NF>(a, p);
  if (a.axis == 0) {
    p.n = a.nx;
    p.seg = (a.bc == 0 && a.nx <= 256) ? a.nx : 255;
    p.nseg = (p.n + p.seg - 1) / p.seg;
    const long blocks = (long)p.nseg * a.ny * a.nz;
    hipLaunchKernelGGL((k_sweep_row<NF, K, LIM, ADAPT>), dim3((unsigned)blocks), dim3(256), 0, a.stream, p);
  } else {
    p.n = (a.axis == 1) ? a.ny : a.nz;
    p.seg = a.seg >= p.n ? p.n : a.seg;
    p.nseg = (p.n + p.seg - 1) / p.seg;
    const int n_other = (a.axis == 1) ? a.nz : a.ny;
    constexpr int LINES = MarchShape<NF, K>::LINES;
    const long ub = ((long)n_other * p.nseg + LINES - 1) / LINES;  // blocks of units per x group
    const long gy = ub < 65535 ? ub : 65535;
    dim3 grid((a.nx + 63) / 64, (unsigned)gy, (unsigned)((ub + gy - 1) / gy));
    hipLaunchKernelGGL((k_sweep_march<NF, K, LIM, ADAPT>), grid, dim3(64, LINES), 0, a.stream, p, a.axis);
  }
  return hipGetLastError();
}

// Tile sweep of any axis: one workgroup per segment (tile_segment) of TX adjacent
// lines.
template <int NF, int K, int LIM, bool ADAPT>
hipError_t launch_tile(const SweepLaunch& a) {
  SweepParams<NF> p;
  fill_sweep<NF>(a, p);
  if (a.axis < 0 || a.axis > 2) return hipErrorInvalidValue;
  p.n = (a.axis == 0) ? a.nx : (a.axis == 1) ? a.ny : a.nz;
  p.seg = tile_segment(a.axis, p.n, a.nx, a.ny, a.nz, a.bc);
  p.nseg = (p.n + p.seg - 1) / p.seg;
  const long tiles = tile_count(a.axis, a.nx, a.ny, a.nz) * p.nseg;
  hipLaunchKernelGGL((k_sweep_tile<NF, K, LIM, ADAPT>), dim3((unsigned)tiles), dim3(256), 0, a.stream, p, a.axis);
  return hipGetLastError();
}

}  // namespace tenom
