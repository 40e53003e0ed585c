// Kernels of single-line grids (1D), where a sweep is a few wavefronts and the
// time is the chain of launches, loads and one face, not throughput.
//
//  k_sweep_fields     one sweep of a 1D Euler line: a workgroup of one wavefront
//                     per characteristic field takes 64 faces, so that a face's
//                     reconstructions run side by side instead of one after the
//                     other in one lane.
//  k_batch_fields     the same for a segment of one problem of a small batch.
//  k_step_line_euler  a whole SSP-RK3 step (and its CFL step size) of a line of
//  k_step_line_scalar at most one workgroup in one launch: the state stays in
//                     LDS through the stages.
//
// The faces, step sizes and updates are those of the row sweep and the rate
// kernels, operation for operation: the same bits.
#pragma once

#include "teno_batch.h"

namespace tenom {

// ---------------------------------------------------------------------------
// One sweep, one wavefront per field
// ---------------------------------------------------------------------------
// Bound by latency: a load, the cell physics, one field's two reconstructions,
// the exchange of the fields' values, a store.  4096 cells at eight points
// (TVD): 7.4 us a sweep, 10.6 by the row sweep.  Wave q also closes component q
// of the cells.
template <int K, int LIM, bool ADAPT>
__global__ __launch_bounds__(192) void k_sweep_fields(SweepParams<3> p) {
  constexpr int NF = 3, FW = 64, NC = FW + K - 1;
  __shared__ double stage[RowStage<NF>::NE * NC];
  __shared__ double fcs[NF * FW];
  const int c_begin = blockIdx.x * p.seg;
  const int ncell = min(p.seg, p.n - c_begin);
  const bool wrap = (p.bc == 0) && (p.seg >= p.n);  // whole periodic line
  const int nface = wrap ? p.n : ncell + 1;
  const int nstage = nface + K - 1;
  const long N = p.n;
  const Line L{0, 1, p.n, p.bc};
  const int t = threadIdx.x, q = threadIdx.y, c = q * FW + t;
  if (c < nstage) stage_cell<NF>(stage, NC, c, p.U, p.fld, p.fp.gamma, N, cell_at(L, c_begin - K / 2 + c));
  // the update's operands, so that their latency hides behind the faces
  const long o = (long)p.fld[q] * N + c_begin + min(t, ncell - 1);
  const double u0 = (p.mode >= EPI_RK && p.a != 0.0) ? p.U0[o] : 0.0;
  const double r = (p.mode == EPI_ACCUM || p.mode == EPI_RK) ? p.R[o] : 0.0;
  const double dt = epi_dt(p);
  __syncthreads();
  StagedCells<NF, K, 1, true> prov{stage, NC, min(t, nface - 1)};
  RoeFrame<NF> fr;
  uint32_t bits[2] = {0u, 0u};
  roe_frame<NF>(prov, p.fp.gamma, fr);
  fcs[q * FW + t] = field_by_index<NF, K, LIM, false, ADAPT>(q, prov, fr, p.fp.tp, bits);
  __syncthreads();
  double fc[NF], Fh[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) fc[i] = fcs[i * FW + t];
  fr.back_project(fc, Fh);
  const double F = q == 0 ? Fh[0] : (q == 1 ? Fh[1] : Fh[2]);
  const double right = __shfl(F, (wrap && t == p.n - 1) ? 0 : (t + 1) & 63, 64);
  if (t >= ncell) return;
  const double div = (F - right) * p.inv_dx;
  const double us = stage[q * NC + t + K / 2];
  if (p.mode == EPI_STORE) {
    p.R[o] = div;
  } else if (p.mode == EPI_ACCUM) {
    p.R[o] = r + div;
  } else {
    const double v = fma(dt, (p.mode == EPI_RK) ? r + div : div, us);
    p.Uout[o] = (p.a != 0.0) ? fma(p.a, u0, p.b * v) : p.b * v;
  }
}

// k_batch_row's segment of 64 faces with one wavefront per field, for batches
// that leave the chip part empty.  Bound by latency: a step of 8 problems of 300
// to 3000 cells at eight points (MP) 36.5 -> 24.0 us.
template <int K, int LIM, bool ADAPT>
__global__ __launch_bounds__(192) void k_batch_fields(BatchParams<3> p) {
  constexpr int NF = 3, FW = 64, NC = FW + K - 1;
  static_assert(kTiles[0].tpb * kTiles[0].fpt == FW, "the segment table of tile 0 serves this kernel");
  __shared__ double stage[RowStage<NF>::NE * NC];
  __shared__ double fcs[NF * FW];
  const int2 sg = p.segs[blockIdx.x];
  const int prob = sg.x, c_begin = sg.y;
  const long base = p.off[prob];
  const int n = (int)(p.off[prob + 1] - base);
  const double dt = p.dt[prob], idx = p.inv_dx[prob];
  const bool wrap = (p.bc == 0) && (n <= FW);  // a whole periodic problem
  const int ncell = wrap ? n : min(FW - 1, n - c_begin);
  const int nface = wrap ? n : ncell + 1;
  const int nstage = nface + K - 1;
  const Line L{base, 1, n, p.bc};
  const int t = threadIdx.x, q = threadIdx.y, c = q * FW + t;
  if (c < nstage) {
    const long cell = cell_at(L, c_begin - K / 2 + c);
    double X[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) X[i] = p.U[i * p.total + cell];
    stage_put<NF>(stage, NC, c, X, p.fp.gamma);
  }
  const long o = q * p.total + base + c_begin + min(t, ncell - 1);
  const double u0 = p.a != 0.0 ? p.U0[o] : 0.0;
  __syncthreads();
  StagedCells<NF, K, 1, true> prov{stage, NC, min(t, nface - 1)};
  RoeFrame<NF> fr;
  uint32_t bits[2] = {0u, 0u};
  roe_frame<NF>(prov, p.fp.gamma, fr);
  fcs[q * FW + t] = field_by_index<NF, K, LIM, false, ADAPT>(q, prov, fr, p.fp.tp, bits);
  __syncthreads();
  double fc[NF], Fh[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) fc[i] = fcs[i * FW + t];
  fr.back_project(fc, Fh);
  const double F = q == 0 ? Fh[0] : (q == 1 ? Fh[1] : Fh[2]);
  const double right = __shfl(F, (wrap && t == n - 1) ? 0 : (t + 1) & 63, 64);
  if (t >= ncell) return;
  const double v = fma(dt, (F - right) * idx, stage[q * NC + t + K / 2]);
  p.Uout[o] = (p.a != 0.0) ? fma(p.a, u0, p.b * v) : p.b * v;
}

// ---------------------------------------------------------------------------
// A whole step in one workgroup
// ---------------------------------------------------------------------------
struct LineStep {
  double* U;    // state, updated in place
  double* U1;   // stage states, written where not NULL
  double* U2;
  int n, bc;
  double inv_dx;
  double dt;       // step size, or
  double cfl;      // > 0: dt = cfl / largest signal rate,
  double* dt_ws;   // written here
  double* dt_out;  // and here where not NULL
  FaceParams fp;
};

constexpr int kLineEuler = 256;    // faces per workgroup
constexpr int kLineScalar = 1024;

// cells of the longest line the step kernels take: n faces on a periodic line,
// n + 1 on a transmissive one
inline bool line_fits(int nf, int n, int bc) {
  return n + (bc == 0 ? 0 : 1) <= (nf == 1 ? kLineScalar : kLineEuler);
}

// SSP-RK3 coefficients of stage st: Uout = a U^n + b (Us + dt L(Us))
__device__ __forceinline__ double rk3_a(int st) { return st == 0 ? 0.0 : (st == 1 ? 0.75 : 1.0 / 3.0); }
__device__ __forceinline__ double rk3_b(int st) { return st == 0 ? 1.0 : (st == 1 ? 0.25 : 2.0 / 3.0); }

__device__ __forceinline__ double line_update(int st, double u0, double us, double dt, double div) {
  const double a = rk3_a(st), b = rk3_b(st), v = fma(dt, div, us);
  return (a != 0.0) ? fma(a, u0, b * v) : b * v;
}

// Bound by latency: three times the chain of k_sweep_fields.  A CFL step by
// itself, wall us, against the rate, step-size and three sweep launches: 64
// cells at six points (MP) 14.1 and 21.6, 255 17.4 and 22.1; 200 at eight 21.2
// and 26.6.
template <int K, int LIM, bool ADAPT>
__global__ __launch_bounds__(3 * kLineEuler) void k_step_line_euler(LineStep p) {
  constexpr int NF = 3, W = kLineEuler, NC = W + K - 1;
  __shared__ double stage[RowStage<NF>::NE * NC];
  __shared__ double sU[NF * W], fcs[NF * W], Fs[NF * W];
  __shared__ unsigned long long rate;
  const int n = p.n, t = threadIdx.x, q = threadIdx.y;
  const int tid = q * (int)blockDim.x + t, nthread = NF * (int)blockDim.x;
  const bool wrap = p.bc == 0;
  const int nface = wrap ? n : n + 1;
  const Line L{0, 1, n, p.bc};
  const double gamma = p.fp.gamma;
  double u0 = 0.0;
  if (t < n) {
    u0 = p.U[(long)q * n + t];
    sU[q * W + t] = u0;
  }
  if (tid == 0) rate = 0ull;
  __syncthreads();
  double dt = p.dt;
  if (p.cfl > 0.0) {
    // the largest signal rate, by the arithmetic of the rate kernel
    for (int i = tid; i < n; i += nthread) {
      const double rho = sU[i], ri = 1.0 / rho, vel = sU[W + i] * ri;
      double q2 = 0.0;
      q2 += vel * vel;
      const double pr = (gamma - 1.0) * (sU[2 * W + i] - 0.5 * rho * q2);
      const double c = sqrt(gamma * pr * ri);
      const double s = (fabs(vel) + c) * p.inv_dx;
      const double best = fmax(0.0, s);
      atomicMax(&rate, (s != s) ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(best));
    }
    __syncthreads();
    dt = p.cfl / __longlong_as_double((long long)rate);
    if (tid == 0) {
      *p.dt_ws = dt;
      if (p.dt_out) *p.dt_out = dt;
    }
  }
  double us = u0;
#pragma unroll 1
  for (int st = 0; st < 3; ++st) {
    for (int c = tid; c < nface + K - 1; c += nthread) {
      const long cell = cell_at(L, c - K / 2);
      double X[NF];
#pragma unroll
      for (int i = 0; i < NF; ++i) X[i] = sU[i * W + cell];
      stage_put<NF>(stage, NC, c, X, gamma);
    }
    __syncthreads();
    StagedCells<NF, K, 1, true> prov{stage, NC, min(t, nface - 1)};
    RoeFrame<NF> fr;
    uint32_t bits[2] = {0u, 0u};
    roe_frame<NF>(prov, gamma, fr);
    fcs[q * W + t] = field_by_index<NF, K, LIM, false, ADAPT>(q, prov, fr, p.fp.tp, bits);
    __syncthreads();
    double fc[NF], Fh[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) fc[i] = fcs[i * W + t];
    fr.back_project(fc, Fh);
    Fs[q * W + t] = q == 0 ? Fh[0] : (q == 1 ? Fh[1] : Fh[2]);
    __syncthreads();
    if (t < n) {
      const int r = (wrap && t == n - 1) ? 0 : t + 1;
      us = line_update(st, u0, us, dt, (Fs[q * W + t] - Fs[q * W + r]) * p.inv_dx);
      sU[q * W + t] = us;
      double* Uo = st == 0 ? p.U1 : (st == 1 ? p.U2 : p.U);
      if (Uo) Uo[(long)q * n + t] = us;
    }
    __syncthreads();
  }
}

// the K cells of a scalar face straight from the line's state in LDS
template <int K>
struct LineCells {
  static constexpr bool kReread = true;
  const double* s;
  Line L;
  int j;
  __device__ __forceinline__ double value(int m) const { return s[cell_at(L, j - K / 2 + m)]; }
};

// Bound by latency.  A step of 200 cells at six points (MP): 3.8 us in the kernel;
// 9.3 a call where calls follow each other, which is the host's enqueue (14.8 by
// three launches), 3.9 in a graph.
template <int K, int LIM, bool ADAPT>
__global__ __launch_bounds__(kLineScalar) void k_step_line_scalar(LineStep p) {
  __shared__ double sU[kLineScalar], Fs[kLineScalar];
  const int n = p.n, t = threadIdx.x;
  const bool wrap = p.bc == 0;
  const int nface = wrap ? n : n + 1;
  const Line L{0, 1, n, p.bc};
  const double u0 = t < n ? p.U[t] : 0.0;
  double dt = p.dt;
  if (p.cfl > 0.0) {
    const double s = fabs(p.fp.adv) * p.inv_dx;
    dt = p.cfl / ((s != s) ? s : fmax(0.0, s));
    if (t == 0) {
      *p.dt_ws = dt;
      if (p.dt_out) *p.dt_out = dt;
    }
  }
  double us = u0;
#pragma unroll 1
  for (int st = 0; st < 3; ++st) {
    if (t < n) sU[t] = us;
    __syncthreads();
    double F;
    uint32_t bits[2] = {0u, 0u};
    LineCells<K> prov{sU, L, min(t, nface - 1)};
    scalar_face<K, LIM, false, ADAPT>(prov, p.fp.adv, p.fp.tp, F, bits);
    Fs[t] = F;
    __syncthreads();
    if (t < n) {
      const int r = (wrap && t == n - 1) ? 0 : t + 1;
      us = line_update(st, u0, us, dt, (Fs[t] - Fs[r]) * p.inv_dx);
      double* Uo = st == 0 ? p.U1 : (st == 1 ? p.U2 : p.U);
      if (Uo) Uo[t] = us;
    }
  }
}

// ---------------------------------------------------------------------------
// Launch descriptors (host side)
// ---------------------------------------------------------------------------
struct LineLaunch {
  LineStep p;
  hipStream_t stream;
};

template <int NF, int K, int LIM, bool ADAPT>
hipError_t launch_step_line(const LineLaunch& a) {
  const int nface = a.p.n + (a.p.bc == 0 ? 0 : 1);
  const unsigned bx = (unsigned)((nface + 63) / 64 * 64);
  if (!line_fits(NF, a.p.n, a.p.bc)) return hipErrorInvalidValue;
  if constexpr (NF == 1)
    hipLaunchKernelGGL((k_step_line_scalar<K, LIM, ADAPT>), dim3(1), dim3(bx), 0, a.stream, a.p);
  else
    hipLaunchKernelGGL((k_step_line_euler<K, LIM, ADAPT>), dim3(1), dim3(bx, 3), 0, a.stream, a.p);
  return hipGetLastError();
}

template <int K, int LIM, bool ADAPT>
hipError_t launch_sweep_fields(const SweepLaunch& a) {
  if (a.ny != 1 || a.nz != 1 || a.axis != 0) return hipErrorInvalidValue;
  SweepParams<3> p;
  fill_sweep<3>(a, p);
  p.n = a.nx;
  p.seg = (a.bc == 0 && a.nx <= 64) ? a.nx : 63;
  p.nseg = (p.n + p.seg - 1) / p.seg;
  hipLaunchKernelGGL((k_sweep_fields<K, LIM, ADAPT>), dim3((unsigned)p.nseg), dim3(64, 3), 0, a.stream, p);
  return hipGetLastError();
}

template <int K, int LIM, bool ADAPT>
hipError_t launch_batch_fields(const BatchLaunch& a) {
  if (a.nseg <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_batch_fields<K, LIM, ADAPT>), dim3(a.nseg), dim3(64, 3), 0, a.stream, batch_params(a));
  return hipGetLastError();
}

}  // namespace tenom
