// Generated by gen_tables.py: exact-rational constants of the TENO-M
// reconstruction in difference form.  Do not edit.
#pragma once

template <int K> struct TenoTables;

// ---- K = 6: stencil values v[0..5] = f_(i-2) .. f_(i+3),
//      differences D[j] = v[j+1] - v[j], j = 0..4
template <> struct TenoTables<6> {
  static constexpr int NK = 4;
  // optimal linear weights d_k (maximum order)
  static __device__ __forceinline__ constexpr double d(int k) {
    return k == 0 ? (9.0 / 20.0) : k == 1 ? (3.0 / 10.0) : k == 2 ? (1.0 / 20.0) : (1.0 / 5.0);
  }
  // every beta below is beta_scale times the measure of Eq. measureTENO;
  // the cutoff scales eps by the same factor
  static constexpr double beta_scale = (3.0 / 4.0);
  // candidate fluxes minus v_i, from the candidate stencils of Table 1
  static __device__ __forceinline__ void candidates(const double* D, double* c) {
    c[0] = fma((1.0 / 3.0), D[2], (1.0 / 6.0) * D[1]);
    c[1] = fma((-1.0 / 6.0), D[3], (2.0 / 3.0) * D[2]);
    c[2] = fma((5.0 / 6.0), D[1], (-1.0 / 3.0) * D[0]);
    c[3] = fma((1.0 / 12.0), D[4], fma((-1.0 / 3.0), D[3], (3.0 / 4.0) * D[2]));
  }
  // sum_k d_k c_k: the linear scheme all smooth candidates assemble to, minus v_i
  static __device__ __forceinline__ double linear(const double* D) {
    return fma((-1.0 / 60.0), D[0] - D[4], fma((7.0 / 60.0), D[1] - D[3], 0.5 * D[2]));
  }
  // weights of the linear scheme's cells (symmetric)
  static __device__ __forceinline__ constexpr double face(int m) {
    return m == 2 || m == 3 ? (37.0 / 60.0) : m == 1 || m == 4 ? (-2.0 / 15.0) : (1.0 / 60.0);
  }
  // adjoint of candidates: Dbar[j] += sum_k (d c_k / d D_j) cbar[k]
  static __device__ __forceinline__ void candidates_vjp(const double* cbar, double* Dbar) {
    Dbar[0] = (-1.0 / 3.0) * cbar[2] + Dbar[0];
    Dbar[1] = fma((5.0 / 6.0), cbar[2], (1.0 / 6.0) * cbar[0]) + Dbar[1];
    Dbar[2] = fma((3.0 / 4.0), cbar[3], fma((2.0 / 3.0), cbar[1], (1.0 / 3.0) * cbar[0])) + Dbar[2];
    Dbar[3] = fma((-1.0 / 3.0), cbar[3], (-1.0 / 6.0) * cbar[1]) + Dbar[3];
    Dbar[4] = (1.0 / 12.0) * cbar[3] + Dbar[4];
  }
  // smoothness measures beta_k (candidates) and beta_K (full stencil)
  static __device__ __forceinline__ void betas(const double* D, double* beta, double& betaK) {
    const double s0 = ((39.0 / 64.0) * D[2]) * D[2];
    const double s1 = ((39.0 / 64.0) * D[1]) * D[1];
    {
      const double y0 = fma((-5.0 / 8.0), D[2], D[1]);
      beta[0] = fma(y0, y0, s0);
    }
    {
      const double y0 = fma((-11.0 / 8.0), D[2], D[3]);
      beta[1] = fma(y0, y0, s0);
    }
    {
      const double y0 = fma((-11.0 / 8.0), D[1], D[0]);
      beta[2] = fma(y0, y0, s1);
    }
    {
      const double y0 = fma((927.0 / 547.0), D[2], fma((-1394.0 / 547.0), D[3], D[4]));
      const double y1 = fma((-3167.0 / 2126.0), D[2], D[3]);
      beta[3] = fma((547.0 / 320.0) * y0, y0, fma((1063.0 / 2188.0) * y1, y1, (3124.0 / 3189.0) * s0));
    }
    {
      const double y0 = fma((1124555.0 / 271779.0), D[2], fma((-606571.0 / 271779.0), D[3], fma((-306207.0 / 90593.0), D[1], fma((122810.0 / 271779.0), D[4], D[0]))));
      const double y1 = fma((94709347673.0 / 22867021007.0), D[2], fma((-81876422035.0 / 22867021007.0), D[3], fma((-33861378837.0 / 22867021007.0), D[1], D[4])));
      const double y2 = fma((-294807913978694.0 / 242805260682217.0), D[2], fma((93932261176693.0 / 242805260682217.0), D[3], D[1]));
      const double y3 = fma((-5806166826175189.0 / 3848503014457426.0), D[2], D[3]);
      betaK = fma((90593.0 / 53760.0) * y0, y0, fma((22867021007.0 / 43832517120.0) * y1, y1, fma((242805260682217.0 / 153666381167040.0) * y2, y2, fma((1924251507228713.0 / 4856105213644340.0) * y3, y3, 0.9782800937737386 * s0))));
    }
  }
};

// ---- K = 8: stencil values v[0..7] = f_(i-3) .. f_(i+4),
//      differences D[j] = v[j+1] - v[j], j = 0..6
template <> struct TenoTables<8> {
  static constexpr int NK = 6;
  // optimal linear weights d_k (maximum order)
  static __device__ __forceinline__ constexpr double d(int k) {
    return k == 0 ? (3.0 / 7.0) : k == 1 ? (9.0 / 35.0) : k == 2 ? (2.0 / 35.0) : k == 3 ? (6.0 / 35.0) : k == 4 ? (1.0 / 70.0) : (1.0 / 14.0);
  }
  // every beta below is beta_scale times the measure of Eq. measureTENO;
  // the cutoff scales eps by the same factor
  static constexpr double beta_scale = (3.0 / 4.0);
  // candidate fluxes minus v_i, from the candidate stencils of Table 1
  static __device__ __forceinline__ void candidates(const double* D, double* c) {
    c[0] = (1.0 / 6.0) * (fma(2.0, D[3], D[2]));
    c[1] = (1.0 / 6.0) * (4.0 * D[3] - D[4]);
    c[2] = (1.0 / 6.0) * (fma(5.0, D[2], -2.0 * D[1]));
    c[3] = (1.0 / 12.0) * (fma(-4.0, D[4], 9.0 * D[3]) + D[5]);
    c[4] = (1.0 / 12.0) * (fma(13.0, D[2], fma(-10.0, D[1], 3.0 * D[0])));
    c[5] = (1.0 / 60.0) * (fma(-3.0, D[6], fma(14.0, D[5], fma(-29.0, D[4], 48.0 * D[3]))));
  }
  // sum_k d_k c_k: the linear scheme all smooth candidates assemble to, minus v_i
  static __device__ __forceinline__ double linear(const double* D) {
    return fma((1.0 / 280.0), D[0] - D[6], fma((-13.0 / 420.0), D[1] - D[5], fma((113.0 / 840.0), D[2] - D[4], 0.5 * D[3])));
  }
  // weights of the linear scheme's cells (symmetric)
  static __device__ __forceinline__ constexpr double face(int m) {
    return m == 3 || m == 4 ? (533.0 / 840.0) : m == 2 || m == 5 ? (-139.0 / 840.0) : m == 1 || m == 6 ? (29.0 / 840.0) : (-1.0 / 280.0);
  }
  // adjoint of candidates: Dbar[j] += sum_k (d c_k / d D_j) cbar[k]
  static __device__ __forceinline__ void candidates_vjp(const double* cbar, double* Dbar) {
    const double s0 = (1.0 / 6.0) * cbar[0];
    const double s1 = (1.0 / 6.0) * cbar[1];
    const double s2 = (1.0 / 6.0) * cbar[2];
    const double s3 = (1.0 / 12.0) * cbar[3];
    const double s4 = (1.0 / 12.0) * cbar[4];
    const double s5 = (1.0 / 60.0) * cbar[5];
    Dbar[0] = 3.0 * s4 + Dbar[0];
    Dbar[1] = fma(-10.0, s4, -2.0 * s2) + Dbar[1];
    Dbar[2] = fma(13.0, s4, fma(5.0, s2, s0)) + Dbar[2];
    Dbar[3] = fma(48.0, s5, fma(9.0, s3, fma(4.0, s1, 2.0 * s0))) + Dbar[3];
    Dbar[4] = fma(-29.0, s5, fma(-4.0, s3, -s1)) + Dbar[4];
    Dbar[5] = fma(14.0, s5, s3) + Dbar[5];
    Dbar[6] = -3.0 * s5 + Dbar[6];
  }
  // smoothness measures beta_k (candidates) and beta_K (full stencil)
  static __device__ __forceinline__ void betas(const double* D, double* beta, double& betaK) {
    const double s0 = ((39.0 / 64.0) * D[3]) * D[3];
    const double s1 = ((39.0 / 64.0) * D[2]) * D[2];
    {
      const double y0 = fma((-5.0 / 8.0), D[3], D[2]);
      beta[0] = fma(y0, y0, s0);
    }
    {
      const double y0 = fma((-11.0 / 8.0), D[3], D[4]);
      beta[1] = fma(y0, y0, s0);
    }
    {
      const double y0 = fma((-11.0 / 8.0), D[2], D[1]);
      beta[2] = fma(y0, y0, s1);
    }
    {
      const double y0 = fma((927.0 / 547.0), D[3], fma((-1394.0 / 547.0), D[4], D[5]));
      const double y1 = fma((-3167.0 / 2126.0), D[3], D[4]);
      beta[3] = fma((547.0 / 320.0) * y0, y0, fma((1063.0 / 2188.0) * y1, y1, (3124.0 / 3189.0) * s0));
    }
    {
      const double y0 = fma((927.0 / 547.0), D[2], fma((-1394.0 / 547.0), D[1], D[0]));
      const double y1 = fma((-3167.0 / 2126.0), D[2], D[1]);
      beta[4] = fma((547.0 / 320.0) * y0, y0, fma((1063.0 / 2188.0) * y1, y1, (3124.0 / 3189.0) * s1));
    }
    {
      const double y0 = fma((-86329.0 / 45316.0), D[3], fma((100839.0 / 22658.0), D[4], fma((-163185.0 / 45316.0), D[5], D[6])));
      const double y1 = fma((1813059.0 / 838195.0), D[3], fma((-41089198.0 / 14249315.0), D[4], D[5]));
      const double y2 = fma((-350813921.0 / 232768856.0), D[3], D[4]);
      beta[5] = fma((11329.0 / 3360.0) * y0, y0, fma((2849863.0 / 5800448.0) * y1, y1, fma((29096107.0 / 71246575.0) * y2, y2, (1110161041.0 / 1134748173.0) * s0)));
    }
    {
      const double y0 = fma((-1985504465170.0 / 139164877641.0), D[3], fma((1291035808745.0 / 139164877641.0), D[4], fma((33287419730.0 / 2728723091.0), D[2], fma((-148180843597.0 / 46388292547.0), D[5], fma((-760759377191.0 / 139164877641.0), D[1], fma((63540330136.0 / 139164877641.0), D[6], D[0]))))));
      const double y1 = fma(-13.515941989697778, D[3], fma(12.478417152406076, D[4], fma(7.105483305004352, D[2], fma(-5.631116607688648, D[5], fma(-1.4522842377772984, D[1], D[6])))));
      const double y2 = fma(3.8771268766168543, D[3], fma(-1.9991216022994762, D[4], fma(-3.2886087899408385, D[2], fma(0.3842944201275226, D[5], D[1]))));
      const double y3 = fma(4.238216248470905, D[3], fma(-3.6269357500773, D[4], fma(-1.5238975608025418, D[2], D[5])));
      const double y4 = fma(-1.2120737331410925, D[3], fma(0.3854478132403791, D[4], D[2]));
      const double y5 = fma(-1.508775853969574, D[3], D[4]);
      betaK = fma((46388292547.0 / 27675648000.0) * y0, y0, fma(0.5581038616642391 * y1, y1, fma(1.5708030070653975 * y2, y2, fma(0.3983582187938113 * y3, y3, fma(1.576857200520724 * y4, y4, fma(0.39470622634302344 * y5, y5, 0.9782785997787286 * s0))))));
    }
  }
};
