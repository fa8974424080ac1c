// Generated by gen_coeffs2d.py -- do not edit.
// Two-dimensional reconstruction operators of Step 5.1 (Section 2.2): the least-squares
// quartic p0 (Figure 1 stencil), the quadratics p1..p4 (Figure 2 sub-stencils) and the
// smoothness indicators of eq. 2dGHYZ for square cells.
#pragma once
namespace hw2 {

// ---------------------------------------------------------------- linear path
// One field: reflection-parity folding of the 19 inputs, then the point values of p0 from the
// folds, with a butterfly per orbit of mirror-image points.
constexpr int NFOLD = 15;
__device__ __forceinline__ void lin2d_fold(const double* in, double* f) {
  const double s0 = in[0] + in[8];
  const double s1 = in[2] + in[6];
  const double d0 = in[8] - in[0];
  const double d1 = in[2] - in[6];
  f[0] = in[4];
  f[1] = in[3] + in[5];
  f[2] = in[1] + in[7];
  f[3] = s0 + s1;
  f[4] = in[12] - in[10];
  f[5] = in[18] - in[14];
  f[6] = in[5] - in[3];
  f[7] = d0 + d1;
  f[8] = in[11];
  f[9] = in[7] - in[1];
  f[10] = d0 - d1;
  f[11] = in[16];
  f[12] = (in[8] - in[2]) - (in[6] - in[0]);
  f[13] = in[13] - in[9];
  f[14] = in[17] - in[15];
}
__device__ __forceinline__ double lin2d_fold_oo0_T(const double* in) { return (in[8] - in[6]) - (in[2] - in[0]); }
// the fold of the stencil with x and y exchanged
__device__ __forceinline__ void lin2d_transpose(const double* f, double* g) {
  g[0] = f[0];
  g[1] = f[2];
  g[2] = f[1];
  g[3] = f[3];
  g[4] = f[5];
  g[5] = f[4];
  g[6] = f[9];
  g[7] = f[10];
  g[8] = f[11];
  g[9] = f[6];
  g[10] = f[7];
  g[11] = f[8];
  g[12] = f[12];
  g[13] = f[14];
  g[14] = f[13];
}

__device__ __forceinline__ void lin2d_inner(const double* f, double* inner) {
  const double Pee_0 = fma(-0.3375, f[5], fma(-0.3375, f[4], fma(0.0011111111111111111, f[3], fma(0.08736111111111111, f[2], fma(0.08736111111111111, f[1], 0.6461111111111111 * f[0])))));
  const double Poe_1 = fma(4.6475800154489, f[8], fma(0.006454972243679028, f[7], -0.012909944487358056 * f[6]));
  const double Peo_2 = fma(4.6475800154489, f[11], fma(0.006454972243679028, f[10], -0.012909944487358056 * f[9]));
  const double Poo_3 = fma(0.9, f[14], fma(0.9, f[13], -0.0375 * f[12]));
  const double p0 = Pee_0 + Poo_3, m0 = Pee_0 - Poo_3;
  const double q0 = Poe_1 + Peo_2, r0 = Poe_1 - Peo_2;
  inner[0] = p0 - q0;
  inner[2] = m0 + r0;
  inner[6] = m0 - r0;
  inner[8] = p0 + q0;
  const double Pee_4 = fma(-0.3375, f[5], fma(0.421875, f[4], fma(-0.001388888888888889, f[3], fma(0.09236111111111112, f[2], fma(-0.10920138888888889, f[1], 1.039236111111111 * f[0])))));
  const double Peo_5 = fma(4.6475800154489, f[11], fma(-0.008068715304598786, f[10], 0.016137430609197572 * f[9]));
  inner[1] = Pee_4 - Peo_5;
  const double Pee_6 = fma(0.421875, f[5], fma(-0.3375, f[4], fma(-0.001388888888888889, f[3], fma(-0.10920138888888889, f[2], fma(0.09236111111111112, f[1], 1.039236111111111 * f[0])))));
  const double Poe_7 = fma(4.6475800154489, f[8], fma(-0.008068715304598786, f[7], 0.016137430609197572 * f[6]));
  inner[3] = Pee_6 - Poe_7;
  const double Pee_8 = fma(0.421875, f[5], fma(0.421875, f[4], fma(0.001736111111111111, f[3], fma(-0.1154513888888889, f[2], fma(-0.1154513888888889, f[1], 1.4548611111111112 * f[0])))));
  inner[4] = Pee_8;
  inner[5] = Pee_6 + Poe_7;
  inner[7] = Pee_4 + Peo_5;
}

// parity parts of the x-face points (ee oe eo oo at the outer pair)
__device__ __forceinline__ void lin2d_xparts_ng2(const double* f, double* p) {
  p[0] = fma(-0.020833333333333332, f[5], fma(-0.75, f[4], fma(0.003472222222222222, f[2], fma(0.20833333333333334, f[1], 0.5763888888888888 * f[0]))));
  p[1] = fma(5.454545454545454, f[8], 0.022727272727272728 * f[6]);
  p[2] = fma(3.674047167570346, f[11], fma(0.012028130608117204, f[10], -0.03280399256759237 * f[9]));
  p[3] = fma(0.9185117918925865, f[14], fma(0.787295821622217, f[13], -0.03499092540543187 * f[12]));
}
__device__ __forceinline__ void lin2d_xface_ng2(const double* p, double side, double* v) {
  v[0] = fma(side, fma(-side, p[2], p[1]), fma(-side, p[3], p[0]));
  v[1] = fma(side, fma(side, p[2], p[1]), fma(side, p[3], p[0]));
}

// parity parts of the x-face points (ee oe eo oo at the outer pair, ee oe at the middle)
__device__ __forceinline__ void lin2d_xparts_ng3(const double* f, double* p) {
  p[0] = fma(-0.3375, f[5], fma(-0.75, f[4], fma(0.002777777777777778, f[3], fma(0.08402777777777778, f[2], fma(0.20277777777777778, f[1], 0.4152777777777778 * f[0])))));
  p[1] = fma(5.454545454545454, f[8], fma(0.008333333333333333, f[7], 0.006060606060606061 * f[6]));
  p[2] = fma(4.6475800154489, f[11], fma(0.016137430609197572, f[10], -0.032274861218395144 * f[9]));
  p[3] = fma(1.161895003862225, f[14], fma(1.0562681853292955, f[13], -0.044011174388720646 * f[12]));
  p[4] = fma(0.421875, f[5], fma(-0.75, f[4], fma(-0.003472222222222222, f[3], fma(-0.10503472222222222, f[2], fma(0.2152777777777778, f[1], 0.7934027777777778 * f[0])))));
  p[5] = fma(5.454545454545454, f[8], fma(-0.010416666666666666, f[7], 0.043560606060606064 * f[6]));
}
__device__ __forceinline__ void lin2d_xface_ng3(const double* p, double side, double* v) {
  v[0] = fma(side, fma(-side, p[2], p[1]), fma(-side, p[3], p[0]));
  v[1] = fma(side, p[5], p[4]);
  v[2] = fma(side, fma(side, p[2], p[1]), fma(side, p[3], p[0]));
}

// ---------------------------------------------------------------- HWENO path
// Monomial order (p, q) for xi^p eta^q: by total degree, then descending p.
// (p0 from the folded inputs)
__device__ __forceinline__ void p0_coeffs(const double* f, double* c) {
  c[0] = fma(0.421875, f[5], fma(0.421875, f[4], fma(0.001736111111111111, f[3], fma(-0.1154513888888889, f[2], fma(-0.1154513888888889, f[1], 1.4548611111111112 * f[0])))));
  c[1] = fma(13.636363636363637, f[8], fma(-0.020833333333333332, f[7], -0.026515151515151516 * f[6]));
  c[2] = fma(13.636363636363637, f[11], fma(-0.020833333333333332, f[10], -0.026515151515151516 * f[9]));
  c[3] = fma(-5.625, f[4], fma(-0.020833333333333332, f[3], fma(0.041666666666666664, f[2], fma(1.4791666666666667, f[1], -2.9583333333333335 * f[0]))));
  c[4] = fma(6.818181818181818, f[14], fma(6.818181818181818, f[13], -0.3181818181818182 * f[12]));
  c[5] = fma(-5.625, f[5], fma(-0.020833333333333332, f[3], fma(1.4791666666666667, f[2], fma(0.041666666666666664, f[1], -2.9583333333333335 * f[0]))));
  c[6] = fma(-10.909090909090908, f[8], 0.45454545454545453 * f[6]);
  c[7] = fma(0.25, f[10], -0.5 * f[9]);
  c[8] = fma(0.25, f[7], -0.5 * f[6]);
  c[9] = fma(-10.909090909090908, f[11], 0.45454545454545453 * f[9]);
  c[10] = fma(3.75, f[4], fma(-0.625, f[1], 1.25 * f[0]));
  c[11] = fma(-5.454545454545454, f[13], 0.22727272727272727 * f[12]);
  c[12] = fma(0.25, f[3], fma(-0.5, f[2], fma(-0.5, f[1], f[0])));
  c[13] = fma(-5.454545454545454, f[14], 0.22727272727272727 * f[12]);
  c[14] = fma(3.75, f[5], fma(-0.625, f[2], 1.25 * f[0]));
}
__device__ __forceinline__ void p1_coeffs(const double* in, double* c) {
  c[0] = fma(-1.0, in[16], fma(-1.0, in[11], fma(1.1666666666666667, in[4], fma(-0.08333333333333333, in[3], -0.08333333333333333 * in[1]))));
  c[1] = 12.0 * in[11];
  c[2] = 12.0 * in[16];
  c[3] = fma(12.0, in[11], fma(-1.0, in[4], in[3]));
  c[4] = fma(1.0, in[4], fma(-1.0, in[3], fma(-1.0, in[1], in[0])));
  c[5] = fma(12.0, in[16], fma(-1.0, in[4], in[1]));
}
__device__ __forceinline__ void p2_coeffs(const double* in, double* c) {
  c[0] = fma(-1.0, in[16], fma(1.0, in[11], fma(-0.08333333333333333, in[5], fma(1.1666666666666667, in[4], -0.08333333333333333 * in[1]))));
  c[1] = 12.0 * in[11];
  c[2] = 12.0 * in[16];
  c[3] = fma(-12.0, in[11], fma(1.0, in[5], -1.0 * in[4]));
  c[4] = fma(1.0, in[5], fma(-1.0, in[4], fma(-1.0, in[2], in[1])));
  c[5] = fma(12.0, in[16], fma(-1.0, in[4], in[1]));
}
__device__ __forceinline__ void p3_coeffs(const double* in, double* c) {
  c[0] = fma(1.0, in[16], fma(-1.0, in[11], fma(-0.08333333333333333, in[7], fma(1.1666666666666667, in[4], -0.08333333333333333 * in[3]))));
  c[1] = 12.0 * in[11];
  c[2] = 12.0 * in[16];
  c[3] = fma(12.0, in[11], fma(-1.0, in[4], in[3]));
  c[4] = fma(1.0, in[7], fma(-1.0, in[6], fma(-1.0, in[4], in[3])));
  c[5] = fma(-12.0, in[16], fma(1.0, in[7], -1.0 * in[4]));
}
__device__ __forceinline__ void p4_coeffs(const double* in, double* c) {
  c[0] = fma(1.0, in[16], fma(1.0, in[11], fma(-0.08333333333333333, in[7], fma(-0.08333333333333333, in[5], 1.1666666666666667 * in[4]))));
  c[1] = 12.0 * in[11];
  c[2] = 12.0 * in[16];
  c[3] = fma(-12.0, in[11], fma(1.0, in[5], -1.0 * in[4]));
  c[4] = fma(1.0, in[8], fma(-1.0, in[7], fma(-1.0, in[5], in[4])));
  c[5] = fma(-12.0, in[16], fma(1.0, in[7], -1.0 * in[4]));
}
__device__ __forceinline__ double beta_p0(const double* c) {
  double b = 0.0;
  b = fma(c[1], fma(0.16666666666666666, c[8], fma(0.5, c[6], c[1])), b);
  b = fma(c[2], fma(0.5, c[9], fma(0.16666666666666666, c[7], c[2])), b);
  b = fma(c[3], fma(0.7222222222222222, c[12], fma(4.2, c[10], 4.333333333333333 * c[3])), b);
  b = fma(c[4], fma(0.5666666666666667, c[13], fma(0.5666666666666667, c[11], 1.1666666666666667 * c[4])), b);
  b = fma(c[5], fma(4.2, c[14], fma(0.7222222222222222, c[12], 4.333333333333333 * c[5])), b);
  b = fma(c[6], fma(0.041666666666666664, c[8], 39.1125 * c[6]), b);
  b = fma(c[7], fma(0.041666666666666664, c[9], 4.706944444444445 * c[7]), b);
  b = fma(c[8], 4.706944444444445 * c[8], b);
  b = fma(c[9], 39.1125 * c[9], b);
  b = fma(c[10], fma(0.35, c[12], 625.8357142857143 * c[10]), b);
  b = fma(c[11], fma(0.1375, c[13], 42.37410714285714 * c[11]), b);
  b = fma(c[12], fma(0.35, c[14], 18.886111111111113 * c[12]), b);
  b = fma(c[13], 42.37410714285714 * c[13], b);
  b = fma(c[14], 625.8357142857143 * c[14], b);
  return b;
}
__device__ __forceinline__ double beta_pq(const double* c) {
  double b = 0.0;
  b = fma(c[1], c[1], b);
  b = fma(c[2], c[2], b);
  b = fma(c[3], 4.333333333333333 * c[3], b);
  b = fma(c[4], 1.1666666666666667 * c[4], b);
  b = fma(c[5], 4.333333333333333 * c[5], b);
  return b;
}
// value of a quadratic (6 coefficients) at edge point i
__device__ __forceinline__ double edge_quad_ng2(const double* c, int i) {
  switch (i) {
  case 0: return fma(0.08333333333333333, c[5], fma(0.14433756729740643, c[4], fma(0.25, c[3], fma(-0.28867513459481287, c[2], fma(-0.5, c[1], c[0])))));
  case 1: return fma(0.08333333333333333, c[5], fma(-0.14433756729740643, c[4], fma(0.25, c[3], fma(0.28867513459481287, c[2], fma(-0.5, c[1], c[0])))));
  case 2: return fma(0.08333333333333333, c[5], fma(-0.14433756729740643, c[4], fma(0.25, c[3], fma(-0.28867513459481287, c[2], fma(0.5, c[1], c[0])))));
  case 3: return fma(0.08333333333333333, c[5], fma(0.14433756729740643, c[4], fma(0.25, c[3], fma(0.28867513459481287, c[2], fma(0.5, c[1], c[0])))));
  case 4: return fma(0.25, c[5], fma(0.14433756729740643, c[4], fma(0.08333333333333333, c[3], fma(-0.5, c[2], fma(-0.28867513459481287, c[1], c[0])))));
  case 5: return fma(0.25, c[5], fma(-0.14433756729740643, c[4], fma(0.08333333333333333, c[3], fma(-0.5, c[2], fma(0.28867513459481287, c[1], c[0])))));
  case 6: return fma(0.25, c[5], fma(-0.14433756729740643, c[4], fma(0.08333333333333333, c[3], fma(0.5, c[2], fma(-0.28867513459481287, c[1], c[0])))));
  case 7: return fma(0.25, c[5], fma(0.14433756729740643, c[4], fma(0.08333333333333333, c[3], fma(0.5, c[2], fma(0.28867513459481287, c[1], c[0])))));
  }
  return 0.0;
}
// value of a quadratic (6 coefficients) at edge point i
__device__ __forceinline__ double edge_quad_ng3(const double* c, int i) {
  switch (i) {
  case 0: return fma(0.15, c[5], fma(0.19364916731037085, c[4], fma(0.25, c[3], fma(-0.3872983346207417, c[2], fma(-0.5, c[1], c[0])))));
  case 1: return fma(0.25, c[3], fma(-0.5, c[1], c[0]));
  case 2: return fma(0.15, c[5], fma(-0.19364916731037085, c[4], fma(0.25, c[3], fma(0.3872983346207417, c[2], fma(-0.5, c[1], c[0])))));
  case 3: return fma(0.15, c[5], fma(-0.19364916731037085, c[4], fma(0.25, c[3], fma(-0.3872983346207417, c[2], fma(0.5, c[1], c[0])))));
  case 4: return fma(0.25, c[3], fma(0.5, c[1], c[0]));
  case 5: return fma(0.15, c[5], fma(0.19364916731037085, c[4], fma(0.25, c[3], fma(0.3872983346207417, c[2], fma(0.5, c[1], c[0])))));
  case 6: return fma(0.25, c[5], fma(0.19364916731037085, c[4], fma(0.15, c[3], fma(-0.5, c[2], fma(-0.3872983346207417, c[1], c[0])))));
  case 7: return fma(0.25, c[5], fma(-0.5, c[2], c[0]));
  case 8: return fma(0.25, c[5], fma(-0.19364916731037085, c[4], fma(0.15, c[3], fma(-0.5, c[2], fma(0.3872983346207417, c[1], c[0])))));
  case 9: return fma(0.25, c[5], fma(-0.19364916731037085, c[4], fma(0.15, c[3], fma(0.5, c[2], fma(-0.3872983346207417, c[1], c[0])))));
  case 10: return fma(0.25, c[5], fma(0.5, c[2], c[0]));
  case 11: return fma(0.25, c[5], fma(0.19364916731037085, c[4], fma(0.15, c[3], fma(0.5, c[2], fma(0.3872983346207417, c[1], c[0])))));
  }
  return 0.0;
}
// ---------------------------------------------------------------- adjoint path
// Transposes (accumulating into fold cotangents fb, or db[19]) of the linear point maps, of the candidate
// coefficient maps and of the edge evaluations; gradients of the indicators.
// db[19] += the transpose of lin2d_fold applied to fb
__device__ __forceinline__ void lin2d_fold_T(const double* fb, double* db) {
  const double s0 = fb[3] + fb[12], s1 = fb[3] - fb[12];
  const double d0 = fb[7] + fb[10], d1 = fb[7] - fb[10];
  db[0] += s0 - d0;
  db[8] += s0 + d0;
  db[2] += s1 + d1;
  db[6] += s1 - d1;
  db[1] += fb[2] - fb[9];
  db[3] += fb[1] - fb[6];
  db[4] += fb[0];
  db[5] += fb[1] + fb[6];
  db[7] += fb[2] + fb[9];
  db[9] += -fb[13];
  db[10] += -fb[4];
  db[11] += fb[8];
  db[12] += fb[4];
  db[13] += fb[13];
  db[14] += -fb[5];
  db[15] += -fb[14];
  db[16] += fb[11];
  db[17] += fb[14];
  db[18] += fb[5];
}

// fb += the transpose of lin2d_inner applied to ub[9]
__device__ __forceinline__ void lin2d_inner_T(const double* ub, double* fb) {
  const double pb = ub[0] + ub[8], qb = ub[8] - ub[0], mb = ub[2] + ub[6], rb = ub[2] - ub[6];
  const double ee0 = pb + mb, oo0 = pb - mb, oe0 = qb + rb, eo0 = qb - rb;
  const double ee1 = ub[1] + ub[7], eo1 = ub[7] - ub[1], ee2 = ub[3] + ub[5], oe2 = ub[5] - ub[3];
  fb[0] = fma(1.4548611111111112, ub[4], fma(1.039236111111111, ee2, fma(1.039236111111111, ee1, fma(0.6461111111111111, ee0, fb[0]))));
  fb[1] = fma(-0.1154513888888889, ub[4], fma(0.09236111111111112, ee2, fma(-0.10920138888888889, ee1, fma(0.08736111111111111, ee0, fb[1]))));
  fb[2] = fma(-0.1154513888888889, ub[4], fma(-0.10920138888888889, ee2, fma(0.09236111111111112, ee1, fma(0.08736111111111111, ee0, fb[2]))));
  fb[3] = fma(0.001736111111111111, ub[4], fma(-0.001388888888888889, ee2, fma(-0.001388888888888889, ee1, fma(0.0011111111111111111, ee0, fb[3]))));
  fb[4] = fma(0.421875, ub[4], fma(-0.3375, ee2, fma(0.421875, ee1, fma(-0.3375, ee0, fb[4]))));
  fb[5] = fma(0.421875, ub[4], fma(0.421875, ee2, fma(-0.3375, ee1, fma(-0.3375, ee0, fb[5]))));
  fb[6] = fma(0.016137430609197572, oe2, fma(-0.012909944487358056, oe0, fb[6]));
  fb[7] = fma(-0.008068715304598786, oe2, fma(0.006454972243679028, oe0, fb[7]));
  fb[8] = fma(4.6475800154489, oe2, fma(4.6475800154489, oe0, fb[8]));
  fb[9] = fma(0.016137430609197572, eo1, fma(-0.012909944487358056, eo0, fb[9]));
  fb[10] = fma(-0.008068715304598786, eo1, fma(0.006454972243679028, eo0, fb[10]));
  fb[11] = fma(4.6475800154489, eo1, fma(4.6475800154489, eo0, fb[11]));
  fb[12] = fma(-0.0375, oo0, fb[12]);
  fb[13] = fma(0.9, oo0, fb[13]);
  fb[14] = fma(0.9, oo0, fb[14]);
}

// fb += the transpose of the x faces' values (low face lo, high face hi)
__device__ __forceinline__ void lin2d_xfaces_ng2_T(const double* lo, const double* hi, double* fb) {
  const double a = lo[0] + hi[1], b = hi[1] - lo[0], c = lo[1] + hi[0], d = hi[0] - lo[1];
  const double p0 = a + c, p1 = b + d, p2 = b - d, p3 = a - c;
  fb[0] = fma(0.5763888888888888, p0, fb[0]);
  fb[1] = fma(0.20833333333333334, p0, fb[1]);
  fb[2] = fma(0.003472222222222222, p0, fb[2]);
  fb[4] = fma(-0.75, p0, fb[4]);
  fb[5] = fma(-0.020833333333333332, p0, fb[5]);
  fb[6] = fma(0.022727272727272728, p1, fb[6]);
  fb[8] = fma(5.454545454545454, p1, fb[8]);
  fb[9] = fma(-0.03280399256759237, p2, fb[9]);
  fb[10] = fma(0.012028130608117204, p2, fb[10]);
  fb[11] = fma(3.674047167570346, p2, fb[11]);
  fb[12] = fma(-0.03499092540543187, p3, fb[12]);
  fb[13] = fma(0.787295821622217, p3, fb[13]);
  fb[14] = fma(0.9185117918925865, p3, fb[14]);
}

// fb += the transpose of the x faces' values (low face lo, high face hi)
__device__ __forceinline__ void lin2d_xfaces_ng3_T(const double* lo, const double* hi, double* fb) {
  const double a = lo[0] + hi[2], b = hi[2] - lo[0], c = lo[2] + hi[0], d = hi[0] - lo[2];
  const double p0 = a + c, p1 = b + d, p2 = b - d, p3 = a - c;
  const double p4 = lo[1] + hi[1], p5 = hi[1] - lo[1];
  fb[0] = fma(0.7934027777777778, p4, fma(0.4152777777777778, p0, fb[0]));
  fb[1] = fma(0.2152777777777778, p4, fma(0.20277777777777778, p0, fb[1]));
  fb[2] = fma(-0.10503472222222222, p4, fma(0.08402777777777778, p0, fb[2]));
  fb[3] = fma(-0.003472222222222222, p4, fma(0.002777777777777778, p0, fb[3]));
  fb[4] = fma(-0.75, p4, fma(-0.75, p0, fb[4]));
  fb[5] = fma(0.421875, p4, fma(-0.3375, p0, fb[5]));
  fb[6] = fma(0.043560606060606064, p5, fma(0.006060606060606061, p1, fb[6]));
  fb[7] = fma(-0.010416666666666666, p5, fma(0.008333333333333333, p1, fb[7]));
  fb[8] = fma(5.454545454545454, p5, fma(5.454545454545454, p1, fb[8]));
  fb[9] = fma(-0.032274861218395144, p2, fb[9]);
  fb[10] = fma(0.016137430609197572, p2, fb[10]);
  fb[11] = fma(4.6475800154489, p2, fb[11]);
  fb[12] = fma(-0.044011174388720646, p3, fb[12]);
  fb[13] = fma(1.0562681853292955, p3, fb[13]);
  fb[14] = fma(1.161895003862225, p3, fb[14]);
}

// fb += the transpose of p0_coeffs applied to cb[15]
__device__ __forceinline__ void p0_coeffs_T(const double* cb, double* fb) {
  fb[0] = fma(1.25, cb[14], fma(1.0, cb[12], fma(1.25, cb[10], fma(-2.9583333333333335, cb[5], fma(-2.9583333333333335, cb[3], fma(1.4548611111111112, cb[0], fb[0]))))));
  fb[1] = fma(-0.5, cb[12], fma(-0.625, cb[10], fma(0.041666666666666664, cb[5], fma(1.4791666666666667, cb[3], fma(-0.1154513888888889, cb[0], fb[1])))));
  fb[2] = fma(-0.625, cb[14], fma(-0.5, cb[12], fma(1.4791666666666667, cb[5], fma(0.041666666666666664, cb[3], fma(-0.1154513888888889, cb[0], fb[2])))));
  fb[3] = fma(0.25, cb[12], fma(-0.020833333333333332, cb[5], fma(-0.020833333333333332, cb[3], fma(0.001736111111111111, cb[0], fb[3]))));
  fb[4] = fma(3.75, cb[10], fma(-5.625, cb[3], fma(0.421875, cb[0], fb[4])));
  fb[5] = fma(3.75, cb[14], fma(-5.625, cb[5], fma(0.421875, cb[0], fb[5])));
  fb[6] = fma(-0.5, cb[8], fma(0.45454545454545453, cb[6], fma(-0.026515151515151516, cb[1], fb[6])));
  fb[7] = fma(0.25, cb[8], fma(-0.020833333333333332, cb[1], fb[7]));
  fb[8] = fma(-10.909090909090908, cb[6], fma(13.636363636363637, cb[1], fb[8]));
  fb[9] = fma(0.45454545454545453, cb[9], fma(-0.5, cb[7], fma(-0.026515151515151516, cb[2], fb[9])));
  fb[10] = fma(0.25, cb[7], fma(-0.020833333333333332, cb[2], fb[10]));
  fb[11] = fma(-10.909090909090908, cb[9], fma(13.636363636363637, cb[2], fb[11]));
  fb[12] = fma(0.22727272727272727, cb[13], fma(0.22727272727272727, cb[11], fma(-0.3181818181818182, cb[4], fb[12])));
  fb[13] = fma(-5.454545454545454, cb[11], fma(6.818181818181818, cb[4], fb[13]));
  fb[14] = fma(-5.454545454545454, cb[13], fma(6.818181818181818, cb[4], fb[14]));
}
__device__ __forceinline__ void p1_coeffs_T(const double* cb, double* db) {
  db[0] = fma(1.0, cb[4], db[0]);
  db[1] = fma(1.0, cb[5], fma(-1.0, cb[4], fma(-0.08333333333333333, cb[0], db[1])));
  db[3] = fma(-1.0, cb[4], fma(1.0, cb[3], fma(-0.08333333333333333, cb[0], db[3])));
  db[4] = fma(-1.0, cb[5], fma(1.0, cb[4], fma(-1.0, cb[3], fma(1.1666666666666667, cb[0], db[4]))));
  db[11] = fma(12.0, cb[3], fma(12.0, cb[1], fma(-1.0, cb[0], db[11])));
  db[16] = fma(12.0, cb[5], fma(12.0, cb[2], fma(-1.0, cb[0], db[16])));
}
__device__ __forceinline__ void p2_coeffs_T(const double* cb, double* db) {
  db[1] = fma(1.0, cb[5], fma(1.0, cb[4], fma(-0.08333333333333333, cb[0], db[1])));
  db[2] = fma(-1.0, cb[4], db[2]);
  db[4] = fma(-1.0, cb[5], fma(-1.0, cb[4], fma(-1.0, cb[3], fma(1.1666666666666667, cb[0], db[4]))));
  db[5] = fma(1.0, cb[4], fma(1.0, cb[3], fma(-0.08333333333333333, cb[0], db[5])));
  db[11] = fma(-12.0, cb[3], fma(12.0, cb[1], fma(1.0, cb[0], db[11])));
  db[16] = fma(12.0, cb[5], fma(12.0, cb[2], fma(-1.0, cb[0], db[16])));
}
__device__ __forceinline__ void p3_coeffs_T(const double* cb, double* db) {
  db[3] = fma(1.0, cb[4], fma(1.0, cb[3], fma(-0.08333333333333333, cb[0], db[3])));
  db[4] = fma(-1.0, cb[5], fma(-1.0, cb[4], fma(-1.0, cb[3], fma(1.1666666666666667, cb[0], db[4]))));
  db[6] = fma(-1.0, cb[4], db[6]);
  db[7] = fma(1.0, cb[5], fma(1.0, cb[4], fma(-0.08333333333333333, cb[0], db[7])));
  db[11] = fma(12.0, cb[3], fma(12.0, cb[1], fma(-1.0, cb[0], db[11])));
  db[16] = fma(-12.0, cb[5], fma(12.0, cb[2], fma(1.0, cb[0], db[16])));
}
__device__ __forceinline__ void p4_coeffs_T(const double* cb, double* db) {
  db[4] = fma(-1.0, cb[5], fma(1.0, cb[4], fma(-1.0, cb[3], fma(1.1666666666666667, cb[0], db[4]))));
  db[5] = fma(-1.0, cb[4], fma(1.0, cb[3], fma(-0.08333333333333333, cb[0], db[5])));
  db[7] = fma(1.0, cb[5], fma(-1.0, cb[4], fma(-0.08333333333333333, cb[0], db[7])));
  db[8] = fma(1.0, cb[4], db[8]);
  db[11] = fma(-12.0, cb[3], fma(12.0, cb[1], fma(1.0, cb[0], db[11])));
  db[16] = fma(-12.0, cb[5], fma(12.0, cb[2], fma(1.0, cb[0], db[16])));
}
// gradient 2 G c of the quadratic form c^T G c
__device__ __forceinline__ void beta_p0_grad(const double* c, double* g) {
  g[0] = 0.0;
  g[1] = fma(0.16666666666666666, c[8], fma(0.5, c[6], 2.0 * c[1]));
  g[2] = fma(0.5, c[9], fma(0.16666666666666666, c[7], 2.0 * c[2]));
  g[3] = fma(0.7222222222222222, c[12], fma(4.2, c[10], 8.666666666666666 * c[3]));
  g[4] = fma(0.5666666666666667, c[13], fma(0.5666666666666667, c[11], 2.3333333333333335 * c[4]));
  g[5] = fma(4.2, c[14], fma(0.7222222222222222, c[12], 8.666666666666666 * c[5]));
  g[6] = fma(0.041666666666666664, c[8], fma(78.225, c[6], 0.5 * c[1]));
  g[7] = fma(0.041666666666666664, c[9], fma(9.41388888888889, c[7], 0.16666666666666666 * c[2]));
  g[8] = fma(9.41388888888889, c[8], fma(0.041666666666666664, c[6], 0.16666666666666666 * c[1]));
  g[9] = fma(78.225, c[9], fma(0.041666666666666664, c[7], 0.5 * c[2]));
  g[10] = fma(0.35, c[12], fma(1251.6714285714286, c[10], 4.2 * c[3]));
  g[11] = fma(0.1375, c[13], fma(84.74821428571428, c[11], 0.5666666666666667 * c[4]));
  g[12] = fma(0.35, c[14], fma(37.772222222222226, c[12], fma(0.35, c[10], fma(0.7222222222222222, c[5], 0.7222222222222222 * c[3]))));
  g[13] = fma(84.74821428571428, c[13], fma(0.1375, c[11], 0.5666666666666667 * c[4]));
  g[14] = fma(1251.6714285714286, c[14], fma(0.35, c[12], 4.2 * c[5]));
}
// gradient 2 G c of the quadratic form c^T G c
__device__ __forceinline__ void beta_pq_grad(const double* c, double* g) {
  g[0] = 0.0;
  g[1] = 2.0 * c[1];
  g[2] = 2.0 * c[2];
  g[3] = 8.666666666666666 * c[3];
  g[4] = 2.3333333333333335 * c[4];
  g[5] = 8.666666666666666 * c[5];
}
// transpose of edge_quad: cb[s] += mono_s(point i) * qb
__device__ __forceinline__ void edge_quad_ng2_T(double qb, int i, double* cb) {
  switch (i) {
  case 0: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.5, qb, cb[1]); cb[2] = fma(-0.28867513459481287, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(0.14433756729740643, qb, cb[4]); cb[5] = fma(0.08333333333333333, qb, cb[5]); break;
  case 1: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.5, qb, cb[1]); cb[2] = fma(0.28867513459481287, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(-0.14433756729740643, qb, cb[4]); cb[5] = fma(0.08333333333333333, qb, cb[5]); break;
  case 2: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.5, qb, cb[1]); cb[2] = fma(-0.28867513459481287, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(-0.14433756729740643, qb, cb[4]); cb[5] = fma(0.08333333333333333, qb, cb[5]); break;
  case 3: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.5, qb, cb[1]); cb[2] = fma(0.28867513459481287, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(0.14433756729740643, qb, cb[4]); cb[5] = fma(0.08333333333333333, qb, cb[5]); break;
  case 4: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.28867513459481287, qb, cb[1]); cb[2] = fma(-0.5, qb, cb[2]); cb[3] = fma(0.08333333333333333, qb, cb[3]); cb[4] = fma(0.14433756729740643, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 5: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.28867513459481287, qb, cb[1]); cb[2] = fma(-0.5, qb, cb[2]); cb[3] = fma(0.08333333333333333, qb, cb[3]); cb[4] = fma(-0.14433756729740643, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 6: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.28867513459481287, qb, cb[1]); cb[2] = fma(0.5, qb, cb[2]); cb[3] = fma(0.08333333333333333, qb, cb[3]); cb[4] = fma(-0.14433756729740643, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 7: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.28867513459481287, qb, cb[1]); cb[2] = fma(0.5, qb, cb[2]); cb[3] = fma(0.08333333333333333, qb, cb[3]); cb[4] = fma(0.14433756729740643, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  }
}
// transpose of edge_quad: cb[s] += mono_s(point i) * qb
__device__ __forceinline__ void edge_quad_ng3_T(double qb, int i, double* cb) {
  switch (i) {
  case 0: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.5, qb, cb[1]); cb[2] = fma(-0.3872983346207417, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(0.19364916731037085, qb, cb[4]); cb[5] = fma(0.15, qb, cb[5]); break;
  case 1: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.5, qb, cb[1]); cb[3] = fma(0.25, qb, cb[3]); break;
  case 2: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.5, qb, cb[1]); cb[2] = fma(0.3872983346207417, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(-0.19364916731037085, qb, cb[4]); cb[5] = fma(0.15, qb, cb[5]); break;
  case 3: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.5, qb, cb[1]); cb[2] = fma(-0.3872983346207417, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(-0.19364916731037085, qb, cb[4]); cb[5] = fma(0.15, qb, cb[5]); break;
  case 4: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.5, qb, cb[1]); cb[3] = fma(0.25, qb, cb[3]); break;
  case 5: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.5, qb, cb[1]); cb[2] = fma(0.3872983346207417, qb, cb[2]); cb[3] = fma(0.25, qb, cb[3]); cb[4] = fma(0.19364916731037085, qb, cb[4]); cb[5] = fma(0.15, qb, cb[5]); break;
  case 6: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.3872983346207417, qb, cb[1]); cb[2] = fma(-0.5, qb, cb[2]); cb[3] = fma(0.15, qb, cb[3]); cb[4] = fma(0.19364916731037085, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 7: cb[0] = fma(1.0, qb, cb[0]); cb[2] = fma(-0.5, qb, cb[2]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 8: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.3872983346207417, qb, cb[1]); cb[2] = fma(-0.5, qb, cb[2]); cb[3] = fma(0.15, qb, cb[3]); cb[4] = fma(-0.19364916731037085, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 9: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(-0.3872983346207417, qb, cb[1]); cb[2] = fma(0.5, qb, cb[2]); cb[3] = fma(0.15, qb, cb[3]); cb[4] = fma(-0.19364916731037085, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 10: cb[0] = fma(1.0, qb, cb[0]); cb[2] = fma(0.5, qb, cb[2]); cb[5] = fma(0.25, qb, cb[5]); break;
  case 11: cb[0] = fma(1.0, qb, cb[0]); cb[1] = fma(0.3872983346207417, qb, cb[1]); cb[2] = fma(0.5, qb, cb[2]); cb[3] = fma(0.15, qb, cb[3]); cb[4] = fma(0.19364916731037085, qb, cb[4]); cb[5] = fma(0.25, qb, cb[5]); break;
  }
}

}  // namespace hw2
