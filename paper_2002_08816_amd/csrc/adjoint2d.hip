// Reverse pass of the two-dimensional stage operator (Zhao & Qiu, arXiv 2002.08816,
// Section 2.2 and eq. RK), with the troubled-cell flags, hybrid masks and Lax-Friedrichs
// speeds of the forward pass held fixed: scalar laws on meshes with periodic and
// transmissive sides, the Euler equations also with reflective sides and on the boundaries
// of Examples 3.10 and 3.11.  A stage is  W = Lim(u)  (Step 4),
// out = a W(u^n) + b (W + dt L(W))  (eq. RK).  For scalar conservation laws its reverse is
// split in two kernels (the Euler equations: five, further below):
//
//  adjL2d   out = cg lam + cl (dL/dW)^T lam + ca acc.  The tile's stage input is staged
//           with three ghost layers, flags, limited moments and hybrid masks are re-derived
//           through the forward's own tile functions, and for every cell j of tile+1 the
//           cotangent d_j of its 19-value stencil is formed: the volume quadrature and the
//           four faces' Lax-Friedrichs fluxes give the cotangents of j's interior and edge
//           values (the flux is a sum of one term per side, so j's edge cotangents need
//           only j's own edge values and lam at j and its neighbours), which are pulled
//           back through the transposed linear maps (Step 5.2) or the reversed HWENO
//           combination (Step 5.1).  Then each tile cell gathers the entries of its
//           neighbours' d_j that refer to it: a scatter-free, deterministic transpose.
//  adjLim2d the transposed limiter Jacobian: every flagged cell of tile+1 differentiates
//           its two modified first moments with respect to their five inputs, and each
//           tile cell gathers what refers to it.
//
// Periodicity makes every LDS position a translate of a mesh cell, so a position's
// stencil cotangent equals that cell's and the gathers above are exact; at a transmissive
// side the ghosts mirror the cells beside it and their slots go back to those cells.
#include <climits>

#include "hw_adjoint.h"
#include "hw_dmr.h"
#include "hw_step.h"

namespace hw {

template <int EQ>
__device__ __forceinline__ double dflux(double u, double a) {
  if constexpr (EQ == EQ_BURGERS) return u;
  else return a;
}

// Threads of the scalar reverse kernels: their per-cell phases run over the 324 cells of tile+1,
// one round of 384 threads instead of two of 256
constexpr int AT = 384;

__device__ __forceinline__ int tq(int ly, int lx) { return (ly - 2) * R1 + (lx - 2); }

// Transmissive sides (scalar laws): the LDS position (ly, lx) of the tile with origin
// (gx0, gy0) is a ghost when it lies beyond such a side; (my, mx) receives the LDS position
// of the mesh cell it mirrors, fx / fy whether it is mirrored in x / y.
__device__ __forceinline__ bool ghost_lds(const Adj2D& P, int gx0, int gy0, int ly, int lx, int& my,
                                          int& mx, bool& fx, bool& fy) {
  const int gx = gx0 + lx, gy = gy0 + ly;
  fx = P.bcx != BC_PERIODIC && (gx < 0 || gx >= P.nx);
  fy = P.bcy != BC_PERIODIC && (gy < 0 || gy >= P.ny);
  double s;
  mx = fx ? map_index(gx, P.nx, P.bcx, s) - gx0 : lx;
  my = fy ? map_index(gy, P.ny, P.bcy, s) - gy0 : ly;
  return fx || fy;
}

// The ghosts of [lo, LX - lo)^2 take the value of the cell they mirror in m (flags, hybrid
// masks), as in the forward stage.  A ghost's mirror is never a ghost.
__device__ __forceinline__ void mirror_ghost_bytes(const Adj2D& P, int gx0, int gy0, uint8_t* m, int lo) {
  const int w = LX - 2 * lo;
  for (int q = threadIdx.x; q < w * w; q += AT) {
    const int ly = lo + q / w, lx = lo + q % w;
    int my, mx;
    bool fx, fy;
    if (ghost_lds(P, gx0, gy0, ly, lx, my, mx, fx, fy)) m[ly * LX + lx] = m[my * LX + mx];
  }
}

// Bound by the latency of its chains (80 KB of LDS and the registers of a reversed
// reconstruction leave a compute unit one or two waves per SIMD).  Burgers NG 3 at 256^2 without hybrid
// cells: 16.0 us with 256 threads, two rounds and both kinds of cells in one loop (more than
// 256 VGPRs, accumulation registers among them); 9.8 us now.  With the stencil of the hybrid loop kept
// across the directions it spilled 820 B a thread; now 96 (20 values, Burgers NG 3; 16 to 32 in the others).
template <int EQ, int NGE>
__global__ __launch_bounds__(AT, 2) void adjL2d_kernel(Adj2D P) {
  static_assert(EQ != EQ_EULER, "scalar equations only");
  constexpr int NQ = R1 * R1;                  // cells of tile+1
  __shared__ double s_in[3 * NPOS];            // stage input, then limited
  __shared__ double s_lam[3 * NPOS];           // lam on tile+2
  __shared__ double s_d[19 * NQ];              // stencil cotangents of tile+1
  __shared__ uint8_t s_T[NPOS];
  __shared__ uint8_t s_H[NPOS];
  __shared__ double s_alpha[2];

  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  int bx, by;
  tile_of_block(nx, bx, by);
  const int gx0 = bx * TX - HL, gy0 = by * TY - HL;
  const size_t plane = (size_t)nx * ny;

  // transmissive sides: ghosts are staged as mirror images (moment normal to the side
  // negated) and take the flags of the cells they mirror; they carry no cotangent of their
  // own (lam = 0, no stencil cotangent).  A ghost's trace on the side is its cell's own
  // trace, so the ghost side of a wall face's flux is added to the wall cell's trace
  // cotangent, and slots of the wall cells' stencils that refer to a ghost go back to the
  // cell it mirrors in the gather
  const bool walls = P.bcx != BC_PERIODIC || P.bcy != BC_PERIODIC;
  reduce_speeds(P.alpha, s_alpha);
  load_tiles<3, 1, AT>(P.in, 0, s_in, P.lam, 1, s_lam, nx, ny, P.bcx, P.bcy, gx0, gy0);
  __syncthreads();
  if (walls) {
    for (int q = tid; q < NPOS; q += AT) {
      int my, mx;
      bool fx, fy;
      if (ghost_lds(P, gx0, gy0, q / LX, q % LX, my, mx, fx, fy))
        s_lam[q] = s_lam[NPOS + q] = s_lam[2 * NPOS + q] = 0.0;
    }
  }
  flags_tile<EQ, AT>(s_in, P.tc_mode, P.adv0, P.adv1, P.dx, P.dy, P.h, s_T);
  __syncthreads();
  if (walls) {
    mirror_ghost_bytes(P, gx0, gy0, s_T, 1);
    __syncthreads();
  }
  if (P.tc_mode != TC_NONE) limit_tile<EQ, AT>(s_in, s_T, 0.0, P.w);
  hybrid_tile<AT>(s_T, s_H);
  __syncthreads();

  const double ax = s_alpha[0], ay = s_alpha[1];
  const double idx = 1.0 / P.dx, idy = 1.0 / P.dy;
  const double* node = Gauss<NGE>::node;
  const double* wt = Gauss<NGE>::wt;

  // the stencil cotangents of one cell of tile+1, by its kind: a hybrid cell's reconstruction
  // takes the registers of several linear ones, so the kinds have loops of their own
  auto stencil_cotangents = [&](int q, auto kind) {
    constexpr bool hyb = decltype(kind)::value;
    const int ly = 2 + q / R1, lx = 2 + q % R1;
    if ((s_H[ly * LX + lx] != 0) != hyb) return;
    double in19[19], fold[hw2::NFOLD], d[19], fb[hw2::NFOLD];
#pragma unroll
    for (int k = 0; k < 19; ++k) d[k] = 0.0;
#pragma unroll
    for (int k = 0; k < hw2::NFOLD; ++k) fb[k] = 0.0;
    int wall = 0;   // bits: low x, high x, low y, high y face on a transmissive side
    if (walls) {
      int my, mx;
      bool fx, fy;
      if (ghost_lds(P, gx0, gy0, ly, lx, my, mx, fx, fy)) {
#pragma unroll
        for (int k = 0; k < 19; ++k) s_d[k * NQ + q] = 0.0;
        return;
      }
      const int gxq = gx0 + lx, gyq = gy0 + ly;
      if (P.bcx != BC_PERIODIC) wall |= (gxq == 0 ? 1 : 0) | (gxq == nx - 1 ? 2 : 0);
      if (P.bcy != BC_PERIODIC) wall |= (gyq == 0 ? 4 : 0) | (gyq == ny - 1 ? 8 : 0);
    }
    gather19<1>(s_in, 0, ly, lx, in19);
    hw2::lin2d_fold(in19, fold);
    const double lU = S(s_lam, 0, ly, lx);
    // volume terms of eq. ode2: the x moment gains (1/dx) sum w f(u(G)), the y moment
    // (1/dy) sum w g(u(G))
    {
      double inner[9], ub[9];
      hw2::lin2d_inner(fold, inner);
      const double lv = S(s_lam, 1, ly, lx) * idx, lw = S(s_lam, 2, ly, lx) * idy;
#pragma unroll
      for (int p = 0; p < 9; ++p) {
        const double wq = VW[p % 3] * VW[p / 3];
        ub[p] = wq * (lv * dflux<EQ>(inner[p], P.adv0) + lw * dflux<EQ>(inner[p], P.adv1));
      }
      hw2::lin2d_inner_T(ub, fb);
    }
    double beta[5], om[5];
    if constexpr (hyb) hweno2d_weights<NGE>(in19, fold, P.w, beta, om);
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      const int oy = dir, ox = 1 - dir;
      const double inv = dir == 0 ? idx : idy;
      const double a = dir == 0 ? ax : ay;
      const double adv = dir == 0 ? P.adv0 : P.adv1;
      // the moment fed by (F_L + F_R)/2 and the one fed by the node-weighted difference
      const int fP = dir == 0 ? 1 : 2, fQ = 3 - fP;
      const double cP = S(s_lam, fP, ly, lx), cQ = S(s_lam, fQ, ly, lx);
      const double mU = S(s_lam, 0, ly - oy, lx - ox), mP = S(s_lam, fP, ly - oy, lx - ox),
                   mQ = S(s_lam, fQ, ly - oy, lx - ox);
      const double pU = S(s_lam, 0, ly + oy, lx + ox), pP = S(s_lam, fP, ly + oy, lx + ox),
                   pQ = S(s_lam, fQ, ly + oy, lx + ox);
      double v[2 * NGE];
      if constexpr (hyb) hweno2d_combine<NGE>(in19, fold, P.w, dir, om, v);
      else lin_faces<NGE>(fold, dir, v, v + NGE);
      double ub[2 * NGE];
#pragma unroll
      for (int k = 0; k < NGE; ++k) {
        const double wk = wt[k] * inv, nk = node[k];
        // low face: this cell's left/bottom face and the neighbour's right/top face
        const double Flo = wk * ((lU - 0.5 * cP + nk * cQ) - (mU + 0.5 * mP + nk * mQ));
        // high face: this cell's right/top face and the neighbour's left/bottom face
        const double Fhi = wk * ((pU - 0.5 * pP + nk * pQ) - (lU + 0.5 * cP + nk * cQ));
        // F = (f(u-) + f(u+))/2 - a (u+ - u-)/2: this cell is u+ on the low face, u- on
        // the high face
        ub[k] = Flo * 0.5 * (dflux<EQ>(v[k], adv) - a);
        ub[NGE + k] = Fhi * 0.5 * (dflux<EQ>(v[NGE + k], adv) + a);
        // a face on a transmissive side: the ghost's trace there is this cell's, so the
        // ghost side of the flux (u- on the low face, u+ on the high face) is this cell's
        if ((wall >> (2 * dir)) & 1) ub[k] += Flo * 0.5 * (dflux<EQ>(v[k], adv) + a);
        if ((wall >> (2 * dir + 1)) & 1) ub[NGE + k] += Fhi * 0.5 * (dflux<EQ>(v[NGE + k], adv) - a);
      }
      if constexpr (hyb) {
        int l2 = ly;   // opaque: the stencil is read again, not kept
        asm volatile("" : "+v"(l2));
        gather19<1>(s_in, 0, l2, lx, in19);
        hw2::lin2d_fold(in19, fold);
        hweno2d_field_adj<NGE>(in19, fold, P.w, dir, beta, om, ub, d);
      }
      else lin_faces_T<NGE>(dir, ub, ub + NGE, fb);
    }
    hw2::lin2d_fold_T(fb, d);
#pragma unroll
    for (int k = 0; k < 19; ++k) s_d[k * NQ + q] = d[k];
  };
  for (int q = tid; q < NQ; q += AT) stencil_cotangents(q, std::false_type());
  for (int q = tid; q < NQ; q += AT) stencil_cotangents(q, std::true_type());
  __syncthreads();

  // gather: slot k of cell j's stencil refers to cell j + offset_k
  const int tx = tid % TX, ty = tid / TX;
  const int lx = tx + HL, ly = ty + HL;
  const int gx = gx0 + lx, gy = gy0 + ly;
  if (ty >= TY || gx >= nx || gy >= ny) return;
  double Wb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 9; ++k) Wb[0] += s_d[k * NQ + tq(ly - (k / 3 - 1), lx - (k % 3 - 1))];
  const int cy[5] = {-1, 0, 0, 0, 1}, cx[5] = {0, -1, 0, 1, 0};
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    Wb[1] += s_d[(9 + k) * NQ + tq(ly - cy[k], lx - cx[k])];
    Wb[2] += s_d[(14 + k) * NQ + tq(ly - cy[k], lx - cx[k])];
  }
  if (walls) {
    // slots of the mesh cells' stencils that refer to a ghost mirroring this cell (one ghost
    // layer beside each transmissive side, and the corner between two; ghosts further out
    // belong to no mesh cell's stencil, and ghosts have no stencil cotangent)
    int xs[3] = {lx, INT_MIN, INT_MIN}, ys[3] = {ly, INT_MIN, INT_MIN};
    int nxs = 1, nys = 1;
    const int gcand[4] = {-1, -2, nx, nx + 1}, hcand[4] = {-1, -2, ny, ny + 1};
    for (int c = 0; c < 4; ++c) {
      double s;
      if (P.bcx != BC_PERIODIC && nxs < 3 && map_index(gcand[c], nx, P.bcx, s) == gx) xs[nxs++] = gcand[c] - gx0;
      if (P.bcy != BC_PERIODIC && nys < 3 && map_index(hcand[c], ny, P.bcy, s) == gy) ys[nys++] = hcand[c] - gy0;
    }
    auto inq = [](int y, int x) { return y >= 2 && y < LX - 2 && x >= 2 && x < LX - 2; };
    for (int a = 0; a < nys; ++a)
      for (int b = 0; b < nxs; ++b) {
        if (a == 0 && b == 0) continue;
        const int qy = ys[a], qx = xs[b];
        const double sx = b > 0 ? -1.0 : 1.0, sy = a > 0 ? -1.0 : 1.0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          const int py = qy - (k / 3 - 1), px = qx - (k % 3 - 1);
          if (inq(py, px)) Wb[0] += s_d[k * NQ + tq(py, px)];
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          const int py = qy - cy[k], px = qx - cx[k];
          if (!inq(py, px)) continue;
          Wb[1] += sx * s_d[(9 + k) * NQ + tq(py, px)];
          Wb[2] += sy * s_d[(14 + k) * NQ + tq(py, px)];
        }
      }
  }
  const size_t gi = (size_t)gy * nx + gx;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const double l = S(s_lam, f, ly, lx);
    double o = P.cg * l + P.cl * Wb[f];
    if (P.ca != 0.0) o = fma(P.ca, P.acc_in[f * plane + gi], o);
    P.out[f * plane + gi] = o;
    if (P.acc_mode == 1) P.acc_out[f * plane + gi] = P.kl * l;
    else if (P.acc_mode == 2) P.acc_out[f * plane + gi] = fma(P.kl, l, P.acc_in[f * plane + gi]);
  }
}

template <int EQ>
__global__ __launch_bounds__(AT, 2) void adjLim2d_kernel(Adj2D P) {
  static_assert(EQ != EQ_EULER, "scalar equations only");
  constexpr int NQ = R1 * R1;
  __shared__ double s_in[3 * NPOS];
  __shared__ double s_g[3 * NPOS];     // cotangent of the limited input, tile+1
  __shared__ double s_c[10 * NQ];      // limiter partials of tile+1: x (um,u0,up,vm,vp), y
  __shared__ uint8_t s_T[NPOS];

  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  int bx, by;
  tile_of_block(nx, bx, by);
  const int gx0 = bx * TX - HL, gy0 = by * TY - HL;
  const size_t plane = (size_t)nx * ny;

  const bool walls = P.bcx != BC_PERIODIC || P.bcy != BC_PERIODIC;
  load_tiles<3, 1, AT>(P.in, 0, s_in, P.lam, 2, s_g, nx, ny, P.bcx, P.bcy, gx0, gy0);
  __syncthreads();
  flags_tile<EQ, AT>(s_in, P.tc_mode, P.adv0, P.adv1, P.dx, P.dy, P.h, s_T);
  __syncthreads();
  if (walls) {
    mirror_ghost_bytes(P, gx0, gy0, s_T, 1);
    __syncthreads();
  }
  const bool lim = P.tc_mode != TC_NONE;
  for (int q = tid; q < NQ; q += AT) {
    const int ly = 2 + q / R1, lx = 2 + q % R1;
    double gxv[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, gyv[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    int my, mx;
    bool fx, fy;
    // a ghost's limited moments are the mirror of its cell's: no limiter of its own
    const bool ghost = walls && ghost_lds(P, gx0, gy0, ly, lx, my, mx, fx, fy);
    if (lim && !ghost && s_T[ly * LX + lx]) {
      limit_moment_adj(S(s_in, 0, ly, lx - 1), S(s_in, 0, ly, lx), S(s_in, 0, ly, lx + 1),
                       S(s_in, 1, ly, lx - 1), S(s_in, 1, ly, lx + 1), P.w.lim, P.w.eps,
                       S(s_g, 1, ly, lx), gxv);
      limit_moment_adj(S(s_in, 0, ly - 1, lx), S(s_in, 0, ly, lx), S(s_in, 0, ly + 1, lx),
                       S(s_in, 2, ly - 1, lx), S(s_in, 2, ly + 1, lx), P.w.lim, P.w.eps,
                       S(s_g, 2, ly, lx), gyv);
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      s_c[m * NQ + q] = gxv[m];
      s_c[(5 + m) * NQ + q] = gyv[m];
    }
  }
  __syncthreads();

  const int tx = tid % TX, ty = tid / TX;
  const int lx = tx + HL, ly = ty + HL;
  const int gx = gx0 + lx, gy = gy0 + ly;
  if (ty >= TY || gx >= nx || gy >= ny) return;
  const int qc = tq(ly, lx), qr = tq(ly, lx + 1), ql = tq(ly, lx - 1);
  const int qt = tq(ly + 1, lx), qb = tq(ly - 1, lx);
  const bool mine = lim && s_T[ly * LX + lx];
  // the right neighbour sees this cell as (um, vm), the left one as (up, vp)
  const double ub = S(s_g, 0, ly, lx) + s_c[1 * NQ + qc] + s_c[0 * NQ + qr] + s_c[2 * NQ + ql] +
                    s_c[6 * NQ + qc] + s_c[5 * NQ + qt] + s_c[7 * NQ + qb];
  double vb = (mine ? 0.0 : S(s_g, 1, ly, lx)) + s_c[3 * NQ + qr] + s_c[4 * NQ + ql];
  double wb = (mine ? 0.0 : S(s_g, 2, ly, lx)) + s_c[8 * NQ + qt] + s_c[9 * NQ + qb];
  double ubw = 0.0;
  if (mine) {
    // beside a transmissive side this cell's own limiter reads the ghost mirroring it
    if (P.bcx != BC_PERIODIC && gx == 0) { ubw += s_c[0 * NQ + qc]; vb -= s_c[3 * NQ + qc]; }
    if (P.bcx != BC_PERIODIC && gx == nx - 1) { ubw += s_c[2 * NQ + qc]; vb -= s_c[4 * NQ + qc]; }
    if (P.bcy != BC_PERIODIC && gy == 0) { ubw += s_c[5 * NQ + qc]; wb -= s_c[8 * NQ + qc]; }
    if (P.bcy != BC_PERIODIC && gy == ny - 1) { ubw += s_c[7 * NQ + qc]; wb -= s_c[9 * NQ + qc]; }
  }
  const size_t gi = (size_t)gy * nx + gx;
  P.out[gi] = ub + ubw;
  P.out[plane + gi] = vb;
  P.out[2 * plane + gi] = wb;
}

// ================================================================== 2D Euler
// The reverse of a 2D Euler stage (eq. euler2) on a mesh with periodic, transmissive or
// reflective sides, with flags, hybrid masks and speeds held fixed.  The forward's own prepasses (flags and work lists, the limiter
// over the flagged list, HWENO over the hybrid list) are rerun on the stored stage input
// first, so the reverse sees the forward's decisions and values bit for bit; then:
//
//  adjEL2d    per tile cell j: the cotangents of j's nine interior values (volume
//             quadrature through the transposed flux Jacobians) and of its edge values
//             (the four faces' Lax-Friedrichs fluxes), pulled back through the transposed
//             linear maps (Step 5.2) to j's 4 x 19 stencil values, which the tile sums by
//             the position they refer to.  For a hybrid cell only the interior part; its
//             edge cotangents are stored for the next pass.
//  adjEhw2d   over the hybrid list, four lanes per cell and direction (lane f:
//             characteristic field f and physical component f), the x and y directions in
//             the two waves of a pair: the reversed characteristic HWENO combination (Step
//             5.1, Remark 4), including the eigenvectors' dependence on the cell average:
//             the hybrid cells' own 4 x 19 stencil cotangents.
//  adjEG2d    per cell: the gather of the sums and the hybrid cells' stencil cotangents,
//             out = cg lam + cl (dL/dW)^T lam + ca acc, and the running cotangent of u^n;
//  adjEC2d    over the forward's flagged list: the reversed characteristic limiter of both
//             directions (Step 4, Remark 4);
//  adjElim2d  per cell: the transposed limiter Jacobian (gathers of the flagged cells'
//             limiter cotangents that refer to it).
// A ghost position beside a transmissive or reflective side holds the mirrored cell's
// values; the kernels never form a ghost's own cotangent but add what refers to a ghost to
// the cell it mirrors (the instances for walls; periodic meshes use plain wrap-around).
// On the forward step, positions beyond the channel's sides and inside the step do the
// same with their source cell, and those beyond the inflow side hold the prescribed free
// stream, which carries no cotangent.

__device__ __forceinline__ int wrap(int g, int n) {
  double s;
  return map_index(g, n, BC_PERIODIC, s);
}

// The four values of a quad of lanes through ds_bpermute.  The reverse list kernels use it
// instead of the DPP quad moves of quad_gather: in several forms of these kernels (a
// run-time direction, mirrored stencil loads) the DPP moves returned values that were not
// the source lanes' with the compiler used here, while the same code through ds_bpermute
// agrees with the complex-step derivative of the oracle.
__device__ __forceinline__ void quad_gather_p(double x, double* out) {
  const int base = (int)(threadIdx.x & 63) & ~3;
#pragma unroll
  for (int g = 0; g < 4; ++g) out[g] = __shfl(x, base + g, 64);
}

// The Euler reverse on meshes with transmissive or reflective sides: a ghost position holds
// the values of the mesh cell it mirrors (Step 4's limiter and the stencils read it), with
// the moment normal to each side it lies beyond negated and, across a reflective side,
// the normal momentum too.  Its own cotangent is never formed: the reverse adds it to the
// cell it mirrors, through the same factors.
struct Mirror {
  int g;          // the mesh cell
  bool mx, my;    // mirrored across an x side / a y side
};
__device__ __forceinline__ Mirror mirror_of(const Adj2D& P, int gy, int gx) {
  double sx, sy;
  const int x = map_index(gx, P.nx, P.bcx, sx), y = map_index(gy, P.ny, P.bcy, sy);
  return {y * P.nx + x, sx < 0.0, sy < 0.0};
}
// factor of moment m (0 average, 1 x moment, 2 y moment) of component c at such a position
__device__ __forceinline__ double mirror_factor(const Adj2D& P, int m, int c, bool mx, bool my) {
  double f = 1.0;
  if (c == 1 && mx && P.bcx == BC_REFLECTIVE) f = -f;
  if (c == 2 && my && P.bcy == BC_REFLECTIVE) f = -f;
  if ((m == 1 && mx) || (m == 2 && my)) f = -f;
  return f;
}

// Boundary forms of the Euler reverse instances: periodic in both directions; a rectangle
// with a transmissive or reflective side (the mirrors above); and the resolver family: the
// forward step (Example 3.11), where a position outside the fluid -- beyond a side of the
// channel or inside the step -- takes the values of one fluid cell under the position rule
// of step::resolve, or the prescribed inflow state beyond the left side; the double Mach
// reflection (Example 3.10), whose positions right of the mesh mirror the outflow side,
// those below it from x = 1/6 on mirror the wall, and all others outside the mesh are
// prescribed (the stage's table of exact cut-cell moments).  Prescribed values carry no
// cotangent.
enum { ADJ_PERIODIC = 0, ADJ_WALLS = 1, ADJ_STEP = 2, ADJ_DMR = 3 };

__device__ __forceinline__ bool step_fluid(const Adj2D& P, int x, int y) {
  return x >= 0 && x < P.nx && y >= 0 && y < P.ny && !step::solid(x, y, P.si, P.sj);
}
// factor of moment m (0 average, 1 x moment, 2 y moment) of component c at a position
// whose source is r
__device__ __forceinline__ double step_factor(const step::Src& r, int m, int c) {
  const double w = step::comp_factor(r, c);
  return m == 0 ? w : (m == 1 ? r.sx * w : r.sy * w);
}
// The non-fluid side of face `side` (0 low, 1 high) of the fluid cell (gx, gy) in
// direction dir under the face rule: -2 a fluid cell or the prescribed inflow (no
// dependence on this cell's trace), -1 the outflow (this cell's own trace), 1 + dir a wall
// (the own trace with the normal momentum, component 1 + dir, reversed).
__device__ __forceinline__ int step_face(const Adj2D& P, int gx, int gy, int dir, int side) {
  const int qx = gx + (dir == 0 ? 2 * side - 1 : 0), qy = gy + (dir == 1 ? 2 * side - 1 : 0);
  if (step_fluid(P, qx, qy) || qx < 0) return -2;
  return qx >= P.nx ? -1 : 1 + dir;
}

// The double Mach reflection's position rule.  A prescribed position's values come from
// the stage's table by position (pres_value); its x, y are only clamped into the mesh.
__device__ __forceinline__ step::Src dmr_src(const Adj2D& P, int gx, int gy) {
  step::Src r{gx, gy, 1.0, 1.0, 1.0, 1.0, false};
  if (dmr::prescribed(gx, gy, P.nx, P.ny, P.x0, P.dx)) {
    r.pres = true;
    r.x = gx < 0 ? 0 : (gx >= P.nx ? P.nx - 1 : gx);
    r.y = gy < 0 ? 0 : (gy >= P.ny ? P.ny - 1 : gy);
    return r;
  }
  if (gx >= P.nx) {               // outflow: the even mirror
    r.x = 2 * P.nx - 1 - gx;
    r.sx = -1.0;
  }
  if (gy < 0) {                   // the wall: rho v reversed
    r.y = -1 - gy;
    r.sy = -1.0;
    r.fv = -1.0;
  }
  // positions beyond the ghost layers (partial tiles) are read by no mesh cell
  r.x = r.x < 0 ? 0 : (r.x >= P.nx ? P.nx - 1 : r.x);
  r.y = r.y < 0 ? 0 : (r.y >= P.ny ? P.ny - 1 : r.y);
  return r;
}
// the resolver family's source of a position, whether a mesh position is a fluid cell,
// field (m, c) of a prescribed position (gx, gy), and the non-fluid side of a face (the
// codes of step_face)
template <int BND>
__device__ __forceinline__ step::Src src_of(const Adj2D& P, int gx, int gy) {
  if constexpr (BND == ADJ_STEP) return step::resolve(gx, gy, P.nx, P.ny, P.si, P.sj);
  else return dmr_src(P, gx, gy);
}
template <int BND>
__device__ __forceinline__ bool fluid_of(const Adj2D& P, int x, int y) {
  if constexpr (BND == ADJ_STEP) return step_fluid(P, x, y);
  else return x >= 0 && x < P.nx && y >= 0 && y < P.ny;
}
template <int BND>
__device__ __forceinline__ double pres_value(const Adj2D& P, int m, int c, int gx, int gy) {
  if constexpr (BND == ADJ_STEP) return m == 0 ? sel4(P.uin, c) : 0.0;
  else return P.dtab[(size_t)(m * 4 + c) * dmr::ring2_size(P.nx, P.ny) + dmr::ring2_index(gx, gy, P.nx, P.ny)];
}
// whether the fluid cell (gx, gy) may be the source of a position outside the fluid that a fluid
// cell's stencil holds: those positions are one layer deep, and their source is the cell
// beside the boundary, or the next one where a step one cell wide meets the outflow
template <int BND>
__device__ __forceinline__ bool beside_boundary(const Adj2D& P, int gx, int gy) {
  bool b = gx == 0 || gx >= P.nx - 2 || gy == 0 || gy == P.ny - 1;
  if constexpr (BND == ADJ_STEP) b = b || (gx >= P.si - 1 && gy <= P.sj);
  return b;
}
template <int BND>
__device__ __forceinline__ int face_of(const Adj2D& P, int gx, int gy, int dir, int side) {
  if constexpr (BND == ADJ_STEP) return step_face(P, gx, gy, dir, side);
  const int qx = gx + (dir == 0 ? 2 * side - 1 : 0), qy = gy + (dir == 1 ? 2 * side - 1 : 0);
  if (fluid_of<BND>(P, qx, qy) || dmr::prescribed(qx, qy, P.nx, P.ny, P.x0, P.dx)) return -2;
  return qx >= P.nx ? -1 : 1 + dir;
}
// The ghost's side of such a face, whose trace is this cell's own trace Uo with component
// cn reversed (cn = -1: none): the flux's derivative on that side, d/du- = (f' + a)/2 on
// the low face (side 0), d/du+ = (f' - a)/2 on the high face, with Fw half the face's
// weight, added to this cell's trace cotangent uo.
__device__ __forceinline__ void own_trace_face(int dir, int side, int cn, double a, double gam,
                                               const double* Fw, const double* Uo, double* uo) {
  constexpr int NC = 4;
  double Ug[NC], fg[NC], gg[NC], ug[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double r = c == cn ? -1.0 : 1.0;
    Ug[c] = r * Uo[c];
    fg[c] = dir == 0 ? Fw[c] : 0.0;
    gg[c] = dir == 0 ? 0.0 : Fw[c];
    ug[c] = (side == 0 ? a : -a) * Fw[c];
  }
  euler_flux2d_vjp(Ug, gam, fg, gg, ug);
#pragma unroll
  for (int c = 0; c < NC; ++c) uo[c] += (c == cn ? -1.0 : 1.0) * ug[c];
}

// The tile kernel's sums: position (ly, lx) of tile + 1 of tile t, moment-major field f
constexpr int W1 = TX + 2, NP1 = W1 * W1;
__device__ __forceinline__ size_t sum_at(int t, int f, int ly, int lx) {
  return ((size_t)t * 12 + f) * NP1 + ly * W1 + lx;
}

// Bound by memory before: the cells' 4 x 19 stencil cotangents went through global memory to
// the gather (80 MB a launch at 256^2 written, and read by it), and one thread per cell held more
// than 256 registers.  Now a tile adds them up in LDS by the position they refer to, two
// components at a time, and stores 12 sums for each of its 18 x 18 positions; two threads work
// on a cell: the first half of the workgroup takes the interior points, the second the edges,
// and each pulls two components back to the stencil, after an exchange of the other two.
// Measured with the two kernels that read the sums, us a launch, before -> now: 256^2 NG 2 with
// shocks 21.3 -> 19.3, the hybrid cells' 24.4 -> 18.3 (its results are stored, not added), the
// gather 14.3 -> 12.4; forward step 480 x 160 NG 3 43.5 -> 39.3, 35.0 -> 27.8, 23.0 -> 26.0.  Of the 19.3 the
// staging and start take 6, the arithmetic 9, the sums 4; 180 to 230 VGPRs: one workgroup per CU, so the
// 300 tiles of the latter mesh take two rounds.
// With the limited moments loaded after the stored ones, not in their place once the flags were
// there: 19.3 -> 18.8 and 39.4 -> 36.4.
template <int NGE, int BND>
__global__ __launch_bounds__(2 * NT, 2) void adjEL2d_kernel(Adj2D P) {
  constexpr bool WALLS = BND == ADJ_WALLS;
  constexpr int NC = 4, NF = 12, W = TX + 2, NP = W * W;   // tile + one ghost layer
  constexpr int NXI = 2 * 9 * NT, NXE = 2 * 4 * NGE * NT;   // exchanged: interior, edge cotangents
  constexpr int ND = 2 * 19 * NT;                           // two components' stencil cotangents
  constexpr int NX = 2 * NF * NP > NXI + NXE ? 2 * NF * NP : NXI + NXE;
  __shared__ double s_buf[NX > ND ? NX : ND];
  double* const s_w = s_buf;             // limited stage input
  double* const s_l = s_buf + NF * NP;   // lam
  __shared__ double s_alpha[2];

  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  int bx, by;
  tile_of_block(nx, bx, by);
  const int gx0 = bx * TX - 1, gy0 = by * TY - 1;
  const size_t plane = (size_t)nx * ny;

  reduce_speeds(P.alpha, s_alpha);
  // the stored values and the flags are loaded together, the limited moments of the (few)
  // flagged cells afterwards
  auto load = [&](size_t g, bool lam, double* v, double* l) {
    const bool t = P.T && P.T[g];
#pragma unroll
    for (int f = 0; f < NF; ++f) v[f] = P.in[f * plane + g];
#pragma unroll
    for (int f = 0; f < NF; ++f) l[f] = lam ? P.lam[f * plane + g] : 0.0;
    if (t) {
#pragma unroll
      for (int f = NC; f < NF; ++f) v[f] = P.lim[(f - NC) * plane + g];
    }
  };
  // ghost positions: the mirrored cell's values with their factors, and no cotangent of
  // their own (lam = 0: a ghost is not updated)
  for (int q = tid; q < NP; q += 2 * NT) {
    const int ly = q / W, lx = q - ly * W;
    if constexpr (BND >= ADJ_STEP) {
      const int px = gx0 + lx, py = gy0 + ly;
      const step::Src r = src_of<BND>(P, px, py);
      if (r.pres) {   // prescribed: never troubled, no cotangent
#pragma unroll
        for (int f = 0; f < NF; ++f) s_w[f * NP + q] = pres_value<BND>(P, f / NC, f % NC, px, py);
#pragma unroll
        for (int f = 0; f < NF; ++f) s_l[f * NP + q] = 0.0;
        continue;
      }
      const size_t g = (size_t)r.y * nx + r.x;
      const bool ghost = r.x != px || r.y != py;   // beyond a side or inside the step
      double v[NF], l[NF];
      load(g, !ghost, v, l);
#pragma unroll
      for (int f = 0; f < NF; ++f) s_w[f * NP + q] = step_factor(r, f / NC, f % NC) * v[f];
#pragma unroll
      for (int f = 0; f < NF; ++f) s_l[f * NP + q] = l[f];
      continue;
    }
    if constexpr (BND == ADJ_PERIODIC) {
      const size_t g = (size_t)wrap(gy0 + ly, ny) * nx + wrap(gx0 + lx, nx);
      double v[NF], l[NF];
      load(g, true, v, l);
#pragma unroll
      for (int f = 0; f < NF; ++f) s_w[f * NP + q] = v[f];
#pragma unroll
      for (int f = 0; f < NF; ++f) s_l[f * NP + q] = l[f];
      continue;
    }
    const Mirror mr = mirror_of(P, gy0 + ly, gx0 + lx);
    const size_t g = (size_t)mr.g;
    const bool ghost = mr.mx || mr.my;
    double v[NF], l[NF];
    load(g, !ghost, v, l);
#pragma unroll
    for (int f = 0; f < NF; ++f) s_w[f * NP + q] = mirror_factor(P, f / NC, f % NC, mr.mx, mr.my) * v[f];
#pragma unroll
    for (int f = 0; f < NF; ++f) s_l[f * NP + q] = l[f];
  }
  __syncthreads();

  const bool first = tid < NT;   // (whole waves)
  const int ct = tid % NT, tx = ct % TX, ty = ct / TX;
  const int lx = tx + 1, ly = ty + 1;
  const int gx = bx * TX + tx, gy = by * TY + ty;
  // the step's solid cells: no right-hand side (their stencil cotangents are never read)
  bool active = gx < nx && gy < ny;
  if constexpr (BND == ADJ_STEP) active = active && !step::solid(gx, gy, P.si, P.sj);
  const size_t gi = active ? (size_t)gy * nx + gx : 0;
  const bool hyb = active && P.H && P.H[gi];
  const double idx = 1.0 / P.dx, idy = 1.0 / P.dy;
  const double* node = Gauss<NGE>::node;
  const double* wt = Gauss<NGE>::wt;
  double* const x_int = s_buf + ct;          // [2][9][NT]: components 0, 1
  double* const x_edge = s_buf + NXI + ct;   // [2][2][2 NGE][NT]: directions, components 2, 3
  // component c's cotangents, pulled back to the stencil values, into this half's space
  double* const s_d = s_buf + (first ? 0 : 19 * NT);
  auto pull_back = [&](const double* ui, const double* e0, const double* e1) {
    double d[19], fb[hw2::NFOLD];
#pragma unroll
    for (int k = 0; k < 19; ++k) d[k] = 0.0;
#pragma unroll
    for (int k = 0; k < hw2::NFOLD; ++k) fb[k] = 0.0;
    hw2::lin2d_inner_T(ui, fb);
    if (!hyb) {
      lin_faces_T<NGE>(0, e0, e0 + NGE, fb);
      lin_faces_T<NGE>(1, e1, e1 + NGE, fb);
    }
    hw2::lin2d_fold_T(fb, d);
#pragma unroll
    for (int k = 0; k < 19; ++k) s_d[k * NT + ct] = active ? d[k] : 0.0;
  };
  // the sums by position of the two components in LDS: c of the first half, c - 2 of the second
  auto add_up = [&](int c) {
    const int cy[5] = {-1, 0, 0, 0, 1}, cx[5] = {0, -1, 0, 1, 0};
    for (int it = tid; it < 2 * NP1; it += 2 * NT) {
      const int half = it >= NP1 ? 1 : 0, q = it - half * NP1, py = q / W1 - 1, px = q % W1 - 1;
      const double* d = s_buf + half * 19 * NT;
      double w[3] = {0.0, 0.0, 0.0};
      // slot k of cell j's stencil refers to the position j + offset_k
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int oy = py - (k / 3 - 1), ox = px - (k % 3 - 1);
        const bool in = (unsigned)oy < TY && (unsigned)ox < TX;   // (outside: read at 0, not added)
        const double v = d[k * NT + (in ? oy * TX + ox : 0)];
        w[0] += in ? v : 0.0;
      }
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const int oy = py - cy[k], ox = px - cx[k];
        const bool in = (unsigned)oy < TY && (unsigned)ox < TX;
        const int j = in ? oy * TX + ox : 0;
        const double v = d[(9 + k) * NT + j], z = d[(14 + k) * NT + j];
        w[1] += in ? v : 0.0;
        w[2] += in ? z : 0.0;
      }
      const int cc = half ? c - 2 : c, t = by * ((nx + TX - 1) / TX) + bx;
#pragma unroll
      for (int m = 0; m < 3; ++m) P.A[sum_at(t, m * NC + cc, q / W1, q % W1)] = w[m];
    }
  };

  // A half's cotangents of the two components it pulls back (interior values, edge values of both
  // directions), and those of the other two, which it hands over.  Both halves meet at every
  // barrier from here on, each a single statement outside the branches.
  double ui[2][9], e[2][2][2 * NGE];
  constexpr int NHAND = 18 > 8 * NGE ? 18 : 8 * NGE;
  double hand[NHAND];
  if (first) {
    // volume terms of eq. ode2: the x moment gains (1/dx) sum w f(u(G)), the y moment
    // (1/dy) sum w g(u(G)); cotangents of the interior values
    double inner[NC][9];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double in[19], fold[hw2::NFOLD];
      gather19<NC, W>(s_w, c, ly, lx, in);
      hw2::lin2d_fold(in, fold);
      hw2::lin2d_inner(fold, inner[c]);
    }
    double lv[NC], lw[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      lv[c] = S<W>(s_l, NC + c, ly, lx) * idx;
      lw[c] = S<W>(s_l, 2 * NC + c, ly, lx) * idy;
    }
#pragma unroll
    for (int p = 0; p < 9; ++p) {
      const double wq = VW[p % 3] * VW[p / 3];
      double U[NC], fb[NC], gb[NC], ub[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        U[c] = inner[c][p];
        fb[c] = wq * lv[c];
        gb[c] = wq * lw[c];
        ub[c] = 0.0;
      }
      euler_flux2d_vjp(U, P.gam, fb, gb, ub);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        hand[c * 9 + p] = ub[c];
        ui[c][p] = ub[2 + c];
      }
    }
  } else {
    // edge values of both directions and the cotangents of the four faces' fluxes
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      double v[NC][2 * NGE];
      if (!hyb) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double in[19], fold[hw2::NFOLD];
          gather19<NC, W>(s_w, c, ly, lx, in);
          hw2::lin2d_fold(in, fold);
          lin_faces<NGE>(fold, dir, v[c], v[c] + NGE);
        }
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int k = 0; k < NGE; ++k) {
            v[c][k] = P.hwv[((((size_t)(dir * 2 + 0) * NGE + k) * NC + c)) * plane + gi];
            v[c][NGE + k] = P.hwv[((((size_t)(dir * 2 + 1) * NGE + k) * NC + c)) * plane + gi];
          }
      }
      const int oy = dir, ox = 1 - dir;
      const double inv = dir == 0 ? idx : idy;
      const double a = s_alpha[dir];
      // the moment fed by (F_L + F_R)/2 and the one fed by the node-weighted difference
      const int fP = dir == 0 ? 1 : 2, fQ = 3 - fP;
#pragma unroll
      for (int k = 0; k < NGE; ++k) {
        const double wk = wt[k] * inv, nk = node[k];
        double flo[NC], fhi[NC], zero[NC], ul[NC], uh[NC], Ul[NC], Uh[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const double lU = S<W>(s_l, c, ly, lx), cP = S<W>(s_l, fP * NC + c, ly, lx),
                       cQ = S<W>(s_l, fQ * NC + c, ly, lx);
          const double mU = S<W>(s_l, c, ly - oy, lx - ox), mP = S<W>(s_l, fP * NC + c, ly - oy, lx - ox),
                       mQ = S<W>(s_l, fQ * NC + c, ly - oy, lx - ox);
          const double pU = S<W>(s_l, c, ly + oy, lx + ox), pP = S<W>(s_l, fP * NC + c, ly + oy, lx + ox),
                       pQ = S<W>(s_l, fQ * NC + c, ly + oy, lx + ox);
          // low face: this cell's left/bottom face and the neighbour's right/top face
          const double Flo = wk * ((lU - 0.5 * cP + nk * cQ) - (mU + 0.5 * mP + nk * mQ));
          // high face: this cell's right/top face and the neighbour's left/bottom face
          const double Fhi = wk * ((pU - 0.5 * pP + nk * pQ) - (lU + 0.5 * cP + nk * cQ));
          // F = (f(u-) + f(u+))/2 - a (u+ - u-)/2: this cell is u+ on the low face, u- on
          // the high face
          flo[c] = 0.5 * Flo;
          fhi[c] = 0.5 * Fhi;
          ul[c] = -0.5 * a * Flo;
          uh[c] = 0.5 * a * Fhi;
          zero[c] = 0.0;
          Ul[c] = v[c][k];
          Uh[c] = v[c][NGE + k];
        }
        if (dir == 0) {
          euler_flux2d_vjp(Ul, P.gam, flo, zero, ul);
          euler_flux2d_vjp(Uh, P.gam, fhi, zero, uh);
        } else {
          euler_flux2d_vjp(Ul, P.gam, zero, flo, ul);
          euler_flux2d_vjp(Uh, P.gam, zero, fhi, uh);
        }
        // a face on a transmissive or reflective side: the ghost's trace there is this
        // cell's own trace (the normal momentum reversed at a reflective side), so the
        // ghost's side of the flux, d/du- on the low face and d/du+ on the high face, also
        // belongs to this cell
        const int bc = dir == 0 ? P.bcx : P.bcy;
        if (WALLS && bc != BC_PERIODIC) {
          const int gd = dir == 0 ? gx : gy, nd = dir == 0 ? nx : ny;
          const int cn = bc == BC_REFLECTIVE ? 1 + dir : -1;
#pragma unroll
          for (int side = 0; side < 2; ++side) {
            if (side == 0 ? gd != 0 : gd != nd - 1) continue;
            double Ug[NC], fg[NC], gg[NC], ug[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
              const double r = c == cn ? -1.0 : 1.0;
              const double Fw = side == 0 ? flo[c] : fhi[c];   // half the face's weight
              Ug[c] = r * (side == 0 ? Ul[c] : Uh[c]);
              fg[c] = dir == 0 ? Fw : 0.0;
              gg[c] = dir == 0 ? 0.0 : Fw;
              ug[c] = (side == 0 ? a : -a) * Fw;   // d/du- = (f' + a)/2, d/du+ = (f' - a)/2
            }
            euler_flux2d_vjp(Ug, P.gam, fg, gg, ug);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
              const double r = c == cn ? -1.0 : 1.0;
              if (side == 0) ul[c] += r * ug[c];
              else uh[c] += r * ug[c];
            }
          }
        }
        // the resolver family: the face rule on faces towards a non-fluid position
        if constexpr (BND >= ADJ_STEP) {
          const int kl = face_of<BND>(P, gx, gy, dir, 0), kh = face_of<BND>(P, gx, gy, dir, 1);
          if (kl != -2) own_trace_face(dir, 0, kl, a, P.gam, flo, Ul, ul);
          if (kh != -2) own_trace_face(dir, 1, kh, a, P.gam, fhi, Uh, uh);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          e[c][dir][k] = ul[c];
          e[c][dir][NGE + k] = uh[c];
          hand[(dir * 2 + c) * 2 * NGE + k] = ul[2 + c];
          hand[(dir * 2 + c) * 2 * NGE + NGE + k] = uh[2 + c];
        }
      }
    }

    if (hyb) {
#pragma unroll
      for (int dir = 0; dir < 2; ++dir)
#pragma unroll
        for (int k = 0; k < 2 * NGE; ++k)
#pragma unroll
          for (int c = 0; c < NC; ++c)
            P.E[((size_t)(dir * 2 * NGE + k) * NC + c) * plane + gi] =
                c < 2 ? e[c & 1][dir][k] : hand[(dir * 2 + (c & 1)) * 2 * NGE + k];
    }
  }
  __syncthreads();   // the staged values are done with
  if (first) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < 9; ++p) x_int[(c * 9 + p) * NT] = hand[c * 9 + p];
  } else {
#pragma unroll
    for (int k = 0; k < 8 * NGE; ++k) x_edge[k * NT] = hand[k];
  }
  __syncthreads();
  if (first) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int dir = 0; dir < 2; ++dir)
#pragma unroll
        for (int k = 0; k < 2 * NGE; ++k) e[c][dir][k] = x_edge[((dir * 2 + c) * 2 * NGE + k) * NT];
  } else {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < 9; ++p) ui[c][p] = x_int[(c * 9 + p) * NT];
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    __syncthreads();   // what was in the space is read
    pull_back(ui[c], e[c][0], e[c][1]);
    __syncthreads();
    add_up(2 + c);
  }
}

// Reversed characteristic HWENO edge values of one hybrid cell in direction DIR (Step 5.1,
// Remark 4), four lanes per cell as in the forward pass: lane f projects onto field f with
// row f of L, reverses field f's reconstruction, and returns in ib the stencil cotangents
// of physical component f; the eigenvectors' dependence on the cell average enters through
// the average's cotangent.  s_x: 19 x 64 doubles of this wave's own, through which the four
// lanes of a cell read each other's stencil components and field cotangents (each value is
// written once and read where it is used; passed round by lane exchanges the components
// stayed in registers, 490 of them, at one wave per SIMD).
template <int NGE, int DIR, int BND>
__device__ __forceinline__ void adjEhw2d_cell(const Adj2D& P, int gi, int f, double* s_x, double* ib) {
  constexpr int NC = 4, dir = DIR;
  constexpr bool WALLS = BND == ADJ_WALLS;
  const size_t plane = (size_t)P.nx * P.ny;
  const int gy = gi / P.nx, gx = gi - gy * P.nx;
  const int cross[5] = {1, 3, 4, 5, 7};
  // component f of the limited stencil (ghost positions: the mirrored cell's values)
  double in[19];
  if constexpr (BND >= ADJ_STEP) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int px = gx + k % 3 - 1, py = gy + k / 3 - 1;
      const step::Src r = src_of<BND>(P, px, py);
      in[k] = r.pres ? pres_value<BND>(P, 0, f, px, py)
                     : step_factor(r, 0, f) * P.in[f * plane + (size_t)r.y * P.nx + r.x];
    }
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int k = cross[j];
      const int px = gx + k % 3 - 1, py = gy + k / 3 - 1;
      const step::Src r = src_of<BND>(P, px, py);
      if (r.pres) {
        in[9 + j] = pres_value<BND>(P, 1, f, px, py);
        in[14 + j] = pres_value<BND>(P, 2, f, px, py);
        continue;
      }
      const size_t g = (size_t)r.y * P.nx + r.x;
      const bool t = P.T[g] != 0;
      in[9 + j] = step_factor(r, 1, f) * (t ? P.lim[f * plane + g] : P.in[(NC + f) * plane + g]);
      in[14 + j] = step_factor(r, 2, f) * (t ? P.lim[(NC + f) * plane + g] : P.in[(2 * NC + f) * plane + g]);
    }
  } else if constexpr (BND == ADJ_PERIODIC) {
    int gb[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) gb[k] = wrap(gy + k / 3 - 1, P.ny) * P.nx + wrap(gx + k % 3 - 1, P.nx);
#pragma unroll
    for (int k = 0; k < 9; ++k) in[k] = P.in[f * plane + gb[k]];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int g = gb[cross[j]];
      const bool t = P.T[g] != 0;
      in[9 + j] = t ? P.lim[f * plane + g] : P.in[(NC + f) * plane + g];
      in[14 + j] = t ? P.lim[(NC + f) * plane + g] : P.in[(2 * NC + f) * plane + g];
    }
  } else {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const Mirror mr = mirror_of(P, gy + k / 3 - 1, gx + k % 3 - 1);
      in[k] = mirror_factor(P, 0, f, mr.mx, mr.my) * P.in[f * plane + mr.g];
    }
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int k = cross[j];
      const Mirror mr = mirror_of(P, gy + k / 3 - 1, gx + k % 3 - 1);
      const int g = mr.g;
      const bool t = P.T[g] != 0;
      in[9 + j] = mirror_factor(P, 1, f, mr.mx, mr.my) * (t ? P.lim[f * plane + g] : P.in[(NC + f) * plane + g]);
      in[14 + j] = mirror_factor(P, 2, f, mr.mx, mr.my) *
                   (t ? P.lim[(NC + f) * plane + g] : P.in[(2 * NC + f) * plane + g]);
    }
  }
  const int lane = threadIdx.x & 63, q0 = lane & ~3;   // the cell's first lane
  auto in_order = [] {   // the wave's LDS operations before this point come before those after
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
#pragma unroll
  for (int k = 0; k < 19; ++k) s_x[k * 64 + lane] = in[k];
  in_order();
  double U[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) U[c] = s_x[4 * 64 + q0 + c];   // the cell average
  double Lr[4], Rc[4], x[4];
  euler_eig2d_field(U, P.gam, dir, f, Lr, Rc);   // row f of L, column f of R
  double w19[19];
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) s = fma(Lr[c], s_x[k * 64 + q0 + c], s);
    w19[k] = s;
  }
  double beta[5], om[5], wv[2 * NGE];
  double fold[hw2::NFOLD];
  hw2::lin2d_fold(w19, fold);
  hweno2d_weights<NGE>(w19, fold, P.w, beta, om);
  hweno2d_combine<NGE>(w19, fold, P.w, dir, om, wv);
  // v_c = sum_f R[c][f] wv_f: the field's cotangent and column f of R-bar
  double wvb[2 * NGE], Rb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 2 * NGE; ++k) {
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = P.E[((size_t)(dir * 2 * NGE + k) * NC + c) * plane + gi];
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      s = fma(Rc[c], x[c], s);
      Rb[c] = fma(x[c], wv[k], Rb[c]);
    }
    wvb[k] = s;
  }
  double w19b[19];
#pragma unroll
  for (int k = 0; k < 19; ++k) w19b[k] = 0.0;
  hweno2d_field_adj<NGE>(w19, fold, P.w, dir, beta, om, wvb, w19b);
  // w_f = sum_c L[f][c] in_c: row f of L-bar, and component f's cotangent through
  // column f of L (lane g holds row g)
  double Lb[4] = {0.0, 0.0, 0.0, 0.0}, Lc[4];
  int q1 = q0;   // opaque: the stencil is read again, not kept
  asm volatile("" : "+v"(q1));
#pragma unroll
  for (int k = 0; k < 19; ++k) {
#pragma unroll
    for (int c = 0; c < 4; ++c) Lb[c] = fma(w19b[k], s_x[k * 64 + q1 + c], Lb[c]);
  }
  in_order();   // every lane has read the stencil: the space takes L's rows, then w19b
#pragma unroll
  for (int c = 0; c < 4; ++c) s_x[c * 64 + lane] = Lr[c];
  in_order();
#pragma unroll
  for (int g = 0; g < 4; ++g) Lc[g] = s_x[f * 64 + q0 + g];
  in_order();
#pragma unroll
  for (int k = 0; k < 19; ++k) s_x[k * 64 + lane] = w19b[k];
  in_order();
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    double s = 0.0;
#pragma unroll
    for (int g = 0; g < 4; ++g) s = fma(Lc[g], s_x[k * 64 + q0 + g], s);
    ib[k] = s;
  }
  // the eigenvectors' dependence on the average: summed over the four fields, lane f
  // keeps the derivative along component f
  double ev[4] = {0.0, 0.0, 0.0, 0.0};
  euler_eig2d_field_vjp(U, P.gam, dir, f, Lb, Rb, ev);
  in_order();
#pragma unroll
  for (int c = 0; c < 4; ++c) s_x[c * 64 + lane] = ev[c];
  in_order();
  double es = 0.0;
#pragma unroll
  for (int g = 0; g < 4; ++g) es += s_x[f * 64 + q0 + g];
  ib[4] += es;
  in_order();
}

// The hybrid list's reversed HWENO reconstruction: the waves of a workgroup form pairs, the
// two waves of a pair take the same 16 cells, one the x direction, the other the y
// direction, and the y wave hands its shares to the x wave through LDS, which stores their
// sum.  The two directions thus run side by side.
// At most 256 VGPRs (two waves per SIMD; 8 to 14 values at NG 2 and 32 to 39 at NG 3 are kept in
// scratch for it, 36 to 160 B a lane), so that no value is kept in accumulation registers:
// forms of this kernel that used them (up to 506 registers) returned stencil cotangents off by
// 1e-9 on some inputs, and exact ones with the registers limited and nothing else changed.
template <int NGE, int BND>
__global__ __launch_bounds__(NT, 2) void adjEhw2d_kernel(Adj2D P) {
  constexpr int NC = 4, CPW = 64 / NC, NPAIR = NT / 128;
  __shared__ double s_x[NT / 64][19 * 64];
  const int ncell = P.lens ? (int)P.lens[3] : P.counts[1];
  if (ncell == 0) return;
  const size_t plane = (size_t)P.nx * P.ny;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, pr = wv >> 1, dir = wv & 1;
  const int f = lane % NC;
  // the loop's bounds are the workgroup's, so every wave meets both barriers
  for (long long base = (long long)blockIdx.x * NPAIR * CPW; base < ncell;
       base += (long long)gridDim.x * NPAIR * CPW) {
    const long long cell = base + pr * CPW + lane / NC;
    const bool on = cell < ncell;   // whole groups of four lanes
    double ib[19];
    int gi = 0;
    if (on) {
      gi = P.hlist[cell];
      if (dir == 0) {
        adjEhw2d_cell<NGE, 0, BND>(P, gi, f, s_x[wv], ib);
      } else {
        adjEhw2d_cell<NGE, 1, BND>(P, gi, f, s_x[wv], ib);
#pragma unroll
        for (int k = 0; k < 19; ++k) s_x[wv][k * 64 + lane] = ib[k];
      }
    }
    __syncthreads();
    if (on && dir == 0) {
#pragma unroll
      for (int k = 0; k < 19; ++k) P.D[(size_t)(f * 19 + k) * plane + gi] = ib[k] + s_x[wv + 1][k * 64 + lane];
    }
    __syncthreads();
  }
}

// The tiles whose sums hold position q in [-1, n] of an axis of n cells, and its place in them
// (b < 0: none): the tile it lies in or beside, the one it is the ring above of, the one it is
// the ring below of (around a periodic axis too)
struct AxisTiles {
  int b[3], l[3];
};
__device__ __forceinline__ AxisTiles axis_tiles(int q, int n, bool periodic) {
  const int nb = (n + TX - 1) / TX, b0 = q < 0 ? 0 : min(q / TX, nb - 1), r = q - b0 * TX;
  AxisTiles a{{b0, -1, -1}, {r + 1, TX + 1, 0}};
  if (r == 0 && b0 > 0) a.b[1] = b0 - 1;
  if (r == TX - 1 && b0 + 1 < nb) a.b[2] = b0 + 1;
  if (periodic && q == 0) {
    a.b[1] = nb - 1;
    a.l[1] = n - (nb - 1) * TX + 1;
  }
  if (periodic && q == n - 1) a.b[2] = 0;
  return a;
}

// Gather of the stencil cotangents and the stage coefficients, one tile of cells per workgroup:
// the tile kernel's sums of every tile that holds the cell's position, the hybrid
// cells' stencil cotangents, and both at the ghosts and solid positions that take the
// cell's values.  Four threads per cell, one per component: bound by the latency of
// dependent loads (masks, then slots; more than one boundary position in a row beside the
// step), which one thread per cell did not hide (19.0 us against 12.4 at 256^2, 42 against 26 on
// the forward step at 480 x 160).
template <int BND>
__global__ __launch_bounds__(NT) void adjEG2d_kernel(Adj2D P) {
  constexpr int NC = 4;
  constexpr bool WALLS = BND == ADJ_WALLS;
  const int nx = P.nx, ny = P.ny, ntx = (nx + TX - 1) / TX;
  const size_t plane = (size_t)nx * ny;
  // wave c of a workgroup: component c of 64 cells, four rows of a tile
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int N = gridDim.x, xcd = blockIdx.x % NXCD, rem = N % NXCD;   // as tile_of_block
  const int q4 = xcd * (N / NXCD) + min(xcd, rem) + blockIdx.x / NXCD, tile = q4 >> 2;
  const int by = tile / ntx, bx = tile - by * ntx;
  const int tx = lane % TX, ty = (q4 & 3) * 4 + lane / TX;
  const int gx = bx * TX + tx, gy = by * TY + ty;
  if (gx >= nx || gy >= ny) return;
  const size_t i = (size_t)gy * nx + gx;
  // a direction that wraps around (the resolver family's do not)
  const bool px = BND < ADJ_STEP && !(WALLS && P.bcx != BC_PERIODIC);
  const bool py = BND < ADJ_STEP && !(WALLS && P.bcy != BC_PERIODIC);
  double Wb[3], l[3], ac[3];
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const size_t g = (size_t)(m * NC + c) * plane + i;
    Wb[m] = P.A[sum_at(tile, m * NC + c, ty + 1, tx + 1)];
    l[m] = P.lam[g];
    ac[m] = P.ca != 0.0 || P.acc_mode == 2 ? P.acc_in[g] : 0.0;
  }
  // position q's sums in the tiles (all, or all but the cell's own) that hold it
  auto add_sums = [&](int qx, int qy, bool own, auto factor) {
    const AxisTiles ax = axis_tiles(qx, nx, px), ay = axis_tiles(qy, ny, py);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (ay.b[a] < 0 || ax.b[b] < 0 || (!own && a == 0 && b == 0)) continue;
        const int t = ay.b[a] * ntx + ax.b[b];
#pragma unroll
        for (int m = 0; m < 3; ++m) Wb[m] += factor(m) * P.A[sum_at(t, m * NC + c, ay.l[a], ax.l[b])];
      }
  };
  const int cross[5] = {1, 3, 4, 5, 7};
  // position q's slots of the hybrid cells around it
  auto add_hybrid = [&](int qx, int qy, auto factor) {
    if (!P.H) return;
    size_t j[9];
    bool h[9], any = false;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      int oy = qy - (k / 3 - 1), ox = qx - (k % 3 - 1);
      if (px) ox = wrap(ox, nx);
      if (py) oy = wrap(oy, ny);
      const bool in = ox >= 0 && ox < nx && oy >= 0 && oy < ny;
      j[k] = in ? (size_t)oy * nx + ox : i;
      h[k] = in && P.H[j[k]] != 0;
      if constexpr (BND == ADJ_STEP) h[k] = h[k] && !step::solid(ox, oy, P.si, P.sj);
      any = any || h[k];
    }
    if (!any) return;
    // every load issued (a slot that is no hybrid cell's is read and not added)
    const double* D = P.D + (size_t)c * 19 * plane;
    double u[9], v[5], w[5];
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = D[k * plane + j[k]];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      v[k] = D[(9 + k) * plane + j[cross[k]]];
      w[k] = D[(14 + k) * plane + j[cross[k]]];
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) Wb[0] += h[k] ? factor(0) * u[k] : 0.0;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      Wb[1] += h[cross[k]] ? factor(1) * v[k] : 0.0;
      Wb[2] += h[cross[k]] ? factor(2) * w[k] : 0.0;
    }
  };
  bool fluid = true;
  if constexpr (BND >= ADJ_STEP) fluid = fluid_of<BND>(P, gx, gy);
  if (!fluid) {   // solid: what refers to its position belongs to its source
#pragma unroll
    for (int m = 0; m < 3; ++m) Wb[m] = 0.0;
  } else {
    const bool rim = tx == 0 || tx == TX - 1 || ty == 0 || ty == TY - 1 || gx == nx - 1 || gy == ny - 1;
    if (rim) add_sums(gx, gy, false, [](int) { return 1.0; });
    add_hybrid(gx, gy, [](int) { return 1.0; });
    if constexpr (BND >= ADJ_STEP) {
      // the non-fluid positions whose source the cell is
      if (beside_boundary<BND>(P, gx, gy))
        for (int ey = -1; ey <= 1; ++ey)
          for (int ex = -2; ex <= 2; ++ex) {
            const int qx = gx + ex, qy = gy + ey;
            if ((ex == 0 && ey == 0) || qx < -1 || qx > nx || qy < -1 || qy > ny || fluid_of<BND>(P, qx, qy)) continue;
            const step::Src r = src_of<BND>(P, qx, qy);
            if (r.pres || r.x != gx || r.y != gy) continue;
            auto factor = [&](int m) { return step_factor(r, m, c); };
            add_sums(qx, qy, true, factor);
            add_hybrid(qx, qy, factor);
          }
    }
    if constexpr (WALLS) {
      // the ghosts that mirror the cell, beside a transmissive or reflective side (at most
      // one per side, and the corner between two)
      const int xs[3] = {gx, !px && gx == 0 ? -1 : INT_MIN, !px && gx == nx - 1 ? nx : INT_MIN};
      const int ys[3] = {gy, !py && gy == 0 ? -1 : INT_MIN, !py && gy == ny - 1 ? ny : INT_MIN};
      const bool edge = xs[1] != INT_MIN || xs[2] != INT_MIN || ys[1] != INT_MIN || ys[2] != INT_MIN;
      for (int a = 0; a < 3 && edge; ++a) {
        if (ys[a] == INT_MIN) continue;
        for (int b = 0; b < 3; ++b) {
          if (xs[b] == INT_MIN || (a == 0 && b == 0)) continue;
          const bool mx = b > 0, my = a > 0;
          auto factor = [&](int m) { return mirror_factor(P, m, c, mx, my); };
          add_sums(xs[b], ys[a], true, factor);
          add_hybrid(xs[b], ys[a], factor);
        }
      }
    }
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const size_t g = (size_t)(m * NC + c) * plane + i;
    double o = P.cg * l[m] + P.cl * Wb[m];
    if (P.ca != 0.0) o = fma(P.ca, ac[m], o);
    P.gw[g] = o;
    if (P.acc_mode == 1) P.acc_out[g] = P.kl * l[m];
    else if (P.acc_mode == 2) P.acc_out[g] = fma(P.kl, l[m], ac[m]);
  }
}

// The reversed characteristic limiter (Step 4, Remark 4) of one flagged cell in direction
// DIR, four lanes per cell: lane f reverses the limiter of characteristic field f and
// stores the cotangents of physical component f of the five stencil values of the
// direction (u_{-1}, u_0, u_{+1}, v_{-1}, v_{+1}), with the eigenvectors' dependence on
// the average added to the centre slot.
template <int DIR, int BND>
__device__ __forceinline__ void adjEC2d_cell(const Adj2D& P, size_t i, int f) {
  constexpr int NC = 4, dir = DIR, mf = 1 + DIR;
  const int nx = P.nx, ny = P.ny;
  const size_t plane = (size_t)nx * ny;
  const int gy = (int)(i / nx), gx = (int)(i - (size_t)gy * nx);
  // the two neighbours along the direction (ghosts: the mirrored cell's values; beyond the
  // forward step's inflow side, the free stream with first moments zero)
  double xm, xp, wm_, wp_;
  if constexpr (BND >= ADJ_STEP) {
    const int xmx = gx - (dir == 0), xmy = gy - (dir == 1), xpx = gx + (dir == 0), xpy = gy + (dir == 1);
    const step::Src rm = src_of<BND>(P, xmx, xmy);
    const step::Src rp = src_of<BND>(P, xpx, xpy);
    const size_t jm = (size_t)rm.y * nx + rm.x, jp = (size_t)rp.y * nx + rp.x;
    xm = rm.pres ? pres_value<BND>(P, 0, f, xmx, xmy) : step_factor(rm, 0, f) * P.in[f * plane + jm];
    xp = rp.pres ? pres_value<BND>(P, 0, f, xpx, xpy) : step_factor(rp, 0, f) * P.in[f * plane + jp];
    wm_ = rm.pres ? pres_value<BND>(P, mf, f, xmx, xmy) : step_factor(rm, mf, f) * P.in[(mf * NC + f) * plane + jm];
    wp_ = rp.pres ? pres_value<BND>(P, mf, f, xpx, xpy) : step_factor(rp, mf, f) * P.in[(mf * NC + f) * plane + jp];
  } else {
    const Mirror mm = dir == 0 ? mirror_of(P, gy, gx - 1) : mirror_of(P, gy - 1, gx);
    const Mirror mp = dir == 0 ? mirror_of(P, gy, gx + 1) : mirror_of(P, gy + 1, gx);
    xm = mirror_factor(P, 0, f, mm.mx, mm.my) * P.in[f * plane + mm.g];
    xp = mirror_factor(P, 0, f, mp.mx, mp.my) * P.in[f * plane + mp.g];
    wm_ = mirror_factor(P, mf, f, mm.mx, mm.my) * P.in[(mf * NC + f) * plane + mm.g];
    wp_ = mirror_factor(P, mf, f, mp.mx, mp.my) * P.in[(mf * NC + f) * plane + mp.g];
  }
  // Jacobi: every input is the unlimited stage input; G is the cotangent of the limited
  // moment of this direction
  double Ui[4], um[4], up[4], vm[4], vp[4], G[4];
  quad_gather_p(P.in[f * plane + i], Ui);
  quad_gather_p(xm, um);
  quad_gather_p(xp, up);
  quad_gather_p(wm_, vm);
  quad_gather_p(wp_, vp);
  quad_gather_p(P.gw[(mf * NC + f) * plane + i], G);
  double Lr[4], Rc[4];
  euler_eig2d_field(Ui, P.gam, dir, f, Lr, Rc);
  double cm = 0.0, c0 = 0.0, cp = 0.0, wm = 0.0, wp = 0.0, wb = 0.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    cm = fma(Lr[c], um[c], cm);
    c0 = fma(Lr[c], Ui[c], c0);
    cp = fma(Lr[c], up[c], cp);
    wm = fma(Lr[c], vm[c], wm);
    wp = fma(Lr[c], vp[c], wp);
    wb = fma(Rc[c], G[c], wb);
  }
  const double vc = limit_moment(cm, c0, cp, wm, wp, P.w.lim, P.w.eps);
  double gbv[5];
  limit_moment_adj(cm, c0, cp, wm, wp, P.w.lim, P.w.eps, wb, gbv);
  double Lb[4], Rb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Lb[c] = gbv[0] * um[c] + gbv[1] * Ui[c] + gbv[2] * up[c] + gbv[3] * vm[c] + gbv[4] * vp[c];
    Rb[c] = G[c] * vc;
  }
  double ev[4] = {0.0, 0.0, 0.0, 0.0};
  euler_eig2d_field_vjp(Ui, P.gam, dir, f, Lb, Rb, ev);
  // component f: sums over the four fields (lane g of the quad holds field g)
  double Lc[4];
  {
    double q0[4], q1[4], q2[4], q3[4];
    quad_gather_p(Lr[0], q0);
    quad_gather_p(Lr[1], q1);
    quad_gather_p(Lr[2], q2);
    quad_gather_p(Lr[3], q3);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const double col[4] = {q0[g], q1[g], q2[g], q3[g]};
      Lc[g] = sel4(col, f);
    }
  }
  double e0[4], e1[4], e2[4], e3[4];
  quad_gather_p(ev[0], e0);
  quad_gather_p(ev[1], e1);
  quad_gather_p(ev[2], e2);
  quad_gather_p(ev[3], e3);
  const double es[4] = {e0[0] + e0[1] + e0[2] + e0[3], e1[0] + e1[1] + e1[2] + e1[3],
                        e2[0] + e2[1] + e2[2] + e2[3], e3[0] + e3[1] + e3[2] + e3[3]};
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    double x[4];
    quad_gather_p(gbv[q], x);
    double s = 0.0;
#pragma unroll
    for (int g = 0; g < 4; ++g) s = fma(Lc[g], x[g], s);
    if (q == 1) s += sel4(es, f);
    P.C[((size_t)(dir * 5 + q) * NC + f) * plane + i] = s;
  }
}

// The reversed limiter over the forward's flagged list: waves alternate between the x and
// the y direction of the same 16 cells.  BND: ADJ_STEP or ADJ_DMR for the resolver family,
// else the mirrors of mirror_of (which reduce to wrap-around on periodic sides).
template <int BND>
__global__ __launch_bounds__(NT) void adjEC2d_kernel(Adj2D P) {
  constexpr int NC = 4, CPW = 64 / NC;
  const int ncnt = P.lens ? (int)P.lens[0] : P.counts[0];
  const long long ngroup = ((long long)ncnt + CPW - 1) / CPW;   // waves per direction
  const int lane = threadIdx.x & 63, f = lane % NC;
  for (long long wq = ((long long)blockIdx.x * NT + threadIdx.x) >> 6; wq < 2 * ngroup;
       wq += ((long long)gridDim.x * NT) >> 6) {
    const long long cell = (wq >> 1) * CPW + lane / NC;
    if (cell >= ncnt) continue;   // whole groups of four lanes
    const size_t i = (size_t)P.flist[cell];
    if (wq & 1) adjEC2d_cell<1, BND>(P, i, f);
    else adjEC2d_cell<0, BND>(P, i, f);
  }
}

// The transposed limiter Jacobian: a flagged cell's limited moments replace its stored
// ones (their cotangent moves to the limiter's inputs); the limiter of a flagged cell
// reads the averages of the cell and its two neighbours along the direction and the
// neighbours' moments (slots um, u0, up, vm, vp).  BND as for adjEC2d_kernel.  Bound by the
// latency of flags, then slots: four threads per cell, one per component (8.2 -> 7.4 us
// at 256^2 with shocks, 14.5 -> 11.1 on the forward step at 480 x 160).
template <int BND>
__global__ __launch_bounds__(NT) void adjElim2d_kernel(Adj2D P) {
  constexpr int NC = 4;
  const int nx = P.nx, ny = P.ny;
  const size_t plane = (size_t)nx * ny;
  // wave c of a workgroup: component c of 64 cells
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t i = (size_t)blockIdx.x * 64 + (threadIdx.x & 63);
  if (blockIdx.x == 0 && threadIdx.x == 0 && P.counts) {   // the list passes are done: empty the lists for the next stage
    P.counts[0] = 0;
    P.counts[1] = 0;
  }
  if (i >= plane) return;
  const int gy = (int)(i / nx), gx = (int)(i - (size_t)gy * nx);
  const bool ti = P.T && P.T[i];
  double ou = P.gw[c * plane + i];
  double ov = ti ? 0.0 : P.gw[(NC + c) * plane + i];
  double ow = ti ? 0.0 : P.gw[(2 * NC + c) * plane + i];
  auto C = [&](int dir, int s, size_t j) { return P.C[((size_t)(dir * 5 + s) * NC + c) * plane + j]; };
  // the forward step: the limiter of a flagged fluid cell j reads the positions j -+ e_dir;
  // this fluid cell gathers what refers to itself and to the non-fluid positions whose
  // source it is (solid cells are never flagged and are nobody's source)
  if (BND >= ADJ_STEP && P.T && !beside_boundary<BND>(P, gx, gy)) {
    // the plain gather: the cell's own slots and its four neighbours' (right / top see it
    // as (um, vm), left / bottom as (up, vp))
    if (ti) ou += C(0, 1, i) + C(1, 1, i);
    const size_t xr = i + 1, xl = i - 1, yt = i + nx, yb = i - nx;
    if (P.T[xr]) {
      ou += C(0, 0, xr);
      ov += C(0, 3, xr);
    }
    if (P.T[xl]) {
      ou += C(0, 2, xl);
      ov += C(0, 4, xl);
    }
    if (P.T[yt]) {
      ou += C(1, 0, yt);
      ow += C(1, 3, yt);
    }
    if (P.T[yb]) {
      ou += C(1, 2, yb);
      ow += C(1, 4, yb);
    }
  } else if (BND >= ADJ_STEP && P.T && fluid_of<BND>(P, gx, gy)) {
    if (ti) ou += C(0, 1, i) + C(1, 1, i);
    for (int ey = -1; ey <= 1; ++ey)
      for (int ex = -2; ex <= 2; ++ex) {
        const int qx = gx + ex, qy = gy + ey;
        step::Src r{gx, gy, 1.0, 1.0, 1.0, 1.0, false};
        if (ex != 0 || ey != 0) {
          if (fluid_of<BND>(P, qx, qy)) continue;
          r = src_of<BND>(P, qx, qy);
          if (r.pres || r.x != gx || r.y != gy) continue;
        }
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
          const int ux = dir == 0, uy = dir == 1;
          // the owner below q sees q as its (up, vp); the owner above, as its (um, vm)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const int ox = s == 0 ? qx - ux : qx + ux, oy = s == 0 ? qy - uy : qy + uy;
            if (!fluid_of<BND>(P, ox, oy)) continue;
            const size_t j = (size_t)oy * nx + ox;
            if (!P.T[j]) continue;
            const int su = s == 0 ? 2 : 0, sv = s == 0 ? 4 : 3;
            ou += step_factor(r, 0, c) * C(dir, su, j);
            const double v = step_factor(r, 1 + dir, c) * C(dir, sv, j);
            if (dir == 0) ov += v;
            else ow += v;
          }
        }
      }
  }
  if (BND < ADJ_STEP && P.T) {
    if (ti) ou += C(0, 1, i) + C(1, 1, i);
    const bool wx = P.bcx != BC_PERIODIC, wy = P.bcy != BC_PERIODIC;
    const size_t xr = (size_t)gy * nx + wrap(gx + 1, nx), xl = (size_t)gy * nx + wrap(gx - 1, nx);
    const size_t yt = (size_t)wrap(gy + 1, ny) * nx + gx, yb = (size_t)wrap(gy - 1, ny) * nx + gx;
    // the right / top neighbour sees this cell as (um, vm), the left / bottom one as (up, vp)
    if (!(wx && gx == nx - 1) && P.T[xr]) {
      ou += C(0, 0, xr);
      ov += C(0, 3, xr);
    }
    if (!(wx && gx == 0) && P.T[xl]) {
      ou += C(0, 2, xl);
      ov += C(0, 4, xl);
    }
    if (!(wy && gy == ny - 1) && P.T[yt]) {
      ou += C(1, 0, yt);
      ow += C(1, 3, yt);
    }
    if (!(wy && gy == 0) && P.T[yb]) {
      ou += C(1, 2, yb);
      ow += C(1, 4, yb);
    }
    // beside a transmissive or reflective side, this cell's own limiter reads the ghost
    // that mirrors it as its neighbour across that side
    if (ti) {
      if (wx && gx == 0) {
        ou += mirror_factor(P, 0, c, true, false) * C(0, 0, i);
        ov += mirror_factor(P, 1, c, true, false) * C(0, 3, i);
      }
      if (wx && gx == nx - 1) {
        ou += mirror_factor(P, 0, c, true, false) * C(0, 2, i);
        ov += mirror_factor(P, 1, c, true, false) * C(0, 4, i);
      }
      if (wy && gy == 0) {
        ou += mirror_factor(P, 0, c, false, true) * C(1, 0, i);
        ow += mirror_factor(P, 2, c, false, true) * C(1, 3, i);
      }
      if (wy && gy == ny - 1) {
        ou += mirror_factor(P, 0, c, false, true) * C(1, 2, i);
        ow += mirror_factor(P, 2, c, false, true) * C(1, 4, i);
      }
    }
  }
  P.out[c * plane + i] = ou;
  P.out[(NC + c) * plane + i] = ov;
  P.out[(2 * NC + c) * plane + i] = ow;
}

}  // namespace hw

extern "C" hipError_t hw_launch_adj2d(int eq, int ng, const hw::Adj2D* P, hipStream_t s) {
  dim3 grid(((P->nx + hw::TX - 1) / hw::TX) * ((P->ny + hw::TY - 1) / hw::TY));
  dim3 block(hw::AT);
#define HW_LA(E, G) hipLaunchKernelGGL((hw::adjL2d_kernel<E, G>), grid, block, 0, s, *P)
  if (eq == hw::EQ_BURGERS && ng == 2) HW_LA(hw::EQ_BURGERS, 2);
  else if (eq == hw::EQ_BURGERS && ng == 3) HW_LA(hw::EQ_BURGERS, 3);
  else if (eq == hw::EQ_ADV && ng == 2) HW_LA(hw::EQ_ADV, 2);
  else if (eq == hw::EQ_ADV && ng == 3) HW_LA(hw::EQ_ADV, 3);
  else return hipErrorInvalidValue;
#undef HW_LA
  return hipGetLastError();
}

extern "C" hipError_t hw_launch_adjlim2d(int eq, const hw::Adj2D* P, hipStream_t s) {
  dim3 grid(((P->nx + hw::TX - 1) / hw::TX) * ((P->ny + hw::TY - 1) / hw::TY));
  dim3 block(hw::AT);
  if (eq == hw::EQ_BURGERS)
    hipLaunchKernelGGL(hw::adjLim2d_kernel<hw::EQ_BURGERS>, grid, block, 0, s, *P);
  else if (eq == hw::EQ_ADV)
    hipLaunchKernelGGL(hw::adjLim2d_kernel<hw::EQ_ADV>, grid, block, 0, s, *P);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

namespace {
// the reverse launches of one Euler stage for edge rule NGE and boundary form BND
template <int NGE, int BND>
void launch_adjE(const hw::Adj2D* P, dim3 grid, dim3 cells, hipStream_t s) {
  // the limiter kernels share one instance between periodic sides and mirrors
  constexpr int LB = BND >= hw::ADJ_STEP ? BND : hw::ADJ_WALLS;
  const dim3 block(hw::NT);
  hipLaunchKernelGGL((hw::adjEL2d_kernel<NGE, BND>), grid, dim3(2 * hw::NT), 0, s, *P);
  if (P->counts) hipLaunchKernelGGL((hw::adjEhw2d_kernel<NGE, BND>), dim3(1024), block, 0, s, *P);
  hipLaunchKernelGGL(hw::adjEG2d_kernel<BND>, dim3(4 * grid.x), block, 0, s, *P);
  if (P->T) hipLaunchKernelGGL(hw::adjEC2d_kernel<LB>, dim3(1024), block, 0, s, *P);
  hipLaunchKernelGGL(hw::adjElim2d_kernel<LB>, cells, block, 0, s, *P);   // 64 cells a workgroup
}
}  // namespace

extern "C" hipError_t hw_launch_adj2d_euler(int ng, const hw::Adj2D* P, hipStream_t s) {
  const size_t plane = (size_t)P->nx * P->ny;
  dim3 grid(((P->nx + hw::TX - 1) / hw::TX) * ((P->ny + hw::TY - 1) / hw::TY));
  dim3 cells((unsigned)((plane + 63) / 64));
  const int bnd = P->bcx == hw::BC_STEP  ? hw::ADJ_STEP
                  : P->bcx == hw::BC_DMR ? hw::ADJ_DMR
                  : (P->bcx != hw::BC_PERIODIC || P->bcy != hw::BC_PERIODIC) ? hw::ADJ_WALLS
                                                                             : hw::ADJ_PERIODIC;
  if (bnd == hw::ADJ_DMR && !P->dtab) return hipErrorInvalidValue;
  if (ng == 2 && bnd == hw::ADJ_PERIODIC) launch_adjE<2, hw::ADJ_PERIODIC>(P, grid, cells, s);
  else if (ng == 2 && bnd == hw::ADJ_WALLS) launch_adjE<2, hw::ADJ_WALLS>(P, grid, cells, s);
  else if (ng == 2 && bnd == hw::ADJ_STEP) launch_adjE<2, hw::ADJ_STEP>(P, grid, cells, s);
  else if (ng == 2) launch_adjE<2, hw::ADJ_DMR>(P, grid, cells, s);
  // the periodic NG = 3 case takes the mirror instances (their mirrors reduce to wrap-around
  // on periodic sides): the plain-wrap tile kernel needs more registers than a wave has there
  else if (ng == 3 && bnd == hw::ADJ_PERIODIC) launch_adjE<3, hw::ADJ_WALLS>(P, grid, cells, s);
  else if (ng == 3 && bnd == hw::ADJ_WALLS) launch_adjE<3, hw::ADJ_WALLS>(P, grid, cells, s);
  else if (ng == 3 && bnd == hw::ADJ_STEP) launch_adjE<3, hw::ADJ_STEP>(P, grid, cells, s);
  else if (ng == 3) launch_adjE<3, hw::ADJ_DMR>(P, grid, cells, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
