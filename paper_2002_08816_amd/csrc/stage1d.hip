// Fused one-dimensional stage kernel of the hybrid Hermite WENO scheme
// (Zhao & Qiu, arXiv 2002.08816, Section 2.1, Steps 1-3 and eq. odeH).
//
// A workgroup (T threads; T = 64, 128, 256 or 512) processes one tile of one instance, one
// position per thread: T - 6 cells and three ghost layers on either side are staged in LDS,
// then KXRCF flags
// (tile+2), the Step-1 limiter on flagged cells (Jacobi, characteristic-wise for Euler),
// the hybrid mask (tile+1), interface values (Step 2.2 linear or Step 2.1 HWENO) and
// interior Gauss-Lobatto values (Step 2.3), each side's share of the Lax-Friedrichs fluxes
// exchanged through LDS, the four-point Gauss-Lobatto volume term, and the TVD-RK3 stage
// combination.
//
// The same tile routine serves a single solver (one instance) and the batched form: many
// independent instances of different sizes, concatenated field by field, advanced by a
// persistent grid that walks an (instance, tile) work list.  Each instance has its own
// Lax-Friedrichs speed, time step and time.
#include "hw_mesh1d.h"

namespace hw {


constexpr int H1 = 3;   // ghost layers: flags on tile+2 read one more cell

// block-wide max over NW waves; red must hold NW doubles
template <int NW>
__device__ __forceinline__ double block_max(double v, double* red) {
  v = wave_max(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  double m = red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) m = fmax(m, red[i]);
  return m;
}

// 1D Euler characteristic fields at a cell-average state, taken one field at a time: row f
// of L = R^{-1} and column f of R (R columns (1, u-c, H-uc), (1, u, u^2/2), (1, u+c, H+uc)).
// Only the derived quantities of the state stay live between fields.
struct Char1 {
  double u, c, H, b1, b2, ic;
};

// a b + c in one rounding, never merged with what uses it.  The characteristic fields, the flux
// shares and the stage update are evaluated through it and otherwise without contraction: the tile
// kernels and the whole-step kernel share out a cell's work differently, and the compiler would contract
// (and, where a factor is the constant 1, regroup) each in its own way; so they give the same values to
// the bit.
__device__ __forceinline__ double mad(double a, double b, double c) {
#pragma clang fp contract(off)
  return __builtin_fma(a, b, c);
}

// a / b from r, 1 / b up to a few ulps: the product corrected by its exact remainder, the rounded
// quotient but for rare last bits
__device__ __forceinline__ double quot(double a, double b, double r) {
#pragma clang fp contract(off)
  const double q = a * r;
  return mad(mad(-b, q, a), r, q);
}

__device__ __forceinline__ Char1 char1d(double rho, double m, double E, double gam) {
#pragma clang fp contract(off)
  Char1 k;
  const double ir = rcp_nr(rho), g1 = gam - 1.0;
  k.u = quot(m, rho, ir);
  const double e = mad(-(0.5 * rho * k.u), k.u, E), p = g1 * e;
  k.c = sqrt(quot(gam * p, rho, ir));
  k.H = quot(mad(g1, e, E), rho, ir);
  k.ic = rcp_nr(k.c);
  k.b1 = quot(g1, k.c * k.c, k.ic * k.ic);
  k.b2 = 0.5 * k.b1 * k.u * k.u;
  return k;
}

__device__ __forceinline__ void char1d_left(const Char1& k, int f, double* Lr) {
#pragma clang fp contract(off)
  if (f == 0) {
    Lr[0] = 0.5 * mad(k.u, k.ic, k.b2);
    Lr[1] = -0.5 * mad(k.b1, k.u, k.ic);
    Lr[2] = 0.5 * k.b1;
  } else if (f == 1) {
    Lr[0] = 1.0 - k.b2;
    Lr[1] = k.b1 * k.u;
    Lr[2] = -k.b1;
  } else {
    Lr[0] = 0.5 * mad(-k.u, k.ic, k.b2);
    Lr[1] = -0.5 * mad(k.b1, k.u, -k.ic);
    Lr[2] = 0.5 * k.b1;
  }
}

__device__ __forceinline__ void char1d_right(const Char1& k, int f, double* Rc) {
#pragma clang fp contract(off)
  Rc[0] = 1.0;
  if (f == 0) {
    Rc[1] = k.u - k.c;
    Rc[2] = mad(-k.u, k.c, k.H);
  } else if (f == 1) {
    Rc[1] = k.u;
    Rc[2] = 0.5 * k.u * k.u;
  } else {
    Rc[1] = k.u + k.c;
    Rc[2] = mad(k.u, k.c, k.H);
  }
}

// row f of L and row f of R (component f of every field's eigenvector), for a lane that works
// on field f and then on component f (f = 3: an idle lane's, never used)
__device__ __forceinline__ void char1d_rows(const Char1& k, int f, double* Lr, double* Rr) {
#pragma clang fp contract(off)
  const double s = f == 0 ? 1.0 : -1.0;
  Lr[0] = f == 1 ? 1.0 - k.b2 : 0.5 * mad(s * k.u, k.ic, k.b2);
  Lr[1] = f == 1 ? k.b1 * k.u : -0.5 * mad(k.b1, k.u, s * k.ic);
  Lr[2] = f == 1 ? -k.b1 : 0.5 * k.b1;
  Rr[0] = f == 0 ? 1.0 : (f == 1 ? k.u - k.c : mad(-k.u, k.c, k.H));
  Rr[1] = f == 0 ? 1.0 : (f == 1 ? k.u : 0.5 * k.u * k.u);
  Rr[2] = f == 0 ? 1.0 : (f == 1 ? k.u + k.c : mad(k.u, k.c, k.H));
}

template <int EQ>
__device__ __forceinline__ void flux1d(const double* U, double gam, double a, double* f) {
  if constexpr (EQ == EQ_EULER) euler_flux1d(U, gam, f);
  else f[0] = scalar_flux<EQ>(U[0], a);
}

// One side's share of twice the Lax-Friedrichs flux f(u-) + f(u+) - alpha (u+ - u-) of a face: fu its
// flux, al = alpha for the low cell's u-, -alpha for the high cell's u+, ref the low cell's average,
// which both sides know.  Without ref (it drops out of the sum) the shares' sum loses the digits that
// alpha u cancels in: 25 % more rounding error in the density's right-hand side on a smooth wave.
__device__ __forceinline__ double flux_share1d(double u, double fu, double al, double ref) {
#pragma clang fp contract(off)
  return mad(al, u - ref, fu);
}

// the ghost's share at a wall face from the inner cell's trace u there: the ghost's trace is the
// same (momentum reversed at a reflective wall)
template <int EQ>
__device__ __forceinline__ void wall_share1d(const double* u, int bc, double gam, double adv, double al,
                                             const double* ref, double* share) {
  constexpr int NC = (EQ == EQ_EULER) ? 3 : 1;
  double g[NC], fg[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) g[c] = ((EQ == EQ_EULER && bc == BC_REFLECTIVE && c == 1) ? -1.0 : 1.0) * u[c];
  flux1d<EQ>(g, gam, adv, fg);
#pragma unroll
  for (int c = 0; c < NC; ++c) share[c] = flux_share1d(g[c], fg[c], al, ref[c]);
}

// the four-point Gauss-Lobatto sum of a cell's fluxes: the interior points' part, then all
__device__ __forceinline__ double lobatto_inner(double fm, double fp) {
#pragma clang fp contract(off)
  return (fm + fp) * (5.0 / 12.0);
}
__device__ __forceinline__ double lobatto_sum(double fL, double fR, double inner) {
#pragma clang fp contract(off)
  return mad(fL + fR, 1.0 / 12.0, inner);
}

// right-hand sides of eq. odeH: the shares of the low face and of the high face (own and other side)
__device__ __forceinline__ void rhs1d(double lo, double ownL, double ownR, double hi, double Fi, double idx,
                                      double& LU, double& LV) {
#pragma clang fp contract(off)
  const double FL = 0.5 * (lo + ownL), FR = 0.5 * (ownR + hi);
  LU = -(FR - FL) * idx;
  LV = (Fi - 0.5 * (FL + FR)) * idx;
}

// the stage combination of eq. RK: wn of u^n, own of the stage input (both limited)
__device__ __forceinline__ double rk_update(int mode, double wn, double own, double dt, double L) {
#pragma clang fp contract(off)
  if (mode == MODE_RK1) return mad(dt, L, own);
  if (mode == MODE_RK2) return mad(0.25 * dt, L, mad(0.75, wn, 0.25 * own));
  return mad((2.0 / 3.0) * dt, L, mad(wn, 1.0 / 3.0, (2.0 / 3.0) * own));
}

// A number of the sign of the velocity m / rho as the rounded quotient has it (zero where the
// quotient underflows): the quotient itself only where the operands do not tell.
__device__ __forceinline__ double velocity_sign(double m, double rho) {
  if (rho > 0.0 && rho < 1e100 && (m == 0.0 || fabs(m) > 1e-200)) return m;
  return m / rho;
}

// spectral radius at a cell average; a non-physical state sets bit 1 of bad
template <int EQ>
__device__ __forceinline__ double speed1d(const double* U, double gam, double adv, int& bad) {
#pragma clang fp contract(off)
  if constexpr (EQ == EQ_EULER) {
    const double ir = rcp_nr(U[0]), u = U[1] * ir;
    const double p = (gam - 1.0) * mad(-0.5 * U[1], u, U[2]);
    if (!(U[0] > 0.0) || !(p > 0.0)) bad |= 2;
    return fabs(u) + sqrt(gam * p * ir);
  } else if constexpr (EQ == EQ_BURGERS) {
    return fabs(U[0]);
  } else {
    return fabs(adv);
  }
}

// One tile: the cells i0 .. i0 + T1 - 7 of an instance, thread l on position i0 + l - 3.
// Bound by VALU issue (FP64), so every phase is one pass of the workgroup.  A tile of T1 cells took a
// second pass of its first or last wave for the two to six positions beyond them in the flags, the
// limiter, the traces and the faces, half as much again with two waves a tile, and evaluated
// each face's fluxes in both of its cells: 52.9 -> 42.9 us a launch for 512 Euler instances of 256 to
// 8192 cells with 128 threads, of which the bytes alone take 32 at the rate of a large copy.
// NU: a single instance on cells of different sizes (per-cell tables, hw_mesh1d.h)
template <int EQ, int T1, bool NU>
__device__ void stage1d_tile(const Stage1D& P, int inst, int i0, double* s_in, double* s_face,
                             uint8_t* s_T, double* s_red) {
  constexpr int L1 = T1;
  constexpr int NC = (EQ == EQ_EULER) ? 3 : 1;
  constexpr int NF = 2 * NC;
  const int tid = threadIdx.x, l = tid;
  const int mode = P.mode;
  const double alpha = __longlong_as_double((long long)P.alpha_in[inst]);
  double dt = 0.0;
  if (mode != MODE_L) {
    dt = P.dt[inst];
    if (dt == 0.0) return;   // uniform over the workgroup
  }
  const int off = P.off[inst], n = P.off[inst + 1] - off;
  const size_t tot = (size_t)P.total;
  // the cell an LDS position holds (a ghost: the cell it wraps to or mirrors) and its table
  auto tab = [&](int l) -> mesh1d::Tab {
    double sg;
    return mesh1d::Tab{P.nu, tot, off + map_index(i0 + l - H1, n, P.bc, sg)};
  };
  const double dx = NU ? tab(l)[mesh1d::K_DX] : P.dxs[inst];
  const double h = 0.5 * dx, idx = 1.0 / dx;

  // stage input -> LDS; a reflective wall's ghost also negates the momentum (average, moment)
  {
    double v[NF], sg;
    const int g = map_index(i0 + l - H1, n, P.bc, sg);
#pragma unroll
    for (int f = 0; f < NF; ++f) v[f] = P.in[f * tot + off + g];
    const bool refl = EQ == EQ_EULER && P.bc == BC_REFLECTIVE;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const double m = (refl && sg < 0.0 && f % NC == 1) ? -1.0 : 1.0;
      s_in[f * L1 + l] = m * (f >= NC ? sg * v[f] : v[f]);
    }
  }
  __syncthreads();
  auto A = [&](int f, int l) -> double { return s_in[f * L1 + l]; };

  // At a transmissive or reflective boundary a ghost cell is the mirror image of the cell
  // it faces in every respect: the ghost next to the boundary takes that cell's flag and
  // its limited moments (under the state's sign rule), and its trace on the boundary face
  // is that cell's trace there.  Ghosts further out only feed values that are replaced.
  // mirror_src: the LDS position whose flag and limited moments the position l takes.
  const bool walls = P.bc != BC_PERIODIC;
  auto mirror_src = [&](int l) -> int {
    if (walls) {
      const int gl = i0 + l - H1;
      if (gl == -1) return l + 1;
      if (gl == n) return l - 1;
    }
    return l;
  };

  // ---------------------------------------------------------------- flags on tile+2
  const bool in2 = l >= 1 && l < L1 - 1, in1 = l >= 2 && l < L1 - 2;   // tile+2, tile+1
  uint8_t myT = 0;
  if (in2) {
    if (P.tc_mode == TC_ALL) {
      myT = 1;
    } else if (P.tc_mode == TC_KXRCF) {
      const int lc = mirror_src(l);
      double vel;
      if constexpr (EQ == EQ_EULER) vel = velocity_sign(A(1, lc), A(0, lc));
      else if constexpr (EQ == EQ_BURGERS) vel = A(0, lc);
      else vel = P.adv;
      constexpr int ncheck = (EQ == EQ_EULER) ? 2 : 1;
      const double hl = NU ? 0.5 * tab(lc)[mesh1d::K_DX] : h;
      for (int k = 0; k < ncheck; ++k) {
        const int c = (k == 0) ? 0 : NC - 1;   // density, then energy
        if (kxrcf1d(A(c, lc), A(NC + c, lc), A(c, lc - 1), A(NC + c, lc - 1), A(c, lc + 1),
                    A(NC + c, lc + 1), vel, hl))
          myT = 1;
      }
    }
  }
  s_T[l] = myT;
  __syncthreads();

  // ---------------------------------------------------------------- limiter (Jacobi)
  double limv[NC];
  {
    if (myT) {
      // the ghost next to a wall takes the mirror of its neighbour's limited moments
      const int l = mirror_src(tid);
      const bool mir = l != tid;
      if constexpr (EQ != EQ_EULER) {
        if constexpr (NU)
          limv[0] = mesh1d::limit_moment_nu(tab(l), A(0, l - 1), A(0, l), A(0, l + 1),
                                                 A(1, l - 1), A(1, l + 1), P.w.lim, P.w.eps);
        else
          limv[0] = limit_moment(A(0, l - 1), A(0, l), A(0, l + 1), A(1, l - 1), A(1, l + 1),
                                      P.w.lim, P.w.eps);
        if (mir) limv[0] = -limv[0];
      } else {
        // field by field: project, limit, and add R's column times the limited moment
        const Char1 k = char1d(A(0, l), A(1, l), A(2, l), P.gam);
#pragma unroll
        for (int c = 0; c < 3; ++c) limv[c] = 0.0;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          double Lr[3], Rc[3];
          char1d_left(k, f, Lr);
          double um = 0.0, u0 = 0.0, up = 0.0, vm = 0.0, vp = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            um = fma(Lr[c], A(c, l - 1), um);
            u0 = fma(Lr[c], A(c, l), u0);
            up = fma(Lr[c], A(c, l + 1), up);
            vm = fma(Lr[c], A(3 + c, l - 1), vm);
            vp = fma(Lr[c], A(3 + c, l + 1), vp);
          }
          double vc;
          if constexpr (NU) vc = mesh1d::limit_moment_nu(tab(l), um, u0, up, vm, vp, P.w.lim, P.w.eps);
          else vc = limit_moment(um, u0, up, vm, vp, P.w.lim, P.w.eps);
          char1d_right(k, f, Rc);
#pragma unroll
          for (int c = 0; c < 3; ++c) limv[c] = mad(Rc[c], vc, limv[c]);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (mir) {
          // first moments are odd under the mirror; a wall also reverses the momentum
          limv[0] = -limv[0];
          if (P.bc != BC_REFLECTIVE) limv[1] = -limv[1];
          limv[2] = -limv[2];
        }
      }
    }
  }
  __syncthreads();
  if (myT) {
#pragma unroll
    for (int c = 0; c < NC; ++c) s_in[(NC + c) * L1 + l] = limv[c];
  }
  const uint8_t myH = in1 ? s_T[l - 1] | s_T[l] | s_T[l + 1] : 0;
  __syncthreads();

  // ---------------------------------------------------------------- reconstruction
  // interface values of cell l: left (u^+_{l-1/2}) and right (u^-_{l+1/2}), and the sum of the
  // Gauss-Lobatto rule over the cell's fluxes
  double left[NC], right[NC], fL[NC], fR[NC], Fi[NC];
  if (in1) {
    const bool hyb = myH != 0;
    // the HWENO branch first, so that no linear value is live across it
    if (hyb) {
      if constexpr (EQ != EQ_EULER) {
        if constexpr (NU) {
          const double d6[6] = {A(0, l - 1), A(0, l), A(0, l + 1), A(1, l - 1), A(1, l), A(1, l + 1)};
          mesh1d::hweno1d_nu(tab(l), d6, P.w.rec, P.w.eps, left[0], right[0]);
        } else {
          hweno1d(A(0, l - 1), A(0, l), A(0, l + 1), A(1, l - 1), A(1, l), A(1, l + 1), P.w.rec,
                  P.w.eps, left[0], right[0]);
        }
      } else {
        // field by field: project, reconstruct, and add R's column times the field's values
        const Char1 k = char1d(A(0, l), A(1, l), A(2, l), P.gam);
#pragma unroll
        for (int c = 0; c < 3; ++c) left[c] = right[c] = 0.0;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          double Lr[3], Rc[3];
          char1d_left(k, f, Lr);
          double d[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            d[0] = fma(Lr[c], A(c, l - 1), d[0]);
            d[1] = fma(Lr[c], A(c, l), d[1]);
            d[2] = fma(Lr[c], A(c, l + 1), d[2]);
            d[3] = fma(Lr[c], A(3 + c, l - 1), d[3]);
            d[4] = fma(Lr[c], A(3 + c, l), d[4]);
            d[5] = fma(Lr[c], A(3 + c, l + 1), d[5]);
          }
          double lf, rf;
          if constexpr (NU) mesh1d::hweno1d_nu(tab(l), d, P.w.rec, P.w.eps, lf, rf);
          else hweno1d(d[0], d[1], d[2], d[3], d[4], d[5], P.w.rec, P.w.eps, lf, rf);
          char1d_right(k, f, Rc);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            left[c] = mad(Rc[c], lf, left[c]);
            right[c] = mad(Rc[c], rf, right[c]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // linear values: the interface values of non-hybrid cells, the interior points of all
    double um[NC], up[NC], fm[NC], fp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double a, b;
      if constexpr (NU) {
        const double d6[6] = {A(c, l - 1), A(c, l), A(c, l + 1), A(NC + c, l - 1), A(NC + c, l),
                              A(NC + c, l + 1)};
        mesh1d::linear1d_nu(tab(l), d6, a, b, um[c], up[c]);
      } else {
        linear1d(A(c, l - 1), A(c, l), A(c, l + 1), A(NC + c, l - 1), A(NC + c, l),
                 A(NC + c, l + 1), a, b, um[c], up[c]);
      }
      if (!hyb) {
        left[c] = a;
        right[c] = b;
      }
    }
    flux1d<EQ>(left, P.gam, P.adv, fL);
    flux1d<EQ>(right, P.gam, P.adv, fR);
    flux1d<EQ>(um, P.gam, P.adv, fm);
    flux1d<EQ>(up, P.gam, P.adv, fp);
    // the cell's shares of its two faces' fluxes
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Fi[c] = lobatto_sum(fL[c], fR[c], lobatto_inner(fm[c], fp[c]));
      fL[c] = flux_share1d(left[c], fL[c], -alpha, A(c, l - 1));
      fR[c] = flux_share1d(right[c], fR[c], alpha, A(c, l));
      s_face[c * T1 + l] = fL[c];
      s_face[(NC + c) * T1 + l] = fR[c];
    }
  }
  const int gi = i0 + l - H1;
  const bool active = l >= H1 && l < T1 - H1 && gi < n;
  __syncthreads();
  double LU[NC], LV[NC];
  if (active) {
    double lo[NC], hi[NC];   // the neighbours' shares
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      lo[c] = s_face[(NC + c) * T1 + l - 1];
      hi[c] = s_face[c * T1 + l + 1];
    }
    if (walls && (gi == 0 || gi == n - 1)) {
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        if (gi != (side == 0 ? 0 : n - 1)) continue;
        double ref[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) ref[c] = A(c, l - 1 + side);
        wall_share1d<EQ>(side == 0 ? left : right, P.bc, P.gam, P.adv, side == 0 ? alpha : -alpha, ref, side == 0 ? lo : hi);
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) rhs1d(lo[c], fL[c], fR[c], hi[c], Fi[c], idx, LU[c], LV[c]);
  }
  double own[NF];   // the (limited) stage input
#pragma unroll
  for (int f = 0; f < NF; ++f) own[f] = A(f, l);
  __syncthreads();   // the LDS is reused by the next work item

  // ---------------------------------------------------------------- epilogue
  // (the ghosts' speeds are left out of the maximum as NaN is: a full tile without a speed that is a
  // number counts as infinitely fast, and the steps after it stand still)
  double sp = l >= H1 && l < T1 - H1 ? 0.0 : __builtin_nan("");
  if (active) {
    const size_t gidx = (size_t)off + gi;
    if (P.flagsT) P.flagsT[gidx] = myT;
    if (P.flagsH) P.flagsH[gidx] = myH;
    if (mode == MODE_L) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        P.out[c * tot + gidx] = LU[c];
        P.out[(NC + c) * tot + gidx] = LV[c];
      }
      if (P.wout) {
#pragma unroll
        for (int f = 0; f < NF; ++f) P.wout[f * tot + gidx] = own[f];
      }
    } else {
      double Wn[NF];
      if (mode == MODE_RK1) {
#pragma unroll
        for (int f = 0; f < NF; ++f) Wn[f] = own[f];
        P.Tn[gidx] = myT;
        if (myT) {
#pragma unroll
          for (int c = 0; c < NC; ++c) P.limn[c * tot + gidx] = own[NC + c];
        }
      } else {
#pragma unroll
        for (int f = 0; f < NF; ++f) Wn[f] = P.base[f * tot + gidx];
        if (P.Tn[gidx]) {
#pragma unroll
          for (int c = 0; c < NC; ++c) Wn[NC + c] = P.limn[c * tot + gidx];
        }
      }
      double res[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        res[f] = rk_update(mode, Wn[f], own[f], dt, f < NC ? LU[f] : LV[f - NC]);
      }
      int bad = 0;
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        P.out[f * tot + gidx] = res[f];
        if (!isfinite(res[f])) bad |= 1;
      }
      sp = speed1d<EQ>(res, P.gam, P.adv, bad);
      if (bad) atomicOr(P.status, bad);
    }
  }
  if (mode != MODE_L) {
    const double m = block_max<T1 / 64>(sp, s_red);
    if (tid == 0) atomic_max_pos(&P.alpha_out[inst], m);
    __syncthreads();
  }
}

template <int EQ, int T1, bool NU>
__global__ __launch_bounds__(T1) void stage1d_kernel(Stage1D P) {
  constexpr int NF = (EQ == EQ_EULER) ? 6 : 2;
  __shared__ double s_in[NF * T1];
  __shared__ double s_face[NF * T1];
  __shared__ uint8_t s_T[T1];
  __shared__ double s_red[T1 / 64];
  const int2 it = P.items[blockIdx.x];
  stage1d_tile<EQ, T1, NU>(P, it.x, it.y, s_in, s_face, s_T, s_red);
}

// persistent form: a grid sized to the machine walks the work list
template <int EQ, int T1>
__global__ __launch_bounds__(T1, 4) void stage1d_persistent(Stage1D P) {
  constexpr int NF = (EQ == EQ_EULER) ? 6 : 2;
  __shared__ double s_in[NF * T1];
  __shared__ double s_face[NF * T1];
  __shared__ uint8_t s_T[T1];
  __shared__ double s_red[T1 / 64];
  for (int item = blockIdx.x; item < P.nitems; item += gridDim.x) {
    const int2 it = P.items[item];
    stage1d_tile<EQ, T1, false>(P, it.x, it.y, s_in, s_face, s_T, s_red);
  }
}

// maximum over a wave of non-negative values (NaN ignored; NaN where all are), in lane 63: register
// moves within rows of 16 lanes, then across them (a lane without a source keeps its own value)
__device__ __forceinline__ double wave_max63(double v) {
#define HW_MAX_DPP(ctrl)                                                                         \
  v = fmax(v, __hiloint2double(__builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), ctrl, 0xF, 0xF, false), \
                               __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), ctrl, 0xF, 0xF, false)))
  HW_MAX_DPP(0x111);   // row_shr:1
  HW_MAX_DPP(0x112);
  HW_MAX_DPP(0x114);
  HW_MAX_DPP(0x118);
  HW_MAX_DPP(0x142);   // row_bcast:15
  HW_MAX_DPP(0x143);   // row_bcast:31
#undef HW_MAX_DPP
  return v;
}

// The instance's speed from its waves' maxima: 256 cells without a speed that is a number count as
// infinitely fast, as a full tile of the stage launches does.
template <int NW>
__device__ __forceinline__ double whole_speed(const double* red) {
  double a = 0.0;
#pragma unroll
  for (int g = 0; g < NW; g += 4) {
    double m = red[g];
#pragma unroll
    for (int i = g + 1; i < g + 4 && i < NW; ++i) m = fmax(m, red[i]);
    if (NW >= 4 && !(m >= 0.0)) m = __longlong_as_double(0x7ff0000000000000ll);
    a = fmax(a, m);
  }
  return a;
}

// LDS of one whole instance of at most T1 cells
template <int EQ, int T1>
struct WholeShared {
  static constexpr int NC = (EQ == EQ_EULER) ? 3 : 1, NF = 2 * NC, L1 = T1 + 2 * H1;
  double in[NF * L1];           // stage input with ghosts, then limited
  double fm[NC * (T1 + 1)];     // u^- at the faces, then the low cell's share of its flux
  double fp[NC * (T1 + 1)];     // u^+, then the high cell's
  double fx[NC * T1];           // limited moments of the flagged cells
  double red[T1 / 64];
  uint16_t fl[T1], hl[T1];      // flagged and hybrid cells
  uint8_t T[L1];
  int cnt[2], bad;
};

// The spatial operator on a whole instance staged in sh.in (its flags' and limiter's ghosts
// are filled here).  Few cells of an instance are troubled, and a cell's characteristic
// limiter or reconstruction is several times as long as the linear path, so the work lists of
// those cells are spread over all lanes, four per Euler cell (lane f: characteristic field f,
// then component f): the wave that holds a shock would otherwise set the stage's time.
template <int EQ, int T1>
__device__ __forceinline__ void whole_operator(const Stage1D& P, WholeShared<EQ, T1>& sh, int n, double h,
                                               double idx, double alpha, double* LU, double* LV, double* own,
                                               uint8_t& myT, uint8_t& myH) {
  constexpr int NC = (EQ == EQ_EULER) ? 3 : 1, NF = 2 * NC, L1 = T1 + 2 * H1, F1 = T1 + 1;
  constexpr int LPC = (EQ == EQ_EULER) ? 4 : 1;   // lanes per listed cell
  const int tid = threadIdx.x, l = tid + H1;
  const bool active = tid < n;
  const bool walls = P.bc != BC_PERIODIC;
  auto A = [&](int f, int q) -> double { return sh.in[f * L1 + q]; };
  // the ghost next to an end that cell i is the source of (0: none)
  auto end_ghost = [&](int i) -> int {
    if (i == 0) return walls ? H1 - 1 : H1 + n;
    if (i == n - 1) return walls ? H1 + n : H1 - 1;
    return 0;
  };
  // ---------------------------------------------------------------- flags, work lists
  myT = myH = 0;
  if (active) {
    if (P.tc_mode == TC_ALL) {
      myT = 1;
    } else if (P.tc_mode == TC_KXRCF) {
      double vel;
      if constexpr (EQ == EQ_EULER) vel = velocity_sign(A(1, l), A(0, l));
      else if constexpr (EQ == EQ_BURGERS) vel = A(0, l);
      else vel = P.adv;
      constexpr int ncheck = (EQ == EQ_EULER) ? 2 : 1;
#pragma unroll
      for (int k = 0; k < ncheck; ++k) {
        const int c = (k == 0) ? 0 : NC - 1;   // density, then energy
        if (kxrcf1d(A(c, l), A(NC + c, l), A(c, l - 1), A(NC + c, l - 1), A(c, l + 1), A(NC + c, l + 1), vel, h))
          myT = 1;
      }
    }
    sh.T[l] = myT;
    const int g = end_ghost(tid);
    if (g) sh.T[g] = myT;
    if (myT) sh.fl[atomicAdd(&sh.cnt[0], 1)] = (uint16_t)tid;
  }
  __syncthreads();
  const int nfl = sh.cnt[0];
  if (active) {
    myH = sh.T[l - 1] | sh.T[l] | sh.T[l + 1];
    if (myH) sh.hl[atomicAdd(&sh.cnt[1], 1)] = (uint16_t)tid;
  }
  // ---------------------------------------------------------------- limiter (Jacobi)
  for (int it = tid; it < nfl * LPC; it += T1) {   // (whole groups of LPC lanes)
    const int f = it % LPC, q = sh.fl[it / LPC] + H1;
    if constexpr (EQ != EQ_EULER) {
      sh.fx[it] = limit_moment(A(0, q - 1), A(0, q), A(0, q + 1), A(1, q - 1), A(1, q + 1), P.w.lim, P.w.eps);
    } else {
      const Char1 k = char1d(A(0, q), A(1, q), A(2, q), P.gam);
      double Lr[3], Rr[3];
      char1d_rows(k, f, Lr, Rr);
      double um = 0.0, u0 = 0.0, up = 0.0, vm = 0.0, vp = 0.0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        um = fma(Lr[c], A(c, q - 1), um);
        u0 = fma(Lr[c], A(c, q), u0);
        up = fma(Lr[c], A(c, q + 1), up);
        vm = fma(Lr[c], A(3 + c, q - 1), vm);
        vp = fma(Lr[c], A(3 + c, q + 1), vp);
      }
      double x[4];
      quad_gather(limit_moment(um, u0, up, vm, vp, P.w.lim, P.w.eps), x);
      double out = 0.0;
#pragma unroll
      for (int g = 0; g < 3; ++g) out = mad(Rr[g], x[g], out);
      if (f < 3) sh.fx[(it / LPC) * NC + f] = out;
    }
  }
  __syncthreads();
  const int nhl = sh.cnt[1];
  for (int it = tid; it < nfl * NC; it += T1) {
    const int c = it % NC, i = sh.fl[it / NC], g = end_ghost(i);
    const double v = sh.fx[it];
    sh.in[(NC + c) * L1 + i + H1] = v;
    // a ghost at a wall holds the mirror image (the moment odd; a reflective wall also
    // reverses the momentum)
    if (g) sh.in[(NC + c) * L1 + g] = walls && !(EQ == EQ_EULER && P.bc == BC_REFLECTIVE && c == 1) ? -v : v;
  }
  __syncthreads();
  // ---------------------------------------------------------------- reconstruction
  auto put = [&](int i, int c, double left, double right) {
    sh.fp[c * F1 + i] = left;
    sh.fm[c * F1 + i + 1] = right;
  };
  for (int it = tid; it < nhl * LPC; it += T1) {
    const int f = it % LPC, i = sh.hl[it / LPC], q = i + H1;
    double left, right;
    if constexpr (EQ != EQ_EULER) {
      hweno1d(A(0, q - 1), A(0, q), A(0, q + 1), A(1, q - 1), A(1, q), A(1, q + 1), P.w.rec, P.w.eps, left, right);
      put(i, 0, left, right);
    } else {
      const Char1 k = char1d(A(0, q), A(1, q), A(2, q), P.gam);
      double Lr[3], Rr[3], d[6] = {0, 0, 0, 0, 0, 0};
      char1d_rows(k, f, Lr, Rr);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        d[0] = fma(Lr[c], A(c, q - 1), d[0]);
        d[1] = fma(Lr[c], A(c, q), d[1]);
        d[2] = fma(Lr[c], A(c, q + 1), d[2]);
        d[3] = fma(Lr[c], A(3 + c, q - 1), d[3]);
        d[4] = fma(Lr[c], A(3 + c, q), d[4]);
        d[5] = fma(Lr[c], A(3 + c, q + 1), d[5]);
      }
      hweno1d(d[0], d[1], d[2], d[3], d[4], d[5], P.w.rec, P.w.eps, left, right);
      double xl[4], xr[4], ol = 0.0, orr = 0.0;
      quad_gather(left, xl);
      quad_gather(right, xr);
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        ol = mad(Rr[g], xl[g], ol);
        orr = mad(Rr[g], xr[g], orr);
      }
      if (f < 3) put(i, f, ol, orr);
    }
  }
  // (what needs no other lane's traces comes before the barrier: it covers the lists' latency)
  double Fi[NC], refL[NC], refR[NC];
  if (active) {
    double um[NC], up[NC], fm[NC], fp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double a, b;
      refL[c] = A(c, l - 1);
      refR[c] = A(c, l);
      linear1d(refL[c], refR[c], A(c, l + 1), A(NC + c, l - 1), A(NC + c, l), A(NC + c, l + 1), a, b, um[c], up[c]);
      if (!myH) put(tid, c, a, b);
    }
    flux1d<EQ>(um, P.gam, P.adv, fm);
    flux1d<EQ>(up, P.gam, P.adv, fp);
#pragma unroll
    for (int c = 0; c < NC; ++c) Fi[c] = lobatto_inner(fm[c], fp[c]);
  }
  __syncthreads();
  // ---------------------------------------------------------------- fluxes
  // the cell's shares of its two faces take the place of its traces
  double left[NC], right[NC], fL[NC], fR[NC];
  if (active) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      left[c] = sh.fp[c * F1 + tid];
      right[c] = sh.fm[c * F1 + tid + 1];
    }
    flux1d<EQ>(left, P.gam, P.adv, fL);
    flux1d<EQ>(right, P.gam, P.adv, fR);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      Fi[c] = lobatto_sum(fL[c], fR[c], Fi[c]);
      fL[c] = flux_share1d(left[c], fL[c], -alpha, refL[c]);
      fR[c] = flux_share1d(right[c], fR[c], alpha, refR[c]);
      sh.fp[c * F1 + tid] = fL[c];
      sh.fm[c * F1 + tid + 1] = fR[c];
      // around the ends of a periodic instance (walls: replaced below)
      if (tid == 0) sh.fp[c * F1 + n] = fL[c];
      if (tid == n - 1) sh.fm[c * F1] = fR[c];
    }
  }
  __syncthreads();
  if (active) {
    double lo[NC], hi[NC];   // the neighbours' shares
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      lo[c] = sh.fm[c * F1 + tid];
      hi[c] = sh.fp[c * F1 + tid + 1];
    }
    if (walls && (tid == 0 || tid == n - 1)) {
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        if (tid != (side == 0 ? 0 : n - 1)) continue;
        wall_share1d<EQ>(side == 0 ? left : right, P.bc, P.gam, P.adv, side == 0 ? alpha : -alpha,
                         side == 0 ? refL : refR, side == 0 ? lo : hi);
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) rhs1d(lo[c], fL[c], fR[c], hi[c], Fi[c], idx, LU[c], LV[c]);
#pragma unroll
    for (int f = 0; f < NF; ++f) own[f] = A(f, l);   // the (limited) stage input
  }
}

// Whole steps of short instances: one workgroup keeps an instance of at most T1 cells in LDS and
// registers for up to nsteps TVD-RK3 steps (time step, three stages, speeds), one cell per
// thread, and reads and writes global memory only at the two ends.  A step of separate
// launches costs their latency, 41 us at 400 cells (time step 4.6, stages 11.5 each, gaps);
// here a stage is six barriers among the instance's own waves, and its 5 us are a chain of
// latencies spread evenly over them: staging and speeds 1.0, flags 0.6, limiter 0.8, write-back
// 0.2, reconstruction 0.8, linear traces 0.8, fluxes 0.7, update 0.8.  The arithmetic per cell is
// the tile routine's, to the bit: an instance's values depend neither on the form nor on the other
// instances of its batch.
//
// Measured, us a step, Euler shock tubes, stage launches in their best width / this: 64 cells 26 /
// 14; 256 25 / 15; 500 26 / 16; 1000 26 / 21.  Batches: hw_step1d_pays.  (1024 threads: 128 VGPRs, 17
// values in scratch.)
template <int EQ, int T1>
__global__ __launch_bounds__(T1) void step1d_kernel(Stage1D P, Step1D Q, int nsteps) {
  constexpr int NC = (EQ == EQ_EULER) ? 3 : 1, NF = 2 * NC, L1 = T1 + 2 * H1, NW = T1 / 64;
  __shared__ WholeShared<EQ, T1> sh;
  double* const s_in = sh.in;
  double* const s_red = sh.red;
  const int inst = blockIdx.x, tid = threadIdx.x;
  const int off = P.off[inst], n = P.off[inst + 1] - off;
  const size_t tot = (size_t)P.total, gidx = (size_t)off + tid;
  const bool active = tid < n;
  const int W = gridDim.x;   // speed entries per slot
  double u[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) u[f] = active ? Q.S[f * tot + gidx] : 0.0;
  double t = Q.t[inst], dt = 0.0;
  long long steps = Q.steps[inst];
  double alpha = __longlong_as_double((long long)Q.alpha[3 * W + inst]);
  const double dxs = P.dxs[inst], idx = 1.0 / dxs;
  if (tid == 0) sh.bad = 0;
  // the ghost position this cell's values also go to (each ghost has one source cell, and no
  // cell is the source of two: n >= 7), and the factor of its first moments and momentum there
  int ghost = -1;
  double gs = 1.0;
#pragma unroll
  for (int g = 0; g < 2 * H1; ++g) {
    const int gg = g < H1 ? g - H1 : n + g - H1;
    double sg;
    if (active && map_index(gg, n, P.bc, sg) == tid) {
      ghost = gg + H1;
      gs = sg;
    }
  }
  const bool refl = EQ == EQ_EULER && P.bc == BC_REFLECTIVE && gs < 0.0;
  int bad = 0;
#pragma unroll 1
  for (int k = 0; k < nsteps; ++k) {
    // a run to a final time: stop on a non-physical state, every 16 steps (as the chunks of
    // separate launches do)
    if (Q.T_end > 0.0 && k > 0 && (k & 15) == 0) {
      if (bad) sh.bad = 1;
      __syncthreads();
      if (sh.bad) break;
    }
    if (k > 0) {
      // speed of the last stage's output (written before barriers of that stage's end)
      __syncthreads();
      alpha = whole_speed<NW>(s_red);
    }
    dt = Q.fixed_dt > 0.0 ? Q.fixed_dt : Q.cfl * dxs / alpha;
    if (Q.T_end > 0.0) {
      if (t >= Q.T_end) dt = 0.0;
      else if (t + dt > Q.T_end) dt = Q.T_end - t;
    }
    if (dt == 0.0) break;
    if (dt > 0.0) {
      t += dt;
      steps += 1;
    }
    double Wn[NF];
#pragma unroll 1
    for (int stage = 0; stage < 3; ++stage) {
      if (active) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          s_in[f * L1 + H1 + tid] = u[f];
          if (ghost >= 0) {
            const double m = (refl && f % NC == 1) ? -1.0 : 1.0;
            s_in[f * L1 + ghost] = m * (f >= NC ? gs * u[f] : u[f]);
          }
        }
      }
      if (tid < 2) sh.cnt[tid] = 0;
      __syncthreads();
      if (stage > 0) alpha = whole_speed<NW>(s_red);
      double LU[NC], LV[NC], own[NF];
      uint8_t myT = 0, myH = 0;
      whole_operator<EQ, T1>(P, sh, n, 0.5 * dxs, idx, alpha, LU, LV, own, myT, myH);
      double sp = 0.0;
      if (active) {
        if (Q.flagsT[0]) {
          uint8_t* fT = stage == 0 ? Q.flagsT[0] : (stage == 1 ? Q.flagsT[1] : Q.flagsT[2]);
          uint8_t* fH = stage == 0 ? Q.flagsH[0] : (stage == 1 ? Q.flagsH[1] : Q.flagsH[2]);
          fT[gidx] = myT;
          fH[gidx] = myH;
        }
        if (stage == 0) {
#pragma unroll
          for (int f = 0; f < NF; ++f) Wn[f] = own[f];
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const double v = rk_update(MODE_RK1 + stage, Wn[f], own[f], dt, f < NC ? LU[f] : LV[f - NC]);
          u[f] = v;
          if (!isfinite(v)) bad |= 1;
        }
        sp = speed1d<EQ>(u, P.gam, P.adv, bad);
      }
      // (the last reads of s_red come before barriers of the operator above)
      sp = wave_max63(sp);
      if ((tid & 63) == 63) s_red[tid >> 6] = sp;
    }
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int f = 0; f < NF; ++f) Q.S[f * tot + gidx] = u[f];
  }
  if (bad) atomicOr(P.status, bad);
  if (tid == 0) {
    if (steps != Q.steps[inst] || !(dt == 0.0)) {
      // (at least one step was taken: the speed of its result)
      Q.alpha[3 * W + inst] = (unsigned long long)__double_as_longlong(whole_speed<NW>(s_red));
    }
    Q.dt[inst] = dt;
    Q.t[inst] = t;
    Q.steps[inst] = steps;
  }
}

// Lax-Friedrichs speed per instance (before the first stage; operator-only calls)
template <int EQ>
__global__ __launch_bounds__(256) void alpha1d_kernel(const double* U, const int* off, int total,
                                                      double gam, double adv,
                                                      unsigned long long* alpha_out) {
  __shared__ double s_red[4];
  const int inst = blockIdx.y;
  const int o = off[inst], n = off[inst + 1] - o;
  double m = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    if constexpr (EQ == EQ_EULER) {
      const double rho = U[o + i], mom = U[(size_t)total + o + i], E = U[2 * (size_t)total + o + i];
      const double p = (gam - 1.0) * (E - mom * mom / (2.0 * rho));
      m = fmax(m, fabs(mom / rho) + sqrt(gam * p / rho));
    } else if constexpr (EQ == EQ_BURGERS) {
      m = fmax(m, fabs(U[o + i]));
    } else {
      m = fabs(adv);
    }
  }
  const double r = block_max256(m, s_red);
  if (threadIdx.x == 0) atomic_max_pos(&alpha_out[inst], r);
}

// ------------------------------------------------------------------ mesh tables
namespace mesh1d {

__device__ __forceinline__ double ipow(double x, int m) {
  double r = 1.0;
  for (int k = 0; k < m; ++k) r *= x;
  return r;
}

// int_lo^hi xi^m dxi
__device__ __forceinline__ double imono(int m, double lo, double hi) {
  return (ipow(hi, m + 1) - ipow(lo, m + 1)) / (m + 1);
}

// Condition row entry m: average (kind 0) or first moment (kind 1) of xi^m over the cell of
// centre c and width w
__device__ __forceinline__ double cond(int kind, double c, double w, int m) {
  const double lo = c - 0.5 * w, hi = c + 0.5 * w;
  if (kind == 0) return imono(m, lo, hi) / w;
  return (imono(m + 1, lo, hi) - c * imono(m, lo, hi)) / (w * w);
}

// Inverse of the N x N matrix A (row-major; destroyed) by Gauss-Jordan elimination with
// partial pivoting
template <int N>
__device__ void invert(double* A, double* X) {
  for (int r = 0; r < N; ++r)
    for (int c = 0; c < N; ++c) X[r * N + c] = r == c ? 1.0 : 0.0;
  for (int k = 0; k < N; ++k) {
    int piv = k;
    for (int r = k + 1; r < N; ++r)
      if (fabs(A[r * N + k]) > fabs(A[piv * N + k])) piv = r;
    if (piv != k)
      for (int c = 0; c < N; ++c) {
        double t = A[k * N + c]; A[k * N + c] = A[piv * N + c]; A[piv * N + c] = t;
        t = X[k * N + c]; X[k * N + c] = X[piv * N + c]; X[piv * N + c] = t;
      }
    const double ip = 1.0 / A[k * N + k];
    for (int c = 0; c < N; ++c) {
      A[k * N + c] *= ip;
      X[k * N + c] *= ip;
    }
    for (int r = 0; r < N; ++r) {
      if (r == k) continue;
      const double f = A[r * N + k];
      for (int c = 0; c < N; ++c) {
        A[r * N + c] -= f * A[k * N + c];
        X[r * N + c] -= f * X[k * N + c];
      }
    }
  }
}

// Upper factor R of the Gram matrix of eq. GHYZ in xi on the monomials xi^1..xi^r
// (G = R^T R; the constant monomial has no derivative), row-major r x r
template <int r>
__device__ void gram_factor(double* R) {
  double G[r * r];
  for (int m = 1; m <= r; ++m)
    for (int n = 1; n <= r; ++n) {
      double s = 0.0;
      for (int l = 1; l <= (m < n ? m : n); ++l) {
        double fm = 1.0, fn = 1.0;
        for (int t = 0; t < l; ++t) {
          fm *= (m - t);
          fn *= (n - t);
        }
        s += fm * fn * imono(m + n - 2 * l, -0.5, 0.5);
      }
      G[(m - 1) * r + (n - 1)] = s;
    }
  for (int i = 0; i < r * r; ++i) R[i] = 0.0;
  for (int j = 0; j < r; ++j) {
    double d = G[j * r + j];
    for (int k = 0; k < j; ++k) d -= R[k * r + j] * R[k * r + j];
    const double rjj = sqrt(d);
    R[j * r + j] = rjj;
    for (int i = j + 1; i < r; ++i) {
      double v = G[j * r + i];
      for (int k = 0; k < j; ++k) v -= R[k * r + j] * R[k * r + i];
      R[j * r + i] = v / rjj;
    }
  }
}

// The polynomial of degree N - 1 fixed by N conditions (kind[q], cell j[q]): its monomial
// coefficients as linear maps of the conditions' data, C[m * N + q]
template <int N>
__device__ void poly_map(const int* kind, const int* j, const double* cc, const double* ww, double* C) {
  double A[N * N];
  for (int q = 0; q < N; ++q)
    for (int m = 0; m < N; ++m) A[q * N + m] = cond(kind[q], cc[j[q] + 1], ww[j[q] + 1], m);
  invert<N>(A, C);
}

// value of the polynomial at xi as a map of its data
template <int N>
__device__ void point_row(const double* C, double xi, double* row) {
  for (int q = 0; q < N; ++q) {
    double s = 0.0;
    for (int m = N - 1; m >= 0; --m) s = s * xi + C[m * N + q];
    row[q] = s;
  }
}

// first moment over [-1/2, 1/2] as a map of the data
template <int N>
__device__ void moment_row(const double* C, double* row) {
  for (int q = 0; q < N; ++q) {
    double s = 0.0;
    for (int m = 0; m < N; ++m) s += imono(m + 1, -0.5, 0.5) * C[m * N + q];
    row[q] = s;
  }
}

// indicator rows R C (rows 0..N-2, over the data) for the Gram factor of degree N - 1
template <int N>
__device__ void beta_rows(const double* C, double* rows) {
  constexpr int r = N - 1;
  double R[r * r];
  gram_factor<r>(R);
  for (int a = 0; a < r; ++a)
    for (int q = 0; q < N; ++q) {
      double s = 0.0;
      for (int m = 1; m <= r; ++m) s += R[a * r + (m - 1)] * C[m * N + q];
      rows[a * N + q] = s;
    }
}

// one instance of n cells whose table columns start at column base of tables with stride
// columns per field
__global__ __launch_bounds__(256) void mesh1d_setup_kernel(const double* faces, int n, int bc,
                                                            double* tab, size_t stride, int base) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const double dx = faces[i + 1] - faces[i];
  double dl, dr;   // neighbour sizes (periodic wrap; a mirrored ghost has the cell's size)
  if (bc == BC_PERIODIC) {
    dl = i > 0 ? faces[i] - faces[i - 1] : faces[n] - faces[n - 1];
    dr = i < n - 1 ? faces[i + 2] - faces[i + 1] : faces[1] - faces[0];
  } else {
    dl = i > 0 ? faces[i] - faces[i - 1] : dx;
    dr = i < n - 1 ? faces[i + 2] - faces[i + 1] : dx;
  }
  const double a = dl / dx, b = dr / dx;
  const double cc[3] = {-0.5 - 0.5 * a, 0.0, 0.5 + 0.5 * b}, ww[3] = {a, 1.0, b};
  auto put = [&](int k, const double* v, int len) {
    for (int q = 0; q < len; ++q) tab[(size_t)(k + q) * stride + base + i] = v[q];
  };
  const double one[1] = {dx};
  put(K_DX, one, 1);
  double row[6];
  {  // Step 1: quartic on the three cells' averages and the neighbours' first moments
    const int kind[5] = {0, 0, 0, 1, 1}, j[5] = {-1, 0, 1, -1, 1};
    double C[25], rows[20];
    poly_map<5>(kind, j, cc, ww, C);
    moment_row<5>(C, row);
    put(K_LQ0, row, 5);
    beta_rows<5>(C, rows);
    put(K_LB0, rows, 20);
  }
  {  // the linear q1, q2 and their slopes
    const int kind[2] = {0, 0}, jm[2] = {-1, 0}, jp[2] = {0, 1};
    double C[4];
    poly_map<2>(kind, jm, cc, ww, C);
    moment_row<2>(C, row);
    put(K_LQ1, row, 2);
    put(K_LB1, C + 2, 2);
    poly_map<2>(kind, jp, cc, ww, C);
    moment_row<2>(C, row);
    put(K_LQ2, row, 2);
    put(K_LB2, C + 2, 2);
  }
  {  // Step 2: quintic on the three cells' averages and first moments
    const int kind[6] = {0, 0, 0, 1, 1, 1}, j[6] = {-1, 0, 1, -1, 0, 1};
    double C[36], rows[30];
    poly_map<6>(kind, j, cc, ww, C);
    point_row<6>(C, -0.5, row);
    put(K_RL0, row, 6);
    point_row<6>(C, 0.5, row);
    put(K_RR0, row, 6);
    const double s5 = 0.223606797749978969640917366873127624;   // sqrt(5) / 10
    point_row<6>(C, -s5, row);
    put(K_RIM, row, 6);
    point_row<6>(C, s5, row);
    put(K_RIP, row, 6);
    beta_rows<6>(C, rows);
    put(K_RB0, rows, 30);
  }
  {  // the quadratics p1 (u_{-1}, u_0, v_0) and p2 (u_0, u_{+1}, v_0)
    const int kind[3] = {0, 0, 1}, jm[3] = {-1, 0, 0}, jp[3] = {0, 1, 0};
    double C[9], rows[6];
    poly_map<3>(kind, jm, cc, ww, C);
    point_row<3>(C, -0.5, row);
    put(K_RL1, row, 3);
    point_row<3>(C, 0.5, row);
    put(K_RR1, row, 3);
    beta_rows<3>(C, rows);
    put(K_RB1, rows, 6);
    poly_map<3>(kind, jp, cc, ww, C);
    point_row<3>(C, -0.5, row);
    put(K_RL2, row, 3);
    point_row<3>(C, 0.5, row);
    put(K_RR2, row, 3);
    beta_rows<3>(C, rows);
    put(K_RB2, rows, 6);
  }
}

}  // namespace mesh1d

}  // namespace hw

template <int EQ, int T>
static void launch1d(int persistent, int grid, const hw::Stage1D* P, hipStream_t s) {
  if (persistent) hipLaunchKernelGGL((hw::stage1d_persistent<EQ, T>), dim3(grid), dim3(T), 0, s, *P);
  else hipLaunchKernelGGL((hw::stage1d_kernel<EQ, T, false>), dim3(P->nitems), dim3(T), 0, s, *P);
}

template <int EQ>
static hipError_t launch1d_tile(int persistent, int grid, int tile, const hw::Stage1D* P, hipStream_t s) {
  switch (tile) {
    case 64: launch1d<EQ, 64>(persistent, grid, P, s); break;
    case 128: launch1d<EQ, 128>(persistent, grid, P, s); break;
    case 256: launch1d<EQ, 256>(persistent, grid, P, s); break;
    case 512: launch1d<EQ, 512>(persistent, grid, P, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

extern "C" hipError_t hw_launch_stage1d(int eq, int persistent, int grid, int tile,
                                        const hw::Stage1D* P, hipStream_t s) {
  if (P->nu) {
    // cells of different sizes: tiles of TILE1D_NU positions, one workgroup per tile.  (The Euler
    // instance keeps 146 values in accumulation registers beside 256 VGPRs: one wave per SIMD.)
    dim3 g(P->nitems), b(256);
    if (eq == hw::EQ_EULER) hipLaunchKernelGGL((hw::stage1d_kernel<hw::EQ_EULER, 256, true>), g, b, 0, s, *P);
    else if (eq == hw::EQ_BURGERS) hipLaunchKernelGGL((hw::stage1d_kernel<hw::EQ_BURGERS, 256, true>), g, b, 0, s, *P);
    else if (eq == hw::EQ_ADV) hipLaunchKernelGGL((hw::stage1d_kernel<hw::EQ_ADV, 256, true>), g, b, 0, s, *P);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  if (eq == hw::EQ_EULER) return launch1d_tile<hw::EQ_EULER>(persistent, grid, tile, P, s);
  if (eq == hw::EQ_BURGERS) return launch1d_tile<hw::EQ_BURGERS>(persistent, grid, tile, P, s);
  if (eq == hw::EQ_ADV) return launch1d_tile<hw::EQ_ADV>(persistent, grid, tile, P, s);
  return hipErrorInvalidValue;
}

// Threads per instance of the one-workgroup form: the smallest count that gives every cell a
// thread, and 0 (separate launches) where an instance is longer than a workgroup, or where
// there are per-cell tables: with those the kernel spills (96 us a step against 61 at 400 cells).
extern "C" int hw_step1d_threads(int maxn, int nonuniform) {
  if (nonuniform || maxn > 1024) return 0;
  return maxn <= 128 ? 128 : (maxn <= 256 ? 256 : (maxn <= 512 ? 512 : 1024));
}

// Whether whole steps take less time than the stage launches, from what both measured (us a step;
// shock tubes).  A round of workgroups takes as long as one of them, whatever its instance fills of it, and
// a compute unit holds 4, 2, 1 and 1 Euler workgroups of 128 to 1024 threads, 8, 4, 2 and 1 scalar ones;
// the stage launches take a time per cell and one per instance (at their default width).
// Whole steps / stage launches, Euler: 1 of 1000 cells 22 / 26; 512 of 64 to 1024 45 / 50, 1024 of them
// 86 / 70, 4096 313 / 169; 4096 of 1000 351 / 406; 2048 of 500 135 / 125; 4096 of 64 77 / 93; 4000 of 64 with one
// of 1000 276 / 93.  Burgers: 512 of 64 to 1024 23 / 26, 4096 of them 158 / 79; 4096 of 256 45 / 65; 4000 of 64
// with one of 1000 140 / 43.
extern "C" int hw_step1d_pays(int eq, int threads, int ninst, long cells) {
  const int w = threads <= 128 ? 0 : (threads <= 256 ? 1 : (threads <= 512 ? 2 : 3));
  const bool euler = eq == hw::EQ_EULER;
  const int round_e[4] = {1024, 512, 256, 256}, round_s[4] = {2048, 1024, 512, 256};
  const double us_e[4] = {19.0, 17.6, 16.7, 23.0}, us_s[4] = {13.0, 11.3, 10.9, 11.5};
  const int per = euler ? round_e[w] : round_s[w];
  const double whole = (euler ? us_e[w] : us_s[w]) * ((ninst + per - 1) / per);
  const double stages = euler ? 30.0 + 8e-5 * cells + 9e-3 * ninst : 18.0 + 3.5e-5 * cells + 4e-3 * ninst;
  return whole <= stages;
}

// Threads per tile where neither the caller nor the tuner has chosen: narrow tiles pack short instances
// better (a tile yields six cells less than it has threads), but every tile of an instance takes the maximum
// of its speeds to one address, 12 ns each in turn.  us a step with 64 / 128 / 256 threads, Euler: 4096
// instances of 256 cells 133 / 174 / 236; 512 of 512 45 / 49 / 68; 2000 of 1100 221 / 236 / 242; 512 of 2048
// 122 / 110 / 118; 64 of 4096 72 / 50 / 50; one of 262144 178 / 98 / 64.  Burgers: 4096 of 256 65 / 77 / 95; 1024 of
// 1000 62 / 58 / 57; 300 of 4096 107 / 71 / 60.
extern "C" int hw_tile1d_default(int eq, int ninst, long cells, int maxn) {
  const bool euler = eq == hw::EQ_EULER;
  if (maxn <= 4096 && cells <= (euler ? 1100L : 600L) * ninst) return 64;
  return euler && maxn <= 16384 ? 128 : 256;
}

template <int EQ>
static hipError_t launch_step1d(int threads, int ninst, const hw::Stage1D* P, const hw::Step1D* Q, int nsteps,
                                hipStream_t s) {
  const dim3 g(ninst), b(threads);
  switch (threads) {
    case 128: hipLaunchKernelGGL((hw::step1d_kernel<EQ, 128>), g, b, 0, s, *P, *Q, nsteps); break;
    case 256: hipLaunchKernelGGL((hw::step1d_kernel<EQ, 256>), g, b, 0, s, *P, *Q, nsteps); break;
    case 512: hipLaunchKernelGGL((hw::step1d_kernel<EQ, 512>), g, b, 0, s, *P, *Q, nsteps); break;
    case 1024: hipLaunchKernelGGL((hw::step1d_kernel<EQ, 1024>), g, b, 0, s, *P, *Q, nsteps); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

extern "C" hipError_t hw_launch_step1d(int eq, int threads, int ninst, const hw::Stage1D* P,
                                       const hw::Step1D* Q, int nsteps, hipStream_t s) {
  if (P->nu) return hipErrorInvalidValue;
  if (eq == hw::EQ_EULER) return launch_step1d<hw::EQ_EULER>(threads, ninst, P, Q, nsteps, s);
  if (eq == hw::EQ_BURGERS) return launch_step1d<hw::EQ_BURGERS>(threads, ninst, P, Q, nsteps, s);
  if (eq == hw::EQ_ADV) return launch_step1d<hw::EQ_ADV>(threads, ninst, P, Q, nsteps, s);
  return hipErrorInvalidValue;
}

extern "C" hipError_t hw_launch_alpha1d(int eq, const double* U, const int* off, int ninst,
                                        int total, int maxn, double gam, double adv,
                                        unsigned long long* alpha_out, hipStream_t s) {
  int bx = (maxn + 255) / 256;
  if (bx > 64) bx = 64;
  dim3 g(bx, ninst), b(256);
  if (eq == hw::EQ_EULER)
    hipLaunchKernelGGL(hw::alpha1d_kernel<hw::EQ_EULER>, g, b, 0, s, U, off, total, gam, adv, alpha_out);
  else if (eq == hw::EQ_BURGERS)
    hipLaunchKernelGGL(hw::alpha1d_kernel<hw::EQ_BURGERS>, g, b, 0, s, U, off, total, gam, adv, alpha_out);
  else
    hipLaunchKernelGGL(hw::alpha1d_kernel<hw::EQ_ADV>, g, b, 0, s, U, off, total, gam, adv, alpha_out);
  return hipGetLastError();
}

extern "C" hipError_t hw_launch_mesh1d_setup(const double* faces, int n, int bc, double* tab,
                                             hipStream_t s) {
  hipLaunchKernelGGL(hw::mesh1d::mesh1d_setup_kernel, dim3((n + 255) / 256), dim3(256), 0, s,
                     faces, n, bc, tab, (size_t)n, 0);
  return hipGetLastError();
}

extern "C" hipError_t hw_launch_mesh1d_setup_batch(const double* faces, const int* off, int ninst,
                                                   int bc, double* tab, int total, hipStream_t s) {
  for (int b = 0; b < ninst; ++b) {
    const int n = off[b + 1] - off[b];
    // instance b's faces follow those of the instances before it (n + 1 each)
    hipLaunchKernelGGL(hw::mesh1d::mesh1d_setup_kernel, dim3((n + 255) / 256), dim3(256), 0, s,
                       faces + off[b] + b, n, bc, tab, (size_t)total, off[b]);
  }
  return hipGetLastError();
}
