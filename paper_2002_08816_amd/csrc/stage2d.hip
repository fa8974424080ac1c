// Two-dimensional stage of the hybrid Hermite WENO scheme (Zhao & Qiu, arXiv 2002.08816,
// Section 2.2, Steps 4-6 and eq. ode2).  Per Runge-Kutta stage, with troubled-cell
// detection on, four launches:
//
//  stage2d_flags  per 16 x 16 tile: KXRCF flags (Step 4, Remark 3) of tile+1 from the
//                 fields the indicator reads; writes the tile's flags and hybrid masks
//                 (a flag in the 3 x 3 block, Step 5) and appends its flagged cells and
//                 its hybrid cells to two work lists.
//  stage2d_limit  the Jacobi limiter of the first moments (Step 4, Remark 4) over the
//                 flagged-cell list, one (cell, direction, characteristic field) per thread.
//  stage2d_hweno  the HWENO edge values (Step 5.1) over the hybrid-cell list, one
//                 (cell, direction, characteristic field) per thread.  Work lists rather
//                 than tiles: the few tiles a shock crosses would otherwise each run their
//                 whole share on one compute unit.
//  stage2d_kernel per 16 x 16 tile with two ghost layers (flags, hybrid masks and
//                 limited moments read back): interior Gauss values of the least-squares quartic -> volume
//                 integrals (Step 5.3); the edge values of the cell (Step 5.2 linear, or the
//                 stored HWENO values), its shares of its four faces' Lax-Friedrichs fluxes and
//                 the edge quadratures of eq. ode2; the TVD-RK3 stage combination (eq. RK) with the
//                 limited moments, the store, and the block's share of the next stage's
//                 speeds.  Each cell evaluates its own edge values and flux shares once; its
//                 neighbours' shares, summed over the edge's Gauss points, come through LDS,
//                 those across the tile's sides from the ring cells the tile evaluates once.
// Without detection only stage2d_kernel runs.  Small rectangular meshes with detection take
// one launch per stage, stage2d_fused_kernel.
//
// The limited first moments of the stage input replace the stored ones in the stage
// combination; the flags and limited moments of u^n (stage 1) are kept for stages 2, 3.
// Ghost cells at transmissive and reflective boundaries are mirror images of the cells
// they copy in every respect (state, flag, hybrid mask, limited moments, edge values); a
// reflective wall also reverses the normal momentum.
#include "hw_dmr.h"
#include "hw_step.h"
#include "hw_tile2d.h"

namespace hw {

// ------------------------------------------------------------------ prepasses
constexpr int H2 = 2, L2 = TX + 2 * H2, NP2 = L2 * L2;   // tile + two ghost layers

// global index of the cell a distance-1 transmissive or reflective ghost mirrors (other
// indices as given)
__device__ __forceinline__ int mirror1(int g, int n, int bc) {
  if (bc == BC_PERIODIC) return g;
  if (g == -1) return 0;
  if (g == n) return n - 1;
  return g;
}

// Factor a reflective wall adds to every value of component c of a ghost cell, on top of
// the mirror's moment signs: the normal momentum (rho u across an x wall, rho v across a y
// wall) is reversed.  xm / ym: the cell is a mirror image across an x / y boundary.
template <int EQ>
__device__ __forceinline__ double wall_factor(int c, bool xm, bool ym, int bcx, int bcy) {
  if constexpr (EQ != EQ_EULER) return 1.0;
  double f = 1.0;
  if (c == 1 && xm && bcx == BC_REFLECTIVE) f = -f;
  if (c == 2 && ym && (bcy == BC_REFLECTIVE || bcy == BC_DMR)) f = -f;
  return f;
}

// double Mach reflection: whether the stencil position (gx, gy) is a prescribed ghost cell,
// and the value of its field f at the stage's time ts.  BK: the boundary kind the kernel
// instance is for (BK_RECT, BK_DMR, BK_STEP); only the instances of the double Mach
// reflection and the forward step carry their boundaries' code.
template <int BK>
__device__ __forceinline__ bool dmr_prescribed(const Stage2D& P, int gx, int gy) {
  if constexpr (BK == BK_DMR) return dmr::prescribed(gx, gy, P.nx, P.ny, P.x0, P.dx);
  return false;
}
// The prescribed ghosts' moments are computed once per stage (dmr_table_kernel) into a
// table over the ring of two ghost layers around the mesh (dmr::ring2_index).
// value of field f of the prescribed ghost (gx, gy) at the stage's time
__device__ __forceinline__ double dmr_value(const Stage2D& P, int f, int gx, int gy, double) {
  return P.dtab[(size_t)f * dmr::ring2_size(P.nx, P.ny) + dmr::ring2_index(gx, gy, P.nx, P.ny)];
}
template <int BK>
__device__ __forceinline__ double stage_time_of(const Stage2D& P, double dtv) {
  if constexpr (BK == BK_DMR) return dmr::stage_time(P.t, dtv, P.mode);
  return 0.0;
}

// Appends the threads marked in a to list a and those marked in b to list b, with one
// atomic per list and workgroup (workgroups with nothing to append touch no counter).
__device__ __forceinline__ void block_append2(bool ma, bool mb, int value, int* counts,
                                              int* list_a, int* list_b,
                                              int* s_wave /* 10 ints */) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long a = __ballot(ma), b = __ballot(mb);
  if (lane == 0) {
    s_wave[w] = __popcll(a);
    s_wave[4 + w] = __popcll(b);
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int* sw = s_wave + 4 * threadIdx.x;
    const int tot = sw[0] + sw[1] + sw[2] + sw[3];
    s_wave[8 + threadIdx.x] = tot ? atomicAdd(&counts[threadIdx.x], tot) : 0;
  }
  __syncthreads();
  const unsigned long long below = (1ull << lane) - 1ull;
  if (ma) {
    int off = s_wave[8];
    for (int i = 0; i < w; ++i) off += s_wave[i];
    list_a[off + __popcll(a & below)] = value;
  }
  if (mb) {
    int off = s_wave[9];
    for (int i = 0; i < w; ++i) off += s_wave[4 + i];
    list_b[off + __popcll(b & below)] = value;
  }
}

// the flag of one fluid cell of the forward step's mesh, from memory
template <int EQ>
__device__ __forceinline__ uint8_t step_flag(const Stage2D& P, int gx, int gy) {
  constexpr int NC = 4;
  if (P.tc_mode == TC_ALL) return 1;
  const size_t plane = (size_t)P.nx * P.ny, g0 = (size_t)gy * P.nx + gx;
  const double velx = P.in[plane + g0] / P.in[g0], vely = P.in[2 * plane + g0] / P.in[g0];
  uint8_t t = 0;
  for (int c = 0; c < NC; c += NC - 1) {   // density, then energy
    double v[5][3];
    for (int k = 0; k < 5; ++k) {   // the cell, its left, right, lower and upper neighbours
      const step::Src r = step::resolve(gx + (k == 2) - (k == 1), gy + (k == 4) - (k == 3), P.nx, P.ny, P.si, P.sj);
      const size_t g = (size_t)r.y * P.nx + r.x;
      v[k][0] = r.pres ? P.uin[c] : P.in[c * plane + g];
      v[k][1] = r.pres ? 0.0 : r.sx * P.in[(NC + c) * plane + g];
      v[k][2] = r.pres ? 0.0 : r.sy * P.in[(2 * NC + c) * plane + g];
    }
    if (kxrcf2d(v[0], v[1], v[2], v[3], v[4], velx, vely, P.dx, P.dy, P.h)) t = 1;
  }
  return t;
}

// KXRCF flags of every cell (Step 4, Remark 3; Euler: density or energy fires).  Each
// tile stages only what the indicator reads, with two ghost layers, and evaluates the
// flags of tile+1 so that it also knows its hybrid cells (a flag in the 3 x 3 block,
// Step 5); transmissive ghosts take the flag of the cell they mirror.  The tile's flags
// and hybrid masks are stored, and its flagged and hybrid cells appended to two work
// lists.
template <int EQ, int BK>
__global__ __launch_bounds__(NT) void stage2d_flags_kernel(Stage2D P) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  constexpr int NK = (EQ == EQ_EULER) ? 2 : 1;   // components checked: density, energy
  constexpr int NV = (EQ == EQ_EULER) ? 2 : 0;   // momentum averages (velocity)
  constexpr int NFK = 3 * NK;                    // averages and moments of those
  constexpr int W1 = L2 - 2;                     // tile+1
  __shared__ double s_k[NFK * NP2];
  __shared__ uint8_t s_vs[NP2];                  // Euler: inflow sides (velocity signs)
  __shared__ uint8_t s_T[NP2];
  __shared__ int s_wave[10];

  // zero once the run has reached its final time (nothing to do); checked after the loads
  // of the tile are issued (the pointer is valid in every mode)
  const double dtv = *P.dt;
  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  int bx, by;
  tile_of_block(nx, bx, by);
  const int gx0 = bx * TX - H2, gy0 = by * TY - H2;
  const size_t plane = (size_t)nx * ny;
  // staging: each thread's (at most NR) positions, every load issued before the stores
  constexpr int NR = (NP2 + NT - 1) / NT;
  double kv[NR][NFK + NV];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = tid + r * NT;
    if (q < NP2) {
      const int ly = q / L2, lx = q - ly * L2;
      double sx, sy;
      size_t gs;
      if constexpr (BK == BK_STEP) {
        // forward step: the position's source cell, or the inflow state
        const step::Src sr = step::resolve(gx0 + lx, gy0 + ly, nx, ny, P.si, P.sj);
        if (sr.pres) {
#pragma unroll
          for (int k = 0; k < NK; ++k) {
            kv[r][3 * k] = P.uin[k == 0 ? 0 : NC - 1];
            kv[r][3 * k + 1] = kv[r][3 * k + 2] = 0.0;
          }
#pragma unroll
          for (int k = 0; k < NV; ++k) kv[r][NFK + k] = P.uin[1 + k];
          continue;
        }
        sx = sr.sx;
        sy = sr.sy;
        gs = (size_t)sr.y * nx + sr.x;
      } else {
        const int gx = map_index(gx0 + lx, nx, P.bcx, sx);
        const int gy = map_index(gy0 + ly, ny, P.bcy, sy);
        gs = (size_t)gy * nx + gx;
      }
      if (dmr_prescribed<BK>(P, gx0 + lx, gy0 + ly)) {
        const double ts = stage_time_of<BK>(P, dtv);
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          const int c = k == 0 ? 0 : NC - 1;
#pragma unroll
          for (int m = 0; m < 3; ++m) kv[r][3 * k + m] = dmr_value(P, m * NC + c, gx0 + lx, gy0 + ly, ts);
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) kv[r][NFK + k] = dmr_value(P, 1 + k, gx0 + lx, gy0 + ly, ts);
        continue;
      }
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const int c = k == 0 ? 0 : NC - 1;
        kv[r][3 * k] = P.in[c * plane + gs];
        kv[r][3 * k + 1] = sx * P.in[(NC + c) * plane + gs];
        kv[r][3 * k + 2] = sy * P.in[(2 * NC + c) * plane + gs];
      }
#pragma unroll
      for (int k = 0; k < NV; ++k) kv[r][NFK + k] = P.in[(1 + k) * plane + gs];
    }
  }
  if (P.mode != MODE_L && dtv == 0.0) return;   // uniform over the grid
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int q = tid + r * NT;
    if (q < NP2) {
#pragma unroll
      for (int f = 0; f < NFK; ++f) s_k[f * NP2 + q] = kv[r][f];
      if constexpr (EQ == EQ_EULER) {
        // velocity (rho u)/rho, (rho v)/rho at the average: which faces are inflow
        const double velx = kv[r][NFK] / kv[r][0], vely = kv[r][NFK + 1] / kv[r][0];
        s_vs[q] = (uint8_t)((velx > 0.0) | ((velx < 0.0) << 1) | ((vely > 0.0) << 2) |
                            ((vely < 0.0) << 3));
      }
    }
  }
  __syncthreads();
  auto K = [&](int f, int y, int x) { return s_k[f * NP2 + y * L2 + x]; };
  for (int q = tid; q < W1 * W1; q += NT) {
    const int ly = 1 + q / W1, lx = 1 + q % W1;
    uint8_t t = 0;
    if (P.tc_mode == TC_ALL) {
      t = 1;
    } else {
      bool lin, rin, bin, tin;
      if constexpr (EQ == EQ_EULER) {
        const unsigned vs = s_vs[ly * L2 + lx];
        lin = vs & 1u; rin = vs & 2u; bin = vs & 4u; tin = vs & 8u;
      } else {
        const double velx = EQ == EQ_BURGERS ? K(0, ly, lx) : P.adv0;
        const double vely = EQ == EQ_BURGERS ? K(0, ly, lx) : P.adv1;
        lin = velx > 0.0; rin = velx < 0.0; bin = vely > 0.0; tin = vely < 0.0;
      }
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        double cc[3], l[3], r[3], b[3], tt[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          cc[m] = K(3 * k + m, ly, lx);
          l[m] = K(3 * k + m, ly, lx - 1);
          r[m] = K(3 * k + m, ly, lx + 1);
          b[m] = K(3 * k + m, ly - 1, lx);
          tt[m] = K(3 * k + m, ly + 1, lx);
        }
        if (kxrcf2d_in(cc, l, r, b, tt, lin, rin, bin, tin, P.dx, P.dy, P.h)) t = 1;
      }
    }
    s_T[ly * L2 + lx] = t;
  }
  __syncthreads();
  if (P.bcx != BC_PERIODIC || P.bcy != BC_PERIODIC) {
    // ghosts take the flag of the cell they mirror; prescribed ghosts are never troubled
    uint8_t tg[(W1 * W1 + NT - 1) / NT];
#pragma unroll
    for (int r = 0; r < (W1 * W1 + NT - 1) / NT; ++r) {
      const int q = tid + r * NT;
      if (q >= W1 * W1) break;
      const int ly = 1 + q / W1, lx = 1 + q % W1;
      if constexpr (BK == BK_STEP) {
        // the flag of the source cell; a source outside tile+1 only belongs to a position
        // that no tile cell's 3 x 3 block holds, but for the step's corner cell, whose
        // source lies across the corner
        const step::Src sr = step::resolve(gx0 + lx, gy0 + ly, nx, ny, P.si, P.sj);
        const int mx = sr.x - gx0, my = sr.y - gy0;
        tg[r] = 0;
        if (!sr.pres && mx >= 1 && mx <= W1 && my >= 1 && my <= W1) tg[r] = s_T[my * L2 + mx];
        else if (gx0 + lx == P.si && gy0 + ly == P.sj - 1) tg[r] = step_flag<EQ>(P, sr.x, sr.y);
      } else {
        const int mx = mirror1(gx0 + lx, nx, P.bcx) - gx0, my = mirror1(gy0 + ly, ny, P.bcy) - gy0;
        tg[r] = dmr_prescribed<BK>(P, gx0 + lx, gy0 + ly) ? 0 : s_T[my * L2 + mx];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < (W1 * W1 + NT - 1) / NT; ++r) {
      const int q = tid + r * NT;
      if (q >= W1 * W1) break;
      const int ly = 1 + q / W1, lx = 1 + q % W1;
      s_T[ly * L2 + lx] = tg[r];
    }
    __syncthreads();
  }
  const int tx = tid % TX, ty = tid / TX;
  const int lx = tx + H2, ly = ty + H2;
  const int gx = gx0 + lx, gy = gy0 + ly;
  const bool inmesh = gx < nx && gy < ny;
  // solid cells of the forward step are never flagged
  bool active = inmesh;
  if constexpr (BK == BK_STEP) active = inmesh && !step::solid(gx, gy, P.si, P.sj);
  const int gi = inmesh ? gy * nx + gx : 0;
  uint8_t t = s_T[ly * L2 + lx];
  uint8_t hm = 0;
  for (int dy = -1; dy <= 1; ++dy)
    for (int dx = -1; dx <= 1; ++dx) hm |= s_T[(ly + dy) * L2 + lx + dx];
  if (!active) t = hm = 0;
  if (inmesh) {
    P.Tcur[gi] = t;
    P.Hcur[gi] = hm;
  }
  block_append2(active && t, active && hm, gi, P.counts, P.flist, P.hlist, s_wave);
}

// Value of field f at the cell (gy, gx) + (dy, dx) as the stencil of that cell sees it:
// boundary mapping (transmissive ghosts negate their normal moment), and the limited
// first moment where the cell is flagged.
template <int BK>
__device__ __forceinline__ double stencil_value(const Stage2D& P, int f, int NC, int gy, int gx,
                                                int dy, int dx, bool limited, double ts) {
  if (dmr_prescribed<BK>(P, gx + dx, gy + dy)) return dmr_value(P, f, gx + dx, gy + dy, ts);
  if constexpr (BK == BK_STEP) {
    const step::Src sr = step::resolve(gx + dx, gy + dy, P.nx, P.ny, P.si, P.sj);
    const int m = f / NC, c = f % NC;
    if (sr.pres) return m == 0 ? P.uin[c] : 0.0;
    const size_t plane = (size_t)P.nx * P.ny, g = (size_t)sr.y * P.nx + sr.x;
    const double wf = step::comp_factor(sr, c);
    if (m == 0) return wf * P.in[f * plane + g];
    const double v = (limited && P.Tcur[g]) ? P.limcur[(f - NC) * plane + g] : P.in[f * plane + g];
    return wf * (m == 1 ? sr.sx * v : sr.sy * v);
  }
  double sx, sy;
  const int x = map_index(gx + dx, P.nx, P.bcx, sx);
  const int y = map_index(gy + dy, P.ny, P.bcy, sy);
  const size_t plane = (size_t)P.nx * P.ny, g = (size_t)y * P.nx + x;
  const int m = f / NC;
  const double wf = NC == 4 ? wall_factor<EQ_EULER>(f % NC, sx < 0.0, sy < 0.0, P.bcx, P.bcy) : 1.0;
  if (m == 0) return wf * P.in[f * plane + g];
  const double v = (limited && P.Tcur[g]) ? P.limcur[(f - NC) * plane + g] : P.in[f * plane + g];
  return wf * (m == 1 ? sx * v : sy * v);
}

// Jacobi limiter of the first moments of every flagged cell (Step 4, Remark 4): one work
// item per (cell, direction, characteristic field).  For Euler the four items of one
// (cell, direction) sit on four consecutive lanes; lane f reads component f of the
// stencil, the group exchanges the components to project onto its characteristic
// fields, and exchanges the limited fields to return to component f.
template <int EQ, int BK>
__global__ __launch_bounds__(NT) void stage2d_limit_kernel(Stage2D P) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  const long long n = (long long)P.counts[0] * 2 * NC;   // whole groups of NC items
  const double dtv = *P.dt;   // loaded together with the list length
  if ((P.mode != MODE_L && dtv == 0.0) || n == 0) return;
  const int lane = threadIdx.x & 63;
  const size_t plane = (size_t)P.nx * P.ny;
  for (long long base = (long long)blockIdx.x * NT + threadIdx.x - lane; base < n;
       base += (long long)gridDim.x * NT) {
    const long long it = base + lane;
    if (it >= n) continue;
    const int f = (int)(it % NC), dir = (int)((it / NC) & 1);
    const int gi = P.flist[(it / NC) >> 1];
    const int gy = gi / P.nx, gx = gi - gy * P.nx;
    const int oy = dir, ox = 1 - dir, mf = 1 + dir;
    // component f of the stencil along dir (unlimited values)
    const double ts = stage_time_of<BK>(P, dtv);
    const double um = stencil_value<BK>(P, f, NC, gy, gx, -oy, -ox, false, ts);
    const double u0 = P.in[f * plane + gi];
    const double up = stencil_value<BK>(P, f, NC, gy, gx, oy, ox, false, ts);
    const double vm = stencil_value<BK>(P, mf * NC + f, NC, gy, gx, -oy, -ox, false, ts);
    const double vp = stencil_value<BK>(P, mf * NC + f, NC, gy, gx, oy, ox, false, ts);
    if constexpr (EQ == EQ_EULER) {
      double U[4], Lr[4], Rr[4], x[4];
      quad_gather(u0, U);
      euler_rows2d(U, P.gam, dir, f, Lr, Rr);
      double cm = 0.0, c0 = 0.0, cp = 0.0, wm = 0.0, wp = 0.0;
      quad_gather(um, x);
#pragma unroll
      for (int c = 0; c < 4; ++c) cm = fma(Lr[c], x[c], cm);
#pragma unroll
      for (int c = 0; c < 4; ++c) c0 = fma(Lr[c], U[c], c0);
      quad_gather(up, x);
#pragma unroll
      for (int c = 0; c < 4; ++c) cp = fma(Lr[c], x[c], cp);
      quad_gather(vm, x);
#pragma unroll
      for (int c = 0; c < 4; ++c) wm = fma(Lr[c], x[c], wm);
      quad_gather(vp, x);
#pragma unroll
      for (int c = 0; c < 4; ++c) wp = fma(Lr[c], x[c], wp);
      const double vc = limit_moment(cm, c0, cp, wm, wp, P.w.lim, P.w.eps);
      quad_gather(vc, x);
      double out = 0.0;
#pragma unroll
      for (int g = 0; g < 4; ++g) out = fma(Rr[g], x[g], out);
      P.limcur[(size_t)(dir * 4 + f) * plane + gi] = out;
    } else {
      P.limcur[(size_t)dir * plane + gi] = limit_moment(um, u0, up, vm, vp, P.w.lim, P.w.eps);
    }
  }
}

// component f of one half of a hybrid cell's 19-value stencil (through the cache, with the
// limited moments of flagged cells), value k to s[64 k]: HALF 0 the nine averages, HALF 1 the ten
// first moments of the cross.  The stored values and the flags are loaded together, the limited
// moments of the (few) flagged cells afterwards.
template <int EQ, int BK, int HALF>
__device__ __forceinline__ void hweno_load(const Stage2D& P, int gi, int f, double dtv, double* s) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1, N = HALF == 0 ? 9 : 5;
  const size_t plane = (size_t)P.nx * P.ny;
  const int gy = gi / P.nx, gx = gi - gy * P.nx;
  const int cross[5] = {1, 3, 4, 5, 7};
  // the positions: stored index, moment signs (mirrored ghosts), prescribed or not
  int gb[N];
  unsigned neg_x = 0, neg_y = 0, neg_w = 0, pres = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int k = HALF == 0 ? j : cross[j];
    if constexpr (BK == BK_STEP) {
      // forward step: the position's source cell (prescribed: the inflow state, below)
      const step::Src sr = step::resolve(gx + k % 3 - 1, gy + k / 3 - 1, P.nx, P.ny, P.si, P.sj);
      gb[j] = sr.y * P.nx + sr.x;
      if (sr.pres) pres |= 1u << j;
      if (sr.sx < 0.0) neg_x |= 1u << j;
      if (sr.sy < 0.0) neg_y |= 1u << j;
      if (step::comp_factor(sr, f) < 0.0) neg_w |= 1u << j;
    } else {
      double sx, sy;
      const int x = map_index(gx + k % 3 - 1, P.nx, P.bcx, sx);
      const int y = map_index(gy + k / 3 - 1, P.ny, P.bcy, sy);
      gb[j] = y * P.nx + x;
      if (sx < 0.0) neg_x |= 1u << j;
      if (sy < 0.0) neg_y |= 1u << j;
      // a reflective wall also reverses the normal momentum of its ghost cells
      if (wall_factor<EQ>(f, sx < 0.0, sy < 0.0, P.bcx, P.bcy) < 0.0) neg_w |= 1u << j;
      // double Mach reflection: prescribed ghosts hold the exact solution (the signs apply to
      // mirrored ghosts only) and are never troubled
      if (dmr_prescribed<BK>(P, gx + k % 3 - 1, gy + k / 3 - 1)) pres |= 1u << j;
    }
  }
  auto value = [&](int m, int j, double v) {   // moment m at position j, prescribed or as stored
    if (!((pres >> j) & 1u)) return ((m == 0 ? neg_w : (m == 1 ? neg_x ^ neg_w : neg_y ^ neg_w)) >> j) & 1u ? -v : v;
    if constexpr (BK == BK_STEP) return m == 0 ? P.uin[f] : 0.0;   // inflow state, zero moments
    if constexpr (BK == BK_DMR) {
      const int k = HALF == 0 ? j : cross[j];
      return dmr_value(P, m * NC + f, gx + k % 3 - 1, gy + k / 3 - 1, stage_time_of<BK>(P, dtv));
    }
    return v;
  };
  if constexpr (HALF == 0) {
    double u[N];
#pragma unroll
    for (int j = 0; j < N; ++j) u[j] = P.in[f * plane + gb[j]];
#pragma unroll
    for (int j = 0; j < N; ++j) s[j * 64] = value(0, j, u[j]);
  } else {
    double v[N], w[N];
    uint8_t t[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      t[j] = P.Tcur[gb[j]];
      v[j] = P.in[(NC + f) * plane + gb[j]];
      w[j] = P.in[(2 * NC + f) * plane + gb[j]];
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (t[j]) {
        v[j] = P.limcur[f * plane + gb[j]];
        w[j] = P.limcur[(NC + f) * plane + gb[j]];
      }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      s[(9 + j) * 64] = value(1, j, v[j]);
      s[(14 + j) * 64] = value(2, j, w[j]);
    }
  }
}

// the edge values of direction DIR of one hybrid cell (lane: field and component f of it, as in
// the limiter) from the stencils in s_x ([19][64])
template <int EQ, int NGE, int DIR>
__device__ __forceinline__ void hweno_list_values(const Stage2D& P, const double* s_x, int lane, int f, double* v) {
  if constexpr (EQ == EQ_EULER) {
    const double* s = s_x + (lane & ~3);   // the cell's four components
    double U[4], Lr[4], Rr[4], x[4], w19[19], wv[2 * NGE];
#pragma unroll
    for (int c = 0; c < 4; ++c) U[c] = s[4 * 64 + c];
    euler_rows2d(U, P.gam, DIR, f, Lr, Rr);
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      double a = 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) a = fma(Lr[c], s[k * 64 + c], a);
      w19[k] = a;
    }
    hweno2d_field<NGE>(w19, P.w, DIR, wv);
#pragma unroll
    for (int k = 0; k < 2 * NGE; ++k) {
      quad_gather(wv[k], x);
      double a = 0.0;
#pragma unroll
      for (int g = 0; g < 4; ++g) a = fma(Rr[g], x[g], a);
      v[k] = a;
    }
  } else {
    double in[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) in[k] = s_x[k * 64 + lane];
    hweno2d_field<NGE>(in, P.w, DIR, v);
  }
}

// HWENO edge values (Step 5.1) of every hybrid cell, one work item per (cell, direction,
// characteristic field), grouped as in the limiter.  The pass waits on its scattered loads and on the
// length of a wave's chain, so the waves of a workgroup form pairs: both waves of a pair take
// the same 64 / NC cells, each loads half of their stencils into LDS, and each reconstructs one
// direction.  Measured against one wave that loaded a cell's whole stencil, passed its components
// round by lane moves and took the directions in turn (236 to 248 VGPRs), us a launch: 15.4 -> 13.6 on
// the forward step at 960 x 320, 14.4 -> 10.9 at 480 x 160, 19.7 -> 15.6 at 1501 x 997, the mean of a
// run 19.7 -> 18.9 at 1024^2 and 25.4 -> 23.4 on the double Mach reflection at 1920 x 480.
template <int EQ, int NGE, int BK>
__global__ __launch_bounds__(NT, 2) void stage2d_hweno_kernel(Stage2D P) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  constexpr int CPW = 64 / NC, NPAIR = NT / 128;   // cells per wave, pairs
  __shared__ double s_x[NPAIR][19 * 64];
  // the list length and the time step are loaded together (the time step pointer is valid
  // in every mode); a finished run or an empty list has nothing to do
  const int ncell = P.counts[1];
  const double dtv = *P.dt;
  if ((P.mode != MODE_L && dtv == 0.0) || ncell == 0) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, pr = wv >> 1, dir = wv & 1, f = lane % NC;
  const size_t plane = (size_t)P.nx * P.ny;
  // the loop's bounds are the workgroup's, so every wave meets both barriers
  for (long long base = (long long)blockIdx.x * NPAIR * CPW; base < ncell;
       base += (long long)gridDim.x * NPAIR * CPW) {
    const long long cell = base + pr * CPW + lane / NC;
    const bool on = cell < ncell;   // whole groups of NC lanes
    const int gi = on ? P.hlist[cell] : 0;
    if (on) {
      if (dir == 0) hweno_load<EQ, BK, 0>(P, gi, f, dtv, s_x[pr] + lane);
      else hweno_load<EQ, BK, 1>(P, gi, f, dtv, s_x[pr] + lane);
    }
    __syncthreads();
    if (on) {
      double v[2 * NGE];
      if (dir == 0) hweno_list_values<EQ, NGE, 0>(P, s_x[pr], lane, f, v);
      else hweno_list_values<EQ, NGE, 1>(P, s_x[pr], lane, f, v);
#pragma unroll
      for (int k = 0; k < NGE; ++k) {
        P.G[((((size_t)(dir * 2 + 0) * NGE + k) * NC + f)) * plane + gi] = v[k];
        P.G[((((size_t)(dir * 2 + 1) * NGE + k) * NC + f)) * plane + gi] = v[NGE + k];
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ main stage kernel

// The 19 stencil values of component c around (ly, lx) as seen along the direction dir of
// each lane: for dir = 1 the stencil is transposed (x and y offsets swapped, x and y moments
// swapped), so that the y-face values are the x-face map of the transposed stencil.  The
// fold of these values (with lin2d_fold_oo0_T) equals lin2d_transpose of the untransposed fold
// to the bit, so a cell's trace is the same whether the cell itself or a neighbouring tile
// evaluates it.
template <int NC, int W>
__device__ __forceinline__ void gather19_dir(const double* s, int c, int ly, int lx, int dir,
                                             double* in) {
  const int sa = dir == 0 ? W : 1, sb = dir == 0 ? 1 : W;   // strides of dy, dx
  const double* p = s + c * W * W + ly * W + lx;
#pragma unroll
  for (int k = 0; k < 9; ++k) in[k] = p[(k / 3 - 1) * sa + (k % 3 - 1) * sb];
  const double* pv = p + (dir == 0 ? NC : 2 * NC) * W * W;   // moment along dir
  const double* pw = p + (dir == 0 ? 2 * NC : NC) * W * W;   // the other moment
  const int cy[5] = {-1, 0, 0, 0, 1}, cx[5] = {0, -1, 0, 1, 0};
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    in[9 + j] = pv[cy[j] * sa + cx[j] * sb];
    in[14 + j] = pw[cy[j] * sa + cx[j] * sb];
  }
}

// The HWENO edge values the prepass stored (Step 5.1) for the hybrid cell at LDS position
// (ly, lx) on its face of direction dir and side (0 low, 1 high).  A ghost's are those of
// the cell it mirrors, faces and edge points reflected.
template <int EQ, int NGE, int BK>
__device__ __forceinline__ void stored_trace(const Stage2D& P, int ly, int lx, int dir, int side,
                                             int gx0, int gy0, double (*v)[NGE]) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  double sx, sy, fu = 1.0, fv = 1.0;
  int gx, gy;
  if constexpr (BK == BK_STEP) {
    const step::Src sr = step::resolve(gx0 + lx, gy0 + ly, P.nx, P.ny, P.si, P.sj);
    gx = sr.x;
    gy = sr.y;
    sx = sr.sx;
    sy = sr.sy;
    fu = sr.fu;
    fv = sr.fv;
  } else {
    gx = map_index(gx0 + lx, P.nx, P.bcx, sx);
    gy = map_index(gy0 + ly, P.ny, P.bcy, sy);
  }
  const bool mx = sx < 0.0, my = sy < 0.0;
  const bool swap = dir == 0 ? mx : my, flip = dir == 0 ? my : mx;
  const size_t plane = (size_t)P.nx * P.ny, gi = (size_t)gy * P.nx + gx;
  const int s = swap ? 1 - side : side;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    double wf;
    if constexpr (BK == BK_STEP) wf = c == 1 ? fu : (c == 2 ? fv : 1.0);
    else wf = wall_factor<EQ>(c, mx, my, P.bcx, P.bcy);
#pragma unroll
    for (int k = 0; k < NGE; ++k) {
      const int kk = flip ? NGE - 1 - k : k;
      v[c][k] = wf * P.G[((((size_t)(dir * 2 + s) * NGE + kk) * NC + c)) * plane + gi];
    }
  }
}

// One side's share f(U) + s U of twice the Lax-Friedrichs flux f(u-) + f(u+) - alpha (u+ - u-)
// at a point: s = alpha for the low cell's trace u-, -alpha for the high cell's u+.  The flux
// is a sum of one term per side, so each cell evaluates its own two sides once and its
// neighbours add theirs: half the point fluxes of a form in which both cells of a face
// evaluate all of it.  (D: direction; adv: the advection speed along it)
template <int EQ, int D>
__device__ __forceinline__ void flux_share(const double* U, double s, double gam, double adv, double* F) {
  if constexpr (EQ == EQ_EULER) {
    constexpr int n = 1 + D, t = 2 - D;   // normal and tangential momentum
    const double r = rcp_nr(U[0]);
    const double un = U[n] * r;
    const double p = (gam - 1.0) * (U[3] - 0.5 * (U[n] * un + U[t] * (U[t] * r)));
    const double us = un + s;
    F[0] = fma(s, U[0], U[n]);
    F[n] = fma(U[n], us, p);
    F[t] = U[t] * us;
    F[3] = fma(U[3], us, p * un);
  } else {
    F[0] = fma(s, U[0], scalar_flux<EQ>(U[0], adv));
  }
}

// Twice the flux's sums over a face's Gauss points enter the right-hand sides only through
// S0 = sum w_k F_k and S1 = sum w_k e_k F_k (both linear in the shares, so neighbours
// exchange two sums instead of NGE point values).  Returned up to the factors C0, C1.
template <int NGE>
struct FaceSums;
template <>
struct FaceSums<2> {
  static constexpr double C0 = 0.5, C1 = 0.5 * 0.28867513459481288225457439025097873;
};
template <>
struct FaceSums<3> {
  static constexpr double C0 = 4.0 / 9.0, C1 = (5.0 / 18.0) * 0.38729833462074168851792653997823996;
};
template <int EQ, int NGE, int D>
__device__ __forceinline__ void face_sums(const double (*tr)[NGE], double s, double gam, double adv,
                                          double* S /* [2][NC] */) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  double F[NGE][NC];
#pragma unroll
  for (int k = 0; k < NGE; ++k) {
    double U[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) U[c] = tr[c][k];
    flux_share<EQ, D>(U, s, gam, adv, F[k]);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if constexpr (NGE == 2) S[c] = F[0][c] + F[1][c];
    else S[c] = fma(0.625, F[0][c] + F[2][c], F[1][c]);
    S[NC + c] = F[NGE - 1][c] - F[0][c];
  }
}

// Faces whose other side follows a boundary's face rule instead of a neighbour's values: the
// forward step's inflow, outflow and walls.  Returns
// 0 (none), 1 (the low face) or 2 (the high face) in the low two bits and above them which
// of the direction's (at most three) such grid lines it is; that side's share sums go to
// entry 16 * line + (position along the line) of s_spec, [sum][NC][64].  (Held in registers
// until the exchange they would not fit beside the traces.)
template <int EQ, int NGE, int BK, int D>
__device__ __forceinline__ int special_face(const Stage2D& P, int gx, int gy, int along,
                                            const double (*lo)[NGE], const double (*hi)[NGE],
                                            double alpha, double* s_spec) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  int which = 0, line = 0;
  double u[NC][NGE];
  if constexpr (BK == BK_STEP) {
    // the inflow state on the left side; at the bottom wall and the step's top face the
    // cell's own trace with rho v reversed
    if (D == 0 ? gx == 0 : (gy == 0 || (gy == P.sj && gx >= P.si))) {
      which = 1;
      line = (D == 1 && gy != 0) ? 1 : 0;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < NGE; ++k) u[c][k] = D == 0 ? P.uin[c] : (c == 2 ? -lo[c][k] : lo[c][k]);
    }
    // the outflow takes the cell's own trace; the step's left face (rho u) and the top wall
    // (rho v) reverse the normal momentum
    if (D == 0 ? (gx == P.nx - 1 || (gx == P.si - 1 && gy < P.sj)) : gy == P.ny - 1) {
      which = 2;
      line = (D == 0 && gx != P.nx - 1) ? 1 : 2;
      const int cn = D == 0 ? (gx == P.nx - 1 ? -1 : 1) : 2;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < NGE; ++k) u[c][k] = c == cn ? -hi[c][k] : hi[c][k];
    }
  }
  if (which) {
    double S[2 * NC];
    face_sums<EQ, NGE, D>(u, which == 1 ? alpha : -alpha, P.gam, 0.0, S);
#pragma unroll
    for (int v = 0; v < 2 * NC; ++v) s_spec[v * 64 + line * 16 + along] = S[v];
  }
  return which | (line << 2);
}

// (1/dx) sum w f(u(G)) and (1/dy) sum w g(u(G)) without the factors 1/dx, 1/dy: the volume
// quadrature over the 3 x 3 interior Gauss points.  The rule is exact for the quartic, so
// the parts of f and g that are linear in u are the cell averages ub themselves.
template <int EQ>
__device__ __forceinline__ void volume_sums(const double (*inner)[9], const double* ub, const Stage2D& P,
                                            double* sf, double* sg) {
  if constexpr (EQ == EQ_EULER) {
    double muu = 0.0, muv = 0.0, mvv = 0.0, mp = 0.0, hu = 0.0, hv = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const double w = VW[q % 3] * VW[q / 3];
      const double m = inner[1][q], n = inner[2][q], E = inner[3][q];
      const double r = rcp_nr(inner[0][q]);
      const double u = m * r, v = n * r;
      const double a = m * u, b = n * v;
      const double p = (P.gam - 1.0) * (E - 0.5 * (a + b));
      const double H = E + p;
      muu = fma(w, a, muu);
      muv = fma(w, n * u, muv);
      mvv = fma(w, b, mvv);
      mp = fma(w, p, mp);
      hu = fma(w, u * H, hu);
      hv = fma(w, v * H, hv);
    }
    sf[0] = ub[1];
    sf[1] = muu + mp;
    sf[2] = muv;
    sf[3] = hu;
    sg[0] = ub[2];
    sg[1] = muv;
    sg[2] = mvv + mp;
    sg[3] = hv;
  } else if constexpr (EQ == EQ_BURGERS) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) s = fma(0.5 * VW[q % 3] * VW[q / 3], inner[0][q] * inner[0][q], s);
    sf[0] = sg[0] = s;
  } else {
    sf[0] = P.adv0 * ub[0];
    sg[0] = P.adv1 * ub[0];
  }
}

// whether the position (gx, gy) lies beyond a transmissive or reflective side
__device__ __forceinline__ bool mirrored(const Stage2D& P, int gx, int gy) {
  return (P.bcx != BC_PERIODIC && (gx < 0 || gx >= P.nx)) || (P.bcy != BC_PERIODIC && (gy < 0 || gy >= P.ny));
}

// LDS of a stage tile beside the staged input
template <int EQ, int NGE, int BK>
struct TileShared {
  static constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  static constexpr int NV = 4 * NC;   // exchanged per direction: [side: high, low][sum][NC]
  static constexpr int NSPEC = BK == BK_STEP ? 2 * NC * 64 : 0;
  double ring[2 * NC * 64];           // ring cells' share sums [sum][NC][ring cell]
  double spec[2 * NSPEC + 1];         // boundary face rules' share sums, per direction
  double red[8];
  double alpha[2];
};

// The stage of one tile from its staged (limited) input s_u, rows of W = TX + 2 HB positions
// with HB ghost layers, and the flags and hybrid masks s_T, s_H of the same positions; the
// space of s_u is reused.  s_rtr: when not null, the HWENO values of hybrid ring cells that are
// no mirror images, [NC][NGE][ring cell]; the tile's own hybrid cells' (and the mirror
// images') are then those this workgroup stored in P.G before the call.
// TH = 2 NT threads: the waves of the second half work on the same cells as those of the first
// and take the ring cells and the y direction's traces over from them.
template <int EQ, int NGE, int BK, int HB, int TH = NT>
__device__ __forceinline__ void stage_tile(const Stage2D& P, TileShared<EQ, NGE, BK>& sh, double* s_u,
                                           const uint8_t* s_T, const uint8_t* s_H,
                                           const double* s_rtr, int bx, int by, double dtv) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  constexpr int NF = 3 * NC, W = TX + 2 * HB;
  constexpr int NV = TileShared<EQ, NGE, BK>::NV;
  constexpr int NSPEC = TileShared<EQ, NGE, BK>::NSPEC;
  static_assert((NT / 64) * NV * 64 <= NF * W * W, "the exchange fits the staged input's space");
  double* const s_ring = sh.ring;
  double* const s_spec = sh.spec;
  double* const s_red = sh.red;
  const double* const s_alpha = sh.alpha;
  constexpr bool HELP = TH > NT;
  static_assert(TH == NT || (TH == 2 * NT && BK == BK_RECT), "one or two threads per cell");
  const bool main = !HELP || threadIdx.x < NT;
  const int mode = P.mode, tid = threadIdx.x % NT, nx = P.nx, ny = P.ny;
  const double dt = mode != MODE_L ? dtv : 0.0;
  const int gx0 = bx * TX - HB, gy0 = by * TY - HB;
  const size_t plane = (size_t)nx * ny;
  const bool tc = P.tc_mode != TC_NONE;
  // the tile's mesh cells (fewer in the last column and row of tiles)
  const int tw = min(TX, nx - bx * TX), th = min(TY, ny - by * TY);

  const int tx = tid % TX, ty = tid / TX;
  const int lx = tx + HB, ly = ty + HB;
  const int gx = gx0 + lx, gy = gy0 + ly;
  const bool inmesh = gx < nx && gy < ny;
  // the solid cells of the forward step are never updated
  bool active = inmesh;
  if constexpr (BK == BK_STEP) active = inmesh && !step::solid(gx, gy, P.si, P.sj);
  const size_t gi = active ? (size_t)gy * nx + gx : 0;
  const int lane = tid & 63, wv = tid >> 6;

  // out = a W(u^n) + b (W(u^(s)) + dt L) with (a, b) of the stage (eq. RK): acc starts with
  // the first two terms, and every part of L is added with the factor b dt.  The operator
  // alone: a = b = 0 and the factor 1.
  double ca, cb;
  rk_coeffs(mode, ca, cb);
  const double cdt = mode == MODE_L ? 1.0 : cb * dt;
  if (mode == MODE_L) cb = 0.0;
  // stages 2 and 3: W(u^n), loaded now and used after the volume quadrature
  double Wn[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) Wn[f] = 0.0;
  if ((mode == MODE_RK2 || mode == MODE_RK3) && active && main) {
    const bool tn = tc && P.Tn[gi] != 0;
#pragma unroll
    for (int f = 0; f < NF; ++f) Wn[f] = P.base[(size_t)f * plane + gi];
    if (tn) {
#pragma unroll
      for (int f = NC; f < NF; ++f) Wn[f] = P.limn[(size_t)(f - NC) * plane + gi];
    }
  }

  double acc[NF];
  if (main) {
    double inner[NC][9], ub[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      double in[19], f[hw2::NFOLD];
      gather19<NC, W>(s_u, c, ly, lx, in);
      ub[c] = in[4];
      acc[c] = cb * in[4];
      acc[NC + c] = cb * in[11];
      acc[2 * NC + c] = cb * in[16];
      hw2::lin2d_fold(in, f);
      hw2::lin2d_inner(f, inner[c]);
      __builtin_amdgcn_sched_barrier(0);
    }
    double sf[NC], sg[NC];
    volume_sums<EQ>(inner, ub, P, sf, sg);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      acc[c] = fma(ca, Wn[c], acc[c]);
      acc[NC + c] = fma(cdt * P.idx, sf[c], fma(ca, Wn[NC + c], acc[NC + c]));
      acc[2 * NC + c] = fma(cdt * P.idy, sg[c], fma(ca, Wn[2 * NC + c], acc[2 * NC + c]));
    }
    // formed here: left to itself the compiler sinks this phase to the stores, holding the
    // interior values in scratch until then
#pragma unroll
    for (int f = 0; f < NF; ++f) asm volatile("" : "+v"(acc[f]));
  }
  if (mode == MODE_L && P.wout && active && main) {
#pragma unroll
    for (int f = 0; f < NF; ++f) P.wout[(size_t)f * plane + gi] = S<W>(s_u, f, ly, lx);
  }

  if (s_rtr) __syncthreads();   // the workgroup's HWENO values are in place
  // ring cells (the tile's neighbours across the four sides of its mesh cells), all 64 by
  // the first wave (of the helpers): lanes
  // 32 d .. 32 d + 31 those of direction d, the low side's high faces and the high side's
  // low faces
  if (wv == 0 && (!HELP || !main)) {
    const int rd = lane / (2 * TX), rs = (lane / TX) & 1, rp = lane % TX;
    const int rly = rd == 0 ? HB + rp : (rs == 0 ? HB - 1 : HB + th);
    const int rlx = rd == 0 ? (rs == 0 ? HB - 1 : HB + tw) : HB + rp;
    double a[NC][NGE];
    if (s_H[rly * W + rlx] == 0) {
      const double side = rs == 0 ? 1.0 : -1.0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        double in[19], f[hw2::NFOLD], p[6];
        gather19_dir<NC, W>(s_u, c, rly, rlx, rd, in);
        hw2::lin2d_fold(in, f);
        if (rd == 1) f[12] = hw2::lin2d_fold_oo0_T(in);
        lin_xparts<NGE>(f, p);
        lin_xface<NGE>(p, side, a[c]);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else if (s_rtr && !mirrored(P, gx0 + rlx, gy0 + rly)) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int k = 0; k < NGE; ++k) a[c][k] = s_rtr[(c * NGE + k) * 64 + lane];
    } else {
      stored_trace<EQ, NGE, BK>(P, rly, rlx, rd, rs == 0 ? 1 : 0, gx0, gy0, a);
    }
    if constexpr (BK == BK_DMR) {
      if (dmr_prescribed<BK>(P, gx0 + rlx, gy0 + rly)) {
        // the face shared with the tile: the ring cell's high face (rs = 0) or low face
        const double ts = stage_time_of<BK>(P, dtv);
        const int gxr = gx0 + rlx, gyr = gy0 + rly;
#pragma unroll
        for (int k = 0; k < NGE; ++k) {
          const double e = Gauss<NGE>::node[k];
          double x, y, U[4];
          if (rd == 0) {
            x = P.x0 + (gxr + (rs == 0 ? 1.0 : 0.0)) * P.dx;
            y = P.y0 + (gyr + 0.5 + e) * P.dy;
          } else {
            x = P.x0 + (gxr + 0.5 + e) * P.dx;
            y = P.y0 + (gyr + (rs == 0 ? 1.0 : 0.0)) * P.dy;
          }
          dmr::point_state(x, y, ts, P.gam, U);
#pragma unroll
          for (int c = 0; c < NC; ++c) a[c][k] = U[c];
        }
      }
    }
    // both directions as x fluxes: the momenta exchanged for y
    if constexpr (EQ == EQ_EULER) {
#pragma unroll
      for (int k = 0; k < NGE; ++k) {
        const double m = a[1][k], n = a[2][k];
        a[1][k] = rd == 0 ? m : n;
        a[2][k] = rd == 0 ? n : m;
      }
    }
    double S[2 * NC];
    const double al = s_alpha[rd];
    face_sums<EQ, NGE, 0>(a, rs == 0 ? al : -al, P.gam, rd == 0 ? P.adv0 : P.adv1, S);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int cc = (c == 0 || c == 3) ? c : (rd == 0 ? c : 3 - c);
        s_ring[(j * NC + cc) * 64 + lane] = S[j * NC + c];
      }
  }

  // ---------------------------------------------------------------- traces and share sums
  // the cell's traces on its four faces (p0, or the stored HWENO values of a hybrid cell)
  // and, per direction, the sums of its shares: E[dir][0] its high face's (u- there),
  // E[dir][1] its low face's (u+ there)
  // the stencils are gathered again (kept from the volume phase they would take 120 VGPRs):
  // the row is made opaque so that the compiler does not keep them
  int ly2 = ly;
  asm volatile("" : "+v"(ly2));
  const bool hyb = active && s_H[ly * W + lx] != 0;
  const double al0 = s_alpha[0], al1 = s_alpha[1];
  double E[2][2][2 * NC];
  int sp[2] = {0, 0};
  if constexpr (HELP) {
    // x by the first half, y by the second
    auto traces = [&](auto D) {
      constexpr int dir = decltype(D)::value;
      double tl[NC][NGE], th[NC][NGE];
      if (!hyb) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double in[19], f[hw2::NFOLD];
          gather19<NC, W>(s_u, c, ly2, lx, in);
          hw2::lin2d_fold(in, f);
          lin_faces<NGE>(f, dir, tl[c], th[c]);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        stored_trace<EQ, NGE, BK>(P, ly, lx, dir, 0, gx0, gy0, tl);
        stored_trace<EQ, NGE, BK>(P, ly, lx, dir, 1, gx0, gy0, th);
      }
      const double al = dir == 0 ? al0 : al1, adv = dir == 0 ? P.adv0 : P.adv1;
      face_sums<EQ, NGE, dir>(th, al, P.gam, adv, E[dir][0]);
      face_sums<EQ, NGE, dir>(tl, -al, P.gam, adv, E[dir][1]);
    };
    if (main) traces(std::integral_constant<int, 0>());
    else traces(std::integral_constant<int, 1>());
  } else if constexpr (NGE == 2) {
    // both directions from one gather
    double xl[NC][NGE], xh[NC][NGE], yl[NC][NGE], yh[NC][NGE];
    if (!hyb) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        double in[19], f[hw2::NFOLD];
        gather19<NC, W>(s_u, c, ly2, lx, in);
        hw2::lin2d_fold(in, f);
        lin_faces<NGE>(f, 0, xl[c], xh[c]);
        lin_faces<NGE>(f, 1, yl[c], yh[c]);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      stored_trace<EQ, NGE, BK>(P, ly, lx, 0, 0, gx0, gy0, xl);
      stored_trace<EQ, NGE, BK>(P, ly, lx, 0, 1, gx0, gy0, xh);
      stored_trace<EQ, NGE, BK>(P, ly, lx, 1, 0, gx0, gy0, yl);
      stored_trace<EQ, NGE, BK>(P, ly, lx, 1, 1, gx0, gy0, yh);
    }
    if constexpr (BK == BK_STEP) {
      sp[0] = special_face<EQ, NGE, BK, 0>(P, gx, gy, ty, xl, xh, al0, s_spec);
      sp[1] = special_face<EQ, NGE, BK, 1>(P, gx, gy, tx, yl, yh, al1, s_spec + NSPEC);
    }
    face_sums<EQ, NGE, 0>(xh, al0, P.gam, P.adv0, E[0][0]);
    face_sums<EQ, NGE, 0>(xl, -al0, P.gam, P.adv0, E[0][1]);
    face_sums<EQ, NGE, 1>(yh, al1, P.gam, P.adv1, E[1][0]);
    face_sums<EQ, NGE, 1>(yl, -al1, P.gam, P.adv1, E[1][1]);
  } else {
    // three points per edge: one direction at a time (96 VGPRs of traces otherwise)
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      double tl[NC][NGE], th[NC][NGE];
      asm volatile("" : "+v"(ly2));
      if (!hyb) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double in[19], f[hw2::NFOLD];
          gather19<NC, W>(s_u, c, ly2, lx, in);
          hw2::lin2d_fold(in, f);
          lin_faces<NGE>(f, dir, tl[c], th[c]);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        stored_trace<EQ, NGE, BK>(P, ly, lx, dir, 0, gx0, gy0, tl);
        stored_trace<EQ, NGE, BK>(P, ly, lx, dir, 1, gx0, gy0, th);
      }
      if (dir == 0) {
        if constexpr (BK == BK_STEP) sp[0] = special_face<EQ, NGE, BK, 0>(P, gx, gy, ty, tl, th, al0, s_spec);
        face_sums<EQ, NGE, 0>(th, al0, P.gam, P.adv0, E[0][0]);
        face_sums<EQ, NGE, 0>(tl, -al0, P.gam, P.adv0, E[0][1]);
      } else {
        if constexpr (BK == BK_STEP) sp[1] = special_face<EQ, NGE, BK, 1>(P, gx, gy, tx, tl, th, al1, s_spec + NSPEC);
        face_sums<EQ, NGE, 1>(th, al1, P.gam, P.adv1, E[1][0]);
        face_sums<EQ, NGE, 1>(tl, -al1, P.gam, P.adv1, E[1][1]);
      }
#pragma unroll
      for (int v = 0; v < 2 * NC; ++v) asm volatile("" : "+v"(E[dir][0][v]), "+v"(E[dir][1][v]));
    }
  }
  __syncthreads();   // the staged input is done with: its space holds the exchange

  // ---------------------------------------------------------------- exchange and faces
  // a cell's two faces of each direction: its own share sums plus the neighbour's, read from
  // the wave's own block (x; y inside the wave's four rows), the neighbouring wave's block,
  // or the ring.  Both cells of a face add the same two values.
  double* const own_blk = s_u + wv * NV * 64 + lane;
#pragma unroll
  for (int dir = 0; dir < 2; ++dir) {
    if (HELP && dir == 1) __syncthreads();   // the x sums are read: the helpers' y sums go there
    if (!HELP || main == (dir == 0)) {
#pragma unroll
      for (int v = 0; v < 2 * NC; ++v) {
        own_blk[v * 64] = E[dir][0][v];
        own_blk[(2 * NC + v) * 64] = E[dir][1][v];
      }
    }
    if (HELP && dir == 1) __syncthreads();
    if (HELP && !main) continue;
    if (HELP && dir == 1) {
#pragma unroll
      for (int v = 0; v < 2 * NC; ++v) {
        E[1][0][v] = own_blk[v * 64];
        E[1][1][v] = own_blk[(2 * NC + v) * 64];
      }
    }
    const double *lo, *hi;   // the low neighbour's high-face sums, the high neighbour's low-face sums
    if (dir == 0) {
      // x neighbours share the wave: its LDS operations stay in order, no barrier
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      lo = tx == 0 ? s_ring + ty : own_blk - 1;
      hi = tx == tw - 1 ? s_ring + TX + ty : own_blk + 2 * NC * 64 + 1;
    } else {
      if (!HELP) __syncthreads();
      lo = (ty & 3) != 0 ? own_blk - TX : (wv == 0 ? s_ring + 2 * TX + tx : own_blk - NV * 64 + 48);
      hi = ty == th - 1 ? s_ring + 3 * TX + tx
                        : ((ty & 3) != 3 ? own_blk + 2 * NC * 64 + TX : own_blk + (NV + 2 * NC) * 64 - 48);
    }
    if (!inmesh) lo = hi = s_ring;   // (nothing is stored for this lane)
    const double k = cdt * (dir == 0 ? P.idx : P.idy);
    const double kU = -0.5 * FaceSums<NGE>::C0 * k, kP = 0.5 * kU, kQ = -0.5 * FaceSums<NGE>::C1 * k;
    const int fP = dir == 0 ? NC : 2 * NC, fQ = dir == 0 ? 2 * NC : NC;
    if constexpr (BK == BK_STEP) {
      const double* spec = s_spec + dir * NSPEC + (sp[dir] >> 2) * 16 + (dir == 0 ? ty : tx);
      if ((sp[dir] & 3) == 1) lo = spec;
      if ((sp[dir] & 3) == 2) hi = spec;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double L0 = lo[c * 64] + E[dir][1][c], R0 = E[dir][0][c] + hi[c * 64];
      const double L1 = lo[(NC + c) * 64] + E[dir][1][NC + c], R1 = E[dir][0][NC + c] + hi[(NC + c) * 64];
      acc[c] = fma(kU, R0 - L0, acc[c]);
      acc[fP + c] = fma(kP, L0 + R0, acc[fP + c]);
      acc[fQ + c] = fma(kQ, R1 - L1, acc[fQ + c]);
    }
    if (dir == 0) {
      // the block is written again for y once every lane of the wave has read it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }

  // ---------------------------------------------------------------- epilogue
  double sp0 = 0.0, sp1 = 0.0;
  if constexpr (BK == BK_STEP) {
    // solid cells: no flags; the operator alone reports zero and the stored state
    if (inmesh && !active) {
      const size_t gs = (size_t)gy * nx + gx;
      if (P.flagsT) P.flagsT[gs] = 0;
      if (P.flagsH) P.flagsH[gs] = 0;
      if (mode == MODE_L) {
#pragma unroll
        for (int f = 0; f < NF; ++f) P.out[(size_t)f * plane + gs] = 0.0;
        if (P.wout) {
#pragma unroll
          for (int f = 0; f < NF; ++f) P.wout[(size_t)f * plane + gs] = P.in[(size_t)f * plane + gs];
        }
      }
    }
  }
  if (active && main) {
    if (P.flagsT) P.flagsT[gi] = s_T[ly * W + lx];
    if (P.flagsH) P.flagsH[gi] = s_H[ly * W + lx];
#pragma unroll
    for (int f = 0; f < NF; ++f) P.out[(size_t)f * plane + gi] = acc[f];
    if (mode != MODE_L) {
      int bad = 0;
#pragma unroll
      for (int f = 0; f < NF; ++f)
        if (!isfinite(acc[f])) bad |= 1;
      if constexpr (EQ == EQ_EULER) {
        double p;
        euler_speeds2d(acc, P.gam, sp0, sp1, p);
        if (!(acc[0] > 0.0) || !(p > 0.0)) bad |= 2;
      } else if constexpr (EQ == EQ_BURGERS) {
        sp0 = sp1 = fabs(acc[0]);
      } else {
        sp0 = fabs(P.adv0);
        sp1 = fabs(P.adv1);
      }
      if (bad) atomicOr(P.status, bad);
    }
  }
  if (mode != MODE_L) {
    // block maxima of both directions with one barrier
    const double w0 = wave_max(sp0), w1 = wave_max(sp1);
    if (lane == 0 && main) {
      s_red[wv] = w0;
      s_red[4 + wv] = w1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const double m0 = fmax(fmax(s_red[0], s_red[1]), fmax(s_red[2], s_red[3]));
      const double m1 = fmax(fmax(s_red[4], s_red[5]), fmax(s_red[6], s_red[7]));
      const int e = blockIdx.x % ASPREAD;
      atomic_max_pos(&P.alpha_out[e], m0);
      atomic_max_pos(&P.alpha_out[ASPREAD + e], m1);
    }
  }
}

// Bound by VALU issue, then by LDS and HBM (1024^2 Euler, NG = 2: 308 MB of HBM traffic a
// launch, about 50 us; the instructions about 45 us; the phases overlap only in part), so the
// arithmetic per cell is what counts: one fold of a stencil serves all its point values of a
// gather, a flux is evaluated once per trace instead of once per cell of the face, and only
// sums over the edge's points are exchanged.  Measured against a form that gathered three
// times, evaluated each face's flux in both of its cells and exchanged point values by lane
// shuffles: 121 -> 96 us at 1024^2 NG = 2; 248 -> 155 us at 1501 x 997 NG = 3, where the smaller
// exchange also lets three workgroups run per CU instead of two; 162 -> 101 us on the double
// Mach reflection at 1920 x 480; 63 -> 40 us on the forward step at 960 x 320.  168 VGPRs and
// 43-52 KB of LDS: three workgroups per CU (the forward step's instance keeps 7 values in scratch at
// NG = 2, the double Mach reflection's one at NG = 3).
template <int EQ, int NGE, int BK>
__global__ __launch_bounds__(NT, 3) void stage2d_kernel(Stage2D P) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  constexpr int NF = 3 * NC;
  __shared__ double s_u[NF * NP2];   // stage input, limited, on tile+2; then the exchange
  __shared__ uint8_t s_T[NP2];
  __shared__ uint8_t s_H[NP2];
  __shared__ TileShared<EQ, NGE, BK> sh;

  const int mode = P.mode;
  // the time step (zero once the run has reached its final time: nothing to do) is
  // checked after the stage input's loads are issued
  const double dtv = *P.dt;   // (valid in every mode)
  const double dt = mode != MODE_L ? dtv : 0.0;
  const int tid = threadIdx.x;
  const int nx = P.nx, ny = P.ny;
  int bx, by;
  tile_of_block(nx, bx, by);
  const int gx0 = bx * TX - H2, gy0 = by * TY - H2;
  const size_t plane = (size_t)nx * ny;
  const bool tc = P.tc_mode != TC_NONE;

  // ---------------------------------------------------------------- stage input -> LDS
  // flagged cells take the prepass's limited first moments; ghosts mirror their cell
  // each thread's (at most NR) positions: flags and stored values are loaded first, the
  // limited moments of the (few) flagged cells replace the moments afterwards
  constexpr int NR = (NP2 + NT - 1) / NT;
  // a tile whose staged positions are all mesh cells needs no boundary mapping: offsets from
  // the tile's corner, below 2^32 bytes for rows of at most 2^24 cells
  bool inside = gx0 >= 0 && gy0 >= 0 && gx0 + L2 <= nx && gy0 + L2 <= ny && nx <= (1 << 24);
  if constexpr (BK == BK_STEP) inside = inside && (gx0 + L2 <= P.si || gy0 >= P.sj);
  if (inside) {
    const size_t corner = (size_t)gy0 * nx + gx0;
    double v[NR][NF];
    uint32_t off[NR];
    uint8_t tr[NR], hr[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = tid + r * NT;
      tr[r] = hr[r] = 0;
      if (q < NP2) {
        const int ly = q / L2, lx = q - ly * L2;
        off[r] = (uint32_t)(ly * nx + lx);
        if (tc) {
          tr[r] = (P.Tcur + corner)[off[r]];
          hr[r] = (P.Hcur + corner)[off[r]];
        }
#pragma unroll
        for (int f = 0; f < NF; ++f)
          v[r][f] = *(const double*)((const char*)(P.in + (f * plane + corner)) + off[r] * 8u);
      }
    }
    if (mode != MODE_L && dt == 0.0) return;   // uniform over the grid
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = tid + r * NT;
      if (q < NP2) {
        if (tr[r]) {
#pragma unroll
          for (int f = NC; f < NF; ++f) v[r][f] = (P.limcur + ((f - NC) * plane + corner))[off[r]];
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) s_u[f * NP2 + q] = v[r][f];
        s_T[q] = tr[r];
        s_H[q] = hr[r];
      }
    }
  } else {
    size_t gsr[NR];
    double sxr[NR], syr[NR];
    uint8_t tr[NR], hr[NR];
    uint8_t fwr[NR];   // forward step: bit 0 rho u, bit 1 rho v reversed
    double v[NR][NF];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = tid + r * NT;
      tr[r] = 0;
      hr[r] = 0;
      fwr[r] = 0;
      if (q < NP2) {
        const int ly = q / L2, lx = q - ly * L2;
        int gx, gy;
        if constexpr (BK == BK_STEP) {
          const step::Src sr = step::resolve(gx0 + lx, gy0 + ly, nx, ny, P.si, P.sj);
          gx = sr.x;
          gy = sr.y;
          sxr[r] = sr.sx;
          syr[r] = sr.sy;
          fwr[r] = (sr.fu < 0.0 ? 1 : 0) | (sr.fv < 0.0 ? 2 : 0);
          if (sr.pres) {
            // inflow: the prescribed state, zero first moments, never troubled
            gsr[r] = 0;
#pragma unroll
            for (int f = 0; f < NF; ++f) v[r][f] = f < NC ? P.uin[f] : 0.0;
            continue;
          }
        } else {
          gx = map_index(gx0 + lx, nx, P.bcx, sxr[r]);
          gy = map_index(gy0 + ly, ny, P.bcy, syr[r]);
        }
        gsr[r] = (size_t)gy * nx + gx;
        if (dmr_prescribed<BK>(P, gx0 + lx, gy0 + ly)) {
          // prescribed ghost: the exact solution, never troubled, no mirror signs
          const double ts = stage_time_of<BK>(P, dtv);
#pragma unroll
          for (int f = 0; f < NF; ++f) v[r][f] = dmr_value(P, f, gx0 + lx, gy0 + ly, ts);
          sxr[r] = syr[r] = 1.0;
          continue;
        }
        if (tc) {
          tr[r] = P.Tcur[gsr[r]];
          hr[r] = P.Hcur[gsr[r]];   // a ghost's mask is that of the cell it mirrors
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) v[r][f] = P.in[f * plane + gsr[r]];
      }
    }
    if (mode != MODE_L && dt == 0.0) return;   // uniform over the grid
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = tid + r * NT;
      if (q < NP2) {
        if (tr[r]) {
#pragma unroll
          for (int f = NC; f < NF; ++f) v[r][f] = P.limcur[(f - NC) * plane + gsr[r]];
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const int m = f / NC, c = f % NC;
          double wf;
          if constexpr (BK == BK_STEP) wf = ((c == 1 && (fwr[r] & 1)) || (c == 2 && (fwr[r] & 2))) ? -1.0 : 1.0;
          else wf = wall_factor<EQ>(c, sxr[r] < 0.0, syr[r] < 0.0, P.bcx, P.bcy);
          s_u[f * NP2 + q] = wf * (m == 1 ? sxr[r] * v[r][f] : (m == 2 ? syr[r] * v[r][f] : v[r][f]));
        }
        s_T[q] = tr[r];
        s_H[q] = hr[r];
      }
    }
  }
  // this stage's prepasses are done: record the list lengths, empty the lists for the next
  // stage
  if (tc && blockIdx.x == 0 && tid == 0) {
    const int st = mode == MODE_L ? 0 : mode - MODE_RK1;
    P.stats[st] = P.counts[0];
    P.stats[3 + st] = P.counts[1];
    P.counts[0] = 0;
    P.counts[1] = 0;
  }
  reduce_speeds(P.alpha_in, sh.alpha);   // visible after the staging barrier
  __syncthreads();

  stage_tile<EQ, NGE, BK, H2>(P, sh, s_u, s_T, s_H, nullptr, bx, by, dtv);
}

// ------------------------------------------------------------------ one-launch stage
// A whole stage of a small rectangular mesh in one launch.  Where the tiles do not fill the
// chip, the four launches of a stage cost their latency (start-up, a round trip of the state
// and the lists through the L2s, the gap to the next launch: 30 us a stage on an 80 x 80 scalar
// mesh, 45 us on 256^2 Euler, whatever the launches compute), so each tile recomputes on idle
// units what it needs of its surroundings: the flags of tile+2 from three staged ghost
// layers, the limited moments of the flagged cells among them, the HWENO edge values of the
// hybrid cells of the tile and its ring.  The arithmetic is that of the four kernels.  Results
// that outlast the stage (flags, masks, limited moments and edge values of the tile's own
// cells, the list lengths, on request the lists) are stored as there.
// Such stages run a step by themselves (Stage2D's sdt): a launch that only sets the time step,
// clears the speeds and advances the time costs its latency and a gap, 3 of 45 us a step at 80^2.
// With at most one tile per compute unit (256 tiles) a tile has two threads per cell: one wave
// per SIMD cannot hide the latency of its own chains.  The second half of the waves takes its share
// of the staging, the flags and the lists, and the ring cells and y traces of the tile phase.
// Measured, us a stage, one thread per cell -> two: Euler NG 2 with shocks 32.2 -> 25.8 at 256^2,
// 27.6 -> 21.6 at 64 x 48; smooth Euler NG 3 15.7 -> 14.1 at 160^2; Burgers NG 3 13.0 -> 11.2 at 80^2.
// With more tiles than units the larger workgroup (172 VGPRs: one at a time on a unit) loses: us a
// step, two threads / one, 131.7 / 129.3 at 288^2 and 133.4 / 125.9 at 320^2 Euler NG 2 with shocks, 102.8 / 84.0
// at 288^2 smooth Euler NG 3, 62.0 / 47.0 at 288^2 advection.
// The rule (one_launch below): at most 400 tiles for Euler, 1600 for scalar laws.  Measured,
// us per step of three stages, one launch against four: Euler with shocks NG 2 105 / 136 at 256^2,
// 126 / 152 at 320^2 (400 tiles), 159 / 160 at 362^2 (529), 208 / 200 at 512^2, NG 3 138 / 153, 172 / 170
// and 235 / 215 at the last three: there two workgroups per CU (79 KB of LDS) run several rounds,
// and the tiles a shock crosses do all their HWENO cells themselves; smooth Euler NG 3 65 / 84 at
// 256^2, 87 / 111 at 320^2, 118 / 123 at 362^2, 217 / 205 at 640^2; Burgers NG 3 with shocks 54 / 97 at
// 256^2, 88 / 121 at 512^2, 103 / 126 at 640^2 (1600 tiles), 127 / 150 at 768^2; advection NG 2 71 / 81 at 512^2,
// 93 / 98 at 640^2, 107 / 114 at 768^2.
// Euler with every cell troubled: a full tile's own HWENO cells are then the stage's time, whatever
// the number of tiles, while four launches spread them over the chip.  One launch / four, us a step,
// NG 2 and NG 3: 87 / 79 and 94 / 86 at 13^2, 99 / 82 and 106 / 87 at 16^2, 101 / 88 and 108 / 94 at 64^2, 103 / 92
// and 111 / 102 at 90^2, 102 / 100 and 110 / 107 at 96^2 (36 tiles), but 103 / 102 and 112 / 114 at 99^2, 103 / 105 and
// 111 / 117 at 100^2; where the tiles are not full 76 / 77 and 81 / 83 at 9^2, 87 / 88 and 93 / 95 at 8 x 512.  Between,
// at 11^2 and 12^2, steps gain (84 / 78, 84 / 82) and a recorded run with its adjoint loses (12 steps 3730 / 3780 and
// 3740 / 3820 us; 3990 / 3790 at 16^2).  So four launches from 13 cells a side to 36 tiles.  A scalar law's
// cells are cheap enough: 37 / 65 at 32^2 and 64^2 Burgers NG 3.

// Appends the threads marked in m (of the workgroup's first four waves) to a work list (no list:
// counts only), the length kept in a 64-bit statistics entry: one atomic per workgroup that has
// something to append.
__device__ __forceinline__ void block_append_stat(bool m, int value, long long* count, int* list,
                                                  int* s_wave /* 6 ints */) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long a = __ballot(m);
  if (lane == 0 && w < NT / 64) s_wave[w] = __popcll(a);
  __syncthreads();
  const int tot = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
  if (!list) {   // uniform over the grid; the atomic's old value is not waited for
    if (threadIdx.x == 0 && tot) atomicAdd((unsigned long long*)count, (unsigned long long)tot);
    return;
  }
  if (threadIdx.x == 0 && tot)
    s_wave[4] = (int)atomicAdd((unsigned long long*)count, (unsigned long long)tot);
  __syncthreads();
  if (m) {
    int off = s_wave[4];
    for (int i = 0; i < w; ++i) off += s_wave[i];
    list[off + __popcll(a & ((1ull << lane) - 1ull))] = value;
  }
}

// characteristic HWENO edge values of direction DIR of the cell at LDS position (ly, lx): the
// Euler lane f projects the stencil onto field f with every component read from LDS (the four
// lanes of a cell read the same address, at less cost than passing their components round),
// reconstructs it, and returns component f of the values
template <int EQ, int NGE, int DIR>
__device__ __forceinline__ void hweno_values(const Stage2D& P, const double* s_u, int ly, int lx, int f,
                                             double* v) {
  if constexpr (EQ == EQ_EULER) {
    double U[4], Lr[4], Rr[4], x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) U[c] = S(s_u, c, ly, lx);   // the cell's own averages
    euler_rows2d(U, P.gam, DIR, f, Lr, Rr);
    double w19[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) w19[k] = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      double in[19];
      gather19<4>(s_u, c, ly, lx, in);
#pragma unroll
      for (int k = 0; k < 19; ++k) w19[k] = fma(Lr[c], in[k], w19[k]);
    }
    double wv[2 * NGE];
    hweno2d_field<NGE>(w19, P.w, DIR, wv);
#pragma unroll
    for (int k = 0; k < 2 * NGE; ++k) {
      quad_gather(wv[k], x);
      double a = 0.0;
#pragma unroll
      for (int g = 0; g < 4; ++g) a = fma(Rr[g], x[g], a);
      v[k] = a;
    }
  } else {
    double in[19];
    gather19<1>(s_u, 0, ly, lx, in);
    hweno2d_field<NGE>(in, P.w, DIR, v);
  }
}

// the limited first moment of direction dir of the cell at LDS position p (lanes as above):
// component f of the limited moment
template <int EQ>
__device__ __forceinline__ double limited_value(const Stage2D& P, const double* s_u, int p, int dir, int f) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  const int o = dir == 0 ? 1 : LX;
  const double* u = s_u + p;
  const double* w = s_u + (1 + dir) * NC * NPOS + p;   // the moment along dir
  if constexpr (EQ == EQ_EULER) {
    double U[4], Lr[4], Rr[4], x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) U[c] = u[c * NPOS];
    euler_rows2d(U, P.gam, dir, f, Lr, Rr);
    double cm = 0.0, c0 = 0.0, cp = 0.0, wm = 0.0, wp = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      cm = fma(Lr[c], u[c * NPOS - o], cm);
      c0 = fma(Lr[c], U[c], c0);
      cp = fma(Lr[c], u[c * NPOS + o], cp);
      wm = fma(Lr[c], w[c * NPOS - o], wm);
      wp = fma(Lr[c], w[c * NPOS + o], wp);
    }
    const double vc = limit_moment(cm, c0, cp, wm, wp, P.w.lim, P.w.eps);
    quad_gather(vc, x);
    double out = 0.0;
#pragma unroll
    for (int g = 0; g < 4; ++g) out = fma(Rr[g], x[g], out);
    return out;
  } else {
    return limit_moment(u[-o], u[0], u[o], w[-o], w[o], P.w.lim, P.w.eps);
  }
}

template <int EQ, int NGE, int TH>
__global__ __launch_bounds__(TH, 2) void stage2d_fused_kernel(Stage2D P) {
  constexpr int NC = (EQ == EQ_EULER) ? 4 : 1;
  constexpr int NF = 3 * NC;
  constexpr int NLIM = R2 * R2 * 2 * NC;         // limited moments of tile+2
  constexpr int NRTR = NC * NGE * 64;            // ring cells' HWENO values
  __shared__ double s_u[NF * NPOS];              // stage input on tile+3, limited on tile+2
  __shared__ double s_lim[NLIM > NRTR ? NLIM : NRTR];
  __shared__ uint8_t s_T[NPOS], s_H[NPOS];
  __shared__ uint16_t s_fl[R2 * R2], s_hl[NT + 64];
  __shared__ int s_cnt[2], s_wave[12];
  __shared__ TileShared<EQ, NGE, BK_RECT> sh;

  const int mode = P.mode, tid = threadIdx.x, nx = P.nx, ny = P.ny;
  const bool begin = mode == MODE_RK1 && P.sdt;   // this stage sets the time step
  double dtv = begin ? 1.0 : *P.dt;   // (valid in every mode; zero: the run has reached its final time)
  const double t0 = begin ? *P.st : 0.0;
  int bx, by;
  tile_of_block(nx, bx, by);
  const int gx0 = bx * TX - HL, gy0 = by * TY - HL;
  const size_t plane = (size_t)nx * ny;
  const int tw = min(TX, nx - bx * TX), th = min(TY, ny - by * TY);
  const int lane = tid & 63;

  // ---------------------------------------------------------------- stage input -> LDS
  {
    constexpr int NR = (NPOS + TH - 1) / TH;
    double v[NR][NF], sxr[NR], syr[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = tid + r * TH;
      if (q < NPOS) {
        const int ly = q / LX, lx = q - ly * LX;
        const int gx = map_index(gx0 + lx, nx, P.bcx, sxr[r]);
        const int gy = map_index(gy0 + ly, ny, P.bcy, syr[r]);
        const size_t gs = (size_t)gy * nx + gx;
#pragma unroll
        for (int f = 0; f < NF; ++f) v[r][f] = P.in[f * plane + gs];
      }
    }
    if (mode != MODE_L && dtv == 0.0) return;   // uniform over the grid
    if (tid < 2) s_cnt[tid] = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = tid + r * TH;
      if (q < NPOS) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          const int m = f / NC, c = f % NC;
          const double wf = wall_factor<EQ>(c, sxr[r] < 0.0, syr[r] < 0.0, P.bcx, P.bcy);
          s_u[f * NPOS + q] = wf * (m == 1 ? sxr[r] * v[r][f] : (m == 2 ? syr[r] * v[r][f] : v[r][f]));
        }
      }
    }
  }
  reduce_speeds(P.alpha_in, sh.alpha);
  __syncthreads();
  if (P.sdt) {   // (uniform over the grid)
    if (begin) {
      dtv = P.fixed_dt > 0.0 ? P.fixed_dt : P.cfl / (sh.alpha[0] / P.dx + sh.alpha[1] / P.dy);
      if (P.T_end > 0.0) {
        if (t0 >= P.T_end) dtv = 0.0;
        else if (t0 + dtv > P.T_end) dtv = P.T_end - t0;
      }
      if (blockIdx.x == 0 && tid == 0) *P.sdt = dtv;   // (read by the later stages)
      if (dtv == 0.0) return;   // uniform over the grid
    }
    if (blockIdx.x == 0) {
      if (mode == MODE_RK2 && tid == 0 && dtv > 0.0) {   // (no other stage reads these)
        *P.st += dtv;
        *P.ssteps += 1;
      }
      if (P.azero && tid < 2 * ASPREAD) P.azero[tid] = 0ull;
      if (P.pub && tid < 2) {
        const int e = 3 * tid + (mode + 2 - MODE_RK1) % 3;   // the stage before
        if (mode != MODE_RK1) P.pub[e] = P.stats[e];
        P.stats[e] = 0;
      }
    }
  }

  // ---------------------------------------------------------------- flags, masks, lists
  // flags of tile+2; a mirror image takes the flag of the cell it mirrors
  flags_tile<EQ, TH>(s_u, P.tc_mode, P.adv0, P.adv1, P.dx, P.dy, P.h, s_T);
  __syncthreads();
  const bool walls = P.bcx != BC_PERIODIC || P.bcy != BC_PERIODIC;
  // the LDS position of the cell a mirror image copies (-1: outside the staged block, which
  // only belongs to positions that no mesh cell's stencil holds)
  auto mirror_pos = [&](int ly, int lx, double& sx, double& sy) -> int {
    const int mx = map_index(gx0 + lx, nx, P.bcx == BC_PERIODIC ? BC_TRANSMISSIVE : P.bcx, sx) - gx0;
    const int my = map_index(gy0 + ly, ny, P.bcy == BC_PERIODIC ? BC_TRANSMISSIVE : P.bcy, sy) - gy0;
    // (a periodic direction wraps: the position itself holds the wrapped cell)
    const int px = P.bcx == BC_PERIODIC ? lx : mx, py = P.bcy == BC_PERIODIC ? ly : my;
    if (P.bcx == BC_PERIODIC) sx = 1.0;
    if (P.bcy == BC_PERIODIC) sy = 1.0;
    return (px < 1 || px >= LX - 1 || py < 1 || py >= LX - 1) ? -1 : py * LX + px;
  };
  if (walls) {
    for (int q = tid; q < R2 * R2; q += TH) {
      const int ly = 1 + q / R2, lx = 1 + q % R2;
      if (!mirrored(P, gx0 + lx, gy0 + ly)) continue;
      double sx, sy;
      const int m = mirror_pos(ly, lx, sx, sy);
      s_T[ly * LX + lx] = m >= 0 ? s_T[m] : 0;   // (the cell mirrored is no mirror image)
    }
    __syncthreads();
  }
  for (int q = tid; q < R2 * R2; q += TH) {
    const int ly = 1 + q / R2, lx = 1 + q % R2, p = ly * LX + lx;
    const bool own = !(walls && mirrored(P, gx0 + lx, gy0 + ly));
    if (own && s_T[p]) s_fl[atomicAdd(&s_cnt[0], 1)] = (uint16_t)p;
    if (ly < 2 || ly >= LX - 2 || lx < 2 || lx >= LX - 2) continue;
    // hybrid mask of tile+1; the tile's mesh cells and the ring's four sides go to the list
    uint8_t hm = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) hm |= s_T[p + (k / 3 - 1) * LX + k % 3 - 1];
    s_H[p] = hm;
    const int cx = lx - HL, cy = ly - HL;
    const bool inx = cx >= 0 && cx < tw, iny = cy >= 0 && cy < th;
    const bool wanted = (inx && iny) || (iny && (cx == -1 || cx == tw)) || (inx && (cy == -1 || cy == th));
    if (own && hm && wanted) s_hl[atomicAdd(&s_cnt[1], 1)] = (uint16_t)p;
  }
  __syncthreads();
  const int tx = tid % TX, ty = tid / TX;
  const bool inmesh = tx < tw && ty < th;   // (no cell for threads from NT on)
  const size_t gi = inmesh ? (size_t)(by * TY + ty) * nx + bx * TX + tx : 0;
  {
    const int p = (ty + HL) * LX + tx + HL;
    const uint8_t t = inmesh ? s_T[p] : 0, hm = inmesh ? s_H[p] : 0;
    if (inmesh) {
      P.Tcur[gi] = t;
      P.Hcur[gi] = hm;
    }
    const int st = mode == MODE_L ? 0 : mode - MODE_RK1;
    block_append_stat(t != 0, (int)gi, &P.stats[st], P.keep_lists ? P.flist : nullptr, s_wave);
    block_append_stat(hm != 0, (int)gi, &P.stats[3 + st], P.keep_lists ? P.hlist : nullptr, s_wave + 6);
  }

  // ---------------------------------------------------------------- limiter (Jacobi)
  // one item per (cell, direction, characteristic field), four lanes side by side for Euler,
  // as in stage2d_limit_kernel; written back once every item has read unlimited values
  const int nfl = s_cnt[0], nhl = s_cnt[1];
  const int nlim = nfl * 2 * NC;
  for (int it = tid; it < nlim; it += TH) {   // (whole groups of NC lanes)
    const int f = it % NC, dir = (it / NC) & 1, p = s_fl[it / (2 * NC)];
    s_lim[it] = limited_value<EQ>(P, s_u, p, dir, f);
  }
  __syncthreads();
  if (nfl) {
    for (int it = tid; it < nlim; it += TH) {
      const int f = it % NC, dir = (it / NC) & 1, p = s_fl[it / (2 * NC)];
      const double v = s_lim[it];
      s_u[((1 + dir) * NC + f) * NPOS + p] = v;
      const int cy = p / LX - HL, cx = p % LX - HL;
      if (cx >= 0 && cx < tw && cy >= 0 && cy < th)
        P.limcur[(size_t)(dir * NC + f) * plane + (size_t)(by * TY + cy) * nx + bx * TX + cx] = v;
    }
    __syncthreads();
    if (walls) {
      for (int q = tid; q < R2 * R2; q += TH) {
        const int ly = 1 + q / R2, lx = 1 + q % R2, p = ly * LX + lx;
        if (!s_T[p] || !mirrored(P, gx0 + lx, gy0 + ly)) continue;
        double sx, sy;
        const int m = mirror_pos(ly, lx, sx, sy);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const double wf = wall_factor<EQ>(c, sx < 0.0, sy < 0.0, P.bcx, P.bcy);
          s_u[(NC + c) * NPOS + p] = wf * (sx * s_u[(NC + c) * NPOS + m]);
          s_u[(2 * NC + c) * NPOS + p] = wf * (sy * s_u[(2 * NC + c) * NPOS + m]);
        }
      }
      __syncthreads();
    }
  }

  // ---------------------------------------------------------------- HWENO edge values
  // groups of 64 / NC cells, the two directions of a group on two waves; the tile's own values
  // go to P.G, the ring cells' towards the tile to LDS
  double* const s_rtr = s_lim;
  constexpr int CPW = 64 / NC;
  for (int w = tid >> 6; w < 2 * ((nhl + CPW - 1) / CPW); w += TH / 64) {
    const int cell = (w >> 1) * CPW + lane / NC, f = lane % NC, dir = w & 1;
    if (cell >= nhl) continue;   // whole groups of NC lanes
    const int p = s_hl[cell], cy = p / LX - HL, cx = p % LX - HL;
    const bool in_tile = cx >= 0 && cx < tw && cy >= 0 && cy < th;
    if (!in_tile && dir != ((cx >= 0 && cx < tw) ? 1 : 0)) continue;   // the ring's other direction
    double v[2 * NGE];
    if (dir == 0) hweno_values<EQ, NGE, 0>(P, s_u, p / LX, p % LX, f, v);
    else hweno_values<EQ, NGE, 1>(P, s_u, p / LX, p % LX, f, v);
    if (in_tile) {
      const size_t g = (size_t)(by * TY + cy) * nx + bx * TX + cx;
#pragma unroll
      for (int k = 0; k < NGE; ++k) {
        P.G[((((size_t)(dir * 2 + 0) * NGE + k) * NC + f)) * plane + g] = v[k];
        P.G[((((size_t)(dir * 2 + 1) * NGE + k) * NC + f)) * plane + g] = v[NGE + k];
      }
    } else {
      // low side of the tile: the ring cell's high face, and the other way round
      const bool low = dir == 0 ? cx < 0 : cy < 0;
      const int rl = dir * 2 * TX + (low ? 0 : TX) + (dir == 0 ? cy : cx);
#pragma unroll
      for (int k = 0; k < NGE; ++k) s_rtr[(f * NGE + k) * 64 + rl] = low ? v[NGE + k] : v[k];
    }
  }
  // (stage_tile waits for these values after its volume phase)
  stage_tile<EQ, NGE, BK_RECT, HL, TH>(P, sh, s_u, s_T, s_H, s_rtr, bx, by, dtv);
}

// Lax-Friedrichs speeds of a state (used before the first stage and by the operator-only
// entry point): per-direction max over cells of the spectral radius at the averages.
template <int EQ>
__global__ __launch_bounds__(256) void alpha2d_kernel(const double* U, int nx, int ny, double gam,
                                                      double a0, double a1, int si, int sj,
                                                      unsigned long long* alpha_out) {
  __shared__ double s_red[4];
  const size_t plane = (size_t)nx * ny;
  double m0 = 0.0, m1 = 0.0;
  for (size_t i = blockIdx.x * 256 + threadIdx.x; i < plane; i += (size_t)gridDim.x * 256) {
    if (si < nx) {
      // the solid cells of the forward step hold no flow
      const size_t gy = i / nx;
      if ((int)(i - gy * nx) >= si && (int)gy < sj) continue;
    }
    if constexpr (EQ == EQ_EULER) {
      double Ub[4], s0, s1, p;
      for (int c = 0; c < 4; ++c) Ub[c] = U[c * plane + i];
      euler_speeds2d(Ub, gam, s0, s1, p);
      m0 = fmax(m0, s0);
      m1 = fmax(m1, s1);
    } else if constexpr (EQ == EQ_BURGERS) {
      m0 = fmax(m0, fabs(U[i]));
      m1 = m0;
    } else {
      m0 = fabs(a0);
      m1 = fabs(a1);
    }
  }
  const double r0 = block_max256(m0, s_red);
  __syncthreads();
  const double r1 = block_max256(m1, s_red);
  if (threadIdx.x == 0) {
    const int e = blockIdx.x % ASPREAD;
    atomic_max_pos(&alpha_out[e], r0);
    atomic_max_pos(&alpha_out[ASPREAD + e], r1);
  }
}

// The double Mach reflection's prescribed ghost cells at the stage's time: the cut-cell
// moments of the exact solution (hw_dmr.h) at every position of the two ghost layers that
// is prescribed, one thread per (position, field); the stage's four kernels read them.
__global__ __launch_bounds__(NT) void dmr_table_kernel(Stage2D P) {
  constexpr int NF = 12;
  const double dtv = *P.dt;
  if (P.mode != MODE_L && dtv == 0.0) return;   // the run has reached its final time
  const double ts = dmr::stage_time(P.t, dtv, P.mode);
  const int nx = P.nx, ny = P.ny, nr = dmr::ring2_size(nx, ny);
  for (int q = blockIdx.x * NT + threadIdx.x; q < NF * nr; q += gridDim.x * NT) {
    const int f = q / nr, r = q - f * nr;
    int gx, gy;
    dmr::ring2_position(r, nx, ny, gx, gy);
    P.dtab[q] = dmr::prescribed(gx, gy, nx, ny, P.x0, P.dx)
                    ? dmr::cell_value(f, P.x0 + (gx + 0.5) * P.dx, P.y0 + (gy + 0.5) * P.dy, P.dx, ts, P.gam)
                    : 0.0;
  }
}

// the rule of stage2d_fused_kernel (with troubled-cell detection; both sides measured there)
constexpr int FUSED_TILES_EULER = 400, FUSED_TILES_SCALAR = 1600;
// two threads per cell up to one tile per compute unit (measured there)
constexpr int HELP_TILES = 256;
// Euler with every cell troubled takes four launches from this many cells a side to that many tiles
constexpr int FULL_SIDE = 13, FULL_TILES = 36;
static bool one_launch(int eq, int tc_mode, int bcx, int nx, int ny) {
  const long long tiles = (long long)((nx + TX - 1) / TX) * ((ny + TY - 1) / TY);
  const bool full = eq == EQ_EULER && tc_mode == TC_ALL && min(nx, ny) >= FULL_SIDE && tiles <= FULL_TILES;
  return tc_mode != TC_NONE && bcx != BC_DMR && bcx != BC_STEP && !full &&
         tiles <= (eq == EQ_EULER ? FUSED_TILES_EULER : FUSED_TILES_SCALAR);
}

}  // namespace hw

// ------------------------------------------------------------------ launch wrappers
extern "C" int hw_one_launch2d(int eq, int tc_mode, int bcx, int nx, int ny) {
  return hw::one_launch(eq, tc_mode, bcx, nx, ny) ? 1 : 0;
}

extern "C" hipError_t hw_launch_stage2d(int eq, int ng, const hw::Stage2D* P, hipStream_t s,
                                        hipEvent_t* ev) {
  dim3 grid(((P->nx + hw::TX - 1) / hw::TX) * ((P->ny + hw::TY - 1) / hw::TY));
  dim3 block(hw::NT);
  const bool pre = P->tc_mode != hw::TC_NONE;
  // work-list passes: a grid of a few workgroups per compute unit strides over the items
  const int wgrid = 2048;
#define HW_MARK(i) \
  if (ev && hipEventRecord(ev[i], s) != hipSuccess) return hipErrorLaunchFailure
  if (hw::one_launch(eq, P->tc_mode, P->bcx, P->nx, P->ny)) {
    HW_MARK(0);
    HW_MARK(1);
    HW_MARK(2);
#define HW_LF(E, G)                                                                               \
  do {                                                                                            \
    if (grid.x <= hw::HELP_TILES)                                                                 \
      hipLaunchKernelGGL((hw::stage2d_fused_kernel<E, G, 2 * hw::NT>), grid, dim3(2 * hw::NT), 0, s, *P); \
    else                                                                                          \
      hipLaunchKernelGGL((hw::stage2d_fused_kernel<E, G, hw::NT>), grid, block, 0, s, *P);        \
  } while (0)
    if (eq == hw::EQ_EULER && ng == 2) HW_LF(hw::EQ_EULER, 2);
    else if (eq == hw::EQ_EULER && ng == 3) HW_LF(hw::EQ_EULER, 3);
    else if (eq == hw::EQ_BURGERS && ng == 2) HW_LF(hw::EQ_BURGERS, 2);
    else if (eq == hw::EQ_BURGERS && ng == 3) HW_LF(hw::EQ_BURGERS, 3);
    else if (eq == hw::EQ_ADV && ng == 2) HW_LF(hw::EQ_ADV, 2);
    else if (eq == hw::EQ_ADV && ng == 3) HW_LF(hw::EQ_ADV, 3);
    else return hipErrorInvalidValue;
#undef HW_LF
    return hipGetLastError();
  }
#define HW_L2(E, G, D)                                                                  \
  do {                                                                                  \
    if (pre) hipLaunchKernelGGL((hw::stage2d_flags_kernel<E, D>), grid, block, 0, s, *P); \
    HW_MARK(0);                                                                         \
    if (pre) hipLaunchKernelGGL((hw::stage2d_limit_kernel<E, D>), dim3(wgrid), block, 0, s, *P); \
    HW_MARK(1);                                                                         \
    if (pre) hipLaunchKernelGGL((hw::stage2d_hweno_kernel<E, G, D>), dim3(wgrid), block, 0, s, *P); \
    HW_MARK(2);                                                                         \
    hipLaunchKernelGGL((hw::stage2d_kernel<E, G, D>), grid, block, 0, s, *P);           \
  } while (0)
  // the double Mach reflection and forward-step boundaries (Euler only) have kernel
  // instances of their own
  const int bk = P->bcx == hw::BC_DMR ? hw::BK_DMR : (P->bcx == hw::BC_STEP ? hw::BK_STEP : hw::BK_RECT);
  if (bk != hw::BK_RECT && eq != hw::EQ_EULER) return hipErrorInvalidValue;
  if (bk == hw::BK_DMR) {
    if (!P->dtab) return hipErrorInvalidValue;
    const int nq = 12 * (4 * (P->nx + 4) + 4 * P->ny);
    hipLaunchKernelGGL(hw::dmr_table_kernel, dim3((nq + hw::NT - 1) / hw::NT), block, 0, s, *P);
  }
  if (eq == hw::EQ_EULER && ng == 2 && bk == hw::BK_DMR) HW_L2(hw::EQ_EULER, 2, hw::BK_DMR);
  else if (eq == hw::EQ_EULER && ng == 3 && bk == hw::BK_DMR) HW_L2(hw::EQ_EULER, 3, hw::BK_DMR);
  else if (eq == hw::EQ_EULER && ng == 2 && bk == hw::BK_STEP) HW_L2(hw::EQ_EULER, 2, hw::BK_STEP);
  else if (eq == hw::EQ_EULER && ng == 3 && bk == hw::BK_STEP) HW_L2(hw::EQ_EULER, 3, hw::BK_STEP);
  else if (eq == hw::EQ_EULER && ng == 2) HW_L2(hw::EQ_EULER, 2, hw::BK_RECT);
  else if (eq == hw::EQ_EULER && ng == 3) HW_L2(hw::EQ_EULER, 3, hw::BK_RECT);
  else if (eq == hw::EQ_BURGERS && ng == 2) HW_L2(hw::EQ_BURGERS, 2, hw::BK_RECT);
  else if (eq == hw::EQ_BURGERS && ng == 3) HW_L2(hw::EQ_BURGERS, 3, hw::BK_RECT);
  else if (eq == hw::EQ_ADV && ng == 2) HW_L2(hw::EQ_ADV, 2, hw::BK_RECT);
  else if (eq == hw::EQ_ADV && ng == 3) HW_L2(hw::EQ_ADV, 3, hw::BK_RECT);
  else return hipErrorInvalidValue;
#undef HW_L2
#undef HW_MARK
  return hipGetLastError();
}

// the forward prepasses alone (the reverse mode reruns them on a stored stage input): flags
// and work lists, the limiter, the HWENO edge values; rectangles with periodic, transmissive
// or reflective sides, and the forward step (si, sj, uin set)
extern "C" hipError_t hw_launch_prepass2d(int eq, int ng, const hw::Stage2D* P, hipStream_t s) {
  if (P->tc_mode == hw::TC_NONE) return hipSuccess;
  dim3 grid(((P->nx + hw::TX - 1) / hw::TX) * ((P->ny + hw::TY - 1) / hw::TY));
  dim3 block(hw::NT);
  const int wgrid = 2048;
#define HW_PP(E, G, B)                                                                         \
  do {                                                                                         \
    hipLaunchKernelGGL((hw::stage2d_flags_kernel<E, B>), grid, block, 0, s, *P);               \
    hipLaunchKernelGGL((hw::stage2d_limit_kernel<E, B>), dim3(wgrid), block, 0, s, *P);        \
    hipLaunchKernelGGL((hw::stage2d_hweno_kernel<E, G, B>), dim3(wgrid), block, 0, s, *P);     \
  } while (0)
  // rectangles with mirrored or periodic sides, and the forward step
  const bool step = P->bcx == hw::BC_STEP;
  // the double Mach reflection: its prescribed ghosts of the stage's time first (dtab)
  const bool dmrb = P->bcx == hw::BC_DMR;
  if (dmrb && eq == hw::EQ_EULER && (ng == 2 || ng == 3)) {
    if (!P->dtab) return hipErrorInvalidValue;
    const int nq = 12 * hw::dmr::ring2_size(P->nx, P->ny);
    hipLaunchKernelGGL(hw::dmr_table_kernel, dim3((nq + hw::NT - 1) / hw::NT), block, 0, s, *P);
  }
  if (eq == hw::EQ_EULER && ng == 2 && dmrb) HW_PP(hw::EQ_EULER, 2, hw::BK_DMR);
  else if (eq == hw::EQ_EULER && ng == 3 && dmrb) HW_PP(hw::EQ_EULER, 3, hw::BK_DMR);
  else if (eq == hw::EQ_EULER && ng == 2 && !step) HW_PP(hw::EQ_EULER, 2, hw::BK_RECT);
  else if (eq == hw::EQ_EULER && ng == 3 && !step) HW_PP(hw::EQ_EULER, 3, hw::BK_RECT);
  else if (eq == hw::EQ_EULER && ng == 2) HW_PP(hw::EQ_EULER, 2, hw::BK_STEP);
  else if (eq == hw::EQ_EULER && ng == 3) HW_PP(hw::EQ_EULER, 3, hw::BK_STEP);
  else return hipErrorInvalidValue;
#undef HW_PP
  return hipGetLastError();
}

extern "C" hipError_t hw_launch_alpha2d(int eq, const double* U, int nx, int ny, double gam,
                                        double a0, double a1, int si, int sj,
                                        unsigned long long* alpha_out, hipStream_t s) {
  const size_t n = (size_t)nx * ny;
  int blocks = (int)((n + 255) / 256);
  if (blocks > 2048) blocks = 2048;
  if (eq == hw::EQ_EULER)
    hipLaunchKernelGGL(hw::alpha2d_kernel<hw::EQ_EULER>, dim3(blocks), dim3(256), 0, s, U, nx, ny, gam, a0, a1, si, sj, alpha_out);
  else if (eq == hw::EQ_BURGERS)
    hipLaunchKernelGGL(hw::alpha2d_kernel<hw::EQ_BURGERS>, dim3(blocks), dim3(256), 0, s, U, nx, ny, gam, a0, a1, si, sj, alpha_out);
  else
    hipLaunchKernelGGL(hw::alpha2d_kernel<hw::EQ_ADV>, dim3(blocks), dim3(256), 0, s, U, nx, ny, gam, a0, a1, si, sj, alpha_out);
  return hipGetLastError();
}
