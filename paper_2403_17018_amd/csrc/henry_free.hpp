// The multigrid smoother, the residual's restriction and the Krylov products of the FP64 forward
// solves with the Jacobian's rows formed from the state instead of read: a row of the five-point
// 2x2-block operator is a function of p, c, phi and K of its cell and its four neighbours.  These
// kernels are bound by memory, and a colour pass reads 8 of those values per row (its own cell's
// and, each shared by the rows around it, its neighbours') where the stored row has 20; a product
// reads 4 per cell.  No Jacobian is assembled or written for them.  256x128 cells, 512 samples, us
// (stored rows, formed rows): colour pass 268, 207 (4.5 TB/s); the two passes of the first
// half-sweep 372, 171 + 207; with the prolongation 361, 340; restriction 209, 184; product 424, 308;
// assembly 788, 304 (its residual alone).  One sample per thread: two took 170 registers (223, 238).
#pragma once

#include <hip/hip_runtime.h>

#include "henry_kernels.hpp"

namespace henry {

// The state and coefficients a grid's operator is taken at.
struct FreeOp {
  const double *p, *c, *phi, *K;
};

struct CellState {
  double p, c, phi, K;
};

__device__ __forceinline__ CellState ld_state(const FreeOp& A, size_t q) { return {A.p[q], A.c[q], A.phi[q], A.K[q]}; }

// The constants of a row, set up on the host (kernel arguments: scalar registers).
struct FreePhys {
  double w[2];      // face area over distance, x and y faces
  double qd[2];     // ... times Dm
  double gA;        // g times the y face's area
  double inv_mu, hd, vt;
  double side_dif;  // 2 Dm hy / hx
  double side_k;    // outflow through the right side per pressure difference and K: hy / (mu hx / 2)
  FreePhys() = default;
  explicit FreePhys(const Phys& P)
      : w{P.hy / P.hx, P.hx / P.hy}, qd{P.Dm * w[0], P.Dm * w[1]}, gA(P.g * P.hx), inv_mu(1.0 / P.mu),
        hd(0.5 * P.drho), vt(P.vol / P.tau), side_dif(2.0 * P.Dm * P.hy / P.hx), side_k(2.0 * P.hy / (P.mu * P.hx)) {}
};

// The left and right sides' share of a cell's centre block (boundary_terms).
__device__ __forceinline__ void side_terms(const Phys& P, const FreePhys& F, int nx, int i, int j, const CellState& o,
                                           double (&D)[4]) {
  const double rP = P.rho0 + P.drho * o.c, dif = o.phi * F.side_dif;
  if (i == 0) D[3] += dif * (P.drho * (o.c - P.c_left) + rP);
  if (i == nx - 1) {
    const double k = o.K * F.side_k, y = -P.Ly + (j + 0.5) * P.hy;
    const double u = k * (o.p + P.rho1 * P.g * y);
    const bool inflow = u < 0.0;
    const double dFdp = (inflow ? P.rho1 : rP) * k, dFdc = inflow ? 0.0 : P.drho * u;
    const double cb = inflow ? 1.0 : o.c;
    D[0] += dFdp;
    D[1] += dFdc;
    D[2] += cb * dFdp;
    D[3] += cb * dFdc + (inflow ? 0.0 : rP * u);
    if (P.right_dir) D[3] += dif * (P.drho * (o.c - 1.0) + rP);
  }
}

// 1/x of a normal x to rounding: the hardware's estimate and two Newton steps.
__device__ __forceinline__ double rcp_normal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// What a face adds to the row of the cell on one side of it, as face_flux's derivatives: the
// neighbour's block [-a, sb; -ac, dN] and the cell's own [a, sb; ac, dP].
struct FaceRow {
  double a, sb, ac, dN, dP;
};

// NORTH: a face between rows; HIGH: the cell is the face's high (east, north) side.
template <bool NORTH, bool HIGH>
__device__ __forceinline__ FaceRow face_row(const Phys& P, const FreePhys& F, const CellState& own,
                                            const CellState& nb) {
  const CellState &L = HIGH ? nb : own, &H = HIGH ? own : nb;
  const double kf = 2.0 * L.K * H.K * rcp_normal(L.K + H.K) * F.inv_mu;
  const double rf = P.rho0 + F.hd * (L.c + H.c);
  const double kw = kf * F.w[NORTH];
  const double rk = rf * kf;
  double uA = kw * (L.p - H.p), grav = 0.0;
  if (NORTH) {
    grav = rk * F.gA;
    uA -= grav;
  }
  const double flux = rf * uA;
  const bool up = flux >= 0.0;
  const double cup = up ? L.c : H.c;
  const double q = 0.5 * (L.phi + H.phi) * F.qd[NORTH];
  const double dif = rf * q;
  const double bF = F.hd * (uA - grav);
  const double g = bF * cup - F.hd * q * (H.c - L.c);
  const double dL = g + (up ? flux : 0.0) + dif, dH = g + (up ? 0.0 : flux) - dif;
  FaceRow r;
  r.a = rk * F.w[NORTH];
  r.ac = r.a * cup;
  r.sb = HIGH ? -bF : bF;
  r.dN = HIGH ? -dL : dH;
  r.dP = HIGH ? -dH : dL;
  return r;
}

// A row being summed: y = the neighbours' part of A x, D = the centre block.
struct RowSum {
  double y0 = 0.0, y1 = 0.0, D[4];
  __device__ __forceinline__ RowSum(const Phys& P, const FreePhys& F, const CellState& own) {
    const double v = F.vt * own.phi;
    D[0] = D[2] = 0.0;
    D[1] = v * P.drho;
    D[3] = v * (P.rho0 + 2.0 * P.drho * own.c);
  }
  __device__ __forceinline__ void centre(const FaceRow& f) {
    D[0] += f.a;
    D[1] += f.sb;
    D[2] += f.ac;
    D[3] += f.dP;
  }
  __device__ __forceinline__ void neighbour(const FaceRow& f, double x0, double x1) {
    y0 += f.sb * x1 - f.a * x0;
    y1 += f.dN * x1 - f.ac * x0;
  }
  // x = D^{-1} (b - y)
  __device__ __forceinline__ void solve(double b0, double b1, double& x0, double& x1) const {
    const double r0 = b0 - y0, r1 = b1 - y1;
    const double det = D[0] * D[3] - D[1] * D[2];
    const double rdet = 1.0 / det;
    x0 = (D[3] * r0 - D[1] * r1) * rdet;
    x1 = (D[0] * r1 - D[2] * r0) * rdet;
  }
};

// Row (i, j): WANT_D the centre block, WANT_Y the neighbours' part; xv(n, q, x0, x1): the values of
// neighbour n (0 W, 1 E, 2 S, 3 N) at index q.  All loads are issued before any arithmetic; a
// neighbour outside the grid reads the cell itself and is left out.
template <bool WANT_D, bool WANT_Y, typename XV>
__device__ __forceinline__ RowSum free_row(const FreeOp& A, const Phys& P, const FreePhys& F, int nx, int ny, int S,
                                           size_t id, int i, int j, const CellState& own, XV&& xv) {
  const bool ok[4] = {i > 0, i < nx - 1, j > 0, j < ny - 1};
  const long long step[4] = {-(long long)S, S, -(long long)nx * S, (long long)nx * S};
  CellState nb[4];
  double xa[4] = {}, xb[4] = {};
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const size_t q = ok[n] ? id + step[n] : id;
    nb[n] = ld_state(A, q);
    if (WANT_Y) xv(n, q, xa[n], xb[n]);
  }
  RowSum r(P, F, own);
  auto add = [&](int n, const FaceRow& f) {
    if (!ok[n]) return;
    if (WANT_D) r.centre(f);
    if (WANT_Y) r.neighbour(f, xa[n], xb[n]);
  };
  add(0, face_row<false, true>(P, F, own, nb[0]));
  add(1, face_row<false, false>(P, F, own, nb[1]));
  add(2, face_row<true, true>(P, F, own, nb[2]));
  add(3, face_row<true, false>(P, F, own, nb[3]));
  if (WANT_D) side_terms(P, F, nx, i, j, own, r.D);
  return r;
}

// One colour of a red-black sweep, as k_gs_colour: MODE 0 plain, 1 from x = 0 (neighbours' x not
// read), 2 with the coarse correction e prolonged onto the neighbours on the fly.
template <int MODE>
__global__ void __launch_bounds__(256) k_gs_free(Map m, Grid2 G, Grid2 Gc, int colour, Phys P, FreePhys F,
                                                 FreeOp A, const double* __restrict__ b, double* __restrict__ x,
                                                 const double* __restrict__ e) {
  int s, mc, sb, cb;
  const int half = (G.nx + 1) >> 1;
  if (!map_cell(m, G.ny * half, s, mc, sb, cb)) return;
  const int j = mc / half;
  const int i = 2 * (mc - j * half) + ((j + colour) & 1);
  if (i >= G.nx) return;
  const size_t N = (size_t)G.ncell * m.S;
  const size_t id = ((size_t)j * G.nx + i) * m.S + s;
  const CellState own = ld_state(A, id);
  const double b0 = b[id], b1 = b[N + id];
  auto xv = [&](int n, size_t q, double& x0, double& x1) {
    x0 = x[q];
    x1 = x[N + q];
    if (MODE == 2) {
      double v0, v1;
      const int qi = i + (n == 0 ? -1 : n == 1 ? 1 : 0), qj = j + (n == 2 ? -1 : n == 3 ? 1 : 0);
      const bool in = qi >= 0 && qi < G.nx && qj >= 0 && qj < G.ny;
      prolong_at<double>(e, (size_t)Gc.ncell * m.S, m.S, s, in ? qi : i, in ? qj : j, Gc, v0, v1);
      x0 += v0;
      x1 += v1;
    }
  };
  const RowSum r = free_row<true, MODE != 1>(A, P, F, G.nx, G.ny, m.S, id, i, j, own, xv);
  double x0, x1;
  r.solve(b0, b1, x0, x1);
  x[id] = x0;
  x[N + id] = x1;
}

// Residual and restriction after a black pass, as k_residual_restrict: only the red rows' residuals
// are not zero.  exact: red x = D^{-1} b (one pre-smoothing sweep from x = 0), so the residual is
// minus the neighbours' part.
__global__ void __launch_bounds__(256) k_restrict_free(Map m, Grid2 G, Grid2 Gc, int exact, Phys P, FreePhys F,
                                                       FreeOp A, const double* __restrict__ b,
                                                       const double* __restrict__ x, double* __restrict__ bH) {
  int s, cc, sb, cb;
  if (!map_cell(m, Gc.ncell, s, cc, sb, cb)) return;
  const int S = m.S;
  const size_t N = (size_t)G.ncell * S, Nc = (size_t)Gc.ncell * S;
  const int Jc = cc / Gc.nx, Ic = cc - Jc * Gc.nx;
  double s0 = 0.0, s1 = 0.0;
  auto xv = [&](int, size_t q, double& x0, double& x1) {
    x0 = x[q];
    x1 = x[N + q];
  };
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int i = 2 * Ic + q, j = 2 * Jc + q;
    const size_t id = ((size_t)j * G.nx + i) * S + s;
    const CellState own = ld_state(A, id);
    if (exact) {
      const RowSum r = free_row<false, true>(A, P, F, G.nx, G.ny, S, id, i, j, own, xv);
      s0 -= r.y0;
      s1 -= r.y1;
    } else {
      const RowSum r = free_row<true, true>(A, P, F, G.nx, G.ny, S, id, i, j, own, xv);
      const double x0 = x[id], x1 = x[N + id];
      s0 += b[id] - r.y0 - r.D[0] * x0 - r.D[1] * x1;
      s1 += b[N + id] - r.y1 - r.D[2] * x0 - r.D[3] * x1;
    }
  }
  const size_t o = (size_t)cc * S + s;
  bH[o] = s0;
  bH[Nc + o] = s1;
}

// y = A x and per-sample dots, as k_spmv_dot (yb: the black rows' product is known).
template <int NDOT, typename TX>
__global__ void __launch_bounds__(256) k_spmv_free(Map m, Grid2 G, Phys P, FreePhys F, FreeOp A,
                                                   const TX* __restrict__ x, double* __restrict__ y,
                                                   const double* __restrict__ d0, double* __restrict__ part,
                                                   const double* __restrict__ yb) {
  __shared__ double lds[2 * 256];
  const int sblk = blockIdx.x % m.nsb, cblk = blockIdx.x / m.nsb;
  const int s = sblk * m.SX + threadIdx.x;
  const bool sv = s < m.S;
  const size_t N = (size_t)G.ncell * m.S;
  double acc[NDOT];
#pragma unroll
  for (int q = 0; q < NDOT; ++q) acc[q] = 0.0;
  for (int k = 0; k < m.CPT; ++k) {
    const int cell = (cblk * m.CPT + k) * m.CY + threadIdx.y;
    if (!sv || cell >= G.ncell) continue;
    const int j = cell / G.nx, i = cell - j * G.nx;
    const size_t id = (size_t)cell * m.S + s;
    double y0, y1;
    if (yb && ((i + j) & 1)) {
      y0 = yb[id];
      y1 = yb[N + id];
    } else {
      auto xv = [&](int, size_t q, double& x0, double& x1) {
        x0 = (double)x[q];
        x1 = (double)x[N + q];
      };
      const CellState own = ld_state(A, id);
      const double x0 = (double)x[id], x1 = (double)x[N + id];
      const RowSum r = free_row<true, true>(A, P, F, G.nx, G.ny, m.S, id, i, j, own, xv);
      y0 = r.y0 + r.D[0] * x0 + r.D[1] * x1;
      y1 = r.y1 + r.D[2] * x0 + r.D[3] * x1;
    }
    y[id] = y0;
    y[N + id] = y1;
    if (NDOT == 1) {
      acc[0] += d0[id] * y0 + d0[N + id] * y1;
    } else {
      acc[0] += y0 * d0[id] + y1 * d0[N + id];
      acc[NDOT - 1] += y0 * y0 + y1 * y1;
    }
  }
  block_sum_y<NDOT>(acc, lds);
  if (threadIdx.y == 0 && sv) {
#pragma unroll
    for (int q = 0; q < NDOT; ++q) part[((size_t)q * m.ncb + cblk) * m.S + s] = acc[q];
  }
}

}  // namespace henry
