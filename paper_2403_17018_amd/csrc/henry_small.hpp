// Grids of up to 2048 cells: the whole Newton iteration of a time step in one launch, a workgroup
// per sample.  The state, the cycle's iterates and the coarse grids' states stay in LDS, the Krylov
// vectors in registers; every decision (convergence, damping, a fresh coarse operator, breakdown)
// is the sample's own, taken on the device.  Operator rows are formed from the state wherever they
// are used (henry_free.hpp): LDS would not hold the Jacobian.
//
// Launch by launch a step of these grids is some 110 launches of 3 to 5 us and four host reads,
// however few the samples, and a batch iterates until its hardest sample is done.  Milliseconds a
// solve, before and with this kernel: 32x16 cells, 48 steps, 16 samples 31.0 and 9.9, 256 samples
// 40.5 and 11.6; 64x32 cells, 48 steps, 64 samples 42.6 and 22.5, 333 samples 88 and 45; 24 steps,
// 1000 samples 147 and 59; 12 steps, 4096 samples 574 and 144 (32x16: 83 and 63): it is taken for
// every batch size.  What bounds it is the chain of a cycle's passes, each a barrier, a few LDS
// reads and some 200 dependent FP64 operations, and of the coarsest operator's inversion; one
// workgroup (LDS, registers) fits a compute unit.
#pragma once

#include <hip/hip_runtime.h>

#include "henry_march.hpp"

namespace henry {

constexpr int SMALL_THREADS = 512, SMALL_CELLS = 2048, SMALL_LEVELS = TAIL_LEVELS + 1;   // smoothed grids at most

struct SmallArgs {
  int S, nl;                                    // samples, smoothed grids (the coarsest follows)
  int nx[SMALL_LEVELS + 1], ny[SMALL_LEVELS + 1];
  int at[SMALL_LEVELS + 2];                     // the grids' places in LDS (small_layout), the rest's
  double hy[SMALL_LEVELS + 1];
  FreePhys F[SMALL_LEVELS + 1];
  double *p, *c;                                // state [cell][S]: the first guess in, the solution out
  const double *c_old, *uin;
  const double *phi[SMALL_LEVELS + 1], *K[SMALL_LEVELS + 1];
  double* inv;                                  // [S][n][n]: the coarsest operators' inverses
  int* status;
  double* stats;                                // [S][4]: Newton, BiCGStab iterations
  int nu_pre, nu_post, newton_maxit, krylov_maxit;
  double rtol2, breakdown, newton_tol, pred_tol, dc_max, jac_reuse, p_ref;
};

// LDS in units of 16 bytes: per grid its state (p c, phi K), iterate and (but for the finest)
// right-hand side; then the red residuals of the finest grid, which the inversion's scratch shares,
// and the reductions.  Returns its bytes.
__host__ __device__ inline int small_scratch(const SmallArgs& A) {
  const int rs = A.nx[0] * A.ny[0] / 2, gj = 10 * A.nx[A.nl] * A.ny[A.nl] + 4 * TAIL_NMAX;
  return rs > gj ? rs : gj;
}
inline size_t small_layout(SmallArgs& A) {
  int n = 0;
  for (int l = 0; l <= A.nl; ++l) {
    A.at[l] = n;
    n += (l == 0 ? 3 : 4) * A.nx[l] * A.ny[l];
  }
  A.at[A.nl + 1] = n;
  return (size_t)(n + small_scratch(A) + 2 * SMALL_THREADS / 64) * 16;
}

// Where the cells of a smoothed grid lie: red ones ((i + j) even) first, row by row, then the black
// ones, so that a colour's cells and each of their neighbours are contiguous.
struct SmallCell {
  int at, i, j, w, e, s, n;   // own place and the neighbours' (a missing one's: another neighbour's)
};
__device__ __forceinline__ SmallCell small_cell(int colour, int u, int i, int j, int nx, int ny) {
  const int hx = nx >> 1, half = hx * ny, ob = (1 - colour) * half, o = i & 1;
  SmallCell c;
  c.i = i;
  c.j = j;
  c.at = colour * half + u;
  c.w = ob + u + o - 1;
  c.e = ob + u + o;
  c.s = ob + u - hx;
  c.n = ob + u + hx;
  if (i == 0) c.w = c.e;
  if (i == nx - 1) c.e = c.w;
  if (j == 0) c.s = c.w;
  if (j == ny - 1) c.n = c.w;
  return c;
}
__device__ __forceinline__ SmallCell small_cell(int colour, int u, int nx, int ny) {
  const int hx = nx >> 1, j = u / hx;
  return small_cell(colour, u, 2 * (u - j * hx) + ((j + colour) & 1), j, nx, ny);
}
__device__ __forceinline__ int small_at(int i, int j, int nx, int ny) {
  const int hx = nx >> 1;
  return ((i + j) & 1) * hx * ny + j * hx + (i >> 1);
}

struct SmallGrid {
  int nx, ny, n;
  Two *pc, *fk, *x, *b;
  __device__ __forceinline__ CellState state(int q) const {
    const Two u = pc[q], v = fk[q];
    return CellState{u[0], u[1], v[0], v[1]};
  }
};

// The four faces' terms of a cell; f(side, face, the neighbour's place), sides 0 W, 1 E, 2 S, 3 N.
template <typename Fn>
__device__ __forceinline__ void small_faces(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c,
                                            const CellState& own, Fn&& f) {
  const double km = 2.0 * F.inv_mu, qx = 0.5 * F.qd[0], qy = 0.5 * F.qd[1];
  const bool w = c.i > 0, e = c.i < G.nx - 1, s = c.j > 0, n = c.j < G.ny - 1;
  f(0, face_terms<false>(P, F, w ? km : 0.0, w ? qx : 0.0, G.state(c.w), own), c.w);
  f(1, face_terms<false>(P, F, e ? km : 0.0, e ? qx : 0.0, own, G.state(c.e)), c.e);
  f(2, face_terms<true>(P, F, s ? km : 0.0, s ? qy : 0.0, G.state(c.s), own), c.s);
  f(3, face_terms<true>(P, F, n ? km : 0.0, n ? qy : 0.0, own, G.state(c.n)), c.n);
}
// the neighbours' part of the row times x
__device__ __forceinline__ Two small_off(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c) {
  Two y{0.0, 0.0};
  small_faces(G, P, F, c, G.state(c.at), [&](int side, const Face& f, int q) {
    const Two v = G.x[q];
    const bool high = (side & 1) == 0;   // the cell is the high side of its west and south faces
    y[0] += (high ? -f.b : f.b) * v[1] - f.a * v[0];
    y[1] += (high ? -f.dL : f.dH) * v[1] - f.ac * v[0];
  });
  return y;
}
struct Inv2 {
  double a, b, c, d;
  __device__ __forceinline__ Two operator()(const Two& r) const { return Two{a * r[0] + b * r[1], c * r[0] + d * r[1]}; }
};
__device__ __forceinline__ Inv2 small_inverse(const double (&D)[4]) {
  const double rdet = 1.0 / (D[0] * D[3] - D[1] * D[2]);
  return Inv2{D[3] * rdet, -D[1] * rdet, -D[2] * rdet, D[0] * rdet};
}
// the centre block; blk(side, values): the neighbours' blocks
template <typename Fn>
__device__ __forceinline__ void small_centre(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c,
                                             double (&D)[4], Fn&& blk) {
  const CellState own = G.state(c.at);
  const double v = F.vt * own.phi;
  D[0] = D[2] = 0.0;
  D[1] = v * P.drho;
  D[3] = v * (P.rho0 + 2.0 * P.drho * own.c);
  small_faces(G, P, F, c, own, [&](int side, const Face& f, int) {
    const bool high = (side & 1) == 0;
    D[0] += f.a;
    D[1] += high ? -f.b : f.b;
    D[2] += f.ac;
    D[3] += high ? -f.dH : f.dL;
    blk(side, -f.a, high ? -f.b : f.b, -f.ac, high ? -f.dL : f.dH);
  });
  side_terms(P, F, G.nx, c.i, c.j, own, D);
}

// D^{-1} (b - the neighbours' part), or D^{-1} b from x = 0
__device__ __forceinline__ Two small_solve(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c,
                                           bool zero) {
  const CellState own = G.state(c.at);
  const double v = F.vt * own.phi;
  double D[4] = {0.0, v * P.drho, 0.0, v * (P.rho0 + 2.0 * P.drho * own.c)};
  Two r = G.b[c.at];
  small_faces(G, P, F, c, own, [&](int side, const Face& f, int q) {
    const bool high = (side & 1) == 0;
    D[0] += f.a;
    D[1] += high ? -f.b : f.b;
    D[2] += f.ac;
    D[3] += high ? -f.dH : f.dL;
    if (zero) return;
    const Two x = G.x[q];
    r[0] -= (high ? -f.b : f.b) * x[1] - f.a * x[0];
    r[1] -= (high ? -f.dL : f.dH) * x[1] - f.ac * x[0];
  });
  side_terms(P, F, G.nx, c.i, c.j, own, D);
  return small_inverse(D)(r);
}
// b - A x of a row
__device__ __forceinline__ Two small_residual(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c) {
  const CellState own = G.state(c.at);
  const double v = F.vt * own.phi;
  double D[4] = {0.0, v * P.drho, 0.0, v * (P.rho0 + 2.0 * P.drho * own.c)};
  Two r = G.b[c.at];
  small_faces(G, P, F, c, own, [&](int side, const Face& f, int q) {
    const bool high = (side & 1) == 0;
    D[0] += f.a;
    D[1] += high ? -f.b : f.b;
    D[2] += f.ac;
    D[3] += high ? -f.dH : f.dL;
    const Two x = G.x[q];
    r[0] -= (high ? -f.b : f.b) * x[1] - f.a * x[0];
    r[1] -= (high ? -f.dL : f.dH) * x[1] - f.ac * x[0];
  });
  side_terms(P, F, G.nx, c.i, c.j, own, D);
  const Two x = G.x[c.at];
  return r - Two{D[0] * x[0] + D[1] * x[1], D[2] * x[0] + D[3] * x[1]};
}

// H: cells of each colour of the finest grid per thread (1 up to 1024 cells, 2 up to 2048); RC, TC:
// the inversion's shape (tail_inverse).
template <int H, int RC, int TC>
__global__ void __launch_bounds__(SMALL_THREADS, 2) k_small_step(SmallArgs A, Phys P) {
  extern __shared__ Two ssh[];
  const int s = tail_sample(A.S), t = threadIdx.x, S = A.S;
  if (s >= S) return;
  const int nl = A.nl;
  auto grid = [&](int l) {
    const int n = A.nx[l] * A.ny[l];
    Two* q = ssh + A.at[l];
    return SmallGrid{A.nx[l], A.ny[l], n, q, q + n, q + 2 * n, q + 3 * n};
  };
  auto phys = [&](int l) {   // what side_terms takes from it
    Phys q = P;
    q.hy = A.hy[l];
    return q;
  };
  const SmallGrid G = grid(0), C = grid(nl);
  Two* const scratch = ssh + A.at[nl + 1];
  double* const red = reinterpret_cast<double*>(scratch + small_scratch(A));   // [2][2][8]
  const int half = G.n >> 1, nu = 2 * C.n;
  // this thread's cells: H red, then H black (i and j kept packed: the rest is found anew, which
  // takes fewer registers)
  int ij[2 * H];
#pragma unroll
  for (int m = 0; m < 2 * H; ++m) {
    const int u = t + SMALL_THREADS * (m % H);
    const SmallCell c = small_cell(m / H, u, G.nx, G.ny);
    ij[m] = u < half ? c.j << 16 | c.i : -1;
  }
  auto cell = [&](int m, SmallCell& c) {
    int k = ij[m];
    asm volatile("" : "+v"(k));
    if (k < 0) return false;
    c = small_cell(m / H, t + SMALL_THREADS * (m % H), k & 0xffff, k >> 16, G.nx, G.ny);
    return true;
  };
  auto global = [&](const SmallCell& c) { return ((size_t)c.j * G.nx + c.i) * S + s; };
  // its cell of a coarser smoothed grid
  auto coarse = [&](const SmallGrid& g, SmallCell& c) {
    const int h = g.n >> 1;
    if (t >= g.n) return false;
    c = t < h ? small_cell(0, t, g.nx, g.ny) : small_cell(1, t - h, g.nx, g.ny);
    return true;
  };
  int flip = 0;
  auto sum2 = [&](double& a, double& b) {
    for (int k = 32; k > 0; k >>= 1) {
      a += __shfl_xor(a, k);
      b += __shfl_xor(b, k);
    }
    double* q = red + 16 * flip;
    flip ^= 1;
    if ((t & 63) == 0) {
      q[t >> 6] = a;
      q[8 + (t >> 6)] = b;
    }
    lds_barrier();
    a = b = 0.0;
#pragma unroll
    for (int k = 0; k < SMALL_THREADS / 64; ++k) {
      a += q[k];
      b += q[8 + k];
    }
  };
  auto larger = [](double a, double b) { return b > a || b != b ? b : a; };   // a NaN stays
  auto max2 = [&](double& a, double& b) {
    for (int k = 32; k > 0; k >>= 1) {
      a = larger(a, __shfl_xor(a, k));
      b = larger(b, __shfl_xor(b, k));
    }
    double* q = red + 16 * flip;
    flip ^= 1;
    if ((t & 63) == 0) {
      q[t >> 6] = a;
      q[8 + (t >> 6)] = b;
    }
    lds_barrier();
    a = b = 0.0;
#pragma unroll
    for (int k = 0; k < SMALL_THREADS / 64; ++k) {
      a = larger(a, q[k]);
      b = larger(b, q[8 + k]);
    }
  };

  // state and coefficients into LDS
#pragma unroll
  for (int m = 0; m < 2 * H; ++m) {
    SmallCell c;
    if (!cell(m, c)) continue;
    const size_t q = global(c);
    G.pc[c.at] = Two{A.p[q], A.c[q]};
    G.fk[c.at] = Two{A.phi[0][q], A.K[0][q]};
  }
  for (int l = 1; l <= nl; ++l) {
    const SmallGrid g = grid(l);
    for (int q = t; q < g.n; q += SMALL_THREADS) {
      const int j = q / g.nx, i = q - j * g.nx;
      g.fk[l < nl ? small_at(i, j, g.nx, g.ny) : q] = Two{A.phi[l][(size_t)q * S + s], A.K[l][(size_t)q * S + s]};
    }
  }
  lds_barrier();

  Inv2 Di[2 * H];   // inverse centre blocks of the fine cells
  double iv[8];                                // the first eight terms of this thread's row of the inverse
  double* const inv = A.inv + (size_t)s * nu * nu;
  const int part = t & 7;
  double last = 0.0, r2prev = 0.0, newtons = 0.0, kits = 0.0;
  int status = 0;
  bool done = false, fresh = true;

  // ---- x = M^{-1} b: b of this thread's fine cells in, x in G.x; rd: the last red right-hand sides
  // less their neighbours' part (D x of the red cells)
  auto cycle = [&](const Two (&b)[2 * H], Two (&rd)[H]) {
    const Phys P0 = phys(0);
    auto pass = [&](int colour, bool zero) {
#pragma unroll
      for (int m = 0; m < H; ++m) {
        const int k = colour * H + m;
        SmallCell c;
        if (!cell(k, c)) continue;
        Two r = b[k];
        if (!zero) r -= small_off(G, P0, A.F[0], c);
        if (colour == 0) rd[m] = r;
        G.x[c.at] = Di[k](r);
      }
      lds_barrier();
    };
    pass(0, true);
    pass(1, false);
    for (int sw = 1; sw < A.nu_pre; ++sw) {
      pass(0, false);
      pass(1, false);
    }
#pragma unroll
    for (int m = 0; m < H; ++m) {   // D x = rd of the last red pass: what is left is the neighbours' change
      SmallCell c;
      if (!cell(m, c)) continue;
      scratch[c.at] = b[m] - rd[m] - small_off(G, P0, A.F[0], c);
    }
    lds_barrier();
    auto gather = [&](const SmallGrid& f, int I, int J) {   // the two red children's residuals
      const int hx = f.nx >> 1;
      return scratch[2 * J * hx + I] + scratch[(2 * J + 1) * hx + I];
    };
#pragma unroll 1
    for (int l = 1; l < nl; ++l) {
      const SmallGrid g = grid(l);
      const Phys Pl = phys(l);
      SmallCell c;
      const bool own = coarse(g, c), is_red = own && t < (g.n >> 1), black = own && !is_red;
      if (own) g.b[c.at] = gather(grid(l - 1), c.i, c.j);
#pragma unroll 1
      for (int sw = 0; sw < A.nu_pre; ++sw) {
        if (is_red) g.x[c.at] = small_solve(g, Pl, A.F[l], c, sw == 0);
        lds_barrier();
        if (black) g.x[c.at] = small_solve(g, Pl, A.F[l], c, false);
        lds_barrier();
      }
      if (is_red) scratch[c.at] = small_residual(g, Pl, A.F[l], c);
      lds_barrier();
    }
    if (t < C.n) C.b[t] = gather(grid(nl - 1), t % C.nx, t / C.nx);
    lds_barrier();
    {
      const double* v = reinterpret_cast<const double*>(C.b);
      double* y = reinterpret_cast<double*>(C.x);
      for (int row = t >> 3, k = 0; row < nu; row += SMALL_THREADS / 8, ++k) {
        double acc = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int q = part + 8 * e;
          if (q < nu) acc += (k == 0 ? iv[e] : inv[(size_t)row * nu + q]) * v[q];
        }
        for (int q = part + 64; q < nu; q += 8) acc += inv[(size_t)row * nu + q] * v[q];
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) acc += __shfl_xor(acc, o);
        if (part == 0) y[row] = acc;
      }
    }
    lds_barrier();
    // the correction prolonged onto a black cell
    auto prolong = [&](const SmallGrid& g, const SmallGrid& e, bool coarsest, const SmallCell& c) {
      const int I = c.i >> 1, J = c.j >> 1;
      const int I2 = min(max(I + ((c.i & 1) ? 1 : -1), 0), e.nx - 1), J2 = min(max(J + ((c.j & 1) ? 1 : -1), 0), e.ny - 1);
      auto v = [&](int i, int j) { return e.x[coarsest ? j * e.nx + i : small_at(i, j, e.nx, e.ny)]; };
      g.x[c.at] += 0.5625 * v(I, J) + 0.1875 * (v(I2, J) + v(I, J2)) + 0.0625 * v(I2, J2);
    };
#pragma unroll 1
    for (int l = nl - 1; l >= 1; --l) {
      const SmallGrid g = grid(l);
      const Phys Pl = phys(l);
      SmallCell c;
      const bool own = coarse(g, c), is_red = own && t < (g.n >> 1), black = own && !is_red;
      if (black) prolong(g, grid(l + 1), l + 1 == nl, c);
      lds_barrier();
#pragma unroll 1
      for (int sw = 0; sw < A.nu_post; ++sw) {
        if (is_red) g.x[c.at] = small_solve(g, Pl, A.F[l], c, false);
        lds_barrier();
        if (black) g.x[c.at] = small_solve(g, Pl, A.F[l], c, false);
        lds_barrier();
      }
    }
#pragma unroll
    for (int m = H; m < 2 * H; ++m) {
      SmallCell c;
      if (cell(m, c)) prolong(G, grid(1), nl == 1, c);
    }
    lds_barrier();
#pragma unroll 1
    for (int sw = 0; sw < A.nu_post; ++sw) {
      pass(0, false);
      pass(1, false);
    }
  };
  // A x after a cycle: its black pass left A x = b on the black cells
  auto apply = [&](const Two (&b)[2 * H], const Two (&rd)[H], Two (&y)[2 * H]) {
    const Phys P0 = phys(0);
#pragma unroll
    for (int m = 0; m < H; ++m) {
      SmallCell c;
      y[m] = y[H + m] = Two{0.0, 0.0};
      if (cell(m, c)) y[m] = rd[m] + small_off(G, P0, A.F[0], c);
      if (cell(H + m, c)) y[H + m] = b[H + m];
    }
  };

  for (int it = 0; it < A.newton_maxit && !done; ++it) {
    // ---- residual and inverse centre blocks at the state (the assembly's formulas)
    Two R[2 * H];
    const Phys& P0 = P;   // of the finest grid
    double r2 = 0.0, zero = 0.0;
#pragma unroll
    for (int m = 0; m < 2 * H; ++m) {
      R[m] = Two{0.0, 0.0};
      SmallCell c;
      if (!cell(m, c)) continue;
      const CellState o = G.state(c.at);
      const double co = A.c_old[global(c)];
      const double rP = P0.rho0 + P0.drho * o.c, ro = P0.rho0 + P0.drho * co;
      double Rp = P0.vol * o.phi * (rP - ro) / P0.tau, Rc = P0.vol * o.phi * (rP * o.c - ro * co) / P0.tau;
      double D[4] = {0.0, P0.vol * o.phi * P0.drho / P0.tau, 0.0,
                     P0.vol * o.phi * (P0.rho0 + 2.0 * P0.drho * o.c) / P0.tau};
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const bool north = d >= 2, high = (d & 1) == 0;
        if (!(d == 0 ? c.i > 0 : d == 1 ? c.i < G.nx - 1 : d == 2 ? c.j > 0 : c.j < G.ny - 1)) continue;
        const CellState q = G.state(d == 0 ? c.w : d == 1 ? c.e : d == 2 ? c.s : c.n);
        FaceFlux f;
        if (high) face_flux(P0, north, q.p, q.c, q.phi, q.K, o.p, o.c, o.phi, o.K, f);
        else face_flux(P0, north, o.p, o.c, o.phi, o.K, q.p, q.c, q.phi, q.K, f);
        const double sg = high ? -1.0 : 1.0;
        Rp += sg * f.F;
        Rc += sg * f.G;
        D[0] += f.a;
        D[1] += sg * f.bF;
        D[2] += f.a * f.cup;
        D[3] += sg * (high ? f.dGH : f.dGL);
      }
      boundary_terms(P0, G.nx, c.i, c.j, o.p, o.c, o.phi, o.K, c.i == 0 ? A.uin[s] : 0.0, Rp, Rc, D);
      R[m] = Two{Rp, Rc};
      Di[m] = small_inverse(D);
      r2 += Rp * Rp + Rc * Rc;
    }
    sum2(r2, zero);
    bool act = r2 > 0.0;
    if (act) {
      // predicted: the next update would be within the tolerance
      if (A.pred_tol > 0.0 && last > 0.0 && r2prev > 0.0 && last * sqrt(r2 / r2prev) <= A.pred_tol) {
        done = true;
        break;
      }
      r2prev = r2;
    }
    if (act && fresh) {
      // ---- coarse operators: restricted states, the coarsest's inverse
      for (int l = 1; l <= nl; ++l) {
        const SmallGrid f = grid(l - 1), g = grid(l);
        for (int q = t; q < g.n; q += SMALL_THREADS) {
          const int J = q / g.nx, I = q - J * g.nx;
          Two v = f.pc[small_at(2 * I, 2 * J, f.nx, f.ny)] + f.pc[small_at(2 * I + 1, 2 * J, f.nx, f.ny)];
          v += f.pc[small_at(2 * I, 2 * J + 1, f.nx, f.ny)] + f.pc[small_at(2 * I + 1, 2 * J + 1, f.nx, f.ny)];
          g.pc[l < nl ? small_at(I, J, g.nx, g.ny) : q] = 0.25 * v;
        }
        lds_barrier();
      }
      double* const Jc = reinterpret_cast<double*>(scratch);   // [20][cells]
      if (t < C.n) {
        SmallCell c;   // row-major places
        c.j = t / C.nx;
        c.i = t - c.j * C.nx;
        c.at = t;
        c.w = c.i > 0 ? t - 1 : t;
        c.e = c.i < C.nx - 1 ? t + 1 : t;
        c.s = c.j > 0 ? t - C.nx : t;
        c.n = c.j < C.ny - 1 ? t + C.nx : t;
        double D[4];
        auto put = [&](int blk, double b0, double b1, double b2, double b3) {
          const double v[4] = {b0, b1, b2, b3};
#pragma unroll
          for (int e = 0; e < 4; ++e) Jc[(blk * 4 + e) * C.n + t] = v[e];
        };
        small_centre(C, phys(nl), A.F[nl], c, D,
                     [&](int side, double b0, double b1, double b2, double b3) { put(side + 1, b0, b1, b2, b3); });
        put(0, D[0], D[1], D[2], D[3]);
      }
      lds_barrier();
      tail_inverse<RC, TC>(Jc, Jc + 20 * C.n, C.n, C.nx, [&](int row, int k, double v) { inv[(size_t)row * nu + k] = v; });
      __threadfence_block();   // the inverse is read back by other threads of the workgroup
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 8; ++e) iv[e] = (t >> 3) < nu && part + 8 * e < nu ? inv[(size_t)(t >> 3) * nu + part + 8 * e] : 0.0;
    }
    // ---- BiCGStab: A dx = -R with the shadow residual R
    Two x[2 * H], r[2 * H], p[2 * H], v[2 * H];
#pragma unroll
    for (int m = 0; m < 2 * H; ++m) {
      x[m] = Two{0.0, 0.0};
      r[m] = p[m] = -R[m];
      v[m] = Two{0.0, 0.0};
    }
    double rho = -r2, al = 0.0, om = 0.0, beta = 0.0;
    for (int k = 0; k < A.krylov_maxit && act; ++k) {
      Two rd[H];
      if (k > 0) {
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) p[m] = r[m] + beta * (p[m] - om * v[m]);
      }
      cycle(p, rd);
      apply(p, rd, v);
      double rv = 0.0, ss = 0.0, d = 0.0;
#pragma unroll
      for (int m = 0; m < 2 * H; ++m) rv += R[m][0] * v[m][0] + R[m][1] * v[m][1];
      sum2(rv, d);
      al = 0.0;
      if (rv != 0.0 && isfinite(rv) && !(fabs(rv) <= A.breakdown * fabs(rho))) {
        al = rho / rv;
      } else {
        status = 2;   // (near) breakdown
        break;
      }
#pragma unroll
      for (int m = 0; m < 2 * H; ++m) {
        r[m] -= al * v[m];   // s
        ss += r[m][0] * r[m][0] + r[m][1] * r[m][1];
        SmallCell c;
        if (cell(m, c)) x[m] += al * G.x[c.at];
      }
      d = 0.0;
      sum2(ss, d);
      const bool at_half = ss <= A.rtol2 * r2;
      om = 0.0;
      if (!at_half) {
        Two y[2 * H];
        cycle(r, rd);
        apply(r, rd, y);
        double ts = 0.0, tt = 0.0;
#pragma unroll
        for (int m = 0; m < 2 * H; ++m) {
          ts += y[m][0] * r[m][0] + y[m][1] * r[m][1];
          tt += y[m][0] * y[m][0] + y[m][1] * y[m][1];
        }
        sum2(ts, tt);
        if (tt > 0.0) om = ts / tt;
        if (om != 0.0) {
#pragma unroll
          for (int m = 0; m < 2 * H; ++m) {
            SmallCell c;
            if (cell(m, c)) x[m] += om * G.x[c.at];
            r[m] -= om * y[m];
          }
        }
      }
      double rn = 0.0, rr = 0.0;
#pragma unroll
      for (int m = 0; m < 2 * H; ++m) {
        rn += R[m][0] * r[m][0] + R[m][1] * r[m][1];
        rr += r[m][0] * r[m][0] + r[m][1] * r[m][1];
      }
      sum2(rn, rr);
      kits += 1.0;
      if (at_half || rr <= A.rtol2 * r2) break;
      if (om == 0.0 || rn == 0.0 || !isfinite(rn)) {
        status = 2;   // breakdown before convergence
        break;
      }
      beta = (rn / rho) * (al / om);
      rho = rn;
    }
    // ---- damped update and convergence
    double mp = 0.0, mc = 0.0;
#pragma unroll
    for (int m = 0; m < 2 * H; ++m) {
      mp = larger(mp, fabs(x[m][0]));
      mc = larger(mc, fabs(x[m][1]));
    }
    max2(mp, mc);
    newtons += 1.0;
    if (!isfinite(mp) || !isfinite(mc)) {
      status = 3;
      done = true;
      break;
    }
    const double lam = mc > A.dc_max ? A.dc_max / mc : 1.0;
    const double size = fmax(mc, mp / A.p_ref);
    last = mc > A.dc_max ? 0.0 : size;
#pragma unroll
    for (int m = 0; m < 2 * H; ++m) {
      SmallCell c;
      if (cell(m, c)) G.pc[c.at] += lam * x[m];
    }
    lds_barrier();
    if (size <= A.newton_tol) done = true;
    else fresh = !(size <= A.jac_reuse);
  }

#pragma unroll
  for (int m = 0; m < 2 * H; ++m) {
    SmallCell c;
    if (!cell(m, c)) continue;
    const size_t q = global(c);
    const Two v = G.pc[c.at];
    A.p[q] = v[0];
    A.c[q] = v[1];
  }
  if (t == 0) {
    A.stats[(size_t)s * 4] += newtons;
    A.stats[(size_t)s * 4 + 1] += kits;
    if (status != 0) A.status[s] = status;
    if (!done && A.status[s] == 0) A.status[s] = 1;
  }
}

}  // namespace henry
