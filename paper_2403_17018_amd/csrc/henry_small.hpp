// Grids of up to 2048 cells: the whole Newton iteration of a time step in one launch, a workgroup
// per sample.  The state, the cycle's iterates and the coarse grids' states stay in LDS, the Krylov
// vectors in registers; every decision (convergence, damping, a fresh coarse operator, breakdown)
// is the sample's own, taken on the device.  Operator rows are formed from the state wherever they
// are used (henry_free.hpp): LDS would not hold the Jacobian.
//
// Launch by launch a step of these grids is some 110 launches of 3 to 5 us and four host reads,
// however few the samples, and a batch iterates until its hardest sample is done.  Milliseconds a
// solve, launch by launch (step_graphs 0) and with this kernel: 32x16 cells, 48 steps, 16 samples
// 40.3 and 7.2, 256 samples 49.0 and 9.5; 64x32 cells, 48 steps, 64 samples 44.7 and 19.6, 333
// samples 99 and 38.9; 24 steps, 1000 samples 133 and 51; 12 steps, 8000 samples 1518 and 250
// (32x16, 30000 samples: 869 and 426): it is taken for every batch size.  What bounds it is latency:
// one workgroup (LDS, registers) fits a compute unit and a step is a chain of passes, each a
// barrier, a few LDS reads and a row.  Of a step's 150 us at 32x16 (3 Newton, 3 BiCGStab iterations)
// the fine passes take 19, the coarser grids 26, the coarsest operator's inversion 24 (or
// twice), residuals and rows 45, the Krylov part 18.  Rows formed from the state in every pass
// instead of kept took 15 % more; with two cells of each colour a thread keeping them spills
// (64x32x64: 20.7 ms with one coarser grid's kept, 22.5 with two).  The step's start and its
// balance as launches of their own took 5 %.
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
  double *p, *c, *c_old;                        // state [cell][S], the step before's in, the new one out; its c
  double *hp[3], *hc[3];                        // the states of the steps before that, newest first
  int guess, order;                             // Newton's first guess: 0 the state, 1 linear, 2 a polynomial
  double gp, gc;                                // (k_extrapolate's factors)
  const double* uin;
  const double *phi[SMALL_LEVELS + 1], *K[SMALL_LEVELS + 1];
  double* inv;                                  // [S][n][n]: the coarsest operators' inverses
  int* status;
  double* stats;                                // [S][4]: Newton, BiCGStab iterations, balance defects
  int nu_pre, nu_post, newton_maxit, krylov_maxit;
  double rtol2, breakdown, newton_tol, pred_tol, dc_max, jac_reuse, p_ref, c_range_tol;
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

// Folds the values of a wavefront's lanes into lane 63's (0 where there is no lane to the left).
template <int CTRL, int ROWS>
__device__ __forceinline__ double lanes_left(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <typename Op>
__device__ __forceinline__ void wave_fold(double& a, double& b, Op&& op) {
  auto step = [&](auto ctrl, auto rows) {
    a = op(a, lanes_left<decltype(ctrl)::value, decltype(rows)::value>(a));
    b = op(b, lanes_left<decltype(ctrl)::value, decltype(rows)::value>(b));
  };
  step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // 1, 2, 4, 8 lanes in rows of 16
  step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // the rows' last lanes on
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
}

// k_extrapolate and k_extrapolate_poly for one value; the history h moves on by one.
__device__ __forceinline__ double small_guess(const SmallArgs& A, double un, double gamma, double* const (&h)[3], size_t q) {
  if (A.guess == 0) return un;
  if (A.guess == 1) {
    const double v = gamma != 0.0 ? un + gamma * (un - h[0][q]) : un;
    h[0][q] = un;
    return v;
  }
  const double a = A.order > 0 ? h[0][q] : un, b = A.order > 1 ? h[1][q] : a;
  const double v = A.order == 3   ? 4.0 * (un + b) - 6.0 * a - h[2][q]
                   : A.order == 2 ? 3.0 * (un - a) + b
                   : A.order == 1 ? 2.0 * un - a
                                  : un;
  if (h[2]) h[2][q] = b;
  h[1][q] = a;
  h[0][q] = un;
  return v;
}

struct SmallGrid {
  int nx, ny, n;
  Two *pc, *fk, *x, *b;
  __device__ __forceinline__ CellState state(int q) const {
    const Two u = pc[q], v = fk[q];
    return CellState{u[0], u[1], v[0], v[1]};
  }
};

// The four faces' terms of a cell; f(side, face, the neighbour's place, the fluxes through it L -> H),
// sides 0 W, 1 E, 2 S, 3 N.
template <typename Fn>
__device__ __forceinline__ void small_faces(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c,
                                            const CellState& own, Fn&& f) {
  const double km = 2.0 * F.inv_mu, qx = 0.5 * F.qd[0], qy = 0.5 * F.qd[1];
  const bool w = c.i > 0, e = c.i < G.nx - 1, s = c.j > 0, n = c.j < G.ny - 1;
  double flow, salt;
  {
    const Face a = face_flows<false>(P, F, w ? km : 0.0, w ? qx : 0.0, G.state(c.w), own, flow, salt);
    f(0, a, c.w, flow, salt);
  }
  {
    const Face a = face_flows<false>(P, F, e ? km : 0.0, e ? qx : 0.0, own, G.state(c.e), flow, salt);
    f(1, a, c.e, flow, salt);
  }
  {
    const Face a = face_flows<true>(P, F, s ? km : 0.0, s ? qy : 0.0, G.state(c.s), own, flow, salt);
    f(2, a, c.s, flow, salt);
  }
  {
    const Face a = face_flows<true>(P, F, n ? km : 0.0, n ? qy : 0.0, own, G.state(c.n), flow, salt);
    f(3, a, c.n, flow, salt);
  }
}
// the neighbours' part of the row times x
__device__ __forceinline__ Two small_off(const SmallGrid& G, const Phys& P, const FreePhys& F, const SmallCell& c) {
  Two y{0.0, 0.0};
  small_faces(G, P, F, c, G.state(c.at), [&](int side, const Face& f, int q, double, double) {
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
  small_faces(G, P, F, c, own, [&](int side, const Face& f, int, double, double) {
    const bool high = (side & 1) == 0;
    D[0] += f.a;
    D[1] += high ? -f.b : f.b;
    D[2] += f.ac;
    D[3] += high ? -f.dH : f.dL;
    blk(side, -f.a, high ? -f.b : f.b, -f.ac, high ? -f.dL : f.dH);
  });
  side_terms(P, F, G.nx, c.i, c.j, own, D);
}

// The neighbours' blocks of a row, kept in registers.
struct SmallRow {
  double o[4][4];
  __device__ __forceinline__ void set(int side, double b0, double b1, double b2, double b3) {
    o[side][0] = b0;
    o[side][1] = b1;
    o[side][2] = b2;
    o[side][3] = b3;
  }
  __device__ __forceinline__ Two off(const SmallGrid& G, const SmallCell& c) const {
    Two y{0.0, 0.0};
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const Two v = G.x[n == 0 ? c.w : n == 1 ? c.e : n == 2 ? c.s : c.n];
      y += Two{o[n][0] * v[0] + o[n][1] * v[1], o[n][2] * v[0] + o[n][3] * v[1]};
    }
    return y;
  }
};

// H: cells of each colour of the finest grid per thread (2 up to 2048 cells), or 0: one cell a thread
// (up to 512), whose rows of the operator and of the first two coarser grids' are kept in registers.
// RC, TC: the inversion's shape (tail_inverse).
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
  // this thread's cells: H red, then H black (their i and j packed: the rest is found anew each time,
  // which takes fewer registers), or one
  constexpr int NC = H ? 2 * H : 1, NR = H ? H : 1;   // cells, of them red (H = 0: or black)
  int ij[NC];
  SmallCell mine{};
  if constexpr (H > 0) {
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      const int u = t + SMALL_THREADS * (m % NR);
      const SmallCell c = small_cell(m / NR, u, G.nx, G.ny);
      ij[m] = u < half ? c.j << 16 | c.i : -1;
    }
  } else if (t < G.n) {
    mine = t < half ? small_cell(0, t, G.nx, G.ny) : small_cell(1, t - half, G.nx, G.ny);
  }
  auto cell = [&](int m, SmallCell& c) {
    if constexpr (H > 0) {
      int k = ij[m];
      asm volatile("" : "+v"(k));
      if (k < 0) return false;
      c = small_cell(m / NR, t + SMALL_THREADS * (m % NR), k & 0xffff, k >> 16, G.nx, G.ny);
      return true;
    } else {
      c = mine;
      return t < G.n;
    }
  };
  // its m-th cell of a colour; k: which of its cells that is
  auto cell_in = [&](int colour, int m, SmallCell& c, int& k) {
    if constexpr (H > 0) {
      k = colour * H + m;
      return cell(k, c);
    } else {
      k = 0;
      c = mine;
      return colour == 0 ? t < half : t >= half && t < G.n;
    }
  };
  auto global = [&](const SmallCell& c) { return ((size_t)c.j * G.nx + c.i) * S + s; };
  // its cell of a coarser smoothed grid
  auto coarse = [&](const SmallGrid& g, SmallCell& c) {
    const int h = g.n >> 1;
    if (t >= g.n) return false;
    c = t < h ? small_cell(0, t, g.nx, g.ny) : small_cell(1, t - h, g.nx, g.ny);
    return true;
  };
  // over the workgroup, for every thread; two buffers by turns, so one barrier each
  int flip = 0;
  auto fold2 = [&](double& a, double& b, auto&& op) {
    wave_fold(a, b, op);
    double* q = red + 16 * flip;
    flip ^= 1;
    if ((t & 63) == 63) {
      q[t >> 6] = a;
      q[8 + (t >> 6)] = b;
    }
    lds_barrier();
    a = b = 0.0;
#pragma unroll
    for (int k = 0; k < SMALL_THREADS / 64; ++k) {
      a = op(a, q[k]);
      b = op(b, q[8 + k]);
    }
  };
  auto larger = [](double a, double b) { return b > a || b != b ? b : a; };   // (of values >= 0; a NaN stays)
  auto sum2 = [&](double& a, double& b) { fold2(a, b, [](double u, double v) { return u + v; }); };
  auto max2 = [&](double& a, double& b) { fold2(a, b, larger); };

  // state and coefficients into LDS
  double co[NC] = {};   // the step before's c
#pragma unroll
  for (int m = 0; m < NC; ++m) {
    SmallCell c;
    if (!cell(m, c)) continue;
    const size_t q = global(c);
    const double pn = A.p[q], cn = A.c[q];
    A.c_old[q] = co[m] = cn;
    G.pc[c.at] = Two{small_guess(A, pn, A.gp, A.hp, q), small_guess(A, cn, A.gc, A.hc, q)};
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

  constexpr int KC = H ? 0 : 2;   // coarser grids whose rows are kept
  Inv2 Di[NC], Dc[2];             // inverse centre blocks
  SmallRow row, rc[2];
  SmallCell cc[2] = {};
  if constexpr (KC > 0) {
    for (int l = 1; l < nl && l <= KC; ++l) (void)coarse(grid(l), l == 1 ? cc[0] : cc[1]);
  }
  double iv[8];                                // the first eight terms of this thread's row of the inverse
  double* const inv = A.inv + (size_t)s * nu * nu;
  const double inflow = -(P.rho0 + P.drho * P.c_left) * A.uin[s] * P.uin_fac * P.hy;
  const int part = t & 7;
  double last = 0.0, r2prev = 0.0, newtons = 0.0, kits = 0.0;
  int status = 0;
  bool done = false, fresh = true;

  // ---- the coarser grids' part of a cycle: one copy of each kind of pass (the kernel's code is
  // read through by every wavefront, and what exceeds the instruction cache is fetched each time)
  auto gather = [&](const SmallGrid& f, int I, int J) {   // the two red children's residuals
    const int hx = f.nx >> 1;
    return scratch[2 * J * hx + I] + scratch[(2 * J + 1) * hx + I];
  };
  // the correction of the grid below prolonged onto a black cell of grid l
  auto prolong = [&](const SmallGrid& g, int l, const SmallCell& c) {
    const SmallGrid e = grid(l + 1);
    const int I = c.i >> 1, J = c.j >> 1;
    const int I2 = min(max(I + ((c.i & 1) ? 1 : -1), 0), e.nx - 1), J2 = min(max(J + ((c.j & 1) ? 1 : -1), 0), e.ny - 1);
    auto v = [&](int i, int j) { return e.x[l + 1 == nl ? j * e.nx + i : small_at(i, j, e.nx, e.ny)]; };
    g.x[c.at] += 0.5625 * v(I, J) + 0.1875 * (v(I2, J) + v(I, J2)) + 0.0625 * v(I2, J2);
  };
  const int cJ = t / C.nx, cI = t - cJ * C.nx;
  auto coarse_cycle = [&] {
#pragma unroll 1
    for (int q = 1; q < 2 * nl; ++q) {   // grids 1 .. nl - 1 down, nl, nl - 1 .. 1 up
      if (q == nl) {
        if (t < C.n) C.b[t] = gather(grid(nl - 1), cI, cJ);
        lds_barrier();
        const double* v = reinterpret_cast<const double*>(C.b);
        double* y = reinterpret_cast<double*>(C.x);
        for (int row = t >> 3, k = 0; row < nu; row += SMALL_THREADS / 8, ++k) {
          double acc = 0.0;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int w = part + 8 * e;
            if (w < nu) acc += (k == 0 ? iv[e] : inv[(size_t)row * nu + w]) * v[w];
          }
          for (int w = part + 64; w < nu; w += 8) acc += inv[(size_t)row * nu + w] * v[w];
#pragma unroll
          for (int o = 1; o < 8; o <<= 1) acc += __shfl_xor(acc, o);
          if (part == 0) y[row] = acc;
        }
        lds_barrier();
        continue;
      }
      const bool down = q < nl;
      const int l = down ? q : 2 * nl - q;
      const SmallGrid g = grid(l);
      const Phys Pl = phys(l);
      SmallCell c;
      const bool own = t < g.n;
      if (KC >= 1 && l == 1) c = cc[0];
      else if (KC >= 2 && l == 2) c = cc[1];
      else (void)coarse(g, c);
      const int colour = own ? t >= (g.n >> 1) : 2;
      if (down && own) {
        g.b[c.at] = gather(grid(l - 1), c.i, c.j);
      } else if (!down && colour == 1) {
        prolong(g, l, c);
      }
      if (!down) lds_barrier();
      const int passes = 2 * (down ? A.nu_pre : A.nu_post) + (down ? 1 : 0);   // the last one down: the residual
      auto sweep = [&](auto&& offd, const Inv2& D) {
        Two rd{0.0, 0.0};
#pragma unroll 1
        for (int k = 0; k < passes; ++k) {
          if (colour == (k & 1)) {
            Two r = g.b[c.at];
            if (!down || k > 0) r -= offd();
            if (down && k == 2 * A.nu_pre) {
              scratch[c.at] = r - rd;
            } else {
              rd = r;
              g.x[c.at] = D(r);
            }
          }
          lds_barrier();
        }
      };
      if (KC >= 1 && l == 1) {
        sweep([&] { return rc[0].off(g, c); }, Dc[0]);
      } else if (KC >= 2 && l == 2) {
        sweep([&] { return rc[1].off(g, c); }, Dc[1]);
      } else {
        Inv2 D{};
        if (own) {
          double d[4];
          small_centre(g, Pl, A.F[l], c, d, [](int, double, double, double, double) {});
          D = small_inverse(d);
        }
        sweep([&] { return small_off(g, Pl, A.F[l], c); }, D);
      }
    }
  };
  // ---- y = A M^{-1} b: b of this thread's fine cells in, the cycle's iterate in G.x.  D x of a red
  // cell is its right-hand side less the neighbours' part when it was last passed over (rd), so a
  // residual or product there is the neighbours' change; the last black pass leaves A x = b there.
  auto off = [&](const SmallCell& c) {
    if constexpr (H > 0) return small_off(G, P, A.F[0], c);
    else return row.off(G, c);
  };
  auto cycle = [&](const Two (&b)[NC], Two (&y)[NC]) {
    Two rd[NR];
    auto pass = [&](int colour, bool zero) {
#pragma unroll
      for (int m = 0; m < NR; ++m) {
        SmallCell c;
        int k;
        if (!cell_in(colour, m, c, k)) continue;
        Two r = b[k];
        if (!zero) r -= off(c);
        if (colour == 0) rd[m] = r;
        G.x[c.at] = Di[k](r);
      }
      lds_barrier();
    };
    pass(0, true);
    pass(1, false);
#pragma unroll 1
    for (int sw = 1; sw < A.nu_pre; ++sw) {
      pass(0, false);
      pass(1, false);
    }
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      SmallCell c;
      int k;
      if (cell_in(0, m, c, k)) scratch[c.at] = b[k] - rd[m] - off(c);
    }
    lds_barrier();
    coarse_cycle();
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      SmallCell c;
      int k;
      if (cell_in(1, m, c, k)) prolong(G, 0, c);
    }
    lds_barrier();
#pragma unroll 1
    for (int sw = 0; sw < A.nu_post; ++sw) {
      pass(0, false);
      pass(1, false);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) y[k] = b[k];   // (black cells; b is 0 where the thread has no cell)
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      SmallCell c;
      int k;
      if (cell_in(0, m, c, k)) y[k] = rd[m] + off(c);
    }
  };

  for (int it = 0; it < A.newton_maxit && !done; ++it) {
    // ---- residual, inverse centre blocks and kept rows at the state
    Two R[NC];
    double r2 = 0.0, zero = 0.0;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      R[m] = Two{0.0, 0.0};
      SmallCell c;
      if (!cell(m, c)) continue;
      const CellState o = G.state(c.at);
      const double v = A.F[0].vt * o.phi;
      const double rP = P.rho0 + P.drho * o.c;
      double Rp = v * (P.drho * (o.c - co[m])), Rc = v * (rP * o.c - (P.rho0 + P.drho * co[m]) * co[m]);
      double D[4] = {0.0, v * P.drho, 0.0, v * (P.rho0 + 2.0 * P.drho * o.c)};
      small_faces(G, P, A.F[0], c, o, [&](int side, const Face& f, int, double flow, double salt) {
        const bool high = (side & 1) == 0;
        Rp += high ? -flow : flow;
        Rc += high ? -salt : salt;
        D[0] += f.a;
        D[1] += high ? -f.b : f.b;
        D[2] += f.ac;
        D[3] += high ? -f.dH : f.dL;
        if (H == 0) row.set(side, -f.a, high ? -f.b : f.b, -f.ac, high ? -f.dL : f.dH);
      });
      const double dif = o.phi * A.F[0].side_dif;
      if (c.i == 0) {   // the inflow, and diffusion to c_left
        Rp += inflow;
        Rc += inflow * P.c_left + dif * rP * (o.c - P.c_left);
      }
      if (c.i == G.nx - 1) {   // the sea: what flows in has its density and concentration
        const double u = o.K * A.F[0].side_k * (o.p + P.rho1 * P.g * (-P.Ly + (c.j + 0.5) * P.hy));
        const double flow = (u < 0.0 ? P.rho1 : rP) * u;
        Rp += flow;
        Rc += flow * (u < 0.0 ? 1.0 : o.c);
        if (P.right_dir) Rc += dif * rP * (o.c - 1.0);
      }
      side_terms(P, A.F[0], G.nx, c.i, c.j, o, D);
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
#pragma unroll
      for (int l = 1; l <= KC; ++l) {
        if (l >= nl || t >= A.nx[l] * A.ny[l]) continue;
        double D[4];
        small_centre(grid(l), phys(l), A.F[l], cc[l - 1], D, [&](int side, double b0, double b1, double b2, double b3) {
          rc[l - 1].set(side, b0, b1, b2, b3);
        });
        Dc[l - 1] = small_inverse(D);
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
    // ---- BiCGStab: A dx = -R with the shadow residual R.  Each iteration is two half-steps, p
    // (half 0) and then s (half 1), through one copy of the cycle.
    Two x[NC], r[NC], p[NC], v[NC];
#pragma unroll
    for (int m = 0; m < NC; ++m) {
      x[m] = Two{0.0, 0.0};
      r[m] = p[m] = -R[m];
      v[m] = Two{0.0, 0.0};
    }
    double rho = -r2, al = 0.0, om = 0.0;
    for (int k = 0; k < 2 * A.krylov_maxit && act; ++k) {
      const bool second = k & 1;
      Two in[NC], y[NC];
#pragma unroll
      for (int m = 0; m < NC; ++m) in[m] = second ? r[m] : p[m];
      cycle(in, y);
      double a = 0.0, b = 0.0;   // half 0: (R, v); half 1: (t, s), (t, t)
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        const Two w = second ? r[m] : R[m];
        a += w[0] * y[m][0] + w[1] * y[m][1];
        b += y[m][0] * y[m][0] + y[m][1] * y[m][1];
      }
      sum2(a, b);
      double step;
      if (!second) {
        if (!(a != 0.0 && isfinite(a) && !(fabs(a) <= A.breakdown * fabs(rho)))) {
          status = 2;   // (near) breakdown
          break;
        }
        step = al = rho / a;
#pragma unroll
        for (int m = 0; m < NC; ++m) v[m] = y[m];
      } else {
        step = om = b > 0.0 ? a / b : 0.0;
      }
      double rn = 0.0, rr = 0.0;
      if (step != 0.0) {
#pragma unroll
        for (int m = 0; m < NC; ++m) {
          SmallCell c;
          if (cell(m, c)) x[m] += step * G.x[c.at];
          r[m] -= step * y[m];
        }
      }
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        rn += R[m][0] * r[m][0] + R[m][1] * r[m][1];
        rr += r[m][0] * r[m][0] + r[m][1] * r[m][1];
      }
      sum2(rn, rr);
      if (!second) {
        if (!(rr <= A.rtol2 * r2)) continue;
        kits += 1.0;
        break;
      }
      kits += 1.0;
      if (rr <= A.rtol2 * r2) break;
      if (om == 0.0 || rn == 0.0 || !isfinite(rn)) {
        status = 2;   // breakdown before convergence
        break;
      }
      const double beta = (rn / rho) * (al / om);
      rho = rn;
#pragma unroll
      for (int m = 0; m < NC; ++m) p[m] = r[m] + beta * (p[m] - om * v[m]);
    }
    // ---- damped update and convergence
    double mp = 0.0, mc = 0.0;
#pragma unroll
    for (int m = 0; m < NC; ++m) {
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
    for (int m = 0; m < NC; ++m) {
      SmallCell c;
      if (cell(m, c)) G.pc[c.at] += lam * x[m];
    }
    lds_barrier();
    if (size <= A.newton_tol) done = true;
    else fresh = !(size <= A.jac_reuse);   // the coarse operators'; the fine rows are always the state's
  }

  // ---- the new state out; mass balance and range (k_balance, k_fin_balance)
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0, low = 0.0, high = 0.0;
#pragma unroll
  for (int m = 0; m < NC; ++m) {
    SmallCell c;
    if (!cell(m, c)) continue;
    const size_t q = global(c);
    const CellState o = G.state(c.at);
    A.p[q] = o.p;
    A.c[q] = o.c;
    const double r = P.rho0 + P.drho * o.c, ro = P.rho0 + P.drho * co[m], dif = o.phi * A.F[0].side_dif;
    a0 += P.vol * o.phi * (r - ro);
    a1 += P.vol * o.phi * (r * o.c - ro * co[m]);
    if (c.i == 0) {
      a2 += P.tau * inflow;
      a3 += P.tau * (inflow * P.c_left + dif * r * (o.c - P.c_left));
    }
    if (c.i == G.nx - 1) {
      const double u = o.K * A.F[0].side_k * (o.p + P.rho1 * P.g * (-P.Ly + (c.j + 0.5) * P.hy));
      const double flow = (u < 0.0 ? P.rho1 : r) * u;
      double salt = flow * (u < 0.0 ? 1.0 : o.c);
      if (P.right_dir) salt += dif * r * (o.c - 1.0);
      a2 += P.tau * flow;
      a3 += P.tau * salt;
    }
    low = larger(low, -o.c);
    high = larger(high, o.c);
  }
  sum2(a0, a1);
  sum2(a2, a3);
  max2(low, high);
  if (t == 0) {
    const double scale = P.tau * P.rho0 * A.uin[s] * P.Ly;
    double* st = A.stats + (size_t)s * 4;
    st[0] += newtons;
    st[1] += kits;
    st[2] = fmax(st[2], fabs(a0 + a2) / scale);
    st[3] = fmax(st[3], fabs(a1 + a3) / scale);
    int v = status ? status : A.status[s];
    if (!done && v == 0) v = 1;
    if (v == 0 && (!(low <= A.c_range_tol) || !(high <= 1.0 + A.c_range_tol))) v = 4;
    A.status[s] = v;
  }
}

}  // namespace henry
