// The coarse end of the multigrid cycle in one launch, one workgroup per sample.
//
// Below about 512 cells a grid's smoother pass is a few microseconds of launch and memory
// latency around a few hundred cells of arithmetic: a V-cycle spent seven launches per coarse
// grid and a serial banded solve there, and each assembly two launches per grid and a serial
// factorisation.  Here a workgroup takes one sample through all of those grids at once:
//   k_tail_setup  restricts the state, assembles the grids' Jacobians and inverts the coarsest;
//   k_mg_tail     runs the cycle.  Each thread owns one cell per grid; its Jacobian row and
//                 right-hand side stay in registers from the way down to the way up, the
//                 iterates live in LDS, and LDS barriers alone separate the passes.
// The coarsest operator is applied as an explicit inverse, a product without serial steps.  It
// is computed, held and applied in FP64 for FP32 cycles too.
//
// The Jacobians are stored sample by sample, in the order of the threads that read them back:
// with the samples fastest, each of a wavefront's lanes would touch a 128-byte line of its own
// for 8 bytes, which bounded the cycle: from a 32x16 grid down to 8x4 with 64 samples, 22.5 us
// that way, 10.7 us this way, and 67 us in 13 launches (333 samples: 41, 19.6 and about 100 us).
// What bounds it now is the chain of some twenty short passes between barriers.
#pragma once

#include <hip/hip_runtime.h>

#include "henry_kernels.hpp"

namespace henry {

// Barrier for LDS traffic only: this wavefront's LDS operations complete, then every wavefront
// of the workgroup arrives.  Unlike __syncthreads() it does not wait for global loads and stores
// in flight (prefetches, results nobody in the kernel reads back), which would put a memory
// latency on every step.  The memory clobber keeps the compiler from moving memory accesses
// across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int TAIL_LEVELS = 3;     // smoothed grids in one launch at most
constexpr int TAIL_CELLS = 512;    // cells of the finest of them at most: one per thread
constexpr int TAIL_NMAX = 128;     // unknowns of the coarsest grid at most (its inverse: n^2 values per sample)

template <typename T>
struct TailArgs {
  int S, nu_pre, nu_post;
  int nx[TAIL_LEVELS + 1], ny[TAIL_LEVELS + 1];   // the smoothed grids, then the coarsest
  const T* J;                                     // k_tail_setup's Jacobians, tail_values() per sample
  const double* inv;                              // [S][n][n]: row r of the inverse (of the transpose when TR)
};

// Workgroups b, b + 8, ... run on one XCD, which gets one eighth of the batch, consecutive samples:
// those of a 128-byte line mostly share its L2.  With whole lines to an XCD (runs of a multiple of
// 16 samples) a batch of 16 ran on one of them, its 16 workgroups behind one L2: 48 steps of 32x16
// cells by k_small_step took 7.7 ms, and 6.7 this way.
__host__ __device__ inline int tail_chunk(int S) { return (S + 7) / 8; }
__device__ __forceinline__ int tail_sample(int S) { return (int)(blockIdx.x & 7) * tail_chunk(S) + (int)(blockIdx.x >> 3); }

template <typename T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};

// One cell's row of a grid's operator (of its transpose when TR): the diagonal block with the
// reciprocal of its determinant, and the four neighbours' blocks (zero outside the grid).
template <typename T>
struct TailRow {
  T d[4], rdet, o[4][4];
  int q[4];       // neighbours' cells (where there is none, another neighbour's: a value that is
                  // set whenever the row is used, for the zero block to multiply)
  int cell;       // -1: this thread owns no cell of the grid
  T b0, b1;
};

// Thread t's cell of a grid of nx (even) x ny cells: red cells ((i + j) even) on the lower half
// of the threads, black ones on the upper half, so that a colour pass fills whole wavefronts.
__device__ __forceinline__ bool tail_cell(int t, int nx, int ny, int& i, int& j) {
  const int hx = nx >> 1, half = hx * ny;
  if (t >= 2 * half) return false;
  const int colour = t >= half ? 1 : 0, u = t - colour * half;
  j = u / hx;
  i = 2 * (u - j * hx) + ((j + colour) & 1);
  return true;
}
// the thread of cell (i, j)
__device__ __forceinline__ int tail_thread(int i, int j, int nx, int ny) {
  const int hx = nx >> 1;
  return ((i + j) & 1) * hx * ny + j * hx + (i >> 1);
}
// Jacobian values per sample: 20 planes of the cells in thread order for each smoothed grid
__host__ __device__ inline size_t tail_values(const int* nx, const int* ny, int nl) {
  size_t n = 0;
  for (int l = 0; l < nl; ++l) n += (size_t)20 * nx[l] * ny[l];
  return n;
}

// J: this sample's 20 planes of the grid
template <typename T, bool TR>
__device__ __forceinline__ void tail_load_row(TailRow<T>& r, const T* __restrict__ J, int nx, int ny) {
  int i, j;
  r.cell = -1;
  if (!tail_cell(threadIdx.x, nx, ny, i, j)) return;
  r.cell = j * nx + i;
  const int nc = nx * ny;
  const bool ok[4] = {i > 0, i < nx - 1, j > 0, j < ny - 1};
  const int di[4] = {-1, 1, 0, 0}, dj[4] = {0, 0, -1, 1};
#pragma unroll
  for (int n = 0; n < 5; ++n) {
    const bool on = n == 0 || ok[n - 1];
    const int slot = !on || n == 0 ? 0 : TR ? (n == 1 ? 2 : n == 2 ? 1 : n == 3 ? 4 : 3) : n;
    const int row = TR && n > 0 && on ? tail_thread(i + di[n - 1], j + dj[n - 1], nx, ny) : (int)threadIdx.x;
    const T* p = J + slot * 4 * nc + row;
    const T e0 = p[0], e1 = p[TR ? 2 * nc : nc], e2 = p[TR ? nc : 2 * nc], e3 = p[3 * nc];
    T* o = n == 0 ? r.d : r.o[n - 1];
    o[0] = on ? e0 : (T)0;
    o[1] = on ? e1 : (T)0;
    o[2] = on ? e2 : (T)0;
    o[3] = on ? e3 : (T)0;
    if (n > 0) r.q[n - 1] = r.cell + (on ? dj[n - 1] * nx + di[n - 1] : i > 0 ? -1 : 1);
  }
}

template <typename T>
__device__ __forceinline__ Pair<T> tail_off(const TailRow<T>& r, const Pair<T>* x) {
  Pair<T> y{(T)0, (T)0};
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const Pair<T> v = x[r.q[n]];
    y.a += r.o[n][0] * v.a + r.o[n][1] * v.b;
    y.b += r.o[n][2] * v.a + r.o[n][3] * v.b;
  }
  return y;
}
// D^{-1} (b - y)
template <typename T>
__device__ __forceinline__ Pair<T> tail_diag(const TailRow<T>& r, const Pair<T>& y) {
  const T r0 = r.b0 - y.a, r1 = r.b1 - y.b;
  return Pair<T>{(r.d[3] * r0 - r.d[1] * r1) * r.rdet, (r.d[0] * r1 - r.d[2] * r0) * r.rdet};
}

// LDS (Pair<T>): the iterates of every smoothed grid, the coarsest grid's right-hand side and
// solution, and one residual vector of the finest of them.
template <typename T>
__host__ inline size_t tail_lds(const TailArgs<T>& A, int nl) {
  size_t n = 0;
  for (int l = 0; l < nl; ++l) n += (size_t)A.nx[l] * A.ny[l];
  n += 2 * (size_t)A.nx[nl] * A.ny[nl] + (nl > 0 ? (size_t)A.nx[0] * A.ny[0] : 0);
  return n * sizeof(Pair<T>);
}
// Threads: one per cell of the finest grid, and eight per unknown of the coarsest where 512 allow.
template <typename T>
__host__ inline int tail_threads(const TailArgs<T>& A, int nl) {
  const int n = 2 * A.nx[nl] * A.ny[nl];
  int t = nl > 0 ? A.nx[0] * A.ny[0] : 0;
  if (t < 8 * n) t = 8 * n < TAIL_CELLS ? 8 * n : TAIL_CELLS;
  return (t + 63) / 64 * 64;
}

// x = M^{-1} b on the grids of A from x = 0 (TR: with the transposed operators).  b, x: vectors
// [2][cells of grid 0][S].  nx of every smoothed grid is even.
template <typename T, bool TR, int NL>
__global__ void __launch_bounds__(TAIL_CELLS) k_mg_tail(TailArgs<T> A, const T* __restrict__ b, T* __restrict__ x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int s = tail_sample(A.S), t = threadIdx.x;
  if (s >= A.S) return;
  Pair<T>* X[NL + 1];
  {
    Pair<T>* p = reinterpret_cast<Pair<T>*>(smem_raw);
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      X[l] = p;
      p += A.nx[l] * A.ny[l];
    }
    X[NL] = p;   // solution of the coarsest grid
  }
  const int nc = A.nx[NL] * A.ny[NL], n = 2 * nc;
  Pair<T>* bc = X[NL] + nc;
  Pair<T>* rs = bc + nc;
  // every global load of the cycle is issued here
  TailRow<T> r[NL > 0 ? NL : 1];
  if constexpr (NL > 0) {
    const T* J = A.J + (size_t)s * tail_values(A.nx, A.ny, NL);
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      tail_load_row<T, TR>(r[l], J, A.nx[l], A.ny[l]);
      J += 20 * A.nx[l] * A.ny[l];
    }
    const size_t N = (size_t)A.nx[0] * A.ny[0] * A.S;
    if (r[0].cell >= 0) {
      r[0].b0 = b[(size_t)r[0].cell * A.S + s];
      r[0].b1 = b[N + (size_t)r[0].cell * A.S + s];
    }
  }
  const int part = t & 7, rstep = blockDim.x >> 3;
  const double* inv = A.inv + (size_t)s * n * n;
  double iv[8];   // the first eight terms of this thread's first row of the inverse
#pragma unroll
  for (int e = 0; e < 8; ++e) iv[e] = (t >> 3) < n && part + 8 * e < n ? inv[(size_t)(t >> 3) * n + part + 8 * e] : 0.0;
  // down: pre-smoothing from x = 0, then the red residuals (black ones vanish after the black
  // pass; a red one is minus the off-diagonal part when x_red was D^{-1} b) summed over children
  if constexpr (NL > 0) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const int half = (A.nx[l] >> 1) * A.ny[l];
      const bool own = r[l].cell >= 0, red = own && t < half, black = own && t >= half;
      const T det = r[l].d[0] * r[l].d[3] - r[l].d[1] * r[l].d[2];
      r[l].rdet = (T)1 / det;
      if (red) X[l][r[l].cell] = tail_diag(r[l], Pair<T>{(T)0, (T)0});
      lds_barrier();
      if (black) X[l][r[l].cell] = tail_diag(r[l], tail_off(r[l], X[l]));
      lds_barrier();
      for (int sw = 1; sw < A.nu_pre; ++sw) {
        if (red) X[l][r[l].cell] = tail_diag(r[l], tail_off(r[l], X[l]));
        lds_barrier();
        if (black) X[l][r[l].cell] = tail_diag(r[l], tail_off(r[l], X[l]));
        lds_barrier();
      }
      if (red) {
        Pair<T> y = tail_off(r[l], X[l]);
        if (A.nu_pre > 1) {
          const Pair<T> v = X[l][r[l].cell];
          y.a += r[l].d[0] * v.a + r[l].d[1] * v.b - r[l].b0;
          y.b += r[l].d[2] * v.a + r[l].d[3] * v.b - r[l].b1;
        }
        rs[r[l].cell] = Pair<T>{-y.a, -y.b};
      }
      lds_barrier();
      // the coarse cell's two red children; the next write to rs is at least two barriers away
      auto gather = [&](int cell) {
        const int nxc = A.nx[l + 1], J = cell / nxc, I = cell - J * nxc;
        const Pair<T> u = rs[2 * J * A.nx[l] + 2 * I], v = rs[(2 * J + 1) * A.nx[l] + 2 * I + 1];
        return Pair<T>{u.a + v.a, u.b + v.b};
      };
      if (l + 1 < NL) {
        if (r[l + 1 < NL ? l + 1 : l].cell >= 0) {
          TailRow<T>& c = r[l + 1 < NL ? l + 1 : l];
          const Pair<T> v = gather(c.cell);
          c.b0 = v.a;
          c.b1 = v.b;
        }
      } else if (t < nc) {
        bc[t] = gather(t);
      }
    }
  } else {
    const size_t N = (size_t)nc * A.S;
    if (t < nc) bc[t] = Pair<T>{b[(size_t)t * A.S + s], b[N + (size_t)t * A.S + s]};
  }
  lds_barrier();
  // coarsest grid: eight threads per row of the inverse
  {
    const T* v = reinterpret_cast<const T*>(bc);
    T* y = reinterpret_cast<T*>(X[NL]);
    for (int row = t >> 3, k = 0; row < n; row += rstep, ++k) {
      double acc = 0.0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = part + 8 * e;
        if (c < n) acc += (k == 0 ? iv[e] : inv[(size_t)row * n + c]) * (double)v[c];
      }
      for (int c = part + 64; c < n; c += 8) acc += inv[(size_t)row * n + c] * (double)v[c];
#pragma unroll
      for (int off = 1; off < 8; off <<= 1) acc += __shfl_xor(acc, off);
      if (part == 0) y[row] = (T)acc;
    }
  }
  lds_barrier();
  // up: the prolonged correction on the black cells (the red pass overwrites the red ones), then
  // the post-smoothing sweeps
  if constexpr (NL > 0) {
#pragma unroll
    for (int l = NL - 1; l >= 0; --l) {
      const int half = (A.nx[l] >> 1) * A.ny[l];
      const bool own = r[l].cell >= 0, red = own && t < half, black = own && t >= half;
      if (black) {
        const int nx = A.nx[l], nxc = A.nx[l + 1], nyc = A.ny[l + 1];
        const int j = r[l].cell / nx, i = r[l].cell - j * nx, I = i >> 1, J = j >> 1;
        int I2 = I + ((i & 1) ? 1 : -1), J2 = J + ((j & 1) ? 1 : -1);
        I2 = I2 < 0 ? 0 : (I2 >= nxc ? nxc - 1 : I2);
        J2 = J2 < 0 ? 0 : (J2 >= nyc ? nyc - 1 : J2);
        const Pair<T>* e = X[l + 1];
        const Pair<T> e0 = e[J * nxc + I], e1 = e[J * nxc + I2], e2 = e[J2 * nxc + I], e3 = e[J2 * nxc + I2];
        const T w9 = (T)0.5625, w3 = (T)0.1875, w1 = (T)0.0625;
        Pair<T> v = X[l][r[l].cell];
        v.a += w9 * e0.a + w3 * e1.a + w3 * e2.a + w1 * e3.a;
        v.b += w9 * e0.b + w3 * e1.b + w3 * e2.b + w1 * e3.b;
        X[l][r[l].cell] = v;
      }
      lds_barrier();
      for (int sw = 0; sw < A.nu_post; ++sw) {
        if (red) X[l][r[l].cell] = tail_diag(r[l], tail_off(r[l], X[l]));
        lds_barrier();
        if (black) X[l][r[l].cell] = tail_diag(r[l], tail_off(r[l], X[l]));
        lds_barrier();
      }
    }
    const size_t N = (size_t)A.nx[0] * A.ny[0] * A.S;
    if (r[0].cell >= 0) {
      const Pair<T> v = X[0][r[0].cell];
      x[(size_t)r[0].cell * A.S + s] = v.a;
      x[N + (size_t)r[0].cell * A.S + s] = v.b;
    }
  } else {
    const size_t N = (size_t)nc * A.S;
    if (t < nc) {
      const Pair<T> v = X[0][t];
      x[(size_t)t * A.S + s] = v.a;
      x[N + (size_t)t * A.S + s] = v.b;
    }
  }
}

template <typename T>
struct TailSetup {
  int S, nl, transposed;
  int nx[TAIL_LEVELS + 1], ny[TAIL_LEVELS + 1];   // as in TailArgs
  const double *p, *c;                            // state on the next finer grid [cell][S]
  const double *phi[TAIL_LEVELS + 1], *K[TAIL_LEVELS + 1];
  T* J;
  double* inv;
};
constexpr int SETUP_THREADS = 512;
// LDS (doubles): the states of two grids by turns; then the coarsest grid's blocks [20][nc] and the
// inversion's pivot rows and columns, double buffered.
template <typename T>
__host__ inline size_t setup_lds(const TailSetup<T>& A) {
  size_t a = 0, b = 0;
  for (int l = 0; l <= A.nl; ++l) {
    size_t& v = l & 1 ? b : a;
    const size_t n = 4 * (size_t)A.nx[l] * A.ny[l];
    v = v > n ? v : n;
  }
  const size_t nc = (size_t)A.nx[A.nl] * A.ny[A.nl];
  return (a + b + 20 * nc + 2 * 4 * TAIL_NMAX) * sizeof(double);
}

// Inverse of an operator of ncc cells (rows of nxc) given by its blocks Jc [20][ncc] in LDS, by a
// workgroup of SETUP_THREADS: Gauss-Jordan by 2x2 blocks without interchanges, as the banded LU
// (the diagonal blocks of this operator are nonsingular and its pressure part is an M-matrix).
// Each of 16 x TC threads holds RC row cells (tr, tr + 16, ..) of two column cells (tc, tc + TC) in
// registers; a step's pivot rows and columns go through LDS (`pivots`, 8 TAIL_NMAX doubles), double
// buffered, so the serial chain is ncc steps of one barrier, a 2x2 inverse and the multiply-adds.
// RC = 2, TC = 16 take 32 cells, RC = 4, TC = 32 take 64.  With the pivots' register slots chosen
// at run time k_tail_setup took 38 us instead of 27.  out(row, column, value).
template <int RC, int TC, typename Out>
__device__ __forceinline__ void tail_inverse(const double* Jc, double* pivots, int ncc, int nxc, Out&& out) {
  struct alignas(16) Blk { double v[4]; };
  Blk* prow = reinterpret_cast<Blk*>(pivots);          // [2][TAIL_NMAX / 2]: blocks of the pivot row
  Blk* pcol = prow + TAIL_NMAX;                        // [2][TAIL_NMAX / 2]: blocks of the pivot column
  const int t = threadIdx.x;
  const bool worker = t < 16 * TC;
  const int tr = t / TC, tc = t % TC;
  double W[RC][2][4];
#pragma unroll
  for (int a = 0; a < RC; ++a)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int q = tr + 16 * a, c = tc + TC * h, d = c - q, qi = q % nxc;
      int blk = -1;
      if (d == 0) blk = 0;
      else if (d == -1 && qi > 0) blk = 1;
      else if (d == 1 && qi < nxc - 1) blk = 2;
      else if (d == -nxc) blk = 3;
      else if (d == nxc) blk = 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) W[a][h][e] = worker && blk >= 0 && q < ncc && c < ncc ? Jc[(blk * 4 + e) * ncc + q] : 0.0;
    }
#pragma unroll
  for (int kh = 0; kh < RC; ++kh) {   // pivots 16 kh .. 16 kh + 15: row cell slot kh, column slot kc
    constexpr int PER = TC / 16;
    const int kc = kh / PER;
    for (int kk = 0; kk < 16 && 16 * kh + kk < ncc; ++kk) {
      const int k = 16 * kh + kk;
      Blk* pr = prow + (kk & 1) * (TAIL_NMAX / 2);
      Blk* pc = pcol + (kk & 1) * (TAIL_NMAX / 2);
      const bool prw = worker && tr == kk, pcl = worker && tc == 16 * (kh % PER) + kk;
      // publish the pivot row and the pivot column; the column becomes the identity's (in the
      // pivot row) and zero, from which the update makes the inverse's
      if (prw)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) pr[tc + TC * h].v[e] = W[kh][h][e];
      if (pcl)
#pragma unroll
        for (int a = 0; a < RC; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            pc[tr + 16 * a].v[e] = W[a][kc][e];
            W[a][kc][e] = 0.0;
          }
      lds_barrier();
      if (!worker) continue;
      const Blk d = pr[k];
      Blk p[2] = {pr[tc], pr[tc + TC]};
      if (pcl) {
        p[kc].v[0] = p[kc].v[3] = 1.0;
        p[kc].v[1] = p[kc].v[2] = 0.0;
      }
      const double rdet = 1.0 / (d.v[0] * d.v[3] - d.v[1] * d.v[2]);
      const double i00 = d.v[3] * rdet, i01 = -d.v[1] * rdet, i10 = -d.v[2] * rdet, i11 = d.v[0] * rdet;
      double g[2][4];   // D^{-1} times the pivot row's blocks
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        g[h][0] = i00 * p[h].v[0] + i01 * p[h].v[2];
        g[h][1] = i00 * p[h].v[1] + i01 * p[h].v[3];
        g[h][2] = i10 * p[h].v[0] + i11 * p[h].v[2];
        g[h][3] = i10 * p[h].v[1] + i11 * p[h].v[3];
      }
#pragma unroll
      for (int a = 0; a < RC; ++a) {
        const Blk l = pc[tr + 16 * a];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            W[a][h][e] -= l.v[2 * (e >> 1)] * g[h][e & 1];
            W[a][h][e] -= l.v[2 * (e >> 1) + 1] * g[h][2 + (e & 1)];
          }
      }
      if (prw)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) W[kh][h][e] = g[h][e];
    }
  }
  if (!worker) return;
#pragma unroll
  for (int a = 0; a < RC; ++a)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int q = tr + 16 * a, c = tc + TC * h;
      if (q >= ncc || c >= ncc) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) out(2 * q + (e >> 1), 2 * c + (e & 1), W[a][h][e]);
    }
}

// Restricted states (means of the four children), rediscretised Jacobians of the grids of A (the
// assembly's formulas), and the inverse of the coarsest operator (of its transpose when
// `transposed`).  The inversion's serial chain bounds the launch: 27 us for 16 samples from a 16x8
// grid down, where the banded factorisation alone took 56 us and the assemblies four launches more.
template <typename T, int RC, int TC>
__global__ void __launch_bounds__(SETUP_THREADS) k_tail_setup(TailSetup<T> A, Phys P) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int s = tail_sample(A.S), t = threadIdx.x, S = A.S;
  if (s >= S) return;
  double* base[2];
  size_t na = 0, nb = 0;
  for (int l = 0; l <= A.nl; ++l) {
    const size_t n = 4 * (size_t)A.nx[l] * A.ny[l];
    if (l & 1) nb = nb > n ? nb : n;
    else na = na > n ? na : n;
  }
  base[0] = reinterpret_cast<double*>(smem_raw);
  base[1] = base[0] + na;
  const int ncc = A.nx[A.nl] * A.ny[A.nl], nu = 2 * ncc;
  double* Jc = base[1] + nb;   // [20][ncc]
  T* Jg = A.J + (size_t)s * tail_values(A.nx, A.ny, A.nl);
  for (int l = 0; l <= A.nl; ++l) {
    const int nx = A.nx[l], ny = A.ny[l], n = nx * ny;
    double* st = (l & 1) ? base[1] : base[0];   // [p, c, phi, K][cell]
    int i = 0, j = 0;
    bool own;
    if (l < A.nl) {
      own = tail_cell(t, nx, ny, i, j);
    } else {
      own = t < n;
      j = t / nx;
      i = t - j * nx;
    }
    const int cell = j * nx + i;
    if (own) {
      double sp = 0.0, sc = 0.0;
      const int fnx = 2 * nx;
      const double* prev = (l & 1) ? base[0] : base[1];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int ch = (2 * j + (q >> 1)) * fnx + 2 * i + (q & 1);
        sp += l == 0 ? A.p[(size_t)ch * S + s] : prev[ch];
        sc += l == 0 ? A.c[(size_t)ch * S + s] : prev[4 * n + ch];
      }
      st[cell] = 0.25 * sp;
      st[n + cell] = 0.25 * sc;
      st[2 * n + cell] = A.phi[l][(size_t)cell * S + s];
      st[3 * n + cell] = A.K[l][(size_t)cell * S + s];
    }
    lds_barrier();
    if (own) {
      Phys Pl = P;
      Pl.hx = P.Lx / nx;
      Pl.hy = P.Ly / ny;
      Pl.vol = Pl.hx * Pl.hy;
      const double pP = st[cell], cP = st[n + cell], phP = st[2 * n + cell], KP = st[3 * n + cell];
      double D[4] = {0.0, Pl.vol * phP * Pl.drho / Pl.tau, 0.0,
                     Pl.vol * phP * (Pl.rho0 + 2.0 * Pl.drho * cP) / Pl.tau};
      auto put = [&](int blk, double b0, double b1, double b2, double b3) {
        const double v[4] = {b0, b1, b2, b3};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (l < A.nl) Jg[(blk * 4 + e) * n + t] = (T)v[e];
          else Jc[(blk * 4 + e) * n + t] = (double)(T)v[e];   // the operator as T holds it
        }
      };
#pragma unroll
      for (int d = 0; d < 4; ++d) {   // west, east, south, north: the cell is the high, low, high, low side
        const bool north = d >= 2, high = (d & 1) == 0;
        const bool on = d == 0 ? i > 0 : d == 1 ? i < nx - 1 : d == 2 ? j > 0 : j < ny - 1;
        if (!on) {
          put(d + 1, 0.0, 0.0, 0.0, 0.0);
          continue;
        }
        const int q = cell + (d == 0 ? -1 : d == 1 ? 1 : d == 2 ? -nx : nx);
        const double pQ = st[q], cQ = st[n + q], phQ = st[2 * n + q], KQ = st[3 * n + q];
        FaceFlux f;
        if (high) face_flux(Pl, north, pQ, cQ, phQ, KQ, pP, cP, phP, KP, f);
        else face_flux(Pl, north, pP, cP, phP, KP, pQ, cQ, phQ, KQ, f);
        const double sg = high ? -1.0 : 1.0;
        D[0] += f.a;
        D[1] += sg * f.bF;
        D[2] += f.a * f.cup;
        D[3] += sg * (high ? f.dGH : f.dGL);
        put(d + 1, -f.a, sg * f.bF, -f.a * f.cup, sg * (high ? f.dGL : f.dGH));
      }
      double r0 = 0.0, r1 = 0.0;
      boundary_terms(Pl, nx, i, j, pP, cP, phP, KP, 0.0, r0, r1, D);
      put(0, D[0], D[1], D[2], D[3]);
    }
    Jg += 20 * n;
  }
  lds_barrier();
  double* out = A.inv + (size_t)s * nu * nu;
  tail_inverse<RC, TC>(Jc, Jc + 20 * ncc, ncc, A.nx[A.nl], [&](int r, int k, double v) {
    out[A.transposed ? (size_t)k * nu + r : (size_t)r * nu + k] = v;
  });
}

}  // namespace henry
