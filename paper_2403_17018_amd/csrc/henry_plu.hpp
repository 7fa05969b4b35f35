// Batched LU with partial pivoting of the coarsest multigrid operator (Gaussian elimination on
// the coarse grid, section 2.3): factorisation by one workgroup and solves by one wavefront per
// sample.
//
// Unknowns r = 2 q + component, cells q numbered along the grid's shorter side first, f of them.
// The five-point 2x2-block operator then has kl = 2 f + 1 scalar diagonals on either side.
// Entries farther out are exact zeros: partial pivoting never picks one, the multipliers of
// such rows are zero, and the rows of U end 2 kl columns right of the diagonal.  So the
// elimination of the full n x n matrix only ever changes a window of PLU_NB + kl rows by
// PLU_NB + 2 kl columns per panel of PLU_NB columns, and that window is all that is worked on:
// n kl^2 operations instead of n^3 / 3.  A 32x16 grid (n = 1024) x 128 samples takes 684 us to
// factor and 166 us to solve.  With the whole trailing matrix updated from memory, its 8 MB a
// sample streamed once per panel, it took 17 300 and 2 350; eliminated column by column in a
// band window, two barriers a column, about 3 000 and 530.
//
// Everything is held and computed in FP64; T is the type of the operator and of the vectors.
#pragma once

#include <hip/hip_runtime.h>

#include "henry_tail.hpp"   // tail_sample, lds_barrier

namespace henry {

typedef double mf_d4 __attribute__((ext_vector_type(4)));

constexpr int PLU_NB = 16;         // panel width: the trailing update works on 16 x 16 matrix-core tiles
constexpr int PLU_THREADS = 512;   // factorisation: wavefront 0 factors the panel, all update

struct PluShape {
  int n, n16;    // unknowns, and padded to whole panels with an identity block
  int kl, m;     // diagonals on a side; rows of the window
  int C;         // columns of the window, padded to whole tiles
  __host__ __device__ PluShape(int nx, int ny) {
    const int f = nx < ny ? nx : ny;
    n = 2 * nx * ny;
    n16 = (n + PLU_NB - 1) / PLU_NB * PLU_NB;
    kl = 2 * f + 1;
    m = PLU_NB + kl;
    C = (PLU_NB + 2 * kl + 15) / 16 * 16;
  }
  __host__ __device__ int panels() const { return n16 / PLU_NB; }
  __host__ __device__ int rows16() const { return (m + 15) / 16 * 16; }
  __host__ __device__ int ld() const { return C + 2; }   // LDS row stride of the window: no power of two
  // factors of a sample: per panel the window's L rows [m][NB] and U rows [NB][C]
  __host__ __device__ size_t panel_values() const { return (size_t)m * PLU_NB + (size_t)PLU_NB * C; }
  __host__ __device__ size_t values() const { return panels() * panel_values(); }
  __host__ __device__ size_t pivots() const { return (size_t)panels() * m; }
  __host__ __device__ size_t factor_lds() const {
    return ((size_t)rows16() * ld() + (size_t)PLU_NB * ld() + (size_t)rows16() * (PLU_NB + 1)) * sizeof(double) +
           rows16() * sizeof(int);
  }
  __host__ __device__ size_t solve_lds() const { return ((size_t)n16 + C + m) * sizeof(double); }
};

// scalar entry (r, c) of the coarse operator J [20][cells][S] (identity beyond n)
template <typename T>
__device__ __forceinline__ double plu_entry(const T* __restrict__ J, int nx, int ny, int S, int s, int r, int c) {
  const int nc = nx * ny, n = 2 * nc;
  if (r >= n || c >= n) return r == c ? 1.0 : 0.0;
  const bool xf = nx < ny;                 // x runs first
  const int f = xf ? nx : ny, slow = xf ? ny : nx;
  const int q = r >> 1, d = (c >> 1) - q, a = q % f, b = q / f;
  int blk = -1;
  if (d == 0) blk = 0;
  else if (d == -f && b > 0) blk = xf ? 3 : 1;
  else if (d == f && b < slow - 1) blk = xf ? 4 : 2;
  else if (d == -1 && a > 0) blk = xf ? 1 : 3;
  else if (d == 1 && a < f - 1) blk = xf ? 2 : 4;
  if (blk < 0) return 0.0;
  const int cell = xf ? b * nx + a : a * nx + b;
  return (double)J[(size_t)(blk * 4 + (r & 1) * 2 + (c & 1)) * nc * S + (size_t)cell * S + s];
}
// grid cell of unknown r
__device__ __forceinline__ int plu_cell(int nx, int ny, int r) {
  const int f = nx < ny ? nx : ny, q = r >> 1, a = q % f, b = q / f;
  return nx < ny ? b * nx + a : a * nx + b;
}

// lane `lane`'s value of v (lane uniform across the wavefront)
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return fmax(v, __longlong_as_double(((long long)hi << 32) | (unsigned int)lo));
}
// the largest of 64 lanes' values, in every lane
__device__ __forceinline__ double wave_max(double v) {
  v = dpp_max<0x111, 0xf>(v);   // lanes 1, 2, 4, 8 to the left in rows of 16
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);   // row 0's last lane into row 1, row 2's into row 3
  v = dpp_max<0x143, 0xc>(v);   // lane 31 into rows 2 and 3
  return lane_value(v, 63);
}

// Per panel: wavefront 0 holds the panel's rows in registers, RPL per lane, and eliminates its 16
// columns without barriers (pivot: the largest magnitude among rows not yet chosen, the first row
// on ties; rows are not moved, the chosen ones become rows 0 .. 15 of the panel and the others
// keep their order); then one thread per column forms U12, and the trailing window is updated
// on the matrix cores and stored 16 rows up and 16 columns left, where the next panel finds it
// beside the 16 rows that enter.  TPW: tiles per wavefront.  The panel's chain bounds it
// (16 columns of a 64-lane maximum, a broadcast row and an update).
template <typename T, int RPL, int TPW>
__global__ void __launch_bounds__(PLU_THREADS) k_plu_factor(int S, int nx, int ny, const T* __restrict__ J,
                                                            double* __restrict__ F, int* __restrict__ piv) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const PluShape sh(nx, ny);
  const int s = tail_sample(S), t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (s >= S) return;
  const int R16 = sh.rows16(), ld = sh.ld(), kl = sh.kl, m = sh.m, C = sh.C;
  double* W = reinterpret_cast<double*>(smem_raw);   // window [R16][ld]
  double* U = W + (size_t)R16 * ld;                  // this panel's rows of U [16][ld]
  double* P = U + (size_t)PLU_NB * ld;               // the factored panel [R16][17], in its row order
  int* src = reinterpret_cast<int*>(P + (size_t)R16 * (PLU_NB + 1));   // window row of each panel row
  double* Fs = F + (size_t)s * sh.values();
  int* ps = piv + (size_t)s * sh.pivots();
  for (int e = t; e < R16 * C; e += PLU_THREADS) {
    const int r = e / C, c = e - r * C, d = c - r;
    W[r * ld + c] = r < m && d >= -kl && d <= kl ? plu_entry(J, nx, ny, S, s, r, c) : 0.0;
  }
  for (int r = t; r < R16; r += PLU_THREADS) src[r] = r;
  lds_barrier();
  const int rt = (kl + 15) / 16, ct = C / 16 - 1;
  for (int k0 = 0; k0 < sh.n16; k0 += PLU_NB) {
    double* Lg = Fs + (size_t)(k0 / PLU_NB) * sh.panel_values();
    double* Ug = Lg + (size_t)m * PLU_NB;
    if (wave == 0) {
      double v[RPL][PLU_NB];
      bool open[RPL];
      int pos[RPL];
#pragma unroll
      for (int a = 0; a < RPL; ++a) {
        const int r = lane + 64 * a;
        open[a] = r < m;
        pos[a] = -1;
#pragma unroll
        for (int c = 0; c < PLU_NB; ++c) v[a][c] = r < m ? W[r * ld + c] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < PLU_NB; ++j) {
        double best = -1.0;
#pragma unroll
        for (int a = 0; a < RPL; ++a) best = fmax(best, open[a] ? fabs(v[a][j]) : -1.0);
        best = wave_max(best);
        int pa = 0, pl = 0;   // the first open row of that magnitude (the first open one if none compares equal: NaN)
        bool found = false;
#pragma unroll
        for (int a = 0; a < RPL; ++a) {
          const unsigned long long hit = __ballot(open[a] && fabs(v[a][j]) == best);
          if (!found && hit) {
            found = true;
            pa = a;
            pl = __ffsll((long long)hit) - 1;
          }
        }
        if (!found) {
#pragma unroll
          for (int a = 0; a < RPL; ++a) {
            const unsigned long long any = __ballot(open[a]);
            if (!found && any) {
              found = true;
              pa = a;
              pl = __ffsll((long long)any) - 1;
            }
          }
        }
        double u[PLU_NB];
#pragma unroll
        for (int c = j; c < PLU_NB; ++c) {
          double w = v[0][c];
          if constexpr (RPL > 1) {
            const double w1 = v[1][c];
            w = pa ? w1 : w;
          }
          u[c] = lane_value(w, pl);
        }
        const double rp = u[j] != 0.0 ? 1.0 / u[j] : 0.0;   // an exactly singular column leaves L = 0 (and 1 / 0 in U)
#pragma unroll
        for (int a = 0; a < RPL; ++a) {
          if (a == pa && lane == pl) {
            open[a] = false;
            pos[a] = j;
          }
          if (open[a]) {
            const double l = v[a][j] * rp;
            v[a][j] = l;
#pragma unroll
            for (int c = j + 1; c < PLU_NB; ++c) v[a][c] -= l * u[c];
          }
        }
      }
      int before = PLU_NB;   // rows not chosen follow in their order
#pragma unroll
      for (int a = 0; a < RPL; ++a) {
        const unsigned long long rest = __ballot(open[a]);
        if (open[a]) pos[a] = before + __popcll(rest & ((1ull << lane) - 1));
        before += __popcll(rest);
        if (pos[a] >= 0) {
          src[pos[a]] = lane + 64 * a;
#pragma unroll
          for (int c = 0; c < PLU_NB; ++c) P[pos[a] * (PLU_NB + 1) + c] = v[a][c];
        }
      }
    }
    lds_barrier();
    // U12 = L11^{-1} A12, one thread per column; the factors go out
    for (int c = PLU_NB + t; c < C; c += PLU_THREADS) {
      double u[PLU_NB];
#pragma unroll
      for (int i = 0; i < PLU_NB; ++i) {
        double x = W[src[i] * ld + c];
#pragma unroll
        for (int k = 0; k < i; ++k) x -= P[i * (PLU_NB + 1) + k] * u[k];
        u[i] = x;
        U[i * ld + c] = x;
        Ug[(size_t)i * C + c] = x;
      }
    }
    for (int e = t; e < m * PLU_NB; e += PLU_THREADS) {
      const int r = e / PLU_NB, c = e - r * PLU_NB;
      const double x = P[r * (PLU_NB + 1) + c];
      Lg[e] = x;
      // U's diagonal as its reciprocal: infinite for a singular operator, whose solves are not finite
      if (r < PLU_NB) Ug[(size_t)r * C + c] = r == c ? 1.0 / x : x;
    }
    for (int r = t; r < m; r += PLU_THREADS) ps[(size_t)(k0 / PLU_NB) * m + r] = src[r];
    lds_barrier();
    // trailing window: lane l of a 16x16x4 step holds A[l % 16][l / 16] and B[l / 16][l % 16], and
    // of the result rows l / 16 + 4 v, column l % 16
    mf_d4 acc[TPW];
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int tile = wave + 8 * u;
      if (tile < rt * ct) {
        const int r0 = PLU_NB + 16 * (tile / ct), c0 = PLU_NB + 16 * (tile % ct);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = W[src[r0 + (lane >> 4) + 4 * v] * ld + c0 + (lane & 15)];
#pragma unroll
        for (int kk = 0; kk < PLU_NB; kk += 4) {
          const double a = -P[(r0 + (lane & 15)) * (PLU_NB + 1) + kk + (lane >> 4)];
          const double b = U[(kk + (lane >> 4)) * ld + c0 + (lane & 15)];
          acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[u], 0, 0, 0);
        }
      }
    }
    lds_barrier();
    const int k1 = k0 + PLU_NB;
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int tile = wave + 8 * u;
      if (tile < rt * ct) {
        const int r0 = 16 * (tile / ct), c0 = 16 * (tile % ct);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = r0 + (lane >> 4) + 4 * v;
          if (r < kl) W[r * ld + c0 + (lane & 15)] = acc[u][v];
        }
      }
    }
    for (int e = t; e < kl * 16; e += PLU_THREADS) W[(e >> 4) * ld + C - 16 + (e & 15)] = 0.0;
    for (int e = t; e < PLU_NB * C; e += PLU_THREADS) {   // the rows that enter
      const int q = e / C, c = e - q * C, r = kl + q, d = c - r;
      W[r * ld + c] = k1 < sh.n16 && d >= -kl && d <= kl ? plu_entry(J, nx, ny, S, s, k1 + r, k1 + c) : 0.0;
    }
    lds_barrier();
  }
}

// x = A^{-1} b (TR: A^{-T} b) with k_plu_factor's factors, one wavefront per sample; b, x:
// [2][cells][S].  Panel by panel, lane r holding the window's row r (RPL rows a lane): the row
// order of the panel, sixteen steps of substitution with the pivot row's value taken from its
// lane, nothing but the wavefront's own LDS in between.  Rows of U are taken four lanes to a
// row.  A solve is this chain of panels; each panel's factors are loaded before the chain of
// the panel before it ends.
template <typename T, bool TR, int RPL>
__global__ void __launch_bounds__(64) k_plu_solve(int S, int nx, int ny, const double* __restrict__ F,
                                                  const int* __restrict__ piv, const T* __restrict__ b,
                                                  T* __restrict__ x) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const PluShape sh(nx, ny);
  const int s = tail_sample(S), lane = threadIdx.x;
  if (s >= S) return;
  const int m = sh.m, C = sh.C, np = sh.panels();
  double* y = reinterpret_cast<double*>(smem_raw);   // [n16] and zeros for the last windows
  const size_t N = (size_t)nx * ny * S;
  const double* Fs = F + (size_t)s * sh.values();
  const int* ps = piv + (size_t)s * sh.pivots();
  for (int r = lane; r < sh.n16 + C + m; r += 64)
    y[r] = r < sh.n ? (double)b[(r & 1) * N + (size_t)plu_cell(nx, ny, r) * S + s] : 0.0;
  const int i4 = lane >> 2, part = lane & 3;
  auto Lp = [&](int p) { return Fs + (size_t)p * sh.panel_values(); };
  auto Up = [&](int p) { return Fs + (size_t)p * sh.panel_values() + (size_t)m * PLU_NB; };
  auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  fence();
  if (!TR) {
    double l[RPL][PLU_NB];
    int q[RPL];
    auto load = [&](int p) {
#pragma unroll
      for (int a = 0; a < RPL; ++a) {
        const int r = lane + 64 * a;
        q[a] = ps[(size_t)p * m + (r < m ? r : 0)];
#pragma unroll
        for (int c = 0; c < PLU_NB; ++c) l[a][c] = Lp(p)[(size_t)(r < m ? r : 0) * PLU_NB + c];
      }
    };
    load(0);
    for (int p = 0; p < np; ++p) {   // L y = P b
      const int k0 = p * PLU_NB;
      double v[RPL];
#pragma unroll
      for (int a = 0; a < RPL; ++a) v[a] = y[k0 + q[a]];
      fence();
#pragma unroll
      for (int j = 0; j < PLU_NB; ++j) {
        const double vj = lane_value(v[0], j);
#pragma unroll
        for (int a = 0; a < RPL; ++a)
          if (a > 0 || lane > j) v[a] -= l[a][j] * vj;
      }
#pragma unroll
      for (int a = 0; a < RPL; ++a)
        if (lane + 64 * a < m) y[k0 + lane + 64 * a] = v[a];
      fence();
      if (p + 1 < np) load(p + 1);
    }
    for (int p = np - 1; p >= 0; --p) {   // U x = y
      const int k0 = p * PLU_NB;
      const double* u = Up(p) + (size_t)i4 * C;
      double d[PLU_NB], acc = 0.0;
#pragma unroll
      for (int c = 0; c < PLU_NB; ++c) d[c] = u[c];
#pragma unroll 8
      for (int c = PLU_NB + part; c < C; c += 4) acc += u[c] * y[k0 + c];
      acc += __shfl_xor(acc, 1);
      acc += __shfl_xor(acc, 2);
      double v = y[k0 + i4] - acc;
#pragma unroll
      for (int j = PLU_NB - 1; j >= 0; --j) {
        const double xj = lane_value(v * d[j], 4 * j);   // the diagonal holds its reciprocal
        if (i4 == j) v = xj;
        else if (i4 < j) v -= d[j] * xj;
      }
      fence();
      if (part == 0) y[k0 + i4] = v;
      fence();
    }
  } else {
    for (int p = 0; p < np; ++p) {   // U^T z = b
      const int k0 = p * PLU_NB;
      const double* u = Up(p);
      double d[PLU_NB], v = lane < PLU_NB ? y[k0 + lane] : 0.0;
#pragma unroll
      for (int j = 0; j < PLU_NB; ++j) d[j] = u[(size_t)j * C + (lane < PLU_NB ? lane : 0)];
      double z[PLU_NB];
#pragma unroll
      for (int j = 0; j < PLU_NB; ++j) {
        z[j] = lane_value(v * d[j], j);
        if (lane == j) v = z[j];
        else if (lane > j) v -= d[j] * z[j];
      }
      fence();
      if (lane < PLU_NB) y[k0 + lane] = v;
      for (int c = PLU_NB + lane; c < C; c += 64) {
        double a = y[k0 + c];
#pragma unroll
        for (int j = 0; j < PLU_NB; ++j) a -= u[(size_t)j * C + c] * z[j];
        y[k0 + c] = a;
      }
      fence();
    }
    for (int r = sh.n16 + lane; r < sh.n16 + C + m; r += 64) y[r] = 0.0;
    fence();
    for (int p = np - 1; p >= 0; --p) {   // L^T w = z, then the panel's row order undone
      const int k0 = p * PLU_NB;
      const double* l = Lp(p);
      double acc = 0.0, d[PLU_NB];
#pragma unroll
      for (int j = 0; j < PLU_NB; ++j) d[j] = l[(size_t)j * PLU_NB + i4];   // L11(j, i4)
#pragma unroll 4
      for (int r = PLU_NB + part; r < m; r += 4) acc += l[(size_t)r * PLU_NB + i4] * y[k0 + r];
      acc += __shfl_xor(acc, 1);
      acc += __shfl_xor(acc, 2);
      double v = y[k0 + i4] - acc;
#pragma unroll
      for (int j = PLU_NB - 1; j > 0; --j) {
        const double wj = lane_value(v, 4 * j);
        if (i4 < j) v -= d[j] * wj;
      }
      double w[RPL];
      int q[RPL];
#pragma unroll
      for (int a = 0; a < RPL; ++a) {
        const int r = lane + 64 * a;
        q[a] = ps[(size_t)p * m + (r < m ? r : 0)];
      }
      fence();
      if (part == 0) y[k0 + i4] = v;
      fence();
#pragma unroll
      for (int a = 0; a < RPL; ++a) w[a] = y[k0 + (lane + 64 * a < m ? lane + 64 * a : 0)];
      fence();
#pragma unroll
      for (int a = 0; a < RPL; ++a)
        if (lane + 64 * a < m) y[k0 + q[a]] = w[a];
      fence();
    }
  }
  for (int r = lane; r < sh.n; r += 64) x[(r & 1) * N + (size_t)plu_cell(nx, ny, r) * S + s] = (T)y[r];
}

}  // namespace henry
