// Several passes of the multigrid cycle over one grid in one launch: a workgroup takes a strip of
// columns for 8 samples and marches through the grid's rows, each pass one row behind the pass
// before it, so that a cell's state, right-hand side and iterate are read from memory once for all
// of them.  Rows are formed from the state (henry_free.hpp), once for all passes.
//
// 256x128 cells, 512 samples: the pre-smoothing sweep with the restriction takes 333 us (three
// launches of a pass each 562), two post-smoothing sweeps with the prolongation 498 us (four
// launches 961); in FP32 (rows formed in FP64, kept rounded) 319 and 444 us.  They move 1.01 and
// 1.28 GB at least, 210 and 270 us at the 4.7 TB/s of a copy; counters show 1.15 and 1.75 GB (FP32
// 1.12 and 1.62) and the vector units busy a third of the time.  What bounds them is
// the issue of two wavefronts a SIMD, all that the registers of a column's rows leave (182 and 243),
// each waiting for its own LDS reads, barrier and instructions most of the time.  Keeping the rows'
// coefficients in registers costs that residency but a third of the arithmetic of forming them in
// every pass (464 and 487 + 421 us); 32-column workgroups waste 8 of 32 columns on halos but are
// tied by smaller barriers than 64-column ones (498 and 552 us).
#pragma once

#include <hip/hip_runtime.h>

#include "henry_free.hpp"
#include "henry_tail.hpp"

namespace henry {

constexpr int MARCH_NS = 8;   // samples a workgroup: 64-byte segments of a cell's row of samples

// PRE: the pre-smoothing sweep from x = 0 and the restricted residual (x: the black half alone).
// POST: two post-smoothing sweeps, the coarse correction e prolonged onto the black cells as they
// are read.
enum { MARCH_PRE = 0, MARCH_POST = 1 };
template <int KIND>
constexpr int march_passes() { return KIND == MARCH_PRE ? 3 : 4; }

// T: the cycle's precision (iterate, coefficients kept and passes; rows are formed in FP64), TB: the
// right-hand side's.
template <typename T, typename TB>
struct MarchArgs {
  int nx, ny, S;
  int halo;            // columns recomputed on each side of a strip (0: one strip is the grid)
  int width, nstrip;   // columns of a strip and strips
  int rows, nseg;      // rows of a segment and segments
  int nsb;             // blocks of MARCH_NS samples
  Phys P;
  FreePhys F;
  FreeOp op;
  const TB* b;
  const T *xin, *e;   // xin: the black cells' values before the sweep
  T *x, *bH;          // x: not xin (strips read their neighbours' cells)
  // (two sample blocks, segment) pairs, each a run of 2 nstrip blocks on one XCD
  __host__ __device__ int pairs() const { return (nsb + 1) / 2 * nseg; }
  __host__ __device__ int blocks() const { return (pairs() + 7) / 8 * 8 * 2 * nstrip; }
};

constexpr int MARCH_WAVES32 = 2;   // wavefronts a SIMD that the FP32 cycle's registers are kept to
constexpr int MARCH_UNROLL = 6;   // steps a group: even, and a row's time in registers
__host__ __device__ constexpr int march_groups(int steps) { return (steps + MARCH_UNROLL - 1) / MARCH_UNROLL; }

typedef double Two __attribute__((ext_vector_type(2)));

template <int KIND, int NC, typename T>
__host__ __device__ constexpr int march_lds() {
  return MARCH_NS * NC * (4 * 16 + MARCH_UNROLL * 2 * (int)sizeof(T)) +
         (KIND == MARCH_PRE ? MARCH_NS * NC / 2 * 2 * (int)sizeof(T) : 0);
}

// A face's share in the rows on its sides, low (L) and high (H): A_LH = [-a, b; -ac, dH],
// A_HL = [-a, -b; -ac, -dL], D_L += [a, b; ac, dL], D_H += [a, -b; ac, -dH].
struct Face {
  double a, b, ac, dL, dH;
};
// km: 2 / mu, qd: half of F.qd; both 0 for a face that is not there.  flow, salt: the fluid and salt
// mass fluxes L -> H.
template <bool NORTH>
__device__ __forceinline__ Face face_flows(const Phys& P, const FreePhys& F, double km, double qd, const CellState& L,
                                           const CellState& H, double& flow, double& salt) {
  const double kf = L.K * H.K * rcp_normal(L.K + H.K) * km;
  const double q = (L.phi + H.phi) * qd;
  const double rf = P.rho0 + F.hd * (L.c + H.c);
  const double rk = rf * kf;
  double uA = kf * F.w[NORTH] * (L.p - H.p), grav = 0.0;
  if (NORTH) {
    grav = rk * F.gA;
    uA -= grav;
  }
  const double flux = rf * uA;
  const double cup = flux >= 0.0 ? L.c : H.c;
  const double dif = rf * q;
  flow = flux;
  salt = flux * cup - dif * (H.c - L.c);
  Face f;
  f.b = F.hd * (uA - grav);
  const double g = f.b * cup - F.hd * q * (H.c - L.c);
  f.dL = g + (fmax(flux, 0.0) + dif);
  f.dH = g + (fmin(flux, 0.0) - dif);
  f.a = rk * F.w[NORTH];
  f.ac = f.a * cup;
  return f;
}
template <bool NORTH>
__device__ __forceinline__ Face face_terms(const Phys& P, const FreePhys& F, double km, double qd, const CellState& L,
                                           const CellState& H) {
  double flow, salt;
  return face_flows<NORTH>(P, F, km, qd, L, H, flow, salt);
}

// A row's coefficients as kept: FaceRow's of the west and east neighbours, its north face's both
// sides, and the inverse of its centre block.
template <typename T>
struct MarchRow {
  T wa, wb, wc, wd, ea, eb, ec, ed;
  T na, nb, nc, nL, nH;
  T i00, i01, i10, i11;
  T b0, b1, x0, x1;
};

// Empty asm statements keep their order: values pinned one after the other are computed one after
// the other, where the scheduler would interleave them and need the registers of all at once.
template <typename V>
__device__ __forceinline__ void pin(V& a, V& b, V& c, V& d) {
  asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
template <typename V>
__device__ __forceinline__ void pin(V& a, V& b) {
  asm volatile("" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void pin(CellState& s) { pin(s.p, s.c, s.phi, s.K); }

// A thread owns a column.  At step t row t enters; row t - 1, whose neighbours are all there, gets
// its operator row (three faces, the south one kept from the row below, and the inverse of the
// centre block), kept in registers for all passes; pass k works on row t - 1 - k.  The passes of a
// column are due at every other step (colours alternate along the column as the passes do along
// the rows): wavefronts hold columns of one parity, due together, and a step's passes read only
// values of the step before and of their own column.  The neighbours' states and iterates come
// through LDS: one barrier a step.  Rows and columns outside the strip's halo hold finite values
// that reach no result: out-of-range loads are clamped to the grid, a missing face's terms are zero.
template <int KIND, int NC, typename T, typename TB>
__global__ void __launch_bounds__(MARCH_NS * NC, sizeof(T) == 8 ? 2 : MARCH_WAVES32) k_march(MarchArgs<T, TB> A) {
  typedef T TwoT __attribute__((ext_vector_type(2)));
  constexpr int K = march_passes<KIND>(), NT = MARCH_NS * NC, RR = MARCH_UNROLL;
  extern __shared__ Two msh[];   // states of two rows [2][p c, phi K][thread], x of RR rows, residuals
  TwoT* const shx = (TwoT*)(msh + 4 * NT);
  const int nx = A.nx, ny = A.ny, S = A.S;
  // The strips of two sample blocks follow one another on one XCD: they share 128-byte lines and
  // read each other's columns, the latter then from its L2.
  const int run = 2 * A.nstrip, seq = blockIdx.x >> 3, half = (A.nsb + 1) / 2;
  const int pair = seq / run * 8 + (blockIdx.x & 7), sb = 2 * (pair % half) + (seq & 1);
  if (pair >= A.pairs() || sb >= A.nsb) return;
  const int x0 = (seq % run >> 1) * A.width, ybeg = (pair / half) * A.rows;
  const int yend = min(ny, ybeg + A.rows), ylo = max(0, ybeg - K), yhi = min(ny, yend + K);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int par = w >= NT / 128 ? 1 : 0;
  const int hc = (w - par * (NT / 128)) * (64 / MARCH_NS) + lane / MARCH_NS, sl = lane % MARCH_NS;
  const int gi = x0 - A.halo + 2 * hc + par, s = min(sb * MARCH_NS + sl, S - 1);
  const int gc = min(max(gi, 0), nx - 1);
  const int odd = (x0 - A.halo + par) & 1;
  const bool mine = sb * MARCH_NS + sl < S && gi >= x0 && gi < min(x0 + A.width, nx);
  // LDS places, even columns of the strip first; a missing neighbour's is the other one's
  const int own = par * (NT / 2) + hc * MARCH_NS + sl;
  int west = par ? hc * MARCH_NS + sl : NT / 2 + max(hc - 1, 0) * MARCH_NS + sl;
  int east = par ? min(hc + 1, NC / 2 - 1) * MARCH_NS + sl : NT / 2 + hc * MARCH_NS + sl;
  if (gi <= 0) west = east;
  if (gi >= nx - 1) east = west;
  const size_t N = (size_t)nx * ny * S, row_step = (size_t)nx * S;
  const unsigned off = (unsigned)gc * S + s;   // march_takes() keeps a row under 4 GiB
  const int ncx = nx >> 1, ncy = ny >> 1;
  const size_t Nc = (size_t)ncx * ncy * S, crow = (size_t)ncx * S;
  const int I = gc >> 1, I2 = min(max(I + ((gc & 1) ? 1 : -1), 0), ncx - 1);
  const unsigned offI = (unsigned)I * S + s, offI2 = (unsigned)I2 * S + s;
  // scalar row address + 32-bit offset (the empty asm keeps the offset from being widened outside
  // the loop, which would cost a 64-bit vector pointer per array)
  auto ld = [](const auto* row, unsigned o) {
    unsigned bytes = o * (unsigned)sizeof(*row);
    asm volatile("" : "+v"(bytes));
    return *(decltype(row))((const char*)row + bytes);
  };
  auto st = [](T* row, unsigned o, T v) {
    unsigned bytes = o * (unsigned)sizeof(T);
    asm volatile("" : "+v"(bytes));
    *(T*)((char*)row + bytes) = v;
  };

  const CellState none{0.0, 0.0, 1.0, 1.0};   // below the first row: finite values, no zero pivot
  MarchRow<T> h[RR] = {};
  CellState cur = none, nst = none;           // of row t - 1, of the row loaded
  Face south = {};                            // the face below row t - 1, not rounded to T
  TB nb0 = 0, nb1 = 0;
  T nx0 = 0, nx1 = 0, e0[4] = {}, e1[4] = {};
  auto add_e = [&] {   // the next row's cell is black
    nx0 += (T)0.5625 * e0[0] + (T)0.1875 * (e0[1] + e0[2]) + (T)0.0625 * e0[3];
    nx1 += (T)0.5625 * e1[0] + (T)0.1875 * (e1[1] + e1[2]) + (T)0.0625 * e1[3];
    pin(nx0, nx1);
  };
  size_t lrow = ylo * row_step;   // the row to load
  int lr = ylo;
  auto load = [&](bool black) {
    // (opaque, so that the addresses stay scalar)
    asm volatile("" : "+s"(lrow));
    nst = CellState{ld(A.op.p + lrow, off), ld(A.op.c + lrow, off), ld(A.op.phi + lrow, off), ld(A.op.K + lrow, off)};
    nb0 = ld(A.b + lrow, off);
    nb1 = ld(A.b + N + lrow, off);
    if (KIND == MARCH_POST && black) {
      nx0 = ld(A.xin + lrow, off);
      nx1 = ld(A.xin + N + lrow, off);
      const int J = lr >> 1, J2 = min(max(J + ((lr & 1) ? 1 : -1), 0), ncy - 1);
      const T *u = A.e + J * crow, *v = A.e + J2 * crow;
      e0[0] = ld(u, offI);
      e0[1] = ld(u, offI2);
      e0[2] = ld(v, offI);
      e0[3] = ld(v, offI2);
      e1[0] = ld(u + Nc, offI);
      e1[1] = ld(u + Nc, offI2);
      e1[2] = ld(v + Nc, offI);
      e1[3] = ld(v + Nc, offI2);
    }
    if (lr + 1 < yhi) {
      ++lr;
      lrow += row_step;
    }
  };
  const double km = 2.0 * A.F.inv_mu, km_w = gi > 0 ? km : 0.0, km_e = gi < nx - 1 ? km : 0.0;
  const double qd_w = gi > 0 ? 0.5 * A.F.qd[0] : 0.0, qd_e = gi < nx - 1 ? 0.5 * A.F.qd[0] : 0.0;
  // a column whose first due step is the second is one phase behind
  const bool late = !((ylo + odd) & 1);
  size_t trow = ylo * row_step;   // row t's
  // x of the row `o` rows behind in a neighbour column, which is one phase off
  auto nx_row = [&](int phase) { return shx + (late ? (phase + 1) % RR : (phase + RR - 1) % RR) * NT; };
  // ph even: the column's passes are due
  auto step = [&](auto ph, int t) {
    constexpr int PH = decltype(ph)::value;
    constexpr bool due = PH % 2 == 0;
    auto at = [&](int o) -> MarchRow<T>& { return h[(PH + RR - o) % RR]; };   // row t - o of the own column
    const CellState entered = nst;
    {
      MarchRow<T>& c = at(0);
      c.b0 = (T)nb0;
      c.b1 = (T)nb1;
      c.x0 = c.x1 = (T)0;
      if (KIND == MARCH_POST && due) {   // a black cell
        c.x0 = nx0;
        c.x1 = nx1;
        shx[PH * NT + own] = TwoT{c.x0, c.x1};
      }
      Two* sh = msh + PH % 2 * 2 * NT + own;
      sh[0] = Two{entered.p, entered.c};
      sh[NT] = Two{entered.phi, entered.K};
    }
    load(!due);
    // a pass's west, east and south terms are old: those of the last passes are taken before the new
    // row is formed, which frees their coefficients for it
    T p0[K], p1[K];
    auto gather = [&](int k) {
      const TwoT* sh = nx_row((PH + RR - 1 - k) % RR);
      const TwoT xw = sh[west], xe = sh[east];
      const MarchRow<T>&c = at(k + 1), &cs = at(k + 2);
      p0[k] = c.eb * xe[1] - c.ea * xe[0] - c.wb * xw[1] - c.wa * xw[0] - cs.nb * cs.x1 - cs.na * cs.x0;
      p1[k] = c.ed * xe[1] - c.ec * xe[0] - c.wd * xw[1] - c.wc * xw[0] - cs.nL * cs.x1 - cs.nc * cs.x0;
      pin(p0[k], p1[k]);
    };
    if constexpr (due) {
#pragma unroll
      for (int k = K - 1; k >= 2; --k) gather(k);
    }
    {
      MarchRow<T>& c = at(1);
      pin(cur);
      const Two* sh = msh + PH % 2 * 2 * NT;   // the neighbours' row t - 1: they are a phase off
      auto nb = [&](int o) {
        const Two u = sh[o], v = sh[NT + o];
        return CellState{u[0], u[1], v[0], v[1]};
      };
      const double vol = A.F.vt * cur.phi;
      double D[4] = {south.a, vol * A.P.drho - south.b, south.ac,
                     vol * (A.P.rho0 + 2.0 * A.P.drho * cur.c) - south.dH};
      {
        const Face f = face_terms<false>(A.P, A.F, km_w, qd_w, nb(west), cur);
        c.wa = (T)f.a;
        c.wb = (T)f.b;
        c.wc = (T)f.ac;
        c.wd = (T)f.dL;
        D[0] += f.a;
        D[1] -= f.b;
        D[2] += f.ac;
        D[3] -= f.dH;
        pin(c.wa, c.wb, c.wc, c.wd);
        pin(D[0], D[1], D[2], D[3]);
        pin(cur);
      }
      {
        const Face f = face_terms<false>(A.P, A.F, km_e, qd_e, cur, nb(east));
        c.ea = (T)f.a;
        c.eb = (T)f.b;
        c.ec = (T)f.ac;
        c.ed = (T)f.dH;
        D[0] += f.a;
        D[1] += f.b;
        D[2] += f.ac;
        D[3] += f.dL;
        pin(c.ea, c.eb, c.ec, c.ed);
        pin(D[0], D[1], D[2], D[3]);
        pin(cur);
      }
      const bool inner = t > ylo && t < ny;
      south = face_terms<true>(A.P, A.F, inner ? km : 0.0, inner ? 0.5 * A.F.qd[1] : 0.0, cur, entered);
      c.na = (T)south.a;
      c.nb = (T)south.b;
      c.nc = (T)south.ac;
      c.nL = (T)south.dL;
      c.nH = (T)south.dH;
      D[0] += south.a;
      D[1] += south.b;
      D[2] += south.ac;
      D[3] += south.dL;
      pin(c.na, c.nb, c.nc, c.nL);
      pin(D[0], D[1], D[2], D[3]);
      side_terms(A.P, A.F, nx, gi, t - 1, cur, D);
      const double rdet = 1.0 / (D[0] * D[3] - D[1] * D[2]);
      c.i00 = (T)(D[3] * rdet);
      c.i01 = (T)(-D[1] * rdet);
      c.i10 = (T)(-D[2] * rdet);
      c.i11 = (T)(D[0] * rdet);
      pin(c.i00, c.i01, c.i10, c.i11);
      cur = entered;
    }
    if constexpr (due) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int r = t - 1 - k;
        MarchRow<T>& c = at(k + 1);
        T y0 = 0, y1 = 0;
        if (!(KIND == MARCH_PRE && k == 0)) {
          if (k < 2) gather(k);
          const MarchRow<T>& cn = at(k);
          y0 = p0[k] + c.nb * cn.x1 - c.na * cn.x0;
          y1 = p1[k] + c.nH * cn.x1 - c.nc * cn.x0;
        }
        const bool out = mine && r >= ybeg && r < yend;
        if (!(KIND == MARCH_PRE && k == 2)) {
          const T r0 = c.b0 - y0, r1 = c.b1 - y1;
          c.x0 = c.i00 * r0 + c.i01 * r1;
          c.x1 = c.i10 * r0 + c.i11 * r1;
          pin(c.x0, c.x1);
          if (k < K - 1) shx[(PH + RR - 1 - k) % RR * NT + own] = TwoT{c.x0, c.x1};
          if ((KIND == MARCH_PRE ? k == 1 : k >= 2) && out) {
            const size_t row = trow - (k + 1) * row_step;
            st(A.x + row, off, c.x0);
            st(A.x + N + row, off, c.x1);
          }
        } else if (out) {
          // the two red cells of a coarse cell are (even, even) and (odd, odd): the first leaves its
          // residual for the other, due in the next step
          TwoT* keep = shx + RR * NT + ((gi - x0) >> 1) * MARCH_NS + sl;
          if (gi & 1) {
            const TwoT v = *keep;
            const size_t row = (r >> 1) * crow;
            st(A.bH + row, offI, v[0] - y0);
            st(A.bH + Nc + row, offI, v[1] - y1);
          } else {
            *keep = TwoT{-y0, -y1};
          }
        }
      }
    }
    if (KIND == MARCH_POST && !due) add_e();   // (its loads have had the step's time)
    trow += row_step;
    lds_barrier();
  };
#pragma unroll
  for (int k = 0; k < RR; ++k) shx[k * NT + own] = TwoT{(T)0, (T)0};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    msh[2 * k * NT + own] = Two{none.p, none.c};
    msh[(2 * k + 1) * NT + own] = Two{none.phi, none.K};
  }
  lds_barrier();
  // A column whose first due step is the second enters its first row ahead of the unrolled steps,
  // the others wait one barrier more at the end.  Whole groups of steps are run (exits between them
  // would keep every register of the group alive); those past the last row write nothing.
  int t = ylo;
  const int groups = march_groups(yend + K - ylo);
  load(!late);
  if (KIND == MARCH_POST && !late) add_e();
  if (late) step(std::integral_constant<int, RR - 1>{}, t++);
  for (int g = 0; g < groups; ++g, t += RR) {
    step(std::integral_constant<int, 0>{}, t);
    step(std::integral_constant<int, 1>{}, t + 1);
    step(std::integral_constant<int, 2>{}, t + 2);
    step(std::integral_constant<int, 3>{}, t + 3);
    step(std::integral_constant<int, 4>{}, t + 4);
    step(std::integral_constant<int, 5>{}, t + 5);
  }
  if (!late) lds_barrier();
}

// Grids marched through: those of at least MARCH_MIN cell-samples (below, too few blocks of too few
// rows are left) whose rows stay under the 4 GiB of the kernel's offsets.  PRE and POST against a
// launch per pass (k_gs_free, k_restrict_free), us: 64x32 cells, 256 samples 24 + 32 and 20 + 32;
// 128x64x64 25 + 38 and 21 + 34; 64x32x333 27 + 41 and 29 + 48; 32x16x2048 28 + 31 and 34 + 59;
// 128x64x128 35 + 43 and 41 + 70; 256x128x512 333 + 498 and 562 + 961.  The FP32 cycle's stored rows
// are half as long: a solve took 130 ms marched and 107 not at 64x32x333; 200 samples of 128x64
// cells 97 and 105 (the middle of eight batches); 256x128x40 98 and 108, 256x128x200 288 and 332,
// 512x256x16 130 and 157.
constexpr size_t MARCH_MIN = 9 << 16, MARCH_MIN32 = 5 << 18;
inline bool march_takes(int nx, int ny, int S, int prec) {
  return (size_t)nx * ny * S >= (prec == 32 ? MARCH_MIN32 : MARCH_MIN) && (size_t)nx * S * 8 < ((size_t)1 << 32);
}

// Strips of a grid and segments of its rows for workgroups of NC columns: the split with the fewest
// steps of a compute unit's wavefronts (their time is that of the wavefronts together: one
// workgroup of 32 columns a unit takes 1.0 us a step, two 2.1).  Returns that number.
template <int KIND, int NC, typename Args>
inline long long march_split(int nx, int ny, int S, Args& A) {
  constexpr int K = march_passes<KIND>();
  A.nx = nx;
  A.ny = ny;
  A.S = S;
  A.nsb = (S + MARCH_NS - 1) / MARCH_NS;
  if (nx <= NC) {
    A.halo = 0;
    A.nstrip = 1;
    A.width = nx;
  } else {
    A.halo = K;
    const int most = (NC - 2 * K) / 2 * 2;
    A.nstrip = (nx + most - 1) / most;
    A.width = ((nx + A.nstrip - 1) / A.nstrip + 1) / 2 * 2;
  }
  long long best = -1;
  for (int seg = 1; seg <= 64; ++seg) {
    const int rows = ((ny + seg - 1) / seg + 1) / 2 * 2;
    const int n = (ny + rows - 1) / rows;
    if (n != seg) continue;
    const long long blocks = (long long)A.nsb * A.nstrip * n;
    const long long cost = (blocks + 255) / 256 * NC * march_groups(rows + K + (n > 1 ? 2 * K : 0));
    if (best >= 0 && cost >= best) continue;
    best = cost;
    A.rows = rows;
    A.nseg = n;
  }
  return best;
}

}  // namespace henry
