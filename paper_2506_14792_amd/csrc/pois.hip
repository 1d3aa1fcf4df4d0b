// Linear stability of plane Poiseuille flow on gfx950: the eigenvalue problem of the paper's
// neutral-curve example (Results, "Parametric sensitivity and numerical continuation";
// Supplementary, "Eigenvalue problems"), its adjoint eigenvectors, the eigenvalue
// sensitivities of equ:eigenvalue_sens and Newton's method on the growth rate, for many
// systems (one streamwise wavenumber alpha at one Reynolds number Re) at once.
//
// Flow between walls y = 0 and y = 2, base flow U = y (2 - y).  Two-dimensional perturbations
// (u, v, p) ~ exp(i alpha x + lambda t) satisfy, with nu = 1/Re, x = y - 1 in [-1, 1], D = d/dx,
// U = 1 - x^2, U' = -2x:
//   lambda u + i alpha U u + U' v + i alpha p - nu (D^2 - alpha^2) u = 0
//   lambda v + i alpha U v + D p - nu (D^2 - alpha^2) v = 0
//   i alpha u + D v = 0,      u = v = 0 at x = -1, 1,
// i.e. (lambda M + L) X = 0.  The discretization is the 2D problem's ultraspherical one (paper:
// Sparse spectral methods): Chebyshev-T unknowns, momentum rows in C2 coefficients, continuity
// in C1, first-order lifted taus, four boundary rows and the row tau_p = 0; a base-flow product
// row holds the first N C2 coefficients of the exact product series.  Slots (S = 3N + 5):
// u[0:N], v[N:2N], p[2N:3N], tau_u1, tau_v1, tau_u2, tau_v2, tau_p.
//
// L = L0 + alpha La + nu Ln + nu alpha^2 Lq, so the host assembles the five parts (with M) once;
// a system's matrix A = sigma M + L(alpha, nu) is formed on the device.  The advection term
// i alpha U is imaginary in the rows where the pressure gradient i alpha p is too, so no
// diagonal phases make A real (unlike the 2D convection problem): A is factored by a complex
// banded LU with partial pivoting.  Rows and columns are interleaved by mode and the u and v
// columns recombined (T_n - T_{n-2}, Dirichlet) so that the boundary rows are short and A is
// banded (kl = 11, ku = 19 at every N).
//
// Every Newton iteration runs: assembly and LU factorization (a block per system), the operators of
// eight rows that the solves use, the right eigenvector by inverse iteration y <- A^{-1} M y and at
// the same time the left eigenvector by w <- A^{-H} M^H w through the same factors, then the sensitivities
// d lambda/dRe = -<w, dL/dRe y> / <w, M y>, d lambda/dalpha likewise, and the Newton update of Re
// (or alpha) on the growth rate Re(lambda) with the next shift at the new eigenvalue.  A
// continuation step (the paper's tracing of the neutral curve) first moves along the curve's
// tangent, the gradient of the growth rate turned by a right angle, then corrects by Newton steps
// along the gradient (the smallest change of the parameters that zeroes the linearized growth
// rate), which also passes the curve's turning points.  All
// vectors stay in the permuted, recombined coordinates of A's band (the eigenvalues and the
// inner products are the same); the eigenvectors are converted to the state layout at the end.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "sps_device.h"
#include "sps_internal.h"
#include "ultra_ops.h"

namespace sps {
namespace {

constexpr int PT = 512;    // threads of a finish or operator block
constexpr int PTF = 256;   // threads of a factor block
// Block operators of the factors, eight rows each (window and width for kl = 11, ku <= 19):
//   L  in block t, with all of its row exchanges done first (permutation pi_t of the PTW-row window),
//      is [A_t | (0; I)] with A_t of PTW x 8;
//   U  back substitution of block t: x_block = G_t [y_block; the next entries], G_t of 8 x PGW.
// The forward solve applies the T_t for t ascending, then the G_t for t descending, the solve with
// the conjugate transpose G_t^H ascending, then T_t^H descending.
constexpr int PB = 8, PTW = 20, PGW = 40;
// A block's operators as the lanes of the right (r) and left (l) iterations read them, entry u of
// lane L at u * lanes + L:
constexpr int PTR = 4 * 2 * PTW;   // A_t: lane 2 row + half, entries 4 half + u
constexpr int PTL = 3 * 64;        // A_t: lane 8 column + q, rows q + 8 u (zero from PTW on)
constexpr int PGR = 5 * 64;        // G_t: lane 8 row + q, columns 5 q + u
constexpr int PGL = 8 * PGW;       // G_t: lane = column, rows u
constexpr int PWIN = 32, PWC = 64; // LDS window of the factorization: rows and columns mod these

__device__ __forceinline__ double cabs1(cplx a) { return fabs(a.x) + fabs(a.y); }
__device__ __forceinline__ cplx cmulc(cplx a, cplx b) {   // conj(a) b
  return cmk(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ cplx cfma(cplx a, cplx b, cplx c) {   // a b + c
  return cmk(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ cplx cfmac(cplx a, cplx b, cplx c) {   // conj(a) b + c
  return cmk(fma(a.x, b.x, fma(a.y, b.y, c.x)), fma(a.x, b.y, fma(-a.y, b.x, c.y)));
}
__device__ __forceinline__ cplx crecip(cplx a) {
  const double s = 1.0 / (a.x * a.x + a.y * a.y);
  return cmk(a.x * s, -a.y * s);
}
__device__ __forceinline__ cplx wave_csum(cplx a) {
  for (int o = 32; o >= 1; o >>= 1) {
    a.x += __shfl_xor(a.x, o);
    a.y += __shfl_xor(a.y, o);
  }
  return a;
}
// Compiler-only barrier between LDS accesses of one wave (a wave's LDS instructions execute in order).
__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A system between the launches of one call.
struct PoisState {
  double alpha, Re;
  cplx sig, lam;
  int stop, solves;
};

struct PoisDev {
  int N, S, kl, ku, bw, ldw;     // bw = kl + ku + 1 (the operators), ldw = 2 kl + ku + 1 (a factor row)
  int nb, mw;                    // blocks of eight rows; most entries of a row of M or of M^H
  const cplx* bM;                // [S][bw] row bands of the permuted, recombined M
  const cplx* bL0;               // parts of L: L0 + alpha La + nu Ln + nu alpha^2 Lq
  const cplx* bLa;
  const cplx* bLn;
  const cplx* bLq;
  const int* mcol[2];            // M and M^H by rows: column of entry e of row i at e S + i (padded rows
  const double* mval[2];         // repeat an entry with value 0); M is real
  const int* rowmap;             // band row i <- state row rowmap[i]
  const int* colinv;             // state column c -> band column colinv[c]
  const double* rho;             // recombination: x[c] = y'[c] + rho[c] y'[c + 2]
  cplx* W;                       // [sys][S][ldw]: U row j (U[j][j + r] at r <= kl + ku), then L's multipliers of step j
  cplx* dinv;                    // [sys][S] reciprocals of U's diagonal
  int* piv;                      // [sys][S] row interchanges (p - j)
  cplx *Tr, *Tl, *Gr, *Gl;       // [sys][nb][PTR] ...: the block operators
  unsigned char* perm;           // [sys][nb][PTW]
  cplx* vec;                     // [2][sys][S] right and left vectors
  PoisState* st;                 // [sys]
  int* active;                   // [solve] systems that go on after it
  int maxsys;
  int* err;
};

struct PoisArgs {
  const double* params;          // [sys][5] alpha, Re, sigma (re, im), continuation step ds
  int iters, mode, maxit;        // inverse iterations per solve; 0: eigenpair only, 1: Newton in Re, 2: in
                                 // alpha, 3: continuation step
  double tol;                    // Newton stops when |Re(lambda)| <= tol
  cplx* lam;                     // [sys]
  cplx* dlam;                    // [sys][2]: d lambda/dRe, d lambda/dalpha
  double* info;                  // [sys][3]: alpha, Re at the end, eigenvalue solves
  cplx* X;                       // [sys][S] right eigenvector, state layout, unit norm (nullable)
  cplx* Y;                       // [sys][S] left eigenvector (nullable)
};

// State of each system and its start vectors (the same for every system), unit norm.  One wave per system.
__global__ void __launch_bounds__(64) pois_start(PoisDev d, PoisArgs a) {
  const int sys = blockIdx.x, lane = threadIdx.x, n = d.S;
  double nn = 0.0;
  auto s0 = [](int i) { return cmk(1.0 / (1 + i % 7), 0.5 / (1 + i % 5)); };
  for (int i = lane; i < n; i += 64) {
    const cplx v = s0(i);
    nn += v.x * v.x + v.y * v.y;
  }
  for (int o = 32; o >= 1; o >>= 1) nn += __shfl_xor(nn, o);
  const double inv = 1.0 / sqrt(nn);
  for (int i = lane; i < n; i += 64)
    for (int side = 0; side < 2; ++side) d.vec[((size_t)side * d.maxsys + sys) * n + i] = cscale(s0(i), inv);
  if (lane == 0) {
    PoisState s;
    s.alpha = a.params[5 * sys];
    s.Re = a.params[5 * sys + 1];
    s.sig = cmk(a.params[5 * sys + 2], a.params[5 * sys + 3]);
    s.lam = czero();
    s.stop = 0;
    s.solves = 0;
    d.st[sys] = s;
  }
}

// Banded LU with partial pivoting of A = sigma M + L0 + alpha La + nu Ln + nu alpha^2 Lq.  One block per
// system.  The rows and columns a step touches (kl + 1 by kl + ku + 1) are in an LDS window of two
// copies: a step reads one and writes the other, two entries per thread, so that a column takes one block
// barrier and its instructions are those of one wave per SIMD (one entry in 512 threads: 0.32 ms against
// 0.25); entry (i, c) is at [i mod 32][(c + i) mod 64], which spreads a column's rows over the banks.  Every wave finds the pivot by itself, the reciprocals of all candidates being formed meanwhile.  The
// next eight rows' parts of A are loaded while eight columns are eliminated.  Bound by the chain of a
// column (pivot search, two LDS round trips, the update, the barrier): 0.64 us, 0.25 ms for 128 systems of
// 389 rows.  With one block per system doing every stage, its band in global memory and four barriers a
// column, the whole call of 20 iterations took 13.7 ms; it takes 0.9.
__global__ void __launch_bounds__(PTF) pois_factor(PoisDev d) {
  __shared__ cplx win[2][PWIN * PWC];
  const int sys = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = d.S, kl = d.kl, kv = d.kl + d.ku, ldw = d.ldw, bw = d.bw;
  const PoisState st = d.st[sys];
  if (st.stop) return;
  const double alpha = st.alpha, nu = 1.0 / st.Re, q2 = nu * alpha * alpha;
  cplx* W = d.W + (size_t)sys * n * ldw;
  cplx* dinv = d.dinv + (size_t)sys * n;
  int* piv = d.piv + (size_t)sys * n;
  auto at = [](int i, int c) { return (i % PWIN) * PWC + ((c + i) % PWC); };
  struct Parts { cplx m, l0, la, ln, lq; };
  auto load = [&](int i, int q) {   // clamped, so that the loads are unconditional
    const size_t e = (size_t)min(i, n - 1) * bw + min(q, bw - 1);
    return Parts{d.bM[e], d.bL0[e], d.bLa[e], d.bLn[e], d.bLq[e]};
  };
  auto form = [&](const Parts& v, int i, int q) {
    const int j = i + q - kl;
    cplx z = cadd(cmul(st.sig, v.m), v.l0);
    z = cadd(z, cscale(v.la, alpha));
    z = cadd(z, cscale(v.ln, nu));
    z = cadd(z, cscale(v.lq, q2));
    return (i < n && j >= 0 && j < n) ? z : czero();
  };
  for (int e = tid; e < 2 * PWIN * PWC; e += PTF) win[0][e] = czero();
  __syncthreads();
  const int r = tid >> 5, cl = tid & 31;   // this thread's rows r, r + 8 and column of the step; as a feeder, row and entry
  for (int i = r; i < kl + PB; i += PTF / 32) {   // the rows of the first eight columns
    const Parts v = load(i, cl);
    if (cl < bw) win[0][at(i, i + cl - kl + PWC)] = win[1][at(i, i + cl - kl + PWC)] = form(v, i, cl);
  }
  __syncthreads();
  for (int j0 = 0; j0 < n; j0 += PB) {
    const int in = j0 + kl + PB + r;       // the row that this thread brings in for the next eight columns
    const Parts nxt = load(in, cl);
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      const int j = j0 + u;
      if (j >= n) break;
      const cplx* wr = win[u & 1];
      cplx* ww = win[(u & 1) ^ 1];
      const int km = min(kl, n - 1 - j), rl = lane & 15;
      const cplx cv = wr[at(j + rl, j)];
      const cplx rv = crecip(cv);
      const double mag = (rl <= km) ? cabs1(cv) : -1.0;
      double best = mag;
      best = fmax(best, dpp_xor1(best));
      best = fmax(best, dpp_xor2(best));
      best = fmax(best, dpp_mirror8(best));
      best = fmax(best, dpp_d<0x140>(best));
      const unsigned hit = (unsigned)__ballot(mag == best) & 0xffffu;   // the first of the largest
      const int p = hit ? __builtin_ctz(hit) : 0;
      const cplx pv = cmk(readlane_d(cv.x, p), readlane_d(cv.y, p));
      const cplx pinv = (pv.x != 0.0 || pv.y != 0.0) ? cmk(readlane_d(rv.x, p), readlane_d(rv.y, p)) : czero();
      const cplx up = wr[at(j + p, j + cl)];
#pragma unroll
      for (int h = 0; h < 2; ++h) {   // this thread's entries: rows j + rr (after the interchange), column j + cl
        const int rr = r + PB * h, src = (rr == p) ? j : j + rr;
        const cplx a0 = wr[at(src, j + cl)], aj = wr[at(src, j)];
        const cplx nv = csub(a0, cmul(cmul(aj, pinv), up));
        if (rr >= 1 && rr <= kl) {
          if (cl >= 1 && cl <= kv) ww[at(j + rr, j + cl)] = (rr <= km) ? nv : czero();
          if (cl == 0) ww[at(j + rr, j + kv + 1)] = czero();   // the column that enters
        }
      }
      if (wv == 2) {          // U's row j
        if (lane <= kv) W[(size_t)j * ldw + lane] = (j + lane < n) ? up : czero();
      } else if (wv == 3) {   // L's multipliers, the pivot
        const cplx c0 = cmk(readlane_d(cv.x, 0), readlane_d(cv.y, 0));
        const cplx l = cmul(rl == p ? c0 : cv, pinv);
        if (lane >= 1 && lane <= kl) W[(size_t)j * ldw + kv + lane] = (lane <= km) ? l : czero();
        if (lane == 0) {
          dinv[j] = pinv;
          piv[j] = p;
          if (!(best > 0.0)) atomicOr(d.err, 1);
        }
      }
      if (u == PB - 1 && cl < bw) {
        const cplx v = form(nxt, in, cl);
        win[0][at(in, in + cl - kl)] = v;
        win[1][at(in, in + cl - kl)] = v;
      }
      __syncthreads();
    }
  }
}

// The block operators of every system's factors, one column per thread.  blockIdx.y: T or G.
__global__ void __launch_bounds__(PT) pois_operators(PoisDev d) {
  const int sys = blockIdx.x, tid = threadIdx.x + blockIdx.z * PT;
  const int n = d.S, kl = d.kl, kv = d.kl + d.ku, ldw = d.ldw;
  if (d.st[sys].stop) return;
  const cplx* W = d.W + (size_t)sys * n * ldw;
  const cplx* dinv = d.dinv + (size_t)sys * n;
  const int* piv = d.piv + (size_t)sys * n;
  // T_t: the image of the window's unit vector c under the block's exchanges and eliminations is column
  // pos of A_t, pos the row that the exchanges bring entry c to (or e_pos for pos >= 8)
  const int nb = d.nb;
  const size_t ob = (size_t)sys * nb;
  for (int e = tid; blockIdx.y == 0 && e < nb * PTW; e += gridDim.z * PT) {
    const int t = e / PTW, c = e - t * PTW, tb = t * PB;
    cplx v[PTW];
#pragma unroll
    for (int i = 0; i < PTW; ++i) v[i] = cmk(i == c ? 1.0 : 0.0, 0.0);
    int pos = c;
    for (int q = 0; q < PB; ++q) {
      const int j = tb + q;
      if (j >= n) break;
      const int p = piv[j], km = min(kl, n - 1 - j);
      if (pos == q) pos = q + p;
      else if (pos == q + p) pos = q;
      cplx vq = czero(), vp = czero();
#pragma unroll
      for (int i = 0; i < PTW; ++i) {
        if (i == q) vq = v[i];
        if (i == q + p) vp = v[i];
      }
#pragma unroll
      for (int i = 0; i < PTW; ++i) {
        if (i == q) v[i] = vp;
        else if (i == q + p) v[i] = vq;
        if (i > q && i - q <= km) v[i] = csub(v[i], cmul(W[(size_t)j * ldw + kv + i - q], vp));
      }
    }
    d.perm[(ob + t) * PTW + pos] = (unsigned char)c;
    if (pos < PB) {
      cplx* Tr = d.Tr + (ob + t) * PTR;
      cplx* Tl = d.Tl + (ob + t) * PTL;
#pragma unroll
      for (int i = 0; i < PTW; ++i) {
        Tr[(pos & 3) * (2 * PTW) + 2 * i + (pos >> 2)] = v[i];
        Tl[(i >> 3) * 64 + pos * 8 + (i & 7)] = v[i];
      }
#pragma unroll
      for (int i = PTW; i < 24; ++i) Tl[(i >> 3) * 64 + pos * 8 + (i & 7)] = czero();
    }
  }
  // G_t by columns: U_tt x = e_c (c < 8), or -U's column tb + c
  for (int e = tid; blockIdx.y == 1 && e < nb * PGW; e += gridDim.z * PT) {
    const int t = e / PGW, c = e - t * PGW, tb = t * PB;
    cplx x[PB];
#pragma unroll
    for (int i = PB - 1; i >= 0; --i) {
      const cplx* Ur = W + (size_t)min(tb + i, n - 1) * ldw;
      cplx s = czero();
      if (c < PB) s.x = (i == c) ? 1.0 : 0.0;
      else if (tb + c < n && c - i <= kv) s = cscale(Ur[c - i], -1.0);
#pragma unroll
      for (int k = i + 1; k < PB; ++k) s = csub(s, cmul(Ur[k - i], x[k]));
      x[i] = (tb + i < n) ? cmul(s, dinv[min(tb + i, n - 1)]) : czero();
    }
    cplx* Gr = d.Gr + (ob + t) * PGR;
    cplx* Gl = d.Gl + (ob + t) * PGL;
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      Gr[(c % 5) * 64 + i * 8 + c / 5] = x[i];
      Gl[i * PGW + c] = x[i];
    }
  }
}

// All inverse iterations of one system's right (blockIdx.y = 0: y <- A^{-1} M y) or left (w <- A^{-H} M^H w)
// vector, in one wave: no barriers; the vector is in LDS, and every block operator goes straight from
// memory to the registers of the lanes that use it, PD blocks ahead (the most that 512 registers hold
// without moving them about: 4 blocks ahead took 0.59 ms, 8 on both sides 0.56, these 0.50 for 20 iterations
// of 128 systems of 389 rows).  A block step is one LDS round trip, a short sum per lane and a DPP sum:
// bound by that chain, 0.25 us a block; either side alone takes the same time, on a CU of its own.
// LDS: x, t (S + PGW each), M's values and columns, the permutations.
template <int side>
__device__ __forceinline__ void iterate_side(const PoisDev& d, int iters, double* sm) {
  const int sys = blockIdx.x, lane = threadIdx.x, n = d.S, nb = d.nb, mw = d.mw;
  const PoisState* st = d.st + sys;
  if (st->stop) return;
  cplx* x = reinterpret_cast<cplx*>(sm);
  cplx* t = x + n;
  double* mv = reinterpret_cast<double*>(t + n + PGW);
  int* mc = reinterpret_cast<int*>(mv + mw * n);
  unsigned char* pm = reinterpret_cast<unsigned char*>(mc + mw * n);
  cplx* gx = d.vec + ((size_t)side * d.maxsys + sys) * n;
  for (int i = lane; i < n; i += 64) x[i] = gx[i];
  for (int i = lane; i < PGW; i += 64) t[n + i] = czero();
  for (int i = lane; i < mw * n; i += 64) {
    mv[i] = d.mval[side][i];
    mc[i] = d.mcol[side][i];
  }
  const size_t ob = (size_t)sys * nb;
  for (int i = lane; i < nb * PTW; i += 64) pm[i] = d.perm[ob * PTW + i];
  wsync();
  const cplx* T = side ? d.Tl + ob * PTL : d.Tr + ob * PTR;
  const cplx* G = side ? d.Gl + ob * PGL : d.Gr + ob * PGR;
  constexpr int PD = side ? 6 : 8;
  cplx ring[PD][8];   // the operators of the next PD steps of the sequence T sweep, G sweep (left: G, T), ...
  const int lt = side ? lane : min(lane, 2 * PTW - 1), lg = side ? min(lane, PGW - 1) : lane;
  // entries of block b for this lane (indices clamped, so that every load is issued)
  auto load_t = [&](int b, cplx (&v)[8]) __attribute__((always_inline)) {
    const cplx* p = T + (size_t)min(max(b, 0), nb - 1) * (side ? PTL : PTR) + lt;
    const int s = side ? 64 : 2 * PTW;
    v[0] = p[0];
    v[1] = p[s];
    v[2] = p[2 * s];
    if (!side) v[3] = p[3 * s];
  };
  auto load_g = [&](int b, cplx (&v)[8]) __attribute__((always_inline)) {
    const cplx* p = G + (size_t)min(max(b, 0), nb - 1) * (side ? PGL : PGR) + lg;
    const int s = side ? PGW : 64;
#pragma unroll
    for (int u = 0; u < 5; ++u) v[u] = p[u * s];
    if (side) {
#pragma unroll
      for (int u = 5; u < 8; ++u) v[u] = p[u * s];
    }
  };
  auto first_t = [&](int u) __attribute__((always_inline)) { return side ? nb - 1 - u : u; };   // T ascends on the right, descends on the left
  auto first_g = [&](int u) __attribute__((always_inline)) { return side ? u : nb - 1 - u; };
  auto load_first = [&](int i, cplx (&v)[8]) __attribute__((always_inline)) { side ? load_g(first_g(i), v) : load_t(first_t(i), v); };
  auto load_second = [&](int i, cplx (&v)[8]) __attribute__((always_inline)) { side ? load_t(first_t(i), v) : load_g(first_g(i), v); };
#pragma unroll
  for (int u = 0; u < PD; ++u) load_first(u, ring[u]);
  // right: rows 2 row + half of A_t; left: column lane / 8, rows lane % 8 + 8 u
  const int rr = lane >> 1, hh = lane & 1, c8 = lane >> 3, q8 = lane & 7;
  const int rc = min(rr, PTW - 1);
  unsigned p4 = 0;   // right: the next block's permutation, entries 4 hh .. 4 hh + 3 and (one byte) rc
  int pk = 0;
  auto next_perm = [&](int b) __attribute__((always_inline)) {
    const unsigned char* pb = pm + min(b, nb - 1) * PTW;
    p4 = *reinterpret_cast<const unsigned*>(pb + 4 * hh);
    pk = pb[rc];
  };
  auto step_t = [&](int b, const cplx (&v)[8]) __attribute__((always_inline)) {
    cplx* w = t + b * PB;
    const unsigned char* pb = pm + b * PTW;
    if (!side) {
      cplx s = (hh == 0 && rc >= PB) ? w[pk] : czero();
      cplx s2 = czero();
      s = cfma(v[0], w[p4 & 255], s);
      s2 = cfma(v[1], w[(p4 >> 8) & 255], s2);
      s = cfma(v[2], w[(p4 >> 16) & 255], s);
      s2 = cfma(v[3], w[p4 >> 24], s2);
      next_perm(b + 1);
      s = cadd(s, s2);
      s = cadd(s, cmk(dpp_xor1(s.x), dpp_xor1(s.y)));
      wsync();
      if (hh == 0 && rr < PTW && b * PB + rr < n) w[rr] = s;
    } else {
      // lane q = 0 stores the sum at pi(c), lanes q = 1, 2 the entries that only move
      const int row = (q8 == 1) ? PB + c8 : 2 * PB + (c8 & 3);
      const cplx keep = w[row];
      cplx s = cfmac(v[0], w[q8], czero());
      s = cfmac(v[1], w[q8 + 8], s);
      s = cfmac(v[2], w[q8 + 16], s);
      s = group_sum<8>(s);
      const int dst = b * PB + pb[(q8 == 0) ? c8 : row];
      s.x = (q8 == 0) ? s.x : keep.x;
      s.y = (q8 == 0) ? s.y : keep.y;
      wsync();
      if ((q8 < 2 || (q8 == 2 && c8 < 4)) && dst < n) t[dst] = s;
    }
    wsync();
  };
  auto step_g = [&](int b, const cplx (&v)[8]) __attribute__((always_inline)) {
    cplx* w = t + b * PB;
    if (!side) {   // row c8, columns 5 q8 + u
      cplx s = czero(), s2 = czero();
      s = cfma(v[0], w[5 * q8], s);
      s2 = cfma(v[1], w[5 * q8 + 1], s2);
      s = cfma(v[2], w[5 * q8 + 2], s);
      s2 = cfma(v[3], w[5 * q8 + 3], s2);
      s = cfma(v[4], w[5 * q8 + 4], s);
      s = group_sum<8>(cadd(s, s2));
      wsync();
      if (q8 == 0 && b * PB + c8 < n) w[c8] = s;
    } else {       // column lane
      cplx s = (lane >= PB && lane < PGW) ? w[lg] : czero(), s2 = czero();
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        s = cfmac(v[u], w[u], s);
        s2 = cfmac(v[u + 1], w[u + 1], s2);
      }
      s = cadd(s, s2);
      wsync();
      if (lane < PGW && b * PB + lane < n) w[lane] = s;
    }
    wsync();
  };
  // one sweep; the last steps load the first blocks of the sweep that follows
  auto sweep = [&](auto step, auto load, auto load_next) __attribute__((always_inline)) {
    int b0 = 0;
    for (; b0 + PD < nb; b0 += PD)
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        step(b0 + u, ring[u]);
        load(b0 + u + PD, ring[u]);
      }
#pragma unroll
    for (int u = 0; u < PD; ++u) {
      if (b0 + u < nb) step(b0 + u, ring[u]);
      load_next(u, ring[u]);
    }
  };
  auto do_t = [&](int i, const cplx (&v)[8]) __attribute__((always_inline)) { step_t(first_t(i), v); };
  auto do_g = [&](int i, const cplx (&v)[8]) __attribute__((always_inline)) { step_g(first_g(i), v); };
  cplx mu = czero();
  for (int k = 0; k < iters; ++k) {
    for (int i = lane; i < n; i += 64) {
      cplx s = czero();
      for (int e = 0; e < mw; ++e) {
        const cplx xv = x[mc[e * n + i]];
        const double m = mv[e * n + i];
        s = cmk(fma(m, xv.x, s.x), fma(m, xv.y, s.y));
      }
      t[i] = s;
    }
    wsync();
    if (!side) {
      next_perm(0);
      sweep(do_t, load_first, load_second);
      sweep(do_g, load_second, load_first);
    } else {
      sweep(do_g, load_first, load_second);
      sweep(do_t, load_second, load_first);
    }
    // x <- t / |t|, mu = <x, t>
    mu = czero();
    double nn = 0.0;
    for (int i = lane; i < n; i += 64) {
      const cplx b = t[i];
      mu = cfmac(x[i], b, mu);
      nn += b.x * b.x + b.y * b.y;
    }
    mu = wave_csum(mu);
    for (int o = 32; o >= 1; o >>= 1) nn += __shfl_xor(nn, o);
    const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
    for (int i = lane; i < n; i += 64) x[i] = cscale(t[i], inv);
    wsync();
  }
  for (int i = lane; i < n; i += 64) gx[i] = x[i];
  if (side == 0 && lane == 0) {
    const double m2 = mu.x * mu.x + mu.y * mu.y;
    d.st[sys].lam = cmk(st->sig.x - mu.x / m2, st->sig.y + mu.y / m2);   // sigma - 1/mu
  }
}
__global__ void __launch_bounds__(64) pois_iterate(PoisDev d, int iters) {
  extern __shared__ double sm[];
  if (blockIdx.y == 0) iterate_side<0>(d, iters, sm);
  else iterate_side<1>(d, iters, sm);
}

template <int NV>
__device__ void block_csums(cplx* v, double* red) {
  const int tid = threadIdx.x, w = tid >> 6;
  for (int q = 0; q < NV; ++q) v[q] = wave_csum(v[q]);
  __syncthreads();
  if ((tid & 63) == 0)
    for (int q = 0; q < NV; ++q) {
      red[(w * NV + q) * 2] = v[q].x;
      red[(w * NV + q) * 2 + 1] = v[q].y;
    }
  __syncthreads();
  for (int q = 0; q < NV; ++q) {
    cplx s = czero();
    for (int ww = 0; ww < PT / 64; ++ww) s = cadd(s, cmk(red[(ww * NV + q) * 2], red[(ww * NV + q) * 2 + 1]));
    v[q] = s;
  }
  __syncthreads();
}

// After eigenvalue solve `it`: the sensitivities, the Newton or continuation update of a system that
// goes on, the outputs of one that is done.  One block per system.  LDS: y, w, t (S complex each).
__global__ void __launch_bounds__(PT) pois_finish(PoisDev d, PoisArgs a, int it) {
  extern __shared__ double sm[];
  __shared__ double red[2 * 3 * PT / 64];
  __shared__ int s_stop;
  cplx* y = reinterpret_cast<cplx*>(sm);
  cplx* w = y + d.S;
  cplx* t0 = w + d.S;
  const int sys = blockIdx.x, tid = threadIdx.x, n = d.S, kl = d.kl, bw = d.bw;
  const PoisState st = d.st[sys];
  if (st.stop) return;
  for (int i = tid; i < n; i += PT) {
    y[i] = d.vec[(size_t)sys * n + i];
    w[i] = d.vec[((size_t)d.maxsys + sys) * n + i];
  }
  __syncthreads();
  const double alpha = st.alpha, Re = st.Re, nu = 1.0 / Re;
  const int solves = st.solves + 1;
  // ---- sensitivities: <w, M y>, <w, dL/dRe y>, <w, dL/dalpha y>
  cplx acc[3] = {czero(), czero(), czero()};
  for (int e = tid; e < n * bw; e += PT) {   // entry by entry: neighbouring lanes read neighbouring entries
    const int i = e / bw, j = i + e - i * bw - kl;
    if (j < 0 || j >= n) continue;
    const cplx wy = cmulc(w[i], y[j]), lq = d.bLq[e];
    // dL/dRe = -nu^2 (Ln + alpha^2 Lq), dL/dalpha = La + 2 nu alpha Lq
    acc[0] = cadd(acc[0], cmul(d.bM[e], wy));
    acc[1] = cadd(acc[1], cmul(cadd(d.bLn[e], cscale(lq, alpha * alpha)), wy));
    acc[2] = cadd(acc[2], cmul(cadd(d.bLa[e], cscale(lq, 2.0 * nu * alpha)), wy));
  }
  block_csums<3>(acc, red);
  const cplx den = acc[0];
  const double dd = den.x * den.x + den.y * den.y;
  auto qdiv = [&](cplx num) { return cscale(cmulc(den, num), -1.0 / dd); };   // -num / den
  const cplx dl0 = cscale(qdiv(acc[1]), -nu * nu), dl1 = qdiv(acc[2]);
  if (tid == 0) {
    const cplx lam = st.lam;
    const double g = lam.x;
    // gradient of the growth rate in (alpha, ln Re)
    const double ga = dl1.x, gr = Re * dl0.x, g2 = ga * ga + gr * gr;
    PoisState ns = st;
    ns.solves = solves;
    int stop = 0;
    if (a.mode == 3 && it == 0) {
      // predictor: a step ds along the tangent of the level curve, the gradient turned by a
      // right angle (the unstable side stays on the same hand)
      const double gn = sqrt(g2), ds = a.params[5 * sys + 4];
      ns.alpha = alpha - ds * gr / gn;
      ns.Re = Re * exp(ds * ga / gn);
      ns.sig = lam;
      if (it + 1 >= max(1, a.maxit)) stop = 1;   // no solve left to correct it
    } else if (a.mode == 0 || fabs(g) <= a.tol || it + 1 >= max(1, a.maxit)) {
      stop = 1;
      if (a.mode != 0 && fabs(g) > a.tol) atomicOr(d.err, 4);
    } else if (a.mode == 3) {
      // corrector: the minimum-norm Newton step in (alpha, ln Re)
      ns.alpha = alpha - g * ga / g2;
      ns.Re = Re * exp(-g * gr / g2);
      ns.sig = lam;
    } else if (a.mode == 1) {
      ns.Re = Re - g / dl0.x;
      ns.sig = lam;
    } else {
      ns.alpha = alpha - g / dl1.x;
      ns.sig = lam;
    }
    ns.stop = stop;
    d.st[sys] = ns;
    if (!stop) atomicAdd(d.active + it, 1);
    s_stop = stop;
    if (stop) {
      a.lam[sys] = lam;
      a.dlam[2 * sys] = dl0;
      a.dlam[2 * sys + 1] = dl1;
      a.info[3 * sys] = ns.alpha;
      a.info[3 * sys + 1] = ns.Re;
      a.info[3 * sys + 2] = solves;
    }
  }
  __syncthreads();
  if (!s_stop) return;
  if (a.X) {
    // X = R P_c y in the state layout, then unit norm
    cplx* X = a.X + (size_t)sys * n;
    double nn = 0.0;
    for (int c = tid; c < n; c += PT) {
      cplx v = y[d.colinv[c]];
      if (d.rho[c] != 0.0) v = cadd(v, cscale(y[d.colinv[c + 2]], d.rho[c]));
      t0[c] = v;
      nn += v.x * v.x + v.y * v.y;
    }
    cplx s[1] = {cmk(nn, 0.0)};
    block_csums<1>(s, red);
    const double inv = 1.0 / sqrt(s[0].x);
    for (int c = tid; c < n; c += PT) X[c] = cscale(t0[c], inv);
  }
  if (a.Y) {
    cplx* Y = a.Y + (size_t)sys * n;
    double nn = 0.0;
    for (int i = tid; i < n; i += PT) nn += w[i].x * w[i].x + w[i].y * w[i].y;
    cplx s[1] = {cmk(nn, 0.0)};
    block_csums<1>(s, red);
    const double inv = 1.0 / sqrt(s[0].x);
    for (int i = tid; i < n; i += PT) Y[d.rowmap[i]] = cscale(w[i], inv);
  }
}

// ---------------------------------------------------------------------------- host assembly
// Dense parts (state slot order) of the operator, written from the formulation above.
struct PoisParts {
  Cmat M, L0, La, Ln, Lq;
  explicit PoisParts(int S) : M(S), L0(S), La(S), Ln(S), Lq(S) {}
};

// rectangular (r x c) row-major products and the exact product operators
static std::vector<double> rmat(const std::vector<double>& A, int ar, int ac, const std::vector<double>& B, int bc) {
  std::vector<double> C((size_t)ar * bc, 0.0);
  for (int i = 0; i < ar; ++i)
    for (int k = 0; k < ac; ++k) {
      const double v = A[(size_t)i * ac + k];
      if (v == 0.0) continue;
      for (int j = 0; j < bc; ++j) C[(size_t)i * bc + j] += v * B[(size_t)k * bc + j];
    }
  return C;
}
// multiplication by x of a T series of m terms: (m + 1) x m
static std::vector<double> mult_x(int m) {
  std::vector<double> A((size_t)(m + 1) * m, 0.0);
  A[(size_t)1 * m + 0] = 1.0;
  for (int k = 1; k < m; ++k) {
    A[(size_t)(k + 1) * m + k] += 0.5;
    A[(size_t)(k - 1) * m + k] += 0.5;
  }
  return A;
}
// first N C2 coefficients (N x N) of the product of a T series of N terms with a polynomial of
// degree deg, given its exact product operator P ((N + deg) x N)
static std::vector<double> c2_rows(const std::vector<double>& P, int N, int deg) {
  const int m = N + deg;
  const std::vector<double> S10 = matmul(op_S1(m), op_S0(m), m);
  const std::vector<double> full = rmat(S10, m, m, P, N);
  return std::vector<double>(full.begin(), full.begin() + (size_t)N * N);
}

static void pois_assemble(int N, PoisParts& P) {
  const int U = 0, V = N, Pp = 2 * N, T = 3 * N;
  const std::vector<double> S0 = op_S0(N), S1 = op_S1(N);
  const std::vector<double> S10 = matmul(S1, S0, N);
  const std::vector<double> D0 = op_D(N, 1.0, true), D1 = op_D(N, 2.0, false);
  const std::vector<double> DZZ = matmul(D1, D0, N), SD = matmul(S1, D0, N);
  const std::vector<double> X1 = mult_x(N);                                   // (N+1) x N
  const std::vector<double> X2 = rmat(mult_x(N + 1), N + 2, N + 1, X1, N);    // (N+2) x N: x^2
  std::vector<double> Uop(X2.size());
  for (int i = 0; i < N + 2; ++i)
    for (int j = 0; j < N; ++j) Uop[(size_t)i * N + j] = (i == j ? 1.0 : 0.0) - X2[(size_t)i * N + j];
  std::vector<double> dU(X1.size());
  for (size_t e = 0; e < X1.size(); ++e) dU[e] = -2.0 * X1[e];
  const std::vector<double> SU = c2_rows(Uop, N, 2), SdU = c2_rows(dU, N, 1);
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j) {
      const size_t e = (size_t)i * N + j;
      for (int f = 0; f < 2; ++f) {
        const int r = f * N + i, c = f * N + j;
        if (S10[e] != 0.0) {
          P.M.add(r, c, S10[e]);
          P.Lq.add(r, c, S10[e]);        // + nu alpha^2 S10
        }
        if (DZZ[e] != 0.0) P.Ln.add(r, c, -DZZ[e]);
        if (SU[e] != 0.0) P.La.add(r, c, 0.0, SU[e]);   // i alpha U
      }
      if (SdU[e] != 0.0) P.L0.add(U + i, V + j, SdU[e]);           // U' v
      if (S10[e] != 0.0) P.La.add(U + i, Pp + j, 0.0, S10[e]);     // i alpha p
      if (SD[e] != 0.0) P.L0.add(V + i, Pp + j, SD[e]);            // dp/dx
      if (S0[e] != 0.0) P.La.add(Pp + i, U + j, 0.0, S0[e]);       // continuity i alpha u
      if (D0[e] != 0.0) P.L0.add(Pp + i, V + j, D0[e]);            // continuity dv/dx
    }
  // lifted taus: -nu 2 C2_{N-2} tau_1 and C2_{N-1} tau_2 in the momentum rows, C1_{N-1} tau_v1 in
  // continuity (d/dx U_{N-1} = 2 C2_{N-2})
  P.Ln.add(U + N - 2, T + 0, -2.0);
  P.Ln.add(V + N - 2, T + 1, -2.0);
  P.L0.add(U + N - 1, T + 2, 1.0);
  P.L0.add(V + N - 1, T + 3, 1.0);
  P.L0.add(Pp + N - 1, T + 1, 1.0);
  // boundary rows u(-1), u(1), v(-1), v(1) and tau_p = 0
  for (int m = 0; m < N; ++m) {
    P.L0.add(T + 0, U + m, (m & 1) ? -1.0 : 1.0);
    P.L0.add(T + 1, U + m, 1.0);
    P.L0.add(T + 2, V + m, (m & 1) ? -1.0 : 1.0);
    P.L0.add(T + 3, V + m, 1.0);
  }
  P.L0.add(T + 4, T + 4, 1.0);
}

struct PoisBands {
  int S = 0, kl = 0, ku = 0;
  std::vector<std::vector<double2>> parts;   // M, L0, La, Ln, Lq: [S][kl+ku+1]
  std::vector<int> rowmap, colmap;
  std::vector<double> rho;
};

static void pois_bands(int N, PoisBands& hb) {
  const int S = 3 * N + 5;
  PoisParts P(S);
  pois_assemble(N, P);
  std::vector<double> rho(S, 0.0);
  for (int f = 0; f < 2; ++f)
    for (int m = 0; m + 2 < N; ++m) rho[f * N + m] = -1.0;
  std::vector<int> rowmap, colmap;
  rowmap.push_back(3 * N + 4);
  for (int q = 0; q < 4; ++q) rowmap.push_back(3 * N + q);
  for (int m = 0; m < N; ++m) {
    rowmap.push_back(2 * N + m);
    rowmap.push_back(m);
    rowmap.push_back(N + m);
  }
  colmap.push_back(3 * N + 4);
  for (int m = 0; m < N; ++m)
    for (int f = 0; f < 3; ++f) colmap.push_back(f * N + m);
  for (int q = 0; q < 4; ++q) colmap.push_back(3 * N + q);
  Cmat* mats[5] = {&P.M, &P.L0, &P.La, &P.Ln, &P.Lq};
  std::vector<std::vector<double2>> dense(5);
  int kl = 0, ku = 0;
  for (int t = 0; t < 5; ++t) {
    Cmat& A = *mats[t];
    dense[t].assign((size_t)S * S, make_double2(0.0, 0.0));
    for (int i = 0; i < S; ++i) {
      const int r = rowmap[i];
      double rowmax = 0.0;
      std::vector<double2> row(S);
      for (int j = 0; j < S; ++j) {
        const int c = colmap[j];
        double2 v = A.at(r, c);
        if (c >= 2 && rho[c - 2] != 0.0) {
          v.x += A.at(r, c - 2).x * rho[c - 2];
          v.y += A.at(r, c - 2).y * rho[c - 2];
        }
        row[j] = v;
        rowmax = std::max(rowmax, std::hypot(v.x, v.y));
      }
      for (int j = 0; j < S; ++j) {
        const double2 v = row[j];
        if (std::hypot(v.x, v.y) <= 1e-14 * rowmax) continue;   // exact cancellations of the recombination
        dense[t][(size_t)i * S + j] = v;
        kl = std::max(kl, i - j);
        ku = std::max(ku, j - i);
      }
    }
  }
  const int bw = kl + ku + 1;
  hb.S = S;
  hb.kl = kl;
  hb.ku = ku;
  hb.parts.assign(5, std::vector<double2>((size_t)S * bw, make_double2(0.0, 0.0)));
  for (int t = 0; t < 5; ++t)
    for (int i = 0; i < S; ++i)
      for (int j = std::max(0, i - kl); j <= std::min(S - 1, i + ku); ++j)
        hb.parts[t][(size_t)i * bw + (j - i + kl)] = dense[t][(size_t)i * S + j];
  hb.rowmap = rowmap;
  hb.colmap = colmap;
  hb.rho = rho;
}

class PoisProblem : public ProblemImpl {
 public:
  PoisProblem(int N, int max_systems, hipStream_t s) {
    stream = s;
    SPS_REQUIRE(N >= 8 && N <= 256, "nz must be in [8, 256]");
    SPS_REQUIRE(max_systems >= 1 && max_systems <= 4096, "max_systems must be in [1, 4096]");
    PoisBands hb;
    pois_bands(N, hb);
    maxsys_ = max_systems;
    dv_.N = N;
    dv_.S = hb.S;
    dv_.kl = hb.kl;
    dv_.ku = hb.ku;
    dv_.bw = hb.kl + hb.ku + 1;
    dv_.ldw = 2 * hb.kl + hb.ku + 1;
    SPS_REQUIRE(hb.kl + 1 <= 32 && hb.kl + hb.ku < 64, "band too wide for the one-wave solves");
    const cplx** dst[5] = {&dv_.bM, &dv_.bL0, &dv_.bLa, &dv_.bLn, &dv_.bLq};
    for (int t = 0; t < 5; ++t) *dst[t] = arena_.upload(hb.parts[t], stream);
    std::vector<int> colinv(hb.S);
    for (int j = 0; j < hb.S; ++j) colinv[hb.colmap[j]] = j;
    dv_.rowmap = arena_.upload(hb.rowmap, stream);
    dv_.colinv = arena_.upload(colinv, stream);
    dv_.rho = arena_.upload(hb.rho, stream);
    dv_.nb = (hb.S + PB - 1) / PB;
    SPS_REQUIRE(hb.kl + PB <= PTW && PB + hb.kl + hb.ku <= PGW && hb.kl < PWIN - 1 && dv_.bw < 32,
                "band too wide for the block operators");
    upload_m(hb);
    const size_t sn = (size_t)maxsys_ * hb.S, sb = (size_t)maxsys_ * dv_.nb;
    dv_.W = arena_.alloc<cplx>(sn * dv_.ldw);
    dv_.dinv = arena_.alloc<cplx>(sn);
    dv_.piv = arena_.alloc<int>(sn);
    // the block operators: 992 complex values per eight rows and system, three times the band factors (W); 0.78 MB a
    // system at nz = 128, 1.5 MB at 256, so 6.3 GB for the largest handle, 4096 systems at 256
    dv_.Tr = arena_.alloc<cplx>(sb * PTR);
    dv_.Tl = arena_.alloc<cplx>(sb * PTL);
    dv_.Gr = arena_.alloc<cplx>(sb * PGR);
    dv_.Gl = arena_.alloc<cplx>(sb * PGL);
    dv_.perm = arena_.alloc<unsigned char>(sb * PTW);
    dv_.vec = arena_.alloc<cplx>(2 * sn);
    dv_.st = arena_.alloc<PoisState>(maxsys_);
    dv_.active = arena_.alloc<int>(kMaxSolves);
    dv_.maxsys = maxsys_;
    dv_.err = arena_.alloc<int>(1);
    params_ = arena_.alloc<double>((size_t)5 * maxsys_);
    SPS_HIP(hipMemsetAsync(dv_.err, 0, sizeof(int), stream));
    SPS_REQUIRE(std::max(iterate_lds(), finish_lds()) <= 160 * 1024, "problem too large for LDS");
    SPS_HIP(hipFuncSetAttribute((const void*)pois_iterate, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)iterate_lds()));
    SPS_HIP(hipFuncSetAttribute((const void*)pois_finish, hipFuncAttributeMaxDynamicSharedMemorySize, (int)finish_lds()));
    SPS_HIP(hipStreamSynchronize(stream));
  }
  static constexpr int kMaxSolves = 1000;   // largest maxit
  size_t iterate_lds() const {
    return sizeof(cplx) * (2 * (size_t)dv_.S + PGW) + (sizeof(double) + sizeof(int)) * (size_t)dv_.mw * dv_.S +
           (size_t)dv_.nb * PTW;
  }
  size_t finish_lds() const { return sizeof(cplx) * 3 * (size_t)dv_.S; }
  // M (real) and its transpose by rows, padded to the longest row
  void upload_m(const PoisBands& hb) {
    const int S = hb.S, bw = hb.kl + hb.ku + 1;
    std::vector<std::vector<std::pair<int, double>>> row[2];
    for (auto& r : row) r.resize(S);
    for (int i = 0; i < S; ++i)
      for (int q = 0; q < bw; ++q) {
        const double2 v = hb.parts[0][(size_t)i * bw + q];
        const int c = i + q - hb.kl;
        if (c < 0 || c >= S || (v.x == 0.0 && v.y == 0.0)) continue;
        SPS_REQUIRE(v.y == 0.0, "the mass matrix is not real");
        row[0][i].push_back({c, v.x});
        row[1][c].push_back({i, v.x});
      }
    int mw = 1;
    for (const auto& r : row)
      for (const auto& e : r) mw = std::max(mw, (int)e.size());
    dv_.mw = mw;
    for (int side = 0; side < 2; ++side) {
      std::vector<int> col((size_t)mw * S, 0);
      std::vector<double> val((size_t)mw * S, 0.0);
      for (int i = 0; i < S; ++i)
        for (size_t e = 0; e < row[side][i].size(); ++e) {
          col[e * S + i] = row[side][i][e].first;
          val[e * S + i] = row[side][i][e].second;
        }
      dv_.mcol[side] = arena_.upload(col, stream);
      dv_.mval[side] = arena_.upload(val, stream);
    }
  }

  void run(int nsys, const double* params, int iters, int mode, double tol, int maxit, double* lam, double* dlam,
           double* info, double* X, double* Y) {
    SPS_REQUIRE(nsys >= 1 && nsys <= maxsys_, "nsys must be in [1, max_systems]");
    SPS_REQUIRE(params && lam && dlam && info, "null argument");
    SPS_REQUIRE(iters >= 1 && iters <= 10000, "iters must be in [1, 10000]");
    SPS_REQUIRE(mode >= 0 && mode <= 3, "mode must be 0, 1, 2 or 3");
    SPS_REQUIRE(maxit >= 1 && maxit <= kMaxSolves, "maxit must be in [1, 1000]");
    SPS_REQUIRE(std::isfinite(tol) && tol >= 0.0, "tol must be finite and >= 0");
    for (int s = 0; s < nsys; ++s) {
      const double* p = params + 5 * s;
      SPS_REQUIRE(std::isfinite(p[0]) && p[0] > 0.0, "alpha must be positive");
      SPS_REQUIRE(std::isfinite(p[1]) && p[1] > 0.0, "Re must be positive");
      SPS_REQUIRE(std::isfinite(p[2]) && std::isfinite(p[3]), "the shift must be finite");
      SPS_REQUIRE(std::isfinite(p[4]), "the continuation step must be finite");
    }
    SPS_HIP(hipMemcpyAsync(params_, params, sizeof(double) * 5 * nsys, hipMemcpyHostToDevice, stream));
    SPS_HIP(hipMemsetAsync(dv_.active, 0, sizeof(int) * maxit, stream));
    PoisArgs a{params_, iters, mode, maxit, tol, reinterpret_cast<cplx*>(lam), reinterpret_cast<cplx*>(dlam), info,
               reinterpret_cast<cplx*>(X), reinterpret_cast<cplx*>(Y)};
    hipLaunchKernelGGL(pois_start, dim3(nsys), dim3(64), 0, stream, dv_, a);
    SPS_CHECK_LAUNCH();
    // one eigenvalue solve per pass; systems that are done skip the later ones, and the passes end when
    // every system is
    for (int it = 0; it < (mode == 0 ? 1 : maxit); ++it) {
      hipLaunchKernelGGL(pois_factor, dim3(nsys), dim3(PTF), 0, stream, dv_);
      hipLaunchKernelGGL(pois_operators, dim3(nsys, 2, (dv_.nb * PGW + PT - 1) / PT), dim3(PT), 0, stream, dv_);
      SPS_CHECK_LAUNCH();
      hipLaunchKernelGGL(pois_iterate, dim3(nsys, 2), dim3(64), iterate_lds(), stream, dv_, iters);
      SPS_CHECK_LAUNCH();
      hipLaunchKernelGGL(pois_finish, dim3(nsys), dim3(PT), finish_lds(), stream, dv_, a, it);
      SPS_CHECK_LAUNCH();
      if (mode != 0 && it + 1 < maxit) {
        int go = 0;
        SPS_HIP(hipMemcpyAsync(&go, dv_.active + it, sizeof(int), hipMemcpyDeviceToHost, stream));
        SPS_HIP(hipStreamSynchronize(stream));
        if (go == 0) break;
      }
    }
    // the host parameters are copied before the call returns
    SPS_HIP(hipStreamSynchronize(stream));
  }

  long long state_size() const override { return 2LL * dv_.S; }
  void factor() override {}
  void step(double*, int) override { unsupported(); }
  void adjoint_step(double*, int) override { unsupported(); }
  void cost(const double*, double*, double*) override { unsupported(); }
  void gradient(const double*, int, const double*, double*, double*, double*, double*) override { unsupported(); }
  void initial_state(const double*, double*) override { unsupported(); }
  void initial_state_adjoint(const double*, double*) override { unsupported(); }
  void eval_F(const double*, double*) override { unsupported(); }
  void eval_F_vjp(const double*, const double*, double*) override { unsupported(); }
  void solve(const double*, double*, int) override { unsupported(); }
  void timer_enable(int, bool) override {}
  void timer_read(long long* l, double* ms) override {
    *l = 0;
    *ms = 0.0;
  }
  int device_error() override {
    int h = 0;
    SPS_HIP(hipMemcpyAsync(&h, dv_.err, sizeof(int), hipMemcpyDeviceToHost, stream));
    SPS_HIP(hipStreamSynchronize(stream));
    if (h) SPS_HIP(hipMemsetAsync(dv_.err, 0, sizeof(int), stream));
    return h;
  }

 private:
  [[noreturn]] static void unsupported() {
    throw Error(SPS_E_UNSUPPORTED, "the plane Poiseuille handle runs the stability problem only");
  }
  DevArena arena_;
  PoisDev dv_{};
  double* params_ = nullptr;
  int maxsys_ = 1;
};

}  // namespace

ProblemImpl* make_poiseuille(int nz, int max_systems, hipStream_t s) { return new PoisProblem(nz, max_systems, s); }

void poiseuille_run(ProblemImpl* p, int nsys, const double* params, int iters, int mode, double tol, int maxit,
                    double* lam, double* dlam, double* info, double* X, double* Y) {
  auto* q = dynamic_cast<PoisProblem*>(p);
  if (!q) throw Error(SPS_E_ARG, "not a plane Poiseuille handle");
  q->run(nsys, params, iters, mode, tol, maxit, lam, dlam, info, X, Y);
}

void poiseuille_host_band(int nz, double alpha, double re, double sig_re, double sig_im, int* S, int* kl, int* ku,
                          double* band, int* rowmap, int* colmap, double* rho) {
  SPS_REQUIRE(nz >= 8 && nz <= 256, "nz must be in [8, 256]");
  PoisBands hb;
  pois_bands(nz, hb);
  *S = hb.S;
  *kl = hb.kl;
  *ku = hb.ku;
  const double nu = 1.0 / re, q2 = nu * alpha * alpha;
  if (band) {
    const size_t cnt = (size_t)hb.S * (hb.kl + hb.ku + 1);
    for (size_t e = 0; e < cnt; ++e) {
      const double2 m = hb.parts[0][e], l0 = hb.parts[1][e], la = hb.parts[2][e], ln = hb.parts[3][e],
                    lq = hb.parts[4][e];
      band[2 * e] = sig_re * m.x - sig_im * m.y + l0.x + alpha * la.x + nu * ln.x + q2 * lq.x;
      band[2 * e + 1] = sig_re * m.y + sig_im * m.x + l0.y + alpha * la.y + nu * ln.y + q2 * lq.y;
    }
  }
  if (rowmap) std::copy(hb.rowmap.begin(), hb.rowmap.end(), rowmap);
  if (colmap) std::copy(hb.colmap.begin(), hb.colmap.end(), colmap);
  if (rho) std::copy(hb.rho.begin(), hb.rho.end(), rho);
}

}  // namespace sps
