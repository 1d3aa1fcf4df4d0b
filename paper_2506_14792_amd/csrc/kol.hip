// 2D Kolmogorov flow in vorticity form on the periodic square [0, 2 pi)^2, a batch of
// independent runs of one size, optionally with a learned closure in the explicit term:
//   omega_t + u . grad omega = nu Laplacian omega - drag omega + f (+ C_theta(omega)),
//   u = (d_y psi, -d_x psi), Laplacian psi = -omega, nu = 1/Re, f = -4 cos 4y.
// IVP form (Supplementary, "Initial value problems"): M = 1, L_k = nu |k|^2 + drag, F = -u.grad omega
// + f (+ closure), the advection formed on the 3/2-padded grid; SBDF2 with an SBDF1 first step
// (equ:imex) and the multistep adjoint recurrence (equ:IMEX_adjoint) with injected cotangents
// of a rollout loss and the closure-parameter gradient (equ:efficient_gradient).
//
// Modes and layouts as the Swift-Hohenberg problem: per instance X[m][iy] (m < N/2 the k_x
// index, iy < N the k_y index in FFT order, iy = N/2 unused), k = integer indices on 2 pi.
// A step is a sequence of launches: column inverse y-FFTs of the fields an evaluation needs
// (u, v, omega_x, omega_y on the 3/2 grid; omega on the N grid for the closure), row x-FFTs
// with the product (or its VJP), the closure network on the N x N vorticity, and a column
// pass with the forward y-FFTs, F and the diagonal solve (or the adjoint combination).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <memory>
#include <type_traits>
#include <vector>

#include "block_fft.h"
#include "cnn.h"
#include "sps_device.h"
#include "sps_internal.h"

namespace sps {
namespace {

constexpr int NTK = 256;
constexpr size_t kLdsMax = 160 * 1024;
constexpr size_t kLdsBudget = 80 * 1024;

struct KolDev {
  int B, N, Nh, Ng;
  double nu, drag, dt;
  int pN, pNg;              // FFT plans of lengths N and Ng
  const FftPlan* plans;
  const cplx* tw;
  const int* twoff;
};

__device__ __forceinline__ int kol_pad_row(int iy, int N, int G) {
  if (iy < N / 2) return iy;
  if (iy == N / 2) return -1;
  return iy - N + G;
}
__device__ __forceinline__ double kol_ky(int iy, int N) { return (iy < N / 2) ? (double)iy : (double)(iy - N); }

struct SbdfC {
  double a0, a1, a2, c1, c2;
};
__device__ __forceinline__ SbdfC sbdf_c(int n, double dt) {
  if (n == 1) return {1.0 / dt, -1.0 / dt, 0.0, 1.0, 0.0};
  return {1.5 / dt, -2.0 / dt, 0.5 / dt, 2.0, -1.0};
}

// spectral factor of derived field f of the vorticity at mode (m, iy): 0 u = i ky/|k|^2,
// 1 v = -i kx/|k|^2, 2 omega_x = i kx, 3 omega_y = i ky; ONE = 1
enum FieldSet { FS_PRIMAL4 = 0, FS_ONE = 1 };
__device__ __forceinline__ cplx field_factor(int f, int m, int iy, int N) {
  const double kx = m, ky = kol_ky(iy, N), k2 = kx * kx + ky * ky;
  const double ik2 = (k2 > 0.0) ? 1.0 / k2 : 0.0;
  switch (f) {
    case 0: return cmk(0.0, ky * ik2);
    case 1: return cmk(0.0, -kx * ik2);
    case 2: return cmk(0.0, kx);
    default: return cmk(0.0, ky);
  }
}

// ---------------------------------------------------------------------------- column inverse
// Z[b][f][y][m] = sum_iy factor_f X[b][m][iy] e^{i k_y y} on a G-point grid, for the tile's
// columns m = c0 .. c0 + tc - 1 and field f = blockIdx.y (of gridDim.y fields).
// Grid (column tiles, fields, instances); LDS twiddles(G) + 2 fpad_size(tc G).
__global__ void __launch_bounds__(NTK) kol_cols_inv(KolDev d, const cplx* X, int set, int G, int plan, int tc,
                                                     cplx* Z) {
  extern __shared__ double smem_d[];
  const int b = blockIdx.z, f = blockIdx.y, nf = gridDim.y, c0 = blockIdx.x * tc, N = d.N, Nh = d.Nh;
  const int tid = threadIdx.x;
  if (c0 >= Nh) return;
  const int tcn = min(tc, Nh - c0);
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  cplx* b1 = b0 + fpad_size(tc * G);
  const cplx* g = d.tw + d.twoff[plan];
  for (int e = tid; e < G; e += NTK) tw[e] = g[e];
  for (int e = tid; e < tcn * G; e += NTK) b0[fpad(e)] = czero();
  __syncthreads();
  const cplx* Xb = X + (long long)b * Nh * N;
  for (int e = tid; e < tcn * N; e += NTK) {
    const int j = e / N, iy = e - j * N, m = c0 + j;
    const int row = kol_pad_row(iy, N, G);
    if (row < 0) continue;
    cplx v = Xb[(long long)m * N + iy];
    if (set == FS_PRIMAL4) v = cmul(v, field_factor(f, m, iy, N));
    b0[fpad(j * G + row)] = v;
  }
  __syncthreads();
  const cplx* o = lds_fft_inline(b0, b1, d.plans[plan], tw, +1, tcn, G, tid, NTK);
  cplx* Zb = Z + ((long long)b * nf + f) * G * Nh + c0;
  for (int e = tid; e < tcn * G; e += NTK) {
    const int y = e / tcn, j = e - y * tcn;
    Zb[(long long)y * Nh + j] = o[fpad(j * G + y)];
  }
}

// ---------------------------------------------------------------------------- rows
// Hermitian packing of two half spectra (rows y, y+1 of one field) into one length-G spectrum
// whose inverse DFT is row_y + i row_(y+1); modes m >= 1 scaled by `scale`.
__device__ __forceinline__ cplx kol_pack(const cplx* U, const cplx* V, int x, int G, int K, double scale) {
  if (x == 0) return cmk(U[0].x, V[0].x);
  if (x < K) return cscale(cmk(U[x].x - V[x].y, U[x].y + V[x].x), scale);
  if (x > G - K) {
    const int q = G - x;
    return cscale(cmk(U[q].x + V[q].y, V[q].x - U[q].y), scale);
  }
  return czero();
}
enum RowMode { R_ADV, R_ADV_VJP, R_GRID, R_FWD_GRID };

// One block per row pair (y, y + 1) of one instance on a G-point grid; y-major field layouts
// Z[b][f][y][m] in and W[b][f][y][m] out.
//  R_ADV:      Z4 (u, v, omega_x, omega_y) -> W = r2c(-(u omega_x + v omega_y))
//  R_ADV_VJP:  Z4 and Zg (the F cotangent, weight-1 modes) -> W4 = r2c of
//              (-qb omega_x, -qb omega_y, -qb u, -qb v), qb = grid cotangent / G^2
//  R_GRID:     Z (one field, modes m >= 1 scaled by `wscale`) -> grid[b][y][x] * gscale
//  R_FWD_GRID: grid[b][y][x] -> W = r2c(grid)
// LDS twiddles(G) + 2 cap, cap >= fpad_size(5 G) when R_ADV_VJP runs, else fpad_size(4 G).
template <int NT>
__global__ void __launch_bounds__(NT) kol_rows(KolDev d, int mode, int G, int plan, int cap, const cplx* Z4,
                                                 const cplx* Zg, double* grid, const double* gin, cplx* W,
                                                 double wscale, double gscale) {
  extern __shared__ double smem_d[];
  const int b = blockIdx.y, y0 = 2 * blockIdx.x, Nh = d.Nh, tid = threadIdx.x;
  const int nin = (mode == R_ADV) ? 4 : (mode == R_ADV_VJP ? 5 : 1);
  const int nout = (mode == R_ADV_VJP) ? 4 : 1;
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  cplx* b1 = b0 + cap;
  const cplx* g = d.tw + d.twoff[plan];
  for (int e = tid; e < G; e += NT) tw[e] = g[e];
  if (mode == R_FWD_GRID) {
    const double* r0 = gin + ((long long)b * G + y0) * G;
    for (int x = tid; x < G; x += NT) b0[fpad(x)] = cmk(r0[x], r0[G + x]);
  } else {
    const int nz = (mode == R_GRID) ? 1 : 4;
    for (int e = tid; e < nin * G; e += NT) {
      const int f = e / G, x = e - f * G;
      const cplx* U = (f == 4) ? Zg + ((long long)b * G + y0) * Nh : Z4 + (((long long)b * nz + f) * G + y0) * Nh;
      const double sc = (mode == R_GRID) ? wscale : (f == 4 ? 0.5 : 1.0);
      b0[fpad(e)] = kol_pack(U, U + Nh, x, G, Nh, sc);
    }
  }
  __syncthreads();
  const FftPlan& P = d.plans[plan];
  cplx* h = (mode == R_FWD_GRID) ? b0 : lds_fft_inline(b0, b1, P, tw, +1, nin, G, tid, NT);
  if (mode == R_GRID) {
    double* r0 = grid + ((long long)b * G + y0) * G;
    for (int x = tid; x < G; x += NT) {
      const cplx v = h[fpad(x)];
      r0[x] = v.x * gscale;
      r0[G + x] = v.y * gscale;
    }
    return;
  }
  cplx* o = h;
  if (mode != R_FWD_GRID) {
    o = (h == b0) ? b1 : b0;
    const double inv2 = 1.0 / ((double)G * G);
    for (int x = tid; x < G; x += NT) {
      const cplx u = h[fpad(x)], v = h[fpad(G + x)], wx = h[fpad(2 * G + x)], wy = h[fpad(3 * G + x)];
      if (mode == R_ADV) {
        o[fpad(x)] = cmk(-(u.x * wx.x + v.x * wy.x), -(u.y * wx.y + v.y * wy.y));
      } else {
        const cplx q = h[fpad(4 * G + x)];
        const double qa = -q.x * inv2, qb = -q.y * inv2;
        o[fpad(x)] = cmk(qa * wx.x, qb * wx.y);           // u bar
        o[fpad(G + x)] = cmk(qa * wy.x, qb * wy.y);       // v bar
        o[fpad(2 * G + x)] = cmk(qa * u.x, qb * u.y);     // omega_x bar
        o[fpad(3 * G + x)] = cmk(qa * v.x, qb * v.y);     // omega_y bar
      }
    }
    __syncthreads();
  }
  cplx* o2 = (o == b0) ? b1 : b0;
  const cplx* r = lds_fft_inline(o, o2, P, tw, -1, nout, G, tid, NT);
  // unpack the two real rows' half spectra: Y_y = (Z_m + conj Z_-m) / 2, Y_y+1 = (Z_m - conj Z_-m) / 2i
  for (int e = tid; e < nout * 2 * Nh; e += NT) {
    const int f = e / (2 * Nh), rr = e - f * 2 * Nh, yy = rr / Nh, m = rr - yy * Nh;
    const cplx zm = r[fpad(f * G + m)], zq = r[fpad(f * G + (m == 0 ? 0 : G - m))];
    const cplx v = yy ? cmk(0.5 * (zm.y + zq.y), -0.5 * (zm.x - zq.x)) : cmk(0.5 * (zm.x + zq.x), 0.5 * (zm.y - zq.y));
    W[(((long long)b * nout + f) * G + y0 + yy) * Nh + m] = v;
  }
}

// The advection product of one row pair in two passes of two fields each (u, omega_x, then
// v, omega_y), so that long rows fit two blocks per CU: LDS twiddles(G) + 2 fpad_size(2 G) +
// fpad_size(G).  Same result as kol_rows in mode R_ADV up to the order of the two products.
template <int NT>
__global__ void __launch_bounds__(NT) kol_rows_adv2(KolDev d, int G, int plan, const cplx* Z4, cplx* W) {
  extern __shared__ double smem_d[];
  const int b = blockIdx.y, y0 = 2 * blockIdx.x, Nh = d.Nh, tid = threadIdx.x;
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  cplx* b1 = b0 + fpad_size(2 * G);
  cplx* pr = b1 + fpad_size(2 * G);
  const cplx* g = d.tw + d.twoff[plan];
  for (int e = tid; e < G; e += NT) tw[e] = g[e];
  const FftPlan& P = d.plans[plan];
  for (int pass = 0; pass < 2; ++pass) {
    // pass 0: fields 0 (u) and 2 (omega_x); pass 1: fields 1 (v) and 3 (omega_y)
    for (int e = tid; e < 2 * G; e += NT) {
      const int q = e / G, x = e - q * G, f = pass + 2 * q;
      const cplx* U = Z4 + (((long long)b * 4 + f) * G + y0) * Nh;
      b0[fpad(e)] = kol_pack(U, U + Nh, x, G, Nh, 1.0);
    }
    __syncthreads();
    const cplx* h = lds_fft_inline(b0, b1, P, tw, +1, 2, G, tid, NT);
    for (int x = tid; x < G; x += NT) {
      const cplx a = h[fpad(x)], c = h[fpad(G + x)];
      const cplx p = cmk(-(a.x * c.x), -(a.y * c.y));
      pr[fpad(x)] = pass ? cmk(pr[fpad(x)].x + p.x, pr[fpad(x)].y + p.y) : p;
    }
    __syncthreads();
  }
  const cplx* r = lds_fft_inline(pr, b0, P, tw, -1, 1, G, tid, NT);
  for (int e = tid; e < 2 * Nh; e += NT) {
    const int yy = e / Nh, m = e - yy * Nh;
    const cplx zm = r[fpad(m)], zq = r[fpad(m == 0 ? 0 : G - m)];
    const cplx v = yy ? cmk(0.5 * (zm.y + zq.y), -0.5 * (zm.x - zq.x)) : cmk(0.5 * (zm.x + zq.x), 0.5 * (zm.y - zq.y));
    W[((long long)b * G + y0 + yy) * Nh + m] = v;
  }
}

// ---------------------------------------------------------------------------- column pass
enum ColMode { K_STEP, K_EVALF, K_ADJ, K_ADJ_INIT, K_VJP };
struct KolCol {
  int mode, n, nsteps, closure;
  const cplx* W;     // [B][nW][Nh][Ng] products' x-spectra (1 field, or 4 for the VJP)
  const cplx* Wc;    // [B][Nh][N] closure x-spectra (nullable)
  cplx* H;           // history [nh][B][Nh][N]
  int hring;         // 0: full history; else ring of hring states
  cplx* Fr;          // F ring [2][B][Nh][N]
  cplx* Yn;          // Y_(k+1) [B][Nh][N]
  cplx* Ln;          // linear part
  cplx* Gk;          // F cotangent for the next VJP
  const cplx* targ;  // rollout targets [nsteps][B][Nh][N] (nullable)
  const cplx* xin;   // K_ADJ_INIT: external dJ/dX_N (nullable)
  cplx* out;         // K_EVALF: F; K_VJP: Xbar; K_ADJ (k = 0): dJ/dX_0; K_STEP (n = nsteps): X_N (nullable)
  cplx* snap;        // K_STEP: filtered snapshots (nullable)
  int snap_every, Nc;
  int* err;          // sticky flags: bit 1 non-finite state
};

__device__ __forceinline__ long long hidx(const KolCol& a, int k, long long st) {
  return (long long)(a.hring ? (k % a.hring) : k) * st;
}

// One mode of a forward step: the SBDF solve with F of state n - 1, its records and (on snapshot steps) the
// truncation to the coarse grid's modes.  keep: not the Nyquist row.
struct StepIn {
  cplx f2, x1, x2;
};
__device__ __forceinline__ StepIn kol_step_load(const KolCol& a, long long st, long long si) {
  const int n = a.n;
  StepIn r;
  r.f2 = (n >= 2) ? a.Fr[(n & 1) * st + si] : czero();
  r.x1 = a.H[hidx(a, n - 1, st) + si];
  r.x2 = (n >= 2) ? a.H[hidx(a, n - 2, st) + si] : czero();
  return r;
}
__device__ __forceinline__ void kol_step_entry(const KolDev& d, const KolCol& a, int b, int m, int iy, bool keep, cplx F,
                                               const StepIn& in, double lin, long long st, long long si) {
  const int n = a.n, N = d.N;
  const SbdfC q = sbdf_c(n, d.dt);
  cplx xn = czero();
  if (keep) {
    cplx rhs = cadd(cscale(F, q.c1), cscale(in.f2, q.c2));
    rhs = csub(rhs, cadd(cscale(in.x1, q.a1), cscale(in.x2, q.a2)));
    xn = cscale(rhs, 1.0 / (q.a0 + lin));
  }
  a.Fr[((n - 1) & 1) * st + si] = F;
  a.H[hidx(a, n, st) + si] = xn;
  if (!(isfinite(xn.x) && isfinite(xn.y))) atomicOr(a.err, 2);
  if (n == a.nsteps && a.out) a.out[si] = xn;
  if (a.snap && n % a.snap_every == 0) {
    // spectral truncation to the Nc x Nc modes of the coarse grid
    const int Nch = a.Nc / 2;
    const int sy = (iy < N / 2) ? iy : iy - N;
    if (m < Nch && sy >= -Nch && sy < Nch) {   // sy = -Nch: the coarse Nyquist row, kept zero
      const int ic = (sy >= 0) ? sy : sy + a.Nc;
      a.snap[((long long)(n / a.snap_every - 1) * d.B + b) * Nch * a.Nc + (long long)m * a.Nc + ic] =
          (sy == -Nch) ? czero() : xn;
    }
  }
}

// Grid (column tiles, instances).  LDS twiddles(Ng) + twiddles(N) + 2 wcap (wcap >=
// fpad_size(nW tc Ng)) + 2 fpad_size(tc N) when the closure runs.
__global__ void __launch_bounds__(NTK) kol_cols_fwd(KolDev d, KolCol a, int tc, int wcap) {
  extern __shared__ double smem_d[];
  const int b = blockIdx.y, c0 = blockIdx.x * tc, N = d.N, Nh = d.Nh, Ng = d.Ng, tid = threadIdx.x;
  if (c0 >= Nh) return;
  const int tcn = min(tc, Nh - c0);
  const bool adj = (a.mode == K_ADJ || a.mode == K_VJP);
  const int nW = (a.mode == K_ADJ_INIT) ? 0 : (adj ? 4 : 1);
  const bool clo = a.closure && a.mode != K_ADJ_INIT;
  cplx* twg = reinterpret_cast<cplx*>(smem_d);
  cplx* twn = twg + Ng;
  cplx* b0 = twn + N;
  cplx* b1 = b0 + wcap;
  cplx* c0b = b1 + wcap;
  cplx* c1b = c0b + fpad_size(tc * N);
  for (int e = tid; e < Ng; e += NTK) twg[e] = d.tw[d.twoff[d.pNg] + e];
  for (int e = tid; e < N; e += NTK) twn[e] = d.tw[d.twoff[d.pN] + e];
  for (int e = tid; e < nW * Ng * tcn; e += NTK) {
    const int f = e / (Ng * tcn), r = e - f * Ng * tcn, y = r / tcn, j = r - y * tcn;
    b0[fpad((f * tcn + j) * Ng + y)] = a.W[(((long long)b * nW + f) * Ng + y) * Nh + c0 + j];
  }
  if (clo)
    for (int e = tid; e < N * tcn; e += NTK) {
      const int y = e / tcn, j = e - y * tcn;
      c0b[fpad(j * N + y)] = a.Wc[((long long)b * N + y) * Nh + c0 + j];
    }
  __syncthreads();
  const cplx* res = (nW > 0) ? lds_fft_inline(b0, b1, d.plans[d.pNg], twg, -1, nW * tcn, Ng, tid, NTK) : nullptr;
  const cplx* rc = clo ? lds_fft_inline(c0b, c1b, d.plans[d.pN], twn, -1, tcn, N, tid, NTK) : nullptr;
  const long long st = (long long)d.B * Nh * N, io = (long long)b * Nh * N;
  const double ng2 = 1.0 / ((double)Ng * Ng), n2 = 1.0 / ((double)N * N);
  for (int e = tid; e < tcn * N; e += NTK) {
    const int j = e / N, iy = e - j * N, m = c0 + j;
    const long long si = io + (long long)m * N + iy;
    const int row = kol_pad_row(iy, N, Ng), rowc = kol_pad_row(iy, N, N);
    const double k2 = (double)m * m + kol_ky(iy, N) * kol_ky(iy, N);
    const double lin = d.nu * k2 + d.drag, wm = (m == 0) ? 1.0 : 2.0;
    if (a.mode == K_STEP || a.mode == K_EVALF) {
      cplx F = czero();
      if (row >= 0) {
        F = cscale(res[fpad(j * Ng + row)], ng2);
        if (m == 0 && N > 8 && (iy == 4 || iy == N - 4)) F = cadd(F, cmk(-2.0, 0.0));   // -4 cos 4y
        if (clo) F = cadd(F, cscale(rc[fpad(j * N + rowc)], n2));
      }
      if (a.mode == K_EVALF) {
        a.out[si] = F;
        continue;
      }
      kol_step_entry(d, a, b, m, iy, row >= 0, F, kol_step_load(a, st, si), lin, st, si);
      continue;
    }
    // reverse sweep: xb of state k (K_ADJ: k = n - 1 from the VJP; K_ADJ_INIT: k = nsteps)
    cplx xb = czero();
    if (a.mode == K_ADJ || a.mode == K_VJP) {
      if (row >= 0) {
        for (int f = 0; f < 4; ++f) {
          const cplx t = cscale(res[fpad((f * tcn + j) * Ng + row)], wm);
          const cplx fac = field_factor(f, m, iy, N);
          xb = cadd(xb, cmul(cconj(fac), t));
        }
        if (clo) xb = cadd(xb, cscale(rc[fpad(j * N + rowc)], wm));
      }
      if (a.mode == K_VJP) {
        a.out[si] = xb;
        continue;
      }
      xb = csub(xb, a.Ln[si]);
    } else if (a.xin && row >= 0) {
      xb = a.xin[si];
    }
    const int k = (a.mode == K_ADJ) ? a.n - 1 : a.nsteps;
    if (a.targ && k >= 1 && row >= 0) {
      // d/dX_k of (1/nsteps) mean over the N x N grid of (omega_k - target_k)^2
      const cplx* T = a.targ + (long long)(k - 1) * st;
      cplx e1 = csub(a.H[hidx(a, k, st) + si], T[si]);
      if (m == 0) {
        const long long sm = io + (long long)((N - iy) % N);
        const cplx e2 = csub(a.H[hidx(a, k, st) + sm], T[sm]);
        e1 = cmk(0.5 * (e1.x + e2.x), 0.5 * (e1.y - e2.y));
      }
      xb = cadd(xb, cscale(e1, 2.0 * wm / a.nsteps));
    }
    if (k == 0) {
      a.out[si] = xb;
      continue;
    }
    cplx y = czero(), g = czero(), l = czero();
    if (row >= 0) {
      const SbdfC q = sbdf_c(k, d.dt);
      y = cscale(xb, 1.0 / (q.a0 + lin));
      g = cscale(y, q.c1);
      l = cscale(y, q.a1);
      if (k + 1 <= a.nsteps) {
        const SbdfC qn = sbdf_c(k + 1, d.dt);
        g = cadd(g, cscale(a.Yn[si], qn.c2));
        l = cadd(l, cscale(a.Yn[si], qn.a2));
      }
    }
    a.Yn[si] = y;
    a.Ln[si] = l;
    a.Gk[si] = g;
  }
}

// ---------------------------------------------------------------------------- steps of a known grid length
// The kernels of a step and of a reverse step on block_fft.h, for the padded lengths it has a plan for: columns
// and row pairs are transformed in place with the first pass read from memory and the last one used in
// registers.  At N = 512, six instances: columns inverse 61 -> 22 us (113 MB moved), rows 87 -> 42 (94 MB), columns
// forward 34 -> 20 (113 MB).  Bound by LDS and the vector unit together in the rows (some 17 and 14 us of the 42), by
// memory in the columns.  At training sizes (N = 64, 16 instances, closure) a launch costs 4 to 5 us whatever it does, most
// of it the launch and the first loads, so independent passes share one: a forward and a reverse step took 6 row
// launches of 6.1 us and one of 5.2, now 4 of 4.1 to 7.4 (42 -> 21 us together), and 6 launches of column inverses of
// 4.8 us and 2 column passes of 12, now 2 of 5.0 and one each of 5.4 and 6.1 (53 -> 22 us).
template <int G>
struct KolFft {
  static constexpr int N = 2 * G / 3, Nh = G / 3, R0 = BlockPlan<G>::R0, R1 = BlockPlan<G>::R1;
  // columns of a block, and row pairs of a block: about 200 to 400 threads of one butterfly each, and no more
  // LDS than lets two blocks share a CU
  static constexpr int TC = G >= 576 ? 4 : 8, PAIRS = G >= 576 ? 1 : (G == 48 ? 4 : 2);
  static constexpr int NTC = TC * G / R0, NTR = 4 * PAIRS * G / R0;
  static constexpr size_t lds_cols = sizeof(cplx) * (G + bf_size(TC * G)), lds_rows = sizeof(cplx) * (G + bf_size(4 * PAIRS * G));
  static constexpr size_t lds_vjp = lds_rows + sizeof(cplx) * bf_size(PAIRS * G);
  // row pairs of a block on the N-point grid: as many as the padded rows' threads take
  static constexpr int PN = 4 * PAIRS, NTN = PN * N / BlockPlan<N>::R0;
  static constexpr size_t lds_n = sizeof(cplx) * (N + bf_size(PN * N));
  // columns of a block with the four products of a reverse step: up to 512 threads (with the closure's) where that
  // leaves two columns, as beyond registers spill.  At 768 points two columns take 768 threads and the closure's 128: 128
  // registers a lane, of which that instantiation (kol_cols_adj_b<768, true>) spills 76 bytes.
  static constexpr int TA = G >= 288 ? 2 : 4, NTA = 4 * TA * G / R0;
  // threads of the closure's columns beside those of the padded ones, from a wave's start
  static constexpr int wave(int n) { return (n + 63) / 64 * 64; }
  static constexpr int step_threads(bool clo) { return clo ? wave(NTC) + TC * N / BlockPlan<N>::R0 : NTC; }
  static constexpr int adj_threads(bool clo) { return clo ? wave(NTA) + TA * N / BlockPlan<N>::R0 : NTA; }
  static constexpr size_t lds_clo(int tc) { return sizeof(cplx) * (N + bf_size(tc * N)); }
  static constexpr size_t lds_step(bool clo) { return lds_cols + (clo ? lds_clo(TC) : 0); }
  static constexpr size_t lds_adj(bool clo) { return sizeof(cplx) * (G + bf_size(4 * TA * G)) + (clo ? lds_clo(TA) : 0); }
  static_assert(Nh % TC == 0 && Nh % TA == 0 && (G / 2) % PAIRS == 0 && (N / 2) % PN == 0, "tiles");
  static_assert(TC * N / BlockPlan<N>::R0 <= NTC && NTN <= NTR, "the N-point grid's blocks fit the padded grid's");
  static_assert(adj_threads(true) <= 1024 && lds_adj(true) <= kLdsMax && lds_vjp <= kLdsMax, "one block");
};
// Column tile of a block.  Tiles of four columns write half of a 128-byte line: the two halves' blocks are
// dealt to the same XCD, one after the other.
template <int TC>
__device__ __forceinline__ int kol_tile(int x, int tiles) {
  return (TC == 4 && tiles % 16 == 0) ? ((x & ~15) | ((x & 7) << 1) | ((x >> 3) & 1)) : x;
}

// One block's columns c0 .. c0 + TC - 1 of kol_cols_inv on an L-point grid: Xb and Zb are the instance's states and
// the field's grid, f < 4 one of the derived fields.
template <int L, int N, int TC, int NT>
__device__ __forceinline__ void kol_inv_columns(const cplx* Xb, int f, cplx* Zb, const cplx* g, int c0, int tid,
                                                double* smem) {
  constexpr int R0 = BlockPlan<L>::R0, NR = L / R0, Nh = N / 2;
  using F = BlockFft<L, TC, NT, 4, 1>;   // the states have a column's modes next to each other, Z a row's
  static_assert(F::First::MB == 1 && F::Last::MB == 1, "one butterfly a thread");
  cplx* tw = reinterpret_cast<cplx*>(smem);
  cplx* buf = tw + L;
  const bool act = F::First::full || tid < F::First::NB;
  const int j = F::First::bfly(tid), m = c0 + F::First::seq(tid);
  const cplx* Xc = Xb + (long long)m * N;
  cplx v[1][R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) {   // grid position p holds mode p (p < N / 2) or p - L + N (p > L - N / 2)
    const int p = j + r * NR;
    v[0][r] = czero();
    if (r * NR >= N / 2 && (r + 1) * NR - 1 <= L - N / 2) continue;
    if (act && (p < N / 2 || p > L - N / 2)) v[0][r] = Xc[p < N / 2 ? p : p - L + N];
  }
  for (int e = tid; e < L; e += NT) tw[e] = g[e];
  if (f < 4) {
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      if (r * NR >= N / 2 && (r + 1) * NR - 1 <= L - N / 2) continue;
      const int p = j + r * NR;
      v[0][r] = cmul(v[0][r], field_factor(f, m, p < N / 2 ? p : p - L + N, N));
    }
  }
  F::First::work(v, tw, +1, tid);   // (the first pass has no twiddles)
  F::First::write(v, buf, tid);
  F::rest(v, buf, tw, +1, tid);
  if (!act) return;
  cplx* Zc = Zb + (long long)F::Last::bfly(tid) * Nh + c0 + F::Last::seq(tid);
#pragma unroll
  for (int r = 0; r < R0; ++r) Zc[(long long)r * NR * Nh] = v[0][r];
}

// All column inverses of an evaluation (or of its VJP with the cotangent Fb) in one launch, which at training
// sizes costs what each of them would: at N = 64, 16 instances, 5.0 us, and 4.6 for the four fields alone.  blockIdx.y: 0 .. 3 the fields of X on the padded grid -> Z4; then with Fb: Fb on the padded grid ->
// Zg; then with the closure: X on the N-point grid -> Zc, and with Fb: Fb on it -> Zgc.
// Grid (column tiles, fields, instances).
struct KolInv {
  const cplx *X, *Fb;
  cplx *Z4, *Zg, *Zc, *Zgc;
};
template <int G, bool CLO>
__global__ void __launch_bounds__(KolFft<G>::NTC) kol_cols_inv_b(KolDev d, KolInv a) {
  using P = KolFft<G>;
  constexpr int N = P::N, Nh = P::Nh, TC = P::TC;
  extern __shared__ double smem_d[];
  const int b = blockIdx.z, c0 = TC * kol_tile<TC>(blockIdx.x, gridDim.x), tid = threadIdx.x;
  const int f = blockIdx.y + (blockIdx.y >= 4 && !a.Fb);   // 4 Zg, 5 Zc, 6 Zgc
  const cplx* Xb = ((f == 4 || f == 6) ? a.Fb : a.X) + (long long)b * Nh * N;
  if (!CLO || f <= 4) {   // (without the closure the kernel keeps to the registers of the padded columns)
    cplx* Zb = (f < 4) ? a.Z4 + ((long long)b * 4 + f) * G * Nh : a.Zg + (long long)b * G * Nh;
    kol_inv_columns<G, N, TC, P::NTC>(Xb, f, Zb, d.tw + d.twoff[d.pNg], c0, tid, smem_d);
  } else {
    kol_inv_columns<N, N, TC, P::NTC>(Xb, f, (f == 5 ? a.Zc : a.Zgc) + (long long)b * N * Nh, d.tw + d.twoff[d.pN], c0, tid,
                                      smem_d);
  }
}

// Inputs of the first inverse pass of butterfly j of a row pair (kol_pack): U the first row's half spectrum of Nh
// modes, the second one's behind it; x < Nh direct, x > L - Nh mirrored, zero between.
template <int L, int Nh>
__device__ __forceinline__ void kol_load_pair(cplx (&v)[BlockPlan<L>::R0], const cplx* U, int j) {
  constexpr int R0 = BlockPlan<L>::R0, NR = L / R0;
  cplx u[R0], w[R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    u[r] = w[r] = czero();
    if (r * NR >= Nh && (r + 1) * NR - 1 <= L - Nh) continue;
    const int x = j + r * NR;
    if (x < Nh || x > L - Nh) {
      const int i = x < Nh ? x : L - x;
      u[r] = U[i];
      w[r] = U[Nh + i];
    }
  }
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    const int x = j + r * NR;
    if (x == 0) u[r].y = w[r].y = 0.0;
    v[r] = (x < Nh) ? cmk(u[r].x - w[r].y, u[r].y + w[r].x) : cmk(u[r].x + w[r].y, w[r].x - u[r].y);
  }
}
// Half spectrum entry m of row yy of the pair in sequence q of TC: Y_y = (Z_m + conj Z_-m) / 2, Y_y+1 = (Z_m -
// conj Z_-m) / 2i.
template <int L, int TC>
__device__ __forceinline__ cplx kol_unpack(const cplx* buf, int m, int yy, int q) {
  const cplx zm = buf[bf_pad(m * TC + q)], zq = buf[bf_pad((m == 0 ? 0 : L - m) * TC + q)];
  return yy ? cmk(0.5 * (zm.y + zq.y), -0.5 * (zm.x - zq.x)) : cmk(0.5 * (zm.x + zq.x), 0.5 * (zm.y - zq.y));
}

// kol_rows in mode R_GRID for the PN row pairs from pair0 of one instance: Zb its field, grid its values.
template <int N, int PN, int NT>
__device__ __forceinline__ void kol_grid_rows(const cplx* Zb, double* grid, const cplx* g, int pair0, double wscale,
                                              double gscale, int tid, double* smem) {
  constexpr int R0 = BlockPlan<N>::R0, NR = N / R0, Nh = N / 2;
  using F = BlockFft<N, PN, NT, 4, 8>;
  static_assert(F::First::MB == 1 && F::Last::MB == 1, "one butterfly a thread");
  cplx* tw = reinterpret_cast<cplx*>(smem);
  cplx* buf = tw + N;
  const bool act = F::First::full || tid < F::First::NB;
  cplx v[1][R0];
  if (act) {
    const int j = F::First::bfly(tid);
    kol_load_pair<N, Nh>(v[0], Zb + (long long)2 * (pair0 + F::First::seq(tid)) * Nh, j);
#pragma unroll
    for (int r = 0; r < R0; ++r)
      if (j + r * NR != 0) v[0][r] = cscale(v[0][r], wscale);
  }
  for (int e = tid; e < N; e += NT) tw[e] = g[e];
  F::First::work(v, tw, +1, tid);
  F::First::write(v, buf, tid);
  F::rest(v, buf, tw, +1, tid);
  if (!act) return;
  double* r0 = grid + (long long)2 * (pair0 + F::Last::seq(tid)) * N + F::Last::bfly(tid);
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    r0[r * NR] = v[0][r].x * gscale;
    r0[N + r * NR] = v[0][r].y * gscale;
  }
}

// Rows of the closure's grids behind the padded ones in the same launch, blocks from G / 2 / PAIRS on: og = X on the
// grid, then (VJP) yg = the F cotangent's transpose.
struct KolGrids {
  const cplx *Zc, *Zgc;
  double *og, *yg;
};
template <int G>
__device__ __forceinline__ bool kol_closure_rows(const KolDev& d, const KolGrids& c, double* smem) {
  using P = KolFft<G>;
  constexpr int N = P::N, blocks = N / 2 / P::PN;
  const int x = blockIdx.x - G / 2 / P::PAIRS;
  if (x < 0) return false;
  const bool cot = x >= blocks;
  const long long b = blockIdx.y;
  kol_grid_rows<N, P::PN, P::NTR>((cot ? c.Zgc : c.Zc) + b * N * P::Nh, (cot ? c.yg : c.og) + b * N * N,
                                  d.tw + d.twoff[d.pN], (x - (cot ? blocks : 0)) * P::PN, cot ? 0.5 : 1.0,
                                  cot ? 1.0 / ((double)N * N) : 1.0, threadIdx.x, smem);
  return true;
}

// kol_rows in mode R_ADV.  The four fields of a row pair are in one row of 16 lanes, so the products are formed
// by lane exchanges in the last inverse pass, whose outputs are the inputs of the forward transform's
// first.  Grid (G / 2 / PAIRS [+ closure rows], instances).
template <int G, bool CLO>
__global__ void __launch_bounds__(KolFft<G>::NTR) kol_rows_adv_b(KolDev d, const cplx* Z4, cplx* W, KolGrids c) {
  using P = KolFft<G>;
  constexpr int Nh = P::Nh, R0 = P::R0, PAIRS = P::PAIRS, TC = 4 * PAIRS, NT = P::NTR;
  using FI = BlockFft<G, TC, NT, 4, 4>;
  using FF = BlockFft<G, PAIRS, NT, 1, 1>;
  static_assert(FI::First::MB == 1 && FI::First::full && FF::Last::MB == 1, "one butterfly a thread");
  extern __shared__ double smem_d[];
  if (CLO && kol_closure_rows<G>(d, c, smem_d)) return;
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  const int b = blockIdx.y, tid = threadIdx.x, j = FI::First::bfly(tid), f = FI::First::seq(tid) & 3, pr = FI::First::seq(tid) >> 2;
  const cplx* g = d.tw + d.twoff[d.pNg];
  cplx v[1][R0];
  kol_load_pair<G, Nh>(v[0], Z4 + (((long long)b * 4 + f) * G + 2 * (blockIdx.x * PAIRS + pr)) * Nh, j);
  for (int e = tid; e < G; e += NT) tw[e] = g[e];
  FI::First::work(v, tw, +1, tid);
  FI::First::write(v, buf, tid);
  FI::rest(v, buf, tw, +1, tid);
  // the fields are on lanes 4 f + (0 .. 3) of a row of 16: u omega_x (f = 0, 2; a turn by 8) + v omega_y (f =
  // 1, 3; by 4), the two rows in the two parts
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    const double x = v[0][r].x * dpp_d<0x128>(v[0][r].x), y = v[0][r].y * dpp_d<0x128>(v[0][r].y);
    v[0][r] = cmk(-(x + dpp_d<0x124>(x)), -(y + dpp_d<0x124>(y)));
  }
  FI::First::work(v, tw, -1, tid);   // the forward transform's first pass: in every field's lanes, one writes
  if (f == 0) {
    const int base = j * R0 * PAIRS + pr;
#pragma unroll
    for (int r = 0; r < R0; ++r) buf[bf_pad(base + r * PAIRS)] = v[0][r];
  }
  FF::rest(v, buf, tw, -1, tid);
  if (FF::Last::full || tid < FF::Last::NB) FF::Last::write(v, buf, tid);
  __syncthreads();
  for (int e = tid; e < PAIRS * 2 * Nh; e += NT) {
    const int rr = e / Nh, m = e - rr * Nh, yy = rr & 1, p = rr >> 1;
    W[((long long)b * G + 2 * (blockIdx.x * PAIRS + p) + yy) * Nh + m] = kol_unpack<G, PAIRS>(buf, m, yy, p);
  }
}

// kol_rows in mode R_ADV_VJP.  As kol_rows_adv_b, with the cotangent's row pairs transformed beside the fields': a
// quarter of the threads has its first two passes' butterflies as well, and the last pass of butterfly j is
// computed in the lanes of all four fields, which then have the cotangent q where they have their field; output f
// is -q times the field a turn by 8 away.  7.4 us at N = 64, 16 instances, with the closure's rows.
template <int G, bool CLO>
__global__ void __launch_bounds__(KolFft<G>::NTR) kol_rows_vjp_b(KolDev d, const cplx* Z4, const cplx* Zg, cplx* W, KolGrids c) {
  using P = KolFft<G>;
  constexpr int Nh = P::Nh, R0 = P::R0, R1 = P::R1, PAIRS = P::PAIRS, TC = 4 * PAIRS, NT = P::NTR;
  using FI = BlockFft<G, TC, NT, 4, 4>;
  using FQ = BlockFft<G, PAIRS, NT, 4, 1>;
  static_assert(FI::First::MB == 1 && FI::First::full, "one butterfly a thread");
  extern __shared__ double smem_d[];
  if (CLO && kol_closure_rows<G>(d, c, smem_d)) return;
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  cplx* bufq = buf + bf_size(TC * G);
  const int b = blockIdx.y, tid = threadIdx.x, j = FI::First::bfly(tid), f = FI::First::seq(tid) & 3, pr = FI::First::seq(tid) >> 2;
  const int y0 = 2 * blockIdx.x * PAIRS;
  const cplx* g = d.tw + d.twoff[d.pNg];
  cplx v[1][R0], q[1][R0];
  kol_load_pair<G, Nh>(v[0], Z4 + (((long long)b * 4 + f) * G + y0 + 2 * pr) * Nh, j);
  if (tid < FQ::First::NB) {
    const int jq = FQ::First::bfly(tid);
    kol_load_pair<G, Nh>(q[0], Zg + ((long long)b * G + y0 + 2 * FQ::First::seq(tid)) * Nh, jq);
#pragma unroll
    for (int r = 0; r < R0; ++r)   // F's cotangent has weight-1 modes
      if (jq + r * (G / R0) != 0) q[0][r] = cscale(q[0][r], 0.5);
    FQ::First::work_one(q[0], tw, +1, tid);
    FQ::First::write_one(q[0], bufq, tid);
  }
  for (int e = tid; e < G; e += NT) tw[e] = g[e];
  FI::First::work(v, tw, +1, tid);
  FI::First::write(v, buf, tid);
  {
    cplx m[FI::Mid::MB][R1], mq[FQ::Mid::MB][R1];
    __syncthreads();
    FI::Mid::read(m, buf, tid);
    FQ::Mid::read(mq, bufq, tid);
    __syncthreads();
    FI::Mid::work(m, tw, +1, tid);
    FI::Mid::write(m, buf, tid);
    FQ::Mid::work(mq, tw, +1, tid);
    FQ::Mid::write(mq, bufq, tid);
  }
  __syncthreads();
  FI::Last::read(v, buf, tid);
  FQ::Last::read_one(q[0], bufq, j * PAIRS + pr);
  __syncthreads();
  FI::Last::work(v, tw, +1, tid);
  FQ::Last::work_one(q[0], tw, +1, j * PAIRS + pr);
  const double inv2 = 1.0 / ((double)G * G);
#pragma unroll
  for (int r = 0; r < R0; ++r)   // u bar = qb omega_x, v bar = qb omega_y, omega_x bar = qb u, omega_y bar = qb v
    v[0][r] = cmk(-q[0][r].x * inv2 * dpp_d<0x128>(v[0][r].x), -q[0][r].y * inv2 * dpp_d<0x128>(v[0][r].y));
  FI::First::work(v, tw, -1, tid);
  FI::First::write(v, buf, tid);
  FI::rest(v, buf, tw, -1, tid);
  FI::Last::write(v, buf, tid);
  __syncthreads();
  for (int e = tid; e < TC * 2 * Nh; e += NT) {
    const int rr = e / Nh, m = e - rr * Nh, yy = rr & 1, s = rr >> 1;
    W[(((long long)b * 4 + (s & 3)) * G + y0 + 2 * (s >> 2) + yy) * Nh + m] = kol_unpack<G, TC>(buf, m, yy, s);
  }
}

// kol_rows in mode R_FWD_GRID.  Grid (N / 2 / PN, instances).
template <int G>
__global__ void __launch_bounds__(KolFft<G>::NTN) kol_rows_fwd_b(KolDev d, const double* gin, cplx* W) {
  using P = KolFft<G>;
  constexpr int N = P::N, Nh = P::Nh, PN = P::PN, NT = P::NTN, R0 = BlockPlan<N>::R0, NR = N / R0;
  using F = BlockFft<N, PN, NT, 8, 1>;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + N;
  const int b = blockIdx.y, tid = threadIdx.x, y0 = 2 * blockIdx.x * PN;
  const cplx* g = d.tw + d.twoff[d.pN];
  const double* r0 = gin + ((long long)b * N + y0 + 2 * F::First::seq(tid)) * N + F::First::bfly(tid);
  cplx v[1][R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) v[0][r] = cmk(r0[r * NR], r0[N + r * NR]);
  for (int e = tid; e < N; e += NT) tw[e] = g[e];
  F::First::work(v, tw, -1, tid);
  F::First::write(v, buf, tid);
  F::rest(v, buf, tw, -1, tid);
  F::Last::write(v, buf, tid);
  __syncthreads();
  for (int e = tid; e < PN * 2 * Nh; e += NT) {
    const int rr = e / Nh, m = e - rr * Nh;
    W[((long long)b * N + y0 + rr) * Nh + m] = kol_unpack<N, PN>(buf, m, rr & 1, rr >> 1);
  }
}

// Forward y-transforms of a block's columns: A the padded grid's (threads from 0), C the closure's on the N-point grid
// (threads from tc0 on, beside them between the same barriers).  v: the first pass's inputs, then A's outputs;
// C's outputs are left in bufc in natural order, synchronized.
template <typename A, typename C, bool CLO, int NTA, int NTC>
__device__ __forceinline__ void kol_fwd_columns(cplx (&v)[1][A::R0], cplx (&vc)[1][C::R0], cplx* buf, cplx* bufc,
                                                const cplx* tw, const cplx* twc, int tid, int tc0) {
  static_assert(A::First::MB == 1 && A::First::full && C::First::MB == 1 && C::First::full, "one butterfly a thread");
  const int itc = tid - tc0;
  const bool aa = !CLO || tid < NTA, ac = CLO && itc >= 0;
  constexpr int MA = A::Mid::MB * A::R1, MC = C::Mid::MB * C::R1;
  cplx x[MA > MC ? MA : MC];
  auto& m = reinterpret_cast<cplx(&)[A::Mid::MB][A::R1]>(x);
  auto& mc = reinterpret_cast<cplx(&)[C::Mid::MB][C::R1]>(x);
  __syncthreads();
  if (aa) A::Mid::read(m, buf, tid);
  if (ac) C::Mid::read(mc, bufc, itc);
  __syncthreads();
  if (aa) {
    A::Mid::work(m, tw, -1, tid);
    A::Mid::write(m, buf, tid);
  }
  if (ac) {
    C::Mid::work(mc, twc, -1, itc);
    C::Mid::write(mc, bufc, itc);
  }
  __syncthreads();
  if (aa) {
    A::Last::read(v, buf, tid);
    A::Last::work(v, tw, -1, tid);
  }
  if (ac) C::Last::read(vc, bufc, itc);
  if (!CLO) return;
  __syncthreads();
  if (ac) {
    C::Last::work(vc, twc, -1, itc);
    C::Last::write(vc, bufc, itc);
  }
  __syncthreads();
}

// kol_cols_fwd in mode K_STEP.  Grid (column tiles, instances).
template <int G, bool CLO>
__global__ void __launch_bounds__(KolFft<G>::step_threads(CLO)) kol_cols_step_b(KolDev d, KolCol a) {
  using P = KolFft<G>;
  constexpr int N = P::N, Nh = P::Nh, R0 = P::R0, TC = P::TC, NR = G / R0, RN = BlockPlan<N>::R0, NTN = TC * N / RN;
  constexpr int NT = P::step_threads(CLO), TC0 = P::wave(P::NTC);
  using F = BlockFft<G, TC, P::NTC, 1, 4>;   // as kol_cols_inv_b, the other way
  using C = BlockFft<N, TC, NTN, 1, 1>;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  cplx* twc = buf + bf_size(TC * G);
  cplx* bufc = twc + N;
  const int b = blockIdx.y, tid = threadIdx.x, c0 = TC * kol_tile<TC>(blockIdx.x, gridDim.x);
  const int j = F::Last::bfly(tid), m = c0 + F::Last::seq(tid);
  const cplx* g = d.tw + d.twoff[d.pNg];
  cplx x[R0 > RN ? R0 : RN];   // a thread has one of the two transforms: the same registers
  auto& v = reinterpret_cast<cplx(&)[1][R0]>(x);
  auto& vc = reinterpret_cast<cplx(&)[1][RN]>(x);
  const bool act = !CLO || tid < P::NTC;
  if (act) {
    const cplx* Wc = a.W + ((long long)b * G + F::First::bfly(tid)) * Nh + c0 + F::First::seq(tid);
#pragma unroll
    for (int r = 0; r < R0; ++r) v[0][r] = Wc[(long long)r * NR * Nh];
  }
  if (CLO && tid >= TC0) {
    const int it = tid - TC0;
    const cplx* Wc = a.Wc + ((long long)b * N + C::First::bfly(it)) * Nh + c0 + C::First::seq(it);
#pragma unroll
    for (int r = 0; r < RN; ++r) vc[0][r] = Wc[(long long)r * (N / RN) * Nh];
  }
  for (int e = tid; e < G; e += NT) tw[e] = g[e];
  if (CLO)
    for (int e = tid; e < N; e += NT) twc[e] = d.tw[d.twoff[d.pN] + e];
  if (act) {
    F::First::work(v, tw, -1, tid);
    F::First::write(v, buf, tid);
  }
  if (CLO && tid >= TC0) {
    C::First::work(vc, twc, -1, tid - TC0);
    C::First::write(vc, bufc, tid - TC0);
  }
  // the previous states and F of this thread's modes: grid position p holds mode p (p < N / 2) or p - G + N
  // (p > G - N / 2); p = N / 2 stands for the Nyquist row, which is kept zero
  const long long st = (long long)d.B * Nh * N, io = ((long long)b * Nh + m) * N;
  constexpr bool early = NT <= 512;   // (beyond, there are no registers to keep them)
  StepIn in[R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    const int p = j + r * NR;
    if (r * NR > N / 2 && (r + 1) * NR - 1 <= G - N / 2) continue;
    if (early && act && (p <= N / 2 || p > G - N / 2)) in[r] = kol_step_load(a, st, io + (p <= N / 2 ? p : p - G + N));
  }
  kol_fwd_columns<F, C, CLO, P::NTC, NTN>(v, vc, buf, bufc, tw, twc, tid, TC0);
  if (!act) return;
  const double ng2 = 1.0 / ((double)G * G), n2 = 1.0 / ((double)N * N);
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    const int p = j + r * NR;
    if (r * NR > N / 2 && (r + 1) * NR - 1 <= G - N / 2) continue;
    if (p <= N / 2 || p > G - N / 2) {
      const int iy = p <= N / 2 ? p : p - G + N;
      const bool keep = p != N / 2;
      cplx f = czero();
      if (keep) {
        f = cscale(v[0][r], ng2);
        if (m == 0 && N > 8 && (iy == 4 || iy == N - 4)) f = cadd(f, cmk(-2.0, 0.0));   // -4 cos 4y
        if (CLO) f = cadd(f, cscale(bufc[bf_pad(iy * TC + (m - c0))], n2));
      }
      const double ky = kol_ky(iy, N), lin = d.nu * ((double)m * m + ky * ky) + d.drag;
      kol_step_entry(d, a, b, m, iy, keep, f, early ? in[r] : kol_step_load(a, st, io + iy), lin, st, io + iy);
    }
  }
}

// kol_cols_fwd in mode K_ADJ: the products of a column's four fields on lanes 4 f + (0 .. 3) of a row of 16, so their
// sum is two lane exchanges, after which the lanes of field f finish the positions j + r G / R0 with r = f
// (mod 4).  12.0 -> 6.1 us at N = 64, 16 instances, with the closure.  Grid (column tiles, instances).
template <int G, bool CLO>
__global__ void __launch_bounds__(KolFft<G>::adj_threads(CLO)) kol_cols_adj_b(KolDev d, KolCol a) {
  using P = KolFft<G>;
  constexpr int N = P::N, Nh = P::Nh, R0 = P::R0, TA = P::TA, TC = 4 * TA, NR = G / R0, RN = BlockPlan<N>::R0, NTN = TA * N / RN;
  constexpr int NT = P::adj_threads(CLO), TC0 = P::wave(P::NTA), RQ = (R0 + 3) / 4;
  using F = BlockFft<G, TC, P::NTA, 1, 4>;
  using C = BlockFft<N, TA, NTN, 1, 1>;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  cplx* twc = buf + bf_size(TC * G);
  cplx* bufc = twc + N;
  const int b = blockIdx.y, tid = threadIdx.x, c0 = TA * blockIdx.x;
  const cplx* g = d.tw + d.twoff[d.pNg];
  cplx x[R0 > RN ? R0 : RN];   // a thread has one of the two transforms: the same registers
  auto& v = reinterpret_cast<cplx(&)[1][R0]>(x);
  auto& vc = reinterpret_cast<cplx(&)[1][RN]>(x);
  const bool act = !CLO || tid < P::NTA;
  if (act) {   // sequence 4 column + field
    const int s = F::First::seq(tid);
    const cplx* Wc = a.W + (((long long)b * 4 + (s & 3)) * G + F::First::bfly(tid)) * Nh + c0 + (s >> 2);
#pragma unroll
    for (int r = 0; r < R0; ++r) v[0][r] = Wc[(long long)r * NR * Nh];
  }
  if (CLO && tid >= TC0) {
    const int it = tid - TC0;
    const cplx* Wc = a.Wc + ((long long)b * N + C::First::bfly(it)) * Nh + c0 + C::First::seq(it);
#pragma unroll
    for (int r = 0; r < RN; ++r) vc[0][r] = Wc[(long long)r * (N / RN) * Nh];
  }
  for (int e = tid; e < G; e += NT) tw[e] = g[e];
  if (CLO)
    for (int e = tid; e < N; e += NT) twc[e] = d.tw[d.twoff[d.pN] + e];
  if (act) {
    F::First::work(v, tw, -1, tid);
    F::First::write(v, buf, tid);
  }
  if (CLO && tid >= TC0) {
    C::First::work(vc, twc, -1, tid - TC0);
    C::First::write(vc, bufc, tid - TC0);
  }
  // what this thread's modes need from memory, positions as in kol_cols_step_b
  const int j = F::Last::bfly(tid), f = F::Last::seq(tid) & 3, m = c0 + (F::Last::seq(tid) >> 2), k = a.n - 1;
  const long long st = (long long)d.B * Nh * N, io = ((long long)b * Nh + m) * N;
  const cplx* H = a.H + hidx(a, k, st);
  const cplx* T = (a.targ && k >= 1) ? a.targ + (long long)(k - 1) * st : nullptr;
  cplx ln[RQ], yn[RQ], dh[RQ], dm[RQ];
#pragma unroll
  for (int i = 0; i < RQ; ++i) {
    ln[i] = yn[i] = dh[i] = dm[i] = czero();
    const int r = f + 4 * i, p = j + r * NR;
    if (!act || r >= R0 || !(p <= N / 2 || p > G - N / 2)) continue;
    const int iy = p <= N / 2 ? p : p - G + N;
    ln[i] = a.Ln[io + iy];
    yn[i] = a.Yn[io + iy];
    if (T) {
      dh[i] = csub(H[io + iy], T[io + iy]);
      if (m == 0) dm[i] = csub(H[io + (N - iy) % N], T[io + (N - iy) % N]);
    }
  }
  kol_fwd_columns<F, C, CLO, P::NTA, NTN>(v, vc, buf, bufc, tw, twc, tid, TC0);
  if (!act) return;
  // the fields' conjugate factors (u: -i ky/|k|^2, v: i kx/|k|^2, omega_x: -i kx, omega_y: -i ky) and their sum
  const double kx = m, wm = (m == 0) ? 1.0 : 2.0;
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    if (r * NR > N / 2 && (r + 1) * NR - 1 <= G - N / 2) continue;
    const int p = j + r * NR;
    const double ky = (p < N / 2) ? p : p - G, k2 = kx * kx + ky * ky;
    const double ik2 = (k2 > 0.0) ? 1.0 / k2 : 0.0;
    const double q = wm * (f == 0 ? ky * ik2 : f == 1 ? -kx * ik2 : f == 2 ? kx : ky);
    double sx = q * v[0][r].y, sy = -q * v[0][r].x;
    sx += dpp_d<0x128>(sx);
    sy += dpp_d<0x128>(sy);
    v[0][r] = cmk(sx + dpp_d<0x124>(sx), sy + dpp_d<0x124>(sy));
  }
  const SbdfC q = sbdf_c(max(k, 1), d.dt), qn = sbdf_c(k + 1, d.dt);
#pragma unroll
  for (int i = 0; i < RQ; ++i) {
    const int r = f + 4 * i, p = j + r * NR;
    cplx xb = czero();
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * i + e < R0) {
        xb.x = (f == e) ? v[0][4 * i + e].x : xb.x;
        xb.y = (f == e) ? v[0][4 * i + e].y : xb.y;
      }
    if (r >= R0 || !(p <= N / 2 || p > G - N / 2)) continue;
    const int iy = p <= N / 2 ? p : p - G + N;
    const bool keep = p != N / 2;
    if (!keep) xb = czero();
    if (CLO && keep) xb = cadd(xb, cscale(bufc[bf_pad(iy * TA + (m - c0))], wm));
    xb = csub(xb, ln[i]);
    if (T && keep) {
      // d/dX_k of (1/nsteps) mean over the N x N grid of (omega_k - target_k)^2
      const cplx e1 = (m == 0) ? cmk(0.5 * (dh[i].x + dm[i].x), 0.5 * (dh[i].y - dm[i].y)) : dh[i];
      xb = cadd(xb, cscale(e1, 2.0 * wm / a.nsteps));
    }
    if (k == 0) {
      a.out[io + iy] = xb;
      continue;
    }
    cplx y = czero(), gk = czero(), l = czero();
    if (keep) {   // (k + 1 <= nsteps: Yn holds the next step's)
      const double ky = kol_ky(iy, N), lin = d.nu * (kx * kx + ky * ky) + d.drag;
      y = cscale(xb, 1.0 / (q.a0 + lin));
      gk = cadd(cscale(y, q.c1), cscale(yn[i], qn.c2));
      l = cadd(cscale(y, q.a1), cscale(yn[i], qn.a2));
    }
    a.Yn[io + iy] = y;
    a.Ln[io + iy] = l;
    a.Gk[io + iy] = gk;
  }
}

// rollout loss per instance: (1/nsteps) sum_k sum_modes w |canon(X_k - T_k)|^2 (= mean over the
// N x N grid of the squared difference).  One block per step and instance writes that step's sum
// (the states and targets are read once, at the memory's rate); kol_loss_sum adds the steps in a
// fixed order.  One block per instance for the whole run: 884 us, now 33 + 5 us (16 runs of
// 64 x 64, 200 steps; 420 MB read).  Beyond kLossBlocks steps a block takes several: a launch of one block per
// step is refused from 2^24 steps on (2^32 threads), which small grids have the memory for.
constexpr int kLossBlocks = 4096;
__global__ void __launch_bounds__(NTK) kol_loss(KolDev d, const cplx* H, const cplx* T, int nsteps, double* part) {
  __shared__ double red[NTK];
  const int b = blockIdx.y, N = d.N, Nh = d.Nh, tid = threadIdx.x;
  const long long st = (long long)d.B * Nh * N, io = (long long)b * Nh * N;
  for (int k = blockIdx.x; k < nsteps; k += gridDim.x) {   // (nsteps + gridDim.x: below 2^31 for every history that fits)
    const cplx* Hk = H + (k + 1LL) * st + io;
    const cplx* Tk = T + (long long)k * st + io;
    double s = 0.0;
    for (int e = tid; e < Nh * N; e += NTK) {
      const int m = e / N, iy = e - m * N;
      if (iy == N / 2) continue;
      cplx c = csub(Hk[e], Tk[e]);
      if (m == 0) {
        const int sm = (N - iy) % N;
        const cplx c2 = csub(Hk[sm], Tk[sm]);
        c = cmk(0.5 * (c.x + c2.x), 0.5 * (c.y - c2.y));
      }
      s += ((m == 0) ? 1.0 : 2.0) * (c.x * c.x + c.y * c.y);
    }
    red[tid] = s;
    __syncthreads();
    for (int w = NTK / 2; w > 0; w >>= 1) {
      if (tid < w) red[tid] += red[tid + w];
      __syncthreads();
    }
    if (tid == 0) part[(long long)b * nsteps + k] = red[0];
    __syncthreads();
  }
}
// J[b] = (1/nsteps) sum of the steps' sums, one block per instance
__global__ void __launch_bounds__(NTK) kol_loss_sum(const double* part, int nsteps, double* J) {
  __shared__ double red[NTK];
  const int tid = threadIdx.x;
  double s = 0.0;
  for (int k = tid; k < nsteps; k += NTK) s += part[(long long)blockIdx.x * nsteps + k];
  red[tid] = s;
  __syncthreads();
  for (int w = NTK / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] += red[tid + w];
    __syncthreads();
  }
  if (tid == 0) J[blockIdx.x] = red[0] / nsteps;
}

// Adam update of the closure parameters (theta, first and second moments in FP64)
__global__ void kol_adam(int n, double* th, const double* g, double* m1, double* m2, double lr, double b1, double b2,
                         double eps, int t) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  m1[i] = b1 * m1[i] + (1.0 - b1) * g[i];
  m2[i] = b2 * m2[i] + (1.0 - b2) * g[i] * g[i];
  const double mh = m1[i] / (1.0 - pow(b1, t)), vh = m2[i] / (1.0 - pow(b2, t));
  th[i] -= lr * mh / (sqrt(vh) + eps);
}

// ---------------------------------------------------------------------------- host
class KolProblem : public ProblemImpl {
 public:
  KolProblem(int batch, int N, double Re, double drag, double dt, int max_steps, int closure, int keep_history,
             hipStream_t s) {
    stream = s;
    SPS_REQUIRE(batch >= 1 && N >= 8 && N % 4 == 0 && N <= 1024, "need batch >= 1 and N a multiple of 4 in [8, 1024]");
    SPS_REQUIRE(Re > 0 && drag >= 0 && dt > 0 && max_steps >= 1, "bad Re / drag / dt / max_steps");
    SPS_REQUIRE(!closure || N % 32 == 0, "the closure needs N a multiple of 32");
    B_ = batch;
    N_ = N;
    Nh_ = N / 2;
    Ng_ = 3 * N / 2;
    max_steps_ = max_steps;
    closure_ = closure;
    hring_ = keep_history ? 0 : 3;
    FftPlan pn{}, png{};
    SPS_REQUIRE(fft_plan(N, &pn) && fft_plan(Ng_, &png), "N and 3N/2 must factor into 2 and 3");
    std::vector<FftPlan> plans = {pn, png};
    std::vector<double2> tw = twiddles(N);
    const auto tg = twiddles(Ng_);
    std::vector<int> off = {0, (int)tw.size()};
    tw.insert(tw.end(), tg.begin(), tg.end());
    d_.B = B_;
    d_.N = N;
    d_.Nh = Nh_;
    d_.Ng = Ng_;
    d_.nu = 1.0 / Re;
    d_.drag = drag;
    d_.dt = dt;
    d_.pN = 0;
    d_.pNg = 1;
    d_.plans = arena_.upload(plans, stream);
    d_.tw = arena_.upload(tw, stream);
    d_.twoff = arena_.upload(off, stream);
    st_ = (long long)B_ * Nh_ * N_;
    err_ = arena_.alloc<int>(1);
    SPS_HIP(hipMemsetAsync(err_, 0, sizeof(int), stream));
    const int nh = keep_history ? max_steps + 1 : 3;
    H_ = arena_.alloc<cplx>((size_t)nh * st_);
    if (keep_history) lpart_ = arena_.alloc<double>((size_t)max_steps * B_);
    Fr_ = arena_.alloc<cplx>(2 * st_);
    Yn_ = arena_.alloc<cplx>(st_);
    Ln_ = arena_.alloc<cplx>(st_);
    Gk_ = arena_.alloc<cplx>(st_);
    Xw_ = arena_.alloc<cplx>(st_);
    Z4_ = arena_.alloc<cplx>((size_t)B_ * 4 * Nh_ * Ng_);
    Zg_ = arena_.alloc<cplx>((size_t)B_ * Nh_ * Ng_);
    W_ = arena_.alloc<cplx>((size_t)B_ * 4 * Nh_ * Ng_);
    if (closure_) {
      net_.reset(new Cnn(B_, N_, N_, stream));
      Zc_ = arena_.alloc<cplx>(st_);
      Zgc_ = arena_.alloc<cplx>(st_);
      Wc_ = arena_.alloc<cplx>(st_);
      og_ = arena_.alloc<double>((size_t)B_ * N_ * N_);
      yg_ = arena_.alloc<double>((size_t)B_ * N_ * N_);
      xg_ = arena_.alloc<double>((size_t)B_ * N_ * N_);
      theta_ = arena_.alloc<double>(Cnn::nparam());
      SPS_HIP(hipMemsetAsync(theta_, 0, sizeof(double) * Cnn::nparam(), stream));
      net_->set_params(theta_);
    }
    // tiles: the widest (up to 8 columns) whose LDS stays within kLdsBudget, so that two
    // blocks fit on a CU; row buffers sized for the widest row mode this problem runs
    nwmax_ = keep_history ? 4 : 1;
    tc_ig_ = pick_tile([&](int tc) { return inv_lds(Ng_, tc); });
    tc_in_ = pick_tile([&](int tc) { return inv_lds(N_, tc); });
    tc_f_ = pick_tile([&](int tc) { return fwd_lds(tc); });
    rcap_ = fpad_size((keep_history ? 5 : 4) * Ng_);
    const size_t rl = sizeof(cplx) * (Ng_ + 2 * (size_t)rcap_);
    const size_t il = std::max(inv_lds(Ng_, tc_ig_), inv_lds(N_, tc_in_));
    SPS_REQUIRE(rl <= kLdsMax && il <= kLdsMax && fwd_lds(tc_f_) <= kLdsMax, "size too large for the Kolmogorov kernels");
    for (const void* k : {(const void*)kol_cols_inv, (const void*)kol_rows<256>, (const void*)kol_rows<512>,
                          (const void*)kol_rows_adv2<512>, (const void*)kol_cols_fwd})
      SPS_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
    block_ = with_block_fft([&](auto g) {
      constexpr int G = decltype(g)::value;
      using P = KolFft<G>;
      const auto lds = [](const void* k, size_t n) { SPS_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)n)); };
      lds((const void*)kol_cols_inv_b<G, false>, P::lds_cols);
      lds((const void*)kol_cols_inv_b<G, true>, P::lds_cols);
      lds((const void*)kol_rows_adv_b<G, false>, P::lds_rows);
      lds((const void*)kol_rows_adv_b<G, true>, P::lds_rows);
      lds((const void*)kol_rows_vjp_b<G, false>, P::lds_vjp);
      lds((const void*)kol_rows_vjp_b<G, true>, P::lds_vjp);
      lds((const void*)kol_rows_fwd_b<G>, P::lds_n);
      lds((const void*)kol_cols_step_b<G, false>, P::lds_step(false));
      lds((const void*)kol_cols_step_b<G, true>, P::lds_step(true));
      lds((const void*)kol_cols_adj_b<G, false>, P::lds_adj(false));
      lds((const void*)kol_cols_adj_b<G, true>, P::lds_adj(true));
    });
    SPS_HIP(hipStreamSynchronize(stream));
  }

  long long state_size() const override { return 2 * st_; }
  // a new step for the following runs: the SBDF2 coefficients take it (diagonal implicit
  // operator); drops the recorded run
  void set_dt(double dt) override {
    SPS_REQUIRE(std::isfinite(dt) && dt > 0.0, "dt must be positive");
    d_.dt = dt;
    tape_ = -1;
  }
  void factor() override {}

  void set_params(const double* theta) {
    SPS_REQUIRE(closure_, "this problem has no closure");
    SPS_HIP(hipMemcpyAsync(theta_, theta, sizeof(double) * Cnn::nparam(), hipMemcpyDeviceToDevice, stream));
    net_->set_params(theta_);
  }

  // forward sweep from X0 (state layout); XN (nullable); snapshots of the run truncated to
  // Nc x Nc modes every `every` steps (nullable)
  void forward(const cplx* X0, int nsteps, cplx* XN, cplx* snap, int every, int Nc) {
    SPS_REQUIRE(X0 && nsteps >= 1, "forward: null state or nsteps < 1");
    SPS_REQUIRE(hring_ || nsteps <= max_steps_, "forward: nsteps exceeds the history the problem was built for");
    SPS_REQUIRE(!snap || (every >= 1 && Nc >= 4 && Nc % 2 == 0 && Nc <= N_), "forward: bad snapshot arguments");
    if (!snap) every = 1;
    SPS_HIP(hipMemcpyAsync(H_, X0, sizeof(cplx) * st_, hipMemcpyDeviceToDevice, stream));
    for (int n = 1; n <= nsteps; ++n) {
      const cplx* Xp = H_ + hslot(n - 1) * st_;
      eval_products(Xp);
      KolCol a = col_args(K_STEP, n, nsteps);
      a.out = XN;
      a.snap = snap;
      a.snap_every = every;
      a.Nc = Nc;
      launch_cols(a);
    }
    tape_ = nsteps;
  }

  // reverse sweep: dJ/dX_0 of the rollout loss against targets (nullable) plus an external
  // dJ/dX_N (nullable); closure-parameter gradient added to th_bar (nullable)
  void reverse(const cplx* targets, const cplx* xbN, int nsteps, cplx* xb0, double* th_bar) {
    SPS_REQUIRE(hring_ == 0, "the reverse sweep needs the full history");
    SPS_REQUIRE(tape_ == nsteps, "reverse: nsteps does not match the recorded forward run");
    KolCol a = col_args(K_ADJ_INIT, nsteps, nsteps);
    a.targ = targets;
    a.xin = xbN;
    a.out = xb0;
    launch_cols(a);
    // the closure-parameter cotangent of every step is summed in the network's accumulators
    // and added to th_bar once at the end of the sweep
    const bool acc = closure_ && th_bar;
    if (acc) net_->grad_reset();
    for (int n = nsteps; n >= 1; --n) {
      const cplx* Xp = H_ + (long long)(n - 1) * st_;
      eval_vjp(Xp, Gk_, acc ? ACC_THETA : NO_THETA, nullptr);
      KolCol c = col_args(K_ADJ, n, nsteps);
      c.targ = targets;
      c.out = xb0;
      launch_cols(c);
    }
    if (acc) net_->grad_flush(th_bar);
  }

  // forward run from X0, the rollout loss J[b] against targets and its gradients: dJdX0
  // (state layout, nullable) and dJdtheta = sum over instances of dJ[b]/dtheta (nullable;
  // needs the closure)
  void rollout(const cplx* X0, const cplx* targets, int nsteps, cplx* XN, double* J, cplx* dJdX0, double* dJdtheta) {
    SPS_REQUIRE(targets, "rollout: targets are required");
    SPS_REQUIRE(!dJdtheta || closure_, "rollout: dJdtheta needs the closure");
    SPS_REQUIRE(!(dJdX0 || dJdtheta) || hring_ == 0, "rollout gradients need a problem built with keep_history");
    forward(X0, nsteps, XN, nullptr, 1, 0);
    if (J) loss(targets, nsteps, J);
    if (dJdX0 || dJdtheta) {
      if (dJdtheta) SPS_HIP(hipMemsetAsync(dJdtheta, 0, sizeof(double) * Cnn::nparam(), stream));
      reverse(targets, nullptr, nsteps, dJdX0 ? dJdX0 : Xw_, dJdtheta);
    }
  }

  void loss(const cplx* targets, int nsteps, double* J) {
    SPS_REQUIRE(hring_ == 0 && tape_ == nsteps, "loss: needs the full history of the last forward run");
    hipLaunchKernelGGL(kol_loss, dim3(std::min(nsteps, kLossBlocks), B_), dim3(NTK), 0, stream, d_, H_, targets, nsteps,
                       lpart_);
    SPS_CHECK_LAUNCH();
    hipLaunchKernelGGL(kol_loss_sum, dim3(B_), dim3(NTK), 0, stream, lpart_, nsteps, J);
    SPS_CHECK_LAUNCH();
  }

  // Adam update of the caller's parameter vector theta, which then becomes the problem's
  void adam(double* theta, const double* grad, double* m1, double* m2, double lr, int t) {
    SPS_REQUIRE(closure_, "this problem has no closure");
    const int n = Cnn::nparam();
    hipLaunchKernelGGL(kol_adam, dim3((n + 255) / 256), dim3(256), 0, stream, n, theta, grad, m1, m2, lr, 0.9, 0.999,
                       1e-8, t);
    SPS_CHECK_LAUNCH();
    set_params(theta);
  }

  // ProblemImpl
  void step(double* X, int nsteps) override {
    SPS_REQUIRE(X && nsteps >= 1 && nsteps <= max_steps_, "bad step arguments");
    forward(reinterpret_cast<const cplx*>(X), nsteps, reinterpret_cast<cplx*>(X), nullptr, 1, 0);
  }
  void adjoint_step(double* Xbar, int nsteps) override {
    SPS_REQUIRE(Xbar, "Xbar is null");
    if (tape_ != nsteps) throw Error(SPS_E_STATE, "adjoint_step: nsteps does not match the recorded forward run");
    SPS_HIP(hipMemcpyAsync(Xw_, Xbar, sizeof(cplx) * st_, hipMemcpyDeviceToDevice, stream));
    reverse(nullptr, Xw_, nsteps, reinterpret_cast<cplx*>(Xbar), nullptr);
  }
  void cost(const double*, double*, double*) override {
    throw Error(SPS_E_UNSUPPORTED, "the Kolmogorov problem's objective is the rollout loss");
  }
  void gradient(const double*, int, const double*, double*, double*, double*, double*) override {
    throw Error(SPS_E_UNSUPPORTED, "use the rollout call of the Kolmogorov problem");
  }
  void initial_state(const double*, double*) override {
    throw Error(SPS_E_UNSUPPORTED, "Kolmogorov states are given as coefficients");
  }
  void initial_state_adjoint(const double*, double*) override {
    throw Error(SPS_E_UNSUPPORTED, "Kolmogorov states are given as coefficients");
  }
  void eval_F(const double* X, double* F) override {
    eval_products(reinterpret_cast<const cplx*>(X));
    KolCol a = col_args(K_EVALF, 0, 0);
    a.out = reinterpret_cast<cplx*>(F);
    launch_cols(a);
  }
  void eval_F_vjp(const double* X, const double* Fbar, double* Xbar) override {
    eval_vjp(reinterpret_cast<const cplx*>(X), reinterpret_cast<const cplx*>(Fbar), NO_THETA, nullptr);
    KolCol a = col_args(K_VJP, 0, 0);
    a.out = reinterpret_cast<cplx*>(Xbar);
    launch_cols(a);
  }
  void param_vjp(const double* X, const double* Fbar, double* th_bar) {
    SPS_REQUIRE(closure_, "this problem has no closure");
    eval_vjp(reinterpret_cast<const cplx*>(X), reinterpret_cast<const cplx*>(Fbar), ADD_THETA, th_bar);
  }
  void solve(const double*, double*, int) override {
    throw Error(SPS_E_UNSUPPORTED, "the Kolmogorov solve is internal to its steps");
  }
  void timer_enable(int, bool) override {}
  void timer_read(long long* l, double* ms) override {
    *l = 0;
    *ms = 0;
  }
  int device_error() override {
    int h = 0;
    SPS_HIP(hipMemcpyAsync(&h, err_, sizeof(int), hipMemcpyDeviceToHost, stream));
    SPS_HIP(hipStreamSynchronize(stream));
    if (h) SPS_HIP(hipMemsetAsync(err_, 0, sizeof(int), stream));
    return h;
  }

 private:
  long long hslot(int k) const { return hring_ ? k % hring_ : k; }
  size_t inv_lds(int G, int tc) const { return sizeof(cplx) * (G + 2 * (size_t)fpad_size(tc * G)); }
  int wcap(int tc) const { return fpad_size(nwmax_ * tc * Ng_); }
  size_t fwd_lds(int tc) const {
    return sizeof(cplx) * (Ng_ + N_ + 2 * (size_t)wcap(tc) + (closure_ ? 2 * (size_t)fpad_size(tc * N_) : 0));
  }
  template <typename F>
  int pick_tile(F lds) const {
    int tc = 8;
    while (tc > 1 && lds(tc) > kLdsBudget) --tc;
    return tc;
  }
  KolCol col_args(int mode, int n, int nsteps) {
    KolCol a{};
    a.mode = mode;
    a.n = n;
    a.nsteps = nsteps;
    a.closure = closure_;
    a.W = W_;
    a.Wc = Wc_;
    a.H = H_;
    a.hring = hring_;
    a.Fr = Fr_;
    a.Yn = Yn_;
    a.Ln = Ln_;
    a.Gk = Gk_;
    a.err = err_;
    return a;
  }
  // fn(the padded length as a type) if the kernels of a known length are built for it.  The others take about twice as
  // long: 16 forward steps of one instance 554 us at N = 144, 270 at 128 and 291 at 192; 332 at N = 48, 191 at 64.
  template <typename Fn>
  bool with_block_fft(Fn fn) const {
    switch (Ng_) {
      case 48: fn(std::integral_constant<int, 48>()); return true;
      case 96: fn(std::integral_constant<int, 96>()); return true;
      case 144: fn(std::integral_constant<int, 144>()); return true;
      case 192: fn(std::integral_constant<int, 192>()); return true;
      case 288: fn(std::integral_constant<int, 288>()); return true;
      case 384: fn(std::integral_constant<int, 384>()); return true;
      case 576: fn(std::integral_constant<int, 576>()); return true;
      case 768: fn(std::integral_constant<int, 768>()); return true;
      default: return false;
    }
  }
  template <int G, bool CLO>
  void launch_cols_b(const KolCol& a) {
    using P = KolFft<G>;
    if (a.mode == K_STEP)
      hipLaunchKernelGGL((kol_cols_step_b<G, CLO>), dim3(P::Nh / P::TC, B_), dim3(P::step_threads(CLO)), P::lds_step(CLO), stream,
                         d_, a);
    else
      hipLaunchKernelGGL((kol_cols_adj_b<G, CLO>), dim3(P::Nh / P::TA, B_), dim3(P::adj_threads(CLO)), P::lds_adj(CLO), stream, d_,
                         a);
  }
  void launch_cols(const KolCol& a) {
    if (block_ && (a.mode == K_STEP || a.mode == K_ADJ)) {
      with_block_fft([&](auto g) {
        constexpr int G = decltype(g)::value;
        if (a.closure) launch_cols_b<G, true>(a);
        else launch_cols_b<G, false>(a);
      });
      SPS_CHECK_LAUNCH();
      return;
    }
    hipLaunchKernelGGL(kol_cols_fwd, dim3((Nh_ + tc_f_ - 1) / tc_f_, B_), dim3(NTK), fwd_lds(tc_f_), stream, d_, a,
                       tc_f_, wcap(tc_f_));
    SPS_CHECK_LAUNCH();
  }
  void cols_inv(const cplx* X, int set, int G, int plan, cplx* Z) {
    const int tc = (G == Ng_) ? tc_ig_ : tc_in_;
    const int nf = (set == FS_PRIMAL4) ? 4 : 1;
    hipLaunchKernelGGL(kol_cols_inv, dim3((Nh_ + tc - 1) / tc, nf, B_), dim3(NTK), inv_lds(G, tc), stream, d_, X,
                       set, G, plan, tc, Z);
    SPS_CHECK_LAUNCH();
  }
  void rows(int mode, int G, int plan, const cplx* Z4, const cplx* Zg, double* grid, const double* gin, cplx* W,
            double wscale, double gscale) {
    if (mode == R_ADV && G >= 384) {
      const size_t l2 = sizeof(cplx) * (G + 2 * (size_t)fpad_size(2 * G) + fpad_size(G));
      hipLaunchKernelGGL(kol_rows_adv2<512>, dim3(G / 2, B_), dim3(512), l2, stream, d_, G, plan, Z4, W);
      SPS_CHECK_LAUNCH();
      return;
    }
    // rows of 384 points or more: 512 threads, so that a CU holding one block (LDS) still has
    // eight waves
    const size_t lds = sizeof(cplx) * (G + 2 * (size_t)rcap_);
    if (G >= 384)
      hipLaunchKernelGGL(kol_rows<512>, dim3(G / 2, B_), dim3(512), lds, stream, d_, mode, G, plan, rcap_, Z4, Zg, grid,
                         gin, W, wscale, gscale);
    else
      hipLaunchKernelGGL(kol_rows<256>, dim3(G / 2, B_), dim3(256), lds, stream, d_, mode, G, plan, rcap_, Z4, Zg, grid,
                         gin, W, wscale, gscale);
    SPS_CHECK_LAUNCH();
  }
  // The column inverses and row passes of F at X, or of its VJP with the cotangent Fb, up to the closure's network,
  // in two launches (padded lengths with a plan).
  void block_products(const cplx* X, const cplx* Fb) {
    with_block_fft([&](auto g) {
      if (closure_) block_products_g<decltype(g)::value, true>(X, Fb);
      else block_products_g<decltype(g)::value, false>(X, Fb);
    });
  }
  template <int G, bool CLO>
  void block_products_g(const cplx* X, const cplx* Fb) {
    using P = KolFft<G>;
    const int grids = CLO ? (Fb ? 2 : 1) : 0, fields = 4 + (Fb ? 1 : 0) + grids;
    hipLaunchKernelGGL((kol_cols_inv_b<G, CLO>), dim3(P::Nh / P::TC, fields, B_), dim3(P::NTC), P::lds_cols, stream, d_,
                       KolInv{X, Fb, Z4_, Zg_, Zc_, Zgc_});
    SPS_CHECK_LAUNCH();
    const dim3 rows(G / 2 / P::PAIRS + grids * (P::N / 2 / P::PN), B_);
    const KolGrids cg{Zc_, Zgc_, og_, yg_};
    if (Fb)
      hipLaunchKernelGGL((kol_rows_vjp_b<G, CLO>), rows, dim3(P::NTR), P::lds_vjp, stream, d_, Z4_, Zg_, W_, cg);
    else
      hipLaunchKernelGGL((kol_rows_adv_b<G, CLO>), rows, dim3(P::NTR), P::lds_rows, stream, d_, Z4_, W_, cg);
    SPS_CHECK_LAUNCH();
  }
  // x-spectra of the network's output on the grid (Wc)
  void closure_spectra(const double* grid) {
    const bool done = with_block_fft([&](auto g) {
      using P = KolFft<decltype(g)::value>;
      hipLaunchKernelGGL(kol_rows_fwd_b<decltype(g)::value>, dim3(P::N / 2 / P::PN, B_), dim3(P::NTN), P::lds_n, stream, d_, grid, Wc_);
      SPS_CHECK_LAUNCH();
    });
    if (!done) rows(R_FWD_GRID, N_, d_.pN, nullptr, nullptr, nullptr, grid, Wc_, 1.0, 1.0);
  }
  // x-spectra of the products of F at X (W) and of the closure output (Wc)
  void eval_products(const cplx* X) {
    if (block_) {
      block_products(X, nullptr);
    } else {
      general_products(X);
    }
    if (closure_) {
      net_->forward(og_, yg_, 1.0, false);
      closure_spectra(yg_);
    }
  }
  void general_products(const cplx* X) {
    cols_inv(X, FS_PRIMAL4, Ng_, d_.pNg, Z4_);
    rows(R_ADV, Ng_, d_.pNg, Z4_, nullptr, nullptr, nullptr, W_, 1.0, 1.0);
    if (closure_) {
      cols_inv(X, FS_ONE, N_, d_.pN, Zc_);
      rows(R_GRID, N_, d_.pN, Zc_, nullptr, og_, nullptr, nullptr, 1.0, 1.0);
    }
  }
  // x-spectra of the VJP of F at X with cotangent G (W: 4 fields; Wc).  The closure's parameter
  // cotangent: dropped (NO_THETA), added to th_bar (ADD_THETA) or to the network's accumulators
  // (ACC_THETA).
  enum ThetaMode { NO_THETA, ADD_THETA, ACC_THETA };
  void eval_vjp(const cplx* X, const cplx* G, ThetaMode tm, double* th_bar) {
    SPS_REQUIRE(nwmax_ == 4, "VJPs need a problem built with keep_history");
    if (block_) {
      block_products(X, G);
    } else {
      general_vjp_products(X, G);
    }
    if (closure_) {
      if (tm == ACC_THETA)
        net_->vjp_accumulate(og_, yg_, xg_, 1.0, false);
      else
        net_->vjp(og_, yg_, xg_, 1.0, false, tm == ADD_THETA ? th_bar : nullptr);
      closure_spectra(xg_);
    }
  }
  void general_vjp_products(const cplx* X, const cplx* G) {
    cols_inv(X, FS_PRIMAL4, Ng_, d_.pNg, Z4_);
    cols_inv(G, FS_ONE, Ng_, d_.pNg, Zg_);
    rows(R_ADV_VJP, Ng_, d_.pNg, Z4_, Zg_, nullptr, nullptr, W_, 1.0, 1.0);
    if (closure_) {
      cols_inv(X, FS_ONE, N_, d_.pN, Zc_);
      rows(R_GRID, N_, d_.pN, Zc_, nullptr, og_, nullptr, nullptr, 1.0, 1.0);
      cols_inv(G, FS_ONE, N_, d_.pN, Zgc_);
      rows(R_GRID, N_, d_.pN, Zgc_, nullptr, yg_, nullptr, nullptr, 0.5, 1.0 / ((double)N_ * N_));
    }
  }

  int B_, N_, Nh_, Ng_, max_steps_, closure_, hring_, nwmax_ = 4, tc_ig_ = 1, tc_in_ = 1, tc_f_ = 1, rcap_ = 0;
  int tape_ = -1;
  bool block_ = false;   // the padded length has a block_fft.h plan
  long long st_ = 0;
  KolDev d_{};
  DevArena arena_;
  std::unique_ptr<Cnn> net_;
  int* err_ = nullptr;
  cplx *H_, *Fr_, *Yn_, *Ln_, *Gk_, *Xw_, *Z4_, *Zg_, *W_, *Zc_ = nullptr, *Zgc_ = nullptr, *Wc_ = nullptr;
  double *og_ = nullptr, *yg_ = nullptr, *xg_ = nullptr, *theta_ = nullptr;
  double* lpart_ = nullptr;   // [B][steps] sums of the rollout loss
};

}  // namespace

ProblemImpl* make_kolmo(int batch, int N, double Re, double drag, double dt, int max_steps, int closure,
                        int keep_history, hipStream_t s) {
  return new KolProblem(batch, N, Re, drag, dt, max_steps, closure, keep_history, s);
}
void kolmo_set_params(ProblemImpl* p, const double* theta) {
  auto* k = dynamic_cast<KolProblem*>(p);
  if (!k) throw Error(SPS_E_ARG, "not a Kolmogorov problem");
  k->set_params(theta);
}
void kolmo_forward(ProblemImpl* p, const double* X0, int nsteps, double* XN, double* snap, int every, int Nc) {
  auto* k = dynamic_cast<KolProblem*>(p);
  if (!k) throw Error(SPS_E_ARG, "not a Kolmogorov problem");
  k->forward(reinterpret_cast<const cplx*>(X0), nsteps, reinterpret_cast<cplx*>(XN), reinterpret_cast<cplx*>(snap),
             every, Nc);
}
void kolmo_rollout(ProblemImpl* p, const double* X0, const double* targets, int nsteps, double* XN, double* J,
                   double* dJdX0, double* dJdtheta) {
  auto* k = dynamic_cast<KolProblem*>(p);
  if (!k) throw Error(SPS_E_ARG, "not a Kolmogorov problem");
  k->rollout(reinterpret_cast<const cplx*>(X0), reinterpret_cast<const cplx*>(targets), nsteps,
             reinterpret_cast<cplx*>(XN), J, reinterpret_cast<cplx*>(dJdX0), dJdtheta);
}
void kolmo_param_vjp(ProblemImpl* p, const double* X, const double* Fbar, double* th_bar) {
  auto* k = dynamic_cast<KolProblem*>(p);
  if (!k) throw Error(SPS_E_ARG, "not a Kolmogorov problem");
  k->param_vjp(X, Fbar, th_bar);
}
void kolmo_adam(ProblemImpl* p, double* theta, const double* grad, double* m1, double* m2, double lr, int t) {
  auto* k = dynamic_cast<KolProblem*>(p);
  if (!k) throw Error(SPS_E_ARG, "not a Kolmogorov problem");
  k->adam(theta, grad, m1, m2, lr, t);
}

}  // namespace sps
