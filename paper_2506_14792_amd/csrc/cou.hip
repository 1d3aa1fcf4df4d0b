// 3D plane Couette flow: the (x, z) plane transforms and products of the explicit term, and their
// vector-Jacobian product.  The per-mode Stokes systems (time derivative, viscous term, pressure,
// continuity, walls) are the per-wavenumber systems of rbc.hip with the buoyancy coupling off:
// for a Fourier mode (kx, kz) with kh = |(kx, kz)| > 0 the horizontal velocity is written in the
// frame of the wave vector, u_par = (kx u + kz w)/kh, u_perp = (-kz u + kx w)/kh, so that the
// pressure acts on u_par alone (i kh p) and continuity reads i kh u_par + v' = 0; u_perp obeys
// the diffusion equation of the buoyancy slot.  At kh = 0, u_par = u and u_perp = w.
//
// The kernels work in the frame scaled to unit wall distance (y' = (y + 1)/2 in [0, 1],
// x' = x/2, z' = z/2, t' = t/2, same velocity and pressure), where the explicit term is
//   N = -(u.grad) u - U u_x - v U' e_x,   U = 2 y' - 1 (the wall-moving laminar profile), U' = 2,
// on the 3/2 padded grid (Supplementary, "Initial value problems": F(X) of the IVP form).
//
// Layouts (complex128): z-grid fields of the per-mode kernels [f][Ngy][K], mode k = m Nz + n
// (m < Kx half-spectrum x modes, n < Nz z modes in FFT order, the z Nyquist n = Nz/2 unforced);
// plane intermediates [f][Ngy][Ngz][Kx] (x modes contiguous).  Steps:
//   A  per (y, tile of x modes, velocity component): the component, its y-derivative and its
//      z-derivative (i kz), inverse z-FFT onto the padded z grid (9 fields);
//   B  per (y, pair of z rows): the x-derivatives (i kx times the components' x spectra, which are at
//      hand here), packed real inverse x-FFTs of the 12 fields, the products, forward real x-FFTs of
//      the 3 densities;
//   C  per (y, tile of x modes): forward z-FFTs, truncation, 1/(Ngx Ngz), rotation to
//      (par, v, perp).
// The VJP runs the transposes in reverse order (C', B' with the primal fields of A, A').
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "block_fft.h"
#include "cou.h"
#include "sps_device.h"
#include "sps_internal.h"

namespace sps {
namespace {

constexpr size_t kCouLdsMax = 160 * 1024;
constexpr size_t kCouLdsBudget = 40 * 1024;

struct CouDev {
  int Kx, Nz, K, Ngx, Ngz, Ngy;
  double lx, lz, du;
  const double* unode;   // [Ngy] base-flow velocity at the y nodes
  FftPlan px, pz;
  const cplx* twx;       // [Ngx]
  const cplx* twz;       // [Ngz]
};

__device__ __forceinline__ int cou_zrow(int n, int Nz, int G) {
  if (n < Nz / 2) return n;
  if (n == Nz / 2) return -1;
  return n - Nz + G;
}

struct Wave {
  double kx, kz, ex, ez;
};
__device__ __forceinline__ Wave cou_wave(const CouDev& d, int m, int n) {
  const int ns = (n < d.Nz / 2) ? n : n - d.Nz;
  Wave w;
  w.kx = 2.0 * M_PI * m / d.lx;
  w.kz = 2.0 * M_PI * ns / d.lz;
  const double kh = sqrt(w.kx * w.kx + w.kz * w.kz);
  if (kh > 0.0) {
    w.ex = w.kx / kh;
    w.ez = w.kz / kh;
  } else {
    w.ex = 1.0;
    w.ez = 0.0;
  }
  return w;
}

__device__ __forceinline__ cplx lin2(double a, cplx p, double b, cplx q) {
  return cmk(a * p.x + b * q.x, a * p.y + b * q.y);
}

// Hermitian packing of two half spectra (z rows z0, z0 + 1 of one field) into one length-G
// spectrum whose inverse DFT is row_z0 + i row_(z0+1); modes m >= 1 scaled by `scale`.
__device__ __forceinline__ cplx cou_pack(const cplx* U, const cplx* V, int x, int G, int K, double scale) {
  if (x == 0) return cmk(U[0].x, V[0].x);
  if (x < K) return cscale(cmk(U[x].x - V[x].y, U[x].y + V[x].x), scale);
  if (x > G - K) {
    const int q = G - x;
    return cscale(cmk(U[q].x + V[q].y, V[q].x - U[q].y), scale);
  }
  return czero();
}
// ---------------------------------------------------------------------------- in-place FFT
// The plane kernels run the mixed-radix Stockham passes in place in one LDS buffer: a thread
// loads and transforms all of its butterflies of a pass into registers, the block
// synchronizes, and the results go to their Stockham positions.  One buffer instead of a
// ping-pong pair lets two or three blocks share a CU.  A pass of radix R holds up to MB
// butterflies per thread, so a block of nt threads transforms up to 6 nt points
// (nbatch * n <= 6 nt, checked on the host).
// HALF: tw holds only the first n/2 twiddles (w^(m + n/2) = -w^m for even n).
template <int R, int MB, bool HALF>
__device__ __forceinline__ void ip_pass(cplx* buf, const FftPlan& p, int s, const cplx* __restrict__ tw, int sign,
                                        int nbatch, int bstride, int tid, int nt) {
  const int nR = p.n / R, Ns = p.ns[s], tst = p.tst[s];
  const unsigned mnr = p.mag_nr[s], mns = p.mag_ns[s];
  const int total = nbatch * nR;
  cplx v[MB][R];
  int dst[MB];
#pragma unroll
  for (int b = 0; b < MB; ++b) {
    const int it = tid + b * nt;
    dst[b] = -1;
    if (it < total) {
      const int q = fdiv(it, mnr);
      const int j = it - q * nR;
      const int jh = fdiv(j, mns);
      const int k = j - jh * Ns;
      const int t = k * tst;
      const int base = q * bstride;
      // all LDS reads of the butterfly first (one wait), then the twiddle products
      cplx w[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[b][r] = buf[fpad(base + j + r * nR)];
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const int ti = r * t;
        if (HALF) {
          const int hn = p.n >> 1;
          const cplx u = tw[ti < hn ? ti : ti - hn];
          w[r] = (ti < hn) ? u : cmk(-u.x, -u.y);
        } else {
          w[r] = tw[ti];
        }
      }
#pragma unroll
      for (int r = 1; r < R; ++r) v[b][r] = cmul(v[b][r], sign > 0 ? cconj(w[r]) : w[r]);
      dft_small<R>(v[b], sign);
      dst[b] = base + jh * Ns * R + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < MB; ++b)
    if (dst[b] >= 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) buf[fpad(dst[b] + r * Ns)] = v[b][r];
    }
  __syncthreads();
}

// nbatch sequences of length p.n at buf + q * bstride (padded indices), transformed in place;
// ends synchronized.  Every thread of the block calls it.
template <bool HALF = false>
__device__ __forceinline__ void ip_fft(cplx* buf, const FftPlan& p, const cplx* tw, int sign, int nbatch, int bstride,
                                       int tid, int nt) {
  for (int s = 0; s < p.nst; ++s) {
    switch (p.radix[s]) {
      case 8: ip_pass<8, 1, HALF>(buf, p, s, tw, sign, nbatch, bstride, tid, nt); break;
      case 6: ip_pass<6, 1, HALF>(buf, p, s, tw, sign, nbatch, bstride, tid, nt); break;
      case 4: ip_pass<4, 2, HALF>(buf, p, s, tw, sign, nbatch, bstride, tid, nt); break;
      case 3: ip_pass<3, 2, HALF>(buf, p, s, tw, sign, nbatch, bstride, tid, nt); break;
      default: ip_pass<2, 3, HALF>(buf, p, s, tw, sign, nbatch, bstride, tid, nt); break;
    }
  }
}

// half spectrum of row yy (0 or 1) of a packed forward DFT r of two real rows
__device__ __forceinline__ cplx cou_unpack(const cplx* r, int base, int m, int G, int yy) {
  const cplx zm = r[fpad(base + m)], zq = r[fpad(base + (m == 0 ? 0 : G - m))];
  return yy ? cmk(0.5 * (zm.y + zq.y), -0.5 * (zm.x - zq.x)) : cmk(0.5 * (zm.x + zq.x), 0.5 * (zm.y - zq.y));
}

// ---------------------------------------------------------------------------- A: z inverse
// Grid (x-mode tiles, 3 components, Ngy).  Component g (u, v, w) writes fields g, 3 + g, 6 + g
// of Z: the component, its y-derivative, i kz times it.  (The x-derivative is a factor per x mode that
// the row kernels apply: a quarter fewer transforms here and fields through memory.)
template <int NT>
__global__ void __launch_bounds__(NT) cou_zinv(CouDev d, const cplx* zg, int tc, cplx* Z) {
  extern __shared__ double smem_d[];
  const int g = blockIdx.y, y = blockIdx.z, m0 = blockIdx.x * tc, tid = threadIdx.x;
  const int Nz = d.Nz, G = d.Ngz, K = d.K, Kx = d.Kx, Ngy = d.Ngy;
  if (m0 >= Kx) return;
  const int tcn = min(tc, Kx - m0);
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  for (int e = tid; e < G; e += NT) tw[e] = d.twz[e];
  for (int e = tid; e < 3 * tcn * G; e += NT) b0[fpad(e)] = czero();
  __syncthreads();
  for (int e = tid; e < tcn * Nz; e += NT) {
    const int j = e / Nz, n = e - j * Nz, m = m0 + j;
    const int row = cou_zrow(n, Nz, G);
    if (row < 0) continue;
    const long long k = (long long)m * Nz + n;
    const Wave w = cou_wave(d, m, n);
    cplx val, dy;
    if (g == 1) {
      val = zg[(1LL * Ngy + y) * K + k];
      dy = zg[(4LL * Ngy + y) * K + k];
    } else {
      const cplx a = zg[(0LL * Ngy + y) * K + k], c = zg[(2LL * Ngy + y) * K + k];
      const cplx da = zg[(3LL * Ngy + y) * K + k], dc = zg[(5LL * Ngy + y) * K + k];
      if (g == 0) {   // u = ex u_par - ez u_perp
        val = lin2(w.ex, a, -w.ez, c);
        dy = lin2(w.ex, da, -w.ez, dc);
      } else {        // w = ez u_par + ex u_perp
        val = lin2(w.ez, a, w.ex, c);
        dy = lin2(w.ez, da, w.ex, dc);
      }
    }
    b0[fpad((0 * tcn + j) * G + row)] = val;
    b0[fpad((1 * tcn + j) * G + row)] = dy;
    b0[fpad((2 * tcn + j) * G + row)] = cscale(cmul_i(val), w.kz);
  }
  __syncthreads();
  ip_fft(b0, d.pz, tw, +1, 3 * tcn, G, tid, NT);
  const cplx* o = b0;
  for (int e = tid; e < 3 * G * tcn; e += NT) {
    const int q = e / (G * tcn), r = e - q * G * tcn, z = r / tcn, j = r - z * tcn;
    Z[(((long long)(3 * q + g) * Ngy + y) * G + z) * Kx + m0 + j] = o[fpad((q * tcn + j) * G + z)];
  }
}

// ---------------------------------------------------------------------------- B: x rows
// densities of one grid point from the 12 fields (one real row of each)
struct Dens {
  double nu, nv, nw;
};
__device__ __forceinline__ Dens cou_dens(const double* f, double U, double dU) {
  // f: u v w uy vy wy ux uz vx vz wx wz
  Dens r;
  r.nu = -(f[0] * f[6] + f[1] * f[3] + f[2] * f[7]) - U * f[6] - dU * f[1];
  r.nv = -(f[0] * f[8] + f[1] * f[4] + f[2] * f[9]) - U * f[8];
  r.nw = -(f[0] * f[10] + f[1] * f[5] + f[2] * f[11]) - U * f[10];
  return r;
}

// Field f of Z (u, v, w, uy, vy, wy, uz, vz, wz) at point x of the packed rows' spectrum p into its
// slot of h (u v w uy vy wy ux uz vx vz wx wz), and a component's x-derivative: i k p with the signed
// wavenumber k of x.
__device__ __forceinline__ void cou_put(const CouDev& d, cplx* h, int f, int x, cplx p) {
  const int G = d.Ngx, Kx = d.Kx;
  h[fpad((f < 6 ? f : 2 * f - 5) * G + x)] = p;
  if (f < 3) {
    const int k = x < Kx ? x : (x > G - Kx ? x - G : 0);
    h[fpad((6 + 2 * f) * G + x)] = cscale(cmul_i(p), 2.0 * M_PI * k / d.lx);
  }
}

// Grid (Ngz / 2, Ngy), 12 Ngx <= 6 NT.  LDS twiddles(Ngx) + fpad_size(12 Ngx).  The densities
// of a grid point overwrite its u, v, w slots (one thread reads and writes each x).
template <int NT>
__global__ void __launch_bounds__(NT) cou_xrow(CouDev d, const cplx* __restrict__ Z, cplx* __restrict__ W) {
  extern __shared__ double smem_d[];
  const int y = blockIdx.y, z0 = 2 * blockIdx.x, tid = threadIdx.x, G = d.Ngx, Kx = d.Kx, Ngy = d.Ngy, Gz = d.Ngz;
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* h = tw + G;
  for (int e = tid; e < G; e += NT) tw[e] = d.twx[e];
  for (int e = tid; e < 9 * G; e += NT) {
    const int f = e / G, x = e - f * G;
    const cplx* U = Z + (((long long)f * Ngy + y) * Gz + z0) * Kx;
    cou_put(d, h, f, x, cou_pack(U, U + Kx, x, G, Kx, 1.0));
  }
  __syncthreads();
  ip_fft(h, d.px, tw, +1, 12, G, tid, NT);
  const double Uy = d.unode[y], dU = d.du;
  for (int x = tid; x < G; x += NT) {
    double fa[12], fb[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const cplx v = h[fpad(i * G + x)];
      fa[i] = v.x;
      fb[i] = v.y;
    }
    const Dens a = cou_dens(fa, Uy, dU), b = cou_dens(fb, Uy, dU);
    h[fpad(x)] = cmk(a.nu, b.nu);
    h[fpad(G + x)] = cmk(a.nv, b.nv);
    h[fpad(2 * G + x)] = cmk(a.nw, b.nw);
  }
  __syncthreads();
  ip_fft(h, d.px, tw, -1, 3, G, tid, NT);
  const cplx* r = h;
  for (int e = tid; e < 3 * 2 * Kx; e += NT) {
    const int f = e / (2 * Kx), rr = e - f * 2 * Kx, yy = rr / Kx, m = rr - yy * Kx;
    W[(((long long)f * Ngy + y) * Gz + z0 + yy) * Kx + m] = cou_unpack(r, f * G, m, G, yy);
  }
}

// ---------------------------------------------------------------------------- C: z forward
// Grid (x-mode tiles, Ngy).
template <int NT>
__global__ void __launch_bounds__(NT) cou_zfwd(CouDev d, const cplx* W, int tc, cplx* nl) {
  extern __shared__ double smem_d[];
  const int y = blockIdx.y, m0 = blockIdx.x * tc, tid = threadIdx.x;
  const int Nz = d.Nz, G = d.Ngz, K = d.K, Kx = d.Kx, Ngy = d.Ngy;
  if (m0 >= Kx) return;
  const int tcn = min(tc, Kx - m0);
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  for (int e = tid; e < G; e += NT) tw[e] = d.twz[e];
  for (int e = tid; e < 3 * G * tcn; e += NT) {
    const int f = e / (G * tcn), r = e - f * G * tcn, z = r / tcn, j = r - z * tcn;
    b0[fpad((f * tcn + j) * G + z)] = W[(((long long)f * Ngy + y) * G + z) * Kx + m0 + j];
  }
  __syncthreads();
  ip_fft(b0, d.pz, tw, -1, 3 * tcn, G, tid, NT);
  const cplx* res = b0;
  const double s = 1.0 / ((double)d.Ngx * G);
  for (int e = tid; e < tcn * Nz; e += NT) {
    const int j = e / Nz, n = e - j * Nz, m = m0 + j;
    const long long k = (long long)m * Nz + n;
    const int row = cou_zrow(n, Nz, G);
    cplx a = czero(), b = czero(), c = czero();
    if (row >= 0) {
      const Wave w = cou_wave(d, m, n);
      const cplx nu = cscale(res[fpad((0 * tcn + j) * G + row)], s);
      const cplx nv = cscale(res[fpad((1 * tcn + j) * G + row)], s);
      const cplx nw = cscale(res[fpad((2 * tcn + j) * G + row)], s);
      a = lin2(w.ex, nu, w.ez, nw);
      b = nv;
      c = lin2(-w.ez, nu, w.ex, nw);
    }
    nl[(0LL * Ngy + y) * K + k] = a;
    nl[(1LL * Ngy + y) * K + k] = b;
    nl[(2LL * Ngy + y) * K + k] = c;
  }
}

// ---------------------------------------------------------------------------- C': transpose of C
template <int NT>
__global__ void __launch_bounds__(NT) cou_zfwd_adj(CouDev d, const cplx* nlbar, int tc, cplx* Wb) {
  extern __shared__ double smem_d[];
  const int y = blockIdx.y, m0 = blockIdx.x * tc, tid = threadIdx.x;
  const int Nz = d.Nz, G = d.Ngz, K = d.K, Kx = d.Kx, Ngy = d.Ngy;
  if (m0 >= Kx) return;
  const int tcn = min(tc, Kx - m0);
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  for (int e = tid; e < G; e += NT) tw[e] = d.twz[e];
  for (int e = tid; e < 3 * tcn * G; e += NT) b0[fpad(e)] = czero();
  __syncthreads();
  const double s = 1.0 / ((double)d.Ngx * G);
  for (int e = tid; e < tcn * Nz; e += NT) {
    const int j = e / Nz, n = e - j * Nz, m = m0 + j;
    const int row = cou_zrow(n, Nz, G);
    if (row < 0) continue;
    const long long k = (long long)m * Nz + n;
    const Wave w = cou_wave(d, m, n);
    const cplx a = nlbar[(0LL * Ngy + y) * K + k], b = nlbar[(1LL * Ngy + y) * K + k];
    const cplx c = nlbar[(2LL * Ngy + y) * K + k];
    b0[fpad((0 * tcn + j) * G + row)] = cscale(lin2(w.ex, a, -w.ez, c), s);
    b0[fpad((1 * tcn + j) * G + row)] = cscale(b, s);
    b0[fpad((2 * tcn + j) * G + row)] = cscale(lin2(w.ez, a, w.ex, c), s);
  }
  __syncthreads();
  ip_fft(b0, d.pz, tw, +1, 3 * tcn, G, tid, NT);
  const cplx* o = b0;
  for (int e = tid; e < 3 * G * tcn; e += NT) {
    const int f = e / (G * tcn), r = e - f * G * tcn, z = r / tcn, j = r - z * tcn;
    Wb[(((long long)f * Ngy + y) * G + z) * Kx + m0 + j] = o[fpad((f * tcn + j) * G + z)];
  }
}

// ---------------------------------------------------------------------------- B': transpose of B
// Grid (Ngz / 2, Ngy), 15 Ngx <= 6 NT.  LDS twiddles(Ngx / 2) + fpad_size(15 Ngx): three
// 512-thread blocks share a CU at Ngx = 192.  The primal fields Zp (9) and
// the density cotangents Wb (3, weight-1 modes) in; the cotangents of the 9 fields out, as x half
// spectra times w_m (the transpose of the inverse transform), the x-derivatives' (times conj(i kx))
// within their components'.  The cotangents of a grid point
// overwrite its first 12 slots (one thread reads and writes each x).
template <int NT>
__global__ void __launch_bounds__(NT)
cou_xrow_adj(CouDev d, const cplx* __restrict__ Zp, const cplx* __restrict__ Wb, cplx* __restrict__ Gb) {
  extern __shared__ double smem_d[];
  const int y = blockIdx.y, z0 = 2 * blockIdx.x, tid = threadIdx.x, G = d.Ngx, Kx = d.Kx, Ngy = d.Ngy, Gz = d.Ngz;
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* h = tw + G / 2;
  cplx* o = h;
  for (int e = tid; e < G / 2; e += NT) tw[e] = d.twx[e];
  for (int e = tid; e < 12 * G; e += NT) {
    const int f = e / G, x = e - f * G;
    const cplx* U = (f < 9) ? Zp + (((long long)f * Ngy + y) * Gz + z0) * Kx
                            : Wb + (((long long)(f - 9) * Ngy + y) * Gz + z0) * Kx;
    const cplx p = cou_pack(U, U + Kx, x, G, Kx, f < 9 ? 1.0 : 0.5);
    if (f < 9) cou_put(d, h, f, x, p);
    else h[fpad((f + 3) * G + x)] = p;
  }
  __syncthreads();
  ip_fft<true>(h, d.px, tw, +1, 15, G, tid, NT);
  const double Uy = d.unode[y], dU = d.du;
  for (int x = tid; x < G; x += NT) {
    // the two packed rows (real and imaginary parts) one after the other, as doubles
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      double* hd = reinterpret_cast<double*>(h) + r;
      double a[12];
#pragma unroll
      for (int i = 0; i < 12; ++i) a[i] = hd[2 * fpad(i * G + x)];
      const double nu = hd[2 * fpad(12 * G + x)], nv = hd[2 * fpad(13 * G + x)], nw = hd[2 * fpad(14 * G + x)];
      const double adv = a[0] + Uy;
      double out[12];
      out[0] = -(nu * a[6] + nv * a[8] + nw * a[10]);
      out[1] = -(nu * a[3] + nv * a[4] + nw * a[5]) - dU * nu;
      out[2] = -(nu * a[7] + nv * a[9] + nw * a[11]);
      out[3] = -nu * a[1];
      out[4] = -nv * a[1];
      out[5] = -nw * a[1];
      out[6] = -nu * adv;
      out[7] = -nu * a[2];
      out[8] = -nv * adv;
      out[9] = -nv * a[2];
      out[10] = -nw * adv;
      out[11] = -nw * a[2];
#pragma unroll
      for (int i = 0; i < 12; ++i) hd[2 * fpad(i * G + x)] = out[i];
    }
  }
  __syncthreads();
  ip_fft<true>(o, d.px, tw, -1, 12, G, tid, NT);
  const cplx* r = o;
  for (int e = tid; e < 9 * 2 * Kx; e += NT) {
    const int f = e / (2 * Kx), rr = e - f * 2 * Kx, yy = rr / Kx, m = rr - yy * Kx;
    cplx v = cou_unpack(r, (f < 6 ? f : 2 * f - 5) * G, m, G, yy);
    if (f < 3) v = cadd(v, cscale(cmul_mi(cou_unpack(r, (6 + 2 * f) * G, m, G, yy)), 2.0 * M_PI * m / d.lx));
    Gb[(((long long)f * Ngy + y) * Gz + z0 + yy) * Kx + m] = (m == 0) ? v : cscale(v, 2.0);
  }
}

// ---------------------------------------------------------------------------- A': transpose of A
// Grid (x-mode tiles, 2 groups, Ngy): group 0 the u and w fields (6: they mix in the rotation),
// group 1 the v fields (3).  Forward z-FFTs of the field cotangents, the transposes of the
// derivative factors and of the rotation, into zbar[6][Ngy][K].
template <int NT>
__global__ void __launch_bounds__(NT) cou_zinv_adj(CouDev d, const cplx* Gb, int tc, cplx* zbar) {
  extern __shared__ double smem_d[];
  const int grp = blockIdx.y, y = blockIdx.z, m0 = blockIdx.x * tc, tid = threadIdx.x;
  const int Nz = d.Nz, G = d.Ngz, K = d.K, Kx = d.Kx, Ngy = d.Ngy;
  if (m0 >= Kx) return;
  const int tcn = min(tc, Kx - m0);
  const int nf = grp == 0 ? 6 : 3;
  // local slot -> field of Gb: group 0: u, uy, uz, w, wy, wz; group 1: v, vy, vz
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* b0 = tw + G;
  for (int e = tid; e < G; e += NT) tw[e] = d.twz[e];
  for (int e = tid; e < nf * G * tcn; e += NT) {
    const int q = e / (G * tcn), r = e - q * G * tcn, z = r / tcn, j = r - z * tcn;
    const int f = 3 * (q % 3) + (grp == 1 ? 1 : (q < 3 ? 0 : 2));
    b0[fpad((q * tcn + j) * G + z)] = Gb[(((long long)f * Ngy + y) * G + z) * Kx + m0 + j];
  }
  __syncthreads();
  ip_fft(b0, d.pz, tw, -1, nf * tcn, G, tid, NT);
  const cplx* res = b0;
  for (int e = tid; e < tcn * Nz; e += NT) {
    const int j = e / Nz, n = e - j * Nz, m = m0 + j;
    const long long k = (long long)m * Nz + n;
    const int row = cou_zrow(n, Nz, G);
    const Wave w = cou_wave(d, m, n);
    auto at = [&](int q) { return row < 0 ? czero() : res[fpad((q * tcn + j) * G + row)]; };
    // total cotangent of a component: value (with the d/dx part) + conj(i kz) d/dz part
    auto total = [&](int qv, int qz) { return cadd(at(qv), cscale(cmul_mi(at(qz)), w.kz)); };
    if (grp == 0) {
      const cplx ut = total(0, 2), wt = total(3, 5);
      const cplx uy = at(1), wy = at(4);
      zbar[(0LL * Ngy + y) * K + k] = lin2(w.ex, ut, w.ez, wt);
      zbar[(2LL * Ngy + y) * K + k] = lin2(-w.ez, ut, w.ex, wt);
      zbar[(3LL * Ngy + y) * K + k] = lin2(w.ex, uy, w.ez, wy);
      zbar[(5LL * Ngy + y) * K + k] = lin2(-w.ez, uy, w.ex, wy);
    } else {
      zbar[(1LL * Ngy + y) * K + k] = total(0, 2);
      zbar[(4LL * Ngy + y) * K + k] = at(1);
    }
  }
}

// ---------------------------------------------------------------------------- kernels of a known grid length
// The six kernels on Block3, for the padded lengths it has a plan for (3/2 padding): three fields at a time, the
// first pass read from memory and the last one used in registers.  A row kernel goes through its 15 or 27
// transforms in threes, holding only what the products still need: u, v, w in LDS (each of a point's nine
// products has one of them as a factor) and in registers the three densities, or their cotangents and three
// sums.  At 128x64x64, us a launch: cou_zinv 46 -> 32 (147 MB moved), cou_xrow 86 -> 60 (113 MB), cou_zfwd 21 -> 13, cou_zfwd_adj
// 18 -> 12, cou_xrow_adj 141 -> 112 (198 MB; 125 with u, v, w in registers), cou_zinv_adj 62 -> 30.  The row kernels are
// held back by their registers: 256 a lane for two waves per SIMD, and some spill beyond those, in cou_xrow_b 88 (96
// and 192 points) and 104 bytes a lane (48), in cou_xrow_adj_b 76 (72), 156 (96) and 172 (48 and 192)
// (tests/test_kernel_resources.py holds them to that).
template <int G>
struct CouRows {
  static constexpr int PAIRS = G >= 144 ? 4 : G >= 72 ? 8 : 16;   // row pairs of a block
  using B = Block3<G, PAIRS, 4, 4>;
  static constexpr bool ok = B::R0 <= 4;   // (six values a field do not fit the registers)
  static constexpr int HELD = 3 * B::R0 * B::NT;   // u, v, w of the block's threads, held in LDS
  static constexpr size_t lds = sizeof(cplx) * (G + 3 * B::BS + HELD);
};
template <int G>
struct CouCols {
  static constexpr int TC = G >= 144 ? 4 : 8;   // x modes of a block: 64 or 128 bytes of a row
  using Inv = Block3<G, TC, 4, 1>;   // modes (z contiguous) to the plane fields (x contiguous)
  using Fwd = Block3<G, TC, 1, 4>;
  static constexpr size_t lds = sizeof(cplx) * (G + 3 * Inv::BS);
};
// The row kernels' blocks are larger and their chain of transforms is longer, so they need a block for nearly
// every CU: 10 steps and their gradient at 240 blocks (72x40x36) 4.58 ms against 4.81 with the general row
// kernels, at 324 (128x24x48) 6.19 against 6.41; at 180 (48x24x48) 3.33 against 3.11, at 48 (32x16x32) 2.64
// against 2.11.  The column kernels gain at every size.
constexpr int kRowBlocks = 240;
template <typename Fn>
bool cou_with_length(int G, Fn fn) {
  switch (G) {
    case 24: fn(std::integral_constant<int, 24>()); return true;
    case 36: fn(std::integral_constant<int, 36>()); return true;
    case 48: fn(std::integral_constant<int, 48>()); return true;
    case 72: fn(std::integral_constant<int, 72>()); return true;
    case 96: fn(std::integral_constant<int, 96>()); return true;
    case 108: fn(std::integral_constant<int, 108>()); return true;
    case 144: fn(std::integral_constant<int, 144>()); return true;
    case 192: fn(std::integral_constant<int, 192>()); return true;
    default: return false;
  }
}

// Packed spectra (cou_pack) of the row pair at U (second row Kx further) for three consecutive fields, fstr
// apart, at this thread's points x = j + r G / R0; on: the pair exists.
template <int G, int R0>
__device__ __forceinline__ void cou_load3(const cplx* U, long long fstr, int j, bool on, double scale, cplx (&p)[3][R0]) {
  constexpr int Kx = G / 3, NR = G / R0;
  asm volatile("" : "+v"(j));   // not loaded before it is wanted
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    asm volatile("" ::: "memory");   // a field at a time: fewer values held (the transpose at 192 points 113 -> 111 us)
    cplx u[R0], w[R0];
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      u[r] = w[r] = czero();
      if (r * NR >= Kx && (r + 1) * NR - 1 <= G - Kx) continue;
      const int x = j + r * NR;
      if (on && (x < Kx || x > G - Kx)) {
        const cplx* q = U + f * fstr + (x < Kx ? x : G - x);
        u[r] = q[0];
        w[r] = q[Kx];
      }
    }
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const int x = j + r * NR;
      if (x == 0) p[f][r] = cmk(u[r].x, w[r].x);
      else p[f][r] = cscale((x < Kx) ? cmk(u[r].x - w[r].y, u[r].y + w[r].x) : cmk(u[r].x + w[r].y, w[r].x - u[r].y), scale);
    }
  }
}
// signed x wavenumber of point x of a packed spectrum, 0 outside the modes
template <int G>
__device__ __forceinline__ int cou_signed(int x) {
  return x < G / 3 ? x : (x > G - G / 3 ? x - G : 0);
}
__device__ __forceinline__ cplx cmul2(cplx a, cplx b) { return cmk(a.x * b.x, a.y * b.y); }   // the two packed rows' products
__device__ __forceinline__ cplx csub2(cplx a, cplx b, cplx c) { return cmk(a.x - b.x * c.x, a.y - b.y * c.y); }

// Half spectra of the packed natural-order spectra of three fields in buf to out (field f at f fstr), times
// (m == 0 ? 1 : wm).
template <int G, int PAIRS, int NT>
__device__ __forceinline__ void cou_unpack3(const cplx* buf, int bs, int z0, int Gz, long long fstr, double wm, cplx* out, int tid) {
  constexpr int Kx = G / 3;
  for (int e = tid; e < 3 * PAIRS * 2 * Kx; e += NT) {
    const int m = e % Kx, rr = e / Kx, yy = rr & 1, pr = (rr >> 1) % PAIRS, f = (rr >> 1) / PAIRS;
    const cplx* h = buf + f * bs;
    const cplx zm = h[bf_pad(m * PAIRS + pr)], zq = h[bf_pad((m == 0 ? 0 : G - m) * PAIRS + pr)];
    const cplx v = yy ? cmk(0.5 * (zm.y + zq.y), -0.5 * (zm.x - zq.x)) : cmk(0.5 * (zm.x + zq.x), 0.5 * (zm.y - zq.y));
    if (z0 + 2 * pr < Gz) out[f * fstr + (long long)(z0 + 2 * pr + yy) * Kx + m] = (m == 0) ? v : cscale(v, wm);
  }
}

// cou_xrow.  Grid (row pairs / PAIRS, Ngy).
template <int G>
__global__ void __launch_bounds__(CouRows<G>::B::NT, 2) cou_xrow_b(CouDev d, const cplx* __restrict__ Z, cplx* __restrict__ W) {
  using B = typename CouRows<G>::B;
  constexpr int PAIRS = CouRows<G>::PAIRS, R0 = B::R0, NR = B::NR, Kx = G / 3;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  cplx* held = buf + 3 * B::BS + threadIdx.x;   // [f R0 + r][thread]
  const int tid = threadIdx.x, y = blockIdx.y, z0 = 2 * PAIRS * blockIdx.x, Gz = d.Ngz;
  const int j = B::First::bfly(tid), zr = z0 + 2 * B::First::seq(tid);
  const bool on = zr < Gz;
  const long long fstr = (long long)d.Ngy * Gz * Kx;
  const cplx* U = Z + ((long long)y * Gz + zr) * Kx;
  cplx p[3][R0], c[3][R0], n[3][R0];
  cou_load3<G>(U, fstr, j, on, 1.0, p);
  for (int e = tid; e < G; e += B::NT) tw[e] = d.twx[e];
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      c[f][r] = p[f][r];
      p[f][r] = cscale(cmul_i(p[f][r]), 2.0 * M_PI * cou_signed<G>(j + r * NR) / d.lx);
    }
  B::transform(c, buf, tw, +1, tid);   // u, v, w
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int r = 0; r < R0; ++r) held[(f * R0 + r) * B::NT] = c[f][r];
  B::transform(p, buf, tw, +1, tid);   // their x-derivatives
  const double Uy = d.unode[y], dU = d.du;
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    const cplx u = held[r * B::NT], a = cmk(-(u.x + Uy), -(u.y + Uy));
#pragma unroll
    for (int f = 0; f < 3; ++f) n[f][r] = cmul2(a, p[f][r]);
    n[0][r] = csub(n[0][r], cscale(held[(R0 + r) * B::NT], dU));
  }
#pragma unroll
  for (int q = 1; q < 3; ++q) {        // the y- and z-derivatives, with v and w
    cou_load3<G>(U + 3 * q * fstr, fstr, j, on, 1.0, p);
    B::transform(p, buf, tw, +1, tid);
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int r = 0; r < R0; ++r) n[f][r] = csub2(n[f][r], held[(q * R0 + r) * B::NT], p[f][r]);
  }
  B::transform(n, buf, tw, -1, tid);
  B::store(n, buf, tid);
  cou_unpack3<G, PAIRS, B::NT>(buf, B::BS, z0, Gz, fstr, 1.0, W + (long long)y * Gz * Kx, tid);
}

// cou_xrow_adj.  Grid (row pairs / PAIRS, Ngy).
template <int G>
__global__ void __launch_bounds__(CouRows<G>::B::NT, 2)
cou_xrow_adj_b(CouDev d, const cplx* __restrict__ Zp, const cplx* __restrict__ Wb, cplx* __restrict__ Gb) {
  using B = typename CouRows<G>::B;
  constexpr int PAIRS = CouRows<G>::PAIRS, R0 = B::R0, NR = B::NR, Kx = G / 3;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  cplx* held = buf + 3 * B::BS + threadIdx.x;   // [f R0 + r][thread]
  const int tid = threadIdx.x, y = blockIdx.y, z0 = 2 * PAIRS * blockIdx.x, Gz = d.Ngz;
  const int j = B::First::bfly(tid), zr = z0 + 2 * B::First::seq(tid);
  const bool on = zr < Gz;
  const long long fstr = (long long)d.Ngy * Gz * Kx, row = ((long long)y * Gz + zr) * Kx;
  cplx* out = Gb + (long long)y * Gz * Kx;
  const double kf = 2.0 * M_PI / d.lx, Uy = d.unode[y], dU = d.du;
  cplx nb[3][R0], c[3][R0], p[3][R0], s[3][R0];
  for (int e = tid; e < G; e += B::NT) tw[e] = d.twx[e];
  cou_load3<G>(Wb + row, fstr, j, on, 0.5, nb);
  B::transform(nb, buf, tw, +1, tid);  // cotangents of the densities
  cou_load3<G>(Zp + row, fstr, j, on, 1.0, c);
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int r = 0; r < R0; ++r) p[f][r] = cscale(cmul_i(c[f][r]), kf * cou_signed<G>(j + r * NR));
  B::transform(c, buf, tw, +1, tid);   // u, v, w
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int r = 0; r < R0; ++r) held[(f * R0 + r) * B::NT] = c[f][r];
#pragma unroll
  for (int q = 0; q < 3; ++q) {        // the x-, y- and z-derivatives: the cotangents of u, v, w
    if (q > 0) cou_load3<G>(Zp + row + 3 * q * fstr, fstr, j, on, 1.0, p);
    B::transform(p, buf, tw, +1, tid);
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      cplx t = (q == 1) ? cscale(nb[0][r], -dU) : czero();
#pragma unroll
      for (int f = 0; f < 3; ++f) t = csub2(t, nb[f][r], p[f][r]);
      s[q][r] = t;
    }
  }
  // the x-derivatives' cotangents, transposed (conj(i kx)) in their spectra, onto the components'
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const cplx u = held[r * B::NT];
      p[f][r] = cmul2(nb[f][r], cmk(-(u.x + Uy), -(u.y + Uy)));
    }
  B::transform(p, buf, tw, -1, tid);
  B::transform(s, buf, tw, -1, tid);
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int r = 0; r < R0; ++r) s[f][r] = cadd(s[f][r], cscale(cmul_mi(p[f][r]), kf * cou_signed<G>(j + r * NR)));
  B::store(s, buf, tid);
  cou_unpack3<G, PAIRS, B::NT>(buf, B::BS, z0, Gz, fstr, 2.0, out, tid);
#pragma unroll
  for (int q = 1; q < 3; ++q) {        // the y- and z-derivatives' cotangents
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int r = 0; r < R0; ++r) p[f][r] = csub2(czero(), nb[f][r], held[(q * R0 + r) * B::NT]);
    __syncthreads();                   // (the unpacking reads buf)
    B::transform(p, buf, tw, -1, tid);
    B::store(p, buf, tid);
    cou_unpack3<G, PAIRS, B::NT>(buf, B::BS, z0, Gz, fstr, 2.0, out + 3 * q * fstr, tid);
  }
}

// z mode of padded position p (p < Nz / 2, or p > G - Nz / 2), Nz = 2 G / 3
template <int G>
__device__ __forceinline__ bool cou_zmode(int p, int& n) {
  constexpr int Nz = 2 * G / 3;
  n = p < Nz / 2 ? p : p - G + Nz;
  return p < Nz / 2 || p > G - Nz / 2;
}
// compile-time: no position j + r NR, j < NR, holds a mode (STRICT: nor stands for the Nyquist mode Nz / 2)
template <int G, int NR>
__device__ constexpr bool cou_nomode(int r, bool strict) {
  constexpr int Nz = 2 * G / 3;
  return (strict ? r * NR > Nz / 2 : r * NR >= Nz / 2) && (r + 1) * NR - 1 <= G - Nz / 2;
}

// cou_zinv (ADJ: cou_zfwd_adj).  Grid (x-mode tiles, 3 components (ADJ: 1), Ngy).
template <int G, bool ADJ>
__global__ void __launch_bounds__(CouCols<G>::Inv::NT) cou_zinv_b(CouDev d, const cplx* in, cplx* out) {
  using B = typename CouCols<G>::Inv;
  constexpr int R0 = B::R0, NR = B::NR, TC = CouCols<G>::TC, Nz = 2 * G / 3;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  const int tid = threadIdx.x, g = blockIdx.y, y = blockIdx.z, m0 = TC * blockIdx.x, Kx = d.Kx;
  const int j = B::First::bfly(tid), m = m0 + B::First::seq(tid);
  const long long fin = (long long)d.Ngy * d.K;
  const cplx* X = in + (long long)y * d.K + (long long)m * Nz;
  const double s = 1.0 / ((double)d.Ngx * G);
  cplx v[3][R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    v[0][r] = v[1][r] = v[2][r] = czero();
    int n;
    if (cou_nomode<G, NR>(r, false) || !cou_zmode<G>(j + r * NR, n) || m >= Kx) continue;
    if (ADJ) {
      v[0][r] = X[n];
      v[1][r] = X[fin + n];
      v[2][r] = X[2 * fin + n];
    } else if (g == 1) {
      v[0][r] = X[fin + n];
      v[1][r] = X[4 * fin + n];
    } else {   // u_par, u_perp and their y-derivatives, rotated below (v[2]: the second, spare until then)
      v[0][r] = X[n];
      v[2][r] = X[2 * fin + n];
      v[1][r] = X[3 * fin + n];
    }
  }
  cplx dc[R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    dc[r] = czero();
    int n;
    if (ADJ || g == 1 || cou_nomode<G, NR>(r, false) || !cou_zmode<G>(j + r * NR, n) || m >= Kx) continue;
    dc[r] = X[5 * fin + n];
  }
  for (int e = tid; e < G; e += B::NT) tw[e] = d.twz[e];
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    int n;
    if (cou_nomode<G, NR>(r, false) || !cou_zmode<G>(j + r * NR, n) || m >= Kx) continue;
    const Wave w = cou_wave(d, m, n);
    const cplx a = v[0][r], b = v[1][r], c = v[2][r];
    if (ADJ) {
      v[0][r] = cscale(lin2(w.ex, a, -w.ez, c), s);
      v[1][r] = cscale(b, s);
      v[2][r] = cscale(lin2(w.ez, a, w.ex, c), s);
    } else {
      if (g == 0) {          // u = ex u_par - ez u_perp
        v[0][r] = lin2(w.ex, a, -w.ez, c);
        v[1][r] = lin2(w.ex, b, -w.ez, dc[r]);
      } else if (g == 2) {   // w = ez u_par + ex u_perp
        v[0][r] = lin2(w.ez, a, w.ex, c);
        v[1][r] = lin2(w.ez, b, w.ex, dc[r]);
      }
      v[2][r] = cscale(cmul_i(v[0][r]), w.kz);
    }
  }
  B::transform(v, buf, tw, +1, tid);
  const int zo = B::Last::bfly(tid), mo = m0 + B::Last::seq(tid);
  if (mo < Kx) {
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int r = 0; r < R0; ++r)
        out[(((long long)(ADJ ? f : 3 * f + g) * d.Ngy + y) * G + zo + r * NR) * Kx + mo] = v[f][r];
  }
}

// cou_zfwd (ADJ: cou_zinv_adj; group 0 the u and w fields, one after the other, group 1 the v fields).  Grid (x-mode
// tiles, groups (1; ADJ: 2), Ngy).
template <int G, bool ADJ>
__global__ void __launch_bounds__(CouCols<G>::Fwd::NT) cou_zfwd_b(CouDev d, const cplx* in, cplx* out) {
  using B = typename CouCols<G>::Fwd;
  constexpr int R0 = B::R0, NR = B::NR, TC = CouCols<G>::TC, Nz = 2 * G / 3;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  const int tid = threadIdx.x, grp = blockIdx.y, y = blockIdx.z, m0 = TC * blockIdx.x, Kx = d.Kx;
  const int zi = B::First::bfly(tid), mi = m0 + B::First::seq(tid);
  auto load = [&](int f0, int fs, cplx (&v)[3][R0]) {   // fields f0, f0 + fs, f0 + 2 fs
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int r = 0; r < R0; ++r)
        v[f][r] = mi < Kx ? in[(((long long)(f0 + f * fs) * d.Ngy + y) * G + zi + r * NR) * Kx + mi] : czero();
  };
  for (int e = tid; e < G; e += B::NT) tw[e] = d.twz[e];
  cplx v[3][R0], u[3][R0];   // u: the u fields' spectra (ADJ, group 0)
  if (!ADJ) {
    load(0, 1, v);
    B::transform(v, buf, tw, -1, tid);
  } else {
    load(grp, 3, v);
    B::transform(v, buf, tw, -1, tid);
    if (grp == 0) {
#pragma unroll
      for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int r = 0; r < R0; ++r) u[f][r] = v[f][r];
      load(2, 3, v);
      B::transform(v, buf, tw, -1, tid);
    }
  }
  const int j = B::Last::bfly(tid), m = m0 + B::Last::seq(tid);
  if (m >= Kx) return;
  const double s = 1.0 / ((double)d.Ngx * G);
  const long long fo = (long long)d.Ngy * d.K;
  cplx* X = out + (long long)y * d.K + (long long)m * Nz;
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    // position Nz / 2 stands for the unforced Nyquist mode
    int n = 0;
    const int p = j + r * NR;
    if (cou_nomode<G, NR>(r, true)) continue;
    const bool keep = cou_zmode<G>(p, n);
    if (!keep && p != Nz / 2) continue;
    if (!keep) n = Nz / 2;
    const Wave w = cou_wave(d, m, n);
    auto put = [&](int f, cplx x) { X[f * fo + n] = keep ? x : czero(); };
    if (!ADJ) {
      const cplx a = cscale(v[0][r], s), b = cscale(v[1][r], s), c = cscale(v[2][r], s);
      put(0, lin2(w.ex, a, w.ez, c));
      put(1, b);
      put(2, lin2(-w.ez, a, w.ex, c));
    } else {
      // total cotangent of a component: value (with the d/dx part) + conj(i kz) d/dz part
      const cplx t = cadd(v[0][r], cscale(cmul_mi(v[2][r]), w.kz));
      if (grp == 1) {
        put(1, t);
        put(4, v[1][r]);
      } else {
        const cplx ut = cadd(u[0][r], cscale(cmul_mi(u[2][r]), w.kz));
        put(0, lin2(w.ex, ut, w.ez, t));
        put(2, lin2(-w.ez, ut, w.ex, t));
        put(3, lin2(w.ex, u[1][r], w.ez, v[1][r]));
        put(5, lin2(-w.ez, u[1][r], w.ex, v[1][r]));
      }
    }
  }
}

// Launch shapes.  A block transforms in place at most 6 NT points (ip_fft); the column kernels
// take x-mode tiles of tc columns of nf fields.  Blocks of 256 threads with at most kCouLdsBudget
// bytes of LDS, so that several share a CU; 1024 threads where one column of nf fields needs
// more.
constexpr int kColSmall = 256, kColLarge = 1024;
size_t lds_bytes(int G, int points) { return sizeof(cplx) * (G + (size_t)fpad_size(points)); }
int pick_nt(int points) { return points <= 6 * 256 ? 256 : (points <= 6 * 512 ? 512 : 1024); }

struct ColShape {
  int nt = kColSmall, tc = 1;
  size_t lds = 0;
};
ColShape col_shape(int G, int nf, int Kx) {
  ColShape c;
  c.nt = (nf * G <= 6 * kColSmall) ? kColSmall : kColLarge;
  SPS_REQUIRE(nf * G <= 6 * c.nt, "padded z grid too large for the plane kernels");
  // (tiles of 8, 4 or 2 columns: whole 64-byte pieces of the plane fields' lines per row; five columns
  // of three fields would also fit, and were 5 to 15 % slower)
  int tc = std::min(8, Kx);
  while (tc > 1 && (nf * tc * G > 6 * c.nt || lds_bytes(G, nf * tc * G) > kCouLdsBudget)) tc = (tc & (tc - 1)) ? tc - 1 : tc / 2;
  c.tc = tc;
  c.lds = lds_bytes(G, nf * tc * G);
  SPS_REQUIRE(c.lds <= kCouLdsMax, "padded z grid too large for LDS");
  return c;
}

template <typename F1, typename F2>
void launch_col(const ColShape& c, F1 small, F2 large, dim3 grid, hipStream_t s) {
  if (c.nt == kColSmall) small(grid, s);
  else large(grid, s);
  SPS_CHECK_LAUNCH();
}

}  // namespace

CouetteKernels couette_kernels(const CouetteGeom& g) {
  CouetteKernels k;
  if (g.Ngx == 3 * g.Kx)
    cou_with_length(g.Ngx, [&](auto n) {
      using R = CouRows<decltype(n)::value>;
      k.rows = R::ok && (g.Ngz / 2 + R::PAIRS - 1) / R::PAIRS * g.Ngy >= kRowBlocks;
    });
  k.cols = 2 * g.Ngz == 3 * g.Nz && cou_with_length(g.Ngz, [](auto) {});
  return k;
}

struct CouettePlanes::Impl {
  CouDev d{};
  DevArena arena;
  ColShape A, C, A2;
  bool rowsb = false, colsb = false;   // the kernels of a known length (couette_kernels)
  int ntB = 256, ntB2 = 256;
  size_t ldsB = 0, ldsB2 = 0;
  cplx *Zf = nullptr, *Wf = nullptr, *Zv = nullptr, *Wbv = nullptr, *Gv = nullptr;
};

CouettePlanes::CouettePlanes(const CouetteGeom& g, hipStream_t s) : p_(new Impl) {
  Impl& m = *p_;
  CouDev& d = m.d;
  SPS_REQUIRE(g.Kx >= 1 && g.Nz >= 2 && g.Nz % 2 == 0 && g.Ngx % 2 == 0 && g.Ngz % 2 == 0, "bad plane sizes");
  SPS_REQUIRE(g.Ngx >= 2 * g.Kx && g.Ngz >= g.Nz, "padded plane grid smaller than the modes");
  d.Kx = g.Kx;
  d.Nz = g.Nz;
  d.K = g.Kx * g.Nz;
  d.Ngx = g.Ngx;
  d.Ngz = g.Ngz;
  d.Ngy = g.Ngy;
  d.lx = g.lx;
  d.lz = g.lz;
  d.du = g.dunode;
  SPS_REQUIRE(fft_plan(g.Ngx, &d.px) && fft_plan(g.Ngz, &d.pz), "padded plane sizes must factor into 2 and 3");
  SPS_REQUIRE(15 * g.Ngx <= 6 * 1024, "padded x grid too large for the plane kernels");
  d.unode = m.arena.upload(std::vector<double>(g.unode, g.unode + g.Ngy), s);
  d.twx = m.arena.upload(twiddles(g.Ngx), s);
  d.twz = m.arena.upload(twiddles(g.Ngz), s);
  SPS_REQUIRE(8 * g.Ngz <= 6 * kColLarge, "padded z grid too large for the plane kernels");
  m.A = col_shape(g.Ngz, 3, g.Kx);
  m.C = col_shape(g.Ngz, 3, g.Kx);
  m.A2 = col_shape(g.Ngz, 6, g.Kx);
  m.ntB = pick_nt(12 * g.Ngx);
  m.ntB2 = pick_nt(15 * g.Ngx);
  m.ldsB = lds_bytes(g.Ngx, 12 * g.Ngx);
  m.ldsB2 = lds_bytes(g.Ngx / 2, 15 * g.Ngx);
  SPS_REQUIRE(m.ldsB2 <= kCouLdsMax, "padded x grid too large for LDS");
  for (const void* k :
       {(const void*)cou_zinv<kColSmall>, (const void*)cou_zinv<kColLarge>, (const void*)cou_zfwd<kColSmall>,
        (const void*)cou_zfwd<kColLarge>, (const void*)cou_zfwd_adj<kColSmall>, (const void*)cou_zfwd_adj<kColLarge>,
        (const void*)cou_zinv_adj<kColSmall>, (const void*)cou_zinv_adj<kColLarge>, (const void*)cou_xrow<256>,
        (const void*)cou_xrow<512>, (const void*)cou_xrow<1024>, (const void*)cou_xrow_adj<256>,
        (const void*)cou_xrow_adj<512>, (const void*)cou_xrow_adj<1024>})
    SPS_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCouLdsMax));
  auto lds_attr = [](const void* k, size_t b) {
    SPS_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)b));
  };
  const CouetteKernels known = couette_kernels(g);
  m.rowsb = known.rows;
  m.colsb = known.cols;
  if (m.rowsb)
    cou_with_length(g.Ngx, [&](auto n) {
      constexpr int G = decltype(n)::value;
      if constexpr (CouRows<G>::ok) {
        lds_attr((const void*)cou_xrow_b<G>, CouRows<G>::lds);
        lds_attr((const void*)cou_xrow_adj_b<G>, CouRows<G>::lds);
      }
    });
  if (m.colsb)
    cou_with_length(g.Ngz, [&](auto n) {
      constexpr int G = decltype(n)::value;
      lds_attr((const void*)cou_zinv_b<G, false>, CouCols<G>::lds);
      lds_attr((const void*)cou_zinv_b<G, true>, CouCols<G>::lds);
      lds_attr((const void*)cou_zfwd_b<G, false>, CouCols<G>::lds);
      lds_attr((const void*)cou_zfwd_b<G, true>, CouCols<G>::lds);
    });
  const size_t plane = (size_t)g.Ngy * g.Ngz * g.Kx;
  m.Zf = m.arena.alloc<cplx>(9 * plane);
  m.Wf = m.arena.alloc<cplx>(3 * plane);
  m.Zv = m.arena.alloc<cplx>(9 * plane);
  m.Wbv = m.arena.alloc<cplx>(3 * plane);
  m.Gv = m.arena.alloc<cplx>(9 * plane);
}
CouettePlanes::~CouettePlanes() = default;

namespace {
// (x-mode tiles, groups, Ngy) for the kernels that read y from blockIdx.z (A, A'); (x-mode
// tiles, Ngy) for C and C', which read it from blockIdx.y.
dim3 col_grid(const CouDev& d, const ColShape& c, int groups) { return dim3((d.Kx + c.tc - 1) / c.tc, groups, d.Ngy); }
dim3 col_grid_y(const CouDev& d, const ColShape& c) { return dim3((d.Kx + c.tc - 1) / c.tc, d.Ngy); }

// one of the column kernels of a known length; kern(length) gives it
template <typename Kern>
void launch_col_b(const CouDev& d, int groups, const cplx* in, cplx* out, hipStream_t s, Kern kern) {
  cou_with_length(d.Ngz, [&](auto n) {
    using C = CouCols<decltype(n)::value>;
    hipLaunchKernelGGL(kern(n), dim3((d.Kx + C::TC - 1) / C::TC, groups, d.Ngy), dim3(C::Inv::NT), C::lds, s, d, in, out);
  });
  SPS_CHECK_LAUNCH();
}

void launch_zinv(const CouDev& d, const ColShape& c, bool block, const cplx* zg, cplx* Z, hipStream_t s) {
  if (block) {
    launch_col_b(d, 3, zg, Z, s, [](auto n) { return cou_zinv_b<decltype(n)::value, false>; });
    return;
  }
  launch_col(
      c, [&](dim3 g, hipStream_t st) { hipLaunchKernelGGL(cou_zinv<kColSmall>, g, dim3(kColSmall), c.lds, st, d, zg, c.tc, Z); },
      [&](dim3 g, hipStream_t st) { hipLaunchKernelGGL(cou_zinv<kColLarge>, g, dim3(kColLarge), c.lds, st, d, zg, c.tc, Z); },
      col_grid(d, c, 3), s);
}

}  // namespace

void CouettePlanes::forward(const double2* zg, double2* nl, hipStream_t s) {
  Impl& m = *p_;
  const CouDev& d = m.d;
  launch_zinv(d, m.A, m.colsb, zg, m.Zf, s);
  const dim3 gb(d.Ngz / 2, d.Ngy);
  if (m.rowsb)
    cou_with_length(d.Ngx, [&](auto n) {
      using R = CouRows<decltype(n)::value>;
      if constexpr (R::ok)
        hipLaunchKernelGGL(cou_xrow_b<decltype(n)::value>, dim3((d.Ngz / 2 + R::PAIRS - 1) / R::PAIRS, d.Ngy), dim3(R::B::NT),
                           R::lds, s, d, m.Zf, m.Wf);
    });
  else if (m.ntB == 256)
    hipLaunchKernelGGL(cou_xrow<256>, gb, dim3(256), m.ldsB, s, d, m.Zf, m.Wf);
  else if (m.ntB == 512)
    hipLaunchKernelGGL(cou_xrow<512>, gb, dim3(512), m.ldsB, s, d, m.Zf, m.Wf);
  else
    hipLaunchKernelGGL(cou_xrow<1024>, gb, dim3(1024), m.ldsB, s, d, m.Zf, m.Wf);
  SPS_CHECK_LAUNCH();
  if (m.colsb) {
    launch_col_b(d, 1, m.Wf, nl, s, [](auto n) { return cou_zfwd_b<decltype(n)::value, false>; });
    return;
  }
  const ColShape& c = m.C;
  launch_col(
      c, [&](dim3 g, hipStream_t st) { hipLaunchKernelGGL(cou_zfwd<kColSmall>, g, dim3(kColSmall), c.lds, st, d, m.Wf, c.tc, nl); },
      [&](dim3 g, hipStream_t st) { hipLaunchKernelGGL(cou_zfwd<kColLarge>, g, dim3(kColLarge), c.lds, st, d, m.Wf, c.tc, nl); },
      col_grid_y(d, c), s);
}

void CouettePlanes::vjp(const double2* nlbar, const double2* zg, double2* zbar, hipStream_t s) {
  Impl& m = *p_;
  const CouDev& d = m.d;
  launch_zinv(d, m.A, m.colsb, zg, m.Zv, s);
  const ColShape& c = m.C;
  if (m.colsb)
    launch_col_b(d, 1, nlbar, m.Wbv, s, [](auto n) { return cou_zinv_b<decltype(n)::value, true>; });
  else
    launch_col(
        c,
        [&](dim3 g, hipStream_t st) {
          hipLaunchKernelGGL(cou_zfwd_adj<kColSmall>, g, dim3(kColSmall), c.lds, st, d, nlbar, c.tc, m.Wbv);
        },
        [&](dim3 g, hipStream_t st) {
          hipLaunchKernelGGL(cou_zfwd_adj<kColLarge>, g, dim3(kColLarge), c.lds, st, d, nlbar, c.tc, m.Wbv);
        },
        col_grid_y(d, c), s);
  const dim3 gb(d.Ngz / 2, d.Ngy);
  if (m.rowsb)
    cou_with_length(d.Ngx, [&](auto n) {
      using R = CouRows<decltype(n)::value>;
      if constexpr (R::ok)
        hipLaunchKernelGGL(cou_xrow_adj_b<decltype(n)::value>, dim3((d.Ngz / 2 + R::PAIRS - 1) / R::PAIRS, d.Ngy),
                           dim3(R::B::NT), R::lds, s, d, m.Zv, m.Wbv, m.Gv);
    });
  else if (m.ntB2 == 256)
    hipLaunchKernelGGL(cou_xrow_adj<256>, gb, dim3(256), m.ldsB2, s, d, m.Zv, m.Wbv, m.Gv);
  else if (m.ntB2 == 512)
    hipLaunchKernelGGL(cou_xrow_adj<512>, gb, dim3(512), m.ldsB2, s, d, m.Zv, m.Wbv, m.Gv);
  else
    hipLaunchKernelGGL(cou_xrow_adj<1024>, gb, dim3(1024), m.ldsB2, s, d, m.Zv, m.Wbv, m.Gv);
  SPS_CHECK_LAUNCH();
  if (m.colsb) {
    launch_col_b(d, 2, m.Gv, zbar, s, [](auto n) { return cou_zfwd_b<decltype(n)::value, true>; });
    return;
  }
  const ColShape& a2 = m.A2;
  launch_col(
      a2,
      [&](dim3 g, hipStream_t st) {
        hipLaunchKernelGGL(cou_zinv_adj<kColSmall>, g, dim3(kColSmall), a2.lds, st, d, m.Gv, a2.tc, zbar);
      },
      [&](dim3 g, hipStream_t st) {
        hipLaunchKernelGGL(cou_zinv_adj<kColLarge>, g, dim3(kColLarge), a2.lds, st, d, m.Gv, a2.tc, zbar);
      },
      col_grid(d, a2, 2), s);
}

}  // namespace sps
