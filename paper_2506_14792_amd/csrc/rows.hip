// Grid-row kernels of the 2D convection problem on block_fft.h (see rows.h): per z row, inverse real x-FFTs of u, w, b
// and their derivatives as four packed pairs, (u, w), (u_x, u_z), (w_x, w_z), (b_x, b_z), the advection products
// N_f = -(u f_x + w f_z) and their forward x-FFTs; and the transpose.
//
// The four pairs of a row are in one row of 16 lanes (4 f + (0 .. 3) holds pair f at four neighbouring points), so
// that the products are formed by lane exchanges from the last inverse pass's registers and go straight
// into the forward transform's first pass.  Blocks of 96 to 192 threads for one or two rows, bound by latency
// (four barriers a transform): us a launch and its transpose, with the general kernels before and with these, 7.4
// and 7.8 -> 4.1 and 5.0 at 24x14 (36 points), 9.9 and 11.5 -> 6.4 and 8.6 at 96x48 (144 points).
#include <type_traits>

#include "block_fft.h"
#include "rows.h"
#include "sps_device.h"
#include "sps_internal.h"

namespace sps {
namespace {

template <int G>
struct RowsPlan {
  static constexpr int K = G / 3, R0 = BlockPlan<G>::R0, NR = G / R0;
  static constexpr int ROWS = G <= 72 ? 2 : 1, TC = 4 * ROWS, NT = TC * NR;
  using Inv = BlockFft<G, TC, NT, 4, 4>;          // four sequences a row
  using Two = BlockFft<G, 2 * ROWS, NT, 1, 1>;    // the two of the products
  static constexpr size_t lds = sizeof(cplx) * (G + bf_size(TC * G));
};

// values of another pair's lane at the same point: of pair f - n (mod 4)
template <int N>
__device__ __forceinline__ double turn(double v) { return dpp_d<0x120 + 4 * N>(v); }
template <int N>
__device__ __forceinline__ cplx turn(cplx v) { return cmk(turn<N>(v.x), turn<N>(v.y)); }
// pair 0's value
__device__ __forceinline__ cplx first_pair(int f, cplx v) {
  const cplx a = turn<1>(v), b = turn<2>(v), c = turn<3>(v);
  return cmk(f == 0 ? v.x : f == 1 ? a.x : f == 2 ? b.x : c.x, f == 0 ? v.y : f == 1 ? a.y : f == 2 ? b.y : c.y);
}

// Hermitian packing of half spectra U, V (null: zero) into the spectrum of u + i v at the points x = j + r NR:
// x < K direct, x > G - K mirrored, zero between.  dx: U is the x-derivative of the spectrum at U.
template <int G, int R0>
__device__ __forceinline__ void pack_points(const cplx* U, const cplx* V, const double* kx, int j, bool on, double scale,
                                            cplx (&p)[1][R0]) {
  constexpr int K = G / 3, NR = G / R0;
  cplx u[R0], w[R0];
  double k[R0];
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    u[r] = w[r] = czero();
    k[r] = 0.0;
    if (r * NR >= K && (r + 1) * NR - 1 <= G - K) continue;
    const int x = j + r * NR;
    if (on && (x < K || x > G - K)) {
      const int m = x < K ? x : G - x;
      u[r] = U[m];
      if (V) w[r] = V[m];
      if (kx) k[r] = kx[m];
    }
  }
#pragma unroll
  for (int r = 0; r < R0; ++r) {
    const int x = j + r * NR;
    cplx a = u[r];
    if (kx) a = cscale(cmul_i(a), k[r]);
    const cplx b = w[r];
    if (x == 0) p[0][r] = cmk(a.x, b.x);
    else p[0][r] = cscale((x < K) ? cmk(a.x - b.y, a.y + b.x) : cmk(a.x + b.y, b.x - a.y), scale);
  }
}
// half spectra m of the two rows packed in the natural-order spectrum of sequence q of TC
template <int G, int TC>
__device__ __forceinline__ void unpack_point(const cplx* buf, int q, int m, cplx& a, cplx& b) {
  const cplx zm = buf[bf_pad(m * TC + q)], zq = buf[bf_pad((m == 0 ? 0 : G - m) * TC + q)];
  a = cmk(0.5 * (zm.x + zq.x), 0.5 * (zm.y - zq.y));
  b = cmk(0.5 * (zm.y + zq.y), -0.5 * (zm.x - zq.x));
}
// pair f of row z: (u, w), (u_x, u_z), (w_x, w_z), (b_x, b_z); zg fields u, w, b, u_z, w_z, b_z
template <int G, int R0>
__device__ __forceinline__ void primal_points(const RowsArgs& r, const cplx* zg, int f, int j, bool on, cplx (&p)[1][R0]) {
  constexpr int K = G / 3;
  const long long fs = (long long)r.Ngz * K;
  const cplx* U = zg + (f == 0 ? 0 : f - 1) * fs;
  const cplx* V = zg + (f == 0 ? 1 : f + 2) * fs;
  cplx q[1][R0];
  pack_points<G>(U, V, (const double*)nullptr, j, on && f == 0, 1.0, p);
  pack_points<G>(U, V, r.kx, j, on && f != 0, 1.0, q);
#pragma unroll
  for (int i = 0; i < R0; ++i)
    if (f != 0) p[0][i] = q[0][i];
}

template <int G>
__global__ void __launch_bounds__(RowsPlan<G>::NT) rows_fwd_b(RowsArgs r, const cplx* __restrict__ zg, cplx* __restrict__ nl) {
  using P = RowsPlan<G>;
  constexpr int K = P::K, R0 = P::R0, ROWS = P::ROWS;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  const int tid = threadIdx.x, s = P::Inv::First::seq(tid), j = P::Inv::First::bfly(tid), f = s & 3, row = s >> 2;
  const int z0 = blockIdx.x * ROWS, z = z0 + row;
  const long long zs = (long long)r.Ngz * K;
  cplx v[1][R0];
  primal_points<G>(r, zg + blockIdx.y * 6 * zs + (long long)min(z, r.Ngz - 1) * K, f, j, z < r.Ngz, v);
  for (int e = tid; e < G; e += P::NT) tw[e] = r.tw[e];
  P::Inv::First::work(v, tw, +1, tid);
  P::Inv::First::write(v, buf, tid);
  P::Inv::rest(v, buf, tw, +1, tid);
  // N_f on pair f's lanes (f >= 1); the sequences (N_u, N_w) on pair 1's and (N_b, 0) on pair 3's
#pragma unroll
  for (int i = 0; i < R0; ++i) {
    const cplx u = first_pair(f, v[0][i]);
    const double n = -(u.x * v[0][i].x + u.y * v[0][i].y), nw = turn<3>(n);
    v[0][i] = cmk(n, f == 1 ? nw : 0.0);
  }
  P::Inv::First::work(v, tw, -1, tid);
  if (f & 1) {
    const int base = j * R0 * 2 * ROWS + 2 * row + (f >> 1);
#pragma unroll
    for (int i = 0; i < R0; ++i) buf[bf_pad(base + i * 2 * ROWS)] = v[0][i];
  }
  P::Two::rest(v, buf, tw, -1, tid);
  if (P::Two::Last::full || tid < P::Two::Last::NB) P::Two::Last::write(v, buf, tid);
  __syncthreads();
  const double inv = 1.0 / G;
  for (int e = tid; e < ROWS * K; e += P::NT) {
    const int q = e / K, m = e % K;
    if (z0 + q >= r.Ngz) break;
    cplx a, b, c, unused;
    unpack_point<G, 2 * ROWS>(buf, 2 * q, m, a, b);
    unpack_point<G, 2 * ROWS>(buf, 2 * q + 1, m, c, unused);
    cplx* o = nl + blockIdx.y * 3 * zs + (long long)(z0 + q) * K + m;
    o[0] = cscale(a, inv);
    o[zs] = cscale(b, inv);
    o[2 * zs] = cscale(c, inv);
  }
}

template <int G>
__global__ void __launch_bounds__(RowsPlan<G>::NT)
rows_adj_b(RowsArgs r, const cplx* __restrict__ nlbar, const cplx* __restrict__ zg, cplx* __restrict__ zbar) {
  using P = RowsPlan<G>;
  constexpr int K = P::K, R0 = P::R0, ROWS = P::ROWS, TC = P::TC;
  extern __shared__ double smem_d[];
  cplx* tw = reinterpret_cast<cplx*>(smem_d);
  cplx* buf = tw + G;
  const int tid = threadIdx.x, s = P::Inv::First::seq(tid), j = P::Inv::First::bfly(tid), f = s & 3, row = s >> 2;
  const int z0 = blockIdx.x * ROWS, z = z0 + row;
  const long long zs = (long long)r.Ngz * K, zr = (long long)min(z, r.Ngz - 1) * K;
  // the cotangents (N_u, N_w) on pair 0's lanes, (N_b, 0) on pair 1's, weights halved for m >= 1
  const cplx* nb = nlbar + blockIdx.y * 3 * zs + zr;
  cplx v[1][R0], c[1][R0];
  {
    cplx t[1][R0];
    pack_points<G>(nb, nb + zs, (const double*)nullptr, j, z < r.Ngz && f == 0, 0.5, c);
    pack_points<G>(nb + 2 * zs, (const cplx*)nullptr, (const double*)nullptr, j, z < r.Ngz && f == 1, 0.5, t);
#pragma unroll
    for (int i = 0; i < R0; ++i)
      if (f == 1) c[0][i] = t[0][i];
  }
  primal_points<G>(r, zg + blockIdx.y * 6 * zs + zr, f, j, z < r.Ngz, v);
  for (int e = tid; e < G; e += P::NT) tw[e] = r.tw[e];
  P::Inv::First::work(c, tw, +1, tid);
  P::Inv::First::write(c, buf, tid);
  P::Inv::rest(c, buf, tw, +1, tid);
  P::Inv::First::work(v, tw, +1, tid);
  P::Inv::First::write(v, buf, tid);
  P::Inv::rest(v, buf, tw, +1, tid);
  // with N_f the cotangent of product f = 1, 2, 3 on its lanes: (u, w) get -sum_f N_f (f_x, f_z), pair f gets
  // -N_f (u, w)
  const double inv = 1.0 / G;
#pragma unroll
  for (int i = 0; i < R0; ++i) {
    const double nu = turn<1>(c[0][i].x), nw = turn<2>(c[0][i].y), nbb = turn<2>(c[0][i].x);
    const double n = (f == 0) ? 0.0 : (f == 1 ? nu : f == 2 ? nw : nbb) * inv;
    const cplx u = first_pair(f, v[0][i]);
    double a = n * v[0][i].x, b = n * v[0][i].y;
    a += turn<2>(a);
    a += turn<1>(a);
    b += turn<2>(b);
    b += turn<1>(b);
    v[0][i] = (f == 0) ? cmk(-a, -b) : cmk(-n * u.x, -n * u.y);
  }
  P::Inv::First::work(v, tw, -1, tid);
  P::Inv::First::write(v, buf, tid);
  P::Inv::rest(v, buf, tw, -1, tid);
  P::Inv::Last::write(v, buf, tid);
  __syncthreads();
  // weight 1 at m = 0, 2 else; the x-derivatives' cotangents, transposed (conj(i kx)), onto the components'
  for (int e = tid; e < ROWS * 3 * K; e += P::NT) {
    const int m = e % K, t = e / K, g = t % 3, q = t / 3;
    if (z0 + q >= r.Ngz) break;
    cplx a0, b0, ad, bd;
    unpack_point<G, TC>(buf, 4 * q, m, a0, b0);
    unpack_point<G, TC>(buf, 4 * q + 1 + g, m, ad, bd);
    const double wgt = (m == 0) ? 1.0 : 2.0;
    cplx base = czero();
    if (g == 0) base = cscale(a0, wgt);
    if (g == 1) base = cscale(b0, wgt);
    cplx* o = zbar + blockIdx.y * 6 * zs + g * zs + (long long)(z0 + q) * K + m;
    o[0] = cadd(base, cscale(cmul_mi(cscale(ad, wgt)), r.kx[m]));
    o[3 * zs] = cscale(bd, wgt);
  }
}

// fn(the length as a type) if it has kernels
template <typename Fn>
bool with_length(int G, Fn fn) {
  switch (G) {
    case 24: fn(std::integral_constant<int, 24>()); return true;
    case 36: fn(std::integral_constant<int, 36>()); return true;
    case 48: fn(std::integral_constant<int, 48>()); return true;
    case 72: fn(std::integral_constant<int, 72>()); return true;
    case 96: fn(std::integral_constant<int, 96>()); return true;
    case 108: fn(std::integral_constant<int, 108>()); return true;
    case 144: fn(std::integral_constant<int, 144>()); return true;
    case 216: fn(std::integral_constant<int, 216>()); return true;
    case 288: fn(std::integral_constant<int, 288>()); return true;
    default: return false;
  }
}

}  // namespace

bool rows_supported(int Ngx, int K) {
  if (Ngx != 3 * K) return false;
  return with_length(Ngx, [](auto n) {
    constexpr int G = decltype(n)::value;
    SPS_HIP(hipFuncSetAttribute((const void*)rows_fwd_b<G>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)RowsPlan<G>::lds));
    SPS_HIP(hipFuncSetAttribute((const void*)rows_adj_b<G>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)RowsPlan<G>::lds));
  });
}
void rows_fwd(const RowsArgs& r, const double2* zg, double2* nl, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  with_length(r.Ngx, [&](auto n) {
    using P = RowsPlan<decltype(n)::value>;
    hipExtLaunchKernelGGL(rows_fwd_b<decltype(n)::value>, dim3((r.Ngz + P::ROWS - 1) / P::ROWS, r.B), dim3(P::NT), P::lds, s, e0, e1,
                          0, r, zg, nl);
  });
  SPS_CHECK_LAUNCH();
}
void rows_adj(const RowsArgs& r, const double2* nlbar, const double2* zg, double2* zbar, hipStream_t s, hipEvent_t e0,
              hipEvent_t e1) {
  with_length(r.Ngx, [&](auto n) {
    using P = RowsPlan<decltype(n)::value>;
    hipExtLaunchKernelGGL(rows_adj_b<decltype(n)::value>, dim3((r.Ngz + P::ROWS - 1) / P::ROWS, r.B), dim3(P::NT), P::lds, s, e0, e1,
                          0, r, nlbar, zg, zbar);
  });
  SPS_CHECK_LAUNCH();
}

}  // namespace sps
