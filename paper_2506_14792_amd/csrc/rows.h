// Grid-row kernels of the 2D convection problem for the padded row lengths that block_fft.h has a plan for.
#pragma once
#include <hip/hip_runtime.h>

namespace sps {

struct RowsArgs {
  int B, Ngx, Ngz;       // instances, padded row length (3 K, K kept modes), rows
  const double* kx;      // [K]
  const double2* tw;     // [Ngx] exp(-2 pi i t / Ngx)
};

// rows of this length have kernels of their own (sets their LDS limits on first use)
bool rows_supported(int Ngx, int K);
// nl[B][3][Ngz][K]: the x-spectra of the advection products of zg[B][6][Ngz][K]
void rows_fwd(const RowsArgs& r, const double2* zg, double2* nl, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
// zbar[B][6][Ngz][K] = (d nl / d zg)^H nlbar at zg
void rows_adj(const RowsArgs& r, const double2* nlbar, const double2* zg, double2* zbar, hipStream_t s, hipEvent_t e0,
              hipEvent_t e1);

}  // namespace sps
