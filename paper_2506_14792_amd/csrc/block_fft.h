// A block's FFT of TC interleaved sequences of a length known at compile time, three Stockham passes in
// place in LDS: entry (position, sequence) is at bf_pad(position TC + sequence).  Every thread holds its
// butterflies of a pass in registers between reading and writing (a block barrier each), so one buffer
// does, a caller can take the first pass's inputs straight from memory and use the last pass's outputs
// in registers, and all index arithmetic but one address a butterfly is in the instructions' constants.
// The general FFT of sps_device.h spends 25 to 30 vector instructions a value and pass, of which the
// transform itself is about 12, and reads and writes LDS once more on either side; a 768-point row took 178
// instructions a value with it.
#pragma once
#include "sps_device.h"

namespace sps {

// Lengths: R0 R1 R0.  The first and the last radix are the same, so that a thread's outputs of one
// transform, positions j + r n / R0, are the inputs of its butterfly of the next one's first pass.
template <int N> struct BlockPlan { static constexpr bool ok = false; };
#define SPS_BLOCK_PLAN(N_, A, B) \
  template <> struct BlockPlan<N_> { static constexpr bool ok = true; static constexpr int R0 = A, R1 = B; \
                                     static_assert(A * B * A == N_, "radices"); };
SPS_BLOCK_PLAN(24, 2, 6)
SPS_BLOCK_PLAN(32, 4, 2)
SPS_BLOCK_PLAN(36, 3, 4)
SPS_BLOCK_PLAN(48, 4, 3)
SPS_BLOCK_PLAN(64, 4, 4)
SPS_BLOCK_PLAN(72, 3, 8)
SPS_BLOCK_PLAN(96, 4, 6)
SPS_BLOCK_PLAN(108, 3, 12)
SPS_BLOCK_PLAN(128, 8, 2)
SPS_BLOCK_PLAN(144, 6, 4)
SPS_BLOCK_PLAN(192, 8, 3)
SPS_BLOCK_PLAN(216, 6, 6)
SPS_BLOCK_PLAN(256, 8, 4)
SPS_BLOCK_PLAN(288, 6, 8)
SPS_BLOCK_PLAN(384, 8, 6)
SPS_BLOCK_PLAN(512, 8, 8)
SPS_BLOCK_PLAN(576, 12, 4)
SPS_BLOCK_PLAN(768, 8, 12)
#undef SPS_BLOCK_PLAN

// Four spare slots after every 32 entries: butterflies of the first pass, 32 entries or a multiple apart,
// write to different banks.
__host__ __device__ constexpr int bf_pad(int e) { return e + ((e >> 5) << 2); }
__host__ __device__ constexpr int bf_size(int n) { return bf_pad(n) + 4; }

// bf_pad(base + OFF), given base and pb = bf_pad(base)
template <int OFF>
__device__ __forceinline__ int bf_at(int base, int pb) {
  return (OFF % 32 == 0) ? pb + OFF + OFF / 8 : bf_pad(base + OFF);
}

// Radix 12 = 3 x 4 (coprime): n = 4 n1 + 3 n2, k = 4 k1 + 9 k2 (mod 12), no twiddles.
template <int R>
__device__ __forceinline__ void bf_dft(cplx* v, int sign) {
  if constexpr (R == 12) {
    cplx a[4][3];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < 3; ++n1) a[n2][n1] = v[(4 * n1 + 3 * n2) % 12];
      dft_small<3>(a[n2], sign);
    }
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) {
      cplx b[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
      dft_small<4>(b, sign);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) v[(4 * k1 + 9 * k2) % 12] = b[k2];
    }
  } else {
    dft_small<R>(v, sign);
  }
}

// One pass: radix R after passes of product NS, over TC sequences of length N by NT threads.  A thread's
// butterfly number it is that of butterfly bfly(it) of sequence seq(it): JF consecutive butterflies of a
// sequence, then the same of the next.  JF = 1 where a caller's memory has the sequences next to each other, 4
// where it has a sequence's positions: four lanes then read or write 64 bytes at a time (lane by lane, the
// advection rows of six 768 x 768 grids took 50 us, so 42).
template <int N, int R, int NS, int TC, int NT, int JF>
struct BlockPass {
  static constexpr int NB = N / R * TC, MB = (NB + NT - 1) / NT, NR = N / R;
  static constexpr bool full = NB % NT == 0;
  static_assert(NR % JF == 0, "whole groups");
  static __device__ __forceinline__ int bfly(int it) { return JF == 1 ? it / TC : it / (JF * TC) * JF + it % JF; }
  static __device__ __forceinline__ int seq(int it) { return it / JF % TC; }
  template <int r = 0>
  static __device__ __forceinline__ void read1(cplx* v, const cplx* buf, int base, int pb) {
    v[r] = buf[bf_at<r * NR * TC>(base, pb)];
    if constexpr (r + 1 < R) read1<r + 1>(v, buf, base, pb);
  }
  static __device__ __forceinline__ void read_one(cplx* v, const cplx* buf, int it) {
    const int base = bfly(it) * TC + seq(it);
    read1(v, buf, base, bf_pad(base));
  }
  static __device__ __forceinline__ void read(cplx (&v)[MB][R], const cplx* buf, int tid) {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int it = tid + i * NT;
      if (full || it < NB) read_one(v[i], buf, it);
    }
  }
  // twiddles (tw[t] = exp(-2 pi i t / N)) and the butterfly
  static __device__ __forceinline__ void work_one(cplx* v, const cplx* tw, int sign, int it) {
    if constexpr (NS > 1) {
      const int t = (bfly(it) % NS) * (N / (NS * R));
#pragma unroll
      for (int r = 1; r < R; ++r) {
        cplx w = tw[r * t];
        if (sign > 0) w = cconj(w);
        v[r] = cmul(v[r], w);
      }
    }
    bf_dft<R>(v, sign);
  }
  static __device__ __forceinline__ void work(cplx (&v)[MB][R], const cplx* tw, int sign, int tid) {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int it = tid + i * NT;
      if (full || it < NB) work_one(v[i], tw, sign, it);
    }
  }
  static __device__ __forceinline__ int out_base(int it) {   // entry of output 0
    const int j = bfly(it), q = seq(it);
    return ((j / NS) * NS * R + j % NS) * TC + q;
  }
  template <int r = 0>
  static __device__ __forceinline__ void write1(const cplx* v, cplx* buf, int base, int pb) {
    // (a butterfly that fills 32 entries exactly has no spare slots inside)
    if constexpr (NS * R * TC == 32) buf[pb + r * NS * TC] = v[r];
    else buf[bf_at<r * NS * TC>(base, pb)] = v[r];
    if constexpr (r + 1 < R) write1<r + 1>(v, buf, base, pb);
  }
  static __device__ __forceinline__ void write_one(const cplx* v, cplx* buf, int it) {
    const int base = out_base(it);
    write1(v, buf, base, bf_pad(base));
  }
  static __device__ __forceinline__ void write(const cplx (&v)[MB][R], cplx* buf, int tid) {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int it = tid + i * NT;
      if (full || it < NB) write_one(v[i], buf, it);
    }
  }
};

// The passes after the first (its outputs are in buf; no barrier since they were written).  Leaves the
// last pass's outputs in v: v[i][r] is position bfly(it) + r N / R0 of sequence seq(it), it = tid +
// i NT; every thread is past its last read of buf.  JF0, JF2: the order of the first and the last pass.
template <int N, int TC, int NT, int JF0, int JF2>
struct BlockFft {
  static constexpr int R0 = BlockPlan<N>::R0, R1 = BlockPlan<N>::R1;
  using First = BlockPass<N, R0, 1, TC, NT, JF0>;
  using Mid = BlockPass<N, R1, R0, TC, NT, 1>;
  using Last = BlockPass<N, R0, R0 * R1, TC, NT, JF2>;
  static __device__ __forceinline__ void rest(cplx (&v)[Last::MB][R0], cplx* buf, const cplx* tw, int sign, int tid) {
    {
      cplx m[Mid::MB][R1];
      __syncthreads();
      Mid::read(m, buf, tid);
      __syncthreads();
      Mid::work(m, tw, sign, tid);
      Mid::write(m, buf, tid);
    }
    __syncthreads();
    Last::read(v, buf, tid);
    __syncthreads();
    Last::work(v, tw, sign, tid);
  }
};

// Three fields of TC sequences each, a thread holding the same butterfly of all three in the first and last
// pass (so that products of the fields stay in its registers); first radices of 2 to 6 keep those few.
template <int N> struct Block3Plan { static constexpr bool ok = false; };
#define SPS_BLOCK3_PLAN(N_, A, B) \
  template <> struct Block3Plan<N_> { static constexpr bool ok = true; static constexpr int R0 = A, R1 = B; \
                                      static_assert(A * B * A == N_, "radices"); };
SPS_BLOCK3_PLAN(24, 2, 6)
SPS_BLOCK3_PLAN(36, 3, 4)
SPS_BLOCK3_PLAN(48, 4, 3)
SPS_BLOCK3_PLAN(72, 3, 8)
SPS_BLOCK3_PLAN(96, 4, 6)
SPS_BLOCK3_PLAN(108, 3, 12)
SPS_BLOCK3_PLAN(144, 6, 4)
SPS_BLOCK3_PLAN(192, 4, 12)
#undef SPS_BLOCK3_PLAN

template <int N, int TC, int JF0, int JF2>
struct Block3 {
  static constexpr int R0 = Block3Plan<N>::R0, R1 = Block3Plan<N>::R1, NT = N / R0 * TC, NR = N / R0;
  static constexpr int BS = bf_size(TC * N);   // entries of a field's buffer
  using First = BlockPass<N, R0, 1, TC, NT, JF0>;
  using Mid = BlockPass<N, R1, R0, TC, NT, 1>;
  using Last = BlockPass<N, R0, R0 * R1, TC, NT, JF2>;
  // v: the inputs at positions First::bfly(tid) + r N / R0 of sequence First::seq(tid), then the outputs at
  // Last's; every thread must be past its reads of buf, and is again on return.
  static __device__ __forceinline__ void transform(cplx (&v)[3][R0], cplx* buf, const cplx* tw, int sign, int tid) {
    asm volatile("" : "+v"(tid));   // index arithmetic is redone for every transform, not kept in registers between them
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      First::work_one(v[f], tw, sign, tid);
      First::write_one(v[f], buf + f * BS, tid);
    }
    constexpr int NM = 3 * Mid::NB, MM = (NM + NT - 1) / NT;
    {
      cplx m[MM][R1];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MM; ++i) {
        const int it = tid + i * NT;
        if (NM % NT == 0 || it < NM) Mid::read_one(m[i], buf + it / Mid::NB * BS, it % Mid::NB);
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MM; ++i) {
        const int it = tid + i * NT;
        if (NM % NT == 0 || it < NM) {
          Mid::work_one(m[i], tw, sign, it % Mid::NB);
          Mid::write_one(m[i], buf + it / Mid::NB * BS, it % Mid::NB);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 3; ++f) Last::read_one(v[f], buf + f * BS, tid);
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 3; ++f) Last::work_one(v[f], tw, sign, tid);
  }
  // the last outputs to buf in natural order, ends synchronized
  static __device__ __forceinline__ void store(const cplx (&v)[3][R0], cplx* buf, int tid) {
#pragma unroll
    for (int f = 0; f < 3; ++f) Last::write_one(v[f], buf + f * BS, tid);
    __syncthreads();
  }
};

}  // namespace sps
