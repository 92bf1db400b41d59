// Epilogue of the GEMM kernels (bf16 and fp32) and the reduction of split-K
// partials, which applies the same epilogue.
#pragma once
#include "common.h"
#include "kernels.h"

namespace lat {

struct Epi {
  const float* bias;    // [N] or null
  int relu;
  const void* mask;     // activation whose sign gates the output, or null
  DType mask_dt;
  int64_t ldm, s_mask;
  const float* addend;  // + addend[m*ld_add + n] (fp32) or null
  int64_t ld_add, s_add;
  int accumulate;       // + the existing (fp32) C
  // BlockNorm / SwishRN (kernels instantiated with NORM = gate): gain [2, N],
  // pre [M, ldp] (C's dtype), rinv [M, nblk]
  const float* gain;
  float eps;
  void* pre;
  int64_t ldp;
  float* rinv;
  int nblk;
};

template <typename CT>
__device__ inline void epi_store(CT* C, int64_t ldc, int row, int col, float v, const Epi& e,
                                 int64_t bz) {
  if (e.bias) v += e.bias[col];
  if (e.addend) v += e.addend[bz * e.s_add + (int64_t)row * e.ld_add + col];
  if (e.accumulate) v += ld(C + (int64_t)row * ldc + col);
  if (e.relu) v = v > 0.f ? v : 0.f;
  if (e.mask) {
    const int64_t mi = bz * e.s_mask + (int64_t)row * e.ldm + col;
    float g = e.mask_dt == DT_BF16 ? bf2f(((const bf16_t*)e.mask)[mi]) : ((const float*)e.mask)[mi];
    v = g > 0.f ? v : 0.f;
  }
  st(C + (int64_t)row * ldc + col, v);
}

inline Epi make_epi(const GemmArgs& g) {
  return Epi{g.bias,   g.relu,     g.mask, g.mask_dt, g.ldm,  g.s_mask, g.addend,
             g.ld_add, g.s_add,    g.accumulate,      g.gain, g.eps,    g.pre,
             g.ldp,    g.rinv,     g.nblk};
}

// Sum of the splits' partials in split order; the loads of 16 splits are
// issued before their adds (a split's partial is a separate [M, N] slice, so
// a plain loop would wait for one load at a time).
__device__ inline float sum_splits(const float* __restrict__ p, int splits, int64_t stride) {
  float s = 0.f;
  int z = 0;
  for (; z + 16 <= splits; z += 16) {
    float v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = p[(int64_t)(z + q) * stride];
#pragma unroll
    for (int q = 0; q < 16; ++q) s += v[q];
  }
  for (; z < splits; ++z) s += p[(int64_t)z * stride];
  return s;
}

template <typename CT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial,
                                                            int splits, int M, int N,
                                                            CT* __restrict__ C, int64_t ldc,
                                                            Epi epi, const float* __restrict__ rs_partial,
                                                            float* __restrict__ rowsum) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (rowsum && i < M) rowsum[i] = sum_splits(rs_partial + i, splits, M);
  if (i >= (int64_t)M * N) return;
  const int row = (int)(i / N), col = (int)(i % N);
  epi_store<CT>(C, ldc, row, col, sum_splits(partial + i, splits, (int64_t)M * N), epi, 0);
}

}  // namespace lat
