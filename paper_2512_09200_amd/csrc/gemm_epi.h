// Epilogue of the GEMM kernels (bf16 and fp32) and the reduction of split-K
// partials, which applies the same epilogue.
#pragma once
#include "common.h"
#include "kernels.h"
#include "swishrn.h"

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

__device__ inline void ld8f(const float* p, float* v) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = a[i];
    v[4 + i] = b[i];
  }
}

// Per-thread coefficients of the BlockNorm epilogue: a thread stores the
// same 8 columns col.. in every row it handles, so bias, g_a, g_b (zeros
// past N) and 1 / |group| are loaded once.
struct NormCoef {
  float b[8], ga[8], gb[8];
  float inv_cnt;
};

__device__ inline void load_norm_coef(const Epi& e, int col, int N, NormCoef& c) {
  load_gains8(e.gain, N, col, c.ga, c.gb);
  if (e.bias && col + 8 <= N && ((uintptr_t)e.bias & 15) == 0) {
    ld8f(e.bias + col, c.b);
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const bool ok = e.bias && col + t < N;
      c.b[t] = ok ? e.bias[ok ? col + t : 0] : 0.f;
    }
  }
  c.inv_cnt = inv_group_size(col, N);
}

// SwishRN with BlockNorm on 8 columns col.. of row `row` of the finished
// fp32 tile (see the header comment).  Every lane of the wave calls it (the
// shuffles need the whole 16-lane group); rows past M and columns past N
// store nothing.
template <typename CT, int GATE>
__device__ inline void epi_blocknorm8(CT* C, int64_t ldc, int row, int col, int M, int N, float* v,
                                      const Epi& e, const NormCoef& nc, int vec) {
  float ss = 0.f;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    v[t] = col + t < N ? v[t] + nc.b[t] : 0.f;
    ss += v[t] * v[t];
  }
  ss = sum16(ss);
  const float r = rsqrtf(ss * nc.inv_cnt + e.eps);
  if (row >= M || col >= N) return;
  if (col % NORM_TILE == 0) e.rinv[(int64_t)row * e.nblk + col / NORM_TILE] = r;
  float o[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const float n = v[t] * r;
    o[t] = (nc.ga[t] * n) * gate_fn<GATE>(nc.gb[t] * n);
  }
  CT* c = C + (int64_t)row * ldc + col;
  CT* p = reinterpret_cast<CT*>(e.pre) + (int64_t)row * e.ldp + col;
  if (vec && col + 8 <= N) {
    if constexpr (sizeof(CT) == 2) {
      stg16(c, Vec16<bf16_t>::pack(o));
      stg16(p, Vec16<bf16_t>::pack(v));
    } else {
      stg16(c, Vec16<float>::pack(o));
      stg16(c + 4, Vec16<float>::pack(o + 4));
      stg16(p, Vec16<float>::pack(v));
      stg16(p + 4, Vec16<float>::pack(v + 4));
    }
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (col + t < N) {
        st(c + t, o[t]);
        st(p + t, v[t]);
      }
  }
}


// Epilogue of 8 consecutive columns of one row with 16-byte vectors (the
// caller guarantees alignment and col + 8 <= N).
template <typename CT>
__device__ inline void epi_store8(CT* C, int64_t ldc, int row, int col, float* v, const Epi& e,
                                  int64_t bz) {
  float t[8];
  if (e.bias) {
    ld8f(e.bias + col, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += t[i];
  }
  if (e.addend) {
    ld8f(e.addend + bz * e.s_add + (int64_t)row * e.ld_add + col, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += t[i];
  }
  CT* c = C + (int64_t)row * ldc + col;
  if (e.accumulate) {  // fp32 C only
    ld8f(reinterpret_cast<const float*>(c), t);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += t[i];
  }
  if (e.relu) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = v[i] > 0.f ? v[i] : 0.f;
  }
  if (e.mask) {
    const int64_t mi = bz * e.s_mask + (int64_t)row * e.ldm + col;
    if (e.mask_dt == DT_BF16) {
      Vec16<bf16_t>::unpack(ldg16(reinterpret_cast<const bf16_t*>(e.mask) + mi), t);
    } else {
      ld8f(reinterpret_cast<const float*>(e.mask) + mi, t);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = t[i] > 0.f ? v[i] : 0.f;
  }
  if constexpr (sizeof(CT) == 2) {
    stg16(c, Vec16<bf16_t>::pack(v));
  } else {
    stg16(c, Vec16<float>::pack(v));
    stg16(c + 4, Vec16<float>::pack(v + 4));
  }
}

inline Epi make_epi(const GemmArgs& g) {
  return Epi{g.bias,   g.relu,     g.mask, g.mask_dt, g.ldm,  g.s_mask, g.addend,
             g.ld_add, g.s_add,    g.accumulate,      g.gain, g.eps,    g.pre,
             g.ldp,    g.rinv,     g.nblk};
}

// Grouped products (parameter untying): blockIdx.z = group.  Rows (gk = 0):
// group z is rows off[z] .. off[z+1]-1 of A, C and the epilogue operands,
// with its own B operand (+ z sB), bias (+ z N) and gains (+ z 2N); blocks
// past a group's rows exit at once.  K (gk = 1): group z sums k = off[z] ..
// off[z+1]-1 into its own C (+ z sC) and row sums (+ z M).
constexpr int GEMM_MAX_GROUPS = 16;
struct GroupSpec {
  int n;    // 0: not grouped
  int gk;
  int off[GEMM_MAX_GROUPS + 1];
  int64_t sB, sC;
};

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
