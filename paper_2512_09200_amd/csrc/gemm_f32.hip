// fp32 contractions of the MLPs and heads (fp32 models), same conventions as
// the bf16 kernels: C[m, n] = epilogue( sum_k A(m, k) * B(n, k) ), each operand
// K-contiguous or M-contiguous.
//
// v_mfma_f32_32x32x2_f32 (full fp32 operands and accumulation).  These
// products are small (a few thousand rows, a few hundred columns): what bounds
// them is how many compute units take part and the chain of K steps each
// walks, then the MFMA rate.  So the block tile is 64x64 (a 2048 x 512 product
// gives 256 blocks where 128x128 tiles would give 64), a K step is 64 and a
// block has two groups of 2x2 waves, one 32x32 fragment each: group g takes
// the step's k 32 g .. 32 g + 31, so two waves share a SIMD and the chain of
// steps is half as long; the groups' sums are added once at the end (through
// LDS, group 0 + group 1).  Two LDS stages and one register stage, one barrier
// per step.  Weight gradients, whose output is
// small and whose K is the batch, split K over the chip (gemm_f32_splits).
// A 415 -> 512 -> 256 -> 8 MLP over 2048 samples, forward, loss and backward:
// 121 us (9 products of about 12 us; 6 us of each is the MFMA rate at full
// occupancy, 5 us a launch's start and end), 1540 us with the VALU kernel of
// unsplit 64x64 tiles and scalar loads it replaced.
//
// LDS layouts: a K-contiguous operand as [row][k] with rows padded to 68
// floats, read 4 k at a time (16 bytes per lane; 16 rows cover the 64 banks
// once); an M-contiguous one as [k][row] with k rows of 72 floats, read one k
// at a time (the two lane halves, 4 k rows apart, fall on the two halves of
// the 64 banks).  Lane half h of a fragment holds k = 4 h + i for MFMA i of a
// group of 8 k, for both operands alike, so the two layouts mix freely.
//
// Loads go through buffer resources based at the tile's first element of the
// K step: what lies past the operand's last element reads zero in hardware
// (per dword), rows need no alignment beyond 4 bytes, and spans are not
// limited (the base advances by 64-bit arithmetic; 64 rows of one operand, or
// 64 k rows, must lie within 2 GiB, else WIDE: checked loads by pointer).
// Elements inside the operand but past the K range (the next row of a
// K-contiguous operand) are zeroed at the last step's LDS store; rows past M
// or N only feed outputs that are never written.
#include "common.h"
#include "gemm_epi.h"
#include "kernels.h"

namespace lat {

constexpr int FT = 64, FK = 64, F_THREADS = 512;
constexpr int FLK = FK + 4;   // [row][k] row stride, floats
constexpr int FLM = FT + 8;   // [k][row] k-row stride, floats
constexpr int F_STAGE = FT * FLK > FK * FLM ? FT * FLK : FK * FLM;

// A 64 x 64 operand tile: 1024 16-byte vectors, two per thread.
template <bool MN>
struct F32Tile {
  f32x4 r[2];
  __device__ static inline int row(int v) { return MN ? (v & 15) * 4 : v >> 4; }
  __device__ static inline int kk(int v) { return MN ? v >> 4 : (v & 15) * 4; }
  // WIDE: rows of 2^23 elements or more; rleft, kleft: rows and k from p on
  __device__ inline void load_wide(const float* p, int64_t ld, int rleft, int kleft) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int v = threadIdx.x + i * F_THREADS;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rr = row(v) + (MN ? e : 0), k = kk(v) + (MN ? 0 : e);
        r[i][e] = rr < rleft && k < kleft ? p[MN ? (int64_t)k * ld + rr : (int64_t)rr * ld + k] : 0.f;
      }
    }
  }
  // p: element (row0, k0); left: elements from p to the operand's end
  __device__ inline void load(const float* p, int64_t left, int64_t ld) {
    const int64_t bytes = left > 0 ? left * 4 : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(p), (short)0, (int)(uint32_t)(bytes < 0x7fffffff ? bytes : 0x7fffffff), BUF_RSRC_WORD3);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int v = threadIdx.x + i * F_THREADS;
      const uint32_t off = (uint32_t)((MN ? (int64_t)kk(v) * ld + row(v) : (int64_t)row(v) * ld + kk(v)) * 4);
      r[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
    }
  }
  // kleft: k of this step inside the range (>= FK: all)
  __device__ inline void mask(int kleft) {
    if (kleft >= FK) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = kk(threadIdx.x + i * F_THREADS);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (k + (MN ? 0 : e) >= kleft) r[i][e] = 0.f;
    }
  }
  __device__ inline void store(float* S) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int v = threadIdx.x + i * F_THREADS;
      *reinterpret_cast<f32x4*>(S + (MN ? kk(v) * FLM + row(v) : row(v) * FLK + kk(v))) = r[i];
    }
  }
};

// the wave's operand values of MFMAs 0..3 of the 8 k from ks
template <bool MN>
__device__ inline f32x4 f32_frag(const float* S, int r0, int ks, int lane) {
  const int row = r0 + (lane & 31), k = ks + 4 * (lane >> 5);
  if (!MN) return *reinterpret_cast<const f32x4*>(S + row * FLK + k);
  f32x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = S[(k + i) * FLM + row];
  return v;
}

// the wave's 32 k of a step from kw on (SHORT: those below K)
template <bool TA, bool TB, bool SHORT>
__device__ inline void f32_step(const float* As, const float* Bs, int wm, int wn, int kw, int K, int lane,
                                f32x16& acc) {
#pragma unroll
  for (int ks = 0; ks < FK / 2; ks += 8) {
    if (SHORT && ks >= K) break;  // uniform
    const f32x4 a = f32_frag<TA>(As, wm * 32, kw + ks, lane), b = f32_frag<TB>(Bs, wn * 32, kw + ks, lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
  }
}

// grid: x = M tiles * N tiles (renumbered per XCD), z = split.  partial: fp32
// split partials [split][M][N] (splits > 1).  rowsum (TA only): sums of A over
// k by the blocks of the first N tile, to rs_partial[split][m] when split.
// SHORT: K <= 32, one step of which only group 0 has a part and only the k
// below K are multiplied (a 13-wide input layer: 30000 x 2048 outputs 147 ->
// 102 us, the step's other 48 k being zeros; in the general kernel the bound
// costs every product 5%).
template <bool TA, bool TB, bool WIDE, bool SHORT>
__global__ __launch_bounds__(F_THREADS) void gemm_f32_kernel(const float* __restrict__ A, int64_t lda,
                                                       const float* __restrict__ Bm, int64_t ldb,
                                                       float* __restrict__ C, int64_t ldc, int M, int N,
                                                       int K, int k_per_split, float* __restrict__ partial,
                                                       Epi epi, float* __restrict__ rowsum,
                                                       float* __restrict__ rs_partial) {
  __shared__ __attribute__((aligned(16))) float smem[4 * F_STAGE];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (w >> 1) & 1, wn = w & 1, kg = w >> 2;
  const int tiles_n = (N + FT - 1) / FT;
  const int tile = xcd_block(blockIdx.x, gridDim.x);
  const int m0 = (tile / tiles_n) * FT, n0 = (tile % tiles_n) * FT;
  const int kbeg = blockIdx.z * k_per_split;
  const int kend = K < kbeg + k_per_split ? K : kbeg + k_per_split;
  const int steps = kend > kbeg ? (kend - kbeg + FK - 1) / FK : 0;
  const int64_t endA = TA ? (int64_t)(K - 1) * lda + M : (int64_t)(M - 1) * lda + K;
  const int64_t endB = TB ? (int64_t)(K - 1) * ldb + N : (int64_t)(N - 1) * ldb + K;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  F32Tile<TA> a;
  F32Tile<TB> b;
  auto load = [&](int t) {
    const int64_t k0 = kbeg + (int64_t)t * FK;
    const int64_t oa = TA ? k0 * lda + m0 : (int64_t)m0 * lda + k0;
    const int64_t ob = TB ? k0 * ldb + n0 : (int64_t)n0 * ldb + k0;
    if constexpr (WIDE) {
      a.load_wide(A + oa, lda, M - m0, (int)(K - k0));
      b.load_wide(Bm + ob, ldb, N - n0, (int)(K - k0));
    } else {
      a.load(A + oa, endA - oa, lda);
      b.load(Bm + ob, endB - ob, ldb);
    }
  };
  const bool rs_on = TA && rowsum != nullptr && n0 == 0;
  f32x4 rs = {0.f, 0.f, 0.f, 0.f};
  auto stage = [&](int t) {
    const int kleft = kend - kbeg - t * FK;
    a.mask(kleft);
    b.mask(kleft);
    if (rs_on) rs += a.r[0] + a.r[1];
    float* S = smem + (t & 1) * 2 * F_STAGE;
    a.store(S);
    b.store(S + F_STAGE);
  };
  load(0);
  stage(0);
  if constexpr (SHORT) {
    __syncthreads();
    if (kg == 0) f32_step<TA, TB, true>(smem, smem + F_STAGE, wm, wn, 0, K, lane, acc);
    __syncthreads();
  } else {
    load(1);
    __syncthreads();
    // one step per iteration and no unrolling: most calls run a handful of
    // steps, and a larger body costs more in instruction fetches than the loop
    // saves.  Loads past the range read zeros (or values that are masked).
#pragma unroll 1
    for (int t = 0; t < steps; ++t) {
      const float* S = smem + (t & 1) * 2 * F_STAGE;
      f32_step<TA, TB, false>(S, S + F_STAGE, wm, wn, kg * (FK / 2), K, lane, acc);
      stage(t + 1);
      load(t + 2);
      __syncthreads();
    }
  }
  if (rs_on) {
    // thread: rows 4 (tid % 16) .. +3 over its k class; the classes of a row
    // are added in class order
    constexpr int CLS = F_THREADS / 16;
    *reinterpret_cast<f32x4*>(smem + (threadIdx.x >> 4) * FT + (threadIdx.x & 15) * 4) = rs;
    __syncthreads();
    const int row = m0 + threadIdx.x;
    if (threadIdx.x < FT && row < M) {
      float s = 0.f;
#pragma unroll
      for (int c = 0; c < CLS; ++c) s += smem[c * FT + threadIdx.x];
      if (rs_partial) rs_partial[(int64_t)blockIdx.z * M + row] = s;
      else rowsum[row] = s;
    }
    __syncthreads();
  }
  // the two groups' sums: group 0 finishes registers 0..7 of the fragment,
  // group 1 registers 8..15 (each hands the other half over through LDS)
  float* xch = smem + (w & 3) * 16 * 64 + lane;
  float v[8];
  if (kg == 0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      xch[r * 64] = acc[8 + r];
      v[r] = acc[r];
    }
  } else {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      xch[(8 + r) * 64] = acc[r];
      v[r] = acc[8 + r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] += xch[((1 - kg) * 8 + r) * 64];
  // lane: column lane % 32, rows 8 (r / 4) + 4 (lane / 32) + r % 4
  const int col = n0 + wn * 32 + (lane & 31);
  const int row0 = m0 + wm * 32 + kg * 16 + 4 * (lane >> 5);
  if (col >= N) return;
  if (partial) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int row = row0 + 8 * (r >> 2) + (r & 3);
      if (row < M) partial[((int64_t)blockIdx.z * M + row) * N + col] = v[r];
    }
    return;
  }
  // the epilogue's operands loaded together, from clamped rows
  float mk[8];
  const float bias = epi.bias ? epi.bias[col] : 0.f;
  if (epi.mask) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int row = row0 + 8 * (r >> 2) + (r & 3);
      mk[r] = static_cast<const float*>(epi.mask)[(int64_t)(row < M ? row : M - 1) * epi.ldm + col];
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int row = row0 + 8 * (r >> 2) + (r & 3);
    float x = v[r] + bias;
    if (epi.relu) x = x > 0.f ? x : 0.f;
    if (epi.mask) x = mk[r] > 0.f ? x : 0.f;
    if (row < M) C[(int64_t)row * ldc + col] = x;
  }
}

// Splits of K.  Only weight gradients split (A M-contiguous: K is the batch,
// the output small), from 512 samples on (below, the reduction's launch costs
// what the split saves), to at most one block per compute unit (a second one
// shares its matrix cores: 512 x 415 over K = 2048 takes 10 us at 4 splits of
// 56 tiles, 14 at 6), at least 4 K steps each.  The count grows with K alone
// for given M and N, so a workspace sized for a batch serves every part of it.
int gemm_f32_splits(const GemmArgs& g) {
  if (!g.ta || g.max_splits <= 1 || g.K < 512) return 1;
  const int64_t tiles = (int64_t)cdiv(g.M, FT) * cdiv(g.N, FT);
  int64_t s = 256 / tiles;
  s = s < g.K / (4 * FK) ? s : g.K / (4 * FK);
  s = s < g.max_splits ? s : g.max_splits;
  return s < 1 ? 1 : (int)s;
}

template <bool TA, bool TB>
static hipError_t gemm_f32_launch(const GemmArgs& g, float* ws, hipStream_t st) {
  int splits = gemm_f32_splits(g);
  if (splits > 1 && !ws) {
    set_error("split-K GEMM without a workspace");
    return hipErrorInvalidValue;
  }
  const int kps = cdiv(cdiv(g.K, splits), FK) * FK;
  splits = g.K > 0 ? cdiv(g.K, kps) : 1;
  float* partial = splits > 1 ? ws : nullptr;
  float* rs_partial = splits > 1 && g.rowsum ? ws + (size_t)splits * g.M * g.N : nullptr;
  const Epi epi = make_epi(g);
  const dim3 grid((unsigned)((int64_t)cdiv(g.M, FT) * cdiv(g.N, FT)), 1, splits);
  const int64_t lim = (int64_t)1 << 31;
  const bool wide = g.lda * (TA ? FK : FT) * 4 >= lim || g.ldb * (TB ? FK : FT) * 4 >= lim;
  auto launch = [&](auto kern) {
    kern<<<grid, F_THREADS, 0, st>>>((const float*)g.A, g.lda, (const float*)g.B, g.ldb, (float*)g.C, g.ldc, g.M, g.N,
                               g.K, kps, partial, epi, g.rowsum, rs_partial);
  };
  if constexpr (!TA) {
    if (!wide && g.K <= FK / 2) {
      launch(gemm_f32_kernel<TA, TB, false, true>);
      LAT_LAUNCH_CHECK();
      return hipSuccess;  // (only a weight gradient is split)
    }
  }
  if (wide) launch(gemm_f32_kernel<TA, TB, true, false>);
  else launch(gemm_f32_kernel<TA, TB, false, false>);
  LAT_LAUNCH_CHECK();
  if (splits > 1) {
    splitk_reduce_kernel<float><<<cdiv((int64_t)g.M * g.N, 256), 256, 0, st>>>(
        ws, splits, g.M, g.N, (float*)g.C, g.ldc, epi, rs_partial, g.rowsum);
    LAT_LAUNCH_CHECK();
  }
  return hipSuccess;
}

hipError_t gemm_f32(const GemmArgs& g, float* ws, hipStream_t st) {
  if (g.c_dt != DT_F32 || (g.rowsum && !g.ta) || g.addend || g.accumulate || (g.mask && g.mask_dt != DT_F32)) {
    set_error("fp32 GEMM: fp32 output and mask, no addend, row sums of an M-contiguous A only");
    return hipErrorInvalidValue;
  }
  if (!g.ta && !g.tb) return gemm_f32_launch<false, false>(g, ws, st);
  if (!g.ta) return gemm_f32_launch<false, true>(g, ws, st);
  if (!g.tb) return gemm_f32_launch<true, false>(g, ws, st);
  return gemm_f32_launch<true, true>(g, ws, st);
}

}  // namespace lat
