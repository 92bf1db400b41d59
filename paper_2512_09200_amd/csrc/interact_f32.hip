// Feature interaction on fp32 MFMA (v_mfma_f32_32x32x2_f32), forward and
// backward: fp32 models, and the bf16 shapes the bf16 MFMA kernels do not
// take (FM ranks other than 32 and 64, d other than 64 and 128).  Both storage
// types are staged in LDS as fp32 and contracted in fp32; values are rounded
// to the storage type exactly where they are stored (P = X^T W, dP and the
// outputs).
//
// What bounds these is the fp32 matrix rate (a quarter of a percent of it was
// reached by the scalar kernels: one FMA per two LDS reads) and, at small n,
// the reads of X.  A block holds one sample's operands (small DOT samples:
// four, one per wave) and its waves share the 32x32 output tiles; the FM
// kernels stay resident, keep W in LDS and hold the next sample's X (and its
// gradient) in registers while the current one is computed.
// fp32, 2048 samples of 65 x 128 at rank 32, each kernel's own time: forward 50
// us, backward with the weight gradient 118 + 5 us (scalar kernels: 208, 1580 +
// 119 us), 162 us a forward and backward in a row of calls; the matrix cores
// are busy 42-46% of that, a third of it on the tiles' padding (65 rows as 96);
// what remains is the phases' barriers and LDS latency at two waves per SIMD.
//
// LDS layouts (floats): a matrix whose rows are read along the contraction
// (16 bytes per lane) or across it (one row element per lane) alike has rows
// of length = 4 or 36 mod 64: 16 rows cover the 64 banks once, and the two
// lane halves, 8 k apart, fall on different halves of them.  Lane half h holds
// k = 8 h + i for MFMA i of a group of 16 k, for both operands.  Contractions
// over n or the rank run to the next multiple of 16 over zeroed rows and
// columns; rows and columns of a tile past the matrix repeat its last one and
// are not stored.
#include "common.h"
#include "kernels.h"
#include "mfma_tile.h"

namespace lat {

constexpr int IF_LDS_MAX = 160 * 1024;
constexpr int IF_MAX_ND = 16384;  // n * d of a sample held in registers by the FM kernels
constexpr int IF_MAX_N = 128, IF_MAX_K = 64;
constexpr int FM_F32_FWD_THREADS = 256, FM_F32_BWD_THREADS = 512;

__host__ __device__ inline int if_up16(int x) { return (x + 15) & ~15; }
__host__ __device__ inline int if_tiles(int x) { return (x + 31) >> 5; }

// a lane's 8 operand values of the 16 k from k0 (k = k0 + 8 (lane / 32) + i)
template <bool KC>
__device__ inline void if_frag(float (&v)[8], const float* p, int ld, int k) {
  if (KC) {
    *reinterpret_cast<f32x4*>(v) = *reinterpret_cast<const f32x4*>(p + k);
    *reinterpret_cast<f32x4*>(v + 4) = *reinterpret_cast<const f32x4*>(p + k + 4);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[(k + i) * ld];
  }
}

// acc += A B^T over K (a multiple of 16).  KA / KB: A / B points at the lane's
// row, k contiguous; otherwise at the lane's column of k row 0, k rows lda /
// ldb apart.  (Reading the next 16 k ahead of the MFMAs measured slower: the
// SIMD's other wave already covers the LDS latency.)
template <bool KA, bool KB>
__device__ inline void mm_f32(f32x16& acc, const float* A, int lda, const float* B, int ldb, int K) {
  const int h8 = ((threadIdx.x & 63) >> 5) * 8;
#pragma unroll 1
  for (int k0 = 0; k0 < K; k0 += 16) {
    float a[8], b[8];
    if_frag<KA>(a, A, lda, k0 + h8);
    if_frag<KB>(b, B, ldb, k0 + h8);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
  }
}

__device__ inline int if_clamp(int i, int n) { return i < n ? i : n - 1; }

// Walk of the elements first, first + step, ... of a row-major matrix with
// rows of d, as (row, column) without a division per element.
struct IfWalk {
  int r, c, dr, dc, d;
  __device__ inline IfWalk(int first, int step, int d_)
      : r(first / d_), c(first % d_), dr(step / d_), dc(step % d_), d(d_) {}
  __device__ inline void next() {
    r += dr;
    c += dc;
    if (c >= d) {
      c -= d;
      ++r;
    }
  }
};

template <typename T>
__device__ inline void if_put(float* p, u32x4 x) {
  constexpr int VE = 16 / (int)sizeof(T);
  float f[VE];
  Vec16<T>::unpack(x, f);
#pragma unroll
  for (int q = 0; q < VE; q += 4) *reinterpret_cast<f32x4*>(p + q) = f32x4{f[q], f[q + 1], f[q + 2], f[q + 3]};
}

// a staged value back to T bit for bit (a conversion would quiet a bf16 NaN)
__device__ inline void if_copy(float* p, float v) { *p = v; }
__device__ inline void if_copy(bf16_t* p, float v) { *p = (bf16_t)(__float_as_uint(v) >> 16); }

// A contiguous [rows, d] matrix of T to fp32 LDS rows of ldx by `threads`
// threads (this one is t), 16-byte loads in rounds of U (all of a round in
// flight together; d a multiple of 16).
template <typename T, int U>
__device__ inline void if_stage(const T* __restrict__ g, int rows, int d, float* xs, int ldx, int t, int threads) {
  constexpr int VE = 16 / (int)sizeof(T);
  const int nv = rows * d / VE;
  IfWalk at(t * VE, threads * VE, d);
#pragma unroll 1
  for (int v0 = t; v0 < nv; v0 += U * threads) {
    u32x4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * threads;
      x[u] = ldg16(g + (int64_t)(v < nv ? v : v0) * VE);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (v0 + u * threads < nv) if_put<T>(xs + at.r * ldx + at.c, x[u]);
      at.next();
    }
  }
}

// One sample's X [n, d] in registers (loaded ahead), then to LDS.
template <typename T, int THREADS>
struct IfSample {
  static constexpr int VE = 16 / (int)sizeof(T);
  static constexpr int NV = IF_MAX_ND / VE / THREADS;
  u32x4 x[NV];
  __device__ inline void load(const T* __restrict__ g, int nd) {
#pragma unroll
    for (int u = 0; u < NV; ++u)
      if (u * THREADS * VE < nd) {  // uniform
        const int e = (threadIdx.x + u * THREADS) * VE;
        x[u] = ldg16(g + (e < nd ? e : 0));
      }
  }
  __device__ inline void store(float* xs, int ldx, int d, int nd) const {
    IfWalk at(threadIdx.x * VE, THREADS * VE, d);
#pragma unroll
    for (int u = 0; u < NV; ++u)
      if (u * THREADS * VE < nd) {
        if ((int)(threadIdx.x + u * THREADS) * VE < nd) if_put<T>(xs + at.r * ldx + at.c, x[u]);
        at.next();
      }
  }
};

__device__ inline void if_zero(float* p, int len, int threads) {
  for (int i = threadIdx.x; i < len; i += threads) p[i] = 0.f;
}

// ---------------------------------------------------------------------------
// FM: P = X^T W, O = X P; backward dP = X^T G, dX = G P^T + W dP^T, dW = sum X dP
// ---------------------------------------------------------------------------
struct FmDims {
  int n, d, k, nk, kk, ldx, ldw;  // nk, kk: n and k to the next multiple of 16
};
static FmDims fm_dims(int n, int d, int k) {
  return FmDims{n, d, k, if_up16(n), if_up16(k), d + 4, if_up16(k) + 4};
}

template <typename T>
__device__ inline void fm_stage_w(const T* __restrict__ W, const FmDims& q, float* ws, int threads) {
  const int nw = q.n * q.k;
  IfWalk at(threadIdx.x, threads, q.k);
#pragma unroll 1
  for (int e0 = threadIdx.x; e0 < nw; e0 += 8 * threads) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ld(W + (e0 + u * threads < nw ? e0 + u * threads : e0));
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (e0 + u * threads < nw) ws[at.r * q.ldw + at.c] = v[u];
      at.next();
    }
  }
}

// tile t of [d, kk] = X^T M (M [nk, kk]) to Ps, rounded to T; columns past the
// rank are zeros whatever X holds (its infinities times M's zero columns are
// not, and dX contracts over all kk columns)
template <typename T>
__device__ inline void fm_p_tile(int t, const FmDims& q, const float* xs, const float* M, float* Ps) {
  const int lane = threadIdx.x & 63, kt = if_tiles(q.kk);
  const int a0 = (t / kt) * 32, c0 = (t % kt) * 32;
  f32x16 acc;
  zero16(acc);
  mm_f32<false, false>(acc, xs + if_clamp(a0 + (lane & 31), q.d), q.ldx, M + if_clamp(c0 + (lane & 31), q.kk), q.ldw,
                       q.nk);
  const int c = c0 + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int a = a0 + frag_row(r);
    if (a < q.d && c < q.kk) Ps[a * q.ldw + c] = c < q.k ? ld_round<T>(acc[r]) : 0.f;
  }
}

template <typename T>
__global__ __launch_bounds__(FM_F32_FWD_THREADS) void fm_fwd_f32_kernel(const T* __restrict__ X,
                                                                        const T* __restrict__ W, FmDims q, int B,
                                                                        T* __restrict__ out, int64_t ostride,
                                                                        int emit0) {
  constexpr int NT = FM_F32_FWD_THREADS;
  extern __shared__ __attribute__((aligned(16))) float if_smem[];
  float* xs = if_smem;                 // [nk][ldx]
  float* ws = xs + q.nk * q.ldx;       // [nk][ldw]
  float* ps = ws + q.nk * q.ldw;       // [d][ldw]
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nd = q.n * q.d;
  IfSample<T, NT> sx;
  sx.load(X + (int64_t)blockIdx.x * nd, nd);
  if_zero(if_smem, q.nk * (q.ldx + q.ldw), NT);
  __syncthreads();
  fm_stage_w(W, q, ws, NT);
  const int kt = if_tiles(q.kk);
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    sx.store(xs, q.ldx, q.d, nd);
    __syncthreads();
    if (b + (int)gridDim.x < B) sx.load(X + (int64_t)(b + gridDim.x) * nd, nd);
    for (int t = w; t < if_tiles(q.d) * kt; t += NT / 64) fm_p_tile<T>(t, q, xs, ws, ps);
    __syncthreads();
    T* ob = out + (int64_t)b * ostride;
    if (emit0) {
      for (int a = threadIdx.x; a < q.d; a += NT) if_copy(ob + a, xs[a]);
      ob += q.d;
    }
    for (int t = w; t < if_tiles(q.n) * kt; t += NT / 64) {
      const int j0 = (t / kt) * 32, c = (t % kt) * 32 + (lane & 31);
      f32x16 acc;
      zero16(acc);
      mm_f32<true, false>(acc, xs + if_clamp(j0 + (lane & 31), q.n) * q.ldx, 0, ps + if_clamp(c, q.kk), q.ldw, q.d);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + frag_row(r);
        if (j < q.n && c < q.k) st(ob + j * q.k + c, acc[r]);
      }
    }
    __syncthreads();  // xs and ps are rewritten for the next sample
  }
}

// 8 waves.  dW stays in registers over the block's samples: wave w holds tile
// w % (8 / kp) over the d range w / (8 / kp) of kp ranges (kp: as many as the
// waves allow); the ranges' sums are added in range order at the end.
template <typename T>
__global__ __launch_bounds__(FM_F32_BWD_THREADS) void fm_bwd_f32_kernel(const T* __restrict__ X,
                                                                        const T* __restrict__ W, FmDims q, int B,
                                                                        const T* __restrict__ dout, int64_t dstride,
                                                                        int emit0, int kp, T* __restrict__ dX,
                                                                        float* __restrict__ dw_part) {
  constexpr int NT = FM_F32_BWD_THREADS, NW = NT / 64;
  constexpr int GV = IF_MAX_N * IF_MAX_K / NT;  // gradient elements per thread
  extern __shared__ __attribute__((aligned(16))) float if_smem[];
  float* xs = if_smem;                  // [nk][ldx]
  float* ws = xs + q.nk * q.ldx;        // [nk][ldw]
  float* gs = ws + q.nk * q.ldw;        // [nk][ldw]
  float* ps = gs + q.nk * q.ldw;        // [d][ldw]
  float* dps = ps + q.d * q.ldw;        // [d][ldw]
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nd = q.n * q.d, ng = q.n * q.k;
  const int off = emit0 ? q.d : 0;
  IfSample<T, NT> sx;
  float g[GV];
  auto load = [&](int b) {
    sx.load(X + (int64_t)b * nd, nd);
    const T* gb = dout + (int64_t)b * dstride + off;
#pragma unroll
    for (int u = 0; u < GV; ++u)
      if (u * NT < ng) {  // uniform
        const int e = threadIdx.x + u * NT;
        g[u] = ld(gb + (e < ng ? e : 0));
      }
  };
  load(blockIdx.x);
  if_zero(if_smem, q.nk * (q.ldx + 2 * q.ldw), NT);
  __syncthreads();
  fm_stage_w(W, q, ws, NT);
  const int kt = if_tiles(q.kk), dt = if_tiles(q.d), nt = if_tiles(q.n);
  const int wt = w % (NW / kp), wk = w / (NW / kp);  // this wave's dW tile and d range
  const int kch = if_up16((q.d + kp - 1) / kp);
  const int dk0 = wk * kch, dkn = dk0 < q.d ? (q.d - dk0 < kch ? q.d - dk0 : kch) : 0;
  const int wj = (wt / kt) * 32, wc = (wt % kt) * 32 + (lane & 31);
  const bool w_on = wt < nt * if_tiles(q.k);
  f32x16 dw;
  zero16(dw);
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    sx.store(xs, q.ldx, q.d, nd);
    IfWalk at(threadIdx.x, NT, q.k);
#pragma unroll
    for (int u = 0; u < GV; ++u)
      if (u * NT < ng) {
        if ((int)threadIdx.x + u * NT < ng) gs[at.r * q.ldw + at.c] = g[u];
        at.next();
      }
    __syncthreads();
    if (b + (int)gridDim.x < B) load(b + gridDim.x);
    for (int t = w; t < 2 * dt * kt; t += NW) {
      if (t & 1) fm_p_tile<T>(t >> 1, q, xs, gs, dps);
      else fm_p_tile<T>(t >> 1, q, xs, ws, ps);
    }
    __syncthreads();
    if (w_on && dkn > 0)
      mm_f32<true, false>(dw, xs + if_clamp(wj + (lane & 31), q.n) * q.ldx + dk0, 0,
                          dps + dk0 * q.ldw + if_clamp(wc, q.kk), q.ldw, dkn);
    T* dxb = dX + (int64_t)b * nd;
    const T* g0 = dout + (int64_t)b * dstride;
    // the waves without dW work first
    for (int t = NW - 1 - w; t < nt * dt; t += NW) {
      const int j0 = (t / dt) * 32, a = (t % dt) * 32 + (lane & 31);
      const int jr = if_clamp(j0 + (lane & 31), q.n) * q.ldw, ar = if_clamp(a, q.d) * q.ldw;
      f32x16 acc;
      zero16(acc);
      mm_f32<true, true>(acc, gs + jr, 0, ps + ar, 0, q.kk);
      mm_f32<true, true>(acc, ws + jr, 0, dps + ar, 0, q.kk);
      if (a < q.d) {
        if (emit0 && j0 == 0 && lane < 32) acc[0] += ld(g0 + a);  // row 0 of the tile
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = j0 + frag_row(r);
          if (j < q.n) st(dxb + j * q.d + a, acc[r]);
        }
      }
    }
    __syncthreads();  // the operands are rewritten for the next sample
  }
  // tiles [nt * 32][kt * 32] of dW in LDS, d ranges added in order
  const int ldt = kt * 32;
  for (int z = 0; z < kp; ++z) {
    if (w_on && wk == z) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float* p = if_smem + (wj + frag_row(r)) * ldt + wc;
        *p = (z ? *p : 0.f) + dw[r];
      }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < ng; e += NT)
    dw_part[(int64_t)blockIdx.x * ng + e] = if_smem[(e / q.k) * ldt + e % q.k];
}

static size_t fm_f32_fwd_lds(const FmDims& q) {
  return ((size_t)q.nk * (q.ldx + q.ldw) + (size_t)q.d * q.ldw) * 4;
}
static size_t fm_f32_bwd_lds(const FmDims& q) {
  const size_t run = ((size_t)q.nk * (q.ldx + 2 * q.ldw) + 2 * (size_t)q.d * q.ldw) * 4;
  const size_t end = (size_t)if_tiles(q.n) * if_tiles(q.kk) * 4096;
  return run > end ? run : end;
}

bool fm_f32_supported(int n, int d, int k, const void* X) {
  if (n < 1 || n > IF_MAX_N || k < 1 || k > IF_MAX_K || d % 16 || d > 256 || n * d > IF_MAX_ND) return false;
  return ((uintptr_t)X & 15) == 0 && fm_f32_bwd_lds(fm_dims(n, d, k)) <= IF_LDS_MAX;
}

// resident blocks: what the LDS holds on each of 256 compute units, at most `most`
static int if_blocks(int B, size_t lds, int most) {
  const int per = (int)(IF_LDS_MAX / lds) < most ? (int)(IF_LDS_MAX / lds) : most;
  return B < 256 * per ? B : 256 * per;
}

template <typename T>
static hipError_t fm_fwd_f32_t(const void* X, const void* W, int B, int n, int d, int k, void* out, int64_t ostride,
                               int emit0, hipStream_t s) {
  static LdsLimit lim;
  LAT_HIP_CHECK(lds_limit(fm_fwd_f32_kernel<T>, IF_LDS_MAX, lim));
  const FmDims q = fm_dims(n, d, k);
  const size_t lds = fm_f32_fwd_lds(q);
  fm_fwd_f32_kernel<T><<<if_blocks(B, lds, 4), FM_F32_FWD_THREADS, lds, s>>>((const T*)X, (const T*)W, q, B, (T*)out,
                                                                          ostride, emit0);
  LAT_LAUNCH_CHECK();
  return hipSuccess;
}

template <typename T>
static hipError_t fm_bwd_f32_t(const void* X, const void* W, int B, int n, int d, int k, const void* dout,
                               int64_t dstride, int emit0, void* dX, float* dW, float* part, hipStream_t s) {
  static LdsLimit lim;
  LAT_HIP_CHECK(lds_limit(fm_bwd_f32_kernel<T>, IF_LDS_MAX, lim));
  const FmDims q = fm_dims(n, d, k);
  const size_t lds = fm_f32_bwd_lds(q);
  const int tiles = if_tiles(n) * if_tiles(k);  // <= 8
  const int kp = tiles <= 1 ? 8 : (tiles <= 2 ? 4 : (tiles <= 4 ? 2 : 1));
  const int blocks = if_blocks(B, lds, 2);  // <= 512: fm_bwd_workspace's partials
  fm_bwd_f32_kernel<T><<<blocks, FM_F32_BWD_THREADS, lds, s>>>((const T*)X, (const T*)W, q, B, (const T*)dout, dstride,
                                                              emit0, kp, (T*)dX, part);
  LAT_LAUNCH_CHECK();
  return sum_parts(part, blocks, (int64_t)n * k, dW, s);
}

hipError_t fm_fwd_f32(DType dt, const void* X, const void* W, int B, int n, int d, int k, void* out, int64_t ostride,
                      int emit0, hipStream_t s) {
  if (B == 0) return hipSuccess;
  return dt == DT_BF16 ? fm_fwd_f32_t<bf16_t>(X, W, B, n, d, k, out, ostride, emit0, s)
                       : fm_fwd_f32_t<float>(X, W, B, n, d, k, out, ostride, emit0, s);
}

hipError_t fm_bwd_f32(DType dt, const void* X, const void* W, int B, int n, int d, int k, const void* dout,
                      int64_t dstride, int emit0, void* dX, float* dW, void* ws, hipStream_t s) {
  return dt == DT_BF16 ? fm_bwd_f32_t<bf16_t>(X, W, B, n, d, k, dout, dstride, emit0, dX, dW, (float*)ws, s)
                       : fm_bwd_f32_t<float>(X, W, B, n, d, k, dout, dstride, emit0, dX, dW, (float*)ws, s);
}

// ---------------------------------------------------------------------------
// DOT: pairs i < j of X X^T, packed row by row; backward dX = S X
// ---------------------------------------------------------------------------
// SPB samples per block, one after the other in memory: 4 when a sample is one
// tile (its one or few tiles go to one wave), else 1.
__device__ inline int if_pair_start(int i, int n) { return i * n - i * (i + 1) / 2; }

template <typename T>
__global__ __launch_bounds__(256) void dot_fwd_f32_kernel(const T* __restrict__ X, int B, int n, int d, int spb,
                                                          T* __restrict__ out, int64_t ostride, int emit0) {
  extern __shared__ __attribute__((aligned(16))) float if_smem[];
  const int ldx = d + 4;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b0 = blockIdx.x * spb, cnt = B - b0 < spb ? B - b0 : spb;
  if_stage<T, 8>(X + (int64_t)b0 * n * d, cnt * n, d, if_smem, ldx, threadIdx.x, 256);
  __syncthreads();
  const int off = emit0 ? d : 0;
  if (emit0)
    for (int e = threadIdx.x; e < cnt * d; e += 256)
      if_copy(out + (int64_t)(b0 + e / d) * ostride + e % d, if_smem[(e / d) * n * ldx + e % d]);
  const int nt = if_tiles(n), zt = nt * (nt + 1) / 2;
  for (int t = w; t < cnt * zt; t += 4) {
    const int sm = t / zt;
    int ti = 0, rem = t % zt;
    while (rem >= nt - ti) {
      rem -= nt - ti;
      ++ti;
    }
    const float* xs = if_smem + sm * n * ldx;
    const int j = (ti + rem) * 32 + (lane & 31);
    f32x16 acc;
    zero16(acc);
    mm_f32<true, true>(acc, xs + if_clamp(ti * 32 + (lane & 31), n) * ldx, 0, xs + if_clamp(j, n) * ldx, 0, d);
    T* ob = out + (int64_t)(b0 + sm) * ostride + off;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = ti * 32 + frag_row(r);
      if (i < j && j < n) st(ob + if_pair_start(i, n) + j - i - 1, acc[r]);
    }
  }
}

template <typename T>
__global__ __launch_bounds__(512) void dot_bwd_f32_kernel(const T* __restrict__ X, int B, int n, int d, int spb,
                                                          const T* __restrict__ dout, int64_t dstride, int emit0,
                                                          T* __restrict__ dX) {
  extern __shared__ __attribute__((aligned(16))) float if_smem[];
  const int threads = blockDim.x;
  const int nk = if_up16(n), ldx = d + 4, lds = nk + 4;
  float* xs = if_smem;                   // [spb][nk][ldx], rows past n zero
  float* S = xs + spb * nk * ldx;        // [spb][n][lds], diagonal and columns past n zero
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b0 = blockIdx.x * spb, cnt = B - b0 < spb ? B - b0 : spb;
  const int P = n * (n - 1) / 2, off = emit0 ? d : 0;
  // threads / spb threads fill each sample's operands
  const int gsz = threads / spb, gsm = threadIdx.x / gsz, gt = threadIdx.x % gsz;
  const bool on = gsm < cnt;
  if (on) {
    if_stage<T, 8>(X + (int64_t)(b0 + gsm) * n * d, n, d, xs + gsm * nk * ldx, ldx, gt, gsz);
    for (int e = gt; e < (nk - n) * ldx; e += gsz) xs[(gsm * nk + n) * ldx + e] = 0.f;
    for (int e = gt; e < n * lds; e += gsz) S[gsm * n * lds + e] = 0.f;
  }
  __syncthreads();
  if (on) {
    const T* gb = dout + (int64_t)(b0 + gsm) * dstride + off;
    float* Sb = S + gsm * n * lds;
#pragma unroll 1
    for (int m0 = gt; m0 < P; m0 += 8 * gsz) {
      float g[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) g[u] = ld(gb + (m0 + u * gsz < P ? m0 + u * gsz : m0));
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        // pair m: the row is the largest i with pair_start(i) <= m, from the
        // quadratic's root (exact integers under the root: off by at most one)
        const int m = m0 + u * gsz;
        const float c = 2.f * n - 1.f;
        int i = (int)((c - sqrtf(fmaxf(c * c - 8.f * m, 0.f))) * 0.5f);
        i = i > n - 2 ? n - 2 : i;
        i -= if_pair_start(i, n) > m ? 1 : 0;
        i += i + 1 <= n - 2 && if_pair_start(i + 1, n) <= m ? 1 : 0;
        const int j = m - if_pair_start(i, n) + i + 1;
        if (m < P) {
          Sb[i * lds + j] = g[u];
          Sb[j * lds + i] = g[u];
        }
      }
    }
  }
  __syncthreads();
  const int nt = if_tiles(n), dt = if_tiles(d);
  for (int t = w; t < cnt * nt * dt; t += threads >> 6) {
    const int sm = t / (nt * dt), tt = t % (nt * dt);
    const int i0 = (tt / dt) * 32, a = (tt % dt) * 32 + (lane & 31);
    const T* g0 = dout + (int64_t)(b0 + sm) * dstride;
    f32x16 acc;
    zero16(acc);
    mm_f32<true, false>(acc, S + (sm * n + if_clamp(i0 + (lane & 31), n)) * lds, 0,
                        xs + sm * nk * ldx + if_clamp(a, d), ldx, nk);
    if (a >= d) continue;
    if (emit0 && i0 == 0 && lane < 32) acc[0] += ld(g0 + a);  // row 0 of the tile
    T* dxb = dX + (int64_t)(b0 + sm) * n * d;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = i0 + frag_row(r);
      if (i < n) st(dxb + i * d + a, acc[r]);
    }
  }
}

static int dot_f32_spb(int n) { return n <= 32 ? 4 : 1; }
static size_t dot_f32_bwd_lds(int n, int d) {
  return (size_t)dot_f32_spb(n) * ((size_t)if_up16(n) * (d + 4) + (size_t)n * (if_up16(n) + 4)) * 4;
}

bool dot_f32_supported(int n, int d, const void* X) {
  return n >= 1 && n <= IF_MAX_N && d % 16 == 0 && d <= 256 && ((uintptr_t)X & 15) == 0 &&
         dot_f32_bwd_lds(n, d) <= IF_LDS_MAX;
}

template <typename T>
static hipError_t dot_f32_t(bool fwd, const void* X, int B, int n, int d, void* out, int64_t ostride, int emit0,
                            const void* dout, int64_t dstride, void* dX, hipStream_t s) {
  const int spb = dot_f32_spb(n);
  if (fwd) {
    static LdsLimit lim;
    LAT_HIP_CHECK(lds_limit(dot_fwd_f32_kernel<T>, IF_LDS_MAX, lim));
    dot_fwd_f32_kernel<T><<<cdiv(B, spb), 256, (size_t)spb * n * (d + 4) * 4, s>>>((const T*)X, B, n, d, spb, (T*)out,
                                                                                  ostride, emit0);
  } else {
    static LdsLimit lim;
    LAT_HIP_CHECK(lds_limit(dot_bwd_f32_kernel<T>, IF_LDS_MAX, lim));
    // large samples leave room for one block per compute unit: twice the waves
    const size_t lds = dot_f32_bwd_lds(n, d);
    dot_bwd_f32_kernel<T><<<cdiv(B, spb), lds > IF_LDS_MAX / 3 ? 512 : 256, lds, s>>>(
        (const T*)X, B, n, d, spb, (const T*)dout, dstride, emit0, (T*)dX);
  }
  LAT_LAUNCH_CHECK();
  return hipSuccess;
}

hipError_t dot_f32(DType dt, bool fwd, const void* X, int B, int n, int d, void* out, int64_t ostride, int emit0,
                   const void* dout, int64_t dstride, void* dX, hipStream_t s) {
  if (B == 0) return hipSuccess;
  return dt == DT_BF16 ? dot_f32_t<bf16_t>(fwd, X, B, n, d, out, ostride, emit0, dout, dstride, dX, s)
                       : dot_f32_t<float>(fwd, X, B, n, d, out, ostride, emit0, dout, dstride, dX, s);
}

}  // namespace lat
