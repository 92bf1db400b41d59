// bf16 contractions of few tiles: C[m, n] = epilogue( sum_k A(m, k) B(n, k) ),
// each operand K-contiguous or M-contiguous, rows aligned to 16 bytes (or, with
// REG, on any element) and operands below 2 GiB.  gemm() takes this kernel for products that would
// leave most of the chip without a 128 x 128 tile (gemm_use_small); such a
// product is bound by the chain of K steps a block walks and by a launch's
// start and end, not by the matrix cores.
//
// So the tile is 64 x 64 (four times the blocks), a block has 8 waves, two
// groups of 2 x 2 waves of 32 x 32 with group g on k 32 g .. 32 g + 31 of each
// 64-k step (sums added at the end, group 0 + group 1), and operands go from
// memory straight to LDS (buffer_load_dwordx4 ... lds) four stages deep: a
// wave issues the loads of the step three ahead, waits by count for those of
// the current step (the later ones stay in flight across the barrier) and
// crosses one barrier per step, which both publishes the step and frees the
// stage the new loads overwrite.  Loads past the range read zeros, so every
// step issues the same number and the count is a constant.  512 x 1024 x 2208
// (32 tiles of 128 x 128): 23.1 -> 13.9 us; 2048 x 512 x 416: 10.8 -> 6.7 us;
// 2048 x 256 x 512: 10.5 -> 6.6 us.  (The same scheme with 128 x 128 and 256 x
// 256 tiles, two stages, measured no faster than the register-staged kernels:
// those products are bound by the LDS port, which it does not relieve.)
//
// LDS layouts, in 16-byte units, one wave load writing 64 consecutive ones.
// K-contiguous operand: [row][64 k], 8 units a row, unit c of row r at c ^
// ((r >> 1) & 7): the 16 rows a fragment read serves at a time fall on
// distinct banks.  M-contiguous operand: [k][64 rows], read back as fragments
// by transposed LDS reads (ds_read_b64_tr_b16), whose four consecutive k rows
// (two to the banks' width) are moved to disjoint 64-byte bank groups by the
// unit's XOR with 4 ((k >> 1) & 1).  The permutation is made by the lanes'
// global addresses, inside one row's 128 bytes.
#include "common.h"
#include "gemm_epi.h"
#include "kernels.h"

namespace lat {

constexpr int DT = 64;                             // tile rows and columns
constexpr int DK = 64;                             // k per step
constexpr int D_THREADS = 512, D_STAGES = 4;
constexpr int D_TILE = DT * DK;                    // elements of an operand's stage
constexpr int CLD = DT + 4;                        // row stride of the staged fp32 tile
constexpr size_t DMA_LDS = (size_t)D_STAGES * 2 * D_TILE * 2;  // 65,536 B: two blocks per compute unit
static_assert((size_t)DT * CLD * 4 <= DMA_LDS / 2, "C staging fits the operand stages");
static_assert(D_TILE / 8 == D_THREADS, "one 16-byte unit per thread, operand and step");

typedef __attribute__((address_space(3))) void lds_void;
typedef short d_i16x4 __attribute__((ext_vector_type(4)));

__device__ inline int dma_swz_mn(int k) { return ((k >> 1) & 1) << 2; }

// An operand's loads: one 16-byte unit per thread and step.
template <bool MN>
struct DmaOp {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t voff;   // byte offset of the unit at k = kbeg
  int kc;          // K-contiguous: first k (in the step) of the unit
  uint32_t kbytes;
  int kbeg, kend;
  __device__ inline void init(const bf16_t* p, int64_t ld, int R, int kbeg_, int kend_, int r0) {
    kbeg = kbeg_;
    kend = kend_;
    int64_t last;
    if (MN) last = kend > 0 ? (int64_t)(kend - 1) * ld + ((R + 7) & ~7) : 0;
    else last = R > 0 ? (int64_t)(R - 1) * ld + ((kend + 7) & ~7) : 0;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), (short)0, (int)(uint32_t)(last * 2),
                                           BUF_RSRC_WORD3);
    kbytes = MN ? (uint32_t)(ld * 2) : 2u;
    const int u = threadIdx.x;  // LDS unit
    if (MN) {
      const int k = u >> 3, c = (u & 7) ^ dma_swz_mn(k);
      voff = (uint32_t)(((int64_t)(kbeg + k) * ld + r0 + c * 8) * 2);
      kc = 0;
    } else {
      const int r = u >> 3, c = (u & 7) ^ ((r >> 1) & 7);
      voff = r0 + r < R ? (uint32_t)(((int64_t)(r0 + r) * ld + kbeg + c * 8) * 2) : 0x80000000u;
      kc = c * 8;
    }
  }
  // the tile at k0 into the stage at S (the wave's 64 units at S + 512 w);
  // what lies past kend reads zero (of a K-contiguous operand whole units:
  // zero_tail() the rest)
  __device__ inline void issue(bf16_t* S, int k0, int w) const {
    const uint32_t d = (uint32_t)(k0 - kbeg) * kbytes;
    const uint32_t o = MN || k0 + kc < kend ? voff + d : 0x80000000u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(S + w * 512), 16, (int)o, 0, 0, 0);
  }
};

// K-contiguous tile whose range ends inside a unit: the unit's elements past
// it (padding of the rows, or other data) become zeros.  klast: k of the
// range's end inside the step, not a multiple of 8.
__device__ inline void zero_tail(bf16_t* S, int klast) {
  const int r = threadIdx.x;
  if (r < DT) {
    bf16_t* p = S + r * DK + (((klast >> 3) ^ ((r >> 1) & 7)) << 3);
    for (int e = klast & 7; e < 8; ++e) p[e] = 0;
  }
}

// Operands whose rows start on any element (odd widths), whose units the LDS
// loads cannot take: the same units of the same layout through registers, by
// 16-byte loads from any address, two steps ahead.  A unit that reaches past a
// row's end is read from the row's last 8 elements and shifted into place at
// the LDS store (its length is at least 8); what lies past kend becomes zeros
// (kend is K or a multiple of 64); rows past R feed outputs that are never
// written.  An MLP of 415 -> 512 -> 8 over 2048 samples, forward and backward,
// whose W rows are such: 85 us with 128 x 128 tiles, 60 with these.
typedef uint32_t d_u32x4 __attribute__((ext_vector_type(4), aligned(2)));
template <bool MN>
struct RegOp {
  const bf16_t* p;  // MN: the unit at k = 0; K-contiguous: its row
  int64_t ld;
  u32x4 x[2];
  int kc, sh, K, kend;
  __device__ inline void init(const bf16_t* base, int64_t ld_, int R, int K_, int kend_, int r0) {
    ld = ld_;
    K = K_;
    kend = kend_;
    const int u = threadIdx.x, q = u >> 3;
    if (MN) {
      const int r = r0 + (((u & 7) ^ dma_swz_mn(q)) << 3);
      const int rr = r >= R ? 0 : (r + 8 > R ? R - 8 : r);
      sh = r >= R ? 0 : r - rr;
      kc = q;
      p = base + rr;
    } else {
      kc = ((u & 7) ^ ((q >> 1) & 7)) << 3;
      sh = 0;
      p = base + (int64_t)(r0 + q < R ? r0 + q : R - 1) * ld;
    }
  }
  __device__ inline int at(int k) const { return k + 8 > K ? K - 8 : k; }
  // a step past the range reads valid elements (k = 0) and is not used
  template <int SLOT>
  __device__ inline void load(int k0) {
    const int k = k0 + kc;
    const bf16_t* g = MN ? p + (k < kend ? (int64_t)k * ld : 0) : p + (k < kend ? at(k) : 0);
    x[SLOT] = *reinterpret_cast<const d_u32x4*>(g);
  }
  template <int SLOT>
  __device__ inline void store(bf16_t* S, int k0) const {
    const int k = k0 + kc;
    const int n = MN ? sh : (k < kend ? k - at(k) : 0);
    u32x4 v = __builtin_bit_cast(u32x4, __builtin_bit_cast(unsigned __int128, x[SLOT]) >> (16 * n));
    if (k >= kend) v = u32x4{0u, 0u, 0u, 0u};
    *reinterpret_cast<u32x4*>(S + threadIdx.x * 8) = v;
  }
};

// MFMA operand fragment: 32 rows from rbase, 16 k from ks (lane: row lane % 32,
// k 8 (lane / 32) .. + 7)
template <bool MN>
__device__ inline bf16x8 dma_frag(const bf16_t* S, int rbase, int ks, int lane) {
  if (!MN) {
    const int r = rbase + (lane & 31);
    const int x = (((lane >> 5) ^ ((r >> 1) & 7)) << 3) ^ ks;
    return *reinterpret_cast<const bf16x8*>(S + r * DK + x);
  }
  // within each 16-lane group a transposed read returns to lane j, as its
  // element e, element j % 4 of the 8-byte piece addressed by lane 4e + j / 4
  const int g = lane >> 4, j = lane & 15;
  const int r = rbase + 16 * (g & 1) + 4 * (j & 3);
  const int k = ks + 8 * (g >> 1) + (j >> 2);
  typedef __attribute__((address_space(3))) d_i16x4 lds_v4;
  auto at = [&](int kk) {
    return (lds_v4*)(S + kk * DT + ((((r >> 3) ^ dma_swz_mn(kk))) << 3) + (r & 7));
  };
  const d_i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(at(k));
  const d_i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(at(k + 4));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// grid: x = M tiles * N tiles (renumbered per XCD), z = split.  rowsum (TA
// only): rowsum[m] = sum over k of A(m, k), by the blocks of the first N tile;
// with split-K each split's sum goes to rs_partial[split][m].
template <bool TA, bool TB, typename CT, bool REG>
__global__ __launch_bounds__(D_THREADS, 4) void gemm_dma_kernel(
    const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ Bm, int64_t ldb, CT* __restrict__ C,
    int64_t ldc, int M, int N, int K, int k_per_split, float* __restrict__ partial, Epi epi, int vec,
    float* __restrict__ rowsum, float* __restrict__ rs_partial) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
  bf16_t* smem = reinterpret_cast<bf16_t*>(gemm_smem);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = w >> 2, wm = (w >> 1) & 1, wn = w & 1;
  const int tiles_n = (N + DT - 1) / DT;
  const int tile = xcd_block(blockIdx.x, gridDim.x);
  const int m0 = (tile / tiles_n) * DT, n0 = (tile % tiles_n) * DT;
  const int kbeg = blockIdx.z * k_per_split;
  const int kend = min(K, kbeg + k_per_split);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  const int steps = kend > kbeg ? (kend - kbeg + DK - 1) / DK : 0;
  // row sums of an M-contiguous A: thread = 8 rows of one k of the step
  const bool rs_on = TA && rowsum != nullptr && n0 == 0;
  float rs[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) rs[e] = 0.f;
  auto mma = [&](const bf16_t* As) {
    const bf16_t* Bs = As + D_TILE;
#pragma unroll
    for (int k = 0; k < DK / 2; k += 16) {
      const int ks = kg * (DK / 2) + k;
      const bf16x8 a = dma_frag<TA>(As, wm * 32, ks, lane), b = dma_frag<TB>(Bs, wn * 32, ks, lane);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
    if constexpr (TA) {
      if (rs_on) {
        const int k = threadIdx.x >> 3;
        float v[8];
        Vec16<bf16_t>::unpack(
            *reinterpret_cast<const u32x4*>(As + k * DT + (((threadIdx.x & 7) ^ dma_swz_mn(k)) << 3)), v);
#pragma unroll
        for (int e = 0; e < 8; ++e) rs[e] += v[e];
      }
    }
  };
  if constexpr (REG) {
    // step t in LDS stage t % 2 and, before that, register slot t % 2
    RegOp<TA> oa;
    RegOp<TB> ob;
    oa.init(A, lda, M, K, kend, m0);
    ob.init(Bm, ldb, N, K, kend, n0);
    bf16_t* S1 = smem + 2 * D_TILE;
    if (steps > 0) {
      oa.template load<0>(kbeg);
      ob.template load<0>(kbeg);
      oa.template load<1>(kbeg + DK);
      ob.template load<1>(kbeg + DK);
      oa.template store<0>(smem, kbeg);
      ob.template store<0>(smem + D_TILE, kbeg);
      oa.template load<0>(kbeg + 2 * DK);
      ob.template load<0>(kbeg + 2 * DK);
    }
    __syncthreads();
#pragma unroll 1
    for (int t = 0; t < steps; t += 2) {
      const int k0 = kbeg + t * DK;
      mma(smem);
      oa.template store<1>(S1, k0 + DK);
      ob.template store<1>(S1 + D_TILE, k0 + DK);
      oa.template load<1>(k0 + 3 * DK);
      ob.template load<1>(k0 + 3 * DK);
      __syncthreads();
      if (t + 1 == steps) break;  // uniform
      mma(S1);
      oa.template store<0>(smem, k0 + 2 * DK);
      ob.template store<0>(smem + D_TILE, k0 + 2 * DK);
      oa.template load<0>(k0 + 4 * DK);
      ob.template load<0>(k0 + 4 * DK);
      __syncthreads();
    }
  } else {
    DmaOp<TA> oa;
    DmaOp<TB> ob;
    oa.init(A, lda, M, kbeg, kend, m0);
    ob.init(Bm, ldb, N, kbeg, kend, n0);
    auto issue = [&](int t) {
      bf16_t* S = smem + (t & (D_STAGES - 1)) * 2 * D_TILE;
      oa.issue(S, kbeg + t * DK, w);
      ob.issue(S + D_TILE, kbeg + t * DK, w);
    };
#pragma unroll
    for (int t = 0; t < D_STAGES - 1; ++t) issue(t);
#pragma unroll 1
    for (int t = 0; t < steps; ++t) {
      // this wave's two loads of step t have landed (those of the two steps
      // after it may be in flight) and its LDS reads of step t - 1 returned; past
      // the barrier everybody's have, so the new loads may overwrite that stage
      static_assert(D_STAGES == 4, "the count below");
      asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      bf16_t* As = smem + (t & (D_STAGES - 1)) * 2 * D_TILE;
      if ((!TA || !TB) && t == steps - 1 && ((kend - kbeg) & 7) != 0) {  // uniform
        const int klast = kend - kbeg - t * DK;
        if (!TA) zero_tail(As, klast);
        if (!TB) zero_tail(As + D_TILE, klast);
        __syncthreads();
      }
      issue(t + D_STAGES - 1);
      mma(As);
    }
    // the loads issued past the last step write LDS: none may be in flight when
    // the epilogue reuses it
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
  float* Cs = reinterpret_cast<float*>(gemm_smem);
  if constexpr (TA) {
    if (rs_on) {
      // the 64 k classes of each row added in class order
#pragma unroll
      for (int e = 0; e < 8; ++e) Cs[(threadIdx.x >> 3) * DT + (threadIdx.x & 7) * 8 + e] = rs[e];
      __syncthreads();
      const int row = m0 + threadIdx.x;
      if (threadIdx.x < DT && row < M) {
        float s = 0.f;
        for (int c = 0; c < DK; ++c) s += Cs[c * DT + threadIdx.x];
        if (rs_partial) rs_partial[(int64_t)blockIdx.z * M + row] = s;
        else rowsum[row] = s;
      }
      __syncthreads();
    }
  }
  // The fp32 tile through LDS, then its rows with 16-byte vectors.  A
  // fragment's lane holds column lane % 32, rows 8 (r / 4) + 4 (lane / 32) + r % 4.
  float* cw = Cs + (wm * 32 + 4 * (lane >> 5)) * CLD + wn * 32 + (lane & 31);
  if (kg == 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) cw[(8 * (r >> 2) + (r & 3)) * CLD] = acc[r];
  }
  __syncthreads();
  if (kg == 1) {
#pragma unroll
    for (int r = 0; r < 16; ++r) cw[(8 * (r >> 2) + (r & 3)) * CLD] += acc[r];
  }
  __syncthreads();
  const int rl = threadIdx.x >> 3, cl = (threadIdx.x & 7) * 8;
  const int row = m0 + rl, col = n0 + cl;
  if (row >= M || col >= N) return;
  float v[8];
  ld8f(Cs + rl * CLD + cl, v);
  if (partial) {
    float* pp = partial + ((int64_t)blockIdx.z * M + row) * N + col;
    if ((N & 3) == 0 && col + 8 <= N) {
      stg16(pp, Vec16<float>::pack(v));
      stg16(pp + 4, Vec16<float>::pack(v + 4));
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (col + e < N) pp[e] = v[e];
    }
  } else if (vec && col + 8 <= N) {
    epi_store8<CT>(C, ldc, row, col, v, epi, 0);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (col + e < N) epi_store<CT>(C, ldc, row, col + e, v[e], epi, 0);
  }
}

template <bool TA, bool TB, typename CT, bool REG>
static hipError_t dma_launch(const GemmArgs& g, const DmaLaunch& L, hipStream_t st) {
  auto kern = gemm_dma_kernel<TA, TB, CT, REG>;
  constexpr size_t lds = REG ? DMA_LDS / 2 : DMA_LDS;  // two stages, four
  static LdsLimit lim;
  LAT_HIP_CHECK(lds_limit(kern, lds, lim));
  const dim3 grid((unsigned)((int64_t)cdiv(g.N, DT) * cdiv(g.M, DT)), 1, L.splits);
  kern<<<grid, D_THREADS, lds, st>>>((const bf16_t*)g.A, g.lda, (const bf16_t*)g.B, g.ldb, (CT*)g.C, g.ldc, g.M,
                                         g.N, g.K, L.kps, L.partial, make_epi(g), L.vec, g.rowsum, L.rs_partial);
  LAT_LAUNCH_CHECK();
  return hipSuccess;
}

template <typename CT, bool REG>
static hipError_t dma_ct(const GemmArgs& g, const DmaLaunch& L, hipStream_t st) {
  if (!g.ta && !g.tb) return dma_launch<false, false, CT, REG>(g, L, st);
  if (!g.ta) return dma_launch<false, true, CT, REG>(g, L, st);
  if (!g.tb) return dma_launch<true, false, CT, REG>(g, L, st);
  return dma_launch<true, true, CT, REG>(g, L, st);
}

hipError_t gemm_dma(const GemmArgs& g, const DmaLaunch& L, hipStream_t st) {
  if (L.reg) return g.c_dt == DT_BF16 ? dma_ct<bf16_t, true>(g, L, st) : dma_ct<float, true>(g, L, st);
  return g.c_dt == DT_BF16 ? dma_ct<bf16_t, false>(g, L, st) : dma_ct<float, false>(g, L, st);
}

}  // namespace lat
