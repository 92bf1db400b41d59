// Dot-product interaction on bf16 MFMA (v_mfma_f32_32x32x16_bf16), forward
// and backward, for n <= 128 vectors and d in {64, 128}: the pairwise inner
// products of a sample's vectors, strict upper triangle packed row by row
// (Section 3.3.2; the DLRM-style baseline of Section 4).
//
// Each block of 4 waves loops over samples; a sample's X [n, d] is loaded
// one sample ahead into registers (the next sample's loads are in flight
// while the current one is computed).
//   forward : X staged row-major; the 32x32 tiles on or above the diagonal of
//             X X^T are computed, the pairs i < j rounded to bf16 into a
//             packed LDS row, which is then written out with 16-byte stores.
//   backward: dX = S X is one contraction over j, where S is the symmetric
//             gradient matrix (S[i][j] = S[j][i] = g of the pair, zero
//             diagonal), of which LDS holds the upper triangle.
// Accumulation is fp32; the pair values and dX are rounded to bf16 once,
// where they are stored.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_tile.h"

namespace lat {

constexpr int DOT_THREADS = 256;
constexpr int DOT_BLOCKS = 512;
constexpr int DOT_MASK_WORDS = 4;  // slot bitmask words per sample (n <= 128)

// first packed position of row i (pairs (i, i+1) .. (i, n-1))
__device__ inline int pair_start(int i, int n) { return i * n - i * (i + 1) / 2; }

typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));  // X rows: 4-byte aligned

// The forward is bound by memory latency: a sample's read, products and write
// follow one another, so what counts is how many samples a compute unit has in
// flight.  LDS therefore holds only the n rows and the packed pairs (lanes of a
// tile's rows past n read row n - 1; their products are not kept), and X moves
// in 16-byte vectors: n = 97, d = 128 takes 36 KB, four blocks per compute
// unit, where tiles padded to 128 rows took 51 KB and 4-byte loads (two blocks:
// 100 us for 8192 samples, now 70).
template <int NP, int D>
__global__ __launch_bounds__(DOT_THREADS, 4) void dot_fwd_mfma_kernel(const bf16_t* __restrict__ X,
                                                                      int B, int n,
                                                                      bf16_t* __restrict__ out,
                                                                      int64_t ostride, int emit0) {
  constexpr int LX = D + 8;
  constexpr int PER = (NP * D / 8 + DOT_THREADS - 1) / DOT_THREADS;  // vectors per thread
  extern __shared__ __attribute__((aligned(16))) bf16_t dot_smem[];
  bf16_t* Xs = dot_smem;            // [n][LX]
  bf16_t* Zp = dot_smem + n * LX;   // packed pairs (n * LX * 2 is a multiple of 16)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int P = n * (n - 1) / 2, nd = n * D;
  const int off = emit0 ? D : 0;
  const int TT = (n + 31) / 32, ZT = TT * (TT + 1) / 2;  // tiles on or above the diagonal
  u32x4 x[PER];
  auto load = [&](int b) {
    const bf16_t* g = X + (int64_t)b * nd;
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (q * DOT_THREADS * 8 < nd) {  // uniform
        const int e = (threadIdx.x + q * DOT_THREADS) * 8;
        x[q] = *reinterpret_cast<const u32x4_a4*>(g + (e < nd ? e : 0));
      }
  };
  load(blockIdx.x);
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = (threadIdx.x + q * DOT_THREADS) * 8;
      if (e < nd) *reinterpret_cast<u32x4*>(Xs + (e / D) * LX + e % D) = x[q];
    }
    __syncthreads();
    if (b + (int)gridDim.x < B) load(b + gridDim.x);
    for (int t = w; t < ZT; t += DOT_THREADS / 64) {
      int ti = 0, rem = t;
      while (rem >= TT - ti) {
        rem -= TT - ti;
        ++ti;
      }
      const int tj = ti + rem;
      const int j = tj * 32 + (lane & 31), ri = ti * 32 + (lane & 31);
      const bf16_t* pa = Xs + (ri < n ? ri : n - 1) * LX + (lane >> 5) * 8;
      const bf16_t* pb = Xs + (j < n ? j : n - 1) * LX + (lane >> 5) * 8;
      f32x16 acc;
      zero16(acc);
#pragma unroll
      for (int k = 0; k < D; k += 16)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(pa + k),
                                                      *reinterpret_cast<const bf16x8*>(pb + k), acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = ti * 32 + frag_row(r);
        if (i < j && j < n) Zp[pair_start(i, n) + (j - i - 1)] = f2bf(acc[r]);
      }
    }
    __syncthreads();
    bf16_t* ob = out + (int64_t)b * ostride;
    if (emit0)
      for (int a = threadIdx.x; a < D; a += DOT_THREADS) ob[a] = Xs[a];
    bf16_t* dst = ob + off;
    int done = 0;
    if ((reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
      const int nv = P / 8;
      for (int v = threadIdx.x; v < nv; v += DOT_THREADS)
        *reinterpret_cast<u32x4*>(dst + v * 8) = *reinterpret_cast<const u32x4*>(Zp + v * 8);
      done = nv * 8;
    }
    for (int m = done + threadIdx.x; m < P; m += DOT_THREADS) dst[m] = Zp[m];
    __syncthreads();  // Xs and Zp are rewritten for the next sample
  }
}

// The backward.  The symmetric gradient matrix S is kept as its strict upper
// triangle U (U[i][j] = g of the pair i < j, zeros elsewhere), written once per
// pair; a 32 x 16 piece of S comes from U's rows right of the diagonal, from
// U's columns (transposed LDS reads) left of it, and from both, their bits
// joined, on it.  X stays as it is in memory ([n][D], 16-byte vectors) and is
// read by columns.  So X and the pairs take n rows each in LDS (50 KB at
// n = 97, d = 128: three blocks per compute unit; with X transposed, both
// triangles of S and a patch for the output it was 80 KB and two), and both are
// loaded a sample ahead.  Wave w takes rows 32 ti .. of dX, its pieces of S in
// registers, computed as dX^T = X^T S so that a lane holds neighbouring columns
// of one row, which exchanges between lanes make 64-byte segments of dX.
//
// Bound by memory traffic (4.5 to 5 TB/s), short batches by latency.  8192
// samples, d = 128: n = 97 130 -> 108 us, 65 75 -> 64, 27 37.6 -> 26.5 (96 and
// 64, whole tiles: 97 -> 98 and 60.6 -> 59.6); d = 64, n = 27: 21.9 -> 12.9;
// 512 samples of n = 97: 16.4 -> 12.2.
//
// LDS units (16 bytes) are permuted within their rows so that neither kind of
// read has bank conflicts: 16 rows at one column, or 4 rows of 64 bytes.
template <int D>
__device__ inline int dot_swz_x(int k) {
  return D == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2;
}
template <int NS>
__device__ inline int dot_swz_u(int r) {
  const int lo = (r >> 2) & 3;
  return NS == 128 ? ((r & 3) << 2) | lo : (NS == 64 ? (((r >> 1) & 1) << 2) | lo : lo);
}

typedef short dot_i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) dot_i16x4 dot_lds_v4;

// MFMA operand of 32 columns from c0 and 16 rows k from ks of a row-major LDS
// matrix (lane: column lane % 32, k 8 (lane / 32) .. + 7), from the positions of its two halves.  Within each
// 16-lane group a transposed read returns to lane j, as its element e, element
// j % 4 of the 8-byte piece addressed by lane 4e + j / 4: a lane's pieces are
// columns c0 + dot_frag_c(lane) .. + 3 of rows ks + dot_frag_k(lane) and + 4.
__device__ inline int dot_frag_c(int lane) { return 16 * ((lane >> 4) & 1) + 4 * (lane & 3); }
__device__ inline int dot_frag_k(int lane) { return 8 * (lane >> 5) + ((lane & 15) >> 2); }
__device__ inline bf16x8 dot_frag_cols(const bf16_t* p0, const bf16_t* p4) {
  const dot_i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dot_lds_v4*)p0);
  const dot_i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((dot_lds_v4*)p4);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// row length of U in LDS
constexpr int dot_u_cols(int np) { return np <= 32 ? 32 : (np <= 64 ? 64 : 128); }
// blocks per compute unit that the registers allow (and about what the LDS holds)
constexpr int dot_bwd_blocks(int np) {
  return np <= 80 ? 4 : (np <= 112 ? 3 : 2);
}

template <int NP, int D>
__global__ __launch_bounds__(DOT_THREADS, dot_bwd_blocks(NP)) void dot_bwd_mfma_kernel(
    const bf16_t* __restrict__ X, int B, int n, const bf16_t* __restrict__ dout, int64_t dstride,
    int emit0, bf16_t* __restrict__ dX) {
  constexpr int NS = dot_u_cols(NP);
  constexpr int PER = (NP * D / 8 + DOT_THREADS - 1) / DOT_THREADS;  // X vectors per thread
  constexpr int PMAX = NP * (NP - 1) / 2;
  constexpr int Q = (PMAX + DOT_THREADS - 1) / DOT_THREADS;          // pairs per thread
  constexpr int KS = NP / 16, AB = D / 32;
  // n > NMIN: what is in range for every such n needs no check
  constexpr int NMIN = NP <= 32 ? 0 : (NP <= 64 ? 32 : NP - 16);
  constexpr int XFULL = (NMIN + 1) * D / (DOT_THREADS * 8), QFULL = (NMIN + 1) * NMIN / 2 / DOT_THREADS;
  extern __shared__ __attribute__((aligned(16))) bf16_t dot_smem[];
  const int nk = (n + 15) & ~15;
  bf16_t* Xs = dot_smem;              // [nk][D], rows past n zeros
  bf16_t* U = Xs + nk * D;            // [n][NS]
  bf16_t* G0 = U + n * NS;            // [D] gradient of the copied row 0
  const bool vec_dx = (reinterpret_cast<uintptr_t>(dX) & 15) == 0;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int P = n * (n - 1) / 2, nd = n * D;
  const int off = emit0 ? D : 0;
  for (int e = threadIdx.x * 8; e < n * NS; e += DOT_THREADS * 8)
    *reinterpret_cast<u32x4*>(U + e) = u32x4{0u, 0u, 0u, 0u};
  for (int e = nd + threadIdx.x * 8; e < nk * D; e += DOT_THREADS * 8)
    *reinterpret_cast<u32x4*>(Xs + e) = u32x4{0u, 0u, 0u, 0u};
  // this thread's pairs m = tid + q * THREADS as positions in U, two 16-bit
  // ones per register (the same for every sample): the row is the largest i
  // with pair_start(i) <= m
  uint32_t pos[(Q + 1) / 2];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int m = threadIdx.x + q * DOT_THREADS;
    uint32_t v = 0;
    if (q < QFULL || m < P) {
      // (the quadratic's root, exact integers under it: off by at most one)
      const float c = 2.f * n - 1.f;
      int i = (int)((c - sqrtf(fmaxf(c * c - 8.f * m, 0.f))) * 0.5f);
      i = i > n - 2 ? n - 2 : i;
      i -= pair_start(i, n) > m ? 1 : 0;
      i += i + 1 <= n - 2 && pair_start(i + 1, n) <= m ? 1 : 0;
      const int j = m - pair_start(i, n) + i + 1;
      v = (uint32_t)(i * NS + (((j >> 3) ^ dot_swz_u<NS>(i)) << 3) + (j & 7));
    }
    if (q % 2 == 0) pos[q / 2] = v;
    else pos[q / 2] |= v << 16;
  }
  u32x4 x[PER];
  uint32_t gv[Q], g0 = 0;
  // straight-line loads (a vector or pair past the last reads the first one
  // and is not used)
  auto load = [&](int b) {
    const bf16_t* gb = dout + (int64_t)b * dstride;
    const bf16_t* xb = X + (int64_t)b * nd;
    const bf16_t* gp = P > 0 ? gb + off : xb;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = (threadIdx.x + q * DOT_THREADS) * 8;
      x[q] = *reinterpret_cast<const u32x4_a4*>(xb + (q < XFULL || e < nd ? e : 0));
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int m = threadIdx.x + q * DOT_THREADS;
      gv[q] = gp[q < QFULL || m < P ? m : 0];
    }
    if (emit0) g0 = gb[threadIdx.x % D];
  };
  load(blockIdx.x);
  __syncthreads();
  // rows of dX and column blocks of this wave
  constexpr int TT = (NP + 31) / 32;
  constexpr int WI = TT <= 1 ? 1 : (TT == 2 ? 2 : 4), WA = 4 / WI;
  const int ti = w % WI, ab0 = w / WI;
  const int row = ti * 32 + (lane & 31);
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    const int e0 = threadIdx.x * 8, r0 = e0 / D;
    bf16_t* xd = Xs + r0 * D + (e0 % D ^ dot_swz_x<D>(r0) << 3);  // (the same 16 rows on)
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (q < XFULL || e0 + q * DOT_THREADS * 8 < nd) *reinterpret_cast<u32x4*>(xd + q * DOT_THREADS * 8) = x[q];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (q < QFULL || threadIdx.x + q * DOT_THREADS < P) U[(pos[q / 2] >> (16 * (q % 2))) & 0xffffu] = (bf16_t)gv[q];
    if (emit0 && threadIdx.x < D) G0[threadIdx.x] = (bf16_t)g0;
    __syncthreads();
    if (b + (int)gridDim.x < B) load(b + gridDim.x);
    if (ti * 32 < n) {  // uniform per wave
      bf16x8 s[KS], dg[2];
      const int fk = dot_frag_k(lane), cu = ti * 32 + dot_frag_c(lane);
      // position of U's columns cu .. cu + 3 at row r
      auto atu = [&](int r) { return r * NS + (((cu >> 3) ^ dot_swz_u<NS>(r)) << 3) + (cu & 7); };
      // (the permutation is the same 16 rows on)
      const bf16_t *u0 = U + atu(fk), *u4 = U + atu(fk + 4);
      const int ru = row < n ? row : n - 1;
      const bf16_t* up = U + ru * NS;
      int fu = (dot_swz_u<NS>(ru) ^ (lane >> 5)) << 3;
      asm volatile("" : "+v"(fu));  // the addresses are not kept in registers
#pragma unroll
      for (int k = 0; k < KS; ++k)
        if (k * 16 <= NMIN || k * 16 < n) {
          if (k / 2 < ti) s[k] = dot_frag_cols(u0 + k * 16 * NS, u4 + k * 16 * NS);
          else s[k] = *reinterpret_cast<const bf16x8*>(up + ((k * 16) ^ fu));
        }
      // rows past the last read row n - 1, which is all zeros
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = ti * 32 + h * 16 + fk;
        dg[h] = dot_frag_cols(U + atu(r < n ? r : n - 1), U + atu(r + 4 < n ? r + 4 : n - 1));
      }
#pragma unroll
      for (int k = 0; k < KS; ++k)
        if (k / 2 == ti)
          s[k] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, s[k]) | __builtin_bit_cast(u32x4, dg[k & 1]));
      bf16_t* dxr = dX + ((int64_t)b * n + ti * 32 + (lane & 15)) * D + ((lane >> 4) & 1) * 16 + (lane >> 5) * 8;
#pragma unroll 1
      for (int ab = ab0; ab < AB; ab += WA) {
        f32x16 acc;
        zero16(acc);
        const int cx = ab * 32 + dot_frag_c(lane);
        const bf16_t* px = Xs + fk * D + (cx ^ dot_swz_x<D>(fk) << 3);  // (the same 4 rows on)
#pragma unroll
        for (int k = 0; k < KS; ++k)
          if (k * 16 <= NMIN || k * 16 < n) {
            const bf16x8 xf = dot_frag_cols(px + k * 16 * D, px + (k * 16 + 4) * D);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, s[k], acc, 0, 0, 0);
          }
        if (emit0 && ti == 0 && lane % 32 == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[r] += bf2f(G0[ab * 32 + frag_row(r)]);
        }
        // registers 4q .. 4q + 3: columns 8q + 4 (lane / 32) .. + 3
        uint32_t p[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) p[q] = (uint32_t)f2bf(acc[2 * q]) | (uint32_t)f2bf(acc[2 * q + 1]) << 16;
        // Half waves exchange, so that a lane has 8 columns (those from 16 h + 8
        // (lane / 32)), then 16-lane groups, so that four lanes have a row's 32
        // (rows lane % 16 and 16 on): 64-byte row segments.
        u32x4 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const auto lo = __builtin_amdgcn_permlane32_swap(p[4 * h], p[4 * h + 2], false, false);
          const auto hi = __builtin_amdgcn_permlane32_swap(p[4 * h + 1], p[4 * h + 3], false, false);
          v[h] = u32x4{lo[0], hi[0], lo[1], hi[1]};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto t = __builtin_amdgcn_permlane16_swap(v[0][e], v[1][e], false, false);
          v[0][e] = t[0];
          v[1][e] = t[1];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (ti * 32 + h * 16 + (lane & 15) >= n) continue;
          bf16_t* d = dxr + h * 16 * D + ab * 32;
          if (vec_dx) stg16(d, v[h]);
          else
#pragma unroll
            for (int e = 0; e < 8; ++e) d[e] = (bf16_t)(v[h][e / 2] >> (16 * (e % 2)));
        }
      }
    }
    __syncthreads();  // Xs, U and G0 are rewritten for the next sample
  }
}

// ---------------------------------------------------------------------------
// Listed slots only (forward).  A per-sample bitmask of DOT_MASK_WORDS
// words (bit s of word s / 32: slot s may be non-zero; bits at or past n are
// ignored) lets the forward work on the listed slots: the caller guarantees
// that every unlisted slot holds a zero vector (absent features are
// zero-padded, Section 3.2), so a pair touching one is exactly 0.  With na
// listed slots (row r of the compact matrix = the r-th listed slot,
// ascending) the listed rows are staged compactly, only the tiles on or above
// the diagonal of the compact Gram matrix are computed (for n = 97 with 42
// listed: 3 tiles instead of 10), and the pairs are scattered into the
// zero-filled packed row; the results equal the full kernel's.  The lists of
// the next sample are built in LDS one iteration ahead, so the prefetch of
// its rows reads its slots from there, and its mask words are loaded one
// more iteration ahead.  (A backward over the listed slots, S [n, na] times
// the compact X, measured slower than the full backward: 156 against 121 us
// at n = 97 with 42 listed, so the backward always runs over every slot.)
struct SlotMask {
  uint32_t m[DOT_MASK_WORDS];
  int na;
};

// sample b's mask words, as a vector load (issued with the row prefetch and
// counted in order with it; a scalar load would be waited for at the next
// barrier).  The offset is a zero held in a vector register the compiler
// cannot see through, so the address stays per lane.
__device__ inline u32x4 slot_mask_load(const uint32_t* __restrict__ mask, int b) {
  int z;
  asm volatile("v_mov_b32 %0, 0" : "=v"(z));
  return *reinterpret_cast<const u32x4*>(mask + (int64_t)b * DOT_MASK_WORDS + z);
}

// the mask with the bits at or past n cleared, and its count
__device__ inline SlotMask slot_mask_of(const u32x4 raw, int n) {
  SlotMask sm;
  sm.na = 0;
#pragma unroll
  for (int w = 0; w < DOT_MASK_WORDS; ++w) {
    const int lim = n - 32 * w;
    const uint32_t valid = lim >= 32 ? 0xffffffffu : (lim <= 0 ? 0u : (1u << lim) - 1u);
    sm.m[w] = raw[w] & valid;
    sm.na += __popc(sm.m[w]);
  }
  return sm;
}

// lst[r] = r-th listed slot (r < na).  Thread t handles slot t (t < n).
__device__ inline void slot_lists(const SlotMask& sm, int n, uint8_t* lst) {
  const int t = threadIdx.x;
  if (t >= n) return;
  const int w = t >> 5, bit = t & 31;
  uint32_t mw = sm.m[0];
  int below = 0;
#pragma unroll
  for (int k = 1; k < DOT_MASK_WORDS; ++k)
    if (w >= k) {
      below += __popc(mw);
      mw = sm.m[k];
    }
  const bool on = (mw >> bit) & 1u;
  const int r = below + __popc(mw & ((1u << bit) - 1u));
  if (on) lst[r] = (uint8_t)t;
}

// Stager over the listed rows: compact row r reads slot lst[r] of the
// sample (r < na), rows past na read slot 0 and are stored as zeros.
template <int RP, int COLS, int THREADS>
struct ListStager {
  static constexpr int ITEMS = (RP / 8) * (COLS / 2);
  static constexpr int PER = (ITEMS + THREADS - 1) / THREADS;
  uint32_t v[PER][8];
  __device__ inline void load(const bf16_t* __restrict__ g, const uint8_t* lst, int na) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      int it = threadIdx.x + q * THREADS;
      it = it < ITEMS ? it : ITEMS - 1;
      const int j0 = (it / (COLS / 2)) * 8, c = (it % (COLS / 2)) * 2;
      const uint2 sl = *reinterpret_cast<const uint2*>(lst + j0);  // 8 slots
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t word = i < 4 ? sl.x : sl.y;
        const int slot = j0 + i < na ? (int)((word >> (8 * (i & 3))) & 0xffu) : 0;
        v[q][i] = *reinterpret_cast<const uint32_t*>(g + (int64_t)slot * COLS + c);
      }
    }
  }
  __device__ inline void store(bf16_t* R, int ldr, bf16_t* T, int ldt, int na) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int it = threadIdx.x + q * THREADS;
      if (it < ITEMS) {
        const int j0 = (it / (COLS / 2)) * 8, c = (it % (COLS / 2)) * 2;
        uint32_t x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = j0 + i < na ? v[q][i] : 0u;
        if (R)
#pragma unroll
          for (int i = 0; i < 8; ++i) *reinterpret_cast<uint32_t*>(R + (j0 + i) * ldr + c) = x[i];
        if (!T) continue;
        u32x4 lo, hi;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          lo[i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x05040100u);
          hi[i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x07060302u);
        }
        *reinterpret_cast<u32x4*>(T + c * ldt + j0) = lo;
        *reinterpret_cast<u32x4*>(T + (c + 1) * ldt + j0) = hi;
      }
    }
  }
};

template <int NP, int D>
__global__ __launch_bounds__(DOT_THREADS) void dot_fwd_listed_kernel(const bf16_t* __restrict__ X,
                                                                     int B, int n,
                                                                     const uint32_t* __restrict__ mask,
                                                                     bf16_t* __restrict__ out,
                                                                     int64_t ostride, int emit0) {
  constexpr int LX = D + 8;
  constexpr int PMAX = NP * (NP - 1) / 2;
  __shared__ __attribute__((aligned(16))) bf16_t Xs[NP * LX];
  __shared__ __attribute__((aligned(16))) bf16_t Zp[(PMAX + 7) / 8 * 8];
  __shared__ __attribute__((aligned(16))) uint8_t lst[2][NP];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int P = n * (n - 1) / 2;
  const int off = emit0 ? D : 0;
  ListStager<NP, D, DOT_THREADS> sx;
  const int G = (int)gridDim.x;
  int na_next = 0;
  u32x4 mraw = {0u, 0u, 0u, 0u};  // mask words of the sample after the next
  if (blockIdx.x < B) {
    const SlotMask sm = slot_mask_of(slot_mask_load(mask, blockIdx.x), n);
    slot_lists(sm, n, lst[0]);
    na_next = sm.na;
  }
  if (blockIdx.x + G < B) mraw = slot_mask_load(mask, blockIdx.x + G);
  __syncthreads();
  if (blockIdx.x < B) sx.load(X + (int64_t)blockIdx.x * n * D, lst[0], na_next);
  int cur = 0;
  for (int b = blockIdx.x; b < B; b += G, cur ^= 1) {
    const int na = na_next;
    const int nb = b + G;
    sx.store(Xs, LX, nullptr, 0, na);
    for (int v = threadIdx.x; v < (P + 7) / 8; v += DOT_THREADS)
      *reinterpret_cast<u32x4*>(Zp + v * 8) = u32x4{0u, 0u, 0u, 0u};
    if (nb < B) {
      const SlotMask sm = slot_mask_of(mraw, n);
      slot_lists(sm, n, lst[cur ^ 1]);
      na_next = sm.na;
    }
    __syncthreads();
    if (nb + G < B) mraw = slot_mask_load(mask, nb + G);
    if (nb < B) sx.load(X + (int64_t)nb * n * D, lst[cur ^ 1], na_next);
    const int TA = (na + 31) / 32;
    const int ZA = TA * (TA + 1) / 2;
    const uint8_t* L = lst[cur];
    for (int t = w; t < ZA; t += DOT_THREADS / 64) {
      int ti = 0, rem = t;
      while (rem >= TA - ti) {
        rem -= TA - ti;
        ++ti;
      }
      const int tj = ti + rem;
      f32x16 acc;
      zero16(acc);
      mfma_tile<D>(acc, Xs + ti * 32 * LX, LX, Xs + tj * 32 * LX, LX);
      const int rj = tj * 32 + (lane & 31);
      const int j = rj < na ? L[rj] : 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ri = ti * 32 + frag_row(r);
        if (ri < rj && rj < na) {
          const int i = L[ri];
          Zp[pair_start(i, n) + (j - i - 1)] = f2bf(acc[r]);
        }
      }
    }
    __syncthreads();
    bf16_t* ob = out + (int64_t)b * ostride;
    if (emit0)
      for (int a = threadIdx.x; a < D; a += DOT_THREADS) ob[a] = X[(int64_t)b * n * D + a];
    bf16_t* dst = ob + off;
    int done = 0;
    if ((reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
      const int nv = P / 8;
      for (int v = threadIdx.x; v < nv; v += DOT_THREADS)
        *reinterpret_cast<u32x4*>(dst + v * 8) = *reinterpret_cast<const u32x4*>(Zp + v * 8);
      done = nv * 8;
    }
    for (int m = done + threadIdx.x; m < P; m += DOT_THREADS) dst[m] = Zp[m];
    __syncthreads();  // Xs, Zp and this sample's list are rewritten next
  }
}

// Slot masks of a batch (feature-major bags): bit 0 when has0 (the dense
// vector), and bit first + f for every feature f whose bag is non-empty.
// Thread (word w, sample b) builds word w of sample b.
__global__ __launch_bounds__(256) void dot_slot_mask_kernel(const int32_t* __restrict__ offsets, int F,
                                                            int B, int first, int has0,
                                                            uint32_t* __restrict__ mask) {
  const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (tid >= (int64_t)DOT_MASK_WORDS * B) return;
  const int wd = (int)(tid / B), b = (int)(tid - (int64_t)wd * B);
  uint32_t m = (has0 && wd == 0) ? 1u : 0u;
  const int s0 = 32 * wd;
  const int f0 = max(0, s0 - first), cnt = min(F, s0 + 32 - first) - f0;
  if (cnt > 0) {
    // the word's (up to 32) bags: both ends of each loaded as straight-line
    // code from clamped positions, so all loads are in flight together
    int32_t lo[32], hi[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int64_t o = (int64_t)(f0 + min(k, cnt - 1)) * B + b;
      lo[k] = offsets[o];
      hi[k] = offsets[o + 1];
    }
#pragma unroll
    for (int k = 0; k < 32; ++k)
      if (k < cnt && hi[k] > lo[k]) m |= 1u << (first + f0 + k - s0);
  }
  mask[(int64_t)b * DOT_MASK_WORDS + wd] = m;
}

hipError_t dot_slot_mask(const int32_t* offsets, int F, int B, int first, int has0, uint32_t* mask,
                         hipStream_t s) {
  if (B == 0) return hipSuccess;
  if (first + F > DOT_MASK_WORDS * 32 || first < 0) {
    set_error("DOT slot mask: slots up to %d exceed %d", first + F, DOT_MASK_WORDS * 32);
    return hipErrorInvalidValue;
  }
  dot_slot_mask_kernel<<<cdiv((int64_t)DOT_MASK_WORDS * B, 256), 256, 0, s>>>(offsets, F, B, first, has0, mask);
  LAT_LAUNCH_CHECK();
  return hipSuccess;
}

bool dot_mfma_supported(int n, int d) { return n >= 1 && n <= 128 && (d == 64 || d == 128); }

// X rows and the packed pairs in whole 16-byte vectors
static size_t dot_fwd_lds(int n, int d) {
  return (size_t)n * (d + 8) * 2 + ((size_t)n * (n - 1) / 2 + 7) / 8 * 16;
}

static size_t dot_bwd_lds(int n, int np, int d) { return ((size_t)((n + 15) / 16 * 16 + 1) * d + (size_t)n * dot_u_cols(np)) * 2; }

template <int NP, int D>
static hipError_t dot_bwd_launch(const void* X, int B, int n, const void* dout, int64_t dstride, int emit0, void* dX,
                                 hipStream_t s) {
  auto kern = dot_bwd_mfma_kernel<NP, D>;
  const size_t lds = dot_bwd_lds(n, NP, D);
  static LdsLimit lim;
  LAT_HIP_CHECK(lds_limit(kern, dot_bwd_lds(NP, NP, D), lim));
  const int per = (int)std::min<size_t>(dot_bwd_blocks(NP), (size_t)160 * 1024 / lds);
  kern<<<B < 256 * per ? B : 256 * per, DOT_THREADS, lds, s>>>((const bf16_t*)X, B, n, (const bf16_t*)dout, dstride,
                                                               emit0, (bf16_t*)dX);
  LAT_LAUNCH_CHECK();
  return hipSuccess;
}

template <int NP, int D>
static hipError_t dot_fwd_launch(const void* X, int B, int n, void* out, int64_t ostride, int emit0,
                                 const uint32_t* mask, hipStream_t s) {
  if (mask) {
    const int blocks = B < DOT_BLOCKS ? B : DOT_BLOCKS;
    dot_fwd_listed_kernel<NP, D><<<blocks, DOT_THREADS, 0, s>>>((const bf16_t*)X, B, n, mask,
                                                               (bf16_t*)out, ostride, emit0);
  } else {
    // as many blocks as the LDS holds, at most 4 per compute unit (registers)
    const size_t lds = dot_fwd_lds(n, D);
    const int per = (int)std::min<size_t>(4, (size_t)160 * 1024 / lds);
    dot_fwd_mfma_kernel<NP, D><<<B < 256 * per ? B : 256 * per, DOT_THREADS, lds, s>>>(
        (const bf16_t*)X, B, n, (bf16_t*)out, ostride, emit0);
  }
  LAT_LAUNCH_CHECK();
  return hipSuccess;
}

hipError_t dot_mfma(bool fwd, const void* X, int B, int n, int d, void* out, int64_t ostride,
                    int emit0, const void* dout, int64_t dstride, void* dX, const uint32_t* mask,
                    hipStream_t s) {
  if (B == 0 && dot_mfma_supported(n, d)) return hipSuccess;
#define LAT_DOTM(NPV, DV)                                                                  \
  if (fwd && n <= NPV && d == DV) return dot_fwd_launch<NPV, DV>(X, B, n, out, ostride, emit0, mask, s);
  LAT_DOTM(32, 64) LAT_DOTM(64, 64) LAT_DOTM(96, 64) LAT_DOTM(128, 64)
  LAT_DOTM(32, 128) LAT_DOTM(64, 128) LAT_DOTM(96, 128) LAT_DOTM(128, 128)
#undef LAT_DOTM
#define LAT_DOTM(NPV, DV)                                                                  \
  if (!fwd && n <= NPV && d == DV) return dot_bwd_launch<NPV, DV>(X, B, n, dout, dstride, emit0, dX, s);
  LAT_DOTM(32, 64) LAT_DOTM(64, 64) LAT_DOTM(80, 64) LAT_DOTM(96, 64) LAT_DOTM(112, 64) LAT_DOTM(128, 64)
  LAT_DOTM(32, 128) LAT_DOTM(64, 128) LAT_DOTM(80, 128) LAT_DOTM(96, 128) LAT_DOTM(112, 128) LAT_DOTM(128, 128)
#undef LAT_DOTM
  set_error("DOT MFMA path: unsupported shape n=%d d=%d", n, d);
  return hipErrorInvalidValue;
}

}  // namespace lat
