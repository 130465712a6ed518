// Plan-time work: the vocabulary fold and weight packing.
//
// Candidate restriction (section 3.2) gathers, once per depth, the rows of the
// correction that the top-M candidates need.  Here the rows are model-only
// quantities, so they are computed once per plan for the whole vocabulary and
// every call just gathers them:
//   P[v] = W_ih E[v] + b_ih (+ b_hh on the r and z gates, which only ever
//          appear summed with it; GRU input projection of token v, 3*d_h)
//   U[v] = W_c^T E[v]         (so delta(v) = U[v] . S + c[v] = E[v] . (W_c S + b_c))
//   c[v] = E[v] . b_c
// This is one GEMM of the embedding table against the packed matrix
// [W_ih ; W_c^T] ([4 d_h, d_e], K = d_e contiguous).  bf16 weights run on the
// gfx950 bf16 MFMA (exact products, fp32 accumulation); fp32 weights on the fp32
// MFMA.  A one-shot call (dt_build_tree_once) folds the rows of its candidates
// only.
#include "dt_internal.h"

namespace dt {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kFoldThreads = 256;
constexpr int kLdsPad = 8;  // bf16 elements of padding per LDS row

// Tile of a GEMM block, one-dimensional grid: blocks are dealt to the XCDs
// round-robin, so the column tiles of a row tile are put on one XCD, one after
// the other, and its embedding rows are read into one L2 (not eight).
// With fewer rows than columns (by_col) it is the row tiles of a column tile that
// share an XCD: an L2 then reads its columns of the weights and all of the
// embedding rows, the smaller part (1,024 rows at d_e = 2560, d_h = 512: 6.6 MB
// instead of 11.2, 37.5 -> 32.5 us).
constexpr int kFoldXcds = 8;
struct FoldTile {
  int col, row;
};
__device__ inline FoldTile fold_tile(int ncol, int nrow, bool by_col) {
  const int xcd = blockIdx.x % kFoldXcds, i = blockIdx.x / kFoldXcds;
  if (by_col) return FoldTile{i / nrow * kFoldXcds + xcd, i % nrow};
  return FoldTile{i % ncol, i / ncol * kFoldXcds + xcd};
}
inline dim3 fold_grid(int ncol, int nrow, bool by_col) {
  const int in = by_col ? nrow : ncol, across = by_col ? ncol : nrow;  // (in: the tiles that share an XCD)
  return dim3((unsigned)in * ((across + kFoldXcds - 1) / kFoldXcds * kFoldXcds));
}

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM: block tile (WR*TI*32) x (WC*TJ*32), 4 waves as WR x WC.
// Bound by the LDS round trip of a K slice: the next slice's global loads are
// issued before the current one is multiplied, so only LDS stands between two
// slices.  151,936 rows at d_e = 4096, d_h = 512 (2.55 TFLOP): 6.9 ms with the
// loads in line, 4.1-4.3 ms (590-620 TFLOP/s) ahead and with a row tile kept on one
// XCD.
// cadd (nullable): c is also added to cadd[row].
// ---------------------------------------------------------------------------
template <int WR, int WC, int TI, int TJ, int BK>
__global__ __launch_bounds__(kFoldThreads) void fold_mfma_kernel(
    const uint16_t *__restrict__ emb, const int32_t *__restrict__ cand, int rows_total, int d_e,
    const uint16_t *__restrict__ wfold, int nf, int d_h, const float *__restrict__ b_ih,
    const float *__restrict__ b_c, float *__restrict__ P, float *__restrict__ U,
    float *__restrict__ cvec, float *__restrict__ cadd, bool by_col) {
  static_assert(WR * WC == 4, "4 waves");
  constexpr int BM = WR * TI * 32, BN = WC * TJ * 32;
  constexpr int LDW = BK + kLdsPad;
  constexpr int TPR = kFoldThreads / BM;  // threads per row of the E . b_c sums
  static_assert(TPR * BM == kFoldThreads && BK % (8 * TPR) == 0, "whole 16-byte segments per thread");
  __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDW];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LDW];
  __shared__ __attribute__((aligned(16))) float bcs[BK];
  __shared__ int32_t rowtok[BM];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / WC, wc = wave % WC;
  const FoldTile tile = fold_tile((nf + BN - 1) / BN, (rows_total + BM - 1) / BM, by_col);
  const int n0 = tile.col * BN, r0 = tile.row * BM;
  if (r0 >= rows_total || n0 >= nf) return;
  const bool do_c = tile.col == 0;  // the first column tile also computes c = E_c b_c

  for (int i = tid; i < BM; i += kFoldThreads) {
    const int r = r0 + i;
    rowtok[i] = (r < rows_total) ? (cand ? cand[r] : r) : -1;
  }
  __syncthreads();

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.0f;
  float cacc = 0.0f;  // c partial of row tid / TPR (do_c only)

  constexpr int SEGS = BK / 8;  // 16-byte segments per tile row
  constexpr int NA = BM * SEGS / kFoldThreads, NB = BN * SEGS / kFoldThreads;
  uint4 ra[NA], rb[NB];
  float rbc = 0.0f;
  auto load = [&](int k0) {  // gathered A rows, packed B rows
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int s = tid + q * kFoldThreads, row = s / SEGS, k = k0 + (s % SEGS) * 8;
      const int tok = rowtok[row];
      ra[q] = make_uint4(0, 0, 0, 0);
      if (tok >= 0 && k + 8 <= d_e) ra[q] = *reinterpret_cast<const uint4 *>(emb + (size_t)tok * d_e + k);
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int s = tid + q * kFoldThreads, row = s / SEGS, k = k0 + (s % SEGS) * 8;
      rb[q] = make_uint4(0, 0, 0, 0);
      if (n0 + row < nf && k + 8 <= d_e)
        rb[q] = *reinterpret_cast<const uint4 *>(wfold + (size_t)(n0 + row) * d_e + k);
    }
    if (do_c && tid < BK) rbc = k0 + tid < d_e ? b_c[k0 + tid] : 0.0f;
  };
  load(0);
  for (int k0 = 0; k0 < d_e; k0 += BK) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int s = tid + q * kFoldThreads;
      *reinterpret_cast<uint4 *>(&As[(s / SEGS) * LDW + (s % SEGS) * 8]) = ra[q];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int s = tid + q * kFoldThreads;
      *reinterpret_cast<uint4 *>(&Bs[(s / SEGS) * LDW + (s % SEGS) * 8]) = rb[q];
    }
    if (do_c && tid < BK) bcs[tid] = rbc;
    __syncthreads();
    if (k0 + BK < d_e) load(k0 + BK);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 a[TI], b[TJ];
      const int kk = ks * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int row = (wr * TI + i) * 32 + (lane & 31);
        a[i] = *reinterpret_cast<const bf16x8 *>(&As[row * LDW + kk]);
      }
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int col = (wc * TJ + j) * 32 + (lane & 31);
        b[j] = *reinterpret_cast<const bf16x8 *>(&Bs[col * LDW + kk]);
      }
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (do_c) {
      // TPR threads per row, each over its part of the K slice
      const int row = tid / TPR, q0 = (tid % TPR) * (BK / TPR);
      float s = 0.0f;
#pragma unroll
      for (int q = q0; q < q0 + BK / TPR; q += 8) {
        const uint4 v = *reinterpret_cast<const uint4 *>(&As[row * LDW + q]);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s += __uint_as_float(w[e] << 16) * bcs[q + 2 * e];
          s += __uint_as_float(w[e] & 0xFFFF0000u) * bcs[q + 2 * e + 1];
        }
      }
      cacc += s;
    }
    __syncthreads();
  }

  // epilogue: 32x32 MFMA output layout -- lane l, register q holds
  // row (q/4)*8 + (l/32)*4 + q%4, column l%32
#pragma unroll
  for (int i = 0; i < TI; ++i) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int col = n0 + (wc * TJ + j) * 32 + (lane & 31);
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int row = r0 + (wr * TI + i) * 32 + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3);
        if (row >= rows_total || col >= nf) continue;
        const float v = acc[i][j][q];
        if (col < 3 * d_h)
          P[(size_t)row * (3 * d_h) + col] = v + b_ih[col];
        else
          U[(size_t)row * d_h + (col - 3 * d_h)] = v;
      }
    }
  }
  if (do_c) {
    __shared__ float cpart[kFoldThreads];
    cpart[tid] = cacc;
    __syncthreads();
    for (int row = tid; row < BM; row += kFoldThreads) {
      const int r = r0 + row;
      if (r >= rows_total) continue;
      float c = cpart[TPR * row];
#pragma unroll
      for (int i = 1; i < TPR; ++i) c += cpart[TPR * row + i];
      cvec[r] = c;
      if (cadd) cadd[r] += c;
    }
  }
}

// ---------------------------------------------------------------------------
// fp32 weights: the same GEMM on the fp32 MFMA (32 x 32 x 2), 64 x 64 tiles,
// K slices of 32, the next slice's loads in flight.  Column nf is b_c: c = E b_c
// comes out of the same products.  32,003 rows at d_e = 1024, d_h = 256 (67
// GFLOP): 0.97 ms (69 TFLOP/s); one thread per output, reading its weight row
// alone, took 127 ms.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kFoldThreads) void fold_f32_kernel(
    const float *__restrict__ emb, const int32_t *__restrict__ cand, int rows_total, int d_e,
    const float *__restrict__ wfold, int nf, int d_h, const float *__restrict__ b_ih,
    const float *__restrict__ b_c, float *__restrict__ P, float *__restrict__ U, float *__restrict__ cvec,
    float *__restrict__ cadd, bool by_col) {
  constexpr int BM = 64, BN = 64, BK = 32, LDW = BK + 2;
  constexpr int NL = BM * BK / kFoldThreads;  // elements per thread and operand
  __shared__ float As[BM * LDW], Bs[BN * LDW];
  __shared__ int32_t rowtok[BM];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const FoldTile tile = fold_tile((nf + 1 + BN - 1) / BN, (rows_total + BM - 1) / BM, by_col);
  const int n0 = tile.col * BN, r0 = tile.row * BM;
  if (r0 >= rows_total || n0 > nf) return;
  if (tid < BM) rowtok[tid] = r0 + tid < rows_total ? (cand ? cand[r0 + tid] : r0 + tid) : -1;
  __syncthreads();
  f32x16 acc;
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
  float ra[NL], rb[NL];
  // (element e of a slice: row e / 32, column e % 32: a row's 32 floats are one line)
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int e = tid + q * kFoldThreads, row = e / BK, k = k0 + e % BK, n = n0 + row;
      const int tok = rowtok[row];
      ra[q] = (tok >= 0 && k < d_e) ? emb[(size_t)tok * d_e + k] : 0.0f;
      rb[q] = (n <= nf && k < d_e) ? (n < nf ? wfold[(size_t)n * d_e + k] : b_c[k]) : 0.0f;
    }
  };
  load(0);
  for (int k0 = 0; k0 < d_e; k0 += BK) {
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int e = tid + q * kFoldThreads;
      As[(e / BK) * LDW + e % BK] = ra[q];
      Bs[(e / BK) * LDW + e % BK] = rb[q];
    }
    __syncthreads();
    if (k0 + BK < d_e) load(k0 + BK);
    const float *ap = As + (wr * 32 + (lane & 31)) * LDW + (lane >> 5), *bp = Bs + (wc * 32 + (lane & 31)) * LDW + (lane >> 5);
#pragma unroll
    for (int k = 0; k < BK; k += 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ap[k], bp[k], acc, 0, 0, 0);
    __syncthreads();
  }
  const int col = n0 + wc * 32 + (lane & 31);
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int row = r0 + wr * 32 + (q >> 2) * 8 + (lane >> 5) * 4 + (q & 3);
    if (row >= rows_total || col > nf) continue;
    const float v = acc[q];
    if (col < 3 * d_h)
      P[(size_t)row * (3 * d_h) + col] = v + b_ih[col];
    else if (col < nf)
      U[(size_t)row * d_h + (col - 3 * d_h)] = v;
    else {
      cvec[row] = v;
      if (cadd) cadd[row] += v;
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 rows of a width the 16-byte loads do not take (d_e % 8 != 0)
// ---------------------------------------------------------------------------
template <typename TW>
__device__ inline float wval(const TW *p, size_t i);
template <>
__device__ inline float wval<uint16_t>(const uint16_t *p, size_t i) {
  return bf16_to_f32(p[i]);
}
template <>
__device__ inline float wval<float>(const float *p, size_t i) {
  return p[i];
}

template <typename TW>
__global__ __launch_bounds__(256) void fold_simple_kernel(
    const TW *__restrict__ emb, const int32_t *__restrict__ cand, int rows_total, int d_e,
    const TW *__restrict__ wfold, int nf, int d_h, const float *__restrict__ b_ih,
    const float *__restrict__ b_c, float *__restrict__ P, float *__restrict__ U,
    float *__restrict__ cvec, float *__restrict__ cadd) {
  // one block per candidate row; threads over the nf+1 outputs
  const int r = blockIdx.x;
  if (r >= rows_total) return;
  const int tok = cand ? cand[r] : r;
  for (int n = threadIdx.x; n <= nf; n += blockDim.x) {
    float s = 0.0f;
    if (tok >= 0) {
      if (n < nf) {
        for (int k = 0; k < d_e; ++k)
          s += wval<TW>(emb, (size_t)tok * d_e + k) * wval<TW>(wfold, (size_t)n * d_e + k);
      } else if (b_c != nullptr) {
        for (int k = 0; k < d_e; ++k) s += wval<TW>(emb, (size_t)tok * d_e + k) * b_c[k];
      }
    }
    if (n < 3 * d_h)
      P[(size_t)r * (3 * d_h) + n] = s + b_ih[n];
    else if (n < nf)
      U[(size_t)r * d_h + (n - 3 * d_h)] = s;
    else {
      cvec[r] = s;
      if (cadd) cadd[r] += s;
    }
  }
}

// ---------------------------------------------------------------------------
// plan-time packing
// ---------------------------------------------------------------------------
// One launch packs everything: a one-shot call runs it each time, and is bound by
// the latency of its few loads (13 MB at d_e = 2560, d_h = 512, 3 us at the
// memory's rate), so every thread has its 16-byte loads in flight together and
// the parts run side by side: 8.6 us (three launches with loads of one element:
// 13.4 + 4.3 + 3.6 us and two gaps).
//   blocks [0, whh)       W_hh in MFMA A-fragment order for the expansion kernels:
//     bf16 (16x16x32 MFMA): fragment (u, g, ks) is 64 lanes x 8 bf16; lane l holds
//       W_hh[g*d_h + 16u + l%16][ks*32 + (l/16)*8 + e], e = 0..7;
//     fp32 (16x16x4 MFMA, four per k-group of 16): fragment (u, g, q) is 64 lanes x
//       4 floats; lane l holds W_hh[g*d_h + 16u + l%16][16q + (l/16)*4 + e];
//     either way 16 bytes a lane, and one k group of 64 bytes a fragment
//   blocks [whh, bias)    b_ih (plus b_hh on the gates r and z), b_hh and b_c in
//     fp32; missing ones are zeros
//   blocks [bias, ih)     [W_ih; W_c^T] as rows of K = d_e: W_ih is copied ...
//   blocks [ih, ...)      ... W_c transposed through LDS in 64 x 64 tiles, and the
//     rows past 4 d_h zeros
struct PackArgs {
  const void *w_ih, *w_hh, *w_c, *b_ih, *b_hh, *b_c;
  void *wfold, *whh;
  float *o_ih, *o_hh, *o_c;
  int d_e, d_h, nf_pad;
  int whh_end, bias_end, ih_end;
};
constexpr int kPackThreads = 256;
constexpr int kPackVecs = 4;  // 16-byte loads a thread has in flight

template <typename TW>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(PackArgs a) {
  constexpr int E = 16 / sizeof(TW);
  // 16 bytes at the elements' own alignment (the callers' weights need no more)
  typedef TW Vec __attribute__((ext_vector_type(E), aligned(sizeof(TW))));
  const int tid = threadIdx.x, blk = blockIdx.x, d_e = a.d_e, d_h = a.d_h;
  if (blk < a.whh_end) {
    const TW *in = static_cast<const TW *>(a.w_hh);
    TW *out = static_cast<TW *>(a.whh);
    const int nk = d_h / (4 * E), total = 3 * d_h * d_h / E;
    Vec v[kPackVecs];
#pragma unroll
    for (int q = 0; q < kPackVecs; ++q) {
      const int i = (blk * kPackVecs + q) * kPackThreads + tid;
      if (i >= total) continue;
      const int l = i & 63, frag = i >> 6, k = frag % nk, g = frag / nk % 3, u = frag / nk / 3;
      v[q] = *reinterpret_cast<const Vec *>(in + (size_t)(g * d_h + 16 * u + (l & 15)) * d_h + k * 4 * E + (l >> 4) * E);
    }
#pragma unroll
    for (int q = 0; q < kPackVecs; ++q) {
      const int i = (blk * kPackVecs + q) * kPackThreads + tid;
      if (i < total) *reinterpret_cast<Vec *>(out + (size_t)i * E) = v[q];
    }
  } else if (blk < a.bias_end) {
    const int i = (blk - a.whh_end) * kPackThreads + tid;
    const TW *b_ih = static_cast<const TW *>(a.b_ih), *b_hh = static_cast<const TW *>(a.b_hh),
             *b_c = static_cast<const TW *>(a.b_c);
    if (i < 3 * d_h) {
      const float h = b_hh ? wval<TW>(b_hh, i) : 0.0f, x = b_ih ? wval<TW>(b_ih, i) : 0.0f;
      a.o_hh[i] = h;
      a.o_ih[i] = i < 2 * d_h ? x + h : x;
    }
    if (i < d_e) a.o_c[i] = b_c ? wval<TW>(b_c, i) : 0.0f;
  } else if (blk < a.ih_end) {
    const TW *in = static_cast<const TW *>(a.w_ih);
    TW *out = static_cast<TW *>(a.wfold);
    const int total = 3 * d_h * d_e / E;  // (whole vectors: d_h % 32 == 0)
    Vec v[kPackVecs];
#pragma unroll
    for (int q = 0; q < kPackVecs; ++q) {
      const int i = ((blk - a.bias_end) * kPackVecs + q) * kPackThreads + tid;
      if (i < total) v[q] = *reinterpret_cast<const Vec *>(in + (size_t)i * E);
    }
#pragma unroll
    for (int q = 0; q < kPackVecs; ++q) {
      const int i = ((blk - a.bias_end) * kPackVecs + q) * kPackThreads + tid;
      if (i < total) *reinterpret_cast<Vec *>(out + (size_t)i * E) = v[q];
    }
  } else {
    constexpr int VR = 64 / E, NV = 64 * VR / kPackThreads;  // vectors per tile row, per thread
    __shared__ TW tile[64][64 + 4 / sizeof(TW)];             // (a dword of padding: rows on other banks)
    const TW *in = static_cast<const TW *>(a.w_c);
    TW *out = static_cast<TW *>(a.wfold);
    const int ncol = (d_e + 63) / 64, t = blk - a.ih_end, k0 = t % ncol * 64, n0 = t / ncol * 64;
    Vec v[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {  // W_c row k, columns n .. n + E - 1 (all in or out: d_h % 32 == 0)
      const int i = q * kPackThreads + tid, k = k0 + i / VR, n = n0 + i % VR * E;
      v[q] = Vec(TW(0));
      if (k < d_e && n < d_h) v[q] = *reinterpret_cast<const Vec *>(in + (size_t)k * d_h + n);
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int i = q * kPackThreads + tid;
#pragma unroll
      for (int e = 0; e < E; ++e) tile[i / VR][i % VR * E + e] = v[q][e];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int i = q * kPackThreads + tid, n = 3 * d_h + n0 + i / VR, kk = i % VR * E;
      if (n >= a.nf_pad) continue;
      TW *o = out + (size_t)n * d_e + k0 + kk;
      Vec r;
#pragma unroll
      for (int e = 0; e < E; ++e) r[e] = tile[kk + e][i / VR];
      if (k0 + kk + E <= d_e) {
        *reinterpret_cast<Vec *>(o) = r;
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (k0 + kk + e < d_e) o[e] = r[e];
      }
    }
  }
}

}  // namespace

hipError_t pack_weights(dt_model *p, const dt_gru *gru, const dt_head *head, hipStream_t s) {
  const int d_e = p->d_e, d_h = p->d_h, per = kPackThreads * kPackVecs * 16 / (p->wdt == DT_BF16 ? 2 : 4);
  auto blocks = [](int n, int each) { return (n + each - 1) / each; };
  PackArgs a{gru->w_ih, gru->w_hh, head->w, gru->b_ih, gru->b_hh, head->b, p->wfold, p->whh_t,
             p->b_ih, p->b_hh, p->b_c, d_e, d_h, p->nf_pad, 0, 0, 0};
  a.whh_end = blocks(3 * d_h * d_h, per);
  a.bias_end = a.whh_end + blocks(3 * d_h > d_e ? 3 * d_h : d_e, kPackThreads);
  a.ih_end = a.bias_end + blocks(3 * d_h * d_e, per);
  const dim3 grid(a.ih_end + blocks(d_e, 64) * blocks(p->nf_pad - 3 * d_h, 64)), block(kPackThreads);
  if (p->wdt == DT_BF16)
    hipLaunchKernelGGL(pack_kernel<uint16_t>, grid, block, 0, s, a);
  else
    hipLaunchKernelGGL(pack_kernel<float>, grid, block, 0, s, a);
  return hipGetLastError();
}

// Fold `rows` embedding rows: all of the vocabulary (cand null), or those of the
// ids in cand (-1: a row of zeros).  cadd: see fold_mfma_kernel.
static hipError_t launch_fold(const dt_model *p, const int32_t *cand, int rows, float *cadd, hipStream_t s) {
  const dim3 block(kFoldThreads);
  const bool by_col = rows <= p->nf;
  if (p->wdt == DT_F32) {
    hipLaunchKernelGGL(fold_f32_kernel, fold_grid((p->nf + 1 + 63) / 64, (rows + 63) / 64, by_col), block, 0, s,
                       (const float *)p->emb, cand, rows, p->d_e, (const float *)p->wfold, p->nf, p->d_h, p->b_ih,
                       p->b_c, p->P_all, p->U_all, p->c_all, cadd, by_col);
  } else if (p->d_e % 8 == 0) {
    // 128 x 128 tiles while they fill the chip twice over; smaller ones leave fewer
    // CUs idle (1,024 rows: 128 against 512 tiles).  Their K slices are twice as
    // long; more in flight, two or four slices of 64 or two of 128, was no faster
    // (35.2, 34.0 and 33.3 us)
    const int t128 = ((p->nf + 127) / 128) * ((rows + 127) / 128);
    if (t128 >= 512)
      hipLaunchKernelGGL((fold_mfma_kernel<2, 2, 2, 2, 64>),
                         fold_grid((p->nf + 127) / 128, (rows + 127) / 128, by_col), block, 0, s,
                         (const uint16_t *)p->emb, cand, rows, p->d_e, (const uint16_t *)p->wfold, p->nf, p->d_h,
                         p->b_ih, p->b_c, p->P_all, p->U_all, p->c_all, cadd, by_col);
    else
      hipLaunchKernelGGL((fold_mfma_kernel<2, 2, 1, 1, 128>),
                         fold_grid((p->nf + 63) / 64, (rows + 63) / 64, by_col), block, 0, s,
                         (const uint16_t *)p->emb, cand, rows, p->d_e, (const uint16_t *)p->wfold, p->nf, p->d_h,
                         p->b_ih, p->b_c, p->P_all, p->U_all, p->c_all, cadd, by_col);
  } else {
    hipLaunchKernelGGL(fold_simple_kernel<uint16_t>, dim3(rows), dim3(256), 0, s, (const uint16_t *)p->emb, cand,
                       rows, p->d_e, (const uint16_t *)p->wfold, p->nf, p->d_h, p->b_ih, p->b_c, p->P_all, p->U_all,
                       p->c_all, cadd);
  }
  return hipGetLastError();
}

hipError_t fold_vocab(const dt_model *p, hipStream_t s) { return launch_fold(p, nullptr, p->V, nullptr, s); }

hipError_t fold_candidates(const dt_model *p, const int32_t *cand, int rows, float *candv, hipStream_t s) {
  return launch_fold(p, cand, rows, candv, s);
}

}  // namespace dt
