// Device building blocks shared by the scan and the expansion kernels:
// order-preserving keys, running log-sum-exp tails, bitonic sorts in registers and
// the per-row merge of sorted chunk lists (Alg. 1 step 1; section 3.2).
#pragma once

#include "dt_internal.h"

namespace dt {
namespace sel {

// Running tail of exp((x - m) / tau) sums: m is the running max, s the sum.
// c = log2(e) / tau so that exp((x - m) / tau) = exp2((x - m) * c).
struct Tail {
  float m, s;
};

__device__ inline Tail tail_empty() { return Tail{-3.402823466e38f, 0.0f}; }

// 2^x on the hardware unit (v_exp_f32): results below 2^-126 flush to zero,
// which a sum of exponentials relative to its running max can ignore
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// SHIFT: the row's candidate values and R are written less the row's largest
// value s0 (R less s0 / tau), which changes no log-probability (a constant
// per row) but keeps the consumer's sums of a value and a correction at the
// magnitude of their difference: logits offset by thousands would otherwise
// leave fp32 ulps of 1e-4 in every score.  (s0 = 0 for a row whose largest
// value is not finite.)
__device__ inline float row_shift(float top) { return __builtin_isfinite(top) ? top : 0.0f; }

template <int N>
__device__ inline void tail_add_group(Tail &t, const float (&x)[N], float c) {
  float mx = t.m;
#pragma unroll
  for (int j = 0; j < N; ++j) mx = fmaxf(mx, x[j]);
  float s = t.s * fast_exp2((t.m - mx) * c);
#pragma unroll
  for (int j = 0; j < N; ++j) s += fast_exp2((x[j] - mx) * c);
  t.m = mx;
  t.s = s;
}

__device__ inline void tail_add1(Tail &t, float x, float c) {
  const float xs[1] = {x};
  tail_add_group<1>(t, xs, c);
}

__device__ inline Tail tail_merge(Tail a, Tail b, float c) {
  Tail r;
  r.m = fmaxf(a.m, b.m);
  r.s = a.s * fast_exp2((a.m - r.m) * c) + b.s * fast_exp2((b.m - r.m) * c);
  return r;
}

// Wave-wide reductions with DPP inside each row of 16 lanes (quad swaps, half
// mirror, mirror) and four lane reads across rows; every lane gets the same
// value.  The whole wave must be active.
__device__ inline float readlane_f(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               0xF, 0xF, false));
}
template <typename Op>
__device__ inline float wave_reduce(float v, Op op) {
  v = op(v, dpp_f<0xB1>(v));   // quad_perm [1,0,3,2]
  v = op(v, dpp_f<0x4E>(v));   // quad_perm [2,3,0,1]
  v = op(v, dpp_f<0x141>(v));  // row_half_mirror
  v = op(v, dpp_f<0x140>(v));  // row_mirror
  return op(op(readlane_f(v, 0), readlane_f(v, 16)), op(readlane_f(v, 32), readlane_f(v, 48)));
}
// block-wide tail reduction in a fixed order (deterministic); red: NT/64 float2.
// The block max first, then every sum rescaled to it once and added up.
template <int NT>
__device__ inline Tail block_tail(Tail t, float c, float2 *red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  (void)lane;
  const float wm = wave_reduce(t.m, [](float x, float y) { return fmaxf(x, y); });
  if ((threadIdx.x & 63) == 0) red[w].x = wm;
  __syncthreads();
  float m = red[0].x;
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) m = fmaxf(m, red[i].x);
  const float s = wave_reduce(t.s > 0.0f ? t.s * fast_exp2((t.m - m) * c) : 0.0f,
                              [](float x, float y) { return x + y; });
  if ((threadIdx.x & 63) == 0) red[w].y = s;
  __syncthreads();
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) sum += red[i].y;
  __syncthreads();
  return Tail{m, sum};
}

template <bool DEV_SCOPE, typename T>
__device__ inline void put(T *p, T v) {
  if constexpr (DEV_SCOPE)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

// The measure of a row's segment lists that the envelope bounds (kRowBoundMax), about
// 22 bytes a list entry and 20 a menu slot, and that the general expansion's LDS
// layout sets aside.  A contract on V and M: the merges themselves need 8 bytes a
// thread for each 64 slots of the menu.
__host__ __device__ inline int up16(int b) { return (b + 15) & ~15; }
__host__ __device__ inline int row_bound_bytes(int nlists, int M) {
  const int n = nlists * M;
  const int q = (M + nlists - 1) / nlists;
  const int nhp = (nlists * q + 1) & ~1;
  const int ns_cap = n < 1024 ? n : 1024;
  int b = up16(8 * n);
  b = up16(b + 8 * M);
  b = up16(b + 4 * M);
  b = up16(b + 8 * nhp);
  b = up16(b + 8 * (ns_cap + 2));
  b = up16(b + 4 * n);
  return up16(b + 2 * n);
}

// ---------------------------------------------------------------------------
// One wave merges a row's segment lists when M <= 64 and there are at most 16
// lists: lane p holds position p of every list, and pairs of lists combine in
// a tree.  Of a descending list A and an ascending list B, max(A[i], B[i]) is
// the better half of A and B as a bitonic sequence (six compare-exchange
// stages sort it) and min(A[i], B[i]) the worse half, which joins the lane's
// tail right away: every key not among the row's M best is added to exactly
// one lane's tail, in an order fixed by the tree.  No LDS and no barrier.

// a 64-bit value from lane ^ J (DPP inside rows of 16 lanes, swizzle across
// rows, permute across halves); the whole wave must be active
template <int J>
__device__ inline uint64_t lane_xor64(uint64_t v) {
  const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
  int plo, phi;
  if constexpr (J == 1 || J == 2 || J == 8) {
    // quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_ror:8
    constexpr int ctrl = J == 1 ? 0xB1 : (J == 2 ? 0x4E : 0x128);
    plo = __builtin_amdgcn_update_dpp(0, lo, ctrl, 0xF, 0xF, false);
    phi = __builtin_amdgcn_update_dpp(0, hi, ctrl, 0xF, 0xF, false);
  } else if constexpr (J == 4) {
    // row_shl:4 (from lane + 4) where bit 2 is clear, row_shr:4 (lane - 4) where set
    const bool up = (threadIdx.x & 4) != 0;
    const int lo_a = __builtin_amdgcn_update_dpp(0, lo, 0x104, 0xF, 0xF, false);
    const int lo_b = __builtin_amdgcn_update_dpp(0, lo, 0x114, 0xF, 0xF, false);
    const int hi_a = __builtin_amdgcn_update_dpp(0, hi, 0x104, 0xF, 0xF, false);
    const int hi_b = __builtin_amdgcn_update_dpp(0, hi, 0x114, 0xF, 0xF, false);
    plo = up ? lo_b : lo_a;
    phi = up ? hi_b : hi_a;
  } else if constexpr (J == 16) {
    // swizzle bit mode inside 32 lanes: and 0x1F, or 0, xor 0x10
    plo = __builtin_amdgcn_ds_swizzle(lo, 0x401F);
    phi = __builtin_amdgcn_ds_swizzle(hi, 0x401F);
  } else {
    static_assert(J == 32, "lane distance");
    const int a = (int)((threadIdx.x & 63) ^ 32) * 4;
    plo = __builtin_amdgcn_ds_bpermute(a, lo);
    phi = __builtin_amdgcn_ds_bpermute(a, hi);
  }
  return ((uint64_t)(uint32_t)phi << 32) | (uint32_t)plo;
}

template <int J>
__device__ inline uint64_t cx_stage(uint64_t v, bool desc) {
  const uint64_t p = lane_xor64<J>(v);
  const bool keep_max = ((threadIdx.x & J) == 0) == desc;
  return ((p > v) == keep_max) ? p : v;  // (equal keys are both empty)
}

// sorts a bitonic sequence of 64 keys (one per lane), descending or ascending
__device__ inline uint64_t bitonic_clean64(uint64_t v, bool desc) {
  v = cx_stage<32>(v, desc);
  v = cx_stage<16>(v, desc);
  v = cx_stage<8>(v, desc);
  v = cx_stage<4>(v, desc);
  v = cx_stage<2>(v, desc);
  return cx_stage<1>(v, desc);
}

// the better half of a descending list a and an ascending list b, sorted in
// direction desc; the worse half joins the lane's tail (empty slots add
// nothing: -inf, whose term is 0 against any reference the tail can hold --
// the least being -FLT_MAX, against which -FLT_MAX itself would add 1)
__device__ inline uint64_t merge_halves(uint64_t a, uint64_t b, bool desc, Tail &t, float c) {
  const bool ga = a > b;
  const uint64_t hi = ga ? a : b, lo = ga ? b : a;
  tail_add1(t, lo ? key_value(lo) : -__builtin_huge_valf(), c);
  return bitonic_clean64(hi, desc);
}

// a wave's list: entry r * 64 + lane, descending (0: empty)
template <int R>
struct WaveList {
  uint64_t k[R];
};

// 64 ascending keys into the list; the 64 that drop out join the lanes' tails
template <int R>
__device__ inline void list_insert(WaveList<R> &l, uint64_t asc, Tail &tail, float c) {
#pragma unroll
  for (int r = 0; r < R - 1; ++r) {
    const bool ga = l.k[r] > asc;
    const uint64_t hi = ga ? l.k[r] : asc, lo = ga ? asc : l.k[r];
    l.k[r] = bitonic_clean64(hi, true);
    asc = bitonic_clean64(lo, false);
  }
  l.k[R - 1] = merge_halves(l.k[R - 1], asc, true, tail, c);
}

// another list (other(i): its entry i, descending) into this wave's: the best 64 R
// stay, the rest join the lanes' tails
template <int R, typename F>
__device__ inline void list_merge(WaveList<R> &l, F other, Tail &tail, float c) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t o = other(R * 64 - 1 - (r * 64 + lane));
    const bool ga = l.k[r] > o;
    const uint64_t lo = ga ? o : l.k[r];
    l.k[r] = ga ? l.k[r] : o;
    tail_add1(tail, lo ? key_value(lo) : -__builtin_huge_valf(), c);
  }
  // (now bitonic over the 64 R entries)
#pragma unroll
  for (int h = R / 2; h > 0; h >>= 1)
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & h) == 0) {
        const uint64_t x = l.k[r], y = l.k[r + h];
        l.k[r] = x > y ? x : y;
        l.k[r + h] = x > y ? y : x;
      }
#pragma unroll
  for (int r = 0; r < R; ++r) l.k[r] = bitonic_clean64(l.k[r], true);
}

// full bitonic sort of 64 keys (one per lane), descending or ascending
__device__ inline uint64_t wave_sort64(uint64_t v, bool desc) {
  const int lane = threadIdx.x & 63;
  // a stage of block size k orders each k-block the way the next block size needs
  auto dir = [&](int k) { return ((lane & k) == 0) == desc; };
  v = cx_stage<1>(v, dir(2));
  v = cx_stage<2>(v, dir(4));
  v = cx_stage<1>(v, dir(4));
  v = cx_stage<4>(v, dir(8));
  v = cx_stage<2>(v, dir(8));
  v = cx_stage<1>(v, dir(8));
  v = cx_stage<8>(v, dir(16));
  v = cx_stage<4>(v, dir(16));
  v = cx_stage<2>(v, dir(16));
  v = cx_stage<1>(v, dir(16));
  v = cx_stage<16>(v, dir(32));
  v = cx_stage<8>(v, dir(32));
  v = cx_stage<4>(v, dir(32));
  v = cx_stage<2>(v, dir(32));
  v = cx_stage<1>(v, dir(32));
  return bitonic_clean64(v, desc);
}

constexpr int kWaveMergeLists = 16;

__host__ __device__ inline bool wave_merge_fits(int nlists, int M) {
  return M <= 64 && nlists <= kWaveMergeLists;
}

// The row's M best keys, R = log sum over every other element of exp(x / tau) and
// the row flag, computed by the calling wave alone; wave_merge_fits must hold.
template <bool DEV_SCOPE, bool SHIFT = false>
__device__ __attribute__((always_inline)) void merge_row_wave(
    const uint64_t *lists, int nlists, int M, const float2 *tails, const int32_t *flags, float c,
    float inv_tau, int32_t *cand, float *candv, float *tailR, int32_t *rflag, const float *vadd) {
  constexpr int NL = kWaveMergeLists;
  const int lane = threadIdx.x & 63;
  // lists at even positions of the tree descending, odd ones reversed (ascending)
  uint64_t k[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int pos = (j & 1) ? 63 - lane : lane;
    k[j] = (j < nlists && pos < M) ? lists[j * M + pos] : 0ull;
  }
  Tail t = tail_empty();
  int bad = 0;
  if (lane < nlists) {
    const float2 tl = tails[lane];
    t = Tail{tl.x, tl.y};
    bad = flags[lane];
  }
  // level s: k[j] (j a multiple of 2s) takes the best 64 of lists j .. j+2s-1,
  // descending when it is the left operand of the next level, else ascending
#pragma unroll
  for (int s = 1; s < NL; s <<= 1) {
#pragma unroll
    for (int j = 0; j < NL; j += 2 * s) {
      if (j >= nlists) break;
      const bool desc = ((j / (2 * s)) & 1) == 0;
      if (j + s < nlists) {
        k[j] = merge_halves(k[j], k[j + s], desc, t, c);
      } else if (!desc) {
        k[j] = bitonic_clean64(k[j], false);  // a lone list, now the right operand
      }
    }
  }
  const uint64_t top = k[0];
  const bool keep = lane < M && top != 0ull;
  if (lane >= M && top) tail_add1(t, key_value(top), c);
  const float va = (keep && vadd) ? vadd[key_index(top)] : 0.0f;
  // the tail: the wave's max, then every lane's sum rescaled to it once
  const float m = wave_reduce(t.m, [](float x, float y) { return fmaxf(x, y); });
  const float sum = wave_reduce(t.s > 0.0f ? t.s * fast_exp2((t.m - m) * c) : 0.0f,
                                [](float x, float y) { return x + y; });
  const bool any_bad = __ballot(bad != 0) != 0ull;
  const float s0 = SHIFT ? row_shift(readlane_f(top ? key_value(top) : 0.0f, 0)) : 0.0f;
  if (lane < M) {
    put<DEV_SCOPE>(cand + lane, keep ? (int32_t)key_index(top) : (int32_t)-1);
    put<DEV_SCOPE>(candv + lane, keep ? (key_value(top) - s0) + va : -__builtin_huge_valf());
  }
  if (lane == 0) {
    put<DEV_SCOPE>(tailR, sum > 0.0f ? (m - s0) * inv_tau + logf(sum) : -__builtin_huge_valf());
    put<DEV_SCOPE>(rflag, (int32_t)(any_bad ? DT_TREE_NONFINITE : 0));
  }
}

// The same merge spread over the NT / 64 waves of a workgroup (every thread
// calls it): wave w merges its kWaveMergeLists / (NT / 64) lists in registers,
// then the tree's levels meet in LDS (xbuf: NT keys), one barrier each; the
// tails combine as in block_tail.
template <bool DEV_SCOPE, int NT, bool SHIFT = false>
__device__ __attribute__((always_inline)) void merge_row_tree(
    const uint64_t *lists, int nlists, int M, const float2 *tails, const int32_t *flags, float c,
    float inv_tau, uint64_t *xbuf, float2 *red, int32_t *cand, float *candv, float *tailR,
    int32_t *rflag, const float *vadd) {
  constexpr int W = NT / 64;
  constexpr int LPW = kWaveMergeLists / W;  // lists per wave
  static_assert(LPW >= 2 && LPW * W == kWaveMergeLists, "at least two lists per wave");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = LPW * wave;  // this wave's first list; the tree as in merge_row_wave
  Tail t = tail_empty();
  int bad = 0;
  if (wave == 0 && lane < nlists) {
    const float2 tl = tails[lane];
    t = Tail{tl.x, tl.y};
    bad = flags[lane];
  }
  uint64_t k[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int pos = (i & 1) ? 63 - lane : lane;
    k[i] = (j + i < nlists && pos < M) ? lists[(j + i) * M + pos] : 0ull;
  }
#pragma unroll
  for (int s = 1; s < LPW; s <<= 1) {
#pragma unroll
    for (int i = 0; i < LPW; i += 2 * s) {
      if (j + i >= nlists) break;
      const bool desc = (((j + i) / (2 * s)) & 1) == 0;
      if (j + i + s < nlists)
        k[i] = merge_halves(k[i], k[i + s], desc, t, c);
      else if (!desc)
        k[i] = bitonic_clean64(k[i], false);  // a lone list, now the right operand
    }
  }
  uint64_t v = k[0];
#pragma unroll
  for (int s = LPW; s < kWaveMergeLists; s <<= 1) {
    // right operands publish; a slot read at this level is never written at the next
    if (j < nlists && (j % (2 * s)) == s) xbuf[wave * 64 + lane] = v;
    __syncthreads();
    if (j < nlists && (j % (2 * s)) == 0) {
      const bool desc = ((j / (2 * s)) & 1) == 0;
      if (j + s < nlists)
        v = merge_halves(v, xbuf[(wave + s / LPW) * 64 + lane], desc, t, c);
      else if (!desc)
        v = bitonic_clean64(v, false);
    }
  }
  const bool keep = wave == 0 && lane < M && v != 0ull;
  if (wave == 0 && lane >= M && v) tail_add1(t, key_value(v), c);
  const float va = (keep && vadd) ? vadd[key_index(v)] : 0.0f;
  const bool any_bad = __ballot(bad != 0) != 0ull;  // (wave 0 holds the flags)
  t = block_tail<NT>(t, c, red);
  if (wave == 0) {
    const float s0 = SHIFT ? row_shift(readlane_f(v ? key_value(v) : 0.0f, 0)) : 0.0f;
    if (lane < M) {
      put<DEV_SCOPE>(cand + lane, keep ? (int32_t)key_index(v) : (int32_t)-1);
      put<DEV_SCOPE>(candv + lane, keep ? (key_value(v) - s0) + va : -__builtin_huge_valf());
    }
    if (lane == 0) {
      put<DEV_SCOPE>(tailR, t.s > 0.0f ? (t.m - s0) * inv_tau + logf(t.s) : -__builtin_huge_valf());
      put<DEV_SCOPE>(rflag, (int32_t)(any_bad ? DT_TREE_NONFINITE : 0));
    }
  }
}

// The same results for any number of lists and M <= 64 R: the lists are dealt to
// the waves, each merges its own in registers (the next one's loads in flight),
// and the waves' lists meet in LDS (xbuf: NT R keys).  Bound by the merges'
// chains of lane exchanges.  Against ranking the survivors of a threshold in LDS:
// 8 lists of 128 keys, 128 rows, 19.6 -> 4.2 us; 4 lists of 64, 512 rows, 6.5 -> 4.8.
// DEV_SCOPE selects device-scope stores (results read by other workgroups).
// vadd (nullable): candv[m] = logit + vadd[cand[m]] instead of the logit.
template <bool DEV_SCOPE, int NT, int R, bool SHIFT = false>
__device__ __attribute__((always_inline)) void merge_row_lists(
    const uint64_t *lists, int nlists, int M, const float2 *tails, const int32_t *flags, float c,
    float inv_tau, uint64_t *xbuf, float2 *red, int *flag_lds, int32_t *cand, float *candv, float *tailR,
    int32_t *rflag, const float *vadd) {
  constexpr int W = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) *flag_lds = 0;
  WaveList<R> l;
  uint64_t nx[R];  // the next list, reversed
  auto next = [&](int j) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = R * 64 - 1 - (r * 64 + lane);
      nx[r] = (j < nlists && i < M) ? lists[(size_t)j * M + i] : 0ull;
    }
  };
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * 64 + lane;
    l.k[r] = (wave < nlists && i < M) ? lists[(size_t)wave * M + i] : 0ull;
  }
  next(wave + W);
  Tail t = tail_empty();
  int bad = 0;
  for (int i = tid; i < nlists; i += NT) {
    const float2 tl = tails[i];
    t = tail_merge(t, Tail{tl.x, tl.y}, c);
    bad |= flags[i];
  }
  __syncthreads();
  if (bad) atomicOr(flag_lds, bad);
  for (int j = wave + W; j < nlists; j += W) {
    uint64_t cur[R];
#pragma unroll
    for (int r = 0; r < R; ++r) cur[r] = nx[r];
    next(j + W);
    // (entry 64 R - 1 - (64 r + lane) is the one loaded as cur[r])
    list_merge<R>(l, [&](int i) { return cur[(R * 64 - 1 - i) >> 6]; }, t, c);
  }
#pragma unroll
  for (int s = 1; s < W; s <<= 1) {
    if (s < nlists) {  // (uniform)
      if ((wave & (2 * s - 1)) == s)
#pragma unroll
        for (int r = 0; r < R; ++r) xbuf[wave * 64 * R + r * 64 + lane] = l.k[r];
      __syncthreads();
      if ((wave & (2 * s - 1)) == 0 && wave + s < nlists)
        list_merge<R>(l, [&](int i) { return xbuf[(wave + s) * 64 * R + i]; }, t, c);
    }
  }
  float va[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool mine = wave == 0 && l.k[r] != 0ull;
    if (mine && r * 64 + lane >= M) tail_add1(t, key_value(l.k[r]), c);
    va[r] = (mine && r * 64 + lane < M && vadd) ? vadd[key_index(l.k[r])] : 0.0f;
  }
  t = block_tail<NT>(t, c, red);
  if (wave == 0) {
    const float s0 = SHIFT ? row_shift(readlane_f(l.k[0] ? key_value(l.k[0]) : 0.0f, 0)) : 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = r * 64 + lane;
      if (i < M) {
        const uint64_t k = l.k[r];
        put<DEV_SCOPE>(cand + i, k ? (int32_t)key_index(k) : (int32_t)-1);
        put<DEV_SCOPE>(candv + i, k ? (key_value(k) - s0) + va[r] : -__builtin_huge_valf());
      }
    }
    if (lane == 0) {
      put<DEV_SCOPE>(tailR, t.s > 0.0f ? (t.m - s0) * inv_tau + logf(t.s) : -__builtin_huge_valf());
      put<DEV_SCOPE>(rflag, (int32_t)(*flag_lds ? DT_TREE_NONFINITE : 0));
    }
  }
  __syncthreads();
}

}  // namespace sel
}  // namespace dt
