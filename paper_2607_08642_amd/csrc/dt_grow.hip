// S3-S5 for menus and budgets of at most 64 (Alg. 1 steps 2-4; section 3.1
// conditional children; section 3.5 verification mask): the same speculative,
// depth-synchronous expansion as the general kernel's, with the candidate list
// in registers.
//
// What bounds it: the chain of dependent steps of one tree (per step: select,
// GRU, correction, exchange between the tree's workgroups, children, ranking),
// every link of it latency.  So each link is kept short:
//
//  * The candidates -- the B best known nodes, the only ones that can still be
//    popped -- are a sorted list, one entry per lane, held by every wave alike.
//    A step's children go through LDS once, and every wave sorts the union for
//    itself: no node table, no append, no second ranking pass.
//  * The list's order is the heap's pop order, ties included, so the final list
//    is the emitted tree and no replay follows.  Nodes are ordered by
//      (score desc, level asc, parent's place asc, sibling's rank),
//    level = how many of its nearest ancestors share the node's score in
//    unbroken succession.  Among nodes of one score the heap works first in,
//    first out (equal keys leave by insertion order, and all of those whose
//    parents score higher are in before the first leaves): level by level, and
//    within a level by the parents' order, then the siblings' rank (log-prob desc,
//    slot asc).  Siblings of one score are rare -- twins, or log-probs that the sum
//    with a low parent's score rounds together -- so entries carry their slot as the
//    rank, and a step whose list holds such siblings ranks its nodes' children and
//    sorts again.  An ancestor always precedes its descendants, so cutting the list
//    at B keeps parents.
//  * A member owns 32 hidden units (G = d_h / 32 members) and keeps its W_hh
//    fragments in registers for the whole launch; two workgroups can share a CU.
//    With more trees than resident groups a group builds several in turn.
//  * W_hh S is formed once per expanded node, right after its state is exchanged
//    and while its children are being scored, and kept in LDS for them: neither
//    the states' loads nor the MFMA stand between a selection and the GRU.
//  * Path states are exchanged as the three bf16 planes the MFMA reads (hi + mid
//    + lo is the fp32 value exactly), split once by their producer.  For at most
//    five nodes the planes take a column each: one MFMA pass instead of three.
//  * Partial corrections are polled for directly: a word still holding the
//    "empty" pattern has not arrived.  Three buffers rotate; a member empties its
//    part of the buffer that the next exchange uses before it sends the current
//    one, so a reader that has all of step s finds the buffer of step s + 1
//    either empty or filled.
//  * Only two depths of an expanded node's products are kept (nodes are expanded
//    in depth order, so a depth's parents are the depth above), and the exchanged
//    states of two steps.
//
// Measured per call (scan included) against the general kernel, us, both in turn on
// the same inputs: one tree at d_h = 512, M = 64, B = 16, L = 16: 31.4 / 37.9; long
// paths (k = 8) 56.3 / 75.0; B = 64: 54.0 / 61.6; 32 trees 122 / 137; 100 trees of
// long paths 500 / 540; d_h = 64, fp32: 29.6 / 48.9.  A step takes about 11,000 cycles (19,000 before):
// exchange 2,600, ranking 1,600, children 1,400, products 1,200, selection 900,
// GRU 850, correction 850, inputs 850, publishing 700.  Weights kept out of the
// registers (spilled) or two kernels of 256 registers per SIMD for one tree were
// slower (33.8 us); a bitonic sort instead of the count took 2,650 cycles.
#include "dt_select.h"
#include <hip/hip_ext.h>

#include <type_traits>

namespace dt {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int GT = kGrowThreads;
constexpr int GW = GT / 64;
constexpr int CH = kChunkNodes;
constexpr int UW = kGrowUnits;
constexpr int MP = 64;                // slots of a menu, padded
constexpr int kTile = 272;            // floats of a 16 x 16 gate tile in LDS (16-row groups of 4, padded)
constexpr int kChainTile = 48;        // ... of its first three columns
constexpr int kGh = 4 * UW;           // floats kept of an expanded node: W_hh S (r, z, n), S
constexpr int SNS = UW + 4;           // row stride of the new states in LDS
constexpr uint32_t kEmptyWord = 0xFFFFFFFFu;  // a partial correction that has not arrived
constexpr int kGrowSpin = 1 << 18;    // default bound of a wait
static_assert(GW == 4 && CH == 16 && UW == 32, "the work split below");
// the children function of an instance: conditional, the depths' marginals, or the
// menus of a greedy chain
enum { kCond = DT_SCORER_COND, kMarg = DT_SCORER_MARG, kStatic = DT_SCORER_STATIC };

struct GrowArgs {
  int L, M, B, k, G, norm_mode, pos_offset, batch, nchunks, nxcd, ngroups, spin_limit;
  int compact;     // rows merged by an earlier launch; table rows are candidate slots
  float inv_tau, c2;
  const uint64_t *ckeys;
  const float2 *ctail;
  const int32_t *cflag;
  int32_t *cand;
  float *candv;
  float *tailR;
  int32_t *rflag;
  const float *P_all, *U_all, *c_all;
  const void *whh;
  const float *b_hh, *h0;
  char *states;    // [ngroups][2][CH][state row]
  float *part;     // [ngroups][3][CH][G][MP]
  int32_t *bar;    // barrier and slot counters (zeroed by the scan kernel)
  int32_t *stats;
  const float *cost;
  dt_tree out;
};

struct GrowLds {
  int list, top, gpart, sn, anc, red, ints, gh, ids, vals, tails, total;
};
__host__ __device__ inline GrowLds grow_layout(int L, int B, int arm) {
  GrowLds l;
  int o = 0;
  auto take = [&](int bytes) {
    const int r = o;
    o += (bytes + 15) / 16 * 16;
    return r;
  };
  l.list = take((CH + 1) * MP * 8);  // a step's children, and the old entries beside them
  l.top = take(64 * 8);
  l.gpart = take(arm == kCond ? GW * 6 * kTile * 4 : arm == kStatic ? GW * 6 * kChainTile * 4 : 0);
  l.sn = take(arm == kCond ? CH * SNS * 4 : arm == kStatic ? GW * UW * 4 : 0);
  l.anc = take(64 * 8);
  l.red = take(GW * 8);
  l.ints = take(16 * 4);
  l.gh = take(arm == kCond ? 2 * B * kGh * 4 : 0);
  const int sets = arm == kStatic ? 2 : 1;  // (the tree a member builds, and the chain under way)
  l.ids = take(sets * L * MP * 4);
  l.vals = take(sets * L * MP * 4);
  l.tails = take(L * 4);
  l.total = o;
  return l;
}
enum { I_STATUS, I_CNT0, I_CNT1, I_SLOT, I_LATE0, I_LATE1 };

// ---- device-scope access, barriers ------------------------------------------
constexpr int kSc1 = 16;  // cache-policy bit: device scope
constexpr int kRange = 0x3FFFFFF0;  // bytes a resource covers ...
constexpr int kOut = 0x40000000;    // ... and an offset past them: loads return zeros
__device__ inline __amdgpu_buffer_rsrc_t rsrc(const void *base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, kRange, 0x00020000);
}
__device__ inline uint4 ld16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kSc1));
}
__device__ inline uint32_t ld4(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kSc1));
}
__device__ inline void st16(__amdgpu_buffer_rsrc_t r, int off, uint4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, kSc1);
}
__device__ inline void st4(__amdgpu_buffer_rsrc_t r, int off, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b32(v, r, off, 0, kSc1);
}
__device__ inline void st2(__amdgpu_buffer_rsrc_t r, int off, uint16_t v) {
  __builtin_amdgcn_raw_buffer_store_b16(v, r, off, 0, kSc1);
}

// a block barrier that orders LDS only (global loads and stores stay in flight)
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// ... after every store of this wave has reached the device's L2
__device__ inline void store_barrier() {
  __builtin_amdgcn_s_waitcnt(0);
  lds_barrier();
}

// ---- wave primitives ----------------------------------------------------------
__device__ inline int pull(int v, int src) { return __builtin_amdgcn_ds_bpermute(src * 4, v); }
__device__ inline int push(int v, int dst) { return __builtin_amdgcn_ds_permute(dst * 4, v); }
__device__ inline float as_f(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ inline uint32_t as_u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ inline int lane_rank(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}
// a + b with a from this half of the wave and b from the other: lanes 0-31 take
// x of both halves, lanes 32-63 y (16: the same with the odd rows of 16 lanes)
__device__ inline float fold32(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(as_u(x), as_u(y), false, false);
  return as_f(r[0]) + as_f(r[1]);
}
__device__ inline float fold16(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(as_u(x), as_u(y), false, false);
  return as_f(r[0]) + as_f(r[1]);
}
template <typename Op>
__device__ inline float wave_all(float v, Op op) {
  v = op(v, sel::dpp_f<0xB1>(v));
  v = op(v, sel::dpp_f<0x4E>(v));
  v = op(v, sel::dpp_f<0x141>(v));
  v = op(v, sel::dpp_f<0x140>(v));
  const auto r = __builtin_amdgcn_permlane16_swap(as_u(v), as_u(v), false, false);
  v = op(as_f(r[0]), as_f(r[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(as_u(v), as_u(v), false, false);
  return op(as_f(q[0]), as_f(q[1]));
}

// How many of the first `total` lanes' keys exceed this lane's.  A count rather
// than a bitonic sort: three VALU instructions per key and no dependent lane
// exchanges (a sort of 64 took 2,650 cycles, 21 dependent exchanges with mask
// arithmetic between them).
__device__ inline int count_above(uint32_t k, int total) {
  int r = 0;
  for (int j = 0; j < total; j += 8) {
    uint32_t s[8], d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = __builtin_amdgcn_readlane((int)k, j + i);
    // min(saturating s - k, 1): no compare masks, whose use stalls the next instruction
#pragma unroll
    for (int i = 0; i < 8; ++i) d[i] = __builtin_elementwise_sub_sat(s[i], k);
#pragma unroll
    for (int i = 0; i < 8; ++i) d[i] = min(d[i], 1u);
    r += (int)(((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7])));
  }
  return r;
}
__device__ inline int count_above(uint64_t k, int total) {
  int r = 0;
  for (int j = 0; j < total; j += 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)k, j + i);
      const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(k >> 32), j + i);
      r += (((uint64_t)hi << 32) | lo) > k;
    }
  }
  return r;
}

// GRU activations on the hardware exp2 and reciprocal (about 1 ulp each)
__device__ inline float sigmoid_fast(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * x));
}
__device__ inline float tanh_fast(float x) { return 2.0f * sigmoid_fast(2.0f * x) - 1.0f; }
__device__ inline float exp_hw(float x) { return __builtin_amdgcn_exp2f(1.44269504088896341f * x); }
__device__ inline float log_hw(float x) { return 0.69314718055994531f * __builtin_amdgcn_logf(x); }

// ---- path states ---------------------------------------------------------------
// bf16 weights: three bf16 planes (hi, mid, lo) of d_h values, each rounded to
// nearest; the residuals are exact, so hi + mid + lo is the fp32 value and the
// three bf16 products carry it to fp32 accuracy.  fp32 weights: fp32 values.
template <typename TW>
struct State;
template <>
struct State<uint16_t> {
  static __host__ __device__ constexpr int row_bytes(int dh) { return 6 * dh; }
  static __device__ inline void store(__amdgpu_buffer_rsrc_t r, int row, int dh, int j, float x) {
    const __bf16 h = (__bf16)x;
    const float r1 = x - (float)h;
    const __bf16 m = (__bf16)r1;
    const __bf16 l = (__bf16)(r1 - (float)m);
    const int o = row + j * 2;
    st2(r, o, __builtin_bit_cast(uint16_t, h));
    st2(r, o + 2 * dh, __builtin_bit_cast(uint16_t, m));
    st2(r, o + 4 * dh, __builtin_bit_cast(uint16_t, l));
  }
  // ... with no half word that reads as empty
  static __device__ inline void send(__amdgpu_buffer_rsrc_t r, int row, int dh, int j, float x) {
    const __bf16 h = (__bf16)x;
    const float r1 = x - (float)h;
    const __bf16 m = (__bf16)r1;
    const __bf16 l = (__bf16)(r1 - (float)m);
    const int o = row + j * 2;
    auto full = [](__bf16 v) {
      const uint16_t b = __builtin_bit_cast(uint16_t, v);
      return b == 0xFFFFu ? (uint16_t)0x7FC0u : b;
    };
    st2(r, o, full(h));
    st2(r, o + 2 * dh, full(m));
    st2(r, o + 4 * dh, full(l));
  }
};
template <>
struct State<float> {
  static __host__ __device__ constexpr int row_bytes(int dh) { return 4 * dh; }
  static __device__ inline void store(__amdgpu_buffer_rsrc_t r, int row, int, int j, float x) {
    st4(r, row + j * 4, as_u(x));
  }
  static __device__ inline void send(__amdgpu_buffer_rsrc_t r, int row, int, int j, float x) {
    st4(r, row + j * 4, as_u(x) == kEmptyWord ? 0x7FC00000u : as_u(x));
  }
};

// W_hh . S of a member's 32 units (two groups of 16, gates r, z, n) over the k
// steps [k0, k1) of 32, k1 - k0 <= KPW, with the weights resident in registers
// (FULL: k1 - k0 = KPW always).  Splitting k over the waves rather than the units
// has every state value loaded by one wave only.
template <typename TW, int KPW, bool FULL, int OCC>
struct Gates;

template <int KPW, bool FULL, int OCC>
struct Gates<uint16_t, KPW, FULL, OCC> {
  static constexpr bool kPlanes = true;
  static constexpr int kH = KPW < 2 || OCC > 1 ? 1 : 2;  // k steps of three planes in flight
  uint4 w[KPW][6];
  static constexpr int kF = KPW > 3 * kH ? KPW : 3 * kH;
  struct Frag {
    uint4 s[kF];
  };
  __device__ inline void load(const void *whh, int u, int nks, int k0, int k1) {
    const uint4 *W = static_cast<const uint4 *>(whh);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < KPW; ++i)
#pragma unroll
      for (int g = 0; g < 6; ++g)
        w[i][g] = FULL || k0 + i < k1 ? W[((size_t)(u * 3 + g) * nks + k0 + i) * 64 + lane] : make_uint4(0, 0, 0, 0);
  }
  static __device__ inline f32x4 mma(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                  0, 0, 0);
  }
  // one: a column per plane (rowoff: the lane's plane of its state row), all k
  // steps; else a column per node, the three planes of kH steps.  The same loads
  // either way (what a mode, or a k step past k1, does not need is out of range:
  // zeros, no traffic), so nothing merges behind a branch and waits there.
  static __device__ inline void fetch(__amdgpu_buffer_rsrc_t st, bool one, int rowoff, int dh, int k0, int k1,
                                      int lane, Frag &f) {
    const int o = rowoff + (k0 * 32 + (lane >> 4) * 8) * 2;
#pragma unroll
    for (int i = 0; i < kF; ++i) {
      const bool in1 = i < KPW && (FULL || k0 + i < k1), in3 = i < 3 * kH && (FULL || k0 + i / 3 < k1);
      const int off = one ? (in1 ? i * 64 : kOut) : (in3 ? (i / 3) * 64 + (i % 3) * 2 * dh : kOut);
      f.s[i] = ld16(st, o + off);
    }
  }
  // a chain's node (off: the lane's plane of its row, or out of range), and whether
  // part of it has not arrived
  static __device__ inline void fetch_one(__amdgpu_buffer_rsrc_t st, int off, int k0, int k1, int lane, Frag &f) {
    const int o = off + (k0 * 32 + (lane >> 4) * 8) * 2;
#pragma unroll
    for (int i = 0; i < KPW; ++i) f.s[i] = ld16(st, FULL || k0 + i < k1 ? o + i * 64 : kOut);
  }
  static __device__ inline bool empty(const Frag &f) {
    u16x2 m = {0, 0};
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
      const uint32_t w[4] = {f.s[i].x, f.s[i].y, f.s[i].z, f.s[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[e]));
    }
    return m.x == 0xFFFFu || m.y == 0xFFFFu;
  }
  template <bool ONE>
  __device__ inline void mul(__amdgpu_buffer_rsrc_t st, int rowoff, int dh, int k0, int k1, int lane, Frag &f,
                             f32x4 (&acc)[6]) const {
#pragma unroll
    for (int g = 0; g < 6; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (ONE) {
#pragma unroll
      for (int i = 0; i < KPW; ++i)
#pragma unroll
        for (int g = 0; g < 6; ++g) acc[g] = mma(w[i][g], f.s[i], acc[g]);
    } else {
#pragma unroll
      for (int i0 = 0; i0 < KPW; i0 += kH) {
        if (i0) fetch(st, false, rowoff + i0 * 64, dh, k0, k1 - i0, lane, f);
#pragma unroll
        for (int i = 0; i < kH; ++i)
#pragma unroll
          for (int p = 2; p >= 0; --p)
#pragma unroll
            for (int g = 0; g < 6; ++g) acc[g] = mma(w[i0 + i][g], f.s[3 * i + p], acc[g]);
      }
    }
  }
};

template <int KPW, bool FULL, int OCC>
struct Gates<float, KPW, FULL, OCC> {
  static constexpr bool kPlanes = false;
  float4 w[2 * KPW][6];
  struct Frag {
    float4 s[2 * KPW];
  };
  __device__ inline void load(const void *whh, int u, int nks, int k0, int k1) {
    const float4 *W = static_cast<const float4 *>(whh);
    const int lane = threadIdx.x & 63, nq = 2 * nks;
#pragma unroll
    for (int i = 0; i < 2 * KPW; ++i)
#pragma unroll
      for (int g = 0; g < 6; ++g)
        w[i][g] = FULL || 2 * k0 + i < 2 * k1 ? W[((size_t)(u * 3 + g) * nq + 2 * k0 + i) * 64 + lane]
                                              : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  static __device__ inline void fetch(__amdgpu_buffer_rsrc_t st, bool, int rowoff, int, int k0, int k1, int lane,
                                      Frag &f) {
    const int o = rowoff + (k0 * 32 + (lane >> 4) * 4) * 4;
#pragma unroll
    for (int i = 0; i < 2 * KPW; ++i)
      f.s[i] = __builtin_bit_cast(float4, ld16(st, o + (FULL || 2 * k0 + i < 2 * k1 ? i * 64 : kOut)));
  }
  static __device__ inline void fetch_one(__amdgpu_buffer_rsrc_t st, int off, int k0, int k1, int lane, Frag &f) {
    fetch(st, true, off, 0, k0, k1, lane, f);
  }
  static __device__ inline bool empty(const Frag &f) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 2 * KPW; ++i)
      m = max(max(m, as_u(f.s[i].x)), max(as_u(f.s[i].y), max(as_u(f.s[i].z), as_u(f.s[i].w))));
    return m == kEmptyWord;
  }
  template <bool ONE>
  __device__ inline void mul(__amdgpu_buffer_rsrc_t, int, int, int, int, int, Frag &f, f32x4 (&acc)[6]) const {
#pragma unroll
    for (int g = 0; g < 6; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2 * KPW; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int g = 0; g < 6; ++g) {
          const float av = e == 0 ? w[i][g].x : e == 1 ? w[i][g].y : e == 2 ? w[i][g].z : w[i][g].w;
          const float bv = e == 0 ? f.s[i].x : e == 1 ? f.s[i].y : e == 2 ? f.s[i].z : f.s[i].w;
          acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[g], 0, 0, 0);
        }
  }
};

// KPW: k steps of 32 hidden units per wave at most (d_h <= 128 KPW); SG > 0 fixes
// the members (and with them d_h) at compile time; OCC: workgroups a CU is to hold;
// ARM: the children function.  A marginal tree needs no state: one workgroup.
// Menus of a greedy chain: the group's members run the chains of up to G trees,
// then each builds one of those trees from its menus.
template <typename TW, int KPW, int SG, int OCC, int ARM>
__global__ __launch_bounds__(GT, OCC) void grow_kernel(GrowArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const GrowLds ly = grow_layout(a.L, a.B, ARM);
  uint64_t *list = reinterpret_cast<uint64_t *>(smem + ly.list);
  uint64_t *top = reinterpret_cast<uint64_t *>(smem + ly.top);
  float *gpart = reinterpret_cast<float *>(smem + ly.gpart);
  float *Sn = reinterpret_cast<float *>(smem + ly.sn);
  float *gh = reinterpret_cast<float *>(smem + ly.gh);
  uint64_t *ancs = reinterpret_cast<uint64_t *>(smem + ly.anc);
  float2 *red = reinterpret_cast<float2 *>(smem + ly.red);
  uint64_t *cut = reinterpret_cast<uint64_t *>(smem + ly.red);  // (the row merges are done by then)
  int *ints = reinterpret_cast<int *>(smem + ly.ints);
  int32_t *ids = reinterpret_cast<int32_t *>(smem + ly.ids);
  float *vals = reinterpret_cast<float *>(smem + ly.vals);
  float *tails = reinterpret_cast<float *>(smem + ly.tails);

  const int tid0 = threadIdx.x, lane0 = tid0 & 63;
  const int tid = tid0, lane = lane0;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = a.L, M = a.M, B = a.B, G = SG > 0 ? SG : a.G;
  constexpr bool FULL = SG == 4 * KPW;
  const int dh = UW * G, nks = G;
  const float NEG_INF = -__builtin_huge_valf();

  // ---- which group, which member -----------------------------------------------
  // (workgroups are dealt to XCDs round-robin and members take their slots in
  // the order they start: a group's members share an XCD, and complete groups
  // form first)
  const int xcd = blockIdx.x % a.nxcd;
  if (xcd >= a.ngroups) return;
  int kk = blockIdx.x / a.nxcd;
  if (G > 1) {
    if (tid == 0)
      ints[I_SLOT] = __hip_atomic_fetch_add(a.bar + a.batch * kBarStride + xcd * kSlotStride, 1, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
    lds_barrier();
    kk = __builtin_amdgcn_readfirstlane(ints[I_SLOT]);
  }
  const int group = xcd + a.nxcd * (kk / G), member = kk % G;
  if (group >= a.ngroups) return;

  // ---- prologue: weights, empty exchange buffers, this member's rows of the scan
  const int k0 = nks * wave / GW, k1 = nks * (wave + 1) / GW;  // this wave's k steps of W_hh S
  using Gt = Gates<TW, KPW, FULL, OCC>;
  Gt gates;
  if constexpr (ARM != kMarg) gates.load(a.whh, member * 2, nks, k0, k1);
  const float bhn = ARM != kMarg ? a.b_hh[2 * dh + member * UW + (lane & 31)] : 0.0f;
  float *const gp = a.part + (size_t)group * 3 * CH * G * MP;
  const __amdgpu_buffer_rsrc_t rpart = rsrc(gp);
  const __amdgpu_buffer_rsrc_t rstate = rsrc(a.states + (size_t)group * 2 * CH * State<TW>::row_bytes(dh));
  const uint4 empty4 = make_uint4(kEmptyWord, kEmptyWord, kEmptyWord, kEmptyWord);
  // byte offset of (buffer, column, member): this thread's 16 bytes of column tid / 16
  auto part_off = [&](int buf, int c, int j) { return ((buf * CH + c) * G + j) * (MP * 4); };
  // chains: one column in four buffers, the states beside them
  constexpr int kPieces = (Gt::kPlanes ? 6 : 4) * UW / 16;  // 16-byte pieces of a member's state
  auto chain_off = [&](int buf, int j) { return (buf * G + j) * (MP * 4); };
  auto chain_piece = [&](int buf, int i) {
    return buf * State<TW>::row_bytes(dh) + (Gt::kPlanes ? (i >> 2) * 2 * dh + member * (2 * UW) + (i & 3) * 16
                                                         : member * (4 * UW) + i * 16);
  };
  if constexpr (ARM == kCond) {
#pragma unroll
    for (int b = 0; b < 3; ++b) st16(rpart, part_off(b, tid >> 4, member) + (tid & 15) * 16, empty4);
  } else if constexpr (ARM == kStatic) {
    if (tid < 64) st16(rpart, chain_off(tid >> 4, member) + (tid & 15) * 16, empty4);
    if (tid < 4 * kPieces) st16(rstate, chain_piece(tid / kPieces, tid % kPieces), empty4);
  }
  if (tid == 0) {
    ints[I_STATUS] = 0;
    ints[I_CNT0] = 0;
    ints[I_CNT1] = 0;
    ints[I_LATE0] = 0;
    ints[I_LATE1] = 0;
  }
  // rows of the group's trees, dealt to its members (a lone workgroup's to its waves)
  int cell = ARM == kMarg ? wave : member;
  for (int t = group; t < a.batch && !a.compact; t += a.ngroups) {
    if constexpr (ARM == kMarg) {
      for (; cell < L; cell += GW) {
        const int row = t * L + cell;
        sel::merge_row_wave<true, true>(a.ckeys + (size_t)row * a.nchunks * M, a.nchunks, M,
                                        a.ctail + (size_t)row * a.nchunks, a.cflag + (size_t)row * a.nchunks, a.c2,
                                        a.inv_tau, a.cand + (size_t)row * M, a.candv + (size_t)row * M,
                                        a.tailR + row, a.rflag + row, nullptr);
      }
      cell -= L;
      continue;
    }
    for (; cell < L; cell += G) {
      const int row = t * L + cell;
      sel::merge_row_tree<true, GT, true>(a.ckeys + (size_t)row * a.nchunks * M, a.nchunks, M,
                                          a.ctail + (size_t)row * a.nchunks, a.cflag + (size_t)row * a.nchunks,
                                          a.c2, a.inv_tau, list, red, a.cand + (size_t)row * M,
                                          a.candv + (size_t)row * M, a.tailR + row, a.rflag + row, a.c_all);
    }
    cell -= L;
  }
  bool dead = false;
  store_barrier();
  if (G > 1) {
    if (tid == 0) {
      int32_t *ctr = a.bar + group * kBarStride;
      __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int spins = 0;
      while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < G) {
        if (++spins > a.spin_limit) {
          ints[I_STATUS] = DT_TREE_TIMEOUT;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    lds_barrier();
    dead = ints[I_STATUS] & DT_TREE_TIMEOUT;
  }

  int xbuf = 0;             // exchange buffer of the next exchange
  int ncb[3] = {0, 0, 0};   // columns of each that hold this member's data
  int par = 0;              // which list counter the next step uses
  int xpar = 0;             // which half of the states the next exchange uses

  // a tree's merged rows: ids, values, tails, flags
  auto load_rows = [&](int t, int32_t *ids, float *vals) {
    lds_barrier();  // (the previous tree's rows are read out)
    if (tid == 0) ints[I_STATUS] = dead ? DT_TREE_TIMEOUT : 0;
    if (!dead) {
      const __amdgpu_buffer_rsrc_t rid = rsrc(a.cand + (size_t)t * L * M), rv = rsrc(a.candv + (size_t)t * L * M);
      const __amdgpu_buffer_rsrc_t rt = rsrc(a.tailR + (size_t)t * L), rf = rsrc(a.rflag + (size_t)t * L);
      const float tl = tid < L ? as_f(ld4(rt, tid * 4)) : 0.0f;
      const int fl = tid < L ? (int)ld4(rf, tid * 4) : 0;
      const int m = lane < M ? lane : M - 1;
      for (int d0 = wave; d0 < L; d0 += 4 * GW) {
        uint32_t id[4], v[4];
  #pragma unroll
        for (int i = 0; i < 4; ++i) {  // (rows past the last: it again)
          const int d = d0 + i * GW < L ? d0 + i * GW : L - 1;
          id[i] = ld4(rid, (d * M + m) * 4);
          v[i] = ld4(rv, (d * M + m) * 4);
        }
        asm volatile("" : "+v"(id[0]), "+v"(id[1]), "+v"(id[2]), "+v"(id[3]));  // (all in flight together)
  #pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = d0 + i * GW < L ? d0 + i * GW : L - 1;
          // (dead slots, -1: row 0, unused)
          ids[d * MP + lane] = a.compact ? (t * L + d) * M + m : max((int)id[i], 0);
          vals[d * MP + lane] = lane < M ? as_f(v[i]) : NEG_INF;
        }
      }
      if (tid < L) tails[tid] = tl;
      if (ARM == kCond && tid < kGh) gh[tid] = 0.0f;  // (a zero root state; h0's is written by the root step)
      lds_barrier();
      if (fl) atomicOr(&ints[I_STATUS], fl);
    }
    lds_barrier();
  };
  // the depths' menus, normalised where they lie (values to be scaled first)
  auto normalise = [&](float scale) {
    for (int d = wave; d < L; d += GW) {
      const float x = vals[d * MP + lane], R = tails[d];
      const float z = x > NEG_INF ? x * scale : NEG_INF;
      const bool tail = a.norm_mode == DT_NORM_TAIL && R > NEG_INF;
      float mx = wave_all(z, [](float p, float q) { return fmaxf(p, q); });
      if (tail) mx = fmaxf(mx, R);
      float sum = wave_all(z > NEG_INF ? exp_hw(z - mx) : 0.0f, [](float p, float q) { return p + q; });
      if (tail) sum += exp_hw(R - mx);
      vals[d * MP + lane] = z > NEG_INF ? z - (mx + log_hw(sum)) : NEG_INF;
    }
    lds_barrier();
  };

  // The greedy chain of a tree (Cond-static): vals becomes each depth's corrected
  // and scaled values.  One node per step, so every wave keeps the state itself
  // and a step is a GRU, a 32-term dot product per slot, one exchange and W_hh S,
  // with one barrier (the waves' parts of W_hh S).  States and corrections are
  // sent together and both polled for, so no store is waited for: four buffers
  // rotate, and the one that step s + 2 uses is emptied at step s by the waves
  // that fill it -- a reader of step s + 2 has seen that wave's words of step
  // s + 1, sent after the wave had waited for loads issued behind the emptying
  // stores; and a wave that empties has seen words of step s - 1 of every wave,
  // sent after the barrier behind their reads of step s - 2, the buffer's last.
  // P and U rows of the next depth's menu are loaded a step ahead (P into L2).
  uint32_t xs = 0;
  auto chain = [&](int t, const int32_t *ids, float *vals) {
    const int u = lane & 31, slot = 4 * (lane & 15) + (lane >> 4), cs = wave * 16 + (lane >> 2);
    const int col = lane & 15;
    float S = a.h0 ? a.h0[(size_t)t * dh + member * UW + u] : 0.0f;
    float gr = 0.0f, gz = 0.0f, gn = 0.0f, xr = 0.0f, xz = 0.0f, xn = 0.0f, pf;
    float4 u0, u1;
    auto ahead = [&](int d) {
      const float *ur = a.U_all + (size_t)ids[d * MP + cs] * dh + member * UW + (lane & 3) * 8;
      u0 = *reinterpret_cast<const float4 *>(ur);
      u1 = *reinterpret_cast<const float4 *>(ur + 4);
      const int i = tid < 3 * MP ? tid : 0;
      pf = a.P_all[(size_t)ids[d * MP + i / 3] * (3 * dh) + (i % 3) * dh + member * UW];
    };
    ahead(0);
    for (int d = 0; d < L; ++d) {
      const float x = vals[d * MP + slot];
      const int my_id = ids[d * MP + slot];
      const bool corr = d > 0 || a.h0 != nullptr, grows = corr && d + 1 < L;
      typename Gt::Frag frag;
      float dl = x;
      if (corr) {
        if (d > 0) {
          const float r = sigmoid_fast(xr + gr);
          const float z = sigmoid_fast(xz + gz);
          const float nn = tanh_fast(xn + r * (gn + bhn));
          S = (1.0f - z) * nn + z * S;
        }
        if (lane < UW) Sn[wave * UW + u] = S;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        const float4 *sp = reinterpret_cast<const float4 *>(Sn + wave * UW + (lane & 3) * 8);
        const float4 s0 = sp[0], s1 = sp[1];
        float dot = ((u0.x * s0.x + u0.y * s0.y) + (u0.z * s0.z + u0.w * s0.w)) +
                    ((u1.x * s1.x + u1.y * s1.y) + (u1.z * s1.z + u1.w * s1.w));
        dot += sel::dpp_f<0xB1>(dot);
        dot += sel::dpp_f<0x4E>(dot);
        const int b = xs & 3, eb = b ^ 2;
        ++xs;
        if ((lane & 3) == 0) st4(rpart, chain_off(b, member) + cs * 4, as_u(dot) == kEmptyWord ? 0x7FC00000u : as_u(dot));
        if (wave == 0 && lane < UW) State<TW>::send(rstate, b * State<TW>::row_bytes(dh), dh, member * UW + u, S);
        if ((lane & 3) == 0) st4(rpart, chain_off(eb, member) + cs * 4, kEmptyWord);
        if (wave == 0 && lane < kPieces) st16(rstate, chain_piece(eb, lane), empty4);
        float4 s;
        int spins = 0;
        const int fo = grows && col < (Gt::kPlanes ? 3 : 1) ? b * State<TW>::row_bytes(dh) + (Gt::kPlanes ? col * 2 * dh : 0)
                                                            : kOut;
        for (;;) {
          uint4 v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int j = 4 * i + (lane >> 4);
            v[i] = ld16(rpart, SG == 16 || j < G ? chain_off(b, j) + (lane & 15) * 16 : kOut);
          }
          gates.fetch_one(rstate, fo, k0, k1, lane, frag);
          bool late = Gt::empty(frag);
          uint32_t mx = 0;
          s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            mx = max(max(mx, v[i].x), max(v[i].y, max(v[i].z, v[i].w)));
            s.x += as_f(v[i].x);
            s.y += as_f(v[i].y);
            s.z += as_f(v[i].z);
            s.w += as_f(v[i].w);
          }
          late |= mx == kEmptyWord;
          if (__ballot(late) == 0) break;
          if (++spins > a.spin_limit) {
            if (lane == 0) ints[I_LATE0 + (d & 1)] = 1;
            break;
          }
          asm volatile("" ::: "memory");  // (load again)
        }
        dl = x + fold16(fold32(s.x, s.z), fold32(s.y, s.w));
      }
      // the next node: the best slot, ties to the lower
      const float z = x > NEG_INF ? dl * a.inv_tau : NEG_INF;
      const float mx = wave_all(z, [](float p, float q) { return fmaxf(p, q); });
      uint64_t best = __ballot(z == mx);
      if (best & (best - 1)) {
        const float ms = wave_all(z == mx ? (float)slot : 64.0f, [](float p, float q) { return fminf(p, q); });
        best = __ballot(z == mx && (float)slot == ms);
      }
      const int id = __builtin_amdgcn_readlane(my_id, best ? __builtin_ctzll(best) : 0);
      const float *pr = a.P_all + (size_t)id * (3 * dh) + member * UW + u;
      xr = pr[0];
      xz = pr[dh];
      xn = pr[2 * dh];
      ahead(d + 1 < L ? d + 1 : d);
      if (grows) {
        f32x4 acc[6];
        gates.template mul<true>(rstate, 0, dh, k0, k1, lane, frag, acc);
        if (col < 3) {
#pragma unroll
          for (int g = 0; g < 6; ++g)
            *reinterpret_cast<f32x4 *>(gpart + (wave * 6 + g) * kChainTile + col * 16 + (lane >> 4) * 4) = acc[g];
        }
      }
      lds_barrier();
      if (wave == 0) vals[d * MP + slot] = z;
      if (ints[I_LATE0 + (d & 1)]) {  // (a wave a step ahead writes the other word)
        dead = true;
        break;
      }
      if (!(mx > NEG_INF)) break;  // (no child: nothing deeper is reached)
      if (grows) {
        // this half's waves' parts, the planes, then the other half's
        const float *p = gpart + ((lane >> 5) * 12 + (u >> 4) * 3) * kChainTile + (u & 15);
        float w3[3];
#pragma unroll
        for (int g = 0; g < 3; ++g) {
          float c3[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) c3[q] = p[g * kChainTile + q * 16] + p[(6 + g) * kChainTile + q * 16];
          w3[g] = (c3[2] + c3[1]) + c3[0];
        }
        gr = fold32(w3[0], w3[0]);
        gz = fold32(w3[1], w3[1]);
        gn = fold32(w3[2], w3[2]);
      }
    }
    asm volatile("" ::"v"(pf));
    lds_barrier();
  };
  constexpr bool ST = ARM == kStatic;
  for (int t0 = group; t0 < a.batch; t0 += ST ? a.ngroups * G : a.ngroups) {
    int t = t0;
    if constexpr (ST) {
      int own = 0;
      for (int j = 0; j < G && t0 + j * a.ngroups < a.batch; ++j) {
        const int tc = t0 + j * a.ngroups;
        int32_t *cids = j == member ? ids : ids + L * MP;
        float *cvals = j == member ? vals : vals + L * MP;
        load_rows(tc, cids, cvals);
        int st = ints[I_STATUS];
        if (!(st & (DT_TREE_NONFINITE | DT_TREE_TIMEOUT))) {
          chain(tc, cids, cvals);
          if (dead) st |= DT_TREE_TIMEOUT;
        }
        if (j == member) own = st;
      }
      t = t0 + member * a.ngroups;
      if (t >= a.batch) return;  // (no tree of this round, nor of a later one)
      lds_barrier();
      if (tid < L) tails[tid] = as_f(ld4(rsrc(a.tailR + (size_t)t * L), tid * 4));
      if (tid == 0) ints[I_STATUS] = own;
      lds_barrier();
      normalise(1.0f);
    } else {
      load_rows(t, ids, vals);
      if constexpr (ARM == kMarg) normalise(a.inv_tau);
    }
    dt_tree o = a.out;
    int32_t *otok = o.tokens + (size_t)t * B;
    int32_t *opar = o.parents + (size_t)t * B;
    int32_t *odep = o.depth + (size_t)t * B;
    int32_t *opos = o.position_ids + (size_t)t * B;
    float *osc = o.scores + (size_t)t * B;
    uint8_t *omask = o.mask + (size_t)t * B * B;
    const bool empty_tree = ints[I_STATUS] & (DT_TREE_NONFINITE | DT_TREE_TIMEOUT);

    // ---- the candidate list: lane i holds entry i -----------------------------
    // hi: order-preserving score bits; lo: the rest of the order, (63 - level) << 26
    // | (126 - parent's place) << 19 | (63 - sibling's rank) << 13 (the root's children:
    // 127), and slot << 6; meta: depth | expanded << 7 | parent's state slot << 8 |
    // state slot << 16
    uint32_t e_hi = 0, e_lo = 0, e_meta = 0;
    int n = 0;
    float vB = NEG_INF;
    // the chunk: lane c < nc holds node c's score bits and place | slot << 6 |
    // parent's state slot << 12 | level << 20; node c's own state slot is sbase + c
    int nc = 1, d = 0, sbase = 0, scount = 0;
    uint32_t q_hi = 0, q_pk = 0;
    int nsteps = 0, nexp = 1;
    float pf[7] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};  // loads into L2 for the next step (see below)
    auto prefetched = [&]() {
      asm volatile("" ::"v"(pf[0]), "v"(pf[1]), "v"(pf[2]), "v"(pf[3]), "v"(pf[4]), "v"(pf[5]), "v"(pf[6]));
    };

    while (!empty_tree) {
      ++nsteps;
      // (opaque, so that addresses are formed where they are used and not kept in
      // registers over the loop: the weights need them)
      int lane_ = lane0;
      asm volatile("" : "+v"(lane_));
      const int lane = lane_, tid = wave * 64 + lane;
      const int slot = 4 * (lane & 15) + (lane >> 4);  // this lane's slot of a menu
      const bool corr = ARM == kCond && (d > 0 || a.h0 != nullptr);  // (a zero root state corrects nothing)
      float4 uf[UW / 16];  // U rows of the menu (rows 16 wave ..), this member's units
      if (corr) {
        const int m = wave * 16 + (lane & 15);
        const float *ur = a.U_all + (size_t)ids[d * MP + m] * dh + member * UW + (lane >> 4) * 4;
        // empty this member's part of the next exchange's buffer
        const int nb = xbuf == 2 ? 0 : xbuf + 1;
        const int nold = nb == 0 ? ncb[0] : (nb == 1 ? ncb[1] : ncb[2]);
        if ((tid >> 4) < nold) st16(rpart, part_off(nb, tid >> 4, member) + (tid & 15) * 16, empty4);
        if (nb == 0) ncb[0] = 0;
        if (nb == 1) ncb[1] = 0;
        if (nb == 2) ncb[2] = 0;
        const int u = lane & 31, srow = xpar * CH;
        if (d == 0) {
          // the root's state is h0
#pragma unroll
          for (int q = 0; q < UW / 16; ++q) uf[q] = *reinterpret_cast<const float4 *>(ur + q * 16);
          if (tid < UW) {
            const float s = a.h0[(size_t)t * dh + member * UW + tid];
            Sn[tid] = s;
            gh[3 * UW + tid] = s;
            State<TW>::store(rstate, srow * State<TW>::row_bytes(dh), dh, member * UW + tid, s);
          }
        } else {
          // 1. path states of this member's units: S = GRU(S_parent, E[token]).
          // W_hh S_parent was formed when the parent was expanded.  (unit, node)
          // pairs of this thread: node 2 wave + (lane / 32), + 8
          float xr[2], xz[2], xn[2];
          int ps[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int c = 2 * wave + (lane >> 5) + 8 * i;
            const int pk = pull(q_pk, c);
            ps[i] = (pk >> 12) & 255;
            xr[i] = xz[i] = xn[i] = 0.0f;
            if (c < nc) {
              const float *pr = a.P_all + (size_t)ids[(d - 1) * MP + ((pk >> 6) & 63)] * (3 * dh) + member * UW + u;
              xr[i] = pr[0];
              xz[i] = pr[dh];
              xn[i] = pr[2 * dh];
            }
          }
#pragma unroll
          for (int q = 0; q < UW / 16; ++q) uf[q] = *reinterpret_cast<const float4 *>(ur + q * 16);
          lds_barrier();  // (the products of the last step's nodes are in gh)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int c = 2 * wave + (lane >> 5) + 8 * i;
            if (c < nc) {
              const float *gp_ = gh + ps[i] * kGh + u;
              // (P_r, P_z carry b_hr, b_hz)
              const float r = sigmoid_fast(xr[i] + gp_[0]);
              const float z = sigmoid_fast(xz[i] + gp_[UW]);
              const float nn = tanh_fast(xn[i] + r * (gp_[2 * UW] + bhn));
              const float s = (1.0f - z) * nn + z * gp_[3 * UW];
              Sn[c * SNS + u] = s;
              gh[(sbase + scount + c) * kGh + 3 * UW + u] = s;
              State<TW>::store(rstate, (srow + c) * State<TW>::row_bytes(dh), dh, member * UW + u, s);
            }
          }
        }
        lds_barrier();
        // 2. this member's part of delta[c][m] = U[cand[m]] . S_c (fp32 MFMA; one
        // tile of 16 slots per wave)
        f32x4 acc;
        {
          const float *sp = Sn + (lane & 15) * SNS + (lane >> 4) * 4;
          f32x4 part[UW / 16];
#pragma unroll
          for (int q = 0; q < UW / 16; ++q) part[q] = f32x4{0.f, 0.f, 0.f, 0.f};
          float4 bv[UW / 16];
#pragma unroll
          for (int q = 0; q < UW / 16; ++q) bv[q] = *reinterpret_cast<const float4 *>(sp + q * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int q = 0; q < UW / 16; ++q) {
              const float av = e == 0 ? uf[q].x : e == 1 ? uf[q].y : e == 2 ? uf[q].z : uf[q].w;
              const float b = e == 0 ? bv[q].x : e == 1 ? bv[q].y : e == 2 ? bv[q].z : bv[q].w;
              part[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b, part[q], 0, 0, 0);
            }
          acc = part[0] + part[1];
        }
        // 3. publish it (16 slots 4 (lane / 16) .. of node lane % 16), after the
        // states and the emptied buffer of every wave
        store_barrier();
        if ((lane & 15) < nc) {
          uint32_t v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[i] = as_u(acc[i]);
            v[i] = v[i] == kEmptyWord ? 0x7FC00000u : v[i];
          }
          st16(rpart, part_off(xbuf, lane & 15, member) + wave * 64 + (lane >> 4) * 16,
               make_uint4(v[0], v[1], v[2], v[3]));
        }
        if (xbuf == 0) ncb[0] = nc;
        if (xbuf == 1) ncb[1] = nc;
        if (xbuf == 2) ncb[2] = nc;
      } else if constexpr (ARM != kCond) {
        // the last step's count and children are read by every wave behind that
        // step's one barrier and written anew below (a conditional step's barriers
        // above stand between the two)
        lds_barrier();
      }
      if (tid == 0) ints[I_CNT0 + (par ^ 1)] = 0;
      // 4. children: nodes wave, wave + 4, ... (pairs); lane = slot
      const float x = vals[d * MP + slot], R = tails[d];
      const int my_id = ids[d * MP + slot];
      const bool tail = a.norm_mode == DT_NORM_TAIL && R > NEG_INF;
      // W_hh S of the chunk's nodes, for their children: the states are loaded once
      // the chunk's corrections are here (every member sends those after its states
      // have arrived), and multiplied while nothing else waits for them
      const bool one = nc <= 5 && Gates<TW, KPW, FULL, OCC>::kPlanes;
      const bool grows = corr && d + 1 < L;
      typename Gates<TW, KPW, FULL, OCC>::Frag frag;
      int rowoff = 0;
      {
        const int col = lane & 15;
        const int node = one ? col / 3 : col;
        rowoff = node < nc ? (xpar * CH + node) * State<TW>::row_bytes(dh) : kOut;  // (unused columns: zeros)
        if (one) rowoff += (col - 3 * (col / 3)) * 2 * dh;
      }
      for (int j0 = 0; j0 < CH / GW; j0 += 2) {
        // (a wave without a node waits for the corrections of another's)
        const bool idle = wave + j0 * GW >= nc;
        if (idle && (j0 > 0 || !grows)) break;
        const int cc[2] = {idle ? 0 : wave + j0 * GW, wave + (j0 + 1) * GW};
        const bool two = cc[1] < nc;
        float dl[2] = {x, x};
        if (corr) {
          // lane (q = lane % 16, r = lane / 16) takes slots 4q .. 4q+3 of members
          // r, r + 4, ...; its sums then meet over r so that lane (q, r) holds slot
          // 4q + r: the same order of summation in every member
          float4 s[2];
          int spins = 0;
          for (;;) {
            uint32_t mx = 0;
            s[0] = s[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            const int base = part_off(xbuf, cc[0], 0) + lane * 16, second = part_off(0, GW, 0);
            for (int g0 = 0; g0 < G; g0 += 16) {
              uint4 v[2][4];
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const bool in = (SG > 0 && SG % 16 == 0) || g0 + 4 * i + (lane >> 4) < G;
                v[0][i] = in ? ld16(rpart, base + (g0 + 4 * i) * (MP * 4)) : make_uint4(0, 0, 0, 0);
              }
              if (two) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const bool in = (SG > 0 && SG % 16 == 0) || g0 + 4 * i + (lane >> 4) < G;
                  v[1][i] = in ? ld16(rpart, base + second + (g0 + 4 * i) * (MP * 4)) : make_uint4(0, 0, 0, 0);
                }
              }
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                if (h == 1 && !two) break;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  mx = max(max(mx, v[h][i].x), max(v[h][i].y, max(v[h][i].z, v[h][i].w)));
                  s[h].x += as_f(v[h][i].x);
                  s[h].y += as_f(v[h][i].y);
                  s[h].z += as_f(v[h][i].z);
                  s[h].w += as_f(v[h][i].w);
                }
              }
            }
            if (__ballot(mx == kEmptyWord) == 0) break;
            if (++spins > a.spin_limit) {
              if (lane == 0) atomicOr(&ints[I_STATUS], DT_TREE_TIMEOUT);
              break;
            }
            asm volatile("" ::: "memory");  // (load again)
          }
          if (j0 == 0) gates.fetch(rstate, one, grows ? rowoff : kOut, dh, k0, k1, lane, frag);
          if (idle) break;
#pragma unroll
          for (int h = 0; h < 2; ++h) dl[h] = x + fold16(fold32(s[h].x, s[h].z), fold32(s[h].y, s[h].w));
        }
        float g2[2], gpar[2];
        uint32_t pk2[2];
        uint64_t em[2] = {0ull, 0ull};
        int kept[2] = {0, 0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (h == 1 && !two) break;
          float lv = x;  // (menus already normalised)
          if constexpr (ARM == kCond) {
            const float z = x > NEG_INF ? dl[h] * a.inv_tau : NEG_INF;  // slots >= M hold -inf
            float mx = wave_all(z, [](float p, float q) { return fmaxf(p, q); });
            if (tail) mx = fmaxf(mx, R);
            float sum = wave_all(z > NEG_INF ? exp_hw(z - mx) : 0.0f, [](float p, float q) { return p + q; });
            if (tail) sum += exp_hw(R - mx);
            lv = z > NEG_INF ? z - (mx + log_hw(sum)) : NEG_INF;
          }
          const uint32_t ghi = __builtin_amdgcn_readlane(q_hi, cc[h] & 63);
          pk2[h] = __builtin_amdgcn_readlane(q_pk, cc[h] & 63);
          gpar[h] = d == 0 ? 0.0f : ordered_to_float(ghi);
          g2[h] = gpar[h] + lv;
          const bool in = lv > NEG_INF && g2[h] >= vB;
          em[h] = __ballot(in);
          kept[h] = __popcll(em[h]);
          if (a.k < B && kept[h] > a.k) {
            // the node's k best, (log-prob desc, slot asc)
            // (equal values leave a place without a lane: counted again by both)
            const uint32_t key = in ? ordered_bits(lv) : 0u;
            int rank = count_above(key, 64);
            const int filled = push((int)key, rank);  // (lanes outside E all go to lane kept, if there is one)
            if (__ballot(lane < kept[h] && filled == 0) != 0)
              rank = count_above(((uint64_t)key << 32) | (uint32_t)(63 - slot), 64);
            em[h] = __ballot(in && rank < a.k);
            kept[h] = a.k;
          }
        }
        int base = 0;
        if (lane == 0) base = atomicAdd(&ints[I_CNT0 + par], kept[0] + kept[1]);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if ((em[h] >> lane) & 1ull) {
            const int level = d > 0 && g2[h] == gpar[h] ? (int)((pk2[h] >> 20) & 63) + 1 : 0;
            const uint32_t place = d == 0 ? 0u : (pk2[h] & 63u) + 1u;  // parent's place + 1
            const uint32_t lo = ((uint32_t)(63 - min(level, 63)) << 26) | ((127u - place) << 19) |
                                ((uint32_t)(63 - slot) << 13) | 0x1000u | ((uint32_t)slot << 6) | (uint32_t)cc[h];
            list[base + (h ? kept[0] : 0) + lane_rank(em[h])] = ((uint64_t)ordered_bits(g2[h]) << 32) | lo;
            // the child's input projection (this member's three gate slices, a
            // line each) is fetched into L2 while the list is sorted
            if (ARM == kCond && d + 1 < L) {
              const float *pr = a.P_all + (size_t)my_id * (3 * dh) + member * UW;
              pf[3 * h] = pr[0];
              pf[3 * h + 1] = pr[dh];
              pf[3 * h + 2] = pr[2 * dh];
            }
          }
        }
      }
      if (grows) {
        f32x4 acc[6];
        if (one)
          gates.template mul<true>(rstate, rowoff, dh, k0, k1, lane, frag, acc);
        else
          gates.template mul<false>(rstate, rowoff, dh, k0, k1, lane, frag, acc);
#pragma unroll
        for (int g = 0; g < 6; ++g)
          *reinterpret_cast<f32x4 *>(gpart + (wave * 6 + g) * kTile + (lane >> 4) * 68 + (lane & 15) * 4) = acc[g];
      }
      // ... and the next depth's U rows (one line each)
      if (ARM == kCond && wave == GW - 1 && d + 1 < L) pf[6] = a.U_all[(size_t)ids[(d + 1) * MP + lane] * dh + member * UW];
      lds_barrier();
      const int nnew = __builtin_amdgcn_readfirstlane(ints[I_CNT0 + par]);
      par ^= 1;
      if (corr) xbuf = xbuf == 2 ? 0 : xbuf + 1;
      if (ints[I_STATUS] & DT_TREE_TIMEOUT) break;  // (uniform: read after the barrier)
      if (grows) {
        // the waves' parts (and the planes) of W_hh S summed, one (unit, node) per thread
        const int u = lane & 31;
        const float *p = gpart + (u >> 4) * 3 * kTile + ((u & 15) >> 2) * 68 + (u & 3);
        float *dst = gh + (sbase + scount) * kGh + u;
        if (one) {
          // (at most five nodes: waves 0-2, nodes 2 wave, 2 wave + 1)
          const int c = 2 * wave + (lane >> 5);
          if (c < nc) {
            float v[3][3][GW];  // every load before the first sum
#pragma unroll
            for (int g = 0; g < 3; ++g)
#pragma unroll
              for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int w = 0; w < GW; ++w) v[g][q][w] = p[(w * 6 + g) * kTile + 12 * c + 4 * q];
#pragma unroll
            for (int g = 0; g < 3; ++g) {
              float s3[3];
#pragma unroll
              for (int q = 0; q < 3; ++q) s3[q] = (v[g][q][0] + v[g][q][1]) + (v[g][q][2] + v[g][q][3]);
              dst[c * kGh + g * UW] = (s3[2] + s3[1]) + s3[0];
            }
          }
        } else {
          float v[2][3][GW];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int c = 2 * wave + (lane >> 5) + 8 * i;  // (columns past nc hold zeros)
#pragma unroll
            for (int g = 0; g < 3; ++g)
#pragma unroll
              for (int w = 0; w < GW; ++w) v[i][g][w] = p[(w * 6 + g) * kTile + 4 * c];
          }
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int c = 2 * wave + (lane >> 5) + 8 * i;
            if (c < nc) {
#pragma unroll
              for (int g = 0; g < 3; ++g)
                dst[c * kGh + g * UW] = (v[i][g][0] + v[i][g][1]) + (v[i][g][2] + v[i][g][3]);
            }
          }
        }
      }
      if (corr) xpar ^= 1;
      // 5. the new list: the best of the old entries (payload: their lane) and the
      // children (payload: 0x1000 | slot << 6 | chunk node)
      const int total = n + nnew;
      uint32_t k = e_hi, p = e_lo | (uint32_t)lane;
      if (lane >= n) k = p = 0u;
      uint64_t ties = 0;  // lanes whose entry is a new sibling of the next one, of one score
      if (total <= 64) {
        if (lane >= n && lane < total) {
          const uint64_t e = list[lane - n];
          k = (uint32_t)(e >> 32);
          p = (uint32_t)e;
        }
        // (lanes without an entry count `total` keys above theirs and meet in a
        // lane that holds none; equal scores would leave a lane without an entry:
        // they are counted again by the whole order)
        int at = count_above(k, total);
        uint32_t ks = push((int)k, at);
        if (__ballot(lane < total && ks == 0) != 0) {
          at = count_above(((uint64_t)k << 32) | p, total);
          ks = push((int)k, at);
          if constexpr (ARM != kMarg) {
            const uint32_t ps = push((int)p, at), pn = pull((int)ps, lane + 1);
            ties = __ballot(lane + 1 < total && (uint32_t)pull((int)ks, lane + 1) == ks &&
                            (pn >> 19) == (ps >> 19) && (ps & 0x1000u));
          }
        }
        p = push((int)p, at);
        k = ks;
      } else {
        // too many for a lane each: wave 0 adds the old entries, every thread ranks
        // its share among all of them, and the best meet in LDS (the first beyond
        // them beside, to be seen as a sibling of the last)
        if (wave == 0 && lane < n) list[nnew + lane] = ((uint64_t)k << 32) | p;
        lds_barrier();
        for (int i = tid; i < total; i += GT) {
          const uint64_t e = list[i];
          const ulonglong2 *l2 = reinterpret_cast<const ulonglong2 *>(list);
          int at = 0;
#pragma unroll 4
          for (int j = 0; j < total >> 1; ++j) {
            const ulonglong2 v = l2[j];
            at += (v.x > e) + (v.y > e);
          }
          if (total & 1) at += list[total - 1] > e;
          if (at < B) top[at] = e;
          if (ARM != kMarg && at == B) *cut = e;
        }
        lds_barrier();
        const uint64_t e = lane < B ? top[lane] : 0ull;  // (total > 64 >= B: all of them are there)
        k = (uint32_t)(e >> 32);
        p = (uint32_t)e;
        if constexpr (ARM != kMarg) {
          const uint64_t en = lane + 1 < B ? top[lane + 1] : *cut;
          ties = __ballot(lane < B && (e >> 19) == (en >> 19) && (p & 0x1000u));
        }
      }
      // (the root's children: score = log-prob, so slots order the equal ones; a
      // marginal menu's log-probs descend with the slot)
      if (__builtin_expect(ARM != kMarg && ties != 0 && d > 0, 0)) {
        // The children by their log-probs' order, formed from their values again.  The
        // partial corrections stay until every member has sent the next ones; the
        // ranks go where the nodes' states were, which nothing reads any more in this
        // step.  A chain's menu is one for all nodes.  (Opaque, as above: nothing of
        // this is kept in registers over the loop; without it, and as a second pass
        // through the code above, a call took 2-6% longer.)
        int lane_ = lane0;
        asm volatile("" : "+v"(lane_));
        const int lane = lane_, tid = wave * 64 + lane, slot = 4 * (lane & 15) + (lane >> 4);
        uint8_t *rk = reinterpret_cast<uint8_t *>(Sn);  // [CH][MP] (a conditional tree's)
        static_assert(CH * MP <= CH * SNS * 4, "the ranks fit the states");
        if constexpr (ARM == kCond) {
#pragma unroll 1
          for (int c = wave; c < nc; c += GW) {
            float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
            const int base = part_off(xbuf == 0 ? 2 : xbuf - 1, c, 0) + lane * 16;
#pragma unroll 1
            for (int j = 0; j + (lane >> 4) < G; j += 4) {
              const uint4 w = ld16(rpart, base + j * (MP * 4));
              s.x += as_f(w.x);
              s.y += as_f(w.y);
              s.z += as_f(w.z);
              s.w += as_f(w.w);
            }
            const float v = vals[d * MP + slot] + fold16(fold32(s.x, s.z), fold32(s.y, s.w));
            const uint64_t key = ((uint64_t)ordered_bits(v) << 32) | (uint32_t)(63 - slot);
            int r = 63;
#pragma unroll 1
            for (int j = 0; j < 64; ++j) {
              const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)key, j);
              const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(key >> 32), j);
              r -= (((uint64_t)hi << 32) | lo) > key;
            }
            rk[c * MP + slot] = (uint8_t)r;
          }
        }
        lds_barrier();
        // ... and the list sorted again, every thread its share
        if (wave == 0 && lane < n) list[nnew + lane] = ((uint64_t)e_hi << 32) | e_lo | (uint32_t)lane;
        for (int i = tid; i < nnew; i += GT) {
          const uint64_t e = list[i];
          uint32_t r;
          if constexpr (ARM == kCond) {
            r = rk[((uint32_t)e & 15u) * MP + (((uint32_t)e >> 6) & 63u)];
          } else {
            const int sl = ((uint32_t)e >> 6) & 63u;
            const float v = vals[d * MP + sl];
            r = 63;
#pragma unroll 1
            for (int j = 0; j < 64; ++j) {
              const float o = vals[d * MP + j];
              r -= o > v || (o == v && j < sl);
            }
          }
          list[i] = (e & ~(63ull << 13)) | (r << 13);
        }
        lds_barrier();
#pragma unroll 1
        for (int i = tid; i < total; i += GT) {
          const uint64_t e = list[i];
          int at = 0;
#pragma unroll 1
          for (int j = 0; j < total; ++j) at += list[j] > e;
          if (at < B) top[at] = e;
        }
        lds_barrier();
        const uint64_t e = lane < B && lane < total ? top[lane] : 0ull;
        k = (uint32_t)(e >> 32);
        p = (uint32_t)e;
      }
      n = total < B ? total : B;
      const bool live = lane < n;
      const bool isnew = p & 0x1000u;
      const int om = pull(e_meta, p & 63);
      // an old entry's new place.  (The old entries that stay are the first ones,
      // so lane 63 is one of them only if all lanes are; the others may push there.)
      const int np = push(lane, live && !isnew ? (int)(p & 63u) : 63);
      const uint32_t place = 127u - ((p >> 19) & 127u);
      const int pnew = pull(np, place ? (int)place - 1 : 0);
      const uint32_t nplace = place ? (uint32_t)pnew + 1u : 0u;
      e_hi = live ? k : 0u;
      e_lo = (p & 0xFC07EFC0u) | ((127u - nplace) << 19);
      e_meta = isnew ? (d + 1) | ((sbase + scount + (int)(p & 15u)) << 8) : om;
      vB = n == B ? ordered_to_float(__builtin_amdgcn_readlane(k, B - 1)) : NEG_INF;
      // 6. the next chunk: up to 16 unexpanded nodes of the least depth, best first
      scount += d > 0 ? nc : 0;
      const int dep = e_meta & 127;
      const bool elig = live && !(e_meta & 128) && dep < L;
      if (__ballot(elig) == 0) break;
      const int dmin = (int)wave_all(elig ? (float)dep : 127.0f, [](float p_, float q_) { return fminf(p_, q_); });
      const int dn = __builtin_amdgcn_readfirstlane(dmin);
      if (dn != d) {
        sbase = (dn & 1) * B;
        scount = 0;
        d = dn;
      }
      const uint64_t use = __ballot(elig && dep == dn);
      const int before = lane_rank(use);
      const bool mine_ = ((use >> lane) & 1ull) && before < CH;
      nc = __popcll(use);
      nc = nc < CH ? nc : CH;
      nexp += nc;
      const int dst = mine_ ? before : 63;  // (lanes nc .. hold nothing)
      q_hi = push(e_hi, dst);
      q_pk = push(lane | (e_lo & 0xFC0u) | (((e_meta >> 8) & 255) << 12) | ((63 - (e_lo >> 26)) << 20), dst);
      if (mine_) e_meta |= 128 | ((sbase + scount + before) << 16);
    }
    prefetched();
    if (ints[I_STATUS] & DT_TREE_TIMEOUT) dead = true;
    if (ARM != kStatic && member != 0) {
      if (dead) return;  // (the others give up at their next wait)
      continue;
    }
    // ---- emission (member 0; of a chain's tree, the member that built it) ------------------------------------------------------
    const int status = ints[I_STATUS];
    if (a.stats && tid == 0) {
      a.stats[2 * t] = nsteps;
      a.stats[2 * t + 1] = nexp;
    }
    int npop = (status & (DT_TREE_NONFINITE | DT_TREE_TIMEOUT)) ? 0 : n;
    if (a.cost && npop) {
      // the adaptive budget (CaDDTree's stopping rule, section 2.5, in the pop
      // loop, section 3.4): pop i is kept while theta(i) = (1 + Phi(i)) / (C_d +
      // C_v(i)) improves on theta(i - 1), Phi(i) = sum of exp(g) over the first i
      const float cd = a.cost[0];
      float phi = 0.0f, theta = 1.0f / (cd + a.cost[1]);
      int keep = 0;
      for (int i = 0; i < npop; ++i) {
        const float pi = exp_hw(ordered_to_float(__builtin_amdgcn_readlane(e_hi, i)));
        const float th = (1.0f + phi + pi) / (cd + a.cost[2 + i]);
        if (!(th > theta)) break;
        phi += pi;
        theta = th;
        keep = i + 1;
      }
      npop = keep;
    }
    const bool emit = lane < npop;
    const int parent = emit ? 126 - (int)((e_lo >> 19) & 127u) : -1;
    // ancestors by pointer jumping (bit j: node j is this node or above it)
    uint64_t anc = emit ? 1ull << lane : 0ull;
    int up = parent;
    while (__ballot(up >= 0) != 0) {
      const int src = up >= 0 ? up : lane;
      const uint32_t alo = pull((int)(uint32_t)anc, src), ahi = pull((int)(uint32_t)(anc >> 32), src);
      const int nu = pull(up, src);
      if (up >= 0) {
        anc |= ((uint64_t)ahi << 32) | alo;
        up = nu;
      }
    }
    if (wave == 0) {
      const int dep = e_meta & 127, m = (int)((e_lo >> 6) & 63u);
      if (lane < B) {
        otok[lane] = !emit ? -1 : a.compact ? a.cand[ids[(dep - 1) * MP + m]] : ids[(dep - 1) * MP + m];
        opar[lane] = parent;
        odep[lane] = emit ? dep : 0;
        opos[lane] = a.pos_offset + (emit ? dep : 0);
        osc[lane] = emit ? ordered_to_float(e_hi) : NEG_INF;
      }
      ancs[lane] = anc;
      if (lane == 0) {
        o.n_nodes[t] = npop;
        o.status[t] = status;
      }
    }
    lds_barrier();
    if ((B & 3) == 0 && (reinterpret_cast<uintptr_t>(o.mask) & 3) == 0) {
      const int wpr = B >> 2;  // four mask bytes per store
      for (int i = tid; i < B * wpr; i += GT) {
        const int r = i / wpr, c = (i - r * wpr) * 4;
        const uint32_t b4 = (uint32_t)(ancs[r] >> c) & 15u;
        *reinterpret_cast<uint32_t *>(omask + r * B + c) = (b4 * 0x00204081u) & 0x01010101u;
      }
    } else {
      for (int i = tid; i < B * B; i += GT) {
        const int r = i / B, c = i - r * B;
        omask[i] = (uint8_t)((ancs[r] >> c) & 1ull);
      }
    }
  }
}

// The instance that takes d_h with `occ` workgroups per CU (null: none).  fp32
// fragments take twice the registers, so they stay resident up to d_h = 256 only.
template <int ARM>
const void *grow_fn_arm(int wdt, int d_h, int occ) {
  if (wdt == DT_BF16) {
    if (d_h == 64) return (const void *)grow_kernel<uint16_t, 1, 2, 2, ARM>;
    if (d_h == 128) return (const void *)grow_kernel<uint16_t, 1, 4, 2, ARM>;
    if (d_h == 256) return (const void *)grow_kernel<uint16_t, 2, 8, 2, ARM>;
    if (d_h == 512)
      return occ > 1 ? (const void *)grow_kernel<uint16_t, 4, 16, 2, ARM>
                     : (const void *)grow_kernel<uint16_t, 4, 16, 1, ARM>;
    return d_h < 512 ? (const void *)grow_kernel<uint16_t, 4, 0, 1, ARM> : nullptr;
  }
  if (d_h == 64) return (const void *)grow_kernel<float, 1, 2, 2, ARM>;
  if (d_h == 128) return (const void *)grow_kernel<float, 1, 4, 2, ARM>;
  if (d_h == 256) return (const void *)grow_kernel<float, 2, 8, 2, ARM>;
  return d_h < 256 ? (const void *)grow_kernel<float, 2, 0, 1, ARM> : nullptr;
}
const void *grow_fn(int arm, int wdt, int d_h, int occ) {
  if (arm == kMarg) return (const void *)grow_kernel<float, 1, 1, 2, kMarg>;  // (reads no weights)
  return arm == kStatic ? grow_fn_arm<kStatic>(wdt, d_h, occ) : grow_fn_arm<kCond>(wdt, d_h, occ);
}
int grow_members(const dt_plan *p) { return p->scorer == kMarg ? 1 : p->d_h / UW; }

// groups of workgroups resident at once with `occ` per CU
int grow_most(const dt_plan *p, int occ) { return p->num_xcd * (occ * (p->num_cus / p->num_xcd) / grow_members(p)); }

// One workgroup per CU while that gives every tree a group (more registers, and
// nothing to share the CU with: 30.2 against 33.8 us for one tree at d_h = 512);
// two when there are more trees and they fit.
int grow_occ(const dt_plan *p, int batch) { return batch > grow_most(p, 1) && p->grow_occ > 1 ? 2 : 1; }

}  // namespace

// Shapes whose menus and budgets fit a wave (M, B <= 64), whose scan lists the
// register merge takes, and whose W_hh slices stay in registers.
bool grow_fits(const dt_plan *p, int batch) {
  return p->M <= 64 && p->B <= 64 && p->frontier_w == 0 && p->grow_occ > 0 &&
         sel::wave_merge_fits(scan_geom(batch * p->L, p->V, p->M).nchunks, p->M);
}

// how many workgroups of the kernel a CU can hold, at most 2 (0: the shape does not fit)
int grow_max_occ(int arm, int wdt, int d_h, int L, int B, int num_cus, int num_xcd) {
  if (arm != kMarg && d_h / UW > num_cus / num_xcd) return 0;
  const int lds = grow_layout(L, B, arm).total;
  for (int occ = 2; occ > 0; --occ) {
    const void *fn = grow_fn(arm, wdt, d_h, occ);
    int nb = 0;
    if (!fn) return 0;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, GT, (size_t)lds) == hipSuccess && nb >= occ)
      return occ;
    (void)hipGetLastError();
  }
  return 0;
}

int grow_groups(const dt_plan *p, int batch) {
  if (p->scorer == kMarg) return batch;  // (workgroups that wait for no other)
  const int most = grow_most(p, grow_occ(p, batch));
  return batch < most ? batch : most;
}

size_t grow_state_bytes(const dt_plan *p, int batch) {
  const size_t row = p->wdt == DT_BF16 ? State<uint16_t>::row_bytes(p->d_h) : State<float>::row_bytes(p->d_h);
  return (size_t)grow_groups(p, batch) * 2 * CH * row;
}
size_t grow_part_bytes(const dt_plan *p, int batch) {
  return (size_t)grow_groups(p, batch) * 3 * CH * grow_members(p) * MP * sizeof(float);
}

hipError_t launch_grow(const dt_plan *p, int batch, const float *h0, float inv_tau, const Workspace &ws,
                       const dt_tree *out, hipStream_t s, hipEvent_t t0, hipEvent_t t1, int32_t *stats,
                       bool compact) {
  GrowArgs a;
  a.compact = compact;
  a.L = p->L;
  a.M = p->M;
  a.B = p->B;
  a.k = p->k;
  a.G = grow_members(p);
  a.norm_mode = p->norm_mode;
  a.pos_offset = p->pos_offset;
  a.batch = batch;
  a.nchunks = scan_geom(batch * p->L, p->V, p->M).nchunks;
  a.nxcd = p->num_xcd;
  a.ngroups = grow_groups(p, batch);
  a.spin_limit = p->spin_limit > 0 ? p->spin_limit : kGrowSpin;
  a.inv_tau = inv_tau;
  a.c2 = 1.4426950408889634f * inv_tau;
  a.ckeys = ws.chunk_keys;
  a.ctail = ws.chunk_tail;
  a.cflag = ws.chunk_flag;
  a.cand = ws.cand;
  a.candv = ws.candv;
  a.tailR = ws.tail;
  a.rflag = ws.row_flag;
  a.P_all = p->P_all;
  a.U_all = p->U_all;
  a.c_all = p->c_all;
  a.whh = p->whh_t;
  a.b_hh = p->b_hh;
  a.h0 = h0;
  a.states = reinterpret_cast<char *>(ws.states);
  a.part = ws.part;
  a.bar = ws.bar;
  a.stats = stats;
  a.cost = p->cost;
  a.out = *out;
  const size_t lds = (size_t)grow_layout(p->L, p->B, p->scorer).total;
  const void *fn = grow_fn(p->scorer, p->wdt, p->d_h, grow_occ(p, batch));
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int grid = a.nxcd * a.G * ((a.ngroups + a.nxcd - 1) / a.nxcd);
  void *args[] = {&a};
  if (t0)
    e = hipExtLaunchKernel(fn, dim3(grid), dim3(GT), args, lds, s, t0, t1, 0);
  else
    e = hipLaunchKernel(fn, dim3(grid), dim3(GT), args, lds, s);
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace dt
