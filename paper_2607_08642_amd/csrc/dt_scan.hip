// S1: per-depth marginal top-M and the tail log-sum-exp (Alg. 1 step 1;
// section 3.2, candidate restriction).
//
// Each logit row [V] is cut into segments of one or more batches (40 elements
// per thread); a workgroup of W waves streams its segment's batches through
// registers, the next batch always in flight.  Keys are 64-bit (order-preserving
// value bits, ~index), so the order (value desc, id asc) is a plain integer order
// without ties.  Every wave keeps its own list of its 64 R best keys in registers
// (M <= 64 R; entry r * 64 + lane, descending) and merges its own candidates into
// it when they gather -- no block barrier while the segment streams, so a wave
// that merges does not hold up the other waves' loads.  A candidate must beat a
// lower bound on the segment's M-th key:
//   * the bound tb of the first two batches (every wave: the ceil(M/W)-th largest
//     of its 64 lanes' maxima over both, found bit by bit with one ballot each;
//     the minimum over the waves leaves at least M elements at or above it; the
//     one block barrier), ties kept.  Drawn from twice the elements, it admits
//     about 40% fewer candidates over an eight-batch segment of Gaussian-like
//     logits than the first batch's alone;
//   * the wave's own list's M-th value, strictly: the wave's later elements
//     have larger indices, so they lose ties with its own list.
// Both depend on nothing but the data, so the candidates, the merges and the
// order of every tail sum are the same from run to run.  (Reading the other
// waves' list values as they stood was faster -- 40.2 against 43.3 us on 512
// rows of 151936 bf16 logits -- but made the candidates, and with them the
// tails' rounding, depend on timing; reading them two batches late, waiting
// for them, gained nothing over the own bound.)
//   * one pass over a batch's registers sends every element at or below the bound
//     into the running tail sum and the few above it, as (index, value) pairs, to
//     the wave's region of LDS through the comparison's lane mask;
//   * a wave merges once 48 candidates have gathered (64 for longer lists): a
//     bitonic sort of 64 keys, then bitonic merges whose losers join the tail;
//   * the wave lists meet once, at the end of the segment, in a tree.
// A wave whose candidates overflow its region (adversarial rows: long runs of
// equal or monotone values) re-reads the batch and merges as it goes; a first
// batch without a finite bound (mostly -inf or padding) takes every element in
// range as a candidate that way.
//
// Rows need no alignment: a row is read from the 16-byte boundary at or below
// its first element, the elements before it (and past its end) made -inf in
// registers.  Those bytes share a 16-byte granule with the row's own, so the
// loads stay on pages that hold the row.  (Reading such rows element by element
// took 64.6 us for 128 rows of 151937 bf16 at M = 128; see launch_scan_chunks.)
//
// The per-row merge of the segment lists (merge_row_lists and its variants)
// runs inside the expansion kernels, or in a small kernel of its own for
// dt_scan_topm; a row of one segment needs none there (its list is the result).
//
// For Domino's own head the launch carries extra workgroups (blockIdx.x >=
// nchunks) that compute a[row][r] = W_1^H H_row, the half of W_1 [H_d; S] that
// does not depend on the path (section 2.3): a small GEMM of 16 x 16 MFMA
// tiles whose memory time hides under the scan's.
#include "dt_select.h"
#include <hip/hip_ext.h>

#include <type_traits>

namespace dt {

namespace {

using sel::Tail;

constexpr int W = kScanThreads / 64;  // waves of a workgroup

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One 16-rank x 16-row tile of a = W_1^H H (tile = rank tile + (rank tiles) x
// row tile) with fp32 accumulation: the K = d_H columns split over the waves
// in chunks of KC (one MFMA group: lane l holds KC/4 consecutive columns of
// rank (tile row) l % 16 and of H row l % 16, at column group l / 16), the
// wave partials summed in LDS (red: W x 256 floats).  Out-of-range ranks,
// rows and columns read as zeros and are not stored.  bf16: 16x16x32 bf16
// MFMAs on the stored values (exact products); fp32: 16x16x4 fp32 MFMAs.
template <typename TW>
__device__ void head_proj_tile(const HeadProj &p, int rows, int tile, float *red) {
  const int nrt = (p.rank + 15) / 16;
  if (tile >= nrt * ((rows + 15) / 16)) return;  // (whole workgroup)
  const int rt = tile % nrt, qt = tile / nrt;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4;
  const int r = rt * 16 + (lane & 15), q = qt * 16 + (lane & 15);
  const bool rok = r < p.rank, qok = q < rows;
  const TW *wr = static_cast<const TW *>(p.w1) + (size_t)(rok ? r : 0) * p.ld1;
  const TW *hr = static_cast<const TW *>(p.H) + (size_t)(qok ? q : 0) * p.d_H;
  constexpr bool kBf = sizeof(TW) == 2;
  constexpr int KC = kBf ? 32 : 16, KL = KC / 4;  // columns per chunk, per lane
  constexpr int U = 4;                             // chunks in flight per wave
  using V = typename std::conditional<kBf, uint4, float4>::type;  // KL columns
  const int nch = (p.d_H + KC - 1) / KC;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int c0 = w; c0 < nch; c0 += W * U) {
    V av[U], bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (c0 + u * W) * KC + g * KL;  // (d_H % 8 == 0: a lane's KL are all in or out)
      const bool ok = c0 + u * W < nch && k < p.d_H;
      av[u] = (ok && rok) ? *reinterpret_cast<const V *>(wr + k) : V{};
      bv[u] = (ok && qok) ? *reinterpret_cast<const V *>(hr + k) : V{};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (kBf) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[u]),
                                                     __builtin_bit_cast(bf16x8, bv[u]), acc, 0, 0, 0);
      } else {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u].x, bv[u].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u].y, bv[u].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u].z, bv[u].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u].w, bv[u].w, acc, 0, 0, 0);
      }
    }
  }
  // lane l, register i: rank rt*16 + (l/16)*4 + i, row qt*16 + l%16
#pragma unroll
  for (int i = 0; i < 4; ++i) red[w * 256 + lane * 4 + i] = acc[i];
  __syncthreads();
  static_assert(kScanThreads == 256, "one thread per tile element");
  const int e = threadIdx.x, el = e >> 2, ei = e & 3;
  float sum = red[e];
  for (int v = 1; v < W; ++v) sum += red[v * 256 + e];
  const int rr = rt * 16 + (el >> 4) * 4 + ei, qq = qt * 16 + (el & 15);
  if (rr < p.rank && qq < rows) p.a[(size_t)qq * p.rank + rr] = sum;
}

template <typename T>
struct Elem;
template <>
struct Elem<uint16_t> {
  static constexpr int EPL = 8;  // elements per 16-byte load
};
template <>
struct Elem<float> {
  static constexpr int EPL = 4;
};

// The bitwise search for a bound runs down to this bit: a bf16 value's
// order-preserving code is set by its high 16 bits (its low 16 are 0 for a
// value >= 0 and all ones below 0), so 16 steps of one ballot each (a serial
// chain) find the high half of the q-th largest code, and full_code restores
// the low half.
template <typename T>
constexpr int kLowBit = 0;
template <>
constexpr int kLowBit<uint16_t> = 16;
template <typename T>
__device__ inline uint32_t full_code(uint32_t pre) {
  if constexpr (kLowBit<T> == 16) return (pre & 0x80000000u) ? pre : (pre | 0xFFFFu);
  return pre;
}

template <typename T>
__device__ inline float to_f32(T x);
template <>
__device__ inline float to_f32<uint16_t>(uint16_t x) {
  return bf16_to_f32(x);
}
template <>
__device__ inline float to_f32<float>(float x) {
  return x;
}

// Raw registers of one batch: kScanPerThread elements per thread as 16-byte loads
template <typename T>
struct Raw {
  static constexpr int NL = kScanPerThread / Elem<T>::EPL;
  uint4 q[NL];
};

// Issue the loads of batch `b` of a segment (element (j, e) of this thread sits at
// batch offset j*STEP + tid*EPL + e): straight-line 16-byte buffer loads; loads
// past the segment's granules return zeros and cost no traffic, and pad_batch
// makes what lies outside the row -inf.  Nothing waits for the data here.
template <typename T>
__device__ inline void load_batch(Raw<T> &r, __amdgpu_buffer_rsrc_t seg, int b) {
  constexpr int EPL = Elem<T>::EPL;
  constexpr int STEP = W * 64 * EPL;
  int lb = (int)threadIdx.x * EPL;
  asm volatile("" : "+v"(lb));
  const int base = (b * (W * 64 * kScanPerThread) + lb) * (int)sizeof(T);
#pragma unroll
  for (int j = 0; j < Raw<T>::NL; ++j)
    r.q[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                           seg, base + j * STEP * (int)sizeof(T), 0, 0));
}

// 16 bytes with the elements outside [lo, hi) made -inf
template <typename T>
__device__ inline uint4 pad_granule(uint4 q, int lo, int hi) {
  constexpr int PER = 4 / sizeof(T);  // elements per dword
  uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = i * PER;
    if constexpr (PER == 2) {
      if (e < lo || e >= hi) w[i] = (w[i] & 0xFFFF0000u) | 0xFF80u;
      if (e + 1 < lo || e + 1 >= hi) w[i] = (w[i] & 0xFFFFu) | 0xFF800000u;
    } else {
      if (e < lo || e >= hi) w[i] = 0xFF800000u;
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// the elements of a batch before `lo` and from `hi` on become -inf (lo < EPL)
template <typename T>
__device__ inline void pad_batch(Raw<T> &r, int lo, int hi) {
  constexpr int EPL = Elem<T>::EPL;
  constexpr int STEP = W * 64 * EPL;
  constexpr uint32_t ninf = EPL == 8 ? 0xFF80FF80u : 0xFF800000u;
  int lb = (int)threadIdx.x * EPL;
  asm volatile("" : "+v"(lb));
  if (lo > 0 && threadIdx.x == 0) r.q[0] = pad_granule<T>(r.q[0], lo, EPL);
#pragma unroll
  for (int j = 0; j < Raw<T>::NL; ++j) {
    // (whole granules past the end, and the one that holds it)
    if (hi < (j + 1) * STEP) {  // (uniform)
      const int in = hi - j * STEP - lb;
      if (in < EPL) r.q[j] = in <= 0 ? make_uint4(ninf, ninf, ninf, ninf) : pad_granule<T>(r.q[j], 0, in);
    }
  }
}

// Opaque to the compiler: each pass unpacks the elements again (one ALU op each)
// instead of keeping every unpacked value live across the passes.
template <typename T>
__device__ inline void fence_regs(Raw<T> &r) {
#pragma unroll
  for (int j = 0; j < Raw<T>::NL; ++j) asm volatile("" : "+v"(r.q[j].x), "+v"(r.q[j].y), "+v"(r.q[j].z), "+v"(r.q[j].w));
}

// element e of 16-byte load j (unpacked from the raw registers on each use)
template <typename T>
__device__ inline float elem(const Raw<T> &r, int j, int e) {
  const uint4 q = r.q[j];
  if constexpr (Elem<T>::EPL == 8) {
    const uint32_t wd = (e >> 1) == 0 ? q.x : (e >> 1) == 1 ? q.y : (e >> 1) == 2 ? q.z : q.w;
    return (e & 1) ? __uint_as_float(wd & 0xFFFF0000u) : __uint_as_float(wd << 16);
  } else {
    return __uint_as_float(e == 0 ? q.x : e == 1 ? q.y : e == 2 ? q.z : q.w);
  }
}

constexpr int kWaveRegion = 512;  // candidates a wave gathers between merges

__device__ inline uint64_t readlane64(uint64_t v, int l) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
  return ((uint64_t)hi << 32) | lo;
}

// a value slightly below v (v finite): comparing x > below(v) keeps x == v
__device__ inline float below(float v) { return v - (fabsf(v) * 0x1p-20f + 0x1p-126f); }

// merge region[0..n) ((index << 32) | value bits each) into the wave's list.
// fresh: the list is still empty, and the first 64 keys become its head sorted,
// with nothing to merge (wave-uniform; cleared here).
template <int R>
__device__ inline void wave_merge(const uint64_t *region, int n, sel::WaveList<R> &list, bool &fresh, Tail &tail,
                                  float c) {
  const int lane = threadIdx.x & 63;
  for (int c0 = 0; c0 < n; c0 += 64) {
    uint64_t k = 0ull;
    if (c0 + lane < n) {
      const uint64_t e = region[c0 + lane];
      k = make_key(__uint_as_float((uint32_t)e), (uint32_t)(e >> 32));
    }
    const uint64_t srt = sel::wave_sort64(k, fresh);
    if (fresh)
      list.k[0] = srt;
    else
      sel::list_insert<R>(list, srt, tail, c);
    fresh = false;
  }
}

// the results of a row of one segment, written by the scan itself
struct RowOut {
  int32_t *ids;   // null: segment lists
  float *vals, *tail;
  int32_t *flag;
  float inv_tau;
};

// K1: exact top-M of one segment (g.chunk elements from the row's 16-byte
// boundary; the last one takes what is left) of one row, plus the tail of the
// rest.  Also clears `zero_n` ints at `zero_ptr` (barrier counters of the
// expansion kernel that follows on the stream).
// R: list registers per lane; TWP: the weights dtype of a head projection carried by
// the launch (void: none)
template <typename T, int R, typename TWP = void>
__global__ __launch_bounds__(kScanThreads) void scan_kernel(
    const T *__restrict__ logits, ScanGeom g, float c, uint64_t *__restrict__ ckeys,
    float2 *__restrict__ ctail, int32_t *__restrict__ cflag, int32_t *__restrict__ zero_ptr,
    int zero_n, RowOut ro, HeadProj hp) {
  constexpr int EPL = Elem<T>::EPL;
  constexpr int NL = Raw<T>::NL;
  constexpr int STEP = W * 64 * EPL;
  constexpr int BATCH = W * 64 * kScanPerThread;
  constexpr float NINF = -__builtin_huge_valf();
  __shared__ alignas(16) uint64_t regions[W * kWaveRegion];
  __shared__ uint64_t wl[W][R * 64];
  __shared__ float wthr[W];
  __shared__ float2 red[W];
  __shared__ int flag;
  if constexpr (!std::is_void<TWP>::value) {
    static_assert(kWaveRegion * 8 >= 256 * 4, "projection partials fit the regions");
    if ((int)blockIdx.x >= g.nchunks) {
      head_proj_tile<TWP>(hp, g.rows, blockIdx.y * hp.extra + blockIdx.x - g.nchunks,
                          reinterpret_cast<float *>(regions));
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int row = blockIdx.y, seg = blockIdx.x;
  const int M = g.M;
  // the row from the 16-byte boundary at or below its start: `mis` elements early
  const T *rowp = logits + (size_t)row * g.V;
  const int mis = (int)((reinterpret_cast<uintptr_t>(rowp) & 15) / sizeof(T));
  const int seg_lo = seg * g.chunk;
  const int seg_n = (seg == g.nchunks - 1 ? g.V + mis : seg_lo + g.chunk) - seg_lo;
  const int seg_start = seg_lo - mis;  // row index of the segment's element 0
  const int nbat = (seg_n + BATCH - 1) / BATCH;
  const int lo0 = seg == 0 ? mis : 0;  // elements of its first batch before the row
  const T *segp = rowp + seg_start;
  if (zero_ptr && blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = tid; i < zero_n; i += W * 64) zero_ptr[i] = 0;
  const __amdgpu_buffer_rsrc_t segr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T *>(segp), 0, (seg_n * (int)sizeof(T) + 15) & ~15, 0x00020000);
  int lb = tid * EPL;
  asm volatile("" : "+v"(lb));
  Raw<T> ra, rb;
  const bool two = nbat > 1;
  load_batch<T>(ra, segr, 0);
  if (two) load_batch<T>(rb, segr, 1);

  // ---- the first two batches' lower bound tb -----------------------------------
  const int bn0 = min(BATCH, seg_n);
  if (bn0 < BATCH || lo0 > 0) pad_batch<T>(ra, lo0, bn0);
  float tmax = NINF;
#pragma unroll
  for (int j = 0; j < NL; ++j)
#pragma unroll
    for (int e = 0; e < EPL; ++e) tmax = fmaxf(tmax, elem<T>(ra, j, e));
  if (two) {
    const int bn1 = min(BATCH, seg_n - BATCH);
    if (bn1 < BATCH) pad_batch<T>(rb, 0, bn1);
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
      for (int e = 0; e < EPL; ++e) tmax = fmaxf(tmax, elem<T>(rb, j, e));
  }
  {
    const int q = (M + W - 1) / W;  // <= 64 since M <= 256 and W >= 4
    const uint32_t code = ordered_bits(tmax);
    uint32_t pre = 0;
#pragma unroll
    for (int bit = 31; bit >= kLowBit<T>; --bit) {
      const uint32_t cand = pre | (1u << bit);
      if (__popcll(__ballot(code >= cand)) >= q) pre = cand;
    }
    pre = full_code<T>(pre);
    if (lane == 0) wthr[w] = ordered_to_float(pre);
  }
  __syncthreads();
  float tb = wthr[0];
#pragma unroll
  for (int i = 1; i < W; ++i) tb = fminf(tb, wthr[i]);
  // (a bound of +inf -- ceil(M/W) lanes of every wave hold one -- lets nothing through
  // that would show it: flagged here, the rest of the row's results unspecified.  The
  // flag's other writers come after the barriers below.)
  if (tid == 0) flag = tb == -NINF;
  const bool all_in = !(tb > NINF);
  const float tlow = all_in ? NINF : below(tb);
  // The tail's reference follows the bound, which every element the tail
  // takes lies at or below, not the segment's maximum: at a small
  // temperature (c large) the tail's terms against the maximum of the
  // candidates would all underflow.
  Tail tail = sel::tail_empty();
  tail.m = fmaxf(tlow, -3.402823466e38f);

  sel::WaveList<R> list;       // this wave's best keys
#pragma unroll
  for (int r = 0; r < R; ++r) list.k[r] = 0ull;
  bool fresh = true;      // no merge yet (the list is empty)
  float v_own = NINF;     // its M-th value once it holds M keys
  int wpos = 0;           // candidates in the region (wave-uniform)
  const int kMergeTrig = R > 1 ? 64 : (M < 16 ? 2 * M : 48);
  uint64_t *region = regions + w * kWaveRegion;

  auto merge_now = [&]() {
    wave_merge<R>(region, wpos, list, fresh, tail, c);
    wpos = 0;
    uint64_t km = 0ull;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r == (M - 1) >> 6) km = readlane64(list.k[r], (M - 1) & 63);
    if (km) v_own = key_value(km);
  };
  // the candidates of batch b read again from memory, merged whenever the
  // region might overflow (the tail already holds the batch's other elements)
  auto slow = [&](int bstart, int lo, int bn, float te, bool in_all) {
#pragma unroll 1
    for (int k = 0; k < NL * EPL; ++k) {
      const int off = lb + (k / EPL) * STEP + k % EPL;
      const bool in = off >= lo && off < bn;
      const float x = in ? to_f32<T>(segp[bstart + off]) : NINF;
      const bool pass = in && (x > te || (in_all && x == NINF));
      if (in_all && in && x != x) tail.s = x;  // (a NaN: the row is flagged)
      const uint64_t bal = __ballot(pass);
      if (bal) {
        if (wpos + 64 > kWaveRegion) merge_now();
        const int at = wpos + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
        if (pass)
          region[at] = ((uint64_t)(uint32_t)(seg_start + bstart + off) << 32) | __float_as_uint(x);
        wpos += __popcll(bal);
      }
    }
  };

  auto process = [&](Raw<T> &raw, int b) {
    const int bstart = b * BATCH;
    const int bn = min(BATCH, seg_n - bstart);
    const int lo = b == 0 ? lo0 : 0;
    if (b > 0 && bn < BATCH) pad_batch<T>(raw, 0, bn);
    // this batch's bound
    float te = tlow;
    if (b > 0) te = fmaxf(te, v_own);
    // every element that cannot enter is <= te: keep the tail's reference above it
    if (te > tail.m) {
      tail.s *= sel::fast_exp2((tail.m - te) * c);
      tail.m = te;
    }
    if (b == 0 && all_in) {
      slow(bstart, lo, bn, NINF, true);
    } else {
      fence_regs<T>(raw);
      const int wprev = wpos;
      const int ibase = seg_start + bstart + lb;  // row index of this thread's element (0, 0)
      // exp((x - m) / tau) = 2^((x - m) c) for every element; a candidate (x >
      // te, rare) is appended to the region and adds nothing.  While |m c| <= 128
      // the exponent is one fma, x c - (m c), off by at most half an ulp of m c
      // (2^-17, the same for every term); otherwise two operations.
      auto tail_pass = [&](auto expo) {
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < NL; ++j)
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            float x = elem<T>(raw, j, e);
            const bool pass = x > te;
            const uint64_t bal = __ballot(pass);
            if (__builtin_expect(bal != 0, 0)) {
              // (past the region's end the last slot is overwritten: the
              // overflow below discards this batch's entries)
              const int at = min(wpos + (int)__builtin_amdgcn_mbcnt_hi(
                                            (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0)),
                                 kWaveRegion - 1);
              if (pass)
                region[at] = ((uint64_t)(uint32_t)(ibase + j * STEP + e) << 32) | __float_as_uint(x);
              wpos += __popcll(bal);
              x = pass ? NINF : x;
            }
            s += sel::fast_exp2(expo(x));
            // (group by group: the sum pinned here keeps the scheduler from
            // holding every converted element at once)
            if (e == EPL - 1) asm volatile("" : "+v"(s));
          }
        tail.s += s;
      };
      const float m = tail.m, mc = m * c;
      if (fabsf(mc) <= 128.0f)
        tail_pass([=](float x) { return __builtin_fmaf(x, c, -mc); });
      else
        tail_pass([=](float x) { return (x - m) * c; });
      if (wpos > kWaveRegion) {
        // overflow: merge what came before, then this batch's candidates again
        wpos = wprev;
        if (wpos) merge_now();
        slow(bstart, lo, bn, te, false);
      }
    }
    if (wpos >= kMergeTrig || (wpos && b == nbat - 1)) merge_now();
  };

  // a buffer is refilled with the batch two ahead as soon as it is processed
  // (loads past the segment's end return zeros and cost no traffic; a third
  // buffer measured slower: 43.2 against 40.0 us on 512 rows of 151936 bf16)
  for (int b = 0; b < nbat; b += 2) {
    process(ra, b);
    if (b + 2 < nbat) load_batch<T>(ra, segr, b + 2);
    if (b + 1 < nbat) {
      process(rb, b + 1);
      if (b + 3 < nbat) load_batch<T>(rb, segr, b + 3);
    }
  }

  // ---- the wave lists meet, pairs side by side: the segment's M best, the rest
  // to the tail
#pragma unroll
  for (int s = 1; s < W; s <<= 1) {
    if ((w & (2 * s - 1)) == s)
#pragma unroll
      for (int r = 0; r < R; ++r) wl[w][r * 64 + lane] = list.k[r];
    __syncthreads();
    if ((w & (2 * s - 1)) == 0) sel::list_merge<R>(list, [&](int i) { return wl[w + s][i]; }, tail, c);
  }
  const size_t cidx = (size_t)row * g.nchunks + seg;
  if (w == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = r * 64 + lane;
      uint64_t f = list.k[r];
      if (p >= M) {
        if (f) sel::tail_add1(tail, key_value(f), c);
        f = 0ull;
      } else if (ro.ids) {
        ro.ids[(size_t)row * M + p] = f ? (int32_t)key_index(f) : -1;
        ro.vals[(size_t)row * M + p] = f ? key_value(f) : NINF;
      } else {
        ckeys[cidx * M + p] = f;
      }
      // +inf heads the list
      if (r == 0 && lane == 0 && f && key_value(f) == __builtin_huge_valf()) atomicOr(&flag, 1);
    }
  }
  // a NaN makes a tail sum NaN (it never passes a comparison)
  if (!(tail.s == tail.s)) atomicOr(&flag, 1);
  const Tail t = sel::block_tail<W * 64>(tail, c, red);
  if (tid == 0) {
    const int fl = flag ? DT_TREE_NONFINITE : 0;
    if (ro.ids) {
      ro.tail[row] = t.s > 0.0f ? t.m * ro.inv_tau + logf(t.s) : NINF;
      ro.flag[row] = fl;
    } else {
      ctail[cidx] = make_float2(t.m, t.s);
      cflag[cidx] = fl;
    }
  }
}

// K2 (dt_scan_topm and one-shot calls): merge the chunk lists of one row
template <int R, bool SHIFT>
__global__ __launch_bounds__(kScanThreads) void scan_merge_kernel(
    ScanGeom g, float c, float inv_tau, const uint64_t *__restrict__ ckeys,
    const float2 *__restrict__ ctail, const int32_t *__restrict__ cflag, int32_t *__restrict__ cand,
    float *__restrict__ candv, float *__restrict__ tailR, int32_t *__restrict__ rflag) {
  __shared__ uint64_t xbuf[kScanThreads * R];
  __shared__ float2 red[kScanThreads / 64];
  __shared__ int flag;
  const int row = blockIdx.x;
  sel::merge_row_lists<false, kScanThreads, R, SHIFT>(
      ckeys + (size_t)row * g.nchunks * g.M, g.nchunks, g.M, ctail + (size_t)row * g.nchunks,
      cflag + (size_t)row * g.nchunks, c, inv_tau, xbuf, red, &flag, cand + (size_t)row * g.M,
      candv + (size_t)row * g.M, tailR + row, rflag + row, nullptr);
}

}  // namespace

ScanGeom scan_geom(int rows, int V, int M) {
  ScanGeom g;
  g.rows = rows;
  g.V = V;
  g.M = M;
  // segments of sb batches: the fewest rounds of kScanSlots resident
  // workgroups (each round pays a workgroup's start-up latency once; within a
  // round the scan streams at the memory's rate whatever the split), then the
  // shortest segments that keep it (the most workgroups in flight)
  const int nb = (V + kScanChunk - 1) / kScanChunk;
  auto rounds = [&](int t) { return ((long long)rows * ((nb + t - 1) / t) + kScanSlots - 1) / kScanSlots; };
  const long long fewest = rounds(nb);
  int sb = 1;
  while (sb < nb && rounds(sb) > fewest) ++sb;
  g.chunk = sb * kScanChunk;
  g.nchunks = (V + g.chunk - 1) / g.chunk;
  return g;
}

size_t row_bound_bytes(const ScanGeom &g) { return (size_t)sel::row_bound_bytes(g.nchunks, g.M); }

size_t scan_bytes(const ScanGeom &g) {
  size_t b = 0;
  const size_t rc = (size_t)g.rows * g.nchunks;
  b += align_up(rc * g.M * sizeof(uint64_t), 256);
  b += align_up(rc * sizeof(float2), 256);
  b += align_up(rc * sizeof(int32_t), 256);
  b += align_up((size_t)g.rows * g.M * sizeof(int32_t), 256);
  b += align_up((size_t)g.rows * g.M * sizeof(float), 256);
  b += align_up((size_t)g.rows * sizeof(float), 256);
  b += align_up((size_t)g.rows * sizeof(int32_t), 256);
  return b;
}

size_t carve_scan(char *base, const ScanGeom &g, Workspace *ws) {
  size_t o = 0;
  const size_t rc = (size_t)g.rows * g.nchunks;
  ws->chunk_keys = reinterpret_cast<uint64_t *>(base + o);
  o += align_up(rc * g.M * sizeof(uint64_t), 256);
  ws->chunk_tail = reinterpret_cast<float2 *>(base + o);
  o += align_up(rc * sizeof(float2), 256);
  ws->chunk_flag = reinterpret_cast<int32_t *>(base + o);
  o += align_up(rc * sizeof(int32_t), 256);
  ws->cand = reinterpret_cast<int32_t *>(base + o);
  o += align_up((size_t)g.rows * g.M * sizeof(int32_t), 256);
  ws->candv = reinterpret_cast<float *>(base + o);
  o += align_up((size_t)g.rows * g.M * sizeof(float), 256);
  ws->tail = reinterpret_cast<float *>(base + o);
  o += align_up((size_t)g.rows * sizeof(float), 256);
  ws->row_flag = reinterpret_cast<int32_t *>(base + o);
  o += align_up((size_t)g.rows * sizeof(int32_t), 256);
  return o;
}

// hipLaunchKernelGGL, or hipExtLaunchKernelGGL with start and end events
template <typename F, typename... Args>
static void launch_maybe_timed(F kernel, dim3 grid, dim3 block, uint32_t lds, hipStream_t s,
                               hipEvent_t t0, hipEvent_t t1, Args... args) {
  if (t0)
    hipExtLaunchKernelGGL(kernel, grid, block, lds, s, t0, t1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
}

template <typename T, int R, typename TWP>
static void launch_scan_k(const T *p, const ScanGeom &g, float c, const Workspace &ws, int32_t *zero_ptr,
                          int zero_n, const RowOut &ro, const HeadProj *hp, hipStream_t s, hipEvent_t t0,
                          hipEvent_t t1) {
  launch_maybe_timed(scan_kernel<T, R, TWP>, dim3(g.nchunks + (hp ? hp->extra : 0), g.rows), dim3(kScanThreads), 0, s,
                     t0, t1, p, g, c, ws.chunk_keys, ws.chunk_tail, ws.chunk_flag, zero_ptr, zero_n, ro,
                     hp ? *hp : HeadProj{});
}

template <typename T, int R>
static void launch_scan_t(const T *p, const ScanGeom &g, float c, const Workspace &ws, int32_t *zero_ptr,
                          int zero_n, const RowOut &ro, const HeadProj *hp, hipStream_t s, hipEvent_t t0,
                          hipEvent_t t1) {
  if (hp && hp->wdt == DT_BF16)
    launch_scan_k<T, R, uint16_t>(p, g, c, ws, zero_ptr, zero_n, ro, hp, s, t0, t1);
  else if (hp)
    launch_scan_k<T, R, float>(p, g, c, ws, zero_ptr, zero_n, ro, hp, s, t0, t1);
  else
    launch_scan_k<T, R, void>(p, g, c, ws, zero_ptr, zero_n, ro, nullptr, s, t0, t1);
}

HeadProj head_proj_args(const dt_plan *p, int rows, const void *H, const dt_domino_head &hd, float *a_out) {
  HeadProj h;
  h.w1 = hd.w1;
  h.H = H;
  h.a = a_out;
  h.d_H = hd.d_H;
  h.ld1 = hd.d_H + p->d_h;
  h.rank = hd.rank;
  h.wdt = p->wdt;
  const int tiles = ((hd.rank + 15) / 16) * ((rows + 15) / 16);
  h.extra = (tiles + rows - 1) / rows;
  return h;
}

// One kernel for every row address, row length and M: the register list grows
// with M (one register per lane for each 64).  A kernel of its own per block for
// M > 64, reading rows that are not 16-byte aligned element by element, took
// 64.6 us for 128 rows of 151937 bf16 at M = 128, this one 19.8 (with the rows'
// merge, dt_scan_topm 87.7 -> 23.6 us); aligned rows at M = 64 run as before (512 rows of 151936
// bf16: 39 us).  direct: rows of one segment give their results here.
hipError_t launch_scan_chunks(const void *logits, int ldt, const ScanGeom &g, float inv_tau,
                              const Workspace &ws, int32_t *zero_ptr, int zero_n, hipStream_t s,
                              hipEvent_t t0, hipEvent_t t1, const HeadProj *hp, bool direct) {
  const float c = 1.4426950408889634f * inv_tau;  // exp(x / tau) = exp2(x * c)
  const RowOut ro = direct ? RowOut{ws.cand, ws.candv, ws.tail, ws.row_flag, inv_tau}
                           : RowOut{nullptr, nullptr, nullptr, nullptr, 0.0f};
  auto launch = [&](auto *p) {
    if (g.M <= 64)
      launch_scan_t<std::remove_cv_t<std::remove_pointer_t<decltype(p)>>, 1>(p, g, c, ws, zero_ptr, zero_n, ro, hp, s, t0, t1);
    else if (g.M <= 128)
      launch_scan_t<std::remove_cv_t<std::remove_pointer_t<decltype(p)>>, 2>(p, g, c, ws, zero_ptr, zero_n, ro, hp, s, t0, t1);
    else
      launch_scan_t<std::remove_cv_t<std::remove_pointer_t<decltype(p)>>, 4>(p, g, c, ws, zero_ptr, zero_n, ro, hp, s, t0, t1);
  };
  if (ldt == DT_BF16)
    launch(static_cast<const uint16_t *>(logits));
  else
    launch(static_cast<const float *>(logits));
  return hipGetLastError();
}

hipError_t launch_scan_merge(const ScanGeom &g, float inv_tau, const Workspace &ws, hipStream_t s, bool shift) {
  const float c = 1.4426950408889634f * inv_tau;
  const auto kernel = g.M <= 64    ? (shift ? scan_merge_kernel<1, true> : scan_merge_kernel<1, false>)
                      : g.M <= 128 ? (shift ? scan_merge_kernel<2, true> : scan_merge_kernel<2, false>)
                                   : (shift ? scan_merge_kernel<4, true> : scan_merge_kernel<4, false>);
  hipLaunchKernelGGL(kernel, dim3(g.rows), dim3(kScanThreads), 0, s, g, c, inv_tau, ws.chunk_keys, ws.chunk_tail,
                     ws.chunk_flag, ws.cand, ws.candv, ws.tail, ws.row_flag);
  return hipGetLastError();
}

}  // namespace dt
