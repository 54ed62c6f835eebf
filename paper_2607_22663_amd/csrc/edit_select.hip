// Confidence-based edit selection over vocabulary logits, gfx950.
//
// Paper, Sec. "Configurable threshold decoding", Eq. (1): per position, the
// prediction is the highest-probability token and its confidence is that
// probability; a visible token is overwritten (the token-to-token set) when
// the prediction differs from it and the confidence clears the threshold.
// MBE keeps this rule for its cross-block passes (Sec. "Training-Free MBE
// Decoding").  Ties go to the lowest index; the test is conf >= threshold.
//
// One HBM pass per row.  Each workgroup (256 threads) reduces one chunk of a
// row; each thread streams 16-byte bf16 vectors (the next iteration's two
// loads in flight while the current one is reduced) and keeps
//   m       its running maximum,
//   s       sum of 2^(x log2(e) - mc), mc = m log2(e) rounded to fp32,
//           rescaled when m grows,
//   it_max  the iteration where m was first reached.
// The exponent is one FMA per element.  Every exponent is off by the same
// delta = m log2(e) - mc (the rounding residual of mc), so the confidence of
// the maximum is 2^delta / s, and the entropy, which does not depend on the
// reference, needs no correction.
// Elements of one thread are visited in increasing index order, so its first
// occurrence of m lies in iteration it_max.  Threads merge (max, rescaled
// sum) in a fixed tree; then only the threads whose own maximum equals the
// chunk maximum re-read their iteration it_max to find its first index, and a
// min over the workgroup picks the lowest.  This keeps the argmax bookkeeping
// out of the per-element loop at the cost of a few cache lines per chunk.
//
// What bounds it: HBM, with the VALU close behind (64 logits cost about 32
// cycles of a SIMD, half of them the exponential, 36 with the entropy; at
// 6.8 TB/s a SIMD has 40).  So the loop keeps no per-iteration copies (two
// register sets in turn; one where that is better, see the launch) and forms
// the reference only when the maximum moves: 2048 x 131072 with entropy 91.5 ->
// 86.3 us for the whole update, 512 x 131072 without 25.3 -> 22.8 us, 8192 x
// 131072 312.9 -> 311.0 us (6.90 TB/s).
// Every row takes 16-byte loads wherever it starts (its up to 7 logits before
// and after the 16-byte grid are read one per thread): 992 rows of 100003
// packed behind each other, with entropy, 276.7 -> 48.4 us; and an iteration
// that is not whole no longer sends the chunk through a second pass: 1024 x
// 32000 39.8 -> 34.2 us.
// Rows split over several workgroups (few rows) write partials that are merged
// in a fixed order by the next kernel (a small one of their own for edit
// selection, the per-block step for the update), so results are bitwise
// reproducible.
#include <hip/hip_runtime.h>
#include <cfloat>
#include <stdint.h>

#include <type_traits>

#include "internal.h"

namespace mbe {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Logits in global memory: said in the type, since an address made from a
// row's start and its offset on the 16-byte grid would otherwise be loaded
// with flat instructions.
typedef const __attribute__((address_space(1))) uint16_t g_bf16;

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kU = kEsVecPerThread;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_at(g_bf16 *p) {
  return __uint_as_float(static_cast<uint32_t>(*p) << 16);
}

// Exponent arguments below this are exactly 0 after exp2 in fp32.  The
// entropy sum adds 2^y * y; a -inf logit would add 0 * (-inf).  The main pass
// does not clamp; a NaN sum sends the chunk through a second pass that clamps
// y here (only rows holding -inf logits take it).
constexpr float kYMin = -256.f;

// The reference of a running maximum m: m log2(e) rounded to fp32.  All sums
// are kept relative to it.  The product is formed by its own instruction:
// fused into a following subtraction (d = ref(m) - ref(M)) it would lose the
// rounding that the sums were accumulated against.  Kept finite: for logits
// near the type's lowest value (rows masked with it instead of -inf) the
// product overflows, and a thread that had met only such logits would hold an
// infinite sum, which no later maximum rescales to 0.  Its terms are 0
// relative to the finite reference.
__device__ __forceinline__ float ref_raw(float m) {
  float r;
  asm("v_mul_f32 %0, %1, %2" : "=v"(r) : "v"(m), "v"(kLog2e));
  return r;
}
__device__ __forceinline__ float at_least_lowest(float r) {
  float f;      // (fmaxf would quiet the product first, one more instruction)
  asm("v_max_f32 %0, %1, %2" : "=v"(f) : "v"(r), "v"(-FLT_MAX));
  return f;
}
__device__ __forceinline__ float ref_of(float m) { return at_least_lowest(ref_raw(m)); }

// max(a, b, c) in one instruction.  fmaxf would first quiet every input
// (one more instruction each): the compiler cannot tell that floats made
// from bf16 bits by shifts are not signalling NaNs.  NaN logits are outside
// the contract; -inf is handled like any value.
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Merge partial (m, s, t) with (m2, s2, t2): the sums are rescaled to the
// common max M.  With d = ref(m) - ref(M): s -> 2^d s, t -> 2^d (t + d s).
template <bool ENT>
__device__ __forceinline__ void merge_ms(float &m, float &s, float &t, float m2, float s2, float t2) {
  const float M = fmaxf(m, m2);
  if (M == -INFINITY) return;     // both empty so far
  float a = 0.f, b = 0.f, ta = 0.f, tb = 0.f;
  // (the product by a positive constant keeps the order, so the larger of the
  // two references is ref_of(M))
  const float r = ref_raw(m), r2 = ref_raw(m2), rM = max3(r, r2, -FLT_MAX);
  // (without the entropy sum an overflowed reference, of a sum that is 0, may
  // stay: d = -inf, f = 0)
  if (m != -INFINITY) {
    const float d = (ENT ? at_least_lowest(r) : r) - rM;
    const float f = __builtin_amdgcn_exp2f(d);
    a = s * f;
    if (ENT) ta = f * __builtin_fmaf(d, s, t);
  }
  if (m2 != -INFINITY) {
    const float d = (ENT ? at_least_lowest(r2) : r2) - rM;
    const float f = __builtin_amdgcn_exp2f(d);
    b = s2 * f;
    if (ENT) tb = f * __builtin_fmaf(d, s2, t2);
  }
  s = a + b;
  if (ENT) t = ta + tb;
  m = M;
}

// Merge partial (m, s, t, i) with (m2, s2, t2, i2): larger max wins, equal
// maxima keep the lower index.
template <bool ENT>
__device__ __forceinline__ void merge(float &m, float &s, float &t, int32_t &i, float m2, float s2, float t2,
                                      int32_t i2) {
  i = (m > m2) ? i : ((m2 > m) ? i2 : min(i, i2));
  merge_ms<ENT>(m, s, t, m2, s2, t2);
}

// Entropy in nats from s = sum 2^y and t = sum 2^y y:
// H = -sum p ln p with p = 2^y / s, i.e. ln 2 (log2 s - t / s).
__device__ __forceinline__ float entropy_nats(float s, float t) {
  return 0.69314718055994531f * (log2f(s) - t / s);
}

// Maximum of the 8 kU logits of one iteration, three at a time (a tree of
// about 4 kU three-input maxima).
__device__ __forceinline__ float max_iter(const float (&x)[kU][8]) {
  constexpr int N = 8 * kU;
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = x[i / 8][i % 8];
  int n = N;
#pragma unroll
  for (int level = 0; level < 8; ++level) {
    if (n == 1) break;
    int m = 0;
#pragma unroll
    for (int i = 0; i < N; i += 3) {
      if (i >= n) break;
      if (i + 2 < n) v[m] = max3(v[i], v[i + 1], v[i + 2]);
      else if (i + 1 < n) v[m] = max3(v[i], v[i + 1], v[i + 1]);
      else v[m] = v[i];
      ++m;
    }
    n = m;
  }
  return v[0];
}

__device__ __forceinline__ uint32_t load16b(g_bf16 *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Eight bf16 logits of one 16-byte vector as floats.
__device__ __forceinline__ void unpack8(const u32x4 &w, float x[8]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    x[2 * k] = bf16_lo(w[k]);
    x[2 * k + 1] = bf16_hi(w[k]);
  }
}

// Streaming load of one 16-byte vector: each logit is read once, so it is
// not kept in cache.
__device__ __forceinline__ u32x4 load16(g_bf16 *grid, int64_t unit) {
  return __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4 *)(grid + unit * 8));
}

// Vector unit `unit` (elements 8*unit .. 8*unit+7 from `grid`) as 8 floats.
// VEC: one 16-byte load of a whole unit.  Otherwise (logits on an odd address)
// one logit at a time; elements at or beyond `end` read as -inf.
template <bool VEC>
__device__ __forceinline__ void load_unit(g_bf16 *grid, int64_t unit, int64_t end, float x[8]) {
  if constexpr (VEC) {
    unpack8(load16(grid, unit), x);
  } else {
    const int64_t e0 = unit * 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = (e0 + k < end) ? bf16_at(grid + e0 + k) : -INFINITY;
  }
}

// it_max of a thread whose maximum is its logit of the row's head or tail
constexpr int32_t kHeadIter = -2, kTailIter = -3;

// The token-to-token decision for one row from its (max, argmax, sum), or,
// for the threshold update, the row's prediction, confidence and entropy.
template <bool ENT>
__device__ __forceinline__ void decide(const EsParams &p, int64_t row, float m, float s, float t, int32_t idx) {
  // the maximum's own term is 2^delta, delta = m log2(e) - ref(m) exactly
  // (0 when the product is exact, e.g. on a constant row of small integers)
  const float delta = __builtin_fmaf(m, kLog2e, -ref_of(m));
  const float conf = (delta == 0.f ? 1.0f : __builtin_amdgcn_exp2f(delta)) / s;   // correctly rounded division
  if (p.update) {
    p.pred[row] = idx;
    p.conf[row] = (m == -INFINITY) ? __builtin_nanf("") : conf;
    if (ENT) p.entropy[row] = entropy_nats(s, t);
    return;
  }
  const int32_t cur = p.cur[row];
  const bool change = (m != -INFINITY) && (idx != cur) && (conf >= p.threshold);
  p.conf[row] = (m == -INFINITY) ? __builtin_nanf("") : conf;
  p.new_tokens[row] = change ? idx : cur;
  p.changed[row] = change ? 1 : 0;
}

// DEEP: the next iteration is requested before the current one is unpacked (two
// register sets in turn, two iterations in flight), otherwise after it.
template <bool VEC, bool ENT, int kT, bool DEEP>
__global__ __launch_bounds__(kT) void edit_select_kernel(EsParams p) {
  __shared__ float sh_m[kT / 64];
  __shared__ float sh_s[kT / 64];
  __shared__ float sh_t[kT / 64];
  __shared__ int32_t sh_i[kT / 64];
  if (p.changed_count && blockIdx.x == 0 && threadIdx.x == 0) *p.changed_count = 0;   // counted per block later
  if (p.gate && *p.gate == 0) return;     // gated off: the block step keeps every row

  const int64_t wg = blockIdx.x;
  const int64_t row = wg / p.chunks;
  const int32_t chunk = static_cast<int32_t>(wg % p.chunks);
  const int tid = threadIdx.x;
  g_bf16 *rowp = (g_bf16 *)(p.logits) + row * p.ld;
  // Units of 8 logits on the 16-byte grid of the addresses.  A row that starts
  // off the grid (an odd vocabulary with packed rows, a padded stride, a view)
  // has a head of up to 7 logits before its first whole unit, and any row a
  // tail of up to 7 after its last.  Both are read one logit per thread (by
  // the first and the last chunk), the units between with vector loads, and
  // no load leaves the row.
  const int off = VEC ? static_cast<int>((reinterpret_cast<uintptr_t>(p.logits + row * p.ld) >> 1) & 7) : 0;
  g_bf16 *grid = rowp - off;                          // dereferenced inside the row only
  const int64_t g_end = p.vocab + off;                // row's end on the grid
  const bool last = chunk + 1 == p.chunks;
  const int head = VEC && off != 0 && chunk == 0 ? static_cast<int>(min(static_cast<int64_t>(8 - off), p.vocab)) : 0;
  const int tail = VEC && last && (g_end >= 8 || off == 0) ? static_cast<int>(g_end & 7) : 0;
  const int64_t tail0 = g_end - tail - off;           // the tail's first index
  const int64_t chunk_units = p.chunk_len / 8;
  const int64_t u0 = chunk * chunk_units + (head ? 1 : 0);
  const int64_t u1 = last ? (VEC ? g_end / 8 : (g_end + 7) / 8) : (chunk + 1) * chunk_units;
  const int64_t c1 = min(g_end, u1 * 8);              // end of the units' logits on the grid

  // This thread's logit of the head and of the tail, if it has one (otherwise
  // the row's first, whose page is read anyway): requested before the first
  // vectors by every workgroup (a branch around the loads would wait for them
  // in it) and used after them.  Relaxed atomic loads stay where they are
  // written; every address lies in the row.
  uint32_t raw_h = 0, raw_t = 0;
  if constexpr (VEC) {
    raw_h = load16b(rowp + (tid < head ? tid : 0));
    raw_t = load16b(rowp + (tid < tail ? tail0 + tid : 0));
  }

  float m = -INFINITY, s = 0.f, t = 0.f;
  float nref = 0.f;      // -ref_of(m), 0 while m is -inf
  int32_t it_max = -1;
  int32_t it = 0;
  // A new maximum, found at `mark`: the sums so far relative to it.
  auto raise = [&](float top, int32_t mark) {
    const float ref = ref_of(top);
    if (m != -INFINITY) {
      const float d = -nref - ref;
      const float f = __builtin_amdgcn_exp2f(d);
      if (ENT) t = f * __builtin_fmaf(d, s, t);
      s *= f;
    } else if (ENT) {     // only -inf so far, whose terms made t NaN (0 * -inf)
      s = 0.f;
      t = 0.f;
    }
    m = top;
    nref = -ref;
    it_max = mark;
  };
  // One iteration's 16 logits of this thread into the running (m, s, t).
  auto accumulate = [&](const float (&x)[kU][8], auto clamp) {
    const float cm = max_iter(x);
    if (cm > m) raise(cm, it);
    float acc = 0.f, acct = 0.f;
#pragma unroll
    for (int j = 0; j < kU; ++j)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float y = __builtin_fmaf(x[j][k], kLog2e, nref);
        if constexpr (decltype(clamp)::value) y = fmaxf(y, kYMin);
        const float e = __builtin_amdgcn_exp2f(y);
        acc += e;
        if (ENT) acct = __builtin_fmaf(e, y, acct);
      }
    s += acc;
    if (ENT) t += acct;
  };
  // The whole chunk, the next iteration's loads issued before the current
  // one is summed.
  auto pass = [&](auto clamp) {
    m = -INFINITY;
    s = 0.f;
    t = 0.f;
    nref = 0.f;
    it_max = -1;
    it = 0;
    constexpr int32_t per_iter = kT * kU;
    // a thread's one logit of the head (visited first: the row's lowest
    // indices) or of the tail (visited last)
    auto single = [&](float x, int32_t mark) {
      // (a NaN counts as a maximum below every logit, so that a thread that
      // holds nothing else does not lose it in the merge)
      const float top = x == x ? x : -FLT_MAX;
      if (top > m) raise(top, mark);
      if (x != -INFINITY) {
        float y = __builtin_fmaf(x, kLog2e, nref);
        if (ENT) y = fmaxf(y, kYMin);    // (the type's lowest value overflows here: 0 * -inf)
        const float e = __builtin_amdgcn_exp2f(y);
        s += e;
        if (ENT) t = __builtin_fmaf(e, y, t);
      }
    };
    if constexpr (VEC) {
      // Iterations 0 .. n - 1 of per_iter units, the last perhaps of fewer.  A
      // request past the last unit reads the last one again, so that
      // every request is unconditional (the compiler would otherwise wait for
      // all loads in flight where a skipped request and a made one meet).
      const int32_t units = static_cast<int32_t>(max(u1 - u0, static_cast<int64_t>(0)));
      const int32_t n_full = units / per_iter, n = (units + per_iter - 1) / per_iter;
      u32x4 wa[kU], wb[kU];
      // 32-bit byte offsets from the chunk's start (a row is below 4 GB): 87
      // instructions an iteration instead of 93 with 64-bit unit indices.
      const __attribute__((address_space(1))) char *base = (const __attribute__((address_space(1))) char *)(grid + u0 * 8);
      const uint32_t last_off = static_cast<uint32_t>(units - 1) * 16u;
      auto request = [&](u32x4 (&w)[kU], int32_t i) {
        const uint32_t at = (static_cast<uint32_t>(i) * per_iter + tid) * 16u;
#pragma unroll
        for (int j = 0; j < kU; ++j)
          w[j] = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4 *)(base + min(at + j * kT * 16u, last_off)));
      };
      auto reduce_iter = [&](const u32x4 (&w)[kU], auto partial) {
        float x[kU][8];
#pragma unroll
        for (int j = 0; j < kU; ++j) {
          unpack8(w[j], x[j]);
          if constexpr (decltype(partial)::value) {
            if (it * per_iter + j * kT + tid >= units) {
#pragma unroll
              for (int k = 0; k < 8; ++k) x[j][k] = -INFINITY;
            }
          }
        }
        // clamped with entropy only: the missing units' -inf must not reach its
        // sum.  Without, a clamp would turn a NaN logit into probability 0.
        if constexpr (ENT && decltype(partial)::value) accumulate(x, std::true_type{});
        else accumulate(x, clamp);
        ++it;
      };
      if (n > 0) request(wa, 0);
      if (tid < head) single(bf16_lo(raw_h), kHeadIter);
      if constexpr (DEEP) {
        while (it + 2 <= n_full) {       // the register sets in turn, so that no vector is copied
          request(wb, it + 1);
          reduce_iter(wa, std::false_type{});
          request(wa, it + 1);
          reduce_iter(wb, std::false_type{});
        }
        while (it < n) {      // at most one whole iteration and one partial one, in one body
          request(wb, it + 1);
          reduce_iter(wa, std::true_type{});
#pragma unroll
          for (int j = 0; j < kU; ++j) wa[j] = wb[j];
        }
      } else {
        while (it < n_full) {
          float x[kU][8];
#pragma unroll
          for (int j = 0; j < kU; ++j) unpack8(wa[j], x[j]);
          request(wa, it + 1);
          accumulate(x, clamp);
          ++it;
        }
        if (it < n) reduce_iter(wa, std::true_type{});
      }
      if (tid < tail) single(bf16_lo(raw_t), kTailIter);
    } else {
      for (int64_t base = u0; base < u1; base += per_iter, ++it) {
        float x[kU][8];
#pragma unroll
        for (int j = 0; j < kU; ++j) {
          const int64_t unit = base + j * kT + tid;
          if (unit < u1) {
            load_unit<VEC>(grid, unit, c1, x[j]);
          } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) x[j][k] = -INFINITY;
          }
        }
        accumulate(x, clamp);
      }
    }
  };
  pass(std::false_type{});

  // (max, rescaled sum) over the workgroup: wave butterfly, then the four
  // wave results in wave order.  Afterwards every thread holds the same
  // (m, s, t).
  const int wave = tid / 64;
  float m_own = m;
  auto reduce = [&]() {
    m_own = m;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const float m2 = __shfl_xor(m, o);
      const float s2 = __shfl_xor(s, o);
      const float t2 = ENT ? __shfl_xor(t, o) : 0.f;
      merge_ms<ENT>(m, s, t, m2, s2, t2);
    }
    if ((tid & 63) == 0) {
      sh_m[wave] = m;
      sh_s[wave] = s;
      sh_t[wave] = t;
    }
    __syncthreads();
    m = sh_m[0];
    s = sh_s[0];
    t = sh_t[0];
#pragma unroll
    for (int w = 1; w < kT / 64; ++w) merge_ms<ENT>(m, s, t, sh_m[w], sh_s[w], sh_t[w]);
  };
  reduce();
  if constexpr (ENT) {
    if (t != t) {          // the chunk holds a -inf logit: clamped second pass
      __syncthreads();     // every thread has read the shared partials
      pass(std::true_type{});
      reduce();
    }
  }

  // First index of the chunk maximum.  Only threads whose own maximum equals
  // it look: their first occurrence lies in iteration it_max, re-read once
  // (the other threads read nothing more, so the re-read costs a few cache
  // lines per chunk instead of one per thread).
  int32_t idx = INT32_MAX;
  if (m != -INFINITY && m_own == m && it_max < -1) {
    idx = static_cast<int32_t>(it_max == kHeadIter ? tid : tail0 + tid);
  } else if (m != -INFINITY && m_own == m) {
    const int64_t base = u0 + static_cast<int64_t>(it_max) * kT * kU;
    for (int j = 0; j < kU && idx == INT32_MAX; ++j) {
      const int64_t unit = base + j * kT + tid;
      if (unit >= u1) break;
      float x[8];
      load_unit<VEC>(grid, unit, c1, x);
      for (int k = 0; k < 8; ++k) {
        if (x[k] == m) {
          idx = static_cast<int32_t>(unit * 8 + k - off);
          break;
        }
      }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) idx = min(idx, __shfl_xor(idx, o));
  if ((tid & 63) == 0) sh_i[wave] = idx;
  __syncthreads();
  if (tid != 0) return;
#pragma unroll
  for (int w = 0; w < kT / 64; ++w) idx = min(idx, sh_i[w]);

  if (p.chunks > 1) {     // merged by the finalize kernel
    p.partials[row * p.chunks + chunk] = EsPartial{m, s, idx, t};
    return;
  }
  decide<ENT>(p, row, m, s, t, idx);
}

// Rows reduced in several chunks: the lanes of a group of L (a power of two
// that holds the chunks, at most 64) merge the chunk partials of one row (the
// kernel boundary makes them visible).  Lane l merges chunks l, l + L, ... in
// order, then a butterfly combines the lanes; every step is a fixed,
// commutative merge, so the result is the same on every lane and in every
// run (and for every L that holds the chunks: merging with an empty partial
// changes no bit).
template <bool ENT>
__device__ __forceinline__ void merge_chunks(const EsParams &p, int64_t row, int lane, int L) {
  const EsPartial *pp = p.partials + row * p.chunks;
  float m = -INFINITY, s = 0.f, t = 0.f;
  int32_t idx = INT32_MAX;
  for (int c = lane; c < p.chunks; c += L) {
    const EsPartial q = pp[c];
    merge<ENT>(m, s, t, idx, q.m, q.s, q.t, q.idx);
  }
  for (int o = 1; o < L; o <<= 1) {
    const float m2 = __shfl_xor(m, o);
    const float s2 = __shfl_xor(s, o);
    const float t2 = ENT ? __shfl_xor(t, o) : 0.f;
    const int32_t i2 = __shfl_xor(idx, o);
    merge<ENT>(m, s, t, idx, m2, s2, t2, i2);
  }
  if (lane == 0) decide<ENT>(p, row, m, s, t, idx);
}

// Edit selection of rows in several chunks: one wave per row.
__global__ __launch_bounds__(256) void edit_select_finalize_kernel(EsParams p) {
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row < p.rows) merge_chunks<false>(p, row, threadIdx.x & 63, 64);
}

// Threshold update, second step: one workgroup per block of block_size rows
// applies the mask-to-token set, the force-unmask and the token-to-token set
// to the rows' predictions and confidences.  Each row's current token is read
// and its new token written by the same thread, so new_tokens may be
// cur_tokens itself (an in-place update).  Rows reduced in several chunks are
// merged here first: they have no launch of their own (a launch of a few
// workgroups is 4 us, the merge well under one: 64 x 131072 with entropy
// 29.6 -> 25.6 us with the calls around it).
template <bool ENT>
__global__ __launch_bounds__(256) void threshold_block_kernel(EsParams p) {
  __shared__ unsigned long long sh_best;
  __shared__ int32_t sh_changed;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * p.block_size;
  const int tid = threadIdx.x;
  if (p.gate && *p.gate == 0) {
    // gated off: the pass changes nothing (its rows were not reduced)
    for (int i = tid; i < p.block_size; i += 256) {
      p.action[r0 + i] = 0;
      p.new_tokens[r0 + i] = p.cur[r0 + i];
    }
    if (tid == 0) p.block_changed[blockIdx.x] = 0;
    return;
  }
  if (tid == 0) {
    sh_best = 0;
    sh_changed = 0;
  }
  if (p.chunks > 1) {
    int L = 2;
    while (L < p.chunks && L < 64) L <<= 1;
    for (int i = tid / L; i < p.block_size; i += 256 / L) merge_chunks<ENT>(p, r0 + i, tid % L, L);
  }
  __syncthreads();      // (the rows' results are read below by other threads of this workgroup)
  bool any_gamma = false, any_masked = false;
  for (int i = tid; i < p.block_size; i += 256) {
    const int64_t r = r0 + i;
    const bool masked = p.cur[r] == p.mask_id;
    const float c = p.conf[r];
    any_masked |= masked;
    any_gamma |= masked && c > p.omega_mask;
    if (masked) {
      // highest confidence first, then the lowest row: conf is positive, so its
      // bits order like the value
      const unsigned long long key = (static_cast<unsigned long long>(__float_as_uint(c)) << 32) |
                                     (0xffffffffu - static_cast<uint32_t>(i));
      atomicMax(&sh_best, key);
    }
  }
  any_gamma = __syncthreads_or(any_gamma);
  any_masked = __syncthreads_or(any_masked);
  const int forced = (any_masked && !any_gamma) ? static_cast<int>(0xffffffffu - static_cast<uint32_t>(sh_best)) : -1;
  int changed = 0;
  for (int i = tid; i < p.block_size; i += 256) {
    const int64_t r = r0 + i;
    const int32_t cur = p.cur[r];
    const int32_t a = p.pred[r];
    const float c = p.conf[r];
    uint8_t act = 0;
    if (cur == p.mask_id) {
      if (c > p.omega_mask) act = 1;
      else if (i == forced) act = 2;
    } else if (a != cur && c >= p.threshold) {
      act = 3;
    }
    p.action[r] = act;
    p.new_tokens[r] = act ? a : cur;
    changed += act != 0;
  }
  if (changed) atomicAdd(&sh_changed, changed);
  __syncthreads();
  if (tid == 0) {
    p.block_changed[blockIdx.x] = sh_changed != 0;
    if (p.changed_count && sh_changed) atomicAdd(p.changed_count, sh_changed);
  }
}

// The second step for blocks of at most 64 rows whose rows are whole (one
// chunk): one wave per block and one row per lane, every value read once, no
// LDS and no barrier.  What bounds it is latency (a launch, one
// round trip, one atomic): 8 x 64 rows in a graph, with attention, 70.4 -> 67.7
// us; 2048 x 131072 with scores (which took the same form) 96.3 -> 92.4 us.
__global__ __launch_bounds__(256) void threshold_block_wave_kernel(EsParams p) {
  const int lane = threadIdx.x & 63;
  const int64_t blk = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int64_t r0 = blk * p.block_size;
  if (r0 >= p.rows) return;
  const bool in = lane < p.block_size;
  const int64_t r = r0 + (in ? lane : 0);
  const int32_t cur = p.cur[r];
  if (p.gate && *p.gate == 0) {      // gated off: the pass changes nothing
    if (in) {
      p.action[r] = 0;
      p.new_tokens[r] = cur;
    }
    if (lane == 0) p.block_changed[blk] = 0;
    return;
  }
  const float c = p.conf[r];
  const int32_t a = p.pred[r];
  const bool masked = in && cur == p.mask_id;
  const bool clear = masked && c > p.omega_mask;
  uint8_t act = 0;
  if (masked) act = clear ? 1 : 0;
  else if (in && a != cur && c >= p.threshold) act = 3;
  if (__builtin_amdgcn_ballot_w64(masked) != 0 && __builtin_amdgcn_ballot_w64(clear) == 0) {
    // force-unmask: highest confidence first (positive, so its bits order like
    // the value), then the lowest row
    const uint32_t bits = masked ? __float_as_uint(c) : 0u;
    uint32_t best = bits;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) best = max(best, static_cast<uint32_t>(__shfl_xor(static_cast<int>(best), o)));
    const uint64_t at = __builtin_amdgcn_ballot_w64(masked && bits == best);
    if (lane == __builtin_ctzll(at)) act = 2;
  }
  const int changed = __builtin_popcountll(__builtin_amdgcn_ballot_w64(act != 0));
  if (in) {
    p.action[r] = act;
    p.new_tokens[r] = act ? a : cur;
  }
  if (lane == 0) {
    p.block_changed[blk] = changed != 0;
    if (p.changed_count && changed) atomicAdd(p.changed_count, changed);
  }
}

}  // namespace

template <bool ENT>
hipError_t launch_rows(const EsParams &p, bool vector_loads, hipStream_t stream) {
  const int64_t wgs = p.rows * p.chunks;
  const dim3 grid(static_cast<unsigned>(wgs));
  // Few rows, each by one workgroup: twice the threads, since a workgroup then
  // has its CU to itself or nearly (256 x 131072: 16.5 us for the call, 18.7
  // with four times the threads or with four loads per thread; from 512 rows
  // on the smaller workgroups are better, 24.8 against 28.0 us).
  if (p.chunks == 1 && p.rows < kEsTargetWgs) {
    if (vector_loads)
      hipLaunchKernelGGL((edit_select_kernel<true, ENT, 2 * kEsThreads, true>), grid, dim3(2 * kEsThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((edit_select_kernel<false, ENT, 2 * kEsThreads, true>), grid, dim3(2 * kEsThreads), 0, stream, p);
    return hipGetLastError();
  }
  // Between two and five workgroups per CU, one iteration in flight per wave
  // and not two: with two, the CUs that hold one workgroup more than the others
  // get no more of the memory rate than those and finish late (all of it goes
  // round-robin by CU), with one every workgroup runs at its own pace.  Measured,
  // two in flight / one, us, without entropy: 528 x 65536 14.8 / 15.6, 640 x
  // 131072 28.4 / 28.1, 784 x 131072 37.9 / 34.5, 832 x 151936 45.3 / 41.6, 1152 x
  // 131072 50.9 / 48.6, 1408 x 131072 58.9 / 58.7, 1536 x 131072 61.7 / 62.7, 512 x
  // 131072 22.8 / 25.6; with it: 528 x 131072 30.7 / 29.7, 784 x 131072 43.1 / 38.6.
  // A row of one iteration has no next one: 8192 x 4096 without 23.7 / 23.6.
  const bool deep = p.chunk_len > kEsThreads * kU * 8 && (wgs < (ENT ? kEsTargetWgs + 1 : 640) || wgs >= 1408);
  if (!vector_loads)
    hipLaunchKernelGGL((edit_select_kernel<false, ENT, kEsThreads, true>), grid, dim3(kEsThreads), 0, stream, p);
  else if (deep)
    hipLaunchKernelGGL((edit_select_kernel<true, ENT, kEsThreads, true>), grid, dim3(kEsThreads), 0, stream, p);
  else
    hipLaunchKernelGGL((edit_select_kernel<true, ENT, kEsThreads, false>), grid, dim3(kEsThreads), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_edit_select(const EsParams &p, bool vector_loads, hipStream_t stream) {
  const hipError_t e = launch_rows<false>(p, vector_loads, stream);
  if (e != hipSuccess || p.chunks == 1) return e;
  hipLaunchKernelGGL(edit_select_finalize_kernel, dim3(static_cast<unsigned>((p.rows + 3) / 4)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_threshold_update(const EsParams &p, bool vector_loads, hipStream_t stream) {
  const hipError_t e =
      p.entropy ? launch_rows<true>(p, vector_loads, stream) : launch_rows<false>(p, vector_loads, stream);
  if (e != hipSuccess) return e;
  const int64_t blocks = p.rows / p.block_size;
  if (p.chunks == 1 && p.block_size <= 64) {
    hipLaunchKernelGGL(threshold_block_wave_kernel, dim3(static_cast<unsigned>((blocks + 3) / 4)), dim3(256), 0, stream, p);
    return hipGetLastError();
  }
  const dim3 grid(static_cast<unsigned>(blocks));
  if (p.entropy) hipLaunchKernelGGL(threshold_block_kernel<true>, grid, dim3(256), 0, stream, p);
  else hipLaunchKernelGGL(threshold_block_kernel<false>, grid, dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace mbe
