// device_common.hpp -- device helpers shared by the encode and decode
// kernels of the 3LC path.
#pragma once

#include <float.h>

#include "lookback.hpp"
#include "tlc_internal.h"
#include "wave_scan.hpp"
#include "zre_scan.hpp"

namespace tlc {

constexpr int kWaves = kThreads / 64;

// Unsigned min/max with both operands of one type.  HIP's mixed-type
// min/max (what min<T>(a, b) selects when b has another type, an int
// constant for instance) converts to double and calls fmin: several f64
// instructions, and values from 2^53 on would round.
__device__ __forceinline__ uint64_t umin64(uint64_t a, uint64_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }

// A store into the pinned host readback (HostMirror) at system scope, so
// that it is in host memory when the kernel completes; p null: nothing.
__device__ __forceinline__ void host_put(uint32_t* p, uint32_t v) {
  if (p) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// A whole result in one 16-byte store: a batch's hundreds of results cross the
// bus one store each (three word stores per tensor kept 335 blocks from
// storing anything else for up to 14 us).  The host checks every word by
// itself, so it need not arrive as one.
__device__ __forceinline__ void host_put_all(EncResult* h, uint32_t err, uint32_t len,
                                             float scale) {
  if (!h) return;
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  u4 w;
  w.x = err;
  w.y = len;
  w.z = __float_as_uint(scale);
  w.w = 0u;
  *reinterpret_cast<volatile u4*>(h) = w;
}
__device__ __forceinline__ void host_put_result(EncResult* h, uint32_t err, float scale) {
  if (h) {
    host_put(&h->err, err);
    host_put(reinterpret_cast<uint32_t*>(&h->scale), __float_as_uint(scale));
  }
}

// ---------------------------------------------------------------- reductions
__device__ __forceinline__ uint32_t abs_bits(float v) {
  return __float_as_uint(v) & 0x7fffffffu;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  return wave_last(wave_incl_scan(v, 0u, OpMax()));
}

// Block-wide max over a block of kW waves; every thread gets the result.
// Uses lds[kW] and one barrier; callers that reuse lds must barrier again
// first.
template <int kW = kWaves>
__device__ __forceinline__ uint32_t block_max(uint32_t v, uint32_t* lds) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t r = lds[0];
#pragma unroll
  for (int w = 1; w < kW; ++w) r = max(r, lds[w]);
  return r;
}

// Block-wide exclusive prefix of u32 values over a block of kW waves:
// returns (exclusive prefix of this thread, block total).  Uses lds[kW] and
// one barrier.
struct ScanU32 {
  uint32_t excl, total;
};
template <int kW = kWaves>
__device__ __forceinline__ ScanU32 block_scan_u32(uint32_t v, uint32_t* lds) {
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(v, 0u, OpAdd());
  if (lane == 63) lds[wid] = incl;
  __syncthreads();
  ScanU32 r;
  r.excl = incl - v;
  r.total = 0;
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    if ((uint32_t)w < wid) r.excl += lds[w];
    r.total += lds[w];
  }
  return r;
}

// Exclusive max-scan over a block of kW waves (0 for thread 0) and the
// block's max (all threads; ends with a barrier-protected read of lds).
template <int kW = kWaves>
__device__ __forceinline__ ScanU32 block_scan_max_u32(uint32_t v, uint32_t* lds) {
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(v, 0u, OpMax());
  const uint32_t excl = wave_prev_lane(incl, 0u);
  if (lane == 63) lds[wid] = incl;
  __syncthreads();
  ScanU32 r;
  r.excl = excl;
  r.total = 0u;
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    if ((uint32_t)w < wid) r.excl = max(r.excl, lds[w]);
    r.total = max(r.total, lds[w]);
  }
  return r;
}

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ uint32_t uniform32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)uniform32((uint32_t)v) | ((uint64_t)uniform32((uint32_t)(v >> 32)) << 32);
}
// A pointer into global memory that is the same in every lane.  The address
// space is said outright: a pointer read from LDS would otherwise be taken for
// one that may point into LDS, and every access made a flat one.
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  typedef __attribute__((address_space(1))) T G;
  return (T*)(G*)uniform64(reinterpret_cast<uint64_t>(p));
}

// Four floats at any dword address: gfx950 loads and stores 16 bytes there
// with the same instruction as at aligned ones, so tensors that are views
// into a flat buffer, and partitions that start anywhere (m % 4 != 0), need
// no path of their own.  (Before, such tensors went value by value, and
// partitions off the 16-byte grid through LDS atomics: on a 7,340,037-value
// view the max pass took 35 us and the encoder 46 us.)
typedef float tlc_f4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ld4(const float* p) {
  const tlc_f4 v = *reinterpret_cast<const tlc_f4*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st4(float* p, float4 v) {
  tlc_f4 w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  *reinterpret_cast<tlc_f4*>(p) = w;
}

// Four bytes at any address, the same way.
typedef uint32_t tlc_u4b __attribute__((aligned(1)));
__device__ __forceinline__ uint32_t ld_word(const uint8_t* p) {
  return *reinterpret_cast<const tlc_u4b*>(p);
}
__device__ __forceinline__ void st_word(uint8_t* p, uint32_t w) {
  *reinterpret_cast<tlc_u4b*>(p) = w;
}

// The same as streaming accesses, with the nontemporal hint, for tensors read or written once per kernel and far
// larger than the caches.  Measured on gfx950: the max reduction reads
// 25 % faster with it, the 8-bit kernels (contiguous read/write streams,
// both sides hinted) 10-15 % faster, and the decoder's partition-by-
// partition sweep gains too (its hinted stores leave no dirty lines for the
// next encode).  The 3LC encoder's flat passes over large tensors hint
// their loads and their stores, as nothing in them is read again before the
// whole tensor has streamed through (the check pass only where the values and
// the buffer don't fit the last-level cache together); its small tensors,
// which are read back from the cache, are not hinted.  The hint changes
// neither values nor visibility: the next kernel on the stream sees the
// stores.
__device__ __forceinline__ float4 ld_stream(const float* p) {
  const tlc_f4 v = __builtin_nontemporal_load(reinterpret_cast<const tlc_f4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_stream(float* p, float4 v) {
  tlc_f4 w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  __builtin_nontemporal_store(w, reinterpret_cast<tlc_f4*>(p));
}

// Place value of partition k's trit in a quartic byte (p0 most significant).
__device__ __forceinline__ uint32_t trit_weight(int k) {
  return k == 0 ? 81u : (k == 1 ? 27u : (k == 2 ? 9u : (k == 3 ? 3u : 1u)));
}

// ---------------------------------------------------------------- Eq. 1-2
struct Scale {
  float M;       // max|acc| * s
  float U;       // smallest fp32 u with rint(u / M) == 1
  uint32_t bad;  // NaN/Inf input or overflowing product
};

// rint(fl(a / M)) for |a| <= M is 1 exactly when fl(a / M) > 0.5, i.e. (the
// tie at 0.5 + 2^-25 rounds down to the even 0.5) when a > T = M * (0.5 +
// 2^-25).  U is the smallest float above T, so the test a >= U gives the same
// q as an IEEE divide followed by round-half-even, and by symmetry a <= -U
// gives q = -1.  M * 2^-25 lies between half and one unit in the last place
// of M / 2, so for M >= 2^-125 U is the float after M / 2; below, where floats
// are k * 2^-149 with k their bit pattern, T lies in [k / 2, k / 2 + 1/2) and U
// is floor(k / 2) + 1 (M = 0: the smallest subnormal, so q = 0 for the
// all-zero tensor).
__device__ __forceinline__ float quant_threshold(float M) {
  const uint32_t k = __float_as_uint(M);
  return __uint_as_float((k < 0x01000000u ? k >> 1 : k - 0x00800000u) + 1u);
}

// M and U from the bit pattern of max|acc|.
__device__ __forceinline__ Scale scale_of(uint32_t A, float s) {
  Scale sc;
  sc.M = 0.0f;
  sc.U = 0.0f;
  sc.bad = 1u;
  if (A >= 0x7f800000u) return sc;
  const float M = __uint_as_float(A) * s;
  if (!(M <= FLT_MAX)) return sc;
  sc.M = M;
  sc.U = quant_threshold(M);
  sc.bad = 0u;
  return sc;
}

// The same from the partial maxima of one tensor (all kT threads of the
// block).
template <int kT = kThreads>
__device__ __forceinline__ Scale finish_scale(const uint32_t* __restrict__ partials,
                                              uint32_t np, float s, uint32_t* lds) {
  static_assert(kT % 64 == 0, "whole waves");
  uint32_t v = 0;
  for (uint32_t i = threadIdx.x; i < np; i += kT) v = max(v, partials[i]);
  return scale_of(block_max<kT / 64>(v, lds), s);
}

// q = round(acc / M) in {-1, 0, 1} as a float: |acc| >= U, with acc's sign.
// The residual acc - M*q is one fused multiply-add: the product is exact, so
// it is the subtraction, and for q = +0 it adds -0, which keeps every acc
// (-0.0 too).
__device__ __forceinline__ float quantize_q(float acc, float U) {
  const float one = __uint_as_float(0x3f800000u | (__float_as_uint(acc) & 0x80000000u));
  return fabsf(acc) >= U ? one : 0.0f;
}
__device__ __forceinline__ float residual_of(float acc, float q, float M) {
  return __builtin_fmaf(-q, M, acc);
}

// The same with the trit q + 1.
__device__ __forceinline__ uint32_t quantize_one(float acc, float M, float U,
                                                 float& res) {
  const bool pos = acc >= U;
  const bool neg = acc <= -U;
  res = pos ? acc - M : (neg ? acc + M : acc);
  return pos ? 2u : (neg ? 0u : 1u);
}

// ---------------------------------------------------------------- stochastic mode
// Philox4x32-10 (Salmon et al., SC 2011): ten rounds, each multiplying two
// counter words by 0xD2511F53 and 0xCD9E8D57 (high halves XORed with the
// other two words and the key), the key advancing by 0x9E3779B9 /
// 0xBB67AE85 between rounds.
struct Philox4 {
  uint32_t v[4];
};
__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                 uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    // one 32 x 32 -> 64 multiply each (v_mad_u64_u32), not a low and a high one
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c0 = n0;
    c1 = (uint32_t)p1;
    c2 = n2;
    c3 = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  Philox4 r;
  r.v[0] = c0;
  r.v[1] = c1;
  r.v[2] = c2;
  r.v[3] = c3;
  return r;
}

// Random words for elements 4b .. 4b+3 of a tensor: counter (b, step),
// key = seed.
__device__ __forceinline__ Philox4 element_words(uint64_t b, uint64_t step, uint64_t seed) {
  return philox4x32_10((uint32_t)b, (uint32_t)(b >> 32), (uint32_t)step,
                       (uint32_t)(step >> 32), (uint32_t)seed, (uint32_t)(seed >> 32));
}

// Stochastic 3-value quantization of one value: sign(x) kept with
// probability |x|/M, i.e. when u*M < |x| for u = (w >> 8) * 2^-24.  The fused
// multiply-add rounds u*M - |x| once, from its exact value, and rounding
// keeps the sign (a negative difference too small for a float becomes -0, a
// zero one +0), so its sign bit is the exact decision; M = 0 (all zeros)
// keeps nothing.  Returns the trit q + 1.
__device__ __forceinline__ uint32_t stochastic_trit(float x, float M, uint32_t w) {
  const float u = (float)(w >> 8) * 0x1p-24f;  // both exact
  const bool keep = (int32_t)__float_as_uint(__builtin_fmaf(u, M, -fabsf(x))) < 0;
  return keep ? (x > 0.0f ? 2u : 0u) : 1u;
}

// ---------------------------------------------------------------- Section 3.3
using EncSW = StatusWord<39>;  // RunSum with a 30-bit count
using DecSW = StatusWord<36>;  // expanded byte count

__device__ __forceinline__ uint64_t rs_to_payload(RunSum a) {
  return (a.v & 0x3fffffffull) | ((a.v >> 32) << 30);
}
__device__ __forceinline__ RunSum rs_from_payload(uint64_t p) {
  RunSum r;
  r.v = (p & 0x3fffffffull) | ((p >> 30) << 32);
  return r;
}

struct EncOp {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const {
    return rs_to_payload(rs_combine(rs_from_payload(a), rs_from_payload(b)));
  }
};
struct SumOp {
  __device__ uint64_t operator()(uint64_t a, uint64_t b) const { return a + b; }
};

// Wave scans of segment summaries (zre_scan.hpp), in lane order.
struct OpRun {
  __device__ __forceinline__ uint64_t operator()(uint64_t a, uint64_t b) const {
    RunSum x, y;
    x.v = a;
    y.v = b;
    return rs_combine(x, y).v;
  }
};
__device__ __forceinline__ RunSum wave_incl_scan_rs(RunSum v) {
  RunSum r;
  r.v = wave_incl_scan(v.v, rs_identity().v, OpRun());
  return r;
}
__device__ __forceinline__ RunSum wave_prev_lane_rs(RunSum v) {
  RunSum r;
  r.v = wave_prev_lane(v.v, rs_identity().v);
  return r;
}

// Number of quartic bytes a stream byte stands for: data bytes (< 243) one,
// run codes 243 + (k - 2) k copies of 121.
__device__ __forceinline__ uint32_t expanded_len(uint32_t b) {
  return b < kRunBase ? 1u : b - (kRunBase - 2u);
}

// What the four stream bytes of w expand to beyond one quartic byte each:
// byte b adds max(b - 242, 0) (expanded_len less one), which is
// (|b - 242| + b - 242) / 2, and two sums of absolute byte differences
// (v_sad_u8) give that for the four bytes at once.  A zero byte adds 0.
__device__ __forceinline__ uint32_t run_extra4(uint32_t w) {
  constexpr uint32_t kPivot = kRunBase - 1u;  // 242 in every byte below
  const uint32_t s =
      __builtin_amdgcn_sad_u8(w, kPivot * 0x01010101u, __builtin_amdgcn_sad_u8(w, 0u, 0u));
  return (s - 4u * kPivot) >> 1;
}

// ---------------------------------------------------------------- Eq. 3
// The dequantized value M*q for trit t = q + 1 is -M, M*0 or M (M*(-1) is
// the exact negation; M*0 is +0, or -0 for a scale of -0.0, which the
// decoder accepts as >= 0).
__device__ __forceinline__ float trit_value(uint32_t t, float M) {
  return t == 0u ? -M : (t == 1u ? M * 0.0f : M);
}

// Eq. 3 accumulated densely into out (every value: out + M*q, so -0.0 + 0
// gives +0.0).  acc_trit4 returns whether any of the four sums has other
// bits than its input: a store of identical bits can be skipped without
// changing any result, and with few values q != 0 most stores are.
__device__ __forceinline__ float acc_trit(float out, uint32_t t, float M) {
  return out + trit_value(t, M);
}

__device__ __forceinline__ bool acc_trit4(float4& o, const uint32_t (&d)[4], float M) {
  const float4 r = make_float4(o.x + trit_value(d[0], M), o.y + trit_value(d[1], M),
                               o.z + trit_value(d[2], M), o.w + trit_value(d[3], M));
  const bool changed = ((__float_as_uint(r.x) ^ __float_as_uint(o.x)) |
                        (__float_as_uint(r.y) ^ __float_as_uint(o.y)) |
                        (__float_as_uint(r.z) ^ __float_as_uint(o.z)) |
                        (__float_as_uint(r.w) ^ __float_as_uint(o.w))) != 0u;
  o = r;
  return changed;
}

// out[e] += M*q, stored only if the bits change.
__device__ __forceinline__ void acc_trit_at(float* __restrict__ out, uint64_t e, uint32_t t,
                                            float M) {
  const float o = out[e];
  const float r = o + trit_value(t, M);
  if (__float_as_uint(r) != __float_as_uint(o)) out[e] = r;
}

// Four bits: byte i of w differs from 121.  x = w ^ 0x79797979 has a zero
// byte exactly where w holds 121; bit 7 of ((x & 0x7f..) + 0x7f..) | x is
// set in every other byte (no carry leaves a byte); the multiply gathers
// the four bit-7 flags, shifted to bits 0, 8, 16, 24, into bits 21..24
// (the partial products occupy distinct bits, so nothing carries).
__device__ __forceinline__ uint32_t nonzero_byte_mask4(uint32_t w) {
  const uint32_t x = w ^ 0x79797979u;
  const uint32_t y = (x | ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u;
  return ((y >> 7) * 0x00204081u) >> 21 & 0xfu;
}

// The same in spread form, bit 2i for byte i (rs_gaps_len<2>): the multiply
// places the four bit-7 flags, shifted to bits 0, 8, 16, 24, at bits 18, 20,
// 22, 24 (again no two partial products share a bit).
__device__ __forceinline__ uint32_t nonzero_byte_mask4_spread(uint32_t w) {
  const uint32_t x = w ^ 0x79797979u;
  const uint32_t y = (x | ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu)) & 0x80808080u;
  return ((y >> 7) * 0x00041041u) >> 18 & 0x55u;
}

// The spread mask of the first cnt (<= 16) quartic bytes that one thread holds.
__device__ __forceinline__ uint32_t nonzero_mask16_spread(const uint4& w, uint32_t cnt) {
  static_assert(kZeroGroup == 0x79u, "the mask compares against bytes of 121");
  const uint32_t nz = nonzero_byte_mask4_spread(w.x) | (nonzero_byte_mask4_spread(w.y) << 8) |
                      (nonzero_byte_mask4_spread(w.z) << 16) |
                      (nonzero_byte_mask4_spread(w.w) << 24);
  return cnt >= 16u ? nz : nz & ((1u << (2u * cnt)) - 1u);
}

// The spread mask of the 16 quartic bytes that five trit words pack (word
// k holds partition k's trits, trit i in bits 2i and 2i + 1, as q + 1):
// byte i is 121 exactly when all five of its trits are 1 (Section 3.2: 121
// is 11111 in base 3), i.e. when bits 2i, 2i + 1 read 01 in every word.
__device__ __forceinline__ uint32_t nonzero_mask_trits(const uint32_t (&d)[5]) {
  constexpr uint32_t kOnes = 0x55555555u;  // trit 1 in every field
  const uint32_t z = (d[0] ^ kOnes) | (d[1] ^ kOnes) | (d[2] ^ kOnes) | (d[3] ^ kOnes) |
                     (d[4] ^ kOnes);
  return (z | (z >> 1)) & kOnes;
}

// Byte i (< 16) of four little-endian words, by selects on the values (an
// indexed array would be placed in LDS or scratch memory).
__device__ __forceinline__ uint32_t byte_of16(uint32_t x, uint32_t y, uint32_t z, uint32_t w,
                                              uint32_t i) {
  const uint32_t lo = (i & 4u) ? y : x, hi = (i & 4u) ? w : z;
  return ((i & 8u) ? hi : lo) >> (8u * (i & 3u)) & 255u;
}

// Base-3 digits of a quartic byte, most significant first (weights 81, 27,
// 9, 3, 1): Section 3.2, decoding step 1.
__device__ __forceinline__ void digits5(uint32_t byte, uint32_t (&t)[5]) {
  t[0] = byte / 81u;
  byte -= t[0] * 81u;
  t[1] = byte / 27u;
  byte -= t[1] * 27u;
  t[2] = byte / 9u;
  byte -= t[2] * 9u;
  t[3] = byte / 3u;
  t[4] = byte - t[3] * 3u;
}

// Index of the last descriptor whose `first` field is <= key (descriptors
// sorted by `first`, descs[0].first == 0).
template <class D, class F>
__device__ __forceinline__ uint32_t find_desc(const D* __restrict__ descs, uint32_t count,
                                              uint32_t key, F first) {
  uint32_t lo = 0, hi = count;  // invariant: first(descs[lo]) <= key
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (first(descs[mid]) <= key)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

}  // namespace tlc
