// encode.hip -- gfx950 encode kernels of the 3LC path.
//
//   tlc_quant_encode_chained_kernel, tlc_quant_encode_batch_kernel
//       a small tensor, or many tensors, in one launch: tiles hold their sums
//       in registers until M is known, and exchange maxima and summaries
//                                                   (Sections 3.1-3.3)
//   tlc_absmax_check_kernel / _batch_kernel
//       partial maxima of |tensor + buffer|, nothing written: lets the
//       default error policy refuse NaN/Inf before the buffer changes
//   tlc_accum_quantize_kernel
//       after the check pass, on large tensors: acc = x + r, 3-value
//       quantization, the residual stored in place and 2-bit trits for the
//       quartic pack                                (Section 3.1, Eq. 1-2)
//   tlc_accum_absmax_kernel / _batch_kernel
//       in place, large tensors: the tensor is added into the buffer with
//       partial maxima of the sums (Fig. 3, Eq. 1) and a bound per float4
//   tlc_quant_encode_kernel, tlc_zre_chunk_kernel, tlc_zre_compact_kernel
//       the quartic pack from the trits and each tile's own zero-run encoding;
//       then a scan of the tile summaries and the compaction into one stream
//                                                   (Sections 3.2-3.3)
//   tlc_quant_encode_bounds_kernel, tlc_quant_pack_bounds_kernel
//       after the in-place max pass: the tiles quantize what its bounds let
//       through themselves, without trits
//
// The batch kernels (and the _many_ ones, for the tensors of a batch that are
// too large for its one launch) run many tensors in one launch: every block
// reads the descriptor of its tensor, then runs the single-tensor device code.
// Everything is HBM streaming or bound by latency; nothing is a dense
// contraction, so there is no MFMA.
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"

namespace tlc {

// ---------------------------------------------------------------- Eq. 1
// Step 1 and Eq. 1 in one read of the tensor: with kResid the buffer
// becomes acc = x + r (the quantizer then rewrites only what can hold a
// q != 0); without, acc = x and nothing is written.  max |acc| is taken on the bit
// patterns with the sign cleared: for non-negative IEEE values integer
// order equals numeric order, so the u32 max is exact and independent of
// reduction order, and any NaN/Inf makes the result >= 0x7f800000.  Block
// `blk` of `nblk` strides over [0, n).  The float4 path marks its loads and
// stores nontemporal: nothing here is read again before the whole tensor
// has streamed through, and the hint measured faster for this kernel and
// for the quantizer that follows.
//
// kStore false (with kResid): the check pass of the default error policy,
// which only reduces max|x + r| and writes nothing.
//
// kBound (in place, large tensors): also store, for each float4 of the buffer,
// the top 16 bits of the bit pattern of its largest |acc|.  That half-word h
// bounds the values from above (|acc| < (h + 1) * 2^16 as bit patterns), so the
// pass that follows can skip every float4 whose h lies below the top half of its
// threshold U: all its values have q = 0 and keep acc.
//
// kKeep: plain loads, which leave what they read in the last-level cache for
// the writing pass (where both tensors fit it).
template <bool kResid = true, bool kStore = kResid, bool kBound = false, bool kKeep = false>
__device__ __forceinline__ uint32_t absmax_part(const float* __restrict__ x,
                                                float* __restrict__ r, uint64_t n,
                                                uint32_t blk, uint32_t nblk,
                                                uint16_t* __restrict__ bound = nullptr) {
  static_assert(!kStore || kResid, "only a buffer is stored");
  static_assert(!kBound || kStore, "bounds are of a stored buffer");
  uint32_t mx = 0;
  const uint64_t tid = (uint64_t)blk * kThreads + threadIdx.x;
  const uint64_t stride = (uint64_t)nblk * kThreads;
  const uint64_t nv = n >> 2;
  auto ld = [](const float* p) { return kKeep ? ld4(p) : ld_stream(p); };
  uint64_t i = tid;
  for (; i + 3 * stride < nv; i += 4 * stride) {
    float4 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = ld(x + 4 * (i + u * stride));
#pragma unroll
    for (int u = 0; u < 4; ++u)
      b[u] = kResid ? ld(r + 4 * (i + u * stride)) : make_float4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float4 v = kResid ? make_float4(a[u].x + b[u].x, a[u].y + b[u].y,
                                            a[u].z + b[u].z, a[u].w + b[u].w)
                              : a[u];
      if (kStore) st_stream(r + 4 * (i + u * stride), v);
      const uint32_t m4 =
          max(max(abs_bits(v.x), abs_bits(v.y)), max(abs_bits(v.z), abs_bits(v.w)));
      if (kBound) bound[i + u * stride] = (uint16_t)(m4 >> 16);
      mx = max(mx, m4);
    }
  }
  for (; i < nv; i += stride) {
    float4 v = ld(x + 4 * i);
    if (kResid) {
      const float4 b = ld(r + 4 * i);
      v = make_float4(v.x + b.x, v.y + b.y, v.z + b.z, v.w + b.w);
      if (kStore) st_stream(r + 4 * i, v);
    }
    const uint32_t m4 = max(max(abs_bits(v.x), abs_bits(v.y)), max(abs_bits(v.z), abs_bits(v.w)));
    if (kBound) bound[i] = (uint16_t)(m4 >> 16);
    mx = max(mx, m4);
  }
  for (uint64_t e = (nv << 2) + tid; e < n; e += stride) {
    const float v = kResid ? x[e] + r[e] : x[e];
    if (kStore) r[e] = v;
    mx = max(mx, abs_bits(v));
  }
  return mx;
}

// The writing pass of large tensors under the default error policy, once the
// check pass has given M (Eq. 1): acc = x + r, q = round(acc / M) and the
// residual acc - M*q (Eq. 2, Fig. 3 steps a-b) for every value; the
// residual is stored in place and q + 1 kept as a 2-bit trit, one byte per
// float4 of the buffer (value 4i + c in bits 2c, 2c + 1), from which the
// quantizer packs the quartic bytes without reading the buffer again.  The
// last n % 4 values are taken by one thread, which writes their byte.
__device__ __forceinline__ void accum_quantize_part(const float* __restrict__ x,
                                                    float* __restrict__ r, uint64_t n,
                                                    uint32_t blk, uint32_t nblk, float M,
                                                    float U, uint8_t* __restrict__ trits) {
  const uint64_t tid = (uint64_t)blk * kThreads + threadIdx.x;
  const uint64_t stride = (uint64_t)nblk * kThreads;
  const uint64_t nv = n >> 2;
  auto put4 = [&](uint64_t i, const float4& a, const float4& b) {
    float4 o;
    const uint32_t t0 = quantize_one(a.x + b.x, M, U, o.x);
    const uint32_t t1 = quantize_one(a.y + b.y, M, U, o.y);
    const uint32_t t2 = quantize_one(a.z + b.z, M, U, o.z);
    const uint32_t t3 = quantize_one(a.w + b.w, M, U, o.w);
    st_stream(r + 4 * i, o);
    trits[i] = (uint8_t)(t0 | (t1 << 2) | (t2 << 4) | (t3 << 6));
  };
  uint64_t i = tid;
  for (; i + 3 * stride < nv; i += 4 * stride) {
    float4 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = ld_stream(x + 4 * (i + u * stride));
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = ld_stream(r + 4 * (i + u * stride));
#pragma unroll
    for (int u = 0; u < 4; ++u) put4(i + u * stride, a[u], b[u]);
  }
  for (; i < nv; i += stride) put4(i, ld_stream(x + 4 * i), ld_stream(r + 4 * i));
  if (tid == 0 && (n & 3u)) {
    uint32_t tb = 0u;
    for (uint64_t e = nv << 2; e < n; ++e) {
      float o;
      tb |= quantize_one(x[e] + r[e], M, U, o) << (2u * (uint32_t)(e & 3u));
      r[e] = o;
    }
    trits[nv] = (uint8_t)tb;
  }
}

// A refused tensor, in place: the buffer gets the sums.
__device__ __forceinline__ void store_sums(const float* __restrict__ x, float* __restrict__ r,
                                           uint64_t n, uint32_t blk, uint32_t nblk) {
  for (uint64_t e = (uint64_t)blk * kThreads + threadIdx.x; e < n; e += (uint64_t)nblk * kThreads)
    r[e] = x[e] + r[e];
}

// Partial maxima of |x + r| that write nothing: the check pass that lets
// the default error policy refuse NaN/Inf before the buffer is touched.
template <bool kKeep>
__global__ __launch_bounds__(kThreads) void tlc_absmax_check_kernel(
    const float* __restrict__ x, const float* __restrict__ r, uint64_t n,
    uint32_t* __restrict__ partials) {
  __shared__ uint32_t lds[kWaves];
  const uint32_t mx = block_max(
      absmax_part<true, false, false, kKeep>(x, const_cast<float*>(r), n, blockIdx.x, gridDim.x),
      lds);
  if (threadIdx.x == 0) partials[blockIdx.x] = mx;
}

// Step 1 into the buffer and its max pass (in place, large tensors), or the
// max pass of a tensor without one.
template <bool kResid>
__global__ __launch_bounds__(kThreads) void tlc_accum_absmax_kernel(
    const float* __restrict__ x, float* __restrict__ r, uint64_t n,
    uint32_t* __restrict__ partials, uint16_t* __restrict__ bound) {
  __shared__ uint32_t lds[kWaves];
  const uint32_t mx = block_max(
      absmax_part<kResid, kResid, kResid>(x, r, n, blockIdx.x, gridDim.x, bound), lds);
  if (threadIdx.x == 0) partials[blockIdx.x] = mx;
}

// The writing pass of large tensors under the default error policy (steps 1,
// a and b of Section 3.1 with Eq. 2): the check pass's partial maxima give M
// (Eq. 1), then every value's acc = x + r is quantized, its residual stored in
// place and q + 1 kept as a 2-bit trit (accum_quantize_part).  A scale that is
// NaN/Inf or overflows leaves the buffer untouched, or with the sums
// (in_place).  Block 0 reports M and the verdict.
__global__ __launch_bounds__(kThreads) void tlc_accum_quantize_kernel(
    const float* __restrict__ x, float* __restrict__ r, uint64_t n, uint8_t* __restrict__ trits,
    const uint32_t* __restrict__ partials, uint32_t np, float s, bool in_place,
    Ctrl* __restrict__ ctrl, HostMirror hm) {
  __shared__ uint32_t lds[kWaves];
  const Scale sc = finish_scale(partials, np, s, lds);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctrl->enc.err = sc.bad;
    ctrl->enc.scale = sc.M;
    host_put_result(hm.res, sc.bad, sc.M);
  }
  if (sc.bad) {
    if (in_place) store_sums(x, r, n, blockIdx.x, gridDim.x);
    return;
  }
  accum_quantize_part(x, r, n, blockIdx.x, gridDim.x, sc.M, sc.U, trits);
}

// The max and the writing passes over a batch's middle tensors, laid end to end
// (v0 counts from the first one's start, in kManyValues).  Groups of blocks take
// equal shares of the whole, and a group's blocks stride over each tensor in
// its share together: equal work wherever the tensors end.  (A share of the
// blocks for each tensor left blocks over or doubled them up on a CU: 130
// tensors of 1M values 625 to 673 us, three of 25M 345 with 258 blocks and 279
// with 255.  A stretch of its own for each block costs a tenth to a fifth of
// the bandwidth, many tensors in a group a tail each.)  Partial maxima: one per
// block, group and tensor, a tensor's from number blk0 on.
template <class Part>
__device__ __forceinline__ void for_many(const EncDesc* __restrict__ descs, uint32_t count,
                                         uint32_t units, uint32_t groups, Part&& part) {
  const uint32_t per = gridDim.x / groups;  // blocks of a group
  const uint32_t g = blockIdx.x / per, b = blockIdx.x - g * per;
  const uint32_t u0 = (uint32_t)((uint64_t)units * g / groups);
  const uint32_t u1 = (uint32_t)((uint64_t)units * (g + 1u) / groups);
  if (u0 >= u1) return;
  uint32_t t = find_desc(descs, count, u0, [](const EncDesc& d) { return d.v0; });
#pragma unroll 1
  for (; t < count; ++t) {
    const EncDesc& d = descs[t];
    if (d.v0 >= u1) break;
    const uint64_t lo = (uint64_t)(umax32(u0, d.v0) - d.v0) * kManyValues;
    const uint64_t hi = umin64(d.n, (uint64_t)(u1 - d.v0) * kManyValues);
    part(t, d, lo, hi > lo ? hi - lo : 0u, (g + t) * (kAbsmaxMaxBlocks / groups) + b, b, per);
    __syncthreads();  // the part's LDS is free again
  }
}

template <bool kKeep>
__global__ __launch_bounds__(kThreads) void tlc_absmax_check_batch_kernel(
    const EncDesc* __restrict__ descs, uint32_t count, uint32_t units, uint32_t groups,
    uint32_t* __restrict__ partials) {
  __shared__ uint32_t lds[kWaves];
  for_many(descs, count, units, groups,
           [&](uint32_t, const EncDesc& d, uint64_t lo, uint64_t n, uint32_t slot, uint32_t blk,
               uint32_t nblk) {
             const uint32_t bm = block_max(
                 absmax_part<true, false, false, kKeep>(uniform_ptr(d.x) + lo,
                                                        uniform_ptr(d.r) + lo, n, blk, nblk),
                 lds);
             if (threadIdx.x == 0) partials[slot] = bm;
           });
}

__global__ __launch_bounds__(kThreads) void tlc_accum_absmax_batch_kernel(
    const EncDesc* __restrict__ descs, uint32_t count, uint32_t units, uint32_t groups,
    uint32_t* __restrict__ partials, uint16_t* __restrict__ bound) {
  __shared__ uint32_t lds[kWaves];
  for_many(descs, count, units, groups,
           [&](uint32_t, const EncDesc& d, uint64_t lo, uint64_t n, uint32_t slot, uint32_t blk,
               uint32_t nblk) {
             const uint64_t at = (uint64_t)d.v0 * kManyValues + lo;
             const uint32_t bm =
                 block_max(absmax_part<true, true, true>(uniform_ptr(d.x) + lo,
                                                         uniform_ptr(d.r) + lo, n, blk, nblk,
                                                         bound + at / 4),
                           lds);
             if (threadIdx.x == 0) partials[slot] = bm;
           });
}

__global__ __launch_bounds__(kThreads) void tlc_quantize_many_kernel(
    const EncDesc* __restrict__ descs, uint32_t count, uint32_t units, uint32_t groups,
    const uint32_t* __restrict__ partials, bool in_place, uint8_t* __restrict__ trits,
    EncResult* __restrict__ results, HostMirror hm) {
  __shared__ uint32_t lds[kWaves];
  for_many(descs, count, units, groups,
           [&](uint32_t t, const EncDesc& d, uint64_t lo, uint64_t n, uint32_t slot, uint32_t blk,
               uint32_t nblk) {
             const Scale sc = finish_scale(partials + d.blk0, d.nblk, d.s, lds);
             if (slot == d.blk0 && threadIdx.x == 0) {  // its first group's first block
               results[t].err = sc.bad;
               results[t].scale = sc.M;
               host_put_result(hm.res ? hm.res + t : nullptr, sc.bad, sc.M);
             }
             const float* x = uniform_ptr(d.x) + lo;
             float* r = uniform_ptr(d.r) + lo;
             const uint64_t at = (uint64_t)d.v0 * kManyValues + lo;
             if (!sc.bad)
               accum_quantize_part(x, r, n, blk, nblk, sc.M, sc.U, trits + at / 4);
             else if (in_place)
               store_sums(x, r, n, blk, nblk);
           });
}

// ---------------------------------------------------------------- Eq. 2, 3.2, 3.3
template <int kW>
struct EncShared {
  uint32_t red[kW];
  uint32_t red2[kW];
  uint32_t lead;   // the tile's first non-121 byte
  __align__(16) uint8_t q[kEncTile];
  __align__(16) uint8_t out[kEncTile + 16];
};

constexpr int kGroupsPerThread = kEncTile / 4 / kThreads;  // groups of 4 bytes per thread

// ---------------------------------------------------------------- single tensor, three passes
// A single tensor is encoded without any wait between tiles:
//   pass A (tlc_quant_encode_kernel, one block per tile): quantize_tile, then
//     zero-run encode the tile from its first non-121 byte on into its own
//     slot.  That part does not depend on earlier tiles: the byte closes the
//     run before it, so the encoder is at phase 0 there.  Each tile records
//     its summary (RunSum), the length of its leading 121 run and the slot
//     length.
//   pass B (tlc_zre_chunk_kernel): every tile's prefix within its chunk of
//     64 tiles and the chunk summaries; the pass's last block scans the
//     chunk summaries.
//   pass C (tlc_zre_compact_kernel, one wave per tile): the tile's prefix
//     (its output offset and incoming run phase) from its chunk's prefix
//     and its own within the chunk, then the leading run's codes, which
//     need the incoming phase (one 255 per 14th byte of the grown run, then
//     its remainder code if the tile has a non-121 byte), and the slot; the
//     last tile adds the remainder of a run that ends the stream.

// Phase 1 of a first-pass tile: every value is quantized already (trits).
// load_trits fetches, for each of this thread's groups (quartic
// bytes j..j+3, g = threadIdx.x + kThreads * it, as in the float4 path) and
// each partition k, the trits of values e = k*m + j .. e + 3 as one byte:
// they start at bit 2*(e mod 4) of trit byte e/4 and run into the next one
// when e mod 4 != 0 (m % 4 != 0).  pack_trits then forms the quartic bytes
// (Section 3.2), with the values past n as the zero padding (trit 0), and
// ends with a barrier.
template <int kT = kThreads>
__device__ __forceinline__ void load_trits(const uint8_t* __restrict__ trits, uint64_t n,
                                           uint32_t m, uint64_t q0, uint32_t tile_bytes,
                                           uint32_t (&tb)[kEncTile / 4 / kT][5]) {
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    // group g's first value is e = base + 4g; q0 is a multiple of 4, so
    // e mod 4 = base mod 4 = a for the whole block, e / 4 = base / 4 + g,
    // and the values before n are those with 4g < n - base
    const uint64_t base = (uint64_t)k * m + q0;
    const uint32_t a = (uint32_t)(base & 3u);
    const uint8_t* tp = trits + (base >> 2);
    const uint64_t left = n > base ? n - base : 0u;  // values of the partition from base on
    const uint32_t lim = (uint32_t)umin64(left, tile_bytes);
    const uint32_t cap = (uint32_t)umin64(left + a, 2u * kEncTile);
#pragma unroll
    for (int it = 0; it < kEncTile / 4 / kT; ++it) {
      const uint32_t g = threadIdx.x + kT * it;
      uint32_t v = 0u;
      if (g * 4u < lim) {
        v = tp[g];
        if (a != 0u) {
          // trit byte e/4 + 1 holds values from e + 4 - a on: it exists when
          // 4g + 4 - a < left (4g + 4 <= tile_bytes + 3 < 2 * kEncTile)
          if (g * 4u + 4u < cap) v |= (uint32_t)tp[g + 1u] << 8;
          v = (v >> (2u * a)) & 0xffu;
        }
      }
      tb[it][k] = v;
    }
  }
}

// The trits of this thread's own 16 * kHalves values in each partition of a
// tile (values k*m + q0 + 16*kHalves*tid + [0, 16*kHalves), so that the
// thread packs the quartic bytes it encodes): consecutive bits of the trit
// array from bit 2*(k*m + q0) + 32*kHalves*tid on, joined from the aligned
// word at or before them and the next ones (alignbit; the bit offset within
// the word is the same for the whole partition, so any m works).  The trit
// area has 64 bytes of slack behind the trits of max_n values, so the word
// past the last one lies inside it too.
template <int kHalves>
__device__ __forceinline__ void load_trit_words(const uint8_t* __restrict__ trits, uint32_t m,
                                                uint64_t q0, uint32_t (&d)[kHalves][5]) {
  const uint32_t* tw = reinterpret_cast<const uint32_t*>(trits);
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const uint64_t e0 = (uint64_t)k * m + q0;  // the partition's first value in the tile
    const uint32_t sh = 2u * (uint32_t)(e0 & 15u);
    const uint32_t* wp = tw + (e0 >> 4) + kHalves * threadIdx.x;
    uint32_t lo = wp[0];
#pragma unroll
    for (int hf = 0; hf < kHalves; ++hf) {
      const uint32_t hi = wp[hf + 1];
      d[hf][k] = sh ? __builtin_amdgcn_alignbit(hi, lo, sh) : lo;
      lo = hi;
    }
  }
}

__device__ __forceinline__ uint32_t spread_trits(uint32_t tb) {
  // the four 2-bit trits of one byte into the low bits of four bytes
  tb = (tb | (tb << 12)) & 0x000f000fu;
  return (tb | (tb << 6)) & 0x03030303u;
}

// Tables of spread trits times the partition's weight (Section 3.2: 81, 27,
// 9, 3, 1): lut[k][b] holds, in byte lane c, 3^(4-k) times trit c of trit
// byte b.  The sum of one entry per partition is the four quartic bytes of
// a group (each at most 242, so no carry crosses a lane): five LDS reads
// and four adds instead of five spreads and four multiply-adds.  Written
// before a barrier of the caller.
template <int kT = kThreads>
__device__ __forceinline__ void init_trit_luts(uint32_t (*lut)[256]) {
  static_assert(256 % kT == 0, "whole rounds of table entries");
#pragma unroll
  for (uint32_t b = threadIdx.x; b < 256u; b += kT) {
    const uint32_t sp = spread_trits(b);
    lut[0][b] = 81u * sp;
    lut[1][b] = 27u * sp;
    lut[2][b] = 9u * sp;
    lut[3][b] = 3u * sp;
    lut[4][b] = sp;
  }
}

// This thread's 16 quartic bytes from its trit words (load_trit_words):
// byte g of each word holds the trits of its values 4g..4g+3.
__device__ __forceinline__ uint4 pack_trit_words(const uint32_t (&d)[5],
                                                 const uint32_t (*lut)[256]) {
  uint32_t o[4];
#pragma unroll
  for (int g = 0; g < 4; ++g)
    o[g] = lut[0][(d[0] >> (8 * g)) & 255u] + lut[1][(d[1] >> (8 * g)) & 255u] +
           lut[2][(d[2] >> (8 * g)) & 255u] + lut[3][(d[3] >> (8 * g)) & 255u] +
           lut[4][(d[4] >> (8 * g)) & 255u];
  return make_uint4(o[0], o[1], o[2], o[3]);
}

template <int kT = kThreads>
__device__ __forceinline__ void pack_trits(const uint32_t (&tb)[kEncTile / 4 / kT][5], uint64_t n,
                                           uint32_t m, uint64_t q0, uint32_t tile_bytes,
                                           const uint32_t (*lut)[256], uint8_t* q) {
  uint32_t* qw = reinterpret_cast<uint32_t*>(q);
#pragma unroll
  for (int it = 0; it < kEncTile / 4 / kT; ++it) {
    const uint32_t g = threadIdx.x + kT * it;
    if (g * 4u >= tile_bytes) break;
    const uint64_t j = q0 + g * 4u;
    if (4ull * m + j + 4u <= n) {
      // all 20 values exist: the four bytes at once
      qw[g] = lut[0][tb[it][0]] + lut[1][tb[it][1]] + lut[2][tb[it][2]] + lut[3][tb[it][3]] +
              lut[4][tb[it][4]];
      continue;
    }
    uint32_t code[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const uint64_t e = (uint64_t)k * m + j;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        code[c] = code[c] * 3u + (e + c < n ? (tb[it][k] >> (2 * c)) & 3u : 0u);
    }
    qw[g] = code[0] | (code[1] << 8) | (code[2] << 16) | (code[3] << 24);
  }
  __syncthreads();
}

// The first pass's tiles, kT threads per tile: each thread packs and
// encodes kEncTile / kT quartic bytes as kHalves pieces of 16, so with fewer
// threads the block scans, the verdict and the record, which cost the same
// per thread, are spread over more bytes (the pass is bound by its vector
// instructions).
constexpr int kTritThreads = 128;
// Below this many tiles the grid is too small to hide the longer work per
// block, and four waves per tile are faster (on gfx950: 13,108 tiles 19.3
// against 23.0 us; a mix of 3,277- and 1,250-tile tensors 10.8 against 9.6).
constexpr uint32_t kTritTwoWaveMinTiles = 8192;

template <int kT>
struct TritTileShared {
  EncShared<kT / 64> enc;
  uint32_t lut[5][256];
};

// Section 3.3 from the tile's first non-121 byte on: the thread's quartic bytes
// w (16 * kHalves, from tile byte lo on) and the masks of the non-121 ones nz
// (of each piece, spread: bit 2i for its byte i) into the tile's slot and its
// record.  left: residuals that the tile leaves to the compaction.
template <int kT>
__device__ __forceinline__ void encode_tile_runs(const uint4 (&w)[kEncTile / kT / 16],
                                                 const uint32_t (&nz)[kEncTile / kT / 16],
                                                 uint32_t tile_bytes, uint8_t* __restrict__ slot,
                                                 TileRec* __restrict__ rec_out,
                                                 EncShared<kT / 64>& sh, uint32_t left) {
  constexpr int kW = kT / 64;
  constexpr int kHalves = kEncTile / kT / 16;
  constexpr uint32_t kBytes = 16u * kHalves;  // quartic bytes per thread
  const uint32_t lo = threadIdx.x * kBytes;
  // From the gaps between non-121 bytes: a max-scan over the threads' last non-121
  // positions gives each thread the previous one, a sum-scan of what each
  // thread emits gives its output offset (zre_scan.hpp: rs_gaps_len,
  // rs_gaps_emit; the pieces take turns, as a gap inside one costs exactly
  // one code); the thread with the tile's last non-121 byte adds the
  // trailing run's codes 255 to its length.
  uint32_t last = 0u, first = 0u;  // position + 1 of the thread's last and first non-121 byte
  uint32_t ends[kHalves];          // last, as it stands before each piece
#pragma unroll
  for (int hf = 0; hf < kHalves; ++hf) {
    const uint32_t l = lo + 16u * hf;
    ends[hf] = last;
    if (nz[hf]) {
      if (first == 0u) first = l + (uint32_t)__builtin_ctz(nz[hf]) / 2u + 1u;
      last = l + (31u - (uint32_t)__builtin_clz(nz[hf])) / 2u + 1u;
    }
  }
  const ScanU32 pm = block_scan_max_u32<kW>(last, sh.red);
  const bool tail = last != 0u && last == pm.total;
  if (first != 0u && pm.excl == 0u) sh.lead = first - 1u;
  const uint32_t trail = tile_bytes - pm.total;  // 121s after the last non-121 byte
  uint32_t mine = tail ? trail / kRunMax : 0u;
#pragma unroll
  for (int hf = 0; hf < kHalves; ++hf)  // the byte before a piece's first: -1 if none
    mine += rs_gaps_len<2>(nz[hf], lo + 16u * hf, (int)umax32(pm.excl, ends[hf]) - 1);
  // every output byte that is not a remainder code or a non-121 byte is a
  // 255: fill the whole output with 255 first (the scan's barrier orders
  // it before the writes below), so runs only advance the offset
  static_assert(sizeof(sh.out) == kBytes * kT + 16, "kHalves uint4 of output per thread, +1");
#pragma unroll
  for (int hf = 0; hf < kHalves; ++hf)
    reinterpret_cast<uint4*>(sh.out)[kHalves * threadIdx.x + hf] = make_uint4(~0u, ~0u, ~0u, ~0u);
  if (threadIdx.x == 0)
    reinterpret_cast<uint4*>(sh.out)[kHalves * kT] = make_uint4(~0u, ~0u, ~0u, ~0u);
  const ScanU32 off = block_scan_u32<kW>(mine, sh.red2);
  uint32_t o = off.excl;
  auto put = [&](uint32_t c) {
    if (o < sizeof(sh.out)) sh.out[o] = (uint8_t)c;
    ++o;
  };
  auto fill = [&](uint32_t k) { o += k; };
#pragma unroll
  for (int hf = 0; hf < kHalves; ++hf) {
    const uint32_t w0 = w[hf].x, w1 = w[hf].y, w2 = w[hf].z, w3 = w[hf].w;
    rs_gaps_emit<2>(nz[hf], lo + 16u * hf, (int)umax32(pm.excl, ends[hf]) - 1,
                    [w0, w1, w2, w3](uint32_t i) { return byte_of16(w0, w1, w2, w3, i); }, put,
                    fill);
  }
  // the slot holds at most the tile's own bytes; the clamp only keeps a
  // logic error inside the slot
  const uint32_t len = umin32(off.total, tile_bytes);
  __syncthreads();
  for (uint32_t i = 16u * threadIdx.x; i < len; i += 16u * kT)
    *reinterpret_cast<uint4*>(slot + i) = *reinterpret_cast<const uint4*>(sh.out + i);
  if (threadIdx.x == 0) {
    TileRec rec;
    if (pm.total == 0u) {  // all 121: one run
      rec.agg = rs_zero_run(tile_bytes).v;
      rec.lead = (uint16_t)tile_bytes;
      rec.len = 0u;
    } else {
      rec.agg = rs_combine(rs_zero_run(sh.lead), rs_make(0u, 0u, trail % kRunMax, off.total)).v;
      rec.lead = (uint16_t)sh.lead;
      rec.len = (uint16_t)len;
    }
    rec.left = left;
    *rec_out = rec;
  }
}

// Tile t of a tensor: its slot and record.  err: the tensor was refused.
template <int kT>
__device__ __forceinline__ void encode_trit_tile(uint64_t n, uint32_t m, uint32_t t,
                                                 const uint8_t* __restrict__ trits,
                                                 const uint32_t* err, uint8_t* __restrict__ slot,
                                                 TileRec* __restrict__ rec_out,
                                                 TritTileShared<kT>& shared) {
  constexpr int kHalves = kEncTile / kT / 16;
  constexpr uint32_t kBytes = 16u * kHalves;  // quartic bytes per thread
  static_assert(kHalves == 1 || kHalves == 2, "one or two pieces of 16 bytes per thread");
  EncShared<kT / 64>& enc = shared.enc;
  uint32_t(&s_lut)[5][256] = shared.lut;
  const uint64_t q0 = (uint64_t)t * kEncTile;
  const uint32_t tile_bytes = (uint32_t)umin64(kEncTile, (uint64_t)m - q0);
  // an interior tile (whole, every value before n): each thread packs its
  // own quartic bytes in registers; other tiles pack through sh.q
  const bool own = tile_bytes == (uint32_t)kEncTile && 4ull * m + q0 + kEncTile <= n;
  const uint32_t lo = threadIdx.x * kBytes;
  uint32_t d[kHalves][5];  // own tile: the trits of the thread's values, 16 per word
  uint32_t h[kEncTile / 4 / kT][5];
  if (own)
    load_trit_words<kHalves>(trits, m, q0, d);
  else
    load_trits<kT>(trits, n, m, q0, tile_bytes, h);
  init_trit_luts<kT>(s_lut);
  __syncthreads();  // the tables
  if (*err) return;  // NaN/Inf or overflow: no stream (every block returns)
  const uint32_t cnt = lo < tile_bytes ? umin32(kBytes, tile_bytes - lo) : 0u;
  uint4 w[kHalves];
  uint32_t nz[kHalves];  // non-121 bytes of each piece, spread: bit 2i for its byte i
  if (own) {
#pragma unroll
    for (int hf = 0; hf < kHalves; ++hf) {
      w[hf] = pack_trit_words(d[hf], s_lut);
      nz[hf] = nonzero_mask_trits(d[hf]);
    }
  } else {
    pack_trits<kT>(h, n, m, q0, tile_bytes, s_lut, enc.q);
#pragma unroll
    for (int hf = 0; hf < kHalves; ++hf) {
      const uint32_t c = cnt > 16u * hf ? umin32(cnt - 16u * hf, 16u) : 0u;
      w[hf] = c ? *reinterpret_cast<const uint4*>(enc.q + lo + 16u * hf) : make_uint4(0, 0, 0, 0);
      nz[hf] = c ? nonzero_mask16_spread(w[hf], c) : 0u;
    }
  }

  encode_tile_runs<kT>(w, nz, tile_bytes, slot, rec_out, enc, 0u);
}

template <int kT>
__global__ __launch_bounds__(kT) void tlc_quant_encode_kernel(
    uint64_t n, uint32_t m, uint8_t* __restrict__ slots, TileRec* __restrict__ recs,
    const uint8_t* __restrict__ trits, const Ctrl* __restrict__ ctrl) {
  __shared__ TritTileShared<kT> sh;
  const uint32_t t = blockIdx.x;
  encode_trit_tile<kT>(n, m, t, trits, &ctrl->enc.err, slots + (uint64_t)t * kEncTile, recs + t,
                       sh);
}

// The tiles of a batch's middle tensors, numbered through (tile0).
__global__ __launch_bounds__(kThreads) void tlc_quant_encode_many_kernel(
    const EncDesc* __restrict__ descs, uint32_t count, uint8_t* __restrict__ slots,
    TileRec* __restrict__ recs, const uint8_t* __restrict__ trits,
    const EncResult* __restrict__ results) {
  __shared__ TritTileShared<kThreads> sh;
  const uint32_t t =
      find_desc(descs, count, blockIdx.x, [](const EncDesc& d) { return d.tile0; });
  const EncDesc& d = descs[t];
  encode_trit_tile<kThreads>(d.n, d.m, blockIdx.x - d.tile0,
                             trits + (uint64_t)d.v0 * (kManyValues / 4), &results[t].err,
                             slots + (uint64_t)blockIdx.x * kEncTile, recs + blockIdx.x, sh);
}

// ---- in place, large tensors: the first pass from the max pass's bounds of
// single float4s.  A slice (four values of a partition) of a group of quartic
// bytes lies in one float4 of the buffer's grid, or with m % 4 != 0 in two, and
// most have q = 0 throughout: the others alone are read.  The residuals of
// q != 0 go through LDS into the tile's list, which the compaction writes back:
// a few scattered stores cost far less in a pass of their own than mixed into a
// stream of reads.  After many steps, a call (through a pass over the 128-byte
// lines that reach the threshold, trits, and tiles from those | this pass): 40M
// values 143 | 128 us, 2^26 224 | 204, 150M 449 | 397, 2^28 785 | 757, most of
// them in zero runs 707 | 682.  At s = 1, where most waves are dense, 2^26 265 |
// 244 and 2^28 1096 | 1057.
//
// Residual v of the tile's value `local` (k * kEncTile + position) when `has`:
// the wave takes consecutive entries of the list with one LDS atomic; what falls
// past kFixCap is stored at dst at once.
__device__ __forceinline__ void fix_put(bool has, uint32_t local, float v, float* dst,
                                        uint32_t* left, uint2* fix) {
  const uint64_t all = __ballot(has);
  if (all == 0u) return;
  const uint32_t leader = (uint32_t)__ffsll((unsigned long long)all) - 1u;
  const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
      (uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0u));
  uint32_t base = 0u;
  if ((threadIdx.x & 63u) == leader) base = atomicAdd(left, (uint32_t)__popcll(all));
  base = (uint32_t)__shfl((int)base, (int)leader, 64);
  if (has) {
    if (base + rank < kFixCap)
      fix[base + rank] = make_uint2(local, __float_as_uint(v));
    else
      *dst = v;
  }
}

// Needed slices that a thread loads together.
constexpr int kSliceBatch = 4;

// Whether every value of group g (quartic bytes 4g .. 4g + 3 of the tile) exists
// and lies in float4s of the buffer that exist whole, so that they have bounds.
__device__ __forceinline__ bool group_whole(uint64_t n, uint32_t m, uint64_t q0,
                                            uint32_t tile_bytes, uint32_t g) {
  return g * 4u + 4u <= tile_bytes && 4ull * m + q0 + g * 4u + 7u <= n;
}

// The tile's quartic bytes into q.  h: the bounds of the thread's slices (group
// it = threadIdx.x + kThreads * it, partition k), the float4's that holds its
// first value below the next one's.  Where no thread of a wave
// needs more than two batches, every group starts from the all-zero byte 121
// and each needed slice moves its bytes by (t - 1) * 3^(4-k); other waves take
// the groups in turn with their needed slices loaded together, and store those
// that change at once: the list would not hold them (through the list and what
// it refused, s = 1, 40M values 170 against 154 us, 2^26 271 against 244).  The
// groups at the end of the tensor are taken value by value.  Ends with a barrier.
template <bool kGrid>
__device__ __forceinline__ void quantize_bounded_tile(
    float* __restrict__ r, uint64_t n, uint32_t m, const Scale& sc, uint64_t q0,
    uint32_t tile_bytes, const uint32_t (&h)[kGroupsPerThread][5], uint8_t* q, uint32_t* left,
    uint2* s_fix) {
  static_assert(kGroupsPerThread * 5 <= 32, "a thread's slices fit one mask");
  uint32_t* qw = reinterpret_cast<uint32_t*>(q);
  const uint32_t hU = __float_as_uint(sc.U) >> 16;
  auto group_of = [](uint32_t it) { return threadIdx.x + kThreads * it; };
  auto slice = [&](uint32_t it, uint32_t k) { return r + (uint64_t)k * m + q0 + group_of(it) * 4u; };
  uint32_t need = 0u;  // bit 5 * it + k
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    // on the grid the second bound is another slice's
    const uint32_t second = !kGrid && (((uint64_t)k * m + q0) & 3u) ? 0xffffu : 0u;
#pragma unroll
    for (int it = 0; it < kGroupsPerThread; ++it) {
      const uint32_t b =
          kGrid ? h[it][k] : umax32(h[it][k] & 0xffffu, (h[it][k] >> 16) & second);
      need |= (group_whole(n, m, q0, tile_bytes, group_of(it)) && b >= hU ? 1u : 0u)
              << (5 * it + k);
    }
  }
  // the four trits of slice k of group it
  auto quantize4 = [&](const float4& a, uint32_t (&t)[4]) {
    float4 o;
    t[0] = quantize_one(a.x, sc.M, sc.U, o.x);
    t[1] = quantize_one(a.y, sc.M, sc.U, o.y);
    t[2] = quantize_one(a.z, sc.M, sc.U, o.z);
    t[3] = quantize_one(a.w, sc.M, sc.U, o.w);
    return o;
  };
  // the same, its residuals to the list
  auto quantize = [&](bool has, const float4& a, uint32_t it, uint32_t k, uint32_t (&t)[4]) {
    const float4 o = quantize4(a, t);
    const uint32_t local = k * kEncTile + group_of(it) * 4u;
    float* e = slice(it, k);
    fix_put(has && t[0] != 1u, local, o.x, e, left, s_fix);
    fix_put(has && t[1] != 1u, local + 1u, o.y, e + 1, left, s_fix);
    fix_put(has && t[2] != 1u, local + 2u, o.z, e + 2, left, s_fix);
    fix_put(has && t[3] != 1u, local + 3u, o.w, e + 3, left, s_fix);
  };
  // a group at the end: its existing values one by one
  auto partial = [&](uint32_t g) {
    uint32_t w = 0u;
    for (uint32_t c = 0; c < 4u && g * 4u + c < tile_bytes; ++c) {
      uint32_t code = 0u;
      for (uint32_t k = 0; k < 5u; ++k) {
        const uint64_t e = (uint64_t)k * m + q0 + g * 4u + c;
        uint32_t t = 0u;  // the padding
        if (e < n) {
          float o;
          t = quantize_one(r[e], sc.M, sc.U, o);
          r[e] = o;
        }
        code = code * 3u + t;
      }
      w |= code << (8u * c);
    }
    return w;
  };
  auto store = [&](uint32_t it, uint32_t w) {
    const uint32_t g = group_of(it);
    if (g * 4u < tile_bytes) qw[g] = group_whole(n, m, q0, tile_bytes, g) ? w : partial(g);
  };
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  if (wave_max((uint32_t)__popc(need)) <= 2u * kSliceBatch) {
    uint32_t bytes[kGroupsPerThread];
#pragma unroll
    for (int it = 0; it < kGroupsPerThread; ++it) bytes[it] = 0x79797979u;  // five zeros each
    uint32_t rest = need;
#pragma unroll 1
    while (__ballot(rest != 0u)) {  // whole waves (fix_put)
      float4 a[kSliceBatch];
      uint32_t sel[kSliceBatch];
#pragma unroll
      for (int b = 0; b < kSliceBatch; ++b) {
        sel[b] = rest ? (uint32_t)__ffs(rest) - 1u : 32u;
        rest &= rest - 1u;
        a[b] = sel[b] < 32u ? ld4(slice(sel[b] / 5u, sel[b] % 5u)) : zero;
      }
#pragma unroll
      for (int b = 0; b < kSliceBatch; ++b) {
        const bool has = sel[b] < 32u;
        if (__ballot(has) == 0u) break;
        const uint32_t it = has ? sel[b] / 5u : 0u, k = has ? sel[b] % 5u : 0u;
        uint32_t t[4];
        quantize(has, a[b], it, k, t);
        // each byte stays in 0 .. 242, so the four move as one word
        const uint32_t by = (t[0] | (t[1] << 8) | (t[2] << 16) | (t[3] << 24)) - 0x01010101u;
        const uint32_t move = has ? by * trit_weight((int)k) : 0u;
#pragma unroll
        for (int gi = 0; gi < kGroupsPerThread; ++gi) bytes[gi] += (uint32_t)gi == it ? move : 0u;
      }
    }
#pragma unroll
    for (int it = 0; it < kGroupsPerThread; ++it) store(it, bytes[it]);
  } else {
#pragma unroll 1
    for (uint32_t it = 0; it < (uint32_t)kGroupsPerThread; ++it) {
      float4 a[5];
#pragma unroll
      for (int k = 0; k < 5; ++k)
        a[k] = (need >> (5 * it + k)) & 1u ? ld4(slice(it, k)) : zero;
      uint32_t w = 0u;
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        uint32_t t[4];
        const float4 o = quantize4(a[k], t);
        const uint32_t tp = t[0] | (t[1] << 8) | (t[2] << 16) | (t[3] << 24);
        if ((need >> (5 * it + k)) & 1u && tp != 0x01010101u) st4(slice(it, k), o);
        w += tp * trit_weight(k);
      }
      store(it, w);
    }
  }
  __syncthreads();
}

struct BoundShared {
  EncShared<kWaves> enc;
  uint2 fix[kFixCap];
  uint32_t left;  // residuals so far, also those that the list did not hold
  uint32_t scale[kWaves];
};

// The tile's quartic bytes in sh.enc.q and its list in sh; false: the tensor is
// refused, and its buffer keeps the sums.  report is called with the scale.
// Bound by its scattered reads.  kGrid: m % 4 == 0 (one bound a slice; with two
// 40M values took 134 us a call, with one 129).
template <bool kGrid, class Report>
__device__ __forceinline__ bool bounded_tile(float* __restrict__ r, uint64_t n, uint32_t m,
                                             uint64_t q0, uint32_t tile_bytes, float s,
                                             const uint32_t* __restrict__ partials, uint32_t np,
                                             const uint16_t* __restrict__ bound, BoundShared& sh,
                                             Report report) {
  if (threadIdx.x == 0) sh.left = 0u;
  // the bounds don't depend on M: loaded before the block reduces it
  typedef uint32_t pair __attribute__((aligned(2)));
  uint32_t h[kGroupsPerThread][5];
#pragma unroll
  for (int it = 0; it < kGroupsPerThread; ++it) {
    const uint32_t g = threadIdx.x + kThreads * it;
    const bool whole = group_whole(n, m, q0, tile_bytes, g);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const uint16_t* p = bound + (((uint64_t)k * m + q0 + g * 4u) >> 2);
      h[it][k] = 0u;
      if (whole) h[it][k] = kGrid ? *p : *reinterpret_cast<const pair*>(p);
    }
  }
  const Scale sc = finish_scale(partials, np, s, sh.scale);  // holds a barrier
  report(sc);
  if (sc.bad) return false;
  quantize_bounded_tile<kGrid>(r, n, m, sc, q0, tile_bytes, h, sh.enc.q, &sh.left, sh.fix);
  return true;
}

template <bool kGrid, class Report>
__device__ __forceinline__ void encode_bounded_tile(float* __restrict__ r, uint64_t n, uint32_t m,
                                                    uint32_t t, float s,
                                                    const uint32_t* __restrict__ partials,
                                                    uint32_t np,
                                                    const uint16_t* __restrict__ bound,
                                                    uint8_t* __restrict__ slot,
                                                    TileRec* __restrict__ rec,
                                                    uint2* __restrict__ fix, BoundShared& sh,
                                                    Report report) {
  const uint64_t q0 = (uint64_t)t * kEncTile;
  const uint32_t tile_bytes = (uint32_t)umin64(kEncTile, (uint64_t)m - q0);
  if (!bounded_tile<kGrid>(r, n, m, q0, tile_bytes, s, partials, np, bound, sh, report)) return;
  const uint32_t left = umin32(sh.left, kFixCap);
  if (threadIdx.x < left) fix[threadIdx.x] = sh.fix[threadIdx.x];
  static_assert(kFixCap <= kThreads, "an entry per thread");
  const uint32_t lo = 16u * threadIdx.x;
  const uint32_t cnt = lo < tile_bytes ? umin32(16u, tile_bytes - lo) : 0u;
  const uint4 w[1] = {cnt ? *reinterpret_cast<const uint4*>(sh.enc.q + lo)
                          : make_uint4(0, 0, 0, 0)};
  const uint32_t nz[1] = {cnt ? nonzero_mask16_spread(w[0], cnt) : 0u};
  encode_tile_runs<kThreads>(w, nz, tile_bytes, slot, rec, sh.enc, left);
}

template <bool kGrid>
__global__ __launch_bounds__(kThreads) void tlc_quant_encode_bounds_kernel(
    float* __restrict__ r, uint64_t n, uint32_t m, float s, const uint32_t* __restrict__ partials,
    uint32_t np, const uint16_t* __restrict__ bound, uint8_t* __restrict__ slots,
    TileRec* __restrict__ recs, uint2* __restrict__ fix, Ctrl* __restrict__ ctrl, HostMirror hm) {
  __shared__ BoundShared sh;
  const uint32_t t = blockIdx.x;
  encode_bounded_tile<kGrid>(r, n, m, t, s, partials, np, bound, slots + (uint64_t)t * kEncTile,
                             recs + t, fix + (uint64_t)t * kFixCap, sh, [&](const Scale& sc) {
                               if (t == 0 && threadIdx.x == 0) {
                                 ctrl->enc.err = sc.bad;
                                 ctrl->enc.scale = sc.M;
                                 host_put_result(hm.res, sc.bad, sc.M);
                               }
                             });
}

// The tiles of a batch's middle tensors.
__global__ __launch_bounds__(kThreads) void tlc_quant_encode_bounds_many_kernel(
    const EncDesc* __restrict__ descs, uint32_t count, const uint32_t* __restrict__ partials,
    const uint16_t* __restrict__ bound, uint8_t* __restrict__ slots, TileRec* __restrict__ recs,
    uint2* __restrict__ fix, EncResult* __restrict__ results, HostMirror hm) {
  __shared__ BoundShared sh;
  const uint32_t T = blockIdx.x;
  const uint32_t t = find_desc(descs, count, T, [](const EncDesc& d) { return d.tile0; });
  const EncDesc& d = descs[t];
  auto report = [&](const Scale& sc) {
    if (T == d.tile0 && threadIdx.x == 0) {
      results[t].err = sc.bad;
      results[t].scale = sc.M;
      host_put_result(hm.res ? hm.res + t : nullptr, sc.bad, sc.M);
    }
  };
  auto tile = [&](auto grid) {
    encode_bounded_tile<decltype(grid)::value>(
        uniform_ptr(d.r), d.n, d.m, T - d.tile0, d.s, partials + d.blk0, d.nblk,
        bound + (uint64_t)d.v0 * (kManyValues / 4), slots + (uint64_t)T * kEncTile, recs + T,
        fix + (uint64_t)T * kFixCap, sh, report);
  };
  if (d.m % 4u == 0u)
    tile(std::true_type{});
  else
    tile(std::false_type{});
}

// Pass B: one wave per chunk of 64 tiles: every tile's prefix within its
// chunk (an ordered wave scan) and the chunk's summary.  The last block to
// finish (a count of finished blocks, each block's summaries released
// before its count) then scans the chunk summaries in place, each entry
// becoming its chunk's exclusive prefix, and clears the count for the next
// call.
constexpr uint32_t kChunkTiles = 64;

__global__ __launch_bounds__(kThreads) void tlc_zre_chunk_kernel(
    const TileRec* __restrict__ recs, uint32_t ntiles, uint64_t* __restrict__ local_pre,
    uint64_t* __restrict__ chunk_agg, Ctrl* __restrict__ ctrl) {
  __shared__ RunSum s_wave[kWaves];
  __shared__ uint32_t s_last;
  if (ctrl->enc.err) return;  // pass A refused the tensor (every block returns)
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  const uint32_t nchunks = (ntiles + kChunkTiles - 1) / kChunkTiles;
  const uint32_t c = blockIdx.x * kWaves + wid;
  if (c < nchunks) {  // whole waves
    const uint32_t i = c * kChunkTiles + lane;
    RunSum a = rs_identity();
    if (i < ntiles) a.v = recs[i].agg;
    const RunSum incl = wave_incl_scan_rs(a);
    const RunSum ex = wave_prev_lane_rs(incl);
    if (i < ntiles) local_pre[i] = ex.v;
    if (lane == 63) chunk_agg[c] = incl.v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    s_last = atomicAdd(&ctrl->chunk_done, 1u) == gridDim.x - 1u ? 1u : 0u;
  }
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  // thread j scans a run of consecutive chunks
  const uint32_t per = (nchunks + kThreads - 1) / kThreads;
  const uint32_t j0 = umin32(threadIdx.x * per, nchunks), j1 = umin32(j0 + per, nchunks);
  RunSum mine = rs_identity();
  for (uint32_t j = j0; j < j1; ++j) {
    RunSum a;
    a.v = chunk_agg[j];
    mine = rs_combine(mine, a);
  }
  const RunSum incl = wave_incl_scan_rs(mine);
  const RunSum ex = wave_prev_lane_rs(incl);
  if (lane == 63) s_wave[wid] = incl;
  __syncthreads();
  RunSum p = rs_identity();
  for (uint32_t w = 0; w < wid; ++w) p = rs_combine(p, s_wave[w]);
  p = rs_combine(p, ex);
  for (uint32_t j = j0; j < j1; ++j) {  // every load of the run came before these stores
    RunSum a;
    a.v = chunk_agg[j];
    chunk_agg[j] = p.v;
    p = rs_combine(p, a);
  }
  if (threadIdx.x == 0)
    __hip_atomic_store(&ctrl->chunk_done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Pass C, the compaction: one wave per tile.  Prefix = the chunk's prefix
// combined with the tile's prefix within the chunk; then the leading run's
// codes and the slot; the last tile also writes the remainder of a run that
// ends the stream and the stream length.  Every write is clamped to
// the m-byte output (the stream never exceeds m bytes; the clamp only
// contains a logic error).
// kPer > 0 (at most kPer * kThreads tiles): no pass B; the block combines the
// summaries of all tiles before its first one itself, kPer per thread.
// fix: the residuals that the bounded first pass left (null: another one ran).
template <uint32_t kPer>
__device__ __forceinline__ void compact_tiles(
    const TileRec* __restrict__ recs, const uint64_t* __restrict__ chunk_pre,
    const uint64_t* __restrict__ local_pre, const uint8_t* __restrict__ slots, uint32_t m,
    uint32_t ntiles, uint32_t t0, uint8_t* __restrict__ out, EncResult* __restrict__ res,
    EncResult* hres, const uint2* __restrict__ fix, float* __restrict__ r, uint64_t n) {
  if (res->err) return;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t t = t0 + (threadIdx.x >> 6);
  RunSum P;
  if constexpr (kPer != 0u) {
    __shared__ uint64_t s_wave[kWaves];
    RunSum a[kPer];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {  // tiles kPer * thread + i, in order
      const uint32_t u = kPer * threadIdx.x + i;
      a[i] = rs_identity();
      if (u < t0) a[i].v = recs[u].agg;
    }
    RunSum sum = a[0];
#pragma unroll
    for (uint32_t i = 1; i < kPer; ++i) sum = rs_combine(sum, a[i]);
    sum = wave_incl_scan_rs(sum);
    if (lane == 63) s_wave[threadIdx.x >> 6] = sum.v;
    __syncthreads();
    P = rs_identity();
#pragma unroll 1
    for (uint32_t i = 0; i < kWaves; ++i) {
      RunSum b;
      b.v = s_wave[i];
      P = rs_combine(P, b);
    }
#pragma unroll 1
    for (uint32_t u = t0; u < t && u < ntiles; ++u) {  // the block's own earlier tiles
      RunSum b;
      b.v = recs[u].agg;
      P = rs_combine(P, b);
    }
  }
  if (t >= ntiles) return;  // whole waves; nothing below synchronises the block
  if constexpr (kPer == 0u) {
    RunSum cp, lp;
    cp.v = chunk_pre[t / kChunkTiles];
    lp.v = local_pre[t];
    P = rs_combine(cp, lp);
  }
  const TileRec rec = recs[t];
  const uint64_t q0 = (uint64_t)t * kEncTile;
  const uint32_t tile_bytes = (uint32_t)umin64(kEncTile, (uint64_t)m - q0);
  const uint32_t off = rs_emitted(P);
  const uint32_t grown = rs_phase(P) + rec.lead;  // the open run after the leading 121s
  const uint32_t n255 = grown / kRunMax, rho = grown % kRunMax;
  const bool rest = rec.lead < tile_bytes;
  const uint32_t code = (rest && rho) ? 1u : 0u;
  for (uint32_t i = lane; i < n255; i += 64u)
    if (off + i < m) out[off + i] = (uint8_t)kFullChunk;
  if (code && lane == 0 && off + n255 < m) out[off + n255] = (uint8_t)rs_code(rho);
  if (rest) {
    const uint32_t at = off + n255 + code;
    const uint32_t len = umin32(rec.len, tile_bytes);
    // dword loads from the slot (4096-byte aligned, len <= 4096), byte stores
    for (uint32_t i = 4u * lane; i < len; i += 256u) {
      const uint32_t w = *reinterpret_cast<const uint32_t*>(slots + q0 + i);
#pragma unroll
      for (uint32_t b = 0; b < 4u; ++b)
        if (i + b < len && at + i + b < m) out[at + i + b] = (uint8_t)(w >> (8u * b));
    }
  }
  if (fix) {
    const uint32_t left = umin32(rec.left, kFixCap);
    for (uint32_t i = lane; i < left; i += 64u) {
      const uint2 f = fix[(uint64_t)t * kFixCap + i];
      const uint64_t e = (uint64_t)(f.x / (uint32_t)kEncTile) * m + q0 + f.x % (uint32_t)kEncTile;
      if (e < n) r[e] = __uint_as_float(f.y);
    }
  }
  if (t + 1 == ntiles && lane == 0) {  // a run that ends the stream; the length
    RunSum a;
    a.v = rec.agg;
    const RunSum T = rs_combine(P, a);
    const uint32_t total = rs_total(T);
    if (rs_phase(T) && total >= 1u && total - 1u < m)
      out[total - 1u] = (uint8_t)rs_code(rs_phase(T));
    res->len = total;
    if (hres) host_put(&hres->len, total);
  }
}

template <uint32_t kPer>
__global__ __launch_bounds__(kThreads) void tlc_zre_compact_kernel(
    const TileRec* __restrict__ recs, const uint64_t* __restrict__ chunk_pre,
    const uint64_t* __restrict__ local_pre, const uint8_t* __restrict__ slots, uint32_t m,
    uint32_t ntiles, uint8_t* __restrict__ out, Ctrl* __restrict__ ctrl, HostMirror hm,
    const uint2* __restrict__ fix, float* __restrict__ r, uint64_t n) {
  compact_tiles<kPer>(recs, chunk_pre, local_pre, slots, m, ntiles, blockIdx.x * kWaves, out,
                      &ctrl->enc, hm.res, fix, r, n);
}

// A batch's middle tensors of at most kPer * kThreads tiles: cblk0 counts the
// compaction's blocks.
template <uint32_t kPer>
__global__ __launch_bounds__(kThreads) void tlc_zre_compact_many_kernel(
    const EncDesc* __restrict__ descs, uint32_t count, const TileRec* __restrict__ recs,
    const uint8_t* __restrict__ slots, EncResult* __restrict__ results, HostMirror hm,
    const uint2* __restrict__ fix) {
  const uint32_t t =
      find_desc(descs, count, blockIdx.x, [](const EncDesc& d) { return d.cblk0; });
  const EncDesc& d = descs[t];
  compact_tiles<kPer>(recs + d.tile0, nullptr, nullptr, slots + (uint64_t)d.tile0 * kEncTile, d.m,
                      (d.m + kEncTile - 1) / kEncTile, (blockIdx.x - d.cblk0) * kWaves,
                      uniform_ptr(d.out), results + t, hm.res ? hm.res + t : nullptr,
                      fix ? fix + (uint64_t)d.tile0 * kFixCap : nullptr, uniform_ptr(d.r), d.n);
}

// ---------------------------------------------------------------- small tensors
// A tile of a small tensor, or of one tensor of a batch, in one go: kT threads
// of kG groups of four quartic bytes each.  Every thread loads the values of
// its own bytes (five slices of x and r per group) before anything else, so
// the tile takes one round trip to memory; the values then stay in registers
// for M, Eq. 2, the residuals and the quartic bytes.
//
// M: a tensor of one tile is all in its block.  Of a tensor of at most
// kExchangeTiles tiles, every tile publishes its largest |acc| in a word of
// its own and reads the others' (nothing is written before all have come), so
// that no check pass runs before.  Those that follow it may not have started:
// a tile that has waited a while reads their values itself (help_maxima), so
// that any number of resident blocks will do.  A longer tensor (of a
// no-allocation call only) takes kT 512 and has its M from a check pass
// (partials).
//
// The zero-run encoding is the first pass's (from the gaps between non-121
// bytes, from the tile's first one on).  Its place in the stream and the
// leading run's codes need the tiles before: every tile publishes its summary
// and, with at most kExchangeTiles, reads all summaries before its own at
// once; in a longer tensor they are chained by decoupled look-back.
//
// Bound by latency (a few dependent round trips and some 1500 instructions per
// wave): tiles of 2048 quartic bytes spread a million values over 103 blocks.
template <int kT, int kG>
struct TileShared {
  uint32_t red[kT / 64];
  uint32_t red2[kT / 64];
  uint32_t lead;   // the tile's first non-121 byte
  uint32_t fault;
  uint32_t help;   // some tile's maximum has not come
  // what the first waves read of the other tiles: maxima, then summaries
  uint64_t wave[kExchangeTiles / 64];
  LookShared<kT / 64> look;
  __align__(16) uint8_t out[kT * kG * 4 + 16];
};

// Where one tensor of a launch lies and where its results go.
struct TileJob {
  const float* x;
  float* r;
  uint8_t* out;
  uint64_t n;
  uint32_t m;
  float s;
  const uint32_t* partials;  // the check pass's (kT 512)
  uint32_t np;
  uint32_t floor;  // status slot of the tensor's first tile
  EncResult* res;
  EncResult* hres;
};

// Waits until every lane's word *p (of the lanes with `mine`) has ready(word);
// each lane gets its own word, the others 0.  False when the wait runs past
// `limit` polls.
template <class Ready>
__device__ __forceinline__ bool wait_words(const uint64_t* p, bool mine, Ready ready,
                                           uint32_t limit, uint64_t* w) {
  *w = 0u;
  for (uint32_t spins = 0;; ++spins) {
    if (mine) *w = status_read(p);
    if (__ballot(mine && !ready(*w)) == 0u) return true;
    if (spins >= limit) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

// The polls (about a microsecond each) before a tile stops waiting for the
// others' maxima.  The stress build helps at the first poll that misses one.
#ifdef TLC_DELAY_INJECT
constexpr uint32_t kHelpPolls = 0u;
#else
constexpr uint32_t kHelpPolls = 1u << 12;
#endif

// The largest |acc| of a whole tensor by one block, for a tile whose wait for
// the others' maxima has run out: those it waits for may not have started, and
// where few blocks are resident (a stream with few CUs, other launches that
// wait) they cannot start before it ends.  A maximum that is still missing is
// taken from the tile's values and published for everybody.  That tile writes
// its buffer only after it has published: where its word is still missing
// after the values have been read, they were the ones before the call; where
// it has come in between, it counts and what was read does not.
template <int kT>
__device__ __forceinline__ uint32_t help_maxima(const TileJob& J, uint32_t tile_values,
                                                uint32_t tiles, uint64_t* __restrict__ maxima,
                                                uint32_t epoch, uint32_t* red, uint64_t* word) {
  uint32_t mx = 0u;
#pragma unroll 1
  for (uint32_t t = 0; t < tiles; ++t) {
    __syncthreads();  // *word and red are free
    if (threadIdx.x == 0) *word = status_read(&maxima[t]);
    __syncthreads();
    if ((uint32_t)(*word >> 32) != epoch) {
      const uint64_t q0 = (uint64_t)t * tile_values;
      const uint32_t len = (uint32_t)umin64(tile_values, J.m - q0);
      uint32_t v = 0u;
#pragma unroll 1
      for (int k = 0; k < 5; ++k) {
        const uint64_t base = (uint64_t)k * J.m + q0;
        const uint32_t lim = J.n > base ? (uint32_t)umin64(J.n - base, len) : 0u;
        for (uint32_t i = threadIdx.x; i < lim; i += kT)
          v = max(v, abs_bits(J.x[base + i] + J.r[base + i]));
      }
      v = block_max<kT / 64>(v, red);  // every thread's values are read
      if (threadIdx.x == 0) {
        uint64_t w = status_read(&maxima[t]);
        if ((uint32_t)(w >> 32) != epoch) {
          w = ((uint64_t)epoch << 32) | v;
          status_publish(&maxima[t], w);
        }
        *word = w;
      }
      __syncthreads();
    }
    mx = max(mx, (uint32_t)*word);
  }
  return mx;
}

template <int kT, int kG>
__device__ __forceinline__ void encode_tile(const TileJob& J, uint32_t lt, bool in_place,
                                            uint64_t* __restrict__ status,
                                            uint64_t* __restrict__ maxima, uint32_t epoch,
                                            Ctrl* __restrict__ ctrl, uint32_t* hfault,
                                            TileShared<kT, kG>& sh) {
  constexpr int kW = kT / 64;
  constexpr uint32_t kBytes = 4u * kG;        // quartic bytes per thread
  constexpr uint32_t kTile = kT * kBytes;
  static_assert(kBytes <= 16, "the gap forms take at most 16 bytes per thread");
  constexpr uint32_t kReaders = kExchangeTiles / 64;  // waves that read a tensor's words
  static_assert(kReaders <= kW && kExchangeTiles % 64 == 0, "a word per lane");
  const uint64_t n = J.n, m = J.m;
  const uint64_t q0 = (uint64_t)lt * kTile;
  const uint32_t tile_bytes = (uint32_t)umin64(kTile, m - q0);
  const uint32_t tiles = (uint32_t)((m + kTile - 1) / kTile);
  constexpr bool kChained = kT > kTileThreads;
  const bool last_tile = q0 + kTile >= m;
  const uint32_t lo = threadIdx.x * kBytes;
  const uint32_t cnt = lo < tile_bytes ? umin32(kBytes, tile_bytes - lo) : 0u;
  const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
  auto fault_out = [&]() {
    __hip_atomic_store(&ctrl->fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    host_put(hfault, 1u);
  };
  if (threadIdx.x == 0) sh.fault = sh.help = 0u;  // read after a barrier

  // ---- step 1: acc = x + r, the thread's 20 * kG values; 0 past the end.
  // Of partition k the tile holds the first lim[k] of the block's bytes'
  // values (all but the last tile: all of them), from a place that is the same
  // for the whole block.
  uint32_t lim[5], least = kTile;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const uint64_t base = (uint64_t)k * m + q0;
    lim[k] = n > base ? (uint32_t)umin64(n - base, tile_bytes) : 0u;
    least = umin32(least, lim[k]);
  }
  auto part = [&](int k) { return lim[k] ? (uint64_t)k * m + q0 : 0u; };  // in bounds in any case
  float4 v[kG][5], b[kG][5];
  bool full[kG];
#pragma unroll
  for (int g = 0; g < kG; ++g) {
    const uint32_t i = lo + 4u * g;
    full[g] = i + 4u <= least;
    if (full[g]) {
#pragma unroll
      for (int k = 0; k < 5; ++k) v[g][k] = ld4(J.r + part(k) + i);
#pragma unroll
      for (int k = 0; k < 5; ++k) b[g][k] = ld4(J.x + part(k) + i);
    } else if (i < tile_bytes) {
      // the group at the end, without branches: a value that does not exist
      // is read as the last one that does, and zeroed below
      auto one = [&](const float* p, int k, uint32_t c) {
        return (p + part(k))[umin32(i + c, lim[k] ? lim[k] - 1u : 0u)];
      };
#pragma unroll
      for (int k = 0; k < 5; ++k)
        v[g][k] = make_float4(one(J.r, k, 0), one(J.r, k, 1), one(J.r, k, 2), one(J.r, k, 3));
#pragma unroll
      for (int k = 0; k < 5; ++k)
        b[g][k] = make_float4(one(J.x, k, 0), one(J.x, k, 1), one(J.x, k, 2), one(J.x, k, 3));
    }
  }
#pragma unroll
  for (int g = 0; g < kG; ++g) {
    const uint32_t i = lo + 4u * g;
    if (i < tile_bytes) {
#pragma unroll
      for (int k = 0; k < 5; ++k)
        v[g][k] = make_float4(b[g][k].x + v[g][k].x, b[g][k].y + v[g][k].y,
                              b[g][k].z + v[g][k].z, b[g][k].w + v[g][k].w);
      if (!full[g]) {
#pragma unroll
        for (int k = 0; k < 5; ++k)
          v[g][k] = make_float4(i < lim[k] ? v[g][k].x : 0.f, i + 1u < lim[k] ? v[g][k].y : 0.f,
                                i + 2u < lim[k] ? v[g][k].z : 0.f,
                                i + 3u < lim[k] ? v[g][k].w : 0.f);
      }
    }
  }

  // ---- Eq. 1
  Scale sc;
  if constexpr (!kChained) {
    uint32_t mx = 0u;
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      if (cnt > 4u * g) {
#pragma unroll
        for (int k = 0; k < 5; ++k)
          mx = max(mx, max(max(abs_bits(v[g][k].x), abs_bits(v[g][k].y)),
                           max(abs_bits(v[g][k].z), abs_bits(v[g][k].w))));
      }
    }
    mx = block_max<kW>(mx, sh.red);
    if (tiles > 1u) {
      if (threadIdx.x == 0)
        status_publish(&maxima[J.floor + lt], ((uint64_t)epoch << 32) | mx);
      if (wid < kReaders) {
        uint64_t w;
        const bool ok = wait_words(
            &maxima[J.floor + threadIdx.x], threadIdx.x < tiles,
            [&](uint64_t v) { return (uint32_t)(v >> 32) == epoch; }, kHelpPolls, &w);
        const uint32_t wm = wave_max((uint32_t)w);
        if (lane == 0) {
          sh.wave[wid] = wm;
          if (!ok) sh.help = 1u;
        }
      }
      __syncthreads();
      if (sh.help) {
        mx = help_maxima<kT>(J, kTile, tiles, maxima + J.floor, epoch, sh.red, &sh.wave[0]);
        __syncthreads();  // sh.wave is written again below
      } else {
#pragma unroll
        for (uint32_t i = 0; i < kReaders; ++i) mx = max(mx, (uint32_t)sh.wave[i]);
      }
    }
    sc = scale_of(mx, J.s);
  } else {
    sc = finish_scale<kT>(J.partials, J.np, J.s, sh.red);
  }
  // one of the last tile's threads reports for the whole tensor
  if (sc.bad && last_tile && threadIdx.x == 0) {
    J.res->err = 1u;
    J.res->len = 0u;
    J.res->scale = 0.0f;
    host_put_all(J.hres, 1u, 0u, 0.0f);
  }
  auto store = [&](int g, int k, const float4& o) {
    const uint32_t i = lo + 4u * g;
    float* p = J.r + part(k) + i;
    if (full[g]) {
      st4(p, o);
    } else {
      if (i < lim[k]) p[0] = o.x;
      if (i + 1u < lim[k]) p[1] = o.y;
      if (i + 2u < lim[k]) p[2] = o.z;
      if (i + 3u < lim[k]) p[3] = o.w;
    }
  };
  if (sc.bad) {
    // NaN/Inf or overflow: no stream, the buffer as it was or, in place, the
    // sums
    if (in_place) {
#pragma unroll
      for (int g = 0; g < kG; ++g)
        if (cnt > 4u * g)
#pragma unroll
          for (int k = 0; k < 5; ++k) store(g, k, v[g][k]);
    }
    return;
  }

  // ---- Eq. 2, residuals, quartic pack: a byte is 121 + sum of 3^(4-k) * q_k,
  // exact in floats, and padding is q = -1 (trit 0)
  uint32_t w[kG];
#pragma unroll
  for (int g = 0; g < kG; ++g) {
    w[g] = 0x79797979u;
    if (cnt > 4u * g) {
      float c0 = 121.f, c1 = 121.f, c2 = 121.f, c3 = 121.f;
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const float wt = (float)trit_weight(k);
        const float4 a = v[g][k];
        float4 q = make_float4(quantize_q(a.x, sc.U), quantize_q(a.y, sc.U),
                               quantize_q(a.z, sc.U), quantize_q(a.w, sc.U));
        store(g, k, make_float4(residual_of(a.x, q.x, sc.M), residual_of(a.y, q.y, sc.M),
                                residual_of(a.z, q.z, sc.M), residual_of(a.w, q.w, sc.M)));
        if (!full[g]) {
          const uint32_t i = lo + 4u * g;
          q.x = i < lim[k] ? q.x : -1.f;
          q.y = i + 1u < lim[k] ? q.y : -1.f;
          q.z = i + 2u < lim[k] ? q.z : -1.f;
          q.w = i + 3u < lim[k] ? q.w : -1.f;
        }
        c0 = __builtin_fmaf(q.x, wt, c0);
        c1 = __builtin_fmaf(q.y, wt, c1);
        c2 = __builtin_fmaf(q.z, wt, c2);
        c3 = __builtin_fmaf(q.w, wt, c3);
      }
      w[g] = __builtin_amdgcn_cvt_pk_u8_f32(
          c3, 3u, __builtin_amdgcn_cvt_pk_u8_f32(
                      c2, 2u, __builtin_amdgcn_cvt_pk_u8_f32(
                                  c1, 1u, __builtin_amdgcn_cvt_pk_u8_f32(c0, 0u, 0u))));
    }
  }

  // ---- Section 3.3 inside the tile, as in tlc_quant_encode_kernel
  uint32_t nz = 0u;
#pragma unroll
  for (int g = 0; g < kG; ++g) nz |= nonzero_byte_mask4(w[g]) << (4 * g);
  nz &= (1u << cnt) - 1u;
  const uint32_t last = nz ? lo + 32u - (uint32_t)__builtin_clz(nz) : 0u;  // position + 1
  const ScanU32 pm = block_scan_max_u32<kW>(last, sh.red2);
  const int prev = (int)pm.excl - 1;  // the previous non-121 byte, -1 if none
  if (nz != 0u && prev < 0) sh.lead = lo + (uint32_t)__builtin_ctz(nz);
  const uint32_t trail = tile_bytes - pm.total;  // 121s after the last non-121 byte
  const uint32_t mine = rs_gaps_len(nz, lo, prev) +
                        (nz != 0u && last == pm.total ? trail / kRunMax : 0u);
  // every output byte that is not a remainder code or a non-121 byte is a 255
#pragma unroll
  for (int g = 0; g < kG; ++g)
    reinterpret_cast<uint32_t*>(sh.out)[kG * threadIdx.x + g] = ~0u;
  if (threadIdx.x < 4u) reinterpret_cast<uint32_t*>(sh.out)[kG * kT + threadIdx.x] = ~0u;
  const ScanU32 off = block_scan_u32<kW>(mine, sh.red);
  const bool some = pm.total != 0u;
  const uint32_t lead = some ? sh.lead : tile_bytes;
  const RunSum agg =
      some ? rs_combine(rs_zero_run(lead), rs_make(0u, 0u, trail % kRunMax, off.total))
           : rs_zero_run(tile_bytes);
  // the tiles after this one can go on before it has emitted anything
  if (tiles > 1u && threadIdx.x == 0)
    status_publish(&status[J.floor + lt],
                   EncSW::pack(rs_to_payload(agg), lt == 0 ? kFlagPrefix : kFlagAgg, epoch));
  uint32_t o = off.excl;
  auto put = [&](uint32_t c) {
    if (o < sizeof(sh.out)) sh.out[o] = (uint8_t)c;
    ++o;
  };
  // the bytes as one 64-bit value: an array indexed at run time would be moved
  // to LDS, at a place each wave computes from the dispatch packet, which lies
  // in host memory (in a batch of 335 tensors the waves waited up to 14 us)
  uint64_t bytes = w[0];
  if (kG > 1) bytes |= (uint64_t)w[kG > 1 ? 1 : 0] << 32;
  rs_gaps_emit(nz, lo, prev, [bytes](uint32_t i) { return (uint32_t)(bytes >> (8u * i)) & 255u; },
               put, [&](uint32_t k) { o += k; });
  static_assert(kG <= 2, "the thread's bytes fit 64 bits");
  RunSum P = rs_identity();
  if (lt != 0) {
    if constexpr (!kChained) {
      if (wid < kReaders) {  // lane i of wave w reads tile 64w + i's summary
        uint64_t w;
        const bool mine = threadIdx.x < lt;
        const bool ok = wait_words(
            &status[J.floor + threadIdx.x], mine,
            [&](uint64_t v) { return EncSW::epoch(v) == epoch && EncSW::flag(v) != 0u; },
            kSpinLimit, &w);
        RunSum a = rs_identity();
        if (mine) a = rs_from_payload(EncSW::payload(w));
        a = wave_incl_scan_rs(a);
        if (lane == 63) {
          sh.wave[wid] = a.v;
          if (!ok) {
            sh.fault = 1u;
            fault_out();
          }
        }
      }
    } else {
      P = rs_from_payload(lookback_block<EncSW, kW>(status, lt, rs_to_payload(agg),
                                                    rs_to_payload(rs_identity()), epoch, EncOp(),
                                                    sh.look, &sh.fault));
      if (sh.fault) {
        if (threadIdx.x == 0) fault_out();
        return;
      }
    }
    if constexpr (!kChained) {
      __syncthreads();
      if (sh.fault) return;
#pragma unroll 1
      for (uint32_t i = 0; i < kReaders; ++i) {
        RunSum a;
        a.v = sh.wave[i];
        P = rs_combine(P, a);
      }
    }
  } else {
    __syncthreads();
  }

  // ---- the tile's part of the stream; the clamps only keep a logic error
  // from writing outside the m-byte output buffer
  const uint32_t at0 = rs_emitted(P);
  const uint32_t grown = rs_phase(P) + lead;  // the open run after the leading 121s
  const uint32_t n255 = grown / kRunMax, rho = grown % kRunMax;
  const uint32_t code = (some && rho) ? 1u : 0u;
  for (uint32_t i = threadIdx.x; i < n255; i += kT)
    if (at0 + i < m) J.out[at0 + i] = (uint8_t)kFullChunk;
  if (code && threadIdx.x == 0 && at0 + n255 < m) J.out[at0 + n255] = (uint8_t)rs_code(rho);
  const uint32_t at = at0 + n255 + code;
  const uint32_t len = umin32(off.total, kTile);
  for (uint32_t i = threadIdx.x; i < len; i += kT)
    if (at + i < m) J.out[at + i] = sh.out[i];
  if (last_tile && threadIdx.x == 0) {  // a run that ends the stream; the length
    const RunSum T = rs_combine(P, agg);
    const uint32_t total = rs_total(T);
    if (rs_phase(T) && total >= 1u && total - 1u < m)
      J.out[total - 1u] = (uint8_t)rs_code(rs_phase(T));
    J.res->err = 0u;
    J.res->len = total;
    J.res->scale = sc.M;
    host_put_all(J.hres, 0u, total, sc.M);
  }
}

// One tensor.  A chained one takes tiles of twice the size (kT 512): its
// look-back is half as long (8,388,608 values: 42 against 51 us).  (Tensors of
// this size in a context take the three passes, alone or in a batch: chained in
// the batch's launch, ten of 2M values took 131 us, four of 8M 197, one of 25.6M
// 166; before the exchange, in 4096-byte tiles, 108, 148 and 126.)
template <int kT>
__global__ __launch_bounds__(kT) void tlc_quant_encode_chained_kernel(
    const float* __restrict__ x, float* __restrict__ r, uint64_t n, uint32_t m, float s,
    bool in_place, const uint32_t* __restrict__ partials, uint32_t np, uint8_t* __restrict__ out,
    uint64_t* __restrict__ status, uint64_t* __restrict__ maxima, uint32_t ticket_base,
    uint32_t epoch, Ctrl* __restrict__ ctrl, HostMirror hm) {
  __shared__ TileShared<kT, kTileGroups> sh;
  __shared__ uint32_t s_tile;
  uint32_t tile = 0u;
  if (m > kT * kTileGroups * 4u) {  // more than one tile
    if (threadIdx.x == 0) s_tile = take_ticket(&ctrl->enc_ticket) - ticket_base;
    __syncthreads();
    tile = uniform32(s_tile);
  }
  const TileJob J = {x, r, out, n, m, s, partials, np, 0u, &ctrl->enc, hm.res};
  encode_tile<kT, kTileGroups>(J, tile, in_place, status, maxima, epoch, ctrl, hm.fault, sh);
}

// Many tensors: the first `shared` tiles, of tensors of more than one, go by
// ticket, and owner says whose each is; every other block has a tensor of its
// own, in descriptor order, and takes none (hundreds of blocks queue for the
// one counter).
__global__ __launch_bounds__(kTileThreads) void tlc_quant_encode_batch_kernel(
    const EncDesc* __restrict__ descs, uint32_t shared, const uint16_t* __restrict__ owner,
    bool in_place, EncResult* __restrict__ results, uint64_t* __restrict__ status,
    uint64_t* __restrict__ maxima, uint32_t ticket_base, uint32_t epoch, Ctrl* __restrict__ ctrl,
    HostMirror hm) {
  __shared__ TileShared<kTileThreads, kTileGroups> sh;
  __shared__ uint32_t s_tile;
  __shared__ EncDesc s_desc;
  uint32_t T = blockIdx.x;
  if (T < shared) {
    if (threadIdx.x == 0) s_tile = take_ticket(&ctrl->enc_ticket) - ticket_base;
    __syncthreads();
    T = uniform32(s_tile);
  }
  const uint32_t t = owner[T];
  // one read of the descriptor per block: it may lie in host memory
  if (threadIdx.x < sizeof(EncDesc) / 4)
    reinterpret_cast<uint32_t*>(&s_desc)[threadIdx.x] =
        reinterpret_cast<const uint32_t*>(descs + t)[threadIdx.x];
  __syncthreads();
  const uint32_t lt = uniform32(T - s_desc.tile0), ut = uniform32(t);
  const TileJob J = {
      uniform_ptr(s_desc.x),
      uniform_ptr(s_desc.r),
      uniform_ptr(s_desc.out),
      uniform64(s_desc.n),
      uniform32(s_desc.m),
      s_desc.s,
      nullptr,
      0u,
      uniform32(s_desc.tile0),
      results + ut,
      hm.res ? hm.res + ut : nullptr};
  encode_tile<kTileThreads, kTileGroups>(J, lt, in_place, status, maxima, epoch, ctrl, hm.fault,
                                         sh);
}

// ---------------------------------------------------------------- comparison modes
// Quantization + quartic pack without zero-run encoding (the quartic bytes
// are the payload, m bytes) goes through trits as well: one flat pass over the
// values leaves them, whatever m and the alignment, and tlc_quant_pack_kernel
// forms the bytes.

// Stochastic 3-value quantization of x with Philox random words (no error
// feedback: there is no buffer) into trits.  One Philox4x32-10 call serves a
// float4.  Bound by the multiplies of its rounds.
__global__ __launch_bounds__(kThreads) void tlc_stochastic_trits_kernel(
    const float* __restrict__ x, uint64_t n, float s, uint64_t seed, uint64_t step,
    const uint32_t* __restrict__ partials, uint32_t np, uint8_t* __restrict__ trits,
    Ctrl* __restrict__ ctrl) {
  __shared__ uint32_t lds[kWaves];
  const Scale sc = finish_scale(partials, np, s, lds);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctrl->enc.err = sc.bad;
    ctrl->enc.scale = sc.M;
  }
  if (sc.bad) return;
  const uint64_t nv = n >> 2;
  const uint64_t tid = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * kThreads;
  for (uint64_t i = tid; i < nv; i += stride) {
    const float4 a = ld_stream(x + 4 * i);
    const Philox4 w = element_words(i, step, seed);
    trits[i] = (uint8_t)(stochastic_trit(a.x, sc.M, w.v[0]) |
                         (stochastic_trit(a.y, sc.M, w.v[1]) << 2) |
                         (stochastic_trit(a.z, sc.M, w.v[2]) << 4) |
                         (stochastic_trit(a.w, sc.M, w.v[3]) << 6));
  }
  if (tid == 0 && (n & 3u)) {
    const Philox4 w = element_words(nv, step, seed);
    uint32_t tb = 0u;
#pragma unroll
    for (uint32_t c = 0; c < 3u; ++c)
      if (c < (n & 3u)) tb |= stochastic_trit(x[4 * nv + c], sc.M, w.v[c]) << (2u * c);
    trits[nv] = (uint8_t)tb;
  }
}

// Sixteen bytes at any address.
typedef uint32_t tlc_u4x1 __attribute__((ext_vector_type(4), aligned(1)));

// The quartic bytes of all values from their trits, one tile per block.
__global__ __launch_bounds__(kThreads) void tlc_quant_pack_kernel(
    uint64_t n, uint32_t m, const uint8_t* __restrict__ trits, uint8_t* __restrict__ out,
    Ctrl* __restrict__ ctrl, HostMirror hm) {
  __shared__ uint32_t s_lut[5][256];
  __shared__ __align__(16) uint8_t s_q[kEncTile];
  const uint32_t bad = ctrl->enc.err;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctrl->enc.len = bad ? 0u : m;
    host_put_all(hm.res, bad, bad ? 0u : m, ctrl->enc.scale);
  }
  if (bad) return;
  const uint64_t q0 = (uint64_t)blockIdx.x * kEncTile;
  const uint32_t tile_bytes = (uint32_t)umin64(kEncTile, (uint64_t)m - q0);
  if (tile_bytes == (uint32_t)kEncTile && 4ull * m + q0 + kEncTile <= n) {
    uint32_t d[1][5];
    load_trit_words<1>(trits, m, q0, d);
    init_trit_luts(s_lut);
    __syncthreads();
    const uint4 w = pack_trit_words(d[0], s_lut);
    tlc_u4x1 o;
    o.x = w.x;
    o.y = w.y;
    o.z = w.z;
    o.w = w.w;
    *reinterpret_cast<tlc_u4x1*>(out + q0 + 16u * threadIdx.x) = o;
  } else {
    uint32_t h[kGroupsPerThread][5];
    load_trits(trits, n, m, q0, tile_bytes, h);
    init_trit_luts(s_lut);
    __syncthreads();
    pack_trits(h, n, m, q0, tile_bytes, s_lut, s_q);
    for (uint32_t i = threadIdx.x; i < tile_bytes; i += kThreads) out[q0 + i] = s_q[i];
  }
}

// The same after the in-place max pass; the residuals that the tile's list holds
// are stored once its reads are through.  (40M values, a call, with a pass over
// lines and trits in between | this one: 132 | 119 us at s = 1.75, 153 | 143 at
// s = 1.)
template <bool kGrid>
__global__ __launch_bounds__(kThreads) void tlc_quant_pack_bounds_kernel(
    float* __restrict__ r, uint64_t n, uint32_t m, float s, const uint32_t* __restrict__ partials,
    uint32_t np, const uint16_t* __restrict__ bound, uint8_t* __restrict__ out,
    Ctrl* __restrict__ ctrl, HostMirror hm) {
  __shared__ BoundShared sh;
  const uint64_t q0 = (uint64_t)blockIdx.x * kEncTile;
  const uint32_t tile_bytes = (uint32_t)umin64(kEncTile, (uint64_t)m - q0);
  if (!bounded_tile<kGrid>(r, n, m, q0, tile_bytes, s, partials, np, bound, sh,
                           [&](const Scale& sc) {
                             if (blockIdx.x == 0 && threadIdx.x == 0) {
                               const uint32_t len = sc.bad ? 0u : m;
                               ctrl->enc.err = sc.bad;
                               ctrl->enc.scale = sc.M;
                               ctrl->enc.len = len;
                               host_put_all(hm.res, sc.bad, len, sc.M);
                             }
                           }))
    return;
  if (threadIdx.x < umin32(sh.left, kFixCap)) {
    const uint2 f = sh.fix[threadIdx.x];
    r[(uint64_t)(f.x / (uint32_t)kEncTile) * m + q0 + f.x % (uint32_t)kEncTile] =
        __uint_as_float(f.y);
  }
  if (tile_bytes == (uint32_t)kEncTile)
    *reinterpret_cast<tlc_u4x1*>(out + q0 + 16u * threadIdx.x) =
        *reinterpret_cast<const tlc_u4x1*>(sh.enc.q + 16u * threadIdx.x);
  else
    for (uint32_t i = threadIdx.x; i < tile_bytes; i += kThreads) out[q0 + i] = sh.enc.q[i];
}

// ---------------------------------------------------------------- launchers
namespace {
uint32_t absmax_blocks(uint64_t n) {
  const uint64_t blocks = ((n >> 2) + kThreads * 4 - 1) / (kThreads * 4);
  return (uint32_t)(blocks < 1 ? 1 : (blocks > kAbsmaxMaxBlocks ? kAbsmaxMaxBlocks : blocks));
}
}  // namespace

// Tensors whose values and buffer fit the last-level cache are read with
// plain loads by the check pass: the writing pass then finds them there (check
// + writing pass, three tensors in turn, nontemporal against plain loads: 12M
// values 16.8 + 27.8 against 18.4 + 22.9 us, 25.6M 32.8 + 53.8 against 35.6 +
// 46.1, 33M 40.5 + 69.0 against 47.3 + 59.9; 45M, which do not fit, 54.4 + 91.9
// against 62.6 + 83.1, and 2^28 lose 40 us).
#ifdef TLC_DELAY_INJECT
// Stress build only: blocks per launch of a small tensor's encode (0: all).
static uint32_t g_stress_blocks = 0u;
extern "C" __attribute__((visibility("default"))) void tlc_stress_blocks(uint32_t blocks) {
  g_stress_blocks = blocks;
}
#endif

hipError_t launch_absmax_check(const float* x, const float* r, uint64_t n, uint32_t* partials,
                               uint32_t* nblocks, hipStream_t st) {
  *nblocks = absmax_blocks(n);
  if (n * 2 * sizeof(float) <= kCacheBytes)
    launch_k(tlc_absmax_check_kernel<true>, *nblocks, kThreads, st, x, r, n, partials);
  else
    launch_k(tlc_absmax_check_kernel<false>, *nblocks, kThreads, st, x, r, n, partials);
  return hipGetLastError();
}

hipError_t launch_accum_absmax(const float* x, float* r, uint64_t n, uint32_t* partials,
                               uint32_t* nblocks, uint16_t* bound, hipStream_t st) {
  *nblocks = absmax_blocks(n);
  if (r)
    launch_k(tlc_accum_absmax_kernel<true>, *nblocks, kThreads, st, x, r, n, partials, bound);
  else
    launch_k(tlc_accum_absmax_kernel<false>, *nblocks, kThreads, st, x, r, n, partials, bound);
  return hipGetLastError();
}

hipError_t launch_accum_quantize(const float* x, float* r, uint64_t n, float s,
                                 bool in_place, const uint32_t* partials, uint32_t np,
                                 uint8_t* trits, Ctrl* ctrl, HostMirror hm, hipStream_t st) {
  launch_k(tlc_accum_quantize_kernel, absmax_blocks(n), kThreads, st, x, r, n, trits, partials,
           np, s, in_place, ctrl, hm);
  return hipGetLastError();
}

hipError_t launch_quant_encode(uint64_t n, uint32_t m, uint8_t* slots, TileRec* recs,
                               const uint8_t* trits, const Ctrl* ctrl, hipStream_t st) {
  const uint32_t ntiles = (uint32_t)((m + kEncTile - 1) / kEncTile);
  if (ntiles >= kTritTwoWaveMinTiles)
    launch_k(tlc_quant_encode_kernel<kTritThreads>, ntiles, kTritThreads, st, n, m, slots, recs,
             trits, ctrl);
  else
    launch_k(tlc_quant_encode_kernel<kThreads>, ntiles, kThreads, st, n, m, slots, recs, trits,
             ctrl);
  return hipGetLastError();
}

hipError_t launch_quant_encode_bounds(float* r, uint64_t n, uint32_t m, float s,
                                      const uint32_t* partials, uint32_t np,
                                      const uint16_t* bound, uint8_t* slots, TileRec* recs,
                                      uint2* fix, Ctrl* ctrl, HostMirror hm, hipStream_t st) {
  const uint32_t tiles = (m + kEncTile - 1) / kEncTile;
  if (m % 4 == 0)
    launch_k(tlc_quant_encode_bounds_kernel<true>, tiles, kThreads, st, r, n, m, s, partials, np,
             bound, slots, recs, fix, ctrl, hm);
  else
    launch_k(tlc_quant_encode_bounds_kernel<false>, tiles, kThreads, st, r, n, m, s, partials, np,
             bound, slots, recs, fix, ctrl, hm);
  return hipGetLastError();
}

hipError_t launch_quant_encode_chained(const float* x, float* r, uint64_t n, uint32_t m, float s,
                                       bool in_place, const uint32_t* partials, uint32_t np,
                                       uint8_t* out, uint64_t* status, uint64_t* maxima,
                                       uint32_t ticket_base, uint32_t epoch, Ctrl* ctrl,
                                       HostMirror hm, hipStream_t st) {
  const uint32_t tiles = small_tiles(m);
  const bool chained = tiles > kExchangeTiles;
  const uint32_t blocks = chained ? (tiles + 1u) / 2u : tiles;
  // one launch; the stress build can launch fewer blocks at a time, each
  // launch ending before the next one starts, as if no more were resident
  uint32_t each = blocks;
#ifdef TLC_DELAY_INJECT
  if (g_stress_blocks) each = std::min(blocks, g_stress_blocks);
#endif
  for (uint32_t b = 0; b < blocks; b += each) {
    const uint32_t grid = std::min(each, blocks - b);
    if (chained)
      launch_k(tlc_quant_encode_chained_kernel<2 * kTileThreads>, grid, 2 * kTileThreads, st, x, r,
               n, m, s, in_place, partials, np, out, status, maxima, ticket_base, epoch, ctrl, hm);
    else
      launch_k(tlc_quant_encode_chained_kernel<kTileThreads>, grid, kTileThreads, st, x, r, n, m, s,
               in_place, partials, np, out, status, maxima, ticket_base, epoch, ctrl, hm);
  }
  return hipGetLastError();
}

hipError_t launch_zre_chunks(const TileRec* recs, uint32_t ntiles, uint64_t* local_pre,
                             uint64_t* chunk_agg, Ctrl* ctrl, hipStream_t st) {
  const uint32_t nchunks = (ntiles + kChunkTiles - 1) / kChunkTiles;
  launch_k(tlc_zre_chunk_kernel, (nchunks + kWaves - 1) / kWaves, kThreads, st,
      recs, ntiles, local_pre, chunk_agg, ctrl);
  return hipGetLastError();
}

hipError_t launch_zre_compact(const TileRec* recs, const uint64_t* chunk_pre,
                              const uint64_t* local_pre, const uint8_t* slots, uint32_t m,
                              uint8_t* out, Ctrl* ctrl, HostMirror hm, const uint2* fix, float* r,
                              uint64_t n, hipStream_t st) {
  const uint32_t ntiles = (uint32_t)((m + kEncTile - 1) / kEncTile);
  const uint32_t blocks = (ntiles + kWaves - 1) / kWaves;
#define TLC_LAUNCH(P)                                                                            \
  launch_k(tlc_zre_compact_kernel<P>, blocks, kThreads, st, recs, chunk_pre, local_pre, slots, m, \
           ntiles, out, ctrl, hm, fix, r, n)
  if (zre_chunked(m))
    TLC_LAUNCH(0u);
  else
    TLC_LAUNCH(kOwnPrefixTiles / kThreads);
#undef TLC_LAUNCH
  return hipGetLastError();
}

hipError_t launch_encode_many(const EncDesc* descs, const ManyPlan& p, bool in_place,
                              uint32_t* partials, uint16_t* bound, uint8_t* trits, uint8_t* slots,
                              TileRec* recs, uint2* fix, EncResult* results, HostMirror hm, int pass,
                              hipStream_t st) {
  constexpr uint32_t kBlocks = kAbsmaxMaxBlocks;  // one per CU, as for a tensor alone
  if (pass == 0) {
    if (p.bounds)
      launch_k(tlc_accum_absmax_batch_kernel, kBlocks, kThreads, st, descs, p.count, p.units,
               p.groups, partials, bound);
    else if (p.values * 2 * sizeof(float) <= kCacheBytes)
      launch_k(tlc_absmax_check_batch_kernel<true>, kBlocks, kThreads, st, descs, p.count, p.units,
               p.groups, partials);
    else
      launch_k(tlc_absmax_check_batch_kernel<false>, kBlocks, kThreads, st, descs, p.count,
               p.units, p.groups, partials);
  } else if (pass == 1) {  // not with bounds: the tiles quantize
    launch_k(tlc_quantize_many_kernel, kBlocks, kThreads, st, descs, p.count, p.units, p.groups,
             partials, in_place, trits, results, hm);
  } else if (pass == 2) {
    if (p.bounds)
      launch_k(tlc_quant_encode_bounds_many_kernel, p.tiles, kThreads, st, descs, p.count,
               partials, bound, slots, recs, fix, results, hm);
    else
      launch_k(tlc_quant_encode_many_kernel, p.tiles, kThreads, st, descs, p.count, slots, recs,
               trits, results);
  } else if (p.most_tiles <= kOwnPrefixTiles) {
    launch_k(tlc_zre_compact_many_kernel<kOwnPrefixTiles / kThreads>, p.compact_blocks, kThreads,
             st, descs, p.count, recs, slots, results, hm, p.bounds ? fix : nullptr);
  } else {
    launch_k(tlc_zre_compact_many_kernel<kManyMaxTiles / kThreads>, p.compact_blocks, kThreads, st,
             descs, p.count, recs, slots, results, hm, p.bounds ? fix : nullptr);
  }
  return hipGetLastError();
}

hipError_t launch_quant_encode_batch(const EncDesc* descs, uint32_t shared, const uint16_t* owner,
                                     uint32_t tiles, bool in_place, EncResult* results,
                                     uint64_t* status, uint64_t* maxima, uint32_t ticket_base,
                                     uint32_t epoch, Ctrl* ctrl, HostMirror hm, hipStream_t st) {
  launch_k(tlc_quant_encode_batch_kernel, tiles, kTileThreads, st, descs, shared, owner, in_place,
           results, status, maxima, ticket_base, epoch, ctrl, hm);
  return hipGetLastError();
}

// Blocks of the stochastic pass: eight per CU, all resident.
constexpr uint32_t kStochMaxBlocks = 2048;

hipError_t launch_stochastic_trits(const float* x, uint64_t n, float s, uint64_t seed,
                                   uint64_t step, const uint32_t* partials, uint32_t np,
                                   uint8_t* trits, Ctrl* ctrl, hipStream_t st) {
  const uint64_t want = std::max<uint64_t>(1, ((n >> 2) + kThreads - 1) / kThreads);
  launch_k(tlc_stochastic_trits_kernel, (uint32_t)std::min<uint64_t>(want, kStochMaxBlocks),
           kThreads, st, x, n, s, seed, step, partials, np, trits, ctrl);
  return hipGetLastError();
}

hipError_t launch_quant_pack(uint64_t n, uint32_t m, const uint8_t* trits, uint8_t* out,
                             Ctrl* ctrl, HostMirror hm, hipStream_t st) {
  const uint32_t blocks = (uint32_t)((m + kEncTile - 1) / kEncTile);
  launch_k(tlc_quant_pack_kernel, blocks, kThreads, st, n, m, trits, out, ctrl, hm);
  return hipGetLastError();
}

hipError_t launch_quant_pack_bounds(float* r, uint64_t n, uint32_t m, float s,
                                    const uint32_t* partials, uint32_t np, const uint16_t* bound,
                                    uint8_t* out, Ctrl* ctrl, HostMirror hm, hipStream_t st) {
  const uint32_t blocks = (m + kEncTile - 1) / kEncTile;
  if (m % 4 == 0)
    launch_k(tlc_quant_pack_bounds_kernel<true>, blocks, kThreads, st, r, n, m, s, partials, np,
             bound, out, ctrl, hm);
  else
    launch_k(tlc_quant_pack_bounds_kernel<false>, blocks, kThreads, st, r, n, m, s, partials, np,
             bound, out, ctrl, hm);
  return hipGetLastError();
}

}  // namespace tlc
