// tlc_internal.h -- definitions shared by the kernels and the host side of
// the library (not part of the public ABI).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "tlc.h"

namespace tlc {

constexpr int kThreads = 256;             // every kernel: 4 wave64 per block
constexpr int kZreBytesPerThread = 64;    // zero-run index scan: four uint4 per thread
constexpr int kZreTile = kThreads * kZreBytesPerThread;  // 16384 stream bytes per tile
// the batched scans, over many streams that mostly fit one tile, and the
// index role of the single-launch decode take half as many bytes per
// thread (shorter per-thread loops on short streams; the fused decode
// kernel then stays within the expanding blocks' 64 registers)
constexpr int kZreBatchBytesPerThread = 32;
constexpr int kZreBatchTile = kThreads * kZreBatchBytesPerThread;  // 8192
constexpr int kEncTile = 4096;            // quartic bytes per encoder tile
constexpr int kDecRange = 4096;           // quartic bytes per expand/dequantize block
// Encoder tiles of small tensors and batches: 256 threads of eight quartic
// bytes.  The tiles of a tensor of at most kExchangeTiles (1,310,720 values)
// exchange their maxima and summaries among themselves.
constexpr int kTileThreads = kThreads;
constexpr int kTileGroups = 2;
constexpr uint32_t kSmallTile = kTileThreads * kTileGroups * 4;  // 2048 quartic bytes
constexpr uint32_t kExchangeTiles = 128;
inline uint32_t small_tiles(uint32_t m) { return (m + kSmallTile - 1) / kSmallTile; }
// Tensors of at least this many encoder tiles take the three-pass encoder
// (no waits between tiles); smaller ones, whose tiles can exchange what they
// need (kExchangeTiles of half the size), a single launch.
constexpr uint32_t kThreePassMinTiles = kExchangeTiles / 2 + 1;
constexpr uint64_t kCacheBytes = 256ull << 20;  // the last-level cache
constexpr uint32_t kCus = 256;
constexpr uint32_t kAbsmaxMaxBlocks = 256;  // partial maxima per encode (one block per CU)
// Up to this many tiles the compaction finds its prefixes without the chunk
// pass, two summaries per thread (9M values, 440 tiles, a call with the chunk
// pass | without: 56.0 | 52.1 us).  With eight summaries, as a batch's middle
// tensors have them, 11M values (538 tiles) would take 59.0 instead of 62.5 us,
// 25.6M 106.3 instead of 108.8 and 41M 162.0 instead of 162.7.
constexpr uint32_t kOwnPrefixTiles = 512;
inline bool zre_chunked(uint32_t m) {
  return (m + (uint32_t)kEncTile - 1) / kEncTile > kOwnPrefixTiles;
}

// Per-tensor encode result (device), written by the encoder's tiles.
struct EncResult {
  uint32_t err;    // 1: NaN/Inf in tensor + residual, or max*s overflow
  uint32_t len;    // zero-run stream length
  float scale;     // M
  uint32_t reserved;
};

// Device control block (one per context, in the workspace).  The first 32
// bytes are copied to pinned host memory by tlc_sync and after the encodes
// whose kernels do not write their result there themselves (HostMirror).
struct Ctrl {
  EncResult enc;           // single-tensor encode result
  uint32_t fault;          // sticky: a look-back wait timed out
  uint32_t dec_corrupt;    // sticky: a decoded stream had the wrong length
  uint32_t dec_bad_epoch;  // epoch of the last decode launch with a bad stream
  uint32_t enc_ticket;     // tile tickets of the encoder
  uint32_t dec_ticket;     // tile tickets of the zero-run index scan
  uint32_t dec_verdict;    // epoch << 1 | bad of the last single-stream decode's stream
  uint32_t chunk_done;     // blocks of the tile-chunk pass done (0 between calls)
  uint32_t pad[53];
};
static_assert(sizeof(Ctrl) == 256, "Ctrl is one 256-byte slot");

struct HostReadback {
  EncResult enc;
  uint32_t fault;
  uint32_t dec_corrupt;
  uint32_t pad[2];
};

// Device pointers into the pinned host readback that the encoders (and the
// decoders, for the fault and bad-stream flags) also write a call's result to,
// so that the host needs no copy before it reads it; null: not mirrored.
// res: the result (one per tensor of a batch); fault: the look-back fault
// flag; corrupt: the decoder's sticky bad-stream flag.
struct HostMirror {
  EncResult* res = nullptr;
  uint32_t* fault = nullptr;
  uint32_t* corrupt = nullptr;
};

// A batch's tensors of more than kExchangeTiles small tiles and at most
// kManyMaxTiles of kEncTile (41,943,040 values) go through the three passes
// together: their trits and bounds start at multiples of kManyValues values of
// the workspace, with as many to spare after each (trit words are read past
// the end).  Larger ones go one after the other: their passes fill the chip.
// (One after the other, four of 12M values took 225 us, together 196.)
// Tensors of kManyMinTiles to kExchangeTiles small tiles join them where they
// don't fit the last-level cache together: the one launch holds a tile's
// values in registers while it waits, which costs more than the check pass's
// second read once the chip is full (64 tensors of 1M values: 265 us; before
// the exchange, in place, 235).
constexpr uint32_t kManyMaxTiles = 2048;
constexpr uint32_t kManyMinTiles = 32;
constexpr uint32_t kManyValues = 1024;
// Groups of blocks over them: as many as tensors, rounded down to a power of
// two, and at most this (130 tensors of 1M values: 16 groups 483 us, 32 474, 64
// 491, 256 554).
constexpr uint32_t kManyMaxGroups = 32;

// One tensor of a batched encode.
struct EncDesc {
  const float* x;
  float* r;
  uint8_t* out;
  uint64_t n;
  uint32_t m;
  float s;
  uint32_t tile0;  // first encoder tile (global tile numbering of the launch)
  // the three passes only:
  uint32_t blk0;   // first partial maximum of the max pass
  uint32_t nblk;   // how many
  uint32_t v0;     // first trit, in kManyValues
  uint32_t cblk0;  // first block of the compaction
  uint32_t pad;
};
static_assert(sizeof(EncDesc) == 64, "EncDesc is 64 bytes");

// Per-tile record of the single-tensor encoder's first pass: the zero-run
// summary of the whole tile (RunSum bits), the length of its leading run of
// 121 bytes and how many bytes it wrote into its slot (its encoding from the
// first non-121 byte on), and how many residuals it left to the compaction
// (kFixCap at most; from bounds only).
struct TileRec {
  uint64_t agg;
  uint16_t lead;  // <= kEncTile
  uint16_t len;   // <= kEncTile
  uint32_t left;
};
static_assert(sizeof(TileRec) == 16, "TileRec is 16 bytes");
// A tile's list of residuals for the compaction: (k * kEncTile + position in
// the tile, value bits) each.  Further ones are stored at once.
constexpr uint32_t kFixCap = 256;

// One stream of a batched decode or of a decode-sum.
struct DecDesc {
  const uint8_t* C;
  float* out;      // batched decode: this stream's output (decode-sum: unused)
  uint64_t n;
  uint32_t c;
  uint32_t m;
  float scale;
  uint32_t tile0;   // first index-scan tile (global numbering of the launch)
  uint32_t range0;  // first start-index entry / expand block of this stream
  uint32_t pad[5];
};
static_assert(sizeof(DecDesc) == 64, "DecDesc is 64 bytes");

// Kernel launches of the library.  While tlc_profile_* times a launcher
// (timed_launch), g_launch_events holds its event pair: the first kernel
// the launcher dispatches takes the start event and every kernel the stop
// event (the last one's stands), recorded by the dispatches themselves
// (hipExtLaunchKernelGGL), so timing adds no marker packets between
// kernels.  Untimed launches are plain launches.
struct LaunchEvents {
  hipEvent_t start = nullptr;
  hipEvent_t stop = nullptr;
};
extern thread_local LaunchEvents g_launch_events;

template <class... Formals, class... Args>
inline void launch_k(void (*kernel)(Formals...), dim3 grid, dim3 block, hipStream_t st,
                     Args... args) {
  LaunchEvents& ev = g_launch_events;
  if (ev.start || ev.stop) {
    hipEvent_t a = ev.start;
    ev.start = nullptr;
    hipExtLaunchKernelGGL(kernel, grid, block, 0, st, a, ev.stop, 0, args...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
  }
}

// Launchers (encode.hip, decode.hip, int8.hip).  All return the hipError_t of the
// launch.
// The check pass: partial maxima of |x + r|, nothing written.
hipError_t launch_absmax_check(const float* x, const float* r, uint64_t n, uint32_t* partials,
                               uint32_t* nblocks, hipStream_t st);
// In place: step 1 into the buffer (r NULL: max |x| alone) and the partial
// maxima; bound (with r): per four values of r, the top half of the largest
// |acc|.
hipError_t launch_accum_absmax(const float* x, float* r, uint64_t n, uint32_t* partials,
                               uint32_t* nblocks, uint16_t* bound, hipStream_t st);
// Eq. 2 for a large tensor after the check pass (its partials): final residuals
// in r and 2-bit trits, one byte per four values (in_place: a refused tensor is
// left with the sums).
hipError_t launch_accum_quantize(const float* x, float* r, uint64_t n, float s, bool in_place,
                                 const uint32_t* partials, uint32_t np, uint8_t* trits,
                                 Ctrl* ctrl, HostMirror hm, hipStream_t st);
// The tiles' own encodings from the trits.
hipError_t launch_quant_encode(uint64_t n, uint32_t m, uint8_t* slots, TileRec* recs,
                               const uint8_t* trits, const Ctrl* ctrl, hipStream_t st);
// The same after the in-place max pass, from its bounds, with Eq. 2: residuals of
// q != 0 go to the tiles' lists, fix.  A bound past the last float4's may be read.
hipError_t launch_quant_encode_bounds(float* r, uint64_t n, uint32_t m, float s,
                                      const uint32_t* partials, uint32_t np,
                                      const uint16_t* bound, uint8_t* slots, TileRec* recs,
                                      uint2* fix, Ctrl* ctrl, HostMirror hm, hipStream_t st);
// A small tensor in one launch (after the check pass, its partials, when it
// has more than kExchangeTiles tiles).  in_place: a refused tensor is left
// with the sums.  status, maxima: a word per tile each.
hipError_t launch_quant_encode_chained(const float* x, float* r, uint64_t n, uint32_t m, float s,
                                       bool in_place, const uint32_t* partials, uint32_t np,
                                       uint8_t* out, uint64_t* status, uint64_t* maxima,
                                       uint32_t ticket_base, uint32_t epoch, Ctrl* ctrl,
                                       HostMirror hm, hipStream_t st);
hipError_t launch_zre_chunks(const TileRec* recs, uint32_t ntiles, uint64_t* local_pre,
                             uint64_t* chunk_agg, Ctrl* ctrl, hipStream_t st);
hipError_t launch_zre_compact(const TileRec* recs, const uint64_t* chunk_pre,
                              const uint64_t* local_pre, const uint8_t* slots, uint32_t m,
                              uint8_t* out, Ctrl* ctrl, HostMirror hm, const uint2* fix, float* r,
                              uint64_t n, hipStream_t st);
// Comparison modes: stochastic trits of x, and the quartic bytes of any trits.
hipError_t launch_stochastic_trits(const float* x, uint64_t n, float s, uint64_t seed,
                                   uint64_t step, const uint32_t* partials, uint32_t np,
                                   uint8_t* trits, Ctrl* ctrl, hipStream_t st);
hipError_t launch_quant_pack(uint64_t n, uint32_t m, const uint8_t* trits, uint8_t* out,
                             Ctrl* ctrl, HostMirror hm, hipStream_t st);
// The quartic bytes after the in-place max pass, with Eq. 2.
hipError_t launch_quant_pack_bounds(float* r, uint64_t n, uint32_t m, float s,
                                    const uint32_t* partials, uint32_t np, const uint16_t* bound,
                                    uint8_t* out, Ctrl* ctrl, HostMirror hm, hipStream_t st);
// x + r after the check pass (its partials), or x alone (r NULL).
hipError_t launch_int8_quant(const float* x, float* r, uint64_t n, float s, bool in_place,
                             const uint32_t* partials, uint32_t npartials, uint8_t* out,
                             Ctrl* ctrl, HostMirror hm, hipStream_t st);
hipError_t launch_int8_dequant(const uint8_t* C, uint64_t n, float M, float* out,
                               int accumulate, hipStream_t st);
// Pass 0 (max), 1 (quantize; not with bounds), 2 (tiles) or 3 (compaction) of a
// batch's middle tensors; descs in device memory, results by descriptor.
struct ManyPlan {
  uint32_t count, tiles, compact_blocks, most_tiles;
  uint32_t units, groups;  // kManyValues each; equal shares of them (a power of two)
  uint64_t values;
  bool bounds;  // the in-place max pass and tiles from its bounds
};
hipError_t launch_encode_many(const EncDesc* descs, const ManyPlan& p, bool in_place,
                              uint32_t* partials, uint16_t* bound, uint8_t* trits, uint8_t* slots,
                              TileRec* recs, uint2* fix, EncResult* results, HostMirror hm,
                              int pass,
                              hipStream_t st);
// owner: the tensor of each of the `tiles` tiles; the first `shared` are those
// of tensors of more than one.
hipError_t launch_quant_encode_batch(const EncDesc* descs, uint32_t shared, const uint16_t* owner,
                                     uint32_t tiles, bool in_place, EncResult* results,
                                     uint64_t* status, uint64_t* maxima, uint32_t ticket_base,
                                     uint32_t epoch, Ctrl* ctrl, HostMirror hm, hipStream_t st);
// One stream's decode.  Small decodes (at most kFusedMaxBlocks blocks in
// all, so every block is resident at once) run in one launch: the first
// blocks scan the stream (kZreBatchTile bytes each), the others expand.
// Larger ones run the scan (kZreTile bytes per block), then the expansion:
// thousands of expanding blocks waiting inside one launch for a scan of
// hundreds of tiles slowed it down more than the launch boundary costs.
constexpr uint32_t kFusedMaxBlocks = 256;
inline uint32_t decode_ranges(uint64_t m) { return (uint32_t)((m + kDecRange - 1) / kDecRange); }
inline bool decode_fused(uint64_t c, uint64_t m) {
  return (c + kZreBatchTile - 1) / kZreBatchTile + decode_ranges(m) <= kFusedMaxBlocks;
}
// The scan's tiles; the tickets a decode takes (the host advances the
// decoder's ticket base by decode_tickets(c, m)).
inline uint32_t decode_index_tiles(uint64_t c, uint64_t m) {
  const uint64_t tile = decode_fused(c, m) ? kZreBatchTile : kZreTile;
  return (uint32_t)((c + tile - 1) / tile);
}
inline uint32_t decode_tickets(uint64_t c, uint64_t m) {
  return decode_index_tiles(c, m) + (decode_fused(c, m) ? decode_ranges(m) : 0u);
}
// The scan of one stream (not decode_fused), then its expansion; or, when
// decode_fused, both in the expansion's launch (ticket_base then counts
// the scan's tiles too).
hipError_t launch_zre_index(const uint8_t* C, uint32_t c, uint32_t m, uint64_t* start,
                            uint64_t* status, uint32_t ntiles, uint32_t ticket_base,
                            uint32_t epoch, Ctrl* ctrl, HostMirror hm, hipStream_t st);
hipError_t launch_expand_dequant(const uint8_t* C, uint32_t c, uint64_t* start,
                                 uint64_t* status, uint32_t ticket_base, uint64_t n, uint64_t m,
                                 float scale, float* out, int accumulate, uint32_t epoch,
                                 Ctrl* ctrl, HostMirror hm, hipStream_t st);
// owner: the stream of each scan tile (not read when every stream has one),
// of each range, in host memory as the descriptors; null: few streams, their
// descriptors in device memory.  wide: tiles of kZreTile stream bytes where the
// streams average more than four of the smaller tiles and are long enough
// together that fewer, longer tiles don't leave the chip idle (16 streams of 366
// KB: 10.1 against 15.0 us; a call of 12 streams, 619 KB together 45.0 us with
// the smaller tiles and 45.1 with these, 1.2 MB 46.1 and 46.0, 2.9 MB 53.4 and
// 50.7; two of 52 KB 20.3 and 20.6), else of kZreBatchTile.
inline bool batch_scan_wide(uint64_t stream_bytes, uint64_t count) {
  return stream_bytes > 4u * std::max<uint64_t>(count, 32u) * kZreBatchTile;
}
hipError_t launch_zre_index_batch(const DecDesc* descs, uint32_t count, const uint16_t* owner,
                                  uint32_t tiles, bool wide, uint64_t* start, uint64_t* status,
                                  uint32_t ticket_base, uint32_t epoch, Ctrl* ctrl, HostMirror hm,
                                  hipStream_t st);
hipError_t launch_expand_dequant_batch(const DecDesc* descs, uint32_t count, const uint16_t* owner,
                                       uint32_t total_ranges, const uint64_t* start,
                                       int accumulate, uint32_t epoch, const Ctrl* ctrl,
                                       hipStream_t st);
hipError_t launch_expand_sum(const DecDesc* descs, uint32_t count, const uint64_t* start,
                             uint64_t n, uint64_t m, float* out, int accumulate, uint32_t epoch,
                             const Ctrl* ctrl, hipStream_t st);

// Epoch widths of the two look-back status layouts.
constexpr uint32_t kEncEpochMax = (1u << 23) - 1u;
constexpr uint32_t kDecEpochMax = (1u << 26) - 1u;
static_assert(kEncEpochMax == TLC_ENC_EPOCH_MAX && kDecEpochMax == TLC_DEC_EPOCH_MAX,
              "the header states the epoch maxima");

// Sets the calling thread's error text (tlc_last_error_string) and returns
// code.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

}  // namespace tlc
