// The signature/probe scan kernel and the tile spaces it walks (one image, or
// a batch of images), Section 3.1: the djb2 signature of each 512-byte sector
// (Eq. (1), 64-bit) and its lookup among the master signatures of the
// sector's cluster position. Device code only; included by carve.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "carve_device.h"

namespace carve {

constexpr int kScanThreads = 256;
constexpr int kScanWaves = kScanThreads / (int)kWave;
// kFlags: hit words and the matched slot of each flagged sector (for
// confirmation); kFlagBits: hit words only; kSigs: the signatures themselves.
enum { kFlags = 0, kSigs = 1, kFlagBits = 2 };

// ------------------------------------------------------------ images
// One image of a scan. tile_begin: its first tile in the scan's tile space.
struct ImageDesc {
  const uint8_t* base;
  uint64_t n_sectors;
  uint64_t tile_begin;
  uint32_t tau0;      // cluster position of the image's first sector
  uint32_t any_tau;   // 1: match at any cluster position
};

// Where a tile's sectors are.
struct TileRef {
  const uint8_t* base;   // its first sector
  uint32_t n_valid;      // 1..64 sectors
  uint32_t tau_first;    // cluster position of its first sector
  uint32_t any_tau;
  uint32_t image;
};

__device__ __forceinline__ TileRef tile_of(const ImageDesc& d, uint64_t g, uint32_t image) {
  const uint64_t first = (g - d.tile_begin) * kTileSectors;
  const uint64_t rem = d.n_sectors - first;
  return TileRef{d.base + first * kSectorBytes, rem >= kTileSectors ? kTileSectors : (uint32_t)rem,
                 (uint32_t)((first + d.tau0) & (kClusterSectors - 1)), d.any_tau, image};
}

// A scan of one image: the descriptor travels by value. Units are sectors:
// unit j is bytes [512j, 512j + 512) of its image.
struct OneImage {
  static constexpr uint32_t kUnitBytes = kSectorBytes, kUnitStride = kSectorBytes;
  static constexpr bool kAnyPosition = false;   // the image's own rule applies
  static constexpr bool kManyImages = false;
  ImageDesc d;
  __device__ __forceinline__ uint64_t n_tiles() const { return (d.n_sectors + kTileSectors - 1) / kTileSectors; }
  __device__ __forceinline__ TileRef tile_at(uint64_t g) const { return tile_of(d, g, 0); }
  // `cursor` is the image of the previous lookup (tiles are visited in increasing order)
  __device__ __forceinline__ TileRef tile(uint64_t g, uint32_t&) const { return tile_of(d, g, 0); }
  __device__ __forceinline__ const ImageDesc& image(uint32_t) const { return d; }
  __device__ __forceinline__ uint32_t image_between(uint64_t, uint32_t, uint32_t) const { return 0; }
};

// A batch: descriptors in device memory, n + 1 of them (the last one only
// carries the total tile count in tile_begin).
struct ManyImages {
  static constexpr uint32_t kUnitBytes = kSectorBytes, kUnitStride = kSectorBytes;
  static constexpr bool kAnyPosition = false, kManyImages = true;
  const ImageDesc* __restrict__ d;
  uint32_t n;
  __device__ __forceinline__ uint64_t n_tiles() const { return d[n].tile_begin; }
  __device__ __forceinline__ TileRef tile_at(uint64_t g) const {
    const uint32_t i = image_of_tile(g);
    return tile_of(d[i], g, i);
  }
  __device__ __forceinline__ TileRef tile(uint64_t g, uint32_t& cursor) const {
    // The image holding tile g is the last i with d[i].tile_begin <= g
    // (empty images are skipped). A wave's tiles are a stride of the grid
    // apart, which can pass several small images: the next 8 starts are
    // read at once (independent loads, one wait), not one after another.
    while (true) {
      uint32_t step = 0;
#pragma unroll
      for (uint32_t k = 1; k <= 8; ++k) {
        const uint32_t i = cursor + k < n ? cursor + k : n;   // d[n] (the total) ends every walk
        step += g >= d[i].tile_begin ? 1u : 0u;
      }
      cursor += step;
      if (step < 8) break;
    }
    return tile_of(d[cursor], g, cursor);
  }
  __device__ __forceinline__ const ImageDesc& image(uint32_t i) const { return d[i]; }
  // The last image i of [lo, hi] with d[i].tile_begin <= g (tile g is in one of them).
  __device__ __forceinline__ uint32_t image_between(uint64_t g, uint32_t lo, uint32_t hi) const {
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (d[mid].tile_begin <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
  }
  __device__ __forceinline__ uint32_t image_of_tile(uint64_t g) const { return image_between(g, 0, n - 1); }
  // The first i of [0, n] with d[i].tile_begin >= g.
  __device__ __forceinline__ uint32_t first_from(uint64_t g) const {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (d[mid].tile_begin >= g) hi = mid; else lo = mid + 1;
    }
    return lo;
  }
};

// ------------------------------------------------------------ tile hashing
// What a wave keeps for hashing its tiles with one signature kind: the
// matrix operands of djb2, or the CRC's staging area in LDS.
template <int kSig>
struct TileHash {
  Djb2Lane d;
  uint32_t first;   // the sixteen sectors it begins a tile with
  __device__ __forceinline__ explicit TileHash(uint32_t wave) : first(wave % (kTileSectors / 16)) { load_djb2_lane(d); }
  template <class Rows>
  __device__ __forceinline__ void load(const Rows& rows, PhaseRegs& r) const {   // a tile's first phase
    load_sectors<true>(rows, first, r);
  }
  // The weights again, for a kernel that needs their registers between tiles.
  __device__ __forceinline__ void reload() {
    uint32_t l = lane_id();
    asm volatile("" : "+v"(l));   // (or the compiler keeps the first ones)
    load_djb2_lane(d, l);
  }
  template <class Rows, class Prefetch>
  __device__ __forceinline__ uint64_t tile(const Rows& rows, PhaseRegs& A, PhaseRegs& B, Prefetch&& prefetch) const {
    return tile_djb2_pipelined<true>(rows, d, first, A, B, prefetch);
  }
};
template <>
struct TileHash<kSigCrc64> {
  uint8_t* my;   // this wave's staging area
  __device__ __forceinline__ explicit TileHash(uint32_t wave) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[kScanWaves * kTileLds];
    my = lds + wave * kTileLds;
  }
  template <class Rows>
  __device__ __forceinline__ void load(const Rows& rows, PhaseRegs& r) const {
    load_phase<true>(rows, 0, r);
  }
  __device__ __forceinline__ void reload() {}
  template <class Rows, class Prefetch>
  __device__ __forceinline__ uint64_t tile(const Rows& rows, PhaseRegs& A, PhaseRegs& B, Prefetch&& prefetch) const {
    return tile_crc_pipelined<true>(rows, my, A, B, prefetch);
  }
};

// ------------------------------------------------------------------ scan
// Persistent grid over the tile space (for launch shapes that cap the grid or
// ask for runs of tiles): wave q takes chunks q, q + W, ... of
// `chunk` consecutive tiles (W = waves in the grid). 4 waves per SIMD (at
// most 128 VGPRs): the more waves, the more sector loads in flight per CU.
// kLayout: the index's probe layout (not for kSigs). kFiltered: the index has a
// filter. Its instance is free of the registers that the probe without one needs
// (with those and the djb2 weights it spilled 6: 256 MiB at 4 blocks a CU 57.3 us,
// now 46.4), and the instance without reads the weights again for each tile
// (65.0 -> 59.0).
template <int kMode, int kSig, class Src, int kLayout, bool kFiltered>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_scan(
    Src src, uint32_t chunk, IndexView ix, uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  // the wave's index, uniform (so tile addresses stay in scalar registers)
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t l = lane_id();
  TileHash<kSig> hash(w);
  const uint64_t n_tiles = src.n_tiles();
  const uint64_t n_waves = (uint64_t)gridDim.x * kScanWaves;
  uint64_t g = ((uint64_t)blockIdx.x * kScanWaves + w) * chunk;
  if (g >= n_tiles) return;
  auto next_of = [&](uint64_t t) {
    return ((t + 1) % chunk != 0) ? t + 1 : t + 1 + (n_waves - 1) * chunk;
  };
  uint32_t cur = 0;
  TileRef tr = src.tile(g, cur);
  PhaseRegs A, B;
  hash.load(ContiguousRows{tr.base, tr.n_valid}, A);
  while (true) {
    const uint64_t gn = next_of(g);
    const bool more = gn < n_tiles;
    uint32_t cur_n = cur;
    TileRef tn = tr;
    // The next tile's first phase is loaded while this tile's last one is
    // hashed. Unconditionally (the last tile reloads itself): a load under a
    // branch would make the compiler wait for every load at the join. The
    // next tile is looked up only here, with this tile's last phase in
    // flight: in a batch the lookup walks the image descriptors (dependent
    // loads), which must not hold back this tile's own loads.
    auto prefetch = [&](PhaseRegs& R) {
      if (more) tn = src.tile(gn, cur_n);
      hash.load(ContiguousRows{tn.base, tn.n_valid}, R);
    };
    const uint64_t h = hash.tile(ContiguousRows{tr.base, tr.n_valid}, A, B, prefetch);
    if constexpr (kMode == kFlags || kMode == kFlagBits) {
      const uint32_t tau = (tr.tau_first + l) & (kClusterSectors - 1);
      uint64_t hits = tile_probe<kLayout, 1, kMode == kFlags, kFiltered>(
          ix, h, tau, tr.any_tau != 0, kMode == kFlags ? hit_slot + g * kTileSectors : nullptr, ix.bloom,
          ix.log2_bloom_words);
      if (tr.n_valid < kTileSectors) hits &= (1ull << tr.n_valid) - 1ull;
      if (l == 0) out[g] = hits;
    } else {
      if (l < tr.n_valid) out[g * kTileSectors + l] = h;   // one image: tile g holds sectors 64g..
    }
    if (!more) break;
    if constexpr (kMode != kSigs && kLayout == kLayoutBucketed && !kFiltered) hash.reload();
    g = gn;
    cur = cur_n;
    tr = tn;
  }
}

// ------------------------------------------------- djb2, a wave per sixteen sectors
// The default djb2 scan: a block is one wave, which requests its 16 sectors (8
// KiB) at once, hashes them on the matrix cores, looks them up and writes their
// 16 bits of the tile's hit word. No loop and no pipeline in the wave: at about
// 60 registers eight waves fit a SIMD, 64 KiB of loads in flight on each, and
// the hardware hands out the next block as a wave ends, so nothing is idle
// before the last few microseconds. Against the persistent grid of tiles of 64
// sectors (k_scan, with the same hashing, 2 blocks a CU), two passes of one run:
// 16 MiB 6.6, 7.4 -> 4.7, 4.6 us; 64 MiB 14.3, 14.9 -> 11.9, 12.6; 700 MiB 113,
// 117 -> 105, 109; 8 GiB 1255, 1262 -> 1214, 1253, 6.9-7.1 TB/s and bound by HBM
// (that grid at 1 block a CU, its best there: 1241, 1245, so 2% slower and 1%
// faster). When they were tried, blocks of four waves were 0-2% slower, 32
// sectors a wave 1% faster on 8 GiB and up to 7% slower below 1 GiB.
constexpr uint32_t kPart = 16;                          // sectors per wave
constexpr uint32_t kTileParts = kTileSectors / kPart;
constexpr uint64_t kMaxPartBlocks = 1ull << 26;         // fewer: a grid has fewer than 2^32 threads

// A wave's sectors `rows` (part `part` of the tile with hit word *out).
template <int kLayout, uint32_t kSlotStride, bool kSlots, bool kFiltered, class Rows>
__device__ __forceinline__ void scan_part(const Rows& rows, uint32_t part, uint32_t tau, bool any_tau,
                                          const IndexView& ix, const uint64_t* bloom, uint32_t log2_bloom,
                                          uint64_t* out, uint32_t* slots) {
  uint16_t* bits = (uint16_t*)out + part;   // little-endian: its bits of the word
  if (rows.n_valid == 0) {                  // past the image's end
    if (lane_id() == 0) *bits = 0;
    return;
  }
  PhaseRegs r;
  load_sectors<true>(rows, 0, r);
  Djb2Lane d;
  load_djb2_lane(d);
  const uint64_t h = sixteen_djb2(r, d);
  const uint64_t hits = tile_probe<kLayout, kSlotStride, kSlots, kFiltered, kPart>(ix, h, tau, any_tau, slots, bloom,
                                                                                   log2_bloom);
  if (lane_id() == 0) *bits = (uint16_t)(hits & ((1u << rows.n_valid) - 1u));
}
// Sectors of a part that starts `first` sectors into a tile of n.
__device__ __forceinline__ uint32_t part_valid(uint64_t n, uint64_t first) {
  return n <= first ? 0u : (n - first < kPart ? (uint32_t)(n - first) : kPart);
}

// The CRC's counterpart: a wave per tile of 64 sectors, since the CRC is a chain
// over a sector's bytes that one lane runs; four waves to a block (their staging
// areas are what bounds the waves of a CU, at 16). Against the persistent grid at
// 2 blocks a CU, two passes: 64 MiB 14.6, 14.5 -> 13.2, 13.4 us; 700 MiB 116, 116
// -> 110, 110; 2 GiB 322, 322 -> 305, 305; 8 GiB 1268, 1271 -> 1195, 1197. When it
// was tried, one wave to a block took 7.0 against 7.1 us on 1 MiB and 1.5% more
// from 700 MiB on.
template <int kMode, class Src, int kLayout>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_scan_tiles(
    Src src, uint64_t n_tiles, IndexView ix, uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t l = lane_id();
  TileHash<kSigCrc64> hash(w);
  const uint64_t g = (uint64_t)blockIdx.x * kScanWaves + w;
  if (g >= n_tiles) return;
  const TileRef tr = src.tile_at(g);
  const ContiguousRows rows{tr.base, tr.n_valid};
  PhaseRegs A, B;
  hash.load(rows, A);
  const uint64_t h = hash.tile(rows, A, B, [](PhaseRegs&) {});
  if constexpr (kMode == kSigs) {
    if (l < tr.n_valid) out[g * kTileSectors + l] = h;
  } else {
    uint64_t hits = tile_probe<kLayout, 1, kMode == kFlags>(
        ix, h, (tr.tau_first + l) & (kClusterSectors - 1), tr.any_tau != 0,
        kMode == kFlags ? hit_slot + g * kTileSectors : nullptr, ix.bloom, ix.log2_bloom_words);
    if (tr.n_valid < kTileSectors) hits &= (1ull << tr.n_valid) - 1ull;
    if (l == 0) out[g] = hits;
  }
}

// Block b takes part b mod 4 of tile b / 4.
template <int kMode, class Src, int kLayout>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(8))) void k_scan_parts(
    Src src, IndexView ix, uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  const uint32_t l = lane_id();
  const uint32_t part = blockIdx.x % kTileParts, first = part * kPart;
  const uint64_t g = blockIdx.x / kTileParts;
  const TileRef tr = src.tile_at(g);
  const ContiguousRows rows{tr.base + first * kSectorBytes, part_valid(tr.n_valid, first)};
  if constexpr (kMode == kSigs) {
    if (rows.n_valid == 0) return;
    PhaseRegs r;
    load_sectors<true>(rows, 0, r);
    Djb2Lane d;
    load_djb2_lane(d);
    const uint64_t h = sixteen_djb2(r, d);
    if (l < rows.n_valid) out[g * kTileSectors + first + l] = h;   // one image: tile g holds sectors 64g..
  } else {
    scan_part<kLayout, 1, kMode == kFlags, false>(
        rows, part, (tr.tau_first + l) & (kClusterSectors - 1), tr.any_tau != 0, ix, ix.bloom, ix.log2_bloom_words,
        out + g, kMode == kFlags ? hit_slot + g * kTileSectors + first : nullptr);
  }
}

// ------------------------------------------------- position-split scan
// One image, per-cluster rule, split by cluster position. Workgroups are
// dispatched to the chip's 8 XCDs in turn (block b runs on XCD b mod 8), so
// block b scans the sectors at position p = b mod 8 and probes position p's
// slice of the Bloom filter: each XCD's L2 holds one eighth of the filter
// instead of all of it (until the last tiles, which go to whichever waves are
// free; see the work sharing below). Tile k of position p is the sectors
// j = 8(64k + i) + r (i = 0..63, r = (p - tau0) mod 8), 512 B each, one
// cluster apart; its 64 hit bits go to tau_words[p * words_per_pos + k]
// (lane i = bit i), to be merged into the ordinary bitmap afterwards.
constexpr uint32_t kPositions = kClusterSectors;

__device__ __forceinline__ uint64_t position_count(uint64_t n_sectors, uint32_t r) {
  return n_sectors > r ? (n_sectors - r + kPositions - 1) / kPositions : 0;
}

// Work sharing of the position-split scan. A position's tiles go in runs of
// `chunk`. The first 7/8 of them are fixed: in round k, wave q of the
// position (of W) takes run kW + q. The rest are handed out by the
// position's counter (32 bits at the start of the p-th 256-byte line of ctr,
// zero at launch): a claim that returns c takes run KW + c (K = the fixed
// rounds). A wave whose position has no run left claims from the next
// positions in turn, so an XCD that finishes early takes over tiles of one
// that lags. On the 64 GiB large image with fixed shares only, the waves'
// finishing times spread over about 1 ms (even XCDs about 0.45 ms behind odd
// ones, and 0.65 ms within an XCD) and the kernel ended with the last; this
// scheme took it from 10.58-10.84 to 10.40-10.42 ms with runs of 2 tiles (the
// same scheme with every run claimed: 10.9-12.0 ms, because adds on one
// counter serialize at about 22 per microsecond; 3/4 or 15/16 fixed: no better).
constexpr uint32_t kCtrStride = 32;
constexpr uint32_t kTauCounters = kPositions * kCtrStride;

struct TauPos {
  uint32_t p;         // cluster position (its slice of the filter, its hit words)
  uint32_t r;         // its first sector: j = 8k + r
  uint64_t count;     // its sectors
  uint64_t n_tiles;
  uint64_t n_static;  // rounds of fixed runs (one run per wave of the position each)
};

__device__ __forceinline__ TauPos tau_pos(uint32_t p, uint64_t n_sectors, uint32_t tau0, uint64_t round_tiles) {
  TauPos t;
  t.p = p;
  t.r = (p - tau0) & (kPositions - 1);
  t.count = position_count(n_sectors, t.r);
  t.n_tiles = (t.count + kTileSectors - 1) / kTileSectors;
  t.n_static = t.n_tiles * 7 / (8 * round_tiles);   // 7/8 of the tiles in fixed runs
  return t;
}

// Lane 0 increments position p's counter (32 bits at the start of its line);
// the result is read later with tau_claim_read, so the atomic's latency hides
// behind the tile in flight. An increment, not an add: the compiler turns an
// add into a wave-wide atomic whose result it broadcasts, and waits for, at
// once.
__device__ __forceinline__ uint32_t tau_claim_issue(unsigned int* ctr, uint32_t p, uint32_t l) {
  uint32_t v = 0;
  if (l == 0) v = atomicInc(ctr + p * (2 * kCtrStride), 0xFFFFFFFFu);
  return v;
}
__device__ __forceinline__ uint64_t tau_claim_read(uint32_t v) {   // lane 0's value, to every lane
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// kSlots = false: no slot records (hit_slot unused). The index has the split filter.
template <int kSig, int kLayout = kLayoutBucketed, bool kSlots = true>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_scan_tau(
    const uint8_t* __restrict__ image, uint64_t n_sectors, uint32_t tau0, uint64_t words_per_pos, uint32_t chunk,
    IndexView ix, uint64_t* __restrict__ tau_words, uint32_t* __restrict__ hit_slot,
    unsigned int* __restrict__ ctr) {
  // the wave's index, uniform (so tile addresses stay in scalar registers)
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t l = lane_id();
  TileHash<kSig> hash(w);
  const uint64_t n_waves = (uint64_t)(gridDim.x / kPositions) * kScanWaves;   // per position
  const uint64_t q = (uint64_t)(blockIdx.x / kPositions) * kScanWaves + w;
  auto rows_of = [&](const TauPos& t, uint64_t k) {
    const uint64_t first = k * kTileSectors;   // its first cluster among the position's
    const uint64_t rem = t.count - first;
    return ClusterStrideRows{image + (first * kPositions + t.r) * kSectorBytes,
                             rem >= kTileSectors ? kTileSectors : (uint32_t)rem};
  };
  // A run claimed from position t's counter (c) or, once t has none left,
  // from the next positions; false when every position is done.
  const uint64_t round_tiles = n_waves * chunk;
  uint32_t visited = 1;
  auto claim_from = [&](TauPos& t, uint64_t c, uint64_t& g, uint64_t& end) {
    while (true) {
      g = (t.n_static * n_waves + c) * chunk;
      end = g + chunk;
      if (g < t.n_tiles) return true;
      if (visited == kPositions) return false;
      t = tau_pos((t.p + 1) & (kPositions - 1), n_sectors, tau0, round_tiles);
      ++visited;
      c = tau_claim_read(tau_claim_issue(ctr, t.p, l));
    }
  };
  TauPos cur = tau_pos(blockIdx.x % kPositions, n_sectors, tau0, round_tiles);
  uint64_t k = 0;          // the wave's fixed run of its own position
  bool fixed = cur.n_static > 0;
  uint64_t g = q * chunk, end = g + chunk;
  if (!fixed && !claim_from(cur, tau_claim_read(tau_claim_issue(ctr, cur.p, l)), g, end)) return;
  ClusterStrideRows tr = rows_of(cur, g);
  PhaseRegs A, B;
  hash.load(tr, A);
  while (true) {
    // the next tile: the rest of this run, else the wave's next fixed run,
    // else a claim issued now and read when the next tile's first loads are due
    const bool in_run = g + 1 < end && g + 1 < cur.n_tiles;
    const bool next_fixed = !in_run && fixed && k + 1 < cur.n_static;
    const bool claim = !in_run && !next_fixed;
    const uint32_t pending = claim ? tau_claim_issue(ctr, cur.p, l) : 0u;
    TauPos nxt = cur;
    uint64_t gn = g + 1, end_n = end;
    bool more = true;
    ClusterStrideRows tn = tr;
    auto prefetch = [&](PhaseRegs& R) {   // unconditionally, as in k_scan
      if (next_fixed) {
        gn = ((k + 1) * n_waves + q) * chunk;
        end_n = gn + chunk;
      } else if (claim) {
        // an empty asm that takes the claim's register here, so the compiler
        // waits for the atomic at this point and not where it was issued
        uint32_t c = pending;
        asm volatile("" : "+v"(c));
        more = claim_from(nxt, tau_claim_read(c), gn, end_n);
      }
      if (more) tn = rows_of(nxt, gn);
      hash.load(tn, R);
    };
    const uint64_t h = hash.tile(tr, A, B, prefetch);
    // this position's slice of the filter
    const uint64_t* bloom = ix.bloom_tau + ((uint64_t)cur.p << ix.log2_bloom_tau);
    uint64_t hits = tile_probe<kLayout, kPositions, kSlots, true>(
        ix, h, cur.p, false, kSlots ? hit_slot + (g * kTileSectors * kPositions + cur.r) : nullptr, bloom,
        ix.log2_bloom_tau);
    if (tr.n_valid < kTileSectors) hits &= (1ull << tr.n_valid) - 1ull;
    if (l == 0) tau_words[cur.p * words_per_pos + g] = hits;
    if (!more) break;
    if (next_fixed) ++k;
    if (claim) fixed = false;
    cur = nxt;
    g = gn;
    end = end_n;
    tr = tn;
  }
}


// The same split for k_scan_parts' way of scanning: block b takes, of position
// p = b mod 8 (so on XCD p), part (b / 8) mod 4 of tile b / 32. The hardware's
// hand-out of blocks balances each XCD's waves, so there are no claims. 16 M
// masters, against k_scan_tau at 2 blocks a CU (and at 1): 64 MiB 13 us against 40
// (29), 1 GiB 164 against 193 (178), 4 GiB 650 against 678 (647), 16 GiB 2583
// against 2649 (2540): k_scan_tau at 1 block a CU is up to 2% faster on large
// images, and 9% slower at 1 GiB. Every word of tau_words is written, the tiles
// past a position's sectors with zeros.
template <int kLayout, bool kSlots>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(8))) void k_scan_tau_parts(
    const uint8_t* __restrict__ image, uint64_t n_sectors, uint32_t tau0, uint64_t words_per_pos, IndexView ix,
    uint64_t* __restrict__ tau_words, uint32_t* __restrict__ hit_slot) {
  const uint32_t p = blockIdx.x % kPositions, r = (p - tau0) & (kPositions - 1);
  const uint32_t part = blockIdx.x / kPositions % kTileParts;
  const uint64_t g = blockIdx.x / (kPositions * kTileParts);
  const uint64_t k0 = g * kTileSectors + part * kPart;   // its first cluster
  const ClusterStrideRows rows{image + (k0 * kPositions + r) * kSectorBytes,
                               part_valid(position_count(n_sectors, r), k0)};
  scan_part<kLayout, kPositions, kSlots, true>(rows, part, p, false, ix,
                                               ix.bloom_tau + ((uint64_t)p << ix.log2_bloom_tau), ix.log2_bloom_tau,
                                               tau_words + p * words_per_pos + g,
                                               kSlots ? hit_slot + (k0 * kPositions + r) : nullptr);
}

// And for k_scan_tiles': block b takes tiles 4(b / 8).. of position b mod 8.
template <int kLayout, bool kSlots>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_scan_tau_tiles(
    const uint8_t* __restrict__ image, uint64_t n_sectors, uint32_t tau0, uint64_t words_per_pos, IndexView ix,
    uint64_t* __restrict__ tau_words, uint32_t* __restrict__ hit_slot) {
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t p = blockIdx.x % kPositions, r = (p - tau0) & (kPositions - 1);
  TileHash<kSigCrc64> hash(w);
  const uint64_t g = (uint64_t)(blockIdx.x / kPositions) * kScanWaves + w;
  if (g >= words_per_pos) return;
  const uint64_t k0 = g * kTileSectors;   // its first cluster
  const uint64_t count = position_count(n_sectors, r);
  uint64_t hits = 0;
  if (count > k0) {
    const uint32_t n = count - k0 < kTileSectors ? (uint32_t)(count - k0) : kTileSectors;
    const ClusterStrideRows rows{image + (k0 * kPositions + r) * kSectorBytes, n};
    PhaseRegs A, B;
    hash.load(rows, A);
    const uint64_t h = hash.tile(rows, A, B, [](PhaseRegs&) {});
    hits = tile_probe<kLayout, kPositions, kSlots, true>(
        ix, h, p, false, kSlots ? hit_slot + (k0 * kPositions + r) : nullptr,
        ix.bloom_tau + ((uint64_t)p << ix.log2_bloom_tau), ix.log2_bloom_tau);
    if (n < kTileSectors) hits &= (1ull << n) - 1ull;
  }
  if (lane_id() == 0) tau_words[p * words_per_pos + g] = hits;
}

}  // namespace carve
