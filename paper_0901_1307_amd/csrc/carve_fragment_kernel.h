// Fragment scan (Section 5): every 64-byte window of an image that starts on
// a 4-byte boundary (window j = bytes [4j, 4j + 64)), hashed with djb2 over
// its 64 bytes (Eq. (1)), looked up among the signatures of the master files'
// 64-byte fragments at any position. Device code only; included by carve.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "carve_device.h"
#include "carve_scan_kernel.h"

namespace carve {

constexpr uint32_t kFragBytes = 64;                          // a master fragment, an image window
constexpr uint32_t kWindowStride = 4;                        // windows start on 4-byte boundaries
constexpr uint32_t kFragThreads = 1024;                      // one block per CU: its LDS holds the filter
constexpr uint32_t kFragWaves = kFragThreads / kWave;
constexpr uint32_t kWaveWindows = 1024;                      // windows per wave task: 4 KiB of image
constexpr uint32_t kBlocks16 = kWaveWindows / 256;           // matrix blocks of a task: 16 rows of 16 windows each
constexpr uint32_t kCandidates = kWave;                      // candidate windows a wave queues at once
// Per wave in LDS: the queue (key, window) and the hit bits of its task.
constexpr uint32_t kFragWaveLds = 2 * kCandidates + kWaveWindows / 32;
// The first filter takes the rest of a CU's 160 KiB of LDS (less what the task
// counter and rounding need): 149.75 KiB.
constexpr uint32_t kLdsFilterMaxWords = 40960 - kFragWaves * kFragWaveLds - 64;
static_assert(kLdsFilterMaxWords % 4 == 0, "copied 16 bytes at a time");
constexpr int kDppWaveShl1 = 0x130;   // DPP controls: lane i takes lane i + 1's value, across the wave
constexpr int kDppRowShl1 = 0x101;    // the same inside each 16 lanes
constexpr int kDppRowRor15 = 0x12F;   // and with lane 15 of the 16 taking lane 0's
// Buffer descriptor word 3 for raw (unformatted, unswizzled) dword access on
// gfx9-family chips: data format 32 in bits 15-18 (value 4), the rest 0.
constexpr int kRawBufferFlags = 0x00020000;

// The two filters of a fragment index, both of 32-bit words, are placed from
// a 32-bit key: the low half of the window's data part H (its
// signature minus the constant 5381*33^64, below) less another constant that
// the matrix units' signed bytes leave in it. Reduction modulo 2^32 respects
// sums and products, so the scan makes k in 32 bits alone, and equal signatures
// give equal keys; the full 64-bit signature is formed only for the rare
// windows that pass both filters.
// Each level takes one 32 x 32 -> 64-bit product of the key (a = k * kFragMulA,
// b = k * kFragMulB; one multiply-add instruction each, the only full 32-bit
// multiplies of a lookup):
// * first level, in LDS: the word from the low 24 bits of a's high half scaled
//   to the word count (a 24-bit multiply, which need not be a power of two),
//   2 bit positions from bits 24-28 of a's high and of a's low half;
// * second level, the Bloom filter in L2: the word from the top bits of b's
//   low half, 3 bit positions from bits 0-4, 16-20 and 24-28 of b's high half.
// Bit positions sit at byte and half-word boundaries so that the scan's shifts
// take them straight from the product's register (sub-dword operand selects).
// A simulation of the logos set's filters on random keys: both levels pass
// 0.033% of windows; 3 Bloom bits keep the exact path rare for two
// instructions fewer than 4. Only windows that pass the first level read the
// second. Key 0 is placed like any other; when a master's whole signature is
// 0 (it lives beside the table, not in it) the build sets the bits of its key
// in both filters, so no value needs special handling in the scan.
constexpr uint32_t kFragMulA = 0x9E3779B1u;
constexpr uint32_t kFragMulB = 0x85EBCA77u;
// A first-level lookup: the word and the 2 bit positions (each < 32).
struct FragLdsProbe {
  uint32_t word, p0, p1;
};
// n_words in 1..kLdsFilterMaxWords (so n_words * 256 < 2^24).
__device__ __forceinline__ FragLdsProbe frag_lds_probe(uint32_t key, uint32_t n_words) {
  const uint64_t a = (uint64_t)key * kFragMulA;
  const uint32_t hi = (uint32_t)(a >> 32), lo = (uint32_t)a;
  FragLdsProbe r;
  const uint32_t n8 = (n_words << 8) & 0xFFFFFFu;   // both factors 24-bit: a 24-bit multiply
  r.word = (uint32_t)(((uint64_t)(hi & 0xFFFFFFu) * n8) >> 32);   // < n_words
  r.p0 = (hi >> 24) & 31u;
  r.p1 = (lo >> 24) & 31u;
  return r;
}
// A second-level lookup: the word's byte offset and the 3 bit positions.
struct FragBloomProbe {
  uint32_t byte_off, p0, p1, p2;
};
// log2_words in 1..30 (the filter has 2 to 2^30 words).
__device__ __forceinline__ FragBloomProbe frag_bloom_probe(uint32_t key, uint32_t log2_words) {
  const uint64_t b = (uint64_t)key * kFragMulB;
  const uint32_t hi = (uint32_t)(b >> 32), lo = (uint32_t)b;
  FragBloomProbe r;
  r.byte_off = (lo >> (30 - log2_words)) & ~3u;   // the word (top log2_words bits of lo) times 4
  r.p0 = hi & 31u;
  r.p1 = (hi >> 16) & 31u;
  r.p2 = (hi >> 24) & 31u;
  return r;
}
// The build's view: the word and its bits.
__device__ __forceinline__ void frag_lds_place(uint32_t key, uint32_t n_words, uint32_t* word, uint32_t* bits) {
  const FragLdsProbe r = frag_lds_probe(key, n_words);
  *word = r.word;
  *bits = (0x80000000u >> r.p0) | (0x80000000u >> r.p1);
}
__device__ __forceinline__ void frag_bloom_place(uint32_t key, uint32_t log2_words, uint32_t* word, uint32_t* bits) {
  const FragBloomProbe r = frag_bloom_probe(key, log2_words);
  *word = r.byte_off >> 2;
  *bits = (0x80000000u >> r.p0) | (0x80000000u >> r.p1) | (0x80000000u >> r.p2);
}
// The scan's view: whether all of a probe's bits are set in the filter word x.
// A position p is bit 31 - p, so a shift left by p brings it to the sign and
// the test is a compare with 0 (a shift by each position, an and, a compare:
// fewer instructions than a mask built and compared).
__device__ __forceinline__ bool frag_lds_has(uint32_t x, const FragLdsProbe& r) {
  return (int32_t)((x << r.p0) & (x << r.p1)) < 0;
}
__device__ __forceinline__ bool frag_bloom_has(uint32_t x, const FragBloomProbe& r) {
  return (int32_t)((x << r.p0) & (x << r.p1) & (x << r.p2)) < 0;
}

// Window keys on the matrix cores. With the window's data part H(j) =
// sum_{i<64} s[4j+i] 33^(63-i) (its signature is 5381*33^64 + H), take the image
// in rows of 64 bytes: the window at word n of row R has its first 64 - 4n bytes
// in row R and the rest in row R + 1. So for the 16 windows n = 0..15 that start
// in a row, H is the row's bytes times one 64 x 16 matrix of weights (zero above
// byte 4n) plus the next row's bytes times another (zero from byte 4n on). Both
// are split into signed base-256 digit planes; the filter key needs H modulo
// 2^32 only, four planes. As in the sector hash the bytes enter as s - 128,
// which shifts every key by the same constant.
constexpr uint64_t kPow4 = pow33(4);
constexpr uint64_t kFragInit = 5381ull * pow33(kFragBytes);
constexpr uint64_t frag_shift() {   // 128 times the sum of a window's weights
  uint64_t c = 0, w = 1;
  for (uint32_t i = 0; i < kFragBytes; ++i, w *= 33) c += 128ull * w;
  return c;
}
constexpr uint32_t kFragKeyShift = (uint32_t)(kFragInit + frag_shift());
// The filter key of a signature: its data part less the shift, modulo 2^32.
__device__ __forceinline__ uint32_t frag_filter_key(uint64_t sig) { return (uint32_t)sig - kFragKeyShift; }

constexpr uint32_t kKeyPlanes = 4;
// A weight depends on the byte's distance from the window's start alone: lane l
// of a wave has column n = l mod 16 (the window) and bytes 16(l/16)..16(l/16)+15
// of the row, so plane q of its weights is 16 consecutive entries of one table
// of 64, from (16(l/16) - 4n) mod 64 on and round its end. (One table of 320
// bytes for every wave, and selects, once: a table of the lanes' registers is 8
// KiB for each wave to read, as much again as the block's filter.)
struct FragWeights {
  uint32_t w[kKeyPlanes][(kFragBytes + 16) / 4];
};
constexpr FragWeights make_frag_weights() {
  FragWeights t{};
  for (uint32_t q = 0; q < kKeyPlanes; ++q)
    for (uint32_t i = 0; i < kFragBytes + 16; ++i)
      t.w[q][i / 4] |= (uint32_t)(signed_digit(pow33(kFragBytes - 1 - i % kFragBytes), q) & 0xFF) << (8 * (i % 4));
  return t;
}
__device__ const FragWeights g_frag_weights = make_frag_weights();
typedef uint32_t u32x4_dw __attribute__((ext_vector_type(4), aligned(4)));
struct FragLane {
  i32x4 w[2][kKeyPlanes];   // [this row, the next][plane]
};
__device__ __forceinline__ void load_frag_lane(FragLane& f) {
  const uint32_t n = lane_id() & 15u, g = lane_id() >> 4;
#pragma unroll
  for (uint32_t q = 0; q < kKeyPlanes; ++q) {
    const u32x4_dw v = *(const u32x4_dw*)(g_frag_weights.w[q] + ((4u * g - n) & 15u));
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const bool next = 4u * g + k < n;
      f.w[0][q][k] = next ? 0 : (int)v[k];
      f.w[1][q][k] = next ? (int)v[k] : 0;
    }
  }
}

// The byte weights of D = b0 33^3 + b1 33^2 + b2 33 + b3 (the bytes of a word in
// address order, D < 2^24) in dot4 form: D = dot(word, low bytes of 33^(3-i))
// + 256 dot(word, second bytes of 33^(3-i)) (33^3 < 2^16).
constexpr uint32_t word_weights(uint32_t shift) {
  uint32_t w = 0;
  for (uint32_t k = 0; k < 4; ++k) w |= (uint32_t)((pow33(3 - k) >> shift) & 0xFFu) << (8 * k);
  return w;
}
constexpr uint32_t kWordWeightsLo = word_weights(0);
constexpr uint32_t kWordWeightsHi = word_weights(8);

__device__ __forceinline__ uint32_t word_djb2(uint32_t x) {
  return __builtin_amdgcn_udot4(x, kWordWeightsLo, 0u, false) +
         (__builtin_amdgcn_udot4(x, kWordWeightsHi, 0u, false) << 8);
}

// Signature of a whole 64-byte fragment (16 words, little-endian dwords).
__device__ __forceinline__ uint64_t fragment_signature(const uint32_t* w) {
  uint64_t H = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) H = H * kPow4 + word_djb2(w[k]);
  return kFragInit + H;
}

// The windows of one image as a tile space for compaction and confirmation:
// unit j is bytes [4j, 4j + 64); d.n_sectors holds the number of windows.
struct FragmentWindows {
  static constexpr uint32_t kUnitBytes = kFragBytes, kUnitStride = kWindowStride;
  static constexpr bool kAnyPosition = true, kManyImages = false;
  ImageDesc d;
  __device__ __forceinline__ uint64_t n_tiles() const { return (d.n_sectors + kTileSectors - 1) / kTileSectors; }
  __device__ __forceinline__ const ImageDesc& image(uint32_t) const { return d; }
  __device__ __forceinline__ uint32_t image_between(uint64_t, uint32_t, uint32_t) const { return 0; }
};

// A task's image words for lane l, as the matrix operand: of block b, 16 bytes
// of row 16b + l mod 16 at byte 16(l/16); and the same piece of the row after
// the task's last (v[kBlocks16]). Every task but the image's last lies wholly
// inside the image (n_dwords >= n_windows + 15); the last task clamps every
// dword to the image's last one (only windows past the end read the repeated
// words).
struct TaskWords {
  u32x4 v[kBlocks16 + 1];
};
// The inside task's words come by buffer loads from a descriptor based at
// the task (scalar base, 32-bit lane offsets: less address arithmetic than
// 64-bit global addresses), cached as any others: streaming and system-scoped
// (nt, sc1) took 1.068 vs 1.041 ms on the 2 GiB logos workload, because a
// candidate's bytes are read again.
__device__ __forceinline__ void load_task_inside(const uint32_t* __restrict__ image, uint64_t t, uint32_t l,
                                                 TaskWords& T) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc((void*)(image + t * kWaveWindows), (short)0,
                                        (int)(kWaveWindows * kWindowStride + kFragBytes), kRawBufferFlags);
  const uint32_t at = (l & 15u) * kFragBytes + (l >> 4) * 16u;
#pragma unroll
  for (uint32_t b = 0; b <= kBlocks16; ++b) {
    const uint32_t off = b < kBlocks16 ? at + b * 16u * kFragBytes : (l >> 4) * 16u + kWaveWindows * kWindowStride;
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    T.v[b] = u32x4{v[0], v[1], v[2], v[3]};
  }
}
__device__ __forceinline__ void load_task_clamped(const uint32_t* __restrict__ image, uint64_t n_dwords, uint64_t t,
                                                  uint32_t l, TaskWords& T) {
#pragma unroll
  for (uint32_t b = 0; b <= kBlocks16; ++b) {
    const uint32_t row = b < kBlocks16 ? 16u * b + (l & 15u) : 16u * kBlocks16;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint64_t g = t * kWaveWindows + row * (kFragBytes / 4) + (l >> 4) * 4u + k;
      T.v[b][k] = image[g < n_dwords ? g : n_dwords - 1];
    }
  }
}

// The candidate windows of a task (few), one per lane with `ok`: window id of
// the task; its bytes read again (from L2), hashed in full and looked up. A hit
// sets the window's bit in `bits` and records its slot.
__device__ __forceinline__ void frag_exact(const uint32_t* __restrict__ image, const IndexView& ix, uint64_t first,
                                           uint32_t id, bool ok, uint32_t* bits, uint32_t* __restrict__ hit_slot) {
  if (!ok) return;
  const uint64_t j = first + id;
  uint32_t w[16];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const u32x4_dw v = ((const u32x4_dw*)(image + j))[k];
    w[4 * k] = v.x;
    w[4 * k + 1] = v.y;
    w[4 * k + 2] = v.z;
    w[4 * k + 3] = v.w;
  }
  const uint64_t sig = fragment_signature(w);
  int64_t slot = -1;
  if (sig == kEmptyKey) {
    if (ix.zero_sig_mask) slot = ix.zero_slot;
  } else {
    slot = find_slot(ix, sig);   // any position: every occupied slot has masters
  }
  if (slot >= 0) {
    hit_slot[j] = (uint32_t)slot;
    atomicOr(&bits[id / 32], 1u << (id % 32));
  }
}

// (x << 8) + y, one instruction. The empty asm keeps nested ones apart: the
// compiler would shift each plane by itself and add, twice as many. (It stays
// empty because the compiler spaces an instruction that reads a matrix result
// from the one that makes it, and knows only its own.)
__device__ __forceinline__ uint32_t shl8_add(uint32_t x, uint32_t y) {
  uint32_t r = (x << 8) + y;
  asm("" : "+v"(r));
  return r;
}

// The keys of a task's windows: key[4b + j] of lane l is that of window
// frag_window(l) + 256b + 16j. Block b is rows 16b..16b+15 of the task; its
// "next rows" are those rows one lane on, with lane 15 of each 16 taking the
// following block's row 0.
__device__ __forceinline__ uint32_t frag_window(uint32_t l) { return 64u * (l >> 4) + (l & 15u); }
__device__ __forceinline__ void frag_keys(const TaskWords& T, const FragLane& f, uint32_t (&key)[4 * kBlocks16]) {
  const u32x4 flip = {0x80808080u, 0x80808080u, 0x80808080u, 0x80808080u};
  i32x4 a = (i32x4)(T.v[0] ^ flip);
#pragma unroll
  for (uint32_t b = 0; b < kBlocks16; ++b) {
    const i32x4 c = (i32x4)(T.v[b + 1] ^ flip);
    i32x4 next;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // (the words after the task are the same in all of a group's lanes)
      const int first = b + 1 < kBlocks16 ? __builtin_amdgcn_update_dpp(0, c[k], kDppRowRor15, 0xF, 0xF, true) : c[k];
      next[k] = __builtin_amdgcn_update_dpp(first, a[k], kDppRowShl1, 0xF, 0xF, false);
    }
    i32x4 p[kKeyPlanes];
#pragma unroll
    for (uint32_t q = 0; q < kKeyPlanes; ++q) {
      const i32x4 zero = {0, 0, 0, 0};
      p[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, f.w[0][q], zero, 0, 0, 0);
    }
#pragma unroll
    for (uint32_t q = 0; q < kKeyPlanes; ++q)
      p[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(next, f.w[1][q], p[q], 0, 0, 0);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      key[4 * b + j] = shl8_add(shl8_add(shl8_add(p[3][j], p[2][j]), p[1][j]), p[0][j]);
    }
    a = c;
  }
}

// One task of a wave (see k_frag_scan). kBloom: the index has the second
// filter. my: the wave's kFragWaveLds words of LDS.
template <bool kBloom>
__device__ __forceinline__ void frag_task(const uint32_t* __restrict__ image, uint64_t n_windows, uint64_t n_words,
                                          const IndexView& ix, const FragLane& f, const uint32_t* lfilter, uint32_t lw,
                                          uint32_t* my, uint64_t t, uint32_t l, const TaskWords& cur,
                                          uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  constexpr uint32_t kLaneWindows = 4 * kBlocks16;
  const char* bloom = (const char*)ix.bloom;   // fragment indexes: 32-bit words
  const uint32_t lwb = ix.log2_bloom_words + 1;
  uint32_t* bits = my + 2 * kCandidates;
  bits[l % (kWaveWindows / 32)] = 0;
  uint32_t h[kLaneWindows];
  frag_keys(cur, f, h);
  const uint64_t first = t * kWaveWindows;
  // windows that pass the first filter: masks of lanes
  uint64_t left[kLaneWindows];
#pragma unroll
  for (uint32_t w = 0; w < kLaneWindows; ++w) {
    const FragLdsProbe r = frag_lds_probe(h[w], lw);
    left[w] = ballot(frag_lds_has(lfilter[r.word], r));
  }
  const uint32_t own = frag_window(l);
  if (n_windows - first < kWaveWindows) {   // the last task: only windows inside the image
    uint32_t n = (uint32_t)(n_windows - first);
    asm volatile("" : "+v"(n));   // kept a branch: these compares are not worth making for every task
#pragma unroll
    for (uint32_t w = 0; w < kLaneWindows; ++w) left[w] &= ballot(own + 256u * (w / 4) + 16u * (w % 4) < n);
  }
  // They are few and scattered over the lanes (20% of random windows at the
  // filter's largest fill), and a wave's load of scattered words costs its 64
  // address cycles however many lanes need theirs, so each four windows'
  // candidates are queued in LDS and the second filter read for up to 64 of
  // them at a time, all four loads in flight together. Four windows of more than
  // 64 candidates queue one window's and leave the rest for another trip.
  constexpr uint32_t kQuarter = 4;
  bool more;
  do {
    more = false;
    uint64_t ok[kQuarter];
    uint32_t id[kQuarter], fw[kQuarter];
    FragBloomProbe r[kQuarter];
#pragma unroll
    for (uint32_t q = 0; q < kQuarter; ++q) {
      uint64_t now[4], later[4] = {0, 0, 0, 0};
      uint32_t n = 0;
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        now[k] = left[4 * q + k];
        n += (uint32_t)__popcll(now[k]);
      }
      if (n > kCandidates) {   // uniform
        more = true;
        bool taken = false;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
          if (taken) {
            later[k] = now[k];
            now[k] = 0;
          }
          if (now[k]) taken = true;
        }
      }
      n = 0;
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint64_t m = now[k];
        const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, n));
        n += (uint32_t)__popcll(m);
        if (__builtin_amdgcn_inverse_ballot_w64(m)) {
          my[pos] = h[4 * q + k];
          my[kCandidates + pos] = own + 256u * q + 16u * k;
        }
        left[4 * q + k] = later[k];
      }
      wave_sync_lds();
      const uint32_t key = my[l];
      id[q] = my[kCandidates + l];
      ok[q] = n < kWave ? (1ull << n) - 1ull : ~0ull;
      wave_sync_lds();
      if constexpr (kBloom) {
        r[q] = frag_bloom_probe(key, lwb);
        fw[q] = *(const uint32_t*)(bloom + (l < n ? r[q].byte_off : 0u));   // unconditional: no branch around it
      }
    }
    uint64_t any = 0;
#pragma unroll
    for (uint32_t q = 0; q < kQuarter; ++q) {
      if constexpr (kBloom) ok[q] &= ballot(frag_bloom_has(fw[q], r[q]));
      any |= ok[q];
    }
    // what passed both, mostly in one of the four: one lookup per lane and turn
    while (any) {   // uniform
      uint32_t at = 0;
      uint64_t turn = 0;
#pragma unroll
      for (uint32_t q = 0; q < kQuarter; ++q) {
        const uint64_t m = ok[q] & ~turn;
        at = __builtin_amdgcn_inverse_ballot_w64(m) ? id[q] : at;
        turn |= m;
        ok[q] &= ~m;
      }
      frag_exact(image, ix, first, at, __builtin_amdgcn_inverse_ballot_w64(turn), bits, hit_slot);
      any = ok[1] | ok[2] | ok[3];
    }
  } while (more);
  wave_sync_lds();
  // the task's 16 hit words
  const uint64_t wi = t * (kWaveWindows / kTileSectors) + l;
  if (l < kWaveWindows / kTileSectors && wi < n_words) out[wi] = ((const uint64_t*)bits)[l];
  wave_sync_lds();
}

// Persistent grid of one block per CU. Task t is windows [1024t, 1024t + 1024);
// hit word 16t + m has bit b for window 64(16t + m) + b, and each hit's table
// slot goes to hit_slot[window]. The block's LDS holds the first filter, the
// waves' queues and their hit bits; the image goes straight to registers.
// What bounds it is the chain of a task (words, keys, first filter, queue,
// second filter) at the 4 waves per SIMD that the filter leaves: 540 M windows
// of the logos image in 1.04 ms, 2.1 TB/s. Before, with every key rolled by
// its lane, a Bloom word read for all windows or none of a wave and fixed
// shares of tasks, 1.12 ms (500 files: 0.71 vs 0.81; 120: 0.71 vs 0.80). Of
// that the claimed tasks give 2-4%: the hardware favours a block's older waves,
// which ended 0.2 ms before its youngest with a fixed share each. Requesting a
// task's words ahead was slower in every form (1.12-1.34 ms): loads return in
// order, so the next task's image words hold up this one's filter words.
template <bool kBloom>
__global__ __launch_bounds__(kFragThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_frag_scan(
    const uint32_t* __restrict__ image, uint64_t n_windows, uint64_t n_dwords, IndexView ix,
    uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  __shared__ __attribute__((aligned(16))) uint32_t lfilter[kLdsFilterMaxWords];
  __shared__ __attribute__((aligned(16))) uint32_t wave_lds[kFragWaves * kFragWaveLds];
  const uint32_t lw = ix.lds_words;   // at most kLdsFilterMaxWords
  // (lw is a multiple of 4)
  for (uint32_t i = 4 * threadIdx.x; i < lw; i += 4 * kFragThreads)
    *(u32x4*)(lfilter + i) = *(const u32x4*)(ix.lds_filter + i);
  FragLane f;
  load_frag_lane(f);
  __shared__ uint32_t claimed;
  if (threadIdx.x == 0) claimed = 0;
  __syncthreads();   // before any wave of the block can leave
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t l = lane_id();
  const uint64_t n_tasks = (n_windows + kWaveWindows - 1) / kWaveWindows;
  const uint64_t n_words = (n_windows + kTileSectors - 1) / kTileSectors;
  const uint64_t n_waves = (uint64_t)gridDim.x * kFragWaves;
  const uint64_t last = n_tasks - 1;   // n_windows >= 1 (the host launches nothing otherwise)
  while (true) {
    uint32_t k = 0;
    if (l == 0) k = atomicAdd(&claimed, 1u);
    k = (uint32_t)__builtin_amdgcn_readfirstlane((int)k);
    const uint64_t t = (uint64_t)(k / kFragWaves) * n_waves + blockIdx.x * kFragWaves + k % kFragWaves;
    if (t >= n_tasks) break;
    TaskWords cur;
    if (t < last) load_task_inside(image, t, l, cur);   // uniform branch
    else load_task_clamped(image, n_dwords, t, l, cur);
    frag_task<kBloom>(image, n_windows, n_words, ix, f, lfilter, lw, wave_lds + wv * kFragWaveLds, t, l, cur, out,
                      hit_slot);
  }
}

// A small image, of at most one task for each wave of the grid: the keys of a
// task are rolled instead, lane l taking windows 16l..16l+15, by
//   H(j+1) = H(j) 33^4 - 33^64 D(j) + D(j+16)        (mod 2^64)
// from Horner over the first window's words. The windows' lookups then lie in
// lanes side by side with no queue between the filters and the candidates' full
// signatures are rolled from words in registers: more instructions, but a
// shorter chain, and one task's chain is all that such a launch waits for. With
// the logos set 10.0 vs 13.2 us at 1 MiB and 15.4 vs 21.2 us at 16 MiB (4,096
// tasks for 4,096 waves), 11.1 vs 15.4 with 120 files; at 32 MiB, two tasks a
// wave, k_frag_scan takes 30 us and a rolling loop 33. The image words are
// requested after the filter: before it, they measured 10.6 and 16.2 us.
constexpr uint32_t kRolled = kWaveWindows / kWave;   // windows of a lane, and its own dwords
constexpr uint64_t kRollAdd = kFragInit - kFragInit * kPow4;          // mod 2^64
constexpr uint64_t kNegPow64 = 0ull - pow33(kFragBytes);              // mod 2^64
template <bool kBloom>
__global__ __launch_bounds__(kFragThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_frag_scan_once(
    const uint32_t* __restrict__ image, uint64_t n_windows, uint64_t n_dwords, IndexView ix,
    uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  __shared__ __attribute__((aligned(16))) uint32_t lfilter[kLdsFilterMaxWords];
  const uint32_t lw = ix.lds_words;   // at most kLdsFilterMaxWords
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t l = lane_id();
  const uint64_t t = (uint64_t)blockIdx.x * kFragWaves + wv;
  const uint64_t first = t * kWaveWindows;
  const uint64_t j0 = first + (uint64_t)l * kRolled;
  for (uint32_t i = 4 * threadIdx.x; i < lw; i += 4 * kFragThreads)
    *(u32x4*)(lfilter + i) = *(const u32x4*)(ix.lds_filter + i);
  __syncthreads();
  if (first >= n_windows) return;
  // the lane's own dwords and, in lanes 0-15, the first of the next task (which
  // lane 63's windows reach); clamped as in k_frag_scan
  uint32_t cur[kRolled], curx;
  if (first + kWaveWindows < n_windows) {   // uniform
#pragma unroll
    for (uint32_t q = 0; q < kRolled / 4; ++q) {
      const u32x4_dw v = *(const u32x4_dw*)(image + j0 + 4 * q);
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) cur[4 * q + k] = v[k];
    }
    curx = image[first + kWaveWindows + (l % kRolled)];
  } else {
    const uint64_t end = n_dwords - 1;
#pragma unroll
    for (uint32_t k = 0; k < kRolled; ++k) {
      const uint64_t g = j0 + k;
      cur[k] = image[g < end ? g : end];
    }
    const uint64_t g = first + kWaveWindows + (l % kRolled);
    curx = image[g < end ? g : end];
  }
  const char* bloom = (const char*)ix.bloom;   // fragment indexes: 32-bit words
  const uint32_t lwb = ix.log2_bloom_words + 1;
  uint32_t d[kRolled];   // D of the lane's dwords
#pragma unroll
  for (uint32_t k = 0; k < kRolled; ++k) d[k] = word_djb2(cur[k]);
  const uint32_t dx = word_djb2(curx);
  // nx[k] = D(dword 16l + 16 + k): the next lane's d[k]; for lane 63, lane k's
  // dx, which a permute brings first (the other lanes read lanes below 31 and
  // are overwritten by the shift across the wave)
  const uint32_t ext_from = l == kWave - 1 ? 0u : 4u * (l % kRolled);   // byte address of a lane
  uint32_t nx[kRolled];
#pragma unroll
  for (uint32_t k = 0; k < kRolled; ++k) {
    const int ext = __builtin_amdgcn_ds_bpermute((int)(ext_from + 4u * k), (int)dx);
    nx[k] = (uint32_t)__builtin_amdgcn_update_dpp(ext, (int)d[k], kDppWaveShl1, 0xF, 0xF, false);
  }
  const uint32_t valid = j0 >= n_windows ? 0u : (n_windows - j0 >= kRolled ? kRolled : (uint32_t)(n_windows - j0));
  uint32_t s = 0;   // H modulo 2^32
#pragma unroll
  for (uint32_t k = 0; k < kRolled; ++k) s = s * (uint32_t)kPow4 + d[k];
  uint32_t h[kRolled];
#pragma unroll
  for (uint32_t w = 0; w < kRolled; ++w) {
    h[w] = s - (kFragKeyShift - (uint32_t)kFragInit);
    s = s * (uint32_t)kPow4 + (uint32_t)kNegPow64 * d[w] + nx[w];   // unused after the last window
  }
  // windows still candidates
  uint32_t pend = valid >= 16 ? 0xFFFFu : (1u << valid) - 1u;
  uint32_t pass = 0;
#pragma unroll
  for (uint32_t w = 0; w < kRolled; ++w) {
    const FragLdsProbe r = frag_lds_probe(h[w], lw);
    pass |= (uint32_t)frag_lds_has(lfilter[r.word], r) << w;
  }
  pend &= pass;
  if constexpr (kBloom) {
    // all in flight together: a window that failed reads the filter's first word
    FragBloomProbe r[kRolled];
    uint32_t fw[kRolled];
#pragma unroll
    for (uint32_t w = 0; w < kRolled; ++w) {
      r[w] = frag_bloom_probe(h[w], lwb);
      const uint32_t keep = 0u - ((pend >> w) & 1u);   // all ones or zero
      fw[w] = *(const uint32_t*)(bloom + (r[w].byte_off & keep));
    }
    pass = 0;
#pragma unroll
    for (uint32_t w = 0; w < kRolled; ++w) pass |= (uint32_t)frag_bloom_has(fw[w], r[w]) << w;
    pend &= pass;
  }
  // few are left: their full signatures, rolled across the lane's windows
  uint32_t mask = 0;
  if (pend) {
    uint64_t H = 0;
#pragma unroll
    for (uint32_t k = 0; k < kRolled; ++k) H = H * kPow4 + d[k];
    uint64_t sig = kFragInit + H;
#pragma unroll
    for (uint32_t w = 0; w < kRolled; ++w) {
      if ((pend >> w) == 0u) break;   // no candidate left in this lane
      if ((pend >> w) & 1u) {
        int64_t slot = -1;
        if (sig == kEmptyKey) {
          if (ix.zero_sig_mask) slot = ix.zero_slot;
        } else {
          slot = find_slot(ix, sig);   // any position: every occupied slot has masters
        }
        if (slot >= 0) {
          mask |= 1u << w;
          hit_slot[j0 + w] = (uint32_t)slot;
        }
      }
      sig = sig * kPow4 + (kRollAdd + kNegPow64 * d[w]) + nx[w];
    }
  }
  // four lanes' 16-bit masks make one 64-bit hit word
  const uint32_t m1 = (uint32_t)__shfl_down((int)mask, 1, kWave);
  const uint32_t m2 = (uint32_t)__shfl_down((int)mask, 2, kWave);
  const uint32_t m3 = (uint32_t)__shfl_down((int)mask, 3, kWave);
  const uint64_t wi = t * (kWaveWindows / kTileSectors) + l / 4;
  if ((l & 3u) == 0 && wi < (n_windows + kTileSectors - 1) / kTileSectors)
    out[wi] = (uint64_t)(mask | (m1 << 16)) | ((uint64_t)(m2 | (m3 << 16)) << 32);
}

}  // namespace carve
