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
// The first filter takes a CU's 160 KiB of LDS, less what the task counter and rounding need.
constexpr uint32_t kLdsFilterMaxWords = 40960 - 16;
static_assert(kLdsFilterMaxWords % 4 == 0, "copied 16 bytes at a time");
constexpr int kDppWaveShl1 = 0x130;   // DPP controls: lane i takes lane i + 1's value, across the wave
// The two filters of a fragment index, both of 32-bit words, are placed from
// a 32-bit key: the low half of the window's data part H (its signature minus the
// constant 5381*33^64, below). Reduction modulo 2^32 respects sums and products,
// so the scan rolls H in 32 bits alone, and equal signatures give equal keys; the
// full 64-bit signature is formed only for the rare windows that pass both
// filters.
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

constexpr uint64_t kPow4 = pow33(4);
constexpr uint64_t kFragInit = 5381ull * pow33(kFragBytes);
// The filter key of a signature: its data part, modulo 2^32.
__device__ __forceinline__ uint32_t frag_filter_key(uint64_t sig) { return (uint32_t)(sig - kFragInit); }

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

// Persistent grid of one block per CU. Task t is windows [1024t, 1024t + 1024);
// hit word 16t + m has bit b for window 64(16t + m) + b, and each hit's table
// slot goes to hit_slot[window]. Lane l takes windows 16l..16l+15 of a task,
// rolled by
//   H(j+1) = H(j) 33^4 - 33^64 D(j) + D(j+16)        (mod 2^64)
// from Horner over the first window's words: the lookups lie in lanes side by
// side, and the candidates' full signatures come from words in registers.
// What bounds it is the chain of a task (words, keys, first filter, second
// filter) at the 4 waves per SIMD that the filter leaves: the 540 M windows of the
// logos image in 0.957 ms, 2.2 TB/s (500 files 0.612, 120 files 0.617), 16 MiB in
// 15.2 us, zeros that all match 256 MiB in 472 us. So the second filter's words of
// a lane's 16 windows are all requested together, whether a window passed the
// first or not (those that failed read one word): reading them for all windows or
// none of a wave took 1.10 ms and 31.8 instead of 22.4 us at 32 MiB. The block's
// waves claim its tasks: with a fixed share each, 1.035 ms, because the hardware
// favours a block's older waves. Keys by matrix instructions, with the candidates
// between the filters gathered in LDS, take fewer instructions and fewer requests
// but add steps to the chain: 1.01 ms, 28 us at 32 MiB, 522 us for the zeros.
// Requesting a task's words ahead was slower too: loads return in order, so the
// next task's words hold up this one's filter words.
constexpr uint32_t kRolled = kWaveWindows / kWave;   // windows of a lane, and its own dwords
constexpr uint64_t kRollAdd = kFragInit - kFragInit * kPow4;          // mod 2^64
constexpr uint64_t kNegPow64 = 0ull - pow33(kFragBytes);              // mod 2^64
template <bool kBloom>
__global__ __launch_bounds__(kFragThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_frag_scan(
    const uint32_t* __restrict__ image, uint64_t n_windows, uint64_t n_dwords, IndexView ix,
    uint64_t* __restrict__ out, uint32_t* __restrict__ hit_slot) {
  __shared__ __attribute__((aligned(16))) uint32_t lfilter[kLdsFilterMaxWords];
  __shared__ uint32_t claimed;
  if (threadIdx.x == 0) claimed = kFragWaves;
  const uint32_t lw = ix.lds_words;   // at most kLdsFilterMaxWords, a multiple of 4
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const uint32_t l = lane_id();
  for (uint32_t i = 4 * threadIdx.x; i < lw; i += 4 * kFragThreads)
    *(u32x4*)(lfilter + i) = *(const u32x4*)(ix.lds_filter + i);
  __syncthreads();
  const uint64_t n_tasks = (n_windows + kWaveWindows - 1) / kWaveWindows;
  // The block's tasks in rounds of one per wave: a wave takes its own of the
  // first round, then claims the block's next.
  for (uint32_t k = wv;;) {
    const uint64_t t = ((uint64_t)(k / kFragWaves) * gridDim.x + blockIdx.x) * kFragWaves + k % kFragWaves;
    if (t >= n_tasks) break;
    uint32_t next = 0;
    if (l == 0) next = atomicAdd(&claimed, 1u);
    const uint64_t first = t * kWaveWindows;
    const uint64_t j0 = first + (uint64_t)l * kRolled;
    // the lane's own dwords and, in lanes 0-15, the first of the next task (which
    // lane 63's windows reach); clamped to the image's
    // last dword in its last task (only windows past the end read that)
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
      h[w] = s;
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
    k = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
  }
}

}  // namespace carve
