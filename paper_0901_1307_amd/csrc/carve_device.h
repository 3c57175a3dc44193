// Device-side building blocks of the carving scan for gfx950 (wave64).
//
// Signature: djb2 with a 64-bit accumulator (Eq. (1), Section 2.2; 64-bit
// accumulator, Section 4). The recurrence is linear modulo 2^64, so for a
// 512-byte sector s_0..s_511 it unrolls to
//     h = 5381*33^512 + sum_b s_b * 33^(511-b)            (mod 2^64),
// a contraction of the sector's bytes with 512 constants, done on the matrix
// cores in 8-bit integers (djb2_phase). Each weight 33^(511-b) mod 2^64 is
// split into 8 signed base-256 digits and each byte is taken as s_b - 128 (one
// xor of four bytes; the 128s go into the constant), so digit plane q gives
//     acc_q = sum_b (s_b - 128) * digit_q(33^(511-b)),   |acc_q| <= 2^23,
// exactly, in 32 bits, and h = const + sum_q acc_q << 8q.
//
// A wave hashes a tile of 64 sectors and ends with one sector per lane, like
// the paper's cohorts (Section 3.2) but 64 wide. The CRC (below) is a serial
// chain over a sector's bytes instead: there each lane runs its own sector,
// handed to it through a per-wave LDS staging area with a padded row pitch
// (the job Fig. 9's skewed tile did for a 16-bank shared memory).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace carve {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_dw __attribute__((ext_vector_type(4), aligned(4)));   // from 4-byte boundaries
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kSectorBytes = 512;
constexpr uint32_t kClusterSectors = 8;
constexpr uint32_t kWave = 64;
constexpr uint32_t kTileSectors = 64;                       // one sector per lane
constexpr uint32_t kPhaseBytes = 128;                       // the CRC: bytes per sector staged at once
constexpr uint32_t kRowPitch = kPhaseBytes + 16;            // padding spreads rows over banks
constexpr uint32_t kTileLds = kTileSectors * kRowPitch;     // 9216 B per wave
constexpr uint32_t kBucketSlots = 16;                       // 16 x 8 B keys = one 128-B line
constexpr uint64_t kEmptyKey = 0;                           // a real signature 0 lives in a side slot
constexpr uint64_t kBucketMul = 0x9E3779B97F4A7C15ull;      // Fibonacci hashing of the signature

// ---------------------------------------------------------------- weights
constexpr uint64_t pow33(uint32_t e) {
  uint64_t r = 1, b = 33;
  while (e) {
    if (e & 1u) r *= b;
    b *= b;
    e >>= 1;
  }
  return r;
}

// 5381*33^512 and 128 times the sum of all weights (the bytes enter as s - 128).
constexpr uint64_t djb2_constant() {
  uint64_t c = 5381ull * pow33(kSectorBytes), w = 1;
  for (uint32_t b = 0; b < kSectorBytes; ++b, w *= 33) c += 128ull * w;
  return c;   // wraps modulo 2^64
}
constexpr uint64_t kDjb2Constant = djb2_constant();

// Signed base-256 digit q of w, in [-128, 127] (modulo 2^64: the carry out of
// the last digit is dropped).
constexpr int32_t signed_digit(uint64_t w, uint32_t q) {
  int32_t d = 0;
  for (uint32_t i = 0; i <= q; ++i) {
    d = (int32_t)(w & 0xFFu);
    if (d > 127) d -= 256;
    w = (w - (uint64_t)(int64_t)d) >> 8;
  }
  return d;
}

// The weights as the matrix instruction's right operand (64 bytes deep, 16
// columns), as each lane holds it: lane l has column n = l mod 16, depth
// 16(l/16)..16(l/16)+15. A row of the left operand is the 16-byte pieces j, j +
// 4, j + 8 and j + 12 of half a sector (256 bytes; j = 0..3), so one row's
// weights are those of another times a power of 33 and need columns of their
// own: columns 0-7 are the digit planes for one j, columns 8-15 for another,
// in two operands: set 0 for j = 3 and 2, set 1 for j = 1 and 0.
struct Djb2Weights {
  uint32_t w[2][2][kWave][4];   // [set][half of the sector][lane][dword]
};
constexpr Djb2Weights make_djb2_weights() {
  Djb2Weights t{};
  for (uint32_t set = 0; set < 2; ++set)
    for (uint32_t half = 0; half < 2; ++half)
      for (uint32_t l = 0; l < kWave; ++l) {
        const uint32_t j = 3u - 2u * set - ((l >> 3) & 1u), q = l & 7u;
        uint64_t w = pow33(kSectorBytes - 1 - (256u * half + 64u * (l >> 4) + 16u * j + 15u));
        for (uint32_t b = 16; b-- > 0; w *= 33)
          t.w[set][half][l][b / 4] |= (uint32_t)(signed_digit(w, q) & 0xFF) << (8 * (b % 4));
      }
  return t;
}
__device__ const Djb2Weights g_djb2_weights = make_djb2_weights();

// ------------------------------------------------------------ static for
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ uint32_t lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, uint32_t src) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  lo = (uint32_t)__shfl((int)lo, (int)src, kWave);
  hi = (uint32_t)__shfl((int)hi, (int)src, kWave);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Byte g of x non-zero -> bit g of the result (x is wave-uniform): fold each
// byte onto its low bit, then gather bits 0, 8, ..., 56 with one multiply
// (the partial products land on distinct bits, so nothing carries).
__device__ __forceinline__ uint32_t bytes_nonzero(uint64_t x) {
  x |= x >> 4;
  x |= x >> 2;
  x |= x >> 1;
  x &= 0x0101010101010101ull;
  return (uint32_t)((x * 0x0102040810204080ull) >> 56);
}

// ------------------------------------------------------------ tile hash
// Sector addresses of a tile: sector s is base + s*512; sectors past n_valid
// are replaced by the last valid one (their hash is discarded), so every load
// stays inside the image without a branch.
struct ContiguousRows {
  const uint8_t* base;
  uint32_t n_valid;   // 1..64
  __device__ __forceinline__ uint32_t offset(uint32_t s) const {
    return (s < n_valid ? s : n_valid - 1) * kSectorBytes;
  }
  __device__ __forceinline__ const uint8_t* row(uint32_t s) const { return base + offset(s); }
};
// A tile of one cluster position: sector s is base + s*4096 (the same
// position in 64 consecutive clusters); past n_valid, the last valid one.
struct ClusterStrideRows {
  const uint8_t* base;
  uint32_t n_valid;   // 1..64
  __device__ __forceinline__ uint32_t offset(uint32_t s) const {
    return (s < n_valid ? s : n_valid - 1) * (kClusterSectors * kSectorBytes);
  }
  __device__ __forceinline__ const uint8_t* row(uint32_t s) const { return base + offset(s); }
};

template <bool kNonTemporal>
__device__ __forceinline__ u32x4 load16(const uint8_t* p) {
  if constexpr (kNonTemporal) return __builtin_nontemporal_load((const u32x4*)p);
  else return *(const u32x4*)p;
}

// Phase p of a tile for the CRC: instruction i, lane l loads 16 B of sector 8i + l/8 at
// byte 128p + 16(l%8); one instruction covers 8 whole 128-byte lines.
struct PhaseRegs {
  u32x4 v[8];
};

template <bool kNonTemporal, class Rows>
__device__ __forceinline__ void load_phase(const Rows& rows, uint32_t p, PhaseRegs& r) {
  const uint32_t l = lane_id();
#pragma unroll
  for (int i = 0; i < 8; ++i) r.v[i] = load16<kNonTemporal>(rows.row(8u * i + (l >> 3)) + p * kPhaseBytes + (l & 7u) * 16u);
}

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// Sixteen sectors of a tile for the matrix path, sectors 16p..16p+15, 8 KiB:
// load 2g + half is 256 bytes of the sectors 16p + 4g + 0..3. Lane l takes
// sector (l/4) mod 4, its 16-byte piece 4(l/16) + l mod 4: each four
// neighbouring lanes read 64 contiguous bytes, an instruction 8 whole 128-byte
// lines, and the lane's bytes are already where the matrix instruction wants
// them (row l mod 16, depth l/16), so nothing goes through LDS.
template <bool kNonTemporal, class Rows>
__device__ __forceinline__ void load_sectors(const Rows& rows, uint32_t p, PhaseRegs& r) {
  const uint32_t l = lane_id();
  const uint32_t at = (l >> 4) * 64u + (l & 3u) * 16u;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    // a 32-bit lane offset from the tile's uniform base: no 64-bit address per load
    const uint8_t* q = rows.base + (rows.offset(16u * p + 4u * g + ((l >> 2) & 3u)) + at);
    r.v[2 * g] = load16<kNonTemporal>(q);
    r.v[2 * g + 1] = load16<kNonTemporal>(q + 256);
  }
}

// This lane's part of the weights.
struct Djb2Lane {
  i32x4 w[2][2];   // [set][half]
};
__device__ __forceinline__ void load_djb2_lane(Djb2Lane& d, uint32_t l = lane_id()) {
#pragma unroll
  for (int set = 0; set < 2; ++set)
#pragma unroll
    for (int half = 0; half < 2; ++half) d.w[set][half] = *(const i32x4*)g_djb2_weights.w[set][half][l];
}

// DPP controls: each lane takes the value of another lane of its 16.
constexpr int kDppXor1 = 0xB1;    // quad_perm 1,0,3,2
constexpr int kDppXor2 = 0x4E;    // quad_perm 2,3,0,1
constexpr int kDppXor7 = 0x141;   // row_half_mirror
constexpr int kDppXor8 = 0x128;   // row_ror 8
template <int kCtrl>
__device__ __forceinline__ int32_t dpp(int32_t v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xF, 0xF, true);
}
template <int kCtrl>
__device__ __forceinline__ uint64_t dpp(uint64_t v) {
  const uint32_t lo = (uint32_t)dpp<kCtrl>((int32_t)(uint32_t)v), hi = (uint32_t)dpp<kCtrl>((int32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}
// One step of a sum over lanes that also deals the values out: a lane keeps a
// (lower) or b (upper, its partner), with the partner's added.
template <int kCtrl, class T>
__device__ __forceinline__ T deal_sum(T a, T b, bool upper) {
  const T keep = upper ? b : a, send = upper ? a : b;
  return keep + dpp<kCtrl>(send);
}

// Four sectors, two loads: the digit plane l mod 8 of sector l/16, over the
// sector's pieces with one parity of j (lanes 0-7 of each 16 the odd ones,
// lanes 8-15 the even ones).
__device__ __forceinline__ int32_t djb2_planes(const u32x4& r0, const u32x4& r1, const Djb2Lane& d, bool upper) {
  const u32x4 flip = {0x80808080u, 0x80808080u, 0x80808080u, 0x80808080u};
  const i32x4 a0 = (i32x4)(r0 ^ flip), a1 = (i32x4)(r1 ^ flip);
  i32x4 x = {0, 0, 0, 0}, y = {0, 0, 0, 0};
  x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, d.w[0][0], x, 0, 0, 0);
  y = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, d.w[1][0], y, 0, 0, 0);
  x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, d.w[0][1], x, 0, 0, 0);
  y = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, d.w[1][1], y, 0, 0, 0);
  // the result's element j of this lane is row 4(l/16) + j: sector l/16, pieces j
  return (upper ? x[2] : x[3]) + (upper ? y[0] : y[1]);
}

// Sixteen sectors (load_sectors): the planes' sums over the two lane pairs
// l, l ^ 8 and l, l ^ 7, which leave a lane with one group of four sectors, the
// one that l's bits 3 and 2 number; what is left to add are the lanes l ^ 1 and
// l ^ 2.
__device__ __forceinline__ uint64_t djb2_phase(const PhaseRegs& r, const Djb2Lane& d) {
  __builtin_amdgcn_sched_barrier(0);   // the loads issued before this call stay above it
  const uint32_t l = lane_id();
  const bool b3 = (l & 8u) != 0, b2 = (l & 4u) != 0;
  uint64_t h[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int32_t lower = djb2_planes(r.v[2 * i], r.v[2 * i + 1], d, b3);
    const int32_t upper = djb2_planes(r.v[2 * i + 4], r.v[2 * i + 5], d, b3);
    h[i] = (uint64_t)(int64_t)deal_sum<kDppXor8>(lower, upper, b3) << (8u * (l & 7u));
    __builtin_amdgcn_sched_barrier(0);   // two groups' results in registers at a time
  }
  return deal_sum<kDppXor7>(h[0], h[1], b2);
}

// Signature of every sector of a tile (lane l = sector l), sixteen after
// sixteen from the one that `first` numbers on and round. A and B are the two
// register buffers of the load pipeline: on entry A holds (or is receiving) the
// first sixteen; the next are requested before these are hashed, and `prefetch`
// (called before the last are hashed) may start the next tile's first into A.
// The waves of a block begin with different sixteens: with all of them reading
// the first 8 KiB of their 32 KiB tiles at the same time, then the second, fewer
// of the memory's channels are busy at once (4 blocks a CU: 256 MiB 47.7 us, and
// 46.0 so).
template <bool kNonTemporal, class Rows, class Prefetch>
__device__ __forceinline__ uint64_t tile_djb2_pipelined(const Rows& rows, const Djb2Lane& d, uint32_t first,
                                                        PhaseRegs& A, PhaseRegs& B, Prefetch&& prefetch) {
  const uint32_t l = lane_id();
  const bool b0 = (l & 1u) != 0, b1 = (l & 2u) != 0;
  load_sectors<kNonTemporal>(rows, (first + 1u) & 3u, B);
  const uint64_t h0 = djb2_phase(A, d);
  load_sectors<kNonTemporal>(rows, (first + 2u) & 3u, A);
  const uint64_t x = deal_sum<kDppXor1>(h0, djb2_phase(B, d), b0);
  load_sectors<kNonTemporal>(rows, (first + 3u) & 3u, B);
  const uint64_t h2 = djb2_phase(A, d);
  prefetch(A);
  const uint64_t y = deal_sum<kDppXor1>(h2, djb2_phase(B, d), b0);
  // the lane that sector l's sum ends in: sector 16p + 4g + k in lane 16k + 4g + (p's place in the order)
  const uint32_t from = 16u * (l & 3u) + (l & 12u) + (((l >> 4) - first) & 3u);
  return shfl_u64(deal_sum<kDppXor2>(x, y, b1), from) + kDjb2Constant;
}

// Signatures of sixteen sectors held in r (lane l: sector l mod 16).
__device__ __forceinline__ uint64_t sixteen_djb2(const PhaseRegs& r, const Djb2Lane& d) {
  uint64_t h = djb2_phase(r, d);
  h += dpp<kDppXor1>(h);
  h += dpp<kDppXor2>(h);
  const uint32_t l = lane_id();
  return shfl_u64(h, 16u * (l & 3u) + (l & 12u)) + kDjb2Constant;
}

// ---------------------------------------------------------------- CRC-64
// The other signature of Section 2.1: a 64-bit CRC, read as CRC-64/GO-ISO
// (generator x^64 + x^4 + x^3 + x + 1, bytes entering least significant bit
// first, register preset to all ones, result complemented).
//
// No table: this generator lets the register absorb a 32-bit word with shifts
// and xors. In the right-shifting (reflected) register a feedback term enters
// at bit 59 or above, so within any 32 steps the bits tested are exactly the
// input bits. Absorbing the little-endian word d (bytes in address order) is
// then, with x = crc ^ d and u = x mod 2^32,
//   crc' = (x >> 32) ^ (u << 28) ^ (u << 29) ^ (u << 31) ^ (u << 32),
// x >> 32 xor the carry-less product of u with the generator's terms below x^64
// (0x1B: bits 0, 1, 3, 4), placed 28 bits up. About 11 VALU operations per word.
enum : int { kSigDjb2 = 0, kSigCrc64 = 1 };   // the values of carve_sig_kind

// The same, on the register's 32-bit halves (full-rate 32-bit shifts):
// the low half becomes hi ^ u<<28 ^ u<<29 ^ u<<31, the high half
// u ^ u>>1 ^ u>>3 ^ u>>4 (the bits the 64-bit shifts carry across).
// a ^ b ^ c in one instruction: gfx950's three-input bit operation with the
// truth table of xor3 (0x96: set where an odd number of inputs is set).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ void crc_word(uint32_t& lo, uint32_t& hi, uint32_t d) {
  const uint32_t u = lo ^ d;
  lo = xor3(hi, u << 28, u << 29) ^ (u << 31);
  hi = xor3(u, u >> 1, u >> 3) ^ (u >> 4);
}

// Stage a phase through this wave's LDS area, then run lane l's register over
// the 128 bytes of its sector, in address order.
__device__ __forceinline__ void crc_phase(const PhaseRegs& r, uint8_t* lds, uint32_t& lo, uint32_t& hi) {
  __builtin_amdgcn_sched_barrier(0);
  const uint32_t l = lane_id();
  const uint32_t col = (l & 7u) * 16u;
#pragma unroll
  for (int i = 0; i < 8; ++i) *(u32x4*)(lds + (8u * i + (l >> 3)) * kRowPitch + col) = r.v[i];
  wave_sync_lds();
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const u32x4 x4 = *(const u32x4*)(lds + l * kRowPitch + c * 16);
#pragma unroll
    for (int k = 0; k < 4; ++k) crc_word(lo, hi, x4[k]);
  }
  asm volatile("" : "+v"(lo), "+v"(hi));
  wave_sync_lds();
  __builtin_amdgcn_sched_barrier(0);
}

// CRC-64 of every sector of a tile, with the same load pipeline as the djb2 path.
template <bool kNonTemporal, class Rows, class Prefetch>
__device__ __forceinline__ uint64_t tile_crc_pipelined(const Rows& rows, uint8_t* lds, PhaseRegs& A, PhaseRegs& B,
                                                       Prefetch&& prefetch) {
  uint32_t lo = ~0u, hi = ~0u;   // preset: all ones
  load_phase<kNonTemporal>(rows, 1, B);
  crc_phase(A, lds, lo, hi);
  load_phase<kNonTemporal>(rows, 2, A);
  crc_phase(B, lds, lo, hi);
  load_phase<kNonTemporal>(rows, 3, B);
  crc_phase(A, lds, lo, hi);
  prefetch(A);
  crc_phase(B, lds, lo, hi);
  return ~(((uint64_t)hi << 32) | lo);   // complemented
}

// ---------------------------------------------------------------- index
struct IndexView {
  const uint64_t* keys;      // n_buckets * 16 slots, kEmptyKey = free
  const uint8_t* tau_mask;   // per slot, bit t = a master with this signature sits at position t
  const uint64_t* bloom;     // blocked Bloom filter of the table's keys, or null
  uint32_t log2_buckets;
  uint32_t log2_bloom_words;
  uint32_t zero_sig_mask;    // positions of signature 0, which has no slot in the table
  uint32_t zero_slot;        // candidate-list id of signature 0 (= number of table slots)
  // other probe layouts, mapping a signature to its slot of the table above
  const uint64_t* lin_keys;  // linear probing per slot from the signature's low bits: 2^log2_lin keys
  const uint32_t* lin_slot;  //   and the table slot of each
  uint32_t log2_lin;
  uint32_t n_sorted;         // sorted distinct signatures (binary search)
  const uint64_t* sorted_keys;
  const uint32_t* sorted_slot;
  const uint32_t* lds_filter;  // fragment indexes: the first-level filter copied into LDS (lds_words words)
  uint32_t lds_words;
  // sector indexes: the Bloom filter split by cluster position, slice t (2^log2_bloom_tau
  // words at bloom_tau + t 2^log2_bloom_tau) holding the keys present at position t; or null
  const uint64_t* bloom_tau;
  uint32_t log2_bloom_tau;
};

// Probe layouts (the values of carve_index_layout).
enum : int { kLayoutBucketed = 0, kLayoutLinear = 1, kLayoutSorted = 2 };

// Register-blocked Bloom filter: a key owns one 64-bit word and sets 4 of
// its bits. Word and bit positions come from the high half of a second
// multiplicative hash (djb2's low bits are weak: 33 = 1 mod 32).
// log2_words must be in 1..40: the word index is a shift by 64 - log2_words,
// and a shift by 64 is not a shift by 64 on this chip (its amount is taken
// mod 64), so a one-word filter would index far past its end.
constexpr uint64_t kBloomMul = 0xD6E8FEB86659FD93ull;
__device__ __forceinline__ void bloom_place(uint64_t h, uint32_t log2_words, uint32_t* word, uint64_t* bits) {
  const uint64_t p = h * kBloomMul;
  *word = (uint32_t)(p >> (64 - log2_words));
  const uint32_t f = (uint32_t)(p >> (40 - log2_words));   // 24 bits below the word index
  *bits = (1ull << (f & 63)) | (1ull << ((f >> 6) & 63)) | (1ull << ((f >> 12) & 63)) | (1ull << ((f >> 18) & 63));
}

__device__ __forceinline__ uint32_t bucket_of(uint64_t h, uint32_t log2_buckets) {
  return (uint32_t)((h * kBucketMul) >> (64 - log2_buckets));
}

// Slot of key h (h != kEmptyKey) or -1. Linear probing over buckets: a key
// lives in its home bucket or, if that bucket filled up first, a later one
// (Eq. (3) at bucket granularity); a bucket with a free slot ends the search.
// A bucket is read as two 64-byte halves in turn: k_insert claims a bucket's
// slots in order (and nothing is ever removed), so the occupied slots are a
// prefix of it and a free slot in the first half ends the search there (about
// 91% of the buckets of a fragment index, half of a sector index's at its
// fullest). A whole bucket at once costs 16 more registers, which the scans
// would spill.
__device__ __forceinline__ int64_t find_slot(const IndexView& ix, uint64_t h) {
  constexpr uint32_t kHalf = kBucketSlots / 2;
  const uint32_t nb_mask = (1u << ix.log2_buckets) - 1u;
  uint32_t b = bucket_of(h, ix.log2_buckets);
  for (uint32_t it = 0; it <= nb_mask; ++it) {
#pragma unroll
    for (uint32_t half = 0; half < 2; ++half) {
      const uint64_t first = (uint64_t)b * kBucketSlots + half * kHalf;
      const u64x2* p = (const u64x2*)(ix.keys + first);
      u64x2 kv[kHalf / 2];
#pragma unroll
      for (int c = 0; c < (int)(kHalf / 2); ++c) kv[c] = p[c];
      int64_t found = -1;
      bool any_empty = false;
#pragma unroll
      for (int c = 0; c < (int)(kHalf / 2); ++c) {
        if (kv[c].x == h) found = (int64_t)(first + 2 * c);
        if (kv[c].y == h) found = (int64_t)(first + 2 * c + 1);
        any_empty |= (kv[c].x == kEmptyKey) | (kv[c].y == kEmptyKey);
      }
      if (found >= 0) return found;
      if (any_empty) return -1;
    }
    b = (b + 1) & nb_mask;
  }
  return -1;
}

// The paper's layout (Eq. (3)): home slot = the w low bits of the signature,
// then the next slots in turn until the key or a free slot. Returns the
// table slot or -1.
__device__ __forceinline__ int64_t find_slot_linear(const IndexView& ix, uint64_t h) {
  const uint64_t mask = (1ull << ix.log2_lin) - 1ull;
  uint64_t s = h & mask;
  for (uint64_t it = 0; it <= mask; ++it) {
    const uint64_t k = ix.lin_keys[s];
    if (k == h) return (int64_t)ix.lin_slot[s];
    if (k == kEmptyKey) return -1;
    s = (s + 1) & mask;
  }
  return -1;
}

// Sorted distinct signatures: lower bound by halving with no data-dependent
// branch (every lane takes the same ceil(log2 n) steps). Returns the table
// slot or -1.
__device__ __forceinline__ int64_t find_slot_sorted(const IndexView& ix, uint64_t h) {
  uint64_t base = 0, n = ix.n_sorted;
  if (n == 0) return -1;
  while (n > 1) {
    const uint64_t half = n >> 1;
    base = ix.sorted_keys[base + half] <= h ? base + half : base;
    n -= half;
  }
  return ix.sorted_keys[base] == h ? (int64_t)ix.sorted_slot[base] : -1;
}

template <int kLayout>
__device__ __forceinline__ int64_t find_slot_in(const IndexView& ix, uint64_t h) {
  if constexpr (kLayout == kLayoutLinear) return find_slot_linear(ix, h);
  else if constexpr (kLayout == kLayoutSorted) return find_slot_sorted(ix, h);
  else return find_slot(ix, h);
}

__device__ __forceinline__ bool tau_ok(uint32_t mask, uint32_t tau, bool any_tau) {
  return any_tau ? (mask != 0) : (((mask >> tau) & 1u) != 0);
}

// Membership of the 64 lane signatures. With a Bloom filter (kept small
// enough to stay in L2): one 8-byte filter word per sector, and only the
// sectors that pass probe the table, each lane its own. Without one: a
// cooperative probe in which, in round r, the 8 lanes of group g read the
// 128-byte home bucket of sector 8r+g (16 B each) and its 16 position masks
// (2 B each); all 16 loads are issued before any is used, so the tile pays
// one memory latency. Returns the tile's hit mask (bit l = sector l); tau is
// this lane's cluster position. For each hit, the slot that matched is
// stored in slot_out[sector * kSlotStride] (the candidate list that
// confirmation walks; the stride is 8 for a tile of one cluster position).
// The linear and sorted layouts probe lane by lane, after the filter if there
// is one.
// bloom / log2_bloom: the filter to consult (the index's, or one position's
// slice of it), or null. kSlots = false records no slots (slot_out unused),
// for scans whose flags are not confirmed afterwards. kFiltered: there always
// is a filter (the cooperative probe's registers are not needed). kSectors: 64,
// or 16 with lane l holding sector l mod 16 (all four lanes of a sector write
// the same slot, and the mask's bits 16 and above repeat).
template <int kLayout = kLayoutBucketed, uint32_t kSlotStride = 1, bool kSlots = true, bool kFiltered = false,
          uint32_t kSectors = kTileSectors>
__device__ __forceinline__ uint64_t tile_probe(const IndexView& ix, uint64_t h, uint32_t tau, bool any_tau,
                                               uint32_t* __restrict__ slot_out, const uint64_t* bloom,
                                               uint32_t log2_bloom) {
  const uint32_t l = lane_id();
  const uint32_t own = l % kSectors;   // this lane's sector
  // signature 0 cannot be stored in the table (it marks free slots)
  const bool ok_zero = (h == kEmptyKey) && tau_ok(ix.zero_sig_mask, tau, any_tau);
  if (kSlots && ok_zero) slot_out[own * kSlotStride] = ix.zero_slot;
  if (kLayout != kLayoutBucketed || kFiltered || bloom) {
    bool maybe = h != kEmptyKey;
    if (kFiltered || bloom) {
      uint32_t w;
      uint64_t bits;
      bloom_place(h, log2_bloom, &w, &bits);
      maybe = maybe && (bloom[w] & bits) == bits;
    }
    bool ok = false;
    if (maybe) {
      const int64_t slot = find_slot_in<kLayout>(ix, h);
      ok = slot >= 0 && tau_ok(ix.tau_mask[slot], tau, any_tau);
      if (kSlots && ok) slot_out[own * kSlotStride] = (uint32_t)slot;
    }
    return ballot(ok) | ballot(ok_zero);
  }
  const uint32_t bkt = bucket_of(h, ix.log2_buckets);
  // per round: the bucket's slots 2(l%8), 2(l%8)+1 and their masks
  constexpr int kRounds = (int)kSectors / 8;
  u64x2 kv[kRounds];
  uint32_t mk[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint32_t s = 8u * r + (l >> 3);
    const uint32_t slot0 = (uint32_t)__shfl((int)bkt, (int)s, kWave) * kBucketSlots + 2u * (l & 7u);
    kv[r] = *(const u64x2*)(ix.keys + slot0);
    mk[r] = *(const uint16_t*)(ix.tau_mask + slot0);
  }
  uint64_t hits = 0, unresolved = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    // the round's sector, fetched again rather than kept live across the loads
    const uint32_t s = 8u * r + (l >> 3);
    const uint64_t hs = shfl_u64(h, s);
    const uint32_t ts = (uint32_t)__shfl((int)tau, (int)s, kWave);
    const bool live = hs != kEmptyKey;
    const bool m0 = live && kv[r].x == hs;
    const bool m1 = live && kv[r].y == hs;
    const bool empty = !live || kv[r].x == kEmptyKey || kv[r].y == kEmptyKey;
    const uint32_t mask = m0 ? (mk[r] & 0xFFu) : (mk[r] >> 8);
    const bool ok = (m0 | m1) && tau_ok(mask, ts, any_tau);
    // cross-lane reads only with every lane active: lane s may be idle inside `if (ok)`
    const uint32_t slot0 = (uint32_t)__shfl((int)bkt, (int)s, kWave) * kBucketSlots + 2u * (l & 7u);
    if (kSlots && ok) slot_out[s * kSlotStride] = slot0 + (m1 ? 1u : 0u);
    hits |= (uint64_t)bytes_nonzero(ballot(ok)) << (8 * r);
    unresolved |= (uint64_t)(~bytes_nonzero(ballot(m0 | m1 | empty)) & 0xFFu) << (8 * r);
  }
  // rare: the home bucket was full and did not hold the key
  bool ok_more = false;
  if ((unresolved >> own) & 1u) {
    const int64_t slot = find_slot(ix, h);
    ok_more = slot >= 0 && tau_ok(ix.tau_mask[slot], tau, any_tau);
    if (kSlots && ok_more) slot_out[own * kSlotStride] = (uint32_t)slot;
  }
  return hits | ballot(ok_more) | ballot(ok_zero);
}

// -------------------------------------------------------- block scans
// Exclusive prefix sum over a 256-thread block; returns this thread's prefix
// and writes the block total to *total (all threads).
template <int kThreads>
__device__ __forceinline__ uint64_t block_exclusive_scan(uint64_t v, uint64_t* lds_w, uint64_t* total) {
  const uint32_t l = lane_id();
  const uint32_t w = threadIdx.x / kWave;
  uint64_t x = v;
#pragma unroll
  for (int o = 1; o < (int)kWave; o <<= 1) {
    const uint64_t y = shfl_u64(x, l >= (uint32_t)o ? l - o : l);
    if (l >= (uint32_t)o) x += y;
  }
  if (l == kWave - 1) lds_w[w] = x;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kThreads / (int)kWave; ++i) {
    const uint64_t t = lds_w[i];
    before += (i < (int)w) ? t : 0;
    all += t;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

}  // namespace carve
