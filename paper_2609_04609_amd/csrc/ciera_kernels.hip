// CIERA codec kernels for CDNA4 (gfx950).
//
// Everything here is integer byte manipulation on HBM-resident streams; the
// roofline is HBM bandwidth, so the kernels are built around wide coalesced
// accesses (16-byte bf16 loads, 8-byte exponent / sign+mantissa accesses per
// lane), whole-tile load batches, and wave64 ballots for the per-block
// reductions. No MFMA: nothing here is a contraction.
//
// Algorithm 1 (appendix of the paper) as kernels:
//   encode   (1) encode_pass_kernel: SplitExpMant, change detection, the
//                sign+mantissa plane, the bitmap and a changed-block count
//                per tile, streaming at copy speed;
//            (2) the exponents of the changed blocks, in block order, read
//                back for those blocks only (from the cache pass 1 brought
//                forward with the fused cache update, else from W'), and
//                the header: encode_exc_blocks_kernel (B = 16 ... 256, lanes
//                over the changed blocks), encode_exc_rows_kernel (B >= 512,
//                over the changed 512-value rows), encode_exc_elems_kernel
//                (B = 1). A workgroup finds its first exception by counting
//                the bitmap bits in front of it (the bitmap is 1/(8B) of the
//                shard and stays in L2), or at B = 1 by adding up pass 1's
//                per-tile counts in front of it; where either would re-read
//                too much, a scan_counts_kernel over those counts stands in.
//            No workgroup ever waits on another: compacting the exception
//            list costs one re-read of the changed blocks (1 or 2 bytes per
//            changed value) instead of a cross-workgroup scan whose waits
//            would hold every tile's slot behind its slowest predecessor.
//            Small shards take encode_small_kernel instead: one workgroup, one
//            launch.
//   decode   for all R gathered shards at once: ExpCache patch + Merge. Each
//            tile finds its first exception by counting the bitmap bits in
//            front of it (the bitmap is 1/(8B) of the shard and stays in L2),
//            so decode tiles never wait on each other. At B = 1 a count
//            kernel takes every tile's bitmap bits first, and each tile adds
//            up the counts in front of it (or, past 128 MB of such reads, a
//            scan of the counts runs in between). Small layers take smaller
//            tiles and one kernel at every B (dec_small).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ciera.h"
#include "ciera_internal.h"

namespace ciera {

namespace {

// ------------------------------------------------------------ bit packing --
// Four bf16 values held as two 32-bit words (a: values 0,1; b: values 2,3)
// become four exponent bytes and four sign|mantissa bytes.
__device__ __forceinline__ void split4(uint32_t a, uint32_t b, uint32_t &e,
                                       uint32_t &sm) {
  const uint32_t hi = __builtin_amdgcn_perm(b, a, 0x07050301u);
  const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x06040200u);
  e = ((hi << 1) & 0xFEFEFEFEu) | ((lo >> 7) & 0x01010101u);
  sm = (hi & 0x80808080u) | (lo & 0x7F7F7F7Fu);
}

// Inverse of split4.
__device__ __forceinline__ void merge4(uint32_t e, uint32_t sm, uint32_t &a,
                                       uint32_t &b) {
  const uint32_t hi = (sm & 0x80808080u) | ((e >> 1) & 0x7F7F7F7Fu);
  const uint32_t lo = ((e << 7) & 0x80808080u) | (sm & 0x7F7F7F7Fu);
  a = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
  b = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
}

// fp16 (sign bit 15, exponent bits 14..10, mantissa bits 9..0): four values
// (a: values 0,1; b: values 2,3) become four 5-bit exponents, four low
// mantissa bytes and four (sign << 2 | mantissa bits 9..8) fields.
__device__ __forceinline__ void split4_f16(uint32_t a, uint32_t b, uint32_t &e,
                                           uint32_t &lo, uint32_t &hi3) {
  const uint32_t hb = __builtin_amdgcn_perm(b, a, 0x07050301u);
  lo = __builtin_amdgcn_perm(b, a, 0x06040200u);
  e = (hb >> 2) & 0x1F1F1F1Fu;
  hi3 = ((hb >> 5) & 0x04040404u) | (hb & 0x03030303u);
}

// Inverse of split4_f16.
__device__ __forceinline__ void merge4_f16(uint32_t e, uint32_t lo,
                                           uint32_t hi3, uint32_t &a,
                                           uint32_t &b) {
  const uint32_t hb = ((hi3 & 0x04040404u) << 5) |
                      ((e & 0x1F1F1F1Fu) << 2) | (hi3 & 0x03030303u);
  a = __builtin_amdgcn_perm(hb, lo, 0x05010400u);
  b = __builtin_amdgcn_perm(hb, lo, 0x07030602u);
}

// Bit p of the eight byte fields of an octet (bytes of x: values 0..3, of
// y: 4..7) gathered into one byte, value k in bit k. The multiply moves the
// bit at 8i to 24 + i; no two partial products share a bit.
__device__ __forceinline__ uint32_t plane_byte(uint32_t x, uint32_t y,
                                               uint32_t p) {
  const uint32_t t0 = (x >> p) & 0x01010101u, t1 = (y >> p) & 0x01010101u;
  return ((t0 * 0x01020408u) >> 24) | (((t1 * 0x01020408u) >> 24) << 4);
}

// Bits 0..3 of x to bit 0 of bytes 0..3 (the inverse gather).
__device__ __forceinline__ uint32_t spread4(uint32_t x) {
  return ((x & 0xFu) * 0x00204081u) & 0x01010101u;
}

// Eight byte fields of an octet from Q plane bytes (byte q: bit q of value
// k in bit k), as two words (values 0..3, 4..7).
template <int Q>
__device__ __forceinline__ uint2 unplane(const uint8_t *g) {
  uint2 v = make_uint2(0u, 0u);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t b = g[q];
    v.x |= spread4(b) << q;
    v.y |= spread4(b >> 4) << q;
  }
  return v;
}

// ---------------------------------------------------- streaming accesses --
// Bytes that a call reads or writes once (the sign|mantissa plane, the
// exception list, the decoded values and the merge's cache patches, W' or
// the cache bytes pass 1 compares, whichever the exception pass does not
// read again) go through non-temporal loads and stores (the nt bit), so
// that they neither push out what is read again (the bitmap words every
// decode tile counts in front of it, what the exception pass re-reads) nor
// leave dirty lines in the Infinity Cache for the next kernel to write back.
// Plain stores of the merge's cache patches, for one, left up to 256 MB of
// them behind a DeepSeek-style decode: the encode after it took 131 instead
// of 84 us.
//
// The callers' buffers (W', caches, decoded values) may start anywhere: a
// shard of n values is a slice at j n of a flat buffer, and n need not be a
// multiple of 8. CDNA4 takes 8- and 16-byte global accesses at any address
// (the compiler emits the same single instruction for them), so every whole
// octet goes through these types, which promise no more than the element's
// own alignment. One kernel then serves every address: 12 shards of
// 34,963,798 values (encode and gathered decode, two iterations) take 768 us
// against 2232 us with element-wise accesses for n % 8 != 0, and aligned
// shards run as before (OLMoE layer encode 23.4 us either way).
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4), aligned(2)));

__device__ __forceinline__ uint2 ld_nt8(const uint8_t *p) {
  const u32x2_t x =
      __builtin_nontemporal_load(reinterpret_cast<const u32x2_t *>(p));
  return make_uint2(x.x, x.y);
}

__device__ __forceinline__ uint4 ld_nt16(const uint16_t *p) {
  const u32x4_t x =
      __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
  return make_uint4(x.x, x.y, x.z, x.w);
}

__device__ __forceinline__ void st_nt8(uint8_t *p, uint2 v) {
  const u32x2_t x = {v.x, v.y};
  __builtin_nontemporal_store(x, reinterpret_cast<u32x2_t *>(p));
}

__device__ __forceinline__ void st_nt16(uint16_t *p, uint4 v) {
  const u32x4_t x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<u32x4_t *>(p));
}

__device__ __forceinline__ uint2 ld8(const uint8_t *p) {
  const u32x2_t x = *reinterpret_cast<const u32x2_t *>(p);
  return make_uint2(x.x, x.y);
}

__device__ __forceinline__ uint4 ld16(const uint16_t *p) {
  const u32x4_t x = *reinterpret_cast<const u32x4_t *>(p);
  return make_uint4(x.x, x.y, x.z, x.w);
}

__device__ __forceinline__ void st8(uint8_t *p, uint2 v) {
  const u32x2_t x = {v.x, v.y};
  *reinterpret_cast<u32x2_t *>(p) = x;
}

__device__ __forceinline__ void st16(uint16_t *p, uint4 v) {
  const u32x4_t x = {v.x, v.y, v.z, v.w};
  *reinterpret_cast<u32x4_t *>(p) = x;
}

// ------------------------------------------------- octet loads and stores --
// `valid` is the number of in-range values of the octet (1..8); the ragged
// last octet of a shard goes element by element.
__device__ __forceinline__ uint4 load_w8(const uint16_t *p, uint32_t valid) {
  if (valid == 8) return ld16(p);
  uint32_t v[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i)
    if (i < valid) v[i >> 1] |= uint32_t(p[i]) << ((i & 1) * 16);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// load_w8 for the encode's second read of W' (non-temporal: its last use)
__device__ __forceinline__ uint4 reread_w8(const uint16_t *p, uint32_t valid) {
  if (valid == 8) return ld_nt16(p);
  return load_w8(p, valid);
}

__device__ __forceinline__ void store_w8(uint16_t *p, uint4 v,
                                         uint32_t valid) {
  if (valid == 8) {
    st16(p, v);
    return;
  }
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i)
    if (i < valid) p[i] = uint16_t(w[i >> 1] >> ((i & 1) * 16));
}

__device__ __forceinline__ uint2 load_b8(const uint8_t *p, uint32_t valid) {
  if (valid == 8) return ld8(p);
  uint32_t v[2] = {0u, 0u};
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i)
    if (i < valid) v[i >> 2] |= uint32_t(p[i]) << ((i & 3) * 8);
  return make_uint2(v[0], v[1]);
}

__device__ __forceinline__ void store_b8(uint8_t *p, uint2 v, uint32_t valid) {
  if (valid == 8) {
    st8(p, v);
    return;
  }
  const uint32_t w[2] = {v.x, v.y};
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i)
    if (i < valid) p[i] = uint8_t(w[i >> 2] >> ((i & 3) * 8));
}

__device__ __forceinline__ uint32_t octet_valid(uint64_t elem, uint64_t n) {
  return elem >= n ? 0u : (n - elem >= 8 ? 8u : uint32_t(n - elem));
}

// ------------------------------------------------------ wave/block sums ----
// Inclusive scan over the wave's 64 lanes with DPP moves (no LDS): shifts
// by 1, 2, 4 and 8 lanes inside each row of 16 (lanes shifted in from
// outside the row read 0), then row 15's last lane added into row 1 and
// row 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, true));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xA, 0xF, false));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xC, 0xF, false));
  return v;
}

// The wave's sum, in every lane (lane 63 of the inclusive scan).
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  return __builtin_amdgcn_readlane(wave_incl_scan(v), 63);
}

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *s_red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_sum(v);
  if (lane == 0) s_red[wave] = v;
  __syncthreads();
  v = s_red[0] + s_red[1] + s_red[2] + s_red[3];
  __syncthreads();
  return v;
}


// Bit i set iff byte i of a and b differ (i = 0..3).
__device__ __forceinline__ uint32_t bytes_ne4(uint32_t a, uint32_t b) {
  const uint32_t x = a ^ b;
  const uint32_t m = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
  // gather bits 7, 15, 23, 31 into bits 0..3
  return (((m >> 7) * 0x00204081u) >> 21) & 0xFu;
}

// Byte i of an 8-byte octet held as two 32-bit words.
__device__ __forceinline__ uint32_t octet_byte(uint2 v, uint32_t i) {
  return ((i < 4 ? v.x : v.y) >> ((i & 3u) * 8u)) & 0xFFu;
}
__device__ __forceinline__ void set_octet_byte(uint2 &v, uint32_t i,
                                               uint32_t b) {
  const uint32_t sh = (i & 3u) * 8u;
  if (i < 4)
    v.x = (v.x & ~(0xFFu << sh)) | (b << sh);
  else
    v.y = (v.y & ~(0xFFu << sh)) | (b << sh);
}

__device__ __forceinline__ void set_error(uint32_t *err, uint32_t bits) {
  __hip_atomic_fetch_or(err, bits, __ATOMIC_RELAXED,
                        __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void set_error(WsCtl *ctl, uint32_t bits) {
  set_error(&ctl->err, bits);
}

__device__ __forceinline__ void put_header(uint8_t *out, uint32_t mode,
                                           uint32_t B, uint64_t n,
                                           uint64_t changed, uint64_t E,
                                           uint64_t P, uint64_t total,
                                           uint32_t i, uint32_t dtype = 0) {
  if (i >= 16) return;
  uint32_t v = 0;
  switch (i) {
    case 0: v = kMagic; break;
    case 1: v = kVersion | (mode << 16); break;
    case 2: v = B; break;
    case 3: v = dtype; break;
    case 4: v = uint32_t(n); break;
    case 5: v = uint32_t(n >> 32); break;
    case 6: v = uint32_t(changed); break;
    case 7: v = uint32_t(changed >> 32); break;
    case 8: v = uint32_t(E); break;
    case 9: v = uint32_t(E >> 32); break;
    case 10: v = uint32_t(P); break;
    case 11: v = uint32_t(P >> 32); break;
    case 12: v = uint32_t(total); break;
    case 13: v = uint32_t(total >> 32); break;
    default: v = 0; break;
  }
  reinterpret_cast<uint32_t *>(out)[i] = v;
}

// Select x[i] for a lane-varying i < N (N small, x uniform). Written as mask
// arithmetic so that the compiler keeps x in registers instead of turning
// the choice into an indexed load from scratch memory.
template <int N>
__device__ __forceinline__ uint64_t pick(const uint64_t (&x)[N], uint32_t i) {
  uint64_t r = 0;
#pragma unroll
  for (int k = 0; k < N; ++k)
    r |= x[k] & (0ull - uint64_t(i == uint32_t(k)));
  return r;
}

// ------------------------------------------------- block hash (Hash128) --
// Two 64-bit hashes per block from SplitMix64 (Steele, Lea and Flood 2014):
// the block's exponent bytes as little-endian 64-bit words u_j, and
//   H_t = sum over j of mix(u_j XOR (s_t + (j + 1) GAMMA))   (mod 2^64)
// with GAMMA the odd integer nearest 2^64 / golden ratio, mix the SplitMix64
// finaliser and the seeds s_0, s_1 the first two 64-bit words of the binary
// fraction of pi. Word j is one octet of the block, so each lane hashes its
// own octets and a wave sum finishes the block.
constexpr uint64_t kSm64Gamma = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kHashSeed0 = 0x243F6A8885A308D3ull;
constexpr uint64_t kHashSeed1 = 0x13198A2E03707344ull;

__device__ __forceinline__ uint64_t sm64_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ================================================================ encode ==
// A tile is one chunk of kEncChunk = 4096 values and belongs to one wave. It
// holds whole blocks at every B (B <= 4096). Lane l handles octets u*64 + l
// (u = 0..7): wave instruction u covers values [512u, 512u + 512) of it.

// Change detectors of pass 1: exact compare with the exponent cache, or the
// sender's block hash (HashCache) of Algorithm 1; kDetHashOnly computes the
// hashes and writes nothing else (seeding HashCache).
enum : int { kDetExact = 0, kDetHash = 1, kDetHashOnly = 2 };

// Block classes, which fix how a chunk's flags map to bitmap bytes: a block
// lies inside a 512-value unit (B <= 512), spans 2 or 4 units, or is the
// whole chunk.
enum : int { kInUnit = 0, kUnits = 1, kChunkBlock = 2 };
constexpr int enc_class(uint32_t log2B) {
  return log2B <= 9 ? kInUnit : log2B < 12 ? kUnits : kChunkBlock;
}

// The terms of unit u: mix(word XOR state) for both hashes, 0 past n. The
// lane's octet in unit u is word j of its block: j = lane mod (B/8) when
// B <= 512, 64 * (u mod (B/512)) + lane above; st0 and st1 are the states of
// word j mod 64.
template <bool BIG>
__device__ __forceinline__ void hash_terms(uint32_t u, uint32_t log2B,
                                           bool live, uint2 e, uint64_t st0,
                                           uint64_t st1, uint64_t &ta,
                                           uint64_t &tb) {
  const uint64_t word = uint64_t(e.x) | (uint64_t(e.y) << 32);
  if (BIG) {
    const uint64_t shift =
        uint64_t(u & ((1u << (log2B - 9)) - 1u)) * 64 * kSm64Gamma;
    st0 += shift;
    st1 += shift;
  }
  ta = live ? sm64_mix(word ^ st0) : 0ull;
  tb = live ? sm64_mix(word ^ st1) : 0ull;
}

// The order in which a chunk's units are hashed: pairs (i, i + 4), or (2i,
// 2i + 1) when blocks span units.
template <bool BIG>
__device__ constexpr int hash_unit(int q) {
  return BIG ? q : (q >> 1) + 4 * (q & 1);
}

// One exchange step over 2H values: each lane hands half of them to its
// partner across lane bit lbit and keeps the sums of the other half.
template <int H>
__device__ __forceinline__ void hash_exchange(uint64_t (&x)[4], uint32_t lane,
                                              uint32_t lbit) {
  const bool hi = (lane >> lbit) & 1u;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const uint64_t sa = hi ? x[i] : x[i + H], ka = hi ? x[i + H] : x[i];
    x[i] = ka + __shfl_xor(sa, int(1u << lbit), 64);
  }
}

// Finish the chunk's block hashes. Summing 8 units (B <= 512: one value per
// unit) with 8 full reductions would take 48 shuffles a hash; each exchange
// step hands half of a lane's values to the partner lane across one lane bit
// and keeps the other half, so 8 values take 4 + 2 + 1 exchanges, and plain
// xor steps finish the remaining lane bits. The first step, units i and i + 4
// across lane bit g - 1, is taken as the units are hashed (B > 512: units 2i
// and 2i + 1 of a block are added), so x and y hold four values here: 60
// VGPRs and eight waves per SIMD, against 87 and five with all sixteen terms
// live (OLMoE shard, B = 512: 24.1 against 25.5 us for the hashed encode; with
// a loop over chunks around it the pass took 121 and four).
// With v = log2 of the values a lane holds per chunk (one per unit when
// B <= 512, one per block above), g = log2 of the lanes sharing a block and
// t = exchange steps, value i then belongs to local index
// k = (sel << (v - t)) + i (sel: the lane's bits g-1 .. g-t) and is complete
// in the lanes whose low g - t bits are 0. Those lanes compare and store the
// hashes; the change flags go to fw, block c of the chunk in bit c mod 64 of
// word c / 64.
template <int DET, bool BIG>
__device__ __forceinline__ void hash_finish(const EncArgs &a, uint64_t cbase,
                                            uint32_t lane, uint64_t (&x)[4],
                                            uint64_t (&y)[4],
                                            uint64_t (&fw)[4]) {
  const uint64_t n = a.n;
  const uint32_t log2B = a.log2B;
  const uint32_t hv = BIG ? 12u - log2B : 3u;
  const uint32_t hg = BIG ? 6u : log2B - 3u;
  const uint32_t ht = hv < hg ? hv : hg;
  if (BIG) {
    if (log2B >= 11) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x[i] = x[2 * i] + x[2 * i + 1];
        y[i] = y[2 * i] + y[2 * i + 1];
      }
    }
    if (log2B >= 12) {
      x[0] += x[1];
      y[0] += y[1];
    }
  }
  // exchange with half size 2^p, p = v-1 .. v-t, across lane bit g-(v-p)
  if (hv >= 2 && hv - ht <= 1) {
    hash_exchange<2>(x, lane, hg - (hv - 1u));
    hash_exchange<2>(y, lane, hg - (hv - 1u));
  }
  if (hv >= 1 && hv == ht) {
    hash_exchange<1>(x, lane, hg - hv);
    hash_exchange<1>(y, lane, hg - hv);
  }
  const uint32_t cnt = 1u << (hv - ht);  // values left per lane
  for (uint32_t off = (1u << (hg - ht)) >> 1; off > 0; off >>= 1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (uint32_t(i) < cnt) {
        x[i] += __shfl_xor(x[i], int(off), 64);
        y[i] += __shfl_xor(y[i], int(off), 64);
      }
    }
  }
  const bool leader = (lane & ((1u << (hg - ht)) - 1u)) == 0;
  const uint32_t sel = (lane >> (hg - ht)) & ((1u << ht) - 1u);
  uint32_t flags = 0;  // bit i: value i's block changed
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (uint32_t(i) >= cnt) continue;
    const uint32_t k = (sel << (hv - ht)) + uint32_t(i);
    const uint64_t b_idx =
        BIG ? (cbase >> log2B) + k
            : ((cbase + uint64_t(k) * 512) >> log2B) + (lane >> hg);
    if (leader && (b_idx << log2B) < n) {
      bool ch = false;
      if (DET == kDetHash)
        ch = x[i] != a.hash_in[2 * b_idx] || y[i] != a.hash_in[2 * b_idx + 1];
      a.hash_out[2 * b_idx] = x[i];
      a.hash_out[2 * b_idx + 1] = y[i];
      flags |= uint32_t(ch) << i;
    }
  }
  if (DET == kDetHashOnly) return;
  if (BIG) {
    const uint64_t m = __ballot(leader && (flags & 1u));
    for (uint32_t k = 0; k < (1u << hv); ++k)
      fw[0] |= ((m >> (k << (6u - ht))) & 1ull) << k;
  } else {
    // chunk block c = (k << (6 - g)) + grp; its value sits in lane
    // (grp << g) + (sel << (g - t)) as value i = k mod cnt
    const uint32_t nb = kEncChunk >> log2B;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t c = uint32_t(q) * 64u + lane;
      const uint32_t k = c >> (6u - hg);
      const uint32_t grp = c & ((1u << (6u - hg)) - 1u);
      const uint32_t src =
          ((grp << hg) + ((k >> (hv - ht)) << (hg - ht))) & 63u;
      const uint32_t fl = __shfl(flags, int(src), 64);
      fw[q] = __ballot(c < nb && ((fl >> (k & (cnt - 1u))) & 1u));
    }
  }
}

// One chunk of pass 1: everything but the exception list and the bitmap. The
// lane's exponents go to e, its octets' change bits to mask (B = 1: a bit per
// value; exact compare: nonzero where an octet differs) and the chunk's block
// flags (B >= 16) to fw, block c in bit c mod 64 of word c / 64.
// NTW (the fused cache update): the exception pass takes the changed
// exponents from the cache brought forward here, so W' is read once and its
// loads are non-temporal, while the cache bytes are loaded plainly for the
// exception pass to find again. Without it the exception pass re-reads W'
// and the cache is read once: the other way round.
template <bool ELEMS, int DET, bool F16, bool NTW, bool BIG>
__device__ __forceinline__ void encode_chunk(const EncArgs &a, uint64_t cbase,
                                             uint32_t lane, uint8_t *sm_out,
                                             uint2 (&e)[8],
                                             uint32_t (&mask)[8],
                                             uint64_t (&fw)[4]) {
  constexpr bool HASH = DET != kDetExact;
  constexpr bool OUT = DET != kDetHashOnly;
  static_assert(!(HASH && ELEMS), "the block hash needs B >= 16");
  static_assert(!(F16 && (HASH || ELEMS)), "fp16: exact compare, B >= 16");
  const uint64_t n = a.n;
  const uint32_t log2B = a.log2B;
#pragma unroll
  for (int k = 0; k < 4; ++k) fw[k] = 0ull;
  // block hash: the states of the lane's words, and the sums of the units
  // hashed so far (see hash_finish)
  uint64_t st0 = 0, st1 = 0, hx[4], hy[4];
  uint32_t hbit = 0;
  if (HASH) {
    const uint64_t j =
        BIG ? lane : uint64_t(lane & ((1u << (log2B - 3)) - 1u));
    st0 = kHashSeed0 + (j + 1) * kSm64Gamma;
    st1 = kHashSeed1 + (j + 1) * kSm64Gamma;
    hbit = BIG ? 0u : log2B - 4u;
  }
  // hash units ua and ub (their octets' exponents known) into value i
  auto hash_pair = [&](int i, uint32_t ua, uint32_t ub, bool la, bool lb) {
    uint64_t xs[4], ys[4];
    hash_terms<BIG>(ua, log2B, la, e[ua], st0, st1, xs[0], ys[0]);
    hash_terms<BIG>(ub, log2B, lb, e[ub], st0, st1, xs[1], ys[1]);
    if (BIG) {
      hx[i] = xs[0] + xs[1];
      hy[i] = ys[0] + ys[1];
    } else {
      hash_exchange<1>(xs, lane, hbit);
      hash_exchange<1>(ys, lane, hbit);
      hx[i] = xs[0];
      hy[i] = ys[0];
    }
  };
  // the octet's exponents and sign|mantissa bytes from its values
  auto split = [&](uint4 wv, uint64_t elem, uint2 &ev, uint2 &sm) {
    if (F16) {
      uint2 hi;
      split4_f16(wv.x, wv.y, ev.x, sm.x, hi.x);
      split4_f16(wv.z, wv.w, ev.y, sm.y, hi.y);
      uint8_t *pl = sm_out + n + 3 * (elem >> 3);
#pragma unroll
      for (uint32_t q = 0; q < 3; ++q)
        pl[q] = uint8_t(plane_byte(hi.x, hi.y, q));
    } else {
      split4(wv.x, wv.y, ev.x, sm.x);
      split4(wv.z, wv.w, ev.y, sm.y);
    }
  };
  auto compare = [&](uint2 ev, uint2 cv) {
    return ELEMS ? (bytes_ne4(ev.x, cv.x) | (bytes_ne4(ev.y, cv.y) << 4))
                 : uint32_t((ev.x != cv.x) || (ev.y != cv.y));
  };
  if (cbase + kEncChunk <= n) {
    uint4 wv[8];
    uint2 cv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      wv[u] = NTW ? ld_nt16(a.w + cbase + (uint64_t(u) * 64 + lane) * 8)
                  : ld16(a.w + cbase + (uint64_t(u) * 64 + lane) * 8);
    if (!HASH) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        cv[u] = NTW ? ld8(a.cache + cbase + (uint64_t(u) * 64 + lane) * 8)
                    : ld_nt8(a.cache + cbase + (uint64_t(u) * 64 + lane) * 8);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int u = HASH ? hash_unit<BIG>(q) : q;
      const uint64_t elem = cbase + (uint64_t(u) * 64 + lane) * 8;
      uint2 sm;
      split(wv[u], elem, e[u], sm);
      if (OUT) st_nt8(sm_out + elem, sm);
      if (HASH) {
        mask[u] = 0;
        if (q & 1)
          hash_pair(q >> 1, uint32_t(hash_unit<BIG>(q - 1)), uint32_t(u),
                    true, true);
      } else {
        mask[u] = compare(e[u], cv[u]);
        // the sender's cache brought forward: only octets that differ
        if (a.cache_out && mask[u]) st8(a.cache_out + elem, e[u]);
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t elem = cbase + (uint64_t(u) * 64 + lane) * 8;
      const uint32_t valid = octet_valid(elem, n);
      mask[u] = 0;
      e[u] = make_uint2(0u, 0u);
      if (valid) {
        // load_w8 zero-fills past n: those fields are 0 in the planes and
        // the hash words, and never a change against a cached 0
        uint2 sm;
        split(load_w8(a.w + elem, valid), elem, e[u], sm);
        if (OUT) store_b8(sm_out + elem, sm, valid);
        if (!HASH) {
          mask[u] = compare(e[u], load_b8(a.cache + elem, valid));
          if (a.cache_out && mask[u])
            store_b8(a.cache_out + elem, e[u], valid);
        }
      }
    }
    if (HASH) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t ua = uint32_t(hash_unit<BIG>(2 * i)),
                       ub = uint32_t(hash_unit<BIG>(2 * i + 1));
        hash_pair(i, ua, ub, cbase + (uint64_t(ua) * 64 + lane) * 8 < n,
                  cbase + (uint64_t(ub) * 64 + lane) * 8 < n);
      }
    }
  }
  if (HASH) {
    hash_finish<DET, BIG>(a, cbase, lane, hx, hy, fw);
  } else if (!ELEMS) {
    uint64_t m[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] = __ballot(mask[u] != 0);
    if (!BIG) {
      // 512/B blocks per 512-value unit, B/8 octets (bits of m[u]) each
      const uint32_t opb_log2 = log2B - 3;
      const uint32_t bpu_log2 = 6 - opb_log2;
      const uint64_t gmask =
          opb_log2 == 6 ? ~0ull : ((1ull << (1u << opb_log2)) - 1ull);
      const uint32_t nb = kEncChunk >> log2B;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t b = uint32_t(k) * 64u + lane;
        bool f = false;
        if (b < nb) {
          const uint64_t word = pick<8>(m, b >> bpu_log2);
          const uint32_t sh = (b & ((1u << bpu_log2) - 1u)) << opb_log2;
          f = ((word >> sh) & gmask) != 0;
        }
        fw[k] = __ballot(f);
      }
    } else {
      // a block spans 2^(log2B-9) units
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (m[u]) fw[0] |= 1ull << (uint32_t(u) >> (log2B - 9));
    }
  }
}

// The padding of the first two sections, and the bitmap bytes that no chunk
// holds, zeroed by one wave.
template <bool ELEMS, bool F16>
__device__ __forceinline__ void pad_sections(const EncArgs &a, uint32_t lane) {
  const uint64_t S_sm = sm_bytes(a.n, F16), n16 = pad16(S_sm);
  const uint64_t bm = bitmap_bytes(a.n, a.log2B), bm16 = pad16(bm);
  uint8_t *const sm_out = a.out + kHeaderBytes;
  for (uint64_t i = S_sm + lane; i < n16; i += 64) sm_out[i] = 0;
  uint64_t written = bm;
  if (!ELEMS)
    written = ((uint64_t(a.num_tiles) << (12 - a.log2B)) + 7) >> 3;
  if (written > bm16) written = bm16;
  for (uint64_t i = written + lane; i < bm16; i += 64) sm_out[n16 + i] = 0;
}

// Pass 1 for blocks of class CLS. A bitmap byte holds 8 blocks. Up to B = 512
// a chunk fills whole bytes; above, 2, 4 or 8 chunks share one, so the
// workgroup's waves put their bits together in LDS: at B = 4096 that takes 8
// waves (elsewhere 4, which keeps the tiles of a workgroup and of the
// exception pass's workgroup alike).
// Bound by HBM (4 bytes a value). A wave that went on over 8 blocks, as it did
// above B = 512, left 768 waves on the chip at B = 4096 and 25.2M values; with
// a chunk a wave the encode of that shard (both passes) takes 25.9 instead of
// 42.4 us, of 88.1M clustered values 84.7 instead of 92.5 us, of 4.0M values
// 11.4 instead of 36.4 us. Without the loop over chunks the kernel also
// needs 58 instead of 78 VGPRs (eight waves per SIMD); at B = 512 the OLMoE
// shard's encode takes 23.2 instead of 23.4 us.
constexpr int enc_waves(int cls) { return cls == kChunkBlock ? 8 : 4; }
template <bool ELEMS, int DET, bool F16, bool NTW, int CLS>
__global__ __launch_bounds__(64 * enc_waves(CLS)) void encode_pass_kernel(
    EncArgs a) {
  constexpr bool OUT = DET != kDetHashOnly;
  constexpr int W = enc_waves(CLS);
  __shared__ uint32_t s_bits[W];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroup L = 8k + x runs on XCD x as its k-th. With runs of
  // G = 2^a.xcd_run_log2 workgroups it takes the tiles of workgroup
  // (k / G) 8G + x G + k mod G, so each XCD streams G neighbouring
  // workgroups' tiles at a time; the tail short of 8G keeps the plain order.
  uint32_t grp = blockIdx.x;
  if (a.xcd_run_log2) {
    const uint32_t g = a.xcd_run_log2;
    if (grp < ((gridDim.x >> (g + 3)) << (g + 3))) {
      const uint32_t k = grp >> 3;
      grp = ((k >> g) << (g + 3)) | ((grp & 7u) << g) | (k & ((1u << g) - 1u));
    }
  }
  const uint32_t tile = grp * uint32_t(W) + wave;
  const uint32_t log2B = a.log2B;
  constexpr bool shared_bytes = OUT && !ELEMS && CLS != kInUnit;
  const bool live = tile < a.num_tiles;
  if (!live && !shared_bytes) return;
  const uint64_t n = a.n;
  const uint64_t cbase = uint64_t(tile) * kEncChunk;
  const uint64_t S_sm = sm_bytes(n, F16);  // sign+mantissa section
  const uint64_t n16 = pad16(S_sm);
  const uint64_t bm = bitmap_bytes(n, log2B);
  const uint64_t bm16 = pad16(bm);
  uint8_t *const sm_out = OUT ? a.out + kHeaderBytes : nullptr;
  uint8_t *const bmp_out = OUT ? sm_out + n16 : nullptr;

  uint32_t mask[8];
  uint2 e[8];
  uint64_t fw[4];
  if (live)
    encode_chunk<ELEMS, DET, F16, NTW, CLS != kInUnit>(a, cbase, lane, sm_out,
                                                       e, mask, fw);
  if (!OUT) return;

  uint32_t count = 0;
  if (ELEMS) {
    // an octet's change byte is its bitmap byte
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t elem = cbase + (uint64_t(u) * 64 + lane) * 8;
      if (elem < n) bmp_out[elem >> 3] = uint8_t(mask[u]);
      count += __popc(mask[u]);
    }
    count = wave_sum(count);
  } else if (CLS == kInUnit) {
    const uint32_t nbytes = uint32_t(kEncChunk >> log2B) >> 3;
    const uint64_t byte0 = uint64_t(tile) * nbytes;
    for (uint32_t i = lane; i < nbytes; i += 64) {
      const uint64_t pos = byte0 + i;
      if (pos < bm16)
        bmp_out[pos] = uint8_t(pick<4>(fw, i >> 3) >> ((i & 7u) * 8u));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) count += uint32_t(__popcll(fw[k]));
  } else {
    const uint32_t nb_log2 = 12 - log2B;  // log2 of the blocks in a chunk
    const uint32_t cpb = 1u << (log2B - 9);  // chunks per bitmap byte
    if (lane == 0) s_bits[wave] = live ? uint32_t(fw[0]) : 0u;
    __syncthreads();
    if (!live) return;
    const uint64_t pos = uint64_t(tile) >> (log2B - 9);
    if (lane == 0 && (wave & (cpb - 1u)) == 0 && pos < bm16) {
      uint32_t b = 0;
      for (uint32_t i = 0; i < cpb && wave + i < uint32_t(W); ++i)
        b |= s_bits[wave + i] << (i << nb_log2);
      bmp_out[pos] = uint8_t(b);
    }
  }
  if ((ELEMS || a.scan_prefix) && lane == 0) a.counts[tile] = count;

  // before the exception pass reads the bitmap back
  if (tile == a.num_tiles - 1) pad_sections<ELEMS, F16>(a, lane);
}

// Exclusive scan of `count` 32-bit counts per segment, in place, one
// 1024-thread workgroup per segment (segment j starts at c + j * stride, a
// 16-byte aligned address); the segment's total goes to c[count]. Each pass
// covers 16384 counts: 16 per thread, loaded as four 16-byte vectors.
constexpr int kScanThreads = 1024;
constexpr uint32_t kScanPer = 16;

__global__ __launch_bounds__(kScanThreads) void scan_counts_kernel(
    uint32_t *counts, uint32_t count, uint64_t stride) {
  __shared__ uint32_t s_wave[kScanThreads / 64];
  __shared__ uint32_t s_total;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t *c = counts + uint64_t(blockIdx.x) * stride;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < count; base += kScanThreads * kScanPer) {
    const uint32_t lo = base + tid * kScanPer;
    uint32_t v[kScanPer];
    if (lo + kScanPer <= count) {
#pragma unroll
      for (uint32_t q = 0; q < kScanPer / 4; ++q) {
        const uint4 x = *reinterpret_cast<const uint4 *>(c + lo + 4 * q);
        v[4 * q] = x.x;
        v[4 * q + 1] = x.y;
        v[4 * q + 2] = x.z;
        v[4 * q + 3] = x.w;
      }
    } else {
#pragma unroll
      for (uint32_t i = 0; i < kScanPer; ++i)
        v[i] = lo + i < count ? c[lo + i] : 0u;
    }
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < kScanPer; ++i) {
      const uint32_t t = v[i];
      v[i] = sum;  // exclusive within the thread
      sum += t;
    }
    const uint32_t incl = wave_incl_scan(sum);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    if (tid == 0) {
      uint32_t run = 0;
      for (int w = 0; w < kScanThreads / 64; ++w) {
        const uint32_t t = s_wave[w];
        s_wave[w] = run;
        run += t;
      }
      s_total = run;
    }
    __syncthreads();
    const uint32_t off = carry + s_wave[wave] + incl - sum;
    if (lo + kScanPer <= count) {
#pragma unroll
      for (uint32_t q = 0; q < kScanPer / 4; ++q)
        *reinterpret_cast<uint4 *>(c + lo + 4 * q) =
            make_uint4(off + v[4 * q], off + v[4 * q + 1], off + v[4 * q + 2],
                       off + v[4 * q + 3]);
    } else {
#pragma unroll
      for (uint32_t i = 0; i < kScanPer; ++i)
        if (lo + i < count) c[lo + i] = off + v[i];
    }
    carry += s_total;
    __syncthreads();
  }
  if (tid == 0) c[count] = carry;
}

// This thread's share of the flagged blocks in bitmap bytes [0, nbytes):
// every load is issued before the first add (clamped addresses, no
// branches), so a workgroup's count costs one round trip per L 16-byte
// words per thread. Sum it over the workgroup with block_sum.
template <uint32_t L>
__device__ __forceinline__ uint32_t popc_bytes_part(const uint8_t *bmp,
                                                    uint64_t nbytes) {
  if (!nbytes) return 0u;
  const uint64_t full16 = nbytes >> 4;
  const uint64_t ti = (full16 << 4) + threadIdx.x;  // < 16 tail bytes
  const uint32_t tb = bmp[ti < nbytes ? ti : nbytes - 1];
  const uint4 *b4 = reinterpret_cast<const uint4 *>(bmp);
  uint32_t c = 0;
  for (uint64_t i0 = 0; i0 < full16; i0 += L * kThreads) {
    uint4 v[L];
#pragma unroll
    for (uint32_t j = 0; j < L; ++j) {
      const uint64_t i = i0 + j * kThreads + threadIdx.x;
      v[j] = b4[i < full16 ? i : full16 - 1];
    }
#pragma unroll
    for (uint32_t j = 0; j < L; ++j) {
      const uint64_t i = i0 + j * kThreads + threadIdx.x;
      const uint32_t w = __popc(v[j].x) + __popc(v[j].y) + __popc(v[j].z) +
                         __popc(v[j].w);
      c += i < full16 ? w : 0u;
    }
  }
  return c + (ti < nbytes ? uint32_t(__popc(tb)) : 0u);
}

// The exponents of one octet (e: one byte per value) at exception index pos:
// bf16 bytes at pos, fp16 five bit-plane bytes at 5 (pos / 8).
template <bool F16>
__device__ __forceinline__ void put_exc_exps(uint8_t *exc_out, uint64_t pos,
                                             uint2 e, uint32_t valid) {
  if (F16) {
    uint8_t *g = exc_out + 5 * (pos >> 3);
#pragma unroll
    for (uint32_t q = 0; q < 5; ++q) g[q] = uint8_t(plane_byte(e.x, e.y, q));
  } else if (valid == 8) {
    st_nt8(exc_out + pos, e);
  } else {
    store_b8(exc_out + pos, e, valid);
  }
}

// Where the exception pass takes a changed octet's exponents from. Without
// the fused cache update it splits W' again (16 bytes an octet). With it,
// pass 1 has already written the new exponent of every changed value into
// the cache, and every other value of a changed block was unchanged, so the
// cache holds exp(W') for the whole block: 8 bytes an octet.
template <bool F16, bool FROMC>
struct ExcSrc {
  using T = typename std::conditional<FROMC, uint2, uint4>::type;
  __device__ static __forceinline__ T load(const EncArgs &a, uint64_t elem,
                                           uint32_t valid) {
    if constexpr (FROMC) {
      if (valid == 8) return ld_nt8(a.cache_out + elem);
      return load_b8(a.cache_out + elem, valid);
    } else {
      return reread_w8(a.w + elem, valid);
    }
  }
  __device__ static __forceinline__ uint2 exps(const T &v) {
    if constexpr (FROMC) {
      return v;
    } else {
      uint2 e, t0, t1;
      if (F16) {
        split4_f16(v.x, v.y, e.x, t0.x, t1.x);
        split4_f16(v.z, v.w, e.y, t0.y, t1.y);
      } else {
        split4(v.x, v.y, e.x, t0.x);
        split4(v.z, v.w, e.y, t0.y);
      }
      return e;
    }
  }
};

// Whether the shard's last block is flagged in its bitmap (B >= 16).
__device__ __forceinline__ bool last_block_changed(const EncArgs &a,
                                                   const uint8_t *bmp) {
  const uint64_t nblk = blocks_of(a.n, a.log2B);
  if (!nblk) return false;
  return (bmp[(nblk - 1) >> 3] >> ((nblk - 1) & 7u)) & 1u;
}

// The totals, known to the wave that holds the last tile: the header, the
// exception section's zero padding and the encoded size. total_changed
// counts changed blocks (B >= 16; last_changed: the last block is one of
// them) or changed values (B = 1).
template <bool ELEMS, bool F16>
__device__ void exc_finish(const EncArgs &a, uint64_t total_changed,
                           uint32_t lane, bool last_changed) {
  const uint64_t n = a.n;
  const uint32_t log2B = a.log2B;
  const uint32_t B = 1u << log2B;
  const uint64_t S_sm = sm_bytes(n, F16);
  const uint64_t n16 = pad16(S_sm);
  const uint64_t bm = bitmap_bytes(n, log2B);
  const uint64_t bm16 = pad16(bm);
  uint8_t *const exc_out = a.out + kHeaderBytes + n16 + bm16;
  uint64_t E = total_changed;
  if (!ELEMS) {
    E = total_changed << log2B;
    // the last block may be short
    if (last_changed) E -= (blocks_of(n, log2B) << log2B) - n;
  }
  if (E > n) {  // only with a count array that was written by someone else
    if (lane == 0) set_error(a.ctl, CIERA_DEVERR_BOUNDS);
    E = n;
  }
  const uint64_t S_exc = exc_bytes(E, F16);
  const uint64_t P = S_sm + bm + S_exc;
  const uint64_t total = kHeaderBytes + n16 + bm16 + pad16(S_exc);
  put_header(a.out, kModeCompressed, B, n, total_changed, E, P, total, lane,
             F16 ? kDtypeFp16 : kDtypeBf16);
  if (lane == 16 && a.out_bytes) *a.out_bytes = total;
  for (uint64_t i = S_exc + lane; i < pad16(S_exc); i += 64) exc_out[i] = 0;
}

// This thread's share of the 32-bit counts c[0, count) (c 16-byte
// aligned): every load issued before the first add, as in popc_bytes_part.
// Sum it over the workgroup with block_sum.
template <uint32_t L>
__device__ __forceinline__ uint32_t sum_words_part(const uint32_t *c,
                                                   uint64_t count) {
  if (!count) return 0u;
  const uint64_t full4 = count >> 2;
  const uint64_t ti = (full4 << 2) + threadIdx.x;  // < 4 tail words
  const uint32_t tw = c[ti < count ? ti : count - 1];
  const uint4 *c4 = reinterpret_cast<const uint4 *>(c);
  uint32_t s = 0;
  for (uint64_t i0 = 0; i0 < full4; i0 += L * kThreads) {
    uint4 v[L];
#pragma unroll
    for (uint32_t j = 0; j < L; ++j) {
      const uint64_t i = i0 + j * kThreads + threadIdx.x;
      v[j] = c4[i < full4 ? i : full4 - 1];
    }
#pragma unroll
    for (uint32_t j = 0; j < L; ++j) {
      const uint64_t i = i0 + j * kThreads + threadIdx.x;
      s += i < full4 ? v[j].x + v[j].y + v[j].z + v[j].w : 0u;
    }
  }
  return s + (ti < count ? tw : 0u);
}

// Pass 2 for B = 1: the tile's changed values, at the tile's offset in the
// list: the per-tile counts of pass 1 in front of the tile, summed here by
// the workgroup, or (a.scan_prefix) read from their scan. The last tile
// writes the header. W' is read again only where the bitmap says so.
template <bool FROMC>
__global__ __launch_bounds__(kThreads) void encode_exc_elems_kernel(
    EncArgs a) {
  using Src = ExcSrc<false, FROMC>;
  __shared__ uint32_t s_red[4];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t nt = a.num_tiles;
  const uint32_t tile = blockIdx.x * 4u + wave;
  const bool live = tile < nt;  // every wave takes part in the count
  const uint64_t n = a.n;
  const uint64_t tbase = uint64_t(tile) * kEncChunk;
  const uint64_t n16 = pad16(sm_bytes(n, false));
  const uint8_t *const bmp = a.out + kHeaderBytes + n16;
  uint8_t *const exc_out =
      a.out + kHeaderBytes + n16 + pad16(bitmap_bytes(n, 0));
  uint32_t mask[8], excl[8];
  uint32_t run = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const uint64_t elem = tbase + (uint64_t(u) * 64 + lane) * 8;
    const uint32_t valid = live ? octet_valid(elem, n) : 0u;
    mask[u] = valid ? uint32_t(bmp[elem >> 3]) & ((1u << valid) - 1u) : 0u;
    const uint32_t c = __popc(mask[u]);
    const uint32_t incl = wave_incl_scan(c);
    excl[u] = run + incl - c;
    run += __shfl(incl, 63, 64);
  }
  typename Src::T wv[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const uint64_t elem = tbase + (uint64_t(u) * 64 + lane) * 8;
    if (mask[u]) wv[u] = Src::load(a, elem, octet_valid(elem, n));
  }
  uint32_t prefix;
  if (a.scan_prefix) {
    prefix = live ? a.counts[tile] : 0u;
  } else {
    const uint32_t g0 = min(blockIdx.x * 4u, nt);
    const uint32_t cg = sum_words_part<kGroupLoads>(a.counts, g0);
    const uint32_t cs =
        (lane < wave && g0 + lane < nt) ? a.counts[g0 + lane] : 0u;
    prefix = block_sum(cg, s_red) + wave_sum(cs);
  }
  if (!live) return;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    uint32_t mm = mask[u];
    if (!mm) continue;
    const uint2 e = Src::exps(wv[u]);
    uint64_t pos = uint64_t(prefix) + excl[u];
    while (mm) {
      const uint32_t i = __builtin_ctz(mm);
      if (pos < n) exc_out[pos] = uint8_t(octet_byte(e, i));
      ++pos;
      mm &= mm - 1u;
    }
  }
  if (tile == nt - 1)
    exc_finish<true, false>(
        a, a.scan_prefix ? uint64_t(a.counts[nt]) : uint64_t(prefix) + run,
        lane, false);
}

// Pass 2 for B >= 512. A row of 512 values lies inside one block, so it is
// changed or unchanged as a whole, and the exceptions of the changed rows
// follow one another in row order: the k-th changed row's exponents start at
// 512 k in the list. A tile is 8 rows (4096 values, whole blocks). Each wave
// takes a run of a.exc_tiles_per_wave tiles and copies its changed rows D at a
// time, so that that many reads of the rows' exponents are in flight per wave;
// the first batch is issued before the offset of the run (the changed blocks
// in front of it) is counted, and the two overlap.
template <bool F16, bool FROMC, uint32_t D>
__global__ __launch_bounds__(kThreads) void encode_exc_rows_kernel(EncArgs a) {
  using Src = ExcSrc<F16, FROMC>;
  __shared__ uint32_t s_red[4];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t n = a.n;
  const uint32_t rpb_log2 = a.log2B - 9;  // rows per block
  const uint64_t S_sm = sm_bytes(n, F16);
  const uint64_t n16 = pad16(S_sm);
  const uint64_t bm = bitmap_bytes(n, a.log2B);
  const uint8_t *const bmp = a.out + kHeaderBytes + n16;
  uint8_t *const exc_out = a.out + kHeaderBytes + n16 + pad16(bm);
  const uint64_t nt = a.num_tiles, tpw = a.exc_tiles_per_wave;
  // the workgroups in runs per XCD (as in pass 1)
  uint32_t grp = blockIdx.x;
  if (a.exc_xcd_run_log2) {
    const uint32_t g = a.exc_xcd_run_log2;
    if (grp < ((gridDim.x >> (g + 3)) << (g + 3))) {
      const uint32_t k = grp >> 3;
      grp = ((k >> g) << (g + 3)) | ((grp & 7u) << g) | (k & ((1u << g) - 1u));
    }
  }
  const uint64_t g0 = min(uint64_t(grp) * 4u * tpw, nt);
  const uint64_t t0 = min(g0 + wave * tpw, nt);
  const uint64_t t1 = min(t0 + tpw, nt);
  const uint64_t rows = (n + 511) >> 9;
  const uint64_t r0 = min(t0 << 3, rows);
  const uint64_t r1 = min(t1 << 3, rows);

  // changed rows among [c, c + 64) of the run, as a wave-uniform mask
  auto chunk_mask = [&](uint64_t c) -> uint64_t {
    const uint64_t row = c + lane;
    bool f = false;
    if (row < r1) {
      const uint64_t b = row >> rpb_log2;
      f = (bmp[b >> 3] >> (b & 7u)) & 1u;
    }
    return __ballot(f);
  };
  uint64_t c = r0, m = r0 < r1 ? chunk_mask(r0) : 0ull;
  uint32_t rr[D], cnt = 0;
  typename Src::T wv[D];
  // the next batch of changed rows of chunk c: positions and W' loads
  auto take_batch = [&]() {
    cnt = 0;
#pragma unroll
    for (uint32_t d = 0; d < D; ++d) {
      if (m) {
        rr[d] = uint32_t(__builtin_ctzll(m));
        m &= m - 1ull;
        cnt = d + 1;
      }
    }
#pragma unroll
    for (uint32_t d = 0; d < D; ++d) {
      if (d < cnt) {
        const uint64_t elem = ((c + rr[d]) << 9) + uint64_t(lane) * 8;
        const uint32_t valid = octet_valid(elem, n);
        if (valid) wv[d] = Src::load(a, elem, valid);
      }
    }
  };
  take_batch();

  // the run's offset in changed blocks: the bitmap bytes in front of it
  uint32_t prefix;
  if (a.scan_prefix) {
    prefix = a.counts[t0];
  } else {
    const uint64_t gb = (g0 << 3) >> (rpb_log2 + 3);  // whole bytes in front
    const uint64_t b0 = (t0 << 3) >> rpb_log2;  // the run's first block
    // bits of byte i in front of b0 (the sibling runs' and the byte they end
    // in): whole bytes, then a partial one
    auto front = [&](uint64_t i, uint32_t v) {
      const uint64_t left = b0 > (i << 3) ? b0 - (i << 3) : 0;
      return uint32_t(__popc(left < 8 ? v & ((1u << left) - 1u) : v));
    };
    const uint64_t si = gb + lane;
    const uint32_t sv = bm ? bmp[min(si, bm - 1)] : 0u;
    const uint32_t cg = popc_bytes_part<kGroupLoads>(bmp, min(gb, bm));
    uint32_t cs = si < bm ? front(si, sv) : 0u;
    for (uint64_t i = si + 64; i < min((b0 + 7) >> 3, bm); i += 64)
      cs += front(i, bmp[i]);  // runs of > 21 tiles
    prefix = block_sum(cg, s_red) + wave_sum(cs);
  }

  uint64_t out_row = uint64_t(prefix) << rpb_log2;
  for (;;) {
#pragma unroll
    for (uint32_t d = 0; d < D; ++d) {
      if (d < cnt) {
        const uint64_t elem = ((c + rr[d]) << 9) + uint64_t(lane) * 8;
        const uint32_t valid = octet_valid(elem, n);
        const uint64_t pos = ((out_row + d) << 9) + uint64_t(lane) * 8;
        if (valid && pos + valid <= n)
          put_exc_exps<F16>(exc_out, pos, Src::exps(wv[d]), valid);
      }
    }
    out_row += cnt;
    while (!m) {
      c += 64;
      if (c >= r1) break;
      m = chunk_mask(c);
    }
    if (c >= r1) break;
    take_batch();
  }

  if (t0 < nt && t1 == nt) {
    uint32_t own = 0;
    const uint64_t b0 = (t0 << 3) >> rpb_log2;
    for (uint64_t i = (b0 >> 3) + lane; i < bm; i += 64) {
      const uint32_t skip = i == (b0 >> 3) ? uint32_t(b0 & 7u) : 0u;
      own += __popc(uint32_t(bmp[i]) >> skip);
    }
    exc_finish<false, F16>(a, uint64_t(prefix) + wave_sum(own), lane,
                           last_block_changed(a, bmp));
  }
}

// Pass 2 for B = 16 ... 256, over the changed blocks only. A block is
// B / 8 octets, so one wave instruction covers 512 / B blocks; the k-th
// changed block's exponents start at B k in the list. Each wave takes a run
// of a.exc_tiles_per_wave tiles (512 / B bitmap bytes each), lists the
// changed blocks of each 64-block chunk of its run in LDS (ballot and mbcnt),
// and copies them kExcBatch instructions at a time: the work follows the
// changed blocks, not the shard. The first batch is issued before the
// offset count of the run, and the two overlap.
template <bool F16, bool FROMC>
__global__ __launch_bounds__(kThreads) void encode_exc_blocks_kernel(
    EncArgs a) {
  using Src = ExcSrc<F16, FROMC>;
  constexpr uint32_t D = kExcBatch;
  __shared__ uint32_t s_red[4];
  __shared__ uint32_t s_list[4][64];  // a wave's changed blocks of a chunk
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t n = a.n;
  const uint32_t log2B = a.log2B;
  const uint32_t lpb_log2 = log2B - 3;  // lanes per block
  const uint32_t bpr_log2 = 9 - log2B;  // blocks per instruction
  const uint32_t slot = lane >> lpb_log2;
  const uint64_t in_blk = uint64_t(lane & ((1u << lpb_log2) - 1u)) * 8u;
  const uint64_t S_sm = sm_bytes(n, F16);
  const uint64_t n16 = pad16(S_sm);
  const uint64_t bm = bitmap_bytes(n, log2B);
  const uint8_t *const bmp = a.out + kHeaderBytes + n16;
  uint8_t *const exc_out = a.out + kHeaderBytes + n16 + pad16(bm);
  const uint64_t nt = a.num_tiles, tpw = a.exc_tiles_per_wave;
  const uint64_t bpt = (kEncChunk >> log2B) >> 3;  // bitmap bytes per tile
  const uint64_t g0 = min(uint64_t(blockIdx.x) * 4u * tpw, nt);
  const uint64_t t0 = min(g0 + wave * tpw, nt);
  const uint64_t t1 = min(t0 + tpw, nt);
  const uint64_t nblk = blocks_of(n, log2B);
  const uint64_t b0 = min(t0 * bpt * 8u, nblk);
  const uint64_t b1 = min(t1 * bpt * 8u, nblk);
  uint32_t *const list = s_list[wave];

  // the changed blocks among [c, c + 64) of the run, listed in order
  uint64_t c = b0;
  uint32_t nm = 0, r = 0;  // listed blocks of chunk c, and those taken
  auto list_chunk = [&]() {
    const uint64_t b = c + lane;
    bool f = false;
    if (b < b1) f = (bmp[b >> 3] >> (b & 7u)) & 1u;
    const uint64_t m = __ballot(f);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the last chunk's list was read
    if (f)
      list[__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u))] =
          uint32_t(b);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    nm = uint32_t(__popcll(m));
    r = 0;
  };
  uint32_t kk[D], valid[D];
  uint64_t elem[D];
  typename Src::T wv[D];
  uint32_t taken = 0;  // list entries this batch covers
  // the next batch: D instructions of 512 / B listed blocks, W' loads issued
  auto take_batch = [&]() {
#pragma unroll
    for (uint32_t d = 0; d < D; ++d) {
      kk[d] = r + (d << bpr_log2) + slot;
      valid[d] = 0;
      if (kk[d] < nm) {
        elem[d] = (uint64_t(list[kk[d]]) << log2B) + in_blk;
        valid[d] = octet_valid(elem[d], n);
        if (valid[d]) wv[d] = Src::load(a, elem[d], valid[d]);
      }
    }
    taken = min(nm - r, D << bpr_log2);
  };
  if (b0 < b1) {
    list_chunk();
    take_batch();
  }

  // the run's offset in changed blocks: the bitmap bytes in front of it
  uint32_t prefix;
  if (a.scan_prefix) {
    prefix = a.counts[t0];
  } else {
    const uint64_t gb = min(g0 * bpt, bm);  // the workgroup's bytes in front
    const uint64_t sb = min(t0 * bpt, bm);  // + the sibling runs in front
    const uint64_t si = gb + lane;
    const uint32_t sv = bm ? bmp[min(si, bm - 1)] : 0u;
    const uint32_t cg = popc_bytes_part<kGroupLoads>(bmp, gb);
    uint32_t cs = si < sb ? uint32_t(__popc(sv)) : 0u;
    for (uint64_t i = si + 64; i < sb; i += 64)
      cs += __popc(uint32_t(bmp[i]));
    prefix = block_sum(cg, s_red) + wave_sum(cs);
  }

  uint64_t out_blk = prefix;  // list index of the batch's first block
  while (b0 < b1) {
#pragma unroll
    for (uint32_t d = 0; d < D; ++d) {
      if (valid[d]) {
        const uint64_t pos = ((out_blk + kk[d] - r) << log2B) + in_blk;
        if (pos + valid[d] <= n)
          put_exc_exps<F16>(exc_out, pos, Src::exps(wv[d]), valid[d]);
      }
    }
    out_blk += taken;
    r += taken;
    while (r >= nm) {
      c += 64;
      if (c >= b1) break;
      list_chunk();
    }
    if (c >= b1) break;
    take_batch();
  }

  if (t0 < nt && t1 == nt) {
    uint32_t own = 0;
    for (uint64_t i = t0 * bpt + lane; i < min(t1 * bpt, bm); i += 64)
      own += __popc(uint32_t(bmp[i]));
    exc_finish<false, F16>(a, uint64_t(prefix) + wave_sum(own), lane,
                           last_block_changed(a, bmp));
  }
}

// The whole encode of a small shard (up to kEncSmall values) in one launch of
// one workgroup, a wave a chunk: the waves put their counts together in LDS
// and write their changed exponents from registers. A second kernel, and the
// re-read of what it copies, would cost more than the other CUs could save.
// Bound by latency: load, compare, count across the waves, store (3.7 us at 128
// values against 5.4 for the two kernels, and one launch of 2.5 us less on the
// host; 4.15 us with 16 waves whatever the shard and a loop over rounds).
constexpr int kSmallWaves = int(kEncSmall / kEncChunk);
static_assert(kEncSmall % kEncChunk == 0 && kSmallWaves >= 1 &&
                  kSmallWaves <= 16,
              "a wave a chunk in one workgroup");
template <bool ELEMS, int DET, bool F16, bool BIG>
__global__ __launch_bounds__(64 * kSmallWaves) void encode_small_kernel(
    EncArgs a) {
  constexpr uint32_t W = kSmallWaves;
  __shared__ uint32_t s_cnt[W];
  __shared__ uint32_t s_bits[W];
  __shared__ uint32_t s_last;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t tile = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t nt = a.num_tiles;  // the workgroup's waves
  const uint64_t n = a.n;
  const uint32_t log2B = a.log2B;
  const uint64_t n16 = pad16(sm_bytes(n, F16));
  const uint64_t bm16 = pad16(bitmap_bytes(n, log2B));
  uint8_t *const sm_out = a.out + kHeaderBytes;
  uint8_t *const bmp_out = sm_out + n16;
  uint8_t *const exc_out = bmp_out + bm16;
  const uint64_t cbase = uint64_t(tile) * kEncChunk;
  uint32_t mask[8], excl[8], count = 0;
  uint2 e[8];
  uint64_t fw[4];
  encode_chunk<ELEMS, DET, F16, true, BIG>(a, cbase, lane, sm_out, e, mask,
                                           fw);
  if (ELEMS) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t elem = cbase + (uint64_t(u) * 64 + lane) * 8;
      if (elem < n) bmp_out[elem >> 3] = uint8_t(mask[u]);
      const uint32_t c = __popc(mask[u]);
      const uint32_t incl = wave_incl_scan(c);
      excl[u] = count + incl - c;
      count += __builtin_amdgcn_readlane(incl, 63);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) count += uint32_t(__popcll(fw[k]));
    const uint32_t nb = kEncChunk >> log2B;  // blocks in a chunk
    if (!BIG) {
      const uint64_t byte0 = uint64_t(tile) * (nb >> 3);
      for (uint32_t i = lane; i < (nb >> 3); i += 64)
        if (byte0 + i < bm16)
          bmp_out[byte0 + i] =
              uint8_t(pick<4>(fw, i >> 3) >> ((i & 7u) * 8u));
    } else if (lane == 0) {
      s_bits[tile] = uint32_t(fw[0]);
    }
    // the last block's flag decides the list's length; no other wave writes
    // it (n = 0: no flag is set)
    if (tile == nt - 1 && lane == 0) {
      const uint32_t k =
          n ? uint32_t(blocks_of(n, log2B) - 1 - (cbase >> log2B)) : 0u;
      s_last = uint32_t(pick<4>(fw, k >> 6) >> (k & 63u)) & 1u;
    }
  }
  if (lane == 0) s_cnt[tile] = count;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (uint32_t w = 0; w < W; ++w) {
    const uint32_t c = w < nt ? s_cnt[w] : 0u;
    before += w < tile ? c : 0u;
    total += c;
  }
  if (BIG) {
    // bitmap byte i: the bits of 8 / nb chunks
    const uint32_t nb_log2 = 12 - log2B, cpb_log2 = log2B - 9;
    const uint32_t t0 = threadIdx.x << cpb_log2;
    if (t0 < nt && threadIdx.x < bm16) {
      uint32_t b = 0;
      for (uint32_t i = 0; i < (1u << cpb_log2) && t0 + i < nt; ++i)
        b |= s_bits[t0 + i] << (i << nb_log2);
      bmp_out[threadIdx.x] = uint8_t(b);
    }
  }
  if (ELEMS) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      uint32_t mm = mask[u], pos = before + excl[u];
      while (mm) {
        exc_out[pos++] = uint8_t(octet_byte(e[u], __builtin_ctz(mm)));
        mm &= mm - 1u;
      }
    }
  } else {
    // values from cbase
    const uint32_t left =
        n > cbase ? uint32_t(min(n - cbase, uint64_t(kEncChunk))) : 0u;
    uint32_t in_front[4];  // flags in the words in front of each
    uint32_t run = before;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      in_front[k] = run;
      run += uint32_t(__popcll(fw[k]));
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t rel = uint32_t(u) * 512u + lane * 8u;
      const uint32_t b = rel >> log2B;
      // a unit's blocks share one word of the flags
      const uint32_t q = (uint32_t(u) * 512u >> log2B) >> 6;
      const uint64_t word =
          q == 0 ? fw[0] : q == 1 ? fw[1] : q == 2 ? fw[2] : fw[3];
      const uint32_t front = q == 0   ? in_front[0]
                             : q == 1 ? in_front[1]
                             : q == 2 ? in_front[2]
                                      : in_front[3];
      // (no flag past n; the exponents past n in the last octet are 0, as
      // the padding that they fall into)
      if (rel < left && ((word >> (b & 63u)) & 1u)) {
        const uint32_t rank =
            front + uint32_t(__popcll(word & ((1ull << (b & 63u)) - 1ull)));
        put_exc_exps<F16>(exc_out,
                          (rank << log2B) | (rel & ((1u << log2B) - 1u)),
                          e[u], 8);
      }
    }
  }
  if (tile == nt - 1) pad_sections<ELEMS, F16>(a, lane);
  if (tile == 0) exc_finish<ELEMS, F16>(a, total, lane, !ELEMS && s_last != 0);
}

// Raw form: header + the values unchanged. One octet per lane, non-temporal:
// 25.2M values just written and then encoded take 30.1 us together, against
// 35.8 with plain accesses (34.0M 40.7 / 49.1; encoded again, out of the cache,
// 22.6 / 21.6).
__global__ __launch_bounds__(kThreads) void encode_raw_kernel(
    const uint16_t *w, uint64_t n, uint32_t B, uint8_t *out,
    uint64_t *out_bytes, uint32_t dtype) {
  const uint64_t total = kHeaderBytes + pad16(2 * n);
  const uint64_t octets = (n + 7) / 8;
  const uint64_t o = uint64_t(blockIdx.x) * kThreads + threadIdx.x;
  uint16_t *body = reinterpret_cast<uint16_t *>(out + kHeaderBytes);
  if (o < octets) {
    const uint64_t elem = o * 8;
    const uint32_t valid = octet_valid(elem, n);
    if (valid == 8)
      st_nt16(body + elem, ld_nt16(w + elem));
    else
      store_w8(body + elem, load_w8(w + elem, valid), valid);
  }
  if (blockIdx.x == 0) {
    const uint32_t tid = threadIdx.x;
    put_header(out, kModeRaw, B, n, 0, 0, 2 * n, total, tid, dtype);
    if (tid == 16 && out_bytes) *out_bytes = total;
    uint8_t *bytes = out + kHeaderBytes;
    for (uint64_t i = 2 * n + tid; i < pad16(2 * n); i += kThreads) bytes[i] = 0;
  }
}

// ================================================================ decode ==
struct ShardView {
  const uint8_t *enc;
  const uint8_t *exc;  // the exception list (decoded, for rANS-coded shards)
  uint32_t mode;
  uint64_t E;
  bool ok;
};

// Every workgroup validates the header of its shard (a 64-byte line that all
// of the shard's tiles share in L2). Tile 0 reports what is wrong. The header
// is read only when it lies inside the caller's buffer, and the shard is used
// only when its total does too.
__device__ __forceinline__ ShardView read_shard(const DecArgs &a, uint32_t j,
                                                bool report) {
  ShardView v;
  const uint64_t off = a.offsets ? a.offsets[j] : 0ull;
  v.enc = a.gathered + off;
  v.ok = false;
  v.exc = nullptr;
  v.mode = 0;
  v.E = 0;
  if (off & 15ull) {
    if (report) set_error(a.err, CIERA_DEVERR_ALIGN);
    return v;
  }
  if (off > a.bytes || a.bytes - off < kHeaderBytes) {
    if (report) set_error(a.err, CIERA_DEVERR_BOUNDS);
    return v;
  }
  const uint32_t *h32 = reinterpret_cast<const uint32_t *>(v.enc);
  const uint64_t *h64 = reinterpret_cast<const uint64_t *>(v.enc);
  const uint32_t magic = h32[0], vm = h32[1], hB = h32[2];
  const uint64_t hn = h64[2], hE = h64[4], hP = h64[5], htotal = h64[6];
  const uint32_t mode = vm >> 16;
  bool ok = magic == kMagic && (vm & 0xFFFFu) == kVersion && hn == a.n &&
            h32[3] == (a.f16 ? kDtypeFp16 : kDtypeBf16);
  const uint64_t bm = bitmap_bytes(hn, a.log2B);
  const uint64_t sm16 = pad16(sm_bytes(hn, a.f16));
  if (ok && mode == kModeCompressed) {
    ok = hB == (1u << a.log2B) && hE <= hn &&
         htotal == kHeaderBytes + sm16 + pad16(bm) +
                       pad16(exc_bytes(hE, a.f16));
  } else if (ok && mode == kModeAns && !a.f16) {
    // rANS-coded exceptions (B >= 16): the list was decoded into the
    // workspace by ans_decode_kernel, which checks the coded section
    ok = a.log2B >= uint32_t(kAnsMinLog2B) && hB == (1u << a.log2B) &&
         hE <= hn && hP >= hn + bm + kAnsFixed &&
         htotal == kHeaderBytes + pad16(hn) + pad16(bm) +
                       pad16(hP - hn - bm);
    if (ok && a.ans_exc == nullptr) {
      if (report) set_error(a.err, CIERA_DEVERR_NOSPACE);
      return v;
    }
  } else if (ok && mode == kModeRaw) {
    ok = htotal == kHeaderBytes + pad16(2 * hn);
  } else {
    ok = false;
  }
  if (!ok) {
    if (report) set_error(a.err, CIERA_DEVERR_FORMAT);
    return v;
  }
  if (htotal > a.bytes - off) {
    if (report) set_error(a.err, CIERA_DEVERR_BOUNDS);
    return v;
  }
  v.ok = true;
  v.mode = mode;
  v.E = hE;
  v.exc = mode == kModeAns ? a.ans_exc + uint64_t(j) * a.ans_stride
                           : v.enc + kHeaderBytes + sm16 + pad16(bm);
  return v;
}

// Decode, B >= 16, step 1: for every shard the flagged blocks in front of
// each decode tile, an exclusive scan of the tiles' bitmap counts (one
// 1024-thread workgroup per shard; the bitmap is 1/(8B) of the shard). Raw
// and malformed shards write nothing: their decode tiles do not read it.
__global__ __launch_bounds__(kScanThreads) void tile_prefix_kernel(DecArgs a) {
  __shared__ uint32_t s_wave[kScanThreads / 64];
  __shared__ uint32_t s_total;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t j = blockIdx.x;
  const ShardView sv = read_shard(a, j, false);
  if (!sv.ok || sv.mode == kModeRaw) return;
  const uint64_t n = a.n;
  const uint32_t tiles = uint32_t(dec_tiles(n));
  const uint32_t *bmp32 = reinterpret_cast<const uint32_t *>(
      sv.enc + kHeaderBytes + pad16(sm_bytes(n, a.f16)));
  // the bitmap section holds pad16(bm) bytes, zero past the last block
  const uint64_t words = pad16(bitmap_bytes(n, a.log2B)) >> 2;
  const uint32_t tb = kDecTileLog2 - a.log2B;  // log2 of the blocks per tile
  uint32_t *c = a.tile_excl + uint64_t(j) * dec_count_stride(tiles);
  uint32_t carry = 0;
  for (uint32_t base = 0; base < tiles; base += kScanThreads) {
    const uint32_t t = base + tid;
    uint32_t cnt = 0;
    if (t < tiles) {
      const uint64_t b0 = uint64_t(t) << tb;  // the tile's first block
      if (tb >= 7) {
        // 4 to 32 words: up to eight 16-byte vectors, all loaded before the
        // sum (the section's word count is a multiple of 4)
        const uint4 *v4 = reinterpret_cast<const uint4 *>(bmp32) + (b0 >> 7);
        const uint64_t left = (words >> 2) - (b0 >> 7);
        const uint32_t nv = 1u << (tb - 7);
        uint4 x[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k)
          x[k] = k < nv && k < left ? v4[k] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k)
          cnt += __popc(x[k].x) + __popc(x[k].y) + __popc(x[k].z) +
                 __popc(x[k].w);
      } else if (tb >= 5) {
        const uint64_t w0 = b0 >> 5, w1 = w0 + (uint64_t(1) << (tb - 5));
        for (uint64_t w = w0; w < w1 && w < words; ++w) cnt += __popc(bmp32[w]);
      } else if ((b0 >> 5) < words) {
        cnt = __popc((bmp32[b0 >> 5] >> (b0 & 31u)) & ((1u << (1u << tb)) - 1u));
      }
    }
    const uint32_t incl = wave_incl_scan(cnt);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    if (tid == 0) {
      uint32_t run = 0;
      for (int w = 0; w < kScanThreads / 64; ++w) {
        const uint32_t x = s_wave[w];
        s_wave[w] = run;
        run += x;
      }
      s_total = run;
    }
    __syncthreads();
    if (t < tiles) c[t] = carry + s_wave[wave] + incl - cnt;
    carry += s_total;
    __syncthreads();
  }
}

// UPDATE_ONLY: the ExpCache patch alone (no sign+mantissa, no output).
// A whole tile issues its loads in two batches (sign|mantissa bytes together
// with the bitmap words, then one cache-or-exception load per octet, chosen
// by address rather than by branch); the ragged last tile goes octet by
// octet. RAWNT: the loads of raw shards (raw_plain_loads); a template argument,
// because a branch on it moved the schedule of the merge (fp16, 16 shards of
// 2.1M values: 31.4 -> 36.8 us).
template <int OCT, bool UPDATE_ONLY, bool F16, bool RAWNT>
__global__ __launch_bounds__(kThreads) void decode_kernel(DecArgs a) {
  constexpr uint32_t T = kThreads * 8 * OCT;
  // tile bitmap words (32 blocks each) covering at most T/16 blocks + 1 word
  constexpr uint32_t kBitWords = T / 16 / 32 + 2;
  static_assert(kBitWords <= kThreads, "one bitmap word per thread");
  __shared__ uint32_t s_bits[kBitWords];
  __shared__ uint32_t s_pre[kBitWords];
  __shared__ uint32_t s_red[4];
  // fp16 whole tiles: the tile's sign/top-mantissa planes (3 bytes per
  // octet) come through LDS in 8-byte loads instead of 3 byte loads a lane
  constexpr uint32_t kHiPairs = F16 && !UPDATE_ONLY ? 3 * T / 64 : 1;
  __shared__ uint2 s_hi[kHiPairs];

  // Workgroups go to the 8 XCDs in turn: workgroup L = 8k + x is XCD x's
  // k-th. With runs of G = 2^a.xcd_run_log2 tiles it takes tile
  // (k / G) 8G + x G + k mod G of the (shard, tile) order, so each XCD walks
  // G neighbouring tiles at a time; the tail short of 8G tiles keeps the
  // plain order.
  const uint32_t ntiles = gridDim.x;
  uint32_t j = blockIdx.y, tix = blockIdx.x;
  if (a.xcd_run_log2) {
    const uint32_t g = a.xcd_run_log2;
    const uint64_t total = uint64_t(ntiles) * gridDim.y;
    uint64_t L = uint64_t(blockIdx.y) * ntiles + blockIdx.x;
    if (L < ((total >> (g + 3)) << (g + 3))) {
      const uint64_t k = L >> 3;
      L = ((k >> g) << (g + 3)) | ((L & 7u) << g) | (k & ((1u << g) - 1u));
      j = uint32_t(L / ntiles);
      tix = uint32_t(L % ntiles);
    }
  }
  const uint64_t base = uint64_t(tix) * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ShardView sv = read_shard(a, j, tix == 0 && tid == 0);
  if (!sv.ok) return;
  const uint64_t n = a.n;
  if (base >= n) return;
  const bool full = base + T <= n;
  uint8_t *const cache = a.cache + uint64_t(j) * n;
  uint16_t *const out = UPDATE_ONLY ? nullptr : a.out + uint64_t(j) * n;

  if (sv.mode == kModeRaw) {
    // (decode_raw_tile is this code for B = 1: a change goes into both)
    // three streams touched once: non-temporal as in the merge, but for the
    // loads of a gather that may lie in the Infinity Cache
    const uint16_t *body =
        reinterpret_cast<const uint16_t *>(sv.enc + kHeaderBytes);
    if (full) {
      uint4 wv[OCT];
#pragma unroll
      for (int u = 0; u < OCT; ++u) {
        const uint16_t *const p =
            body + base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
        wv[u] = RAWNT ? ld_nt16(p) : ld16(p);
      }
#pragma unroll
      for (int u = 0; u < OCT; ++u) {
        const uint64_t elem =
            base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
        uint2 e, sm, hi;
        if (F16) {
          split4_f16(wv[u].x, wv[u].y, e.x, sm.x, hi.x);
          split4_f16(wv[u].z, wv[u].w, e.y, sm.y, hi.y);
        } else {
          split4(wv[u].x, wv[u].y, e.x, sm.x);
          split4(wv[u].z, wv[u].w, e.y, sm.y);
        }
        if (!UPDATE_ONLY) st_nt16(out + elem, wv[u]);
        st_nt8(cache + elem, e);
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      const uint32_t o = uint32_t(wave * OCT + u) * 64u + lane;
      const uint64_t elem = base + uint64_t(o) * 8u;
      const uint32_t valid = octet_valid(elem, n);
      if (!valid) continue;
      const uint4 wv = load_w8(body + elem, valid);
      uint2 e, sm, hi;
      if (F16) {
        split4_f16(wv.x, wv.y, e.x, sm.x, hi.x);
        split4_f16(wv.z, wv.w, e.y, sm.y, hi.y);
      } else {
        split4(wv.x, wv.y, e.x, sm.x);
        split4(wv.z, wv.w, e.y, sm.y);
      }
      if (!UPDATE_ONLY) store_w8(out + elem, wv, valid);
      store_b8(cache + elem, e, valid);
    }
    return;
  }

  const uint32_t log2B = a.log2B;
  const uint32_t B = 1u << log2B;
  const uint8_t *const sm_in = sv.enc + kHeaderBytes;
  const uint8_t *const bmp = sm_in + pad16(sm_bytes(n, F16));
  const uint32_t *const bmp32 = reinterpret_cast<const uint32_t *>(bmp);
  const uint8_t *const exc = sv.exc;

  // sign|mantissa bytes first: they do not depend on the bitmap (fp16: the
  // low mantissa bytes, and the sign and top mantissa bits from 3 planes)
  uint2 smv[OCT], hiv[OCT];
  if (F16 && !UPDATE_ONLY) {
    if (full) {
      // the barriers of the prefix sum below order these stores
      const uint8_t *hp = sm_in + n + 3 * (base >> 3);
      for (uint32_t i = tid; i < kHiPairs; i += kThreads)
        s_hi[i] = ld_nt8(hp + 8 * i);
    } else {
#pragma unroll
      for (int u = 0; u < OCT; ++u) {
        const uint64_t elem =
            base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
        hiv[u] = elem < n ? unplane<3>(sm_in + n + 3 * (elem >> 3))
                          : make_uint2(0u, 0u);
      }
    }
  }
  if (!UPDATE_ONLY) {
    if (full) {
#pragma unroll
      for (int u = 0; u < OCT; ++u)
        smv[u] =
            ld_nt8(sm_in + base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u);
    } else {
#pragma unroll
      for (int u = 0; u < OCT; ++u) {
        const uint64_t elem =
            base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
        const uint32_t valid = octet_valid(elem, n);
        smv[u] =
            valid ? load_b8(sm_in + elem, valid) : make_uint2(0u, 0u);
      }
    }
  }

  // this tile's bitmap words, and the count of flagged blocks before it
  const uint64_t end = (base + T < n) ? base + T : n;
  const uint64_t fb = base >> log2B;             // first block of the tile
  const uint64_t lbk = (end - 1) >> log2B;       // last block of the tile
  const uint64_t w0 = fb >> 5;
  const uint32_t nw = uint32_t((lbk >> 5) - w0 + 1);  // <= 33 < kThreads
  // one word per thread (clamped address, no branch), stored below, so that
  // the count's loads are issued before anything waits for it
  uint32_t word = bmp32[w0 + (tid < nw ? tid : nw - 1u)];
  if (tid == 0) word &= ~((1u << (fb & 31u)) - 1u);
  // flagged blocks in front of the tile: from tile_prefix_kernel, or
  // counted here straight from the bitmap, every load issued before the
  // first count
  uint32_t prefix;
  if (a.prefix_pass) {
    prefix = a.tile_excl[uint64_t(j) * dec_count_stride(ntiles) + tix];
    if (tid < nw) s_bits[tid] = word;
    __syncthreads();  // s_bits, and the fp16 planes in s_hi
  } else {
    const uint64_t full4 = w0 >> 2;  // whole 16-byte chunks before word w0
    const uint64_t wr = (full4 << 2) + tid;  // leftover words before w0
    const uint32_t wl = bmp32[wr < w0 ? wr : 0u];
    const uint32_t wf = bmp32[w0];
    const uint4 *b4 = reinterpret_cast<const uint4 *>(bmp);
    uint32_t cnt = 0;
    for (uint64_t i0 = 0; i0 < full4; i0 += kGroupLoads * kThreads) {
      uint4 v[kGroupLoads];
#pragma unroll
      for (uint32_t k = 0; k < kGroupLoads; ++k) {
        const uint64_t i = i0 + k * kThreads + tid;
        v[k] = b4[i < full4 ? i : full4 - 1];
      }
#pragma unroll
      for (uint32_t k = 0; k < kGroupLoads; ++k) {
        const uint64_t i = i0 + k * kThreads + tid;
        const uint32_t c = __popc(v[k].x) + __popc(v[k].y) + __popc(v[k].z) +
                           __popc(v[k].w);
        cnt += i < full4 ? c : 0u;
      }
    }
    if (tid < nw) s_bits[tid] = word;
    cnt += (tid < 4 && wr < w0) ? uint32_t(__popc(wl)) : 0u;
    if (tid == 4 && (fb & 31u))
      cnt += __popc(wf & ((1u << (fb & 31u)) - 1u));
    prefix = block_sum(cnt, s_red);  // also orders s_bits and s_hi
  }
  if (tid == 0) {
    uint32_t run = 0;
    for (uint32_t i = 0; i < nw; ++i) {
      s_pre[i] = run;
      run += __popc(s_bits[i]);
    }
  }
  __syncthreads();

  bool bad = false;
  if (full) {
    bool ch[OCT];
    const uint8_t *src[OCT];
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      const uint64_t elem = base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
      const uint32_t rel = uint32_t((elem >> log2B) - (w0 << 5));
      const uint32_t word = s_bits[rel >> 5];
      ch[u] = (word >> (rel & 31u)) & 1u;
      const uint32_t rank =
          s_pre[rel >> 5] + __popc(word & ((1u << (rel & 31u)) - 1u));
      const uint64_t pos =
          (uint64_t(prefix + rank) << log2B) | (elem & uint64_t(B - 1u));
      if (ch[u] && pos + 8 > sv.E) {  // inconsistent shard: stay in bounds
        bad = true;
        ch[u] = false;
      }
      // fp16: the octet's exponents are the 5 plane bytes of group pos / 8
      src[u] = ch[u] ? (F16 ? exc + 5 * (pos >> 3) : exc + pos) : cache + elem;
    }
    uint2 ev[OCT];
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      if (F16 && ch[u])
        ev[u] = unplane<5>(src[u]);
      else if (!UPDATE_ONLY)
        ev[u] = ld_nt8(src[u]);
      else if (ch[u])  // the cache update alone: plain loads measured faster
        ev[u] = ld8(src[u]);
    }
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      const uint64_t elem = base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
      if (ch[u]) {
        if (UPDATE_ONLY)
          st8(cache + elem, ev[u]);
        else  // the merge's patches: non-temporal, like its other streams
          st_nt8(cache + elem, ev[u]);
      }
      if (!UPDATE_ONLY) {
        uint4 wv;
        if (F16) {
          const uint32_t o = uint32_t(wave * OCT + u) * 64u + lane;
          const uint2 hv = unplane<3>(
              reinterpret_cast<const uint8_t *>(s_hi) + 3 * o);
          merge4_f16(ev[u].x, smv[u].x, hv.x, wv.x, wv.y);
          merge4_f16(ev[u].y, smv[u].y, hv.y, wv.z, wv.w);
        } else {
          merge4(ev[u].x, smv[u].x, wv.x, wv.y);
          merge4(ev[u].y, smv[u].y, wv.z, wv.w);
        }
        st_nt16(out + elem, wv);
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      const uint32_t o = uint32_t(wave * OCT + u) * 64u + lane;
      const uint64_t elem = base + uint64_t(o) * 8u;
      const uint32_t valid = octet_valid(elem, n);
      if (!valid) continue;
      const uint32_t rel = uint32_t((elem >> log2B) - (w0 << 5));
      const uint32_t word = s_bits[rel >> 5];
      uint2 ev;
      if ((word >> (rel & 31u)) & 1u) {
        const uint32_t rank =
            s_pre[rel >> 5] + __popc(word & ((1u << (rel & 31u)) - 1u));
        const uint64_t pos =
            (uint64_t(prefix + rank) << log2B) | (elem & uint64_t(B - 1u));
        if (pos + valid > sv.E) {
          bad = true;
          continue;
        }
        ev = F16 ? unplane<5>(exc + 5 * (pos >> 3))
                 : load_b8(exc + pos, valid);
        store_b8(cache + elem, ev, valid);
      } else {
        if (UPDATE_ONLY) continue;
        ev = load_b8(cache + elem, valid);
      }
      if (!UPDATE_ONLY) {
        uint4 wv;
        if (F16) {
          merge4_f16(ev.x, smv[u].x, hiv[u].x, wv.x, wv.y);
          merge4_f16(ev.y, smv[u].y, hiv[u].y, wv.z, wv.w);
        } else {
          merge4(ev.x, smv[u].x, wv.x, wv.y);
          merge4(ev.y, smv[u].y, wv.z, wv.w);
        }
        store_w8(out + elem, wv, valid);
      }
    }
  }
  if (bad) set_error(a.err, CIERA_DEVERR_BOUNDS);
}

// ============================================== element exceptions (B = 1) ==
// At B = 1 the bitmap has one bit per value: octet o of the shard owns bitmap
// byte o, and the exception list holds the changed exponent bytes in value
// order (the encoder is encode_pass_kernel<..., true, ...>). Within a decode tile
// the octets are ranked by a wave scan per 64-octet segment and a scan of the
// segment totals; the per-tile counts in front of the tile (added up by the
// tile's workgroup, or scanned per shard) give the tile start.

// Exclusive rank of this lane's octet among the set bits of its tile, for
// every u; returns the tile total. `cnt[u]` are the per-octet bit counts.
template <int OCT>
__device__ __forceinline__ uint32_t rank_octets(const uint32_t (&cnt)[OCT],
                                                uint32_t (&excl)[OCT],
                                                uint32_t *s_seg) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl[OCT];
#pragma unroll
  for (int u = 0; u < OCT; ++u) {
    incl[u] = wave_incl_scan(cnt[u]);
    if (lane == 63) s_seg[wave * OCT + u] = incl[u];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int i = 0; i < 4 * OCT; ++i) {
      const uint32_t t = s_seg[i];
      s_seg[i] = run;
      run += t;
    }
    s_seg[4 * OCT] = run;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < OCT; ++u)
    excl[u] = s_seg[wave * OCT + u] + incl[u] - cnt[u];
  return s_seg[4 * OCT];
}

// Decode, B = 1, step 1: the number of set bitmap bits in every decode tile
// of every shard (one wave per tile; raw or malformed shards count 0).
__global__ __launch_bounds__(kThreads) void count_tile_bits_kernel(
    DecArgs a, uint32_t tiles) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t j = blockIdx.y;
  const uint32_t t = blockIdx.x * 4u + uint32_t(wave);
  if (t >= tiles) return;
  const ShardView sv = read_shard(a, j, false);
  uint32_t c = 0;
  if (sv.ok && sv.mode == kModeCompressed) {
    const uint8_t *bmp = sv.enc + kHeaderBytes + pad16(a.n);
    const uint64_t bm = (a.n + 7) / 8;
    const uint64_t lo = uint64_t(t) * (kDecTile / 8);
    const uint64_t hi = (lo + kDecTile / 8 < bm) ? lo + kDecTile / 8 : bm;
    for (uint64_t i = lo + uint64_t(lane) * 16u; i < hi; i += 64u * 16u) {
      if (i + 16 <= hi) {
        const uint4 v = *reinterpret_cast<const uint4 *>(bmp + i);
        c += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
      } else {
        for (uint64_t k = i; k < hi; ++k) c += __popc(uint32_t(bmp[k]));
      }
    }
  }
  c = wave_sum(c);
  if (lane == 0) a.tile_excl[uint64_t(j) * dec_count_stride(tiles) + t] = c;
}

// A tile of a raw shard in the B = 1 decode: the values copied, their
// exponents to the cache, as in decode_kernel (a change goes into both; that
// kernel keeps the code in place:
// with a call here it takes 81 instead of 72 VGPRs and 2% longer on every
// layer). 16 raw shards of 1.06M values: 18.0 us against 21.9 octet by octet.
template <int OCT, bool UPDATE_ONLY, bool RAWNT>
__device__ __forceinline__ void decode_raw_tile(const ShardView &sv,
                                                uint64_t base, uint64_t n,
                                                bool full, int wave, int lane,
                                                uint8_t *cache,
                                                uint16_t *out) {
  const uint16_t *body =
      reinterpret_cast<const uint16_t *>(sv.enc + kHeaderBytes);
  if (full) {
    uint4 wv[OCT];
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      const uint16_t *const p =
          body + base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
      wv[u] = RAWNT ? ld_nt16(p) : ld16(p);
    }
#pragma unroll
    for (int u = 0; u < OCT; ++u) {
      const uint64_t elem =
          base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
      uint2 e, sm;
      split4(wv[u].x, wv[u].y, e.x, sm.x);
      split4(wv[u].z, wv[u].w, e.y, sm.y);
      if (!UPDATE_ONLY) st_nt16(out + elem, wv[u]);
      st_nt8(cache + elem, e);
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < OCT; ++u) {
    const uint32_t o = uint32_t(wave * OCT + u) * 64u + lane;
    const uint64_t elem = base + uint64_t(o) * 8u;
    const uint32_t valid = octet_valid(elem, n);
    if (!valid) continue;
    const uint4 wv = load_w8(body + elem, valid);
    uint2 e, sm;
    split4(wv.x, wv.y, e.x, sm.x);
    split4(wv.z, wv.w, e.y, sm.y);
    if (!UPDATE_ONLY) store_w8(out + elem, wv, valid);
    store_b8(cache + elem, e, valid);
  }
}

// Decode, B = 1, step 2 (step 3 after a scan of the counts): patch and merge
// (UPDATE_ONLY: patch only; SMALL: the only step, the tile counts the bitmap
// in front of it).
template <int OCT, bool UPDATE_ONLY, bool SMALL, bool RAWNT>
__global__ __launch_bounds__(kThreads) void decode_elems_kernel(DecArgs a) {
  constexpr uint32_t T = kThreads * 8 * OCT;
  __shared__ uint32_t s_seg[4 * OCT + 1];
  __shared__ uint32_t s_red[4];

  const uint32_t j = blockIdx.y;
  const uint32_t t = blockIdx.x;
  const uint64_t base = uint64_t(t) * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ShardView sv = read_shard(a, j, t == 0 && tid == 0);
  if (!sv.ok) return;
  const uint64_t n = a.n;
  if (base >= n) return;
  uint8_t *const cache = a.cache + uint64_t(j) * n;
  uint16_t *const out = UPDATE_ONLY ? nullptr : a.out + uint64_t(j) * n;

  if (sv.mode == kModeRaw) {
    decode_raw_tile<OCT, UPDATE_ONLY, RAWNT>(sv, base, n, base + T <= n, wave,
                                             lane, cache, out);
    return;
  }

  const uint8_t *const sm_in = sv.enc + kHeaderBytes;
  const uint8_t *const bmp = sm_in + pad16(n);
  const uint8_t *const exc = bmp + pad16((n + 7) / 8);
  const uint32_t tiles = uint32_t(dec_tiles(n));
  const bool full = base + T <= n;

  uint32_t mask[OCT], cnt[OCT];
  uint2 smv[OCT], ev[OCT];
#pragma unroll
  for (int u = 0; u < OCT; ++u) {
    const uint64_t elem = base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
    const uint32_t valid = full ? 8u : octet_valid(elem, n);
    mask[u] = valid ? uint32_t(bmp[elem >> 3]) : 0u;
    if (valid < 8) mask[u] &= (1u << valid) - 1u;
    cnt[u] = __popc(mask[u]);
    if (full) {
      // streams this call touches once: non-temporal, as in decode_kernel
      // (the cache update alone keeps plain loads there too)
      if (!UPDATE_ONLY) smv[u] = ld_nt8(sm_in + elem);
      ev[u] = UPDATE_ONLY ? ld8(cache + elem) : ld_nt8(cache + elem);
    } else {
      smv[u] = make_uint2(0u, 0u);
      ev[u] = make_uint2(0u, 0u);
      if (valid) {
        if (!UPDATE_ONLY) smv[u] = load_b8(sm_in + elem, valid);
        ev[u] = load_b8(cache + elem, valid);
      }
    }
  }
  // the changed values in front of the tile: counted from the bitmap (small
  // layers, no count kernel), scanned, or the counts in front of it added up
  // here, the loads of either sum behind the tile's own
  uint32_t tile_first;
  if constexpr (SMALL) {
    tile_first = block_sum(popc_bytes_part<kGroupLoads>(bmp, base >> 3), s_red);
  } else {
    const uint32_t *const counts =
        a.tile_excl + uint64_t(j) * dec_count_stride(tiles);
    tile_first = a.prefix_pass
                     ? counts[t]
                     : block_sum(sum_words_part<kGroupLoads>(counts, t), s_red);
  }
  uint32_t excl[OCT];
  rank_octets<OCT>(cnt, excl, s_seg);

  bool bad = false;
#pragma unroll
  for (int u = 0; u < OCT; ++u) {
    const uint64_t elem = base + (uint64_t(wave * OCT + u) * 64u + lane) * 8u;
    const uint32_t valid = full ? 8u : octet_valid(elem, n);
    if (!valid) continue;
    uint32_t m = mask[u];
    if (m) {
      uint64_t pos = uint64_t(tile_first) + excl[u];
      if (pos + cnt[u] > sv.E) {
        bad = true;
        continue;
      }
      while (m) {
        const uint32_t i = __builtin_ctz(m);
        set_octet_byte(ev[u], i, exc[pos++]);
        m &= m - 1u;
      }
      if (!UPDATE_ONLY && full)
        st_nt8(cache + elem, ev[u]);
      else
        store_b8(cache + elem, ev[u], valid);
    }
    if (!UPDATE_ONLY) {
      uint4 wv;
      merge4(ev[u].x, smv[u].x, wv.x, wv.y);
      merge4(ev[u].y, smv[u].y, wv.z, wv.w);
      if (full)
        st_nt16(out + elem, wv);
      else
        store_w8(out + elem, wv, valid);
    }
  }
  if (bad) set_error(a.err, CIERA_DEVERR_BOUNDS);
}

__global__ void fill_zero_kernel(uint32_t *p, uint64_t words) {
  for (uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < words;
       i += uint64_t(gridDim.x) * blockDim.x)
    p[i] = 0u;
}

}  // namespace

// ============================================================= launchers ==
namespace {
template <bool B>
using bool_c = std::integral_constant<bool, B>;
template <int I>
using int_c = std::integral_constant<int, I>;

// go(class of the block size), as a template argument
template <typename Go>
void by_class(uint32_t log2B, Go go) {
  switch (enc_class(log2B)) {
    case kInUnit: go(int_c<kInUnit>{}); break;
    case kUnits: go(int_c<kUnits>{}); break;
    default: go(int_c<kChunkBlock>{}); break;
  }
}

// Launch the exception-pass kernel that pick(f16, from_cache) names, with the
// two flags as template arguments (f16 is always false at B = 1).
template <bool ELEMS, typename Pick>
void launch_exc(dim3 grid, const EncArgs &a, bool f16, bool fromc,
                hipStream_t s, Pick pick) {
  auto go = [&](auto f, auto c) {
    hipLaunchKernelGGL(pick(f, c), grid, dim3(kThreads), 0, s, a);
  };
  auto with_c = [&](auto f) {
    if (fromc) go(f, bool_c<true>{}); else go(f, bool_c<false>{});
  };
  if (!ELEMS && f16) with_c(bool_c<!ELEMS>{});
  else with_c(bool_c<false>{});
}
}  // namespace

namespace {
hipError_t launch_encode_small(const EncArgs &a, hipStream_t s) {
  auto go = [&](auto e, auto det, auto f, auto big) {
    hipLaunchKernelGGL((encode_small_kernel<decltype(e)::value,
                                            decltype(det)::value,
                                            decltype(f)::value,
                                            decltype(big)::value>),
                       dim3(1), dim3(64 * a.num_tiles), 0, s, a);
  };
  auto blocks = [&](auto det, auto f) {
    if (enc_class(a.log2B) == kInUnit)
      go(bool_c<false>{}, det, f, bool_c<false>{});
    else
      go(bool_c<false>{}, det, f, bool_c<true>{});
  };
  if (a.log2B == 0)
    go(bool_c<true>{}, int_c<kDetExact>{}, bool_c<false>{}, bool_c<false>{});
  else if (a.f16)
    blocks(int_c<kDetExact>{}, bool_c<true>{});
  else if (a.hashed)
    blocks(int_c<kDetHash>{}, bool_c<false>{});
  else
    blocks(int_c<kDetExact>{}, bool_c<false>{});
  return hipGetLastError();
}
}  // namespace

hipError_t launch_encode(const EncArgs &a, hipStream_t s) {
  if (enc_small(a.n, a.log2B, a.f16)) return launch_encode_small(a, s);
  const dim3 grid((a.num_tiles + 3) / 4);
  const bool elems = a.log2B == 0;
  // with the fused cache update the exception pass reads the cache, not W'
  const bool fromc = a.cache_out != nullptr;
  auto pass = [&](auto e, auto det, auto f, auto c) {
    constexpr bool E = decltype(e)::value, F = decltype(f)::value,
                   C = decltype(c)::value;
    constexpr int D = decltype(det)::value;
    auto go = [&](auto cls) {
      constexpr int K = E ? int(kInUnit) : decltype(cls)::value;
      constexpr uint32_t W = enc_waves(K);
      hipLaunchKernelGGL((encode_pass_kernel<E, D, F, C, K>),
                         dim3((a.num_tiles + W - 1) / W), dim3(64 * W), 0, s,
                         a);
    };
    by_class(a.log2B, go);
  };
  auto exact = [&](auto e, auto f) {
    constexpr int_c<kDetExact> det{};
    if (fromc) pass(e, det, f, bool_c<true>{});
    else pass(e, det, f, bool_c<false>{});
  };
  if (elems)
    exact(bool_c<true>{}, bool_c<false>{});
  else if (a.f16)
    exact(bool_c<false>{}, bool_c<true>{});
  else if (a.hashed)
    pass(bool_c<false>{}, int_c<kDetHash>{}, bool_c<false>{}, bool_c<false>{});
  else
    exact(bool_c<false>{}, bool_c<false>{});
  if (a.scan_prefix)
    hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(kScanThreads), 0, s,
                       a.counts, a.num_tiles, uint64_t(0));
  if (elems) {
    launch_exc<true>(grid, a, false, fromc, s, [](auto, auto c) {
      return encode_exc_elems_kernel<decltype(c)::value>;
    });
    return hipGetLastError();
  }
  // B >= 16: runs of tiles per wave, over the changed blocks (B <= 256) or
  // the changed 512-value rows (B >= 512)
  EncArgs r = a;
  if (r.exc_tiles_per_wave == 0) r.exc_tiles_per_wave = 1;
  const uint64_t waves = (uint64_t(r.num_tiles) + r.exc_tiles_per_wave - 1) /
                         r.exc_tiles_per_wave;
  const dim3 rgrid(uint32_t((waves + 3) / 4));
  if (r.log2B < 9)
    launch_exc<false>(rgrid, r, r.f16, fromc, s, [](auto f, auto c) {
      return encode_exc_blocks_kernel<decltype(f)::value, decltype(c)::value>;
    });
  else if (fromc && r.exc_tiles_per_wave >= 2)
    launch_exc<false>(rgrid, r, r.f16, fromc, s, [](auto f, auto c) {
      return encode_exc_rows_kernel<decltype(f)::value, decltype(c)::value,
                                    kExcBatchDeep>;
    });
  else
    launch_exc<false>(rgrid, r, r.f16, fromc, s, [](auto f, auto c) {
      return encode_exc_rows_kernel<decltype(f)::value, decltype(c)::value,
                                    kExcBatch>;
    });
  return hipGetLastError();
}

hipError_t launch_hash_blocks(const EncArgs &a, hipStream_t s) {
  by_class(a.log2B, [&](auto cls) {
    constexpr int K = decltype(cls)::value;
    constexpr uint32_t W = enc_waves(K);
    hipLaunchKernelGGL((encode_pass_kernel<false, kDetHashOnly, false, false,
                                           K>),
                       dim3((a.num_tiles + W - 1) / W), dim3(64 * W), 0, s, a);
  });
  return hipGetLastError();
}

hipError_t launch_encode_raw(const uint16_t *w, uint64_t n, uint32_t B,
                             uint8_t *out, uint64_t *out_bytes, bool f16,
                             hipStream_t s) {
  const uint32_t dtype = f16 ? kDtypeFp16 : kDtypeBf16;
  const uint64_t octets = (n + 7) / 8;
  uint64_t blocks = (octets + kThreads - 1) / kThreads;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(encode_raw_kernel, dim3(uint32_t(blocks)),
                     dim3(kThreads), 0, s, w, n, B, out, out_bytes, dtype);
  return hipGetLastError();
}

namespace {
template <int OCT, bool SMALL, bool RAWNT>
void launch_decode_tiles(const DecArgs &a, hipStream_t s) {
  constexpr uint64_t T = uint64_t(kThreads) * 8 * OCT;
  const dim3 grid(uint32_t((a.n + T - 1) / T), a.nshards);
  auto go = [&](auto upd) {
    constexpr bool U = decltype(upd)::value;
    auto k = a.log2B == 0 ? decode_elems_kernel<OCT, U, SMALL, RAWNT>
             : a.f16      ? decode_kernel<OCT, U, true, RAWNT>
                          : decode_kernel<OCT, U, false, RAWNT>;
    hipLaunchKernelGGL(k, grid, dim3(kThreads), 0, s, a);
  };
  if (a.out == nullptr)
    go(bool_c<true>{});
  else
    go(bool_c<false>{});
}
}  // namespace

hipError_t launch_decode(const DecArgs &a, hipStream_t s) {
  const uint64_t tiles = dec_tiles(a.n);
  if (tiles == 0 || a.nshards == 0) return hipSuccess;
  if (dec_small(a.n, a.nshards, a.log2B, a.f16, a.out == nullptr)) {
    launch_decode_tiles<int(kDecOctSmall), true, false>(a, s);
    return hipGetLastError();
  }
  if (a.log2B == 0) {
    hipLaunchKernelGGL(count_tile_bits_kernel,
                       dim3(uint32_t((tiles + 3) / 4), a.nshards),
                       dim3(kThreads), 0, s, a, uint32_t(tiles));
    if (a.prefix_pass)
      hipLaunchKernelGGL(scan_counts_kernel, dim3(a.nshards),
                         dim3(kScanThreads), 0, s, a.tile_excl,
                         uint32_t(tiles), dec_count_stride(tiles));
  } else if (a.prefix_pass) {
    hipLaunchKernelGGL(tile_prefix_kernel, dim3(a.nshards), dim3(kScanThreads),
                       0, s, a);
  }
  if (raw_plain_loads(a.n, a.nshards))
    launch_decode_tiles<int(kDecOct), false, false>(a, s);
  else
    launch_decode_tiles<int(kDecOct), false, true>(a, s);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void *p, uint64_t bytes, hipStream_t s) {
  const uint64_t words = bytes / 4;
  if (words == 0) return hipSuccess;
  uint64_t blocks = (words + kThreads - 1) / kThreads;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(uint32_t(blocks)), dim3(kThreads),
                     0, s, static_cast<uint32_t *>(p), words);
  return hipGetLastError();
}

}  // namespace ciera
