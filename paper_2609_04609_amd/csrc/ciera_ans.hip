// rANS coding of the exception section (Section 3.1: the changed blocks'
// exponents travel ANS-coded; the receiver ANS-decodes them before the
// ExpCache patch). Range ANS (Duda 2013) with 16-bit renormalisation and 64
// interleaved states per chunk (Giesen 2014): one wave codes one chunk of
// 4096 exception bytes, lane l owning the chunk's bytes l, l + 64, ... The
// format is given in include/ciera.h.
//
// Coding (ciera_ans_code), in place on an encoded shard:
//   ans_hist_kernel    byte histogram of the exception list, a row of counts
//                      per workgroup
//   ans_encode_kernel  every workgroup adds up the rows and quantises the
//                      frequencies (sum 4096) for itself, then every wave codes
//                      chunks backwards; words go to the end of the chunk's
//                      workspace slot, lane order within a step
//   ans_copy_kernel    every workgroup adds up the stream sizes: the size
//                      decision and its chunks' offsets; then section tables,
//                      header and the chunk streams (only when the coded
//                      section is smaller)
// or, for shards of up to kAnsSmallChunks chunks, all of it in one workgroup
// (ans_code_small_kernel). What the kernels compute again in every workgroup
// is less than a launch of one workgroup that computes it once: 4.5 to 5 us
// each for zeroing the counters, the table and the offsets.
// Decoding (inside ciera_decode_gathered / ciera_update_cache):
//   ans_decode_kernel    every chunk of every rANS-coded shard into the
//                        shard's exception list in the workspace; the decode
//                        kernel then reads the list from there.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "ciera.h"
#include "ciera_internal.h"

namespace ciera {

namespace {

#ifndef CIERA_ANS_DEC_THREADS
#define CIERA_ANS_DEC_THREADS 1024
#endif
// threads per rANS decode workgroup: its waves share one slot table
constexpr int kAnsDecThreads = CIERA_ANS_DEC_THREADS;

__device__ __forceinline__ void set_err(uint32_t *err, uint32_t bits) {
  __hip_atomic_fetch_or(err, bits, __ATOMIC_RELAXED,
                        __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t ld32(const uint8_t *p) {
  return *reinterpret_cast<const uint32_t *>(p);
}
__device__ __forceinline__ uint64_t ld64(const uint8_t *p) {
  return *reinterpret_cast<const uint64_t *>(p);
}

__host__ __device__ inline uint64_t exc_offset(uint64_t n, uint32_t log2B) {
  return kHeaderBytes + pad16(n) + pad16(bitmap_bytes(n, log2B));
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
}

// Workgroup-wide sum and exclusive scan of one value per thread, NW waves.
template <int NW>
__device__ uint32_t block_sum32(uint32_t v, uint32_t *s_red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if (lane == 0) s_red[wave] = v;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += s_red[w];
  return t;
}

template <int NW>
__device__ uint32_t block_excl_scan32(uint32_t v, uint32_t *s_red,
                                      uint32_t *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(inc, d, 64);
    if (lane >= d) inc += t;
  }
  __syncthreads();
  if (lane == 63) s_red[wave] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) before += s_red[w];
    all += s_red[w];
  }
  *total = all;
  return before + inc - v;
}

// The symbol (thread idx < 256) holding the largest v, the lowest on ties.
// Some v is above 0; threads past 255 pass 0.
template <int NW>
__device__ uint32_t block_argmax(uint64_t v, uint32_t idx, uint64_t *s_key) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t key = idx < 256 ? (v << 8) | uint64_t(255u - idx) : 0ull;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t o = __shfl_xor(key, off, 64);
    key = o > key ? o : key;
  }
  __syncthreads();
  if (lane == 0) s_key[wave] = key;
  __syncthreads();
  uint64_t best = s_key[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) best = s_key[w] > best ? s_key[w] : best;
  return 255u - uint32_t(best & 255u);
}

// ================================================================ coding ==

// The number of exception bytes to code, 0 for a shard that stays as it is.
__device__ __forceinline__ uint64_t ans_to_code(const AnsEncArgs &a) {
  const uint64_t E = ld64(a.enc + 32);
  if ((ld32(a.enc + 4) >> 16) != kModeCompressed ||
      ld32(a.enc + 12) != kDtypeBf16 || E > a.n)
    return 0;
  return E;
}

// Row g of the histogram: 256 counts at the start of chunk g's slot of words.
// A chunk's words end at most 64 * 49 words from the slot's end (each state
// takes up 16 bits a word and 12 bits a symbol), so coding leaves it alone.
__device__ __forceinline__ uint32_t *hist_row(const AnsEncArgs &a,
                                              uint32_t g) {
  return reinterpret_cast<uint32_t *>(a.words + uint64_t(g) * kAnsChunk);
}
static_assert((kAnsChunk - 64 * 49) * 2 >= 1024, "a row fits in front");

// The exponents of the changed blocks crowd into a few values, so the lanes
// of one instruction adding into a single LDS histogram would mostly hit the
// same counters. The workgroup keeps kHistCopies copies, thread t adding into
// copy t mod kHistCopies; a copy is 257 words long, so one symbol's counters
// in different copies fall in different LDS banks. Counts exception bytes
// first, first + stride, ... (16 at a time); s_h is zero before.
constexpr int kHistCopies = 16;
constexpr int kHistStride = 257;
__device__ __forceinline__ void hist_bytes(const uint8_t *exc, uint64_t E,
                                           uint64_t first, uint64_t stride,
                                           uint32_t *s_h) {
  uint32_t *const h = s_h + (threadIdx.x & (kHistCopies - 1)) * kHistStride;
  for (uint64_t i = first; i < E; i += stride) {
    if (i + 16 <= E) {
      const uint4 v = *reinterpret_cast<const uint4 *>(exc + i);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          atomicAdd(&h[(w[k] >> (8 * b)) & 255u], 1u);
    } else {
      for (uint64_t k = i; k < E; ++k) atomicAdd(&h[exc[k]], 1u);
    }
  }
}

// Bound by the latency of its loads until 4096 waves run: 128 workgroups of
// 512 threads left the coding of the OLMoE shard 2 us and of a shard with
// every exponent sent 8 us slower than 256 of 1024; more rows than that would
// cost the coder as much to add up.
constexpr int kHistThreads = 1024;
constexpr uint32_t kHistRows = 256;  // workgroups of ans_hist_kernel at most
__global__ __launch_bounds__(kHistThreads) void ans_hist_kernel(AnsEncArgs a) {
  __shared__ uint32_t s_h[kHistCopies * kHistStride];
  const uint64_t E = ans_to_code(a);
  if (E == 0) return;
  const int tid = threadIdx.x;
  for (int i = tid; i < kHistCopies * kHistStride; i += kHistThreads)
    s_h[i] = 0u;
  __syncthreads();
  hist_bytes(a.enc + exc_offset(a.n, a.log2B), E,
             (uint64_t(blockIdx.x) * kHistThreads + tid) * 16,
             uint64_t(gridDim.x) * kHistThreads * 16, s_h);
  __syncthreads();
  if (tid < 256) {
    uint32_t t = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) t += s_h[c * kHistStride + tid];
    hist_row(a, blockIdx.x)[tid] = t;
  }
}

// Thread s < 256 owns symbol s with count h (the others: h = 0). Quantisation:
// every present symbol gets max(1, floor(h_s M / E)); a deficit goes to the
// most frequent symbol, an excess comes off the largest frequency (lowest
// symbol on ties), never below 1, until the total is M. Returns the frequency;
// *cum its exclusive prefix sum.
struct TableScratch {
  uint32_t red[16];
  uint64_t key[16];
  uint32_t fbest;
};
template <int NW>
__device__ __forceinline__ uint32_t quantise(uint32_t h, uint64_t E,
                                             uint32_t *cum, TableScratch &t) {
  const uint32_t s = threadIdx.x;
  uint32_t f = 0;
  if (h) {
    const uint64_t q = (uint64_t(h) << kAnsScale) / E;
    f = q ? uint32_t(q) : 1u;
  }
  uint32_t sum = block_sum32<NW>(f, t.red);
  if (sum < kAnsM) {
    const uint32_t best = block_argmax<NW>(h, s, t.key);
    if (s == best) f += kAnsM - sum;
    sum = kAnsM;
  }
  while (sum > kAnsM) {
    const uint32_t best = block_argmax<NW>(f, s, t.key);
    if (s == best) t.fbest = f;
    __syncthreads();
    const uint32_t fbest = t.fbest;
    uint32_t take = sum - kAnsM;
    if (take > fbest - 1u) take = fbest - 1u;
    if (s == best) f -= take;
    sum -= take;
  }
  uint32_t total = 0;
  *cum = block_excl_scan32<NW>(f, t.red, &total);
  return f;
}

// A symbol's coding entry. x / f without a divide (Granlund and Montgomery
// 1994, division by invariant integers, Fig. 4.1): with l = ceil(log2 f) and
// m = floor(2^32 (2^l - f) / f) + 1 < 2^32, t = mulhi(x, m) gives
// x / f = (t + ((x - t) >> min(l, 1))) >> max(l - 1, 0) for every 32-bit x.
// y: the largest state that takes the symbol without a word, 2^20 f - 1;
// z: M - f; w: cum, the shifts at bits 16 and 20. Absent symbols (f = 0) are
// never coded.
__device__ __forceinline__ uint4 coding_entry(uint32_t f, uint32_t cum) {
  const uint32_t l = f > 1u ? 32u - uint32_t(__clz(f - 1u)) : 0u;
  const uint32_t m =
      f ? uint32_t(((((uint64_t(1) << l) - f) << 32) / f) + 1u) : 0u;
  const uint32_t sh1 = l < 1u ? l : 1u, sh2 = l > 1u ? l - 1u : 0u;
  return make_uint4(m, (f << 20) - 1u, kAnsM - f,
                    cum | (sh1 << 16) | (sh2 << 20));
}

// One wave codes chunk c backwards: its final states and its words (at the end
// of its slot) go to the workspace. Returns the words. A step's table entries
// do not depend on the states, so those of kAhead steps are read before the
// first of them is coded.
__device__ __forceinline__ uint32_t code_chunk(const AnsEncArgs &a, uint32_t c,
                                               const uint8_t *exc, uint64_t E,
                                               const uint4 *s_tab,
                                               uint8_t *s_sym) {
  constexpr int kAhead = 4;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t lo = uint64_t(c) * kAnsChunk;
  const uint32_t len = uint32_t(E - lo < kAnsChunk ? E - lo : kAnsChunk);
  __builtin_amdgcn_wave_barrier();  // the previous chunk's symbols are read
  if (len == kAnsChunk) {
    const uint4 *src = reinterpret_cast<const uint4 *>(exc + lo) + lane;
    uint4 *const dst = reinterpret_cast<uint4 *>(s_sym) + lane;
    const uint4 v0 = src[0], v1 = src[64], v2 = src[128], v3 = src[192];
    dst[0] = v0;
    dst[64] = v1;
    dst[128] = v2;
    dst[192] = v3;
  } else {
    for (uint32_t b = lane; b < len; b += 64) s_sym[b] = exc[lo + b];
  }
  __builtin_amdgcn_wave_barrier();
  uint32_t x = kAnsL;
  uint32_t p = kAnsChunk;  // the words of this chunk fill [p, kAnsChunk)
  uint16_t *const slot = a.words + lo;
  auto step = [&](uint4 e, bool live) {
    const bool emit = live && x > e.y;
    const uint64_t m = __ballot(emit);
    p -= uint32_t(__popcll(m));
    if (emit) {
      slot[p + lanes_below(m)] = uint16_t(x & 0xFFFFu);
      x >>= 16;
    }
    const uint32_t t = __umulhi(x, e.x);
    const uint32_t q = (t + ((x - t) >> ((e.w >> 16) & 1u))) >> (e.w >> 20);
    // q M + (x - q f) + cum (q < 2^20)
    const uint32_t xn = __umul24(q, e.z) + x + (e.w & 0xFFFFu);
    x = live ? xn : x;
  };
  int t = int(len / 64) - 1;
  if (len % 64) {  // only the last chunk's first step
    const uint32_t i = uint32_t(t + 1) * 64 + lane;
    step(s_tab[i < len ? s_sym[i] : 0u], i < len);
  }
  for (; t >= kAhead - 1; t -= kAhead) {
    uint4 e[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      e[k] = s_tab[s_sym[uint32_t(t - k) * 64 + lane]];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) step(e[k], true);
  }
  for (; t >= 0; --t) step(s_tab[s_sym[uint32_t(t) * 64 + lane]], true);
  a.states[uint64_t(c) * 64 + lane] = x;
  const uint32_t words = kAnsChunk - p;
  if (lane == 0) a.counts[c] = words;
  return words;
}

// A wave codes chunk (round * grid + workgroup) * waves + wave. Bound by
// latency: the chain of 64 state updates, after the histogram rows.
// OLMoE shard (10.1 MB of exceptions): the three kernels take 35 us, against 52
// for a counter fill, histogram with global atomics, table, coder, offsets and
// copy in six launches; 16 x 131,072 values with every block sent, coded and
// decoded with the rest of the step, 47 against 62 us.
constexpr int kCodeThreads = 512;
constexpr uint32_t kCodeWaves = kCodeThreads / 64;
__global__ __launch_bounds__(kCodeThreads) void ans_encode_kernel(
    AnsEncArgs a, uint32_t rows) {
  __shared__ uint4 s_tab[256];
  __shared__ __align__(16) uint8_t s_sym[kCodeWaves][kAnsChunk];
  __shared__ TableScratch s_t;
  const uint32_t tid = threadIdx.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t E = ans_to_code(a);
  const uint32_t K = uint32_t((E + kAnsChunk - 1) / kAnsChunk);
  if (blockIdx.x == 0 && tid == 0) a.ans->K = K;
  if (blockIdx.x * kCodeWaves >= K) return;
  // the rows, two threads a symbol, through the LDS the symbols take later
  uint32_t h = 0;
  {
    constexpr uint32_t kParts = kCodeThreads / 256;
    const uint32_t s = tid & 255u;
#pragma unroll 32
    for (uint32_t g = tid >> 8; g < rows; g += kParts) h += hist_row(a, g)[s];
    uint32_t *const part = reinterpret_cast<uint32_t *>(&s_sym[0][0]);
    part[tid] = h;
    __syncthreads();
    h = 0;
    if (tid < 256)
#pragma unroll
      for (uint32_t q = 0; q < kParts; ++q) h += part[q * 256 + tid];
  }
  uint32_t cum;
  const uint32_t f = quantise<kCodeWaves>(h, E, &cum, s_t);
  if (tid < 256) {
    s_tab[tid] = coding_entry(f, cum);
    if (blockIdx.x == 0) a.ans->freq[tid] = f;
  }
  __syncthreads();
  const uint8_t *exc = a.enc + exc_offset(a.n, a.log2B);
  for (uint32_t c = blockIdx.x * kCodeWaves + wave; c < K;
       c += gridDim.x * kCodeWaves)
    code_chunk(a, c, exc, E, s_tab, s_sym[wave]);
}

// Bytes of chunk c's stream: the states and its words, padded to 4 bytes.
__device__ __forceinline__ uint32_t stream_bytes(uint32_t words) {
  return (256u + 2u * words + 3u) & ~3u;
}

// One wave copies chunk c's stream to the section, start bytes into the
// streams; the last chunk (end bytes in) also zeroes the section's padding.
__device__ __forceinline__ void copy_chunk(const AnsEncArgs &a, uint32_t c,
                                           uint32_t K, uint8_t *sec,
                                           uint32_t start, uint32_t end,
                                           uint32_t words) {
  const uint32_t lane = threadIdx.x & 63;
  uint8_t *const dst = sec + kAnsFixed + 4ull * K + start;
  reinterpret_cast<uint32_t *>(dst)[lane] = a.states[uint64_t(c) * 64 + lane];
  const uint16_t *src = a.words + uint64_t(c) * kAnsChunk + (kAnsChunk - words);
  uint16_t *d16 = reinterpret_cast<uint16_t *>(dst + 256);
  // 8 words a lane (16-byte accesses at the 2- and 4-byte aligned places that
  // they start at), then the last few
  typedef uint32_t words8_t __attribute__((ext_vector_type(4), aligned(2)));
  const uint32_t whole = words & ~7u;
#pragma unroll 2
  for (uint32_t k = lane * 8; k < whole; k += 512)
    *reinterpret_cast<words8_t *>(d16 + k) =
        *reinterpret_cast<const words8_t *>(src + k);
  if (whole + lane < words) d16[whole + lane] = src[whole + lane];
  if ((words & 1u) && lane == 0) d16[words] = 0;
  if (c == K - 1) {
    const uint64_t C = kAnsFixed + 4ull * K + end;
    for (uint64_t b = C + lane; b < pad16(C); b += 64) sec[b] = 0;
  }
}

// The coded section's fixed part and the shard's new header fields, by the
// first 256 threads (freq: symbol tid's frequency).
__device__ __forceinline__ void put_section(const AnsEncArgs &a, uint32_t K,
                                            uint8_t *sec, uint64_t C,
                                            uint32_t freq) {
  const uint32_t tid = threadIdx.x;
  const uint64_t bm = bitmap_bytes(a.n, a.log2B);
  if (tid < 256) reinterpret_cast<uint16_t *>(sec + 8)[tid] = uint16_t(freq);
  if (tid == 0) {
    reinterpret_cast<uint32_t *>(sec)[0] = K;
    reinterpret_cast<uint32_t *>(sec)[1] = kAnsChunk;
    const uint64_t total = kHeaderBytes + pad16(a.n) + pad16(bm) + pad16(C);
    reinterpret_cast<uint32_t *>(a.enc)[1] = kVersion | (kModeAns << 16);
    reinterpret_cast<uint64_t *>(a.enc)[5] = a.n + bm + C;
    reinterpret_cast<uint64_t *>(a.enc)[6] = total;
    if (a.out_bytes) *a.out_bytes = total;
  }
}

// Workgroup b copies chunks [b per, (b + 1) per). The header's mode, P and
// total change under the other workgroups, which read none of them.
__global__ __launch_bounds__(kThreads) void ans_copy_kernel(AnsEncArgs a) {
  constexpr int NW = kThreads / 64;
  __shared__ uint32_t s_red[NW];
  __shared__ uint32_t s_start[kThreads + 1];
  const uint32_t tid = threadIdx.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t K = a.ans->K;
  if (K == 0) {
    if (blockIdx.x == 0 && tid == 0 && a.out_bytes)
      *a.out_bytes = ld64(a.enc + 48);
    return;
  }
  const uint32_t per = (K + gridDim.x - 1) / gridDim.x;
  const uint32_t k0 = min(blockIdx.x * per, K), k1 = min(k0 + per, K);
  if (k0 == k1 && blockIdx.x) return;
  // stream dwords in front of k0, and in all. In bytes the sum of a list of
  // nearly 2^32 that does not compress would pass 2^32; streams are whole
  // dwords, and 2^20 of at most kAnsStreamMax bytes stay below that. Byte
  // offsets fit 32 bits once C < E.
  static_assert((kAnsStreamMax / 4ull) << 20 < 1ull << 32, "sum in dwords");
  uint32_t front = 0, all = 0;
#pragma unroll 8
  for (uint32_t c = tid; c < K; c += kThreads) {
    const uint32_t d = stream_bytes(a.counts[c]) >> 2;
    all += d;
    front += c < k0 ? d : 0u;
  }
  all = block_sum32<NW>(all, s_red);
  front = 4u * block_sum32<NW>(front, s_red);
  const uint64_t E = ld64(a.enc + 32);
  const uint64_t C = kAnsFixed + 4ull * K + 4ull * all;
  if (C >= E) {
    if (blockIdx.x == 0 && tid == 0 && a.out_bytes)
      *a.out_bytes = ld64(a.enc + 48);
    return;
  }
  uint8_t *const sec = a.enc + exc_offset(a.n, a.log2B);
  uint32_t *const ends = reinterpret_cast<uint32_t *>(sec + kAnsFixed);
  if (blockIdx.x == 0) put_section(a, K, sec, C, a.ans->freq[tid]);
  for (uint32_t r0 = k0; r0 < k1; r0 += kThreads) {
    const uint32_t c = r0 + tid;
    const uint32_t b = c < k1 ? stream_bytes(a.counts[c]) : 0u;
    uint32_t sum = 0;
    const uint32_t at = front + block_excl_scan32<NW>(b, s_red, &sum);
    s_start[tid] = at;
    if (c < k1) ends[c] = at + b;
    front += sum;
    if (tid == 0) s_start[kThreads] = front;
    __syncthreads();
    for (uint32_t i = wave; i < kThreads && r0 + i < k1; i += NW)
      copy_chunk(a, r0 + i, K, sec, s_start[i], s_start[i + 1],
                 a.counts[r0 + i]);
    __syncthreads();
  }
}

// All of it for shards of up to kAnsSmallChunks chunks (65,536 values), a wave
// a chunk. One CU's time grows with the exceptions, so with the share of blocks
// that changed. Three launches / one from a HIP graph, in us:
//   values                  16,384       32,768       49,152       65,536
//   40 to 50% changed    14.7 / 11.5  16.5 / 12.2  18.6 / 13.9  18.0 / 14.2
//   all changed          16.4 / 12.4  18.1 / 15.5  18.7 / 17.9  18.6 / 21.0
// The line is a workgroup's 16 waves: tensors that keep about half of their
// blocks gain on all of the range, those that keep none up to 49,152 values.
constexpr uint32_t kAnsSmallChunks = 16;
__global__ __launch_bounds__(64 * kAnsSmallChunks) void ans_code_small_kernel(
    AnsEncArgs a) {
  constexpr int NW = int(kAnsSmallChunks);
  __shared__ uint4 s_tab[256];
  __shared__ __align__(16) uint8_t s_sym[NW][kAnsChunk];
  __shared__ TableScratch s_t;
  __shared__ uint32_t s_words[NW];
  const uint32_t tid = threadIdx.x;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t E = ans_to_code(a);
  const uint32_t K = uint32_t((E + kAnsChunk - 1) / kAnsChunk);
  if (K == 0) {
    if (tid == 0 && a.out_bytes) *a.out_bytes = ld64(a.enc + 48);
    return;
  }
  uint8_t *const sec = a.enc + exc_offset(a.n, a.log2B);
  uint32_t *const s_h = reinterpret_cast<uint32_t *>(&s_sym[0][0]);
  static_assert(sizeof(s_sym) >= 4 * kHistCopies * kHistStride, "histogram");
  for (uint32_t i = tid; i < kHistCopies * kHistStride; i += 64 * NW)
    s_h[i] = 0u;
  __syncthreads();
  hist_bytes(sec, E, uint64_t(tid) * 16, uint64_t(64 * NW) * 16, s_h);
  __syncthreads();
  uint32_t h = 0, cum;
  if (tid < 256)
    for (int c = 0; c < kHistCopies; ++c) h += s_h[c * kHistStride + tid];
  const uint32_t f = quantise<NW>(h, E, &cum, s_t);
  if (tid < 256) s_tab[tid] = coding_entry(f, cum);
  __syncthreads();
  const uint32_t words =
      wave < K ? code_chunk(a, wave, sec, E, s_tab, s_sym[wave]) : 0u;
  if ((tid & 63) == 0) s_words[wave] = words;
  __syncthreads();  // and every symbol has been read
  uint32_t start = 0, all = 0;
#pragma unroll
  for (uint32_t w = 0; w < uint32_t(NW); ++w) {
    const uint32_t b = w < K ? stream_bytes(s_words[w]) : 0u;
    start += w < wave ? b : 0u;
    all += b;
  }
  const uint64_t C = kAnsFixed + 4ull * K + all;
  if (C >= E) {
    if (tid == 0 && a.out_bytes) *a.out_bytes = ld64(a.enc + 48);
    return;
  }
  put_section(a, K, sec, C, f);
  if (wave < K) {
    const uint32_t end = start + stream_bytes(words);
    if ((tid & 63) == 0)
      reinterpret_cast<uint32_t *>(sec + kAnsFixed)[wave] = end;
    copy_chunk(a, wave, K, sec, start, end, words);
  }
}

// ============================================================== decoding ==

// A wave's chunk stream in LDS: up to kAnsStage bytes of words are staged
// whole, longer ones (over 6 bits a symbol) go through a ring of two 256-byte
// blocks in the same place.
constexpr uint32_t kAnsStage = 3072;

// Grid (workgroups per shard, shards). A workgroup checks its shard's coded
// section and builds the slot table in LDS; then every wave decodes chunks on
// its own (no further barrier). Any inconsistency sets CIERA_DEVERR_FORMAT;
// every access stays inside the section and the shard's exception list.
//
// Bound by the instructions of a step (64 symbols, one per lane), not by
// bandwidth: a step is 11 VALU, 2 LDS and 1 store. A slot's entry is
// symbol | (f mod 4096) << 8 | (slot - cum) << 20, so the next state is one
// multiply-add of two extracted fields; the one shard that f = 4096 leaves
// out, with a single symbol, never moves its states and is filled instead. A
// chunk's words are staged in LDS whole, so a step only adds the words it used
// to the count: no window to slide and no load to wait for behind the byte
// stores. OLMoE layer, 16 shards (161 M symbols): 78 us, against 98 with the
// words in a ring of two blocks, f - 1 in the entry (17 VALU a step) and the
// slots' symbols found by binary search.
template <int NT>
__global__ __launch_bounds__(NT) void ans_decode_kernel(DecArgs a) {
  constexpr int NW = NT / 64;
  static_assert(NT >= 256 && NT % 256 == 0, "a thread per symbol at least");
  constexpr uint32_t kLoads = kAnsStage / 256;  // dwords a lane, whole chunk
  constexpr uint32_t kUnroll = 8;               // steps per loop iteration
  // the waves' streams, then the slot table: a bad stream makes its wave read
  // at most 64 * 64 words on from its start, which is still in here
  __shared__ __align__(16) uint32_t s_mem[NW * kAnsStage / 4 + kAnsM];
  uint32_t *const s_slot = s_mem + NW * kAnsStage / 4;
  static_assert(kAnsM * 4 + kAnsStage >= (kAnsChunk + 64) * 2, "stays inside");
  __shared__ uint32_t s_freq[256];
  __shared__ uint32_t s_cum[256];
  __shared__ uint32_t s_red[4];
  __shared__ uint32_t s_top[NW];
  const uint32_t j = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  // wave-uniform, so that the chunk loop and its lengths stay scalar
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t *const words32 = s_mem + wave * int(kAnsStage / 4);
  const uint16_t *const words16 = reinterpret_cast<const uint16_t *>(words32);
  const uint64_t off = a.offsets ? a.offsets[j] : 0ull;
  // the decode kernel reports a misplaced shard
  if ((off & 15ull) || off > a.bytes || a.bytes - off < kHeaderBytes) return;
  const uint8_t *enc = a.gathered + off;
  const uint64_t n = a.n;
  const uint32_t vm = ld32(enc + 4);
  if (ld32(enc) != kMagic || (vm & 0xFFFFu) != kVersion ||
      (vm >> 16) != kModeAns || ld32(enc + 12) != kDtypeBf16 ||
      ld64(enc + 16) != n ||
      ld32(enc + 8) != (1u << a.log2B) || a.log2B < 4)
    return;
  const uint64_t E = ld64(enc + 32), P = ld64(enc + 40);
  const uint64_t bm = bitmap_bytes(n, a.log2B);
  if (E > n || P < n + bm + kAnsFixed) return;
  const uint64_t C = P - n - bm;
  const uint64_t htotal = ld64(enc + 48);
  if (htotal != kHeaderBytes + pad16(n) + pad16(bm) + pad16(C) ||
      htotal > a.bytes - off)
    return;
  const uint8_t *sec = enc + exc_offset(n, a.log2B);
  const uint32_t K = ld32(sec);
  const uint64_t want_k = (E + kAnsChunk - 1) / kAnsChunk;
  bool ok = K == want_k && ld32(sec + 4) == kAnsChunk &&
            C >= kAnsFixed + 4ull * K;
  // the 256 frequencies (the first four waves), their total and exclusive
  // prefix sums
  uint32_t f = 0, inc = 0;
  if (tid < 256) {
    f = reinterpret_cast<const uint16_t *>(sec + 8)[tid];
    s_freq[tid] = f;
    inc = f;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t t = __shfl_up(inc, d, 64);
      if (lane >= d) inc += t;
    }
    if (lane == 63) s_red[wave] = inc;
  }
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before += s_red[w];
    total += s_red[w];
  }
  if (tid < 256) s_cum[tid] = before + inc - f;
  ok = ok && total == kAnsM;
  if (!ok) {
    if (blockIdx.x == 0 && tid == 0) set_err(a.err, CIERA_DEVERR_FORMAT);
    return;
  }
  __syncthreads();
  // the symbol of every slot: symbol + 1 at each run's first slot, then a
  // running maximum over the slots, kPer consecutive ones a thread (a binary
  // search a slot over the prefix sums took a third of the kernel's time)
  constexpr uint32_t kPer = kAnsM / NT;
  static_assert(kPer % 4 == 0, "whole 16-byte vectors a thread");
  uint4 *const mine = reinterpret_cast<uint4 *>(s_slot) + tid * (kPer / 4);
#pragma unroll
  for (uint32_t q = 0; q < kPer / 4; ++q) mine[q] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  if (tid < 256 && f) s_slot[before + inc - f] = uint32_t(tid) + 1u;
  __syncthreads();
  uint32_t sym[kPer];
#pragma unroll
  for (uint32_t q = 0; q < kPer / 4; ++q) {
    const uint4 v = mine[q];
    sym[4 * q] = v.x;
    sym[4 * q + 1] = v.y;
    sym[4 * q + 2] = v.z;
    sym[4 * q + 3] = v.w;
  }
#pragma unroll
  for (uint32_t q = 1; q < kPer; ++q) sym[q] = max(sym[q], sym[q - 1]);
  uint32_t top = sym[kPer - 1];  // the maximum up to this thread, in its wave
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(top, d, 64);
    if (lane >= d) top = max(top, t);
  }
  if (lane == 63) s_top[wave] = top;
  __syncthreads();
  uint32_t front = __shfl_up(top, 1, 64);
  if (lane == 0) front = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wave) front = max(front, s_top[w]);
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t s = max(sym[q], front) - 1u;
    const uint32_t slot = uint32_t(tid) * kPer + q;
    sym[q] = s | ((s_freq[s] & (kAnsM - 1u)) << 8) | ((slot - s_cum[s]) << 20);
  }
#pragma unroll
  for (uint32_t q = 0; q < kPer / 4; ++q)
    mine[q] = make_uint4(sym[4 * q], sym[4 * q + 1], sym[4 * q + 2],
                         sym[4 * q + 3]);
  __syncthreads();
  // f = 4096: the only symbol, in every slot
  const uint32_t only = __builtin_amdgcn_readfirstlane(s_slot[0] & 255u);
  const bool single = s_freq[only] == kAnsM;
  const uint32_t *ends = reinterpret_cast<const uint32_t *>(sec + kAnsFixed);
  const uint8_t *streams = sec + kAnsFixed + 4ull * K;
  const uint64_t avail = C - kAnsFixed - 4ull * K;
  uint8_t *const list = a.ans_exc + uint64_t(j) * a.ans_stride;

  for (uint32_t c = blockIdx.x * NW + uint32_t(wave); c < K;
       c += gridDim.x * NW) {
    const uint32_t start = c ? ends[c - 1] : 0u;
    const uint32_t end = ends[c];
    if (!(start <= end && end <= avail && ((start | end) & 3u) == 0 &&
          end - start >= 256u && end - start <= kAnsStreamMax)) {
      if (lane == 0) set_err(a.err, CIERA_DEVERR_FORMAT);
      continue;
    }
    const uint8_t *st = streams + start;
    const uint32_t wbytes = end - start - 256u;  // words and padding
    const uint32_t nwords = wbytes / 2u;
    const uint8_t *wsrc = st + 256;
    // block b of the words: 256 bytes, a dword a lane
    auto block = [&](uint32_t b) -> uint32_t {
      const uint32_t o = b * 256u + 4u * uint32_t(lane);
      return o < wbytes ? ld32(wsrc + o) : 0u;
    };
    uint32_t x = ld32(st + 4u * uint32_t(lane));
    {
      uint32_t w[kLoads];
#pragma unroll
      for (uint32_t q = 0; q < kLoads; ++q) w[q] = block(q);
      __builtin_amdgcn_wave_barrier();  // the previous chunk's reads are done
#pragma unroll
      for (uint32_t q = 0; q < kLoads; ++q) words32[q * 64 + lane] = w[q];
      __builtin_amdgcn_wave_barrier();
    }
    const uint64_t lo = uint64_t(c) * kAnsChunk;
    const uint32_t len = uint32_t(E - lo < kAnsChunk ? E - lo : kAnsChunk);
    uint8_t *dst = list + lo;
    bool bad = x < kAnsL;
    uint32_t rd = 0;
    // 64 symbols a step, one per lane; only the last step of the last chunk
    // can be partial (TAIL)
    auto state = [&](uint32_t e) {
      return __umul24((e >> 8) & (kAnsM - 1u), x >> kAnsScale) + (e >> 20);
    };
    auto step = [&](uint32_t t, auto tail) {
      constexpr bool TAIL = decltype(tail)::value;
      const uint32_t i = t * 64 + uint32_t(lane);
      const bool live = !TAIL || i < len;
      const uint32_t e = s_slot[x & (kAnsM - 1u)];
      const uint32_t xd = state(e);
      if (live) dst[i] = uint8_t(e);
      x = live ? xd : x;
      const bool need = live && x < kAnsL;
      const uint64_t m = __ballot(need);
      // word rd + (needing lanes below); past a bad stream's end some other
      // LDS of this block is read, and the check after the chunk fails
      const uint32_t w = words16[rd + lanes_below(m)];
      x = need ? ((x << 16) | w) : x;
      rd += uint32_t(__popcll(m));
    };
    // the same with the words in a ring of two blocks of 128 words: the next
    // block is loaded ahead into a register and written over the one that the
    // window leaves
    uint32_t base = 0, next = 3, pre = 0;  // base: the window's first word
    auto ring_step = [&](uint32_t t, auto tail) {
      constexpr bool TAIL = decltype(tail)::value;
      const uint32_t i = t * 64 + uint32_t(lane);
      const bool live = !TAIL || i < len;
      const uint32_t e = s_slot[x & (kAnsM - 1u)];
      const uint32_t xd = state(e);
      if (live) dst[i] = uint8_t(e);
      x = live ? xd : x;
      const bool need = live && x < kAnsL;
      const uint64_t m = __ballot(need);
      // word w of the stream sits at w mod 256 of the ring (rd - base < 128)
      const uint32_t w = words16[(rd + lanes_below(m)) & 255u];
      x = need ? ((x << 16) | w) : x;
      rd += uint32_t(__popcll(m));
      if (rd - base >= 128u) {  // uniform: slide the window by one block
        __builtin_amdgcn_wave_barrier();
        words32[((base >> 7) & 1u) * 64u + uint32_t(lane)] = pre;
        __builtin_amdgcn_wave_barrier();
        pre = block(next++);
        base += 128u;
      }
    };
    const uint32_t full = len / 64;
    if (single) {
      for (uint32_t i = uint32_t(lane); i < len; i += 64)
        dst[i] = uint8_t(only);
    } else if (wbytes <= kAnsStage) {
      uint32_t t = 0;
      for (; t + kUnroll <= full; t += kUnroll) {
#pragma unroll
        for (uint32_t u = 0; u < kUnroll; ++u)
          step(t + u, std::integral_constant<bool, false>{});
      }
      for (; t < full; ++t) step(t, std::integral_constant<bool, false>{});
      if (len % 64) step(full, std::integral_constant<bool, true>{});
    } else {
      pre = block(2);
#pragma unroll 1
      for (uint32_t t = 0; t < full; ++t)
        ring_step(t, std::integral_constant<bool, false>{});
      if (len % 64) ring_step(full, std::integral_constant<bool, true>{});
    }
    // every state back at L, the words used up exactly (none read past the
    // stream's end), only zero padding after
    bad = bad || x != kAnsL;
    const uint32_t used = 256u + 2u * rd;
    if (((used + 3u) & ~3u) != end - start) bad = true;
    else if (rd < nwords &&
             reinterpret_cast<const uint16_t *>(wsrc)[rd] != 0)
      bad = true;
    if (__ballot(bad) != 0ull && lane == 0) set_err(a.err, CIERA_DEVERR_FORMAT);
  }
}

}  // namespace

hipError_t launch_ans_code(const AnsEncArgs &a, hipStream_t s) {
  if (a.kmax == 0) return hipSuccess;
  if (a.kmax <= kAnsSmallChunks) {
    hipLaunchKernelGGL(ans_code_small_kernel, dim3(1),
                       dim3(64 * kAnsSmallChunks), 0, s, a);
    return hipGetLastError();
  }
  const uint32_t rows = std::min(a.kmax / 4 + 1, kHistRows);
  const uint32_t g =
      std::min((a.kmax + kCodeWaves - 1) / kCodeWaves, uint32_t(512));
  hipLaunchKernelGGL(ans_hist_kernel, dim3(rows), dim3(kHistThreads), 0, s, a);
  hipLaunchKernelGGL(ans_encode_kernel, dim3(g), dim3(kCodeThreads), 0, s, a,
                     rows);
  hipLaunchKernelGGL(ans_copy_kernel, dim3(std::min(a.kmax / 4 + 1, 1024u)),
                     dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ans_decode(const DecArgs &a, hipStream_t s) {
  if (a.ans_exc == nullptr || a.nshards == 0) return hipSuccess;
  const uint64_t kmax = ans_kmax(a.n);
  if (kmax == 0) return hipSuccess;
  // about 8192 waves over all shards
  constexpr int NT = kAnsDecThreads;
  constexpr uint32_t kGroups = 8192u / (NT / 64);
  uint64_t g = (kGroups + a.nshards - 1) / a.nshards;
  const uint64_t need = (kmax + NT / 64 - 1) / (NT / 64);
  if (g > need) g = need;
  if (g == 0) g = 1;
  hipLaunchKernelGGL(ans_decode_kernel<NT>, dim3(uint32_t(g), a.nshards),
                     dim3(NT), 0, s, a);
  return hipGetLastError();
}

}  // namespace ciera
