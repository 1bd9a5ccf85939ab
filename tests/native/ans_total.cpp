// The rANS size decision for incompressible lists close to 2^32 bytes, in the
// host model: workgroup 0 of the copy kernel alone, on sparse memory (its
// neighbours would decide alike). Prints, for each words-a-chunk given, the
// shard's mode and size afterwards.
#include "ciera_ans.hip"

using namespace ciera;

static void *sparse(uint64_t bytes) {
  void *p = mmap(nullptr, bytes, PROT_READ | PROT_WRITE,
                 MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (p == MAP_FAILED) abort();
  return p;
}

int main(int argc, char **argv) {
  const uint64_t n = 0xFFFFFF00ull;
  const uint32_t log2B = 9;
  const uint64_t raw =
      kHeaderBytes + pad16(n) + pad16(bitmap_bytes(n, log2B)) + pad16(n);
  const uint32_t K = uint32_t(ans_kmax(n));
  for (int i = 1; i < argc; ++i) {
    uint64_t out_bytes = 0;
    AnsEncArgs a{};
    a.enc = static_cast<uint8_t *>(sparse(raw));
    a.n = n;
    a.log2B = log2B;
    a.kmax = K;
    a.out_bytes = &out_bytes;
    a.ans = static_cast<AnsCtl *>(sparse(sizeof(AnsCtl)));
    a.counts = static_cast<uint32_t *>(sparse(4ull * K));
    a.states = static_cast<uint32_t *>(sparse(256ull * K));
    a.words = static_cast<uint16_t *>(sparse(2ull * kAnsChunk * K));
    uint32_t *const h32 = reinterpret_cast<uint32_t *>(a.enc);
    uint64_t *const h64 = reinterpret_cast<uint64_t *>(a.enc);
    h32[1] = kVersion | (kModeCompressed << 16);
    h64[2] = n;
    h64[4] = n;  // E: every block changed
    h64[6] = raw;
    a.ans->K = K;
    for (uint32_t c = 0; c < K; ++c) a.counts[c] = uint32_t(atol(argv[i]));
    wave_host::max_groups = 1;
    hipLaunchKernelGGL(ans_copy_kernel, dim3(1024), dim3(kThreads), 0,
                       nullptr, a);
    printf("%u %llu\n", h32[1] >> 16, (unsigned long long)out_bytes);
    munmap(a.enc, raw);
    munmap(a.words, 2ull * kAnsChunk * K);
    munmap(a.states, 256ull * K);
  }
  return 0;
}
