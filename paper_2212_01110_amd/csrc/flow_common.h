// Copies into LDS and bounded waits for tagged values, shared by the two
// dataflow forms of the sweeps (flow.hip, walk.hip).
#pragma once
#include "device_common.h"

namespace spk {

namespace {

constexpr int kFW = 256;                   // threads per workgroup (4 wavefronts)

typedef __attribute__((address_space(3))) void lds_void;

// Copies nwords 32-bit words from global memory into LDS (dst = word
// offset, a multiple of 64). From a 16-byte aligned source, whole rows of
// 256 words go as 16 bytes per lane (lane l fills words 4l..4l+3 of the
// row); the rest (all of it from an unaligned source) goes in rows of 64
// words, 4 bytes per lane, lanes past the end re-reading the last word (in
// bounds) into the region's padding. Wavefront w issues rows w', w' + 4, ...
// (w' = w rotated by `rot`, so that small copies spread over the
// wavefronts).
__device__ __forceinline__ void dma_words(const void* src, unsigned* lds, int dst, int nwords, int rot) {
  const int lane = threadIdx.x & 63, w = ((threadIdx.x >> 6) + rot) & 3;
  // uniform base + 32-bit lane byte offset (scalar-base addressing)
  const char* s = static_cast<const char*>(src);
  int done = 0;
  if ((reinterpret_cast<uintptr_t>(src) & 15u) == 0) {
    const int rows = nwords >> 8;
    for (int r = w; r < rows; r += 4)
      __builtin_amdgcn_global_load_lds(s + (unsigned)((r * 256 + lane * 4) * 4), (lds_void*)(lds + dst + r * 256), 16, 0,
                                       0);
    done = rows << 8;
  }
  const int rest = nwords - done;
  for (int r = w; r * 64 < rest; r += 4) {
    int e = r * 64 + lane;
    e = e < rest ? e : rest - 1;
    __builtin_amdgcn_global_load_lds(s + (unsigned)((done + e) * 4), (lds_void*)(lds + dst + done + r * 64), 4, 0, 0);
  }
}

__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
}

__device__ __forceinline__ unsigned ld_flag(const unsigned* f) {
  return __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One wavefront polls the n tagged elements at src until all carry `tag`
// (bounded), copying the values to dst (LDS).
template <typename S>
__device__ __forceinline__ void wait_tagged(const unsigned long long* src, int n, unsigned tag, S* dst,
                                            unsigned* err, unsigned spin) {
  const int lane = threadIdx.x & 63;
  for (unsigned it = 0; it < spin; ++it) {
    bool ok = true;
    for (int e = lane; e < n; e += 64) {
      S v;
      ok = get_tagged<S>(src + (size_t)e * kTW<S>, tag, v) && ok;
      dst[e] = v;
    }
    if (__all(ok)) return;
    if ((it & 255u) == 255u && ld_flag(err) != 0u) return;
    __builtin_amdgcn_s_sleep(1);
  }
  __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Same for two sources at once (one memory round trip per poll).
template <typename S>
__device__ __forceinline__ void wait_tagged2(const unsigned long long* srcA, int nA, S* dstA,
                                             const unsigned long long* srcB, int nB, S* dstB, unsigned tag,
                                             unsigned* err, unsigned spin) {
  const int lane = threadIdx.x & 63;
  for (unsigned it = 0; it < spin; ++it) {
    bool ok = true;
    for (int e = lane; e < nA; e += 64) {
      S v;
      ok = get_tagged<S>(srcA + (size_t)e * kTW<S>, tag, v) && ok;
      dstA[e] = v;
    }
    for (int e = lane; e < nB; e += 64) {
      S v;
      ok = get_tagged<S>(srcB + (size_t)e * kTW<S>, tag, v) && ok;
      dstB[e] = v;
    }
    if (__all(ok)) return;
    if ((it & 255u) == 255u && ld_flag(err) != 0u) return;
    __builtin_amdgcn_s_sleep(1);
  }
  __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

}  // namespace spk
