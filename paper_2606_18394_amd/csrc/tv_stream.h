// Loads for data read exactly once (the vocabulary scans over logits): the
// non-temporal hint lets them stream past the caches instead of allocating
// lines that are never read again.  Measured on the greedy acceptance scan:
// 35.2 -> 32.4 us over 155.6 MB of bf16 logits (512 rows of 151936) and
// 60.2 -> 52.9 us over 311 MB (1024 rows).
//
// Rows of a vocabulary that is no multiple of 16 bytes start at any element.
// They are still read 16 bytes at a time: gfx950's global loads need no
// alignment, and from a 4-byte boundary they stream within 4% of the aligned
// rate (512 fp32 rows of 151935: 50.4 us in the greedy scan, of 151936: 48.6;
// one element per load: 114 us).  From a 2-byte boundary they are slower (1024
// bf16 rows of 151935: 64.4 us, of 151936: 50.3), so a bf16 row that starts on
// one leaves its first element out of its chunks (49.1 us; one element per
// load: 169 us).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tv {

typedef unsigned int stream_u32x4 __attribute__((ext_vector_type(4), aligned(1)));

// 16 bytes from any address
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  const stream_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const stream_u32x4*>(p));
  return uint4{v.x, v.y, v.z, v.w};
}
// A row of V logits as 16-byte chunks: elements [head, head + E * chunks), E
// the elements per chunk, and fewer than 2 E others: spare(t) is the t-th.
template <bool F32>
struct RowSpan {
  static constexpr int E = F32 ? 4 : 8;
  const char* first;  // of chunk 0
  int head, chunks, V;
  __device__ __forceinline__ RowSpan(const void* row, int V_)
      : head(!F32 && ((uintptr_t)row & 2) != 0), V(V_) {
    chunks = (V - head) / E;
    first = (const char*)row + head * 2;
  }
  __device__ __forceinline__ uint4 load(long long c) const { return load_stream16(first + c * 16); }
  __device__ __forceinline__ int index(long long c) const { return head + (int)c * E; }
  // index of the t-th element outside the chunks (V or more: no such element)
  __device__ __forceinline__ long long spare(int t) const {
    return t < head ? t : (long long)chunks * E + t;
  }
};

// logit i of a row, as fp32
template <bool F32>
__device__ __forceinline__ float load_logit_stream(const void* row, long long i) {
  if (F32) return __builtin_nontemporal_load(reinterpret_cast<const float*>(row) + i);
  return __uint_as_float(
      (unsigned int)__builtin_nontemporal_load(reinterpret_cast<const unsigned short*>(row) + i) << 16);
}

}  // namespace tv
