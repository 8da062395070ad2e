// device.h -- device functions shared by the fixpoint kernels: wave sums, the
// block order over the XCDs, and the device-scope accesses that hand data from
// one workgroup of a launch to another.
#pragma once

#include "common.h"

namespace dl {

// 16 bytes at any address: one global access each (the compiler knows the
// alignment; the memory system splits what crosses a line).  A caller's rows
// are rarely aligned: their stride is often n itself.
typedef u32x4 u32x4_any __attribute__((aligned(1)));
__device__ inline u32x4 load16_any(const uint8_t* p) { return *(const u32x4_any*)p; }
__device__ inline void store16_any(uint8_t* p, u32x4 v) { *(u32x4_any*)p = v; }

// Nonzero bytes as ones: each byte's bits folded into its bit 0.
__device__ inline u32x4 bytes01(u32x4 x) {
  x |= x >> 4;
  x |= x >> 2;
  x |= x >> 1;
  return x & 0x01010101u;
}

// 16 bytes as 16 bits (nonzero or not), and back to 0/1 bytes.
__device__ inline unsigned bit16_of_bytes(u32x4 x) {
  const u32x4 b = bytes01(x);
  unsigned m = 0u;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    unsigned v = b[w];
    v |= v >> 7;
    v |= v >> 14;
    m |= (v & 15u) << (4 * w);
  }
  return m;
}

__device__ inline u32x4 bytes_of_bit16(unsigned m) {
  u32x4 x;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const unsigned v = (m >> (4 * w)) & 15u;
    x[w] = (v * 0x00204081u) & 0x01010101u;
  }
  return x;
}

__device__ inline int wave_sum(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Block index -> logical index.  The hardware deals workgroups round-robin
// over the 8 XCDs (block b on XCD b % 8); the blocks of XCD x get the
// contiguous run of logical indices [x q + min(x, r), ...), q = nblocks / 8,
// r = nblocks % 8 (a bijection on [0, nblocks) for any nblocks).
__device__ inline int xcd_logical(int b, int nblocks) {
  const int q = nblocks >> 3, r = nblocks & 7;
  const int x = b & 7, local = b >> 3;
  return x * q + (x < r ? x : r) + local;
}

__device__ inline unsigned ld_agent(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long ld_agent64(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_agent(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Stores to host memory that the host polls: system scope, so that a wait for
// them (wait_stores) means the host can see them.  Plain stores may still sit
// in the L2 then, and the host saw a status word before the results it
// announces (once in about 80 thousand calls).
__device__ inline void st_system(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ inline void st_system64(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Waits until this wave's stores and atomics have completed.
__device__ inline void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Device-scope (write-through, sc1) stores of 16 and 8 bytes at byte offset
// off of a buffer (buffer instructions: the compiler knows them as stores
// and keeps the wait states their data registers need).
constexpr int kCpolSc1 = 16;  // cache-policy bits of a device-scope access
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000);
}
__device__ inline void st_agent_x4(__amdgpu_buffer_rsrc_t r, int off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, kCpolSc1);
}
__device__ inline void st_agent_x2(__amdgpu_buffer_rsrc_t r, int off, unsigned lo, unsigned hi) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 v = {lo, hi};
  __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, kCpolSc1);
}

// The same for a caller's buffer, of any alignment: the first `count` bytes
// of v at p.  A kernel whose status word ends the call stores its results so:
// a plain store may sit in its XCD's L2 until the launch ends, where other
// streams do not see it.
__device__ inline void st_agent_u8(uint8_t* p, unsigned v) {
  __hip_atomic_store(p, (uint8_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store4_agent_any(uint8_t* p, unsigned v, int count) {
  if (count >= 4 && ((uintptr_t)p & 3) == 0) {
    st_agent((unsigned*)p, v);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < count) st_agent_u8(p + e, v >> (8 * e));
  }
}
__device__ inline void store16_agent_any(uint8_t* p, u32x4 v, int count) {
  const int head = (int)(-(uintptr_t)p & 3);
  if (count >= 16 && head != 0) {  // bytes up to a word, three words, the bytes left
#pragma unroll
    for (int w = 0; w < 3; ++w) st_agent((unsigned*)(p + head + 4 * w), __builtin_amdgcn_alignbyte(v[w + 1], v[w], head));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (e < head) st_agent_u8(p + e, v[0] >> (8 * e));
      else st_agent_u8(p + 12 + e, v[3] >> (8 * e));
    }
  } else {
#pragma unroll
    for (int w = 0; w < 4; ++w) store4_agent_any(p + 4 * w, v[w], count - 4 * w);
  }
}

}  // namespace dl
