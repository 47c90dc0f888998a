// Device helpers shared by the HIP sources.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

// Loads and stores at any address, in global memory and in LDS (one access
// each: the device takes unaligned ones)
typedef uint32_t u32x4 __attribute__((vector_size(16)));
typedef uint32_t u32x2 __attribute__((vector_size(8)));
template <class T> struct __attribute__((packed)) Any { T v; };
template <class T> __device__ __forceinline__ T ld_any(const uint8_t* p) { return reinterpret_cast<const Any<T>*>(p)->v; }
template <class T> __device__ __forceinline__ void st_any(uint8_t* p, T v) { reinterpret_cast<Any<T>*>(p)->v = v; }
__device__ __forceinline__ uint32_t ld32(const uint8_t* p) { return ld_any<uint32_t>(p); }
__device__ __forceinline__ uint64_t ld64(const uint8_t* p) { return ld_any<uint64_t>(p); }
__device__ __forceinline__ u32x4 ld128(const uint8_t* p) { return ld_any<u32x4>(p); }
// the first n <= 16 bytes of v to p
__device__ __forceinline__ void st_upto16(uint8_t* p, u32x4 v, uint32_t n) {
  if (n == 16) {
    st_any<u32x4>(p, v);
    return;
  }
  uint32_t a = v[0], b = v[1];
  if (n & 8) {
    st_any<u32x2>(p, (u32x2){a, b});
    p += 8;
    a = v[2];
    b = v[3];
  }
  if (n & 4) {
    st_any<uint32_t>(p, a);
    p += 4;
    a = b;
  }
  if (n & 2) {
    st_any<uint16_t>(p, (uint16_t)a);
    p += 2;
    a >>= 16;
  }
  if (n & 1) *p = (uint8_t)a;
}

}  // namespace
