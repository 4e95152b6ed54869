// cf_fine_reg.h -- shared by the simulators that keep their control state in
// registers (k_fine_reg.hip, k_fine_gate.hip): lane reads and writes, the
// request block and its attributes.
#pragma once
#include "cf_fine.h"

namespace cf {
namespace fine {

// A request's block: executors of its path (byte c, 0xFF off the path), join
// counters (4 bits per component), outputs left (4 bits) and type (bits
// 8..10); its length attributes; first token time and output tokens of its
// TTFT stage; last token and media times.
struct __attribute__((aligned(64))) RReq {
  uint64_t ex;
  uint32_t join, misc;
  uint32_t attr[4];  // prompt | out << 16, patches, audio in ms, audio out ms
  double tfirst;
  uint32_t n1, pad;
  double tlast, tmedia;
};
static_assert(sizeof(RReq) == 64, "request block");
constexpr uint32_t kOffAttr = 16, kOffTim = 32, kOffLast = 48;

// info word of a (component, type) pair
constexpr uint32_t IN_TTFT = 1u << 8;   // c is the type's TTFT stage
constexpr uint32_t IN_OUT = 1u << 9;    // c is one of its outputs
constexpr uint32_t IN_PFO = 1u << 10;   // c emits one token for it
constexpr uint32_t IN_GENO = 1u << 11;  // the type has a GEN output
constexpr uint32_t IN_LLM = 1u << 12;   // the type has a TTFT stage
// the compiler's lane write (lane and value wave-uniform); it has no builtin
extern "C" __device__ int cf_writelane(int x, int lane, int v) __asm("llvm.amdgcn.writelane.i32");

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ uint32_t rl(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
// v as a value of its own per lane: the compiler derives from a lane write's
// arguments whether its result is the same in every lane, so a register that
// starts uniform and only sees lane writes would be taken for uniform
__device__ __forceinline__ uint32_t per_lane(uint32_t v) {
  asm("" : "+v"(v));
  return v;
}
__device__ __forceinline__ double per_lane(double v) {
  asm("" : "+v"(v));
  return v;
}
__device__ __forceinline__ void wl(uint32_t &v, int lane, uint32_t x) {
  v = per_lane((uint32_t)cf_writelane((int)x, lane, (int)v));
}
__device__ __forceinline__ void wld(double &v, int lane, double x) {
  const uint64_t o = (uint64_t)__double_as_longlong(v), n = ru64((uint64_t)__double_as_longlong(x));
  uint32_t lo = (uint32_t)o, hi = (uint32_t)(o >> 32);
  wl(lo, lane, (uint32_t)n);
  wl(hi, lane, (uint32_t)(n >> 32));
  v = __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ uint64_t rl64(uint64_t v, int lane) {
  return ((uint64_t)rl((uint32_t)(v >> 32), lane) << 32) | rl((uint32_t)v, lane);
}
__device__ __forceinline__ int ff1(uint64_t m) { return __builtin_ctzll(m); }  // m != 0
__device__ __forceinline__ double words_double(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The launch's arguments in the constant address space (scalar loads), read
// where they are used: without the barrier the compiler loads every field
// ahead of the event loop and spills the scalar registers.
typedef const __attribute__((address_space(4))) FineArgs CArgs;
typedef const __attribute__((address_space(4))) KModel CModel;
__device__ __forceinline__ CArgs &args(const FineArgs *p) {
  CArgs *A = (CArgs *)p;
  asm volatile("" : "+s"(A));
  return *A;
}

// attribute a (wave-uniform) of a request's attributes w
__device__ __forceinline__ uint32_t attr_in(const u32x4 &w, uint32_t a) {
  uint32_t v;
  if (a < CF_ATTR_AUDIN_MS) {
    v = a == CF_ATTR_PATCHES ? w.y : w.x;
    v = a == CF_ATTR_OUT ? v >> 16 : v & 0xFFFFu;
  } else {
    v = (a & 1u) ? w.z : w.w;
    if (a >= CF_ATTR_AUDIN_TOK) v = (v + 79u) / 80u;
  }
  return v;
}
// the sum of the attributes in sel (wave-uniform): the 16-bit ones by dot
// products with 0/1 weights, the 32-bit ones under masks
__device__ __forceinline__ uint32_t x_in(const u32x4 &w, uint32_t sel) {
  typedef unsigned short us2 __attribute__((ext_vector_type(2)));
  const uint32_t p0 = (sel & 1u) | ((sel & 2u) << 15), p1 = (sel >> 2) & 1u;
  uint32_t x = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, (uint32_t)w.y), __builtin_bit_cast(us2, p1), 0u, false);
  x = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, (uint32_t)w.x), __builtin_bit_cast(us2, p0), x, false);
  if (sel & 0x78u) {
    if (sel & 0x08u) x += w.z;
    if (sel & 0x10u) x += w.w;
    if (sel & 0x20u) x += (w.z + 79u) / 80u;
    if (sel & 0x40u) x += (w.w + 79u) / 80u;
  }
  return x;
}

}  // namespace fine
}  // namespace cf
