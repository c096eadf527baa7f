// Device-side helpers shared by the gfx950 kernels: the fp64 MFMA tile type
// and the counter-based Philox4x32-10 generator used for Klein's draws.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ojbkq {

// Accumulator of one v_mfma_f64_16x16x4_f64: a 16x16 fp64 tile spread over a
// wave, four values per lane.  Lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] of the 16x4 and 4x16 operands and holds
// D[l / 16 + 4 r][l % 16], r = 0..3 (measured on gfx950).
typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
// 32x32->64-bit products (one v_mad_u64_u32 each) on a 128-bit counter, key
// bumped by the two Weyl constants between rounds.

// Uniform double in [0, 1) for the Klein draw of (row i, column j, candidate
// k): counter (i, j, k, 0), key (seed lo, seed hi), 53 bits from the first
// two words (27 high bits of x0, 26 high bits of x1).
__device__ __forceinline__ double uniform53(uint32_t x0, uint32_t x1) {
  const double hi = (double)(x0 >> 5);
  const double lo = (double)(x1 >> 6);
  return (hi * 67108864.0 + lo) * (1.0 / 9007199254740992.0);
}

// philox4x32_10 of those counters for a lane that walks the rows i: the first
// round's product with k and the second's with its result are the same for
// every row.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);   // one v_bitop3_b32
}
struct KleinLane {
  uint32_t lo1;        // low word of kM1 k
  uint32_t hi2, lo2;   // kM0 c0 of the second round
};
__device__ __forceinline__ KleinLane klein_lane(uint32_t j, uint32_t k, uint32_t k0) {
  const uint64_t p1 = 0xCD9E8D57ull * k;
  const uint64_t p0 = 0xD2511F53ull * ((uint32_t)(p1 >> 32) ^ j ^ k0);
  return KleinLane{(uint32_t)p1, (uint32_t)(p0 >> 32), (uint32_t)p0};
}
__device__ __forceinline__ void klein_words(const KleinLane& w, uint32_t i, uint32_t k0,
                                            uint32_t k1, uint32_t& x0, uint32_t& x1) {
  constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u;
  constexpr uint32_t kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
  // rounds one and two (the row's own words are the same for every lane)
  const uint64_t pi = (uint64_t)kM0 * i;
  const uint32_t c2i = (uint32_t)(pi >> 32) ^ k1;
  k0 += kW0;
  k1 += kW1;
  const uint64_t q1 = (uint64_t)kM1 * c2i;
  uint32_t c0 = (uint32_t)(q1 >> 32) ^ w.lo1 ^ k0, c1 = (uint32_t)q1;
  uint32_t c2 = w.hi2 ^ (uint32_t)pi ^ k1, c3 = w.lo2;
#pragma unroll
  for (int round = 2; round < 10; ++round) {
    k0 += kW0;
    k1 += kW1;
    const uint64_t p0 = (uint64_t)kM0 * c0, p1 = (uint64_t)kM1 * c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c0 = n0;
    c1 = (uint32_t)p1;
    c2 = n2;
    c3 = (uint32_t)p0;
  }
  x0 = c0;
  x1 = c1;
}

// LDS address of a generic pointer into LDS: its low word (the shared
// aperture is aligned to 4 GB).
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>(p);
}

// 16 bytes per lane from global memory straight to LDS: lane i reads base +
// off_i (base the same for every lane) and its bytes land at LDS address
// lds + 16 i.  Issued as its own instruction so that the compiler's wait
// counting for the LDS reads around it stays exact (it would otherwise treat
// every LDS read after such a load as possibly out of order and wait for all
// of them); a vmcnt(0) wait before the barrier that publishes the data covers
// its completion.  The LDS address goes in M0, set by the compiler; one wait
// state separates that write from the load reading it.  A base that the
// vector ALU wrote (readfirstlane, or readlane where the compiler keeps it in
// a spilled lane) may be read by the load only five wait states later, and
// the compiler, which does not see that the asm is a load, inserts none: the
// load reads a copy that the scalar ALU makes (reads by it are interlocked),
// which is the wait state for M0 as well.
__device__ __forceinline__ void load_to_lds16(const void* base, uint32_t off, const void* lds) {
  const uint32_t a = __builtin_amdgcn_readfirstlane(lds_address(lds));
  uint64_t copy;
  asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
               : "=&s"(copy)
               : "v"(off), "s"(base), "{m0}"(a)
               : "memory");
}

// The same with a full 64-bit global address per lane.
__device__ __forceinline__ void load_to_lds16_at(const void* src, const void* lds) {
  const uint32_t a = __builtin_amdgcn_readfirstlane(lds_address(lds));
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "{m0}"(a) : "memory");
}

}  // namespace ojbkq
