// cand_device.hpp -- device helpers shared by the candidate passes: operand
// transfers into LDS, wave-uniform values, the staged candidate queue.
#pragma once

#include "join_params.hpp"

namespace dl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = 512;  // eight waves, two per SIMD

typedef __attribute__((address_space(1))) void gvoid_t;
typedef __attribute__((address_space(3))) void lvoid_t;

// 16 bytes per lane from global memory into LDS (global_load_lds_dwordx4):
// lane l's bytes land at lds_dst + 16 l.  Issued as inline assembly so that
// the compiler's wait-count insertion does not treat the transfer as a
// write to the stage being read; the kernel orders it explicitly (vmcnt(0)
// and a barrier before a stage is read or overwritten).
__device__ inline uint32_t lds_addr(const void* lds_ptr) {
  return __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>((const lvoid_t*)lds_ptr));
}
// the same with the LDS destination given as a wave-uniform LDS address
__device__ inline void lds_dma16_at(const void* gsrc, uint32_t m0) {
  // M0 (the LDS base of the transfer) is an operand bound to the register,
  // so the compiler knows it is written; one wait state separates the M0
  // write from the LDS-DMA instruction that reads it.
  asm volatile(
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, off"
      :
      : "v"(gsrc), "{m0}"(m0)
      : "memory");
}
__device__ inline void lds_dma16(const void* gsrc, void* lds_dst) { lds_dma16_at(gsrc, lds_addr(lds_dst)); }

// Marks a block-uniform 64-bit value as such, so that it lives in scalar
// registers (the uniformity analysis loses tile indices carried around the
// persistent loop, and 64-bit vector copies of them crowd out the
// accumulators).
__device__ inline int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// This lane's index (0..63), recomputed from the lane-count instructions at
// every use.  Lane-derived offsets formed from it are not hoisted out of the
// persistent loop, where they would stay live beside the 128 accumulator
// registers and be spilled.
__device__ inline int fresh_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

constexpr int kQueue = 256;  // staged hits per wave (eps candidates or band entries)

// Writes a wave's staged (i, j) candidates to the global list from slot base
// on.  Positions past the list's capacity are counted but not written (the
// caller then retries with room).  With kP, each record's P~ (qp, staged
// beside q) goes to p.candp too.
template <bool kP>
__device__ inline void write_eps(const CandParams& p, const uint2* q, const uint32_t* qp, int nq,
                                 unsigned long long base) {
  // the records that fit; addresses are a scalar base and a 32-bit offset
  const unsigned long long cap = (unsigned long long)p.ccap;
  const int fit = base >= cap ? 0 : (cap - base < (unsigned long long)nq ? (int)(cap - base) : nq);
  uint2* const dst = p.cand + base;
  float* const dstp = kP && p.candp ? p.candp + base : nullptr;
  for (int s = fresh_lane(); s < fit; s += 64) {
    dst[s] = q[s];
    if constexpr (kP)
      if (dstp) dstp[s] = __uint_as_float(qp[s]);
  }
}

// The wave's staged candidates, with one atomic for the whole batch.
template <bool kP>
__device__ inline void flush_eps(const CandParams& p, const uint2* q, const uint32_t* qp, int nq) {
  unsigned long long base = 0;
  if (fresh_lane() == 0) base = atomicAdd(p.ccount, (unsigned long long)nq);
  write_eps<kP>(p, q, qp, nq, (unsigned long long)uniform64((int64_t)base));
}

// What every wave of the workgroup has left, at the end of its work: one
// atomic for the workgroup (one counter serves the whole grid, and its atomics
// queue at 10 ns or more each, so one per wave would add 20 us to a call).
// s_left: one word per wave and two for the base; every wave calls it.
template <bool kP>
__device__ inline void flush_eps_last(const CandParams& p, const uint2* q, const uint32_t* qp, int nq, int* s_left) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned long long* const s_base = reinterpret_cast<unsigned long long*>(s_left + kThreads / 64);
  if ((threadIdx.x & 63) == 0) s_left[wave] = nq;
  __syncthreads();
  int before = 0, all = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    const int n = __builtin_amdgcn_readfirstlane(s_left[w]);
    if (w < wave) before += n;
    all += n;
  }
  if (all == 0) return;
  if (threadIdx.x == 0) *s_base = atomicAdd(p.ccount, (unsigned long long)all);
  __syncthreads();
  write_eps<kP>(p, q, qp, nq, (unsigned long long)uniform64((int64_t)*s_base) + before);
}

}  // namespace dl
