// Stage 1 of Sec. 3, the per-workgroup half of the threshold: a sample
// workgroup of BS threads holds up to 4*BS draws, 4 per thread (draw
// 4*tid + q in kv[q]), and keeps its own top-t of them.  The t-th largest
// key of the whole sample (with multiplicity) is among the union of the
// workgroups' lists, so stage 2 selects from that union only.
#pragma once

#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace profk {

// Vector y of a batch: a workspace pointer (null stays null), the values.
template <class T>
__device__ __forceinline__ void at_vector(T*& p, uint64_t bytes) {
  // (byte arithmetic on the pointer: through an integer the compiler would
  // lose its address space and load with flat instructions)
  using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  if (p) p = reinterpret_cast<T*>(reinterpret_cast<Byte*>(p) + bytes * blockIdx.y);
}

// Clears the per-call counters; fhist (kLogBins words, or null) is the
// refinement histogram the filter accumulates into.
// (bcur: the large-k path's bucket fill counters, one per kBktPad words, and
// ghist its radix digit histogram, kBigBins words; both null when the call
// does not take that path)
__device__ __forceinline__ void reset_state(CallState* st, uint32_t* seg_cnt, uint32_t* fhist, uint32_t* bcur,
                                            uint32_t* ghist) {
  if (threadIdx.x < kSegs) seg_cnt[threadIdx.x * kSegStride] = 0;
  if (fhist)
    for (uint32_t i = threadIdx.x; i < kLogBins; i += blockDim.x) fhist[i] = 0;
  if (bcur)
    for (uint32_t i = threadIdx.x; i < kLogBins; i += blockDim.x) bcur[i * kBktPad] = 0;
  if (ghist)
    for (uint32_t i = threadIdx.x; i < kBigBins; i += blockDim.x) ghist[i] = 0;
  if (threadIdx.x == 0) {
    st->ticket = 0;
    st->status = 0;
    st->tie_above = 0;
    st->tie_n = 0;
    st->tie_ticket = 0;
    st->big_ticket = 0;
  }
  if (threadIdx.x < 16) st->grp_ticket[threadIdx.x] = 0;
}

// LDS of sample_block_top.
template <int BS>
struct SampleUnionShared {
  static constexpr int kDigit = BS <= kSampBS ? 10 : 11;  // about a bin per draw, half a bin on wide blocks
  alignas(16) uint32_t hist[1 << kDigit];
  alignas(16) uint32_t list[kListWords];
  alignas(16) uint32_t red[kKthRed];
  SelectScratch sc;
  uint32_t emitted;
};

// Writes the workgroup's top-min(t, nb) draws to dst, in no particular order
// (nb: draws it holds, valid bit q of `valid` for kv[q]).  Every thread of
// the workgroup calls it.  *cut (when not null) receives the t-th largest
// draw if the workgroup dropped any (nb > t), else 0.
template <int BS>
__device__ __forceinline__ void sample_block_top(uint32_t (&kv)[4], uint32_t valid, uint32_t nb, uint32_t t,
                                                 uint32_t* dst, SampleUnionShared<BS>& sh,
                                                 uint32_t* cut = nullptr) {
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
  if (t >= nb) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((valid >> q) & 1u) dst[4 * tid + q] = kv[q];
    if (cut && tid == 0) *cut = 0u;
    return;
  }
  if (tid == 0) sh.emitted = 0;  // (the select's barriers order it)
  const uint2 r = block_kth_regs<BS, 4, SampleUnionShared<BS>::kDigit>(kv, valid, (nb + 3) / 4, t, sh.hist, sh.list,
                                                                               sh.red, sh.sc);
  // the keys above the t-th, then copies of it up to t
  uint32_t m = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) m |= (((valid >> q) & 1u) && kv[q] > r.x ? 1u : 0u) << q;
  const uint32_t c = static_cast<uint32_t>(__popc(m)), incl = wave_incl_sum(c);
  const uint32_t tot = __builtin_amdgcn_readlane(incl, kWave - 1);
  if (tot) {
    uint32_t slot = 0;
    if (lane == 0) slot = atomicAdd(&sh.emitted, tot);
    slot = __builtin_amdgcn_readlane(slot, 0) + incl - c;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((m >> q) & 1u) dst[slot++] = kv[q];
  }
  for (uint32_t j = r.y + tid; j < t; j += BS) dst[j] = r.x;
  if (cut && tid == 0) *cut = r.x;
}

}  // namespace profk
