// Blocks that solve one problem together inside one launch ("a team"): the
// exchange of per-block records that stands in for a kernel boundary.
//
// Every block posts its record of NV doubles into a slot of its own and reads
// the records of all the others, so one exchange is one store and one load
// trip through memory (2-3 us for 256 blocks against 12-15 us for a pass
// kernel, a one-block reduction kernel and the gaps between them).  A double
// travels as two 8-byte words that each hold 32 of its bits and a 32-bit tag;
// the words are relaxed agent-scope atomics, so a word with the expected tag
// carries its data and no fence or flag is needed.  Tags rise by one with
// every exchange and never repeat in a context's slots (the host hands each
// launch a fresh range), and the two parities of a tag use different slots: a
// block can be one exchange ahead of a slower one, never two, because each
// exchange waits for every record of the one before.
//
// The blocks of a team have to run at the same time.  The grid never exceeds
// one block per compute unit, but another stream's kernels may hold compute
// units back, so every wait is bounded: a block that has waited `limit` ticks
// of the 100 MHz clock gives up, says so in the launch's result and ends;
// the others then run out of their own limit.  The host takes the
// multi-launch route when any block gave up.
#pragma once

#include "cqk_device.h"

namespace cqk {

constexpr int kTeamBlock = 512;
constexpr int kTeamMax = 256;     // blocks of a team
constexpr int kSlotWords = 32;    // 8-byte words of one record slot (up to 16 doubles)
constexpr size_t kTeamCtlBytes = 16384;  // behind the slots: a solver's control block
constexpr size_t kTeamSlotBytes = (size_t)2 * kTeamMax * kSlotWords * sizeof(uint64_t);

struct Team {
  uint64_t* slots;
  uint32_t tag;      // tag of the last exchange; the next one uses tag + 1
  uint32_t pad_;
  uint64_t limit;    // longest wait of one exchange, 100 MHz ticks
};

// One exchange: `mine` (LDS, NV doubles, written before a barrier by the
// caller) goes out, all[v * T + g] (LDS) receives value v of block g.
// Returns false when a wait ran into its limit (the same answer for the
// whole block).  Ends with a barrier.
template <int NV>
__device__ __forceinline__ bool team_exchange(Team& team, const double* mine, double* all,
                                              int* gave_up) {
  static_assert(2 * NV <= kSlotWords, "a record fits its slot");
  const int T = gridDim.x, me = blockIdx.x, tid = threadIdx.x;
  if (T == 1) {
    if (tid < NV) all[tid] = mine[tid];
    __syncthreads();
    return true;
  }
  const uint32_t tag = ++team.tag;
  uint64_t* slots = team.slots + (size_t)(tag & 1u) * kTeamMax * kSlotWords;
  if (tid < 2 * NV) {
    const uint64_t u = __builtin_bit_cast(uint64_t, mine[tid >> 1]);
    const uint64_t half = (tid & 1) ? (u >> 32) : (u & 0xffffffffull);
    __hip_atomic_store(&slots[(size_t)me * kSlotWords + tid], (half << 32) | tag,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (tid == 0) *gave_up = 0;
  // word j of block g is item g * 2 NV + j; T <= kTeamMax = kTeamBlock / 2,
  // so a thread has at most NV of them, all loaded before the first test
  const int total = T * 2 * NV;
  uint64_t w[NV];
  bool ok = false, late = false;
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  while (!ok && !late) {
    ok = true;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int i = tid + k * kTeamBlock;
      w[k] = tag;
      if (i < total)
        w[k] = __hip_atomic_load(&slots[(size_t)(i / (2 * NV)) * kSlotWords + i % (2 * NV)],
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) ok = ok && (uint32_t)w[k] == tag;
    late = !ok && __builtin_amdgcn_s_memrealtime() - t0 > team.limit;
  }
  __syncthreads();  // *gave_up is clear
  if (late) *gave_up = 1;
  uint32_t* out = reinterpret_cast<uint32_t*>(all);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int i = tid + k * kTeamBlock;
    if (i < total) {
      const int g = i / (2 * NV), j = i % (2 * NV);
      out[2 * ((j >> 1) * T + g) + (j & 1)] = (uint32_t)(w[k] >> 32);
    }
  }
  __syncthreads();
  return *gave_up == 0;
}

// Sums of the NV values over the T records, in record order per lane: wave v
// takes value v, v + waves, ...; out[v] (LDS) is valid after the barrier it
// ends with, the same bits in every block.
template <int NV>
__device__ __forceinline__ void team_sum(const double* all, double* out) {
  const int T = gridDim.x;
  const int lane = threadIdx.x & (kWave - 1);
  for (int v = (int)(threadIdx.x / kWave); v < NV; v += kTeamBlock / kWave) {
    double a = 0.0;
    for (int g = lane; g < T; g += kWave) a += all[v * T + g];
    a = wave_sum(a);
    if (lane == 0) out[v] = a;
  }
  __syncthreads();
}

}  // namespace cqk
