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
// what the GPU holds at once, but another stream's kernels may hold compute
// units back, so every wait is bounded: a block that has waited `limit` ticks
// of the 100 MHz clock gives up, says so in the launch's result and ends.
// The others then run out of their own limit, but for the last exchange: a
// block posts its record before it waits, so there the rest of the team can
// finish without it.  A result that any block besides block 0 has a part in
// (x, the sums over it) therefore counts only when no block gave up, whatever
// block 0 found; one that block 0 writes alone (a run state) stands on its
// own.  Where it does not count, the multi-launch route answers.
#pragma once

#include "cqk_device.h"
#include "cqk_internal.h"

namespace cqk {

constexpr int kTeamBlock = 512;
constexpr int kTeamMax = 512;     // blocks of a team: up to two per compute unit
constexpr int kSlotWords = 16;    // 8-byte words of one record slot (up to 8 doubles)
constexpr size_t kTeamCtlBytes = 16384;  // behind the slots: a solver's control block
constexpr size_t kTeamSlotBytes = (size_t)2 * kTeamMax * kSlotWords * sizeof(uint64_t);

// The slots of teams that change size during a launch (the batched calls):
// the smaller teams of a later class of rows are parts of the larger ones of
// an earlier class, so their members agree on the tag, but a member of the
// larger team may still be reading when another part moves on: every team
// size has slots of its own.
constexpr int kBatTeamBlocks = 1024;      // blocks of such a launch
constexpr int kBatTeamLogs = 9;           // team sizes 1, 2, ... kBatTeamMax
constexpr int kBatTeamMax = 1 << (kBatTeamLogs - 1);
constexpr size_t kBatTeamBytes =
    (size_t)kBatTeamLogs * 2 * kBatTeamBlocks * kSlotWords * sizeof(uint64_t);
// The context's team buffer: slots and control block of the single solves,
// then those of the batched calls.
constexpr size_t kTeamBatCtl = kTeamSlotBytes + kTeamCtlBytes;
constexpr size_t kTeamBatSlots = kTeamBatCtl + 256;
constexpr size_t kTeamBytes = kTeamBatSlots + kBatTeamBytes;

struct Team {
  uint64_t* slots;   // the first member's slot of parity 0
  uint64_t limit;    // longest wait of one exchange, 100 MHz ticks
  uint32_t tag;      // tag of the last exchange; the next one uses tag + 1
  int T, me;         // blocks of the team, this block's place in it
  int parity;        // words from one parity's slots to the other's
  uint32_t late;     // tag of the exchange this block gives up at (tests), 0: none
};

// The tag of the exchange a test has this block give up at: 0 (no exchange
// has it) unless the block is the chosen one.
__device__ __forceinline__ uint32_t late_tag(TeamLate late, uint32_t tag) {
  return (late.exchange > 0 && (int)blockIdx.x == late.block) ? tag + (uint32_t)late.exchange : 0u;
}

__device__ __forceinline__ Team grid_team(uint64_t* slots, uint32_t tag, uint64_t limit,
                                          TeamLate late) {
  return Team{slots, limit, tag, (int)gridDim.x, (int)blockIdx.x, kTeamMax * kSlotWords,
              late_tag(late, tag)};
}

// A block by itself: nothing is exchanged and nothing waited for.
__device__ __forceinline__ Team team_alone() { return Team{nullptr, 0, 0, 1, 0, 0, 0}; }

// LDS of the reductions below.
template <int BLOCK>
struct TeamLds {
  double red[2][8 * (BLOCK / kWave)];  // the waves' sums, by the parity of the reduction
  double part[2][8 * (BLOCK / kWave)];
  int gave_up;                         // clear at the start of the kernel
};

// Posts a record: value v sits, the same in all of them, in the NW lanes from
// v * NW on of the calling wave.
template <int NV, int NW>
__device__ __forceinline__ void team_post(const Team& team, uint64_t* slots, uint32_t tag,
                                          double y, int lane) {
  static_assert(NW >= 2 && NV * NW <= kWave, "two lanes of a wave per value");
  if (lane < NV * NW && lane % NW < 2) {
    const uint64_t u = __builtin_bit_cast(uint64_t, y);
    const uint64_t half = (lane % NW) ? (u >> 32) : (u & 0xffffffffull);
    __hip_atomic_store(&slots[(size_t)team.me * kSlotWords + 2 * (lane / NW) + lane % NW],
                       (half << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A wave reads the records from, from + 4, ... (steps of `step` groups of
// four) below T: lane l takes word l % 16 of record l / 16 of a group, so one
// load instruction covers four whole records, R of them in flight.  Each
// record's value v is then in lanes 2v and 2v + 1 of its row of 16; the lane
// adds it up (lane_min: takes the minimum), or (MIN) takes the (key, weight)
// minimum with the value two lanes on as the weight.  (A lane per record instead, ten loads each of its
// own line, took the exchange of 256 blocks from 3 to 7 us.)
struct TeamRead {
  double sum;
  KeySum min;
  bool late;   // a wait ran into its limit
};

template <int NV, bool MIN>
__device__ __forceinline__ TeamRead team_read(const Team& team, const uint64_t* slots,
                                              uint32_t tag, int from, int step, int lane,
                                              bool lane_min = false) {
  constexpr int R = 4;
  TeamRead out{lane_min ? inf_d() : 0.0, KeySum{inf_d(), 0.0}, tag == team.late};
  const bool mine = (lane & 15) < 2 * NV;
  const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
  for (int g0 = from * 4; g0 < team.T && !out.late; g0 += R * step * 4) {
    uint64_t w[R];
    bool ok = false;
    while (!ok && !out.late) {
      ok = true;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int g = g0 + k * step * 4 + lane / 16;
        w[k] = tag;
        if (mine && g < team.T)
          w[k] = __hip_atomic_load(&slots[(size_t)g * kSlotWords + (lane & 15)],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int k = 0; k < R; ++k) ok = ok && (uint32_t)w[k] == tag;
      ok = __ballot(!ok) == 0;  // the wave goes round together
      out.late = !ok && __builtin_amdgcn_s_memrealtime() - t0 > team.limit;
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t half = (uint32_t)(w[k] >> 32);
      const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)half, dpp::kXor1, 0xF,
                                                                   0xF, false);
      const uint32_t lo = (lane & 1) ? other : half, hi = (lane & 1) ? half : other;
      const double v = __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
      const bool in = g0 + k * step * 4 + lane / 16 < team.T;
      if constexpr (MIN) {
        const double weight = dpp_move<dpp::kXor2, 0xF>(v, 0.0);
        out.min = ks_min(out.min, in ? KeySum{v, weight} : KeySum{inf_d(), 0.0});
      } else {
        out.sum = lane_min ? fmin(out.sum, in ? v : inf_d()) : out.sum + (in ? v : 0.0);
      }
    }
  }
  return out;
}

// Records are read by every wave of the block while a team is small (the
// totals are then in every wave with no further trip through LDS), shared
// among the waves in larger teams.
constexpr int kTeamAllRead = 16;

// Sums of NV values over the threads of a team's blocks, the last NM of them
// minima instead; tot[] holds the
// totals as scalars in every wave, the same bits in every block.  par: a
// counter of the block's reductions (parity of the LDS buffers).  Returns
// false, in the whole block, when a wait ran into its limit.  One barrier,
// two with more than one block.
template <int NV, int BLOCK, int NM = 0>
__device__ __forceinline__ bool team_reduce(Team& team, TeamLds<BLOCK>& S, int& par,
                                            const double* v, double* tot) {
  constexpr int NW = BLOCK / kWave;
  constexpr int N = (NV <= 4) ? 4 : 8;
  constexpr int SH = 6 - detail::ilog2(N);
  static_assert(NV <= 8 && NV * NW <= kWave, "one lane per wave and value");
  static_assert(2 * NV <= kSlotWords, "a record fits its slot");
  static_assert(NW == 4 || NW == 8, "the sums over NW lanes below");
  int tid = threadIdx.x;
  // what is made from the thread index stays here: hoisted out of a loop of
  // reductions the addresses would be spilled
  asm volatile("" : "+v"(tid));
  const int lane = tid & (kWave - 1), wid = scalar(tid / kWave);
  constexpr int NS = NV - NM;
  double x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = (i < NS) ? v[i] : 0.0;
  wave_sum_many<N>(x);
  par ^= 1;
  double* red = S.red[par];
  const int idx = lane >> SH;
  if ((lane & ((1 << SH) - 1)) == 0 && idx < NS) red[idx * NW + wid] = x[0];
#pragma unroll
  for (int i = NS; i < NV; ++i) {
    const double m = wave_min(v[i]);
    if (lane == 0) red[i * NW + wid] = m;
  }
  __syncthreads();
  // op: the sum, or the minimum in the lanes that hold one of the last NM
  auto op = [](double a, double b, bool min) { return (NM > 0 && min) ? fmin(a, b) : a + b; };
  double y = (lane < NV * NW) ? red[lane] : 0.0;
  const bool ym = lane >= NS * NW;
  y = op(y, dpp_move<dpp::kXor1, 0xF>(y, 0.0), ym);
  y = op(y, dpp_move<dpp::kXor2, 0xF>(y, 0.0), ym);
  if constexpr (NW == 8) y = op(y, dpp_move<dpp::kHalfMirror, 0xF>(y, 0.0), ym);
  if (team.T == 1) {
#pragma unroll
    for (int i = 0; i < NV; ++i) tot[i] = lane_value(y, i * NW);
    return true;
  }
  const uint32_t tag = ++team.tag;
  uint64_t* slots = team.slots + (size_t)(tag & 1u) * team.parity;
  if (wid == 0) team_post<NV, NW>(team, slots, tag, y, lane);
  const bool split = team.T > kTeamAllRead;
  const bool zm = NM > 0 && (lane & 15) >= 2 * NS;
  const TeamRead got =
      team_read<NV, false>(team, slots, tag, split ? wid : 0, split ? NW : 1, lane, zm);
  if (got.late) S.gave_up = 1;
  double z = got.sum;
  // the four rows of 16 lanes
  z = op(z, __shfl_xor(z, 32, kWave), zm);
  z = op(z, __shfl_xor(z, 16, kWave), zm);
  if (split && lane < 16 && (lane & 1) == 0) S.part[par][8 * wid + lane / 2] = z;
  __syncthreads();
  if (S.gave_up) return false;
  if (!split) {
#pragma unroll
    for (int i = 0; i < NV; ++i) tot[i] = lane_value(z, 2 * i);
    return true;
  }
  // value i of wave w at w * 8 + i: the waves' parts in lanes 8 apart
  const bool pm = NM > 0 && (lane & 7) >= NS;
  double p = (lane < 8 * NW) ? S.part[par][lane] : (pm ? inf_d() : 0.0);
  p = op(p, dpp_move<dpp::kRor8, 0xF>(p, 0.0), pm);
  p = op(p, __shfl_xor(p, 32, kWave), pm);
  p = op(p, __shfl_xor(p, 16, kWave), pm);
#pragma unroll
  for (int i = 0; i < NV; ++i) tot[i] = lane_value(p, i);
  return true;
}

// The two (key, weight) minima over the threads of a team's blocks, as
// team_reduce.
template <int BLOCK>
__device__ __forceinline__ bool team_reduce_ks(Team& team, TeamLds<BLOCK>& S, int& par,
                                               KeySum* ks) {
  constexpr int NW = BLOCK / kWave;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & (kWave - 1), wid = scalar(tid / kWave);
  par ^= 1;
  double* red = S.red[par];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const KeySum k = wave_ks_min(ks[i]);
    if (lane == 0) {
      red[(2 * i) * NW + wid] = k.k;
      red[(2 * i + 1) * NW + wid] = k.w;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i)
    ks[i] = wave_ks_min(lane < NW ? KeySum{red[2 * i * NW + lane], red[(2 * i + 1) * NW + lane]}
                                  : KeySum{inf_d(), 0.0});
  if (team.T == 1) return true;
  const uint32_t tag = ++team.tag;
  uint64_t* slots = team.slots + (size_t)(tag & 1u) * team.parity;
  const int q = lane / NW;
  const KeySum k0 = ks[0], k1 = ks[1];  // read before the choice: both stay in registers
  const double y = (q == 0) ? k0.k : (q == 1) ? k0.w : (q == 2) ? k1.k : k1.w;
  if (wid == 0) team_post<4, NW>(team, slots, tag, y, lane);
  // keys are in lanes 0, 1 and 4, 5 of a row of 16, their weights two lanes
  // on; lane 0 (4) of each row takes both
  const bool split = team.T > kTeamAllRead;
  const TeamRead got = team_read<4, true>(team, slots, tag, split ? wid : 0, split ? NW : 1, lane);
  if (got.late) S.gave_up = 1;
  const KeySum k2 = got.min;
#pragma unroll
  for (int i = 0; i < 2; ++i)
    ks[i] = wave_ks_min((lane & 15) == 4 * i ? k2 : KeySum{inf_d(), 0.0});
  const KeySum m0 = ks[0], m1 = ks[1];
  if (split && lane < 4)
    S.part[par][8 * wid + lane] = (lane == 0) ? m0.k : (lane == 1) ? m0.w
                                  : (lane == 2) ? m1.k : m1.w;
  __syncthreads();
  if (S.gave_up) return false;
  if (!split) return true;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    ks[i] = KeySum{inf_d(), 0.0};
    for (int k = 0; k < NW; ++k)
      ks[i] = ks_min(ks[i], KeySum{S.part[par][8 * k + 2 * i], S.part[par][8 * k + 2 * i + 1]});
  }
  return true;
}

// The sum of one value per block over the team, and over the blocks before
// this one, in every thread.  false as team_reduce.
template <int BLOCK>
__device__ __forceinline__ bool team_prefix(Team& team, TeamLds<BLOCK>& S, int& par, double mine,
                                            double* total, double* before) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & (kWave - 1), wid = scalar(tid / kWave);
  const uint32_t tag = ++team.tag;
  uint64_t* slots = team.slots + (size_t)(tag & 1u) * team.parity;
  par ^= 1;
  if (wid == 0) {
    team_post<1, 2>(team, slots, tag, mine, lane);
    double all = 0.0, low = 0.0;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    bool late = tag == team.late;
    for (int g = lane; g < team.T; g += kWave) {
      uint64_t w0, w1;
      bool ok = false;
      while (!ok && !late) {
        w0 = __hip_atomic_load(&slots[(size_t)g * kSlotWords], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        w1 = __hip_atomic_load(&slots[(size_t)g * kSlotWords + 1], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        ok = (uint32_t)w0 == tag && (uint32_t)w1 == tag;
        late = !ok && __builtin_amdgcn_s_memrealtime() - t0 > team.limit;
      }
      if (ok) {
        const double v =
            __builtin_bit_cast(double, (w0 >> 32) | (w1 & 0xffffffff00000000ull));
        all += v;
        low += (g < team.me) ? v : 0.0;
      }
    }
    if (late) S.gave_up = 1;
    all = wave_sum(all);
    low = wave_sum(low);
    if (lane == 0) {
      S.part[par][0] = all;
      S.part[par][1] = low;
    }
  }
  __syncthreads();
  if (S.gave_up) return false;
  *total = scalar(S.part[par][0]);
  *before = scalar(S.part[par][1]);
  return true;
}

// Tags of queued and captured launches, in device memory (a replay must not
// repeat its tags): those of the current launch, and the first never used.
// They have the top bit set, those of waiting calls clear.
struct TeamTags {
  uint32_t base, next;
  TeamFlags flags;   // of the current launch
  TeamPause pause;
  uint32_t epoch;    // of the pause
};
constexpr uint32_t kTeamDeviceTags = 0x80000000u;

// What a launch's flags are at its start, from those of the one before.
__device__ __forceinline__ TeamFlags next_flags(const TeamFlags& last, TeamPause& pause,
                                                bool forget) {
  if (forget) pause = TeamPause{0, 0, 0};
  else if (last.gave_up != kNotRun) pause.outcome(last.gave_up != 0);
  return TeamFlags{pause.turn() ? 0 : (int32_t)kNotRun, 0};
}

// Whether a queued launch's kernel is to return at once, the same in the
// whole block: not to run, or a block gave up before this one started.
__device__ __forceinline__ bool team_is_off(const TeamFlags* flags, int* lds) {
  if (threadIdx.x == 0)
    *lds = __hip_atomic_load(&flags->gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int off = *lds;
  __syncthreads();
  return off != 0;
}

// Before a queued or captured one-launch call: the run state of the kernels
// queued behind it, a fresh range of tags (the slots are cleared when the
// range starts over) and its flags.
template <typename State>
__global__ __launch_bounds__(256) void team_init_kernel(State* st, State init, TeamTags* tags,
                                                        uint64_t* slots, uint32_t need,
                                                        uint32_t epoch) {
  const uint32_t next = tags->next;
  const bool wrap = next == 0 || next > 0xffffffffu - need;
  __syncthreads();
  if (wrap)
    for (size_t i = threadIdx.x; i < kTeamSlotBytes / sizeof(uint64_t); i += 256) slots[i] = 0;
  if (threadIdx.x == 0) {
    *st = init;
    const uint32_t base = wrap ? kTeamDeviceTags : next;
    tags->base = base;
    tags->next = base + need;
    TeamPause pause = tags->pause;
    tags->flags = next_flags(tags->flags, pause, tags->epoch != epoch);
    tags->pause = pause;
    tags->epoch = epoch;
  }
}

}  // namespace cqk
