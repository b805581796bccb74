// Batched simplex projections (many rows of uneven length in one launch) and
// the vector-Jacobian product of the projection.
//
// Per row the method is the one of the single-instance path: Algorithm 2 per
// thread chunk merged into lam_J bounds (Section 2.2 eq. (lambdaJ),
// Section 4), then Algorithm 4 from that start (Section 3, Theorem 1), then
// x = max(0, y + lam*).  The backward pass follows from eq. (lambdaJ) on a
// fixed support S = {x > 0}: lam* = (r - sum_S y)/|S|, so
//   dx_S/dy_S = I - 11^T/|S|,  dx_S/dr = 1/|S|,
//   grad_y = [x > 0](g - mean_S g),  grad_r = mean_S g.
//
// Schedule.  Rows are classified on the device by length: rows of at most
// 64 * small_per values go to one wave each (four per workgroup), longer rows
// get a whole workgroup.  Workgroup rows are listed by decreasing length
// bucket; one persistent kernel pulls work items from an atomic counter
// (wave rows first or workgroup rows first) until the list is exhausted.
// small_per, the number of persistent workgroups per compute unit and that
// order form the schedule, which the tuner picks by timing every candidate
// on the caller's rows.
//
// A workgroup row is read once from HBM and x written once: each wave takes
// every fourth tile of 1024 values, writes zeros to that part of x, runs
// Algorithm 2 on 16 values per lane on its first tile with values above its
// running bound and keeps every such value of later tiles (wave reductions
// only), appending them with their indices to its LDS list.  After one barrier every wave combines the four lists'
// bounds, runs Algorithm 4 on the lists from the combined bound (all waves
// get the same multiplier) and writes x for its own list's entries; every
// other x is the zero already written.  The backward pass
// does the same with the support: zeros first, then g - mean_S g on S.
// A wave row keeps its values in registers from load to store.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "cqk_alg1.h"
#include "cqk_device.h"
#include "cqk_internal.h"
#include "cqk_team.h"

namespace cqk {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
constexpr int kK = 16;               // values per lane per wave tile (workgroup rows)
constexpr int kWTile = kWave * kK;   // 1024
constexpr int kSurvW = 1024;         // LDS list slots per wave (value + index)
constexpr int kNBW = 24;             // length buckets (bit length) of each row class
constexpr int kNB = 2 * kNBW;        // wave rows 0 .. kNBW - 1, workgroup rows kNBW .. kNB - 1
constexpr int kRefine = 8;
constexpr int kMaxNewton = 100;

enum BatFlags : int32_t { kBadRadius = 1, kBadValue = 2, kInfeasible = 4, kNotConverged = 8 };

struct BatArgs {
  int32_t nseg;
  int32_t small_max;    // longest row solved from one wave's registers
  int32_t med_max;      // longest row solved by one wave (tile by tile above small_max)
  int32_t short_first;  // 1: wave rows are handed out first
  const int64_t* off;
  const float* y;
  const double* r;
  double r_scalar;
  float* x;
  double* lam_out;
  int32_t* nfree_out;
  const float* g;       // backward: upstream gradient
  float* gy;            // backward: grad_y
  double* gr;           // backward: grad_r
  int32_t* list;        // row ids: workgroup rows by bucket, then wave rows
  int64_t* lrow;        // per list entry: the row's first element and its length
  int32_t* counters;    // CTR_* below
  int32_t* bhist;       // planning: rows per length bucket of each block of kPBlock rows
};

// The call's counters, in lines of 32 ints (128 bytes): line 0 holds the rows
// of each class, the work items, whether a team gave up and where each length
// bucket of the workgroup rows starts in the list; then kQueues lines with
// the call's outcome, each as summed by the blocks of one queue (flags,
// survivors, rows whose lists overflowed), kQueues more for the rows solved
// by teams (they count only when no team gave up), and two sets of work
// queues, one line each (the second for the rows of teams of one).  Atomics on one
// address take turns at about 13 ns each on this part, so one shared queue
// and one shared survivor total, updated per row, bounded every call of many
// rows (65 536 rows of 64-512 values: 1.70 ms for 147 456 atomics): blocks
// now share a queue in groups of grid / kQueues and add their outcome once.
constexpr int CTR_NLONG = 0, CTR_NSHORT = 1, CTR_NITEMS = 2, CTR_GAVE_UP = 3, CTR_LBASE = 4;
constexpr int CTR_FLAGS = 0, CTR_SURV = 1, CTR_OVER = 2;
constexpr int kQueues = 32, kCtrLine = 32;
constexpr int CTR_STAT0 = kCtrLine, CTR_STAT1 = (1 + kQueues) * kCtrLine,
              CTR_OUTCOME = (1 + 2 * kQueues) * kCtrLine,  // what the host reads
              CTR_QUEUE0 = CTR_OUTCOME, CTR_QUEUE1 = CTR_QUEUE0 + kQueues * kCtrLine,
              CTR_TOTAL = CTR_QUEUE1 + kQueues * kCtrLine;
// rows whose length has at most kGroupBucket bits (general form, four to a
// wave): where they start in the list
constexpr int kGroupBucket = 7;
constexpr int CTR_GROUPS = CTR_LBASE + kNBW;
static_assert(CTR_GROUPS < kCtrLine, "the bucket starts fit line 0");

// A block's outcome, in LDS until the block ends.
struct BatStat {
  int32_t flags, surv, over;
};

__device__ __forceinline__ void stat_init(BatStat& t) {
  if (threadIdx.x == 0) t.flags = t.surv = t.over = 0;
}

// Adds the block's outcome to its group's line.  MAXOVER: `over` is a maximum
// (the general form's iteration count), not a sum.
template <bool MAXOVER>
__device__ __forceinline__ void stat_flush(const BatStat& t, int32_t* lines) {
  if (threadIdx.x == 0) {
    int32_t* line = lines + (blockIdx.x % kQueues) * kCtrLine;
    if (t.flags) atomicOr(&line[CTR_FLAGS], t.flags);
    if (t.surv) atomicAdd(&line[CTR_SURV], t.surv);
    if (t.over) {
      if (MAXOVER) atomicMax(&line[CTR_OVER], t.over);
      else atomicAdd(&line[CTR_OVER], t.over);
    }
  }
}

// The work items of one block: those of its group's queue (queue q holds
// items q, q + kQueues, ...), then those of the queues that still hold some.
// No item is a block's by its number: a grid larger than the GPU can hold
// starts its last blocks late, and their items (long rows, at the list's
// start) would wait for them.  Called by the whole first wave of the block;
// returns nitems or more once every queue is empty.
struct ItemSource {
  int own = (int)(blockIdx.x % kQueues);
  __device__ __forceinline__ int next(int32_t* queues, int nitems) {
    const int lane = threadIdx.x & (kWave - 1);
    for (;;) {
      int k = 0;
      if (lane == 0) k = atomicAdd(&queues[own * kCtrLine], 1);
      k = __builtin_amdgcn_readfirstlane(k);
      const int64_t item = own + (int64_t)k * kQueues;
      if (item < nitems) return (int)item;
      // the queues that still hold items, in one round trip; the next one
      // after this block's
      int64_t at = nitems;
      if (lane < kQueues)
        at = lane + (int64_t)__hip_atomic_load(&queues[lane * kCtrLine],
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) *
                        kQueues;
      const uint64_t m = __ballot(at < nitems);
      if (m == 0) return nitems;
      const uint64_t up = m >> own << own;
      own = __builtin_ctzll(up ? up : m);
    }
  }
};

// Length bucket of a row of L values: its bit length, in the wave-row range
// if L <= wave_max, else in the workgroup-row range.  (Finer buckets, with
// the two bits below the leading one, made the solve kernel slower.)
__device__ __forceinline__ int bucket_of(int64_t L, int wave_max) {
  int b = 64 - __clzll((unsigned long long)L);
  b = b >= kNBW ? kNBW - 1 : b;
  return (L <= wave_max) ? b : kNBW + b;
}

// Tags of the teams' exchanges, in device memory (replays must not repeat
// them): every launch starts above the largest tag of the one before; near
// the end of the range the slots are cleared and it starts over.
struct BatTeamCtl {
  uint32_t base, last;
  TeamFlags flags;   // of the current launch (done: not used)
  TeamPause pause;
  uint32_t epoch;    // of the pause
};
constexpr uint32_t kTagRestart = 0xc0000000u, kTagEnd = 0xfffffff0u;

// The planning's part in it, by one block.
template <typename Args>
__device__ __forceinline__ void start_teams(const Args&) {}
// CTR_GAVE_UP at the start of a launch.
template <typename Args>
__device__ __forceinline__ int32_t teams_off(const Args&) {
  return 0;
}

// Planning: the rows are listed by length bucket (workgroup rows longest
// bucket first, then the wave rows longest bucket first, so the four wave
// rows of one work item have about the same length), in row order inside a
// bucket, without atomics: each block of kPBlock rows counts its buckets
// with ballots, then each block places its rows after the rows of its bucket
// in earlier blocks.
constexpr int kPBlock = 1024;
constexpr int kPW = kPBlock / kWave;

// Longest row one wave solves: the simplex forward's medium limit, else the
// register limit.
template <typename Args>
__device__ __forceinline__ int wave_row_max(const Args& A) {
  return A.small_max;
}

template <>
__device__ __forceinline__ int wave_row_max<BatArgs>(const BatArgs& A) {
  return A.med_max;
}

// length bucket of row s, -1 past the last row.  Args: the simplex or the
// general form's argument record (both carry nseg, small_max, off and the
// planning buffers).
template <typename Args>
__device__ __forceinline__ int plan_bucket(const Args& A, int s) {
  return (s < A.nseg) ? bucket_of(A.off[s + 1] - A.off[s], wave_row_max(A)) : -1;
}

template <typename Args>
__device__ __forceinline__ void clear_counters(const Args& A) {
  for (int i = CTR_STAT0 + (int)threadIdx.x; i < CTR_TOTAL; i += kPBlock) A.counters[i] = 0;
  start_teams(A);
}

template <typename Args>
__global__ __launch_bounds__(kPBlock) void bat_count_kernel(Args A) {
  __shared__ int wh[kPW][kNB];
  const int s = blockIdx.x * kPBlock + (int)threadIdx.x;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int b = plan_bucket(A, s);
  for (int k = 0; k < kNB; ++k) {
    const uint64_t m = __ballot(b == k);
    if (lane == 0) wh[w][k] = __popcll(m);
  }
  __syncthreads();
  if (threadIdx.x < kNB) {
    int c = 0;
    for (int q = 0; q < kPW; ++q) c += wh[q][threadIdx.x];
    A.bhist[(size_t)blockIdx.x * kNB + threadIdx.x] = c;
  }
  if (blockIdx.x == 0) clear_counters(A);
}

template <typename Args>
__global__ __launch_bounds__(kPBlock) void bat_place_kernel(Args A) {
  __shared__ int part[2][kNB][32];
  __shared__ int base[kNB], pre[kNB];
  __shared__ int wh[kPW][kNB];
  const int nblk = gridDim.x;
  // one block (up to kPBlock rows) needs no counts of the others and no
  // launch before it
  const bool alone = nblk == 1;
  if (alone) clear_counters(A);
  // bucket totals over all blocks and over the blocks before this one,
  // 32 threads per bucket
  for (int idx = threadIdx.x; idx < kNB * 32; idx += kPBlock) {
    const int k = idx / 32, sub = idx % 32;
    int t = 0, p = 0;
    for (int q = sub; q < nblk && !alone; q += 32) {
      const int v = A.bhist[(size_t)q * kNB + k];
      t += v;
      p += (q < (int)blockIdx.x) ? v : 0;
    }
    part[0][k][sub] = t;
    part[1][k][sub] = p;
  }
  const int s = blockIdx.x * kPBlock + (int)threadIdx.x;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int b = plan_bucket(A, s);
  int rank = 0;
  for (int k = 0; k < kNB; ++k) {
    const uint64_t m = __ballot(b == k);
    if (b == k) rank = lane_prefix(m);
    if (lane == 0) wh[w][k] = __popcll(m);
  }
  __syncthreads();
  if (threadIdx.x < kNB) {
    const int k = threadIdx.x;
    int t = 0, p = 0;
    for (int q = 0; q < 32; ++q) {
      t += part[0][k][q];
      p += part[1][k][q];
    }
    pre[k] = p;
    // exclusive scan of the per-wave counts of this block
    int c = 0;
    for (int q = 0; q < kPW; ++q) {
      const int v = wh[q][k];
      wh[q][k] = c;
      c += v;
    }
    base[k] = alone ? c : t;  // totals for now
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    // workgroup rows, longest bucket first, then the wave rows, longest first
    int acc = 0;
    for (int k = kNB - 1; k >= kNBW; --k) {
      const int t = base[k];
      base[k] = acc;
      acc += t;
    }
    const int nlong = acc;
    for (int k = kNBW - 1; k >= 0; --k) {
      const int t = base[k];
      base[k] = acc;
      acc += t;
    }
    const int nshort = acc - nlong;
    if (blockIdx.x == 0) {
      A.counters[CTR_NLONG] = nlong;
      A.counters[CTR_NSHORT] = nshort;
      A.counters[CTR_NITEMS] = nlong + (nshort + kWaves - 1) / kWaves;
      A.counters[CTR_GAVE_UP] = teams_off(A);
      for (int k = 0; k < kNBW; ++k) A.counters[CTR_LBASE + k] = base[kNBW + k];
      A.counters[CTR_GROUPS] = base[kGroupBucket];
    }
  }
  __syncthreads();
  if (b >= 0) {
    const int pos = base[b] + pre[b] + wh[w][b] + rank;
    A.list[pos] = s;
    // the solve kernels read the row's extent with its id, in one round trip
    A.lrow[2 * (size_t)pos] = A.off[s];
    A.lrow[2 * (size_t)pos + 1] = A.off[s + 1] - A.off[s];
  }
}

__device__ __forceinline__ double row_radius(const BatArgs& A, int s) {
  return A.r ? A.r[s] : A.r_scalar;
}

// Block sum of three doubles; every thread gets the totals.
__device__ __forceinline__ void block_sum3(double a, double b, double c, double* lds, double* o) {
  __shared__ double bc[3];
  double in[3] = {a, b, c};
  block_reduce<3, 0, 0, kBlock>(in, nullptr, nullptr, lds, bc);
  o[0] = bc[0];
  o[1] = bc[1];
  o[2] = bc[2];
  __syncthreads();
}

// Algorithm 2 over K values (division-free comparisons, see the simplex
// kernels): returns the J mask, its count and sum.
template <int K>
__device__ __forceinline__ uint32_t alg2(const float* v, uint32_t active, float r, int& c,
                                         float& S) {
  uint32_t J = 0, Jt = 0;
  c = 0;
  S = 0.f;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const uint32_t bit = 1u << j;
    if (!(active & bit)) continue;
    const float vj = v[j];
    if (c == 0) {
      J = bit;
      c = 1;
      S = vj;
      continue;
    }
    if ((float)c * vj + (r - S) > 0.f) {
      if ((r - S - vj) < (float)(c + 1) * (r - vj)) {
        J |= bit;
        S += vj;
        c += 1;
      } else {
        Jt |= J;
        J = bit;
        S = vj;
        c = 1;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const uint32_t bit = 1u << j;
    if ((Jt & bit) && ((float)c * v[j] + (r - S) > 0.f)) {
      J |= bit;
      S += v[j];
      c += 1;
    }
  }
  return J;
}

// LDS of one workgroup: the four waves' lists and their bound records.
struct BatLds {
  float sv[kWaves][kSurvW];
  int32_t si[kWaves][kSurvW];
  double ws[kWaves][8];
  double red[3 * kWaves];
  BatStat stat;
  int item;
};

enum { W_C = 0, W_S, W_LMIN, W_VMAX, W_BAD, W_N, W_NF };

// One wave's share of Algorithm 2 on a tile of kK values per lane already in
// registers (v, active): the lanes' sets, the wave's bound refined against
// its running survivors (run_c, run_s), the values kept.  Returns the keep
// mask; nk/ks are the lane's kept count and sum; lam_min takes the new bound.
__device__ __forceinline__ uint32_t wave_tile_alg2(const float* v, uint32_t active, double rd,
                                                   double run_c, double run_s, double& lam_min,
                                                   double& nk, double& ks) {
  const float r = (float)rd;
  int c = 0;
  float S = 0.f;
  uint32_t J;
  if (__ballot(__popc(active) > 1) != 0) {
    J = alg2<kK>(v, active, r, c, S);
  } else {
    // at most one value per lane: Algorithm 2 keeps it
    J = active;
    c = __popc(active);
#pragma unroll
    for (int e = 0; e < kK; ++e)
      if ((active >> e) & 1u) S = v[e];
  }
  const double lam_t = (c > 0) ? (rd - (double)S) / (double)c : inf_d();
  // every bound below is lam_J of a non-empty J, hence >= lam* (eq. (lambdaJ))
  const double ct = wave_sum((double)c), skt = wave_sum((double)S);
  double lam_b = (ct > 0.0) ? (rd - skt) / ct : inf_d();
  if (ct > 0.0 && run_c > 0.0) lam_b = fmin(lam_b, (rd - (skt + run_s)) / (ct + run_c));
  if (run_c > 0.0) lam_b = fmin(lam_b, (rd - run_s) / run_c);
  uint32_t keep = 0;
  auto select = [&](double lb) {
    const double lt = fmin(lam_t, lb);
    keep = 0;
    nk = 0.0;
    ks = 0.0;
#pragma unroll
    for (int e = 0; e < kK; ++e) {
      if (((J >> e) & 1u) && ((double)v[e] + lt > 0.0)) {
        keep |= 1u << e;
        nk += 1.0;
        ks += (double)v[e];
      }
    }
  };
  for (int it = 0; it < kRefine; ++it) {
    select(lam_b);
    const double kc = wave_sum(nk), kss = wave_sum(ks);
    if (kc == 0.0) break;
    double nl = (rd - kss) / kc;
    if (run_c > 0.0) nl = fmin(nl, (rd - (kss + run_s)) / (kc + run_c));
    if (!(nl < lam_b)) break;
    lam_b = nl;
  }
  select(lam_b);
  lam_min = fmin(lam_min, lam_b);
  return keep;
}

// One wave tile of a row: kK values per lane, four 16-byte vectors at
// t0 + q*256 + lane*4 (q < 4); when the tile is in range every load is
// issued before the first use.  Rows start at any element, so the vectors
// are only element-aligned.
__device__ __forceinline__ void load_wtile(const float* p, int64_t t0, int lane, int64_t n,
                                           float* o) {
  if (t0 + kWTile <= n) {
    flt4u r[kK / 4];
#pragma unroll
    for (int q = 0; q < kK / 4; ++q) r[q] = ld16(p + t0 + q * kWave * 4 + lane * 4);
#pragma unroll
    for (int q = 0; q < kK / 4; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) o[4 * q + k] = r[q][k];
  } else {
    // a part tile: whole vectors still move 16 bytes, the one that crosses
    // the end value by value
#pragma unroll
    for (int q = 0; q < kK / 4; ++q) {
      const int64_t i = t0 + q * kWave * 4 + lane * 4;
      if (i + 4 <= n) {
        const flt4u r = ld16(p + i);
#pragma unroll
        for (int k = 0; k < 4; ++k) o[4 * q + k] = r[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) o[4 * q + k] = (i + k < n) ? p[i + k] : 0.f;
      }
    }
  }
}

__device__ __forceinline__ void zero_wtile(float* p, int64_t t0, int lane, int64_t n) {
  const flt4u z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kK / 4; ++q) {
    const int64_t i = t0 + q * kWave * 4 + lane * 4;
    if (i + 4 <= n) {
      st16(p + i, z);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i + k < n) p[i + k] = 0.f;
    }
  }
}

// The largest float not above x: v > result exactly when v + x' > 0 for
// x' = -x, so a bound filters FP32 values with one FP32 compare.
__device__ __forceinline__ float float_at_or_below(double x) {
  float f = (float)x;
  if ((double)f > x) f = nextafterf(f, -__builtin_huge_valf());
  return f;
}

// Algorithm 4 from lam (>= lam*) on the four LDS lists, run by one wave:
// lam_{k+1} = lam_J(J_k), J_k = {v + lam_k > 0}; stops as the paper's
// Algorithm 4 (phi(lam_k) <= r for k >= 1) or when J no longer changes.
__device__ __forceinline__ double wave_newton_lists(const BatLds& L, const int* nw, double rd,
                                                    double lam) {
  const int lane = threadIdx.x & (kWave - 1);
  double prev_c = -1.0;
  for (int it = 0; it < kMaxNewton; ++it) {
    double cc = 0.0, ss = 0.0, ph = 0.0;
    for (int w = 0; w < kWaves; ++w) {
      for (int i = lane; i < nw[w]; i += kWave) {
        const double v = (double)L.sv[w][i];
        const double z = v + lam;
        if (z > 0.0) {
          cc += 1.0;
          ss += v;
          ph += z;
        }
      }
    }
    cc = wave_sum(cc);
    ss = wave_sum(ss);
    ph = wave_sum(ph);
    if (cc == prev_c) break;
    if (it > 0 && ph <= rd) break;
    if (cc == 0.0) break;
    const double nl = (rd - ss) / cc;
    if (!(nl < lam)) break;
    prev_c = cc;
    lam = nl;
  }
  return lam;
}

// A wave's running state over its tiles of one row: the values kept so far
// (count, sum, list length), the smallest bound found (each bound lam_J of
// some set J, so >= lam*), the largest value and a NaN once a value is NaN
// or infinite.
struct WaveRun {
  double c = 0.0, s = 0.0, lam = inf_d();
  float vmx = -__builtin_huge_valf();
  float badf = 0.f;
  int nw = 0;
};

// One tile (values t0 .. t0 + 1023) of a row of n values for the calling
// wave: x = 0 over the tile; on the wave's first tile of the row Algorithm 2
// per lane with the wave's refinement, on a later one the running bound;
// the values kept are appended with their positions to the wave's list
// (sv, si; entries past kSurvW are counted, not stored).  A tile whose
// largest value is at or below the running bound costs one test.
__device__ __forceinline__ void wave_row_tile(const float* y, float* x, int64_t n, int64_t t0,
                                              double rd, WaveRun& R, float* sv, int32_t* si) {
  static_assert(kK < 32, "a lane's kept count must fit in five bits");
  const int lane = threadIdx.x & (kWave - 1);
  float v[kK];
  uint32_t active = 0;
  float tmax = -__builtin_huge_valf();
  load_wtile(y, t0, lane, n, v);
  if (t0 + kWTile <= n) {
    // a tile wholly in the row: no per-value range tests
    const flt4u z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kK / 4; ++q) st16(x + t0 + q * kWave * 4 + lane * 4, z);
    active = (1u << kK) - 1u;
#pragma unroll
    for (int e = 0; e < kK; ++e) {
      R.badf += v[e] * 0.f;
      tmax = fmaxf(tmax, v[e]);
    }
  } else {
    // x is zero wherever the lists do not write it
    zero_wtile(x, t0, lane, n);
#pragma unroll
    for (int q = 0; q < kK / 4; ++q) {
      const int64_t i = t0 + (int64_t)q * kWave * 4 + (int64_t)lane * 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (i + k < n) {
          active |= 1u << (4 * q + k);
          R.badf += v[4 * q + k] * 0.f;
          tmax = fmaxf(tmax, v[4 * q + k]);
        }
      }
    }
  }
  R.vmx = fmaxf(R.vmx, tmax);
  // the first bound of the row: lam_J of the tile's largest value alone
  // (Algorithm 2's first set), so that Algorithm 2 below only scans the
  // values above it
  if (R.lam == inf_d()) {
    const double m = wave_max((double)tmax);
    if (m > -inf_d()) R.lam = rd - m;
  }
  // values at or below the wave's best bound so far are zero at the
  // solution (v <= thr exactly when v + lam <= 0)
  if (R.lam < inf_d()) {
    const float thr = float_at_or_below(-R.lam);
    if (__ballot(tmax > thr) == 0) return;
#pragma unroll
    for (int e = 0; e < kK; ++e)
      if (!(v[e] > thr)) active &= ~(1u << e);
  }
  if (__ballot(active != 0u) == 0) return;
  uint32_t keep;
  if (R.c > 0.0) {
    // a later tile: the running bound has already filtered it and every
    // value left is kept; lam_J of everything kept so far becomes the
    // bound below (again >= lam*)
    keep = active;
  } else {
    double nk, ks;
    keep = wave_tile_alg2(v, active, rd, R.c, R.s, R.lam, nk, ks);
  }
  // this lane's place in the list: its kept count (five bits) summed over
  // the lanes below it, one bit at a time
  const int c = __popc(keep);
  int pre = 0, nt = 0;
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    const uint64_t m = __ballot((c >> b) & 1);
    pre += lane_prefix(m) << b;
    nt += __popcll(m) << b;
  }
  if (nt == 0) return;
  int pos = R.nw + pre;
  double ks = 0.0;
#pragma unroll
  for (int q = 0; q < kK / 4; ++q) {
    if ((keep >> (4 * q)) & 0xFu) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = 4 * q + k;
        if ((keep >> e) & 1u) {
          if (pos < kSurvW) {
            sv[pos] = v[e];
            si[pos] = (int32_t)(t0 + q * kWave * 4 + lane * 4 + k);
          }
          ++pos;
          ks += (double)v[e];
        }
      }
    }
  }
  R.nw += nt;
  R.c += (double)nt;
  R.s += wave_sum(ks);
  R.lam = fmin(R.lam, (rd - R.s) / R.c);
}

// ---------------------------------------------------------------------------
// One workgroup row.
// ---------------------------------------------------------------------------
__device__ void solve_long_row(const BatArgs& A, int s, int64_t base, int64_t n, BatLds& L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const double rd = row_radius(A, s);
  const float* y = A.y + base;
  float* x = A.x + base;
  if (!(rd >= 0.0) || !(rd < inf_d())) {
    for (int64_t i = threadIdx.x; i < n; i += kBlock) x[i] = 0.f;
    if (threadIdx.x == 0) {
      atomicOr(&L.stat.flags, kBadRadius);
      if (A.lam_out) A.lam_out[s] = __builtin_nan("");
      if (A.nfree_out) A.nfree_out[s] = 0;
    }
    return;
  }
  WaveRun R;
  const int64_t ntiles = (n + kWTile - 1) / kWTile;
  for (int64_t t = wid; t < ntiles; t += kWaves)
    wave_row_tile(y, x, n, t * kWTile, rd, R, L.sv[wid], L.si[wid]);
  const double run_c = R.c, run_s = R.s, lam_min = R.lam;
  const float vmx = R.vmx, badf = R.badf;
  const int nw = R.nw;
  const double wbad = wave_sum((badf == 0.f) ? 0.0 : 1.0);
  const double wmax = wave_max((double)vmx);
  if (lane == 0) {
    L.ws[wid][W_C] = run_c;
    L.ws[wid][W_S] = run_s;
    L.ws[wid][W_LMIN] = lam_min;
    L.ws[wid][W_VMAX] = wmax;
    L.ws[wid][W_BAD] = wbad;
    L.ws[wid][W_N] = (double)nw;
  }
  __syncthreads();
  // every wave combines the four records in the same order
  double C = 0.0, S = 0.0, lmin = inf_d(), vmax = -inf_d(), bad = 0.0;
  bool over = false;
  int nws[kWaves];
  int ntot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    C += L.ws[w][W_C];
    S += L.ws[w][W_S];
    lmin = fmin(lmin, L.ws[w][W_LMIN]);
    vmax = fmax(vmax, L.ws[w][W_VMAX]);
    bad += L.ws[w][W_BAD];
    nws[w] = (int)L.ws[w][W_N];
    over = over || nws[w] > kSurvW;
    ntot += nws[w];
  }
  if (bad > 0.0 || n == 0 || rd == 0.0) {
    // x is already zero
    if (threadIdx.x == 0) {
      if (bad > 0.0) atomicOr(&L.stat.flags, kBadValue);
      if (n == 0 && rd > 0.0) atomicOr(&L.stat.flags, kInfeasible);
      if (A.lam_out) A.lam_out[s] = (bad > 0.0 || n == 0) ? __builtin_nan("") : 0.0;
      if (A.nfree_out) A.nfree_out[s] = 0;
    }
    return;
  }
  const double lam0 = (C > 0.0) ? fmin((rd - S) / C, lmin) : lmin;
  if (over) {
    // a list overflowed: Algorithm 4 over the row itself (re-read from cache)
    double lam = lam0, prev_c = -1.0;
    for (int it = 0; it < kMaxNewton; ++it) {
      double cc = 0.0, ss = 0.0, ph = 0.0;
      for (int64_t i = threadIdx.x; i < n; i += kBlock) {
        const double yv = (double)y[i];
        const double z = yv + lam;
        if (z > 0.0) {
          cc += 1.0;
          ss += yv;
          ph += z;
        }
      }
      double tt[3];
      block_sum3(cc, ss, ph, L.red, tt);
      if (tt[0] == prev_c) break;
      if (it > 0 && tt[2] <= rd) break;
      if (tt[0] == 0.0) break;
      const double nl = (rd - tt[1]) / tt[0];
      if (!(nl < lam)) break;
      prev_c = tt[0];
      lam = nl;
    }
    double nf = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kBlock) {
      const float o = (float)fmax((double)y[i] + lam, 0.0);
      nf += (o > 0.f) ? 1.0 : 0.0;
      x[i] = o;
    }
    double tn[3];
    block_sum3(nf, 0.0, 0.0, L.red, tn);
    if (threadIdx.x == 0) {
      if (A.lam_out) A.lam_out[s] = lam;
      if (A.nfree_out) A.nfree_out[s] = (int32_t)tn[0];
      atomicAdd(&L.stat.surv, ntot);
      atomicAdd(&L.stat.over, 1);
    }
    return;
  }
  // Algorithm 4 from lam_0 (>= lam*) on the lists.  (The start refinement of
  // the single-instance path, 12 candidate sets, is left out here: on lists
  // in LDS it cost more than the Newton steps it saves.)
  double lam = lam0;
  lam = wave_newton_lists(L, nws, rd, lam);
  // x for this wave's list; every other x of the row is already zero
  double nf = 0.0;
  for (int i = lane; i < nws[wid]; i += kWave) {
    const float o = (float)fmax((double)L.sv[wid][i] + lam, 0.0);
    x[L.si[wid][i]] = o;
    nf += (o > 0.f) ? 1.0 : 0.0;
  }
  nf = wave_sum(nf);
  if (lane == 0) L.ws[wid][W_NF] = nf;
  __syncthreads();
  if (threadIdx.x == 0) {
    double nft = 0.0;
    for (int w = 0; w < kWaves; ++w) nft += L.ws[w][W_NF];
    if (A.lam_out) A.lam_out[s] = lam;
    if (A.nfree_out) A.nfree_out[s] = (int32_t)nft;
    atomicAdd(&L.stat.surv, ntot);
  }
}

// Algorithm 4 from lam (>= lam*) on one wave's LDS list of n values.
__device__ __forceinline__ double wave_newton_list(const float* lv, int n, double rd, double lam) {
  const int lane = threadIdx.x & (kWave - 1);
  double prev_c = -1.0;
  for (int it = 0; it < kMaxNewton; ++it) {
    double cc = 0.0, ss = 0.0, ph = 0.0;
    for (int i = lane; i < n; i += kWave) {
      const double v = (double)lv[i];
      const double z = v + lam;
      if (z > 0.0) {
        cc += 1.0;
        ss += v;
        ph += z;
      }
    }
    cc = wave_sum(cc);
    ss = wave_sum(ss);
    ph = wave_sum(ph);
    if (cc == prev_c) break;
    if (it > 0 && ph <= rd) break;
    if (cc == 0.0) break;
    const double nl = (rd - ss) / cc;
    if (!(nl < lam)) break;
    prev_c = cc;
    lam = nl;
  }
  return lam;
}

// ---------------------------------------------------------------------------
// One medium row (64 * SP < n <= med_max): one wave takes every tile of the
// row, as each wave of a workgroup row takes every fourth, then runs
// Algorithm 4 on its own list.  No workgroup barrier: the four waves of a
// work item solve four rows of about the same length at once.
// ---------------------------------------------------------------------------
__device__ void solve_medium_row(const BatArgs& A, int s, int64_t base, int64_t n, BatLds& L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const double rd = row_radius(A, s);
  const float* y = A.y + base;
  float* x = A.x + base;
  if (!(rd >= 0.0) || !(rd < inf_d())) {
    for (int64_t i = lane; i < n; i += kWave) x[i] = 0.f;
    if (lane == 0) {
      atomicOr(&L.stat.flags, kBadRadius);
      if (A.lam_out) A.lam_out[s] = __builtin_nan("");
      if (A.nfree_out) A.nfree_out[s] = 0;
    }
    return;
  }
  WaveRun R;
  const int64_t ntiles = (n + kWTile - 1) / kWTile;
  for (int64_t t = 0; t < ntiles; ++t)
    wave_row_tile(y, x, n, t * kWTile, rd, R, L.sv[wid], L.si[wid]);
  const bool bad = wave_sum((R.badf == 0.f) ? 0.0 : 1.0) > 0.0;
  if (bad || rd == 0.0) {
    // x is already zero
    if (lane == 0) {
      if (bad) atomicOr(&L.stat.flags, kBadValue);
      if (A.lam_out) A.lam_out[s] = bad ? __builtin_nan("") : 0.0;
      if (A.nfree_out) A.nfree_out[s] = 0;
    }
    return;
  }
  double lam = (R.c > 0.0) ? fmin((rd - R.s) / R.c, R.lam) : R.lam;
  double nf = 0.0;
  const bool over = R.nw > kSurvW;
  if (over) {
    // the list overflowed: Algorithm 4 over the row itself (re-read)
    double prev_c = -1.0;
    for (int it = 0; it < kMaxNewton; ++it) {
      double cc = 0.0, ss = 0.0, ph = 0.0;
      for (int64_t i = lane; i < n; i += kWave) {
        const double yv = (double)y[i];
        const double z = yv + lam;
        if (z > 0.0) {
          cc += 1.0;
          ss += yv;
          ph += z;
        }
      }
      cc = wave_sum(cc);
      ss = wave_sum(ss);
      ph = wave_sum(ph);
      if (cc == prev_c) break;
      if (it > 0 && ph <= rd) break;
      if (cc == 0.0) break;
      const double nl = (rd - ss) / cc;
      if (!(nl < lam)) break;
      prev_c = cc;
      lam = nl;
    }
    for (int64_t i = lane; i < n; i += kWave) {
      const float o = (float)fmax((double)y[i] + lam, 0.0);
      nf += (o > 0.f) ? 1.0 : 0.0;
      x[i] = o;
    }
  } else {
    lam = wave_newton_list(L.sv[wid], R.nw, rd, lam);
    // x for the list; every other x of the row is already zero
    for (int i = lane; i < R.nw; i += kWave) {
      const float o = (float)fmax((double)L.sv[wid][i] + lam, 0.0);
      x[L.si[wid][i]] = o;
      nf += (o > 0.f) ? 1.0 : 0.0;
    }
  }
  nf = wave_sum(nf);
  if (lane == 0) {
    if (A.lam_out) A.lam_out[s] = lam;
    if (A.nfree_out) A.nfree_out[s] = (int32_t)nf;
    atomicAdd(&L.stat.surv, R.nw);
    if (over) atomicAdd(&L.stat.over, 1);
  }
}

// ---------------------------------------------------------------------------
// One wave row (L <= 64 * SP), values in registers.
// ---------------------------------------------------------------------------
template <int SP>
__device__ void solve_short_row(const BatArgs& A, int s, int64_t base, int64_t L, BatStat& stat) {
  const int lane = threadIdx.x & (kWave - 1);
  const double rd = row_radius(A, s);
  const float* y = A.y + base;
  float* x = A.x + base;
  float v[SP];
  uint32_t active = 0;
  double bad = 0.0;
#pragma unroll
  for (int k = 0; k < SP; ++k) v[k] = 0.f;
  if (L > 0) {
    // every load issued before the first use (index clamped to the row)
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      const int64_t i = (int64_t)k * kWave + lane;
      v[k] = y[i < L ? i : L - 1];
    }
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      const int64_t i = (int64_t)k * kWave + lane;
      if (i < L) {
        active |= 1u << k;
        bad += (fabsf(v[k]) < __builtin_huge_valf()) ? 0.0 : 1.0;
      } else {
        v[k] = 0.f;
      }
    }
  }
  bad = wave_sum(bad);
  const bool bad_r = !(rd >= 0.0) || !(rd < inf_d());
  if (bad_r || bad > 0.0 || L == 0 || rd == 0.0) {
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      const int64_t i = (int64_t)k * kWave + lane;
      if (i < L) x[i] = 0.f;
    }
    if (lane == 0) {
      int f = 0;
      if (bad_r) f |= kBadRadius;
      if (bad > 0.0) f |= kBadValue;
      if (L == 0 && rd > 0.0) f |= kInfeasible;
      if (f) atomicOr(&stat.flags, f);
      if (A.lam_out) A.lam_out[s] = (f) ? __builtin_nan("") : 0.0;
      if (A.nfree_out) A.nfree_out[s] = 0;
    }
    return;
  }
  const float r = (float)rd;
  // Algorithm 2 scans only the values above the first bound, lam_J of the
  // row's largest value alone
  float vm = -__builtin_huge_valf();
#pragma unroll
  for (int k = 0; k < SP; ++k)
    if ((active >> k) & 1u) vm = fmaxf(vm, v[k]);
  const double lam_first = rd - wave_max((double)vm);
  const float thr = float_at_or_below(-lam_first);
  uint32_t scan = 0;
#pragma unroll
  for (int k = 0; k < SP; ++k) scan |= (((active >> k) & 1u) && v[k] > thr) ? (1u << k) : 0u;
  int c;
  float S;
  const uint32_t J = alg2<SP>(v, scan, r, c, S);
  const double lam_t = (c > 0) ? (rd - (double)S) / (double)c : inf_d();
  const double cw = wave_sum((double)c), sw = wave_sum((double)S);
  double lam_b = (cw > 0) ? fmin((rd - sw) / cw, lam_first) : lam_first;
  // refinement on the wave's own sub-problem, then Algorithm 4 on the row
  for (int it = 0; it < kRefine; ++it) {
    const double lt = fmin(lam_t, lam_b);
    double nk = 0.0, ks = 0.0;
#pragma unroll
    for (int e = 0; e < SP; ++e)
      if (((J >> e) & 1u) && (double)v[e] + lt > 0.0) {
        nk += 1.0;
        ks += (double)v[e];
      }
    nk = wave_sum(nk);
    ks = wave_sum(ks);
    if (nk == 0.0) break;
    const double nl = (rd - ks) / nk;
    if (!(nl < lam_b)) break;
    lam_b = nl;
  }
  // every value of the row is still in registers: run Algorithm 4 on all of it
  double lam = fmin(lam_b, wave_min(lam_t));
  double prev_c = -1.0;
  for (int it = 0; it < kMaxNewton; ++it) {
    double cc = 0.0, ss = 0.0, ph = 0.0;
#pragma unroll
    for (int e = 0; e < SP; ++e) {
      const double z = (double)v[e] + lam;
      if (((active >> e) & 1u) && z > 0.0) {
        cc += 1.0;
        ss += (double)v[e];
        ph += z;
      }
    }
    cc = wave_sum(cc);
    ss = wave_sum(ss);
    ph = wave_sum(ph);
    if (cc == prev_c) break;
    if (it > 0 && ph <= rd) break;
    if (cc == 0.0) break;
    const double nl = (rd - ss) / cc;
    if (!(nl < lam)) break;
    prev_c = cc;
    lam = nl;
  }
  double nf = 0.0;
#pragma unroll
  for (int k = 0; k < SP; ++k) {
    const int64_t i = (int64_t)k * kWave + lane;
    if (i < L) {
      const float o = (float)fmax((double)v[k] + lam, 0.0);
      nf += (o > 0.f) ? 1.0 : 0.0;
      x[i] = o;
    }
  }
  nf = wave_sum(nf);
  if (lane == 0) {
    if (A.lam_out) A.lam_out[s] = lam;
    if (A.nfree_out) A.nfree_out[s] = (int32_t)nf;
  }
}

// Work item -> workgroup row (true) or group of four wave rows (false), and
// its index in that class, under the schedule's order.
__device__ __forceinline__ bool item_is_long(const BatArgs& A, int item, int nlong, int nsg,
                                             int* idx) {
  if (A.short_first) {
    if (item < nsg) {
      *idx = item;
      return false;
    }
    *idx = item - nsg;
    return true;
  }
  if (item < nlong) {
    *idx = item;
    return true;
  }
  *idx = item - nlong;
  return false;
}

template <int SP>
__global__ __launch_bounds__(kBlock, 3) void bat_solve_kernel(BatArgs A) {
  __shared__ BatLds L;
  const int nlong = A.counters[CTR_NLONG];
  const int nshort = A.counters[CTR_NSHORT];
  const int nitems = A.counters[CTR_NITEMS];
  const int nsg = nitems - nlong;
  ItemSource src;
  stat_init(L.stat);
  for (;;) {
    if (threadIdx.x < kWave) {
      const int next = src.next(A.counters + CTR_QUEUE0, nitems);
      if (threadIdx.x == 0) L.item = next;
    }
    __syncthreads();
    const int item = L.item;
    __syncthreads();
    if (item >= nitems) break;
    int idx;
    if (item_is_long(A, item, nlong, nsg, &idx)) {
      solve_long_row(A, A.list[idx], A.lrow[2 * (size_t)idx], A.lrow[2 * (size_t)idx + 1], L);
    } else {
      const int k = idx * kWaves + (int)(threadIdx.x / kWave);
      if (k < nshort) {
        const size_t e = (size_t)nlong + k;
        const int64_t Lr = A.lrow[2 * e + 1];
        if (Lr <= A.small_max) solve_short_row<SP>(A, A.list[e], A.lrow[2 * e], Lr, L.stat);
        else solve_medium_row(A, A.list[e], A.lrow[2 * e], Lr, L);
      }
    }
    __syncthreads();
  }
  stat_flush<false>(L.stat, A.counters + CTR_STAT0);
}

// ---------------------------------------------------------------------------
// Backward: grad_y = [x > 0](g - mean_S g), grad_r = mean_S g.
// ---------------------------------------------------------------------------
// One tile (values t0 .. t0 + 1023) of a row of n values for the calling
// wave's VJP: grad_y = 0 over the tile, the support's count and sum of g
// added to (cnt, sum), its (g, position) pairs appended to the wave's list
// (sv, si; entries past kSurvW are counted, not stored).
__device__ __forceinline__ void vjp_row_tile(const float* x, const float* g, float* gy, int64_t n,
                                             int64_t t0, double& cnt, double& sum, int& nw,
                                             float* sv, int32_t* si) {
  const int lane = threadIdx.x & (kWave - 1);
  float xs[kK], gs[kK];
  uint32_t sup = 0;
  load_wtile(x, t0, lane, n, xs);
  load_wtile(g, t0, lane, n, gs);
  // grad_y is zero off the support
  zero_wtile(gy, t0, lane, n);
#pragma unroll
  for (int q = 0; q < kK / 4; ++q) {
    const int64_t i = t0 + (int64_t)q * kWave * 4 + (int64_t)lane * 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = 4 * q + k;
      if (i + k < n && xs[e] > 0.f) {
        sup |= 1u << e;
        cnt += 1.0;
        sum += (double)gs[e];
      }
    }
  }
  if (__ballot(sup != 0u) == 0) return;
#pragma unroll
  for (int e = 0; e < kK; ++e) {
    const bool kb = (sup >> e) & 1u;
    const uint64_t m = __ballot(kb);
    if (kb) {
      const int pos = nw + lane_prefix(m);
      if (pos < kSurvW) {
        sv[pos] = gs[e];
        si[pos] = (int32_t)(t0 + (e / 4) * kWave * 4 + lane * 4 + (e % 4));
      }
    }
    nw += __popcll(m);
  }
}

__device__ void vjp_long_row(const BatArgs& A, int s, int64_t base, int64_t n, BatLds& L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const float* x = A.x + base;
  const float* g = A.g + base;
  float* gy = A.gy + base;
  double cnt = 0.0, sum = 0.0;
  int nw = 0;
  const int64_t ntiles = (n + kWTile - 1) / kWTile;
  for (int64_t t = wid; t < ntiles; t += kWaves)
    vjp_row_tile(x, g, gy, n, t * kWTile, cnt, sum, nw, L.sv[wid], L.si[wid]);
  cnt = wave_sum(cnt);
  sum = wave_sum(sum);
  if (lane == 0) {
    L.ws[wid][W_C] = cnt;
    L.ws[wid][W_S] = sum;
    L.ws[wid][W_N] = (double)nw;
  }
  __syncthreads();
  double C = 0.0, Sg = 0.0;
  bool over = false;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    C += L.ws[w][W_C];
    Sg += L.ws[w][W_S];
    over = over || L.ws[w][W_N] > (double)kSurvW;
  }
  const double gbar = (C > 0.0) ? Sg / C : 0.0;
  const float gb = (float)gbar;
  if (over) {
    // the support did not fit the lists: a second pass over the row
    for (int64_t i = threadIdx.x; i < n; i += kBlock)
      if (x[i] > 0.f) gy[i] = g[i] - gb;
  } else {
    for (int i = lane; i < nw; i += kWave) gy[L.si[wid][i]] = L.sv[wid][i] - gb;
  }
  if (threadIdx.x == 0 && A.gr) A.gr[s] = gbar;
}

// A medium row's VJP (64 * SP < n <= med_max) by one wave, tile after tile.
__device__ void vjp_medium_row(const BatArgs& A, int s, int64_t base, int64_t n, BatLds& L) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const float* x = A.x + base;
  const float* g = A.g + base;
  float* gy = A.gy + base;
  double cnt = 0.0, sum = 0.0;
  int nw = 0;
  const int64_t ntiles = (n + kWTile - 1) / kWTile;
  for (int64_t t = 0; t < ntiles; ++t)
    vjp_row_tile(x, g, gy, n, t * kWTile, cnt, sum, nw, L.sv[wid], L.si[wid]);
  const double C = wave_sum(cnt), Sg = wave_sum(sum);
  const double gbar = (C > 0.0) ? Sg / C : 0.0;
  const float gb = (float)gbar;
  if (nw > kSurvW) {
    // the support did not fit the list: a second pass over the row
    for (int64_t i = lane; i < n; i += kWave)
      if (x[i] > 0.f) gy[i] = g[i] - gb;
  } else {
    for (int i = lane; i < nw; i += kWave) gy[L.si[wid][i]] = L.sv[wid][i] - gb;
  }
  if (lane == 0 && A.gr) A.gr[s] = gbar;
}

template <int SP>
__device__ void vjp_short_row(const BatArgs& A, int s, int64_t base, int64_t L) {
  const int lane = threadIdx.x & (kWave - 1);
  float xs[SP], gs[SP];
  double cnt = 0.0, sum = 0.0;
#pragma unroll
  for (int k = 0; k < SP; ++k) xs[k] = gs[k] = 0.f;
  if (L > 0) {
    // every load issued before the first use (index clamped to the row)
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      const int64_t i = (int64_t)k * kWave + lane;
      const int64_t e = base + (i < L ? i : L - 1);
      xs[k] = A.x[e];
      gs[k] = A.g[e];
    }
#pragma unroll
    for (int k = 0; k < SP; ++k)
      if ((int64_t)k * kWave + lane >= L) xs[k] = gs[k] = 0.f;
  }
#pragma unroll
  for (int k = 0; k < SP; ++k) {
    if (xs[k] > 0.f) {
      cnt += 1.0;
      sum += (double)gs[k];
    }
  }
  cnt = wave_sum(cnt);
  sum = wave_sum(sum);
  const double gbar = (cnt > 0.0) ? sum / cnt : 0.0;
  const float gb = (float)gbar;
#pragma unroll
  for (int k = 0; k < SP; ++k) {
    const int64_t i = (int64_t)k * kWave + lane;
    if (i < L) A.gy[base + i] = (xs[k] > 0.f) ? gs[k] - gb : 0.f;
  }
  if (lane == 0 && A.gr) A.gr[s] = gbar;
}

template <int SP>
__global__ __launch_bounds__(kBlock) void bat_vjp_kernel(BatArgs A) {
  __shared__ BatLds L;
  const int nlong = A.counters[CTR_NLONG];
  const int nshort = A.counters[CTR_NSHORT];
  const int nitems = A.counters[CTR_NITEMS];
  const int nsg = nitems - nlong;
  ItemSource src;
  for (;;) {
    if (threadIdx.x < kWave) {
      const int next = src.next(A.counters + CTR_QUEUE0, nitems);
      if (threadIdx.x == 0) L.item = next;
    }
    __syncthreads();
    const int item = L.item;
    __syncthreads();
    if (item >= nitems) break;
    int idx;
    if (item_is_long(A, item, nlong, nsg, &idx)) {
      vjp_long_row(A, A.list[idx], A.lrow[2 * (size_t)idx], A.lrow[2 * (size_t)idx + 1], L);
    } else {
      const int k = idx * kWaves + (int)(threadIdx.x / kWave);
      if (k < nshort) {
        const size_t e = (size_t)nlong + k;
        const int64_t Lr = A.lrow[2 * e + 1];
        if (Lr <= A.small_max) vjp_short_row<SP>(A, A.list[e], A.lrow[2 * e], Lr);
        else vjp_medium_row(A, A.list[e], A.lrow[2 * e], Lr, L);
      }
    }
    __syncthreads();
  }
}


// ===========================================================================
// Batched general CQK (Section 2.1, Algorithm 1 per row) and its VJP.
//
// Row s is (d, a, b, l, u)[off[s] .. off[s+1]) with its own r[s].  Every row
// runs Algorithm 1 from lam = 0 (or eq. (CQKlambda0) over the row) with its
// own bracket, breakpoint and secant state: the scalar update of the
// single-instance solver on a state record each wave or workgroup keeps in
// registers, every lane updating its own copy from the same reduced sums (so
// all copies stay identical and the control flow uniform).  A row of at most
// 64 * small_per values is one wave's, its per-index form (c, s, bl, bu) held in
// registers from load to store (4 or 8 values per lane, by the schedule); a
// longer row is a workgroup's, which re-reads the row from memory at every
// evaluation.  x = clamp((a + lam b)/d, l, u)
// (eq. (xopt)) is written once.
//
// Backward, on a locally constant free set F = {l < x < u} (eq. (xopt) on F
// and eq. (opt) differentiated): with q = sum_F b^2/d and
// mu = (sum_F g b/d)/q,
//   grad_a = [F](g - b mu)/d,   grad_r = mu   (both 0 when F is empty).
// ===========================================================================
constexpr int kCqkU = 4;    // values per thread in flight in a workgroup pass

struct BatCqkArgs {
  int32_t nseg;
  int32_t small_max;    // longest wave row
  int32_t short_first;  // 1: wave rows are handed out first
  int32_t grouped;      // 1: rows of up to kGroupBucket bits are the group kernel's
  int32_t lambda0_mode; // CQK_LAMBDA0_ZERO, _FORMULA or _USER
  int32_t max_iter;
  double tol;
  double lam0_user;     // the start of every row with CQK_LAMBDA0_USER
  const int64_t* off;
  const void *d, *a, *b, *l, *u;  // TIn (float or double)
  const double* r;
  void* x;              // forward output; backward input (TIn)
  double* lam_out;
  int32_t* status_out;
  const void* g;        // backward: upstream gradient (TIn)
  void* ga;             // backward: grad_a (TIn)
  double* gr;           // backward: grad_r
  int32_t* list;
  int64_t* lrow;
  int32_t* counters;
  int32_t* bhist;
  uint64_t* tslots;     // teams: record slots, control words (BatTeamCtl), wait
  BatTeamCtl* tctl;     // limit; tslots null: no teams
  uint64_t tlimit;
  uint32_t tepoch;
  TeamLate tlate;
};

template <>
__device__ __forceinline__ void start_teams<BatCqkArgs>(const BatCqkArgs& A) {
  if (A.tslots == nullptr) return;
  const uint32_t last = A.tctl->last;
  __syncthreads();
  if (last >= kTagRestart)
    for (size_t i = threadIdx.x; i < kBatTeamBytes / sizeof(uint64_t); i += kPBlock)
      A.tslots[i] = 0;
  if (threadIdx.x == 0) {
    BatTeamCtl& T = *A.tctl;
    T.base = T.last = (last >= kTagRestart) ? 0u : last;
    TeamPause pause = T.pause;
    T.flags = next_flags(T.flags, pause, T.epoch != A.tepoch);
    T.pause = pause;
    T.epoch = A.tepoch;
  }
}
template <>
__device__ __forceinline__ int32_t teams_off<BatCqkArgs>(const BatCqkArgs& A) {
  return A.tslots != nullptr ? A.tctl->flags.gave_up : 0;
}

__device__ __forceinline__ GenState cqk_row_state(const BatCqkArgs& A, double r) {
  GenState st{};
  st.lam = (A.lambda0_mode == CQK_LAMBDA0_USER) ? A.lam0_user : 0.0;
  st.lam0 = st.lam;
  st.lam_prev = __builtin_nan("");
  st.lam_final = __builtin_nan("");
  st.lo = -inf_d();
  st.hi = inf_d();
  st.phi_lo = st.phi_hi = __builtin_nan("");
  st.r = r;
  st.tol = A.tol;
  st.status = kRunning;
  st.max_iter = A.max_iter;
  st.compaction = CQK_COMPACT_OFF;
  st.mode = kModeEval;
  return st;
}

// Per-row outputs and the call's flags, by one thread of the row's owner.
__device__ __forceinline__ void cqk_row_report(const BatCqkArgs& A, int s, const GenState& st,
                                               double lam, BatStat& stat) {
  if (A.lam_out) A.lam_out[s] = lam;
  if (A.status_out) A.status_out[s] = st.status;
  int f = 0;
  if (st.status == CQK_INVALID_ARG) f = kBadValue;
  else if (st.status == CQK_INFEASIBLE) f = kInfeasible;
  else if (st.status == CQK_NOT_CONVERGED) f = kNotConverged;
  if (f) atomicOr(&stat.flags, f);
  atomicAdd(&stat.surv, st.iter);
  atomicMax(&stat.over, st.iter);
}

// The arrays of a call in their element type (FP64 values are used as
// they are, FP32 values are widened to FP64 for the arithmetic).
template <typename TIn>
struct CqkArrays {
  const TIn *d, *a, *b, *l, *u, *g;
  TIn *x, *ga;
  __device__ explicit CqkArrays(const BatCqkArgs& A)
      : d((const TIn*)A.d), a((const TIn*)A.a), b((const TIn*)A.b), l((const TIn*)A.l),
        u((const TIn*)A.u), g((const TIn*)A.g), x((TIn*)A.x), ga((TIn*)A.ga) {}
};

__device__ __forceinline__ bool cqk_has_lambda(const GenState& st) {
  return st.status == CQK_OK || st.status == CQK_NOT_CONVERGED;
}

// ---------------------------------------------------------------------------
// One wave row (L <= 64 * SP), per-index form in registers.
// ---------------------------------------------------------------------------
template <int SP, typename TIn>
__device__ __forceinline__ void cqk_short_row(const BatCqkArgs& A, int s, int64_t base, int64_t L,
                              double r, BatStat& stat) {
  const CqkArrays<TIn> V(A);
  const int lane = threadIdx.x & (kWave - 1);
  double c[SP], sv[SP], bl[SP], bu[SP];
  double bad = 0.0, sc = 0.0, ss = 0.0;
#pragma unroll
  for (int k = 0; k < SP; ++k) c[k] = sv[k] = bl[k] = bu[k] = 0.0;
  if (L > 0) {
    // every load issued before the first use (index clamped to the row), so
    // the row costs one memory round trip, not one per value of a lane
    TIn rd[SP], ra[SP], rb[SP], rl[SP], ru[SP];
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      const int64_t i = lane + (int64_t)k * kWave;
      const int64_t e = base + (i < L ? i : L - 1);
      rd[k] = V.d[e];
      ra[k] = V.a[e];
      rb[k] = V.b[e];
      rl[k] = V.l[e];
      ru[k] = V.u[e];
    }
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      if (lane + (int64_t)k * kWave < L) {
        to_form((double)rd[k], (double)ra[k], (double)rb[k], (double)rl[k], (double)ru[k], c[k],
                sv[k], bl[k], bu[k], bad);
        sc += c[k];
        ss += sv[k];
      }
    }
  }
  // slots in use, the same for the whole wave: a short row skips the others
  // (the lanes past its end hold zeros, which add nothing to any sum)
  const int nk = __builtin_amdgcn_readfirstlane((int)((L + kWave - 1) / kWave));
  GenState st = cqk_row_state(A, r);
  if (wave_sum(bad) > 0.0 || !(fabs(r) < inf_d())) {
    st.status = CQK_INVALID_ARG;
  } else if (L == 0) {
    st.status = (r == 0.0) ? CQK_OK : CQK_INFEASIBLE;
    st.lam_final = 0.0;
  } else if (A.lambda0_mode == CQK_LAMBDA0_FORMULA) {
    const double tc = wave_sum(sc), ts = wave_sum(ss);
    st.lam = st.lam0 = (ts > 0.0) ? (r - tc) / ts : 0.0;
  }
  while (st.status == kRunning) {
    if (st.mode == kModeEval) {
      Acc acc;
      acc_init(acc);
#pragma unroll
      for (int k = 0; k < SP; ++k)
        if (k < nk) eval_index<false>(acc, c[k], sv[k], bl[k], bu[k], st.lam, 0.0, 0.0);
      double t[NSUM];
#pragma unroll
      for (int i = 0; i < NSUM; ++i) t[i] = 0.0;
      static_assert(P_P == 0 && P_A == 1 && P_QP == 2 && P_QM == 3, "the four sums");
      wave_sum4(acc.s, t);
      t[P_NIN] = (double)L;
      update_after_eval<false>(&st, t, nullptr);
    } else {
      KeySum ks[2] = {KeySum{inf_d(), 0.0}, KeySum{inf_d(), 0.0}};
#pragma unroll
      for (int k = 0; k < SP; ++k)
        if (k < nk) bkpt_index(ks, c[k], sv[k], bl[k], bu[k], st.lam);
      ks[0] = wave_ks_min(ks[0]);
      ks[1] = wave_ks_min(ks[1]);
      update_after_bkpt<false>(&st, ks, nullptr);
    }
    state_to_scalars(st);
  }
  const bool ok = cqk_has_lambda(st);
  const double lam = ok ? st.lam_final : __builtin_nan("");
  if (L > 0) {
    // the row again (from cache): a slot's loads unguarded, issued together
    constexpr int H = 4;
#pragma unroll
    for (int k0 = 0; k0 < SP; k0 += H) {
      if (k0 < nk) {
        TIn rd[H], ra[H], rb[H], rl[H], ru[H];
#pragma unroll
        for (int k = 0; k < H; ++k) {
          const int64_t i = lane + (int64_t)(k0 + k) * kWave;
          const int64_t e = base + (i < L ? i : L - 1);
          rd[k] = V.d[e];
          ra[k] = V.a[e];
          rb[k] = V.b[e];
          rl[k] = V.l[e];
          ru[k] = V.u[e];
        }
#pragma unroll
        for (int k = 0; k < H; ++k) {
          const int64_t i = lane + (int64_t)(k0 + k) * kWave;
          if (k0 + k < nk) {
            const double xv = fmin(fmax(fma((double)rb[k], lam, (double)ra[k]) / (double)rd[k],
                                        (double)rl[k]), (double)ru[k]);
            if (i < L) V.x[base + i] = (TIn)(ok ? xv : __builtin_nan(""));
          }
        }
      }
    }
  }
  if (lane == 0) cqk_row_report(A, s, st, lam, stat);
}

// Rows of at most kGroupLanes * kGroupSlots values, kWave / kGroupLanes of
// them side by side in a wave.
constexpr int kGroupLanes = 16, kGroupSlots = 8;
// Calls of at least this many rows take the group kernel: 16 384 FP32 rows of
// 16 to 127 values 95 -> 75 us; a call without such rows pays for the empty
// launch (128 to 512 values 111 -> 113 us), which at 8192 rows is as much as
// it saves on a mixed call.
constexpr int kGroupMinRows = 16384;
static_assert(kGroupLanes * kGroupSlots >= (1 << kGroupBucket) - 1, "every row of the bucket fits");

// Sum over a group's lanes (a DPP row), the same bits in each of them.
__device__ __forceinline__ double group_sum(double v) {
  v += dpp_move<dpp::kXor1, 0xF>(v, 0.0);
  v += dpp_move<dpp::kXor2, 0xF>(v, 0.0);
  v += dpp_move<dpp::kHalfMirror, 0xF>(v, 0.0);
  v += dpp_move<dpp::kMirror, 0xF>(v, 0.0);
  return v;
}

__device__ __forceinline__ KeySum group_ks_min(KeySum v) {
#pragma unroll
  for (int o = kGroupLanes / 2; o > 0; o >>= 1)
    v = ks_min(v, KeySum{__shfl_xor(v.k, o, kWave), __shfl_xor(v.w, o, kWave)});
  return v;
}

// Short rows side by side: the reductions and the scalar update, which cost a
// wave the same however short its row is, run once for four of them.  A group
// without a row has L < 0.
template <typename TIn>
__device__ __forceinline__ void cqk_group_rows(const BatCqkArgs& A, int s, int64_t base,
                                               int64_t L, double r, BatStat& stat) {
  constexpr int SP = kGroupSlots, GL = kGroupLanes;
  const CqkArrays<TIn> V(A);
  // what is made from the thread index stays here: hoisted out of the loop
  // over the work items it would be spilled
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & (GL - 1);
  double c[SP], sv[SP], bl[SP], bu[SP];
  double bad = 0.0, sc = 0.0, ss = 0.0;
#pragma unroll
  for (int k = 0; k < SP; ++k) c[k] = sv[k] = bl[k] = bu[k] = 0.0;
  // slots in use by any of the rows
  int nk = 0;
#pragma unroll
  for (int g = 0; g < kWave; g += GL)
    nk = max(nk, (__builtin_amdgcn_readlane((int)L, g) + GL - 1) / GL);
  {
    // every load issued before the first use (index clamped to the row; a
    // group without values reads place 0 of the call's arrays)
    TIn rd[SP], ra[SP], rb[SP], rl[SP], ru[SP];
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      if (k < nk) {
        const int64_t i = lane + k * GL;
        const int64_t e = (L > 0) ? base + (i < L ? i : L - 1) : 0;
        rd[k] = V.d[e];
        ra[k] = V.a[e];
        rb[k] = V.b[e];
        rl[k] = V.l[e];
        ru[k] = V.u[e];
      }
    }
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      if (k < nk && lane + k * GL < L) {
        to_form((double)rd[k], (double)ra[k], (double)rb[k], (double)rl[k], (double)ru[k], c[k],
                sv[k], bl[k], bu[k], bad);
        sc += c[k];
        ss += sv[k];
      }
    }
  }
  GenState st = cqk_row_state(A, r);
  bad = group_sum(bad);
  if (A.lambda0_mode == CQK_LAMBDA0_FORMULA) {
    const double tc = group_sum(sc), ts = group_sum(ss);
    if (L > 0) st.lam = st.lam0 = (ts > 0.0) ? (r - tc) / ts : 0.0;
  }
  if (L < 0) {
    st.status = CQK_OK;
  } else if (bad > 0.0 || !(fabs(r) < inf_d())) {
    st.status = CQK_INVALID_ARG;
  } else if (L == 0) {
    st.status = (r == 0.0) ? CQK_OK : CQK_INFEASIBLE;
    st.lam_final = 0.0;
  }
  while (__ballot(st.status == kRunning) != 0) {
    if (st.status == kRunning && st.mode == kModeEval) {
      Acc acc;
      acc_init(acc);
#pragma unroll
      for (int k = 0; k < SP; ++k)
        if (k < nk) eval_index<false>(acc, c[k], sv[k], bl[k], bu[k], st.lam, 0.0, 0.0);
      double t[NSUM];
#pragma unroll
      for (int i = 0; i < NSUM; ++i) t[i] = 0.0;
      t[P_P] = group_sum(acc.s[P_P]);
      t[P_A] = group_sum(acc.s[P_A]);
      t[P_QP] = group_sum(acc.s[P_QP]);
      t[P_QM] = group_sum(acc.s[P_QM]);
      update_after_eval<false>(&st, t, nullptr);
    } else if (st.status == kRunning) {
      KeySum ks[2] = {KeySum{inf_d(), 0.0}, KeySum{inf_d(), 0.0}};
#pragma unroll
      for (int k = 0; k < SP; ++k)
        if (k < nk) bkpt_index(ks, c[k], sv[k], bl[k], bu[k], st.lam);
      ks[0] = group_ks_min(ks[0]);
      ks[1] = group_ks_min(ks[1]);
      update_after_bkpt<false>(&st, ks, nullptr);
    }
  }
  const bool ok = cqk_has_lambda(st);
  const double lam = ok ? st.lam_final : __builtin_nan("");
  // the rows again (from cache): a slot's loads unguarded, issued together
  constexpr int H = 4;
#pragma unroll
  for (int k0 = 0; k0 < SP; k0 += H) {
    if (k0 < nk) {
      TIn rd[H], ra[H], rb[H], rl[H], ru[H];
#pragma unroll
      for (int k = 0; k < H; ++k) {
        const int64_t i = lane + (k0 + k) * GL;
        const int64_t e = (L > 0) ? base + (i < L ? i : L - 1) : 0;
        rd[k] = V.d[e];
        ra[k] = V.a[e];
        rb[k] = V.b[e];
        rl[k] = V.l[e];
        ru[k] = V.u[e];
      }
#pragma unroll
      for (int k = 0; k < H; ++k) {
        const int64_t i = lane + (k0 + k) * GL;
        if (k0 + k < nk) {
          const double xv = fmin(fmax(fma((double)rb[k], lam, (double)ra[k]) / (double)rd[k],
                                      (double)rl[k]), (double)ru[k]);
          if (i < L) V.x[base + i] = (TIn)(ok ? xv : __builtin_nan(""));
        }
      }
    }
  }
  if (lane == 0 && L >= 0) cqk_row_report(A, s, st, lam, stat);
}

// ---------------------------------------------------------------------------
// One workgroup row: every evaluation streams the row.
// ---------------------------------------------------------------------------
struct CqkLds {
  double red[8 * kWaves];
  double tot[8];
  KeySum ks[2];
  int item;
};

template <typename TIn>
__device__ __forceinline__ void cqk_long_row(const BatCqkArgs& A, int s, int64_t base, int64_t L, CqkLds& S,
                             BatStat& stat) {
  const CqkArrays<TIn> V(A);
  const double r = A.r[s];
  GenState st = cqk_row_state(A, r);
  const TIn* d = V.d + base;
  const TIn* a = V.a + base;
  const TIn* b = V.b + base;
  const TIn* l = V.l + base;
  const TIn* u = V.u + base;
  constexpr int64_t STEP = (int64_t)kBlock * kCqkU;
  // kCqkU values per thread with every load issued before the first use:
  // the loads are unconditional (a lane past the end re-reads the last value,
  // L > i0 >= 0 inside the loop) and the neutral values are selected after,
  // so no load sits behind a branch and its own wait
  auto stream = [&](auto&& fn) {
    for (int64_t i0 = threadIdx.x; i0 < L; i0 += STEP) {
      TIn rd[kCqkU], ra[kCqkU], rb[kCqkU], rl[kCqkU], ru[kCqkU];
#pragma unroll
      for (int k = 0; k < kCqkU; ++k) {
        const int64_t i = i0 + (int64_t)k * kBlock;
        const int64_t ic = i < L ? i : L - 1;
        rd[k] = d[ic];
        ra[k] = a[ic];
        rb[k] = b[ic];
        rl[k] = l[ic];
        ru[k] = u[ic];
      }
      double vd[kCqkU], va[kCqkU], vb[kCqkU], vl[kCqkU], vu[kCqkU];
#pragma unroll
      for (int k = 0; k < kCqkU; ++k) {
        const bool in = i0 + (int64_t)k * kBlock < L;
        vd[k] = in ? (double)rd[k] : 1.0;
        va[k] = in ? (double)ra[k] : 0.0;
        vb[k] = in ? (double)rb[k] : 1.0;
        vl[k] = in ? (double)rl[k] : 0.0;
        vu[k] = in ? (double)ru[k] : 0.0;
      }
#pragma unroll
      for (int k = 0; k < kCqkU; ++k)
        if (i0 + (int64_t)k * kBlock < L) fn(i0 + (int64_t)k * kBlock, vd[k], va[k], vb[k], vl[k], vu[k]);
    }
  };
  if (!(fabs(r) < inf_d())) {
    st.status = CQK_INVALID_ARG;
  } else if (A.lambda0_mode == CQK_LAMBDA0_FORMULA) {
    double acc[3] = {0.0, 0.0, 0.0};
    stream([&](int64_t, double vd, double va, double vb, double vl, double vu) {
      double c, sv, bl, bu;
      to_form(vd, va, vb, vl, vu, c, sv, bl, bu, acc[2]);
      acc[0] += c;
      acc[1] += sv;
    });
    block_reduce<3, 0, 0, kBlock>(acc, nullptr, nullptr, S.red, S.tot);
    if (S.tot[2] > 0.0) st.status = CQK_INVALID_ARG;
    else st.lam = st.lam0 = (S.tot[1] > 0.0) ? (r - S.tot[0]) / S.tot[1] : 0.0;
  }
  while (st.status == kRunning) {
    if (st.mode == kModeEval) {
      Acc acc;
      acc_init(acc);
      double bad = 0.0;
      const double lam = st.lam, lo = st.lo, hi = st.hi;
      stream([&](int64_t, double vd, double va, double vb, double vl, double vu) {
        double c, sv, bl, bu;
        to_form(vd, va, vb, vl, vu, c, sv, bl, bu, bad);
        eval_index<false>(acc, c, sv, bl, bu, lam, lo, hi);
      });
      double v[5] = {acc.s[P_P], acc.s[P_A], acc.s[P_QP], acc.s[P_QM], bad};
      block_reduce<5, 0, 0, kBlock>(v, nullptr, nullptr, S.red, S.tot);
      double t[NSUM];
#pragma unroll
      for (int i = 0; i < NSUM; ++i) t[i] = 0.0;
      t[P_P] = S.tot[0];
      t[P_A] = S.tot[1];
      t[P_QP] = S.tot[2];
      t[P_QM] = S.tot[3];
      t[P_BAD] = S.tot[4];
      t[P_NIN] = (double)L;
      update_after_eval(&st, t, nullptr);
    } else {
      KeySum ks[2] = {KeySum{inf_d(), 0.0}, KeySum{inf_d(), 0.0}};
      const double lam = st.lam;
      double bad = 0.0;
      stream([&](int64_t, double vd, double va, double vb, double vl, double vu) {
        double c, sv, bl, bu;
        to_form(vd, va, vb, vl, vu, c, sv, bl, bu, bad);
        bkpt_index(ks, c, sv, bl, bu, lam);
      });
      block_ks_min<2, kBlock>(ks, S.red, S.ks);
      const KeySum kt[2] = {S.ks[0], S.ks[1]};
      __syncthreads();
      update_after_bkpt(&st, kt, nullptr);
    }
  }
  const bool ok = cqk_has_lambda(st);
  const double lam = ok ? st.lam_final : __builtin_nan("");
  TIn* x = V.x + base;
  stream([&](int64_t i, double vd, double va, double vb, double vl, double vu) {
    const double t = fma(vb, lam, va) / vd;
    x[i] = (TIn)(ok ? fmin(fmax(t, vl), vu) : __builtin_nan(""));
  });
  if (threadIdx.x == 0) cqk_row_report(A, s, st, lam, stat);
}

// ---------------------------------------------------------------------------
// Workgroup rows held on chip by teams of blocks.  A block of kRowBlock
// threads holds E values per thread of the five arrays in registers (FP64: 8,
// FP32: 16, 80 registers either way); a row of bit length b is shared evenly
// by 2^(b - log2(kRowBlock E)) blocks, so it is read from memory once for all its
// evaluations, the blocks exchanging their sums as the single solve's do
// (cqk_team.h).  Four blocks per compute unit: some load while others wait
// for their sums.  Bound by latency (a row's load 10 us, 2 us per evaluation,
// 4-5 us with an exchange) against four rows in flight per compute unit.
// 4e7 values from lambda_0 = 0, streamed / held, FP64: rows of 600 1557 /
// 978 us, 2000 1022 / 541, 8000 1176 / 712, 60 000 1914 / 839, 500 000 4750 /
// 1210; FP32: 1244 / 936, 716 / 480, 697 / 503, 1052 / 570, 4230 / 657.  VJP,
// FP64: 757 / 497, 590 / 493, 775 / 459, 854 / 455, 2330 / 530 (4.9 TB/s).
// ---------------------------------------------------------------------------
constexpr int kRowBlock = 256;
constexpr int kRowBlocksPerCu = 4;
template <typename TIn>
struct RowShape {
  static constexpr int E = 64 / (int)sizeof(TIn);
  static constexpr int kLog = sizeof(TIn) == 8 ? 11 : 12;  // bit length of one block's rows
  static constexpr int kMaxLog = kLog + kBatTeamLogs - 1;  // longest team rows
  static_assert(kRowBlock * E == 1 << kLog, "a row of bit length kLog fits one block");
  static_assert(kMaxLog < kNBW - 1, "and every team row has a bucket of its own length");
  static_assert(kBatTeamMax == 1 << (kMaxLog - kLog), "the longest rows take the largest teams");
};

// Which workgroup rows teams hold in a call of nlong of them: all, where a
// team has anything to hold; otherwise they stay beside the wave rows, where
// the forward kernel may hold a row of one block and streams the others.
// The team kernel comes before those, so it adds its launch, a load and its
// exchanges to the call's time, where a short row's evaluations find it in the
// cache; once it runs, a short row in it costs less than a second round in the
// kernel behind (by each row's own length / all held, us: FP32 6000 rows of
// 600 to 1500 167 / 159, backward 100 / 89, 100 of 5000 to 90 000 backward 97 /
// 70; FP64 3000 of 513 to 1999 backward 98 / 85).
// Rows of bit length kAlways are held in any call; each bit less wants so many
// workgroup rows.
// Rows of one length, streamed / held, us.  FP64: 8 of 1000 values 47 / 52,
// 3000 57 / 54 (but 58 / 73 among rows of 10 to 3000), 6000 81 / 55; 256 of
// 3000 68 / 66 (300 of 600 to 4000 76 / 87), 512 of 3000 87 / 78, 1024 of 1200
// 87 / 81, 2048 of 800 97 / 91.
// FP32: 8 of 3000 53 / 55, 6000 74 / 60; 512 of 3000 70 / 70, 2048 of 2000 113
// / 107, 8192 of 800 180 / 175.  Backward, FP64: 8 of 3000 37 / 42, 6000 44 /
// 42; 512 of 3000 57 / 55, 1024 of 1200 57 / 58, 4096 of 800 81 / 79; FP32: 8
// of 12 000 49 / 43 (but 47 / 58 among rows of 3000 to 9000), 256 of 8000 52 /
// 51, 512 of 6000 56 / 57, 1024 of 3000 67 / 67, 4096 of 2000 99 / 87.
template <typename TIn, bool BACKWARD>
__device__ __forceinline__ int held_from(int nlong) {
  constexpr bool k64 = sizeof(TIn) == 8;
  constexpr int kAlways = (BACKWARD && !k64) ? 15 : 13;
  // from one bit less down to 9, that of the shortest workgroup rows
  constexpr int kLeast[6] = {BACKWARD ? (k64 ? 384 : 256) : 512,
                             BACKWARD ? (k64 ? 1024 : 512) : (k64 ? 1024 : 2048),
                             BACKWARD ? (k64 ? 3072 : 1024) : (k64 ? 2048 : 8192),
                             BACKWARD ? (k64 ? 8192 : 3072) : (k64 ? 4096 : 16384),
                             16384, 32768};
  int b = kAlways;
  while (b > 9 && nlong >= kLeast[kAlways - b]) --b;
  return b;
}

// Where the held rows end in the list (they follow those too long); start: of
// its length buckets, longest first.
template <typename TIn, bool BACKWARD, typename F>
__device__ __forceinline__ int held_end(int nlong, F&& start) {
  const int longer = start(RowShape<TIn>::kMaxLog);
  return start(held_from<TIn, BACKWARD>(nlong) - 1) > longer ? nlong : longer;
}

// The rows of this block one after the other, each with its team.  Longest
// classes first.  Rows of a class go to its teams in turn, starting where the
// class before left off; the rows of one block each come last, from the work
// queue.  Ids, extents and right-hand sides are fetched for kWin rows at a
// time, one lane each.  (Larger teams for a class of few rows, an equal share
// per block of a smaller piece, were slower throughout: 1 row of 12 000 FP64
// values 67 against 56 us, 8 of 30 000 79 / 59, 32 of 100 000 121 / 118.)
template <typename TIn, bool BACKWARD>
struct TeamRows {
  static constexpr int kTeamLog = RowShape<TIn>::kLog, kTeamMaxLog = RowShape<TIn>::kMaxLog;
  static constexpr int kWin = 4;
  Team team;            // of the current row
  int id;               // the row, its first element and length, its r
  int64_t first, len;
  double rhs;
  int b, from, cnt, j, NT, off, per, wi, wn;
  int w_id;             // the window, a row per lane
  int64_t w_first, w_len;
  double w_rhs;
  int bases;            // bucket starts, one per lane
  int end;              // of the held rows in the list
  ItemSource src;

  __device__ __forceinline__ explicit TeamRows(const BatCqkArgs& A) {
    const int lane = threadIdx.x & (kWave - 1);
    bases = (lane < kNBW) ? A.counters[CTR_LBASE + lane] : 0;
    end = held_end<TIn, BACKWARD>(scalar(A.counters[CTR_NLONG]),
                                  [&](int k) { return base_of(k); });
    const uint32_t tag = scalar(A.tctl->base);
    team = Team{nullptr, A.tlimit, tag, 1, 0, kBatTeamBlocks * kSlotWords, late_tag(A.tlate, tag)};
    b = kTeamMaxLog + 1;
    from = cnt = j = off = wi = wn = 0;
    NT = per = 1;
  }

  __device__ __forceinline__ bool none() const { return end <= base_of(kTeamMaxLog); }

  __device__ __forceinline__ int base_of(int k) const {
    return __builtin_amdgcn_readlane(bases, k);
  }

  // rows at + k * step of the list, k < n, into the window
  __device__ __forceinline__ void fetch(const BatCqkArgs& A, int at, int step, int n) {
    const int lane = threadIdx.x & (kWave - 1);
    w_id = 0;
    w_first = w_len = 0;
    w_rhs = 0.0;
    if (lane < n) {
      const size_t e = (size_t)at + (size_t)lane * step;
      w_id = A.list[e];
      w_first = A.lrow[2 * e];
      w_len = A.lrow[2 * e + 1];
      w_rhs = (A.r != nullptr) ? A.r[w_id] : 0.0;
    }
    wi = 0;
    wn = n;
  }

  // The next row (called by the whole block; item: a word of LDS); false at
  // the end.
  __device__ __forceinline__ bool next(const BatCqkArgs& A, int* item) {
    const int G = gridDim.x;
    if (wi == wn && b > kTeamLog) {
      while (j >= cnt) {
        if (b <= kTeamMaxLog) off = (off + cnt % NT * team.T) % (NT * team.T);
        if (--b == kTeamLog) break;
        from = base_of(b);
        cnt = min(end, base_of(b - 1)) - from;
        const int lg = b - kTeamLog, T = 1 << lg, mine = (int)blockIdx.x / T;
        NT = G / T;
        off -= off % T;
        team.T = T;
        team.me = (int)blockIdx.x % T;
        team.slots = A.tslots +
                     ((size_t)lg * 2 * kBatTeamBlocks + (size_t)mine * T) * kSlotWords;
        // a block past the last whole team has no rows of this class
        j = (mine < NT) ? (mine - off / T % NT + NT) % NT : cnt;
      }
      if (b > kTeamLog) {
        const int n = min(kWin, (cnt - j + NT - 1) / NT);
        fetch(A, from + j, NT, n);
        j += n * NT;
      } else {
        from = base_of(kTeamLog);
        cnt = end - from;
        per = min(kWin, max(1, cnt / (G * 4)));
        team.T = 1;
        team.me = 0;
      }
    }
    if (wi == wn) {
      if (cnt <= 0) return false;
      const int nitems = (cnt + per - 1) / per;
      if (threadIdx.x < kWave) {
        const int k = src.next(A.counters + CTR_QUEUE1, nitems);
        if (threadIdx.x == 0) *item = k;
      }
      __syncthreads();
      const int k = scalar(*item);
      __syncthreads();
      if (k >= nitems) return false;
      fetch(A, from + k * per, 1, min(per, cnt - k * per));
    }
    id = __builtin_amdgcn_readlane(w_id, wi);
    first = lane_value(w_first, wi);
    len = lane_value(w_len, wi);
    rhs = lane_value(w_rhs, wi);
    ++wi;
    return true;
  }
};

// This block's share of a row of L values: [lo, hi), whole cache lines of
// FP32 apart.
__device__ __forceinline__ void team_share(const Team& team, int L, int& lo, int& hi) {
  const int per = ((L + team.T - 1) / team.T + 31) / 32 * 32;
  lo = min(L, per * team.me);
  hi = min(L, lo + per);
}

// Vectors q = 0, 1, ... of an array for one thread: values lo + (q kRowBlock +
// tid) V ... of a share [lo, hi) of a row of at least V values.  A vector that
// would pass hi is moved back to end there, and the thread then owns only the
// values no other thread holds; so every load is a whole vector with no test
// before it, and all of a share's loads are in flight together.
template <typename TIn>
struct ShareVec {
  static constexpr int V = VecWidth<TIn>::value;
  typedef typename Raw16<TIn>::type Raw;
  int lo, hi;   // a team row has fewer than 2^31 values
  int tid;
  __device__ __forceinline__ int want(int q) const { return lo + (q * kRowBlock + tid) * V; }
  __device__ __forceinline__ int at(int q) const { return min(want(q), hi - V); }
  __device__ __forceinline__ bool owns(int q, int k) const { return at(q) + k >= want(q); }
  __device__ __forceinline__ int groups() const {
    return (hi - lo + kRowBlock * V - 1) / (kRowBlock * V);
  }
  __device__ __forceinline__ Raw load(const TIn* p, int q) const {
    return *reinterpret_cast<const Raw*>(p + (unsigned)at(q));
  }
  __device__ __forceinline__ void store(TIn* p, int q, Raw o) const {
    const unsigned i = (unsigned)at(q);
    if ((int)i == want(q)) {
      st16(p + i, o);
    } else {
#pragma unroll
      for (int k = 1; k < V; ++k)
        if (owns(q, k)) p[i + k] = o[k];
    }
  }
};

// One row of a team.  The block keeps its share of the five arrays as loaded
// and makes the per-index form again at every evaluation: holding the form
// instead would mean reading the arrays a second time for x (eq. (xopt) from
// the arrays' own values), which took twice as long as the load itself.
template <typename TIn, int E>
__device__ __forceinline__ bool cqk_team_row(const BatCqkArgs& A, TeamLds<kRowBlock>& S,
                                             BatStat& stat, int& par, Team& team, int s,
                                             int64_t base, int64_t L, double r) {
  constexpr int V = VecWidth<TIn>::value;
  constexpr int Q = E / V;
  typedef typename Raw16<TIn>::type Raw;
  const CqkArrays<TIn> P(A);
  ShareVec<TIn> B;
  B.tid = threadIdx.x;
  asm volatile("" : "+v"(B.tid));  // nothing made from it is hoisted out of the loop over rows
  team_share(team, (int)L, B.lo, B.hi);
  const int nq = B.groups();
  Raw rd[Q], ra[Q], rb[Q], rl[Q], ru[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q < nq) {
      rd[q] = B.load(P.d + base, q);
      ra[q] = B.load(P.a + base, q);
      rb[q] = B.load(P.b + base, q);
      rl[q] = B.load(P.l + base, q);
      ru[q] = B.load(P.u + base, q);
    }
  }
  // The form is made anew for each use, one vector after the other: kept
  // across the evaluations by the compiler, or made for all values at once,
  // it would be spilled.  (What the kernel does spill, 19 VGPRs and 80 B of
  // scratch a lane, and 72 to 75 SGPRs into VGPR lanes, is the rest of its
  // state: four blocks per compute unit leave it 128 VGPRs.)
  auto hold = [&]() {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      asm volatile("" : "+v"(rd[q]), "+v"(ra[q]), "+v"(rb[q]), "+v"(rl[q]), "+v"(ru[q]));
  };
  auto each = [&](auto&& fn) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (q < nq) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < V; ++k) {
          double c, sv, bl, bu, b1 = 0.0;
          to_form((double)rd[q][k], (double)ra[q][k], (double)rb[q][k], (double)rl[q][k],
                  (double)ru[q][k], c, sv, bl, bu, b1);
          fn(c, sv, bl, bu);
        }
      }
    }
  };
  double bad = 0.0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q >= nq) break;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      double c, sv, bl, bu, b1 = 0.0;
      to_form((double)rd[q][k], (double)ra[q][k], (double)rb[q][k], (double)rl[q][k],
              (double)ru[q][k], c, sv, bl, bu, b1);
      const bool in = B.owns(q, k);
      bad += in ? b1 : 0.0;
      // a value another thread owns: b = 0, so it adds nothing to any sum
      rd[q][k] = in ? rd[q][k] : (TIn)1;
      ra[q][k] = in ? ra[q][k] : (TIn)0;
      rb[q][k] = in ? rb[q][k] : (TIn)0;
      rl[q][k] = in ? rl[q][k] : (TIn)0;
      ru[q][k] = in ? ru[q][k] : (TIn)0;
    }
  }
  hold();
  GenState st = cqk_row_state(A, r);
  if (!(fabs(r) < inf_d())) st.status = CQK_INVALID_ARG;
  bool ok = true;
  if (A.lambda0_mode == CQK_LAMBDA0_FORMULA && st.status == kRunning) {
    double v[3] = {0.0, 0.0, bad}, tot[3];
    each([&](double c, double sv, double, double) {
      v[0] += c;
      v[1] += sv;
    });
    ok = team_reduce<3, kRowBlock>(team, S, par, v, tot);
    if (tot[2] > 0.0) st.status = CQK_INVALID_ARG;
    else st.lam = st.lam0 = scalar((tot[1] > 0.0) ? (r - tot[0]) / tot[1] : 0.0);
  }
  while (ok && st.status == kRunning) {
    hold();
    const double lam = st.lam;
    if (st.mode == kModeEval) {
      Acc acc;
      acc_init(acc);
      each([&](double c, double sv, double bl, double bu) {
        eval_index<false>(acc, c, sv, bl, bu, lam, 0.0, 0.0);
      });
      const double v[5] = {acc.s[P_P], acc.s[P_A], acc.s[P_QP], acc.s[P_QM], bad};
      double tot[5], t[NSUM];
      ok = team_reduce<5, kRowBlock>(team, S, par, v, tot);
      t[P_P] = tot[0];
      t[P_A] = tot[1];
      t[P_QP] = tot[2];
      t[P_QM] = tot[3];
      t[P_BAD] = tot[4];
      update_after_eval<false>(&st, t, nullptr);
    } else {
      KeySum ks[2] = {KeySum{inf_d(), 0.0}, KeySum{inf_d(), 0.0}};
      each([&](double c, double sv, double bl, double bu) {
        bkpt_index(ks, c, sv, bl, bu, lam);
      });
      ok = team_reduce_ks<kRowBlock>(team, S, par, ks);
      update_after_bkpt<false>(&st, ks, nullptr);
    }
    state_to_scalars(st);
  }
  if (!ok) return false;
  const bool has = cqk_has_lambda(st);
  const double lam = has ? st.lam_final : __builtin_nan("");
  hold();
  asm volatile("" : "+v"(B.tid));  // the addresses again
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q < nq) {
      __builtin_amdgcn_sched_barrier(0);
      Raw o;
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const double t = fma((double)rb[q][k], lam, (double)ra[q][k]) / (double)rd[q][k];
        o[k] = (TIn)(has ? fmin(fmax(t, (double)rl[q][k]), (double)ru[q][k])
                         : __builtin_nan(""));
      }
      B.store(P.x + base, q, o);
    }
  }
  if (threadIdx.x == 0 && team.me == 0) cqk_row_report(A, s, st, lam, stat);
  return true;
}

// What a team kernel does after its last row.
__device__ __forceinline__ void team_end(const BatCqkArgs& A, const Team& team, uint32_t base_tag,
                                         bool ok) {
  if (threadIdx.x == 0) {
    if (!ok) {
      atomicOr(&A.counters[CTR_GAVE_UP], (int)kGaveUp);
      A.tctl->flags.gave_up = kGaveUp;
    }
    if (team.tag != base_tag) atomicMax(&A.tctl->last, team.tag);
  }
}

template <typename TIn>
__global__ __launch_bounds__(kRowBlock, kRowBlocksPerCu) void bat_cqk_team_kernel(BatCqkArgs A) {
  __shared__ TeamLds<kRowBlock> S;
  __shared__ BatStat stat;
  __shared__ int item;
  TeamRows<TIn, false> rows(A);
  if (rows.none() || team_is_off(&A.tctl->flags, &S.gave_up)) return;
  stat_init(stat);
  if (threadIdx.x == 0) S.gave_up = 0;
  __syncthreads();
  const uint32_t base_tag = rows.team.tag;
  int par = 0;
  bool ok = true;
  while (ok && rows.next(A, &item))
    ok = rows.team.tag < kTagEnd - 4096u &&
         cqk_team_row<TIn, RowShape<TIn>::E>(A, S, stat, par, rows.team, rows.id, rows.first, rows.len, rows.rhs);
  team_end(A, rows.team, base_tag, ok);
  __syncthreads();
  stat_flush<true>(stat, A.counters + CTR_STAT1);
}

// Workgroup rows that no team holds (their number, of nlong): those past the
// longest team rows and, by the rule above, all shorter ones or none, or all
// of them when a team gave up or there are none; and the list entry of one.
template <typename TIn, bool BACKWARD>
__device__ __forceinline__ int streamed_rows(const BatCqkArgs& A, int nlong) {
  if (A.tslots == nullptr || A.counters[CTR_GAVE_UP]) return nlong;
  auto start = [&](int k) { return A.counters[CTR_LBASE + k]; };
  return nlong - (held_end<TIn, BACKWARD>(nlong, start) - start(RowShape<TIn>::kMaxLog));
}
template <typename TIn>
__device__ __forceinline__ size_t streamed_entry(const BatCqkArgs& A, int row, int nlong,
                                                 int nstream) {
  const int longer = scalar(A.counters[CTR_LBASE + RowShape<TIn>::kMaxLog]);
  return (size_t)(row < longer ? row : row + (nlong - nstream));
}

// The wave rows, four to a block at a time; each wave takes kRowsPerWave rows
// of an item one after the other when there are enough items to go round, so
// the block meets less often.  A kernel of its own: the registers of a
// workgroup row's loads would cost its waves' occupancy.
constexpr int kRowsPerWave = 4;

//
// Workgroup rows that no team holds come beside them.  HOLD: those of one block
// are held, as a team of one would, with the same sums in the same order, so a
// row's result does not depend on how many others the call has (6000 FP32 rows
// of 513 to 999 values take 121 us, streamed 146, in teams 145; FP64 144, 177
// and 145).  Not in calls of so many rows that the shortest have a kernel of
// their own: there the wave rows bound the time, and the code for the others
// costs them 4 of 256 us (65 536 FP32 rows of 64 to 512 values).  The other
// workgroup rows stream from memory at every evaluation.
template <int SP, typename TIn, bool HOLD>
__global__ __launch_bounds__(kBlock, 3) void bat_cqk_solve_kernel(BatCqkArgs A) {
  __shared__ BatStat stat;
  __shared__ CqkLds S;
  __shared__ TeamLds<kRowBlock> one;
  Team alone = team_alone();
  int par = 0;
  const int nlong = A.counters[CTR_NLONG];
  const int nstream = streamed_rows<TIn, false>(A, nlong);
  // the shortest may be the group kernel's
  const int nshort = A.grouped ? A.counters[CTR_GROUPS] - nlong : A.counters[CTR_NSHORT];
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int per = min(kRowsPerWave, max(1, nshort / ((int)gridDim.x * kWaves * kRowsPerWave)));
  const int ngroups = (nshort + kWaves * per - 1) / (kWaves * per);
  const int nitems = nstream + ngroups;
  ItemSource src;
  stat_init(stat);
  for (;;) {
    if (threadIdx.x < kWave) {
      const int next = src.next(A.counters + CTR_QUEUE0, nitems);
      if (threadIdx.x == 0) S.item = next;
    }
    __syncthreads();
    int item = scalar(S.item);
    __syncthreads();
    if (item >= nitems) break;
    const int row = A.short_first ? item - ngroups : item;
    if (row >= 0 && row < nstream) {
      const size_t e = streamed_entry<TIn>(A, row, nlong, nstream);
      const int id = A.list[e];
      const int64_t first = A.lrow[2 * e], len = A.lrow[2 * e + 1];
      if (HOLD && len < (1 << RowShape<TIn>::kLog))
        cqk_team_row<TIn, RowShape<TIn>::E>(A, one, stat, par, alone, id, first, len, A.r[id]);
      else
        cqk_long_row<TIn>(A, id, first, len, S, stat);
      __syncthreads();
      continue;
    }
    if (!A.short_first) item -= nstream;
    // the wave's rows of this item: ids, extents and right-hand sides in two
    // round trips for all of them, one lane each
    const int lane = threadIdx.x & (kWave - 1);
    const int k0 = item * per * kWaves + wid;
    int id = 0;
    int64_t first = 0, len = 0;
    double rhs = 0.0;
    if (lane < per && k0 + lane * kWaves < nshort) {
      const size_t e = (size_t)nlong + k0 + lane * kWaves;
      id = A.list[e];
      first = A.lrow[2 * e];
      len = A.lrow[2 * e + 1];
      rhs = A.r[id];
    }
    for (int j = 0; j < per && k0 + j * kWaves < nshort; ++j)
      cqk_short_row<SP, TIn>(A, __builtin_amdgcn_readlane(id, j), lane_value(first, j),
                             lane_value(len, j), lane_value(rhs, j), stat);
  }
  __syncthreads();
  stat_flush<true>(stat, A.counters + CTR_STAT0);
}

// The shortest rows (list entries from CTR_GROUPS on), four to a wave at a
// time; all about as long, so they are handed out by number.  Bound by FP64
// instructions, of which a row to a wave spends about half on reductions and
// the scalar update.  65 536 rows, whole calls, a row to a wave against this:
// 100 values FP32 212 -> 144 us, FP64 264 -> 153; 16 values FP32 202 -> 120,
// FP64 220 -> 116.  (Two rows of up to 256 values to a wave gained nothing.)
template <typename TIn>
__global__ __launch_bounds__(kBlock, 3) void bat_cqk_group_kernel(BatCqkArgs A) {
  __shared__ BatStat stat;
  stat_init(stat);
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  constexpr int NG = kWave / kGroupLanes;
  const int first = A.counters[CTR_GROUPS];
  const int end = A.counters[CTR_NLONG] + A.counters[CTR_NSHORT];
  const int wave = blockIdx.x * kWaves + scalar((int)(threadIdx.x / kWave));
  for (int64_t k = first + (int64_t)wave * NG; k < end; k += (int64_t)gridDim.x * kWaves * NG) {
    const int64_t e = k + lane / kGroupLanes;
    int id = 0;
    int64_t base = 0, len = -1;
    double r = 0.0;
    if (e < end) {
      id = A.list[e];
      base = A.lrow[2 * e];
      len = A.lrow[2 * e + 1];
      r = A.r[id];
    }
    cqk_group_rows<TIn>(A, id, base, len, r, stat);
  }
  __syncthreads();
  stat_flush<true>(stat, A.counters + CTR_STAT0);
}

// Backward of one wave row.
template <int SP, typename TIn>
__device__ void cqk_vjp_short_row(const BatCqkArgs& A, int s, int64_t base, int64_t L) {
  const CqkArrays<TIn> V(A);
  const int lane = threadIdx.x & (kWave - 1);
  double q = 0.0, m = 0.0;
  double gv[SP], bd[SP], dv[SP];
  bool fr[SP];
#pragma unroll
  for (int k = 0; k < SP; ++k) {
    fr[k] = false;
    gv[k] = bd[k] = 0.0;
    dv[k] = 1.0;
  }
  if (L > 0) {
    // every load issued before the first use (index clamped to the row)
    TIn rx[SP], rl[SP], ru[SP], rg[SP], rd[SP], rb[SP];
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      const int64_t i = lane + (int64_t)k * kWave;
      const int64_t e = base + (i < L ? i : L - 1);
      rx[k] = V.x[e];
      rl[k] = V.l[e];
      ru[k] = V.u[e];
      rg[k] = V.g[e];
      rd[k] = V.d[e];
      rb[k] = V.b[e];
    }
#pragma unroll
    for (int k = 0; k < SP; ++k) {
      if (lane + (int64_t)k * kWave < L) {
        const double xv = (double)rx[k];
        fr[k] = (xv > (double)rl[k]) && (xv < (double)ru[k]);
        gv[k] = (double)rg[k];
        dv[k] = (double)rd[k];
        bd[k] = (double)rb[k];
        if (fr[k]) {
          q += bd[k] * bd[k] / dv[k];
          m += gv[k] * bd[k] / dv[k];
        }
      }
    }
  }
  q = wave_sum(q);
  m = wave_sum(m);
  const double mu = (q > 0.0) ? m / q : 0.0;
#pragma unroll
  for (int k = 0; k < SP; ++k) {
    const int64_t i = lane + (int64_t)k * kWave;
    if (i < L) V.ga[base + i] = (TIn)(fr[k] ? (gv[k] - bd[k] * mu) / dv[k] : 0.0);
  }
  if (lane == 0 && A.gr) A.gr[s] = mu;
}

// Backward of one workgroup row: the two sums, then the map.
template <typename TIn>
__device__ void cqk_vjp_long_row(const BatCqkArgs& A, int s, int64_t base, int64_t L,
                                 CqkLds& S) {
  const CqkArrays<TIn> V(A);
  constexpr int64_t STEP = (int64_t)kBlock * kCqkU;
  // kCqkU values per thread, all six loads of each issued before the first
  // use (index clamped to the row, L > i0 >= 0 inside the loop); lanes past
  // the end count as not free
  auto stream = [&](int64_t i0, bool (&fr)[kCqkU], double (&xg)[kCqkU], double (&xb)[kCqkU],
                    double (&xd)[kCqkU]) {
    TIn rx[kCqkU], rl[kCqkU], ru[kCqkU], rb[kCqkU], rd[kCqkU], rg[kCqkU];
#pragma unroll
    for (int k = 0; k < kCqkU; ++k) {
      const int64_t i = i0 + (int64_t)k * kBlock;
      const int64_t e = base + (i < L ? i : L - 1);
      rx[k] = V.x[e];
      rl[k] = V.l[e];
      ru[k] = V.u[e];
      rb[k] = V.b[e];
      rd[k] = V.d[e];
      rg[k] = V.g[e];
    }
#pragma unroll
    for (int k = 0; k < kCqkU; ++k) {
      const double xv = (double)rx[k];
      fr[k] = (i0 + (int64_t)k * kBlock < L) && (xv > (double)rl[k]) && (xv < (double)ru[k]);
      xg[k] = (double)rg[k];
      xb[k] = (double)rb[k];
      xd[k] = (double)rd[k];
    }
  };
  double acc[2] = {0.0, 0.0};
  for (int64_t i0 = threadIdx.x; i0 < L; i0 += STEP) {
    bool fr[kCqkU];
    double xg[kCqkU], xb[kCqkU], xd[kCqkU];
    stream(i0, fr, xg, xb, xd);
#pragma unroll
    for (int k = 0; k < kCqkU; ++k) {
      if (fr[k]) {
        acc[0] += xb[k] * xb[k] / xd[k];
        acc[1] += xg[k] * xb[k] / xd[k];
      }
    }
  }
  block_reduce<2, 0, 0, kBlock>(acc, nullptr, nullptr, S.red, S.tot);
  const double q = S.tot[0];
  const double mu = (q > 0.0) ? S.tot[1] / q : 0.0;
  for (int64_t i0 = threadIdx.x; i0 < L; i0 += STEP) {
    bool fr[kCqkU];
    double xg[kCqkU], xb[kCqkU], xd[kCqkU];
    stream(i0, fr, xg, xb, xd);
#pragma unroll
    for (int k = 0; k < kCqkU; ++k) {
      const int64_t i = i0 + (int64_t)k * kBlock;
      if (i < L) V.ga[base + i] = (TIn)(fr[k] ? (xg[k] - xb[k] * mu) / xd[k] : 0.0);
    }
  }
  if (threadIdx.x == 0 && A.gr) A.gr[s] = mu;
}

// Backward of one team row: the share's g, d and b stay in registers from the
// sums to the map, so the row is read once.
template <typename TIn, int E>
__device__ __forceinline__ bool cqk_team_vjp_row(const BatCqkArgs& A, TeamLds<kRowBlock>& S,
                                                 int& par, Team& team, int s, int64_t base,
                                                 int64_t L) {
  constexpr int V = VecWidth<TIn>::value;
  constexpr int Q = E / V;
  typedef typename Raw16<TIn>::type Raw;
  const CqkArrays<TIn> P(A);
  ShareVec<TIn> B;
  B.tid = threadIdx.x;
  asm volatile("" : "+v"(B.tid));  // nothing made from it is hoisted out of the loop over rows
  team_share(team, (int)L, B.lo, B.hi);
  const int nq = B.groups();
  Raw rg[Q], rd[Q], rb[Q];
  uint32_t fr = 0;  // free and owned by this thread
  {
    Raw rx[Q], rl[Q], ru[Q];
    // FP32: a vector past the share is not loaded (rows of 600 values 391 ->
    // 344 us for 40e6); FP64 has half as many to save, and the branches cost
    // it more registers than they save loads (rows of 60000 455 -> 480 us)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (sizeof(TIn) == 8 || q < nq) {
        rx[q] = B.load(P.x + base, q);
        rl[q] = B.load(P.l + base, q);
        ru[q] = B.load(P.u + base, q);
        rg[q] = B.load(P.g + base, q);
        rd[q] = B.load(P.d + base, q);
        rb[q] = B.load(P.b + base, q);
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int k = 0; k < V; ++k)
        if ((sizeof(TIn) == 8 || q < nq) && B.owns(q, k) && rx[q][k] > rl[q][k] && rx[q][k] < ru[q][k]) fr |= 1u << (q * V + k);
  }
  double v[2] = {0.0, 0.0}, tot[2];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      if ((fr >> (q * V + k)) & 1u) {
        const double xb = (double)rb[q][k], xd = (double)rd[q][k];
        v[0] += xb * xb / xd;
        v[1] += (double)rg[q][k] * xb / xd;
      }
    }
  }
  if (!team_reduce<2, kRowBlock>(team, S, par, v, tot)) return false;
  const double mu = (tot[0] > 0.0) ? tot[1] / tot[0] : 0.0;
  asm volatile("" : "+v"(B.tid));  // the addresses again
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q < nq) {
      __builtin_amdgcn_sched_barrier(0);
      Raw o;
#pragma unroll
      for (int k = 0; k < V; ++k)
        o[k] = (TIn)(((fr >> (q * V + k)) & 1u)
                         ? ((double)rg[q][k] - (double)rb[q][k] * mu) / (double)rd[q][k]
                         : 0.0);
      B.store(P.ga + base, q, o);
    }
  }
  if (threadIdx.x == 0 && team.me == 0 && A.gr) A.gr[s] = mu;
  return true;
}

template <typename TIn>
__global__ __launch_bounds__(kRowBlock, kRowBlocksPerCu) void bat_cqk_team_vjp_kernel(
    BatCqkArgs A) {
  __shared__ TeamLds<kRowBlock> S;
  __shared__ int item;
  TeamRows<TIn, true> rows(A);
  if (rows.none() || team_is_off(&A.tctl->flags, &S.gave_up)) return;
  if (threadIdx.x == 0) S.gave_up = 0;
  __syncthreads();
  const uint32_t base_tag = rows.team.tag;
  int par = 0;
  bool ok = true;
  while (ok && rows.next(A, &item))
    ok = rows.team.tag < kTagEnd - 4096u &&
         cqk_team_vjp_row<TIn, RowShape<TIn>::E>(A, S, par, rows.team, rows.id, rows.first,
                                                 rows.len);
  team_end(A, rows.team, base_tag, ok);
}

// The wave rows and the workgroup rows that no team holds.
template <int SP, typename TIn>
__global__ __launch_bounds__(kBlock) void bat_cqk_vjp_kernel(BatCqkArgs A) {
  __shared__ CqkLds S;
  const int nlong = A.counters[CTR_NLONG];
  const int nshort = A.counters[CTR_NSHORT];
  const int nstream = streamed_rows<TIn, true>(A, nlong);
  const int nsg = (nshort + kWaves - 1) / kWaves;
  const int nitems = nstream + nsg;
  ItemSource src;
  for (;;) {
    if (threadIdx.x < kWave) {
      const int next = src.next(A.counters + CTR_QUEUE0, nitems);
      if (threadIdx.x == 0) S.item = next;
    }
    __syncthreads();
    const int item = S.item;
    __syncthreads();
    if (item >= nitems) break;
    int idx;
    bool is_long;
    if (A.short_first) {
      is_long = item >= nsg;
      idx = is_long ? item - nsg : item;
    } else {
      is_long = item < nstream;
      idx = is_long ? item : item - nstream;
    }
    if (is_long) {
      const size_t e = streamed_entry<TIn>(A, idx, nlong, nstream);
      cqk_vjp_long_row<TIn>(A, A.list[e], A.lrow[2 * e], A.lrow[2 * e + 1],
                            S);
    } else {
      const int k = idx * kWaves + (int)(threadIdx.x / kWave);
      if (k < nshort) {
        const size_t e = (size_t)nlong + k;
        cqk_vjp_short_row<SP, TIn>(A, A.list[e], A.lrow[2 * e], A.lrow[2 * e + 1]);
      }
    }
    __syncthreads();
  }
}

// The outcome of a forward call from the host copy of its counters: the
// groups' lines combined.
BatStat host_stat(const int32_t* hc, bool max_over) {
  BatStat t{0, 0, 0};
  const int lines = hc[CTR_GAVE_UP] ? kQueues : 2 * kQueues;
  for (int q = 0; q < lines; ++q) {
    const int32_t* line = hc + CTR_STAT0 + q * kCtrLine;
    t.flags |= line[CTR_FLAGS];
    t.surv += line[CTR_SURV];
    t.over = max_over ? std::max(t.over, line[CTR_OVER]) : t.over + line[CTR_OVER];
  }
  return t;
}

struct BatWs {
  int32_t* list;
  int32_t* counters;
  int32_t* bhist;
  int64_t* lrow;
};

constexpr size_t round256(size_t v) { return (v + 255) / 256 * 256; }

// Bytes of the planning buffers of a batched call on nseg rows: the row list,
// the counters, the bucket histogram of each planning block and the row
// extents, each on a 256-byte boundary.
constexpr size_t bat_ws_bytes(size_t nseg) {
  return round256(nseg * sizeof(int32_t)) + round256(CTR_TOTAL * sizeof(int32_t)) +
         round256((nseg > kPBlock ? (nseg + kPBlock - 1) / kPBlock : 1) * kNB * sizeof(int32_t)) +
         round256(nseg * 2 * sizeof(int64_t));
}

// Carves the planning buffers out of base (bat_ws_bytes(nseg) bytes).
void bat_layout(void* base, int32_t nseg, BatWs* w) {
  const size_t list_bytes = round256((size_t)nseg * sizeof(int32_t));
  const size_t ctr_bytes = round256(CTR_TOTAL * sizeof(int32_t));
  const size_t nblk = std::max<size_t>(1, ((size_t)nseg + kPBlock - 1) / kPBlock);
  const size_t hist_bytes = round256(nblk * kNB * sizeof(int32_t));
  char* p = (char*)base;
  w->list = (int32_t*)p;
  w->counters = (int32_t*)(p + list_bytes);
  w->bhist = (int32_t*)(p + list_bytes + ctr_bytes);
  w->lrow = (int64_t*)(p + list_bytes + ctr_bytes + hist_bytes);
}

cqk_status bat_workspace(cqk_ctx* ctx, int32_t nseg, BatWs* w) {
  cqk_status st = ensure_buffer(ctx, ctx->ws, bat_ws_bytes((size_t)nseg));
  if (st != CQK_OK) return st;
  bat_layout(ctx->ws.ptr, nseg, w);
  return CQK_OK;
}

// The planning buffers of cqk_project_simplex_batched_noalloc_f32: a fixed
// device array (one copy per GPU, alive until the process ends) for up to
// CQK_NOALLOC_MAX_SEG rows.  Host code never names it in a launch or a copy:
// its address on a device comes from hipGetSymbolAddress (noalloc_scratch).
static_assert(CQK_NOALLOC_MAX_SEG > 0, "row limit of the no-allocation call");
constexpr size_t kScratchBytes = bat_ws_bytes(CQK_NOALLOC_MAX_SEG);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

int persistent_grid(cqk_ctx* ctx, const cqk_batch_schedule& sc, int nseg) {
  const int g = ctx->num_cus * sc.blocks_per_cu;
  return std::max(1, std::min(g, nseg));
}

template <typename Args>
void plan(cqk_ctx* ctx, const Args& A) {
  hipStream_t s = ctx->stream;
  const int gb = std::max(1, (A.nseg + kPBlock - 1) / kPBlock);
  if (gb > 1) hipLaunchKernelGGL(bat_count_kernel<Args>, dim3(gb), dim3(kPBlock), 0, s, A);
  hipLaunchKernelGGL(bat_place_kernel<Args>, dim3(gb), dim3(kPBlock), 0, s, A);
}

// Rows above the register limit and up to medium_tiles tiles are solved by
// one wave.
void apply_schedule(const cqk_batch_schedule& sc, BatArgs* A) {
  A->small_max = kWave * sc.small_per;
  A->med_max = std::max(A->small_max, sc.medium_tiles * kWTile);
  A->short_first = sc.short_first;
}

// Queues one forward call under schedule sc.
void launch_forward(cqk_ctx* ctx, const cqk_batch_schedule& sc, BatArgs A) {
  apply_schedule(sc, &A);
  plan(ctx, A);
  const dim3 grid(persistent_grid(ctx, sc, A.nseg));
  if (sc.small_per == 4)
    hipLaunchKernelGGL(bat_solve_kernel<4>, grid, dim3(kBlock), 0, ctx->stream, A);
  else
    hipLaunchKernelGGL(bat_solve_kernel<8>, grid, dim3(kBlock), 0, ctx->stream, A);
}

void launch_backward(cqk_ctx* ctx, const cqk_batch_schedule& sc, BatArgs A) {
  apply_schedule(sc, &A);
  plan(ctx, A);
  const dim3 grid(persistent_grid(ctx, sc, A.nseg));
  if (sc.small_per == 4)
    hipLaunchKernelGGL(bat_vjp_kernel<4>, grid, dim3(kBlock), 0, ctx->stream, A);
  else
    hipLaunchKernelGGL(bat_vjp_kernel<8>, grid, dim3(kBlock), 0, ctx->stream, A);
}

BatArgs forward_args(int32_t nseg, const int64_t* offsets, const float* y, const double* r,
                     double r_scalar, float* x, double* lambda_out, int32_t* nfree_out,
                     const BatWs& w) {
  BatArgs A{};
  A.nseg = nseg;
  A.off = offsets;
  A.y = y;
  A.r = r;
  A.r_scalar = r_scalar;
  A.x = x;
  A.lam_out = lambda_out;
  A.nfree_out = nfree_out;
  A.list = w.list;
  A.counters = w.counters;
  A.bhist = w.bhist;
  A.lrow = w.lrow;
  return A;
}

BatArgs backward_args(int32_t nseg, const int64_t* offsets, const float* x, const float* g,
                      float* grad_y, double* grad_r, const BatWs& w) {
  BatArgs A{};
  A.nseg = nseg;
  A.off = offsets;
  A.x = const_cast<float*>(x);
  A.g = g;
  A.gy = grad_y;
  A.gr = grad_r;
  A.list = w.list;
  A.counters = w.counters;
  A.bhist = w.bhist;
  A.lrow = w.lrow;
  return A;
}

// The candidate schedules the tuner times.
// The batched simplex candidates: also the medium-row limit (medium_tiles,
// in tiles of 1024 values; 0: none).
int candidate_schedules_fwd(cqk_batch_schedule* out, int cap) {
  int k = 0;
  for (int sp : {4, 8})
    for (int bpc : {2, 3, 4, 6})
      for (int sf : {0, 1})
        for (int med : {0, 4, 8, 16, 32, 64})
          if (k < cap) out[k++] = cqk_batch_schedule{sp, bpc, sf, med};
  return k;
}

int candidate_schedules(cqk_batch_schedule* out, int cap) {
  int k = 0;
  for (int sp : {4, 8})
    for (int bpc : {1, 2, 3, 4})
      for (int sf : {0, 1})
        if (k < cap) out[k++] = cqk_batch_schedule{sp, bpc, sf, 0};
  return k;
}

// Times `launch` for each candidate (`repeats` runs each after one warm-up,
// the fastest counts) and returns the index of the best.
template <typename Launch>
cqk_status tune(cqk_ctx* ctx, const cqk_batch_schedule* cand, int ncand, int repeats,
                Launch launch, int* best, double* best_ms) {
  cqk_status st = ensure_events(ctx, 2);
  if (st != CQK_OK) return st;
  hipStream_t s = ctx->stream;
  *best = 0;
  *best_ms = 1e300;
  for (int c = 0; c < ncand; ++c) {
    launch(cand[c]);
    double t = 1e300;
    for (int k = 0; k < repeats; ++k) {
      hipEventRecord(ctx->events[0], s);
      launch(cand[c]);
      hipEventRecord(ctx->events[1], s);
      if (hip_ok(hipEventSynchronize(ctx->events[1])) != CQK_OK) return CQK_DEVICE_ERROR;
      float ms = 0.f;
      hipEventElapsedTime(&ms, ctx->events[0], ctx->events[1]);
      t = std::min(t, (double)ms);
    }
    if (hip_ok(hipGetLastError()) != CQK_OK) return CQK_DEVICE_ERROR;
    if (t < *best_ms) {
      *best_ms = t;
      *best = c;
    }
  }
  return CQK_OK;
}


// Batched general CQK: the plan, then one persistent launch.
BatCqkArgs cqk_args(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets, const void* d, const void* a,
                    const void* b, const void* l, const void* u, const BatWs& w) {
  BatCqkArgs A{};
  A.nseg = nseg;
  A.off = offsets;
  A.d = d;
  A.a = a;
  A.b = b;
  A.l = l;
  A.u = u;
  A.list = w.list;
  A.counters = w.counters;
  A.bhist = w.bhist;
  A.lrow = w.lrow;
  // every team size finds its blocks on the GPU at once
  if (kRowBlocksPerCu * ctx->num_cus >= kBatTeamMax && team_ready(ctx, 0)) {
    A.tctl = (BatTeamCtl*)((char*)ctx->team.ptr + kTeamBatCtl);
    A.tslots = (uint64_t*)((char*)ctx->team.ptr + kTeamBatSlots);
    A.tlimit = ctx->team_wait;
    A.tlate = ctx->team_late;
    A.tepoch = ctx->team_epoch;
  }
  return A;
}

// The batched general CQK under schedule sc: rows of at most
// 64 * small_per values go to one wave (small_per 4 or 8 values per lane in
// registers), blocks_per_cu persistent workgroups per compute unit.
void cqk_apply_schedule(cqk_ctx* ctx, const cqk_batch_schedule& sc, BatCqkArgs* A, dim3* grid) {
  A->small_max = kWave * sc.small_per;
  A->short_first = sc.short_first;
  *grid = dim3(std::max(1, std::min(ctx->num_cus * sc.blocks_per_cu, A->nseg)));
}

// The rows of teams; the rows it leaves (all of them when a team gave up) go
// to the kernel queued behind it.
template <typename Kern>
void launch_teams(cqk_ctx* ctx, const BatCqkArgs& A, Kern kern) {
  if (A.tslots == nullptr) return;
  const dim3 grid(std::min(kBatTeamBlocks, kRowBlocksPerCu * ctx->num_cus));
  hipLaunchKernelGGL(kern, grid, dim3(kRowBlock), 0, ctx->stream, A);
}

template <typename TIn>
void launch_cqk_forward(cqk_ctx* ctx, const cqk_batch_schedule& sc, BatCqkArgs A) {
  dim3 grid;
  cqk_apply_schedule(ctx, sc, &A, &grid);
  plan(ctx, A);
  launch_teams(ctx, A, bat_cqk_team_kernel<TIn>);
  // the shortest rows side by side, when there are enough of them to go round
  A.grouped = A.nseg >= kGroupMinRows ? 1 : 0;
  if (A.grouped)
    hipLaunchKernelGGL((bat_cqk_group_kernel<TIn>), dim3(3 * ctx->num_cus), dim3(kBlock), 0,
                       ctx->stream, A);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(kBlock), 0, ctx->stream, A); };
  if (A.grouped)
    sc.small_per == 4 ? go(bat_cqk_solve_kernel<4, TIn, false>)
                      : go(bat_cqk_solve_kernel<8, TIn, false>);
  else
    sc.small_per == 4 ? go(bat_cqk_solve_kernel<4, TIn, true>)
                      : go(bat_cqk_solve_kernel<8, TIn, true>);
}

template <typename TIn>
void launch_cqk_backward(cqk_ctx* ctx, const cqk_batch_schedule& sc, BatCqkArgs A) {
  dim3 grid;
  cqk_apply_schedule(ctx, sc, &A, &grid);
  plan(ctx, A);
  launch_teams(ctx, A, bat_cqk_team_vjp_kernel<TIn>);
  if (sc.small_per == 4)
    hipLaunchKernelGGL((bat_cqk_vjp_kernel<4, TIn>), grid, dim3(kBlock), 0, ctx->stream, A);
  else
    hipLaunchKernelGGL((bat_cqk_vjp_kernel<8, TIn>), grid, dim3(kBlock), 0, ctx->stream, A);
}

}  // namespace

namespace {
template <typename TIn>
cqk_status run_batched_cqk(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets, const TIn* d,
                           const TIn* a, const TIn* b, const TIn* l, const TIn* u,
                           const double* r, TIn* x, double* lambda_out, int32_t* status_out,
                           const cqk_opts& o, cqk_info* info) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  BatCqkArgs A = cqk_args(ctx, nseg, offsets, d, a, b, l, u, w);
  A.r = r;
  A.x = x;
  A.lam_out = lambda_out;
  A.status_out = status_out;
  A.lambda0_mode = o.lambda0_mode;
  A.lam0_user = o.lambda0_user;
  A.max_iter = o.max_iter;
  A.tol = (o.tol > 0.0) ? o.tol : std::pow(2.220446049250313e-16, 0.75);
  hipStream_t s = ctx->stream;
  if (o.timing) {
    st = ensure_events(ctx, 2);
    if (st != CQK_OK) return st;
    hipEventRecord(ctx->events[0], s);
  }
  launch_cqk_forward<TIn>(ctx, ctx->sched_cqk_fwd, A);
  if (o.timing) hipEventRecord(ctx->events[1], s);
  if (hip_ok(hipGetLastError()) != CQK_OK) return CQK_DEVICE_ERROR;
  // the call's result from the device counters (host copy in hc)
  int32_t* hc = (int32_t*)ctx->host_pinned;
  const bool timing = o.timing != 0;
  auto fill = [ctx, hc, timing](cqk_info* inf) {
    const BatStat t = host_stat(hc, true);
    const int flags = t.flags;
    int status = CQK_OK;
    if (flags & kBadValue) status = CQK_INVALID_ARG;
    else if (flags & kInfeasible) status = CQK_INFEASIBLE;
    else if (flags & kNotConverged) status = CQK_NOT_CONVERGED;
    std::memset(inf, 0, sizeof(*inf));
    inf->status = status;
    inf->iterations = t.over;
    inf->passes = t.surv;
    if (timing) {
      float ms = 0.f;
      hipEventElapsedTime(&ms, ctx->events[0], ctx->events[1]);
      inf->pass_ms = ms;
    }
  };
  int32_t* dc = A.counters;
  ctx->last = [hc, dc, fill](cqk_info* inf) -> cqk_status {
    if (hip_ok(hipMemcpy(hc, dc, CTR_OUTCOME * sizeof(int32_t), hipMemcpyDeviceToHost)) != CQK_OK)
      return CQK_DEVICE_ERROR;
    fill(inf);
    return CQK_OK;
  };
  if (info) std::memset(info, 0, sizeof(*info));
  if (!o.sync) return CQK_OK;
  if (hip_ok(hipMemcpyAsync(hc, A.counters, CTR_OUTCOME * sizeof(int32_t), hipMemcpyDeviceToHost,
                            s)) != CQK_OK)
    return CQK_DEVICE_ERROR;
  if (hip_ok(hipStreamSynchronize(s)) != CQK_OK) return CQK_DEVICE_ERROR;
  if (info) fill(info);
  return CQK_OK;
}

template <typename TIn>
cqk_status run_batched_cqk_backward(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                    const TIn* x, const TIn* g, const TIn* d, const TIn* b,
                                    const TIn* l, const TIn* u, TIn* grad_a, double* grad_r,
                                    const cqk_opts& o) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  BatCqkArgs A = cqk_args(ctx, nseg, offsets, d, nullptr, b, l, u, w);
  A.x = const_cast<TIn*>(x);
  A.g = g;
  A.ga = grad_a;
  A.gr = grad_r;
  launch_cqk_backward<TIn>(ctx, ctx->sched_cqk_bwd, A);
  if (hip_ok(hipGetLastError()) != CQK_OK) return CQK_DEVICE_ERROR;
  ctx->last = ok_info;
  if (o.sync && hip_ok(hipStreamSynchronize(ctx->stream)) != CQK_OK) return CQK_DEVICE_ERROR;
  return CQK_OK;
}
}  // namespace

cqk_status run_batched_cqk_f64(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                               const double* d, const double* a, const double* b,
                               const double* l, const double* u, const double* r, double* x,
                               double* lambda_out, int32_t* status_out, const cqk_opts& o,
                               cqk_info* info) {
  return run_batched_cqk<double>(ctx, nseg, offsets, d, a, b, l, u, r, x, lambda_out,
                                 status_out, o, info);
}

cqk_status run_batched_cqk_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                               const float* d, const float* a, const float* b, const float* l,
                               const float* u, const double* r, float* x, double* lambda_out,
                               int32_t* status_out, const cqk_opts& o, cqk_info* info) {
  return run_batched_cqk<float>(ctx, nseg, offsets, d, a, b, l, u, r, x, lambda_out, status_out,
                                o, info);
}

cqk_status run_batched_cqk_backward_f64(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                        const double* x, const double* g, const double* d,
                                        const double* b, const double* l, const double* u,
                                        double* grad_a, double* grad_r, const cqk_opts& o) {
  return run_batched_cqk_backward<double>(ctx, nseg, offsets, x, g, d, b, l, u, grad_a, grad_r,
                                          o);
}

cqk_status run_batched_cqk_backward_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                        const float* x, const float* g, const float* d,
                                        const float* b, const float* l, const float* u,
                                        float* grad_a, double* grad_r, const cqk_opts& o) {
  return run_batched_cqk_backward<float>(ctx, nseg, offsets, x, g, d, b, l, u, grad_a, grad_r,
                                         o);
}

namespace {
template <typename TIn>
cqk_status tune_batched_cqk(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets, const TIn* d,
                            const TIn* a, const TIn* b, const TIn* l, const TIn* u,
                            const double* r, TIn* x, const TIn* g, TIn* grad_a,
                            int32_t backward, int32_t repeats, cqk_batch_schedule* best,
                            double* best_ms) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  BatCqkArgs A = cqk_args(ctx, nseg, offsets, d, a, b, l, u, w);
  A.r = r;
  A.x = x;
  A.g = g;
  A.ga = grad_a;
  A.lambda0_mode = CQK_LAMBDA0_ZERO;
  A.max_iter = 100;
  A.tol = std::pow(2.220446049250313e-16, 0.75);
  cqk_batch_schedule cand[32];
  const int nc = candidate_schedules(cand, 32);
  int bi = 0;
  double ms = 0.0;
  if (backward)
    st = tune(ctx, cand, nc, repeats,
              [&](const cqk_batch_schedule& sc) { launch_cqk_backward<TIn>(ctx, sc, A); }, &bi,
              &ms);
  else
    st = tune(ctx, cand, nc, repeats,
              [&](const cqk_batch_schedule& sc) { launch_cqk_forward<TIn>(ctx, sc, A); }, &bi,
              &ms);
  if (st != CQK_OK) return st;
  (backward ? ctx->sched_cqk_bwd : ctx->sched_cqk_fwd) = cand[bi];
  if (best) *best = cand[bi];
  if (best_ms) *best_ms = ms;
  return CQK_OK;
}
}  // namespace

cqk_status tune_batched_cqk_f64(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                const double* d, const double* a, const double* b,
                                const double* l, const double* u, const double* r, double* x,
                                const double* g, double* grad_a, int32_t backward,
                                int32_t repeats, cqk_batch_schedule* best, double* best_ms) {
  return tune_batched_cqk<double>(ctx, nseg, offsets, d, a, b, l, u, r, x, g, grad_a, backward,
                                  repeats, best, best_ms);
}

cqk_status tune_batched_cqk_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                const float* d, const float* a, const float* b, const float* l,
                                const float* u, const double* r, float* x, const float* g,
                                float* grad_a, int32_t backward, int32_t repeats,
                                cqk_batch_schedule* best, double* best_ms) {
  return tune_batched_cqk<float>(ctx, nseg, offsets, d, a, b, l, u, r, x, g, grad_a, backward,
                                 repeats, best, best_ms);
}

bool valid_schedule(const cqk_batch_schedule& sc) {
  return (sc.small_per == 4 || sc.small_per == 8) && sc.blocks_per_cu >= 1 &&
         sc.blocks_per_cu <= 8 && (sc.short_first == 0 || sc.short_first == 1) &&
         sc.medium_tiles >= 0 && sc.medium_tiles <= 64;
}


// The info record of the last batched forward call from the host copy of its
// counters.
void bat_fill_info(cqk_ctx* ctx, cqk_info* inf) {
  const int32_t* hc = (const int32_t*)ctx->host_pinned;
  const BatStat t = host_stat(hc, false);
  const int flags = t.flags;
  int status = CQK_OK;
  if (flags & (kBadRadius | kBadValue)) status = CQK_INVALID_ARG;
  else if (flags & kInfeasible) status = CQK_INFEASIBLE;
  std::memset(inf, 0, sizeof(*inf));
  inf->status = status;
  inf->n_after_init = t.surv;
  inf->iterations = 0;
  inf->passes = 1;
  inf->rows_spilled = t.over;
  if (ctx->bat_timing) {
    float ms = 0.f;
    hipEventElapsedTime(&ms, ctx->events[0], ctx->events[1]);
    inf->pass_ms = ms;
  }
}

// Reads the outcome of the last batched forward call from its device
// counters (ctx->bat_counters) once the stream has finished it.
cqk_status bat_read_last(cqk_ctx* ctx, cqk_info* inf) {
  int32_t* hc = (int32_t*)ctx->host_pinned;
  if (hip_ok(hipMemcpy(hc, ctx->bat_counters, CTR_OUTCOME * sizeof(int32_t),
                       hipMemcpyDeviceToHost)) != CQK_OK)
    return CQK_DEVICE_ERROR;
  bat_fill_info(ctx, inf);
  return CQK_OK;
}

// One batched forward call with its planning buffers in w.  Allocates
// nothing unless o.timing asks for events the context does not have yet.
cqk_status run_batched_f32_on(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                              const float* y, const double* r, double r_scalar, float* x,
                              double* lambda_out, int32_t* nfree_out, const BatWs& w,
                              const cqk_opts& o, cqk_info* info) {
  const BatArgs A = forward_args(nseg, offsets, y, r, r_scalar, x, lambda_out, nfree_out, w);
  hipStream_t s = ctx->stream;
  if (o.timing) {
    cqk_status st = ensure_events(ctx, 2);
    if (st != CQK_OK) return st;
    hipEventRecord(ctx->events[0], s);
  }
  launch_forward(ctx, ctx->sched_fwd, A);
  if (o.timing) hipEventRecord(ctx->events[1], s);
  if (hip_ok(hipGetLastError()) != CQK_OK) return CQK_DEVICE_ERROR;
  ctx->bat_counters = A.counters;
  ctx->bat_timing = o.timing != 0;
  // one captured pointer: std::function keeps it without a heap allocation
  ctx->last = [ctx](cqk_info* inf) -> cqk_status { return bat_read_last(ctx, inf); };
  if (info) std::memset(info, 0, sizeof(*info));
  if (!o.sync) return CQK_OK;
  if (hip_ok(hipMemcpyAsync(ctx->host_pinned, A.counters, CTR_OUTCOME * sizeof(int32_t),
                            hipMemcpyDeviceToHost, s)) != CQK_OK)
    return CQK_DEVICE_ERROR;
  if (hip_ok(hipStreamSynchronize(s)) != CQK_OK) return CQK_DEVICE_ERROR;
  if (info) bat_fill_info(ctx, info);
  return CQK_OK;
}

cqk_status run_batched_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets, const float* y,
                           const double* r, double r_scalar, float* x, double* lambda_out,
                           int32_t* nfree_out, const cqk_opts& o, cqk_info* info) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  return run_batched_f32_on(ctx, nseg, offsets, y, r, r_scalar, x, lambda_out, nfree_out, w, o,
                            info);
}

cqk_status noalloc_scratch(int device, void** out) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return CQK_DEVICE_ERROR;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    void* p = nullptr;
    // the caller made `device` current
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return CQK_DEVICE_ERROR;
    }
    addr[device] = p;
  }
  *out = addr[device];
  return CQK_OK;
}

cqk_status run_batched_noalloc_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                   const float* y, const double* r, double r_scalar, float* x,
                                   double* lambda_out, int32_t* nfree_out, const cqk_opts& o,
                                   cqk_info* info) {
  if (nseg > CQK_NOALLOC_MAX_SEG) return CQK_BUFFER_TOO_SMALL;
  if (!ctx->scratch) return CQK_DEVICE_ERROR;
  BatWs w;
  bat_layout(ctx->scratch, nseg, &w);
  cqk_opts o2 = o;
  o2.timing = 0;  // events would be created on first use
  return run_batched_f32_on(ctx, nseg, offsets, y, r, r_scalar, x, lambda_out, nfree_out, w, o2,
                            info);
}

cqk_status run_batched_backward_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                    const float* x, const float* g, float* grad_y,
                                    double* grad_r, const cqk_opts& o) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  launch_backward(ctx, ctx->sched_bwd, backward_args(nseg, offsets, x, g, grad_y, grad_r, w));
  if (hip_ok(hipGetLastError()) != CQK_OK) return CQK_DEVICE_ERROR;
  ctx->last = ok_info;
  if (o.sync && hip_ok(hipStreamSynchronize(ctx->stream)) != CQK_OK) return CQK_DEVICE_ERROR;
  return CQK_OK;
}

cqk_status tune_batched_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets, const float* y,
                            const double* r, double r_scalar, float* x, int32_t repeats,
                            cqk_batch_schedule* best, double* best_ms) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  const BatArgs A = forward_args(nseg, offsets, y, r, r_scalar, x, nullptr, nullptr, w);
  cqk_batch_schedule cand[128];
  const int nc = candidate_schedules_fwd(cand, 128);
  int bi = 0;
  double ms = 0.0;
  st = tune(ctx, cand, nc, repeats,
            [&](const cqk_batch_schedule& sc) { launch_forward(ctx, sc, A); }, &bi, &ms);
  if (st != CQK_OK) return st;
  ctx->sched_fwd = cand[bi];
  if (best) *best = cand[bi];
  if (best_ms) *best_ms = ms;
  return CQK_OK;
}

cqk_status tune_batched_backward_f32(cqk_ctx* ctx, int32_t nseg, const int64_t* offsets,
                                     const float* x, const float* g, float* grad_y,
                                     int32_t repeats, cqk_batch_schedule* best,
                                     double* best_ms) {
  BatWs w;
  cqk_status st = bat_workspace(ctx, nseg, &w);
  if (st != CQK_OK) return st;
  const BatArgs A = backward_args(nseg, offsets, x, g, grad_y, nullptr, w);
  cqk_batch_schedule cand[128];
  const int nc = candidate_schedules_fwd(cand, 128);
  int bi = 0;
  double ms = 0.0;
  st = tune(ctx, cand, nc, repeats,
            [&](const cqk_batch_schedule& sc) { launch_backward(ctx, sc, A); }, &bi, &ms);
  if (st != CQK_OK) return st;
  ctx->sched_bwd = cand[bi];
  if (best) *best = cand[bi];
  if (best_ms) *best_ms = ms;
  return CQK_OK;
}

}  // namespace cqk
