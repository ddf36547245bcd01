// Task advantage normalisation (AgentRL Sec. 3.2) on top of GRPO's group-relative
// advantage (App. B.2), for a global batch of trajectories.
//
// Compiled with -ffp-contract=off: every + - * / and sqrtf below is one correctly
// rounded fp32 operation, so the results are bit-identical to any implementation
// that follows the same summation order (see agrl.h).
#include <math.h>

#include "../../include/agrl.h"
#include "common.hpp"

namespace agrl {
namespace {

constexpr int kCountPerLane = 16;

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// n_tau: a lane walks kCountPerLane consecutive tokens, adding each run of one
// trajectory's action tokens at its end; the last run is left in (cur, cnt).  Integer
// atomics are exact, so the counts do not depend on the order.
struct Run {
  int cur = -1, cnt = 0;
  __device__ __forceinline__ void token(int id, bool m, int32_t n_traj, int32_t* count, int* err) {
    if (id >= n_traj) {
      set_error(err, ERR_TRAJ_ID);
      return;
    }
    if (id < 0 || !m) return;
    if (id != cur) {
      if (cnt) atomicAdd(&count[cur], cnt);
      cur = id;
      cnt = 0;
    }
    ++cnt;
  }
};

// Four values in one 16-byte access at any element's address (global memory takes one that
// is only 4-byte aligned)
typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// Tokens are taken in runs of N whose mask bytes start at a multiple of N in memory: a
// micro-batch's arrays may start anywhere in the batch's.  The first run then begins up to
// N - 1 tokens before the arrays.  Read element by element where the arrays are not aligned,
// sequence weights of 65536 tokens took 46.6 us a call and an advantage call of 512
// trajectories and 32000 tokens 56.2, now 11.6 and 27.6 (aligned 8.4 and 26.2).
template <int N>
__host__ __device__ __forceinline__ int run_shift(const uint8_t* mask) {
  return (int)((uintptr_t)mask & (N - 1));
}

// The ids and mask bytes of a lane's tokens [t0, t0 + 16), with four 16-byte id loads and one
// 16-byte mask load; the tokens of the first and the last run that lie outside the arrays are
// padding.
struct Tokens {
  i32x4 ids[4];
  u32x4 m;
  __device__ __forceinline__ void load(int64_t t0, int64_t T_g, const int32_t* __restrict__ traj_id,
                                       const uint8_t* __restrict__ mask) {
    static_assert(kCountPerLane == 16, "one 16-byte mask load per lane");
    if (t0 >= 0 && t0 + kCountPerLane <= T_g) {
#pragma unroll
      for (int k = 0; k < 4; ++k) ids[k] = *(const i32x4*)(traj_id + t0 + 4 * k);
      m = *(const u32x4*)(mask + t0);
      return;
    }
    m = u32x4{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < kCountPerLane; ++i) {
      const bool in = t0 + i >= 0 && t0 + i < T_g;
      ids[i >> 2][i & 3] = in ? traj_id[t0 + i] : -1;
      m[i >> 2] |= (in && mask[t0 + i] ? 1u : 0u) << (8 * (i & 3));
    }
  }
  // Trajectories are mostly longer than 16 tokens, so a lane nearly always has one of them or
  // two: their action tokens are then counted as bits, about half the instructions of the walk,
  // which is what bounded a workgroup that counts all the tokens: 12.5 -> 8.4 us a call of
  // sequence weights at 65536 tokens, 640 trajectories; 33.1 -> 31.7 us a large advantage call.
  __device__ __forceinline__ Run count(int32_t n_traj, int32_t* count, int* err) const {
    uint32_t changes = 0;                  // bit i: token i's id differs from the one before
#pragma unroll
    for (int i = 1; i < kCountPerLane; ++i)
      changes |= (ids[i >> 2][i & 3] != ids[(i - 1) >> 2][(i - 1) & 3] ? 1u : 0u) << i;
    Run r;
    if (changes & (changes - 1)) {
#pragma unroll
      for (int i = 0; i < kCountPerLane; ++i)
        r.token(ids[i >> 2][i & 3], (m[i >> 2] >> (8 * (i & 3))) & 0xFFu, n_traj, count, err);
      return r;
    }
    uint32_t act = 0;                      // bit 8 j + k: token 4 k + j is an action token
#pragma unroll
    for (int k = 0; k < 4; ++k)
      act |= ((((m[k] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | m[k]) & 0x80808080u) >> (7 - k);
    const int first = ids[0][0], last = ids[3][3];
    if (max(first, last) >= n_traj) set_error(err, ERR_TRAJ_ID);
    uint32_t head = 0;                     // the tokens before the change, if there is one
    if (changes) {
      const int at = __builtin_ctz(changes), k = at >> 2, j = at & 3;
      head = ((0x01010101u << k) - 0x01010101u) | ((0x01010101u & ((1u << (8 * j)) - 1)) << k);
      const int n = __popc(act & head);
      if (n && first >= 0 && first < n_traj) atomicAdd(&count[first], n);
    }
    if (last >= 0 && last < n_traj) {
      r.cur = last;
      r.cnt = __popc(act & ~head);
    }
    return r;
  }
};

// A wave's tokens from t0 (each lane's first) into counters in memory: lanes that end on
// the same trajectory are merged into one atomic.
__device__ __forceinline__ void count_tokens(int64_t t0, int64_t T_g, int32_t n_traj,
                                             const int32_t* traj_id, const uint8_t* mask,
                                             int32_t* count, int* err) {
  Tokens tok;
  tok.load(t0, T_g, traj_id, mask);
  Run r = tok.count(n_traj, count, err);
  const int lane = threadIdx.x & 63;
  for (;;) {
    const uint64_t pend = __ballot(r.cnt > 0);
    if (!pend) break;
    const int leader = __ffsll((unsigned long long)pend) - 1;
    const int lid = __shfl(r.cur, leader);
    int mine = (r.cnt > 0 && r.cur == lid) ? r.cnt : 0;
    for (int o = 32; o >= 1; o >>= 1) mine += __shfl_xor(mine, o);
    if (lane == leader) atomicAdd(&count[lid], mine);
    if (r.cnt > 0 && r.cur == lid) r.cnt = 0;
  }
}

// All T_g tokens by one workgroup of 1024 threads into counters in LDS, two batches of
// loads in flight.
__device__ __forceinline__ void count_in_lds(int64_t T_g, int32_t n_traj, const int32_t* traj_id,
                                             const uint8_t* mask, int32_t* count, int* err) {
  constexpr int B = 2;
  constexpr int64_t step = 1024 * kCountPerLane;
  const int shift = run_shift<kCountPerLane>(mask);
  for (int64_t t0 = (int64_t)threadIdx.x * kCountPerLane - shift; t0 < T_g; t0 += B * step) {
    Tokens tok[B];
#pragma unroll
    for (int b = 0; b < B; ++b) tok[b].load(t0 + b * step, T_g, traj_id, mask);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const Run r = tok[b].count(n_traj, count, err);
      if (r.cnt) atomicAdd(&count[r.cur], r.cnt);
    }
  }
}

// Lowest and highest trajectory index per segment key, one atomic pair per
// distinct key of the wave: the wave's trajectories are consecutive, so the
// lowest lane holding a key has its lowest index and the highest lane its highest.
__device__ __forceinline__ void wave_range(bool valid, int key, int tau, int32_t* range) {
  const int lane = threadIdx.x & 63;
  uint64_t pend = __ballot(valid);
  while (pend) {
    const int k = __shfl(key, __ffsll((unsigned long long)pend) - 1);
    const uint64_t m = __ballot(valid && key == k);
    if (lane == __ffsll((unsigned long long)m) - 1) atomicMin(&range[2 * k], tau);
    if (lane == 63 - __clzll((unsigned long long)m)) atomicMax(&range[2 * k + 1], tau);
    pend &= ~m;
  }
}

// Zero the per-trajectory counts, preset the n_range member ranges to empty (lowest =
// n_traj, highest = -1), one launch.
__global__ void init_kernel(int32_t n_traj, int32_t* act_count, int32_t n_range, int32_t* range) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_traj) act_count[k] = 0;
  if (k < n_range) range[k] = (k & 1) ? -1 : n_traj;
}

// Check a trajectory's task and group ids; with `range` (2 ints per group, then 2 per
// task) also record the lowest and the highest index of each group's and each task's
// members (integer atomics: the result does not depend on the order).
struct IdArgs {
  int32_t n_task, n_group;
  const int32_t* traj_task;
  const int32_t* traj_group;
  int32_t* range;
};
__device__ __forceinline__ void check_ids(const IdArgs& a, int j, int32_t n_traj, int* err) {
  const bool in = j < n_traj;
  const int i = in ? a.traj_task[j] : 0;
  const int g = in && a.traj_group ? a.traj_group[j] : 0;
  const bool ok_task = in && i >= 0 && i < a.n_task;
  const bool ok_group = in && a.traj_group && g >= 0 && g < a.n_group;
  if (in && !ok_task) set_error(err, ERR_TASK_ID);
  if (in && a.traj_group && !ok_group) set_error(err, ERR_GROUP_ID);
  if (a.range) {
    if (a.traj_group) wave_range(ok_group, g, j, a.range);
    wave_range(ok_task, i, j, a.range + 2 * a.n_group);
  }
}

// The token counts, and beside them the id checks, which do not need them: the first
// id_blocks blocks take 256 trajectories each, the others 256 * kCountPerLane tokens.
// One launch less at 2560 trajectories and 9M tokens: 38.6 -> 33.6 us a call (31.7 since).  (Ranges
// preset and recorded by one block: 16.3 us for that launch alone.)
__global__ __launch_bounds__(256) void count_kernel(int64_t T_g, int32_t n_traj,
                                                    const int32_t* __restrict__ traj_id,
                                                    const uint8_t* __restrict__ mask,
                                                    int32_t* act_count, int32_t id_blocks,
                                                    IdArgs ids, int* err) {
  if ((int)blockIdx.x < id_blocks) {
    check_ids(ids, blockIdx.x * 256 + threadIdx.x, n_traj, err);
    return;
  }
  count_tokens(((int64_t)(blockIdx.x - id_blocks) * 256 + threadIdx.x) * kCountPerLane -
                   run_shift<kCountPerLane>(mask),
               T_g, n_traj, traj_id, mask, act_count, err);
}

void launch_count(int64_t T_g, int32_t n_traj, const int32_t* traj_id, const uint8_t* mask,
                  int32_t* act_count, int32_t id_blocks, const IdArgs& ids, int* err,
                  hipStream_t s) {
  const int64_t tokens = T_g > 0 ? T_g + run_shift<kCountPerLane>(mask) : 0;
  const int64_t blocks = id_blocks + cdiv<int64_t>(tokens, 256 * kCountPerLane);
  if (blocks == 0) return;
  hipLaunchKernelGGL(count_kernel, dim3((unsigned)blocks), dim3(256), 0, s, T_g, n_traj, traj_id,
                     mask, act_count, id_blocks, ids, err);
}

// The trajectories a segment's wave visits: [first, last] of its members when
// the ranges were recorded, else all of them.  The wave walks them in steps of
// 64 from first rounded down to a multiple of 64, so that lane l always takes
// the trajectories tau = l mod 64 in ascending order: the summation order, and
// so every bit of the result, is the same either way.
struct Span {
  int first, last;
};
__device__ __forceinline__ Span segment_span(const int32_t* range, int k, int32_t n_traj) {
  if (!range) return Span{0, n_traj - 1};
  return Span{range[2 * k], range[2 * k + 1]};
}

// The fixed combination of a wave's 64 partial sums: acc_l += acc_{l xor o},
// o = 32 .. 1.  All lanes end with the same bits.
__device__ __forceinline__ float butterfly_sum(float acc) {
  for (int o = 32; o >= 1; o >>= 1) acc = acc + __shfl_xor(acc, o);
  return acc;
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// GRPO stage: one wave per group.  Lane l owns trajectories l, l+64, ...
// With drop_uniform, a group whose rewards are all equal is marked dropped by a
// quiet NaN in a_hat (the task stage leaves such trajectories out and gives
// them advantage 0).
__device__ void group_wave(int g, int lane, int32_t n_traj, Span sp,
                           const int32_t* __restrict__ traj_group,
                           const float* __restrict__ reward, int32_t ddof, float eps,
                           int32_t drop_uniform, float* a_hat) {
  if (sp.last < sp.first) return;      // no members
  const int t0 = (sp.first & ~63) + lane, end = sp.last + 1;
  float acc = 0.0f;
  int K = 0;
  for (int base = sp.first & ~63; base < end; base += 64) {
    const int tau = base + lane;
    const bool mem = tau < end && traj_group[tau] == g;
    if (mem) acc = acc + reward[tau];
    K += __popcll(__ballot(mem));
  }
  if (K == 0) return;
  if (drop_uniform) {
    // exact: min and max over the members do not depend on the order
    float lo = INFINITY, hi = -INFINITY;
    for (int tau = t0; tau < end; tau += 64)
      if (traj_group[tau] == g) {
        lo = fminf(lo, reward[tau]);
        hi = fmaxf(hi, reward[tau]);
      }
    for (int o = 32; o >= 1; o >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, o));
      hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if (lo == hi) {
      for (int tau = t0; tau < end; tau += 64)
        if (traj_group[tau] == g) a_hat[tau] = __builtin_nanf("");
      return;
    }
  }
  if (K - ddof <= 0) {
    for (int tau = t0; tau < end; tau += 64)
      if (traj_group[tau] == g) a_hat[tau] = 0.0f;
    return;
  }
  const float mu = butterfly_sum(acc) / (float)K;
  acc = 0.0f;
  for (int tau = t0; tau < end; tau += 64) {
    if (traj_group[tau] == g) {
      const float dv = reward[tau] - mu;
      acc = acc + dv * dv;
    }
  }
  const float var = butterfly_sum(acc) / (float)(K - ddof);
  const float den = sqrtf(var) + eps;
  for (int tau = t0; tau < end; tau += 64)
    if (traj_group[tau] == g) a_hat[tau] = (reward[tau] - mu) / den;
}

__global__ __launch_bounds__(256) void group_kernel(int32_t n_group, int32_t n_traj,
                                                    const int32_t* __restrict__ traj_group,
                                                    const float* __restrict__ reward,
                                                    const int32_t* range, int32_t ddof, float eps,
                                                    int32_t drop_uniform, float* a_hat) {
  const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g < n_group)
    group_wave(g, threadIdx.x & 63, n_traj, segment_span(range, g, n_traj), traj_group, reward,
               ddof, eps, drop_uniform, a_hat);
}

// Task stage: one wave per task; statistics of the token-level set, where
// trajectory tau contributes its advantage with multiplicity n_tau.
// src may alias adv_traj: each lane reads its own trajectories before writing them.
// With drop_uniform, trajectories whose group stage left a NaN mark (dropped
// groups) are not members of their task's set and get advantage 0.
__device__ void task_wave(int i, int lane, int32_t n_traj, Span sp,
                          const int32_t* __restrict__ traj_task,
                          const int32_t* __restrict__ act_count, const float* src, int32_t ddof,
                          float eps, int32_t drop_uniform, int64_t* task_count, float* task_mean,
                          float* task_std, float* adv_traj) {
  auto member = [&](int tau) {
    return traj_task[tau] == i && !(drop_uniform && isnan(src[tau]));
  };
  const int t0 = (sp.first & ~63) + lane, end = sp.last + 1;   // empty when last < first
  float acc = 0.0f;
  int64_t n_lane = 0;
  for (int tau = t0; tau < end; tau += 64) {
    if (member(tau)) {
      const int n = act_count[tau];
      n_lane += n;
      acc = acc + (float)n * src[tau];
    }
  }
  const int64_t N = wave_sum_i64(n_lane);
  if (N == 0) {
    for (int tau = t0; tau < end; tau += 64)
      if (traj_task[tau] == i) adv_traj[tau] = 0.0f;       // dropped ones included
    if (lane == 0) {
      task_count[i] = 0;
      task_mean[i] = 0.0f;
      task_std[i] = 0.0f;
    }
    return;
  }
  const float mu = butterfly_sum(acc) / (float)N;
  acc = 0.0f;
  for (int tau = t0; tau < end; tau += 64) {
    if (member(tau)) {
      const float dv = src[tau] - mu;
      acc = acc + (float)act_count[tau] * (dv * dv);
    }
  }
  const float q = butterfly_sum(acc);
  const float sigma = (N - ddof > 0) ? sqrtf(q / (float)(N - ddof)) : 0.0f;
  const float den = sigma + eps;
  for (int tau = t0; tau < end; tau += 64)
    if (traj_task[tau] == i) adv_traj[tau] = member(tau) ? (src[tau] - mu) / den : 0.0f;
  if (lane == 0) {
    task_count[i] = N;
    task_mean[i] = mu;
    task_std[i] = sigma;
  }
}

__global__ __launch_bounds__(256) void task_kernel(int32_t n_task, int32_t n_group, int32_t n_traj,
                                                   const int32_t* __restrict__ traj_task,
                                                   const int32_t* __restrict__ act_count,
                                                   const float* src, const int32_t* range,
                                                   int32_t ddof, float eps, int32_t drop_uniform,
                                                   int64_t* task_count, float* task_mean,
                                                   float* task_std, float* adv_traj) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i < n_task)
    task_wave(i, threadIdx.x & 63, n_traj, segment_span(range, n_group + i, n_traj),
              traj_task, act_count, src, ddof, eps, drop_uniform, task_count, task_mean,
              task_std, adv_traj);
}

// tok = value[traj_id] on action tokens, 0 elsewhere: run r of four tokens, with one 16-byte id
// load, one 4-byte mask load and one 16-byte store.
__device__ __forceinline__ void spread_tokens(int64_t r, int64_t T, int32_t n_traj,
                                              const int32_t* __restrict__ traj_id,
                                              const uint8_t* __restrict__ mask,
                                              const float* value, float* tok) {
  auto one = [&](int id, bool m) { return (m && id >= 0 && id < n_traj) ? value[id] : 0.0f; };
  const int64_t t = 4 * r - run_shift<4>(mask);
  if (t >= 0 && t + 4 <= T) {
    const i32x4 id = *(const i32x4*)(traj_id + t);
    const uint32_t m = *(const uint32_t*)(mask + t);
    *(f32x4_any*)(tok + t) = f32x4_any{one(id[0], m & 0xFFu), one(id[1], (m >> 8) & 0xFFu),
                                       one(id[2], (m >> 16) & 0xFFu), one(id[3], m >> 24)};
    return;
  }
  for (int64_t u = t < 0 ? 0 : t; u < T && u < t + 4; ++u) tok[u] = one(traj_id[u], mask[u] != 0);
}
// runs that cover T tokens
__host__ __device__ __forceinline__ int64_t spread_runs(int64_t T, const uint8_t* mask) {
  return cdiv<int64_t>(T + run_shift<4>(mask), 4);
}

__global__ void broadcast_kernel(int64_t T_g, int32_t n_traj, const int32_t* __restrict__ traj_id,
                                 const uint8_t* __restrict__ mask,
                                 const float* __restrict__ adv_traj, float* adv_tok) {
  spread_tokens((int64_t)blockIdx.x * blockDim.x + threadIdx.x, T_g, n_traj, traj_id, mask,
                adv_traj, adv_tok);
}

// A whole call in one workgroup, for batches small enough that launches are what they
// cost: the same stages on arrays in LDS.  32 trajectories, 3.8k tokens, 8 groups, 2
// tasks: 8.0 us, against 18.6 us of six kernels and as much between them.
constexpr int kSmallTraj = 1024;          // trajectories
// Two lots of 16 tokens a thread.  One workgroup against several launches, 64 trajectories:
// 10.7 and 19.7 us at 32768 tokens, 15.3 and 19.7 at 65536, 20.3 and 19.7 at 98304; 256
// trajectories: 15.6 and 23.2, 21.4 and 23.1, 26.4 and 23.1.
constexpr int64_t kSmallTokens = 32768;
// The stages: 16 waves take a segment each, in turn, and walk the trajectories in steps of
// 64; a turn costs about 0.2 us and 0.32 us a step (5 and 8 units), an empty segment's too.
// Several launches cost 6 us more than the rest of this kernel, more with many trajectories,
// and merge a wave's 1024 tokens trajectory by trajectory.  One workgroup against several
// launches, groups and tasks 7 : 1 (tokens 32768; 2000): 256 trajectories, 64 segments 17.7
// and 24.6 us (15.7 and 37.0), 128 segments 25.0 and 26.5 (20.8 and 36.9), 256 segments
// 38.2 and 30.9 (33.2 and 36.8); 1024 trajectories, 64 segments 38.3 and 46.6 (35.1 and
// 57.6), 128 segments 55.5 and 46.6 (50.1 and 57.0); 64 trajectories, 128 segments 16.5 and
// 21.6 (11.1 and 22.3), 512 segments 24.2 and 30.3 (19.1 and 30.6); one trajectory and
// 65535 tasks 2441 against 25.
__host__ inline bool stages_are_short(int64_t T, int32_t n_traj, int32_t n_group, int32_t n_task) {
  const int64_t turns = cdiv<int64_t>(n_group, 16) + cdiv<int64_t>(n_task, 16);
  const int64_t merged = T > 0 ? (int64_t)1024 * n_traj / T : 0;   // trajectories in a wave's tokens
  return turns * (5 + 8 * cdiv(n_traj, 64)) <= 155 + n_traj / 2 + 5 * (merged < 64 ? merged : 64);
}
struct SmallArgs {
  int64_t T_g;
  int32_t n_traj, n_task, n_group;
  const int32_t* traj_id;
  const uint8_t* mask;
  const int32_t* traj_task;
  const int32_t* traj_group;
  const float* reward;
  int32_t ddof;
  float eps;
  int32_t drop;
  int32_t* act_count;
  int64_t* task_count;
  float* task_mean;
  float* task_std;
  float* adv_traj;
  float* adv_tok;
  int* err;
};
__global__ __launch_bounds__(1024) void adv_small_kernel(SmallArgs a) {
  __shared__ int32_t s_count[kSmallTraj], s_task[kSmallTraj], s_group[kSmallTraj];
  __shared__ float s_reward[kSmallTraj], s_adv[kSmallTraj];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < a.n_traj) {
    const int i = a.traj_task[tid], g = a.traj_group ? a.traj_group[tid] : 0;
    s_count[tid] = 0;
    s_task[tid] = i;
    s_group[tid] = g;
    const float r = a.reward[tid];
    s_reward[tid] = r;
    s_adv[tid] = a.traj_group ? 0.0f : r;
    if (i < 0 || i >= a.n_task) set_error(a.err, ERR_TASK_ID);
    if (a.traj_group && (g < 0 || g >= a.n_group)) set_error(a.err, ERR_GROUP_ID);
  }
  __syncthreads();
  count_in_lds(a.T_g, a.n_traj, a.traj_id, a.mask, s_count, a.err);
  const Span all{0, a.n_traj - 1};
  if (a.traj_group)
    for (int g = wave; g < a.n_group; g += 16)
      group_wave(g, lane, a.n_traj, all, s_group, s_reward, a.ddof, a.eps, a.drop, s_adv);
  __syncthreads();
  if (tid < a.n_traj) a.act_count[tid] = s_count[tid];
  for (int i = wave; i < a.n_task; i += 16)
    task_wave(i, lane, a.n_traj, all, s_task, s_count, s_adv, a.ddof, a.eps, a.drop, a.task_count,
              a.task_mean, a.task_std, s_adv);
  __syncthreads();
  if (tid < a.n_traj) a.adv_traj[tid] = s_adv[tid];
  if (a.adv_tok) {
#pragma unroll 4
    for (int64_t r = tid; r < spread_runs(a.T_g, a.mask); r += 1024)
      spread_tokens(r, a.T_g, a.n_traj, a.traj_id, a.mask, s_adv, a.adv_tok);
  }
}

int fail(int code, const char* msg) {
  set_last_error(msg);
  return code;
}

// Sequence-level weights: every block counts the non-empty trajectories
// (n_traj is small) and then weighs its tokens.
__global__ __launch_bounds__(256) void seq_weight_kernel(int64_t T, int32_t n_traj,
                                                         const int32_t* __restrict__ traj_id,
                                                         const uint8_t* __restrict__ mask,
                                                         const int32_t* __restrict__ seq_count,
                                                         float* __restrict__ w) {
  __shared__ int part[256 / 64];
  int n = 0;
  for (int j = threadIdx.x; j < n_traj; j += blockDim.x) n += seq_count[j] > 0;
  for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
  __syncthreads();
  const int n_seq = part[0] + part[1] + part[2] + part[3];
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < T;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int id = traj_id[t];
    float v = 0.0f;
    if (id >= 0 && id < n_traj && mask[t])
      v = (float)(1.0 / ((double)n_seq * (double)seq_count[id]));
    w[t] = v;
  }
}

// The same in one launch, counters in LDS: every workgroup counts all the tokens itself
// (kSeqTokens: 4 lots of 16 a thread, from L2) and weighs its share of them.  One launch
// against three, 640 trajectories: 8.5 and 11.7 us a call at 65536 tokens, 10.7 and 11.7 at
// 98304, 12.4 and 11.6 at 131072; with arrays one element off alignment 11.6 and 12.7, 14.0
// and 11.9, 16.0 and 11.7.
constexpr int kSeqTraj = 4096;
constexpr int64_t kSeqTokens = 65536;
constexpr int kSeqShare = 4096;          // tokens a workgroup weighs
__global__ __launch_bounds__(1024) void seq_small_kernel(int64_t T, int32_t n_traj,
                                                         const int32_t* __restrict__ traj_id,
                                                         const uint8_t* __restrict__ mask,
                                                         int32_t* __restrict__ seq_count,
                                                         float* __restrict__ w, int* err) {
  __shared__ int32_t count[kSeqTraj];
  __shared__ int part[16];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int j = tid; j < n_traj; j += 1024) count[j] = 0;
  __syncthreads();
  count_in_lds(T, n_traj, traj_id, mask, count, err);
  __syncthreads();
  int n = 0;
  for (int j = tid; j < n_traj; j += 1024) {
    if (blockIdx.x == 0) seq_count[j] = count[j];
    n += count[j] > 0;
  }
  for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o);
  if (lane == 0) part[tid >> 6] = n;
  __syncthreads();
  int n_seq = 0;
  for (int k = 0; k < 16; ++k) n_seq += part[k];
  // the quotients of the trajectories with action tokens, in place of their counts
  for (int j = tid; j < n_traj; j += 1024)
    if (count[j] > 0)
      count[j] = __float_as_int((float)(1.0 / ((double)n_seq * (double)count[j])));
  __syncthreads();
  static_assert(kSeqShare == 4 * 1024, "four tokens a thread");
  spread_tokens((int64_t)blockIdx.x * (kSeqShare / 4) + tid, T, n_traj, traj_id, mask,
                (const float*)count, w);
}

}  // namespace
}  // namespace agrl

extern "C" int agrl_task_adv_norm(int64_t T_g, int32_t n_traj, int32_t n_task, int32_t n_group,
                                  const int32_t* traj_id, const uint8_t* action_mask,
                                  const int32_t* traj_task, const int32_t* traj_group,
                                  const float* reward, const agrl_options* opt,
                                  int32_t* act_count, int64_t* task_count, float* task_mean,
                                  float* task_std, float* adv_traj, float* adv_tok,
                                  void* stream) {
  using namespace agrl;
  if (T_g < 0 || n_traj < 0 || n_task < 0 || n_group < 0)
    return fail(AGRL_E_SHAPE, "agrl_task_adv_norm: negative size");
  if (T_g > ((int64_t)1 << 40)) return fail(AGRL_E_SHAPE, "agrl_task_adv_norm: T_g too large");
  if (traj_group && n_traj > 0 && n_group == 0)
    return fail(AGRL_E_SHAPE, "agrl_task_adv_norm: traj_group given with n_group == 0");
  if (T_g > 0 && (!traj_id || !action_mask))
    return fail(AGRL_E_NULL, "agrl_task_adv_norm: traj_id/action_mask is NULL");
  if (n_traj > 0 && (!traj_task || !reward || !act_count || !adv_traj))
    return fail(AGRL_E_NULL, "agrl_task_adv_norm: per-trajectory array is NULL");
  if (n_task > 0 && (!task_count || !task_mean || !task_std))
    return fail(AGRL_E_NULL, "agrl_task_adv_norm: per-task output is NULL");
  agrl_options o = {};
  if (opt) o = *opt;
  if (o.std_ddof != 0 && o.std_ddof != 1)
    return fail(AGRL_E_FLAGS, "agrl_task_adv_norm: std_ddof must be 0 or 1");
  if (!(o.std_eps >= 0.0f) || !isfinite(o.std_eps))
    return fail(AGRL_E_FLAGS, "agrl_task_adv_norm: std_eps must be finite and >= 0");
  const float eps = o.std_eps == 0.0f ? 1e-6f : o.std_eps;
  if (o.drop_uniform_groups != 0 && o.drop_uniform_groups != 1)
    return fail(AGRL_E_FLAGS, "agrl_task_adv_norm: drop_uniform_groups must be 0 or 1");
  if (o.drop_uniform_groups && !traj_group && n_traj > 0)
    return fail(AGRL_E_FLAGS, "agrl_task_adv_norm: drop_uniform_groups needs traj_group");

  hipStream_t s = (hipStream_t)stream;
  int* err = device_error_ptr();
  if (!err) return hip_status(hipErrorInvalidSymbol);

  const int32_t n_group_used = traj_group ? n_group : 0;
  const int32_t ddof = (int32_t)o.std_ddof;
  const int32_t drop = traj_group ? o.drop_uniform_groups : 0;
  if (T_g <= kSmallTokens && n_traj <= kSmallTraj &&
      stages_are_short(T_g, n_traj, n_group_used, n_task)) {
    const SmallArgs a = {T_g, n_traj, n_task, n_group_used, traj_id, action_mask, traj_task,
                         traj_group, reward, ddof, eps, drop, act_count, task_count, task_mean,
                         task_std, adv_traj, adv_tok, err};
    hipLaunchKernelGGL(adv_small_kernel, dim3(1), dim3(1024), 0, s, a);
    return hip_status(hipGetLastError());
  }

  // member ranges (optional scratch): groups first, then tasks
  int32_t* range = n_traj > 0 ? o.adv_ranges : nullptr;
  const int32_t n_range = range ? 2 * (n_group_used + n_task) : 0;
  const int32_t n_init = n_traj > n_range ? n_traj : n_range;
  if (n_init > 0)
    hipLaunchKernelGGL(init_kernel, dim3(cdiv(n_init, 256)), dim3(256), 0, s, n_traj, act_count,
                       n_range, range);
  launch_count(T_g, n_traj, traj_id, action_mask, act_count, cdiv(n_traj, 256),
               IdArgs{n_task, n_group_used, traj_task, traj_group, range}, err, s);
  if (n_group_used > 0)
    hipLaunchKernelGGL(group_kernel, dim3(cdiv(n_group, 4)), dim3(256), 0, s, n_group, n_traj,
                       traj_group, reward, (const int32_t*)range, ddof, eps, drop, adv_traj);
  if (n_task > 0)
    hipLaunchKernelGGL(task_kernel, dim3(cdiv(n_task, 4)), dim3(256), 0, s, n_task, n_group_used,
                       n_traj, traj_task, act_count,
                       traj_group ? (const float*)adv_traj : reward, (const int32_t*)range, ddof,
                       eps, drop, task_count, task_mean, task_std, adv_traj);
  if (adv_tok && T_g > 0) {
    const dim3 grid((unsigned)cdiv<int64_t>(spread_runs(T_g, action_mask), 256));
    hipLaunchKernelGGL(broadcast_kernel, grid, dim3(256), 0, s, T_g, n_traj, traj_id, action_mask,
                       (const float*)adv_traj, adv_tok);
  }
  return hip_status(hipGetLastError());
}

extern "C" int agrl_sequence_mean_weights(int64_t T, int32_t n_traj, const int32_t* traj_id,
                                          const uint8_t* action_mask, int32_t* seq_count,
                                          float* token_weight, void* stream) {
  using namespace agrl;
  if (T < 0 || n_traj < 0) return fail(AGRL_E_SHAPE, "agrl_sequence_mean_weights: negative size");
  if (T > ((int64_t)1 << 40))
    return fail(AGRL_E_SHAPE, "agrl_sequence_mean_weights: T too large");
  if (T > 0 && (!traj_id || !action_mask || !token_weight))
    return fail(AGRL_E_NULL, "agrl_sequence_mean_weights: traj_id/action_mask/token_weight is NULL");
  if (n_traj > 0 && !seq_count)
    return fail(AGRL_E_NULL, "agrl_sequence_mean_weights: seq_count is NULL");
  hipStream_t s = (hipStream_t)stream;
  int* err = device_error_ptr();
  if (!err) return hip_status(hipErrorInvalidSymbol);
  if (T <= kSeqTokens && n_traj <= kSeqTraj) {
    const dim3 grid((unsigned)(T > 0 ? cdiv<int64_t>(spread_runs(T, action_mask), kSeqShare / 4) : 1));
    hipLaunchKernelGGL(seq_small_kernel, grid, dim3(1024), 0, s, T, n_traj, traj_id, action_mask,
                       seq_count, token_weight, err);
    return hip_status(hipGetLastError());
  }
  if (n_traj > 0)
    hipLaunchKernelGGL(fill_i32_kernel, dim3(cdiv(n_traj, 256)), dim3(256), 0, s, seq_count,
                       (int64_t)n_traj, 0);
  if (T > 0) {
    launch_count(T, n_traj, traj_id, action_mask, seq_count, 0, IdArgs{}, err, s);
    const int64_t blocks = cdiv<int64_t>(T, 256);
    hipLaunchKernelGGL(seq_weight_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)),
                       dim3(256), 0, s, T, n_traj, traj_id, action_mask,
                       (const int32_t*)seq_count, token_weight);
  }
  return hip_status(hipGetLastError());
}
