// Fused LM-head + token log-probability + clipped policy-gradient loss, forward
// and backward, over a packed micro-batch (AgentRL App. B.1 token-level
// factorisation; App. B.2 PPO/GRPO clipped surrogate; App. A DAPO decoupled
// clip bounds and token-level normalisation).
//
// Forward:  compact the action tokens -> logits H_act W^T by 256 x 256 tiles on
//           the matrix cores with a per-tile max / sum-exp epilogue (logits are
//           never written) -> merge the vocabulary tiles into lse -> logp,
//           ratio, clipped surrogate, fixed-order loss sum.
// Backward: recompute the logit tiles, form G = dL/dz in bf16 (one stage-tiled
//           layout, which dW reads transposed), then dW = G^T H and dH = G W on
//           the matrix cores; the vocabulary is processed in chunks that bound
//           the G buffer.
#include <math.h>

#include "../../include/agrl.h"
#include "common.hpp"
#include "gemm.hpp"
#include "gemm_f32.hpp"

namespace agrl {
namespace {

constexpr int kScanTile = 4096;          // tokens per block of the compaction scan
constexpr int kScanThreads = 256;
constexpr int kScanPer = kScanTile / kScanThreads;   // 16 tokens per thread
constexpr int kRowPad = 256;             // compacted rows are padded to the GEMM tile
constexpr int kMergeRows = 64;         // action tokens per merge block
constexpr int kMergeWaves = 16;        // waves per merge block
constexpr int kCompactRows = 256;      // tokens per compaction block
// words of the control block: action tokens the launches work on (0 when there are more
// than max_act), that fault's flag, action tokens counted, merge blocks finished; from
// byte 64 two tile queues of 16 words, which the matrix-core launches use in turn
enum : int { CTRL_N = 0, CTRL_OVER = 1, CTRL_COUNT = 2, CTRL_MERGED = 3, CTRL_QUEUE = 16 };

__host__ __device__ inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

// ------------------------------------------------------------------ compaction
__global__ __launch_bounds__(kScanThreads) void scan_count_kernel(int64_t T,
                                                                  const uint8_t* __restrict__ mask,
                                                                  int32_t* blk_cnt) {
  __shared__ int wsum[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanPer;
  int c = 0;
  for (int i = 0; i < kScanPer; ++i) {
    const int64_t t = base + i;
    if (t < T) c += mask[t] != 0;
  }
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) s += wsum[w];
    blk_cnt[blockIdx.x] = s;
  }
}

__device__ __forceinline__ void set_ctrl(int32_t* ctrl, int total, int64_t max_act, int* err) {
  const bool over = (int64_t)total > max_act;
  if (over) set_error(err, ERR_MAX_ACT);
  ctrl[CTRL_N] = over ? 0 : total;
  ctrl[CTRL_OVER] = over;      // the loss becomes NaN
  ctrl[CTRL_COUNT] = total;
  ctrl[CTRL_MERGED] = 0;
  for (int i = 0; i < 32; ++i) ctrl[CTRL_QUEUE + i] = 0;
}

// Single block: exclusive offsets of the scan blocks and the control words.
__global__ __launch_bounds__(1024) void scan_offsets_kernel(int32_t nblk,
                                                            const int32_t* __restrict__ blk_cnt,
                                                            int32_t* blk_off, int32_t* ctrl,
                                                            int64_t max_act, int* err) {
  __shared__ int wsum[16];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int base = 0; base < nblk; base += 1024) {
    const int i = base + threadIdx.x;
    const int v = i < nblk ? blk_cnt[i] : 0;
    int incl = v;   // inclusive prefix within the wave
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = carry;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    if (i < nblk) blk_off[i] = before + incl - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry = before + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) set_ctrl(ctrl, carry, max_act, err);
}

// The last rows of W padded with zero rows to kTailRows, for a K extent over W's rows.
constexpr int kTailRows = 2 * bf16k::SK;
struct TailCopy {
  const uint8_t* src;      // nullable
  int64_t rows;            // rows of src
  uint8_t* dst;
};

struct CompactArgs {
  int64_t T;
  int32_t V, d;
  const uint8_t* mask;
  const int32_t* token_id;
  const float* adv_tok;
  const float* old_logp;
  const float* lse_in;      // backward only
  const float* logp_in;     // backward only
  const int32_t* blk_off;   // nullable: action tokens before each scan tile, ctrl then set
  int32_t* ctrl;
  int64_t max_act;
  int32_t* idx;
  int32_t* y_act;
  float* adv_act;
  float* old_act;
  float* lse_act;           // backward only
  float* gs_act;            // backward only: dL/dlogp / temperature
  float* logp_out;          // forward only: zeroed on masked tokens
  float* lse_out;
  const float* ref_logp;    // nullable: reference log-probs of the KL penalty
  const float* token_weight;  // nullable: per-token loss weights
  float* ref_act;           // forward only: compacted ref_logp / weights
  float* w_act;
  float kl_beta;
  int32_t kl_est;
  float eps_lo, eps_hi;
  float grad_loss;
  int64_t n_norm;
  float inv_temp;
  int* err;
  const uint8_t* H;
  uint8_t* H_act;
  int64_t row_bytes;        // of H
  float* dH;                // backward only: masked rows zeroed
  TailCopy tail;
};

// one wave: dst[0, bytes) = src (nullptr: zeros), 16 bytes a lane
__device__ __forceinline__ void copy_row(u32x4* dst, const u32x4* src, int64_t chunks, int lane) {
  for (int64_t c = lane; c < chunks; c += 4 * 64) {
    u32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c + 64 * k < chunks) v[k] = src ? src[c + 64 * k] : u32x4{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c + 64 * k < chunks) dst[c + 64 * k] = v[k];
  }
}

// nonzero bytes of a word
__device__ __forceinline__ int nonzero_bytes(uint32_t x) {
  return __popc((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u);
}

// Everything the products need of the action tokens, in one launch: their positions,
// their scalars and H rows compacted (zero rows up to the next multiple of 256), and what
// masked tokens get (logp = lse = 0; dH row +0).  Block (b, r) covers the tokens
// [256 b, 256 b + 256); the blocks of one b share its rows out, the first writes the
// scalars.  Every block counts the action tokens before its own, and all of them, from
// the mask itself: for a mask of up to 64 KiB (kOneLaunchTokens) that is a few loads of
// 16 bytes in flight per thread, cheaper than the two launches (5 us each) that it
// replaces; beyond, scan_count / scan_offsets come first and blk_off is given.  Against
// the scan, scatter, gather and zero kernels it replaces (forward + backward): 79 and 22 us
// at T = 2304, d = 3584, 170 and 128 at T = 32768, 370 and 378 at T = 65536, d = 5120, where
// all that counts is the 1.8 GB of rows.
__global__ __launch_bounds__(kCompactRows) void compact_kernel(CompactArgs a) {
  __shared__ int wsum[kCompactRows / 64][3];
  __shared__ int16_t row_of[kCompactRows];     // action tokens from 0 up, masked from 255 down
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kCompactRows, t = base + tid;
  const bool first = blockIdx.y == 0;
  const bool in = t < a.T, m = in && a.mask[t] != 0;
  int before = 0, total = 0;
  const int64_t from = a.blk_off ? base / kScanTile * kScanTile : 0;
  const int64_t to = a.blk_off ? base : a.T;
  // 16-byte words of the mask between the bytes before its first and after its last whole
  // word (a micro-batch's mask may start anywhere in the batch's)
  const int64_t head = min(to, from + (int64_t)((16 - ((uintptr_t)a.mask & 15)) & 15));
  const int64_t whole = head + (to - head) / 16 * 16;
#pragma unroll 4
  for (int64_t c = head + 16 * tid; c < whole; c += 16 * kCompactRows) {
    const u32x4 v = *(const u32x4*)(a.mask + c);
    const int n = nonzero_bytes(v[0]) + nonzero_bytes(v[1]) + nonzero_bytes(v[2]) +
                  nonzero_bytes(v[3]);
    total += n;
    if (c + 16 <= base) {
      before += n;
    } else if (c < base) {                     // base lies inside the word
      const int in_base = (int)(base - c);
#pragma unroll
      for (int e = 0; e < 16; ++e)
        before += e < in_base && ((v[e >> 2] >> (8 * (e & 3))) & 0xFFu) != 0;
    }
  }
  const int odd = (int)(head - from);          // bytes before the words; fewer than 16 after
  if (tid < odd + (int)(to - whole)) {
    const int64_t c = tid < odd ? from + tid : whole + tid - odd;
    const int n = a.mask[c] != 0;
    total += n;
    before += c < base ? n : 0;
  }
  for (int o = 32; o >= 1; o >>= 1) {
    before += __shfl_xor(before, o);
    total += __shfl_xor(total, o);
  }
  const uint64_t act = __ballot(m);
  const int below = __popcll(act & (((uint64_t)1 << lane) - 1));
  if (lane == 0) {
    wsum[wave][0] = before;
    wsum[wave][1] = total;
    wsum[wave][2] = __popcll(act);
  }
  __syncthreads();
  before = total = 0;
  int rank = below, mine = 0;                  // action tokens of the block
  for (int w = 0; w < kCompactRows / 64; ++w) {
    before += wsum[w][0];
    total += wsum[w][1];
    rank += w < wave ? wsum[w][2] : 0;
    mine += wsum[w][2];
  }
  if (a.blk_off) {
    before += a.blk_off[base / kScanTile];
    total = a.ctrl[CTRL_COUNT];
  } else if (first && blockIdx.x == 0 && tid == 0) {
    set_ctrl(a.ctrl, total, a.max_act, a.err);
  }
  const bool ok = total <= a.max_act;
  if (m)
    row_of[rank] = (int16_t)tid;
  else
    row_of[kCompactRows - 1 - (tid - rank)] = (int16_t)tid;
  __syncthreads();

  if (first && in) {
    if (!m) {
      if (a.logp_out) {
        a.logp_out[t] = 0.0f;
        a.lse_out[t] = 0.0f;
      }
    } else {
      const int y_in = a.token_id[t];
      // an id outside the vocabulary poisons the call: the token is kept with
      // id -1 (it matches no logit), its logp / lse and the loss become NaN in the
      // merge, its logit-gradient row NaN in the backward
      const bool bad = y_in < 0 || y_in >= a.V;
      if (bad) set_error(a.err, ERR_TOKEN_ID);
      if (ok) {
        const int pos = before + rank;
        a.idx[pos] = (int32_t)t;
        a.y_act[pos] = bad ? -1 : y_in;
        // the forward-only log-prob pass has neither (its merge then forms a zero surrogate)
        const float adv = a.adv_tok ? a.adv_tok[t] : 0.0f;
        const float old = a.old_logp ? a.old_logp[t] : 0.0f;
        a.adv_act[pos] = adv;
        a.old_act[pos] = old;
        if (a.gs_act) {
          // dL/dlogp of -w (min(rho A, clip(rho) A) - beta KL), w = 1/N or the
          // token's weight: the unclipped branch's derivative, or 0 where the
          // clipped branch is the active minimum, plus w beta dKL/dlogp.
          const float lp = a.logp_in[t];
          const float rho = expf(lp - old);
          const bool cut = (adv > 0.0f && rho > 1.0f + a.eps_hi) || (adv < 0.0f && rho < 1.0f - a.eps_lo);
          const float N = a.n_norm > 0 ? (float)a.n_norm : (float)total;
          const float scale = a.token_weight ? a.grad_loss * a.token_weight[t] : a.grad_loss / N;
          float g = cut ? 0.0f : -scale * adv * rho;
          if (a.kl_beta != 0.0f) {
            // k3: dKL/dl = 1 - exp(r - l) = -expm1(r - l); k1: 1
            const float dkl = a.kl_est == 1 ? 1.0f : -expm1f(a.ref_logp[t] - lp);
            g += scale * a.kl_beta * dkl;
          }
          a.lse_act[pos] = a.lse_in[t];
          a.gs_act[pos] = bad ? NAN : g * a.inv_temp;
        } else {
          a.ref_act[pos] = a.ref_logp ? a.ref_logp[t] : 0.0f;
          a.w_act[pos] = a.token_weight ? a.token_weight[t] : 0.0f;
        }
      }
    }
  }

  // rows, one wave each
  const int R = gridDim.y * (kCompactRows / 64), r = blockIdx.y * (kCompactRows / 64) + wave;
  const int64_t chunks = a.row_bytes / 16;
  if (ok)
    for (int i = r; i < mine; i += R)
      copy_row((u32x4*)(a.H_act + (before + i) * a.row_bytes),
               (const u32x4*)(a.H + (base + row_of[i]) * a.row_bytes), chunks, lane);
  if (a.dH) {
    const int masked = (int)min((int64_t)kCompactRows, a.T - base) - mine;
    // (the threads past T come last in the masked list)
    for (int i = r; i < masked; i += R)
      copy_row((u32x4*)(a.dH + (base + row_of[kCompactRows - 1 - i]) * a.d), nullptr, a.d / 4,
               lane);
  }
  // zero rows after the last action token, and the tail copy
  const int64_t waves = (int64_t)gridDim.x * R, w = (int64_t)blockIdx.x * R + r;
  const int n_act = ok ? total : 0;
  const int64_t pad = round_up(n_act, kRowPad) - n_act;
  for (int64_t i = w; i < pad; i += waves)
    copy_row((u32x4*)(a.H_act + (n_act + i) * a.row_bytes), nullptr, chunks, lane);
  if (a.tail.src)
    for (int64_t i = w; i < kTailRows; i += waves)
      copy_row((u32x4*)(a.tail.dst + i * a.row_bytes),
               i < a.tail.rows ? (const u32x4*)(a.tail.src + i * a.row_bytes) : nullptr, chunks,
               lane);
}

// dst = src^T, stage-tiled (tiled_index, K = r padded to ld_dst); rows r in
// [n_rows, n_rows_pad) are written as 0.  n_rows comes from ctrl[0] (rounded up to
// 256 for the padded extent) when ctrl is given.  bf16 as raw bits, 16-byte global
// accesses: each 64 x 64 tile is read as 8-element row chunks, written to LDS
// transposed (66-element rows: the 16-bit stores of a wave hit distinct banks), and
// read back as 8-element chunks of the output rows; d (the source row length) is a
// multiple of 64.
__global__ __launch_bounds__(256) void transpose16_kernel(const uint16_t* __restrict__ src,
                                                          int64_t ld_src, uint16_t* dst,
                                                          int64_t ld_dst, int64_t n_rows,
                                                          int64_t n_rows_pad, int64_t n_cols,
                                                          const int32_t* ctrl) {
  constexpr int P = 66;
  __shared__ uint16_t tile_t[64 * P];
  if (ctrl) {
    n_rows = ctrl[0];
    n_rows_pad = round_up(n_rows, kRowPad);
  }
  const int64_t r0 = (int64_t)blockIdx.x * 64, c0 = (int64_t)blockIdx.y * 64;
  if (r0 >= n_rows_pad) return;
  for (int k = 0; k < 2; ++k) {
    const int id = threadIdx.x + 256 * k;
    const int rr = id >> 3, c8 = id & 7;
    const int64_t r = r0 + rr;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (r < n_rows) v = *(const u32x4*)(src + r * ld_src + c0 + 8 * c8);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile_t[(8 * c8 + 2 * e) * P + rr] = (uint16_t)v[e];
      tile_t[(8 * c8 + 2 * e + 1) * P + rr] = (uint16_t)(v[e] >> 16);
    }
  }
  __syncthreads();
  for (int k = 0; k < 2; ++k) {
    const int id = threadIdx.x + 256 * k;
    const int c = id >> 3, r8 = id & 7;
    const uint32_t* t32 = (const uint32_t*)(tile_t + c * P + 8 * r8);   // 4-byte aligned
    const u32x4 v = {t32[0], t32[1], t32[2], t32[3]};
    const int64_t oc = c0 + c, orr = r0 + 8 * r8;
    if (oc < n_cols && orr < n_rows_pad)
      *(u32x4*)(dst + tiled_index(oc, orr, ld_dst)) = v;
  }
}

// ------------------------------------------------------------------ forward epilogue
struct MergeArgs {
  int32_t* ctrl;
  int32_t tiles_v;
  const f32x2* part;
  int64_t ld_part;
  const float* zy;
  const int32_t* y_act;    // -1 marks an action token whose id was out of range
  const float* old_act;
  const float* adv_act;
  const float* ref_act;
  const float* w_act;
  const int32_t* idx;
  float eps_lo, eps_hi;
  float kl_beta;
  int32_t kl_est;
  int32_t weighted;        // loss partials are w_n f_n (else f_n, divided by N at the end)
  int64_t n_norm;
  float* logp_out;
  float* lse_out;
  double* blk_sum;
  unsigned long long* blk_clip;     // [2 * blocks]
  float* loss;             // nullptr: log-probs only
  int64_t* n_clip;
};

// (max, sum of exp) joined by another; an empty sum carries no weight whatever its max
__device__ __forceinline__ float mass(float sum, float at, float to) {
  return sum == 0.0f ? 0.0f : sum * expf(at - to);
}

// 64 action tokens per block.  Each of the 16 waves folds a sixteenth of the
// vocabulary-tile partials of its lane's token, eight loads in flight (what bounds the
// kernel is their latency: at V = 152064, with 4 waves and one load at a time, 74 us at 150
// tokens and 86 at 22793; now 14 and 41); wave 0
// combines them, then forms logp, rho and the clipped surrogate and writes the block's
// fixed-order partial sums.  The block that finishes last adds those in block order; blocks
// past the last action token leave at once (a bound of 281575 tokens launches 4400: counting
// themselves finished took them 106 us, 7 now).
__global__ __launch_bounds__(64 * kMergeWaves) void merge_loss_kernel(MergeArgs a) {
  constexpr int U = 8;
  __shared__ f32x2 wpart[kMergeWaves][kMergeRows];
  const int n_act = a.ctrl[CTRL_N];
  const int blocks = max(1, cdiv(n_act, kMergeRows));
  if ((int)blockIdx.x >= blocks) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = blockIdx.x * kMergeRows + lane;
  float m = -INFINITY, s = 0.0f;
  if (n < n_act) {
    for (int t = wave; t < a.tiles_v; t += U * kMergeWaves) {
      f32x2 p[U];
      float mn = m;
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int tk = t + k * kMergeWaves;
        p[k] = tk < a.tiles_v ? a.part[(int64_t)tk * a.ld_part + n] : f32x2{-INFINITY, 0.0f};
      }
#pragma unroll
      for (int k = 0; k < U; ++k) mn = fmaxf(mn, p[k].x);
      s = mass(s, m, mn);
#pragma unroll
      for (int k = 0; k < U; ++k) s += mass(p[k].y, p[k].x, mn);
      m = mn;
    }
  }
  wpart[wave][lane] = f32x2{m, s};
  __syncthreads();
  if (wave != 0) return;
  double sv = 0.0;
  long long hi = 0, lo = 0;
  if (n < n_act) {
    float mm = -INFINITY;
    for (int w = 0; w < kMergeWaves; ++w) mm = fmaxf(mm, wpart[w][lane].x);
    float sum = 0.0f;
    for (int w = 0; w < kMergeWaves; ++w) sum += mass(wpart[w][lane].y, wpart[w][lane].x, mm);
    const bool bad = a.y_act[n] < 0;
    const float lse = bad ? NAN : mm + logf(sum);
    const float logp = bad ? NAN : a.zy[n] - lse;
    const float A = a.adv_act[n];
    const float rho = expf(logp - a.old_act[n]);
    const float rc = fminf(fmaxf(rho, 1.0f - a.eps_lo), 1.0f + a.eps_hi);
    float f = fminf(rho * A, rc * A);
    if (a.kl_beta != 0.0f) {
      // k3: exp(u) - u - 1 = expm1(u) - u with u = r - l (no cancellation near u = 0)
      const float u = a.ref_act[n] - logp;
      f -= a.kl_beta * (a.kl_est == 1 ? -u : expm1f(u) - u);
    }
    sv = a.weighted ? (double)a.w_act[n] * (double)f : (double)f;
    if (isnan(rho)) sv = NAN;      // (the clamps above take the bound for a NaN; bad ids too)
    hi = (A > 0.0f && rho > 1.0f + a.eps_hi);
    lo = (A < 0.0f && rho < 1.0f - a.eps_lo);
    const int t = a.idx[n];
    a.logp_out[t] = logp;
    a.lse_out[t] = lse;
  }
  if (!a.loss) return;
  for (int o = 32; o >= 1; o >>= 1) {
    sv += __shfl_xor(sv, o);
    hi += __shfl_xor(hi, o);
    lo += __shfl_xor(lo, o);
  }
  // blocks run on XCDs whose L2 caches are not coherent: sums are written and read at
  // device scope, the counter orders them
  unsigned long long* sums = (unsigned long long*)a.blk_sum;
  int done = 0;
  if (lane == 0) {
    const int b = blockIdx.x;
    __hip_atomic_store(sums + b, __builtin_bit_cast(unsigned long long, sv), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.blk_clip + 2 * b, (unsigned long long)hi, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.blk_clip + 2 * b + 1, (unsigned long long)lo, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    done = __hip_atomic_fetch_add(a.ctrl + CTRL_MERGED, 1, __ATOMIC_ACQ_REL,
                                  __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__shfl(done, 0) != blocks - 1) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  sv = 0.0;
  hi = lo = 0;
  for (int b = lane; b < blocks; b += 64) {
    sv += __builtin_bit_cast(double, __hip_atomic_load(sums + b, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT));
    hi += (long long)__hip_atomic_load(a.blk_clip + 2 * b, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
    lo += (long long)__hip_atomic_load(a.blk_clip + 2 * b + 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int o = 32; o >= 1; o >>= 1) {
    sv += __shfl_xor(sv, o);
    hi += __shfl_xor(hi, o);
    lo += __shfl_xor(lo, o);
  }
  if (lane == 0) {
    const double N = a.n_norm > 0 ? (double)a.n_norm : (double)n_act;
    const float L = a.weighted ? (float)(-sv) : (N > 0 ? (float)(-sv / N) : 0.0f);
    *a.loss = a.ctrl[CTRL_OVER] ? NAN : L;
    if (a.n_clip) {
      a.n_clip[0] = hi;
      a.n_clip[1] = lo;
    }
  }
}

__global__ void zero_loss_kernel(float* loss, int64_t* n_clip) {
  *loss = 0.0f;
  if (n_clip) {
    n_clip[0] = 0;
    n_clip[1] = 0;
  }
}

// dH[idx[n]][c] (+)= the parts of (c, n) in ascending order: parts [part][d][ld], turned
// through LDS by 64 x 64 tiles (dh_split says how many there are, as in the launch).
__global__ __launch_bounds__(256) void dh_reduce_kernel(const float* __restrict__ parts,
                                                        int64_t ld, const int32_t* ctrl,
                                                        const int32_t* idx, int32_t nv, int32_t d,
                                                        int32_t cus, int32_t split_max,
                                                        int32_t add, float* dH) {
  __shared__ float tile[64][65];
  const int n_act = ctrl[0];
  const int n0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  if (n0 >= n_act) return;
  const int n_parts = dh_split(n_act, nv, d, cus, split_max);
  const int q = threadIdx.x & 15, r = threadIdx.x >> 4;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float* p = parts + (int64_t)(c0 + r + 16 * k) * ld + n0 + 4 * q;
    f32x4 v = *(const f32x4*)p;
    for (int i = 1; i < n_parts; ++i) v += *(const f32x4*)(p + i * (int64_t)d * ld);
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[r + 16 * k][4 * q + e] = v[e];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int n = r + 16 * k;
    if (n0 + n >= n_act) continue;
    f32x4* out = (f32x4*)(dH + (int64_t)idx[n0 + n] * d + c0 + 4 * q);
    f32x4 v = {tile[4 * q][n], tile[4 * q + 1][n], tile[4 * q + 2][n], tile[4 * q + 3][n]};
    if (add) v += *out;
    *out = v;
  }
}

__global__ __launch_bounds__(256) void zero_f32_kernel(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0f;
}

// ------------------------------------------------------------------ host side
int fail(int code, const char* msg) {
  set_last_error(msg);
  return code;
}

struct Layout {
  int64_t T, A_pad, V_pad, Vc;
  int32_t d, V, esize, nblk, tiles_v, merge_blocks;
  size_t ctrl, blk_cnt, blk_off, idx, y_act, adv_act, old_act, ref_act, w_act, lse_act, gs_act,
      zy, blk_sum,
      blk_clip, H_act, part, Ht, Wt, G, ph, pw, fwd_total, total;
  int32_t ph_max, pw_max;      // parts the gradient products' partial buffers hold
  bool w_rows;                 // bf16: dH reads W as it lies (no W^T; its place holds W's
  size_t tail;                 // padded tail rows and dH's parts)
};

constexpr int64_t kDefaultChunkBytes = (int64_t)4 << 30;

// Up to a bound of this many (padded) action tokens dH reads W as it lies, transposing in the
// LDS read, instead of a W^T built first.  (The bound, not the tokens there are: it sizes the
// parts' buffers, in W^T's place, which must hold one part: about V_pad >= 2 A_pad.)  The transpose costs a pass over W whatever the
// tokens, the transposing reads a share of dH's time.  Backward products and transpose,
// W^T against W (V = 152064): 7.33 against 6.53 ms at d = 5120 and 2871 tokens, 15.70
// against 15.57 ms at d = 3584 and 10515, 45.0 against 45.8 ms at d = 5120 and 22793.
constexpr int64_t kWRowsMax = 8192;

bool make_layout(int64_t T, int64_t max_act, int32_t d, int32_t V, int32_t dtype,
                 const agrl_options& o, Layout* L) {
  if (T < 0 || d <= 0 || V <= 0 || (dtype != AGRL_BF16 && dtype != AGRL_F32)) return false;
  if (max_act <= 0 || max_act > T) max_act = T;
  L->T = T;
  L->d = d;
  L->V = V;
  L->esize = dtype == AGRL_BF16 ? 2 : 4;
  L->A_pad = round_up(max_act > 0 ? max_act : 1, kRowPad);
  L->V_pad = round_up(V, kRowPad);
  L->nblk = (int32_t)((T + kScanTile - 1) / kScanTile);
  if (L->nblk < 1) L->nblk = 1;
  L->tiles_v = (int32_t)(L->V_pad / GBN);
  L->merge_blocks = (int32_t)(L->A_pad / kMergeRows);
  // vocabulary chunk of the backward: the widest multiple of 256 whose logit
  // gradient buffers (bf16: G; fp32: twice G, the second half serving the gradient
  // products' parts) fit the budget, then evened out over the chunks this needs
  const int64_t budget = o.g_chunk_bytes > 0 ? o.g_chunk_bytes : kDefaultChunkBytes;
  const int64_t g_copies = dtype == AGRL_BF16 ? 1 : 2;
  int64_t vc_max = budget / (g_copies * L->A_pad * L->esize) / kRowPad * kRowPad;
  if (vc_max < kRowPad) vc_max = kRowPad;
  const int64_t n_chunks = (L->V_pad + vc_max - 1) / vc_max;
  L->Vc = round_up((V + n_chunks - 1) / n_chunks, kRowPad);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t at = off;
    off += (bytes + 255) / 256 * 256;
    return at;
  };
  const size_t A = (size_t)L->A_pad;
  L->ctrl = take(256);
  L->blk_cnt = take(sizeof(int32_t) * L->nblk);
  L->blk_off = take(sizeof(int32_t) * L->nblk);
  L->idx = take(4 * A);
  L->y_act = take(4 * A);
  L->adv_act = take(4 * A);
  L->old_act = take(4 * A);
  L->ref_act = take(4 * A);
  L->w_act = take(4 * A);
  L->lse_act = take(4 * A);
  L->gs_act = take(4 * A);
  L->zy = take(4 * A);
  L->blk_sum = take(sizeof(double) * L->merge_blocks);
  L->blk_clip = take(2 * sizeof(long long) * L->merge_blocks);
  L->H_act = take(A * d * L->esize);
  // the forward's partials and the backward's buffers share one region
  const size_t shared_at = off;
  L->part = take((size_t)L->tiles_v * A * 8);
  const size_t fwd_end = off;
  L->fwd_total = fwd_end;
  off = shared_at;
  // H^T and W^T: d rows padded to a whole 256-row tile (bf16 stage-tiled layout)
  const size_t d_pad = (size_t)round_up(d, kRowPad);
  L->Ht = take(d_pad * A * L->esize);
  L->Wt = take(d_pad * L->V_pad * L->esize);
  L->G = take(A * (size_t)L->Vc * L->esize);
  L->w_rows = dtype == AGRL_BF16 && L->A_pad <= kWRowsMax;
  if (L->w_rows) {
    L->tail = L->Wt;
    L->ph = L->Wt + round_up((int64_t)kTailRows * d * 2, 256);
    const size_t n = L->ph < L->G ? (L->G - L->ph) / (A * d * 4) : 0;
    L->ph_max = (int32_t)(n > 32 ? 32 : n);
    L->w_rows = n > 0;        // (a tiny vocabulary's W^T is smaller than dH)
  }
  if (dtype == AGRL_F32) {
    // The fp32 products read H_act and W as they lie: no H^T and W^T.  G, then half
    // of the rest for the parts of each gradient product (G is budgeted twice)
    take((size_t)L->Vc * A * L->esize);
    const size_t g_bytes = A * (size_t)L->Vc * 4;
    L->G = shared_at;
    L->ph = shared_at + g_bytes;
    const size_t half = (off - L->ph) / 2 / 256 * 256;
    L->pw = L->ph + half;
    auto parts = [&](size_t rows) {
      const size_t n = half / (rows * d * 4);
      return (int32_t)(n < 1 ? 1 : n > 32 ? 32 : n);
    };
    L->ph_max = parts(A);
    L->pw_max = parts((size_t)L->Vc);
  }
  if (fwd_end > off) off = fwd_end;
  L->total = off;
  return true;
}

struct Common {
  int64_t T, max_act;
  int32_t d, V, dtype;
  float eps_lo, eps_hi, inv_temp;
  agrl_options o;
};

int validate(const char* fn, int64_t T, int64_t max_act, int32_t d, int32_t V, int32_t dtype,
             const void* H, const void* W, const int32_t* token_id, const uint8_t* mask,
             const float* adv, const float* old, float eps_lo, float eps_hi, int64_t n_norm,
             const agrl_options* opt, void* ws, size_t ws_bytes, Common* c,
             bool loss_inputs = true) {
  char buf[200];
  auto bad = [&](int code, const char* what) {
    snprintf(buf, sizeof buf, "%s: %s", fn, what);
    return fail(code, buf);
  };
  if (dtype != AGRL_BF16 && dtype != AGRL_F32) return bad(AGRL_E_DTYPE, "dtype must be AGRL_BF16 or AGRL_F32");
  if (T < 0) return bad(AGRL_E_SHAPE, "T < 0");
  if (T > ((int64_t)1 << 31) - kScanTile) return bad(AGRL_E_SHAPE, "T too large");
  if (d <= 0 || V <= 0) return bad(AGRL_E_SHAPE, "d and V must be positive");
  if (d % 64 != 0) return bad(AGRL_E_UNSUPPORTED, "d must be a multiple of 64");
  if (n_norm < 0) return bad(AGRL_E_SHAPE, "n_norm < 0");
  if (!(eps_lo >= 0.0f && eps_lo < 1.0f) || !(eps_hi >= 0.0f) || !isfinite(eps_hi))
    return bad(AGRL_E_FLAGS, "clip bounds must satisfy 0 <= low < 1 and 0 <= high < inf");
  agrl_options o = {};
  if (opt) o = *opt;
  if (!(o.temperature >= 0.0f) || !isfinite(o.temperature))
    return bad(AGRL_E_FLAGS, "temperature must be finite and >= 0");
  if (o.dw_accumulate != 0 && o.dw_accumulate != 1) return bad(AGRL_E_FLAGS, "dw_accumulate must be 0 or 1");
  if (o.g_chunk_bytes < 0) return bad(AGRL_E_FLAGS, "g_chunk_bytes < 0");
  if (!isfinite(o.kl_beta)) return bad(AGRL_E_FLAGS, "kl_beta must be finite");
  if (o.kl_estimator != 0 && o.kl_estimator != 1) return bad(AGRL_E_FLAGS, "kl_estimator must be 0 or 1");
  if (loss_inputs && o.kl_beta != 0.0f && T > 0 && !o.ref_logp)
    return bad(AGRL_E_NULL, "kl_beta != 0 needs ref_logp");
  if (T > 0 && (!H || !token_id || !mask || (loss_inputs && (!adv || !old))))
    return bad(AGRL_E_NULL, "input pointer is NULL");
  if (!W) return bad(AGRL_E_NULL, "W is NULL");
  if (max_act <= 0 || max_act > T) max_act = T;
  // every tile row offset and the G buffers use 32-bit row indices
  // operand rows are addressed as 32-bit offsets within a 256-row tile, so a row
  // of any operand (d, V or the padded action count, in elements) stays below 8M
  // (this also bounds dW's transposed read of G: three block columns of at most
  // 2^15 blocks of 32 KiB)
  if (round_up(max_act > 0 ? max_act : 1, kRowPad) > ((int64_t)1 << 23)) return bad(AGRL_E_SHAPE, "max_act too large");
  if (round_up(V, kRowPad) > ((int64_t)1 << 23) || d > (1 << 23)) return bad(AGRL_E_SHAPE, "V or d too large");
  Layout L;
  make_layout(T, max_act, d, V, dtype, o, &L);
  const size_t need = loss_inputs ? L.total : L.fwd_total;
  if (T > 0 && (!ws || ws_bytes < need)) return bad(AGRL_E_WORKSPACE, "workspace missing or too small");
  if ((((uintptr_t)H | (uintptr_t)W | (uintptr_t)ws) & 15) != 0)
    return bad(AGRL_E_SHAPE, "H, W and workspace must be 16-byte aligned");
  c->T = T;
  c->max_act = max_act;
  c->d = d;
  c->V = V;
  c->dtype = dtype;
  c->eps_lo = eps_lo;
  c->eps_hi = eps_hi;
  c->inv_temp = o.temperature == 0.0f ? 1.0f : 1.0f / o.temperature;
  c->o = o;
  return AGRL_OK;
}

enum Phase { PH_FWD = 0, PH_RECOMPUTE = 1, PH_DW = 2, PH_DH = 3 };

void record(const agrl_options& o, int event, hipStream_t s) {
  if (o.phase_events) hipEventRecord(((hipEvent_t*)o.phase_events)[event], s);
}

// Launch n (1 or 2) independent bf16 products: one persistent launch.  `launch` counts
// the call's launches: they use the control block's two tile queues in turn, each
// clearing the next one's (the first is clear).  The phase's events bracket the whole launch (a second phase
// slot, when given, is recorded empty).
template <class Epi>
void launch_gemm(const GemmShape* g, const Epi* e, int n, int max_tiles, int32_t* ctrl, int launch,
                 const agrl_options& o, Phase ph, int ph2, hipStream_t s, int split_max = 1) {
  int grid = device_cu_count();
  if (max_tiles < grid) grid = max_tiles < 1 ? 1 : max_tiles;
  GemmBatch<Epi> b;
  for (int i = 0; i < 2; ++i) {
    b.g[i] = g[i < n ? i : 0];
    b.e[i] = e[i < n ? i : 0];
  }
  b.n = n;
  b.queue = ctrl + CTRL_QUEUE + 16 * (launch & 1);
  b.queue_next = ctrl + CTRL_QUEUE + 16 * (~launch & 1);
  b.cus = device_cu_count();
  b.split_max = split_max;
  record(o, 2 * ph, s);
  // The bf16 store launch is the backward's dH + dW: its operands are
  // stage-tiled, dW reads G transposed, and both K extents are whole stage
  // pairs (the vocabulary chunk rounded up to 128, the device-read token count
  // rounded up in the kernel), so it always runs the 16 x 16 loop.
  if constexpr (std::is_base_of<EpiStore, Epi>::value) {
    hipLaunchKernelGGL((gemm_bf16_kernel<Epi, true>), dim3(grid), dim3(GEMM_THREADS), 0, s, b);
  } else {
    // K, the hidden size: a whole number of stage pairs, or one stage more
    if (g[0].K % (2 * bf16k::SK) == 0)
      hipLaunchKernelGGL((gemm_bf16_kernel<Epi, false>), dim3(grid), dim3(GEMM_THREADS), 0, s, b);
    else
      hipLaunchKernelGGL((gemm_bf16_kernel<Epi, false, true>), dim3(grid), dim3(GEMM_THREADS), 0,
                         s, b);
  }
  record(o, 2 * ph + 1, s);
  if (ph2 >= 0) {
    record(o, 2 * ph2, s);
    record(o, 2 * ph2 + 1, s);
  }
}

// fp32 logits: forward partials, or G of a vocabulary chunk.  64 tokens per tile read
// W half as often; 32 give twice the tiles, for launches whose wide tiles would not
// fill the two workgroups that fit a compute unit.  Either side of the line is flat:
// 38.0 + 42.5 us wide against 41.0 + 36.5 us at V = 4096, d = 256, 1519 tokens (384 wide
// tiles), 419 + 425 against 430 + 418 us at V = 16391, d = 1024, 1333 tokens.
// (A launch holds fewer than 2^32 threads, 2^24 of these workgroups: 2^20 tokens on 2^18
// vocabulary entries have more, so a launch stops at half of that.)
template <bool GRAD>
void launch_logits_f32(f32k::LogitsArgs g, int64_t rows, hipStream_t s) {
  constexpr int64_t kMost = (int64_t)1 << 23;
  const int tiles_m = cdiv(g.nv, 256);
  const int64_t wide = cdiv<int64_t>(rows, 64) * tiles_m;
  const bool is_wide = wide >= 2 * device_cu_count();
  const int64_t blocks = round_up(is_wide ? wide : cdiv<int64_t>(rows, 32) * tiles_m, 8);
  for (int64_t at = 0; at < blocks; at += kMost) {
    const dim3 grid((unsigned)(blocks - at < kMost ? blocks - at : kMost));
    g.block0 = (int32_t)at;
    if (is_wide)
      hipLaunchKernelGGL((f32k::f32_logits_kernel<2, GRAD>), grid, dim3(f32k::THREADS), 0, s, g);
    else
      hipLaunchKernelGGL((f32k::f32_logits_kernel<1, GRAD>), grid, dim3(f32k::THREADS), 0, s, g);
  }
}

// Up to this many tokens the compaction is one launch, whose blocks each count the mask:
// T^2 / 256 bytes read, against two short launches.  Log-prob pass, V = 300, one launch
// against three: 24.2 and 29.3 us at T = 1024, 28.6 and 31.5 at 32768, 30.7 and 31.4 at
// 65536, 34.3 and 32.1 at 98304, 51.1 and 32.5 at 262144 (d = 64, 64 action tokens); 180.4
// and 183.6 at 65536, 326.6 and 325.5 at 131072 (d = 4096, a third action tokens).
constexpr int64_t kOneLaunchTokens = (int64_t)1 << 16;

void compact(const Common& c, const Layout& L, uint8_t* ws, const uint8_t* mask,
             const int32_t* token_id, const float* adv, const float* old, const float* lse_in,
             const float* logp_in, float grad_loss, int64_t n_norm, float* logp_out,
             float* lse_out, const void* H, int* err, hipStream_t s, float* dH = nullptr,
             TailCopy tail = {}) {
  int32_t* ctrl = (int32_t*)(ws + L.ctrl);
  CompactArgs a;
  a.T = c.T;
  a.V = c.V;
  a.d = c.d;
  a.mask = mask;
  a.token_id = token_id;
  a.adv_tok = adv;
  a.old_logp = old;
  a.lse_in = lse_in;
  a.logp_in = logp_in;
  a.blk_off = nullptr;
  a.ctrl = ctrl;
  a.max_act = c.max_act;
  a.idx = (int32_t*)(ws + L.idx);
  a.y_act = (int32_t*)(ws + L.y_act);
  a.adv_act = (float*)(ws + L.adv_act);
  a.old_act = (float*)(ws + L.old_act);
  a.lse_act = lse_in ? (float*)(ws + L.lse_act) : nullptr;
  a.gs_act = lse_in ? (float*)(ws + L.gs_act) : nullptr;
  a.logp_out = logp_out;
  a.lse_out = lse_out;
  a.ref_logp = c.o.kl_beta != 0.0f ? c.o.ref_logp : nullptr;
  a.token_weight = c.o.token_weight;
  a.ref_act = (float*)(ws + L.ref_act);
  a.w_act = (float*)(ws + L.w_act);
  a.kl_beta = c.o.kl_beta;
  a.kl_est = c.o.kl_estimator;
  a.eps_lo = c.eps_lo;
  a.eps_hi = c.eps_hi;
  a.grad_loss = grad_loss;
  a.n_norm = n_norm;
  a.inv_temp = c.inv_temp;
  a.err = err;
  a.H = (const uint8_t*)H;
  a.H_act = ws + L.H_act;
  a.row_bytes = (int64_t)c.d * L.esize;
  a.dH = dH;
  a.tail = tail;
  if (c.T > kOneLaunchTokens) {
    hipLaunchKernelGGL(scan_count_kernel, dim3(L.nblk), dim3(kScanThreads), 0, s, c.T, mask,
                       (int32_t*)(ws + L.blk_cnt));
    hipLaunchKernelGGL(scan_offsets_kernel, dim3(1), dim3(1024), 0, s, L.nblk,
                       (const int32_t*)(ws + L.blk_cnt), (int32_t*)(ws + L.blk_off), ctrl,
                       c.max_act, err);
    a.blk_off = (const int32_t*)(ws + L.blk_off);
  }
  // about eight blocks a compute unit, up to 64 for the same tokens
  const int64_t blocks = cdiv<int64_t>(c.T, kCompactRows);
  const int64_t share = 8 * device_cu_count() / blocks;
  hipLaunchKernelGGL(compact_kernel,
                     dim3((unsigned)blocks, (unsigned)(share < 1 ? 1 : share > 64 ? 64 : share)),
                     dim3(kCompactRows), 0, s, a);
}

void fwd_gemm_bf16(const Common& c, const Layout& L, uint8_t* ws, const void* W, hipStream_t s) {
  const int max_tiles = (int)(L.A_pad / GBM) * L.tiles_v;
  GemmShape g = {};
  g.K = c.d;
  g.group_m = 8;
  // transposed tile (rows: vocabulary, columns: action tokens), so that the
  // log-sum-exp over the vocabulary reduces mostly inside each lane
  g.A = W;
  g.lda = c.d;
  g.M = c.V;
  g.B = ws + L.H_act;
  g.ldb = c.d;
  g.N = (int32_t)L.A_pad;
  g.n_dev = (const int32_t*)(ws + L.ctrl);
  EpiLseCols e;
  e.y = (const int32_t*)(ws + L.y_act);
  e.part = (f32x2*)(ws + L.part);
  e.ld_part = L.A_pad;
  e.zy = (float*)(ws + L.zy);
  e.scale = c.inv_temp;
  launch_gemm(&g, &e, 1, max_tiles, (int32_t*)(ws + L.ctrl), 0, c.o, PH_FWD, -1, s);
}

// loss == nullptr: lse and logp, formed exactly as in the policy-loss forward
void merge(const Common& c, const Layout& L, uint8_t* ws, int64_t n_norm, float* loss, float* logp,
           float* lse, int64_t* n_clip, hipStream_t s) {
  MergeArgs m;
  m.ctrl = (int32_t*)(ws + L.ctrl);
  m.tiles_v = L.tiles_v;
  m.part = (const f32x2*)(ws + L.part);
  m.ld_part = L.A_pad;
  m.zy = (const float*)(ws + L.zy);
  m.y_act = (const int32_t*)(ws + L.y_act);
  m.old_act = (const float*)(ws + L.old_act);
  m.adv_act = (const float*)(ws + L.adv_act);
  m.idx = (const int32_t*)(ws + L.idx);
  m.eps_lo = c.eps_lo;
  m.eps_hi = c.eps_hi;
  m.ref_act = (const float*)(ws + L.ref_act);
  m.w_act = (const float*)(ws + L.w_act);
  m.kl_beta = c.o.kl_beta;
  m.kl_est = c.o.kl_estimator;
  m.weighted = c.o.token_weight != nullptr;
  m.n_norm = n_norm;
  m.logp_out = logp;
  m.lse_out = lse;
  m.blk_sum = (double*)(ws + L.blk_sum);
  m.blk_clip = (unsigned long long*)(ws + L.blk_clip);
  m.loss = loss;
  m.n_clip = n_clip;
  hipLaunchKernelGGL(merge_loss_kernel, dim3(L.merge_blocks), dim3(64 * kMergeWaves), 0, s, m);
}

f32k::LogitsArgs logits_args_f32(const Common& c, const Layout& L, uint8_t* ws, const void* W,
                                 int64_t v0, int32_t nv) {
  f32k::LogitsArgs g = {};
  g.W = (const float*)W + v0 * c.d;
  g.H = (const float*)(ws + L.H_act);
  g.K = c.d;
  g.nv = nv;
  g.n_act = (const int32_t*)(ws + L.ctrl);
  g.y = (const int32_t*)(ws + L.y_act);
  g.scale = c.inv_temp;
  g.col0 = (int32_t)v0;
  return g;
}

void fwd_gemm_f32(const Common& c, const Layout& L, uint8_t* ws, const void* W, hipStream_t s) {
  f32k::LogitsArgs g = logits_args_f32(c, L, ws, W, 0, c.V);
  g.part = (f32x2*)(ws + L.part);
  g.ld_part = L.A_pad;
  g.zy = (float*)(ws + L.zy);
  record(c.o, 2 * PH_FWD, s);
  launch_logits_f32<false>(g, L.A_pad, s);
  record(c.o, 2 * PH_FWD + 1, s);
}

void fwd_gemm(const Common& c, const Layout& L, uint8_t* ws, const void* W, hipStream_t s) {
  if (c.dtype == AGRL_BF16)
    fwd_gemm_bf16(c, L, ws, W, s);
  else
    fwd_gemm_f32(c, L, ws, W, s);
}

void bwd_gemms_f32(const Common& c, const Layout& L, uint8_t* ws, const void* W, float* dH,
                   float* dW, hipStream_t s) {
  const int cus = device_cu_count();
  for (int64_t v0 = 0; v0 < c.V; v0 += L.Vc) {
    const int32_t nv = (int32_t)((c.V - v0) < L.Vc ? (c.V - v0) : L.Vc);
    f32k::LogitsArgs g = logits_args_f32(c, L, ws, W, v0, nv);
    g.lse = (const float*)(ws + L.lse_act);
    g.gs = (const float*)(ws + L.gs_act);
    g.G = (float*)(ws + L.G);
    g.ldg = L.Vc;
    record(c.o, 2 * PH_RECOMPUTE, s);
    launch_logits_f32<true>(g, L.A_pad, s);
    record(c.o, 2 * PH_RECOMPUTE + 1, s);
    f32k::GradArgs a;
    a.G = g.G;
    a.ldg = L.Vc;
    a.W = g.W;
    a.H = g.H;
    a.d = c.d;
    a.nv = nv;
    a.n_act = g.n_act;
    a.dH = dH;
    a.idx = (const int32_t*)(ws + L.idx);
    a.dh_add = v0 > 0;
    a.dW = dW + v0 * c.d;
    a.dw_add = c.o.dw_accumulate;
    a.ph = (float*)(ws + L.ph);
    a.ph_rows = L.A_pad;
    a.ph_max = L.ph_max;
    a.pw = (float*)(ws + L.pw);
    a.pw_max = L.pw_max;
    a.cus = cus;
    record(c.o, 2 * PH_DW, s);
    hipLaunchKernelGGL(f32k::f32_grad_kernel, dim3(f32k::max_blocks((int)L.A_pad, nv, c.d, cus)),
                       dim3(f32k::THREADS), 0, s, a);
    record(c.o, 2 * PH_DW + 1, s);
    record(c.o, 2 * PH_DH, s);
    record(c.o, 2 * PH_DH + 1, s);
    if (L.ph_max > 1 || L.pw_max > 1)
      hipLaunchKernelGGL(f32k::f32_reduce_kernel, dim3(4 * cus), dim3(f32k::THREADS), 0, s, a);
  }
}

void bwd_gemms_bf16(const Common& c, const Layout& L, uint8_t* ws, const void* W, float* dH,
                    float* dW, hipStream_t s) {
  const int32_t* ctrl = (const int32_t*)(ws + L.ctrl);
  __bf16* Ht = (__bf16*)(ws + L.Ht);
  __bf16* Wt = (__bf16*)(ws + L.Wt);
  __bf16* G = (__bf16*)(ws + L.G);
  // H_act^T [d][A_pad] (zero beyond the action rows) and W^T [d][V_pad] (zero
  // beyond V); both, and G, are stage-tiled: every stage of the two products
  // below is a contiguous 32 KiB block per operand tile (8 KiB in each of four
  // blocks for dW's transposed read of G)
  const dim3 gh((unsigned)(L.A_pad / 64), (unsigned)cdiv(c.d, 64));
  const dim3 gw((unsigned)(L.V_pad / 64), (unsigned)cdiv(c.d, 64));
  hipLaunchKernelGGL(transpose16_kernel, gh, dim3(256), 0, s, (const uint16_t*)(ws + L.H_act),
                     (int64_t)c.d, (uint16_t*)Ht, L.A_pad, (int64_t)0, (int64_t)0, (int64_t)c.d,
                     ctrl);
  if (!L.w_rows)
    hipLaunchKernelGGL(transpose16_kernel, gw, dim3(256), 0, s, (const uint16_t*)W, (int64_t)c.d,
                       (uint16_t*)Wt, L.V_pad, (int64_t)c.V, L.V_pad, (int64_t)c.d,
                       (const int32_t*)nullptr);
  const int row_tiles = (int)(L.A_pad / GBM);
  const int d_tiles = cdiv(c.d, GBN);
  for (int64_t v0 = 0; v0 < c.V; v0 += L.Vc) {
    const int32_t nv = (int32_t)((c.V - v0) < L.Vc ? (c.V - v0) : L.Vc);
    const int nv_tiles = cdiv(nv, GBN);
    {  // logits of the chunk -> G
      GemmShape g = {};
      g.A = ws + L.H_act;
      g.lda = c.d;
      g.B = (const __bf16*)W + v0 * c.d;
      g.ldb = c.d;
      g.m_dev = ctrl;
      g.N = nv;
      g.K = c.d;
      // groups of 8 vocabulary tiles sweep every token tile: each W panel of the
      // chunk is read from memory once (the compacted H is small enough to stay
      // in the Infinity Cache), not once per group of 8 token tiles
      g.group_m = 8;
      g.group_cols = 1;
      EpiLogitGrad e;
      e.y = (const int32_t*)(ws + L.y_act);
      e.lse = (const float*)(ws + L.lse_act);
      e.gs = (const float*)(ws + L.gs_act);
      e.G = G;
      e.ldg = L.A_pad;
      e.scale = c.inv_temp;
      e.col0 = (int32_t)v0;
      launch_gemm(&g, &e, 1, row_tiles * nv_tiles, (int32_t*)(ws + L.ctrl), 0, c.o, PH_RECOMPUTE,
                  -1, s);
    }
    {  // dH[idx] (+)= G W[v0 : v0 + nv] (K = the chunk's vocabulary columns) and
       // dW[v0 : v0 + nv] = G^T H_act (K = action tokens), one launch, dH first:
       // its tiles are the long ones.  G is column-block stage-tiled; dW reads it
       // transposed
      GemmShape g[2] = {};
      g[0].A = G;
      g[0].lda = L.A_pad;
      g[0].B = Wt + v0 * 256;    // the chunk's first column: whole 64-column blocks
      g[0].ldb = L.V_pad;
      g[0].a_tiled = 2;
      g[0].b_tiled = 1;
      g[0].m_dev = ctrl;
      g[0].N = c.d;
      // (a whole number of stage pairs; G and W^T are zero up to Vc and V_pad)
      g[0].K = (int32_t)round_up(nv, 2 * bf16k::SK);
      g[0].group_m = 8;
      g[1].A = G;
      g[1].lda = L.A_pad;
      g[1].B = Ht;
      g[1].ldb = L.A_pad;
      g[1].a_tiled = 2;
      g[1].a_trans = 1;
      g[1].b_tiled = 1;
      g[1].M = nv;
      g[1].N = c.d;
      g[1].k_dev = ctrl;
      g[1].group_m = 8;
      EpiGrad e[2] = {};
      e[0].out = dH;
      e[0].ldo = c.d;
      e[0].row_map = (const int32_t*)(ws + L.idx);
      e[0].accumulate = v0 > 0;
      e[1].out = dW + v0 * c.d;
      e[1].ldo = c.d;
      e[1].row_map = nullptr;
      e[1].accumulate = c.o.dw_accumulate;
      int32_t* queue = (int32_t*)(ws + L.ctrl);
      if (!L.w_rows) {
        const EpiStore es[2] = {e[0], e[1]};
        launch_gemm(g, es, 2, row_tiles * d_tiles + nv_tiles * d_tiles, queue, 1, c.o, PH_DW, PH_DH,
                    s);
        continue;
      }
      // dH^T = W^T G^T: W's rows are K as they lie, the last ones from the padded copy
      GemmShape& h = g[0];
      h.B = h.A;
      h.ldb = h.lda;
      h.b_tiled = 2;
      h.N = (int32_t)L.A_pad;
      h.n_dev = ctrl;
      h.A = (const __bf16*)W + v0 * c.d;
      h.lda = c.d;
      h.a_tiled = 0;
      h.a_trans = 2;
      h.M = c.d;
      h.m_dev = nullptr;
      h.a_tail = ws + L.tail;
      h.a_tail_stage = (int32_t)((c.V / kTailRows * kTailRows - v0) / bf16k::SK);
      const bool add = e[0].accumulate;
      e[0].out = (float*)(ws + L.ph);
      e[0].ldo = L.A_pad;
      e[0].row_map = nullptr;
      e[0].accumulate = 0;
      e[0].part_stride = c.d * L.A_pad;
      launch_gemm(g, e, 2, row_tiles * d_tiles * L.ph_max + nv_tiles * d_tiles, queue, 1, c.o, PH_DW,
                  PH_DH, s, L.ph_max);
      hipLaunchKernelGGL(dh_reduce_kernel, gh, dim3(256), 0, s, (const float*)(ws + L.ph), L.A_pad,
                         ctrl, (const int32_t*)(ws + L.idx), nv, c.d, device_cu_count(), L.ph_max,
                         (int32_t)add, dH);
    }
  }
}

}  // namespace
}  // namespace agrl

extern "C" int64_t agrl_policy_loss_vocab_chunk(int64_t T, int64_t max_act, int32_t d,
                                                int32_t V, int32_t dtype,
                                                const agrl_options* opt) {
  agrl_options o = {};
  if (opt) o = *opt;
  agrl::Layout L;
  if (T <= 0 || o.g_chunk_bytes < 0 || !agrl::make_layout(T, max_act, d, V, dtype, o, &L)) return 0;
  return L.Vc;
}

extern "C" size_t agrl_policy_loss_workspace_size(int64_t T, int64_t max_act, int32_t d,
                                                  int32_t V, int32_t dtype,
                                                  const agrl_options* opt) {
  agrl_options o = {};
  if (opt) o = *opt;
  agrl::Layout L;
  if (T <= 0 || o.g_chunk_bytes < 0 || !agrl::make_layout(T, max_act, d, V, dtype, o, &L)) return 0;
  return L.total;
}

extern "C" int agrl_policy_loss_fwd(int64_t T, int64_t max_act, int32_t d, int32_t V,
                                    int32_t dtype, const void* H, const void* W,
                                    const int32_t* token_id, const uint8_t* action_mask,
                                    const float* adv_tok, const float* old_logp,
                                    float clip_eps_low, float clip_eps_high, int64_t n_norm,
                                    const agrl_options* opt, void* workspace, size_t ws_bytes,
                                    float* loss, float* logp, float* lse, int64_t* n_clip,
                                    void* stream) {
  using namespace agrl;
  Common c;
  int rc = validate("agrl_policy_loss_fwd", T, max_act, d, V, dtype, H, W, token_id, action_mask,
                    adv_tok, old_logp, clip_eps_low, clip_eps_high, n_norm, opt, workspace,
                    ws_bytes, &c);
  if (rc) return rc;
  if (!loss || (T > 0 && (!logp || !lse))) return fail(AGRL_E_NULL, "agrl_policy_loss_fwd: output pointer is NULL");
  hipStream_t s = (hipStream_t)stream;
  int* err = device_error_ptr();
  if (!err) return hip_status(hipErrorInvalidSymbol);
  if (T == 0) {
    hipLaunchKernelGGL(zero_loss_kernel, dim3(1), dim3(1), 0, s, loss, n_clip);
    return hip_status(hipGetLastError());
  }
  Layout L;
  make_layout(T, c.max_act, d, V, dtype, c.o, &L);
  uint8_t* ws = (uint8_t*)workspace;
  compact(c, L, ws, action_mask, token_id, adv_tok, old_logp, nullptr, nullptr, 0.0f, n_norm,
          logp, lse, H, err, s);
  fwd_gemm(c, L, ws, W, s);
  merge(c, L, ws, n_norm, loss, logp, lse, n_clip, s);
  return hip_status(hipGetLastError());
}

extern "C" size_t agrl_token_logprob_workspace_size(int64_t T, int64_t max_act, int32_t d,
                                                    int32_t V, int32_t dtype,
                                                    const agrl_options* opt) {
  agrl_options o = {};
  if (opt) o = *opt;
  agrl::Layout L;
  if (T <= 0 || o.g_chunk_bytes < 0 || !agrl::make_layout(T, max_act, d, V, dtype, o, &L)) return 0;
  return L.fwd_total;
}

extern "C" int agrl_token_logprob(int64_t T, int64_t max_act, int32_t d, int32_t V, int32_t dtype,
                                  const void* H, const void* W, const int32_t* token_id,
                                  const uint8_t* action_mask, const agrl_options* opt,
                                  void* workspace, size_t ws_bytes, float* logp, float* lse,
                                  void* stream) {
  using namespace agrl;
  Common c;
  int rc = validate("agrl_token_logprob", T, max_act, d, V, dtype, H, W, token_id, action_mask,
                    nullptr, nullptr, 0.0f, 0.0f, 0, opt, workspace, ws_bytes, &c, false);
  if (rc) return rc;
  if (T > 0 && (!logp || !lse)) return fail(AGRL_E_NULL, "agrl_token_logprob: output pointer is NULL");
  if (T == 0) return AGRL_OK;
  c.o.kl_beta = 0.0f;          // loss-only options play no part here
  c.o.token_weight = nullptr;
  hipStream_t s = (hipStream_t)stream;
  int* err = device_error_ptr();
  if (!err) return hip_status(hipErrorInvalidSymbol);
  Layout L;
  make_layout(T, c.max_act, d, V, dtype, c.o, &L);
  uint8_t* ws = (uint8_t*)workspace;
  compact(c, L, ws, action_mask, token_id, nullptr, nullptr, nullptr, nullptr, 0.0f, 0, logp,
          lse, H, err, s);
  fwd_gemm(c, L, ws, W, s);
  merge(c, L, ws, 0, nullptr, logp, lse, nullptr, s);
  return hip_status(hipGetLastError());
}

extern "C" int agrl_policy_loss_bwd(int64_t T, int64_t max_act, int32_t d, int32_t V,
                                    int32_t dtype, const void* H, const void* W,
                                    const int32_t* token_id, const uint8_t* action_mask,
                                    const float* adv_tok, const float* old_logp,
                                    float clip_eps_low, float clip_eps_high, int64_t n_norm,
                                    const agrl_options* opt, const float* lse, const float* logp,
                                    float grad_loss, void* workspace, size_t ws_bytes, float* dH,
                                    float* dW, void* stream) {
  using namespace agrl;
  Common c;
  int rc = validate("agrl_policy_loss_bwd", T, max_act, d, V, dtype, H, W, token_id, action_mask,
                    adv_tok, old_logp, clip_eps_low, clip_eps_high, n_norm, opt, workspace,
                    ws_bytes, &c);
  if (rc) return rc;
  if (!dW || (T > 0 && (!dH || !lse || !logp)))
    return fail(AGRL_E_NULL, "agrl_policy_loss_bwd: lse/logp/dH/dW pointer is NULL");
  if (((uintptr_t)dH | (uintptr_t)dW) % 16 != 0)
    return fail(AGRL_E_UNSUPPORTED, "agrl_policy_loss_bwd: dH and dW must be 16-byte aligned");
  if (!isfinite(grad_loss)) return fail(AGRL_E_FLAGS, "agrl_policy_loss_bwd: grad_loss must be finite");
  hipStream_t s = (hipStream_t)stream;
  int* err = device_error_ptr();
  if (!err) return hip_status(hipErrorInvalidSymbol);
  if (T == 0) {
    if (!c.o.dw_accumulate) {
      const int64_t n = (int64_t)V * d;
      hipLaunchKernelGGL(zero_f32_kernel, dim3((unsigned)(n / 256 < 4096 ? n / 256 + 1 : 4096)),
                         dim3(256), 0, s, dW, n);
    }
    return hip_status(hipGetLastError());
  }
  Layout L;
  make_layout(T, c.max_act, d, V, dtype, c.o, &L);
  uint8_t* ws = (uint8_t*)workspace;
  TailCopy tail = {};
  const int64_t tail0 = V / kTailRows * kTailRows;
  if (L.w_rows && tail0 < V)
    tail = TailCopy{(const uint8_t*)W + tail0 * d * 2, V - tail0, ws + L.tail};
  compact(c, L, ws, action_mask, token_id, adv_tok, old_logp, lse, logp, grad_loss, n_norm,
          nullptr, nullptr, H, err, s, dH, tail);
  if (dtype == AGRL_BF16)
    bwd_gemms_bf16(c, L, ws, W, dH, dW, s);
  else
    bwd_gemms_f32(c, L, ws, W, dH, dW, s);
  return hip_status(hipGetLastError());
}
