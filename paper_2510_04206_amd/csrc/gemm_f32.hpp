// fp32 products of the policy loss on the matrix cores (v_mfma_f32_32x32x2_f32).
//
// The fp32 matrix rate is a sixteenth of the bf16 one: 64 cycles per MFMA, so
// operands read from LDS four bytes a lane keep up with it, and what bounds these
// products is how evenly a small problem spreads over the chip.  Hence small tiles
// with several workgroups resident per compute unit, K split where the tiles are
// few, and no transposed copies: an operand whose K runs along its rows is staged
// as it lies and read column-wise.
//
//   logits    z^T = W H_act^T, tile 256 vocabulary rows x 32 BJ tokens, each wave 64
//             rows: the log-sum-exp over the vocabulary is lane-local but for one
//             exchange.  Forward (log-sum-exp partials) and recompute (G) run the
//             same loop, so the backward's logits are the forward's to the bit.
//   gradients dH = G W (K = vocabulary) and dW = G^T H_act (K = tokens) in one
//             launch, tile 64 x 64, K split so that every part is a fraction
//             of a compute unit's share; parts go to fp32 partial buffers that one
//             more kernel adds in a fixed order.
//
// A K stage is 32 floats deep, double-buffered, one barrier per stage.
#pragma once
#include "common.hpp"
#include "gemm.hpp"

namespace agrl {
namespace f32k {

using bf16k::copy16;
constexpr int SK = 32;                 // k per stage
constexpr int ROW = SK * 4;            // bytes per row of a K-contiguous operand and stage
constexpr int THREADS = 256;

__device__ __forceinline__ void stage_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One operand tile of R rows (of the product) per stage.  KM = false: K-contiguous,
// row-major rows of the tile, 128 bytes each, in the swizzle of the bf16 kernel.
// KM = true: the K index runs along memory rows; a stage is 32 k-rows of R floats,
// stored as they come.  Rows (KM: 4-float column chunks, k-rows) past the end are
// clamped to the last valid one; the epilogue drops what comes of them (a clamped
// k-row meets zeros in the other operand).
template <int R, bool KM>
struct Tile {
  static constexpr int BYTES = R * ROW;
  static constexpr int NC = R / 32;                     // copies per wave per stage
  static constexpr int KPC = KM ? 256 / R : 0;          // k-rows per copy
  const uint8_t* base;
  int64_t step;        // bytes per stage
  uint32_t off[NC];    // K-contiguous: the lane's byte offset; KM: its column offset
  int kr[NC];          // KM: the lane's k-row of each copy
  uint32_t ld_b;

  // p: element (row r0, k = 0) of the operand; rows: rows from r0 to the end
  __device__ __forceinline__ void init(const float* p, int64_t ld, int rows, int wave, int lane) {
    // The base is the first row that the wave copies (64 rows of at most 2^23 floats, or 32
    // k-rows, stay within the 32-bit offsets; a tile's 256 rows would not)
    const int first = KM ? 0 : min(wave * NC * 8, rows - 1);
    base = (const uint8_t*)(p + first * ld);
    ld_b = (uint32_t)(ld * 4);
    if constexpr (KM) {
      step = (int64_t)SK * ld * 4;
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        kr[b] = (wave * NC + b) * KPC + lane / (R / 4);
        off[b] = (uint32_t)(min((lane % (R / 4)) * 4, rows - 4) * 4);
      }
    } else {
      step = ROW;
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        const int row = (wave * NC + b) * 8 + (lane >> 3);
        off[b] = (uint32_t)(min(row, rows - 1) - first) * ld_b +
                 (uint32_t)(((lane & 7) ^ row_swizzle(row)) << 4);
      }
    }
  }
  // stage s into LDS at byte address lds (already offset by the wave); KM: k-rows
  // past klast (relative to the operand's start) are clamped
  __device__ __forceinline__ void copy(int s, uint32_t lds, int klast) const {
    const uint8_t* at = base + s * step;
#pragma unroll
    for (int b = 0; b < NC; ++b) {
      uint32_t o = off[b];
      if constexpr (KM) o += (uint32_t)min(kr[b], klast - s * SK) * ld_b;
      copy16<0>(at, o, lds + b * 1024);
    }
  }
  // the 8 k values of slice kk (k = 16 kk + 8 (lane / 32) + e) of block row blk + lane % 32
  static __device__ __forceinline__ void read(const uint8_t* st, int blk, int kk, int lane,
                                              float (&v)[8]) {
    const int r = lane & 31, h = lane >> 5;
    if constexpr (KM) {
      const float* p = (const float*)st + (kk * 16 + h * 8) * R + blk + r;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = p[e * R];
    } else {
      const uint8_t* p = st + (blk + r) * ROW;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4 x = *(const f32x4*)(p + (((kk * 4 + h * 2 + c) ^ row_swizzle(r)) << 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * c + e] = x[e];
      }
    }
  }
};

// The K loop over stages [s0, s1): waves in a WM x WN arrangement, each owning
// BI x BJ blocks of 32 x 32.  LDS: two buffers of the A tile then the B tile.
template <int WM, int WN, int BI, int BJ, bool AKM, bool BKM>
__device__ __forceinline__ void main_loop(f32x16 (&acc)[BI][BJ], uint8_t* smem,
                                          const Tile<WM * BI * 32, AKM>& A,
                                          const Tile<WN * BJ * 32, BKM>& B, int s0, int s1,
                                          int b_klast, int wave, int lane) {
  typedef Tile<WM * BI * 32, AKM> TA;
  typedef Tile<WN * BJ * 32, BKM> TB;
  constexpr int BUF = TA::BYTES + TB::BYTES;
  const int wm = wave / WN, wn = wave % WN;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)smem);
  auto copy = [&](int s) {
    const uint32_t at = lds0 + (uint32_t)((s & 1) * BUF);
    A.copy(s, at + wave * TA::NC * 1024, 1 << 30);
    B.copy(s, at + TA::BYTES + wave * TB::NC * 1024, b_klast);
  };
  if (s0 >= s1) return;
  copy(s0);
  for (int s = s0; s < s1; ++s) {
    // stage s has landed and every wave is done with stage s - 1's buffer
    stage_barrier();
    if (s + 1 < s1) copy(s + 1);
    const uint8_t* st = smem + (s & 1) * BUF;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      float a[BI][8], b[BJ][8];
#pragma unroll
      for (int i = 0; i < BI; ++i) TA::read(st, (wm * BI + i) * 32, kk, lane, a[i]);
#pragma unroll
      for (int j = 0; j < BJ; ++j) TB::read(st + TA::BYTES, (wn * BJ + j) * 32, kk, lane, b[j]);
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < BI; ++i)
#pragma unroll
          for (int j = 0; j < BJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
    }
  }
}

template <int BI, int BJ>
__device__ __forceinline__ void clear(f32x16 (&acc)[BI][BJ]) {
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
}

// Accumulator element r of a 32 x 32 block: row acc_r(r, lane), column lane & 31.
__device__ __forceinline__ int acc_r(int r, int lane) {
  return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

// Workgroup b of a launch runs on XCD b mod 8; this gives every XCD a run of
// consecutive items, so that the tiles it works on share operand panels in its L2.
// Returns total or more for a surplus workgroup.
__device__ __forceinline__ int xcd_item(int b, int total) {
  const int per = cdiv(total, 8);
  return b / 8 < per ? (b & 7) * per + b / 8 : total;
}

// ------------------------------------------------------------------ logits
struct LogitsArgs {
  const float* W;          // [nv][K] (the chunk's first row)
  const float* H;          // [tokens][K], compacted
  int32_t K;               // hidden size, a multiple of 64
  int32_t nv;              // vocabulary rows
  const int32_t* n_act;
  const int32_t* y;        // [tokens] target id
  float scale;             // 1 / temperature
  // forward
  f32x2* part;             // [ceil(nv / 256)][ld_part] (max, sum exp)
  int64_t ld_part;
  float* zy;               // [tokens] target logit
  // recompute
  const float* lse;
  const float* gs;         // dL/dlogp / temperature
  float* G;                // [tokens][ldg]
  int64_t ldg;
  int32_t col0;            // vocabulary index of row 0
  int32_t block0;          // workgroups of the launch before this one's (a multiple of 8)
};

// Two workgroups per compute unit: 72 or 80 KiB of LDS each.  A tile spans the 256
// vocabulary rows of one partial.  419 us at V = 16391, d = 1024, 1333 tokens (107
// TFLOP/s; 2.7 rounds of tiles), 41 us at V = 4096, d = 256, 1519 tokens, against 556
// and 82 us with 256 x 256 tiles.
template <int BJ, bool GRAD>
__global__ __launch_bounds__(THREADS, 2) void f32_logits_kernel(LogitsArgs g) {
  typedef Tile<256, false> TA;
  typedef Tile<32 * BJ, false> TB;
  __shared__ __attribute__((aligned(16))) uint8_t smem[2 * (TA::BYTES + TB::BYTES)];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_act = __builtin_amdgcn_readfirstlane(*g.n_act);
  const int tiles_n = cdiv(n_act, 32 * BJ), tiles_m = cdiv(g.nv, 256);
  const int total = tiles_m * tiles_n;
  const int t = xcd_item(blockIdx.x + g.block0, total);
  if (t >= total) return;
  // all token tiles of a vocabulary tile in a row: its panel of W is read once
  const int m0 = (t / tiles_n) * 256, n0 = (t % tiles_n) * 32 * BJ;
  TA A;
  TB B;
  A.init(g.W + (int64_t)m0 * g.K, g.K, g.nv - m0, wave, lane);
  // (H_act's rows past n_act are zero up to a multiple of 256: no clamp)
  B.init(g.H + (int64_t)n0 * g.K, g.K, 32 * BJ, wave, lane);
  f32x16 acc[2][BJ];
  clear(acc);
  main_loop<4, 1, 2, BJ>(acc, smem, A, B, 0, g.K / SK, 1 << 30, wave, lane);
  // this lane's vocabulary rows are m0 + wave * 64 + 4 (lane / 32) + o,
  // o = 32 i + 8 (r / 4) + r % 4, of the tokens n0 + 32 j + lane % 32
  const int rb = wave * 64 + 4 * (lane >> 5);
  const int lim = g.nv - m0 - rb;      // rows o >= lim are beyond the vocabulary
  const float k1 = g.scale * 1.44269504088896341f;
  if constexpr (GRAD) {
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int n = n0 + 32 * j + (lane & 31);
      const bool live = n < n_act;
      const float lse = live ? g.lse[n] : INFINITY;      // dead tokens: exp(-inf) = 0
      const float gs = live ? g.gs[n] : 0.0f;
      const int o_y = live ? g.y[n] - g.col0 - m0 - rb : -1;
      float* row = g.G + (int64_t)n * g.ldg + m0 + rb;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          f32x4 v;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int o = 32 * i + 8 * r4 + q;
            const float p = __expf(fmaf(acc[i][j][4 * r4 + q], g.scale, -lse));
            v[q] = o < lim ? gs * ((o == o_y ? 1.0f : 0.0f) - p) : 0.0f;
          }
          *(f32x4*)(row + 32 * i + 8 * r4) = v;
        }
    }
  } else {
    f32x2* red = (f32x2*)smem;       // [4 waves][32 BJ]
    __syncthreads();                 // the last stage has been read
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int c = 32 * j + (lane & 31);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          mx = fmaxf(mx, 32 * i + 8 * (r >> 2) + (r & 3) < lim ? acc[i][j][r] : -INFINITY);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mk = mx != -INFINITY ? -mx * k1 : 0.0f;
      const int o_y = n0 + c < n_act ? g.y[n0 + c] - m0 - rb : -1;
      float sm = 0.0f, zy = 0.0f;
      bool mine = false;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int o = 32 * i + 8 * (r >> 2) + (r & 3);
          const float e = __builtin_amdgcn_exp2f(fmaf(acc[i][j][r], k1, mk));
          sm += o < lim ? e : 0.0f;
          zy = o == o_y ? acc[i][j][r] : zy;
          mine = mine || o == o_y;
        }
      sm += __shfl_xor(sm, 32);
      if (lane < 32) red[wave * 32 * BJ + c] = f32x2{mx * g.scale, sm};
      if (mine) g.zy[n0 + c] = zy * g.scale;
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < 32 * BJ && n0 + c < n_act) {
      float m = red[c].x, s = 0.0f;
#pragma unroll
      for (int w = 1; w < 4; ++w) m = fmaxf(m, red[w * 32 * BJ + c].x);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const f32x2 p = red[w * 32 * BJ + c];
        s += p.y == 0.0f ? 0.0f : p.y * __expf(p.x - m);   // (a NaN sum stays)
      }
      g.part[(int64_t)(m0 / 256) * g.ld_part + n0 + c] = f32x2{m, s};
    }
  }
}

// ------------------------------------------------------------------ gradients
struct GradArgs {
  const float* G;          // [tokens][ldg], zero past the chunk's columns and n_act
  int64_t ldg;
  const float* W;          // [nv][d], the chunk's rows
  const float* H;          // [tokens][d], compacted, zero rows past n_act
  int32_t d, nv;
  const int32_t* n_act;
  float* dH;               // [T][d]
  const int32_t* idx;      // token of each compacted row
  int32_t dh_add;          // add to dH (chunks after the first)
  float* dW;               // [nv][d]
  int32_t dw_add;
  float* ph;               // dH partials [split][ph_rows][d]
  int64_t ph_rows;
  int32_t ph_max;          // most splits its buffer holds (1: none)
  float* pw;               // dW partials [split][nv][d]
  int32_t pw_max;
  int32_t cus;             // compute units
};

// How the launch's K extents are split: an item is at most 1 / PARTS of a compute
// unit's share of the stages, and not shorter than MIN_STAGES (below that a part's
// epilogue costs as much as its loop).  Device code decides, from the action tokens
// there are; max_blocks bounds the grid from the tokens there may be.
// (PARTS 2, 4, 8: 80.6, 74.0, 71.2 us at V = 4096, d = 256, 1519 tokens, and 871, 803,
// 816 us at V = 16391, d = 1024, 1333 tokens, where dW's 4112 tiles need no split.)
constexpr int PARTS = 4;
constexpr int MIN_STAGES = 12;
constexpr int GT = 64;                 // rows and columns of a tile
struct Split {
  int tiles_d, th, tw;     // column tiles; tiles of dH and dW
  int kh, kw;              // stages
  int sh, sw;              // splits
};
__host__ __device__ inline Split grad_split(int n_act, int nv, int d, int cus, int ph_max,
                                            int pw_max) {
  Split s;
  s.tiles_d = cdiv(d, GT);
  s.th = cdiv(n_act, GT) * s.tiles_d;
  s.tw = cdiv(nv, GT) * s.tiles_d;
  s.kh = cdiv(nv, SK);
  s.kw = cdiv(n_act, SK);
  const int64_t work = (int64_t)s.th * s.kh + (int64_t)s.tw * s.kw;
  int64_t most = work / ((int64_t)cus * PARTS);
  if (most < MIN_STAGES) most = MIN_STAGES;
  const int64_t sh = (s.kh + most - 1) / most, sw = (s.kw + most - 1) / most;
  s.sh = (int)(sh < ph_max ? sh : ph_max);
  s.sw = (int)(sw < pw_max ? sw : pw_max);
  if (s.sw < 1) s.sw = 1;      // no action tokens: dW is written as zeros
  return s;
}

// Items <= tiles + work / most, and most is PARTS' share rounded down (>= 12: by at
// most a twelfth); each product's blocks are a multiple of 8.
__host__ inline int max_blocks(int rows, int nv, int d, int cus) {
  const int64_t tiles = (int64_t)(cdiv(rows, GT) + cdiv(nv, GT)) * cdiv(d, GT);
  return (int)(tiles + cus * PARTS * 13 / 12 + 16);
}

__device__ __forceinline__ void store_tile(const f32x16 (&acc)[1][1], float* out, int64_t ld,
                                           const int32_t* row_map, bool add, int m0, int M, int n0,
                                           int N, int wm, int wn, int lane) {
  const int c = n0 + wn * 32 + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = m0 + wm * 32 + acc_r(r, lane);
    if (row < M) {
      float* dst = out + (int64_t)(row_map ? row_map[row] : row) * ld;
      if (c < N) dst[c] = add ? dst[c] + acc[0][0][r] : acc[0][0][r];
    }
  }
}

// 64 x 64 tiles, five workgroups per compute unit: 74 us at V = 4096, d = 256, 1519
// tokens (6.4 GF; 87 TFLOP/s) and 803 us at V = 16391, d = 1024, 1333 tokens (112 TFLOP/s
// of the 151 a large fp32 library product reaches); 256 x 256 tiles over the whole K
// and transposed copies took 1352 and 4614 us, with 6 and 24 workgroups for dH.
// 128 x 64, 64 x 128 and 128 x 128 tiles are within 6% of it at both sizes.
__global__ __launch_bounds__(THREADS, 2) void f32_grad_kernel(GradArgs g) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[2 * (GT + GT) * ROW];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_act = __builtin_amdgcn_readfirstlane(*g.n_act);
  const Split s = grad_split(n_act, g.nv, g.d, g.cus, g.ph_max, g.pw_max);
  // dH's items first, each product's spread over all XCDs
  const int items_h = s.th * s.sh, items_w = s.tw * s.sw, blocks_h = 8 * cdiv(items_h, 8);
  const bool is_h = (int)blockIdx.x < blocks_h;
  int t = is_h ? xcd_item(blockIdx.x, items_h) : xcd_item(blockIdx.x - blocks_h, items_w);
  if (t >= (is_h ? items_h : items_w)) return;
  f32x16 acc[1][1];
  clear(acc);
  const int wm = wave >> 1, wn = wave & 1;
  if (is_h) {
    // dH: rows tokens, K = the chunk's vocabulary
    const int part = t / s.th;
    t -= part * s.th;
    const int m0 = (t / s.tiles_d) * GT, n0 = (t % s.tiles_d) * GT;
    const int per = cdiv(s.kh, s.sh), k0 = part * per, k1 = min(s.kh, k0 + per);
    Tile<GT, false> A;
    Tile<GT, true> B;
    A.init(g.G + (int64_t)m0 * g.ldg, g.ldg, n_act - m0, wave, lane);
    B.init(g.W + n0, g.d, g.d - n0, wave, lane);
    main_loop<2, 2, 1, 1>(acc, smem, A, B, k0, k1, g.nv - 1, wave, lane);
    if (s.sh > 1)
      store_tile(acc, g.ph + (int64_t)part * g.ph_rows * g.d, g.d, nullptr, false, m0, n_act, n0,
                 g.d, wm, wn, lane);
    else
      store_tile(acc, g.dH, g.d, g.idx, g.dh_add, m0, n_act, n0, g.d, wm, wn, lane);
  } else {
    // dW: rows vocabulary, K = tokens
    const int part = t / s.tw;
    t -= part * s.tw;
    const int m0 = (t / s.tiles_d) * GT, n0 = (t % s.tiles_d) * GT;
    const int per = cdiv(s.kw, s.sw), k0 = part * per, k1 = min(s.kw, k0 + per);
    Tile<GT, true> A;
    Tile<GT, true> B;
    A.init(g.G + m0, g.ldg, (int)g.ldg - m0, wave, lane);
    B.init(g.H + n0, g.d, g.d - n0, wave, lane);
    main_loop<2, 2, 1, 1>(acc, smem, A, B, k0, k1, 1 << 30, wave, lane);
    if (s.sw > 1)
      store_tile(acc, g.pw + (int64_t)part * g.nv * g.d, g.d, nullptr, false, m0, g.nv, n0, g.d,
                 wm, wn, lane);
    else
      store_tile(acc, g.dW, g.d, nullptr, g.dw_add, m0, g.nv, n0, g.d, wm, wn, lane);
  }
}

// The split products' parts, added in ascending order: dH rows go to their tokens.
__global__ __launch_bounds__(THREADS) void f32_reduce_kernel(GradArgs g) {
  const int n_act = *g.n_act;
  const Split s = grad_split(n_act, g.nv, g.d, g.cus, g.ph_max, g.pw_max);
  const int64_t c4 = g.d / 4;
  const int64_t nh = s.sh > 1 ? n_act * c4 : 0, nw = s.sw > 1 ? g.nv * c4 : 0;
  for (int64_t i = (int64_t)blockIdx.x * THREADS + threadIdx.x; i < nh + nw;
       i += (int64_t)gridDim.x * THREADS) {
    const bool h = i < nh;
    const int64_t e = h ? i : i - nh;
    const f32x4* p = (const f32x4*)(h ? g.ph : g.pw) + e;
    const int64_t stride = h ? g.ph_rows * c4 : g.nv * c4;
    const int parts = h ? s.sh : s.sw;
    f32x4* out = h ? (f32x4*)g.dH + (int64_t)g.idx[e / c4] * c4 + e % c4 : (f32x4*)g.dW + e;
    f32x4 v = p[0];
    for (int k = 1; k < parts; ++k) v += p[k * stride];
    if (h ? g.dh_add : g.dw_add) v += *out;
    *out = v;
  }
}

}  // namespace f32k
}  // namespace agrl
