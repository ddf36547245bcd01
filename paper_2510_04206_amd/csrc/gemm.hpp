// Persistent bf16 "NT" GEMM on the gfx950 matrix cores: C[M, N] = A[M, K] * B[N, K]^T,
// both operands K-contiguous (A can also be read transposed from its stage-tiled
// storage), fp32 accumulation, with a fused epilogue functor.
//
// Block tile 256 x 256, 4 waves in a 2 x 2 arrangement, each wave owning a
// 128 x 128 sub-tile as 8 x 8 blocks of v_mfma_f32_16x16x32_bf16 accumulators (half
// the accumulator traffic per flop of the 32 x 32 shape: under the board power limit
// the chip then holds a higher clock).
// Each K stage moves 128 bytes of every tile row from global memory straight into
// LDS (no register staging), double-buffered (a second barrier in the middle of the
// stage gives a stage's copies until then to land).  The 16-byte chunk c of tile row r is
// stored at chunk c ^ ((r >> 1) & 7): a 128-bit LDS read serves 16 lanes per pass
// from a 256-byte window (two 128-byte rows), and this places the 16 rows such a
// pass touches in 16 distinct bank groups.
//
// The grid is persistent (about one workgroup per compute unit, since a block
// holds 128 KiB of LDS).  The row counts M and N and the K extent may be read
// from device memory, so a launch sized for an upper bound does only the work
// the data needs without a host round trip.  Workgroups are dealt to the 8 XCDs
// round-robin, and the tile queues (below) keep an XCD's workgroups on a compact
// block of tiles that shares its A and B panels in the XCD's L2.
#pragma once
#include <type_traits>
#include <utility>

#include "common.hpp"

namespace agrl {

constexpr int GBM = 256;
constexpr int GBN = 256;
constexpr int LDS_ROW = 128;                            // bytes per tile row per stage
constexpr int STAGE_BYTES = (GBM + GBN) * LDS_ROW;      // 64 KiB
constexpr int GEMM_LDS = 2 * STAGE_BYTES;               // 128 KiB of stage buffers
// bf16 logit-gradient epilogue (two passes of 128 tile rows): G rows staged
// row-major with 528-byte pitch; three 256-entry per-row arrays at EPI_META, above both the
// stage buffers and the store epilogue's 130 KiB staging of a pass
constexpr int EPI_G_ROW = 528;
constexpr int EPI_GS = 0;
// fp32 store epilogue of the 16 x 16 layout: a pass of 128 tile rows staged
// row-major, 260 floats per row (see EpiStore::tile16)
constexpr int EPI_F32_ROW = 260;
constexpr int EPI_ROWS_LDS = 128 * EPI_F32_ROW * 4;         // 133120
constexpr int EPI_META = EPI_ROWS_LDS > GEMM_LDS ? EPI_ROWS_LDS : GEMM_LDS;
constexpr int EPI_STAGE_LDS = EPI_META + 3 * 1024;          // 136192 B
static_assert(EPI_GS + 128 * EPI_G_ROW <= EPI_META, "G staging below the per-row arrays");
constexpr int BF16_KERNEL_LDS = EPI_STAGE_LDS > GEMM_LDS ? EPI_STAGE_LDS : GEMM_LDS;
constexpr int GEMM_THREADS = 256;

struct GemmShape {
  const void* A;
  int64_t lda;             // elements
  const void* B;
  int64_t ldb;
  int32_t M;               // rows of A (used when m_dev == nullptr)
  const int32_t* m_dev;    // rows of A read on the device
  int32_t N;               // rows of B (used when n_dev == nullptr)
  const int32_t* n_dev;    // rows of B read on the device
  int32_t K;               // multiple of 64 (used when k_dev == nullptr)
  const int32_t* k_dev;    // K read on the device, rounded up to a stage
  int32_t group_m;         // row-tiles per tile-order group
  // bf16 kernel only.  a_tiled / b_tiled: the operand is stored stage-tiled,
  // 1 in row-block order (tiled_index; lda / ldb = its padded K extent, a
  // multiple of 64), 2 in column-block order (tiled_cm_index; lda / ldb = its
  // padded row count, a multiple of 256).  a_trans: A is read transposed out
  // of a column-block tiled matrix whose rows are the product's K and whose
  // columns are the product's rows (lda = its padded row count), or (2) out of a
  // row-major one (lda = its row length; EpiGrad's launches only), whose rows from
  // stage a_tail_stage on are read from a_tail instead (a copy that is zero-padded
  // to a whole number of stages).
  int32_t a_tiled, b_tiled, a_trans;
  const void* a_tail;
  int32_t a_tail_stage;
  // bf16 kernel only: 1 makes the tile-order groups run over column tiles
  // (group_m column tiles deep, sweeping every row tile) instead of row tiles
  int32_t group_cols;
};

// Stage-tiled bf16 layout of a matrix with rows r and K-columns k (K padded to
// k_pad, a multiple of 64; rows padded to a multiple of 256): the 256 x 64
// block (r / 256, k / 64) is 32 KiB contiguous, row-major with 128-byte rows,
// and 16-byte chunk c of a block row rr sits at chunk c ^ ((rr >> 1) & 7), the
// LDS swizzle of the kernel below.  One K stage of a 256-row tile is then one
// contiguous 32 KiB block that copies into LDS unchanged (every copy moves
// 1 KiB of consecutive bytes), and a stage's rows share DRAM pages.
__host__ __device__ __forceinline__ int64_t tiled_index(int64_t r, int64_t k, int64_t k_pad) {
  return (((r >> 8) * (k_pad >> 6) + (k >> 6)) << 14) + ((r & 255) << 6) +
         ((((k & 63) >> 3) ^ ((r >> 1) & 7)) << 3) + (k & 7);
}

// The same blocks in column-block order: block (r / 256, k / 64) at index
// (k / 64) * (r_pad / 256) + r / 256.  This is the layout of the backward's
// logit gradient G (r = token, k = vocabulary entry).  dH reads it with K =
// vocabulary (the stages of a 256-token tile are r_pad / 256 blocks apart); dW
// reads it transposed with K = tokens (a 64-token stage lies 8 KiB further in
// each of the tile's four block columns).  Both are uniform strides.
__host__ __device__ __forceinline__ int64_t tiled_cm_index(int64_t r, int64_t k, int64_t r_pad) {
  return (((k >> 6) * (r_pad >> 8) + (r >> 8)) << 14) + ((r & 255) << 6) +
         ((((k & 63) >> 3) ^ ((r >> 1) & 7)) << 3) + (k & 7);
}

// Swizzle of a tile row: the chunk offset XORed into its 16-byte chunks.
__device__ __forceinline__ int row_swizzle(int r) { return (r >> 1) & 7; }

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

// ---------------------------------------------------------------------------
// The kernel: the tile, waves and swizzle described at the top, with a software
// pipeline tuned for one wave per SIMD:
//   * the per-lane global offsets of the stage copies are computed once per
//     tile (32-bit, relative to the tile's first row); each stage only moves a
//     scalar base, so a copy costs one instruction;
//   * every MFMA of a slice is paired with at most one LDS fragment read or
//     one stage copy (sched_barrier keeps that order), so the matrix pipe is
//     never left waiting behind a burst of memory instructions;
//   * the barriers are bare s_barrier: __syncthreads() would also wait for the
//     copies still in flight.
namespace bf16k {
constexpr int SK = 64;                        // k per stage
constexpr int ROW = SK * 2;                   // bytes per tile row per stage
constexpr int STAGE = (GBM + GBN) * ROW;      // 64 KiB
constexpr int HALF = GBM * ROW;               // one operand's part of a stage (32 KiB)
constexpr int NB = 2;                         // stage buffers
constexpr int RPI = 1024 / ROW;               // tile rows per copy instruction (8)
constexpr int IPW = 64 / RPI;                 // copy instructions per wave per operand (8)
constexpr int NCOPY = 2 * IPW;                // per wave per stage (16)
static_assert(NB * STAGE <= GEMM_LDS, "LDS");
static_assert((NB - 1) * HALF + 7 * 16 * ROW < 65536, "fragment offsets fit a DS immediate");
// Transposed A (a_trans).  The stage's A half holds 64 k-rows of the tile's 256
// rows of A, 512 bytes per k-row: the 64-byte window w (rows 32 w .. 32 w + 31)
// of k-row k sits at window w ^ (k & 3) (see loop16 for the reads).
constexpr int TR_KROW = GBM * 2;                // bytes per k-row (512)
static_assert((NB - 1) * HALF + 32 * TR_KROW + 4 * TR_KROW < 65536,
              "transposed fragment offsets fit a DS immediate");
// B rows first, then A rows
__device__ __forceinline__ constexpr int copy_order(int c) { return (c + IPW) % NCOPY; }
static_assert(NB == 2, "the vmcnt waits assume two stage buffers");

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// One 1 KiB global -> LDS copy (16 bytes per lane, LDS written contiguously
// from the wave-uniform byte address `lds`).  Issued as inline assembly on
// purpose: the compiler then does not see an in-flight LDS write, so it does
// not wait for the copy before later LDS reads of the other stage buffer
// (its alias analysis cannot tell the buffers apart and would serialise the
// prefetch).  The kernel orders copies and reads itself: vmcnt wait + barrier
// before a buffer is read, barrier before it is refilled.  Nothing else in
// these kernels uses M0.
template <uint32_t LDS_OFF>
__device__ __forceinline__ void copy16(const void* base, uint32_t off, uint32_t lds) {
  // scalar base + 32-bit per-lane offset: no 64-bit address arithmetic per copy;
  // M0 = lds + LDS_OFF in one scalar add (which writes SCC: undeclared, the compiler may
  // put a copy between the two halves of a 64-bit address add and lose the carry)
  asm volatile("s_add_u32 m0, %2, %3\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base),
               "s"(lds), "n"(LDS_OFF)
               : "memory", "scc");
}

// 16 x 16 x 32 loop: what rides along with MFMA slot q of a stage (slot
// q = 16 i + 2 j + kk is block (i, j), slice kk).  Copy c of the stage after
// next in slot CS c (even slots, spread over the stage: a burst of copies
// stalls issue when the memory pipeline is backed up, and the wave's matrix
// pipe waits with it).  The next stage's fragments are read in the odd slots
// of the second half only: a wait for the copies of the next stage and a
// barrier sit before slot 64, so a copy has until the middle of the stage
// after the one that issued it to land.  A rows 4..6 are replaced in place,
// two slots after row i's last MFMA; the other odd slots from 65 on carry the
// 16 B fragments, then A rows 0..3, then row 7 (into the spare set).
constexpr int MF16_NONE = -1, MF16_COPY = 0, MF16_BREAD = 16, MF16_AREAD = 32;
constexpr int MF16_MID = 64;   // slot of the mid-stage wait and barrier
__device__ __forceinline__ constexpr bool mf16_inplace_slot(int q) {
  return (q & 1) == 1 && q >= 81 && (q - 81) % 16 < 4 && (q - 81) / 16 < 3;
}
// rank of odd slot q >= 65 among those not taken by the in-place rows (-1: none)
__device__ __forceinline__ constexpr int mf16_late_rank(int q) {
  if ((q & 1) == 0 || q <= MF16_MID || mf16_inplace_slot(q)) return -1;
  int n = 0;
  for (int p = MF16_MID + 1; p < q; p += 2)
    if (!mf16_inplace_slot(p)) ++n;
  return n;
}
// SPLIT (transposed A, whose fragments take two LDS reads each): the B
// fragments come first, in the odd slots 33..63 behind a wait for the next
// stage's B copies (a stage issues B's copies before A's) at slot 32, so that
// the second half carries only A's reads.
constexpr int MF16_MID_B = 32;   // slot of the wait for B's copies (SPLIT)
// CS: slots between two copies (even, so that copies never share a slot with
// a fragment read)
template <int CS, bool SPLIT = false>
__device__ __forceinline__ constexpr int mf16_slot(int q) {
  static_assert(CS % 2 == 0 && 15 * CS < 128, "copy spacing");
  if (q < 16 * CS && q % CS == 0) return MF16_COPY + q / CS;
  if (mf16_inplace_slot(q)) return MF16_AREAD + 8 + 2 * ((q - 81) / 16) + ((q - 81) % 16) / 2;
  if (SPLIT) {
    if ((q & 1) == 1 && q > MF16_MID_B && q < MF16_MID) return MF16_BREAD + (q - MF16_MID_B) / 2;
    const int r = mf16_late_rank(q);
    if (r >= 0 && r < 8) return MF16_AREAD + r;
    if (r >= 8 && r < 10) return MF16_AREAD + 14 + (r - 8);
    return MF16_NONE;
  }
  const int r = mf16_late_rank(q);
  if (r >= 0 && r < 16) return MF16_BREAD + r;
  if (r >= 16 && r < 24) return MF16_AREAD + (r - 16);
  if (r >= 24 && r < 26) return MF16_AREAD + 14 + (r - 24);
  return MF16_NONE;
}
// copies a wave issues in a stage before slot q
template <int CS>
__device__ __forceinline__ constexpr int mf16_copies_before(int q) {
  return (q - 1) / CS + 1 < 16 ? (q - 1) / CS + 1 : 16;
}
// every fragment of the next stage is read exactly once, after the wait for
// its copies
template <int CS, bool SPLIT = false>
__device__ __forceinline__ constexpr bool mf16_schedule_ok() {
  int reads[32] = {}, copies[16] = {};
  for (int q = 0; q < 128; ++q) {
    const int op = mf16_slot<CS, SPLIT>(q);
    if (op >= MF16_COPY && op < MF16_COPY + 16) ++copies[op - MF16_COPY];
    if (op >= MF16_BREAD && op < MF16_AREAD + 16) {
      if (q <= (SPLIT && op < MF16_AREAD ? MF16_MID_B : MF16_MID)) return false;
      ++reads[op - MF16_BREAD];
    }
    // an in-place A row only after the last MFMA of that row
    if (op >= MF16_AREAD && op < MF16_AREAD + 14 && q < 16 * ((op - MF16_AREAD) >> 1) + 17) return false;
  }
  for (int n = 0; n < 32; ++n)
    if (reads[n] != 1) return false;
  for (int n = 0; n < 16; ++n)
    if (copies[n] != 1) return false;
  return true;
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
__device__ __forceinline__ bf16x4 read_tr(const uint8_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p));
}

}  // namespace bf16k

// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{})
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// The lane index computed afresh (from the exec mask, not from threadIdx.x), so
// that quantities derived from it are formed where they are used instead of
// being hoisted out of loops into spill slots
__device__ __forceinline__ int fresh_lane() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// Barrier that orders LDS accesses only: unlike __syncthreads() it does not
// wait for this wave's global stores to complete.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Up to two independent problems in one launch (the backward's dH and dW).
template <class Epi>
struct GemmBatch {
  GemmShape g[2];
  Epi e[2];
  int32_t n;          // number of problems
  int32_t cus;        // EpiGrad: compute units, and the most parts K of problem 0
  int32_t split_max;  // may be split into (see dh_split)
  int32_t* queue;     // 8 tile counters, then 8 finished-tile counters, zero at launch
  int32_t* queue_next;  // the next launch's: zeroed by this one
};

// Copy schedule of the 16 x 16 loop, per epilogue (measured on the 32B-shaped
// workload): MFMA slots between two stage copies, and whether odd rounds of tiles sweep K backwards (a round then starts
// on the operand chunks the previous round of its XCD read last: 2% faster for
// the long-K dH + dW tiles, while the forward and recompute gained nothing and
// their L2 hit rate dropped).
struct EpiLseCols;
struct EpiStore;
struct EpiGrad;
template <class Epi>
struct CopySched {
  static constexpr int spacing = 6;
  static constexpr bool serpentine = false;
  static constexpr bool round_sync = false;
};
template <>
struct CopySched<EpiLseCols> {
  static constexpr int spacing = 8;
  static constexpr bool serpentine = false;
  static constexpr bool round_sync = false;
};
template <>
struct CopySched<EpiStore> {
  static constexpr int spacing = 8;
  static constexpr bool serpentine = true;
  static constexpr bool round_sync = true;
};
// (with few tokens dW's tiles are short and the sync costs more than the panels it keeps
// in step: 1.80 -> 1.56 ms at 700 tokens, 6.44 -> 6.37 at 2871, 8.90 -> 8.92 at 6000)
template <>
struct CopySched<EpiGrad> : CopySched<EpiStore> {
  static constexpr bool round_sync = false;
};
constexpr int ROUND_SLACK = 2;   // tiles of the earlier rounds that may still run
constexpr int ROUND_SPIN = 32;   // polls of the finished-tile counter (~0.3 us apart)

// Tile scheduling.  Workgroups are dealt round-robin to the 8 XCDs, so
// workgroup b serves queue b % nq (nq = 8, fewer for a small grid).  A
// problem's tiles are ordered 8 row tiles deep, column-major inside a group,
// and cut into rounds of 32 nq tiles; queue q owns slots [32 q, 32 q + 32) of
// every round (the final partial round is dealt round-robin).  So at any time
// all XCDs work on the same few row panels (shared through the Infinity
// Cache) and each XCD on a compact 8 x 4 block of tiles (shared through its
// L2), while the workgroups of a queue take its tiles with an atomic counter
// and balance tiles of unequal length.  Problem 0's tiles come first.  A
// workgroup whose queue is empty takes the remaining tiles of the others.
__device__ __forceinline__ void grouped_tile(int L, int tiles_m, int tiles_n, int group_m,
                                             int& tm, int& tn) {
  const int width = group_m * tiles_n;
  const int grp = L / width;
  const int first = grp * group_m;
  const int gsz = min(tiles_m - first, group_m);
  const int rem = L - grp * width;
  tm = first + rem % gsz;
  tn = rem / gsz;
}

struct QueueShare {
  int full;     // tiles of this queue in the full rounds
  int len;      // all tiles of this queue
};

__device__ __forceinline__ QueueShare queue_share(int total, int q, int nq) {
  const int round = 32 * nq;
  const int rounds = total / round;
  const int tail = total - rounds * round;
  QueueShare s;
  s.full = 32 * rounds;
  s.len = s.full + (tail > q ? (tail - q + nq - 1) / nq : 0);
  return s;
}

// k-th tile of queue q -> tile index in the problem's order
__device__ __forceinline__ int queue_tile(int k, const QueueShare& s, int q, int nq) {
  if (k < s.full) return (k >> 5) * (32 * nq) + 32 * q + (k & 31);
  return (s.full / 32) * (32 * nq) + (k - s.full) * nq + q;
}

// Parts of dH's K extent (a vocabulary chunk of nv columns) in an EpiGrad launch.  With
// few action tokens dH has few tiles, each a chain over the whole chunk (2376 stages at
// V = 152064, 3 ms, whatever the chip could do beside it): parts of a third of a compute
// unit's share of the launch let the queues balance them against dW's tiles, whose
// epilogue (256 KiB written) costs about 12 stages.  dH + dW at V = 152064, d = 3584, 700
// tokens, dW accumulated: 3250 us in one piece (and 400 us of W^T before it), 1830 us in
// parts; V = 43776, d = 1088, 2122 tokens: 750 and 418 us.  2 or 5 instead of 3, or 24
// stages for the epilogue, are within the runs' noise.
constexpr int DH_PARTS = 3, DW_EPI_STAGES = 12, DH_MIN_STAGES = 16;
__host__ __device__ inline int dh_split(int n_act, int nv, int d, int cus, int most) {
  const int td = cdiv(d, GBN);
  const int64_t th = (int64_t)cdiv(n_act, GBM) * td, tw = (int64_t)cdiv(nv, GBM) * td;
  const int kh = 2 * cdiv(nv, 2 * bf16k::SK), kw = 2 * cdiv(n_act, 2 * bf16k::SK);
  const int64_t work = th * kh + tw * (kw + DW_EPI_STAGES);
  int64_t part = work / ((int64_t)cus * DH_PARTS);
  if (part < DH_MIN_STAGES) part = DH_MIN_STAGES;
  const int64_t parts = (kh + part - 1) / part;
  return (int)(parts < most ? parts : most);
}

// Stages run in pairs, so that which LDS buffer a stage reads and refills is known at
// compile time and every LDS address of the loop is a base register plus an immediate.
// ODD: K is an odd number of stages (a hidden size that is no multiple of 128; forward
// and recompute only): the first stage runs before the pairs, slice by slice, so that its
// second slice and the next stage's fragments are read under MFMAs.  The forward of 29440
// tokens on 157952 entries at 3 stages takes 3125 us, with the first stage's reads and the
// next's in the open 3387, in a loop on 32 x 32 blocks that chose its buffer at run time
// 3089; at 17 stages (d = 1088, V = 131001, 2122 tokens) 549 us, 560 and 582, and the
// recompute per 43776 columns 213 us against 218 (and 272, on a slower box where the second
// took 240).  ATR: a problem may read A transposed (GemmShape::a_trans).
template <class Epi, bool ATR, bool ODD = false>
__global__ void __launch_bounds__(GEMM_THREADS)
    __attribute__((amdgpu_waves_per_eu(1, 1))) gemm_bf16_kernel(GemmBatch<Epi> bat) {
  static_assert(!(ATR && ODD), "the products that read A transposed have whole stage pairs");
  // both products read A transposed, problem 0 (dH) out of row-major W with K split
  constexpr bool GRAD = std::is_same<Epi, EpiGrad>::value;
  using namespace bf16k;
  __shared__ __attribute__((aligned(16))) uint8_t smem[BF16_KERNEL_LDS];
  __shared__ int s_tile[2];   // claimed tile (-1: none left) and its queue
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  if (blockIdx.x == 0 && tid < 16) bat.queue_next[tid] = 0;
  const int nq = min(8, (int)gridDim.x);
  const int qi = blockIdx.x % nq;
  int Mp[2], Np[2], Kp[2], tmp[2], tnp[2], totp[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const GemmShape& gp = bat.g[p];
    // device-read sizes are the same in every lane; keep them scalar (see below)
    Mp[p] = __builtin_amdgcn_readfirstlane(gp.m_dev ? *gp.m_dev : gp.M);
    Np[p] = __builtin_amdgcn_readfirstlane(gp.n_dev ? *gp.n_dev : gp.N);
    constexpr int KR = 2 * SK;
    Kp[p] = __builtin_amdgcn_readfirstlane(gp.k_dev ? cdiv(*gp.k_dev, KR) * KR : gp.K);
    tmp[p] = cdiv(Mp[p], GBM);
    tnp[p] = cdiv(Np[p], GBN);
    totp[p] = (p < bat.n && Mp[p] > 0 && Np[p] > 0) ? tmp[p] * tnp[p] : 0;
  }
  int parts = 1;
  if constexpr (GRAD) {
    parts = __builtin_amdgcn_readfirstlane(
        dh_split(Np[0], Mp[1], Mp[0], bat.cus, bat.split_max));
    totp[0] *= parts;
  }

  // LDS holds the A halves of the two stage buffers first, then the B halves.
  // LDS byte address of the stage buffers
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)smem);

  // Tiles come from the queue of this workgroup's XCD until it runs dry, then
  // from the other queues in turn (cq: the first queue the next claim tries).
  // The XCDs do not run at one clock under the power limit (up to 9% apart on
  // one chip), so without this the slowest XCD's share sets the launch time.
  // A counter only grows, so a queue found empty stays empty, and a workgroup
  // leaves after one claim per queue has come back empty.
  int cq = qi, done_q = -1;
  for (;;) {
    if (wave == 0 && fresh_lane() == 0) {
      if (CopySched<Epi>::round_sync && done_q >= 0) atomicAdd(bat.queue + 8 + done_q, 1);
      int q = cq, k = -1;
      for (int n = 0; n < nq; ++n) {
        const int len = queue_share(totp[0], q, nq).len + queue_share(totp[1], q, nq).len;
        const int c = atomicAdd(bat.queue + q, 1);
        if (c < len) {
          k = c;
          break;
        }
        q = q + 1 == nq ? 0 : q + 1;
      }
      if constexpr (CopySched<Epi>::round_sync) {
        // a tile of a full round starts once all but a few tiles of the queue's
        // earlier rounds of the same problem have finished (bounded wait)
        if (k >= 0) {
          const QueueShare s0 = queue_share(totp[0], q, nq), s1 = queue_share(totp[1], q, nq);
          int target = 0;
          if (k < s0.full)
            target = k & ~31;
          else if (k >= s0.len && k - s0.len < s1.full)
            target = s0.full + ((k - s0.len) & ~31);
          target -= ROUND_SLACK;
          for (int it = 0; it < ROUND_SPIN && target > 0 &&
                           __hip_atomic_load(bat.queue + 8 + q, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT) < target;
               ++it)
            __builtin_amdgcn_s_sleep(8);
        }
      }
      s_tile[0] = k;
      s_tile[1] = q;
    }
    __syncthreads();
    // the same value in every lane: make it a scalar, otherwise every quantity
    // derived from it (loop bounds, the copies' LDS base in M0) is treated as
    // divergent and each copy becomes a waterfall loop
    const int t = __builtin_amdgcn_readfirstlane(s_tile[0]);
    if (t < 0) break;
    cq = __builtin_amdgcn_readfirstlane(s_tile[1]);
    done_q = cq;
    QueueShare sh[2];
    sh[0] = queue_share(totp[0], cq, nq);
    sh[1] = queue_share(totp[1], cq, nq);
    const int p = t < sh[0].len ? 0 : 1;
    const GemmShape g = p ? bat.g[1] : bat.g[0];
    const Epi epi = p ? bat.e[1] : bat.e[0];
    const int M = p ? Mp[1] : Mp[0];
    const int N = p ? Np[1] : Np[0];
    int nk = (p ? Kp[1] : Kp[0]) / SK;
    int tm, tn;
    int L = p ? queue_tile(t - sh[0].len, sh[1], cq, nq) : queue_tile(t, sh[0], cq, nq);
    int k0 = 0, at_part = 0;     // first stage of this item's part of K; the part
    if constexpr (GRAD) {
      if (p == 0) {
        const int tiles = tmp[0] * tnp[0];
        const int part = __builtin_amdgcn_readfirstlane(L / tiles);
        const int per = __builtin_amdgcn_readfirstlane(2 * cdiv(nk / 2, parts));
        L -= part * tiles;
        k0 = part * per;
        nk = max(0, min(per, nk - k0));
        at_part = part;
      }
    }
    if (g.group_cols)
      grouped_tile(L, p ? tnp[1] : tnp[0], p ? tmp[1] : tmp[0], g.group_m, tn, tm);
    else
      grouped_tile(L, p ? tmp[1] : tmp[0], p ? tnp[1] : tnp[0], g.group_m, tm, tn);
    const int64_t lda_b = g.lda * 2, ldb_b = g.ldb * 2;
    const int m0 = tm * GBM, n0 = tn * GBN;
    const bool atr = ATR && g.a_trans;
    // where a tile starts and how far a stage advances.  Row-major: the tile's
    // first row, 128 bytes.  Stage-tiled, row-block order: the tile's first
    // 32 KiB block, one block.  Column-block order: the same, ld / 256 blocks.
    // Transposed A: the tile's first block column, 64 k-rows of 128 bytes.
    auto place = [&](int tiled, int64_t ld, int64_t ld_b, int t, int r0, int64_t& off,
                     int64_t& ks) {
      if (tiled == 2) {
        off = (int64_t)t * HALF;
        ks = (ld >> 8) * HALF;
      } else if (tiled) {
        off = (int64_t)t * (ld >> 6) * HALF;
        ks = HALF;
      } else {
        off = (int64_t)r0 * ld_b;
        ks = ROW;
      }
    };
    int64_t a_off, a_ks, b_off, b_ks;
    const bool atr_rows = GRAD && g.a_trans == 2;
    if (atr_rows) {
      a_off = (int64_t)m0 * 2;
      a_ks = SK * lda_b;
    } else if (atr) {
      a_off = (int64_t)tm * 4 * (g.lda >> 8) * HALF;
      a_ks = SK * ROW;
    } else {
      place(g.a_tiled, g.lda, lda_b, tm, m0, a_off, a_ks);
    }
    place(g.b_tiled, g.ldb, ldb_b, tn, n0, b_off, b_ks);
    // serpentine K: odd rounds of the problem's tile order copy
    // the stages last to first
    // (an item of row-major W goes forwards: its tail is another buffer)
    if constexpr (GRAD) {
      a_off += k0 * a_ks;
      b_off += k0 * b_ks;
    }
    int64_t tail_delta = 0;      // from a tail stage's place in W to its copy
    if constexpr (GRAD) {
      if (atr_rows)
        tail_delta = ((const uint8_t*)g.a_tail - (int64_t)g.a_tail_stage * a_ks) -
                     (const uint8_t*)g.A;
    }
    if (CopySched<Epi>::serpentine && !atr_rows && ((L / (32 * nq)) & 1)) {
      a_off += (int64_t)(nk - 1) * a_ks;
      b_off += (int64_t)(nk - 1) * b_ks;
      a_ks = -a_ks;
      b_ks = -b_ks;
    }
    const uint8_t* a_base = (const uint8_t*)g.A + a_off;
    const uint8_t* b_base = (const uint8_t*)g.B + b_off;
    // copy q < 8 moves A rows [64 wave + 8 q, +8), q >= 8 the same rows of B;
    // lane i fetches chunk (i & 7) ^ swizzle(row) of row i / 8 (row-major: clamped
    // to the last valid row, those products are discarded by the epilogue;
    // stage-tiled: the chunk is already in place, the copy is 1 KiB contiguous)
    // (the lane index is re-read here: lane-derived constants hoisted out of the
    // tile loop end up in spill slots, and every reload is a round trip to memory
    // that the streaming operands have evicted from the caches)
    const int ln = fresh_lane();
    uint32_t offa[IPW], offb[IPW];
#pragma unroll
    for (int b = 0; b < IPW; ++b) {
      const int row = wave * 64 + b * RPI + (ln >> 3);
      const int ch = ((ln & 7) ^ row_swizzle(row)) << 4;
      offa[b] = g.a_tiled ? (uint32_t)(row * ROW + (ln & 7) * 16)
                          : (uint32_t)(min(row, M - 1 - m0) * lda_b + ch);
      offb[b] = g.b_tiled ? (uint32_t)(row * ROW + (ln & 7) * 16)
                          : (uint32_t)(min(row, N - 1 - n0) * ldb_b + ch);
    }
    if (atr) {
      // transposed A: copy b of a wave fills k-rows 16 wave + 2 b, + 1 (the
      // same LDS bytes as above); lane i lands in physical 16-byte chunk i & 31
      // of its k-row, which holds rows 32 w + 8 (i & 3) .. + 7 of window
      // w = ((i & 31) >> 2) ^ (k-row & 3).  In the source those rows are a
      // 16-byte chunk of k-row (token) 64 s + kr of block column w / 2.
#pragma unroll
      for (int b = 0; b < IPW; ++b) {
        const int kr = wave * 16 + 2 * b + (ln >> 5);
        const int p = ln & 31;
        const int w = (p >> 2) ^ (kr & 3);
        // the 32-byte halves of a window are swapped when bit 3 of the k-row is
        // set, so lane i holds rows 32 w + 16 hf + 8 (i & 1) .. + 7
        const int c16 = (w & 1) * 4 + ((((p >> 1) & 1) ^ ((kr >> 3) & 1)) << 1) + (p & 1);
        // (lda <= 2^23 rows: at most 3 * 2^15 blocks of 32 KiB, within 32 bits)
        offa[b] = (uint32_t)((w >> 1) * (uint32_t)((g.lda >> 8) * HALF) + kr * ROW +
                             ((c16 ^ ((kr >> 1) & 7)) << 4));
        // row-major: k-row kr of the stage, the same columns (those past the last
        // are clamped; the epilogue drops their rows)
        if constexpr (GRAD) {
          if (atr_rows)
            offa[b] = (uint32_t)(kr * (uint32_t)lda_b) +
                      (uint32_t)(min((w >> 1) * 64 + c16 * 8, M - 8 - m0) * 2);
        }
      }
    }

    // (the LDS address is formed from scalars only, so it stays in SGPRs)
    // copy Q of stage s into stage buffer BUF: the LDS address is a scalar base plus
    // a constant of the copy site
    const uint32_t lds_w = lds0 + (uint32_t)(wave * 64 * ROW);
    auto copy = [&](int s, auto q_c, auto buf_c) {
      constexpr int Q = decltype(q_c)::value;
      constexpr int BUF = decltype(buf_c)::value;
      constexpr uint32_t b = Q % IPW;
      constexpr uint32_t fixed = (uint32_t)BUF * HALF;
      if constexpr (Q < IPW && GRAD)
        copy16<fixed + b * RPI * ROW>(
            a_base + s * a_ks + (atr_rows && k0 + s >= g.a_tail_stage ? tail_delta : 0), offa[b],
            lds_w);
      else if constexpr (Q < IPW)
        copy16<fixed + b * RPI * ROW>(a_base + s * a_ks, offa[b], lds_w);
      else
        copy16<NB * HALF + fixed + b * RPI * ROW>(b_base + s * b_ks, offb[b], lds_w);
    };
    // q is a constant at every call site once the loops are unrolled
    auto copy_q = [&](int s, int q, auto buf_c) {
      static_assert(NCOPY == 16, "one case per copy");
      switch (q) {
        case 0: copy(s, std::integral_constant<int, 0>{}, buf_c); break;
        case 1: copy(s, std::integral_constant<int, 1>{}, buf_c); break;
        case 2: copy(s, std::integral_constant<int, 2>{}, buf_c); break;
        case 3: copy(s, std::integral_constant<int, 3>{}, buf_c); break;
        case 4: copy(s, std::integral_constant<int, 4>{}, buf_c); break;
        case 5: copy(s, std::integral_constant<int, 5>{}, buf_c); break;
        case 6: copy(s, std::integral_constant<int, 6>{}, buf_c); break;
        case 7: copy(s, std::integral_constant<int, 7>{}, buf_c); break;
        case 8: copy(s, std::integral_constant<int, 8>{}, buf_c); break;
        case 9: copy(s, std::integral_constant<int, 9>{}, buf_c); break;
        case 10: copy(s, std::integral_constant<int, 10>{}, buf_c); break;
        case 11: copy(s, std::integral_constant<int, 11>{}, buf_c); break;
        case 12: copy(s, std::integral_constant<int, 12>{}, buf_c); break;
        case 13: copy(s, std::integral_constant<int, 13>{}, buf_c); break;
        case 14: copy(s, std::integral_constant<int, 14>{}, buf_c); break;
        case 15: copy(s, std::integral_constant<int, 15>{}, buf_c); break;
        default: break;
      }
    };

    {
      // 16 x 16 x 32 loop.  acc[i][j] is the 16 x 16 block (i, j) of the wave's
      // 128 x 128 sub-tile: lane l holds column 16 j + (l & 15), rows 16 i +
      // 4 (l >> 4) .. + 3 (Epi::SWAP: row 16 i + (l & 15), columns 16 j +
      // 4 (l >> 4) .. + 3).  A stage is two 32-deep slices; the MFMAs of a stage
      // run rows i = 0..7, columns j = 0..7, and the two slices of block (i, j)
      // back to back (the second accumulates onto the first).  The stage's
      // fragments are in registers before it starts: fa[i][kk] (A, replaced in
      // place by the next stage's row i once row i's MFMAs are issued; row 7 of
      // odd stages lives in fa7) and fb[P][j][kk] (B, two sets by stage parity).
      // Two barriers per stage: at its start every wave is done reading this
      // stage's buffer, which the copies of the stage after next then refill;
      // before slot 64 the next stage has landed, and its fragments are read
      // in the second half.
      // one accumulator set and one epilogue for both operand modes (TR: A
      // read transposed); only the main loop is instantiated per mode
      f32x4 acc[8][8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      auto loop16 = [&](auto tr_c) {
      constexpr bool TR = decltype(tr_c)::value;
      {
        // lane l reads row l & 15 of each 16-row block, 16-byte chunk
        // 4 kk + (l >> 4) of slice kk; the row swizzle depends on the row within
        // the block only, so a block is an immediate offset of 2 KiB.
        // Transposed A: the stage's A half holds 64 k-rows of 512 bytes; the
        // 64-byte window w (rows 32 w .. + 31) of k-row k sits at w ^ (k & 3)
        // and its 32-byte halves are swapped when bit 3 of k is set.  Block i
        // of slice kk is two transposing reads (ds_read_b64_tr_b16): in 16-lane
        // group g, lane s supplies k-row 32 kk + 8 g + (s >> 2) (+ 4 for the
        // second read) and rows 4 (s & 3) .. + 3 of the block, and lane s
        // receives row s of those 4 k-rows.  A 32-lane half touches 8 k-rows,
        // spread over 4 bank windows by (k & 3) and 2 halves by bit 3 of k.
        const int l16 = fresh_lane();
        const int fr = l16 & 15;
        int ra16[2], rb16[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int chk = ((kk * 4 + (l16 >> 4)) ^ row_swizzle(fr)) << 4;
          ra16[kk] = (wm * 128 + fr) * ROW + chk;
          rb16[kk] = NB * HALF + (wn * 128 + fr) * ROW + chk;
        }
        // block i's transposed read: ta16 ^ (64 (i >> 1) + 32 (i & 1)) (the
        // window and half bits of ta16 hold the lane's XOR pattern; the block's
        // bits go in by one XOR per read instead of eight live addresses)
        int ta16 = 0;
        if constexpr (TR) {
          const int g = l16 >> 4, q4 = (l16 >> 2) & 3;
          ta16 = (8 * g + q4) * TR_KROW + 4 * wm * 64 + (q4 << 6) + ((g & 1) << 5) + 8 * (l16 & 3);
        }
        auto rd_a = [&](int i, int kk, int buf) {
          if constexpr (TR) {
            const uint8_t* p = smem + (ta16 ^ ((i >> 1) << 6 | (i & 1) << 5)) + buf * HALF +
                               kk * 32 * TR_KROW;
            bf16x8 v;
            v.lo = read_tr(p);
            v.hi = read_tr(p + 4 * TR_KROW);
            return v;
          } else {
            return *(const bf16x8*)(smem + ra16[kk] + buf * HALF + i * 16 * ROW);
          }
        };
        auto rd_b = [&](int j, int kk, int buf) {
          return *(const bf16x8*)(smem + rb16[kk] + buf * HALF + j * 16 * ROW);
        };
        using P0 = std::integral_constant<int, 0>;
        using P1 = std::integral_constant<int, 1>;
        bf16x8 fa[8][2], fa7[2], fb[2][8][2];
        if constexpr (ODD) {
          // The first stage, through buffer 1, slice by slice: under the first slice's MFMAs
          // the second slice's fragments are read, under the second's the fragments of the
          // next stage, which went through buffer 0, and the copies of the one after it (a
          // single stage is copied in place of either and read for nothing).
#pragma unroll
          for (int q = 0; q < NCOPY; ++q) copy_q(0, q, P1{});
          const int more = nk > 1 ? 1 : 0;
          a_base += more * a_ks;
          b_base += more * b_ks;
          nk -= 1;
#pragma unroll
          for (int q = 0; q < NCOPY; ++q) copy_q(0, q, P0{});
          wait_vmcnt<NCOPY>();
          __builtin_amdgcn_s_barrier();
          bf16x8 a[2][8], b[2][8];
          a[0][0] = rd_a(0, 0, 1);
          static_for<8>([&](auto j_c) { b[0][j_c.value] = rd_b(j_c.value, 0, 1); });
          static_for<7>([&](auto i_c) { a[0][i_c.value + 1] = rd_a(i_c.value + 1, 0, 1); });
          __builtin_amdgcn_sched_barrier(0);
          static_for<128>([&](auto q_c) {
            constexpr int kk = q_c.value >> 6, q = q_c.value & 63, i = q >> 3, j = q & 7;
            if constexpr (kk == 1 && q == 0) {
              // buffer 1 is in registers, buffer 0 has landed, in every wave
              asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
              __builtin_amdgcn_sched_barrier(0);
            }
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                Epi::SWAP ? b[kk][j] : a[kk][i], Epi::SWAP ? a[kk][i] : b[kk][j], acc[i][j], 0, 0, 0);
            if constexpr (kk == 0 && q % 4 == 1) {
              constexpr int n = q >> 2;
              if constexpr (n < 8)
                b[1][n] = rd_b(n, 1, 1);
              else
                a[1][n - 8] = rd_a(n - 8, 1, 1);
            }
            if constexpr (kk == 1 && q % 4 == 0) copy_q(more, copy_order(q >> 2), P1{});
            if constexpr (kk == 1 && q % 2 == 1) {
              constexpr int n = q >> 1, r = (n >> 1) & 7, k = n & 1;
              if constexpr (n < 16)
                fb[0][r][k] = rd_b(r, k, 0);
              else
                fa[r][k] = rd_a(r, k, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
          });
          if (nk == 0) return;
        } else {
          // stages 0 and 1 whole (stage 1 in the loop's copy order, which the
          // first stage's waits assume)
#pragma unroll
          for (int q = 0; q < NCOPY; ++q) copy_q(0, q, P0{});
#pragma unroll
          for (int q = 0; q < NCOPY; ++q) copy_q(1, copy_order(q), P1{});
          wait_vmcnt<NCOPY>();        // stage 0 landed (stage pairs: nk >= 2)
          __builtin_amdgcn_s_barrier();
          // stage 0's fragments
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
              fa[i][kk] = rd_a(i, kk, 0);
              fb[0][i][kk] = rd_b(i, kk, 0);
            }
        }
        // Every stage runs the same code (one register assignment for the whole
        // loop): the last two stages copy the last stage again into the buffer
        // they free (its data is in registers already, nothing reads it again),
        // and the last stage reads stale fragments of a stage that does not
        // exist; both stay within the operands and the LDS.
        auto stage16 = [&](int kt, auto par_c) {
          constexpr int P = decltype(par_c)::value;            // kt % 2
          using PC = std::integral_constant<int, P>;
          constexpr int CS = CopySched<Epi>::spacing;
          constexpr bool SPLIT = TR;
          static_assert(mf16_schedule_ok<CS, SPLIT>(), "16 x 16 slot schedule");
          const int kc = min(kt + 2, nk - 1);                  // stage to copy
          // every wave has read its fragments of this stage's buffer, which the
          // copies below refill
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
          // (every index below is a compile-time constant, so that the
          // fragment and accumulator arrays stay in registers)
          static_for<128>([&](auto q_c) {
            constexpr int q = decltype(q_c)::value;
            constexpr int i = q >> 4, j = (q >> 1) & 7, kk = q & 1;
            constexpr int op = mf16_slot<CS, SPLIT>(q);
            if constexpr (SPLIT && q == MF16_MID_B) {
              // stage kt + 1's B half landed: this wave's first 8 copies of the
              // previous stage, before its 8 A copies and this stage's copies
              wait_vmcnt<8 + mf16_copies_before<CS>(MF16_MID_B)>();
              __builtin_amdgcn_s_barrier();
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (q == MF16_MID) {
              // stage kt + 1 landed: this wave's copies of it are all but the
              // ones issued so far in this stage, then the other waves'
              wait_vmcnt<mf16_copies_before<CS>(MF16_MID)>();
              __builtin_amdgcn_s_barrier();
              __builtin_amdgcn_sched_barrier(0);
            }
            // (operands swapped: each block transposed, the same sums)
            const bf16x8 a = i == 7 && P == 1 ? fa7[kk] : fa[i][kk], b = fb[P][j][kk];
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Epi::SWAP ? b : a,
                                                                Epi::SWAP ? a : b, acc[i][j], 0, 0, 0);
            if constexpr (op >= MF16_COPY && op < MF16_COPY + 16) {
              constexpr int c = op - MF16_COPY;
              copy_q(kc, copy_order(c), PC{});
            } else if constexpr (op >= MF16_BREAD && op < MF16_BREAD + 16) {
              constexpr int n = op - MF16_BREAD;
              fb[P ^ 1][n >> 1][n & 1] = rd_b(n >> 1, n & 1, P ^ 1);
            } else if constexpr (op >= MF16_AREAD && op < MF16_AREAD + 16) {
              constexpr int n = op - MF16_AREAD, ia = n >> 1, ka = n & 1;
              // the next stage's row 7 goes to the set this stage does not use
              if constexpr (ia == 7 && P == 0)
                fa7[ka] = rd_a(7, ka, P ^ 1);
              else
                fa[ia][ka] = rd_a(ia, ka, P ^ 1);
            }
            __builtin_amdgcn_sched_barrier(0);
          });
        };
        for (int kt = 0; kt < nk; kt += 2) {
          stage16(kt, P0{});
          stage16(kt + 1, P1{});
        }
      }
      };
      if (nk > 0) {
        if constexpr (GRAD) {
          loop16(std::true_type{});
        } else if constexpr (ATR) {
          if (atr)
            loop16(std::true_type{});
          else
            loop16(std::false_type{});
        } else {
          loop16(std::false_type{});
        }
      }
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __syncthreads();
      {
        const int lane_e = fresh_lane();
        if constexpr (GRAD) {
          Epi ep = epi;
          ep.to_part(at_part);
          ep.tile16(acc, m0, n0, tn, M, N, smem, wm, wn, lane_e, wave * 64 + lane_e);
        } else
        epi.tile16(acc, m0, n0, tn, M, N, smem, wm, wn, lane_e, wave * 64 + lane_e);
      }
    }
    // the next tile's copies overwrite what the epilogue staged in LDS; its stores stay
    // in flight under the next tile's claim and first copies
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// Epilogues.  Each receives the finished accumulators of one tile.

// Forward partial log-sum-exp on a transposed tile: rows are vocabulary
// entries (A = W), columns are compacted tokens (B = H_act).  Lane l holds 8 token
// columns (16 j + (l & 15)) and 32 vocabulary rows of each (16 i + 4 (l >> 4) + r);
// the other 96 rows of the wave's half sit in lanes l ^ 16, l ^ 32, l ^ 48.  So the
// reduction over the tile's vocabulary is lane-local except for two exchanges and one
// merge of the two row waves through LDS: (max, sum exp) per token and vocabulary
// tile, and the target logit.
struct EpiLseCols {
  static constexpr bool SWAP = false;
  const int32_t* y;      // [tokens] target id of each compacted row
  f32x2* part;           // [tiles_v][ld_part] (max, sum exp) per token and vocabulary tile
  int64_t ld_part;
  float* zy;             // [tokens] logit of the target token
  float scale;           // 1 / temperature

  template <bool FULL>
  __device__ __forceinline__ void cols16(const f32x4 (&acc)[8][8], int m0, int n0, int M,
                                         const int* sy, f32x2* red, int wm, int wn,
                                         int lane) const {
    const float k1 = scale * 1.44269504088896341f;
    const int g4 = 4 * (lane >> 4);
    const int lim = M - m0 - wm * 128 - g4;     // rows 16 i + r >= lim are beyond the vocabulary
    auto live = [&](int i, int r) { return FULL || 16 * i + r < lim; };
    float mx[8], sm[8], mk[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      mx[j] = -INFINITY;
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[j] = fmaxf(mx[j], live(i, r) ? acc[i][j][r] : -INFINITY);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 16));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      mx[j] = fmaxf(mx[j], __shfl_xor(mx[j], 32));
      mk[j] = mx[j] != -INFINITY ? -mx[j] * k1 : 0.0f;
      sm[j] = 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float e = __builtin_amdgcn_exp2f(fmaf(acc[i][j][r], k1, mk[j]));
          sm[j] += live(i, r) ? e : 0.0f;
        }
#pragma unroll
    for (int j = 0; j < 8; ++j) sm[j] += __shfl_xor(sm[j], 16);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sm[j] += __shfl_xor(sm[j], 32);
      const int c = wn * 128 + j * 16 + (lane & 15);
      if (lane < 16) red[wm * GBN + c] = f32x2{mx[j] * scale, sm[j]};
      // target logit: local row o of the target, held here iff 0 <= o < 128 and
      // bits 2..3 of o equal lane / 16; the register is picked by a select tree
      // over o's block (bits 4..6) and row (bits 0..1)
      const int o = sy[c] - wm * 128;
      float v[32];
#pragma unroll
      for (int q = 0; q < 32; ++q) v[q] = acc[q >> 2][j][q & 3];
      const int idx = ((o >> 4) << 2) | (o & 3);
#pragma unroll
      for (int b = 0, w = 16; b < 5; ++b, w >>= 1) {
        const bool hi = (idx >> b) & 1;
#pragma unroll
        for (int q = 0; q < w; ++q) v[q] = hi ? v[2 * q + 1] : v[2 * q];
      }
      if ((unsigned)o < 128u && (o & 12) == g4) zy[n0 + c] = v[0] * scale;
    }
  }

  __device__ __forceinline__ void tile16(f32x4 (&acc)[8][8], int m0, int n0, int tn, int M,
                                         int N, uint8_t* smem, int wm, int wn, int lane,
                                         int tid) const {
    int* sy = (int*)smem;
    f32x2* red = (f32x2*)(smem + 1024);
    sy[tid] = (n0 + tid < N) ? y[n0 + tid] - m0 : -1;
    __syncthreads();
    if (m0 + GBM <= M)
      cols16<true>(acc, m0, n0, M, sy, red, wm, wn, lane);
    else
      cols16<false>(acc, m0, n0, M, sy, red, wm, wn, lane);
    __syncthreads();
    const int col = n0 + tid;
    if (col < N) {
      const f32x2 a = red[tid], b = red[GBN + tid];
      const float m = fmaxf(a.x, b.x);
      // only an empty sum is left out (its max may be -inf): a NaN or infinite logit makes
      // its half's sum NaN, and with it the token's lse
      const float s = (a.y == 0.0f ? 0.0f : a.y * __expf(a.x - m)) +
                      (b.y == 0.0f ? 0.0f : b.y * __expf(b.x - m));
      part[(int64_t)(m0 / GBM) * ld_part + col] = f32x2{m, s};
    }
  }
};

// Backward recompute: G = gs_n * (1[v == y_n] - exp(z - lse_n)), rounded to bf16.
// Rows >= M and columns >= N are written as 0 (they pad the K extent of the next
// products).  The tile is finished in two passes of 128 rows (accumulator blocks
// i = 2h and 2h + 1 of both wave rows).  A pass stages its G rows row-major in LDS,
// then they leave as full 128-byte lines of G's column-block stage-tiled layout (dW
// reads the same G transposed, so no transposed copy is written).  The exponent is
// evaluated in base 2 with the scale folded in:
// exp(z - lse) = exp2(acc * scale * log2(e) - lse * log2(e)).
struct EpiLogitGrad {
  static constexpr bool SWAP = true;
  const int32_t* y;
  const float* lse;
  const float* gs;       // dL/dlogp / temperature, per compacted row
  __bf16* G;             // column-block stage-tiled
  int64_t ldg;           // G's padded row count
  float scale;
  int32_t col0;          // vocabulary index of this chunk's column 0

  // per tile row: target column relative to the tile, -lse * log2(e) (-inf on
  // dead rows, so their exponentials are 0 and G is +0 there), dL/dlogp
  __device__ __forceinline__ void meta(int m0, int n0, int M, uint8_t* smem, int tid) const {
    const bool live = m0 + tid < M;
    ((int*)(smem + EPI_META))[tid] = live ? y[m0 + tid] - col0 - n0 : -1;
    ((float*)(smem + EPI_META + 1024))[tid] =
        live ? -lse[m0 + tid] * 1.44269504088896341f : -INFINITY;
    ((float*)(smem + EPI_META + 2048))[tid] = live ? gs[m0 + tid] : 0.0f;
  }

  // Swapped accumulators: pass h takes blocks i = 4 h .. 4 h + 3 of both wave rows; lane l holds
  // columns 16 j + 4 (l >> 4) .. + 3 of row 16 i + (l & 15): its token's values are
  // read once per block row and four entries of G leave as one 8-byte LDS write (four
  // 2-byte writes before: 11830 -> 11750 us per 76032-column chunk at d = 5120, 22793
  // tokens).
  template <bool FULL, int h>
  __device__ __forceinline__ void stage_pass16(const f32x4 (&acc)[8][8], int n0, int N,
                                               uint8_t* smem, int wm, int wn, int lane) const {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const float k1 = scale * 1.44269504088896341f;
    const int c0 = wn * 128 + 4 * (lane >> 4);                  // tile column of j = q = 0
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      const int i = 4 * h + ii;
      const int rt = wm * 128 + 16 * i + (lane & 15);           // tile row
      const int oy = *(const int*)(smem + EPI_META + 4 * rt) - c0;
      const float rn = *(const float*)(smem + EPI_META + 1024 + 4 * rt);
      const float rg = *(const float*)(smem + EPI_META + 2048 + 4 * rt);
      uint8_t* gs_at = smem + EPI_GS + (wm * 64 + 16 * ii + (lane & 15)) * EPI_G_ROW + c0 * 2;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float gv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float p = __builtin_amdgcn_exp2f(fmaf(acc[i][j][q], k1, rn));
          gv[q] = fmaf(-rg, p, 0.0f);
          if constexpr (!FULL) gv[q] = n0 + c0 + 16 * j + q < N ? gv[q] : 0.0f;
        }
        *(u32x2*)(gs_at + 32 * j) =
            u32x2{__builtin_bit_cast(uint32_t,
                                     __builtin_convertvector(f32x2{gv[0], gv[1]}, bf16x2_t)),
                  __builtin_bit_cast(uint32_t,
                                     __builtin_convertvector(f32x2{gv[2], gv[3]}, bf16x2_t))};
      }
      // a token whose target lies in this lane's columns (rare: one tile in V / 256 per
      // token) gets that entry again, instead of a compare and a select per entry: 11780
      // -> 11700 us per chunk at d = 5120, 22793 tokens, 3205 -> 3157 at 2871
      const bool held = (unsigned)oy < 128u && (oy & 12) == 0;
      if (__any(held)) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (oy == 16 * j + q) {
              const float p = __builtin_amdgcn_exp2f(fmaf(acc[i][j][q], k1, rn));
              *(uint16_t*)(gs_at + 32 * j + 2 * q) = f32_to_bf16_bits(fmaf(-rg, p, rg));
            }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  __device__ __forceinline__ void tile16(f32x4 (&acc)[8][8], int m0, int n0, int tn, int M,
                                         int N, uint8_t* smem, int wm, int wn, int lane,
                                         int tid) const {
    meta(m0, n0, M, smem, tid);
    __syncthreads();
    const bool full = n0 + GBN <= N;
    if (full)
      stage_pass16<true, 0>(acc, n0, N, smem, wm, wn, lane);
    else
      stage_pass16<false, 0>(acc, n0, N, smem, wm, wn, lane);
    __syncthreads();
    copy_out<0>(m0, n0, smem, tid);
    __syncthreads();
    if (full)
      stage_pass16<true, 1>(acc, n0, N, smem, wm, wn, lane);
    else
      stage_pass16<false, 1>(acc, n0, N, smem, wm, wn, lane);
    __syncthreads();
    copy_out<1>(m0, n0, smem, tid);
  }

  // G: 128 rows of 512 bytes staged in LDS by pass h; pass rows 0..63 are tile
  // rows 64h + r, rows 64..127 are tile rows 128 + 64h + (r - 64).
  // Column-block stage-tiled addresses: m0 and n0 are multiples of 256, so a
  // thread's block and chunk are fixed and only the row within the block
  // changes from store to store.  The loop reads all its LDS chunks before
  // the first store, so the reads overlap.  The stores are non-temporal: G is
  // read back only by the next launch, and a round of tiles writes as much G
  // as an XCD's L2 holds, which would otherwise evict the operand panels the
  // running tiles share.
  template <int h>
  __device__ __forceinline__ void copy_out(int m0, int n0, uint8_t* smem, int tid) const {
    const int c16 = tid & 31;
    __bf16* base = G + (((int64_t)((n0 >> 6) + (c16 >> 3)) * (ldg >> 8) + (m0 >> 8)) << 14);
    u32x4 v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k)
      v[k] = *(const u32x4*)(smem + EPI_GS + ((tid >> 5) + 8 * k) * EPI_G_ROW + c16 * 16);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int row = (tid >> 5) + 8 * k;
      const int trow = 64 * h + (row < 64 ? row : row + 64);
      __builtin_nontemporal_store(
          v[k], (u32x4*)(base + ((trow << 6) + (((c16 & 7) ^ ((trow >> 1) & 7)) << 3))));
    }
  }
};

// Plain fp32 store (or accumulate) of the tile, rows optionally remapped.  Swapped
// accumulators: lane l's f32x4 of block (i, j) is columns 16 j + 4 (l >> 4) .. + 3 of row
// 16 i + (l & 15).  Pass h stages blocks i = 4 h .. 4 h + 3 of both wave rows row-major,
// one 16-byte LDS write per accumulator (260 floats a row: the 16 rows of a write are 16
// distinct bank groups), and a row leaves as one 16-byte access per lane, 1 KiB
// contiguous.  With few action tokens dW's tiles are mostly this (12 K stages at 700
// tokens): what bounds them is how many bytes a workgroup has in flight, so 16 rows a
// wave are read ahead when accumulating (64 KiB per compute unit).
struct EpiStore {
  static constexpr bool SWAP = true;
  float* out;
  int64_t ldo;
  const int32_t* row_map;   // nullable: output row of each tile row
  int32_t accumulate;

  __device__ __forceinline__ void tile16(f32x4 (&acc)[8][8], int m0, int n0, int tn, int M, int N,
                                         uint8_t* smem, int wm, int wn, int lane, int tid) const {
    int* sr = (int*)(smem + EPI_META);
    if (row_map) {
      sr[tid] = (m0 + tid < M) ? row_map[m0 + tid] : 0;
      lds_barrier();
    }
    if (accumulate)
      out16<true>(acc, m0, n0, M, N, (float*)smem, sr, wm, wn, lane);
    else
      out16<false>(acc, m0, n0, M, N, (float*)smem, sr, wm, wn, lane);
  }

  template <bool ACC>
  __device__ __forceinline__ void out16(const f32x4 (&acc)[8][8], int m0, int n0, int M, int N,
                                        float* st, const int* sr, int wm, int wn, int lane) const {
    const int wave = wm * 2 + wn;
    // (a column past the last is one of the row's padding: N is a multiple of 64, or a token
    // count in rows of a multiple of 256, of which the reduce takes the first N columns)
    const bool col_ok = n0 + 4 * lane < N;
    // Staged row pr of pass h is tile row 64 h + pr (pr < 64) or 64 h + pr + 64; wave w
    // handles rows w, w + 4, ... in two batches of 16, the first below 64.  Lane k forms
    // output row k of a batch; a row's address is then a scalar, two multiplies and an add
    // (with a 64-bit address and an exec mask formed per row and lane, the 32 stores of a
    // pass took 7.7k cycles; dH + dW at V = 152064, d = 3584, 700 tokens 1.60 -> 1.47 ms).
    // The scalars are read outside the branches on col_ok: inside, lanes 1..15 may be off
    // (257 tokens leave one column of the last tile).
    const uint32_t ld_b = (uint32_t)(ldo * 4);
    struct Rows {
      uint32_t of[16];
    };
    auto first = [&](int h, int b) { return 64 * h + 128 * b + wave; };     // tile row
    auto batch = [&](int h, int b) {
      const int tr = first(h, b) + 4 * (lane & 15);
      const int rows = row_map ? sr[tr] : m0 + tr;
      Rows r;
#pragma unroll
      for (int k = 0; k < 16; ++k) r.of[k] = __builtin_amdgcn_readlane(rows, k);
      return r;
    };
    auto at = [&](uint32_t row) {
      return (f32x4*)((char*)(out + n0) + (uint64_t)row * ld_b + (uint32_t)(16 * lane));
    };
    f32x4 old[16];
    // (vmcnt counts stores too and in order: the next rows are read before a batch is
    // stored, also across the passes, so that no read waits for a store)
    auto read = [&](int h, int b) {
      const Rows r = batch(h, b);
      if (col_ok) {
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (m0 + first(h, b) + 4 * k < M) old[k] = *at(r.of[k]);
      }
    };
    if constexpr (ACC) read(0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h) lds_barrier();                        // pass 0's rows have been read
#pragma unroll
      for (int ii = 0; ii < 4; ++ii)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          *(f32x4*)(st + (wm * 64 + 16 * ii + (lane & 15)) * EPI_F32_ROW + wn * 128 + 16 * j +
                    4 * (lane >> 4)) = acc[4 * h + ii][j];
      lds_barrier();                               // rows staged
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        f32x4 v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          v[k] = *(const f32x4*)(st + (wave + 64 * b + 4 * k) * EPI_F32_ROW + 4 * lane);
          if constexpr (ACC) v[k] += old[k];
        }
        if constexpr (ACC) {
          if (h == 0 || b == 0) read(h + b, 1 - b);
        }
        const Rows r = batch(h, b);
        if (col_ok) {
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (m0 + first(h, b) + 4 * k < M) *at(r.of[k]) = v[k];
        }
      }
    }
  }
};

// The two products of a launch for few action tokens: dW as above; dH computed
// transposed (rows: hidden units, columns: compacted tokens), so that W is the operand
// read transposed, as it lies in memory, and no W^T is built.  Its items write their
// part of K to parts [part][rows][ldo]; the reduce kernel adds the parts in order and
// turns them into dH's rows.
struct EpiGrad : EpiStore {
  int64_t part_stride;

  __device__ __forceinline__ void to_part(int part) { out += part * part_stride; }
};

}  // namespace agrl
