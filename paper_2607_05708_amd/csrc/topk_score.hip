// General selection path: any dtype, any d <= 8192, any row stride and
// alignment, k <= 64, optional full probability output.  It serves what the
// fused matrix-core kernel does not take (fp32 embeddings, k > 32, d not a
// multiple of 32, full probabilities) and calls too small to fill it.
//
// Two kernels.  A score kernel forms s_ij = <q_i, b_j> on the matrix cores
// (fp32 inputs on the fp32 MFMA, bf16 inputs on the bf16 MFMA, fp32
// accumulation) and writes a block of scores [queries, rows]; a select kernel
// folds each query's scores into its softmax state and sorted top-k list.
// The block is at most 96 MiB (kScoreBlock), so that it stays in the last
// level cache between the two, and larger problems run block by block, the
// select kernel resuming each list.  Where a query has one split, its last
// select writes the final results (and its full probability row), else the
// merge kernels combine the splits.
//
// A thread-per-row fp32 kernel did this before (3.8 TFLOP/s whatever the
// type, every query re-reading the bank).  64 fp32 queries against 65,536 x
// 768 rows, k = 16: 1,706 -> 75 us (scores 66 us, 98 TFLOP/s); 200 bf16
// queries against 100,003 x 1024, k = 64: 12.2 -> 0.136 ms (430 TFLOP/s, bound
// by the 8 TB/s that the 128 x 128 tiles draw from L2); 16 fp32 queries against
// 1,024 x 256 with full probabilities: 20.9 -> 11.3 us, half of it the launches
// and the caller's own time.
//
// Dense-only relevance of the paper's Section 5.5 applied to LLMSelect of
// Algorithm 1.
#include "device_common.h"
#include "launch.h"
#include "select.h"

namespace memattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// acc += A B over the 16 bytes of K that every lane holds of its row: one
// 32x32x16 bf16 MFMA, or four 32x32x2 fp32 ones.  Lane l's 16 bytes belong to
// row l % 32 of the block; lanes 0-31 and 32-63 hold different 16-byte
// pieces of the rows.  Which piece a half holds is free, as long as A and B
// agree: the sum runs over all of them.
__device__ __forceinline__ void mma16(f32x16& acc, u32x4 a, u32x4 b, uint16_t) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0,
                                                0, 0);
}
__device__ __forceinline__ void mma16(f32x16& acc, u32x4 a, u32x4 b, float) {
  const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[e], fb[e], acc, 0, 0, 0);
}

// 16 bytes of a row from element k on, elements at or past d as zeros.  Rows
// need only their elements' own alignment.
template <typename T>
__device__ __forceinline__ u32x4 load16(const T* row, int k, int d, bool whole) {
  constexpr int E = 16 / sizeof(T);
  u32x4 v = {0u, 0u, 0u, 0u};
  if (whole || k + E <= d) {
    __builtin_memcpy(&v, row + k, 16);
  } else if (k < d) {
    T e[E];
#pragma unroll
    for (int i = 0; i < E; ++i) e[i] = k + i < d ? row[k + i] : T(0);
    __builtin_memcpy(&v, e, 16);
  }
  return v;
}

// The same without a branch around the load, so that the compiler's wait
// counts stay exact: a piece that would pass the row's end is read from its
// last 16 bytes (d >= 16 / sizeof(T)) and shifted into place by fix_tail.
template <typename T>
__device__ __forceinline__ u32x4 load16_within(const T* row, int k, int d) {
  u32x4 v;
  __builtin_memcpy(&v, row + min(k, d - static_cast<int>(16 / sizeof(T))), 16);
  return v;
}
template <typename T>
__device__ __forceinline__ u32x4 fix_tail(u32x4 v, int k, int d) {
  const int over = k + static_cast<int>(16 / sizeof(T)) - d;  // elements past the row
  if (over <= 0) return v;
  if (k >= d) return u32x4{0u, 0u, 0u, 0u};
  const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v);
  return __builtin_bit_cast(u32x4, x >> (over * static_cast<int>(sizeof(T)) * 8));
}

struct ScoreArgs {
  const void* bank;      // first row of the block
  int64_t bank_stride;
  int64_t rows;          // rows of the block
  const void* queries;   // first query of the block
  int64_t q_stride;
  int64_t nq;            // queries of the block
  int32_t d;
  float* out;            // [nq, ld]
  int64_t ld;
};

// Tiled score kernel: 4 waves, QW x RW of them (queries x rows), each scoring
// QB query blocks against RB row blocks of 32.  Each stage holds 128 bytes of
// K of every row in LDS (two buffers), loaded into registers two stages
// ahead; the 16-byte pieces of a row are XOR swizzled by the row so that
// fragment reads (32 consecutive rows, one piece) and the staging writes
// (whole rows) are free of bank conflicts.  On fp32 rows this runs at the
// rate of a library matrix product of the same shape (512 x 131,072 x 768: 931
// against 902 us), both at about 2.1 GHz with the matrix cores 80-86 % busy;
// tiles of other sizes and more waves per SIMD change nothing.
constexpr int kStageBytes = 128;
// STREAM: bank rows, 16-byte aligned, are loaded non-temporally (a stage takes
// whole lines, which no other workgroup reads).  It pays for tiles of 32
// queries over long rows of a bank that the last level cache cannot hold: one
// query over 1M x 1024 rows 367 -> 350 us, 1,024 over 256 tables of them 474 ->
// 463 us; shorter rows lose (1M x 256: 233 -> 245 us), and so do 400 MB banks,
// parts of which stay cached from call to call (193 -> 224 us).
constexpr int64_t kStreamRowBytes = 1536;
constexpr int64_t kStreamBankBytes = int64_t{1} << 30;
bool streams(int64_t rows, int64_t row_bytes) {
  return row_bytes >= kStreamRowBytes && rows * row_bytes >= kStreamBankBytes;
}

template <typename T, int QB, int QW, int RB, int RW, bool STREAM = false>
struct ScoreTile {
  static_assert(QW * RW == 4, "four waves");
  static constexpr int kTileQ = 32 * QB * QW;
  static constexpr int kTileR = 32 * RB * RW;
  static constexpr int kLines = kTileR + kTileQ;  // staged rows: bank rows, then query rows
  static constexpr int kLoads = kLines / 32;      // 16-byte pieces per thread and stage: piece
  static constexpr int kRowLoads = kTileR / 32;   // tid % 8 of staged rows tid / 8 + 32 i
  static constexpr int E = 16 / sizeof(T);            // elements per piece
  static constexpr int KE = kStageBytes / sizeof(T);  // elements per stage

  // acc += the tile's scores, src[i] being the thread's staged rows.  Every
  // thread of the workgroup calls it; it may be called again at once (past
  // its last barrier only unused fragments are read).
  static __device__ __forceinline__ void run(u32x4 (&st)[2][kLines * 8], const T* const (&src)[kLoads], int d,
                                             f32x16 (&acc)[QB][RB]) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int c = tid & 7;
    const int n_st = (d + KE - 1) / KE;
    // (stages past the last read the rows' last bytes again and are not used)
    auto load = [&](int s, u32x4 (&v)[kLoads]) {
      const int k = s * KE + c * E;
#pragma unroll
      for (int i = 0; i < kRowLoads; ++i) {
        if constexpr (STREAM)
          v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src[i] + min(k, d - E)));
        else
          v[i] = load16_within<T>(src[i], k, d);
      }
#pragma unroll
      for (int i = kRowLoads; i < kLoads; ++i) v[i] = load16_within<T>(src[i], k, d);
    };
    const int wr = c ^ ((tid >> 4) & 7);  // (32 rows on, the swizzle is the same)
    // (the last stage's tail is mended in LDS: a use of the registers there
    // would make the compiler copy them in every stage, and wait for them)
    auto store = [&](int s, int buf, const u32x4 (&v)[kLoads]) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) st[buf][((tid >> 3) + 32 * i) * 8 + wr] = v[i];
      if ((s + 1) * KE > d && s < n_st) {
#pragma unroll 1
        for (int i = 0; i < kLoads; ++i) {
          u32x4* at = &st[buf][((tid >> 3) + 32 * i) * 8 + wr];
          *at = fix_tail<T>(*at, s * KE + c * E, d);
        }
      }
    };
    const int frow = lane & 31;
    const int part = lane >> 5;
    const int wq = wave % QW;                // the wave's query group
    const int wrow = (wave / QW) * 32 * RB;  // and its first row of the tile
    struct Frag {
      u32x4 q[QB], r[RB];
    };
    auto read = [&](int buf, int step, Frag& f) {
      const int p = (2 * step + part) ^ ((frow >> 1) & 7);
#pragma unroll
      for (int x = 0; x < QB; ++x) f.q[x] = st[buf][(kTileR + (wq * QB + x) * 32 + frow) * 8 + p];
#pragma unroll
      for (int y = 0; y < RB; ++y) f.r[y] = st[buf][(wrow + y * 32 + frow) * 8 + p];
    };
    auto mma = [&](const Frag& f) {
      __builtin_amdgcn_sched_barrier(0);  // the reads before it are issued before it
#pragma unroll
      for (int x = 0; x < QB; ++x)
#pragma unroll
        for (int y = 0; y < RB; ++y) mma16(acc[x][y], f.q[x], f.r[y], T{});
      __builtin_amdgcn_sched_barrier(0);
    };
    // Stage s is computed from buffer s % 2 while the loads of stages s + 2
    // and s + 3 are in flight.  Its staging writes of stage s + 1 go first
    // (that buffer was last read in stage s - 1, before the barrier in it),
    // each step's fragments are read ahead of the MFMAs of the step before,
    // and the barrier stands before the last step, whose MFMAs cover the
    // reads of the next stage's first fragments.
    Frag f0, f1;
    auto stage = [&](int s, int buf, u32x4 (&v)[kLoads]) {
      store(s + 1, buf ^ 1, v);
      load(s + 3, v);
      read(buf, 1, f1);
      mma(f0);
      read(buf, 2, f0);
      mma(f1);
      read(buf, 3, f1);
      mma(f0);
      __syncthreads();
      read(buf ^ 1, 0, f0);
      mma(f1);
    };
    u32x4 va[kLoads], vb[kLoads];
    load(0, va);
    load(1, vb);
    store(0, 0, va);
    load(2, va);
    __syncthreads();
    read(0, 0, f0);
    // (no exit inside the loop: the wait counts at its head stay exact; the
    // last stage writes a buffer that is not read)
    int s = 0;
    for (; s + 1 < n_st; s += 2) {
      stage(s, 0, vb);
      stage(s + 1, 1, va);
    }
    if (s < n_st) stage(s, 0, vb);
  }
};

template <typename T, int QB, int QW, int RB, int RW, bool STREAM>
__global__ __launch_bounds__(256) void score_tile_kernel(ScoreArgs a) {
  using S = ScoreTile<T, QB, QW, RB, RW, STREAM>;
  __shared__ u32x4 st[2][S::kLines * 8];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // Workgroups b, b + 8, ... run on one XCD: the query tiles of one row tile
  // are neighbours there and share its rows through that XCD's L2.
  const int q_tiles = static_cast<int>((a.nq + S::kTileQ - 1) / S::kTileQ);
  const int i8 = blockIdx.x >> 3;
  const int64_t r0 = (static_cast<int64_t>(i8 / q_tiles) * 8 + (blockIdx.x & 7)) * S::kTileR;
  const int64_t q0 = static_cast<int64_t>(i8 % q_tiles) * S::kTileQ;
  if (r0 >= a.rows) return;
  // rows past the block repeat its last one (their scores are not written)
  const T* src[S::kLoads];
#pragma unroll
  for (int i = 0; i < S::kLoads; ++i) {
    const int line = (tid >> 3) + 32 * i;
    src[i] = i < S::kRowLoads
                 ? static_cast<const T*>(a.bank) + min(r0 + line, a.rows - 1) * a.bank_stride
                 : static_cast<const T*>(a.queries) + min(q0 + line - S::kTileR, a.nq - 1) * a.q_stride;
  }
  f32x16 acc[QB][RB];
#pragma unroll
  for (int x = 0; x < QB; ++x)
#pragma unroll
    for (int y = 0; y < RB; ++y) acc[x][y] = f32x16{};
  S::run(st, src, a.d, acc);
  // accumulator lane: row lane % 32 of its block, queries 8 (r / 4) + 4 (lane / 32) + r % 4
#pragma unroll
  for (int y = 0; y < RB; ++y) {
    const int64_t row = r0 + (wave / QW) * 32 * RB + y * 32 + (lane & 31);
    if (row < a.rows) {
#pragma unroll
      for (int x = 0; x < QB; ++x)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t q = q0 + (wave % QW * QB + x) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (q < a.nq) a.out[q * a.ld + row] = acc[x][y][r];
        }
    }
  }
}

// Small problems: 32 queries against 32 rows per workgroup, its four waves
// taking every fourth 128-byte block of K each and adding their sums up in
// LDS.  Fragments come straight from global memory (lane: 64 contiguous
// bytes of its row), all of a block's loads in flight, so a call costs little
// more than one trip to memory, and four times as many workgroups share it
// as with the tiles above.
template <typename T>
__global__ __launch_bounds__(256) void score_small_kernel(ScoreArgs a) {
  constexpr int E = 16 / sizeof(T);
  constexpr int KE = kStageBytes / sizeof(T);
  __shared__ float red[4][1024];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int q_tiles = static_cast<int>((a.nq + 31) / 32);
  const int64_t r0 = static_cast<int64_t>(blockIdx.x / q_tiles) * 32;
  const int64_t q0 = static_cast<int64_t>(blockIdx.x % q_tiles) * 32;
  const int frow = lane & 31;
  const int part = lane >> 5;
  const T* br = static_cast<const T*>(a.bank) + min(r0 + frow, a.rows - 1) * a.bank_stride;
  const T* qr = static_cast<const T*>(a.queries) + min(q0 + frow, a.nq - 1) * a.q_stride;
  const int d = a.d;
  const int n_blk = (d + KE - 1) / KE;
  const int n_whole = d / KE;
  f32x16 acc = {};
  auto load = [&](int b, u32x4 (&x)[4], u32x4 (&y)[4]) {
    if (b >= n_blk) return;
    const int k = b * KE + part * 4 * E;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = load16<T>(qr, k + i * E, d, b < n_whole);
      y[i] = load16<T>(br, k + i * E, d, b < n_whole);
    }
  };
  auto compute = [&](int b, const u32x4 (&x)[4], const u32x4 (&y)[4]) {
    if (b >= n_blk) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) mma16(acc, x[i], y[i], T{});
  };
  u32x4 xa[4], ya[4], xb[4], yb[4];
  load(wave, xa, ya);
  for (int b = wave; b < n_blk; b += 8) {
    load(b + 4, xb, yb);
    compute(b, xa, ya);
    load(b + 8, xa, ya);
    compute(b + 4, xb, yb);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][r * 64 + lane] = acc[r];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = wave * 4 + j;
    const int64_t q = q0 + 8 * (r >> 2) + 4 * part + (r & 3);
    const float s = (red[0][r * 64 + lane] + red[1][r * 64 + lane]) + (red[2][r * 64 + lane] + red[3][r * 64 + lane]);
    if (q < a.nq && r0 + frow < a.rows) a.out[q * a.ld + r0 + frow] = s;
  }
}

// ---------------------------------------------------------------- selection

struct SelectArgs {
  float* scores;          // [nq, ld]: column c is bank row c0 + c
  int64_t ld;
  int64_t q0;             // first query of the block
  int64_t c0, c1;         // bank rows of the block
  int64_t rows_per_split;
  int n_splits;           // splits of a query (all of them)
  int split0;             // first split that meets the block
  int block_splits;       // and how many do
  int k, kcap;
  float c2;
  int64_t self_base;
  const int32_t* row_ns;
  const int32_t* key_ns;
  int64_t part_q0;        // first query of the partials: 0, or with one split the block's
  uint64_t* part_keys;    // [queries, n_splits, kcap]
  float2* part_ms;        // [queries, n_splits]: max, sum
  float* part_lo;         // [queries, n_splits]: what the sum's rounding left
  int full;               // the scores are the caller's full probability rows
  int64_t n;
  // final results (one split per query, last block), else idx is NULL
  int32_t* idx;
  float* score;
  float* prob;
  float* lse;
};

// Folds a step's scores into the thread's softmax state (-inf adds nothing)
// and returns the largest order key among them; bit j of `out`: value j is no
// candidate.
template <int PER>
__device__ __forceinline__ uint32_t fold_step(const float (&v)[PER], uint32_t out, float c2, float& m_run,
                                              double& s_run) {
  float best = v[0];
#pragma unroll
  for (int j = 1; j < PER; ++j) best = fmaxf(best, v[j]);
  const float mx = fmaxf(m_run, best * c2);
  double part = 0.0;
  if (mx != -INFINITY) {
#pragma unroll
    for (int j = 0; j < PER; ++j) part += static_cast<double>(fast_exp2(v[j] * c2 - mx));
    s_run = s_run * static_cast<double>(fast_exp2(m_run - mx)) + part;
    m_run = mx;
  }
  uint32_t top = f2ord(best);
  // (not so where a value is no candidate or a NaN, which fmaxf passes by but
  // the sum above does not)
  if (out != 0 || !(best > -INFINITY) || !(part < INFINITY)) {
    top = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) top = max(top, ((out >> j) & 1u) ? 0u : f2ord(v[j]));
  }
  return top;
}

// One workgroup per (query, split): the split's scores of this block, 4,096
// a step.  A split that an earlier block began resumes from its list and
// softmax state (the sum in two floats, so that nothing of the double is
// lost between blocks).  PER: scores per thread and step, 16 but for banks of
// at most 1,024 (4) or 2,048 rows (8), whose one step has no more (16 queries
// x 1,024 rows: 9.7 -> 6.7 us, the reductions by DPP included).
template <int PER>
__global__ __launch_bounds__(kSelThreads, 4) void select_kernel(SelectArgs a) {
  constexpr int kStep = kSelThreads * PER;
  __shared__ SelectLds L;
  const int tid = threadIdx.x;
  const int64_t ql = blockIdx.x / a.block_splits;
  const int64_t q = a.q0 + ql;
  const int split = a.split0 + static_cast<int>(blockIdx.x % a.block_splits);
  const int64_t slot = (q - a.part_q0) * a.n_splits + split;
  const int64_t s0 = static_cast<int64_t>(split) * a.rows_per_split;
  const int64_t row0 = max(s0, a.c0);
  const int64_t row1 = min(min(s0 + a.rows_per_split, a.n), a.c1);
  const bool resume = s0 < a.c0;
  float* row = a.scores + ql * a.ld;  // column c: bank row c0 + c
  const int64_t self_row = a.self_base >= 0 ? a.self_base + q : -1;
  const int32_t my_ns = a.row_ns ? a.key_ns[q] : 0;
  int cur = 0;
  if (tid < kMaxK) L.list[0][tid] = (resume && tid < a.k) ? a.part_keys[slot * a.kcap + tid] : 0;
  float m_run = -INFINITY;
  double s_run = 0.0;
  if (resume && tid == 0) {
    const float2 ms = a.part_ms[slot];
    m_run = ms.x;
    s_run = static_cast<double>(ms.y) + static_cast<double>(a.part_lo[slot]);
  }
  __syncthreads();
  // value j of a step is its element 1024 (j / 4) + 4 tid + j % 4: four
  // 16-byte loads where the rows allow it
  const bool vec = (reinterpret_cast<uintptr_t>(a.scores) % 16 | a.ld % 4 | (row0 - a.c0) % 4) == 0;
  auto at = [&](int j) { return 1024 * (j >> 2) + 4 * tid + (j & 3); };
  float v[PER];  // a step's scores, -inf where no candidate
  uint32_t out = 0;  // bit j: value j is no candidate
  for (int64_t base = row0; base < row1; base += kStep) {
    const int left = static_cast<int>(min(row1 - base, static_cast<int64_t>(kStep)));
    float* src = row + (base - a.c0);
    if (vec && left == kStep) {
#pragma unroll
      for (int j = 0; j < PER; j += 4) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(src + at(j));
        v[j] = x.x, v[j + 1] = x.y, v[j + 2] = x.z, v[j + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < PER; ++j) v[j] = at(j) < left ? src[at(j)] : -INFINITY;
    }
    out = 0;
    if (left < kStep || a.row_ns || (self_row >= base && self_row < base + left)) {  // (uniform)
      const int64_t self = self_row - base;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int e = at(j);
        bool cand = e < left && e != self;
        if (a.row_ns && cand) cand = my_ns >= 0 && a.row_ns[base + e] == my_ns;
        if (!cand) {
          // a row outside the candidates gets probability 0 in the full output
          if (a.full && e < left) src[e] = -INFINITY;
          out |= 1u << j;
          v[j] = -INFINITY;
        }
      }
    }
    auto hi = [&](int j) { return ((out >> j) & 1u) ? 0u : f2ord(v[j]); };
    const uint32_t low = 0xFFFFFFFFu - static_cast<uint32_t>(base) - 4 * tid;
    const uint32_t top = fold_step(v, out, a.c2, m_run, s_run);
    cur = select_step<true, PER>(
        L, hi,
        [&](int j) {
          const uint32_t h = hi(j);
          return h ? (static_cast<uint64_t>(h) << 32) | (low - (1024 * (j >> 2) + (j & 3))) : uint64_t{0};
        },
        top, a.k, cur);
  }

  const SoftmaxSum all = block_softmax(L, m_run, s_run);
  if (a.idx == nullptr) {
    if (tid < a.kcap) a.part_keys[slot * a.kcap + tid] = L.list[cur][tid];
    if (tid == 0) {
      const float hi = static_cast<float>(all.sum);
      a.part_ms[slot] = make_float2(all.max, hi);
      a.part_lo[slot] = static_cast<float>(all.sum - static_cast<double>(hi));
    }
    return;
  }
  const float lse2 = all.max + static_cast<float>(log2(all.sum));
  if (tid < a.k) write_selected(L.list[cur][tid], a.c2, lse2, q * a.k + tid, a.idx, a.score, a.prob);
  if (tid == 0 && a.lse) a.lse[q] = lse2 * kLn2;
  if (!a.full) return;
  const bool none = lse2 == -INFINITY;
  const bool one = row1 - row0 <= kStep;  // the only step's scores are still here
  for (int64_t base = row0; base < row1; base += kStep) {
    const int left = static_cast<int>(min(row1 - base, static_cast<int64_t>(kStep)));
    float* src = row + (base - a.c0);
    const bool wide = vec && left == kStep;
    if (!one) {
      // (the writes of -inf above were this thread's own)
      if (wide) {
#pragma unroll
        for (int j = 0; j < PER; j += 4) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(src + at(j));
          v[j] = x.x, v[j + 1] = x.y, v[j + 2] = x.z, v[j + 3] = x.w;
        }
      } else {
#pragma unroll
        for (int j = 0; j < PER; ++j) v[j] = at(j) < left ? src[at(j)] : 0.f;
      }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) v[j] = none ? 0.f : fast_exp2(v[j] * a.c2 - lse2);
    if (wide) {
#pragma unroll
      for (int j = 0; j < PER; j += 4)
        *reinterpret_cast<f32x4*>(src + at(j)) = f32x4{v[j], v[j + 1], v[j + 2], v[j + 3]};
    } else {
#pragma unroll
      for (int j = 0; j < PER; ++j)
        if (at(j) < left) src[at(j)] = v[j];
    }
  }
}

// ---------------------------------------------------------------- chunk tables

// The same two steps over chunk tables: every query against the rows its
// own namespace's table lists.  One workgroup plans: the tiles of each
// namespace (32 of its queries x 128 of its rows), where its scores go (a row
// of the table's length per query), and whether it is done this way at all:
// the scores have to fit their room and no table may be so long that one
// workgroup's selection from it would be waited for.  Otherwise the fused
// grouped pass does it; the losing side's launches return at once.
//
// The fused pass takes a whole table per workgroup: with 256 tables of 5 to
// 11 of its 512-row tiles the longest set the time, and lists that start
// empty take most of their first tile's time.  1,024 queries over 256 tables
// of about 3,700 x 1024 rows, k = 5: 578 us, k = 32: 690 + 65 us (sample);
// this way 380 us of scores (5.0 TB/s of bank rows) and 24-26 us of selection.
constexpr int kTablePlanThreads = 1024;
constexpr int kTablePlanPer = static_cast<int>(kTableMaxNs) / kTablePlanThreads;

__device__ __forceinline__ int64_t table_first(const TableArgs& a, int u) {
  return min(max(static_cast<int64_t>(a.ns_off[static_cast<int64_t>(u) * a.off_step]), int64_t{0}), a.n_entries);
}
// (offsets are clamped so a malformed table cannot send reads past it)
__device__ __forceinline__ int table_length(const TableArgs& a, int u) {
  const int64_t lo = table_first(a, u);
  const int64_t hi = min(static_cast<int64_t>(a.ns_off[static_cast<int64_t>(u) * a.off_step + 1]), a.n_entries);
  return static_cast<int>(max(hi - lo, int64_t{0}));
}

__global__ __launch_bounds__(kTablePlanThreads) void table_plan_kernel(TableArgs a) {
  __shared__ int64_t red[2][kTablePlanThreads / 64];
  __shared__ int longest;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  if (a.gate != nullptr && *a.gate == 0) {  // (uniform) no tables
    if (tid == 0) {
      a.flag[0] = a.flag[1] = 0;
      a.tile_off[a.n_ns] = 0;
    }
    return;
  }
  if (tid == 0) longest = 0;
  __syncthreads();
  int64_t tiles[kTablePlanPer], room[kTablePlanPer], sum_t = 0, sum_r = 0;
#pragma unroll
  for (int j = 0; j < kTablePlanPer; ++j) {
    const int u = tid * kTablePlanPer + j;
    tiles[j] = room[j] = 0;
    if (u < a.n_ns) {
      const int64_t nq = a.q_off[u + 1] - a.q_off[u];
      if (nq > 0) {
        const int len = table_length(a, u);
        tiles[j] = (nq + 31) / 32 * ((len + 127) / 128);
        room[j] = nq * ((len + 3) / 4 * 4);
        atomicMax(&longest, len);
      }
    }
    sum_t += tiles[j];
    sum_r += room[j];
  }
  int64_t inc_t = sum_t, inc_r = sum_r;
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t t = __shfl_up(inc_t, off), r = __shfl_up(inc_r, off);
    if (lane >= off) {
      inc_t += t;
      inc_r += r;
    }
  }
  if (lane == 63) {
    red[0][wave] = inc_t;
    red[1][wave] = inc_r;
  }
  __syncthreads();
  int64_t at_t = inc_t - sum_t, at_r = inc_r - sum_r, all_t = 0, all_r = 0;
  for (int w = 0; w < kTablePlanThreads / 64; ++w) {
    at_t += w < wave ? red[0][w] : 0;
    at_r += w < wave ? red[1][w] : 0;
    all_t += red[0][w];
    all_r += red[1][w];
  }
  const bool use = all_r <= a.max_scores && longest <= kTableMaxRows;
#pragma unroll
  for (int j = 0; j < kTablePlanPer; ++j) {
    const int u = tid * kTablePlanPer + j;
    if (u < a.n_ns) {
      a.tile_off[u] = use ? static_cast<int32_t>(at_t) : 0;
      a.score_off[u] = at_r;
    }
    at_t += tiles[j];
    at_r += room[j];
  }
  if (tid == 0) {
    a.flag[0] = use ? 1 : 0;
    a.flag[1] = use ? 0 : 1;
    a.tile_off[a.n_ns] = use ? static_cast<int32_t>(all_t) : 0;
    if (use) a.item_off[a.n_ns] = 0;  // no work item for the fused pass
  }
}

// The last of off[0 .. n) that is <= x (off ascends from 0, n <= 4096): two
// loads per lane instead of a chain of twelve.
template <typename I>
__device__ __forceinline__ int find_last(const I* off, int n, I x) {
  const int lane = threadIdx.x & 63;
  const I a = 64 * lane < n ? off[64 * lane] : x + 1;
  const int hi = __builtin_popcountll(__ballot(a <= x)) - 1;
  const I b = 64 * hi + lane < n ? off[64 * hi + lane] : x + 1;
  return __builtin_amdgcn_readfirstlane(64 * hi + __builtin_popcountll(__ballot(b <= x)) - 1);
}

template <bool STREAM>
__global__ __launch_bounds__(256) void score_tables_kernel(TableArgs a) {
  using S = ScoreTile<uint16_t, 1, 1, 1, 4, STREAM>;
  __shared__ u32x4 st[2][S::kLines * 8];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int total = a.tile_off[a.n_ns];
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int u = find_last(a.tile_off, a.n_ns, item);
    const int local = item - a.tile_off[u];
    const int len = table_length(a, u);
    const int row_tiles = (len + 127) / 128;
    const int r0 = local % row_tiles * 128;
    const int q0 = local / row_tiles * 32;
    const int64_t q_first = a.q_off[u];
    const int nq = static_cast<int>(a.q_off[u + 1] - q_first);
    const int32_t* rows = a.chunks + table_first(a, u);
    const uint16_t* src[S::kLoads];
#pragma unroll
    for (int i = 0; i < S::kLoads; ++i) {
      const int line = (tid >> 3) + 32 * i;
      if (i < S::kRowLoads) {
        // an entry outside the bank reads row 0 (and is no candidate)
        const int32_t r = rows[min(r0 + line, len - 1)];
        src[i] = a.bank + (r >= 0 && r < a.n ? r : 0) * a.bank_stride;
      } else {
        src[i] = a.queries + a.perm[q_first + min(q0 + line - S::kTileR, nq - 1)] * a.q_stride;
      }
    }
    f32x16 acc[1][1] = {{f32x16{}}};
    S::run(st, src, a.d, acc);
    const int row = r0 + wave * 32 + (lane & 31);
    const int64_t pitch = (len + 3) / 4 * 4;
    float* out = a.scores + a.score_off[u] + row;
    if (row < len) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int q = q0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (q < nq) out[q * pitch] = acc[0][0][r];
      }
    }
  }
}

// One workgroup per query: the selection over its table's scores.
__global__ __launch_bounds__(kSelThreads, 4) void select_tables_kernel(TableArgs a) {
  if (a.flag[0] == 0) return;
  __shared__ SelectLds L;
  const int tid = threadIdx.x;
  const int64_t q = blockIdx.x;
  const int32_t pos = a.q_pos[q];
  int cur = 0;
  if (tid < kMaxK) L.list[0][tid] = 0;
  float m_run = -INFINITY;
  double s_run = 0.0;
  __syncthreads();
  if (pos >= 0) {  // (uniform: a query without a namespace has no candidates)
    const int u = find_last(a.q_off, a.n_ns, static_cast<int64_t>(pos));
    const int len = table_length(a, u);
    const int32_t* rows = a.chunks + table_first(a, u);
    const float* row = a.scores + a.score_off[u] + (pos - a.q_off[u]) * static_cast<int64_t>((len + 3) / 4 * 4);
    auto at = [&](int j) { return 1024 * (j >> 2) + 4 * tid + (j & 3); };
    for (int base = 0; base < len; base += kSelStep) {
      const int left = min(len - base, kSelStep);
      float v[kSelPer];
      int32_t id[kSelPer];
#pragma unroll
      for (int j = 0; j < kSelPer; j += 4) {
        const int e = at(j);
        // (a row's room is a multiple of 4 scores)
        const f32x4 x = e < left ? *reinterpret_cast<const f32x4*>(row + base + e) : f32x4{};
        v[j] = x.x, v[j + 1] = x.y, v[j + 2] = x.z, v[j + 3] = x.w;
        if (e + 4 <= left) {
          __builtin_memcpy(&id[j], rows + base + e, 16);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) id[j + i] = e + i < left ? rows[base + e + i] : -1;
        }
      }
      uint32_t out = 0;  // an entry outside the bank is no candidate
#pragma unroll
      for (int j = 0; j < kSelPer; ++j) {
        if (id[j] < 0 || id[j] >= a.n) {
          out |= 1u << j;
          v[j] = -INFINITY;
        }
      }
      const uint32_t top = fold_step(v, out, a.c2, m_run, s_run);
      auto hi = [&](int j) { return ((out >> j) & 1u) ? 0u : f2ord(v[j]); };
      // (ids ascend within a table)
      cur = select_step<true, kSelPer>(
          L, hi,
          [&](int j) {
            const uint32_t h = hi(j);
            return h ? (static_cast<uint64_t>(h) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(id[j])) : uint64_t{0};
          },
          top, a.k, cur);
    }
  }
  const SoftmaxSum all = block_softmax(L, m_run, s_run);
  const float lse2 = all.max + static_cast<float>(log2(all.sum));
  if (tid < a.k) write_selected(L.list[cur][tid], a.c2, lse2, q * a.k + tid, a.idx, a.score, a.prob);
  if (tid == 0 && a.lse) a.lse[q] = lse2 * kLn2;
}

// Queries per tile: 128, 64 or 32, no more than the queries need, and fewer
// while that leaves fewer tiles than CUs.  128 queries x 30,000 rows (235 tiles
// of 128 queries, so the small kernel before, against 470 of 64), d = 64, 256
// and 1,024: 30 -> 29, 37 -> 29 and 86 -> 34 us; 200 x 6,000 (tiles of 32): 21
// -> 20, 24 -> 21 and 42 -> 27 us; fp32, d = 1,024: 183 -> 88 and 79 -> 54 us.
// (Tiles sum a row in one chain, as the fused pass does, the small kernel in
// four: relative error against 64 bits at d = 1,024 3.6e-7 and 3.3e-7 in bf16,
// 5.2e-7 and 3.4e-7 in fp32.)
int64_t tiles_of(int64_t nq, int64_t n, int64_t tq) { return (n + 127) / 128 * ((nq + tq - 1) / tq); }
int64_t tile_queries(int64_t nq, int64_t n) {
  int64_t tq = nq <= 32 ? 32 : (nq <= 64 ? 64 : 128);
  while (tq > 32 && tiles_of(nq, n, tq) < 256) tq /= 2;
  return tq;
}

// Whether the whole call (not one block of it, so that scores do not depend
// on how it is cut into blocks: tiles of all sizes sum alike) takes the small
// kernel: fewer tiles than CUs whatever their size, which smaller ones spread
// over four times as many, or rows shorter than the 16 bytes the tiles read at
// a time.
bool small_scores(int64_t m, int64_t n, int64_t row_bytes) {
  return row_bytes < 16 || tiles_of(m, n, tile_queries(m, n)) < 256;
}

template <typename T, int QB, int QW, int RB, int RW, bool STREAM = false>
void launch_tiles(const ScoreArgs& a, hipStream_t stream) {
  const int64_t row_tiles = (a.rows + 32 * RB * RW - 1) / (32 * RB * RW);
  const int64_t q_tiles = (a.nq + 32 * QB * QW - 1) / (32 * QB * QW);
  const dim3 grid(static_cast<unsigned>((row_tiles + 7) / 8 * 8 * q_tiles));
  score_tile_kernel<T, QB, QW, RB, RW, STREAM><<<grid, 256, 0, stream>>>(a);
}

template <typename T>
hipError_t launch_score(const ScoreArgs& a, bool small, hipStream_t stream) {
  const int64_t tq = tile_queries(a.nq, a.rows);
  if (small) {
    const int64_t wgs = (a.rows + 31) / 32 * ((a.nq + 31) / 32);
    score_small_kernel<T><<<dim3(static_cast<unsigned>(wgs)), 256, 0, stream>>>(a);
  } else if (tq == 32) {
    const uintptr_t place = reinterpret_cast<uintptr_t>(a.bank) | static_cast<uintptr_t>(a.bank_stride * sizeof(T)) |
                            static_cast<uintptr_t>(a.d * sizeof(T));
    if (a.nq <= 32 && place % 16 == 0 && streams(a.rows, a.d * sizeof(T)))
      launch_tiles<T, 1, 1, 1, 4, true>(a, stream);
    else
      launch_tiles<T, 1, 1, 1, 4>(a, stream);
  } else if (tq == 64) {
    launch_tiles<T, 2, 1, 1, 4>(a, stream);
  } else {
    launch_tiles<T, 2, 2, 2, 2>(a, stream);
  }
  return hipGetLastError();
}

// The block's scores, in launches of at most 2^23 workgroups even of the
// smallest blocks: a launch has fewer than 2^32 threads, and a block with full
// probabilities is the whole bank.
template <typename T>
hipError_t launch_scores(const ScoreArgs& a, bool small, hipStream_t stream) {
  const int64_t most = (int64_t{1} << 28) / ((a.nq + 31) / 32) / 1024 * 1024;
  const int64_t per = most > 1024 ? most : 1024;
  for (int64_t r0 = 0; r0 < a.rows; r0 += per) {
    ScoreArgs part = a;
    part.bank = static_cast<const T*>(a.bank) + r0 * a.bank_stride;
    part.rows = a.rows - r0 < per ? a.rows - r0 : per;
    part.out = a.out + r0;
    const hipError_t e = launch_score<T>(part, small, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_topk_tables(const TableArgs& a, hipStream_t stream) {
  table_plan_kernel<<<1, kTablePlanThreads, 0, stream>>>(a);
  // four workgroups per CU, each taking every 1,024th tile
  if (streams(a.n, a.d * 2))
    score_tables_kernel<true><<<1024, 256, 0, stream>>>(a);
  else
    score_tables_kernel<false><<<1024, 256, 0, stream>>>(a);
  select_tables_kernel<<<dim3(static_cast<unsigned>(a.m)), kSelThreads, 0, stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_topk_score(const Plan& p, const void* bank, int64_t bank_stride, int64_t n, const void* queries,
                             int64_t q_stride, int64_t m, int32_t d, int32_t dtype, float c2, int64_t self_base,
                             int32_t k, const Scope& scope, void* ws, float* full_scores, int32_t* idx, float* score,
                             float* prob, float* lse, hipStream_t stream) {
  char* w = static_cast<char*>(ws);
  const int64_t elem = dtype == 0 ? 4 : 2;
  // with full probabilities the scores go to the caller's rows, all at once
  const int64_t mb = full_scores ? m : p.blk_queries;
  const int64_t nb = full_scores ? n : p.blk_rows;
  const bool small = small_scores(m, n, d * elem);
  for (int64_t q0 = 0; q0 < m; q0 += mb) {
    const int64_t nq = m - q0 < mb ? m - q0 : mb;
    for (int64_t c0 = 0; c0 < n; c0 += nb) {
      const int64_t c1 = c0 + nb < n ? c0 + nb : n;
      ScoreArgs sa{};
      sa.bank = static_cast<const char*>(bank) + c0 * bank_stride * elem;
      sa.bank_stride = bank_stride;
      sa.rows = c1 - c0;
      sa.queries = static_cast<const char*>(queries) + q0 * q_stride * elem;
      sa.q_stride = q_stride;
      sa.nq = nq;
      sa.d = d;
      sa.out = full_scores ? full_scores : reinterpret_cast<float*>(w + p.ws_scores);
      sa.ld = full_scores ? n : p.blk_rows;
      hipError_t e = dtype == 0 ? launch_scores<float>(sa, small, stream) : launch_scores<uint16_t>(sa, small, stream);
      if (e != hipSuccess) return e;
      SelectArgs a{};
      a.scores = sa.out;
      a.ld = sa.ld;
      a.q0 = q0;
      a.c0 = c0;
      a.c1 = c1;
      a.rows_per_split = p.rows_per_split;
      a.n_splits = p.n_splits;
      a.split0 = static_cast<int>(c0 / p.rows_per_split);
      a.block_splits = static_cast<int>((c1 - 1) / p.rows_per_split) - a.split0 + 1;
      a.k = k;
      a.kcap = p.kcap;
      a.c2 = c2;
      a.self_base = self_base;
      a.row_ns = scope.row_ns;
      a.key_ns = scope.key_ns;
      a.part_q0 = p.n_splits == 1 ? q0 : 0;
      a.part_keys = reinterpret_cast<uint64_t*>(w + p.ws_part_keys);
      a.part_ms = reinterpret_cast<float2*>(w + p.ws_part_ms);
      a.part_lo = reinterpret_cast<float*>(w + p.ws_part_lo);
      a.full = full_scores != nullptr;
      a.n = n;
      if (p.n_splits == 1 && c1 == n) {
        a.idx = idx;
        a.score = score;
        a.prob = prob;
        a.lse = lse;
      }
      const dim3 grid(static_cast<unsigned>(nq * a.block_splits));
      if (n <= 1024)
        select_kernel<4><<<grid, kSelThreads, 0, stream>>>(a);
      else if (n <= 2048)
        select_kernel<8><<<grid, kSelThreads, 0, stream>>>(a);
      else
        select_kernel<16><<<grid, kSelThreads, 0, stream>>>(a);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace memattn
