// Top-k selection by one workgroup of 256 threads, shared by the general
// path's select kernel and the merge of partial lists.  Internal to the
// library.
#pragma once

#include "device_common.h"
#include "launch.h"

namespace memattn {
namespace {

constexpr int kSelThreads = 256;
constexpr int kSelPer = 16;                          // most keys per thread and step
constexpr int kSelStep = kSelThreads * kSelPer;      // and keys per step
constexpr int kSelCand = kMaxK * kSelPer;            // most candidates of a step
constexpr int kSelDirect = 160;                      // up to so many are ranked without a better bound

// A descending list of 64-bit keys (zeros past its last) in two buffers, of
// which the caller tracks the current one, and scratch.
struct SelectLds {
  uint64_t list[2][kMaxK];
  __attribute__((aligned(16))) uint64_t cand[kSelCand + 2];
  uint32_t tops[kSelThreads];
  uint64_t thr;
  int wcount[4];
  float red_m[4];
  double red_s[4];
};

// Counts, over the workgroup, the in(j), j < PER, of every thread (only
// those with `any` have one); every wave's own count stays in wcount.
template <int PER, class In>
__device__ __forceinline__ int select_count(SelectLds& L, const In& in, bool any) {
  int mine = 0;
  if (__ballot(any) != 0) {
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += __builtin_popcountll(__ballot(in(j)));
  }
  if ((threadIdx.x & 63) == 0) L.wcount[threadIdx.x >> 6] = mine;
  __syncthreads();
  return L.wcount[0] + L.wcount[1] + L.wcount[2] + L.wcount[3];
}

// How many of cand[0, total) are above x (total even or followed by a 0).
__device__ __forceinline__ int count_above(const SelectLds& L, int total, uint64_t x) {
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  const u64x2* c = reinterpret_cast<const u64x2*>(L.cand);
  int r = 0;
#pragma unroll 8
  for (int i = 0; i < (total + 1) / 2; ++i) {
    const u64x2 v = c[i];
    r += (v.x > x ? 1 : 0) + (v.y > x ? 1 : 0);
  }
  return r;
}

// Offers a step's keys to the list: key(j), j < PER, are this thread's
// (0 = none; all distinct, or equal ones may be lost), hi(j) their upper halves
// and top the largest of those.  Only keys above the list's k-th matter; with
// RISING (every key is of a later row than the list's) those with a larger
// upper half.  If many are (as in the first step), the k-th largest of the
// threads' tops is a better bound: k keys lie at or above it, so none below can
// be among the k best, and but for ties only those k threads hold candidates,
// at most 16 each.
// One wave finds its upper kBoundBits bits from ballots.  (With fewer than k
// threads holding any there is no such bound, and at most 16 (k - 1)
// candidates.)  Where ties let in too many, the bound is found once more on
// whole keys, by counting.  The candidates are compacted by ballots and
// ranked in the union with the list by counting; every rank below k is
// written once into the other buffer.  Returns the buffer then current.
// A step without candidates costs one barrier and touches no key; every
// thread of the workgroup calls it, in every step.
constexpr int kBoundBits = 22;  // (the rest, 2^-13 of a score, lets few more in)
template <bool RISING, int PER, class Hi, class Key>
__device__ __forceinline__ int select_step(SelectLds& L, const Hi& hi, const Key& key, uint32_t top, int k, int cur) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const uint64_t last = L.list[cur][k - 1];
  uint32_t least = static_cast<uint32_t>(last >> 32) + (RISING ? 1u : 0u);
  least = least < 1u ? 1u : least;
  auto above = [&](int j) { return hi(j) >= least; };
  int total = 0;
  if (last != 0) {
    if (!__syncthreads_or(top >= least)) return cur;
    total = select_count<PER>(L, above, top >= least);
  }
  bool whole = false;  // the bound is a whole key
  uint64_t least64 = 0;
  if (last == 0 || total > kSelDirect) {
    L.tops[tid] = top;
    __syncthreads();
    if (wave == 0) {
      uint32_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = L.tops[64 * i + lane];
      uint32_t t = 0;
      for (int b = 31; b >= 32 - kBoundBits; --b) {
        const uint32_t c = t | (1u << b);
        int n = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) n += __builtin_popcountll(__ballot(h[i] >= c));
        if (n >= k) t = c;
      }
      if (lane == 0) L.thr = t;
    }
    __syncthreads();
    const uint32_t t = static_cast<uint32_t>(L.thr);
    least = t > least ? t : least;
    total = select_count<PER>(L, above, top >= least);
    if (total > kSelCand) {
      // (more than kSelCand: over k threads hold a candidate, so the k-th
      // largest of their largest keys is one thread's.  Fewer than k threads
      // hold keys above it, also where a chunk table repeats a row and keys
      // are equal: those and one copy of it are the candidates.)
      uint64_t best = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const uint64_t x = key(j);
        best = x > best ? x : best;
      }
      L.cand[tid] = best;
      __syncthreads();
      if (best != 0 && count_above(L, kSelThreads, best) < k && count_above(L, kSelThreads, best - 1) >= k) L.thr = best;
      __syncthreads();
      least64 = L.thr;
      whole = true;
      if (tid == 0) L.cand[0] = least64;
      total = 1 + select_count<PER>(L, [&](int j) { return key(j) > least64; }, true);
    }
  }
  int at = whole ? 1 : 0;
  for (int w = 0; w < wave; ++w) at += L.wcount[w];
  if (L.wcount[wave] != 0) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool in = whole ? key(j) > least64 : above(j);
      const uint64_t bal = __ballot(in);
      if (in) L.cand[at + __popcll(bal & ((uint64_t{1} << lane) - 1))] = key(j);
      at += __popcll(bal);
    }
  }
  const int nxt = cur ^ 1;
  if (tid < kMaxK) L.list[nxt][tid] = 0;
  if (tid == 0) L.cand[total] = 0;
  __syncthreads();
  for (int i = tid; i < total; i += kSelThreads) {
    const uint64_t x = L.cand[i];
    int lo = 0, up = k;  // list keys above x
    while (lo < up) {
      const int mid = (lo + up) >> 1;
      if (L.list[cur][mid] > x) lo = mid + 1; else up = mid;
    }
    const int r = lo + count_above(L, total, x);
    if (r < k) L.list[nxt][r] = x;
  }
  // (the last wave ranks the list's own keys: it has the fewest candidates)
  const int li = kSelThreads - 1 - tid;
  if (li < k) {
    const uint64_t y = L.list[cur][li];
    if (y != 0) {
      const int r = li + count_above(L, total, y);
      if (r < k) L.list[nxt][r] = y;
    }
  }
  __syncthreads();
  return nxt;
}

// The threads' softmax states (max, sum of exp2(x - max)) as one.
struct SoftmaxSum {
  float max;
  double sum;
};
__device__ __forceinline__ SoftmaxSum block_softmax(SelectLds& L, float m_run, double s_run) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const float m_w = wave_max_f32(m_run);
  if (lane == 0) L.red_m[wave] = m_w;
  __syncthreads();
  const float m_all = fmaxf(fmaxf(L.red_m[0], L.red_m[1]), fmaxf(L.red_m[2], L.red_m[3]));
  const double s_w = wave_sum_f64((m_run == -INFINITY) ? 0.0 : s_run * static_cast<double>(fast_exp2(m_run - m_all)));
  if (lane == 0) L.red_s[wave] = s_w;
  __syncthreads();
  return SoftmaxSum{m_all, (L.red_s[0] + L.red_s[1]) + (L.red_s[2] + L.red_s[3])};
}

}  // namespace
}  // namespace memattn
