// Top-k selection by one workgroup of 256 threads, shared by the general
// path's select kernel and the merge of partial lists.  Internal to the
// library.
#pragma once

#include "device_common.h"
#include "launch.h"

namespace memattn {
namespace {

constexpr int kSelThreads = 256;
constexpr int kSelPer = 16;                          // keys per thread and step
constexpr int kSelStep = kSelThreads * kSelPer;      // keys per step
constexpr int kSelCand = kMaxK * kSelPer;            // most candidates of a step
constexpr int kSelDirect = 160;                      // up to so many are ranked without a better bound

// A descending list of 64-bit keys (zeros past its last) in two buffers, of
// which the caller tracks the current one, and scratch.
struct SelectLds {
  uint64_t list[2][kMaxK];
  uint64_t cand[kSelCand];
  uint64_t tops[kSelThreads];
  uint64_t thr;
  int wcount[4];
  float red_m[4];
  double red_s[4];
};

// Counts, over the workgroup, the keys at or above `least`; every wave's own
// count stays in wcount.  Leaves a barrier between the counts and their use.
template <class Key>
__device__ __forceinline__ int select_count(SelectLds& L, const Key& key, uint64_t least) {
  int mine = 0;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) mine += __builtin_popcountll(__ballot(key(j) >= least));
  if ((threadIdx.x & 63) == 0) L.wcount[threadIdx.x >> 6] = mine;
  __syncthreads();
  return L.wcount[0] + L.wcount[1] + L.wcount[2] + L.wcount[3];
}

// Offers a step's keys to the list: key(j), j < kSelPer, are this thread's
// (0 = none; all keys distinct).  Only keys above the list's k-th matter.  If
// many are (as in the first step), the k-th largest of the threads' own
// largest keys is a better bound: k keys lie at or above it, so no other can
// be among the k best, and only those k threads hold candidates, at most 16
// each.  One wave finds it on the keys' upper halves, bit by bit from
// ballots; where ties there let in too many, by counting over the whole keys.
// (With fewer than k threads holding a candidate there is no such bound, and
// at most 16 (k - 1) candidates.)  The candidates are compacted by ballots
// and ranked in the union with the list by counting; every rank below k is
// written once into the other buffer.  Returns the buffer then current.
// Every thread of the workgroup calls it.
template <class Key>
__device__ __forceinline__ int select_step(SelectLds& L, const Key& key, int k, int cur) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  uint64_t least = L.list[cur][k - 1] + 1;
  int total = select_count(L, key, least);
  if (total == 0) {  // (uniform)
    __syncthreads();  // wcount is free for the next step
    return cur;
  }
  if (total > kSelDirect) {
    uint64_t top = 0;
#pragma unroll
    for (int j = 0; j < kSelPer; ++j) {
      const uint64_t x = key(j);
      top = x > top ? x : top;
    }
    top = top >= least ? top : 0;
    L.tops[tid] = top;
    __syncthreads();
    if (wave == 0) {
      uint32_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = static_cast<uint32_t>(L.tops[64 * i + lane] >> 32);
      uint32_t t = 0;
      for (int b = 31; b >= 0; --b) {
        const uint32_t c = t | (1u << b);
        int n = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) n += __builtin_popcountll(__ballot(h[i] >= c));
        if (n >= k) t = c;
      }
      if (lane == 0) L.thr = static_cast<uint64_t>(t) << 32;
    }
    __syncthreads();
    least = L.thr > least ? L.thr : least;
    total = select_count(L, key, least);
    if (total > kSelCand) {
      // (more than kSelCand candidates: over k threads hold one, and the
      // k-th largest top is one thread's)
      int above = 0;
#pragma unroll 8
      for (int i = 0; i < kSelThreads; ++i) above += L.tops[i] > top ? 1 : 0;
      if (above == k - 1 && top != 0) L.thr = top;
      __syncthreads();
      least = L.thr;
      total = select_count(L, key, least);
    }
  }
  int at = 0;
  for (int w = 0; w < wave; ++w) at += L.wcount[w];
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    const uint64_t x = key(j);
    const uint64_t bal = __ballot(x >= least);
    if (x >= least) L.cand[at + __popcll(bal & ((uint64_t{1} << lane) - 1))] = x;
    at += __popcll(bal);
  }
  const int nxt = cur ^ 1;
  if (tid < kMaxK) L.list[nxt][tid] = 0;
  __syncthreads();
  for (int i = tid; i < total; i += kSelThreads) {
    const uint64_t x = L.cand[i];
    int lo = 0, hi = k;  // list keys above x
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (L.list[cur][mid] > x) lo = mid + 1; else hi = mid;
    }
    int r = lo;
#pragma unroll 4
    for (int c = 0; c < total; ++c) r += L.cand[c] > x ? 1 : 0;
    if (r < k) L.list[nxt][r] = x;
  }
  // (the last wave ranks the list's own keys: it has the fewest candidates)
  const int li = kSelThreads - 1 - tid;
  if (li < k) {
    const uint64_t y = L.list[cur][li];
    if (y != 0) {
      int r = li;
#pragma unroll 4
      for (int c = 0; c < total; ++c) r += L.cand[c] > y ? 1 : 0;
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
  float m_w = m_run;
  for (int off = 32; off > 0; off >>= 1) m_w = fmaxf(m_w, __shfl_xor(m_w, off));
  if (lane == 0) L.red_m[wave] = m_w;
  __syncthreads();
  const float m_all = fmaxf(fmaxf(L.red_m[0], L.red_m[1]), fmaxf(L.red_m[2], L.red_m[3]));
  double s_w = (m_run == -INFINITY) ? 0.0 : s_run * static_cast<double>(fast_exp2(m_run - m_all));
  for (int off = 32; off > 0; off >>= 1) s_w += __shfl_xor(s_w, off);
  if (lane == 0) L.red_s[wave] = s_w;
  __syncthreads();
  return SoftmaxSum{m_all, (L.red_s[0] + L.red_s[1]) + (L.red_s[2] + L.red_s[3])};
}

}  // namespace
}  // namespace memattn
