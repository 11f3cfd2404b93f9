// Merges of partial selections (one sorted list and softmax partial per
// bank split) into the final top-k, probabilities and normaliser, and the
// full probability rows of banks that took several splits.
#include "device_common.h"
#include "launch.h"
#include "select.h"

namespace memattn {

namespace {

// Softmax partials of one query (at most 64), combined by one wave: lse2 =
// log2 of the normaliser in the scaled log2 domain (max, then the rescaled sum
// in fp64).
__device__ __forceinline__ float wave_lse2(const float2* __restrict__ ms, int n_parts, int lane) {
  const float2 v = lane < n_parts ? ms[lane] : make_float2(-INFINITY, 0.f);
  float m = v.x;
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  double s = v.x != -INFINITY ? static_cast<double>(v.y) * static_cast<double>(fast_exp2(v.x - m)) : 0.0;
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  return m + static_cast<float>(log2(s));
}

// Copy the first k keys of lists [l0, l0 + nl) (list l at keys + l * kcap)
// into dst[(l - l0) * k + j] with one wave, 16 loads in flight per lane.
__device__ __forceinline__ void stage_list_heads(uint64_t* dst, const uint64_t* __restrict__ keys, int l0, int nl,
                                                 int k, int kcap, int lane) {
  constexpr int kU = 16;
  const int total = nl * k;
  for (int base = 0; base < total; base += 64 * kU) {
    uint64_t v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = base + u * 64 + lane;
      v[u] = i < total ? keys[static_cast<int64_t>(l0 + i / k) * kcap + i % k] : 0;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = base + u * 64 + lane;
      if (i < total) dst[i] = v[u];
    }
  }
}

// One wave per key, four keys per workgroup, for few partial lists
// (S * k <= kRankMaxKeys): the first k keys of every list are staged in LDS
// and each staged key finds its rank in the union by a binary search in
// every (descending) list; keys are unique (except empty slots, which rank
// below every real key), so the keys of rank < k are exactly the top-k and
// each lands in its own output slot.
// LDS is sized per launch (rank_lds_bytes): four waves' staged keys and
// chosen keys, so that short rows leave room for more workgroups per CU.
// With `full` set (a bank of at most kRankFullMax rows) the wave also turns
// its query's row of raw scores there into probabilities, saving the
// separate launch of full_prob_kernel (same arithmetic).
constexpr int kRankMaxKeys = 1024;
constexpr int64_t kRankFullMax = 4096;
size_t rank_lds_bytes(int n_parts, int k) {
  return 4 * (static_cast<size_t>(n_parts) * k + kMaxK) * sizeof(uint64_t);
}

__global__ __launch_bounds__(256) void topk_merge_rank_kernel(const uint64_t* __restrict__ part_keys,
                                                              const float2* __restrict__ part_ms, int64_t m,
                                                              int n_parts, int kcap, int k, float c2,
                                                              int32_t* __restrict__ idx, float* __restrict__ score,
                                                              float* __restrict__ prob, float* __restrict__ lse,
                                                              float* __restrict__ lse2_out, float* __restrict__ full,
                                                              int64_t n_full, int64_t self_base,
                                                              const int32_t* done) {
  if (done != nullptr && *done != 0) return;
  extern __shared__ uint64_t rank_smem[];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + wave;
  if (q >= m) return;  // whole waves only; no workgroup barrier below
  const int total = n_parts * k;
  uint64_t* st = rank_smem + static_cast<int64_t>(wave) * (total + kMaxK);
  uint64_t* chosen = st + total;
  const uint64_t* keys = part_keys + q * static_cast<int64_t>(n_parts) * kcap;
  // ranks that no key takes (fewer than k candidates) stay empty
  if (lane < k) chosen[lane] = 0;
  const float lse2 = wave_lse2(part_ms + q * n_parts, n_parts, lane);
  stage_list_heads(st, keys, 0, n_parts, k, kcap, lane);
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  for (int i = lane; i < total; i += 64) {
    const uint64_t x = st[i];
    if (x == 0) continue;
    int rank = 0;
    for (int s = 0; s < n_parts; ++s) {
      // number of keys > x in list s: first position holding a key <= x
      const uint64_t* l = st + s * k;
      int lo = 0, hi = k;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (l[mid] > x) lo = mid + 1; else hi = mid;
      }
      rank += lo;
    }
    if (rank < k) chosen[rank] = x;
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  if (lane < k) write_selected(chosen[lane], c2, lse2, q * k + lane, idx, score, prob);
  if (lane == 0) {
    if (lse) lse[q] = lse2 * kLn2;
    lse2_out[q] = lse2;
  }
  if (full != nullptr) {
    // 16 values per lane in flight at a time (n_full <= kRankFullMax)
    float* row = full + q * n_full;
    constexpr int kU = 16;
    for (int64_t base = 0; base < n_full; base += 64 * kU) {
      float v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t j = base + u * 64 + lane;
        v[u] = j < n_full ? row[j] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t j = base + u * 64 + lane;
        if (j < n_full)
          row[j] = ((self_base >= 0 && j == self_base + q) || lse2 == -INFINITY) ? 0.f : fast_exp2(v[u] * c2 - lse2);
      }
    }
  }
}

// One workgroup per key, for more partial lists: the lists' keys, 4,096 a
// step, go through the selection of select.h.  A step's thread t reads rank
// (t + j) % kk of list j * (256 / kk) + t / kk (kk: k rounded up to a power of
// two, which divides 256), so that each thread gets every rank in turn and
// the lists' heads, which hold the answer, fall to all threads alike: the
// selection's bound comes from the threads' own best keys.  (A k-step
// tournament over the lists' heads did this: 27 -> 9 us for 16 keys with 256
// lists of 32, 30 -> 9 us for 200 with 13 of 64, 20 -> 8 us for 1,024 with 64
// of 32.)
__global__ __launch_bounds__(kSelThreads) void topk_merge_select_kernel(
    const uint64_t* __restrict__ part_keys, const float2* __restrict__ part_ms, int n_parts, int kcap, int k, int kk,
    float c2, int32_t* __restrict__ idx, float* __restrict__ score, float* __restrict__ prob, float* __restrict__ lse,
    float* __restrict__ lse2_out, MergeAlt alt) {
  if (alt.done != nullptr && *alt.done != 0) return;
  __shared__ SelectLds L;
  const int tid = threadIdx.x;
  const int64_t q = blockIdx.x;
  const uint64_t* keys = part_keys + q * static_cast<int64_t>(n_parts) * kcap;
  const float2* ms = part_ms + q * n_parts;
  if (alt.flag != nullptr && *alt.flag != 0) {  // (uniform)
    keys = alt.keys + q * static_cast<int64_t>(alt.n_parts) * alt.kcap;
    ms = alt.ms + q * alt.n_parts;
    kcap = alt.kcap;
    n_parts = *alt.parts;
  }
  const int per = kSelThreads / kk;  // lists read at a time
  if (tid < kMaxK) L.list[0][tid] = 0;
  float m_run = -INFINITY;
  double s_run = 0.0;
  for (int s = tid; s < n_parts; s += kSelThreads) {
    const float2 v = ms[s];
    if (v.x == -INFINITY) continue;
    const float mx = fmaxf(m_run, v.x);
    s_run = s_run * static_cast<double>(fast_exp2(m_run - mx)) +
            static_cast<double>(v.y) * static_cast<double>(fast_exp2(v.x - mx));
    m_run = mx;
  }
  __syncthreads();
  int cur = 0;
  const int l0 = tid / kk;
  for (int l = 0; l < n_parts; l += per * kSelPer) {
    uint64_t x[kSelPer];
#pragma unroll
    for (int j = 0; j < kSelPer; ++j) {
      const int s = l + j * per + l0;
      const int r = (tid + j) & (kk - 1);
      x[j] = (s < n_parts && r < k) ? keys[static_cast<int64_t>(s) * kcap + r] : 0;
    }
    uint32_t top = 0;
#pragma unroll
    for (int j = 0; j < kSelPer; ++j) top = max(top, static_cast<uint32_t>(x[j] >> 32));
    cur = select_step<false>(
        L, [&](int j) { return static_cast<uint32_t>(x[j] >> 32); }, [&](int j) { return x[j]; }, top, k, cur);
  }
  const SoftmaxSum all = block_softmax(L, m_run, s_run);
  const float lse2 = all.max + static_cast<float>(log2(all.sum));
  if (tid < k) write_selected(L.list[cur][tid], c2, lse2, q * k + tid, idx, score, prob);
  if (tid == 0) {
    if (lse) lse[q] = lse2 * kLn2;
    // (for the full probability rows; the other partials may lie there)
    if (alt.flag == nullptr) lse2_out[q] = lse2;
  }
}

__global__ __launch_bounds__(256) void full_prob_kernel(float* __restrict__ full, int64_t n, float c2,
                                                        int64_t self_base, const float* __restrict__ lse2) {
  const int64_t q = blockIdx.y;
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (j >= n) return;
  const float l = lse2[q];
  float* p = full + q * n + j;
  // rows outside the candidates hold -inf scores; with no candidate at all
  // (an empty namespace) lse is -inf and every probability is 0
  *p = ((self_base >= 0 && j == self_base + q) || l == -INFINITY) ? 0.f : fast_exp2(*p * c2 - l);
}

}  // namespace

hipError_t launch_topk_merge(const Plan& p, int64_t m, int32_t k, float c2, int32_t* idx, float* score, float* prob,
                             float* lse, void* ws, hipStream_t stream, const FullProb& fp, const MergeAlt& alt) {
  // every merge but the fused rank merge leaves the full rows to full_prob_kernel
  auto finish = [&](hipError_t e) -> hipError_t {
    if (e != hipSuccess || fp.full == nullptr) return e;
    return launch_full_prob(p, m, fp.n, c2, fp.self_base, fp.full, ws, stream);
  };
  char* w = static_cast<char*>(ws);
  const auto* keys = reinterpret_cast<const uint64_t*>(w + p.ws_part_keys);
  const auto* ms = reinterpret_cast<const float2*>(w + p.ws_part_ms);
  auto* lse2 = reinterpret_cast<float*>(w + p.ws_lse2);
  const int64_t S = p.n_parts;
  // consecutive lists of a key start kcap_eff keys apart (every part_stride-th slot)
  const int kcap_eff = p.kcap * p.part_stride;
  if (S * k <= kRankMaxKeys && S <= 4 && alt.flag == nullptr) {
    const bool fused = fp.full != nullptr && fp.n <= kRankFullMax;
    topk_merge_rank_kernel<<<dim3(static_cast<unsigned>((m + 3) / 4)), 256, rank_lds_bytes(p.n_parts, k), stream>>>(
        keys, ms, m, p.n_parts, kcap_eff, k, c2, idx, score, prob, lse, lse2, fused ? fp.full : nullptr, fp.n,
        fp.self_base, alt.done);
    return fused ? hipGetLastError() : finish(hipGetLastError());
  }
  int kk = 1;
  while (kk < k) kk <<= 1;
  topk_merge_select_kernel<<<dim3(static_cast<unsigned>(m)), kSelThreads, 0, stream>>>(
      keys, ms, p.n_parts, kcap_eff, k, kk, c2, idx, score, prob, lse, lse2, alt);
  return finish(hipGetLastError());
}

hipError_t launch_full_prob(const Plan& p, int64_t m, int64_t n, float c2, int64_t self_base, float* full, void* ws,
                            hipStream_t stream) {
  char* w = static_cast<char*>(ws);
  const dim3 grid(static_cast<unsigned>((n + 255) / 256), static_cast<unsigned>(m));
  full_prob_kernel<<<grid, 256, 0, stream>>>(full, n, c2, self_base, reinterpret_cast<const float*>(w + p.ws_lse2));
  return hipGetLastError();
}

}  // namespace memattn
