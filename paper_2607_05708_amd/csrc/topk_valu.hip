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
  const float m = wave_max_f32(v.x);
  const double s =
      wave_sum_f64(v.x != -INFINITY ? static_cast<double>(v.y) * static_cast<double>(fast_exp2(v.x - m)) : 0.0);
  return m + static_cast<float>(log2(s));
}

// One wave per key, four keys per workgroup, for at most 64 lists of at most
// 64 * PER keys in all (PER <= 16) and k <= 32: lane l's j-th key is rank
// (l + j) % kk of list j * (64 / kk) + l / kk (kk: k rounded up to a power of
// two), so that each lane gets every rank in turn.  As in select.h the k-th largest of the
// lanes' own largest upper halves bounds the candidates, which are compacted
// by ballots and ranked by counting, here without a workgroup barrier.
// Against a rank by binary search in every other list (few lists) and a
// k-step tournament over the list heads (more), whole calls: relation builds
// of 12,288 keys (5 lists of 32) 402 -> 366 us, of 8,192 (8 of 32) 245 -> 222
// us, 8,000 queries (8 of 32) 669 -> 645 us, 4,096 (16 of 32) 693 -> 685 us.
template <int PER>
__global__ __launch_bounds__(256) void topk_merge_wave_kernel(const uint64_t* __restrict__ part_keys,
                                                              const float2* __restrict__ part_ms, int64_t m,
                                                              int n_parts, int kcap, int k, int kk, float c2,
                                                              int32_t* __restrict__ idx, float* __restrict__ score,
                                                              float* __restrict__ prob, float* __restrict__ lse,
                                                              float* __restrict__ lse2_out,
                                                              const int32_t* __restrict__ done) {
  if (done != nullptr && *done != 0) return;
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) uint64_t all_cand[4][64 * PER + 2];
  __shared__ uint64_t all_chosen[4][32];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 4 + wave;
  if (q >= m) return;  // whole waves only; no workgroup barrier below
  uint64_t* cand = all_cand[wave];
  uint64_t* chosen = all_chosen[wave];
  const uint64_t* keys = part_keys + q * static_cast<int64_t>(n_parts) * kcap;
  const int per = 64 / kk;  // lists read at a time
  uint64_t x[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int s = j * per + lane / kk;
    const int r = (lane + j) & (kk - 1);
    x[j] = (s < n_parts && r < k) ? keys[static_cast<int64_t>(s) * kcap + r] : 0;
  }
  const float lse2 = wave_lse2(part_ms + q * n_parts, n_parts, lane);
  if (lane < k) chosen[lane] = 0;  // ranks that no key takes (fewer than k candidates) stay empty
  uint32_t top = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) top = max(top, static_cast<uint32_t>(x[j] >> 32));
  uint32_t least = 0;
  for (int b = 31; b >= 32 - kBoundBits; --b) {
    const uint32_t c = least | (1u << b);
    if (__builtin_popcountll(__ballot(top >= c)) >= k) least = c;
  }
  least = least < 1u ? 1u : least;
  int total = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const bool in = static_cast<uint32_t>(x[j] >> 32) >= least;
    const uint64_t bal = __ballot(in);
    if (in) cand[total + __popcll(bal & ((uint64_t{1} << lane) - 1))] = x[j];
    total += __popcll(bal);
  }
  if (lane == 0) cand[total] = 0;
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  for (int i = lane; i < total; i += 64) {
    const uint64_t y = cand[i];
    const u64x2* c = reinterpret_cast<const u64x2*>(cand);
    int r = 0;
#pragma unroll 8
    for (int e = 0; e < (total + 1) / 2; ++e) {
      const u64x2 v = c[e];
      r += (v.x > y ? 1 : 0) + (v.y > y ? 1 : 0);
    }
    if (r < k) chosen[r] = y;
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  if (lane < k) write_selected(chosen[lane], c2, lse2, q * k + lane, idx, score, prob);
  if (lane == 0) {
    if (lse) lse[q] = lse2 * kLn2;
    lse2_out[q] = lse2;
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
    cur = select_step<false, kSelPer>(
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
  char* w = static_cast<char*>(ws);
  const auto* keys = reinterpret_cast<const uint64_t*>(w + p.ws_part_keys);
  const auto* ms = reinterpret_cast<const float2*>(w + p.ws_part_ms);
  auto* lse2 = reinterpret_cast<float*>(w + p.ws_lse2);
  // consecutive lists of a key start kcap_eff keys apart (every part_stride-th slot)
  const int kcap_eff = p.kcap * p.part_stride;
  int kk = 8;
  while (kk < k) kk <<= 1;
  const int64_t total = static_cast<int64_t>(p.n_parts) * kk;
  // One wave up to 64 lists of 1,024 keys in all (1,000 queries with 59 lists
  // of 16: 124 us for the whole call, 132 by workgroups; 2,000 with 30 of 32:
  // 346 and 360); a workgroup is sooner done with more lists (100 queries with
  // 128 lists of 8: 344 against 352 us).
  if (k <= 32 && total <= 1024 && p.n_parts <= 64 && alt.flag == nullptr) {
    const dim3 grid(static_cast<unsigned>((m + 3) / 4));
    if (total <= 64)
      topk_merge_wave_kernel<1><<<grid, 256, 0, stream>>>(keys, ms, m, p.n_parts, kcap_eff, k, kk, c2, idx, score, prob,
                                                          lse, lse2, alt.done);
    else if (total <= 256)
      topk_merge_wave_kernel<4><<<grid, 256, 0, stream>>>(keys, ms, m, p.n_parts, kcap_eff, k, kk, c2, idx, score, prob,
                                                          lse, lse2, alt.done);
    else if (total <= 512)
      topk_merge_wave_kernel<8><<<grid, 256, 0, stream>>>(keys, ms, m, p.n_parts, kcap_eff, k, kk, c2, idx, score, prob,
                                                          lse, lse2, alt.done);
    else
      topk_merge_wave_kernel<16><<<grid, 256, 0, stream>>>(keys, ms, m, p.n_parts, kcap_eff, k, kk, c2, idx, score, prob,
                                                           lse, lse2, alt.done);
  } else {
    topk_merge_select_kernel<<<dim3(static_cast<unsigned>(m)), kSelThreads, 0, stream>>>(
        keys, ms, p.n_parts, kcap_eff, k, kk, c2, idx, score, prob, lse, lse2, alt);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || fp.full == nullptr) return e;
  return launch_full_prob(p, m, fp.n, c2, fp.self_base, fp.full, ws, stream);
}

hipError_t launch_full_prob(const Plan& p, int64_t m, int64_t n, float c2, int64_t self_base, float* full, void* ws,
                            hipStream_t stream) {
  char* w = static_cast<char*>(ws);
  const dim3 grid(static_cast<unsigned>((n + 255) / 256), static_cast<unsigned>(m));
  full_prob_kernel<<<grid, 256, 0, stream>>>(full, n, c2, self_base, reinterpret_cast<const float*>(w + p.ws_lse2));
  return hipGetLastError();
}

}  // namespace memattn
