// Chunk tables for a scoped selection over a shared bank.  The scoped call
// names a namespace per bank row and per query; scoring the whole bank and
// masking it costs every query the whole bank.  Where the queries' own rows
// are few enough, it is cheaper to collect them first (for each queried
// namespace the ascending ids of its live rows, the chunk table T[u][s] of
// Section 4.1) and to score each query against its own table only, as the
// grouped call does.
//
//   1. scope_plan_kernel (one workgroup): the distinct namespaces of the
//      queries (a hash table; namespace ids are any non-negative int32), the
//      queries in namespace order, and a sample of the bank's rows, from
//      which it decides whether the tables pay.  If not, it leaves no work
//      item and the flag 0, and the kernels after it return at once.
//   2. scope_count_kernel: rows per (namespace, 1,024-row block).
//   3. scope_scan_kernel (one workgroup per namespace): those counts become
//      positions within the namespace's table, and the table gets its place.
//   4. scope_fill_kernel: every row of a queried namespace to its position.
//      A wave takes its block in order, 64 rows at a time; a row's rank among
//      the 64 comes from ballots over the bits of its namespace's number, so
//      ids ascend within a table.  Workgroups past the bank's copy the
//      queries into grouped order.
//
// 1,024 queries against 1M x 1024 rows in 256 namespaces, k = 32: 2.95 ms
// masked, 0.49 ms through the tables (rows in bursts of 64), 2.38 and 0.49 ms
// (mixed rows); 8 namespaces 2.43 and 1.33 ms.  The four launches take 55 us.
// One namespace, where the plan declines, costs 17 us and the idle launches:
// 2.39 and 2.43 ms.
#include "device_common.h"
#include "launch.h"

namespace memattn {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPlanThreads = 1024;
constexpr int kPlanPer = static_cast<int>(kScopeMaxQueries) / kPlanThreads;  // queries (and namespaces) per thread
constexpr int kPlanSample = 4096;  // bank rows sampled for the decision

__device__ __forceinline__ uint32_t hash_slot(int32_t ns, int bits) {
  return (static_cast<uint32_t>(ns) * 2654435761u) >> (32 - bits);
}

// The number of namespace `ns` among the queried ones, -1 if it is none.
__device__ __forceinline__ int32_t find_ns(const int32_t* key, const int32_t* num, int bits, int32_t ns) {
  if (ns < 0) return -1;
  uint32_t s = hash_slot(ns, bits);
  const uint32_t mask = (1u << bits) - 1;
  for (;;) {  // (the table is at most half full: an empty slot ends every search)
    const int32_t k = key[s];
    if (k == ns) return num[s];
    if (k < 0) return -1;
    s = (s + 1) & mask;
  }
}

// Exclusive sum over the workgroup's threads; `total` gets the sum of all.
__device__ __forceinline__ int32_t plan_exclusive(int32_t mine, int32_t* red, int32_t& total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int32_t inc = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t o = __shfl_up(inc, off);
    if (lane >= off) inc += o;
  }
  __syncthreads();
  if (lane == 63) red[wave] = inc;
  __syncthreads();
  int32_t before = 0;
  total = 0;
  for (int w = 0; w < kPlanThreads / 64; ++w) {
    before += w < wave ? red[w] : 0;
    total += red[w];
  }
  return before + inc - mine;
}

__global__ __launch_bounds__(kPlanThreads) void scope_plan_kernel(ScopeArgs a) {
  __shared__ int32_t key[2 * kScopeMaxQueries];
  __shared__ int32_t num[2 * kScopeMaxQueries];
  __shared__ int32_t cnt[kScopeMaxQueries];
  __shared__ int32_t start[kScopeMaxQueries];
  __shared__ int32_t red[kPlanThreads / 64];
  __shared__ int32_t n_groups;
  const int tid = threadIdx.x;
  const int m = static_cast<int>(a.m);
  const int slots = 1 << a.bits;
  // (the sampled rows' namespaces, needed last, are asked for first)
  constexpr int kPer = kPlanSample / kPlanThreads;
  const int64_t sampled = a.n < kPlanSample ? a.n : kPlanSample;
  int32_t seen[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int64_t i = tid + j * kPlanThreads;
    seen[j] = i < sampled ? a.row_ns[i * a.n / sampled] : -1;
  }
  for (int s = tid; s < slots; s += kPlanThreads) key[s] = -1;
  for (int i = tid; i < m; i += kPlanThreads) cnt[i] = 0;
  if (tid == 0) n_groups = 0;
  __syncthreads();
  int32_t slot[kPlanPer];
#pragma unroll
  for (int j = 0; j < kPlanPer; ++j) {
    const int i = tid + j * kPlanThreads;
    const int32_t ns = i < m ? a.query_ns[i] : -1;
    slot[j] = -1;
    if (ns >= 0) {
      uint32_t s = hash_slot(ns, a.bits);
      for (;;) {
        const int32_t old = atomicCAS(&key[s], -1, ns);
        if (old < 0 || old == ns) break;
        s = (s + 1) & (slots - 1);
      }
      slot[j] = static_cast<int32_t>(s);
    }
  }
  __syncthreads();
  for (int s = tid; s < slots; s += kPlanThreads) {
    if (key[s] >= 0) num[s] = atomicAdd(&n_groups, 1);
  }
  __syncthreads();
  const int groups = n_groups;
  int32_t group[kPlanPer], rank[kPlanPer];
#pragma unroll
  for (int j = 0; j < kPlanPer; ++j) {
    group[j] = slot[j] >= 0 ? num[slot[j]] : -1;
    rank[j] = group[j] >= 0 ? atomicAdd(&cnt[group[j]], 1) : 0;
  }
  __syncthreads();
  // first grouped position and first 64-query tile of each namespace
  int32_t c[kPlanPer], sum_q = 0, sum_t = 0;
#pragma unroll
  for (int j = 0; j < kPlanPer; ++j) {
    const int u = tid * kPlanPer + j;
    c[j] = u < groups ? cnt[u] : 0;
    sum_q += c[j];
    sum_t += (c[j] + 63) / 64;
  }
  int32_t grouped, tiles;
  int32_t at_q = plan_exclusive(sum_q, red, grouped);
  int32_t at_t = plan_exclusive(sum_t, red, tiles);
  // the sample: bank rows that lie in a queried namespace, and how many
  // 64-query tiles would score them
  int32_t in = 0, work = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int32_t g = find_ns(key, num, a.bits, seen[j]);
    if (g >= 0) {
      ++in;
      work += (cnt[g] + 63) / 64;
    }
  }
  int32_t rows_in, row_tiles;
  plan_exclusive(in, red, rows_in);
  plan_exclusive(work, red, row_tiles);
  // A 64-query tile costs a row about 0.72 ns (d = 1,024), the masked pass
  // 2.7 ns per 1,024 queries, so the tables pay below m / 267 tiles per row
  // of the bank; the line lies a sixth below that.
  const bool use = static_cast<double>(row_tiles) * 320.0 < static_cast<double>(sampled) * static_cast<double>(m);
  // about one work item per CU, but no more splits than an average table has tiles
  const int64_t mean_rows =
      static_cast<int64_t>(rows_in) * a.n / sampled / (groups > 0 ? groups : 1);
  int64_t S = tiles > 0 ? 256 / tiles : 1;
  const int64_t mean_tiles = (mean_rows + 511) / 512;
  S = S > mean_tiles ? mean_tiles : S;
  S = S > a.max_splits ? a.max_splits : S;
  S = S < 1 ? 1 : S;
#pragma unroll
  for (int j = 0; j < kPlanPer; ++j) {
    const int u = tid * kPlanPer + j;
    if (u < m) {
      start[u] = at_q;
      a.q_off[u] = at_q;
      a.item_off[u] = use ? at_t * S : 0;
      a.table[2 * u] = a.table[2 * u + 1] = 0;
      at_q += c[j];
      at_t += (c[j] + 63) / 64;
    }
  }
  if (tid == 0) {
    a.q_off[m] = use ? grouped : 0;
    a.item_off[m] = use ? tiles * S : 0;
    a.flags[0] = use ? 1 : 0;
    a.flags[1] = static_cast<int32_t>(S);
    a.flags[2] = groups;
    a.flags[3] = 0;  // table entries handed out
  }
  for (int s = tid; s < slots; s += kPlanThreads) {
    a.key[s] = key[s];
    a.num[s] = key[s] >= 0 ? num[s] : -1;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPlanPer; ++j) {
    const int i = tid + j * kPlanThreads;
    if (i >= m) continue;
    a.thr[i] = 0u;
    if (group[j] >= 0) {
      a.perm[start[group[j]] + rank[j]] = i;
      a.q_pos[i] = start[group[j]] + rank[j];
    } else {
      a.q_pos[i] = -1;
      // no work item covers a query without a namespace: empty partials
      for (int64_t s = 0; s < S; ++s) {
        for (int e = 0; e < a.kcap; ++e) a.part_keys[((i * a.max_splits + s) * a.part_stride) * a.kcap + e] = 0;
        a.part_ms[i * a.max_splits + s] = make_float2(-INFINITY, 0.f);
      }
    }
  }
}

// Loads the hash table into LDS: keys, then numbers.
__device__ __forceinline__ void load_table(const ScopeArgs& a, int32_t* lds) {
  const int slots = 1 << a.bits;
  for (int s = threadIdx.x; s < slots; s += 256) {
    lds[s] = a.key[s];
    lds[slots + s] = a.num[s];
  }
}

__global__ __launch_bounds__(256) void scope_count_kernel(ScopeArgs a) {
  if (a.flags[0] == 0) return;
  extern __shared__ int32_t lds[];
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int groups = a.flags[2];
  const int slots = 1 << a.bits;
  int32_t* cnt = lds + 2 * slots;  // [groups][4 waves]
  load_table(a, lds);
  for (int i = tid; i < 4 * groups; i += 256) cnt[i] = 0;
  __syncthreads();
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kScopeRows + wave * (kScopeRows / 4) + (tid & 63);
#pragma unroll 4
  for (int i = 0; i < kScopeRows / 256; ++i) {
    const int64_t r = r0 + 64 * i;
    const int32_t g = r < a.n ? find_ns(lds, lds + slots, a.bits, a.row_ns[r]) : -1;
    if (g >= 0) atomicAdd(&cnt[4 * g + wave], 1);
  }
  __syncthreads();
  for (int g = tid; g < groups; g += 256) {
    const int4 v = make_int4(cnt[4 * g], cnt[4 * g + 1], cnt[4 * g + 2], cnt[4 * g + 3]);
    *reinterpret_cast<int4*>(a.counts + g * a.n_blocks + 4 * static_cast<int64_t>(blockIdx.x)) = v;
  }
}

__global__ __launch_bounds__(256) void scope_scan_kernel(ScopeArgs a) {
  if (a.flags[0] == 0 || static_cast<int32_t>(blockIdx.x) >= a.flags[2]) return;
  __shared__ int32_t red[4];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  int32_t* c = a.counts + static_cast<int64_t>(blockIdx.x) * a.n_blocks;
  int32_t carry = 0;
  for (int64_t b0 = 0; b0 < a.n_blocks; b0 += 1024) {  // (n_blocks is a multiple of 4)
    const int64_t b = b0 + 4 * tid;
    int4 v = b < a.n_blocks ? *reinterpret_cast<int4*>(c + b) : make_int4(0, 0, 0, 0);
    const int32_t mine = v.x + v.y + v.z + v.w;
    int32_t inc = mine;
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t o = __shfl_up(inc, off);
      if (lane >= off) inc += o;
    }
    if (lane == 63) red[wave] = inc;
    __syncthreads();
    int32_t before = carry + inc - mine;
    for (int w = 0; w < wave; ++w) before += red[w];
    carry += red[0] + red[1] + red[2] + red[3];
    if (b < a.n_blocks)
      *reinterpret_cast<int4*>(c + b) =
          make_int4(before, before + v.x, before + v.x + v.y, before + v.x + v.y + v.z);
    __syncthreads();  // red is free
  }
  if (tid == 0) {
    // (the tables' order in memory does not matter)
    const int32_t base = atomicAdd(&a.flags[3], carry);
    a.table[2 * blockIdx.x] = base;
    a.table[2 * blockIdx.x + 1] = base + carry;
  }
}

__global__ __launch_bounds__(256) void scope_fill_kernel(ScopeArgs a) {
  if (a.flags[0] == 0) return;
  extern __shared__ int32_t lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t row_wgs = a.n_blocks / 4;
  if (blockIdx.x >= row_wgs) {
    // one wave per grouped position: copy its query's row (16-byte vectors)
    const int64_t pos = 4 * (blockIdx.x - row_wgs) + wave;
    if (pos >= a.q_off[a.m]) return;
    const u32x4* src = static_cast<const u32x4*>(a.queries) + a.perm[pos] * (a.q_stride / 8);
    u32x4* dst = static_cast<u32x4*>(a.qbuf) + pos * (a.d / 8);
    for (int v = lane; v < a.d / 8; v += 64) dst[v] = src[v];
    return;
  }
  const int groups = a.flags[2];
  const int slots = 1 << a.bits;
  int32_t* next = lds + 2 * slots;  // [groups][4 waves]: the wave's next entry
  load_table(a, lds);
  for (int g = tid; g < groups; g += 256) {
    const int4 v = *reinterpret_cast<const int4*>(a.counts + g * a.n_blocks + 4 * static_cast<int64_t>(blockIdx.x));
    const int32_t t = a.table[2 * g];
    next[4 * g] = t + v.x;
    next[4 * g + 1] = t + v.y;
    next[4 * g + 2] = t + v.z;
    next[4 * g + 3] = t + v.w;
  }
  __syncthreads();
  int bits = 0;  // bits of a namespace's number
  while ((1 << bits) < groups) ++bits;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kScopeRows + wave * (kScopeRows / 4) + lane;
  for (int i = 0; i < kScopeRows / 256; ++i) {
    const int64_t r = r0 + 64 * i;
    const int32_t g = r < a.n ? find_ns(lds, lds + slots, a.bits, a.row_ns[r]) : -1;
    uint64_t same = __ballot(g >= 0);  // lanes of the same namespace
    for (int b = 0; b < bits; ++b) {
      const uint64_t bal = __ballot((g >> b) & 1);
      same &= ((g >> b) & 1) ? bal : ~bal;
    }
    if (g >= 0) {
      const uint64_t before = same & ((uint64_t{1} << lane) - 1);
      const int32_t at = next[4 * g + wave];
      a.chunks[at + __popcll(before)] = static_cast<int32_t>(r);
      // (the lanes of a wave run together: every lane has read its entry)
      __builtin_amdgcn_wave_barrier();
      if (before == 0) next[4 * g + wave] = at + __popcll(same);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
}

}  // namespace

hipError_t launch_scope_tables(const ScopeArgs& a, hipStream_t stream) {
  const unsigned blocks = static_cast<unsigned>(a.n_blocks / 4);
  // hash table, and four counters per namespace (at most one per query)
  const size_t lds = (size_t{2} << a.bits) * 4 + static_cast<size_t>(a.m) * 16;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&scope_count_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&scope_fill_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  scope_plan_kernel<<<1, kPlanThreads, 0, stream>>>(a);
  scope_count_kernel<<<blocks, 256, lds, stream>>>(a);
  scope_scan_kernel<<<dim3(static_cast<unsigned>(a.m)), 256, 0, stream>>>(a);
  scope_fill_kernel<<<dim3(blocks + static_cast<unsigned>((a.m + 3) / 4)), 256, lds, stream>>>(a);
  return hipGetLastError();
}

}  // namespace memattn
