// Stage 3 as device code: fused gather + weighted flash-decode + split combine
// (paper Sec. 4.3 Eq. 8 and Eq. 9; the "weighted attention" of Sec. 4.4), shared by
// the decode kernel (dp_decode.hip) and by the selection kernel, which runs the
// same queue after its own selections when a launch serves few heads.
//
// A head's work is a list of rows: the tokens of its exact clusters (K row,
// V row, additive weight 0) followed by one pseudo-token per approximated
// cluster (key-centroid row, mean-value row, additive weight ln s_i, which
// makes its softmax weight s_i * exp(xbar_i) = Zhat_i).  Rows are read IN
// PLACE from the cluster-contiguous cache: no gather buffer is materialised, so
// the traffic is the 512 B per row the method itself needs.
//
// Work split: a head with R rows is cut into ceil(R / c) items of
// c = 64 * max(g, ceil(R / (64 * S))) rows (S = partial slots per head; g grows
// with the launch's total rows up to the rows one workgroup step covers: a light
// launch spreads over the whole chip in small items, a heavy one amortises its
// merges, yet keeps several items per workgroup so that the last round is short).
// Item boundaries are multiples of 64 rows, so the first list entry of an item
// comes from the plan's chunk table in O(1).  Heads differ by orders of magnitude
// in rows and the host knows none of the counts, so the grid is a fixed number of
// workgroups that pull items from a device-side queue: every workgroup builds
// the same prefix of items per head in LDS from head_rows[], then claims item
// numbers with an atomic counter until they run out (nobody waits for anybody).
// Inside a workgroup the waves take units of 16, 32 or 64 rows of an item, each for
// itself: a wave reads the list entries that cover its unit, works out per lane where
// one row lies, and then each 16-lane DPP row owns one cache row per
// load (lane t holds dims [8t, 8t+8) of K for the dot and of V for the
// accumulation) and keeps its own online-softmax state in base-2 exponent form;
// the states are merged through LDS at the end of the item.  (With the lists staged
// in LDS for the whole workgroup and walked row by row the decode launch took 155 us
// against 134 for 256 heads, half of them flat, over 128 k tokens, 765 MB of rows; and
// 27.1 against 23.2 for a fixed budget, 70 MB of rows.)  Partials (m, l, acc[128]) go to the
// workspace; the item of a head that finishes last (an arrival counter, no
// waiting) merges them (log-sum-exp merge), normalises and writes the output.
#pragma once

#include "dp_attend.hpp"
#include "dp_device.hpp"
#include "dp_kernels.hpp"

namespace dp {

typedef unsigned long long u64_t;
constexpr int kPartialStride = kHeadDim + 2;  // m, l, acc[128]

struct DecodeArgs {
  const void *q, *k_cache, *v_cache, *k_centroids, *v_centroids;
  const int64_t *seg_row_base;
  const int32_t *seg_cluster_ptr, *cluster_sizes;
  const int32_t *n_exact, *n_retained;
  Plan plan;
  float *partials;
  void *out;
  float *lse;  // nullable
  int32_t n_kv_heads, n_q_heads, group, max_k, splits, out_is_bf16;
  int32_t head0, n_heads;  // this launch serves heads [head0, head0 + n_heads), n_heads <= kMaxQueueHeads
  int32_t *queue_next;     // the launch's item counter (zeroed before the first claim)
  const int32_t *pending;  // nullable: heads of this launch that have work; 0 = return at once
  // A/B variant (kGathered): per-head buffers that hold the gathered exact rows of heads with at most rows_cap of them
  const void *k_gather, *v_gather;
  int32_t rows_cap;
  float scale_log2;  // sm_scale * log2(e)
};

// everything but the launch's slice of heads and its counters (head0, n_heads, queue_next, pending)
inline DecodeArgs decode_args_of(const CacheView &c, const int32_t *n_exact, const int32_t *n_retained,
                                 const Plan &plan, float *partials, int splits, const AttnOut &attn) {
  DecodeArgs a;
  a.q = c.q;
  a.k_cache = c.k_cache;
  a.v_cache = c.v_cache;
  a.k_centroids = c.k_centroids;
  a.v_centroids = c.v_centroids;
  a.seg_row_base = c.seg_row_base;
  a.seg_cluster_ptr = c.seg_cluster_ptr;
  a.cluster_sizes = c.cluster_sizes;
  a.n_exact = n_exact;
  a.n_retained = n_retained;
  a.plan = plan;
  a.partials = partials;
  a.out = attn.out;
  a.lse = attn.lse;
  a.out_is_bf16 = attn.out_is_bf16;
  a.n_kv_heads = c.n_kv_heads;
  a.n_q_heads = c.n_q_heads;
  a.group = c.group;
  a.max_k = c.max_clusters_per_seg;
  a.splits = splits;
  a.scale_log2 = c.sm_scale * kLog2e;
  a.k_gather = a.v_gather = nullptr;
  a.rows_cap = 0;
  a.head0 = 0;
  a.n_heads = 0;
  a.queue_next = nullptr;
  a.pending = nullptr;
  return a;
}

// An int32 that another workgroup of the SAME launch may have written (kCoherent, a template parameter in scope):
// a device-coherent load that does not hit a stale line of this compute die's L2; data of an earlier launch is read
// with a plain load.  (A macro: through a function the plain loads of uniform addresses were no longer scalar loads,
// eight more vector registers and a wave of occupancy on the decode kernel.)
#define DP_LD_I32(lvalue) \
  (kCoherent ? __hip_atomic_load(&(lvalue), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (lvalue))

// Rows in flight per 16-lane row in the queue.  Inside the selection's launch a CU holds one large workgroup (8 or 16 waves,
// against 20 of the decode kernel's small ones): the rows in flight per wave are doubled there (at 4 / at 8, 32 flat heads
// over 32 k tokens, four layers 141.2 / 137.5 us; over 128 k, one head in eight flat, two layers 86.5 / 85.8, all of them
// flat 140.0 both).
__host__ __device__ constexpr int queue_batch(bool coherent) { return coherent ? 8 : kAttendBatch; }

// rows per item of a head with R rows (multiple of kChunkRows); g: least chunks per item of this launch
__device__ __forceinline__ int rows_per_item(int R, int S, int g) {
  return kChunkRows * max(g, (R + kChunkRows * S - 1) / (kChunkRows * S));
}

// LDS of the queue, declared by the kernel that runs it (separate arrays: as members of one struct the same code
// needed 16 more vector registers and lost a wave of occupancy on the decode kernel)
#define DP_DECODE_LDS(T, HEADS)                                                                    \
  __shared__ float s_m[(T) / 64], s_l[(T) / 64];                                                   \
  __shared__ float s_acc[(T) / 64][kHeadDim];                                                      \
  __shared__ int s_last, s_item;                                                                   \
  __shared__ int s_rows[(HEADS)]
#define DP_DECODE_LDS_ARGS s_m, s_l, s_acc, &s_last, &s_item, s_rows

// What the rows [r0, r1) of a head's list are, one row per lane: lane 16 g + j takes row j of group g, `per` rows per
// group (4 per <= 64 rows, inside one 64-row chunk of the list whose first row lies in entry ent0).  Lane k holds the
// start and the source of entry ent0 + k: every entry has at least one row, so 64 of them cover the chunk.  The entry
// of a row is then the number of entries that start at or before it, counted in a 64-bit mask of the starts: no walk.
struct UnitLists {
  int start, source;
};
template <bool kGathered>
__device__ __forceinline__ UnitRows unit_rows(int lane, const UnitLists &li, const RowSources &src, const int32_t *row_start, const int32_t *ent_src,
                                              bool check, int ent0, int n_ex, int n_rt, int r0, int r1, int per) {
  const int rc = r0 & ~(kChunkRows - 1);
  const int d = li.start - rc;
  const uint32_t lo = wave_or(lane > 0 && d < 32 ? 1u << (d & 31) : 0u);
  const uint32_t hi = wave_or(lane > 0 && d >= 32 && d < 64 ? 1u << (d & 31) : 0u);
  const int j = lane & 15;
  const int mine = r0 + (lane >> 4) * per + j;
  const bool valid = j < per && mine < r1;
  const int row = valid ? mine : r1 - 1;
  const int at = row - rc;
  const uint32_t upto_lo = at >= 31 ? 0xffffffffu : (2u << at) - 1u;
  const uint32_t upto_hi = at >= 63 ? 0xffffffffu : at >= 32 ? (2u << (at - 32)) - 1u : 0u;
  int k = __popc(lo & upto_lo) + __popc(hi & upto_hi);
  int source = __shfl(li.source, k, 64), start = __shfl(li.start, k, 64);
  if (check) {
    // lists given by a caller: an entry without rows (not allowed, and it adds nothing) shares its start with the next
    // one, and the count is off: look the rows up one by one.  The entry behind the last lane's is none of the 64: its
    // start is read where it matters, behind 63 tokens of one-row clusters.
    const int next = __shfl_down(li.start, 1, 64);
    bool empty = lane < 63 && ent0 + lane + 1 < n_rt && next == li.start;
    if (lane == 63 && d < kChunkRows && ent0 + 63 < n_ex) empty = row_start[ent0 + 64] == li.start;
    if (__any(empty)) {
      k = 0;
      while (ent0 + k + 1 < n_rt && row_start[ent0 + k + 1] <= row) ++k;
      source = ent_src[ent0 + k];
      start = row_start[ent0 + k];
    }
  }
  const bool exact = ent0 + k < n_ex;
  // (unconditional, and an atomic load so that it stays so: inside a condition it is waited for on its own)
  const int size = __hip_atomic_load(src.seg_sizes + (exact ? 0 : source), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  UnitRows u;
  const int64_t token = kGathered && src.gather_row0 >= 0 ? src.gather_row0 + row : src.seg_row0 + source + (row - start);
  const int64_t g = exact ? token : src.c0 + source;
  const uint64_t ka = (uint64_t)(exact ? src.k_cache : src.k_centroids) + g * kRowBytes;
  const uint64_t va = (uint64_t)(exact ? src.v_cache : src.v_centroids) + g * kRowBytes;
  u.klo = (uint32_t)ka;
  u.khi = (uint32_t)(ka >> 32);
  u.vlo = (uint32_t)va;
  u.vhi = (uint32_t)(va >> 32);
  u.size = size;
  u.weight = !valid ? 0 : exact ? 1 : -1;
  return u;
}

// Merge of n partials (m, l, acc[128]; written by workgroups of this launch) by a workgroup, a 16-lane row per partial.
template <int T>
__device__ __forceinline__ void gather_partials(const float *P, int n, RowState &st, int lane16, int grp) {
  typedef unsigned long long u64;
  row_state_init(st);
#pragma unroll 1
  for (int s = grp; s < n; s += T / 16) {
    const u64 *Q = reinterpret_cast<const u64 *>(P + (int64_t)s * kPartialStride);  // 520 bytes apart: 8-byte aligned
    u64 w[5];
    w[0] = __hip_atomic_load(Q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[1 + i] = __hip_atomic_load(Q + 1 + 4 * lane16 + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float m = __uint_as_float((uint32_t)w[0]), l = __uint_as_float((uint32_t)(w[0] >> 32));
    const float M = fmaxf(st.m, m);
    const float wa = st.m == -INFINITY ? 0.f : exp2f(st.m - M), wb = m == -INFINITY ? 0.f : exp2f(m - M);
    st.l = st.l * wa + l * wb;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float o = __uint_as_float((uint32_t)(w[1 + i / 2] >> (32 * (i & 1))));
      st.acc[i] = st.acc[i] * wa + o * wb;
    }
    st.m = M;
  }
}

// Merge of a few partials by a thread per dimension: all loads go out together and nothing passes through LDS.
constexpr int kFewPartials = 8;
__device__ __forceinline__ void merge_few(const float *P, int n, int d, float &M, float &L, float &o) {
  float m[kFewPartials], l[kFewPartials], v[kFewPartials];
#pragma unroll
  for (int u = 0; u < kFewPartials; ++u) {
    const float *Q = P + min(u, n - 1) * kPartialStride;
    m[u] = __hip_atomic_load(Q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    l[u] = __hip_atomic_load(Q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v[u] = __hip_atomic_load(Q + 2 + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  M = m[0];
#pragma unroll
  for (int u = 1; u < kFewPartials; ++u) M = fmaxf(M, m[u]);
  L = o = 0.f;
#pragma unroll
  for (int u = 0; u < kFewPartials; ++u) {
    const float w = u >= n || m[u] == -INFINITY ? 0.f : exp2f(m[u] - M);
    L += u < n ? l[u] * w : 0.f;
    o += u < n ? v[u] * w : 0.f;
  }
}

// One item, the rows [split * c, + c) of a head: attend them, publish the partial, and merge the head if this item
// arrives last.  c is a multiple of 64.  The waves of the workgroup take units of the item in turn, each for itself:
// nothing but the merge at the end makes them wait for one another, so one wave's list lookups hide behind another
// one's rows.
template <int T, bool kGathered, bool kCoherent>
__device__ __forceinline__ void decode_item(const DecodeArgs &a, int head, int split, int R, int c, float *s_m, float *s_l,
                                            float (*s_acc)[kHeadDim], int *s_last) {
  constexpr int kWaves = T / 64;
  // (a thread number that is new with every item: addresses made from it are not kept in registers from item to item,
  // which cost a wave of occupancy)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, lane16 = tid & 15;
  const int row_a = split * c;
  const int row_b = min(R, row_a + c);
  const int n_active = (R + c - 1) / c;

  const int b = head / a.n_q_heads, h = head % a.n_q_heads;
  const int seg = b * a.n_kv_heads + h / a.group;
  const int c0 = a.seg_cluster_ptr[seg];
  const int n_ex = DP_LD_I32(a.n_exact[head]), n_rt = DP_LD_I32(a.n_retained[head]);
  const int32_t *ent_src = a.plan.ent_src + (int64_t)head * a.max_k;
  const int32_t *row_start = a.plan.row_start + (int64_t)head * (a.max_k + 1);
  const int32_t *chunk_entry = a.plan.chunk_entry + (int64_t)head * a.plan.chunk_stride;

  const uint4 qv = load_row_slice(a.q, (int64_t)head, lane16);

  RowSources src;
  src.k_cache = a.k_cache;
  src.v_cache = a.v_cache;
  src.k_centroids = a.k_centroids;
  src.v_centroids = a.v_centroids;
  src.seg_sizes = a.cluster_sizes + c0;
  src.seg_row0 = a.seg_row_base[seg];
  src.c0 = c0;
  src.gather_row0 = -1;
  // a head whose exact rows did not fit the buffer was not gathered: it is read in place
  if (kGathered && n_ex > 0 && row_start[n_ex] <= a.rows_cap) {
    src.k_cache = a.k_gather;
    src.v_cache = a.v_gather;
    src.gather_row0 = (int64_t)head * a.rows_cap;
  }

  RowState st;
  row_state_init(st);

  // rows per unit: 64, or fewer where the item would not give every wave one (at least one batch of every group)
  constexpr int kB = queue_batch(kCoherent);
  const int n_rows = row_b - row_a;
  const int unit = n_rows > kWaves * 32 ? 64 : (kB == 8 || n_rows > kWaves * 16) ? 32 : 16;
  const int wave = __builtin_amdgcn_readfirstlane(wave_id());
  int r0 = row_a + wave * unit;
  if (r0 < row_b) {
    int ent0 = DP_LD_I32(chunk_entry[r0 / kChunkRows]);
    int ent_next = DP_LD_I32(chunk_entry[min(r0 + kWaves * unit, R - 1) / kChunkRows]);
    UnitLists li;
    li.start = DP_LD_I32(row_start[min(ent0 + lane, n_rt)]);
    li.source = DP_LD_I32(ent_src[min(ent0 + lane, n_rt - 1)]);
#pragma unroll 1
    for (;;) {
      const int r1 = min(row_b, r0 + unit), next = r0 + kWaves * unit;
      const UnitRows rows = unit_rows<kGathered>(lane, li, src, row_start, ent_src, !kCoherent, ent0, n_ex, n_rt, r0, r1, unit / 4);
      // the next unit's lists are fetched in front of this one's rows
      ent0 = ent_next;
      ent_next = DP_LD_I32(chunk_entry[min(next + kWaves * unit, R - 1) / kChunkRows]);
      li.start = DP_LD_I32(row_start[min(ent0 + lane, n_rt)]);
      li.source = DP_LD_I32(ent_src[min(ent0 + lane, n_rt - 1)]);
      attend_unit<kB>(st, qv, a.scale_log2, rows, unit / (4 * kB), lane16);
      if (next >= row_b) break;
      r0 = next;
    }
  }

  tid = threadIdx.x;  // (anew: nothing made from it is held over the rows)
  asm volatile("" : "+v"(tid));
  float M, L, o;
  // (waves beyond the item's rows hold the empty state: they are not merged)
  block_merge<kWaves>(st, s_m, s_l, s_acc, min(kWaves, (n_rows + unit - 1) / unit), M, L, o, tid);

  if (n_active == 1) {  // the only split of this head: finish here
    if (tid < kHeadDim) {
      store_out(a.out, a.out_is_bf16, head, tid, o / L);
      if (a.lse && tid == 0) a.lse[head] = (M + log2f(L)) * kLn2;
    }
    return;
  }

  // Partials are exchanged through device-coherent (agent-scope) stores and loads, which go
  // straight to memory: no L2 write-back or invalidate of the whole cache is needed around the
  // arrival counter, only "my stores have completed" before the ticket is taken.  (This leans on
  // how gfx950 handles such accesses -- they are performed at the memory side in issue order once
  // s_waitcnt has seen them complete -- rather than on release / acquire fences, which here write
  // back and invalidate the whole L2 and made the kernel four times slower.)
  float *P = a.partials + (int64_t)head * a.splits * kPartialStride;
  if (tid < kHeadDim) {
    float *mine = P + (int64_t)split * kPartialStride;
    if (tid == 0) {
      __hip_atomic_store(mine + 0, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(mine + 1, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __hip_atomic_store(mine + 2 + tid, o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __builtin_amdgcn_s_waitcnt(0);  // all of this thread's memory operations have completed
  __syncthreads();
  // The split that arrives last merges all partials of the head (log-sum-exp merge).
  if (tid == 0) {
    const int ticket = __hip_atomic_fetch_add(&a.plan.done[head], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    (*s_last) = (ticket == n_active - 1);
  }
  __syncthreads();
  if (!(*s_last)) return;
  // Few partials are merged by a thread per dimension in the decode launch, whose light launches consist of them: 64 heads of
  // a budget, some 270 rows each, four layers 108.6 -> 106.3 us, 512 heads half of them flat, two layers 73.9 -> 73.3.  In the
  // selection's launch the code costs more than it saves (four layers of 32 flat heads over 32 k tokens 137.0 -> 139.1).
  if (!kCoherent && n_active <= kFewPartials) {
    if (tid < kHeadDim) merge_few(P, n_active, tid, M, L, o);
  } else {
    gather_partials<T>(P, n_active, st, tid & 15, tid >> 4);
    block_merge<kWaves>(st, s_m, s_l, s_acc, min(kWaves, (n_active + 3) / 4), M, L, o, tid);
  }
  if (tid < kHeadDim) {
    store_out(a.out, a.out_is_bf16, head, tid, o / L);
    if (a.lse && tid == 0) a.lse[head] = (M + log2f(L)) * kLn2;
  }
}

// The queue of a decode launch: the plan was written by an earlier launch.  A workgroup's first item is its block index,
// further items are claimed from the counter.  Call with the whole workgroup.
// s_first [kMaxQueueHeads + 1]: first item number of each head of this launch; s_scan [T / 64 + 1].
template <int T, bool kGathered>
__device__ __forceinline__ void decode_queue(const DecodeArgs &a, float *s_m, float *s_l, float (*s_acc)[kHeadDim],
                                             int *s_last, int *s_item, int *s_rows, int *s_first, int *s_scan) {
  const int tid = threadIdx.x;

  // ---- the queue: items per head from head_rows[], exclusive prefix in LDS ----
  // least chunks per item of a heavy launch: two 64-row units for every wave (256 heads, half of them flat, over 128 k
  // tokens: 166 us per step with one, 164.5 with two, 167.5 with four)
  constexpr int kMinItemChunks = T / 32;
  constexpr int kPer = kMaxQueueHeads / T;  // consecutive heads per thread
  int rows[kPer], chunks = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int hh = tid * kPer + u;
    // (an unconditional load at a clamped index, the value chosen afterwards: loads inside a condition are waited
    // for one by one, four dependent round trips at the start of every workgroup)
    const int got = a.plan.head_rows[a.head0 + min(hh, a.n_heads - 1)];
    rows[u] = hh < a.n_heads ? got : 0;  // <= 0: nothing to do (empty, or attended already)
    s_rows[hh] = rows[u];
    if (rows[u] > 0) chunks += min(1 << 20, (rows[u] + kChunkRows - 1) / kChunkRows);  // capped: the sum stays in range
  }
  // least chunks per item, between 1 and kMinItemChunks: the launch aims at about one item for every second workgroup
  const int all_chunks = block_sum<int, (T / 64)>(chunks, s_scan);
  const int half_grid = max(1, (int)gridDim.x / 2);
  const int g = min(kMinItemChunks, max(1, (all_chunks + half_grid - 1) / half_grid));
  int cnt[kPer], mine = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    int n = 0;
    if (rows[u] > 0) {
      const int c = rows_per_item(rows[u], a.splits, g);
      n = (rows[u] + c - 1) / c;
    }
    cnt[u] = n;
    mine += n;
  }
  int total;
  int run = block_excl_scan<int, (T / 64)>(mine, s_scan, total);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    s_first[tid * kPer + u] = run;
    run += cnt[u];
  }
  if (tid == T - 1) s_first[kMaxQueueHeads] = total;
  __syncthreads();
  if (total == 0) return;
#pragma unroll 1
  for (int item = blockIdx.x; item < total;) {
    // head that owns the item: the largest hh with s_first[hh] <= item (heads without items repeat the
    // next head's value, so the largest such hh is the one with s_first[hh + 1] > item)
    int lo = 0, hi = kMaxQueueHeads;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_first[mid] <= item) lo = mid; else hi = mid;
    }
    // (uniform: in scalar registers, and what is computed from them too)
    const int head = __builtin_amdgcn_readfirstlane(a.head0 + lo), split = __builtin_amdgcn_readfirstlane(item - s_first[lo]);
    const int R = __builtin_amdgcn_readfirstlane(s_rows[lo]);
    decode_item<T, kGathered, false>(a, head, split, R, rows_per_item(R, a.splits, g), s_m, s_l, s_acc, s_last);
    if (total <= (int)gridDim.x) break;  // every item had its workgroup: nothing to claim
    if (tid == 0)
      *s_item = gridDim.x + __hip_atomic_fetch_add(a.queue_next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();  // also: LDS is reused by the next item
    item = *s_item;
    __syncthreads();
  }
}

// The queue inside the selection's launch (at most kSameLaunchMaxHeads heads; s_rows[] holds their rows, 0 where there is
// nothing to do; call with the whole workgroup after a barrier).  The plan was written by workgroups of this same launch:
// it is read with device-coherent loads, and EVERY item is claimed from the counter (a workgroup may be missing): `first`
// is this workgroup's first claim, known to the last wave only.
// The rows are cut so that there is about one item for every workgroup that serves: helpers and heads that left rows.
// (Items of 512 rows, three or four of them for a workgroup, all waves in step at five barriers each, left the memory idle
// while an item began and ended: 32 flat heads over 8 x 131072 tokens, 94 us per step; now 74, of which the queue takes 45
// for 240 MB.)
template <int T>
__device__ __forceinline__ void decode_queue_here(const DecodeArgs &a, int first, float *s_m, float *s_l, float (*s_acc)[kHeadDim],
                                                  int *s_last, int *s_item, int *s_rows) {
  static_assert(kSameLaunchMaxHeads == 128, "two heads per lane");
  const int tid = threadIdx.x, lane = lane_id();
  // every wave works the cut out for itself
  const int R0 = s_rows[lane], R1 = s_rows[64 + lane];
  const int ch0 = (R0 + kChunkRows - 1) / kChunkRows, ch1 = (R1 + kChunkRows - 1) / kChunkRows;
  const int all = wave_sum(min(ch0, 1 << 23) + min(ch1, 1 << 23));
  const int n_left = __popcll(__ballot(R0 > 0)) + __popcll(__ballot(R1 > 0));
  const int helpers = max(1, (int)gridDim.x - a.n_heads), servers = helpers + n_left;
  // g chunks per item: all / helpers gives at most `servers` items (every head may add a short one); finer if that
  // already does
  int g = max(1, (all + helpers - 1) / helpers);
  int n0, n1, total;
  auto cut = [&](int gg) {
    const int c0 = rows_per_item(R0, a.splits, gg), c1 = rows_per_item(R1, a.splits, gg);
    n0 = R0 > 0 ? (R0 + c0 - 1) / c0 : 0;
    n1 = R1 > 0 ? (R1 + c1 - 1) / c1 : 0;
    total = wave_sum(n0 + n1);
  };
  {
    const int finer = max(1, (all + servers - 1) / servers);
    const int mid = (finer + g) / 2;
    cut(finer);
    if (total <= servers) {
      g = finer;
    } else {
      cut(mid);
      if (total <= servers) g = mid;
      else cut(g);
    }
  }
  const int i0 = wave_incl_scan(n0), i1 = wave_incl_scan(n1);
  const int f0 = i0 - n0, f1 = lane_u32((uint32_t)i0, 63) + i1 - n1;
  int item = first;
#pragma unroll 1
  for (;;) {
    if (tid == T - 64) *s_item = item;
    __syncthreads();  // also: LDS is reused by the next item
    item = __builtin_amdgcn_readfirstlane(*s_item);
    if (item >= total) return;
    const u64_t own0 = __ballot(item >= f0 && item < f0 + n0), own1 = __ballot(item >= f1 && item < f1 + n1);
    const int at = own0 ? __builtin_ctzll(own0) : __builtin_ctzll(own1);
    const int head = own0 ? at : 64 + at;
    const int R = __builtin_amdgcn_readlane(own0 ? R0 : R1, at);
    const int split = item - __builtin_amdgcn_readlane(own0 ? f0 : f1, at);
    // the next item is claimed before this one is attended
    int next = 0;
    if (tid == T - 64) next = __hip_atomic_fetch_add(a.queue_next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    decode_item<T, false, true>(a, head, split, R, rows_per_item(R, a.splits, g), s_m, s_l, s_acc, s_last);
    item = next;
    __syncthreads();
  }
}

}  // namespace dp
