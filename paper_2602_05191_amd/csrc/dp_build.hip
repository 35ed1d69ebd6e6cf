// Prefill side of the clustered cache (paper Sec. 4.1, Eq. 2): from K / V in
// token order and one cluster id per token, build what the decode step reads:
// the cluster-contiguous K / V rows, per-cluster sizes and offsets, the key
// centroids C_i (mean key) and the value aggregates V^Sigma_i and V-bar_i.
//
// A stable counting sort by cluster id with the segmented mean taken while the
// rows move.  HBM-bound: every K / V row is read once (a 256 B run at its token's
// place) and written once (clusters are written as contiguous runs); nothing
// is read back.  Everything is deterministic: counts are integers, a token's
// place inside its cluster is its token order, and the means are fp64 sums
// taken in row order and rounded once to bf16.
//
// The sort has two levels, so that its tables stay small: tokens are first put
// into bins of 16 consecutive clusters, in token order; the workgroup that moves a
// bin then orders the bin's tokens (some hundreds) by cluster itself.
//   rank     per 4096-token block: a token's rank among the earlier tokens of its
//            block in the same bin, and the block's count of every bin
//   scan     per segment: exclusive prefix of those counts over the blocks, and
//            of the bins' totals
//   place    position of a token = start of its bin + its bin's count in earlier
//            blocks + rank: the token's number and cluster go there
// (one kernel does all three for short segments)
//   move     a workgroup per bin orders the bin's tokens by cluster, walks the rows
//            (one contiguous run of the cache) in chunks, fetches each row's token,
//            stores it in place, and sums the chunk's rows column by column from a
//            copy in LDS
// A lane finds the earlier tokens of its bin (its cluster) inside its wave from one
// ballot per bit of the id; a wave takes its tokens in order and keeps a count of its
// own per bin.  So the cost does not depend on how the ids are distributed.
// (One level with a count per 1024-token block and cluster needed 33 MB of counts for
// 8 x 131072 tokens and 8192 clusters, and compared tokens of equal id pairwise: 64 us in
// four kernels in front of the move; the three kernels here take 25.)
// The update step of k-means (mean key of every cluster, nothing moved) is the same
// sequence with the cache pointers left null: the last kernel then fetches keys only and stores no row.
#include "dp_device.hpp"
#include "dp_kernels.hpp"

namespace dp {
namespace {

constexpr int kRankThreads = 1024, kRankWaves = kRankThreads / 64;
constexpr int kRankRounds = 4;                            // tokens per thread
constexpr int kBuildBlock = kRankThreads * kRankRounds;  // tokens per workgroup of the rank kernel
constexpr int kBinClusters = 16;

struct BuildArgs {
  const void *k_tokens, *v_tokens;
  const int32_t *assignment;
  const int64_t *seg_row_base;
  const int32_t *seg_rows, *seg_cluster_ptr;
  void *k_cache, *v_cache, *k_centroids, *v_centroids;
  int32_t *cluster_offsets, *cluster_sizes, *token_row;  // all nullable
  float *v_sums;                                         // nullable
  int32_t *hist;                                         // [n_seg, n_blocks, bin_stride]
  uint16_t *rank;                                        // [n_seg, max_rows], in the place of row_token until the move
  int32_t *bin_start;                                    // [n_seg, bin_stride + 1] (there is none if max_rows is 0)
  void *binned;                                          // [n_seg, max_rows]: 16 x token + cluster of the bin
  int32_t *row_token;                                    // [n_seg, max_rows]: token of each row, for runs too long for LDS
  int32_t n_blocks, bin_stride, max_kc, max_rows;
};

// LDS of one wave, read by lanes other than the writer: the wave's LDS operations execute in order, the compiler must
// keep them in order too.
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

__device__ __forceinline__ uint64_t lanes_below() { return (1ull << lane_id()) - 1; }

// ---- shared by the sort in three launches and the one in a single one ----

// a thread's tokens t0, t0 + 64, ..: their clusters, -1 for a token without a valid one
template <int R>
__device__ __forceinline__ void leave_out_invalid(const BuildArgs &a, int (&c)[R], int t0, int n, int kc, int64_t r0) {
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int t = t0 + 64 * u;
    if (t >= n || (unsigned)c[u] >= (unsigned)kc) {
      c[u] = -1;
      if (a.token_row && t < n) a.token_row[r0 + t] = -1;
    }
  }
}

// rank of each token among the wave's earlier tokens of its bin; mine: the wave's counts per bin, 0 so far
template <int R>
__device__ __forceinline__ void rank_in_bins(const int (&c)[R], int (&rank)[R], uint16_t *mine, int n_bins) {
  const int bits = n_bins > 1 ? 32 - __clz(n_bins - 1) : 0;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int bin = c[u] >> 4;
    const bool live = c[u] >= 0;
    uint64_t peers = __ballot(live);
    rank[u] = 0;
    if (peers == 0) continue;
    for (int b = 0; b < bits; ++b) {
      const bool bit = (bin >> b) & 1;
      const uint64_t ones = __ballot(bit);
      peers &= bit ? ones : ~ones;
    }
    const int before = live ? mine[bin] : 0;
    const int ahead = __popcll(peers & lanes_below());
    rank[u] = before + ahead;
    wave_lds_order();
    if (live && ahead == 0) mine[bin] = (uint16_t)(before + __popcll(peers));
    wave_lds_order();
  }
}

// exclusive prefix of a bin's counts over the waves, in place; returns their sum
template <int W>
__device__ __forceinline__ int prefix_over_waves(uint16_t *bin, int stride) {
  int run = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int v = bin[w * stride];
    bin[w * stride] = (uint16_t)run;
    run += v;
  }
  return run;
}

// clusters beyond the host's bound received no token: they are reported empty
template <int T>
__device__ __forceinline__ void report_unbounded_empty(const BuildArgs &a, int c0, int kc_all, int n_placed, int tid) {
  for (int i = a.max_kc + tid; i < kc_all; i += T) {
    if (a.cluster_offsets) a.cluster_offsets[c0 + i] = n_placed;
    if (a.cluster_sizes) a.cluster_sizes[c0 + i] = 0;
  }
}

__global__ __launch_bounds__(kRankThreads) void build_rank_kernel(BuildArgs a) {
  extern __shared__ uint32_t s_words[];  // 16-bit counts [kRankWaves][bin_stride]
  uint16_t *const tab = reinterpret_cast<uint16_t *>(s_words);
  const int seg = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x, wave = wave_id();
  const int n = min(a.seg_rows[seg], a.max_rows);
  if (blk * kBuildBlock >= n) return;
  const int c0 = a.seg_cluster_ptr[seg], kc = min(a.seg_cluster_ptr[seg + 1] - c0, a.max_kc);
  const int n_bins = (kc + kBinClusters - 1) / kBinClusters;
  const int64_t r0 = a.seg_row_base[seg];
  const int t0 = blk * kBuildBlock + wave * (64 * kRankRounds) + lane_id();  // a wave owns consecutive tokens
  int c[kRankRounds];
#pragma unroll
  for (int u = 0; u < kRankRounds; ++u) c[u] = a.assignment[r0 + min(t0 + 64 * u, n - 1)];
  for (int i = tid; i < kRankWaves * a.bin_stride / 2; i += kRankThreads) s_words[i] = 0;
  leave_out_invalid(a, c, t0, n, kc, r0);
  __syncthreads();
  uint16_t *const mine = tab + wave * a.bin_stride;
  int rank[kRankRounds];
  rank_in_bins(c, rank, mine, n_bins);
  __syncthreads();
  // per bin: exclusive prefix over the waves, in place; the block's count
  int32_t *row = a.hist + ((size_t)seg * a.n_blocks + blk) * a.bin_stride;
  for (int i = tid; i < n_bins; i += kRankThreads) row[i] = prefix_over_waves<kRankWaves>(tab + i, a.bin_stride);
  __syncthreads();
  uint16_t *out = a.rank + (size_t)seg * a.max_rows + t0;
#pragma unroll
  for (int u = 0; u < kRankRounds; ++u)
    if (c[u] >= 0) out[64 * u] = (uint16_t)(mine[c[u] >> 4] + rank[u]);
}

// T threads per segment: one wave where the bins of a segment fit it (2048 segments of 30 tokens: 21 -> 4.6 us).
template <int T>
__global__ __launch_bounds__(T) void build_scan_kernel(BuildArgs a) {
  __shared__ int scr[T / 64 + 1];
  const int seg = blockIdx.x, tid = threadIdx.x;
  const int c0 = a.seg_cluster_ptr[seg], kc_all = a.seg_cluster_ptr[seg + 1] - c0, kc = min(kc_all, a.max_kc);
  const int n_bins = (kc + kBinClusters - 1) / kBinClusters;
  const int n = min(a.seg_rows[seg], a.max_rows);
  const int blocks = (n + kBuildBlock - 1) / kBuildBlock;
  int32_t *start = a.bin_start + (size_t)seg * (a.bin_stride + 1);
  int carry = 0;
  for (int i0 = 0; i0 < (a.max_rows > 0 ? n_bins : 0); i0 += T) {
    const int i = i0 + tid;
    int run = 0;
    if (i < n_bins) {
      int32_t *h = a.hist + (size_t)seg * a.n_blocks * a.bin_stride + i;
      constexpr int kBatch = 16;  // independent loads in flight, then the running prefix
      for (int b0 = 0; b0 < blocks; b0 += kBatch) {
        int v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) v[u] = h[(size_t)min(b0 + u, blocks - 1) * a.bin_stride];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
          if (b0 + u < blocks) {
            h[(size_t)(b0 + u) * a.bin_stride] = run;
            run += v[u];
          }
      }
    }
    int tot;
    const int ex = block_excl_scan<int, T / 64>(run, scr, tot);
    if (i < n_bins) start[i] = carry + ex;
    carry += tot;
  }
  if (tid == 0 && a.max_rows > 0) start[n_bins] = carry;
  report_unbounded_empty<T>(a, c0, kc_all, carry, tid);
}

// The word of a token in its bin is 16 x token + cluster: 32 bits hold it for segments of less than kShortRows tokens.
constexpr int kShortRows = 1 << 28;

template <class Word>
__global__ __launch_bounds__(256) void build_place_kernel(BuildArgs a) {
  const int seg = blockIdx.y;
  const int n = min(a.seg_rows[seg], a.max_rows);
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= n) return;
  const int c0 = a.seg_cluster_ptr[seg], kc = min(a.seg_cluster_ptr[seg + 1] - c0, a.max_kc);
  const int c = a.assignment[a.seg_row_base[seg] + t];
  const int rank = a.rank[(size_t)seg * a.max_rows + t];  // (undefined for a token that is left out)
  if ((unsigned)c >= (unsigned)kc) return;
  const int bin = c / kBinClusters;
  const int at = a.bin_start[(size_t)seg * (a.bin_stride + 1) + bin] +
                 a.hist[((size_t)seg * a.n_blocks + t / kBuildBlock) * a.bin_stride + bin] + rank;
  static_cast<Word *>(a.binned)[(size_t)seg * a.max_rows + at] = (Word)t * kBinClusters + (Word)(c % kBinClusters);
}

// rank, scan and place of a segment of at most T * R tokens by one workgroup: the counts stay in LDS and a token's cluster and
// rank in registers.  Bounded by latency (the ids in, the words out; a few LDS round trips per 64 tokens of a wave): 24
// segments of 1.2 k to 5 k tokens take 7.2 us, in three launches they took 5.0, 4.1 and 3.0 and the gaps between.
template <int T, int R>
__global__ __launch_bounds__(T) void build_sort_kernel(BuildArgs a) {
  extern __shared__ uint32_t s_words[];  // 16-bit counts [T / 64][bin_stride], then the starts of the bins
  __shared__ int scr[T / 64 + 1];
  constexpr int kWaves = T / 64;
  uint16_t *const tab = reinterpret_cast<uint16_t *>(s_words);
  int *const s_start = reinterpret_cast<int *>(s_words + kWaves * a.bin_stride / 2);
  const int seg = blockIdx.x, tid = threadIdx.x, wave = wave_id();
  const int n = min(a.seg_rows[seg], a.max_rows);
  const int c0 = a.seg_cluster_ptr[seg], kc_all = a.seg_cluster_ptr[seg + 1] - c0, kc = min(kc_all, a.max_kc);
  const int n_bins = (kc + kBinClusters - 1) / kBinClusters;
  const int64_t r0 = a.seg_row_base[seg];
  const int t0 = wave * (64 * R) + lane_id();  // a wave owns consecutive tokens
  int c[R], rank[R];
#pragma unroll
  for (int u = 0; u < R; ++u) c[u] = -1;
  if (n > 0) {
#pragma unroll
    for (int u = 0; u < R; ++u) c[u] = a.assignment[r0 + min(t0 + 64 * u, n - 1)];
  }
  for (int i = tid; i < kWaves * a.bin_stride / 2; i += T) s_words[i] = 0;
  leave_out_invalid(a, c, t0, n, kc, r0);
  __syncthreads();
  uint16_t *const mine = tab + wave * a.bin_stride;
  rank_in_bins(c, rank, mine, n_bins);
  __syncthreads();
  int32_t *start = a.bin_start + (size_t)seg * (a.bin_stride + 1);
  int carry = 0;
  for (int i0 = 0; i0 < n_bins; i0 += T) {
    const int i = i0 + tid;
    const int run = i < n_bins ? prefix_over_waves<kWaves>(tab + i, a.bin_stride) : 0;
    int tot;
    const int ex = block_excl_scan<int, kWaves>(run, scr, tot);
    if (i < n_bins) start[i] = s_start[i] = carry + ex;
    carry += tot;
  }
  if (tid == 0) start[n_bins] = carry;
  report_unbounded_empty<T>(a, c0, kc_all, carry, tid);
  __syncthreads();
  uint32_t *out = static_cast<uint32_t *>(a.binned) + (size_t)seg * a.max_rows;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    if (c[u] < 0) continue;
    const int bin = c[u] >> 4;
    out[s_start[bin] + mine[bin] + rank[u]] = (uint32_t)(t0 + 64 * u) * kBinClusters + (uint32_t)(c[u] % kBinClusters);
  }
}

// double -> bf16 bits with ONE rounding to 8 significant bits, ties to even.  Values whose magnitude
// is below the bf16 normal range go through float (two roundings, irrelevant at 1e-38).
__device__ __forceinline__ uint32_t f64_to_bf16_rne(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const int e = (int)((u >> 52) & 0x7ff) - 1023 + 127;  // bf16 / float exponent field
  if (e <= 0 || e >= 255) return f32_to_bf16_rne((float)x);
  const unsigned long long man = u & 0xfffffffffffffull;
  unsigned long long top = man >> 45;                   // 7 explicit mantissa bits
  const unsigned long long rest = man & ((1ull << 45) - 1), half = 1ull << 44;
  uint32_t bits = ((uint32_t)(u >> 63) << 15) | ((uint32_t)e << 7) | (uint32_t)top;
  if (rest > half || (rest == half && (top & 1))) bits += 1;  // a carry runs into the exponent, as it should
  return bits;
}

// The move.  A workgroup owns a bin of 16 consecutive clusters, whose rows are one contiguous run of the cache.  It
// first orders the bin's tokens by cluster (stable: a wave takes a consecutive share of the bin's list, 64 tokens at a
// time; lane i < 16 counts cluster i); the list stays in LDS, or in global memory when the run is too long for that.
// The run is then taken in chunks of 64 rows: the sixteen 16-lane rows of the workgroup fetch four rows each (whatever
// the sizes of the clusters, every lane has the same number of loads in flight), leave a copy in LDS and store them in
// place; the next chunk's rows are fetched while the chunk is summed.  Thread d sums column d (key dimensions, then
// value dimensions) of the chunk's rows in row order, in fp64, and writes a cluster's means when its last row has gone
// by.  A sum carries over from chunk to chunk.
// One long run is one workgroup's serial work (a cluster of 131072 tokens: 2048 chunks of 2.4 us), so nothing in it
// may wait in turn: the list is read in batches, one ahead, the tokens of a chunk come a chunk before its rows and the
// rows a chunk before they are summed (all tokens of 8 segments in one cluster each: 6311 -> 5025 us; half of them 3812 ->
// 2659; with the list read in front of every chunk's rows these were slower than the one-level sort: 5390, 2860).
// Rows go by once: non-temporal loads and stores (move of 8 x 131072 tokens 228 -> 215 us = 5.2 TB/s over 1.11 GB; a
// plain copy of 2 GB runs at 4.7 TB/s on the same card).
// kMove = false: keys only (the update step of k-means): nothing is stored in place, no value is read, the two halves
// of the workgroup take the clusters in turn, and a cluster without tokens keeps the centroid it has.
constexpr int kMoveRows = 64;
constexpr int kListRows = 1024;  // longest run whose list stays in LDS

template <bool kMove, class Word>
__global__ __launch_bounds__(256) void build_move_kernel(BuildArgs a) {
  constexpr int kCols = kMove ? 2 * kHeadDim : kHeadDim;
  __shared__ __align__(16) uint16_t s_rows[kMoveRows][kCols];  // key | value of every row of the chunk
  __shared__ int s_list[kListRows];
  __shared__ int s_cnt[4][kBinClusters];
  const int seg = blockIdx.y, bin = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int c0 = a.seg_cluster_ptr[seg], kc = min(a.seg_cluster_ptr[seg + 1] - c0, a.max_kc);
  const int64_t r0 = a.seg_row_base[seg];
  const int cf = bin * kBinClusters;
  if (cf >= kc) return;
  const int ncl = min(kBinClusters, kc - cf);
  const int lane16 = tid & 15, grp = tid >> 4;
  const int32_t *start = a.bin_start + (size_t)seg * (a.bin_stride + 1) + bin;
  const int run0 = a.max_rows > 0 ? start[0] : 0, n_run = a.max_rows > 0 ? start[1] - run0 : 0;
  const Word *binned = static_cast<const Word *>(a.binned) + (size_t)seg * a.max_rows + run0;
  int32_t *far_list = a.row_token + (size_t)seg * a.max_rows + run0;
  const bool in_lds = n_run <= kListRows;

  // ---- order the bin's tokens by cluster ----
  const int share = 64 * ((n_run + 255) / 256), j0 = wave * share, j1 = min(n_run, j0 + share);
  // the lanes of the wave that hold a token of cluster v, from the ballots of the id's four bits
  struct Ballots {
    uint64_t live, bit[4];
    __device__ __forceinline__ uint64_t of(int v) const {
      uint64_t m = live;
#pragma unroll
      for (int b = 0; b < 4; ++b) m &= ((v >> b) & 1) ? bit[b] : ~bit[b];
      return m;
    }
  };
  auto ballots = [&](Word word, bool live) {
    Ballots s;
    s.live = __ballot(live);
#pragma unroll
    for (int b = 0; b < 4; ++b) s.bit[b] = __ballot((word >> b) & 1);
    return s;
  };
  // The wave's share, 64 words at a time: the first kKeep of a lane stay in registers from the first pass to the second,
  // the others are loaded kAhead at a time, one batch ahead.
  constexpr int kKeep = 2, kAhead = 8;
  Word kept[kKeep];
  auto word_at = [&](int u) { return binned[min(j0 + 64 * u + lane, n_run - 1)]; };
#pragma unroll
  for (int u = 0; u < kKeep; ++u) kept[u] = n_run > 0 ? word_at(u) : 0;
  auto each_word = [&](auto use) {  // use(word, whether it is one of the share)
#pragma unroll
    for (int u = 0; u < kKeep; ++u)
      if (j0 + 64 * u < j1) use(kept[u], j0 + 64 * u + lane < j1);
    if (j0 + 64 * kKeep >= j1) return;
    Word w[kAhead], next[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) next[k] = word_at(kKeep + k);
    for (int u0 = kKeep; j0 + 64 * u0 < j1; u0 += kAhead) {
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        w[k] = next[k];
        next[k] = word_at(u0 + kAhead + k);
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
        if (j0 + 64 * (u0 + k) < j1) use(w[k], j0 + 64 * (u0 + k) + lane < j1);
    }
  };
  int count = 0;
  each_word([&](Word word, bool live) { count += __popcll(ballots(word, live).of(lane16)); });
  if (lane < kBinClusters) s_cnt[wave][lane] = count;
  __syncthreads();
  int sz = 0, before = 0;  // of cluster lane16, in every 16-lane row: its size; its tokens in earlier waves' shares
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int v = s_cnt[w][lane16];
    sz += v;
    before += w < wave ? v : 0;
  }
  const int my_end = row16_incl_scan(sz), my_off = my_end - sz;  // where the cluster lies inside the run
  int next = my_off + before;
  each_word([&](Word word, bool live) {
    const Ballots s = ballots(word, live);
    const int v = (int)(word & (kBinClusters - 1)), t = (int)(word / kBinClusters);
    const int dest = __shfl(next, v, 16) + __popcll(s.of(v) & lanes_below());
    next += __popcll(s.of(lane16));
    if (live) {
      if (in_lds) s_list[dest] = t;
      else far_list[dest] = t;
      if (a.token_row) a.token_row[r0 + t] = run0 + dest;
    }
  });
  if (tid < ncl) {
    if (a.cluster_offsets) a.cluster_offsets[c0 + cf + tid] = run0 + my_off;
    if (a.cluster_sizes) a.cluster_sizes[c0 + cf + tid] = sz;
  }
  if (in_lds) lds_barrier();
  else __syncthreads();  // (waits for the list's stores)

  // ---- fetch, store in place, sum ----
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 kr[4], vr[4];
  // Lanes u, u + 4, ... of a 16-lane row: the token of the row's u-th share of the chunk (row 16 u + grp); shares beyond
  // the run repeat its last row and are not stored.
  auto token_of = [&](int base) {
    const int j = min(base + 16 * (lane16 & 3) + grp, n_run - 1);
    int t = s_list[min(j, kListRows - 1)];
    // (two loads: merged into one through a flat address they would be waited for at the next LDS barrier)
    asm volatile("" : "+v"(t));
    if (!in_lds) t = far_list[j];
    return t;
  };
  auto fetch = [&](int tokens, u32x4 (&kr)[4], u32x4 (&vr)[4]) {
    const int t[4] = {(int)dpp_mov_u32<0x00>((uint32_t)tokens), (int)dpp_mov_u32<0x55>((uint32_t)tokens),
                      (int)dpp_mov_u32<0xAA>((uint32_t)tokens), (int)dpp_mov_u32<0xFF>((uint32_t)tokens)};  // of the quad
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t at = (r0 + t[u]) * kRowBytes + lane16 * 16;
      const u32x4 *k = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.k_tokens) + at);
      // (the keys-only form reads rows that the next round reads again: plain loads, so that they may stay cached)
      kr[u] = kMove ? __builtin_nontemporal_load(k) : *k;
      if (kMove)
        vr[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.v_tokens) + at));
    }
  };
  auto flush = [&](int c, int s, double sum) {
    if (!kMove && s == 0) return;
    const uint32_t bits = s > 0 ? f64_to_bf16_rne(sum / (double)s) : 0u;
    const size_t o = (size_t)(c0 + cf + c) * kHeadDim;
    if (!kMove) {
      static_cast<uint16_t *>(a.k_centroids)[o + (tid & (kHeadDim - 1))] = (uint16_t)bits;
    } else if (tid < kHeadDim) {
      static_cast<uint16_t *>(a.k_centroids)[o + tid] = (uint16_t)bits;
    } else {
      static_cast<uint16_t *>(a.v_centroids)[o + tid - kHeadDim] = (uint16_t)bits;
      if (a.v_sums) a.v_sums[o + tid - kHeadDim] = (float)sum;
    }
  };
  const int col = kMove ? tid : tid & (kHeadDim - 1);
  constexpr int kStep = kMove ? 1 : 2;
  double acc = 0.0;
  // the cluster whose rows are being summed: the same in every thread (of a half)
  int cur = kMove ? 0 : __builtin_amdgcn_readfirstlane(tid / kHeadDim);
  int cur_off, cur_end;
  auto bounds = [&]() {
    cur_off = __builtin_amdgcn_readfirstlane(__shfl(my_off, cur & 15, 16));
    cur_end = __builtin_amdgcn_readfirstlane(__shfl(my_end, cur & 15, 16));
  };
  bounds();
  int tokens = 0;
  if (n_run > 0) {
    fetch(token_of(0), kr, vr);
    tokens = token_of(kMoveRows);
  }
  for (int base = 0; base < n_run; base += kMoveRows) {
    const int nb = min(kMoveRows, n_run - base);
    lds_barrier();  // the previous chunk has been summed
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      *reinterpret_cast<u32x4 *>(&s_rows[16 * u + grp][lane16 * 8]) = kr[u];
      if constexpr (kMove) *reinterpret_cast<u32x4 *>(&s_rows[16 * u + grp][kHeadDim + lane16 * 8]) = vr[u];
    }
    asm volatile("" : "+v"(tokens));  // arrived, too (loaded behind the rows): no wait for them behind the stores
    if constexpr (kMove) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // after the copies: a wait placed behind a store would wait for the store
        const int j = 16 * u + grp;
        if (j < nb) {
          const int64_t at = (r0 + run0 + base + j) * kRowBytes + lane16 * 16;
          __builtin_nontemporal_store(kr[u], reinterpret_cast<u32x4 *>(static_cast<char *>(a.k_cache) + at));
          __builtin_nontemporal_store(vr[u], reinterpret_cast<u32x4 *>(static_cast<char *>(a.v_cache) + at));
        }
      }
    }
    if (base + kMoveRows < n_run) {  // in flight while this chunk is summed, with the tokens of the chunk after it
      fetch(tokens, kr, vr);
      tokens = token_of(base + 2 * kMoveRows);
    }
    lds_barrier();
    while (cur < ncl) {
      int j = max(cur_off - base, 0);
      const int hi = min(cur_end - base, nb);
      for (; j + 8 <= hi; j += 8) {
        uint16_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = s_rows[j + u][col];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += (double)__uint_as_float((uint32_t)x[u] << 16);
      }
      for (; j < hi; ++j) acc += (double)__uint_as_float((uint32_t)s_rows[j][col] << 16);
      if (cur_end - base > nb) break;  // the cluster goes on in the next chunk
      flush(cur, cur_end - cur_off, acc);
      acc = 0.0;
      cur += kStep;
      bounds();
    }
  }
  for (; cur < ncl; cur += kStep)  // a workgroup without rows: its clusters are empty
    flush(cur, 0, 0.0);
}

struct BuildLayout {
  size_t hist, row_token, bin_start, binned, total;  // byte offsets
  int n_blocks, bin_stride;
};
BuildLayout layout_of(int n_seg, int max_rows, int max_kc) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t rows = (size_t)n_seg * max_rows, word = max_rows < kShortRows ? sizeof(uint32_t) : sizeof(uint64_t);
  BuildLayout L;
  L.n_blocks = (int)(((int64_t)max_rows + kBuildBlock - 1) / kBuildBlock);
  L.bin_stride = ((max_kc + kBinClusters - 1) / kBinClusters + 1) / 2 * 2;  // even: the tables are cleared word by word
  L.hist = 0;
  L.row_token = up((size_t)n_seg * L.n_blocks * L.bin_stride * sizeof(int32_t));
  L.bin_start = L.row_token + up(rows * sizeof(int32_t));  // (the ranks lie where row_token comes: half of it)
  L.binned = L.bin_start + up((size_t)n_seg * (L.bin_stride + 1) * sizeof(int32_t));
  L.total = L.binned + up(rows * word);
  return L;
}

template <class Word>
void place(const BuildArgs &a, int n_seg, hipStream_t s) {
  if (a.max_rows > 0 && a.max_kc > 0)
    hipLaunchKernelGGL(build_place_kernel<Word>, dim3(((unsigned)a.max_rows + 255) / 256, n_seg), dim3(256), 0, s, a);
}
template <class Word>
void move(const BuildArgs &a, int n_seg, hipStream_t s) {
  if (a.max_kc == 0) return;
  const dim3 grid((a.max_kc + kBinClusters - 1) / kBinClusters, n_seg);
  if (a.k_cache) hipLaunchKernelGGL((build_move_kernel<true, Word>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((build_move_kernel<false, Word>), grid, dim3(256), 0, s, a);
}
template <int T, int R>
void sort_short(const BuildArgs &a, int n_seg, hipStream_t s) {
  const size_t lds = (size_t)a.bin_stride * (T / 64 * sizeof(uint16_t) + sizeof(int));
  hipLaunchKernelGGL((build_sort_kernel<T, R>), dim3(n_seg), dim3(T), lds, s, a);
}

}  // namespace

// (without rows nothing is sorted: no workspace)
size_t build_workspace_bytes(int n_seg, int max_rows, int max_kc) {
  return max_rows > 0 ? layout_of(n_seg, max_rows, max_kc).total : 0;
}

hipError_t launch_build(const BuildProblem &p, void *workspace, hipStream_t s) {
  if (p.n_seg == 0) return hipSuccess;
  const BuildLayout L = layout_of(p.n_seg, p.max_rows, p.max_kc);
  char *ws = static_cast<char *>(workspace);
  BuildArgs a;
  a.k_tokens = p.k_tokens;
  a.v_tokens = p.v_tokens;
  a.assignment = p.assignment;
  a.seg_row_base = p.seg_row_base;
  a.seg_rows = p.seg_rows;
  a.seg_cluster_ptr = p.seg_cluster_ptr;
  a.k_cache = p.k_cache;
  a.v_cache = p.v_cache;
  a.k_centroids = p.k_centroids;
  a.v_centroids = p.v_centroids;
  a.cluster_offsets = p.cluster_offsets;
  a.cluster_sizes = p.cluster_sizes;
  a.token_row = p.token_row;
  a.v_sums = p.v_sums;
  a.hist = reinterpret_cast<int32_t *>(ws + L.hist);
  a.rank = reinterpret_cast<uint16_t *>(ws + L.row_token);
  a.bin_start = reinterpret_cast<int32_t *>(ws + L.bin_start);
  a.binned = ws + L.binned;
  a.row_token = reinterpret_cast<int32_t *>(ws + L.row_token);
  a.n_blocks = L.n_blocks;
  a.bin_stride = L.bin_stride;
  a.max_kc = p.max_kc;
  a.max_rows = p.max_rows;
  // Short segments are sorted by a workgroup each, us per call against three launches: one segment of 2048 tokens 21.3 / 26.0,
  // 20 of 3644 31.2 / 35.9, 24 of up to 7000 44.0 / 46.4, 128 of up to 2300 54.3 / 59.9, 128 of up to 8000 144.7 / 148.7, 8 of
  // 8100 28.7 / 30.2.  The gain shrinks with the length, which one CU works through alone, so longer ones keep the three;
  // and tables of many clusters would take more LDS than leaves room for a second workgroup.
  if (p.max_rows > 0 && p.max_rows <= 8192 && L.bin_stride > 0 && L.bin_stride <= 512) {
    if (p.max_rows <= 1024) sort_short<256, 4>(a, p.n_seg, s);
    else if (p.max_rows <= 4096) sort_short<1024, 4>(a, p.n_seg, s);
    else sort_short<1024, 8>(a, p.n_seg, s);
    move<uint32_t>(a, p.n_seg, s);
    return hipGetLastError();
  }
  if (L.n_blocks > 0 && (L.bin_stride > 0 || p.token_row)) {  // (no cluster at all: every token is left out)
    // a count per wave and bin lives in LDS: 2 bytes per cluster of the longest segment (128 KB at the 65536 limit)
    const size_t lds = (size_t)kRankWaves * L.bin_stride * sizeof(uint16_t);
    if (lds > 32768) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(build_rank_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(build_rank_kernel, dim3(L.n_blocks, p.n_seg), dim3(kRankThreads), lds, s, a);
  }
  if (L.bin_stride <= 64) hipLaunchKernelGGL(build_scan_kernel<64>, dim3(p.n_seg), dim3(64), 0, s, a);
  else hipLaunchKernelGGL(build_scan_kernel<1024>, dim3(p.n_seg), dim3(1024), 0, s, a);
  if (p.max_rows < kShortRows) {
    place<uint32_t>(a, p.n_seg, s);
    move<uint32_t>(a, p.n_seg, s);
  } else {
    place<uint64_t>(a, p.n_seg, s);
    move<uint64_t>(a, p.n_seg, s);
  }
  return hipGetLastError();
}

}  // namespace dp
