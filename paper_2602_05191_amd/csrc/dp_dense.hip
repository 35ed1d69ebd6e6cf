// Dense decode attention over every token of a KV segment (paper Sec. 2.1,
// Eq. 1): the full-attention baseline that the paper's efficiency figures are
// measured against (Sec. 5.3).
//
// HBM-bound streaming kernel (512 B per token).  The K and V rows of a segment are
// contiguous, so a workgroup streams a range of rows once and scores each row against
// up to 16 query heads of the GQA group at once: the cache is read once per KV head.  Both contractions run on the matrix cores, and the
// operands go from global memory straight into the instructions' register layouts,
// with nothing exchanged between lanes and nothing staged in LDS:
//   scores  S[16 rows x 16 heads] = K Q^T, four v_mfma_f32_16x16x32_bf16.  Lane l
//           loads chunks l / 16 + 4 j of key row l % 16 (64 contiguous bytes of 16
//           rows per load instruction); it receives the scores of head l % 16 for
//           rows 4 (l / 16) + i, i = 0 .. 3, and turns them into weights in place.
//   output  O^T[dims x heads] += V^T P^T, v_mfma_f32_16x16x4_f32 with k = l / 16
//           standing for row 4 (l / 16) + i: the weight operand is the register that
//           the scores left, unrounded, and the value operand of lane l is element
//           l % 16 of row 4 (l / 16) + i.  "Element" may be any 16 dimensions as long as
//           the output is read back alike: load instruction i fetches 16 B per lane
//           (whole rows, dims 8 (l % 16) .. + 7), and its n-th value widened to fp32 is
//           the operand of the n-th of eight output tiles.
// Precision: scores are four products over 32 dimensions summed pairwise (4.7e-8 of their size against fp64; one chain
// through the four instructions: 5.9e-8), scaled inside the subtraction of the maximum (one rounding less).  An fp32
// matrix instruction adds its four rows one after the other, so a tile's 16 rows are summed by themselves and added to
// the accumulator: its chain is as long as the wave has tiles, not rows (output against fp64, 131072 rows x 8 KV heads:
// 4.1e-7 -> 1.7e-7 with flat weights, 1.0e-6 -> 5.0e-7 with scores of deviation 3; the vector-ALU form had 3.0e-7 and
// 6.5e-7).
// The running maximum of a head is the same in the four lanes that hold it, so the
// rescaling of the accumulators is lane-local; it is skipped while no maximum moves.
// Values that are not finite stay where they belong: a row that is loaded in place of one past the range has its
// value replaced by zero (an infinite value times the weight 0 would be NaN); a maximum of -inf (no row yet, or only
// rows that score -inf) is taken as the lowest finite number when it is subtracted (-inf - -inf would be NaN); weights
// keep the range below 2^-126 (exp2f, not the bare instruction, which flushes it: a value of 1e38 there still counts).
// Matrix-core time per 16 rows: 4 x 16 + 32 x 32 cycles, whatever the group size is:
// 29 us at 2.4 GHz for the million rows of 8 x 131072 tokens, behind 87 us of HBM
// time at 6.2 TB/s.  Measured there at G = 4: 81 us = 6.6 TB/s (87 us = 6.1 TB/s over
// buffers in turn that no cache holds a part of); with plain loads 95 (111 us with the dot
// products, G softmaxes per row in 16 lanes each and G x 128 multiply-adds per row on the
// vector ALU; that form was vector-bound at G = 8).  Calls of one to five thousand rows per
// segment at G = 1 are up to 15 % (one of 5003 x 8: 20 %) slower than that form was where the
// rows come from the caches (40 x 1024 tokens x 8 KV heads 34.2 against 30.1 us, 8 x 2048
// 17.1 / 16.8), not where they come from HBM (8 x 1024 12.5 / 13.7, 5003 x 8 14.6 / 14.6;
// 2400 segments of 64 rows 23.0 / 21.4).
// Work split: the segments' rows, in chunks of 64, are dealt out evenly to one round of resident workgroups, whatever
// the lengths of the segments (the lengths are on the device: every wave derives its share from them).  A share may end
// one segment and begin the next (three segments of 24 to 45 k tokens x 8 KV heads, G = 8: 83 -> 73.5 us against equal
// ranges of the longest segment).  The partials (m, l, acc[128]) of the pieces of a segment are merged by a second small
// kernel: no counters, no atomics.  Short or very many segments are taken whole, a workgroup each, which then writes the
// output itself: one launch.
#include <type_traits>

#include "dp_attend.hpp"
#include "dp_device.hpp"
#include "dp_kernels.hpp"

namespace dp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDenseThreads = 256;
constexpr int kDenseWaves = kDenseThreads / 64;
constexpr int kDenseHeads = 16;  // query heads per pass: the columns of one MFMA tile
constexpr int kDenseTile = 16;   // cache rows per wave and step
constexpr int kPartialStride = kHeadDim + 2;

struct DenseArgs {
  const void *q, *k_cache, *v_cache;
  const int64_t *seg_row_base;
  const int32_t *seg_rows;
  float *partials;  // [nh, splits, kPartialStride]
  void *out;
  float *lse;  // nullable
  int32_t n_seg, n_kv_heads, n_q_heads, group;
  int32_t head0;  // this launch serves heads [head0, head0 + 16) of every group
  int32_t splits;            // partial slots per head
  int32_t min_share, grid;   // chunks dealt out: fewest per workgroup, workgroups
  int32_t whole;             // nothing dealt out: a workgroup per segment
  int32_t max_rows, out_is_bf16;
  float scale_log2;
};

constexpr int kDealtSegs = 64 * 64;  // most segments that the lookup can hold

__device__ __forceinline__ int dense_rows(const DenseArgs &a, int seg) { return max(0, min(a.seg_rows[seg], a.max_rows)); }
__device__ __forceinline__ int dense_chunks(int rows) { return (rows + kChunkRows - 1) / kChunkRows; }

// The chunks of all segments, numbered through in segment order: workgroup w takes chunks [w share, (w + 1) share).
__device__ __forceinline__ int dealt_share(const DenseArgs &a, int total) {
  return max(a.min_share, (total + a.grid - 1) / a.grid);
}
// The segment that holds chunk c = blockIdx.x * share, by every wave for itself: a lane adds up `per` consecutive
// segments, then the lane that holds the chunk has its segments spread over the lanes.  The row base comes along, so that
// nothing but the rows themselves is left to wait for.  false: no chunk is left.
struct DenseStart {
  int seg, first, rows;  // segment, its first chunk, its rows
  int64_t row0;
  int c, c_end, share;   // the workgroup's chunks
};
__device__ __forceinline__ bool dense_start(const DenseArgs &a, DenseStart &d) {
  const int lane = lane_id(), per = (a.n_seg + 63) / 64;
  int rows = 0, mine = 0;
  int64_t base = 0;
  auto look = [&](int seg, bool valid) {
    const int s = min(seg, a.n_seg - 1);
    rows = dense_rows(a, s);
    base = a.seg_row_base[s];
    return valid && seg < a.n_seg ? dense_chunks(rows) : 0;
  };
  if (per == 1) {
    mine = look(lane, true);
  } else {
#pragma unroll 4
    for (int u = 0; u < per; ++u) {
      const int seg = lane * per + u, n = dense_chunks(dense_rows(a, min(seg, a.n_seg - 1)));
      mine += seg < a.n_seg ? n : 0;
    }
  }
  int upto = wave_incl_scan(mine);
  const int total = (int)lane_u32((uint32_t)upto, 63);
  d.share = dealt_share(a, total);
  d.c = blockIdx.x * d.share;
  d.c_end = min(total, d.c + d.share);
  if (d.c >= d.c_end) return false;
  int at = __builtin_ctzll(__ballot(upto - mine <= d.c && d.c < upto));
  d.seg = at * per;
  d.first = (int)lane_u32((uint32_t)(upto - mine), at);
  if (per > 1) {
    mine = look(d.seg + lane, lane < per);
    upto = d.first + wave_incl_scan(mine);
    at = __builtin_ctzll(__ballot(upto - mine <= d.c && d.c < upto));
    d.seg += at;
    d.first = (int)lane_u32((uint32_t)(upto - mine), at);
  }
  d.rows = (int)lane_u32((uint32_t)rows, at);
  d.row0 = (int64_t)lane_u64((unsigned long long)base, at);
  return true;
}

// Number of pieces of segment my_seg (which has rows), by every wave for itself.
__device__ __forceinline__ int dense_pieces(const DenseArgs &a, int my_seg, int chunks) {
  int total = 0, first = 0;
#pragma unroll 4
  for (int u = 0; u < a.n_seg; u += 64) {
    const int seg = u + lane_id(), rows = dense_rows(a, min(seg, a.n_seg - 1));
    const int n = seg < a.n_seg ? dense_chunks(rows) : 0;
    total += n;
    first += seg < my_seg ? n : 0;
  }
  total = wave_sum(total);
  first = wave_sum(first);
  const int share = dealt_share(a, total);
  return (first + chunks - 1) / share - first / share + 1;
}

// what is subtracted from a score whose running maximum is m
__device__ __forceinline__ float finite_max(float m) { return fmaxf(m, -3.402823466e38f); }

// one wave's 16 cache rows as the two contractions want them
struct DenseTile {
  uint4 k[4], v[4];
};

// Rows beyond the range read its last row: a lane's loads never leave the segment, and their weight and values are
// made zero before they are used.
// (row0 and t are uniform in the wave: the tile's base is a scalar, a lane adds a 32-bit offset.)
__device__ __forceinline__ void load_dense_tile(const DenseArgs &a, int64_t row0, int t, int last, int r, int kq,
                                                DenseTile &d) {
  const int base = min(t, last), more = last - base;
  const char *k = static_cast<const char *>(a.k_cache) + (row0 + base) * kRowBytes;
  const char *v = static_cast<const char *>(a.v_cache) + (row0 + base) * kRowBytes;
  const uint32_t ko = (uint32_t)min(r, more) * kRowBytes + kq * 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) d.k[j] = load_stream16(k + (ko + j * 64));
#pragma unroll
  for (int i = 0; i < 4; ++i) d.v[i] = load_stream16(v + ((uint32_t)min(4 * kq + i, more) * kRowBytes + r * 16));
}

__global__ __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void dense_kernel(DenseArgs a) {
  __shared__ float s_m[kDenseWaves][kDenseHeads], s_l[kDenseWaves][kDenseHeads];
  __shared__ __align__(16) float s_acc[kDenseWaves][kDenseHeads][kHeadDim + 4];
  const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
  const int r = lane & 15, kq = lane >> 4;
  const int n_live = min(kDenseHeads, a.group - a.head0);
  DenseStart at;
  if (a.whole) {
    at.seg = blockIdx.x;
    at.rows = dense_rows(a, at.seg);
    at.row0 = a.seg_row_base[at.seg];
    at.first = at.c = 0;
    at.c_end = dense_chunks(at.rows);
    at.share = 1;
    if (at.rows == 0) {  // zero output
      const int64_t head = (int64_t)(at.seg / a.n_kv_heads) * a.n_q_heads + at.seg % a.n_kv_heads * a.group + a.head0;
      for (int j = tid / kHeadDim; j < n_live; j += kDenseThreads / kHeadDim) {
        store_out(a.out, a.out_is_bf16, head + j, tid % kHeadDim, 0.f);
        if (a.lse && tid % kHeadDim == 0) a.lse[head + j] = -INFINITY;
      }
      return;
    }
  } else if (!dense_start(a, at)) {
    return;
  }
  int seg = at.seg, first = at.first, R = at.rows, c0 = at.c;
  int64_t row0 = at.row0;
  const int c_end = at.c_end, share = at.share;

  // one piece of a segment after the other, usually one
  while (true) {
    const int seg_end = first + dense_chunks(R);
    const int ra = (c0 - first) * kChunkRows, rb = min(R, (min(c_end, seg_end) - first) * kChunkRows);
    const int split = blockIdx.x - first / share;  // number of the piece inside its segment
    c0 = seg_end;
    first = seg_end;
    const int b = seg / a.n_kv_heads, g = seg % a.n_kv_heads;
    const int64_t head_first = (int64_t)b * a.n_q_heads + g * a.group + a.head0;

    // query head r of the pass (beyond the group: its last head again, not stored), chunks kq + 4 j
    uint4 Q[4];
    {
      const char *row = static_cast<const char *>(a.q) + (head_first + min(r, n_live - 1)) * kRowBytes + kq * 16;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        Q[j] = *reinterpret_cast<const uint4 *>(row + j * 64);
    }
    f32x4 acc[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;  // head r: the maximum of all rows so far, the weights of this lane's rows

    // (rows beyond the range exist in a wave's last tile only)
    auto attend = [&](DenseTile &d, int t, auto last) {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      f32x4 part[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        part[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, d.k[j]),
                                                          __builtin_bit_cast(bf16x8, Q[j]), zero, 0, 0, 0);
      f32x4 x = (part[0] + part[1]) + (part[2] + part[3]);  // unscaled
      if constexpr (last) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = t + 4 * kq + i < rb ? x[i] : -INFINITY;
      }
      float top = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
      top = fmaxf(top, xor16(top));
      top = fmaxf(top, xor32(top));
      top = fmaxf(m, top * a.scale_log2);
      if (__ballot(top > m)) {
        const float alpha = exp2f(m - finite_max(top));
        l *= alpha;
#pragma unroll
        for (int n = 0; n < 8; ++n) acc[n] *= alpha;
        m = top;
      }
      const float sub = finite_max(m);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = exp2f(fmaf(x[i], a.scale_log2, -sub));
      l += (x[0] + x[1]) + (x[2] + x[3]);
      if constexpr (last) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t + 4 * kq + i >= rb) d.v[i] = make_uint4(0, 0, 0, 0);
      }
      f32x4 sum[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v[8];
        unpack8(d.v[i], v);
#pragma unroll
        for (int n = 0; n < 8; ++n)
          sum[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[n], x[i], i == 0 ? zero : sum[n], 0, 0, 0);
      }
#pragma unroll
      for (int n = 0; n < 8; ++n) acc[n] += sum[n];
    };

    // the workgroup's waves take tiles in turn; the next tile's loads are in flight during a tile's arithmetic
    // (none is issued behind the last one: 2048 tokens x 8 KV heads 11.2 -> 10.2 us)
    constexpr int kStep = kDenseWaves * kDenseTile;
    int t = ra + wave * kDenseTile;
    constexpr std::integral_constant<bool, false> kFull{};
    constexpr std::integral_constant<bool, true> kLast{};
    if (t < rb) {
      DenseTile d0, d1;
      load_dense_tile(a, row0, t, rb - 1, r, kq, d0);
      while (true) {
        if (t + kStep >= rb) {
          attend(d0, t, kLast);
          break;
        }
        load_dense_tile(a, row0, t + kStep, rb - 1, r, kq, d1);
        attend(d0, t, kFull);
        t += kStep;
        if (t + kStep >= rb) {
          attend(d1, t, kLast);
          break;
        }
        load_dense_tile(a, row0, t + kStep, rb - 1, r, kq, d0);
        attend(d1, t, kFull);
        t += kStep;
      }
    }
    l += xor16(l);
    l += xor32(l);

    // merge the waves through LDS: lane (r, kq) holds dims 8 (4 kq + i) + n of head r
    if (r < n_live) {
      if (kq == 0) {
        s_m[wave][r] = m;
        s_l[wave][r] = l;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float4 *dst = reinterpret_cast<float4 *>(&s_acc[wave][r][8 * (4 * kq + i)]);
        dst[0] = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
        dst[1] = make_float4(acc[4][i], acc[5][i], acc[6][i], acc[7][i]);
      }
    }
    __syncthreads();
    // thread t: dim t % 128 of heads t / 128, t / 128 + 2, ...
    for (int j = tid / kHeadDim; j < n_live; j += kDenseThreads / kHeadDim) {
      const int d = tid % kHeadDim;
      float M = -INFINITY, L = 0.f, o = 0.f;
#pragma unroll
      for (int w = 0; w < kDenseWaves; ++w) M = fmaxf(M, s_m[w][j]);
#pragma unroll
      for (int w = 0; w < kDenseWaves; ++w) {
        const float wg = (s_m[w][j] == -INFINITY) ? 0.f : exp2f(s_m[w][j] - M);
        L += s_l[w][j] * wg;
        o += s_acc[w][j][d] * wg;
      }
      if (a.whole) {
        store_out(a.out, a.out_is_bf16, head_first + j, d, o / L);
        if (a.lse && d == 0) a.lse[head_first + j] = (M + log2f(L)) * kLn2;
        continue;
      }
      float *P = a.partials + ((head_first + j) * a.splits + split) * kPartialStride;
      if (d == 0) {
        P[0] = M;
        P[1] = L;
      }
      P[2 + d] = o;
    }
    if (c0 >= c_end) break;
    __syncthreads();  // LDS is reused by the next piece
    do R = dense_rows(a, ++seg);
    while (R == 0);  // (a segment with rows follows: chunks are left)
    row0 = a.seg_row_base[seg];
  }
}

// One workgroup per head; its groups of 128 threads (one dimension each) take the splits in turn, so that the partials
// of a head are fetched in a round or two of loads, and meet in LDS.  (One group walking all splits of a head eight at
// a time took 20 us for the 96 splits of 8 x 131072 tokens: a dozen dependent round trips on 32 CUs.)
template <int kGroups>
__global__ __launch_bounds__(kGroups * kHeadDim) void dense_merge_kernel(DenseArgs a) {
  __shared__ float s_m[kGroups], s_l[kGroups], s_o[kGroups][kHeadDim];
  const int head = blockIdx.x, t = threadIdx.x % kHeadDim, grp = threadIdx.x / kHeadDim;
  const int b = head / a.n_q_heads, h = head % a.n_q_heads;
  const int seg = b * a.n_kv_heads + h / a.group;
  const int chunks = dense_chunks(dense_rows(a, seg));
  if (chunks == 0) {  // an empty segment: zero output
    if (grp > 0) return;
    store_out(a.out, a.out_is_bf16, head, t, 0.f);
    if (a.lse && t == 0) a.lse[head] = -INFINITY;
    return;
  }
  const int n_active = dense_pieces(a, seg, chunks);
  const float *P = a.partials + (int64_t)head * a.splits * kPartialStride;
  constexpr int kBatch = 8;
  float Mx = -INFINITY, Ls = 0.f, os = 0.f;
  for (int s0 = grp; s0 < n_active; s0 += kGroups * kBatch) {
    float ms[kBatch], ll[kBatch], oo[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float *Q = P + min(s0 + kGroups * u, n_active - 1) * kPartialStride;
      ms[u] = Q[0];
      ll[u] = Q[1];
      oo[u] = Q[2 + t];
    }
    float Mn = Mx;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (s0 + kGroups * u >= n_active) {
        ms[u] = -INFINITY;
        ll[u] = oo[u] = 0.f;
      }
      Mn = fmaxf(Mn, ms[u]);
    }
    const float sub = finite_max(Mn), sc = exp2f(Mx - sub);
    Ls *= sc;
    os *= sc;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float w = exp2f(ms[u] - sub);
      Ls = fmaf(ll[u], w, Ls);
      os = fmaf(oo[u], w, os);
    }
    Mx = Mn;
  }
  s_o[grp][t] = os;
  if (t == 0) {
    s_m[grp] = Mx;
    s_l[grp] = Ls;
  }
  __syncthreads();
  if (grp > 0) return;
  float M = s_m[0], L = 0.f, o = 0.f;  // the first group has at least one split
#pragma unroll
  for (int v = 1; v < kGroups; ++v) M = fmaxf(M, s_m[v]);
#pragma unroll
  for (int v = 0; v < kGroups; ++v) {
    const float w = exp2f(s_m[v] - finite_max(M));
    L = fmaf(s_l[v], w, L);
    o = fmaf(s_o[v][t], w, o);
  }
  store_out(a.out, a.out_is_bf16, head, t, o / L);
  if (a.lse && t == 0) a.lse[head] = (M + log2f(L)) * kLn2;
}

}  // namespace

hipError_t launch_dense(const CacheView &c, const int32_t *seg_rows, float *partials, int max_splits,
                        const AttnOut &attn, hipStream_t s) {
  const int n_seg = c.batch * c.n_kv_heads, nh = c.batch * c.n_q_heads;
  if (nh == 0) return hipSuccess;
  DenseArgs a;
  a.q = c.q;
  a.k_cache = c.k_cache;
  a.v_cache = c.v_cache;
  a.seg_row_base = c.seg_row_base;
  a.seg_rows = seg_rows;
  a.partials = partials;
  a.out = attn.out;
  a.lse = attn.lse;
  a.out_is_bf16 = attn.out_is_bf16;
  a.n_seg = n_seg;
  a.n_kv_heads = c.n_kv_heads;
  a.n_q_heads = c.n_q_heads;
  a.group = c.group;
  a.head0 = 0;
  a.splits = max_splits;
  a.max_rows = c.max_rows_per_seg;
  a.scale_log2 = c.sm_scale * kLog2e;
  // One round of workgroups: as many as are resident at once (two waves per SIMD x 256 CUs; at three waves per SIMD
  // the next tile's registers spill: 113 against 86 us over 8 x 131072 tokens).  A small call is cut down to one step
  // per workgroup (2 x 3001 tokens: 11.1 us, 13.9 with at least four steps each; no difference on large calls).
  // A segment of n chunks has at most ceil(n / share) + 1 pieces, and never more than n: the share is large enough for
  // the partial slots of a head.
  constexpr int kResident = 2 * 256;
  const int max_chunks = (c.max_rows_per_seg + kChunkRows - 1) / kChunkRows;
  a.min_share = 1;
  if (max_chunks > max_splits && max_splits > 1) {
    const int least = (max_chunks + max_splits - 2) / (max_splits - 1);
    if (a.min_share < least) a.min_share = least;
  }
  const long want = ((long)n_seg * max_chunks + a.min_share - 1) / a.min_share;
  a.grid = (int)(want < 1 ? 1 : want < kResident ? want : kResident);
  // Whole segments against dealt-out chunks (us; G = 4): 8 segments of 320 rows 8.8 / 11.0, of 512 11.8 / 11.0; 128 of 512
  // 12.6 / 13.4, 320 of 512 22.1 / 23.3, 320 of 1024 39 / 36; 512 of 1024 42.6 / 50.0, 2048 of 64 20 / 57 with the lookup
  // in front of every workgroup.  Longer segments are dealt out (512 of 512 to 2048: 66 / 116) as far as the lookup goes.
  a.whole = n_seg > kDealtSegs || c.max_rows_per_seg <= (n_seg >= 512 ? 1024 : n_seg >= 128 ? 512 : 320);
  if (c.max_rows_per_seg > 0 || a.whole) {
    for (int h0 = 0; h0 < c.group; h0 += kDenseHeads) {  // one pass over the cache for up to 16 heads of a group
      a.head0 = h0;
      hipLaunchKernelGGL(dense_kernel, dim3(a.whole ? n_seg : a.grid), dim3(kDenseThreads), 0, s, a);
    }
  }
  if (a.whole) return hipGetLastError();
  // A head with at most 32 pieces (as many chunks, or partial slots, which is so from 512 heads on) is merged by one group
  // of threads in four rounds of loads.  One group against eight: 512 heads (16 x 2048 tokens) 29.5 against 31.5 us for the
  // call, 4096 heads (64 x 1024) 54.9 / 74.0; 8 x 1024 tokens x 8 KV heads, G = 1: 11.8 / 13.5, 2048 x 8, G = 4: 10.9 / 11.6.
  // (Few heads with many pieces: at the kernel.)
  if (nh >= 512 || max_chunks <= 32)
    hipLaunchKernelGGL(dense_merge_kernel<1>, dim3(nh), dim3(kHeadDim), 0, s, a);
  else
    hipLaunchKernelGGL(dense_merge_kernel<8>, dim3(nh), dim3(8 * kHeadDim), 0, s, a);
  return hipGetLastError();
}

}  // namespace dp
