// Dense decode attention over every token of a KV segment (paper Sec. 2.1,
// Eq. 1): the full-attention baseline that the paper's efficiency figures are
// measured against (Sec. 5.3).
//
// HBM-bound streaming kernel (512 B per token).  The K and V rows of a segment are
// contiguous, so a workgroup streams a row range [split * c, split * c + c) once and
// scores each row against up to 16 query heads of the GQA group at once: the cache
// is read once per KV head.  Both contractions run on the matrix cores, and the
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
// The running maximum of a head is the same in the four lanes that hold it, so the
// rescaling of the accumulators is lane-local; it is skipped while no maximum moves.
// Matrix-core time per 16 rows: 4 x 16 + 32 x 32 cycles, whatever the group size is:
// 29 us at 2.4 GHz for the million rows of 8 x 131072 tokens, behind 87 us of HBM
// time at 6.2 TB/s.  Measured there at G = 4: 94.5 us = 5.7 TB/s (108 us with the dot
// products, G softmaxes per row in 16 lanes each and G x 128 multiply-adds per row on
// the vector ALU; that form was vector-bound at G = 8).  The per-split partials (m, l, acc[128]) are merged
// by a second small kernel: no counters, no atomics.
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
  int32_t n_kv_heads, n_q_heads, group;
  int32_t head0;  // this launch serves heads [head0, head0 + 16) of every group
  int32_t splits, rows_per_split, max_rows;
  float scale_log2;
};

// one wave's 16 cache rows as the two contractions want them
struct DenseTile {
  uint4 k[4], v[4];
};

// Rows beyond the range read its last row: a lane's loads never leave the segment, and their weight is zero.
__device__ __forceinline__ void load_dense_tile(const DenseArgs &a, int64_t row0, int t, int last, int r, int kq,
                                                DenseTile &d) {
  const char *k = static_cast<const char *>(a.k_cache) + (row0 + min(t + r, last)) * kRowBytes + kq * 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) d.k[j] = *reinterpret_cast<const uint4 *>(k + j * 64);
#pragma unroll
  for (int i = 0; i < 4; ++i) d.v[i] = load_row_slice(a.v_cache, row0 + min(t + 4 * kq + i, last), r);
}

__global__ __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void dense_kernel(DenseArgs a) {
  __shared__ float s_m[kDenseWaves][kDenseHeads], s_l[kDenseWaves][kDenseHeads];
  __shared__ __align__(16) float s_acc[kDenseWaves][kDenseHeads][kHeadDim + 4];
  const int seg = blockIdx.y, split = blockIdx.x;
  const int R = min(a.seg_rows[seg], a.max_rows);
  const int ra = split * a.rows_per_split;
  const int rb = min(R, ra + a.rows_per_split);
  if (ra >= rb) return;  // the merge kernel derives the number of live splits from R as well

  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int r = lane & 15, kq = lane >> 4;
  const int b = seg / a.n_kv_heads, g = seg % a.n_kv_heads;
  const int64_t head_first = (int64_t)b * a.n_q_heads + g * a.group + a.head0;
  const int n_live = min(kDenseHeads, a.group - a.head0);
  const int64_t row0 = a.seg_row_base[seg];

  // query head r of the pass (a zero column beyond the group), chunks kq + 4 j
  uint4 Q[4];
  {
    const char *row = static_cast<const char *>(a.q) + (head_first + min(r, n_live - 1)) * kRowBytes + kq * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j) Q[j] = r < n_live ? *reinterpret_cast<const uint4 *>(row + j * 64) : make_uint4(0, 0, 0, 0);
  }
  f32x4 acc[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;  // head r: the maximum of all rows so far, the weights of this lane's rows

  auto attend = [&](const DenseTile &d, int t) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, d.k[j]), __builtin_bit_cast(bf16x8, Q[j]),
                                                  x, 0, 0, 0);
    float top = m;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = t + 4 * kq + i < rb ? x[i] * a.scale_log2 : -INFINITY;
      top = fmaxf(top, x[i]);
    }
    top = fmaxf(top, xor16(top));
    top = fmaxf(top, xor32(top));
    if (__ballot(top > m)) {  // finite from the first tile on: its first row is inside the range
      const float alpha = __builtin_amdgcn_exp2f(m - top);
      l *= alpha;
#pragma unroll
      for (int n = 0; n < 8; ++n) acc[n] *= alpha;
      m = top;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = __builtin_amdgcn_exp2f(x[i] - m);
      l += x[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v[8];
      unpack8(d.v[i], v);
#pragma unroll
      for (int n = 0; n < 8; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[n], x[i], acc[n], 0, 0, 0);
    }
  };

  // the workgroup's waves take tiles in turn; the next tile's loads are in flight during a tile's arithmetic
  constexpr int kStep = kDenseWaves * kDenseTile;
  int t = ra + wave * kDenseTile;
  if (t < rb) {
    DenseTile d0, d1;
    load_dense_tile(a, row0, t, rb - 1, r, kq, d0);
    while (true) {
      load_dense_tile(a, row0, t + kStep, rb - 1, r, kq, d1);
      attend(d0, t);
      t += kStep;
      if (t >= rb) break;
      load_dense_tile(a, row0, t + kStep, rb - 1, r, kq, d0);
      attend(d1, t);
      t += kStep;
      if (t >= rb) break;
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
      const float wg = (s_m[w][j] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(s_m[w][j] - M);
      L += s_l[w][j] * wg;
      o += s_acc[w][j][d] * wg;
    }
    float *P = a.partials + ((head_first + j) * a.splits + split) * kPartialStride;
    if (d == 0) {
      P[0] = M;
      P[1] = L;
    }
    P[2 + d] = o;
  }
}

struct DenseMergeArgs {
  const float *partials;
  const int32_t *seg_rows;
  void *out;
  float *lse;  // nullable
  int32_t n_kv_heads, n_q_heads, group, splits, rows_per_split, max_rows, out_is_bf16;
};

// One workgroup per head; its eight groups of 128 threads (one dimension each) take the splits in turn, so that the
// partials of a head are fetched in a round or two of loads, and meet in LDS.  (One group walking all splits of a head
// eight at a time took 20 us for the 96 splits of 8 x 131072 tokens: a dozen dependent round trips on 32 CUs.)
constexpr int kMergeGroups = 8;
__global__ __launch_bounds__(kMergeGroups * kHeadDim) void dense_merge_kernel(DenseMergeArgs a) {
  __shared__ float s_m[kMergeGroups], s_l[kMergeGroups], s_o[kMergeGroups][kHeadDim];
  const int head = blockIdx.x, t = threadIdx.x % kHeadDim, grp = threadIdx.x / kHeadDim;
  const int b = head / a.n_q_heads, h = head % a.n_q_heads;
  const int seg = b * a.n_kv_heads + h / a.group;
  const int R = min(a.seg_rows[seg], a.max_rows);
  const int n_active = (R + a.rows_per_split - 1) / a.rows_per_split;
  if (n_active <= 0) {  // an empty segment: zero output
    if (grp > 0) return;
    store_out(a.out, a.out_is_bf16, head, t, 0.f);
    if (a.lse && t == 0) a.lse[head] = -INFINITY;
    return;
  }
  const float *P = a.partials + (int64_t)head * a.splits * kPartialStride;
  constexpr int kBatch = 8;
  float Mx = -INFINITY, Ls = 0.f, os = 0.f;
  for (int s0 = grp; s0 < n_active; s0 += kMergeGroups * kBatch) {
    float ms[kBatch], ll[kBatch], oo[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float *Q = P + min(s0 + kMergeGroups * u, n_active - 1) * kPartialStride;
      ms[u] = Q[0];
      ll[u] = Q[1];
      oo[u] = Q[2 + t];
    }
    float Mn = Mx;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (s0 + kMergeGroups * u >= n_active) ms[u] = -INFINITY;  // every live split has at least one row: its m is finite
      Mn = fmaxf(Mn, ms[u]);
    }
    const float sc = __builtin_amdgcn_exp2f(Mx - Mn);
    Ls *= sc;
    os *= sc;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float w = __builtin_amdgcn_exp2f(ms[u] - Mn);
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
  for (int v = 1; v < kMergeGroups; ++v) M = fmaxf(M, s_m[v]);
#pragma unroll
  for (int v = 0; v < kMergeGroups; ++v) {
    const float w = __builtin_amdgcn_exp2f(s_m[v] - M);
    L = fmaf(s_l[v], w, L);
    o = fmaf(s_o[v][t], w, o);
  }
  store_out(a.out, a.out_is_bf16, head, t, o / L);
  if (a.lse && t == 0) a.lse[head] = (M + log2f(L)) * kLn2;
}

}  // namespace

// Equal row ranges stream at equal speed, so the grid is ONE round of workgroups: as many as are resident
// at once (three waves per SIMD x 256 CUs), each with at least 256 rows (four steps).
void dense_split(int max_rows, int n_seg, int max_splits, int *splits, int *rows_per_split) {
  constexpr int resident = 3 * 256;
  long want = resident / n_seg;
  if (want > max_splits) want = max_splits;
  const long by_rows = ((long)max_rows + 255) / 256;
  if (want > by_rows) want = by_rows;
  if (want < 1) want = 1;
  const long c = kChunkRows * (((long)max_rows + kChunkRows * want - 1) / (kChunkRows * want));
  *rows_per_split = (int)(c > 0 ? c : kChunkRows);
  *splits = (int)(((long)max_rows + *rows_per_split - 1) / *rows_per_split);
  if (*splits < 1) *splits = 1;
}

hipError_t launch_dense(const CacheView &c, const int32_t *seg_rows, float *partials, int max_splits,
                        const AttnOut &attn, hipStream_t s) {
  const int n_seg = c.batch * c.n_kv_heads, nh = c.batch * c.n_q_heads;
  if (nh == 0) return hipSuccess;
  int splits, rows_per_split;
  dense_split(c.max_rows_per_seg, n_seg, max_splits, &splits, &rows_per_split);
  if (c.max_rows_per_seg > 0) {
    DenseArgs a;
    a.q = c.q;
    a.k_cache = c.k_cache;
    a.v_cache = c.v_cache;
    a.seg_row_base = c.seg_row_base;
    a.seg_rows = seg_rows;
    a.partials = partials;
    a.n_kv_heads = c.n_kv_heads;
    a.n_q_heads = c.n_q_heads;
    a.group = c.group;
    a.splits = splits;
    a.rows_per_split = rows_per_split;
    a.max_rows = c.max_rows_per_seg;
    a.scale_log2 = c.sm_scale * kLog2e;
    const dim3 grid(splits, n_seg);
    // one pass over the cache for up to 16 heads of a group
    for (int h0 = 0; h0 < c.group; h0 += kDenseHeads) {
      a.head0 = h0;
      hipLaunchKernelGGL(dense_kernel, grid, dim3(kDenseThreads), 0, s, a);
    }
  }
  DenseMergeArgs m;
  m.partials = partials;
  m.seg_rows = seg_rows;
  m.out = attn.out;
  m.lse = attn.lse;
  m.n_kv_heads = c.n_kv_heads;
  m.n_q_heads = c.n_q_heads;
  m.group = c.group;
  m.splits = splits;
  m.rows_per_split = rows_per_split;
  m.max_rows = c.max_rows_per_seg;
  m.out_is_bf16 = attn.out_is_bf16;
  hipLaunchKernelGGL(dense_merge_kernel, dim3(nh), dim3(kMergeGroups * kHeadDim), 0, s, m);
  return hipGetLastError();
}

}  // namespace dp
