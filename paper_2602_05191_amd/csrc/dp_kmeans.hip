// Assignment step of the k-means clustering that builds the clustered cache at
// prefill (paper Sec. 4.1): every key goes to its nearest centroid,
//   argmin_c |x - c|^2  =  argmax_c ( x . c - |c|^2 / 2 ),
// ties to the lower centroid index.  Together with dp_build_cluster_cache (the
// update step: centroids = cluster means) this is one Lloyd iteration.
//
// The one dense contraction of this library: tokens x centroids x 128 per KV
// segment (2.2 TFLOP per iteration at 8 x 131072 tokens x 8192 centroids), so
// it runs on the matrix cores: v_mfma_f32_16x16x32_bf16, bf16 operands as
// stored, fp32 accumulation.  MFMA-bound; the operands come from cache (a
// segment's centroids are 2 MB).
//
// A wave owns 16 x TM tokens (the B operand: the columns of TM result tiles, held in registers for the whole kernel).
// The workgroup walks the segment's centroids 64 at a time: the block is fetched once from global memory by all 256
// threads, kept in LDS (three blocks in rotation, rows padded to 272 B so that the 16 rows an operand read touches
// fall into different banks) and read from there by the four waves as the A operand, 16 centroids (a tile) at a time;
// the block after the next travels global -> registers -> LDS meanwhile.
// Operand layout of the instruction: lane l holds row (column) l % 16 and the 8 consecutive k of block l / 16; the
// result tile holds, in lane l, column l % 16 and rows 4 (l / 16) .. + 3.  So the four results of a lane are four
// consecutive centroids of ONE token: its running best is one (score, index) per token tile.  The accumulator starts
// at -|c|^2 / 2 of those centroids (read from LDS), so a result element IS the score.  The four classes of centroids
// of a token are merged once at the end (lower index wins a tie).
// Bounds: the matrix cores' time, and next to it the issue of vector instructions (one per 4 cycles and SIMD, four in
// the time of one MFMA).  With the tokens as rows each score cost three of these, more than there is room for.  Here,
// per four scores: two v_max3, a comparison and a select keep the best quad (kQuads), and which of its four it was is
// found at the end by scoring the quad again; or twelve keep the index itself (small launches, where latency counts).
// A tile's tokens are taken in two halves: the MFMAs of one run while the results of the other are looked at, in an
// order given to the scheduler, so that a wave alone keeps both units busy (two waves in step would wait for the same
// unit).  No load may be pending when the loop begins (below).
// 8 x 131072 tokens x 8192 centroids: 1860 -> 1450 us = 1.52 PFLOP/s in the rounds of a fit; matrix cores busy 71 % of the
// cycles, at the 1.9 GHz the card runs at under this load.  (bench.py's line, five calls on keys of its own, reads 1545 to
// 1565 us = 1.41 PFLOP/s: so does the kernel's own time there.)  Tried and worse: the position inside the quad as lane masks in scalar
// registers (1660: ten scalar instructions per quad), a pair instead of a quad scored again (1510), the index itself
// at 128 tokens per wave (1705).
#include "dp_device.hpp"
#include "dp_kernels.hpp"

namespace dp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kKmThreads = 256;
constexpr int kKmCus = 256;                   // compute units of the chip
constexpr int kKmCB = 64;                     // centroids per LDS block: 256 threads fetch 64 rows at once
constexpr int kKmBufs = 3;                              // LDS blocks in rotation: computed on, next (already stored), being filled
constexpr int kKmRowPad = kRowBytes + 16;              // LDS row stride: 68 words, 4 r mod 64 banks for row r

constexpr int kNoCentroid = 0x7fffffff;  // no centroid has scored above -inf
constexpr int kNoQuad = kNoCentroid / 4;
constexpr int kWaitLoads = 0x0f70;   // s_waitcnt vmcnt(0), the other counters at their maxima (not waited for)

struct KmArgs {
  const void *k_tokens, *centroids;
  const int64_t *seg_row_base;
  const int32_t *seg_rows, *seg_cluster_ptr;
  float *half_norm;      // [total_clusters]
  int32_t *assignment;   // [total_rows]
  float *best_score;     // nullable
  int32_t max_rows, total_clusters;
};

// half_norm[c] = |c|^2 / 2 in fp32; one 16-lane DPP row per centroid
__global__ __launch_bounds__(256) void km_norm_kernel(KmArgs a) {
  const int c = blockIdx.x * 16 + (threadIdx.x >> 4), lane16 = threadIdx.x & 15;
  if (c >= a.total_clusters) return;
  float f[8];
  unpack8(load_row_slice(a.centroids, c, lane16), f);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) s = fmaf(f[i], f[i], s);
  s = row16_sum(s);
  if (lane16 == 0) a.half_norm[c] = 0.5f * s;
}

// 16 B of row `row` at dims [32 j + 8 kq, + 8): the operand slice of lane (row % 16, kq) for k-step j
__device__ __forceinline__ bf16x8 operand_slice(const void *base, int64_t row, int j, int kq) {
  return *reinterpret_cast<const bf16x8 *>(static_cast<const char *>(base) + row * kRowBytes + j * 64 + kq * 16);
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// kNorms: the workgroup works out |c|^2 / 2 of the centroids it stages itself (half_norm is not read): the same products
// and sums in the same order as km_norm_kernel's, so the same bits.
template <int TM, bool kQuads, bool kNorms = false>
__device__ __forceinline__ void km_assign(const KmArgs &a) {
  constexpr int kTokensPerWave = 16 * TM, kTokensPerBlock = kTokensPerWave * (kKmThreads / 64);
  __shared__ __attribute__((aligned(16))) char s_c[kKmBufs][kKmCB * kKmRowPad];
  __shared__ __attribute__((aligned(16))) float s_hn[kKmBufs][kKmCB];  // -|c|^2 / 2
  const int seg = blockIdx.y;
  const int n = min(a.seg_rows[seg], a.max_rows);
  const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
  const int blk0 = blockIdx.x * kTokensPerBlock;
  if (blk0 >= n) return;  // uniform in the workgroup
  const int t0 = blk0 + wave * kTokensPerWave;  // first token of this wave (a wave past the end only helps to load)
  const int c0 = a.seg_cluster_ptr[seg], kc = a.seg_cluster_ptr[seg + 1] - c0;
  const int64_t r0 = a.seg_row_base[seg];
  const int r = lane & 15, kq = lane >> 4;

  // B operand: column r of tile tm is token t0 + 16 tm + r; beyond the segment its last token (not stored)
  bf16x8 tok[TM][4];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int t = min(t0 + 16 * tm + r, n - 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) tok[tm][j] = operand_slice(a.k_tokens, r0 + t, j, kq);
  }
  // of token t0 + 16 tm + r among the centroids 4 x + 0 .. 3 with x % 4 == kq: the best score and its centroid, or
  // (kQuads) its x
  float best[TM];
  int bidx[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    best[tm] = -INFINITY;
    bidx[tm] = kQuads ? kNoQuad : kNoCentroid;
  }

  // global -> registers -> LDS: thread tid fetches 64 B (quarter tid & 3) of row tid >> 2
  const int lrow = tid >> 2, lq = tid & 3;
  struct Staged {
    bf16x8 slice[4];
    float half_norm;
  };
  auto fetch_block = [&](int blk, Staged &x) {
    const int cc = c0 + min(blk * kKmCB + lrow, kc - 1);
    const char *src = static_cast<const char *>(a.centroids) + (int64_t)cc * kRowBytes + lq * 64;
#pragma unroll
    for (int u = 0; u < 4; ++u) x.slice[u] = *reinterpret_cast<const bf16x8 *>(src + 16 * u);
    if (!kNorms) x.half_norm = a.half_norm[cc];
  };
  auto store_block = [&](int buf, int blk, const Staged &x) {
    char *dst = s_c[buf] + lrow * kKmRowPad + lq * 64;
#pragma unroll
    for (int u = 0; u < 4; ++u) *reinterpret_cast<bf16x8 *>(dst + 16 * u) = x.slice[u];
    float half_norm;
    if constexpr (kNorms) {
      float part[4];  // of 8 dimensions each: a lane of the norm kernel's 16; then the order of its row sum
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float f[8];
        unpack8(__builtin_bit_cast(uint4, x.slice[u]), f);
        part[u] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) part[u] = fmaf(f[i], f[i], part[u]);
      }
      float sum = (part[0] + part[1]) + (part[2] + part[3]);
      sum += dpp_mov<0xB1>(sum);  // the neighbouring quarter of the row, then the other half
      sum += dpp_mov<0x4E>(sum);
      half_norm = 0.5f * sum;
    } else {
      half_norm = x.half_norm;
    }
    // past the segment's centroids: rows that can never win (a finite product - inf, or NaN: neither is > best)
    if (lq == 0) s_hn[buf][lrow] = blk * kKmCB + lrow < kc ? -half_norm : -INFINITY;
  };
  const char *const my_slices = s_c[0] + r * kKmRowPad + kq * 16;
  const f32x4 *const my_starts = reinterpret_cast<const f32x4 *>(s_hn[0]) + kq;
  auto read_slice = [&](int row, int j) {
    return *reinterpret_cast<const bf16x8 *>(my_slices + (unsigned)row * kKmRowPad + j * 64);
  };
  auto read_start = [&](int row) { return my_starts[(unsigned)row / 4]; };

  const int n_blocks = (kc + kKmCB - 1) / kKmCB;
  Staged stage;
  if (n_blocks > 0) {
    Staged first;
    fetch_block(0, first);
    fetch_block(1, stage);  // (past the last block: the last centroid, as rows that cannot win)
    store_block(0, 0, first);
    store_block(1, 1, stage);
  }
  // The tokens have arrived before the loop begins: a load still open there would put a wait for ALL loads, the
  // staged block's among them, in front of the loop's first MFMA.
  __builtin_amdgcn_s_waitcnt(kWaitLoads);
  lds_barrier();
  bf16x8 cur[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) cur[j] = read_slice(0, j);  // harmless when there is no block: never used
  f32x4 start = read_start(0);
  constexpr int kHalf = TM / 2, kPer = kQuads ? 2 : 4;
  f32x4 acc[TM];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) acc[tm] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  auto update = [&](int tm, int quad) {  // centroids come in ascending order: strict comparisons keep the lowest
    const f32x4 x = acc[tm];
    if constexpr (kQuads) {
      const float m = fmaxf(fmaxf(fmaxf(fmaxf(best[tm], x[0]), x[1]), x[2]), x[3]);
      bidx[tm] = m > best[tm] ? quad : bidx[tm];
      best[tm] = m;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool better = x[i] > best[tm];
        best[tm] = better ? x[i] : best[tm];
        bidx[tm] = better ? 4 * quad + i : bidx[tm];
      }
    }
  };
  // the updates stay in the half they are written in
  auto keep = [&](int first) {
#pragma unroll
    for (int tm = 0; tm < kHalf; ++tm) asm volatile("" : "+v"(best[first + tm]), "+v"(bidx[first + tm]));
  };
  // one matrix instruction, then the vector instructions that fit behind it
  auto groups = [&](bool reads) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int i = 0; i < kHalf; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, kPer, 0);
      }
      if (reads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  int buf = 0, quad = kq, row = 0;  // row: of the tile, in the three blocks together
  for (int blk = 0; blk < n_blocks; ++blk) {
    const int buf2 = buf == 0 ? kKmBufs - 1 : buf - 1;
    if (blk + 2 < n_blocks) fetch_block(blk + 2, stage);  // in flight during this block's MFMAs
#pragma unroll 1
    for (int tt = 0; tt < kKmCB / 16; ++tt) {
      row = row == kKmBufs * kKmCB - 16 ? 0 : row + 16;  // past the last block: a stale block, never used
      // first half of the token tiles; meanwhile the second half's results of the tile before
#pragma unroll
      for (int tm = kHalf; tm < TM; ++tm) update(tm, quad - 4);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int tm = 0; tm < kHalf; ++tm) acc[tm] = mfma(cur[j], tok[tm][j], j == 0 ? start : acc[tm]);
      keep(kHalf);
      groups(false);
      // second half; meanwhile the first half's results, and the next tile's slices
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int tm = kHalf; tm < TM; ++tm) acc[tm] = mfma(cur[j], tok[tm][j], j == 0 ? start : acc[tm]);
        if (j == 0) start = read_start(row);
        cur[j] = read_slice(row, j);
      }
#pragma unroll
      for (int tm = 0; tm < kHalf; ++tm) update(tm, quad);
      quad += 4;
      keep(0);
      groups(true);
    }
    // buf2 held block blk - 1, last read before the barrier that ended the previous iteration
    if (blk + 2 < n_blocks) store_block(buf2, blk + 2, stage);
    lds_barrier();
    buf = buf == kKmBufs - 1 ? 0 : buf + 1;
  }
#pragma unroll
  for (int tm = kHalf; tm < TM; ++tm) update(tm, quad - 4);

  // merge the four classes of each token: max score, the lower index on a tie
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int m = 16; m < 64; m *= 2) {
      const float os = __shfl_xor(best[tm], m, 64);
      const int oq = __shfl_xor(bidx[tm], m, 64);
      const bool take = os > best[tm] || (os == best[tm] && oq < bidx[tm]);
      best[tm] = take ? os : best[tm];
      bidx[tm] = take ? oq : bidx[tm];
    }
  // Which centroid of the quad?  The four scores once more by the same instructions (so to the same bit): the quads of
  // four tokens are the 16 rows of one tile; token 4 y + z has rows 4 z .. + 3, whose results lie in the lanes of
  // kq == z.  (A token without a quad: kNoQuad is past the last centroid, its scores stay -inf.)
  if (kQuads && kc > 0) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
      f32x4 four{};  // the scores of column r's token, in the lanes of kq == r % 4
#pragma unroll
      for (int y0 = 0; y0 < 4; y0 += 2) {
        bf16x8 rows[2][4];
        f32x4 res[2];
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int row_c = c0 + min(4 * __shfl(bidx[tm], 4 * (y0 + y) + (r >> 2), 64) + (r & 3), kc - 1);
          const int c = 4 * __shfl(bidx[tm], 4 * (y0 + y) + kq, 64);
#pragma unroll
          for (int j = 0; j < 4; ++j) rows[y][j] = operand_slice(a.centroids, row_c, j, kq);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float hn = a.half_norm[c0 + min(c + i, kc - 1)];
            res[y][i] = c + i < kc ? -hn : -INFINITY;
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int y = 0; y < 2; ++y) res[y] = mfma(rows[y][j], tok[tm][j], res[y]);
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int i = 0; i < 4; ++i) four[i] = (r >> 2) == y0 + y ? res[y][i] : four[i];
      }
      float s = -INFINITY;
      int id = kNoCentroid;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool better = four[i] > s;
        s = better ? four[i] : s;
        id = better ? 4 * bidx[tm] + i : id;
      }
      bidx[tm] = __shfl(id, 16 * (r & 3) + r, 64);
      __builtin_amdgcn_sched_barrier(0);  // one token tile's rows at a time: all of them do not fit the registers
    }
  }
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
    const int t = t0 + 16 * tm + r;
    if (kq == 0 && t < n) {
      a.assignment[r0 + t] = kc > 0 ? bidx[tm] : -1;
      if (a.best_score) a.best_score[r0 + t] = best[tm];
    }
  }
}

__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void km_assign8_kernel(KmArgs a) { km_assign<8, true>(a); }
__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void km_assign4_kernel(KmArgs a) { km_assign<4, false>(a); }
__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void km_assign2_kernel(KmArgs a) { km_assign<2, false>(a); }
__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void km_assign4_norms_kernel(KmArgs a) { km_assign<4, false, true>(a); }
__global__ __launch_bounds__(kKmThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void km_assign2_norms_kernel(KmArgs a) { km_assign<2, false, true>(a); }

// One 16-lane row copies one key row: centroid c of the segment starts as the key of token floor(c * n / kc).
__global__ __launch_bounds__(256) void km_init_strided_kernel(KmArgs a, void *centroids) {
  const int seg = blockIdx.y;
  const int c0 = a.seg_cluster_ptr[seg], kc = a.seg_cluster_ptr[seg + 1] - c0;
  const int lane16 = threadIdx.x & 15, c = blockIdx.x * 16 + (threadIdx.x >> 4);
  if (c >= kc) return;
  const int n = min(a.seg_rows[seg], a.max_rows);
  uint4 row = make_uint4(0, 0, 0, 0);
  if (n > 0) row = load_row_slice(a.k_tokens, a.seg_row_base[seg] + (int64_t)c * n / kc, lane16);
  *reinterpret_cast<uint4 *>(static_cast<char *>(centroids) + (size_t)(c0 + c) * kRowBytes + lane16 * 16) = row;
}

}  // namespace

hipError_t launch_kmeans_init_strided(const KmeansProblem &p, void *centroids, int max_kc, hipStream_t s) {
  if (p.n_seg == 0 || max_kc == 0) return hipSuccess;
  KmArgs a{};
  a.k_tokens = p.k_tokens;
  a.seg_row_base = p.seg_row_base;
  a.seg_rows = p.seg_rows;
  a.seg_cluster_ptr = p.seg_cluster_ptr;
  a.max_rows = p.max_rows;
  hipLaunchKernelGGL(km_init_strided_kernel, dim3((max_kc + 15) / 16, p.n_seg), dim3(256), 0, s, a, centroids);
  return hipGetLastError();
}

hipError_t launch_kmeans_assign(const KmeansProblem &p, float *half_norm, hipStream_t s) {
  if (p.n_seg == 0 || p.max_rows == 0) return hipSuccess;
  KmArgs a;
  a.k_tokens = p.k_tokens;
  a.centroids = p.centroids;
  a.seg_row_base = p.seg_row_base;
  a.seg_rows = p.seg_rows;
  a.seg_cluster_ptr = p.seg_cluster_ptr;
  a.half_norm = half_norm;
  a.assignment = p.assignment;
  a.best_score = p.best_score;
  a.max_rows = p.max_rows;
  a.total_clusters = p.total_clusters;
  // Tokens per workgroup.  128 per wave need the fewest operand bytes per product and the fewest instructions per score,
  // but end with 14 us in which every token's last four candidates are scored again.  Against 64 per wave, where the
  // launch fills the chip at its two workgroups per CU (us):
  //   centroids             1024       1280       1536       1792       2048       4096
  //   8 x 32768 tokens     79 / 72    88 / 87    99 / 102  111 / 117  121 / 132  211 / 252
  //   8 x 65536           143 / 130  162 / 160  182 / 188  203 / 217  223 / 245  398 / 475
  //   8 x 131072          260 / 250  299 / 306  341 / 364  382 / 419  426 / 477  773 / 928
  // and where it does not (8 x 24576, 384 workgroups) they lose up to 4096 (192 / 191).  Below that 32 per wave while these
  // fit one round at three workgroups per CU (8 x 12000 tokens: 33.2 against 35.4 us; 8192 tokens, one segment: 13.2
  // against 17.5), then 64 (8 x 16384: 46 against 52; 64 x 4096: 22 against 25).
  // The host sees the mean of the centroids and the longest segment only: workgroups past the end of a shorter segment
  // leave at once, but count here (one segment of 131072 x 8192 among 31 of 1000 x 64 takes 64 per wave, 260 us, where 128
  // would take 226; four of 40000 x 2500 among 28 of 3000 x 200: 120, and 131 with 128).
  auto grid = [&](int tm) {
    const int per_block = 16 * tm * (kKmThreads / 64);
    return dim3((p.max_rows + per_block - 1) / per_block, p.n_seg);
  };
  auto blocks = [&](int tm) { return (int64_t)grid(tm).x * grid(tm).y; };
  const bool wide = p.total_clusters / p.n_seg >= 1536 && blocks(8) >= 2 * kKmCus, narrow = !wide && blocks(2) <= 3 * kKmCus;
  // The norms: by a launch in front (5 us with the gap), or by every workgroup for the centroids it stages, which costs each
  // 70 instructions per wave and block of 64 centroids.  That pays up to 16 blocks in a row and 16384 in the launch.  Fits of
  // 3 rounds, us, norms by the workgroups / by a launch: one segment of 2048 x 128 66.4 / 72.7, 24 of up to 7000 x 218 146 / 157,
  // 128 of up to 2300 x 143 129 / 137, 8 of 8100 x 506 124.5 / 134, 8 of 16384 x 1024 210 / 214; 128 of up to 8000 x 500 385 / 387,
  // one of 32768 x 2048 200 / 196, two of 65536 x 2048 348 / 336.
  const int64_t n_blocks = (p.total_clusters / p.n_seg + kKmCB - 1) / kKmCB;
  const bool own_norms = !wide && n_blocks <= 16 && blocks(narrow ? 2 : 4) * n_blocks <= 16384;
  if (p.total_clusters > 0 && !own_norms)
    hipLaunchKernelGGL(km_norm_kernel, dim3((p.total_clusters + 15) / 16), dim3(256), 0, s, a);
  if (wide)
    hipLaunchKernelGGL(km_assign8_kernel, grid(8), dim3(kKmThreads), 0, s, a);
  else if (narrow && own_norms)
    hipLaunchKernelGGL(km_assign2_norms_kernel, grid(2), dim3(kKmThreads), 0, s, a);
  else if (narrow)
    hipLaunchKernelGGL(km_assign2_kernel, grid(2), dim3(kKmThreads), 0, s, a);
  else if (own_norms)
    hipLaunchKernelGGL(km_assign4_norms_kernel, grid(4), dim3(kKmThreads), 0, s, a);
  else
    hipLaunchKernelGGL(km_assign4_kernel, grid(4), dim3(kKmThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace dp
