// merge.hip -- log-sum-exp merge of partition partials (gfx950).
//
// Paper Sec. 4.1(2): the final output is the sum of the partitions' partial
// outputs once each is weighted by its share of the global softmax
// denominator (l^(j) = exp(lse_j)).  Per row r = (sequence, query head):
//   M = max_p lse_p,  w_p = exp(lse_p - M),
//   out = sum_p w_p out_p / sum_p w_p,  lse_out = M + ln sum_p w_p,
// skipping parts with lse_p = -inf (their out_p never enters a sum); no live part
// gives out = 0, lse_out = -inf.  A NaN lse is not in M but has a NaN weight, so
// a row is empty where it has no live part (its weights sum to 0) and not where
// M is -inf: a row with parts whose lse is NaN, and no others, is NaN.
//
// HBM-bound.  32 consecutive threads cover one 128-float row (16 bytes each,
// one coalesced 512-byte access per part).  Three kernels:
//  * up to four parts (the usual local + migrated split): every lse and every
//    partial row is loaded up front, before any of them is used, so the
//    kernel waits on one round of memory latency;
//  * more parts of few rows (the chunks of few sequences): a row's parts spread
//    over 2 to 16 thread groups of 4 parts a round: one such round up to 64 parts,
//    further ones beyond (plans make up to 256 chunks);
//  * more parts of many rows, and the balanced launch's pieces: the 32 lanes of
//    a row first read 32 parts' lse at once and reduce their max with lane
//    shuffles, then stream the partial rows with loads that do not depend on
//    any lse (the weights come from the lanes by shuffle), so loads of
//    consecutive parts overlap.
// Where a row has KP thread groups, each keeps its sums relative to its own max
// and the groups are combined through LDS, rescaled to the common max (the same
// log-sum-exp algebra once more).
// The part-to-group assignment and every summation order depend only on
// n_parts and the number of merged rows, so results are deterministic.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "kernels.h"

namespace bana {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Rows of merged row r (below 2^26: a launch counts 32 threads each in 32 bits) in a part and in the
// result.  Where all heads are merged, both are r; a kv-head range's rows take a division.
struct Rows {
  int64_t in, out;

  static __device__ __forceinline__ unsigned sequence(const MergeRows& mr, unsigned r) { return r / (unsigned)mr.hn; }
  __device__ __forceinline__ Rows(const MergeRows& mr, unsigned r) {
    if (mr.hn == mr.in_hq && mr.hn == mr.out_hq) {
      in = out = r;
    } else {
      const unsigned b = sequence(mr, r), i = r - b * mr.hn;
      in = (int64_t)b * mr.in_hq + mr.in_h0 + i;
      out = (int64_t)b * mr.out_hq + mr.out_h0 + i;
    }
  }
};

// The parts of a merged row: part p is row first + p * stride of the part buffers, p < n.  Partials
// [n_parts][B][in_hq]: n_parts rows B x in_hq apart.  Pieces of the balanced launch: the pieces of a
// sequence are consecutive slots of in_hq rows, counted from the block-count prefix sums (pieces =
// intervals of S blocks that overlap the sequence's blocks [prefix[b], prefix[b + 1])).
struct Parts {
  int n;
  int64_t first, stride;

  __device__ __forceinline__ Parts(const MergeRows& mr, const Rows& at, int n_parts)
      : n(n_parts), first(at.in), stride(mr.B * mr.in_hq) {}
  __device__ __forceinline__ Parts(const MergeRows& mr, unsigned r, const int32_t* __restrict__ prefix, int K)
      : n(0), first(0), stride(mr.in_hq) {
    const unsigned b = Rows::sequence(mr, r), i = r - b * mr.hn;
    const int p0 = prefix[b], p1 = prefix[b + 1], total = prefix[mr.B];
    const unsigned S = total > K ? ((unsigned)total + K - 1) / (unsigned)K : 1u;
    if (p1 > p0) {  // slots clamped to [b, K + b): prefix sums from another call cannot reach outside
      const unsigned p = min((unsigned)p0 / S, (unsigned)K - 1);
      const unsigned last = min(max((unsigned)(p1 - 1) / S, p), (unsigned)K - 1);
      n = (int)(last - p + 1);
      first = (int64_t)(p + b) * mr.in_hq + mr.in_h0 + i;
    }
  }
};

// At most NP parts, all loaded before use.  Parts with lse = -inf are loaded
// too (their rows lie inside the partial buffer) but never enter a sum.
template <int NP>
__global__ __launch_bounds__(256) void merge_few_kernel(const float* __restrict__ outs,
                                                        const float* __restrict__ lses, int n_parts, MergeRows mr,
                                                        float* __restrict__ out, float* __restrict__ lse_out) {
  const int t = threadIdx.x;
  const int d4 = t & 31;
  const int64_t r = (int64_t)blockIdx.x * 8 + (t >> 5);
  if (r >= mr.B * mr.hn) return;
  const int64_t rows = mr.B * mr.in_hq;
  const Rows at(mr, (unsigned)r);
  const int64_t row = at.in, orow = at.out;
  float l[NP];
  f32x4 o[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (p < n_parts) {
      l[p] = lses[(int64_t)p * rows + row];
      o[p] = reinterpret_cast<const f32x4*>(outs + ((int64_t)p * rows + row) * 128)[d4];
    }
  }
  float M = -INFINITY;
  bool empty = true;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (p < n_parts) {
      M = fmaxf(M, l[p]);
      empty &= l[p] == -INFINITY;
    }
  }
  f32x4* dst = reinterpret_cast<f32x4*>(out + orow * 128) + d4;
  if (empty) {
    *dst = f32x4{0.f, 0.f, 0.f, 0.f};
    if (lse_out != nullptr && d4 == 0) lse_out[orow] = -INFINITY;
    return;
  }
  float wsum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (p < n_parts && l[p] != -INFINITY) {
      const float w = expf(l[p] - M);
      wsum += w;
      acc += w * o[p];
    }
  }
  *dst = acc * (1.0f / wsum);
  if (lse_out != nullptr && d4 == 0) lse_out[orow] = M + logf(wsum);
}

// 1 / the sum of a row's weights; 0 for an empty row, whose sums are 0.  A select costs a short merge
// less than a branch on the sum (32 rows of 32 parts 3.18 against 3.26 us).
__device__ __forceinline__ float inverse_sum(float wsum) { return wsum == 0.f ? 0.f : 1.0f / wsum; }

// Any number of parts of many rows.  Group k (of KP) of a row takes parts k, k + KP, ...;
// its q-th part is p = k + KP q.
//
// Rows stream in rounds of U parts, each round requested before the previous one is summed (the
// waits the compiler places keep about one round in flight per lane, its loads overlapping the
// sums of the round before).  The many-part merge of many rows takes one part per round: with fewer
// part streams in flight per wavefront the 16-part merge of 32,768 rows runs in 50 us instead of
// 57 (U = 4) or 62 (U = 8) on MI355X, cold caches; the piece merges, few pieces per row, keep
// U = 4 (U = 1 costs them 2 us).
template <int KP, bool PIECES, int U>
__global__ __launch_bounds__(256) void merge_many_kernel(const float* __restrict__ outs,
                                                         const float* __restrict__ lses, int n_parts, MergeRows mr,
                                                         float* __restrict__ out, float* __restrict__ lse_out,
                                                         const int32_t* __restrict__ prefix, int K) {
  constexpr int R = 256 / (32 * KP);  // rows per workgroup
  __shared__ f32x4 sm_acc[KP > 1 ? R * KP * 32 : 1];
  __shared__ float sm_m[KP > 1 ? R * KP : 1];
  __shared__ float sm_w[KP > 1 ? R * KP : 1];
  const int t = threadIdx.x;
  const int d4 = t & 31;
  const int k = (t >> 5) % KP;
  const int rl = t / (32 * KP);
  const int64_t r = (int64_t)blockIdx.x * R + rl;  // row among the B x hn merged rows
  const bool live = r < mr.B * mr.hn;
  const Rows at(mr, live ? (unsigned)r : 0u);
  const int64_t dst_row = at.out;
  Parts parts(mr, at, live ? n_parts : 0);
  if (PIECES && live) parts = Parts(mr, (unsigned)r, prefix, K);
  const int n = parts.n;
  const int64_t base = parts.first, prow = parts.stride;
  const int nq = live && n > k ? (n - k + KP - 1) / KP : 0;
  const int64_t lstride = (int64_t)KP * prow;                   // from the q-th part of the group to the next
  const float* lrow = lses + (int64_t)k * prow + base;           // lse of the q-th part: lrow[q * lstride]
  const float* orow = outs + ((int64_t)k * prow + base) * 128;  // its row: orow + q * lstride * 128

  // Group max: lane d4 reads parts q = d4, d4 + 32, ...  The first round of partial rows is
  // requested at the same time: rows do not depend on any lse (the weights reach them by
  // shuffle), so the group waits on one round of memory latency for both.  Then the rows stream
  // in rounds of U, the next round requested before the current one is summed.  Rows of
  // empty parts are loaded too (they lie inside the part buffer) but never enter a sum.
  float l0 = -INFINITY;
  if (d4 < nq) l0 = lrow[d4 * lstride];
  f32x4 o[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < nq) o[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(orow + u * lstride * 128) + d4);
  float m = l0;
  bool full = l0 != -INFINITY;  // a NaN part is not empty
  for (int q = d4 + 32; q < nq; q += 32) {
    const float lq = lrow[q * lstride];
    m = fmaxf(m, lq);
    full |= lq != -INFINITY;
  }
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 32));

  float wsum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if ((uint32_t)(__ballot(full) >> (t & 32)) != 0) {  // any part of the group's 32 lanes
    // Weight of part 32r + d4 on lane d4 for the current round r of 32 parts (0 past the end
    // and for empty parts).
    float wq = l0 == -INFINITY ? 0.f : expf(l0 - m);
#pragma unroll 1
    for (int q = 0; q < nq; q += U) {
      if (q > 0 && (q & 31) == 0) {
        const float lq = q + d4 < nq ? lrow[(q + d4) * lstride] : -INFINITY;
        wq = lq == -INFINITY ? 0.f : expf(lq - m);
      }
      f32x4 cur[U];
#pragma unroll
      for (int u = 0; u < U; ++u) cur[u] = o[u];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q + U + u < nq)
          o[u] = __builtin_nontemporal_load(
              reinterpret_cast<const f32x4*>(orow + (q + U + u) * lstride * 128) + d4);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (q + u < nq) {
          const float w = __shfl(wq, (q + u) & 31, 32);
          wsum += w;
          if (w != 0.f) acc += w * cur[u];
        }
      }
    }
  }
  float M = m;
  if (KP > 1) {
    race_check_delay(t >> 6);
    sm_acc[(rl * KP + k) * 32 + d4] = acc;
    if (d4 == 0) {
      sm_m[rl * KP + k] = m;
      sm_w[rl * KP + k] = wsum;
    }
    __syncthreads();
    race_check_barrier();
    if (k != 0) return;
    M = -INFINITY;
#pragma unroll
    for (int j = 0; j < KP; ++j) M = fmaxf(M, sm_m[rl * KP + j]);
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    wsum = 0.f;
    const float ref = M == -INFINITY ? 0.f : M;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const float s = expf(sm_m[rl * KP + j] - ref);  // 0 for a group of empty parts, whose sums are 0 (or NaN)
      acc += s * sm_acc[(rl * KP + j) * 32 + d4];
      wsum += s * sm_w[rl * KP + j];
    }
  }
  if (!live) return;
  f32x4* dst = reinterpret_cast<f32x4*>(out + dst_row * 128) + d4;
  const float inv = inverse_sum(wsum);
  // Many rows: stored past the caches, so that the launch does not end with them dirty in the L2s
  // (fine's 32,768 rows, 16.8 MB: 2 us of 48).
  if (KP == 1 && !PIECES) __builtin_nontemporal_store(acc * inv, dst);
  else *dst = acc * inv;
  if (lse_out != nullptr && d4 == 0) lse_out[dst_row] = M + logf(wsum);  // -inf where wsum = 0
}

// Few rows of more than four parts (the chunks of few sequences, few partitions of a small batch): a
// workgroup per row, its parts spread over KP thread groups, U per group and round.  Each thread
// reads the lse of its parts itself, beside the rows (32 threads one word), so the group waits on one
// round of memory latency and no shuffle: 32 rows of 32 parts 4.1 -> 3.5 us, 256 rows of 8 parts
// 3.5 -> 3.0 us per call on MI355X (HIP graph).  Later rounds rescale to the running max.
template <int KP, int U>
__global__ __launch_bounds__(32 * KP) void merge_spread_kernel(const float* __restrict__ outs,
                                                               const float* __restrict__ lses, int n_parts,
                                                               MergeRows mr, float* __restrict__ out,
                                                               float* __restrict__ lse_out) {
  __shared__ f32x4 sm_acc[KP * 32];
  __shared__ float sm_m[KP];
  __shared__ float sm_w[KP];
  const int d4 = threadIdx.x & 31;
  const int k = threadIdx.x >> 5;
  const Rows at(mr, blockIdx.x);
  const Parts parts(mr, at, n_parts);
  float m = -INFINITY, wsum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float l[U];
  f32x4 o[U];
  auto request = [&](int p0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u * KP;
      l[u] = -INFINITY;
      if (p < parts.n) {
        const int64_t row = parts.first + p * parts.stride;
        l[u] = lses[row];
        o[u] = reinterpret_cast<const f32x4*>(outs + row * 128)[d4];
      }
    }
  };
  request(k);
  for (int p0 = k; p0 < parts.n; p0 += KP * U) {
    float lc[U];
    f32x4 oc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      lc[u] = l[u];
      oc[u] = o[u];
    }
    if (p0 + KP * U < parts.n) request(p0 + KP * U);  // the next round, before this one is summed
    float top = m;
#pragma unroll
    for (int u = 0; u < U; ++u) top = fmaxf(top, lc[u]);
    // A NaN lse is not in the max but must reach the result, also from a group or round whose other
    // parts are empty: its weight is NaN below, and no sum is left out on account of a max of -inf.
    const float scale = m == top ? 1.f : expf(m - top);
    acc *= scale;
    wsum *= scale;
    m = top;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (lc[u] != -INFINITY) {  // rows of empty parts never enter a sum
        const float w = expf(lc[u] - top);
        wsum += w;
        acc += w * oc[u];
      }
    }
  }
  race_check_delay(threadIdx.x >> 6);
  sm_acc[k * 32 + d4] = acc;
  if (d4 == 0) {
    sm_m[k] = m;
    sm_w[k] = wsum;
  }
  __syncthreads();
  race_check_barrier();
  if (k != 0) return;
  float M = -INFINITY;
#pragma unroll
  for (int j = 0; j < KP; ++j) M = fmaxf(M, sm_m[j]);
  f32x4* dst = reinterpret_cast<f32x4*>(out + at.out * 128) + d4;
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
  wsum = 0.f;
  const float ref = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int j = 0; j < KP; ++j) {
    const float s = expf(sm_m[j] - ref);  // 0 for a group of empty parts, whose sums are 0 (or NaN)
    acc += s * sm_acc[j * 32 + d4];
    wsum += s * sm_w[j];
  }
  // An infinite element times a weight or a rescale that underflowed to 0 is NaN.  Where a sum is not
  // finite the row is summed again, part after part relative to its own max, and parts of weight 0 are
  // left out, as merge_many_kernel does.
  if (!(fabsf((acc[0] + acc[1]) + (acc[2] + acc[3])) < INFINITY)) {
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
    wsum = 0.f;
    for (int p = 0; p < parts.n; ++p) {
      const int64_t row = parts.first + p * parts.stride;
      const float lp = lses[row];
      const float w = lp == -INFINITY ? 0.f : expf(lp - M);
      wsum += w;
      if (w != 0.f) acc += w * reinterpret_cast<const f32x4*>(outs + row * 128)[d4];
    }
  }
  *dst = acc * inverse_sum(wsum);
  if (lse_out != nullptr && d4 == 0) lse_out[at.out] = M + logf(wsum);  // -inf where wsum = 0
}

template <int KP>
hipError_t launch_spread(const float* outs, const float* lses, int n_parts, const MergeRows& m, float* out,
                         float* lse_out, hipStream_t stream) {
  hipLaunchKernelGGL((merge_spread_kernel<KP, 4>), dim3((unsigned)(m.B * m.hn)), dim3(32 * KP), 0, stream, outs, lses,
                     n_parts, m, out, lse_out);
  return hipGetLastError();
}

template <int KP, bool PIECES = false>
hipError_t launch_many(const float* outs, const float* lses, int n_parts, const MergeRows& m, float* out,
                       float* lse_out, hipStream_t stream, const int32_t* prefix = nullptr, int K = 0) {
  constexpr int R = 256 / (32 * KP);
  const int64_t rows = m.B * m.hn;
  const unsigned grid = (unsigned)((rows + R - 1) / R);
  constexpr int U = KP == 1 && !PIECES ? 1 : 4;
  hipLaunchKernelGGL((merge_many_kernel<KP, PIECES, U>), dim3(grid), dim3(256), 0, stream, outs, lses, n_parts, m,
                     out, lse_out, prefix, K);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_merge(const float* outs, const float* lses, int n_parts, MergeRows m, float* out, float* lse_out,
                        hipStream_t stream) {
  const int64_t rows = m.B * m.hn;
  if (rows == 0) return hipSuccess;
  if (n_parts <= 4) {
    hipLaunchKernelGGL(merge_few_kernel<4>, dim3((unsigned)((rows + 7) / 8)), dim3(256), 0, stream, outs, lses,
                       n_parts, m, out, lse_out);
    return hipGetLastError();
  }
  // With enough rows to fill the GPU, one thread group per row streams best.
  // With few rows (the chunks of few sequences, few partitions), spread a row's
  // parts over enough thread groups that each takes them in one round of loads, up to 64 parts (more
  // in further rounds).
  // More rows stream better with one group each, the more parts the sooner (us per call, spread /
  // one group: 8,192 rows of 5, 8, 16, 40 parts 6.9 / 6.9, 8.5 / 9.2, 13.5 / 15.2, 39.6 / 32.9; 16,384
  // rows of 5, 16 parts 10.7 / 9.7, 30.9 / 24.6).
  if (rows < 4096 || (rows <= 8192 && n_parts >= 8 && n_parts <= 16)) {
    if (n_parts <= 8) return launch_spread<2>(outs, lses, n_parts, m, out, lse_out, stream);
    if (n_parts <= 16) return launch_spread<4>(outs, lses, n_parts, m, out, lse_out, stream);
    if (n_parts <= 32) return launch_spread<8>(outs, lses, n_parts, m, out, lse_out, stream);
    return launch_spread<16>(outs, lses, n_parts, m, out, lse_out, stream);
  }
  return launch_many<1>(outs, lses, n_parts, m, out, lse_out, stream);
}

hipError_t launch_merge_pieces(const float* outs, const float* lses, const int32_t* prefix, int K, int kp,
                               MergeRows m, float* out, float* lse_out, hipStream_t stream) {
  const int64_t rows = m.B * m.hn;
  if (rows == 0) return hipSuccess;
  switch (kp) {
    case 1: return launch_many<1, true>(outs, lses, 0, m, out, lse_out, stream, prefix, K);
    case 2: return launch_many<2, true>(outs, lses, 0, m, out, lse_out, stream, prefix, K);
    case 8: return launch_many<8, true>(outs, lses, 0, m, out, lse_out, stream, prefix, K);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bana
