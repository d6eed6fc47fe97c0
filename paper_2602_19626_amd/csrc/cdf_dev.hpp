// Device building blocks of the CDF-24 quantiser (paper section 3.4).
//
// Counts: c_i = max(1, floor(p_i * (T - V))) where the floor is that of the exact product (never
// of a rounded one, see floor_count); the residual T - sum(c), which may be negative, goes to the
// lowest index among the maximal p_i;
// cdf[i + 1] = c_0 + ... + c_i.
//
// Work split: a row of V entries is cut into segments of kSeg = 4096 entries, one 256-thread
// workgroup per (row, segment).  A first pass reduces each segment to a SegPartial (sum of
// counts, argmax, validity); a second pass combines the row's partials in segment order (so the
// result never depends on scheduling), re-reads its segment, and scans it.  Inside a segment,
// thread t owns the four contiguous entries 4t..4t+3 of each of the four 1024-entry quarters,
// so every load and store instruction of a wave covers one contiguous 1 KiB span.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave_dev.hpp"

namespace nc {

constexpr int kSegThreads = 256;
constexpr int kSegWaves = kSegThreads / 64;
constexpr int kQuarter = kSegThreads * 4;  // 1024 entries
constexpr int kSeg = kQuarter * 4;         // 4096 entries per segment
constexpr int kMaxSegs = 64;               // vocab <= 262,144

typedef float f4v __attribute__((ext_vector_type(4)));

// max(1, floor(p * m)) of the exact real product, for finite p in [0, 1] and m < 2^24.  c, the
// truncated float product, is the floor or one above it: rounding is monotonic and every integer
// up to 2^24 is a float, so the rounded product is never below an integer that the exact product
// reaches.  The fused p * m - c rounds once, so its sign is exact and tells the two apart.  Eight
// full-rate instructions for every entry of a row (a 24-bit integer product with its 64-bit shift
// takes thirteen, the shift at quarter rate).  A NaN gives 0, an interval that no coder accepts.
__device__ __forceinline__ uint32_t floor_count(float p, uint32_t m) {
  const float fm = float(m);
  const float c = truncf(p * fm);
  const float f = __builtin_fmaf(p, fm, -c) < 0.f ? c - 1.f : c;
  return uint32_t(f < 1.f ? 1.f : f);
}

// (value, index) maximum with the lowest index winning ties.
__device__ __forceinline__ void argmax_merge(float& v, uint32_t& i, float v2, uint32_t i2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

// Key of (value, index) for valid probabilities: the larger value, then the lower index (the bits of
// floats that are not negative order them; -0 counts as 0).
__device__ __forceinline__ uint64_t max_key(float v, uint32_t i) {
  return (uint64_t(__float_as_uint(v + 0.f)) << 32) | (0xFFFFFFFFu - i);
}
__device__ __forceinline__ float key_value(uint64_t k) { return __uint_as_float(uint32_t(k >> 32)); }
__device__ __forceinline__ uint32_t key_index(uint64_t k) { return 0xFFFFFFFFu - uint32_t(k); }

// Per-(row, segment) reduction result.
struct SegPartial {
  uint32_t sum;   // sum of floor counts of the segment (saturated at 2^32 - 1)
  float maxv;     // largest probability of the segment
  uint32_t maxi;  // its lowest index (row-global)
  int32_t bad;    // 1 if a probability is NaN, negative or above one
};

// Whole-row quantities derived from the partials of one row, combined in segment order.
struct RowQuant {
  uint32_t argmax;
  int32_t residual;
  uint32_t m;      // T - V
  int status;      // 0 valid; 1 bad probability or mass above the total
  uint32_t start;  // cdf value at the first entry of this workgroup's segment
};

__device__ __forceinline__ uint32_t corrected_count(float x, uint32_t idx, const RowQuant& q) {
  const uint32_t cc = floor_count(x, q.m);
  return idx == q.argmax ? uint32_t(int32_t(cc) + q.residual) : cc;
}

// Element index of quarter j, sub-entry i of thread tid in segment seg.
__device__ __forceinline__ uint32_t seg_index(uint32_t seg, int j, int tid, int i) {
  return seg * kSeg + uint32_t(j) * kQuarter + 4u * uint32_t(tid) + uint32_t(i);
}

struct SegLds {
  uint64_t u64[kSegWaves];
  uint64_t best[kSegWaves];
  int flag[kSegWaves];
  uint32_t cols[kSegWaves * 4];
  SegPartial parts[kMaxSegs];
};

// First pass: reduce one segment of probabilities p[j][i] (already zero at or beyond V); tid is
// the thread's index within its 256-thread segment group.
__device__ __forceinline__ SegPartial seg_reduce(const float (&p)[4][4], uint32_t seg, uint32_t V,
                                                 uint32_t m, SegLds& L, int tid) {
  const int lane = tid & 63, w = tid >> 6;
  int bad = 0;
  uint32_t sum = 0;  // (valid probabilities: at most 16 times 2^24)
  uint64_t best = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t idx = seg_index(seg, j, tid, i);
      const float x = p[j][i];
      if (idx < V) {
        if (!(x >= 0.f && x <= 1.f)) bad = 1;  // also catches NaN
        sum += floor_count(x, m);
        const uint64_t k = max_key(x, idx);
        best = k > best ? k : best;
      }
    }
  const uint64_t wsum = wave_sum_u64(sum);
  best = wave_max_u64(best);
  const int wbad = __any(bad) ? 1 : 0;
  if (lane == 0) {
    L.u64[w] = wsum;
    L.best[w] = best;
    L.flag[w] = wbad;
  }
  __syncthreads();
  SegPartial r;
  uint64_t tot = 0;
  best = 0;
  r.bad = 0;
#pragma unroll
  for (int k = 0; k < kSegWaves; ++k) {
    tot += L.u64[k];
    best = L.best[k] > best ? L.best[k] : best;
    r.bad |= L.flag[k];
  }
  r.maxv = key_value(best);
  r.maxi = key_index(best);
  r.sum = tot >= 0xFFFFFFFFull ? 0xFFFFFFFFu : uint32_t(tot);
  return r;
}

// Second pass, row part: combine the row's partials (in LDS) in segment order into the residual,
// the argmax and this segment's starting CDF value.
// parts: kMaxSegs entries (in LDS), the first nseg of them the row's partials.
__device__ __forceinline__ RowQuant seg_combine(const SegPartial* parts, uint32_t nseg,
                                                uint32_t seg, uint32_t V, uint32_t total) {
  RowQuant q;
  q.m = total - V;
  uint64_t tot = 0, before = 0;
  float bv = -1.f;
  uint32_t bi = 0xFFFFFFFFu;
  int bad = 0;
  // partials read sixteen at a time (parts holds kMaxSegs entries, so every read is in range)
  // and combined in segment order
  for (uint32_t k0 = 0; k0 < nseg; k0 += 16) {
    SegPartial buf[16];
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) buf[u] = parts[k0 + u];
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) {
      const uint32_t k = k0 + u;
      if (k < nseg) {
        const SegPartial& s = buf[u];
        if (k < seg) before += s.sum;
        tot += s.sum;
        argmax_merge(bv, bi, s.maxv, s.maxi);
        bad |= s.bad;
      }
    }
  }
  const int64_t r = int64_t(total) - int64_t(tot);
  q.argmax = bi;
  q.residual = int32_t(r);
  q.status = bad | (tot >= 0xFFFFFFFFull ? 1 : 0) | (bi < V ? 0 : 1);
  if (!q.status && int64_t(floor_count(bv, q.m)) + r < 1) q.status = 1;
  if (bi < V && bi / kSeg < seg) before += uint64_t(int64_t(r));
  q.start = uint32_t(before);
  return q;
}

// Second pass, segment part: exclusive scan of the corrected counts of this segment.  On return
// base[j] = cdf[seg_index(seg, j, tid, 0)] and c[j][i] is the corrected count of entry (j, i)
// (0 at or beyond V), so cdf[idx + 1] = base[j] + c[j][0] + ... + c[j][i].
__device__ __forceinline__ void seg_scan(const float (&p)[4][4], uint32_t seg, uint32_t V,
                                         const RowQuant& q, uint32_t (&base)[4],
                                         uint32_t (&c)[4][4], SegLds& L, int tid) {
  const int lane = tid & 63, w = tid >> 6;
  uint32_t excl[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t idx = seg_index(seg, j, tid, i);
      c[j][i] = idx < V ? corrected_count(p[j][i], idx, q) : 0u;
      s += c[j][i];
    }
    const uint32_t v = wave_scan_u32(s);
    if (lane == 63) L.cols[w * 4 + j] = v;
    excl[j] = v - s;
  }
  __syncthreads();
  uint32_t acc = q.start;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t off = 0, coltot = 0;
#pragma unroll
    for (int k = 0; k < kSegWaves; ++k) {
      const uint32_t s = L.cols[k * 4 + j];
      off += (k < w) ? s : 0u;
      coltot += s;
    }
    base[j] = acc + off + excl[j];
    acc += coltot;
  }
}

}  // namespace nc
