// Per-token vocabulary chain over a batch of streams (one row per stream and step):
//   softmax of z + b (paper section 3.3 with the section 3.7 bias, temperature 1),
//   coding distribution: bias head alone (warmup), n-gram alone (section 3.8 skip), the linear
//   mix of section 3.6, or the softmax-gated ensemble,
//   CDF-24 quantisation and scan (section 3.4) with the interval gather (encode) or the target
//   search (decode) of section 3.9,
//   online updates: bias head SGD (section 3.7), exponential-weights mixer (section 3.6), n-gram
//   counts with the 64-slot cap (section 3.5), ensemble backward + SGD,
//   n-gram prediction of the next position, its entropy and the skip decision (section 3.8).
//
// Rows are cut into 4096-entry segments, one 256-thread workgroup per (segment, row), and every
// cross-segment combination runs in segment order, so each row's result is independent of the
// launch shape and of the other rows.  No float atomics are used.
#include "cdf_dev.hpp"
#include "common.hpp"
#include "vocab_dev.hpp"

// The same probability must come out of the counting pass and the scanning pass bit for bit, so
// no multiply-add contraction is allowed to differ between them: contraction is off here.
#pragma clang fp contract(off)

namespace nc {

// ---- shared row arithmetic -----------------------------------------------------------------

__device__ __forceinline__ LsePart lse_merge(LsePart a, LsePart b) {
  const float M = fmaxf(a.m, b.m);
  if (M == -INFINITY) return LsePart{-INFINITY, 0.f};
  return LsePart{M, a.s * expf(a.m - M) + b.s * expf(b.m - M)};
}

// The logsumexp partial of a wave's 64 partials by one tree: lane L merges lane L + d for
// d = 1, 2, 4, ... with the lower lane first.  Lanes whose partner is another tree node's (or
// missing) hold values that no node of lane 0's tree reads.
template <int kCtrl>
__device__ __forceinline__ LsePart dpp_lse(LsePart a) {
  return lse_merge(a, LsePart{dpp_f<kCtrl>(a.m), dpp_f<kCtrl>(a.s)});
}
__device__ __forceinline__ LsePart wave_lse(LsePart p) {
  p = dpp_lse<kShl + 1>(p);
  p = dpp_lse<kShl + 2>(p);
  p = dpp_lse<kShl + 4>(p);
  p = dpp_lse<kShl + 8>(p);
  LsePart q[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) q[k] = LsePart{read_lane(p.m, 16 * k), read_lane(p.s, 16 * k)};
  return lse_merge(lse_merge(q[0], q[1]), lse_merge(q[2], q[3]));
}

// Logsumexp of a row from its segment partials, merged in segment order; lane k of the wave holds
// partial k (mine).  The running maxima of the fold are exact whatever the order, so lane k computes
// the two factors of merge k and only the products and sums are serial.
__device__ __forceinline__ float row_lse(const LsePart mine, int nseg, int lane) {
  const float run = wave_scan_max(lane < nseg ? mine.m : -INFINITY);
  const float prev = dpp_f<kWaveShr1>(run, -INFINITY);
  const bool empty = run == -INFINITY;
  const float e1 = empty ? 0.f : expf(prev - run);
  const float e2 = empty ? 0.f : mine.s * expf(mine.m - run);
  float acc = read_lane(mine.s, 0);
  for (int k = 1; k < nseg; ++k) acc = acc * read_lane(e1, k) + read_lane(e2, k);
  return read_lane(run, nseg - 1) + logf(acc);
}

struct RowIn {
  const float* z;   // logits of the row (modes that use the LLM)
  const float* b;   // bias vector of the stream
  const float* png; // n-gram distribution of the stream
  const float* pk;  // P_1..P_K (ensemble)
  float lse;
  int mode, use_head, K, V;
  float w[kMaxExperts];
};

// Mixture / gate weights of a stream: mixer w = exp(log w); ensemble w = softmax(theta).
__device__ __forceinline__ void row_weights(const VocabParams& P, const float* lw, float* w) {
  if (P.ensemble) {
    // every one of the kMaxOrder + 1 slots is read and written unconditionally (entries past n
    // masked by selects), so that w stays in registers; the kept terms are combined in order
    const int n = P.K + 1;
    float l[kMaxOrder + 1];
#pragma unroll
    for (int j = 0; j <= kMaxOrder; ++j) l[j] = lw[j];
    float mx = l[0];
#pragma unroll
    for (int j = 1; j <= kMaxOrder; ++j) mx = j < n ? fmaxf(mx, l[j]) : mx;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j <= kMaxOrder; ++j) {
      const float e = expf(l[j] - mx);
      s = j < n ? s + e : s;
    }
#pragma unroll
    for (int j = 0; j <= kMaxOrder; ++j) w[j] = j < n ? expf(l[j] - mx) / s : 0.f;
  } else {
    // (the same slots written as by the ensemble branch, so that the two merge by value)
    w[0] = expf(lw[0]);
    w[1] = expf(lw[1]);
#pragma unroll
    for (int j = 2; j <= kMaxOrder; ++j) w[j] = 0.f;
  }
}

__device__ __forceinline__ bool uses_llm(int mode) { return mode != M_SKIP; }

// ---- the per-segment steps ------------------------------------------------------------------
//
// Each step is a device function of (segment, row, thread index within a 256-thread segment
// group), run by one workgroup per (segment, row).  Steps that contain barriers take an `active`
// flag: an inactive group passes through the barriers and touches nothing, so several groups of
// one workgroup could share them.

// V1: logsumexp partial of z + b over one segment
__device__ __forceinline__ void v1_seg(const VocabParams& P, const StreamState& S,
                                       const StepArgs& A, int seg, int r, int nseg, int tid,
                                       bool active, LsePart* wl) {
  const int lane = tid & 63, w = tid >> 6;
  const int V = P.V;
  const int s = A.rows[r];
  LsePart part{-INFINITY, 0.f};
  if (active && uses_llm(S.mode[s])) {
    const float* z = A.z + (size_t)r * V;
    const float* b = S.b + (size_t)s * V;
    float u[4][4];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t0 = seg_index(seg, j, tid, 0);
      if (t0 + 3 < uint32_t(V)) {
        const f4v zz = *reinterpret_cast<const f4v*>(z + t0);
        const f4v bb = P.use_head ? *reinterpret_cast<const f4v*>(b + t0) : f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) u[j][i] = P.use_head ? zz[i] + bb[i] : zz[i];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t t = t0 + i;
          u[j][i] = t < uint32_t(V) ? (P.use_head ? z[t] + b[t] : z[t]) : -INFINITY;
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) m = fmaxf(m, u[j][i]);
    }
    float sum = 0.f;
    if (m != -INFINITY)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum += expf(u[j][i] - m);
    part = LsePart{m, sum};
  }
  part = wave_lse(part);
  if (lane == 0) wl[w] = part;
  __syncthreads();
  if (active && tid == 0) {
    LsePart acc = wl[0];
    for (int k = 1; k < kSegWaves; ++k) acc = lse_merge(acc, wl[k]);
    A.lse_parts[(size_t)r * nseg + seg] = acc;
  }
  __syncthreads();  // wl is reused by the next call
}

// Row setup shared by V2 and V3 (identical code, identical results).
__device__ __forceinline__ RowIn make_row(const VocabParams& P, const StreamState& S,
                                          const StepArgs& A, int r, int s, int nseg) {
  RowIn R;
  R.V = P.V;
  R.K = P.K;
  R.mode = S.mode[s];
  R.use_head = P.use_head;
  R.z = A.z + (size_t)r * P.V;
  R.b = S.b + (size_t)s * P.V;
  R.png = S.png + (size_t)s * P.V;
  R.pk = S.pk ? S.pk + (size_t)s * P.K * P.V : nullptr;
  const int lane = threadIdx.x & 63;
  const LsePart mine = A.lse_parts[(size_t)r * nseg + min(lane, nseg - 1)];
  R.lse = uses_llm(R.mode) ? row_lse(mine, nseg, lane) : 0.f;
  for (int j = 0; j < kMaxExperts; ++j) R.w[j] = 0.f;
  row_weights(P, S.lw + (size_t)s * kMaxExperts, R.w);
  return R;
}

// This thread's 16 entries of segment seg (4 contiguous per quarter) of the row's logits, bias and
// n-gram probabilities, loaded as vectors before the row's mode is known (the mode only selects
// among them), so that these loads overlap the row-metadata loads.  V % 4 == 0: a group of four
// is whole or past the end (zero).
struct RowVec {
  f4v z[4], b[4], g[4];
};
__device__ __forceinline__ void row_fetch(const VocabParams& P, const StreamState& S,
                                          const StepArgs& A, int r, int s, uint32_t seg, int tid,
                                          RowVec& v) {
  const float* z = A.z + (size_t)r * P.V;
  const float* b = S.b + (size_t)s * P.V;
  const float* g = S.png + (size_t)s * P.V;
  const f4v zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t t0 = seg_index(seg, j, tid, 0);
    const bool in = t0 < uint32_t(P.V);
    v.z[j] = in ? *reinterpret_cast<const f4v*>(z + t0) : zero4;
    v.b[j] = in && P.use_head ? *reinterpret_cast<const f4v*>(b + t0) : zero4;
    v.g[j] = in ? *reinterpret_cast<const f4v*>(g + t0) : zero4;
  }
}

// Probabilities of this thread's 16 entries of segment seg from the fetched vectors, zero at or
// beyond V (kEns: the row may be an ensemble's).
template <bool kEns = true>
__device__ __forceinline__ void row_probs(const RowIn& R, const RowVec& v, uint32_t seg, int tid,
                                          float (&p)[4][4], float (&pt)[4][4]) {
  if (kEns && R.mode == M_ENS) {
    // The ensemble also reads P_1..P_K at the thread's 16 entries: every vector is requested
    // (clamped into the row, masked after) before the first is used, rather than one dependent
    // load per entry and order.  p = w0 q + w1 P_1 + ... + wK P_K, added in that order.
    f4v pk[4][kMaxOrder];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t0 = seg_index(seg, j, tid, 0);
      const uint32_t tc = t0 < uint32_t(R.V) ? t0 : 0u;
#pragma unroll
      for (int k = 0; k < kMaxOrder; ++k)
        pk[j][k] = *reinterpret_cast<const f4v*>(R.pk + (size_t)min(k, R.K - 1) * R.V + tc);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t0 = seg_index(seg, j, tid, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (t0 >= uint32_t(R.V)) {
          p[j][i] = pt[j][i] = 0.f;
          continue;
        }
        const float q = expf((R.use_head ? v.z[j][i] + v.b[j][i] : v.z[j][i]) - R.lse);
        pt[j][i] = q;
        float pv = R.w[0] * q;
#pragma unroll
        for (int k = 1; k <= kMaxOrder; ++k)
          if (k <= R.K) pv = pv + R.w[k] * pk[j][k - 1][i];
        p[j][i] = pv;
      }
    }
    return;
  }
  // The other forms, one loop per form (the mode is the row's, uniform over the workgroup):
  // SKIP p = g; LLM p = q; MIX p = w0 q + w1 g; with q = exp(z (+ b) - lse) the bias-head
  // probability, returned in pt (0 for SKIP).
  if (R.mode == M_SKIP) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = seg_index(seg, j, tid, 0) < uint32_t(R.V);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[j][i] = in ? v.g[j][i] : 0.f;
        pt[j][i] = 0.f;
      }
    }
    return;
  }
  const bool mix = R.mode == M_MIX;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool in = seg_index(seg, j, tid, 0) < uint32_t(R.V);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float q = expf((R.use_head ? v.z[j][i] + v.b[j][i] : v.z[j][i]) - R.lse);
      pt[j][i] = in ? q : 0.f;
      p[j][i] = in ? (mix ? R.w[0] * q + R.w[1] * v.g[j][i] : q) : 0.f;
    }
  }
}

// V2: count partial of one segment
__device__ __forceinline__ void v2_seg(const VocabParams& P, const StreamState& S,
                                       const StepArgs& A, int seg, int r, int nseg, int tid,
                                       bool active, SegLds& L) {
  float p[4][4], pt[4][4];
  RowIn R;
  if (active) {
    const int s = A.rows[r];
    RowVec v;
    row_fetch(P, S, A, r, s, seg, tid, v);
    R = make_row(P, S, A, r, s, nseg);
    row_probs(R, v, seg, tid, p, pt);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) p[j][i] = 0.f;
  }
  const SegPartial sp = seg_reduce(p, seg, P.V, P.total - P.V, L, tid);
  if (active && tid == 0) static_cast<SegPartial*>(A.seg_parts)[(size_t)r * nseg + seg] = sp;
  __syncthreads();  // L is reused by the next call
}

// V3: scan of one segment, the interval (encode) or the target search (decode), the outcome and
// the bias-head step on the segment's entries
__device__ __forceinline__ void v3_seg(const VocabParams& P, const StreamState& S,
                                       const StepArgs& A, int seg, int r, int nseg, int tid,
                                       bool active, SegLds& L, int* s_sym) {
  const int V = P.V;
  const int s = A.rows[r];
  // Issue order: the count partials of the row's segments (into registers; an LDS store right
  // after the load would wait for it before anything else is issued), the row's vectors and
  // metadata, then the key (decode: the host's target; encode: the token at the stream's next
  // position, behind the committed count), all before the scan needs any of them.
  SegPartial part{};
  if (active)
    part = static_cast<const SegPartial*>(A.seg_parts)[(size_t)r * nseg + min(tid, nseg - 1)];
  RowIn R;
  RowVec v;
  float p[4][4], pt[4][4];
  if (active) {
    row_fetch(P, S, A, r, s, seg, tid, v);
    R = make_row(P, S, A, r, s, nseg);
  }
  const int i_pos = !active ? 0 : (A.pos >= 0 ? A.pos : S.ncommit[s]);
  const uint32_t key =
      !active ? 0u
              : (A.decode ? (A.targets ? A.targets[r] : A.targets_in[r])
                          : uint32_t(S.hist[(size_t)s * S.maxT + i_pos]));
  if (active && tid < nseg) L.parts[tid] = part;
  if (tid == 0) *s_sym = -1;
  if (active) {
    row_probs(R, v, seg, tid, p, pt);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) p[j][i] = pt[j][i] = 0.f;
  }
  __syncthreads();
  RowQuant q{};
  if (active) q = seg_combine(L.parts, nseg, seg, V, P.total);
  uint32_t base[4], cnt[4][4];
  seg_scan(p, seg, V, q, base, cnt, L, tid);
  int found = -1;
  uint32_t fcl = 0, fch = 0;
  float fp = 0.f, fpt = 0.f, fpng = 0.f;
  if (active) {
    // the entry whose interval holds the key (decode) or the key's entry (encode), by selects
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t run = base[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t t = seg_index(seg, j, tid, i);
        const uint32_t c = cnt[j][i];
        const bool hit = t < uint32_t(V) &&
                         (A.decode ? (key >= run && key - run < c) : (t == key));
        found = hit ? int(t) : found;
        fcl = hit ? run : fcl;
        fch = hit ? run + c : fch;
        fp = hit ? p[j][i] : fp;
        fpt = hit ? pt[j][i] : fpt;
        fpng = hit ? v.g[j][i] : fpng;  // the row's p_ng at t, fetched with the row
        run += c;
      }
    }
    // full-row diagnostics (single-row probes)
    if (A.dbg_cdf || A.dbg_p || A.dbg_pt) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t run = base[j];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t t = seg_index(seg, j, tid, i);
          run += cnt[j][i];
          if (t >= uint32_t(V)) continue;
          if (A.dbg_cdf) A.dbg_cdf[(size_t)r * (V + 1) + t + 1] = run;
          if (A.dbg_p) A.dbg_p[(size_t)r * V + t] = p[j][i];
          if (A.dbg_pt) A.dbg_pt[(size_t)r * V + t] = pt[j][i];
        }
      }
    }
    if (A.dbg_cdf && seg == 0 && tid == 0) A.dbg_cdf[(size_t)r * (V + 1)] = 0;
    if (found >= 0 && !A.no_update) {
      *s_sym = found;
      Outcome o;
      o.sym = q.status ? -1 : found;
      o.cl = fcl;
      o.ch = fch;
      o.mode = R.mode;
      o.p = fp;
      o.pt = fpt;
      o.png = fpng;
      o.lse = R.lse;
      for (int k = 0; k < kMaxOrder; ++k)
        o.pk[k] = (R.pk && k < P.K) ? R.pk[(size_t)k * V + found] : 0.f;
      for (int k = 0; k < kMaxExperts; ++k) o.r[k] = 0.f;
      if (R.mode == M_ENS) {
        o.r[0] = R.w[0] * fpt / fp;
#pragma unroll
        for (int k = 1; k <= kMaxOrder; ++k)
          if (k <= P.K) o.r[k] = R.w[k] * o.pk[k - 1] / fp;
      }
      A.out[r] = o;
      if (A.iv) {
        A.iv[((size_t)s * S.maxT + i_pos) * 2 + 0] = fcl;
        A.iv[((size_t)s * S.maxT + i_pos) * 2 + 1] = fch;
      }
      if (A.ptok) A.ptok[(size_t)s * S.maxT + i_pos] = fp;
    }
    if (found >= 0 && A.no_update) *s_sym = found;
    if (q.status && seg == 0 && tid == 0) {
      // invalid distribution: report through the outcome; no symbol can be coded
      Outcome o{};
      o.sym = -1;
      o.mode = R.mode;
      A.out[r] = o;
    }
  }
  // bias-head SGD step on -log ptilde(t*), section 3.7 (entries of this segment only)
  __syncthreads();
  if (active && P.use_head && !P.ensemble && (R.mode == M_LLM || R.mode == M_MIX) && !q.status &&
      !A.no_update) {
    const int sym = A.decode ? *s_sym : int(key);
    float* b = S.b + (size_t)s * V;
    // b was fetched with the row (use_head) and only this workgroup writes these entries
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t0 = seg_index(seg, j, tid, 0);
      if (t0 >= uint32_t(V)) continue;
      f4v nb;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float ind = int(t0) + i == sym ? 1.f : 0.f;
        nb[i] = v.b[j][i] - P.head_lr * (pt[j][i] - ind);
      }
      *reinterpret_cast<f4v*>(b + t0) = nb;
    }
  }
  __syncthreads();  // L and s_sym are reused by the next call
}

// V4: ensemble backward + SGD on b over one segment (no barriers)
__device__ __forceinline__ void v4_seg(const VocabParams& P, const StreamState& S,
                                       const StepArgs& A, int seg, int r, int tid) {
  const int s = A.rows[r];
  const Outcome o = A.out[r];
  if (o.sym < 0 || o.mode != M_ENS) return;
  const int V = P.V;
  const float* z = A.z + (size_t)r * V;
  float* b = S.b + (size_t)s * V;
  const float r0 = o.r[0];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t t = seg_index(seg, j, tid, i);
      if (t < uint32_t(V)) {
        const float q0 = expf(z[t] + b[t] - o.lse);
        const float ind = int(t) == o.sym ? 1.f : 0.f;
        b[t] = b[t] - P.head_lr * (r0 * (q0 - ind));
      }
    }
}

// ---- V5: n-gram + mixer / gate update with the coded symbol --------------------------------

// A context of up to kMaxOrder tokens.  Held by value and walked by loops unrolled to the
// compile-time bound (with the order k as a guard), so that it stays in registers.
struct Ctx {
  int32_t v[kMaxOrder];
};

__device__ __forceinline__ uint32_t ctx_hash(const Ctx& c, int k) {
  uint64_t h = 0x9E3779B97F4A7C15ull * uint64_t(k + 1);
#pragma unroll
  for (int i = 0; i < kMaxOrder; ++i)
    if (i < k) {
      h ^= uint64_t(uint32_t(c.v[i])) + 0x632BE59BD9B4E019ull + (h << 6) + (h >> 2);
      h *= 0xBF58476D1CE4E5B9ull;
    }
  h ^= h >> 31;
  return uint32_t(h);
}

// Probe the order-k table t for the context c.v[0..k); returns the pool index or -1, and the
// empty table slot where it would go in *ins.
__device__ __forceinline__ int ctx_find(const StreamState& S, size_t t, const Ctx& c, int k,
                                         int* ins) {
  typedef int32_t i4 __attribute__((ext_vector_type(4)));
  static_assert(kMaxOrder == 4, "a table key is one 16-byte vector");
  const i4* keys = reinterpret_cast<const i4*>(S.keys + t * S.cap * 4);
  const int32_t* kidx = S.kidx + t * S.cap;
  uint32_t h = ctx_hash(c, k) & uint32_t(S.cap - 1);
  for (int probe = 0; probe < S.cap; ++probe) {
    // the slot's pool index and key are requested together (the key is read whether or not the
    // slot is in use)
    const int id = kidx[h];
    const i4 kk = keys[h];
    bool eq = true;
#pragma unroll
    for (int i = 0; i < kMaxOrder; ++i)
      if (i < k) eq = eq && kk[i] == c.v[i];
    if (id < 0) {
      *ins = int(h);
      return -1;
    }
    if (eq) return id;
    h = (h + 1) & uint32_t(S.cap - 1);
  }
  *ins = -1;
  return -1;
}

// thread k of the row's update (k = 0: unigram, history, mixer / gate; k = 1..K: order-k table);
// k < 0 does nothing but pass the barriers
__device__ __forceinline__ void v5_row(const VocabParams& P, const StreamState& S,
                                       const StepArgs& A, int r, int k) {
  const int s = A.rows[r];
  const int32_t* hist = S.hist + (size_t)s * S.maxT;
  // With the position given (encode) the counts take the known token in hist, whatever the step's
  // outcome; the mixer update reads the outcome.
  const bool given = A.pos >= 0 && !A.decode;
  const Outcome o = A.out[r];
  const int i = k < 0 ? 0 : (A.pos >= 0 ? A.pos : S.ncommit[s]);
  const int sym = given ? hist[i] : o.sym;
  const bool on = k >= 0 && sym >= 0 && (given || o.sym >= 0);
  __syncthreads();
  if (on && k == 0) {
    if (A.decode) S.hist[(size_t)s * S.maxT + i] = sym;
    if (P.use_ngram || P.ensemble) {
      S.uni[(size_t)s * P.V + sym] += 1;
      S.nseen[s] += 1;
    }
  }
  if (on && k == 0 && o.sym >= 0) {
    float* lw = S.lw + (size_t)s * kMaxExperts;
    if (o.mode == M_MIX) {
      // exponential weights (section 3.6): log w_j += eta log p_j(t*), then renormalise
      lw[0] = lw[0] + P.mix_eta * logf(o.pt);
      lw[1] = lw[1] + P.mix_eta * logf(o.png);
      const float mx = fmaxf(lw[0], lw[1]);
      const float ls = mx + logf(expf(lw[0] - mx) + expf(lw[1] - mx));
      lw[0] = lw[0] - ls;
      lw[1] = lw[1] - ls;
    } else if (o.mode == M_ENS) {
      float w[kMaxExperts];
      row_weights(P, lw, w);
#pragma unroll
      for (int j = 0; j <= kMaxOrder; ++j)
        if (j <= P.K) lw[j] = lw[j] - P.head_lr * (w[j] - o.r[j]);
    }
  }
  if (on && (P.use_ngram || P.ensemble) && k >= 1 && k <= P.K) {
    const size_t t = (size_t)s * P.K + (k - 1);
    Ctx ctx{};
    // insert t* as a continuation of the order-k context ending at t_{i-1}
    if (i >= k) {
#pragma unroll
      for (int q = 0; q < kMaxOrder; ++q)
        if (q < k) ctx.v[q] = hist[i - k + q];
      int ins = -1;
      int id = ctx_find(S, t, ctx, k, &ins);
      if (id < 0) {
        if (ins >= 0 && S.nctx[t] < min(S.maxctx, P.ngram_max_contexts)) {
          id = S.nctx[t]++;
#pragma unroll
          for (int q = 0; q < 4; ++q) S.keys[(t * S.cap + ins) * 4 + q] = q < k ? ctx.v[q] : -1;
          S.kidx[t * S.cap + ins] = id;
          int32_t* sl = S.pool + (t * S.maxctx + id) * kSlots * 2;
          sl[0] = sym;
          sl[1] = 1;
          S.pool_n[t * S.maxctx + id] = 1;
          S.pool_sum[t * S.maxctx + id] = 1;
        }
      } else {
        int32_t* sl = S.pool + (t * S.maxctx + id) * kSlots * 2;
        const int n = S.pool_n[t * S.maxctx + id];
        // first slot holding t*, or n: eight slots per round of loads rather than one dependent
        // load per slot (kSlots is a multiple of 8, so a round stays inside the pool)
        static_assert(kSlots % 8 == 0, "slot rounds of eight");
        int j = n;
        for (int j0 = 0; j0 < n; j0 += 8) {
          typedef int32_t i4 __attribute__((ext_vector_type(4)));
          const i4* q4 = reinterpret_cast<const i4*>(sl + 2 * j0);
          const i4 a0 = q4[0], a1 = q4[1], a2 = q4[2], a3 = q4[3];
          const int32_t tk[8] = {a0.x, a0.z, a1.x, a1.z, a2.x, a2.z, a3.x, a3.z};
          int hit = -1;
#pragma unroll
          for (int u = 7; u >= 0; --u)
            if (j0 + u < n && tk[u] == sym) hit = j0 + u;
          if (hit >= 0) {
            j = hit;
            break;
          }
        }
        if (j < n) {
          sl[2 * j + 1] += 1;
          S.pool_sum[t * S.maxctx + id] += 1;
        } else if (n < kSlots) {
          sl[2 * n] = sym;
          sl[2 * n + 1] = 1;
          S.pool_n[t * S.maxctx + id] = n + 1;
          S.pool_sum[t * S.maxctx + id] += 1;
        } else {
          int ev = 0;  // lowest count, lowest slot index on ties
          for (int q = 1; q < kSlots; ++q)
            if (sl[2 * q + 1] < sl[2 * ev + 1]) ev = q;
          S.pool_sum[t * S.maxctx + id] += 1 - sl[2 * ev + 1];
          sl[2 * ev] = sym;
          sl[2 * ev + 1] = 1;
        }
      }
    }
    // context of the next position: t_{i-k+1} .. t_i (= t*)
    int nid = -1;
    if (i + 1 >= k) {
#pragma unroll
      for (int q = 0; q < kMaxOrder; ++q) {
        if (q < k - 1) ctx.v[q] = hist[i - k + 1 + q];
        if (q == k - 1) ctx.v[q] = sym;
      }
      int ins;
      nid = ctx_find(S, t, ctx, k, &ins);
    }
    S.next_ctx[(size_t)s * kMaxOrder + (k - 1)] = nid;
  }
  __syncthreads();
  if (on && k == 0) S.ncommit[s] = i + 1;
}

// ---- V6: dense n-gram prediction of the current position ------------------------------------

struct NgRow {
  float lam[kMaxOrder];
  int present[kMaxOrder];
  int id[kMaxOrder];  // pool index of the order-k context of the next position, or -1
  int n[kMaxOrder];   // its total count n_k
  float inv_norm;     // 1 / (N + V)
};

// The row's n-gram weights.  Lane q (mod kMaxOrder) of each wave fetches order q's context index
// and then that context's total count, and every lane reads the four orders' values from those
// lanes: two vector loads per row.  (Per-order scalar loads of the same values were issued one
// after the other, each behind the previous one's wait.)  Must be called by whole waves.
__device__ __forceinline__ NgRow ng_row(const VocabParams& P, const StreamState& S, int s) {
  static_assert((kMaxOrder & (kMaxOrder - 1)) == 0, "kMaxOrder must be a power of two");
  NgRow g;
  const int q = threadIdx.x & (kMaxOrder - 1);
  const int raw = S.next_ctx[(size_t)s * kMaxOrder + q];
  const int seen = S.nseen[s];
  const int idq = q < P.K ? raw : -1;
  // (indices clamped into the tables; a missing context's count is masked)
  const int nraw = S.pool_sum[((size_t)s * P.K + min(q, P.K - 1)) * S.maxctx + max(idq, 0)];
  const int nq = idq >= 0 ? nraw : 0;
#pragma unroll
  for (int k = 0; k < kMaxOrder; ++k) {
    g.id[k] = __builtin_amdgcn_readlane(idq, k);
    g.n[k] = __builtin_amdgcn_readlane(nq, k);
  }
#pragma unroll
  for (int k = 0; k < kMaxOrder; ++k) {
    g.present[k] = g.n[k] > 0 ? 1 : 0;
    g.lam[k] = g.present[k] ? float(g.n[k]) / (float(g.n[k]) + P.ngram_eps) : 0.f;
  }
  g.inv_norm = 1.0f / float(seen + P.V);
  return g;
}

__device__ __forceinline__ void v6_seg(const VocabParams& P, const StreamState& S,
                                       const int32_t* rows, NgPart* parts, int seg, int r,
                                       int nseg, int tid, bool active, NgPart* wl) {
  const int lane = tid & 63, w = tid >> 6;
  const int V = P.V;
  const int s = rows[r];
  float h = 0.f, mx = 0.f;
  if (active) {
    // unigram counts in, dense P_K out, four contiguous entries per load and store (V % 4 == 0)
    typedef int32_t i4v __attribute__((ext_vector_type(4)));
    i4v u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t0 = seg_index(seg, j, tid, 0);
      u[j] = t0 < uint32_t(V) ? *reinterpret_cast<const i4v*>(S.uni + (size_t)s * V + t0)
                              : i4v{0, 0, 0, 0};
    }
    const NgRow g = ng_row(P, S, s);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t0 = seg_index(seg, j, tid, 0);
      if (t0 >= uint32_t(V)) continue;
      f4v out;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t t = t0 + i;
        float pv = float(u[j][i] + 1) * g.inv_norm;  // unigram base (n_t + 1) / (N + V)
        // orders unrolled to the compile-time bound: with a runtime trip count the row weights
        // were indexed dynamically and kept in LDS, two LDS round trips per entry and order
#pragma unroll
        for (int k = 1; k <= kMaxOrder; ++k) {
          if (k > P.K) break;
          if (g.present[k - 1]) pv = (1.0f - g.lam[k - 1]) * pv;
          if (S.pk) S.pk[((size_t)s * P.K + (k - 1)) * V + t] = pv;
        }
        out[i] = pv;
        h = h - pv * log2f(pv);
        mx = fmaxf(mx, pv);
      }
      *reinterpret_cast<f4v*>(S.png + (size_t)s * V + t0) = out;
    }
  }
  h = wave_sum_f(h);
  mx = wave_max_f(mx);
  if (lane == 0) wl[w] = NgPart{h, mx};
  __syncthreads();
  if (active && tid == 0) {
    NgPart acc = wl[0];
    for (int k = 1; k < kSegWaves; ++k) {
      acc.h += wl[k].h;
      acc.mx = fmaxf(acc.mx, wl[k].mx);
    }
    parts[(size_t)r * nseg + seg] = acc;
  }
  __syncthreads();  // wl is reused by the next call
}

// ---- V7: sparse n-gram entries, entropy, skip decision ---------------------------------------

struct alignas(16) FixLds {
  int lt[kMaxOrder][kSlots], lc[kMaxOrder][kSlots], ln[kMaxOrder];
  float sh[kSegThreads], smx[kSegThreads];
};

// The last of the first ln slots of order row q holding tok, or -1 (a pool holds a token at most
// once, so it is also the first); four slots per LDS read.
__device__ __forceinline__ int slot_last(const FixLds& F, int q, int ln, int tok) {
  static_assert(kSlots % 4 == 0, "slot rows are read four at a time");
  typedef int32_t i4 __attribute__((ext_vector_type(4)));
  const i4* row = reinterpret_cast<const i4*>(F.lt[q]);
  int at = -1;
  for (int j0 = 0; j0 < ln; j0 += 4) {
    const i4 v = row[j0 >> 2];
    if (v.x == tok) at = j0;
    if (v.y == tok && j0 + 1 < ln) at = j0 + 1;
    if (v.z == tok && j0 + 2 < ln) at = j0 + 2;
    if (v.w == tok && j0 + 3 < ln) at = j0 + 3;
  }
  return at;
}

// 256 threads (tid) of one row; active == false only passes the barriers
__device__ __forceinline__ void v7_row(const VocabParams& P, const StreamState& S,
                                       const int32_t* rows, const NgPart* parts, int nseg,
                                       StepOut* step_out, const Outcome* out, int r, int tid,
                                       bool active, FixLds& F) {
  const int nt = kSegThreads;
  const int V = P.V;
  const int s = rows[r];
  // inputs of the final reduction and of the packed outcome, fetched now so that their latency
  // overlaps the n-gram chain below
  NgPart pre_part{0.f, 0.f};
  if (active && tid < nseg) pre_part = parts[(size_t)r * nseg + tid];
  int pre_pos = 0, pre_sym = 0;
  uint32_t pre_cl = 0, pre_ch = 0;
  float pre_p = 0.f;
  if (active && tid == 0) {
    pre_pos = S.ncommit[s];
    if (step_out) {
      pre_sym = out[r].sym;
      pre_cl = out[r].cl;
      pre_ch = out[r].ch;
      pre_p = out[r].p;
    }
  }
  NgRow g{};
  if (active) g = ng_row(P, S, s);
  if (active && tid < kMaxOrder) F.ln[tid] = 0;
  __syncthreads();
  // wave w reads the kSlots slots of order w + 1 (one slot per lane), so the order is
  // wave-uniform and the row's per-order values are picked without indexing
  static_assert(kSlots == 64 && kMaxOrder * kSlots <= kSegThreads, "one wave per order");
  const int kw = __builtin_amdgcn_readfirstlane(tid >> 6);  // order - 1 of this wave
  int w_present = 0, w_id = -1;
#pragma unroll
  for (int q = 0; q < kMaxOrder; ++q)
    if (kw == q) {
      w_present = g.present[q];
      w_id = g.id[q];
    }
  if (active && kw < P.K && w_present) {
    const int k = kw + 1, j = tid & 63, id = w_id;
    const size_t t = (size_t)s * P.K + (k - 1);
    // the slot is read whether or not it is in use (readers stop at ln), so the slot and the
    // slot count load together
    const int2 tc = *reinterpret_cast<const int2*>(S.pool + ((t * S.maxctx + id) * kSlots + j) * 2);
    const int n = S.pool_n[t * S.maxctx + id];
    if (j == 0) F.ln[k - 1] = n;
    F.lt[k - 1][j] = tc.x;
    F.lc[k - 1][j] = tc.y;
  }
  __syncthreads();
  float dh = 0.f, dmx = 0.f;
  if (active)
    for (int e = tid; e < P.K * kSlots; e += nt) {
      const int k = e / kSlots + 1, j = e % kSlots;
      if (j >= F.ln[k - 1]) continue;
      const int tok = F.lt[k - 1][j];
      // the entry's unigram count and current p_ng are requested before the slot scans
      const int32_t u_tok = S.uni[(size_t)s * V + tok];
      const float old = S.png[(size_t)s * V + tok];
      bool owner = true;  // first occurrence over (order, slot) in increasing order
      for (int k2 = 1; k2 < k && owner; ++k2) owner = slot_last(F, k2 - 1, F.ln[k2 - 1], tok) < 0;
      if (!owner) continue;
      // P_k(tok) = lambda_k Phat_k(tok) + (1 - lambda_k) P_{k-1}(tok), k = 1..K (section 3.5)
      float pv = float(u_tok + 1) * g.inv_norm;  // unigram base (n_t + 1) / (N + V)
#pragma unroll
      for (int k2 = 1; k2 <= kMaxOrder; ++k2) {
        if (k2 > P.K) break;
        if (g.present[k2 - 1]) {
          const int at = slot_last(F, k2 - 1, F.ln[k2 - 1], tok);
          const int cnt = at >= 0 ? F.lc[k2 - 1][at] : 0;
          const float n = float(g.n[k2 - 1]);
          pv = g.lam[k2 - 1] * (float(cnt) / n) + (1.0f - g.lam[k2 - 1]) * pv;
        }
        if (S.pk) S.pk[((size_t)s * P.K + (k2 - 1)) * V + tok] = pv;
      }
      S.png[(size_t)s * V + tok] = pv;
      dh = dh + (old * log2f(old) - pv * log2f(pv));
      dmx = fmaxf(dmx, pv);
    }
  // sparse corrections: wave sums, then the four waves' in order; the dense segment partials are
  // staged in LDS by as many threads, then added in segment order
  dh = wave_sum_f(dh);
  dmx = wave_max_f(dmx);
  if (active && (tid & 63) == 0) {
    F.sh[tid >> 6] = dh;
    F.smx[tid >> 6] = dmx;
  }
  if (active && tid < nseg) {
    F.sh[kSegWaves + tid] = pre_part.h;
    F.smx[kSegWaves + tid] = pre_part.mx;
  }
  __syncthreads();
  if (active && tid == 0) {
    float H = 0.f, mx = 0.f;
    for (int k = 0; k < nseg; ++k) {
      H += F.sh[kSegWaves + k];
      mx = fmaxf(mx, F.smx[kSegWaves + k]);
    }
    float sh = F.sh[0], smx = F.smx[0];
    for (int k = 1; k < kSegWaves; ++k) {
      sh = sh + F.sh[k];
      smx = fmaxf(smx, F.smx[k]);
    }
    H = H + sh;
    mx = fmaxf(mx, smx);
    S.H[s] = H;
    S.pmax[s] = mx;
    const int pos = pre_pos;
    int mode;
    if (P.ensemble) {
      mode = M_ENS;
    } else {
      const bool warm = pos < P.warmup;
      bool skip = false;
      if (P.use_skip && !warm) {
        if (P.skip_mode == 1) skip = H < P.skip_bits;
        if (P.skip_mode == 2) skip = mx >= P.skip_pmax;
      }
      mode = skip ? M_SKIP : ((warm || !P.use_mixer) ? M_LLM : M_MIX);
    }
    S.mode[s] = mode;
    if (step_out) {
      StepOut so{};
      so.sym = pre_sym;
      so.cl = pre_cl;
      so.ch = pre_ch;
      so.next_mode = mode;
      so.p = pre_p;
      step_out[r] = so;
    }
  }
}

// ---- the segmented kernels: one workgroup per (segment, row) ---------------------------------

__global__ __launch_bounds__(kSegThreads) void vocab_lse_kernel(VocabParams P, StreamState S,
                                                                StepArgs A) {
  __shared__ LsePart wl[kSegWaves];
  v1_seg(P, S, A, blockIdx.x, blockIdx.y, gridDim.x, threadIdx.x, true, wl);
}

__global__ __launch_bounds__(kSegThreads) void vocab_count_kernel(VocabParams P, StreamState S,
                                                                  StepArgs A) {
  __shared__ SegLds L;
  v2_seg(P, S, A, blockIdx.x, blockIdx.y, gridDim.x, threadIdx.x, true, L);
}

__global__ __launch_bounds__(kSegThreads) void vocab_scan_kernel(VocabParams P, StreamState S,
                                                                 StepArgs A) {
  __shared__ SegLds L;
  __shared__ int s_sym;
  v3_seg(P, S, A, blockIdx.x, blockIdx.y, gridDim.x, threadIdx.x, true, L, &s_sym);
}

__global__ __launch_bounds__(kSegThreads) void ensemble_bias_kernel(VocabParams P, StreamState S,
                                                                    StepArgs A) {
  v4_seg(P, S, A, blockIdx.x, blockIdx.y, threadIdx.x);
}

__global__ __launch_bounds__(64) void ngram_update_kernel(VocabParams P, StreamState S,
                                                          StepArgs A) {
  v5_row(P, S, A, blockIdx.x, threadIdx.x);
}

__global__ __launch_bounds__(kSegThreads) void ngram_dense_kernel(VocabParams P, StreamState S,
                                                                  const int32_t* rows,
                                                                  NgPart* parts) {
  __shared__ NgPart wl[kSegWaves];
  v6_seg(P, S, rows, parts, blockIdx.x, blockIdx.y, gridDim.x, threadIdx.x, true, wl);
}

__global__ __launch_bounds__(kSegThreads) void ngram_fix_kernel(VocabParams P, StreamState S,
                                                                const int32_t* rows,
                                                                const NgPart* parts, int nseg,
                                                                StepOut* step_out,
                                                                const Outcome* out) {
  __shared__ FixLds F;
  v7_row(P, S, rows, parts, nseg, step_out, out, blockIdx.x, threadIdx.x, true, F);
}

// ---- chunks of known tokens (encode, committed prompts) ----------------------------------------
//
// Where the tokens of a run of positions are known, neither the n-gram models nor the logits of
// those positions depend on the coding of any of them; only the bias head and the mixer weights
// run from position to position.  A chunk of positions is therefore taken apart:
//   known_advance   updates the tables with the chunk's tokens, one wave per (order, stream), and
//                   leaves what each position's prediction needs: its contexts' slots and counts;
//   known_dense,    the n-gram distribution, entropy and mode of every position of the chunk at
//   known_fix       once;
//   known_commit    unigram counts;
//   known_first     the logsumexp partials of the chunk's first position;
//   known_run,      up to kRunGroups workgroups: probabilities and the bias step of all positions in
//   known_count     one launch, then every position's count partials;
//   known_step      more workgroups, one launch per position: probabilities, count partials, the bias
//                   step and the logsumexp partials of the next position, whose bias is then known;
//   known_finish    the intervals of every position from the count partials.
// Every value is computed by the expressions, and reduced in the order, of the step-by-step
// kernels above, so the coded bits are those of the sequential decode.

// The order-k context of position i (tokens i - k .. i - 1) in table t: its pool index or -1, and
// the empty slot where it would go.  Eight slots of the probe sequence per round of loads, one per
// lane (ctx_find's sequence and result).
__device__ __forceinline__ int wave_ctx_find(const StreamState& S, size_t t, const Ctx& c, int k,
                                             int lane, int* ins) {
  typedef int32_t i4 __attribute__((ext_vector_type(4)));
  const i4* keys = reinterpret_cast<const i4*>(S.keys + t * S.cap * 4);
  const int32_t* kidx = S.kidx + t * S.cap;
  const uint32_t h = ctx_hash(c, k);
  for (int p0 = 0; p0 < S.cap; p0 += 8) {
    const uint32_t at = (h + p0 + (lane & 7)) & uint32_t(S.cap - 1);
    const int id = kidx[at];
    const i4 kk = keys[at];
    bool eq = true;
#pragma unroll
    for (int i = 0; i < kMaxOrder; ++i)
      if (i < k) eq = eq && kk[i] == c.v[i];
    const uint64_t stop = __ballot(id < 0 || eq) & 0xFF;
    if (stop) {
      const int l = __builtin_ctzll(stop);
      *ins = __builtin_amdgcn_readlane(int(at), l);
      const int found = __builtin_amdgcn_readlane(id, l);
      return found < 0 ? -1 : found;
    }
  }
  *ins = -1;
  return -1;
}

// One wave per (order k = blockIdx.x + 1, row): the chunk's tokens are inserted one after the other
// (the update kernel's rules), the current context's slots held one per lane.  Before each token
// the slots and counts are left in the snapshot of its position.  Bound by two dependent reads per
// token, the table slot and then the slots of the context found there.
__global__ __launch_bounds__(64) void known_advance_kernel(VocabParams P, StreamState S,
                                                           KnownChunk C, int p0) {
  const int k = blockIdx.x + 1, r = blockIdx.y, lane = threadIdx.x;
  const int s = C.s0 + r, np = min(C.np, C.left[r]);
  const size_t t = (size_t)s * P.K + (k - 1);
  const int32_t* hist = S.hist + (size_t)s * S.maxT;
  const int most = min(S.maxctx, P.ngram_max_contexts);
  int nctx = S.nctx[t];
  int id = -1, ins = -1, n = 0, sum = 0;  // the context of the position
  int2 slot{-1, 0};                       // this lane's slot of it
  auto take = [&](int i) {                // the context of position i
    Ctx c{};
#pragma unroll
    for (int q = 0; q < kMaxOrder; ++q)
      if (q < k) c.v[q] = hist[i - k + q];
    const int old = id;
    id = wave_ctx_find(S, t, c, k, lane, &ins);
    if (id < 0) {
      n = sum = 0;
    } else if (id != old) {
      slot = *reinterpret_cast<const int2*>(S.pool + ((t * S.maxctx + id) * kSlots + lane) * 2);
      n = S.pool_n[t * S.maxctx + id];
      sum = S.pool_sum[t * S.maxctx + id];
    }
  };
  if (p0 >= k) take(p0);
  for (int j = 0; j < np; ++j) {
    const int i = p0 + j;
    const size_t at = ((size_t)j * C.B + r) * P.K + (k - 1);
    C.slots[at * kSlots + lane] = slot;
    if (lane == 0) C.counts[at] = int2{n, sum};
    const int tok = hist[i];
    if (i >= k) {
      int32_t* sl = S.pool + (t * S.maxctx + max(id, 0)) * kSlots * 2;
      int put = -1;  // the slot that changes
      if (id < 0) {
        if (ins >= 0 && nctx < most) {
          id = nctx++;
          sl = S.pool + (t * S.maxctx + id) * kSlots * 2;
          if (lane < 4) {
            int v = -1;
#pragma unroll
            for (int q = 0; q < kMaxOrder; ++q)
              if (q == lane && q < k) v = hist[i - k + q];
            S.keys[(t * S.cap + ins) * 4 + lane] = v;
          }
          if (lane == 0) S.kidx[t * S.cap + ins] = id;
          put = 0;
          n = sum = 1;
          if (lane == put) slot = int2{tok, 1};
        }
      } else {
        const uint64_t hit = __ballot(lane < n && slot.x == tok);
        if (hit) {
          put = __builtin_ctzll(hit);
          if (lane == put) slot.y += 1;
          sum += 1;
        } else if (n < kSlots) {
          put = n++;
          if (lane == put) slot = int2{tok, 1};
          sum += 1;
        } else {  // the lowest count, the lowest slot index on ties
          const uint32_t key = (uint32_t(slot.y) << 6) | uint32_t(lane);
          uint32_t low = key;
#pragma unroll
          for (int d = 1; d < 64; d <<= 1) low = min(low, uint32_t(__shfl_xor(low, d, 64)));
          put = int(low & 63);
          sum += 1 - int(low >> 6);
          if (lane == put) slot = int2{tok, 1};
        }
      }
      if (put >= 0) {
        if (lane == put) *reinterpret_cast<int2*>(sl + 2 * lane) = slot;
        if (lane == 0) {
          S.pool_n[t * S.maxctx + id] = n;
          S.pool_sum[t * S.maxctx + id] = sum;
        }
        // the wave's later reads of these places come after the writes
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      }
    }
    if (i + 1 >= k) take(i + 1);
  }
  if (lane == 0) {
    S.nctx[t] = nctx;
    S.next_ctx[(size_t)s * kMaxOrder + (k - 1)] = id;
  }
}

// The n-gram weights of a position from its snapshot (ng_row's expressions).
__device__ __forceinline__ void known_row(const VocabParams& P, const KnownChunk& C, int j, int r,
                                          int seen, NgRow& g) {
  const int2* cnt = C.counts + ((size_t)j * C.B + r) * P.K;
#pragma unroll
  for (int k = 0; k < kMaxOrder; ++k) {
    g.id[k] = -1;
    const int sum = cnt[min(k, P.K - 1)].y;
    g.n[k] = k < P.K ? sum : 0;
    g.present[k] = g.n[k] > 0 ? 1 : 0;
    g.lam[k] = g.present[k] ? float(g.n[k]) / (float(g.n[k]) + P.ngram_eps) : 0.f;
  }
  g.inv_norm = 1.0f / float(seen + P.V);
}

// The dense distribution of kKnownRun positions of one row over one segment (v6_seg for each): the
// unigram counts stay in registers and take each position's token.  The tokens of the chunk before
// the first of these positions are added through LDS.
constexpr int kKnownRun = 4;
__global__ __launch_bounds__(kSegThreads) void known_dense_kernel(VocabParams P, StreamState S,
                                                                  KnownChunk C, int p0) {
  typedef int32_t i4v __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) int32_t s_u[kSeg];
  __shared__ NgPart wl[2][kSegWaves];
  const int seg = blockIdx.x, r = blockIdx.z, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j0 = blockIdx.y * kKnownRun;
  const int s = C.s0 + r, V = P.V, np = min(C.np, C.left[r]), nseg = gridDim.x;
  if (j0 >= np) return;
  const int32_t* hist = S.hist + (size_t)s * S.maxT + p0;
  i4v u[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t t0 = seg_index(seg, q, tid, 0);
    u[q] = t0 < uint32_t(V) ? *reinterpret_cast<const i4v*>(S.uni + (size_t)s * V + t0)
                            : i4v{0, 0, 0, 0};
  }
  if (j0 > 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) reinterpret_cast<i4v*>(s_u)[q * kSegThreads + tid] = i4v{0, 0, 0, 0};
    __syncthreads();
    for (int q = tid; q < j0; q += kSegThreads) {
      const uint32_t off = uint32_t(hist[q]) - uint32_t(seg) * kSeg;
      if (off < uint32_t(kSeg)) atomicAdd(s_u + off, 1);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] += reinterpret_cast<const i4v*>(s_u)[q * kSegThreads + tid];
  }
  const int seen = S.nseen[s];
  const int j1 = min(j0 + kKnownRun, np);
  for (int j = j0; j < j1; ++j) {
    NgRow g;
    known_row(P, C, j, r, seen + j, g);
    float h = 0.f, mx = 0.f;
    float* png = C.png + ((size_t)j * C.B + r) * V;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t t0 = seg_index(seg, q, tid, 0);
      if (t0 >= uint32_t(V)) continue;
      f4v out;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float pv = float(u[q][i] + 1) * g.inv_norm;
#pragma unroll
        for (int k = 1; k <= kMaxOrder; ++k) {
          if (k > P.K) break;
          if (g.present[k - 1]) pv = (1.0f - g.lam[k - 1]) * pv;
        }
        out[i] = pv;
        h = h - pv * log2f(pv);
        mx = fmaxf(mx, pv);
      }
      *reinterpret_cast<f4v*>(png + t0) = out;
    }
    h = wave_sum_f(h);
    mx = wave_max_f(mx);
    if (lane == 0) wl[j & 1][w] = NgPart{h, mx};
    __syncthreads();
    if (tid == 0) {
      NgPart acc = wl[j & 1][0];
      for (int k = 1; k < kSegWaves; ++k) {
        acc.h += wl[j & 1][k].h;
        acc.mx = fmaxf(acc.mx, wl[j & 1][k].mx);
      }
      C.ngp[((size_t)j * C.B + r) * nseg + seg] = acc;
    }
    const uint32_t off = uint32_t(hist[j]) - uint32_t(seg) * kSeg;
    if (off < uint32_t(kSeg) && int((off % kQuarter) >> 2) == tid) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (int(off / kQuarter) == q && int(off & 3) == i) u[q][i] += 1;
    }
  }
}

// The sparse entries, entropy and mode of one position of one row (v7_row), and its token.
__global__ __launch_bounds__(kSegThreads) void known_fix_kernel(VocabParams P, StreamState S,
                                                                KnownChunk C, int p0, int nseg) {
  __shared__ FixLds F;
  extern __shared__ int32_t s_tok[];  // the chunk's tokens before the position
  const int j = blockIdx.x, r = blockIdx.y, tid = threadIdx.x;
  const int s = C.s0 + r, V = P.V;
  if (j >= min(C.np, C.left[r])) return;
  const size_t row = (size_t)j * C.B + r;
  const int32_t* hist = S.hist + (size_t)s * S.maxT + p0;
  float* png = C.png + row * V;
  NgPart pre_part{0.f, 0.f};
  if (tid < nseg) pre_part = C.ngp[row * nseg + tid];
  for (int q = tid; q < j; q += kSegThreads) s_tok[q] = hist[q];
  if (tid == 0) C.tok[row] = hist[j];
  NgRow g;
  known_row(P, C, j, r, S.nseen[s] + j, g);
  const int kw = __builtin_amdgcn_readfirstlane(tid >> 6);  // order - 1 of this wave
  if (kw < kMaxOrder) {
    const int kc = min(kw, P.K - 1);
    const int2 tc = C.slots[(row * P.K + kc) * kSlots + (tid & 63)];
    const int n = C.counts[row * P.K + kc].x;
    if ((tid & 63) == 0) F.ln[kw] = kw < P.K ? n : 0;
    F.lt[kw][tid & 63] = tc.x;
    F.lc[kw][tid & 63] = tc.y;
  }
  __syncthreads();
  float dh = 0.f, dmx = 0.f;
  // (one entry per thread: P.K * kSlots <= kSegThreads)
  if (kw < P.K && (tid & 63) < F.ln[kw]) {
    const int k = kw + 1, tok = F.lt[kw][tid & 63];
    int u_tok = S.uni[(size_t)s * V + tok];
    const float old = png[tok];
    bool owner = true;
    for (int k2 = 1; k2 < k && owner; ++k2) owner = slot_last(F, k2 - 1, F.ln[k2 - 1], tok) < 0;
    if (owner) {
#pragma unroll 8
      for (int q = 0; q < j; ++q) u_tok += s_tok[q] == tok ? 1 : 0;
      float pv = float(u_tok + 1) * g.inv_norm;
#pragma unroll
      for (int k2 = 1; k2 <= kMaxOrder; ++k2) {
        if (k2 > P.K) break;
        if (g.present[k2 - 1]) {
          const int at = slot_last(F, k2 - 1, F.ln[k2 - 1], tok);
          const int cnt = at >= 0 ? F.lc[k2 - 1][at] : 0;
          const float n = float(g.n[k2 - 1]);
          pv = g.lam[k2 - 1] * (float(cnt) / n) + (1.0f - g.lam[k2 - 1]) * pv;
        }
      }
      png[tok] = pv;
      dh = dh + (old * log2f(old) - pv * log2f(pv));
      dmx = fmaxf(dmx, pv);
    }
  }
  dh = wave_sum_f(dh);
  dmx = wave_max_f(dmx);
  if ((tid & 63) == 0) {
    F.sh[tid >> 6] = dh;
    F.smx[tid >> 6] = dmx;
  }
  if (tid < nseg) {
    F.sh[kSegWaves + tid] = pre_part.h;
    F.smx[kSegWaves + tid] = pre_part.mx;
  }
  __syncthreads();
  if (tid != 0) return;
  float H = 0.f, mx = 0.f;
  for (int k = 0; k < nseg; ++k) {
    H += F.sh[kSegWaves + k];
    mx = fmaxf(mx, F.smx[kSegWaves + k]);
  }
  float sh = F.sh[0], smx = F.smx[0];
  for (int k = 1; k < kSegWaves; ++k) {
    sh = sh + F.sh[k];
    smx = fmaxf(smx, F.smx[k]);
  }
  H = H + sh;
  mx = fmaxf(mx, smx);
  const bool warm = p0 + j < P.warmup;
  bool skip = false;
  if (P.use_skip && !warm) {
    if (P.skip_mode == 1) skip = H < P.skip_bits;
    if (P.skip_mode == 2) skip = mx >= P.skip_pmax;
  }
  C.mode[row] = skip ? M_SKIP : ((warm || !P.use_mixer) ? M_LLM : M_MIX);
}

// Without the n-gram: every position is the model's.
__global__ void known_tokens_kernel(StreamState S, KnownChunk C, int p0) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= C.np * C.B) return;
  const int j = e / C.B, r = e % C.B;
  if (j >= C.left[r]) return;
  C.tok[e] = S.hist[(size_t)(C.s0 + r) * S.maxT + p0 + j];
  C.mode[e] = M_LLM;
}

// Unigram counts (integer adds, any order) and the committed position of each row.
__global__ __launch_bounds__(kSegThreads) void known_commit_kernel(VocabParams P, StreamState S,
                                                                   KnownChunk C, int p0) {
  const int r = blockIdx.x, s = C.s0 + r, np = min(C.np, C.left[r]);
  const int32_t* hist = S.hist + (size_t)s * S.maxT + p0;
  if (P.use_ngram)
    for (int j = threadIdx.x; j < np; j += blockDim.x)
      atomicAdd(S.uni + (size_t)s * P.V + hist[j], 1);
  if (threadIdx.x == 0) {
    if (P.use_ngram) S.nseen[s] += np;
    if (np > 0) S.ncommit[s] = p0 + np;
  }
}

// The mixer weights after a position: exponential weights (section 3.6), then renormalised.
__device__ __forceinline__ void mixer_step(const VocabParams& P, int mode, float pt, float png,
                                           float (&lw)[2]) {
  if (mode != M_MIX) return;
  lw[0] = lw[0] + P.mix_eta * logf(pt);
  lw[1] = lw[1] + P.mix_eta * logf(png);
  const float mx = fmaxf(lw[0], lw[1]);
  const float ls = mx + logf(expf(lw[0] - mx) + expf(lw[1] - mx));
  lw[0] = lw[0] - ls;
  lw[1] = lw[1] - ls;
}

// Logsumexp partials of position j over u = z_j + b (v1_seg's reduction): every thread's 16 values.
__device__ __forceinline__ LsePart known_lse(const float (&u)[4][4]) {
  float m = -INFINITY;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) m = fmaxf(m, u[q][i]);
  float sum = 0.f;
  if (m != -INFINITY)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) sum += expf(u[q][i] - m);
  return wave_lse(LsePart{m, sum});
}
__device__ __forceinline__ LsePart known_lse_sum(const LsePart* wl) {
  LsePart acc = wl[0];
  for (int k = 1; k < kSegWaves; ++k) acc = lse_merge(acc, wl[k]);
  return acc;
}
__device__ __forceinline__ void known_lse_store(const KnownChunk& C, int j, int r, int seg,
                                                int nseg, const LsePart* wl) {
  C.lse[((size_t)(j & 1) * C.B + r) * nseg + seg] = known_lse_sum(wl);
}

// Two floats as one word that is not kUnset.
constexpr uint64_t kUnset = ~uint64_t(0);
__device__ __forceinline__ uint64_t sync_word(float lo, float hi) {
  const uint64_t v = uint64_t(__float_as_uint(hi)) << 32 | __float_as_uint(lo);
  return v == kUnset ? 0x7FC000007FC00000ull : v;  // (both NaN either way)
}
__device__ __forceinline__ uint64_t sync_word(const LsePart& p) { return sync_word(p.m, p.s); }

// The chunk's first position: its logsumexp partials.
__global__ __launch_bounds__(kSegThreads) void known_first_kernel(VocabParams P, StreamState S,
                                                                  KnownChunk C) {
  __shared__ LsePart wl[kSegWaves];
  const int seg = blockIdx.x, r = blockIdx.y, tid = threadIdx.x;
  const float* z = C.z + (size_t)r * P.V;
  const float* b = S.b + (size_t)(C.s0 + r) * P.V;
  float u[4][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t t0 = seg_index(seg, q, tid, 0);
    const bool in = t0 < uint32_t(P.V);
    const f4v zz = *reinterpret_cast<const f4v*>(z + (in ? t0 : 0));
    const f4v bb = *reinterpret_cast<const f4v*>(b + (in ? t0 : 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) u[q][i] = !in ? -INFINITY : (P.use_head ? zz[i] + bb[i] : zz[i]);
  }
  const LsePart part = known_lse(u);
  if ((tid & 63) == 0) wl[tid >> 6] = part;
  __syncthreads();
  if (tid == 0) known_lse_store(C, 0, r, seg, gridDim.x, wl);
  if (!C.sync) return;
  const int ns = gridDim.x + 1;
  uint64_t* sync = C.sync + (size_t)r * ns;
  if (tid == 0) sync[seg] = sync_word(known_lse_sum(wl));
  for (int j = tid; j < C.np; j += kSegThreads) {
    if (j > 0) sync[(size_t)j * C.B * ns + seg] = kUnset;
    if (seg == 0) sync[(size_t)j * C.B * ns + ns - 1] = kUnset;
  }
}

// A wave's part of a position's counts: their sum, the sum before the token, the largest entry.
struct KnownSums {
  uint64_t sum, best;
  uint32_t before;
  int bad;
};

// The probabilities of the position's token, recorded by the thread that holds its entry; word, if
// any, tells them to the row's other workgroups.
__device__ __forceinline__ void known_outcome(const KnownChunk& C, size_t row, int seg, int tid,
                                              int mode, int tok, const float (&p)[4][4],
                                              const float (&pt)[4][4], const f4v (&g)[4],
                                              uint64_t* word) {
  if (uint32_t(tok) / kSeg != uint32_t(seg)) return;  // (uniform)
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (seg_index(seg, q, tid, i) == uint32_t(tok)) {
        const float png = C.png ? g[q][i] : 0.f;
        if (word)
          __hip_atomic_store(word, sync_word(pt[q][i], png), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        KnownRec& o = C.rec[row];
        o.p = p[q][i];
        o.pt = pt[q][i];
        o.png = png;
        o.mode = mode;
      }
}

// The wave's counts of row's position; the thread that holds the token's entry records its count.
__device__ __forceinline__ KnownSums known_counts(const VocabParams& P, const KnownChunk& C,
                                                  size_t row, int seg, int tid, int tok,
                                                  const float (&p)[4][4]) {
  const int V = P.V;
  const uint32_t m = P.total - uint32_t(V);
  uint32_t sum = 0, before = 0;
  int bad = 0;
  uint64_t best = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t t = seg_index(seg, q, tid, i);
      const float x = p[q][i];
      const uint32_t c = t < uint32_t(V) ? floor_count(x, m) : 0u;
      sum += c;
      before += t < uint32_t(tok) ? c : 0u;
      if (t < uint32_t(V)) {
        if (!(x >= 0.f && x <= 1.f)) bad = 1;
        const uint64_t key = max_key(x, t);
        best = key > best ? key : best;
      }
      if (t == uint32_t(tok)) C.rec[row].c = c;
    }
  return KnownSums{wave_sum_u64(sum), wave_max_u64(best), wave_sum_u32(before), __any(bad) ? 1 : 0};
}

// The position's count partial of the segment from its waves', and the counts before the token.
__device__ __forceinline__ void known_store(const KnownChunk& C, size_t row, int seg, int nseg,
                                            int tok, const KnownSums* ws) {
  uint64_t tot = 0, bk = 0;
  uint32_t bf = 0;
  int bd = 0;
#pragma unroll
  for (int k = 0; k < kSegWaves; ++k) {
    tot += ws[k].sum;
    bf += ws[k].before;
    bk = ws[k].best > bk ? ws[k].best : bk;
    bd |= ws[k].bad;
  }
  SegPartial sp;
  sp.sum = tot >= 0xFFFFFFFFull ? 0xFFFFFFFFu : uint32_t(tot);
  sp.maxv = key_value(bk);
  sp.maxi = key_index(bk);
  sp.bad = bd;
  static_cast<SegPartial*>(C.segs)[row * nseg + seg] = sp;
  if (uint32_t(tok) / kSeg == uint32_t(seg)) C.rec[row].before = bf;
}

// Bias-head step on -log ptilde(t*), section 3.7 (b in place), and u = z2 + b of the next position.
__device__ __forceinline__ void known_bias(const VocabParams& P, bool learn, int seg, int tid,
                                           int tok, const float (&pt)[4][4], const f4v (&z2)[4],
                                           f4v (&b)[4], float (&u)[4][4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t t0 = seg_index(seg, q, tid, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float ind = int(t0) + i == tok ? 1.f : 0.f;
      if (learn) b[q][i] = b[q][i] - P.head_lr * (pt[q][i] - ind);
      u[q][i] = t0 >= uint32_t(P.V) ? -INFINITY : (P.use_head ? z2[q][i] + b[q][i] : z2[q][i]);
    }
  }
}

// Position j of the chunk, one workgroup per (segment, row); see above for what it leaves.  A chain
// of np such launches is what a stream's encoding takes, so what counts is the time of one: every
// load goes out at once, and the reductions stay in registers.  7.0 us a position at one stream
// (V = 49,152), where logsumexp, count, scan and update were four dependent launches of 21.9 us
// ordered against the n-gram's three by events.  64 streams: 15.3 us a
// position against 39.9 us, bound by memory.
__global__ __launch_bounds__(kSegThreads) void known_step_kernel(VocabParams P, StreamState S,
                                                                 KnownChunk C, int j) {
  __shared__ LsePart s_lse[kSegWaves];
  __shared__ KnownSums s_sums[kSegWaves];
  const int seg = blockIdx.x, r = blockIdx.y, nseg = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int V = P.V, s = C.s0 + r;
  const size_t row = (size_t)j * C.B + r;
  const bool more = j + 1 < C.np;
  const float* z = C.z + row * V;
  const float* zn = more ? z + (size_t)C.B * V : z;
  const float* gp = C.png ? C.png + row * V : z;
  float* b = S.b + (size_t)s * V;
  RowVec v;
  f4v z2[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    // (an index past the end reads the row's start; masked below)
    const uint32_t t0 = seg_index(seg, q, tid, 0), tc = t0 < uint32_t(V) ? t0 : 0;
    v.z[q] = *reinterpret_cast<const f4v*>(z + tc);
    v.b[q] = *reinterpret_cast<const f4v*>(b + tc);
    v.g[q] = *reinterpret_cast<const f4v*>(gp + tc);
    z2[q] = *reinterpret_cast<const f4v*>(zn + tc);
  }
  const LsePart mine = C.lse[((size_t)(j & 1) * C.B + r) * nseg + min(lane, nseg - 1)];
  const KnownRec last = C.rec[j > 0 ? row - C.B : row];
  const float* lws = j > 1 ? C.lw + ((size_t)((j - 1) & 1) * C.B + r) * 2
                           : S.lw + (size_t)s * kMaxExperts;
  float lw[2] = {lws[0], lws[1]};
  const int mode = C.mode[row], tok = C.tok[row];
  const int mode2 = C.mode[more ? row + C.B : row];
  const int left = C.left[r];
  if (j >= left) return;  // the row has ended (uniform over the workgroup)
  // mixer weights of this position: the last position's outcome, taken by every workgroup alike
  if (j > 0) {
    mixer_step(P, last.mode, last.pt, last.png, lw);
    if (seg == 0 && tid < 2) C.lw[((size_t)(j & 1) * C.B + r) * 2 + tid] = tid ? lw[1] : lw[0];
  }
  RowIn R;
  R.V = V;
  R.K = P.K;
  R.mode = mode;
  R.use_head = P.use_head;
  R.lse = uses_llm(mode) ? row_lse(mine, nseg, lane) : 0.f;
  R.w[0] = expf(lw[0]);
  R.w[1] = expf(lw[1]);
  float p[4][4], pt[4][4];
  row_probs<false>(R, v, seg, tid, p, pt);
  known_outcome(C, row, seg, tid, mode, tok, p, pt, v.g, nullptr);
  const KnownSums sums = known_counts(P, C, row, seg, tid, tok, p);
  // the bias-head step, then the next position's logsumexp with it
  const bool learn = P.use_head && uses_llm(mode);
  float u[4][4];
  known_bias(P, learn, seg, tid, tok, pt, z2, v.b, u);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t t0 = seg_index(seg, q, tid, 0);
    if (learn && t0 < uint32_t(V)) *reinterpret_cast<f4v*>(b + t0) = v.b[q];
  }
  const bool lse2 = more && j + 1 < left && uses_llm(mode2);
  const LsePart part = lse2 ? known_lse(u) : LsePart{-INFINITY, 0.f};
  if (lane == 0) {
    s_sums[w] = sums;
    s_lse[w] = part;
  }
  __syncthreads();
  if (tid == 0) known_store(C, row, seg, nseg, tok, s_sums);
  if (tid == 64 && lse2) known_lse_store(C, j + 1, r, seg, nseg, s_lse);
}

// The chunk's positions in one launch, one workgroup per (segment, row) over all of them: the bias
// stays in registers and the next position's logits and n-gram probabilities arrive while this one is
// computed.  Between two positions the row's workgroups exchange the segments' logsumexp partials and
// the token's probabilities (which move the mixer): each is one 64-bit word of its own per position,
// unset at first, stored and polled at device scope, so a word that is set is also whole.  A position is
// bound by its instructions (one wave a SIMD), so the counts are left to known_count_kernel, which
// takes all positions at once from the probabilities that this kernel leaves.  One stream, V = 49,152:
// 3.1 us a position alone and 4.1 beside a transformer pass (5.2 and 7.2 with the counts in it), where
// a launch per position took 6.2 and 9.8; encoding 4,096 tokens 42.5 to 33.8 ms, bound by the passes.
// A workgroup waits for those of its own row only, so all that a wait needs is that they get to run:
// two workgroups fit a CU, and kRunGroups is half of what the chip holds, which leaves room for a second
// context's.  If they still do not run (many contexts at once) a wait ends after C.polls polls, a
// few tenths of a second, and raises its flag, with which the caller takes the positions one by one.
// More rows than that gain less: 33 BF16 streams of 1,000 tokens (396 workgroups) 39.5 ms, or 36.8 in
// one launch; 64 streams 68.1 and 68.2, 200 streams 66.4 and 68.0.
constexpr int kRunGroups = 256;

__device__ __forceinline__ uint64_t sync_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void sync_store(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kSegThreads) void known_run_kernel(VocabParams P, StreamState S,
                                                                KnownChunk C) {
  __shared__ LsePart s_lse[2][kSegWaves];
  const int seg = blockIdx.x, r = blockIdx.y, nseg = gridDim.x, ns = nseg + 1;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int V = P.V, s = C.s0 + r;
  const int n = min(C.np, C.left[r]);
  if (n <= 0) return;
  const size_t step = (size_t)C.B * V;
  float* b = S.b + (size_t)s * V;
  uint32_t tc[4];  // (an index past the end reads the row's start; masked below)
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t t0 = seg_index(seg, q, tid, 0);
    tc[q] = t0 < uint32_t(V) ? t0 : 0;
  }
  auto fetch = [&](f4v(&d)[4], const float* src) {
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = *reinterpret_cast<const f4v*>(src + tc[q]);
  };
  float* z0 = C.z + (size_t)r * V;
  const float* g0 = C.png ? C.png + (size_t)r * V : z0;
  RowVec v;
  f4v z2[4], z3[4], g2[4];
  fetch(v.b, b);
  fetch(v.z, z0);
  fetch(v.g, g0);
  fetch(z2, z0 + (n > 1 ? step : 0));
  float lw[2] = {S.lw[(size_t)s * kMaxExperts], S.lw[(size_t)s * kMaxExperts + 1]};
  int mode = C.mode[r], tok = C.tok[r], mode2 = C.mode[n > 1 ? C.B + r : r];
  int last_mode = 0;
  bool late = false;  // a wait of this wave has ended without its words
  for (int j = 0; j < n; ++j) {
    const size_t row = (size_t)j * C.B + r;
    const bool more = j + 1 < n;
    // the next position's inputs (the one after it for the logits)
    fetch(z3, z0 + min(j + 2, n - 1) * step);
    fetch(g2, g0 + min(j + 1, n - 1) * step);
    const int tok2 = C.tok[more ? row + C.B : row];
    const int mode3 = C.mode[(size_t)min(j + 2, n - 1) * C.B + r];
    // the words of this position
    const uint64_t* words = C.sync + row * ns;
    const bool llm = uses_llm(mode);
    uint64_t part = 0, out = 0;
    for (int spin = 0;; ++spin) {
      part = sync_load(words + min(lane, nseg - 1));
      if (j > 0) out = sync_load(words - (size_t)C.B * ns + nseg);
      const bool wait = (llm && part == kUnset) || out == kUnset;
      if (__builtin_amdgcn_ballot_w64(wait) == 0) break;
      if (late || spin >= C.polls) {
        late = true;
        if (lane == 0) atomicOr(C.bad, KB_EXPIRED);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    auto lo = [](uint64_t x) { return __uint_as_float(uint32_t(x)); };
    auto hi = [](uint64_t x) { return __uint_as_float(uint32_t(x >> 32)); };
    if (j > 0) mixer_step(P, last_mode, lo(out), hi(out), lw);
    RowIn R;
    R.V = V;
    R.K = P.K;
    R.mode = mode;
    R.use_head = P.use_head;
    R.lse = llm ? row_lse(LsePart{lo(part), hi(part)}, nseg, lane) : 0.f;
    R.w[0] = expf(lw[0]);
    R.w[1] = expf(lw[1]);
    float p[4][4], pt[4][4], u[4][4];
    row_probs<false>(R, v, seg, tid, p, pt);
    known_outcome(C, row, seg, tid, mode, tok, p, pt, v.g, C.sync + row * ns + nseg);
    known_bias(P, P.use_head && llm, seg, tid, tok, pt, z2, v.b, u);
    const bool lse2 = more && uses_llm(mode2);
    if (lse2) {
      const LsePart mine = known_lse(u);
      if (lane == 0) s_lse[j & 1][w] = mine;
    }
    __syncthreads();
    if (tid == 0 && lse2)
      sync_store(C.sync + (row + C.B) * ns + seg, sync_word(known_lse_sum(s_lse[j & 1])));
    // the probabilities take the place of the logits, which are in registers two positions on
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (seg_index(seg, q, tid, 0) < uint32_t(V))
        *reinterpret_cast<f4v*>(z0 + j * step + tc[q]) = f4v{p[q][0], p[q][1], p[q][2], p[q][3]};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v.z[q] = z2[q];
      z2[q] = z3[q];
      v.g[q] = g2[q];
    }
    last_mode = mode;
    mode = mode2;
    mode2 = mode3;
    tok = tok2;
  }
  if (seg == 0 && tid < 2) C.lw[((size_t)((n - 1) & 1) * C.B + r) * 2 + tid] = tid ? lw[1] : lw[0];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (seg_index(seg, q, tid, 0) < uint32_t(V)) *reinterpret_cast<f4v*>(b + tc[q]) = v.b[q];
}

// Count partials of every position of the chunk, a workgroup per (segment, position and row).
__global__ __launch_bounds__(kSegThreads) void known_count_kernel(VocabParams P, KnownChunk C) {
  __shared__ KnownSums s_sums[kSegWaves];
  const int seg = blockIdx.x, nseg = gridDim.x, tid = threadIdx.x;
  const size_t row = blockIdx.y;
  if (int(row) / C.B >= C.left[int(row) % C.B]) return;
  const float* z = C.z + row * P.V;
  const int tok = C.tok[row];
  float p[4][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t t0 = seg_index(seg, q, tid, 0);
    const bool in = t0 < uint32_t(P.V);
    const f4v x = *reinterpret_cast<const f4v*>(z + (in ? t0 : 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) p[q][i] = in ? x[i] : 0.f;
  }
  const KnownSums sums = known_counts(P, C, row, seg, tid, tok, p);
  if ((tid & 63) == 0) s_sums[tid >> 6] = sums;
  __syncthreads();
  if (tid == 0) known_store(C, row, seg, nseg, tok, s_sums);
}

// The intervals of the chunk's positions from their count partials, and the mixer weights after
// each row's last position.  A position whose distribution is invalid raises the flag: the caller
// then takes the positions one by one, where the models stop at such a position.
__global__ __launch_bounds__(64) void known_finish_kernel(VocabParams P, StreamState S,
                                                          KnownChunk C, int p0, int nseg) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= C.np * C.B) return;
  const int j = e / C.B, r = e % C.B, s = C.s0 + r;
  const int np = min(C.np, C.left[r]);
  if (j >= np) return;
  const KnownRec o = C.rec[e];
  const uint32_t tok = uint32_t(C.tok[e]), seg = tok / kSeg;
  const SegPartial* parts = static_cast<const SegPartial*>(C.segs) + (size_t)e * nseg;
  const RowQuant q = seg_combine(parts, nseg, seg, P.V, P.total);
  uint32_t cl = q.start + o.before, c = o.c;
  if (q.argmax / kSeg == seg && q.argmax < tok) cl += uint32_t(q.residual);
  if (q.argmax == tok) c += uint32_t(q.residual);
  if (q.status) atomicOr(C.bad, KB_INVALID);
  if (C.iv) {
    const size_t at = (size_t)s * S.maxT + p0 + j;
    C.iv[2 * at] = cl;
    C.iv[2 * at + 1] = cl + c;
    C.ptok[at] = o.p;
  }
  if (j == np - 1) {
    float* out = S.lw + (size_t)s * kMaxExperts;
    const float* src = j > 0 ? C.lw + ((size_t)(j & 1) * C.B + r) * 2 : out;
    float lw[2] = {src[0], src[1]};
    mixer_step(P, o.mode, o.pt, o.png, lw);
    out[0] = lw[0];
    out[1] = lw[1];
  }
}

// ---- reset -----------------------------------------------------------------------------------

__global__ void state_reset_kernel(VocabParams P, StreamState S, int s0, float w_llm) {
  const int s = s0 + blockIdx.x;
  const int V = P.V;
  for (int t = threadIdx.x; t < V; t += blockDim.x) {
    S.b[(size_t)s * V + t] = 0.f;
    S.uni[(size_t)s * V + t] = 0;
  }
  if (threadIdx.x == 0) {
    S.nseen[s] = 0;
    S.ncommit[s] = 0;
    float* lw = S.lw + (size_t)s * kMaxExperts;
    for (int j = 0; j < kMaxExperts; ++j) lw[j] = 0.f;  // ensemble gate: uniform
    if (!P.ensemble) {
      lw[0] = logf(w_llm);
      lw[1] = logf(1.0f - w_llm);
    }
    for (int k = 0; k < kMaxOrder; ++k) S.next_ctx[(size_t)s * kMaxOrder + k] = -1;
    if (S.nctx)  // n-gram tables exist only when the n-gram (or the ensemble) is enabled
      for (int k = 0; k < P.K; ++k) S.nctx[(size_t)s * P.K + k] = 0;
    S.mode[s] = P.ensemble ? M_ENS : M_LLM;
    S.H[s] = 0.f;
    S.pmax[s] = 0.f;
  }
}

// ---- standalone ensemble head (shared b and theta over a batch of rows) --------------------

// w = softmax(theta): every one of the kMaxExperts slots is computed and masked by selects, so that
// w stays in registers; the kept terms are combined in order.
__device__ __forceinline__ void gate_weights(const float* theta, int n, float (&w)[kMaxExperts]) {
  float l[kMaxExperts];
#pragma unroll
  for (int j = 0; j < kMaxExperts; ++j) l[j] = theta[min(j, n - 1)];
  float mx = l[0];
#pragma unroll
  for (int j = 1; j < kMaxExperts; ++j) mx = j < n ? fmaxf(mx, l[j]) : mx;
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < kMaxExperts; ++j) {
    w[j] = expf(l[j] - mx);
    s = j < n ? s + w[j] : s;
  }
#pragma unroll
  for (int j = 0; j < kMaxExperts; ++j) w[j] = w[j] / s;
}

// Four consecutive floats at any 4-byte boundary (a row of odd length starts at one); the hardware
// takes one 16-byte load.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// Logsumexp partials of z_r + b per (segment, row).  Bound by memory (z read once); a thread's
// four consecutive entries go out as one load whatever V is: 7.5 us for 64 rows of 49,152 entries,
// 12.3 us with scalar loads.
__global__ __launch_bounds__(kSegThreads) void ens_lse_kernel(const float* __restrict__ z,
                                                              const float* __restrict__ b, int V,
                                                              LsePart* __restrict__ parts) {
  __shared__ LsePart wl[kSegWaves];
  const int seg = blockIdx.x, r = blockIdx.y, nseg = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const float* zr = z + (size_t)r * V;
  float u[4][4];
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t t0 = seg_index(seg, j, tid, 0);
    if (t0 + 3 < uint32_t(V)) {
      const f4u zz = *reinterpret_cast<const f4u*>(zr + t0);
      const f4u bb = *reinterpret_cast<const f4u*>(b + t0);
#pragma unroll
      for (int i = 0; i < 4; ++i) u[j][i] = zz[i] + bb[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) u[j][i] = t0 + i < uint32_t(V) ? zr[t0 + i] + b[t0 + i] : -INFINITY;
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) m = fmaxf(m, u[j][i]);
  float sum = 0.f;
  if (m != -INFINITY)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) sum += expf(u[j][i] - m);
  LsePart part{m, sum};
  part = wave_lse(part);
  if (lane == 0) wl[w] = part;
  __syncthreads();
  if (tid == 0) {
    LsePart acc = wl[0];
    for (int k = 1; k < kSegWaves; ++k) acc = lse_merge(acc, wl[k]);
    parts[(size_t)r * nseg + seg] = acc;
  }
}

// Per row: lse, loss = -log p(t*), responsibilities r_j = w_j q_j(t*) / p(t*).  A chain of a few
// dependent loads per row, so one wave takes one row (kEnsRows per workgroup) and its lanes fetch
// the row's partials and experts side by side.
constexpr int kEnsRows = 4;
__global__ __launch_bounds__(64 * kEnsRows) void ens_row_kernel(
    const float* __restrict__ z, const float* __restrict__ b, const float* __restrict__ theta,
    const float* __restrict__ Pk, const int32_t* __restrict__ target, int rows, int V, int nexp,
    const LsePart* __restrict__ parts, int nseg, float* __restrict__ lse_out,
    float* __restrict__ loss, float* __restrict__ resp) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * kEnsRows + (threadIdx.x >> 6);
  if (r >= rows) return;  // whole waves
  const int t = target[r];
  // lane 0: the logit and bias of t*; lane j >= 1: expert j's probability of t*
  const float* src = z + (size_t)r * V + t;
  if (lane >= 1 && lane < nexp) src = Pk + ((size_t)r * (nexp - 1) + (lane - 1)) * V + t;
  const float v = *src, bt = b[t];
  float w[kMaxExperts];
  gate_weights(theta, nexp, w);
  const float lse = row_lse(parts[(size_t)r * nseg + min(lane, nseg - 1)], nseg, lane);
  float q[kMaxExperts];
  q[0] = expf(read_lane(v, 0) + bt - lse);
  float p = w[0] * q[0];
#pragma unroll
  for (int j = 1; j < kMaxExperts; ++j) {
    q[j] = read_lane(v, j);
    p = j < nexp ? p + w[j] * q[j] : p;
  }
  if (lane == 0) {
    lse_out[r] = lse;
    if (loss) loss[r] = -logf(p);
  }
#pragma unroll
  for (int j = 0; j < kMaxExperts; ++j)
    if (lane == j && j < nexp) resp[(size_t)r * nexp + j] = w[j] * q[j] / p;
}

// each row's logsumexp from its partials, one wave per row
__global__ __launch_bounds__(64 * kEnsRows) void ens_lse_to_row_kernel(
    const LsePart* __restrict__ parts, int rows, int nseg, float* __restrict__ lse) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * kEnsRows + (threadIdx.x >> 6);
  if (r >= rows) return;
  const float v = row_lse(parts[(size_t)r * nseg + min(lane, nseg - 1)], nseg, lane);
  if (lane == 0) lse[r] = v;
}

// optional full coding distribution p_r
__global__ void ens_prob_kernel(const float* __restrict__ z, const float* __restrict__ b,
                                const float* __restrict__ theta, const float* __restrict__ Pk,
                                int rows, int V, int nexp, const float* __restrict__ lse,
                                float* __restrict__ p) {
  const int r = blockIdx.y;
  float w[kMaxExperts];
  gate_weights(theta, nexp, w);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < V; t += gridDim.x * blockDim.x) {
    float v = w[0] * expf(z[(size_t)r * V + t] + b[t] - lse[r]);
#pragma unroll
    for (int j = 1; j < kMaxExperts; ++j)
      if (j < nexp) v = v + w[j] * Pk[((size_t)r * (nexp - 1) + (j - 1)) * V + t];
    p[(size_t)r * V + t] = v;
  }
}

// Backward of the head over all rows, in one launch.
//   Workgroups 0 .. gridDim.x - 2, 64 vocabulary entries each, one per lane:
//     grad_b[t] = sum_r g_r r_{r,0} (q0_r(t) - 1[t = t*_r]); SGD on b.  Wave w sums the rows of
//     blocks w, w + 4, ... (kGradRows rows each) in order, then the four sums are added in order.
//     Bound by reading z once: a block's loads are in flight together and the waves' side by side,
//     so 64 rows take one memory round trip.
//   The last workgroup: grad_theta[j] = sum_r g_r (w_j - r_{r,j}), each thread over its rows, then
//     a fixed tree; SGD on theta (nothing else in the launch reads theta).
// 64 rows of 49,152 entries and 5 experts: 5.4 us.  One thread per entry walking all rows took 16.4
// us, and a launch of its own whose one thread walked the rows for theta 30.8 us.
constexpr int kGradWaves = 4, kGradThreads = 64 * kGradWaves, kGradRows = 16;
__global__ __launch_bounds__(kGradThreads) void ens_grad_kernel(
    const float* __restrict__ z, float* __restrict__ b, float* __restrict__ theta,
    const float* __restrict__ resp, const int32_t* __restrict__ target,
    const float* __restrict__ gl, int rows, int V, int nexp, const float* __restrict__ lse,
    float lr, float* __restrict__ gb, float* __restrict__ gth) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ float s_part[kGradWaves][kMaxExperts];
    float w[kMaxExperts], g[kMaxExperts];
    gate_weights(theta, nexp, w);
#pragma unroll
    for (int j = 0; j < kMaxExperts; ++j) g[j] = 0.f;
    for (int r = tid; r < rows; r += kGradThreads) {
      const float f = gl ? gl[r] : 1.f;
#pragma unroll
      for (int j = 0; j < kMaxExperts; ++j)
        if (j < nexp) g[j] = g[j] + f * (w[j] - resp[(size_t)r * nexp + j]);
    }
#pragma unroll
    for (int j = 0; j < kMaxExperts; ++j) {
      g[j] = wave_sum_f(g[j]);
      if (lane == 0) s_part[wave][j] = g[j];
    }
    __syncthreads();
    if (tid < nexp) {
      float v = s_part[0][tid];
      for (int k = 1; k < kGradWaves; ++k) v = v + s_part[k][tid];
      if (gth) gth[tid] = v;
      if (lr != 0.f) theta[tid] = theta[tid] - lr * v;
    }
    return;
  }
  __shared__ float s_g[kGradWaves][64];
  const int t = blockIdx.x * 64 + lane;
  const int tc = min(t, V - 1);
  const float bt = b[tc];
  float g = 0.f;
  for (int r0 = wave * kGradRows; r0 < rows; r0 += kGradWaves * kGradRows) {
    // lane u (mod kGradRows) holds row u's factors; rows past the end repeat the last one, unused
    const int ru = min(r0 + (lane & (kGradRows - 1)), rows - 1);
    float x[kGradRows];
#pragma unroll
    for (int u = 0; u < kGradRows; ++u) x[u] = z[(size_t)min(r0 + u, rows - 1) * V + tc];
    const float l = lse[ru], f = (gl ? gl[ru] : 1.f) * resp[(size_t)ru * nexp];
    const int tt = target[ru];
#pragma unroll
    for (int u = 0; u < kGradRows; ++u) {
      const float q0 = expf(x[u] + bt - read_lane(l, u));
      const float ind = __builtin_amdgcn_readlane(tt, u) == t ? 1.f : 0.f;
      const float d = read_lane(f, u) * (q0 - ind);
      g = r0 + u < rows ? g + d : g;
    }
  }
  s_g[wave][lane] = g;
  __syncthreads();
  if (wave == 0 && t < V) {
    for (int k = 1; k < kGradWaves; ++k) g = g + s_g[k][lane];
    if (gb) gb[t] = g;
    if (lr != 0.f) b[t] = bt - lr * g;
  }
}

size_t ensemble_workspace_bytes(int rows, int V) {
  return size_t(rows) * (ceil_div(V, kSeg) * sizeof(LsePart) + sizeof(float)) + 256;
}

void launch_ensemble_forward(const float* z, const float* b, const float* theta, const float* Pk,
                             const int32_t* target, int rows, int V, int nexp, float* loss,
                             float* p, float* resp, float* lse_out, void* ws, hipStream_t s) {
  if (rows <= 0) return;
  const int nseg = int(ceil_div(V, kSeg));
  LsePart* parts = static_cast<LsePart*>(ws);
  float* lse = lse_out ? lse_out : reinterpret_cast<float*>(parts + (size_t)rows * nseg);
  hipLaunchKernelGGL(ens_lse_kernel, dim3(nseg, rows), dim3(kSegThreads), 0, s, z, b, V, parts);
  hipLaunchKernelGGL(ens_row_kernel, dim3(ceil_div(rows, kEnsRows)), dim3(64 * kEnsRows), 0, s, z,
                     b, theta, Pk, target, rows, V, nexp, parts, nseg, lse, loss, resp);
  if (p)
    hipLaunchKernelGGL(ens_prob_kernel, dim3(ceil_div(V, 256), rows), dim3(256), 0, s, z, b,
                       theta, Pk, rows, V, nexp, lse, p);
  NC_HIP(hipGetLastError());
}

void launch_ensemble_backward(const float* z, float* b, float* theta, const float* resp,
                              const int32_t* target, const float* gl, int rows, int V, int nexp,
                              float lr, float* gb, float* gth, const float* lse_in, void* ws,
                              hipStream_t s) {
  if (rows <= 0) return;
  const float* lse = lse_in;
  if (!lse) {  // each row's lse, the forward's bits, recomputed
    const int nseg = int(ceil_div(V, kSeg));
    LsePart* parts = static_cast<LsePart*>(ws);
    float* out = reinterpret_cast<float*>(parts + (size_t)rows * nseg);
    hipLaunchKernelGGL(ens_lse_kernel, dim3(nseg, rows), dim3(kSegThreads), 0, s, z, b, V, parts);
    hipLaunchKernelGGL(ens_lse_to_row_kernel, dim3(ceil_div(rows, kEnsRows)), dim3(64 * kEnsRows),
                       0, s, parts, rows, nseg, out);
    lse = out;
  }
  hipLaunchKernelGGL(ens_grad_kernel, dim3(ceil_div(V, 64) + 1), dim3(kGradThreads), 0, s, z,
                     b, theta, resp, target, gl, rows, V, nexp, lse, lr, gb, gth);
  NC_HIP(hipGetLastError());
}

// ---- launchers ------------------------------------------------------------------------------

void launch_vocab_step(const VocabParams& P, const StreamState& S, const StepArgs& A,
                       hipStream_t s) {
  if (A.B <= 0) return;
  const int nseg = int(ceil_div(P.V, kSeg));
  const dim3 grid(nseg, A.B);
  if (A.lse) hipLaunchKernelGGL(vocab_lse_kernel, grid, dim3(kSegThreads), 0, s, P, S, A);
  hipLaunchKernelGGL(vocab_count_kernel, grid, dim3(kSegThreads), 0, s, P, S, A);
  hipLaunchKernelGGL(vocab_scan_kernel, grid, dim3(kSegThreads), 0, s, P, S, A);
  if (!A.no_update && P.ensemble)
    hipLaunchKernelGGL(ensemble_bias_kernel, grid, dim3(kSegThreads), 0, s, P, S, A);
  if (!A.no_update)
    hipLaunchKernelGGL(ngram_update_kernel, dim3(A.B), dim3(64), 0, s, P, S, A);
  NC_HIP(hipGetLastError());
}

void launch_ngram_predict(const VocabParams& P, const StreamState& S, const int32_t* rows, int B,
                          NgPart* parts, StepOut* step_out, const Outcome* out, hipStream_t s) {
  if (B <= 0) return;
  const int nseg = int(ceil_div(P.V, kSeg));
  hipLaunchKernelGGL(ngram_dense_kernel, dim3(nseg, B), dim3(kSegThreads), 0, s, P, S, rows,
                     parts);
  hipLaunchKernelGGL(ngram_fix_kernel, dim3(B), dim3(256), 0, s, P, S, rows, parts, nseg,
                     step_out, out);
  NC_HIP(hipGetLastError());
}

void launch_known_ngram(const VocabParams& P, const StreamState& S, const KnownChunk& C, int p0,
                        hipStream_t s) {
  if (C.B <= 0 || C.np <= 0) return;
  const int nseg = int(ceil_div(P.V, kSeg));
  if (P.use_ngram) {
    hipLaunchKernelGGL(known_advance_kernel, dim3(P.K, C.B), dim3(64), 0, s, P, S, C, p0);
    hipLaunchKernelGGL(known_dense_kernel, dim3(nseg, ceil_div(C.np, kKnownRun), C.B),
                       dim3(kSegThreads), 0, s, P, S, C, p0);
    hipLaunchKernelGGL(known_fix_kernel, dim3(C.np, C.B), dim3(kSegThreads),
                       C.np * sizeof(int32_t), s, P, S, C, p0, nseg);
  } else {
    hipLaunchKernelGGL(known_tokens_kernel, dim3(ceil_div(C.np * C.B, 256)), dim3(256), 0, s, S, C,
                       p0);
  }
  hipLaunchKernelGGL(known_commit_kernel, dim3(C.B), dim3(kSegThreads), 0, s, P, S, C, p0);
  NC_HIP(hipGetLastError());
}

bool known_in_one_launch(int B, int V) { return B * ceil_div(V, kSeg) <= kRunGroups; }

void launch_known_steps(const VocabParams& P, const StreamState& S, const KnownChunk& C,
                        hipStream_t s) {
  if (C.B <= 0 || C.np <= 0) return;
  const dim3 grid(ceil_div(P.V, kSeg), C.B);
  hipLaunchKernelGGL(known_first_kernel, grid, dim3(kSegThreads), 0, s, P, S, C);
  if (C.sync) {
    hipLaunchKernelGGL(known_run_kernel, grid, dim3(kSegThreads), 0, s, P, S, C);
    hipLaunchKernelGGL(known_count_kernel, dim3(grid.x, C.np * C.B), dim3(kSegThreads), 0, s, P, C);
    NC_HIP(hipGetLastError());
    return;
  }
  for (int j = 0; j < C.np; ++j)
    hipLaunchKernelGGL(known_step_kernel, grid, dim3(kSegThreads), 0, s, P, S, C, j);
  NC_HIP(hipGetLastError());
}

void launch_known_finish(const VocabParams& P, const StreamState& S, const KnownChunk& C, int p0,
                         hipStream_t s) {
  if (C.B <= 0 || C.np <= 0) return;
  hipLaunchKernelGGL(known_finish_kernel, dim3(ceil_div(C.np * C.B, 64)), dim3(64), 0, s, P, S, C,
                     p0, int(ceil_div(P.V, kSeg)));
  NC_HIP(hipGetLastError());
}

void launch_state_reset(const VocabParams& P, const StreamState& S, int s0, int n_streams,
                        float w_llm, hipStream_t s) {
  if (n_streams <= 0) return;
  hipLaunchKernelGGL(state_reset_kernel, dim3(n_streams), dim3(256), 0, s, P, S, s0, w_llm);
  NC_HIP(hipGetLastError());
}

}  // namespace nc
