// Transformer kernels of the 135M-shape decoder (paper section 3.2 Eq. (lm), section 3.10):
// MFMA GEMMs with a fused RMSNorm prologue and fused epilogues (RoPE + KV-ring write, residual
// add, SiLU-gated MLP, logits), GQA attention over the sliding window, embedding gather and
// precision conversion.
//
// Batch invariance.  Every output element of a GEMM is the sum over K in chunks of 32 taken in
// increasing order, each chunk by the same MFMA instruction (f32 16x16x4, bf16 16x16x32, fp8
// 16x16x32), whatever the tile shape or the number of rows M.  Attention splits the keys into
// 64-key chunks at fixed absolute positions and combines the chunk partials with one fixed
// two-level fold.  A token's logits are therefore bitwise the same whether it is evaluated in a
// 32,768-row prefill or in a one-row decode step, which the coder relies on.
#include "cdf_dev.hpp"
#include "common.hpp"
#include "llm_dev.hpp"

#include <algorithm>
#include <type_traits>

// Prefill and decode must round every shared expression identically: no contraction.
#pragma clang fp contract(off)

namespace nc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

// ---- number formats ------------------------------------------------------------------------

__device__ __forceinline__ uint16_t f2bf(float f) {  // round to nearest even (finite inputs)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}

// float -> OCP fp8 e4m3 (bias 7, max 448, no infinity), round to nearest even, saturating.
__device__ __forceinline__ uint8_t f2fp8(float f) {
  const uint32_t b = __float_as_uint(f);
  const uint32_t sign = (b >> 24) & 0x80u;
  const uint32_t u = b & 0x7FFFFFFFu;
  uint32_t r;
  if (u >= 0x43E00000u) {           // |f| >= 448
    r = 0x7Eu;
  } else if (u < 0x3C800000u) {     // |f| < 2^-6: subnormal grid of 2^-9
    r = uint32_t(rintf(__uint_as_float(u) * 512.0f));
  } else {
    const uint32_t ue = u - (120u << 23);  // rebias 127 -> 7
    r = (ue + 0x7FFFFu + ((ue >> 20) & 1u)) >> 20;
    if (r > 0x7Eu) r = 0x7Eu;
  }
  return uint8_t(r | sign);
}

template <int P>
struct PT;
template <>
struct PT<P_F32> {
  static constexpr int ES = 4;
  __device__ static void store(void* base, long long i, float v, float) {
    static_cast<float*>(base)[i] = v;
  }
};
template <>
struct PT<P_BF16> {
  static constexpr int ES = 2;
  __device__ static void store(void* base, long long i, float v, float) {
    static_cast<uint16_t*>(base)[i] = f2bf(v);
  }
};
template <>
struct PT<P_FP8> {
  static constexpr int ES = 1;
  __device__ static void store(void* base, long long i, float v, float inv_scale) {
    static_cast<uint8_t*>(base)[i] = f2fp8(v * inv_scale);
  }
};

__device__ __forceinline__ void atomic_max_abs(float* p, float v) {
  // |v| >= 0, so the IEEE bit pattern orders like an unsigned integer: integer atomic max
  atomicMax(reinterpret_cast<unsigned int*>(p), __float_as_uint(fabsf(v)));
}

// ---- GEMM -----------------------------------------------------------------------------------
//
// Arithmetic of every output element (the same in every kernel and tile shape):
//   out = ((0 + P_0) + P_1) + ... + P_{S-1},  S = ceil(K / 64),
//   P_s = the chain of MFMAs over the 64 K entries of part s, starting from zero, where
//     f32 16x16x4:            16 steps, step t / lane group g consumes k = 16 g + t,
//     bf16 / fp8 16x16x32:     2 steps, step t / lane group g consumes k = 32 t + 8 g .. + 7,
//   with entries beyond K read as zero.
// A normed GEMM (A_NORM) then multiplies by deq (FP8) and by the row's RMSNorm scale, in that
// order.  The tile kernels (many rows) sum the parts as they walk K; the split kernel (few rows)
// computes each part in its own wave and the workgroup adds the parts in order.  All apply the
// same epilogue functions, so a row's outputs do not depend on how many rows are in the launch.

constexpr int KP = 64;

// RMSNorm scale of a row, 1 / sqrt(mean(x^2) + eps), from block sums of squares.  Whatever writes
// a residual row x (embedding, residual epilogues) also writes, for each 16-column block b,
// ssq[b] = sum of x^2 over the block by one fixed tree (block_ssq16); the scale adds the block
// sums in block order.  Prefill and decode kernels therefore derive bitwise equal scales.

// Block sum of squares of 16 values held by 16 consecutive lanes (lane % 16 = column); every lane
// of the group returns the same bits: the tree of partners c ^ 8, c ^ 4, c ^ 2, c ^ 1 (after each
// step the values repeat with half the period, so rotating by 8, 4, 2, 1 fetches the partner's).
__device__ __forceinline__ float block_ssq16(float x) {
  float v = x * x;
  v += dpp_f<kRor + 8>(v);
  v += dpp_f<kRor + 4>(v);
  v += dpp_f<kRor + 2>(v);
  v += dpp_f<kRor + 1>(v);
  return v;
}

__device__ __forceinline__ float inv_from_ssq(const float* ssq, int K, float eps) {
  const int nb = K / 16;
  float t = 0.f;
  int b = 0;
  if (nb % 4 == 0) {
    // (rows of 16-byte multiples: 48 blocks' sums requested together)
    const v4f* q = reinterpret_cast<const v4f*>(ssq);
    for (; b < nb; b += 48) {
      v4f v[12];
#pragma unroll
      for (int u = 0; u < 12; ++u) v[u] = q[min(b / 4 + u, nb / 4 - 1)];
#pragma unroll
      for (int u = 0; u < 12; ++u) {
        const bool in = b + 4 * u < nb;
#pragma unroll
        for (int e = 0; e < 4; ++e) t = in ? t + v[u][e] : t;
      }
    }
  }
  for (; b < nb; ++b) t += ssq[b];
  return 1.0f / sqrtf(t / float(K) + eps);
}

// the scale of A row ar of a normed GEMM
__device__ __forceinline__ float a_row_inv(const GemmArgs& a, int ar) {
  return a.inv ? a.inv[ar] : inv_from_ssq(a.ssq + (long long)ar * (a.K / 16), a.K, a.eps);
}

// ---- epilogue emitters ----

// q/k/v output (m, n) = v (partner: the RoPE partner column's value) with the row's metadata rm
// and, for q/k columns, its RoPE entry cs (cos, sin)
__device__ __forceinline__ void emit_qkv_core(const GemmArgs& a, int prec_att, int m, int n,
                                              float v, float partner, const RowMeta& rm,
                                              float2 cs) {
  const int hd = a.hd, h2 = hd / 2;
  const int nq = a.Hq * hd, nk = a.Hk * hd;
  const int within = n % hd;
  if (n < nq + nk)  // rotate-half RoPE on q and k
    v = within < h2 ? v * cs.x - partner * cs.y : v * cs.x + partner * cs.y;
  long long idx;
  void* base;
  if (n < nq) {
    idx = (long long)m * nq + n;
    base = a.q_out;
  } else {
    const int kv = n < nq + nk ? n - nq : n - nq - nk;
    const int kvh = kv / hd;
    const long long slot = rm.slot;
    const long long sb = (long long)rm.stream * a.kv_stride + (long long)kvh * a.ring * hd;
    if (n < nq + nk) {
      idx = sb + slot * hd + within;
      base = a.k_cache;
    } else {
      idx = sb + (long long)within * a.ring + slot;
      base = a.vt_cache;
    }
  }
  if (prec_att == P_F32)
    PT<P_F32>::store(base, idx, v, 1.f);
  else
    PT<P_BF16>::store(base, idx, v, 1.f);
}

// emit_qkv_core for rows m .. m + 3 of one column (BF16 attention operands), element for element
// the same arithmetic, with the rows' metadata rm and RoPE table rows rr (cos, sin pairs of
// position rm[e].pos, in global memory or LDS) supplied by the caller; V^T gets one 8-byte store
// when the rows are 4 consecutive ring slots of one stream.
__device__ __forceinline__ void emit_qkv4_rows(const GemmArgs& a, int n, const RowMeta (&rm)[4],
                                               const bool (&ok)[4], const float* const (&rr)[4],
                                               const float (&v)[4], const float (&partner)[4],
                                               int m) {
  const int hd = a.hd, h2 = hd / 2;
  const int nq = a.Hq * hd, nk = a.Hk * hd;
  const int within = n % hd;
  uint16_t h[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = v[e];
    if (n < nq + nk && ok[e]) {
      const int i = within < h2 ? within : within - h2;
      const float cs = rr[e][i * 2 + 0];
      const float sn = rr[e][i * 2 + 1];
      x = within < h2 ? x * cs - partner[e] * sn : x * cs + partner[e] * sn;
    }
    h[e] = f2bf(x);
  }
  if (n < nq) {
    uint16_t* Q = static_cast<uint16_t*>(a.q_out);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (ok[e]) Q[(long long)(m + e) * nq + n] = h[e];
    return;
  }
  const int kv = n < nq + nk ? n - nq : n - nq - nk;
  const int kvh = kv / hd;
  if (n < nq + nk) {
    uint16_t* Kc = static_cast<uint16_t*>(a.k_cache);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (ok[e]) {
        const long long sb = (long long)rm[e].stream * a.kv_stride + (long long)kvh * a.ring * hd;
        Kc[sb + (long long)rm[e].slot * hd + within] = h[e];
      }
    return;
  }
  uint16_t* Vt = static_cast<uint16_t*>(a.vt_cache);
  const int slot0 = rm[0].slot;
  bool run = ok[3] && (slot0 & 3) == 0 && slot0 + 3 < a.ring;
#pragma unroll
  for (int e = 1; e < 4; ++e)
    run = run && rm[e].stream == rm[0].stream && rm[e].pos == rm[0].pos + e;
  if (run) {
    const long long sb = (long long)rm[0].stream * a.kv_stride + (long long)kvh * a.ring * hd;
    uint2 w;
    w.x = uint32_t(h[0]) | (uint32_t(h[1]) << 16);
    w.y = uint32_t(h[2]) | (uint32_t(h[3]) << 16);
    *reinterpret_cast<uint2*>(Vt + sb + (long long)within * a.ring + slot0) = w;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (ok[e]) {
      const long long sb = (long long)rm[e].stream * a.kv_stride + (long long)kvh * a.ring * hd;
      Vt[sb + (long long)within * a.ring + rm[e].slot] = h[e];
    }
}

template <int P>
__device__ __forceinline__ float emit_glu(const GemmArgs& a, int m, int col, float g, float u) {
  const float h = g / (1.0f + expf(-g)) * u;
  const float oinv = (P == P_FP8) ? 1.0f / a.out_scale : 1.0f;
  PT<P>::store(a.out_p, (long long)m * (a.N / 2) + col, h, oinv);
  return fabsf(h);
}

// ---- operand fragments (from LDS or global, row-major with K contiguous) ----

template <int P>
struct Frag;
template <>
struct Frag<P_F32> {
  typedef float T[16];  // 16 steps of one float
  __device__ static void load(T& f, const uint8_t* row, int g) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const v4f v = *reinterpret_cast<const v4f*>(row + (16 * g + 4 * q) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) f[4 * q + e] = v[e];
    }
  }
  // straight from a global row: entries k0 + 16 g + 0..15, zero at or beyond K.  The load itself is
  // unconditional (its offset clamped into the row), so that no branch separates it from the loads
  // issued around it
  __device__ static void load_clamped(T& f, const uint8_t* row, int k0, int K, int g) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + 16 * g + 4 * q;
      const v4f v = *reinterpret_cast<const v4f*>(row + (long long)min(k, K - 4) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) f[4 * q + e] = k < K ? v[e] : 0.f;
    }
  }
  static constexpr int STEPS = 16;
  __device__ static void step(v4f& acc, const T& a, const T& b, int t) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[t], acc, 0, 0, 0);
  }
  __device__ static void mma(v4f& acc, const T& a, const T& b) {
#pragma unroll
    for (int t = 0; t < STEPS; ++t) step(acc, a, b, t);
  }
};
template <>
struct Frag<P_BF16> {
  typedef v4i T[2];
  __device__ static void load(T& f, const uint8_t* row, int g) {
#pragma unroll
    for (int t = 0; t < 2; ++t) f[t] = *reinterpret_cast<const v4i*>(row + (32 * t + 8 * g) * 2);
  }
  __device__ static void load_clamped(T& f, const uint8_t* row, int k0, int K, int g) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int k = k0 + 32 * t + 8 * g;
      const v4i v = *reinterpret_cast<const v4i*>(row + (long long)min(k, K - 8) * 2);
      f[t] = k < K ? v : v4i{0, 0, 0, 0};
    }
  }
  static constexpr int STEPS = 2;
  __device__ static void step(v4f& acc, const T& a, const T& b, int t) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a[t]),
                                                  __builtin_bit_cast(v8bf, b[t]), acc, 0, 0, 0);
  }
  __device__ static void mma(v4f& acc, const T& a, const T& b) {
#pragma unroll
    for (int t = 0; t < STEPS; ++t) step(acc, a, b, t);
  }
};
template <>
struct Frag<P_FP8> {
  typedef long T[2];
  __device__ static void load(T& f, const uint8_t* row, int g) {
#pragma unroll
    for (int t = 0; t < 2; ++t) f[t] = *reinterpret_cast<const long*>(row + 32 * t + 8 * g);
  }
  __device__ static void load_clamped(T& f, const uint8_t* row, int k0, int K, int g) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int k = k0 + 32 * t + 8 * g;
      const long v = *reinterpret_cast<const long*>(row + min(k, K - 8));
      f[t] = k < K ? v : 0;
    }
  }
  static constexpr int STEPS = 2;
  __device__ static void step(v4f& acc, const T& a, const T& b, int t) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a[t], b[t], acc, 0, 0, 0);
  }
  __device__ static void mma(v4f& acc, const T& a, const T& b) {
#pragma unroll
    for (int t = 0; t < STEPS; ++t) step(acc, a, b, t);
  }
};

// Residual epilogue of element (m, n) after x[m][n] was updated to xn: the block sum of squares of
// row m over the 16-column block of n (held by the 16 lanes with lane % 16 = column), and the
// next normed GEMM's operand quantise(xn * y_gain[n]).  Every lane of the wave must call this;
// lanes with ok == false pass xn = 0 and store nothing.  Returns |xn * y_gain[n]|.
template <int P>
__device__ __forceinline__ float resid_out(const GemmArgs& a, int m, int n, float xn, int c,
                                             bool ok, float gain) {
  const float sq = block_ssq16(xn);
  if (!ok) return 0.f;
  if (a.ssq_out && c == 0) a.ssq_out[(long long)m * (a.N / 16) + n / 16] = sq;
  if (!a.y_out) return 0.f;
  const float yv = xn * gain;
  PT<P>::store(a.y_out, (long long)m * a.N + n, yv, a.y_inv_scale);
  return fabsf(yv);
}
__device__ __forceinline__ void amax_flush(float* dst, float v, int lane) {
  if (!dst) return;
  v = wave_max_f(v);
  if (lane == 0) atomic_max_abs(dst, v);
}

// Column blocks of an epilogue group: a RoPE pair {b, b + hd/32} for QKV (a single block when hd =
// 16), a gate/up block pair for the SiLU-gated MLP, two adjacent blocks otherwise.
__host__ __device__ __forceinline__ int group_block(int epi, int hd, int gi, int j) {
  if (epi == E_QKV && hd > 16) {
    const int nb = hd / 16, half = nb / 2;  // blocks per head
    return (gi / half) * nb + gi % half + j * half;
  }
  return 2 * gi + j;
}

// ---- tile kernel (many rows) ----
//
// WVM x WVN waves, each RB x CB blocks of 16 x 16 outputs; the workgroup's operand rows of one
// 64-wide K part are staged in LDS.  Parts go global -> registers -> LDS ahead of their MFMAs:
// while part s is multiplied, the loads of the parts after it are in flight, with one barrier per
// part.  Tiles are ordered so that the
// workgroups of one XCD (dispatch is round-robin over the 8 XCDs) take consecutive tiles of the
// same A rows, which then stay in that XCD's L2 while every column tile reads them.  A tile's
// column blocks are taken in epilogue groups (group_block), so a wave holds both halves of a RoPE
// pair, and both of a gate/up pair, in one lane.
//
// Every residual value and gain of a lane is loaded before its first store, so the loads overlap
// instead of each waiting behind the previous output's store.
template <int P, int AM, int EPI, int RB, int CB, int WVM, int WVN, bool kDeep>
__global__ __launch_bounds__(64 * WVM * WVN, 2) void gemm_tile_kernel(
    const GemmArgs a, int tiles_m, int tiles_n) {
  constexpr int NT = 64 * WVM * WVN;
  constexpr int BM = 16 * RB * WVM, BN = 16 * CB * WVN;
  constexpr int ES = PT<P>::ES;
  constexpr int ROWB = KP * ES + 16;  // padded LDS row (bytes)
  constexpr int TILEB = (BM + BN) * ROWB;
  constexpr int CPR = KP * ES / 16;                          // 16-byte chunks per staged row
  constexpr int NCH = ((BM + BN) * CPR + NT - 1) / NT;       // chunks per thread
  constexpr bool kEven = (BM + BN) * CPR % NT == 0;
  static_assert(CB % 2 == 0 || EPI == E_RESID || EPI == E_STORE, "column groups are block pairs");
  // (QKV: the epilogue keeps the tile rows' metadata and RoPE entries there)
  constexpr int QKVB = EPI == E_QKV ? BM * int(sizeof(RowMeta) + 32 * 8) : 0;
  __shared__ __align__(16) uint8_t lds[2 * TILEB > QKVB ? 2 * TILEB : QKVB];
  __shared__ float s_inv[BM];
  __shared__ int s_arow[BM];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WVN, wn = wave % WVN;
  const int fr = lane & 15, fg = lane >> 4;
  const int K = a.K, S = (K + KP - 1) / KP;
  const int hd = EPI == E_QKV ? a.hd : 64;

  // XCD-aware tile order (a bijection of [0, tiles)): XCD x owns a contiguous range of tiles
  const int nt = tiles_m * tiles_n, q8 = nt / 8, r8 = nt % 8;
  const int bx = blockIdx.x, xcd = bx % 8;
  const int t = xcd * q8 + min(xcd, r8) + bx / 8;
  const int m0 = (t / tiles_n) * BM, cb0 = (t % tiles_n) * (BN / 16);
  // first column of the tile's block j
  auto col0 = [&](int j) {
    const int jb = cb0 + j;
    return 16 * (EPI == E_QKV ? group_block(EPI, hd, jb >> 1, jb & 1) : jb);
  };

  // rows past M repeat row M - 1 and columns past N column N - 1 (never stored)
  for (int r = tid; r < BM; r += NT) {
    const int m = min(m0 + r, a.M - 1);
    s_arow[r] = a.a_rows ? a.a_rows[m] : m;
  }
  __syncthreads();
  for (int r = tid; r < BM; r += NT) s_inv[r] = AM == A_NORM ? a_row_inv(a, s_arow[r]) : 1.f;

  // global -> register staging of one K part; each thread's row addresses are resolved once.  The
  // loads of a part are the same number on every path, and parts past the last repeat it: a load
  // under a branch of its own would make the number in flight path-dependent, and the wait for one
  // part would drain the parts behind it.  (Only a part that K ends in clamps its loads into the
  // rows and zeroes the entries beyond K: a wave that has its SIMD to itself pays for every
  // instruction between its MFMAs.)
  constexpr int NBUF = kDeep ? 2 : 1;
  constexpr int CE = 16 / ES;  // entries per chunk
  v4i rg[NBUF][NCH];
  const uint8_t* src[NCH];
  int dst[NCH];
#pragma unroll
  for (int u = 0; u < NCH; ++u) {
    const int c = min(tid + u * NT, (BM + BN) * CPR - 1), r = c / CPR, k = (c % CPR) * CE;
    dst[u] = r * ROWB + (c % CPR) * 16;
    if (r < BM) {
      src[u] = static_cast<const uint8_t*>(a.A) + ((long long)s_arow[r] * K + k) * ES;
    } else {
      const int rr = r - BM, n = min(col0(rr / 16) + rr % 16, a.N - 1);
      src[u] = static_cast<const uint8_t*>(a.W) + ((long long)n * K + k) * ES;
    }
  }
  // entries of chunk u's row from its own first on (its position in the row is implied by dst)
  auto room = [&](int u) { return K - ((min(tid + u * NT, (BM + BN) * CPR - 1)) % CPR) * CE; };
  auto fetch = [&](int q, int s) {
    const int k0 = min(s, S - 1) * KP;
    if (k0 + KP <= K) {
#pragma unroll
      for (int u = 0; u < NCH; ++u)
        rg[q][u] = *reinterpret_cast<const v4i*>(src[u] + (long long)k0 * ES);
    } else {
#pragma unroll
      for (int u = 0; u < NCH; ++u)
        rg[q][u] = *reinterpret_cast<const v4i*>(src[u] + (long long)min(k0, room(u) - CE) * ES);
    }
    // parts' loads stay in order, so that waiting for one leaves the later ones in flight
    __builtin_amdgcn_sched_barrier(0);
  };
  auto stage = [&](int q, int s, uint8_t* buf) {
    const int k0 = min(s, S - 1) * KP;
    __builtin_amdgcn_sched_barrier(0);  // no wait for these loads before the MFMAs
    if (k0 + KP > K) {
#pragma unroll
      for (int u = 0; u < NCH; ++u)
        if (k0 >= room(u)) rg[q][u] = v4i{0, 0, 0, 0};
    }
#pragma unroll
    for (int u = 0; u < NCH; ++u)
      if (kEven || tid + u * NT < (BM + BN) * CPR) *reinterpret_cast<v4i*>(buf + dst[u]) = rg[q][u];
  };

  v4f tot[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) tot[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  const int ra = (wm * RB * 16 + fr) * ROWB, rb = (BM + wn * CB * 16 + fr) * ROWB;
  fetch(0, 0);
  if constexpr (kDeep) {
    // Few tiles (a wave has its SIMD to itself): nothing else hides a wave's own waits.  Two parts'
    // loads are in flight, and with kAhead (BF16 / FP8) the fragments of part s + 1 are read while
    // part s is multiplied, part s + 2 then written to the buffer whose fragments are all in
    // registers.  (FP32's fragments are four times as large and its MFMAs four times as long: there
    // it gains 3% at 512 rows and loses 12% at 16,384.)
    constexpr bool kAhead = P != P_F32;
    typename Frag<P>::T fa[2][RB], fb[2][CB];
    auto frags = [&](int q, const uint8_t* buf) {
#pragma unroll
      for (int j = 0; j < CB; ++j) Frag<P>::load(fb[q][j], buf + rb + j * 16 * ROWB, fg);
#pragma unroll
      for (int i = 0; i < RB; ++i) Frag<P>::load(fa[q][i], buf + ra + i * 16 * ROWB, fg);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int q) {
      v4f acc[RB][CB];
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < Frag<P>::STEPS; ++t)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < CB; ++j) Frag<P>::step(acc[i][j], fa[q][i], fb[q][j], t);
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) tot[i][j] += acc[i][j];
    };
    // (two parts an iteration and no exit between them, so that the loads in flight are the same
    // on every path)
    fetch(1, 1);
    stage(0, 0, lds);
    if constexpr (kAhead) {
      stage(1, 1, lds + TILEB);
      __syncthreads();
      frags(0, lds);
      __syncthreads();
      fetch(0, 2);
      fetch(1, 3);
      // register set s % 2 holds part s + 2, and fragment set s % 2 part s
      for (int s = 0; s + 1 < S; s += 2) {
        frags(1, lds + TILEB);
        multiply(0);
        stage(0, s + 2, lds);
        fetch(0, s + 4);
        __syncthreads();
        frags(0, lds);
        multiply(1);
        stage(1, s + 3, lds + TILEB);
        fetch(1, s + 5);
        __syncthreads();
      }
      if (S & 1) multiply(0);
    } else {
      __syncthreads();
      fetch(0, 2);
      // register set (s + 1) % 2 holds part s + 1
      for (int s = 0; s + 1 < S; s += 2) {
        frags(0, lds);
        multiply(0);
        stage(1, s + 1, lds + TILEB);
        fetch(1, s + 3);
        __syncthreads();
        frags(0, lds + TILEB);
        multiply(0);
        stage(0, s + 2, lds);
        fetch(0, s + 4);
        __syncthreads();
      }
      if (S & 1) {
        frags(0, lds);
        multiply(0);
      }
    }
    __syncthreads();
  } else {
    stage(0, 0, lds);
    __syncthreads();
    for (int s = 0; s < S; ++s) {
      fetch(0, s + 1);
      const uint8_t* buf = lds + (s & 1) * TILEB;
      typename Frag<P>::T bf[CB];
#pragma unroll
      for (int j = 0; j < CB; ++j) Frag<P>::load(bf[j], buf + rb + j * 16 * ROWB, fg);
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        typename Frag<P>::T af;
        Frag<P>::load(af, buf + ra + i * 16 * ROWB, fg);
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          v4f acc = {0.f, 0.f, 0.f, 0.f};
          Frag<P>::mma(acc, af, bf[j]);
          tot[i][j] += acc;
        }
      }
      stage(0, s + 1, lds + ((s + 1) & 1) * TILEB);
      __syncthreads();
    }
  }

  const float deq = (P == P_FP8) ? a.a_scale * a.w_scale : 1.0f;
  const int rw = wm * RB * 16, jw = wn * CB;  // the wave's first tile row and column block
  // output value of accumulator (i, j, e): (sum of parts) * deq * row scale
  auto val = [&](int i, int j, int e) { return tot[i][j][e] * deq * s_inv[rw + i * 16 + fg * 4 + e]; };
  if constexpr (EPI == E_RESID) {
    float xo[RB][CB][4], gn[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const int n = col0(jw + j) + fr;
      gn[j] = (a.y_out && n < a.N) ? a.y_gain[n] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + rw + i * 16 + fg * 4 + e;
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          const int n = col0(jw + j) + fr;
          xo[i][j][e] = (m < a.M && n < a.N) ? a.out_f32[(long long)m * a.ldo + n] : 0.f;
        }
      }
    float ymax = 0.f;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + rw + i * 16 + fg * 4 + e;
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          const int n = col0(jw + j) + fr;
          const bool ok = m < a.M && n < a.N;
          float xn = 0.f;
          if (ok) {
            xn = xo[i][j][e] + val(i, j, e);
            a.out_f32[(long long)m * a.ldo + n] = xn;
          }
          ymax = fmaxf(ymax, resid_out<P>(a, m, n, xn, fr, ok, gn[j]));
        }
      }
    amax_flush(a.y_amax, ymax, lane);
  } else if constexpr (EPI == E_STORE) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + rw + i * 16 + fg * 4 + e;
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          const int n = col0(jw + j) + fr;
          if (m < a.M && n < a.N) a.out_f32[(long long)m * a.ldo + n] = val(i, j, e);
        }
      }
  } else if constexpr (EPI == E_GLU) {
    // W rows are interleaved in 16-row groups (gate, up, gate, up, ...)
    float omax = 0.f;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + rw + i * 16 + fg * 4 + e;
        if (m >= a.M) continue;
#pragma unroll
        for (int j = 0; j < CB; j += 2) {
          const int col = ((cb0 + jw + j) / 2) * 16 + fr;
          if (col < a.N / 2)
            omax = fmaxf(omax, emit_glu<P>(a, m, col, val(i, j, e), val(i, j + 1, e)));
        }
      }
    amax_flush(a.out_amax, omax, lane);
  } else if constexpr (EPI == E_QKV) {
    // the staging LDS is free after the last part's barrier: stage the tile rows' metadata and,
    // when the tile holds q/k columns, their RoPE table rows, so that the epilogue issues no
    // dependent global loads
    const int nqk = (a.Hq + a.Hk) * a.hd, h2 = a.hd / 2;
    RowMeta* s_rm = reinterpret_cast<RowMeta*>(lds);
    float* s_rope = reinterpret_cast<float*>(lds + BM * sizeof(RowMeta));
    for (int r = tid; r < BM; r += NT)
      s_rm[r] = m0 + r < a.M ? a.rows[m0 + r] : RowMeta{0, 0, 0, 0};
    __syncthreads();
    if (col0(0) < nqk) {
      for (int q = tid; q < BM * h2; q += NT) {
        const int r = q / h2, i = q % h2;
        if (m0 + r < a.M)
          *reinterpret_cast<float2*>(s_rope + (r * h2 + i) * 2) = *reinterpret_cast<const float2*>(
              a.rope + ((long long)s_rm[r].pos * h2 + i) * 2);
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int rl = rw + i * 16 + fg * 4;  // tile row of e = 0
      const int m = m0 + rl;
      RowMeta rm[4];
      bool ok[4];
      const float* rr[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ok[e] = m + e < a.M;
        rm[e] = s_rm[rl + e];
        rr[e] = s_rope + (rl + e) * h2 * 2;
      }
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        const int n = col0(jw + j) + fr;
        float v[4], pr[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = val(i, j, e);
          // the other half of the head: the pair's other block, or (hd = 16) the lane 8 further
          const float other = val(i, j ^ 1, e), across = dpp_f<kRor + 8>(v[e]);
          pr[e] = n < nqk ? (a.hd == 16 ? across : other) : 0.f;
        }
        if (m >= a.M || n >= a.N) continue;
        if constexpr (P == P_F32) {
          const int i2 = (n % a.hd) % h2;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (ok[e])
              emit_qkv_core(a, P_F32, m + e, n, v[e], pr[e], rm[e],
                            n < nqk ? *reinterpret_cast<const float2*>(rr[e] + 2 * i2)
                                    : float2{1.f, 0.f});
        } else {
          emit_qkv4_rows(a, n, rm, ok, rr, v, pr, m);
        }
      }
    }
  }
}

template <int P, int AM, int EPI, int RB, int CB, int WVM, int WVN, bool kDeep>
static void gemm_tile(const GemmArgs& a, hipStream_t s) {
  constexpr int BM = 16 * RB * WVM, BN = 16 * CB * WVN;
  const int tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
  hipLaunchKernelGGL((gemm_tile_kernel<P, AM, EPI, RB, CB, WVM, WVN, kDeep>), dim3(tm * tn),
                     dim3(64 * WVM * WVN), 0, s, a, tm, tn);
}

// ---- split kernel (few rows) ----
//
// One workgroup per (group of 16 columns, or 32 for plain stores, and mb (1-4) blocks of 16 rows).
// Wave w of nw takes K parts w, w + nw, ...: it loads the part's weights and operand rows, runs
// every MFMA chain from zero and leaves the partials in LDS; after one barrier the workgroup adds
// each output's partials in part order and applies the epilogue.  No communication between
// workgroups.  A normed GEMM has one more wave, which derives the rows' RMSNorm scales meanwhile.
//
// A group of a RoPE GEMM is eight columns i .. i + 7 of a head's first half and their partners
// i + hd/2 ..., one of the gated MLP eight gate columns and their eight up columns, so both halves
// of a pair are eight lanes apart.  (Pairs of whole blocks give half as many workgroups, each with
// twice the weights and chains.)
//
// One-row launches at the 135M shape, BF16 / FP32, before in brackets: QKV 4.6 (6.1) / 4.6 (8.2) us,
// gate/up 4.1 (5.1) / 4.6 (7.6), O and down on average 5.3 (5.4) / 5.9 (7.3).
//
// What a decode step's GEMM waits for is a chain: weights from HBM, the MFMA chains, the sum and the
// epilogue.  FP32 weights go through LDS (kStage): a load instruction then covers four rows of 256
// bytes, eight cache lines; taken straight in fragment order it touches 32, and a CU's vector cache
// takes about one a cycle: with nine waves' fragments queued there, a one-row gate/up spent 8,000 of
// its 14,400 cycles before the first MFMA.

constexpr int SPLIT_WAVES = 16;
constexpr int SPLIT_ROWS = 64;

// inv[a_rows[m]] = the RMSNorm scale of row a_rows[m] (for the output layer)
__global__ void row_rms_kernel(const GemmArgs a, float* __restrict__ inv) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= a.M) return;
  const int ar = a.a_rows ? a.a_rows[m] : m;
  inv[ar] = inv_from_ssq(a.ssq + (long long)ar * (a.K / 16), a.K, a.eps);
}

// 16-column blocks per split group.  With several row blocks the gated MLP takes a gate and an up
// block in BF16 / FP8: half as many workgroups then read the operand rows (64 rows BF16: 5.8 us
// against 6.8; FP32, where the chains weigh more, 25 rows: 9.8 us against 7.3).
__host__ __device__ __forceinline__ constexpr int group_size(int prec, int epi, int mb) {
  return epi == E_STORE || (epi == E_GLU && mb > 1 && prec != P_F32) ? 2 : 1;
}

// log2 of head_dim (16, 32 or 64)
__device__ __forceinline__ int log2_hd(int hd) { return 31 - __builtin_clz(hd); }

// The column of lane c (0..15) in block j of split group gi.
__device__ __forceinline__ int split_col(int epi, int gs, int hd, int gi, int j, int c) {
  if (epi == E_QKV) {
    const int lg = log2_hd(hd), head = gi >> (lg - 4), i = (gi & ((hd >> 4) - 1)) * 8 + (c & 7);
    return head * hd + i + (c >> 3) * (hd >> 1);
  }
  if (epi == E_GLU && gs == 1) return ((gi >> 1) * 2 + (c >> 3)) * 16 + (gi & 1) * 8 + (c & 7);
  return (gi * gs + j) * 16 + c;
}

// Floats of a part's slot in LDS: its staged weights (kStage), then its partials in their place.
__host__ __device__ __forceinline__ constexpr int split_slot(int prec, int epi, int mb,
                                                             bool stage) {
  const int gs = group_size(prec, epi, mb), part = gs * mb * 256, w = stage ? gs * 1024 : 0;
  return part > w ? part : w;
}

template <int P, int AM, int EPI, int MB, bool kStage>
__global__ __launch_bounds__(64 * SPLIT_WAVES) void gemm_split_kernel(const GemmArgs a, int nw) {
  static_assert(!kStage || P == P_F32, "only FP32 weights are staged");
  constexpr int ES = PT<P>::ES;
  constexpr int GS = group_size(P, EPI, MB);
  constexpr int SLOT = split_slot(P, EPI, MB, kStage);
  extern __shared__ __align__(16) float lds[];  // [part][SLOT], then the rows' scales [64]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  const int K = a.K, N = a.N;
  const int S = (K + KP - 1) / KP;
  const int gi = blockIdx.x, r0 = blockIdx.y * MB * 16;
  const int M = min(a.M - r0, MB * 16);
  float* s_inv = lds + S * SLOT;
  const uint8_t* A8 = static_cast<const uint8_t*>(a.A);
  const uint8_t* W8 = static_cast<const uint8_t*>(a.W);
  // only the output layer gathers its A rows (launch_gemm checks this)
  const int32_t* const a_rows = EPI == E_STORE ? a.a_rows : nullptr;

  // The inputs of this thread's first epilogue item (row t / 16, column t % 16) are requested first:
  // the row metadata of a q/k/v output, or the residual value and gain.
  int pre_stream = 0, pre_pos = 0, pre_slot = 0;
  float2 pre_cs{1.f, 0.f};
  float pre_x = 0.f, pre_g = 0.f;
  const int em = min(int(threadIdx.x) >> 4, M - 1);
  const int en = split_col(EPI, GS, EPI == E_QKV ? a.hd : 64, gi, 0, threadIdx.x & 15);
  if constexpr (EPI == E_QKV) {
    const v4i rm = *reinterpret_cast<const v4i*>(a.rows + r0 + em);  // stream, pos, tok, slot
    pre_stream = rm[0];
    pre_pos = rm[1];
    pre_slot = rm[3];
  } else if constexpr (EPI == E_RESID) {
    const int n = min(en, N - 1);
    const float* xp = a.out_f32 + (long long)(r0 + em) * a.ldo + n;
    pre_x = *xp;
    pre_g = *(a.y_out ? a.y_gain + n : xp);  // (unused without y_out)
  }

  if (AM == A_NORM && wave == nw) {
    // the rows' scales, one row per lane
    if (lane < M) {
      const int ar = a_rows ? a_rows[r0 + lane] : r0 + lane;
      s_inv[lane] = a_row_inv(a, ar);
    }
  } else {
    // This lane's A row of each row block (rows past M repeat row M - 1; never stored).
    int arow[MB];
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
      arow[rb] = r0 + min(rb * 16 + fr, M - 1);
      if (a_rows) arow[rb] = a_rows[arow[rb]];
    }
    // W rows of this lane: fragment row fr, or when staged rows 4 q + fg, chunk fr of the part
    // (columns past N repeat column N - 1; never stored)
    constexpr int WR = kStage ? 4 : 1;
    const uint8_t* wrow[GS][WR];
#pragma unroll
    for (int j = 0; j < GS; ++j)
#pragma unroll
      for (int q = 0; q < WR; ++q) {
        const int c = kStage ? 4 * q + fg : fr;
        const int n = min(split_col(EPI, GS, EPI == E_QKV ? a.hd : 64, gi, j, c), N - 1);
        wrow[j][q] = W8 + (long long)n * K * ES;
      }
    // two parts of a wave are requested together where their registers allow
    constexpr bool kTwo = GS == 1 && MB <= 2;
    constexpr int NB = kTwo ? 2 : 1;
    typename Frag<P>::T bf[NB][GS], af[NB][MB];
    v4f wv[NB][GS][WR];  // staged: the part's weights as loaded
    // every load of a part is issued unconditionally (clamped into its row; entries at or beyond K
    // are zeroed), so that the number in flight is the same on every path
    auto load = [&](int q, int s) {
      const int k0 = s * KP;
      if constexpr (kStage) {
        const int k = k0 + 4 * fr;
#pragma unroll
        for (int j = 0; j < GS; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const v4f v = *reinterpret_cast<const v4f*>(wrow[j][u] + min(k, K - 4) * 4);
            wv[q][j][u] = v;
          }
      } else {
#pragma unroll
        for (int j = 0; j < GS; ++j) Frag<P>::load_clamped(bf[q][j], wrow[j][0], k0, K, fg);
      }
#pragma unroll
      for (int rb = 0; rb < MB; ++rb)
        Frag<P>::load_clamped(af[q][rb], A8 + (long long)arow[rb] * K * ES, k0, K, fg);
    };
    auto part = [&](int q, int s) {
      float* slot = lds + s * SLOT;
      if constexpr (kStage) {
        // Rows of 256 bytes; chunk c of row r lies at chunk c ^ r, so that neither the writes
        // (sixteen chunks of a row) nor the reads (one chunk of sixteen rows) meet in a bank.
        // Only this wave uses the slot before the barrier.
        const bool in = s * KP + 4 * fr < K;
#pragma unroll
        for (int j = 0; j < GS; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int r = 4 * u + fg;
            *reinterpret_cast<v4f*>(slot + j * 1024 + r * 64 + ((fr ^ r) & 15) * 4) =
                in ? wv[q][j][u] : v4f{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
        for (int j = 0; j < GS; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const v4f v = *reinterpret_cast<const v4f*>(slot + j * 1024 + fr * 64 +
                                                        (((4 * fg + u) ^ fr) & 15) * 4);
            if constexpr (P == P_F32) {
#pragma unroll
              for (int e = 0; e < 4; ++e) bf[q][j][4 * u + e] = v[e];
            }
          }
      }
      v4f acc[GS][MB];
#pragma unroll
      for (int j = 0; j < GS; ++j)
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) {
          acc[j][rb] = v4f{0.f, 0.f, 0.f, 0.f};
          Frag<P>::mma(acc[j][rb], af[q][rb], bf[q][j]);
        }
#pragma unroll
      for (int j = 0; j < GS; ++j)
#pragma unroll
        for (int rb = 0; rb < MB; ++rb) {
          float* dst = slot + ((j * MB + rb) << 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) dst[(fg * 4 + e) * 16 + fr] = acc[j][rb][e];
        }
    };
    for (int s = wave; s < S; s += NB * nw) {
      load(0, s);
      if (kTwo && s + nw < S) {
        load(NB - 1, s + nw);
        part(0, s);
        part(NB - 1, s + nw);
      } else {
        part(0, s);
      }
    }
  }
  // the RoPE entry of this thread's first q/k output (its metadata was requested first)
  if constexpr (EPI == E_QKV) {
    const int h2 = a.hd >> 1, i = (gi & ((a.hd >> 4) - 1)) * 8 + (threadIdx.x & 7);
    pre_cs = *reinterpret_cast<const float2*>(a.rope + ((long long)pre_pos * h2 + i) * 2);
  }
  __syncthreads();
  const float deq = (P == P_FP8) ? a.a_scale * a.w_scale : 1.0f;
  // output (row m of the chunk, block j, lane c) = (partials summed in part order) * deq * scale
  auto sum = [&](int m, int j, int c) {
    const float* src = lds + ((j * MB + (m >> 4)) << 8) + (m & 15) * 16 + c;
    float v = 0.f;
    int s = 0;
    for (; s + 8 <= S; s += 8) {  // eight LDS reads at a time
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = src[(s + u) * SLOT];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += x[u];
    }
    for (; s < S; ++s) v += src[s * SLOT];
    return v * deq * (AM == A_NORM ? s_inv[m] : 1.f);
  };
  if constexpr (EPI == E_GLU) {
    // one block: lanes 0-7 of sixteen hold the gate columns, lanes 8-15 their up columns
    float omax = 0.f;
    for (int t0 = 0; t0 < M * 16; t0 += blockDim.x) {
      const int t = t0 + threadIdx.x;
      const int m = min(t >> 4, M - 1), c = t & 15;
      const float v = sum(m, 0, c);
      const float up = GS == 2 ? sum(m, GS - 1, c) : dpp_f<kRor + 8>(v);
      const int col = GS == 2 ? gi * 16 + c : gi * 8 + (c & 7);
      if (t < M * 16 && (GS == 2 || c < 8) && col < N / 2)
        omax = fmaxf(omax, emit_glu<P>(a, r0 + m, col, v, up));
    }
    amax_flush(a.out_amax, omax, lane);
  } else if constexpr (EPI == E_RESID) {
    // one block per group; every lane takes part in the block sums of squares
    float ymax = 0.f;
    for (int t0 = 0; t0 < M * 16; t0 += blockDim.x) {
      const int t = t0 + threadIdx.x;
      const int m = t >> 4, c = t & 15;
      const int n = gi * 16 + c;
      const bool ok = t < M * 16 && n < N;
      float xn = 0.f;
      float* o = a.out_f32 + (long long)(r0 + m) * a.ldo + n;
      if (ok) {
        xn = (t0 == 0 ? pre_x : *o) + sum(m, 0, c);
        *o = xn;
      }
      const float g = t0 == 0 ? pre_g : (ok && a.y_out ? a.y_gain[n] : 0.f);
      ymax = fmaxf(ymax, resid_out<P>(a, r0 + m, n, xn, c, ok, g));
    }
    amax_flush(a.y_amax, ymax, lane);
  } else if constexpr (EPI == E_STORE) {
    for (int t = threadIdx.x; t < M * 32; t += blockDim.x) {
      const int m = t >> 5, j = (t >> 4) & 1, c = t & 15;
      const int n = (2 * gi + j) * 16 + c;
      if (n < N) a.out_f32[(long long)(r0 + m) * a.ldo + n] = sum(m, j, c);
    }
  } else {
    // the group's head: a q head, a k head or a v head (head_dim is a power of two)
    const int lg = log2_hd(a.hd), hd = a.hd, h2 = hd >> 1;
    const int head = gi >> (lg - 4);
    for (int t0 = 0; t0 < M * 16; t0 += blockDim.x) {
      const int t = t0 + threadIdx.x;
      const int m = min(t >> 4, M - 1), c = t & 15;
      float v = sum(m, 0, c);
      const float partner = dpp_f<kRor + 8>(v);  // the other half of the RoPE pair
      if (t >= M * 16) continue;
      const int i = (gi & ((hd >> 4) - 1)) * 8 + (c & 7), within = i + (c >> 3) * h2;
      if (t0 > 0) {
        const v4i rm = *reinterpret_cast<const v4i*>(a.rows + r0 + m);
        pre_stream = rm[0];
        pre_slot = rm[3];
        pre_cs = *reinterpret_cast<const float2*>(a.rope + ((long long)rm[1] * h2 + i) * 2);
      }
      if (head < a.Hq + a.Hk) {
        const float2 cs = pre_cs;
        v = c < 8 ? v * cs.x - partner * cs.y : v * cs.x + partner * cs.y;
      }
      void* base = a.q_out;
      long long idx = (long long)(r0 + m) * a.Hq * hd + head * hd + within;
      if (head >= a.Hq) {
        const bool is_k = head < a.Hq + a.Hk;
        const int kvh = head - a.Hq - (is_k ? 0 : a.Hk);
        const long long sb = (long long)pre_stream * a.kv_stride + (long long)kvh * a.ring * hd;
        base = is_k ? a.k_cache : a.vt_cache;
        idx = sb + (is_k ? (long long)pre_slot * hd + within : (long long)within * a.ring + pre_slot);
      }
      if constexpr (P == P_F32)
        PT<P_F32>::store(base, idx, v, 1.f);
      else
        PT<P_BF16>::store(base, idx, v, 1.f);
    }
  }
}

// ---- attention ------------------------------------------------------------------------------
//
// Keys of a query's window [s(pos), pos] are cut into 64-key chunks at fixed absolute positions,
// chunks into quads of 4 (256 keys) and quads into groups of 4 (1,024 keys).  A chunk partial is
// one softmax pass over its 64 keys:
//   m = max score, p = 2^(score - m), l = sum p (fixed order), o = V^T P^T (chained MFMAs).
// Partials are combined by the left fold
//   (m, l, o) <- (M, l 2^(m - M) + l' 2^(m' - M), o 2^(m - M) + o' 2^(m' - M)),  M = max(m, m'),
// at three levels, each from the empty state (-inf, 0, 0) and in order: the chunks of a quad, the
// quads of a group, then the groups; the output is o / l.  Folding the empty state is exact in
// either operand, so chunks outside a column's window drop out and a column's result does not
// depend on the other columns of its launch, nor on which kernel computes it.
// S^T = K Q^T puts keys on MFMA rows and (query, head) pairs on columns, so the probabilities
// leave the QK MFMA in the B-operand layout of the P*V MFMA and no transpose is needed.  Within a
// chunk, MFMA row r of block b holds key 16 (r / 4) + 4 b + r % 4: a lane's P*V operand then
// covers 16 consecutive keys over the 4 blocks, so its V^T reads are contiguous.

constexpr int KCH = kAttnChunk;  // keys per chunk
constexpr int QCH = 4;       // chunks per quad
constexpr int GQ = 4;        // quads per group
constexpr int MAXQ = 12;     // quads an item may span (window <= 2,048 keys + 15 query positions)
constexpr int HDMAX = 64;
constexpr int QSTATE = 2 + HDMAX / 4;  // floats per lane of a stored state: m, l, o[16]

__device__ __forceinline__ int window_start(int pos, int L, int C) {
  return pos < L ? 0 : C * (1 + (pos - L) / C);
}

// key offset within its chunk of MFMA row r of block b
__device__ __forceinline__ int chunk_key(int b, int r) { return (r >> 2) * 16 + b * 4 + (r & 3); }

struct AttnCol {
  bool valid;
  int pos, cs, row, head;
};

struct ChunkState {
  float m, l;
  v4f o[HDMAX / 16];  // o[hb][j]: hd index hb*16 + 4 (lane/16) + j of column lane%16
};

__device__ __forceinline__ void state_empty(ChunkState& a) {
  a.m = -INFINITY;
  a.l = 0.f;
#pragma unroll
  for (int hb = 0; hb < HDMAX / 16; ++hb) a.o[hb] = v4f{0.f, 0.f, 0.f, 0.f};
}

__device__ __forceinline__ void fold(ChunkState& a, const ChunkState& b, int nhb) {
  const float M = fmaxf(a.m, b.m);
  if (M == -INFINITY) return;
  const float e1 = exp2f(a.m - M), e2 = exp2f(b.m - M);
  a.l = a.l * e1 + b.l * e2;
#pragma unroll
  for (int hb = 0; hb < HDMAX / 16; ++hb)
    if (hb < nhb) a.o[hb] = a.o[hb] * e1 + b.o[hb] * e2;
  a.m = M;
}

// state of one lane <-> 18 floats (wave-interleaved: float i of lane l at i * 64 + l)
__device__ __forceinline__ void state_put(float* dst, const ChunkState& st, int lane) {
  dst[lane] = st.m;
  dst[64 + lane] = st.l;
#pragma unroll
  for (int hb = 0; hb < HDMAX / 16; ++hb)
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[(2 + hb * 4 + j) * 64 + lane] = st.o[hb][j];
}
__device__ __forceinline__ void state_get(ChunkState& st, const float* src, int lane) {
  st.m = src[lane];
  st.l = src[64 + lane];
#pragma unroll
  for (int hb = 0; hb < HDMAX / 16; ++hb)
#pragma unroll
    for (int j = 0; j < 4; ++j) st.o[hb][j] = src[(2 + hb * 4 + j) * 64 + lane];
}

template <int PA>
struct QFrag {
  v8bf b[2];
  float f[HDMAX / 4];
};

template <int PA>
__device__ __forceinline__ void load_q(QFrag<PA>& q, const AttnArgs& a, const AttnCol& c,
                                       int grp) {
  const int hd = a.hd;
  const long long qbase = ((long long)c.row * a.Hq + c.head) * hd;
  // every load is issued (clamped into the row; c's row is valid even for an invalid column) and
  // the entries outside are zeroed afterwards, so that no branch makes the loads' count
  // path-dependent (a later wait would then drain every load in flight)
  if constexpr (PA == P_BF16) {
    const uint16_t* Q = static_cast<const uint16_t*>(a.q);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int k = s * 32 + grp * 8;
      const v4i v = *reinterpret_cast<const v4i*>(Q + qbase + min(k, hd - 8));
      q.b[s] = __builtin_bit_cast(v8bf, (c.valid && k < hd) ? v : v4i{0, 0, 0, 0});
    }
  } else {
    // step s, lane group g: hd entry 16 g + s (the same mapping is used for K)
    const float* Q = static_cast<const float*>(a.q);
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      const int k = 16 * grp + 4 * qd;
      const v4f v = *reinterpret_cast<const v4f*>(Q + qbase + min(k, hd - 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) q.f[4 * qd + e] = (c.valid && k < hd) ? v[e] : 0.f;
    }
  }
}

// Every key of the chunk is in every column's window.
__device__ __forceinline__ bool chunk_inside(const AttnItem& it, int g, int key0) {
  return key0 >= it.cs_hi && key0 + KCH - 1 <= it.pos_base + it.c0 / g;
}

// Softmax of one chunk's masked scores st (in place: scores -> probabilities); returns (m, l).
// exp2f is the hardware's exponential but below -126, where it scales its argument and result
// to reach the denormals; a lane's smallest score tells whether any of its 16 needs that.  A chunk
// inside every window has no masks.  Both are uniform branches; together they take a chunk
// of BF16 attention, which is bound by these instructions, from about 900 to 350 of them.
__device__ __forceinline__ void chunk_softmax(v4f (&st)[4], const AttnArgs& a, const AttnCol& c,
                                              int key0, int grp, bool inside, float& m,
                                              float& l) {
  float mx = -INFINITY, mn = INFINITY;
  if (inside) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        st[b][j] *= a.scale_log2;
        mx = fmaxf(mx, st[b][j]);
        mn = fminf(mn, st[b][j]);
      }
  } else {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int key = key0 + chunk_key(b, grp * 4 + j);
        const bool ok = c.valid && key >= c.cs && key <= c.pos;
        st[b][j] = ok ? st[b][j] * a.scale_log2 : -INFINITY;
        mx = fmaxf(mx, st[b][j]);
      }
    mn = -INFINITY;
  }
  auto larger = [](float x, float y) { return fmaxf(x, y); };
  auto plus = [](float x, float y) { return x + y; };
  mx = combine_x32(combine_x16(mx, larger), larger);
  float ls = 0.f;
  if (__builtin_amdgcn_ballot_w64(!(mn <= mx && mn - mx >= -126.f)) == 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int j = 0; j < 4; ++j) st[b][j] = __builtin_amdgcn_exp2f(st[b][j] - mx);
      ls += (st[b][0] + st[b][1]) + (st[b][2] + st[b][3]);
    }
  } else {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int j = 0; j < 4; ++j) st[b][j] = mx == -INFINITY ? 0.f : exp2f(st[b][j] - mx);
      ls += (st[b][0] + st[b][1]) + (st[b][2] + st[b][3]);
    }
  }
  ls = combine_x32(combine_x16(ls, plus), plus);
  m = mx;
  l = ls;
}

// The probabilities of four keys as BF16, round to nearest even.
__device__ __forceinline__ v4s prob_bf16(const v4f& p) {
  typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(v4s, __builtin_convertvector(p, v4bf));
}

// One chunk partial for the 16 columns of this wave.
template <int PA>
__device__ __forceinline__ ChunkState chunk_partial(const AttnArgs& a, const AttnItem& it,
                                                    const AttnCol& c, const QFrag<PA>& q,
                                                    int chunk, int col, int grp) {
  const int hd = a.hd, nhb = hd / 16;
  const long long sbase = (long long)it.stream * a.kv_stride + (long long)it.kvh * a.ring * hd;
  const int key0 = chunk * KCH;
  // ring slot of key key0 + off (0 <= off < 64 <= ring): one wave-uniform modulo per chunk
  const int base = key0 % a.ring;
  auto slot_of = [&](int off) {
    const int t = base + off;
    return t >= a.ring ? t - a.ring : t;
  };
  // V^T operand of this lane: keys key0 + 16 grp .. + 15 (never wrapping: ring % 16 == 0)
  const int vslot = slot_of(16 * grp);
  v4f st[4];
  ChunkState r;
#pragma unroll
  for (int hb = 0; hb < HDMAX / 16; ++hb) r.o[hb] = v4f{0.f, 0.f, 0.f, 0.f};
  if constexpr (PA == P_BF16) {
    const uint16_t* Kc = static_cast<const uint16_t*>(a.k_cache);
    const uint16_t* Vt = static_cast<const uint16_t*>(a.vt_cache);
    // K and V^T fragments of the 4 blocks, all loads in flight together
    v4i kf[4][2];
    v4i vf[HDMAX / 16][2];  // 16 keys per lane per hd block
    // (loads clamped into range and masked afterwards, as for q)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const long long ks = sbase + (long long)slot_of(chunk_key(b, col)) * hd;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = s * 32 + grp * 8;
        const v4i v = *reinterpret_cast<const v4i*>(Kc + ks + min(k, hd - 8));
        kf[b][s] = k < hd ? v : v4i{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int hb = 0; hb < HDMAX / 16; ++hb)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int hc = min(hb, nhb - 1);
        const v4i v = *reinterpret_cast<const v4i*>(
            Vt + sbase + (long long)(hc * 16 + col) * a.ring + vslot + 8 * h);
        vf[hb][h] = hb < nhb ? v : v4i{0, 0, 0, 0};
      }
    __builtin_amdgcn_sched_barrier(0);  // every load above is issued before the first MFMA
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      st[b] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (s * 32 < hd)
          st[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, kf[b][s]),
                                                          q.b[s], st[b], 0, 0, 0);
    }
    chunk_softmax(st, a, c, key0, grp, chunk_inside(it, a.Hq / a.Hk, key0), r.m, r.l);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const v4s pb = prob_bf16(st[b]);
#pragma unroll
      for (int hb = 0; hb < HDMAX / 16; ++hb)
        if (hb < nhb) {
          // keys 4 b .. 4 b + 3 of the lane's 16: dwords 2 (b % 2) .. + 1 of half b / 2
          const v4i w = vf[hb][b >> 1];
          const v4s va = __builtin_bit_cast(v4s, (b & 1) ? int2{w[2], w[3]} : int2{w[0], w[1]});
          r.o[hb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, pb, r.o[hb], 0, 0, 0);
        }
    }
  } else {
    const float* Kc = static_cast<const float*>(a.k_cache);
    const float* Vt = static_cast<const float*>(a.vt_cache);
    // every K and V^T fragment of the chunk requested before the first MFMA
    v4f kf[4][4], vf[HDMAX / 16][4];
    // (loads clamped into range and masked afterwards, as for q)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const long long ks = sbase + (long long)slot_of(chunk_key(b, col)) * hd;
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int k = 16 * grp + 4 * qd;
        const v4f v = *reinterpret_cast<const v4f*>(Kc + ks + min(k, hd - 4));
        kf[b][qd] = k < hd ? v : v4f{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int hb = 0; hb < HDMAX / 16; ++hb)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int hc = min(hb, nhb - 1);
        const v4f v = *reinterpret_cast<const v4f*>(
            Vt + sbase + (long long)(hc * 16 + col) * a.ring + vslot + 4 * b);
        vf[hb][b] = hb < nhb ? v : v4f{0.f, 0.f, 0.f, 0.f};
      }
    // every load above is issued before the first MFMA (the scheduler would otherwise sink the
    // V^T loads behind the score chains, adding a memory round trip)
    __builtin_amdgcn_sched_barrier(0);
    // the four blocks' MFMA chains interleaved step by step
#pragma unroll
    for (int b = 0; b < 4; ++b) st[b] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < HDMAX / 4; ++s)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        st[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][s >> 2][s & 3], q.f[s], st[b], 0, 0, 0);
    chunk_softmax(st, a, c, key0, grp, chunk_inside(it, a.Hq / a.Hk, key0), r.m, r.l);
    // the four hd blocks' P*V chains interleaved step by step (same order per chain)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int hb = 0; hb < HDMAX / 16; ++hb)
          if (hb < nhb)
            r.o[hb] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[hb][b][j], st[b][j], r.o[hb], 0, 0, 0);
  }
  return r;
}

// Column col of an item; a column past ncols is invalid and takes the last valid column's row,
// head and position, so that every address derived from it stays inside the pass.
__device__ __forceinline__ AttnCol attn_col(const AttnArgs& a, const AttnItem& it, int col) {
  const int g = a.Hq / a.Hk;
  const int cc = it.c0 + min(col, it.ncols - 1);
  AttnCol c;
  c.valid = col < it.ncols;
  const int qo = cc / g;
  c.head = it.kvh * g + cc % g;
  c.pos = it.pos_base + qo;
  c.row = it.row_base + qo;
  c.cs = it.cs_lo;
  if (it.cs_lo != it.cs_hi) c.cs = window_start(c.pos, a.ctx_len, a.slide);
  return c;
}

template <int PO>
__device__ __forceinline__ float attn_store(const AttnArgs& a, const AttnItem& it,
                                            const ChunkState& s, int col, int grp) {
  const int g = a.Hq / a.Hk, hd = a.hd, nhb = hd / 16;
  float omax = 0.f;
  if (col >= it.ncols) return omax;
  const int cc = it.c0 + col;
  const long long orow = it.row_base + cc / g;
  const int oh = it.kvh * g + cc % g;
  const float oinv = (PO == P_FP8) ? 1.0f / a.out_scale : 1.0f;
#pragma unroll
  for (int hb = 0; hb < HDMAX / 16; ++hb)
    if (hb < nhb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int d = hb * 16 + grp * 4 + j;
        const float o = s.o[hb][j] / s.l;
        const long long idx = orow * ((long long)a.Hq * hd) + (long long)oh * hd + d;
        omax = fmaxf(omax, fabsf(o));
        if constexpr (PO == P_F32)
          PT<P_F32>::store(a.out, idx, o, 1.f);
        else if constexpr (PO == P_BF16)
          PT<P_BF16>::store(a.out, idx, o, 1.f);
        else
          PT<P_FP8>::store(a.out, idx, o, oinv);
      }
  return omax;
}

// Groups of up to 4 consecutive items of one stream's kv head (several rows of a stream: prompts and
// encode): a workgroup stages each K and V^T chunk of their windows in LDS once, and each wave takes
// one item.  In the MFMA layouts a load asks for 16 bytes of each of 16 to 64 cache lines, one line a
// cycle, for each item again; staged, the rows come whole and once.  LDS holds K rows of hd entries
// and V^T rows of 64 keys in units of 16 bytes, XORed with the row so that the 16 rows of a fragment
// read fall on different banks; the next chunk's units are in registers while this one is computed.
// Every item folds its own chunks in the order of the other kernels, so the bits are theirs.  Full
// shape, 512 rows of one FP32 stream: 67.8 us a layer (a wave per chunk, K and V for itself) to 37
// (the FP32 matrix rate alone is 16); 32,768 rows of 64 BF16 streams: 177 to 81, bound by the
// softmax's vector instructions.
//  * kQuads (too few items to fill the chip with one wave each): a workgroup per (group, quad), the
//    quads' states to the fold kernel as in attention_quad_kernel;
//  * otherwise a workgroup per group runs over all its chunks, the three fold levels in registers.
// Units of work are placed as in attention_quad_kernel, so that a stream's groups read one L2.
constexpr int GI = 4;  // items of a group

template <int PA, int PO, bool kQuads, bool kFull>
__global__ __launch_bounds__(256) void attention_group_kernel(const AttnArgs a) {
  constexpr int ES = PA == P_BF16 ? 2 : 4;
  constexpr int U = KCH * ES / 16;     // 16-byte units of a row (64 hd entries or 64 keys)
  constexpr int E = KCH * U / 256;     // units of K, and of V^T, that a thread stages
  constexpr int NBUF = PA == P_BF16 ? 2 : 1;
  __shared__ v4i s_kv[NBUF][2][KCH * U];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int nu = gridDim.x, q8 = nu / 8, r8 = nu % 8, xcd = blockIdx.x % 8;
  const int u = xcd * q8 + min(xcd, r8) + int(blockIdx.x) / 8;
  const int gi = kQuads ? u % a.n_groups : u, qi = kQuads ? u / a.n_groups : 0;
  const int gw = __builtin_amdgcn_readfirstlane(a.items[gi].group);
  const int first = gw >> 2, last = first + (gw & 3);
  int lo = a.items[first].c_lo, hi = a.items[last].c_hi;  // positions do not decrease
  const int slot_lo = a.items[first].slot_lo;
  const int item = __builtin_amdgcn_readfirstlane(min(first + wave, last));
  const bool mine = first + wave <= last;
  const AttnItem it = a.items[item];
  const int hd = kFull ? HDMAX : a.hd, nhb = hd / 16, g = a.Hq / a.Hk;
  int base = slot_lo;
  if constexpr (kQuads) {
    const int q0 = (lo / QCH + qi) * QCH, c_first = lo;
    lo = max(lo, q0);
    hi = min(hi, q0 + QCH - 1);
    if (lo > hi) return;
    base += (lo - c_first) * KCH;
    while (base >= a.ring) base -= a.ring;
  }
  const AttnCol c = attn_col(a, it, col);
  QFrag<PA> q;
  load_q<PA>(q, a, c, grp);
  const long long sbase = (long long)it.stream * a.kv_stride + (long long)it.kvh * a.ring * hd;
  const char* Kc = static_cast<const char*>(a.k_cache) + sbase * ES;
  const char* Vt = static_cast<const char*>(a.vt_cache) + sbase * ES;
  constexpr int EPU = 16 / ES;  // entries of a unit
  // the rows' XORs: the 16 K rows of a fragment are 16 (col / 4) + col % 4 (+ 4 b), the 16 V^T rows
  // col (+ 16 hb); a BF16 row fills half the banks, so a row's lowest bit chooses the half
  auto kx = [](int r) {
    return PA == P_BF16 ? ((r >> 1) & 1) | ((r >> 3) & 6) : (r & 3) | ((r >> 2) & 12);
  };
  auto vx = [](int r) { return PA == P_BF16 ? (r >> 1) & 7 : r & 15; };
  v4i kr[E], vr[E];
  auto fetch = [&]() {  // the chunk at ring slot base (loads clamped into the head's rows)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + 256 * e, r = i / U, un = i % U;
      int ks = base + r;
      ks = ks >= a.ring ? ks - a.ring : ks;
      const int k = kFull ? un * EPU : min(un * EPU, hd - EPU);
      const v4i v = *reinterpret_cast<const v4i*>(Kc + ((long long)ks * hd + k) * ES);
      kr[e] = kFull || un * EPU < hd ? v : v4i{0, 0, 0, 0};
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + 256 * e, r = i / U, un = i % U;
      int vs = base + un * EPU;  // never wraps inside a unit: ring and chunk starts are 16 n
      vs = vs >= a.ring ? vs - a.ring : vs;
      const int d = kFull ? r : min(r, hd - 1);
      const v4i v = *reinterpret_cast<const v4i*>(Vt + ((long long)d * a.ring + vs) * ES);
      vr[e] = kFull || r < hd ? v : v4i{0, 0, 0, 0};
    }
  };
  ChunkState run, gs, qs;
  state_empty(run);
  state_empty(gs);
  state_empty(qs);
  const int i_lo = mine ? it.c_lo : hi + 1, i_hi = it.c_hi;
  fetch();
  for (int ch = lo; ch <= hi; ++ch) {
    v4i(*kv)[KCH * U] = s_kv[NBUF == 2 ? ch & 1 : 0];
    if (NBUF == 1 && ch > lo) __syncthreads();  // the chunk before has been read
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + 256 * e, r = i / U, un = i % U;
      kv[0][r * U + (un ^ kx(r))] = kr[e];
      kv[1][r * U + (un ^ vx(r))] = vr[e];
    }
    __syncthreads();
    if (ch < hi) {
      base += KCH;
      base = base >= a.ring ? base - a.ring : base;
      fetch();
    }
    if (ch < i_lo || ch > i_hi) continue;
    const int key0 = ch * KCH;
    const int krow = (col >> 2) * 16 + (col & 3), kxr = kx(krow), vxr = vx(col);
    v4f st[4];
    ChunkState r;
#pragma unroll
    for (int hb = 0; hb < HDMAX / 16; ++hb) r.o[hb] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 4; ++b) st[b] = v4f{0.f, 0.f, 0.f, 0.f};
    if constexpr (PA == P_BF16) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (kFull || s * 32 < hd)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            st[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(v8bf, kv[0][(krow + 4 * b) * U + ((4 * s + grp) ^ kxr)]),
                q.b[s], st[b], 0, 0, 0);
    } else {
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        v4f kf[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
          kf[b] = __builtin_bit_cast(v4f, kv[0][(krow + 4 * b) * U + ((4 * grp + qd) ^ kxr)]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            st[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][e], q.f[4 * qd + e], st[b], 0, 0, 0);
      }
    }
    chunk_softmax(st, a, c, key0, grp, chunk_inside(it, g, key0), r.m, r.l);
    if constexpr (PA == P_BF16) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v4i vf[HDMAX / 16];
#pragma unroll
        for (int hb = 0; hb < HDMAX / 16; ++hb)
          vf[hb] = kv[1][(hb * 16 + col) * U + ((2 * grp + h) ^ vxr)];
#pragma unroll
        for (int b = 2 * h; b < 2 * h + 2; ++b) {
          const v4s pb = prob_bf16(st[b]);
#pragma unroll
          for (int hb = 0; hb < HDMAX / 16; ++hb)
            if (hb < nhb) {
              const v4i w = vf[hb];
              const v4s va =
                  __builtin_bit_cast(v4s, (b & 1) ? int2{w[2], w[3]} : int2{w[0], w[1]});
              r.o[hb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(va, pb, r.o[hb], 0, 0, 0);
            }
        }
      }
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        v4f vf[HDMAX / 16];
#pragma unroll
        for (int hb = 0; hb < HDMAX / 16; ++hb)
          vf[hb] = __builtin_bit_cast(v4f, kv[1][(hb * 16 + col) * U + ((4 * grp + b) ^ vxr)]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int hb = 0; hb < HDMAX / 16; ++hb)
            if (hb < nhb)
              r.o[hb] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(vf[hb][j], st[b][j], r.o[hb], 0, 0, 0);
      }
    }
    fold(qs, r, nhb);
    if constexpr (!kQuads) {
      if (ch % QCH == QCH - 1 || ch == i_hi) {
        fold(gs, qs, nhb);
        state_empty(qs);
        if (ch % (QCH * GQ) == QCH * GQ - 1 || ch == i_hi) {
          fold(run, gs, nhb);
          state_empty(gs);
        }
      }
    }
  }
  if (!mine) return;
  if constexpr (kQuads) {
    if (hi < i_lo || lo > i_hi) return;
    state_put(a.ws + ((long long)item * MAXQ + lo / QCH - i_lo / QCH) * QSTATE * 64, qs, lane);
  } else {
    float omax = attn_store<PO>(a, it, run, col, grp);
    if (a.out_amax) {
      omax = wave_max_f(omax);
      if (lane == 0) atomic_max_abs(a.out_amax, omax);
    }
  }
}

// Few items (decode), first kernel: one 4-wave workgroup per (item, quad); wave w computes chunk
// 4 Q + w, wave 0 folds the quad in order and stores its state.  When several items share a
// stream's K/V (the column blocks of a multi-row pass, consecutive in the item list), work unit
// u = item + n_items * qi is placed by an XCD-aware bijection of the 1-D grid (dispatch is
// round-robin over the 8 XCDs): XCD x runs a contiguous range of units, so those items read the
// same K/V chunks from one L2.  Otherwise (one row per stream, where contiguous ranges would
// gather the empty units past short windows on a few XCDs) the units keep the round-robin order.
template <int PA>
__global__ __launch_bounds__(256) void attention_quad_kernel(const AttnArgs a) {
  __shared__ float part[QCH][QSTATE * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int nu = gridDim.x;
  int item = blockIdx.x % a.n_items, qi = blockIdx.x / a.n_items;
  if (a.xcd_place) {
    const int q8 = nu / 8, r8 = nu % 8, xcd = blockIdx.x % 8;
    const int u = xcd * q8 + min(xcd, r8) + blockIdx.x / 8;
    item = u % a.n_items;
    qi = u / a.n_items;
  }
  const AttnItem it = a.items[item];
  const int c_lo = it.c_lo, c_hi = it.c_hi;
  const int q0 = (c_lo / QCH + qi) * QCH;
  if (q0 > c_hi) return;  // beyond the item: its fold never reads this quad
  const AttnCol c = attn_col(a, it, col);
  const int nhb = a.hd / 16;
  const int ch = q0 + wave;
  if (ch >= c_lo && ch <= c_hi) {
    QFrag<PA> q;
    load_q<PA>(q, a, c, grp);
    state_put(part[wave], chunk_partial<PA>(a, it, c, q, ch, col, grp), lane);
  }
  __syncthreads();
  if (wave != 0) return;
  ChunkState qs, p;
  state_empty(qs);
  for (int w = 0; w < QCH; ++w) {
    if (q0 + w < c_lo || q0 + w > c_hi) continue;
    state_get(p, part[w], lane);
    fold(qs, p, nhb);
  }
  state_put(a.ws + ((long long)item * MAXQ + qi) * QSTATE * 64, qs, lane);
}

constexpr int BSTATE = 2 + 4;  // floats per lane of a one-block state

// Block hb of a state as a one-block state: o[0] holds what state_put laid out as o[hb].
__device__ __forceinline__ void block_get(ChunkState& st, const float* q, int hb, int lane) {
  st.m = q[lane];
  st.l = q[64 + lane];
#pragma unroll
  for (int j = 0; j < 4; ++j) st.o[0][j] = q[(2 + hb * 4 + j) * 64 + lane];
}

// Output block hb of the lane's column from its one-block state: attn_store for one block.
template <int PO>
__device__ __forceinline__ void block_store(const AttnArgs& a, const AttnItem& it,
                                            const ChunkState& run, int hb, int lane) {
  const int col = lane & 15, grp = lane >> 4;
  float omax = 0.f;
  if (col < it.ncols) {
    const int g = a.Hq / a.Hk, hd = a.hd;
    const int cc = it.c0 + col;
    const long long orow = it.row_base + cc / g;
    const int oh = it.kvh * g + cc % g;
    const float oinv = (PO == P_FP8) ? 1.0f / a.out_scale : 1.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int d = hb * 16 + grp * 4 + j;
      const float o = run.o[0][j] / run.l;
      const long long idx = orow * ((long long)a.Hq * hd) + (long long)oh * hd + d;
      omax = fmaxf(omax, fabsf(o));
      if constexpr (PO == P_F32)
        PT<P_F32>::store(a.out, idx, o, 1.f);
      else if constexpr (PO == P_BF16)
        PT<P_BF16>::store(a.out, idx, o, 1.f);
      else
        PT<P_FP8>::store(a.out, idx, o, oinv);
    }
  }
  if (a.out_amax) {
    omax = wave_max_f(omax);
    if (lane == 0) atomic_max_abs(a.out_amax, omax);
  }
}

// Few items, second kernel: quads -> groups -> output, one workgroup per (item, head-dimension
// block hb): a state's m and l and its block hb fold on their own (the other blocks only scale
// alike), so the four blocks' folds run side by side.  Wave w folds the quads of the item's w-th
// group (their states loaded together) and leaves the group state in LDS; wave 0 then folds the
// groups in order.  The folds are the group kernel's, in the same order, so the output is
// the same.
constexpr int FOLD_WAVES = (MAXQ + GQ - 2) / GQ + 1;  // groups an item may span
template <int PO>
__global__ __launch_bounds__(64 * FOLD_WAVES) void attention_fold_kernel(const AttnArgs a) {
  __shared__ float gst[FOLD_WAVES][BSTATE * 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col = lane & 15, grp = lane >> 4;
  const int item = blockIdx.x, hb = blockIdx.y;
  const AttnItem it = a.items[item];
  const int c_lo = it.c_lo, c_hi = it.c_hi;
  const int qlo = c_lo / QCH, qhi = c_hi / QCH;
  const int gfirst = (qlo / GQ) * GQ;
  const int ng = (qhi - gfirst) / GQ + 1;  // <= FOLD_WAVES: qhi - qlo < MAXQ
  const float* src = a.ws + (long long)item * MAXQ * QSTATE * 64;
  if (w < ng) {
    const int g0 = gfirst + w * GQ;
    ChunkState gs, p[GQ];
#pragma unroll
    for (int u = 0; u < GQ; ++u)
      if (g0 + u >= qlo && g0 + u <= qhi) block_get(p[u], src + (g0 + u - qlo) * QSTATE * 64, hb, lane);
    state_empty(gs);
#pragma unroll
    for (int u = 0; u < GQ; ++u)
      if (g0 + u >= qlo && g0 + u <= qhi) fold(gs, p[u], 1);
    gst[w][lane] = gs.m;
    gst[w][64 + lane] = gs.l;
#pragma unroll
    for (int j = 0; j < 4; ++j) gst[w][(2 + j) * 64 + lane] = gs.o[0][j];
  }
  __syncthreads();
  if (w != 0) return;
  ChunkState run, gs;
  state_empty(run);
  state_empty(gs);
  for (int k = 0; k < ng; ++k) {
    gs.m = gst[k][lane];
    gs.l = gst[k][64 + lane];
#pragma unroll
    for (int j = 0; j < 4; ++j) gs.o[0][j] = gst[k][(2 + j) * 64 + lane];
    fold(run, gs, 1);
  }
  block_store<PO>(a, it, run, hb, lane);
}

// Windows of one quad: a workgroup per item, one wave per chunk; wave hb then folds the chunks of
// head-dimension block hb, takes the (one) quad through the group's fold and the last one, and
// writes the output, so that no second kernel is needed.  A pass of 64 BF16 streams of 250 tokens: 6.6 us
// a layer in place of 6.3 + 3.0 and the gap between two launches (64 streams' decode 245 to 220 ms).
// Longer windows stay with two kernels: 16 waves and 4 quads in one workgroup, with the partials in
// 98 KB of LDS, took 12.8 us for one BF16 row after 700 tokens where the two take 11.5.
template <int PA, int PO>
__global__ __launch_bounds__(256) void attention_item_kernel(const AttnArgs a) {
  __shared__ float part[QCH][QSTATE * 64];
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const AttnItem it = a.items[blockIdx.x];
  const int ch = (it.c_lo / QCH) * QCH + w;
  const AttnCol c = attn_col(a, it, col);
  if (ch >= it.c_lo && ch <= it.c_hi) {
    QFrag<PA> q;
    load_q<PA>(q, a, c, grp);
    state_put(part[w], chunk_partial<PA>(a, it, c, q, ch, col, grp), lane);
  }
  __syncthreads();
  if (w >= a.hd / 16) return;
  ChunkState run, gs, qs, p;
  state_empty(run);
  state_empty(gs);
  state_empty(qs);
  state_empty(p);
  for (int k = 0; k < QCH; ++k) {
    if (ch - w + k < it.c_lo || ch - w + k > it.c_hi) continue;
    block_get(p, part[k], w, lane);
    fold(qs, p, 1);
  }
  fold(gs, qs, 1);
  fold(run, gs, 1);
  block_store<PO>(a, it, run, w, lane);
}

// Few items, FP32 (decode): the quad kernel's work spread over a workgroup per chunk, so that each
// chunk's MFMA chains run on four SIMDs instead of one.  Wave w runs the score chain of key
// block w, the four blocks' scores meet in LDS, every wave takes the chunk's softmax (the same
// code, the same bits), and wave w runs the P*V chain of head-dimension block w.  A wave's 16 K rows
// and 16 V^T rows arrive as whole rows, 1 KB an instruction (in the MFMA layout an instruction asks for
// 16 bytes of each of 64 lines, and the vector cache takes a line a cycle), and turn in LDS of the
// wave's own, their 16-byte units XORed with the row.  The chunk states go to memory for
// attention_chunk_fold_kernel: handed over inside this kernel instead, by device-scope stores and a
// counter a quad, they cost two more round trips to the coherence point than a wider fold costs.  One
// FP32 row after 1,200 tokens, both kernels: 13.4 us a layer with the handover, 12.1 without; the
// chain is the bound (item, K and V, 16 + 16 dependent MFMAs, states, folds), not the 1.8 MB of keys.
constexpr int kChunkItems = 24;  // largest item count of the chunk-parallel path
constexpr int CST = 6;           // floats per lane of one wave's chunk state: m, l, o[4]

__device__ __forceinline__ float* chunk_slot(const AttnArgs& a, int item, int qi, int cw, int w) {
  return a.ws + ((((size_t)item * MAXQ + qi) * QCH + cw) * 4 + w) * CST * 64;
}

__global__ __launch_bounds__(256) void attention_chunk_kernel(const AttnArgs a) {
  __shared__ v4f s_kv[4][2][16 * 16];  // [wave][K, V^T][row * 16 + (unit ^ row)]
  __shared__ float s_st[4][4][64];     // scores [key block][element][lane]
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int cw = blockIdx.x, item = blockIdx.y, qi = blockIdx.z;
  const AttnItem it = a.items[item];
  const int q0 = (it.c_lo / QCH + qi) * QCH, ch = q0 + cw;
  if (ch < it.c_lo || ch > it.c_hi) return;  // not a chunk of the item (the fold skips it)
  const int hd = a.hd, nhb = hd / 16, g = a.Hq / a.Hk;
  const float* Kc = static_cast<const float*>(a.k_cache);
  const float* Vt = static_cast<const float*>(a.vt_cache);
  const long long sbase = (long long)it.stream * a.kv_stride + (long long)it.kvh * a.ring * hd;
  const int key0 = ch * KCH;
  int base = it.slot_lo + (ch - it.c_lo) * KCH;
  while (base >= a.ring) base -= a.ring;
  // row 4 e + grp of the wave's K and V^T rows, unit col (loads clamped into the head's rows and
  // masked afterwards, as in chunk_partial): key chunk_key(w, row), head entry 16 w + row
  v4f kr[4], vr[4];
  {
    const int kc = min(4 * col, hd - 4);
    int vs = base + 4 * col;
    vs = vs >= a.ring ? vs - a.ring : vs;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int ks = base + 16 * e + 4 * w + grp;
      ks = ks >= a.ring ? ks - a.ring : ks;
      kr[e] = *reinterpret_cast<const v4f*>(Kc + sbase + (long long)ks * hd + kc);
    }
    const int d0 = 16 * min(w, nhb - 1) + grp;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      vr[e] = *reinterpret_cast<const v4f*>(Vt + sbase + (long long)(d0 + 4 * e) * a.ring + vs);
  }
  const AttnCol c = attn_col(a, it, col);
  QFrag<P_F32> q;
  load_q<P_F32>(q, a, c, grp);
  __builtin_amdgcn_sched_barrier(0);  // every load above is issued before the first use
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = 4 * e + grp;
    s_kv[w][0][r * 16 + (col ^ r)] = 4 * col < hd ? kr[e] : zero;
    s_kv[w][1][r * 16 + (col ^ r)] = w < nhb ? vr[e] : zero;
  }
  // the wave reads what its own lanes wrote: LDS serves a wave's accesses in order
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  v4f kf[4], vf[4];
#pragma unroll
  for (int qd = 0; qd < 4; ++qd) kf[qd] = s_kv[w][0][col * 16 + ((4 * grp + qd) ^ col)];
#pragma unroll
  for (int b = 0; b < 4; ++b) vf[b] = s_kv[w][1][col * 16 + ((4 * grp + b) ^ col)];
  v4f sw = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < HDMAX / 4; ++s)
    sw = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[s >> 2][s & 3], q.f[s], sw, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) s_st[w][j][lane] = sw[j];
  __syncthreads();
  v4f st[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int j = 0; j < 4; ++j) st[b][j] = s_st[b][j][lane];
  ChunkState r;
  state_empty(r);
  chunk_softmax(st, a, c, key0, grp, chunk_inside(it, g, key0), r.m, r.l);
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      r.o[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[b][j], st[b][j], r.o[0], 0, 0, 0);
  float* dst = chunk_slot(a, item, qi, cw, w) + lane;
  dst[0] = r.m;
  dst[64] = r.l;
#pragma unroll
  for (int j = 0; j < 4; ++j) dst[(2 + j) * 64] = r.o[0][j];
}

// The chunk kernel's states -> quads -> groups -> output, one workgroup per (item, head-dimension
// block hb).  Wave w folds the chunks of the item's w-th quad (their states loaded together), the
// first waves then fold the quads of a group each and wave 0 the groups: the other kernels' folds
// in their order.
__global__ __launch_bounds__(64 * MAXQ) void attention_chunk_fold_kernel(const AttnArgs a) {
  __shared__ float qst[MAXQ][CST * 64];
  __shared__ float gst[FOLD_WAVES][CST * 64];
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int item = blockIdx.x, hb = blockIdx.y;
  const AttnItem it = a.items[item];
  const int qlo = it.c_lo / QCH, qhi = it.c_hi / QCH, gfirst = (qlo / GQ) * GQ;
  const int ng = (qhi - gfirst) / GQ + 1;  // <= FOLD_WAVES: qhi - qlo < MAXQ
  auto get = [&](ChunkState& st, const float* p) {
    st.m = p[lane];
    st.l = p[64 + lane];
#pragma unroll
    for (int j = 0; j < 4; ++j) st.o[0][j] = p[(2 + j) * 64 + lane];
  };
  auto put = [&](float* p, const ChunkState& st) {
    p[lane] = st.m;
    p[64 + lane] = st.l;
#pragma unroll
    for (int j = 0; j < 4; ++j) p[(2 + j) * 64 + lane] = st.o[0][j];
  };
  if (qlo + w <= qhi) {
    const int q0 = (qlo + w) * QCH;
    ChunkState qs, p[QCH];
    // (a slot outside the item is inside the workspace, and is not folded)
#pragma unroll
    for (int k = 0; k < QCH; ++k) get(p[k], chunk_slot(a, item, w, k, hb));
    state_empty(qs);
#pragma unroll
    for (int k = 0; k < QCH; ++k)
      if (q0 + k >= it.c_lo && q0 + k <= it.c_hi) fold(qs, p[k], 1);
    put(qst[w], qs);
  }
  __syncthreads();
  // waves 0 .. ng - 1 exist: an item of one quad has one group, of q quads at most q
  ChunkState run, gs;
  state_empty(run);
  state_empty(gs);
  ChunkState t;
  state_empty(t);
  if (w < ng) {
    const int g0 = gfirst + w * GQ;
    for (int u = max(g0, qlo); u <= min(g0 + GQ - 1, qhi); ++u) {
      get(t, qst[u - qlo]);
      fold(gs, t, 1);
    }
    put(gst[w], gs);
  }
  __syncthreads();
  if (w != 0) return;
  for (int k = 0; k < ng; ++k) {
    get(t, gst[k]);
    fold(run, t, 1);
  }
  block_store<P_F32>(a, it, run, hb, lane);
}

// ---- small kernels ------------------------------------------------------------------------

// x[r] = E[tok], the block sums of squares of the row, and y[r] = quantise(x[r] * gain)
template <int P>
__global__ void embed_kernel(const float* __restrict__ E, const RowMeta* __restrict__ rows, int n,
                             int d, float* __restrict__ x, float* __restrict__ ssq, void* y,
                             const float* __restrict__ gain, float inv_scale, float* y_amax) {
  const int r = blockIdx.x;
  if (r >= n) return;
  const int lane = threadIdx.x, c = lane & 15, q = lane >> 4;
  const int nb = d / 16;
  const long long t = rows[r].tok;
  float ymax = 0.f;
  for (int b0 = 0; b0 < nb; b0 += 4) {
    const int b = b0 + q;
    const bool ok = b < nb;
    const int k = 16 * b + c;
    const float v = ok ? E[t * d + k] : 0.f;
    const float sq = block_ssq16(v);
    if (ok) {
      x[(long long)r * d + k] = v;
      if (c == 0) ssq[(long long)r * nb + b] = sq;
      const float yv = v * gain[k];
      PT<P>::store(y, (long long)r * d + k, yv, inv_scale);
      ymax = fmaxf(ymax, fabsf(yv));
    }
  }
  amax_flush(y_amax, ymax, lane);
}

template <int P>
__global__ void convert_kernel(const float* __restrict__ src, void* __restrict__ dst, long long n,
                               float inv_scale) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    PT<P>::store(dst, i, src[i], inv_scale);
}

// ---- launchers ------------------------------------------------------------------------------

constexpr size_t kSplitLdsMax = 144 * 1024;  // of the 160 KiB LDS of a gfx950 CU

template <int P, int AM, int EPI, int MB, bool kStage>
static void launch_split(dim3 grid, int waves, size_t lds, const GemmArgs& a, hipStream_t s) {
  static bool raised = false;  // allow more than the default 64 KiB of dynamic LDS, once
  if (!raised) {
    NC_HIP(hipFuncSetAttribute(
        reinterpret_cast<const void*>(&gemm_split_kernel<P, AM, EPI, MB, kStage>),
        hipFuncAttributeMaxDynamicSharedMemorySize, int(kSplitLdsMax)));
    raised = true;
  }
  // a normed GEMM's row scales have a wave of their own
  const int extra = AM == A_NORM ? 1 : 0, nw = std::min(waves, SPLIT_WAVES - extra);
  hipLaunchKernelGGL((gemm_split_kernel<P, AM, EPI, MB, kStage>), grid, dim3(64 * (nw + extra)),
                     lds, s, a, nw);
}

static int split_groups(const GemmArgs& a, int prec, int epi, int mb) {
  const int w = 16 * group_size(prec, epi, mb);
  return (a.N + w - 1) / w;
}

// Row blocks (16 rows each) per workgroup: GEMMs with few column groups cut M finer, so that
// more workgroups share the work and each one's chain of loads, MFMAs and epilogue is shorter.
static int split_mb(const GemmArgs& a, int prec, int epi) {
  const int ngroups = split_groups(a, prec, epi, SPLIT_ROWS / 16);
  const int cap = ngroups < 64 ? 1 : ngroups < 256 ? 2 : SPLIT_ROWS / 16;
  return std::min((a.M + 15) / 16, cap);
}

static int split_parts(const GemmArgs& a) { return (a.K + KP - 1) / KP; }

static size_t split_lds(const GemmArgs& a, int prec, int epi, int mb, bool stage) {
  return (size_t(split_parts(a)) * split_slot(prec, epi, mb, stage) + SPLIT_ROWS) * sizeof(float);
}

// The shapes that are accepted: S partials of mb 16 x 16 blocks per column block, for the pair of
// blocks that an epilogue works on, with the rows' block sums, in kSplitLdsMax.  (The kernel needs
// no more than that.)
static bool split_fits(const GemmArgs& a, int epi, int mb) {
  const int nb16 = a.K / 16, pair = epi == E_RESID || (epi == E_QKV && a.hd == 16) ? 1 : 2;
  const size_t ssq = epi != E_RESID && nb16 <= 64 ? size_t(mb) * 16 * nb16 : 0;
  return (size_t(split_parts(a)) * pair * mb * 256 + SPLIT_ROWS + ssq) * sizeof(float) <=
         kSplitLdsMax;
}

template <int P, int AM, int EPI, int MB>
static void gemm_split_mb(const GemmArgs& a, hipStream_t s, int waves) {
  const dim3 grid(split_groups(a, P, EPI, MB), (a.M + 16 * MB - 1) / (16 * MB));
  if constexpr (P == P_F32 && MB <= 2) {  // (more row blocks would spill)
    const size_t lds = split_lds(a, P, EPI, MB, true);
    if (lds <= kSplitLdsMax) return launch_split<P, AM, EPI, MB, true>(grid, waves, lds, a, s);
  }
  launch_split<P, AM, EPI, MB, false>(grid, waves, split_lds(a, P, EPI, MB, false), a, s);
}

template <int P, int AM, int EPI>
static void gemm_split(const GemmArgs& a, hipStream_t s, int mb, int waves) {
  switch (mb) {
    case 1: return gemm_split_mb<P, AM, EPI, 1>(a, s, waves);
    case 2: return gemm_split_mb<P, AM, EPI, 2>(a, s, waves);
    case 3: return gemm_split_mb<P, AM, EPI, 3>(a, s, waves);
    default: return gemm_split_mb<P, AM, EPI, 4>(a, s, waves);
  }
}

void launch_row_rms(const GemmArgs& a, float* inv, hipStream_t s) {
  if (a.M <= 0) return;
  hipLaunchKernelGGL(row_rms_kernel, dim3((a.M + 255) / 256), dim3(256), 0, s, a, inv);
  NC_HIP(hipGetLastError());
}

static bool wide_ok(int prec, int epi, const GemmArgs& a) {
  return prec != P_F32 && (epi != E_QKV || a.hd == 32 || a.hd == 64);
}

static bool tile_valid(int prec, int epi, const GemmArgs& a, const GemmTile& t) {
  switch (t.kind) {
    case T_AUTO: return true;
    case T_SPLIT:
      return t.mb >= 1 && t.mb <= SPLIT_ROWS / 16 && t.waves >= 1 && t.waves <= SPLIT_WAVES &&
             split_fits(a, epi, t.mb);
    case T_TILE_S:
    case T_TILE_M: return true;
    case T_WIDE: return wide_ok(prec, epi, a);
    default: return false;
  }
}

// The fixed rule used when no measured choice is given, from the number of tiles that a shape gives
// (256 CUs of four SIMDs).  Times per launch at the 135M shape, microseconds:
//  - split up to 32 rows, and while 64 x 32 tiles are fewer than 128 (half the CUs): FP32 QKV at 256
//    rows (120 tiles) 16.8 against 22.4, gate/up at 128 rows (192 tiles) 22.1 against 18.5; output
//    layer at 64 rows (1,536 tiles) 92 against 53.
//  - then 64 x 32 tiles while larger ones leave SIMDs idle: FP32 O projection at 512 / 4,096 rows
//    16.3 / 43.3 against 23.5 / 52.6 with 64 x 64; BF16 at 1,024 rows 12.1 against 14.0, but at 4,096
//    rows (576 tiles of 64 x 64) 21.7 against 20.2.
//  - 128 x 128 in BF16 / FP8 from 384 tiles on: gate/up at 4,096 rows 45.7 against 55.2, output layer
//    at 512 rows 73 against 102; for the residual GEMMs, whose N = 576 fills 4.5 of 5 column tiles,
//    from 1,024 on (down projection at 16,384 rows, 640 tiles, 93 against 77; at 32,768 rows
//    146 against 157).
static GemmTile default_tile(int prec, int epi, const GemmArgs& a) {
  const int S = split_parts(a);
  const GemmTile sp{T_SPLIT, split_mb(a, prec, epi), S < SPLIT_WAVES ? S : SPLIT_WAVES};
  auto tiles = [&](long long bm, long long bn) {
    return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn);
  };
  if ((a.M <= 32 || tiles(64, 32) < 128) && split_fits(a, epi, sp.mb)) return sp;
  if (tiles(128, 128) >= (epi == E_RESID ? 1024 : 384) && wide_ok(prec, epi, a))
    return GemmTile{T_WIDE, 0, 0};
  return GemmTile{tiles(64, 64) < (prec == P_F32 ? 1024 : 512) ? T_TILE_S : T_TILE_M, 0, 0};
}

bool gemm_tile_fits(int prec, int epi, const GemmArgs& a, const GemmTile& t) {
  return tile_valid(prec, epi, a, t);
}

std::vector<GemmTile> gemm_candidates(int prec, int epi, const GemmArgs& a) {
  std::vector<GemmTile> out;
  const int S = split_parts(a);
  const int wmax = S < SPLIT_WAVES ? S : SPLIT_WAVES;
  if (a.M <= 1024) {
    const int mbmax = std::min((a.M + 15) / 16, SPLIT_ROWS / 16);
    for (int mb = 1; mb <= mbmax; ++mb) {
      int prev = 0;
      for (int div = 1; div <= 4; div *= 2) {
        const int w = (wmax + div - 1) / div;
        const GemmTile t{T_SPLIT, mb, w};
        if (w != prev && tile_valid(prec, epi, a, t)) out.push_back(t);
        prev = w;
      }
    }
  }
  out.push_back(GemmTile{T_TILE_S, 0, 0});
  out.push_back(GemmTile{T_TILE_M, 0, 0});
  if (wide_ok(prec, epi, a)) out.push_back(GemmTile{T_WIDE, 0, 0});
  return out;
}

template <int P, int AM, int EPI>
static void gemm_shape(const GemmArgs& a, hipStream_t s, GemmTile t) {
  if (t.kind == T_AUTO) t = default_tile(P, EPI, a);
  if (t.kind == T_SPLIT) return gemm_split<P, AM, EPI>(a, s, t.mb, t.waves);
  if constexpr (P != P_F32) {
    if (t.kind == T_WIDE) return gemm_tile<P, AM, EPI, 4, 4, 2, 2, false>(a, s);
  }
  if (t.kind == T_TILE_S)
    gemm_tile<P, AM, EPI, 1, 2, 4, 1, true>(a, s);
  else
    gemm_tile<P, AM, EPI, 2, 2, 2, 2, true>(a, s);
}

template <int P>
static void gemm_prec(int amode, int epi, const GemmArgs& a, hipStream_t s, GemmTile t) {
  if (amode == A_NORM) {
    switch (epi) {
      case E_STORE: return gemm_shape<P, A_NORM, E_STORE>(a, s, t);
      case E_GLU: return gemm_shape<P, A_NORM, E_GLU>(a, s, t);
      case E_QKV: return gemm_shape<P, A_NORM, E_QKV>(a, s, t);
      default: break;
    }
  } else if (epi == E_RESID) {
    return gemm_shape<P, A_DIRECT, E_RESID>(a, s, t);
  }
  fail(NC_E_INVALID, "unsupported GEMM variant");
}

void launch_gemm(int prec, int amode, int epi, const GemmArgs& a, hipStream_t s, GemmTile t) {
  if (a.M <= 0) return;
  NC_CHECK(a.K % 16 == 0, NC_E_INVALID, "GEMM K must be a multiple of 16");
  if (epi == E_QKV) NC_CHECK(64 % a.hd == 0, NC_E_INVALID, "head_dim must divide 64");
  if (epi == E_GLU) NC_CHECK(a.N % 32 == 0, NC_E_INVALID, "d_ffn must be a multiple of 16");
  if (amode == A_NORM) NC_CHECK(a.ssq || a.inv, NC_E_INVALID, "normed GEMM needs row statistics");
  NC_CHECK(!a.a_rows || epi == E_STORE, NC_E_INVALID, "only the output layer gathers A rows");
  if (epi == E_RESID)
    NC_CHECK(a.N % 16 == 0 && (!a.y_out || a.y_gain), NC_E_INVALID, "bad residual epilogue");
  NC_CHECK(tile_valid(prec, epi, a, t), NC_E_INVALID, "GEMM launch shape does not fit this GEMM");
  if (prec == P_F32)
    gemm_prec<P_F32>(amode, epi, a, s, t);
  else if (prec == P_BF16)
    gemm_prec<P_BF16>(amode, epi, a, s, t);
  else
    gemm_prec<P_FP8>(amode, epi, a, s, t);
  NC_HIP(hipGetLastError());
}

// Quads that consecutive items of one stream can span: their keys run from the window start of the
// first query to the last query, at most ctx_len + 16 items - 1 keys (a window holds at most
// ctx_len keys, an item at most 16 query positions), i.e. at most nch chunks at any alignment.
static int attention_quads(int ctx_len, int items = 1) {
  const int nch = (ctx_len + 16 * items - 1 + KCH - 1) / KCH + 1;
  return (nch - 1 + QCH - 1) / QCH + 1;
}

template <int PA, int PO>
static void attn_go(const AttnArgs& a, bool parallel, hipStream_t s) {
  // Shared staging needs 2 items a group to pay (FP32, 64 streams: of 4 rows, one item a group,
  // 15.7 us alone and 23.5 grouped; of 6 rows, two, 36.6 and 28.2) and work for the chip (one BF16
  // stream after 1,200 tokens: 18 items 13.7 and 14.7, 27 items 15.1 and 14.3).  FP32 chunk by chunk is
  // the shorter chain for few items also where one quad is the whole window (one row after 200 tokens:
  // 11.1 us, and 12.5 an item a workgroup).
  // From 1,024 items on (not parallel) a workgroup takes a group over its whole window whatever the
  // group's size: where groups are one item (decode of over 340 streams, three kv heads) three of its
  // waves only stage, but the chip is full.  Against four items a workgroup, each wave reading keys
  // for itself, on average over a decode of 250 tokens: BF16 400 / 1,000 streams 18.2 / 36.2 us and
  // 20.6 / 35.5, FP32 36.1 / 77.0 and 41.9 / 70.5; 700 tokens, 400 streams, 33.2 and 39.9, 67.2 and 80.5.
  const bool grouped = a.n_items > kChunkItems && a.n_items >= 2 * a.n_groups;
  if (parallel) {
    const int nq = std::min(a.quads, attention_quads(a.ctx_len));
    if (PA == P_F32 && a.n_items <= kChunkItems) {
      hipLaunchKernelGGL(attention_chunk_kernel, dim3(QCH, a.n_items, nq), dim3(256), 0, s, a);
      hipLaunchKernelGGL(attention_chunk_fold_kernel, dim3(a.n_items, a.hd / 16), dim3(64 * nq), 0,
                         s, a);
      return;
    }
    if (!grouped && nq == 1) {
      hipLaunchKernelGGL((attention_item_kernel<PA, PO>), dim3(a.n_items), dim3(256), 0, s, a);
      return;
    }
    if (grouped) {
      hipLaunchKernelGGL((a.hd == HDMAX ? attention_group_kernel<PA, PO, true, true>
                                        : attention_group_kernel<PA, PO, true, false>),
                         dim3(a.n_groups * std::min(a.quads, attention_quads(a.ctx_len, GI))),
                         dim3(256), 0, s, a);
    } else {
      hipLaunchKernelGGL((attention_quad_kernel<PA>), dim3(a.n_items * nq), dim3(256), 0, s, a);
    }
    hipLaunchKernelGGL((attention_fold_kernel<PO>), dim3(a.n_items, a.hd / 16),
                       dim3(64 * FOLD_WAVES), 0, s, a);
  } else {
    hipLaunchKernelGGL((a.hd == HDMAX ? attention_group_kernel<PA, PO, false, true>
                                      : attention_group_kernel<PA, PO, false, false>),
                       dim3(a.n_groups), dim3(256), 0, s, a);
  }
}

size_t attention_ws_bytes(int n_items) {
  const size_t quads = size_t(n_items) * MAXQ * QSTATE * 64;
  const size_t chunks = n_items <= kChunkItems ? size_t(n_items) * MAXQ * QCH * 4 * CST * 64 : 0;
  return std::max(quads, chunks) * sizeof(float);
}

// parallel: the work of an item or group is spread over workgroups, with a fold kernel (few items);
// otherwise a workgroup per group of items (prefill).  Both produce the same bits.
void launch_attention(int prec_att, int prec_out, const AttnArgs& a, bool parallel,
                      hipStream_t s) {
  if (a.n_items <= 0) return;
  NC_CHECK(a.hd % 16 == 0 && a.hd <= HDMAX, NC_E_INVALID, "head_dim must be 16..64, x16");
  NC_CHECK(attention_quads(a.ctx_len) <= MAXQ, NC_E_INVALID, "context window too large");
  NC_CHECK(a.ring % 16 == 0 && a.ring >= KCH, NC_E_INVALID,
           "ring must be a multiple of 16 and hold a chunk");
  NC_CHECK(a.n_groups > 0 && a.n_groups <= a.n_items, NC_E_INVALID, "attention groups");
  if (parallel)
    NC_CHECK(a.ws && a.ws_bytes >= attention_ws_bytes(a.n_items), NC_E_INVALID,
             "attention workspace too small");
  if (prec_att == P_F32) {
    NC_CHECK(prec_out == P_F32, NC_E_INVALID, "fp32 attention feeds fp32 GEMMs");
    attn_go<P_F32, P_F32>(a, parallel, s);
  } else if (prec_out == P_BF16) {
    attn_go<P_BF16, P_BF16>(a, parallel, s);
  } else {
    attn_go<P_BF16, P_FP8>(a, parallel, s);
  }
  NC_HIP(hipGetLastError());
}

void launch_embed(const float* E, const RowMeta* rows, int n, int d, float* x, float* ssq,
                  void* y, const float* gain, int prec, float inv_scale, float* y_amax,
                  hipStream_t s) {
  if (n <= 0) return;
  NC_CHECK(d % 16 == 0, NC_E_INVALID, "d_model must be a multiple of 16");
  if (prec == P_F32)
    hipLaunchKernelGGL(embed_kernel<P_F32>, dim3(n), dim3(64), 0, s, E, rows, n, d, x, ssq, y,
                       gain, inv_scale, y_amax);
  else if (prec == P_BF16)
    hipLaunchKernelGGL(embed_kernel<P_BF16>, dim3(n), dim3(64), 0, s, E, rows, n, d, x, ssq, y,
                       gain, inv_scale, y_amax);
  else
    hipLaunchKernelGGL(embed_kernel<P_FP8>, dim3(n), dim3(64), 0, s, E, rows, n, d, x, ssq, y,
                       gain, inv_scale, y_amax);
  NC_HIP(hipGetLastError());
}

void launch_convert(const float* src, void* dst, long long n, int prec, float inv_scale,
                    hipStream_t s) {
  const int blocks = int(std::min<long long>((n + 255) / 256, 65536));
  if (prec == P_F32)
    hipLaunchKernelGGL(convert_kernel<P_F32>, dim3(blocks), dim3(256), 0, s, src, dst, n, inv_scale);
  else if (prec == P_BF16)
    hipLaunchKernelGGL(convert_kernel<P_BF16>, dim3(blocks), dim3(256), 0, s, src, dst, n,
                       inv_scale);
  else
    hipLaunchKernelGGL(convert_kernel<P_FP8>, dim3(blocks), dim3(256), 0, s, src, dst, n,
                       inv_scale);
  NC_HIP(hipGetLastError());
}

}  // namespace nc
