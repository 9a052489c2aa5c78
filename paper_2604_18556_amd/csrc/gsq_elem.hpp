// What the elementwise kernels of both precisions share: the state's layout, its accesses, the
// relaxed sample of one coordinate and the optimiser's update of one parameter.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "gsq_device.hpp"
#include "gsq_internal.h"

namespace gsq {
namespace {

constexpr int kBlock = 256;   // 4 wavefronts
constexpr int kCols = 256;    // columns per wavefront

template <bool kF64>
using Real = typename std::conditional<kF64, double, float>::type;

__device__ __forceinline__ float f4get(const float4& v, int q) {
  return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w;
}

__device__ __forceinline__ void f4set(float4& v, int q, float x) {
  if (q == 0) v.x = x; else if (q == 1) v.y = x; else if (q == 2) v.z = x; else v.w = x;
}

__device__ __forceinline__ bool finite4(const float4& v) {
  return __builtin_isfinite(v.x) && __builtin_isfinite(v.y) && __builtin_isfinite(v.z) &&
         __builtin_isfinite(v.w);
}

// Float offset of logit (or moment) k of coordinate e in the blocked state layout.  Four
// consecutive coordinates from a multiple of 4 lie in one block, so a lane's float4 is
// contiguous and 16-byte aligned.
__device__ __forceinline__ int64_t state_off(int64_t e, int k, int K) {
  return (e / kStateBlock) * (K * kStateBlock) + (int64_t)k * kStateBlock + (e % kStateBlock);
}

// Streaming accesses of the state and G: each is touched once per launch, so the loads and
// stores carry the non-temporal hint (no cache allocation).  On the backward's access pattern
// this moves 14-21 % more bytes per second than plain accesses.  W and R keep plain accesses:
// R is read next by the contraction, and the hint on them measured slightly slower.
__device__ __forceinline__ float4 ld_stream(const float* p) {
  float4 v;
  v.x = __builtin_nontemporal_load(p);
  v.y = __builtin_nontemporal_load(p + 1);
  v.z = __builtin_nontemporal_load(p + 2);
  v.w = __builtin_nontemporal_load(p + 3);
  return v;
}

__device__ __forceinline__ void st_stream(float* p, const float4& v) {
  __builtin_nontemporal_store(v.x, p);
  __builtin_nontemporal_store(v.y, p + 1);
  __builtin_nontemporal_store(v.z, p + 2);
  __builtin_nontemporal_store(v.w, p + 3);
}

__device__ __forceinline__ void load_w4(const void* W, int w_bf16, int64_t e, float (&w)[4]) {
  if (w_bf16) {
    const uint2 u = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(W) + e);
    w[0] = __uint_as_float(u.x << 16);
    w[1] = __uint_as_float(u.x & 0xFFFF0000u);
    w[2] = __uint_as_float(u.y << 16);
    w[3] = __uint_as_float(u.y & 0xFFFF0000u);
  } else {
    const float4 v = *reinterpret_cast<const float4*>(static_cast<const float*>(W) + e);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  }
}

// R is stored in the contraction's padded layout: row (b, o) at (b*Opad + o)*Ipad.
__device__ __forceinline__ int64_t padded_index(const ElemArgs& a, int64_t row, int64_t col) {
  const int64_t b = row / a.O;
  return (b * a.Opad + (row - b * a.O)) * a.Ipad + col;
}

template <bool kF64>
__device__ __forceinline__ void store_r4(void* R, int64_t idx, const float (&r)[4]) {
  if constexpr (kF64) {
    *reinterpret_cast<float4*>(static_cast<float*>(R) + idx) = make_float4(r[0], r[1], r[2], r[3]);
  } else {
    uint2 u;
    u.x = (uint32_t)bf16_rne(r[0]) | ((uint32_t)bf16_rne(r[1]) << 16);
    u.y = (uint32_t)bf16_rne(r[2]) | ((uint32_t)bf16_rne(r[3]) << 16);
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(R) + idx) = u;
  }
}

// R = W - s v before the contraction's rounding; the forward, the fused next sample and the
// backward's loss all form it with this one expression.
template <bool kF64>
__device__ __forceinline__ float residual(float w, Real<kF64> s, Real<kF64> v) {
  return (float)((Real<kF64>)w - s * v);
}

// fp32 path: hardware exp2 / reciprocal / square root (about 1 ulp); fp64 path: about 1 ulp of fp64.
constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// One coordinate's relaxed sample (Alg. 1): p = softmax((kappa l + g) / tau), with the
// largest perturbed logit r subtracted first.  vp = sum_k p_k (c_k - c_r), so that the soft
// level v = c_r + vp and c_k - v = (c_k - c_r) - vp keep full relative accuracy when one
// level holds almost all the mass.  c holds the values the K logits stand for.
template <int K, bool kF64>
__device__ __forceinline__ void soft_sample(const float (&l)[K], const float (&c)[K], const float (&g)[K],
                                            float kappa, Real<kF64> inv_tau, Real<kF64> (&p)[K],
                                            Real<kF64>& vp, Real<kF64>& cr) {
  using T = Real<kF64>;
  T b[K];
#pragma unroll
  for (int k = 0; k < K; ++k) b[k] = (T)kappa * (T)l[k] + (T)g[k];
  T bmax = b[0];
  cr = (T)c[0];
#pragma unroll
  for (int k = 1; k < K; ++k) {
    if (b[k] > bmax) { bmax = b[k]; cr = (T)c[k]; }
  }
  T z = 0;
  if constexpr (kF64) {
#pragma unroll
    for (int k = 0; k < K; ++k) { p[k] = exp_nonpos((b[k] - bmax) * inv_tau); z += p[k]; }
  } else {
    const float s2 = inv_tau * kLog2e;   // exp(a) = exp2(a log2 e)
#pragma unroll
    for (int k = 0; k < K; ++k) { p[k] = __builtin_amdgcn_exp2f((b[k] - bmax) * s2); z += p[k]; }
  }
  T rz;
  if constexpr (kF64) rz = T(1) / z; else rz = fast_rcp(z);
  vp = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) { p[k] *= rz; vp += p[k] * ((T)c[k] - cr); }
}

// Two-value relaxation with logits {-l, l} (§3): p1 = softmax over (-kappa l + g0,
// kappa l + g1) / tau, i.e. a sigmoid of (2 kappa l + g1 - g0) / tau.  The pair's noise dn is
// drawn as the difference g1 - g0 itself (a logistic value).  The smaller probability is formed
// as e / (1 + e) with e = exp(-|a|), never as 1 - p.
template <bool kF64>
__device__ __forceinline__ void pair_probs(float l, float dn, float kappa, Real<kF64> inv_tau,
                                           Real<kF64>& p0, Real<kF64>& p1) {
  using T = Real<kF64>;
  const T d = (T)2 * (T)kappa * (T)l + (T)dn;
  const T a = d * inv_tau;
  T e, big;
  if constexpr (kF64) {
    e = exp_nonpos(-fabs(a));
    big = T(1) / (T(1) + e);
  } else {
    e = __builtin_amdgcn_exp2f(-fabsf(a) * kLog2e);
    big = fast_rcp(1.f + e);
  }
  const T small = e * big;
  p1 = a >= T(0) ? big : small;
  p0 = a >= T(0) ? small : big;
}

// Noise values per coordinate and draw: one Gumbel value per logit of a categorical, or one
// logistic value per binary pair (the mask's, then the sign's).
template <int K, int kMode>
constexpr int noise_count() { return kMode == GSQ_RELAX_TERNARY ? 2 : K; }

template <int kMode>
constexpr int noise_kind() { return kMode == GSQ_RELAX_TERNARY ? kLogistic : kGumbel; }

// One coordinate's relaxed sample in any relaxation: the soft level v (W_hat = s v) and
// jac[k] = (tau / kappa) dv/dl_k.
//   GRID / SHIFT: v = sum_k p_k c_k, jac[k] = p_k (c_k - v).
//   TERNARY: v = m~ b~ with m~ = p1 of the mask pair (values 0, 1) and b~ = p1 - p0 of the
//   sign pair (values -1, 1); a pair with logits {-l, l} and values (y0, y1) has
//   (tau / kappa) dy/dl = 2 p0 p1 (y1 - y0), so jac = (2 p0 p1 b~, 4 p0 p1 m~).
template <int K, int Z, bool kF64, int kMode>
__device__ __forceinline__ void coord_sample(const float (&l)[K], const float (&c)[K], const float (&g)[Z],
                                             float kappa, Real<kF64> inv_tau, Real<kF64>& v,
                                             Real<kF64> (&jac)[K]) {
  using T = Real<kF64>;
  if constexpr (kMode == GSQ_RELAX_TERNARY) {
    static_assert(K == 2 && Z == 2, "ternary: two logits, one noise value per pair");
    T pm0, pm1, pb0, pb1;
    pair_probs<kF64>(l[0], g[0], kappa, inv_tau, pm0, pm1);
    pair_probs<kF64>(l[1], g[1], kappa, inv_tau, pb0, pb1);
    const T m = pm1, b = pb1 - pb0;
    v = m * b;
    jac[0] = b * (T(2) * pm0 * pm1);
    jac[1] = m * (T(4) * pb0 * pb1);
  } else {
    static_assert(K == Z, "one noise value per logit");
    T p[K], vp, cr;
    soft_sample<K, kF64>(l, c, g, kappa, inv_tau, p, vp, cr);
    v = cr + vp;
#pragma unroll
    for (int k = 0; k < K; ++k) jac[k] = p[k] * (((T)c[k] - cr) - vp);
  }
}

// Local-shift windows in LDS: row j (a grid index) holds the levels of the five shifts around
// it, c[clip(j + k - 2, 0, n - 1)] for k < 5, padded to 8 floats.  Rows past the grid are
// filled like the last one, so a clamped index never reads an unset row.
constexpr int kWinRow = 8;
__device__ __forceinline__ void fill_windows(float* win, const ElemArgs& a) {
  for (int i = threadIdx.x; i < GSQ_MAX_LEVELS * kWinRow; i += blockDim.x) {
    const int j = i / kWinRow, k = i % kWinRow;
    int idx = j + k - 2;
    idx = idx < 0 ? 0 : idx;
    idx = idx > a.n_grid - 1 ? a.n_grid - 1 : idx;
    float v = 0.f;
#pragma unroll
    for (int m = 0; m < GSQ_MAX_LEVELS; ++m) v = (m == idx) ? a.c[m] : v;
    win[i] = k < GSQ_SHIFT_WINDOW ? v : 0.f;
  }
  __syncthreads();
}

// Base indices of the chunk's four coordinates (local shift; one byte each), or 0.
template <int kMode>
__device__ __forceinline__ uint32_t chunk_bases(const ElemArgs& a, int64_t e0) {
  if constexpr (kMode == GSQ_RELAX_SHIFT) return *reinterpret_cast<const uint32_t*>(a.J0 + e0);
  else return 0u;
}

// The values the logits of coordinate q of the chunk stand for: the grid (GRID), or the
// window of its base index read from the LDS table (SHIFT; read where needed rather than
// held in registers).
template <int K, int kMode>
__device__ __forceinline__ void coord_candidates(float (&cand)[K], const ElemArgs& a, const float* win,
                                                 uint32_t j4, int q) {
  if constexpr (kMode == GSQ_RELAX_SHIFT) {
    static_assert(K == GSQ_SHIFT_WINDOW, "five shifts");
    int j = (int)((j4 >> (8 * q)) & 0xFFu);
    j = j < a.n_grid ? j : a.n_grid - 1;          // a corrupt index cannot leave the table
    const float4 lo = *reinterpret_cast<const float4*>(win + j * kWinRow);
    cand[0] = lo.x; cand[1] = lo.y; cand[2] = lo.z; cand[3] = lo.w;
    cand[4] = win[j * kWinRow + 4];
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) cand[k] = a.c[k];
  }
}

// Noise of the thread's chunk of four coordinates (or zeros when sampling is off).
template <int Z, int kMode>
__device__ __forceinline__ void chunk_noise(float (&g)[4][Z], const ElemArgs& a, uint64_t e0,
                                            uint32_t t, uint32_t sample) {
  if (a.noise) {
    draw_chunk<Z, false, noise_kind<kMode>()>(g, a.seed, e0, t, sample);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < Z; ++k) g[q][k] = 0.f;
  }
}

// One parameter's optimiser update.  Adam: bias-corrected (step = lr / (1 - b1^n),
// rbc2 = 1 / sqrt(1 - b2^n)), plus decoupled decay lr wd theta (AdamW).  Lion: the sign of
// b1 m + (1 - b1) d, plus decoupled decay; the moment then moves with b2; v is untouched.
template <bool kF64, bool kLion>
__device__ __forceinline__ void opt_update(Real<kF64> d, Real<kF64>& th, Real<kF64>& m,
                                           Real<kF64>& v, Real<kF64> lr, Real<kF64> step,
                                           Real<kF64> b1, Real<kF64> b2, Real<kF64> omb1,
                                           Real<kF64> omb2, Real<kF64> rbc2, Real<kF64> eps,
                                           Real<kF64> wd) {
  using T = Real<kF64>;
  if constexpr (kLion) {
    const T c = b1 * m + omb1 * d;
    const T sg = (T)((c > T(0)) - (c < T(0)));
    th = th - lr * (sg + wd * th);
    m = b2 * m + omb2 * d;
  } else {
    m = b1 * m + omb1 * d;
    v = b2 * v + omb2 * d * d;
    if constexpr (kF64) th = th - (step * m / (sqrt_f64(v) * rbc2 + eps) + lr * wd * th);
    else th = th - (step * m * fast_rcp(fast_sqrt(v) * rbc2 + eps) + lr * wd * th);
  }
}

}  // namespace
}  // namespace gsq
