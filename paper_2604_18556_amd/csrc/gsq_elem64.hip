// The forward and the backward of the FP32 precision: fp64 arithmetic on the state's fp32 values.
//
// Bound by the fp64 vector units: a logit's step takes four logarithms, two exponentials, a root
// and a division.  One coordinate per lane: with four, as in the other precision, the 8-level
// kernel held 362 registers, ran one wavefront per SIMD and waited for its own chains, and a small
// layer had few wavefronts, each with four coordinates' chains one after the other.  The state's
// accesses of 256 bytes per wavefront are wide enough for it.  A workgroup owns 256 columns of a
// row, so a scale group lies inside it; what crosses its wavefronts goes through LDS in a fixed
// order.  With the short fp64 functions, 1024 x 2048, K = 8: backward 332 -> 206 us, forward
// 109 -> 57; 256 x 256, K = 4: backward 24.5 -> 9.8 us.
#include <hip/hip_runtime.h>

#include "gsq_elem.hpp"

namespace gsq {
namespace {

// Most Philox calls that the Z values of one coordinate lie in.
template <int Z>
constexpr int lane_calls() {
  int most = 0;
  for (int q = 0; q < 4; ++q) {
    const int n = (q * Z % 4 + Z - 1) / 4 + 1;
    most = n > most ? n : most;
  }
  return most;
}

// w moved down by n places where `on`.  Both values are read before one is chosen: of a choice
// between two array elements the compiler makes one between their addresses and keeps the array in
// LDS, 4 to 12 KB per workgroup.  2048 x 256, K = 2: forward 22 -> 9.4 us, backward 32.6 -> 20.9;
// 1024 x 2048, K = 6: 58 -> 47, 174 -> 146.
template <int n, int N>
__device__ __forceinline__ void shift_words(uint32_t (&w)[N], bool on) {
#pragma unroll
  for (int i = 0; i + n < N; ++i) {
    const uint32_t here = w[i], there = w[i + n];
    w[i] = on ? there : here;
  }
}

// Noise of coordinate e: positions (e mod 4) Z .. + Z - 1 of its chunk's stream (or zeros when
// sampling is off).
template <int Z, int kMode>
__device__ __forceinline__ void lane_noise(float (&g)[Z], const ElemArgs& a, uint64_t e, uint32_t t,
                                           uint32_t sample) {
  if (!a.noise) {
#pragma unroll
    for (int k = 0; k < Z; ++k) g[k] = 0.f;
    return;
  }
  constexpr int kCalls = lane_calls<Z>();
  const int f0 = (int)(e & 3) * Z;
  uint32_t w[4 * kCalls];
#pragma unroll
  for (int j = 0; j < kCalls; ++j) {
    const U4 x = noise_words(a.seed, e & ~(uint64_t)3, t, sample * 256u, (uint32_t)((f0 >> 2) + j));
#pragma unroll
    for (int r = 0; r < 4; ++r) w[4 * j + r] = word_of(x, r);
  }
  // the coordinate's first word to w[0]
  if constexpr (Z % 2 != 0) shift_words<1>(w, f0 & 1);
  if constexpr (Z % 4 != 0) shift_words<2>(w, f0 & 2);
#pragma unroll
  for (int k = 0; k < Z; ++k) g[k] = noise_value<noise_kind<kMode>(), true>(w[k]);
}

__device__ __forceinline__ float load_w(const ElemArgs& a, int64_t e) {
  return a.w_bf16 ? bf16_to_f32(static_cast<const uint16_t*>(a.W)[e])
                  : static_cast<const float*>(a.W)[e];
}

// Row of the workgroup, of which there are `cols` per row (split_rows); past the last one: none.  The
// rows and those of a further grid.y fit 31 bits: in 64 the backward takes 1 % more.
__device__ __forceinline__ int lane_row(const ElemArgs& a, int cols) {
  return (int)(blockIdx.y * (uint32_t)a.rows_x + blockIdx.x / (uint32_t)cols);
}

template <int K, int kMode>
__global__ __launch_bounds__(kBlock) void k_forward_f64(ElemArgs a) {
  constexpr int Z = noise_count<K, kMode>();
  __shared__ __align__(16) float win[kMode == GSQ_RELAX_SHIFT ? GSQ_MAX_LEVELS * kWinRow : 4];
  if constexpr (kMode == GSQ_RELAX_SHIFT) fill_windows(win, a);
  const int cols = (a.I + kBlock - 1) / kBlock;   // blocks per row
  const int row = lane_row(a, cols);
  const int64_t col = (int64_t)(blockIdx.x % cols) * kBlock + threadIdx.x;
  if (row >= a.rows || col >= a.I) return;
  const int64_t e = (int64_t)row * a.I + col;
  float l[K], cand[K], g[Z];
#pragma unroll
  for (int k = 0; k < K; ++k) l[k] = a.L[state_off(e, k, K)];
  const float w = load_w(a, e);
  const double s = (double)a.S[(int64_t)row * (a.I / a.gs) + col / a.gs];
  const uint32_t j0 = kMode == GSQ_RELAX_SHIFT ? a.J0[e] : 0u;
  coord_candidates<K, kMode>(cand, a, win, j0, 0);
  lane_noise<Z, kMode>(g, a, (uint64_t)e, a.t, (uint32_t)a.sample);
  double v, jac[K];
  coord_sample<K, Z, true, kMode>(l, cand, g, a.kappa, a.inv_tau_d, v, jac);
  static_cast<float*>(a.Rout)[padded_index(a, row, col)] = residual<true>(w, s, v);
}

// Gradient, update and (a.fuse) the next sample, as k_backward.
template <int K, bool kScales, bool kMulti, int kMode, bool kLion>
__global__ __launch_bounds__(kBlock) void k_backward_f64(ElemArgs a) {
  constexpr int Z = noise_count<K, kMode>();
  constexpr int kWaves = kBlock / 64;
  __shared__ __align__(16) float win[kMode == GSQ_RELAX_SHIFT ? GSQ_MAX_LEVELS * kWinRow : 4];
  if constexpr (kMode == GSQ_RELAX_SHIFT) fill_windows(win, a);
  __shared__ double part[2][kWaves];   // the wavefronts' sums: loss, scale gradient
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cols = (a.I + kBlock - 1) / kBlock;   // blocks per row
  const int row = lane_row(a, cols);
  const int64_t col = (int64_t)(blockIdx.x % cols) * kBlock + threadIdx.x;
  if (row >= a.rows) return;   // the whole workgroup
  const bool active = col < a.I;
  const double kt = (double)a.kappa * a.inv_tau_d;
  const double b1 = a.b1, b2 = a.b2, omb1 = 1.0 - b1, omb2 = 1.0 - b2;
  const double eps = a.eps, wd = a.wd;
  const int64_t gpr = a.I / a.gs;
  const int in_wave = min(a.gs, 64);
  const bool wide = kScales && a.gs > 64;   // a group spans gs / 64 wavefronts
  bool bad = false;
  const int64_t e = (int64_t)row * a.I + (active ? col : 0);
  const int64_t sidx = (int64_t)row * gpr + (active ? col / a.gs : 0);
  const int64_t gidx = active ? padded_index(a, row, col) : 0;
  const float s32 = a.S[sidx];
  const double s = s32;
  float l[K], m[K], v[K], ms = 0.f, vs = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t o = state_off(e, k, K);
    l[k] = active ? __builtin_nontemporal_load(a.L + o) : 0.f;
    m[k] = active ? __builtin_nontemporal_load(a.M + o) : 0.f;
    v[k] = active && !kLion ? __builtin_nontemporal_load(a.V + o) : 0.f;
  }
  if constexpr (kScales) {
    ms = a.MS[sidx];
    vs = a.VS[sidx];
  }
  const float w = active && (a.want_loss || a.fuse) ? load_w(a, e) : 0.f;
  const uint32_t j0 = kMode == GSQ_RELAX_SHIFT ? a.J0[e] : 0u;
  float cand[K];
  coord_candidates<K, kMode>(cand, a, win, j0, 0);

  double lsum = 0.0, ds = 0.0, d[K];
#pragma unroll
  for (int k = 0; k < K; ++k) d[k] = 0.0;
  const int M = kMulti ? a.samples : 1;
  for (int smp = 0; smp < M; ++smp) {
    const double gq = active ? (double)__builtin_nontemporal_load(a.G + smp * a.g_stride + gidx) : 0.0;
    float g[Z];
    lane_noise<Z, kMode>(g, a, (uint64_t)e, a.t, (uint32_t)smp);
    double val, jac[K];
    coord_sample<K, Z, true, kMode>(l, cand, g, a.kappa, a.inv_tau_d, val, jac);
    ds += gq * val;
    const double coef = kt * (gq * s);
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] += coef * jac[k];
    if (a.want_loss) lsum += (double)residual<true>(w, s, val) * gq;
  }
  if constexpr (kMulti) {
    const double inv_m = 1.0 / (double)M;
    ds *= inv_m;
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] *= inv_m;
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double th = l[k], m1 = m[k], v1 = v[k];
    opt_update<true, kLion>(d[k], th, m1, v1, (double)a.lr, a.step_l_d, b1, b2, omb1, omb2,
                            a.rbc2_d, eps, wd);
    l[k] = (float)th;
    m[k] = (float)m1;
    v[k] = (float)v1;
    if (active) {
      bad |= !(__builtin_isfinite(l[k]) && __builtin_isfinite(kLion ? m[k] : v[k]));
      const int64_t o = state_off(e, k, K);
      __builtin_nontemporal_store(l[k], a.L + o);
      __builtin_nontemporal_store(m[k], a.M + o);
      if (!kLion) __builtin_nontemporal_store(v[k], a.V + o);
    }
  }
  // sums over the wavefront, then over the workgroup, whose partial is that of its place in the grid
  // (row cols + x % cols, but no division that is kept in registers until here)
  if (a.want_loss) {
    const double x = wave_sum_to_lane63(-0.5 * lsum);   // P = -G / 2
    if (lane == 63) part[0][wave] = x;
  }
  if constexpr (kScales) {
    for (int off = 1; off < in_wave; off <<= 1) ds += __shfl_xor(ds, off, 64);
    if (wide && lane == 0) part[1][wave] = ds;
  }
  if (a.want_loss || wide) __syncthreads();   // the same for the whole workgroup
  if (a.want_loss && threadIdx.x == 0) {
    double x = part[0][0];
#pragma unroll
    for (int i = 1; i < kWaves; ++i) x += part[0][i];
    a.loss_part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = x;
  }
  float s_new = s32;
  if constexpr (kScales) {
    if (wide) {
      const int n = a.gs / 64, first = wave & ~(n - 1);
      ds = part[1][first];
      for (int i = 1; i < n; ++i) ds += part[1][first + i];
    }
    // every lane of the group forms the new scale; the old ones were read before the barrier (or
    // by this wavefront alone), so the first lane may write it
    double th = s, m1 = ms, v1 = vs;
    opt_update<true, kLion>(ds, th, m1, v1, (double)a.lr_s, a.step_s_d, b1, b2, omb1, omb2,
                            a.rbc2_d, eps, wd);
    s_new = (float)th;
    if (active && (threadIdx.x & (a.gs - 1)) == 0) {
      bad |= !(__builtin_isfinite(s_new) && __builtin_isfinite((float)(kLion ? m1 : v1)));
      a.MS[sidx] = (float)m1;
      a.VS[sidx] = (float)v1;
      a.S[sidx] = s_new;
    }
  }
  if (a.fuse && active) {
    float g[Z];
    lane_noise<Z, kMode>(g, a, (uint64_t)e, a.t_next, 0u);
    double val, jac[K];
    coord_sample<K, Z, true, kMode>(l, cand, g, a.kappa_n, a.inv_tau_n_d, val, jac);
    static_cast<float*>(a.Rout)[gidx] = residual<true>(w, (double)s_new, val);
  }
  if (bad) *a.flag = 1;
}

// One block per row and 256 columns: with a loop over rows the compiler keeps the polynomials'
// constants in scalar registers across it, more than there are, and reads them back one lane at a
// time (385 such moves per row at 8 levels).  Fills a.rows_x.
dim3 lane_grid(const Layer& L, ElemArgs& a) {
  const RowSplit sp = split_rows(L.B * L.O, (L.I + kBlock - 1) / kBlock);
  a.rows_x = sp.rows_x;
  return dim3(sp.gx, sp.gy);
}

template <int K, int kMode = GSQ_RELAX_GRID>
hipError_t forward_k(const Layer& L, ElemArgs a, hipStream_t s) {
  const dim3 g = lane_grid(L, a);
  hipLaunchKernelGGL((k_forward_f64<K, kMode>), g, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

template <int K, bool kMulti, int kMode, bool kLion>
void backward_km(const Layer& L, ElemArgs a, bool sc, hipStream_t s) {
  const dim3 g = lane_grid(L, a), b(kBlock);
  if (sc) hipLaunchKernelGGL((k_backward_f64<K, true, kMulti, kMode, kLion>), g, b, 0, s, a);
  else hipLaunchKernelGGL((k_backward_f64<K, false, kMulti, kMode, kLion>), g, b, 0, s, a);
}

template <int K, int kMode = GSQ_RELAX_GRID>
hipError_t backward_k(const Layer& L, const ElemArgs& a, bool sc, hipStream_t s) {
  if (a.lion) {
    if (a.samples > 1) backward_km<K, true, kMode, true>(L, a, sc, s);
    else backward_km<K, false, kMode, true>(L, a, sc, s);
  } else {
    if (a.samples > 1) backward_km<K, true, kMode, false>(L, a, sc, s);
    else backward_km<K, false, kMode, false>(L, a, sc, s);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_forward_f64(const Layer& L, const ElemArgs& a, hipStream_t s) {
  if (L.relax == GSQ_RELAX_SHIFT) return forward_k<GSQ_SHIFT_WINDOW, GSQ_RELAX_SHIFT>(L, a, s);
  if (L.relax == GSQ_RELAX_TERNARY) return forward_k<2, GSQ_RELAX_TERNARY>(L, a, s);
  switch (L.K) {
    case 2: return forward_k<2>(L, a, s);
    case 3: return forward_k<3>(L, a, s);
    case 4: return forward_k<4>(L, a, s);
    case 5: return forward_k<5>(L, a, s);
    case 6: return forward_k<6>(L, a, s);
    case 7: return forward_k<7>(L, a, s);
    default: return forward_k<8>(L, a, s);
  }
}

hipError_t launch_backward_f64(const Layer& L, const ElemArgs& a, bool update_scales, hipStream_t s) {
  if (L.relax == GSQ_RELAX_SHIFT)
    return backward_k<GSQ_SHIFT_WINDOW, GSQ_RELAX_SHIFT>(L, a, update_scales, s);
  if (L.relax == GSQ_RELAX_TERNARY) return backward_k<2, GSQ_RELAX_TERNARY>(L, a, update_scales, s);
  switch (L.K) {
    case 2: return backward_k<2>(L, a, update_scales, s);
    case 3: return backward_k<3>(L, a, update_scales, s);
    case 4: return backward_k<4>(L, a, update_scales, s);
    case 5: return backward_k<5>(L, a, update_scales, s);
    case 6: return backward_k<6>(L, a, update_scales, s);
    case 7: return backward_k<7>(L, a, update_scales, s);
    default: return backward_k<8>(L, a, update_scales, s);
  }
}

}  // namespace gsq
