// Device kernels of the learned smoother scaling (see learned.h).
#include "learned.h"

#include <algorithm>
#include <cmath>

namespace mfgmg {
namespace learned {

namespace {

constexpr int kBlock = 256;

inline unsigned grid_for(int64_t n, int block = kBlock, int64_t cap = 1 << 20) {
  int64_t g = (n + block - 1) / block;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return unsigned(g);
}

// velocity slot of local node a of cell c: node >= 0 when free, < 0 otherwise
// (on general levels a free slot also marks the components fixed by the
// no-normal-flux condition: slot_node / slot_fixed)
__device__ __forceinline__ int32_t lslot(const DevLevel& L, int64_t c, int a) {
  if (!L.uniform) return L.slots[27 * c + a];
  const int64_t n = L.n_edge, m = 2 * n + 1;
  const int64_t i = c % n, j = (c / n) % n, k = c / (n * n);
  const int64_t X = 2 * i + a % 3, Y = 2 * j + (a / 3) % 3, Z = 2 * k + a / 9;
  if (X == 0 || Y == 0 || Z == 0 || X == m - 1 || Y == m - 1 || Z == m - 1) return -1;
  return int32_t(X + m * (Y + m * Z));
}

__global__ void k_scal_accum(DevLevel L, const double* __restrict__ y, double* __restrict__ acc,
                             double* __restrict__ cnt) {
  for (int64_t c = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; c < L.ncell; c += int64_t(gridDim.x) * blockDim.x) {
    const double y0 = y[3 * c], y1 = y[3 * c + 1], y2 = y[3 * c + 2];
    for (int a = 0; a < 27; ++a) {
      const int32_t s = lslot(L, c, a);
      if (s < 0) continue;
      // a fixed component keeps s = 1 (its acc stays 0)
      const int64_t b = 3 * int64_t(slot_node(s));
      if (!slot_fixed(s, 0)) atomicAdd(&acc[b], y0);
      if (!slot_fixed(s, 1)) atomicAdd(&acc[b + 1], y1);
      if (!slot_fixed(s, 2)) atomicAdd(&acc[b + 2], y2);
      if (cnt) atomicAdd(&cnt[slot_node(s)], 1.0);
    }
  }
}

__global__ void k_scal_finish(int64_t nn, const double* __restrict__ acc, const double* __restrict__ cnt,
                              const double* __restrict__ minv, double* __restrict__ sdof, double* __restrict__ md,
                              float* __restrict__ mf) {
  for (int64_t v = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; v < nn; v += int64_t(gridDim.x) * blockDim.x) {
    const double k = cnt[v];
    for (int q = 0; q < 3; ++q) {
      const double sv = k > 0 ? exp(acc[3 * v + q] / k) : 1.0;
      const double ms = k > 0 ? sv * minv[3 * v + q] : minv[3 * v + q];
      if (sdof) sdof[3 * v + q] = sv;
      if (md) md[3 * v + q] = ms;
      if (mf) mf[3 * v + q] = float(ms);
    }
  }
}

__global__ void k_scal_grad(DevLevel L, const double* __restrict__ sbar, const double* __restrict__ sdof,
                            const double* __restrict__ cnt, double* __restrict__ ybar) {
  for (int64_t c = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; c < L.ncell; c += int64_t(gridDim.x) * blockDim.x) {
    double g0 = 0, g1 = 0, g2 = 0;
    for (int a = 0; a < 27; ++a) {
      const int32_t s = lslot(L, c, a);
      if (s < 0) continue;
      const int64_t b = 3 * int64_t(slot_node(s));
      const double ic = 1.0 / cnt[slot_node(s)];
      if (!slot_fixed(s, 0)) g0 += sbar[b] * sdof[b] * ic;
      if (!slot_fixed(s, 1)) g1 += sbar[b + 1] * sdof[b + 1] * ic;
      if (!slot_fixed(s, 2)) g2 += sbar[b + 2] * sdof[b + 2] * ic;
    }
    ybar[3 * c] = g0, ybar[3 * c + 1] = g1, ybar[3 * c + 2] = g2;
  }
}

__global__ void k_chebrev_a(int64_t n, const double* __restrict__ xbar, const double* __restrict__ minv,
                            const double* __restrict__ mp, const double* __restrict__ rk, double* __restrict__ dbar,
                            double* __restrict__ rbar, double* __restrict__ sbar, double beta, double sgn) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const double d = dbar[i] + xbar[i];
    dbar[i] = d;
    rbar[i] += beta * minv[i] * d;
    sbar[i] += sgn * beta * d * rk[i] * mp[i];
  }
}

// M-weight of the Ritz vector: out_i = v_i M_ii = v_i / minv_i
__global__ void k_ritz_mass(int64_t n, const double* __restrict__ v, const double* __restrict__ minv,
                            double* __restrict__ out) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    out[i] = v[i] / minv[i];
}

// term of dJ/ds through lambda(s): sbar_i -= coef v_i^2 M_ii / s_i
__global__ void k_lambda_term(int64_t n, const double* __restrict__ v, const double* __restrict__ minv,
                              const double* __restrict__ sdof, double coef, double* __restrict__ sbar) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    sbar[i] -= coef * v[i] * v[i] / (minv[i] * sdof[i]);
}

__global__ void k_chebrev_b(int64_t n, double* __restrict__ dbar, const double* __restrict__ t, double alpha) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    dbar[i] = alpha * dbar[i] - t[i];
}

template <typename T>
__global__ void k_adam(int64_t n, T* __restrict__ w, const T* __restrict__ g, T* __restrict__ m, T* __restrict__ v,
                       T lr, T b1, T b2, T eps, T bc1, T bc2, T clamp) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const T gi = g[i];
    const T mi = b1 * m[i] + (T(1) - b1) * gi;
    const T vi = b2 * v[i] + (T(1) - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    T wi = w[i] - lr * (mi / bc1) / (sqrt(vi / bc2) + eps);
    if (clamp > T(0)) wi = wi > clamp ? clamp : (wi < -clamp ? -clamp : wi);
    w[i] = wi;
  }
}

__global__ void k_features(int64_t ncell, const int32_t* __restrict__ nbr, const int32_t* __restrict__ self,
                           const double* __restrict__ mu, float* __restrict__ feat) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < 27 * ncell;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int64_t c = e / 27;
    feat[e] = float(log10(mu[nbr[e]]) - log10(mu[self[c]]));
  }
}

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// The network on the matrix cores: v_mfma_f32_16x16x4_f32 (FP32 in and out),
// 16 samples a tile.  Lane l of a wave holds, with col = l mod 16 and g = l
// div 16, the A entry (row col, k g), the B entry (k g, column col) and, in
// its four results r, the D entries (row 4 g + r, column col).  Rows are
// units, columns samples, wave w of the workgroup owns units 16 w .. 16 w + 15
// of each hidden layer.  Since a contraction's k order is free, k step (t, i)
// takes units 16 t + 4 g + i, so results feed the next layer as they lie.
// One thread per sample left the matrix cores idle and, at the training batch
// of 4,096, filled 32 workgroups: forward 57 -> 5.5 us, backward 207 -> 19.3 us.
using f4 = __attribute__((ext_vector_type(4))) float;
__device__ __forceinline__ f4 mfma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
constexpr int kTile = 16;               // samples a tile
constexpr int kK1 = (kIn + 3) / 4;      // k steps over the inputs
constexpr int kPitch = 80;              // LDS row of 64 units: 16 banks between the four k groups

__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ w, const float* __restrict__ x,
                                                     int64_t n, float* __restrict__ y, float* __restrict__ cache) {
  __shared__ float zc[kTile * kCache];              // z1, z2, z3 as the cache lays them out
  __shared__ __attribute__((aligned(16))) float hs[kTile][kPitch];
  __shared__ float z3[4][kTile][kOut];
  const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = l & 15, g = l >> 4, unit = 16 * wv + col;   // A row of the hidden layers
  float a1[kK1], a2[4][4], a3[4];
#pragma unroll
  for (int k = 0; k < kK1; ++k) a1[k] = 4 * k + g < kIn ? w[unit * kIn + min(4 * k + g, kIn - 1)] : 0.0f;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) a2[t][i] = w[kOffW2 + unit * kH + 16 * t + 4 * g + i];
#pragma unroll
  for (int i = 0; i < 4; ++i) a3[i] = col < kOut ? w[kOffW3 + min(col, kOut - 1) * kH + 16 * wv + 4 * g + i] : 0.0f;
  f4 b1, b2;
#pragma unroll
  for (int r = 0; r < 4; ++r) b1[r] = w[kOffB1 + 16 * wv + 4 * g + r], b2[r] = w[kOffB2 + 16 * wv + 4 * g + r];
  const int64_t tiles = (n + kTile - 1) / kTile;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t s0 = tile * kTile;
    const int ns = int(n - s0 < kTile ? n - s0 : kTile);
    const float* xs = x + (s0 + min(col, ns - 1)) * kIn;
    f4 z = b1;
    float xv[kK1];
#pragma unroll
    for (int k = 0; k < kK1; ++k) xv[k] = 4 * k + g < kIn ? xs[min(4 * k + g, kIn - 1)] : 0.0f;
#pragma unroll
    for (int k = 0; k < kK1; ++k) z = mfma(a1[k], xv[k], z);
    f4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) zc[col * kCache + 16 * wv + 4 * g + r] = z[r], h[r] = gelu(z[r]);
    *reinterpret_cast<f4*>(&hs[col][16 * wv + 4 * g]) = h;
    __syncthreads();
    z = b2;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f4 hv = *reinterpret_cast<const f4*>(&hs[col][16 * t + 4 * g]);
#pragma unroll
      for (int i = 0; i < 4; ++i) z = mfma(a2[t][i], hv[i], z);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) zc[col * kCache + kH + 16 * wv + 4 * g + r] = z[r], h[r] = gelu(z[r]);
    // the output layer: each wave over its own 16 units
    f4 o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i) o = mfma(a3[i], h[i], o);
    if (g == 0) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) z3[wv][col][c] = o[c];
    }
    __syncthreads();
    if (tid < kTile * kOut) {
      const int s = tid / kOut, c = tid % kOut;
      const float q = w[kOffB3 + c] + ((z3[0][s][c] + z3[1][s][c]) + (z3[2][s][c] + z3[3][s][c]));
      zc[s * kCache + 2 * kH + c] = q;
      if (s < ns) y[s0 * kOut + tid] = q > kClamp ? kClamp : (q < -kClamp ? -kClamp : q);
    }
    __syncthreads();
    for (int i = tid; i < ns * kCache; i += 256) cache[s0 * kCache + i] = zc[i];
    __syncthreads();
  }
}

// Backward: d3 = dy where the clamp passes, d2 = W3^T d3 gelu'(z2), d1 = W2^T
// d2 gelu'(z1); then the weight gradients contract over the tile's samples
// (A: deltas, B: activations, both through LDS), accumulated in registers over
// the workgroup's tiles and written as one partial per workgroup.  The bias
// gradients are a column of ones beside the inputs (b1) and sums over columns
// (b2, b3).  Deltas and activations never go to memory.
__global__ __launch_bounds__(256) void k_mlp_backward(const float* __restrict__ w, const float* __restrict__ x,
                                                      const float* __restrict__ cache, const float* __restrict__ dy,
                                                      int64_t n, float* __restrict__ part) {
  __shared__ float zc[kTile * kCache];
  __shared__ __attribute__((aligned(16))) float d1s[kTile][kPitch], h1s[kTile][kPitch], d2s[kTile][kPitch],
      h2s[kTile][kPitch];
  __shared__ float xs[kTile][kIn + 1], d3s[kTile][4];
  const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = l & 15, g = l >> 4, unit = 16 * wv + col;
  float a2[4][4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) a2[t][i] = w[kOffW2 + (16 * t + 4 * g + i) * kH + unit];
  const float a3 = g < kOut ? w[kOffW3 + min(g, kOut - 1) * kH + unit] : 0.0f;
  const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f4 g1[2] = {zero, zero}, g2[4] = {zero, zero, zero, zero}, g3 = zero, gb2 = zero;
  float gb3 = 0.0f;
  const int64_t tiles = (n + kTile - 1) / kTile;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t s0 = tile * kTile;
    const int ns = int(n - s0 < kTile ? n - s0 : kTile);
    for (int i = tid; i < kTile * kCache; i += 256) zc[i] = i < ns * kCache ? cache[s0 * kCache + i] : 0.0f;
    for (int i = tid; i < kTile * (kIn + 1); i += 256) {
      const int s = i / (kIn + 1), c = i % (kIn + 1);
      xs[s][c] = s >= ns ? 0.0f : c < kIn ? x[(s0 + s) * kIn + c] : 1.0f;
    }
    const float dyv = g < kOut && col < ns ? dy[(s0 + col) * kOut + g] : 0.0f;
    __syncthreads();
    const float zo = zc[col * kCache + 2 * kH + min(g, kOut - 1)];
    const float d3 = g < kOut && zo > -kClamp && zo < kClamp ? dyv : 0.0f;
    if (wv == 0) d3s[col][g] = d3, gb3 += d3;
    f4 d = mfma(a3, d3, zero), h;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float z = zc[col * kCache + kH + 16 * wv + 4 * g + r];
      d[r] *= gelu_d(z);
      h[r] = gelu(z);
    }
    gb2 += d;
    *reinterpret_cast<f4*>(&d2s[col][16 * wv + 4 * g]) = d;
    *reinterpret_cast<f4*>(&h2s[col][16 * wv + 4 * g]) = h;
    __syncthreads();
    d = zero;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f4 dv = *reinterpret_cast<const f4*>(&d2s[col][16 * t + 4 * g]);
#pragma unroll
      for (int i = 0; i < 4; ++i) d = mfma(a2[t][i], dv[i], d);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float z = zc[col * kCache + 16 * wv + 4 * g + r];
      d[r] *= gelu_d(z);
      h[r] = gelu(z);
    }
    *reinterpret_cast<f4*>(&d1s[col][16 * wv + 4 * g]) = d;
    *reinterpret_cast<f4*>(&h1s[col][16 * wv + 4 * g]) = h;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTile / 4; ++k) {
      const int s = 4 * k + g;   // the sample of this lane's k
      const float e1 = d1s[s][unit], e2 = d2s[s][unit], e3 = col < kOut ? d3s[s][min(col, kOut - 1)] : 0.0f;
      g1[0] = mfma(e1, xs[s][col], g1[0]);
      g1[1] = mfma(e1, col < kIn + 1 - 16 ? xs[s][min(16 + col, kIn)] : 0.0f, g1[1]);
#pragma unroll
      for (int t = 0; t < 4; ++t) g2[t] = mfma(e2, h1s[s][16 * t + col], g2[t]);
      g3 = mfma(e3, h2s[s][unit], g3);
    }
    __syncthreads();
  }
  float* out = part + int64_t(blockIdx.x) * kParams;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int o = 16 * wv + 4 * g + r;
    out[o * kIn + col] = g1[0][r];
    if (16 + col < kIn) out[o * kIn + 16 + col] = g1[1][r];
    else if (16 + col == kIn) out[kOffB1 + o] = g1[1][r];
#pragma unroll
    for (int t = 0; t < 4; ++t) out[kOffW2 + o * kH + 16 * t + col] = g2[t][r];
    if (g == 0 && r < kOut) out[kOffW3 + r * kH + unit] = g3[r];
    float sb = gb2[r];
#pragma unroll
    for (int q = 8; q > 0; q >>= 1) sb += __shfl_xor(sb, q);
    if (col == 0) out[kOffB2 + o] = sb;
  }
#pragma unroll
  for (int q = 8; q > 0; q >>= 1) gb3 += __shfl_xor(gb3, q);
  if (wv == 0 && col == 0 && g < kOut) out[kOffB3 + g] = gb3;
}

// dw = sum of the partials: 64 parameters a workgroup, 16 waves that each sum
// every 16th partial (eight loads in flight), then meet in LDS
__global__ __launch_bounds__(1024) void k_sum_parts(int np, const float* __restrict__ part, float* __restrict__ dw) {
  __shared__ float sh[16][64];
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, i = blockIdx.x * 64 + l, ic = min(i, kParams - 1);
  float a = 0.0f;
  for (int k0 = wv; k0 < np; k0 += 16 * 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[int64_t(min(k0 + 16 * u, np - 1)) * kParams + ic];
#pragma unroll
    for (int u = 0; u < 8; ++u) a += k0 + 16 * u < np ? v[u] : 0.0f;
  }
  sh[wv][l] = a;
  __syncthreads();
  if (wv != 0 || i >= kParams) return;
  a = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k) a += sh[k][l];
  dw[i] = a;
}
__global__ __launch_bounds__(kBlock) void k_mse(int64_t n, const float* __restrict__ y, const float* __restrict__ t,
                                                float* __restrict__ dy, float scale, double* __restrict__ loss) {
  __shared__ double sm[kBlock / 64];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const float d = y[i] - t[i];
    dy[i] = scale * d;
    acc += double(d) * double(d);
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0 && loss) {
    double b = 0.0;
    for (int i = 0; i < int(blockDim.x >> 6); ++i) b += sm[i];
    atomicAdd(loss, b);
  }
}

__global__ void k_gather_rows(const float* __restrict__ src, int cols, const int64_t* __restrict__ idx, int64_t n,
                              float* __restrict__ dst) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n * cols; e += int64_t(gridDim.x) * blockDim.x) {
    const int64_t i = e / cols, j = e % cols;
    dst[e] = src[idx[i] * cols + j];
  }
}

__global__ void k_d2f(int64_t n, const double* __restrict__ a, float* __restrict__ b) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    b[i] = float(a[i]);
}
__global__ void k_f2d(int64_t n, const float* __restrict__ a, double* __restrict__ b) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    b[i] = double(a[i]);
}

}  // namespace

void launch_scaling_accum(const DevLevel& L, const double* y, double* acc, double* cnt, hipStream_t s) {
  k_scal_accum<<<grid_for(L.ncell), kBlock, 0, s>>>(L, y, acc, cnt);
}
void launch_scaling_finish(int64_t nn, const double* acc, const double* cnt, const double* minv, double* sdof,
                           double* md, float* mf, hipStream_t s) {
  k_scal_finish<<<grid_for(nn), kBlock, 0, s>>>(nn, acc, cnt, minv, sdof, md, mf);
}
void launch_scaling_grad(const DevLevel& L, const double* sbar, const double* sdof, const double* cnt, double* ybar,
                         hipStream_t s) {
  k_scal_grad<<<grid_for(L.ncell), kBlock, 0, s>>>(L, sbar, sdof, cnt, ybar);
}
void launch_chebrev_a(int64_t n, const double* xbar, const double* minv, const double* mp, const double* rk,
                      double* dbar, double* rbar, double* sbar, double beta, double sgn, hipStream_t s) {
  k_chebrev_a<<<grid_for(n), kBlock, 0, s>>>(n, xbar, minv, mp, rk, dbar, rbar, sbar, beta, sgn);
}
void launch_ritz_mass(int64_t n, const double* v, const double* minv, double* out, hipStream_t s) {
  k_ritz_mass<<<grid_for(n), kBlock, 0, s>>>(n, v, minv, out);
}
void launch_lambda_term(int64_t n, const double* v, const double* minv, const double* sdof, double coef, double* sbar,
                        hipStream_t s) {
  k_lambda_term<<<grid_for(n), kBlock, 0, s>>>(n, v, minv, sdof, coef, sbar);
}
void launch_chebrev_b(int64_t n, double* dbar, const double* t, double alpha, hipStream_t s) {
  k_chebrev_b<<<grid_for(n), kBlock, 0, s>>>(n, dbar, t, alpha);
}
template <typename T>
void launch_adam(int64_t n, T* w, const T* g, T* m, T* v, double lr, double b1, double b2, double eps, int64_t t,
                 double clamp, hipStream_t s) {
  const double bc1 = 1.0 - std::pow(b1, double(t)), bc2 = 1.0 - std::pow(b2, double(t));
  k_adam<T><<<grid_for(n), kBlock, 0, s>>>(n, w, g, m, v, T(lr), T(b1), T(b2), T(eps), T(bc1), T(bc2), T(clamp));
}
template void launch_adam<float>(int64_t, float*, const float*, float*, float*, double, double, double, double,
                                 int64_t, double, hipStream_t);
template void launch_adam<double>(int64_t, double*, const double*, double*, double*, double, double, double, double,
                                  int64_t, double, hipStream_t);
void launch_features(int64_t ncell, const int32_t* nbr, const int32_t* self, const double* mu, float* feat,
                     hipStream_t s) {
  k_features<<<grid_for(27 * ncell), kBlock, 0, s>>>(ncell, nbr, self, mu, feat);
}
void launch_mlp_forward(const float* w, const float* x, int64_t n, float* y, float* cache, hipStream_t s) {
  if (n <= 0) return;
  // at most six workgroups a CU, which keep their weights in registers over their tiles
  k_mlp_forward<<<unsigned(std::min<int64_t>((n + kTile - 1) / kTile, 1536)), 256, 0, s>>>(w, x, n, y, cache);
}
void launch_mlp_backward(const float* w, const float* x, const float* cache, const float* dy, int64_t n, float* dw,
                         float* work, hipStream_t s) {
  if (n <= 0) return;
  // Two tiles a workgroup (its 24.6 KB partial costs about as much as a tile)
  // until the chip is full; the work array holds that many partials from n = 1 up
  const int64_t tiles = (n + kTile - 1) / kTile;
  const int np = int(std::min<int64_t>((tiles + 1) / 2, 1024));
  k_mlp_backward<<<unsigned(np), 256, 0, s>>>(w, x, cache, dy, n, work);
  k_sum_parts<<<(kParams + 63) / 64, 1024, 0, s>>>(np, work, dw);
}
void launch_mse(int64_t n3, const float* y, const float* t, float* dy, float scale, double* loss, hipStream_t s) {
  k_mse<<<grid_for(n3, kBlock, 1024), kBlock, 0, s>>>(n3, y, t, dy, scale, loss);
}
void launch_gather_rows(const float* src, int cols, const int64_t* idx, int64_t n, float* dst, hipStream_t s) {
  k_gather_rows<<<grid_for(n * cols), kBlock, 0, s>>>(src, cols, idx, n, dst);
}
void launch_d2f(int64_t n, const double* a, float* b, hipStream_t s) { k_d2f<<<grid_for(n), kBlock, 0, s>>>(n, a, b); }
void launch_f2d(int64_t n, const float* a, double* b, hipStream_t s) { k_f2d<<<grid_for(n), kBlock, 0, s>>>(n, a, b); }

}  // namespace learned
}  // namespace mfgmg
