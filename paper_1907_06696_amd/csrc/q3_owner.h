// The Q3 operator on lattice levels, fused with what consumes A x (device
// code).
//
// Small levels, where a kernel's time is its chain of latencies: a workgroup
// owns the nodes of 2 x 2 x 2 cells (half-open box) and computes the 3 x 3 x 3
// cells that touch them, so A x of an owned node is complete inside the
// workgroup and the smoother's update is formed there, in one kernel.  Large
// levels: a workgroup computes its own 4 x 2 x 2 cells and leaves the sums of
// its high faces in halo slots; a second kernel adds them and forms the update.
// Each cell and component is four lanes, a quad, one lane for each plane of
// 4 x 4 nodes.
//
// In tensor products of Legendre polynomials P_0 .. P_3 of the cell the mass
// matrix is diagonal and a derivative has four entries a line, P_1' = 2 P_0,
// P_2' = 6 P_1, P_3' = 10 P_2 + 2 P_0 on [0, 1], so the exact integrals of the
// strain rate are a few multiply-adds a value, where the interpolation to
// Gauss points and the derivatives there are 36 dense 4 x 4 contractions a
// cell.  The transforms use the symmetry of the Lobatto points: with A = u_0 +
// u_3, B = u_1 + u_2, C = u_3 - u_0, D = u_2 - u_1 the scaled modes are
//   q_0 = A + 5 B, q_1 = C + sqrt 5 D, q_2 = A - B, q_3 = C - sqrt 5 D
// (12, 4, 12/5 and 4 times the Legendre coefficients); x and y run inside a
// lane, z between the quad's lanes.
//
// One smoothing step, FP64, against a wavefront per cell with dense
// contractions, halo kernel and update kernel: 32^3 95 -> 53 us, 16^3 25 -> 13
// us, 8^3 17 -> 9 us, 4^3 16 -> 9 us.  The small levels are bound by that
// chain, the brick by LDS and vector operations alike (per wave some 120 LDS
// reads and 1000 operations of which half are indices; 84 registers hold a
// plane, 77 in the fused kernel), the halo kernel by memory (5.5 TB/s).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "owner_kernel.h"

namespace mfgmg {
namespace q3own {

using owner::Op;

template <typename T>
struct Args {
  int n;              // cells per edge
  const T* mu;
  const T* x;
  const T* b;
  const T* minv;
  T* d;
  T* y;               // never x: neighbouring workgroups read x
  T alpha, beta, it0;
};

struct Brick {
  static constexpr int BX = 2, CX = BX + 1, C = 3, cells = CX * C * C, quads = 4 * cells;
  static constexpr int NX = 3 * CX + 1, N = 10;         // node box, from 3 points below
  static constexpr int RS = NX + 1, PS = RS * N;        // its row and plane strides in LDS
  static constexpr int waves = (quads + 63) / 64;       // of one component
  static constexpr int threads = 3 * 64 * waves;
};

// value of another lane of the quad (PERM: DPP quad_perm)
template <int PERM>
__device__ __forceinline__ float quad(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), PERM, 0xF, 0xF, false));
}
template <int PERM>
__device__ __forceinline__ double quad(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp(int(b & 0xffffffffLL), PERM, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(int(b >> 32), PERM, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
constexpr int perm(int a, int b, int c, int d) { return a | b << 2 | c << 4 | d << 6; }
constexpr int kRev = perm(3, 2, 1, 0), kSwap = perm(1, 0, 3, 2);

constexpr double kR5 = 2.23606797749978969641;   // sqrt 5

template <typename T>
__device__ __forceinline__ void to_modes(T& a, T& b, T& c, T& d) {
  const T A = a + d, C = d - a, B = b + c, D = c - b;
  a = A + T(5) * B, b = C + T(kR5) * D, c = A - B, d = C - T(kR5) * D;
}
template <typename T>
__device__ __forceinline__ void from_modes(T& a, T& b, T& c, T& d) {   // its transpose
  const T P = a + c, Q = b + d, R = T(5) * a - c, S = T(kR5) * (b - d);
  a = P - Q, b = R - S, c = R + S, d = P + Q;
}

// Weights of a mode (index) along an axis, products of scaling and mass: value
// against value, derivative against value, derivative against derivative,
// where the derivative of (q_0 .. q_3) is (q_1 + q_3, q_2, q_3, 0)
constexpr double kW00[4] = {1.0 / 144, 1.0 / 48, 5.0 / 144, 1.0 / 112};
constexpr double kWD0[4] = {1.0 / 24, 5.0 / 24, 5.0 / 24, 0.0};

// The quad's lanes hold modes 0, 2, 1, 3 along z.  Per-lane factors: built
// again for each phase from the lane number (fresh), for together they would
// hold 22 registers through the kernel.
__device__ __forceinline__ int fresh(int l) {
  asm volatile("" : "+v"(l));
  return l;
}
template <typename T>
__device__ __forceinline__ T pick(int l, double a, double b, double c, double d) {
  return (l & 2) ? (l & 1) ? T(d) : T(c) : (l & 1) ? T(b) : T(a);
}
template <typename T>
struct Transform {
  T sg, al, be, bt;
  __device__ explicit Transform(int l)
      : sg(l < 2 ? T(1) : T(-1)), al(pick<T>(l, 1, -1, kR5, 1)), be(pick<T>(l, 5, 1, 1, -kR5)),
        bt(pick<T>(l, 1, 5, -kR5, 1)) {}
  __device__ __forceinline__ T to_modes(T v) const {
    const T e = v + sg * quad<kRev>(v);
    return al * e + be * quad<kSwap>(e);
  }
  __device__ __forceinline__ T from_modes(T v) const {
    const T e = al * v + bt * quad<kSwap>(v);
    return e - sg * quad<kRev>(e);
  }
};
template <typename T>
struct Weights {
  T z00, zd0, ta, tb;   // mu h times the weights along z; d_z^T d_z = ta own + tb partner's
  int l;
  __device__ Weights(int l_, T mu_h)
      : z00(mu_h * pick<T>(l_, kW00[0], kW00[2], kW00[1], kW00[3])),
        zd0(mu_h * pick<T>(l_, kWD0[0], kWD0[2], kWD0[1], kWD0[3])), ta(mu_h * pick<T>(l_, 0, 25.0 / 12, 0.25, 1.5)),
        tb(mu_h * pick<T>(l_, 0, 0, 0.25, 0.25)), l(l_) {}
};

// Component C of mu h K applied in modes.  other(c, s): mode s = i + 4 j of
// component c on this lane; at(c, s, l): on lane l of the quad.  The own
// component is read again where it is needed: held in registers it would halve
// the waves in flight.
template <int C, typename T, typename G, typename H>
__device__ __forceinline__ void apply_modes(int z, T mu_h, T (&y)[16], G other, H at) {
  const Weights<T> L(z, mu_h);
  constexpr T fx = C == 0 ? 2 : 1, fy = C == 1 ? 2 : 1, fz = C == 2 ? 2 : 1;
  // in the plane: second derivatives of the own component ...
#pragma unroll
  for (int i = 0; i < 16; ++i) y[i] = T(0);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const T wx = fx * T(kW00[j]), wy = fy * T(kW00[j]);
    const T x1 = other(C, 1 + 4 * j), x2 = other(C, 2 + 4 * j), x3 = other(C, 3 + 4 * j);
    const T y1 = at(C, j + 4, L.l), y2 = at(C, j + 8, L.l), y3 = at(C, j + 12, L.l);
    const T a = T(0.25) * (x1 + x3), c = T(0.25) * (y1 + y3);
    y[1 + 4 * j] += wx * a;
    y[2 + 4 * j] += wx * T(25.0 / 12) * x2;
    y[3 + 4 * j] += wx * (a + T(1.25) * x3);
    y[j + 4] += wy * c;
    y[j + 8] += wy * T(25.0 / 12) * y2;
    y[j + 12] += wy * (c + T(1.25) * y3);
    __builtin_amdgcn_sched_barrier(0);   // or every LDS read moves to the front, and registers spill
  }
  // ... and the other in-plane component
  if constexpr (C == 0) {   // d_y^T d_x u_y
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const T q1 = other(1, 1 + 4 * j), q2 = other(1, 2 + 4 * j), q3 = other(1, 3 + 4 * j);
      const T f[3] = {T(kWD0[0] * kWD0[j]) * (q1 + q3), T(kWD0[1] * kWD0[j]) * q2, T(kWD0[2] * kWD0[j]) * q3};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (j == 0) y[i + 4] += f[i], y[i + 12] += f[i];
        else if (j == 1) y[i + 8] += f[i];
        else y[i + 12] += f[i];
      }
    }
  } else if constexpr (C == 1) {   // d_x^T d_y u_x
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T q1 = other(0, i + 4), q2 = other(0, i + 8), q3 = other(0, i + 12);
      const T f[3] = {T(kWD0[0] * kWD0[i]) * (q1 + q3), T(kWD0[1] * kWD0[i]) * q2, T(kWD0[2] * kWD0[i]) * q3};
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (i == 0) y[1 + 4 * j] += f[j], y[3 + 4 * j] += f[j];
        else if (i == 1) y[2 + 4 * j] += f[j];
        else y[3 + 4 * j] += f[j];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i % 8 == 0) __builtin_amdgcn_sched_barrier(0);
    y[i] = L.z00 * y[i] + T(fz * kW00[i & 3] * kW00[i >> 2]) * (L.ta * at(C, i, L.l) + L.tb * at(C, i, L.l ^ 1));
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (C < 2) {   // d_z^T d_C u_z
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // line along axis C (stride S), the other in-plane index j
      constexpr int S = C == 0 ? 1 : 4, R = 5 - S;
      const T q1 = other(2, S + R * j), q2 = other(2, 2 * S + R * j), q3 = other(2, 3 * S + R * j);
      const T f[3] = {T(kWD0[0] * kW00[j]) * (q1 + q3), T(kWD0[1] * kW00[j]) * q2, T(kWD0[2] * kW00[j]) * q3};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const T g = L.zd0 * f[i];
        // mode 1 takes mode 0, mode 2 mode 1, mode 3 both 0 and 2; lane 3's g is 0
        y[S * i + R * j] += quad<perm(3, 2, 0, 0)>(g) + quad<perm(3, 3, 3, 1)>(g);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {   // d_x^T d_z u_x and d_y^T d_z u_y
    // source lanes: mode 0 takes modes 1 and 3, mode 1 mode 2, mode 2 mode 3
    const int sa = (2 | 3 << 2 | 1 << 4) >> (2 * L.l) & 3;
    const T m0 = L.l == 0 ? T(1) : T(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const T gx = L.zd0 * T(kWD0[i] * kW00[j]) * (at(0, i + 4 * j, sa) + m0 * at(0, i + 4 * j, 3));
        const T gy = L.zd0 * T(kWD0[i] * kW00[j]) * (at(1, 4 * i + j, sa) + m0 * at(1, 4 * i + j, 3));
        if (i == 0) y[1 + 4 * j] += gx, y[3 + 4 * j] += gx, y[4 + j] += gy, y[12 + j] += gy;
        else if (i == 1) y[2 + 4 * j] += gx, y[8 + j] += gy;
        else y[3 + 4 * j] += gx, y[12 + j] += gy;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The cells' share of A x in the workgroup: w, the component's 4 x 4 nodes of
// this lane's plane, becomes the cell's results there, left in mem
// ([component][16][quad lane], read after the caller's barrier).  mem may hold
// the box that w came from.
template <int L4, typename T>
__device__ __forceinline__ void apply_cells(T* mem, int comp, int li, bool live, T mu_h, T (&w)[16]) {
  auto ex = [&](int q, int s, int l) -> T& { return mem[(16 * q + s) * L4 + l]; };
  const int z = li & 3;
#pragma unroll
  for (int j = 0; j < 4; ++j) to_modes(w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]);
#pragma unroll
  for (int i = 0; i < 4; ++i) to_modes(w[i], w[i + 4], w[i + 8], w[i + 12]);
  {
    const Transform<T> tz(fresh(z));
#pragma unroll
    for (int s = 0; s < 16; ++s) w[s] = tz.to_modes(w[s]);
  }
  __syncthreads();
  if (live) {
#pragma unroll
    for (int s = 0; s < 16; ++s) ex(comp, s, li) = w[s];
  }
  __syncthreads();
  auto other = [&](int c, int s) { return ex(c, s, li); };
  auto at = [&](int c, int s, int l) { return ex(c, s, (li & ~3) + l); };
  if (comp == 0) apply_modes<0>(fresh(z), mu_h, w, other, at);
  else if (comp == 1) apply_modes<1>(fresh(z), mu_h, w, other, at);
  else apply_modes<2>(fresh(z), mu_h, w, other, at);
  {
    const Transform<T> tz(fresh(z));
#pragma unroll
    for (int s = 0; s < 16; ++s) w[s] = tz.from_modes(w[s]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) from_modes(w[i], w[i + 4], w[i + 8], w[i + 12]);
#pragma unroll
  for (int j = 0; j < 4; ++j) from_modes(w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]);
  __syncthreads();
  if (live) {
#pragma unroll
    for (int s = 0; s < 16; ++s) ex(comp, s, li) = w[s];
  }
}

// What is done with A x at an entry (x there: xe, for Add y: de)
template <Op OP, typename T>
__device__ __forceinline__ void finish(const Args<T>& a, int64_t i, T ax, bool fixed, T xe, T be, T me, T de) {
  if (fixed) ax = xe;
  if constexpr (OP == Op::Apply) {
    a.y[i] = ax;
  } else if constexpr (OP == Op::Add) {
    if (!fixed) a.y[i] = de + ax;
  } else if constexpr (OP == Op::Residual) {
    a.y[i] = be - ax;
  } else {
    T dn = a.beta * me * (be - ax);
    if constexpr (OP == Op::First) dn = a.alpha * xe + dn;
    if constexpr (OP == Op::Step || OP == Op::Last) dn = a.alpha * de + dn;
    if constexpr (OP != Op::Last) a.d[i] = dn;
    a.y[i] = xe + dn;
  }
}

// Small levels
template <typename T, Op OP>
__global__ __launch_bounds__(Brick::threads) void k_owner_q3(Args<T> a) {
  using S = Brick;
  constexpr int BX = S::BX, CX = S::CX, C = S::C, NX = S::NX, N = S::N, RS = S::RS, PS = S::PS, L4 = S::quads;
  constexpr int kThreads = S::threads, kBox = PS * N, kIn = 3 * kBox, kOut = 48 * L4;
  __shared__ T mem[kIn > kOut ? kIn : kOut];   // x on the box; then modes, then results, [component][16][quad lane]
  const int n = a.n, m = 3 * n + 1, nbx = n / BX, nb = n / 2;
  const int blk = int(brick::xcd_order(blockIdx.x, gridDim.x));
  const int bx = blk % nbx, by = blk / nbx % nb, bz = blk / (nbx * nb);
  const int X0 = 3 * BX * bx, Y0 = 6 * by, Z0 = 6 * bz, t = threadIdx.x;
  // entries of the box: its own first node's (uniform) plus an offset
  const int64_t first = 3 * (X0 + int64_t(m) * (Y0 + int64_t(m) * Z0));
  auto inside = [m](int p) { return p > 0 && p < m - 1; };
  // box planes, one at a time; fixed nodes and points outside the level stage
  // zero.  Every load is issued before use.
  constexpr int RW = 3 * NX;
  const int plane = 3 * m * m;
  const int sw = t % RW, sx = sw / 3, sq = sw - 3 * sx, sy = t / RW;
  const bool stages = sy < N, sin = stages && inside(X0 - 3 + sx) && inside(Y0 - 3 + sy);
  const int so = sin ? 3 * (sx - 3 + m * (sy - 3)) + sq : 0;
  T v[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const bool in = inside(Z0 - 3 + k);   // uniform
    const int64_t at = first + (in ? (k - 3) * plane : 0);
    if constexpr (OP == Op::First) v[k] = (a.minv + at)[so] * (a.b + at)[so] * a.it0;
    else v[k] = (a.x + at)[so];
    if (!in || !sin) v[k] = T(0);
  }
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), comp = wave / S::waves;
  const int ql = t - 64 * S::waves * comp;
  const bool live = ql < L4;
  const int li = live ? ql : ql & 3, z = li & 3, ci = li >> 2;
  const int cx = ci % CX, cy = ci / CX % C, cz = ci / (CX * C);
  const int gx = BX * bx - 1 + cx, gy = 2 * by - 1 + cy, gz = 2 * bz - 1 + cz;
  const bool cell = gx >= 0 && gy >= 0 && gz >= 0;
  // mu h; zero for cells outside the mesh, whose points are all zero
  T mu_h = a.mu[cell ? gx + int64_t(n) * (gy + int64_t(n) * gz) : 0] / T(n);
  if (!cell) mu_h = T(0);
  if (stages) {
#pragma unroll
    for (int k = 0; k < N; ++k) mem[sq * kBox + sx + RS * sy + PS * k] = v[k];
  }
  __syncthreads();
  T w[16];
  const T* in = mem + comp * kBox + 3 * cx + RS * 3 * cy + PS * (3 * cz + z);
#pragma unroll
  for (int s = 0; s < 16; ++s) w[s] = in[(s & 3) + RS * (s >> 2)];
  apply_cells<L4>(mem, comp, li, live, mu_h, w);
  // this thread's owned entries, in KP planes at a time, loaded before the
  // results' barrier
  constexpr int OW = 9 * BX, OP1 = 6 * OW, KP = kThreads / OP1, KO = 6 / KP;   // words of a row, of a plane
  static_assert(6 % KP == 0);
  const int oz = t / OP1, ow = t % OW, oy = t % OP1 / OW, ox = ow / 3, oq = ow - 3 * ox;
  const bool owns = oz < KP;
  const int oxy = 3 * (ox + m * oy) + oq;
  T b[KO], mi[KO], d[KO], x[KO];
#pragma unroll
  for (int k = 0; k < KO; ++k) {
    const int i = oxy + plane * (owns ? KP * k + oz : 0);
    if constexpr (OP != Op::Apply && OP != Op::Add) b[k] = (a.b + first)[i];
    if constexpr (owner::is_update<OP>) mi[k] = (a.minv + first)[i];
    if constexpr (OP == Op::Step || OP == Op::Last) d[k] = (a.d + first)[i];
    if constexpr (OP == Op::Add) d[k] = (a.y + first)[i];
    if constexpr (OP == Op::First) x[k] = mi[k] * b[k] * a.it0;
    else x[k] = (a.x + first)[i];
  }
  __syncthreads();
  // A x of an owned entry: along each axis node 0 of the point's cell and node
  // 3 of the one below, or one node inside the cell
  const int cox = ox / 3, coy = oy / 3, pox = ox - 3 * cox, poy = oy - 3 * coy;
  const int oxyl = 16 * L4 * oq + 4 * (cox + 1 + CX * (coy + 1)) + L4 * (pox + 4 * poy);
  const int lowx = pox ? 0 : 3 * L4 - 4, lowy = poy ? 0 : 12 * L4 - 4 * CX;
#pragma unroll
  for (int k = 0; k < KO; ++k) {
    const int Z = KP * k + oz, coz = Z / 3, poz = Z - 3 * coz;
    const int at = oxyl + 4 * CX * C * (coz + 1) + poz, lowz = poz ? 0 : 3 - 4 * CX * C;
    if (!owns) break;
    T ax = T(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const T rv = mem[at + ((s & 1) ? lowx : 0) + ((s & 2) ? lowy : 0) + ((s & 4) ? lowz : 0)];
      const bool use = !(((s & 1) && pox) || ((s & 2) && poy) || ((s & 4) && poz));
      ax += use ? rv : T(0);
    }
    finish<OP>(a, first + oxy + plane * Z, ax, X0 + ox == 0 || Y0 + oy == 0 || Z0 + Z == 0, x[k], b[k], mi[k], d[k]);
  }
  // the closing planes, fixed throughout, belong to the last bricks
  if (OP == Op::Add || (bx < nbx - 1 && by < nb - 1 && bz < nb - 1)) return;
  constexpr int WX = 3 * BX + 1, W = 7;
  for (int e = t; e < 3 * WX * W * W; e += kThreads) {
    const int q = e % 3, lx = e / 3 % WX, ly = e / (3 * WX) % W, lz = e / (3 * WX * W);
    const bool c0 = lx == WX - 1, c1 = ly == W - 1, c2 = lz == W - 1;
    const bool mine = (c0 && bx == nbx - 1) || (c1 && by == nb - 1) || (c2 && bz == nb - 1);
    const bool theirs = (c0 && bx < nbx - 1) || (c1 && by < nb - 1) || (c2 && bz < nb - 1);
    if (!mine || theirs) continue;
    const int i = 3 * (lx + m * ly) + q + plane * lz;
    T be = T(0), me = T(0), de = T(0), xe;
    if constexpr (OP != Op::Apply && OP != Op::Add) be = (a.b + first)[i];
    if constexpr (owner::is_update<OP>) me = (a.minv + first)[i];
    if constexpr (OP == Op::Step || OP == Op::Last) de = (a.d + first)[i];
    if constexpr (OP == Op::First) xe = me * be * a.it0;
    else xe = (a.x + first)[i];
    finish<OP>(a, first + i, T(0), true, xe, be, me, de);
  }
}

// Large levels: the brick's own 4 x 2 x 2 cells only, 64 quad lanes, a wave a
// component.  y takes the sums of the points that the brick owns (Add: on top
// of y; x on fixed points), halo those of its 205 high-face points, which the
// kernel below adds.
struct Large {
  static constexpr int BX = 4, B = 2, NX = 3 * BX + 1, N = 3 * B + 1;
  static constexpr int threads = 192, L4 = 64;
  static constexpr int RS = NX + 1, PS = RS * N;
  static constexpr int rows = 4;   // box rows at a time: 39 words each
  static constexpr int halo = NX * N * N - (NX - 1) * (N - 1) * (N - 1);
};
// index of a high-face point in the brick's halo slot
__device__ __forceinline__ int halo_point(int lx, int ly, int lz) {
  constexpr int N = Large::N, L = Large::NX - 1, M = N - 1;
  if (lx == L) return ly + N * lz;
  if (ly == M) return N * N + lx + L * lz;
  return N * N + L * N + lx + L * ly;
}

template <typename T, Op OP>
__global__ __launch_bounds__(Large::threads) void k_brick_q3(Args<T> a, T* __restrict__ halo) {
  using S = Large;
  constexpr int NX = S::NX, N = S::N, RS = S::RS, PS = S::PS, L4 = S::L4, BX = S::BX;
  constexpr int kBox = PS * N, kIn = 3 * kBox, kOut = 48 * L4;
  __shared__ T mem[kIn > kOut ? kIn : kOut];
  const int n = a.n, m = 3 * n + 1, nbx = n / BX, nb = n / 2;
  const int blk = int(brick::xcd_order(blockIdx.x, gridDim.x));
  const int bx = blk % nbx, by = blk / nbx % nb, bz = blk / (nbx * nb);
  const int X0 = 3 * BX * bx, Y0 = 6 * by, Z0 = 6 * bz, t = threadIdx.x;
  const int64_t first = 3 * (X0 + int64_t(m) * (Y0 + int64_t(m) * Z0));
  const int plane = 3 * m * m;
  auto inside = [m](int p) { return p > 0 && p < m - 1; };
  const int sw = t % (3 * NX), sx = sw / 3, sq = sw - 3 * sx, r0 = t / (3 * NX);
  // rows r0 and r0 + 4 of the box's 7, all planes
  bool row[2], sin[2];
  T v[2][N];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int ly = r0 + S::rows * h;
    row[h] = r0 < S::rows && ly < N;
    sin[h] = row[h] && inside(X0 + sx) && inside(Y0 + ly);
    const int so = sin[h] ? sw + 3 * m * ly : 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const bool in = inside(Z0 + k);   // uniform
      const int64_t at = first + (in ? k * plane : 0);
      if constexpr (OP == Op::First) v[h][k] = (a.minv + at)[so] * (a.b + at)[so] * a.it0;
      else v[h][k] = (a.x + at)[so];
      if (!in || !sin[h]) v[h][k] = T(0);
    }
  }
  const int comp = __builtin_amdgcn_readfirstlane(t >> 6), li = t & 63, ci = li >> 2;
  const int cx = ci & 3, cy = ci >> 2 & 1, cz = ci >> 3;
  const T mu_h = a.mu[BX * bx + cx + int64_t(n) * (2 * by + cy + int64_t(n) * (2 * bz + cz))] / T(n);
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (row[h]) {
#pragma unroll
      for (int k = 0; k < N; ++k) mem[sq * kBox + sx + RS * (r0 + S::rows * h) + PS * k] = v[h][k];
    }
  __syncthreads();
  T w[16];
  const T* in = mem + comp * kBox + 3 * cx + RS * 3 * cy + PS * (3 * cz + (li & 3));
#pragma unroll
  for (int s = 0; s < 16; ++s) w[s] = in[(s & 3) + RS * (s >> 2)];
  apply_cells<L4>(mem, comp, li, true, mu_h, w);
  __syncthreads();
  const bool lastx = bx == nbx - 1, lasty = by == nb - 1, lastz = bz == nb - 1;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (!row[h]) break;
    // cells and nodes along x and y: a cell's node 0 and node 3 of the one below
    const int ly = r0 + S::rows * h;
    const int ax = sx == NX - 1 ? 3 : sx % 3, ay = ly == N - 1 ? 3 : ly % 3;
    const int kx = sx == NX - 1 ? BX - 1 : sx / 3, ky = ly == N - 1 ? 1 : ly / 3;
    const bool onex = ax != 0 || sx == 0, oney = ay != 0 || ly == 0;
    const int base = 16 * L4 * sq + 4 * (kx + BX * ky) + L4 * (ax + 4 * ay);
    const int lowx = onex ? 0 : 3 * L4 - 4, lowy = oney ? 0 : 12 * L4 - 4 * BX;
    const bool ownxy = (sx < NX - 1 || lastx) && (ly < N - 1 || lasty);
    const bool fixxy = !inside(X0 + sx) || !inside(Y0 + ly);
    const int oxy = sw + 3 * m * ly;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int az = k == N - 1 ? 3 : k % 3, kz = k == N - 1 ? 1 : k / 3;
      const bool own = ownxy && (k < N - 1 || lastz);
      const int64_t i = first + oxy + plane * k;
      if (fixxy || !inside(Z0 + k)) {
        if constexpr (OP != Op::Add) {
          if (own) a.y[i] = OP == Op::First ? a.minv[i] * a.b[i] * a.it0 : a.x[i];
        }
        continue;
      }
      T s = T(0);
#pragma unroll
      for (int u = 0; u < (k == 3 ? 8 : 4); ++u) {
        const int at = base + 4 * BX * 2 * kz + az + ((u & 1) ? lowx : 0) + ((u & 2) ? lowy : 0) +
                       ((u & 4) ? 3 - 4 * BX * 2 : 0);
        const T r = mem[at];
        s += ((u & 1) && onex) || ((u & 2) && oney) ? T(0) : r;
      }
      if (own) a.y[i] = OP == Op::Add ? a.y[i] + s : s;
      else halo[(int64_t(blk) * S::halo + halo_point(sx, ly, k)) * 3 + sq] = s;
    }
  }
}

// Adds the lower neighbours' halo values on the bricks' low faces and does
// what is done with A x, so that the smoother's update shares the pass.  One
// wave for 64 words of a lattice row.
template <typename T, Op OP>
__global__ __launch_bounds__(256) void k_halo_q3(Args<T> a, const T* __restrict__ halo) {
  using S = Large;
  constexpr int LX = S::NX - 1, L = S::N - 1;
  const int n = a.n, m = 3 * n + 1, nbx = n / S::BX, nb = n / 2, chunks = (3 * m + 63) / 64;
  const int wave = __builtin_amdgcn_readfirstlane(int(blockIdx.x * 4 + (threadIdx.x >> 6)));
  const int r = wave / chunks, word = (wave - r * chunks) * 64 + int(threadIdx.x & 63);
  const int Z = r / m, Y = r - Z * m, X = word / 3, q = word - 3 * X;
  if (Z >= m || word >= 3 * m) return;
  const bool yz = Y > 0 && Y < m - 1 && Z > 0 && Z < m - 1;
  const bool fixed = !yz || X == 0 || X == m - 1;
  const bool fx = X % LX == 0, fy = Y % L == 0, fz = Z % L == 0;
  if constexpr (OP == Op::Apply || OP == Op::Add) {   // y is there already
    if (fixed || !(fx || fy || fz)) return;
  }
  const int64_t i = 3 * int64_t(m) * r + word;
  T ax = a.y[i], xe = T(0), be = T(0), me = T(0), de = T(0);
  if constexpr (OP != Op::Apply && OP != Op::Add) be = a.b[i];
  if constexpr (owner::is_update<OP>) me = a.minv[i];
  if constexpr (OP == Op::Step || OP == Op::Last) de = a.d[i];
  if constexpr (OP == Op::First) xe = me * be * a.it0;
  else if constexpr (OP != Op::Apply && OP != Op::Add) xe = a.x[i];
  if (!fixed) {
    const int ox = X / LX, oy = Y / L, oz = Z / L, px = X - LX * ox, py = Y - L * oy, pz = Z - L * oz;
#pragma unroll
    for (int s = 1; s < 8; ++s) {
      const int ux = s & 1, uy = s >> 1 & 1, uz = s >> 2;
      if ((ux && !fx) || (uy && !fy) || (uz && !fz)) continue;
      const int64_t nbr = (ox - ux) + int64_t(nbx) * ((oy - uy) + int64_t(nb) * (oz - uz));
      ax += halo[(nbr * S::halo + halo_point(px + LX * ux, py + L * uy, pz + L * uz)) * 3 + q];
    }
  }
  if constexpr (OP == Op::Apply || OP == Op::Add) a.y[i] = ax;
  else finish<OP>(a, i, ax, fixed, xe, be, me, de);
}

}  // namespace q3own
}  // namespace mfgmg
