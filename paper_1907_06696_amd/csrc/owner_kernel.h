// Small uniform Q2 levels: the operator fused with what consumes A x (device
// code).
//
// On a level of 16^3 cells or fewer a kernel's time is its chain of latencies
// (launch, loads, LDS, barriers), not its bytes or operations, so the number
// of kernels and the length of that chain count.  One workgroup owns the nodes
// of 2 x 2 x 2 cells (the half-open node box; the last ones along an axis also
// the closing plane) and computes the 3 x 3 x 3 cells that touch them, three
// threads (components) a cell: A x of an owned node is complete inside the
// workgroup, so there is no output initialisation, no atomic and no second
// kernel, and the smoother's update is formed where A x is.  Each cell is
// computed by 3.4 workgroups on average, which costs less than the atomics
// (device scope, served beyond the XCD's L2) and the launch that it saves.
// One smoothing step against cell kernel with atomics plus update kernel, FP64
// / FP32: 16^3 13.5 -> 6.9 / 11.0 -> 5.5 us, 8^3 11.0 -> 5.7 / 9.4 -> 5.0 us.
// At 32^3 the brick is 4 x 2 x 2 cells (2.8 computed per cell; FP64 21.5
// against 28.2 us, FP32 14.8 against 18.6 us), still below the brick and halo
// kernels plus the update (23.6 / 19.3 us); from 64^3 up the redundant cells
// cost more than the halo pass (FP32 step 100 against 61 us).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "brick_kernel.h"
#include "cell_kernel.h"

namespace mfgmg {
namespace owner {

// What is done with A x.  The Chebyshev updates are d = alpha d + beta minv
// (b - A x), y = x + d:
//   Apply     y = A x (x on Dirichlet nodes)       Add   y += A x on free nodes
//   Residual  y = b - A x
//   First     x is x0 = d0 = it0 minv b, formed while it is staged (x and d are
//             not read); then an update
//   Start     an update with alpha = 0 (d is not read)
//   Step      an update;  Last: an update whose d is not stored
enum class Op { Apply, Add, Residual, First, Start, Step, Last };

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
  // MAP: storage node and cell of each lattice node and cell
  const int32_t* node;
  const int32_t* cell;
};

template <Op OP>
constexpr bool is_update = OP == Op::First || OP == Op::Start || OP == Op::Step || OP == Op::Last;

// Own cells 2 E x 2 x 2 (E = 1, 2), computed cells (2 E + 1) x 3 x 3.
template <int E>
struct Brick {
  static constexpr int BX = 2 * E, CX = BX + 1, C = 3, cells = CX * C * C;
  static constexpr int NX = 2 * BX + 3, N = 7, points = NX * N * N;   // node box, from 2 points below
};
constexpr int kThreads = 192;   // wave c: component c of the cells
// own nodes: 4 E x 4 x 4, three entries each, E a thread

// I: node index type (int up to 256 cells per edge).  MAP: a level under u . n
// = 0 whose cells are all of one size, stored in the general order: nodes and
// cells go through a.node and a.cell, and component c is fixed on the two
// faces normal to axis c only.
template <typename T, int E, typename I, bool MAP, Op OP>
__global__ __launch_bounds__(kThreads) void k_owner(Args<T> a) {
  using S = Brick<E>;
  constexpr int BX = S::BX, CX = S::CX, C = S::C, NX = S::NX, N = S::N, kCells = S::cells;
  // LDS: x on the box (x fastest) and the modes that other components read;
  // then, in the same place, the cells' results
  constexpr int kIn = 3 * S::points + 3 * cellop::kSharedModes * kCells, kOut = 3 * 27 * kCells;
  __shared__ T mem[kIn > kOut ? kIn : kOut];
  auto buf = [&](int q, int p) -> T& { return mem[q * S::points + p]; };
  auto ex = [&](int q, int s, int c) -> T& {
    return mem[3 * S::points + (q * cellop::kSharedModes + s) * kCells + c];
  };
  const int n = a.n, m = 2 * n + 1, nbx = n / BX, nb = n / 2;
  const int blk = int(brick::xcd_order(blockIdx.x, gridDim.x));
  const int bx = blk % nbx, by = blk / nbx % nb, bz = blk / (nbx * nb);
  const int X0 = 2 * BX * bx, Y0 = 4 * by, Z0 = 4 * bz;
  const int t = threadIdx.x;
  // index of component q at a lattice point, and whether it is fixed
  auto entry = [&](int X, int Y, int Z, int q) -> I {
    const I p = X + I(m) * (Y + I(m) * Z);
    return 3 * I(MAP ? a.node[p] : p) + q;
  };
  auto fixed = [&](int X, int Y, int Z, int q) {
    if constexpr (MAP) {
      const int w = q == 0 ? X : q == 1 ? Y : Z;
      return w == 0 || w == m - 1;
    }
    return X == 0 || X == m - 1 || Y == 0 || Y == m - 1 || Z == 0 || Z == m - 1;
  };
  // box rows, RP at a time; fixed entries and points outside
  // the level stage zero (their index is 0).  Every load is issued before use.
  constexpr int RW = 3 * NX, RP = kThreads / RW, NR = N * N, KS = (NR + RP - 1) / RP;
  const int word = t % RW, sx = word / 3, sq = word - 3 * sx, r0 = t / RW;
  T v[KS];
  {
    const int X = X0 - 2 + sx;
    const bool xin = r0 < RP && (MAP ? X >= 0 && X < m : X > 0 && X < m - 1);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const int r = r0 + RP * k, Y = Y0 - 2 + r % N, Z = Z0 - 2 + r / N;
      const bool in = xin && r < NR && (MAP ? Y >= 0 && Y < m && Z >= 0 && Z < m && !fixed(X, Y, Z, sq)
                                            : Y > 0 && Y < m - 1 && Z > 0 && Z < m - 1);
      const I i = in ? entry(X, Y, Z, sq) : 0;
      if constexpr (OP == Op::First) v[k] = a.minv[i] * a.b[i] * a.it0;
      else v[k] = a.x[i];
      if (!in) v[k] = T(0);
    }
  }
  // this thread's owned entries
  I own[E];
  bool dir[E];
  T b[E], mi[E], d[E], x[E];
  const int oq = t % 3, oy = t / (3 * 4) % 4, oz = t / (3 * 16);   // point 4 e + t / 3 % 4 along x
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int X = X0 + 4 * e + t / 3 % 4;
    own[e] = entry(X, Y0 + oy, Z0 + oz, oq);
    dir[e] = MAP ? fixed(X, Y0 + oy, Z0 + oz, oq) : X == 0 || Y0 + oy == 0 || Z0 + oz == 0;
    if constexpr (OP != Op::Apply && OP != Op::Add) b[e] = a.b[own[e]];
    if constexpr (is_update<OP>) mi[e] = a.minv[own[e]];
    if constexpr (OP == Op::Step || OP == Op::Last) d[e] = a.d[own[e]];
    if constexpr (OP == Op::Add) d[e] = a.y[own[e]];
    if constexpr (OP == Op::First) x[e] = mi[e] * b[e] * a.it0;
    else x[e] = a.x[own[e]];
  }
  const int comp = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const bool live = lane < kCells;
  const int ci = live ? lane : 0, cx = ci % CX, cy = ci / CX % C, cz = ci / (CX * C);
  const int gx = BX * bx - 1 + cx, gy = 2 * by - 1 + cy, gz = 2 * bz - 1 + cz;
  const bool cell = gx >= 0 && gy >= 0 && gz >= 0;
  // mu h; zero for cells outside the mesh, whose points are all zero
  const I mc = cell ? gx + I(n) * (gy + I(n) * gz) : 0;
  T mu_h = a.mu[MAP ? I(a.cell[mc]) : mc] / T(n);
  if (!cell) mu_h = T(0);
#pragma unroll
  for (int k = 0; k < KS; ++k)
    if (r0 < RP && r0 + RP * k < NR) buf(sq, sx + NX * (r0 + RP * k)) = v[k];
  __syncthreads();
  T w[27];
#pragma unroll
  for (int p = 0; p < 27; ++p)
    w[p] = buf(comp, (2 * cx + p % 3) + NX * ((2 * cy + p / 3 % 3) + N * (2 * cz + p / 9)));
  cellop::modes_all(w);
  auto put = [&](int s, T q) {
    if (live) ex(comp, s, ci) = q;
  };
  if (comp == 0) cellop::share_modes<0>(w, put);
  else if (comp == 1) cellop::share_modes<1>(w, put);
  else cellop::share_modes<2>(w, put);
  __syncthreads();
  auto modes = [&](auto e, auto j) { return ex(e, cellop::mode_slot(e, j), ci); };
  if (comp == 0) cellop::apply_component<0>(w, modes);
  else if (comp == 1) cellop::apply_component<1>(w, modes);
  else cellop::apply_component<2>(w, modes);
  __syncthreads();
  if (live) {
#pragma unroll
    for (int p = 0; p < 27; ++p) mem[(comp * 27 + p) * kCells + ci] = mu_h * w[p];
  }
  __syncthreads();
  // A x of component q at box point l: along each axis a point on a cell edge
  // (even) takes node 2 of one cell and node 0 of the next (not computed past
  // the brick's last point: top), else node 1 of one
  auto sum = [&](int q, int lx, int ly, int lz, bool top0, bool top1, bool top2) {
    const int l[3] = {lx, ly, lz};
    const bool top[3] = {top0, top1, top2};
    constexpr int step[3] = {1, CX, CX * C}, node[3] = {1, 3, 9};
    int at = q * 27 * kCells, up[3];
    bool one[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const bool odd = l[e] & 1;
      one[e] = odd || top[e];
      at += (odd ? l[e] >> 1 : (l[e] >> 1) - 1) * step[e] + (odd ? 1 : 2) * node[e] * kCells;
      up[e] = one[e] ? 0 : step[e] - 2 * node[e] * kCells;
    }
    T ax = T(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const T r = mem[at + ((s & 1) ? up[0] : 0) + ((s & 2) ? up[1] : 0) + ((s & 4) ? up[2] : 0)];
      const bool use = !(((s & 1) && one[0]) || ((s & 2) && one[1]) || ((s & 4) && one[2]));
      ax += use ? r : T(0);
    }
    return ax;
  };
  auto finish = [&](I i, T ax, bool fx, T xe, T be, T me, T de) {
    if (fx) ax = xe;
    if constexpr (OP == Op::Apply) {
      a.y[i] = ax;
    } else if constexpr (OP == Op::Add) {
      if (!fx) a.y[i] = de + ax;
    } else if constexpr (OP == Op::Residual) {
      a.y[i] = be - ax;
    } else {
      T dn = a.beta * me * (be - ax);
      if constexpr (OP == Op::First) dn = a.alpha * xe + dn;
      if constexpr (OP == Op::Step || OP == Op::Last) dn = a.alpha * de + dn;
      if constexpr (OP != Op::Last) a.d[i] = dn;
      a.y[i] = xe + dn;
    }
  };
#pragma unroll
  for (int e = 0; e < E; ++e)
    finish(own[e], sum(oq, t / 3 % 4 + 4 * e + 2, oy + 2, oz + 2, false, false, false), dir[e], x[e], b[e], mi[e], d[e]);
  // the closing planes belong to the last bricks (fixed throughout under u = 0)
  if ((OP == Op::Add && !MAP) || (bx < nbx - 1 && by < nb - 1 && bz < nb - 1)) return;
  constexpr int WX = 2 * BX + 1, W = 5;
  for (int e = t; e < 3 * WX * W * W; e += kThreads) {
    const int q = e % 3, lx = e / 3 % WX, ly = e / (3 * WX) % W, lz = e / (3 * WX * W);
    const bool c0 = lx == WX - 1, c1 = ly == W - 1, c2 = lz == W - 1;
    const bool mine = (c0 && bx == nbx - 1) || (c1 && by == nb - 1) || (c2 && bz == nb - 1);
    const bool other = (c0 && bx < nbx - 1) || (c1 && by < nb - 1) || (c2 && bz < nb - 1);
    if (!mine || other) continue;
    const I i = entry(X0 + lx, Y0 + ly, Z0 + lz, q);
    const bool fx = fixed(X0 + lx, Y0 + ly, Z0 + lz, q);
    T be = T(0), me = T(0), de = T(0), xe;
    if constexpr (OP != Op::Apply && OP != Op::Add) be = a.b[i];
    if constexpr (is_update<OP>) me = a.minv[i];
    if constexpr (OP == Op::Step || OP == Op::Last) de = a.d[i];
    if constexpr (OP == Op::Add) de = a.y[i];
    if constexpr (OP == Op::First) xe = me * be * a.it0;
    else xe = a.x[i];
    T ax = T(0);
    if constexpr (MAP) ax = sum(q, lx + 2, ly + 2, lz + 2, c0, c1, c2);
    finish(i, ax, fx, xe, be, me, de);
  }
}

}  // namespace owner
}  // namespace mfgmg
