// Per-cell Q2 strain-rate operator in Legendre modes (device code).
//
// Paper: A_ij = int 2 mu eps(phi_i) : eps(phi_j) (Sec. 2.1).  On an
// axis-aligned cube of side h with cell-constant mu the cell contribution is
// mu h K_hat u_cell, and the 3x3x3 Gauss rule of the method integrates K_hat
// exactly, so any exact evaluation gives the same operator.  Here each axis
// goes from the nodal basis {0, 1/2, 1} to the Legendre polynomials P0, P1,
// P2 of 2 t - 1 (value at the nodes: 1 1 1 | -1 0 1 | 1 -1/2 1), in which the
// 1D mass matrix is diag(1, 1/3, 1/5), the stiffness diag(0, 4, 12), and a
// derivative maps P1 -> 2 P0, P2 -> 6 P1.  K_hat then has 150 nonzeros out of
// 6561: 78 on the diagonal (the three rigid translations have none) and 72
// from d_d v_c d_c u_d, c != d.  A transform of a line of three values takes
// four operations, so a cell takes 324 + 150 + 324 = 798 operations; the
// sum-factorised evaluation at the 27 Gauss points took ~2,360, at
// one issue slot each the larger part of every cell kernel's issue time (one
// application: 64^3 FP64 65.7 -> 56.0 us, 128^3 FP32 256 -> 229 us, adaptive
// 32^3 + 2 FP64 387 -> 300 us).  Every index is a compile-time constant, so
// the 81 values live in registers and are transformed in place.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

namespace mfgmg {
namespace cellop {

// ---- Legendre modes of a line of nodal values
// a0, a1, a2 -> 6 c0, 2 c1, 3 c2 (c: coefficients of P0, P1, P2)
template <typename T>
__device__ __forceinline__ void to_modes(T& a0, T& a1, T& a2) {
  const T s = a0 + a2, p = a2 - a0;
  const T q = s - T(2) * a1, m = s + T(4) * a1;
  a0 = m;
  a1 = p;
  a2 = q;
}
// the transpose, for mode residuals scaled by 4/6, 1/2, 1/3
template <typename T>
__device__ __forceinline__ void to_nodes(T& m, T& p, T& q) {
  const T t = T(0.25) * m + q;
  const T y1 = m - T(2) * q;
  m = t - p;
  q = t + p;
  p = y1;
}

// the same along every line of a 27-value tensor (x fastest), axis by axis
template <typename T>
__device__ __forceinline__ void modes_all(T* v) {
#pragma unroll
  for (int l = 0; l < 9; ++l) to_modes(v[3 * l], v[3 * l + 1], v[3 * l + 2]);
#pragma unroll
  for (int z = 0; z < 3; ++z)
#pragma unroll
    for (int x = 0; x < 3; ++x) to_modes(v[x + 9 * z], v[x + 3 + 9 * z], v[x + 6 + 9 * z]);
#pragma unroll
  for (int l = 0; l < 9; ++l) to_modes(v[l], v[l + 9], v[l + 18]);
}
template <typename T>
__device__ __forceinline__ void nodes_all(T* v) {
#pragma unroll
  for (int l = 0; l < 9; ++l) to_nodes(v[l], v[l + 9], v[l + 18]);
#pragma unroll
  for (int z = 0; z < 3; ++z)
#pragma unroll
    for (int x = 0; x < 3; ++x) to_nodes(v[x + 9 * z], v[x + 3 + 9 * z], v[x + 6 + 9 * z]);
#pragma unroll
  for (int l = 0; l < 9; ++l) to_nodes(v[3 * l], v[3 * l + 1], v[3 * l + 2]);
}

// ---- K_hat between modes, with the scalings of to_modes and to_nodes
constexpr double mode_mass(int i) { return i == 0 ? 1.0 : i == 1 ? 1.0 / 3.0 : 0.2; }
constexpr double mode_stiff(int i) { return i == 0 ? 0.0 : i == 1 ? 4.0 : 12.0; }
constexpr double mode_in(int i) { return i == 0 ? 1.0 / 6.0 : i == 1 ? 0.5 : 1.0 / 3.0; }
constexpr double mode_out(int i) { return i == 0 ? 4.0 / 6.0 : i == 1 ? 0.5 : 1.0 / 3.0; }
constexpr int mode_axis(int i, int axis) { return axis == 0 ? i % 3 : axis == 1 ? i / 3 % 3 : i / 9; }
constexpr int mode_step(int axis) { return axis == 0 ? 1 : axis == 1 ? 3 : 9; }
constexpr double mode_scale(int i, int j) {
  double s = 1.0;
  for (int a = 0; a < 3; ++a) s *= mode_out(mode_axis(i, a)) * mode_in(mode_axis(j, a));
  return s;
}
// diagonal entry of mode i, component c: the derivative along axis c counts twice
constexpr double mode_diag(int c, int i) {
  double s = 0.0;
  for (int d = 0; d < 3; ++d) {
    double f = (d == c ? 2.0 : 1.0) * mode_stiff(mode_axis(i, d));
    for (int e = 0; e < 3; ++e)
      if (e != d) f *= mode_mass(mode_axis(i, e));
    s += f;
  }
  return s * mode_scale(i, i);
}
// int d_d v_c d_c u_d: test mode i of component c sees mode j of component d,
// j = i raised by one along c and lowered by one along d
constexpr bool mode_couples(int c, int d, int i) { return mode_axis(i, c) < 2 && mode_axis(i, d) > 0; }
constexpr int mode_partner(int c, int d, int i) { return i + mode_step(c) - mode_step(d); }
constexpr double mode_coupling(int c, int d, int i) {
  const int ic = mode_axis(i, c), id = mode_axis(i, d), e = 3 - c - d;
  const double up = ic == 0 ? 2.0 : 6.0, down = id == 1 ? 2.0 : 6.0;
  return up * down * mode_mass(ic) * mode_mass(id - 1) * mode_mass(mode_axis(i, e)) *
         mode_scale(i, mode_partner(c, d, i));
}

// row of K_hat: mode i of component C; u(d, j) gives mode j of component d
template <int C, int I, typename T, typename U>
__device__ __forceinline__ T mode_row(const U& u) {
  constexpr int D = (C + 1) % 3, E = (C + 2) % 3;
  T r = I == 0 ? T(0) : T(mode_diag(C, I)) * u(std::integral_constant<int, C>(), std::integral_constant<int, I>());
  if constexpr (mode_couples(C, D, I))
    r += T(mode_coupling(C, D, I)) *
         u(std::integral_constant<int, D>(), std::integral_constant<int, mode_partner(C, D, I)>());
  if constexpr (mode_couples(C, E, I))
    r += T(mode_coupling(C, E, I)) *
         u(std::integral_constant<int, E>(), std::integral_constant<int, mode_partner(C, E, I)>());
  return r;
}

// The modes split by parity into eight blocks that K_hat does not couple:
// block B (bit a: parity along axis a) holds the modes of component c whose
// parities are B with bit c flipped, 6 to 12 values, so the product runs in
// place with one block's inputs beside the 81 values.
constexpr bool in_parity_block(int B, int c, int i) {
  for (int a = 0; a < 3; ++a)
    if ((mode_axis(i, a) & 1) != (((B >> a) & 1) ^ (a == c ? 1 : 0))) return false;
  return true;
}
template <int B, int K, typename T>
__device__ __forceinline__ void parity_entry(const T (&U)[3][27], T (&R)[3][27]) {
  constexpr int C = K / 27, I = K % 27;
  if constexpr (in_parity_block(B, C, I))
    R[C][I] = mode_row<C, I, T>([&](auto d, auto j) { return U[decltype(d)::value][decltype(j)::value]; });
}
template <int B, int K, typename T>
__device__ __forceinline__ void parity_store(const T (&R)[3][27], T (&U)[3][27]) {
  constexpr int C = K / 27, I = K % 27;
  if constexpr (in_parity_block(B, C, I)) U[C][I] = R[C][I];
}
template <int B, typename T, int... K>
__device__ __forceinline__ void parity_block(T (&U)[3][27], std::integer_sequence<int, K...>) {
  T R[3][27];
  (parity_entry<B, K>(U, R), ...);
  (parity_store<B, K>(R, U), ...);
}
template <typename T, int... B>
__device__ __forceinline__ void all_blocks(T (&U)[3][27], std::integer_sequence<int, B...>) {
  (parity_block<B>(U, std::make_integer_sequence<int, 81>()), ...);
}

// U[c][a]: nodal values of component c at local node a (x fastest) on input,
// K_hat U on return; the caller multiplies by mu h.
template <typename T>
__device__ __forceinline__ void apply_cell(T (&U)[3][27]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) modes_all(U[c]);
  all_blocks(U, std::make_integer_sequence<int, 8>());
#pragma unroll
  for (int c = 0; c < 3; ++c) nodes_all(U[c]);
}

// Component C of K_hat U where one thread holds one component: w, this
// component's modes (modes_all applied), on return its nodal results; modes
// of the other components are fetched with get(component, mode) (24 of them;
// both arguments are integral constants).
// Of a component's modes the other components read 16: those at most linear
// along the component's own axis and not constant along both others.
// mode_slot: a mode's rank among them (-1: not read).
constexpr int kSharedModes = 16;
constexpr bool mode_shared(int c, int i) {
  return mode_axis(i, c) < 2 && (mode_axis(i, (c + 1) % 3) > 0 || mode_axis(i, (c + 2) % 3) > 0);
}
constexpr int mode_slot(int c, int i) {
  if (!mode_shared(c, i)) return -1;
  int s = 0;
  for (int j = 0; j < i; ++j) s += mode_shared(c, j) ? 1 : 0;
  return s;
}

// put(slot, value) for the modes of component C that the others read
template <int C, int I, typename T, typename Put>
__device__ __forceinline__ void share_mode(const T (&w)[27], const Put& put) {
  if constexpr (mode_shared(C, I)) put(mode_slot(C, I), w[I]);
}
template <int C, typename T, typename Put, int... I>
__device__ __forceinline__ void share_modes(const T (&w)[27], const Put& put, std::integer_sequence<int, I...>) {
  (share_mode<C, I>(w, put), ...);
}
template <int C, typename T, typename Put>
__device__ __forceinline__ void share_modes(const T (&w)[27], const Put& put) {
  share_modes<C>(w, put, std::make_integer_sequence<int, 27>());
}

template <int C, typename T, typename Get, int... I>
__device__ __forceinline__ void component_rows(T (&w)[27], const Get& get, std::integer_sequence<int, I...>) {
  T r[27];
  ((r[I] = mode_row<C, I, T>([&](auto d, auto j) {
      if constexpr (decltype(d)::value == C) return w[decltype(j)::value];
      else return get(d, j);
    })), ...);
  ((w[I] = r[I]), ...);
}
template <int C, typename T, typename Get>
__device__ __forceinline__ void apply_component(T (&w)[27], const Get& get) {
  component_rows<C>(w, get, std::make_integer_sequence<int, 27>());
  nodes_all(w);
}

// ---- Gauss points (right-hand side assembly)
// Interpolation from the Q2 nodes {0, 1/2, 1} to the Gauss points
// 1/2 -+ g, 1/2, g = sqrt(15)/10:
//   N = [[0.3+g, 0.4, 0.3-g], [0, 1, 0], [0.3-g, 0.4, 0.3+g]].
constexpr double kG = 0.38729833462074168852;
constexpr double kNa = 0.3 + kG;
constexpr double kNb = 0.3 - kG;

template <typename T>
__device__ __forceinline__ void interp3_t(T& v0, T& v1, T& v2) {
  const T a = T(kNa), b = T(kNb), f = T(0.4);
  const T o0 = a * v0 + b * v2;
  const T o1 = v1 + f * (v0 + v2);
  const T o2 = b * v0 + a * v2;
  v0 = o0;
  v1 = o1;
  v2 = o2;
}

// transpose of N x N x N on a 27-value tensor, x fastest
template <typename T>
__device__ __forceinline__ void interp_all_t(T* v) {
#pragma unroll
  for (int l = 0; l < 9; ++l) interp3_t(v[l], v[l + 9], v[l + 18]);
#pragma unroll
  for (int z = 0; z < 3; ++z)
#pragma unroll
    for (int x = 0; x < 3; ++x) interp3_t(v[x + 9 * z], v[x + 3 + 9 * z], v[x + 6 + 9 * z]);
#pragma unroll
  for (int l = 0; l < 9; ++l) interp3_t(v[3 * l], v[3 * l + 1], v[3 * l + 2]);
}

}  // namespace cellop
}  // namespace mfgmg
