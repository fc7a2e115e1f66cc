// rhs_common.h -- device building blocks of the BSSN right-hand sides and
// constraints: gridfunction indices, stencil loads, difference weights.
//
// Notation follows Sec. 2.1-2.2 of arXiv:2505.00097: eps_ij = gammabar_ij -
// gammahat_ij, Delta^k_ij = Gammabar^k_ij - Gammahat^k_ij, W = exp(-2 phi),
// rescaled variables h_ij = eps_ij/(S_i S_j), lambda^i = S_i Lambdabar^i, ...
#pragma once

#include "bhah_internal.h"

namespace bhah {

enum {
  G_ADD00 = 0, G_ALPHA = 6, G_BETU0 = 7, G_CF = 10, G_HDD00 = 11, G_LAMU0 = 17,
  G_TRK = 20, G_VETU0 = 21
};

// symmetric pair (i,j) -> 0..5 in the order 00,01,02,11,12,22
__host__ __device__ constexpr int sy(int i, int j) {
  return i <= j ? (i * (5 - i)) / 2 + j : (j * (5 - j)) / 2 + i;
}

// Stencil loads through buffer descriptors: one descriptor per group of four
// gridfunctions (base = the group's first element, range = its size in
// bytes), the gridfunction's place in its group and the wave-uniform part of
// the stencil offset as scalar offset, the per-lane part as vector offset.
// Few descriptors stay live (scalar registers are scarce in the stencil
// kernels); an access outside the group returns 0 instead of faulting.
// Grids are limited to 2^26 points so every offset fits 31 bits.
typedef unsigned int bhah_u2 __attribute__((ext_vector_type(2)));

typedef unsigned int bhah_u4 __attribute__((ext_vector_type(4)));

// two consecutive doubles (along i0) in one 16-byte load: a wave's vector
// memory pipeline moves twice the data per instruction
__device__ __forceinline__ void gf_ld2(const double* y, long long sgf, int g, unsigned voff, int soff, double& lo,
                                       double& hi) {
  const __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc((void*)(y + (g >> 2) * 4 * sgf), (short)0, (int)(4 * sgf * 8), 0x00020000);
  const bhah_u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff + (g & 3) * (int)(sgf * 8), 0);
  lo = __builtin_bit_cast(double, (unsigned long long)v.x | ((unsigned long long)v.y << 32));
  hi = __builtin_bit_cast(double, (unsigned long long)v.z | ((unsigned long long)v.w << 32));
}

__device__ __forceinline__ double gf_ld(const double* y, long long sgf, int g, unsigned voff, int soff) {
  const __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc((void*)(y + (g >> 2) * 4 * sgf), (short)0, (int)(4 * sgf * 8), 0x00020000);
  const bhah_u2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff + (g & 3) * (int)(sgf * 8), 0);
  return __builtin_bit_cast(double, v);
}

// Finite-difference weights of order N_FD = 2R (Sec. 3: N_G = R + 1 ghost
// layers, the extra layer for the upwinded advection stencils), as integers
// over a common denominator, unit spacing:
//   D f  = sum_{j=1..R} d1[j] (f_j - f_-j) / den1
//   D2 f = (sum_{j=1..R} d2[j] (f_j + f_-j) + d2[0] f_0) / den2
//   U f  = the centred first difference shifted one point upwind (UpW in
//          rhs_stencil.h), over den1
//   KO f = (sum_{j=1..R+1} ko[j] (f_j + f_-j) + ko[0] f_0) / kden, the
//          difference of order 2(R+1) scaled to the Fourier symbol
//          -sin^(2R+2)(theta/2) (Kreiss-Oliger dissipation of order 2R+1,
//          Sec. 4.1)
// R = 2: the 4th-order stencils; R = 4: the 8th-order ones of the
// production head-on run (Sec. 4.1).
template <int R>
struct FdW;
template <>
struct FdW<2> {
  static constexpr double d1[3] = {0.0, 8.0, -1.0}, den1 = 12.0;
  static constexpr double d2[3] = {-30.0, 16.0, -1.0}, den2 = 12.0;
  static constexpr double ko[4] = {-20.0, 15.0, -6.0, 1.0}, kden = 64.0;
};
template <>
struct FdW<4> {
  static constexpr double d1[5] = {0.0, 672.0, -168.0, 32.0, -3.0}, den1 = 840.0;
  static constexpr double d2[5] = {-14350.0, 8064.0, -1008.0, 128.0, -9.0}, den2 = 5040.0;
  static constexpr double ko[6] = {-252.0, 210.0, -120.0, 45.0, -10.0, 1.0}, kden = 1024.0;
};

// inverse of a symmetric matrix
__device__ __forceinline__ void sym_inverse(const double g[6], double gi[6]) {
  const double c00 = g[3] * g[5] - g[4] * g[4];
  const double c01 = g[2] * g[4] - g[1] * g[5];
  const double c02 = g[1] * g[4] - g[2] * g[3];
  const double det = g[0] * c00 + g[1] * c01 + g[2] * c02;
  const double id = 1.0 / det;
  gi[0] = c00 * id;
  gi[1] = c01 * id;
  gi[2] = c02 * id;
  gi[3] = (g[0] * g[5] - g[2] * g[2]) * id;
  gi[4] = (g[1] * g[2] - g[0] * g[4]) * id;
  gi[5] = (g[0] * g[3] - g[1] * g[1]) * id;
}

}  // namespace bhah
