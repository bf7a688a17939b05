// Elimination of a 32 x 32 Hermitian block in the registers of one workgroup, for the Cholesky factor of a panel's
// diagonal block and of a Gram matrix.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

namespace gwi {

// 1 / x for a positive finite x: the hardware estimate refined by two Newton steps r <- r + r (1 - x r), each of which
// squares the relative error (within an ulp or two of the rounded quotient); three dependent operations fewer
// than the correctly rounded division
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int i = 0; i < 2; ++i) r = fma(r, fma(-x, r, 1.0), r);
  return r;
}

// z / r for a positive finite r with ir = rcp_nr(r): the quotient's remainder is added once, which leaves the rounded
// quotient where z ir alone has a second rounding
__device__ __forceinline__ double div_nr(double z, double r, double ir) {
  const double q = z * ir;
  return fma(fma(-q, r, z), ir, q);
}

// v of lane K of each row of 16 lanes, in all its lanes (DPP row_newbcast)
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  const int2 u = __builtin_bit_cast(int2, v);
  const int2 b = make_int2(__builtin_amdgcn_update_dpp(0, u.x, 0x150 + K, 0xf, 0xf, true),
                           __builtin_amdgcn_update_dpp(0, u.y, 0x150 + K, 0xf, 0xf, true));
  return __builtin_bit_cast(double, b);
}

// f(integral_constant<int, J>) for J = 0, 1, ...: loop bodies whose index must be a constant
template <typename F, int... J>
__device__ __forceinline__ void static_for(F &&f, std::integer_sequence<int, J...>) {
  (f(std::integral_constant<int, J>{}), ...);
}

// Unblocked right-looking elimination of the whole Hermitian block, A = Lu D Lu^H with Lu unit lower: step j
// subtracts p_j(i) row_j(m) / d_j from every entry (i, m) below it, with p_j column j, row_j = p_j^H and d_j
// the pivot.  The same step applies Lu's j-th elimination to X (started as I): row i > j loses p_j(i) / d_j
// times row j of X, on the columns m <= j where that row is non-zero.  After the last step X = Lu^-1, and
// L = Lu D^1/2, L^-1 = D^-1/2 X follow by scaling.  Column m of A changes only in the steps j < m and
// column m of X only in the steps j >= m, so A and X share the registers: X's column takes the place of
// A's in step m, and row j of both together is one row of 32 entries.
//
// The steps are one latency chain, so they are laid out for few instructions and little LDS
// traffic per step: lane (c, m) = (tid / 16, tid % 16) of the 512 holds the entries (c, m) and (c, 16 + m) in z.  A
// row of the block is then one row of 16 lanes, in which p_j(c) is a register broadcast (DPP) from lane j % 16; the
// row of the pivot, divided by it, goes through LDS (w[j], a row of its own for every step, so one
// barrier per step orders the writes before the reads), written by the wave that holds it and read as two
// words of 16 bytes per lane by the waves that still have rows below it.  inv(d) stands for 1 / d; pivots
// that are not positive are the caller's to find.  About 450 cycles per step.
//
// Out: w[j][m] = row_j(m) inv(d_j), A's entries right of the diagonal, X's on it (X_jj = 1) and left of it; dv[j] = d_j;
// for j < n, complete after the caller's next barrier; row = row_c(m) and row_c(16 + m) of the lane's own row c < n, as
// they were before inv(d_c), for callers that scale them by another factor.  wave is the uniform tid / 64.
template <typename Inv>
__device__ __forceinline__ void eliminate32(double2 (&z)[2], double2 (&row)[2], double2 (*__restrict__ w)[32],
                                            double *__restrict__ dv, int wave, int n, Inv inv) {
  const int m = threadIdx.x % 16, c = threadIdx.x / 16;    // the wave's rows are 4 wave ... 4 wave + 3
  double2 p;                                               // p_j(c)
  // p of step j, X's column in place of A's, and row j of w by the wave that holds it
  auto pivot_row = [&](auto jc) {
    constexpr int j = decltype(jc)::value;
    p = make_double2(row_bcast<j % 16>(z[j / 16].x), row_bcast<j % 16>(z[j / 16].y));
    if (m == j % 16) z[j / 16] = make_double2(c == j ? 1.0 : 0.0, 0.0);
    if (wave == j / 4) {
      if (c == j) {
        const double dinv = inv(p.x);
        w[j][m] = make_double2(z[0].x * dinv, z[0].y * dinv);
        w[j][16 + m] = make_double2(z[1].x * dinv, z[1].y * dinv);
        if (m == 0) dv[j] = p.x;
        row[0] = z[0];
        row[1] = z[1];
      }
    }
  };
  auto step = [&](auto jc) {
    constexpr int j = decltype(jc)::value;
    if (j + 1 >= n) return;                                // uniform
    __syncthreads();
    if (wave >= (j + 1) / 4) {                             // this wave has rows below j
      if (wave == (j + 1) / 4) __builtin_amdgcn_s_setprio(3);      // every wave waits for the next pivot row
      const double2 q0 = w[j][m], q1 = w[j][16 + m];
      // The whole term first, then one subtraction: two chained fma round twice at the size of z, which is the larger
      // of the two where the diagonal dominates (eps^-1 19% further from the exact inverse at N = 130 and 6% at 410,
      // with the block's partial sums subtracted one by one; 410 rows took 337 us so, and 341 us as it is).
      z[0].x -= fma(p.x, q0.x, -(p.y * q0.y));
      z[0].y -= fma(p.x, q0.y, p.y * q0.x);
      z[1].x -= fma(p.x, q1.x, -(p.y * q1.y));
      z[1].y -= fma(p.x, q1.y, p.y * q1.x);
      pivot_row(std::integral_constant<int, j + 1>{});
    }
  };
  pivot_row(std::integral_constant<int, 0>{});
  static_for(step, std::make_integer_sequence<int, 31>{});
}

}  // namespace gwi
