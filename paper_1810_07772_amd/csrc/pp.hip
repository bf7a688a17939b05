// Plasmon-pole model of the dynamic inverse dielectric matrix (the paper's section on it):
//   S = sqrt(V) (eps^-1 - I) sqrt(V)            the polarization part of the static W
//   S = A diag(sigma) A^H                       Eq.(eigdecomp), the few most negative sigma
//   omega_a^2 = (A^H M A)_aa / |sigma_a|,  M(g,g') = V V' [(q+g).(q+g')] rho_{g-g'}   Eq.(ppfreq)
//   S(w) = sum_a A_a sigma_a omega_a^2 / (omega_a^2 - w^2) A_a^H                  Eq.(ppform)
// Kernels for the density and its transform, S and M, the products, small dense eigenproblems and
// orthonormalisation of the block iteration, and the pole-form evaluation (its large product is the complex
// FP64 MFMA GEMM).
#include <algorithm>

#include "elim32.h"
#include "gw_internal.h"

namespace gwi {

// rho(r) = occ sum_v |psi_v(r)|^2, written as complex (rho, 0) for the transform that follows
__global__ void density_kernel(const float2 *__restrict__ psi, int nv, int nr, double occ, double2 *__restrict__ rho) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nr) return;
  double a = 0.0;
  for (int v = 0; v < nv; ++v) {
    const float2 p = psi[(size_t)v * nr + r];
    a += (double)p.x * p.x + (double)p.y * p.y;
  }
  rho[r] = make_double2(occ * a, 0.0);
}

// One axis of the FP64 forward DFT on the full grid: out[.. k ..] = sum_i in[.. i ..] exp(-2 pi i k i / n_d).
// Lengths are at most 48, so each output is a direct sum; the phase comes from sincospi in FP64.
__global__ void dft_axis_f64_kernel(const double2 *__restrict__ in, double2 *__restrict__ out, int n1, int n2, int n3,
                                    int axis) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int nr = n1 * n2 * n3;
  if (idx >= nr) return;
  const int i3 = idx % n3, i2 = (idx / n3) % n2, i1 = idx / (n2 * n3);
  int n, k, stride, base;
  if (axis == 0) { n = n1; k = i1; stride = n2 * n3; base = idx - i1 * stride; }
  else if (axis == 1) { n = n2; k = i2; stride = n3; base = idx - i2 * stride; }
  else { n = n3; k = i3; stride = 1; base = idx - i3; }
  double re = 0.0, im = 0.0;
  for (int i = 0; i < n; ++i) {
    double sn, cs;
    sincospi(-2.0 * (double)((k * i) % n) / (double)n, &sn, &cs);
    const double2 x = in[base + i * stride];
    re += x.x * cs - x.y * sn;
    im += x.x * sn + x.y * cs;
  }
  out[idx] = make_double2(re, im);
}

// s = sv_g (eps_inv - delta) sv_g'
__global__ void screening_kernel(const double2 *__restrict__ ei, const double *__restrict__ sv, int ng, long long lds,
                                 double2 *__restrict__ s) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ng * ng) return;
  const int g = (int)(idx / ng), h = (int)(idx % ng);
  double2 e = ei[idx];
  if (g == h) e.x -= 1.0;
  const double f = sv[g] * sv[h];
  s[g * lds + h] = make_double2(f * e.x, f * e.y);
}

// m = V_g V_h (2pi/a)^2 [(q+m_g).(q+m_h)] rho[(m_g - m_h) mod n]
__global__ void sum_rule_kernel(const int *__restrict__ miller, int ng, double q0, double q1, double q2, double b,
                                const double *__restrict__ sv, const double2 *__restrict__ rho_g, int n1, int n2,
                                int n3, double2 *__restrict__ m) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ng * ng) return;
  const int g = (int)(idx / ng), h = (int)(idx % ng);
  const int *mg = miller + 3 * g, *mh = miller + 3 * h;
  const double dot = b * b * ((q0 + mg[0]) * (q0 + mh[0]) + (q1 + mg[1]) * (q1 + mh[1]) + (q2 + mg[2]) * (q2 + mh[2]));
  const double vg = sv[g] * sv[g], vh = sv[h] * sv[h];
  const int d1 = ((mg[0] - mh[0]) % n1 + n1) % n1, d2 = ((mg[1] - mh[1]) % n2 + n2) % n2,
            d3 = ((mg[2] - mh[2]) % n3 + n3) % n3;
  const double2 r = rho_g[((size_t)d1 * n2 + d2) * n3 + d3];
  const double f = vg * vh * dot;
  m[idx] = make_double2(f * r.x, f * r.y);
}

// Start block: entries uniform in [-1, 1) (real and imaginary parts) from SplitMix64 (Steele, Lea and
// Flood, 2014) of a counter, so the iteration is deterministic.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}
__global__ void start_block_kernel(double2 *__restrict__ x, int ng, int b, unsigned long long seed) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ng * b) return;
  const unsigned long long u = splitmix64(seed * 0x100000000ull + 2 * idx);
  const unsigned long long w = splitmix64(seed * 0x100000000ull + 2 * idx + 1);
  const double s = 1.0 / 9007199254740992.0;     // 2^-53
  x[idx] = make_double2(2.0 * (double)(u >> 11) * s - 1.0, 2.0 * (double)(w >> 11) * s - 1.0);
}

// ---- the block iteration's products: blocks are [ng][b] complex128 row-major, b <= 32 -----------------------
constexpr int JMAX = 32;         // largest block
typedef double f64x4 __attribute__((ext_vector_type(4)));

// part[z] = A B over k in split z, A [M][K] (read once, from memory) and B [K][N], N <= 32 (from cache).
// 64 rows per workgroup, 16 complex k per stage, so a workgroup has 16 KB of A in flight in registers while the
// FP64 MFMAs of the stage before run (k' = (k, re/im) as in zgemm_kernel: Re C += [Re A, Im A] . [Re B; -Im B],
// Im C += [Re A, Im A] . [Im B; Re B]); wave w owns rows 16 w .. +15 and all 32 columns.  Bound by memory and the
// matrix cores alike (16 bytes and 256 flop per entry of A).  3071 x 3071 by 32 columns: 103 us in the 64 x 64 tiles
// of zgemm_kernel, half of whose columns are padding here, 59 us so with one stage of loads in flight, 50 us with two
// and no branch between a load and its use.
constexpr int TPM = 64, TPK = 16;
__global__ __launch_bounds__(256) void thin_product_kernel(int M, int N, int K, const double2 *__restrict__ A,
                                                           long long lda, const double2 *__restrict__ B, int ldb,
                                                           double2 *__restrict__ part, int kchunk) {
  constexpr int LA = TPM + 1, LB = JMAX + 1;      // odd strides: the transposing LDS writes spread over the banks
  __shared__ double sA[2][TPK][2][LA];
  __shared__ double sB[2][TPK][2][LB];            // [Re B; -Im B]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, kl = lane >> 4, li = lane & 15;
  const int row0 = blockIdx.x * TPM, k_beg = blockIdx.y * kchunk, k_end = min(K, k_beg + kchunk);
  double2 va[2][4], vb[2][2];                     // the loads of two stages
  const int ar = tid / TPK, ak = tid % TPK;       // A: rows ar + 16 i, offset ak
  const int bc = tid % JMAX, bk = tid / JMAX;     // B: k offsets bk + 8 i, column bc
  // Every stage loads, without a branch (behind one the compiler waits for all outstanding loads): elements outside
  // the operands read an address inside, and zero takes their place on the way to LDS.
  auto gload = [&](int k0, auto setc) {
    constexpr int set = decltype(setc)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i) va[set][i] = A[(long long)min(row0 + ar + 16 * i, M - 1) * lda + min(k0 + ak, k_end - 1)];
#pragma unroll
    for (int i = 0; i < 2; ++i) vb[set][i] = B[(long long)min(k0 + bk + 8 * i, k_end - 1) * ldb + min(bc, N - 1)];
  };
  auto lstore = [&](int k0, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    if (k0 + TPK > k_end || N < JMAX) {           // uniform; rows past M are not stored
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k0 + ak >= k_end) va[buf][i] = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (bc >= N || k0 + bk + 8 * i >= k_end) vb[buf][i] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sA[buf][ak][0][ar + 16 * i] = va[buf][i].x;
      sA[buf][ak][1][ar + 16 * i] = va[buf][i].y;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      sB[buf][bk + 8 * i][0][bc] = vb[buf][i].x;
      sB[buf][bk + 8 * i][1][bc] = -vb[buf][i].y;
    }
  };
  f64x4 accR[2], accI[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) { accR[c][e] = 0.0; accI[c][e] = 0.0; }
  const int comp = kl & 1, kh = kl >> 1;
  const unsigned long long flip = comp ? 0ull : 0x8000000000000000ull;   // [Im B; Re B] = [-X_1; X_0]
  // Operands are read AHEAD steps of two k before they are multiplied, the barrier stands before a stage's last AHEAD
  // steps, and the reads past the last stage are unused, as in zgemm_kernel.
  struct Ops { double a, x[2], y[2]; };
  constexpr int AHEAD = 2, ST = TPK / 2;
  auto rd = [&](int buf, int s) {
    const int kk = 2 * s + kh;
    Ops o;
    o.a = sA[buf][kk][comp][16 * wave + li];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      o.x[c] = sB[buf][kk][comp][16 * c + li];
      o.y[c] = sB[buf][kk][comp ^ 1][16 * c + li];
    }
    return o;
  };
  Ops q[AHEAD];
  auto stage = [&](int k0, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    gload(k0 + 2 * TPK, bufc);
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      if (s == ST - AHEAD) {
        if (k0 + TPK < k_end) lstore(k0 + TPK, std::integral_constant<int, buf ^ 1>{});
        __syncthreads();
      }
      const Ops o = q[s % AHEAD];
      q[s % AHEAD] = s + AHEAD < ST ? rd(buf, s + AHEAD) : rd(buf ^ 1, s + AHEAD - ST);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double yv = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, o.y[c]) ^ flip);
        accR[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a, o.x[c], accR[c], 0, 0, 0);
        accI[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a, yv, accI[c], 0, 0, 0);
      }
    }
  };
  if (k_beg < k_end) {
    gload(k_beg, std::integral_constant<int, 0>{});
    gload(k_beg + TPK, std::integral_constant<int, 1>{});
    lstore(k_beg, std::integral_constant<int, 0>{});
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < AHEAD; ++s) q[s] = rd(0, s);
  for (int k0 = k_beg; k0 < k_end; k0 += 2 * TPK) {
    stage(k0, std::integral_constant<int, 0>{});
    if (k0 + TPK < k_end) stage(k0 + TPK, std::integral_constant<int, 1>{});
  }
  double2 *out = part + (size_t)blockIdx.y * M * N;
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = row0 + 16 * wave + 4 * e + kl, col = 16 * c + li;
      if (row < M && col < N) out[(size_t)row * N + col] = make_double2(accR[c][e], accI[c][e]);
    }
}

// Splits of K: three workgroups per CU (their LDS fits; at 3071 rows, before the second stage of loads, 58.6 us against
// 67.9 with two and 77.6 with one and a half), at least four stages each.
static int thin_splits(int M, int K) {
  const int tiles = (M + TPM - 1) / TPM;
  return std::max(1, std::min(768 / tiles, K / (4 * TPK)));
}
size_t thin_part_elems(int M, int N, int K) { return (size_t)thin_splits(M, K) * M * N; }

// The share of X^H Y of the rows [blockIdx.x chunk, +chunk) into gpart[block].  Up to GRAM_ROWS rows of both at a
// time in LDS, all their loads in flight together; each of eight waves forms the real or imaginary part of one
// 16 x 16 tile on the FP64 MFMA, with k' = (row, re/im): Re = [Re X; Im X]^T [Re Y; Im Y],
// Im = [Re X; Im X]^T [Im Y; -Re Y].  Bound by latency, and so is its consumer, one workgroup that reads every
// partial matrix: the split is the one that keeps their sum shortest.  3071 rows, b = 32: 64 blocks of
// 48 rows on the vector units took 8.6 us, their sum 12 us of the consumer's; 32 of 96 rows 6.5 us and 7 (48 blocks
// 5.5 and 10, 24 blocks 8.7 and 6).  From 3073 rows on every block makes a second pass: 7.9 us there and 8.9 at
// 4067; more blocks of one pass each would lengthen the consumer's sum by as much.
constexpr int GRAM_ROWS = 96;
constexpr int GRAM_BLOCKS = 32;
__global__ __launch_bounds__(512) void block_gram_kernel(const double2 *__restrict__ x, const double2 *__restrict__ y,
                                                         int ng, int b, int chunk, double2 *__restrict__ gpart) {
  __shared__ double2 sx[GRAM_ROWS][JMAX + 1], sy[GRAM_ROWS][JMAX + 1];
  static_assert(JMAX == 32, "two tiles a side");
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int kl = lane >> 4, li = lane & 15, comp = kl & 1, kh = kl >> 1;
  const int ti = 16 * (wave & 1), tj = 16 * ((wave >> 1) & 1), im = wave >> 2;
  const unsigned long long flip = comp && im ? 0x8000000000000000ull : 0ull;
  const int r_beg = blockIdx.x * chunk, r_end = min(ng, r_beg + chunk);
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int r0 = r_beg; r0 < r_end; r0 += GRAM_ROWS) {
    if (r0 != r_beg) __syncthreads();
    const int i = tid % JMAX;
    double2 xv[GRAM_ROWS / 16], yv[GRAM_ROWS / 16];
#pragma unroll
    for (int h = 0; h < GRAM_ROWS / 16; ++h) {
      const int r = r0 + tid / JMAX + 16 * h;
      xv[h] = yv[h] = make_double2(0.0, 0.0);
      if (r < r_end && i < b) {
        const size_t at = (size_t)r * b + i;
        xv[h] = x[at];
        yv[h] = y[at];
      }
    }
#pragma unroll
    for (int h = 0; h < GRAM_ROWS / 16; ++h) {
      sx[tid / JMAX + 16 * h][i] = xv[h];
      sy[tid / JMAX + 16 * h][i] = yv[h];
    }
    __syncthreads();
    if (ti < b && tj < b) {                              // uniform over the wave
      const double *px = &reinterpret_cast<const double *>(&sx[kh][ti + li])[comp];
      const double *py = &reinterpret_cast<const double *>(&sy[kh][tj + li])[comp ^ im];
      const int groups = (min(GRAM_ROWS, r_end - r0) + 15) / 16;
      for (int g = 0; g < groups; ++g) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {                    // two rows each
          const int at = (16 * g + 2 * t) * 2 * (JMAX + 1);
          const double yy = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, py[at]) ^ flip);
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(px[at], yy, acc, 0, 0, 0);
        }
      }
    }
  }
  // lane holds tile entry (4 e + kl, li) in register e
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = ti + 4 * e + kl, j = tj + li;
    if (i < b && j < b) reinterpret_cast<double *>(gpart + (size_t)blockIdx.x * b * b + i * b + j)[im] = acc[e];
  }
}

static int gram_chunk(int ng) {
  const int c = std::max(48, (ng + GRAM_BLOCKS - 1) / GRAM_BLOCKS);
  return (c + 15) / 16 * 16;
}
static int gram_blocks(int ng) { return (ng + gram_chunk(ng) - 1) / gram_chunk(ng); }
size_t gram_part_elems(int ng, int b) { return (size_t)gram_blocks(ng) * b * b; }

// Entries tid, tid + THREADS, ... (i JMAX + j each) of the sum of the partial Gram matrices, in block order, into
// g; entries outside b x b are zero.  32 loads are in flight per thread: one workgroup reads all parts, and
// eight at a time cost it 20 us of the factorisation's 29 us for 48 parts.
template <int THREADS>
__device__ __forceinline__ void gram_sum(const double2 *__restrict__ gpart, int nblk, int b,
                                         double2 (*__restrict__ g)[JMAX + 1]) {
  constexpr int NE = JMAX * JMAX / THREADS, U = 32 / NE;
  double2 a[NE];
  const double2 *src[NE];
  bool in[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int idx = threadIdx.x + e * THREADS, i = idx / JMAX, j = idx % JMAX;
    in[e] = i < b && j < b;
    src[e] = gpart + (in[e] ? i * b + j : 0);
    a[e] = make_double2(0.0, 0.0);
  }
  const size_t bb = (size_t)b * b;
  int q = 0;
  for (; q + U <= nblk; q += U) {
    double2 v[NE][U];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int k = 0; k < U; ++k) v[e][k] = src[e][(q + k) * bb];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int k = 0; k < U; ++k) {
        a[e].x += v[e][k].x;
        a[e].y += v[e][k].y;
      }
  }
  for (; q < nblk; ++q)
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const double2 v = src[e][q * bb];
      a[e].x += v.x;
      a[e].y += v.y;
    }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const int idx = threadIdx.x + e * THREADS;
    g[idx / JMAX][idx % JMAX] = in[e] ? a[e] : make_double2(0.0, 0.0);
  }
}

// ---- Hermitian Jacobi eigensolver for b <= 32, one workgroup ------------------------------------
// Cyclic two-sided Jacobi with the round-robin (circle) ordering: each round rotates m/2 disjoint
// index pairs at once.  For a pair (p, q) the rotation is J = [[c, s], [-conj(s), c]] with complex s:
// with d = (a_qq - a_pp) / 2 and r = sqrt(d^2 + |a_pq|^2), c = sqrt((1 + |d| / r) / 2) and
// s = sign(d) a_pq / (2 r c), two reciprocal square roots in all; A <- J^H A J, V <- V J.
// A round's time is its serial chain, so it has one barrier: thread (k, l) of the first four waves computes
// the rotation of pair l from A, takes that of pair k from the lane that holds it (its own row of 16 lanes
// has all 16 pairs), and applies both sides to the 2 x 2 block (pair k, pair l) in registers, from one
// copy of A in LDS to the other.  The other four waves apply the previous round's rotations to V meanwhile, at a
// lower wave priority, since they share the SIMDs.
// (With the rotations passed through LDS and one barrier each for them, the columns and the rows, a round took
// 2.4 us; about 0.55 us.)  At 3071 G and 16 modes the solves of the iteration went from 522 us each (two per
// iteration) to 102 us (one), 95 us with fewer partial matrices to add, and 91 us with the priority and the
// shorter square roots.  The matrix is the Hermitian part of the sum of nblk partial ones, [b][b] each.
// Eigenvalues are returned in descending order with their vectors as columns of z (row-major, leading dimension b).

// 1 / sqrt(x), x > 0 normal: the hardware estimate r (5e-8 relative) refined by r (1 + e / 2 + 3 e^2 / 8),
// e = 1 - x r^2, the binomial series to third order: 1.4e-16 at most over 2^20 values, as with two Newton
// steps, and two dependent operations fewer
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * r, r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}

// Sum of v over the 64 lanes of a wave.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Pair t of a round over m indices (m even): (round + t, round - t) modulo m - 1, with m - 1 in place of the
// second for t = 0; the next round's pair is one step on.
struct JacobiPair {
  int p, q, n;
  bool fixed;
  __device__ __forceinline__ JacobiPair(int t, int m) : p(t), q(t == 0 ? m - 1 : m - 1 - t), n(m - 1), fixed(t == 0) {}
  __device__ __forceinline__ void step() {
    p = p + 1 == n ? 0 : p + 1;
    if (!fixed) q = q + 1 == n ? 0 : q + 1;
  }
};

__global__ __launch_bounds__(512) void herm_jacobi_kernel(const double2 *__restrict__ gpart, int nblk, int b,
                                                          double *__restrict__ evals, double2 *__restrict__ z,
                                                          int max_sweeps) {
  __shared__ double2 A[2][JMAX][JMAX + 1];
  __shared__ double2 V[JMAX][JMAX + 1];
  __shared__ double rc[2][JMAX / 2];
  __shared__ double2 rs[2][JMAX / 2];
  __shared__ double red_off[8], red_all[8];
  __shared__ int perm[JMAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = (b + 1) & ~1;          // even size; a padding index has a zero row and column
  const int half = m / 2;
  gram_sum<512>(gpart, nblk, b, A[1]);
  for (int idx = tid; idx < JMAX * JMAX; idx += 512) {
    const int i = idx / JMAX, j = idx % JMAX;
    V[i][j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  for (int idx = tid; idx < JMAX * JMAX; idx += 512) {
    const int i = idx / JMAX, j = idx % JMAX;
    const double2 a = A[1][i][j], c = A[1][j][i];
    A[0][i][j] = make_double2(0.5 * (a.x + c.x), 0.5 * (a.y - c.y));     // Hermitian part
  }
  __syncthreads();
  int cur = 0, done = 0;               // A's current copy; rounds done
  if (wave < 4) __builtin_amdgcn_s_setprio(3);     // V's waves share their SIMDs and have time to spare
  const int l = lane & 15;             // this lane's pair of columns, and of rows (first four waves) k
  const int k = (wave & 3) * 4 + (lane >> 4), i0 = (wave & 3) * 8 + (lane >> 4) * 2;
  JacobiPair cols(l < half ? l : 0, m), rows(k < half ? k : 0, m);
  auto rotate_v = [&](int par) {       // by waves 4 to 7: the last round's rotations on rows i0, i0 + 1
    if (l >= half) return;
    const int p = cols.p, q = cols.q;
    const double c = rc[par][l];
    const double2 s = rs[par][l];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double2 x = V[i0 + h][p], y = V[i0 + h][q];
      // x' = c x - conj(s) y,  y' = s x + c y
      V[i0 + h][p] = make_double2(c * x.x - (s.x * y.x + s.y * y.y), c * x.y - (s.x * y.y - s.y * y.x));
      V[i0 + h][q] = make_double2(c * y.x + (s.x * x.x - s.y * x.y), c * y.y + (s.x * x.y + s.y * x.x));
    }
  };
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    // convergence: off-diagonal mass against the whole (norm below 1e-15 relative)
    double off = 0.0, all = 0.0;
    for (int idx = tid; idx < m * m; idx += 512) {
      const int i = idx / m, j = idx % m;
      const double2 v = A[cur][i][j];
      const double s2 = v.x * v.x + v.y * v.y;
      all += s2;
      if (i != j) off += s2;
    }
    off = wave_sum(off);
    all = wave_sum(all);
    if (lane == 0) { red_off[wave] = off; red_all[wave] = all; }
    __syncthreads();
    double o = 0.0, a = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) { o += red_off[w]; a += red_all[w]; }
    if (o <= 1e-30 * a || a == 0.0) break;       // the same in every thread
    for (int round = 0; round < m - 1; ++round) {
      if (wave < 4) {
        const int pl = cols.p, ql = cols.q, pk = rows.p, qk = rows.q;
        cols.step();
        rows.step();
        const double2(*Ac)[JMAX + 1] = A[cur];
        const double app = Ac[pl][pl].x, aqq = Ac[ql][ql].x;
        const double2 apq = Ac[pl][ql];
        double2 x00 = Ac[pk][pl], x01 = Ac[pk][ql], x10 = Ac[qk][pl], x11 = Ac[qk][ql];
        const double dd = 0.5 * (aqq - app);
        const double r2 = fma(dd, dd, fma(apq.x, apq.x, apq.y * apq.y));
        double c = 1.0;
        double2 s = make_double2(0.0, 0.0);
        if (r2 > 1e-290) {                        // below it the block is diagonal to any relative accuracy
          const double ir = rsqrt_nr(r2);
          const double c2 = fma(0.5 * fabs(dd), ir, 0.5);
          const double ic = rsqrt_nr(c2);
          c = c2 * ic;
          const double f = copysign(0.5 * ir * ic, dd);
          s = make_double2(f * apq.x, f * apq.y);
        }
        const int src = (lane & 48) | (k & 15);
        const double ck = __shfl(c, src, 64);
        const double2 sk = make_double2(__shfl(s.x, src, 64), __shfl(s.y, src, 64));
        if (lane < 16 && wave == 0 && l < half) { rc[done & 1][l] = c; rs[done & 1][l] = s; }
        if (k < half && l < half) {
          // columns: x_i0' = c x_i0 - conj(s) x_i1,  x_i1' = s x_i0 + c x_i1 (pair l), then rows with the
          // conjugates: x_0j' = ck x_0j - sk x_1j,  x_1j' = conj(sk) x_0j + ck x_1j (pair k)
          auto col = [&](double2 &u, double2 &v) {
            const double2 a0 = u, a1 = v;
            u = make_double2(c * a0.x - (s.x * a1.x + s.y * a1.y), c * a0.y - (s.x * a1.y - s.y * a1.x));
            v = make_double2(c * a1.x + (s.x * a0.x - s.y * a0.y), c * a1.y + (s.x * a0.y + s.y * a0.x));
          };
          auto row = [&](double2 &u, double2 &v) {
            const double2 a0 = u, a1 = v;
            u = make_double2(ck * a0.x - (sk.x * a1.x - sk.y * a1.y), ck * a0.y - (sk.x * a1.y + sk.y * a1.x));
            v = make_double2(ck * a1.x + (sk.x * a0.x + sk.y * a0.y), ck * a1.y + (sk.x * a0.y - sk.y * a0.x));
          };
          col(x00, x01);
          col(x10, x11);
          row(x00, x10);
          row(x01, x11);
          if (k == l) {                            // the rotated pair itself: real diagonal, zero off it
            x00.y = 0.0;
            x11.y = 0.0;
            x01 = make_double2(0.0, 0.0);
            x10 = make_double2(0.0, 0.0);
          }
          double2(*An)[JMAX + 1] = A[cur ^ 1];
          An[pk][pl] = x00;
          An[pk][ql] = x01;
          An[qk][pl] = x10;
          An[qk][ql] = x11;
        }
      } else if (done > 0) {
        rotate_v((done - 1) & 1);
        cols.step();
      }
      ++done;
      cur ^= 1;
      __syncthreads();
    }
  }
  if (done > 0 && wave >= 4) rotate_v((done - 1) & 1);
  // descending order of the b real eigenvalues (padding excluded): each one's rank
  if (tid < b) perm[tid] = tid;        // stays in range whatever the values are
  __syncthreads();
  if (tid < b) {
    const double mine = A[cur][tid][tid].x;
    int rank = 0;
    for (int j = 0; j < b; ++j) {
      const double v = A[cur][j][j].x;
      rank += v > mine || (v == mine && j < tid);
    }
    perm[rank] = tid;
  }
  __syncthreads();
  for (int idx = tid; idx < b * b; idx += 512) {
    const int i = idx / b, j = idx % b;
    z[(size_t)i * b + j] = V[i][perm[j]];
  }
  if (tid < b) evals[tid] = A[cur][perm[tid]][perm[tid]].x;
}

// ---- orthonormalisation of a block -------------------------------------------------------------------
// From the Gram matrix G = W^H W (sum of nblk partial ones) the upper triangular u with W u orthonormal: with
// D = diag(G), D^-1/2 G D^-1/2 = L L^H (Cholesky), u = D^-1/2 L^-H.  The columns of W, -S times the Ritz vectors,
// are close to orthogonal once the iteration settles, so W u stays close to them and the next Rayleigh-Ritz
// problem close to diagonal, which saves its Jacobi sweeps.  A direction whose squared length falls below
// 1e-14 of its column's once the earlier columns are projected out is dropped (u gets a zero column), as is a zero
// column.  One workgroup; the pivots are its time.
// (b = 32 from 64 partial matrices: 28.2 us with a column per lane, one pivot's column and row through LDS; 24.4 us in
// this form, 12 us of it the sum, and 16.7 us from 32.)
__global__ __launch_bounds__(512) void block_chol_kernel(const double2 *__restrict__ gpart, int nblk, int b,
                                                         double2 *__restrict__ u) {
  __shared__ double2 g[JMAX][JMAX + 1];
  __shared__ double2 w[JMAX][JMAX];
  __shared__ double dinv[JMAX], dv[JMAX];
  const int tid = threadIdx.x, m = tid % 16, c = tid / 16;
  static_assert(JMAX == 32, "eliminate32");
  gram_sum<512>(gpart, nblk, b, g);
  __syncthreads();
  if (tid < JMAX) {
    const double d = g[tid][tid].x;
    dinv[tid] = d > 0.0 && isfinite(d) ? 1.0 / sqrt(d) : 0.0;
  }
  __syncthreads();
  double2 z[2], row[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int k = 16 * h + m;
    const double2 a = g[c][k], t = g[k][c];
    const double f = 0.5 * dinv[c] * dinv[k];
    z[h] = make_double2(f * (a.x + t.x), f * (a.y - t.y));
  }
  eliminate32(z, row, w, dv, __builtin_amdgcn_readfirstlane(tid >> 6), b, [](double d) { return d > 1e-14 ? rcp_nr(d) : 0.0; });
  __syncthreads();
  // row c of the inverse of L is sqrt(d_c) w[c]; u[k][c] = dinv[k] conj(Linv[c][k])
  if (c < b) {
    const double d = dv[c], r = d > 1e-14 ? sqrt(d) : 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = 16 * h + m;
      if (k < b) {
        const double f = c >= k ? dinv[k] * r : 0.0;
        const double2 v = w[c][k];
        u[k * b + c] = make_double2(f * v.x, -f * v.y);
      }
    }
  }
}

// w = x z and, with y, t = y z for [ng][b] blocks and a b x b matrix z: 16 rows per workgroup, thread (row, column
// j) of 8 x 32 forms two rows of each.  With y also the rows' share of ||t_j - theta_j w_j||^2 into rpart[block][b].
constexpr int ROT_ROWS = 16;
__global__ __launch_bounds__(256) void block_rotate_kernel(const double2 *__restrict__ x, const double2 *__restrict__ y,
                                                           const double2 *__restrict__ z, int ng, int b,
                                                           const double *__restrict__ theta, double2 *__restrict__ w,
                                                           double2 *__restrict__ t, double *__restrict__ rpart) {
  __shared__ double2 sz[JMAX][JMAX];
  __shared__ double2 sx[ROT_ROWS][JMAX], sy[ROT_ROWS][JMAX];
  __shared__ double red[8][JMAX];
  const int tid = threadIdx.x, j = tid % JMAX, rg = tid / JMAX;
  const int r0 = blockIdx.x * ROT_ROWS;
  const double2 zero = make_double2(0.0, 0.0);
#pragma unroll
  for (int h = 0; h < JMAX / 8; ++h) {
    const int k = rg + 8 * h;
    sz[k][j] = (k < b && j < b) ? z[k * b + j] : zero;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int rr = rg + 8 * h, r = r0 + rr;
    const bool in = r < ng && j < b;
    sx[rr][j] = in ? x[(size_t)r * b + j] : zero;
    sy[rr][j] = in && y ? y[(size_t)r * b + j] : zero;
  }
  __syncthreads();
  double2 aw[2] = {zero, zero}, at[2] = {zero, zero};
#pragma unroll 4
  for (int k = 0; k < JMAX; ++k) {
    const double2 zv = sz[k][j];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double2 xv = sx[rg + 8 * h][k];
      aw[h].x += xv.x * zv.x - xv.y * zv.y;
      aw[h].y += xv.x * zv.y + xv.y * zv.x;
      if (y) {
        const double2 yv = sy[rg + 8 * h][k];
        at[h].x += yv.x * zv.x - yv.y * zv.y;
        at[h].y += yv.x * zv.y + yv.y * zv.x;
      }
    }
  }
  double res = 0.0;
  const double th = y && j < b ? theta[j] : 0.0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = r0 + rg + 8 * h;
    if (r < ng && j < b) {
      w[(size_t)r * b + j] = aw[h];
      if (y) {
        t[(size_t)r * b + j] = at[h];
        const double dx = at[h].x - th * aw[h].x, dy = at[h].y - th * aw[h].y;
        res += dx * dx + dy * dy;
      }
    }
  }
  if (!y) return;
  red[rg][j] = res;
  __syncthreads();
  if (rg == 0) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) a += red[q][j];
    if (j < b) rpart[(size_t)blockIdx.x * b + j] = a;
  }
}

// out[0] = max_{j < nm} ||y_j - theta_j x_j|| / theta_0 from the blocks' shares (one workgroup)
__global__ __launch_bounds__(256) void ritz_residual_kernel(const double *__restrict__ rpart, int nblk, int b,
                                                            const double *__restrict__ theta, int nm,
                                                            double *__restrict__ out) {
  __shared__ double red[8][JMAX];
  const int j = threadIdx.x % JMAX, g = threadIdx.x / JMAX;
  double a = 0.0;
#pragma unroll 8
  for (int q = g; q < nblk; q += 8) a += j < b ? rpart[(size_t)q * b + j] : 0.0;
  red[g][j] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double mx = 0.0;
    for (int i = 0; i < nm; ++i) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) s += red[q][i];
      mx = fmax(mx, sqrt(s));                        // a mode that is NaN does not count: its values are passed on
    }
    out[0] = theta[0] > 0.0 ? mx / theta[0] : (mx == 0.0 ? 0.0 : INFINITY);
  }
}

// y = alpha sum_z part[z] (the thin product's splits)
__global__ void thin_sum_kernel(const double2 *__restrict__ part, int kz, size_t n, double alpha,
                                double2 *__restrict__ y) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double2 a = make_double2(0.0, 0.0);
#pragma unroll 4
  for (int z = 0; z < kz; ++z) {
    const double2 v = part[(size_t)z * n + i];
    a.x += v.x;
    a.y += v.y;
  }
  y[i] = make_double2(alpha * a.x, alpha * a.y);
}

// sigma_a = -theta_a, omega_a = sqrt(Re(a^H t_a) / theta_a) with t = M A (one workgroup per mode)
__global__ void pp_frequency_kernel(const double2 *__restrict__ a, int lda, const double2 *__restrict__ t, int ldt,
                                    int ng, const double *__restrict__ theta, double *__restrict__ sigma,
                                    double *__restrict__ omega) {
  const int j = blockIdx.x;
  __shared__ double red[256];
  double s = 0.0;
  for (int g = threadIdx.x; g < ng; g += 256) {
    const double2 av = a[(size_t)g * lda + j], tv = t[(size_t)g * ldt + j];
    s += av.x * tv.x + av.y * tv.y;         // Re(conj(a) t)
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double th = theta[j];
    sigma[j] = -th;
    omega[j] = sqrt(fmax(red[0], 0.0) / th);
  }
}

// b[g][a] = A[g][a] * sigma_a omega_a^2 / (omega_a^2 - w^2)
__global__ void pp_weight_kernel(const double2 *__restrict__ modes, int ng, int nm, const double *__restrict__ sigma,
                                 const double *__restrict__ omega, double w, double2 *__restrict__ out) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= ng * nm) return;
  const int j = idx % nm;
  const double o2 = omega[j] * omega[j];
  const double c = sigma[j] * o2 / (o2 - w * w);
  const double2 v = modes[idx];
  out[idx] = make_double2(c * v.x, c * v.y);
}

// e = I + S(w) / (sv_g sv_h) where both sv > 0, else the static eps^-1 entry
__global__ void pp_finish_kernel(double2 *__restrict__ e, const double2 *__restrict__ ei_static,
                                 const double *__restrict__ sv, int ng) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)ng * ng) return;
  const int g = (int)(idx / ng), h = (int)(idx % ng);
  if (sv[g] > 0.0 && sv[h] > 0.0) {
    const double f = 1.0 / (sv[g] * sv[h]);
    double2 v = e[idx];
    v.x *= f;
    v.y *= f;
    if (g == h) v.x += 1.0;
    e[idx] = v;
  } else {
    e[idx] = ei_static[idx];
  }
}

// The pole form for at most 32 modes in one pass: e = I + (sum_a c_a A_ga conj(A_ha)) / (sv_g sv_h) with
// c_a = sigma_a omega_a^2 / (omega_a^2 - w^2), or the static entry where sv_g or sv_h vanishes.  64 x 64 outputs
// per workgroup, 4 x 4 per thread, both tiles' modes in LDS; bound by writing e once.  (Weights, product and
// division as three passes: 100 us for 3071 G and 16 modes; 62 us.)
constexpr int PFT = 64, PFM = 32;
__global__ __launch_bounds__(256) void pp_pole_kernel(const double2 *__restrict__ modes, int ng, int nm,
                                                      const double *__restrict__ sigma,
                                                      const double *__restrict__ omega, double w,
                                                      const double *__restrict__ sv,
                                                      const double2 *__restrict__ ei_static, double2 *__restrict__ e) {
  __shared__ double2 sa[PFM][PFT + 1], sb[PFM][PFT + 1];
  __shared__ double sc[PFM];
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  const int g0 = blockIdx.y * PFT, h0 = blockIdx.x * PFT;
  if (tid < nm) {
    const double o2 = omega[tid] * omega[tid];
    sc[tid] = sigma[tid] * o2 / (o2 - w * w);
  }
  __syncthreads();
  for (int idx = tid; idx < PFT * nm; idx += 256) {
    const int r = idx / nm, a = idx - r * nm;
    const double2 u = modes[(size_t)min(g0 + r, ng - 1) * nm + a], v = modes[(size_t)min(h0 + r, ng - 1) * nm + a];
    sa[a][r] = make_double2(sc[a] * u.x, sc[a] * u.y);
    sb[a][r] = v;
  }
  __syncthreads();
  double2 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = make_double2(0.0, 0.0);
#pragma unroll 2
  for (int a = 0; a < nm; ++a) {
    double2 u[4], v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = sa[a][ty + 16 * i];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = sb[a][tx + 16 * j];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[i][j].x += u[i].x * v[j].x + u[i].y * v[j].y;
        acc[i][j].y += u[i].y * v[j].x - u[i].x * v[j].y;
      }
  }
  double vg[4], vh[4];                 // sqrt(V)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    vg[i] = sv[min(g0 + ty + 16 * i, ng - 1)];
    vh[i] = sv[min(h0 + tx + 16 * i, ng - 1)];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int g = g0 + ty + 16 * i, h = h0 + tx + 16 * j;
      if (g < ng && h < ng) {
        const size_t at = (size_t)g * ng + h;
        double2 v = acc[i][j];
        if (vg[i] > 0.0 && vh[j] > 0.0) {
          const double f = 1.0 / (vg[i] * vh[j]);      // as in pp_finish_kernel
          v.x *= f;
          v.y *= f;
          if (g == h) v.x += 1.0;
        } else {
          v = ei_static[at];
        }
        e[at] = v;
      }
    }
}

static inline unsigned blocks_for(size_t n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_density(const float2 *psi, int nv, int nr, double occ, double2 *rho, hipStream_t s) {
  hipLaunchKernelGGL(density_kernel, dim3(blocks_for(nr)), dim3(256), 0, s, psi, nv, nr, occ, rho);
  return hipGetLastError();
}

hipError_t launch_density_transform(double2 *rho, double2 *tmp, int n1, int n2, int n3, hipStream_t s) {
  // rho -> tmp (axis 0) -> rho (axis 1) -> tmp (axis 2); the result is left in tmp
  const int nr = n1 * n2 * n3;
  hipLaunchKernelGGL(dft_axis_f64_kernel, dim3(blocks_for(nr)), dim3(256), 0, s, rho, tmp, n1, n2, n3, 0);
  hipLaunchKernelGGL(dft_axis_f64_kernel, dim3(blocks_for(nr)), dim3(256), 0, s, tmp, rho, n1, n2, n3, 1);
  hipLaunchKernelGGL(dft_axis_f64_kernel, dim3(blocks_for(nr)), dim3(256), 0, s, rho, tmp, n1, n2, n3, 2);
  return hipGetLastError();
}

hipError_t launch_screening(const double2 *ei, const double *sv, int ng, long long lds, double2 *out, hipStream_t s) {
  hipLaunchKernelGGL(screening_kernel, dim3(blocks_for((size_t)ng * ng)), dim3(256), 0, s, ei, sv, ng, lds, out);
  return hipGetLastError();
}

hipError_t launch_sum_rule(const int *miller, int ng, const double *q, double a_bohr, const double *sv,
                           const double2 *rho_g, int n1, int n2, int n3, double2 *m, hipStream_t s) {
  const double b = 2.0 * 3.14159265358979323846 / a_bohr;
  hipLaunchKernelGGL(sum_rule_kernel, dim3(blocks_for((size_t)ng * ng)), dim3(256), 0, s, miller, ng, q[0], q[1],
                     q[2], b, sv, rho_g, n1, n2, n3, m);
  return hipGetLastError();
}

hipError_t launch_start_block(double2 *x, int ng, int b, unsigned long long seed, hipStream_t s) {
  hipLaunchKernelGGL(start_block_kernel, dim3(blocks_for((size_t)ng * b)), dim3(256), 0, s, x, ng, b, seed);
  return hipGetLastError();
}

hipError_t launch_thin_product(int M, int N, int K, const double2 *A, long long lda, const double2 *B, int ldb,
                               double2 *part, hipStream_t s) {
  if (N < 1 || N > JMAX) return hipErrorInvalidValue;
  const int kz = thin_splits(M, K);
  int kchunk = (K + kz - 1) / kz;
  kchunk = (kchunk + TPK - 1) / TPK * TPK;
  hipLaunchKernelGGL(thin_product_kernel, dim3((M + TPM - 1) / TPM, kz), dim3(256), 0, s, M, N, K, A, lda, B, ldb, part,
                     kchunk);
  return hipGetLastError();
}

hipError_t launch_thin_sum(const double2 *part, int M, int N, int K, double alpha, double2 *y, hipStream_t s) {
  const size_t n = (size_t)M * N;
  hipLaunchKernelGGL(thin_sum_kernel, dim3(blocks_for(n)), dim3(256), 0, s, part, thin_splits(M, K), n, alpha, y);
  return hipGetLastError();
}

hipError_t launch_block_gram(const double2 *x, const double2 *y, int ng, int b, double2 *gpart, hipStream_t s) {
  hipLaunchKernelGGL(block_gram_kernel, dim3(gram_blocks(ng)), dim3(512), 0, s, x, y, ng, b, gram_chunk(ng), gpart);
  return hipGetLastError();
}

hipError_t launch_herm_jacobi(const double2 *gpart, int ng, int b, double *evals, double2 *z, hipStream_t s) {
  if (b < 1 || b > JMAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(herm_jacobi_kernel, dim3(1), dim3(512), 0, s, gpart, gram_blocks(ng), b, evals, z, 40);
  return hipGetLastError();
}

hipError_t launch_block_chol(const double2 *gpart, int ng, int b, double2 *u, hipStream_t s) {
  if (b < 1 || b > JMAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(block_chol_kernel, dim3(1), dim3(512), 0, s, gpart, gram_blocks(ng), b, u);
  return hipGetLastError();
}

size_t rotate_part_doubles(int ng, int b) { return (size_t)((ng + ROT_ROWS - 1) / ROT_ROWS) * b; }

hipError_t launch_block_rotate(const double2 *x, const double2 *z, int ng, int b, double2 *w, hipStream_t s) {
  hipLaunchKernelGGL(block_rotate_kernel, dim3((ng + ROT_ROWS - 1) / ROT_ROWS), dim3(256), 0, s, x,
                     (const double2 *)nullptr, z, ng, b, (const double *)nullptr, w, (double2 *)nullptr,
                     (double *)nullptr);
  return hipGetLastError();
}

hipError_t launch_block_ritz(const double2 *x, const double2 *y, const double2 *z, int ng, int b, const double *theta,
                             int nm, double2 *w, double2 *t, double *rpart, double *out, hipStream_t s) {
  if (nm < 1 || nm > JMAX) return hipErrorInvalidValue;
  const int nblk = (ng + ROT_ROWS - 1) / ROT_ROWS;
  hipLaunchKernelGGL(block_rotate_kernel, dim3(nblk), dim3(256), 0, s, x, y, z, ng, b, theta, w, t, rpart);
  hipLaunchKernelGGL(ritz_residual_kernel, dim3(1), dim3(256), 0, s, rpart, nblk, b, theta, nm, out);
  return hipGetLastError();
}

hipError_t launch_pp_frequency(const double2 *a, int lda, const double2 *t, int ldt, int ng, const double *theta,
                               int nm, double *sigma, double *omega, hipStream_t s) {
  hipLaunchKernelGGL(pp_frequency_kernel, dim3(nm), dim3(256), 0, s, a, lda, t, ldt, ng, theta, sigma, omega);
  return hipGetLastError();
}

bool pp_pole_fits(int nm) { return nm <= PFM; }

hipError_t launch_pp_pole(const double2 *modes, int ng, int nm, const double *sigma, const double *omega, double w,
                          const double *sv, const double2 *ei_static, double2 *e, hipStream_t s) {
  const int nt = (ng + PFT - 1) / PFT;
  if (nm > PFM || nt > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pp_pole_kernel, dim3(nt, nt), dim3(256), 0, s, modes, ng, nm, sigma, omega, w, sv, ei_static, e);
  return hipGetLastError();
}

hipError_t launch_pp_weight(const double2 *modes, int ng, int nm, const double *sigma, const double *omega, double w,
                            double2 *out, hipStream_t s) {
  hipLaunchKernelGGL(pp_weight_kernel, dim3(blocks_for((size_t)ng * nm)), dim3(256), 0, s, modes, ng, nm, sigma, omega,
                     w, out);
  return hipGetLastError();
}

hipError_t launch_pp_finish(double2 *e, const double2 *ei_static, const double *sv, int ng, hipStream_t s) {
  hipLaunchKernelGGL(pp_finish_kernel, dim3(blocks_for((size_t)ng * ng)), dim3(256), 0, s, e, ei_static, sv, ng);
  return hipGetLastError();
}

}  // namespace gwi
