// FP64 inverse of a Hermitian positive definite matrix (eps of Sec. 5.1) by Cholesky:
//   eps = L L^H  (blocked: right-looking between panels of 128 columns, left-looking inside one),
//   X = L^-1 (blocked forward substitution on I, panel by panel behind the factorisation),
//   eps^-1 = X^H X.
// The paper inverts eps with a Newton iteration built on matrix products because that
// parallelises across distributed memory; on one GPU the factorisation costs about a
// third of the flops and every large step below is still a matrix product (zgemm).
//
// zgemm: C = alpha * op(A) op(B) + beta * C for complex128 (B also complex64, widened on the way into LDS), op =
// identity, transpose, conjugate or both, on v_mfma_f64_16x16x4f64.  Complex products use real MFMA with k' = (k, re/im):
//   Re C += [Re A, Im A] . [Re B; -Im B],   Im C += [Re A, Im A] . [Im B; Re B].
#include <algorithm>

#include <type_traits>
#include <utility>

#include "elim32.h"
#include "gw_internal.h"

namespace gwi {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// Two shapes of the product kernel: 64 x 64 tiles with 4 complex k per stage (20 KB of LDS, four workgroups per CU; 8
// complex k per stage: 2% slower for the inverse at N = 4067, 16: 18% slower) for outputs that fill the chip, and
// 32 x 32 tiles with 16 complex k per stage where they do not: four times the workgroups, and stages long enough
// to cover the loads of the stage after the next on a CU that holds a single workgroup.  GK: complex k per
// stage; WGS: workgroups per CU; SETS: stages whose global loads are in registers; AHEAD: steps of two complex k
// between reading an operand from LDS and multiplying it.
template <int GT> struct ZgShape;
template <> struct ZgShape<64> { static constexpr int GK = 4, WGS = 4, SETS = 1, AHEAD = 1; };
template <> struct ZgShape<32> { static constexpr int GK = 16, WGS = 3, SETS = 2, AHEAD = 4; };

// The second product of a combined launch (lower_only == 3): same A, K, alpha, beta and leading dimension of C, its
// own B (leading dimension ldb), C and column count, over a full grid of tiles numbered after the first product's
// ntile1 lower tiles.
struct Zg2 {
  const double2 *B;
  double2 *C;
  long long ldb;
  int opB, N, ntile1;
};

template <int GT, typename TB>
__global__ __launch_bounds__(256, ZgShape<GT>::WGS) void zgemm_kernel(int M, int N, int K, const double2 *__restrict__ A,
                                                    long long lda, int opA, const TB *__restrict__ B,
                                                    long long ldb, int opB, double2 *__restrict__ C, long long ldc,
                                                    double alpha, double beta, int lower_only, int tri_k, Zg2 z2) {
  constexpr int GK = ZgShape<GT>::GK, RB = GT / 32;     // 16 x 16 blocks per wave and side
  constexpr int LP = GT == 64 ? 64 : 36;                // LDS row stride
  // lower_only == 2: a square product over a one-dimensional grid of its lower tiles only, numbered row
  // by row (t = r (r + 1) / 2 + c), so consecutive workgroups, which the dispatcher deals out to the XCDs
  // in turn, carry equal work and no workgroup is launched for an upper tile
  int row0, col0;
  if (lower_only == 3 && (int)blockIdx.x >= z2.ntile1) {
    const int t = (int)blockIdx.x - z2.ntile1, nct = (z2.N + GT - 1) / GT;
    row0 = (t / nct) * GT;
    col0 = (t % nct) * GT;
    if constexpr (std::is_same_v<TB, double2>) B = z2.B;
    C = z2.C;
    ldb = z2.ldb;
    opB = z2.opB;
    N = z2.N;
  } else if (lower_only >= 2) {
    const int t = blockIdx.x;
    int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    while (r * (r + 1) / 2 > t) --r;
    row0 = r * GT;
    col0 = (t - r * (r + 1) / 2) * GT;
  } else {
    row0 = blockIdx.y * GT;
    col0 = blockIdx.x * GT;
  }
  const int kend = K;
  const bool transA = opA & Z_T, transB = opB & Z_T;
  // two LDS stages: the global loads of stage k+1 are in flight in registers while stage k's MFMAs run
  __shared__ double sA[2][GK][2][LP];
  __shared__ double sX[2][GK][3][LP];   // planes Re B, -Im B, Im B: [Re B; -Im B] is planes 0, 1, [Im B; Re B] 2, 0
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wr = wave >> 1, wc = wave & 1;
  f64x4 accR[RB][RB], accI[RB][RB];
#pragma unroll
  for (int a = 0; a < RB; ++a)
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) { accR[a][b][e] = 0.0; accI[a][b][e] = 0.0; }

  int kbeg = 0;
  if (tri_k) kbeg = (max(row0, col0) / GK) * GK;
  const int kl = lane >> 4, li = lane & 15;
  constexpr int PER = (GT * GK) / 256;   // elements of each operand per thread and stage
  constexpr int SETS = ZgShape<GT>::SETS;
  double2 va[SETS][PER];
  TB vb[SETS][PER];
  // element idx of a stage: A row r / B column c and its k offset kk, in the order that keeps the
  // global reads contiguous for either layout
  auto a_coord = [&](int idx, int &r, int &kk) {
    if (transA) { r = idx % GT; kk = idx / GT; } else { r = idx / GK; kk = idx % GK; }
  };
  auto b_coord = [&](int idx, int &c, int &kk) {
    if (transB) { c = idx / GK; kk = idx % GK; } else { c = idx % GT; kk = idx / GT; }
  };
  // Loads keep the raw values; the conjugation of a transposed operand is applied when they are
  // written to LDS, so no instruction waits on a load before the stage's MFMAs have been issued.
  // Each thread's elements advance by GK along k per stage: running pointers.  With one set of registers the loads of
  // stage k + 1 are issued in stage k, without a bounds test in the stages of a whole tile that lie inside
  // [kbeg, kend).  With two sets they are issued two stages ahead, and without a branch, behind which the
  // compiler would wait for all outstanding loads, not for the stage's own: an element outside the tile or past
  // kend reads an address inside its operand, and zero takes its place on the way to LDS.
  // (N = 410, K = 128, 32 x 32 tiles: 15.2 us with one set, 12.6 us with two; 64 x 64 tiles, where four waves
  // per SIMD hide the loads: 67.8 TFLOP/s with one set at N = 4067, 66 without the branches.)
  const double2 *pa[PER];
  const TB *pb[PER];
  int ka[PER], kb[PER];
  bool ra[PER], cb_ok[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int idx = tid + it * 256;
    int r, c, kk;
    a_coord(idx, r, kk);
    ka[it] = kk;
    ra[it] = row0 + r < M;
    const int rr = min(row0 + r, M - 1), kr = min(kbeg + kk, kend - 1);
    pa[it] = transA ? A + (long long)kr * lda + rr : A + (long long)rr * lda + kr;
    b_coord(idx, c, kk);
    kb[it] = kk;
    cb_ok[it] = col0 + c < N;
    const int cc = min(col0 + c, N - 1), kc = min(kbeg + kk, kend - 1);
    pb[it] = transB ? B + (long long)cc * ldb + kc : B + (long long)kc * ldb + cc;
  }
  const long long step_a = transA ? (long long)GK * lda : GK, step_b = transB ? GK : (long long)GK * ldb;
  const bool whole = row0 + GT <= M && col0 + GT <= N;
  auto gload = [&](int k0, auto setc) {      // the stage from k0 on, and the pointers to the next
    constexpr int set = decltype(setc)::value % SETS;
    if constexpr (SETS == 2) {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        va[set][it] = *pa[it];
        vb[set][it] = *pb[it];
        pa[it] += k0 + GK + ka[it] < kend ? step_a : 0;
        pb[it] += k0 + GK + kb[it] < kend ? step_b : 0;
      }
      return;
    }
    if (whole && k0 + GK <= kend) {          // uniform
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        va[set][it] = *pa[it];
        vb[set][it] = *pb[it];
      }
    } else {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        va[set][it] = make_double2(0.0, 0.0);
        if (ra[it] && k0 + ka[it] < kend) va[set][it] = *pa[it];
        vb[set][it] = TB{0, 0};
        if (cb_ok[it] && k0 + kb[it] < kend) vb[set][it] = *pb[it];
      }
    }
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      pa[it] += step_a;
      pb[it] += step_b;
    }
  };
  const double sa = opA & Z_J ? -1.0 : 1.0, sb = opB & Z_J ? -1.0 : 1.0;
  auto lstore = [&](int k0, auto bufc) {
    constexpr int buf = decltype(bufc)::value, set = buf % SETS;
    if (SETS == 2 && !(whole && k0 + GK <= kend)) {       // uniform
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        if (!(ra[it] && k0 + ka[it] < kend)) va[set][it] = make_double2(0.0, 0.0);
        if (!(cb_ok[it] && k0 + kb[it] < kend)) vb[set][it] = TB{0, 0};
      }
    }
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int idx = tid + it * 256;
      int r, c, kk;
      a_coord(idx, r, kk);
      sA[buf][kk][0][r] = va[set][it].x;
      sA[buf][kk][1][r] = sa * va[set][it].y;
      b_coord(idx, c, kk);
      const double by = sb * (double)vb[set][it].y;
      sX[buf][kk][0][c] = (double)vb[set][it].x;
      sX[buf][kk][1][c] = -by;
      sX[buf][kk][2][c] = by;
    }
  };
  // operands of one step of two complex k
  struct Ops { double a[RB], x[RB], y[RB]; };
  const int comp = kl & 1, kh = kl >> 1, yp = comp ? 0 : 2;
  const int ar = wr * 16 * RB + li, bc = wc * 16 * RB + li;
  auto rd = [&](int buf, int s) {
    const int kk = 2 * s + kh;
    Ops o;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      o.a[i] = sA[buf][kk][comp][ar + 16 * i];
      o.x[i] = sX[buf][kk][comp][bc + 16 * i];
      o.y[i] = sX[buf][kk][yp][bc + 16 * i];
    }
    return o;
  };
  auto mul = [&](const Ops &o) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        accR[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[i], o.x[j], accR[i][j], 0, 0, 0);
        accI[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.a[i], o.y[j], accI[i][j], 0, 0, 0);
      }
  };
  // Each step's operands are read from LDS AHEAD steps before they are multiplied, and the barrier stands before
  // a stage's last AHEAD steps, so LDS latency and the wait for the other waves pass while MFMAs run.  Once a wave
  // passes the barrier of stage k every wave has the stage's operands in registers, so stage k + 1 may refill
  // its buffer.  The reads past the last stage return whatever the buffer holds, unused: with a test around them
  // the MFMAs behind it waited for all reads (4096^3: 67.7 TFLOP/s with the test, 70.4 without).
  constexpr int AHEAD = ZgShape<GT>::AHEAD, ST = GK / 2;   // steps per stage
  static_assert(ST % AHEAD == 0, "a step's slot is its index modulo AHEAD");
  if (kbeg < kend) {
    gload(kbeg, std::integral_constant<int, 0>{});
    if constexpr (SETS == 2) gload(kbeg + GK, std::integral_constant<int, 1>{});
    lstore(kbeg, std::integral_constant<int, 0>{});
  }
  __syncthreads();
  Ops q[AHEAD];
#pragma unroll
  for (int st = 0; st < AHEAD; ++st) q[st] = rd(0, st);
  auto stage = [&](int k0, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    const bool more = k0 + GK < kend;
    if (SETS == 2 || more) gload(k0 + SETS * GK, bufc);
#pragma unroll
    for (int st = 0; st < ST; ++st) {
      if (st == ST - AHEAD) {
        if (more) lstore(k0 + GK, std::integral_constant<int, buf ^ 1>{});
        __syncthreads();
      }
      const Ops cur = q[st % AHEAD];
      q[st % AHEAD] = st + AHEAD < ST ? rd(buf, st + AHEAD) : rd(buf ^ 1, st + AHEAD - ST);
      mul(cur);
    }
  };
  for (int k0 = kbeg; k0 < kend; k0 += 2 * GK) {
    stage(k0, std::integral_constant<int, 0>{});
    if (k0 + GK < kend) stage(k0 + GK, std::integral_constant<int, 1>{});
  }
  // lane holds D[i][j] of each 16x16 block in register e with i = 4*e + (lane>>4), j = lane & 15
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < RB; ++cb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = row0 + wr * 16 * RB + rb * 16 + 4 * e + kl;
        const int col = col0 + wc * 16 * RB + cb * 16 + li;
        if (row < M && col < N) {
          double2 *d = C + (long long)row * ldc + col;
          double2 v = make_double2(alpha * accR[rb][cb][e], alpha * accI[rb][cb][e]);
          if (beta != 0.0) { const double2 o = *d; v.x += beta * o.x; v.y += beta * o.y; }
          *d = v;
        }
      }
}

// Tile side for a product of `tiles` 64 x 64 tiles.  Small tiles win while four times as many still find a place at
// once (three per CU), and further for short K, where a 64 x 64 tile's prologue and store are most of its time, and
// for X^H X, whose tiles are of uneven length.  Inverse, us, the limits 400, 600, 192 -> these: N = 1800 1870 -> 1723,
// 2109 2367 -> 2221, 2500 3065 -> 2936, 3071 4325 -> 4280; 2200 in place of 600 takes 4617 at 3071 and 900 takes 4366;
// 925 x 925 products of the Newton iteration (225 tiles, K = 925) take 4.99 ms, and 5.11 with a limit of 256.
static int zg_tile(long long tiles, int K, int tri_k) {
  return tiles < (tri_k ? 1200 : K <= 256 ? 600 : 192) ? 32 : 64;
}

template <int GT, typename TB>
static hipError_t zgemm_t(int M, int N, int K, const double2 *A, long long lda, int opA, const TB *B,
                          long long ldb, int opB, double2 *C, long long ldc, double alpha, double beta,
                          int lower_only, int tri_k, hipStream_t s) {
  if (lower_only) {
    const long long nt = (N + GT - 1) / GT;
    hipLaunchKernelGGL(HIP_KERNEL_NAME(zgemm_kernel<GT, TB>), dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), 0, s, M, N,
                       K, A, lda, opA, B, ldb, opB, C, ldc, alpha, beta, 2, tri_k, Zg2{});
    return hipGetLastError();
  }
  dim3 grid((N + GT - 1) / GT, (M + GT - 1) / GT);
  hipLaunchKernelGGL(HIP_KERNEL_NAME(zgemm_kernel<GT, TB>), grid, dim3(256), 0, s, M, N, K, A, lda, opA, B, ldb, opB,
                     C, ldc, alpha, beta, 0, tri_k, Zg2{});
  return hipGetLastError();
}

// lower_only: a square product, its lower tiles only
template <typename TB>
static hipError_t zgemm(int M, int N, int K, const double2 *A, long long lda, int opA, const TB *B,
                        long long ldb, int opB, double2 *C, long long ldc, double alpha, double beta,
                        int lower_only, int tri_k, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const long long mt = (M + 63) / 64, nt = (N + 63) / 64, tiles = lower_only ? nt * (nt + 1) / 2 : mt * nt;
  return zg_tile(tiles, K, tri_k) == 32
             ? zgemm_t<32>(M, N, K, A, lda, opA, B, ldb, opB, C, ldc, alpha, beta, lower_only, tri_k, s)
             : zgemm_t<64>(M, N, K, A, lda, opA, B, ldb, opB, C, ldc, alpha, beta, lower_only, tri_k, s);
}

// C1 = alpha A B1^H + beta C1 on the lower tiles of the square M x M C1, and C2 = alpha A B2 + beta C2 on
// all tiles of the M x N2 C2, in one launch
template <int GT>
static hipError_t zgemm_lower_and_full_t(int M, int N2, int K, const double2 *A, long long lda, const double2 *B1,
                                         long long ldb1, double2 *C1, const double2 *B2, long long ldb2, double2 *C2,
                                         long long ldc, double alpha, double beta, hipStream_t s) {
  const long long nt = (M + GT - 1) / GT, nt1 = nt * (nt + 1) / 2, nt2 = N2 > 0 ? nt * ((N2 + GT - 1) / GT) : 0;
  hipLaunchKernelGGL(HIP_KERNEL_NAME(zgemm_kernel<GT, double2>), dim3((unsigned)(nt1 + nt2)), dim3(256), 0, s, M, M, K,
                     A, lda, Z_N, B1, ldb1, Z_H, C1, ldc, alpha, beta, 3, 0, Zg2{B2, C2, ldb2, Z_N, N2, (int)nt1});
  return hipGetLastError();
}

static hipError_t zgemm_lower_and_full(int M, int N2, int K, const double2 *A, long long lda, const double2 *B1,
                                       long long ldb1, double2 *C1, const double2 *B2, long long ldb2, double2 *C2,
                                       long long ldc, double alpha, double beta, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const long long nt = (M + 63) / 64, tiles = nt * (nt + 1) / 2 + nt * ((N2 + 63) / 64);
  return zg_tile(tiles, K, 0) == 32
             ? zgemm_lower_and_full_t<32>(M, N2, K, A, lda, B1, ldb1, C1, B2, ldb2, C2, ldc, alpha, beta, s)
             : zgemm_lower_and_full_t<64>(M, N2, K, A, lda, B1, ldb1, C1, B2, ldb2, C2, ldc, alpha, beta, s);
}

hipError_t launch_zgemm(int M, int N, int K, const double2 *A, long long lda, int opA, const double2 *B, long long ldb,
                        int opB, double2 *C, long long ldc, double alpha, double beta, hipStream_t s) {
  return zgemm(M, N, K, A, lda, opA, B, ldb, opB, C, ldc, alpha, beta, 0, 0, s);
}

hipError_t launch_zgemm(int M, int N, int K, const double2 *A, long long lda, int opA, const float2 *B, long long ldb,
                        int opB, double2 *C, long long ldc, double alpha, double beta, hipStream_t s) {
  return zgemm(M, N, K, A, lda, opA, B, ldb, opB, C, ldc, alpha, beta, 0, 0, s);
}

// ---- diagonal block L_kk = chol(A_kk), Linv_kk = L_kk^-1, and the panel column below it -------------
// Every workgroup first applies the panel's earlier columns to the block and to its panel rows, then
// factors and inverts the 32 x 32 block in LDS (cheap, and it saves a dependent launch per step);
// workgroup 0 stores L_kk, Linv_kk and the pivot flag, and workgroup g forms PR rows of the panel
// L[k0+nb+PR g : +PR, k0 : k0+nb] = A Linv_kk^H.  With PR = 16 the panel product of a 4067-row
// matrix spreads over about 250 CUs (64 rows per workgroup left three quarters of the CUs idle).
constexpr int NB = 32;
constexpr int PR = 16;    // panel rows per workgroup of the diagonal-block kernel
constexpr int CHOL_PW = 128;   // panel width of the factorisation and the substitution
constexpr int PD_THREADS = PR * NB;   // diagonal-block kernel: eight waves, one panel entry per thread

// L is the panel buffer: row i of the panel's columns at L + i ldl
__global__ __launch_bounds__(PD_THREADS) void potrf_diag_kernel(const double2 *__restrict__ A, int n, int p0,
                                                                int k0, double2 *__restrict__ L, int ldl,
                                                                double2 *__restrict__ linv, int *__restrict__ pivot) {
  __shared__ double2 a[NB][NB + 1];
  // L[k0 + i][p0 + k] (the block's rows, the panel's earlier columns) and the same columns of this
  // workgroup's panel rows, planar: [k][re, im][row], the operand layout of the FP64 MFMA
  __shared__ double lbp[CHOL_PW - NB][2][NB + 1];
  __shared__ double lrp[CHOL_PW - NB][2][PR + 1];
  __shared__ double2 x[NB][NB + 1];
  __shared__ double2 pa[PR][NB + 1];
  __shared__ int bad;
  const int tid = threadIdx.x;
  const int nb = min(NB, n - k0);
  const int kp = k0 - p0;                                   // a multiple of NB
  // Every load is issued before the first use, so that one memory latency covers them all: this workgroup's PR
  // panel rows below the block (thread (pib, pj) holds A[r0 + pib][k0 + pj]), the block's lower triangle
  // (rows pib and pib + PR), and the panel's earlier columns of both.
  const int r0 = k0 + nb + (int)blockIdx.x * PR;
  const int pj = tid % NB, pib = tid / NB;
  static_assert(PR * NB == PD_THREADS, "one panel entry per thread");
  static_assert(2 * PR == NB, "rows pib and pib + PR cover the block");
  const double2 zero2 = make_double2(0.0, 0.0);
  const double2 pv = (r0 + pib < n && pj < nb) ? A[(size_t)(r0 + pib) * n + k0 + pj] : zero2;
  double2 bv[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = pib + PR * h;
    bv[h] = i >= nb && i == pj ? make_double2(1.0, 0.0) : zero2;      // padded with the identity
    if (i < nb && pj <= i) bv[h] = A[(size_t)(k0 + i) * n + k0 + pj];
  }
  constexpr int Q = (CHOL_PW - NB) / NB;
  double2 lu[Q], lw[Q], lv[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    lu[q] = lw[q] = lv[q] = zero2;
    if (NB * q < kp) {                                       // column k = pj + NB q; rows pib and pib + PR
      const int k = pj + NB * q;
      if (pib < nb) lu[q] = L[(size_t)(k0 + pib) * ldl + k];
      if (pib + PR < nb) lw[q] = L[(size_t)(k0 + pib + PR) * ldl + k];
      if (r0 + pib < n) lv[q] = L[(size_t)(r0 + pib) * ldl + k];
    }
  }
  a[pib][pj] = bv[0];
  a[pib + PR][pj] = bv[1];
  pa[pib][pj] = pv;
  // Left-looking inside the panel: the kp columns of this panel factored by the earlier steps are applied
  // here, A[k0:, k0:k0+nb] -= L[k0:, p0:k0] L[k0:k0+nb, p0:k0]^H, to this workgroup's copy of the diagonal
  // block and to its panel rows, instead of by a separate product after every step.  The FP64 MFMA forms five
  // 16 x 16 tiles, with k' = (k, re/im) as in zgemm_kernel: Re C += [Re A, Im A] . [Re B; Im B] and
  // Im C += [Re A, Im A] . [-Im B; Re B] for C = A B^H.  Waves 0 and 1 take the panel rows' two column
  // halves, waves 2 and 3 the block's tiles (0,0) and (1,0), and waves 4 to 7 a quarter of the columns each of tile
  // (1,1), so that the four SIMDs carry the same number of MFMAs (five whole tiles on five waves leave
  // one SIMD with two); the quarters are added where the block is next read.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, kl = lane >> 4, li = lane & 15;
  const int comp = kl & 1;
  const unsigned long long flip = comp ? 0ull : 0x8000000000000000ull;   // Y = [-Im B; Re B]
  double2 (*quarter)[16][16] = reinterpret_cast<double2 (*)[16][16]>(&x[0][0]);   // x is free until the factor is done
  static_assert(4 * 16 * 16 <= NB * (NB + 1), "the quarters fit in x");
  if (kp > 0) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (NB * q < kp) {
        const int k = pj + NB * q;
        lbp[k][0][pib] = lu[q].x;
        lbp[k][1][pib] = lu[q].y;
        lbp[k][0][pib + PR] = lw[q].x;
        lbp[k][1][pib + PR] = lw[q].y;
        lrp[k][0][pib] = lv[q].x;
        lrp[k][1][pib] = lv[q].y;
      }
    }
    __syncthreads();
    const bool rows = wave < 2;                              // wave-uniform
    const int ra = wave < 3 ? 0 : 16;                        // first row of the tile (panel rows or block)
    const int cb = wave == 1 || wave >= 4 ? 16 : 0;          // first column (block row of B)
    const int kb = wave < 4 ? 0 : (wave - 4) * (kp / 4), ke = wave < 4 ? kp : kb + kp / 4;   // multiples of 8
    f64x4 accR = {0.0, 0.0, 0.0, 0.0}, accI = {0.0, 0.0, 0.0, 0.0};
    // groups of eight columns, the next group's operands read while one is multiplied, in two register sets
    struct Group {
      double a[4], x[4], y[4];
    } g0, g1;
    const double *ap = rows ? &lrp[kl >> 1][comp][li] : &lbp[kl >> 1][comp][ra + li];
    const int as = rows ? 2 * (PR + 1) : 2 * (NB + 1);       // doubles per column
    auto fetch = [&](Group &g, int s8) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kk = s8 + 2 * u;
        g.a[u] = ap[kk * as];
        g.x[u] = lbp[kk + (kl >> 1)][comp][cb + li];
        g.y[u] = lbp[kk + (kl >> 1)][comp ^ 1][cb + li];
      }
    };
    auto multiply = [&](Group &g) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        g.y[u] = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, g.y[u]) ^ flip);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        accR = __builtin_amdgcn_mfma_f64_16x16x4f64(g.a[u], g.x[u], accR, 0, 0, 0);
        accI = __builtin_amdgcn_mfma_f64_16x16x4f64(g.a[u], g.y[u], accI, 0, 0, 0);
      }
    };
    fetch(g0, kb);
    for (int s8 = kb; s8 < ke; s8 += 16) {
      fetch(g1, min(s8 + 8, ke - 8));                        // unconditional: a branch would make the MFMAs wait for it
      multiply(g0);
      if (s8 + 8 < ke) {
        fetch(g0, min(s8 + 16, ke - 8));
        multiply(g1);
      }
    }
    // lane holds tile entry (4 e + kl, li) in register e
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * e + kl;
      if (rows) {
        pa[i][cb + li].x -= accR[e];
        pa[i][cb + li].y -= accI[e];
      } else if (wave >= 4) {
        quarter[wave - 4][i][li] = make_double2(accR[e], accI[e]);
      } else if (ra + i >= li) {                             // lower entries of the block only
        a[ra + i][li].x -= accR[e];
        a[ra + i][li].y -= accI[e];
      }
    }
  }
  // Elimination of the whole block: the kernel's latency chain.
  // (Four waves with four rows each, the column and the row both through LDS, the pivot checked and the row
  // bounds tested in every step: 20.4 us per call on average at N = 410 against 13.3 us.)
  __shared__ double2 w[NB][NB];
  __shared__ double dv[NB];
  const int m = tid % 16, c = tid / 16;
  static_assert(PD_THREADS == 16 * NB && NB == 32, "one row per 16 lanes, two columns per lane");
  double2 row[2];
  {
    double2 z[2];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {                            // the upper triangle from the lower one
      const int k = 16 * h + m;
      z[h] = a[max(c, k)][min(c, k)];
      if (kp > 0 && min(c, k) >= 16) {
        double2 v[4];                                        // added first, so that the entry is rounded once
#pragma unroll
        for (int g = 0; g < 4; ++g) v[g] = quarter[g][max(c, k) - 16][min(c, k) - 16];
        z[h].x -= (v[0].x + v[1].x) + (v[2].x + v[3].x);
        z[h].y -= (v[0].y + v[1].y) + (v[2].y + v[3].y);
      }
      if (k > c) z[h].y = -z[h].y;
    }
    eliminate32(z, row, w, dv, wave, NB, [](double d) { return rcp_nr(d); });
  }
  __syncthreads();
  // With r_j = sqrt(d_j): row j of L^-1 is row_j / r_j up to the diagonal, column j of L is conj(row_j) / r_j from it on
  // (w[j] r_j would round once more).  The first pivot that is not positive and finite (1-based, over the whole matrix)
  // is flagged; it scales by 1.
  if (wave == 0) {
    const bool wrong = tid < nb && !(dv[tid % NB] > 0.0 && isfinite(dv[tid % NB]));
    const unsigned long long first = __ballot(wrong);
    if (tid == 0) bad = first ? k0 + __ffsll(first) : 0;
  }
  {
    const double d = dv[c], r = d > 0.0 && isfinite(d) ? sqrt(d) : 1.0, ir = rcp_nr(r);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = 16 * h + m;
      const double2 v = make_double2(div_nr(row[h].x, r, ir), div_nr(row[h].y, r, ir));
      x[c][k] = k <= c ? v : make_double2(0.0, 0.0);
      if (k >= c) a[k][c] = k == c ? make_double2(r, 0.0) : make_double2(v.x, -v.y);
    }
  }
  __syncthreads();
  // Waves 4 to 7 of workgroup 0 store the block while waves 0 to 3 form the panel below it.
  if (wave >= 4) {
    if (blockIdx.x != 0) return;
    for (int idx = tid - 256; idx < NB * NB; idx += PD_THREADS - 256) {
      const int i = idx / NB, j = idx % NB;
      if (i < nb && j < nb) L[(size_t)(k0 + i) * ldl + kp + j] = (j <= i) ? a[i][j] : make_double2(0.0, 0.0);
      linv[idx] = (i < nb && j < nb) ? x[i][j] : make_double2(0.0, 0.0);
    }
    if (tid == 256 && bad != 0 && *pivot == 0) *pivot = bad;
    return;
  }
  // L[r][k0 + j] = sum_{k <= j} A[r][k0 + k] conj(Linv[j][k]) (every workgroup factored the block for itself),
  // the tiles of columns 0-15 and 16-31 on the MFMA: waves 0 and 1 form the first tile's real and imaginary
  // part (k < 16: Linv is lower triangular, its upper part zeros), waves 2 and 3 the second's.
  if (r0 >= n) return;
  const int cb = 16 * (wave >> 1), im = wave & 1;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0}, acc2 = {0.0, 0.0, 0.0, 0.0};
  for (int s16 = 0; s16 <= cb; s16 += 16) {
#pragma unroll
    for (int s2 = 0; s2 < 16; s2 += 2) {
      const int kk = s16 + s2 + (kl >> 1);
      const double2 av = pa[li][kk], xv = x[cb + li][kk];
      const double left = comp ? av.y : av.x;
      const double right = im ? (comp ? xv.x : -xv.y) : (comp ? xv.y : xv.x);
      f64x4 &to = s2 & 2 ? acc2 : acc;
      to = __builtin_amdgcn_mfma_f64_16x16x4f64(left, right, to, 0, 0, 0);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = r0 + 4 * e + kl, j = cb + li;
    if (i < n && j < nb) reinterpret_cast<double *>(&L[(size_t)i * ldl + kp + j])[im] = acc[e] + acc2[e];
  }
}

__global__ void fill_identity_kernel(double2 *__restrict__ a, int n, double diag) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)n * n) return;
  const size_t i = idx / n, j = idx % n;
  a[idx] = make_double2(i == j ? diag : 0.0, 0.0);
}

// out[j][i] = conj(out[i][j]) for i > j (upper triangle from the lower), 32x32 tiles via LDS.
__global__ __launch_bounds__(256) void mirror_lower_kernel(double2 *__restrict__ a, int n) {
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj > bi) return;
  __shared__ double2 t[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = 0; k < 32; k += 8) {
    const int i = bi * 32 + ty + k, j = bj * 32 + tx;
    if (i < n && j < n) t[ty + k][tx] = a[(size_t)i * n + j];
  }
  __syncthreads();
  for (int k = 0; k < 32; k += 8) {
    const int i = bj * 32 + ty + k, j = bi * 32 + tx;     // destination (i, j) in the upper tile
    if (i < n && j < n && j > i) {
      const double2 v = t[tx][ty + k];                    // a[j][i]
      a[(size_t)i * n + j] = make_double2(v.x, -v.y);
    }
  }
}

__global__ void fill_int_kernel(int *p, int v) { *p = v; }

hipError_t launch_fill_int(int *p, int value, hipStream_t s) {
  hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(1), 0, s, p, value);
  return hipGetLastError();
}

// ---- block substitution of one panel of rows, X[p0:p1, :] from B[p0:p1, :] ----------------------------
// The columns of B are independent, so a workgroup carries its SUB_CW columns through the panel's
// 32-row steps in LDS: X_k = Linv_kk B_k, then B_i -= L_ik X_k for the panel's later row blocks.
// One launch per panel replaces two small GEMMs per step.
constexpr int SUB_CW = 8;      // columns per workgroup
constexpr int SUB_RS = 256 / SUB_CW;   // row stride of a thread's rows in a 32-row block

__global__ __launch_bounds__(256) void subst_panel_kernel(const double2 *__restrict__ B, const double2 *__restrict__ L,
                                                          int ldl, const double2 *__restrict__ linv_all,
                                                          double2 *__restrict__ X, int n, int p0, int p1) {
  __shared__ double2 sB[CHOL_PW][SUB_CW + 1];
  __shared__ double2 sM[NB][NB + 1];   // Linv_kk, then one L_ik block at a time
  constexpr int PER = NB * SUB_CW / 256;
  const int tid = threadIdx.x;
  const int c0 = blockIdx.x * SUB_CW;
  const int rows = p1 - p0;
  for (int idx = tid; idx < CHOL_PW * SUB_CW; idx += 256) {
    const int i = idx / SUB_CW, c = idx % SUB_CW;
    sB[i][c] = (i < rows && c0 + c < n) ? B[(size_t)(p0 + i) * n + c0 + c] : make_double2(0.0, 0.0);
  }
  // The 32 x 32 blocks pass through sM in the order Linv_(k0), L_(k0+32, k0), ..., Linv_(k0+32), ...; each
  // is loaded into registers (pf) while the block before it is in use, and written to sM when that is free.
  double2 pf[NB * NB / 256];
  auto fetch = [&](int k0, int j0) {   // j0 < 0: Linv of block k0; else L[j0 : j0 + 32, k0 : k0 + 32], zero-padded
    const int nb = min(NB, n - k0), jn = min(NB, p1 - j0);
#pragma unroll
    for (int t = 0; t < NB * NB / 256; ++t) {
      const int idx = tid + 256 * t, i = idx / NB, m = idx % NB;
      if (j0 < 0)
        pf[t] = linv_all[(size_t)(k0 / NB) * NB * NB + idx];
      else
        pf[t] = (i < jn && m < nb) ? L[(size_t)(j0 + i) * ldl + k0 - p0 + m] : make_double2(0.0, 0.0);
    }
  };
  auto commit = [&]() {
#pragma unroll
    for (int t = 0; t < NB * NB / 256; ++t) {
      const int idx = tid + 256 * t;
      sM[idx / NB][idx % NB] = pf[t];
    }
  };
  fetch(p0, -1);
  for (int k0 = p0; k0 < p1; k0 += NB) {
    const int nb = min(NB, n - k0), kr = k0 - p0;
    commit();
    __syncthreads();
    if (k0 + NB < p1) fetch(k0, k0 + NB);
    // X_k = Linv_kk B_k.  Linv_kk is stored with zeros above its diagonal, so m runs over the whole
    // block for every thread: thread (i = ib + SUB_RS t, c) keeps PER independent sums.
    const int ib = tid / SUB_CW, c = tid % SUB_CW;
    double2 xv[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t) xv[t] = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int m = 0; m < NB; ++m) {
      const double2 v = sB[kr + m][c];
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const double2 u = sM[ib + SUB_RS * t][m];
        xv[t].x += u.x * v.x - u.y * v.y;
        xv[t].y += u.x * v.y + u.y * v.x;
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int idx = tid + 256 * t, i = idx / SUB_CW, c = idx % SUB_CW;
      if (i < nb) {
        sB[kr + i][c] = xv[t];
        if (c0 + c < n) X[(size_t)(k0 + i) * n + c0 + c] = xv[t];
      }
    }
    // the panel's later row blocks: B_i -= L_ik X_k
    for (int j0 = k0 + NB; j0 < p1; j0 += NB) {
      const int jn = min(NB, p1 - j0), jr = j0 - p0;
      __syncthreads();
      commit();
      __syncthreads();
      if (j0 + NB < p1)
        fetch(k0, j0 + NB);
      else if (k0 + NB < p1)
        fetch(k0 + NB, -1);
      // sM is zero for m >= nb, so m runs over the whole block here too
      double2 acc[PER];
#pragma unroll
      for (int t = 0; t < PER; ++t) acc[t] = make_double2(0.0, 0.0);
#pragma unroll 4
      for (int m = 0; m < NB; ++m) {
        const double2 v = sB[kr + m][c];
#pragma unroll
        for (int t = 0; t < PER; ++t) {
          const double2 u = sM[ib + SUB_RS * t][m];
          acc[t].x += u.x * v.x - u.y * v.y;
          acc[t].y += u.x * v.y + u.y * v.x;
        }
      }
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int i = ib + SUB_RS * t;
        if (i < jn) {
          sB[jr + i][c].x -= acc[t].x;
          sB[jr + i][c].y -= acc[t].y;
        }
      }
    }
    __syncthreads();
  }
}

// L is needed one panel of columns at a time: rows of CHOL_PW values, aligned to memory lines whatever n is.  (With
// the n x n factor at n = 4067, whose rows of 65072 bytes start anywhere in a line, the products' 64-byte runs of
// L touched half as many lines again.)
size_t chol_panel_elems(int n) { return (size_t)n * std::min(n, CHOL_PW); }

size_t chol_small_bytes(int n) {
  const int nblk = (n + NB - 1) / NB;
  return (size_t)nblk * NB * NB * sizeof(double2);
}

#define GW_TRY(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) return e_; } while (0)

hipError_t hpd_inverse(double2 *a, int n, double2 *l, double2 *x, double2 *small, int *pivot_dev, double2 *out,
                       hipStream_t s) {
  const size_t nn = (size_t)n * n;
  const unsigned fill_blocks = (unsigned)((nn + 255) / 256);
  GW_TRY(launch_fill_int(pivot_dev, 0, s));
  // the substitution's right-hand side B = I lives in out until X^H X overwrites it
  hipLaunchKernelGGL(fill_identity_kernel, dim3(fill_blocks), dim3(256), 0, s, out, n, 1.0);
  GW_TRY(hipGetLastError());
  // Panels of PW columns, factorisation and substitution interleaved.  Inside a panel each NB-wide step of
  // the factorisation first applies the panel's earlier columns to its own (left-looking, inside the
  // diagonal-block kernel, so a step is one launch).  The panel's rows of X = L^-1 need only L's rows of
  // this panel and B's rows, so they follow at once.  Then one launch of K = PW products updates both
  // what lies right of the panel in A and below it in B, with the same left operand L[p1:, p0:p1]: the
  // large trailing matrices are read and written once per panel, and the two products fill the GPU
  // together where one alone would leave CUs idle (few trailing rows late, few B columns early).
  // (A look-ahead that moved each panel's trailing product to a second stream, so that the next panel's
  // chain could start at once, measured slower at N = 4067: the product's workgroups fill the CUs the
  // chain's small launches wait for.)
  const int ldl = std::min(n, CHOL_PW);
  constexpr int PW = CHOL_PW;   // 128, 256 and 512 measured alike; 32 (no panels) 5% slower at N = 4067
  for (int p0 = 0; p0 < n; p0 += PW) {
    const int p1 = min(n, p0 + PW);
    // 1. factor the panel: L[p0:, p0:p1]
    for (int k0 = p0; k0 < p1; k0 += NB) {
      const int kb = k0 / NB, nb = min(NB, n - k0), rest = n - k0 - nb;
      double2 *linv = small + (size_t)kb * NB * NB;
      // the diagonal block and, in the same launch, the panel column L[k0+nb:, k0:k0+nb] = A Linv^H
      hipLaunchKernelGGL(potrf_diag_kernel, dim3(std::max(1, (rest + PR - 1) / PR)), dim3(PD_THREADS), 0, s, a, n, p0,
                         k0, l, ldl, linv, pivot_dev);
      GW_TRY(hipGetLastError());
    }
    // 2. the panel's rows of X (columns < p1; beyond them X is zero, never read and not written), all 32-row
    // steps in one launch
    hipLaunchKernelGGL(subst_panel_kernel, dim3((p1 + SUB_CW - 1) / SUB_CW), dim3(256), 0, s, out, l, ldl, small, x, n, p0,
                       p1);
    GW_TRY(hipGetLastError());
    // 3. A[p1:, p1:] -= Lp Lp^H (lower tiles) and B[p1:, :p1] -= Lp X[p0:p1, :p1], Lp = L[p1:, p0:p1]
    const int rest = n - p1;
    if (rest > 0) {
      const double2 *lp = l + (size_t)p1 * ldl;
      GW_TRY(zgemm_lower_and_full(rest, p1, p1 - p0, lp, ldl, lp, ldl, a + (size_t)p1 * n + p1,
                                  x + (size_t)p0 * n, n, out + (size_t)p1 * n, n, -1.0, 1.0, s));
    }
  }
  // 3. out = X^H X (lower tiles, k from max(row, col) since X is lower triangular), then mirror
  GW_TRY(zgemm(n, n, n, x, n, Z_H, x, n, Z_N, out, n, 1.0, 0.0, 1, 1, s));
  dim3 mg((n + 31) / 32, (n + 31) / 32);
  hipLaunchKernelGGL(mirror_lower_kernel, mg, dim3(256), 0, s, out, n);
  return hipGetLastError();
}

// ---- Newton iteration for the inverse (Sec. 5.1): X_{n+1} = X_n (2I - A X_n), X_0 = alpha A^H -------
// alpha = 1 / max_i sum_j |(A A^H)_ij| (absolute values make alpha <= 1/sigma_max^2, so the iteration
// converges for any nonsingular A).  Every product is the complex FP64 MFMA GEMM above.

// per-row sum of |m_ij| into rs[i]
__global__ void row_abs_sum_kernel(const double2 *__restrict__ m, int n, double *__restrict__ rs) {
  const int i = blockIdx.x;
  __shared__ double red[256];
  double a = 0.0;
  for (int j = threadIdx.x; j < n; j += 256) {
    const double2 v = m[(size_t)i * n + j];
    a += sqrt(v.x * v.x + v.y * v.y);
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) rs[i] = red[0];
}

// out[0] = max of v[0..n) (one workgroup); with inv set, out[0] = 1 / max
__global__ void max_reduce_kernel(const double *__restrict__ v, int n, double *__restrict__ out, int inv) {
  __shared__ double red[256];
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) a = fmax(a, v[i]);
  red[threadIdx.x] = a;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = inv ? 1.0 / red[0] : red[0];
}

// x = alpha * a^H with alpha read from device memory
__global__ __launch_bounds__(256) void scaled_conj_transpose_kernel(const double2 *__restrict__ a, int n,
                                                                    const double *__restrict__ alpha,
                                                                    double2 *__restrict__ x) {
  __shared__ double2 t[32][33];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const double al = alpha[0];
  for (int k = 0; k < 32; k += 8) {
    const int r = r0 + ty + k, c = c0 + tx;
    if (r < n && c < n) t[ty + k][tx] = a[(size_t)r * n + c];
  }
  __syncthreads();
  for (int k = 0; k < 32; k += 8) {
    const int r = c0 + ty + k, c = r0 + tx;        // x[r][c] = alpha conj(a[c][r])
    if (r < n && c < n) {
      const double2 v = t[tx][ty + k];
      x[(size_t)r * n + c] = make_double2(al * v.x, -al * v.y);
    }
  }
}

// per-row max |x_ij - y_ij| into rm[i]
__global__ void row_max_diff_kernel(const double2 *__restrict__ x, const double2 *__restrict__ y, int n,
                                    double *__restrict__ rm) {
  const int i = blockIdx.x;
  __shared__ double red[256];
  double a = 0.0;
  for (int j = threadIdx.x; j < n; j += 256) {
    const double2 u = x[(size_t)i * n + j], v = y[(size_t)i * n + j];
    const double dx = u.x - v.x, dy = u.y - v.y;
    a = fmax(a, sqrt(dx * dx + dy * dy));
  }
  red[threadIdx.x] = a;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
    __syncthreads();
  }
  if (threadIdx.x == 0) rm[i] = red[0];
}

size_t newton_ws_bytes(int n) { return 3 * (size_t)n * n * sizeof(double2) + ((size_t)n + 64) * sizeof(double); }

hipError_t newton_start(const double2 *a, int n, double2 *x, double2 *t, double *scratch, hipStream_t s) {
  // t = A A^H, alpha = 1 / max_i sum_j |t_ij|, x = alpha A^H
  GW_TRY(zgemm(n, n, n, a, n, Z_N, a, n, Z_H, t, n, 1.0, 0.0, 0, 0, s));
  hipLaunchKernelGGL(row_abs_sum_kernel, dim3(n), dim3(256), 0, s, t, n, scratch + 64);
  GW_TRY(hipGetLastError());
  hipLaunchKernelGGL(max_reduce_kernel, dim3(1), dim3(256), 0, s, scratch + 64, n, scratch, 1);
  GW_TRY(hipGetLastError());
  dim3 g((n + 31) / 32, (n + 31) / 32);
  hipLaunchKernelGGL(scaled_conj_transpose_kernel, g, dim3(256), 0, s, a, n, scratch, x);
  return hipGetLastError();
}

hipError_t newton_step(const double2 *a, int n, const double2 *x, double2 *t, double2 *xn, double *scratch,
                       hipStream_t s) {
  // t = 2I - A X, xn = X t, scratch[1] = max |xn - x|
  const size_t nn = (size_t)n * n;
  hipLaunchKernelGGL(fill_identity_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, t, n, 2.0);
  GW_TRY(hipGetLastError());
  GW_TRY(zgemm(n, n, n, a, n, Z_N, x, n, Z_N, t, n, -1.0, 1.0, 0, 0, s));
  GW_TRY(zgemm(n, n, n, x, n, Z_N, t, n, Z_N, xn, n, 1.0, 0.0, 0, 0, s));
  hipLaunchKernelGGL(row_max_diff_kernel, dim3(n), dim3(256), 0, s, xn, x, n, scratch + 64);
  GW_TRY(hipGetLastError());
  hipLaunchKernelGGL(max_reduce_kernel, dim3(1), dim3(256), 0, s, scratch + 64, n, scratch + 1, 0);
  return hipGetLastError();
}

}  // namespace gwi
