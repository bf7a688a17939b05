// Static self-energy matrix elements in g-space (the paper's self-energy section):
//   f~_g^{nv} = sum_r exp(-i G.r) conj(u_n(r)) u_v(r)            (pair products + row transform)
//   Sigma_x(n,n')   = -sum_g V(q+g) sum_v f~_g^{nv} conj(f~_g^{n'v})
//   Sigma_sex(n,n') =  sum_v sum_g f~_g^{nv} T_g^{n'v},  T = -S conj(f~)   (T form; S on FP64 MFMA)
//   Sigma_sex(n,n') = -sum_a sigma_a sum_v zeta_a^{nv} conj(zeta_a^{n'v}),  zeta = f~^T A   (eigen form)
// The transforms are FP32 (the library's sphere passes); every contraction accumulates in FP64.
#include <algorithm>

#include "gw_internal.h"

namespace gwi {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 to_d2(float2 v) { return make_double2(v.x, v.y); }
__device__ __forceinline__ double2 to_d2(double2 v) { return v; }

// part[block][tile][16][16] = the block's share of sum_g w_g sum_v f[g][n nv + v] op(b[g][n' nv + v]) for a 16 x 16
// tile of (n, n'), op = conjugation if CONJ, on the FP64 MFMA straight from memory: in a unit of 16 consecutive v of
// one g, lane (i, kk) holds four of them (v0 + 4 kk + j) of band n0 + i of f and of band n0' + i of b, and step j
// multiplies the real and imaginary parts of all lanes' j-th values (the order of k' is free as long as both sides
// share it).  With s = -1 for op = conjugation, 1 else:
//   Re C += [Re f] . [Re b] + [-s Im f] . [Im b],   Im C += [Im f] . [Re b] + [s Re f] . [Im b].
// Bound by reading f and b once per tile row and column; one workgroup per (n, n') over all of K read them nn times
// each (16 bands, 128 occupied, 4067 G: 0.87 ms for b = f and 1.12 ms for b in FP64; 43 us each and 5 us for the sum).
constexpr int CTV = 16;         // v per unit
constexpr int CT_BLOCKS = 512;  // workgroups, over all tiles
template <bool CONJ, typename TB>
__global__ __launch_bounds__(256) void contract_kernel(const float2 *__restrict__ f, const TB *__restrict__ b, int nn,
                                                       int nv, int ng, const double *__restrict__ sv, int nt,
                                                       double2 *__restrict__ part) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int i = lane & 15, kk = lane >> 4;
  const int tn = (int)blockIdx.y / nt, tm = (int)blockIdx.y % nt;
  const int n = tn * 16 + i, m = tm * 16 + i;
  const bool nok = n < nn, mok = m < nn;
  const int nvu = (nv + CTV - 1) / CTV;
  const long long units = (long long)ng * nvu, nw = (long long)gridDim.x * 4, ld = (long long)nn * nv;
  f64x4 accR = {0.0, 0.0, 0.0, 0.0}, accI = {0.0, 0.0, 0.0, 0.0};
  const float2 *fr = f + (long long)min(n, nn - 1) * nv;
  const TB *br = b + (long long)min(m, nn - 1) * nv;
  constexpr double sg = CONJ ? -1.0 : 1.0;
#pragma unroll 2
  for (long long u = (long long)blockIdx.x * 4 + wave; u < units; u += nw) {
    const int g = (int)(u / nvu), v0 = (int)(u - (long long)g * nvu) * CTV + 4 * kk;
    const double w = sv ? sv[g] * sv[g] : 1.0;
    double2 x[4], y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = min(v0 + j, nv - 1);
      const bool in = v0 + j < nv;
      const double2 a = to_d2(fr[g * ld + v]), c = to_d2(br[g * ld + v]);
      x[j] = in && nok ? make_double2(w * a.x, w * a.y) : make_double2(0.0, 0.0);
      y[j] = in && mok ? c : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      accR = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j].x, y[j].x, accR, 0, 0, 0);
      accI = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j].y, y[j].x, accI, 0, 0, 0);
      accR = __builtin_amdgcn_mfma_f64_16x16x4f64(-sg * x[j].y, y[j].y, accR, 0, 0, 0);
      accI = __builtin_amdgcn_mfma_f64_16x16x4f64(sg * x[j].x, y[j].y, accI, 0, 0, 0);
    }
  }
  // lane holds D[4 e + kk][i] in register e: the four waves' sums in wave order
  __shared__ double2 red[4][16][17];
#pragma unroll
  for (int e = 0; e < 4; ++e) red[wave][4 * e + kk][i] = make_double2(accR[e], accI[e]);
  __syncthreads();
  const int r = tid >> 4, c = tid & 15;
  double2 s = red[0][r][c];
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    s.x += red[w][r][c].x;
    s.y += red[w][r][c].y;
  }
  part[((size_t)blockIdx.x * nt * nt + blockIdx.y) * 256 + tid] = s;
}

// out[n][n'] = scale times the sum of the blocks' shares: one wave per output
__global__ __launch_bounds__(64) void contract_sum_kernel(const double2 *__restrict__ part, int nblk, int nt, int nn,
                                                          double scale, double2 *__restrict__ out) {
  const int n = blockIdx.x / nn, m = blockIdx.x % nn;
  const size_t at = (size_t)((n >> 4) * nt + (m >> 4)) * 256 + (n & 15) * 16 + (m & 15);
  double re = 0.0, im = 0.0;
  for (int q = threadIdx.x; q < nblk; q += 64) {
    const double2 v = part[(size_t)q * nt * nt * 256 + at];
    re += v.x;
    im += v.y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    re += __shfl_xor(re, off, 64);
    im += __shfl_xor(im, off, 64);
  }
  if (threadIdx.x == 0) out[blockIdx.x] = make_double2(scale * re, scale * im);
}

// out[n][n'] = -sum_a sigma_a sum_v zeta[a][n*nv+v] conj(zeta[a][n'*nv+v]); one workgroup per (n, n')
__global__ __launch_bounds__(256) void contract_modes_kernel(const double2 *__restrict__ zeta, int nm, int nv, int nn,
                                                             const double *__restrict__ sigma,
                                                             double2 *__restrict__ out) {
  const int n = blockIdx.x / nn, np = blockIdx.x % nn;
  __shared__ double rr[256], ri[256];
  double sr = 0.0, si = 0.0;
  for (int idx = threadIdx.x; idx < nm * nv; idx += 256) {
    const int a = idx / nv, v = idx % nv;
    const double2 x = zeta[((size_t)a * nn + n) * nv + v], y = zeta[((size_t)a * nn + np) * nv + v];
    const double s = sigma[a];
    sr += s * (x.x * y.x + x.y * y.y);       // x conj(y)
    si += s * (x.y * y.x - x.x * y.y);
  }
  rr[threadIdx.x] = sr;
  ri[threadIdx.x] = si;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      rr[threadIdx.x] += rr[threadIdx.x + st];
      ri[threadIdx.x] += ri[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[(size_t)n * nn + np] = make_double2(-rr[0], -ri[0]);
}

// blocks of K: at least four units for each of a block's four waves, and partial sums no larger than two copies of
// the pair products on the grid (which bounds calls with one pair)
int contract_blocks(int nn, int nv, int ng, int nr) {
  const long long units = (long long)ng * ((nv + CTV - 1) / CTV), nt2 = (long long)((nn + 15) / 16) * ((nn + 15) / 16);
  return (int)std::max(1LL, std::min({CT_BLOCKS / nt2, units / 16, (long long)nn * nv * nr / (256 * nt2)}));
}
size_t contract_part_elems(int nn, int nblk) {
  const int nt = (nn + 15) / 16;
  return (size_t)nblk * nt * nt * 256;
}

template <bool CONJ, typename TB>
static hipError_t contract(const float2 *f, const TB *b, int nn, int nv, int ng, const double *sv, double scale,
                           int nblk, double2 *part, double2 *out, hipStream_t s) {
  const int nt = (nn + 15) / 16;
  hipLaunchKernelGGL(HIP_KERNEL_NAME(contract_kernel<CONJ, TB>), dim3(nblk, nt * nt), dim3(256), 0, s, f, b, nn, nv, ng,
                     sv, nt, part);
  hipLaunchKernelGGL(contract_sum_kernel, dim3(nn * nn), dim3(64), 0, s, part, nblk, nt, nn, scale, out);
  return hipGetLastError();
}

hipError_t launch_contract_x(const float2 *f, int nn, int nv, int ng, const double *sv, double scale, int nblk,
                             double2 *part, double2 *out, hipStream_t s) {
  return contract<true>(f, f, nn, nv, ng, sv, scale, nblk, part, out, s);
}

hipError_t launch_contract_t(const float2 *f, const double2 *t, int nn, int nv, int ng, double scale, int nblk,
                             double2 *part, double2 *out, hipStream_t s) {
  return contract<false>(f, t, nn, nv, ng, (const double *)nullptr, scale, nblk, part, out, s);
}

hipError_t launch_contract_modes(const double2 *zeta, int nm, int nv, int nn, const double *sigma, double2 *out,
                                 hipStream_t s) {
  hipLaunchKernelGGL(contract_modes_kernel, dim3(nn * nn), dim3(256), 0, s, zeta, nm, nv, nn, sigma, out);
  return hipGetLastError();
}

}  // namespace gwi
