// Pair products f_vc(r) = conj(u_v(r)) u_c(r) sqrt(p/(E_c - E_v))  (Eq.(fdef)) and the scale table.
//
// Bound by writing nv*nc*nr complex64 values.  A workgroup owns a segment of P grid points, VB occupied
// and CB unoccupied bands: their values at the segment pass through LDS once and serve VB * CB rows of F.
// Rows of F start anywhere in a 128-byte line (nr need not be a multiple of 16), so each row's segment runs from
// line boundary to line boundary, and a wave stores whole lines, 1 KB per instruction, whatever nr is: stores
// that straddled lines reached 3.6 TB/s at nr = 19683 (27^3) and 4.2 at 19684, against 5.1 on rows that are aligned
// anyway; with whole lines 5.2 to 5.4 on all of them (12 x 200 bands; a plain fill of that size 6.9).  On small grids
// the segment of 512 points (1024 before) also leaves fewer CUs idle: 16 x 100 bands on 15^3 38 -> 20 us a call.
// Segments by VB x CB at nr = 19683: 512 by 8 x 4 79 us, 256 by 8 x 8 79, 384 by 8 x 8 80, 512 by 8 x 8 83, 1024 by
// 4 x 4 86, 512 by 4 x 8 88; at 36^3, 8 x 256 bands, 142, 150, 148, 145, 148 and 146 us.  Stores that are not
// non-temporal: 3 to 20% slower.
// The occupied bands are split evenly over as few blocks of at most 8 as hold them, and a block loads as many rows as
// it has: with blocks of 8 throughout, 9 x 500 bands on 24^3 took 112 us (kernel alone; blocks of 5 87, a kernel that
// loops over the occupied bands 100), 12 x 200 on 27^3 74 (6: 70), 10 x 490 on 18^3 54 (5: 45).  With four bands or
// fewer the segment is 256 points by 4 x 4 or 3 x 4 (2 x 600 bands on 20^3 23.4 -> 18.7 us, 3 x 500 on 24^3 37.5 ->
// 34.1), with one 512 by 1 x 4 (600 bands on 20^3 17.8 -> 12.2).
#include <algorithm>
#include <type_traits>

#include "gw_internal.h"

namespace gwi {

int scale_ld(int nc) { return (nc + 31) / 32 * 32; }
size_t scale_table_floats(int nv, int nc) { return (size_t)2 * nv * scale_ld(nc); }

// s_vc = sqrt(p / (E_c - E_v)) in [nv][ldsc], then s_vc^2 = p / (E_c - E_v) in a second [nv][ldsc] table
// (the planar wide update scales only its row side, by s^2); zero for c >= nc in both
__global__ void scale_table_kernel(const double *__restrict__ e_v, int nv, const double *__restrict__ e_c, int nc,
                                   double prefactor, float *__restrict__ scale, int ldsc) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nv * ldsc) return;
  const int v = idx / ldsc, c = idx - v * ldsc;
  const double q = c < nc ? prefactor / (e_c[c] - e_v[v]) : 0.0;
  scale[idx] = (float)sqrt(q);
  scale[(size_t)nv * ldsc + idx] = (float)q;
}

// Energies in the kernel's own arguments (a copy made at the launch) instead of two copies from pageable memory,
// which the host stages and waits for: 12 x 200 bands on 27^3 138.8 -> 136.2 us a call, 12^3 FP32 build 130 -> 127.
// ENERGY_ARG doubles fit beside the other arguments into the 4 KB a launch takes; a longer list goes by the copies
// (2 x 600 bands on 20^3: in three launches 30.1 us a call, 29.3 by copies; 2 x 800 on 16^3 26.3 and 23.2).  Under capture any list goes by
// copies: a graph whose launches held the energies would replay those of the capture, copies read the caller's arrays
// at every replay.
constexpr int ENERGY_ARG = 488;
struct EnergyArg { double e[ENERGY_ARG]; };

__global__ void energies_kernel(EnergyArg a, int n, double *__restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a.e[i];
}

bool pair_energies_fit(int nv, int nc) { return (long long)nv + nc <= ENERGY_ARG; }

// dev[0 .. nv) = e_v, dev[nv .. nv + nc) = e_c (host arrays, read before the call returns unless it is captured)
hipError_t upload_energies(const double *e_v, int nv, const double *e_c, int nc, double *dev, hipStream_t s) {
  if (pair_energies_fit(nv, nc) && !stream_capturing(s)) {
    EnergyArg a;
    std::copy(e_v, e_v + nv, a.e);
    std::copy(e_c, e_c + nc, a.e + nv);
    hipLaunchKernelGGL(energies_kernel, dim3((nv + nc + 255) / 256), dim3(256), 0, s, a, nv + nc, dev);
    return hipGetLastError();
  }
  const hipError_t e = hipMemcpyAsync(dev, e_v, (size_t)nv * sizeof(double), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return e;
  return hipMemcpyAsync(dev + nv, e_c, (size_t)nc * sizeof(double), hipMemcpyHostToDevice, s);
}

hipError_t launch_scale_table(const double *e_v, int nv, const double *e_c, int nc, double prefactor, float *scale,
                              int ldsc, hipStream_t s) {
  const int n = nv * ldsc;
  hipLaunchKernelGGL(scale_table_kernel, dim3((n + 255) / 256), dim3(256), 0, s, e_v, nv, e_c, nc, prefactor, scale,
                     ldsc);
  return hipGetLastError();
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float2 conj_mul_scale(float2 v, float2 c, float s) {
  // conj(v) * c * s
  return make_float2((v.x * c.x + v.y * c.y) * s, (v.x * c.y - v.y * c.x) * s);
}

constexpr int PP_THREADS = 256;
constexpr int PP_CB = 4;       // unoccupied bands per workgroup
constexpr int PP_LINE = 16;    // values in a 128-byte line

// The pair scales come from the table, or (ARG) from the energies in the arguments: no launch before this one.
// P points of VB occupied bands per workgroup.
template <int P, int VB, bool ARG>
__global__ __launch_bounds__(PP_THREADS) void pair_products_kernel(const float2 *__restrict__ psi_v, int nv,
                                                                   const float2 *__restrict__ psi_c, int nc, int nr,
                                                                   int cbase, const float *__restrict__ scale, int ldsc,
                                                                   double prefactor, float2 *__restrict__ f,
                                                                   std::conditional_t<ARG, EnergyArg, int> energies) {
  __shared__ float2 sv[VB][P + PP_LINE], sc[PP_CB][P + PP_LINE];
  __shared__ float ss[VB][PP_CB];
  static_assert(P % PP_LINE == 0, "a segment's end falls on the line boundary its start is shifted to");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nvb = (nv + VB - 1) / VB;
  const int v0 = ((int)blockIdx.x % nvb) * VB, p0 = ((int)blockIdx.x / nvb) * P;
  const int c0 = cbase + (int)blockIdx.y * PP_CB;
  const int mv = min(VB, nv - v0), mc = min(PP_CB, nc - c0);
  const int np = min(P + PP_LINE, nr - p0);
  for (int i = tid; i < P + PP_LINE; i += PP_THREADS) {
    const int q = min(i, np - 1);
#pragma unroll
    for (int k = 0; k < VB; ++k) sv[k][i] = psi_v[(size_t)min(v0 + k, nv - 1) * nr + p0 + q];
#pragma unroll
    for (int k = 0; k < PP_CB; ++k) sc[k][i] = psi_c[(size_t)min(c0 + k, nc - 1) * nr + p0 + q];
  }
  if (tid < VB * PP_CB) {
    const int k = tid / PP_CB, j = tid % PP_CB;
    const int v = min(v0 + k, nv - 1), c = min(c0 + j, nc - 1);
    if constexpr (ARG) ss[k][j] = (float)sqrt(prefactor / (energies.e[nv + c] - energies.e[v]));
    else ss[k][j] = scale[(size_t)v * ldsc + c];
  }
  __syncthreads();
  const int a0 = (int)((reinterpret_cast<uintptr_t>(f) >> 3) & (PP_LINE - 1));
  for (int row = wave; row < mv * PP_CB; row += PP_THREADS / 64) {
    const int k = row / PP_CB, j = row % PP_CB;
    if (j >= mc) continue;
    const size_t at = ((size_t)(v0 + k) * nc + c0 + j) * nr + p0;      // the segment's first value in F
    float2 *out = f + at;
    // From the first line boundary (the row's start for its first segment) to the first one past the segment
    // (the row's end for its last); a wave's stores start at a boundary, if need be before the row's start.
    const int off = (int)((a0 + at) & (PP_LINE - 1)), sh = (PP_LINE - off) & (PP_LINE - 1);
    const int beg = p0 == 0 ? 0 : sh, end = min(P + sh, nr - p0);   // P is a multiple of a line
    const float s = ss[k][j];
    for (int i = (p0 == 0 ? -off : sh) + 2 * lane; i < end; i += 128) {
      const int x = max(i, 0), y = max(min(i + 1, np - 1), 0);
      const float2 a = conj_mul_scale(sv[k][x], sc[j][x], s), b = conj_mul_scale(sv[k][y], sc[j][y], s);
      if (i >= beg && i + 1 < end) {
        const f32x4 w = {a.x, a.y, b.x, b.y};
        __builtin_nontemporal_store(w, reinterpret_cast<f32x4 *>(out + i));
      } else {
        if (i >= beg && i < end) out[i] = a;
        if (i + 1 >= beg && i + 1 < end) out[i + 1] = b;
      }
    }
  }
}

template <int P, int VB, bool ARG>
static hipError_t launch_pairs_tile(const float2 *psi_v, int nv, const float2 *psi_c, int nc, int nr, const float *scale,
                                    int ldsc, double prefactor, float2 *f, std::conditional_t<ARG, EnergyArg, int> e,
                                    hipStream_t s) {
  constexpr int CY = 65535 * PP_CB;                    // unoccupied bands per launch
  for (int cb = 0; cb < nc; cb += CY) {
    const dim3 grid(((nr + P - 1) / P) * ((nv + VB - 1) / VB), (std::min(CY, nc - cb) + PP_CB - 1) / PP_CB);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(pair_products_kernel<P, VB, ARG>), grid, dim3(PP_THREADS), 0, s, psi_v, nv, psi_c,
                       nc, nr, cb, scale, ldsc, prefactor, f, e);
  }
  return hipGetLastError();
}

template <bool ARG>
static hipError_t launch_pairs(const float2 *psi_v, int nv, const float2 *psi_c, int nc, int nr, const float *scale,
                               int ldsc, double prefactor, float2 *f, std::conditional_t<ARG, EnergyArg, int> e,
                               hipStream_t s) {
  const int blocks = (int)((nv + 7ll) / 8);
  switch ((nv + blocks - 1) / blocks) {
    case 1: return launch_pairs_tile<512, 1, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
    case 3: return launch_pairs_tile<256, 3, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
    case 2:
    case 4: return launch_pairs_tile<256, 4, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
    case 5: return launch_pairs_tile<512, 5, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
    case 6: return launch_pairs_tile<512, 6, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
    case 7: return launch_pairs_tile<512, 7, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
    default: return launch_pairs_tile<512, 8, ARG>(psi_v, nv, psi_c, nc, nr, scale, ldsc, prefactor, f, e, s);
  }
}

hipError_t launch_pair_products(const float2 *psi_v, int nv, const float2 *psi_c, int nc, int nr, const float *scale,
                                int ldsc, float2 *f, hipStream_t s) {
  return launch_pairs<false>(psi_v, nv, psi_c, nc, nr, scale, ldsc, 1.0, f, 0, s);
}

hipError_t launch_pair_products_e(const float2 *psi_v, int nv, const float2 *psi_c, int nc, int nr, const double *e_v,
                                  const double *e_c, double prefactor, float2 *f, hipStream_t s) {
  if (!pair_energies_fit(nv, nc)) return hipErrorInvalidValue;
  EnergyArg a;
  std::copy(e_v, e_v + nv, a.e);
  std::copy(e_c, e_c + nc, a.e + nv);
  return launch_pairs<true>(psi_v, nv, psi_c, nc, nr, nullptr, 0, prefactor, f, a, s);
}

}  // namespace gwi
