// Learned band-tail correction of the truncated unoccupied-band sum.
//
// The paper lists the truncation of the unoccupied-band sum of Eq.(Pstatic) as its first
// technical issue.  This correction predicts, per G, the missing part of P~ from a truncated
// build:  dP~ = -(diag(d) + U U^H) with d_G = softplus(o_G0) s_G and
// u_Gk = (o_G,1+k + i o_G,17+k) sqrt(s_G) for k < r (zero beyond; the rank r <= 16 is a model setting),
// s_G = |Re P~_Nc(G,G)|, where o_G is a 4-128-128-33
// MLP (SiLU, BF16 weights, FP32 arithmetic) of the raw features
// x_G = (|q+G|, log|Re P~_Nc(G,G)|, Nc/N_g, E_max) normalised by stored mean and std.
// Training minimises ||dP~ - T||_F^2 / ||T||_F^2 with T = H(P~_4Nc) - H(P~_Nc), H(X) = (X+X^H)/2.
//
// These are small dense products (widths <= 128, N_g <= a few thousand), bound by latency rather than by
// arithmetic, so a training step is four launches, each carrying blocks of rows through every stage that needs
// no other rows, with FP32 accumulation.
#include <algorithm>

#include "gw_internal.h"

namespace gwi {

constexpr int TW = 128;     // hidden width
constexpr int TO = 33;      // outputs: 1 + 2 * TR
constexpr int TR = 16;      // rank of the off-diagonal part

__device__ __forceinline__ float bf2f(const __bf16 x) { return (float)x; }
__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = sigm(z);
  return s * (1.0f + z * (1.0f - s));
}
__device__ __forceinline__ float softplus(float z) { return z > 20.f ? z : log1pf(expf(z)); }

// ---- features and target -------------------------------------------------------------------------
__global__ void tail_features_kernel(const float2 *__restrict__ p, int ng, const int *__restrict__ miller, double q0,
                                     double q1, double q2, double a_bohr, int nc, double e_max,
                                     float *__restrict__ feat) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ng) return;
  const double b = 2.0 * 3.14159265358979323846 / a_bohr;
  const double x = (miller[3 * g] + q0) * b, y = (miller[3 * g + 1] + q1) * b, z = (miller[3 * g + 2] + q2) * b;
  const float diag = fabsf(p[(size_t)g * ng + g].x);
  feat[4 * g + 0] = (float)sqrt(x * x + y * y + z * z);
  feat[4 * g + 1] = logf(fmaxf(diag, 1e-30f));
  feat[4 * g + 2] = (float)nc / (float)ng;
  feat[4 * g + 3] = (float)e_max;
}

// T = H(full) - H(trunc), 32x32 tiles with the transposed partners through LDS.
__global__ __launch_bounds__(256) void tail_target_kernel(const float2 *__restrict__ full,
                                                          const float2 *__restrict__ trunc, int ng,
                                                          float2 *__restrict__ t) {
  __shared__ float2 tf[32][33], tt[32][33];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = 0; k < 32; k += 8) {
    const int r = c0 + ty + k, c = r0 + tx;
    if (r < ng && c < ng) {
      tf[ty + k][tx] = full[(size_t)r * ng + c];
      tt[ty + k][tx] = trunc[(size_t)r * ng + c];
    }
  }
  __syncthreads();
  for (int k = 0; k < 32; k += 8) {
    const int g = r0 + ty + k, gp = c0 + tx;
    if (g < ng && gp < ng) {
      const float2 a = full[(size_t)g * ng + gp], at = tf[tx][ty + k];
      const float2 b = trunc[(size_t)g * ng + gp], bt = tt[tx][ty + k];
      t[(size_t)g * ng + gp] = make_float2(0.5f * (a.x + at.x) - 0.5f * (b.x + bt.x),
                                           0.5f * (a.y - at.y) - 0.5f * (b.y - bt.y));
    }
  }
}

// ---- MLP forward and head ---------------------------------------------------------------------------
// Every layer and the head depend on one row of the features only, so one workgroup carries TRB rows
// through all of them: the weights and the rows' activations stay in LDS, the launches and the memory
// round trips between layers go.  What bounds it is latency (20 kFMA per row): at 925 rows the four
// separate kernels took 28 us and four launches, this one takes 20 us and writes the parts of U^H U too.
//
// Row blocks of TRB rows; 256 threads: thread (j = t % 128, half = t / 128) forms output j of eight rows,
// one weight read and two broadcast reads of eight activations per input ([input][row] layout).
constexpr int TRB = 16;          // rows per block
constexpr int TRS = TRB + 4;     // LDS stride of an [input][row] activation tile, in floats

// word i of the BF16 array src (values 2i, 2i + 1); the caller's array may be aligned to two bytes only
__device__ __forceinline__ unsigned bf16_pair(const __bf16 *__restrict__ src, int i, bool aligned) {
  if (aligned) return reinterpret_cast<const unsigned *>(src)[i];           // uniform
  const unsigned short *h = reinterpret_cast<const unsigned short *>(src);
  return (unsigned)h[2 * i] | ((unsigned)h[2 * i + 1] << 16);
}

// o = MLP(x) for every row; with a training or head pass also the stored intermediates (xn, z1, h1, z2, h2),
// d_G and u_Gk, and each block's part of U^H U (gpart [block][16][16]).  The first workgroup also sets
// (set_step >= 0) or advances (set_step < 0) the Adam step count for the launches that follow.
__global__ __launch_bounds__(256) void tail_forward_kernel(const float *__restrict__ feat, int n,
                                                           const __bf16 *__restrict__ w, const float *__restrict__ bias,
                                                           const float *__restrict__ norm, int rank,
                                                           float *__restrict__ xn, float *__restrict__ z1,
                                                           float *__restrict__ h1, float *__restrict__ z2,
                                                           float *__restrict__ h2, float *__restrict__ o,
                                                           float *__restrict__ d, float2 *__restrict__ u,
                                                           float2 *__restrict__ gpart, int *__restrict__ step_dev,
                                                           int set_step) {
  __shared__ __attribute__((aligned(16))) unsigned sw[(4 * TW + TW * TW + TW * TO) / 2];   // W1, W2, W3
  __shared__ __attribute__((aligned(16))) float sa[TW][TRS], sb[TW][TRS];   // h1 and h2, [unit][row]
  __shared__ float so[TRB][TO + 1];
  __shared__ float2 su[TRB][TR];
  __shared__ float sx[TRB][4];
  const int tid = threadIdx.x;
  const int g0 = blockIdx.x * TRB, rows = min(TRB, n - g0);
  if (step_dev && blockIdx.x == 0 && tid == 0) step_dev[0] = set_step >= 0 ? set_step : step_dev[0] + 1;
  static_assert((4 * TW + TW * TW + TW * TO) % 2 == 0, "weights copied as 32-bit words");
  {
    const bool al = (reinterpret_cast<uintptr_t>(w) & 3) == 0;
#pragma unroll 8
    for (int i = tid; i < (4 * TW + TW * TW + TW * TO) / 2; i += 256) sw[i] = bf16_pair(w, i, al);
  }
  if (tid < TRB * 4) {
    const int r = tid / 4, i = tid % 4;
    const float x = r < rows ? (feat[4 * (size_t)(g0 + r) + i] - norm[i]) / norm[4 + i] : 0.f;
    sx[r][i] = x;
    if (xn && r < rows) xn[4 * (size_t)(g0 + r) + i] = x;
  }
  __syncthreads();
  const __bf16 *w1 = reinterpret_cast<const __bf16 *>(sw), *w2 = w1 + 4 * TW, *w3 = w2 + TW * TW;
  const int j = tid & (TW - 1), r0 = (tid >> 7) * (TRB / 2);
  {
    float acc[TRB / 2];
    const float b0 = bias[j];
#pragma unroll
    for (int r = 0; r < TRB / 2; ++r) acc[r] = b0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float wv = bf2f(w1[i * TW + j]);
#pragma unroll
      for (int r = 0; r < TRB / 2; ++r) acc[r] += sx[r0 + r][i] * wv;
    }
#pragma unroll
    for (int r = 0; r < TRB / 2; ++r) {
      const float h = silu(acc[r]);
      sa[j][r0 + r] = h;
      if (z1 && r0 + r < rows) {
        z1[(size_t)(g0 + r0 + r) * TW + j] = acc[r];
        h1[(size_t)(g0 + r0 + r) * TW + j] = h;
      }
    }
  }
  __syncthreads();
  {
    float acc[TRB / 2];
    const float b0 = bias[TW + j];
#pragma unroll
    for (int r = 0; r < TRB / 2; ++r) acc[r] = b0;
#pragma unroll 8
    for (int k = 0; k < TW; ++k) {
      const float wv = bf2f(w2[k * TW + j]);
#pragma unroll
      for (int r = 0; r < TRB / 2; ++r) acc[r] += sa[k][r0 + r] * wv;
    }
#pragma unroll
    for (int r = 0; r < TRB / 2; ++r) {
      const float h = silu(acc[r]);
      sb[j][r0 + r] = h;
      if (z2 && r0 + r < rows) {
        z2[(size_t)(g0 + r0 + r) * TW + j] = acc[r];
        h2[(size_t)(g0 + r0 + r) * TW + j] = h;
      }
    }
  }
  __syncthreads();
  for (int idx = tid; idx < TRB * TO; idx += 256) {
    const int r = idx / TO, m = idx - r * TO;
    float acc = bias[2 * TW + m];
#pragma unroll 8
    for (int k = 0; k < TW; ++k) acc += sb[k][r] * bf2f(w3[k * TO + m]);
    so[r][m] = acc;
    if (r < rows) o[(size_t)g0 * TO + idx] = acc;
  }
  if (!d) return;
  __syncthreads();
  const int r = tid / TR, k = tid % TR;
  static_assert(TRB * TR == 256, "one (row, column of U) per thread");
  float2 uv = make_float2(0.f, 0.f);
  if (r < rows) {
    const float s = expf(feat[4 * (size_t)(g0 + r) + 1]);
    const float rs = sqrtf(s);
    if (k == 0) d[g0 + r] = softplus(so[r][0]) * s;
    if (k < rank) uv = make_float2(so[r][1 + k] * rs, so[r][1 + TR + k] * rs);
    u[(size_t)(g0 + r) * TR + k] = uv;
  }
  if (!gpart) return;
  su[r][k] = uv;
  __syncthreads();
  const int gk = tid / TR, gl = tid % TR;
  float2 acc = make_float2(0.f, 0.f);
#pragma unroll
  for (int q = 0; q < TRB; ++q) {
    const float2 a = su[q][gk], b = su[q][gl];      // conj(a) b
    acc.x += a.x * b.x + a.y * b.y;
    acc.y += a.x * b.y - a.y * b.x;
  }
  gpart[(size_t)blockIdx.x * TR * TR + tid] = acc;
}

// ---- W = T U, ||T||^2 and G = U^H U ----------------------------------------------------------------
// TUR rows of T per workgroup, 256 threads = 16 columns of U x 16 parts of the sum over g': a row's values
// pass through LDS once (coalesced) and each U value loaded serves TUR rows, so the kernel reads T once and
// U n / TUR times from cache.  (One workgroup per row with every thread holding all 33 sums spent its time in a
// 33-value LDS tree: 20.7 us at n = 925, against 11 us.)  The last workgroup sums the forward pass's
// parts of G; tpart holds each workgroup's part of ||T||^2.
constexpr int TUR = 4;
constexpr int TUC = 1024;        // g' per LDS chunk
__global__ __launch_bounds__(256) void tail_tu_kernel(const float2 *__restrict__ t, const float2 *__restrict__ u,
                                                      int n, float2 *__restrict__ w, float *__restrict__ tpart,
                                                      const float2 *gpart, int ngpart, float2 *gm) {
  __shared__ float2 st[TUR][TUC];
  __shared__ float2 red[16][TUR][TR];
  __shared__ float rt[4];
  const int tid = threadIdx.x;
  const int nblk = (n + TUR - 1) / TUR;
  if ((int)blockIdx.x == nblk) {                    // G = sum of the parts, in block order
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll 8
    for (int b = 0; b < ngpart; ++b) {
      const float2 v = gpart[(size_t)b * TR * TR + tid];
      acc.x += v.x;
      acc.y += v.y;
    }
    gm[tid] = acc;
    return;
  }
  const int g0 = blockIdx.x * TUR, rows = min(TUR, n - g0);
  const int k = tid % TR, part = tid / TR;
  float2 acc[TUR];
#pragma unroll
  for (int r = 0; r < TUR; ++r) acc[r] = make_float2(0.f, 0.f);
  float tn = 0.f;
  for (int c0 = 0; c0 < n; c0 += TUC) {
    const int cn = min(TUC, n - c0);
    if (c0) __syncthreads();
#pragma unroll
    for (int r = 0; r < TUR; ++r)
#pragma unroll
      for (int i = 0; i < TUC / 256; ++i) {
        const int c = tid + 256 * i;
        float2 v = make_float2(0.f, 0.f);
        if (r < rows && c < cn) v = t[(size_t)(g0 + r) * n + c0 + c];
        st[r][c] = v;
        tn += v.x * v.x + v.y * v.y;
      }
    __syncthreads();
#pragma unroll 8
    for (int c = part; c < cn; c += 16) {
      const float2 b = u[(size_t)(c0 + c) * TR + k];
#pragma unroll
      for (int r = 0; r < TUR; ++r) {
        const float2 a = st[r][c];
        acc[r].x += a.x * b.x - a.y * b.y;
        acc[r].y += a.x * b.y + a.y * b.x;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < TUR; ++r) red[part][r][k] = acc[r];
  for (int off = 32; off > 0; off >>= 1) tn += __shfl_down(tn, off, 64);
  if ((tid & 63) == 0) rt[tid >> 6] = tn;
  __syncthreads();
  if (tid < TUR * TR) {
    const int r = tid / TR, kk = tid % TR;
    float2 s = make_float2(0.f, 0.f);
#pragma unroll
    for (int p = 0; p < 16; ++p) {
      s.x += red[p][r][kk].x;
      s.y += red[p][r][kk].y;
    }
    if (r < rows) w[(size_t)(g0 + r) * TR + kk] = s;
  }
  if (tid == 0) tpart[blockIdx.x] = (rt[0] + rt[1]) + (rt[2] + rt[3]);
}

// Sum of v[0..n) over the workgroup's 256 threads, the result in every thread.
__device__ __forceinline__ float block_sum(const float *__restrict__ v, int n, float *red4) {
  float a = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) a += v[i];
  for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red4[threadIdx.x >> 6] = a;
  __syncthreads();
  return (red4[0] + red4[1]) + (red4[2] + red4[3]);
}

// ---- d loss / d o, the way back through the layers, and the weight gradients --------------------------
// Per row g: B U = d U + U G + W, B_gg = d + |u|^2 + Re T_gg, the loss terms of row g and d loss / d o; then
// dz2 = (go W3^T) silu'(z2) and dz1 = (dz2 W2^T) silu'(z1), which need nothing but the row.  So one workgroup
// takes blocks of TRB rows through all of it in LDS and adds their outer products h2 go, h1 dz2, xn dz1 to
// gradients that it keeps in registers (85 per thread) over all its blocks; it stores one partial gradient
// at the end, and the Adam kernel adds the partials.  (Before: one thread per weight walking all rows, a
// serial chain of n loads: three weight, three bias and two backward kernels took 970 us at n = 925 against
// 27 us for this one.)  lpart receives each workgroup's part of the loss; with gpar = nullptr only that.
constexpr int TWS = TW + 2;      // LDS row stride of W2 in BF16 values: 65 words, so lanes on rows hit all banks
constexpr int TGP = 21409 + 31;  // floats of one partial gradient, padded (a multiple of 32)
__global__ __launch_bounds__(256) void tail_backward_kernel(
    const float *__restrict__ o, const float *__restrict__ feat, const float *__restrict__ d,
    const float2 *__restrict__ u, const float2 *__restrict__ w, const float2 *__restrict__ gm,
    const float2 *__restrict__ t, int n, int rank, const float *__restrict__ tpart, int ntpart,
    const __bf16 *__restrict__ wts, const float *__restrict__ xn, const float *__restrict__ z1,
    const float *__restrict__ h1, const float *__restrict__ z2, const float *__restrict__ h2,
    float *__restrict__ lpart, float *__restrict__ gpar) {
  __shared__ __attribute__((aligned(16))) unsigned sw2[TW * TWS / 2];
  __shared__ __bf16 sw3[TW * TO];
  __shared__ float2 sg[TR][TR];
  __shared__ __attribute__((aligned(16))) float sh1[TRB][TW], sh2[TRB][TW], sd1[TRB][TW], sd2[TRB][TW];
  __shared__ float sgo[TRB][TO + 1];
  __shared__ float2 su[TRB][TR], sv[TRB][TR];
  __shared__ float sx[TRB][4], sdg[TRB], stg[TRB], srs[TRB], sl[TRB];
  __shared__ float red4[4];
  const int tid = threadIdx.x;
  const bool grads = gpar != nullptr;
  if (grads) {
    const bool al = (reinterpret_cast<uintptr_t>(wts) & 3) == 0;
#pragma unroll 8
    for (int i = tid; i < TW * TW / 2; i += 256)
      sw2[(i / (TW / 2)) * (TWS / 2) + i % (TW / 2)] = bf16_pair(wts + 4 * TW, i, al);
#pragma unroll 8
    for (int i = tid; i < TW * TO; i += 256) sw3[i] = wts[4 * TW + TW * TW + i];
  }
  sg[tid / TR][tid % TR] = gm[tid];
  const float inv = 1.0f / block_sum(tpart, ntpart, red4);
  // gradient accumulators: W2 rows 8 ti .. +7 x columns 8 tj .. +7, W3 row tid / 2 x 17 (16) columns,
  // W1 row tid / 64 x two columns, two biases at most
  const int ti = tid / 16, tj = tid % 16;
  float a2[8][8], a3[17], a1[2] = {0.f, 0.f}, ab[2] = {0.f, 0.f};
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) a2[a][b] = 0.f;
#pragma unroll
  for (int a = 0; a < 17; ++a) a3[a] = 0.f;
  float lsum = 0.f;
  const int nblk = (n + TRB - 1) / TRB;
  for (int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int g0 = blk * TRB, rows = min(TRB, n - g0);
    __syncthreads();
    {
      const int r = tid / TR, k = tid % TR;
      const bool in = r < rows;
      su[r][k] = in ? u[(size_t)(g0 + r) * TR + k] : make_float2(0.f, 0.f);
      sv[r][k] = in ? w[(size_t)(g0 + r) * TR + k] : make_float2(0.f, 0.f);
      if (k == 0) {
        sdg[r] = in ? d[g0 + r] : 0.f;
        stg[r] = in ? t[(size_t)(g0 + r) * n + g0 + r].x : 0.f;
        srs[r] = in ? expf(feat[4 * (size_t)(g0 + r) + 1]) : 0.f;
      }
      if (grads) {
        if (k < 4) sx[r][k] = in ? xn[4 * (size_t)(g0 + r) + k] : 0.f;
#pragma unroll
        for (int i = 0; i < TRB * TW / 256; ++i) {
          const int idx = tid + 256 * i, q = idx / TW, c = idx % TW;
          sh1[q][c] = q < rows ? h1[(size_t)(g0 + q) * TW + c] : 0.f;
          sh2[q][c] = q < rows ? h2[(size_t)(g0 + q) * TW + c] : 0.f;
        }
      }
    }
    __syncthreads();
    {
      const int r = tid / TR, k = tid % TR;
      const float s = srs[r], rs = sqrtf(s), dg = sdg[r], tgg = stg[r];
      // |u|^2 and Re(conj(u) w) of the row, over its 16 lanes
      const float2 uk = su[r][k], wk = sv[r][k];
      float u2 = uk.x * uk.x + uk.y * uk.y, uw = uk.x * wk.x + uk.y * wk.y;
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) {
        u2 += __shfl_xor(u2, off, 64);
        uw += __shfl_xor(uw, off, 64);
      }
      if (k == 0) {
        const float bgg = dg + u2 + tgg;
        sgo[r][0] = r < rows ? 2.0f * bgg * sigm(o[(size_t)(g0 + r) * TO]) * s * inv : 0.f;
        sl[r] = dg * dg + 2.0f * dg * tgg + 2.0f * dg * u2 + 2.0f * uw;
      }
      float2 bu = make_float2(dg * uk.x + wk.x, dg * uk.y + wk.y);
#pragma unroll
      for (int l = 0; l < TR; ++l) {
        const float2 a = su[r][l], c = sg[l][k];
        bu.x += a.x * c.x - a.y * c.y;
        bu.y += a.x * c.y + a.y * c.x;
      }
      sgo[r][1 + k] = k < rank ? 4.0f * bu.x * rs * inv : 0.f;        // unused columns: no gradient
      sgo[r][1 + TR + k] = k < rank ? 4.0f * bu.y * rs * inv : 0.f;
    }
    __syncthreads();
    if (tid == 0) {
      float a = 0.f;
      for (int r = 0; r < rows; ++r) a += sl[r];
      lsum += a;
    }
    if (!grads) continue;
    const int i = tid & (TW - 1), r0 = (tid >> 7) * (TRB / 2);       // unit i of rows r0 .. r0 + 7
    {
      float acc[TRB / 2];
#pragma unroll
      for (int r = 0; r < TRB / 2; ++r) acc[r] = 0.f;
#pragma unroll
      for (int j = 0; j < TO; ++j) {
        const float wv = bf2f(sw3[i * TO + j]);
#pragma unroll
        for (int r = 0; r < TRB / 2; ++r) acc[r] += sgo[r0 + r][j] * wv;
      }
#pragma unroll
      for (int r = 0; r < TRB / 2; ++r)
        sd2[r0 + r][i] = r0 + r < rows ? acc[r] * dsilu(z2[(size_t)(g0 + r0 + r) * TW + i]) : 0.f;
    }
    __syncthreads();
    {
      float acc[TRB / 2];
#pragma unroll
      for (int r = 0; r < TRB / 2; ++r) acc[r] = 0.f;
#pragma unroll 4
      for (int j2 = 0; j2 < TW / 2; ++j2) {
        const unsigned wp = sw2[i * (TWS / 2) + j2];                  // W2[i][2 j2], W2[i][2 j2 + 1]
        const float wa = __builtin_bit_cast(float, wp << 16), wb = __builtin_bit_cast(float, wp & 0xffff0000u);
#pragma unroll
        for (int r = 0; r < TRB / 2; ++r) {
          const float2 b = *reinterpret_cast<const float2 *>(&sd2[r0 + r][2 * j2]);
          acc[r] += b.x * wa;
          acc[r] += b.y * wb;
        }
      }
#pragma unroll
      for (int r = 0; r < TRB / 2; ++r)
        sd1[r0 + r][i] = r0 + r < rows ? acc[r] * dsilu(z1[(size_t)(g0 + r0 + r) * TW + i]) : 0.f;
    }
    __syncthreads();
    // outer products of the block's rows (rows past n hold zeros)
#pragma unroll 1
    for (int r = 0; r < TRB; ++r) {
      float ha[8], db[8];
#pragma unroll
      for (int a = 0; a < 8; ++a) ha[a] = sh1[r][8 * ti + a];
#pragma unroll
      for (int b = 0; b < 8; ++b) db[b] = sd2[r][8 * tj + b];
#pragma unroll
      for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) a2[a][b] += ha[a] * db[b];
      const float hv = sh2[r][tid >> 1];
      const int j0 = 17 * (tid & 1);
#pragma unroll
      for (int j = 0; j < 17; ++j) a3[j] += hv * sgo[r][j0 + j];      // column 33 is the row's padding
      const float xv = sx[r][tid >> 6];
      a1[0] += xv * sd1[r][tid & 63];
      a1[1] += xv * sd1[r][64 + (tid & 63)];
      ab[0] += tid < TW ? sd1[r][tid] : sd2[r][tid - TW];
      if (tid < TO) ab[1] += sgo[r][tid];
    }
  }
  if (tid == 0) lpart[blockIdx.x] = lsum;
  if (!grads) return;
  // one partial gradient in the master's layout
  float *gp = gpar + (size_t)blockIdx.x * TGP;
  float *g1 = gp, *gb1 = g1 + 4 * TW, *g2 = gb1 + TW, *gb2 = g2 + TW * TW, *g3 = gb2 + TW, *gb3 = g3 + TW * TO;
  g1[(tid >> 6) * TW + (tid & 63)] = a1[0];
  g1[(tid >> 6) * TW + 64 + (tid & 63)] = a1[1];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) g2[(8 * ti + a) * TW + 8 * tj + b] = a2[a][b];
#pragma unroll
  for (int j = 0; j < 17; ++j)
    if (17 * (tid & 1) + j < TO) g3[(tid >> 1) * TO + 17 * (tid & 1) + j] = a3[j];
  if (tid < TW) gb1[tid] = ab[0];
  else gb2[tid - TW] = ab[0];
  if (tid < TO) gb3[tid] = ab[1];
}

// loss = (||T||^2 + sum of the rows' terms + ||G||_F^2) / ||T||^2 (one workgroup)
__device__ __forceinline__ void tail_loss_sum(const float *__restrict__ tpart, int ntpart,
                                              const float *__restrict__ lpart, int nlpart,
                                              const float2 *__restrict__ gm, float *__restrict__ loss, float *red4) {
  const float tn = block_sum(tpart, ntpart, red4);
  const float ls = block_sum(lpart, nlpart, red4);
  const float2 g = gm[threadIdx.x];
  float a = g.x * g.x + g.y * g.y;
  for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red4[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) loss[0] = (tn + (ls + ((red4[0] + red4[1]) + (red4[2] + red4[3])))) / tn;
}

__global__ __launch_bounds__(256) void tail_loss_kernel(const float *__restrict__ tpart, int ntpart,
                                                        const float *__restrict__ lpart, int nlpart,
                                                        const float2 *__restrict__ gm, float *__restrict__ loss) {
  __shared__ float red4[4];
  tail_loss_sum(tpart, ntpart, lpart, nlpart, gm, loss, red4);
}

// ---- Adam on the FP32 master copy, then the BF16 weights / FP32 biases of the next forward ------
// master layout: W1 [4][128], b1 [128], W2 [128][128], b2 [128], W3 [128][33], b3 [33]
__device__ __forceinline__ void tail_put_weight(int i, float p, __bf16 *__restrict__ wout, float *__restrict__ bout) {
  const int o1 = 4 * TW, o2 = o1 + TW, o3 = o2 + TW * TW, o4 = o3 + TW, o5 = o4 + TW * TO;
  if (i < o1) wout[i] = (__bf16)p;
  else if (i < o2) bout[i - o1] = p;
  else if (i < o3) wout[o1 + (i - o2)] = (__bf16)p;
  else if (i < o4) bout[TW + (i - o3)] = p;
  else if (i < o5) wout[o1 + TW * TW + (i - o4)] = (__bf16)p;
  else bout[2 * TW + (i - o5)] = p;
}

__global__ void tail_sync_kernel(const float *__restrict__ master, int np, __bf16 *__restrict__ wout,
                                 float *__restrict__ bout) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < np) tail_put_weight(i, master[i], wout, bout);
}

// Sums the npart partial gradients (32 parameters per workgroup, eight threads each: consecutive lanes read
// consecutive parameters, eight parts at a time), then the Adam step of each parameter.  The step count t
// comes from device memory (step_dev), so the same launch replays correctly from a graph; the bias
// corrections are 1 - beta^t.  The last workgroup forms the loss.  A single part may live in grad itself.
constexpr int TAP = 32;
__global__ __launch_bounds__(256) void tail_adam_kernel(float *__restrict__ master, float *__restrict__ m,
                                                        float *__restrict__ v, float *grad, const float *gpar,
                                                        int npart, int np, float lr,
                                                        float b1, float b2, float eps,
                                                        const int *__restrict__ step_dev, __bf16 *__restrict__ wout,
                                                        float *__restrict__ bout, const float *__restrict__ tpart,
                                                        int ntpart, const float *__restrict__ lpart, int nlpart,
                                                        const float2 *__restrict__ gm, float *__restrict__ loss) {
  __shared__ float red[256 / TAP][TAP];
  __shared__ float red4[4];
  if (blockIdx.x == gridDim.x - 1) {
    tail_loss_sum(tpart, ntpart, lpart, nlpart, gm, loss, red4);
    return;
  }
  const int c = threadIdx.x % TAP, part = threadIdx.x / TAP;
  const int i = blockIdx.x * TAP + c, ic = min(i, np - 1);
  float a = 0.f;
#pragma unroll 4
  for (int q = part; q < npart; q += 256 / TAP) a += gpar[(size_t)q * TGP + ic];
  red[part][c] = a;
  __syncthreads();
  if (part != 0 || i >= np) return;
  float gi = 0.f;
#pragma unroll
  for (int q = 0; q < 256 / TAP; ++q) gi += red[q][c];
  grad[i] = gi;
  const float t = (float)step_dev[0];
  const float c1 = 1.0f - powf(b1, t), c2 = 1.0f - powf(b2, t);
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float p = master[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  master[i] = p;
  tail_put_weight(i, p, wout, bout);
}

// ---- corrected P~ and the training-box check -------------------------------------------------------
// flag[0] = 1 if any raw feature leaves [lo - 5% w, hi + 5% w], w = hi - lo (per feature).
__global__ void tail_box_kernel(const float *__restrict__ feat, int n, const float *__restrict__ norm,
                                int *__restrict__ flag) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  for (int i = 0; i < 4; ++i) {
    const float lo = norm[8 + i], hi = norm[12 + i], m = 0.05f * (hi - lo);
    const float x = feat[4 * g + i];
    if (!(x >= lo - m && x <= hi + m)) flag[0] = 1;
  }
}

// p_corr = p_trunc - (diag(d) + U U^H)
__global__ void tail_apply_kernel(const float2 *__restrict__ p, const float *__restrict__ d,
                                  const float2 *__restrict__ u, int n, float2 *__restrict__ out) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)n * n) return;
  const int g = (int)(idx / n), gp = (int)(idx % n);
  float2 acc = make_float2(g == gp ? d[g] : 0.f, 0.f);
  for (int k = 0; k < TR; ++k) {
    const float2 a = u[g * TR + k], b = u[gp * TR + k];     // a conj(b)
    acc.x += a.x * b.x + a.y * b.y;
    acc.y += a.y * b.x - a.x * b.y;
  }
  const float2 x = p[idx];
  out[idx] = make_float2(x.x - acc.x, x.y - acc.y);
}

// Residual parts of one row g of dP~ - T with dP~ = -(diag(d) + U U^H): one workgroup per row; part[g][0..3] =
// off-diagonal |residual|^2, off-diagonal |T|^2, diagonal |residual|^2, diagonal |T|^2.
__global__ __launch_bounds__(256) void tail_parts_kernel(const float *__restrict__ d, const float2 *__restrict__ u,
                                                         const float2 *__restrict__ t, int n,
                                                         float *__restrict__ part) {
  const int g = blockIdx.x;
  __shared__ float2 ug[TR];
  __shared__ float red[4][256];
  if (threadIdx.x < TR) ug[threadIdx.x] = u[g * TR + threadIdx.x];
  __syncthreads();
  float a[4] = {0.f, 0.f, 0.f, 0.f};
  for (int gp = threadIdx.x; gp < n; gp += 256) {
    float2 c = make_float2(gp == g ? d[g] : 0.f, 0.f);
    for (int k = 0; k < TR; ++k) {
      const float2 x = ug[k], y = u[gp * TR + k];          // x conj(y)
      c.x += x.x * y.x + x.y * y.y;
      c.y += x.y * y.x - x.x * y.y;
    }
    const float2 tv = t[(size_t)g * n + gp];
    const float rx = -c.x - tv.x, ry = -c.y - tv.y;
    const int b = gp == g ? 2 : 0;
    a[b] += rx * rx + ry * ry;
    a[b + 1] += tv.x * tv.x + tv.y * tv.y;
  }
  for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = a[k];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[4 * g + threadIdx.x] = red[threadIdx.x][0];
}

// Column sums of part [n][4] into out[4] (one workgroup, double accumulation).
__global__ __launch_bounds__(256) void tail_parts_sum_kernel(const float *__restrict__ part, int n,
                                                             float *__restrict__ out) {
  __shared__ double red[4][256];
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int g = threadIdx.x; g < n; g += 256)
    for (int k = 0; k < 4; ++k) a[k] += part[4 * g + k];
  for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = a[k];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 4) out[threadIdx.x] = (float)red[threadIdx.x][0];
}

// Feature statistics over a training set, one system per launch (one workgroup), merged into acc
// (double [16]): pass 0 adds the sums (acc[0..4)) and folds min / max (acc[8..12), acc[12..16)); pass 1
// adds the squared deviations from mean = acc[0..4) / total (acc[4..8)).  The first launch of a pass
// initialises its entries.
__global__ __launch_bounds__(256) void tail_stats_kernel(const float *__restrict__ feat, int n, int pass, int first,
                                                         double total, double *__restrict__ acc) {
  __shared__ double red[12][256];
  double a[12];
  for (int k = 0; k < 4; ++k) {
    a[k] = 0.0;
    a[4 + k] = INFINITY;
    a[8 + k] = -INFINITY;
  }
  for (int g = threadIdx.x; g < n; g += 256)
    for (int k = 0; k < 4; ++k) {
      const double x = feat[4 * g + k];
      if (pass == 0) {
        a[k] += x;
        a[4 + k] = fmin(a[4 + k], x);
        a[8 + k] = fmax(a[8 + k], x);
      } else {
        const double dx = x - acc[k] / total;
        a[k] += dx * dx;
      }
    }
  for (int k = 0; k < 12; ++k) red[k][threadIdx.x] = a[k];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int k = 0; k < 4; ++k) {
        red[k][threadIdx.x] += red[k][threadIdx.x + st];
        red[4 + k][threadIdx.x] = fmin(red[4 + k][threadIdx.x], red[4 + k][threadIdx.x + st]);
        red[8 + k][threadIdx.x] = fmax(red[8 + k][threadIdx.x], red[8 + k][threadIdx.x + st]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 4) {
    const int k = threadIdx.x;
    if (pass == 0) {
      acc[k] = (first ? 0.0 : acc[k]) + red[k][0];
      acc[8 + k] = first ? red[4 + k][0] : fmin(acc[8 + k], red[4 + k][0]);
      acc[12 + k] = first ? red[8 + k][0] : fmax(acc[12 + k], red[8 + k][0]);
    } else {
      acc[4 + k] = (first ? 0.0 : acc[4 + k]) + red[k][0];
    }
  }
}

// norm = mean[4], std[4] (1 where std <= 1e-12 max(1, |mean|)), min[4], max[4] as floats.
__global__ void tail_stats_final_kernel(const double *__restrict__ acc, double total, float *__restrict__ norm) {
  const int k = threadIdx.x;
  if (k >= 4) return;
  const double mean = acc[k] / total;
  double sd = sqrt(acc[4 + k] / total);
  if (sd <= 1e-12 * fmax(1.0, fabs(mean))) sd = 1.0;
  norm[k] = (float)mean;
  norm[4 + k] = (float)sd;
  norm[8 + k] = (float)acc[8 + k];
  norm[12 + k] = (float)acc[12 + k];
}

// ---- launch sequences ------------------------------------------------------------------------------
#define T_LAUNCH(kernel, total, ...)                                                                      \
  do {                                                                                                    \
    hipLaunchKernelGGL(kernel, dim3((unsigned)(((size_t)(total) + 255) / 256)), dim3(256), 0, s, __VA_ARGS__); \
    hipError_t e_ = hipGetLastError();                                                                    \
    if (e_ != hipSuccess) return e_;                                                                      \
  } while (0)

static int row_blocks(int n) { return (n + TRB - 1) / TRB; }
static int tu_blocks(int n) { return (n + TUR - 1) / TUR; }

// Partial gradients of a training step: one workgroup per block of rows up to one per CU.  Where there is no
// room for so many, a step runs with as many as fit into the room of two arrays of back-propagated rows
// (2 TW n floats); none: a single workgroup, whose part lives in the caller's gradient.
constexpr int TAIL_WGS = 256;
int tail_parts_most(int n) { return std::min(row_blocks(n), TAIL_WGS); }
int tail_parts_least(int n) { return std::min(tail_parts_most(n), std::max(0, (int)((2LL * TW * n - 1024) / TGP))); }

size_t tail_part_floats() { return TGP; }

size_t tail_ws_floats(int n, bool train) {
  // xn 4n, z1 h1 z2 h2 4*128n, o 33n, d n, u w 2*(32n), residual parts 4n, ||T||^2 parts, G parts and G,
  // loss parts, partial gradients
  return (size_t)n * (4 + 4 * TW + TO + 1 + 4 * TR + 4) + tu_blocks(n) +
         2 * TR * TR * ((size_t)row_blocks(n) + (row_blocks(n) > 1 ? 1 : 0)) + tail_parts_most(n) +
         (train ? (size_t)tail_parts_least(n) * TGP : 0);
}

struct TailWs {
  float *xn, *z1, *h1, *z2, *h2, *o, *d, *tpart, *lpart, *part, *gpar;
  float2 *u, *w, *gm, *gpart;
};

static TailWs carve(float *base, int n) {
  TailWs t;
  float *p = base;
  t.z1 = p; p += (size_t)TW * n;
  t.h1 = p; p += (size_t)TW * n;
  t.z2 = p; p += (size_t)TW * n;
  t.h2 = p; p += (size_t)TW * n;
  t.u = (float2 *)p; p += 2 * (size_t)TR * n;
  t.w = (float2 *)p; p += 2 * (size_t)TR * n;
  t.gm = (float2 *)p; p += row_blocks(n) > 1 ? 2 * TR * TR : 0;   // a single part of G is G
  t.gpart = (float2 *)p; p += 2 * (size_t)TR * TR * row_blocks(n);
  t.xn = p; p += 4 * (size_t)n;
  t.part = p; p += 4 * (size_t)n;
  t.o = p; p += (size_t)TO * n;
  t.d = p; p += n;
  t.tpart = p; p += tu_blocks(n);
  t.lpart = p; p += tail_parts_most(n);
  t.gpar = p;
  return t;
}

hipError_t tail_features(const float2 *p, int ng, const int *miller, const double *q, double a_bohr, int nc,
                         double e_max, float *feat, hipStream_t s) {
  T_LAUNCH(tail_features_kernel, ng, p, ng, miller, q[0], q[1], q[2], a_bohr, nc, e_max, feat);
  return hipSuccess;
}

hipError_t tail_target(const float2 *full, const float2 *trunc, int ng, float2 *t, hipStream_t s) {
  dim3 grid((ng + 31) / 32, (ng + 31) / 32);
  hipLaunchKernelGGL(tail_target_kernel, grid, dim3(256), 0, s, full, trunc, ng, t);
  return hipGetLastError();
}

// MLP outputs into out; with `t` also the head (d, u) and with `train` what the backward pass needs
static hipError_t forward(const gw_mlp &w, const float *feat, int n, const TailWs *t, bool train, float *out,
                          int *step_dev, int set_step, hipStream_t s) {
  float *z = nullptr;
  hipLaunchKernelGGL(tail_forward_kernel, dim3(row_blocks(n)), dim3(256), 0, s, feat, n, (const __bf16 *)w.w, w.b,
                     w.norm, w.rank, train ? t->xn : z, train ? t->z1 : z, train ? t->h1 : z, train ? t->z2 : z,
                     train ? t->h2 : z, out, t ? t->d : z, t ? t->u : (float2 *)nullptr,
                     train ? t->gpart : (float2 *)nullptr, step_dev, set_step);
  return hipGetLastError();
}

hipError_t tail_forward(const gw_mlp &w, const float *feat, int n, float *out, hipStream_t s) {
  return forward(w, feat, n, nullptr, false, out, nullptr, 0, s);
}

// forward, W = T U and the row terms; with gpar also the wgs partial gradients
static hipError_t loss_pass(const gw_mlp &w, const float *feat, const float2 *target, int n, const TailWs &t, int wgs,
                            float *gpar, int *step_dev, int set_step, hipStream_t s) {
  hipError_t e = forward(w, feat, n, &t, true, t.o, step_dev, set_step, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tail_tu_kernel, dim3(tu_blocks(n) + 1), dim3(256), 0, s, target, t.u, n, t.w, t.tpart, t.gpart,
                     row_blocks(n), t.gm);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(tail_backward_kernel, dim3(wgs), dim3(256), 0, s, t.o, feat, t.d, t.u, t.w, t.gm, target, n,
                     w.rank, t.tpart, tu_blocks(n), (const __bf16 *)w.w, t.xn, t.z1, t.h1, t.z2, t.h2, t.lpart, gpar);
  return hipGetLastError();
}

hipError_t tail_loss(const gw_mlp &w, const float *feat, const float2 *target, int n, float *ws, float *loss_out,
                     hipStream_t s) {
  const TailWs t = carve(ws, n);
  const int wgs = tail_parts_most(n);
  hipError_t e = loss_pass(w, feat, target, n, t, wgs, nullptr, nullptr, 0, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tail_loss_kernel, dim3(1), dim3(256), 0, s, t.tpart, tu_blocks(n), t.lpart, wgs, t.gm, loss_out);
  return hipGetLastError();
}

// One training step, four launches; the partial gradients go to `parts` (tail_parts_most(n) of them) or, where
// that is NULL, to the fewer that the workspace holds.  The Adam step count lives in step_dev: with set_step >= 0 the forward
// kernel writes it (eager calls), with set_step < 0 it advances it by one (the form a captured graph replays).
hipError_t tail_train_step(const gw_mlp &w, const gw_adam &a, const float *feat, const float2 *target, int n,
                           float *ws, float *parts, float *loss_out, int *step_dev, int set_step, hipStream_t s) {
  const TailWs t = carve(ws, n);
  const int least = tail_parts_least(n), wgs = parts ? tail_parts_most(n) : std::max(1, least);
  float *gpar = parts ? parts : least > 0 ? t.gpar : a.grad;
  hipError_t e = loss_pass(w, feat, target, n, t, wgs, gpar, step_dev, set_step, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tail_adam_kernel, dim3((GW_TAIL_NPARAM + TAP - 1) / TAP + 1), dim3(256), 0, s, a.master, a.m, a.v,
                     a.grad, gpar, wgs, GW_TAIL_NPARAM, a.lr, a.beta1, a.beta2, a.eps, (const int *)step_dev,
                     (__bf16 *)w.w, w.b, t.tpart, tu_blocks(n), t.lpart, wgs, t.gm, loss_out);
  return hipGetLastError();
}

hipError_t tail_sync_weights(gw_mlp &w, const float *master, hipStream_t s) {
  T_LAUNCH(tail_sync_kernel, GW_TAIL_NPARAM, master, GW_TAIL_NPARAM, (__bf16 *)w.w, w.b);
  return hipSuccess;
}

hipError_t tail_check_box(const float *feat, int n, const float *norm, int *flag, hipStream_t s) {
  hipError_t e = launch_fill_int(flag, 0, s);
  if (e != hipSuccess) return e;
  T_LAUNCH(tail_box_kernel, n, feat, n, norm, flag);
  return hipSuccess;
}

hipError_t tail_apply(const gw_mlp &w, const float *feat, const float2 *p, int n, float *ws, float2 *out,
                      hipStream_t s) {
  const TailWs t = carve(ws, n);
  hipError_t e = forward(w, feat, n, &t, false, t.o, nullptr, 0, s);
  if (e != hipSuccess) return e;
  T_LAUNCH(tail_apply_kernel, (size_t)n * n, p, t.d, t.u, n, out);
  return hipSuccess;
}

hipError_t tail_residual_parts(const gw_mlp &w, const float *feat, const float2 *target, int n, float *ws,
                               float *parts, hipStream_t s) {
  const TailWs t = carve(ws, n);
  hipError_t e = forward(w, feat, n, &t, false, t.o, nullptr, 0, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tail_parts_kernel, dim3(n), dim3(256), 0, s, t.d, t.u, target, n, t.part);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(tail_parts_sum_kernel, dim3(1), dim3(256), 0, s, t.part, n, parts);
  return hipGetLastError();
}

hipError_t tail_fit_norm(int nsys, const float *const *feats, const int *ngs, double *acc, float *norm,
                         hipStream_t s) {
  double total = 0.0;
  for (int i = 0; i < nsys; ++i) total += ngs[i];
  for (int pass = 0; pass < 2; ++pass)
    for (int i = 0; i < nsys; ++i) {
      hipLaunchKernelGGL(tail_stats_kernel, dim3(1), dim3(256), 0, s, feats[i], ngs[i], pass, i == 0 ? 1 : 0, total,
                         acc);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  hipLaunchKernelGGL(tail_stats_final_kernel, dim3(1), dim3(64), 0, s, (const double *)acc, total, norm);
  return hipGetLastError();
}

}  // namespace gwi
