// C ABI of the plasmon-pole model (the paper's section on the dynamic inverse dielectric matrix):
// the few most negative eigenpairs of S = sqrt(V)(eps^-1 - I)sqrt(V) by block subspace iteration
// with a Rayleigh-Ritz step per iteration, their frequencies from the Johnson sum rule, and the
// pole-form eps^-1(w).  Kernels in pp.hip; the pole form's product on the FP64 MFMA GEMM.
//
// Iteration (all on the device, one host read of the residual per iteration):
//   Y = -S X;  H = X^H Y;  H = Z diag(theta) Z^H (Jacobi, descending);  W = X Z, T = Y Z
//   stop when max_{a < n_modes} ||T_a - theta_a W_a|| <= tol * theta_0
//   X <- T u, u from the Cholesky factor of T^H T: an orthonormal basis of T
// The next X is formed while the host waits for the residual.
#include <algorithm>
#include <cmath>
#include <cstdio>

#include "gw_internal.h"

using namespace gwi;

namespace {

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

constexpr int kBlock = 32;      // subspace size (the Jacobi kernel's limit)
constexpr int kMaxModes = 24;   // at least 8 guard vectors beyond the wanted modes

enum {
  PP_MILLER = 40, PP_SQRTV, PP_RHO, PP_RHO_T, PP_S, PP_M, PP_X, PP_Y, PP_W, PP_T, PP_SMALL, PP_B
};

struct Small {            // b x b matrices, eigenvalues and partial sums of the iteration
  double2 *z, *u, *gpart;
  double *theta, *res, *rpart;
};

int upload_sphere(gw_ctx *ctx, const int *miller, int ng, const double *q, double a_bohr, int **dm, double **dsv,
                  hipStream_t s) {
  void *sv;
  GWX_STATUS(upload_miller(ctx, miller, ng, PP_MILLER, dm, s));
  GWX_STATUS(api_ws_get(ctx, PP_SQRTV, (size_t)ng * sizeof(double), &sv, s));
  GWX_HIP(ctx, launch_sqrtv(*dm, ng, q[0], q[1], q[2], a_bohr, (double *)sv, s));
  *dsv = (double *)sv;
  return GW_OK;
}

// x = orthonormal basis of the columns of w
int orthonormalize(gw_ctx *ctx, double2 *w, int ng, int b, const Small &sm, double2 *x, hipStream_t s) {
  GWX_HIP(ctx, launch_block_gram(w, w, ng, b, sm.gpart, s));
  GWX_HIP(ctx, launch_block_chol(sm.gpart, ng, b, sm.u, s));
  GWX_HIP(ctx, launch_block_rotate(w, sm.u, ng, b, x, s));
  return GW_OK;
}

}  // namespace

extern "C" {

int gw_plasmon_pole(gw_ctx *ctx, const gw_c64 *eps_inv, int ng, gw_grid grid, const double *q, const int *g_miller,
                    const gw_c32 *psi_v, int nv, double occupation, int n_modes, double tol, int max_iter,
                    double *sigma, double *omega, gw_c64 *modes, int *iterations, double *residual, void *stream) {
  GWX_STATUS(api_begin(ctx));
  GWX_CHECK(ctx, eps_inv && psi_v && sigma && omega && modes && iterations && q,
            "eps_inv, psi_v, sigma, omega, modes, iterations and q must not be NULL");
  GWX_STATUS(api_check_grid(ctx, grid));
  const long long nrl = (long long)grid.n1 * grid.n2 * grid.n3;
  GWX_CHECK(ctx, nrl <= (1 << 24), "grid too large");
  GWX_STATUS(api_check_sphere(ctx, grid, g_miller, ng));
  GWX_CHECK(ctx, std::isfinite(q[0]) && std::isfinite(q[1]) && std::isfinite(q[2]), "q must be finite");
  GWX_CHECK(ctx, nv > 0, "nv must be positive");
  GWX_CHECK(ctx, std::isfinite(occupation) && occupation > 0.0, "occupation must be positive");
  GWX_CHECK(ctx, n_modes >= 1 && n_modes <= std::min(kMaxModes, ng), "n_modes must be in [1, min(24, ng)]");
  GWX_CHECK(ctx, std::isfinite(tol) && tol > 0.0, "tol must be positive");
  GWX_CHECK(ctx, max_iter >= 1 && max_iter <= 100000, "max_iter must be in [1, 100000]");
  if (ctx->device < 0) {
    *iterations = 0;
    return GW_OK;
  }
  hipStream_t s = as_stream(stream);
  const int nr = (int)nrl, b = std::min(kBlock, ng);
  int *dm;
  double *sv;
  GWX_STATUS(upload_sphere(ctx, g_miller, ng, q, grid.a_bohr, &dm, &sv, s));
  // density and its transform on the full grid, then S and the sum-rule matrix M
  void *rho, *rho_t, *sp, *mp;
  GWX_STATUS(api_ws_get(ctx, PP_RHO, (size_t)nr * sizeof(double2), &rho, s));
  GWX_STATUS(api_ws_get(ctx, PP_RHO_T, (size_t)nr * sizeof(double2), &rho_t, s));
  GWX_STATUS(api_ws_get(ctx, PP_S, (size_t)ng * ng * sizeof(double2), &sp, s));
  // M's buffer, filled after the iteration, holds the iteration's partial sums until then; the last product's
  // are left in S's
  const size_t tp_el = thin_part_elems(ng, b, ng), gp_el = gram_part_elems(ng, b);
  GWX_STATUS(api_ws_get(ctx, PP_M, std::max((size_t)ng * ng * sizeof(double2), (tp_el + gp_el) * sizeof(double2) +
                                                                      rotate_part_doubles(ng, b) * sizeof(double)),
                        &mp, s));
  GWX_HIP(ctx, launch_density((const float2 *)psi_v, nv, nr, occupation, (double2 *)rho, s));
  GWX_HIP(ctx, launch_density_transform((double2 *)rho, (double2 *)rho_t, grid.n1, grid.n2, grid.n3, s));
  double2 *S = (double2 *)sp, *M = (double2 *)mp;
  GWX_HIP(ctx, launch_screening((const double2 *)eps_inv, sv, ng, ng, S, s));
  // block buffers
  void *xp, *yp, *wp, *tp, *smp;
  const size_t blk = (size_t)ng * b * sizeof(double2);
  GWX_STATUS(api_ws_get(ctx, PP_X, blk, &xp, s));
  GWX_STATUS(api_ws_get(ctx, PP_Y, blk, &yp, s));
  GWX_STATUS(api_ws_get(ctx, PP_W, blk, &wp, s));
  GWX_STATUS(api_ws_get(ctx, PP_T, blk, &tp, s));
  const size_t bb = (size_t)b * b;
  GWX_STATUS(api_ws_get(ctx, PP_SMALL, 2 * bb * sizeof(double2) + (b + 8) * sizeof(double), &smp, s));
  Small sm;
  sm.z = (double2 *)smp;
  sm.u = sm.z + bb;
  sm.theta = (double *)(sm.u + bb);
  sm.res = sm.theta + b;
  double2 *part = M;
  sm.gpart = part + tp_el;
  sm.rpart = (double *)(sm.gpart + gp_el);
  double2 *X = (double2 *)xp, *Y = (double2 *)yp, *W = (double2 *)wp, *T = (double2 *)tp;
  GWX_HIP(ctx, launch_start_block(T, ng, b, 0x5eedULL, s));
  GWX_STATUS(orthonormalize(ctx, T, ng, b, sm, X, s));
  double res = INFINITY;
  int it = 0;
  for (it = 1; it <= max_iter; ++it) {
    GWX_HIP(ctx, launch_thin_product(ng, b, ng, S, ng, X, b, part, s));
    GWX_HIP(ctx, launch_thin_sum(part, ng, b, ng, -1.0, Y, s));                      // Y = -S X
    GWX_HIP(ctx, launch_block_gram(X, Y, ng, b, sm.gpart, s));                       // X^H Y
    GWX_HIP(ctx, launch_herm_jacobi(sm.gpart, ng, b, sm.theta, sm.z, s));
    GWX_HIP(ctx, launch_block_ritz(X, Y, sm.z, ng, b, sm.theta, n_modes, W, T, sm.rpart, sm.res, s));
    GWX_HIP(ctx, hipMemcpyAsync(ctx->result_host, sm.res, sizeof(double), hipMemcpyDeviceToHost, s));
    GWX_HIP(ctx, hipEventRecord(ctx->result_event, s));
    if (it < max_iter && b < ng) GWX_STATUS(orthonormalize(ctx, T, ng, b, sm, X, s));
    GWX_HIP(ctx, hipEventSynchronize(ctx->result_event));
    res = *ctx->result_host;
    if (!std::isfinite(res)) break;
    if (res <= tol || b == ng) break;      // converged (a full-space block is exact after one step)
  }
  *iterations = std::min(it, max_iter);
  if (residual) *residual = res;
  // frequencies from the sum rule: t = M A, omega_a^2 = Re(a^H t_a) / theta_a
  GWX_HIP(ctx, launch_sum_rule(dm, ng, q, grid.a_bohr, sv, (const double2 *)rho_t, grid.n1, grid.n2, grid.n3, M, s));
  GWX_HIP(ctx, launch_thin_product(ng, n_modes, ng, M, ng, W, b, S, s));
  GWX_HIP(ctx, launch_thin_sum(S, ng, n_modes, ng, 1.0, Y, s));
  GWX_HIP(ctx, launch_pp_frequency(W, b, Y, n_modes, ng, sm.theta, n_modes, sigma, omega, s));
  GWX_HIP(ctx, hipMemcpy2DAsync(modes, (size_t)n_modes * sizeof(double2), W, (size_t)b * sizeof(double2),
                                (size_t)n_modes * sizeof(double2), ng, hipMemcpyDeviceToDevice, s));
  GWX_HIP(ctx, hipStreamSynchronize(s));
  if (!std::isfinite(res)) {
    api_set_err(ctx, "plasmon-pole iteration produced a non-finite residual");
    return GW_E_HIP;
  }
  if (res > tol) {
    char m[200];
    snprintf(m, sizeof(m), "plasmon-pole iteration did not reach tol %.3g in %d iterations (residual %.3g)", tol,
             max_iter, res);
    api_set_err(ctx, m);
    return GW_E_UNSUPPORTED;
  }
  return GW_OK;
}

int gw_pp_eps_inverse(gw_ctx *ctx, const gw_c64 *eps_inv_static, int ng, gw_grid grid, const double *q,
                      const int *g_miller, const gw_c64 *modes, const double *sigma, const double *omega, int n_modes,
                      const double *freqs, int nf, gw_c64 *out, void *stream) {
  GWX_STATUS(api_begin(ctx));
  GWX_CHECK(ctx, eps_inv_static && modes && sigma && omega && freqs && out && q,
            "eps_inv_static, modes, sigma, omega, freqs, out and q must not be NULL");
  GWX_STATUS(api_check_grid(ctx, grid));
  GWX_STATUS(api_check_sphere(ctx, grid, g_miller, ng));
  GWX_CHECK(ctx, n_modes >= 1 && n_modes <= ng, "n_modes must be in [1, ng]");
  GWX_CHECK(ctx, nf >= 1, "nf must be positive");
  for (int f = 0; f < nf; ++f) GWX_CHECK(ctx, std::isfinite(freqs[f]), "frequencies must be finite");
  if (ctx->device < 0) return GW_OK;
  hipStream_t s = as_stream(stream);
  int *dm;
  double *sv;
  GWX_STATUS(upload_sphere(ctx, g_miller, ng, q, grid.a_bohr, &dm, &sv, s));
  if (pp_pole_fits(n_modes)) {
    for (int f = 0; f < nf; ++f)
      GWX_HIP(ctx, launch_pp_pole((const double2 *)modes, ng, n_modes, sigma, omega, freqs[f], sv,
                                  (const double2 *)eps_inv_static, (double2 *)out + (size_t)f * ng * ng, s));
    return GW_OK;
  }
  void *bp;
  GWX_STATUS(api_ws_get(ctx, PP_B, (size_t)ng * n_modes * sizeof(double2), &bp, s));
  for (int f = 0; f < nf; ++f) {
    double2 *e = (double2 *)out + (size_t)f * ng * ng;
    GWX_HIP(ctx, launch_pp_weight((const double2 *)modes, ng, n_modes, sigma, omega, freqs[f], (double2 *)bp, s));
    GWX_HIP(ctx, launch_zgemm(ng, ng, n_modes, (const double2 *)bp, n_modes, Z_N, (const double2 *)modes, n_modes, Z_H, e,
                              ng, 1.0, 0.0, s));
    GWX_HIP(ctx, launch_pp_finish(e, (const double2 *)eps_inv_static, sv, ng, s));
  }
  return GW_OK;
}

}  // extern "C"
