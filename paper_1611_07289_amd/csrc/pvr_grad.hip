// Derivative of the forward model with respect to the per-patch motion:
//   grad_theta_s = sum_{j in s} g_j d y_hat_j / d theta_s.
//
// y_hat_j = sum_i g_hat_ji X_i / Z_j with Z_j = sum_i g_hat_ji, so
//   d y_hat_j / d theta = sum_i (X_i - y_hat_j) d g_hat_ji / d theta / Z_j,
// with d g_hat / d theta as derived in pvr_grad.h.
//
// One workgroup per patch; FP64 accumulation of the six per-patch sums.  One
// walk per sample gathers the nine offset moments of pvr_grad.h and forms the
// six derivatives once per sample: in FP32 the exact registration's walk, in
// FP64 the plane walk's (k_grad_theta_planes), or for patches off it two walks
// (y_hat, then the derivative evaluated at every voxel).  The FP32 derivative
// keeps the per-sample walk: its error is the voxels that rounding puts on the
// other side of the support's edge, where the derivative jumps, so another
// rounding would move a few per patch.
#include <math.h>

#include "pvr_geometry.h"
#include "pvr_grad.h"
#include "pvr_internal.h"
#include "pvr_planes.h"
#include "pvr_util.h"

using namespace pvr;

constexpr int GR_THREADS = 256;

// The patch's derivative constants, built by the first wavefront (all threads
// call; ends with a barrier).
__device__ __forceinline__ void shared_grad_const(const ProbDev &pr, const StackDev &st,
                                                  const PatchDev &pt, const double *th,
                                                  GradConst &gc) {
  if (threadIdx.x < 64) {
    const Trig trig = wave_trig(th);
    if (threadIdx.x == 0) make_grad_const(pr, st, pt, th, trig, gc);
  }
  __syncthreads();
}

// sum6 over the workgroup in a fixed order into grad[0..6); whether all are finite
// (the same in every thread)
template <typename T>
__device__ __forceinline__ bool grad_out(const double sum6[6], T *__restrict__ grad) {
  __shared__ double red[6][GR_THREADS / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double x = sum6[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[k][wave] = x;
  }
  __syncthreads();
  double x = 0;
  if (lane < 6) {
    for (int w = 0; w < GR_THREADS / 64; ++w) x += red[lane][w];
    if (wave == 0) grad[lane] = (T)x;
  }
  return __all(__builtin_isfinite(x));
}

// q = x_world - (c + t) of pixel (u, v), x_world = Vl x_vox + o
template <typename T>
__device__ __forceinline__ void grad_q(const GradConst &gc, const double *H, int u, int v, int slice,
                                       T qt[3]) {
  double xv[3];
#pragma unroll
  for (int r = 0; r < 3; ++r)
    xv[r] = fma(H[4 * r], (double)u, fma(H[4 * r + 1], (double)v,
                                         fma(H[4 * r + 2], (double)slice, H[4 * r + 3])));
#pragma unroll
  for (int r = 0; r < 3; ++r)
    qt[r] = (T)(gc.Vl[3 * r] * xv[0] + gc.Vl[3 * r + 1] * xv[1] + gc.Vl[3 * r + 2] * xv[2] +
                gc.v2w_o[r] - gc.ct[r]);
}

template <typename T>
__global__ void __launch_bounds__(GR_THREADS)
k_grad_theta(const ProbDev *__restrict__ probs, const StackDev *__restrict__ stacks,
             const PatchDev *__restrict__ patches, const typename GeoOf<T>::type *__restrict__ geo,
             const double *__restrict__ theta, const T *__restrict__ invz,
             const T *__restrict__ X, const T *__restrict__ gy, T *__restrict__ grad) {
  const int s = blockIdx.x;
  const PatchDev pt = patches[s];
  const ProbDev pr = probs[pt.problem];
  const StackDev st = stacks[pt.stack];
  const typename GeoOf<T>::type &g = geo[s];
  GradConst gc;
  make_grad_const(pr, st, pt, theta + 6 * s, make_trig(theta + 6 * s), gc);
  const T *Xp = X + pr.vol_off;
  GradMom gm;
  if constexpr (sizeof(T) == 4) make_grad_mom(gc, g.perm, gm);
  const unsigned nbytes = (unsigned)(pr.nx * pr.ny * pr.nz) * (unsigned)sizeof(T);
  const __amdgpu_buffer_rsrc_t xr = raw_buffer(Xp, nbytes);
  double sum6[6] = {0, 0, 0, 0, 0, 0};
  const int n = pt.w * pt.h;
  for (int l = threadIdx.x; l < n; l += GR_THREADS) {
    const long long j = pt.off + l;
    const T iz = invz[j];
    if (!(iz > (T)0)) continue;
    const T gj = gy[j];
    if (gj == (T)0) continue;
    const int u = pt.x0 + l % pt.w, v = pt.y0 + l / pt.w;
    int b[3];
    T f[3];
    sample_centre(g, pr, u, v, pt.slice, b, f);
    T qt[3];
    grad_q(gc, g.H, u, v, pt.slice, qt);
    T a6[6] = {0, 0, 0, 0, 0, 0};
    if constexpr (sizeof(T) == 4) {
      // moments of w_i = e^{-Q_i/2} (X_i - y_hat) from those relative to the
      // centre voxel's value X_b: y_hat - X_b = sum g_hat (X - X_b) / Z
      float xb, a, z, mx[9], me[9];
      if (g.perm[2] == 0)
        psf_walk_grad<1, false>(g, pr, b, f, xr, nbytes, xb, a, z, mx, me);
      else
        psf_walk_grad<2, false>(g, pr, b, f, xr, nbytes, xb, a, z, mx, me);
      const float dl = a * iz;
      float m[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) m[c] = fma(-dl, me[c], mx[c]);
      grad_from_moments(gm, m, qt, a6);
    } else {
      T z = 0, acc = 0;
      psf_walk<T, typename GeoOf<T>::type, true>(g, pr, b, f, Xp, z, acc);
      const T yh = acc * iz;
      grad_walk<T>(g, pr, gc, b, f, qt, Xp, yh, a6);
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) sum6[k] += (double)gj * (double)(a6[k] * iz);
  }
  grad_out(sum6, grad + 6 * s);
}

// FP64 by the plane walk, a lane's 2 x 2 samples two at a time; patches off it are
// walked sample by sample, as by k_grad_theta.  187 000 samples at 48^3: 117 -> 88 us
// (two walks before, the derivative at every voxel, an FP64 exponential for each
// voxel and walk; here eight for eighteen).  Two wavefronts a SIMD: all four samples
// at once take six exponentials less but 420 registers, so that one wavefront ran,
// no faster on the walk (88 us) and slow off it (all patches turned by 60 degrees:
// 336 us, 133 here and before).
__global__ void __launch_bounds__(GR_THREADS, 2)
k_grad_theta_planes(const ProbDev *__restrict__ probs, const StackDev *__restrict__ stacks,
                    const PatchDev *__restrict__ patches, const GeoD *__restrict__ geo,
                    const FwdPatch<double> *__restrict__ fwd, const double *__restrict__ theta,
                    const double *__restrict__ invz, const double *__restrict__ X,
                    const double *__restrict__ gy, double *__restrict__ grad) {
  __shared__ GradConst gc;
  __shared__ GradMomT<double> gm;
  __shared__ FwdPatch<double> fw;
  const int s = blockIdx.x;
  const PatchDev pt = patches[s];
  const ProbDev pr = probs[pt.problem];
  const GeoD &g = geo[s];
  static_assert(sizeof fw % 4 == 0, "copied by words");
  for (int i = threadIdx.x; i < (int)sizeof fw / 4; i += GR_THREADS)
    reinterpret_cast<int *>(&fw)[i] = reinterpret_cast<const int *>(fwd + s)[i];
  shared_grad_const(pr, stacks[pt.stack], pt, theta + 6 * s, gc);
  if (threadIdx.x == 0) make_grad_mom(gc, fw.rows ? fw.ax : g.perm, gm);
  __syncthreads();
  const double *Xp = X + pr.vol_off;
  const unsigned nbytes = (unsigned)(pr.nx * pr.ny * pr.nz) * (unsigned)sizeof(double);
  const __amdgpu_buffer_rsrc_t xr = raw_buffer(Xp, nbytes);
  double sum6[6] = {0, 0, 0, 0, 0, 0};
  auto add = [&](double gj, double iz, const double a6[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) sum6[k] += gj * (a6[k] * iz);
  };
  if (fw.rows) {
    const int nbu = (pt.w + 1) / 2, nblk = nbu * ((pt.h + 1) / 2);
    for (int blk = threadIdx.x; blk < nblk; blk += GR_THREADS) {
      const int u0 = 2 * (blk % nbu), v0 = 2 * (blk / nbu);
      double iz[4], gj[4];  // pixel (u0 + i, v0 + j) at 2 j + i; off: 0
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int u = u0 + (t & 1), v = v0 + (t >> 1);
        const long long j = pt.off + (long long)v * pt.w + u;
        const bool in = u < pt.w && v < pt.h;
        gj[t] = in ? gy[j] : 0.0;
        iz[t] = in && gj[t] != 0.0 ? invz[j] : 0.0;
      }
      const bool live = iz[0] > 0 || iz[1] > 0 || iz[2] > 0 || iz[3] > 0;
      if (!live) continue;
#pragma unroll 1
      for (int j = 0; j < 2; ++j) {
        double xb, a[2], z[2], mx[2][9], me[2][9];
        if (fw.rows == 3) plane_walk_grad<double, 3>(fw, u0, v0, j, xr, nbytes, xb, a, z, mx, me);
        else plane_walk_grad<double, 4>(fw, u0, v0, j, xr, nbytes, xb, a, z, mx, me);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int p = (2 * j + t) ^ fw.flip;  // the sub-window's pixel
          const double izp = p == 0 ? iz[0] : p == 1 ? iz[1] : p == 2 ? iz[2] : iz[3];
          const double gp = p == 0 ? gj[0] : p == 1 ? gj[1] : p == 2 ? gj[2] : gj[3];
          if (!(izp > 0)) continue;
          const double dl = a[t] * izp;
          double m[9], qt[3], a6[6];
#pragma unroll
          for (int c = 0; c < 9; ++c) m[c] = fma(-dl, me[t][c], mx[t][c]);
          grad_q(gc, g.H, pt.x0 + u0 + (p & 1), pt.y0 + v0 + (p >> 1), pt.slice, qt);
          grad_from_moments(gm, m, qt, a6);
          add(gp, izp, a6);
        }
      }
    }
    // a voxel of the walk's windows outside every support may have made a sum not finite
    if (grad_out(sum6, grad + 6 * s)) return;
#pragma unroll
    for (int k = 0; k < 6; ++k) sum6[k] = 0.0;
    __syncthreads();
  }
  // sample by sample, as k_grad_theta
  const int n = pt.w * pt.h;
  for (int l = threadIdx.x; l < n; l += GR_THREADS) {
    const long long j = pt.off + l;
    const double gj = gy[j], iz = invz[j];
    if (!(iz > 0) || gj == 0.0) continue;
    const int u = pt.x0 + l % pt.w, v = pt.y0 + l / pt.w;
    int b[3];
    double f[3], qt[3], a6[6] = {0, 0, 0, 0, 0, 0}, z = 0, acc = 0;
    sample_centre(g, pr, u, v, pt.slice, b, f);
    grad_q(gc, g.H, u, v, pt.slice, qt);
    psf_walk<double, GeoD, true>(g, pr, b, f, Xp, z, acc);
    grad_walk<double>(g, pr, gc, b, f, qt, Xp, acc * iz, a6);
    add(gj, iz, a6);
  }
  grad_out(sum6, grad + 6 * s);
}

template <typename T>
static pvr_status grad_impl(const pvr_plan *p, const T *X, const T *gy, T *grad, const T *invz,
                            hipStream_t stream) {
  if (!X || !gy || !grad) return fail(PVR_EINVAL, "pvr_simulate_grad_theta: NULL argument");
  if (p->psf != PVR_PSF_GAUSSIAN)
    return fail(PVR_EUNSUPPORTED, "pvr_simulate_grad_theta: the theta-derivative is implemented for the Gaussian PSF");
  const auto *geo = (const typename GeoOf<T>::type *)(sizeof(T) == 4 ? (const void *)p->d_geof
                                                                     : (const void *)p->d_geod);
  if constexpr (sizeof(T) == 8) {
    if (p->planes64) {
      hipLaunchKernelGGL(k_grad_theta_planes, dim3(p->M), dim3(GR_THREADS), 0, stream, p->d_prob,
                         p->d_stack, p->d_patch, p->d_geod, p->d_fwd64, p->d_theta, invz, X, gy, grad);
      HIP_TRY(hipGetLastError());
      return PVR_OK;
    }
  }
  hipLaunchKernelGGL(k_grad_theta<T>, dim3(p->M), dim3(GR_THREADS), 0, stream, p->d_prob, p->d_stack,
                     p->d_patch, geo, p->d_theta, invz, X, gy, grad);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
}

extern "C" pvr_status pvr_simulate_grad_theta(const pvr_plan *p, const float *X, const float *gy,
                                              float *grad_theta, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_simulate_grad_theta", X, 4);
  PVR_ALIGNED("pvr_simulate_grad_theta", gy, 4);
  PVR_ALIGNED("pvr_simulate_grad_theta", grad_theta, 4);
  if (!p) return fail(PVR_EINVAL, "pvr_simulate_grad_theta: plan is NULL");
  if (!p->built) return fail(PVR_EINVAL, "pvr_simulate_grad_theta: plan has not been built");
  PVR_TRY_STATUS(debug_finite(p, "pvr_simulate_grad_theta", "X", X, p->V, stream));
  PVR_TRY_STATUS(debug_finite(p, "pvr_simulate_grad_theta", "grad_y", gy, p->N, stream));
  return grad_impl<float>(p, X, gy, grad_theta, p->d_invz, stream);
  PVR_API_END();
}

extern "C" pvr_status pvr_simulate_grad_theta_f64(const pvr_plan *p, const double *X,
                                                  const double *gy, double *grad_theta,
                                                  hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_simulate_grad_theta_f64", X, 8);
  PVR_ALIGNED("pvr_simulate_grad_theta_f64", gy, 8);
  PVR_ALIGNED("pvr_simulate_grad_theta_f64", grad_theta, 8);
  if (!p) return fail(PVR_EINVAL, "pvr_simulate_grad_theta_f64: plan is NULL");
  if (!p->built || !p->built64)
    return fail(PVR_EINVAL, "pvr_simulate_grad_theta_f64: plan needs pvr_plan_build_f64 on a "
                            "workspace attached with PVR_WS_F64");
  PVR_TRY_STATUS(debug_finite(p, "pvr_simulate_grad_theta_f64", "X", X, p->V, stream));
  PVR_TRY_STATUS(debug_finite(p, "pvr_simulate_grad_theta_f64", "grad_y", gy, p->N, stream));
  return grad_impl<double>(p, X, gy, grad_theta, p->d_invz64, stream);
  PVR_API_END();
}

// ---------------------------------------------------------------------------
// Cross-correlation of every patch with its simulation and its derivative
// with respect to the simulated samples (Sec. IV-A eq. CC over the samples
// valid at the last build, population statistics):
//   NCC_s = cov(y, yh) / (sd_y sd_yh),
//   d NCC_s / d yh_j = ((y_j - mu_y) / (sd_y sd_yh)
//                       - NCC_s (yh_j - mu_yh) / sd_yh^2) / n_s.
// Flat patches (a variance at or below 1e-12 of the squared mean) get NCC 0
// and a zero derivative.  One workgroup per patch.
__global__ void __launch_bounds__(GR_THREADS)
k_ncc_grad(const PatchDev *__restrict__ patches, const float *__restrict__ invz,
           const float *__restrict__ y, const float *__restrict__ yh,
           float *__restrict__ gout, float *__restrict__ ncc) {
  __shared__ double red[6][GR_THREADS / 64];
  const int s = blockIdx.x;
  const PatchDev pt = patches[s];
  const int n = pt.w * pt.h;
  double a6[6] = {0, 0, 0, 0, 0, 0};
  for (int l = threadIdx.x; l < n; l += GR_THREADS) {
    const long long j = pt.off + l;
    if (!(invz[j] > 0.f)) continue;
    const double yo = y[j], ys = yh[j];
    a6[0] += 1.0; a6[1] += yo; a6[2] += yo * yo; a6[3] += ys; a6[4] += ys * ys; a6[5] += yo * ys;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double x = a6[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[k][wave] = x;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    double x = 0;
    for (int w = 0; w < GR_THREADS / 64; ++w) x += red[k][w];
    a6[k] = x;
  }
  const double cnt = a6[0];
  double my = 0, mh = 0, vy = 0, vh = 0, cv = 0, r = 0;
  bool ok = cnt > 0;
  if (ok) {
    my = a6[1] / cnt; mh = a6[3] / cnt;
    vy = a6[2] / cnt - my * my; vh = a6[4] / cnt - mh * mh; cv = a6[5] / cnt - my * mh;
    ok = vy > 1e-12 * my * my && vh > 1e-12 * mh * mh && vy > 0 && vh > 0;
  }
  double sy = 0, sh = 0;
  if (ok) {
    sy = sqrt(vy); sh = sqrt(vh);
    r = cv / (sy * sh);
  }
  if (ncc && threadIdx.x == 0) ncc[s] = (float)r;
  if (!gout) return;
  for (int l = threadIdx.x; l < n; l += GR_THREADS) {
    const long long j = pt.off + l;
    float gj = 0.f;
    if (ok && invz[j] > 0.f) {
      const double yo = y[j], ys = yh[j];
      gj = (float)(((yo - my) / (sy * sh) - r * (ys - mh) / vh) / cnt);
    }
    gout[j] = gj;
  }
}

extern "C" pvr_status pvr_ncc_grad(const pvr_plan *p, const float *y_obs, const float *y_sim,
                                   float *grad_y, float *ncc, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_ncc_grad", y_obs, 4);
  PVR_ALIGNED("pvr_ncc_grad", y_sim, 4);
  PVR_ALIGNED("pvr_ncc_grad", grad_y, 4);
  PVR_ALIGNED("pvr_ncc_grad", ncc, 4);
  if (!p || !y_obs || !y_sim) return fail(PVR_EINVAL, "pvr_ncc_grad: NULL argument");
  if (!p->built) return fail(PVR_EINVAL, "pvr_ncc_grad: plan has not been built");
  hipLaunchKernelGGL(k_ncc_grad, dim3(p->M), dim3(GR_THREADS), 0, stream, p->d_patch, p->d_invz,
                     y_obs, y_sim, grad_y, ncc);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}
