// Registration of all patches in step.
//
// Every patch runs its own optimiser (see pvr_register_patches), but the
// patches move together through its stages: one launch evaluates a stage for
// every patch that needs it, one chunk of 1024 samples per workgroup, then a
// wavefront per patch combines its partial sums, takes the decision and builds
// the next stage's geometry.  Against one workgroup per patch running its whole
// optimiser (k_register), which bound the launch by its slowest patches and by
// the geometry chain that 255 threads waited for in every evaluation, each
// launch fills the chip whatever the patches' number and size, and the
// evaluation kernels hold no optimiser state in registers (the gradient's walk:
// 128 registers instead of 254).  The samples are the same bit for bit.  Passes
// of up to forty steps from zero motion, one workgroup per patch -> in step (ms):
// 256^3, 11 760 patches of 64 x 64: exact gradient 115 -> 67.6, central differences
// 329 -> 226; 128^3, 1 152 patches: 15.3 -> 10.9 and 59.1 -> 29.1; 64^3, 432 patches
// of 32 x 32: central differences 11.0 -> 5.8.  Bound by the walks' vector issue
// (256^3), by the launches' latency (64^3).
//
// Stages: POINT (NCC at the start), then per trial step GRAD (exact gradient) or
// FD (central differences, `nv` of the twelve points per launch), and TRIAL.  A
// patch takes part in a stage while its optimiser still runs and the stage
// applies to it (a rejected trial keeps its gradient).
#include <math.h>

#include <algorithm>

#include "pvr_geometry.h"
#include "pvr_grad.h"
#include "pvr_internal.h"
#include "pvr_util.h"

using namespace pvr;

namespace {

enum Stage { ST_BEGIN, ST_POINT, ST_GRAD, ST_FD, ST_TRIAL, ST_END };

struct RegState {
  double q[6], sc[6];   // current point in scaled variables, and the scales
  double grad[6], fd[12];
  double f0, delta;
  double walked[2];     // samples walked, plain and exact-gradient evaluations
  int evals[2];
  int run, have_grad, moved, pad_;
};

// One evaluated transform; on: the patch takes part in the stage.
struct EvalGeo {
  GeoF g;
  int on, pad_;
};
struct GradGeo {
  double Q[9];  // (u, v, 1) -> x_j - (c + t) in world mm
  GradMom gm;
};

constexpr int RG_THREADS = SIM_THREADS;
constexpr long long RG_ENTRIES = 32768, RG_ITEMS = 262144;  // bounds of an FD launch

// Workgroups per chunk: small plans of full chunks take a quarter of a chunk
// each, one sample per thread (a pass of forty exact-gradient steps over 432
// chunks: 3.78 -> 2.98 ms).  With 4 608 chunks, which fill the chip by
// themselves, four samples per thread share the reductions (10.9 ms, split
// 13.1 ms), and patches of 256 samples leave nothing to split (FD 2.35 ms, split
// 2.99 ms).
constexpr int RG_SPLIT_MAX_ITEMS = 2048;
__host__ __device__ inline int chunk_split(long long N, int items) {
  return items <= RG_SPLIT_MAX_ITEMS && N > 512LL * items ? 4 : 1;
}

// Central-difference points evaluated per launch.
__host__ __device__ inline int fd_width(int M, int items) {
  long long v = RG_ENTRIES / M;
  if (RG_ITEMS / items < v) v = RG_ITEMS / items;
  return v < 1 ? 1 : v > 12 ? 12 : (int)v;
}

// Population NCC from its six sums (0 for flat patches).
__device__ __forceinline__ double ncc_of(const double s[6]) {
  const double cnt = s[0];
  if (!(cnt > 0)) return 0.0;
  const double my = s[1] / cnt, mh = s[3] / cnt;
  const double vy = s[2] / cnt - my * my, vh = s[4] / cnt - mh * mh;
  const double cv = s[5] / cnt - my * mh;
  if (!(vy > 1e-12 * my * my) || !(vh > 1e-12 * mh * mh) || !(vy > 0) || !(vh > 0)) return 0.0;
  return cv / sqrt(vy * vh);
}

// Sums of N doubles per thread over the workgroup (wave butterflies, then the
// wave results in order), written by thread 0.
template <int N>
__device__ __forceinline__ void sums_out(const double v[N], double *__restrict__ out) {
  __shared__ double red[N][RG_THREADS / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < N; ++q) {
    double x = v[q];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[q][wave] = x;
  }
  __syncthreads();
  if (threadIdx.x < N) {
    double x = 0;
#pragma unroll
    for (int w = 0; w < RG_THREADS / 64; ++w) x += red[threadIdx.x][w];
    out[threadIdx.x] = x;
  }
}

}  // namespace

// Optimiser start: standard deviation of the observed (unmasked) samples, the
// scaled variables.  One workgroup per patch.
__global__ void __launch_bounds__(256)
k_reg_begin(const StackDev *__restrict__ stacks, const PatchDev *__restrict__ patches,
            const float *__restrict__ y, const uint8_t *__restrict__ mask,
            const float *__restrict__ theta, const uint8_t *__restrict__ reg, pvr_reg_params prm,
            RegState *__restrict__ state, int *__restrict__ live) {
  __shared__ double red[3][4];
  const int s = blockIdx.x;
  if (s == 0 && threadIdx.x == 0) *live = 0;
  const PatchDev pt = patches[s];
  const int n = pt.w * pt.h;
  double v[3] = {0, 0, 0};
  for (int l = threadIdx.x; l < n; l += 256) {
    const long long j = pt.off + l;
    if (!mask[j]) continue;
    const double yo = y[j];
    v[0] += 1.0;
    v[1] += yo;
    v[2] += yo * yo;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
    if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = v[q];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = ((red[q][0] + red[q][1]) + red[q][2]) + red[q][3];
  double sd = 0;
  if (v[0] > 0) {
    const double m = v[1] / v[0];
    sd = sqrt(fmax(v[2] / v[0] - m * m, 0.0));
  }
  RegState &o = state[s];
  const StackDev &st = stacks[pt.stack];
  const double su = st.spacing[0], sv = st.spacing[1];
  double rho = 0.5 * sqrt((pt.w - 1) * (pt.w - 1) * su * su + (pt.h - 1) * (pt.h - 1) * sv * sv);
  rho = rho < 1.0 ? 1.0 : rho;
  for (int a = 0; a < 6; ++a) {
    o.sc[a] = a < 3 ? rho : 1.0;
    o.q[a] = (double)theta[6 * s + a] * o.sc[a];
    o.grad[a] = 0.0;
  }
  o.f0 = 0.0;
  o.delta = prm.step0;
  o.walked[0] = o.walked[1] = 0.0;
  o.evals[0] = o.evals[1] = 0;
  o.have_grad = o.moved = 0;
  o.run = (reg ? reg[s] != 0 : true) && sd >= prm.min_std && prm.max_iter > 0;
}

// Per patch (one wavefront): combines the partial sums of the stage `prev`
// (points v0 .. v0 + nv - 1 for FD), moves the optimiser on, and prepares the
// stage `next` (points w0 .. w0 + nw - 1 for FD: lane i builds point w0 + i;
// one transform: the lanes share its sines and cosines).
__global__ void __launch_bounds__(64)
k_reg_advance(const ProbDev *__restrict__ probs, const StackDev *__restrict__ stacks,
              const PatchDev *__restrict__ patches, const int *__restrict__ item_off, int M,
              int items, int split, int psf, int prev, int v0, int nv, int next, int w0, int nw,
              pvr_reg_params prm, double k, RegState *__restrict__ state, EvalGeo *__restrict__ eg,
              GradGeo *__restrict__ gg, const double *__restrict__ part,
              float *__restrict__ theta, float *__restrict__ ncc,
              unsigned long long *__restrict__ stats, int *__restrict__ live, int stage) {
  __shared__ double sum[72];
  __shared__ double thl[6];
  __shared__ int go;
  const int s = blockIdx.x, lane = threadIdx.x;
  RegState &st = state[s];
  const bool was = prev != ST_BEGIN && eg[s].on;
  const int i0 = item_off[s] * split, i1 = item_off[s + 1] * split;
  if (was) {
    const int n = prev == ST_GRAD ? 24 : 6 * nv;
    for (int q = lane; q < n; q += 64) {
      double x = 0;
      if (prev == ST_GRAD)
        for (int i = i0; i < i1; ++i) x += part[24LL * i + q];
      else
        for (int i = i0; i < i1; ++i) x += part[6 * ((long long)(q / 6) * items * split + i) + q % 6];
      sum[q] = x;
    }
  }
  __syncthreads();
  if (lane == 0) {
    if (was) {
      if (prev == ST_GRAD) {
        const double ncc0 = ncc_of(sum), cnt = sum[0];
        double g[6] = {0, 0, 0, 0, 0, 0};
        const double my = sum[1] / cnt, mh = sum[3] / cnt;
        const double vy = sum[2] / cnt - my * my, vh = sum[4] / cnt - mh * mh;
        if (cnt > 0 && vy > 1e-12 * my * my && vh > 1e-12 * mh * mh && vy > 0 && vh > 0) {
          const double sab = cnt * sqrt(vy * vh), sb = cnt * vh;
          for (int c = 0; c < 6; ++c)
            g[c] = (sum[12 + c] - my * sum[6 + c]) / sab - ncc0 * (sum[18 + c] - mh * sum[6 + c]) / sb;
        }
        for (int a = 0; a < 6; ++a) st.grad[a] = g[a] / st.sc[a];
        st.have_grad = 1;
        st.walked[1] += cnt;
        st.evals[1] += 1;
      } else {
        for (int v = 0; v < nv; ++v) {
          const double f = ncc_of(sum + 6 * v);
          st.walked[0] += sum[6 * v];
          st.evals[0] += 1;
          if (prev == ST_POINT) {
            st.f0 = f;
          } else if (prev == ST_FD) {
            st.fd[v0 + v] = f;
          } else if (f > st.f0) {  // TRIAL
            double gn = 0;
            for (int a = 0; a < 6; ++a) gn += st.grad[a] * st.grad[a];
            gn = sqrt(gn);
            for (int a = 0; a < 6; ++a) st.q[a] = st.q[a] + st.delta * st.grad[a] / gn;
            st.f0 = f;
            st.have_grad = 0;
            st.moved = 1;
            st.delta = fmin(2.0 * st.delta, prm.step0);
          } else {
            st.delta *= 0.5;
          }
        }
        if (prev == ST_FD && v0 + nv == 12) {
          for (int a = 0; a < 6; ++a) st.grad[a] = (st.fd[2 * a] - st.fd[2 * a + 1]) / (2.0 * prm.fd_h);
          st.have_grad = 1;
        }
      }
    }
    if (st.delta < prm.step_min) st.run = 0;
    bool on = next == ST_POINT;
    if (next == ST_GRAD || next == ST_FD) on = st.run && !st.have_grad;
    for (int a = 0; a < 6; ++a) thl[a] = st.q[a] / st.sc[a];
    if (next == ST_TRIAL && st.run) {
      double gn = 0;
      for (int a = 0; a < 6; ++a) gn += st.grad[a] * st.grad[a];
      gn = sqrt(gn);
      if (!(gn > 0)) st.run = 0;
      else
        for (int a = 0; a < 6; ++a) thl[a] = (st.q[a] + st.delta * st.grad[a] / gn) / st.sc[a];
      on = st.run != 0;
    }
    go = on;
    if (on) *live = stage;  // (the same value from every patch)
    if (next == ST_END) {
      if (st.moved)
        for (int a = 0; a < 6; ++a) theta[6 * s + a] = (float)(st.q[a] / st.sc[a]);
      if (ncc) ncc[s] = (float)st.f0;
      atomicAdd(&stats[0], (unsigned long long)st.evals[0]);
      atomicAdd(&stats[1], (unsigned long long)st.walked[0]);
      atomicAdd(&stats[2], (unsigned long long)st.evals[1]);
      atomicAdd(&stats[3], (unsigned long long)st.walked[1]);
    }
  }
  __syncthreads();
  if (next == ST_END) return;
  if (!go) {
    if (lane < nw) eg[(long long)lane * M + s].on = 0;
    return;
  }
  const PatchDev pt = patches[s];
  const ProbDev &pr = probs[pt.problem];
  const StackDev &sk = stacks[pt.stack];
  auto build = [&](EvalGeo &e, const double *th, const Trig &trig) {
    GeoD gd;
    int bb[6];
    if (psf == PVR_PSF_SINC) make_geometry<PVR_PSF_SINC>(pr, sk, pt, th, trig, k, gd, e.g, bb);
    else make_geometry<PVR_PSF_GAUSSIAN>(pr, sk, pt, th, trig, k, gd, e.g, bb);
    e.on = 1;
    return gd;
  };
  if (next == ST_FD) {
    if (lane >= nw) return;
    const int w = w0 + lane;
    double th[6];
    for (int a = 0; a < 6; ++a)
      th[a] = a == w / 2 ? (st.q[a] + (w % 2 ? -prm.fd_h : prm.fd_h)) / st.sc[a] : thl[a];
    build(eg[(long long)lane * M + s], th, make_trig(th));
    return;
  }
  const Trig trig = wave_trig(thl);
  if (lane != 0) return;
  const GeoD gd = build(eg[s], thl, trig);
  if (next == ST_GRAD) {
    GradConst gc;
    make_grad_const(pr, sk, pt, thl, trig, gc);
    GradGeo &o = gg[s];
    make_grad_mom(gc, gd.perm, o.gm);
    for (int r = 0; r < 3; ++r) {
      const double *V = gc.Vl + 3 * r;
      double c[4];
      for (int q = 0; q < 4; ++q) c[q] = V[0] * gd.H[q] + V[1] * gd.H[4 + q] + V[2] * gd.H[8 + q];
      o.Q[3 * r] = c[0];
      o.Q[3 * r + 1] = c[1];
      o.Q[3 * r + 2] = c[2] * pt.slice + c[3] + gc.v2w_o[r] - gc.ct[r];
    }
  }
}

// NCC sums of one chunk (its part blockIdx.z) at the transforms blockIdx.y: count, sum y, y^2, yh, yh^2,
// y yh over the chunk's valid samples.  A launch that no patch takes part in ends at
// its first load, before the chunk's and the patch's (256 central-difference steps of
// 8 064 patches of 64 x 64 of which none moves: 51 -> 32 ms, 1 152 patches 8.4 -> 5.6).
template <int PSF>
__global__ void __launch_bounds__(RG_THREADS)
k_reg_eval(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
           const BlockWork *__restrict__ work, const EvalGeo *__restrict__ eg, int M,
           const float *__restrict__ X, const float *__restrict__ XT, const float *__restrict__ y,
           const uint8_t *__restrict__ mask, double *__restrict__ part, int items, int granule,
           const int *__restrict__ live, int stage) {
  if (*live != stage) return;
  const int wi = xcd_work(blockIdx.x, granule);
  if (wi >= items) return;
  const BlockWork wk = work[wi];
  const EvalGeo &e = eg[(long long)blockIdx.y * M + wk.patch];
  if (!e.on) return;
  const GeoF &g = e.g;
  const PatchDev pt = patches[wk.patch];
  const ProbDev pr = probs[pt.problem];
  const unsigned nbytes = (unsigned)(pr.nx * pr.ny * pr.nz) * 4u;
  const bool xt = XT != nullptr && pt.layout == 1;
  const __amdgpu_buffer_rsrc_t xr = raw_buffer((xt ? XT : X) + pr.vol_off, nbytes);
  const int len = SIM_CHUNK / gridDim.z, l0 = wk.l0 + blockIdx.z * len;
  const int l1 = min(pt.w * pt.h, l0 + len);
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int l = l0 + threadIdx.x; l < l1; l += RG_THREADS) {
    const long long j = pt.off + l;
    if (!mask[j]) continue;
    int b[3];
    float f[3];
    if (!sample_centre(g, pr, pt.x0 + l % pt.w, pt.y0 + l / pt.w, pt.slice, b, f)) continue;
    float z = 0.f, a;
    if constexpr (PSF == PVR_PSF_SINC) {
      if (xt)
        a = g.perm[2] == 1 ? psf_walk_sinc<float, GeoF, true, 1, true>(g, pr, b, f, xr, nbytes, &z)
                           : psf_walk_sinc<float, GeoF, true, 2, true>(g, pr, b, f, xr, nbytes, &z);
      else
        a = g.perm[2] == 0 ? psf_walk_sinc<float, GeoF, true, 1>(g, pr, b, f, xr, nbytes, &z)
                           : psf_walk_sinc<float, GeoF, true, 2>(g, pr, b, f, xr, nbytes, &z);
    } else {
      if (xt)
        a = g.perm[2] == 1 ? psf_walk_fwd<float, GeoF, true, 1, true>(g, pr, b, f, xr, nbytes, &z)
                           : psf_walk_fwd<float, GeoF, true, 2, true>(g, pr, b, f, xr, nbytes, &z);
      else
        a = g.perm[2] == 0 ? psf_walk_fwd<float, GeoF, true, 1>(g, pr, b, f, xr, nbytes, &z)
                           : psf_walk_fwd<float, GeoF, true, 2>(g, pr, b, f, xr, nbytes, &z);
    }
    if (!(z > 0.f)) continue;
    const double yh = (double)(a / z), yo = (double)y[j];
    acc[0] += 1.0;
    acc[1] += yo;
    acc[2] += yo * yo;
    acc[3] += yh;
    acc[4] += yh * yh;
    acc[5] += yo * yh;
  }
  sums_out<6>(acc, part + 6 * (((long long)blockIdx.y * items + wi) * gridDim.z + blockIdx.z));
}

// The six NCC sums and, with d = d yh / d theta_c, the sums of d, y d and yh d
// of one chunk (Gaussian PSF).  Held to 128 registers, four waves per SIMD: a
// pass over 11 760 patches of 64 x 64 at 256^3 takes 67.6 ms, with 140 registers 69.3.
__global__ void __launch_bounds__(RG_THREADS, 4)
k_reg_grad(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
           const BlockWork *__restrict__ work, const EvalGeo *__restrict__ eg,
           const GradGeo *__restrict__ gg, const float *__restrict__ X,
           const float *__restrict__ XT, const float *__restrict__ y,
           const uint8_t *__restrict__ mask, double *__restrict__ part, int items, int granule,
           const int *__restrict__ live, int stage) {
  if (*live != stage) return;
  const int wi = xcd_work(blockIdx.x, granule);
  if (wi >= items) return;
  const BlockWork wk = work[wi];
  const EvalGeo &e = eg[wk.patch];
  if (!e.on) return;
  const GeoF &g = e.g;
  const GradGeo &gr = gg[wk.patch];
  const PatchDev pt = patches[wk.patch];
  const ProbDev pr = probs[pt.problem];
  const unsigned nbytes = (unsigned)(pr.nx * pr.ny * pr.nz) * 4u;
  const bool xt = XT != nullptr && pt.layout == 1;
  const __amdgpu_buffer_rsrc_t xr = raw_buffer((xt ? XT : X) + pr.vol_off, nbytes);
  const int len = SIM_CHUNK / gridDim.z, l0 = wk.l0 + blockIdx.z * len;
  const int l1 = min(pt.w * pt.h, l0 + len);
  double acc[24];
#pragma unroll
  for (int q = 0; q < 24; ++q) acc[q] = 0.0;
  for (int l = l0 + threadIdx.x; l < l1; l += RG_THREADS) {
    const long long j = pt.off + l;
    if (!mask[j]) continue;
    const int u = pt.x0 + l % pt.w, v = pt.y0 + l / pt.w;
    int b[3];
    float f[3], xb, a, z, mx[9], me[9];
    if (!sample_centre(g, pr, u, v, pt.slice, b, f)) continue;
    if (xt) {
      if (g.perm[2] == 1) psf_walk_grad<1, true>(g, pr, b, f, xr, nbytes, xb, a, z, mx, me);
      else psf_walk_grad<2, true>(g, pr, b, f, xr, nbytes, xb, a, z, mx, me);
    } else {
      if (g.perm[2] == 0) psf_walk_grad<1, false>(g, pr, b, f, xr, nbytes, xb, a, z, mx, me);
      else psf_walk_grad<2, false>(g, pr, b, f, xr, nbytes, xb, a, z, mx, me);
    }
    if (!(z > 0.f)) continue;
    const float iz = 1.f / z;
    const float dl = a * iz;  // y_hat - X_b
    const float yhf = xb + dl;
    float m[9], qt[3], a6[6];
#pragma unroll
    for (int c = 0; c < 9; ++c) m[c] = fma(-dl, me[c], mx[c]);
    // q = x_j - (c + t)
#pragma unroll
    for (int r = 0; r < 3; ++r)
      qt[r] = (float)fma(gr.Q[3 * r], (double)u, fma(gr.Q[3 * r + 1], (double)v, gr.Q[3 * r + 2]));
    grad_from_moments(gr.gm, m, qt, a6);
    const double yh = (double)yhf, yo = (double)y[j];
    acc[0] += 1.0;
    acc[1] += yo;
    acc[2] += yo * yo;
    acc[3] += yh;
    acc[4] += yh * yh;
    acc[5] += yo * yh;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const double d = (double)(a6[c] * iz);
      acc[6 + c] += d;
      acc[12 + c] += yo * d;
      acc[18 + c] += yh * d;
    }
  }
  sums_out<24>(acc, part + 24LL * ((long long)wi * gridDim.z + blockIdx.z));
}

// Byte offsets of the states, the evaluated transforms, the gradient constants,
// the partial sums and the last stage that a patch took part in, in the plan's registration scratch; returns its size.
size_t pvr::reg_state_bytes(const pvr_plan *p, size_t off[5]) {
  const size_t M = p->M, items = p->n_sim_blocks, nv = fd_width(p->M, p->n_sim_blocks);
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  off[0] = 0;
  off[1] = off[0] + up(M * sizeof(RegState));
  off[2] = off[1] + up(M * nv * sizeof(EvalGeo));
  off[3] = off[2] + up(M * sizeof(GradGeo));
  off[4] = off[3] + up(items * chunk_split(p->N, p->n_sim_blocks) * std::max<size_t>(24, 6 * nv) * sizeof(double));
  return off[4] + up(sizeof(int));
}

pvr_status pvr::register_in_step(const pvr_plan *p, const float *X, const float *XT,
                                 const float *y, float *theta, float *ncc, const uint8_t *reg,
                                 const pvr_reg_params &prm, hipStream_t stream) {
  size_t off[5];
  reg_state_bytes(p, off);
  RegState *state = (RegState *)(p->d_reg + off[0]);
  EvalGeo *eg = (EvalGeo *)(p->d_reg + off[1]);
  GradGeo *gg = (GradGeo *)(p->d_reg + off[2]);
  double *part = (double *)(p->d_reg + off[3]);
  int *live = (int *)(p->d_reg + off[4]), stage = 0;
  const int M = p->M, items = p->n_sim_blocks, width = fd_width(M, items);
  const bool exact = prm.gradient == PVR_REG_GRAD_EXACT;
  const unsigned grid = xcd_blocks(items, p->sim_granule), split = chunk_split(p->N, items);
  hipLaunchKernelGGL(k_reg_begin, dim3(M), dim3(256), 0, stream, p->d_stack, p->d_patch, y, p->d_mask,
                     theta, reg, prm, state, live);
  HIP_TRY(hipGetLastError());
  int prev = ST_BEGIN, v0 = 0, nv = 1;  // the stage whose sums are waiting
  auto advance = [&](int next, int w0, int nw) {
    hipLaunchKernelGGL(k_reg_advance, dim3(M), dim3(64), 0, stream, p->d_prob, p->d_stack, p->d_patch,
                       p->d_item_off, M, items, (int)split, p->psf, prev, v0, nv, next, w0, nw, prm, p->k, state, eg, gg,
                       part, theta, ncc, p->d_reg_stats, live, ++stage);
    prev = next; v0 = w0; nv = nw;
  };
  auto eval = [&](int n) {
    if (p->psf == PVR_PSF_SINC)
      hipLaunchKernelGGL(k_reg_eval<PVR_PSF_SINC>, dim3(grid, n, split), dim3(RG_THREADS), 0, stream,
                         p->d_prob, p->d_patch, p->d_sim_blocks, eg, M, X, XT, y, p->d_mask, part, items,
                         p->sim_granule, live, stage);
    else
      hipLaunchKernelGGL(k_reg_eval<PVR_PSF_GAUSSIAN>, dim3(grid, n, split), dim3(RG_THREADS), 0, stream,
                         p->d_prob, p->d_patch, p->d_sim_blocks, eg, M, X, XT, y, p->d_mask, part, items,
                         p->sim_granule, live, stage);
  };
  advance(ST_POINT, 0, 1);
  eval(1);
  for (int it = 0; it < prm.max_iter; ++it) {
    if (exact) {
      advance(ST_GRAD, 0, 1);
      hipLaunchKernelGGL(k_reg_grad, dim3(grid, 1, split), dim3(RG_THREADS), 0, stream, p->d_prob, p->d_patch,
                         p->d_sim_blocks, eg, gg, X, XT, y, p->d_mask, part, items, p->sim_granule,
                         live, stage);
    } else {
      for (int w = 0; w < 12; w += width) {
        const int n = std::min(width, 12 - w);
        advance(ST_FD, w, n);
        eval(n);
      }
    }
    advance(ST_TRIAL, 0, 1);
    eval(1);
    HIP_TRY(hipGetLastError());
  }
  advance(ST_END, 0, 1);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
}
