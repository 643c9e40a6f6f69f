// EM robust weights of one SR iteration (inlier Gaussian, uniform outlier
// density, inlier posterior p, patch potential p_bar, patch classification,
// M-step).  All sums are FP64 and reduced in a fixed order.
//
// Kernels, in call order:
//   k_em_patch_stats  one workgroup per patch: min / max residual, max |y|,
//                     sum e^2 and count over the patch's valid samples
//   k_em_problem      one workgroup per problem: m = 1/(max e - min e), and at
//                     the start of a cycle sigma^2 = mean(e^2), c = 0.9
//   k_em_estep        one workgroup per patch: p_j, N_s, sum p^2, sum p,
//                     sum p e^2, p_bar_s
//   k_em_patches      one workgroup per problem: two-component mixture on
//                     {p_bar_s} (median split start, 20 EM iterations), W_s,
//                     and the M-step for the next iteration
#include <math.h>

#include "pvr_internal.h"
#include "pvr_util.h"

using namespace pvr;

constexpr int EM_T = 256;     // per-patch workgroups
constexpr int EMP_T = 1024;   // per-problem workgroups
constexpr int PSTAT = 5;      // doubles per patch of the residual statistics
constexpr int EMP_LDS = 12288; // patches per problem whose potentials fit the LDS copy

// Workgroup reductions in a fixed order: a butterfly inside every wave, then
// the wave results combined in wave order by every lane.  lds must hold
// NT / 64 doubles per reduced value.
enum class Op { Sum, Min, Max };

template <Op OP>
__device__ __forceinline__ double combine(double a, double b) {
  if (OP == Op::Sum) return a + b;
  if (OP == Op::Min) return fmin(a, b);
  return fmax(a, b);
}

// The value of lane ^ O (O = 32, 16: swaps of half wavefronts and rows of 16;
// 8 .. 1: rotations within a row, where the values repeat every 2 O lanes, as
// they do in a butterfly from 32 down), a few cycles instead of an LDS
// permutation's hundred.
template <int O>
__device__ __forceinline__ double from_xor(double x) {
  const uint2 u = __builtin_bit_cast(uint2, x);
  uint2 r;
  if constexpr (O == 32 || O == 16) {
    // {own half or row's low, high}: the sum of both is wanted, so either order
    // will do; the other lane's value is the one that is not this lane's
    const auto a = O == 32 ? __builtin_amdgcn_permlane32_swap(u.x, u.x, false, false)
                           : __builtin_amdgcn_permlane16_swap(u.x, u.x, false, false);
    const auto b = O == 32 ? __builtin_amdgcn_permlane32_swap(u.y, u.y, false, false)
                           : __builtin_amdgcn_permlane16_swap(u.y, u.y, false, false);
    const bool high = threadIdx.x & O;
    r = make_uint2(high ? a[0] : a[1], high ? b[0] : b[1]);
  } else {
    r = make_uint2(__builtin_amdgcn_update_dpp(0u, u.x, 0x120 + O, 0xf, 0xf, false),
                   __builtin_amdgcn_update_dpp(0u, u.y, 0x120 + O, 0xf, 0xf, false));
  }
  return __builtin_bit_cast(double, r);
}
// Reduction over the wavefront in every lane, by a butterfly from lane ^ 32 down.
template <Op OP>
__device__ __forceinline__ double wave_reduce(double x) {
  x = combine<OP>(x, from_xor<32>(x));
  x = combine<OP>(x, from_xor<16>(x));
  x = combine<OP>(x, from_xor<8>(x));
  x = combine<OP>(x, from_xor<4>(x));
  x = combine<OP>(x, from_xor<2>(x));
  return combine<OP>(x, from_xor<1>(x));
}

template <int NT, Op OP>
__device__ __forceinline__ double breduce(double v, double *lds) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_reduce<OP>(v);
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  double r = lds[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) r = combine<OP>(r, lds[w]);
  __syncthreads();
  return r;
}

// K sums at once (one pair of barriers)
template <int NT, int K>
__device__ __forceinline__ void bsumk(double (&v)[K], double *lds) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    const double x = wave_reduce<Op::Sum>(v[q]);
    if (lane == 0) lds[q * NW + wave] = x;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < K; ++q) {
    double r = lds[q * NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) r += lds[q * NW + w];
    v[q] = r;
  }
  __syncthreads();
}

template <int NT> __device__ __forceinline__ double bsum(double v, double *lds) { return breduce<NT, Op::Sum>(v, lds); }
template <int NT> __device__ __forceinline__ double bmin(double v, double *lds) { return breduce<NT, Op::Min>(v, lds); }
template <int NT> __device__ __forceinline__ double bmax(double v, double *lds) { return breduce<NT, Op::Max>(v, lds); }

__global__ void __launch_bounds__(EM_T)
k_em_patch_stats(const PatchDev *__restrict__ patches, const float *__restrict__ invz,
                 const float *__restrict__ e, const float *__restrict__ y,
                 double *__restrict__ pstat) {
  __shared__ double lds[8 * (EM_T / 64)];
  const int s = blockIdx.x;
  const PatchDev pt = patches[s];
  const int n = pt.w * pt.h;
  double mn = INFINITY, mx = -INFINITY, ym = 0, se2 = 0, cnt = 0;
  for (int l = threadIdx.x; l < n; l += EM_T) {
    const long long j = pt.off + l;
    if (!(invz[j] > 0.f)) continue;
    const double ev = e[j];
    mn = fmin(mn, ev);
    mx = fmax(mx, ev);
    ym = fmax(ym, fabs((double)y[j]));
    se2 += ev * ev;
    cnt += 1.0;
  }
  mn = bmin<EM_T>(mn, lds);
  mx = bmax<EM_T>(mx, lds);
  ym = bmax<EM_T>(ym, lds);
  double red[2] = {se2, cnt};
  bsumk<EM_T, 2>(red, lds);
  se2 = red[0]; cnt = red[1];
  if (threadIdx.x == 0) {
    double *o = pstat + PSTAT * s;
    o[0] = mn; o[1] = mx; o[2] = ym; o[3] = se2; o[4] = cnt;
  }
}

// Per-problem reduction of the residual statistics: from the per-patch table
// (pstat, stride PSTAT), or with chunk_stats from the forward kernel's
// per-chunk records (stride 5) over the problem's chunk range.
__global__ void __launch_bounds__(EMP_T)
k_em_problem(const ProbDev *__restrict__ probs, const double *__restrict__ pstat,
             const double *__restrict__ chunk_stats, int planes, pvr_em_state *__restrict__ em, int init,
             unsigned *__restrict__ status) {
  __shared__ double lds[8 * (EMP_T / 64)];
  const ProbDev pr = probs[blockIdx.x];
  double mn = INFINITY, mx = -INFINITY, ym = 0, se2 = 0, cnt = 0;
  const int r0 = chunk_stats ? (planes ? pr.pblk_begin : pr.chunk_begin) : pr.patch_begin;
  const int r1 = chunk_stats ? (planes ? pr.pblk_end : pr.chunk_end) : pr.patch_end;
  const double *rec = chunk_stats ? chunk_stats : pstat;
  const long long stride = chunk_stats ? 5 : PSTAT;
  // four records per thread in flight, taken in the order of one at a time
  int s = r0 + threadIdx.x;
  for (; s + 3 * EMP_T < r1; s += 4 * EMP_T) {
    double o[4][5];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < 5; ++k) o[u][k] = rec[stride * (s + u * EMP_T) + k];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      mn = fmin(mn, o[u][0]);
      mx = fmax(mx, o[u][1]);
      ym = fmax(ym, o[u][2]);
      se2 += o[u][3];
      cnt += o[u][4];
    }
  }
  for (; s < r1; s += EMP_T) {
    const double *o = rec + stride * s;
    mn = fmin(mn, o[0]);
    mx = fmax(mx, o[1]);
    ym = fmax(ym, o[2]);
    se2 += o[3];
    cnt += o[4];
  }
  // the five reductions at once: a butterfly inside every wave, then thread 0
  // combines the wave results in wave order (the order of breduce / bsumk)
  {
    constexpr int NW = EMP_T / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    mn = wave_reduce<Op::Min>(mn);
    mx = wave_reduce<Op::Max>(mx);
    ym = wave_reduce<Op::Max>(ym);
    se2 = wave_reduce<Op::Sum>(se2);
    cnt = wave_reduce<Op::Sum>(cnt);
    if (lane == 0) {
      lds[0 * NW + wave] = mn;
      lds[1 * NW + wave] = mx;
      lds[2 * NW + wave] = ym;
      lds[3 * NW + wave] = se2;
      lds[4 * NW + wave] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      mn = lds[0]; mx = lds[NW]; ym = lds[2 * NW]; se2 = lds[3 * NW]; cnt = lds[4 * NW];
      for (int w = 1; w < NW; ++w) {
        mn = fmin(mn, lds[w]);
        mx = fmax(mx, lds[NW + w]);
        ym = fmax(ym, lds[2 * NW + w]);
        se2 += lds[3 * NW + w];
        cnt += lds[4 * NW + w];
      }
    }
  }
  if (threadIdx.x == 0) {
    // min / max skip NaN residuals, their squares' sum does not
    if (!isfinite(se2) || !isfinite(mx - mn) || !isfinite(ym)) atomicOr(status, PVR_FAULT_RESIDUAL);
    pvr_em_state &st = em[blockIdx.x];
    const double eps = 1e-6 * ym;
    const double range = cnt > 0 ? fmax(mx - mn, eps) : 0.0;
    st.m = range > 0 ? 1.0 / range : 1.0;
    st.y_abs_max = ym;
    if (init || !st.started) {
      const double floor2 = (1e-4 * ym) * (1e-4 * ym);
      double s2 = cnt > 0 ? se2 / cnt : 0.0;
      s2 = s2 > 0 ? fmax(s2, floor2) : fmax(floor2, 1.0);
      st.sigma2 = s2;
      st.c = 0.9;
      st.started = 1;
    }
  }
}

__global__ void __launch_bounds__(EM_T)
k_em_estep(const PatchDev *__restrict__ patches, const float *__restrict__ invz,
           const float *__restrict__ e, const pvr_em_state *__restrict__ em,
           float *__restrict__ p_out, float *__restrict__ pbar, double *__restrict__ esum, int M) {
  __shared__ double lds[8 * (EM_T / 64)];
  const int s = blockIdx.x;
  const PatchDev pt = patches[s];
  const pvr_em_state st = em[pt.problem];
  const float sigma2 = (float)st.sigma2;
  const float inv2s2 = (float)(0.5 / st.sigma2);
  const float cG0 = (float)(st.c / sqrt(2.0 * M_PI * st.sigma2));
  const float mo = (float)(st.m * (1.0 - st.c));
  (void)sigma2;
  const int n = pt.w * pt.h;
  double ns = 0, sp2 = 0, sp = 0, spe2 = 0;
  // one sample: the posterior and the sums (invalid samples, 1/Z = 0, get 0)
  auto one = [&](long long j, float iz, float ev) {
    float pj = 0.f;
    if (iz > 0.f) {
      const float Gc = cG0 * expf(-ev * ev * inv2s2);
      const float dd = Gc + mo;
      pj = dd > 0.f ? Gc / dd : 0.f;
      ns += 1.0;
      sp2 += (double)pj * pj;
      sp += pj;
      spe2 += (double)pj * ev * ev;
    }
    if (p_out) p_out[j] = pj;
  };
  // four samples per thread in flight (the loop is latency-bound), taken in
  // the same order as one at a time; e is read for invalid samples too (it
  // is defined for every sample)
  int l = threadIdx.x;
  for (; l + 3 * EM_T < n; l += 4 * EM_T) {
    float iz[4], ev[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long j = pt.off + l + u * EM_T;
      iz[u] = invz[j];
      ev[u] = e[j];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) one(pt.off + l + u * EM_T, iz[u], ev[u]);
  }
  for (; l < n; l += EM_T) {
    const long long j = pt.off + l;
    one(j, invz[j], e[j]);
  }
  double red[4] = {ns, sp2, sp, spe2};
  bsumk<EM_T, 4>(red, lds);
  ns = red[0]; sp2 = red[1]; sp = red[2]; spe2 = red[3];
  if (threadIdx.x == 0) {
    esum[s] = ns;
    esum[M + s] = sp2;
    esum[2LL * M + s] = sp;
    esum[3LL * M + s] = spe2;
    if (pbar) pbar[s] = ns > 0 ? (float)sqrt(sp2 / ns) : 0.f;
  }
}

// Inlier responsibility 1 / (1 + exp(l0 - l1)) with
// l_c = log(weight_c) - log(sd_c) - (v - mu_c)^2 / (2 sd_c^2); the constant
// 0.5 log(2 pi) cancels.  The per-component constants are computed once per
// mixture iteration.
struct Mix {
  double mu0, mu1, h0, h1, c0, c1;  // h = 1 / (2 sd^2), c = log(weight) - log(sd)
};

__device__ __forceinline__ Mix make_mix(double mu0, double sd0, double mu1, double sd1, double w1) {
  Mix m;
  m.mu0 = mu0; m.mu1 = mu1;
  m.h0 = 0.5 / (sd0 * sd0); m.h1 = 0.5 / (sd1 * sd1);
  m.c1 = w1 > 0 ? log(w1) - log(sd1) : -INFINITY;
  m.c0 = w1 < 1 ? log(1.0 - w1) - log(sd0) : -INFINITY;
  return m;
}

__device__ __forceinline__ double inlier_resp(double v, const Mix &m) {
  const double d0 = v - m.mu0, d1 = v - m.mu1;
  const double l1 = m.c1 - d1 * d1 * m.h1;
  const double l0 = m.c0 - d0 * d0 * m.h0;
  return 1.0 / (1.0 + exp(l0 - l1));
}

// The same for the mixture iterations: the exponent in FP64, its whole part
// taken off before the single-precision exponential, so the responsibilities (FP32)
// are right to ~1e-7 relative whatever the exponent (up to hundreds where the
// components are narrow); the sums over patches stay FP64.
__device__ __forceinline__ float inlier_resp_f(double v, const Mix &m) {
  const double d0 = v - m.mu0, d1 = v - m.mu1;
  const double l = (m.c0 - d0 * d0 * m.h0) - (m.c1 - d1 * d1 * m.h1);
  // +-inf when a component has zero weight: 2^200 is inf, 1 / (1 + inf) = 0
  const double t = fmin(fmax(l * 1.4426950408889634, -200.0), 200.0), n = rint(t);
  return __builtin_amdgcn_rcpf(1.f + ldexpf(__builtin_amdgcn_exp2f((float)(t - n)), (int)n));
}

// Lane l's value in every lane.
__device__ __forceinline__ double lane_value(double x, int l) {
  const int2 u = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(u.x, l), __builtin_amdgcn_readlane(u.y, l)));
}

// Two-component mixture on the potentials of one problem, patch weights and
// the M-step.  The start splits the potentials at the median: the n/2 smallest
// form the low component.  The split value is found exactly by a radix select
// on the float bit patterns (potentials are >= 0, so the patterns are ordered
// like the values).
//
// The potentials of the problem's patches (FP64: where the components are narrow,
// 1e-3 at least, an FP32 one's rounding would move a patch's posterior by 1e-4) are
// first gathered into a compact array (-1 marks a patch that takes no part): in LDS when
// the problem has at most EMP_LDS patches, else in the plan's scratch array, so the
// 20 mixture iterations touch only that array.  One pass per iteration gathers
// the high component's sums of r, r v and r v^2; the low component's follow
// from the totals (sum 1, sum v, sum v^2), and each variance is
// E[v^2] - mean^2 (values in [0, 1], FP64: the cancellation costs ~1e-16 /
// var relative, against a floor of 1e-6 on the variance).  Inside the
// iterations the responsibilities are single precision (inlier_resp_f).
//
// Bound by the chain of the iterations: the wavefronts' sums, a barrier, the
// wavefronts' sums in order, the step to the next parameters with its divisions, roots and
// logarithms side by side in lanes.  Few wavefronts shorten the chain, many share the
// patches.  Up to 1 280 patches four wavefronts (64: one), one a SIMD, take the step
// each for itself; beyond, eight (up to 4 096) or sixteen, of which one takes it for
// all, at one more barrier.  Robust weights of one problem with four / eight /
// sixteen wavefronts (us): 300 patches 45 / 49 / 61, 600 50 / 53 / 63, 1 152 58 / 60 /
// 70, 1 600 69 / 67 / 75, 3 000 97 / 86 / 89, 4 000 116 / 104 / 106, 6 000 - / 131 /
// 126.  256^3, 11 760 patches, the fit alone: 170 us; 216 with LDS permutations, one
// lane taking the step and flat reads of the potentials.  CAP: potentials the workgroup keeps in LDS
// (0: none).
// K sums of the workgroup into every lane, in the order of bsumk; two calls with
// the same lds need a barrier in between.
template <int NT, int K>
__device__ __forceinline__ void wsumk(double (&v)[K], double *lds) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double x = wave_reduce<Op::Sum>(v[k]);
    if (lane == 0) lds[k * NW + wave] = x;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    v[k] = lds[k * NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) v[k] += lds[k * NW + w];
  }
}

template <int NT, int CAP>
__global__ void __launch_bounds__(NT)
k_em_patches(const ProbDev *__restrict__ probs,
             const uint8_t *__restrict__ active, const double *__restrict__ esum, int M,
             double *__restrict__ gval, float *__restrict__ patch_w, pvr_em_state *__restrict__ em,
             int fix_w) {
  constexpr int U = CAP == NT ? 1 : 4;             // patches of a lane in flight
  constexpr bool ONE = NT > 256;                   // one wavefront takes the step
  __shared__ double lds[2][4 * (NT / 64)];         // in turn: one barrier a sum
  __shared__ double par[3];                        // variances, weight
  __shared__ Mix mixs;
  __shared__ int stop;
  __shared__ unsigned int hist[256];
  __shared__ unsigned int sel_prefix, sel_rank;
  __shared__ double sval[CAP ? CAP : 1];
  const ProbDev pr = probs[blockIdx.x];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int pb = pr.patch_begin, np = pr.patch_end - pr.patch_begin;
  double *V = CAP ? sval : gval + pb;  // (a choice at run time would make every read a flat one)
  // the patches taking part (valid samples, active) and their potentials; the
  // reads of a patch, and of U patches, are independent
  double n, s_all, q_all;
  {
    double r3[3] = {0, 0, 0};
    for (int q0 = t; q0 < np; q0 += U * NT) {
      double ns[U], sp2[U];
      uint8_t act[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = pb + min(q0 + u * NT, np - 1);
        ns[u] = esum[s];
        sp2[u] = esum[M + s];
        act[u] = active[s];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (q0 + u * NT >= np) continue;
        const double v = (ns[u] > 0 && act[u] != 0) ? sqrt(sp2[u] / ns[u]) : -1.0;
        V[q0 + u * NT] = v;
        if (v >= 0) {
          r3[0] += 1.0;
          r3[1] += v;
          r3[2] += v * v;
        }
      }
    }
    wsumk<NT, 3>(r3, lds[0]);  // its barrier also publishes V
    n = r3[0]; s_all = r3[1]; q_all = r3[2];
  }
  const int nu = (int)n;
  double mu0 = 0, sd0 = 1, mu1 = 0, sd1 = 1, w1 = 0.9;
  const bool fit = nu >= 2;
  if (fit) {
    const int n_lo = nu / 2;
    // radix select of the value of rank n_lo - 1
    if (t == 0) { sel_prefix = 0; sel_rank = (unsigned)(n_lo - 1); }
    __syncthreads();
    for (int pass = 0; pass < 4; ++pass) {
      const int shift = 24 - 8 * pass;
      for (int b = t; b < 256; b += NT) hist[b] = 0;
      __syncthreads();
      const unsigned pref = sel_prefix;
      const unsigned mask_hi = pass == 0 ? 0u : (0xffffffffu << (32 - 8 * pass));
      for (int q0 = t - lane; q0 < np; q0 += NT) {
        const float v = q0 + lane < np ? (float)V[q0 + lane] : -1.f;
        const unsigned bits = __float_as_uint(v), bin = (bits >> shift) & 255u;
        bool on = v >= 0.f && (bits & mask_hi) == pref;
        // the potentials crowd in a few bins: equal ones of a wavefront at once
        for (int k = 0; k < 4; ++k) {
          const unsigned long long left = __ballot(on);
          if (!left) break;
          const int first = __builtin_ctzll(left);
          const unsigned b = __builtin_amdgcn_readlane(bin, first);
          const unsigned long long same = __ballot(on && bin == b);
          if (lane == first) atomicAdd(&hist[b], (unsigned)__popcll(same));
          on = on && bin != b;
        }
        if (on) atomicAdd(&hist[bin], 1u);
      }
      __syncthreads();
      // the bin holding rank r: wave 0 scans the 256 counts (4 per lane)
      if (t < 64) {
        const unsigned r = sel_rank;
        const unsigned h0 = hist[4 * t], h1 = hist[4 * t + 1], h2 = hist[4 * t + 2],
                       h3 = hist[4 * t + 3];
        const unsigned tot = h0 + h1 + h2 + h3;
        unsigned incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const unsigned v = __shfl_up(incl, o, 64);
          if (t >= o) incl += v;
        }
        const unsigned long long hit = __ballot(incl > r);
        if (hit != 0ull && t == __ffsll((long long)hit) - 1) {
          unsigned acc = incl - tot;
          int b = 4 * t;
          if (acc + h0 <= r) {
            acc += h0; ++b;
            if (acc + h1 <= r) {
              acc += h1; ++b;
              if (acc + h2 <= r) { acc += h2; ++b; }
            }
          }
          sel_prefix = pref | ((unsigned)b << shift);
          sel_rank = r - acc;
        }
      }
      __syncthreads();
    }
    const double tv = (double)__uint_as_float(sel_prefix);
    double red3[3] = {0, 0, 0};
    for (int q = t; q < np; q += NT) {
      const double v = V[q];
      if (v >= 0 && (float)v < (float)tv) { red3[0] += 1; red3[1] += v; red3[2] += v * v; }
    }
    wsumk<NT, 3>(red3, lds[1]);
    const double c_lt = red3[0], s_lt = red3[1], q_lt = red3[2];
    Mix mx;
    double var0 = 1, var1 = 1;
    // the parameters from the components' sums of r v and r v^2 and their weights
    // (n1 / nu returned), and the constants of make_mix at the weight `wt` (0: that
    // one): every lane's result, the operations side by side in lanes
    const auto step = [&](double v1, double v0, double q1, double q0, double n1, double n0, double wt) {
      const double num = lane == 0 ? v1 : lane == 1 ? v0 : lane == 2 ? q1 : lane == 3 ? q0 : n1;
      const double den = lane == 4 ? (double)nu : (lane & 1) ? n0 : n1;
      const double m = num / den;
      mx.mu1 = lane_value(m, 0);
      mx.mu0 = lane_value(m, 1);
      w1 = wt > 0 ? wt : lane_value(m, 4);
      const double mu = (lane & 1) ? mx.mu0 : mx.mu1, sq = (lane & 1) ? lane_value(m, 3) : lane_value(m, 2);
      const double var = fmax(sq - mu * mu, 1e-6);  // sd at least 1e-3
      const double h = 0.5 / var;
      const double lg = log(lane < 2 ? var : lane == 2 ? w1 : 1.0 - w1);
      var1 = lane_value(var, 0);
      var0 = lane_value(var, 1);
      mx.h1 = lane_value(h, 0);
      mx.h0 = lane_value(h, 1);
      mx.c1 = lane_value(lg, 2) - 0.5 * lane_value(lg, 0);
      mx.c0 = lane_value(lg, 3) - 0.5 * lane_value(lg, 1);
    };
    const double fill = n_lo - c_lt;
    const double s0 = s_lt + fill * tv, q0 = q_lt + fill * tv * tv;
    step(s_all - s0, s0, q_all - q0, q0, nu - n_lo, n_lo, 0.9);
    for (int it = 0; it < 20; ++it) {
      double red[3] = {0, 0, 0};  // sums of r1, r1 v, r1 v^2
#pragma unroll 4
      for (int q = t; q < np; q += NT) {
        const double v = V[q];
        const double r1 = inlier_resp_f(v, mx);
        if (v >= 0) {
          red[0] += r1;
          red[1] += r1 * v;
          red[2] += r1 * v * v;
        }
      }
      bool last = false;
      if constexpr (ONE) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double x = wave_reduce<Op::Sum>(red[k]);
          if (lane == 0) lds[0][k * (NT / 64) + wave] = x;
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            red[k] = lds[0][k * (NT / 64)];
#pragma unroll
            for (int w = 1; w < NT / 64; ++w) red[k] += lds[0][k * (NT / 64) + w];
          }
          const double r1s = red[0], r0s = nu - r1s;
          last = !(r1s > 0) || !(r0s > 0);
          if (!last) step(red[1], s_all - red[1], red[2], q_all - red[2], r1s, r0s, 0.0);
          if (lane == 0) {
            mixs = mx;
            par[0] = var0; par[1] = var1; par[2] = w1;
            stop = last;
          }
        }
        __syncthreads();
        mx = mixs;
        last = stop;
      } else {
        wsumk<NT, 3>(red, lds[it & 1]);
        const double r1s = red[0], r0s = nu - r1s;
        last = !(r1s > 0) || !(r0s > 0);  // (the same in every lane)
        if (!last) step(red[1], s_all - red[1], red[2], q_all - red[2], r1s, r0s, 0.0);
      }
      if (last) break;
    }
    if constexpr (ONE) {
      var0 = par[0]; var1 = par[1]; w1 = par[2];
    }
    mu0 = mx.mu0; sd0 = sqrt(var0); mu1 = mx.mu1; sd1 = sqrt(var1);
  }
  const bool swap = fit && mu0 > mu1;
  const Mix mfin = make_mix(mu0, sd0, mu1, sd1, w1);
  // patch weights (given, or from the fitted mixture), then the M-step sums over
  // the problem's patches from their partials o = (N_s, sum p, sum p e^2)
  double red4[4] = {0, 0, 0, 0};
  for (int q0 = t; q0 < np; q0 += U * NT) {
    double o5[U], o7[U], o8[U];
    float wg[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = pb + min(q0 + u * NT, np - 1);
      o5[u] = esum[s];
      o7[u] = esum[2LL * M + s];
      o8[u] = esum[3LL * M + s];
      wg[u] = fix_w ? patch_w[s] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * NT, s = pb + q;
      if (q >= np) continue;
      double W;
      const bool on = V[q] >= 0;
      if (fix_w) {
        W = wg[u];
      } else {
        double pi = 0;
        if (on) {
          pi = fit ? inlier_resp(V[q], mfin) : 1.0;
          if (swap) pi = 1.0 - pi;
        }
        W = (on && pi >= 0.5) ? pi : 0.0;
        patch_w[s] = (float)W;
        W = (double)(float)W;
      }
      red4[0] += W * o8[u];
      red4[1] += W * o7[u];
      red4[2] += W * o5[u];
      red4[3] += (on && W == 0) ? 1.0 : 0.0;
    }
  }
  __syncthreads();  // both halves of lds are free
  wsumk<NT, 4>(red4, lds[0]);
  const double swpe2 = red4[0], swp = red4[1], sw = red4[2], nex = red4[3];
  if (t == 0) {
    pvr_em_state &st = em[blockIdx.x];
    const double floor2 = (1e-4 * st.y_abs_max) * (1e-4 * st.y_abs_max);
    st.sum_wp = swp;
    st.sum_wpe2 = swpe2;
    st.sum_w = sw;
    if (swp > 0) st.sigma2 = fmax(swpe2 / swp, floor2);
    if (sw > 0) st.c = swp / sw;
    st.n_used = nu;
    st.n_excluded = (int)nex;
  }
}

extern "C" pvr_status pvr_robust_weights(pvr_plan *p, const float *resid, const float *y_obs,
                                         pvr_em_state *em, float *pp, float *pbar,
                                         float *patch_w, int32_t flags, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_robust_weights", resid, 4);
  PVR_ALIGNED("pvr_robust_weights", y_obs, 4);
  PVR_ALIGNED("pvr_robust_weights", em, 8);
  PVR_ALIGNED("pvr_robust_weights", pp, 4);
  PVR_ALIGNED("pvr_robust_weights", pbar, 4);
  PVR_ALIGNED("pvr_robust_weights", patch_w, 4);
  if (!p || !resid || !y_obs || !em || !patch_w) return fail(PVR_EINVAL, "pvr_robust_weights: NULL argument");
  if (!p->built) return fail(PVR_EINVAL, "pvr_robust_weights: plan has not been built");
  PVR_TRY_STATUS(debug_finite(p, "pvr_robust_weights", "resid", resid, p->N, stream));
  PVR_TRY_STATUS(debug_finite(p, "pvr_robust_weights", "y_obs", y_obs, p->N, stream));
  const int init = (flags & PVR_EM_INIT) != 0;
  const int fix = (flags & PVR_EM_FIX_W) != 0;
  // residual statistics: reused from the forward kernel when the caller vouches
  // that resid is unchanged since the plan's last pvr_simulate wrote it
  const bool fresh = (flags & PVR_EM_RESID_FRESH) && p->stats_valid && p->stats_resid == resid &&
                     p->stats_y == y_obs && p->stats_capture == capture_id(stream);
  if (!fresh) {
    hipLaunchKernelGGL(k_em_patch_stats, dim3(p->M), dim3(EM_T), 0, stream, p->d_patch, p->d_invz,
                       resid, y_obs, p->d_pstat);
    HIP_TRY(hipGetLastError());
  }
  hipLaunchKernelGGL(k_em_problem, dim3(p->P), dim3(EMP_T), 0, stream, p->d_prob, p->d_pstat,
                     fresh ? (const double *)p->d_chunk_stats : nullptr, p->stats_planes ? 1 : 0, em,
                     init, p->d_status);
  HIP_TRY(hipGetLastError());
  hipLaunchKernelGGL(k_em_estep, dim3(p->M), dim3(EM_T), 0, stream, p->d_patch, p->d_invz, resid,
                     em, pp, pbar, p->d_pstat + PSTAT * (long long)p->M, p->M);
  HIP_TRY(hipGetLastError());
  // the adjoint's inputs need the posteriors only, not the patch weights: on
  // request they are prepared on the plan's second stream while the patch
  // classification (one workgroup per problem) runs on this one
  const bool prep = (flags & PVR_EM_PREP_ADJOINT) && pp != nullptr;
  p->rq_fresh = false;
  if (prep) {
    HIP_TRY(hipEventRecord(p->ev_fork, stream));
    HIP_TRY(hipStreamWaitEvent(p->side, p->ev_fork, 0));
    const pvr_status st = launch_bp_prep(p, resid, pp, p->side);
    if (st != PVR_OK) return st;
    HIP_TRY(hipEventRecord(p->ev_join, p->side));
  }
#define PATCHES_LAUNCH(NT, CAP)                                                                   \
  hipLaunchKernelGGL((k_em_patches<NT, CAP>), dim3(p->P), dim3(NT),                              \
                     0, stream, p->d_prob, p->d_active, p->d_pstat + PSTAT * (long long)p->M, \
                     p->M, p->d_pval, patch_w, em, fix)
  if (p->max_problem_patches <= 64) PATCHES_LAUNCH(64, 64);
  else if (p->max_problem_patches <= 256) PATCHES_LAUNCH(256, 256);
  else if (p->max_problem_patches <= 1280) PATCHES_LAUNCH(256, 1280);
  else if (p->max_problem_patches <= 4096) PATCHES_LAUNCH(512, 4096);
  else if (p->max_problem_patches <= EMP_LDS) PATCHES_LAUNCH(EMP_T, EMP_LDS);
  else PATCHES_LAUNCH(EMP_T, 0);
#undef PATCHES_LAUNCH
  HIP_TRY(hipGetLastError());
  if (prep) {
    HIP_TRY(hipStreamWaitEvent(stream, p->ev_join, 0));
    p->rq_fresh = true;
    p->rq_capture = capture_id(stream);
    p->rq_e = resid;
    p->rq_p = pp;
  }
  return PVR_OK;
  PVR_API_END();
}
