// Adjoint direction ("pixel-volume") as a gather: every voxel sums, in a fixed
// order, the contributions of the samples whose PSF support covers it, so no
// two lanes ever write the same address and the result is bitwise repeatable.
//
// For a voxel and a patch, the voxel is mapped (FP64 affine G) into the
// patch's unmoved pixel frame; the PSF is axis-aligned there, so the candidate
// pixels are the integer (u, v) inside an ellipse around the mapped point, on
// the patch's single slice.  Two kernels: k_gather_blocks (2 x 2 voxels per
// lane, where pixels are about as wide as voxels and the PSF about as wide as
// a pixel: pvr_plan::gather_blocks) and k_backproject (one voxel per lane, any
// sizes; patches indexed per 4^3 sub-brick).
#include <math.h>

#include "pvr_internal.h"
#include "pvr_util.h"

using namespace pvr;

constexpr int BP_THREADS = BRICK * BRICK * BRICK;

template <typename T> struct Vec2Of;
template <> struct Vec2Of<float> { using type = float2; };
template <> struct Vec2Of<double> { using type = double2; };

// Where the inputs rq of a patch lie.  FP32: rows padded by RQ_PAD zeros, from
// the patch's rq_off; FP64: packed like the samples, one guard entry before and
// after all N.  lead: index of pixel (0, 0) in the view; pitch: entries per row.
template <typename T> struct Rq;
template <> struct Rq<float> {
  static constexpr int lead = RQ_PAD;
  static __device__ __forceinline__ int pitch(int w) { return rq_pitch(w); }
  static __device__ __forceinline__ __amdgpu_buffer_rsrc_t view(const float2 *rq, const PatchDev &pt) {
    return raw_buffer(rq + pt.rq_off, (unsigned)rq_entries(pt.w, pt.h) * (unsigned)sizeof(float2));
  }
};
template <> struct Rq<double> {
  static constexpr int lead = 1;
  static __device__ __forceinline__ int pitch(int w) { return w; }
  static __device__ __forceinline__ __amdgpu_buffer_rsrc_t view(const double2 *rq, const PatchDev &pt) {
    return raw_buffer(rq + pt.off - 1, (unsigned)(pt.w * pt.h + 2) * (unsigned)sizeof(double2));
  }
};

// rq_j = (p_j e_j / Z_j, p_j / Z_j) for valid samples, 0 otherwise (the
// patch weight W_s is applied by the gather, per patch).  Leaves its number in *odd
// where one is not finite (see k_gather_blocks).
template <typename T>
__global__ void __launch_bounds__(SIM_THREADS)
k_bp_prep(const PatchDev *__restrict__ patches, const BlockWork *__restrict__ work,
          const T *__restrict__ invz, const T *__restrict__ e, const T *__restrict__ p,
          typename Vec2Of<T>::type *__restrict__ rq, unsigned *__restrict__ odd, unsigned call) {
  const BlockWork wk = work[blockIdx.x];
  const PatchDev pt = patches[wk.patch];
  const int n = pt.w * pt.h;
  const int l1 = min(n, wk.l0 + SIM_CHUNK);
  typename Vec2Of<T>::type *out =
      sizeof(T) == 4 ? rq + pt.rq_off + RQ_PAD : rq + pt.off;
  // one sample (invalid samples, 1/Z = 0, get 0); a padded row adds RQ_PAD
  // entries per pixel row before it
  bool bad = false;
  auto one = [&](int l, T iz, T pj, T ej) {
    typename Vec2Of<T>::type o;
    if (iz > (T)0) {
      const T q = pj * iz;
      o.x = q * ej;
      o.y = q;
      bad = bad || !__builtin_isfinite(o.x) || !__builtin_isfinite(q);
    } else {
      o.x = 0;
      o.y = 0;
    }
    out[sizeof(T) == 4 ? l + RQ_PAD * (l / pt.w) : l] = o;
  };
  // four samples per thread in flight: their reads are independent (e and p
  // are defined for every sample)
  int l = wk.l0 + threadIdx.x;
  for (; l + 3 * SIM_THREADS < l1; l += 4 * SIM_THREADS) {
    T iz[4], pj[4], ej[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long j = pt.off + l + u * SIM_THREADS;
      iz[u] = invz[j];
      pj[u] = p ? p[j] : (T)1;
      ej[u] = e[j];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) one(l + u * SIM_THREADS, iz[u], pj[u], ej[u]);
  }
  for (; l < l1; l += SIM_THREADS) {
    const long long j = pt.off + l;
    one(l, invz[j], p ? p[j] : (T)1, e[j]);
  }
  if (bad) *odd = call;
}

// A buffer load never faults: outside the patch's view it returns 0, so
// candidate pixels off the patch need no address clamp.  Their weights are
// zeroed explicitly, so whatever such a load returns never contributes.  The
// margin around the patch's entries (Rq::lead, the row padding) matters
// because the compiler merges the loads of two adjacent candidates into one
// 16-byte load, and a partly out-of-range load may return 0 for all of it:
// with the margin, a pair holding an in-patch entry is always wholly in range.
template <typename V2> __device__ __forceinline__ V2 load_rq(__amdgpu_buffer_rsrc_t r, int off);
template <> __device__ __forceinline__ float2 load_rq<float2>(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <> __device__ __forceinline__ double2 load_rq<double2>(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// max(a b - c, 0) for a b - c in [-1, 1]: one FMA with the output clamp.
template <typename T> __device__ __forceinline__ T fma_clamp0(T a, T b, T c);
template <> __device__ __forceinline__ float fma_clamp0<float>(float a, float b, float c) {
  return __builtin_amdgcn_fmed3f(fmaf(a, b, -c), 0.f, 1.f);
}
template <> __device__ __forceinline__ double fma_clamp0<double>(double a, double b, double c) {
  return fmax(fma(a, b, -c), 0.0);
}

// Contribution of one patch to one voxel mapped to pixel coordinates
// (pu, pv) with normalised through-plane term qk.  The candidate pixels are
// rint(p) + [-HU, HU] x [-HV, HV] (a superset of the integers inside the
// in-plane support ellipse).  The weight factorises over the axes of the
// patch frame, 2^-Q = 2^-(qk + wv^2) 2^-(wu^2), so a candidate costs one
// product; rows and columns outside the patch get the factor 0, and
// 2^-Q - 2^-K2 is clamped at 0 outside the support (every value lies in
// [-1, 1], so the clamp to [0, 1] is exact).
template <typename T, typename GEO, typename V2, int HU, int HV, bool DEN>
__device__ __forceinline__ void adj_patch(const GEO &g, const PatchDev &pt, double pu, double pv,
                                          T qk, const V2 *__restrict__ rq, T &sn, T &sd) {
  const double rud = rint(pu), rvd = rint(pv);
  const int ru = (int)rud - pt.x0, rv = (int)rvd - pt.y0;  // patch-local nearest pixel
  const T fu = (T)(pu - rud), fv = (T)(pv - rvd);
  const T cu = (T)g.cu, cv = (T)g.cv, cut = (T)g.cut;
  T U[2 * HU + 1], E[2 * HV + 1];
#pragma unroll
  for (int a = -HU; a <= HU; ++a) {
    const T wu = ((T)a - fu) * cu;
    const bool in = (unsigned)(ru + a) < (unsigned)pt.w;
    U[a + HU] = in ? fast_exp2<T>(-wu * wu) : (T)0;
  }
#pragma unroll
  for (int b = -HV; b <= HV; ++b) {
    const T wv = ((T)b - fv) * cv;
    const bool in = (unsigned)(rv + b) < (unsigned)pt.h;
    E[b + HV] = in ? fast_exp2<T>(-fma(wv, wv, qk)) : (T)0;
  }
  const __amdgpu_buffer_rsrc_t r = Rq<T>::view(rq, pt);
  const int pitch = Rq<T>::pitch(pt.w), row_bytes = pitch * (int)sizeof(V2);
  int off = ((rv - HV) * pitch + (ru - HU) + Rq<T>::lead) * (int)sizeof(V2);
#pragma unroll
  for (int b = 0; b < 2 * HV + 1; ++b) {
#pragma unroll
    for (int a = 0; a < 2 * HU + 1; ++a) {
      const T gh = fma_clamp0<T>(E[b], U[a], cut);
      const V2 q = load_rq<V2>(r, off + a * (int)sizeof(V2));
      sn = fma(gh, q.x, sn);
      if (DEN) sd = fma(gh, q.y, sd);
    }
    off += row_bytes;
  }
}

// Candidate grids wider than the unrolled shapes (PSF much wider than a
// pixel): the same arithmetic with run-time half-widths, one exponential
// per candidate.
template <typename T, typename GEO, typename V2, bool DEN>
__device__ __forceinline__ void adj_patch_rt(const GEO &g, const PatchDev &pt, double pu, double pv,
                                             T qk, const V2 *__restrict__ rq, T &sn, T &sd) {
  const int hu = g.hu, hv = g.hv;
  const double rud = rint(pu), rvd = rint(pv);
  const int ru = (int)rud - pt.x0, rv = (int)rvd - pt.y0;
  const T fu = (T)(pu - rud), fv = (T)(pv - rvd);
  const T cu = (T)g.cu, cv = (T)g.cv, cut = (T)g.cut;
  const __amdgpu_buffer_rsrc_t r = Rq<T>::view(rq, pt);
  const int pitch = Rq<T>::pitch(pt.w);
  for (int b = -hv; b <= hv; ++b) {
    const T wv = ((T)b - fv) * cv;
    const T qkv = fma(wv, wv, qk);
    const int row = (rv + b) * pitch;
    for (int a = -hu; a <= hu; ++a) {
      const T wu = ((T)a - fu) * cu;
      const bool in = ((unsigned)(ru + a) < (unsigned)pt.w) & ((unsigned)(rv + b) < (unsigned)pt.h);
      const T gh = in ? fma_clamp0<T>(fast_exp2<T>(-fma(wu, wu, qkv)), (T)1, cut) : (T)0;
      const V2 q = load_rq<V2>(r, (row + ru + a + Rq<T>::lead) * (int)sizeof(V2));
      sn = fma(gh, q.x, sn);
      if (DEN) sd = fma(gh, q.y, sd);
    }
  }
}

// The sinc PSF (PVR_PSF_SINC): the weight factorises over the patch frame as
// s(t_u) s(t_v) g(t_n) with t = pixel offset * (spacing / first zero) in-plane
// and g = 2^-qk - 2^-K2 (clamped at 0) through-plane; candidates outside the
// main lobe (|t| >= 1) or the patch get the factor 0.  HU, HV > 0: the
// candidate half-widths every patch fits; 0 reads them per patch.
template <typename T, typename GEO, typename V2, int HU, int HV, bool DEN>
__device__ __forceinline__ void adj_patch_sinc(const GEO &g, const PatchDev &pt, double pu,
                                               double pv, T qk, const V2 *__restrict__ rq, T &sn,
                                               T &sd) {
  const int hu = HU > 0 ? HU : g.hu, hv = HV > 0 ? HV : g.hv;
  const double rud = rint(pu), rvd = rint(pv);
  const int ru = (int)rud - pt.x0, rv = (int)rvd - pt.y0;
  const T fu = (T)(pu - rud), fv = (T)(pv - rvd);
  const T cu = (T)g.cu, cv = (T)g.cv, cut = (T)g.cut;
  T gz = fast_exp2<T>(-qk) - cut;
  gz = gz > (T)0 ? gz : (T)0;
  const __amdgpu_buffer_rsrc_t r = Rq<T>::view(rq, pt);
  const int pitch = Rq<T>::pitch(pt.w);
  for (int b = -hv; b <= hv; ++b) {
    const T tv = ((T)b - fv) * cv;
    const T e = (unsigned)(rv + b) < (unsigned)pt.h ? sinc_lobe<T>(tv) * gz : (T)0;
    const int row = (rv + b) * pitch;
    for (int a = -hu; a <= hu; ++a) {
      const T tu = ((T)a - fu) * cu;
      const T gh = (unsigned)(ru + a) < (unsigned)pt.w ? sinc_lobe<T>(tu) * e : (T)0;
      const V2 q = load_rq<V2>(r, (row + ru + a + Rq<T>::lead) * (int)sizeof(V2));
      sn = fma(gh, q.x, sn);
      if (DEN) sd = fma(gh, q.y, sd);
    }
  }
}

// One workgroup = one 8^3 brick; each wavefront owns one 4^3 sub-brick and
// walks that sub-brick's patch list (wave-uniform), one voxel per lane.
// HW: the candidate half-width every patch of the plan fits (1 or 2, fixed
// at compile time), or 0 to read it per patch.
template <typename T, bool DEN, int HW, bool SINC>
__global__ void __launch_bounds__(BP_THREADS)
k_backproject(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
              const typename GeoOf<T>::type *__restrict__ geo, const int *__restrict__ brick_prob,
              const int *__restrict__ sub_off, const int *__restrict__ sub_patch,
              const typename Vec2Of<T>::type *__restrict__ rq, const T *__restrict__ patch_w,
              T *__restrict__ num, T *__restrict__ den, int n_bricks, int granule) {
  using GEO = typename GeoOf<T>::type;
  using V2 = typename Vec2Of<T>::type;
  const int bi = xcd_work(blockIdx.x, granule);
  if (bi >= n_bricks) return;
  const ProbDev pr = probs[brick_prob[bi]];
  const int local = bi - pr.brick_base;
  const int bx = local % pr.nbx, by = (local / pr.nbx) % pr.nby, bz = local / (pr.nbx * pr.nby);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63;
  const int i = bx * BRICK + (w & 1) * SUB + (l & 3);
  const int jj = by * BRICK + ((w >> 1) & 1) * SUB + ((l >> 2) & 3);
  const int kk = bz * BRICK + (w >> 2) * SUB + (l >> 4);
  const bool inside = i < pr.nx && jj < pr.ny && kk < pr.nz;
  T sn = 0, sd = 0;
  const int sbi = bi * 9 + w;
  const int q0 = sub_off[sbi], q1 = sub_off[sbi + 1];
  const double fi = i, fj = jj, fk = kk;
  for (int q = q0; q < q1; ++q) {
    const int s = sub_patch[q];
    // the patch weight scales the patch's whole contribution; an excluded
    // patch (weight 0) is skipped
    const T ws = patch_w ? patch_w[s] : (T)1;
    if (ws == (T)0) continue;
    const GEO &g = geo[s];
    const PatchDev pt = patches[s];
    const double pk = fma(g.G[8], fi, fma(g.G[9], fj, fma(g.G[10], fk, g.G[11])));
    const T wk = (T)(pk - (double)pt.slice) * (T)g.ck;
    const T qk = wk * wk;
    if (!(qk <= (T)g.K2)) continue;
    const double pu = fma(g.G[0], fi, fma(g.G[1], fj, fma(g.G[2], fk, g.G[3])));
    const double pv = fma(g.G[4], fi, fma(g.G[5], fj, fma(g.G[6], fk, g.G[7])));
    T pn = 0, pd = 0;
    if (SINC)
      adj_patch_sinc<T, GEO, V2, HW, HW, DEN>(g, pt, pu, pv, qk, rq, pn, pd);
    else if (HW == 1)
      adj_patch<T, GEO, V2, 1, 1, DEN>(g, pt, pu, pv, qk, rq, pn, pd);
    else if (HW == 2)
      adj_patch<T, GEO, V2, 2, 2, DEN>(g, pt, pu, pv, qk, rq, pn, pd);
    else
      adj_patch_rt<T, GEO, V2, DEN>(g, pt, pu, pv, qk, rq, pn, pd);
    sn = fma(ws, pn, sn);
    if (DEN) sd = fma(ws, pd, sd);
  }
  if (inside) {
    const long long idx = pr.vol_off + ((long long)kk * pr.ny + jj) * pr.nx + i;
    num[idx] = sn;
    if (DEN) den[idx] = sd;
  }
}

// ---------------------------------------------------------------------------
// Block gather: each lane owns the 2 x 2 voxels (along the patch's in-plane
// axes) of one layer along its normal axis, a wavefront 8 x 8 x 4 voxels, a
// workgroup of two wavefronts one 8^3 brick.  See AdjPatch for the voxels'
// forced nearest pixels.  The four voxels share
//  * the 4 x 4 pixel window, 16 bytes per load (8 loads for four voxels instead
//    of 6 per voxel: the per-voxel gather kept the vector-memory path 80-90 %
//    busy);
//  * the FP64 voxel -> pixel map, taken once at the block's centre;
//  * with the Gaussian, the factors 2^-(c (a - f))^2 of the six candidate rows
//    and columns: a voxel's own deviation d enters as 2^(2 c^2 a d), a constant
//    of the patch, and one exponential per voxel that also holds its
//    through-plane term (10 exponentials instead of 24).
// About 70 vector issue slots per voxel and patch instead of 111: the kernel is
// bound by vector issue.  256^3 benchmark, 11 760 patches: 2.27 ms per launch with
// the per-voxel gather, 1.31 ms with this one.  The
// patches of a brick are taken normal axis by normal axis (lists of
// k_adj_lists), so that the two wavefronts' voxels are disjoint; between axes
// the sums move through LDS.  The order (axis, then patch, then candidate) is
// fixed: the result is bitwise repeatable.
//
// A voxel's three rows and columns of the shared window may hold a sample that its
// own nearest pixel's do not, weighed by zero, and zero times a value that is not
// finite is NaN: where the inputs hold one (k_bp_prep left its number, `call`, in *odd),
// every patch goes voxel by voxel.
//
// A brick's lists are split over `parts` pairs of wavefronts (entry q to part
// (q - q0) mod parts, each part with its own LDS sums, added in part order at
// the end), so that a small grid still fills the chip: gather_parts.
constexpr int GB_THREADS = 128;  // of one part
template <typename T> constexpr int GB_MAX_PARTS = sizeof(T) == 4 ? 8 : 4;  // registers

// Measured, whole passes in us with 1 / 2 / 4 / 8 parts: build and first volume at
// 160^3 (16 000 wavefronts at one part) 766 / 743 / 767 / 952; SR iteration at 128^3,
// sinc PSF (8 192) 696 / 674 / 718 / 805; gradients at 96^3 (3 456) 494 / - / 448 /
// 484; SR iteration at 32^3 (128) 198 / - / - / 142.  A workgroup of 8 parts waits for
// 16 free wavefront slots of one CU, so it pays only where a CU has one
// workgroup at most, below 256 bricks (56^3, 343 bricks: 28.9 us a call with 8 parts,
// 24.4 with 4).
static int gather_parts(int n_bricks, int most) {
  int parts = 1;
  while (parts < most && 2LL * n_bricks * parts < (parts < 4 ? 16384 : 2048)) parts *= 2;
  return parts;
}

template <typename T, bool DEN> struct GbAcc;
template <typename T> struct GbAcc<T, true> { T n, d; };
template <typename T> struct GbAcc<T, false> { T n; };

// The 4 x 4 window whose first column and row are the patch-local pixel
// (u0, v0); in: the window meets the patch.  Pixels outside the patch read 0.
__device__ __forceinline__ void load_window(const AdjPatch<float> &g, const float2 *__restrict__ rq,
                                            int u0, int v0, bool in, float2 q[4][4]) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const int pitch = rq_pitch(g.w);
  const __amdgpu_buffer_rsrc_t r =
      raw_buffer(rq + g.rq_off, (unsigned)rq_entries(g.w, g.h) * (unsigned)sizeof(float2));
  int off = in ? (v0 * pitch + u0 + RQ_PAD) * (int)sizeof(float2) : -64;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    // a row before the patch gives a negative offset, out of range as unsigned
    const f4 x = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    const f4 y = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off + 16, 0, 0));
    q[b][0] = make_float2(x.x, x.y);
    q[b][1] = make_float2(x.z, x.w);
    q[b][2] = make_float2(y.x, y.y);
    q[b][3] = make_float2(y.z, y.w);
    off += pitch * (int)sizeof(float2);
  }
}
__device__ __forceinline__ void load_window(const AdjPatch<double> &g, const double2 *__restrict__ rq,
                                            int u0, int v0, bool in, double2 q[4][4]) {
  const __amdgpu_buffer_rsrc_t r =
      raw_buffer(rq + g.rq_off, (unsigned)(g.w * g.h) * (unsigned)sizeof(double2));
  int off[4];  // packed rows: a column outside the patch reads past the view
#pragma unroll
  for (int a = 0; a < 4; ++a)
    off[a] = in && (unsigned)(u0 + a) < (unsigned)g.w ? (v0 * g.w + u0 + a) * (int)sizeof(double2)
                                                      : 0x70000000;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      q[b][a] = __builtin_bit_cast(
          double2, __builtin_amdgcn_raw_buffer_load_b128(r, off[a] + b * g.w * (int)sizeof(double2), 0, 0));
}

// Rounds x (|x| < 2^51) to the nearest integer, ties to even; returns it and
// its value as a double (the low word of x + 1.5 2^52 holds the integer).
__device__ __forceinline__ int round_split(double x, double &r) {
  const double m = x + 6755399441055744.0;
  r = m - 6755399441055744.0;
  return (int)(__builtin_bit_cast(long long, m) & 0xffffffffll);
}

template <typename T, bool DEN, bool SINC>
__global__ void __launch_bounds__(GB_THREADS * GB_MAX_PARTS<T>)
k_gather_blocks(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
                const typename GeoOf<T>::type *__restrict__ geo,
                const AdjPatch<T> *__restrict__ adj, const int *__restrict__ brick_prob,
                const int *__restrict__ off, const int *__restrict__ list,
                const typename Vec2Of<T>::type *__restrict__ rq, const T *__restrict__ patch_w,
                T *__restrict__ num, T *__restrict__ den, int n_bricks, int granule,
                const unsigned *__restrict__ odd, unsigned call) {
  using GEO = typename GeoOf<T>::type;
  using V2 = typename Vec2Of<T>::type;
  using Acc = GbAcc<T, DEN>;
  constexpr int NV = BRICK * BRICK * BRICK;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int may_fast = *odd == call ? 0 : ADJ_FAST;
  const int bi = xcd_work(blockIdx.x, granule);
  if (bi >= n_bricks) return;
  const ProbDev pr = probs[brick_prob[bi]];
  const int local = bi - pr.brick_base;
  const int bx = local % pr.nbx, by = (local / pr.nbx) % pr.nby, bz = local / (pr.nbx * pr.nby);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = wave & 1, part = wave >> 1, parts = blockDim.x / GB_THREADS;
  const int l = threadIdx.x & 63;
  const int lp = l & 3, lq = (l >> 2) & 3, ln = l >> 4;
  Acc *const acc = reinterpret_cast<Acc *>(lds) + part * NV;
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q * GB_THREADS + (threadIdx.x & (GB_THREADS - 1))] = Acc{};
  T sn[4], sd[4];  // sub-window (ou, ov) at 2 ov + ou
  for (int an = 0; an < 3; ++an) {
    __syncthreads();
    const int li = bi * 7 + 2 * an + w;
    const int q0 = off[li] + part, q1 = off[li + 1];
    int cur = -1;
    double xu = 0, xv = 0, xn = 0;  // the block's centre along (au, av, an)
#pragma unroll
    for (int t = 0; t < 4; ++t) sn[t] = sd[t] = (T)0;
    // adds the lane's sums of the class `cur` to its voxels and clears them
    auto flush = [&]() {
      const int au = cur & 3, av = (cur >> 2) & 3;
      const int tu = au == 0 ? 1 : au == 1 ? BRICK : BRICK * BRICK;
      const int tv = av == 0 ? 1 : av == 1 ? BRICK : BRICK * BRICK;
      const int tn = an == 0 ? 1 : an == 1 ? BRICK : BRICK * BRICK;
      // a lane's voxels: 2 x 2 side by side, or (off the fast path) one of each 4^3
      const int lane_step = cur & ADJ_OFF ? 1 : 2, own_step = cur & ADJ_OFF ? SUB : 1;
      const int base = lane_step * (lp * tu + lq * tv) + (SUB * w + ln) * tn;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int du = (t & 1) ^ ((cur >> 4) & 1), dv = (t >> 1) ^ ((cur >> 5) & 1);
        Acc &o = acc[base + own_step * (du * tu + dv * tv)];
        o.n += sn[t];
        if constexpr (DEN) o.d += sd[t];
        sn[t] = sd[t] = (T)0;
      }
    };
    for (int q = q0; q < q1; q += parts) {
      const int s = list[q];
      // the patch weight scales the patch's whole contribution; an excluded
      // patch (weight 0) is skipped
      const T ws = patch_w ? patch_w[s] : (T)1;
      if (ws == (T)0) continue;
      const AdjPatch<T> &g = adj[s];
      const bool fast = g.cls & may_fast;
      const int cls = fast ? g.cls & ADJ_MAP : (an == 0 ? 1 : 0) | (an == 2 ? 1 : 2) << 2 | ADJ_OFF;
      if (cls != cur) {  // (uniform; the patches of a stack share their class)
        if (cur >= 0) flush();
        cur = cls;
        const int au = cls & 3, av = (cls >> 2) & 3;
        xu = sel3(au, bx, by, bz) * BRICK + 2 * lp + 0.5;
        xv = sel3(av, bx, by, bz) * BRICK + 2 * lq + 0.5;
        xn = sel3(an, bx, by, bz) * BRICK + SUB * w + ln;
      }
      if (fast) {
        const T wk = (T)fma(g.Gk[0], xu, fma(g.Gk[1], xv, fma(g.Gk[2], xn, g.Gk[3])));
        const double pu = fma(g.Gu[0], xu, fma(g.Gu[1], xv, fma(g.Gu[2], xn, g.Gu[3])));
        const double pv = fma(g.Gv[0], xu, fma(g.Gv[1], xv, fma(g.Gv[2], xn, g.Gv[3])));
        double rud, rvd;
        const int ru = round_split(pu, rud), rv = round_split(pv, rvd);
        const T f = (T)(pu - rud), h = (T)(pv - rvd);
        // through-plane offsets of the four voxels, and the lanes with none
        // inside the support or off the patch
        const T wt[4] = {wk - g.dk11, wk + g.dk10, wk - g.dk10, wk + g.dk11};
        const T reach = fmin(fmin(wt[0] * wt[0], wt[1] * wt[1]), fmin(wt[2] * wt[2], wt[3] * wt[3]));
        const bool in = reach <= g.K2 && (unsigned)(ru + 2) <= (unsigned)(g.w + 2) &&
                        (unsigned)(rv + 2) <= (unsigned)(g.h + 2);
        if (!__any(in)) continue;
        V2 x[4][4];
        load_window(g, rq, ru - 1, rv - 1, in, x);
        const T cut = g.cut;
        T U[4][3], E[4][3];  // column and row factors of the four voxels
        if constexpr (SINC) {
          const T du[4] = {-g.P11, g.P10, -g.P10, g.P11}, dv[4] = {-g.Q11, g.Q10, -g.Q10, g.Q11};
          // pixels -1, 0, 1 of an axis, from 0 at distance d: the lobe holds 0 and the
          // one on the point's side, and the other only where it reaches over a pixel:
          // two lobes an axis instead of three, and the products summed row by row:
          // 217 -> 205 us at 128^3, 406 -> 381 at 160^3 (held to six wavefronts a SIMD, with
          // spills, 205 and 394)
          const bool wide = g.cu < (T)1 || g.cv < (T)1;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const T gz = fmax(fast_exp2<T>(-wt[t] * wt[t]) - cut, (T)0);
            const T pu = f + du[t], pv = h + dv[t], au = fabs(pu), av = fabs(pv);
            const T su = sinc_lobe<T>(((T)1 - au) * g.cu), sv = sinc_lobe<T>(((T)1 - av) * g.cv) * gz;
            T ou = (T)0, ov = (T)0;
            if (wide) {
              ou = sinc_lobe<T>(((T)1 + au) * g.cu);
              ov = sinc_lobe<T>(((T)1 + av) * g.cv) * gz;
            }
            U[t][0] = pu < (T)0 ? su : ou;
            U[t][1] = sinc_lobe<T>(pu * g.cu);
            U[t][2] = pu < (T)0 ? ou : su;
            E[t][0] = pv < (T)0 ? sv : ov;
            E[t][1] = sinc_lobe<T>(pv * g.cv) * gz;
            E[t][2] = pv < (T)0 ? ov : sv;
          }
        } else {
          const T fu = f * g.cu, hv = h * g.cv;
          T B[3], C[3];
#pragma unroll
          for (int a = -1; a <= 1; ++a) {
            const T yu = (T)a * g.cu - fu, yv = (T)a * g.cv - hv;
            B[a + 1] = fast_exp2<T>(-yu * yu);
            C[a + 1] = fast_exp2<T>(-yv * yv);
          }
          const T P[4] = {-g.P11, g.P10, -g.P10, g.P11}, Q[4] = {-g.Q11, g.Q10, -g.Q10, g.Q11};
          const T R[4] = {g.R11, g.R10, g.R10, g.R11};
          const T ku[4] = {g.ki11, g.ku10, g.ki10, g.ku11}, ki[4] = {g.ku11, g.ki10, g.ku10, g.ki11};
          const T kv[4] = {g.ji11, g.kv10, g.ji10, g.kv11}, ji[4] = {g.kv11, g.ji10, g.kv10, g.ji11};
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const T S = fast_exp2<T>(-fma(wt[t], wt[t], fma(f, P[t], fma(h, Q[t], R[t]))));
            U[t][0] = B[0] * ki[t];
            U[t][1] = B[1];
            U[t][2] = B[2] * ku[t];
            E[t][0] = (C[0] * ji[t]) * S;
            E[t][1] = C[1] * S;
            E[t][2] = (C[2] * kv[t]) * S;
          }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int ou = t & 1, ov = t >> 1;
          T pn = 0, pd = 0;
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            T rn = 0, rd = 0;  // the sinc's weights are products: sum row by row
#pragma unroll
            for (int a = 0; a < 3; ++a) {
              const T gh = SINC ? U[t][a] : fma_clamp0<T>(E[t][b], U[t][a], cut);
              const V2 &e = x[ov + b][ou + a];
              T &n = SINC ? rn : pn, &d = SINC ? rd : pd;
              n = fma(gh, e.x, n);
              if (DEN) d = fma(gh, e.y, d);
            }
            if (SINC) {
              pn = fma(E[t][b], rn, pn);
              if (DEN) pd = fma(E[t][b], rd, pd);
            }
          }
          if (in && wt[t] * wt[t] <= g.K2) {  // outside, a non-finite input stays out
            sn[t] = fma(ws, pn, sn[t]);
            if (DEN) sd[t] = fma(ws, pd, sd[t]);
          }
        }
      } else {
        // deviations too large for shared windows: voxel by voxel, a 4^3 sub-brick at
        // a time, where the patch reaches it (192^3, 37 x 37 patches, all turned by 60
        // degrees: 1540 us; 2041 with the lane's 2 x 2 voxels in turn, which spread every
        // step over the whole half brick)
        const GEO &ge = geo[s];
        const PatchDev pt = patches[s];
        const int au = cls & 3, av = (cls >> 2) & 3;
#pragma unroll 1
        for (int t = 0; t < 4; ++t) {
          const int vu = sel3(au, bx, by, bz) * BRICK + SUB * (t & 1) + lp;
          const int vv = sel3(av, bx, by, bz) * BRICK + SUB * (t >> 1) + lq;
          const int vn = sel3(an, bx, by, bz) * BRICK + SUB * w + ln;
          const double fi = au == 0 ? vu : av == 0 ? vv : vn, fj = au == 1 ? vu : av == 1 ? vv : vn,
                       fk = au == 2 ? vu : av == 2 ? vv : vn;
          const double pk = fma(ge.G[8], fi, fma(ge.G[9], fj, fma(ge.G[10], fk, ge.G[11])));
          const T wk = (T)(pk - (double)pt.slice) * (T)ge.ck;
          const T qk = wk * wk;
          const double pu = fma(ge.G[0], fi, fma(ge.G[1], fj, fma(ge.G[2], fk, ge.G[3])));
          const double pv = fma(ge.G[4], fi, fma(ge.G[5], fj, fma(ge.G[6], fk, ge.G[7])));
          // (candidates reach one pixel from the nearest one)
          if (!(qk <= (T)ge.K2 && fabs(pu - (pt.x0 + 0.5 * (pt.w - 1))) <= 0.5 * pt.w + 1.0 &&
                fabs(pv - (pt.y0 + 0.5 * (pt.h - 1))) <= 0.5 * pt.h + 1.0))
            continue;
          T pn = 0, pd = 0;
          if (SINC) adj_patch_sinc<T, GEO, V2, 1, 1, DEN>(ge, pt, pu, pv, qk, rq, pn, pd);
          else adj_patch<T, GEO, V2, 1, 1, DEN>(ge, pt, pu, pv, qk, rq, pn, pd);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            sn[k] = k == t ? fma(ws, pn, sn[k]) : sn[k];
            if (DEN) sd[k] = k == t ? fma(ws, pd, sd[k]) : sd[k];
          }
        }
      }
    }
    if (cur >= 0) flush();
  }
  __syncthreads();
  for (int v = threadIdx.x; v < NV; v += blockDim.x) {
    Acc r = reinterpret_cast<Acc *>(lds)[v];
    for (int q = 1; q < parts; ++q) {
      const Acc &o = reinterpret_cast<Acc *>(lds)[q * NV + v];
      r.n += o.n;
      if constexpr (DEN) r.d += o.d;
    }
    const int i = bx * BRICK + (v & 7), jj = by * BRICK + ((v >> 3) & 7), kk = bz * BRICK + (v >> 6);
    if (i < pr.nx && jj < pr.ny && kk < pr.nz) {
      const long long idx = pr.vol_off + ((long long)kk * pr.ny + jj) * pr.nx + i;
      num[idx] = r.n;
      if constexpr (DEN) den[idx] = r.d;
    }
  }
}

// The preparation pass.  Each has a number of its own, so that what an earlier one left
// in d_odd says nothing of this one; a captured one keeps its number from replay to
// replay and clears the place first.
template <typename T>
static pvr_status prepare(const pvr_plan *p, const T *invz, const T *e, const T *pp,
                          typename Vec2Of<T>::type *rq, hipStream_t stream) {
  const int f64 = sizeof(T) == 8;
  unsigned &call = const_cast<pvr_plan *>(p)->odd_call[f64];
  if (++call == 0) call = 1;
  if (capture_id(stream)) launch_fill_i32((int *)p->d_odd + f64, 0, 1, stream);
  hipLaunchKernelGGL(k_bp_prep<T>, dim3(p->n_sim_blocks), dim3(SIM_THREADS), 0, stream, p->d_patch,
                     p->d_sim_blocks, invz, e, pp, rq, p->d_odd + f64, call);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
}

// On its own (FP32), for pvr_robust_weights.
pvr_status pvr::launch_bp_prep(const pvr_plan *p, const float *e, const float *pp,
                               hipStream_t stream) {
  return prepare<float>(p, p->d_invz, e, pp, p->d_rq, stream);
}

template <typename T>
static pvr_status backproject_impl(const pvr_plan *p, const T *e, const T *pp, const T *patch_w,
                                   T *num, T *den, const T *invz, typename Vec2Of<T>::type *rq,
                                   hipStream_t stream) {
  if (!e || !num) return fail(PVR_EINVAL, "pvr_backproject: e and num are required");
  const int f64 = sizeof(T) == 8;
  const unsigned long long capture = capture_id(stream);
  if (!p->index_valid || (p->index_capture && p->index_capture != capture)) {
    const pvr_status st = plan_build_index(const_cast<pvr_plan *>(p), stream);
    if (st != PVR_OK) return st;
  }
  // the preparation pass, unless pvr_robust_weights (PVR_EM_PREP_ADJOINT)
  // already ran it for these residuals and posteriors (in this capture, if any)
  const bool prepared = sizeof(T) == 4 && p->rq_fresh && p->rq_e == (const void *)e &&
                        p->rq_p == (const void *)pp && p->rq_capture == capture;
  if (!prepared) {
    if (sizeof(T) == 4) const_cast<pvr_plan *>(p)->rq_fresh = false;  // d_rq changes
    const pvr_status st = prepare<T>(p, invz, e, pp, rq, stream);
    if (st != PVR_OK) return st;
  }
  const void *geo = sizeof(T) == 4 ? (const void *)p->d_geof : (const void *)p->d_geod;
  const dim3 grid(xcd_blocks(p->n_bricks, p->bp_granule));
  hipEvent_t *ev = timing_slot(p, PVR_KERNEL_BACKPROJECT);
  if (ev) HIP_TRY(hipEventRecord(ev[0], stream));
  const int hw = (p->max_hu <= 1 && p->max_hv <= 1) ? 1 : (p->max_hu <= 2 && p->max_hv <= 2) ? 2 : 0;
  const auto *geot = (const typename GeoOf<T>::type *)geo;
#define BP_LAUNCH(D, H, SC)                                                                     \
  hipLaunchKernelGGL((k_backproject<T, D, H, SC>), grid, dim3(BP_THREADS), 0, stream, p->d_prob, \
                     p->d_patch, geot, p->d_brick_prob, p->d_sub_off, p->d_sub_patch, rq,         \
                     patch_w, num, den, p->n_bricks, p->bp_granule)
#define BP_LAUNCH_HW(D, SC)            \
  if (hw == 1) BP_LAUNCH(D, 1, SC);    \
  else if (hw == 2) BP_LAUNCH(D, 2, SC); \
  else BP_LAUNCH(D, 0, SC)
  const bool sinc = p->psf == PVR_PSF_SINC;
  if (p->gather_blocks) {
    const void *adj = sizeof(T) == 4 ? (const void *)p->d_adj : (const void *)p->d_adj64;
    const int parts = gather_parts(p->n_bricks, GB_MAX_PARTS<T>);
#define GB_LAUNCH(D, SC)                                                                          \
  hipLaunchKernelGGL((k_gather_blocks<T, D, SC>), grid, dim3(GB_THREADS * parts),                 \
                     sizeof(GbAcc<T, D>) * BRICK * BRICK * BRICK * parts, stream, p->d_prob,      \
                     p->d_patch, geot, (const AdjPatch<T> *)adj, p->d_brick_prob, p->d_sub_off,   \
                     p->d_sub_patch, rq, patch_w, num, den, p->n_bricks, p->bp_granule, \
                     p->d_odd + f64, p->odd_call[f64])
    if (den) {
      if (sinc) GB_LAUNCH(true, true);
      else GB_LAUNCH(true, false);
    } else {
      if (sinc) GB_LAUNCH(false, true);
      else GB_LAUNCH(false, false);
    }
#undef GB_LAUNCH
  } else if (den) {
    if (sinc) { BP_LAUNCH_HW(true, true); }
    else { BP_LAUNCH_HW(true, false); }
  } else {
    if (sinc) { BP_LAUNCH_HW(false, true); }
    else { BP_LAUNCH_HW(false, false); }
  }
#undef BP_LAUNCH_HW
#undef BP_LAUNCH
  HIP_TRY(hipGetLastError());
  if (ev) HIP_TRY(hipEventRecord(ev[1], stream));
  return PVR_OK;
}

extern "C" pvr_status pvr_backproject(const pvr_plan *p, const float *e, const float *pp,
                                      const float *patch_w, float *num, float *den,
                                      hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_backproject", e, 4);
  PVR_ALIGNED("pvr_backproject", pp, 4);
  PVR_ALIGNED("pvr_backproject", patch_w, 4);
  PVR_ALIGNED("pvr_backproject", num, 4);
  PVR_ALIGNED("pvr_backproject", den, 4);
  if (!p) return fail(PVR_EINVAL, "pvr_backproject: plan is NULL");
  if (!p->built) return fail(PVR_EINVAL, "pvr_backproject: plan has not been built");
  PVR_TRY_STATUS(debug_finite(p, "pvr_backproject", "e", e, p->N, stream));
  PVR_TRY_STATUS(debug_finite(p, "pvr_backproject", "p", pp, p->N, stream));
  PVR_TRY_STATUS(debug_weights(p, "pvr_backproject", "patch_w", patch_w, p->M, stream));
  return backproject_impl<float>(p, e, pp, patch_w, num, den, p->d_invz, p->d_rq, stream);
  PVR_API_END();
}

extern "C" pvr_status pvr_backproject_f64(const pvr_plan *p, const double *e, const double *pp,
                                          const double *patch_w, double *num, double *den,
                                          hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_backproject_f64", e, 8);
  PVR_ALIGNED("pvr_backproject_f64", pp, 8);
  PVR_ALIGNED("pvr_backproject_f64", patch_w, 8);
  PVR_ALIGNED("pvr_backproject_f64", num, 8);
  PVR_ALIGNED("pvr_backproject_f64", den, 8);
  if (!p) return fail(PVR_EINVAL, "pvr_backproject_f64: plan is NULL");
  if (!p->built || !p->built64)
    return fail(PVR_EINVAL, "pvr_backproject_f64: plan needs pvr_plan_build_f64 on a workspace "
                            "attached with PVR_WS_F64");
  PVR_TRY_STATUS(debug_finite(p, "pvr_backproject_f64", "e", e, p->N, stream));
  PVR_TRY_STATUS(debug_finite(p, "pvr_backproject_f64", "p", pp, p->N, stream));
  PVR_TRY_STATUS(debug_weights(p, "pvr_backproject_f64", "patch_w", patch_w, p->M, stream));
  return backproject_impl<double>(p, e, pp, patch_w, num, den, p->d_invz64, p->d_rq64 + 1, stream);
  PVR_API_END();
}
