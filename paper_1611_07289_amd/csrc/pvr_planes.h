// Plane walk of the Gaussian PSF ("volume-pixel" direction): a lane takes the
// 2 x 2 samples of one pixel block and walks the voxel planes across their
// supports along the voxel axis c nearest the patch's normal; in a plane the
// four samples share one window of voxels.
//
// With the quadratic form conditioned on c (t_a, t_b the slope of the
// conditional centre, S_cc the Schur complement),
//   Q = S_cc (c - x_c)^2 + q(a - p_a, b - p_b),  p = x + t (c - x_c),
// q the 2 x 2 in-plane form.  Stepping one pixel along u moves the centre in a
// plane by one voxel along a (the voxel axis u runs along, with sign su) plus
// a small deviation, and v likewise along b: the sample of sub-window (i, j)
// in {0, 1}^2 is centred at (r_a + i + f + d_a, r_b + j + h + d_b) with (r, f),
// (r, h) the rounded block position and its fraction and d the sample's own
// deviation (constants of the patch, antisymmetric about the block's centre).
// Its weight at the voxel (alpha, beta) from its own nearest one is
//   2^-Q = U_alpha V_beta kappa_a^alpha kappa_b^beta 2^(-2 A_ab alpha beta) S,
// U and V exponentials of the lane shared by the four samples, kappa constants
// of the sample, and S one exponential of the sample: 10 exponentials for 36
// weights, no row bounds, and loads of whole window rows.  A patch takes this
// walk when every voxel that can carry weight lies in the window (3 x 3 per
// sample, or 3 x 4 for planes cut at a larger tilt): make_fwd.
#pragma once

#include "pvr_geometry.h"
#include "pvr_internal.h"

namespace pvr {

// Constants of the walk; a, b, c as above, suffix 11 / 10: sub-window (1, 1) /
// (1, 0), the opposite ones having the opposite sign (reciprocal factor).
// ex: the exponents of o.kap, which the caller raises (all zero off the walk).
template <typename T>
__host__ __device__ inline void make_fwd_args(const GeoD &g, const ProbDev &pr, const PatchDev &pt,
                                              FwdPatch<T> &o, double ex[10]) {
  for (int i = 0; i < 10; ++i) ex[i] = 0.0;
  o.rows = 0;
  if (g.psf != PVR_PSF_GAUSSIAN) return;
  int a = 0;
  for (int r = 1; r < 3; ++r) if (fabs(g.H[4 * r]) > fabs(g.H[4 * a])) a = r;
  const int b0 = a == 0 ? 1 : 0, b1 = 3 - a - b0;
  const int b = fabs(g.H[4 * b0 + 1]) >= fabs(g.H[4 * b1 + 1]) ? b0 : b1, c = 3 - a - b;
  const int ax[3] = {a, b, c};
  double A[9];
  const double w2[3] = {g.cu * g.cu, g.cv * g.cv, g.ck * g.ck};
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      A[3 * i + j] = w2[0] * g.G[ax[i]] * g.G[ax[j]] + w2[1] * g.G[4 + ax[i]] * g.G[4 + ax[j]] +
                     w2[2] * g.G[8 + ax[i]] * g.G[8 + ax[j]];
  const double Aaa = A[0], Aab = A[1], Aac = A[2], Abb = A[4], Abc = A[5], Acc = A[8];
  const double idet = 1.0 / (Aaa * Abb - Aab * Aab);
  const double ta = -(Abb * Aac - Aab * Abc) * idet, tb = -(Aaa * Abc - Aab * Aac) * idet;
  const double Scc = Acc + ta * Aac + tb * Abc;
  const double *Ha = g.H + 4 * a, *Hb = g.H + 4 * b, *Hc = g.H + 4 * c;
  const double su = Ha[0] < 0 ? -1.0 : 1.0, sv = Hb[1] < 0 ? -1.0 : 1.0;
  const double Au = su * (Ha[0] - ta * Hc[0]) - 1.0, Av = sv * (Ha[1] - ta * Hc[1]);
  const double Bu = su * (Hb[0] - tb * Hc[0]), Bv = sv * (Hb[1] - tb * Hc[1]) - 1.0;
  const double da11 = 0.5 * (Au + Av), da10 = 0.5 * (Au - Av);
  const double db11 = 0.5 * (Bu + Bv), db10 = 0.5 * (Bu - Bv);
  const double e11 = 0.5 * (su * Hc[0] + sv * Hc[1]), e10 = 0.5 * (su * Hc[0] - sv * Hc[1]);
  const double Ra = sqrt(g.K2 * Abb * idet) + fmax(fabs(da11), fabs(da10));
  const double Rb = sqrt(g.K2 * Aaa * idet) + fmax(fabs(db11), fabs(db10));
  const double Rc = sqrt(g.K2 / Scc) + 0.5 + fmax(fabs(e11), fabs(e10));
  // the voxels of a window row are read together: u must run along the fastest
  // axis of the volume copy the patch reads (FP32; the FP64 walk reads voxel
  // by voxel).  In-plane scales beyond 7 would make the shared exponentials'
  // FP32 rounding larger than the per-voxel form's.  (All comparisons are
  // false for a motion that is not finite.)
  const bool xt = sizeof(T) == 4 && pt.layout == 1;
  const bool ok = Ra < 1.5 - 1e-4 && Rb < 2.0 - 1e-4 && Rc < 32.0 && Aaa <= 7.0 && Abb <= 7.0 &&
                  (sizeof(T) == 8 || a == (xt ? 1 : 0));
  if (!ok) return;
  o.rows = Rb < 1.5 - 1e-4 ? 3 : 4;
  o.half = (int)floor(Rc + 1e-6);
  for (int i = 0; i < 2; ++i) { o.Ha[i] = Ha[i]; o.Hb[i] = Hb[i]; o.Hc[i] = Hc[i]; }
  // block centre: pixel (u, v) + 1/2 of the block's first pixel, patch-local
  for (int r = 0; r < 3; ++r) {
    const double *H = g.H + 4 * ax[r];
    double *t = r == 0 ? o.Ha : r == 1 ? o.Hb : o.Hc;
    t[2] = H[0] * (pt.x0 + 0.5) + H[1] * (pt.y0 + 0.5) + H[2] * pt.slice + H[3];
  }
  o.ta = ta; o.tb = tb;
  o.fta = (T)ta; o.ftb = (T)tb;
  o.Aaa = (T)Aaa; o.Aab2 = (T)(2 * Aab); o.Abb = (T)Abb; o.Scc = (T)Scc; o.cut = (T)g.cut;
  const double ga11 = 2 * (Aaa * da11 + Aab * db11), gb11 = 2 * (Aab * da11 + Abb * db11);
  const double ga10 = 2 * (Aaa * da10 + Aab * db10), gb10 = 2 * (Aab * da10 + Abb * db10);
  o.ga11 = (T)ga11; o.ga10 = (T)ga10; o.gb11 = (T)gb11; o.gb10 = (T)gb10;
  o.D11 = (T)(0.5 * (ga11 * da11 + gb11 * db11));
  o.D10 = (T)(0.5 * (ga10 * da10 + gb10 * db10));
  o.e11 = (T)e11; o.e10 = (T)e10;
  o.da11 = (T)da11; o.da10 = (T)da10; o.db11 = (T)db11; o.db10 = (T)db10;
  const double x[10] = {ga11, -ga11, ga10, -ga10, gb11, -gb11, gb10, -gb10, -2 * Aab, 2 * Aab};
  for (int i = 0; i < 10; ++i) ex[i] = x[i];
  for (int i = 0; i < 3; ++i) o.ax[i] = ax[i];
  const int sx = xt ? pr.ny : 1, sy = xt ? 1 : pr.nx, sz = pr.nx * pr.ny;
  o.st_a = sel3(a, sx, sy, sz); o.st_b = sel3(b, sx, sy, sz); o.st_c = sel3(c, sx, sy, sz);
  o.na = sel3(a, pr.nx, pr.ny, pr.nz); o.nb = sel3(b, pr.nx, pr.ny, pr.nz);
  o.nc = sel3(c, pr.nx, pr.ny, pr.nz);
  o.flip = (su < 0 ? 1 : 0) | (sv < 0 ? 2 : 0);
}

// The pixel block and the share of its planes of a thread: a work item's nb
// blocks (at most PLANE_BLOCKS) take ceil(nb / 64) of the workgroup's four
// wavefronts, and where two or four times as many fit, the others share the
// planes of the same blocks (16-pixel patches at 32^3: 14.9 -> 10.5 us; larger
// workgroups, to split the planes of larger patches too, gained nothing at
// 32^3 and 48^3 and lost 8 % at 96^3).  Part 0 ends with the sums
// (combine_parts).
struct PlaneLane {
  int blk, part, parts, span;
  bool on;  // holds a block
};
__device__ __forceinline__ PlaneLane plane_lane(const PatchDev &pt, int l0) {
  PlaneLane p;
  const int nblk = ((pt.w + 1) / 2) * ((pt.h + 1) / 2);
  const int nb = min(PLANE_BLOCKS, nblk - l0);
  p.span = (nb + 63) & ~63;
  p.parts = (int)blockDim.x / p.span;
  const int thread = threadIdx.x;
  p.part = __builtin_amdgcn_readfirstlane(thread / p.span);
  const int i = thread - p.part * p.span;
  p.blk = l0 + i;
  p.on = i < nb && p.part < p.parts;
  return p;
}
// Adds the parts' sums s[4] in part order into part 0's (all threads of the
// workgroup call; lds: blockDim.x entries of 4 T).
template <typename T>
__device__ __forceinline__ void combine_parts(const PlaneLane &p, T s[4], T (*lds)[4]) {
  if (p.parts == 1) return;  // uniform over the workgroup
#pragma unroll
  for (int t = 0; t < 4; ++t) lds[threadIdx.x][t] = s[t];
  __syncthreads();
  if (p.part == 0) {
    for (int q = 1; q < p.parts; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) s[t] += lds[threadIdx.x + q * p.span][t];
  }
}

// The same work item one sample at a time, for patches off the walk: calls f(u, v)
// for the item's pixels, every thread of the workgroup its share, a wavefront 16
// blocks at a time (two rows of 32 pixels where they lie side by side).  MIXED and
// not all: for the pixels of the lane's own block `blk` that `bits` names (2 j + i).
template <bool MIXED, typename F>
__device__ __forceinline__ void each_pixel(const PatchDev &pt, int l0, bool all, int blk,
                                           unsigned bits, F &&f) {
  const int nbu = (pt.w + 1) / 2, nb = min(PLANE_BLOCKS, nbu * ((pt.h + 1) / 2) - l0);
  const int end = MIXED && !all ? 4 * PLANE_BLOCKS : 4 * ((nb + 15) & ~15);
#pragma unroll 1
  for (int q = threadIdx.x; q < end; q += PLANE_BLOCKS) {
    const int o = (q >> 6) * 16 + ((q & 31) >> 1), i = q / PLANE_BLOCKS;
    const bool mine = MIXED && !all;
    const int b = mine ? blk : l0 + o;
    const int u = 2 * (b % nbu) + ((mine ? i : q) & 1), v = 2 * (b / nbu) + (mine ? i >> 1 : (q >> 5) & 1);
    if (mine ? ((bits >> i) & 1u) != 0 : o < nb && u < pt.w && v < pt.h) f(u, v);
  }
}

template <typename T>
__host__ __device__ inline void make_fwd(const GeoD &g, const ProbDev &pr, const PatchDev &pt, FwdPatch<T> &o) {
  double ex[10];
  make_fwd_args(g, pr, pt, o, ex);
  for (int i = 0; i < 10; ++i) o.kap[i] = (T)exp2(ex[i]);
}

// Nearest integer (ties to even) or floor of a float / double as a value.
template <bool FLOOR> __device__ __forceinline__ float round_val(float x) {
  return FLOOR ? __builtin_floorf(x) : __builtin_rintf(x);
}
template <bool FLOOR> __device__ __forceinline__ double round_val(double x) {
  return FLOOR ? __builtin_floor(x) : __builtin_rint(x);
}

// The window rows: NB + 1 rows of four voxels from (ia, ib) in plane ic.
// A voxel outside the grid reads 0 (inside: the whole window is in the grid).
template <int NB>
__device__ __forceinline__ void load_rows(const FwdPatch<float> &g, __amdgpu_buffer_rsrc_t xr,
                                          unsigned nbytes, int ia, int ib, int ic, bool inside,
                                          float x[NB + 1][4]) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  int off = (ic * g.st_c + ib * g.st_b + ia) * 4;
  const int row = g.st_b * 4;
  if (__all(inside)) {
#pragma unroll
    for (int r = 0; r <= NB; ++r) {
      const f4 v = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
      x[r][0] = v.x; x[r][1] = v.y; x[r][2] = v.z; x[r][3] = v.w;
      off += row;
    }
  } else {
    const bool pc = (unsigned)ic < (unsigned)g.nc;
#pragma unroll
    for (int r = 0; r <= NB; ++r) {
      const bool pr = pc && (unsigned)(ib + r) < (unsigned)g.nb;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool in = pr && (unsigned)(ia + k) < (unsigned)g.na;
        x[r][k] = load_vox<float>(xr, in ? (unsigned)(off + 4 * k) : nbytes);
      }
      off += row;
    }
  }
}
template <int NB>
__device__ __forceinline__ void load_rows(const FwdPatch<double> &g, __amdgpu_buffer_rsrc_t xr,
                                          unsigned nbytes, int ia, int ib, int ic, bool inside,
                                          double x[NB + 1][4]) {
  unsigned off = (unsigned)(ic * g.st_c + ib * g.st_b + ia * g.st_a) * 8u;
  const bool pc = (unsigned)ic < (unsigned)g.nc;
#pragma unroll
  for (int r = 0; r <= NB; ++r) {
    const bool pr = pc && (unsigned)(ib + r) < (unsigned)g.nb;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = inside || (pr && (unsigned)(ia + k) < (unsigned)g.na);
      x[r][k] = load_vox<double>(xr, in ? off + (unsigned)(k * g.st_a) * 8u : nbytes);
    }
    off += (unsigned)g.st_b * 8u;
  }
}

// The walk for the block whose first pixel is (u, v), patch-local: sums
// g_hat X (HAS_X) and g_hat (HAS_Z) over in-grid voxels of the four samples,
// sub-window (i, j) at 2 j + i.  live: the lane's sums are used (a wavefront
// whose live lanes stay inside the grid skips the border handling).  The
// planes part, part + parts, ... are taken (PlaneLane).
template <typename T, int NB, bool HAS_X, bool HAS_Z>
__device__ __forceinline__ void plane_walk(const FwdPatch<T> &g, int u, int v, bool live, int part,
                                           int parts,
                                           __amdgpu_buffer_rsrc_t xr, unsigned nbytes, T y[4], T z[4]) {
  const double du = u, dv = v;
  const double xa = fma(g.Ha[0], du, fma(g.Ha[1], dv, g.Ha[2]));
  const double xb = fma(g.Hb[0], du, fma(g.Hb[1], dv, g.Hb[2]));
  const double xc = fma(g.Hc[0], du, fma(g.Hc[1], dv, g.Hc[2]));
  const double rc = __builtin_rint(xc), dc = rc - xc;
  // block position in the middle plane, minus the half of sub-window (0, 0)
  const double pa = fma(g.ta, dc, xa) - 0.5, pb = fma(g.tb, dc, xb) - 0.5;
  const double ra = __builtin_rint(pa), rb = __builtin_rint(pb);
  const T f0 = (T)(pa - ra), h0 = (T)(pb - rb), z0 = (T)dc;
  const int ia0 = (int)ra - 1, ib0 = (int)rb - 1, ic0 = (int)rc;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (HAS_X) y[t] = (T)0;
    if (HAS_Z) z[t] = (T)0;
  }
  const T ga[4] = {-g.ga11, g.ga10, -g.ga10, g.ga11}, gb[4] = {-g.gb11, g.gb10, -g.gb10, g.gb11};
  const T D[4] = {g.D11, g.D10, g.D10, g.D11}, e[4] = {-g.e11, g.e10, -g.e10, g.e11};
  const T ka[4] = {g.kap[IA11], g.kap[KA10], g.kap[IA10], g.kap[KA11]},
          ja[4] = {g.kap[KA11], g.kap[IA10], g.kap[KA10], g.kap[IA11]},
          kb[4] = {g.kap[IB11], g.kap[KB10], g.kap[IB10], g.kap[KB11]},
          jb[4] = {g.kap[KB11], g.kap[IB10], g.kap[KB10], g.kap[IB11]}, xm = g.kap[XM], xp = g.kap[XP];
  const T cut = g.cut;
#pragma unroll 1
  for (int k = part - g.half; k <= g.half; k += parts) {
    const T kk = (T)k;
    const T qa = fma(kk, g.fta, f0), qb = fma(kk, g.ftb, h0);
    const T sa = round_val<false>(qa), sb = round_val<NB == 4>(qb);
    const T f = qa - sa, h = qb - sb, wz = z0 + kk;
    const int ia = ia0 + (int)sa, ib = ib0 + (int)sb, ic = ic0 + k;
    const bool inside = !live || ((unsigned)ic < (unsigned)g.nc && ia >= 0 && ia + 4 <= g.na &&
                                  ib >= 0 && ib + NB + 1 <= g.nb);
    T x[NB + 1][4];
    if (HAS_X) load_rows<NB>(g, xr, nbytes, ia, ib, ic, inside, x);
    // U_alpha, V_beta: exponents -A (alpha - f)^2 + 2 A_ab alpha h as sums of small terms
    const T m = g.Aab2 * f * h;
    const T ea = -g.Aaa * f * f, eb = -g.Abb * h * h;
    const T sla = fma(g.Aab2, h, (T)2 * g.Aaa * f), slb = fma(g.Aab2, f, (T)2 * g.Abb * h);
    T U[3], V[NB];
    U[0] = fast_exp2<T>(ea - g.Aaa - sla);
    U[1] = fast_exp2<T>(ea);
    U[2] = fast_exp2<T>(ea - g.Aaa + sla);
    V[0] = fast_exp2<T>(eb - g.Abb - slb);
    V[1] = fast_exp2<T>(eb);
    V[2] = fast_exp2<T>(eb - g.Abb + slb);
    if constexpr (NB == 4) V[3] = fast_exp2<T>(fma((T)-4, g.Abb, fma((T)2, slb, eb)));
    if (HAS_Z && !__all(inside)) {
      // voxels outside the grid do not count: window columns and rows are
      // masked per sample below through the factors of their own columns
      const bool pc = (unsigned)ic < (unsigned)g.nc;
      T ca[4], cb[NB + 1];
#pragma unroll
      for (int i = 0; i < 4; ++i) ca[i] = (unsigned)(ia + i) < (unsigned)g.na ? (T)1 : (T)0;
#pragma unroll
      for (int j = 0; j <= NB; ++j) cb[j] = pc && (unsigned)(ib + j) < (unsigned)g.nb ? (T)1 : (T)0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = t & 1, j = t >> 1;
        const T w = wz - e[t];
        const T S = fast_exp2<T>(-fma(g.Scc * w, w, fma(f, ga[t], fma(h, gb[t], D[t] + m))));
        const T Um = U[0] * ja[t] * ca[i], Uc = U[1] * ca[i + 1], Up = U[2] * ka[t] * ca[i + 2];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          T E = V[b] * S * cb[j + b];
          if (b == 0) E *= jb[t];
          if (b == 2) E *= kb[t];
          if (b == 3) E *= kb[t] * kb[t];
          const T Em = b == 0 ? E * xm : b == 1 ? E : b == 2 ? E * xp : E * xp * xp;
          const T Ep = b == 0 ? E * xp : b == 1 ? E : b == 2 ? E * xm : E * xm * xm;
          const T g0 = clamp01<T>(fma(Em, Um, -cut)), g1 = clamp01<T>(fma(E, Uc, -cut)),
                  g2 = clamp01<T>(fma(Ep, Up, -cut));
          z[t] += g0 + g1 + g2;
          if (HAS_X) {
            y[t] = fma(g0, x[j + b][i], y[t]);
            y[t] = fma(g1, x[j + b][i + 1], y[t]);
            y[t] = fma(g2, x[j + b][i + 2], y[t]);
          }
        }
      }
      continue;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = t & 1, j = t >> 1;
      const T w = wz - e[t];
      const T S = fast_exp2<T>(-fma(g.Scc * w, w, fma(f, ga[t], fma(h, gb[t], D[t] + m))));
      const T Um = U[0] * ja[t], Up = U[2] * ka[t];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        T E = V[b] * S;
        if (b == 0) E *= jb[t];
        if (b == 2) E *= kb[t];
        if (b == 3) E *= kb[t] * kb[t];
        const T Em = b == 0 ? E * xm : b == 1 ? E : b == 2 ? E * xp : E * (xp * xp);
        const T Ep = b == 0 ? E * xp : b == 1 ? E : b == 2 ? E * xm : E * (xm * xm);
        const T g0 = clamp01<T>(fma(Em, Um, -cut)), g1 = clamp01<T>(fma(E, U[1], -cut)),
                g2 = clamp01<T>(fma(Ep, Up, -cut));
        if (HAS_Z) z[t] += g0 + g1 + g2;
        if (HAS_X) {
          y[t] = fma(g0, x[j + b][i], y[t]);
          y[t] = fma(g1, x[j + b][i + 1], y[t]);
          y[t] = fma(g2, x[j + b][i + 2], y[t]);
        }
      }
    }
  }
}

// Walk of one sample by planes for the sinc PSF (FP32).  Row by row along the
// longest axis, the walk (psf_walk_sinc) intersects three slabs for every row of
// the support's bounding box, and a wavefront takes as many groups of four as the
// longest of its lanes' rows: about 83 voxels where a support holds 41.  In a
// plane across axis c, nearest the patch's normal, the support is a
// parallelogram |t_u| < 1, |t_v| < 1 around the line t_u = t_v = 0, about two
// voxels wide each way: the four voxels of the cell that holds the line's point
// carry 98 % of all nonzero weights.  A third column or row (the one on the nearer
// side, and their corner) is tested voxel by voxel where the point lies near
// enough to the cell's border, and the voxels inside are taken one by one.
// Bound by vector issue: 25 instructions a voxel, about 150 a plane.  6.3 M samples
// of 37 x 37 patches, whole forward pass: 483 us by rows, 387 here; putting the
// tested voxels off to the end of six planes gained nothing (421 and 419 in an
// earlier form).  The error against 64 bits falls from 2.1e-7 to 1.3e-7, most of it
// by summing plane by plane.  Patches whose parallelogram reaches 3/2 voxels or more,
// whose normal runs along the copy's fastest axis, or which lie so nearly along the
// axes with zeros over a voxel away that the rows cost less (make_sinc), keep the row
// walk, and so does the registration, which compares the values of trials.
__host__ __device__ inline void make_sinc(const GeoD &g, const ProbDev &pr, const PatchDev &pt,
                                          SincPatch &o) {
  o.on = 0;
  if (g.psf != PVR_PSF_SINC) return;
  const double *L = g.L;
  int c = 0;
  for (int r = 1; r < 3; ++r) if (fabs(L[6 + r]) > fabs(L[6 + c])) c = r;
  // the cell's columns are read together: a is the fastest axis of the volume
  // copy the patch reads
  const bool xt = pt.layout == 1;
  const int a = xt ? 1 : 0;
  if (c == a) return;
  const int b = 3 - a - c, ax[3] = {a, b, c};
  const double det = L[a] * L[3 + b] - L[b] * L[3 + a];
  const double i00 = L[3 + b] / det, i01 = -L[b] / det, i10 = -L[3 + a] / det, i11 = L[a] / det;
  const double ra = fabs(i00) + fabs(i01), rb = fabs(i10) + fabs(i11);
  // (false for a motion that is not finite)
  const int sx = xt ? pr.ny : 1, sy = xt ? 1 : pr.nx, sz = pr.nx * pr.ny;
  o.st_a = sel3(a, sx, sy, sz); o.st_b = sel3(b, sx, sy, sz); o.st_c = sel3(c, sx, sy, sz);
  const bool ok = fabs(det) > 1e-6 && ra < 1.5 - 1e-3 && rb < 1.5 - 1e-3 && g.ext[c] < 64.0 &&
                  o.st_b < 1 << 23;  // (24-bit products)
  if (!ok) return;
  // What the rows cost goes with the cross-section of the support's bounding box (4
  // area voxels), what the planes cost with the parallelogram (4 share voxels, of
  // which the cell holds four).  The line fits the crossovers of the forward pass at
  // 96^3 (rows / planes, us): zeros 1 voxel off at rest 75 / 70, 1.05 at rest 89 / 102,
  // at 3 degrees 116 / 122, at 10 147 / 130, 1.1 at 6 degrees 134 / 138, at 15 174 / 154,
  // 1.2 at rest 114 / 142, at 10 degrees 167 / 170, at 15 195 / 174.
  const double share = 1.0 / fabs(det), area = g.ext[a] * g.ext[b];
  if (area < fmin(1.0 + 8.0 * (share - 1.0), 3.3) - 0.02) return;
  for (int i = 0; i < 3; ++i) {
    o.Lu[i] = (float)L[ax[i]];
    o.Lv[i] = (float)L[3 + ax[i]];
    o.Ln[i] = (float)(L[6 + ax[i]] * SQRT_KAPPA);
    o.ax[i] = ax[i];
  }
  const double ta = -(i00 * L[c] + i01 * L[3 + c]), tb = -(i10 * L[c] + i11 * L[3 + c]);
  o.ta = (float)ta;
  o.tb = (float)tb;
  o.tn = (float)((L[6 + c] + ta * L[6 + a] + tb * L[6 + b]) * SQRT_KAPPA);
  o.qa = (float)(1.5 - 1e-4 - ra);
  o.qb = (float)(1.5 - 1e-4 - rb);
  // (with the third columns and rows, which lie up to two voxels off the line)
  o.ra = (float)(fabs(ta) * g.ext[c] + 2.01);
  o.rb = (float)(fabs(tb) * g.ext[c] + 2.01);
  o.rc = (float)g.ext[c];
  o.cut = (float)g.cut;
  o.na = sel3(a, pr.nx, pr.ny, pr.nz); o.nb = sel3(b, pr.nx, pr.ny, pr.nz);
  o.nc = sel3(c, pr.nx, pr.ny, pr.nz);
  o.on = 1;
}

// Sum of g_hat X (HAS_X) or of g_hat over the in-grid voxels of the sample
// centred f beside voxel b (sample_centre).  EDGE: cells may reach outside the
// grid.
template <bool HAS_X, bool EDGE>
__device__ __forceinline__ float sinc_cells(const SincPatch &g, const int b[3], const float f[3],
                                            __amdgpu_buffer_rsrc_t xr, unsigned nbytes) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  const float fc = f[2], cut = g.cut;
  const int lo = max((int)ceilf(fc - g.rc), -b[2]), hi = min((int)floorf(fc + g.rc), g.nc - 1 - b[2]);
  const auto weight = [&](float u, float v, float n) {
    return sinc_lobe<float>(u) * sinc_lobe<float>(v) * clamp01<float>(fast_exp2<float>(-n * n) - cut);
  };
  const auto step = [](float t, const float L[3], int i, int j) {
    const float r = i ? t + L[0] : t;
    return j ? r + L[1] : r;
  };
  float acc = 0.f, wc = (float)lo - fc;
  int plane = (b[2] + lo) * g.st_c + b[1] * g.st_b + b[0];  // of voxel (b[0], b[1])
  for (int oc = lo; oc <= hi; ++oc, wc += 1.f, plane += g.st_c) {
    // the line's point, the corner of its cell and t there
    const float pa = fmaf(g.ta, wc, f[0]), pb = fmaf(g.tb, wc, f[1]);
    const float fa = floorf(pa), fb = floorf(pb), ga = pa - fa, gb = pb - fb;
    const float u = -fmaf(g.Lu[0], ga, g.Lu[1] * gb), v = -fmaf(g.Lv[0], ga, g.Lv[1] * gb),
                n = fmaf(g.tn, wc, -fmaf(g.Ln[0], ga, g.Ln[1] * gb));
    const int a0 = (int)fa, b0 = (int)fb;
    const unsigned off = (unsigned)(plane + __mul24(b0, g.st_b) + a0) * 4u;
    const auto inside = [&](int a, int c) {
      return !EDGE || ((unsigned)(b[0] + a) < (unsigned)g.na && (unsigned)(b[1] + c) < (unsigned)g.nb);
    };
    float sum = 0.f;  // the plane's: fewer roundings than one running sum
    float x[2][2];    // a voxel outside the grid reads 0
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (HAS_X && !EDGE) {
        const f2 r = __builtin_bit_cast(
            f2, __builtin_amdgcn_raw_buffer_load_b64(xr, (int)off, j * g.st_b * 4, 0));
        x[j][0] = r.x;
        x[j][1] = r.y;
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bool in = inside(a0 + i, b0 + j);
          x[j][i] = HAS_X ? load_vox<float>(xr, in ? off + (unsigned)(j * g.st_b + i) * 4u : nbytes)
                          : in ? 1.f : 0.f;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float w = weight(step(u, g.Lu, i, j), step(v, g.Lv, i, j), step(n, g.Ln, i, j));
        sum = HAS_X || EDGE ? fmaf(w, x[j][i], sum) : sum + w;
      }
    // the third column and row, on the nearer side
    if (fabsf(ga - 0.5f) > g.qa || fabsf(gb - 0.5f) > g.qb) {
      const float sa = ga < 0.5f ? -1.f : 2.f, sb = gb < 0.5f ? -1.f : 2.f;
      const float ua = fmaf(sa, g.Lu[0], u), va = fmaf(sa, g.Lv[0], v);
      const float ub = fmaf(sb, g.Lu[1], u), vb = fmaf(sb, g.Lv[1], v);
      const auto in = [](float s, float t) { return fmaxf(fabsf(s), fabsf(t)) < 1.f; };
      unsigned m = (in(ua, va) ? 1u : 0u) | (in(ua + g.Lu[1], va + g.Lv[1]) ? 2u : 0u) |
                   (in(ub, vb) ? 4u : 0u) | (in(ub + g.Lu[0], vb + g.Lv[0]) ? 8u : 0u) |
                   (in(fmaf(sb, g.Lu[1], ua), fmaf(sb, g.Lv[1], va)) ? 16u : 0u);
      while (m) {
        const unsigned k = m & (0u - m);
        m ^= k;
        const float ea = k == 4u ? 0.f : k == 8u ? 1.f : sa, eb = k == 1u ? 0.f : k == 2u ? 1.f : sb;
        const int ja = (int)ea, jb = (int)eb;
        const bool on = inside(a0 + ja, b0 + jb);
        const float x1 = HAS_X ? load_vox<float>(xr, on ? off + (unsigned)(__mul24(jb, g.st_b) + ja) * 4u : nbytes)
                               : on ? 1.f : 0.f;
        sum = fmaf(weight(fmaf(ea, g.Lu[0], fmaf(eb, g.Lu[1], u)), fmaf(ea, g.Lv[0], fmaf(eb, g.Lv[1], v)),
                          fmaf(ea, g.Ln[0], fmaf(eb, g.Ln[1], n))), x1, sum);
      }
    }
    acc += sum;
  }
  return acc;
}
template <bool HAS_X>
__device__ __forceinline__ float sinc_planes(const SincPatch &g, const int b[3], const float f[3],
                                             __amdgpu_buffer_rsrc_t xr, unsigned nbytes) {
  const int p[3] = {sel3(g.ax[0], b[0], b[1], b[2]), sel3(g.ax[1], b[0], b[1], b[2]),
                    sel3(g.ax[2], b[0], b[1], b[2])};
  const float q[3] = {sel3f<float>(g.ax[0], f[0], f[1], f[2]), sel3f<float>(g.ax[1], f[0], f[1], f[2]),
                      sel3f<float>(g.ax[2], f[0], f[1], f[2])};
  const float xa = (float)p[0] + q[0], xb = (float)p[1] + q[1];
  const bool inner = xa >= g.ra && xa <= (float)(g.na - 1) - g.ra && xb >= g.rb &&
                     xb <= (float)(g.nb - 1) - g.rb;
  return __all(inner) ? sinc_cells<HAS_X, false>(g, p, q, xr, nbytes)
                      : sinc_cells<HAS_X, true>(g, p, q, xr, nbytes);
}

// The plane walk with the derivative's moments (pvr_grad.h: psf_walk_grad, along
// the axes a, b, c), for the two samples of the block's sub-window row j: relative
// to the value xb of one voxel near the block, per sample acc = sum g_hat (X - xb),
// z = sum g_hat, and the nine offset moments of e^{-Q/2} (X - xb) in mx and of
// e^{-Q/2} in me.  (All four at once share more exponentials but hold 420
// registers, one wavefront a SIMD.)  In a plane the
// moments are taken about each sample's nearest voxel, where they are sums and
// differences, and moved to the sample's centre once.
template <typename T, int NB>
__device__ __forceinline__ void plane_walk_grad(const FwdPatch<T> &g, int u, int v, int j,
                                                __amdgpu_buffer_rsrc_t xr, unsigned nbytes, T &xb,
                                                T acc[2], T z[2], T mx[2][9], T me[2][9]) {
  const double du = u, dv = v;
  const double xa = fma(g.Ha[0], du, fma(g.Ha[1], dv, g.Ha[2]));
  const double xbd = fma(g.Hb[0], du, fma(g.Hb[1], dv, g.Hb[2]));
  const double xc = fma(g.Hc[0], du, fma(g.Hc[1], dv, g.Hc[2]));
  const double rc = __builtin_rint(xc), dc = rc - xc;
  const double pa = fma(g.ta, dc, xa) - 0.5, pb = fma(g.tb, dc, xbd) - 0.5;
  const double ra = __builtin_rint(pa), rb = __builtin_rint(pb);
  const T f0 = (T)(pa - ra), h0 = (T)(pb - rb), z0 = (T)dc;
  const int ia0 = (int)ra - 1, ib0 = (int)rb - 1, ic0 = (int)rc;
  {
    const int a = min(max(ia0 + 1, 0), g.na - 1), b = min(max(ib0 + 1, 0), g.nb - 1),
              c = min(max(ic0, 0), g.nc - 1);
    xb = load_vox<T>(xr, (unsigned)(c * g.st_c + b * g.st_b + a * g.st_a) * (unsigned)sizeof(T));
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    acc[t] = z[t] = (T)0;
#pragma unroll
    for (int q = 0; q < 9; ++q) mx[t][q] = me[t][q] = (T)0;
  }
#pragma unroll 1
  for (int k = -g.half; k <= g.half; ++k) {
    asm volatile("" ::: "memory");  // the constants (in LDS) are read again: held, they would spill
    const T cut = g.cut;
    const T kk = (T)k;
    const T qa = fma(kk, g.fta, f0), qb = fma(kk, g.ftb, h0);
    const T sa = round_val<false>(qa), sb = round_val<NB == 4>(qb);
    const T f = qa - sa, h = qb - sb, wz = z0 + kk;
    const int ia = ia0 + (int)sa, ib = ib0 + j + (int)sb, ic = ic0 + k;
    const bool inside = (unsigned)ic < (unsigned)g.nc && ia >= 0 && ia + 4 <= g.na && ib >= 0 && ib + NB <= g.nb;
    T x[NB][4];
    load_rows<NB - 1>(g, xr, nbytes, ia, ib, ic, inside, x);
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[r][i] -= xb;
    const T m = g.Aab2 * f * h;
    const T ea = -g.Aaa * f * f, eb = -g.Abb * h * h;
    const T sla = fma(g.Aab2, h, (T)2 * g.Aaa * f), slb = fma(g.Aab2, f, (T)2 * g.Abb * h);
    T U[3], V[NB];
    U[0] = fast_exp2<T>(ea - g.Aaa - sla);
    U[1] = fast_exp2<T>(ea);
    U[2] = fast_exp2<T>(ea - g.Aaa + sla);
    V[0] = fast_exp2<T>(eb - g.Abb - slb);
    V[1] = fast_exp2<T>(eb);
    V[2] = fast_exp2<T>(eb - g.Abb + slb);
    if constexpr (NB == 4) V[3] = fast_exp2<T>(fma((T)-4, g.Abb, fma((T)2, slb, eb)));
    T ca[4] = {(T)1, (T)1, (T)1, (T)1}, cb[NB];
#pragma unroll
    for (int r = 0; r < NB; ++r) cb[r] = (T)1;
    const bool edge = !__all(inside);  // voxels outside the grid do not count
    if (edge) {
      const bool pc = (unsigned)ic < (unsigned)g.nc;
#pragma unroll
      for (int i = 0; i < 4; ++i) ca[i] = (unsigned)(ia + i) < (unsigned)g.na ? (T)1 : (T)0;
#pragma unroll
      for (int r = 0; r < NB; ++r) cb[r] = pc && (unsigned)(ib + r) < (unsigned)g.nb ? (T)1 : (T)0;
    }
    const T xm = g.kap[XM], xp = g.kap[XP];
#pragma unroll
    for (int t = 0; t < 2; ++t) {  // sub-window (t, j)
      const bool same = t == j;
      const auto pick = [&](T v11, T v10) { const T v = same ? v11 : v10; return t ? v : -v; };
      const T w = wz - pick(g.e11, g.e10), D = same ? g.D11 : g.D10;
      const T ka = g.kap[(same ? KA11 : KA10) + (t ? 0 : 1)], ja = g.kap[(same ? KA11 : KA10) + (t ? 1 : 0)];
      const T kb = g.kap[(same ? KB11 : KB10) + (t ? 0 : 1)], jb = g.kap[(same ? KB11 : KB10) + (t ? 1 : 0)];
      const T S = fast_exp2<T>(-fma(g.Scc * w, w, fma(f, pick(g.ga11, g.ga10), fma(h, pick(g.gb11, g.gb10), D + m))));
      const T Um = U[0] * ja * ca[t], Uc = U[1] * ca[t + 1], Up = U[2] * ka * ca[t + 2];
      // plane moments about the nearest voxel: m00, m10, m20, m01, m11, m02
      T px[6] = {(T)0, (T)0, (T)0, (T)0, (T)0, (T)0}, pe[6] = {(T)0, (T)0, (T)0, (T)0, (T)0, (T)0};
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        T E = V[b] * S * cb[b];
        if (b == 0) E *= jb;
        if (b == 2) E *= kb;
        if (b == 3) E *= kb * kb;
        const T Em = b == 0 ? E * xm : b == 1 ? E : b == 2 ? E * xp : E * (xp * xp);
        const T Ep = b == 0 ? E * xp : b == 1 ? E : b == 2 ? E * xm : E * (xm * xm);
        const T w0 = Em * Um, w1 = E * Uc, w2 = Ep * Up;
        const T g0 = clamp01<T>(w0 - cut), g1 = clamp01<T>(w1 - cut),
                    g2 = clamp01<T>(w2 - cut);
        const T e0 = g0 > (T)0 ? w0 : (T)0, e1 = g1 > (T)0 ? w1 : (T)0, e2 = g2 > (T)0 ? w2 : (T)0;
        const T v0 = x[b][t], v1 = x[b][t + 1], v2 = x[b][t + 2];
        acc[t] = fma(g0, v0, acc[t]);
        acc[t] = fma(g1, v1, acc[t]);
        acc[t] = fma(g2, v2, acc[t]);
        z[t] += g0 + g1 + g2;
        const T a0 = e0 * v0, a1 = e1 * v1, a2 = e2 * v2;
        const T xs = a0 + a2, es = e0 + e2, xd = a2 - a0, ed = e2 - e0;
        const T x0 = xs + a1, n0 = es + e1;
        px[0] += x0; px[1] += xd; px[2] += xs;
        pe[0] += n0; pe[1] += ed; pe[2] += es;
        if (b != 1) {
          const T s1 = b == 0 ? -(T)1 : b == 2 ? (T)1 : (T)2, s2 = s1 * s1;
          px[3] = fma(s1, x0, px[3]); px[4] = fma(s1, xd, px[4]); px[5] = fma(s2, x0, px[5]);
          pe[3] = fma(s1, n0, pe[3]); pe[4] = fma(s1, ed, pe[4]); pe[5] = fma(s2, n0, pe[5]);
        }
      }
      // about the sample's centre, at (fa, hb) from its nearest voxel (the plane's
      // conditional centre lies t w beside it)
      const T fa = fma(-g.fta, w, f + pick(g.da11, g.da10)), hb = fma(-g.ftb, w, h + pick(g.db11, g.db10));
      auto move = [&](const T p[6], T o[9]) {
        const T sa1 = fma(-fa, p[0], p[1]), sb1 = fma(-hb, p[0], p[3]);
        o[0] += sa1;
        o[1] += sb1;
        o[2] = fma(w, p[0], o[2]);
        o[3] += fma(-fa, p[1] + sa1, p[2]);
        o[4] += fma(-fa, sb1, fma(-hb, p[1], p[4]));
        o[5] = fma(w, sa1, o[5]);
        o[6] += fma(-hb, p[3] + sb1, p[5]);
        o[7] = fma(w, sb1, o[7]);
        o[8] = fma(w * w, p[0], o[8]);
      };
      move(px, mx[t]);
      move(pe, me[t]);
    }
  }
}

}  // namespace pvr
