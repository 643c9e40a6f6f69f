// Plan creation and the motion-dependent build: per-patch geometry, per-sample
// PSF normalisers and the brick -> patch index of the gather adjoint.
#include <limits.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "pvr_internal.h"
#include "pvr_util.h"
#include "pvr_geometry.h"
#include "pvr_planes.h"

using namespace pvr;

static pvr_status make_tiles(pvr_plan *p, int tile_w, int tile_h);

// Which walks the plan uses, from every stack's first patch at rest: the block
// gather (make_adj) and the plane walks (make_fwd) where at least half of the
// samples lie in stacks on their fast path, i.e. pixels about as wide as voxels
// and the PSF about as wide as a pixel.  The motion is not known here: the patches
// of such a plan that leave it (a large tilt, or a stack of another kind) run the
// per-voxel or per-sample walk inside the same kernels.  What that costs against
// the walks' own kernels, all patches turned by 60 degrees (us, own / here): forward
// 128^3 562 / 513, 32^3 17 / 18; adjoint 128^3 420 / 346, 192^3 with 37 x 37 patches
// 1494 / 1540; FP64 48^3 forward 52 / 51, adjoint 144 / 150, derivative 133 / 133.
static void choose_walks(pvr_plan *p) {
  std::vector<char> adj(p->S, 0), fwd(p->S, 0), fwd64(p->S, 0), seen(p->S, 0);
  long long n_adj = 0, n_fwd = 0, n_fwd64 = 0;
  for (int s = 0; s < p->M; ++s) {
    const PatchDev &q = p->h_patch[s];
    const int t = q.stack;
    if (!seen[t]) {
      seen[t] = 1;
      const double th[6] = {0, 0, 0, 0, 0, 0};
      GeoD g;
      GeoF f;
      int bb[6];
      if (p->psf == PVR_PSF_SINC)
        make_geometry<PVR_PSF_SINC>(p->h_prob[q.problem], p->h_stack[t], q, th, p->k, g, f, bb);
      else
        make_geometry<PVR_PSF_GAUSSIAN>(p->h_prob[q.problem], p->h_stack[t], q, th, p->k, g, f, bb);
      AdjPatch<float> a;
      FwdPatch<float> w;
      FwdPatch<double> w64;
      make_adj(g, q, a);
      make_fwd(g, p->h_prob[q.problem], q, w);
      make_fwd(g, p->h_prob[q.problem], q, w64);
      adj[t] = (a.cls & ADJ_FAST) != 0;
      fwd[t] = w.rows != 0;
      fwd64[t] = w64.rows != 0;
    }
    const long long n = (long long)q.w * q.h;
    n_adj += adj[t] ? n : 0;
    n_fwd += fwd[t] ? n : 0;
    n_fwd64 += fwd64[t] ? n : 0;
  }
  p->gather_blocks = p->max_hu <= 1 && p->max_hv <= 1 && 2 * n_adj >= p->N;
  p->planes = 2 * n_fwd >= p->N;
  p->planes64 = 2 * n_fwd64 >= p->N;
}

// Largest capacity of an adjoint index list (its offsets are int32).
constexpr long long INDEX_CAP_MAX = 0x7ffffff0LL;

// Upper bound, over every motion and either PSF, on the number of bricks of
// e^3 voxels (a lattice of step e voxels) that the separating-axis test of
// the index kernels lists for one patch.  A brick is listed only if its
// voxel-centre box meets each of the three slabs of the patch's pixel-frame
// support box, so its centre lies in the support box widened on every side
// by the box's largest projected half-width hb = (e - 1)/2 sum_c |V_c| (V_c
// the voxel axes in mm).  That widened box K is a rotated box with sides
// D_a (mm), and the cells of the centres inside it are disjoint and lie in K
// grown by the cell's circumradius R, so the count is at most
// (D0 D1 D2 + 2 (D0 D1 + D1 D2 + D2 D0) R + pi (D0 + D1 + D2) R^2 +
// 4/3 pi R^3) / (e^3 |det V|), the Steiner volume of the grown box over the
// cell volume.  At most `cap` (the grid's own count).
static long long pair_bound(const ProbDev &pr, const StackDev &st, const PatchDev &q, double k,
                            int e, long long cap) {
  double V[3][3], sumn = 0;
  for (int c = 0; c < 3; ++c) {
    double n2 = 0;
    for (int r = 0; r < 3; ++r) {
      V[c][r] = pr.v2w[4 * r + c];
      n2 += V[c][r] * V[c][r];
    }
    sumn += sqrt(n2);
  }
  double R = 0;
  for (int sgn = 0; sgn < 8; ++sgn) {
    double n2 = 0;
    for (int r = 0; r < 3; ++r) {
      double x = 0;
      for (int c = 0; c < 3; ++c) x += ((sgn >> c) & 1 ? -1.0 : 1.0) * V[c][r];
      n2 += x * x;
    }
    R = std::max(R, sqrt(n2));
  }
  R *= 0.5 * e;
  const double det = fabs(V[0][0] * (V[1][1] * V[2][2] - V[1][2] * V[2][1]) -
                          V[1][0] * (V[0][1] * V[2][2] - V[0][2] * V[2][1]) +
                          V[2][0] * (V[0][1] * V[1][2] - V[0][2] * V[1][1]));
  const double hb = 0.5 * (e - 1) * sumn;
  const double reach_u = std::max(k * st.sigma[0], st.wz[0]);
  const double reach_v = std::max(k * st.sigma[1], st.wz[1]);
  const double reach_n = k * st.sigma[2];
  double D[3] = {(q.w - 1) * st.spacing[0] + 2 * reach_u + 2 * hb,
                 (q.h - 1) * st.spacing[1] + 2 * reach_v + 2 * hb, 2 * reach_n + 2 * hb};
  for (double &d : D) d = d * (1 + 1e-6) + 1e-6;  // room for the test's rounding
  const double pi = 3.14159265358979323846;
  const double vol = D[0] * D[1] * D[2] + 2 * (D[0] * D[1] + D[1] * D[2] + D[2] * D[0]) * R +
                     pi * (D[0] + D[1] + D[2]) * R * R + 4.0 / 3.0 * pi * R * R * R;
  const double n = ceil(vol / (det * e * e * e)) + 1;
  return n >= (double)cap ? cap : (long long)n;
}

// Per-patch geometry of a build: four wavefronts per 64 patches.  The first
// runs the motion geometry, one patch per lane; then the wavefronts derive from
// it (through LDS) the support boxes and the group's brick range, the block
// gather's constants, the plane walk's, and the FP64 versions of both, side by
// side: the launch is as long as its longest chain of dependent FP64 steps and
// strided stores (29 us with one thread per patch doing all in turn, 16 here, 2 560
// patches).  The FP64 geometry is stored for FP64 builds only.  Keeps
// the motion and the active set (all patches if null) for later passes.
struct MiniGeo {
  double G[12], H[12], cu, cv, ck, K2, cut;
};
template <typename TH>
__global__ void __launch_bounds__(256)
k_geometry(const ProbDev *__restrict__ probs, const StackDev *__restrict__ stacks,
           const PatchDev *__restrict__ patches, const TH *__restrict__ theta_in,
           const uint8_t *__restrict__ active_in, int M, double k, int psf, int f64,
           double *__restrict__ theta, uint8_t *__restrict__ active, GeoD *__restrict__ gd,
           GeoF *__restrict__ gf, AdjPatch<float> *__restrict__ adj,
           AdjPatch<double> *__restrict__ adj64, FwdPatch<float> *__restrict__ fwd,
           FwdPatch<double> *__restrict__ fwd64, SincPatch *__restrict__ sp, int *__restrict__ bb, int *__restrict__ gbox,
           double *__restrict__ sbox) {
  __shared__ MiniGeo mini[64];
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = blockIdx.x * 64 + lane;
  const bool on = s < M;
  int r6[6] = {INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN};
  if (role == 0 && on) {
    const PatchDev pt = patches[s];
    const StackDev &st = stacks[pt.stack];
    double th[6];
    for (int a = 0; a < 6; ++a) {
      th[a] = (double)theta_in[6 * s + a];
      theta[6 * s + a] = th[a];
    }
    GeoD g;
    GeoF f;
    if (psf == PVR_PSF_SINC) make_geometry<PVR_PSF_SINC>(probs[pt.problem], st, pt, th, k, g, f, r6);
    else make_geometry<PVR_PSF_GAUSSIAN>(probs[pt.problem], st, pt, th, k, g, f, r6);
    MiniGeo &m = mini[lane];
    for (int q = 0; q < 12; ++q) {
      m.G[q] = g.G[q];
      m.H[q] = g.H[q];
    }
    m.cu = g.cu; m.cv = g.cv; m.ck = g.ck; m.K2 = g.K2; m.cut = g.cut;
    gf[s] = f;
    if (f64) gd[s] = g;
    if (psf == PVR_PSF_SINC) make_sinc(g, probs[pt.problem], pt, sp[s]);
    active[s] = active_in ? active_in[s] : 1;
  }
  __syncthreads();
  if (role == 0) {
    if (on)
      for (int q = 0; q < 6; ++q) bb[6 * s + q] = r6[q];
    // union of the brick ranges of the 64 patches: a brick outside it meets none
    // of them (empty ranges, low end above the high end, only widen it)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        r6[r] = min(r6[r], __shfl_xor(r6[r], o, 64));
        r6[3 + r] = max(r6[3 + r], __shfl_xor(r6[3 + r], o, 64));
      }
    int v = r6[0];
#pragma unroll
    for (int r = 1; r < 6; ++r) v = lane == r ? r6[r] : v;
    if (lane < 6) gbox[6 * blockIdx.x + lane] = v;
  }
  if (!on) return;
  const PatchDev pt = patches[s];
  const MiniGeo &m = mini[lane];
  if (role == 0) {
    // voxel -> pixel map and the pixel-frame support box of the patch
    const StackDev &st = stacks[pt.stack];
    double *o = sbox + 18 * s;
    for (int q = 0; q < 12; ++q) o[q] = m.G[q];
    const bool sinc = psf == PVR_PSF_SINC;
    const double ru = sinc ? st.wz[0] / st.spacing[0] : k * st.sigma[0] / st.spacing[0],
                 rv = sinc ? st.wz[1] / st.spacing[1] : k * st.sigma[1] / st.spacing[1],
                 rk = k * st.sigma[2] / st.spacing[2];
    o[12] = pt.x0 - ru; o[13] = pt.x0 + pt.w - 1 + ru;
    o[14] = pt.y0 - rv; o[15] = pt.y0 + pt.h - 1 + rv;
    o[16] = pt.slice - rk; o[17] = pt.slice + rk;
    return;
  }
  if (role == 3 && !f64) return;
  GeoD g;
  for (int q = 0; q < 12; ++q) {
    g.G[q] = m.G[q];
    g.H[q] = m.H[q];
  }
  g.cu = m.cu; g.cv = m.cv; g.ck = m.ck; g.K2 = m.K2; g.cut = m.cut;
  g.psf = psf;
  if (role == 1) make_adj(g, pt, adj[s]);
  if (role == 2) make_fwd(g, probs[pt.problem], pt, fwd[s]);
  if (role == 3) {
    make_adj(g, pt, adj64[s]);
    make_fwd(g, probs[pt.problem], pt, fwd64[s]);
  }
}

// Per-sample inverse normaliser 1/Z_j (0 marks an invalid sample).  Keeps the
// sample mask (all ones if null) for later passes.
template <typename T>
__global__ void __launch_bounds__(SIM_THREADS)
k_normalisers(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
              const BlockWork *__restrict__ work, const typename GeoOf<T>::type *__restrict__ geo,
              const SincPatch *__restrict__ sp, const uint8_t *__restrict__ mask,
              const uint8_t *__restrict__ active, uint8_t *__restrict__ keep,
              float *__restrict__ invz, double *__restrict__ invz64) {
  const BlockWork wk = work[blockIdx.x];
  const PatchDev pt = patches[wk.patch];
  const ProbDev pr = probs[pt.problem];
  const typename GeoOf<T>::type &g = geo[wk.patch];
  const int n = pt.w * pt.h;
  const int l1 = min(n, wk.l0 + SIM_CHUNK);
  const bool act = active[wk.patch] != 0;
  for (int l = wk.l0 + threadIdx.x; l < l1; l += SIM_THREADS) {
    const long long j = pt.off + l;
    const int u = pt.x0 + l % pt.w, v = pt.y0 + l / pt.w;
    int b[3];
    T f[3];
    const uint8_t kept = mask ? mask[j] : 1;
    keep[j] = kept;
    bool ok = sample_centre(g, pr, u, v, pt.slice, b, f) && act && kept;
    T z = 0, acc = 0;
    if (ok && g.psf == PVR_PSF_SINC) {
      const __amdgpu_buffer_rsrc_t none = raw_buffer((const T *)nullptr, 0u);
      bool planes = false;
      if constexpr (sizeof(T) == 4) {
        planes = sp[wk.patch].on != 0;
        if (planes) z = sinc_planes<false>(sp[wk.patch], b, f, none, 0u);
      }
      if (!planes) psf_walk_sinc<T, typename GeoOf<T>::type, false>(g, pr, b, f, none, 0u, &z);
    } else if (ok) {
      psf_walk<T, typename GeoOf<T>::type, false>(g, pr, b, f, nullptr, z, acc);
    }
    ok = ok && z > (T)0;
    const T iz = ok ? (T)1 / z : (T)0;
    invz[j] = (float)iz;
    if (invz64) invz64[j] = (double)iz;
  }
}

// The same by the plane walk: one lane per 2 x 2 pixel block.  Bound by vector
// issue: 10.5 M samples of a 160^3 plan take 198 us one sample per lane, 167 us here
// (1.8 M at 96^3: 45 and 37 us).
template <typename T>
__global__ void __launch_bounds__(PLANE_BLOCKS)
k_normalisers_planes(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
                     const BlockWork *__restrict__ work,
                     const typename GeoOf<T>::type *__restrict__ geo,
                     const FwdPatch<T> *__restrict__ fwd, const uint8_t *__restrict__ mask,
                     const uint8_t *__restrict__ active, uint8_t *__restrict__ keep,
                     float *__restrict__ invz, double *__restrict__ invz64) {
  const BlockWork wk = work[blockIdx.x];
  const PatchDev pt = patches[wk.patch];
  const ProbDev pr = probs[pt.problem];
  const typename GeoOf<T>::type &g = geo[wk.patch];
  const FwdPatch<T> &fw = fwd[wk.patch];
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const bool act = active[wk.patch] != 0;
  const __amdgpu_buffer_rsrc_t none = raw_buffer((const T *)nullptr, 0u);
  const auto put = [&](long long j, bool ok, T z) {
    const T iz = ok && z > (T)0 ? (T)1 / z : (T)0;
    invz[j] = (float)iz;
    if (invz64) invz64[j] = (double)iz;
  };
  if (fw.rows) {
    const PlaneLane pl = plane_lane(pt, wk.l0);
    const int nbu = (pt.w + 1) / 2;
    const int u0 = 2 * (pl.blk % nbu), v0 = 2 * (pl.blk / nbu);
    bool ok[4];  // pixel (u0 + i, v0 + j) at 2 j + i
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int u = u0 + (t & 1), v = v0 + (t >> 1);
      int b[3];
      T f[3];
      ok[t] = pl.on && u < pt.w && v < pt.h && act &&
              sample_centre(g, pr, pt.x0 + u, pt.y0 + v, pt.slice, b, f);
      if (pl.on && u < pt.w && v < pt.h) {
        const long long j = pt.off + (long long)v * pt.w + u;
        const uint8_t kept = mask ? mask[j] : 1;
        if (pl.part == 0) keep[j] = kept;
        ok[t] = ok[t] && kept;
      }
    }
    const bool live = ok[0] || ok[1] || ok[2] || ok[3];
    T zw[4] = {0, 0, 0, 0};  // by sub-window
    if (__any(live)) {
      if (fw.rows == 3) plane_walk<T, 3, false, true>(fw, u0, v0, live, pl.part, pl.parts, none, 0u, nullptr, zw);
      else plane_walk<T, 4, false, true>(fw, u0, v0, live, pl.part, pl.parts, none, 0u, nullptr, zw);
    }
    combine_parts(pl, zw, reinterpret_cast<T(*)[4]>(lds));
    if (pl.part != 0 || !pl.on) return;
    const bool fu = fw.flip & 1, fv = fw.flip & 2;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int u = u0 + (t & 1), v = v0 + (t >> 1);
      const T a = fu ? zw[t ^ 1] : zw[t], c = fu ? zw[t ^ 3] : zw[t ^ 2];
      if (u < pt.w && v < pt.h) put(pt.off + (long long)v * pt.w + u, ok[t], fv ? c : a);
    }
  } else {
    each_pixel<false>(pt, wk.l0, true, 0, 0u, [&](int u, int v) {
      const long long j = pt.off + (long long)v * pt.w + u;
      const uint8_t kept = mask ? mask[j] : 1;
      keep[j] = kept;
      int b[3];
      T f[3], z = 0, acc = 0;
      const bool ok = sample_centre(g, pr, pt.x0 + u, pt.y0 + v, pt.slice, b, f) && act && kept;
      if (ok) psf_walk<T, typename GeoOf<T>::type, false>(g, pr, b, f, nullptr, z, acc);
      put(j, ok, z);
    });
  }
}

// Adjoint index: per brick the lists of the patches that reach its parts.  A
// patch is listed when the brick is inside its voxel bounding box and the
// part's corner voxels, mapped into the patch's pixel frame, overlap the
// patch's support box on each of the three stack axes (separating-axis test;
// conservative).
__device__ __forceinline__ bool box_meets_patch(const double *sb, const double lo[3],
                                                const double hi[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double *g = sb + 4 * a;
    double mn = g[3], mx = g[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double p = g[c] * lo[c], q = g[c] * hi[c];
      mn += fmin(p, q);
      mx += fmax(p, q);
    }
    if (mx < sb[12 + 2 * a] || mn > sb[13 + 2 * a]) return false;
  }
  return true;
}

// The parts of brick b that a patch reaches, one bit each.  NL = 8: the
// sub-bricks (SUB^3 voxels, one wavefront of the per-voxel gather each).
// NL = 6: the halves along the patch's normal axis an (bit 2 an + half,
// 8 x 8 x 4 voxels, one wavefront of the block gather each).
template <int NL>
__device__ __forceinline__ unsigned part_mask(const int b[3], int an, const double *__restrict__ sb) {
  double g[18];
  const double2 *s2 = reinterpret_cast<const double2 *>(sb);  // 144-byte rows
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const double2 v = s2[q];
    g[2 * q] = v.x;
    g[2 * q + 1] = v.y;
  }
  unsigned m = 0;
#pragma unroll
  for (int w = 0; w < (NL == 6 ? 2 : 8); ++w) {
    double lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const bool cut = NL == 8 || a == an;
      const int o = NL == 8 ? (w >> a) & 1 : w;
      lo[a] = b[a] * BRICK + (cut ? o * SUB : 0);
      hi[a] = lo[a] + (cut ? SUB : BRICK) - 1;
    }
    m |= box_meets_patch(g, lo, hi) ? (NL == 6 ? 1u << (2 * an + w) : 1u << w) : 0u;
  }
  return m;
}

constexpr int PGROUP = 64;  // patches per range union (k_geometry)
__device__ __forceinline__ bool brick_in_range(const int *__restrict__ r, const int b[3]) {
  return b[0] >= r[0] && b[0] <= r[3] && b[1] >= r[1] && b[1] <= r[4] && b[2] >= r[2] && b[2] <= r[5];
}

// The lists of NL parts per brick in one launch, one wavefront per brick: the
// lanes first test 64 patch groups' range unions at once, then the 64 patches
// of each group whose union holds the brick, four groups' loads in flight; the
// patches whose own range holds it queue up in LDS and are taken 64 at a time
// through the separating-axis tests.  The hits (patch and parts) wait in LDS
// until the workgroup has reserved space for its bricks' lists with one
// addition to the cursor; then each list is written in ascending patch order
// (ballot prefix counts), the order that fixes the adjoint's summation order.
// Where the reserved space lies varies from run to run, the lists do not.  A
// brick with more hits than LDS holds tests its patches again instead.  off:
// NL + 1 entries per brick, clamped to the capacity `cap`; a total beyond it
// (which the host bound on the pairs rules out) raises PVR_FAULT_INDEX.
// Bound by each wavefront's chain of loads.  Before, eleven launches (brick
// lists, then lists of their parts, each counted, scanned and filled): 160^3,
// 2 560 patches 195 us, now 33; 96^3 92 and 15, 48^3 66 and 12; testing each group's
// 64 patches where they stand, with no queue, 107, 36 and 20.  At 80 registers
// (6 wavefronts a SIMD) 256^3 with 11 760 patches takes 208 us, at 82 registers 230,
// at 64 (spills) 336.
constexpr int LIST_BRICKS = 8, LIST_HITS = 512;
template <int NL>
__global__ void __launch_bounds__(64 * LIST_BRICKS, NL == 6 ? 6 : 4)
k_adj_lists(const ProbDev *__restrict__ probs, const int *__restrict__ brick_prob,
            const int *__restrict__ bb, const int *__restrict__ gbox,
            const double *__restrict__ sbox, const AdjPatch<float> *__restrict__ adj, int nb,
            unsigned long long *__restrict__ cursor, int *__restrict__ off,
            int *__restrict__ list, long long cap, unsigned *__restrict__ status) {
  __shared__ unsigned hits[LIST_BRICKS][LIST_HITS];  // (patch - patch_begin) << 8 | parts
  __shared__ int queue[LIST_BRICKS][320];            // candidates: under 64 left, four groups added
  __shared__ int total[LIST_BRICKS];
  __shared__ unsigned long long base;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bi = blockIdx.x * LIST_BRICKS + wv;
  const bool on = bi < nb;  // uniform over the wavefront
  const ProbDev &pr = probs[brick_prob[on ? bi : 0]];
  const int local = bi - pr.brick_base;
  const int b[3] = {local % pr.nbx, (local / pr.nbx) % pr.nby, local / (pr.nbx * pr.nby)};
  const int p0 = pr.patch_begin, p1 = pr.patch_end;
  const unsigned long long below = (1ull << lane) - 1ull;
  int c[NL];
#pragma unroll
  for (int w = 0; w < NL; ++w) c[w] = 0;
  // calls f(s, m) for 64 candidate patches at a time, m the lane's parts
  auto each = [&](auto &&f) {
    if (!on || p1 <= p0) return;
    int nq = 0;
    auto take = [&](int q0, int n) {  // queue[q0 .. q0 + n), n <= 64
      const int s = lane < n ? queue[wv][q0 + lane] : -1;
      unsigned m = 0;
      if (s >= 0)
        m = part_mask<NL>(b, NL == 6 ? adj_normal_axis(adj[s].cls) : 0, sbox + 18 * s);
      f(s, m);
    };
    const int g1 = (p1 - 1) / PGROUP;
    for (int G0 = p0 / PGROUP; G0 <= g1; G0 += 64) {
      const int Gl = G0 + lane;
      unsigned long long hit = __ballot(Gl <= g1 && brick_in_range(gbox + 6 * Gl, b));
      while (hit) {
        int s[4];
        int2 r[4][3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[i] = hit ? (G0 + __builtin_ctzll(hit)) * PGROUP + lane : -1;
          hit &= hit - 1;
          if (s[i] < p0 || s[i] >= p1) s[i] = -1;
          const int2 *q = reinterpret_cast<const int2 *>(bb + 6 * (s[i] < 0 ? p0 : s[i]));
#pragma unroll
          for (int k = 0; k < 3; ++k) r[i][k] = q[k];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int rr[6] = {r[i][0].x, r[i][0].y, r[i][1].x, r[i][1].y, r[i][2].x, r[i][2].y};
          const bool in = s[i] >= 0 && brick_in_range(rr, b);
          const unsigned long long bal = __ballot(in);
          if (in) queue[wv][nq + __popcll(bal & below)] = s[i];
          nq += __popcll(bal);
        }
        if (nq >= 64) {
          __builtin_amdgcn_wave_barrier();
          int q0 = 0;
          for (; q0 + 64 <= nq; q0 += 64) take(q0, 64);
          const int rest = nq - q0;
          const int keep = lane < rest ? queue[wv][q0 + lane] : 0;
          __builtin_amdgcn_wave_barrier();
          if (lane < rest) queue[wv][lane] = keep;
          nq = rest;
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (nq) take(0, nq);
  };
  int n = 0;
  each([&](int s, unsigned m) {
    const unsigned long long any = __ballot(m != 0);
    if (!any) return;
    const int pos = n + __popcll(any & below);
    if (m && pos < LIST_HITS) hits[wv][pos] = (unsigned)(s - p0) << 8 | m;
    n += __popcll(any);
#pragma unroll
    for (int w = 0; w < NL; ++w) c[w] += __popcll(__ballot((m >> w) & 1u));
  });
  int sum = 0;
#pragma unroll
  for (int w = 0; w < NL; ++w) sum += c[w];
  if (lane == 0) total[wv] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int w = 0; w < LIST_BRICKS; ++w) t += (unsigned)total[w];
    // low 40 bits: pairs reserved, above: workgroups that did; the last one
    // leaves the cursor at zero for the next index and the total beside it
    const unsigned long long was = atomicAdd(cursor, t | 1ull << 40);
    base = was & ((1ull << 40) - 1);
    if (base + t > (unsigned long long)cap) atomicOr(status, PVR_FAULT_INDEX);
    if ((was >> 40) == gridDim.x - 1) {
      cursor[1] = base + t;
      cursor[0] = 0;
    }
  }
  __syncthreads();
  if (!on) return;
  long long at = (long long)base;
  for (int w = 0; w < wv; ++w) at += total[w];
  int end[NL];
  int first = 0;  // lane w: start of list w, lane NL: the end
#pragma unroll
  for (int w = 0; w < NL; ++w) {
    const int start = (int)min(at, cap);
    first = lane == w ? start : first;
    at += c[w];
    end[w] = (int)min(at, cap);
    c[w] = start;
  }
  first = lane == NL ? end[NL - 1] : first;
  if (lane <= NL) off[(long long)bi * (NL + 1) + lane] = first;
  auto put = [&](int s, unsigned m) {
#pragma unroll
    for (int w = 0; w < NL; ++w) {
      const bool h = (m >> w) & 1u;
      const unsigned long long bal = __ballot(h);
      const int pos = c[w] + __popcll(bal & below);
      if (h && pos < end[w]) list[pos] = s;
      c[w] += __popcll(bal);
    }
  };
  static_assert(PVR_MAX_PROBLEM_PATCHES <= 1 << 24, "24 bits of a hit hold the patch");
  if (n > LIST_HITS) {
    each(put);
    return;
  }
  for (int q0 = 0; q0 < n; q0 += 64) {
    const int q = q0 + lane;
    const unsigned e = q < n ? hits[wv][q] : 0u;
    put(p0 + (int)(e >> 8), e & 255u);
  }
}

// Largest voxel box over the forward tiles (sizes the staged LDS).
__global__ void k_tile_boxmax(const ProbDev *__restrict__ probs, const PatchDev *__restrict__ patches,
                              const int *__restrict__ tile_off, int M, int tile_w, int tile_h,
                              int n_tiles, const GeoF *__restrict__ geo, int *__restrict__ out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_tiles) return;
  const TileWork tw = tile_at(tile_off, M, patches, tile_w, tile_h, t);
  const PatchDev pt = patches[tw.patch];
  int lo[3], hi[3];
  const int c = tile_box(geo[tw.patch], probs[pt.problem], pt, tw, lo, hi);
  atomicMax(out, c);
}

// ---------------------------------------------------------------------------
// host API
// ---------------------------------------------------------------------------
static void host_mat3_from_aff(const double *a, double *L) {
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) L[3 * r + c] = a[4 * r + c];
}

extern "C" pvr_status pvr_plan_create(const pvr_grid *grids, int32_t n_problems,
                                      const pvr_stack *stacks, int32_t n_stacks,
                                      const pvr_patch *patches, int32_t n_patches,
                                      double cutoff_k, pvr_plan **out) {
  PVR_API_BEGIN();
  if (!out) return fail(PVR_EINVAL, "pvr_plan_create: out is NULL");
  *out = nullptr;
  if (!grids || !stacks || !patches) return fail(PVR_EINVAL, "pvr_plan_create: NULL descriptor array");
  if (n_problems <= 0 || n_stacks <= 0 || n_patches <= 0)
    return fail(PVR_ESHAPE, "pvr_plan_create: empty problem / stack / patch set");
  if (!(cutoff_k > 0 && cutoff_k < 20)) return fail(PVR_EINVAL, "pvr_plan_create: cutoff_k out of (0, 20)");
  pvr_plan *p = (pvr_plan *)calloc(1, sizeof(pvr_plan));
  PlanGuard guard(p);
  p->P = n_problems; p->S = n_stacks; p->M = n_patches; p->k = cutoff_k;
  p->h_prob = (ProbDev *)calloc(n_problems, sizeof(ProbDev));
  p->h_stack = (StackDev *)calloc(n_stacks, sizeof(StackDev));
  p->h_patch = (PatchDev *)calloc(n_patches, sizeof(PatchDev));
  p->h_sample_off = (long long *)calloc(n_patches + 1, sizeof(long long));
  p->h_vol_off = (long long *)calloc(n_problems + 1, sizeof(long long));
  // problems
  long long vo = 0;
  int nbr = 0;
  for (int b = 0; b < n_problems; ++b) {
    const pvr_grid &g = grids[b];
    if (g.nx <= 0 || g.ny <= 0 || g.nz <= 0) return fail(PVR_ESHAPE, "pvr_plan_create: grid %d has an empty size", b);
    if ((long long)g.nx * g.ny * g.nz > (1LL << 28))
      return fail(PVR_ESHAPE, "pvr_plan_create: grid %d has more than 2^28 voxels", b);
    ProbDev &d = p->h_prob[b];
    d.nx = g.nx; d.ny = g.ny; d.nz = g.nz;
    d.nbx = (g.nx + BRICK - 1) / BRICK; d.nby = (g.ny + BRICK - 1) / BRICK; d.nbz = (g.nz + BRICK - 1) / BRICK;
    d.brick_base = nbr;
    d.n_bricks = d.nbx * d.nby * d.nbz;
    nbr += d.n_bricks;
    d.vol_off = vo;
    p->h_vol_off[b] = vo;
    vo += (long long)g.nx * g.ny * g.nz;
    memcpy(d.v2w, g.vox2world, sizeof(d.v2w));
    double L[9], Li[9];
    host_mat3_from_aff(g.vox2world, L);
    double det = mat3_inv(L, Li);
    if (!(fabs(det) > 1e-12)) return fail(PVR_ESHAPE, "pvr_plan_create: grid %d vox2world is singular", b);
    aff_inv(g.vox2world, d.w2v);
  }
  p->h_vol_off[n_problems] = vo;
  p->V = vo;
  p->n_bricks = nbr;
  // stacks
  for (int s = 0; s < n_stacks; ++s) {
    const pvr_stack &st = stacks[s];
    if (st.problem < 0 || st.problem >= n_problems) return fail(PVR_EINVAL, "pvr_plan_create: stack %d names problem %d", s, st.problem);
    if (st.nx <= 0 || st.ny <= 0 || st.nslices <= 0) return fail(PVR_ESHAPE, "pvr_plan_create: stack %d has an empty size", s);
    StackDev &d = p->h_stack[s];
    d.problem = st.problem; d.nx = st.nx; d.ny = st.ny; d.ns = st.nslices;
    memcpy(d.p2w, st.pix2world, sizeof(d.p2w));
    double L[9];
    host_mat3_from_aff(st.pix2world, L);
    for (int a = 0; a < 3; ++a) {
      double n = sqrt(L[a] * L[a] + L[3 + a] * L[3 + a] + L[6 + a] * L[6 + a]);
      if (!(n > 0)) return fail(PVR_ESHAPE, "pvr_plan_create: stack %d axis %d has zero length", s, a);
      d.spacing[a] = n;
      for (int r = 0; r < 3; ++r) d.E[3 * r + a] = L[3 * r + a] / n;
      if (!(st.fwhm_mm[a] > 0)) return fail(PVR_EINVAL, "pvr_plan_create: stack %d fwhm[%d] <= 0", s, a);
      d.sigma[a] = st.fwhm_mm[a] / (2.0 * sqrt(2.0 * log(2.0)));
      if (a < 2) d.wz[a] = st.fwhm_mm[a];
    }
    for (int a = 0; a < 3; ++a)
      for (int c = a + 1; c < 3; ++c) {
        double dt = d.E[a] * d.E[c] + d.E[3 + a] * d.E[3 + c] + d.E[6 + a] * d.E[6 + c];
        if (fabs(dt) > 1e-9) return fail(PVR_ESHAPE, "pvr_plan_create: stack %d axes %d and %d are not orthogonal", s, a, c);
      }
  }
  // the adjoint's candidate grid depends on the stacks only
  p->max_hu = p->max_hv = 0;
  {
    const double sk = sqrt(KAPPA), K2 = KAPPA * cutoff_k * cutoff_k;
    for (int s = 0; s < n_stacks; ++s) {
      const StackDev &d = p->h_stack[s];
      p->max_hu = std::max(p->max_hu, cand_halfwidth(K2, sk * d.spacing[0] / d.sigma[0]));
      p->max_hv = std::max(p->max_hv, cand_halfwidth(K2, sk * d.spacing[1] / d.sigma[1]));
    }
  }
  // patches: grouped by problem in problem order, each inside its slice
  long long so = 0;
  int prev_prob = 0;
  std::vector<BlockWork> blocks, pblocks;
  std::vector<int> pcount(n_problems, 0);
  std::vector<long long> scount(n_problems, 0);
  for (int s = 0; s < n_patches; ++s) {
    const pvr_patch &q = patches[s];
    if (q.stack < 0 || q.stack >= n_stacks) return fail(PVR_EINVAL, "pvr_plan_create: patch %d names stack %d", s, q.stack);
    const StackDev &st = p->h_stack[q.stack];
    if (q.w <= 0 || q.h <= 0 || q.x0 < 0 || q.y0 < 0 || q.x0 + q.w > st.nx || q.y0 + q.h > st.ny ||
        q.slice < 0 || q.slice >= st.ns)
      return fail(PVR_ESHAPE, "pvr_plan_create: patch %d does not fit its slice", s);
    const int prob = st.problem;
    if (prob < prev_prob) return fail(PVR_EINVAL, "pvr_plan_create: patches must be ordered by problem (patch %d)", s);
    prev_prob = prob;
    PatchDev &d = p->h_patch[s];
    d.stack = q.stack; d.slice = q.slice; d.x0 = q.x0; d.y0 = q.y0; d.w = q.w; d.h = q.h;
    d.problem = prob; d.off = so;
    d.rq_off = p->n_rq;
    p->n_rq += rq_entries(q.w, q.h);
    {
      // rows of the patch run along the stack's u axis: when that is closer
      // to voxel y than to voxel x, the forward walks read the y-fastest copy
      const double *W = p->h_prob[prob].w2v, *A = st.p2w;
      double du[3];
      for (int r = 0; r < 3; ++r) du[r] = W[4 * r] * A[0] + W[4 * r + 1] * A[4] + W[4 * r + 2] * A[8];
      d.layout = fabs(du[1]) > fabs(du[0]) ? 1 : 0;
      if (d.layout) p->any_xt = true;
    }
    p->h_sample_off[s] = so;
    const int n = q.w * q.h;
    for (int l0 = 0; l0 < n; l0 += SIM_CHUNK) blocks.push_back(BlockWork{s, l0});
    const int nblk = ((q.w + 1) / 2) * ((q.h + 1) / 2);
    for (int l0 = 0; l0 < nblk; l0 += PLANE_BLOCKS) pblocks.push_back(BlockWork{s, l0});
    so += n;
    pcount[prob] += 1;
    scount[prob] += n;
  }
  {
    int pb = 0;
    long long sb = 0;
    p->max_problem_patches = 0;
    for (int b = 0; b < n_problems; ++b) {
      if (pcount[b] > PVR_MAX_PROBLEM_PATCHES)
        return fail(PVR_ESHAPE, "pvr_plan_create: problem %d has more than %d patches", b,
                    PVR_MAX_PROBLEM_PATCHES);
      p->max_problem_patches = std::max(p->max_problem_patches, pcount[b]);
      p->h_prob[b].patch_begin = pb; p->h_prob[b].patch_end = pb + pcount[b];
      p->h_prob[b].sample_begin = sb; p->h_prob[b].sample_end = sb + scount[b];
      pb += pcount[b];
      sb += scount[b];
    }
  }
  {
    // forward chunks are patch-major, so every problem's chunks form a range
    int c = 0;
    for (int b = 0; b < n_problems; ++b) {
      p->h_prob[b].chunk_begin = c;
      while (c < (int)blocks.size() && blocks[c].patch < p->h_prob[b].patch_end) ++c;
      p->h_prob[b].chunk_end = c;
    }
    c = 0;
    for (int b = 0; b < n_problems; ++b) {
      p->h_prob[b].pblk_begin = c;
      while (c < (int)pblocks.size() && pblocks[c].patch < p->h_prob[b].patch_end) ++c;
      p->h_prob[b].pblk_end = c;
    }
  }
  p->h_sample_off[n_patches] = so;
  p->N = so;
  if (so > 0x7fffffffLL * 4) return fail(PVR_ESHAPE, "pvr_plan_create: too many samples");
  p->n_sim_blocks = (int)blocks.size();
  p->n_pblocks = (int)pblocks.size();
  for (int s = 0; s < n_patches; ++s)
    if (patches[s].w > 32767 || patches[s].h > 32767 ||
        (long long)patches[s].w * patches[s].h > (1LL << 26))
      return fail(PVR_ESHAPE, "pvr_plan_create: patch %d too large (w, h <= 32767, w * h <= 2^26)", s);
  p->tile_w = TILE;
  p->tile_h = TILE;
  p->use_tiles = false;
  p->sim_granule = SIM_XCD_GRANULE;
  p->bp_granule = BP_XCD_GRANULE;
  p->h_item_off = (int *)calloc(n_patches + 1, sizeof(int));
  for (const BlockWork &w : blocks) p->h_item_off[w.patch + 1] += 1;
  for (int s = 0; s < n_patches; ++s) p->h_item_off[s + 1] += p->h_item_off[s];
  p->h_tile_off = (int *)calloc(n_patches + 1, sizeof(int));
  {
    const pvr_status st = make_tiles(p, TILE, TILE);
    if (st != PVR_OK) return st;
  }
  std::vector<int> plane_prob;
  std::vector<int> plane_first(n_problems);
  p->max_nx = p->max_ny = 0;
  for (int b = 0; b < n_problems; ++b) {
    plane_first[b] = (int)plane_prob.size();
    for (int z = 0; z < p->h_prob[b].nz; ++z) plane_prob.push_back(b);
    p->max_nx = std::max(p->max_nx, p->h_prob[b].nx);
    p->max_ny = std::max(p->max_ny, p->h_prob[b].ny);
  }
  p->n_planes = (int)plane_prob.size();
  if (p->n_planes > 65535) return fail(PVR_ESHAPE, "pvr_plan_create: more than 65535 z-planes in total");
  plane_prob.insert(plane_prob.end(), plane_first.begin(), plane_first.end());
  p->h_plane_prob = (int *)malloc(sizeof(int) * plane_prob.size());
  std::copy(plane_prob.begin(), plane_prob.end(), p->h_plane_prob);
  p->h_brick_prob = (int *)malloc(sizeof(int) * (size_t)std::max(nbr, 1));
  for (int b = 0; b < n_problems; ++b)
    for (int i = 0; i < p->h_prob[b].n_bricks; ++i) p->h_brick_prob[p->h_prob[b].brick_base + i] = b;
  p->h_sim_blocks = (BlockWork *)malloc(sizeof(BlockWork) * std::max<size_t>(blocks.size(), 1));
  std::copy(blocks.begin(), blocks.end(), p->h_sim_blocks);
  p->h_pblocks = (BlockWork *)malloc(sizeof(BlockWork) * std::max<size_t>(pblocks.size(), 1));
  std::copy(pblocks.begin(), pblocks.end(), p->h_pblocks);
  // capacity of the adjoint's index: bounds over every motion, so that no
  // build needs to read a count back or to grow a list
  {
    long long bins = 0, subs = 0;
    for (int s = 0; s < n_patches; ++s) {
      const PatchDev &q = p->h_patch[s];
      const ProbDev &pr = p->h_prob[q.problem];
      const long long b = pair_bound(pr, p->h_stack[q.stack], q, cutoff_k, BRICK, pr.n_bricks);
      bins += b;
      // the 4^3 lists, or the block gather's (at most two halves of every brick)
      subs += std::max(2 * b, std::min(8 * b, pair_bound(pr, p->h_stack[q.stack], q, cutoff_k, SUB,
                                                         8LL * pr.n_bricks)));
    }
    p->bin_cap = std::min(bins, (long long)INDEX_CAP_MAX);
    p->sub_cap = std::min(subs, (long long)INDEX_CAP_MAX);
  }
  choose_walks(p);
  p->device = -1;  // the device of the first workspace
  guard.release();
  *out = p;
  return PVR_OK;
  PVR_API_END();
}

// The plan's device state, in one fixed order: with a NULL base this only
// measures the workspace (the same calls size and carve it).
static size_t layout(pvr_plan *p, char *base, int flags) {
  WsCursor c{base, 0};
  const long long M = p->M, N = p->N, nb = p->n_bricks;
  p->d_prob = ws_take<ProbDev>(c, p->P);
  p->d_stack = ws_take<StackDev>(c, p->S);
  p->d_patch = ws_take<PatchDev>(c, M);
  p->d_sim_blocks = ws_take<BlockWork>(c, p->n_sim_blocks);
  p->d_pblocks = ws_take<BlockWork>(c, p->n_pblocks);
  p->d_item_off = ws_take<int>(c, M + 1);
  p->d_tile_off = ws_take<int>(c, M + 1);
  p->d_box_max = ws_take<int>(c, 4);
  p->d_brick_prob = ws_take<int>(c, nb);
  p->d_plane_prob = ws_take<int>(c, p->n_planes + p->P);
  p->d_theta = ws_take<double>(c, 6 * M);
  p->d_geod = ws_take<GeoD>(c, M);
  p->d_geof = ws_take<GeoF>(c, M);
  p->d_adj = ws_take<AdjPatch<float>>(c, M);
  p->d_adj64 = ws_take<AdjPatch<double>>(c, M);
  p->d_fwd = ws_take<FwdPatch<float>>(c, M);
  p->d_sinc = ws_take<SincPatch>(c, M);
  p->d_fwd64 = ws_take<FwdPatch<double>>(c, M);
  p->d_bb = ws_take<int>(c, 6 * M);
  p->d_gbox = ws_take<int>(c, 6 * ((M + 63) / 64));
  p->d_sbox = ws_take<double>(c, 18 * M);
  p->d_invz = ws_take<float>(c, N);
  p->d_mask = ws_take<uint8_t>(c, N);
  p->d_active = ws_take<uint8_t>(c, M);
  p->d_sub_off = ws_take<int>(c, 9 * nb);
  p->d_sub_patch = ws_take<int>(c, p->sub_cap);
  p->d_rq = ws_take<float2>(c, p->n_rq);
  p->d_odd = ws_take<unsigned>(c, 2);
  p->d_pstat = ws_take<double>(c, 9 * M);
  p->d_pval = ws_take<double>(c, M);
  p->d_chunk_stats = ws_take<double>(c, 5LL * std::max(p->n_sim_blocks, p->n_pblocks));
  p->d_xt = p->any_xt ? ws_take<float>(c, p->V) : nullptr;
  p->d_cursor = ws_take<unsigned long long>(c, 2);
  p->d_reg_stats = ws_take<unsigned long long>(c, 4);
  {
    size_t off[5];
    p->d_reg = ws_take<char>(c, (long long)reg_state_bytes(p, off));
  }
  p->d_status = ws_take<unsigned>(c, 1);
  p->d_dbg = ws_take<unsigned long long>(c, 1);
  p->d_invz64 = (flags & PVR_WS_F64) ? ws_take<double>(c, N) : nullptr;
  // one guard entry (zero) before and after the N entries: the FP64 adjoint's
  // candidates may reach one entry past a patch
  p->d_rq64 = (flags & PVR_WS_F64) ? ws_take<double2>(c, N + 2) : nullptr;
  return (c.off + 255) & ~(size_t)255;
}

extern "C" pvr_status pvr_plan_workspace_size(const pvr_plan *p, int32_t flags, size_t *bytes) {
  PVR_API_BEGIN();
  if (!p || !bytes) return fail(PVR_EINVAL, "pvr_plan_workspace_size: NULL argument");
  if (flags & ~PVR_WS_F64) return fail(PVR_EINVAL, "pvr_plan_workspace_size: unknown flags 0x%x", flags);
  pvr_plan q = *p;  // layout() writes pointers: measure on a copy
  *bytes = layout(&q, nullptr, flags);
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_plan_attach(pvr_plan *p, void *workspace, size_t bytes, int32_t flags,
                                      hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_plan_attach", workspace, 256);
  if (!p || !workspace) return fail(PVR_EINVAL, "pvr_plan_attach: NULL argument");
  if (flags & ~PVR_WS_F64) return fail(PVR_EINVAL, "pvr_plan_attach: unknown flags 0x%x", flags);
  {
    pvr_plan q = *p;
    const size_t need = layout(&q, nullptr, flags);
    if (bytes < need)
      return fail(PVR_ESHAPE, "pvr_plan_attach: workspace of %zu bytes, %zu needed", bytes, need);
  }
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (p->device >= 0 && dev != p->device)
    return fail(PVR_EINVAL, "pvr_plan_attach: device %d is current, the plan belongs to device %d",
                dev, p->device);
  if (p->attached) HIP_TRY(hipStreamSynchronize(stream));  // the old workspace may be in use
  if (!p->side) {
    HIP_TRY(hipStreamCreateWithFlags(&p->side, hipStreamNonBlocking));
    HIP_TRY(hipEventCreateWithFlags(&p->ev_fork, hipEventDisableTiming));
    HIP_TRY(hipEventCreateWithFlags(&p->ev_join, hipEventDisableTiming));
  }
  p->device = dev;
  layout(p, (char *)workspace, flags);
  p->ws = workspace;
  p->ws_bytes = bytes;
  p->ws_flags = flags;
  const int M = p->M;
  HIP_TRY(hipMemcpyAsync(p->d_prob, p->h_prob, sizeof(ProbDev) * p->P, hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_stack, p->h_stack, sizeof(StackDev) * p->S, hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_patch, p->h_patch, sizeof(PatchDev) * M, hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_sim_blocks, p->h_sim_blocks, sizeof(BlockWork) * p->n_sim_blocks,
                         hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_item_off, p->h_item_off, sizeof(int) * (M + 1), hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_pblocks, p->h_pblocks, sizeof(BlockWork) * p->n_pblocks,
                         hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_tile_off, p->h_tile_off, sizeof(int) * (M + 1), hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_brick_prob, p->h_brick_prob, sizeof(int) * p->n_bricks,
                         hipMemcpyHostToDevice, stream));
  HIP_TRY(hipMemcpyAsync(p->d_plane_prob, p->h_plane_prob, sizeof(int) * (p->n_planes + p->P),
                         hipMemcpyHostToDevice, stream));
  launch_fill_f32((float *)p->d_rq, 0.f, 2 * p->n_rq, stream);
  if (p->d_rq64) launch_fill_f64((double *)p->d_rq64, 0.0, 2 * (p->N + 2), stream);
  launch_fill_i32((int *)p->d_status, 0, 1, stream);
  launch_fill_i32((int *)p->d_cursor, 0, 4, stream);
  launch_fill_i32((int *)p->d_odd, 0, 2, stream);
  launch_fill_i32((int *)p->d_reg_stats, 0, 8, stream);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipStreamSynchronize(stream));  // the uploads read pageable host tables of the plan
  p->attached = true;
  p->built = p->built64 = false;
  p->index_valid = false;
  p->stats_valid = false;
  p->rq_fresh = false;
  ++p->generation;
  return PVR_OK;
  PVR_API_END();
}

extern "C" void pvr_plan_destroy(pvr_plan *p) {
  if (!p) return;
  plan_free(p);
}

extern "C" pvr_status pvr_plan_info(const pvr_plan *p, pvr_plan_sizes *out) {
  PVR_API_BEGIN();
  if (!p || !out) return fail(PVR_EINVAL, "pvr_plan_info: NULL argument");
  out->n_samples = p->N;
  out->n_voxels = p->V;
  out->n_patches = p->M;
  out->n_problems = p->P;
  out->n_stacks = p->S;
  out->n_bricks = p->n_bricks;
  out->n_bin_pairs = 0;
  if (p->attached && p->index_valid) {
    unsigned long long n = 0;
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(&n, p->d_cursor + 1, sizeof n, hipMemcpyDeviceToHost));
    out->n_bin_pairs = std::min((long long)n, p->sub_cap);
  }
  out->device_bytes = p->attached ? (int64_t)p->ws_bytes : 0;
  out->bin_capacity = p->bin_cap;
  out->sub_capacity = p->sub_cap;
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_plan_offsets(const pvr_plan *p, int64_t *sample_off, int64_t *vol_off) {
  PVR_API_BEGIN();
  if (!p) return fail(PVR_EINVAL, "pvr_plan_offsets: plan is NULL");
  if (sample_off) for (int s = 0; s <= p->M; ++s) sample_off[s] = p->h_sample_off[s];
  if (vol_off) for (int b = 0; b <= p->P; ++b) vol_off[b] = p->h_vol_off[b];
  return PVR_OK;
  PVR_API_END();
}

extern "C" const float *pvr_plan_inv_z(const pvr_plan *p) {
  return p && p->attached ? p->d_invz : nullptr;
}

// Forward tiles: every patch cut into tile_w x tile_h rectangles (edge tiles
// smaller), row of tiles after row of tiles; h_tile_off counts the tiles
// before each patch (a workgroup finds its tile with tile_at).
static pvr_status make_tiles(pvr_plan *p, int tile_w, int tile_h) {
  long long t = 0;
  for (int s = 0; s < p->M; ++s) {
    const PatchDev &q = p->h_patch[s];
    const int tw = std::min(q.w, tile_w), th = std::min(q.h, tile_h);
    p->h_tile_off[s] = (int)t;
    t += (long long)((q.w + tw - 1) / tw) * ((q.h + th - 1) / th);
    if (t > 0x7fffffffLL)
      return fail(PVR_ESHAPE, "forward tiles of %dx%d: more than 2^31 tiles", tile_w, tile_h);
  }
  p->h_tile_off[p->M] = (int)t;
  p->n_tiles = (int)t;
  p->tile_w = tile_w;
  p->tile_h = tile_h;
  return PVR_OK;
}

static pvr_status update_lds_box(pvr_plan *p, hipStream_t stream) {
  const int T = 256;
  launch_fill_i32(p->d_box_max, 0, 1, stream);
  hipLaunchKernelGGL(k_tile_boxmax, dim3((p->n_tiles + T - 1) / T), dim3(T), 0, stream, p->d_prob,
                     p->d_patch, p->d_tile_off, p->M, p->tile_w, p->tile_h, p->n_tiles, p->d_geof,
                     p->d_box_max);
  HIP_TRY(hipGetLastError());
  HIP_TRY(hipMemcpyAsync(p->h_total + 2, p->d_box_max, sizeof(int), hipMemcpyDeviceToHost, stream));
  HIP_TRY(hipStreamSynchronize(stream));
  p->lds_box = std::min(p->h_total[2], LDS_BOX_MAX);
  return PVR_OK;
}

extern "C" pvr_status pvr_plan_set_psf(pvr_plan *p, int32_t kind) {
  PVR_API_BEGIN();
  if (!p) return fail(PVR_EINVAL, "pvr_plan_set_psf: plan is NULL");
  if (kind != PVR_PSF_GAUSSIAN && kind != PVR_PSF_SINC)
    return fail(PVR_EINVAL, "pvr_plan_set_psf: kind must be PVR_PSF_GAUSSIAN or PVR_PSF_SINC");
  p->psf = kind;
  // the adjoint's candidate grid follows the PSF's in-plane reach
  const double sk = sqrt(KAPPA), K2 = KAPPA * p->k * p->k;
  p->max_hu = p->max_hv = 0;
  for (int s = 0; s < p->S; ++s) {
    const StackDev &d = p->h_stack[s];
    const int hu = kind == PVR_PSF_SINC ? sinc_halfwidth(d.spacing[0] / d.wz[0])
                                        : cand_halfwidth(K2, sk * d.spacing[0] / d.sigma[0]);
    const int hv = kind == PVR_PSF_SINC ? sinc_halfwidth(d.spacing[1] / d.wz[1])
                                        : cand_halfwidth(K2, sk * d.spacing[1] / d.sigma[1]);
    p->max_hu = std::max(p->max_hu, hu);
    p->max_hv = std::max(p->max_hv, hv);
  }
  choose_walks(p);
  p->built = p->built64 = false;
  p->index_valid = false;
  p->stats_valid = false;
  p->rq_fresh = false;
  ++p->generation;
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_plan_set_tiles(pvr_plan *p, int32_t tile_w, int32_t tile_h,
                                         hipStream_t stream) {
  PVR_API_BEGIN();
  if (!p) return fail(PVR_EINVAL, "pvr_plan_set_tiles: plan is NULL");
  if (!p->attached) return fail(PVR_EINVAL, "pvr_plan_set_tiles: no workspace attached");
  ++p->generation;
  if (tile_w == 0 && tile_h == 0) {
    p->use_tiles = false;
    return PVR_OK;
  }
  if (tile_w <= 0 || tile_h <= 0 || tile_w * tile_h > 256)
    return fail(PVR_EINVAL, "pvr_plan_set_tiles: need 0 < tile_w * tile_h <= 256 (or 0 x 0)");
  HIP_TRY(hipStreamSynchronize(stream));  // earlier launches may still read the tile table
  const pvr_status st = make_tiles(p, tile_w, tile_h);
  if (st != PVR_OK) {
    p->use_tiles = false;
    return st;
  }
  HIP_TRY(hipMemcpyAsync(p->d_tile_off, p->h_tile_off, sizeof(int) * (p->M + 1),
                         hipMemcpyHostToDevice, stream));
  p->use_tiles = true;
  if (p->built) return update_lds_box(p, stream);
  HIP_TRY(hipStreamSynchronize(stream));
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_plan_set_granules(pvr_plan *p, int32_t sim_granule,
                                            int32_t bp_granule) {
  PVR_API_BEGIN();
  if (!p) return fail(PVR_EINVAL, "pvr_plan_set_granules: plan is NULL");
  if (sim_granule < 1 || sim_granule > 4096 || bp_granule < 1 || bp_granule > 4096)
    return fail(PVR_EINVAL, "pvr_plan_set_granules: granules must lie in [1, 4096]");
  p->sim_granule = sim_granule;
  p->bp_granule = bp_granule;
  ++p->generation;
  return PVR_OK;
  PVR_API_END();
}

// The gather adjoint's lists for the geometry of the last build, into a list
// array of the capacity bounded at plan creation: no count is read back,
// nothing is synchronised.
pvr_status pvr::plan_build_index(pvr_plan *p, hipStream_t stream) {
  const int nb = p->n_bricks;
  const dim3 grid((nb + LIST_BRICKS - 1) / LIST_BRICKS), block(64 * LIST_BRICKS);
#define LIST_LAUNCH(NL)                                                                            \
  hipLaunchKernelGGL(k_adj_lists<NL>, grid, block, 0, stream, p->d_prob, p->d_brick_prob, p->d_bb, \
                     p->d_gbox, p->d_sbox, p->d_adj, nb, p->d_cursor, p->d_sub_off, p->d_sub_patch, \
                     p->sub_cap, p->d_status)
  if (p->gather_blocks) LIST_LAUNCH(6);
  else LIST_LAUNCH(8);
#undef LIST_LAUNCH
  HIP_TRY(hipGetLastError());
  p->index_valid = true;
  p->index_capture = capture_id(stream);
  ++p->generation;
  return PVR_OK;
}

template <typename TH>
static pvr_status plan_build_common(pvr_plan *p, const TH *theta, const uint8_t *active,
                                    const uint8_t *mask, hipStream_t stream) {
  const int M = p->M;
  const bool f64 = sizeof(TH) == 8;
  const bool wide = f64 && p->d_invz64;
  hipLaunchKernelGGL(k_geometry<TH>, dim3((M + 63) / 64), dim3(256), 0, stream, p->d_prob, p->d_stack,
                     p->d_patch, theta, active, M, p->k, p->psf, wide ? 1 : 0, p->d_theta,
                     p->d_active, p->d_geod, p->d_geof, p->d_adj, p->d_adj64, p->d_fwd, p->d_fwd64, p->d_sinc,
                     p->d_bb, p->d_gbox,
                     p->d_sbox);
  HIP_TRY(hipGetLastError());
  // an FP64 build also writes FP64 normalisers when the workspace has room
  // for them (PVR_WS_F64); the FP32 ones are written either way
#define NORM_LAUNCH(T, GEO, FWD, OUT64)                                                            \
  if (wide ? p->planes64 : p->planes)                                                              \
    hipLaunchKernelGGL(k_normalisers_planes<T>, dim3(p->n_pblocks), dim3(PLANE_BLOCKS),              \
                       PLANE_BLOCKS * 4 * sizeof(T), stream,                                       \
                       p->d_prob, p->d_patch, p->d_pblocks, GEO, FWD, mask, p->d_active, p->d_mask,  \
                       p->d_invz, OUT64);                                                          \
  else                                                                                             \
    hipLaunchKernelGGL(k_normalisers<T>, dim3(p->n_sim_blocks), dim3(SIM_THREADS), 0, stream,      \
                       p->d_prob, p->d_patch, p->d_sim_blocks, GEO, p->d_sinc, mask, p->d_active, p->d_mask,    \
                       p->d_invz, OUT64)
  if (wide) { NORM_LAUNCH(double, p->d_geod, p->d_fwd64, p->d_invz64); }
  else { NORM_LAUNCH(float, p->d_geof, p->d_fwd, (double *)nullptr); }
#undef NORM_LAUNCH
  HIP_TRY(hipGetLastError());
  // forward-tile boxes (LDS size of the staged forward pass)
  if (p->use_tiles) {
    const pvr_status st = update_lds_box(p, stream);
    if (st != PVR_OK) return st;
  }
  p->index_valid = false;
  p->stats_valid = false;
  p->rq_fresh = false;
  p->built = true;
  p->built64 = f64 && p->d_invz64;
  ++p->generation;
  return PVR_OK;
}

extern "C" pvr_status pvr_plan_build(pvr_plan *p, const float *theta, const uint8_t *active,
                                     const uint8_t *sample_mask, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_plan_build", theta, 4);
  if (!p || !theta) return fail(PVR_EINVAL, "pvr_plan_build: NULL plan or theta");
  if (!p->attached) return fail(PVR_EINVAL, "pvr_plan_build: no workspace attached (pvr_plan_attach)");
  PVR_TRY_STATUS(debug_finite(p, "pvr_plan_build", "theta", theta, 6LL * p->M, stream));
  return plan_build_common(p, theta, active, sample_mask, stream);
  PVR_API_END();
}

extern "C" pvr_status pvr_plan_build_f64(pvr_plan *p, const double *theta, const uint8_t *active,
                                         const uint8_t *sample_mask, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_plan_build_f64", theta, 8);
  if (!p || !theta) return fail(PVR_EINVAL, "pvr_plan_build_f64: NULL plan or theta");
  if (!p->attached) return fail(PVR_EINVAL, "pvr_plan_build_f64: no workspace attached (pvr_plan_attach)");
  PVR_TRY_STATUS(debug_finite(p, "pvr_plan_build_f64", "theta", theta, 6LL * p->M, stream));
  return plan_build_common(p, theta, active, sample_mask, stream);
  PVR_API_END();
}
