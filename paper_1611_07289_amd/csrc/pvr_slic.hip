// Superpixel patch extraction: SLIC on every observed slice (see
// include/pvr_slic.h for the definition).  Assignment is a gather over pixel
// tiles: the centres that can reach a tile are listed in LDS in ascending
// order, and every pixel keeps the first of least D^2 (FP32 bits; D^2 >= 0, so
// they order like the values, a NaN after infinity).  The update gathers too:
// one workgroup per centre sums the pixels of its window that carry its label.
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "pvr_internal.h"
#include "pvr_slic.h"
#include "pvr_util.h"

#include <algorithm>
#include <mutex>
#include <type_traits>

using namespace pvr;

namespace {

constexpr int SLIC_T = 256;

__device__ __forceinline__ void cell_of(int k, int kx, int a, int h, int w, float &x, float &y) {
  const int i = k % kx, j = k / kx;
  x = 0.5f * (float)(i * a + min(w, (i + 1) * a) - 1);
  y = 0.5f * (float)(j * a + min(h, (j + 1) * a) - 1);
}

// window of a centre: integer pixel ranges with |x - cx| <= a, clipped to the
// image (empty when x0 > x1 or y0 > y1).  The centre is first clamped to a
// band around the image that leaves every window inside the image unchanged,
// so that any input (NaN, infinities, far-off centres) gives small integers.
__device__ __forceinline__ void window(float cx, float cy, int a, int h, int w, int &x0, int &x1,
                                       int &y0, int &y1) {
  const float fa = (float)a;
  cx = fminf(fmaxf(cx, -2.f * fa - 1.f), (float)w + 2.f * fa);
  cy = fminf(fmaxf(cy, -2.f * fa - 1.f), (float)h + 2.f * fa);
  x0 = max(0, (int)ceilf(cx - fa));
  x1 = min(w - 1, (int)floorf(cx + fa));
  y0 = max(0, (int)ceilf(cy - fa));
  y1 = min(h - 1, (int)floorf(cy + fa));
}

// The image and the item (centre or pixel block, `per` of them an image) of a
// workgroup of a per x n_img grid.  Workgroups go to the XCDs in turn, so of
// eight images each is worked on by one XCD, in whose L2 its pixels and labels
// are read several times over; the images beyond a multiple of eight keep the
// grid's order.
__device__ __forceinline__ void image_item(int per, int n_img, int &im, int &item) {
  im = blockIdx.y;
  item = blockIdx.x;
  const unsigned L = blockIdx.y * (unsigned)per + blockIdx.x;  // at most 2^31 - 1
  if (im < (n_img & ~7)) {
    const unsigned slot = L >> 3;
    im = (int)(slot / (unsigned)per) * 8 + (int)(L & 7);
    item = (int)(slot % (unsigned)per);
  }
}

// Wavefront reductions over data-parallel primitives (rows of 16 lanes, then
// the rows): the sum and the greatest of the 64 lanes' values.
template <int CTRL, int ROWS_ON>
__device__ __forceinline__ int dpp(int idle, int v) {
  return __builtin_amdgcn_update_dpp(idle, v, CTRL, ROWS_ON, 0xf, false);
}
__device__ __forceinline__ int wave_sum(int v) {
  v += dpp<0x111, 0xf>(0, v);  // row_shr 1, 2, 4, 8
  v += dpp<0x112, 0xf>(0, v);
  v += dpp<0x114, 0xf>(0, v);
  v += dpp<0x118, 0xf>(0, v);
  v += dpp<0x142, 0xa>(0, v);  // row_bcast 15, 31
  v += dpp<0x143, 0xc>(0, v);
  return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ float wave_max(float v) {
  const auto take = [&](int o) {
    const float f = __int_as_float(o);
    v = f > v ? f : v;
  };
  take(dpp<0x111, 0xf>(__float_as_int(v), __float_as_int(v)));
  take(dpp<0x112, 0xf>(__float_as_int(v), __float_as_int(v)));
  take(dpp<0x114, 0xf>(__float_as_int(v), __float_as_int(v)));
  take(dpp<0x118, 0xf>(__float_as_int(v), __float_as_int(v)));
  take(dpp<0x142, 0xa>(__float_as_int(v), __float_as_int(v)));
  take(dpp<0x143, 0xc>(__float_as_int(v), __float_as_int(v)));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

}  // namespace

__global__ void k_slic_init(const float *__restrict__ img, int n_img, int h, int w, int a, int kx,
                            int K, float t0, float *__restrict__ C) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)n_img * K) return;
  const int im = (int)(t / K), k = (int)(t % K);
  float x, y;
  cell_of(k, kx, a, h, w, x, y);
  const int px = (int)floorf(x + 0.5f), py = (int)floorf(y + 0.5f);
  float *c = C + 4 * t;
  c[0] = x;
  c[1] = y;
  c[2] = img[((long long)im * h + py) * w + px];
  c[3] = t0;
}

// Largest distance of a centre from its grid cell's middle, per image: a
// centre whose window covers a pixel sits in a cell at most a + drift away.
__global__ void __launch_bounds__(SLIC_T)
k_slic_drift(const float *__restrict__ C, int h, int w, int a, int kx, int K,
             float *__restrict__ drift) {
  __shared__ float red[SLIC_T / 64];
  const int im = blockIdx.x;
  float d = 0.0f;
  for (int k = threadIdx.x; k < K; k += SLIC_T) {
    const float *c = C + 4 * ((long long)im * K + k);
    float gx, gy;
    cell_of(k, kx, a, h, w, gx, gy);
    const float e = fmaxf(fabsf(c[0] - gx), fabsf(c[1] - gy));
    d = (e == e) ? fmaxf(d, e) : INFINITY;  // a NaN centre widens the search to all cells
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) d = fmaxf(d, __shfl_xor(d, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = d;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < SLIC_T / 64; ++q) d = fmaxf(d, red[q]);
    drift[im] = fmaxf(d, red[0]);
  }
}

// Assignment as a gather: a wavefront takes TILE_X x TILE_Y pixels (four a
// lane, TILE_X / 4 apart in x), a workgroup four such tiles below each other.
// Each wavefront lists the centres whose window can reach its tile in LDS, in
// ascending order (64 centres at a time: all of the image, or, DRIFT, those of
// the cells within a + drift of the tile), then every pixel takes the first of
// least D^2.  Bound by vector issue, about 10 instructions per pixel and listed
// centre (6.75 of them a tile at full reach, of which a pixel is inside 4 windows):
// 240 images of 256 x 256, a = 32, 34 us; 86 with one pixel per lane, packed
// 64-bit keys and one list per workgroup.
constexpr int TILE_X = 32, TILE_Y = 8, TILE_WAVES = SLIC_T / 64;
// All centres are listed up to this many an image (four rounds of 64, no
// drift launch, which takes 5 us); beyond it the cells near the tile are.
constexpr int SLIC_LIST_ALL = 256;

// v, but no NaN whose bits without the sign are all ones (quietened or not): a D^2 of
// all ones is a pixel's start and would not be taken.
__device__ __forceinline__ float not_all_ones(float v) {
  const unsigned b = __float_as_uint(v);
  return (b | 0x80400000u) == ~0u ? __uint_as_float(b & ~1u) : v;
}

template <bool DRIFT>
__global__ void __launch_bounds__(SLIC_T)
k_slic_gather(const float *__restrict__ img, int n_img, int h, int w, int a, int kx, int ky, int K,
              const float *__restrict__ C, const float *__restrict__ drift,
              int32_t *__restrict__ labels) {
  __shared__ float4 list_c[TILE_WAVES][64];  // (cx, cy, ci, t^2 / a^2)
  __shared__ int list_k[TILE_WAVES][64];
  const int tiles_x = (w + TILE_X - 1) / TILE_X, rows = TILE_WAVES * TILE_Y;
  int im, blk;
  image_item(tiles_x * ((h + rows - 1) / rows), n_img, im, blk);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tx0 = (blk % tiles_x) * TILE_X, ty0 = (blk / tiles_x) * rows + wv * TILE_Y;
  if (ty0 >= h) return;
  const int tx1 = min(w, tx0 + TILE_X) - 1, ty1 = min(h, ty0 + TILE_Y) - 1;
  const int x = tx0 + (lane & 7), y = ty0 + (lane >> 3);
  const long long row = ((long long)im * h + min(y, h - 1)) * w;
  float I[4];
  unsigned bits[4];
  int best[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float v = img[row + min(x + 8 * t, w - 1)];
    I[t] = v == v ? v : __builtin_nanf("");
    bits[t] = ~0u;
    best[t] = -1;
  }
  int i0 = 0, j0 = 0, ni = kx, ncand = K;
  if constexpr (DRIFT) {
    // cells i whose middle (in [i a, i a + (a-1)/2]) lies within a + drift of the tile
    int i1 = kx - 1, j1 = ky - 1;
    const float D = drift[im];
    if (D <= 4.0f * (float)(h + w)) {
      const float r = (float)a + D + 1.0f;
      i0 = max(0, (int)floorf(((float)tx0 - r - 0.5f * (float)(a - 1)) / (float)a));
      i1 = min(kx - 1, (int)floorf(((float)tx1 + r) / (float)a));
      j0 = max(0, (int)floorf(((float)ty0 - r - 0.5f * (float)(a - 1)) / (float)a));
      j1 = min(ky - 1, (int)floorf(((float)ty1 + r) / (float)a));
    }
    ni = i1 - i0 + 1;
    ncand = (ni > 0 && j1 >= j0) ? ni * (j1 - j0 + 1) : 0;
  }
  const float fa = (float)a;
  const float4 *Ci = reinterpret_cast<const float4 *>(C) + (long long)im * K;
  for (int c0 = 0; c0 < ncand; c0 += 64) {
    const int c = c0 + lane;
    int k = c;
    if constexpr (DRIFT) k = (j0 + c / ni) * kx + i0 + c % ni;
    float4 cc = c < ncand ? Ci[k] : float4{0, 0, 0, 0};
    // the window |x - cx| <= a meets the tile (one pixel of slack for rounding)
    const bool in = c < ncand && cc.x - fa <= (float)(tx1 + 1) && cc.x + fa >= (float)(tx0 - 1) &&
                    cc.y - fa <= (float)(ty1 + 1) && cc.y + fa >= (float)(ty0 - 1);
    const unsigned long long hit = __ballot(in);
    if (in) {
      const int slot = __popcll(hit & ((1ull << lane) - 1ull));
      cc.z = not_all_ones(cc.z);
      cc.w = not_all_ones(cc.w * cc.w / (float)(a * a));
      list_c[wv][slot] = cc;
      list_k[wv][slot] = k;
    }
    __builtin_amdgcn_wave_barrier();
    const int n = __popcll(hit);
    for (int e = 0; e < n; ++e) {
      const float4 cd = list_c[wv][e];
      const int ke = list_k[wv][e];
      const float dy = (float)y - cd.y, dy2 = dy * dy;
      const bool iny = fabsf(dy) <= fa;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float dx = (float)(x + 8 * t) - cd.x, dc = I[t] - cd.z;
        const unsigned d = __float_as_uint(fmaf(dc, dc, fmaf(dx, dx, dy2) * cd.w));
        const bool take = iny & (fabsf(dx) <= fa) & (d < bits[t]);
        bits[t] = take ? d : bits[t];
        best[t] = take ? ke : best[t];
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (y < h)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (x + 8 * t < w) labels[row + x + 8 * t] = best[t];
}

constexpr int ROWS = 8;  // rows a wavefront reads at once
constexpr int SLIC_SMALL = 512;

// Update: one workgroup per centre over its window, one pass: count, sums of
// x, y and I (FP64; the first three whole numbers, SMALL: in 32 bits, summed by
// data-parallel primitives), and the extreme intensities (max |I - mean| is
// reached at one of them).  Waves take rows, lanes consecutive pixels of a row.
// Each pixel lies in four windows on average: bound by instruction issue,
// scalar and vector alike, and then by the pixels' and labels' first read.
// Eight rows' labels and pixels are read at once and unconditionally (SMALL:
// buffer loads, the row in a scalar offset), and a row without a pixel of the
// centre ends after the comparison.  240 images of 256 x 256, 64 centres each:
// 42 us (126 MB of labels and pixels, 3.0 TB/s); 97 one row at a time, pixels
// only where the label is the centre's; 38 to 41 with one wavefront per centre.
constexpr int UPD_WAVES = SLIC_T / 64;
template <bool SMALL>
__global__ void __launch_bounds__(SLIC_T)
k_slic_update(const float *__restrict__ img, int n_img, int h, int w, int a, int K,
              const int32_t *__restrict__ labels, float t_min, float *__restrict__ C) {
  __shared__ double lds[4][UPD_WAVES];
  __shared__ float lim[2][UPD_WAVES];
  int im, k;
  image_item(K, n_img, im, k);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float *c = C + 4 * ((long long)im * K + k);
  int x0, x1, y0, y1;
  window(c[0], c[1], a, h, w, x0, x1, y0, y1);
  if (x0 > x1 || y0 > y1) return;  // no pixels: the centre stays
  using Sum = typename std::conditional<SMALL, int, double>::type;
  using Off = typename std::conditional<SMALL, int, long long>::type;
  Sum cnt = 0, sx = 0, sy = 0;  // of x and y less their starts x0, y0
  double sI = 0;
  float imax = -INFINITY, imin = INFINITY;
  const long long first = ((long long)im * h + y0) * w;  // of the window's rows
  const int32_t *lp = labels + first;
  const float *ip = img + first;
  const unsigned nbytes = SMALL ? (unsigned)(y1 - y0 + 1) * (unsigned)w * 4u : 0u;
  const __amdgpu_buffer_rsrc_t lr = raw_buffer(lp, nbytes), ir = raw_buffer(ip, nbytes);
  for (int x = x0 + lane; x <= x1; x += 64) {
    int col = 0;  // this column's pixels
    for (int yb = y0 + wave; yb <= y1; yb += ROWS * UPD_WAVES) {
      const int rows = min(ROWS, (y1 - yb) / UPD_WAVES + 1);
      int lab[ROWS], mine = 0, pre = 0;
      float I[ROWS];
      Off at = (Off)(yb - y0) * w;  // a clamped row repeats the last one
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        if constexpr (SMALL) {
          lab[r] = (int)__builtin_amdgcn_raw_buffer_load_b32(lr, 4 * x, 4 * (int)at, 0);
          I[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ir, 4 * x, 4 * (int)at, 0));
        } else {
          lab[r] = lp[at + x];
          I[r] = ip[at + x];
        }
        at += r + 1 < rows ? (Off)w * UPD_WAVES : 0;
      }
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const bool hit = (lab[r] == k) & (r < rows);
        mine += hit ? 1 : 0;
        if (__any(hit)) {
          sI += (double)(hit ? I[r] : 0.0f);
          imax = (hit & (I[r] > imax)) ? I[r] : imax;
          imin = (hit & (I[r] < imin)) ? I[r] : imin;
        }
        pre += mine;
      }
      // pre = sum over the rows r with a pixel of 8 - r, row r at yb + UPD_WAVES r
      col += mine;
      sy += (Sum)(mine * (yb - y0 + ROWS * UPD_WAVES) - pre * UPD_WAVES);
    }
    cnt += (Sum)col;
    sx += (Sum)col * (Sum)(x - x0);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sI += __shfl_xor(sI, o, 64);
    if constexpr (!SMALL) {
      cnt += __shfl_xor(cnt, o, 64);
      sx += __shfl_xor(sx, o, 64);
      sy += __shfl_xor(sy, o, 64);
    }
  }
  if constexpr (SMALL) {
    cnt = wave_sum(cnt);
    sx = wave_sum(sx);
    sy = wave_sum(sy);
  }
  imax = wave_max(imax);
  imin = -wave_max(-imin);
  if (lane == 0) {
    lds[0][wave] = (double)cnt;
    lds[1][wave] = (double)sx;
    lds[2][wave] = (double)sy;
    lds[3][wave] = sI;
    lim[0][wave] = imax;
    lim[1][wave] = imin;
  }
  __syncthreads();
  if (wave != 0) return;
  double t[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    t[r] = 0.0;
    for (int q = 0; q < UPD_WAVES; ++q) t[r] += lds[r][q];
  }
  for (int q = 1; q < UPD_WAVES; ++q) {
    imax = fmaxf(imax, lim[0][q]);
    imin = fminf(imin, lim[1][q]);
  }
  if (!(t[0] > 0)) return;  // no pixels: the centre stays
  t[1] += t[0] * (double)x0;
  t[2] += t[0] * (double)y0;
  // lanes 0, 1, 2: the mean x, y and intensity; lane 3: the deviation from it
  const double mean = (lane == 0 ? t[1] : lane == 1 ? t[2] : t[3]) / t[0];
  const double dev = fmax((double)imax - mean, mean - (double)imin);
  if (lane < 4) c[lane] = (float)(lane < 3 ? mean : fmax(dev, (double)t_min));
}

static pvr_status check_sizes(const char *fn, int n_img, int h, int w, int a) {
  // a = 0: no centre grid to check (pack)
  if (n_img <= 0 || h <= 0 || w <= 0 || a < 0) return fail(PVR_EINVAL, "%s: sizes must be positive", fn);
  if ((long long)n_img * h * w > (1LL << 31)) return fail(PVR_ESHAPE, "%s: more than 2^31 pixels", fn);
  if (h > (1 << 20) || w > (1 << 20)) return fail(PVR_ESHAPE, "%s: a side beyond 2^20 pixels", fn);
  const long long K = a > 0 ? (long long)((h + a - 1) / a) * ((w + a - 1) / a) : 0;
  if (K > (1 << 20)) return fail(PVR_ESHAPE, "%s: more than 2^20 centres per image", fn);
  if ((long long)n_img > 65535) return fail(PVR_ESHAPE, "%s: more than 65535 images", fn);
  return PVR_OK;
}

extern "C" int64_t pvr_slic_centres(int32_t h, int32_t w, int32_t a) {
  if (h <= 0 || w <= 0 || a <= 0) return 0;
  return (int64_t)((h + a - 1) / a) * ((w + a - 1) / a);
}

extern "C" pvr_status pvr_slic_init(const float *img, int32_t n_img, int32_t h, int32_t w,
                                    int32_t a, float t0, float *centres, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic_init", img, 4);
  PVR_ALIGNED("pvr_slic_init", centres, 16);
  if (!img || !centres) return fail(PVR_EINVAL, "pvr_slic_init: NULL argument");
  if (a <= 0 || a > (1 << 20)) return fail(PVR_EINVAL, "pvr_slic_init: a must be in [1, 2^20]");
  pvr_status st = check_sizes("pvr_slic_init", n_img, h, w, a);
  if (st != PVR_OK) return st;
  const int kx = (w + a - 1) / a, K = kx * ((h + a - 1) / a);
  const long long n = (long long)n_img * K;
  hipLaunchKernelGGL(k_slic_init, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, img,
                     n_img, h, w, a, kx, K, t0, centres);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_slic_assign(const float *img, int32_t n_img, int32_t h, int32_t w,
                                      int32_t a, const float *centres, uint64_t *ws,
                                      int32_t *labels, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic_assign", img, 4);
  PVR_ALIGNED("pvr_slic_assign", centres, 16);
  PVR_ALIGNED("pvr_slic_assign", ws, 8);
  PVR_ALIGNED("pvr_slic_assign", labels, 4);
  if (!img || !centres || !ws || !labels) return fail(PVR_EINVAL, "pvr_slic_assign: NULL argument");
  if (a <= 0 || a > (1 << 20)) return fail(PVR_EINVAL, "pvr_slic_assign: a must be in [1, 2^20]");
  pvr_status st = check_sizes("pvr_slic_assign", n_img, h, w, a);
  if (st != PVR_OK) return st;
  const int kx = (w + a - 1) / a, ky = (h + a - 1) / a, K = kx * ky;
  const int rows = TILE_WAVES * TILE_Y;
  const dim3 grid((unsigned)(((w + TILE_X - 1) / TILE_X) * ((h + rows - 1) / rows)), n_img);
  float *drift = (float *)ws;  // n_img floats
  if (K <= SLIC_LIST_ALL) {
    hipLaunchKernelGGL(k_slic_gather<false>, grid, dim3(SLIC_T), 0, stream, img, n_img, h, w, a, kx,
                       ky, K, centres, nullptr, labels);
  } else {
    hipLaunchKernelGGL(k_slic_drift, dim3(n_img), dim3(SLIC_T), 0, stream, centres, h, w, a, kx, K,
                       drift);
    hipLaunchKernelGGL(k_slic_gather<true>, grid, dim3(SLIC_T), 0, stream, img, n_img, h, w, a, kx,
                       ky, K, centres, drift, labels);
  }
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_slic_update(const float *img, int32_t n_img, int32_t h, int32_t w,
                                      int32_t a, const int32_t *labels, float t_min,
                                      float *centres, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic_update", img, 4);
  PVR_ALIGNED("pvr_slic_update", labels, 4);
  PVR_ALIGNED("pvr_slic_update", centres, 16);
  if (!img || !labels || !centres) return fail(PVR_EINVAL, "pvr_slic_update: NULL argument");
  if (a <= 0 || a > (1 << 20)) return fail(PVR_EINVAL, "pvr_slic_update: a must be in [1, 2^20]");
  pvr_status st = check_sizes("pvr_slic_update", n_img, h, w, a);
  if (st != PVR_OK) return st;
  const int K = ((w + a - 1) / a) * ((h + a - 1) / a);
  // windows of at most 2 SLIC_SMALL + 1 pixels a side: sums and offsets below 2^31
  if (a <= SLIC_SMALL && w <= 1 << 18)
    hipLaunchKernelGGL(k_slic_update<true>, dim3(K, n_img), dim3(SLIC_T), 0, stream, img, n_img, h,
                       w, a, K, labels, t_min, centres);
  else
    hipLaunchKernelGGL(k_slic_update<false>, dim3(K, n_img), dim3(SLIC_T), 0, stream, img, n_img, h,
                       w, a, K, labels, t_min, centres);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_slic(const float *img, int32_t n_img, int32_t h, int32_t w, int32_t a,
                               float t0, float t_min, int32_t iters, uint64_t *ws,
                               float *centres, int32_t *labels, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic", img, 4);
  PVR_ALIGNED("pvr_slic", centres, 16);
  PVR_ALIGNED("pvr_slic", ws, 8);
  PVR_ALIGNED("pvr_slic", labels, 4);
  if (iters < 0) return fail(PVR_EINVAL, "pvr_slic: iters < 0");
  pvr_status st = pvr_slic_init(img, n_img, h, w, a, t0, centres, stream);
  for (int it = 0; st == PVR_OK && it < iters; ++it) {
    st = pvr_slic_assign(img, n_img, h, w, a, centres, ws, labels, stream);
    if (st == PVR_OK) st = pvr_slic_update(img, n_img, h, w, a, labels, t_min, centres, stream);
  }
  if (st == PVR_OK) st = pvr_slic_assign(img, n_img, h, w, a, centres, ws, labels, stream);
  return st;
  PVR_API_END();
}

// ---------------------------------------------------------------------------
// Superpixel patches: dilated bounding boxes and the packed samples.

// One workgroup per centre over its window, as the update: the extreme rows
// and columns that carry its label come from a bit per row and lane, sixteen
// rows read at once (64 centres of 256 x 256, 240 images: 22 us, 25 with eight
// rows; 65 one pixel at a time).
constexpr int BOX_ROWS = 16;
__global__ void __launch_bounds__(SLIC_T)
k_slic_boxes(const int32_t *__restrict__ labels, int n_img, int h, int w, int a, int K,
             const float *__restrict__ C, int gamma, int32_t *__restrict__ boxes) {
  __shared__ int red[4][SLIC_T / 64];
  int im, k;
  image_item(K, n_img, im, k);
  const float *c = C + 4 * ((long long)im * K + k);
  int x0, x1, y0, y1;
  window(c[0], c[1], a, h, w, x0, x1, y0, y1);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long base = (long long)im * h * w;
  int b[4] = {INT_MAX, INT_MAX, INT_MIN, INT_MIN};  // min x, min y, max x, max y
  const unsigned step = (unsigned)w * (SLIC_T / 64);
  for (int xb = x0; xb <= x1; xb += 64) {
    const int x = xb + lane;
    for (int yb = y0 + wave; yb <= y1; yb += BOX_ROWS * (SLIC_T / 64)) {
      const int rows = min(BOX_ROWS, (y1 - yb) / (SLIC_T / 64) + 1);
      unsigned seen = 0;  // bit 15 - r: the centre's label in row r
      if (x <= x1) {
        const int32_t *lp = labels + base + (long long)yb * w;
        int lab[BOX_ROWS];
#pragma unroll
        for (int r = 0; r < BOX_ROWS; ++r) lab[r] = lp[(unsigned)min(r, rows - 1) * step + x];
#pragma unroll
        for (int r = 0; r < BOX_ROWS; ++r) seen = seen + seen + (lab[r] == k ? 1u : 0u);
      }
      const unsigned long long cols = __ballot(seen != 0);
      if (!cols) continue;
      b[0] = min(b[0], xb + __builtin_ctzll(cols));
      b[2] = max(b[2], xb + 63 - __builtin_clzll(cols));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) seen |= __shfl_xor(seen, o, 64);
      // (a clamped row repeats the last one: the largest row is bounded by it)
      b[1] = min(b[1], yb + (SLIC_T / 64) * (__builtin_clz(seen) - (32 - BOX_ROWS)));
      b[3] = max(b[3], yb + (SLIC_T / 64) * min(rows - 1, BOX_ROWS - 1 - __builtin_ctz(seen)));
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[r][wave] = b[r];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < SLIC_T / 64; ++q) {
      b[0] = min(b[0], red[0][q]); b[1] = min(b[1], red[1][q]);
      b[2] = max(b[2], red[2][q]); b[3] = max(b[3], red[3][q]);
    }
    int32_t *o = boxes + 4 * ((long long)im * K + k);
    if (b[2] < b[0]) {
      o[0] = o[1] = o[2] = o[3] = 0;
    } else {
      const int bx0 = max(0, b[0] - gamma), by0 = max(0, b[1] - gamma);
      const int bx1 = min(w - 1, b[2] + gamma), by1 = min(h - 1, b[3] + gamma);
      o[0] = bx0; o[1] = by0; o[2] = bx1 - bx0 + 1; o[3] = by1 - by0 + 1;
    }
  }
}

constexpr int PACK_MAX_PIXELS = 65536;

// The device table of the packing: the caller's rows (image, label, x0, y0,
// width, height), M of them, then the M sample offsets.
struct PackTable {
  const int32_t *row;
  const long long *off;
};
__host__ __device__ __forceinline__ PackTable pack_table(const void *ws, int M) {
  return PackTable{(const int32_t *)ws, (const long long *)((const char *)ws + 24 * (size_t)M)};
}
struct PackDesc {
  int32_t img, label, x0, y0, bw, bh;
  long long off;
};
__device__ __forceinline__ PackDesc pack_desc(PackTable t, int s) {
  const int32_t *r = t.row + 6 * (size_t)s;
  return PackDesc{r[0], r[1], r[2], r[3], r[4], r[5], t.off[s]};
}

// Sample offsets: exclusive sums of the boxes' pixels, one workgroup, 16 384
// rows at a time with all their loads in flight (15 360 rows 13 us; 34 with a run
// of rows per thread).
constexpr int OFF_T = 1024, OFF_N = 16;
__global__ void __launch_bounds__(OFF_T)
k_slic_pack_off(const int32_t *__restrict__ row, int M, long long *__restrict__ off) {
  __shared__ long long part[OFF_N * (OFF_T / 64)];  // pixels of 64 rows, then those before them
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  long long base = 0;
  for (int s0 = 0; s0 < M; s0 += OFF_T * OFF_N) {
    int own[OFF_N], inc[OFF_N];  // a box holds at most 2^16 pixels
#pragma unroll
    for (int i = 0; i < OFF_N; ++i) {
      const int s = s0 + i * OFF_T + t;
      const int2 wh = s < M ? *reinterpret_cast<const int2 *>(row + 6 * (size_t)s + 4) : int2{0, 0};
      own[i] = wh.x * wh.y;
    }
#pragma unroll
    for (int i = 0; i < OFF_N; ++i) {
      inc[i] = own[i];
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(inc[i], o, 64);
        inc[i] += lane >= o ? v : 0;
      }
      if (lane == 63) part[i * (OFF_T / 64) + wave] = inc[i];
    }
    __syncthreads();
    if (wave == 0) {
      long long sum = 0;
      constexpr int EACH = OFF_N * (OFF_T / 64) / 64;
      for (int q = 0; q < EACH; ++q) sum += part[lane * EACH + q];
      long long run = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const long long v = __shfl_up(run, o, 64);
        run += lane >= o ? v : 0;
      }
      run -= sum;
      for (int q = 0; q < EACH; ++q) {
        const long long v = part[lane * EACH + q];
        part[lane * EACH + q] = run;
        run += v;
      }
    }
    __syncthreads();
    long long at = 0;
#pragma unroll
    for (int i = 0; i < OFF_N; ++i) {
      const int s = s0 + i * OFF_T + t;
      at = base + part[i * (OFF_T / 64) + wave] + inc[i];
      if (s < M) off[s] = at - own[i];
    }
    __syncthreads();
    if (s0 + OFF_T * OFF_N < M) {  // the sum so far, for the next rows
      if (t == OFF_T - 1) part[0] = at;
      __syncthreads();
      base = part[0];
      __syncthreads();
    }
  }
}

// One workgroup per patch, for gamma < 64 and boxes of at most
// PACK_MAX_WORDS 64-pixel words (rows cut into words): the label's indicator
// is a bit per pixel, dilated along the rows by shifts over a word and its
// neighbours and along the columns by the union of 2 gamma + 1 words, eight at
// a time.  Then
// the box's pixels are copied and the mask bytes written, four a lane.  Bound
// by the stores: 15 360 patches of 98 M samples in 150 us (3.3 TB/s written); 331 a byte
// per pixel, with counts slid along whole rows and columns by single threads.
// A larger gamma or box, or an image beyond 32-bit offsets, goes to k_slic_pack.
constexpr int PACK_GAMMA = 64, PACK_MAX_WORDS = 2048, PACK_MAX_IMAGE = 1 << 29;

__global__ void __launch_bounds__(SLIC_T)
k_slic_pack_bits(const float *__restrict__ img, const int32_t *__restrict__ labels, int h, int w,
                 int gamma, int M, const void *__restrict__ ws, int words,
                 float *__restrict__ y, uint8_t *__restrict__ mask) {
  extern __shared__ __attribute__((aligned(16))) unsigned long long bits[];  // [3][words] + 1
  unsigned long long *wide = bits + words;
  // patches come image by image: an eighth of them to each XCD, so that an
  // image's pixels and labels are read into one L2
  const int per = (M + 7) >> 3, s = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (s >= M) return;
  const PackDesc d = pack_desc(pack_table(ws, M), s);
  const int bw = d.bw, bh = d.bh, n = bw * bh, W = (bw + 63) >> 6, nw = W * bh;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long base = ((long long)d.img * h + d.y0) * w + d.x0;  // box corner
  const unsigned step = (unsigned)w * (SLIC_T / 64);
  for (int cw = 0; cw < W; ++cw) {
    const int x = 64 * cw + lane;
    const unsigned xc = min(x, bw - 1);
    for (int rb = wave; rb < bh; rb += ROWS * (SLIC_T / 64)) {
      const int rows = min(ROWS, (bh - 1 - rb) / (SLIC_T / 64) + 1);
      const int32_t *lp = labels + base + (long long)rb * w;
      int lab[ROWS];
      if (rows == ROWS) {
        unsigned o = xc;
#pragma unroll
        for (int i = 0; i < ROWS; ++i, o += step) lab[i] = lp[o];
      } else {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) lab[i] = lp[(unsigned)min(i, rows - 1) * step + xc];
      }
      int lo = 0, hi = 0;  // lane i: row i of the eight
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        const unsigned long long hit = __ballot(lab[i] == d.label && x < bw);
        lo = lane == i ? (int)hit : lo;
        hi = lane == i ? (int)(hit >> 32) : hi;
      }
      if (lane < rows)
        bits[(rb + lane * (SLIC_T / 64)) * W + cw] = (unsigned long long)(unsigned)hi << 32 | (unsigned)lo;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nw; q += SLIC_T) {
    const int cw = q % W;
    unsigned long long up = bits[q], dn = up, lo = cw > 0 ? bits[q - 1] : 0ull,
                       hi = cw + 1 < W ? bits[q + 1] : 0ull;
    for (int c = 1; c <= gamma;) {  // up, dn cover shifts of 0 .. c - 1
      const int s = min(c, gamma + 1 - c);
      up |= up << s | lo >> (64 - s);
      lo |= lo << s;
      dn |= dn >> s | hi << (64 - s);
      hi |= hi >> s;
      c += s;
    }
    wide[q] = up | dn;
  }
  __syncthreads();
  // unions of eight rows from each row on, then of those (2 gamma + 1 rows)
  for (int q = threadIdx.x; q < nw; q += SLIC_T) {
    unsigned long long m = wide[q];
#pragma unroll
    for (int i = 1; i < 8; ++i) m |= q + i * W < nw ? wide[q + i * W] : 0ull;
    bits[q] = m;
  }
  __syncthreads();
  unsigned long long *out = bits + 2 * words;
  for (int q = threadIdx.x; q < nw; q += SLIC_T) {
    const int r = q / W, cw = q - r * W;
    const int r0 = max(0, r - gamma), r1 = min(bh - 1, r + gamma);
    unsigned long long m = 0;
    if (r1 - r0 >= 7) {
      for (int rr = r0; rr <= r1 - 7; rr += 8) m |= bits[rr * W + cw];
      m |= bits[(r1 - 7) * W + cw];
    } else {
      for (int rr = r0; rr <= r1; ++rr) m |= wide[rr * W + cw];
    }
    out[q] = m;
  }
  __syncthreads();
  const unsigned *b32 = reinterpret_cast<const unsigned *>(out);
  float *yo = y + d.off;
  uint8_t *mo = mask + d.off;
  const float *src = img + base;
  const float rcp = 1.0f / (float)bw;
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef float f4 __attribute__((ext_vector_type(4)));
  const auto one = [&](int q, int r, int x) {
    yo[q] = src[(unsigned)(r * w + x)];
    mo[q] = b32[2 * r * W + (x >> 5)] >> (x & 31) & 1u;
  };
  // quads from the first 16-byte boundary of y on, those inside one row
  const int head = min(n, (int)(-(reinterpret_cast<uintptr_t>(yo) >> 2) & 3));
  const int quads = (n - head) >> 2;
  for (int t = threadIdx.x; t < quads; t += SLIC_T) {
    const int q = head + 4 * t;
    const int r = (int)(((float)q + 0.5f) * rcp);  // exact: q < 2^16
    const int x = q - __mul24(r, bw);
    if (x + 3 < bw) {
      const unsigned *b = b32 + __mul24(r, 2 * W) + (x >> 5);  // (a word of padding behind)
      const unsigned m = __builtin_amdgcn_alignbit(b[1], b[0], x & 31) & 15u;
      *reinterpret_cast<f4 *>(yo + q) = *reinterpret_cast<const f4u *>(src + (unsigned)(__mul24(r, w) + x));
      const unsigned m4 = (unsigned)__mul24((int)m, 0x204081) & 0x01010101u;
      __builtin_memcpy(mo + q, &m4, 4);
    }
  }
  // the quads across two or more rows, one thread per quad (by the row its
  // first sample lies in), and the up to three samples before and after the quads
  for (int r = threadIdx.x; r < bh; r += SLIC_T) {
    const int e = (r + 1) * bw;                        // the next row's first sample
    const int q0 = head + ((e - head - 1) & ~3);       // the quad of this row's last
    if (q0 < head || q0 < r * bw || q0 + 4 > head + 4 * quads || q0 + 4 <= e) continue;
    int rr = r, x = q0 - r * bw;
    for (int i = 0; i < 4; ++i) {
      one(q0 + i, rr, x);
      if (++x == bw) {
        x = 0;
        ++rr;
      }
    }
  }
  const int t = threadIdx.x;
  const int q = t < 4 ? t : head + 4 * quads + t - 4;
  if (t < 8 && (t < 4 ? q < head : q < n)) one(q, q / bw, q % bw);
}

// One workgroup per patch.  The label's indicator over the box sits in LDS as
// bit 0 of a byte; a sliding-window count along the rows gives the row
// dilation (bit 1), the same along the columns of bit 1 the square dilation
// (bit 2).
__global__ void __launch_bounds__(SLIC_T)
k_slic_pack(const float *__restrict__ img, const int32_t *__restrict__ labels, int h, int w,
            int gamma, int M, const void *__restrict__ ws, float *__restrict__ y,
            uint8_t *__restrict__ mask) {
  extern __shared__ uint8_t bytes[];
  uint8_t *bits = bytes;
  const PackDesc d = pack_desc(pack_table(ws, M), blockIdx.x);
  const int bw = d.bw, bh = d.bh, n = bw * bh;
  const long long base = (long long)d.img * h * w;
  for (int q = threadIdx.x; q < n; q += SLIC_T) {
    const long long p = base + (long long)(d.y0 + q / bw) * w + d.x0 + q % bw;
    bits[q] = labels[p] == d.label ? 1 : 0;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < bh; r += SLIC_T) {
    uint8_t *row = bits + r * bw;
    int cnt = 0;
    for (int x = 0; x < min(gamma, bw); ++x) cnt += row[x] & 1;
    for (int x = 0; x < bw; ++x) {
      if (x + gamma < bw) cnt += row[x + gamma] & 1;
      if (x - gamma - 1 >= 0) cnt -= row[x - gamma - 1] & 1;
      if (cnt > 0) row[x] |= 2;
    }
  }
  __syncthreads();
  for (int col = threadIdx.x; col < bw; col += SLIC_T) {
    uint8_t *cp = bits + col;
    int cnt = 0;
    for (int yy = 0; yy < min(gamma, bh); ++yy) cnt += (cp[yy * bw] >> 1) & 1;
    for (int yy = 0; yy < bh; ++yy) {
      if (yy + gamma < bh) cnt += (cp[(yy + gamma) * bw] >> 1) & 1;
      if (yy - gamma - 1 >= 0) cnt -= (cp[(yy - gamma - 1) * bw] >> 1) & 1;
      if (cnt > 0) cp[yy * bw] |= 4;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < n; q += SLIC_T) {
    const long long p = base + (long long)(d.y0 + q / bw) * w + d.x0 + q % bw;
    y[d.off + q] = img[p];
    mask[d.off + q] = (bits[q] >> 2) & 1;
  }
}

extern "C" pvr_status pvr_slic_boxes(const int32_t *labels, int32_t n_img, int32_t h, int32_t w,
                                     int32_t a, const float *centres, int32_t gamma,
                                     int32_t *boxes, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic_boxes", labels, 4);
  PVR_ALIGNED("pvr_slic_boxes", centres, 16);
  PVR_ALIGNED("pvr_slic_boxes", boxes, 4);
  if (!labels || !centres || !boxes) return fail(PVR_EINVAL, "pvr_slic_boxes: NULL argument");
  if (gamma < 0) return fail(PVR_EINVAL, "pvr_slic_boxes: gamma < 0");
  if (a <= 0 || a > (1 << 20)) return fail(PVR_EINVAL, "pvr_slic_boxes: a must be in [1, 2^20]");
  pvr_status st = check_sizes("pvr_slic_boxes", n_img, h, w, a);
  if (st != PVR_OK) return st;
  const int K = ((w + a - 1) / a) * ((h + a - 1) / a);
  hipLaunchKernelGGL(k_slic_boxes, dim3(K, n_img), dim3(SLIC_T), 0, stream, labels, n_img, h,
                     w, a, K, centres, gamma, boxes);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}

// Checks the host table of pvr_slic_pack and returns the largest box (pixels,
// k_slic_pack's LDS bytes) and the most words of one (k_slic_pack_bits).
static pvr_status pack_check(const char *fn, int32_t n_img, int32_t h, int32_t w, int32_t M,
                             const int32_t *table, int *most, int *words) {
  *most = *words = 0;
  for (int s = 0; s < M; ++s) {
    const int32_t *t = table + 6 * (size_t)s;
    if (t[0] < 0 || t[0] >= n_img || t[4] <= 0 || t[5] <= 0 || t[2] < 0 || t[3] < 0 ||
        t[2] > w - t[4] || t[3] > h - t[5])
      return fail(PVR_ESHAPE, "%s: patch %d (image %d, box %d,%d %dx%d) leaves its image", fn, s,
                  t[0], t[2], t[3], t[4], t[5]);
    if ((long long)t[4] * t[5] > PACK_MAX_PIXELS)
      return fail(PVR_ESHAPE, "%s: patch %d holds %lld pixels (at most %d)", fn, s,
                  (long long)t[4] * t[5], PACK_MAX_PIXELS);
    *most = std::max(*most, t[4] * t[5]);
    *words = std::max(*words, (t[4] + 63) / 64 * t[5]);
  }
  return PVR_OK;
}

// Copies the M rows into the device table `ws` (one synchronised copy: the
// rows are the caller's), sums their offsets behind them, then launches the
// packing.  No memory is allocated.
static pvr_status pack_launch(const float *img, const int32_t *labels, int32_t h, int32_t w,
                              int32_t gamma, int32_t M, const int32_t *table, int most, int words,
                              void *ws, float *y, uint8_t *mask, hipStream_t stream) {
  HIP_TRY(hipMemcpyAsync(ws, table, 24 * (size_t)M, hipMemcpyHostToDevice, stream));
  HIP_TRY(hipStreamSynchronize(stream));
  const PackTable tab = pack_table(ws, M);
  hipLaunchKernelGGL(k_slic_pack_off, dim3(1), dim3(OFF_T), 0, stream, tab.row, M,
                     const_cast<long long *>(tab.off));
  if (gamma < PACK_GAMMA && words <= PACK_MAX_WORDS && (long long)h * w < PACK_MAX_IMAGE)
    hipLaunchKernelGGL(k_slic_pack_bits, dim3((M + 7) / 8 * 8), dim3(SLIC_T), 24 * (size_t)words + 8, stream, img,
                       labels, h, w, gamma, M, (const void *)ws, words, y, mask);
  else
    hipLaunchKernelGGL(k_slic_pack, dim3(M), dim3(SLIC_T), (size_t)most, stream, img, labels, h, w,
                       gamma, M, (const void *)ws, y, mask);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
}

extern "C" size_t pvr_slic_pack_workspace(int32_t M) {
  return M > 0 ? sizeof(PackDesc) * (size_t)M : 0;
}

extern "C" pvr_status pvr_slic_pack(const float *img, const int32_t *labels, int32_t n_img,
                                    int32_t h, int32_t w, int32_t gamma, int32_t M,
                                    const int32_t *table, void *workspace, size_t workspace_bytes,
                                    float *y, uint8_t *mask, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic_pack", img, 4);
  PVR_ALIGNED("pvr_slic_pack", labels, 4);
  PVR_ALIGNED("pvr_slic_pack", y, 4);
  PVR_ALIGNED("pvr_slic_pack", workspace, 16);
  if (!img || !labels || !table || (M > 0 && (!y || !mask || !workspace)))
    return fail(PVR_EINVAL, "pvr_slic_pack: NULL argument");
  if (gamma < 0 || M < 0) return fail(PVR_EINVAL, "pvr_slic_pack: gamma < 0 or M < 0");
  pvr_status st = check_sizes("pvr_slic_pack", n_img, h, w, 0);
  if (st != PVR_OK) return st;
  if (M == 0) return PVR_OK;
  if (workspace_bytes < pvr_slic_pack_workspace(M))
    return fail(PVR_ESHAPE, "pvr_slic_pack: workspace of %zu bytes, %zu needed for %d patches",
                workspace_bytes, pvr_slic_pack_workspace(M), M);
  int most = 0, words = 0;
  st = pack_check("pvr_slic_pack", n_img, h, w, M, table, &most, &words);
  if (st != PVR_OK) return st;
  return pack_launch(img, labels, h, w, gamma, M, table, most, words, workspace, y, mask, stream);
  PVR_API_END();
}

// ---------------------------------------------------------------------------
// pvr_slic_pack_noalloc: the same packing for callers that cannot allocate
// device memory.  The table lives in `scratch`, a file-scope device
// array for PVR_SLIC_PACK_NOALLOC_MAX patches; every device holds its
// own copy, whose address is looked up once per device.  In host code the
// array's name is only a host-side stand-in: the kernels receive the looked
// up device address.
// ---------------------------------------------------------------------------
static __device__ __align__(256) PackDesc scratch[PVR_SLIC_PACK_NOALLOC_MAX];

namespace {
constexpr int SCRATCH_DEVICES = 64;
std::mutex g_scratch_mu;
PackDesc *g_scratch_ptr[SCRATCH_DEVICES];  // device address of `scratch` per device
}  // namespace

static pvr_status scratch_on_current_device(PackDesc **out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= SCRATCH_DEVICES)
    return fail(PVR_EUNSUPPORTED, "pvr_slic_pack_noalloc: device %d beyond %d", dev, SCRATCH_DEVICES);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(PVR_EHIP, "pvr_slic_pack_noalloc: no device address for the table");
    g_scratch_ptr[dev] = (PackDesc *)ptr;
  }
  *out = g_scratch_ptr[dev];
  return PVR_OK;
}

extern "C" pvr_status pvr_slic_pack_noalloc(const float *img, const int32_t *labels,
                                            int32_t n_img, int32_t h, int32_t w, int32_t gamma,
                                            int32_t M, const int32_t *table, float *y,
                                            uint8_t *mask, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_slic_pack_noalloc", img, 4);
  PVR_ALIGNED("pvr_slic_pack_noalloc", labels, 4);
  PVR_ALIGNED("pvr_slic_pack_noalloc", y, 4);
  if (!img || !labels || !table || (M > 0 && (!y || !mask)))
    return fail(PVR_EINVAL, "pvr_slic_pack_noalloc: NULL argument");
  if (gamma < 0 || M < 0) return fail(PVR_EINVAL, "pvr_slic_pack_noalloc: gamma < 0 or M < 0");
  if (M > PVR_SLIC_PACK_NOALLOC_MAX)
    return fail(PVR_ESHAPE, "pvr_slic_pack_noalloc: %d patches, at most %d", M,
                PVR_SLIC_PACK_NOALLOC_MAX);
  pvr_status st = check_sizes("pvr_slic_pack_noalloc", n_img, h, w, 0);
  if (st != PVR_OK) return st;
  if (M == 0) return PVR_OK;
  int most = 0, words = 0;
  st = pack_check("pvr_slic_pack_noalloc", n_img, h, w, M, table, &most, &words);
  if (st != PVR_OK) return st;
  PackDesc *tab = nullptr;
  st = scratch_on_current_device(&tab);
  if (st != PVR_OK) return st;
  st = pack_launch(img, labels, h, w, gamma, M, table, most, words, tab, y, mask, stream);
  if (st != PVR_OK) return st;
  HIP_TRY(hipStreamSynchronize(stream));  // the device's table is free again on return
  return PVR_OK;
  PVR_API_END();
}
