// Learned registration initialiser: a small 2D CNN that maps a pair
// (observed patch, patch simulated from the current volume) to a 6-DoF rigid
// correction.  Hand-written training and inference kernels for gfx950:
// convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16 (BF16 operands,
// FP32 accumulation); pooling, head, loss and Adam run in FP32.
//
// Layouts: activations NHWC BF16 ([B][H][W][C]); conv weights BF16
// [Cout][3][3][Cin] for the forward pass and [3][3][Cin][Cout] for the data
// gradient, FP32 master copies [Cout][3][3][Cin]; gradients FP32.
//
// MFMA 16x16x32 lane layout (lane l, i = 0..7 for operands, 0..3 for the
// result): A row l%16, k = 8*(l/16)+i; B column l%16, k = 8*(l/16)+i;
// D column l%16, row 4*(l/16)+i.
#include <math.h>
#include <stdint.h>

#include "pvr_cnn.h"
#include "pvr_internal.h"
#include "pvr_util.h"

#include <algorithm>

using namespace pvr;

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// two FP32 values to BF16, round to nearest even (one instruction)
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}
__device__ __forceinline__ uint16_t f2bf(float f) { return (uint16_t)f2bf2(f, f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

union V8 {
  uint4 u;
  bf16x8 v;
  uint16_t h[8];
};

__device__ __forceinline__ bf16x8 load8(const uint16_t *p) {
  V8 t;
  t.u = *reinterpret_cast<const uint4 *>(p);
  return t.v;
}

}  // namespace

// ---------------------------------------------------------------------------
// Tiled 3x3 convolution, the forward pass (out = relu(conv3x3(in, W, stride S,
// pad 1) + bias)) and, DG, the stride-1 data gradient (the same sum with the
// taps mirrored, over gout * [out > 0], no bias).
//
// Implicit GEMM with the weights as the A operand (M = NO output channels)
// and the input as B (N = output pixels), K = 9 KC, tap after tap, so that each
// lane ends with four consecutive channels of one pixel and stores them as one
// 8-byte word.  A workgroup stages the layer's weights into LDS once (rows of
// K padded by 8 elements) and loops over groups of NSUB tiles of TW x TH output
// pixels; the tiles' input, with its border, zero outside the image, is staged
// too (pixels padded by 8 channels; for stride 2 even columns before odd ones,
// so that neighbouring lanes read neighbouring pixels), the next group's read
// into registers while this one is multiplied.  A wavefront takes PB blocks of 16
// pixels times all channels: NT + PB 16-byte LDS reads per lane and NT PB matrix
// instructions a step, and every input value is read once from memory instead of
// once a tap, and masked (DG) once.
// Bound by memory where the layer is large (32x32, 32 -> 64 channels, 1024 images:
// 201 MB in 58 us, 3.5 TB/s; 87 with each tap gathered from memory by 16 pixels a
// wavefront), by LDS reads where it is not (16x16, 64 -> 64: 29 us; 51).  Weights in
// registers instead of LDS were as fast (no room for the next group's input).
// ---------------------------------------------------------------------------
template <int KC_, int NO_, int S, int TW, int TH, int NSUB, int WAVES>
struct TileShape {
  static constexpr int KC = KC_, NO = NO_, K = 9 * KC, LS = K + 8;
  static constexpr int IW = (TW - 1) * S + 3, IH = (TH - 1) * S + 3;  // input tile with its border
  static constexpr int NE = S == 2 ? (IW + 1) / 2 : 0;                // even columns
  static constexpr int CS = KC + 8;                                   // LDS stride of a pixel
  static constexpr int PIX = IW * IH;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int CHUNKS = NSUB * PIX * (KC / 8);
  static constexpr int NL = (CHUNKS + THREADS - 1) / THREADS;
  static constexpr int PB = NSUB * TW * TH / 16 / WAVES, NT = NO / 16;
  static constexpr int W_ELEMS = NO * LS, I_ELEMS = NSUB * PIX * CS;
  static constexpr int LDS_BYTES = (W_ELEMS + I_ELEMS) * 2;
  // column ix of an input row in LDS
  __device__ static constexpr int slot(int ix) { return S == 2 ? (ix >> 1) + (ix & 1) * NE : ix; }
};

// One block group's products: acc[pb][nt] += W x input, tap after tap.
template <class SH, int S, bool DG>
__device__ __forceinline__ void tile_mma(const uint16_t *Wl, const uint16_t *It, const int (&px)[SH::PB],
                                         int r16, int kq, f32x4 (&acc)[SH::PB][SH::NT]) {
  constexpr int CB = SH::KC / 32;
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    const int dy = DG ? 2 - tap / 3 : tap / 3, dx = DG ? 2 - tap % 3 : tap % 3;
    const int o = (dy * SH::IW + SH::slot(dx)) * SH::CS;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      bf16x8 a[SH::PB];
#pragma unroll
      for (int b = 0; b < SH::PB; ++b)
        a[b] = *reinterpret_cast<const bf16x8 *>(It + px[b] + o + cb * 32);
#pragma unroll
      for (int nt = 0; nt < SH::NT; ++nt) {
        const bf16x8 w = *reinterpret_cast<const bf16x8 *>(
            Wl + (nt * 16 + r16) * SH::LS + tap * SH::KC + cb * 32 + 8 * kq);
#pragma unroll
        for (int b = 0; b < SH::PB; ++b)
          acc[b][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a[b], acc[b][nt], 0, 0, 0);
      }
    }
  }
}

// bias, ReLU, BF16: lane (kq, r16) holds channels nt*16 + 4kq .. +3 of
// pixel p, one 8-byte store per 16-channel block
template <int COUT, int NT>
__device__ __forceinline__ void conv_store(uint16_t *__restrict__ out, long long p, int kq,
                                           const f32x4 (&acc)[NT], const float (&bb)[NT][4],
                                           int relu) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = acc[nt][i] + bb[nt][i];
      if (relu) v[i] = fmaxf(v[i], 0.f);  // (NaN gives 0)
    }
    *reinterpret_cast<uint2 *>(out + p * COUT + nt * 16 + 4 * kq) =
        make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
  }
}

// Image, row and column of a tile, ntx by nty an image.  ONE: a single tile an
// image (8 x 8 tiles are used for images no larger), which saves the divisions
// where the tile differs from lane to lane.
struct TileAt {
  int im, y, x;
};
template <bool ONE>
__device__ __forceinline__ TileAt tile_of(int sid, int ntx, int nty) {
  if constexpr (ONE) return TileAt{sid, 0, 0};
  const int im = sid / (ntx * nty), t = sid - im * (ntx * nty), y = t / ntx;
  return TileAt{im, y, t - y * ntx};
}

// Hi x Wi: the input's size, Ho x Wo the output's; n_sub tiles, ntx by nty an
// image.
template <int KC, int NO, int S, int TW, int TH, int NSUB, int WAVES, bool DG>
__global__ void __launch_bounds__(64 * WAVES)
k_conv_tile(const uint16_t *__restrict__ in, const uint16_t *__restrict__ mask,
            const uint16_t *__restrict__ W, const float *__restrict__ bias,
            uint16_t *__restrict__ out, int Hi, int Wi, int Ho, int Wo, int relu, int n_sub, int ntx,
            int nty) {
  using SH = TileShape<KC, NO, S, TW, TH, NSUB, WAVES>;
  constexpr int NL = SH::NL, PB = SH::PB, NT = SH::NT, C8 = KC / 8;
  __shared__ __attribute__((aligned(16))) uint16_t Wl[SH::W_ELEMS];
  __shared__ __attribute__((aligned(16))) uint16_t It[SH::I_ELEMS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, r16 = lane & 15;
  const int n_groups = (n_sub + NSUB - 1) / NSUB;
  uint4 g[NL], y[DG ? NL : 1];
  const auto load = [&](int group) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int e = j * SH::THREADS + threadIdx.x;
      g[j] = make_uint4(0, 0, 0, 0);
      if constexpr (DG) y[j] = g[j];
      const int pix = e / C8, sub = NSUB == 1 ? 0 : pix / SH::PIX, rr = pix - sub * SH::PIX;
      const int sid = group * NSUB + sub;
      const TileAt t = tile_of<TW == 8>(sid, ntx, nty);
      const int iy = t.y * (TH * S) - 1 + rr / SH::IW, ix = t.x * (TW * S) - 1 + rr % SH::IW;
      if (e < SH::CHUNKS && sid < n_sub && (unsigned)iy < (unsigned)Hi && (unsigned)ix < (unsigned)Wi) {
        const long long o = (((long long)t.im * Hi + iy) * Wi + ix) * KC + 8 * (e % C8);
        g[j] = *reinterpret_cast<const uint4 *>(in + o);
        if constexpr (DG) y[j] = *reinterpret_cast<const uint4 *>(mask + o);
      }
    }
  };
  const auto put = [&]() {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int e = j * SH::THREADS + threadIdx.x;
      if (e >= SH::CHUNKS) break;
      const int pix = e / C8, sub = NSUB == 1 ? 0 : pix / SH::PIX, rr = pix - sub * SH::PIX;
      V8 v;
      v.u = g[j];
      if constexpr (DG) {
        V8 m;
        m.u = y[j];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (!(bf2f(m.h[i]) > 0.f)) v.h[i] = 0;
      }
      *reinterpret_cast<uint4 *>(
          &It[(sub * SH::PIX + (rr / SH::IW) * SH::IW + SH::slot(rr % SH::IW)) * SH::CS + 8 * (e % C8)]) = v.u;
    }
  };
  load(blockIdx.x);
  if constexpr (DG) {  // [tap][NO][KC] -> rows of K per output channel
    for (int e = threadIdx.x; e < 9 * NO * C8; e += SH::THREADS) {
      const int k8 = e % C8, q = e / C8, tap = q / NO, no = q % NO;
      *reinterpret_cast<uint4 *>(&Wl[no * SH::LS + tap * KC + 8 * k8]) =
          *reinterpret_cast<const uint4 *>(W + (long long)q * KC + 8 * k8);
    }
  } else {
    for (int e = threadIdx.x; e < NO * (SH::K / 8); e += SH::THREADS) {
      const int no = e / (SH::K / 8), k8 = e % (SH::K / 8);
      *reinterpret_cast<uint4 *>(&Wl[no * SH::LS + 8 * k8]) =
          *reinterpret_cast<const uint4 *>(W + (long long)no * SH::K + 8 * k8);
    }
  }
  float bb[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int i = 0; i < 4; ++i) bb[nt][i] = DG ? 0.f : bias[nt * 16 + 4 * kq + i];
  int px[PB];  // LDS offset of the lane's pixel of each block (upper left tap, 8 kq channels on)
#pragma unroll
  for (int b = 0; b < PB; ++b) {
    const int q = (wave * PB + b) * 16 + r16, sub = q / (TW * TH), rr = q % (TW * TH);
    px[b] = (sub * SH::PIX + (rr / TW) * S * SH::IW + rr % TW) * SH::CS + 8 * kq;
  }
  put();
  __syncthreads();
  for (int group = blockIdx.x; group < n_groups; group += gridDim.x) {
    const bool more = group + (int)gridDim.x < n_groups;
    if (more) load(group + gridDim.x);
    f32x4 acc[PB][NT];
#pragma unroll
    for (int b = 0; b < PB; ++b)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[b][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    tile_mma<SH, S, DG>(Wl, It, px, r16, kq, acc);
#pragma unroll
    for (int b = 0; b < PB; ++b) {
      const int q = (wave * PB + b) * 16 + r16, sub = q / (TW * TH), rr = q % (TW * TH);
      const int sid = group * NSUB + sub;
      const TileAt t = tile_of<TW == 8>(sid, ntx, nty);
      const int oy = t.y * TH + rr / TW, ox = t.x * TW + rr % TW;
      if (sid < n_sub && oy < Ho && ox < Wo)
        conv_store<NO, NT>(out, ((long long)t.im * Ho + oy) * Wo + ox, kq, acc[b], bb, DG ? 0 : relu);
    }
    if (!more) break;
    __syncthreads();
    put();
    __syncthreads();
  }
}

// Workgroups: as many as fit on the chip at once by LDS, at most one a group.
template <class SH>
static unsigned tile_grid(long long n_groups) {
  const long long cap = 256LL * std::max(1, std::min(4, 160 * 1024 / SH::LDS_BYTES));
  return (unsigned)std::min(n_groups, cap);
}

template <int KC, int NO, int S, int TW, int TH, int NSUB, int WAVES, bool DG>
static pvr_status tile_launch(const uint16_t *in, const uint16_t *mask, const uint16_t *W,
                              const float *bias, uint16_t *out, int B, int Hi, int Wi, int Ho, int Wo,
                              int relu, hipStream_t stream) {
  using SH = TileShape<KC, NO, S, TW, TH, NSUB, WAVES>;
  const int ntx = (Wo + TW - 1) / TW, nty = (Ho + TH - 1) / TH;
  const long long n_sub = (long long)B * ntx * nty;
  if (n_sub > 0x7fff0000LL) return fail(PVR_ESHAPE, "pvr_cnn: more than 2^31 tiles");
  hipLaunchKernelGGL((k_conv_tile<KC, NO, S, TW, TH, NSUB, WAVES, DG>),
                     dim3(tile_grid<SH>((n_sub + NSUB - 1) / NSUB)), dim3(SH::THREADS), 0, stream, in,
                     mask, W, bias, out, Hi, Wi, Ho, Wo, relu, (int)n_sub, ntx, nty);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
}

// Tiles of a layer: 16 x 16 pixels, 16 x 8 with stride 2 (their input is as
// large), or 8 x 8 ones, four or two at a time, where the image is no larger and
// one image a workgroup would take the chip more than a round (8x8, 64 -> 64
// channels: 1024 images 10.4 us, 20.2 in 16 x 16 tiles; 256 images 9.2 and 7.5).
constexpr int SMALL_MIN = 257;
template <int KC, int NO, int S, bool DG>
static pvr_status conv_tiled(const uint16_t *in, const uint16_t *mask, const uint16_t *W,
                             const float *bias, uint16_t *out, int B, int Hi, int Wi, int relu,
                             hipStream_t stream) {
  const int Ho = (Hi - 1) / S + 1, Wo = (Wi - 1) / S + 1;
  if (Ho <= 8 && Wo <= 8 && B >= SMALL_MIN)
    return tile_launch<KC, NO, S, 8, 8, 4 / S, 8, DG>(in, mask, W, bias, out, B, Hi, Wi, Ho, Wo, relu, stream);
  if constexpr (S == 2 && KC == 32)  // four wavefronts, two workgroups a compute unit by LDS
    return tile_launch<KC, NO, S, 16, 8, 1, 4, DG>(in, mask, W, bias, out, B, Hi, Wi, Ho, Wo, relu, stream);
  else
    return tile_launch<KC, NO, S, 16, 16 / S, 1, 8, DG>(in, mask, W, bias, out, B, Hi, Wi, Ho, Wo, relu, stream);
}

// ---------------------------------------------------------------------------
// forward pass of a layer of fewer than 32 input channels: K = 9 CIN <= 32 in
// one matrix step, each lane gathering its taps from memory; the workgroup (16
// waves) loops over tiles of 256 output pixels, one 16-pixel column block per
// wave.  Bound by the output's stores.
// ---------------------------------------------------------------------------
constexpr int FW_THREADS = 1024;                       // 16 waves share the staged weights
constexpr int FW_TILE = (FW_THREADS / 64) * 16;       // 16 output pixels per wave

template <int CIN, int COUT>
struct FwdShape {
  static constexpr int K = 9 * CIN;
  static constexpr int KP = K < 32 ? 32 : K;  // K padded to one MFMA step when CIN < 32
  static constexpr int LS = KP + 8;           // LDS row stride (elements), 16-byte rows
  static constexpr int LDS_BYTES = COUT * LS * 2;
};

template <int CIN, int COUT, int S>
__global__ void __launch_bounds__(FW_THREADS)
k_conv_fwd(const uint16_t *__restrict__ in, const uint16_t *__restrict__ W,
           const float *__restrict__ bias, uint16_t *__restrict__ out, int B, int H, int Wd,
           int relu) {
  using SH = FwdShape<CIN, COUT>;
  constexpr int NT = COUT / 16, K = SH::K, KP = SH::KP, LS = SH::LS;
  __shared__ __attribute__((aligned(16))) uint16_t Wl[COUT * LS];
  for (int e = threadIdx.x; e < COUT * KP; e += FW_THREADS) {
    const int co = e / KP, k = e % KP;
    Wl[co * LS + k] = k < K ? W[co * K + k] : (uint16_t)0;
  }
  __syncthreads();
  const int Ho = (H - 1) / S + 1, Wo = (Wd - 1) / S + 1;
  const long long P = (long long)B * Ho * Wo;
  const long long n_tiles = (P + FW_TILE - 1) / FW_TILE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, r16 = lane & 15;
  float bb[NT][4];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int i = 0; i < 4; ++i) bb[nt][i] = bias[nt * 16 + 4 * kq + i];
  for (long long tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const long long pbase = tile * FW_TILE + wave * 16;
    if (pbase >= P) continue;  // wave-uniform; no barrier below
    const long long p = pbase + r16;
    const bool pv = p < P;
    const long long pp = pv ? p : 0;
    const int pb = (int)(pp / (Ho * Wo));
    const int rr = (int)(pp % (Ho * Wo));
    const int py = rr / Wo, px = rr % Wo;
    // lane group kq holds taps 4 kq .. 4 kq + 3, both channels (one dword each)
    static_assert(CIN == 2, "two input channels");
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int tap = 4 * kq + j;
      const int iy = py * S + tap / 3 - 1, ix = px * S + tap % 3 - 1;
      d[j] = (pv && tap < 9 && iy >= 0 && iy < H && ix >= 0 && ix < Wd)
                 ? *reinterpret_cast<const uint32_t *>(in + (((long long)pb * H + iy) * Wd + ix) * 2)
                 : 0u;
    }
    V8 ta;
    ta.u = make_uint4(d[0], d[1], d[2], d[3]);
    f32x4 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const bf16x8 w = *reinterpret_cast<const bf16x8 *>(&Wl[(nt * 16 + r16) * LS + 8 * kq]);
      acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, ta.v, (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    if (pv) conv_store<COUT, NT>(out, p, kq, acc, bb, relu);
  }
}

// Persistent grid: as many workgroups as fit on the chip at once with the
// layer's LDS, at most one per tile.
static unsigned persistent_grid(long long n_tiles, int lds_bytes) {
  int per_cu = (150 * 1024) / (lds_bytes > 0 ? lds_bytes : 1);
  per_cu = per_cu < 1 ? 1 : (per_cu > 2 ? 2 : per_cu);  // 1024-thread workgroups
  const long long cap = 256LL * per_cu;
  return (unsigned)(n_tiles < cap ? n_tiles : cap);
}

// ---------------------------------------------------------------------------
// The first two layers at once (2 -> 32 channels, then 32 -> 32 with stride 2,
// both with ReLU), for a forward pass that keeps no activations: a workgroup
// computes the 33 x 17 first-layer pixels under a tile of 16 x 8 outputs into LDS
// (BF16, zero outside the image, as the layer by itself would store them) and
// the second layer from there; both layers' weights stay in registers.  Bound by
// vector issue (the first layer's bias, ReLU and rounding).  1024 images of 64 x 64:
// 54 us; 85 + 70 layer by layer, which write and read 268 MB in between.
// ---------------------------------------------------------------------------
constexpr int ST_W = 16, ST_H = 8, ST_WAVES = 4;           // output tile
constexpr int ST_XW = 2 * ST_W + 3, ST_XH = 2 * ST_H + 3;  // input tile of the first layer

__global__ void __launch_bounds__(64 * ST_WAVES, 3)
k_conv_stem(const uint32_t *__restrict__ in, const uint16_t *__restrict__ W1,
            const float *__restrict__ b1, const uint16_t *__restrict__ W2,
            const float *__restrict__ b2, uint16_t *__restrict__ out, int H, int Wd, int Ho, int Wo,
            int n_tiles, int ntx, int nty) {
  using SH = TileShape<32, 32, 2, ST_W, ST_H, 1, ST_WAVES>;
  constexpr int XN = ST_XW * ST_XH, NX = (XN + SH::THREADS - 1) / SH::THREADS;
  static_assert(SH::IW == 33 && SH::IH == 17, "two blocks and a column");
  __shared__ __attribute__((aligned(16))) uint16_t It[SH::I_ELEMS];
  __shared__ uint32_t Xt[XN + 1];  // the last entry stays zero
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kq = lane >> 4, r16 = lane & 15;
  const int per = ntx * nty;
  bf16x8 w1[2], w2[9][2];
  float bb1[2][4], bb2[2][4];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    V8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 8 * kq + i;
      v.h[i] = k < 18 ? W1[(nt * 16 + r16) * 18 + k] : (uint16_t)0;
    }
    w1[nt] = v.v;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) w2[tap][nt] = load8(W2 + (nt * 16 + r16) * 288 + tap * 32 + 8 * kq);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bb1[nt][i] = b1[nt * 16 + 4 * kq + i];
      bb2[nt][i] = b2[nt * 16 + 4 * kq + i];
    }
  }
  // LDS entry of the lane's tap 4 kq + j for the pixel block at row 0, column r16,
  // and its step a row and a column (taps from 9 on stay at the zero)
  int tap_at[4], tap_row[4], tap_col[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int tap = 4 * kq + j;
    tap_at[j] = tap < 9 ? (tap / 3) * ST_XW + tap % 3 : XN;
    tap_row[j] = tap < 9 ? ST_XW : 0;
    tap_col[j] = tap < 9 ? 1 : 0;
  }
  // a block of 16 first-layer pixels: rows qy, columns qx of the lane's pixel
  // (on: it is one; edge: some may lie outside the image)
  const auto first = [&](int qy, int qx, bool on, bool edge, int iy0, int ix0) {
    V8 a;
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = Xt[tap_at[j] + qy * tap_row[j] + qx * tap_col[j]];
    a.u = make_uint4(d[0], d[1], d[2], d[3]);
    const bool inside = !edge || ((unsigned)(iy0 + qy) < (unsigned)H && (unsigned)(ix0 + qx) < (unsigned)Wd);
    uint16_t *o = &It[(qy * SH::IW + SH::slot(qx)) * SH::CS + 4 * kq];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[nt], a.v, (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = fmaxf(c[i] + bb1[nt][i], 0.f);
      uint2 u = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
      if (edge) u = inside ? u : make_uint2(0u, 0u);
      if (on) *reinterpret_cast<uint2 *>(o + nt * 16) = u;
    }
  };
  uint32_t x[NX];
  const auto load = [&](int tile) {
    const int im = tile / per, t = tile - im * per;
    const int y0 = (t / ntx) * (2 * ST_H) - 2, x0 = (t % ntx) * (2 * ST_W) - 2;
    const uint32_t *src = in + (long long)im * H * Wd;
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      const int e = j * SH::THREADS + threadIdx.x;
      const int iy = y0 + e / ST_XW, ix = x0 + e % ST_XW;
      x[j] = e < XN && (unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)Wd
                 ? src[(long long)iy * Wd + ix] : 0u;
    }
  };
  const auto put = [&]() {
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      const int e = j * SH::THREADS + threadIdx.x;
      if (e < XN) Xt[e] = x[j];
    }
  };
  if (threadIdx.x == 0) Xt[XN] = 0u;
  load(blockIdx.x);
  put();
  __syncthreads();
  for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int im = tile / per, t = tile - im * per;
    const int oy0 = (t / ntx) * ST_H, ox0 = (t % ntx) * ST_W;
    const bool more = tile + (int)gridDim.x < n_tiles;
    if (more) load(tile + gridDim.x);
    const int iy0 = 2 * oy0 - 1, ix0 = 2 * ox0 - 1;
    const bool edge = iy0 < 0 || ix0 < 0 || iy0 + SH::IH > H || ix0 + SH::IW > Wd;
    const auto rows = [&](bool e) {  // two blocks a row, rows in turn; then column 32
      for (int qy = wave; qy < SH::IH; qy += ST_WAVES) {
        first(qy, r16, true, e, iy0, ix0);
        first(qy, 16 + r16, true, e, iy0, ix0);
      }
      if (wave == 1) first(r16, 32, true, e, iy0, ix0);
      if (wave == 2) first(16, 32, r16 == 0, e, iy0, ix0);
    };
    if (edge) rows(true);
    else rows(false);
    __syncthreads();
    if (more) put();
    f32x4 acc[SH::PB][2];
    int px[SH::PB];
#pragma unroll
    for (int b = 0; b < SH::PB; ++b) {
      const int rr = (wave * SH::PB + b) * 16 + r16;
      px[b] = ((rr / ST_W) * 2 * SH::IW + rr % ST_W) * SH::CS + 8 * kq;
      acc[b][0] = acc[b][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int o = ((tap / 3) * SH::IW + SH::slot(tap % 3)) * SH::CS;
#pragma unroll
      for (int b = 0; b < SH::PB; ++b) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(It + px[b] + o);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          acc[b][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2[tap][nt], a, acc[b][nt], 0, 0, 0);
      }
    }
#pragma unroll
    for (int b = 0; b < SH::PB; ++b) {
      const int rr = (wave * SH::PB + b) * 16 + r16, oy = oy0 + rr / ST_W, ox = ox0 + rr % ST_W;
      if (oy < Ho && ox < Wo)
        conv_store<32, 2>(out, ((long long)im * Ho + oy) * Wo + ox, kq, acc[b], bb2, 1);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Data gradient of a stride-2 layer: gin = conv^T(gpre), gpre = gout * [out > 0].
// An input pixel meets the taps of its own row and column parity only, 1, 2, 2 or
// 4 of them (2.25 on average instead of 9 mostly empty ones): a 16-pixel matrix
// column block holds pixels of one parity, and a wavefront takes the four blocks of
// the same pixel pairs, nine taps in all.  Weights ([tap][CIN][COUT] as rows of K per
// input channel) and the group's masked gpre (NSUB tiles of 9 x (BW + 1) outputs
// under 16 x 2 BW inputs, zero outside the image) in LDS, staged as by the tiled
// convolution.  Bound by memory: 64x64, 32 -> 32 channels, 256 images 26 us; 58
// with every tap gathered and masked from memory.
// ---------------------------------------------------------------------------
template <int CIN, int COUT, int BW>
struct Dgrad2Shape {
  static constexpr int NSUB = 16 / BW, K = 9 * COUT, LS = K + 8, CS = COUT + 8, NT = CIN / 16;
  static constexpr int IW = BW + 1, PIX = 9 * IW, THREADS = 512;
  static constexpr int CHUNKS = NSUB * PIX * (COUT / 8), NL = (CHUNKS + THREADS - 1) / THREADS;
  static constexpr int W_ELEMS = CIN * LS, I_ELEMS = NSUB * PIX * CS;
  static constexpr int LDS_BYTES = (W_ELEMS + I_ELEMS) * 2;
};

template <int CIN, int COUT, int BW>
__global__ void __launch_bounds__(512)
k_dgrad2_tile(const uint16_t *__restrict__ gout, const uint16_t *__restrict__ out,
              const uint16_t *__restrict__ Wt, uint16_t *__restrict__ gin, int H, int Wd, int Ho,
              int Wo, int n_sub, int ntx, int nty) {
  using SH = Dgrad2Shape<CIN, COUT, BW>;
  constexpr int NL = SH::NL, NT = SH::NT, C8 = COUT / 8, CB = COUT / 32, NSUB = SH::NSUB;
  __shared__ __attribute__((aligned(16))) uint16_t Wl[SH::W_ELEMS];
  __shared__ __attribute__((aligned(16))) uint16_t Gt[SH::I_ELEMS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, r16 = lane & 15;
  const int n_groups = (n_sub + NSUB - 1) / NSUB;
  uint4 g[NL], y[NL];
  const auto load = [&](int group) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int e = j * SH::THREADS + threadIdx.x;
      g[j] = y[j] = make_uint4(0, 0, 0, 0);
      const int pix = e / C8, sub = pix / SH::PIX, rr = pix - sub * SH::PIX;
      const int sid = group * NSUB + sub;
      const TileAt t = tile_of<BW == 8>(sid, ntx, nty);
      const int oy = t.y * 8 + rr / SH::IW, ox = t.x * BW + rr % SH::IW;
      if (e < SH::CHUNKS && sid < n_sub && oy < Ho && ox < Wo) {
        const long long o = (((long long)t.im * Ho + oy) * Wo + ox) * COUT + 8 * (e % C8);
        g[j] = *reinterpret_cast<const uint4 *>(gout + o);
        y[j] = *reinterpret_cast<const uint4 *>(out + o);
      }
    }
  };
  const auto put = [&]() {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int e = j * SH::THREADS + threadIdx.x;
      V8 v, m;
      v.u = g[j];
      m.u = y[j];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (!(bf2f(m.h[i]) > 0.f)) v.h[i] = 0;
      if (e < SH::CHUNKS) *reinterpret_cast<uint4 *>(&Gt[(e / C8) * SH::CS + 8 * (e % C8)]) = v.u;
    }
  };
  load(blockIdx.x);
  for (int e = threadIdx.x; e < 9 * CIN * C8; e += SH::THREADS) {
    const int k8 = e % C8, q = e / C8, tap = q / CIN, ci = q % CIN;
    *reinterpret_cast<uint4 *>(&Wl[ci * SH::LS + tap * COUT + 8 * k8]) =
        *reinterpret_cast<const uint4 *>(Wt + (long long)q * COUT + 8 * k8);
  }
  put();
  __syncthreads();
  // the lane's pixel pair: column bx, row pair rp of tile sub
  const int u = wave * 16 + r16, bx = u % BW, rp = (u / BW) % 8, sub = u / (BW * 8);
  const uint16_t *gp = Gt + (sub * SH::PIX + rp * SH::IW + bx) * SH::CS + 8 * kq;
  const uint16_t *wp = Wl + r16 * SH::LS + 8 * kq;
  for (int group = blockIdx.x; group < n_groups; group += gridDim.x) {
    const bool more = group + (int)gridDim.x < n_groups;
    if (more) load(group + gridDim.x);
    const int sid = group * NSUB + sub;
    const TileAt t = tile_of<BW == 8>(sid, ntx, nty);
    const int py0 = t.y * 16 + 2 * rp, px0 = t.x * (2 * BW) + 2 * bx;
#pragma unroll
    for (int cls = 0; cls < 4; ++cls) {
      const int ay = cls >> 1, ax = cls & 1;  // row and column parity
      f32x4 acc[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
      // odd: taps 0 (the next output on) and 2; even: tap 1
#pragma unroll
      for (int ky = 1 - ay; ky < 3; ky += 2)
#pragma unroll
        for (int kx = 1 - ax; kx < 3; kx += 2)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(
                gp + ((ky == 0 ? SH::IW : 0) + (kx == 0 ? 1 : 0)) * SH::CS + cb * 32);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              const bf16x8 w = *reinterpret_cast<const bf16x8 *>(
                  wp + nt * 16 * SH::LS + (ky * 3 + kx) * COUT + cb * 32);
              acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, acc[nt], 0, 0, 0);
            }
          }
      const int py = py0 + ay, px = px0 + ax;
      if (sid < n_sub && py < H && px < Wd) {
        uint16_t *o = gin + (((long long)t.im * H + py) * Wd + px) * CIN + 4 * kq;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          *reinterpret_cast<uint2 *>(o + nt * 16) =
              make_uint2(f2bf2(acc[nt][0], acc[nt][1]), f2bf2(acc[nt][2], acc[nt][3]));
      }
    }
    if (!more) break;
    __syncthreads();
    put();
    __syncthreads();
  }
}

template <int CIN, int COUT, int BW>
static pvr_status dgrad2_launch(const uint16_t *gout, const uint16_t *out, const uint16_t *wt,
                                uint16_t *gin, int B, int H, int W, hipStream_t stream) {
  using SH = Dgrad2Shape<CIN, COUT, BW>;
  const int ntx = (W + 2 * BW - 1) / (2 * BW), nty = (H + 15) / 16;
  const long long n_sub = (long long)B * ntx * nty;
  if (n_sub > 0x7fff0000LL) return fail(PVR_ESHAPE, "pvr_cnn: more than 2^31 tiles");
  hipLaunchKernelGGL((k_dgrad2_tile<CIN, COUT, BW>),
                     dim3(tile_grid<SH>((n_sub + SH::NSUB - 1) / SH::NSUB)), dim3(SH::THREADS), 0, stream,
                     gout, out, wt, gin, H, W, (H - 1) / 2 + 1, (W - 1) / 2 + 1, (int)n_sub, ntx, nty);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
}

// ---------------------------------------------------------------------------
// weight gradient: dW[co][tap][ci] = sum_p gpre[p][co] in[p @ tap][ci],
// gpre = gout * [out > 0], a GEMM with K = output pixels.
//
// Layers of 32 and 64 input channels, tiled: a workgroup of 16 wavefronts loops over
// groups of output tiles, as the tiled convolution.  A group's gpre (masked once)
// and its input with border, zero outside the image, are staged in LDS as they lie
// in memory, pixels padded by 8 channels; both matrix operands, eight consecutive
// pixels of one channel per lane, come from it by transposing reads (four pixels of
// 16 channels each), so a tap is an address offset and every value is staged once.
// A wavefront owns 16 output by 16 input channels of all nine taps (and, for the
// first 16 input channels, the bias: the product with ones); where a layer has fewer
// such blocks than wavefronts, KS sets of wavefronts share out the pixels.  After
// every `chain` steps of 32 pixels each set writes its sums as a partial block and
// starts anew: k_wgrad_reduce adds the blocks in FP64, in order (deterministic), so
// that no FP32 sum grows longer than wgrad_chain's pixels.  Bound by LDS reads, 10 for 9
// matrix instructions, and by the blocks written and reduced: 32x32, 32 -> 64 channels,
// 256 images 44.6 us with the reduction (35 with the KS sets' sums added in FP32, half
// the blocks); 73 with both operands transposed on their way into LDS, once a tap.
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int CIN, int COUT, int S, int TW, int TH, int NSUB>
struct WgTile {
  static constexpr int MT = COUT / 16, NC = CIN / 16, KS = 16 / (MT * NC);
  static constexpr int IW = (TW - 1) * S + 3, IH = (TH - 1) * S + 3, PIX = IW * IH;
  static constexpr int NE = S == 2 ? (IW + 1) / 2 : 0;
  static constexpr int CI = CIN + 8, CG = COUT + 8;
  static constexpr int PXO = NSUB * TW * TH, STEPS = PXO / 32;
  static constexpr int ICH = NSUB * PIX * (CIN / 8), GCH = PXO * (COUT / 8);
  static constexpr int NI = (ICH + 1023) / 1024, NG = (GCH + 1023) / 1024;
  static constexpr int I_ELEMS = NSUB * PIX * CI, G_ELEMS = PXO * CG;
  static constexpr long long REC = 9LL * COUT * CIN;  // floats per partial block
  __device__ static constexpr int slot(int ix) { return S == 2 ? (ix >> 1) + (ix & 1) * NE : ix; }
};

// Lane (kq, r16): pixels 8 kq .. 8 kq + 7 of channel r16, from p = the address
// of pixel 8 kq + r16 / 4, channels 4 (r16 % 4) on, STRIDE elements a pixel.
template <int STRIDE>
__device__ __forceinline__ bf16x8 read_transposed(const uint16_t *p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * STRIDE));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int CIN, int COUT, int S, int TW, int TH, int NSUB>
__global__ void __launch_bounds__(1024)
k_wgrad_tile(const uint16_t *__restrict__ gout, const uint16_t *__restrict__ out,
             const uint16_t *__restrict__ in, float *__restrict__ part, float *__restrict__ bpart,
             int H, int Wd, int Ho, int Wo, int n_sub, int ntx, int nty, int chain, int blocks) {
  using SH = WgTile<CIN, COUT, S, TW, TH, NSUB>;
  constexpr int NI = SH::NI, NG = SH::NG, C8 = CIN / 8, G8 = COUT / 8;
  __shared__ __attribute__((aligned(16))) uint16_t lds[SH::I_ELEMS + SH::G_ELEMS];
  uint16_t *It = lds, *Gt = lds + SH::I_ELEMS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kq = lane >> 4, r16 = lane & 15;
  const int ks = wave / (SH::MT * SH::NC), wl = wave % (SH::MT * SH::NC);
  const int cm = wl / SH::NC, cn = wl % SH::NC;
  const int n_groups = (n_sub + NSUB - 1) / NSUB;
  uint4 gi[NI], gg[NG], gy[NG];
  const auto load = [&](int group) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int e = j * 1024 + threadIdx.x;
      gi[j] = make_uint4(0, 0, 0, 0);
      const int pix = e / C8, sub = NSUB == 1 ? 0 : pix / SH::PIX, rr = pix - sub * SH::PIX;
      const int sid = group * NSUB + sub;
      const TileAt t = tile_of<TW == 8>(sid, ntx, nty);
      const int iy = t.y * (TH * S) - 1 + rr / SH::IW, ix = t.x * (TW * S) - 1 + rr % SH::IW;
      if (e < SH::ICH && sid < n_sub && (unsigned)iy < (unsigned)H && (unsigned)ix < (unsigned)Wd)
        gi[j] = *reinterpret_cast<const uint4 *>(in + (((long long)t.im * H + iy) * Wd + ix) * CIN + 8 * (e % C8));
    }
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const int e = j * 1024 + threadIdx.x;
      gg[j] = gy[j] = make_uint4(0, 0, 0, 0);
      const int q = e / G8, sub = NSUB == 1 ? 0 : q / (TW * TH), rr = q - sub * (TW * TH);
      const int sid = group * NSUB + sub;
      const TileAt t = tile_of<TW == 8>(sid, ntx, nty);
      const int oy = t.y * TH + rr / TW, ox = t.x * TW + rr % TW;
      if (e < SH::GCH && sid < n_sub && oy < Ho && ox < Wo) {
        const long long o = (((long long)t.im * Ho + oy) * Wo + ox) * COUT + 8 * (e % G8);
        gg[j] = *reinterpret_cast<const uint4 *>(gout + o);
        gy[j] = *reinterpret_cast<const uint4 *>(out + o);
      }
    }
  };
  const auto put = [&]() {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int e = j * 1024 + threadIdx.x;
      const int pix = e / C8, sub = NSUB == 1 ? 0 : pix / SH::PIX, rr = pix - sub * SH::PIX;
      if (e < SH::ICH)
        *reinterpret_cast<uint4 *>(&It[(sub * SH::PIX + (rr / SH::IW) * SH::IW + SH::slot(rr % SH::IW)) * SH::CI +
                                       8 * (e % C8)]) = gi[j];
    }
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const int e = j * 1024 + threadIdx.x;
      V8 v, m;
      v.u = gg[j];
      m.u = gy[j];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (!(bf2f(m.h[i]) > 0.f)) v.h[i] = 0;
      if (e < SH::GCH) *reinterpret_cast<uint4 *>(&Gt[(e / G8) * SH::CG + 8 * (e % G8)]) = v.u;
    }
  };
  f32x4 acc[10];  // nine taps; the bias where cn = 0
#pragma unroll
  for (int t = 0; t < 10; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  bf16x8 ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = 0x3f80;
  // the set's partial blocks: block 0, 1, .. of each set in turn
  long long row = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * blocks * SH::KS + ks;
  int left = chain;
  const auto write = [&]() {
    float *dst = part + row * SH::REC;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dst[((long long)t * COUT + cm * 16 + 4 * kq + i) * CIN + cn * 16 + r16] = acc[t][i];
    if (cn == 0 && r16 == 0)
#pragma unroll
      for (int i = 0; i < 4; ++i) bpart[row * COUT + cm * 16 + 4 * kq + i] = acc[9][i];
#pragma unroll
    for (int t = 0; t < 10; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    row += SH::KS;
    left = chain;
    --blocks;
  };
  load(blockIdx.x);
  put();
  __syncthreads();
  for (int group = blockIdx.x; group < n_groups; group += gridDim.x) {
    const bool more = group + (int)gridDim.x < n_groups;
    if (more) load(group + gridDim.x);
    for (int st = ks + SH::KS * blockIdx.y; st < SH::STEPS; st += SH::KS * gridDim.y) {
      if (left == 0) write();
      --left;
      const int q = st * 32 + 8 * kq + (r16 >> 2);  // (its eight pixels lie in one row)
      const int sub = q / (TW * TH), rr = q % (TW * TH);
      const uint16_t *gp = Gt + q * SH::CG + cm * 16 + 4 * (r16 & 3);
      const uint16_t *ip = It + (sub * SH::PIX + (rr / TW) * S * SH::IW + rr % TW) * SH::CI + cn * 16 + 4 * (r16 & 3);
      const bf16x8 a = read_transposed<SH::CG>(gp);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const bf16x8 b = read_transposed<SH::CI>(ip + ((t / 3) * SH::IW + SH::slot(t % 3)) * SH::CI);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
      }
      if (cn == 0) acc[9] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, acc[9], 0, 0, 0);
    }
    __syncthreads();
    if (more) {
      put();
      __syncthreads();
    }
  }
  while (blocks > 0) write();  // the last sums, and zeros where a workgroup had fewer groups
}

// The first layer (2 input channels): the columns are (tap, ci) flattened and
// padded to 32 with one "tap".  One workgroup (16 waves) takes a chunk of
// pixels and every (co, column) tile.  Per step, each of KSPLIT wave groups
// stages 32 pixels into LDS, transposed so that both MFMA operands are
// 16-byte reads of 8 consecutive pixels: G[co][px] (gpre, with the ReLU mask)
// and I[column][px] (the input at every tap, zero outside the image).  The
// waves of a group share the group's tiles; each group writes its own partial
// block (row chunk * KSPLIT + group).
template <int CIN>
struct WCols {
  static constexpr int n = CIN >= 32 ? CIN : ((9 * CIN + 15) / 16) * 16;
};

template <int CIN, int COUT>
struct WgradShape {
  static constexpr int NC = WCols<CIN>::n;
  static constexpr int TN = NC / 16, TILES = COUT / 16 * TN;
  static constexpr int KSPLIT = 16;                       // one wave a group
  static constexpr int PS = 40;                           // LDS row stride (32 pixels + 8)
  static constexpr int G_ELEMS = COUT * PS, I_ELEMS = NC * PS;
  static constexpr long long REC = (long long)COUT * NC;  // floats per partial block
};

// Pixels per chunk (a multiple of 32 KSPLIT), chosen for about 256 chunks.
static long long wgrad_chunk(long long P, int ksplit) {
  const long long step = 32LL * ksplit;
  long long c = (P + 255) / 256;
  c = (c + step - 1) / step * step;
  return c < step ? step : c;
}

template <int CIN, int COUT, int S>
__global__ void __launch_bounds__(1024)
k_conv_wgrad(const uint16_t *__restrict__ gout, const uint16_t *__restrict__ out,
             const uint16_t *__restrict__ in, float *__restrict__ part,
             float *__restrict__ bpart, int B, int H, int Wd, long long wch) {
  using SH = WgradShape<CIN, COUT>;
  constexpr int NC = SH::NC, TN = SH::TN, TILES = SH::TILES, KSPLIT = SH::KSPLIT, PS = SH::PS;
  __shared__ __attribute__((aligned(16))) uint16_t Gs[KSPLIT * SH::G_ELEMS];
  __shared__ __attribute__((aligned(16))) uint16_t Is[KSPLIT * SH::I_ELEMS];
  const int Ho = (H - 1) / S + 1, Wo = (Wd - 1) / S + 1;
  const long long P = (long long)B * Ho * Wo;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, r16 = lane & 15;
  const int kg = wave;
  // the padding columns (tap, ci) >= 9 CIN stay zero
  for (int e = threadIdx.x; e < KSPLIT * SH::I_ELEMS; e += 1024) Is[e] = 0;
  __syncthreads();
  f32x4 acc[TILES];
#pragma unroll
  for (int q = 0; q < TILES; ++q) acc[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;  // bias partial of (group kg, channel lane) when < COUT
  const long long p0 = (long long)blockIdx.x * wch;
  const long long p1 = p0 + wch < P ? p0 + wch : P;
  for (long long ps = p0; ps < p1; ps += 32 * KSPLIT) {
    // stage gpre (masked by the ReLU) transposed: Gs[g][co][px]
    for (int e = threadIdx.x; e < KSPLIT * 32 * (COUT / 8); e += 1024) {
      const int c8 = e % (COUT / 8), r = e / (COUT / 8);  // r = g * 32 + px
      const int g = r / 32, px = r % 32;
      const long long p = ps + r;
      V8 gv;
      gv.u = make_uint4(0, 0, 0, 0);
      if (p < p1) {
        V8 y;
        gv.u = *reinterpret_cast<const uint4 *>(gout + p * COUT + 8 * c8);
        y.u = *reinterpret_cast<const uint4 *>(out + p * COUT + 8 * c8);
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (!(bf2f(y.h[i]) > 0.f)) gv.h[i] = 0;
      }
      uint16_t *dst = Gs + g * SH::G_ELEMS + (8 * c8) * PS + px;
#pragma unroll
      for (int i = 0; i < 8; ++i) dst[i * PS] = gv.h[i];
    }
    // stage the input at every tap transposed: Is[g][tap][col][px]
    {
      for (int e = threadIdx.x; e < KSPLIT * 32 * 9; e += 1024) {
        const int tap = e % 9, r = e / 9;  // r = g * 32 + px
        const int g = r / 32, px = r % 32;
        const long long p = ps + r;
        uint16_t v[CIN];
#pragma unroll
        for (int c = 0; c < CIN; ++c) v[c] = 0;
        if (p < p1) {
          const int b = (int)(p / (Ho * Wo));
          const int rr = (int)(p % (Ho * Wo));
          const int iy = (rr / Wo) * S + tap / 3 - 1, ix = (rr % Wo) * S + tap % 3 - 1;
          if (iy >= 0 && iy < H && ix >= 0 && ix < Wd)
#pragma unroll
            for (int c = 0; c < CIN; ++c) v[c] = in[(((long long)b * H + iy) * Wd + ix) * CIN + c];
        }
#pragma unroll
        for (int c = 0; c < CIN; ++c) Is[g * SH::I_ELEMS + (tap * CIN + c) * PS + px] = v[c];
      }
    }
    __syncthreads();
    {
      const int co = lane;
      if (co < COUT) {
        const uint16_t *gr = Gs + kg * SH::G_ELEMS + co * PS;
        for (int px = 0; px < 32; ++px) bsum += bf2f(gr[px]);
      }
    }
#pragma unroll
    for (int q = 0; q < TILES; ++q) {
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(
          Gs + kg * SH::G_ELEMS + (q / TN * 16 + r16) * PS + 8 * kq);
      const bf16x8 b = *reinterpret_cast<const bf16x8 *>(
          Is + kg * SH::I_ELEMS + (q % TN * 16 + r16) * PS + 8 * kq);
      acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[q], 0, 0, 0);
    }
    __syncthreads();
  }
  // partial block of this group: part[row][co][col], row = chunk * KSPLIT + group
  const long long row = (long long)blockIdx.x * KSPLIT + kg;
  float *dst = part + row * SH::REC;
#pragma unroll
  for (int q = 0; q < TILES; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      dst[(q / TN * 16 + 4 * kq + i) * NC + q % TN * 16 + r16] = acc[q][i];
  {
    const int co = lane;
    if (co < COUT) bpart[row * COUT + co] = bsum;
  }
}

// dW[co][tap][ci] (FP32, layout of the master weights) and db[co] = sums over
// the partial blocks (rows).  A workgroup of 16 waves takes 64 consecutive
// outputs (one per lane, coalesced loads) and a range of up to RED_ROWS rows;
// wave g sums rows g, g + 16, ... of the range in order (FP64) and the 16
// partial sums are added in wave order.  With one range the result is
// written directly; with several, each range's sums go to `partial` and
// k_wgrad_finish adds them in range order: the result does not depend on the
// launch.  Outputs past COUT * 9 CIN are the bias entries (row stride COUT).
constexpr int RED_WAVES = 16;
constexpr int RED_ROWS = 256;

template <int CIN, int COUT>
__global__ void __launch_bounds__(RED_WAVES * 64)
k_wgrad_reduce(const float *__restrict__ part, const float *__restrict__ bpart, int n_rows,
               float *__restrict__ dW, float *__restrict__ db, double *__restrict__ partial) {
  constexpr int NC = WCols<CIN>::n;
  constexpr int taps = CIN >= 32 ? 9 : 1;
  constexpr int K = 9 * CIN;
  constexpr int NRED = COUT * K + COUT;
  constexpr long long REC = (long long)taps * COUT * NC;
  __shared__ double red[RED_WAVES][64];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int idx = blockIdx.x * 64 + lane;
  const int r0 = blockIdx.y * RED_ROWS;
  const int r1 = n_rows < r0 + RED_ROWS ? n_rows : r0 + RED_ROWS;
  double sum = 0;
  if (idx < COUT * K) {
    const int co = idx / K, k = idx % K;
    const int tap = CIN >= 32 ? k / CIN : 0;
    const int col = CIN >= 32 ? k % CIN : k;
    const float *src = part + ((long long)tap * COUT + co) * NC + col;
    for (int c = r0 + g; c < r1; c += RED_WAVES) sum += src[c * REC];
  } else if (idx < NRED) {
    const float *src = bpart + (idx - COUT * K);
    for (int c = r0 + g; c < r1; c += RED_WAVES) sum += src[(long long)c * COUT];
  }
  red[g][lane] = sum;
  __syncthreads();
  if (g == 0 && idx < NRED) {
    double t = 0;
    for (int w = 0; w < RED_WAVES; ++w) t += red[w][lane];
    if (gridDim.y > 1) partial[(long long)blockIdx.y * NRED + idx] = t;
    else if (idx < COUT * K) dW[idx] = (float)t;
    else db[idx - COUT * K] = (float)t;
  }
}

__global__ void k_wgrad_finish(const double *__restrict__ partial, int ranges, int n_w, int nred,
                               float *__restrict__ dW, float *__restrict__ db) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nred) return;
  double t = 0;
  for (int r = 0; r < ranges; ++r) t += partial[(long long)r * nred + idx];
  if (idx < n_w) dW[idx] = (float)t;
  else db[idx - n_w] = (float)t;
}

// ---------------------------------------------------------------------------
// pair packing: channel 0 = observed patch, channel 1 = simulated patch, each
// normalised to zero mean / unit variance over the patch's valid samples
// (invalid samples 0).  One workgroup per pair; patches are 64 x 64.  Bound by
// memory: a thread's 16 samples of each array are read at once and kept for both
// passes (1024 pairs, 67 MB: 18 us; 36 reading them twice, one at a time).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_pack_pairs(const PatchDev *__restrict__ patches, const int *__restrict__ ids,
             const float *__restrict__ invz, const float *__restrict__ y,
             const float *__restrict__ ys, uint16_t *__restrict__ outp, int M) {
  __shared__ double red[5][4];
  const int bi = blockIdx.x;
  constexpr int n = PVR_CNN_SIDE * PVR_CNN_SIDE, N = n / 256;  // samples, of them a thread's
  const int id = ids[bi];
  if (id < 0 || id >= M) {  // not a patch of the plan: an all-zero pair (uniform per workgroup)
    uint32_t *o32 = reinterpret_cast<uint32_t *>(outp) + (long long)bi * n;
    for (int l = threadIdx.x; l < n; l += 256) o32[l] = 0u;
    return;
  }
  const long long off = patches[id].off + threadIdx.x;
  float yu[N], yv[N], z[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    z[i] = invz[off + 256 * i];
    yu[i] = y[off + 256 * i];
    yv[i] = ys[off + 256 * i];
  }
  double a[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (z[i] > 0.f) {
      const double u = yu[i], v = yv[i];
      a[0] += 1; a[1] += u; a[2] += u * u; a[3] += v; a[4] += v * v;
    }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    double x = a[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[k][wave] = x;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 5; ++k) a[k] = red[k][0] + red[k][1] + red[k][2] + red[k][3];
  const double c = a[0] > 0 ? a[0] : 1.0;
  const double m0 = a[1] / c, m1 = a[3] / c;
  const double s0 = sqrt(fmax(a[2] / c - m0 * m0, 0.0)) + 1e-3;
  const double s1 = sqrt(fmax(a[4] / c - m1 * m1, 0.0)) + 1e-3;
  const double r0 = 1.0 / s0, r1 = 1.0 / s1;
  uint32_t *o32 = reinterpret_cast<uint32_t *>(outp) + (long long)bi * n;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float u = 0.f, v = 0.f;
    if (z[i] > 0.f) {
      u = (float)((yu[i] - m0) * r0);
      v = (float)((yv[i] - m1) * r1);
    }
    o32[threadIdx.x + 256 * i] = f2bf2(u, v);  // both channels of a pixel
  }
}

// ---------------------------------------------------------------------------
// head: fully connected layer from the whole last feature map (hw positions
// x 64 channels, so the weights can depend on position) to 6 outputs,
// weighted squared loss and its gradients.  One workgroup of 256 lanes per
// sample; lane t owns the flattened inputs t, t + 256, ...
// ---------------------------------------------------------------------------
constexpr int HEAD_THREADS = 256;

__global__ void __launch_bounds__(HEAD_THREADS)
k_head(const uint16_t *__restrict__ act, int n_in, const float *__restrict__ Wfc,
       const float *__restrict__ bfc, const float *__restrict__ target,
       const float *__restrict__ lw, float *__restrict__ pred, float *__restrict__ loss_part,
       float *__restrict__ dp_out, uint16_t *__restrict__ gact, float inv_batch) {
  __shared__ float red[6][HEAD_THREADS / 64];
  __shared__ float dp[6];
  const int b = blockIdx.x, t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const uint16_t *a = act + (long long)b * n_in;
  float s[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int e = t; e < n_in; e += HEAD_THREADS) {
    const float x = bf2f(a[e]);
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = fmaf(x, Wfc[e * 6 + k], s[k]);
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    float x = s[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (lane == 0) red[k][wave] = x;
  }
  __syncthreads();
  if (t < 6) {
    float o = bfc[t];
    for (int w = 0; w < HEAD_THREADS / 64; ++w) o += red[t][w];
    pred[b * 6 + t] = o;
    if (target) {
      const float d = o - target[b * 6 + t];
      dp[t] = lw[t] * d * inv_batch;
      dp_out[b * 6 + t] = dp[t];
      loss_part[b * 6 + t] = 0.5f * lw[t] * d * d * inv_batch;
    }
  }
  if (!target) return;
  __syncthreads();
  // dL/dact[e] = sum_k Wfc[e][k] dp[k]
  for (int e = t; e < n_in; e += HEAD_THREADS) {
    float g = 0.f;
#pragma unroll
    for (int k = 0; k < 6; ++k) g = fmaf(Wfc[e * 6 + k], dp[k], g);
    gact[(long long)b * n_in + e] = f2bf(g);
  }
}

// dL/dWfc[e][k] = sum_b act[b][e] dp[b][k], dL/dbfc[k] = sum_b dp[b][k].  A
// workgroup of 16 waves takes 64 inputs e (one per lane; the last lanes past
// n_in take the bias); wave g sums the samples b = g, g + 16, ... in order and
// the 16 partial sums are added in wave order (fixed summation order).
__global__ void __launch_bounds__(RED_WAVES * 64)
k_head_wgrad(const uint16_t *__restrict__ act, const float *__restrict__ dp, int B, int n_in,
             float *__restrict__ dW, float *__restrict__ db) {
  __shared__ float red[RED_WAVES][64][6];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  float acc[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (e < n_in) {
    for (int b = g; b < B; b += RED_WAVES) {
      const float x = bf2f(act[(long long)b * n_in + e]);
#pragma unroll
      for (int k = 0; k < 6; ++k) acc[k] = fmaf(x, dp[b * 6 + k], acc[k]);
    }
  } else if (e < n_in + 6) {
    const int k = e - n_in;
    for (int b = g; b < B; b += RED_WAVES) acc[0] += dp[b * 6 + k];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) red[g][lane][k] = acc[k];
  __syncthreads();
  if (g == 0) {
    float t[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < RED_WAVES; ++w)
#pragma unroll
      for (int k = 0; k < 6; ++k) t[k] += red[w][lane][k];
    if (e < n_in) {
#pragma unroll
      for (int k = 0; k < 6; ++k) dW[e * 6 + k] = t[k];
    } else if (e < n_in + 6) {
      db[e - n_in] = t[0];
    }
  }
}

// sum of per-sample partials (fixed order)
// out[0] = sum of x[0..n) by one workgroup: thread t sums t, t + 1024, ...
// in order (FP64), then a fixed tree over the threads.
__global__ void __launch_bounds__(1024) k_sum_all(const float *__restrict__ x, int n,
                                                  float *__restrict__ out) {
  __shared__ double red[1024];
  double s = 0;
  for (int i = threadIdx.x; i < n; i += 1024) s += x[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (float)red[0];
}

// ---------------------------------------------------------------------------
// Adam on FP32 master weights, refreshing the BF16 copies (forward layout
// [Cout][9][Cin] and, for conv layers, the transposed [9][Cin][Cout]).
// ---------------------------------------------------------------------------
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2, uint16_t *__restrict__ wb, uint16_t *__restrict__ wt,
                       int cout, int cin) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  w[i] = wi;
  if (wb) wb[i] = f2bf(wi);
  if (wt) {
    const int co = i / (9 * cin), k = i % (9 * cin);
    const int tap = k / cin, ci = k % cin;
    wt[((long long)tap * cin + ci) * cout + co] = f2bf(wi);
  }
}

__global__ void k_to_bf16(const float *__restrict__ w, int n, uint16_t *__restrict__ wb,
                          uint16_t *__restrict__ wt, int cout, int cin) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float wi = w[i];
  if (wb) wb[i] = f2bf(wi);
  if (wt) {
    const int co = i / (9 * cin), k = i % (9 * cin);
    const int tap = k / cin, ci = k % cin;
    wt[((long long)tap * cin + ci) * cout + co] = f2bf(wi);
  }
}

// ---------------------------------------------------------------------------
// host entry points
// ---------------------------------------------------------------------------
#define CONV_CASES(X)  \
  X(2, 32, 1)          \
  X(32, 32, 2)         \
  X(32, 64, 1)         \
  X(64, 64, 2)         \
  X(64, 64, 1)         \
  X(32, 32, 1)         \
  X(64, 32, 1)

static int out_size(int n, int s) { return (n - 1) / s + 1; }

template <int CIN, int COUT, int S>
static pvr_status conv_fwd(const uint16_t *in, const uint16_t *w, const float *bias, uint16_t *out,
                           int B, int H, int W, int relu, hipStream_t stream) {
  if constexpr (CIN >= 32) {
    return conv_tiled<CIN, COUT, S, false>(in, nullptr, w, bias, out, B, H, W, relu, stream);
  } else {
    const long long P = (long long)B * out_size(H, S) * out_size(W, S);
    const dim3 grid(persistent_grid((P + FW_TILE - 1) / FW_TILE, FwdShape<CIN, COUT>::LDS_BYTES));
    hipLaunchKernelGGL((k_conv_fwd<CIN, COUT, S>), grid, dim3(FW_THREADS), 0, stream, in, w, bias,
                       out, B, H, W, relu);
    HIP_TRY(hipGetLastError());
    return PVR_OK;
  }
}

template <int CIN, int COUT, int S>
static pvr_status conv_dgrad(const uint16_t *gout, const uint16_t *out, const uint16_t *wt,
                             uint16_t *gin, int B, int H, int W, hipStream_t stream) {
  if constexpr (S == 1) {
    return conv_tiled<COUT, CIN, 1, true>(gout, out, wt, nullptr, gin, B, H, W, 0, stream);
  } else {
    // images of at most 16 x 16 two at a time where there are many, as above (64 -> 64
    // channels: 1024 images 18.0 us, 23.4 in 32 x 16 tiles; 256 images 9.0 and 8.0)
    if (W <= 16 && H <= 16 && B >= SMALL_MIN) return dgrad2_launch<CIN, COUT, 8>(gout, out, wt, gin, B, H, W, stream);
    return dgrad2_launch<CIN, COUT, 16>(gout, out, wt, gin, B, H, W, stream);
  }
}

extern "C" pvr_status pvr_cnn_conv_fwd(const uint16_t *in, const uint16_t *w, const float *bias,
                                       uint16_t *out, int32_t B, int32_t H, int32_t W,
                                       int32_t cin, int32_t cout, int32_t stride, int32_t relu,
                                       hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_conv_fwd", in, 16);
  PVR_ALIGNED("pvr_cnn_conv_fwd", w, 16);
  PVR_ALIGNED("pvr_cnn_conv_fwd", bias, 4);
  PVR_ALIGNED("pvr_cnn_conv_fwd", out, 16);
  if (!in || !w || !bias || !out || B <= 0 || H <= 0 || W <= 0)
    return fail(PVR_EINVAL, "pvr_cnn_conv_fwd: invalid argument");
#define LAUNCH(CI, CO, ST)                                                  \
  if (cin == CI && cout == CO && stride == ST)                              \
    return conv_fwd<CI, CO, ST>(in, w, bias, out, B, H, W, relu, stream);
  CONV_CASES(LAUNCH)
#undef LAUNCH
  return fail(PVR_EUNSUPPORTED, "pvr_cnn_conv_fwd: no kernel for cin %d cout %d stride %d", cin,
              cout, stride);
  PVR_API_END();
}

extern "C" pvr_status pvr_cnn_stem_fwd(const uint16_t *in, const uint16_t *w1, const float *b1,
                                       const uint16_t *w2, const float *b2, uint16_t *out,
                                       int32_t B, int32_t H, int32_t W, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_stem_fwd", in, 16);
  PVR_ALIGNED("pvr_cnn_stem_fwd", w1, 16);
  PVR_ALIGNED("pvr_cnn_stem_fwd", b1, 4);
  PVR_ALIGNED("pvr_cnn_stem_fwd", w2, 16);
  PVR_ALIGNED("pvr_cnn_stem_fwd", b2, 4);
  PVR_ALIGNED("pvr_cnn_stem_fwd", out, 16);
  if (!in || !w1 || !b1 || !w2 || !b2 || !out || B <= 0 || H <= 0 || W <= 0)
    return fail(PVR_EINVAL, "pvr_cnn_stem_fwd: invalid argument");
  const int Ho = out_size(H, 2), Wo = out_size(W, 2);
  const int ntx = (Wo + ST_W - 1) / ST_W, nty = (Ho + ST_H - 1) / ST_H;
  const long long n = (long long)B * ntx * nty;
  if (n > 0x7fff0000LL) return fail(PVR_ESHAPE, "pvr_cnn_stem_fwd: more than 2^31 tiles");
  hipLaunchKernelGGL(k_conv_stem, dim3((unsigned)std::min(n, 768LL)), dim3(64 * ST_WAVES), 0, stream,
                     reinterpret_cast<const uint32_t *>(in), w1, b1, w2, b2, out, H, W, Ho, Wo, (int)n,
                     ntx, nty);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_cnn_conv_dgrad(const uint16_t *gout, const uint16_t *out,
                                         const uint16_t *wt, uint16_t *gin, int32_t B, int32_t H,
                                         int32_t W, int32_t cin, int32_t cout, int32_t stride,
                                         hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_conv_dgrad", gout, 16);
  PVR_ALIGNED("pvr_cnn_conv_dgrad", out, 16);
  PVR_ALIGNED("pvr_cnn_conv_dgrad", wt, 16);
  PVR_ALIGNED("pvr_cnn_conv_dgrad", gin, 16);
  if (!gout || !out || !wt || !gin || B <= 0 || H <= 0 || W <= 0)
    return fail(PVR_EINVAL, "pvr_cnn_conv_dgrad: invalid argument");
#define LAUNCH(CI, CO, ST)                                                \
  if constexpr (CI >= 16)                                                 \
    if (cin == CI && cout == CO && stride == ST)                          \
      return conv_dgrad<(CI >= 16 ? CI : 16), CO, ST>(gout, out, wt, gin, B, H, W, stream);
  CONV_CASES(LAUNCH)
#undef LAUNCH
  return fail(PVR_EUNSUPPORTED, "pvr_cnn_conv_dgrad: no kernel for cin %d cout %d stride %d", cin,
              cout, stride);
  PVR_API_END();
}

// The launch of a layer's weight gradient: partial blocks (rows), floats of each.
struct WgradPlan {
  long long rows, rec, wch;  // wch: pixels per chunk (first layer)
  int n_sub, ntx, nty;       // tiles (other layers)
  int sub;                   // of them a group
  int wgs, split;            // workgroups, and of them to a group
  int chain, blocks;         // steps of a partial block, blocks of a set of wavefronts
  bool small;                // 8 x 8 tiles
};
// Steps of 32 pixels that a set of wavefronts (KS share a layer's pixels) adds up in
// FP32 before it writes a partial block: about 256 KS blocks a layer.  The rounding
// of a weight's sum grows with it.
static int wgrad_chain(long long P, int ks) {
  const long long c = ((P + 255) / 256 + 32LL * ks - 1) / (32LL * ks);
  return c < 1 ? 1 : (int)c;
}
// Workgroups of the tiled kernel: at most one a compute unit, its groups of tiles as
// even as they go; a group of more than one partial block is split over several
// workgroups while there are fewer (16x16, 64 -> 64, 4 images: 11.4 us, 24.6 unsplit).
constexpr int WG_MAX = 256, WG_ONE_TILE = 64;

template <int CIN, int COUT>
static bool wgrad_plan(int B, int H, int W, int stride, WgradPlan &pl) {
  const int Ho = out_size(H, stride), Wo = out_size(W, stride);
  if constexpr (CIN < 32) {
    using SH = WgradShape<CIN, COUT>;
    const long long P = (long long)B * Ho * Wo;
    pl.wch = wgrad_chunk(P, SH::KSPLIT);
    pl.rows = (P + pl.wch - 1) / pl.wch * SH::KSPLIT;
    pl.rec = SH::REC;
    return true;
  } else {
    pl.small = Ho <= 8 && Wo <= 8;
    const int tw = pl.small ? 8 : 16, th = pl.small ? 8 : 16 / stride;
    pl.ntx = (Wo + tw - 1) / tw;
    pl.nty = (Ho + th - 1) / th;
    const long long n_sub = (long long)B * pl.ntx * pl.nty;
    pl.n_sub = (int)n_sub;
    pl.sub = pl.small && n_sub > WG_ONE_TILE ? 4 / stride : 1;
    const long long groups = (n_sub + pl.sub - 1) / pl.sub;
    constexpr int KS = 16 / ((COUT / 16) * (CIN / 16));
    const long long per = std::max(1LL, (groups + WG_MAX - 1) / WG_MAX), wgs = (groups + per - 1) / per;
    const int steps = (pl.sub * tw * th / 32 + KS - 1) / KS;  // of a set, a group
    pl.chain = wgrad_chain((long long)B * Ho * Wo, KS);
    pl.split = wgs < WG_MAX && wgs > 0 ? (int)std::min<long long>((steps + pl.chain - 1) / pl.chain, WG_MAX / wgs) : 1;
    pl.wgs = (int)wgs;
    pl.blocks = (int)((per * ((steps + pl.split - 1) / pl.split) + pl.chain - 1) / pl.chain);
    pl.rows = wgs * pl.split * pl.blocks * KS;
    pl.rec = 9LL * CIN * COUT;
    return n_sub <= 0x7fff0000LL;
  }
}

static long long wgrad_ranges(long long rows) { return (rows + RED_ROWS - 1) / RED_ROWS; }

extern "C" int64_t pvr_cnn_wgrad_scratch(int32_t B, int32_t H, int32_t W, int32_t cin,
                                         int32_t cout, int32_t stride) {
  if (stride != 1 && stride != 2) return 0;
  WgradPlan pl = {};
#define SCR(CI, CO, ST)                                                                     \
  if (cin == CI && cout == CO) {                                                            \
    wgrad_plan<CI, CO>(B, H, W, stride, pl);                                                \
    const long long ranges = wgrad_ranges(pl.rows);                                         \
    return pl.rows * (pl.rec + CO) * (long long)sizeof(float) +                             \
           (ranges > 1 ? ranges * (9LL * CI * CO + CO) * (long long)sizeof(double) : 0);    \
  }
  CONV_CASES(SCR)
#undef SCR
  return 0;
}

template <int CIN, int COUT, int S>
static pvr_status conv_wgrad(const uint16_t *gout, const uint16_t *out, const uint16_t *in,
                             float *scratch, float *dw, float *db, int B, int H, int W,
                             hipStream_t stream) {
  WgradPlan pl = {};
  if (!wgrad_plan<CIN, COUT>(B, H, W, S, pl)) return fail(PVR_ESHAPE, "pvr_cnn: more than 2^31 tiles");
  float *part = scratch, *bpart = scratch + pl.rows * pl.rec;
  if constexpr (CIN < 32) {
    const int chunks = (int)(pl.rows / WgradShape<CIN, COUT>::KSPLIT);
    hipLaunchKernelGGL((k_conv_wgrad<CIN, COUT, S>), dim3(chunks), dim3(1024), 0, stream, gout, out,
                       in, part, bpart, B, H, W, pl.wch);
  } else {
    const int Ho = out_size(H, S), Wo = out_size(W, S);
#define WG_LAUNCH(TW, TH, NSUB)                                                                \
  hipLaunchKernelGGL((k_wgrad_tile<CIN, COUT, S, TW, TH, NSUB>), dim3(pl.wgs, pl.split), dim3(1024), 0, stream, \
                     gout, out, in, part, bpart, H, W, Ho, Wo, pl.n_sub, pl.ntx, pl.nty, pl.chain, pl.blocks)
    if (!pl.small) WG_LAUNCH(16, 16 / S, 1);
    else if (pl.sub == 1) WG_LAUNCH(8, 8, 1);
    else WG_LAUNCH(8, 8, 4 / S);
#undef WG_LAUNCH
  }
  HIP_TRY(hipGetLastError());
  const int nred = COUT * 9 * CIN + COUT;  // weights, then biases
  const int ranges = (int)wgrad_ranges(pl.rows);
  double *partial = ranges > 1 ? (double *)(bpart + pl.rows * COUT) : nullptr;
  hipLaunchKernelGGL((k_wgrad_reduce<CIN, COUT>), dim3((nred + 63) / 64, ranges), dim3(RED_WAVES * 64),
                     0, stream, part, bpart, (int)pl.rows, dw, db, partial);
  HIP_TRY(hipGetLastError());
  if (ranges > 1) {
    hipLaunchKernelGGL(k_wgrad_finish, dim3((nred + 255) / 256), dim3(256), 0, stream, partial, ranges,
                       nred - COUT, nred, dw, db);
    HIP_TRY(hipGetLastError());
  }
  return PVR_OK;
}

extern "C" pvr_status pvr_cnn_conv_wgrad(const uint16_t *gout, const uint16_t *out,
                                         const uint16_t *in, float *scratch, float *dw, float *db,
                                         int32_t B, int32_t H, int32_t W, int32_t cin,
                                         int32_t cout, int32_t stride, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_conv_wgrad", gout, 16);
  PVR_ALIGNED("pvr_cnn_conv_wgrad", out, 16);
  PVR_ALIGNED("pvr_cnn_conv_wgrad", in, 16);
  PVR_ALIGNED("pvr_cnn_conv_wgrad", scratch, 16);
  PVR_ALIGNED("pvr_cnn_conv_wgrad", dw, 4);
  PVR_ALIGNED("pvr_cnn_conv_wgrad", db, 4);
  if (!gout || !out || !in || !scratch || !dw || !db || B <= 0 || H <= 0 || W <= 0)
    return fail(PVR_EINVAL, "pvr_cnn_conv_wgrad: invalid argument");
#define LAUNCH(CI, CO, ST)                                                           \
  if (cin == CI && cout == CO && stride == ST)                                       \
    return conv_wgrad<CI, CO, ST>(gout, out, in, scratch, dw, db, B, H, W, stream);
  CONV_CASES(LAUNCH)
#undef LAUNCH
  return fail(PVR_EUNSUPPORTED, "pvr_cnn_conv_wgrad: no kernel for cin %d cout %d stride %d", cin,
              cout, stride);
  PVR_API_END();
}

extern "C" pvr_status pvr_cnn_pack_pairs(const pvr_plan *p, const int32_t *patch_ids, int32_t B,
                                         const float *y_obs, const float *y_sim, uint16_t *out,
                                         hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_pack_pairs", patch_ids, 4);
  PVR_ALIGNED("pvr_cnn_pack_pairs", y_obs, 4);
  PVR_ALIGNED("pvr_cnn_pack_pairs", y_sim, 4);
  PVR_ALIGNED("pvr_cnn_pack_pairs", out, 4);
  if (!p || !patch_ids || !y_obs || !y_sim || !out || B <= 0)
    return fail(PVR_EINVAL, "pvr_cnn_pack_pairs: invalid argument");
  if (!p->built) return fail(PVR_EINVAL, "pvr_cnn_pack_pairs: plan has not been built");
  for (int s = 0; s < p->M; ++s)
    if (p->h_patch[s].w != PVR_CNN_SIDE || p->h_patch[s].h != PVR_CNN_SIDE)
      return fail(PVR_ESHAPE, "pvr_cnn_pack_pairs: patch %d is not %dx%d", s, PVR_CNN_SIDE,
                  PVR_CNN_SIDE);
  hipLaunchKernelGGL(k_pack_pairs, dim3(B), dim3(256), 0, stream, p->d_patch, patch_ids, p->d_invz,
                     y_obs, y_sim, out, p->M);
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}

extern "C" pvr_status pvr_cnn_head(const uint16_t *act, int32_t B, int32_t hw, const float *wfc,
                                   const float *bfc, const float *target, const float *loss_w,
                                   float *pred, float *loss, uint16_t *gact, float *dwfc,
                                   float *dbfc, float *scratch, hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_head", act, 16);
  PVR_ALIGNED("pvr_cnn_head", wfc, 4);
  PVR_ALIGNED("pvr_cnn_head", bfc, 4);
  PVR_ALIGNED("pvr_cnn_head", target, 4);
  PVR_ALIGNED("pvr_cnn_head", loss_w, 4);
  PVR_ALIGNED("pvr_cnn_head", pred, 4);
  PVR_ALIGNED("pvr_cnn_head", loss, 4);
  PVR_ALIGNED("pvr_cnn_head", gact, 16);
  PVR_ALIGNED("pvr_cnn_head", dwfc, 4);
  PVR_ALIGNED("pvr_cnn_head", dbfc, 4);
  PVR_ALIGNED("pvr_cnn_head", scratch, 16);
  if (!act || !wfc || !bfc || !pred || B <= 0 || hw <= 0) return fail(PVR_EINVAL, "pvr_cnn_head: invalid argument");
  if ((long long)hw * 64 > (1 << 24)) return fail(PVR_ESHAPE, "pvr_cnn_head: hw too large");
  if (target && (!loss_w || !loss || !gact || !dwfc || !dbfc || !scratch))
    return fail(PVR_EINVAL, "pvr_cnn_head: training needs loss weights, outputs and scratch");
  const int n_in = hw * 64;
  float *lp = scratch, *dp = scratch ? scratch + (long long)B * 6 : nullptr;
  hipLaunchKernelGGL(k_head, dim3(B), dim3(HEAD_THREADS), 0, stream, act, n_in, wfc, bfc, target,
                     loss_w, pred, lp, dp, gact, 1.0f / B);
  HIP_TRY(hipGetLastError());
  if (target) {
    hipLaunchKernelGGL(k_sum_all, dim3(1), dim3(1024), 0, stream, lp, B * 6, loss);
    hipLaunchKernelGGL(k_head_wgrad, dim3((n_in + 6 + 63) / 64), dim3(RED_WAVES * 64), 0, stream,
                       act, dp, B, n_in, dwfc, dbfc);
    HIP_TRY(hipGetLastError());
  }
  return PVR_OK;
  PVR_API_END();
}

extern "C" int64_t pvr_cnn_head_scratch(int32_t B) {
  return (long long)B * 12 * (long long)sizeof(float);
}

extern "C" pvr_status pvr_cnn_adam(float *w, const float *g, float *m, float *v, int32_t n,
                                   float lr, float beta1, float beta2, float eps, int32_t step,
                                   uint16_t *w_bf16, uint16_t *wt_bf16, int32_t cout, int32_t cin,
                                   hipStream_t stream) {
  PVR_API_BEGIN();
  PVR_ALIGNED("pvr_cnn_adam", w, 4);
  PVR_ALIGNED("pvr_cnn_adam", g, 4);
  PVR_ALIGNED("pvr_cnn_adam", m, 4);
  PVR_ALIGNED("pvr_cnn_adam", v, 4);
  PVR_ALIGNED("pvr_cnn_adam", w_bf16, 16);
  PVR_ALIGNED("pvr_cnn_adam", wt_bf16, 16);
  if (!w || !m || !v || n <= 0 || step < 0) return fail(PVR_EINVAL, "pvr_cnn_adam: invalid argument");
  if (wt_bf16 && (cout <= 0 || cin <= 0 || cout * 9 * cin != n))
    return fail(PVR_EINVAL, "pvr_cnn_adam: transposed copy needs n = cout * 9 * cin");
  if (step == 0) {
    hipLaunchKernelGGL(k_to_bf16, dim3((n + 255) / 256), dim3(256), 0, stream, w, n, w_bf16,
                       wt_bf16, cout, cin);
  } else {
    if (!g) return fail(PVR_EINVAL, "pvr_cnn_adam: gradient is NULL");
    const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, stream, w, g, m, v, n, lr,
                       beta1, beta2, eps, c1, c2, w_bf16, wt_bf16, cout, cin);
  }
  HIP_TRY(hipGetLastError());
  return PVR_OK;
  PVR_API_END();
}
