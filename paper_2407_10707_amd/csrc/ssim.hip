// Image loss of the training section (Sec. 3.3, image-loss equation):
// L = (1 - lambda) L_1 + lambda (1 - mean SSIM), SSIM with an 11 x 11
// Gaussian window (std 1.5), C1 = 0.01^2, C2 = 0.03^2, every channel filtered
// on its own with zero padding.
//
// With mu = G * x, E_xx = G * x^2, E_xy = G * (x y) (G the separable window)
// and sigma_x^2 = E_xx - mu_x^2, sigma_xy = E_xy - mu_x mu_y, the SSIM of a
// pixel p depends on x through (mu_x, E_xx, E_xy) only, so
//   dS/dx_q = (G * a)_q + 2 x_q (G * b)_q + y_q (G * c)_q
// with a = dS/dmu_x (through the sigmas as well), b = dS/dE_xx and
// c = dS/dE_xy per pixel (G is symmetric, so its adjoint is itself).
//
//   forward   per 32 x 54 tile and channel: x and y with a 5-pixel halo in
//             LDS, the five horizontal sums, the five vertical sums, the
//             SSIM, the (a, b, c) maps for the adjoint, per-tile sums of
//             SSIM and |x - y|
//   adjoint   per tile: (a, b, c) with halo in LDS, the same two passes,
//             then the image gradient with the L1 term
//   final     fixed-order sum of the tile sums -> the loss, by the adjoint's first
//             workgroup (a kernel of its own where no gradient is asked for)
//
// A thread takes eight outputs of a row, then eight of a column, so a value is
// read from LDS once for up to eight windows (one output per thread: 11 reads
// per output and map, and the products of x and y once per tap).  With 54 rows
// and their halo every thread has one row piece in the first pass, and its sums
// stay in registers while the second pass's LDS replaces the first's.  At 3 x
// 1080 x 1080, forward and adjoint: 52 -> 32 us and 38 -> 23 us, of which the tiles
// divided among the XCDs are 1 and 8 (42 and 34 us where each load of the halo
// waited for the one before).  Vector issue is about two thirds and half of that;
// the rest is the loads' latency at four waves per SIMD.
#include "common.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int kThreads = 256;
constexpr int kR = 5;                  // window radius
constexpr int kOut = 8;                // outputs per thread and pass
constexpr int kTW = 32;                // output tile: columns,
constexpr int kTH = kThreads * kOut / kTW - 2 * kR;   // rows: 54
constexpr int kSW = kTW + 2 * kR;      // tile with halo: 42 columns,
constexpr int kSH = kTH + 2 * kR;      // 64 rows
constexpr int kPI = 44, kPH = 36;      // row pitches in LDS (16-byte rows, banks spread)
constexpr int kTaps = kOut + 2 * kR;   // values under eight windows: 18
constexpr float kC1 = 0.0001f;
constexpr float kC2 = 0.0009f;

struct Window {
  float g[2 * kR + 1];
};

Window window() {
  Window w{};
  double s = 0.0, v[2 * kR + 1];
  for (int i = 0; i <= 2 * kR; ++i) {
    const double t = i - kR;
    v[i] = std::exp(-t * t / (2.0 * 1.5 * 1.5));
    s += v[i];
  }
  for (int i = 0; i <= 2 * kR; ++i) w.g[i] = (float)(v[i] / s);
  return w;
}

// Workgroups per row of the grid (a dimension holds less than 2^32 threads).
constexpr int kGridX = 1 << 23;

// The tile of a workgroup (the count of them: none).  Workgroups that share a remainder modulo 8 run on
// the same XCD and take one contiguous eighth of the tiles (row by row), so
// that a tile's halo and the cache lines its rows share with its neighbours are
// in the XCD's L2.
struct Tile {
  int ch, y0, x0, index;
};

__device__ inline Tile tile_of(int tx, int ty, int count) {
  const int per = (count + 7) / 8;
  const int block = blockIdx.y * kGridX + blockIdx.x;
  Tile t;
  t.index = block >= 8 * per ? count : (block % 8) * per + block / 8;
  const int row = t.index / tx;
  t.x0 = kTW * (t.index - row * tx);
  t.ch = row / ty;
  t.y0 = kTH * (row - t.ch * ty);
  return t;
}

// Loads N maps of a tile with halo (zero outside the image) into LDS: a wave
// per row (every fourth), lane = column.  All loads are issued before the first
// is used; those outside the image read its nearest pixel, so none is
// predicated.
template <int N>
__device__ inline void load_halo(const float* const (&src)[N], int H, int W, int y0, int x0,
                                 float (*dst)[kSH][kPI]) {
  constexpr int kWaves = kThreads / 64, kRows = kSH / kWaves;
  const int c = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xx = x0 - kR + c;
  const bool in = xx >= 0 && xx < W;
  const unsigned xc = (unsigned)rga::clampi(xx, 0, W - 1);
  if (c >= kSW) return;
  float v[N][kRows];
#pragma unroll
  for (int t = 0; t < kRows; ++t) {
    const int yc = rga::clampi(y0 - kR + wave + kWaves * t, 0, H - 1);
#pragma unroll
    for (int m = 0; m < N; ++m) v[m][t] = (src[m] + (size_t)yc * W)[xc];
  }
#pragma unroll
  for (int t = 0; t < kRows; ++t) {
    const int r = wave + kWaves * t, yy = y0 - kR + r;
    const bool ok = in && yy >= 0 && yy < H;
#pragma unroll
    for (int m = 0; m < N; ++m) dst[m][r][c] = ok ? v[m][t] : 0.f;
  }
}

// The kTaps (and two more) values of a row from a 16-byte boundary.
__device__ inline void row_read(const float* p, float (&v)[kTaps + 2]) {
#pragma unroll
  for (int q = 0; q < (kTaps + 2) / 4; ++q) {
    const float4 f = *reinterpret_cast<const float4*>(p + 4 * q);
    v[4 * q] = f.x;
    v[4 * q + 1] = f.y;
    v[4 * q + 2] = f.z;
    v[4 * q + 3] = f.w;
  }
}

// Eight window sums over v[0 .. kTaps), taps in order.
__device__ inline void windows(const Window& w, const float (&v)[kTaps + 2], float (&s)[kOut]) {
#pragma unroll
  for (int o = 0; o < kOut; ++o) {
    s[o] = 0.f;
#pragma unroll
    for (int j = 0; j <= 2 * kR; ++j) s[o] = fmaf(w.g[j], v[o + j], s[o]);
  }
}

template <int N>
__device__ inline void rows_write(const float (&s)[N][kOut], float (*hs)[kSH][kPH], int r, int c0) {
#pragma unroll
  for (int q = 0; q < N; ++q) {
    *reinterpret_cast<float4*>(&hs[q][r][c0]) = make_float4(s[q][0], s[q][1], s[q][2], s[q][3]);
    *reinterpret_cast<float4*>(&hs[q][r][c0 + 4]) = make_float4(s[q][4], s[q][5], s[q][6], s[q][7]);
  }
}

// Eight outputs of column c from row r0 on.  (The last group of a tile's rows
// has fewer: the rows past the tile repeat its last one and are not used.)
template <int N>
__device__ inline void columns(const Window& w, float (*hs)[kSH][kPH], int r0, int c,
                               float (&m)[N][kOut]) {
#pragma unroll
  for (int q = 0; q < N; ++q) {
    float v[kTaps + 2] = {};
#pragma unroll
    for (int j = 0; j < kTaps; ++j) v[j] = hs[q][min(r0 + j, kSH - 1)][c];
    windows(w, v, m[q]);
  }
}

// The variances are filtered apart, each less its own squared mean: their sum from
// one map of x^2 + y^2 cancels at twice the magnitude (the gradient's error against
// 64 bits grew by 8 to 14 % on smooth and textured images and by 58 % on flat ones),
// and (x - y)^2 in its place is better near the target only.  LDS holds four maps
// of sums, so that four workgroups fit a CU; those of y^2 follow in the place of
// x's once these are read.
__global__ void __launch_bounds__(kThreads)
ssim_fwd_kernel(int C, int H, int W, int tx, int ty, Window win, const float* __restrict__ img,
                const float* __restrict__ tgt, float* __restrict__ abc, float* __restrict__ part) {
  __shared__ __align__(16) float smem[4 * kSH * kPH];
  static_assert(2 * kPI <= 4 * kPH, "the inputs fit the sums' space");
  __shared__ float red[2][kThreads];
  float (*in)[kSH][kPI] = reinterpret_cast<float (*)[kSH][kPI]>(smem);
  float (*hs)[kSH][kPH] = reinterpret_cast<float (*)[kSH][kPH]>(smem);
  const Tile tile = tile_of(tx, ty, C * tx * ty);
  if (tile.index >= C * tx * ty) return;
  const int ch = tile.ch, x0 = tile.x0, y0 = tile.y0;
  const size_t HW = (size_t)H * W;
  const float* x = img + ch * HW;
  const float* y = tgt + ch * HW;
  {
    const float* const src[2] = {x, y};
    load_halo<2>(src, H, W, y0, x0, in);
  }
  __syncthreads();
  float ssum = 0.f, lsum = 0.f;
  const int hr = threadIdx.x / (kTW / kOut), hc = kOut * (threadIdx.x % (kTW / kOut));
  float syy[1][kOut];
  {
    float a[kTaps + 2], b[kTaps + 2], t[kTaps + 2], s[4][kOut];
    row_read(&in[0][hr][hc], a);
    row_read(&in[1][hr][hc], b);
    // |x - y| of this thread's pixels that belong to the tile and the image
    if (hr >= kR && hr < kR + kTH && y0 + hr - kR < H) {
#pragma unroll
      for (int o = 0; o < kOut; ++o)
        if (x0 + hc + o < W) lsum += fabsf(a[o + kR] - b[o + kR]);
    }
    windows(win, a, s[0]);
    windows(win, b, s[1]);
#pragma unroll
    for (int j = 0; j < kTaps; ++j) t[j] = a[j] * b[j];
    windows(win, t, s[3]);
#pragma unroll
    for (int j = 0; j < kTaps; ++j) {
      a[j] *= a[j];
      b[j] *= b[j];
    }
    windows(win, a, s[2]);
    windows(win, b, syy[0]);
    __syncthreads();
    rows_write<4>(s, hs, hr, hc);
  }
  __syncthreads();
  const int c = threadIdx.x % kTW, r0 = kOut * (threadIdx.x / kTW);
  float m[4][kOut], myy[1][kOut];
  columns<4>(win, hs, r0, c, m);
  __syncthreads();
  rows_write<1>(syy, hs, hr, hc);
  __syncthreads();
  if (r0 < kTH) {
    columns<1>(win, hs, r0, c, myy);
#pragma unroll
    for (int o = 0; o < kOut; ++o) {
      const int yy = y0 + r0 + o, xx = x0 + c;
      if (r0 + o >= kTH || yy >= H || xx >= W) continue;
      const float mx = m[0][o], my = m[1][o];
      const float sxx = m[2][o] - mx * mx, sy2 = myy[0][o] - my * my, sxy = m[3][o] - mx * my;
      const float A1 = 2.f * mx * my + kC1, A2 = 2.f * sxy + kC2;
      const float B1 = mx * mx + my * my + kC1, B2 = sxx + sy2 + kC2;
      const float iB = 1.f / (B1 * B2);
      const float S = A1 * A2 * iB;
      // dS/dmu_x holding the sigmas, dS/dsigma_x^2, dS/dsigma_xy
      const float dmu = 2.f * my * A2 * iB - 2.f * mx * S * (iB * B2);
      const float dsx = -S * (iB * B1);
      const float dsxy = 2.f * A1 * iB;
      const size_t p = (size_t)yy * W + xx;
      abc[ch * HW + p] = dmu - 2.f * mx * dsx - my * dsxy;     // a
      abc[(C + ch) * HW + p] = dsx;                     // b
      abc[(2 * C + ch) * HW + p] = dsxy;                // c
      ssum += S;
    }
  }
  red[0][threadIdx.x] = ssum;
  red[1][threadIdx.x] = lsum;
  __syncthreads();
  for (int o = kThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      red[0][threadIdx.x] += red[0][threadIdx.x + o];
      red[1][threadIdx.x] += red[1][threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[tile.index] = red[0][0];
    part[C * tx * ty + tile.index] = red[1][0];
  }
}

// The loss from the tile sums, in a fixed order, by one workgroup.
struct Final {
  int nb;
  float inv, lam;
  const float* part;
  float* loss;
};

__device__ inline void loss_of(const Final& f, float* red) {
  constexpr int kWaves = kThreads / 64;
  float s = 0.f, l = 0.f;
#pragma unroll 4
  for (int b = threadIdx.x; b < f.nb; b += kThreads) {
    s += f.part[b];
    l += f.part[f.nb + b];
  }
  s = rga::wave_sum(s);
  l = rga::wave_sum(l);
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = s;
    red[kWaves + (threadIdx.x >> 6)] = l;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float ts = 0.f, tl = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      ts += red[w];
      tl += red[kWaves + w];
    }
    f.loss[0] = (1.f - f.lam) * tl * f.inv + f.lam * (1.f - ts * f.inv);
  }
}

__global__ void __launch_bounds__(kThreads)
ssim_bwd_kernel(int C, int H, int W, int tx, int ty, Window win, Final f, float ks, float kl,
                const float* __restrict__ img, const float* __restrict__ tgt, const float* __restrict__ abc,
                float* __restrict__ dimg) {
  __shared__ __align__(16) float smem[3 * kSH * kPI];
  float (*in)[kSH][kPI] = reinterpret_cast<float (*)[kSH][kPI]>(smem);
  float (*hs)[kSH][kPH] = reinterpret_cast<float (*)[kSH][kPH]>(smem);
  const Tile tile = tile_of(tx, ty, C * tx * ty);
  if (tile.index >= C * tx * ty) return;
  const int ch = tile.ch, x0 = tile.x0, y0 = tile.y0;
  const size_t HW = (size_t)H * W;
  // (the first workgroup also forms the loss: a launch of its own took 5 us)
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    loss_of(f, smem);
    __syncthreads();
  }
  {
    const float* const src[3] = {abc + ch * HW, abc + (C + ch) * HW,
                                 abc + (2 * C + ch) * HW};
    load_halo<3>(src, H, W, y0, x0, in);
  }
  // this thread's eight pixels (the nearest inside the image where there is none)
  const int c = threadIdx.x % kTW, r0 = kOut * (threadIdx.x / kTW);
  float xv[kOut], yv[kOut];
#pragma unroll
  for (int o = 0; o < kOut; ++o) {
    const size_t p = ch * HW + (size_t)min(y0 + r0 + o, H - 1) * W + min(x0 + c, W - 1);
    xv[o] = img[p];
    yv[o] = tgt[p];
  }
  __syncthreads();
  {
    const int r = threadIdx.x / (kTW / kOut), c0 = kOut * (threadIdx.x % (kTW / kOut));
    float v[kTaps + 2], s[3][kOut];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      row_read(&in[q][r][c0], v);
      windows(win, v, s[q]);
    }
    __syncthreads();
    rows_write<3>(s, hs, r, c0);
  }
  __syncthreads();
  if (r0 >= kTH || x0 + c >= W) return;
  float m[3][kOut];
  columns<3>(win, hs, r0, c, m);
#pragma unroll
  for (int o = 0; o < kOut; ++o) {
    const int yy = y0 + r0 + o;
    if (r0 + o >= kTH || yy >= H) continue;
    const float dS = m[0][o] + 2.f * xv[o] * m[1][o] + yv[o] * m[2][o];
    const float sg = xv[o] > yv[o] ? 1.f : (xv[o] < yv[o] ? -1.f : 0.f);
    dimg[ch * HW + (size_t)yy * W + x0 + c] = fmaf(ks, dS, kl * sg);
  }
}

__global__ void __launch_bounds__(kThreads)
ssim_final_kernel(Final f) {
  __shared__ float red[2 * kThreads / 64];
  loss_of(f, red);
}

size_t tiles(int C, int H, int W) {
  return (size_t)rga::ceil_div(W, kTW) * rga::ceil_div(H, kTH) * C;
}

}  // namespace

extern "C" size_t image_loss_workspace(int C, int H, int W) {
  if (C < 1 || H < 1 || W < 1) return 0;
  return rga::align_up((size_t)3 * C * H * W * 4, 256) + 2 * tiles(C, H, W) * 4;
}

extern "C" int image_loss(void* stream, int C, int H, int W, const float* image,
                          const float* target, float lambda, float* loss, float* dimage, void* ws,
                          size_t ws_bytes) {
  if (C < 1 || H < 1 || W < 1 || C > 65535 || H > (1 << 20) || W > (1 << 20))
    return rga::fail(RGA_EINVAL, "image_loss: C in 1..65535, H and W in 1..2^20");
  if (!(lambda >= 0.f && lambda <= 1.f)) return rga::fail(RGA_EINVAL, "image_loss: lambda in [0, 1]");
  if (!image || !target || !loss || !ws) return rga::fail(RGA_EINVAL, "image_loss: null pointer");
  if (ws_bytes < image_loss_workspace(C, H, W))
    return rga::fail(RGA_ECAPACITY, "image_loss: workspace too small");
  hipStream_t s = static_cast<hipStream_t>(stream);
  static const Window win = window();
  float* abc = static_cast<float*>(ws);
  float* part = reinterpret_cast<float*>(static_cast<char*>(ws) +
                                         rga::align_up((size_t)3 * C * H * W * 4, 256));
  const int tx = (int)rga::ceil_div(W, kTW), ty = (int)rga::ceil_div(H, kTH);
  const int nb = (int)tiles(C, H, W);
  const int64_t blocks = (int64_t)rga::align_up(nb, 8);
  const dim3 grid((unsigned)std::min<int64_t>(blocks, kGridX), (unsigned)rga::ceil_div(blocks, kGridX));
  const double count = (double)C * H * W;
  RGA_LAUNCH("ssim_fwd", ssim_fwd_kernel, grid, dim3(kThreads), 0, s, C, H, W, tx, ty, win, image, target, abc,
             part);
  const Final fin = {nb, (float)(1.0 / count), lambda, part, loss};
  if (dimage)
    RGA_LAUNCH("ssim_bwd", ssim_bwd_kernel, grid, dim3(kThreads), 0, s, C, H, W, tx, ty, win, fin,
               (float)(-lambda / count), (float)((1.0 - lambda) / count), image, target, abc,
               dimage);
  else
    RGA_LAUNCH("ssim_final", ssim_final_kernel, dim3(1), dim3(kThreads), 0, s, fin);
  RGA_CHECK_LAUNCH("image_loss");
  return RGA_OK;
}
