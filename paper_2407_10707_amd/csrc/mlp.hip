// The pose-dependent vertex displacement dx = d(x, theta) (Sec. 3.1,
// attribute paragraph; Sec. 3.5, implementation details): four hidden layers
// of width 256 with ReLU and a linear output of 3, the coordinates encoded by
// random Fourier features gamma(x) = [sin(2 pi B x), cos(2 pi B x)] (B is
// 64 x 3) and the pose theta (72) appended to every vertex's input.
//
// Every layer is a dense product over the vertices, so it runs on MFMA
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation) in a split form that keeps
// FP32 accuracy: each operand is a bf16 high part plus a bf16 low part and
// a product is taken as hi.hi + lo.hi + hi.lo (the lo.lo term is below FP32
// rounding).
//
//   pack      weights -> bf16 hi/lo operands in the exact per-lane order of
//             the MFMA B operand (one 16-byte load per lane and step), once
//             in forward order and once transposed for the adjoint; the pose
//             is folded into the first layer's bias (b_1 + W_1[:, 128:] theta)
//   forward   one workgroup per 64 vertices, all layers in one kernel: the
//             activations stay in LDS, already split, each wave computes 32
//             of a layer's columns with the weights streaming from L2; the
//             features and the hidden activations are kept for the weight
//             gradient, and a bit each (h > 0) for the adjoint
//   backward  the same shape: dz_5 = ddx, dh = dz W (transposed pack),
//             dz = dh where h > 0; every dz is kept
//   wgrad     dW_l = sum over vertices of dz_l h_{l-1}^T: a workgroup per
//             (layer, chunk of vertices), the inputs staged through LDS once
//             per workgroup; partial sums per chunk (no atomics), then a
//             fixed-order sum over the chunks; dW_1's pose columns are
//             db_1 theta^T and dtheta = W_1[:, 128:]^T db_1
//
// The kept arrays (163 MB each at 39,780 vertices) are laid out by blocks of 32
// vertices, [layer][block][column][32], so that every kernel's workgroup moves
// whole contiguous blocks.
#include "common.h"

#include <algorithm>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kFreqs = RGA_MLP_FREQS;     // 64
constexpr int kPose = RGA_MLP_POSE;       // 72
constexpr int kWidth = RGA_MLP_WIDTH;     // 256
constexpr int kIn1 = 2 * kFreqs + kPose;  // 200
constexpr int kLayers = 5;
constexpr int kParams = RGA_MLP_PARAMS;
constexpr int kAS = kWidth + 8;           // LDS row stride of the activations (bf16)
constexpr int kRows = 32;                 // vertices per block
// forward and adjoint: a workgroup of eight waves, two blocks, each wave 32
// columns of a layer (NQ tiles of 16) for all 64 rows (RT tiles)
constexpr int kWaves = 8;
constexpr int kWgRows = 64;
constexpr int kRT = kWgRows / 16;
constexpr int kNQ = kWidth / 16 / kWaves;
constexpr int kWgBlocks = kWgRows / kRows;
// Chunks of vertices per layer of the weight gradient: its workgroups fit the
// 256 CUs at once, and the layers' shares are as their work (the first has half
// the columns, the last reads half and multiplies little).
__host__ __device__ constexpr int max_chunks(int l) { return l == 0 ? 40 : (l < 4 ? 58 : 40); }
constexpr int kMaxChunks = 58;

// parameter layout: W_1 [256][200], b_1, W_2 [256][256], b_2, W_3, b_3, W_4, b_4, W_5 [3][256], b_5
__host__ __device__ constexpr int n_out(int l) { return l < 4 ? kWidth : 3; }
__host__ __device__ constexpr int n_in(int l) { return l == 0 ? kIn1 : kWidth; }
__host__ __device__ constexpr int w_off(int l) {
  int o = 0;
  for (int i = 0; i < l; ++i) o += n_out(i) * n_in(i) + n_out(i);
  return o;
}
__host__ __device__ constexpr int b_off(int l) { return w_off(l) + n_out(l) * n_in(l); }
static_assert(w_off(kLayers) == kParams, "parameter count");

// forward operand of layer l: reduction over its MFMA inputs (the 128
// Fourier features for l = 0), columns = outputs padded to 16
__host__ __device__ constexpr int f_k(int l) { return l == 0 ? 2 * kFreqs : kWidth; }
__host__ __device__ constexpr int f_n(int l) { return l < 4 ? kWidth : 16; }
__host__ __device__ constexpr int f_off(int l) {
  int o = 0;
  for (int i = 0; i < l; ++i) o += f_k(i) * f_n(i);
  return o;
}
constexpr int kFwdElems = f_off(kLayers);
// transposed operand of layer l = 1..4: reduction over its outputs (padded
// to 32), columns = its 256 inputs
__host__ __device__ constexpr int t_k(int l) { return l < 4 ? kWidth : 32; }
__host__ __device__ constexpr int t_off(int l) {
  int o = kFwdElems;
  for (int i = 1; i < l; ++i) o += t_k(i) * kWidth;
  return o;
}
constexpr int kPackElems = t_off(kLayers);   // per hi and lo

struct MlpLayout {
  int nvp, least;          // padded vertices; at most this many chunks per layer
  size_t pack, bias, feat, h, mask, dz, part, total;
};

// chunks of a layer, and the vertices of each (whole blocks)
__host__ __device__ inline int chunks_of(int l, int least) {
  return max_chunks(l) < least ? max_chunks(l) : least;
}
__host__ __device__ inline int chunk_len(int nvp, int chunks) {
  return (nvp / kRows + chunks - 1) / chunks * kRows;
}

MlpLayout mlp_layout(int nv) {
  MlpLayout L{};
  L.nvp = (int)rga::align_up((size_t)(nv > 0 ? nv : 1), 32);
  L.least = std::max(1, std::min(kMaxChunks, L.nvp / 256));
  const size_t V = (size_t)L.nvp;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t a = o;
    o = rga::align_up(o + bytes, 256);
    return a;
  };
  L.pack = take((size_t)2 * kPackElems * 2);
  L.bias = take((size_t)kLayers * kWidth * 4);
  L.feat = take((size_t)2 * kFreqs * V * 4);
  L.h = take((size_t)4 * kWidth * V * 4);
  L.mask = take((size_t)4 * kWidth * (V / kRows) * 4);
  L.dz = take(((size_t)4 * kWidth + 16) * V * 4);
  L.part = take((size_t)L.least * kParams * 4);
  L.total = o;
  return L;
}

template <typename T>
T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// 8 floats -> bf16 high parts and bf16 low parts (the remainders)
__device__ inline void split8(const float* v, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = (__bf16)v[e];
    hi[e] = h;
    lo[e] = (__bf16)(v[e] - (float)h);
  }
}

__device__ inline f32x4 mfma3(const bf16x8& ah, const bf16x8& al, const bf16x8& bh,
                              const bf16x8& bl, f32x4 acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
  return acc;
}

__device__ inline void load8(const float* p, float* v) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Fragment order of an operand with KS reduction steps of 32: element
// ((ct * KS + ks) * 64 + lane) * 8 + e holds column ct * 16 + lane % 16 and
// reduction index ks * 32 + 8 (lane / 16) + e.
// Workgroups of one wave, one group of 8 elements (or one bias) per thread: bound
// by the latency of the loads, which 256 threads of a workgroup waited for
// together (12.4 -> 7.5 us with the launch).  The pose's share of the first bias is
// one chain of kPose products per row, whose rows are brought to LDS in whole
// lines first (-> 6.9 us).
constexpr int kPackThreads = 64;
constexpr int kPackItems = kPackElems / 8 + kLayers * kWidth;
static_assert(kPackElems / 8 % kPackThreads == 0 && kWidth % kPackThreads == 0,
              "a workgroup packs one kind");

__global__ void __launch_bounds__(kPackThreads)
mlp_pack_kernel(const float* __restrict__ P, const float* __restrict__ theta,
                __bf16* __restrict__ hi, __bf16* __restrict__ lo, float* __restrict__ bias) {
  const int groups = kPackElems / 8;
  const int i = blockIdx.x * kPackThreads + threadIdx.x;
  if (i < groups) {
    const int e0 = 8 * i;
    float v[8];
    if (e0 < kFwdElems) {
      int l = 0;
      while (l + 1 < kLayers && e0 >= f_off(l + 1)) ++l;
      const int KS = f_k(l) / 32, frag = (e0 - f_off(l)) / 8;
      const int lane = frag & 63, t = frag >> 6, ks = t % KS, ct = t / KS;
      const int n = ct * 16 + (lane & 15), kb = ks * 32 + 8 * (lane >> 4);
      for (int e = 0; e < 8; ++e)
        v[e] = n < n_out(l) ? P[w_off(l) + n * n_in(l) + kb + e] : 0.f;
    } else {
      int l = 1;
      while (l + 1 < kLayers && e0 >= t_off(l + 1)) ++l;
      const int KS = t_k(l) / 32, frag = (e0 - t_off(l)) / 8;
      const int lane = frag & 63, t = frag >> 6, ks = t % KS, ct = t / KS;
      const int k = ct * 16 + (lane & 15), nb = ks * 32 + 8 * (lane >> 4);
      for (int e = 0; e < 8; ++e)
        v[e] = nb + e < n_out(l) ? P[w_off(l) + (nb + e) * n_in(l) + k] : 0.f;
    }
    bf16x8 h, l8;
    split8(v, h, l8);
    *reinterpret_cast<bf16x8*>(hi + e0) = h;
    *reinterpret_cast<bf16x8*>(lo + e0) = l8;
  } else {
    const int j = i - groups, l = j / kWidth, n = j % kWidth;
    float b = 0.f;
    if (l == 0) {
      __shared__ float w[kPackThreads][kPose + 1];
      const float* rows = P + w_off(0) + (n - (int)threadIdx.x) * kIn1 + 2 * kFreqs;
#pragma unroll 24
      for (int q = threadIdx.x; q < kPackThreads * kPose; q += kPackThreads)
        w[q / kPose][q % kPose] = rows[q / kPose * kIn1 + q % kPose];
      b = P[b_off(0) + n];
      __syncthreads();
      for (int t = 0; t < kPose; ++t) b = fmaf(w[threadIdx.x][t], theta[t], b);
    } else if (n < n_out(l)) {
      b = P[b_off(l) + n];
    }
    bias[j] = b;
  }
}

// gamma(x): sin and cos of 2 pi (B_j . x), with the 2 folded into the
// argument of sinpi / cospi
__device__ inline float fourier_arg(const float* __restrict__ freqs, int j, float x0, float x1,
                                    float x2) {
  const float a = fmaf(freqs[3 * j + 2], x2, fmaf(freqs[3 * j + 1], x1, freqs[3 * j] * x0));
  return 2.f * a;
}

// Weight fragments (hi, lo) of NQ column tiles at one reduction step.
template <int NQ>
struct Frags {
  bf16x8 h[NQ], l[NQ];
};

template <int NQ>
__device__ inline void frags_load(Frags<NQ>& F, const bf16x8* __restrict__ bh,
                                  const bf16x8* __restrict__ bl, int fo, int KS, int ct0, int ks) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int fi = fo + ((ct0 + q) * KS + ks) * 64 + lane;
    F.h[q] = bh[fi];
    F.l[q] = bl[fi];
  }
}

// The activations of a workgroup's rows, split.  (Split where they are made:
// split where they are read, every wave repeated it for all rows.)
struct Act {
  __bf16 h[kWgRows][kAS], l[kWgRows][kAS];
};

__device__ inline void act_put(Act& A, int r, int n, float v) {
  const __bf16 h = (__bf16)v;
  A.h[r][n] = h;
  A.l[r][n] = (__bf16)(v - (float)h);
}

// One layer's product for a workgroup's rows: wave w takes the kNQ column
// tiles from `ct0`; the activations come from LDS, the weights from global
// memory, those of the next reduction step loaded before the products of the
// current one.  F holds the first step's on entry, and on exit those of the
// next product's first step (`nfo`, `nKS`; none if nKS is 0).
__device__ inline void layer_mm(const Act& A, const bf16x8* __restrict__ bh,
                                const bf16x8* __restrict__ bl, int fo, int KS, int nfo, int nKS,
                                int ct0, Frags<kNQ>& F, f32x4 (&acc)[kRT][kNQ]) {
  const int lane = threadIdx.x & 63, row = lane & 15, g = lane >> 4;
#pragma unroll
  for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
    for (int q = 0; q < kNQ; ++q) acc[rt][q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int ks = 0; ks < KS; ++ks) {
    Frags<kNQ> N;
    if (ks + 1 < KS)
      frags_load<kNQ>(N, bh, bl, fo, KS, ct0, ks + 1);
    else if (nKS > 0)
      frags_load<kNQ>(N, bh, bl, nfo, nKS, ct0, 0);
    else
      N = F;
#pragma unroll
    for (int rt = 0; rt < kRT; ++rt) {
      const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&A.h[rt * 16 + row][ks * 32 + 8 * g]);
      const bf16x8 al = *reinterpret_cast<const bf16x8*>(&A.l[rt * 16 + row][ks * 32 + 8 * g]);
#pragma unroll
      for (int q = 0; q < kNQ; ++q) acc[rt][q] = mfma3(ah, al, F.h[q], F.l[q], acc[rt][q]);
    }
    F = N;
  }
}

// Forward and adjoint: the products take 22 us of the matrix units at 39,780
// vertices, the kept arrays 32 us of memory each way; the rest is the latency of
// a workgroup's steps and stores (one alone takes 30 and 20 us, and 2.4 follow
// each other on a CU in pairs).  Activations split where they are made, one LDS
// set instead of two, sign bits instead of the activations in the adjoint and
// contiguous blocks: 100 -> 80 us and 110 -> 70 us.  (Twice the rows per
// workgroup halves the weights' traffic at the same time; three more steps of
// weights in flight do not fit the registers.)
__global__ void __launch_bounds__(64 * kWaves, 4)
mlp_forward_kernel(int nv, int nblk, const float* __restrict__ x, const float* __restrict__ freqs,
                   const __bf16* __restrict__ phi, const __bf16* __restrict__ plo,
                   const float* __restrict__ bias, float* __restrict__ feat,
                   float* __restrict__ H, uint32_t* __restrict__ mask, float* __restrict__ out) {
  __shared__ __align__(16) Act act;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = lane & 15, g = lane >> 4;
  const int blk0 = kWgBlocks * blockIdx.x, r0 = blk0 * kRows;
  const bf16x8* bh = reinterpret_cast<const bf16x8*>(phi);
  const bf16x8* bl = reinterpret_cast<const bf16x8*>(plo);
  Frags<kNQ> F;
  frags_load<kNQ>(F, bh, bl, f_off(0) / 8, f_k(0) / 32, kNQ * wave, 0);
  // Fourier features: lane = frequency, eight rows per wave
  {
    constexpr int U = kWgRows / kWaves;
    const int u0 = U * wave;
    float sn[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = r0 + u0 + u;
      const bool in = v < nv;
      const int vc = in ? v : 0;
      const float x0 = in ? x[vc] : 0.f, x1 = in ? x[nv + vc] : 0.f, x2 = in ? x[2 * nv + vc] : 0.f;
      const float f = fourier_arg(freqs, lane, x0, x1, x2);
      sn[u] = sinpif(f);
      cs[u] = cospif(f);
      act_put(act, u0 + u, lane, sn[u]);
      act_put(act, u0 + u, kFreqs + lane, cs[u]);
    }
    const int blk = blk0 + u0 / kRows;
    if (blk < nblk) {
      float* fs = feat + ((size_t)blk * 2 * kFreqs + lane) * kRows + u0 % kRows;
      float* fc = fs + kFreqs * kRows;
#pragma unroll
      for (int u = 0; u < U; u += 4) {
        *reinterpret_cast<float4*>(fs + u) = make_float4(sn[u], sn[u + 1], sn[u + 2], sn[u + 3]);
        *reinterpret_cast<float4*>(fc + u) = make_float4(cs[u], cs[u + 1], cs[u + 2], cs[u + 3]);
      }
    }
  }
  __syncthreads();
  for (int l = 0; l < kLayers - 1; ++l) {
    f32x4 acc[kRT][kNQ];
    const bool last = l == kLayers - 2;
    layer_mm(act, bh, bl, f_off(l) / 8, f_k(l) / 32, f_off(l + 1) / 8, last ? 0 : f_k(l + 1) / 32,
             kNQ * wave, F, acc);
    __syncthreads();                     // every wave is done with the inputs
#pragma unroll
    for (int q = 0; q < kNQ; ++q) {
      const int n = (kNQ * wave + q) * 16 + row;
      const float bn = bias[l * kWidth + n];
#pragma unroll
      for (int b = 0; b < kWgBlocks; ++b) {
        uint32_t on = 0u;
        const size_t at = ((size_t)l * nblk + blk0 + b) * kWidth + n;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          float hv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 16 * t + 4 * g + i;
            const float h = fmaxf(acc[2 * b + t][q][i] + bn, 0.f);
            act_put(act, kRows * b + r, n, h);
            hv[i] = r0 + kRows * b + r < nv ? h : 0.f;
            on |= hv[i] > 0.f ? 1u << r : 0u;
          }
          if (blk0 + b < nblk)
            *reinterpret_cast<float4*>(H + at * kRows + 16 * t + 4 * g) =
                make_float4(hv[0], hv[1], hv[2], hv[3]);
        }
        on |= __shfl_xor(on, 16);
        on |= __shfl_xor(on, 32);
        if (g == 0 && blk0 + b < nblk) mask[at] = on;
      }
    }
    __syncthreads();
  }
  if (wave < kRT) {                      // the output layer: one column tile, a row tile per wave
    constexpr int KS = f_k(kLayers - 1) / 32;
    Frags<KS> W;                         // (tile 0 of each reduction step)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int fi = f_off(kLayers - 1) / 8 + ks * 64 + lane;
      W.h[ks] = bh[fi];
      W.l[ks] = bl[fi];
    }
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&act.h[wave * 16 + row][ks * 32 + 8 * g]);
      const bf16x8 al = *reinterpret_cast<const bf16x8*>(&act.l[wave * 16 + row][ks * 32 + 8 * g]);
      acc = mfma3(ah, al, W.h[ks], W.l[ks], acc);
    }
    if (row < 3)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int v = r0 + wave * 16 + 4 * g + i;
        if (v < nv) out[(size_t)row * nv + v] = acc[i] + bias[(kLayers - 1) * kWidth + row];
      }
  }
}

__global__ void __launch_bounds__(64 * kWaves, 4)
mlp_backward_kernel(int nv, int nblk, const float* __restrict__ ddx,
                    const __bf16* __restrict__ phi, const __bf16* __restrict__ plo,
                    const uint32_t* __restrict__ mask, float* __restrict__ dZ) {
  __shared__ __align__(16) Act act;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = lane & 15, g = lane >> 4;
  const int blk0 = kWgBlocks * blockIdx.x, r0 = blk0 * kRows;
  const bf16x8* bh = reinterpret_cast<const bf16x8*>(phi);
  const bf16x8* bl = reinterpret_cast<const bf16x8*>(plo);
  Frags<kNQ> F;
  frags_load<kNQ>(F, bh, bl, t_off(kLayers - 1) / 8, t_k(kLayers - 1) / 32, kNQ * wave, 0);
  // dz_5 = ddx, as 32 reduction columns (3 used)
  for (int t = threadIdx.x; t < kWgRows * 32; t += blockDim.x) {
    const int r = t % kWgRows, c = t / kWgRows, v = r0 + r;
    const float d = (c < 3 && v < nv) ? ddx[(size_t)c * nv + v] : 0.f;
    act_put(act, r, c, d);
    const int blk = blk0 + r / kRows;
    if (c < 16 && blk < nblk)
      dZ[((size_t)4 * nblk * kWidth + (size_t)blk * 16 + c) * kRows + r % kRows] = d;
  }
  __syncthreads();
  for (int l = kLayers - 1; l >= 1; --l) {
    f32x4 acc[kRT][kNQ];
    uint32_t on[kWgBlocks][kNQ];
#pragma unroll
    for (int b = 0; b < kWgBlocks; ++b)
#pragma unroll
      for (int q = 0; q < kNQ; ++q)
        on[b][q] = mask[((size_t)(l - 1) * nblk + min(blk0 + b, nblk - 1)) * kWidth +
                        (kNQ * wave + q) * 16 + row];
    layer_mm(act, bh, bl, t_off(l) / 8, t_k(l) / 32, t_off(l - 1) / 8, l > 1 ? t_k(l - 1) / 32 : 0,
             kNQ * wave, F, acc);
    __syncthreads();
    // dz of hidden layer l - 1 (the input of layer l): dh where h > 0
#pragma unroll
    for (int q = 0; q < kNQ; ++q) {
      const int n = (kNQ * wave + q) * 16 + row;
#pragma unroll
      for (int b = 0; b < kWgBlocks; ++b)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          float dv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = 16 * t + 4 * g + i;
            dv[i] = (on[b][q] >> r) & 1u ? acc[2 * b + t][q][i] : 0.f;
            act_put(act, kRows * b + r, n, dv[i]);
          }
          if (blk0 + b < nblk)
            *reinterpret_cast<float4*>(dZ + (((size_t)(l - 1) * nblk + blk0 + b) * kWidth + n) * kRows +
                                       16 * t + 4 * g) = make_float4(dv[0], dv[1], dv[2], dv[3]);
        }
    }
    __syncthreads();
  }
}

// dW_l of one layer over one chunk of vertices, the whole layer per
// workgroup so that every operand row is read once per chunk (a workgroup
// per 64 x 128 tile re-reads dz twice and h four times); all five layers run
// side by side: the first layer's Fourier columns (256 x 128), the hidden
// layers (256 x 256, h_{l-1} from the forward) and the output layer (3 x 256,
// its dz padded to 16 rows).  Eight waves, each RT row tiles x NCT column
// tiles of 16 x 16.  Both operands of a 32-vertex step are split into bf16
// hi / lo fragments in LDS (A = dz rows, B = the layer's inputs),
// double-buffered: each thread loads its share of the next step into
// registers before this step's MFMAs and splits and stores it after them, so
// the loads' latency is spent under the products.  The db sums come from the
// same loads.
// Bound by the reading of the kept arrays (340 MB, 3.6 TB/s): 110 -> 96 us at
// 39,780 vertices by reading contiguous blocks, keeping the features (20 MB;
// computed again they made the first layer's workgroups the slowest) and
// dividing the chunks by the layers' work.
constexpr int kLayerThreads = 512;
constexpr int kLayerWaves = kLayerThreads / 64;
constexpr int kFragA = 16 * 64;   // A fragments per step buffer (256 rows)
constexpr int kFragB = 16 * 64;   // B fragments per step buffer (256 columns)

struct WgradLds {
  bf16x8 a[2][2][kFragA];   // [buffer][hi, lo][row tile * 64 + lane]
  bf16x8 b[2][2][kFragB];   // [buffer][hi, lo][column tile * 64 + lane]
};

template <int NQ, int NRT, int RT, int NCT>
__device__ inline void wgrad_layer(int l, int c, int v0, int v1, int nvp, const float* hin,
                                   const float* dZ, float* part, WgradLds& S) {
  constexpr int NRG = kLayerWaves * NCT / NQ;                  // row groups of waves
  static_assert(NRG * RT == NRT, "the waves cover the layer's rows");
  constexpr int FA = NRT * 64, FB = NQ * 64;                   // fragments per step
  constexpr int PA = (FA + kLayerThreads - 1) / kLayerThreads;  // per thread
  constexpr int PB = FB / kLayerThreads;                        // loaded per thread (B)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, g = lane >> 4;
  const int n0 = 16 * RT * (wave % NRG), q0 = NCT * (wave / NRG);
  const int nrows = l < 4 ? kWidth : 16;
  const float* dz = dZ + (size_t)l * kWidth * nvp;
  // fragment f = 64 t + L of either operand: row (or column) 16 t + L % 16,
  // vertices vb + 8 (L / 16) .. + 7 (the MFMA operand order)
  float ra[PA][8], rb[PB][8];
  float dsum[PA];
#pragma unroll
  for (int p = 0; p < PA; ++p) dsum[p] = 0.f;
  auto load = [&](int vb) {
#pragma unroll
    for (int p = 0; p < PA; ++p) {
      const int f = threadIdx.x + p * kLayerThreads;
      const int n = 16 * (f >> 6) + (f & 15), va = 8 * ((f & 63) >> 4);
      if (f < FA && n < nrows) {
        load8(dz + (size_t)vb * nrows + n * kRows + va, ra[p]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) ra[p][e] = 0.f;
      }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int f = threadIdx.x + p * kLayerThreads;
      const int col = 16 * (f >> 6) + (f & 15), va = 8 * ((f & 63) >> 4);
      load8(hin + (size_t)vb * 16 * NQ + col * kRows + va, rb[p]);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int p = 0; p < PA; ++p) {
      const int f = threadIdx.x + p * kLayerThreads;
      if (f < FA) {
        bf16x8 h, lo;
        split8(ra[p], h, lo);
        S.a[buf][0][f] = h;
        S.a[buf][1][f] = lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) dsum[p] += ra[p][e];
      }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int f = threadIdx.x + p * kLayerThreads;
      bf16x8 h, lo;
      split8(rb[p], h, lo);
      S.b[buf][0][f] = h;
      S.b[buf][1][f] = lo;
    }
  };
  f32x4 acc[RT][NCT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int j = 0; j < NCT; ++j) acc[rt][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int buf = 0;
  if (v0 < v1) {
    load(v0);
    store(0);
  }
  __syncthreads();
  for (int vb = v0; vb < v1; vb += 32) {
    const bool more = vb + 32 < v1;
    if (more) load(vb + 32);
    bf16x8 ah[RT], al[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int f = (n0 / 16 + rt) * 64 + lane;
      ah[rt] = S.a[buf][0][f];
      al[rt] = S.a[buf][1][f];
    }
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
      const bf16x8 bh = S.b[buf][0][(q0 + j) * 64 + lane];
      const bf16x8 bl = S.b[buf][1][(q0 + j) * 64 + lane];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt][j] = mfma3(ah[rt], al[rt], bh, bl, acc[rt][j]);
    }
    // the other buffer's readers all passed the barrier that ended the
    // previous step
    if (more) store(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  float* pc = part + (size_t)c * kParams;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
      const int k = 16 * (q0 + j) + row;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = n0 + 16 * rt + 4 * g + i;
        if (n < n_out(l)) pc[w_off(l) + n * n_in(l) + k] = acc[rt][j][i];
      }
    }
  // db: fragment f's thread summed row 16 (f >> 6) + f % 16 over its
  // vertex quarter (f % 64) / 16; the four quarters are lanes L, L ^ 16,
  // L ^ 32, L ^ 48 of one wave
#pragma unroll
  for (int p = 0; p < PA; ++p) {
    float d = dsum[p];
    d += __shfl_xor(d, 16);
    d += __shfl_xor(d, 32);
    const int f = threadIdx.x + p * kLayerThreads;
    const int n = 16 * (f >> 6) + (f & 15);
    if (f < FA && lane < 16 && n < n_out(l)) pc[b_off(l) + n] = d;
  }
}

__global__ void __launch_bounds__(kLayerThreads)
mlp_wgrad_layer_kernel(int nvp, int least, const float* __restrict__ feat,
                       const float* __restrict__ H, const float* __restrict__ dZ,
                       float* __restrict__ part) {
  __shared__ WgradLds S;
  // the workgroups run over the layers' chunks, the full layers first
  int l = 1, c = blockIdx.x;
  while (c >= chunks_of(l, least)) {
    c -= chunks_of(l, least);
    l = l == 3 ? 0 : (l == 0 ? 4 : l + 1);
  }
  const int len = chunk_len(nvp, chunks_of(l, least));
  const int v0 = min(nvp, c * len), v1 = min(nvp, v0 + len);
  const float* hin = l == 0 ? feat : H + (size_t)(l - 1) * kWidth * nvp;
  if (l == 0)
    wgrad_layer<2 * kFreqs / 16, 16, 4, 4>(l, c, v0, v1, nvp, hin, dZ, part, S);
  else if (l < 4)
    wgrad_layer<kWidth / 16, 16, 4, 8>(l, c, v0, v1, nvp, hin, dZ, part, S);
  else
    wgrad_layer<kWidth / 16, 1, 1, 2>(l, c, v0, v1, nvp, hin, dZ, part, S);
}

// Sum of one parameter's partials over the chunks, in order (the loads of 16
// are in flight together: one at a time, the sums of 51 chunks took 27 us).
__device__ inline float chunk_sum(const float* __restrict__ part, int p, int chunks) {
  float s = 0.f;
  int c = 0;
  for (; c + 16 <= chunks; c += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = part[(size_t)(c + u) * kParams + p];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += v[u];
  }
  for (; c < chunks; ++c) s += part[(size_t)c * kParams + p];
  return s;
}

// dparams = sum over the chunks (fixed order); W_1's pose columns are
// db_1 theta^T (the pose is shared by every vertex).  The first workgroup:
// dtheta = W_1[:, 128:]^T db_1 (db_1 summed over the chunks first; the
// 256-term products in four fixed quarters, then added in order).
__global__ void __launch_bounds__(256)
mlp_reduce_kernel(int least, const float* __restrict__ theta, const float* __restrict__ P,
                  const float* __restrict__ part, float* __restrict__ dP,
                  float* __restrict__ dtheta) {
  if (blockIdx.x == 0) {
    __shared__ float db[kWidth];
    __shared__ float quarter[4 * kPose];
    static_assert(kWidth == 256, "a thread per bias");
    db[threadIdx.x] = chunk_sum(part, b_off(0) + threadIdx.x, chunks_of(0, least));
    __syncthreads();
    for (int t = threadIdx.x; t < 4 * kPose; t += 256) {
      const int k = t % kPose, q = t / kPose;
      float a = 0.f;
#pragma unroll 16
      for (int n = 64 * q; n < 64 * q + 64; ++n)
        a = fmaf(P[w_off(0) + n * kIn1 + 2 * kFreqs + k], db[n], a);
      quarter[t] = a;
    }
    __syncthreads();
    if (threadIdx.x < kPose) {
      const float* q = quarter + threadIdx.x;
      dtheta[threadIdx.x] = ((q[0] + q[kPose]) + q[2 * kPose]) + q[3 * kPose];
    }
    return;
  }
  const int p = (blockIdx.x - 1) * blockDim.x + threadIdx.x;
  if (p >= kParams) return;
  const int l = p < w_off(1) ? 0 : (p < w_off(4) ? 1 : 4);    // (layers 1 to 3 have alike many)
  const int chunks = chunks_of(l, least);
  const int k = p % kIn1;
  if (p < b_off(0) && k >= 2 * kFreqs)
    dP[p] = chunk_sum(part, b_off(0) + p / kIn1, chunks) * theta[k - 2 * kFreqs];
  else
    dP[p] = chunk_sum(part, p, chunks);
}

}  // namespace

extern "C" size_t mlp_workspace(int nv) {
  if (nv < 0) return 0;
  return mlp_layout(nv).total;
}

extern "C" int mlp_forward(void* stream, int nv, const float* x, const float* freqs,
                           const float* theta, const float* params, void* ws, size_t ws_bytes,
                           float* dx) {
  if (nv < 0 || nv > (1 << 26)) return rga::fail(RGA_EINVAL, "mlp_forward: nv in 0..2^26");
  if (!freqs || !theta || !params || !ws || (nv > 0 && (!x || !dx)))
    return rga::fail(RGA_EINVAL, "mlp_forward: null pointer");
  const MlpLayout L = mlp_layout(nv);
  if (ws_bytes < L.total) return rga::fail(RGA_ECAPACITY, "mlp_forward: workspace too small");
  if (!rga::aligned16(ws)) return rga::fail(RGA_EINVAL, "mlp_forward: workspace not 16-byte aligned");
  hipStream_t s = static_cast<hipStream_t>(stream);
  __bf16* hi = at<__bf16>(ws, L.pack);
  __bf16* lo = hi + kPackElems;
  RGA_LAUNCH("mlp_pack", mlp_pack_kernel, dim3(kPackItems / kPackThreads), dim3(kPackThreads), 0,
             s, params, theta, hi, lo, at<float>(ws, L.bias));
  // with no vertices the kernel still clears the kept activations of the
  // padding rows, which the adjoint reads
  RGA_LAUNCH("mlp_fwd", mlp_forward_kernel, dim3(rga::ceil_div(L.nvp, kWgRows)), dim3(64 * kWaves), 0,
             s, nv, L.nvp / kRows, x, freqs, hi, lo, at<float>(ws, L.bias), at<float>(ws, L.feat),
             at<float>(ws, L.h), at<uint32_t>(ws, L.mask), dx);
  RGA_CHECK_LAUNCH("mlp_forward");
  return RGA_OK;
}

extern "C" int mlp_backward(void* stream, int nv, const float* x, const float* freqs,
                            const float* theta, const float* params, const float* ddx, void* ws,
                            size_t ws_bytes, float* dparams, float* dtheta) {
  if (nv < 0 || nv > (1 << 26)) return rga::fail(RGA_EINVAL, "mlp_backward: nv in 0..2^26");
  if (!freqs || !theta || !params || !ws || !dparams || !dtheta || (nv > 0 && (!x || !ddx)))
    return rga::fail(RGA_EINVAL, "mlp_backward: null pointer");
  const MlpLayout L = mlp_layout(nv);
  if (ws_bytes < L.total) return rga::fail(RGA_ECAPACITY, "mlp_backward: workspace too small");
  if (!rga::aligned16(ws)) return rga::fail(RGA_EINVAL, "mlp_backward: workspace not 16-byte aligned");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const __bf16* hi = at<__bf16>(ws, L.pack);
  const __bf16* lo = hi + kPackElems;
  float* part = at<float>(ws, L.part);
  // with no vertices every partial sum is zero: the backward and the
  // weight-gradient kernels still run over the (zero) padding rows
  RGA_LAUNCH("mlp_bwd", mlp_backward_kernel, dim3(rga::ceil_div(L.nvp, kWgRows)), dim3(64 * kWaves), 0,
             s, nv, L.nvp / kRows, ddx, hi, lo, at<uint32_t>(ws, L.mask), at<float>(ws, L.dz));
  int groups = 0;
  for (int l = 0; l < kLayers; ++l) groups += chunks_of(l, L.least);
  RGA_LAUNCH("mlp_wgrad", mlp_wgrad_layer_kernel, dim3(groups), dim3(kLayerThreads), 0, s, L.nvp,
             L.least, at<float>(ws, L.feat), at<float>(ws, L.h), at<float>(ws, L.dz), part);
  RGA_LAUNCH("mlp_reduce", mlp_reduce_kernel, dim3(1 + rga::ceil_div(kParams, 256)), dim3(256), 0, s,
             L.least, theta, params, part, dparams, dtheta);
  RGA_CHECK_LAUNCH("mlp_backward");
  return RGA_OK;
}
