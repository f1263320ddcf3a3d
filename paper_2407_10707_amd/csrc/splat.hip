// Tile-based Gaussian splatting (the 3DGS rasterizer used in Sec. 3.1 of the
// paper): projection, tile binning, depth + tile radix sort, front-to-back
// alpha compositing, and the hand-written adjoint.
//
// Pipeline on one stream, no host synchronisation:
//   preprocess        1 thread / splat: camera transform, covariance, conic,
//                     opacity-aware tile rectangle, packed 48-byte record;
//                     also clears the frame's ranges, counters and sums
//   depth sort        of (depth bits, index): up to 16,384 splats by counting
//                     the keys before each, else a stable LSD radix sort in
//                     3 passes of 11-bit digits, each [upsweep of per-block
//                     digit counts, per-digit scan, ranked scatter]; culled
//                     splats carry key 0xFFFFFFFF and leave with the first
//   touched sums      tiles touched by each block of splats in depth order
//                     (with few splats the depth sort adds them up)
//   duplicate         one (tile, splat) entry per touched tile, emitted in
//                     depth order -> D
//   tile sort         stable LSD radix sort of the entries by tile id (one
//                     pass up to 4096 tiles) -> per tile, entries in
//                     (depth bits, index) order
//   ranges            tile boundaries in the sorted entries (written by the
//                     tile sort's scatter when it takes one pass)
//   blend             one workgroup per 8 x 8 pixel block walks the tile's list
//                     until the block has stopped, each wave for one of its
//                     4 x 4 sub-blocks; the adjoint over the 64-entry
//                     sub-chunks that were composited
// Stable ranking inside a radix pass uses wave64 ballots (one per digit bit
// gives the lanes that share a digit) and mbcnt-style lane masks.
#include "common.h"

#include <algorithm>

#include <math.h>

namespace {

constexpr int kTile = 16;
constexpr int kRadixThreads = 256;
constexpr int kItemsD = 8;       // per thread, passes over the duplicates
constexpr int kItemsN = 2;       // per thread, passes over the splats
constexpr int kBlockD = kRadixThreads * kItemsD;
constexpr int kBlockN = kRadixThreads * kItemsN;
constexpr int kSub = 64;         // list entries per sub-chunk of the blend passes
constexpr int kBlocks = 4;       // 8 x 8 pixel blocks of a tile
constexpr int kGrad = 16;        // floats per splat of the adjoint sums (9 used, one 64-byte line)
constexpr float kHalfNegLog2e = -0.72134752f;   // -log2(e) / 2
constexpr float kInvHalfLog2e = 1.38629436f;    // 2 / log2(e) = 2 ln 2
// Digit widths of the tile sort: one pass of the narrowest that holds the tiles
// up to 4096 of them, two of 7 bits up to 16,384 and of 8 up to 65,536 (4,624
// tiles, 3.4 million entries: two passes of 11 bits 185 us with their scans, of 7
// bits 70: the digit tables are 16 times smaller), else of 11.
constexpr int kDigitBits = 11;
constexpr int kRadix = 1 << kDigitBits;
constexpr int kMaxBits = 12;
constexpr int kDepthBits = 11;   // digit width of the depth sort: 3 passes over 32-bit keys
constexpr int kDepthPasses = (32 + kDepthBits - 1) / kDepthBits;
constexpr int kManySplats = 1 << 17;

// Deep lists are walked in parts, side by side (see the blend): a list of two part
// lengths or more.  Up to 65,536 entries in all a part is 1/64 of them, one workgroup
// per CU, at least 256; beyond that 1,024 (a walk of 22 us, where the launches of a
// frame's other steps take longer than a shorter one saves: 100k splats over 500^2,
// paper's mesh, frame 308 us with 1,024, 312 with 512, 314 with 256; 30k splats on 37
// tiles, 22,699 entries, blend and adjoint 108, 85 and 73, now 79) or, so that all parts
// together are about as many workgroups as the chip holds, 1/256 of all entries.
// What decides is each list's own length, known on the device: the mean over an
// image's tiles says nothing of an avatar that covers a few of them.
constexpr int kPart = 1024;
constexpr int kPartMin = 256;
constexpr int kPartsMin = 64;    // of all lists, up to kPart * kPartsMin entries
constexpr int kParts = 256;      // the same of more entries, about
constexpr int kListParts = 128;  // of one list
constexpr int kPartBits = 7;     // an item of the part list: tile << kPartBits | part

__device__ inline uint32_t part_length(int64_t entries) {   // (at most 2^31 - 1)
  static_assert(kParts == 256 && kPartsMin == 64, "shifts");
  const uint32_t n = (uint32_t)entries, few = min(max((n + 63u) >> 6, (uint32_t)kPartMin), (uint32_t)kPart);
  return (max((n + 255u) >> 8, few) + kSub - 1) / kSub * kSub;
}

__device__ inline bool is_deep(int L, uint32_t part) { return (uint32_t)L >= 2 * part; }

// parts of a deep list of L entries
__device__ inline int list_parts(int L, uint32_t part) {
  return (int)min(((uint32_t)L + part - 1) / part, (uint32_t)kListParts);
}

// Room for the parts: lists of more than two lengths each have at most half as
// many parts again as whole lengths.  None where no list can be that long.
inline int part_slots(int64_t n, int64_t cap) {
  if (n < 2 * kPartMin) return 0;
  const int64_t few = std::min<int64_t>(kPartsMin, cap / kPartMin);
  return (int)std::max(few, std::min<int64_t>(kParts, cap / kPart)) * 3 / 2 + 1;
}

// What the blend keeps of the parts, one array behind the other (one address keeps
// its scalar registers free): per (place, block, pixel) the (C, T) of a part, then
// the (C, T) before it; T alone for the parts beside it; per (first place, block)
// the number of arrived parts; per (place, block) the sub-chunks entered; the
// items, a deep list's parts but the first; the lists' first places by tile.
constexpr int kPartWords = kBlocks * 64 + kBlocks;   // cleared per place: T and arrivals

struct Parts {
  char* ws;
  int slots;               // 0: no list can be deep
  __device__ float4* state() const { return reinterpret_cast<float4*>(ws); }
  __device__ __host__ uint32_t* T() const {
    return reinterpret_cast<uint32_t*>(ws + (size_t)slots * kBlocks * 64 * 16);
  }
  __device__ uint32_t* arrived() const { return T() + (size_t)slots * kBlocks * 64; }
  __device__ uint32_t* live() const { return arrived() + slots * kBlocks; }
  __device__ uint32_t* items() const { return live() + slots * kBlocks; }
  __device__ uint32_t* base() const { return items() + slots; }
};

inline size_t parts_bytes(int slots, int64_t tiles) {
  return slots ? (size_t)slots * (kBlocks * 64 * 16 + 4 * (kPartWords + kBlocks + 1)) + 4 * tiles : 0;
}

struct Layout {
  size_t rec, mean2d, conic, depth, rect, touched, fp64, keys0, vals0, keys1, vals1;
  size_t tk0, tv0, tk1, tv1, ranges, hist, binoff, bintot, bsum, count, grad;
  size_t nlive, last, mask, state, part, total;
  int tiles_x, tiles_y, nb_n, nb_cap, nb_max, tile_passes;
  int slots;       // parts that the deep lists have room for
  int tile_bits;   // digit width of the tile sort: 7, 8, 10, 11 or 12
};

Layout make_layout(int n, int width, int height, int64_t cap) {
  Layout L{};
  L.tiles_x = (width + kTile - 1) / kTile;
  L.tiles_y = (height + kTile - 1) / kTile;
  const int64_t tiles = (int64_t)L.tiles_x * L.tiles_y;
  L.nb_n = (int)rga::ceil_div(n > 0 ? n : 1, kBlockN);
  L.nb_cap = (int)rga::ceil_div(cap > 0 ? cap : 1, kBlockD);
  L.nb_max = L.nb_n > L.nb_cap ? L.nb_n : L.nb_cap;
  int bits = 0;
  while ((1ll << bits) < tiles) ++bits;
  L.tile_passes = bits <= kMaxBits ? 1 : (bits <= 2 * kDigitBits ? 2 : 3);
  L.tile_bits = bits > 16 ? kDigitBits
                          : (bits > 14 || bits <= 8 ? 8 : (bits > kMaxBits ? 7 : (bits <= 10 ? 10 : bits)));
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = rga::align_up(o + bytes, 256);
    return at;
  };
  const size_t N = (size_t)(n > 0 ? n : 1);
  const size_t C = (size_t)(cap > 0 ? cap : 1);
  L.rec = take(N * 48);
  L.mean2d = take(N * 8);
  L.conic = take(N * 12);
  L.depth = take(N * 4);
  L.rect = take(N * 16);
  L.touched = take(N * 4);
  L.fp64 = take(N);
  L.keys0 = take(N * 4);
  L.vals0 = take(N * 4);
  L.keys1 = take(N * 4);
  L.vals1 = take(N * 4);
  L.tk0 = take(C * 4);
  L.tv0 = take(C * 4);
  L.tk1 = take(C * 4);
  L.tv1 = take(C * 4);
  L.ranges = take((size_t)tiles * 8);
  L.hist = take((size_t)L.nb_max * (1 << kMaxBits) * 4);
  L.binoff = take((size_t)L.nb_max * (1 << kMaxBits) * 4);
  L.bintot = take((1 << kMaxBits) * 4);
  L.bsum = take((size_t)L.nb_n * 4);
  L.count = take(32);   // int64 [0] = D, [1] = places and items of the deep lists (32 bits each),
                        // [3] = splats that touch a tile
  L.grad = take(N * kGrad * 4);   // adjoint sums per splat: mean2d, conic, opacity, colour
  // blend state: tile t's sub-chunk m of its list [start, end) has the slot
  // start / 64 + t + m, distinct for every (tile, sub-chunk)
  const size_t slots = C / kSub + (size_t)tiles + 1;
  L.nlive = take((size_t)tiles * kBlocks * 4);
  L.last = take((size_t)tiles * kBlocks * 64 * 4);
  L.mask = take(slots * kBlocks * 8);
  L.state = take(slots * 4 * 256 * 4);
  L.slots = part_slots(n, cap);
  L.part = take(parts_bytes(L.slots, tiles));
  L.total = o;
  return L;
}

template <typename T>
__device__ __host__ inline T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

struct CamDev {
  float R[9], t[3], fx, fy, cx, cy;
  int W, H;
};

CamDev to_dev(const rga_camera* c) {
  CamDev d;
  for (int i = 0; i < 9; ++i) d.R[i] = c->R[i];
  for (int i = 0; i < 3; ++i) d.t[i] = c->t[i];
  d.fx = c->fx;
  d.fy = c->fy;
  d.cx = c->cx;
  d.cy = c->cy;
  d.W = c->width;
  d.H = c->height;
  return d;
}

constexpr uint32_t kCulled = 0xFFFFFFFFu;   // depth key of a splat that touches no tile
constexpr uint32_t kNoPart = 0xFFFFFFFFu;   // a part not finished (the bits of a NaN)

// exp for the scales: Cody-Waite reduction by ln 2, degree-7 Taylor
// polynomial, fixed FP32 operation order (reproducible bit for bit).
__device__ inline float exp_repro(float x) {
  x = fminf(fmaxf(x, -87.f), 88.f);
  const float k = rintf(x * 1.44269502f);
  float r = fmaf(-k, 0.693145752f, x);
  r = fmaf(-k, 1.42860677e-6f, r);
  float p = 1.f / 5040.f;
  p = fmaf(p, r, 1.f / 720.f);
  p = fmaf(p, r, 1.f / 120.f);
  p = fmaf(p, r, 1.f / 24.f);
  p = fmaf(p, r, 1.f / 6.f);
  p = fmaf(p, r, 0.5f);
  p = fmaf(p, r, 1.f);
  p = fmaf(p, r, 1.f);
  return ldexpf(p, (int)k);
}

// Upper bound of ln y (y >= 1) from exact operations: y = m 2^e, m in [1,2),
// ln y <= e ln 2 + (m - 1) / sqrt(m).
__device__ inline float ln_upper(float y) {
  int e;
  const float m = frexpf(y, &e) * 2.f;
  return (float)(e - 1) * 0.693147182f + (m - 1.f) / sqrtf(m);
}

// ---- forward geometry shared by preprocess and its adjoint ----------------
struct Geo {
  float X, Y, Z, xzr, yzr, J00, J11, J02, J12;
  float s[3], q[4], inv, Rq[9], A[9], M[9], V[9], T[6];
  float a, b, c;
};

__device__ inline void geo_forward(const CamDev& cam, const float* __restrict__ x,
                                   const float* __restrict__ A, const float* __restrict__ quat,
                                   const float* __restrict__ log_s, int n, int g, Geo& G,
                                   bool& ok_quat) {
  const float* Rc = cam.R;
  const float x0 = x[g], x1 = x[n + g], x2 = x[2 * n + g];
  G.X = fmaf(Rc[2], x2, fmaf(Rc[1], x1, fmaf(Rc[0], x0, cam.t[0])));
  G.Y = fmaf(Rc[5], x2, fmaf(Rc[4], x1, fmaf(Rc[3], x0, cam.t[1])));
  G.Z = fmaf(Rc[8], x2, fmaf(Rc[7], x1, fmaf(Rc[6], x0, cam.t[2])));
  for (int j = 0; j < 3; ++j) G.s[j] = exp_repro(log_s[j * n + g]);
  const float q0 = quat[g], q1 = quat[n + g], q2 = quat[2 * n + g], q3 = quat[3 * n + g];
  const float qq = fmaf(q3, q3, fmaf(q2, q2, fmaf(q1, q1, q0 * q0)));
  ok_quat = qq > 0.f;
  G.inv = 1.f / sqrtf(ok_quat ? qq : 1.f);
  const float qw = q0 * G.inv, qx = q1 * G.inv, qy = q2 * G.inv, qz = q3 * G.inv;
  G.q[0] = qw;
  G.q[1] = qx;
  G.q[2] = qy;
  G.q[3] = qz;
  const float xx = qx * qx, yy = qy * qy, zz = qz * qz;
  const float xy = qx * qy, xz = qx * qz, yz = qy * qz;
  const float wx = qw * qx, wy = qw * qy, wz = qw * qz;
  G.Rq[0] = 1.f - 2.f * (yy + zz);
  G.Rq[1] = 2.f * (xy - wz);
  G.Rq[2] = 2.f * (xz + wy);
  G.Rq[3] = 2.f * (xy + wz);
  G.Rq[4] = 1.f - 2.f * (xx + zz);
  G.Rq[5] = 2.f * (yz - wx);
  G.Rq[6] = 2.f * (xz - wy);
  G.Rq[7] = 2.f * (yz + wx);
  G.Rq[8] = 1.f - 2.f * (xx + yy);
  for (int k = 0; k < 9; ++k) G.A[k] = A[k * n + g];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      G.M[3 * i + j] = fmaf(G.A[3 * i + 2], G.Rq[6 + j],
                            fmaf(G.A[3 * i + 1], G.Rq[3 + j], G.A[3 * i] * G.Rq[j])) * G.s[j];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      G.V[3 * i + j] = fmaf(Rc[3 * i + 2], G.M[6 + j], fmaf(Rc[3 * i + 1], G.M[3 + j], Rc[3 * i] * G.M[j]));
  G.xzr = G.X / G.Z;
  G.yzr = G.Y / G.Z;
  G.J00 = cam.fx / G.Z;
  G.J11 = cam.fy / G.Z;
  G.J02 = -(G.J00 * G.xzr);
  G.J12 = -(G.J11 * G.yzr);
  for (int j = 0; j < 3; ++j) {
    G.T[j] = fmaf(G.J02, G.V[6 + j], G.J00 * G.V[j]);
    G.T[3 + j] = fmaf(G.J12, G.V[6 + j], G.J11 * G.V[3 + j]);
  }
  G.a = fmaf(G.T[2], G.T[2], fmaf(G.T[1], G.T[1], G.T[0] * G.T[0])) + 0.3f;
  G.b = fmaf(G.T[2], G.T[5], fmaf(G.T[1], G.T[4], G.T[0] * G.T[3]));
  G.c = fmaf(G.T[5], G.T[5], fmaf(G.T[4], G.T[4], G.T[3] * G.T[3])) + 0.3f;
}

// FP64 2x2 covariance of a near-degenerate splat from the same FP32 inputs.
struct Geo64 {
  double M[9], V[9], T[6], J00, J11, J02, J12, a, b, c, det;
};

__device__ inline void geo_forward64(const CamDev& cam, const Geo& G, Geo64& D) {
  const float* Rc = cam.R;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      D.M[3 * i + j] = fma((double)G.A[3 * i + 2], (double)G.Rq[6 + j],
                           fma((double)G.A[3 * i + 1], (double)G.Rq[3 + j],
                               (double)G.A[3 * i] * (double)G.Rq[j])) * (double)G.s[j];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      D.V[3 * i + j] = fma((double)Rc[3 * i + 2], D.M[6 + j],
                           fma((double)Rc[3 * i + 1], D.M[3 + j], (double)Rc[3 * i] * D.M[j]));
  const double Zd = (double)G.Z;
  D.J00 = (double)cam.fx / Zd;
  D.J11 = (double)cam.fy / Zd;
  D.J02 = -(D.J00 * ((double)G.X / Zd));
  D.J12 = -(D.J11 * ((double)G.Y / Zd));
  for (int j = 0; j < 3; ++j) {
    D.T[j] = fma(D.J02, D.V[6 + j], D.J00 * D.V[j]);
    D.T[3 + j] = fma(D.J12, D.V[6 + j], D.J11 * D.V[3 + j]);
  }
  D.a = fma(D.T[2], D.T[2], fma(D.T[1], D.T[1], D.T[0] * D.T[0])) + 0.3;
  D.b = fma(D.T[2], D.T[5], fma(D.T[1], D.T[4], D.T[0] * D.T[3]));
  D.c = fma(D.T[5], D.T[5], fma(D.T[4], D.T[4], D.T[3] * D.T[3])) + 0.3;
  D.det = fma(D.a, D.c, -(D.b * D.b));
}

// ---- preprocess -------------------------------------------------------------
__global__ void __launch_bounds__(256)
preprocess_kernel(int n, CamDev cam, int TX, int TY, const float* __restrict__ x,
                  const float* __restrict__ A, const float* __restrict__ quat,
                  const float* __restrict__ log_s, const float* __restrict__ opac,
                  const uint8_t* __restrict__ front,
                  float4* __restrict__ rec, float* __restrict__ mean2d, float* __restrict__ conic,
                  float* __restrict__ depth, int32_t* __restrict__ rect,
                  int32_t* __restrict__ touched, uint8_t* __restrict__ fp64,
                  uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                  uint32_t* __restrict__ ranges_u32, int64_t nranges, uint32_t* __restrict__ cnt4,
                  float4* __restrict__ grad, uint4* __restrict__ part_t, int64_t nparts4,
                  uint32_t* __restrict__ bsum, int nsums) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  // the frame's tile ranges start empty, its counters at zero, and so do the
  // adjoint's sums of the splats in the lists (below); no part is finished
  for (int64_t i = g; i < nparts4; i += (int64_t)gridDim.x * blockDim.x)
    part_t[i] = make_uint4(kNoPart, kNoPart, kNoPart, kNoPart);
  if (g < nranges) ranges_u32[g] = 0u;
  if (g < 8) cnt4[g] = 0u;
  if (g < nsums) bsum[g] = 0u;
  if (g >= n) return;
  Geo G;
  bool okq;
  geo_forward(cam, x, A, quat, log_s, n, g, G, okq);
  const float o = opac[g];
  bool valid = (G.Z > 0.2f) && front[g] && (o >= 1.f / 255.f) && okq;
  float ca = 0.f, cb = 0.f, cc = 0.f;
  uint8_t used64 = 0;
  if (valid) {
    const float det = fmaf(G.a, G.c, -(G.b * G.b));
    if (det <= (G.a * G.c) * 0x1p-12f) {
      Geo64 D;
      geo_forward64(cam, G, D);
      if (D.det > 0.0) {
        ca = (float)(D.c / D.det);
        cb = (float)(-D.b / D.det);
        cc = (float)(D.a / D.det);
        used64 = 1;
      } else {
        valid = false;
      }
    } else {
      ca = G.c / det;
      cb = -G.b / det;
      cc = G.a / det;
    }
  }
  const float u = fmaf(cam.fx, G.xzr, cam.cx);
  const float v = fmaf(cam.fy, G.yzr, cam.cy);
  int tx0 = 0, ty0 = 0, tx1 = -1, ty1 = -1, cnt = 0;
  float r2_cull = 0.f;
  if (valid) {
    const float r2 = 2.f * ln_upper(255.f * o);
    r2_cull = r2;
    const float hx = sqrtf(r2 * G.a) * 1.001f + 1e-3f;
    const float hy = sqrtf(r2 * G.c) * 1.001f + 1e-3f;
    float fx0 = floorf((u - hx) * 0.0625f), fx1 = floorf((u + hx) * 0.0625f);
    float fy0 = floorf((v - hy) * 0.0625f), fy1 = floorf((v + hy) * 0.0625f);
    const bool finite = (fx0 == fx0) && (fx1 == fx1) && (fy0 == fy0) && (fy1 == fy1);
    fx0 = fmaxf(fx0, 0.f);
    fy0 = fmaxf(fy0, 0.f);
    fx1 = fminf(fx1, (float)(TX - 1));
    fy1 = fminf(fy1, (float)(TY - 1));
    if (finite && fx0 <= fx1 && fy0 <= fy1) {
      tx0 = (int)fx0;
      ty0 = (int)fy0;
      tx1 = (int)fx1;
      ty1 = (int)fy1;
      cnt = (tx1 - tx0 + 1) * (ty1 - ty0 + 1);
    }
  }
  // the blend evaluates the exponent of alpha in base 2: the record holds
  // the conic scaled by -log2(e) / 2 (cross term by -log2(e)); the blend
  // passes put the colour into its empty slots when they stage it
  rec[3 * g + 0] = make_float4(u, v, ca * kHalfNegLog2e, cb * (2.f * kHalfNegLog2e));
  rec[3 * g + 1] = make_float4(cc * kHalfNegLog2e, o, 0.f, 0.f);
  // for the blend's per-wave culling: the slopes of the exponent's maxima
  // along vertical and horizontal lines, and a lower bound of the exponent
  // any pixel with alpha >= 1/255 can have (r2 bounds 2 ln(255 o) from
  // above; the margin covers the rounding of both evaluations)
  const float thr = valid ? (r2_cull * kHalfNegLog2e) * 1.01f - 0.01f : 0.f;
  rec[3 * g + 2] = make_float4(0.f, valid ? -cb / cc : 0.f, valid ? -cb / ca : 0.f, thr);
  mean2d[g] = valid ? u : 0.f;
  mean2d[n + g] = valid ? v : 0.f;
  conic[g] = ca;
  conic[n + g] = cb;
  conic[2 * n + g] = cc;
  depth[g] = G.Z;
  rect[g] = tx0;
  rect[n + g] = ty0;
  rect[2 * n + g] = tx1;
  rect[3 * n + g] = ty1;
  touched[g] = cnt;
  if (cnt > 0) {
#pragma unroll
    for (int q = 0; q < 3; ++q) grad[(size_t)g * (kGrad / 4) + q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  fp64[g] = used64;
  keys[g] = cnt > 0 ? __float_as_uint(G.Z) : kCulled;
  vals[g] = (uint32_t)g;
}

// The back-face rule (a Gaussian whose normal faces away from the camera
// gets zero opacity), for a caller that bins before it shades: the same
// FP32 expression, in the same order, as the shading kernels' decision, so
// the flags agree bit for bit.
__global__ void __launch_bounds__(256)
back_face_kernel(int n, const float* __restrict__ x, const float* __restrict__ nrm, float c0,
                 float c1, float c2, uint8_t* __restrict__ front) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const float w0 = c0 - x[g], w1 = c1 - x[n + g], w2 = c2 - x[2 * (size_t)n + g];
  const float m0 = nrm[g], m1 = nrm[n + g], m2 = nrm[2 * (size_t)n + g];
  front[g] = fmaf(m2, w2, fmaf(m1, w1, m0 * w0)) > 0.f ? 1 : 0;
}

// A splat's record for the blend passes, with its colour (slots 6-8, left
// empty by the projection: the binning runs before the colours exist).
struct SplatRec {
  float4 r0, r1, r2;
};
__device__ inline SplatRec load_rec(const float4* __restrict__ rec, const float* __restrict__ color,
                                    int n, uint32_t g) {
  SplatRec R{rec[3 * g], rec[3 * g + 1], rec[3 * g + 2]};
  R.r1.z = color[g];
  R.r1.w = color[(size_t)n + g];
  R.r2.x = color[2 * (size_t)n + g];
  return R;
}

// A tile's deep list of L entries among the parts; `next` gives out the places and
// the items (two words behind D, or LDS where one workgroup has all lists).
__device__ inline void deep_list(const Parts& P, uint32_t* next, int t, int L, uint32_t part) {
  const int k = list_parts(L, part);
  P.base()[t] = atomicAdd(next, (uint32_t)k);
  uint32_t* const item = P.items() + atomicAdd(next + 1, (uint32_t)(k - 1));
  for (int y = 1; y < k; ++y) item[y - 1] = (uint32_t)t << kPartBits | (uint32_t)y;
}

// ---- radix sort (reduce-then-scan, stable) ----------------------------------
__device__ inline int64_t live_count(const int64_t* cnt_ptr, int64_t fixed, int64_t cap) {
  int64_t c = cnt_ptr ? *cnt_ptr : fixed;
  return c < cap ? c : cap;
}

// The digit tables hold a block's 2^BITS counts side by side, or (narrow digits,
// whose tables are short) a digit's counts of all nb blocks, so that the scan
// reads and writes whole lines: 1,655 blocks of 128 digits 13 -> 5 us.
template <int BITS>
__device__ inline size_t table_at(int block, int d, int nb) {
  return BITS <= 8 ? (size_t)d * nb + block : (size_t)block * (1 << BITS) + d;
}

// Per-block digit histogram (LDS integer atomics), digits of BITS bits.  With
// LIVE the items of key kCulled are left out (by the scatter too).
template <int ITEMS, int BITS, bool LIVE = false>
__global__ void __launch_bounds__(kRadixThreads)
radix_upsweep(const uint32_t* __restrict__ keys, const int64_t* cnt_ptr, int64_t fixed,
              int64_t cap, int shift, uint32_t* __restrict__ hist) {
  constexpr int kRadix = 1 << BITS;
  __shared__ uint32_t h[kRadix];
  const int64_t count = live_count(cnt_ptr, fixed, cap);
  const int64_t base = (int64_t)blockIdx.x * (kRadixThreads * ITEMS);
  if (base >= count) return;              // no items: the scan skips this block
  for (int d = threadIdx.x; d < kRadix; d += kRadixThreads) h[d] = 0;
  __syncthreads();
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = base + (int64_t)r * kRadixThreads + threadIdx.x;
    if (i < count) {
      const uint32_t k = keys[i];
      if (!LIVE || k != kCulled) atomicAdd(&h[(k >> shift) & (kRadix - 1)], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < kRadix; d += kRadixThreads)
    hist[table_at<BITS>(blockIdx.x, d, gridDim.x)] = h[d];
}

// Exclusive scan of each digit's counts over the blocks that hold items
// (the rest of a capacity-sized grid is skipped): 8 digits per workgroup,
// 32 threads per digit each summing a run of blocks (held in registers for
// runs of up to kHeld blocks); the 32 run sums of a digit are scanned with
// wave shuffles (lanes d, d + 8, ..., of each wave) and the four wave totals.
template <int BITS>
__global__ void __launch_bounds__(256)
radix_binscan(const uint32_t* __restrict__ hist, int nb, const int64_t* cnt_ptr, int64_t fixed,
              int64_t cap, int block_items, uint32_t* __restrict__ binoff,
              uint32_t* __restrict__ bintot) {
  constexpr int kRadix = 1 << BITS;
  constexpr int kHeld = 8;
  static_assert(BITS > 8, "a table of blocks");
  __shared__ uint32_t wtot[4][8];
  const int dl = threadIdx.x & 7, c = threadIdx.x >> 3;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d = blockIdx.x * 8 + dl;
  const int64_t count = live_count(cnt_ptr, fixed, cap);
  const int nbl = (int)min((int64_t)nb, (count + block_items - 1) / block_items);
  const int chunk = (nbl + 31) / 32;
  const int j0 = c * chunk, j1 = min(nbl, j0 + chunk);
  uint32_t held[kHeld];
  uint32_t s = 0;
#pragma unroll
  for (int q = 0; q < kHeld; ++q) {
    held[q] = j0 + q < j1 ? hist[(size_t)(j0 + q) * kRadix + d] : 0u;
    s += held[q];
  }
  for (int j = j0 + kHeld; j < j1; ++j) s += hist[(size_t)j * kRadix + d];
  uint32_t incl = s;                      // inclusive scan over c within the wave
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane >= 56) wtot[wave][dl] = incl;
  __syncthreads();
  uint32_t run = incl - s, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t x = wtot[w][dl];
    run += w < wave ? x : 0u;
    total += x;
  }
  if (c == 0) bintot[d] = total;
#pragma unroll
  for (int q = 0; q < kHeld; ++q)
    if (j0 + q < j1) {
      binoff[(size_t)(j0 + q) * kRadix + d] = run;
      run += held[q];
    }
  for (int j = j0 + kHeld; j < j1; ++j) {
    const uint32_t v = hist[(size_t)j * kRadix + d];
    binoff[(size_t)j * kRadix + d] = run;
    run += v;
  }
}

// The same for narrow digits: one workgroup per digit walks its row of the table,
// four blocks per thread at a time.
template <int BITS>
__global__ void __launch_bounds__(256)
radix_rowscan(const uint32_t* __restrict__ hist, int nb, const int64_t* cnt_ptr, int64_t fixed,
              int64_t cap, int block_items, uint32_t* __restrict__ binoff,
              uint32_t* __restrict__ bintot) {
  __shared__ uint32_t wtot[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t count = live_count(cnt_ptr, fixed, cap);
  const int nbl = (int)min((int64_t)nb, (count + block_items - 1) / block_items);
  const uint32_t* in = hist + (size_t)blockIdx.x * nb;
  uint32_t* out = binoff + (size_t)blockIdx.x * nb;
  uint32_t carry = 0u;
  for (int j0 = 0, r = 0; j0 < nbl; j0 += 1024, r ^= 1) {
    const int j = j0 + 4 * threadIdx.x;
    uint32_t v[4], s = 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = j + q < nbl ? in[j + q] : 0u;
      s += v[q];
    }
    const uint32_t incl = rga::wave_scan(s);
    if (lane == 63) wtot[r][wave] = incl;
    __syncthreads();
    uint32_t run = carry + incl - s;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      run += w < wave ? wtot[r][w] : 0u;
      carry += wtot[r][w];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (j + q < nbl) out[j + q] = run;
      run += v[q];
    }
  }
  if (threadIdx.x == 0) bintot[blockIdx.x] = carry;
}

// Stable scatter of one block.  Each wave owns a contiguous run of
// 64 ITEMS items (so the block's order is wave by wave, round by round, lane
// by lane) and keeps them in registers.  Pass 1: per round, items with the
// same digit are matched with one ballot per digit bit (rank = number of
// lower lanes with that digit, group = their number) and each group's
// lowest lane adds the group to the wave's own digit counts in LDS.  Then,
// after one barrier, digit d of wave w starts at
//   (sum of bintot over digits < d) + binoff[block][d] + (counts of d in
//   waves < w),
// written over the wave's counts; after a second barrier each wave scatters
// its rounds with no further barrier: position = running start of the digit
// + rank, and the group's lowest lane advances the running start (the
// wave's LDS operations complete in order).  Narrow digits (16 items of 2048 and
// more each) are first put in order in LDS, so that a wave stores runs of a
// digit side by side: stored one by one, each item was a write of its own at the
// L2 (3.4 million entries, two passes of 7 bits: 51 -> 35 us).
template <int ITEMS, int BITS, bool LIVE = false>
__global__ void __launch_bounds__(kRadixThreads)
radix_downsweep(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                const int64_t* cnt_ptr, int64_t fixed, int64_t cap, int shift,
                const uint32_t* __restrict__ binoff, const uint32_t* __restrict__ bintot,
                int32_t* __restrict__ ranges, int nranges, Parts P, uint32_t* __restrict__ items,
                int64_t* __restrict__ live, int nb) {
  constexpr int kRadix = 1 << BITS;
  constexpr int kWavesR = kRadixThreads / 64;
  // digits per thread in the digit scan (the threads past the digits have none)
  constexpr int kPer = (kRadix + kRadixThreads - 1) / kRadixThreads;
  constexpr bool kNarrow = BITS <= 8;
  __shared__ uint32_t run[kWavesR][kRadix];
  __shared__ uint32_t wtot[kWavesR], ltot[kWavesR], deep_next[2];
  __shared__ uint32_t shift_to[kNarrow ? kRadix : 1];
  __shared__ uint2 sorted[kNarrow ? kRadixThreads * ITEMS : 1];
  uint32_t mine = 0u;   // items of this thread's digit in the block
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t count = live_count(cnt_ptr, fixed, cap);
  const int block = blockIdx.x;
  const int64_t blk = (int64_t)block * (kRadixThreads * ITEMS);
  // block 0 of a one-pass tile sort writes the ranges even when there are no
  // entries
  if (blk >= count && !(ranges && block == 0)) return;
  uint32_t* wrun = run[wave];
  for (int d = lane; d < kRadix; d += 64) wrun[d] = 0u;
  if (tid < 2) deep_next[tid] = 0u;
  const uint32_t part = part_length(count);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t wbeg = blk + (int64_t)wave * 64 * ITEMS;
  uint32_t key[ITEMS], val[ITEMS], info[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = wbeg + 64 * r + lane;
    const bool ok = i < count;
    key[r] = ok ? kin[i] : 0u;
    val[r] = ok ? vin[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool ok = wbeg + 64 * r + lane < count && (!LIVE || key[r] != kCulled);
    const uint32_t d = (key[r] >> shift) & (kRadix - 1);
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t rank = __popcll(peers & lt);
    const uint32_t group = __popcll(peers);
    if (ok && rank == 0) wrun[d] += group;
    // rank (6 bits), group size (7 bits); all ones = no item
    info[r] = ok ? (rank | (group << 6)) : 0xFFFFFFFFu;
  }
  // digit starts: each thread sums kPer consecutive digit totals, a wave
  // scan, then the waves' totals
  uint32_t tot[kPer];
  uint32_t s = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    tot[q] = tid * kPer + q < kRadix ? bintot[tid * kPer + q] : 0u;
    s += tot[q];
  }
  uint32_t incl = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  uint32_t start = incl - s;
  for (int w = 0; w < wave; ++w) start += wtot[w];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int d = tid * kPer + q;
    if (d >= kRadix) break;
    // a one-pass tile sort: digit d is tile d, and its entries land at
    // [start of the digit, + its total)
    if (ranges && block == 0 && d < nranges) {
      ranges[2 * d] = (int32_t)start;
      ranges[2 * d + 1] = (int32_t)(start + tot[q]);
      if (P.slots && is_deep((int)tot[q], part)) {
        deep_list(P, deep_next, d, (int)tot[q], part);
        atomicAdd(items, (uint32_t)(list_parts((int)tot[q], part) - 1));
      }
    }
    uint32_t acc = start + binoff[table_at<BITS>(block, d, nb)];
    if constexpr (kNarrow) {
      shift_to[d] = acc;
      for (int w = 0; w < kWavesR; ++w) mine += run[w][d];
    } else {
#pragma unroll
      for (int w = 0; w < kWavesR; ++w) {
        const uint32_t h = run[w][d];
        run[w][d] = acc;
        acc += h;
      }
    }
    start += tot[q];
  }
  if (LIVE && block == 0 && tid == kRadixThreads - 1) *live = (int64_t)start;
  if constexpr (kNarrow) {
    // the digits' places in the block, and how far each is from its place in
    // the output
    const uint32_t li = rga::wave_scan(mine);
    if (lane == 63) ltot[wave] = li;
    __syncthreads();
    uint32_t at = li - mine, items = 0u;
#pragma unroll
    for (int w = 0; w < kWavesR; ++w) {
      at += w < wave ? ltot[w] : 0u;
      items += ltot[w];
    }
    if (tid < kRadix) {
      shift_to[tid] -= at;
#pragma unroll
      for (int w = 0; w < kWavesR; ++w) {
        const uint32_t h = run[w][tid];
        run[w][tid] = at;
        at += h;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      if (info[r] != 0xFFFFFFFFu) {
        const uint32_t d = (key[r] >> shift) & (kRadix - 1);
        const uint32_t rank = info[r] & 63u, group = info[r] >> 6;
        const uint32_t pos = wrun[d] + rank;
        sorted[pos] = make_uint2(key[r], val[r]);
        if (rank == 0) wrun[d] += group;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t i = (uint32_t)(r * kRadixThreads + tid);
      if (i < items) {
        const uint2 e = sorted[i];
        const uint32_t pos = i + shift_to[(e.x >> shift) & (kRadix - 1)];
        kout[pos] = e.x;
        vout[pos] = e.y;
      }
    }
    return;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    if (info[r] != 0xFFFFFFFFu) {
      const uint32_t d = (key[r] >> shift) & (kRadix - 1);
      const uint32_t rank = info[r] & 63u, group = info[r] >> 6;
      const uint32_t pos = wrun[d] + rank;
      kout[pos] = key[r];
      vout[pos] = val[r];
      if (rank == 0) wrun[d] += group;
    }
  }
}

// ---- depth sort of few splats -----------------------------------------------
// Every splat's place by counting the keys before its own, with the live count and
// the sums of tiles touched: n^2 / 64 comparisons of a scalar key with 64 lanes',
// but one launch with no pass waiting for another, where the radix passes are ten
// (forward and back on 256^2: 8,000 splats 102 -> 78 us, 16,384 113 -> 98 us, and an
// LSD sort in one workgroup's LDS took 75 us against 65 at 4,096).  A workgroup
// places 64 splats, its sixteen waves share the keys: up to one workgroup per CU,
// beyond which 20,000 take 118 -> 122 us.  (Equal keys keep their order: those before
// the splat count up to its own key, those after it below.)
constexpr int kRankSort = 64 * 256;

__global__ void __launch_bounds__(1024)
rank_sort_kernel(int n, const uint32_t* __restrict__ keys, const int32_t* __restrict__ touched,
                 uint32_t* __restrict__ order, uint32_t* __restrict__ bsum,
                 int64_t* __restrict__ live) {
  constexpr int kW = 16;
  __shared__ uint32_t counts[kW][64], bs[kRankSort / kBlockN], alive;
  const int lane = threadIdx.x & 63, b = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = 64 * b + lane, groups = (n + 63) / 64;
  if (threadIdx.x < kRankSort / kBlockN) bs[threadIdx.x] = 0u;
  if (threadIdx.x == 0) alive = 0u;
  const uint32_t own = i < n ? keys[i] : kCulled;
  uint32_t c = 0u;
  for (int q = wave; q < groups; q += kW) {
    const uint32_t* __restrict__ k = keys + 64 * q;
    if (q != b && 64 * q + 64 <= n) {
      const uint32_t limit = own + (q < b ? 1u : 0u);
#pragma unroll
      for (int j = 0; j < 64; ++j) c += k[j] < limit ? 1u : 0u;
    } else {
      const int m = min(64, n - 64 * q);
      for (int j = 0; j < m; ++j) c += k[j] < own + (64 * q + j < i ? 1u : 0u) ? 1u : 0u;
    }
  }
  counts[wave][lane] = c;
  __syncthreads();
  if (b == 0) {
    uint32_t a = 0u;
    for (int j = threadIdx.x; j - lane < n; j += 64 * kW)
      a += (uint32_t)__popcll(__ballot(j < n && keys[j] != kCulled));
    if (lane == 0) atomicAdd(&alive, a);
  }
  if (wave == 0 && own != kCulled) {
    uint32_t at = 0u;
#pragma unroll
    for (int w = 0; w < kW; ++w) at += counts[w][lane];
    order[at] = (uint32_t)i;
    atomicAdd(&bs[at / kBlockN], (uint32_t)touched[i]);
  }
  __syncthreads();
  if (threadIdx.x < kRankSort / kBlockN && bs[threadIdx.x] != 0u)
    atomicAdd(&bsum[threadIdx.x], bs[threadIdx.x]);
  if (b == 0 && threadIdx.x == 0) *live = alive;
}

// ---- entries: one per (splat, tile touched), in depth order -----------------
// Tiles touched by each block of kBlockN splats in depth order (those that touch
// any come first: *live of them).
__global__ void __launch_bounds__(kBlockN)
touched_sum_kernel(const int64_t* __restrict__ live, const uint32_t* __restrict__ order,
                   const int32_t* __restrict__ touched, uint32_t* __restrict__ bsum) {
  __shared__ uint32_t red[kBlockN / 64];
  const int64_t n = *live, i = (int64_t)blockIdx.x * kBlockN + threadIdx.x;
  if ((int64_t)blockIdx.x * kBlockN >= n) return;
  const uint32_t v = rga::wave_scan(i < n ? (uint32_t)touched[order[i]] : 0u);
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0u;
#pragma unroll
    for (int w = 0; w < kBlockN / 64; ++w) s += red[w];
    bsum[blockIdx.x] = s;
  }
}

// One thread per splat in depth order: the sums of the blocks before and a
// workgroup scan of tiles-touched (wave scans, then the waves' totals) give each
// splat its first entry; the last block knows D.  Then one thread per entry,
// kDupChunk entries at a time: a splat marks its first entry in LDS, a running
// maximum over the marks gives every entry its splat, and the entries leave in
// whole lines.  With one thread storing each splat's entries the 3.4 million of
// 300k splats took 49 us, now 17.
constexpr int kDupItems = 8;
constexpr int kDupChunk = kBlockN * kDupItems;

__global__ void __launch_bounds__(kBlockN)
duplicate_kernel(int n, int TX, int64_t cap, const int64_t* __restrict__ live,
                 const uint32_t* __restrict__ order, const int32_t* __restrict__ touched,
                 const int32_t* __restrict__ rect, const uint32_t* __restrict__ bsum,
                 uint32_t* __restrict__ tkeys, uint32_t* __restrict__ tvals,
                 int64_t* __restrict__ total) {
  constexpr int kW = kBlockN / 64;
  __shared__ uint32_t wt[kW];
  __shared__ uint64_t wb[kW];
  __shared__ int wm[kW];
  __shared__ __align__(16) uint16_t own[kDupChunk];   // 1 + the entry's splat in the block
  __shared__ uint32_t splat[kBlockN], begin[kBlockN], corner[kBlockN], width[kBlockN];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t nl = *live, i0 = (int64_t)blockIdx.x * kBlockN, i = i0 + tid;
  if (i0 >= nl) return;
  uint64_t before = 0ull;
  for (int j = tid; j < (int)blockIdx.x; j += kBlockN) before += bsum[j];
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) before += __shfl_xor(before, o, 64);
  uint32_t g = 0u, cnt = 0u;
  if (i < nl) {
    g = order[i];
    cnt = (uint32_t)touched[g];
  }
  const uint32_t incl = rga::wave_scan(cnt);
  if (lane == 63) wt[wave] = incl;
  if (lane == 0) wb[wave] = before;
  splat[tid] = g;
  if (cnt > 0u) {
    const int x0 = rect[g], y0 = rect[n + g];
    corner[tid] = (uint32_t)(y0 * TX + x0);
    width[tid] = (uint32_t)(rect[2 * n + g] - x0 + 1);
  }
  __syncthreads();
  uint64_t base = 0ull;
  uint32_t first = incl - cnt, sum = 0u;
#pragma unroll
  for (int v = 0; v < kW; ++v) {
    base += wb[v];
    first += v < wave ? wt[v] : 0u;
    sum += wt[v];
  }
  begin[tid] = first;
  if (tid == 0 && i0 + kBlockN >= nl) *total = (int64_t)(base + sum);
  for (uint32_t c0 = 0u; c0 < sum && (int64_t)(base + c0) < cap; c0 += kDupChunk) {
    uint4* mine = reinterpret_cast<uint4*>(own) + tid;   // kDupItems marks
    static_assert(kDupItems == 8, "eight marks of two bytes");
    *mine = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    // a splat's mark: at its first entry, or at the chunk's if it began before
    if (cnt > 0u && first < c0 + kDupChunk && first + cnt > c0)
      own[first > c0 ? first - c0 : 0u] = (uint16_t)(tid + 1);
    __syncthreads();
    const uint4 q = *mine;
    const uint32_t words[4] = {q.x, q.y, q.z, q.w};
    int m[kDupItems], top = 0;
#pragma unroll
    for (int u = 0; u < kDupItems; ++u) {
      top = max(top, (int)((words[u >> 1] >> (16 * (u & 1))) & 0xFFFFu));
      m[u] = top;
    }
    int run = top;                       // inclusive maximum over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(run, o, 64);
      if (lane >= o) run = max(run, t);
    }
    if (lane == 63) wm[wave] = run;
    int prev = __shfl_up(run, 1, 64);
    if (lane == 0) prev = 0;
    __syncthreads();
    for (int v = 0; v < wave; ++v) prev = max(prev, wm[v]);
#pragma unroll
    for (int u = 0; u < kDupItems; ++u) m[u] = max(m[u], prev);
    *mine = make_uint4((uint32_t)m[0] | (uint32_t)m[1] << 16, (uint32_t)m[2] | (uint32_t)m[3] << 16,
                       (uint32_t)m[4] | (uint32_t)m[5] << 16, (uint32_t)m[6] | (uint32_t)m[7] << 16);
    __syncthreads();
    const uint32_t left = min((uint32_t)kDupChunk, sum - c0);
#pragma unroll
    for (int u = 0; u < kDupItems; ++u) {
      const uint32_t e = (uint32_t)(u * kBlockN + tid);
      const int64_t off = (int64_t)(base + c0) + e;
      if (e >= left || off >= cap) continue;
      const int o = (int)own[e] - 1;
      const uint32_t k = c0 + e - begin[o], w = width[o];
      // k / w from an approximate reciprocal, put right (k is below 2^24)
      uint32_t y = (uint32_t)((float)k * __builtin_amdgcn_rcpf((float)w));
      y -= y * w > k ? 1u : 0u;
      y += k - y * w >= w ? 1u : 0u;
      tkeys[off] = corner[o] + y * (uint32_t)TX + (k - y * w);
      tvals[off] = splat[o];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256)
fill_u32(uint32_t* __restrict__ p, int64_t count, uint32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

__global__ void __launch_bounds__(256)
tile_ranges_kernel(const uint32_t* __restrict__ tkeys, const int64_t* cnt_ptr, int64_t cap,
                   int32_t* __restrict__ ranges, Parts P,
                   uint32_t* __restrict__ next) {
  const int64_t count = live_count(cnt_ptr, 0, cap);
  const uint32_t part = part_length(count);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t t = tkeys[i];
    if (i == 0 || tkeys[i - 1] != t) ranges[2 * t] = (int32_t)i;
    if (i == count - 1 || tkeys[i + 1] != t) {
      ranges[2 * t + 1] = (int32_t)(i + 1);
      if (P.slots && i + 1 >= 2 * (int64_t)part && tkeys[i + 1 - 2 * (int64_t)part] == t) {
        int64_t lo = 0, hi = i + 1 - 2 * (int64_t)part;   // the list's first entry: search
        while (lo < hi) {
          const int64_t m = (lo + hi) / 2;
          if (tkeys[m] < t) lo = m + 1; else hi = m;
        }
        deep_list(P, next, (int)t, (int)(i + 1 - lo), part);
      }
    }
  }
}

// ---- blend ------------------------------------------------------------------
// One workgroup of four waves per 8 x 8 pixel block of a tile walks the
// tile's list front to back, 256 entries a round: each wave stages 64 of them
// (lane = entry) and tests them against the block's four 4 x 4 sub-blocks;
// then each wave composites the entries that can reach its sub-block, four at
// a time: lane = (pixel, one of four consecutive entries), the transmittance
// before each entry by a product scan over the four lanes of a pixel.  The
// product T of every listed entry's 1 - alpha is monotone, so an entry
// contributes exactly if T after it is still >= 1e-4 (the stop rule), and
// the pixel has stopped once T is not.
// The workgroup ends with its list or when its 64 pixels have stopped.
//
// Bound by vector issue and, per block, by the chain of its rounds.  Stopping
// is what counts: of the (entry, 8 x 8 block) pairs that can meet, 35 % lie
// before the block's stop at 100k Gaussians / 512^2 and 16 % at 300k / 1080^2.
// (Compositing 256-entry chunks of every list side by side, then combining
// them per pixel and restarting the chunk with the stop, walked all of them:
// 85 us at 100k / 512^2 and 416 us at 300k / 1080^2, this 72 and 162 us.)
// Four entries per step shorten the chain of the longest walk (1,250 entries)
// fourfold, and the 4 x 4 sub-blocks waste fewer lanes on pixels an entry
// does not reach than 8 x 8 blocks do.  Two steps are taken together: all but
// one product of a step does not depend on the step before.
//
// What the adjoint needs is left per (sub-chunk of 64 entries, pixel): the
// (C, T) before it, T negative once the pixel has stopped; per (sub-chunk,
// block) the entries that can reach pixels not stopped before it; per block
// the number of sub-chunks that some pixel entered; per pixel T after the last
// entry that counted.
//
// A deep list (is_deep) is walked in parts side by side, each from T = 1, C = 0:
// the first by the block's own workgroup, the others by workgroups behind those of
// the blocks, so that they wait for slots, not the other way round.  The last of a
// block's workgroups to arrive (counted; none waits) finds every part's incoming
// (C, T) per pixel and the part in which the pixel stops, and walks that part's
// sub-chunk with the stop again from its true state.  The states of such a list
// are relative to their part.  A part leaves its pixels' T where the later parts of
// the block look for it before they start: pixels that the earlier parts finished
// so far have stopped for certain need no walk any more.  The join decides on its
// own; what it reads of a part that ended early lies past the stop.
// One walk takes 22 ns per entry where pixels do not stop, as at an avatar's rim.
// Blend and its adjoint, every list in one walk (or equal parts of all, chosen by
// their mean, at 128^2 and 200^2) -> deep ones in parts: 300k splats on 8 tiles of
// 1080^2, the longest list 101,728 entries, 2,257 and 1,604 -> 107 and 76 us; on 40
// tiles of 512^2, 25,667 entries, 434 and 185 -> 102 and 67; 30k on 39 tiles, 2,576
// entries, 56 and 36 -> 40 and 34; 100k on 128^2 139 and 80 -> 75 and 48; 200k on
// 200^2 111 and 75 -> 87 and 74; 100k on 372 tiles, 4,570 entries, 75 and 71 -> 72 and
// 74; 300k on 1,627 tiles, no deep list, 157 and 202 -> 162 and 202 (the join's
// registers leave six waves per SIMD instead of seven, and seven by a launch bound
// cost 100k on 372 tiles 6 us).
constexpr float kPastStop = -2.f;

// One front-to-back compositing step of the adjoint for the pixel centre (px, py),
// written with selects instead of divergent branches: an entry is skipped when its
// exponent is positive or its alpha is below 1/255, and the walk stops at the first
// entry that would take T below `last` (stop_after).  Returns the weight alpha * T
// (0 if the entry is skipped or the walk has stopped); `applied` tells whether the
// entry contributed.
__device__ inline float blend_step(const float4& a, const float4& c1, float px, float py, float last,
                                   float& T, bool& stopped, bool& applied, float& alpha, float& dx,
                                   float& dy, float& G, float& araw) {
  dx = a.x - px;
  dy = a.y - py;
  // power log2(e) = -(A dx^2 + 2 B dx dy + C dy^2) log2(e) / 2 from the
  // scaled conic; exp(power) = 2^(power log2 e)
  const float e2 = fmaf(a.z * dx, dx, fmaf(c1.x * dy, dy, (a.w * dx) * dy));
  G = __builtin_amdgcn_exp2f(e2);
  araw = c1.y * G;
  alpha = fminf(0.99f, araw);
  const bool use = !stopped && e2 <= 0.f && alpha >= 1.f / 255.f;
  const float Tn = T * (1.f - alpha);
  const bool stop = use && Tn < last;
  stopped = stopped || stop;
  applied = use && !stop;
  const float w = applied ? alpha * T : 0.f;
  T = applied ? Tn : T;
  return w;
}

// The forward multiplies T in another order than the adjoint, so within the rounding
// of 1e-4 the two could stop one entry apart.  The forward keeps its T after the last
// entry that counted; one more that is used takes it down by 1/255 at least, so the
// adjoint stops halfway between.
__device__ inline float stop_after(float T) { return T * (1.f - 0x1p-9f); }

// The 8 x 8 block (tile, index in the tile) of a blend workgroup, and the part of
// the tile's list it walks: the four blocks of a tile, which read the same
// records, follow each other on one XCD (workgroups with equal index mod 8), and
// neighbouring tiles go to different ones; the same of the items (a tile's further
// part).  Of an image around an avatar most workgroups find nothing and leave: what
// they work out before that counts (37,000 of them at 1080^2, the grid's layout taken
// apart in the kernel 30 instead of 26 us for the adjoint of 4,000 entries).
struct PixelBlock {
  int t, blk, ox, oy;     // tile (-1: none), block in the tile, first pixel
  int y;                  // part
  __device__ inline int id() const { return kBlocks * t + blk; }
};
__device__ inline PixelBlock pixel_block(int e, bool own, int TX, int tiles, const Parts& P,
                                         const int64_t* counters) {
  PixelBlock b;
  const int k = e >> 3;
  b.t = (k >> 2) * 8 + (e & 7);
  b.blk = k & 3;
  b.y = 0;
  if (!own) {
    const bool have = b.t < (int)((uint64_t)counters[1] >> 32);
    const uint32_t item = have ? P.items()[b.t] : 0u;
    b.t = have ? (int)(item >> kPartBits) : -1;
    b.y = (int)(item & ((1u << kPartBits) - 1u));
  } else if (b.t >= tiles) {
    b.t = -1;
  }
  b.ox = (b.t % TX) * kTile + 8 * (b.blk & 1);
  b.oy = (b.t / TX) * kTile + 8 * (b.blk >> 1);
  return b;
}
inline int64_t block_grid(int64_t tiles) { return (tiles + 7) / 8 * 8 * kBlocks; }

__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Whether a splat record can give alpha >= 1/255 at any pixel centre of
// the rectangle [x0, x1] x [y0, y1]: the base-2 exponent is a concave
// quadratic, so its largest value there is 0 when the mean is inside, else
// the best of the four edges, each maximised along its line in closed form
// (slopes in the record) and clamped to the edge.  The record's threshold
// is a lower bound with a margin, so the test never drops an entry that a
// pixel would use.
__device__ inline bool reaches(const float4& r0, const float4& r1, const float4& r2, float x0,
                               float x1, float y0, float y1) {
  const float A = r0.z, B = r0.w, C = r1.x;
  const float lx = x0 - r0.x, hx = x1 - r0.x, ly = y0 - r0.y, hy = y1 - r0.y;
  auto ex = [&](float dx, float dy) { return fmaf(A * dx, dx, fmaf(C * dy, dy, (B * dx) * dy)); };
  const float e0 = ex(lx, fminf(fmaxf(r2.y * lx, ly), hy));
  const float e1 = ex(hx, fminf(fmaxf(r2.y * hx, ly), hy));
  const float e2 = ex(fminf(fmaxf(r2.z * ly, lx), hx), ly);
  const float e3 = ex(fminf(fmaxf(r2.z * hy, lx), hx), hy);
  const bool inside = lx <= 0.f && hx >= 0.f && ly <= 0.f && hy >= 0.f;
  return inside || !(fmaxf(fmaxf(e0, e1), fmaxf(e2, e3)) < r2.w);
}

// Sub-chunks per part of a list of L entries walked in `parts` parts.
__device__ inline int part_subs(int L, int parts) {
  return ((L + kSub - 1) / kSub + parts - 1) / parts;
}

template <int CTRL>
__device__ inline float quad(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// sum over the four lanes of a pixel, in each of them
__device__ inline float quad_sum(float v) {
  v += quad<0xB1>(v);
  return v + quad<0x4E>(v);
}

// Of four entries in a pixel's lanes, front to back: the product of the factors up
// to this lane's, and before it (quad_perm [0, 0, 1, 2], then [0, 1, 0, 1]).
__device__ inline float quad_product(float m, int e, float& before) {
  const float m1 = m * quad<0x90>(m);
  m = e >= 1 ? m1 : m;
  const float m2 = m * quad<0x44>(m);
  m = e >= 2 ? m2 : m;
  const float ml = quad<0x90>(m);
  before = e >= 1 ? ml : 1.f;
  return m;
}

// What a block's workgroups leave for the one that arrives last goes past the L2 of
// their XCD, and is read past that of the reader's (device-scope accesses), and the
// arrivals are counted once it is there: a fence instead would write the L2 back
// for each of them (1,000 parts: 290 us).
template <typename T>
__device__ inline void put_shared(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline T get_shared(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void shared_is_out() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The parts of a block joined, by the workgroup that arrived last.  Each part's
// (C, T) becomes the (C, T) before it, with the code of T_in that only flips signs:
// T_in for a whole part, -T_in for the part where the pixel stops (its own walk
// stopped, or T_in T < 1e-4), kPastStop past it (the first wave, lane = pixel).
// Pixels that stop in the first part, walked from the true T = 1, and pixels that
// never stop are written at once; the others walk the sub-chunk of their part in
// which they stop -- T_in T >= 1e-4 before it, not after it -- from that state with
// the stop: each pixel its own, four lanes and entries at a time as in the blend.
// (A pixel that does not stop there because of rounding ends with the sub-chunk.)
__device__ inline void blend_join(int W, int H, const PixelBlock& B, int parts, int home, int per,
                                  int start, int slot0, int L, int n,
                                  const uint32_t* __restrict__ sorted, const float4* __restrict__ rec,
                                  const float* __restrict__ color, const float* state, const Parts& P,
                                  float* last, float* image, float* Tfinal, float4* before,
                                  int* stops) {
  const int lane = threadIdx.x & 63, e = lane & 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const size_t HW = (size_t)H * W;
  if (wave == 0) {
    const int px = B.ox + (lane & 7), py = B.oy + (lane >> 3);
    const bool inside = px < W && py < H;
    float4* p = P.state() + (size_t)home * 64 + lane;
    float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f, Tout = 1.f;
    bool active = inside, first = false;
    int stop_part = -1;
    float4 in = make_float4(0.f, 0.f, 0.f, 0.f);   // (C, T) before the part of the stop
    for (int y0 = 0; y0 < parts; y0 += 4) {
      float4 r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t* f = reinterpret_cast<const uint64_t*>(p + min(y0 + u, parts - 1) * kBlocks * 64);
        const uint64_t a = get_shared(f), b = get_shared(f + 1);
        r[u] = make_float4(__uint_as_float((uint32_t)a), __uint_as_float((uint32_t)(a >> 32)),
                           __uint_as_float((uint32_t)b), __uint_as_float((uint32_t)(b >> 32)));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int y = y0 + u;
        if (y >= parts) continue;
        const bool stop = active && (r[u].w < 0.f || T * r[u].w < 1e-4f);
        p[y * kBlocks * 64] = make_float4(C0, C1, C2, active ? (stop ? -T : T) : kPastStop);
        if (stop) {
          active = false;
          first = y == 0;
          stop_part = y > 0 ? y : -1;
          in = make_float4(C0, C1, C2, T);
        }
        if (active || (stop && y == 0)) {
          C0 = fmaf(T, r[u].x, C0);
          C1 = fmaf(T, r[u].y, C1);
          C2 = fmaf(T, r[u].z, C2);
          T = active ? T * r[u].w : T;
          Tout = active ? T : -r[u].w;
        }
      }
    }
    if (inside && (active || first)) {
      const size_t q = (size_t)py * W + px;
      image[q] = C0;
      image[HW + q] = C1;
      image[2 * HW + q] = C2;
      Tfinal[q] = Tout;
      last[B.id() * 64 + lane] = Tout;
    }
    before[lane] = in;
    stops[lane] = stop_part;
  }
  __syncthreads();
  const int bx = 4 * (wave & 1) + ((lane >> 2) & 3), by = 4 * (wave >> 1) + (lane >> 4);
  const float4 in = before[8 * by + bx];
  const int y = stops[8 * by + bx];
  if (y < 0) return;                       // (a pixel's four lanes)
  const float* const st = state + (size_t)slot0 * 1024 + 64 * B.blk + 8 * by + bx;
  // the last sub-chunk entered with T_in T >= 1e-4 (T falls along the part)
  int sub = per * y;
  for (int hi = sub + min((int)get_shared(P.live() + home + kBlocks * y), per); hi - sub > 1;) {
    const int m = (sub + hi) / 2;
    const bool above = in.w * get_shared(st + (size_t)m * 1024 + 768) >= 1e-4f;
    sub = above ? m : sub;
    hi = above ? hi : m;
  }
  const float* const sj = st + (size_t)sub * 1024;
  float T = in.w * get_shared(sj + 768), Tl = T;
  float C0 = 0.f, C1 = 0.f, C2 = 0.f;
  const float base = e < 3 ? fmaf(in.w, get_shared(sj + 256 * e), e == 0 ? in.x : (e == 1 ? in.y : in.z)) : 0.f;
  const float fpx = (float)(B.ox + bx) + 0.5f, fpy = (float)(B.oy + by) + 0.5f;
  const int e0 = sub * kSub + e;
  auto index = [&](int i) { return sorted[start + min(e0 + 4 * i, L - 1)]; };
  SplatRec R = load_rec(rec, color, n, index(0));
  uint32_t g1 = index(1), g2 = index(2);
#pragma unroll 1
  for (int i = 0; i < kSub / 4; ++i) {
    const SplatRec N = load_rec(rec, color, n, g1);
    g1 = g2;
    g2 = index(i + 3);
    const float dx = R.r0.x - fpx, dy = R.r0.y - fpy;
    const float e2 = fmaf(R.r0.z * dx, dx, fmaf(R.r1.x * dy, dy, (R.r0.w * dx) * dy));
    const float alpha = fminf(0.99f, R.r1.y * __builtin_amdgcn_exp2f(e2));
    const bool use = e2 <= 0.f && alpha >= 1.f / 255.f && e0 + 4 * i < L;
    float ml;
    const float m = quad_product(use ? 1.f - alpha : 1.f, e, ml);
    const float after = T * m, prior = T * ml;
    const bool on = use && after >= 1e-4f;
    const float w = on ? alpha * prior : 0.f;
    C0 = fmaf(R.r1.z, w, C0);
    C1 = fmaf(R.r1.w, w, C1);
    C2 = fmaf(R.r2.x, w, C2);
    Tl = on ? after : Tl;
    T = quad<0xFF>(after);
    R = N;
  }
  C0 = quad_sum(C0);
  C1 = quad_sum(C1);
  C2 = quad_sum(C2);
  Tl = fminf(Tl, quad<0xB1>(Tl));
  Tl = fminf(Tl, quad<0x4E>(Tl));
  const size_t q = (size_t)(B.oy + by) * W + B.ox + bx;
  (e == 3 ? Tfinal : image + e * HW)[q] = e == 3 ? Tl : base + (e == 0 ? C0 : (e == 1 ? C1 : C2));
  if (e == 3) last[B.id() * 64 + 8 * by + bx] = Tl;
}

__global__ void __launch_bounds__(256)
blend_kernel(int W, int H, int TX, int tiles, int n, const int32_t* __restrict__ ranges,
             const uint32_t* __restrict__ sorted, const float4* __restrict__ rec,
             const float* __restrict__ color, const int64_t* __restrict__ counters,
             int64_t capacity, float* __restrict__ state, uint64_t* __restrict__ mask,
             uint32_t* __restrict__ nlive, float* __restrict__ last, Parts P, int blocks,
             float* __restrict__ image, float* __restrict__ Tfinal) {
  constexpr int kRound = 4 * kSub;        // entries per round
  // the staged records of two rounds, each with an entry past them with
  // opacity 0 that fills up a step of four
  __shared__ float4 s0[2][kRound + 1], s1[2][kRound + 1];
  __shared__ float s2[2][kRound + 1];
  __shared__ uint64_t reach[2][4][4];     // [round][sub-block][sub-chunk]
  __shared__ uint64_t used[2][4][4];      // the same, of sub-blocks not stopped yet
  // a wave's entries, each sub-chunk's padded to eights; per eight the two of
  // lane e (the e-th of either four) follow each other
  __shared__ uint16_t lists[4][kRound];
  __shared__ int open[2][4];              // sub-chunks entered in the round, per wave; 0: stopped
  const bool own = (int)blockIdx.x < blocks;
  const PixelBlock B = pixel_block(blockIdx.x - (own ? 0 : blocks), own, TX, tiles, P, counters);
  if (B.t < 0) return;
  const int lane = threadIdx.x & 63, e = lane & 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this lane's pixel in the block, wave w having the sub-block (w & 1, w >> 1)
  const int bx = 4 * (wave & 1) + ((lane >> 2) & 3), by = 4 * (wave >> 1) + (lane >> 4);
  const int px = B.ox + bx, py = B.oy + by;
  const bool inside = px < W && py < H;
  // lane e < 3 of a pixel writes channel e, lane 3 the transmittance
  auto put_pixel = [&](float c0, float c1, float c2, float T) {
    const size_t p = (size_t)py * W + px, HW = (size_t)H * W;
    const float v = e == 0 ? c0 : (e == 1 ? c1 : (e == 2 ? c2 : T));
    if (inside) (e == 3 ? Tfinal : image + e * HW)[p] = v;
  };
  // more duplicates than the workspace holds: the lists were truncated, so
  // the frame is poisoned (NaN) rather than silently wrong
  if (counters[0] > capacity) {
    const float nan = __builtin_nanf("");
    if (B.y == 0) {
      put_pixel(nan, nan, nan, nan);
      if (threadIdx.x == 0) nlive[B.id()] = 0u;
    }
    return;
  }
  const int start = ranges[2 * B.t], L = ranges[2 * B.t + 1] - start;
  if (L <= 0) {                           // (most tiles of an image around an avatar)
    put_pixel(0.f, 0.f, 0.f, 1.f);
    if (threadIdx.x == 0) nlive[B.id()] = 0u;
    return;
  }
  const int slot0 = start / kSub + B.t;
  // this workgroup's entries; of a deep list its part, the place of the first
  // part's block and of its own
  int parts = 1, per = L, a0 = 0, a1 = L, home = 0, place = 0;
  const uint32_t part = part_length(counters[0]);
  if (is_deep(L, part)) {
    parts = list_parts(L, part);
    per = kSub * part_subs(L, parts);
    a0 = min(L, per * B.y);
    a1 = min(L, a0 + per);
    home = kBlocks * (int)P.base()[B.t] + B.blk;
    place = home + kBlocks * B.y;
  }
  const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
  if (threadIdx.x < 2) {
    s0[threadIdx.x][kRound] = make_float4(0.f, 0.f, 0.f, 0.f);
    s1[threadIdx.x][kRound] = make_float4(0.f, 0.f, 0.f, 0.f);
    s2[threadIdx.x][kRound] = 0.f;
  }
  float T = inside ? 1.f : 0.f;           // the pixel is live while T >= 1e-4
  // this lane's entries only: their colour, T after the last that counted
  float Tl = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
  int nl = 0;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  // this wave's entry of the round and of the next one, read ahead
  const int mine = a0 + kSub * wave + lane;
  SplatRec R = {};
  uint32_t gnext = 0u;
  if (mine < a1) R = load_rec(rec, color, n, sorted[start + mine]);
  if (mine + kRound < a1) gnext = sorted[start + mine + kRound];
  // the masks of a finished round (all waves are past it) for the adjoint
  auto finish = [&](int r, int c0) {
    if (threadIdx.x < 4 && (int)threadIdx.x < (a1 - c0 + kSub - 1) / kSub)
      mask[(size_t)(slot0 + c0 / kSub + threadIdx.x) * kBlocks + B.blk] =
          (used[r][0][threadIdx.x] | used[r][1][threadIdx.x]) |
          (used[r][2][threadIdx.x] | used[r][3][threadIdx.x]);
    int m = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) m = max(m, open[r][w] >> 1);
    if (m) nl = (c0 - a0) / kSub + m;
    return ((open[r][0] | open[r][1]) | (open[r][2] | open[r][3])) & 1;   // some wave goes on
  };
  // A further part first looks what the block's earlier ones (the first 32) have
  // left at this pixel, as far as they are finished: with less than the stop's T
  // before it the pixel needs no walk (a margin for the order of the product).
  bool walk = true;
  if (B.y > 0) {
    uint32_t seen[8];
    float before = 1.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      seen[u] = kNoPart;
      if (4 * u + e < B.y)
        seen[u] = get_shared(P.T() + (uint32_t)((home + kBlocks * (4 * u + e)) * 64 + 8 * by + bx));
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (seen[u] != kNoPart) before *= __uint_as_float(seen[u]);
    before *= quad<0xB1>(before);
    before *= quad<0x4E>(before);
    if (before < 0.9e-4f) T = 0.f;
    walk = __syncthreads_or(T >= 1e-4f);
  }
  int par = 0, c0 = walk ? a0 : a1 + 1;
  for (; c0 < a1; c0 += kRound, par ^= 1) {
    {
      const bool ok = c0 - a0 + mine < a1;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float x0 = (float)(B.ox + 4 * (w & 1)) + 0.5f, y0 = (float)(B.oy + 4 * (w >> 1)) + 0.5f;
        const uint64_t m = __ballot(ok && reaches(R.r0, R.r1, R.r2, x0, x0 + 3.f, y0, y0 + 3.f));
        if (lane == 0) reach[par][w][wave] = m;
      }
      if (ok) {
        s0[par][kSub * wave + lane] = R.r0;
        s1[par][kSub * wave + lane] = R.r1;
        s2[par][kSub * wave + lane] = R.r2.x;
      }
      if (c0 - a0 + kRound + mine < a1) R = load_rec(rec, color, n, gnext);
      if (c0 - a0 + 2 * kRound + mine < a1) gnext = sorted[start + c0 - a0 + 2 * kRound + mine];
    }
    __syncthreads();
    // every wave is done with the round before this one: its masks go out,
    // and if all its waves had stopped, so does the workgroup
    if (c0 > a0 && !finish(par ^ 1, c0 - kRound)) break;
    const int nq = min(4, (a1 - c0 + kSub - 1) / kSub);
    // this wave's entries as a list
    uint16_t* lst = lists[wave];
    int pairq[5];                         // first pair of steps of each sub-chunk
    pairq[0] = 0;
    auto place = [](int i) { return (i & ~7) | ((i & 3) << 1) | ((i >> 2) & 1); };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t m = reach[par][wave][q];
      const int cnt = __popcll(m), at = 8 * pairq[q];
      if ((m >> lane) & 1ull) lst[place(at + __popcll(m & below))] = (uint16_t)(q * kSub + lane);
      if (lane < ((8 - cnt) & 7)) lst[place(at + cnt + lane)] = (uint16_t)kRound;
      pairq[q + 1] = __builtin_amdgcn_readfirstlane(pairq[q] + (cnt + 7) / 8);
    }
    wave_fence();
    const uint32_t* pairs = reinterpret_cast<const uint32_t*>(lst) + e;
    auto take = [&](uint32_t k, float4 (&a)[2], float4 (&c1)[2], float (&c2)[2]) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t ku = u ? k >> 16 : k & 0xFFFFu;
        a[u] = s0[par][ku];
        c1[u] = s1[par][ku];
        c2[u] = s2[par][ku];
      }
    };
    int entered = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q >= nq) break;
      const bool live = __ballot(T >= 1e-4f) != 0ull;
      if (lane == 0) used[par][wave][q] = live ? reach[par][wave][q] : 0ull;
      {
        // the state before the sub-chunk
        const float c0s = quad_sum(C0), c1s = quad_sum(C1), c2s = quad_sum(C2);
        float* st = state + (size_t)(slot0 + c0 / kSub + q) * 1024 + 64 * B.blk + 8 * by + bx;
        const float v = e == 0 ? c0s : (e == 1 ? c1s : (e == 2 ? c2s : (T >= 1e-4f ? T : kPastStop)));
        if (parts > 1)
          put_shared(st + 256 * e, v);
        else
          st[256 * e] = v;
      }
      if (!live) continue;
      entered = q + 1;
      const int i1 = pairq[q + 1];
      if (pairq[q] == i1) continue;
      float4 a[2], c1[2];
      float c2[2];
      take(pairs[4 * pairq[q]], a, c1, c2);
      uint32_t kn = pairs[4 * min(pairq[q] + 1, i1 - 1)];
      for (int i = pairq[q]; i < i1; ++i) {
        // the next pair's entries are read while this one is composited
        float4 an[2], c1n[2];
        float c2n[2];
        take(kn, an, c1n, c2n);
        kn = pairs[4 * min(i + 2, i1 - 1)];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float dx = a[u].x - fpx, dy = a[u].y - fpy;
          const float e2 = fmaf(a[u].z * dx, dx, fmaf(c1[u].x * dy, dy, (a[u].w * dx) * dy));
          const float alpha = fminf(0.99f, c1[u].y * __builtin_amdgcn_exp2f(e2));
          const bool use = e2 <= 0.f && alpha >= 1.f / 255.f;
          float ml;
          const float m = quad_product(use ? 1.f - alpha : 1.f, e, ml);
          const float after = T * m, before = T * ml;
          const bool on = use && after >= 1e-4f;
          const float w = on ? alpha * before : 0.f;
          C0 = fmaf(c1[u].z, w, C0);
          C1 = fmaf(c1[u].w, w, C1);
          C2 = fmaf(c2[u], w, C2);
          Tl = on ? after : Tl;
          T = quad<0xFF>(after);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          a[u] = an[u];
          c1[u] = c1n[u];
          c2[u] = c2n[u];
        }
        if (__ballot(T >= 1e-4f) == 0ull) break;
      }
    }
    const int on = __ballot(T >= 1e-4f) != 0ull ? 1 : 0;
    if (lane == 0) open[par][wave] = 2 * entered + on;
  }
  if (walk && c0 >= a1 && a1 > a0) {      // the list ended: its last round's masks
    __syncthreads();
    finish(par ^ 1, c0 - kRound);
  }
  C0 = quad_sum(C0);
  C1 = quad_sum(C1);
  C2 = quad_sum(C2);
  Tl = fminf(Tl, quad<0xB1>(Tl));
  Tl = fminf(Tl, quad<0x4E>(Tl));
  if (B.y == 0 && threadIdx.x == 0) nlive[B.id()] = (uint32_t)nl;
  if (parts == 1) {
    put_pixel(C0, C1, C2, Tl);
    if (e == 3) last[B.id() * 64 + 8 * by + bx] = Tl;
    return;
  }
  if (e == 0) {
    const bool whole = T >= 1e-4f || !inside;
    const size_t q = (size_t)place * 64 + 8 * by + bx;
    uint64_t* const f = reinterpret_cast<uint64_t*>(P.state() + q);
    put_shared(f, (uint64_t)__float_as_uint(C1) << 32 | __float_as_uint(C0));
    put_shared(f + 1, (uint64_t)__float_as_uint(whole ? T : -Tl) << 32 | __float_as_uint(C2));
    put_shared(P.T() + q, __float_as_uint(whole ? T : 0.f));
  }
  if (threadIdx.x == 0) put_shared(P.live() + place, (uint32_t)nl);
  shared_is_out();
  __syncthreads();
  int* const turn = &open[0][0];
  uint32_t* const arrived = P.arrived() + home;   // from kNoPart on
  if (threadIdx.x == 0) *turn = (int)(atomicAdd(arrived, 1u) + 2u);
  __syncthreads();
  if (*turn != parts) return;
  if (threadIdx.x == 0) *arrived = kNoPart;   // for another blend of the same lists
  blend_join(W, H, B, parts, home, per / kSub, start, slot0, L, n, sorted, rec, color, state, P, last,
             image, Tfinal, &s0[0][0], reinterpret_cast<int*>(&s2[0][0]));
}

// Workgroups per block of the adjoint (a block's sub-chunks are dealt out to
// them four at a time), so that a long list does not keep one of them alone;
// with many blocks fewer do, since every further workgroup of a short list
// is started for nothing.
inline int splits(int64_t tiles) { return tiles >= 4096 ? 2 : 4; }
constexpr int kSplitsPart = 2;           // the same, per further part of a deep list

// ---- adjoint: blend ----------------------------------------------------------
// One workgroup per 8 x 8 pixel block again; its waves take the sub-chunks
// that the forward entered, wave by wave, each from the recorded state, and
// re-walk the entries that contributed front to back with the same decisions:
//   dL/dc_i     = alpha_i T_i g
//   dL/dalpha_i = T_i g.c_i - Q_i / (1 - alpha_i),  Q_i = g.(C - C_<=i)
// with C the forward colour, then alpha = o exp(power) (unless clamped).
// A wave takes eight entries at a time.  The exponent is quadratic in the
// offset (dx, dy), dx depends on the pixel's column and dy on its row, so
// only s = dL/dpower, s dy, s dy^2 and the three colour terms are summed
// over the pixels' rows (eight entries together, ending with entry l / 8 and
// column l % 8 in lane l); the terms in dx are formed per column and nine
// values are summed over the columns.  Each entry's nine sums go to its
// splat's line of the sums in one 32-byte atomic request and one single add
// (as nine planes they were 64 scattered lines per request).
//
// Bound by vector issue (about 500 slots per eight entries): 61 us at 100k /
// 512^2 and 202 us at 300k / 1080^2, where one item queue over the sub-chunks
// of whole lists, most of them past the stop, took 88 and 390 us.  No
// workgroup waits for another and the waves share nothing; the next
// sub-chunk's loads are issued before the current one is walked.
__global__ void __launch_bounds__(256)
blend_bwd_kernel(int W, int H, int TX, int tiles, int n, const int32_t* __restrict__ ranges,
                 const uint32_t* __restrict__ sorted, const float4* __restrict__ rec,
                 const float* __restrict__ color, const float* __restrict__ state,
                 const uint64_t* __restrict__ mask, const uint32_t* __restrict__ nlive,
                 const float* __restrict__ last, const int64_t* __restrict__ counters, int64_t capacity,
                 Parts P, int front,
                 const float* __restrict__ image, const float* __restrict__ dimage,
                 float* __restrict__ grad) {
  __shared__ float4 s0[4][kSub], s1[4][kSub];
  __shared__ float s2[4][kSub];
  __shared__ uint32_t sg[4][kSub];
  // the workgroups of the items before those of the blocks (the items, of long lists,
  // at the end would be a tail: 71 us instead of 61 at 100k / 512^2 of the avatar); of
  // a part's sub-chunks each takes every so many'th four
  const bool own = (int)blockIdx.x >= front;
  const int split = blockIdx.y;
  if (!own && split >= kSplitsPart) return;
  const PixelBlock B = pixel_block(blockIdx.x - (own ? front : 0), own, TX, tiles, P, counters);
  if (B.t < 0) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int myslot = lane >> 3, col = lane & 7;
  const int step = 4 * (own ? (int)gridDim.y : kSplitsPart);
  int first = wave + 4 * split, end = own ? (int)nlive[B.id()] : first + 1;
  if (first >= end || counters[0] > capacity) return;
  const int start = ranges[2 * B.t], L = ranges[2 * B.t + 1] - start;
  const int slot0 = start / kSub + B.t;
  const uint32_t part = part_length(counters[0]);
  float4 base = make_float4(0.f, 0.f, 0.f, 1.f);
  if (is_deep(L, part)) {
    const int parts = list_parts(L, part);
    const int place = kBlocks * ((int)P.base()[B.t] + B.y) + B.blk;
    const int per = part_subs(L, parts), m0 = per * B.y;
    first += m0;
    end = m0 + min((int)P.live()[place], per);
    base = P.state()[(size_t)place * 64 + lane];
  }
  end = min(end, (L + kSub - 1) / kSub);
  if (first >= end) return;
  const int px = B.ox + (lane & 7), py = B.oy + (lane >> 3);
  const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
  float Cf0 = 0.f, Cf1 = 0.f, Cf2 = 0.f, g0 = 0.f, g1 = 0.f, g2 = 0.f;
  if (px < W && py < H) {
    const size_t p = (size_t)py * W + px, HW = (size_t)H * W;
    Cf0 = image[p];
    Cf1 = image[HW + p];
    Cf2 = image[2 * HW + p];
    g0 = dimage[p];
    g1 = dimage[HW + p];
    g2 = dimage[2 * HW + p];
  }
  const float Tin = fabsf(base.w), stop = stop_after(last[B.id() * 64 + lane]);
  // a sub-chunk's loads (entry indices, then the masks, records and states)
  // are issued while the one before is walked
  auto index = [&](int sub) {
    const int e = sub * kSub + lane;
    return sub < end && e < L ? sorted[start + e] : 0u;
  };
  struct Item {
    uint64_t mm;
    uint32_t g;
    SplatRec R;
    float C0, C1, C2, T;
  };
  auto fetch = [&](int sub, uint32_t g) {
    Item I = {};
    if (sub < end) {
      I.mm = mask[(size_t)(slot0 + sub) * kBlocks + B.blk];
      I.g = g;
      I.R = load_rec(rec, color, n, g);
      const float* st = state + (size_t)(slot0 + sub) * 1024 + 64 * B.blk + lane;
      I.C0 = st[0];
      I.C1 = st[256];
      I.C2 = st[512];
      I.T = st[768];
    }
    return I;
  };
  Item I = fetch(first, index(first));
  uint32_t gnext = index(first + step);
  for (int sub = first; sub < end; sub += step) {
    uint64_t mm = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(I.mm >> 32)) << 32) |
                  (uint32_t)__builtin_amdgcn_readfirstlane((int)I.mm);
    s0[wave][lane] = I.R.r0;
    s1[wave][lane] = I.R.r1;
    s2[wave][lane] = I.R.r2.x;
    sg[wave][lane] = I.g;
    // the pixel's state before the sub-chunk (base: 0, 1 for a whole list)
    float T = Tin * I.T;
    bool done = !(T >= 1e-4f) || base.w < -1.f;
    float Q = 0.f;
    if (!done)
      Q = fmaf(g2, Cf2 - fmaf(Tin, I.C2, base.z),
               fmaf(g1, Cf1 - fmaf(Tin, I.C1, base.y), g0 * (Cf0 - fmaf(Tin, I.C0, base.x))));
    I = fetch(sub + step, gnext);
    gnext = index(sub + 2 * step);
    wave_fence();
    while (mm && __ballot(!done) != 0ull) {
      float v[8][6];
      int kv = 0;                             // entry of this lane's slot
      int ns = 0;                             // slots filled
#pragma unroll
      for (int s = 0; s < 8; ++s) {
#pragma unroll
        for (int q = 0; q < 6; ++q) v[s][q] = 0.f;
        if (mm) {
          const int k = (int)__builtin_ctzll(mm);
          mm &= mm - 1;
          const float4 a = s0[wave][k], c1 = s1[wave][k];
          const float gc = fmaf(g2, s2[wave][k], fmaf(g1, c1.w, g0 * c1.z));
          const float Tb = T;
          bool applied;
          float alpha, dx, dy, G, araw;
          const float w = blend_step(a, c1, fpx, fpy, stop, T, done, applied, alpha, dx, dy, G, araw);
          Q = fmaf(-gc, w, Q);
          const float dal = fmaf(gc, Tb, -(Q * __builtin_amdgcn_rcpf(1.f - alpha)));   // alpha <= 0.99
          const float dp = applied && araw <= 0.99f ? dal * alpha : 0.f;   // unless clamped
          v[s][0] = dp;
          v[s][1] = dp * dy;
          v[s][2] = dp * dy * dy;
          v[s][3] = w * g0;
          v[s][4] = w * g1;
          v[s][5] = w * g2;
          kv = myslot == s ? k : kv;
          ++ns;
        }
      }
      float c[6];
      rga::slot_row_sums8(v, c);
      // this lane's entry and column: the sums over the column's pixels
      const float4 a = s0[wave][kv], c1 = s1[wave][kv];
      const float dx = a.x - fpx, hb = 0.5f * a.w;
      float r[9];
      r[0] = kInvHalfLog2e * fmaf(hb, c[1], a.z * dx * c[0]);   // d/d mean x (the record's conic unscaled)
      r[1] = kInvHalfLog2e * fmaf(c1.x, c[1], hb * dx * c[0]);  // d/d mean y
      r[2] = -0.5f * dx * dx * c[0];                            // d/d conic A
      r[3] = -dx * c[1];                                        // d/d conic B
      r[4] = -0.5f * c[2];                                      // d/d conic C
      r[5] = c[0] / c1.y;                                       // d/d opacity
      r[6] = c[3];                                              // d/d colour
      r[7] = c[4];
      r[8] = c[5];
      rga::group_sums8(r);
      if (myslot < ns) {
        float* row = grad + (size_t)sg[wave][kv] * kGrad;
        float x = r[0];
#pragma unroll
        for (int q = 1; q < 8; ++q) x = col == q ? r[q] : x;
        atomicAdd(row + col, x);
        if (col == 0) atomicAdd(row + 8, r[8]);
      }
    }
    wave_fence();   // the next sub-chunk's records replace these
  }
}

// ---- adjoint: projection --------------------------------------------------
template <typename R>
struct Chain {
  // Inputs: forward quantities in precision R and upstream gradients.
  // Outputs: camera-space gradient gXYZ, dRq (3x3), ds (3).
  static __device__ void run(const CamDev& cam, const R* Tm, const R* Vm, R J00, R J11, R J02,
                             R J12, R X, R Y, R Z, R ca, R cb, R cc, R dca, R dcb, R dcc, R du,
                             R dv, R* gM /*3x3 out*/, R* gXYZ) {
    const R h = dcb * R(0.5);
    const R P00 = dca * ca + h * cb, P01 = dca * cb + h * cc;
    const R P10 = h * ca + dcc * cb, P11 = h * cb + dcc * cc;
    const R S00 = -(ca * P00 + cb * P10);
    const R S01 = -(ca * P01 + cb * P11);
    const R S11 = -(cb * P01 + cc * P11);
    R gT[6];
    for (int j = 0; j < 3; ++j) {
      gT[j] = R(2) * (S00 * Tm[j] + S01 * Tm[3 + j]);
      gT[3 + j] = R(2) * (S01 * Tm[j] + S11 * Tm[3 + j]);
    }
    R gJ00 = 0, gJ02 = 0, gJ11 = 0, gJ12 = 0;
    for (int j = 0; j < 3; ++j) {
      gJ00 += gT[j] * Vm[j];
      gJ02 += gT[j] * Vm[6 + j];
      gJ11 += gT[3 + j] * Vm[3 + j];
      gJ12 += gT[3 + j] * Vm[6 + j];
    }
    R gV[9];
    for (int j = 0; j < 3; ++j) {
      gV[j] = J00 * gT[j];
      gV[3 + j] = J11 * gT[3 + j];
      gV[6 + j] = J02 * gT[j] + J12 * gT[3 + j];
    }
    const R fx = (R)cam.fx, fy = (R)cam.fy;
    const R iz = R(1) / Z, iz2 = iz * iz, iz3 = iz2 * iz;
    R gX = gJ02 * (-fx * iz2) + du * fx * iz;
    R gY = gJ12 * (-fy * iz2) + dv * fy * iz;
    R gZ = gJ00 * (-fx * iz2) + gJ02 * (R(2) * fx * X * iz3) + gJ11 * (-fy * iz2) +
           gJ12 * (R(2) * fy * Y * iz3) - du * fx * X * iz2 - dv * fy * Y * iz2;
    gXYZ[0] = gX;
    gXYZ[1] = gY;
    gXYZ[2] = gZ;
    // gM = Rc^T gV
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j)
        gM[3 * i + j] = (R)cam.R[i] * gV[j] + (R)cam.R[3 + i] * gV[3 + j] + (R)cam.R[6 + i] * gV[6 + j];
  }
};

__global__ void __launch_bounds__(256)
preprocess_bwd_kernel(int n, CamDev cam, const float* __restrict__ x, const float* __restrict__ A,
                      const float* __restrict__ quat, const float* __restrict__ log_s,
                      const float* __restrict__ opac, const uint8_t* __restrict__ front,
                      const int32_t* __restrict__ touched, float* __restrict__ grad,
                      float* __restrict__ dx, float* __restrict__ dquat,
                      float* __restrict__ dlog_s, float* __restrict__ dopac,
                      float* __restrict__ dcolor, float* __restrict__ dA,
                      const int64_t* __restrict__ counters, int64_t capacity) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  // take the blend adjoint's sums and leave them zero for another backward
  // (a splat in no list has none)
  float gs[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (touched[g] > 0) {
    float4* row = reinterpret_cast<float4*>(grad + (size_t)g * kGrad);
    const float4 a = row[0], b = row[1], c = row[2];
    gs[0] = a.x; gs[1] = a.y; gs[2] = a.z; gs[3] = a.w;
    gs[4] = b.x; gs[5] = b.y; gs[6] = b.z; gs[7] = b.w;
    gs[8] = c.x;
#pragma unroll
    for (int q = 0; q < 3; ++q) row[q] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (counters[0] > capacity) {
    // the forward's lists were truncated: poison the gradients (NaN)
    const float nan = __builtin_nanf("");
    for (int k = 0; k < 3; ++k) dx[(size_t)k * n + g] = nan;
    for (int k = 0; k < 4; ++k) dquat[(size_t)k * n + g] = nan;
    for (int k = 0; k < 3; ++k) dlog_s[(size_t)k * n + g] = nan;
    for (int k = 0; k < 3; ++k) dcolor[(size_t)k * n + g] = nan;
    dopac[g] = nan;
    if (dA)
      for (int k = 0; k < 9; ++k) dA[(size_t)k * n + g] = nan;
    return;
  }
  dopac[g] = gs[5];
  for (int k = 0; k < 3; ++k) dcolor[(size_t)k * n + g] = gs[6 + k];
  Geo G;
  bool okq;
  geo_forward(cam, x, A, quat, log_s, n, g, G, okq);
  bool valid = (G.Z > 0.2f) && front[g] && (opac[g] >= 1.f / 255.f) && okq;
  float gM[9], gXYZ[3];
  if (valid) {
    const float du = gs[0], dv = gs[1], dca = gs[2], dcb = gs[3], dcc = gs[4];
    const float det = fmaf(G.a, G.c, -(G.b * G.b));
    if (det <= (G.a * G.c) * 0x1p-12f) {
      Geo64 D;
      geo_forward64(cam, G, D);
      if (D.det > 0.0) {
        const double ca = D.c / D.det, cb = -D.b / D.det, cc = D.a / D.det;
        double gM64[9], g64[3];
        Chain<double>::run(cam, D.T, D.V, D.J00, D.J11, D.J02, D.J12, (double)G.X, (double)G.Y,
                           (double)G.Z, ca, cb, cc, dca, dcb, dcc, du, dv, gM64, g64);
        for (int k = 0; k < 9; ++k) gM[k] = (float)gM64[k];
        for (int k = 0; k < 3; ++k) gXYZ[k] = (float)g64[k];
      } else {
        valid = false;
      }
    } else {
      const float ca = G.c / det, cb = -G.b / det, cc = G.a / det;
      Chain<float>::run(cam, G.T, G.V, G.J00, G.J11, G.J02, G.J12, G.X, G.Y, G.Z, ca, cb, cc, dca,
                        dcb, dcc, du, dv, gM, gXYZ);
    }
  }
  if (!valid) {
    for (int k = 0; k < 3; ++k) dx[(size_t)k * n + g] = 0.f;
    for (int k = 0; k < 4; ++k) dquat[(size_t)k * n + g] = 0.f;
    for (int k = 0; k < 3; ++k) dlog_s[(size_t)k * n + g] = 0.f;
    if (dA)
      for (int k = 0; k < 9; ++k) dA[(size_t)k * n + g] = 0.f;
    return;
  }
  // x' -> camera: dx' = Rc^T gXYZ
  for (int k = 0; k < 3; ++k)
    dx[(size_t)k * n + g] = cam.R[k] * gXYZ[0] + cam.R[3 + k] * gXYZ[1] + cam.R[6 + k] * gXYZ[2];
  // M = (A Rq) diag(s)
  float B[9];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      B[3 * i + j] = G.A[3 * i] * G.Rq[j] + G.A[3 * i + 1] * G.Rq[3 + j] + G.A[3 * i + 2] * G.Rq[6 + j];
  float gB[9];
  for (int j = 0; j < 3; ++j) {
    float gs = 0.f;
    for (int i = 0; i < 3; ++i) {
      gs += gM[3 * i + j] * B[3 * i + j];
      gB[3 * i + j] = gM[3 * i + j] * G.s[j];
    }
    dlog_s[(size_t)j * n + g] = gs * G.s[j];
  }
  // dA = gB Rq^T (the skinning's linear part, for the pose gradient)
  if (dA)
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < 3; ++k)
        dA[(size_t)(3 * i + k) * n + g] =
            gB[3 * i] * G.Rq[3 * k] + gB[3 * i + 1] * G.Rq[3 * k + 1] + gB[3 * i + 2] * G.Rq[3 * k + 2];
  // gRq = A^T gB
  float gR[9];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      gR[3 * i + j] = G.A[i] * gB[j] + G.A[3 + i] * gB[3 + j] + G.A[6 + i] * gB[6 + j];
  const float w = G.q[0], qx = G.q[1], qy = G.q[2], qz = G.q[3];
  float gw = 2.f * (-qz * gR[1] + qy * gR[2] + qz * gR[3] - qx * gR[5] - qy * gR[6] + qx * gR[7]);
  float gx = 2.f * (qy * gR[1] + qz * gR[2] + qy * gR[3] - 2.f * qx * gR[4] - w * gR[5] +
                    qz * gR[6] + w * gR[7] - 2.f * qx * gR[8]);
  float gy = 2.f * (-2.f * qy * gR[0] + qx * gR[1] + w * gR[2] + qx * gR[3] + qz * gR[5] -
                    w * gR[6] + qz * gR[7] - 2.f * qy * gR[8]);
  float gz = 2.f * (-2.f * qz * gR[0] - w * gR[1] + qx * gR[2] + w * gR[3] - 2.f * qz * gR[4] +
                    qy * gR[5] + qx * gR[6] + qy * gR[7]);
  const float dot = w * gw + qx * gx + qy * gy + qz * gz;
  dquat[g] = (gw - w * dot) * G.inv;
  dquat[(size_t)n + g] = (gx - qx * dot) * G.inv;
  dquat[(size_t)2 * n + g] = (gy - qy * dot) * G.inv;
  dquat[(size_t)3 * n + g] = (gz - qz * dot) * G.inv;
}

// ---- storage order of the Gaussians --------------------------------------------
// The Gaussians sorted by their nearest mesh vertex (vidx row 0), stably (ties
// keep their index order), with the binning's radix sort: keys = vertex,
// values = index, 11-bit digits, as many passes as the vertex count needs.
__global__ void __launch_bounds__(256)
vertex_keys_kernel(int n, const int32_t* __restrict__ vidx, int nv, uint32_t* __restrict__ keys,
                   uint32_t* __restrict__ vals) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g < n) {
    keys[g] = (uint32_t)rga::clampi(vidx[g], 0, nv - 1);
    vals[g] = (uint32_t)g;
  }
}

// dst[r][j] = src[r][order[j]] for rows of 4-byte elements
__global__ void __launch_bounds__(256)
gather_columns_kernel(int rows, int n, const uint32_t* __restrict__ src,
                      const int32_t* __restrict__ order, uint32_t* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)rows * n) return;
  const int64_t r = i / n, j = i - r * n;
  dst[i] = src[r * n + rga::clampi(order[j], 0, n - 1)];
}

struct VertexOrderLayout {
  size_t keys0, keys1, vals0, vals1, hist, binoff, bintot, total;
  int nb;
};

VertexOrderLayout vertex_order_layout(int n) {
  VertexOrderLayout L;
  L.nb = (int)rga::ceil_div(n > 0 ? n : 1, kBlockN);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += rga::align_up(bytes, 256);
    return o;
  };
  const size_t items = (size_t)(n > 0 ? n : 1) * sizeof(uint32_t);
  L.keys0 = take(items);
  L.keys1 = take(items);
  L.vals0 = take(items);
  L.vals1 = take(items);
  L.hist = take((size_t)L.nb * kRadix * sizeof(uint32_t));
  L.binoff = take((size_t)L.nb * kRadix * sizeof(uint32_t));
  L.bintot = take((size_t)kRadix * sizeof(uint32_t));
  L.total = off;
  return L;
}

Parts parts_of(void* ws, const Layout& L) { return Parts{at<char>(ws, L.part), L.slots}; }

int check_common(const char* fn, int n, const rga_camera* cam, const void* ws, size_t ws_bytes,
                 int64_t cap, Layout& L) {
  if (n < 0) return rga::fail(RGA_EINVAL, "%s: n < 0", fn);
  if (!cam) return rga::fail(RGA_EINVAL, "%s: null camera", fn);
  if (cam->width < 1 || cam->height < 1 || cam->width > 16384 || cam->height > 16384)
    return rga::fail(RGA_EINVAL, "%s: image size must be in 1..16384", fn);
  if (cap < 1 || cap > 0x7FFFFFFFll) return rga::fail(RGA_EINVAL, "%s: capacity must be in 1..2^31-1", fn);
  if (n > 0x7FFFFFFF / 16) return rga::fail(RGA_EUNSUPPORTED, "%s: n too large", fn);
  L = make_layout(n, cam->width, cam->height, cap);
  if (!ws) return rga::fail(RGA_EINVAL, "%s: null workspace", fn);
  if (!rga::aligned16(ws)) return rga::fail(RGA_EINVAL, "%s: workspace must be 16-byte aligned", fn);
  if (ws_bytes < L.total)
    return rga::fail(RGA_ECAPACITY, "%s: workspace %zu < %zu bytes", fn, ws_bytes, L.total);
  return RGA_OK;
}

}  // namespace

extern "C" int back_face(void* stream, int n, const float* x, const float* nrm,
                         const float* cam_pos, uint8_t* front) {
  if (n < 0) return rga::fail(RGA_EINVAL, "back_face: n < 0");
  if (n == 0) return RGA_OK;
  if (!x || !nrm || !cam_pos || !front) return rga::fail(RGA_EINVAL, "back_face: null pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  RGA_LAUNCH("back_face", back_face_kernel, dim3(rga::ceil_div(n, 256)), dim3(256), 0, s, n, x,
             nrm, cam_pos[0], cam_pos[1], cam_pos[2], front);
  RGA_CHECK_LAUNCH("back_face");
  return RGA_OK;
}

extern "C" size_t splat_workspace_size(int n, int width, int height, int64_t capacity) {
  if (n < 0 || width < 1 || height < 1 || capacity < 1) return 0;
  return make_layout(n, width, height, capacity).total;
}

extern "C" int splat_state(void* ws, int n, int width, int height, int64_t capacity,
                           rga_splat_state* st) {
  if (!ws || !st || n < 0 || width < 1 || height < 1 || capacity < 1)
    return rga::fail(RGA_EINVAL, "splat_state: bad argument");
  Layout L = make_layout(n, width, height, capacity);
  st->mean2d = at<float>(ws, L.mean2d);
  st->conic = at<float>(ws, L.conic);
  st->depth = at<float>(ws, L.depth);
  st->rect = at<int32_t>(ws, L.rect);
  st->touched = at<int32_t>(ws, L.touched);
  st->fp64 = at<uint8_t>(ws, L.fp64);
  // after the tile sort the entries sit in the buffer of the final pass
  st->sorted = at<int32_t>(ws, (L.tile_passes & 1) ? L.tv1 : L.tv0);
  st->ranges = at<int32_t>(ws, L.ranges);
  st->count = at<int64_t>(ws, L.count);
  st->tiles_x = L.tiles_x;
  st->tiles_y = L.tiles_y;
  return RGA_OK;
}

extern "C" int splat_read_count(void* stream, const void* ws, int n, int width, int height,
                                int64_t capacity, int64_t* D) {
  if (!ws || !D || n < 0 || width < 1 || height < 1 || capacity < 1)
    return rga::fail(RGA_EINVAL, "splat_read_count: bad argument");
  Layout L = make_layout(n, width, height, capacity);
  hipStream_t s = static_cast<hipStream_t>(stream);
  int64_t h = 0;
  if (hipMemcpyAsync(&h, at<int64_t>(const_cast<void*>(ws), L.count), sizeof(int64_t),
                     hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return rga::fail(RGA_EHIP, "splat_read_count: copy failed");
  *D = h;
  return RGA_OK;
}

// Projection, depth sort, duplication, tile sort, tile ranges: everything of
// the forward that the colours do not enter.
extern "C" int splat_bin(void* stream, int n, const rga_camera* cam, const float* x,
                         const float* A, const float* quat, const float* log_s,
                         const float* opac, const uint8_t* front, void* ws, size_t ws_bytes,
                         int64_t capacity) {
  Layout L;
  int rc = check_common("splat_bin", n, cam, ws, ws_bytes, capacity, L);
  if (rc) return rc;
  if (n > 0 && (!x || !A || !quat || !log_s || !opac || !front))
    return rga::fail(RGA_EINVAL, "splat_bin: null input");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const CamDev cd = to_dev(cam);
  const int64_t tiles = (int64_t)L.tiles_x * L.tiles_y;
  int64_t* cnt = at<int64_t>(ws, L.count);
  uint32_t* k0 = at<uint32_t>(ws, L.keys0);
  uint32_t* v0 = at<uint32_t>(ws, L.vals0);
  uint32_t* k1 = at<uint32_t>(ws, L.keys1);
  uint32_t* v1 = at<uint32_t>(ws, L.vals1);
  uint32_t* hist = at<uint32_t>(ws, L.hist);
  uint32_t* binoff = at<uint32_t>(ws, L.binoff);
  uint32_t* bintot = at<uint32_t>(ws, L.bintot);
  int32_t* ranges = at<int32_t>(ws, L.ranges);
  if (n == 0) {
    // ranges := empty; count := 0
    RGA_LAUNCH("splat_fill", fill_u32, dim3(rga::ceil_div(2 * tiles + 4, 256)), dim3(256), 0, s,
               reinterpret_cast<uint32_t*>(ranges), 2 * tiles, 0u);
    RGA_LAUNCH("splat_fill", fill_u32, dim3(1), dim3(256), 0, s, reinterpret_cast<uint32_t*>(cnt),
               (int64_t)8, 0u);
  } else {
    const bool small = n <= kRankSort;
    uint32_t* bsum = at<uint32_t>(ws, L.bsum);
    // the projection also clears the tile ranges, the counters and, for the sort
    // of few splats, the sums of tiles touched
    const int64_t pre_threads = std::max<int64_t>(std::max<int64_t>(n, 2 * tiles), 8);
    RGA_LAUNCH("splat_preprocess", preprocess_kernel, dim3(rga::ceil_div(pre_threads, 256)),
               dim3(256), 0, s, n, cd, L.tiles_x, L.tiles_y, x, A, quat, log_s, opac, front, at<float4>(ws, L.rec), at<float>(ws, L.mean2d), at<float>(ws, L.conic),
               at<float>(ws, L.depth), at<int32_t>(ws, L.rect), at<int32_t>(ws, L.touched),
               at<uint8_t>(ws, L.fp64), k0, v0, reinterpret_cast<uint32_t*>(ranges), 2 * tiles,
               reinterpret_cast<uint32_t*>(cnt), at<float4>(ws, L.grad), reinterpret_cast<uint4*>(parts_of(ws, L).T()),
               (int64_t)L.slots * kPartWords / 4, bsum, small ? L.nb_n : 0);
    // depth sort: 3 passes of 11 bits over n 32-bit keys (4 passes of 8
    // bits, with 8x smaller digit tables, take longer: the passes are
    // latency-bound launches).  The first leaves out the culled splats (half of
    // an avatar's face away), the rest of the binning has the others only.
    int64_t* live = cnt + 3;
    if (small)
      RGA_LAUNCH("rank_sort", rank_sort_kernel, dim3(rga::ceil_div(n, 64)), dim3(1024), 0, s, n, k0,
                 at<int32_t>(ws, L.touched), v0, bsum, live);
    // Twice the keys per block from kManySplats on, half the digit tables (forward
    // and back on 1080^2: 300k splats 540 -> 528 us, 240k 481 -> 477, 140k 377 either
    // way; 100k on 512^2, where the blocks fill the chip no more, 370 -> 376).
    const bool many = n >= kManySplats;
    const int block = many ? 2 * kBlockN : kBlockN, nb = (int)rga::ceil_div(n, block);
    for (int pass = 0; pass < kDepthPasses && !small; ++pass) {
      const int shift = kDepthBits * pass;
      const int64_t* count = pass > 0 ? live : nullptr;
      auto up = pass > 0 ? (many ? radix_upsweep<2 * kItemsN, kDepthBits>
                                 : radix_upsweep<kItemsN, kDepthBits>)
                         : (many ? radix_upsweep<2 * kItemsN, kDepthBits, true>
                                 : radix_upsweep<kItemsN, kDepthBits, true>);
      auto down = pass > 0 ? (many ? radix_downsweep<2 * kItemsN, kDepthBits>
                                   : radix_downsweep<kItemsN, kDepthBits>)
                           : (many ? radix_downsweep<2 * kItemsN, kDepthBits, true>
                                   : radix_downsweep<kItemsN, kDepthBits, true>);
      RGA_LAUNCH("radix_upsweep", up, dim3(nb), dim3(kRadixThreads), 0, s, k0, count, (int64_t)n,
                 (int64_t)n, shift, hist);
      RGA_LAUNCH("radix_binscan", radix_binscan<kDepthBits>, dim3((1 << kDepthBits) / 8), dim3(256), 0, s,
                 hist, nb, count, (int64_t)n, (int64_t)n, block, binoff, bintot);
      RGA_LAUNCH("radix_downsweep", down, dim3(nb), dim3(kRadixThreads), 0, s, k0, v0, k1, v1, count,
                 (int64_t)n, (int64_t)n, shift, binoff, bintot, (int32_t*)nullptr, 0, Parts{}, (uint32_t*)nullptr, live, nb);
      uint32_t* t = k0; k0 = k1; k1 = t;
      t = v0; v0 = v1; v1 = t;
    }
    // v0 now holds the live splats' indices in (depth, index) order
    if (!small)
      RGA_LAUNCH("touched_sum", touched_sum_kernel, dim3(L.nb_n), dim3(kBlockN), 0, s, live, v0,
               at<int32_t>(ws, L.touched), bsum);
    uint32_t* tk0 = at<uint32_t>(ws, L.tk0);
    uint32_t* tv0 = at<uint32_t>(ws, L.tv0);
    uint32_t* tk1 = at<uint32_t>(ws, L.tk1);
    uint32_t* tv1 = at<uint32_t>(ws, L.tv1);
    RGA_LAUNCH("splat_duplicate", duplicate_kernel, dim3(L.nb_n), dim3(kBlockN), 0, s, n,
               L.tiles_x, capacity, live, v0, at<int32_t>(ws, L.touched), at<int32_t>(ws, L.rect), bsum,
               tk0, tv0, cnt);
    // with one tile pass its scatter also writes the tile ranges
    const bool one = L.tile_passes == 1;
    for (int pass = 0; pass < L.tile_passes; ++pass) {
      const int shift = L.tile_bits * pass;
      auto up = L.tile_bits == 7 ? radix_upsweep<kItemsD, 7> : L.tile_bits == 8 ? radix_upsweep<kItemsD, 8>
                : (L.tile_bits == 10 ? radix_upsweep<kItemsD, 10>
                   : (L.tile_bits == 11 ? radix_upsweep<kItemsD, 11> : radix_upsweep<kItemsD, 12>));
      auto scan = L.tile_bits == 7 ? radix_rowscan<7> : L.tile_bits == 8 ? radix_rowscan<8>
                  : (L.tile_bits == 10 ? radix_binscan<10>
                     : (L.tile_bits == 11 ? radix_binscan<11> : radix_binscan<12>));
      auto down = L.tile_bits == 7 ? radix_downsweep<kItemsD, 7> : L.tile_bits == 8 ? radix_downsweep<kItemsD, 8>
                  : (L.tile_bits == 10 ? radix_downsweep<kItemsD, 10>
                     : (L.tile_bits == 11 ? radix_downsweep<kItemsD, 11> : radix_downsweep<kItemsD, 12>));
      RGA_LAUNCH("radix_upsweep", up, dim3(L.nb_cap), dim3(kRadixThreads), 0, s, tk0,
                 (const int64_t*)cnt, (int64_t)0, capacity, shift, hist);
      RGA_LAUNCH("radix_binscan", scan, dim3((1 << L.tile_bits) / (L.tile_bits <= 8 ? 1 : 8)), dim3(256), 0, s, hist, L.nb_cap,
                 (const int64_t*)cnt, (int64_t)0, capacity, kBlockD, binoff, bintot);
      RGA_LAUNCH("radix_downsweep", down, dim3(L.nb_cap), dim3(kRadixThreads), 0, s, tk0, tv0, tk1, tv1,
                 (const int64_t*)cnt, (int64_t)0, capacity, shift, binoff, bintot,
                 one ? ranges : (int32_t*)nullptr, one ? (int)tiles : 0, parts_of(ws, L),
                 reinterpret_cast<uint32_t*>(cnt) + 3, (int64_t*)nullptr, L.nb_cap);
      uint32_t* t = tk0; tk0 = tk1; tk1 = t;
      t = tv0; tv0 = tv1; tv1 = t;
    }
    if (!one)
      RGA_LAUNCH("tile_ranges", tile_ranges_kernel,
                 dim3(std::min<int64_t>(rga::ceil_div(capacity, 256), 2048)), dim3(256), 0, s, tk0,
                 (const int64_t*)cnt, capacity, ranges, parts_of(ws, L),
                 reinterpret_cast<uint32_t*>(cnt) + 2);
  }
  RGA_CHECK_LAUNCH("splat_bin");
  return RGA_OK;
}

// The compositing: the rest of the forward, on the lists splat_bin left in ws.
extern "C" int splat_blend(void* stream, int n, const rga_camera* cam, const float* color,
                           void* ws, size_t ws_bytes, int64_t capacity, float* image,
                           float* T_final) {
  Layout L;
  int rc = check_common("splat_blend", n, cam, ws, ws_bytes, capacity, L);
  if (rc) return rc;
  if (!image || !T_final) return rga::fail(RGA_EINVAL, "splat_blend: null output");
  if (n > 0 && !color) return rga::fail(RGA_EINVAL, "splat_blend: null input");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int W = cam->width, H = cam->height;
  const int64_t tiles = (int64_t)L.tiles_x * L.tiles_y;
  int64_t* cnt = at<int64_t>(ws, L.count);
  int32_t* ranges = at<int32_t>(ws, L.ranges);
  const uint32_t* sorted = at<uint32_t>(ws, (L.tile_passes & 1) ? L.tv1 : L.tv0);
  RGA_LAUNCH("blend", blend_kernel, dim3(block_grid(tiles) + block_grid(L.slots)), dim3(256), 0, s, W, H,
             L.tiles_x, (int)tiles, n, ranges, sorted, at<float4>(ws, L.rec), color, cnt, capacity,
             at<float>(ws, L.state), at<uint64_t>(ws, L.mask), at<uint32_t>(ws, L.nlive),
             at<float>(ws, L.last), parts_of(ws, L), (int)block_grid(tiles), image, T_final);
  RGA_CHECK_LAUNCH("splat_blend");
  return RGA_OK;
}

extern "C" int splat_forward(void* stream, int n, const rga_camera* cam, const float* x,
                             const float* A, const float* quat, const float* log_s,
                             const float* opac, const float* color, const uint8_t* front,
                             void* ws, size_t ws_bytes, int64_t capacity, float* image,
                             float* T_final) {
  Layout L;
  int rc = check_common("splat_forward", n, cam, ws, ws_bytes, capacity, L);
  if (rc) return rc;
  if (!image || !T_final) return rga::fail(RGA_EINVAL, "splat_forward: null output");
  if (n > 0 && (!x || !A || !quat || !log_s || !opac || !color || !front))
    return rga::fail(RGA_EINVAL, "splat_forward: null input");
  rc = splat_bin(stream, n, cam, x, A, quat, log_s, opac, front, ws, ws_bytes, capacity);
  if (rc) return rc;
  return splat_blend(stream, n, cam, color, ws, ws_bytes, capacity, image, T_final);
}

extern "C" int splat_backward(void* stream, int n, const rga_camera* cam, const float* x,
                              const float* A, const float* quat, const float* log_s,
                              const float* opac, const float* color, const uint8_t* front,
                              void* ws, size_t ws_bytes, int64_t capacity, const float* image,
                              const float* dimage, float* dx, float* dquat, float* dlog_s,
                              float* dopac, float* dcolor, float* dA) {
  Layout L;
  int rc = check_common("splat_backward", n, cam, ws, ws_bytes, capacity, L);
  if (rc) return rc;
  if (n == 0) return RGA_OK;
  if (!x || !A || !quat || !log_s || !opac || !color || !front || !image || !dimage || !dx ||
      !dquat || !dlog_s || !dopac || !dcolor)
    return rga::fail(RGA_EINVAL, "splat_backward: null pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const CamDev cd = to_dev(cam);
  // The per-splat sums were zeroed by splat_forward's projection, and the
  // projection adjoint zeroes them again after use.
  float* grad = at<float>(ws, L.grad);
  const int64_t tiles = (int64_t)L.tiles_x * L.tiles_y;
  const uint32_t* sorted = at<uint32_t>(ws, (L.tile_passes & 1) ? L.tv1 : L.tv0);
  RGA_LAUNCH("blend_bwd", blend_bwd_kernel,
             dim3(block_grid(L.slots) + block_grid(tiles), splits(tiles)), dim3(256), 0, s,
             cam->width, cam->height, L.tiles_x, (int)tiles, n, at<int32_t>(ws, L.ranges), sorted,
             at<float4>(ws, L.rec), color, at<float>(ws, L.state), at<uint64_t>(ws, L.mask),
             at<uint32_t>(ws, L.nlive), at<float>(ws, L.last), (const int64_t*)at<int64_t>(ws, L.count),
             capacity, parts_of(ws, L), (int)block_grid(L.slots), image, dimage, grad);
  RGA_LAUNCH("preprocess_bwd", preprocess_bwd_kernel, dim3(rga::ceil_div(n, 256)), dim3(256), 0, s,
             n, cd, x, A, quat, log_s, opac, front, at<int32_t>(ws, L.touched), grad, dx, dquat,
             dlog_s, dopac, dcolor, dA, (const int64_t*)at<int64_t>(ws, L.count), capacity);
  RGA_CHECK_LAUNCH("splat_backward");
  return RGA_OK;
}

extern "C" size_t vertex_order_workspace(int n) {
  if (n < 0) return 0;
  return vertex_order_layout(n).total;
}

extern "C" int vertex_order(void* stream, int n, const int32_t* vidx, int nv, int32_t* order,
                            void* ws, size_t ws_bytes) {
  if (n < 0 || nv < 1) return rga::fail(RGA_EINVAL, "vertex_order: n >= 0 and nv >= 1");
  if (n > 0x7FFFFFFF / 16) return rga::fail(RGA_EUNSUPPORTED, "vertex_order: n too large");
  if (n == 0) return RGA_OK;
  if (!vidx || !order || !ws) return rga::fail(RGA_EINVAL, "vertex_order: null pointer");
  if (!rga::aligned16(ws)) return rga::fail(RGA_EINVAL, "vertex_order: workspace must be 16-byte aligned");
  const VertexOrderLayout L = vertex_order_layout(n);
  if (ws_bytes < L.total)
    return rga::fail(RGA_ECAPACITY, "vertex_order: workspace %zu < %zu bytes", ws_bytes, L.total);
  hipStream_t s = static_cast<hipStream_t>(stream);
  uint32_t* k0 = at<uint32_t>(ws, L.keys0);
  uint32_t* k1 = at<uint32_t>(ws, L.keys1);
  uint32_t* v0 = at<uint32_t>(ws, L.vals0);
  uint32_t* v1 = at<uint32_t>(ws, L.vals1);
  uint32_t* hist = at<uint32_t>(ws, L.hist);
  uint32_t* binoff = at<uint32_t>(ws, L.binoff);
  uint32_t* bintot = at<uint32_t>(ws, L.bintot);
  int bits = 0;
  while (bits < 31 && ((uint32_t)(nv - 1) >> bits) != 0u) ++bits;
  const int passes = bits <= kDigitBits ? 1 : (bits <= 2 * kDigitBits ? 2 : 3);
  RGA_LAUNCH("vertex_keys", vertex_keys_kernel, dim3(rga::ceil_div(n, 256)), dim3(256), 0, s, n,
             vidx, nv, k0, v0);
  for (int pass = 0; pass < passes; ++pass) {
    const int shift = kDigitBits * pass;
    const bool last = pass == passes - 1;
    uint32_t* vout = last ? reinterpret_cast<uint32_t*>(order) : v1;
    RGA_LAUNCH("radix_upsweep", (radix_upsweep<kItemsN, kDigitBits>), dim3(L.nb), dim3(kRadixThreads), 0, s, k0,
               (const int64_t*)nullptr, (int64_t)n, (int64_t)n, shift, hist);
    RGA_LAUNCH("radix_binscan", radix_binscan<kDigitBits>, dim3(kRadix / 8), dim3(256), 0, s, hist, L.nb,
               (const int64_t*)nullptr, (int64_t)n, (int64_t)n, kBlockN, binoff, bintot);
    RGA_LAUNCH("radix_downsweep", (radix_downsweep<kItemsN, kDigitBits>), dim3(L.nb), dim3(kRadixThreads), 0, s,
               k0, v0, k1, vout, (const int64_t*)nullptr, (int64_t)n, (int64_t)n, shift, binoff,
               bintot, (int32_t*)nullptr, 0, Parts{}, (uint32_t*)nullptr, (int64_t*)nullptr, L.nb);
    uint32_t* t = k0; k0 = k1; k1 = t;
    t = v0; v0 = v1; v1 = t;
  }
  RGA_CHECK_LAUNCH("vertex_order");
  return RGA_OK;
}

extern "C" int gather_columns(void* stream, int rows, int n, const void* src, const int32_t* order,
                              void* dst) {
  if (rows < 0 || n < 0) return rga::fail(RGA_EINVAL, "gather_columns: rows >= 0 and n >= 0");
  if ((int64_t)rows * n == 0) return RGA_OK;
  if (!src || !order || !dst) return rga::fail(RGA_EINVAL, "gather_columns: null pointer");
  if (src == dst) return rga::fail(RGA_EINVAL, "gather_columns: src and dst must not overlap");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t total = (int64_t)rows * n;
  if (rga::ceil_div(total, 256) > 0x7FFFFFFF)
    return rga::fail(RGA_EUNSUPPORTED, "gather_columns: rows * n too large");
  RGA_LAUNCH("gather_columns", gather_columns_kernel, dim3(rga::ceil_div(total, 256)), dim3(256), 0,
             s, rows, n, static_cast<const uint32_t*>(src), order, static_cast<uint32_t*>(dst));
  RGA_CHECK_LAUNCH("gather_columns");
  return RGA_OK;
}
