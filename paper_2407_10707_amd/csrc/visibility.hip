// Per-vertex visibility from orthographic rasterization of the posed mesh
// (Sec. 3.2 of the paper), bit-exact.
//
//   frame      the mesh's bounding box (partial boxes of a few workgroups,
//              joined by every raster workgroup: min and max are exact) and
//              the range of vertices that each batch of triangles uses
//   raster     one workgroup per view: the res x res z-buffer of 64-bit keys
//              (float bits of depth << 32 | triangle id) lives in LDS
//              (128 KB at 128^2, within gfx950's 160 KB), filled with LDS
//              64-bit atomic-min; winning triangles mark their three
//              vertices in an LDS bitmask that is written out view-major
//   transpose  32x32 bit-matrix transposes by wave ballots -> vertex-major words
//              raw[v][w] whose bit b is view 32w + b
//   filter     bit-sliced: one 32-bit word carries 32 views, so the median
//              of kv neighbours is a bitwise majority vote computed with a
//              5-plane ripple counter (two passes), and the final pass
//              expands the counter planes into count bytes [nv][V]
#include <algorithm>
#include <mutex>

#include "common.h"

namespace {

constexpr int kMaxRes = 128;
constexpr int kRasterThreads = 1024;
constexpr int kWideWords = 1 << 18;
constexpr int kRing = 256;               // entries of a raster wave's ring
constexpr int kGroup = 2;                // steps tested together; 63 + 64 kGroup <= kRing
constexpr int kRingFaces = 4096;         // the fewest triangles that go through the rings

__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a value that is the same in all lanes, in a scalar register
__device__ inline float uni(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ inline void basis(const float* d, float* t, float* b) {
  const float sgn = copysignf(1.f, d[2]);
  const float a = -1.f / (sgn + d[2]);
  const float bb = (d[0] * d[1]) * a;
  t[0] = 1.f + ((sgn * d[0]) * d[0]) * a;
  t[1] = sgn * bb;
  t[2] = -(sgn * d[0]);
  b[0] = bb;
  b[1] = sgn + (d[1] * d[1]) * a;
  b[2] = -d[1];
}

__device__ inline int64_t edge(int64_t ax, int64_t ay, int64_t bx, int64_t by, int64_t sx,
                               int64_t sy) {
  return (bx - ax) * (sy - ay) - (by - ay) * (sx - ax);
}

__device__ inline bool owns(int64_t ax, int64_t ay, int64_t bx, int64_t by) {
  const int64_t dx = bx - ax, dy = by - ay;
  return dy > 0 || (dy == 0 && dx < 0);
}

__device__ inline int64_t fdiv(int64_t a, int64_t b) {
  int64_t q = a / b;
  if ((a % b != 0) && ((a < 0) != (b < 0))) --q;
  return q;
}

struct Proj {
  float c[3], rho, irho, t[3], b[3], d[3], scale;
};

// The vertices: the caller's [3][nv], or the frame kernel's copy of 16 bytes
// each, which a triangle reads by three loads instead of nine (the addresses of
// 64 triangles lie in up to 64 lines, one of which the CU's cache serves per
// cycle).
struct Verts {
  const float* v;
  const float4* v4;
  int nv;
};

template <bool V4>
__device__ inline void vertex(const Verts& m, int i, float (&q)[3]) {
  if constexpr (V4) {
    const float4 x = m.v4[i];
    q[0] = x.x;
    q[1] = x.y;
    q[2] = x.z;
  } else {
    q[0] = m.v[i];
    q[1] = m.v[m.nv + i];
    q[2] = m.v[2 * m.nv + i];
  }
}

__device__ inline void project(const Proj& P, const float (&x)[3], int32_t& U, int32_t& V,
                               float& z) {
  const float q0 = x[0] - P.c[0], q1 = x[1] - P.c[1], q2 = x[2] - P.c[2];
  const float pu = fmaf(P.t[2], q2, fmaf(P.t[1], q1, P.t[0] * q0));
  const float pv = fmaf(P.b[2], q2, fmaf(P.b[1], q1, P.b[0] * q0));
  const float pd = fmaf(P.d[2], q2, fmaf(P.d[1], q1, P.d[0] * q0));
  // u = (t.(x - c) (1/rho) + 1) res / 2
  const float u = (pu * P.irho + 1.f) * P.scale;
  const float w = (pv * P.irho + 1.f) * P.scale;
  U = (int32_t)rintf(u * 256.f);
  V = (int32_t)rintf(w * 256.f);
  z = P.rho - pd;
}

__device__ inline unsigned long long depth_key(float bz, int f) {
  return ((unsigned long long)__float_as_uint(bz) << 32) | (unsigned long long)(uint32_t)f;
}

// General triangle (any extent): edge functions in 64-bit integers.
__device__ void raster_tri_wide(unsigned long long* zb, int res, int f, int64_t x0, int64_t y0,
                                float z0, int64_t x1, int64_t y1, float z1, int64_t x2,
                                int64_t y2, float z2) {
  int64_t area = edge(x0, y0, x1, y1, x2, y2);
  if (area == 0) return;
  if (area < 0) {
    int64_t tx = x1, ty = y1;
    x1 = x2; y1 = y2; x2 = tx; y2 = ty;
    float tz = z1; z1 = z2; z2 = tz;
    area = -area;
  }
  int64_t mnx = min(x0, min(x1, x2)), mxx = max(x0, max(x1, x2));
  int64_t mny = min(y0, min(y1, y2)), mxy = max(y0, max(y1, y2));
  int64_t i_lo = -fdiv(-(mnx - 128), 256), i_hi = fdiv(mxx - 128, 256);
  int64_t j_lo = -fdiv(-(mny - 128), 256), j_hi = fdiv(mxy - 128, 256);
  if (i_lo < 0) i_lo = 0;
  if (j_lo < 0) j_lo = 0;
  if (i_hi > res - 1) i_hi = res - 1;
  if (j_hi > res - 1) j_hi = res - 1;
  const bool o12 = owns(x1, y1, x2, y2), o20 = owns(x2, y2, x0, y0), o01 = owns(x0, y0, x1, y1);
  const float ia = 1.f / (float)area;   // barycentric weights w_e / area
  for (int64_t j = j_lo; j <= j_hi; ++j) {
    const int64_t sy = 256 * j + 128;
    for (int64_t i = i_lo; i <= i_hi; ++i) {
      const int64_t sx = 256 * i + 128;
      const int64_t w0 = edge(x1, y1, x2, y2, sx, sy);
      const int64_t w1 = edge(x2, y2, x0, y0, sx, sy);
      const int64_t w2 = edge(x0, y0, x1, y1, sx, sy);
      const bool in0 = w0 > 0 || (w0 == 0 && o12);
      const bool in1 = w1 > 0 || (w1 == 0 && o20);
      const bool in2 = w2 > 0 || (w2 == 0 && o01);
      if (!(in0 && in1 && in2)) continue;
      const float bz = fmaf((float)w2, z2, fmaf((float)w1, z1, (float)w0 * z0)) * ia;
      atomicMin(&zb[j * res + i], depth_key(bz, f));
    }
  }
}

// Triangle whose bounding box spans fewer than 2^14 fixed-point units on
// both axes (64 pixels): every coordinate difference inside the box (and
// one sample step past it) is below 2^14 + 256, so each edge-function
// product is below 2^29 and the edge functions are exact in 32-bit
// integers (and its factors fit the 24-bit multiplier, which takes a quarter of
// the 32-bit one's time).  They are stepped incrementally along rows and from
// row to row (exact integer updates), and the top-left rule becomes a
// sign test after subtracting 1 from the edges a sample on them does not
// belong to.  Same integers, same depth arithmetic as the wide form.
__device__ inline void raster_tri(unsigned long long* zb, int res, int f, int32_t x0, int32_t y0,
                                  float z0, int32_t x1, int32_t y1, float z1, int32_t x2,
                                  int32_t y2, float z2) {
  const int32_t mnx = min(x0, min(x1, x2)), mxx = max(x0, max(x1, x2));
  const int32_t mny = min(y0, min(y1, y2)), mxy = max(y0, max(y1, y2));
  if ((uint32_t)mxx - (uint32_t)mnx >= 16384u || (uint32_t)mxy - (uint32_t)mny >= 16384u) {
    raster_tri_wide(zb, res, f, x0, y0, z0, x1, y1, z1, x2, y2, z2);
    return;
  }
  int32_t area = __mul24(x1 - x0, y2 - y0) - __mul24(y1 - y0, x2 - x0);
  if (area == 0) return;
  if (area < 0) {
    int32_t tx = x1, ty = y1;
    x1 = x2; y1 = y2; x2 = tx; y2 = ty;
    float tz = z1; z1 = z2; z2 = tz;
    area = -area;
  }
  // sample columns i with mnx <= 256 i + 128 <= mxx (arithmetic shifts floor)
  const int i_lo = max(0, -((128 - mnx) >> 8)), i_hi = min(res - 1, (mxx - 128) >> 8);
  const int j_lo = max(0, -((128 - mny) >> 8)), j_hi = min(res - 1, (mxy - 128) >> 8);
  if (i_lo > i_hi || j_lo > j_hi) return;
  // w_e(s) = a_e (sx - x_e) + b_e (sy - y_e) for the edge opposite vertex e
  const int32_t a0 = y1 - y2, b0 = x2 - x1;
  const int32_t a1 = y2 - y0, b1 = x0 - x2;
  const int32_t a2 = y0 - y1, b2 = x1 - x0;
  // 0 if a sample on the edge belongs to the triangle, else 1
  // (edge A -> B owns its samples iff B.y > A.y, or B.y == A.y and B.x < A.x)
  const int32_t c0 = (a0 < 0 || (a0 == 0 && b0 < 0)) ? 0 : 1;   // edge v1 -> v2
  const int32_t c1 = (a1 < 0 || (a1 == 0 && b1 < 0)) ? 0 : 1;   // edge v2 -> v0
  const int32_t c2 = (a2 < 0 || (a2 == 0 && b2 < 0)) ? 0 : 1;   // edge v0 -> v1
  const float ia = 1.f / (float)area;   // barycentric weights w_e / area
  const int32_t sx = 256 * i_lo + 128, sy = 256 * j_lo + 128;
  int32_t r0 = __mul24(a0, sx - x1) + __mul24(b0, sy - y1) - c0;
  int32_t r1 = __mul24(a1, sx - x2) + __mul24(b1, sy - y2) - c1;
  int32_t r2 = __mul24(a2, sx - x0) + __mul24(b2, sy - y0) - c2;
  unsigned long long* row = zb + __mul24(j_lo, res);
  for (int j = j_lo; j <= j_hi; ++j) {
    int32_t w0 = r0, w1 = r1, w2 = r2;
    for (int i = i_lo; i <= i_hi; ++i) {
      if ((w0 | w1 | w2) >= 0) {
        const float bz = fmaf((float)(w2 + c2), z2, fmaf((float)(w1 + c1), z1,
                                                        (float)(w0 + c0) * z0)) * ia;
        atomicMin(&row[i], depth_key(bz, f));
      }
      w0 += 256 * a0;
      w1 += 256 * a1;
      w2 += 256 * a2;
    }
    r0 += 256 * b0;
    r1 += 256 * b1;
    r2 += 256 * b2;
    row += res;
  }
}

// min / max over the 64 lanes of a wave (DPP row shifts, then the two row
// broadcasts; a lane with no source keeps its own value), result in lane 63
template <int CTRL, int ROWS>
__device__ inline float dpp_same(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROWS, 0xf, false));
}

template <bool MAX>
__device__ inline float wave_extreme(float v) {
  auto op = [](float a, float b) { return MAX ? fmaxf(a, b) : fminf(a, b); };
  v = op(v, dpp_same<0x111, 0xf>(v));
  v = op(v, dpp_same<0x112, 0xf>(v));
  v = op(v, dpp_same<0x114, 0xf>(v));
  v = op(v, dpp_same<0x118, 0xf>(v));
  v = op(v, dpp_same<0x142, 0xa>(v));
  v = op(v, dpp_same<0x143, 0xc>(v));
  return v;
}

// Centre and radius of the frame of a bounding box (lo, hi).
__device__ inline void frame_from(const float (&r)[6], Proj& P) {
  float e[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    P.c[a] = (r[a] + r[3 + a]) * 0.5f;
    e[a] = r[3 + a] - r[a];
  }
  float rr = 1.01f * (0.5f * sqrtf(fmaf(e[2], e[2], fmaf(e[1], e[1], e[0] * e[0]))));
  if (!(rr > 0.f)) rr = 1.f;
  P.rho = rr;
}

// Workgroups [0, nbox): partial bounding boxes of the vertices (lo, hi per axis, six
// floats each; where there is one, the frame behind kBoxes of them) and, for the
// raster, a copy of 16 bytes per vertex (v4, if there is room).  The other workgroups
// write the triangles as the byte offsets of three entries of the raster's table: where
// that holds all vertices
// (nv <= cap) workgroup nbox + i 1024 of them, else workgroup nbox + b those
// of batch b, counted from the batch's lowest vertex, if its range of vertices
// fits.  (min and max are exact and independent of the reduction order.)  One
// workgroup over 39,780 vertices took 16 us.
constexpr int kBoxes = 16;
constexpr int kBatch = 16384;            // triangles per batch, a multiple of the raster's threads

__global__ void __launch_bounds__(1024)
frame_kernel(int nv, int nf, int nbox, const float* __restrict__ v, const int32_t* __restrict__ faces,
             int cap, float* __restrict__ boxes, int2* __restrict__ ranges,
             uint2* __restrict__ packed, float4* __restrict__ v4) {
  __shared__ float ext[6][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = (int)blockIdx.x - nbox;
  auto pack = [&](int f, int i0, int i1, int i2) {
    packed[f] = make_uint2((uint32_t)(2 * i0) | ((uint32_t)(2 * i1) << 16), (uint32_t)(2 * i2));
  };
  if (b >= 0 && nv <= cap) {
    const int f = b * 1024 + (int)threadIdx.x;
    if (f < nf)
      pack(f, rga::clampi(faces[3 * f], 0, nv - 1), rga::clampi(faces[3 * f + 1], 0, nv - 1),
           rga::clampi(faces[3 * f + 2], 0, nv - 1));
    return;
  }
  if (b >= 0) {
    __shared__ int lo16[16], hi16[16];
    int t[kBatch / 1024][3];
    int lo = nv - 1, hi = 0;
#pragma unroll
    for (int q = 0; q < kBatch / 1024; ++q) {
      const int f = min(b * kBatch + q * 1024 + (int)threadIdx.x, nf - 1);
#pragma unroll
      for (int c = 0; c < 3; ++c) t[q][c] = faces[3 * f + c];
    }
#pragma unroll
    for (int q = 0; q < kBatch / 1024; ++q) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        t[q][c] = rga::clampi(t[q][c], 0, nv - 1);
        lo = min(lo, t[q][c]);
        hi = max(hi, t[q][c]);
      }
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      lo = min(lo, __shfl_xor(lo, o, 64));
      hi = max(hi, __shfl_xor(hi, o, 64));
    }
    if (lane == 0) {
      lo16[wave] = lo;
      hi16[wave] = hi;
    }
    __syncthreads();
    for (int w = 0; w < 16; ++w) {
      lo = min(lo, lo16[w]);
      hi = max(hi, hi16[w]);
    }
    if (threadIdx.x == 0) ranges[b] = make_int2(lo, hi);
    if (hi - lo >= cap) return;
#pragma unroll
    for (int q = 0; q < kBatch / 1024; ++q) {
      const int f = b * kBatch + q * 1024 + (int)threadIdx.x;
      if (f < nf) pack(f, t[q][0] - lo, t[q][1] - lo, t[q][2] - lo);
    }
    return;
  }
  float lo3[3], hi3[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) lo3[a] = hi3[a] = v[a * nv];
  for (int i = blockIdx.x * 1024 + threadIdx.x; i < nv; i += nbox * 1024) {
    float c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      c[a] = v[a * nv + i];
      lo3[a] = fminf(lo3[a], c[a]);
      hi3[a] = fmaxf(hi3[a], c[a]);
    }
    if (v4) v4[i] = make_float4(c[0], c[1], c[2], 0.f);
  }
  float r[6];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    r[a] = wave_extreme<false>(lo3[a]);
    r[3 + a] = wave_extreme<true>(hi3[a]);
  }
  if (lane == 63) {
#pragma unroll
    for (int q = 0; q < 6; ++q) ext[q][wave] = r[q];
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    float x = ext[threadIdx.x][0];
    for (int w = 1; w < 16; ++w)
      x = threadIdx.x < 3 ? fminf(x, ext[threadIdx.x][w]) : fmaxf(x, ext[threadIdx.x][w]);
    boxes[6 * blockIdx.x + threadIdx.x] = x;
    if (nbox == 1) ext[threadIdx.x][0] = x;
  }
  if (nbox > 1 || wave > 0) return;
  wave_fence();
  if (threadIdx.x == 0) {
    float box[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) box[q] = ext[q][0];
    Proj P;
    frame_from(box, P);
    boxes[6 * kBoxes] = P.c[0];
    boxes[6 * kBoxes + 1] = P.c[1];
    boxes[6 * kBoxes + 2] = P.c[2];
    boxes[6 * kBoxes + 3] = P.rho;
  }
}

// The frame of the posed mesh from the partial boxes, joined by the lanes of
// every row of 16: centre of its bounding box and rho = 1.01 x half its
// diagonal.
__device__ inline void frame_of(const float* __restrict__ boxes, Proj& P) {
  static_assert(kBoxes == 16, "one box per lane of a row");
  float r[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const bool mx = q >= 3;
    auto op = [mx](float x, float y) { return mx ? fmaxf(x, y) : fminf(x, y); };
    float x = boxes[6 * (threadIdx.x & 15) + q];
    x = op(x, dpp_same<0x121, 0xf>(x));
    x = op(x, dpp_same<0x122, 0xf>(x));
    x = op(x, dpp_same<0x124, 0xf>(x));
    x = op(x, dpp_same<0x128, 0xf>(x));
    r[q] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
  }
  frame_from(r, P);
}

// A vertex's place between the sample centres 256 i + 128, for one axis: how many
// are below it and, in bit 7, whether it lies on one (for x in 0 .. 32640).
__device__ inline uint32_t place(int32_t x) {
  return (uint32_t)(x + 127) >> 8 | ((x & 255) == 128 ? 0x80u : 0u);
}

// A workgroup rasterizes views blockIdx.x, + gridDim.x, ...: one fits a CU at 128^2
// (its z-buffer takes 128 KB of the 160), and a new one for every view cost 6 of 116
// us at four views each; with ONE it has one view, in 64 registers, so that two fit a
// CU where the z-buffer leaves room for another.  Bound by vector issue, of which the
// rasterizer takes some 240 instructions per wave of triangles, and by its addresses.
//
// RING: many triangles of a mesh cover no sample (41 % at 13k triangles and
// 128^2, 96 % at 79k).  Each is tested first, by its bounding box alone: that
// holds a sample centre on an axis unless the places of the three vertices are
// equal there and on no centre.  Those that pass are gathered in an LDS ring per
// wave and rasterized by whole waves.  Where the range of a batch's vertices fits
// the LDS left beside the z-buffer (`cap`), their places, a byte per axis, are
// computed once into a table there (a mesh's triangles and vertices are numbered
// alike, so a batch uses a short range; each vertex is used by six triangles),
// else by each triangle.  A finite vertex lies inside the frame's sphere of
// 1 / 1.01 of rho, so its coordinates lie in 0 .. 255 res, and a NaN projects to
// 0; where that does not hold (rho from squares below the normal floats, view
// directions that are not unit vectors) there is no table.  1024 views at 128^2,
// in place -> 4-byte coordinates in the table, tested axis by axis -> this: 79k
// triangles 474 -> 365 -> 260 us; 512 views 241 -> 194 -> 139 us.
__host__ __device__ inline int ring_bytes() {
  return (int)sizeof(uint16_t) * kRing * (kRasterThreads / 64);
}
__host__ __device__ inline int table_bytes(int cap) { return (2 * cap + 15) / 16 * 16; }

template <bool RING, bool V4, bool ONE>
__global__ void __launch_bounds__(kRasterThreads, ONE ? 8 : 4)
raster_kernel(Verts verts, int nf, const int32_t* __restrict__ faces,
              int views, const float* __restrict__ dirs, int res, int nbox, const float* __restrict__ boxes,
              const int2* __restrict__ ranges, const uint2* __restrict__ packed, int cap,
              uint32_t* __restrict__ bits_vm /*[V][nwv]*/, int nwv, int shadow, float bias_px) {
  // the table first: its byte offsets are LDS addresses
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned long long* zb =
      reinterpret_cast<unsigned long long*>(smem + (RING ? table_bytes(cap) + ring_bytes() : 0));
  const int nv = verts.nv, pixels = res * res;
  uint32_t* mark = reinterpret_cast<uint32_t*>(zb + pixels);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Proj P;
  if (ONE && nbox == 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) P.c[a] = boxes[6 * kBoxes + a];
    P.rho = boxes[6 * kBoxes + 3];
  } else {
    frame_of(boxes, P);
  }
  P.irho = 1.f / P.rho;
  P.scale = 0.5f * (float)res;
  // (with ONE what all lanes share is in scalar registers; where a CU's only workgroup
  // takes four views in turn that costs 90 us instead of 87)
  auto uniform = [](float& v) {
    if constexpr (ONE) v = uni(v);
  };
#pragma unroll
  for (int a = 0; a < 3; ++a) uniform(P.c[a]);
  uniform(P.rho);
  uniform(P.irho);
  uniform(P.scale);
  auto corner = [&](int i, int32_t& U, int32_t& V, float& z) {
    float q[3];
    vertex<V4>(verts, i, q);
    project(P, q, U, V, z);
  };
  auto fill = [&](int lo, int hi) {
    for (int i = lo + threadIdx.x; i <= hi; i += kRasterThreads) {
      int32_t U, V;
      float z;
      corner(i, U, V, z);
      reinterpret_cast<uint16_t*>(smem)[i - lo] = (uint16_t)(place(U) | place(V) << 8);
    }
  };
  for (int w = threadIdx.x; w < nwv; w += kRasterThreads) mark[w] = 0u;
  for (int view = blockIdx.x; view < views; view += gridDim.x) {
    P.d[0] = dirs[3 * view];
    P.d[1] = dirs[3 * view + 1];
    P.d[2] = dirs[3 * view + 2];
    basis(P.d, P.t, P.b);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      uniform(P.t[a]);
      uniform(P.b[a]);
    }
    // (see above; a table's entries hold what the frame keeps its vertices to)
    const bool tables = RING && cap > 0 && P.irho < 1e17f &&
                        P.t[0] * P.t[0] + P.t[1] * P.t[1] + P.t[2] * P.t[2] < 1.001f &&
                        P.b[0] * P.b[0] + P.b[1] * P.b[1] + P.b[2] * P.b[2] < 1.001f;
    const bool whole = tables && nv <= cap;
    // (the next view's z-buffer is cleared as the marks are taken)
    if (ONE || view == (int)blockIdx.x || shadow)
      for (int p = threadIdx.x; p < pixels; p += kRasterThreads) zb[p] = ~0ull;
    if (whole) fill(0, nv - 1);
    __syncthreads();
    auto raster = [&](int f) {
      const int i0 = rga::clampi(faces[3 * f], 0, nv - 1);
      const int i1 = rga::clampi(faces[3 * f + 1], 0, nv - 1);
      const int i2 = rga::clampi(faces[3 * f + 2], 0, nv - 1);
      int32_t x0, y0, x1, y1, x2, y2;
      float z0, z1, z2;
      corner(i0, x0, y0, z0);
      corner(i1, x1, y1, z1);
      corner(i2, x2, y2, z2);
      raster_tri(zb, res, f, x0, y0, z0, x1, y1, z1, x2, y2, z2);
    };
    if constexpr (!RING) {
      for (int f = threadIdx.x; f < nf; f += kRasterThreads) raster(f);
    }
    uint16_t* ring = reinterpret_cast<uint16_t*>(smem + table_bytes(cap)) + kRing * wave;
    int head = 0, tail = 0;
    int base = 0;                           // first triangle the ring's entries count from
    for (int f0 = 0, b = 0; RING && f0 < nf; f0 += kBatch, ++b) {
      const int f1 = min(nf, f0 + kBatch);
      bool table = whole;
      if (tables && !whole) {
        const int2 r = ranges[b];
        table = r.y - r.x < cap;
        if (table) {
          if (b > 0) __syncthreads();       // the last batch's table is done with
          fill(r.x, r.y);
          __syncthreads();
        }
      }
      // the wave's triangles: lane's of fw, fw + kRasterThreads, ... below f1 (counts
      // are the same in all lanes: the ring's ends stay in scalar registers)
      const int fw = f0 + 64 * wave;
      constexpr int per = kGroup * kRasterThreads;
      const int groups = max(1, (f1 - fw + per - 1) / per);
      // the ring is emptied after the last batch and where its 16-bit entries end
      const bool drain = f1 == nf || f0 + kBatch - base >= 1024 * kRasterThreads;
      for (int g = 0; g < groups; ++g) {
        const int fg = fw + per * g;
        bool keep[kGroup];
        if (table) {
          uint2 t[kGroup];
  #pragma unroll
          for (int q = 0; q < kGroup; ++q)
            t[q] = *reinterpret_cast<const uint2*>(
                reinterpret_cast<const char*>(packed) +
                8u * (uint32_t)min(fg + lane + kRasterThreads * q, f1 - 1));
  #pragma unroll
          for (int q = 0; q < kGroup; ++q) {
            const uint32_t a = *reinterpret_cast<const uint16_t*>(smem + (t[q].x & 0xFFFFu));
            const uint32_t c = *reinterpret_cast<const uint16_t*>(smem + (t[q].x >> 16));
            const uint32_t d = *reinterpret_cast<const uint16_t*>(smem + t[q].y);
            const uint32_t w = (a ^ c) | (a ^ d) | (a & 0x8080u);
            keep[q] = (w & 0xFFu) != 0u && w > 0xFFu;
          }
        } else {
  #pragma unroll
          for (int q = 0; q < kGroup; ++q) {
            const int f = min(fg + lane + kRasterThreads * q, f1 - 1);
            int32_t x0, y0, x1, y1, x2, y2;
            float z;
            corner(rga::clampi(faces[3 * f], 0, nv - 1), x0, y0, z);
            corner(rga::clampi(faces[3 * f + 1], 0, nv - 1), x1, y1, z);
            corner(rga::clampi(faces[3 * f + 2], 0, nv - 1), x2, y2, z);
            const int32_t mnx = min(x0, min(x1, x2)), mxx = max(x0, max(x1, x2));
            const int32_t mny = min(y0, min(y1, y2)), mxy = max(y0, max(y1, y2));
            // (a coordinate may be the lowest integer: what lies left of the frame
            // lies left of its first sample)
            keep[q] = max(0, -((128 - max(mnx, 0)) >> 8)) <= min(res - 1, (mxx - 128) >> 8) &&
                      max(0, -((128 - max(mny, 0)) >> 8)) <= min(res - 1, (mxy - 128) >> 8);
          }
        }
  #pragma unroll
        for (int q = 0; q < kGroup; ++q) {
          const bool k = keep[q] && fg + lane + kRasterThreads * q < f1;
          const uint64_t m = __ballot(k);
          // entry = 64 x the wave's step + its lane there
          const int step = (fg - 64 * wave - base) / kRasterThreads + q;
          const uint32_t at = __builtin_amdgcn_mbcnt_hi(
              (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, tail));
          if (k) ring[at & (kRing - 1)] = (uint16_t)(step << 6 | lane);
          tail += __popcll(m);
        }
        const int need = drain && g == groups - 1 ? 1 : 64;
        while (tail - head >= need) {
          wave_fence();
          if (head + lane < tail) {
            const int en = ring[(head + lane) & (kRing - 1)];
            raster(base + 64 * wave + (en >> 6) * kRasterThreads + (en & 63));
          }
          head = min(head + 64, tail);
          wave_fence();
        }
      }
      if (drain) base = f0 + kBatch;
    }
    __syncthreads();
    if (shadow) {
      // shadow-mapping test: the vertex's depth against the depth map's
      // sample in the pixel it projects into, plus bias_px pixel widths; an
      // empty sample occludes nothing
      const float bias = bias_px * (2.f * P.rho) / (float)res;
      for (int i = threadIdx.x; i < nv; i += blockDim.x) {
        int32_t U, V;
        float z;
        corner(i, U, V, z);
        const int px = rga::clampi(U >> 8, 0, res - 1), py = rga::clampi(V >> 8, 0, res - 1);
        const unsigned long long k = zb[py * res + px];
        if (k == ~0ull || z <= __uint_as_float((uint32_t)(k >> 32)) + bias)
          atomicOr(&mark[i >> 5], 1u << (i & 31));
      }
    } else {
      for (int p = threadIdx.x; p < pixels; p += kRasterThreads) {
        const unsigned long long k = zb[p];
        if (k == ~0ull) continue;
        if (!ONE) zb[p] = ~0ull;
        const int f = (int)(uint32_t)(k & 0xffffffffull);
        for (int c = 0; c < 3; ++c) {
          const int vi = rga::clampi(faces[3 * f + c], 0, nv - 1);
          atomicOr(&mark[vi >> 5], 1u << (vi & 31));
        }
      }
    }
    __syncthreads();
    for (int w = threadIdx.x; w < nwv; w += kRasterThreads) {
      bits_vm[(size_t)view * nwv + w] = mark[w];
      if (!ONE) mark[w] = 0u;
    }
    if constexpr (ONE) return;   // (it has this view alone)
  }
}

// view-major [V][nwv] (bit i&31 of word i>>5 = vertex i) -> vertex-major
// [nv][nwV] (bit k&31 of word k>>5 = view k).  Each half-wave transposes one
// 32 x 32 bit block: lane r holds the row of view 32 kw + r, and the ballot
// of bit c over the half-wave is the column of vertex 32 vw + c, which
// lane c keeps and writes.
__global__ void __launch_bounds__(256)
transpose_kernel(int nv, int V, int nwv, int nwV, const uint32_t* __restrict__ vm,
                 uint32_t* __restrict__ out) {
  const int64_t blk = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 5;
  const int64_t total = (int64_t)nwv * nwV;
  const int lane = threadIdx.x & 63, r = lane & 31;
  const bool live = blk < total;            // both halves of a wave run the ballots
  const int vw = live ? (int)(blk / nwV) : 0;  // word of vertices
  const int kw = live ? (int)(blk % nwV) : 0;  // word of views
  const int k = 32 * kw + r;
  const uint32_t a = live && k < V ? vm[(size_t)k * nwv + vw] : 0u;
  uint32_t col = 0u;
#pragma unroll
  for (int c = 0; c < 32; ++c) {
    const uint64_t m = __ballot((a >> c) & 1u);
    const uint32_t half = lane < 32 ? (uint32_t)m : (uint32_t)(m >> 32);
    col = r == c ? half : col;
  }
  const int i = 32 * vw + r;
  if (live && i < nv) out[(size_t)i * nwV + kw] = col;
}

struct Planes {
  uint32_t p[5];
};

__device__ inline void add_word(Planes& s, uint32_t x) {
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const uint32_t c = s.p[k] & x;
    s.p[k] ^= x;
    x = c;
  }
}

// lanes whose 5-bit count >= thr
__device__ inline uint32_t at_least(const Planes& s, int thr) {
  uint32_t ge = 0u, eq = 0xFFFFFFFFu;
#pragma unroll
  for (int k = 4; k >= 0; --k) {
    if ((thr >> k) & 1) {
      eq &= s.p[k];
    } else {
      ge |= eq & s.p[k];
      eq &= ~s.p[k];
    }
  }
  return ge | eq;
}

// Bit planes of the number of neighbours (kv <= 31) whose word has each bit
// set, for VEC consecutive words.  All neighbour indices are read first and
// then all words, so the loads overlap instead of forming a chain of
// dependent round trips.
template <int VEC>
struct Words {
  uint32_t x[VEC];
};

template <int VEC>
__device__ inline void neighbour_planes(const int32_t* __restrict__ knn, int i, int kv, int nv,
                                        const uint32_t* __restrict__ src, int nwV, int w,
                                        Planes (&s)[VEC]) {
  const int32_t* row = knn + (size_t)i * kv;
  int idx[31];
#pragma unroll
  for (int j = 0; j < 31; ++j) idx[j] = j < kv ? rga::clampi(row[j], 0, nv - 1) : 0;
  Words<VEC> x[31];
#pragma unroll
  for (int j = 0; j < 31; ++j) {
    if (j >= kv) continue;
    const uint32_t* p = src + (size_t)idx[j] * nwV + w;
    if constexpr (VEC == 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(p);
      x[j] = {v.x, v.y, v.z, v.w};
    } else {
      x[j].x[0] = p[0];
    }
  }
#pragma unroll
  for (int u = 0; u < VEC; ++u) s[u] = {{0u, 0u, 0u, 0u, 0u}};
#pragma unroll
  for (int j = 0; j < 31; ++j)
    if (j < kv) {
#pragma unroll
      for (int u = 0; u < VEC; ++u) add_word(s[u], x[j].x[u]);
    }
}

// One thread per vertex and VEC words (VEC views' words in one load; words a
// multiple of VEC and 4 VEC-byte aligned rows).  With one word per thread the
// neighbour indices were read once per word.
template <int VEC>
__global__ void __launch_bounds__(256)
majority_kernel(int nv, int nwV, const int32_t* __restrict__ knn, int kv,
                const uint32_t* __restrict__ src, uint32_t* __restrict__ dst) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per = nwV / VEC;
  if (id >= (int64_t)nv * per) return;
  const int i = (int)(id / per), w = VEC * (int)(id % per);
  Planes s[VEC];
  neighbour_planes<VEC>(knn, i, kv, nv, src, nwV, w, s);
  uint32_t* out = dst + (size_t)i * nwV + w;
  const int thr = (kv + 1) / 2;
  if constexpr (VEC == 4)
    *reinterpret_cast<uint4*>(out) = make_uint4(at_least(s[0], thr), at_least(s[1], thr),
                                                at_least(s[2], thr), at_least(s[3], thr));
  else
    out[0] = at_least(s[0], thr);
}

template <int VEC>
__global__ void __launch_bounds__(256)
count_kernel(int nv, int V, int nwV, const int32_t* __restrict__ knn, int kv,
             const uint32_t* __restrict__ src, uint8_t* __restrict__ count) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per = nwV / VEC;
  if (id >= (int64_t)nv * per) return;
  const int i = (int)(id / per), w = VEC * (int)(id % per);
  Planes s[VEC];
  neighbour_planes<VEC>(knn, i, kv, nv, src, nwV, w, s);
  uint8_t* row = count + (size_t)i * V;
#pragma unroll
  for (int u = 0; u < VEC; ++u) {
    uint32_t words[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      // bits 4q .. 4q+3 of each plane to the lowest bit of four bytes: the
      // product puts bit j at positions j + 7 m, of which 8 j is kept
      uint32_t packed = 0u;
#pragma unroll
      for (int k = 0; k < 5; ++k)
        packed |= (__umul24((s[u].p[k] >> (4 * q)) & 0xFu, 0x204081u) & 0x01010101u) << k;
      words[q] = packed;
    }
    const int k0 = 32 * (w + u);
    if ((V & 15) == 0 && k0 + 32 <= V) {
      uint4* dst = reinterpret_cast<uint4*>(row + k0);
      dst[0] = make_uint4(words[0], words[1], words[2], words[3]);
      dst[1] = make_uint4(words[4], words[5], words[6], words[7]);
    } else {
      for (int b = 0; b < 32 && k0 + b < V; ++b) row[k0 + b] = (uint8_t)((words[b >> 2] >> (8 * (b & 3))) & 0xFFu);
    }
  }
}

struct VisLayout {
  size_t vm, raw, m1, m2, total;
  int nwv, nwV;
};

VisLayout vis_layout(int nv, int V) {
  VisLayout L{};
  L.nwv = (nv + 31) / 32;
  L.nwV = (V + 31) / 32;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t a = o;
    o = rga::align_up(o + bytes, 256);
    return a;
  };
  take(16);   // (kept: sizes a caller has computed stay enough)
  L.vm = take((size_t)V * L.nwv * 4);
  L.raw = take((size_t)nv * L.nwV * 4);
  L.m1 = take((size_t)nv * L.nwV * 4);
  L.m2 = take((size_t)nv * L.nwV * 4);
  L.total = o;
  return L;
}

}  // namespace

// (beyond the layout: room for the raster's copy of the vertices and for twice
// as many packed triangles, which it does without in a smaller workspace)
extern "C" size_t mesh_visibility_workspace(int nv, int V) {
  if (nv < 1 || V < 1) return 0;
  const VisLayout L = vis_layout(nv, V);
  return std::max(L.total, L.raw + 1024 + (size_t)33 * nv);
}

namespace {

int visibility_impl(void* stream, int nv, int nf, const float* verts, const int32_t* faces, int V,
                    const float* view_dirs, int res, const int32_t* knn, int kv,
                    uint32_t* raw_bits, uint8_t* count, void* ws, size_t ws_bytes, int shadow,
                    float bias_px) {
  if (nv < 1 || nf < 0 || V < 1) return rga::fail(RGA_EINVAL, "mesh_visibility: nv >= 1, nf >= 0, V >= 1");
  if (res < 1 || res > kMaxRes)
    return rga::fail(RGA_EUNSUPPORTED, "mesh_visibility: res must be in 1..%d", kMaxRes);
  if (kv < 1 || kv > 31 || (kv & 1) == 0)
    return rga::fail(RGA_EINVAL, "mesh_visibility: kv must be odd and in 1..31");
  if (!verts || (nf > 0 && !faces) || !view_dirs || !knn || !count || !ws)
    return rga::fail(RGA_EINVAL, "mesh_visibility: null pointer");
  if (!rga::aligned16(ws) || !rga::aligned16(count))
    return rga::fail(RGA_EINVAL, "mesh_visibility: ws and count must be 16-byte aligned");
  VisLayout L = vis_layout(nv, V);
  if (ws_bytes < L.total)
    return rga::fail(RGA_ECAPACITY, "mesh_visibility: workspace %zu < %zu bytes", ws_bytes, L.total);
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* w = static_cast<char*>(ws);
  uint32_t* vm = reinterpret_cast<uint32_t*>(w + L.vm);
  uint32_t* raw = raw_bits ? raw_bits : reinterpret_cast<uint32_t*>(w + L.raw);
  uint32_t* m1 = reinterpret_cast<uint32_t*>(w + L.m1);
  uint32_t* m2 = reinterpret_cast<uint32_t*>(w + L.m2);
  // z-buffer and marks; what is left of the LDS (beside the rings) holds
  // projected vertices
  const size_t zm = sizeof(unsigned long long) * (size_t)res * res + 4 * (size_t)L.nwv;
  if (zm > 160 * 1024)
    return rga::fail(RGA_EUNSUPPORTED, "mesh_visibility: %d vertices need too much LDS", nv);
  // A workgroup has one view where two workgroups' LDS fits a CU (up to 100^2 samples
  // in place, 94^2 through the rings, with half of the LDS for each one's table): one's
  // clearing, marking and tails run beside the other's triangles (1024 views, one per
  // CU -> two: in place 1k triangles at 96^2 62 -> 49 us, 3.6k 67 -> 58; through the
  // rings 13.6k at 64^2 93 -> 81, 79k 257 -> 213); and in place where there are no more
  // views than CUs (1k triangles at 128^2, 256 views 41.6 -> 40.2; through the rings
  // 27k at 64^2 51.0 -> 52.4).  Else a workgroup per CU takes the views in turn.
  // From one triangle per sample and 4,096 of them on, they go through the rings, if
  // the LDS has room for them; from two per sample on where that costs the second
  // workgroup (1024 views, in place -> rings: 79k at 128^2 526 -> 344 us, 13.6k at
  // 64^2 109 -> 81, 3.6k at 48^2 47 -> 50, 27k at 96^2 177 -> 157 but 13.6k 109 ->
  // 117; 256 views, 3.6k at 48^2 31 -> 32).
  const size_t rings = ring_bytes();
  const int cus = rga::compute_units();
  const size_t whole = 160 * 1024, half = whole / 2;
  const bool pairs = V > cus && V < 1 << 21;   // (a launch's threads count to 2^32)
  const bool pair_ring = pairs && zm + rings + 2048 <= half, pair_place = pairs && zm <= half;
  const int least = (pair_place && !pair_ring ? 2 : 1) * res * res;
  const bool ring = nf > kRingFaces && nf > least && zm + rings <= whole;
  const bool one = ring ? pair_ring : pair_place || V <= cus;
  // the partial boxes, the vertices' copy, the batches' ranges and the packed
  // triangles live in the filters' buffers, which are written after the raster
  // only; without room for them, or with a table too small to be of use, every
  // triangle projects its own.  (In place the copy pays from more than one view
  // per CU on: 13k triangles, 1024 views 114 -> 110 us; 5k, 64 views 31.5 -> 32 us
  // with the frame kernel.)
  char* const end = w + ws_bytes;
  float* boxes = reinterpret_cast<float*>(w + L.raw);
  float4* v4 = reinterpret_cast<float4*>(boxes + 8 * kBoxes);
  const int batches = (int)rga::ceil_div(nf, kBatch);
  int2* ranges = reinterpret_cast<int2*>(v4 + nv);
  uint2* packed = reinterpret_cast<uint2*>(ranges + batches);
  int64_t cap = ring ? std::min<int64_t>(((one ? half : whole) - zm - rings) / 16 * 8, nv) : 0;
  if (cap < 1024 && cap < nv) cap = 0;
  cap = std::min<int64_t>(cap, 32768);
  if (nf >= 1 << 28 || reinterpret_cast<char*>(packed + nf) > end) cap = 0;
  if (reinterpret_cast<char*>(v4 + nv) > end || !(ring || V > cus)) v4 = nullptr;
  // One workgroup takes the bounding box of few vertices and forms the frame: where a
  // workgroup has one view, joining partial boxes in it takes longer (2 us) than the
  // box does (1024 views of 13.6k triangles at 64^2 84 -> 81 us).
  const int nbox = one && nv <= 8192 ? 1 : kBoxes;
  const int packers = cap == 0 ? 0 : (int)(nv <= cap ? rga::ceil_div(nf, 1024) : batches);
  const size_t lds = zm + (ring ? rings + table_bytes((int)cap) : 0);
  auto raster =
      one ? (ring ? (v4 ? raster_kernel<true, true, true> : raster_kernel<true, false, true>)
                  : (v4 ? raster_kernel<false, true, true> : raster_kernel<false, false, true>))
          : (ring ? (v4 ? raster_kernel<true, true, false> : raster_kernel<true, false, false>)
                  : (v4 ? raster_kernel<false, true, false> : raster_kernel<false, false, false>));
  static bool attr_set = false;
  if (!attr_set) {
    for (auto k : {raster_kernel<true, true, false>, raster_kernel<true, false, false>,
                   raster_kernel<false, true, false>, raster_kernel<false, false, false>,
                   raster_kernel<true, true, true>, raster_kernel<true, false, true>,
                   raster_kernel<false, true, true>, raster_kernel<false, false, true>})
      hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    attr_set = true;
  }
  RGA_LAUNCH("vis_frame", frame_kernel, dim3(nbox + packers), dim3(1024), 0, s, nv,
             nf, nbox, verts, faces, (int)cap, boxes, ranges, packed, v4);
  const Verts mesh = {verts, v4, nv};
  const int grid = one ? V : std::min(V, cus);
  RGA_LAUNCH("vis_raster", raster, dim3(grid), dim3(kRasterThreads), lds, s, mesh, nf, faces,
             V, view_dirs, res, nbox, boxes, ranges, packed, (int)cap, vm, L.nwv, shadow, bias_px);
  const int64_t tw = (int64_t)L.nwv * L.nwV;
  RGA_LAUNCH("vis_transpose", transpose_kernel, dim3(rga::ceil_div(tw * 32, 256)), dim3(256), 0, s, nv,
             V, L.nwv, L.nwV, vm, raw);
  // Four words per thread of the filters where whole 16-byte groups make a row
  // and enough threads are left (the three filter launches together, one word
  // -> four: 1.27M words 79 -> 61 us, 433k 38 -> 34 us, 219k 28 us either way,
  // 27k 22 -> 27 us).
  const int64_t nw = (int64_t)nv * L.nwV;
  const bool wide = L.nwV % 4 == 0 && rga::aligned16(raw) && nw >= kWideWords;
  const dim3 fgrid(rga::ceil_div(wide ? nw / 4 : nw, 256));
  auto majority = wide ? majority_kernel<4> : majority_kernel<1>;
  auto counts = wide ? count_kernel<4> : count_kernel<1>;
  RGA_LAUNCH("vis_majority", majority, fgrid, dim3(256), 0, s, nv, L.nwV, knn, kv, raw, m1);
  RGA_LAUNCH("vis_majority", majority, fgrid, dim3(256), 0, s, nv, L.nwV, knn, kv, m1, m2);
  RGA_LAUNCH("vis_count", counts, fgrid, dim3(256), 0, s, nv, V, L.nwV, knn, kv, m2, count);
  RGA_CHECK_LAUNCH("mesh_visibility");
  return RGA_OK;
}

}  // namespace

extern "C" int mesh_visibility(void* stream, int nv, int nf, const float* verts,
                               const int32_t* faces, int V, const float* view_dirs, int res,
                               const int32_t* knn, int kv, uint32_t* raw_bits, uint8_t* count,
                               void* ws, size_t ws_bytes) {
  return visibility_impl(stream, nv, nf, verts, faces, V, view_dirs, res, knn, kv, raw_bits, count,
                         ws, ws_bytes, 0, 0.f);
}

namespace {

// ---- the variant that allocates nothing ----------------------------------
// Its workspace is this file-scope device array.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the
// symbol): the device address comes from hipGetSymbolAddress, taken once per
// device with that device current, and is kept per device.
constexpr size_t kNoAllocBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int scratch_for_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return rga::fail(RGA_EHIP, "mesh_visibility_noalloc: no current device");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return rga::fail(RGA_EHIP, "mesh_visibility_noalloc: hipGetSymbolAddress: %s",
                       hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return RGA_OK;
}

}  // namespace

extern "C" size_t mesh_visibility_noalloc_limit(void) { return kNoAllocBytes; }

extern "C" int mesh_visibility_noalloc(void* stream, int nv, int nf, const float* verts,
                                       const int32_t* faces, int V, const float* view_dirs,
                                       int res, const int32_t* knn, int kv, uint32_t* raw_bits,
                                       uint8_t* count) {
  if (nv < 1 || nf < 0 || V < 1)
    return rga::fail(RGA_EINVAL, "mesh_visibility_noalloc: nv >= 1, nf >= 0, V >= 1");
  const size_t need = vis_layout(nv, V).total;
  if (need > kNoAllocBytes)
    return rga::fail(RGA_ECAPACITY,
                     "mesh_visibility_noalloc: %d vertices x %d views need %zu B of scratch, "
                     "above its %zu B",
                     nv, V, need, kNoAllocBytes);
  void* ws = nullptr;
  const int rc = scratch_for_current_device(&ws);
  if (rc != RGA_OK) return rc;
  // every byte of the workspace that a kernel reads was written earlier in
  // the same call, so nothing is cleared
  return visibility_impl(stream, nv, nf, verts, faces, V, view_dirs, res, knn, kv, raw_bits, count,
                         ws, kNoAllocBytes, 0, 0.f);
}

extern "C" int mesh_visibility_shadowmap(void* stream, int nv, int nf, const float* verts,
                                         const int32_t* faces, int V, const float* view_dirs,
                                         int res, const int32_t* knn, int kv, float bias_px,
                                         uint32_t* raw_bits, uint8_t* count, void* ws,
                                         size_t ws_bytes) {
  if (!(bias_px >= 0.f && bias_px <= 64.f))
    return rga::fail(RGA_EINVAL, "mesh_visibility_shadowmap: bias_px in [0, 64]");
  return visibility_impl(stream, nv, nf, verts, faces, V, view_dirs, res, knn, kv, raw_bits, count,
                         ws, ws_bytes, 1, bias_px);
}
