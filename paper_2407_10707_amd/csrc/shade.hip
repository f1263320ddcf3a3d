// Per-Gaussian shading (Sec. 3.1 rendering equation, App. A BRDF) and its
// adjoint, FP32 form.
//
// Work mapping: one wave64 per Gaussian, lanes over light directions.  Per
// chunk of 64 directions each lane evaluates n.w_k and the interpolated
// visibility v_g[k] (three coalesced byte loads from the vertex-major count
// rows); a wave ballot compacts the live directions (n.w_k > 0 and
// v_g[k] > 0) into a 128-slot LDS ring, and the BRDF weights are evaluated
// only for full waves of live directions.  For a typical body roughly a
// third of the K directions are live, so the expensive part (GGX, Fresnel,
// Smith) runs at full SIMD width on that third only.  The per-lane sums are
// reduced across the wave once per Gaussian.
//
// The direction table (unit direction, radiance x solid angle, view index)
// is built in LDS by every workgroup; workgroups are persistent and loop
// over Gaussians.
//
// Given a tape, the forward also writes each Gaussian's live (direction,
// visibility) pairs, in the order and 64-pair groups of its walk; the
// adjoint of the same inputs then replays them instead of walking every
// direction again (same pairs, same lanes, same sums), which removes the
// direction test, the count rows and the ring from the adjoint.  The MFMA
// forward of the BF16X3 form writes the same tape (its pairs in step order),
// and the adjoint given one is this replay.
#include <algorithm>

#include "common.h"

#include <math.h>

namespace {

constexpr int kRing = 128;
constexpr float kPi = 3.14159265358979323846f;

struct ShadeArgs {
  int n, nv, V, kv, he, we, hv, wv, K;
  float cam[3];
  const float *x, *nrm, *albedo, *rough, *tint, *vw, *env;
  const int32_t* vidx;
  const uint8_t* count;
  int patch;   // table slots in 4 x 8 texel patches (the BF16X3 form), else texel order
  int split;   // factors of the contraction rounded to bf16 hi + lo (BF16X3 on the FP32 kernel)
  // the live-pair tape (NULL: none): per Gaussian its count and its live
  // (direction, visibility) pairs in the order visited, [n][K]
  int32_t* tape_n;
  uint2* tape;
};

// Direction k held by table slot s.  In texel order s = k.  In patch order
// (he % 4 == 0, we % 8 == 0) the slots run over patches of 4 texel rows x 8
// columns, patch-major along each band of 4 rows: slot 32 p + 8 i + j is
// texel (4 (p / (we / 8)) + i, 8 (p % (we / 8)) + j).  A patch is the
// 32-direction reduction step of the MFMA kernels, so the directions of one
// step lie close together and are often all below the horizon (or all
// occluded) for the 16 Gaussians of a tile.
__device__ inline int slot_k(int s, int we, int patch) {
  if (!patch) return s;
  const int p = s >> 5, q = s & 31;
  const int pw = we >> 3;
  const int pr = p / pw, pc = p - pr * pw;
  return (4 * pr + (q >> 3)) * we + 8 * pc + (q & 7);
}

// What the MFMA contraction keeps of a factor: its bf16 part and that of the rest.
__device__ inline float split2(float w) {
  const float hi = (float)(__bf16)w;
  return hi + (float)(__bf16)(w - hi);
}

// Table in LDS, two float4 per slot s (direction k = slot_k(s)): [s] =
// (direction x, y, z, view index as int bits), [K + s] = (E = radiance x
// texel solid angle, r, g, b, and k as int bits).  One 16-byte LDS read
// fetches either half.
__device__ inline void build_table(const ShadeArgs& a, float* tab) {
  float4* t4 = reinterpret_cast<float4*>(tab);
  const int K = a.K;
  const float dth = kPi / (float)a.he, dph = 2.f * kPi / (float)a.we;
  // exact solid angle of a texel row: (2 pi / we) * 2 sin(theta_r) sin(pi / (2 he))
  const float band = (2.f * kPi / (float)a.we) * 2.f * sinf(0.5f * dth);
  for (int sl = threadIdx.x; sl < K; sl += blockDim.x) {
    const int k = slot_k(sl, a.we, a.patch);
    const int r = k / a.we, c = k - r * a.we;
    float st, ct, sp, cp;
    sincosf(((float)r + 0.5f) * dth, &st, &ct);
    sincosf(((float)c + 0.5f) * dph, &sp, &cp);
    const float area = band * st;
    const int view = ((r * a.hv) / a.he) * a.wv + (c * a.wv) / a.we;
    t4[sl] = make_float4(st * sp, ct, st * cp, __int_as_float(view));
    float e[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      e[i] = a.env[3 * k + i] * area;
      if (a.split) e[i] = split2(e[i]);
    }
    t4[K + sl] = make_float4(e[0], e[1], e[2], __int_as_float(k));
  }
}

__device__ inline float4 dir_of(const float* tab, int k) {
  return reinterpret_cast<const float4*>(tab)[k];
}
__device__ inline float4 rad_of(const float* tab, int K, int k) {
  return reinterpret_cast<const float4*>(tab)[K + k];
}

struct Attr {
  float x[3], m[3], alb[3], rough, tint, vw[3];
  int vidx[3];
};

__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ inline void attr_load(const ShadeArgs& a, int g, Attr& A) {
  const int n = a.n, nvm = a.nv - 1;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    A.x[c] = a.x[(size_t)c * n + g];
    A.m[c] = a.nrm[(size_t)c * n + g];
    A.alb[c] = a.albedo[(size_t)c * n + g];
    A.vw[c] = a.vw[(size_t)c * n + g];
    A.vidx[c] = rga::clampi(a.vidx[(size_t)c * n + g], 0, nvm);
  }
  A.rough = a.rough[g];
  A.tint = a.tint[g];
}

// Reciprocal and reciprocal square root on the transcendental unit (about
// 1 ulp).  The shading sums are compared with the FP64 oracle under a
// relative tolerance, never bit for bit, so the correctly rounded
// division sequence buys nothing here.
__device__ inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

struct GaussCtx {
  float nn[3], wo[3], co, a2, kG, Go, Gq, inn, iwo, alpha, ialpha, gamma;
  float u0, u1, u2;
  const uint8_t* rows;   // LDS copy of the three count rows
  bool front;
};

// (In the wave-per-Gaussian kernels the constants are the same in every lane.
// They stay in vector registers all the same: to move 19 of them to scalar ones
// per Gaussian took 4 of 118 us, forward and back, at 100k Gaussians and 512
// directions, and occupancy does not ask for it.)
__device__ inline void gauss_setup(const ShadeArgs& a, const Attr& A, const uint8_t* rows,
                                   GaussCtx& G) {
  const float m0 = A.m[0], m1 = A.m[1], m2 = A.m[2];
  const float w0 = a.cam[0] - A.x[0], w1 = a.cam[1] - A.x[1], w2 = a.cam[2] - A.x[2];
  // back-face decision in FP32 with a fixed operation order
  const float dotf = fmaf(m2, w2, fmaf(m1, w1, m0 * w0));
  G.front = dotf > 0.f;
  G.inn = rsq(fmaf(m2, m2, fmaf(m1, m1, m0 * m0)));
  G.nn[0] = m0 * G.inn;
  G.nn[1] = m1 * G.inn;
  G.nn[2] = m2 * G.inn;
  G.iwo = rsq(fmaf(w2, w2, fmaf(w1, w1, w0 * w0)));
  G.wo[0] = w0 * G.iwo;
  G.wo[1] = w1 * G.iwo;
  G.wo[2] = w2 * G.iwo;
  G.co = fmaf(G.nn[2], G.wo[2], fmaf(G.nn[1], G.wo[1], G.nn[0] * G.wo[0]));
  G.gamma = A.rough;
  G.alpha = G.gamma * G.gamma;
  G.ialpha = rcp(G.alpha);
  G.a2 = G.alpha * G.alpha;
  G.kG = (G.gamma + 1.f) * (G.gamma + 1.f) * 0.125f;
  G.Go = rcp(fmaf(G.co, 1.f - G.kG, G.kG));
  G.Gq = G.Go * (0.25f / kPi);                      // the constant factors of W0
  const float ikv = 1.f / (float)a.kv;
  G.u0 = A.vw[0] * ikv;
  G.u1 = A.vw[1] * ikv;
  G.u2 = A.vw[2] * ikv;
  G.rows = rows;
}

struct Pair {
  float d[3], E[3], ci, ok, hh, nht, s2, den, invh, nh, oh, e2, F, hd, D, G1i, deni, ideni, W0F, W0, Ws,
      Wd;
};

// BRDF weights of one live (Gaussian, direction) pair.  The GGX denominator
// 1 - nh^2 (1 - alpha^2) is formed as (|n x h~|^2 + (n.h~)^2 alpha^2)/|h~|^2
// with h~ = w_k + w_o, which keeps its relative accuracy when nh -> 1.
__device__ inline void pair_eval(const GaussCtx& G, const float* tab, int K, int k, float v,
                                 Pair& P) {
  const float4 dv = dir_of(tab, k), er = rad_of(tab, K, k);
  P.d[0] = dv.x;
  P.d[1] = dv.y;
  P.d[2] = dv.z;
  P.E[0] = er.x;
  P.E[1] = er.y;
  P.E[2] = er.z;
  P.ci = fmaf(G.nn[2], P.d[2], fmaf(G.nn[1], P.d[1], G.nn[0] * P.d[0]));
  P.ok = fmaf(G.wo[2], P.d[2], fmaf(G.wo[1], P.d[1], G.wo[0] * P.d[0]));
  const float h0 = P.d[0] + G.wo[0], h1 = P.d[1] + G.wo[1], h2 = P.d[2] + G.wo[2];
  P.hh = fmaf(h2, h2, fmaf(h1, h1, h0 * h0));
  P.nht = P.ci + G.co;
  const float s0 = G.nn[1] * h2 - G.nn[2] * h1;
  const float s1 = G.nn[2] * h0 - G.nn[0] * h2;
  const float s2 = G.nn[0] * h1 - G.nn[1] * h0;
  P.s2 = fmaf(s2, s2, fmaf(s1, s1, s0 * s0));
  P.den = fmaf(P.nht * P.nht, G.a2, P.s2);           // (1 - nh^2 (1 - a^2)) |h~|^2
  P.invh = rsq(P.hh);
  P.nh = P.nht * P.invh;
  P.oh = (1.f + P.ok) * P.invh;
  // exponent in [-12.6, 0] (o.h in [0, 1]): the hardware exp2 needs no range step
  P.e2 = __builtin_amdgcn_exp2f((-5.55473f * P.oh - 6.98316f) * P.oh);
  P.F = 0.04f + 0.96f * P.e2;
  P.hd = P.hh * rcp(P.den);                         // 1 / (1 - nh^2 (1 - a^2))
  P.D = G.a2 * P.hd * P.hd;                         // pi D
  P.deni = fmaf(P.ci, 1.f - G.kG, G.kG);
  P.ideni = rcp(P.deni);
  P.G1i = P.ci * P.ideni;
  P.W0F = v * P.D * G.Gq;                          // W0 / F
  P.W0 = P.W0F * P.F;
  P.Ws = P.W0 * P.G1i;
  P.Wd = v * P.ci;
}

// x^p for x > 0 (normal) as 2^(p log2 x) on the transcendental unit: a
// few ulp, where the library powf spends ~180 instructions on special
// cases that cannot occur here.
__device__ inline float pos_pow(float x, float p) {
  return __builtin_amdgcn_exp2f(p * __builtin_amdgcn_logf(x));
}

// sRGB transfer curve (gamma correction of L_o)
__device__ inline float srgb(float L) {
  return L <= 0.0031308f ? 12.92f * L : 1.055f * pos_pow(L, 1.f / 2.4f) - 0.055f;
}

// dL/dL_o from dL/dcolour, with L_o recovered from the colour by inverting
// the transfer curve
__device__ inline float srgb_adjoint(float col, float dc) {
  if (col <= 0.04045f) return dc * 12.92f;
  const float Lo = pos_pow((col + 0.055f) / 1.055f, 2.4f);
  return dc * (col + 0.055f) / (2.4f * Lo);
}

__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- FP32 form: one wave per front-facing Gaussian ---------------------------
// A workgroup takes up to `cap` Gaussians at a time: each thread loads one
// Gaussian's position and normal and decides the back-face rule; a back-facing
// Gaussian's outputs are written at once (it needs nothing else, and its count
// rows are never read), and the front-facing ones are listed in LDS with their
// three nearest vertices.  The waves then take entries of the list from a
// shared counter until it is empty: per chunk of 64 directions each lane tests
// its direction, a ballot compacts the live ones into the wave's LDS ring, and
// whole waves of ring entries go to the BRDF stage.  The next entry's count
// rows and attributes are loaded into registers while the current one is
// shaded, and the rows then written to the wave's LDS slot.
//
// Bound by vector issue (87 % of the slots forward, 95 % adjoint at 200k
// Gaussians and 2048 directions).  A wave that walked its own fixed share of
// the Gaussians left the others waiting (the back-facing ones come in runs),
// and two sets of rows per wave in LDS left two waves per SIMD at 2048
// directions: 200k Gaussians there 663 -> 294 us forward, 457 -> 280 us adjoint;
// 100k at 512 directions 80 -> 53 us and 85 -> 65 us.

// Per-lane plan of the count-row copies (depends only on the lane and V):
// 16-byte piece q = lane + 64 i is byte 16 q of the three rows laid end to
// end, i.e. row j = 16 q / V at offset 16 q - j V; packed as off << 2 | j
// (j = 3: no piece).
template <int NQ>
struct RowPlan {
  int p[NQ];
};

template <int NQ>
__device__ inline void row_plan(int V, int lane, RowPlan<NQ>& P) {
  const int nq = 3 * V / 16;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int q = lane + 64 * i;
    const int j = (16 * q) / V;
    P.p[i] = q < nq ? ((16 * q - j * V) << 2) | j : 3;
  }
}

// the three count rows of a Gaussian, in registers
template <int NQ>
struct Rows {
  uint4 q[NQ];
};

template <int NQ>
__device__ inline void rows_load(const ShadeArgs& a, const RowPlan<NQ>& P, const int* vidx,
                                 Rows<NQ>& R) {
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int j = P.p[i] & 3;
    const int vi = j == 0 ? vidx[0] : (j == 1 ? vidx[1] : vidx[2]);
    R.q[i] = make_uint4(0u, 0u, 0u, 0u);
    if (j != 3)
      R.q[i] = *reinterpret_cast<const uint4*>(a.count + (size_t)vi * a.V + (P.p[i] >> 2));
  }
}

template <int NQ>
__device__ inline void rows_store(const RowPlan<NQ>& P, const Rows<NQ>& R, uint8_t* lds, int lane) {
#pragma unroll
  for (int i = 0; i < NQ; ++i)
    if ((P.p[i] & 3) != 3) *reinterpret_cast<uint4*>(lds + 16 * lane + 1024 * i) = R.q[i];
}

// The workgroup's Gaussians at(0) .. at(count - 1).  With a grid of whole
// groups of 8 workgroups, those that share a remainder modulo 8 (dispatched to
// the same XCD, whose L2 they share) take every eighth of 64 contiguous
// segments: with the Gaussians stored grouped by nearest vertex, each XCD
// gathers count rows from about an eighth of the table, and its L2 holds them,
// and each has its share of every part of the body.  Within the XCD the
// workgroups take every (grid / 8)-th.
constexpr int kSegments = 64;

struct Walk {
  int first, stride, count, seg, x;
};

__device__ inline Walk group_walk(int n) {
  Walk w;
  const int grid = gridDim.x, b = blockIdx.x;
  const bool xcd = grid % 8 == 0;
  w.x = xcd ? b % 8 : -1;
  w.first = xcd ? b / 8 : b;
  w.stride = xcd ? grid / 8 : grid;
  w.seg = (n + kSegments - 1) / kSegments;
  const int len = xcd ? (kSegments / 8) * w.seg : n;
  w.count = w.first < len ? (len - 1 - w.first) / w.stride + 1 : 0;
  return w;
}

// index of the m-th Gaussian, -1 if there is none
__device__ inline int walk_at(const Walk& w, int n, int m) {
  if (m >= w.count) return -1;
  const int q = w.first + m * w.stride;
  if (w.x < 0) return q;
  const int s = q / w.seg;
  const int g = (8 * s + w.x) * w.seg + (q - s * w.seg);
  return g < n ? g : -1;
}

// Fill the list with the front-facing ones of the workgroup's Gaussians m0 ..
// m0 + cap - 1 (FP32 test, fixed order, as gauss_setup); back(g) finishes a
// back-facing one, each(g, front) sees every one.
template <class Each>
__device__ inline void list_fill(const ShadeArgs& a, const Walk& w, int m0, int cap, int4* list,
                                 int* count, uint64_t lt, Each&& each) {
  for (int t = threadIdx.x; t - (int)(threadIdx.x & 63) < cap; t += blockDim.x) {
    const int g = t < cap ? walk_at(w, a.n, m0 + t) : -1;
    bool front = false;
    int4 e = make_int4(g, 0, 0, 0);
    if (g >= 0) {
      const int n = a.n;
      float x[3], m[3];
      int vi[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        x[c] = a.x[(size_t)c * n + g];
        m[c] = a.nrm[(size_t)c * n + g];
        vi[c] = a.vidx[(size_t)c * n + g];
      }
      const float w0 = a.cam[0] - x[0], w1 = a.cam[1] - x[1], w2 = a.cam[2] - x[2];
      front = fmaf(m[2], w2, fmaf(m[1], w1, m[0] * w0)) > 0.f;
      each(g, front);
      e.y = rga::clampi(vi[0], 0, a.nv - 1);
      e.z = rga::clampi(vi[1], 0, a.nv - 1);
      e.w = rga::clampi(vi[2], 0, a.nv - 1);
    }
    const uint64_t f = __ballot(front);
    if (f == 0ull) continue;
    int at = 0;
    if ((threadIdx.x & 63) == 0) at = atomicAdd(count, (int)__popcll(f));
    at = __builtin_amdgcn_readfirstlane(at);
    if (front) list[at + __popcll(f & lt)] = e;
  }
}

// The wave's next entry of the list: its number, from the shared counter.
__device__ inline int list_take(int* next, int lane) {
  int t = 0;
  if (lane == 0) t = atomicAdd(next, 1);
  return __builtin_amdgcn_readfirstlane(t);
}

// A listed Gaussian's attributes are loaded by one instruction, lane i the i-th
// of x, n, albedo, weights (three each), roughness and tint, and read from the
// lanes when its turn comes (held in scalar registers from the load on, with
// the arrays' addresses, they were spilled).
__device__ inline const float* attr_lane(const ShadeArgs& a, int lane) {
  const int c = lane % 3, q = lane / 3;
  const float* p = q == 0 ? a.x : (q == 1 ? a.nrm : (q == 2 ? a.albedo : a.vw));
  p += (size_t)c * a.n;
  return lane < 12 ? p : (lane == 12 ? a.rough : a.tint);
}

__device__ inline void attr_read(float v, Attr& A) {
  auto at = [v](int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i)); };
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    A.x[c] = at(c);
    A.m[c] = at(3 + c);
    A.alb[c] = at(6 + c);
    A.vw[c] = at(9 + c);
  }
  A.rough = at(12);
  A.tint = at(13);
}

// Walk the K directions of one Gaussian 64 at a time: lane = direction,
// the live ones (n.w_k > 0 and visibility > 0) appended with their
// visibility to the wave's ring; flush(k, v, on, base) on every whole wave
// of ring entries as it fills and on the remainder (base = the number of
// live pairs flushed before).  Returns the number of live pairs.  Two waves of
// directions are looked up together: each lookup is two dependent LDS reads, for
// whose latency four waves per SIMD are too few (200k Gaussians, 2048 directions
// 312 -> 271 us, one at a time without the branches 301, four 267 but 63 us
// against 60 at 128 directions).
template <class Flush>
__device__ inline int live_walk(const GaussCtx& G, const float* tab, int K, int V, int* qk,
                                float* qv, int lane, Flush&& flush) {
  int head = 0, tail = 0;
  auto append = [&](int k, float v) {
    const bool live = v > 0.f;
    const uint64_t m = __ballot(live);
    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)m, tail));
    if (live) {
      qk[at & (kRing - 1)] = k;
      qv[at & (kRing - 1)] = v;
    }
    tail += __popcll(m);
    if (tail - head >= 64) {
      wave_fence();
      const int slot = (head + lane) & (kRing - 1);
      flush(qk[slot], qv[slot], true, head);
      head += 64;
      wave_fence();
    }
  };
  for (int k0 = 0; k0 < K; k0 += 128) {
    float ci[2], v[2] = {0.f, 0.f};
    int view[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = k0 + 64 * h + lane;
      const float4 dv = dir_of(tab, min(k, K - 1));
      ci[h] = fmaf(G.nn[2], dv.z, fmaf(G.nn[1], dv.y, G.nn[0] * dv.x));
      if (k >= K) ci[h] = 0.f;
      view[h] = __float_as_int(dv.w);
    }
    if (__ballot(ci[0] > 0.f || ci[1] > 0.f) == 0ull) continue;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float c0 = (float)G.rows[view[h]], c1 = (float)G.rows[V + view[h]],
                  c2 = (float)G.rows[2 * V + view[h]];
      v[h] = ci[h] > 0.f ? fmaf(G.u2, c2, fmaf(G.u1, c1, G.u0 * c0)) : 0.f;
    }
    append(k0 + lane, v[0]);
    append(k0 + 64 + lane, v[1]);
  }
  if (tail > head) {
    wave_fence();
    const int slot = (head + lane) & (kRing - 1);
    flush(qk[slot], qv[slot], lane < tail - head, head);
    wave_fence();
  }
  return tail;
}

// LDS of the FP32 kernels: the direction table (8 K floats; the adjoint adds
// 3 K for the environment gradient), then per wave the count rows (3 V bytes)
// and the ring (none in the adjoint that reads a tape), then the list.
template <int WAVES>
struct Lds {
  float* tab;
  uint8_t* rows;
  int* qk;
  float* qv;
  int4* list;
};

template <int WAVES>
__device__ inline Lds<WAVES> lds_of(float* smem, int tab_floats, int V, int wave, bool walks) {
  Lds<WAVES> L;
  L.tab = smem;
  uint8_t* p = reinterpret_cast<uint8_t*>(smem + tab_floats);
  L.rows = p + (size_t)wave * 3 * V;
  if (walks) p += (size_t)WAVES * 3 * V;
  L.qk = reinterpret_cast<int*>(p) + wave * kRing;
  L.qv = reinterpret_cast<float*>(p) + (WAVES + wave) * kRing;
  if (walks) p += (size_t)WAVES * kRing * 8;
  L.list = reinterpret_cast<int4*>(p);
  return L;
}

template <int NQ, int WAVES>
__global__ void __launch_bounds__(WAVES * 64, NQ <= 2 ? 8 : 4)
shade_fwd_kernel(ShadeArgs a, int cap, float* __restrict__ color, uint8_t* __restrict__ front) {
  extern __shared__ __align__(16) float smem[];
  __shared__ int ctl[2][2];   // entries listed and taken, of alternate rounds
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int K = a.K, n = a.n, V = a.V;
  const Lds<WAVES> L = lds_of<WAVES>(smem, 8 * K, V, wave, true);
  const float* tab = L.tab;
  if (threadIdx.x < 4) (&ctl[0][0])[threadIdx.x] = 0;
  build_table(a, smem);
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  RowPlan<NQ> plan;
  row_plan<NQ>(V, lane, plan);
  const float* pattr = attr_lane(a, lane);
  const Walk walk = group_walk(n);
  for (int m0 = 0, r = 0; m0 < walk.count; m0 += cap, r ^= 1) {
    __syncthreads();          // the last round's list is done with
    if (threadIdx.x < 2) ctl[r ^ 1][threadIdx.x] = 0;
    list_fill(a, walk, m0, cap, L.list, &ctl[r][0], lt, [&](int g, bool f) {
      front[g] = f ? 1 : 0;
      if (f) return;
#pragma unroll
      for (int c = 0; c < 3; ++c) color[(size_t)c * n + g] = 0.f;
      if (a.tape_n) a.tape_n[g] = 0;
    });
    __syncthreads();
    const int entries = ctl[r][0];
    int t = list_take(&ctl[r][1], lane);
    Rows<NQ> R;
    int g = 0;
    float v = 0.f;
    auto load = [&](int e) {
      const int4 le = L.list[e];
      const int gg = uni(le.x);
      const int vidx[3] = {uni(le.y), uni(le.z), uni(le.w)};
      v = pattr[gg];
      rows_load(a, plan, vidx, R);
      return gg;
    };
    if (t < entries) {
      g = load(t);
      rows_store(plan, R, L.rows, lane);
    }
    while (t < entries) {
      Attr A;
      attr_read(v, A);
      t = list_take(&ctl[r][1], lane);
      int gn = 0;
      if (t < entries) gn = load(t);
      wave_fence();
      GaussCtx G;
      gauss_setup(a, A, L.rows, G);
      float sd0 = 0.f, sd1 = 0.f, sd2 = 0.f, ss0 = 0.f, ss1 = 0.f, ss2 = 0.f;
      // this Gaussian's row of the tape (a wave-uniform address)
      uint2* const trow = a.tape ? a.tape + (size_t)uni(g) * K : nullptr;
      const int nlive = live_walk(G, tab, K, V, L.qk, L.qv, lane,
                                  [&](int k, float v, bool on, int base) {
        if (on) {
          Pair P;
          pair_eval(G, tab, K, k, v, P);
          if (trow)
            trow[base + lane] = make_uint2(__float_as_uint(rad_of(tab, K, k).w), __float_as_uint(v));
          if (a.split) {
            P.Wd = split2(P.Wd);
            P.Ws = split2(P.Ws);
          }
          sd0 = fmaf(P.Wd, P.E[0], sd0);
          sd1 = fmaf(P.Wd, P.E[1], sd1);
          sd2 = fmaf(P.Wd, P.E[2], sd2);
          ss0 = fmaf(P.Ws, P.E[0], ss0);
          ss1 = fmaf(P.Ws, P.E[1], ss1);
          ss2 = fmaf(P.Ws, P.E[2], ss2);
        }
      });
      if (trow && lane == 0) a.tape_n[g] = nlive;
      sd0 = rga::wave_sum(sd0);
      sd1 = rga::wave_sum(sd1);
      sd2 = rga::wave_sum(sd2);
      ss0 = rga::wave_sum(ss0);
      ss1 = rga::wave_sum(ss1);
      ss2 = rga::wave_sum(ss2);
      if (lane < 3) {
        const float sd = lane == 0 ? sd0 : (lane == 1 ? sd1 : sd2);
        const float ss = lane == 0 ? ss0 : (lane == 1 ? ss1 : ss2);
        const float alb = lane == 0 ? A.alb[0] : (lane == 1 ? A.alb[1] : A.alb[2]);
        color[(size_t)lane * n + g] = srgb(alb * (1.f / kPi) * sd + A.tint * ss);
      }
      wave_fence();
      if (t < entries) rows_store(plan, R, L.rows, lane);
      g = gn;
    }
  }
}

// ---- BF16X3 form: the contraction on MFMA -----------------------------------
// A wave owns 16 Gaussians (MFMA rows) and walks the light directions 32 at
// a time (the MFMA reduction dimension).  Lane l evaluates the BRDF weights of
// Gaussian l % 16 for the 8 directions 8 (l / 16) .. + 7 of the step -- exactly
// its slots of the A operand -- on VALU, splits each weight into bf16 hi + lo,
// and the contraction with B = [E_hi | E_lo] (columns 0-2 and 3-5) runs on
// v_mfma_f32_16x16x32_bf16 with FP32 accumulation:
//   S_c = A_hi E_hi + A_hi E_lo + A_lo E_hi + A_lo E_lo (columns c and c+3).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMWaves = 4;
constexpr int kMThreads = kMWaves * 64;

// LDS: dir x,y,z | E r,g,b | view (int) [K each], then B [16 cols][K] bf16
// B operand of the shading contraction in LDS, [6 columns][K] bf16:
// columns 0-2 the high parts of E (r, g, b), 3-5 the low parts.  The other
// ten columns of the 16-wide MFMA operand are zero and never stored.
__device__ inline void build_btab(const float* tab, int K, __bf16* bt) {
  for (int i = threadIdx.x; i < 6 * K; i += blockDim.x) {
    const int col = i / K, k = i - col * K;
    float v = 0.f;
    const float4 er = rad_of(tab, K, k);
    const int cc = col < 3 ? col : col - 3;
    const float e = cc == 0 ? er.x : (cc == 1 ? er.y : er.z);
    v = col < 3 ? (float)(__bf16)e : e - (float)(__bf16)e;
    bt[i] = (__bf16)v;
  }
}

// 8 consecutive k of column `col` of the B operand (zero for col >= 6).
__device__ inline bf16x8 btab_load(const __bf16* bt, int K, int col, int kb) {
  const bf16x8 b = *reinterpret_cast<const bf16x8*>(bt + (size_t)min(col, 5) * K + kb);
  const bf16x8 z = {};
  return col < 6 ? b : z;
}

// visibility bytes of 8 consecutive directions k..k+7 (k % 8 == 0, same
// texel row) for one count row: identity view map (view = k), two texels
// per view (view = k / 2), or the table's view indices
__device__ inline void vis8(const uint8_t* row, const float* tab, int k, int ratio, float* c) {
  if (ratio == 1) {
    const uint2 w = *reinterpret_cast<const uint2*>(row + k);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      c[i] = (float)((w.x >> (8 * i)) & 0xFFu);
      c[4 + i] = (float)((w.y >> (8 * i)) & 0xFFu);
    }
  } else if (ratio == 2) {
    const uint32_t w = *reinterpret_cast<const uint32_t*>(row + (k >> 1));
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = (float)((w >> (8 * (i >> 1))) & 0xFFu);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = (float)row[__float_as_int(dir_of(tab, k + i).w)];
  }
}

// Slots kb .. kb+7 of one lane (8 texels of one row, consecutive in the
// texel order too): the interpolated visibility of each and the mask of
// the live ones (front-facing, n.w_k > 0, visibility > 0).
__device__ inline uint32_t live8(const ShadeArgs& a, const GaussCtx& G, const float* tab,
                                 const uint8_t* r0, const uint8_t* r1, const uint8_t* r2, int kb,
                                 int ratio, bool on, float (&vv)[8]) {
  const int kv = ratio ? slot_k(kb, a.we, a.patch) : kb;
  float c0[8], c1[8], c2[8];
  vis8(r0, tab, kv, ratio, c0);
  vis8(r1, tab, kv, ratio, c1);
  vis8(r2, tab, kv, ratio, c2);
  uint32_t lm = 0u;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float4 dv = dir_of(tab, kb + i);
    const float ci = fmaf(G.nn[2], dv.z, fmaf(G.nn[1], dv.y, G.nn[0] * dv.x));
    vv[i] = fmaf(G.u2, c2[i], fmaf(G.u1, c1[i], G.u0 * c0[i]));
    if (on && ci > 0.f && vv[i] > 0.f) lm |= 1u << i;
  }
  return lm;
}

__global__ void __launch_bounds__(kMThreads)
shade_fwd_mfma_kernel(ShadeArgs a, int ratio, float* __restrict__ color,
                      uint8_t* __restrict__ front) {
  extern __shared__ __align__(16) float tab[];
  const int K = a.K, n = a.n, V = a.V;
  __bf16* bt = reinterpret_cast<__bf16*>(tab + 8 * K);
  float* stage = reinterpret_cast<float*>(bt + 6 * K) + (threadIdx.x >> 6) * 512;
  build_table(a, tab);
  __syncthreads();
  build_btab(tab, K, bt);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, kg = lane >> 4;
  const int ntiles = (n + 15) / 16;
  for (int tile = blockIdx.x * kMWaves + wave; tile < ntiles; tile += gridDim.x * kMWaves) {
    const int g = tile * 16 + row;
    const bool have = g < n;
    Attr A;
    attr_load(a, have ? g : n - 1, A);
    GaussCtx G;
    gauss_setup(a, A, nullptr, G);
    const bool on = have && G.front;
    const uint8_t* r0 = a.count + (size_t)A.vidx[0] * V;
    const uint8_t* r1 = a.count + (size_t)A.vidx[1] * V;
    const uint8_t* r2 = a.count + (size_t)A.vidx[2] * V;
    f32x4 accD = {0.f, 0.f, 0.f, 0.f}, accS = {0.f, 0.f, 0.f, 0.f};
    // the tape: this Gaussian's live pairs so far (the same in the four
    // lanes of its row), written step by step in (step, lane group, i) order
    int tcount = 0;
    uint2* const trow = (a.tape && on) ? a.tape + (size_t)g * K : nullptr;
    for (int k0 = 0; k0 < K; k0 += 32) {
      const int kb = k0 + 8 * kg;
      float vv[8];
      const uint32_t lm = live8(a, G, tab, r0, r1, r2, kb, ratio, on, vv);
      // a step with no live pair in the tile adds nothing
      if (__ballot(lm != 0u) == 0ull) continue;
      if (a.tape) {
        // this lane's pairs follow those of the row's lanes with smaller kg
        const int p = __popc(lm);
        const int p0 = __shfl(p, row), p1 = __shfl(p, row + 16), p2 = __shfl(p, row + 32),
                  p3 = __shfl(p, row + 48);
        int pos = tcount + (kg > 0 ? p0 : 0) + (kg > 1 ? p1 : 0) + (kg > 2 ? p2 : 0);
        if (trow) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if ((lm >> i) & 1u)
              trow[pos++] = make_uint2((uint32_t)slot_k(kb + i, a.we, a.patch),
                                       __float_as_uint(vv[i]));
        }
        tcount += p0 + p1 + p2 + p3;
      }
      bf16x8 dh, dl, sh, sl;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = kb + i;
        float Wd = 0.f, Ws = 0.f;
        if ((lm >> i) & 1u) {
          Pair P;
          pair_eval(G, tab, K, k, vv[i], P);
          Wd = P.Wd;
          Ws = P.Ws;
        }
        const __bf16 hd = (__bf16)Wd, hs = (__bf16)Ws;
        dh[i] = hd;
        dl[i] = (__bf16)(Wd - (float)hd);
        sh[i] = hs;
        sl[i] = (__bf16)(Ws - (float)hs);
      }
      const bf16x8 b = btab_load(bt, K, row, kb);
      accD = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dh, b, accD, 0, 0, 0);
      accD = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dl, b, accD, 0, 0, 0);
      accS = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sh, b, accS, 0, 0, 0);
      accS = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sl, b, accS, 0, 0, 0);
    }
    if (a.tape_n && have && kg == 0) a.tape_n[g] = tcount;
    // D[row 4 kg + i][col] -> stage; then one lane per (Gaussian, channel)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      stage[(4 * kg + i) * 16 + row] = accD[i];
      stage[256 + (4 * kg + i) * 16 + row] = accS[i];
    }
    wave_fence();
    if (lane < 48) {
      const int gr = lane / 3, c = lane - 3 * gr;
      const int gg = tile * 16 + gr;
      if (gg < n) {
        const float sd = stage[gr * 16 + c] + stage[gr * 16 + 3 + c];
        const float ss = stage[256 + gr * 16 + c] + stage[256 + gr * 16 + 3 + c];
        // this Gaussian's inputs (lane gr of the tile holds them)
        const float alb = a.albedo[(size_t)c * n + gg];
        const float tnt = a.tint[gg];
        const float m0 = a.nrm[gg], m1 = a.nrm[n + gg], m2 = a.nrm[2 * n + gg];
        const float w0 = a.cam[0] - a.x[gg], w1 = a.cam[1] - a.x[n + gg],
                    w2 = a.cam[2] - a.x[2 * n + gg];
        const bool fr = fmaf(m2, w2, fmaf(m1, w1, m0 * w0)) > 0.f;
        color[(size_t)c * n + gg] = fr ? srgb(alb * (1.f / kPi) * sd + tnt * ss) : 0.f;
        if (c == 0) front[gg] = fr ? 1 : 0;
      }
    }
    wave_fence();
  }
}

// ---- adjoint ------------------------------------------------------------
struct BwdAcc {
  float gn[3], gw[3], gco, gga, sd[3], ts;
};

// Chain rule through one live pair's weights: upstream gWd = dL/dW_d and
// gWs = dL/dW_s give the pair's share of dL/dn^, dL/dw_o, dL/d(n.w_o) and
// dL/dgamma.  Uses the logarithmic derivatives of D (in n.h and alpha), F
// (through dF/d(o.h)) and G1.  Only the part of dL/dw_o orthogonal to w_o
// reaches x, so the w_o terms are taken along h = h~/|h~|: n.h changes by
// (n - (n.h) h)/|h~| and o.h = |h~|/2 by h/2 (up to multiples of w_o).  The
// same derivative taken through o.w_k (d(n.h)/d(o.w_k) = -(n.h~)/|h~|^3)
// is of size 1/|h~|^2 near w_k = -w_o, almost all of it along w_o, and the
// projection onto the tangent plane then cancels it in FP32.
__device__ inline void pair_grads(const GaussCtx& G, const Pair& P, float v, float gWd, float gWs,
                                  BwdAcc& acc) {
  const float one_m_a2 = 1.f - G.a2;
  const float dlnD_dnh = 4.f * P.nh * one_m_a2 * P.hd;
  const float dlnD_da = 2.f * G.ialpha - 4.f * G.alpha * P.nh * P.nh * P.hd;
  // dF/d(o.h); gs dlnF/d(o.h) = gWs (W_s / F) dF/d(o.h) needs no 1/F
  const float dF_doh = 0.96f * P.e2 * 0.69314718f * (-2.f * 5.55473f * P.oh - 6.98316f);
  const float gs = gWs * P.Ws;
  const float gsF = gWs * P.W0F * P.G1i * dF_doh;
  const float gnh = gs * dlnD_dnh * P.invh;          // dL/d(n.h~) through D
  const float gci = gWd * v + gWs * P.W0 * G.kG * (P.ideni * P.ideni) + gnh;
  const float gco = gnh - gs * (1.f - G.kG) * G.Go;
  // dL/dw_o = gco n + ghh h~ (modulo w_o)
  const float ghh = fmaf(-gnh, P.nh, 0.5f * gsF) * P.invh;
  const float dlnG_dk = -(1.f - P.ci) * P.ideni - (1.f - G.co) * G.Go;
  const float gga = gs * (dlnD_da * 2.f * G.gamma + dlnG_dk * (G.gamma + 1.f) * 0.25f);
  acc.gn[0] = fmaf(gci, P.d[0], acc.gn[0]);
  acc.gn[1] = fmaf(gci, P.d[1], acc.gn[1]);
  acc.gn[2] = fmaf(gci, P.d[2], acc.gn[2]);
  acc.gw[0] = fmaf(ghh, P.d[0] + G.wo[0], acc.gw[0]);
  acc.gw[1] = fmaf(ghh, P.d[1] + G.wo[1], acc.gw[1]);
  acc.gw[2] = fmaf(ghh, P.d[2] + G.wo[2], acc.gw[2]);
  acc.gco += gco;
  acc.gga += gga;
}

__device__ inline void pair_bwd(const GaussCtx& G, const float* tab, float* denv_lds, int K, int k,
                                float v, const float* qd, const float* dLo, float tint,
                                const float* aop, BwdAcc& acc) {
  Pair P;
  pair_eval(G, tab, K, k, v, P);
  // upstream weights of W_d and W_s
  const float gWd = fmaf(qd[2], P.E[2], fmaf(qd[1], P.E[1], qd[0] * P.E[0]));
  const float sE = fmaf(dLo[2], P.E[2], fmaf(dLo[1], P.E[1], dLo[0] * P.E[0]));
  const float gWs = tint * sE;
  acc.sd[0] = fmaf(P.Wd, P.E[0], acc.sd[0]);
  acc.sd[1] = fmaf(P.Wd, P.E[1], acc.sd[1]);
  acc.sd[2] = fmaf(P.Wd, P.E[2], acc.sd[2]);
  acc.ts = fmaf(P.Ws, sE, acc.ts);
  // environment: dL/d(L_k,c A_k) = dLo_c (a_c/pi W_d + p W_s); the area
  // factor is applied when the per-workgroup sums are reduced
  rga::lds_add3(&denv_lds[3 * k], dLo[0] * fmaf(aop[0], P.Wd, tint * P.Ws),
                dLo[1] * fmaf(aop[1], P.Wd, tint * P.Ws), dLo[2] * fmaf(aop[2], P.Wd, tint * P.Ws));
  pair_grads(G, P, v, gWd, gWs, acc);
}

// BF16X3 adjoint.  Same tiling (16 Gaussians x 32 directions per step).  On
// MFMA: the per-Gaussian sums S_d = W_d E and S_s = W_s E (for the albedo and
// tint gradients, 16x16x32 as in the forward), and the environment gradient
// dE[k][c] = sum_g W_d[g][k] Qd[g][c] + W_s[g][k] Qs[g][c] with
// Qd = dL/dL_o a / pi, Qs = dL/dL_o p -- a reduction over Gaussians, so W is
// transposed through LDS and fed to v_mfma_f32_32x32x16_bf16 (A = W^T,
// 32 directions x 16 Gaussians; B = [Q_hi | Q_lo]).  The direction-dependent
// derivative terms of the BRDF weights stay on VALU in FP32.
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ void __launch_bounds__(kMThreads)
shade_bwd_mfma_kernel(ShadeArgs a, int ratio, const float* __restrict__ color,
                      const float* __restrict__ dcolor, float* __restrict__ dx,
                      float* __restrict__ dn, float* __restrict__ dalbedo,
                      float* __restrict__ drough, float* __restrict__ dtint,
                      float* __restrict__ denv_part) {
  extern __shared__ __align__(16) float tab[];
  const int K = a.K, n = a.n, V = a.V;
  __bf16* bt = reinterpret_cast<__bf16*>(tab + 8 * K);
  float* denv_lds = reinterpret_cast<float*>(bt + 6 * K);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // per-wave scratch: W^T stage (4 x [32 k][16 g] bf16 = 4 KB), Q (16 x 6 f32),
  // per-Gaussian sums (2 x 256 f32)
  char* wbase = reinterpret_cast<char*>(denv_lds + 3 * K) + (size_t)wave * (4096 + 384 + 2048);
  __bf16* wt = reinterpret_cast<__bf16*>(wbase);
  float* qst = reinterpret_cast<float*>(wbase + 4096);
  float* stage = reinterpret_cast<float*>(wbase + 4096 + 384);
  build_table(a, tab);
  for (int i = threadIdx.x; i < 3 * K; i += blockDim.x) denv_lds[i] = 0.f;
  __syncthreads();
  build_btab(tab, K, bt);
  __syncthreads();
  const int row = lane & 15, kg = lane >> 4;
  const int ntiles = (n + 15) / 16;
  for (int tile = blockIdx.x * kMWaves + wave; tile < ntiles; tile += gridDim.x * kMWaves) {
    const int g = tile * 16 + row;
    const bool have = g < n;
    const int gc = have ? g : n - 1;
    Attr A;
    attr_load(a, gc, A);
    GaussCtx G;
    gauss_setup(a, A, nullptr, G);
    const bool on = have && G.front;
    float dLo[3], aop[3], qd[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float col = color[(size_t)c * n + gc];
      const float dc = on ? dcolor[(size_t)c * n + gc] : 0.f;
      dLo[c] = srgb_adjoint(col, dc);
      aop[c] = A.alb[c] * (1.f / kPi);
      qd[c] = dLo[c] * aop[c];
    }
    const float tint = A.tint;
    // B operand of the environment contraction: Q of the tile's 16 Gaussians
    if (kg == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        qst[row * 6 + c] = qd[c];
        qst[row * 6 + 3 + c] = dLo[c] * tint;
      }
    }
    wave_fence();
    bf16x8 bqd, bqs;   // B [16 g][32 cols]: lane holds col lane % 32, g = 8 (lane / 32) + i
    {
      const int col = lane & 31, g0 = 8 * (lane >> 5);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float vd = 0.f, vs = 0.f;
        if (col < 6) {
          const float qdv = qst[(g0 + i) * 6 + (col % 3)];
          const float qsv = qst[(g0 + i) * 6 + 3 + (col % 3)];
          vd = col < 3 ? (float)(__bf16)qdv : qdv - (float)(__bf16)qdv;
          vs = col < 3 ? (float)(__bf16)qsv : qsv - (float)(__bf16)qsv;
        }
        bqd[i] = (__bf16)vd;
        bqs[i] = (__bf16)vs;
      }
    }
    const uint8_t* r0 = a.count + (size_t)A.vidx[0] * V;
    const uint8_t* r1 = a.count + (size_t)A.vidx[1] * V;
    const uint8_t* r2 = a.count + (size_t)A.vidx[2] * V;
    f32x4 accD = {0.f, 0.f, 0.f, 0.f}, accS = {0.f, 0.f, 0.f, 0.f};
    BwdAcc acc = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, 0.f, 0.f, {0.f, 0.f, 0.f}, 0.f};
    for (int k0 = 0; k0 < K; k0 += 32) {
      const int kb = k0 + 8 * kg;
      float vv[8];
      const uint32_t lm = live8(a, G, tab, r0, r1, r2, kb, ratio, on, vv);
      // a step with no live pair in the tile adds nothing (W = 0)
      if (__ballot(lm != 0u) == 0ull) continue;
      bf16x8 dh, dl, sh, sl;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = kb + i;
        float Wd = 0.f, Ws = 0.f;
        if ((lm >> i) & 1u) {
          Pair P;
          pair_eval(G, tab, K, k, vv[i], P);
          Wd = P.Wd;
          Ws = P.Ws;
          const float gWd = fmaf(qd[2], P.E[2], fmaf(qd[1], P.E[1], qd[0] * P.E[0]));
          const float sE = fmaf(dLo[2], P.E[2], fmaf(dLo[1], P.E[1], dLo[0] * P.E[0]));
          const float gWs = tint * sE;
          pair_grads(G, P, vv[i], gWd, gWs, acc);
        }
        const __bf16 hd = (__bf16)Wd, hs = (__bf16)Ws;
        dh[i] = hd;
        dl[i] = (__bf16)(Wd - (float)hd);
        sh[i] = hs;
        sl[i] = (__bf16)(Ws - (float)hs);
        // W^T stage [k local][g]
        const int kl = 8 * kg + i;
        wt[0 * 512 + kl * 16 + row] = dh[i];
        wt[1 * 512 + kl * 16 + row] = dl[i];
        wt[2 * 512 + kl * 16 + row] = sh[i];
        wt[3 * 512 + kl * 16 + row] = sl[i];
      }
      const bf16x8 b = btab_load(bt, K, row, kb);
      accD = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dh, b, accD, 0, 0, 0);
      accD = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dl, b, accD, 0, 0, 0);
      accS = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sh, b, accS, 0, 0, 0);
      accS = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sl, b, accS, 0, 0, 0);
      wave_fence();
      // environment: A = W^T [32 k][16 g]; lane holds k = lane % 32, g = 8 (lane / 32) + i
      const int kr = lane & 31, gq = 8 * (lane >> 5);
      const bf16x8 adh = *reinterpret_cast<const bf16x8*>(wt + 0 * 512 + kr * 16 + gq);
      const bf16x8 adl = *reinterpret_cast<const bf16x8*>(wt + 1 * 512 + kr * 16 + gq);
      const bf16x8 ash = *reinterpret_cast<const bf16x8*>(wt + 2 * 512 + kr * 16 + gq);
      const bf16x8 asl = *reinterpret_cast<const bf16x8*>(wt + 3 * 512 + kr * 16 + gq);
      f32x16 de;
#pragma unroll
      for (int i = 0; i < 16; ++i) de[i] = 0.f;
      de = __builtin_amdgcn_mfma_f32_32x32x16_bf16(adh, bqd, de, 0, 0, 0);
      de = __builtin_amdgcn_mfma_f32_32x32x16_bf16(adl, bqd, de, 0, 0, 0);
      de = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ash, bqs, de, 0, 0, 0);
      de = __builtin_amdgcn_mfma_f32_32x32x16_bf16(asl, bqs, de, 0, 0, 0);
      // D[k][col]: lane holds col = lane % 32, rows 8 (i / 4) + 4 (lane / 32) + i % 4
      const int col = lane & 31;
      if (col < 6) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int kk = k0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
          atomicAdd(&denv_lds[3 * kk + (col % 3)], de[i]);
        }
      }
      wave_fence();
    }
    // per-Gaussian sums from the forward-style MFMA: D[row 4 kg + i][col]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      stage[(4 * kg + i) * 16 + row] = accD[i];
      stage[256 + (4 * kg + i) * 16 + row] = accS[i];
    }
    // VALU partial sums of the four lanes of each Gaussian row
    float r8[8] = {acc.gn[0], acc.gn[1], acc.gn[2], acc.gw[0], acc.gw[1], acc.gw[2], acc.gco, acc.gga};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      r8[q] += __shfl_xor(r8[q], 16, 64);
      r8[q] += __shfl_xor(r8[q], 32, 64);
    }
    wave_fence();
    if (kg == 0 && have) {
      if (!G.front) {
        for (int c = 0; c < 3; ++c) {
          dn[(size_t)c * n + g] = 0.f;
          dalbedo[(size_t)c * n + g] = 0.f;
        }
        drough[g] = 0.f;
        dtint[g] = 0.f;
      } else {
        const float gco = r8[6];
        float gn3[3] = {r8[0] + gco * G.wo[0], r8[1] + gco * G.wo[1], r8[2] + gco * G.wo[2]};
        float gw[3] = {r8[3] + gco * G.nn[0], r8[4] + gco * G.nn[1], r8[5] + gco * G.nn[2]};
        const float pn = gn3[0] * G.nn[0] + gn3[1] * G.nn[1] + gn3[2] * G.nn[2];
        const float pw = gw[0] * G.wo[0] + gw[1] * G.wo[1] + gw[2] * G.wo[2];
        float ts = 0.f;
        for (int c = 0; c < 3; ++c) {
          const float sd = stage[row * 16 + c] + stage[row * 16 + 3 + c];
          const float ss = stage[256 + row * 16 + c] + stage[256 + row * 16 + 3 + c];
          dn[(size_t)c * n + g] = (gn3[c] - G.nn[c] * pn) * G.inn;
          dx[(size_t)c * n + g] += -(gw[c] - G.wo[c] * pw) * G.iwo;
          dalbedo[(size_t)c * n + g] = dLo[c] * sd * (1.f / kPi);
          ts = fmaf(dLo[c], ss, ts);
        }
        drough[g] = r8[7];
        dtint[g] = ts;
      }
    }
    wave_fence();
  }
  __syncthreads();
  // LDS sums are in slot order; the partials in texel order
  float* out = denv_part + (size_t)blockIdx.x * 3 * K;
  for (int i = threadIdx.x; i < 3 * K; i += blockDim.x) {
    const int sl = i / 3, c = i - 3 * sl;
    out[3 * slot_k(sl, a.we, a.patch) + c] = denv_lds[i];
  }
}

// With TAPE the live pairs of each Gaussian are read from the forward's tape,
// in the order and 64-pair groups the walk would produce them (so the sums are
// the same), instead of testing every direction: no count rows, no ring.  (At
// most 128 VGPRs: four waves per SIMD.)
template <int NQ, bool TAPE, int WAVES>
__global__ void __launch_bounds__(WAVES * 64, TAPE || NQ <= 2 ? 4 : 2)
shade_bwd_kernel(ShadeArgs a, int cap, const float* __restrict__ color,
                 const float* __restrict__ dcolor, float* __restrict__ dx, float* __restrict__ dn,
                 float* __restrict__ dalbedo, float* __restrict__ drough,
                 float* __restrict__ dtint, float* __restrict__ denv_part /*[grid][K][3]*/) {
  extern __shared__ __align__(16) float smem[];
  __shared__ int ctl[2][2];   // entries listed and taken, of alternate rounds
  const int K = a.K, n = a.n, V = a.V;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const Lds<WAVES> L = lds_of<WAVES>(smem, 11 * K, V, wave, !TAPE);
  const float* tab = L.tab;
  float* denv_lds = smem + 8 * K;
  if (threadIdx.x < 4) (&ctl[0][0])[threadIdx.x] = 0;
  build_table(a, smem);
  for (int i = threadIdx.x; i < 3 * K; i += blockDim.x) denv_lds[i] = 0.f;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  RowPlan<NQ> plan;
  row_plan<NQ>(V, lane, plan);
  const float* pattr = attr_lane(a, lane);
  const Walk walk = group_walk(n);
  // Lane c < 3 handles channel c of the per-Gaussian inputs and outputs.
  const int ch = min(lane, 2);
  for (int m0 = 0, r = 0; m0 < walk.count; m0 += cap, r ^= 1) {
    __syncthreads();          // the last round's list is done with
    if (threadIdx.x < 2) ctl[r ^ 1][threadIdx.x] = 0;
    // a back-facing Gaussian gets zero gradients (dx, accumulated, is left as
    // it is)
    list_fill(a, walk, m0, cap, L.list, &ctl[r][0], lt, [&](int g, bool f) {
      if (f) return;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        dn[(size_t)c * n + g] = 0.f;
        dalbedo[(size_t)c * n + g] = 0.f;
      }
      drough[g] = 0.f;
      dtint[g] = 0.f;
    });
    __syncthreads();
    const int entries = ctl[r][0];
    int t = list_take(&ctl[r][1], lane);
    Rows<NQ> R;
    int g = 0;
    float v = 0.f;
    // TAPE: the Gaussian's live count and first 64 pairs (lane < K keeps
    // the read inside the Gaussian's row of the tape)
    int tl = 0;
    uint2 tw = make_uint2(0u, 0u);
    float pcol = 0.f, pdc = 0.f, pdx = 0.f;
    auto load = [&](int e, int& len, uint2& w) {
      const int4 le = L.list[e];
      const int gg = uni(le.x);
      v = pattr[gg];
      if constexpr (TAPE) {
        len = a.tape_n[gg];
        if (lane < K) w = a.tape[(size_t)gg * K + lane];
      } else {
        const int vidx[3] = {uni(le.y), uni(le.z), uni(le.w)};
        rows_load(a, plan, vidx, R);
      }
      pcol = color[(size_t)ch * n + gg];
      pdc = dcolor[(size_t)ch * n + gg];
      pdx = dx[(size_t)ch * n + gg];
      return gg;
    };
    if (t < entries) {
      g = load(t, tl, tw);
      if constexpr (!TAPE) rows_store(plan, R, L.rows, lane);
    }
    while (t < entries) {
      const float col = pcol, dcol = pdc, dx_in = pdx;
      Attr A;
      attr_read(v, A);
      t = list_take(&ctl[r][1], lane);
      int gn = 0;
      int tln = 0;
      uint2 twn = make_uint2(0u, 0u);
      if (t < entries) gn = load(t, tln, twn);
      wave_fence();
      GaussCtx G;
      gauss_setup(a, A, L.rows, G);
      // dL/dL_o: lane c < 3 takes channel c, every lane reads the three
      float dLo[3], aop[3], qd[3];
      {
        const float d = srgb_adjoint(col, dcol);
#pragma unroll
        for (int q = 0; q < 3; ++q)
          dLo[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(d), q));
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        aop[c] = A.alb[c] * (1.f / kPi);
        qd[c] = dLo[c] * aop[c];
      }
      const float tint = A.tint;
      BwdAcc acc = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, 0.f, 0.f, {0.f, 0.f, 0.f}, 0.f};
      if constexpr (TAPE) {
        // 64 pairs at a time, the next group's read issued before this one
        uint2 w = tw;
        for (int base = 0; base < tl; base += 64) {
          uint2 wn2 = make_uint2(0u, 0u);
          if (base + 64 < tl && base + 64 + lane < K) wn2 = a.tape[(size_t)g * K + base + 64 + lane];
          if (base + lane < tl)
            pair_bwd(G, tab, denv_lds, K, (int)w.x, __uint_as_float(w.y), qd, dLo, tint, aop, acc);
          w = wn2;
        }
      } else {
        live_walk(G, tab, K, V, L.qk, L.qv, lane, [&](int k, float v, bool on, int) {
          if (on) pair_bwd(G, tab, denv_lds, K, k, v, qd, dLo, tint, aop, acc);
        });
      }
      // per-Gaussian sums of the twelve partials over the wave: four slots
      // of three values (lane swaps and DPP), slot s summed in row s
      float r12[12];
      {
        float v4[4][3] = {{acc.gn[0], acc.gn[1], acc.gn[2]},
                          {acc.gw[0], acc.gw[1], acc.gw[2]},
                          {acc.gco, acc.gga, acc.ts},
                          {acc.sd[0], acc.sd[1], acc.sd[2]}};
        float o3[3];
        rga::slot_sums4<3>(v4, o3);
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
#pragma unroll
          for (int q = 0; q < 3; ++q)
            r12[3 * sl + q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(o3[q]), 16 * sl));
      }
      // r12: gn 0-2, gw 3-5, gco 6, gga 7, ts 8, sd 9-11
      {
        const float gco = r12[6];
        float gn3[3] = {r12[0] + gco * G.wo[0], r12[1] + gco * G.wo[1], r12[2] + gco * G.wo[2]};
        float gw[3] = {r12[3] + gco * G.nn[0], r12[4] + gco * G.nn[1], r12[5] + gco * G.nn[2]};
        const float pn = gn3[0] * G.nn[0] + gn3[1] * G.nn[1] + gn3[2] * G.nn[2];
        const float pw = gw[0] * G.wo[0] + gw[1] * G.wo[1] + gw[2] * G.wo[2];
        const int c = ch;
        const float gnc = c == 0 ? gn3[0] : (c == 1 ? gn3[1] : gn3[2]);
        const float gwc = c == 0 ? gw[0] : (c == 1 ? gw[1] : gw[2]);
        const float nnc = c == 0 ? G.nn[0] : (c == 1 ? G.nn[1] : G.nn[2]);
        const float woc = c == 0 ? G.wo[0] : (c == 1 ? G.wo[1] : G.wo[2]);
        const float dlc = c == 0 ? dLo[0] : (c == 1 ? dLo[1] : dLo[2]);
        const float sdc = c == 0 ? r12[9] : (c == 1 ? r12[10] : r12[11]);
        if (lane < 3) {
          dn[(size_t)lane * n + g] = (gnc - nnc * pn) * G.inn;
          // w_o = (cam - x)/|cam - x|: d/dx = -(I - w w^T)/|cam - x|
          dx[(size_t)lane * n + g] = dx_in - (gwc - woc * pw) * G.iwo;
          dalbedo[(size_t)lane * n + g] = dlc * sdc * (1.f / kPi);
        }
        if (lane == 0) {
          drough[g] = r12[7];
          dtint[g] = r12[8];
        }
      }
      wave_fence();
      if constexpr (!TAPE) {
        if (t < entries) rows_store(plan, R, L.rows, lane);
      }
      g = gn;
      tl = tln;
      tw = twn;
    }
  }
  __syncthreads();
  float* out = denv_part + (size_t)blockIdx.x * 3 * K;
  for (int i = threadIdx.x; i < 3 * K; i += blockDim.x) out[i] = denv_lds[i];
}

// denv[k][c] = area_k * sum over workgroups.  Each block owns 64 outputs;
// its 1024 threads split the partials into 16 interleaved groups and the
// groups are added in a fixed tree order (deterministic).
__global__ void __launch_bounds__(1024)
denv_reduce_kernel(int K, int he, int we, int parts, const float* __restrict__ part,
                   float* __restrict__ denv) {
  __shared__ float red[16][64];
  const int o = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + o;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  if (i < 3 * K) {
    int p = grp;
    for (; p + 48 < parts; p += 64) {
      s0 += part[(size_t)p * 3 * K + i];
      s1 += part[(size_t)(p + 16) * 3 * K + i];
      s2 += part[(size_t)(p + 32) * 3 * K + i];
      s3 += part[(size_t)(p + 48) * 3 * K + i];
    }
    for (; p < parts; p += 16) s0 += part[(size_t)p * 3 * K + i];
  }
  red[grp][o] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  for (int h = 8; h > 0; h >>= 1) {
    if (grp < h) red[grp][o] += red[grp + h][o];
    __syncthreads();
  }
  if (grp == 0 && i < 3 * K) {
    const int k = i / 3, r = k / we;
    const float dth = kPi / (float)he;
    const float area = (2.f * kPi / (float)we) * 2.f * sinf(0.5f * dth) * sinf(((float)r + 0.5f) * dth);
    denv[i] = red[0][o] * area;
  }
}

constexpr size_t kLdsMax = 160 * 1024;
constexpr size_t kLdsStatic = 64;    // the kernels' counters

// What the FP32 kernels accept: the direction table (8 K floats; the adjoint
// adds 3 K for the environment gradient) and two sets of count rows for each of
// eight waves in 152 KB (with a tape: the table and the environment sums).
inline size_t fp32_need(int K, int V, bool adjoint, bool taped) {
  return (size_t)(adjoint ? 11 : 8) * K * sizeof(float) + (taped ? 0 : (size_t)48 * V);
}

// LDS of a kernel of `waves` waves without its list
inline size_t fp32_lds(int K, int V, bool adjoint, bool taped, int waves) {
  return (size_t)(adjoint ? 11 : 8) * K * sizeof(float) +
         (taped ? 0 : (size_t)waves * (3 * (size_t)V + 8 * kRing));
}

template <int NQ, int WAVES>
const void* fp32_kernel_of(bool adjoint, bool taped) {
  // (the adjoint that reads a tape copies no rows: one instance serves every
  // view count)
  if (adjoint && taped) return reinterpret_cast<const void*>(shade_bwd_kernel<2, true, WAVES>);
  // (the adjoint without one keeps six pieces of rows in eight waves only: 128
  // registers of 16 do not hold them)
  if (adjoint) return reinterpret_cast<const void*>(shade_bwd_kernel<NQ, false, NQ <= 2 ? WAVES : 8>);
  return reinterpret_cast<const void*>(shade_fwd_kernel<NQ, WAVES>);
}

// texels per view along the azimuth that the MFMA kernels read in whole words
// (1 or 2), 0 for any other view grid
int view_ratio(int he, int we, int hv, int wv) {
  return (hv == he && we == wv) ? 1 : ((hv == he && we == 2 * wv && we % 8 == 0) ? 2 : 0);
}

// 4 x 8 texel patches where they divide the map
int patches(int he, int we) { return (he % 4 == 0 && we % 8 == 0) ? 1 : 0; }

// Whether the forward of a BF16X3 call runs on MFMA.  Three output channels
// leave the matrix units idle; what counts is the BRDF weights, which the MFMA
// kernel evaluates for whole patches of 16 Gaussians x 32 directions and the FP32
// kernel for the live pairs alone, after a walk and a set-up per Gaussian.  So few
// directions go to MFMA, in one or two texels per view, if there are Gaussians to
// fill the chip; 129 to 512, fewer Gaussians and other view grids to the FP32
// kernel.  MFMA -> FP32: 300k Gaussians 128 directions 56 -> 80 us, 256 102 -> 97;
// 100k 512 100 -> 57, in other view grids 237 -> 56; 30k 128 14 us both, 500 17 -> 9.
// The FP32 kernel then walks the same patches, so the tape is the same, and rounds
// the factors as MFMA takes them (3 us of the 57).  What differs is the order of the
// sums: a colour changes by up to 6e-7 of the colours' rms where the route does, so
// also from 32,767 Gaussians to 32,768 at 128 directions, and dx and dn, sums that
// cancel, by up to 1.4e-4 of theirs (1,200 Gaussians, 512 to 2048 directions).  Neither
// is nearer to FP64: errors in units of the rms, MFMA and the FP32 kernel, 512
// directions colour 3.9e-7 and 3.9e-7, dx 5.7e-6 and 5.7e-6, dn 6.0e-6 and 4.9e-6; 1024
// colour 2.8e-7 and 2.6e-7, dx 5.0e-6 and 4.8e-6, dn 6.5e-6 and 5.9e-6; 2048 colour
// 2.4e-7 and 2.0e-7, dx 1.40e-5 and 1.40e-5, dn 7.9e-6 and 8.2e-6.  So the line at 512
// is none of accuracy, nor of time (100k Gaussians, 2048 directions: 828 us on MFMA, 144
// on the FP32 kernel): up to there the form has moved to the FP32 kernel, beyond it runs
// on MFMA as it always has, and RGA_FP32 is the form to ask for.
bool forward_on_mfma(const ShadeArgs& a) {
  if (fp32_lds(a.K, a.V, false, false, 8) + 16 * 64 > kLdsMax - kLdsStatic || a.K > 512) return true;
  return a.K <= 128 && a.n >= 32768 && view_ratio(a.he, a.we, a.hv, a.wv) > 0;
}

struct Launch {
  const void* kernel;
  int waves, grid, cap;
  size_t lds;
};

// The FP32 kernel for these sizes and its launch.  A persistent grid, as many
// workgroups as the device holds at once (from the occupancy of the exact
// kernel at its LDS size), never more than one wave per Gaussian; beside other
// work half as many, where two or more fit a CU: a full grid leaves the other
// stream's short kernels no wave slots until it ends (100k Gaussians, 512
// directions beside their binning, training step 381 -> 366 us; alone the forward
// would take 61 us instead of 55).  Frames and training steps of 20k to 300k Gaussians,
// 128, 512 and 2048 directions, 128^2 to 1080^2 take 0.91 to 1.00 times as long with
// the half as with the whole; 1.01 to 1.03 times where the two streams were given one
// hardware queue, so that nothing overlaps (one pair in four).
Launch fp32_launch(int n, int K, int V, bool adjoint, bool taped, bool beside) {
  Launch l;
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
    ncu = 256;
  const bool small = 3 * V <= 2048;      // pieces of 1024 bytes of three count rows: at most 2
  const size_t room = kLdsMax - kLdsStatic;
  // Sixteen waves share one table where the LDS holds their rows and a list, so
  // that four waves per SIMD are resident up to 2048 directions and 1024 views
  // (eight -> sixteen, forward: 200k Gaussians there 491 -> 294 us, 100k at 512
  // directions 57 -> 53 us, 10k 18 -> 17 us); below one Gaussian per wave of
  // such workgroups on every CU, eight spread over more CUs.
  l.waves = n > 16 * ncu && fp32_lds(K, V, adjoint, taped, 16) + 16 * 256 <= room &&
                    !(adjoint && !taped && !small) ? 16 : 8;
  if (l.waves == 16)
    l.kernel = small ? fp32_kernel_of<2, 16>(adjoint, taped) : fp32_kernel_of<6, 16>(adjoint, taped);
  else
    l.kernel = small ? fp32_kernel_of<2, 8>(adjoint, taped) : fp32_kernel_of<6, 8>(adjoint, taped);
  const size_t base = fp32_lds(K, V, adjoint, taped, l.waves);
  const size_t least = base + std::min<size_t>(16 * 128, room - base);
  if (2 * least > kLdsMax)   // (the attribute is kept per device)
    hipFuncSetAttribute(l.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)room);
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, l.kernel, 64 * l.waves, least) !=
          hipSuccess || per_cu < 1)
    per_cu = 1;
  // the longest list, up to 1024 entries, that leaves room for as many
  // workgroups (LDS is given in steps of 1280 bytes)
  const size_t share = kLdsMax / 1280 / per_cu * 1280 - kLdsStatic;
  l.cap = (int)(std::min<size_t>(share > least ? share - base : least - base, 16 * 1024) / 16);
  l.lds = base + 16 * (size_t)l.cap;
  const int groups = ncu * (beside && per_cu > 1 ? per_cu / 2 : per_cu);
  l.grid = std::max(1, std::min(groups, (int)rga::ceil_div(n, l.waves)));
  return l;
}

int check_args(const char* fn, int n, const float* x, const float* nrm, const float* albedo,
               const float* rough, const float* tint, const int32_t* vidx, const float* vw,
               const uint8_t* count, int nv, int kv, int he, int we, int hv, int wv,
               const float* env, const float* cam_pos, int precision) {
  if (n < 0) return rga::fail(RGA_EINVAL, "%s: n < 0", fn);
  if (he < 1 || we < 1 || hv < 1 || wv < 1 || he % hv || we % wv)
    return rga::fail(RGA_EINVAL, "%s: view grid %dx%d must divide the map %dx%d", fn, hv, wv, he, we);
  if ((int64_t)he * we > 3584)
    return rga::fail(RGA_EUNSUPPORTED, "%s: at most 3584 light directions (LDS table)", fn);
  if (nv < 1 || kv < 1) return rga::fail(RGA_EINVAL, "%s: nv, kv >= 1", fn);
  if ((hv * wv) % 16 != 0 || hv * wv > 2048)
    return rga::fail(RGA_EUNSUPPORTED, "%s: the view count must be a multiple of 16, at most 2048", fn);
  if (count && !rga::aligned16(count))
    return rga::fail(RGA_EINVAL, "%s: count must be 16-byte aligned", fn);
  if (!cam_pos || !env) return rga::fail(RGA_EINVAL, "%s: null env or cam_pos", fn);
  if (precision != RGA_FP32 && precision != RGA_BF16X3)
    return rga::fail(RGA_EINVAL, "%s: unknown precision %d", fn, precision);
  if (n > 0 && (!x || !nrm || !albedo || !rough || !tint || !vidx || !vw || !count))
    return rga::fail(RGA_EINVAL, "%s: null input", fn);
  return RGA_OK;
}

ShadeArgs make_args(int n, const float* x, const float* nrm, const float* albedo,
                    const float* rough, const float* tint, const int32_t* vidx, const float* vw,
                    const uint8_t* count, int nv, int kv, int he, int we, int hv, int wv,
                    const float* env, const float* cam_pos) {
  ShadeArgs a;
  a.n = n;
  a.nv = nv;
  a.V = hv * wv;
  a.kv = kv;
  a.he = he;
  a.we = we;
  a.hv = hv;
  a.wv = wv;
  a.K = he * we;
  for (int i = 0; i < 3; ++i) a.cam[i] = cam_pos[i];
  a.x = x;
  a.nrm = nrm;
  a.albedo = albedo;
  a.rough = rough;
  a.tint = tint;
  a.vw = vw;
  a.env = env;
  a.vidx = vidx;
  a.count = count;
  a.patch = 0;
  a.split = 0;
  a.tape_n = nullptr;
  a.tape = nullptr;
  return a;
}

}  // namespace

// The live-pair tape: [n] int32 counts (256-byte aligned block), then
// [n][K] (direction, visibility bits) pairs.
extern "C" size_t shade_tape_bytes(int n, int he, int we) {
  if (n < 0 || he < 1 || we < 1) return 0;
  return rga::align_up((size_t)4 * (n > 0 ? n : 1), 256) + (size_t)8 * n * he * we;
}

namespace {
int attach_tape(const char* fn, ShadeArgs& a, const void* tape, size_t tape_bytes) {
  if (!tape) return RGA_OK;
  if (!rga::aligned16(tape)) return rga::fail(RGA_EINVAL, "%s: tape must be 16-byte aligned", fn);
  if (tape_bytes < shade_tape_bytes(a.n, a.he, a.we))
    return rga::fail(RGA_ECAPACITY, "%s: tape %zu < %zu bytes", fn, tape_bytes,
                     shade_tape_bytes(a.n, a.he, a.we));
  char* t = static_cast<char*>(const_cast<void*>(tape));
  a.tape_n = reinterpret_cast<int32_t*>(t);
  a.tape = reinterpret_cast<uint2*>(t + rga::align_up((size_t)4 * (a.n > 0 ? a.n : 1), 256));
  return RGA_OK;
}
}  // namespace

namespace {

int shade_forward(bool beside, void* stream, int n, const float* x, const float* nrm, const
                  float* albedo, const float* rough, const float* tint, const int32_t* vidx,
                  const float* vw, const uint8_t* count, int nv, int kv, int he, int we, int hv,
                  int wv, const float* env, const float* cam_pos, int precision, float* color,
                  uint8_t* front, void* tape, size_t tape_bytes) {
  int rc = check_args("shade_gaussians", n, x, nrm, albedo, rough, tint, vidx, vw, count, nv, kv,
                      he, we, hv, wv, env, cam_pos, precision);
  if (rc) return rc;
  if (n == 0) return RGA_OK;
  if (!color || !front) return rga::fail(RGA_EINVAL, "shade_gaussians: null output");
  ShadeArgs a = make_args(n, x, nrm, albedo, rough, tint, vidx, vw, count, nv, kv, he, we, hv, wv,
                          env, cam_pos);
  rc = attach_tape("shade_gaussians", a, tape, tape_bytes);
  if (rc) return rc;
  if (precision == RGA_BF16X3) {
    if (a.K % 32 != 0)
      return rga::fail(RGA_EUNSUPPORTED, "shade_gaussians: BF16X3 needs a multiple of 32 directions");
    const size_t lds = (size_t)8 * a.K * sizeof(float) + (size_t)6 * a.K * 2 + kMWaves * 512 * 4;
    if (lds > 150 * 1024) return rga::fail(RGA_EUNSUPPORTED, "shade_gaussians: too many directions");
  }
  if (precision == RGA_BF16X3) {
    a.patch = patches(he, we);
    a.split = !forward_on_mfma(a);
  }
  if (precision == RGA_BF16X3 && !a.split) {
    const int ratio = view_ratio(he, we, hv, wv);
    const size_t lds = (size_t)8 * a.K * sizeof(float) + (size_t)6 * a.K * 2 + kMWaves * 512 * 4;
    static bool mattr = false;
    if (!mattr) {
      hipFuncSetAttribute(reinterpret_cast<const void*>(shade_fwd_mfma_kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
      mattr = true;
    }
    int ncu = 0, dev = 0;
    hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
      ncu = 256;
    const int per_cu = lds <= 40 * 1024 ? 4 : (lds <= 76 * 1024 ? 2 : 1);
    const int tiles = (int)rga::ceil_div(n, 16);
    int grid = ncu * per_cu;
    const int need = (int)rga::ceil_div(tiles, kMWaves);
    if (grid > need) grid = need;
    hipStream_t s = static_cast<hipStream_t>(stream);
    RGA_LAUNCH("shade_fwd_bf16x3", shade_fwd_mfma_kernel, dim3(grid), dim3(kMThreads), lds, s, a,
               ratio, color, front);
    RGA_CHECK_LAUNCH("shade_gaussians");
    return RGA_OK;
  }
  const size_t need = fp32_need(a.K, a.V, false, false);
  if (precision == RGA_FP32 && need > 152 * 1024)
    return rga::fail(RGA_EUNSUPPORTED, "shade_gaussians: %d directions and %d views need %zu B of LDS",
                     a.K, a.V, need);
  hipStream_t s = static_cast<hipStream_t>(stream);
  Launch l = fp32_launch(n, a.K, a.V, false, false, beside);
  {
    rga::TimedLaunch tl("shade_fwd", s);
    void* args[] = {&a, &l.cap, &color, &front};
    if (hipLaunchKernel(l.kernel, dim3(l.grid), dim3(64 * l.waves), args, l.lds, s) != hipSuccess)
      return rga::fail(RGA_EHIP, "shade_gaussians: launch failed");
  }
  RGA_CHECK_LAUNCH("shade_gaussians");
  return RGA_OK;
}

}  // namespace

extern "C" int shade_gaussians(void* stream, int n, const float* x, const float* nrm, const
                               float* albedo, const float* rough, const float* tint, const
                               int32_t* vidx, const float* vw, const uint8_t* count, int nv, int
                               kv, int he, int we, int hv, int wv, const float* env, const
                               float* cam_pos, int precision, float* color, uint8_t* front,
                               void* tape, size_t tape_bytes) {
  return shade_forward(false, stream, n, x, nrm, albedo, rough, tint, vidx, vw, count, nv, kv,
                         he, we, hv, wv, env, cam_pos, precision, color, front, tape,
                         tape_bytes);
}

extern "C" int shade_gaussians_beside(void* stream, int n, const float* x, const float* nrm,
                                      const float* albedo, const float* rough, const float*
                                      tint, const int32_t* vidx, const float* vw, const uint8_t*
                                      count, int nv, int kv, int he, int we, int hv, int wv,
                                      const float* env, const float* cam_pos, int precision,
                                      float* color, uint8_t* front, void* tape, size_t
                                      tape_bytes) {
  return shade_forward(true, stream, n, x, nrm, albedo, rough, tint, vidx, vw, count, nv, kv,
                         he, we, hv, wv, env, cam_pos, precision, color, front, tape,
                         tape_bytes);
}

extern "C" size_t shade_gaussians_workspace(int n, int he, int we) {
  if (n < 0 || he < 1 || we < 1) return 0;
  const size_t K = (size_t)he * we;
  // at most 4 workgroups per CU on up to 512 CUs
  return 4 * 512 * 3 * K * sizeof(float);
}

extern "C" int shade_gaussians_backward(void* stream, int n, const float* x, const float* nrm,
                                        const float* albedo, const float* rough, const float* tint,
                                        const int32_t* vidx, const float* vw, const uint8_t* count,
                                        int nv, int kv, int he, int we, int hv, int wv,
                                        const float* env, const float* cam_pos, int precision,
                                        const float* color, const uint8_t* front,
                                        const float* dcolor, float* dx, float* dn,
                                        float* dalbedo, float* drough, float* dtint, float* denv,
                                        void* ws, size_t ws_bytes, const void* tape,
                                        size_t tape_bytes) {
  (void)front;
  int rc = check_args("shade_gaussians_backward", n, x, nrm, albedo, rough, tint, vidx, vw, count,
                      nv, kv, he, we, hv, wv, env, cam_pos, precision);
  if (rc) return rc;
  if (!denv) return rga::fail(RGA_EINVAL, "shade_gaussians_backward: null denv");
  if (n > 0 && (!color || !dcolor || !dx || !dn || !dalbedo || !drough || !dtint))
    return rga::fail(RGA_EINVAL, "shade_gaussians_backward: null pointer");
  ShadeArgs a = make_args(n, x, nrm, albedo, rough, tint, vidx, vw, count, nv, kv, he, we, hv, wv,
                          env, cam_pos);
  rc = attach_tape("shade_gaussians_backward", a, tape, tape_bytes);
  if (rc) return rc;
  // given a tape (of either form's forward), the adjoint replays its live
  // pairs in FP32; the MFMA adjoint is the BF16X3 form's without one
  if (precision == RGA_BF16X3 && !a.tape) {
    if (a.K % 32 != 0)
      return rga::fail(RGA_EUNSUPPORTED, "shade_gaussians_backward: BF16X3 needs a multiple of 32 directions");
    const size_t lds = (size_t)11 * a.K * sizeof(float) + (size_t)6 * a.K * 2 +
                       (size_t)kMWaves * (4096 + 384 + 2048);
    if (lds > 150 * 1024)
      return rga::fail(RGA_EUNSUPPORTED, "shade_gaussians_backward: too many directions");
    const int ratio = view_ratio(he, we, hv, wv);
    a.patch = patches(he, we);
    static bool mattr = false;
    if (!mattr) {
      hipFuncSetAttribute(reinterpret_cast<const void*>(shade_bwd_mfma_kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
      mattr = true;
    }
    int ncu = 0, dev = 0;
    hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
      ncu = 256;
    const int per_cu = lds <= 40 * 1024 ? 4 : (lds <= 76 * 1024 ? 2 : 1);
    int grid = ncu * per_cu;
    const int need = (int)rga::ceil_div(rga::ceil_div(n, 16), kMWaves);
    if (grid > need) grid = need;
    if (grid < 1) grid = 1;
    if (!ws || ws_bytes < (size_t)grid * 3 * a.K * sizeof(float))
      return rga::fail(RGA_ECAPACITY, "shade_gaussians_backward: workspace too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    float* part = static_cast<float*>(ws);
    if (n > 0)
      RGA_LAUNCH("shade_bwd_bf16x3", shade_bwd_mfma_kernel, dim3(grid), dim3(kMThreads), lds, s, a,
                 ratio, color, dcolor, dx, dn, dalbedo, drough, dtint, part);
    RGA_LAUNCH("shade_denv", denv_reduce_kernel, dim3(rga::ceil_div(3 * a.K, 64)), dim3(1024), 0, s,
               a.K, he, we, n > 0 ? grid : 0, part, denv);
    RGA_CHECK_LAUNCH("shade_gaussians_backward");
    return RGA_OK;
  }
  const bool taped = a.tape != nullptr;
  const size_t need = fp32_need(a.K, a.V, true, taped);
  if (need > 152 * 1024)
    return rga::fail(RGA_EUNSUPPORTED,
                     "shade_gaussians_backward: %d directions and %d views need %zu B of LDS", a.K,
                     a.V, need);
  Launch l = fp32_launch(n, a.K, a.V, true, taped, false);
  const int grid = l.grid;
  if (!ws || ws_bytes < (size_t)grid * 3 * a.K * sizeof(float))
    return rga::fail(RGA_ECAPACITY, "shade_gaussians_backward: workspace too small");
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* part = static_cast<float*>(ws);
  if (n > 0) {
    rga::TimedLaunch tl("shade_bwd", s);
    void* args[] = {&a, &l.cap, &color, &dcolor, &dx, &dn, &dalbedo, &drough, &dtint, &part};
    if (hipLaunchKernel(l.kernel, dim3(grid), dim3(64 * l.waves), args, l.lds, s) != hipSuccess)
      return rga::fail(RGA_EHIP, "shade_gaussians_backward: launch failed");
  }
  RGA_LAUNCH("shade_denv", denv_reduce_kernel, dim3(rga::ceil_div(3 * a.K, 64)), dim3(1024), 0, s,
             a.K, he, we, n > 0 ? grid : 0, part, denv);
  RGA_CHECK_LAUNCH("shade_gaussians_backward");
  return RGA_OK;
}
