// Forward linear blend skinning and its adjoint (Sec. 3.1, deformation).
//
// One thread per point; the joint table ([J][3][4], <= 12 KB) is staged in
// LDS once per workgroup, SoA planes are read and written fully coalesced.
// HBM-bound: 72 B in, 60 B out per point with normal and A.
#include "common.h"

namespace {

constexpr int kMaxJoints = 256;
constexpr int kBlock = 256;

__global__ void __launch_bounds__(kBlock)
lbs_fwd_kernel(int n, int J, const float* __restrict__ skin, const int32_t* __restrict__ jidx,
               const float* __restrict__ jw, const float* __restrict__ x,
               const float* __restrict__ disp, const float* __restrict__ nrm,
               float* __restrict__ x_out, float* __restrict__ n_out, float* __restrict__ A_out) {
  __shared__ float S[kMaxJoints * 12];
  for (int k = threadIdx.x; k < J * 12; k += blockDim.x) S[k] = skin[k];
  __syncthreads();
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  // the optional displacement is added first (x + dx rounded to FP32)
  const float p0 = disp ? x[i] + disp[i] : x[i];
  const float p1 = disp ? x[n + i] + disp[n + i] : x[n + i];
  const float p2 = disp ? x[2 * n + i] + disp[2 * n + i] : x[2 * n + i];
  float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f;
  float Aa[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float w = jw[j * n + i];
    const float* Sj = S + 12 * rga::clampi(jidx[j * n + i], 0, J - 1);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float d0 = Sj[4 * a + 0] - (a == 0 ? 1.f : 0.f);
      const float d1 = Sj[4 * a + 1] - (a == 1 ? 1.f : 0.f);
      const float d2 = Sj[4 * a + 2] - (a == 2 ? 1.f : 0.f);
      const float pa = fmaf(d2, p2, fmaf(d1, p1, fmaf(d0, p0, Sj[4 * a + 3])));
      if (a == 0) acc0 = fmaf(w, pa, acc0);
      if (a == 1) acc1 = fmaf(w, pa, acc1);
      if (a == 2) acc2 = fmaf(w, pa, acc2);
      Aa[3 * a + 0] = fmaf(w, d0, Aa[3 * a + 0]);
      Aa[3 * a + 1] = fmaf(w, d1, Aa[3 * a + 1]);
      Aa[3 * a + 2] = fmaf(w, d2, Aa[3 * a + 2]);
    }
  }
  x_out[i] = p0 + acc0;
  x_out[n + i] = p1 + acc1;
  x_out[2 * n + i] = p2 + acc2;
  float A[9];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) A[3 * a + b] = (a == b ? 1.f : 0.f) + Aa[3 * a + b];
  if (A_out) {
#pragma unroll
    for (int k = 0; k < 9; ++k) A_out[k * n + i] = A[k];
  }
  if (nrm && n_out) {
    const float m0 = nrm[i], m1 = nrm[n + i], m2 = nrm[2 * n + i];
#pragma unroll
    for (int a = 0; a < 3; ++a)
      n_out[a * n + i] = fmaf(A[3 * a + 2], m2, fmaf(A[3 * a + 1], m1, A[3 * a + 0] * m0));
  }
}

__global__ void __launch_bounds__(kBlock)
lbs_bwd_kernel(int n, int J, const float* __restrict__ skin, const int32_t* __restrict__ jidx,
               const float* __restrict__ jw, const float* __restrict__ dx_out,
               const float* __restrict__ dn_out, float* __restrict__ dx, float* __restrict__ dn) {
  __shared__ float S[kMaxJoints * 12];
  for (int k = threadIdx.x; k < J * 12; k += blockDim.x) S[k] = skin[k];
  __syncthreads();
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float A[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float w = jw[j * n + i];
    const float* Sj = S + 12 * rga::clampi(jidx[j * n + i], 0, J - 1);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) A[3 * a + b] = fmaf(w, Sj[4 * a + b] - (a == b ? 1.f : 0.f), A[3 * a + b]);
  }
  const float g0 = dx_out[i], g1 = dx_out[n + i], g2 = dx_out[2 * n + i];
#pragma unroll
  for (int b = 0; b < 3; ++b) dx[b * n + i] = fmaf(A[6 + b], g2, fmaf(A[3 + b], g1, A[b] * g0));
  if (dn_out && dn) {
    const float h0 = dn_out[i], h1 = dn_out[n + i], h2 = dn_out[2 * n + i];
#pragma unroll
    for (int b = 0; b < 3; ++b) dn[b * n + i] = fmaf(A[6 + b], h2, fmaf(A[3 + b], h1, A[b] * h0));
  }
}

}  // namespace

namespace {

// Pose gradient: dS_j[r][c] = sum_i w_ij (dx'_i[r] (x_i, 1)[c] + dn'_i[r] (n_i, 0)[c]
// + dA_i[r][c] for c < 3), w_ij the summed weights of joint j in Gaussian i's
// slots.  A wave owns two Gaussians per lane: the twelve factors of each, which
// all of its joints share, stay in registers, and the wave takes the distinct
// joints of its 512 slots one after the other (Gaussians that are neighbours
// share them) and adds each joint's wave sum into its own LDS row.  The waves'
// rows, then the workgroups' rows, are added in a fixed order (no atomics).
// A workgroup adds up the joints [per blockIdx.y, + per) of its chunk.
// Every input is read once: with a workgroup per joint and chunk that read all
// indices and skipped the other joints', 100k Gaussians and 24 joints took
// 33 us and the sum over the chunks 12 us, now 9 and 4 us.
constexpr int kPoseWaves = 4;
constexpr int kPoseLane = 2;                                   // Gaussians per lane
constexpr int kPoseChunk = kPoseWaves * 64 * kPoseLane;        // per workgroup

__global__ void __launch_bounds__(kPoseWaves * 64)
lbs_pose_grad_kernel(int n, int n_joints, int per, const int32_t* __restrict__ jidx, const float* __restrict__ jw,
                     const float* __restrict__ x, const float* __restrict__ disp,
                     const float* __restrict__ nrm, const float* __restrict__ dxo,
                     const float* __restrict__ dno, const float* __restrict__ dA,
                     float* __restrict__ part) {
  extern __shared__ float rows[];                              // [wave][joint][12]
  const int j0 = blockIdx.y * per, J = min(per, n_joints - j0);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int k = threadIdx.x; k < kPoseWaves * J * 12; k += blockDim.x) rows[k] = 0.f;
  __syncthreads();
  float* row = rows + wave * J * 12;
  const int i0 = blockIdx.x * kPoseChunk + wave * 64 * kPoseLane + lane;
  float M[kPoseLane][12], w[kPoseLane][4];
  int id[kPoseLane][4];
#pragma unroll
  for (int k = 0; k < kPoseLane; ++k) {
    const int i = i0 + 64 * k;
    const bool have = i < n;
    const size_t c = have ? i : 0;
    // (slots that add nothing: no weight, or no such joint)
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      id[k][sl] = jidx[(size_t)sl * n + c] - j0;
      w[k][sl] = jw[(size_t)sl * n + c];
    }
#pragma unroll
    for (int sl = 0; sl < 4; ++sl)
      if (!have || w[k][sl] == 0.f || id[k][sl] < 0 || id[k][sl] >= J) id[k][sl] = -1;
    float xv[3], g[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      xv[q] = x[(size_t)q * n + c];
      if (disp) xv[q] += disp[(size_t)q * n + c];
      g[q] = dxo[(size_t)q * n + c];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
      for (int q = 0; q < 3; ++q) M[k][4 * r + q] = g[r] * xv[q];
      M[k][4 * r + 3] = g[r];
    }
    if (dA)
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) M[k][4 * r + q] += dA[(size_t)(3 * r + q) * n + c];
    if (dno)
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          M[k][4 * r + q] = fmaf(dno[(size_t)r * n + c], nrm[(size_t)q * n + c], M[k][4 * r + q]);
  }
  for (;;) {
    // the next joint: that of the first lane with a slot left
    int mine = -1;
#pragma unroll
    for (int k = 0; k < kPoseLane; ++k)
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) mine = max(mine, id[k][sl]);
    const uint64_t left = __ballot(mine >= 0);
    if (left == 0ull) break;
    const int j = __builtin_amdgcn_readlane(mine, __builtin_ctzll(left));
    float v[4][3] = {};
#pragma unroll
    for (int k = 0; k < kPoseLane; ++k) {
      float wj = 0.f;
      bool has = false;
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        const bool hit = id[k][sl] == j;
        wj += hit ? w[k][sl] : 0.f;
        has |= hit;
        id[k][sl] = hit ? -1 : id[k][sl];
      }
      if (has) {
#pragma unroll
        for (int q = 0; q < 12; ++q) v[q / 3][q % 3] = fmaf(wj, M[k][q], v[q / 3][q % 3]);
      }
    }
    float o[3];
    rga::slot_sums4<3>(v, o);
    // row s of the wave holds values 3 s .. 3 s + 2
    if ((lane & 15) < 3) {
      const int q = lane & 15;
      row[12 * j + 3 * (lane >> 4) + q] = q == 0 ? o[0] : (q == 1 ? o[1] : o[2]);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < J * 12; k += blockDim.x) {
    float t = rows[k];
#pragma unroll
    for (int v = 1; v < kPoseWaves; ++v) t += rows[v * J * 12 + k];
    part[((size_t)blockIdx.x * n_joints + j0) * 12 + k] = t;
  }
}

// 64 values per workgroup; its 16 waves add every sixteenth chunk each.
__global__ void __launch_bounds__(1024)
lbs_pose_grad_final(int n_joints, int chunks, const float* __restrict__ part,
                    float* __restrict__ dskin) {
  __shared__ float red[16][64];
  const int o = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int t = blockIdx.x * 64 + o, count = 12 * n_joints;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  if (t < count) {
    const float* p = part + t;
    int c = grp;
    for (; c + 48 < chunks; c += 64) {
      s0 += p[(size_t)c * count];
      s1 += p[(size_t)(c + 16) * count];
      s2 += p[(size_t)(c + 32) * count];
      s3 += p[(size_t)(c + 48) * count];
    }
    for (; c < chunks; c += 16) s0 += p[(size_t)c * count];
  }
  red[grp][o] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  for (int h = 8; h > 0; h >>= 1) {
    if (grp < h) red[grp][o] += red[grp + h][o];
    __syncthreads();
  }
  if (grp == 0 && t < count) dskin[t] = red[0][o];
}

int pose_chunks(int n) { return (int)rga::ceil_div(n > 0 ? n : 1, kPoseChunk); }

}  // namespace

namespace {

// ---- pose -> skinning matrices (forward kinematics of the axis-angle pose)
// R_j = exp([theta_j]x) = I + a K + b K^2 (a = sin t / t, b = (1 - cos t) / t^2,
// series near t = 0), G_j = G_p R_j, P_j = P_p + G_p (J_j - J_p), a root
// (parent outside 0..j-1) has G = R, P = J; skin_j = [G_j | P_j - G_j J_j].
// One workgroup, a thread per joint (at most 256): the Rodrigues matrices, then
// the chain one depth of the tree at a time, its joints in parallel.  Bound by
// latency (one thread walked the joints in order: 24 joints of a body 14 us, the
// adjoint 34; now 7.5 and 10).
__device__ inline void rodrigues(const float* th, float* R, float& a, float& b, float& ap,
                                 float& bp) {
  const float t2 = fmaf(th[2], th[2], fmaf(th[1], th[1], th[0] * th[0]));
  const float t = sqrtf(t2);
  if (t2 < 1e-12f) {
    a = 1.f - t2 / 6.f;
    b = 0.5f - t2 / 24.f;
  } else {
    const float h = sinf(0.5f * t);      // 1 - cos t = 2 sin^2(t/2), no cancellation
    a = sinf(t) / t;
    b = 2.f * h * h / t2;
  }
  // (da/dt) / t and (db/dt) / t: Taylor series below t = 0.5 (the closed
  // forms cancel there), the closed forms above
  if (t2 < 0.25f) {
    ap = -1.f / 3.f + t2 * (1.f / 30.f + t2 * (-1.f / 840.f + t2 * (1.f / 45360.f)));
    bp = -1.f / 12.f + t2 * (1.f / 180.f + t2 * (-1.f / 6720.f + t2 * (1.f / 453600.f)));
  } else {
    const float sn = sinf(t), cs = cosf(t);
    ap = (t * cs - sn) / (t2 * t);
    bp = (t * sn - 2.f * (1.f - cs)) / (t2 * t2);
  }
  const float K[9] = {0.f, -th[2], th[1], th[2], 0.f, -th[0], -th[1], th[0], 0.f};
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) {
      float k2 = 0.f;
      for (int m = 0; m < 3; ++m) k2 = fmaf(K[3 * r + m], K[3 * m + c], k2);
      R[3 * r + c] = (r == c ? 1.f : 0.f) + a * K[3 * r + c] + b * k2;
    }
}

__device__ inline void mat3_mul(const float* A, const float* B, float* C) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float v = 0.f;
#pragma unroll
      for (int m = 0; m < 3; ++m) v = fmaf(A[3 * r + m], B[3 * m + c], v);
      C[3 * r + c] = v;
    }
}

__device__ inline int parent_of(const int32_t* parents, int j) {
  const int p = parents[j];
  return (p >= 0 && p < j) ? p : -1;
}

static_assert(kMaxJoints <= kBlock, "a thread per joint");

struct Chain {
  float G[kMaxJoints][9], P[kMaxJoints][3];
  float at[kMaxJoints][3];   // rest joints
  int parent[kMaxJoints];
  int jump[2][kMaxJoints];   // 512 times the way up to an ancestor, and that one + 1
  int deepest;
};

// This thread's joint: Rodrigues factors and matrix, the rest position and its offset
// from the parent's, G and P, parent and depth.
struct Joint {
  float a, b, ap, bp;
  float R[9], at[3], off[3], G[9], P[3];
  int p, depth;
};

// The depths take log2 J rounds, in which a joint jumps to its ancestor's ancestor, and
// a step of the chain reads its parent's G and P alone (one chain of 256 joints: 154 us
// where each joint walked up through its parents and a step read five tables, 133 where
// one thread walked all joints, now 60; the adjoint 264, 337 and 155).
__device__ inline void forward_chain(int J, const float* theta, const float* joints,
                                     const int32_t* parents, Chain& ch, Joint& t) {
  const int j = threadIdx.x;
  t.p = -1;
  t.depth = -1;
  if (j == 0) ch.deepest = 0;
  int mine = 0;
  if (j < J) {
    t.p = parent_of(parents, j);
    ch.parent[j] = t.p;
#pragma unroll
    for (int q = 0; q < 3; ++q) ch.at[j][q] = t.at[q] = joints[3 * j + q];
    rodrigues(theta + 3 * j, t.R, t.a, t.b, t.ap, t.bp);
    mine = t.p < 0 ? 0 : 512 + t.p + 1;
    ch.jump[0][j] = mine;
  }
  __syncthreads();
  if (t.p >= 0) {
#pragma unroll
    for (int q = 0; q < 3; ++q) t.off[q] = t.at[q] - ch.at[t.p][q];
  }
  for (int span = 1, from = 0; span < J; span *= 2, from ^= 1) {
    const int up = mine & 511;
    if (up > 0) mine += ch.jump[from][up - 1] - up;
    if (j < J) ch.jump[from ^ 1][j] = mine;
    __syncthreads();
  }
  if (j < J) {
    t.depth = mine >> 9;
    if (t.depth > 0) atomicMax(&ch.deepest, t.depth);
  }
  __syncthreads();
  const int deepest = ch.deepest;
  for (int d = 0; d <= deepest; ++d) {
    if (t.depth == d) {
      if (t.p < 0) {
#pragma unroll
        for (int q = 0; q < 9; ++q) t.G[q] = t.R[q];
#pragma unroll
        for (int q = 0; q < 3; ++q) t.P[q] = t.at[q];
      } else {
        float Gp[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) Gp[q] = ch.G[t.p][q];
        mat3_mul(Gp, t.R, t.G);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          float v = ch.P[t.p][r];
#pragma unroll
          for (int m = 0; m < 3; ++m) v = fmaf(Gp[3 * r + m], t.off[m], v);
          t.P[r] = v;
        }
      }
#pragma unroll
      for (int q = 0; q < 9; ++q) ch.G[j][q] = t.G[q];
#pragma unroll
      for (int q = 0; q < 3; ++q) ch.P[j][q] = t.P[q];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kBlock)
pose_skin_kernel(int J, const float* __restrict__ theta, const float* __restrict__ joints,
                 const int32_t* __restrict__ parents, float* __restrict__ skin) {
  __shared__ Chain ch;
  Joint t;
  forward_chain(J, theta, joints, parents, ch, t);
  const int j = threadIdx.x;
  if (j >= J) return;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    float v = t.P[r];
#pragma unroll
    for (int m = 0; m < 3; ++m) v = fmaf(-t.G[3 * r + m], t.at[m], v);
#pragma unroll
    for (int c = 0; c < 3; ++c) skin[12 * j + 4 * r + c] = t.G[3 * r + c];
    skin[12 * j + 4 * r + 3] = v;
  }
}

// Adjoint: dG_j = dS_j[:, :3] - dt_j J_j^T, dP_j = dt_j; from the deepest joints
// up dG_p += dG_j R_j^T + dP_j (J_j - J_p)^T, dP_p += dP_j (a joint adds its
// children's shares in descending order), dR_j = G_p^T dG_j (dR_j = dG_j at a
// root); then dtheta_j from dR_j through Rodrigues.
__global__ void __launch_bounds__(kBlock)
pose_skin_bwd_kernel(int J, const float* __restrict__ theta, const float* __restrict__ joints,
                     const int32_t* __restrict__ parents, const float* __restrict__ dskin,
                     float* __restrict__ dtheta, int accumulate) {
  __shared__ Chain ch;
  __shared__ float share[kMaxJoints][12];   // a joint's addition to its parent's dG and dP
  __shared__ int child[kMaxJoints], next[kMaxJoints];   // highest child, next lower sibling
  const int j = threadIdx.x;
  float dG[9], dP[3], D[9], Gp[9];
  if (j < J) {
    child[j] = -1;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      dP[r] = dskin[12 * j + 4 * r + 3];
#pragma unroll
      for (int c = 0; c < 3; ++c) dG[3 * r + c] = dskin[12 * j + 4 * r + c];
    }
  }
  Joint t;
  forward_chain(J, theta, joints, parents, ch, t);
  if (j < J) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) dG[3 * r + c] -= dP[r] * t.at[c];
    int s = -1;
    if (t.p >= 0) {
#pragma unroll
      for (int q = 0; q < 9; ++q) Gp[q] = ch.G[t.p][q];
      atomicMax(&child[t.p], j);
      for (int k = t.p + 1; k < j; ++k)
        if (ch.parent[k] == t.p) s = k;
    }
    next[j] = s;
  }
  __syncthreads();
  for (int d = ch.deepest; d >= 0; --d) {
    if (t.depth == d) {
      for (int k = child[j]; k >= 0; k = next[k]) {
#pragma unroll
        for (int q = 0; q < 9; ++q) dG[q] += share[k][q];
#pragma unroll
        for (int q = 0; q < 3; ++q) dP[q] += share[k][9 + q];
      }
      if (t.p < 0) {
#pragma unroll
        for (int q = 0; q < 9; ++q) D[q] = dG[q];
      } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            float vR = 0.f, vG = 0.f;
#pragma unroll
            for (int m = 0; m < 3; ++m) {
              vR = fmaf(Gp[3 * m + r], dG[3 * m + c], vR);             // G_p^T dG_j
              vG = fmaf(dG[3 * r + m], t.R[3 * c + m], vG);            // dG_j R_j^T
            }
            D[3 * r + c] = vR;
            share[j][3 * r + c] = vG + dP[r] * t.off[c];
          }
#pragma unroll
        for (int r = 0; r < 3; ++r) share[j][9 + r] = dP[r];
      }
    }
    __syncthreads();
  }
  if (j < J) {
    const float* th = theta + 3 * j;
    const float a = t.a, b = t.b, ap = t.ap, bp = t.bp;
    const float K[9] = {0.f, -th[2], th[1], th[2], 0.f, -th[0], -th[1], th[0], 0.f};
    float K2[9];
    mat3_mul(K, K, K2);
    float dK = 0.f, dK2 = 0.f;
    for (int q = 0; q < 9; ++q) {
      dK = fmaf(D[q], K[q], dK);
      dK2 = fmaf(D[q], K2[q], dK2);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      float E[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (k == 0) { E[5] = -1.f; E[7] = 1.f; }
      if (k == 1) { E[2] = 1.f; E[6] = -1.f; }
      if (k == 2) { E[1] = -1.f; E[3] = 1.f; }
      float EK[9], KE[9];
      mat3_mul(E, K, EK);
      mat3_mul(K, E, KE);
      float dE = 0.f, dS = 0.f;
      for (int q = 0; q < 9; ++q) {
        dE = fmaf(D[q], E[q], dE);
        dS = fmaf(D[q], EK[q] + KE[q], dS);
      }
      const float v = ap * th[k] * dK + a * dE + bp * th[k] * dK2 + b * dS;
      dtheta[3 * j + k] = accumulate ? dtheta[3 * j + k] + v : v;
    }
  }
}

}  // namespace

extern "C" int pose_to_skin(void* stream, int n_joints, const float* theta, const float* joints,
                            const int32_t* parents, float* skin) {
  if (n_joints < 1 || n_joints > kMaxJoints)
    return rga::fail(RGA_EINVAL, "pose_to_skin: n_joints must be in 1..%d", kMaxJoints);
  if (!theta || !joints || !parents || !skin) return rga::fail(RGA_EINVAL, "pose_to_skin: null pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  RGA_LAUNCH("pose_skin", pose_skin_kernel, dim3(1), dim3(kBlock), 0, s, n_joints, theta, joints,
             parents, skin);
  RGA_CHECK_LAUNCH("pose_to_skin");
  return RGA_OK;
}

extern "C" int pose_to_skin_backward(void* stream, int n_joints, const float* theta,
                                     const float* joints, const int32_t* parents,
                                     const float* dskin, float* dtheta, int accumulate) {
  if (n_joints < 1 || n_joints > kMaxJoints)
    return rga::fail(RGA_EINVAL, "pose_to_skin_backward: n_joints must be in 1..%d", kMaxJoints);
  if (!theta || !joints || !parents || !dskin || !dtheta)
    return rga::fail(RGA_EINVAL, "pose_to_skin_backward: null pointer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  RGA_LAUNCH("pose_skin_bwd", pose_skin_bwd_kernel, dim3(1), dim3(kBlock), 0, s, n_joints, theta,
             joints, parents, dskin, dtheta, accumulate);
  RGA_CHECK_LAUNCH("pose_to_skin_backward");
  return RGA_OK;
}

extern "C" size_t lbs_skin_pose_grad_workspace(int n, int n_joints) {
  if (n < 0 || n_joints < 1 || n_joints > kMaxJoints) return 0;
  return (size_t)pose_chunks(n) * n_joints * 12 * 4;
}

extern "C" int lbs_skin_pose_grad(void* stream, int n, int n_joints, const int32_t* jidx,
                                  const float* jw, const float* x, const float* disp,
                                  const float* nrm, const float* dx_out, const float* dn_out,
                                  const float* dA, float* dskin, void* ws, size_t ws_bytes) {
  if (n < 0) return rga::fail(RGA_EINVAL, "lbs_skin_pose_grad: n < 0");
  if (n_joints < 1 || n_joints > kMaxJoints)
    return rga::fail(RGA_EINVAL, "lbs_skin_pose_grad: n_joints must be in 1..%d", kMaxJoints);
  if (!dskin || !ws || (n > 0 && (!jidx || !jw || !x || !dx_out)))
    return rga::fail(RGA_EINVAL, "lbs_skin_pose_grad: null pointer");
  if ((dn_out == nullptr) != (nrm == nullptr))
    return rga::fail(RGA_EINVAL, "lbs_skin_pose_grad: nrm and dn_out must both be set or both NULL");
  if (ws_bytes < lbs_skin_pose_grad_workspace(n, n_joints))
    return rga::fail(RGA_ECAPACITY, "lbs_skin_pose_grad: workspace too small");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int chunks = pose_chunks(n);
  float* part = static_cast<float*>(ws);
  // Joints are split over workgroups while the chunks alone leave CUs idle, down to four
  // a workgroup: the walk over a wave's joints is as long as they are many there (256
  // joints in no order, one workgroup per chunk -> split: 300 Gaussians 83 -> 14 us, 20k
  // 85 -> 23, 60k 86 -> 44; 24 joints 19 -> 13), and every workgroup of a chunk reads all
  // of it (100k Gaussians in the body's order, 24 joints, one workgroup 13.4 us, two 14.9).
  const int cus = rga::compute_units();
  const int split = std::min((n_joints + 3) / 4, std::max(1, 3 * cus / 2 / chunks));
  const int per = rga::ceil_div(n_joints, split);
  RGA_LAUNCH("lbs_pose_grad", lbs_pose_grad_kernel, dim3(chunks, rga::ceil_div(n_joints, per)), dim3(kPoseWaves * 64),
             (size_t)kPoseWaves * per * 12 * sizeof(float), s, n, n_joints, per, jidx, jw, x, disp, nrm,
             dx_out, dn_out, dA, part);
  RGA_LAUNCH("lbs_pose_grad_final", lbs_pose_grad_final, dim3(rga::ceil_div(12 * n_joints, 64)),
             dim3(1024), 0, s, n_joints, chunks, part, dskin);
  RGA_CHECK_LAUNCH("lbs_skin_pose_grad");
  return RGA_OK;
}

extern "C" int lbs_skin(void* stream, int n, int n_joints, const float* skin, const int32_t* jidx,
                        const float* jw, const float* x, const float* disp, const float* nrm,
                        float* x_out, float* n_out, float* A_out) {
  if (n < 0) return rga::fail(RGA_EINVAL, "lbs_skin: n < 0");
  if (n_joints < 1 || n_joints > kMaxJoints)
    return rga::fail(RGA_EINVAL, "lbs_skin: n_joints must be in 1..%d", kMaxJoints);
  if (n == 0) return RGA_OK;
  if (!skin || !jidx || !jw || !x || !x_out) return rga::fail(RGA_EINVAL, "lbs_skin: null pointer");
  if (n_out && !nrm) return rga::fail(RGA_EINVAL, "lbs_skin: n_out requires nrm");
  hipStream_t s = static_cast<hipStream_t>(stream);
  RGA_LAUNCH("lbs_fwd", lbs_fwd_kernel, dim3(rga::ceil_div(n, kBlock)), dim3(kBlock), 0, s, n,
             n_joints, skin, jidx, jw, x, disp, nrm, x_out, n_out, A_out);
  RGA_CHECK_LAUNCH("lbs_skin");
  return RGA_OK;
}

extern "C" int lbs_skin_backward(void* stream, int n, int n_joints, const float* skin,
                                 const int32_t* jidx, const float* jw, const float* dx_out,
                                 const float* dn_out, float* dx, float* dn) {
  if (n < 0) return rga::fail(RGA_EINVAL, "lbs_skin_backward: n < 0");
  if (n_joints < 1 || n_joints > kMaxJoints)
    return rga::fail(RGA_EINVAL, "lbs_skin_backward: n_joints must be in 1..%d", kMaxJoints);
  if (n == 0) return RGA_OK;
  if (!skin || !jidx || !jw || !dx_out || !dx)
    return rga::fail(RGA_EINVAL, "lbs_skin_backward: null pointer");
  if ((dn_out == nullptr) != (dn == nullptr))
    return rga::fail(RGA_EINVAL, "lbs_skin_backward: dn_out and dn must both be set or both NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  RGA_LAUNCH("lbs_bwd", lbs_bwd_kernel, dim3(rga::ceil_div(n, kBlock)), dim3(kBlock), 0, s, n,
             n_joints, skin, jidx, jw, dx_out, dn_out, dx, dn);
  RGA_CHECK_LAUNCH("lbs_skin_backward");
  return RGA_OK;
}
