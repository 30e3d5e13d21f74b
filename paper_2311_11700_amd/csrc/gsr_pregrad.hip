// Chain rule from the per-view 2D gradients back to the Gaussian parameters
// and the camera pose (GS-SLAM Eq. 2-3, Eq. 11 and supplement Sec. A).
#include <math.h>

#include "gsr_internal.h"

namespace gsr {

struct PreConstsB {
  float z_near, lowpass, cutoff;
  uint32_t flags;
  float fov_guard;
};

// dst += v, or dst = v when the gradients are overwritten.
__device__ __forceinline__ void put(float &dst, double v, bool overwrite) {
  dst = overwrite ? (float)v : dst + (float)v;
}

// The chain runs in FP64: gfx950 executes FP64 vector arithmetic at the
// non-packed FP32 rate, and near-camera Gaussians put 1/z^3 factors and
// cancelling terms into this chain.
using R = double;

// v of the lane that the DPP control names (0 where there is none).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_d(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Sum over the wavefront, in lane 63.
__device__ __forceinline__ double wave_sum_d(double v) {
  v += dpp_d<0x111, 0xf>(v);  // row_shr:1
  v += dpp_d<0x112, 0xf>(v);  // row_shr:2
  v += dpp_d<0x114, 0xf>(v);  // row_shr:4
  v += dpp_d<0x118, 0xf>(v);  // row_shr:8
  v += dpp_d<0x142, 0xa>(v);  // row_bcast:15
  v += dpp_d<0x143, 0xc>(v);  // row_bcast:31
  return v;
}

// Rotation matrix of a unit quaternion (w, x, y, z) (supplement eq. q2R).
__device__ __forceinline__ void quat_rot_r(R w, R x, R y, R z, R M[9]) {
  M[0] = R(1) - R(2) * (y * y + z * z);
  M[1] = R(2) * (x * y - w * z);
  M[2] = R(2) * (x * z + w * y);
  M[3] = R(2) * (x * y + w * z);
  M[4] = R(1) - R(2) * (x * x + z * z);
  M[5] = R(2) * (y * z - w * x);
  M[6] = R(2) * (x * z - w * y);
  M[7] = R(2) * (y * z + w * x);
  M[8] = R(1) - R(2) * (x * x + y * y);
}

// Gradient rows of the visible records (the others are neither added to nor
// read) cleared, BLOCK records of a view a block.  Bound by the stores: a row of
// GEO_ROW doubles is written by four lanes, one of COL_ROW by two, so that a
// wavefront writes whole cache lines.  (Two fills over the rows of all records,
// 96 bytes each: a backward of 300 000 Gaussians at 1200x680 147 us, 143 so; of
// 500 000 in 16 views of 600x340 698 and 655 us.)
__global__ __launch_bounds__(BLOCK) void k_clear_rows(Workspace ws, int64_t n, int64_t vis_words, int colours) {
  const int view = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint64_t visible =
      reinterpret_cast<const uint64_t *>(ws.visible)[(int64_t)view * (vis_words / 2) + (int64_t)blockIdx.x * (BLOCK / 64) + wave];
  if (visible == 0ull) return;
  const int64_t rec = (int64_t)view * n + (int64_t)blockIdx.x * BLOCK + wave * 64;
  constexpr int GP = GEO_ROW / 2, CP = COL_ROW / 2;  // lanes of a row
  double2 *geo = reinterpret_cast<double2 *>(ws.grad2d + rec * GEO_ROW);
  double2 *col = reinterpret_cast<double2 *>(ws.grad_col + rec * COL_ROW);
#pragma unroll
  for (int k = lane; k < 64 * GP; k += 64)
    if (visible >> (k / GP) & 1ull) geo[k] = make_double2(0., 0.);
  if (!colours) return;
#pragma unroll
  for (int k = lane; k < 64 * CP; k += 64)
    if (visible >> (k / CP) & 1ull) col[k] = make_double2(0., 0.);
}

void launch_clear_grads(const Plan &p, const Workspace &ws, const RenderConsts &rc, hipStream_t s) {
  if (p.n > 0)
    hipLaunchKernelGGL(k_clear_rows, dim3((unsigned)((p.n + BLOCK - 1) / BLOCK), (unsigned)p.n_views), dim3(BLOCK), 0, s, ws,
                       p.n, p.vis_words, (rc.grad_fields >> GEO_FIELDS) != 0u ? 1 : 0);
}

// ----------------------------------------------------------------------------
// Backward: per Gaussian, loop over the views, chain the per-view 2D
// gradients (u, v, conic, depth, opacity, colour) through Eq. 3 to the
// camera-frame point and to L = R_q diag(s) (Sigma = L L^T), accumulate
// dL/dmean and dL/dL over the views, then chain dL/dL to the log-scales and
// the quaternion once.  With P = J W (2x3) and T = P L the projected covariance
// is T T^T + lowpass, so that with G = dL/dSigma'
//   H = 2 G T,  dL/dP = H L^T,  dL/dL += P^T H,  dL/dJ = dL/dP W^T,
// and no 3x3 covariance is formed.  The pose gradient of each view is the
// left-perturbation derivative rho = sum gX, phi = sum (X_c x gX + v) with
// v_i = sum_jk eps_ijk Q_kj, Q = dL/dW W^T and dL/dW = J^T dL/dP, reduced per
// block into fixed slots (deterministic order).
//
// A block takes BLOCK Gaussians and `vpb` views: all of them when the
// Gaussians' gradients are wanted (they are summed in registers), otherwise
// POSE_VIEWS, so that the views spread over the chip.  Bound by the latency of
// the dependent reads (visibility bits, then the gradients of the records that
// are visible) and, over many views, by FP64 work in wavefronts of which a
// quarter to a half of the lanes is visible.  The bits of VCHUNK views are
// read at a time and the next view's gradients ahead; the covariance form
// (three 3x3 products more, 224 registers) took 755 us for the poses of 72
// views of 500 000 Gaussians, 237 us for 16 views of a million, 11 us for the
// pose of one view of 150 000: 304, 205 and 6.5 us now (300 000 Gaussians and
// one view 19 us before and after).  72, 16, 8 and 4 views a block for the 72:
// 460, 412, 415 and 440 us (with 80-byte gradient rows).

// SH: the colour is degree-1 spherical harmonics; GAUSS: the Gaussians'
// gradients are wanted (instantiated separately for their registers).
constexpr int VCHUNK = 8;
constexpr int POSE_VIEWS = 8;  // views of a block without Gaussian gradients

template <bool SH, bool GAUSS>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(2))) void k_preprocess_bwd(
    gsr_gaussians g, const gsr_camera *__restrict__ cams, int n_views, int vpb, int64_t vis_words, PreConstsB pc, Workspace ws,
    gsr_grads gr) {
  extern __shared__ double s_dyn[];  // [4 waves][vpb][6]
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const bool active = i < g.n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int view0 = blockIdx.y * vpb, view1 = min(view0 + vpb, n_views);
  const bool want_pose = (pc.flags & GSR_POSE_GRAD) && gr.d_pose;
  const bool approx = (pc.flags & GSR_PAPER_POSE_APPROX) != 0;

  if (want_pose) {
    for (int k = threadIdx.x; k < 4 * vpb * 6; k += BLOCK) s_dyn[k] = 0.;
    __syncthreads();
  }

  R mx = 0, my = 0, mz = 0;
  // The linear spherical-harmonic coefficients as stored (float32, widened
  // where used); the constant term does not enter the direction gradient.
  float shc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) shc[k] = 0.f;
  if (active && SH) {
#pragma unroll
    for (int k = 0; k < 9; ++k) shc[k] = g.sh[12 * i + 3 + k];
  }
  // Gradients of the linear coefficients; the constant term's is Y_0 times
  // the colour gradient summed over the views (gc0..gc2).
  R gsh[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) gsh[k] = 0.;
  // L = R_q diag(s); the scales and the rotation are found again at the end,
  // which costs less than their registers in between.
  auto factors = [&](R sc[3], R &w, R &x, R &y, R &z, R &inv, R M[9]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) sc[k] = exp((R)g.log_scale[3 * i + k]);
    const float4 fq = reinterpret_cast<const float4 *>(g.quat)[i];
    const R q0 = fq.x, q1 = fq.y, q2 = fq.z, q3 = fq.w;
    const R qn = sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
    inv = qn > 0 ? R(1) / qn : R(0);
    w = q0 * inv; x = q1 * inv; y = q2 * inv; z = q3 * inv;
    quat_rot_r(w, x, y, z, M);
  };
  R L[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) L[k] = 0.;
  if (active) {
    mx = g.mean[3 * i]; my = g.mean[3 * i + 1]; mz = g.mean[3 * i + 2];
    R sc[3], w, x, y, z, inv;
    factors(sc, w, x, y, z, inv, L);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int k = 0; k < 3; ++k) L[3 * c + k] *= sc[k];
  }

  R gm[3] = {0, 0, 0};
  R gL[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  R gop = 0., gc0 = 0., gc1 = 0., gc2 = 0.;

  for (int v0 = view0; v0 < view1; v0 += VCHUNK) {
    uint32_t visible = 0u;  // bit k: in view v0 + k
    {
      // (a word per wavefront and view)
      const uint64_t *words = reinterpret_cast<const uint64_t *>(ws.visible) + blockIdx.x * (BLOCK / 64) + wave;
      uint64_t w[VCHUNK];
#pragma unroll
      for (int k = 0; k < VCHUNK; ++k) w[k] = v0 + k < view1 ? words[(int64_t)(v0 + k) * (vis_words / 2)] : 0ull;
#pragma unroll
      for (int k = 0; k < VCHUNK; ++k) visible |= (uint32_t)(w[k] >> lane & 1u) << k;
    }
    uint32_t todo = 0u;  // views in which some lane is visible
#pragma unroll
    for (int k = 0; k < VCHUNK; ++k) todo |= __any((visible >> k) & 1u) ? 1u << k : 0u;
    constexpr bool COL = SH || GAUSS;  // the colour fields matter
    constexpr int NG = GEO_ROW / 2, NC = COL ? COL_ROW / 2 : 0;
    auto read = [&](int k, double2 d[NG + NC]) {
      const int64_t rec = (int64_t)(v0 + k) * g.n + i;
      const double2 *geo = reinterpret_cast<const double2 *>(ws.grad2d + rec * GEO_ROW);
      const double2 *col = reinterpret_cast<const double2 *>(ws.grad_col + rec * COL_ROW);
      const bool vis = (visible >> k) & 1u;
#pragma unroll
      for (int f = 0; f < NG - (COL ? 0 : 1); ++f) d[f] = vis ? geo[f] : make_double2(0., 0.);
#pragma unroll
      for (int f = 0; f < NC; ++f) d[NG + f] = vis ? col[f] : make_double2(0., 0.);
    };
    double2 next[NG + NC];
    if (todo) read(__builtin_ctz(todo), next);
    while (todo) {
      const int view = v0 + __builtin_ctz(todo);
      todo &= todo - 1u;
      R g2[NGRAD2D];
      bool has = false;
#pragma unroll
      for (int f = 0; f < NGRAD2D; ++f) {
        const int at = f < GEO_FIELDS ? f : GEO_ROW + f - GEO_FIELDS;
        g2[f] = f < (COL ? NGRAD2D : 6) ? (at & 1 ? next[at >> 1].y : next[at >> 1].x) : 0.;
        has = has || g2[f] != 0.;
      }
      // The next view's gradients are read while this one's are chained.
      if (todo) read(__builtin_ctz(todo), next);
      if (!__any(has)) continue;
      R pr[6] = {0, 0, 0, 0, 0, 0};
      if (has) {
        if (GAUSS) {
          gop += g2[6];
          gc0 += g2[7]; gc1 += g2[8]; gc2 += g2[9];
        }
        const gsr_camera &cam = cams[view];
        R W[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) W[k] = cam.R[k];
        const R x = W[0] * mx + W[1] * my + W[2] * mz + (R)cam.t[0];
        const R y = W[3] * mx + W[4] * my + W[5] * mz + (R)cam.t[1];
        const R z = W[6] * mx + W[7] * my + W[8] * mz + (R)cam.t[2];
        const R fx = cam.fx, fy = cam.fy;
        const R iz = R(1) / z, iz2 = iz * iz;
        // x/z, y/z as they enter J (limited by the guard); a limited ratio no
        // longer depends on x (or y), and J then depends on z through 1/z only.
        R rxz = x * iz, ryz = y * iz;
        R free_x = 1., free_y = 1.;
        if (pc.fov_guard > 0.f) {
          const R lx = (R)pc.fov_guard * (0.5 * (R)cam.width) / fx;
          const R ly = (R)pc.fov_guard * (0.5 * (R)cam.height) / fy;
          if (rxz > lx || rxz < -lx) { rxz = rxz > 0. ? lx : -lx; free_x = 0.; }
          if (ryz > ly || ryz < -ly) { ryz = ryz > 0. ? ly : -ly; free_y = 0.; }
        }
        const R J00 = fx * iz, J02 = -fx * rxz * iz, J11 = fy * iz, J12 = -fy * ryz * iz;
        R P0[3], P1[3], T0[3], T1[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          P0[c] = J00 * W[c] + J02 * W[6 + c];
          P1[c] = J11 * W[3 + c] + J12 * W[6 + c];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          T0[k] = P0[0] * L[k] + P0[1] * L[3 + k] + P0[2] * L[6 + k];
          T1[k] = P1[0] * L[k] + P1[1] * L[3 + k] + P1[2] * L[6 + k];
        }
        const R A = T0[0] * T0[0] + T0[1] * T0[1] + T0[2] * T0[2] + pc.lowpass;
        const R B = T0[0] * T1[0] + T0[1] * T1[1] + T0[2] * T1[2];
        const R C = T1[0] * T1[0] + T1[1] * T1[1] + T1[2] * T1[2] + pc.lowpass;
        const R idet = 1. / (A * C - B * B);
        const R ca = C * idet, cb = -B * idet, cc = A * idet;
        // dL/dSigma' = -M G_M M with M the conic, G_M = [[ga, gb/2], [gb/2, gc]];
        // twice that, for H.
        const R n00 = g2[2], n01 = 0.5 * g2[3], n11 = g2[4];
        const R P00 = ca * n00 + cb * n01, P01 = ca * n01 + cb * n11;
        const R P10 = cb * n00 + cc * n01, P11 = cb * n01 + cc * n11;
        const R G00 = -2. * (P00 * ca + P01 * cb), G01 = -2. * (P00 * cb + P01 * cc),
                G11 = -2. * (P10 * cb + P11 * cc);
        R H0[3], H1[3], D0[3], D1[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          H0[k] = G00 * T0[k] + G01 * T1[k];
          H1[k] = G01 * T0[k] + G11 * T1[k];
        }
        if (GAUSS) {
#pragma unroll
          for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < 3; ++k) gL[3 * c + k] += P0[c] * H0[k] + P1[c] * H1[k];
        }
        // dL/dP, and D_r = dL/dP_r W^T.
        {
          R dP0[3], dP1[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            dP0[c] = H0[0] * L[3 * c] + H0[1] * L[3 * c + 1] + H0[2] * L[3 * c + 2];
            dP1[c] = H1[0] * L[3 * c] + H1[1] * L[3 * c + 1] + H1[2] * L[3 * c + 2];
          }
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            D0[r] = dP0[0] * W[3 * r] + dP0[1] * W[3 * r + 1] + dP0[2] * W[3 * r + 2];
            D1[r] = dP1[0] * W[3 * r] + dP1[1] * W[3 * r + 1] + dP1[2] * W[3 * r + 2];
          }
        }
        const R GJ00 = D0[0], GJ02 = D0[2], GJ11 = D1[1], GJ12 = D1[2];
        const R gu = g2[0], gv = g2[1], gzd = g2[5];
        // Through the projected centre and depth.
        const R pX0 = gu * fx * iz;
        const R pX1 = gv * fy * iz;
        const R pX2 = gzd - (gu * fx * x + gv * fy * y) * iz2;
        // Through J (part of the Sigma' path): J02 = -fx r/z with r = x/z (or
        // its limit), dJ02/dx = -fx/z^2 while r is free, dJ02/dz = fx r/z^2
        // (+ fx x/z^3 while r is free); J12 likewise.
        const R jX0 = -GJ02 * fx * iz2 * free_x;
        const R jX1 = -GJ12 * fy * iz2 * free_y;
        const R jX2 = (fx * (GJ02 * (rxz + free_x * x * iz) - GJ00) + fy * (GJ12 * (ryz + free_y * y * iz) - GJ11)) * iz2;
        const R gX0 = pX0 + jX0, gX1 = pX1 + jX1, gX2 = pX2 + jX2;
        if (GAUSS) {
          gm[0] += W[0] * gX0 + W[3] * gX1 + W[6] * gX2;
          gm[1] += W[1] * gX0 + W[4] * gX1 + W[7] * gX2;
          gm[2] += W[2] * gX0 + W[5] * gX1 + W[8] * gX2;
        }
        // Spherical-harmonic colour: coefficient gradient Y (x) dL/dc and, through
        // the viewing direction d = v / |v| (v = mean - o, o = -W^T t),
        // dL/dv = (I - d d^T) dL/dd / |v|, which adds to the mean and, since a
        // left perturbation moves o by -W^T rho, W dL/dv to the pose's rho.
        R gv0 = 0., gv1 = 0., gv2 = 0.;
        if (SH) {
          const R t0 = cam.t[0], t1 = cam.t[1], t2 = cam.t[2];
          const R vx = mx + (W[0] * t0 + W[3] * t1 + W[6] * t2);
          const R vy = my + (W[1] * t0 + W[4] * t1 + W[7] * t2);
          const R vz = mz + (W[2] * t0 + W[5] * t1 + W[8] * t2);
          const R il = R(1) / sqrt(vx * vx + vy * vy + vz * vz);
          const R dx = vx * il, dy = vy * il, dz = vz * il;
          const R Y[3] = {SH_C1 * dy, SH_C1 * dz, SH_C1 * dx};
          const R gc[3] = {g2[7], g2[8], g2[9]};
          if (GAUSS) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
              for (int ch = 0; ch < 3; ++ch) gsh[3 * k + ch] += Y[k] * gc[ch];
          }
          R gY1 = 0., gY2 = 0., gY3 = 0.;
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) {
            gY1 += (R)shc[ch] * gc[ch];
            gY2 += (R)shc[3 + ch] * gc[ch];
            gY3 += (R)shc[6 + ch] * gc[ch];
          }
          const R gdx = SH_C1 * gY3, gdy = SH_C1 * gY1, gdz = SH_C1 * gY2;
          const R dot = dx * gdx + dy * gdy + dz * gdz;
          gv0 = (gdx - dx * dot) * il;
          gv1 = (gdy - dy * dot) * il;
          gv2 = (gdz - dz * dot) * il;
          if (GAUSS) {
            gm[0] += gv0;
            gm[1] += gv1;
            gm[2] += gv2;
          }
        }
        if (want_pose) {
          const R rX0 = approx ? pX0 : gX0, rX1 = approx ? pX1 : gX1, rX2 = approx ? pX2 : gX2;
          pr[0] = rX0; pr[1] = rX1; pr[2] = rX2;
          pr[3] = y * rX2 - z * rX1;
          pr[4] = z * rX0 - x * rX2;
          pr[5] = x * rX1 - y * rX0;
          if (!approx) {
            // Q = dL/dW W^T: rows J00 D0, J11 D1, J02 D0 + J12 D1.
            pr[3] += (J02 * D0[1] + J12 * D1[1]) - J11 * D1[2];
            pr[4] += J00 * D0[2] - (J02 * D0[0] + J12 * D1[0]);
            pr[5] += J11 * D1[0] - J00 * D0[1];
          }
          if (SH) {
            pr[0] += W[0] * gv0 + W[1] * gv1 + W[2] * gv2;
            pr[1] += W[3] * gv0 + W[4] * gv1 + W[5] * gv2;
            pr[2] += W[6] * gv0 + W[7] * gv1 + W[8] * gv2;
          }
        }
      }
      if (want_pose) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          const R t = wave_sum_d(pr[k]);
          if (lane == 63) s_dyn[(wave * vpb + (view - view0)) * 6 + k] = t;
        }
      }
    }
  }

  if (active && GAUSS) {
    // Eq. 2 backward: L = Rq diag(s).
    R Rq[9], GR[9];
    R sc[3], w, x, y, z, iq;
    __asm__ volatile("" ::: "memory");  // (read again, not kept)
    factors(sc, w, x, y, z, iq, Rq);
    R gl[3] = {0., 0., 0.};
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        GR[3 * c + k] = gL[3 * c + k] * sc[k];
        gl[k] += GR[3 * c + k] * Rq[3 * c + k];
      }
    const R gw = 2. * (-z * GR[1] + y * GR[2] + z * GR[3] - x * GR[5] - y * GR[6] + x * GR[7]);
    const R gx = 2. * (y * GR[1] + z * GR[2] + y * GR[3] - 2. * x * GR[4] - w * GR[5] + z * GR[6] +
                            w * GR[7] - 2. * x * GR[8]);
    const R gy = 2. * (-2. * y * GR[0] + x * GR[1] + w * GR[2] + x * GR[3] + z * GR[5] - w * GR[6] +
                            z * GR[7] - 2. * y * GR[8]);
    const R gz = 2. * (-2. * z * GR[0] - w * GR[1] + x * GR[2] + w * GR[3] - 2. * z * GR[4] + y * GR[5] +
                            x * GR[6] + y * GR[7]);
    const R dotq = w * gw + x * gx + y * gy + z * gz;
    const bool ow = (pc.flags & GSR_GRAD_OVERWRITE) != 0;
    if (gr.d_mean) {
      put(gr.d_mean[3 * i], gm[0], ow);
      put(gr.d_mean[3 * i + 1], gm[1], ow);
      put(gr.d_mean[3 * i + 2], gm[2], ow);
    }
    if (gr.d_log_scale) {
      put(gr.d_log_scale[3 * i], gl[0], ow);
      put(gr.d_log_scale[3 * i + 1], gl[1], ow);
      put(gr.d_log_scale[3 * i + 2], gl[2], ow);
    }
    if (gr.d_quat) {
      float4 *dq = reinterpret_cast<float4 *>(gr.d_quat) + i;
      float4 cur = ow ? make_float4(0.f, 0.f, 0.f, 0.f) : *dq;
      cur.x += (float)((gw - w * dotq) * iq);
      cur.y += (float)((gx - x * dotq) * iq);
      cur.z += (float)((gy - y * dotq) * iq);
      cur.w += (float)((gz - z * dotq) * iq);
      *dq = cur;
    }
    if (gr.d_opacity_logit) {
      const R o = R(1) / (R(1) + exp(-(R)g.opacity_logit[i]));
      put(gr.d_opacity_logit[i], gop * o * (R(1) - o), ow);
    }
    if (SH && gr.d_sh) {
      put(gr.d_sh[12 * i], SH_C0 * gc0, ow);
      put(gr.d_sh[12 * i + 1], SH_C0 * gc1, ow);
      put(gr.d_sh[12 * i + 2], SH_C0 * gc2, ow);
#pragma unroll
      for (int k = 0; k < 9; ++k) put(gr.d_sh[12 * i + 3 + k], gsh[k], ow);
    }
    if (gr.d_rgb && !SH) {
      put(gr.d_rgb[3 * i], gc0, ow);
      put(gr.d_rgb[3 * i + 1], gc1, ow);
      put(gr.d_rgb[3 * i + 2], gc2, ow);
    }
  }

  if (want_pose) {
    __syncthreads();
    const int V6 = vpb * 6;
    for (int k = threadIdx.x; k < (view1 - view0) * 6; k += BLOCK)
      ws.pose_part[(int64_t)(view0 * 6 + k) * gridDim.x + blockIdx.x] =
          s_dyn[k] + s_dyn[V6 + k] + s_dyn[2 * V6 + k] + s_dyn[3 * V6 + k];
  }
}

// Deterministic reduction of the per-block pose partials: one block per
// (view, component), fixed summation order; with tile_loss a last block sums
// the tiles' losses the same way (in FP64: a float sum over the tiles in the
// order they finish differs between two runs in its sixth digit).
__global__ __launch_bounds__(BLOCK) void k_step_reduce(const double *__restrict__ part, int n_blocks, int n_pose, int overwrite, float *__restrict__ d_pose,
                                                       const float *__restrict__ tile_loss, int n_tiles,
                                                       float *__restrict__ loss) {
  __shared__ double red[BLOCK];
  const int vc = blockIdx.x;  // view * 6 + component
  double acc = 0.0;
  if (vc < n_pose) {
    for (int b = threadIdx.x; b < n_blocks; b += BLOCK) acc += part[(int64_t)vc * n_blocks + b];
  } else {
#pragma unroll 8
    for (int t = threadIdx.x; t < n_tiles; t += BLOCK) acc += (double)tile_loss[t];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = BLOCK / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) put(vc < n_pose ? d_pose[vc] : *loss, red[0], overwrite != 0);
}

void launch_preprocess_backward(const Plan &p, const gsr_gaussians &g, const gsr_camera *cams,
                                const gsr_config &cfg, const Workspace &ws, const gsr_grads &gr, float *loss,
                                hipStream_t s) {
  const bool want_pose = (cfg.flags & GSR_POSE_GRAD) && gr.d_pose;
  const int overwrite = (cfg.flags & GSR_GRAD_OVERWRITE) ? 1 : 0;
  if (g.n > 0) {
    PreConstsB pc{cfg.z_near, cfg.lowpass, cfg.cutoff_sigma, cfg.flags, cfg.fov_guard};
    const bool gauss = (cfg.flags & GSR_GAUSS_GRAD) != 0;
    const int vpb = gauss ? p.n_views : std::min(p.n_views, POSE_VIEWS);
    const size_t lds = want_pose ? (size_t)4 * vpb * 6 * sizeof(double) : 0;
    const auto kernel = g.sh ? (gauss ? k_preprocess_bwd<true, true> : k_preprocess_bwd<true, false>)
                             : (gauss ? k_preprocess_bwd<false, true> : k_preprocess_bwd<false, false>);
    hipLaunchKernelGGL(kernel, dim3(p.n_pose_blocks, (unsigned)((p.n_views + vpb - 1) / vpb)), dim3(BLOCK), lds, s, g,
                       cams, p.n_views, vpb, p.vis_words, pc, ws, gr);
  } else if (want_pose && overwrite) {
    // No Gaussian, no gradient: an overwritten pose gradient is zero.
    launch_fill_f32(gr.d_pose, 0.f, (int64_t)p.n_views * 6, s);
  }
  const int n_pose = g.n > 0 && want_pose ? p.n_views * 6 : 0;
  if (n_pose > 0 || loss)
    hipLaunchKernelGGL(k_step_reduce, dim3((unsigned)(n_pose + (loss ? 1 : 0))), dim3(BLOCK), 0, s, ws.pose_part,
                       p.n_pose_blocks, n_pose, overwrite, gr.d_pose, ws.tile_loss, p.total_tiles, loss);
}

}  // namespace gsr
