// Per-(view, Gaussian) projection: camera-frame centre, EWA screen-space
// covariance and its conic, opacity, tile rectangle and depth sort key
// (GS-SLAM Eq. 2-3, supplement eq. q2R).
//
// Forward geometry runs in FP64: gfx950 executes FP64 vector arithmetic at
// the FP32 non-packed rate.  The camera-frame centre, and so the depth sort key,
// agrees bit for bit with an FP64 reference evaluated in the same order
// (contraction is off); the covariance and the tile rectangle, formed without
// the 3x3 covariance and with reciprocals, agree up to FP64 rounding.  The
// values the rasteriser consumes are rounded to FP32 once, at the end.
#pragma clang fp contract(off)

#include <math.h>

#include "gsr_internal.h"

namespace gsr {

struct PreConsts {
  float z_near, lowpass, cutoff;
  uint32_t flags;
  float fov_guard;
  float alpha_min;
  double inv_alpha_min;
  int clear_grads;  // zero each record's geometry row (1) or both gradient rows (2): start of a fused step
};

// Rotation matrix of a unit quaternion (w, x, y, z) (GS-SLAM supplement,
// eq. q2R), row-major.
template <typename T>
__device__ __forceinline__ void quat_rot(T w, T x, T y, T z, T R[9]) {
  R[0] = T(1) - T(2) * (y * y + z * z);
  R[1] = T(2) * (x * y - w * z);
  R[2] = T(2) * (x * z + w * y);
  R[3] = T(2) * (x * y + w * z);
  R[4] = T(1) - T(2) * (x * x + z * z);
  R[5] = T(2) * (y * z - w * x);
  R[6] = T(2) * (x * z - w * y);
  R[7] = T(2) * (y * z + w * x);
  R[8] = T(1) - T(2) * (x * x + y * y);
}

// Upper bound of the squared spectral norm of the view's matrix W: the largest
// row sum of |W W^T|.  1 for a rotation; the projection takes W as it is, a
// similarity's scale or a drifted product of rotations too.
__device__ __forceinline__ float norm2_bound(const float *W) {
  float g[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      g[i][j] = fabsf(W[3 * i] * W[3 * j] + W[3 * i + 1] * W[3 * j + 1] + W[3 * i + 2] * W[3 * j + 2]);
  return fmaxf(fmaxf(g[0][0] + g[0][1] + g[0][2], g[1][0] + g[1][1] + g[1][2]), g[2][0] + g[2][1] + g[2][2]);
}

// Whether record i of the view is certainly culled: masked, not beyond the near
// plane, or its tile rectangle empty.  The rectangle's half-width is
// cutoff sqrt(A) with A <= |J_0|^2 |W|^2 max(scale)^2 + lowpass; the bound is
// evaluated in float32 with margins far above its rounding, and any
// comparison with a NaN keeps the record for the exact tests.  norm2: at least
// |W|^2.
struct Early {
  float m[3], ls[3];  // mean, log scales
  uint8_t keep;       // mask
};

__device__ __forceinline__ bool surely_culled(const Early &e, const gsr_camera &cam, const ViewInfo &vi,
                                              const PreConsts &pc, float norm2) {
  if (e.keep == 0) return true;
  const double mx = e.m[0], my = e.m[1], mz = e.m[2];
  const double x = (((double)cam.R[0] * mx + (double)cam.R[1] * my) + (double)cam.R[2] * mz) + (double)cam.t[0];
  const double y = (((double)cam.R[3] * mx + (double)cam.R[4] * my) + (double)cam.R[5] * mz) + (double)cam.t[1];
  const double z = (((double)cam.R[6] * mx + (double)cam.R[7] * my) + (double)cam.R[8] * mz) + (double)cam.t[2];
  if (z <= (double)pc.z_near) return true;
  if ((pc.flags & GSR_FULL_RECT) || !(cam.fx > 0.f) || !(cam.fy > 0.f)) return false;
  const float ls = fmaxf(fmaxf(e.ls[0], e.ls[1]), e.ls[2]);
  const float smax = __expf(ls) * 1.001f;
  const float rz = 1.f / (float)z, xz = (float)x * rz, yz = (float)y * rz;
  float tx = fabsf(xz), ty = fabsf(yz);
  if (pc.fov_guard > 0.f) {
    tx = fminf(tx, pc.fov_guard * (0.5f * (float)vi.W) / cam.fx * 1.001f);
    ty = fminf(ty, pc.fov_guard * (0.5f * (float)vi.H) / cam.fy * 1.001f);
  }
  const float jx = cam.fx * rz, jy = cam.fy * rz;
  const float rx = pc.cutoff * sqrtf(jx * jx * (1.f + tx * tx) * smax * smax * norm2 + fabsf(pc.lowpass));
  const float ry = pc.cutoff * sqrtf(jy * jy * (1.f + ty * ty) * smax * smax * norm2 + fabsf(pc.lowpass));
  const float u = cam.fx * xz + cam.cx, v = cam.fy * yz + cam.cy;
  const float mu = rx * 1.001f + 1e-4f * (fabsf(u) + fabsf(cam.cx)) + 0.5f;
  const float mv = ry * 1.001f + 1e-4f * (fabsf(v) + fabsf(cam.cy)) + 0.5f;
  return u + mu < 0.f || u - mu > (float)(vi.TX * TILE) || v + mv < 0.f || v - mv > (float)(vi.TY * TILE);
}

// What the binning needs of a visible record: its tile rectangle, depth key,
// conic (its alpha support lies apart).
struct Staged {
  float a, b, c;
  uint32_t key, rec;
  uint16_t tx0, tx1, ty0, ty1;
};

// The projection's arguments, in LDS.
struct ProjArgs {
  gsr_gaussians g;
  ViewInfo vi;
  PreConsts pc;
  float4 *rec;
  double *grad2d, *grad_col;
  int cull;
};

// Project record rec = view * n + i; returns whether it is visible (`out` is
// then filled in).  SH: spherical-harmonic colour.  Out of line, with its
// arguments in LDS: inside the loop over the batches the compiler keeps the
// camera's FP64 values and the coefficients of exp and log in registers
// (170 instead of 90, and one block per CU less).
template <bool SH>
__device__ __attribute__((noinline)) bool project_record(const ProjArgs *args, const gsr_camera *camp, int64_t i,
                                                         int64_t rec, Staged *out, Support *support) {
  const gsr_gaussians &g = args->g;
  const ViewInfo &vi = args->vi;
  const PreConsts &pc = args->pc;
  const ProjArgs &ws = *args;
  const gsr_camera &cam = *camp;
  const float fm0 = g.mean[3 * i], fm1 = g.mean[3 * i + 1], fm2 = g.mean[3 * i + 2];
  const float fl0 = g.log_scale[3 * i], fl1 = g.log_scale[3 * i + 1], fl2 = g.log_scale[3 * i + 2];
  const float4 fq = reinterpret_cast<const float4 *>(g.quat)[i];
  const float fop = g.opacity_logit[i];
  // Colour: RGB, or the 12 spherical-harmonic coefficients [4][3].
  constexpr int ncol = SH ? 12 : 3;
  float col[ncol];
  const float *csrc = SH ? g.sh + 12 * i : g.rgb + 3 * i;
  bool colour_ok = true;
#pragma unroll
  for (int k = 0; k < ncol; ++k) {
    col[k] = csrc[k];
    colour_ok = colour_ok && isfinite(col[k]);
  }

  bool ok = isfinite(fm0) && isfinite(fm1) && isfinite(fm2) && isfinite(fl0) && isfinite(fl1) &&
            isfinite(fl2) && isfinite(fq.x) && isfinite(fq.y) && isfinite(fq.z) && isfinite(fq.w) &&
            isfinite(fop) && colour_ok;
  if (g.mask) ok = ok && g.mask[i] != 0;

  // Camera-frame centre, each row summed left to right (this is the exact
  // sequence behind the float32 depth key).
  const double mx = fm0, my = fm1, mz = fm2;
  const double W0 = cam.R[0], W1 = cam.R[1], W2 = cam.R[2], W3 = cam.R[3], W4 = cam.R[4],
               W5 = cam.R[5], W6 = cam.R[6], W7 = cam.R[7], W8 = cam.R[8];
  const double x = ((W0 * mx + W1 * my) + W2 * mz) + (double)cam.t[0];
  const double y = ((W3 * mx + W4 * my) + W5 * mz) + (double)cam.t[1];
  const double z = ((W6 * mx + W7 * my) + W8 * mz) + (double)cam.t[2];
  ok = ok && (z > (double)pc.z_near);

  // Rotation of Eq. 2.
  double qw = fq.x, qx = fq.y, qy = fq.z, qz = fq.w;
  const double qn = sqrt(((qw * qw + qx * qx) + qy * qy) + qz * qz);
  ok = ok && (qn > 0.0);
  double Rq[9];
  {
    const double inv = 1.0 / (ok ? qn : 1.0);
    qw *= inv; qx *= inv; qy *= inv; qz *= inv;
    quat_rot<double>(qw, qx, qy, qz, Rq);
  }
  const double s0 = exp((double)fl0), s1 = exp((double)fl1), s2 = exp((double)fl2);
  // EWA projection (Eq. 3): J = [[fx/z, 0, -fx (x/z)/z], [0, fy/z, -fy (y/z)/z]],
  // with x/z and y/z limited to +-g W/(2 fx), +-g H/(2 fy) when the guard g
  // is on (the projected centre below is not limited).  With T = J W R_q S
  // the projected covariance is T T^T: no 3x3 covariance is formed.
  const double fx = cam.fx, fy = cam.fy;
  const double iz = 1.0 / (ok ? z : 1.0);
  const double px = (fx * x) * iz, py = (fy * y) * iz;
  double gx = px, gy = py;
  if (pc.fov_guard > 0.f) {
    const double lx = (double)pc.fov_guard * (0.5 * (double)vi.W), ly = (double)pc.fov_guard * (0.5 * (double)vi.H);
    gx = fx >= 0.0 ? fmin(lx, fmax(-lx, px)) : lx;
    gy = fy >= 0.0 ? fmin(ly, fmax(-ly, py)) : ly;
  }
  const double J00 = fx * iz, J02 = -gx * iz;
  const double J11 = fy * iz, J12 = -gy * iz;
  double T0[3], T1[3];
  {
    const double P0[3] = {fma(J00, W0, J02 * W6), fma(J00, W1, J02 * W7), fma(J00, W2, J02 * W8)};
    const double P1[3] = {fma(J11, W3, J12 * W6), fma(J11, W4, J12 * W7), fma(J11, W5, J12 * W8)};
    const double sc[3] = {s0, s1, s2};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      T0[k] = fma(P0[0], Rq[k], fma(P0[1], Rq[3 + k], P0[2] * Rq[6 + k])) * sc[k];
      T1[k] = fma(P1[0], Rq[k], fma(P1[1], Rq[3 + k], P1[2] * Rq[6 + k])) * sc[k];
    }
  }
  const double A = fma(T0[0], T0[0], fma(T0[1], T0[1], T0[2] * T0[2])) + (double)pc.lowpass;
  const double B = fma(T0[0], T1[0], fma(T0[1], T1[1], T0[2] * T1[2]));
  const double C = fma(T1[0], T1[0], fma(T1[1], T1[1], T1[2] * T1[2])) + (double)pc.lowpass;
  const double det = A * C - B * B;
  ok = ok && (det > 0.0);

  const double u = px + (double)cam.cx;
  const double v = py + (double)cam.cy;

  int tx0 = 0, tx1 = vi.TX - 1, ty0 = 0, ty1 = vi.TY - 1;
  if (!(pc.flags & GSR_FULL_RECT) && ok) {
    const double rx = (double)pc.cutoff * sqrt(A), ry = (double)pc.cutoff * sqrt(C);
    const double bx0 = floor((u - rx) / (double)TILE), bx1 = floor((u + rx) / (double)TILE);
    const double by0 = floor((v - ry) / (double)TILE), by1 = floor((v + ry) / (double)TILE);
    const double cx0 = fmax(0.0, bx0), cx1 = fmin((double)(vi.TX - 1), bx1);
    const double cy0 = fmax(0.0, by0), cy1 = fmin((double)(vi.TY - 1), by1);
    ok = ok && (cx0 <= cx1) && (cy0 <= cy1);
    if (ok) {
      tx0 = (int)cx0; tx1 = (int)cx1; ty0 = (int)cy0; ty1 = (int)cy1;
    }
  }

  if (!ok) return false;
  // Only records that enter tile lists receive or give back 2D gradients.
  // (whole cache lines are written here and below, pads included: a line
  // written in part is read first)
  if (pc.clear_grads) {
    double2 *gz = reinterpret_cast<double2 *>(ws.grad2d + rec * GEO_ROW);
#pragma unroll
    for (int k = 0; k < GEO_ROW / 2; ++k) gz[k] = make_double2(0.0, 0.0);
    if (pc.clear_grads > 1) {
      double2 *gc = reinterpret_cast<double2 *>(ws.grad_col + rec * COL_ROW);
#pragma unroll
      for (int k = 0; k < COL_ROW / 2; ++k) gc[k] = make_double2(0.0, 0.0);
    }
  }
  const float zf = (float)z;
  const float uh = (float)u, vh = (float)v;
  const float op = (float)(1.0 / (1.0 + exp(-(double)fop)));
  const float4 fa = make_float4(uh, (float)(u - (double)uh), vh, (float)(v - (double)vh));
  const double idet = 1.0 / det;
  const float4 fb = make_float4((float)(C * idet), (float)(-B * idet), (float)(A * idet), op);
  float fc0 = col[0], fc1 = col[1], fc2 = col[2];
  if constexpr (SH) {
    // Degree-1 spherical harmonics of the viewing direction d from the
    // camera centre -W^T t to the mean: Y_0 = 1/(2 sqrt(pi)),
    // (Y_1, Y_2, Y_3) = sqrt(3/(4 pi)) (d_y, d_z, d_x).
    const double t0 = cam.t[0], t1 = cam.t[1], t2 = cam.t[2];
    const double vx = mx + ((W0 * t0 + W3 * t1) + W6 * t2);
    const double vy = my + ((W1 * t0 + W4 * t1) + W7 * t2);
    const double vz = mz + ((W2 * t0 + W5 * t1) + W8 * t2);
    const double il = 1.0 / sqrt((vx * vx + vy * vy) + vz * vz);
    const double Y0 = SH_C0, Y1 = SH_C1 * (vy * il), Y2 = SH_C1 * (vz * il), Y3 = SH_C1 * (vx * il);
    double c[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
      c[ch] = ((Y0 * (double)col[ch] + Y1 * (double)col[3 + ch]) + Y2 * (double)col[6 + ch]) + Y3 * (double)col[9 + ch];
    fc0 = (float)c[0];
    fc1 = (float)c[1];
    fc2 = (float)c[2];
  }
  float4 *row = ws.rec + rec * REC_ROW;
  row[0] = fa;
  row[1] = fb;
  row[2] = make_float4(fc0, fc1, fc2, zf);
  row[3] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (args->cull) {
    Support sp;
    if (!support_of(fa, fb, pc.inv_alpha_min, sp)) {
      sp.U = sp.V = sp.t = sp.dys = sp.ra = 0.0;
      sp.hy = -1.0;  // no row reaches it
    }
    *support = sp;
  }
  out->a = fb.x;
  out->b = fb.y;
  out->c = fb.z;
  out->key = __float_as_uint(zf);
  out->rec = (uint32_t)rec;
  out->tx0 = (uint16_t)tx0;
  out->tx1 = (uint16_t)tx1;
  out->ty0 = (uint16_t)ty0;
  out->ty1 = (uint16_t)ty1;
  return true;
}

// One block per `rounds` x PRE_BLOCK Gaussians of one view: an early test
// drops most of the records outside the view (a third to four fifths of a room
// seen from inside), and the rest, packed into full wavefronts, go through the
// projection in batches of PRE_BLOCK.  Then the block writes an entry of every
// visible one for every bin of tiles it reaches, in three steps spread evenly
// over the block whatever the records' sizes: the column range inside the alpha
// support of every tile row of every record (FP64, once; ROW_CACHE rows are
// kept in LDS, the rest found again where they are used); then, per bin row of
// every record, the entries per bin are counted (lds_bins bins at a time) and
// one global add reserves the batch's place; then they are written grouped by
// bin, from the list that the count kept of them (in the supports' place) or,
// where that does not hold them all, by walking the bin rows again.
// Bound by the latency of these phases where the grid is about a block a CU
// (2 048 records of 160x120 and 300 000 of 1200x680: 24 and 44 us before the
// early test read its rounds together, rows and bin rows knew their record
// without a search and the second sweep gave way to the list; 19 and 36 now),
// by memory over many views: 36 M records in 72 views wrote 3.5 GB in 1.9 ms
// with records in three arrays and gradient rows of 80 bytes (lines written in
// part), and write 2.65 GB in 1.45 ms in whole cache lines with bits for the
// visible ones.
constexpr int ROW_CACHE = 3072;
constexpr int UNIT_CACHE = 2048;  // bin rows whose record is kept

// An entry of the batch: its record and mask, its bin and its number there.
struct Item {
  uint16_t rec, mask, bin, at;
};
constexpr int ITEMS = PRE_BLOCK * (int)(sizeof(Support) / sizeof(Item));
static_assert(BIN_MAX * BIN_MAX <= 16 && ITEMS <= 65536, "16-bit fields");

// Column range of one tile row of a record: first column | length << 16 (length
// 0 where the alpha support does not reach the row).
__device__ __forceinline__ uint32_t row_range(const Staged &t, const Support &sp, bool cull, int ty) {
  int c0 = t.tx0, len = (int)t.tx1 - (int)t.tx0 + 1;
  if (cull) {
    c0 = 0;
    len = support_row(sp, (double)t.a, (double)t.b, (double)t.c, ty, t.tx0, t.tx1, c0);
  }
  return (uint32_t)c0 | (uint32_t)len << 16;
}

// Last of the n ascending values first[] that is <= i.
__device__ __forceinline__ int owner_of(const uint32_t *first, int n, uint32_t i) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= i) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Mask of the tiles of bin column bx that the rows cover (bit r S + column).
__device__ __forceinline__ uint32_t unit_mask(const uint32_t rows[BIN_MAX], int bx, int shift) {
  const int S = 1 << shift;
  uint32_t m = 0u;
#pragma unroll
  for (int r = 0; r < BIN_MAX; ++r) {
    const int c0 = (int)(rows[r] & 0xFFFFu), len = (int)(rows[r] >> 16);
    const int a = max(c0 - (bx << shift), 0), b = min(c0 + len - (bx << shift), S);
    if (b > a) m |= ((1u << b) - (1u << a)) << (r * S);
  }
  return m;
}

template <bool SH>
__global__ __launch_bounds__(PRE_BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_preprocess(gsr_gaussians g, const gsr_camera *__restrict__ cams,
                                                          const ViewInfo *__restrict__ views, PreConsts pc,
                                                          Workspace ws, int bpv, int rounds, int lds_bins,
                                                          unsigned long long cap, int shared_bins) {
  constexpr int NW = PRE_BLOCK / 64;
  extern __shared__ uint32_t s_cur[];  // [lds_bins]
  __shared__ ProjArgs s_args;
  __shared__ Staged s_rec[PRE_BLOCK];  // the records of a batch (the visible ones filled in)
  __shared__ union {
    Support support[PRE_BLOCK];
    Item item[ITEMS];
  } s_u;
  __shared__ uint16_t s_unit[UNIT_CACHE];
  __shared__ uint32_t s_first[PRE_BLOCK];
  __shared__ uint32_t s_rowat[PRE_BLOCK];  // first tile row of each record
  __shared__ uint32_t s_rows[ROW_CACHE];
  __shared__ uint16_t s_left[PRE_BLOCK * PRE_ROUNDS_MAX];  // records the early test leaves
  __shared__ uint32_t s_visible[PRE_ROUNDS_MAX * PRE_BLOCK / 32];
  __shared__ uint32_t s_w[NW];
  __shared__ unsigned long long s_pairs[NW];
  __shared__ uint32_t s_base, s_nleft, s_nitem, s_used;
  const int view = blockIdx.x / bpv, blk = blockIdx.x - view * bpv;
  const ViewInfo vi = views[view];
  const gsr_camera &cam = cams[view];
  const int wave = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blk * PRE_BLOCK * rounds;
  const int64_t rec0 = (int64_t)view * g.n;
  // Every tile of a record's rectangle is a pair; the lists leave out the
  // tiles its alpha support does not reach (none in the full-rectangle mode
  // or without an alpha threshold).
  const bool cull = !(pc.flags & GSR_FULL_RECT) && pc.alpha_min > 0.f;
  if (threadIdx.x < PRE_ROUNDS_MAX * PRE_BLOCK / 32) s_visible[threadIdx.x] = 0u;
  for (int b = blockIdx.x * PRE_BLOCK + threadIdx.x; b < shared_bins; b += gridDim.x * PRE_BLOCK) ws.shared_place[b] = 0ull;
  if (threadIdx.x == 0) {
    s_used = header_used(ws.hdr) ? 1u : 0u;
    if (blockIdx.x == 0) reset_header_words(ws.hdr);  // (read by the kernels behind this one)
    s_nleft = 0u;
    s_args = ProjArgs{g, vi, pc, ws.rec, ws.grad2d, ws.grad_col, cull ? 1 : 0};
  }
  __syncthreads();
  {
    const float norm2 = norm2_bound(cam.R);
    // (the reads of all rounds are in flight together)
    Early e[PRE_ROUNDS_MAX];
#pragma unroll
    for (int r = 0; r < PRE_ROUNDS_MAX; ++r) {
      const int64_t i = i0 + r * PRE_BLOCK + threadIdx.x;
      if (r < rounds && i < g.n) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          e[r].m[k] = g.mean[3 * i + k];
          e[r].ls[k] = g.log_scale[3 * i + k];
        }
        e[r].keep = g.mask ? g.mask[i] : 1;
      }
    }
#pragma unroll
    for (int r = 0; r < PRE_ROUNDS_MAX; ++r) {
      if (r >= rounds) break;
      const int64_t i = i0 + r * PRE_BLOCK + threadIdx.x;
      bool left = false;
      if (i < g.n) left = !surely_culled(e[r], cam, vi, pc, norm2);
      const uint64_t m = __ballot(left);
      uint32_t at = 0u;
      if ((threadIdx.x & 63) == 0 && m) at = atomicAdd(&s_nleft, (uint32_t)__popcll(m));
      at = __shfl(at, 0);
      if (left) s_left[at + (uint32_t)__popcll(m & lanemask_lt())] = (uint16_t)(r * PRE_BLOCK + threadIdx.x);
    }
  }
  __syncthreads();
  const int nleft = (int)s_nleft;
  const int shift = vi.bin_shift, S = 1 << shift, nb = vi.BX * vi.BY;
  unsigned long long pairs = 0ull;
  uint32_t largest = 0u;  // the batches' largest groups among this thread's bins, summed
  for (int batch = 0; batch < rounds; ++batch) {
    const int group = blockIdx.x * rounds + batch;
    if (batch * PRE_BLOCK >= nleft) {
      if (threadIdx.x == 0) ws.block_base[group] = NO_BASE;
      continue;
    }
    const int k = batch * PRE_BLOCK + (int)threadIdx.x;
    const int nrec = min(nleft - batch * PRE_BLOCK, PRE_BLOCK);
    bool vis = false;
    if (k < nleft) {
      const int local = s_left[k];
      const int64_t i = i0 + local;
      vis = project_record<SH>(&s_args, &cam, i, rec0 + i, &s_rec[threadIdx.x], &s_u.support[threadIdx.x]);
      if (vis) atomicOr(&s_visible[local >> 5], 1u << (local & 31));
    }
    uint32_t units, tile_rows;
    {
      // (records without rows share the next one's first row and unit)
      uint32_t nu = 0u, nr = 0u;
      if (vis) {
        const Staged &t = s_rec[threadIdx.x];
        nr = (uint32_t)(t.ty1 - t.ty0 + 1);
        nu = (uint32_t)((t.ty1 >> shift) - (t.ty0 >> shift) + 1);
        pairs += (unsigned long long)(t.tx1 - t.tx0 + 1) * nr;
      }
      if (threadIdx.x == 0) s_nitem = 0u;
      const uint32_t u0 = block_exclusive_scan<PRE_BLOCK>(nu, s_w, units);
      const uint32_t r0 = block_exclusive_scan<PRE_BLOCK>(nr, s_w, tile_rows);
      s_first[threadIdx.x] = u0;
      s_rowat[threadIdx.x] = r0;
      // The rows and bin rows in the caches name their record.
      for (uint32_t u = u0; u < min(u0 + nu, (uint32_t)UNIT_CACHE); ++u) s_unit[u] = (uint16_t)threadIdx.x;
      for (uint32_t u = r0; u < min(r0 + nr, (uint32_t)ROW_CACHE); ++u) s_rows[u] = threadIdx.x;
    }
    __syncthreads();
    for (uint32_t u = threadIdx.x; u < min(tile_rows, (uint32_t)ROW_CACHE); u += PRE_BLOCK) {
      const int o = (int)s_rows[u];
      s_rows[u] = row_range(s_rec[o], s_u.support[o], cull, s_rec[o].ty0 + (int)(u - s_rowat[o]));
    }
    __syncthreads();
    // The supports are needed no more, unless rows are to be found again.
    const bool listing = tile_rows <= (uint32_t)ROW_CACHE && nb <= lds_bins;
    uint32_t *row = ws.group_off + vi.mat_off + ((int64_t)blk * rounds + batch) * (nb + 1);
    uint32_t carry = 0u, most = 0u;
    // Sweep 0 over all bins (counts and offsets), then sweep 1 (entries).
    for (int sweep = 0; sweep < 2; ++sweep) {
      for (int c0 = 0; c0 < nb; c0 += lds_bins) {
        const int cn = min(lds_bins, nb - c0);  // bins of this turn
        if (sweep == 0) {
          for (int b = threadIdx.x; b < cn; b += PRE_BLOCK) s_cur[b] = 0u;
          __syncthreads();
        } else if (nb > lds_bins) {
          for (int b = threadIdx.x; b < cn; b += PRE_BLOCK) s_cur[b] = row[c0 + b];
          __syncthreads();
        }
        for (uint32_t u = threadIdx.x; u < units; u += PRE_BLOCK) {
          const int o = u < (uint32_t)UNIT_CACHE ? (int)s_unit[u] : owner_of(s_first, nrec, u);
          const Staged &t = s_rec[o];
          const int by = (t.ty0 >> shift) + (int)(u - s_first[o]);
          uint32_t rows[BIN_MAX];
#pragma unroll
          for (int r = 0; r < BIN_MAX; ++r) {
            const int ty = (by << shift) + r;
            rows[r] = 0u;
            if (r < S && ty >= (int)t.ty0 && ty <= (int)t.ty1) {
              const uint32_t at = s_rowat[o] + (uint32_t)(ty - (int)t.ty0);
              rows[r] = at < (uint32_t)ROW_CACHE ? s_rows[at] : row_range(t, s_u.support[o], cull, ty);
            }
          }
          for (int bx = t.tx0 >> shift; bx <= t.tx1 >> shift; ++bx) {
            const int b = by * vi.BX + bx - c0;
            if (b < 0 || b >= cn) continue;
            const uint32_t m = unit_mask(rows, bx, shift);
            if (m == 0u) continue;
            const uint32_t p = atomicAdd(&s_cur[b], 1u);
            if (sweep == 1) {
              ws.entries[s_base + p] = Entry{t.key, t.rec, m};
            } else if (listing) {
              const uint32_t k = atomicAdd(&s_nitem, 1u);
              if (k < (uint32_t)ITEMS) s_u.item[k] = Item{(uint16_t)o, (uint16_t)m, (uint16_t)b, (uint16_t)p};
            }
          }
        }
        __syncthreads();
        if (sweep == 0) {
          for (int b0 = 0; b0 < cn; b0 += PRE_BLOCK) {
            const int b = b0 + (int)threadIdx.x;
            uint32_t total;
            const uint32_t count = b < cn ? s_cur[b] : 0u;
            most = max(most, count);
            const uint32_t pre = block_exclusive_scan<PRE_BLOCK>(count, s_w, total) + carry;
            if (b < cn) {
              s_cur[b] = pre;
              row[c0 + b] = pre;
            }
            carry += total;
          }
          __syncthreads();
        }
      }
      if (sweep == 0) {
        largest += most;
        if (threadIdx.x == 0) {
          row[nb] = carry;
          uint32_t base = NO_BASE;
          if (carry > 0u) {
            const unsigned long long at = reserve_entries(ws.hdr, s_used != 0u, carry);
            if (at + carry <= cap) base = (uint32_t)at;
          }
          ws.block_base[group] = base;
          s_base = base;
        }
        __syncthreads();
        if (s_base == NO_BASE) break;
        if (listing && carry <= (uint32_t)ITEMS) {
          for (uint32_t k = threadIdx.x; k < carry; k += PRE_BLOCK) {
            const Item it = s_u.item[k];
            const Staged &t = s_rec[it.rec];
            ws.entries[s_base + s_cur[it.bin] + it.at] = Entry{t.key, t.rec, it.mask};
          }
          break;
        }
      }
    }
    __syncthreads();  // the next batch takes the staging
  }
  const int words = rounds * (PRE_BLOCK / 32);
  if ((int)threadIdx.x < words)
    ws.visible[(int64_t)blockIdx.x * words + threadIdx.x] = s_visible[threadIdx.x];
  for (int o = 32; o > 0; o >>= 1) pairs += __shfl_xor(pairs, o);
  largest = (uint32_t)wave_max((int)largest);
  if ((threadIdx.x & 63) == 0) s_pairs[wave] = pairs | (unsigned long long)largest << PAIRS_BITS;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NW; ++w) {
      pairs += s_pairs[w] & PAIRS_MASK;
      largest = max(largest, (uint32_t)(s_pairs[w] >> PAIRS_BITS));
    }
    ws.block_pairs[blockIdx.x] = pairs | (unsigned long long)largest << PAIRS_BITS;
  }
}

void launch_preprocess(const Plan &p, const gsr_gaussians &g, const gsr_camera *cams, const ViewInfo *views,
                       const gsr_config &cfg, const Workspace &ws, bool clear_grads, hipStream_t s) {
  PreConsts pc{cfg.z_near, cfg.lowpass, cfg.cutoff_sigma, cfg.flags, cfg.fov_guard, cfg.alpha_min,
               cfg.alpha_min > 0.f ? 1.0 / (double)cfg.alpha_min : 0.0, clear_grads ? ((cfg.flags & GSR_GAUSS_GRAD) || g.sh ? 2 : 1) : 0};
  if (g.n > 0)
    hipLaunchKernelGGL(g.sh ? k_preprocess<true> : k_preprocess<false>,
                       dim3((unsigned)(p.blocks_per_view * p.n_views)), dim3(PRE_BLOCK), (size_t)4 * p.lds_bins, s, g,
                       cams, views, pc, ws, p.blocks_per_view, p.pre_rounds, p.lds_bins,
                       (unsigned long long)p.capacity, p.lists_helpers > 0 ? p.total_bins : 0);
}

// Reliable-Gaussian selection (Eq. 12): compare each centre's camera depth
// with the observed depth at the nearest pixel.
__global__ __launch_bounds__(BLOCK) void k_select_reliable(gsr_gaussians g, const gsr_camera *__restrict__ cam,
                                                           const float *__restrict__ depth, int W, int H,
                                                           double eps, double z_near, uint8_t *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i >= g.n) return;
  uint8_t keep = 1;
  if (g.mask && g.mask[i] == 0) {
    keep = 0;
  } else {
    const double mx = g.mean[3 * i], my = g.mean[3 * i + 1], mz = g.mean[3 * i + 2];
    const float *R = cam->R;
    const double x = (((double)R[0] * mx + (double)R[1] * my) + (double)R[2] * mz) + (double)cam->t[0];
    const double y = (((double)R[3] * mx + (double)R[4] * my) + (double)R[5] * mz) + (double)cam->t[1];
    const double z = (((double)R[6] * mx + (double)R[7] * my) + (double)R[8] * mz) + (double)cam->t[2];
    if (z > z_near) {
      const double u = ((double)cam->fx * x) / z + (double)cam->cx;
      const double v = ((double)cam->fy * y) / z + (double)cam->cy;
      const double pxd = floor(u + 0.5), pyd = floor(v + 0.5);
      if (pxd >= 0.0 && pxd < (double)W && pyd >= 0.0 && pyd < (double)H) {
        const double D = depth[(int64_t)pyd * W + (int64_t)pxd];
        if (D > 0.0 && fabs(D - z) > eps) keep = 0;
      }
    }
  }
  out[i] = keep;
}

void launch_select_reliable(const gsr_gaussians &g, const gsr_camera *cam, const float *depth, int W, int H,
                            float eps, float z_near, uint8_t *out, hipStream_t s) {
  if (g.n > 0)
    hipLaunchKernelGGL(k_select_reliable, dim3((unsigned)((g.n + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s, g, cam,
                       depth, W, H, (double)eps, (double)z_near, out);
}

}  // namespace gsr
