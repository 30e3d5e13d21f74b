// Per-tile compositing: front-to-back alpha blending of colour and depth
// (GS-SLAM Eq. 4-5), its backward pass (supplement eq. grad_depth and the
// colour analogue), and the weighted L1 loss gradient (Eq. 6 / Eq. 10).
//
// One 256-thread block (four wave64) renders one 16x16 tile, one thread per
// pixel.  The tile's Gaussians are staged through LDS in batches: each
// thread loads one record, converts its centre to tile-relative FP32
// coordinates (the record keeps the centre as a float pair, so the offset to
// a pixel keeps full precision even at x ~ 1000 px), and pre-scales the
// conic so that alpha = min(alpha_max, o * 2^P) with
// P = a'' dx^2 + 2 b'' dx dy + c'' dy^2 and (a'', b'', c'') = -log2(e)/2 * conic
// (the staged record holds 2 b'').  The forward and the backward evaluate
// alpha with the same inlined function and contraction disabled, so both
// take every threshold decision identically.
#pragma clang fp contract(off)

#include "gsr_internal.h"

namespace gsr {

constexpr int BATCH = 192;  // staged records per forward round (<= BLOCK; the fused kernel's is tunable)
constexpr int FGROUP = 4;   // list entries that the forward walk takes at a time
constexpr int BGROUP = 8;   // and the backward walk (one contraction), in two halves
constexpr int BHALF = 4;
constexpr float NEG_HALF_LOG2E = -0.72134752044448170368f;  // -log2(e) / 2
constexpr float LN2 = 0.69314718055994530942f;
// Alpha threshold of a pixel that has stopped (or lies outside the image):
// above any alpha (alpha <= alpha_max <= 1) and an inline constant of the
// instruction set, so that no register holds it.
constexpr float A_STOPPED = 2.f;

struct Staged {
  float4 geo;  // (u_rel, v_rel, opacity, depth)
  float4 con;  // (a'', 2 b'', c'', unused)
  float4 col;  // (r, g, b, depth)
};

struct TileInfo {
  int view;
  int tx, ty;
  int W, H;
  int64_t pix;     // global pixel index of this thread (valid if inside)
  int64_t HW;      // pixels of the view
  int64_t pix_off; // first pixel of the view
  bool inside;
  int2 range;
  float x0, y0;
};

__device__ __forceinline__ TileInfo tile_info(int tile, const ViewInfo *__restrict__ views,
                                              const int32_t *__restrict__ tile_view,
                                              const int2 *__restrict__ ranges) {
  TileInfo ti;
  ti.view = tile_view[tile];
  const ViewInfo vi = views[ti.view];
  const int local = tile - vi.tile_off;
  ti.ty = local / vi.TX;
  ti.tx = local - ti.ty * vi.TX;
  ti.W = vi.W;
  ti.H = vi.H;
  const int px = ti.tx * TILE + (threadIdx.x & (TILE - 1));
  const int py = ti.ty * TILE + (threadIdx.x >> 4);
  ti.inside = px < vi.W && py < vi.H;
  ti.HW = (int64_t)vi.W * vi.H;
  ti.pix_off = vi.pix_off;
  ti.pix = vi.pix_off + (int64_t)py * vi.W + px;
  ti.range = ranges[tile];
  ti.x0 = (float)(ti.tx * TILE);
  ti.y0 = (float)(ti.ty * TILE);
  return ti;
}

// Load record `id` into this thread's staging slot (three 16-byte loads of one
// cache line).
__device__ __forceinline__ Staged stage_record(uint32_t id, float x0, float y0, const float4 *__restrict__ rec) {
  const float4 *row = rec + (size_t)id * REC_ROW;
  const float4 A = row[0];
  const float4 Bc = row[1];
  const float4 C = row[2];
  Staged s;
  // (u_hi - x0) is exact for |u_hi| < 2^24 and integer x0; the low word adds
  // the remaining bits.
  s.geo = make_float4((A.x - x0) + A.y, (A.z - y0) + A.w, Bc.w, C.w);
  s.con = make_float4(NEG_HALF_LOG2E * Bc.x, 2.f * (NEG_HALF_LOG2E * Bc.y), NEG_HALF_LOG2E * Bc.z, 0.f);
  s.col = C;
  return s;
}

// Staging of list entry t of a batch of cnt: the walks take whole groups, so
// the slots up to the next multiple of BGROUP hold records of opacity 0.
__device__ __forceinline__ int padded(int cnt) { return (cnt + BGROUP - 1) & ~(BGROUP - 1); }

__device__ __forceinline__ Staged empty_record() {
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  return Staged{z, z, z};
}

// alpha of a staged Gaussian at pixel offset (dx, dy) = centre - pixel;
// oG >= 0, so the clamp to [0, alpha_max] is min(oG, alpha_max).
__device__ __forceinline__ float splat_alpha(const float4 &geo, const float3 &con, float dx, float dy,
                                             float alpha_max, float &oG) {
  const float t = __fmaf_rn(con.x, dx, con.y * dy);
  const float P = __fmaf_rn(con.z * dy, dy, dx * t);
  oG = geo.z * __builtin_amdgcn_exp2f(P);
  return __builtin_amdgcn_fmed3f(oG, 0.f, alpha_max);
}

// Geometry of GROUP consecutive staged records, read one group ahead of its
// use: the compiler places the reads next to the use, so a scheduling barrier
// follows them.
template <int G>
struct GroupGeo {
  float4 geo[G];
  float3 con[G];
  __device__ __forceinline__ void load(const Staged *rec) {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      geo[u] = rec[u].geo;
      con[u] = *reinterpret_cast<const float3 *>(&rec[u].con);
    }
  }
};

typedef float float4v __attribute__((ext_vector_type(4)));

// v_mfma_f32_4x4x1_16b_f32: lane l = 4 b + j supplies a (row j) and b (column
// j) of block b; D[i] of the lane is row i, column j: D[i] += a of lane
// 4 b + i * b of lane l.  (All lanes take part, whatever the EXEC mask.)
__device__ __forceinline__ float4v outer4(float a, float b, float4v D) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, D, 0, 0, 0);
}

// Element (j, i) <- (i, j) of the 4x4 matrices that four neighbouring lanes
// hold (D[i] of lane 4 b + j).
__device__ __forceinline__ float4v transpose4(float4v D) {
  const int i = __lane_id() & 3;
  float4v r;
#define GSR_ROW(J)                                                                                              \
  {                                                                                                             \
    float v[4];                                                                                                 \
    for (int k = 0; k < 4; ++k)                                                                                 \
      v[k] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(D[k]), (J) * 0x55, 0xf, 0xf, true));        \
    r[J] = i == 0 ? v[0] : (i == 1 ? v[1] : (i == 2 ? v[2] : v[3]));                                            \
  }
  GSR_ROW(0) GSR_ROW(1) GSR_ROW(2) GSR_ROW(3)
#undef GSR_ROW
  return r;
}

// ------------------------------------------------------------------ forward

struct FwdState {
  float T, C0, C1, C2, D;
  int last;
  float zr;  // depth of the last blended entry (0 if none): the backward's reference depth
};

// Depth of list entry pos of the tile, from the staged batch that starts at
// entry lo when it holds pos, else from the record.
__device__ __forceinline__ float entry_depth(int pos, int lo, const Staged *s_rec, const TileInfo &ti,
                                            const uint32_t *__restrict__ ids, const float4 *__restrict__ rec) {
  if (pos >= lo) return s_rec[pos - lo].geo.w;
  return rec[(size_t)ids[ti.range.x + pos] * REC_ROW + 2].w;
}

// With COUNT, the walk also adds its work to counts (wave totals, once per
// tile): counts[1] += list entries examined by live pixels (including the
// entry that stopped a pixel), counts[2] += entries blended.  The render
// kernels do not count; gsr_work_counts re-walks the lists with counting on.
template <bool COUNT, int NB = BATCH>
__device__ __forceinline__ void tile_forward(const TileInfo &ti, const float4 *__restrict__ rec,
                                             const uint32_t *__restrict__ ids, const RenderConsts &rc,
                                             Staged *s_rec, FwdState &st, unsigned long long *counts,
                                             uint32_t *s_id = nullptr, int *staged_lo = nullptr) {
  st.T = 1.f;
  // Colour and depth, transposed among four lanes: lane 4 b + j holds channel
  // j (r, g, b, depth) of the four pixels 4 b + i (one matrix instruction adds
  // an entry where four FMAs would).
  float4v C = {0.f, 0.f, 0.f, 0.f};
  const float *s_col = reinterpret_cast<const float *>(&s_rec[0].col) + (threadIdx.x & 3);
  constexpr int COL_STRIDE = sizeof(Staged) / sizeof(float);
  st.last = 0;
  st.zr = 0.f;
  // The pixel's alpha threshold; A_STOPPED once it has stopped (or outside
  // the image), so that no later entry is accepted.
  float amin = ti.inside ? rc.alpha_min : A_STOPPED;
  int lo_last = -1;  // first entry of the staged batch (-1: none staged)
  uint32_t nev_w = 0u, nbl_w = 0u;
  const float lx = (float)(threadIdx.x & (TILE - 1));
  const float ly = (float)(threadIdx.x >> 4);
  // This thread's list word of the next batch, loaded one batch ahead.
  uint32_t next_id = 0u;
  static_assert(NB % 64 == 0 && NB <= BLOCK, "whole wavefronts of staging threads");
  if ((int)threadIdx.x < NB && ti.range.x + (int)threadIdx.x < ti.range.y) next_id = ids[ti.range.x + threadIdx.x];
  for (int base = ti.range.x; base < ti.range.y; base += NB) {
    if (__syncthreads_and(amin == A_STOPPED)) break;
    const int pos = base + threadIdx.x;
    const int cnt = min(NB, ti.range.y - base);
    if ((int)threadIdx.x < cnt) {
      const uint32_t id = next_id;
      if (s_id) s_id[threadIdx.x] = id;
      s_rec[threadIdx.x] = stage_record(id, ti.x0, ti.y0, rec);
      if (pos + NB < ti.range.y) next_id = ids[pos + NB];
    } else if ((int)threadIdx.x < padded(cnt)) {
      s_rec[threadIdx.x] = empty_record();
    }
    const int first = base - ti.range.x;
    lo_last = first;
    __syncthreads();
    // Every lane evaluates every entry and keeps or drops the result with
    // selects.  `live` (wave-uniform) holds the lanes still blending; it
    // changes only where a pixel stops, and the wave leaves the batch when it
    // is empty.
    uint64_t live = __builtin_amdgcn_ballot_w64(amin != A_STOPPED);
    GroupGeo<FGROUP> g;
    g.load(s_rec);
    for (int k = 0; k < cnt && live; k += FGROUP) {
      float w[FGROUP], T[FGROUP], alpha[FGROUP], col[FGROUP];
      bool acc[FGROUP];
#pragma unroll
      for (int u = 0; u < FGROUP; ++u) col[u] = s_col[(k + u) * COL_STRIDE];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < FGROUP; ++u) {
        float oG;
        alpha[u] = splat_alpha(g.geo[u], g.con[u], g.geo[u].x - lx, g.geo[u].y - ly, rc.alpha_max, oG);
      }
      g.load(s_rec + min(k + FGROUP, NB - FGROUP));
      __builtin_amdgcn_sched_barrier(0);
      float Tc = st.T;
      int rel = -1;  // last entry of the group that blends
#pragma unroll
      for (int u = 0; u < FGROUP; ++u) {
        acc[u] = alpha[u] >= amin;
        // Blend weight alpha T and the transmittance behind, T - alpha T.
        w[u] = (acc[u] ? alpha[u] : 0.f) * Tc;
        Tc = Tc - w[u];
        T[u] = Tc;
        rel = acc[u] ? u : rel;
      }
      // T never grows: no pixel stops in the group unless its last value is
      // below T_min (that of a stopped pixel is not: it keeps the value that
      // it had in front of the entry that stopped it).
      const uint64_t stop = __builtin_amdgcn_ballot_w64(Tc < rc.T_min);
      uint64_t ran[FGROUP], blends[FGROUP];  // (counted only)
      if (COUNT) {
#pragma unroll
        for (int u = 0; u < FGROUP; ++u) {
          ran[u] = live;
          blends[u] = __builtin_amdgcn_ballot_w64(acc[u]);
        }
      }
      if (stop) {
        bool run = true;
        Tc = st.T;
        rel = -1;
#pragma unroll
        for (int u = 0; u < FGROUP; ++u) {
          const bool a = alpha[u] >= amin;
          if (COUNT) ran[u] = __builtin_amdgcn_ballot_w64(run) & live;
          run = run && !(a && T[u] < rc.T_min);
          w[u] = run ? w[u] : 0.f;
          Tc = run ? T[u] : Tc;
          rel = a && run ? u : rel;
          if (COUNT) blends[u] = __builtin_amdgcn_ballot_w64(a && run);
        }
        amin = run ? amin : A_STOPPED;
        live = __builtin_amdgcn_ballot_w64(amin != A_STOPPED);
      }
      st.T = Tc;
      // (an entry behind the list's end has alpha 0: an alpha_min of 0 accepts it)
      st.last = rel >= 0 ? min(first + k + 1 + rel, first + cnt) : st.last;
#pragma unroll
      for (int u = 0; u < FGROUP; ++u) {
        if (COUNT && k + u < cnt) {
          nev_w += (uint32_t)__popcll(ran[u]);
          nbl_w += (uint32_t)__popcll(blends[u]);
        }
        C = outer4(w[u], col[u], C);
      }
    }
  }
  if (staged_lo) *staged_lo = lo_last;
  // The reference depth: the last blended entry's, read once per pixel (an
  // entry was blended, so a batch was staged).
  if (st.last > 0) st.zr = entry_depth(st.last - 1, lo_last, s_rec, ti, ids, rec);
  if (COUNT && __lane_id() == 0 && nev_w) {
    atomicAdd(counts + 1, (unsigned long long)nev_w);
    atomicAdd(counts + 2, (unsigned long long)nbl_w);
  }
  C = transpose4(C);
  st.C0 = __fmaf_rn(st.T, rc.bg[0], C[0]);
  st.C1 = __fmaf_rn(st.T, rc.bg[1], C[1]);
  st.C2 = __fmaf_rn(st.T, rc.bg[2], C[2]);
  st.D = C[3];
}

// ----------------------------------------------------------------- backward
//
// Per list entry the backward needs, summed over the 256 pixels of the tile,
//   S1 = sum dLdP, Sx = sum dLdP dx, Sy = sum dLdP dy,
//   Sxx = sum dLdP dx^2, Sxy = sum dLdP dx dy, Syy = sum dLdP dy^2,
//   Sc = sum w gC_c (c = r, g, b), Sd = sum w gD,
// with dx = u - x, dy = v - y.  Expanding dx, dy about the tile centre turns
// all of them into moments of two per-pixel values (dLdP and w) against
// per-pixel constants: the matrix [dLdP; w] (entries x pixels) times the
// matrix [1, xc, yc, xc^2, xc yc, yc^2, gC_r, gC_g, gC_b, gD] (pixels x 10),
// a dense contraction over the pixels.  Each wavefront collects dLdP and w of
// BGROUP = 8 entries (16 rows) for its 64 pixels in LDS and contracts them on
// the bf16 matrix cores (v_mfma_f32_16x16x32_bf16, 4 steps); the four
// wavefronts' sums are added at the flush.

constexpr int SUB = 64;                   // entries per backward sub-batch
constexpr int MA_ROWS = 2 * BGROUP;       // high and low parts of (dLdP, w) of a group's entries
constexpr int MA_STRIDE = 64 + 4;         // words (pixels, bf16 pairs) per row (padding spreads LDS banks)
constexpr int MA_WAVE = MA_ROWS * MA_STRIDE;
constexpr int NMOM = 10;                  // per-entry sums kept in LDS

struct BwdIn {
  float T;         // final transmittance
  int last;        // list positions [0, last) to walk
  float zr;        // depth of the last contributor (0 if none)
  float gC0, gC1, gC2, gD, gT;
  // The fused step's upstream colour and depth gradients divided by their
  // weights (sC = gC / w_rgb, sD = gD / w_depth), values that bf16 holds
  // exactly (signs of the L1 residuals).
  float sC0, sC1, sC2, sD;
};

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));

// dLdP and w of one entry at this lane's pixel, each as the sum of two bf16
// (h = x rounded, l = x - h rounded: 16 significant bits, a relative error of
// at most 2^-17): words (h, h) and (l, l) of the pair.  x - h is exact.
__device__ __forceinline__ void split_pair(float dLdP, float w, uint32_t &hi, uint32_t &lo) {
  const float2v x = {dLdP, w};
  const bf16x2 h = __builtin_convertvector(x, bf16x2);
  hi = __builtin_bit_cast(uint32_t, h);
  const float2v r = {dLdP - __uint_as_float(hi << 16), w - __uint_as_float(hi & 0xFFFF0000u)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
}

// Contract the wave's collected rows (rows 2 e and 2 e + 1: the high and low
// words of entry e) with the per-pixel constants B.  A pixel's word is two
// consecutive K slots, dLdP and w: the B entries of the first slot are the
// moment columns, of the second the upstream columns, 0 in the others.  B is
// exact in bf16 for the moment polynomials of half-integer coordinates (at
// most 8 significant bits) and for residual signs; with BLO it is not, and Bl
// holds the low halves (B - Bb rounded to bf16) for a second set of steps.
// K = 128 slots (64 pixels x 2) in 4 steps; step j covers the wave's pixel row
// j.  Lane l supplies A[l % 16][k] and B[k][l % 16] for the 8 slots k of its
// group l / 16; D[i][l % 16] lands in register i % 4 of lane 16 (i / 4) +
// l % 16.  The accumulation is FP32.  (In FP32, v_mfma_f32_16x16x4_f32, the
// 16 steps of a group run on the vector units and cost more than the split.)
template <bool BLO>
__device__ __forceinline__ float4v contract(const uint32_t *mA, const bf16x8 Bb[4], const bf16x8 *Bl) {
  const int lane = __lane_id();
  wave_lds_sync();
  // Lane (g, r): row r, words (pixels) 16 j + 4 g .. + 3 of step j.
  const uint4 *src = reinterpret_cast<const uint4 *>(mA + (lane & 15) * MA_STRIDE + 4 * (lane >> 4));
  bf16x8 a[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = __builtin_bit_cast(bf16x8, src[4 * j]);
  // In registers: the next group may rewrite the rows.
  wave_lds_sync();
  float4v D = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 4; ++j) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], Bb[j], D, 0, 0, 0);
  if constexpr (BLO) {
#pragma unroll
    for (int j = 0; j < 4; ++j) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], Bl[j], D, 0, 0, 0);
  }
  return D;
}

// Store a group's contraction into the wavefront's own per-entry sums
// (sum[e][NMOM]; a wavefront meets each entry once, so plain stores suffice).
// Lane (g, col) holds rows 4g..4g+3: entry 2g (high row, low row) and entry
// 2g+1.  Bit e of used: some pixel of the wave blended entry e; the sums of
// the others are 0 (the products are too, unless an upstream gradient is not
// finite).
__device__ __forceinline__ void store_sums(const float4v &D, uint32_t used, float *sum) {
  const int lane = __lane_id();
  const int g = lane >> 4;
  const int col = lane & 15;
  if (col < NMOM) {
    const uint32_t u = used >> (2 * g);
    sum[(2 * g) * NMOM + col] = (u & 1u) ? D[0] + D[1] : 0.f;
    sum[(2 * g + 1) * NMOM + col] = (u & 2u) ? D[2] + D[3] : 0.f;
  }
}

// State of a pixel's backward walk (see tile_backward).
struct BwdPixel {
  float T, B;           // transmittance behind the current entry; blend behind it
  float Kf, zr;
  float gC0, gC1, gC2, gD;
  int last;
  float lx, ly;
};

// The chain of half a group, back to front: dLdP and w of this lane's pixel go
// to its rows.  PLAIN: every lane walks every entry of the half, some lane
// blends each and none has its alpha clamped, which saves the selects.
template <bool PLAIN>
__device__ __forceinline__ void backward_half(const float alpha[BHALF], const float oG[BHALF], const float4v &Q,
                                              int first, const RenderConsts &rc, BwdPixel &px, uint32_t *rows) {
#pragma unroll
  for (int u = BHALF - 1; u >= 0; --u) {
    const bool has = (PLAIN || first + u < px.last) && alpha[u] >= rc.alpha_min;
    // Lanes without a contribution take alpha = 0, which leaves T and B
    // unchanged (1 / (1 - 0) is exactly 1) and gives w = dLdP = 0.
    const float ae = has ? alpha[u] : 0.f;
    const float rinv = __builtin_amdgcn_rcpf(1.f - ae);
    const float Tk = px.T * rinv;  // transmittance in front of this Gaussian
    px.T = Tk;
    const float w = ae * Tk;
    const float QB = PLAIN || has ? Q[u] - px.B : 0.f;
    const float dLda = __fmaf_rn(Tk, QB, px.Kf * rinv);
    px.B = __fmaf_rn(ae, QB, px.B);
    // dL/dP with G = 2^P (the ln 2 and the conic pre-scale are applied at the
    // flush); dL/d(opacity) = dLdP / o there.  Below the clamp o G is alpha.
    const float dLdP = PLAIN || oG[u] <= rc.alpha_max ? dLda * ae : 0.f;
    split_pair(dLdP, w, rows[(2 * u) * MA_STRIDE], rows[(2 * u + 1) * MA_STRIDE]);
  }
}

// One group of entries.  slot: its first entry's place in s_rec, first: in the
// list; g holds the geometry of its upper half, then of the group in front.
// all: every entry lies below the last contributor of every pixel of the wave.
// Returns the entries that some pixel of the wave blends.
__device__ __forceinline__ uint32_t backward_group(const Staged *s_rec, int slot, int first, bool all,
                                                   const RenderConsts &rc, BwdPixel &px, uint32_t *rows,
                                                   GroupGeo<BHALF> &g) {
  static_assert(BHALF == 4, "one outer4 step per channel");
  uint32_t used = 0u;
#pragma unroll
  for (int h = BGROUP / BHALF - 1; h >= 0; --h) {
    float alpha[BHALF], oG[BHALF];
    // Q of the half's four entries at this lane's pixel (see tile_backward):
    // lane 4 b + i supplies the colour of entry i.
    const float3 col = *reinterpret_cast<const float3 *>(&s_rec[slot + h * BHALF + (threadIdx.x & 3)].col);
    float4v Q;
#pragma unroll
    for (int u = 0; u < BHALF; ++u) Q[u] = px.gD * (g.geo[u].w - px.zr);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = BHALF - 1; u >= 0; --u)
      alpha[u] = splat_alpha(g.geo[u], g.con[u], g.geo[u].x - px.lx, g.geo[u].y - px.ly, rc.alpha_max, oG[u]);
    Q = outer4(col.x, px.gC0, Q);
    Q = outer4(col.y, px.gC1, Q);
    Q = outer4(col.z, px.gC2, Q);
    g.load(s_rec + max(slot + (h - 1) * BHALF, 0));
    __builtin_amdgcn_sched_barrier(0);
    uint32_t u4 = 0u;
#pragma unroll
    for (int u = 0; u < BHALF; ++u) u4 |= __builtin_amdgcn_ballot_w64(alpha[u] >= rc.alpha_min) != 0 ? 1u << u : 0u;
    const bool clamped =
        __builtin_amdgcn_ballot_w64(fmaxf(fmaxf(oG[0], oG[1]), fmaxf(oG[2], oG[3])) > rc.alpha_max) != 0;
    if (all && u4 == 15u && !clamped) {
      backward_half<true>(alpha, oG, Q, first + h * BHALF, rc, px, rows + 2 * h * BHALF * MA_STRIDE);
    } else {
      u4 = 0u;
#pragma unroll
      for (int u = 0; u < BHALF; ++u)
        u4 |= __builtin_amdgcn_ballot_w64(first + h * BHALF + u < px.last && alpha[u] >= rc.alpha_min) != 0 ? 1u << u : 0u;
      backward_half<false>(alpha, oG, Q, first + h * BHALF, rc, px, rows + 2 * h * BHALF * MA_STRIDE);
    }
    used |= u4 << (h * BHALF);
  }
  return used;
}

// A dLdP or w that is not finite would reach every sum of its entry, and those
// of entries that its pixel does not blend: 0 times it, in a lane without a
// contribution or beside a 0 of B, is NaN.  So in a wild wavefront (see
// tile_backward) they are taken out of the group's rows in front of the
// contraction, and the sums that they belong to are made NaN behind it.
// Bits 8 + e and 16 + e of the result: the dLdP, resp. w, of entry e was not
// finite at some pixel, the dLdP at one that blends it.  (Found again here, so
// that the walk itself pays one test a group.  Measured in the fused step, which
// needs none: three ragged views, whose longest tile is the tail of the step,
// 282 us without it, 286 with it, 297 with the selects in the walk, 303 with a
// second loop over the groups, which spills 50 registers; 300 000 Gaussians at
// 1200x680 257.5, 256.4, 258.6, 280 us.)
__device__ __forceinline__ uint32_t clean_rows(const Staged *s_rec, int slot, int first, const RenderConsts &rc,
                                               const BwdPixel &px, uint32_t *rows) {
  uint32_t bad = 0u;
#pragma unroll 1
  for (int e = 0; e < BGROUP; ++e) {
    const Staged *r = s_rec + slot + e;
    float oG;
    const float alpha = splat_alpha(r->geo, *reinterpret_cast<const float3 *>(&r->con), r->geo.x - px.lx,
                                    r->geo.y - px.ly, rc.alpha_max, oG);
    const bool has = first + e < px.last && alpha >= rc.alpha_min;
    const uint32_t h = rows[2 * e * MA_STRIDE], l = rows[(2 * e + 1) * MA_STRIDE];
    auto wrong = [](uint32_t x, uint32_t exponent) { return (x & exponent) == exponent; };
    const bool p = wrong(h, 0x7F80u) || wrong(l, 0x7F80u), w = wrong(h, 0x7F800000u) || wrong(l, 0x7F800000u);
    const uint32_t keep = (p ? 0u : 0xFFFFu) | (w ? 0u : 0xFFFF0000u);
    rows[2 * e * MA_STRIDE] = h & keep;
    rows[(2 * e + 1) * MA_STRIDE] = l & keep;
    bad |= (__builtin_amdgcn_ballot_w64(p && has) != 0 ? 0x100u << e : 0u) |
           (__builtin_amdgcn_ballot_w64(w) != 0 ? 0x10000u << e : 0u);
  }
  return bad;
}

// The sums of a group whose clean_rows gave the bits of bad: moments from dLdP,
// the others from w.
__device__ __forceinline__ void spoil_sums(uint32_t bad, float *sum) {
  for (int k = __lane_id(); k < BGROUP * NMOM; k += 64) {
    const int e = k / NMOM, f = k - e * NMOM;
    if (bad >> ((f < 6 ? 8 : 16) + e) & 1u) sum[k] = __builtin_nanf("");
  }
}

// Walk the tile's list back to front; per entry, dLdP and w of every pixel
// go through the contraction above, and the flush turns the per-entry sums
// into the 2D gradients, added to grad2d with one FP64 atomic per field (a
// Gaussian that covers many tiles sums partials of both signs; the FP64 sum
// keeps the result independent of the order the tiles finish in).  grad2d
// fields: (u, v, conic a, b, c, depth, opacity), grad_col: (r, g, b).
//
// Without BLO (the fused step) the upstream columns are the residual signs
// in.sC / in.sD and the colour and depth sums are scaled by w_rgb and
// w_depth at the flush; with BLO (the separate backward, any upstream
// gradient) they are in.gC / in.gD themselves, split into high and low bf16
// halves like the A values.
template <bool BLO>
__device__ __forceinline__ void tile_backward(const TileInfo &ti, const float4 *__restrict__ rec,
                                              const uint32_t *__restrict__ ids, const RenderConsts &rc,
                                              const BwdIn &in, double *__restrict__ grad2d, double *__restrict__ grad_col,
                                              Staged *s_rec, float *s_part, uint32_t *s_id, int *s_max,
                                              float *s_mA, int staged_lo = -1, float w_rgb = 1.f,
                                              float w_depth = 1.f) {
  const float lx = (float)(threadIdx.x & (TILE - 1));
  const float ly = (float)(threadIdx.x >> 4);
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float *mA = s_mA + wv * MA_WAVE;
  float *my_part = s_part + wv * SUB * NMOM;  // this wavefront's per-entry sums
  const int wmax = wave_max(in.last);
  const int wmin = INT_MAX - wave_max(INT_MAX - in.last);
  if (lane == 0) s_max[wv] = wmax;
  __syncthreads();
  const int maxlast = __builtin_amdgcn_readfirstlane(max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3])));
  if (maxlast == 0) return;

  // Per-pixel constants of the contraction, in the B-operand layout,
  // coordinates relative to the tile centre.  The upstream gradients reach
  // those lanes through the wave's LDS rows.
  bf16x8 Bb[4];
  bf16x8 Bl[BLO ? 4 : 1];
  {
    // Step j, lane (g, col): elements 2 i and 2 i + 1 hold column col of the
    // moments and of the upstream values of pixel x = 4 g + i of the wave's
    // row j (y = 4 wv + j).
    mA[0 * MA_STRIDE + lane] = BLO ? in.gC0 : in.sC0;
    mA[1 * MA_STRIDE + lane] = BLO ? in.gC1 : in.sC1;
    mA[2 * MA_STRIDE + lane] = BLO ? in.gC2 : in.sC2;
    mA[3 * MA_STRIDE + lane] = BLO ? in.gD : in.sD;
    mA[4 * MA_STRIDE + lane] = 0.f;  // (read by the lanes of the other columns)
    wave_lds_sync();
    // Rebuilt per tile from an opaque copy of the lane index: kept out of
    // the tile loop, these tile-invariant values would be held in registers
    // (or spilled) across the forward walk.
    int lane_t = lane;
    __asm__ volatile("" : "+v"(lane_t));
    const int col = lane_t & 15, g = lane_t >> 4;
    const int row = col >= 6 && col < NMOM ? col - 6 : 4;
    // Moment columns 1, xc, yc, xc^2, xc yc, yc^2: products fx fy.
    float fx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float xc = (float)(4 * g + i) - 7.5f;
      fx[i] = col == 1 || col == 4 ? xc : (col == 3 ? xc * xc : (col < 6 ? 1.f : 0.f));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float yc = (float)(4 * wv + j) - 7.5f;
      const float fy = col == 2 || col == 4 ? yc : (col == 5 ? yc * yc : 1.f);
      const float4v q = *reinterpret_cast<const float4v *>(mA + row * MA_STRIDE + 16 * j + 4 * g);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        Bb[j][2 * i] = (__bf16)(fx[i] * fy);
        Bb[j][2 * i + 1] = (__bf16)q[i];
        if constexpr (BLO) {
          Bl[j][2 * i] = (__bf16)0.f;
          Bl[j][2 * i + 1] = (__bf16)(q[i] - (float)Bb[j][2 * i + 1]);
        }
      }
    }
    wave_lds_sync();
  }

  // Blend behind the current entry, normalised by the transmittance in front
  // of it, enters dL/dalpha only through the upstream-weighted scalar
  //   B = gC . aC + gD . aDs,
  // (aC: colour behind, starting at the background; aDs: depth behind,
  // relative to the depth zr of the pixel's last contributor), which obeys
  // the same recurrence B <- B + alpha (Q - B) with Q = gC . c + gD (z - zr).
  // With the telescoping identity sum_m alpha_m T_m = 1 - T_f,
  //   dL/dalpha_k = T_k (Q_k - B_k) + (gD zr - gT) T_f / (1 - alpha_k).
  // On a surface all depths agree to a few mm, so the shifted terms keep
  // their float32 digits (z_k - aD_k itself would cancel).
  BwdPixel px;
  px.T = in.T;
  px.B = in.gC0 * rc.bg[0] + in.gC1 * rc.bg[1] + in.gC2 * rc.bg[2];
  px.Kf = (in.gD * in.zr - in.gT) * in.T;
  px.zr = in.zr;
  px.gC0 = in.gC0;
  px.gC1 = in.gC1;
  px.gC2 = in.gC2;
  px.gD = in.gD;
  px.last = in.last;
  px.lx = lx;
  px.ly = ly;
  // Wild: some pixel's upstream gradient is infinite or NaN (or so large that a
  // product might be), or its transmittance has reached 0, which the walk
  // divides.  Only the sums of the Gaussians that the pixel blends may see it,
  // and of these only the ones that it enters.  (Not in the fused step, whose
  // upstream gradients are the weights with a sign; an alpha of exactly 1, which
  // alone makes a 0 that is divided by 0, spoils the sums in front there.)
  const bool wild = BLO && __builtin_amdgcn_ballot_w64(!(fabsf(px.gC0) + fabsf(px.gC1) + fabsf(px.gC2) + fabsf(px.gD) +
                                                  fabsf(px.Kf) < 1e30f) || !(px.T > 0.f)) != 0;

  // Sub-batches [b SUB, (b + 1) SUB), walked from the last one that holds
  // an entry below maxlast.  Those inside the forward's last batch (still
  // staged, records and ids, from list position staged_lo on) are read in
  // place; the others are staged into the first SUB slots.
  uint32_t next_id = 0u;  // list word of this thread's slot in sub-batch next_lo, loaded ahead
  int next_lo = -1;
  for (int lo = ((maxlast - 1) / SUB) * SUB; lo >= 0; lo -= SUB) {
    const int hi = min(lo + SUB, maxlast);
    const int cnt = hi - lo;
    int off = 0;  // slot of entry lo in s_rec / s_id
    if (staged_lo >= 0 && lo >= staged_lo) {
      off = lo - staged_lo;
    } else {
      staged_lo = -1;
      if ((int)threadIdx.x < cnt) {
        const uint32_t id = next_lo == lo ? next_id : ids[ti.range.x + lo + threadIdx.x];
        s_id[threadIdx.x] = id;
        s_rec[threadIdx.x] = stage_record(id, ti.x0, ti.y0, rec);
      } else if ((int)threadIdx.x < padded(cnt)) {
        s_rec[threadIdx.x] = empty_record();
      }
    }
    if (lo >= SUB && !(staged_lo >= 0 && lo - SUB >= staged_lo)) {
      if ((int)threadIdx.x < SUB) next_id = ids[ti.range.x + lo - SUB + threadIdx.x];
      next_lo = lo - SUB;
    }
    // This wavefront's groups of the sub-batch, from the one that holds the
    // last contributor of any of its pixels; the entries behind keep zero sums.
    const int ng = (min(max(wmax - lo, 0), cnt) + BGROUP - 1) / BGROUP;
    {
      float4 *z = reinterpret_cast<float4 *>(my_part);
      for (int k = ng * (BGROUP * NMOM / 4) + lane; k < SUB * NMOM / 4; k += 64) z[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    if (ng > 0) {
      // A group's sums are stored behind the next group's walk, so that the
      // matrix cores work beside it.
      uint32_t used = 0u;
      GroupGeo<BHALF> g;
      g.load(s_rec + off + ng * BGROUP - BHALF);
      float4v D = {0.f, 0.f, 0.f, 0.f};
      uint32_t *rows = reinterpret_cast<uint32_t *>(mA);
      for (int q = ng - 1; q >= 0; --q) {
        const int first = lo + q * BGROUP;
        uint32_t now =
            backward_group(s_rec, off + q * BGROUP, first, first + BGROUP <= wmin, rc, px, rows + lane, g);
        if (q < ng - 1) store_sums(D, used, my_part + (q + 1) * BGROUP * NMOM);
        if (__builtin_expect(wild, false)) {
          if (q < ng - 1) spoil_sums(used, my_part + (q + 1) * BGROUP * NMOM);
          now |= clean_rows(s_rec, off + q * BGROUP, first, rc, px, rows + lane);
        }
        D = contract<BLO>(rows, Bb, Bl);
        used = now;
      }
      store_sums(D, used, my_part);
      if (__builtin_expect(wild, false)) spoil_sums(used, my_part);
    }
    __syncthreads();
    // Flush.  First one thread per Gaussian of the batch converts its sums:
    // with the centre relative to the tile centre (uc, vc) and the pixel
    // moments M about it,
    //   Sx = uc M1 - Mx, Sy = vc M1 - My, Sxx = uc^2 M1 - 2 uc Mx + Mxx,
    //   Sxy = uc vc M1 - uc My - vc Mx + Mxy, Syy = vc^2 M1 - 2 vc My + Myy;
    // then dL/du = 2 ln2 (a'' Sx + b'' Sy), dL/dv = 2 ln2 (b'' Sx + c'' Sy)
    // with the pre-scaled conic (a'', b'', c'') = -log2(e)/2 (a, b, c), and
    //   dL/da = -Sxx/2, dL/db = -Sxy, dL/dc = -Syy/2, dL/do = M1 / o.
    // Then the block adds them to grad2d field-parallel: consecutive lanes
    // take consecutive fields of one Gaussian, so each atomic instruction
    // touches a few cache lines.
    double *s_out = reinterpret_cast<double *>(s_mA);  // [SUB][NGRAD2D], free during the flush
    if ((int)threadIdx.x < cnt) {
      // The four wavefronts' sums, added in a fixed order.
      const float *src = s_part + threadIdx.x * NMOM;
      double m[NMOM];
#pragma unroll
      for (int f = 0; f < NMOM; ++f)
        m[f] = (double)((src[f] + src[SUB * NMOM + f]) + (src[2 * SUB * NMOM + f] + src[3 * SUB * NMOM + f]));
      const Staged &sr = s_rec[off + threadIdx.x];
      const double uc = (double)sr.geo.x - 7.5, vc = (double)sr.geo.y - 7.5;
      const double M1 = m[0], Mx = m[1], My = m[2], Mxx = m[3], Mxy = m[4], Myy = m[5];
      const double Sx = uc * M1 - Mx, Sy = vc * M1 - My;
      const double Sxx = (uc * uc * M1 - 2.0 * uc * Mx) + Mxx;
      const double Sxy = ((uc * vc * M1 - uc * My) - vc * Mx) + Mxy;
      const double Syy = (vc * vc * M1 - 2.0 * vc * My) + Myy;
      const double a2 = (double)sr.con.x, b2 = 0.5 * (double)sr.con.y, c2 = (double)sr.con.z;
      double *o = s_out + threadIdx.x * NGRAD2D;
      o[0] = 2.0 * (double)LN2 * (a2 * Sx + b2 * Sy);
      o[1] = 2.0 * (double)LN2 * (b2 * Sx + c2 * Sy);
      o[2] = -0.5 * Sxx;
      o[3] = -Sxy;
      o[4] = -0.5 * Syy;
      o[6] = M1 / (double)sr.geo.z;
      constexpr bool SCALED = !BLO;  // the upstream columns were the residual signs
      o[5] = SCALED ? m[9] * (double)w_depth : m[9];
      o[7] = SCALED ? m[6] * (double)w_rgb : m[6];
      o[8] = SCALED ? m[7] * (double)w_rgb : m[7];
      o[9] = SCALED ? m[8] * (double)w_rgb : m[8];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < cnt * NGRAD2D; t += BLOCK) {
      const int e = t / NGRAD2D, f = t - e * NGRAD2D;
      const double v = s_out[t];
      const size_t id = s_id[off + e];
      double *to = f < GEO_FIELDS ? grad2d + id * GEO_ROW + f : grad_col + id * COL_ROW + (f - GEO_FIELDS);
      if (v != 0.0 && ((rc.grad_fields >> f) & 1u)) atomicAdd(to, v);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ kernels

struct RasterArgs {
  const float4 *rec;
  const uint32_t *ids;
  const int2 *ranges;
  const ViewInfo *views;
  const int32_t *tile_view;
  RenderConsts rc;
};

static RasterArgs raster_args(const Workspace &ws, const ViewInfo *views, const int32_t *tile_view,
                              const RenderConsts &rc) {
  return RasterArgs{ws.rec, ws.ids, ws.ranges, views, tile_view, rc};
}

// Per-pixel forward state that a separate backward reads (the unfused
// forward); all null in the fused step, whose backward keeps it in registers.
struct PixelState {
  float *T;
  int32_t *last;
  float *zr;
};

__device__ __forceinline__ void save_state(const PixelState &ps, int64_t pix, const FwdState &st) {
  if (ps.T) ps.T[pix] = st.T;
  if (ps.last) ps.last[pix] = st.last;
  if (ps.zr) ps.zr[pix] = st.zr;
}

__global__ __launch_bounds__(BLOCK) void k_render_fwd(RasterArgs a, PixelState ps, gsr_images out) {
  __shared__ Staged s_rec[BATCH];
  const TileInfo ti = tile_info(blockIdx.x, a.views, a.tile_view, a.ranges);
  FwdState st;
  tile_forward<false>(ti, a.rec, a.ids, a.rc, s_rec, st, nullptr);
  if (!ti.inside) return;
  save_state(ps, ti.pix, st);
  const int64_t loc = ti.pix - ti.pix_off;
  if (out.rgb) {
    float *o = out.rgb + 3 * ti.pix_off + loc;
    o[0] = st.C0;
    o[ti.HW] = st.C1;
    o[2 * ti.HW] = st.C2;
  }
  if (out.depth) out.depth[ti.pix] = st.D;
  if (out.T_final) out.T_final[ti.pix] = st.T;
  if (out.last) out.last[ti.pix] = st.last;
}

__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_render_bwd(RasterArgs a, const float *__restrict__ T_ws,
                                                      const int32_t *__restrict__ last_ws,
                                                      const float *__restrict__ zr_ws,
                                                      const float *__restrict__ g_rgb,
                                                      const float *__restrict__ g_depth,
                                                      const float *__restrict__ g_T,
                                                      double *__restrict__ grad2d, double *__restrict__ grad_col) {
  // Without a forward in the same kernel the walk stages SUB entries at a time.
  __shared__ Staged s_rec[SUB];
  __shared__ __align__(16) float s_part[4 * SUB * NMOM];
  __shared__ uint32_t s_id[SUB];
  __shared__ int s_max[4];
  __shared__ __align__(16) float s_mA[4 * MA_WAVE];
  const TileInfo ti = tile_info(blockIdx.x, a.views, a.tile_view, a.ranges);
  BwdIn in{1.f, 0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (ti.inside) {
    const int64_t loc = ti.pix - ti.pix_off;
    in.zr = zr_ws[ti.pix];
    in.T = T_ws[ti.pix];
    in.last = last_ws[ti.pix];
    const float *gc = g_rgb + 3 * ti.pix_off + loc;
    in.gC0 = gc[0];
    in.gC1 = gc[ti.HW];
    in.gC2 = gc[2 * ti.HW];
    in.gD = g_depth ? g_depth[ti.pix] : 0.f;
    in.gT = g_T ? g_T[ti.pix] : 0.f;
  }
  tile_backward<true>(ti, a.rec, a.ids, a.rc, in, grad2d, grad_col, s_rec, s_part, s_id, s_max, s_mA);
}

__device__ __forceinline__ float sgnf(float x) { return (float)((x > 0.f) - (x < 0.f)); }

// The walks are bound by the vector units: at 1200x680 (300 000 Gaussians,
// 3 225 tiles) a step evaluates 1.16 M wave-entries in each direction, and a
// wave-entry cost 25 vector instructions forward and 44 backward when entries
// were taken one at a time.  It costs about 17 and 29 now, and k_render_fused
// went from 210 to 160 us (86 % of the vector units' issue slots in use):
//  - records are read a group ahead, and the tile's number, view and list are
//    scalar: 317 -> 290 us a step;
//  - a group asks once whether any of its pixels stops, resp. whether every
//    entry is plain (backward_half), instead of selecting at each entry;
//  - colours run on v_mfma_f32_4x4x1 (an FP32 matrix instruction that uses the
//    vector units, but half the cycles of the four FMAs): 290 -> 283 us;
//  - the two halves of dLdP and w are split as a pair (split_pair).
// Measured and dropped: two pixels a thread (355 us: half the wavefronts and
// 158 registers), the contraction in FP32 (290 us against 274), the residual
// of the split from v_dot2c (the same time).
//
// Persistent fused step: blocks take tiles from an atomic counter (in index
// order, or in the longest-first order of `queue`); per tile run the
// forward blend, the L1 loss gradient of every pixel, and the backward walk
// without leaving the block (per-pixel state stays in registers).  Each
// tile's duration goes to tile_cost, the next step's longest-first order, and
// its loss to tile_loss (summed in tile order at the end of the step).
template <int NB>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_render_fused(RasterArgs a, uint32_t *__restrict__ hdr,
                                                        const uint32_t *__restrict__ queue, int total_tiles,
                                                        int tiles_per_pop, const float *__restrict__ t_rgb,
                                                        const float *__restrict__ t_depth,
                                                        const uint8_t *__restrict__ pmask, float w_rgb,
                                                        float w_depth, const float *__restrict__ loss_cap,
                                                        gsr_images out, float *__restrict__ tile_loss,
                                                        double *__restrict__ grad2d, double *__restrict__ grad_col, PixelState ps,
                                                        uint32_t *__restrict__ tile_cost) {
  __shared__ Staged s_rec[NB];
  __shared__ __align__(16) float s_part[4 * SUB * NMOM];
  __shared__ uint32_t s_id[NB];
  __shared__ int s_max[4];
  __shared__ __align__(16) float s_mA[4 * MA_WAVE];
  __shared__ int s_q;
  __shared__ float s_loss[4];
  for (;;) {
    if (threadIdx.x == 0) s_q = (int)atomicAdd(hdr + HDR_QUEUE, (uint32_t)tiles_per_pop);
    __syncthreads();
    const int q0 = __builtin_amdgcn_readfirstlane(s_q);  // (scalar: so are the tile's number, view and list)
    __syncthreads();
    if (q0 >= total_tiles) break;
    const int q1 = min(q0 + tiles_per_pop, total_tiles);
    for (int q = q0; q < q1; ++q) {
      const int tile = queue ? (int)queue[q] : q;
      const TileInfo ti = tile_info(tile, a.views, a.tile_view, a.ranges);
      const uint64_t clk0 = wall_clock64();
      // The pixel's targets, loaded before the forward walk hides their latency.
      float tc0 = 0.f, tc1 = 0.f, tc2 = 0.f, td = 0.f, cap = __builtin_inff();
      bool m = false;
      if (ti.inside) {
        const float *tc = t_rgb + 3 * ti.pix_off + (ti.pix - ti.pix_off);
        tc0 = tc[0];
        tc1 = tc[ti.HW];
        tc2 = tc[2 * ti.HW];
        td = t_depth[ti.pix];
        m = pmask ? pmask[ti.pix] != 0 : true;
        if (loss_cap) cap = loss_cap[ti.view];
      }
      FwdState st;
      int staged_lo;
      tile_forward<false, NB>(ti, a.rec, a.ids, a.rc, s_rec, st, nullptr, s_id,
                          &staged_lo);
      BwdIn in{st.T, ti.inside ? st.last : 0, st.zr, 0.f, 0.f, 0.f, 0.f, 0.f};
      float lpx = 0.f;
      if (ti.inside) {
        const int64_t loc = ti.pix - ti.pix_off;
        const float e0 = st.C0 - tc0, e1 = st.C1 - tc1, e2 = st.C2 - tc2;
        const bool md = m && td > 0.f;
        const float ed = st.D - td;
        if (m) {
          lpx = w_rgb * (fabsf(e0) + fabsf(e1) + fabsf(e2));
          if (md) lpx += w_depth * fabsf(ed);
        }
        if (out.loss) out.loss[ti.pix] = lpx;
        // Outlier pixels (own loss above the view's cap) are ignored.
        const bool keep = m && !(lpx > cap);
        lpx = keep ? lpx : 0.f;
        if (keep) {
          in.sC0 = sgnf(e0);
          in.sC1 = sgnf(e1);
          in.sC2 = sgnf(e2);
          if (md) in.sD = sgnf(ed);
          in.gC0 = w_rgb * in.sC0;
          in.gC1 = w_rgb * in.sC1;
          in.gC2 = w_rgb * in.sC2;
          in.gD = w_depth * in.sD;
        }
        save_state(ps, ti.pix, st);
        if (out.rgb) {
          float *o = out.rgb + 3 * ti.pix_off + loc;
          o[0] = st.C0;
          o[ti.HW] = st.C1;
          o[2 * ti.HW] = st.C2;
        }
        if (out.depth) out.depth[ti.pix] = st.D;
        if (out.T_final) out.T_final[ti.pix] = st.T;
        if (out.last) out.last[ti.pix] = st.last;
      }
      const float ls = wave_sum(lpx);
      if ((threadIdx.x & 63) == 0) s_loss[threadIdx.x >> 6] = ls;
      tile_backward<false>(ti, a.rec, a.ids, a.rc, in, grad2d, grad_col, s_rec, s_part, s_id, s_max,
                           s_mA, staged_lo, w_rgb, w_depth);
      if (threadIdx.x == 0) {
        tile_loss[tile] = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
        const uint64_t d = wall_clock64() - clk0;
        tile_cost[tile] = d < 0xFFFFFFFFull ? (uint32_t)d : 0xFFFFFFFFu;
        if (blockIdx.x == 0) hdr[HDR_COSTS] = 1u;
      }
      // The next tile may have an empty list (no barrier in its forward):
      // keep its shared-memory writes behind this tile's reads.
      __syncthreads();
    }
  }
}

// Standalone L1 loss gradient for the autograd path (grid.y = view).
__global__ __launch_bounds__(BLOCK) void k_l1(const ViewInfo *__restrict__ views, const float *__restrict__ rgb,
                                              const float *__restrict__ depth,
                                              const float *__restrict__ t_rgb,
                                              const float *__restrict__ t_depth,
                                              const uint8_t *__restrict__ pmask, float w_rgb, float w_depth,
                                              const float *__restrict__ loss_cap,
                                              float *__restrict__ g_rgb, float *__restrict__ g_depth,
                                              float *__restrict__ loss) {
  __shared__ float s_w[4];
  const ViewInfo vi = views[blockIdx.y];
  const int64_t HW = (int64_t)vi.W * vi.H;
  float l = 0.f;
  for (int64_t q = (int64_t)blockIdx.x * BLOCK + threadIdx.x; q < HW; q += (int64_t)gridDim.x * BLOCK) {
    const int64_t pix = vi.pix_off + q;
    const int64_t c0 = 3 * vi.pix_off + q;
    const bool m0 = pmask ? pmask[pix] != 0 : true;
    const float td = t_depth[pix];
    const float ed = depth[pix] - td;
    float e[3];
    float lp = 0.f;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      e[ch] = rgb[c0 + ch * HW] - t_rgb[c0 + ch * HW];
      lp += fabsf(e[ch]);
    }
    lp = w_rgb * lp;
    if (td > 0.f) lp += w_depth * fabsf(ed);
    // Outlier pixels (own loss above the view's cap) are ignored.
    const bool m = m0 && !(loss_cap && lp > loss_cap[blockIdx.y]);
    const bool md = m && td > 0.f;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) g_rgb[c0 + ch * HW] = m ? w_rgb * sgnf(e[ch]) : 0.f;
    g_depth[pix] = md ? w_depth * sgnf(ed) : 0.f;
    l += m ? lp : 0.f;
  }
  l = wave_sum(l);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0 && loss) atomicAdd(loss, (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]));
}

void launch_l1(const Plan &p, const ViewInfo *views, const float *rgb, const float *depth,
               const float *t_rgb, const float *t_depth, const uint8_t *pmask, float w_rgb,
               float w_depth, const float *loss_cap, float *g_rgb, float *g_depth, float *loss, hipStream_t s) {
  const unsigned gx = (unsigned)((p.total_pixels / p.n_views + BLOCK - 1) / BLOCK);
  dim3 grid(gx < 1024 ? (gx < 1 ? 1 : gx) : 1024, (unsigned)p.n_views);
  hipLaunchKernelGGL(k_l1, grid, dim3(BLOCK), 0, s, views, rgb, depth, t_rgb, t_depth, pmask, w_rgb, w_depth,
                     loss_cap, g_rgb, g_depth, loss);
}

void launch_render_forward(const Plan &p, const Workspace &ws, const ViewInfo *views,
                           const int32_t *tile_view, const RenderConsts &rc,
                           const gsr_images *out, hipStream_t s) {
  const RasterArgs a = raster_args(ws, views, tile_view, rc);
  gsr_images o{nullptr, nullptr, nullptr, nullptr, nullptr};
  if (out) o = *out;
  PixelState ps{ws.T_final, ws.last, ws.zr};
  hipLaunchKernelGGL(k_render_fwd, dim3(p.total_tiles), dim3(BLOCK), 0, s, a, ps, o);
}

void launch_render_backward(const Plan &p, const Workspace &ws, const ViewInfo *views,
                            const int32_t *tile_view, const RenderConsts &rc,
                            const float *g_rgb, const float *g_depth, const float *g_T, hipStream_t s) {
  const RasterArgs a = raster_args(ws, views, tile_view, rc);
  hipLaunchKernelGGL(k_render_bwd, dim3(p.total_tiles), dim3(BLOCK), 0, s, a, ws.T_final, ws.last, ws.zr, g_rgb,
                     g_depth, g_T, ws.grad2d, ws.grad_col);
}

void launch_render_fused(const Plan &p, const Workspace &ws, const ViewInfo *views,
                         const int32_t *tile_view, const RenderConsts &rc,
                         const float *t_rgb, const float *t_depth, const uint8_t *pmask, float w_rgb,
                         float w_depth, const float *loss_cap, const gsr_images *out,
                         const Tuning &tun, int num_cus, hipStream_t s) {
  const RasterArgs a = raster_args(ws, views, tile_view, rc);
  gsr_images o{nullptr, nullptr, nullptr, nullptr, nullptr};
  if (out) o = *out;
  int grid = tun.blocks_per_cu * num_cus;
  const int need = (p.total_tiles + tun.tiles_per_pop - 1) / tun.tiles_per_pop;
  if (grid > need) grid = need;
  if (grid < 1) grid = 1;
  PixelState ps{nullptr, nullptr, nullptr};  // the fused backward keeps the forward state in registers
  const uint32_t *queue = tun.lpt_order ? ws.queue : nullptr;
#define GSR_LAUNCH_FUSED(NB_)                                                                                  \
  hipLaunchKernelGGL(k_render_fused<NB_>, dim3(grid), dim3(BLOCK), 0, s, a, ws.hdr, queue, p.total_tiles,            \
                     tun.tiles_per_pop, t_rgb, t_depth, pmask, w_rgb, w_depth, loss_cap, o, ws.tile_loss, ws.grad2d, ws.grad_col, ps,      \
                     ws.tile_cost)
  switch (tun.batch) {
    case 64: GSR_LAUNCH_FUSED(64); break;
    case 128: GSR_LAUNCH_FUSED(128); break;
    case 256: GSR_LAUNCH_FUSED(256); break;
    default: GSR_LAUNCH_FUSED(192); break;
  }
#undef GSR_LAUNCH_FUSED
}

// Totals of the per-pixel work counters: counts[0] pairs, [1] entries the
// forward examined, [2] entries blended, [3] sum of last.
// Work of the last forward, for the roofline: the forward walk of every
// tile again, with counting on and no outputs (the workspace still holds the
// records, lists and ranges of that call).
// The walk also sums every pixel's `last` (the entries the backward walk
// examines) into counts[3], and block 0 copies the pair count into counts[0].
__global__ __launch_bounds__(BLOCK) void k_count_walk(RasterArgs a, const uint32_t *__restrict__ hdr,
                                                      unsigned long long *__restrict__ counts) {
  __shared__ Staged s_rec[BATCH];
  const TileInfo ti = tile_info(blockIdx.x, a.views, a.tile_view, a.ranges);
  FwdState st;
  tile_forward<true>(ti, a.rec, a.ids, a.rc, s_rec, st, counts);
  unsigned long long c = ti.inside ? (unsigned long long)st.last : 0ull;
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(counts + 3, c);
  if (blockIdx.x == 0 && threadIdx.x == 0)
    counts[0] = *reinterpret_cast<const unsigned long long *>(hdr + HDR_NPAIRS);
}

void launch_work_counts(const Plan &p, const Workspace &ws, const ViewInfo *views, const int32_t *tile_view,
                        const RenderConsts &rc, hipStream_t s) {
  launch_fill_u32(reinterpret_cast<uint32_t *>(ws.counts), 0u, 8, s);
  const RasterArgs a = raster_args(ws, views, tile_view, rc);
  if (p.total_tiles > 0)
    hipLaunchKernelGGL(k_count_walk, dim3(p.total_tiles), dim3(BLOCK), 0, s, a, ws.hdr, ws.counts);
}

}  // namespace gsr
