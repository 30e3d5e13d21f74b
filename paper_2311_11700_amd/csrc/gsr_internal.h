// Internal declarations of the gfx950 splatting renderer: the view table,
// the workspace layout, device helpers shared by the kernels, and the kernel
// launchers the C ABI calls.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gsr.h"

namespace gsr {

constexpr int TILE = 16;          // tile edge in pixels
constexpr int BLOCK = 256;        // one thread per pixel of a tile
constexpr int NGRAD2D = 10;       // 2D gradient fields: u, v, conic a, b, c, depth, opacity, r, g, b
constexpr int GEO_FIELDS = 7;     // of these in a geometry row (GEO_ROW doubles, one cache line);
constexpr int GEO_ROW = 8;        // the others in a colour row of COL_ROW
constexpr int COL_ROW = 4;
constexpr int REC_ROW = 4;        // float4s of a record (one cache line)
constexpr int PRE_BLOCK = 512;    // records projected at a time by a projection block
constexpr int PRE_ROUNDS_MAX = 4; // PRE_BLOCKs of records per block, at most
constexpr int BIN_MAX = 4;        // largest bin edge S in tiles
// Entries the lists kernel sorts in LDS at a time (12 bytes each beside 10 KB
// of counters): chosen by gsr_plan in this range.
constexpr int LISTS_CAP_MIN = 4096, LISTS_CAP_MAX = 12288, LISTS_ENTRY_BYTES = 12;
constexpr int RADIX_BITS = 8;     // buckets of the rasteriser's work order
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int EXPAND_CHUNK = 2048;  // pixels per block of the adding step (eight rounds of BLOCK)
// Real spherical harmonics of degree <= 1: 1/(2 sqrt(pi)) and sqrt(3/(4 pi)).
constexpr double SH_C0 = 0.28209479177387814;
constexpr double SH_C1 = 0.48860251190291992;

// Per-view geometry of the concatenated output (device copy lives in the
// context, written at plan time).
struct ViewInfo {
  int32_t W, H, TX, TY;
  int32_t tile_off;   // first global tile id of the view
  int32_t bin_shift;  // log2 of the bins' edge S in tiles (0, 1 or 2)
  int32_t BX, BY;     // bins of the view, ceil(TX / S) x ceil(TY / S)
  int32_t bin_off;    // first global bin id of the view
  int32_t _pad;
  int64_t mat_off;    // first word of the view's group offsets
  int64_t pix_off;    // first pixel of the view in the concatenated images
};

// Header words at the start of the workspace.
enum HeaderWord {
  HDR_NPAIRS = 0,      // u64 (words 0-1): pairs (rectangle tiles) of the last forward
  HDR_REQUIRED = 2,    // u64 (words 2-3): largest pair count seen that overflowed
  HDR_OVERFLOW = 4,    // u32: set when a forward overflowed the pair buffer
  HDR_QUEUE = 5,       // u32: persistent rasteriser work counter
  HDR_MAGIC = 8,       // u32 x 2 (words 8-9): set once the header has been initialised
  HDR_NLISTED = 12,    // u64 (words 12-13): pairs inside the alpha support (the tile lists)
  HDR_COSTS = 14,      // u32: a fused step has recorded every tile's duration (sticky)
  HDR_ENTRIES = 32,    // u64 (words 32-33): bin entries reserved; in a cache line apart from the words above
  HDR_WORDS = 64
};
// Header magic: a workspace whose words 8-9 do not hold it has never been
// used (its sticky words may hold any leftover bytes) and is cleared.
constexpr uint32_t HDR_MAGIC0 = 0x67737248u, HDR_MAGIC1 = 0x2311B700u;

// The cursor of the bin entries: a tag above a count.  The lists kernel leaves
// it at 0 for the next call, so that the projection needs no kernel in front of
// it.  In a workspace that was never used (no magic, which the lists kernel
// writes) the cursor may hold anything: there the blocks start the count with a
// compare-and-swap that only one of them can win.
// A kernel of one block in front that reset it cost every call 2-4 us: a
// forward of 2000 Gaussians at 160x120 74 -> 72 us without it, the fused step
// of 300k at 1200x680 262 -> 258 us.  The word has a cache line of its own, and
// a block looks at the magic, not at the cursor, when it starts: with a read of
// the cursor in each block, among the others' adds, the step took 266 us and
// one over 16 views 2740 us instead of 2615.
constexpr int ENTRY_COUNT_BITS = 44;
constexpr unsigned long long ENTRY_COUNT_MASK = (1ull << ENTRY_COUNT_BITS) - 1ull;
constexpr unsigned long long ENTRY_TAG = 0xA53C7ull << ENTRY_COUNT_BITS;

// ------------------------------------------------------- alpha support
//
// Tiles of a Gaussian's rectangle that it can reach with alpha >= alpha_min.
// Its alpha at a pixel is o exp(-Q/2), Q the conic quadratic form of the
// offset, so it reaches alpha_min only where Q <= t = 2 ln(o / alpha_min);
// a margin of 1e-4 on t keeps tiles where a float32 alpha could round up to
// alpha_min.  Inside one row of tiles the ellipse {Q <= t} meets a
// contiguous run of tiles: the x-range of the ellipse within the row's band
// of pixel-centre rows [16 ty, 16 ty + 15], mapped to the columns whose
// pixel centres [16 tx, 16 tx + 15] it overlaps.  Every input is a stored
// float32 value (centre as hi + lo, conic, opacity), so the runs agree with an
// FP64 reference evaluated in the same order.
struct Support {
  double U, V, t, hy, dys, ra;  // centre, level, half-height, dy of the rightmost point, 1 / a
};

__device__ inline bool support_of(float4 A, float4 B, double inv_alpha_min, Support &s) {
#pragma clang fp contract(off)
  s.U = (double)A.x + (double)A.y;
  s.V = (double)A.z + (double)A.w;
  const double a = (double)B.x, b = (double)B.y, c = (double)B.z;
  const double det = a * c - b * b;
  s.t = 2.0 * log((double)B.w * inv_alpha_min) + 1e-4;
  if (!(det > 0.0) || !(s.t > 0.0)) return false;
  // Half-height sqrt(t a / det); the rightmost point lies at
  // dy = (-b / det) sqrt(t det / c).
  const double r = 1.0 / det, k = s.t * r;
  s.hy = sqrt(k * a);
  s.dys = -b * sqrt(k / c);
  s.ra = 1.0 / a;
  return true;
}

// Run of tile columns of row ty (within [tx0, tx1]) reached by the support
// of the Gaussian with conic (a, b, c): returns its length and writes its
// first column to lo.
__device__ inline int support_row(const Support &s, double a, double b, double c, int ty, int tx0, int tx1,
                                  int &lo) {
#pragma clang fp contract(off)
  const double p = (double)(16 * ty) - s.V, q = (double)(16 * ty + 15) - s.V;
  if (q < -s.hy || p > s.hy) return 0;
  const double dr = fmin(fmax(s.dys, p), q), dl = fmin(fmax(-s.dys, p), q);
  const double br = b * dr, bl = b * dl;
  const double er = fmax(br * br - a * ((c * dr) * dr - s.t), 0.0);
  const double el = fmax(bl * bl - a * ((c * dl) * dl - s.t), 0.0);
  const double R = (-br + sqrt(er)) * s.ra, L = (-bl - sqrt(el)) * s.ra;
  const double clo = fmax(ceil(((s.U + L) - 15.0) * 0.0625), (double)tx0);
  const double chi = fmin(floor((s.U + R) * 0.0625), (double)tx1);
  if (!(clo <= chi)) return 0;
  lo = (int)clo;
  return (int)(chi - clo) + 1;
}

// A record in a bin of tiles: its depth key (float32 bits), its id and the
// tiles of the bin it reaches (bit row S + column).
struct Entry {
  uint32_t key, id, mask;
};
constexpr uint32_t NO_BASE = 0xFFFFFFFFu;
// (a block has at most 2 048 records of 2^24 tiles, and as many entries in a bin)
constexpr int PAIRS_BITS = 48;
constexpr unsigned long long PAIRS_MASK = (1ull << PAIRS_BITS) - 1ull;

// Device pointers into the caller's workspace (computed on the host).
struct Workspace {
  uint32_t *hdr;
  // [n_rec][REC_ROW]: (u_hi, u_lo, v_hi, v_lo), (conic a, b, c, opacity),
  // (r, g, b, camera-frame depth), 0.
  float4 *rec;
  uint32_t *visible;       // [n_views][vis_words] bit i: record i of the view is not culled
  // Bin entries: each projection batch's, grouped by bin, from block_base on;
  // group_off[view][batch][bin] .. [bin + 1] is the bin's group among them.
  Entry *entries;          // [capacity]
  uint32_t *group_off;
  uint32_t *block_base;    // [projection batches] (NO_BASE: none, or past the capacity)
  unsigned long long *block_pairs;  // [projection blocks] pairs (rectangle tiles) of the block's records, and from
                                    // PAIRS_BITS on a bound of its entries in any bin
  uint32_t *ids;           // [capacity] record ids of the tile lists
  unsigned long long *shared_place;  // [total_bins] place of a bin's lists that several blocks write (0: none yet)
  int2 *ranges;            // [total_tiles]
  float *T_final;          // [total_pixels]
  int32_t *last;           // [total_pixels]
  float *zr;               // [total_pixels] depth of the last blended entry (forward -> backward)
  unsigned long long *counts;  // [4] work totals (gsr_work_counts)
  // FP64 sums over tiles: [n_rec][GEO_ROW] (a pose-only step touches only
  // these) and [n_rec][COL_ROW].
  double *grad2d, *grad_col;
  double *pose_part;       // [n_views][6][n_pose_blocks]
  uint32_t *queue;         // [total_tiles] work order of the persistent rasteriser
  unsigned long long *expand_bits;  // [chunks][8][4] adding step: one bit per pixel (ballot words)
  uint32_t *expand_cnt;    // [chunks] adding step: unreliable pixels per chunk, then their exclusive scan
  uint32_t *tile_cost;     // [total_tiles] duration of each tile in the last fused step (10 ns ticks)
  float *tile_loss;        // [total_tiles] loss of each tile in the fused step
};

struct Plan {
  int64_t n = 0;
  int n_views = 0;
  int64_t n_rec = 0;
  int total_tiles = 0;
  int64_t total_pixels = 0;
  int64_t capacity = 0;
  int blocks_per_view = 0; // projection blocks of each view
  int pre_rounds = 1;      // PRE_BLOCKs of records (and batches of entries) per projection block
  int total_bins = 0;
  int lds_bins = 0;        // bins that a projection block counts in LDS at a time
  int lists_cap = 0;       // bin entries that the lists kernel sorts at a time
  int lists_helpers = 0;   // blocks of the lists kernel beside the bins' own, for crowded bins
  int n_pose_blocks = 0;
  int64_t vis_words = 0;   // words of a view's visibility bits
  size_t bytes = 0;
  // byte offsets inside the workspace
  size_t off_hdr, off_rec, off_visible, off_entries, off_group, off_base, off_pairs, off_ids, off_shared, off_ranges,
      off_T, off_last, off_zr, off_grad2d, off_grad_col, off_pose, off_queue, off_counts, off_tile_cost, off_expand_bits,
      off_expand_cnt;
};

struct Tuning {
  int blocks_per_cu = 4;  // four blocks fit a CU (LDS): every resident slot busy
  int tiles_per_pop = 1;
  int lpt_order = 1;
  int batch = 192;  // records staged per forward round of the fused rasteriser (64, 128, 192, 256)
};

// Scalar renderer constants passed by value to kernels.
struct RenderConsts {
  float alpha_min, alpha_max, T_min;
  float bg[3];
  uint32_t grad_fields;  // bit f set: the backward accumulates grad2d field f
};

// ---------------------------------------------------------------- device helpers

__device__ __forceinline__ float wave_sum(float v) {
  // Butterfly over the 64 lanes of a wavefront.
  v += __shfl_xor(v, 32);
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 8);
  v += __shfl_xor(v, 4);
  v += __shfl_xor(v, 2);
  v += __shfl_xor(v, 1);
  return v;
}

// Maximum over the wavefront of v >= 0, in a scalar register.
__device__ __forceinline__ int wave_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));  // row_shr:1
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));  // row_shr:2
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));  // row_shr:4
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));  // row_shr:8
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));  // row_bcast:15
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));  // row_bcast:31
  return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ bool header_used(const uint32_t *hdr) {
  return hdr[HDR_MAGIC] == HDR_MAGIC0 && hdr[HDR_MAGIC + 1] == HDR_MAGIC1;
}

// Per-call header reset (one thread), but for the magic and the entries'
// cursor, which the lists kernel writes.  The overflow flag and required count
// are sticky until gsr_check_overflow reads them; on a workspace's first use
// (no magic yet) they are cleared too.
__device__ __forceinline__ void reset_header_words(uint32_t *hdr) {
  if (!header_used(hdr)) {
    hdr[HDR_REQUIRED] = 0u;
    hdr[HDR_REQUIRED + 1] = 0u;
    hdr[HDR_OVERFLOW] = 0u;
    hdr[HDR_COSTS] = 0u;
  }
  hdr[HDR_NPAIRS] = 0u;
  hdr[HDR_NPAIRS + 1] = 0u;
  hdr[HDR_NLISTED] = 0u;
  hdr[HDR_NLISTED + 1] = 0u;
  hdr[HDR_QUEUE] = 0u;
}

__device__ __forceinline__ unsigned long long *entry_cursor(uint32_t *hdr) {
  return reinterpret_cast<unsigned long long *>(hdr + HDR_ENTRIES);
}

__device__ __forceinline__ unsigned long long read_entry_cursor(uint32_t *hdr) {
  return __hip_atomic_load(entry_cursor(hdr), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// First of n entries; used: header_used at the call's start.  (An untagged
// word changes once, to a tagged one, so the loop runs twice at most.)  Should
// the word of a used workspace hold no tag, the place is past any capacity.
__device__ __forceinline__ unsigned long long reserve_entries(uint32_t *hdr, bool used, uint32_t n) {
  if (!used) {
    unsigned long long seen = read_entry_cursor(hdr);
    while ((seen & ~ENTRY_COUNT_MASK) != ENTRY_TAG) {
      const unsigned long long old = atomicCAS(entry_cursor(hdr), seen, ENTRY_TAG | n);
      if (old == seen) return 0ull;
      seen = old;
    }
  }
  const unsigned long long at = atomicAdd(entry_cursor(hdr), (unsigned long long)n);
  return (at & ~ENTRY_COUNT_MASK) == ENTRY_TAG ? at & ENTRY_COUNT_MASK : 1ull << 62;
}

__device__ __forceinline__ unsigned long long lanemask_lt() {
  const unsigned lane = __lane_id();
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Lanes of the wavefront whose digit equals this lane's digit (and valid).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, int nbits, uint64_t valid) {
  uint64_t m = valid;
  for (int b = 0; b < nbits; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t bb = __ballot(bit);
    m &= bit ? bb : ~bb;
  }
  return m;
}

// Exclusive scan of one value per thread over a block of NT threads; s_w
// holds NT / 64 words.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *s_w, uint32_t &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_w[wave] = x;
  __syncthreads();
  uint32_t pre = 0u, tot = 0u;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const uint32_t c = s_w[w];
    pre += w < wave ? c : 0u;
    tot += c;
  }
  total = tot;
  __syncthreads();
  return pre + x - v;
}

// --------------------------------------------------------------- tile order

// Log-scale bucket of a tile length (eight buckets per octave), 0 .. 255.
__device__ __forceinline__ uint32_t length_bucket(uint32_t x) {
  if (x == 0u) return 0u;
  const int b = 31 - __clz(x);  // floor(log2 x)
  const uint32_t m = b >= 3 ? (x >> (b - 3)) & 7u : (x << (3 - b)) & 7u;
  const uint32_t k = 1u + 8u * (uint32_t)b + m;
  return k < (uint32_t)RADIX ? k : (uint32_t)(RADIX - 1);
}

// Work order of the persistent rasteriser, computed by one block of NT
// threads: with `timed` (the last fused step on this workspace recorded every
// tile's duration in tile_cost) the tiles longest first, by a counting sort
// over length_bucket (order inside a bucket arbitrary; equal buckets inside a
// wavefront grouped by ballot matching, one LDS atomic per group); otherwise
// index order.  The queue is a permutation of the tiles whatever the recorded
// values.  `timed` must be the same in every thread; s_cnt, s_cur hold RADIX
// words and s_w NT / 64.
template <int NT>
__device__ __forceinline__ void order_tiles(const uint32_t *__restrict__ tile_cost, bool timed, int total,
                                            uint32_t *__restrict__ queue, uint32_t *s_cnt, uint32_t *s_cur,
                                            uint32_t *s_w) {
  static_assert(NT >= RADIX && NT % 64 == 0, "one thread per bucket, whole wavefronts");
  if (!timed) {
    for (int t = threadIdx.x; t < total; t += NT) queue[t] = (uint32_t)t;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x < RADIX) s_cnt[threadIdx.x] = 0u;
  __syncthreads();
  for (int base = 0; base < total; base += NT) {
    const int t = base + (int)threadIdx.x;
    const bool valid = t < total;
    const uint32_t d = valid ? length_bucket(tile_cost[t]) : 0u;
    const uint64_t peers = match_digit(d, RADIX_BITS, __ballot(valid));
    if (valid && (peers & lanemask_lt()) == 0ull) atomicAdd(&s_cnt[d], (uint32_t)__popcll(peers));
  }
  __syncthreads();
  // Start of each bucket: the tiles of all longer buckets (bucket RADIX - 1 - k
  // is the k-th in the order).
  {
    const int k = threadIdx.x;
    const uint32_t v = k < RADIX ? s_cnt[RADIX - 1 - k] : 0u;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    uint32_t pre = 0u;
    for (int w = 0; w < wave; ++w) pre += s_w[w];
    if (k < RADIX) s_cur[RADIX - 1 - k] = pre + x - v;
  }
  __syncthreads();
  for (int base = 0; base < total; base += NT) {
    const int t = base + (int)threadIdx.x;
    const bool valid = t < total;
    const uint32_t d = valid ? length_bucket(tile_cost[t]) : 0u;
    const uint64_t peers = match_digit(d, RADIX_BITS, __ballot(valid));
    const int leader = __ffsll((long long)peers) - 1;
    uint32_t first = 0u;
    if (valid && lane == leader) first = atomicAdd(&s_cur[d], (uint32_t)__popcll(peers));
    first = __shfl(first, leader < 0 ? 0 : leader);
    if (valid) queue[first + (uint32_t)__popcll(peers & lanemask_lt())] = (uint32_t)t;
  }
}

// --------------------------------------------------------------- launchers (host)

// Preprocess (projection and bin entries) for every (view, Gaussian).  Also
// clears grad2d when clear_grad2d (start of a fused step).
void launch_preprocess(const Plan &p, const gsr_gaussians &g, const gsr_camera *cams, const ViewInfo *views,
                       const gsr_config &cfg, const Workspace &ws, bool clear_grad2d, hipStream_t s);

// Reliable-Gaussian selection (fine tracking stage).
void launch_select_reliable(const gsr_gaussians &g, const gsr_camera *cam, const float *depth, int W, int H,
                            float eps, float z_near, uint8_t *out, hipStream_t s);

// Start of a call without Gaussians (in any other the projection does it), and
// the tile lists from the bin entries.  With order_total > 0 the lists kernel also writes the rasteriser's
// longest-first work order of that many tiles (from the durations the last
// fused step recorded).
void launch_lists_begin(const Workspace &ws, hipStream_t s);
void launch_bin_lists(const Plan &p, const Workspace &ws, const ViewInfo *views, const int32_t *bin_view,
                      int order_total, hipStream_t s);
// The lists moved into tile order without gaps (inspection).
void launch_lists_in_tile_order(const Plan &p, const Workspace &ws, hipStream_t s);
void launch_fill_u32(uint32_t *ptr, uint32_t value, int64_t count, hipStream_t s);
void launch_fill_f32(float *ptr, float value, int64_t count, hipStream_t s);
// The rasteriser's work order (order_tiles) as a one-block kernel.
void launch_queue_order(const Workspace &ws, int total_tiles, hipStream_t s);

// Rasterisation.
void launch_render_forward(const Plan &p, const Workspace &ws, const ViewInfo *views,
                           const int32_t *tile_view, const RenderConsts &rc,
                           const gsr_images *out, hipStream_t s);
void launch_render_backward(const Plan &p, const Workspace &ws, const ViewInfo *views,
                            const int32_t *tile_view, const RenderConsts &rc,
                            const float *g_rgb, const float *g_depth, const float *g_T,
                            hipStream_t s);
void launch_render_fused(const Plan &p, const Workspace &ws, const ViewInfo *views,
                         const int32_t *tile_view, const RenderConsts &rc,
                         const float *t_rgb, const float *t_depth, const uint8_t *pmask,
                         float w_rgb, float w_depth, const float *loss_cap, const gsr_images *out, const Tuning &tun, int num_cus, hipStream_t s);
// Work totals of the last forward (re-walks its lists; needs the constants of
// that call).
void launch_work_counts(const Plan &p, const Workspace &ws, const ViewInfo *views, const int32_t *tile_view,
                        const RenderConsts &rc, hipStream_t s);
void launch_l1(const Plan &p, const ViewInfo *views, const float *rgb, const float *depth,
               const float *t_rgb, const float *t_depth, const uint8_t *pmask, float w_rgb,
               float w_depth, const float *loss_cap, float *g_rgb, float *g_depth, float *loss, hipStream_t s);
// Loss cap: factor x lower median of each view's per-pixel loss.  With scratch
// (median_scratch_bytes, zero before the first call; every call leaves it
// zero) many blocks share a view; without, one block a view.
size_t median_scratch_bytes(int n_views);
bool median_wants_scratch(int64_t largest_view);
void launch_loss_median(const Plan &p, const ViewInfo *views, int64_t largest_view, const float *px_loss,
                        const uint8_t *pmask, float factor, float *cap_out, uint32_t *scratch, hipStream_t s);

// Pose parameterisations (one thread per view).
void launch_pose_apply(int n, const float *xi, const gsr_camera *cin, gsr_camera *cout, hipStream_t s);
void launch_pose_xi_grad(int n, const float *xi, const float *d_pose, float *d_xi, hipStream_t s);
void launch_pose_from_qt(int n, const float *q, const float *t, const gsr_camera *cin, gsr_camera *cout,
                         hipStream_t s);
void launch_pose_qt_grad(int n, const float *q, const float *t, const float *d_pose, float *d_q, float *d_t,
                         hipStream_t s);

// Adaptive expansion (adding step over the planned views; deleting step).
void launch_expand_add(const Plan &p, const ViewInfo *views, const gsr_camera *cams, const float *T_final,
                       const float *depth, const float *depth_obs, const float *rgb_obs, float tau_T, float tau_D,
                       float scale_factor, float logit_init, const Workspace &ws, int64_t n, int64_t capacity,
                       const gsr_gaussians_out &out, uint8_t *pixel_flag, int64_t *count, hipStream_t s);
void launch_expand_delete(const gsr_gaussians &g, const gsr_camera *cam, const float *depth_obs, int W, int H,
                          float gamma, float eta, float z_near, float *logit_out, uint8_t *decayed, hipStream_t s);

// Clears the gradient rows that a backward with these constants adds to: those
// of the records that the last projection on the workspace found visible.
void launch_clear_grads(const Plan &p, const Workspace &ws, const RenderConsts &rc, hipStream_t s);

// Backward preprocess (chain to parameters and pose; with loss, also the fused
// step's tile losses summed into *loss).
void launch_preprocess_backward(const Plan &p, const gsr_gaussians &g, const gsr_camera *cams,
                                const gsr_config &cfg, const Workspace &ws, const gsr_grads &gr, float *loss,
                                hipStream_t s);

}  // namespace gsr
