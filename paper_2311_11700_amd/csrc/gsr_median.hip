// Loss cap of the tracking loss: factor x the lower median of every view's
// per-pixel loss (the paper's implementation details drop tracking pixels
// whose loss exceeds ten times the median).  Exact radix select on the float
// bit patterns: three histograms of 11, 10 and 10 bits (the sign is gone), each
// over the values that share the digits already found.
//
// A view of up to MED_SMALL pixels is one block's work.  More pixels are
// counted by many blocks: a block reads its share a few values at a time
// into an LDS histogram and adds the non-zero counts to the view's histogram
// in the scratch; each later kernel finds the digit from the histogram of the
// one before, redundantly in every block (8 KB), and the last one writes the
// cap and leaves the scratch cleared.  640x480: one block 348 us (its loads
// came one at a time), the four kernels together 19 us.
#include <math.h>

#include "gsr_internal.h"

namespace gsr {

constexpr int MED_BLOCK = 1024;
constexpr int MED_WAVES = MED_BLOCK / 64;
constexpr int64_t MED_SMALL = 32768;  // pixels that one block counts in the time of the passes' extra launches
constexpr int64_t MED_CHUNK = 8192;   // pixels per block of a pass

// Order key of a loss value: non-negative floats order like their bit
// patterns; negative values and -0 count as 0, NaN sorts above +inf.
__device__ __forceinline__ uint32_t loss_key(float v) {
  const uint32_t b = __float_as_uint(v);
  const uint32_t a = b & 0x7FFFFFFFu;
  if (a > 0x7F800000u) return a;  // NaN of either sign
  return (b & 0x80000000u) ? 0u : b;
}

// Exclusive scan of one value per thread over the 1024-thread block; the
// block total goes to *total.
__device__ __forceinline__ uint32_t med_block_scan(uint32_t v, uint32_t *s_w, uint32_t *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_w[wave] = x;
  __syncthreads();
  if (wave == 0) {
    uint32_t w = lane < MED_WAVES ? s_w[lane] : 0u;
    for (int o = 1; o < MED_WAVES; o <<= 1) {
      const uint32_t y = __shfl_up(w, o);
      if (lane >= o) w += y;
    }
    if (lane < MED_WAVES) s_w[lane] = w;  // inclusive wave prefix
  }
  __syncthreads();
  const uint32_t before = wave > 0 ? s_w[wave - 1] : 0u;
  *total = s_w[MED_WAVES - 1];
  return before + x - v;
}

constexpr int MED_BITS[3] = {11, 10, 10};
constexpr int MED_SHIFT[3] = {20, 10, 0};

// Digit of the histogram (2^11 counters, the later digits use 2^10) that holds
// rank k, and k's rank inside it; in the first pass k is the lower median's
// rank among all counted values.  Every thread gets the answer; false where
// nothing was counted.  s_sel holds two words.
__device__ __forceinline__ bool med_select(const uint32_t *hist, bool first, uint32_t *s_w, uint32_t *s_sel,
                                           uint32_t &digit, uint32_t &k) {
  const uint32_t c0 = hist[2 * threadIdx.x], c1 = hist[2 * threadIdx.x + 1];
  uint32_t total;
  const uint32_t base = med_block_scan(c0 + c1, s_w, &total);
  if (first) {
    if (total == 0u) return false;
    k = (total - 1u) / 2u;
  }
  if (base <= k && k < base + c0) {
    s_sel[0] = 2u * threadIdx.x;
    s_sel[1] = base;
  } else if (base + c0 <= k && k < base + c0 + c1) {
    s_sel[0] = 2u * threadIdx.x + 1u;
    s_sel[1] = base + c0;
  }
  __syncthreads();
  digit = s_sel[0];
  k -= s_sel[1];
  __syncthreads();
  return true;
}

// Adds the values [q0, q1) of a view that match the prefix to hist (LDS).
__device__ __forceinline__ void med_count(const float *__restrict__ L, const uint8_t *__restrict__ M, int64_t q0,
                                          int64_t q1, int pass, uint32_t prefix, uint32_t *hist) {
  constexpr int PER = 8;  // values in flight per thread
  const int sh = MED_SHIFT[pass], hi = sh + MED_BITS[pass];
  const uint32_t mask = (1u << MED_BITS[pass]) - 1u;
  for (int64_t b = q0; b < q1; b += (int64_t)MED_BLOCK * PER) {
    float v[PER];
    uint8_t m[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t q = b + (int64_t)j * MED_BLOCK + threadIdx.x;
      m[j] = q < q1 ? 1 : 0;
      v[j] = q < q1 ? L[q] : 0.f;
    }
    if (M) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int64_t q = b + (int64_t)j * MED_BLOCK + threadIdx.x;
        if (q < q1) m[j] = M[q];
      }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const uint32_t key = loss_key(v[j]);
      if (m[j] != 0 && (pass == 0 || (key >> hi) == prefix)) atomicAdd(&hist[(key >> sh) & mask], 1u);
    }
  }
}

__global__ __launch_bounds__(MED_BLOCK) void k_loss_median(const ViewInfo *__restrict__ views,
                                                           const float *__restrict__ px_loss,
                                                           const uint8_t *__restrict__ pmask, float factor,
                                                           float *__restrict__ cap_out) {
  __shared__ uint32_t hist[2 * MED_BLOCK];
  __shared__ uint32_t s_w[MED_WAVES];
  __shared__ uint32_t s_sel[2];
  const ViewInfo vi = views[blockIdx.x];
  const int64_t HW = (int64_t)vi.W * vi.H;
  uint32_t prefix = 0u, k = 0u;
  for (int pass = 0; pass < 3; ++pass) {
    hist[threadIdx.x] = 0u;
    hist[threadIdx.x + MED_BLOCK] = 0u;
    __syncthreads();
    med_count(px_loss + vi.pix_off, pmask ? pmask + vi.pix_off : nullptr, 0, HW, pass, prefix, hist);
    __syncthreads();
    uint32_t digit;
    if (!med_select(hist, pass == 0, s_w, s_sel, digit, k)) {  // no eligible pixel: no cap
      if (threadIdx.x == 0) cap_out[blockIdx.x] = INFINITY;
      return;
    }
    prefix = prefix << MED_BITS[pass] | digit;
  }
  if (threadIdx.x == 0) cap_out[blockIdx.x] = factor * __uint_as_float(prefix);
}

// One pass over every view (grid: blocks x views), or with pass = 3 the result
// (one block a view).  scratch: [views][3][2 MED_BLOCK] counters, zero before
// pass 0.
__global__ __launch_bounds__(MED_BLOCK) void k_loss_median_pass(const ViewInfo *__restrict__ views,
                                                                const float *__restrict__ px_loss,
                                                                const uint8_t *__restrict__ pmask, int pass,
                                                                uint32_t *__restrict__ scratch, float factor,
                                                                float *__restrict__ cap_out) {
  __shared__ uint32_t hist[2 * MED_BLOCK];
  __shared__ uint32_t s_w[MED_WAVES];
  __shared__ uint32_t s_sel[2];
  const ViewInfo vi = views[blockIdx.y];
  const int64_t HW = (int64_t)vi.W * vi.H;
  uint32_t *view_hist = scratch + (size_t)blockIdx.y * 3 * 2 * MED_BLOCK;
  const int64_t q0 = (int64_t)blockIdx.x * MED_CHUNK;
  if (pass < 3 && q0 >= HW) return;
  uint32_t prefix = 0u, k = 0u;
  for (int p = 0; p < pass; ++p) {
    uint32_t digit;
    if (!med_select(view_hist + p * 2 * MED_BLOCK, p == 0, s_w, s_sel, digit, k)) {  // no eligible pixel: no cap
      if (pass == 3 && threadIdx.x == 0) cap_out[blockIdx.y] = INFINITY;
      return;  // (nothing was counted, so the scratch is clear)
    }
    prefix = prefix << MED_BITS[p] | digit;
  }
  if (pass == 3) {
    if (threadIdx.x == 0) cap_out[blockIdx.y] = factor * __uint_as_float(prefix);
    for (int t = threadIdx.x; t < 3 * 2 * MED_BLOCK; t += MED_BLOCK) view_hist[t] = 0u;
    return;
  }
  hist[threadIdx.x] = 0u;
  hist[threadIdx.x + MED_BLOCK] = 0u;
  __syncthreads();
  med_count(px_loss + vi.pix_off, pmask ? pmask + vi.pix_off : nullptr, q0, q0 + MED_CHUNK < HW ? q0 + MED_CHUNK : HW,
            pass, prefix, hist);
  __syncthreads();
  for (int t = threadIdx.x; t < 2 * MED_BLOCK; t += MED_BLOCK)
    if (hist[t]) atomicAdd(&view_hist[pass * 2 * MED_BLOCK + t], hist[t]);
}

size_t median_scratch_bytes(int n_views) { return (size_t)n_views * 3 * 2 * MED_BLOCK * sizeof(uint32_t); }

bool median_wants_scratch(int64_t largest_view) { return largest_view > MED_SMALL; }

void launch_loss_median(const Plan &p, const ViewInfo *views, int64_t largest_view, const float *px_loss,
                        const uint8_t *pmask, float factor, float *cap_out, uint32_t *scratch, hipStream_t s) {
  if (!scratch) {
    hipLaunchKernelGGL(k_loss_median, dim3((unsigned)p.n_views), dim3(MED_BLOCK), 0, s, views, px_loss, pmask, factor,
                       cap_out);
    return;
  }
  const unsigned blocks = (unsigned)((largest_view + MED_CHUNK - 1) / MED_CHUNK);
  for (int pass = 0; pass <= 3; ++pass)
    hipLaunchKernelGGL(k_loss_median_pass, dim3(pass < 3 ? blocks : 1u, (unsigned)p.n_views), dim3(MED_BLOCK), 0, s,
                       views, px_loss, pmask, pass, scratch, factor, cap_out);
}

}  // namespace gsr
