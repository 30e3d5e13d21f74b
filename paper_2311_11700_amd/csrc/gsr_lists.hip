// Tile lists: every tile's Gaussians in blending order, the lexicographic
// (tile, float32 depth bits, index) order.
//
// The tiles of a view are grouped into bins of S x S (S = 1, 2 or 4, chosen
// per view by gsr_plan).  A record (one Gaussian in one view) becomes one
// entry (depth key, record id, mask of the bin's tiles it reaches) in every
// bin it reaches: a few entries instead of one pair per tile.  The projection
// writes each block's entries grouped by bin, with the offsets of the groups;
// one block per bin then collects its groups, sorts them by depth in LDS and
// writes the lists of all its tiles from the masks.  So the lists take two
// kernels beside the projection whatever the sizes, with no global sort.
// Every grid is fixed by the plan and every count is read on the device, so
// the sequence can be captured in a HIP graph.
//
// Measured against radix passes over the records and the pairs (17 dependent
// kernels): 300k Gaussians at 1200x680, projection and lists 171 us -> 78 us;
// 72 views of 500k, 12.2 ms -> 3.2 ms; 2 000 Gaussians at 160x120 as a whole
// call 155 us -> 81 us.
#include "gsr_internal.h"

namespace gsr {

__global__ void k_fill_u32(uint32_t *__restrict__ p, uint32_t v, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x)
    p[k] = v;
}

__global__ void k_fill_f32(float *__restrict__ p, float v, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x)
    p[k] = v;
}

static unsigned fill_grid(int64_t n) {
  int64_t b = (n + BLOCK - 1) / BLOCK;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return (unsigned)b;
}

void launch_fill_u32(uint32_t *ptr, uint32_t value, int64_t count, hipStream_t s) {
  if (count > 0) hipLaunchKernelGGL(k_fill_u32, dim3(fill_grid(count)), dim3(BLOCK), 0, s, ptr, value, count);
}

void launch_fill_f32(float *ptr, float value, int64_t count, hipStream_t s) {
  if (count > 0) hipLaunchKernelGGL(k_fill_f32, dim3(fill_grid(count)), dim3(BLOCK), 0, s, ptr, value, count);
}

// ----------------------------------------------------------------- header

// Start of a call without Gaussians; otherwise the projection does it.
__global__ void k_lists_begin(uint32_t *__restrict__ hdr) {
  if (threadIdx.x != 0) return;
  reset_header_words(hdr);
  *entry_cursor(hdr) = ENTRY_TAG;
}

void launch_lists_begin(const Workspace &ws, hipStream_t s) {
  hipLaunchKernelGGL(k_lists_begin, dim3(1), dim3(64), 0, s, ws.hdr);
}

// ----------------------------------------------------------------- lists

// One block per bin: collects the bin's groups (one per projection block),
// sorts the entries in LDS by (depth, record id) and writes the lists.
// Entries are sorted by reference: the keys stay in place and 16-bit positions
// move.  Counting into LPARTS equal parts of the bin's depth range gives each
// key an estimated rank (walls crowd most depths of a bin into a few parts, so
// the rank is interpolated inside the part); a second count by estimated rank
// leaves about one entry a slot, and one thread orders the few that share one.
// Depths that crowd even there (a slot over LSLOT) take stable
// least-significant-digit passes over the differing bits instead, and equal
// depths are put in index order afterwards.  A bin with more than `cap`
// entries is taken in rounds of consecutive key ranges.  A tile's list is the
// sorted entries whose mask has the tile's bit: per row of 64 entries one
// ballot gives the tile's entries and each lane's place, so consecutive lanes
// write consecutive words.
//
// Bound by the latency of the reads of the entries and by the block's LDS (one
// block a CU at its 12 288 entries).  A bin of 7 000 entries (72 views of
// 500 000 Gaussians) took 67 us: 20 to collect its groups, 10 to order the
// slots, 8 for the masks and 21 to write.  It takes 51 us with the group table
// read at once and four groups in flight (13), up to four entries of a slot
// ordered in registers (8), id and mask read together, and the places counted
// from the tile's next one in the lanes' registers (12): 5 512 bins 1.65 -> 1.2
// ms, the 209 bins of 2 500 of a 1200x680 view 39 -> 33 us.
constexpr int LB = 1024;         // threads
constexpr int LW = LB / 64;      // wavefronts
constexpr int LBITS = 8;         // bits per digit pass
constexpr int LDIGITS = 1 << LBITS;
constexpr int LRUN = 24;         // longest run of equal depths that one thread orders
constexpr int LPARTS = 4096;     // parts of the depth range
constexpr uint32_t LSLOT = 24;   // most entries of a slot that one thread orders
constexpr int NTILE = BIN_MAX * BIN_MAX;
static_assert(LPARTS <= LISTS_CAP_MIN, "the rounds' histogram takes the keys' place");

// Arrays of `cap` entries in dynamic LDS.
struct ListsArrays {
  uint32_t *key;   // depth key
  uint32_t *at;    // entry index
  uint16_t *from, *to;  // positions before and after a sorting pass
};

struct ListsLds {
  union {
    uint16_t cnt[LW][LDIGITS];  // per-wavefront digit counts, then next positions
    uint32_t part[LPARTS / 2];  // counts of the parts (two per word), then next positions
    uint2 group[LB];            // first entry and place of the groups that are being read
  };
  uint32_t w[LW];
  uint32_t tile[LW][NTILE];    // per-wavefront entries of each tile, then their first places
  uint32_t next[NTILE];        // next place of each tile's list
  uint32_t kmin, kmax, n, most, end;
};

// One stable digit pass over n positions, from -> to, by `per` bits at sh of
// value(position).  A wavefront takes I rows of 64 positions; it counts its
// digits, and after the scan of the counts walks its rows again: the place of
// an entry is its digit's next position plus the equal digits in front of it
// in its row.
template <typename V>
__device__ __forceinline__ void digit_pass(ListsLds &s, const uint16_t *from, uint16_t *to, int n, int I, int at,
                                           int sh, int per, V value) {
  const int wave = threadIdx.x >> 6;
  const uint32_t mask = (1u << per) - 1u;
  __syncthreads();
  for (int t = threadIdx.x; t < LW * LDIGITS / 2; t += LB) s.part[t] = 0u;
  for (int walk = 0; walk < 2; ++walk) {
    __syncthreads();
    for (int r = 0; r < I; ++r) {
      const bool valid = at + 64 * r < n;
      const uint16_t q = valid ? from[at + 64 * r] : 0;
      const uint32_t d = valid ? (value(q) >> sh) & mask : 0u;
      const uint64_t peers = match_digit(d, per, __ballot(valid));
      const uint64_t below = peers & lanemask_lt();
      // Every lane reads before the group's first lane adds the group's size
      // (program order within the wavefront).
      const uint32_t next = valid ? s.cnt[wave][d] : 0u;
      if (walk == 1 && valid) to[next + (uint32_t)__popcll(below)] = q;
      if (valid && below == 0ull) s.cnt[wave][d] = (uint16_t)(next + (uint32_t)__popcll(peers));
    }
    __syncthreads();
    if (walk == 0) {
      uint32_t sum = 0u, total;
      if (threadIdx.x < LDIGITS)
        for (int w = 0; w < LW; ++w) sum += s.cnt[w][threadIdx.x];
      uint32_t pre = block_exclusive_scan<LB>(sum, s.w, total);
      if (threadIdx.x < LDIGITS)
        for (int w = 0; w < LW; ++w) {
          const uint32_t c = s.cnt[w][threadIdx.x];
          s.cnt[w][threadIdx.x] = (uint16_t)pre;
          pre += c;
        }
    }
  }
}

// LSD passes over the low `bits` bits of value(position) (at least one).
template <typename V>
__device__ __forceinline__ void sort_digits(ListsLds &s, ListsArrays &a, int n, int I, int at, int bits, V value) {
  const int passes = bits ? (bits + LBITS - 1) / LBITS : 1;
  const int per = bits ? (bits + passes - 1) / passes : 1;
  for (int p = 0; p < passes; ++p) {
    digit_pass(s, a.from, a.to, n, I, at, p * per, per, value);
    uint16_t *t = a.from;
    a.from = a.to;
    a.to = t;
  }
}

// Orders the positions from[first .. last] by (key, record id) in place.
__device__ __forceinline__ void order_span(const ListsArrays &a, uint16_t *from, int first, int last,
                                           const Entry *__restrict__ entries) {
  for (int i = first + 1; i <= last; ++i) {
    const uint16_t me = from[i];
    const uint32_t k = a.key[me];
    int j = i;
    for (; j > first; --j) {
      const uint16_t o = from[j - 1];
      const uint32_t ko = a.key[o];
      if (ko < k || (ko == k && entries[a.at[o]].id < entries[a.at[me]].id)) break;
      from[j] = o;
    }
    from[j] = me;
  }
}

// The same for the entries of one slot: up to four distinct keys (a slot holds
// one entry on average) are ordered in registers, since an insertion step
// waits for two dependent LDS reads.
__device__ __forceinline__ void order_slot(const ListsArrays &a, uint16_t *from, int first, int last,
                                           const Entry *__restrict__ entries) {
  constexpr int N = 4;
  const int n = last - first + 1;
  if (n <= N) {
    uint32_t f[N], k[N];
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = i < n ? from[first + i] : 0u;
#pragma unroll
    for (int i = 0; i < N; ++i) k[i] = i < n ? a.key[f[i]] : 0xFFFFFFFFu;  // (keys are below 2^31)
    auto order = [&](int i, int j) {
      const bool swap = k[j] < k[i];
      const uint32_t ki = k[i], fi = f[i];
      k[i] = swap ? k[j] : ki;
      f[i] = swap ? f[j] : fi;
      k[j] = swap ? ki : k[j];
      f[j] = swap ? fi : f[j];
    };
    order(0, 1);
    order(2, 3);
    order(0, 2);
    order(1, 3);
    order(1, 2);
    if (k[0] != k[1] && (n < 3 || k[1] != k[2]) && (n < 4 || k[2] != k[3])) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (i < n) from[first + i] = (uint16_t)f[i];
      return;
    }
  }
  order_span(a, from, first, last, entries);
}

// Exclusive scan of `count` 16-bit counters in place (two per word); s.most
// becomes the largest of them if that exceeds `limit`.
__device__ __forceinline__ void scan_counters(ListsLds &s, uint32_t *words, int count, uint32_t limit) {
  const int nw = (count + 1) / 2, per = (nw + LB - 1) / LB;
  const int w0 = min((int)threadIdx.x * per, nw), w1 = min(w0 + per, nw);
  uint32_t sum = 0u, most = 0u, total;
  for (int w = w0; w < w1; ++w) {
    const uint32_t c = words[w];
    sum += (c & 0xFFFFu) + (c >> 16);
    most = max(most, max(c & 0xFFFFu, c >> 16));
  }
  if (most > limit) s.most = most;
  uint32_t pre = block_exclusive_scan<LB>(sum, s.w, total);
  for (int w = w0; w < w1; ++w) {
    const uint32_t c = words[w], mid = pre + (c & 0xFFFFu);
    words[w] = pre | mid << 16;
    pre = mid + (c >> 16);
  }
  __syncthreads();
}

// Positions of the n entries in (key, record id) order into a.from; the keys
// are key0 + [0, 2^key_bits).
__device__ __forceinline__ void sort_entries(ListsLds &s, ListsArrays &a, int n, int I, int at, uint32_t key0,
                                             int key_bits, const Entry *__restrict__ entries, uint32_t id0,
                                             int id_bits) {
  constexpr int PBITS = 12;
  static_assert(LPARTS == 1 << PBITS, "parts per key range");
  const int sh = key_bits > PBITS ? key_bits - PBITS : 0;
  uint32_t *slots = reinterpret_cast<uint32_t *>(a.to);
  for (int t = threadIdx.x; t < LPARTS / 2; t += LB) s.part[t] = 0u;
  for (int t = threadIdx.x; t < (n + 1) / 2; t += LB) slots[t] = 0u;
  if (threadIdx.x == 0) s.most = 0u;
  __syncthreads();
  for (int q = threadIdx.x; q < n; q += LB) {
    const uint32_t p = (a.key[q] - key0) >> sh;
    atomicAdd(&s.part[p >> 1], 1u << (16u * (p & 1u)));
  }
  __syncthreads();
  scan_counters(s, s.part, LPARTS, 0xFFFFu);
  // The slot of a key: its rank if the keys of its part lay evenly in it.
  const uint16_t *start = reinterpret_cast<const uint16_t *>(s.part);
  auto slot = [&](uint32_t k) {
    const uint32_t d = k - key0, p = d >> sh;
    const uint32_t f = start[p], c = (p + 1u < (uint32_t)LPARTS ? start[p + 1u] : (uint32_t)n) - f;
    return f + (sh > 0 ? __umulhi(d << (32 - sh), c) : 0u);
  };
  for (int q = threadIdx.x; q < n; q += LB) {
    const uint32_t t = slot(a.key[q]);
    atomicAdd(&slots[t >> 1], 1u << (16u * (t & 1u)));
  }
  __syncthreads();
  scan_counters(s, slots, n, LSLOT);
  if (s.most <= LSLOT) {
    // A slot's next position ends up as its end.
    for (int q = threadIdx.x; q < n; q += LB) {
      const uint32_t t = slot(a.key[q]), half = 16u * (t & 1u);
      a.from[(atomicAdd(&slots[t >> 1], 1u << half) >> half) & 0xFFFFu] = (uint16_t)q;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < n; t += LB) {
      const int first = t ? a.to[t - 1] : 0, last = (int)a.to[t] - 1;
      if (last > first) order_slot(a, a.from, first, last, entries);
    }
    __syncthreads();
    return;
  }
  // By depth digits; with a long run of equal depths by record id and then
  // (stable) by depth again.
  for (int q = threadIdx.x; q < n; q += LB) a.from[q] = (uint16_t)q;
  for (int stage = 0; stage < 3; ++stage) {
    const bool by_id = stage == 1;
    sort_digits(s, a, n, I, at, by_id ? id_bits : key_bits, [&](uint32_t q) {
      return by_id ? entries[a.at[q]].id - id0 : a.key[q] - key0;
    });
    if (stage > 0) continue;
    int tie = 0;
    for (int q = threadIdx.x; q + 1 < n; q += LB)
      if (a.key[a.from[q]] == a.key[a.from[q + 1]])
        tie = max(tie, q + LRUN < n && a.key[a.from[q]] == a.key[a.from[q + LRUN]] ? 2 : 1);
    if (__syncthreads_or(tie > 1)) continue;
    // Short runs of equal depths: ordered by the thread of their first entry.
    for (int q = threadIdx.x; q < n; q += LB) {
      const uint32_t k = a.key[a.from[q]];
      if (q > 0 && a.key[a.from[q - 1]] == k) continue;
      int last = q;
      while (last + 1 < n && a.key[a.from[last + 1]] == k) ++last;
      if (last > q) order_span(a, a.from, q, last, entries);
    }
    break;
  }
  __syncthreads();
}

// Calls use(place, entry, load(entry)) for every entry of the bin, place
// counting them group after group (the entries one projection batch wrote for
// the bin); returns their number.  The groups' first entries and places come
// from one read of the group table by the whole block, so that the reads of
// the entries depend on LDS alone and LUNROLL groups of a team of LTEAM lanes
// are in flight at a time: reading a group's place, then its entries, one
// group after the other, took 20 of a bin's 67 us with 980 groups of 7 entries.
constexpr int LTEAM = 16;
constexpr int LUNROLL = 4;
template <typename L, typename U>
__device__ __forceinline__ int for_entries(ListsLds &s, const Workspace &ws, const ViewInfo &vi, int view, int local,
                                           int groups, L load, U use) {
  const int stride = vi.BX * vi.BY + 1;
  const int sub = threadIdx.x & (LTEAM - 1);
  constexpr int TEAMS = LB / LTEAM;
  const uint32_t *bases = ws.block_base + (size_t)view * groups;
  uint32_t E = 0u;
  for (int g0 = 0; g0 < groups; g0 += LB) {
    const int j = g0 + (int)threadIdx.x;
    uint32_t first = 0u, n = 0u, total;
    if (j < groups) {
      const uint32_t base = bases[j];
      const uint32_t *row = ws.group_off + vi.mat_off + (int64_t)j * stride + local;
      const uint32_t r0 = row[0], r1 = row[1];  // (not written where base is NO_BASE)
      if (base != NO_BASE) {
        first = base + r0;
        n = r1 - r0;
      }
    }
    __syncthreads();  // (the table's place: s.part, s.w)
    const uint32_t pre = block_exclusive_scan<LB>(n, s.w, total) + E;
    s.group[threadIdx.x] = make_uint2(first, pre);
    if (threadIdx.x == 0) s.end = E + total;
    E += total;
    __syncthreads();
    const int ng = min(LB, groups - g0);
    for (int t0 = threadIdx.x / LTEAM; t0 < ng; t0 += TEAMS * LUNROLL) {
      uint32_t e[LUNROLL], q[LUNROLL], left[LUNROLL];
      decltype(load(0u)) v[LUNROLL];
#pragma unroll
      for (int u = 0; u < LUNROLL; ++u) {
        const int t = t0 + u * TEAMS;
        left[u] = 0u;
        if (t < ng) {
          const uint2 g = s.group[t];
          const uint32_t next = t + 1 < ng ? s.group[t + 1].y : s.end;
          e[u] = g.x + sub;
          q[u] = g.y + sub;
          left[u] = next > q[u] ? next - q[u] : 0u;
        }
      }
#pragma unroll
      for (int u = 0; u < LUNROLL; ++u)
        if (left[u]) v[u] = load(e[u]);
#pragma unroll
      for (int u = 0; u < LUNROLL; ++u)
        if (left[u]) {
          use(q[u], e[u], v[u]);
          for (uint32_t k = LTEAM; k < left[u]; k += LTEAM) use(q[u] + k, e[u] + k, load(e[u] + k));
        }
    }
  }
  __syncthreads();
  return (int)E;
}

// The sorted entries' record ids and masks in order, in the place of the keys
// and of the free positions (a thread reads and writes its own places only),
// and the wavefront's entries of each of the bin's NT tiles.
template <int NT>
__device__ __forceinline__ void order_masks(ListsLds &s, const ListsArrays &a, const Entry *__restrict__ entries, int n,
                                            int I, int at) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t c[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) c[t] = 0u;
  for (int r0 = 0; r0 < I; r0 += LUNROLL) {
    // (LUNROLL rows' reads in flight)
    uint32_t m[LUNROLL], id[LUNROLL];
#pragma unroll
    for (int u = 0; u < LUNROLL; ++u) {
      const int q = at + 64 * (r0 + u);
      m[u] = 0u;
      if (r0 + u < I && q < n) {
        const Entry *e = entries + a.at[a.from[q]];
        id[u] = e->id;
        m[u] = e->mask;
      }
    }
#pragma unroll
    for (int u = 0; u < LUNROLL; ++u) {
      if (r0 + u >= I) break;
      const int q = at + 64 * (r0 + u);
      if (q < n) {
        a.key[q] = id[u];
        a.to[q] = (uint16_t)m[u];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) c[t] += (uint32_t)__popcll(__ballot((m[u] & (1u << t)) != 0u));
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (lane == t) s.tile[wave][t] = c[t];
}

// The wavefront's part of the NT lists, from s.tile on: in a row of 64 entries
// the lanes whose mask has the tile's bit write consecutive words.
template <int NT>
__device__ __forceinline__ void write_lists(const ListsLds &s, const ListsArrays &a, uint32_t *__restrict__ ids, int n,
                                            int I, int at) {
  const int wave = threadIdx.x >> 6;
  uint32_t c[NT];  // next place (held per lane: the count of the lanes in front starts from it)
#pragma unroll
  for (int t = 0; t < NT; ++t) c[t] = s.tile[wave][t];
  for (int r = 0; r < I; ++r) {
    const int q = at + 64 * r;
    uint32_t m = 0u, id = 0u;
    if (q < n) {
      m = a.to[q];
      id = a.key[q];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bool in = (m & (1u << t)) != 0u;
      const uint64_t b = __builtin_amdgcn_ballot_w64(in);
      const uint32_t place =
          __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, c[t]));
      if (in) ids[place] = id;
      c[t] += (uint32_t)__popcll(b);
    }
  }
}

__global__ __launch_bounds__(LB) void k_bin_lists(const ViewInfo *__restrict__ views,
                                                  const int32_t *__restrict__ bin_view, Workspace ws, int64_t n_gauss,
                                                  int id_bits, int groups, int pre_blocks, unsigned long long cap_pairs,
                                                  int cap, int order_total) {
  extern __shared__ uint32_t dyn[];
  __shared__ ListsLds s;
  if (blockIdx.x == 0) {
    // The pair count, and the overflow record when it exceeds the capacity.
    unsigned long long x = 0ull;
    for (int j = threadIdx.x; j < pre_blocks; j += LB) x += ws.block_pairs[j];
    unsigned long long *part = reinterpret_cast<unsigned long long *>(s.part);
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < LW; ++w) x += part[w];
      *reinterpret_cast<unsigned long long *>(ws.hdr + HDR_NPAIRS) = x;
      // Entries are no more than pairs: a count above the capacity with fewer
      // pairs did not start at 0 (a call that ended between the projection and
      // here, a word overwritten).  It is reported as an overflow, and the next
      // call starts clean.  No tag in a workspace never used: no entries.
      const unsigned long long cur = read_entry_cursor(ws.hdr);
      const bool tagged = (cur & ~ENTRY_COUNT_MASK) == ENTRY_TAG;
      const unsigned long long used = tagged || header_used(ws.hdr) ? cur - ENTRY_TAG : 0ull;
      *entry_cursor(ws.hdr) = ENTRY_TAG;
      ws.hdr[HDR_MAGIC] = HDR_MAGIC0;
      ws.hdr[HDR_MAGIC + 1] = HDR_MAGIC1;
      if (x > cap_pairs || used > cap_pairs) {
        unsigned long long *req = reinterpret_cast<unsigned long long *>(ws.hdr + HDR_REQUIRED);
        ws.hdr[HDR_OVERFLOW] = 1u;
        if (x > *req) *req = x;
      }
    }
    return;
  }
  if (blockIdx.x == 1) {
    // The rasteriser's work order for this step, from the tile durations the
    // last fused step recorded (the other blocks cover its time).
    if (order_total > 0)
      order_tiles<LB>(ws.tile_cost, ws.hdr[HDR_COSTS] != 0u, order_total, ws.queue, s.part, s.part + RADIX, s.w);
    return;
  }
  ListsArrays a;
  a.key = dyn;
  a.at = dyn + cap;
  a.from = reinterpret_cast<uint16_t *>(dyn + 2 * cap);
  a.to = a.from + cap;
  const int bin = blockIdx.x - 2;
  const int view = bin_view[bin];
  const ViewInfo vi = views[view];
  const int shift = vi.bin_shift, S = 1 << shift, nt = S * S;
  const int local = bin - vi.bin_off;
  const int by = local / vi.BX, bx = local - by * vi.BX;
  const Entry *entries = ws.entries;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tx = (bx << shift) + ((int)threadIdx.x & (S - 1)), ty = (by << shift) + ((int)threadIdx.x >> shift);
  const bool my_tile = (int)threadIdx.x < nt && tx < vi.TX && ty < vi.TY;
  const int tile = vi.tile_off + ty * vi.TX + tx;
  const uint32_t id0 = (uint32_t)((int64_t)view * n_gauss);

  if (threadIdx.x == 0) {
    s.kmin = 0xFFFFFFFFu;
    s.kmax = 0u;
  }
  int E;
  {
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
    E = for_entries(
        s, ws, vi, view, local, groups, [&](uint32_t e) { return entries[e].key; },
        [&](uint32_t q, uint32_t e, uint32_t key) {
          kmin = min(kmin, key);
          kmax = max(kmax, key);
          if (q < (uint32_t)cap) {
            a.key[q] = key;
            a.at[q] = e;
          }
        });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmin = min(kmin, __shfl_xor(kmin, o));
      kmax = max(kmax, __shfl_xor(kmax, o));
    }
    if (lane == 0) {
      atomicMin(&s.kmin, kmin);
      atomicMax(&s.kmax, kmax);
    }
  }
  __syncthreads();
  if (E == 0) {
    if (my_tile) ws.ranges[tile] = make_int2(0, 0);
    return;
  }
  const bool all_fit = E <= cap;
  const uint32_t kmin = s.kmin, kmax = s.kmax;
  if (!all_fit) {
    // The tiles' totals, needed before the first round writes.
    if (threadIdx.x < NTILE) s.next[threadIdx.x] = 0u;
    __syncthreads();
    for_entries(
        s, ws, vi, view, local, groups, [&](uint32_t e) { return entries[e].mask; },
        [&](uint32_t, uint32_t, uint32_t mask) {
          for (uint32_t m = mask; m; m &= m - 1u) atomicAdd(&s.next[__ffs(m) - 1], 1u);
        });
    __syncthreads();
  }

  // Rounds over consecutive ranges [lo, hi) of the unique key (depth, record
  // id) with at most cap entries each; one round when all entries fit.
  const uint64_t end = ((uint64_t)kmax << 32 | 0xFFFFFFFFull) + 1ull;  // depth keys are below 2^31
  uint64_t lo = (uint64_t)kmin << 32;
  for (bool placed = false; lo < end;) {
    uint64_t hi = end;
    int n = E;
    if (!all_fit) {
      // The range's end comes from a histogram over LPARTS equal parts of
      // what is left; a part that alone exceeds cap is divided again.
      uint32_t *hist = a.key;
      int sh = 0;
      while ((end - lo) >> sh > (uint64_t)LPARTS) ++sh;
      for (;;) {
        __syncthreads();
        for (int b = threadIdx.x; b < LPARTS; b += LB) hist[b] = 0u;
        if (threadIdx.x == 0) s.n = (uint32_t)LPARTS;
        __syncthreads();
        for_entries(
            s, ws, vi, view, local, groups,
            [&](uint32_t e) { return (uint64_t)entries[e].key << 32 | entries[e].id; },
            [&](uint32_t, uint32_t, uint64_t k) {
              if (k >= lo && (k - lo) >> sh < (uint64_t)LPARTS) atomicAdd(&hist[(k - lo) >> sh], 1u);
            });
        __syncthreads();
        // Parts in order while their sum fits: the first part whose
        // inclusive sum exceeds cap ends the range.
        constexpr int PER = LPARTS / LB;
        uint32_t sum = 0u, total;
#pragma unroll
        for (int k = 0; k < PER; ++k) sum += hist[threadIdx.x * PER + k];
        uint32_t run = block_exclusive_scan<LB>(sum, s.w, total);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const uint32_t h = hist[threadIdx.x * PER + k];
          if (run <= (uint32_t)cap && run + h > (uint32_t)cap) s.n = threadIdx.x * PER + k;
          run += h;
        }
        __syncthreads();
        const uint32_t parts = s.n;
        if (parts > 0u) {
          hi = lo + ((uint64_t)parts << sh);
          break;
        }
        sh = sh > 12 ? sh - 12 : 0;  // (at sh = 0 a part is one key, which one entry has)
      }
      __syncthreads();
      if (threadIdx.x == 0) s.n = 0u;
      __syncthreads();
      for_entries(
          s, ws, vi, view, local, groups,
          [&](uint32_t e) { return (uint64_t)entries[e].key << 32 | entries[e].id; },
          [&](uint32_t, uint32_t e, uint64_t k) {
            if (k >= lo && k < hi) {
              const uint32_t q = atomicAdd(&s.n, 1u);
              a.key[q] = (uint32_t)(k >> 32);
              a.at[q] = e;
            }
          });
      __syncthreads();
      n = (int)s.n;
    }
    const uint32_t key0 = (uint32_t)(lo >> 32), key1 = min((uint32_t)((hi - 1ull) >> 32), kmax);
    lo = hi;
    if (n == 0) continue;
    const int I = (n + LB - 1) / LB;
    const int at = wave * 64 * I + lane;
    sort_entries(s, a, n, I, at, key0, key1 <= key0 ? 0 : 32 - __clz(key1 - key0), entries, id0, id_bits);
    if (shift == 2) order_masks<16>(s, a, entries, n, I, at);
    else if (shift == 1) order_masks<4>(s, a, entries, n, I, at);
    else order_masks<1>(s, a, entries, n, I, at);
    __syncthreads();
    if (threadIdx.x < 64) {
      uint32_t mine = 0u;
      if (lane < nt) {
#pragma unroll
        for (int w = 0; w < LW; ++w) mine += s.tile[w][lane];
      }
      uint32_t place = 0u;
      if (!placed) {
        // The bin's lists take consecutive places, tile after tile, reserved
        // with one add on the listed-pair count.  Past the capacity (an
        // overflow) they stay empty.
        const uint32_t tot = all_fit ? mine : lane < NTILE ? s.next[lane] : 0u;
        uint32_t x = tot;
#pragma unroll
        for (int o = 1; o < NTILE; o <<= 1) {
          const uint32_t y = __shfl_up(x, o);
          if (lane >= o) x += y;
        }
        const uint32_t all = __shfl(x, NTILE - 1);
        unsigned long long first = 0ull;
        if (lane == 0)
          first = atomicAdd(reinterpret_cast<unsigned long long *>(ws.hdr + HDR_NLISTED), (unsigned long long)all);
        first = __shfl(first, 0);
        const bool fits = first + all <= cap_pairs;
        place = (uint32_t)first + x - tot;
        if (lane == 0) s.most = fits ? 0u : 0xFFFFFFFFu;
        if (my_tile) ws.ranges[tile] = fits ? make_int2((int)place, (int)(place + tot)) : make_int2(0, 0);
      } else if (lane < nt) {
        place = s.next[lane];
      }
      if (lane < nt) {
#pragma unroll
        for (int w = 0; w < LW; ++w) {
          const uint32_t k = s.tile[w][lane];
          s.tile[w][lane] = place;
          place += k;
        }
        s.next[lane] = place;
      }
    }
    __syncthreads();
    if (!placed && s.most == 0xFFFFFFFFu) return;
    placed = true;
    if (shift == 2) write_lists<16>(s, a, ws.ids, n, I, at);
    else if (shift == 1) write_lists<4>(s, a, ws.ids, n, I, at);
    else write_lists<1>(s, a, ws.ids, n, I, at);
    __syncthreads();
  }
}

void launch_bin_lists(const Plan &p, const Workspace &ws, const ViewInfo *views, const int32_t *bin_view,
                      int order_total, hipStream_t s) {
  int id_bits = 1;
  while ((1ll << id_bits) < p.n) ++id_bits;
  hipLaunchKernelGGL(k_bin_lists, dim3((unsigned)p.total_bins + 2u), dim3(LB), (size_t)p.lists_cap * LISTS_ENTRY_BYTES,
                     s, views, bin_view, ws, p.n, id_bits, p.blocks_per_view * p.pre_rounds, p.blocks_per_view * p.n_views,
                     (unsigned long long)p.capacity, p.lists_cap, order_total);
}

// ------------------------------------------------------- lists for inspection

// The bins' blocks place their lists in the order they finish.  For
// inspection the lists are moved into tile order without gaps (through the
// entries, which nothing reads once the lists are written); everything
// that reads the lists goes by the ranges.  Ranges that cannot be lists (a
// workspace no forward has filled) count as empty.
constexpr int QUEUE_BLOCK = 1024;

__device__ __forceinline__ uint32_t list_length(int2 r, uint32_t cap) {
  const uint32_t a = (uint32_t)r.x, b = (uint32_t)r.y;
  return a <= b && b <= cap ? b - a : 0u;
}

__global__ __launch_bounds__(QUEUE_BLOCK) void k_tile_starts(const int2 *__restrict__ ranges, int n_tiles, uint32_t cap,
                                                            uint32_t *__restrict__ starts) {
  __shared__ uint32_t s_w[QUEUE_BLOCK / 64];
  uint32_t carry = 0u;
  for (int base = 0; base < n_tiles; base += QUEUE_BLOCK) {
    const int t = base + (int)threadIdx.x;
    const uint32_t v = t < n_tiles ? list_length(ranges[t], cap) : 0u;
    uint32_t total;
    const uint32_t pre = block_exclusive_scan<QUEUE_BLOCK>(v, s_w, total) + carry;
    if (t < n_tiles) starts[t] = pre;
    carry += total;
  }
}

__global__ __launch_bounds__(BLOCK) void k_tile_gather(const int2 *__restrict__ ranges,
                                                       const uint32_t *__restrict__ starts, uint32_t cap,
                                                       const uint32_t *__restrict__ ids, uint32_t *__restrict__ out) {
  const int2 r = ranges[blockIdx.x];
  const uint32_t len = list_length(r, cap), to = starts[blockIdx.x];
  for (uint32_t k = threadIdx.x; k < len && to + k < cap; k += BLOCK) out[to + k] = ids[(uint32_t)r.x + k];
}

__global__ __launch_bounds__(BLOCK) void k_tile_place(int2 *__restrict__ ranges, const uint32_t *__restrict__ starts,
                                                      uint32_t cap, const uint32_t *__restrict__ in,
                                                      uint32_t *__restrict__ ids) {
  const uint32_t len = list_length(ranges[blockIdx.x], cap), to = starts[blockIdx.x];
  for (uint32_t k = threadIdx.x; k < len && to + k < cap; k += BLOCK) ids[to + k] = in[to + k];
  __syncthreads();
  if (threadIdx.x == 0) ranges[blockIdx.x] = make_int2((int)to, (int)(to + len));
}

void launch_lists_in_tile_order(const Plan &p, const Workspace &ws, hipStream_t s) {
  const uint32_t cap = (uint32_t)p.capacity;
  // (the work order of the last step is not read again)
  hipLaunchKernelGGL(k_tile_starts, dim3(1), dim3(QUEUE_BLOCK), 0, s, ws.ranges, p.total_tiles, cap, ws.queue);
  hipLaunchKernelGGL(k_tile_gather, dim3((unsigned)p.total_tiles), dim3(BLOCK), 0, s, ws.ranges, ws.queue, cap, ws.ids,
                     reinterpret_cast<uint32_t *>(ws.entries));
  hipLaunchKernelGGL(k_tile_place, dim3((unsigned)p.total_tiles), dim3(BLOCK), 0, s, ws.ranges, ws.queue, cap,
                     reinterpret_cast<const uint32_t *>(ws.entries), ws.ids);
}

// ------------------------------------------------------- work order

// The rasteriser's work order as a kernel of its own (one block), for the
// autotuner's trials.
__global__ __launch_bounds__(QUEUE_BLOCK) void k_queue_order(const uint32_t *__restrict__ tile_cost,
                                                             const uint32_t *__restrict__ hdr, int total,
                                                             uint32_t *__restrict__ queue) {
  __shared__ uint32_t s_cnt[RADIX];
  __shared__ uint32_t s_cur[RADIX];
  __shared__ uint32_t s_w[QUEUE_BLOCK / 64];
  order_tiles<QUEUE_BLOCK>(tile_cost, hdr[HDR_COSTS] != 0u, total, queue, s_cnt, s_cur, s_w);
}

void launch_queue_order(const Workspace &ws, int total_tiles, hipStream_t s) {
  if (total_tiles > 0)
    hipLaunchKernelGGL(k_queue_order, dim3(1), dim3(QUEUE_BLOCK), 0, s, ws.tile_cost, ws.hdr, total_tiles,
                       ws.queue);
}

}  // namespace gsr
