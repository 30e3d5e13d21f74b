// Tile lists: every tile's Gaussians in blending order, the lexicographic
// (tile, float32 depth bits, index) order.
//
// The tiles of a view are grouped into bins of S x S (S = 1, 2 or 4, chosen
// per view by gsr_plan).  A record (one Gaussian in one view) becomes one
// entry (depth key, record id, mask of the bin's tiles it reaches) in every
// bin it reaches: a few entries instead of one pair per tile.  The projection
// writes each block's entries grouped by bin, with the offsets of the groups;
// one block per bin then collects its groups, sorts them by depth in LDS and
// writes the lists of all its tiles from the masks.  So the lists take one
// kernel beside the projection whatever the sizes, with no global sort.
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
// depths are put in index order afterwards (entries of a single depth are sorted
// by their index at once).  A bin with more than `cap` entries is taken in
// rounds of consecutive key ranges, which several blocks share (see "crowded
// bins").  A tile's list is the sorted entries whose mask has the tile's bit: per row of 64 entries one
// ballot gives the tile's entries and each lane's place, so consecutive lanes
// write consecutive words.
//
// Bound by the latency of the reads of the entries and by the block's LDS (one
// block a CU at its 12 288 entries).  A bin of 7 000 entries (72 views of
// 500 000 Gaussians) took 67 us: 20 to collect its groups, 10 to order the
// slots, 8 for the masks and 21 to write.  It takes 51 us with the group table
// read at once and four groups in flight (13), up to four entries of a slot
// ordered in registers (8), id and mask read together, and the places counted
// from the tile's next one in the lanes' registers (12): 5 512 bins 1.65 -> 1.14
// ms, the 209 bins of 2 500 of a 1200x680 view 39 -> 33 us.
constexpr int LB = 1024;         // threads
constexpr int LW = LB / 64;      // wavefronts
constexpr int LBITS = 8;         // bits per digit pass
constexpr int LDIGITS = 1 << LBITS;
constexpr int LRUN = 24;         // longest run of equal depths that one thread orders
constexpr int LPARTS = 4096;     // parts of the depth range
constexpr uint32_t LSLOT = 24;   // most entries of a slot that one thread orders
constexpr int NTILE = BIN_MAX * BIN_MAX;
constexpr int LBOUNDS = 256;     // rounds that one histogram gives the ends of
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
  uint32_t total[NTILE], before[NTILE];  // a crowded bin's entries of each tile, and those in front of the round
  uint16_t bound[LBOUNDS];     // ends of its rounds
  uint32_t bounds;
  uint32_t share[3];           // crowd_share's answer
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
    for (int i = 0; i < N; ++i) k[i] = i < n ? a.key[f[i]] : 0xFFFFFFFFu;  // (no key: neither a depth nor an id)
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
      uint32_t e[LUNROLL], q[LUNROLL], left[LUNROLL], most = 0u;
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
          most = max(most, left[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < LUNROLL; ++u)
        if (left[u]) v[u] = load(e[u]);
#pragma unroll
      for (int u = 0; u < LUNROLL; ++u)
        if (left[u]) use(q[u], e[u], v[u]);
      // What longer groups have left.
      for (uint32_t k = LTEAM; k < most; k += LTEAM) {
#pragma unroll
        for (int u = 0; u < LUNROLL; ++u)
          if (k < left[u]) v[u] = load(e[u] + k);
#pragma unroll
        for (int u = 0; u < LUNROLL; ++u)
          if (k < left[u]) use(q[u] + k, e[u] + k, v[u]);
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

// order_masks and write_lists by the bin's edge.
__device__ __forceinline__ void masks_of(int shift, ListsLds &s, const ListsArrays &a, const Entry *entries, int n, int I,
                                         int at) {
  if (shift == 2) order_masks<16>(s, a, entries, n, I, at);
  else if (shift == 1) order_masks<4>(s, a, entries, n, I, at);
  else order_masks<1>(s, a, entries, n, I, at);
}

__device__ __forceinline__ void lists_of(int shift, const ListsLds &s, const ListsArrays &a, uint32_t *ids, int n, int I,
                                         int at) {
  if (shift == 2) write_lists<16>(s, a, ids, n, I, at);
  else if (shift == 1) write_lists<4>(s, a, ids, n, I, at);
  else write_lists<1>(s, a, ids, n, I, at);
}

// Exclusive scan over the tiles (lanes below NTILE of a whole wavefront; the
// other lanes have v = 0), and the sum.
__device__ __forceinline__ uint32_t tile_scan(uint32_t v, uint32_t &all) {
  const int lane = threadIdx.x & 63;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < NTILE; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  all = __shfl(x, NTILE - 1);
  return x - v;
}

// ---------------------------------------------------------- crowded bins
//
// A map seen from afar lies in a few bins, which then have hundreds of
// thousands of entries.  Each pass over them is the work of one block, but the
// rounds are independent once their ends are known, so they are shared: the
// plan adds blocks behind the bins' own (lists_helpers) that look for crowded
// bins.  A helper finds the bin's entries, the rounds' ends and the tiles'
// totals for itself, as the bin's own block does, and takes every parts-th
// round.  What they must agree on depends on the entries alone, but for the
// place of the lists (shared_reserve).
//
// Bound by what one CU reads: a pass over 120 000 entries takes a block 60 to
// 80 us (25 GB/s), and a block makes three, for the keys, the histogram and its
// round; a round of 12 288 is sorted and written in 55.  Lists of 400 000 and
// 1.6 M Gaussians in four bins of 640x480: 3.1 and 57 ms by one block a bin with
// two passes for every round, 0.41 and 1.4 ms so.  A forward of a million at a
// quarter, a tenth and a twentieth of the view's width 3.6, 14 and 26 ms -> 0.78,
// 1.27 and 2.8 (by radix passes over all pairs 0.89, 1.25, 3.9); with all of
// them in view, where every bin has 1.3 rounds, 405 -> 343 us.

// Entries of each tile of the bin among a thread's own.
__device__ __forceinline__ void count_mask(uint32_t c[NTILE], uint32_t mask) {
#pragma unroll
  for (int t = 0; t < NTILE; ++t) c[t] += (mask >> t) & 1u;
}

// to[] += the block's counts (by all threads).
__device__ __forceinline__ void add_counts(const uint32_t c[NTILE], uint32_t to[NTILE]) {
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    int x = (int)c[t];
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    if ((threadIdx.x & 63) == 63 && x) atomicAdd(&to[t], (uint32_t)x);
  }
}

// Ends of the rounds (s.bound, in parts) by one wavefront: rounds of about equal
// size, cap entries at most, up to a part that alone has more than cap.
// front[]: entries in front of each part, s.end: of all.
__device__ __forceinline__ void round_ends(ListsLds &s, const uint32_t *front, int cap) {
  const int lane = threadIdx.x;
  const uint32_t total = s.end;
  const auto at = [&](int p) { return p < LPARTS ? front[p] : total; };
  const uint32_t rounds = (total + (uint32_t)cap - 1u) / (uint32_t)cap;
  // (a sixteenth more than an equal share, lest what the parts leave over makes
  // a round of its own)
  const uint32_t even = rounds ? total / rounds + total / (16u * rounds) + 64u : 0u;
  int start = 0, bounds = 0;
  while (start < LPARTS && bounds < LBOUNDS) {
    int q = start;
    for (uint32_t most = min(even, (uint32_t)cap);; most = (uint32_t)cap) {
      // Last part boundary q with at most that many entries between start and
      // it: 64 boundaries 64 apart, then the 64 from there on.  (The counts
      // ascend: those in front of the first that fails.)
      const uint32_t limit = at(start) + most;
#pragma unroll
      for (int step = 64; step > 0; step /= 64) {
        const int p = q + (lane + 1) * step;
        q += step * __popcll(__ballot(p <= LPARTS && at(p) <= limit));
      }
      if (q > start || most == (uint32_t)cap) break;
    }
    if (q == start) break;
    if (lane == 0) s.bound[bounds] = (uint16_t)q;
    ++bounds;
    start = q;
  }
  if (lane == 0) s.bounds = (uint32_t)bounds;
}

// Helpers and their bins.  Every block that asks finds the same: the entries of
// each bin are estimated from some of its view's groups, a bin that may be
// crowded asks for as many blocks as it has rounds, and the helpers are dealt
// out in the order of the bins.  The estimate decides on speed alone.  For
// helper number `idx` (want < 0) returns its bin, -1 for none; for the bin
// `want` itself; with the block's part of how many.
constexpr int CROWD_WORDS = 65536;  // of the group table, read by a block at most (but for 8 groups a view)
__device__ __forceinline__ int crowd_share(ListsLds &s, uint32_t *est, const Workspace &ws,
                                           const ViewInfo *__restrict__ views, const int32_t *__restrict__ bin_view,
                                           int total_bins, int groups, int cap, int helpers, int want, int idx, int &part,
                                           int &parts) {
  const int sample = min(groups, max(8, min(64, CROWD_WORDS / total_bins)));
  const int slices = max(1, min(sample, LB / total_bins));
  for (int b = threadIdx.x; b < total_bins; b += LB) est[b] = 0u;
  if (threadIdx.x == 0) s.share[0] = 0xFFFFFFFFu;
  __syncthreads();
  for (int t = threadIdx.x; t < total_bins * slices; t += LB) {
    const int b = t % total_bins, view = bin_view[b];
    const ViewInfo &vi = views[view];
    const int stride = vi.BX * vi.BY + 1;
    const uint32_t *row0 = ws.group_off + vi.mat_off + (b - vi.bin_off);
    const uint32_t *bases = ws.block_base + (size_t)view * groups;
    uint32_t sum = 0u;
#pragma unroll 4
    for (int j = t / total_bins; j < sample; j += slices) {
      const int g = (int)((int64_t)j * groups / sample);
      const uint32_t *row = row0 + (int64_t)g * stride;
      const uint32_t base = bases[g], r0 = row[0], r1 = row[1];
      sum += base != NO_BASE ? r1 - r0 : 0u;
    }
    if (sum) atomicAdd(&est[b], sum);
  }
  __syncthreads();
  // Blocks that a bin asks for beside its own.
  const auto asked = [&](int b) {
    const uint64_t e = (uint64_t)est[b] * (uint32_t)groups / (uint32_t)sample;
    return (uint32_t)min((e + (e >> 3) + (uint64_t)cap - 1ull) / (uint32_t)cap, (uint64_t)helpers + 1ull);
  };
  const int per = (total_bins + LB - 1) / LB;
  const int b0 = min((int)threadIdx.x * per, total_bins), b1 = min(b0 + per, total_bins);
  uint32_t sum = 0u, all, dealt;
  for (int b = b0; b < b1; ++b) {
    const uint32_t k = asked(b);
    sum += k > 1u ? k - 1u : 0u;
  }
  (void)block_exclusive_scan<LB>(sum, s.w, all);
  const auto gets = [&](int b) {
    const uint32_t k = asked(b), more = k > 1u ? k - 1u : 0u;
    return all > (uint32_t)helpers ? (uint32_t)((uint64_t)more * (uint32_t)helpers / all) : more;
  };
  sum = 0u;
  for (int b = b0; b < b1; ++b) sum += gets(b);
  uint32_t first = block_exclusive_scan<LB>(sum, s.w, dealt);
  for (int b = b0; b < b1; ++b) {
    const uint32_t k = gets(b);
    if (want < 0 ? (uint32_t)idx - first < k : b == want) {
      s.share[0] = (uint32_t)b;
      s.share[1] = want < 0 ? (uint32_t)idx - first + 1u : 0u;
      s.share[2] = k + 1u;
    }
    first += k;
  }
  __syncthreads();
  part = (int)s.share[1];
  parts = (int)s.share[2];
  return (int)s.share[0];
}

// Place of the lists of a bin that several blocks write.  The first of them that
// comes to shared_reserve (one thread, once the tiles' totals are known) takes
// it and tells the others in shared_place: 0 before that, 1 while it is taken,
// then the place + 2, or NO_PLACE past the capacity.  shared_wait, needed a
// collecting pass and a sort later, hardly ever waits, and always ends: 1 was
// written by a block that is running and waits for nothing before the place
// follows.  Relaxed atomics do: the words carry all that is told.  (Acquire and
// release at device scope write back and invalidate the L2 under the other
// blocks' reads and writes, and a chain of compare-and-swaps on one word, which
// needs no wait, takes 1.4 us a bin: 990 and 660 us for 209 bins.)
constexpr unsigned long long NO_PLACE = ~0ull;

__device__ __forceinline__ void shared_reserve(const Workspace &ws, int bin, uint32_t all, unsigned long long cap_pairs) {
  unsigned long long *word = ws.shared_place + bin;
  if (atomicCAS(word, 0ull, 1ull) != 0ull) return;
  const unsigned long long first =
      atomicAdd(reinterpret_cast<unsigned long long *>(ws.hdr + HDR_NLISTED), (unsigned long long)all);
  (void)atomicExch(word, first + all <= cap_pairs ? first + 2ull : NO_PLACE);
}

__device__ __forceinline__ unsigned long long shared_wait(const Workspace &ws, int bin) {
  unsigned long long v;
  while ((v = __hip_atomic_load(ws.shared_place + bin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < 2ull)
    __builtin_amdgcn_s_sleep(4);
  return v == NO_PLACE ? NO_PLACE : v - 2ull;
}

__global__ __launch_bounds__(LB) void k_bin_lists(const ViewInfo *__restrict__ views,
                                                  const int32_t *__restrict__ bin_view, Workspace ws, int64_t n_gauss,
                                                  int id_bits, int groups, int pre_blocks, unsigned long long cap_pairs,
                                                  int cap, int order_total, int n_views, int total_bins, int helpers) {
  extern __shared__ uint32_t dyn[];
  __shared__ ListsLds s;
  if (blockIdx.x == 0) {
    // The pair count, and the overflow record when it exceeds the capacity.
    unsigned long long x = 0ull;
    for (int j = threadIdx.x; j < pre_blocks; j += LB) x += ws.block_pairs[j] & PAIRS_MASK;
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
  // Blocks behind the bins' help with the crowded ones.
  int bin = (int)blockIdx.x - 2, part = 0, parts = 1;
  const bool helper = bin >= total_bins;
  if (helper) {
    // No bin has more entries than the blocks of its view together allow: most
    // calls end here, and their helpers on the CUs that no bin needs (the ones of
    // 1200x680 are gone in half the time of its bins; those that went on to the
    // estimate, on a bound of the largest group alone, made its lists 1.5 us
    // longer).
    const int bpv = pre_blocks / n_views;
    bool crowd = false;
    for (int v = threadIdx.x >> 6; v < n_views; v += LW) {
      uint32_t sum = 0u;
      for (int j = threadIdx.x & 63; j < bpv; j += 64) sum += (uint32_t)(ws.block_pairs[(size_t)v * bpv + j] >> PAIRS_BITS);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
      crowd = crowd || sum > (uint32_t)cap;
    }
    if (!__syncthreads_or(crowd)) return;
    bin = crowd_share(s, dyn, ws, views, bin_view, total_bins, groups, cap, helpers, -1, bin - total_bins, part, parts);
    if (bin < 0) return;
  }
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
  if (E <= cap) {
    if (helper) return;
    if (E == 0) {
      if (my_tile) ws.ranges[tile] = make_int2(0, 0);
      return;
    }
    uint32_t key0 = s.kmin, key1 = s.kmax;
    if (key0 == key1) {
      // One depth: by index.
      for (int q = threadIdx.x; q < E; q += LB) a.key[q] = entries[a.at[q]].id;
      key0 = id0;
      key1 = id0 + (uint32_t)n_gauss - 1u;
      __syncthreads();
    }
    const int I = (E + LB - 1) / LB;
    const int at = wave * 64 * I + lane;
    sort_entries(s, a, E, I, at, key0, key1 == key0 ? 0 : 32 - __clz(key1 - key0), entries, id0, id_bits);
    masks_of(shift, s, a, entries, E, I, at);
    __syncthreads();
    if (threadIdx.x < 64) {
      uint32_t tot = 0u;
      if (lane < nt) {
#pragma unroll
        for (int w = 0; w < LW; ++w) tot += s.tile[w][lane];
      }
      // The bin's lists take consecutive places, tile after tile, reserved
      // with one add on the listed-pair count.  Past the capacity (an
      // overflow) they stay empty.
      uint32_t all;
      const uint32_t pre = tile_scan(tot, all);
      unsigned long long first = 0ull;
      if (lane == 0)
        first = atomicAdd(reinterpret_cast<unsigned long long *>(ws.hdr + HDR_NLISTED), (unsigned long long)all);
      first = __shfl(first, 0);
      const bool fits = first + all <= cap_pairs;
      uint32_t place = (uint32_t)first + pre;
      if (lane == 0) s.most = fits ? 0u : 0xFFFFFFFFu;
      if (my_tile) ws.ranges[tile] = fits ? make_int2((int)place, (int)(place + tot)) : make_int2(0, 0);
      if (lane < nt) {
#pragma unroll
        for (int w = 0; w < LW; ++w) {
          const uint32_t k = s.tile[w][lane];
          s.tile[w][lane] = place;
          place += k;
        }
      }
    }
    __syncthreads();
    if (s.most == 0xFFFFFFFFu) return;
    lists_of(shift, s, a, ws.ids, E, I, at);
    return;
  }

  // A crowded bin: its rounds, every parts-th of them from `part` on.
  if (!helper) {
    part = 0;
    parts = 1;
    if (helpers > 0) crowd_share(s, dyn, ws, views, bin_view, total_bins, groups, cap, helpers, bin, -1, part, parts);
  }
  const uint32_t kmin = s.kmin, kmax = s.kmax;
  const uint64_t end = ((uint64_t)kmax << 32 | 0xFFFFFFFFull) + 1ull;
  uint64_t lo = (uint64_t)kmin << 32;
  uint64_t counted = lo;  // s.before holds the entries below it
  if (threadIdx.x < NTILE) s.total[threadIdx.x] = s.before[threadIdx.x] = 0u;
  const auto whole = [&](uint32_t e) { return entries[e]; };
  const auto unique = [](const Entry &e) { return (uint64_t)e.key << 32 | e.id; };
  int turn = 0;
  bool totals = false, reserved = false, placed = false;
  while (lo < end) {
    // The ends of the rounds come from a histogram over LPARTS equal parts of
    // what is left; where the first part alone exceeds cap it is divided
    // again.
    uint32_t *hist = a.key;
    int sh = 0;
    while ((end - lo) >> sh > (uint64_t)LPARTS) ++sh;
    for (;;) {
      __syncthreads();
      for (int b = threadIdx.x; b < LPARTS; b += LB) hist[b] = 0u;
      __syncthreads();
      uint32_t c[NTILE];
#pragma unroll
      for (int t = 0; t < NTILE; ++t) c[t] = 0u;
      for_entries(s, ws, vi, view, local, groups, whole, [&](uint32_t, uint32_t, const Entry &e) {
        const uint64_t k = unique(e);
        if (k >= lo && (k - lo) >> sh < (uint64_t)LPARTS) atomicAdd(&hist[(k - lo) >> sh], 1u);
        if (!totals) count_mask(c, e.mask);
      });
      if (!totals) add_counts(c, s.total);
      totals = true;
      // Entries in front of each part, then the rounds' ends.
      {
        constexpr int PER = LPARTS / LB;
        uint32_t h[PER], sum = 0u, total;
#pragma unroll
        for (int k = 0; k < PER; ++k) sum += h[k] = hist[threadIdx.x * PER + k];
        uint32_t run = block_exclusive_scan<LB>(sum, s.w, total);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          hist[threadIdx.x * PER + k] = run;
          run += h[k];
        }
        if (threadIdx.x == 0) s.end = total;
      }
      __syncthreads();
      if (threadIdx.x < 64) round_ends(s, hist, cap);
      if (threadIdx.x == 64 && parts > 1 && !reserved) {
        uint32_t all = 0u;
        for (int t = 0; t < NTILE; ++t) all += s.total[t];
        shared_reserve(ws, bin, all, cap_pairs);
      }
      reserved = true;
      __syncthreads();
      if (s.bounds > 0u) break;
      sh = sh > 12 ? sh - 12 : 0;  // (at sh = 0 a part is one key, which one entry has)
    }
    const int bounds = (int)s.bounds;
    uint64_t from = lo;
    for (int r = 0; r < bounds; ++r, ++turn) {
      const uint64_t first = from, last = min(lo + ((uint64_t)s.bound[r] << sh), end);
      from = last;
      if (turn % parts != part) continue;
      // The round's entries, and the tiles' entries in front of it.
      const bool one = first >> 32 == (last - 1ull) >> 32;  // a single depth: by index
      __syncthreads();
      if (threadIdx.x == 0) s.n = 0u;
      __syncthreads();
      uint32_t c[NTILE];
#pragma unroll
      for (int t = 0; t < NTILE; ++t) c[t] = 0u;
      for_entries(s, ws, vi, view, local, groups, whole, [&](uint32_t, uint32_t i, const Entry &e) {
        const uint64_t k = unique(e);
        if (k >= first && k < last) {
          const uint32_t q = atomicAdd(&s.n, 1u);
          a.key[q] = one ? e.id : e.key;
          a.at[q] = i;
        } else if (k >= counted && k < first) {
          count_mask(c, e.mask);
        }
      });
      add_counts(c, s.before);
      counted = last;
      __syncthreads();
      const int n = (int)s.n;
      if (n == 0) continue;
      const uint32_t key0 = one ? max((uint32_t)first, id0) : (uint32_t)(first >> 32);
      const uint32_t key1 = one ? min((uint32_t)(last - 1ull), id0 + (uint32_t)n_gauss - 1u)
                                : min((uint32_t)((last - 1ull) >> 32), kmax);
      const int I = (n + LB - 1) / LB;
      const int at = wave * 64 * I + lane;
      sort_entries(s, a, n, I, at, key0, key1 <= key0 ? 0 : 32 - __clz(key1 - key0), entries, id0, id_bits);
      masks_of(shift, s, a, entries, n, I, at);
      __syncthreads();
      if (threadIdx.x < 64) {
        if (!placed) {
          const uint32_t tot = lane < NTILE ? s.total[lane] : 0u;
          uint32_t all, start;
          const uint32_t pre = tile_scan(tot, all);
          unsigned long long at0 = 0ull;
          if (lane == 0) {
            if (parts > 1) {
              at0 = shared_wait(ws, bin);
            } else {
              at0 = atomicAdd(reinterpret_cast<unsigned long long *>(ws.hdr + HDR_NLISTED), (unsigned long long)all);
              if (at0 + all > cap_pairs) at0 = NO_PLACE;
            }
          }
          at0 = __shfl(at0, 0);
          const bool fits = at0 != NO_PLACE;
          start = (uint32_t)at0 + pre;
          if (lane == 0) s.most = fits ? 0u : 0xFFFFFFFFu;
          if (lane < NTILE) s.next[lane] = start;
          if (part == 0 && my_tile)
            ws.ranges[tile] = fits ? make_int2((int)start, (int)(start + tot)) : make_int2(0, 0);
        }
        if (lane < nt) {
          uint32_t seen = s.before[lane];
          const uint32_t start = s.next[lane];
#pragma unroll
          for (int w = 0; w < LW; ++w) {
            const uint32_t k = s.tile[w][lane];
            s.tile[w][lane] = start + seen;
            seen += k;
          }
          s.before[lane] = seen;
        }
      }
      __syncthreads();
      if (!placed && s.most == 0xFFFFFFFFu) return;
      placed = true;
      lists_of(shift, s, a, ws.ids, n, I, at);
    }
    lo = from;
  }
}

void launch_bin_lists(const Plan &p, const Workspace &ws, const ViewInfo *views, const int32_t *bin_view,
                      int order_total, hipStream_t s) {
  int id_bits = 1;
  while ((1ll << id_bits) < p.n) ++id_bits;
  hipLaunchKernelGGL(k_bin_lists, dim3((unsigned)(p.total_bins + p.lists_helpers) + 2u), dim3(LB), (size_t)p.lists_cap * LISTS_ENTRY_BYTES,
                     s, views, bin_view, ws, p.n, id_bits, p.blocks_per_view * p.pre_rounds, p.blocks_per_view * p.n_views,
                     (unsigned long long)p.capacity, p.lists_cap, order_total, p.n_views, p.total_bins, p.lists_helpers);
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
