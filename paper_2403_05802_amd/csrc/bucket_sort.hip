// The Sort operator for lists of many entries: most significant digits first.  The list is cut into parents, equal
// shares of the range of the key (one pass over memory), every parent into children of about BK_TARGET entries by splitters
// drawn from a sample of its own keys (a second pass), and a child is sorted where it lies in LDS while its sorted entries
// and the pointers of its rows are written.  Keys are unique, so splitters tell apart what one share leaves together
// (a heavy row of a power-law matrix fills several children), and no pass but the last has an order to keep: places inside
// a tile come from one LDS atomic per entry.
//
// Against the least-significant-digit passes of sort.hip: an entry travels as 8 bytes {key less the parent's first, value}
// instead of 12 and a digit byte, through two passes and the finish (52 bytes read and written in all, pointers of the
// rows included) instead of one pass per eight key bits (26 each).  COO -> CSR, digit passes / this, us: 16.8 M entries of a
// power-law matrix, 40 key bits, 695 / 425; 40 M with local columns, 42 bits, 1630 / 964; 4 M 238 / 172; 1 M, even rows
// 155 / 103; 300 k 138 / 94; 41 k, 24 bits (one parent) 88 / 78.
#include "device.h"
#include "sort_key.h"

namespace us {

constexpr int BK_CAP = 2048;        // most entries of a child: what the finish holds in LDS
constexpr int BK_TARGET = 1024;     // ... and how many it gets on average
constexpr int BK_MAXK = 128;        // most children of a parent
constexpr int BK_OVERSAMPLE = 64;   // sampled keys per child
constexpr int BK_MAXBITS = 10, BK_MAXSHARES = 1 << BK_MAXBITS;

// The parents are equal shares of the range that the major index really has, whole rows where there are more of them than
// parents (rows >= 1: share = major / rows, an exact division of 31 bits by multiplication), else pieces of 2^shift keys.
// (By the key's top bits half of the parents are empty when the row count lies just above a power of two, and the others
// twice as full: 40 M entries of a power-law matrix of 1,050,000 rows had a parent of more than BK_MAXK children, which sent
// the call back to the digit passes, 1657 us; now 933.  2,000,000 rows 933 / 937.)
struct KeyShares {
  uint32_t count, rows;
  uint32_t mul; int mul_shift;
  int shift;
  uint64_t width;              // keys of a share: at most 2^32
};

struct BkParent { uint32_t start, size, child0, k, tile0, region0; };

// BkArgs::child, third word: the share (BK_MAXBITS bits), where its entries are, the region of its parent's first child in rec2
constexpr uint32_t BK_SHARED = 1u << BK_MAXBITS;   // it has siblings (or comes from the caller's list): in its region, else in rec1
constexpr int BK_REGION_SHIFT = BK_MAXBITS + 1;

struct BkArgs {
  const int32_t *row, *col; const uint32_t *val;   // the caller's list
  uint32_t n; KeySpec ks;
  KeyShares share;
  // sample of the caller's list: if a share has crowded_at of its keys, those of heavy_at are cut into parents of about `unit`
  uint32_t nsamples, crowded_at, heavy_at, unit;
  uint16_t *sample_share;      // [nsamples rounded up to 8]
  uint32_t *sample_low;        // [nsamples]
  int clear_flags;             // the first kernel clears them
  uint32_t max_parents;        // shares + nsamples / unit
  uint16_t *first;             // [shares + 1] the first parent of every share, if any of them is cut, and ...
  uint32_t *split;             // ... [parents - shares] the smallest low keys of the further ones, share after share ...
  uint2 *origin;               // ... [max_parents] {share, smallest low key}
  int coo_vec;                 // row, col and val are 16-byte aligned
  // first pass: every workgroup takes per_group consecutive entries
  uint32_t per_group, ngroups, groups_per_xcd;
  uint32_t *hist;              // [ngroups][max_parents] entries per group and parent, then where they start inside the parent
  uint32_t *ptotal;            // [max_parents] entries per parent
  uint2 *rec1;                 // [n] {low key, value}, by parent
  // second pass
  BkParent *parent;            // [max_parents]
  uint32_t *totals;            // [0] children, [1] tiles of parents with more than one child, [2] parents: more than shares if any is cut
  uint4 *child;                // [max_children] {start of the parent, its first child, share and BK_*, smallest low key}
  uint32_t *cursor;            // [max_children] entries of the child
  uint32_t *tile_parent;       // [max_tiles]
  uint32_t max_children, max_regions, max_tiles;
  int tile_chunk, child_chunk;   // (xcd_chunk_item)
  uint2 *rec2;                 // [max_regions][BK_CAP]: the children that share a parent
  // output
  int32_t *major_out, *minor_out; uint32_t *val_out;
  int32_t *ptr; uint32_t ngroups_out;   // pointers over the major indices 0..ngroups_out, or null
  Flags *flags;
};

// (a coordinate out of range is reported, not sorted: it only has to fall into some share)
__device__ __forceinline__ uint32_t share_of_lead(const KeyShares &s, uint32_t lead) {
  return min(__umulhi(lead << 1, s.mul) >> s.mul_shift, s.count - 1);
}
// the entry's share and the rest of its key
__device__ __forceinline__ uint32_t share_of_entry(const BkArgs &a, uint32_t r, uint32_t c, uint32_t *low) {
  const uint32_t lead = a.ks.swap ? c : r, minor = a.ks.swap ? r : c;
  if (a.share.rows) {
    const uint32_t s = share_of_lead(a.share, lead);
    *low = ((lead - s * a.share.rows) << a.ks.b_bits) | minor;
    return s;
  }
  const Key key = ((Key)lead << a.ks.b_bits) | minor;
  *low = (uint32_t)key & (uint32_t)(a.share.width - 1);
  return (uint32_t)min(key >> a.share.shift, (Key)(a.share.count - 1));
}

// A kernel of the call has given up: a coordinate out of range, or an input this sort does not take.  The tables that later
// kernels index with may then be unwritten.  Read once per workgroup, because workgroups of the same launch may set it.
__device__ __forceinline__ bool gave_up(const BkArgs &a, bool range) {
  __shared__ int32_t s_stop;
  if (threadIdx.x == 0) s_stop = (range ? a.flags->index_range : 0) | a.flags->retry;
  __syncthreads();
  return s_stop != 0;
}

// Neighbouring items (a parent's tiles, the ends of what children write) on the same XCD, 2^shift of them: how many there are
// only the GPU knows, and a contiguous range of the most possible for each XCD would leave the last one with less to do.
__device__ __forceinline__ uint32_t xcd_chunk_item(uint32_t i, int shift) {
  const uint32_t at = i >> 3;
  return ((at >> shift) * 8 + (i & 7u)) << shift | (at & ((1u << shift) - 1u));
}

// Exclusive prefix sum over the workgroup with one barrier; s_wave: T / 64 words, free again after the next barrier.
template <int T>
__device__ __forceinline__ uint32_t scan_one_barrier(uint32_t v, uint32_t *s_wave) {
  const uint32_t inc = wave_inclusive_sum_dpp(v);
  if (lane_id() == 63) s_wave[wave_id()] = inc;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) before += w < wave_id() ? s_wave[w] : 0u;
  return before + inc - v;
}

// ------------------------------------------------------------------ first pass: parents
// Some shares hold more entries than a parent may (rows in order of their length, the quadrants of an R-MAT graph, a few
// rows that are used at all).  A sample of the caller's list, 64 keys per 131,072 entries while there are up to 33.5 M, tells
// whether one does and where to cut the heavy ones: into parents of 41 k entries on average, 20 keys of the sample.  Every
// workgroup of the histogram looks through the sample by itself, so no launch waits for one of them; only where a share
// has to be cut the keys are sorted, by all of them the same.  A parent that is too large all the same is noticed by the scan.
// Digit passes / a failed first pass, then the digit passes / this, us: 16.8 M entries with rows in order of their length 688 /
// 784 / 555, R-MAT 681 / 755 / 543; 4 M 215 / 296 / 189 and 228 / 300 / 188; 1 M 153 / 224 / 118 and 164 / 235 / 118.  Without
// a share too many the sample costs what the clearing of the flags, which it takes over, did (16.8 M entries 405 -> 411, 40 M
// 935 -> 937, 1 M 103 -> 104); a histogram with cut shares takes 150 instead of 24 (sort and searches; 512 threads instead of
// 1024: 280), the scatter 139 instead of 102.
constexpr int BL_T = 256;
__global__ __launch_bounds__(BL_T) void bucket_probe_kernel(BkArgs a) {
  const uint32_t i = blockIdx.x * BL_T + threadIdx.x;
  if (a.clear_flags && i < sizeof(Flags) / 4) reinterpret_cast<uint32_t *>(a.flags)[i] = 0;
  if (i >= ((a.nsamples + 7) & ~7u)) return;
  uint32_t share = 0xFFFFu;   // (none)
  if (i < a.nsamples) {
    // evenly spaced pieces of the list, at a scattered place in each (lists often come in a regular order)
    const uint32_t piece = a.n / a.nsamples, at = (uint32_t)((uint64_t)i * a.n / a.nsamples) + ((i * 0x9E3779B1u) >> 8) % piece;
    uint32_t low;
    share = share_of_entry(a, (uint32_t)a.row[at], (uint32_t)a.col[at], &low);
    a.sample_low[i] = low;
  }
  a.sample_share[i] = (uint16_t)share;
}

// the parent of an entry where shares are cut: the last one of its share whose smallest low key is not above the entry's
__device__ __forceinline__ uint32_t parent_of(const uint16_t *first, const uint32_t *split, uint32_t share, uint32_t low) {
  const uint32_t f = first[share];
  uint32_t b = f - share, e = first[share + 1] - share - 1;   // the splitters of the share
  while (b < e) {
    const uint32_t mid = (b + e) >> 1;
    if (split[mid] <= low) b = mid + 1; else e = mid;
  }
  return share + b;
}

constexpr int BH_COPIES = 4;

// NS: room for the sample, MAXX: most parents beside the shares
template <int BH_T, int NS, int MAXX>
__global__ __launch_bounds__(BH_T) void bucket_hist_kernel(BkArgs a) {
  __shared__ union {
    uint32_t hist[(BK_MAXSHARES + MAXX) * BH_COPIES];   // (copies picked by lane: LDS adds to one address take turns)
    uint64_t key[NS];
  } s;
  __shared__ uint32_t s_cnt[BK_MAXSHARES];   // keys of the sample per share
  __shared__ uint16_t s_at[BK_MAXSHARES], s_first[BK_MAXSHARES + 2];
  __shared__ uint32_t s_split[MAXX], s_wave[2][BH_T / 64], s_n;
  const uint32_t group = xcd_tile(blockIdx.x, a.groups_per_xcd);
  if (group >= a.ngroups) return;
  const int tid = threadIdx.x;
  const uint32_t nshares = a.share.count;
  bool cut = false;
  if (a.nsamples) {
    for (uint32_t p = tid; p < BK_MAXSHARES; p += BH_T) s_cnt[p] = 0;
    if (tid == 0) s_n = 0;
    __syncthreads();
    const uint4 *v8 = reinterpret_cast<const uint4 *>(a.sample_share);   // eight at a time
    constexpr int EACH = NS / 8 / BH_T;
    uint4 x[EACH];
#pragma unroll
    for (int q = 0; q < EACH; ++q) {
      x[q] = make_uint4(~0u, ~0u, ~0u, ~0u);
      if (8u * (q * BH_T + tid) < a.nsamples) x[q] = v8[q * BH_T + tid];
    }
#pragma unroll
    for (int q = 0; q < EACH; ++q) {
      const uint32_t w[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        if ((w[y] & 0xFFFFu) != 0xFFFFu) atomicAdd(&s_cnt[w[y] & 0xFFFFu], 1u);
        if (w[y] >> 16 != 0xFFFFu) atomicAdd(&s_cnt[w[y] >> 16], 1u);
      }
    }
    __syncthreads();
    bool crowded = false;
    for (uint32_t p = tid; p < nshares; p += BH_T) crowded |= s_cnt[p] >= a.crowded_at;
    if (crowded) s_n = 1;
    __syncthreads();
    cut = s_n != 0;
  }
  uint32_t np = nshares;
  if (cut) {
    constexpr int PER = BK_MAXSHARES / BH_T;
    uint32_t c[PER], more[PER], msum = 0, csum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      c[q] = s_cnt[tid * PER + q];
      more[q] = c[q] >= a.heavy_at ? (c[q] - 1) / a.unit : 0u;
      if (!more[q]) c[q] = 0;
      msum += more[q]; csum += c[q];
    }
    uint32_t m0 = scan_one_barrier<BH_T>(msum, s_wave[0]), c0 = scan_one_barrier<BH_T>(csum, s_wave[1]);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t p = tid * PER + q;
      s_first[p] = (uint16_t)(p + m0); s_at[p] = (uint16_t)c0;
      m0 += more[q]; c0 += c[q];
      if (p + 1 == (uint32_t)BK_MAXSHARES) s_first[p + 1] = (uint16_t)(p + 1 + m0);
    }
    if (tid == 0) s_n = 0;
    __syncthreads();
    for (uint32_t i = tid; i < a.nsamples; i += BH_T) {
      const uint32_t p = a.sample_share[i];
      if (s_first[p + 1] - s_first[p] > 1) s.key[atomicAdd(&s_n, 1u)] = (uint64_t)p << 32 | a.sample_low[i];   // nsamples <= NS
    }
    __syncthreads();
    const uint32_t m = s_n;
    uint32_t size = 1;
    while (size < m) size <<= 1;
    for (uint32_t i = m + tid; i < size; i += BH_T) s.key[i] = ~0ull;   // (NS is a power of two)
    __syncthreads();
    for (uint32_t k = 2; k <= size; k <<= 1) {
      for (uint32_t half = k >> 1; half > 0; half >>= 1) {   // all comparisons ascending
        const uint32_t flip = half == k >> 1 ? k - 1 : half;
        for (uint32_t t = tid; t < size / 2; t += BH_T) {
          const uint32_t x = (t & (half - 1)) + ((t & ~(half - 1)) << 1), y = x ^ flip;
          const uint64_t kx = s.key[x], ky = s.key[y];
          if (kx > ky) { s.key[x] = ky; s.key[y] = kx; }
        }
        __syncthreads();
      }
    }
    for (uint32_t i = tid; i < m; i += BH_T) {   // key j * count / parents of a share starts its parent j
      const uint32_t p = (uint32_t)(s.key[i] >> 32), q = i - s_at[p], parents = s_first[p + 1] - s_first[p];
      const uint32_t j = (q * parents + s_cnt[p] - 1) / s_cnt[p];
      if (j >= 1 && j < parents && j * s_cnt[p] / parents == q) s_split[s_first[p] - p + j - 1] = (uint32_t)s.key[i];
    }
    np = s_first[nshares];
    __syncthreads();
    if (group == 0) {
      for (uint32_t p = tid; p <= nshares; p += BH_T) a.first[p] = s_first[p];
      for (uint32_t p = tid; p < np - nshares; p += BH_T) a.split[p] = s_split[p];
      for (uint32_t p = tid; p < nshares; p += BH_T)
        for (uint32_t f = s_first[p], x = f; x < s_first[p + 1]; ++x) a.origin[x] = make_uint2(p, x > f ? s_split[x - p - 1] : 0u);
    }
  }
  if (group == 0 && tid == 0) a.totals[2] = np;
  for (uint32_t i = tid; i < np * BH_COPIES; i += BH_T) s.hist[i] = 0;
  __syncthreads();
  const uint32_t begin = group * a.per_group, end = min(begin + a.per_group, a.n);
  const uint32_t copy = tid & (BH_COPIES - 1);
  const int32_t *lead = a.ks.swap ? a.col : a.row;
  auto count = [&](uint32_t p) { atomicAdd(&s.hist[p * BH_COPIES + copy], 1u); };
  auto of_lead = [&](uint32_t x) { return share_of_lead(a.share, x); };
  uint32_t i = begin;
  if (a.share.rows && a.coo_vec && !cut) {
    for (; i + 8 * BH_T <= end; i += 8 * BH_T) {   // (begin is a multiple of four entries)
      const uint4 *p4 = reinterpret_cast<const uint4 *>(lead + i);
      const uint4 x = p4[tid], y = p4[BH_T + tid];
      count(of_lead(x.x)); count(of_lead(x.y)); count(of_lead(x.z)); count(of_lead(x.w));
      count(of_lead(y.x)); count(of_lead(y.y)); count(of_lead(y.z)); count(of_lead(y.w));
    }
  }
  if (a.share.rows && !cut) {
    for (uint32_t e = i + tid; e < end; e += BH_T) count(of_lead((uint32_t)lead[e]));
  } else {
    constexpr int N = 4;
    for (; i < end; i += N * BH_T) {
      uint32_t r[N], c[N], p[N], low[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const uint32_t e = min(i + j * BH_T + tid, end - 1);
        r[j] = (uint32_t)a.row[e]; c[j] = (uint32_t)a.col[e];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        p[j] = share_of_entry(a, r[j], c[j], &low[j]);
        if (i + j * BH_T + tid >= end) p[j] = 0xFFFFFFFFu;
      }
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (p[j] != 0xFFFFFFFFu) count(cut ? parent_of(s_first, s_split, p[j], low[j]) : p[j]);
    }
  }
  __syncthreads();
  for (uint32_t p = tid; p < np; p += BH_T) {
    uint32_t sum = 0;
#pragma unroll
    for (int c = 0; c < BH_COPIES; ++c) sum += s.hist[p * BH_COPIES + c];
    a.hist[(size_t)group * a.max_parents + p] = sum;
  }
}

// where the entries of every group start inside their parent, and the parents' sizes: a workgroup takes 32 parents, its
// threads 32 consecutive ranges of groups each
constexpr int BS_T = 1024, BS_BINS = 32, BS_PARTS = BS_T / BS_BINS;
__global__ __launch_bounds__(BS_T) void bucket_scan_kernel(BkArgs a) {
  __shared__ uint32_t s_part[BS_PARTS][BS_BINS];
  const uint32_t q = threadIdx.x % BS_BINS, part = threadIdx.x / BS_BINS, p = blockIdx.x * BS_BINS + q;
  const uint32_t np = a.totals[2], each = (a.ngroups + BS_PARTS - 1) / BS_PARTS, g0 = min(part * each, a.ngroups), g1 = min(g0 + each, a.ngroups);
  uint32_t sum = 0;
  if (p < a.share.count || p < np) {   // (the loads of a share's own parent do not wait for the number of parents)
#pragma unroll 8
    for (uint32_t g = g0; g < g1; ++g) sum += a.hist[(size_t)g * a.max_parents + p];
  }
  s_part[part][q] = sum;
  __syncthreads();
  uint32_t run = 0;
  for (uint32_t w = 0; w < part; ++w) run += s_part[w][q];
  if (p >= np) return;
  if (part == BS_PARTS - 1) {
    a.ptotal[p] = run + sum;
    if (run + sum > (uint32_t)(BK_MAXK * BK_TARGET)) a.flags->retry = RETRY_SORT_LDS;   // (the kernels that follow leave at once)
  }
#pragma unroll 8
  for (uint32_t g = g0; g < g1; ++g) {
    uint32_t *h = a.hist + (size_t)g * a.max_parents + p;
    const uint32_t v = *h;
    *h = run;
    run += v;
  }
}

// A workgroup walks its range tile by tile: places inside the tile by LDS atomics, the tile put in order of the parents
// in LDS, every parent's run written as one piece behind the workgroup's earlier ones.  Its runs are short (12 entries of a
// tile of 12,288 in 1024 parents) and leave lines partly written: ngroups x nparents of them are open at a time, 128 bytes
// each, against 4 MB of L2 per XCD.  By the counters it writes a quarter more than the records take (400 MB for 320, 40 M
// entries) and fetches the list once, 3.4 TB/s in all: scattered pieces and, with one workgroup per CU, its phases one
// after the other are what is left.  Few
// workgroups and large tiles where there are many entries.  512 threads x 8 entries and 768 workgroups / 1024 x 8 and 256
// / 1024 x 12 and 256, us: 40 M entries, 1024 parents 329 / 283 / 260; 16.8 M, 512 parents 110 / 98 / 101; 4 M, 128
// parents 22 / 24 / 28; 1 M 12 / 15 / 17.
template <int T, int IPT, int MAXX>
__global__ __launch_bounds__(T, T == 512 ? 6 : 4) void bucket_scatter_kernel(BkArgs a) {
  constexpr int TILE = T * IPT, MAXP = BK_MAXSHARES + MAXX, PER = (MAXP + T - 1) / T;
  __shared__ uint2 s_rec[TILE];
  __shared__ uint16_t s_bin[TILE];
  __shared__ uint32_t s_cnt[MAXP];    // entries of the tile per parent, then where they start in the tile
  __shared__ uint32_t s_goff[MAXP];   // position of the parent's run of this tile in rec1, minus its start in the tile
  __shared__ uint32_t s_split[MAXX];
  __shared__ uint16_t s_first[BK_MAXSHARES + 2];
  __shared__ uint32_t s_wave[2][T / 64];
  const uint32_t group = xcd_tile(blockIdx.x, a.groups_per_xcd);
  if (group >= a.ngroups || a.flags->retry) return;   // (set, if at all, by the kernel before)
  const uint32_t begin = group * a.per_group, end = min(begin + a.per_group, a.n);
  const int tid = threadIdx.x;
  const uint32_t np = a.totals[2], nshares = a.share.count;
  const bool cut = np != nshares;
  if (cut) {
    for (uint32_t p = tid; p <= nshares; p += T) s_first[p] = a.first[p];
    for (uint32_t p = tid; p < np - nshares; p += T) s_split[p] = a.split[p];
  }   // (read behind the scan's barrier)
  uint32_t next[PER];   // parents PER * tid ..: where the group's next entry goes
  {
    uint32_t t[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t p = tid * PER + q;
      t[q] = p < nshares || p < np ? a.ptotal[p] : 0u;
      next[q] = p < nshares || p < np ? a.hist[(size_t)group * a.max_parents + p] : 0u;
      if (p < MAXP) s_cnt[p] = 0;
      sum += t[q];
    }
    uint32_t run = scan_one_barrier<T>(sum, s_wave[0]);
#pragma unroll
    for (int q = 0; q < PER; ++q) { next[q] += run; run += t[q]; }
  }
  bool bad = false;
  for (uint32_t base = begin; base < end; base += TILE) {
    const uint32_t in_tile = min((uint32_t)TILE, end - base);
    uint32_t key[IPT], val[IPT], bin[IPT], arr[IPT];
    if (a.coo_vec && in_tile == (uint32_t)TILE) {
      const uint4 *r4 = reinterpret_cast<const uint4 *>(a.row + base), *c4 = reinterpret_cast<const uint4 *>(a.col + base);
      const uint4 *v4 = reinterpret_cast<const uint4 *>(a.val + base);
      uint4 rr[IPT / 4], cc[IPT / 4], vv[IPT / 4];
#pragma unroll
      for (int q = 0; q < IPT / 4; ++q) { rr[q] = r4[q * T + tid]; cc[q] = c4[q * T + tid]; vv[q] = v4[q * T + tid]; }
#pragma unroll
      for (int q = 0; q < IPT / 4; ++q) {
        const uint32_t r[4] = {rr[q].x, rr[q].y, rr[q].z, rr[q].w}, c[4] = {cc[q].x, cc[q].y, cc[q].z, cc[q].w};
        const uint32_t v[4] = {vv[q].x, vv[q].y, vv[q].z, vv[q].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bad |= coo_out_of_range(a.ks, r[e], c[e]);
          bin[4 * q + e] = share_of_entry(a, r[e], c[e], &key[4 * q + e]);
          val[4 * q + e] = v[e];
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        const uint32_t i = j * T + tid;
        bin[j] = 0xFFFFFFFFu; key[j] = 0; val[j] = 0;
        if (i < in_tile) {
          const uint32_t r = (uint32_t)a.row[base + i], c = (uint32_t)a.col[base + i];
          bad |= coo_out_of_range(a.ks, r, c);
          bin[j] = share_of_entry(a, r, c, &key[j]);
          val[j] = a.val[base + i];
        }
      }
    }
    if (cut) {
#pragma unroll
      for (int j = 0; j < IPT; ++j)
        if (bin[j] != 0xFFFFFFFFu) bin[j] = parent_of(s_first, s_split, bin[j], key[j]);
    }
    __syncthreads();   // s_cnt is clear, the previous tile is written
#pragma unroll
    for (int j = 0; j < IPT; ++j) arr[j] = bin[j] != 0xFFFFFFFFu ? atomicAdd(&s_cnt[bin[j]], 1u) : 0u;
    __syncthreads();
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) { c[q] = tid * PER + q < MAXP ? s_cnt[tid * PER + q] : 0u; sum += c[q]; }
    uint32_t run = scan_one_barrier<T>(sum, s_wave[1]);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (tid * PER + q < MAXP) {
        s_cnt[tid * PER + q] = run;
        s_goff[tid * PER + q] = next[q] - run;
      }
      next[q] += c[q]; run += c[q];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (bin[j] != 0xFFFFFFFFu) {
        const uint32_t pos = s_cnt[bin[j]] + arr[j];
        s_rec[pos] = make_uint2(key[j], val[j]);
        s_bin[pos] = (uint16_t)bin[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      const uint32_t i = j * T + tid;
      if (i < in_tile) {
        const uint32_t g = s_goff[s_bin[i]] + i;
        if (g < a.n) a.rec1[g] = s_rec[i];
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (tid * PER + q < MAXP) s_cnt[tid * PER + q] = 0;
  }
  if (bad) a.flags->index_range = 1;
}

// ------------------------------------------------------------------ a few thousand keys in LDS
// The keys go into bins that keep their order: 64 of the keys themselves, sorted by one wavefront, cut them into intervals of
// similar numbers of keys whatever their distribution, and every interval is cut evenly over its range into the same number
// of bins.  What is left together, one or two keys on average, fix_order puts in order.  A bin of more than LIMIT keys is
// cut again before, evenly between its own smallest and largest key, into as many bins as it has keys.  LDS and the
// chain of steps bound this: the splitters are held one per lane, every eighth in a scalar, and a key finds its
// interval by three comparisons with scalars and three with splitters fetched by ds_bpermute, which knows no bank
// conflicts; then it costs an atomic, a read and two writes at scattered places.
constexpr uint32_t BP_MOST = 129;
constexpr int BP_ROUNDS = 4;

// LIMIT 0: no bin is cut again, and the counters and the values share their place
template <int T, int IPT, uint32_t LIMIT>
struct BinScratch {
  static constexpr int NW = T / 64, Q = IPT / 4;   // wavefronts; blocks of four bins or slots per thread
  uint32_t a[T * IPT];
  uint32_t cnt[T * IPT + 4];
  uint32_t b_own[LIMIT ? T * IPT : 4];
  __device__ __forceinline__ uint32_t *b() { return LIMIT ? b_own : cnt; }
  uint32_t split[64];
  uint32_t wave[Q * NW], big[NW];
  uint32_t reach[Q * NW];   // per 256 slots: the most keys of a bin that touches them
};

// key[j] belongs to item j * T + threadIdx.x < m <= T * IPT, lo <= key <= hi; sample: the key of item threadIdx.x * m / 64
// (wavefront 0).  Leaves the slot of every item in order of the bins, s.reach, and returns the most keys of a bin, rounded
// up to 1, 5, 9, 17, 33, 65, BP_MOST or ~0 (the same for every thread).  Ends with a barrier: s.a and s.b() are free.
template <int T, int IPT, uint32_t LIMIT>
__device__ __forceinline__ uint32_t bin_slots(const uint32_t (&key)[IPT], uint32_t m, uint32_t lo, uint32_t hi, uint32_t sample,
                                              BinScratch<T, IPT, LIMIT> &s, uint32_t (&slot)[IPT]) {
  constexpr int CAP = T * IPT, NW = T / 64, Q = IPT / 4;
  static_assert(IPT % 4 == 0, "counters are cleared and read four at a time");
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  uint32_t bin[IPT], arr[IPT];
#pragma unroll
  for (int q = 0; q < Q; ++q) reinterpret_cast<uint4 *>(s.cnt)[q * T + tid] = make_uint4(0, 0, 0, 0);
  if (tid < Q * NW) s.reach[tid] = 0;
  if (w == 0) {
    s.split[lane] = ~0u;
    uint32_t rank = 0;
#pragma unroll 16
    for (int q = 0; q < 64; ++q) rank += (uint32_t)__builtin_amdgcn_readlane((int)sample, q) < sample;
    __builtin_amdgcn_wave_barrier();
    if (m >= 64) s.split[rank] = sample;
  }
  __syncthreads();
  {
    // lane i: interval i = [split i, split i + 1); two equal samples (a duplicate), the largest possible key among them or too
    // few keys leave a gap in the list: one interval then
    uint32_t sp = s.split[lane];
    const bool one = __any(sp == ~0u);
    if (one) sp = ~0u;
    if (lane == 0) sp = lo;
    const uint32_t per = one ? CAP : CAP / 64;
    uint32_t next = (uint32_t)__shfl_down((int)sp, 1);
    if (lane == 63 || next > hi) next = hi;
    const float scale = (float)per * __builtin_amdgcn_rcpf((float)(next - sp) + 1.f);
    uint32_t by8[8];
#pragma unroll
    for (int q = 1; q < 8; ++q) by8[q] = (uint32_t)__builtin_amdgcn_readlane((int)sp, 8 * q);
    uint32_t from[IPT];   // where the key's interval begins
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      bin[j] = 0; arr[j] = 0; from[j] = lo;
      if (j * T < m) {
        const uint32_t k = key[j];
        const bool c4 = by8[4] <= k;
        const uint32_t t2 = c4 ? by8[6] : by8[2];
        const bool c2 = t2 <= k;
        const uint32_t t1 = c4 ? (c2 ? by8[7] : by8[5]) : (c2 ? by8[3] : by8[1]);
        const bool c1 = t1 <= k;
        bin[j] = (c4 ? 32u : 0u) + (c2 ? 16u : 0u) + (c1 ? 8u : 0u);
        from[j] = c1 ? t1 : (c2 ? t2 : (c4 ? by8[4] : lo));
      }
    }
#pragma unroll
    for (int step = 4; step; step >>= 1) {
#pragma unroll
      for (int j = 0; j < IPT; ++j) {
        if (j * T < m) {
          const uint32_t v = (uint32_t)__shfl((int)sp, (int)(bin[j] + step));
          if (v <= key[j]) { bin[j] += step; from[j] = v; }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (j * T < m) {   // (rounding keeps the order of the keys)
        const float sc = __builtin_bit_cast(float, __shfl(__builtin_bit_cast(int, scale), (int)bin[j]));
        bin[j] = min(bin[j] * per + min((uint32_t)((float)(key[j] - from[j]) * sc), per - 1), (uint32_t)(CAP - 1));
      }
    }
  }
  uint32_t worst;
  for (int round = 0;; ++round) {
#pragma unroll
    for (int j = 0; j < IPT; ++j)
      if (j * T + tid < m) arr[j] = atomicAdd(&s.cnt[bin[j]], 1u);
    __syncthreads();
    uint32_t c[IPT], inc[Q], most = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint4 v = reinterpret_cast<const uint4 *>(s.cnt)[q * T + tid];
      c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
      most = max(max(most, max(v.x, v.y)), max(v.z, v.w));
      inc[q] = wave_inclusive_sum_dpp(v.x + v.y + v.z + v.w);
      if (lane == 63) s.wave[q * NW + w] = inc[q];
    }
    uint32_t big = 1;
    if (__any(most > 1)) {
      big = 5;
      if (__any(most > 5)) big = 9;
      if (__any(most > 9)) big = 17;
      if (__any(most > 17)) big = !__any(most > 33) ? 33u : !__any(most > 65) ? 65u : !__any(most > BP_MOST) ? BP_MOST : ~0u;
    }
    if (lane == 0) s.big[w] = big;
    __syncthreads();
    worst = 1;
#pragma unroll
    for (int x = 0; x < NW; ++x) worst = max(worst, s.big[x]);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint32_t run = inc[q] - (c[4 * q] + c[4 * q + 1] + c[4 * q + 2] + c[4 * q + 3]);
#pragma unroll
      for (int x = 0; x < Q * NW; ++x) run += x < q * NW + w ? s.wave[x] : 0u;
      uint4 v;
      v.x = run; v.y = v.x + c[4 * q]; v.z = v.y + c[4 * q + 1]; v.w = v.z + c[4 * q + 2];
      reinterpret_cast<uint4 *>(s.cnt)[q * T + tid] = v;
      if (q == Q - 1 && tid == T - 1) s.cnt[CAP] = v.w + c[4 * q + 3];
    }
    if (LIMIT == 0 || worst <= LIMIT || round == BP_ROUNDS) break;
    if constexpr (LIMIT > 0) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      reinterpret_cast<uint4 *>(s.a)[q * T + tid] = make_uint4(~0u, ~0u, ~0u, ~0u);
      reinterpret_cast<uint4 *>(s.b())[q * T + tid] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (j * T + tid < m) {
        const uint32_t st = s.cnt[bin[j]], count = s.cnt[bin[j] + 1] - st;
        slot[j] = bin[j];
        bin[j] = st;
        arr[j] = count;
        if (count > LIMIT) {
          atomicMin(&s.a[slot[j]], key[j]);
          atomicMax(&s.b()[slot[j]], key[j]);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
      if (j * T + tid < m && arr[j] > LIMIT) {
        const uint32_t mn = s.a[slot[j]], mx = s.b()[slot[j]];
        bin[j] += min((uint32_t)((float)(key[j] - mn) * ((float)arr[j] * __builtin_amdgcn_rcpf((float)(mx - mn) + 1.f))), arr[j] - 1);
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) reinterpret_cast<uint4 *>(s.cnt)[q * T + tid] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < IPT; ++j) {
    slot[j] = 0;
    if (j * T + tid < m) {
      const uint32_t st = s.cnt[bin[j]];
      slot[j] = st + arr[j];
      if (arr[j] >= 5) {   // (the last of a bin's keys to arrive says how many there are, where the bin begins and where it ends)
        atomicMax(&s.reach[st >> 8], arr[j] + 1);
        atomicMax(&s.reach[slot[j] >> 8], arr[j] + 1);
      }
    }
  }
  __syncthreads();
  return worst;
}

// The m items in s.a (keys) and s.b(), in order of the bins, into order of the keys: a key moves by the smaller ones behind it
// and the larger ones before it, and those lie fewer places away than its bin has keys; nothing beyond a bin's ends
// counts, so the bins need not be known.  Four items per thread and 16 bytes per read.  Ends with a barrier.
template <int T, int IPT, uint32_t LIMIT>
__device__ __forceinline__ void fix_order(uint32_t m, BinScratch<T, IPT, LIMIT> &s) {
  const uint4 *a4 = reinterpret_cast<const uint4 *>(s.a), *b4 = reinterpret_cast<const uint4 *>(s.b());
  const uint32_t n4 = (m + 3) / 4;
  if (threadIdx.x < 4 * n4 - m) s.a[m + threadIdx.x] = ~0u;
  __syncthreads();
  uint32_t k[IPT], v[IPT], pos[IPT];
#pragma unroll
  for (int q = 0; q < IPT / 4; ++q) {
    const uint32_t t = q * T + threadIdx.x;
    const uint32_t most = max(s.reach[t >> 6], 5u), reach = (most + 2) / 4;   // ceil((most - 1) / 4) blocks to either side
    if (t < n4) {
      const uint4 own = a4[t], pay = b4[t];
      uint32_t *kq = k + 4 * q, *pq = pos + 4 * q;
      kq[0] = own.x; kq[1] = own.y; kq[2] = own.z; kq[3] = own.w;
      v[4 * q] = pay.x; v[4 * q + 1] = pay.y; v[4 * q + 2] = pay.z; v[4 * q + 3] = pay.w;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        pq[x] = 4 * t + x;
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          if (y > x) pq[x] += kq[y] < kq[x];
          if (y < x) pq[x] -= kq[y] > kq[x];
        }
      }
      for (uint32_t d = 1; d <= reach; ++d) {
        if (t >= d) {
          const uint4 o = a4[t - d];
#pragma unroll
          for (int x = 0; x < 4; ++x) pq[x] -= (uint32_t)(o.x > kq[x]) + (o.y > kq[x]) + (o.z > kq[x]) + (o.w > kq[x]);
        }
        if (t + d < n4) {
          const uint4 o = a4[t + d];
#pragma unroll
          for (int x = 0; x < 4; ++x) pq[x] += (uint32_t)(o.x < kq[x]) + (o.y < kq[x]) + (o.z < kq[x]) + (o.w < kq[x]);
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < IPT / 4; ++q) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (4 * (q * T + threadIdx.x) + x < m) {
        s.a[pos[4 * q + x]] = k[4 * q + x];
        s.b()[pos[4 * q + x]] = v[4 * q + x];
      }
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------------ children: splitters from a sample, second pass
constexpr int SM_T = 512, SM_IPT = 8, SM_MOST = SM_T * SM_IPT;   // sampled keys of a parent
constexpr int BX_T = 512, BX_IPT = 8, BX_TILE = BX_T * BX_IPT;

// One workgroup per parent: its place among the parents, its children and tiles, their splitters.  A child of
// twice the average is more than the finish holds: with s sampled keys per child its odds are those of a Poisson number of mean
// 2 s below s, 1e-10 for 64 keys, which parents of up to 64 children have, 8e-8 for the 44 of 93 children (the fullest parents
// of a power-law list of 40 M entries), 4e-6 for the 32 of 128.  The call is then run again with the digit passes, as it is when a parent is
// too large for BK_MAXK children.
// COO: the whole list is one parent, its keys are built from the coordinates.  PER: parents for a thread to add up, SM_T * PER
// in all.
template <bool COO, int PER>
__global__ __launch_bounds__(SM_T) void bucket_sample_kernel(BkArgs a) {
  __shared__ BinScratch<SM_T, SM_IPT, 33> s;
  __shared__ uint32_t s_wave[3][SM_T / 64];
  __shared__ BkParent s_me;
  const int tid = threadIdx.x;
  const uint32_t p = blockIdx.x;
  const uint32_t np = COO ? 1u : a.totals[2];   // (written by an earlier kernel of the call whatever happens)
  if (COO && a.clear_flags) {   // the first kernel of the call, in one workgroup: the flags start here, not in a launch of their own
    if (tid < (int)(sizeof(Flags) / 4)) reinterpret_cast<uint32_t *>(a.flags)[tid] = 0;   // (the scans' barriers lie before any flag)
  } else if (gave_up(a, true)) return;
  if (p >= np) return;
  const uint2 origin = np != a.share.count ? a.origin[p] : make_uint2(p, 0u);
  {
    // children and parents of a single child, summed up together: below 2^18 and 2^14 of them
    constexpr uint32_t ALONE = 1u << 18;
    uint32_t size[PER], k[PER], tiles[PER], ssum = 0, ksum = 0, tsum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t x = tid * PER + q;
      size[q] = x >= np && x >= a.share.count ? 0u : COO ? a.n : a.ptotal[x];
      k[q] = x < np ? max((size[q] + BK_TARGET - 1) / BK_TARGET, 1u) : 0u;
      tiles[q] = (COO || k[q] > 1) ? (size[q] + BX_TILE - 1) / BX_TILE : 0u;
      const bool alone = !COO && k[q] == 1;
      ssum += size[q]; ksum += k[q] + (alone ? ALONE : 0u); tsum += tiles[q];
    }
    uint32_t s0 = scan_one_barrier<SM_T>(ssum, s_wave[0]), k0 = scan_one_barrier<SM_T>(ksum, s_wave[1]),
             t0 = scan_one_barrier<SM_T>(tsum, s_wave[2]);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t child0 = k0 % ALONE;
      if ((uint32_t)(tid * PER + q) == p) s_me = BkParent{s0, size[q], child0, k[q], t0, child0 - k0 / ALONE};
      s0 += size[q]; k0 += k[q] + (!COO && k[q] == 1 ? ALONE : 0u); t0 += tiles[q];
    }
    if (p == 0 && tid == SM_T - 1) { a.totals[0] = k0 % ALONE; a.totals[1] = t0; }
  }
  __syncthreads();
  const BkParent me = s_me;
  const bool shared = COO || me.k > 1;
  if (tid == 0) a.parent[p] = me;
  // (the sums are bounded by what the host allocated for; the guards keep it so whatever the sizes say)
  if (me.k > (uint32_t)BK_MAXK || me.child0 + me.k > a.max_children || (shared && me.region0 + me.k > a.max_regions)) {
    if (tid == 0) a.flags->retry = RETRY_SORT_LDS;
    return;
  }
  auto child = [&](uint32_t c, uint32_t low) {
    const uint32_t kind = origin.x | (shared ? BK_SHARED : 0u) | me.region0 << BK_REGION_SHIFT;
    a.child[me.child0 + c] = make_uint4(me.start, me.child0, kind, low);
    a.cursor[me.child0 + c] = shared ? 0u : me.size;
  };
  if (tid == 0) child(0, origin.y);
  if (me.k == 1) return;
  const uint32_t ntiles = (me.size + BX_TILE - 1) / BX_TILE;
  for (uint32_t t = tid; t < ntiles && me.tile0 + t < a.max_tiles; t += SM_T) a.tile_parent[me.tile0 + t] = p;
  // keys from evenly spaced pieces of the parent, at a scattered place in each (lists often come in a regular order)
  const uint32_t ns = min(min((uint32_t)SM_MOST, me.k * BK_OVERSAMPLE), me.size), piece = me.size / ns;
  uint32_t key[SM_IPT], pos[SM_IPT];
#pragma unroll
  for (int j = 0; j < SM_IPT; ++j) {
    const uint32_t i = j * SM_T + tid;
    key[j] = 0;
    if (i < ns) {
      const uint32_t at = me.start + (uint32_t)((uint64_t)i * me.size / ns) + ((i * 0x9E3779B1u + p * 0x85EBCA6Bu) >> 8) % piece;
      if (COO) share_of_entry(a, (uint32_t)a.row[at], (uint32_t)a.col[at], &key[j]);
      else key[j] = a.rec1[at].x;
    }
  }
  __shared__ uint32_t s_sample[64];
#pragma unroll
  for (int j = 0; j < SM_IPT; ++j) {
    const uint32_t i = j * SM_T + tid, x = (i * 64 + ns - 1) / ns;   // item x * ns / 64 for some x < 64?
    if (i < ns && x < 64 && x * ns / 64 == i) s_sample[x] = key[j];
  }
  __syncthreads();
  const uint32_t most = bin_slots<SM_T, SM_IPT, 33>(key, ns, origin.y, (uint32_t)(a.share.width - 1), s_sample[lane_id()], s, pos);
  if (most > BP_MOST) {
    if (tid == 0) a.flags->retry = RETRY_SORT_LDS;
    return;
  }
#pragma unroll
  for (int j = 0; j < SM_IPT; ++j)
    if (j * SM_T + tid < ns) { s.a[pos[j]] = key[j]; s.b()[pos[j]] = 0; }
  fix_order<SM_T, SM_IPT, 33>(ns, s);
  for (uint32_t c = tid; c < me.k; c += SM_T)
    if (c > 0) child(c, s.a[c * ns / me.k]);
}

// 16.8 M entries 59 us, 40 M 135: 4.5 and 4.7 TB/s, near the rate of a copy (runs of some 200 entries).
// A tile of a parent with more than one child: every entry finds its child among the splitters, the tile is put in
// order of the children in LDS, every child's run goes behind what it already holds (one device atomic per tile and
// child: a parent's tiles are few).
template <bool COO>
__global__ __launch_bounds__(BX_T) void bucket_split_kernel(BkArgs a) {
  __shared__ uint2 s_rec[BX_TILE];
  __shared__ uint8_t s_bin[BX_TILE];
  __shared__ uint32_t s_split[BK_MAXK], s_cnt[BK_MAXK], s_goff[BK_MAXK];
  __shared__ uint32_t s_wave[BX_T / 64];
  const uint32_t t = xcd_chunk_item(blockIdx.x, a.tile_chunk);
  if (gave_up(a, !COO)) return;   // (COO: this kernel is the one that finds coordinates out of range)
  if (t >= min(a.totals[1], a.max_tiles)) return;
  const BkParent me = a.parent[COO ? 0u : a.tile_parent[t]];
  const int tid = threadIdx.x;
  if (me.k > (uint32_t)BK_MAXK) return;
  const uint32_t first = me.start + (t - me.tile0) * BX_TILE, in_tile = min((uint32_t)BX_TILE, me.start + me.size - first);
  if (tid < BK_MAXK) {
    s_split[tid] = (uint32_t)tid < me.k ? a.child[me.child0 + tid].w : 0xFFFFFFFFu;
    s_cnt[tid] = 0;
  }
  uint32_t key[BX_IPT], val[BX_IPT], bin[BX_IPT], arr[BX_IPT];
  bool bad = false;
#pragma unroll
  for (int j = 0; j < BX_IPT; ++j) {
    const uint32_t i = j * BX_T + tid;
    key[j] = 0; val[j] = 0;
    if (i < in_tile) {
      if (COO) {
        const uint32_t r = (uint32_t)a.row[first + i], c = (uint32_t)a.col[first + i];
        bad |= coo_out_of_range(a.ks, r, c);
        share_of_entry(a, r, c, &key[j]);
        val[j] = a.val[first + i];
      } else {
        const uint2 r = a.rec1[first + i];
        key[j] = r.x; val[j] = r.y;
      }
    }
  }
  if (COO && bad) a.flags->index_range = 1;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < BX_IPT; ++j) bin[j] = 0;
  for (uint32_t step = 1u << (31 - __clz((int)me.k)); step; step >>= 1) {   // last child whose splitter is not above the key
#pragma unroll
    for (int j = 0; j < BX_IPT; ++j) {
      const uint32_t at = bin[j] + step;
      if (at < me.k && s_split[at] <= key[j]) bin[j] = at;
    }
  }
#pragma unroll
  for (int j = 0; j < BX_IPT; ++j) arr[j] = j * BX_T + tid < in_tile ? atomicAdd(&s_cnt[bin[j]], 1u) : 0u;
  __syncthreads();
  const uint32_t c = tid < BK_MAXK ? s_cnt[tid] : 0u;
  const uint32_t start = scan_one_barrier<BX_T>(c, s_wave);
  if (tid < BK_MAXK) {
    uint32_t at = 0;
    if (c) {
      at = atomicAdd(&a.cursor[me.child0 + tid], c);
      if (at + c > (uint32_t)BK_CAP) a.flags->retry = RETRY_SORT_LDS;
    }
    s_cnt[tid] = start;
    s_goff[tid] = at - start;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < BX_IPT; ++j) {
    if (j * BX_T + tid < in_tile) {
      const uint32_t pos = s_cnt[bin[j]] + arr[j];
      s_rec[pos] = make_uint2(key[j], val[j]);
      s_bin[pos] = (uint8_t)bin[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < BX_IPT; ++j) {
    const uint32_t i = j * BX_T + tid;
    if (i < in_tile) {
      const uint32_t child = s_bin[i], at = s_goff[child] + i;
      if (at < (uint32_t)BK_CAP) a.rec2[(size_t)(me.region0 + child) * BK_CAP + at] = s_rec[i];
    }
  }
}

// ------------------------------------------------------------------ finish: a child per workgroup
// 16.8 M entries of the power-law matrix 147 us, 40 M with local columns 367 (65 and 152 when it only reads and writes), in
// six workgroups per CU (71 registers; 8 at 64 with spills: 149 and 369).  A workgroup takes some 12 us, mostly a chain of
// dependent steps, so what counts is how many are resident: counters and values share their place in LDS, bins that
// crowd are not cut again; children of 2048 entries on average with twice the LDS: 297 and 810, of 1024 with room for 2560
// or 3072: 237 and 621, 282 and 750; as many workgroups as are resident, walking the children with the next one's entries on
// their way, some 40 and 110 us longer (the loop's state takes the registers that the steps need).  (Bins by row or range, cut again by smallest and largest key until none
// holds more than 9: 177 and 602, three quarters of it LDS atomics and reads that meet in a bank; four digit passes of
// ballot ranking would take 280 vector instructions an entry, this takes 200.)
constexpr int BF_T = 256, BF_IPT = BK_CAP / BF_T;
static_assert(BF_T % 64 == 0 && BF_T * BF_IPT == BK_CAP && BK_MAXK <= BF_T, "a workgroup holds a child and sees its siblings");

__global__ __launch_bounds__(BF_T, 6) void bucket_finish_kernel(BkArgs a) {
  __shared__ BinScratch<BF_T, BF_IPT, 0> s;
  __shared__ uint32_t s_before;
  const int tid = threadIdx.x;
  const uint32_t c = xcd_chunk_item(blockIdx.x, a.child_chunk), at = min(c, a.max_children - 1);
  // everything that does not hang on something else first; what an earlier kernel has left unwritten is not used
  const uint4 me = a.child[at], after = a.child[min(at + 1, a.max_children - 1)];
  const uint32_t m = a.cursor[at], nchildren = min(a.totals[0], a.max_children);
  if (tid == 0) s_before = 0;
  if (gave_up(a, true) || c >= nchildren) return;
  const uint32_t start = me.x, child0 = me.y, share = me.z & (BK_MAXSHARES - 1), j0 = c - child0;
  if (m > (uint32_t)BK_CAP) return;   // (the call will be run again)
  if ((uint32_t)tid < j0) atomicAdd(&s_before, a.cursor[child0 + tid]);   // j0 < BK_MAXK <= BF_T
  const uint2 *src = me.z & BK_SHARED ? a.rec2 + (size_t)((me.z >> BK_REGION_SHIFT) + j0) * BK_CAP : a.rec1 + start;
  const bool last = c + 1 == nchildren || (after.z & (BK_MAXSHARES - 1)) != share;   // of the share
  const Key behind = last ? a.share.width : after.w;
  const uint32_t lo = me.w, hi = (uint32_t)min(behind, (Key)0xFFFFFFFFu);   // (hi itself may be the next child's)
  uint32_t key[BF_IPT], val[BF_IPT], pos[BF_IPT];
#pragma unroll
  for (int j = 0; j < BF_IPT; ++j) {
    key[j] = 0; val[j] = 0;
    if (j * BF_T + tid < m) {
      const uint2 r = src[j * BF_T + tid];
      key[j] = r.x; val[j] = r.y;
    }
  }
  const uint32_t sample = tid < 64 && m >= 64 ? src[(uint32_t)tid * m / 64].x : 0u;
  const uint32_t most = bin_slots<BF_T, BF_IPT, 0>(key, m, lo, hi, sample, s, pos);
#pragma unroll
  for (int j = 0; j < BF_IPT; ++j)
    if (j * BF_T + tid < m) { s.a[pos[j]] = key[j]; s.b()[pos[j]] = val[j]; }
  if (most <= BP_MOST) {
    fix_order<BF_T, BF_IPT, 0>(m, s);
  } else {   // keys that crowd in more than a few places of their range
    __syncthreads();
    for (uint32_t size = 2; size < 2 * m; size <<= 1) {   // bitonic, all comparisons ascending; items past m are not there
      for (uint32_t half = size >> 1; half > 0; half >>= 1) {
        const uint32_t flip = half == size >> 1 ? size - 1 : half;
        for (uint32_t t = tid; t < 1u << (31 - __clz(BK_CAP - 1)); t += BF_T) {   // half of the next power of two
          const uint32_t i = (t & (half - 1)) + ((t & ~(half - 1)) << 1), k = i ^ flip;
          if (k < m && s.a[i] > s.a[k]) {
            const uint32_t x = s.a[i], y = s.b()[i];
            s.a[i] = s.a[k]; s.a[k] = x; s.b()[i] = s.b()[k]; s.b()[k] = y;
          }
        }
        __syncthreads();
      }
    }
  }
  const uint32_t out = start + s_before;
  const Key base = share * a.share.width;
  const Key bmask = ((Key)1 << a.ks.b_bits) - 1;
  bool dup = false;
  for (uint32_t i = tid; i < m; i += BF_T) {
    const Key full = base + s.a[i];
    dup |= i > 0 && s.a[i - 1] == s.a[i];
    if (out + i < a.n) {
      if (a.major_out) a.major_out[out + i] = (int32_t)(full >> a.ks.b_bits);
      a.minor_out[out + i] = (int32_t)(full & bmask);
      a.val_out[out + i] = s.b()[i];
    }
  }
  if (dup) a.flags->duplicate = 1;
  if (a.ptr) {   // the major indices whose first possible key lies in this child's range: entries below that key
    Key g0 = (base + lo + bmask) >> a.ks.b_bits, g1 = (base + behind + bmask) >> a.ks.b_bits;
    if (c + 1 == nchildren) g1 = (Key)a.ngroups_out + 1;
    if (g1 > (Key)a.ngroups_out + 1) g1 = (Key)a.ngroups_out + 1;
    for (Key g = g0 + tid; g < g1; g += BF_T) {
      const Key first = (g << a.ks.b_bits) - base;   // may lie beyond 32 bits (behind the last key): all entries are below
      uint32_t b = 0, e = m;
      while (b < e) {
        const uint32_t mid = (b + e) >> 1;
        if ((Key)s.a[mid] < first) b = mid + 1; else e = mid;
      }
      a.ptr[g] = (int32_t)(out + b);
    }
  }
}

// ------------------------------------------------------------------ host
// first pass, threads and entries per thread, and workgroups: as many as are resident at once
constexpr int BP_T = 512, BP_IPT = 8, BP_GROUPS = 768, BPL_T = 1024, BPL_IPT = 12, BPL_GROUPS = 256;
constexpr int64_t BK_LARGE = 1 << 23;
// most keys of the sample and parents beside the shares: what leaves the LDS of the first pass its workgroups per CU (3 / 1)
constexpr int BP_SAMPLES = 4096, BP_MAXX = 192, BPL_SAMPLES = 16384, BPL_MAXX = 1024;
static_assert(BK_MAXSHARES + BPL_MAXX <= 4 * SM_T && BP_MAXX <= BPL_MAXX, "a workgroup of the sample sees all parents");

struct BucketPlan {
  bool direct;     // one parent: the caller's list
  KeyShares share;
  bool large;      // the first pass takes large tiles
  uint32_t nsamples, crowded_at, heavy_at, unit, max_parents, per_group, ngroups, max_children, max_regions, max_tiles;
};

static int chunk_shift(uint32_t items) { return std::min(std::max(bits_for(items / 64) - 1, 0), 6); }
static uint32_t chunk_grid(uint32_t items, int shift) { return ceil_div(items, 8u << shift) * (8u << shift); }

// at most `most` shares, or what keeps them at 2^32 keys (BK_MAXSHARES where the key has BK_MAXBITS + 32 bits)
static KeyShares key_shares(const KeySpec &ks, uint32_t most) {
  KeyShares s{};
  if (ks.a_extent >= most && ks.b_bits <= 32) {
    s.rows = std::min(ceil_div(ks.a_extent, most), (uint32_t)std::min<uint64_t>((1ull << 32) >> ks.b_bits, 1u << 31));
    s.count = ceil_div(ks.a_extent, s.rows);
    s.width = (uint64_t)s.rows << ks.b_bits;
    s.mul_shift = bits_for(s.rows - 1);
    s.mul = (uint32_t)((1ull << (31 + s.mul_shift)) / s.rows + 1);
  } else {
    const uint64_t span = (uint64_t)ks.a_extent << ks.b_bits;
    while (s.shift < 32 && ((span - 1) >> s.shift) + 1 > most) ++s.shift;
    s.count = (uint32_t)((span - 1) >> s.shift) + 1;
    s.width = 1ull << s.shift;
  }
  return s;
}

static BucketPlan bucket_plan(int64_t nnz, const KeySpec &ks) {
  BucketPlan b{};
  b.direct = ks.total_bits <= 32 && nnz <= BK_MAXK / 2 * BK_TARGET;
  if (b.direct) {
    b.share.count = 1; b.share.shift = ks.total_bits; b.share.width = 1ull << ks.total_bits;
  } else {
    // 32 children per parent; 6 where the first pass writes whole lines all the same and the sample's sort is a chain of steps
    // that its size makes longer (1 M entries: 24 -> 17 us in the sample, the other kernels as they were)
    const int64_t want = ceil_div<int64_t>(nnz, (nnz < (1 << 22) ? 6 : 32) * BK_TARGET);
    b.share = key_shares(ks, (uint32_t)std::min<int64_t>(want, BK_MAXSHARES));
    b.large = nnz >= BK_LARGE;
    const uint32_t tile = b.large ? BPL_T * BPL_IPT : BP_T * BP_IPT, groups = b.large ? BPL_GROUPS : BP_GROUPS;
    const uint32_t tiles = (uint32_t)ceil_div<int64_t>(nnz, tile), each = ceil_div(tiles, groups);
    b.per_group = each * tile;
    b.ngroups = ceil_div(tiles, each);
    if (nnz > BK_MAXK * BK_TARGET) {
      b.nsamples = (uint32_t)std::min<int64_t>(nnz / 2048, b.large ? BPL_SAMPLES : BP_SAMPLES);
      auto keys_of = [&](int64_t entries) { return (uint32_t)ceil_div<int64_t>(entries * b.nsamples, nnz); };
      // (three quarters are enough to be cut, but it takes a share that is too large: a first pass with cut shares takes longer)
      b.crowded_at = keys_of(BK_MAXK * BK_TARGET);
      b.heavy_at = keys_of(BK_MAXK * BK_TARGET * 3 / 4);
      b.unit = std::max({8u, keys_of(40 * BK_TARGET), ceil_div<uint32_t>(b.nsamples, b.large ? BPL_MAXX : BP_MAXX)});
    }
  }
  // (the cut shares' parents beside the first: (keys - 1) / unit each)
  b.max_parents = b.share.count + (b.nsamples ? b.nsamples / b.unit : 0);
  const uint32_t full = (uint32_t)(nnz / BK_TARGET), shared = std::min(b.max_parents, full);   // parents of more than one child, at most
  b.max_children = full + b.max_parents + 1;
  b.max_regions = b.direct ? full + 1 : full + shared;
  b.max_tiles = (uint32_t)(nnz / BX_TILE) + shared + 1;
  return b;
}

// (row, col) tuples whose share of the key's range fits 32 bits, in numbers that leave parents room for uneven sizes:
// a parent of twice the average has children enough up to 67 M entries.
bool bucket_sort_takes(int64_t nnz, const KeySpec &ks) {
  return nnz >= 1 && ks.mode == 0 && ks.total_bits >= 1 && ks.total_bits - BK_MAXBITS <= 32 &&
         (nnz >> (ks.total_bits < BK_MAXBITS ? ks.total_bits : BK_MAXBITS)) <= BK_MAXK / 2 * BK_TARGET;
}

size_t bucket_sort_temp_bytes(int64_t nnz, const KeySpec &ks) {
  const BucketPlan b = bucket_plan(nnz, ks);
  auto g = [](size_t bytes) { return Env::granule(bytes); };
  return (b.direct ? 0 : g(4ull * b.ngroups * b.max_parents) + g(4ull * b.max_parents) + g(8ull * nnz)) +
         (b.nsamples ? g(2ull * (b.nsamples + 7)) + g(4ull * b.nsamples) + g(2ull * (b.share.count + 1)) + g(4ull * (b.max_parents - b.share.count)) + g(8ull * b.max_parents) : 0) +
         g(sizeof(BkParent) * b.max_parents) + g(12) + g(16ull * b.max_children) + g(4ull * b.max_children) + g(4ull * b.max_tiles) + g(8ull * BK_CAP * b.max_regions);
}

void bucket_sort(Env &env, const int32_t *row, const int32_t *col, const float *val, int64_t nnz, const KeySpec &ks,
                 SortOut &out, Flags *flags) {
  const BucketPlan b = bucket_plan(nnz, ks);
  BkArgs a{};
  a.row = row; a.col = col; a.val = (const uint32_t *)val;
  a.n = (uint32_t)nnz; a.ks = ks; a.flags = flags;
  a.share = b.share;
  a.nsamples = b.nsamples; a.crowded_at = b.crowded_at; a.heavy_at = b.heavy_at; a.unit = b.unit; a.max_parents = b.max_parents;
  a.per_group = b.per_group; a.ngroups = b.ngroups;
  a.groups_per_xcd = ceil_div<uint32_t>(b.ngroups, 8u);
  a.coo_vec = ((reinterpret_cast<uintptr_t>(row) | reinterpret_cast<uintptr_t>(col) | reinterpret_cast<uintptr_t>(val)) & 15u) == 0;
  a.max_children = b.max_children; a.max_regions = b.max_regions; a.max_tiles = b.max_tiles;
  a.tile_chunk = chunk_shift(b.max_tiles); a.child_chunk = chunk_shift(b.max_children);
  env.reserve(bucket_sort_temp_bytes(nnz, ks));
  if (!b.direct) {
    a.hist = env.temp<uint32_t>((size_t)b.ngroups * b.max_parents);
    a.ptotal = env.temp<uint32_t>(b.max_parents);
    a.rec1 = env.temp<uint2>(nnz);
  }
  if (b.nsamples) {
    a.sample_share = env.temp<uint16_t>(b.nsamples + 7);
    a.sample_low = env.temp<uint32_t>(b.nsamples);
    a.first = env.temp<uint16_t>(b.share.count + 1);
    a.split = env.temp<uint32_t>(b.max_parents - b.share.count);
    a.origin = env.temp<uint2>(b.max_parents);
  }
  a.parent = env.temp<BkParent>(b.max_parents);
  a.totals = env.temp<uint32_t>(3);
  a.child = env.temp<uint4>(b.max_children);
  a.cursor = env.temp<uint32_t>(b.max_children);
  a.tile_parent = env.temp<uint32_t>(b.max_tiles);
  a.rec2 = env.temp<uint2>((size_t)b.max_regions * BK_CAP);
  if (!env.ok()) return;
  a.clear_flags = (b.nsamples || b.direct) && out.clear_flags;   // by the first kernel
  if (out.clear_flags && !a.clear_flags) fill_u32(env, (uint32_t *)flags, sizeof(Flags) / 4, 0u);
  if (!b.direct) {
    if (b.nsamples) US_LAUNCH(env, "bucket_probe", 8.0 * b.nsamples, bucket_probe_kernel, ceil_div<uint32_t>(b.nsamples, BL_T), BL_T, a);
    const double hist_bytes = (a.share.rows ? 4.0 : 8.0) * nnz;
    if (b.large) US_LAUNCH(env, "bucket_hist", hist_bytes, (bucket_hist_kernel<BPL_T, BPL_SAMPLES, BPL_MAXX>), a.groups_per_xcd * 8, BPL_T, a);
    else US_LAUNCH(env, "bucket_hist", hist_bytes, (bucket_hist_kernel<BP_T, BP_SAMPLES, BP_MAXX>), a.groups_per_xcd * 8, BP_T, a);
    US_LAUNCH(env, "bucket_scan", 8.0 * b.ngroups * b.share.count, bucket_scan_kernel, ceil_div<uint32_t>(b.max_parents, BS_BINS), BS_T, a);
    if (b.large) US_LAUNCH(env, "bucket_scatter", 20.0 * nnz, (bucket_scatter_kernel<BPL_T, BPL_IPT, BPL_MAXX>), a.groups_per_xcd * 8, BPL_T, a);
    else US_LAUNCH(env, "bucket_scatter", 20.0 * nnz, (bucket_scatter_kernel<BP_T, BP_IPT, BP_MAXX>), a.groups_per_xcd * 8, BP_T, a);
    if (b.max_parents <= SM_T) US_LAUNCH(env, "bucket_sample", 0.0, (bucket_sample_kernel<false, 1>), b.max_parents, SM_T, a);
    else if (b.max_parents <= 2 * SM_T) US_LAUNCH(env, "bucket_sample", 0.0, (bucket_sample_kernel<false, 2>), b.max_parents, SM_T, a);
    else US_LAUNCH(env, "bucket_sample", 0.0, (bucket_sample_kernel<false, 4>), b.max_parents, SM_T, a);
    US_LAUNCH(env, "bucket_split", 16.0 * nnz, (bucket_split_kernel<false>), chunk_grid(b.max_tiles, a.tile_chunk), BX_T, a);
  } else {
    US_LAUNCH(env, "bucket_sample", 0.0, (bucket_sample_kernel<true, 1>), 1, SM_T, a);
    US_LAUNCH(env, "bucket_split", 20.0 * nnz, (bucket_split_kernel<true>), chunk_grid(b.max_tiles, a.tile_chunk), BX_T, a);
  }
  if (out.late) {
    out.late(out); out.late = nullptr;
    if (!env.ok()) return;
  }
  a.major_out = out.major; a.minor_out = out.minor; a.val_out = (uint32_t *)out.val;
  a.ptr = out.ptr; a.ngroups_out = ks.a_extent;
  US_LAUNCH(env, "bucket_finish", (out.major ? 20.0 : 16.0) * nnz, bucket_finish_kernel, chunk_grid(b.max_children, a.child_chunk), BF_T, a);
}

}  // namespace us
