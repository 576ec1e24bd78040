// Y (+)= A X, a panel of columns of X at a time: over entries grouped by row (row-major COO, CSR, DCSR, CISR-plus) in equal shares
// of the entries, and over the rows of an ELL slab.
#include "common.h"
#include "device.h"
#include "spmm_internal.h"

#include <algorithm>
#include <type_traits>

namespace us {

// VEC columns in registers, and in memory, where rows may begin at any float
template <int VEC> struct PanelVec {
  typedef float reg __attribute__((ext_vector_type(VEC)));
  typedef float mem __attribute__((ext_vector_type(VEC), aligned(4)));
};
template <> struct PanelVec<1> { typedef float reg; typedef float mem; };

// lane K of every 16 lanes to all of them (all lanes must be active: a lane that is not reads as 0)
template <int K>
__device__ __forceinline__ int bcast16(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xf, 0xf, true); }
template <int K>
__device__ __forceinline__ float bcast16(float v) { return __builtin_bit_cast(float, bcast16<K>(__builtin_bit_cast(int, v))); }

template <int K, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (K < N) { f(std::integral_constant<int, K>{}); static_for<K + 1, N>(static_cast<F &&>(f)); }
}

constexpr uint64_t FIRST16 = 0x0001000100010001ull;   // the first lane of every 16
__device__ __forceinline__ uint64_t spread16(uint64_t firsts) { return (firsts << 16) - firsts; }   // ... to all 16

// largest value so far across the wavefront (all lanes active)
__device__ __forceinline__ uint32_t wave_inclusive_max_dpp(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, true));
  return v;
}

// Parents between the ends of a tile up to which all of them are walked, 512 at a time (0.85 us); beyond, every entry looks for its
// own, at some 3 us whatever lies between.  us, walk / search, N = 1: 20,000 entries of 200,000 / 400,000 / 1 M rows (5,120 / 10,240 /
// 25,600 parents a tile) 13.3 / 12.2, 17.9 / 12.9, 29.8 / 12.3; 150,000 of 1 M / 400,000 (3,413 / 1,365) 17.2 / 16.8, 15.1 / 15.7;
// 500 of 10 M 8,470 / 14.4.
constexpr int32_t PS_FAR = 4096;
constexpr int PS_WAVES = 8, PS_T = 64 * PS_WAVES, PS_GROUPS = 4 * PS_WAVES, PS_TILE = PS_T;
static_assert(PS_GROUPS < 64, "bit masks over the groups of a workgroup");

// Sixteen lanes ("a group") take sixteen consecutive entries, one after the other, a lane VEC * H columns of a panel: H parts of
// 16 * VEC columns.  FULL: the panel has all its columns.  WIDE: X or Y has 4 GB or more.  U: rows of X in flight.
template <int VEC, int H, bool FULL, bool WIDE, int U>
struct PanelWalk {
  typedef typename PanelVec<VEC>::reg V;
  typedef typename PanelVec<VEC>::mem M;
  static constexpr int PART = 16 * VEC, PW = PART * H;
  // first column of the lane in every part of the panel.  Not FULL: where the panel's columns end inside the vector the lane takes
  // the last VEC of them: what it shares with the lane before it both compute, and store, alike.  No two panels share a column (they
  // would both add to it): where fewer than VEC are left for the last panel, the one before it leaves it VEC (N >= VEC)
  uint32_t c0[H];
  uint64_t cols_ok[H];              // lanes with a column
  V x[16][H], acc[H];

  __device__ __forceinline__ void columns(uint32_t panel, uint32_t N, int s) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      c0[h] = panel * PW + h * PART + s * VEC;
      cols_ok[h] = ~0ull;
      if constexpr (!FULL) {
        uint32_t begin = panel * PW, end = min(begin + PW, N);
        if (end < N && N - end < VEC) end = N - VEC;
        begin = min(begin, N - VEC);
        c0[h] = begin + h * PART + s * VEC;
        const bool ok = c0[h] < end;
        cols_ok[h] = __ballot(ok);
        c0[h] = ok ? min(c0[h], end - VEC) : begin;   // (the others load as well: from a line that is loaded anyway)
      }
    }
  }
  // part h of the lane's columns in the row that begins `o` bytes into X or Y
  template <typename T, typename O>
  __device__ __forceinline__ T *at(T *base, O o, int h) const {
    if constexpr (FULL) return base + (o + c0[0] * 4u) + h * (PART * 4);
    else return base + (o + c0[h] * 4u);
  }
  // bytes from a row's number to where it begins, and from the lane of entry K to all of its group (all lanes take part)
  struct Offset { int lo, hi; };
  static __device__ __forceinline__ Offset offset(int32_t row, int64_t ld) {
    const uint64_t o = (uint64_t)(uint32_t)row * (uint64_t)ld * 4u;
    return {(int)(uint32_t)o, (int)(uint32_t)(o >> 32)};
  }
  template <int K>
  static __device__ __forceinline__ auto of(const Offset &o) {
    if constexpr (WIDE) return (uint64_t)(uint32_t)bcast16<K>(o.hi) << 32 | (uint32_t)bcast16<K>(o.lo);
    else return (uint32_t)bcast16<K>(o.lo);
  }
  template <int K>
  __device__ __forceinline__ void gather(const char *X, const Offset &xo) {
    const auto o = of<K>(xo);
#pragma unroll
    for (int h = 0; h < H; ++h) x[K][h] = *reinterpret_cast<const M *>(at(X, o, h));
  }
  __device__ __forceinline__ void first_gathers(const char *X, const Offset &xo) {
    static_for<0, U>([&](auto kc) { gather<decltype(kc)::value>(X, xo); });
  }
  // the sums of the lanes in to[] to (add: onto) the rows of Y that begin at byte y; all is read before anything is written
  template <typename O>
  __device__ __forceinline__ void put(char *Y, O y, const uint64_t (&to)[H], bool add) const {
    V out[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      out[h] = acc[h];
      if (add) {
        if (__builtin_amdgcn_inverse_ballot_w64(to[h])) { const V old = *reinterpret_cast<const M *>(at(Y, y, h)); out[h] = old + acc[h]; }
      }
    }
#pragma unroll
    for (int h = 0; h < H; ++h)
      if (__builtin_amdgcn_inverse_ballot_w64(to[h])) *reinterpret_cast<M *>(at(Y, y, h)) = out[h];
  }
  // All entries of the group: sm = lanes whose entry is the first of its row, dead = lanes without an entry.  Sums of rows that
  // begin and end among them go to Y; the part of a row that began before them to s_head[group]; what begins and is still open
  // at their end stays in acc.
  __device__ __forceinline__ void walk(const char *X, const Offset &xo, float v, uint64_t sm, uint64_t dead, char *Y, const Offset &yo,
                                       bool add, V (*s_head)[16], int s) {
    uint64_t seen = spread16(sm & FIRST16);   // lanes whose run began among their own entries
#pragma unroll
    for (int h = 0; h < H; ++h) acc[h] = V(0.f);
    static_for<0, 16>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      if constexpr (k > 0) {
        const uint64_t m = (sm >> k) & FIRST16;
        if (m) {   // (scalar, like all masks here) some of the four runs end in front of entry k
          const uint64_t lanes = spread16(m), head = lanes & ~seen, full = lanes & seen & ~spread16((dead >> (k - 1)) & FIRST16);
          if (head) {
            if (__builtin_amdgcn_inverse_ballot_w64(head)) {
#pragma unroll
              for (int h = 0; h < H; ++h) s_head[h][s] = acc[h];
            }
          }
          if (full) {
            const auto y = of<k - 1>(yo);
            uint64_t to[H];
#pragma unroll
            for (int h = 0; h < H; ++h) to[h] = full & cols_ok[h];
            put(Y, y, to, add);
          }
          if (__builtin_amdgcn_inverse_ballot_w64(lanes)) {
#pragma unroll
            for (int h = 0; h < H; ++h) acc[h] = V(0.f);
          }
          seen |= lanes;
        }
      }
      const float t = bcast16<k>(v);
#pragma unroll
      for (int h = 0; h < H; ++h) acc[h] += t * x[k][h];
      if constexpr (k + U < 16) gather<k + U>(X, xo);
    });
    if (((uint32_t)(sm >> (lane_id() & 48)) & 0xffffu) == 0) {
#pragma unroll
      for (int h = 0; h < H; ++h) s_head[h][s] = acc[h];
    }
  }
};

// a + s_head[j0 .. end)[h][s], in this order
template <int H, typename V>
__device__ __forceinline__ V panel_heads(const V (*s_head)[H][16], int h, int s, int j0, int end, V a) {
  int j = j0;
  for (; j + 4 <= end; j += 4) {
    V t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = s_head[j + u][h][s];
#pragma unroll
    for (int u = 0; u < 4; ++u) a += t[u];
  }
  for (; j < end; ++j) a += s_head[j][h][s];
  return a;
}
// The groups of a workgroup as masks: `some` have a first entry of a row at all, `fresh` begin with one (bits from PS_GROUPS on
// set).  A run that is open in front of group j0 ends before the next group that is fresh, or inside the next that has a start.
struct PanelRuns {
  uint64_t some, fresh;
  __device__ __forceinline__ int next(int j0) const { return __builtin_ctzll(some >> j0) + j0; }
  __device__ __forceinline__ int end(int j0) const {
    const int k = next(j0);
    return k >= PS_GROUPS ? PS_GROUPS : k + !(fresh >> k & 1);
  }
};
__device__ __forceinline__ PanelRuns panel_runs(const uint32_t *s_starts) {
  const uint32_t st = lane_id() < PS_GROUPS ? s_starts[lane_id()] : 1u;
  return {__ballot(st != 0), __ballot((st & 1u) != 0)};
}

struct PanelJob {
  const int32_t *row;      // COO: row of every entry, else null
  const int32_t *ptr, *ids;// compressed rows: children of parent p are [ptr[p], ptr[p + 1]); row of a stored row, or null
  const int2 *bounds;      // compressed rows: parents of the entries around every tile boundary (tile_bounds_kernel), or null: the
  int64_t nparents;        // workgroup looks for its own among all parents
  const int32_t *col;
  const float *val;
  uint32_t n;              // entries
  const float *X; int64_t ldx;
  float *Y; int64_t ldy;
  uint32_t N;              // columns of this launch
  int32_t *carry_row;      // null: another launch of the product writes them
  float *carry; int64_t carry_ld;
};

// bounds[k] = parents of the last entry before tile k and of its first one, for all tiles side by side: a bisection over all
// parents is 20 dependent loads
__global__ __launch_bounds__(256) void tile_bounds_kernel(const int32_t *ptr, int64_t nparents, int64_t nnz, int64_t ntiles,
                                                          int2 *bounds) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k > ntiles) return;
  const int64_t e = min(k * PS_TILE, nnz);     // nnz > 0
  const int64_t behind = parent_of(ptr, nparents, e < nnz ? e : nnz - 1);
  int64_t before = behind;                     // the parent of e - 1: behind itself, or the last one before it with entries
  if (e > 0 && e < nnz && (int64_t)ptr[behind] == e) before = parent_of(ptr, behind, e - 1);
  bounds[k] = make_int2((int32_t)before, (int32_t)behind);
}

// The parent of an entry e is the number of parents p with ptr[p + 1] <= e.  Of two entries at once, by all threads of the
// workgroup: 512 places at a time, three trips to memory for 16 M parents where a bisection takes 24.
__device__ __forceinline__ int2 find_parents(const int32_t *ptr, uint32_t nparents, uint32_t e0, uint32_t e1, uint32_t *s_count) {
  const uint32_t e[2] = {e0, e1};
  uint32_t lo[2] = {0, 0}, hi[2] = {nparents - 1, nparents - 1};   // (an entry that no other parent holds is the last one's)
  while (lo[0] < hi[0] || lo[1] < hi[1]) {
    uint32_t step[2], p[2];
    int32_t end[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {   // both loads before either is looked at: at a place that there is, whether it counts or not
      step[q] = (hi[q] - lo[q] + PS_T - 1) / PS_T;
      p[q] = lo[q] + (threadIdx.x + 1) * step[q] - 1;
      end[q] = ptr[min(p[q], nparents - 1) + 1];
    }
    uint32_t c = 0;   // of the wavefront, of either entry in 16 bits
#pragma unroll
    for (int q = 0; q < 2; ++q) c |= (uint32_t)__popcll(__ballot(lo[q] < hi[q] && p[q] < hi[q] && (uint32_t)end[q] <= e[q])) << (16 * q);
    if (lane_id() == 0) s_count[wave_id()] = c;
    __syncthreads();
    c = 0;
#pragma unroll
    for (int w = 0; w < PS_WAVES; ++w) c += s_count[w];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (lo[q] < hi[q]) {
        lo[q] += (c >> (16 * q) & 0xFFFFu) * step[q];
        hi[q] = min(hi[q], lo[q] + step[q] - 1);
      }
    }
  }
  return make_int2((int32_t)lo[0], (int32_t)lo[1]);
}

// The same of every thread's entry, all of them held by parents from `before` to `last`: 512 pointers between the two through LDS,
// then, for every entry by itself, three at a time of those between its neighbours among the 512.
__device__ __forceinline__ uint32_t find_parent(const int32_t *ptr, int32_t before, int32_t last, uint32_t e, bool live, uint32_t *s_pivot) {
  const int32_t *end = ptr + before + 1;
  const uint32_t span = (uint32_t)(last - before), step = (span + PS_T - 1) / PS_T, mine = (threadIdx.x + 1) * step - 1;
  s_pivot[threadIdx.x] = mine < span ? (uint32_t)end[mine] : 0xFFFFFFFFu;   // (entries have 31 bits)
  __syncthreads();
  uint32_t c = 0;   // pivots at or below e
#pragma unroll
  for (int d = PS_T / 2; d >= 1; d >>= 1)
    if (s_pivot[c + d - 1] <= e) c += d;
  if (s_pivot[c] <= e) ++c;
  uint32_t lo = min(c * step, span), hi = live ? min(lo + step - 1, span) : lo;
  while (lo < hi) {
    const uint32_t q = (hi - lo + 3) / 4;
    uint32_t p[3], n = 0;
    int32_t v[3];
#pragma unroll
    for (uint32_t j = 0; j < 3; ++j) {   // (as above)
      p[j] = lo + (j + 1) * q - 1;
      v[j] = end[min(p[j], span - 1)];
    }
#pragma unroll
    for (uint32_t j = 0; j < 3; ++j) n += p[j] < hi && (uint32_t)v[j] <= e;
    lo += n * q;
    if (n < 3) hi = min(hi, lo + q - 1);
  }
  return (uint32_t)before + lo;
}

// A workgroup takes 512 consecutive entries and a panel of 16 * VEC * H columns, a wavefront 64 entries, sixteen lanes
// ("a group") sixteen of them one after the other, VEC * H columns a lane.  So a load of one instruction brings pieces of four
// rows of X, and column, value and row of an entry reach the lanes of their group as DPP operands (row_newbcast), not as LDS
// traffic or scalars.  Sixteen loads are in flight before the first multiply-add; the rows of a tile's entries are looked up
// behind them.
//
// What bounds it: the misses of the L2s.  They come over the fabric in 128-byte lines at 6.5 to 7.5 TB/s whether HBM or the
// memory-side cache answers, hits at 23 to 27 TB/s (measured with bare gathers of 64 to 1024 bytes from spans of 2 MB to 1 GB;
// pieces of 64 bytes cost as much as of 128).  So the columns go by panels, all entries for a panel, then for the next: in a
// panel of 64 columns a row of X takes two lines instead of its whole length, and the entries in flight on an XCD (which walks a
// contiguous range of tiles) find more rows with local columns again.  By counters: 25.6 M entries of long rows, N = 128, two panels
// of 64: 27 % of 113 M requests hit, 10.6 GB fetched and stored at 7.1 TB/s; 5.2 M, N = 1000, rows off whole lines,
// three panels of 256 and one of 232: 32 and 34 % hit, 13.2 and 4.0 GB at 7.4 TB/s (with whole rows of X 10 % and 23.4 GB).  The next bound is
// instruction issue (a wave64 instruction holds its SIMD for four cycles): where a run ends is kept as scalar masks, rows and panels
// that need no bounds have none.
//
// us, one wavefront per 256 entries with whole rows of X (64 lanes across 64, 128 or 256 columns) -> this; 5.2 M entries of
// 262,144 rows, local columns, N = 8 / 16 / 32 / 64 / 128 / 256 / 1000: 251 / 248 / 246 / 248 / 385 / 745 / 3010 -> 81 / 84 / 96 /
// 154 / 277 / 535 / 2400; 40 M of 2 M rows, N = 16 / 64 / 128: 1560 / 1679 / 2732 -> 526 / 1205 / 2349; 10 M uniformly drawn,
// N = 32 / 128 / 500: 424 / 808 / 3448 -> 222 / 750 / 3180.  Tried and left: four wavefronts a workgroup (0 to 7 % slower), a persistent grid
// that fetches the next tile's entries early (15 % slower), three workgroups per CU by spilling four registers (6 % slower),
// less resident by LDS (no faster), X copied into panels of whole lines (no faster than wider panels, and a copy of X), and the
// rows of 512 entries and more taken out, ordered by ranges of columns that an L2 holds and summed range by range (their hits
// 27 -> 75 %, but what is left runs at 5.6 TB/s, and the lists and the sums cost what it gains: 2570 -> 2850 at N = 1000).
template <int VEC, int H, bool FULL, bool WIDE, bool SEARCH, bool ADD>
__global__ __launch_bounds__(PS_T, VEC * H <= 2 ? 8 : H == 1 ? 5 : 4) void panel_spmm_kernel(PanelJob job) {
  typedef PanelWalk<VEC, H, FULL, WIDE, 16 / H> Walk;
  typedef typename Walk::V V;
  typedef typename Walk::M M;
  __shared__ V s_head[PS_GROUPS][H][16];
  __shared__ uint32_t s_starts[PS_GROUPS];
  __shared__ uint32_t s_mark[SEARCH ? PS_TILE : 1], s_last[SEARCH ? PS_WAVES : 1];
  const int lane = lane_id(), s = lane & 15, w = wave_id(), group = w * 4 + (lane >> 4);
  const uint32_t n = job.n, ntiles = (n + PS_TILE - 1) / PS_TILE, per_xcd = (ntiles + 7) / 8;
  const uint32_t tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= ntiles) return;
  const uint32_t t0 = tile * PS_TILE, t1 = min(t0 + PS_TILE, n), e = t0 + threadIdx.x;
  const bool live = e < t1;
  const int32_t c = live ? __builtin_nontemporal_load(job.col + e) : 0;
  const float v = live ? __builtin_nontemporal_load(job.val + e) : 0.f;
  int32_t r = -1;
  bool start = true, next_same;     // the entry is the first of its row; the row of the tile's last entry goes on behind it
  int2 b0, b1;                      // parents of the entries around the tile's ends (at an end of the list the one inside)
  if constexpr (SEARCH) {
    s_mark[threadIdx.x] = 0;
  } else {
    if (live) r = job.row[e];
    if (live && e > 0) start = job.row[e - 1] != r;
    next_same = t1 < n && job.row[t1] == job.row[t1 - 1];
  }
  Walk walk;
  walk.columns(blockIdx.y, job.N, s);
  const char *X = reinterpret_cast<const char *>(job.X);
  char *Y = reinterpret_cast<char *>(job.Y);
  const auto xo = Walk::offset(c, job.ldx);
  // rows that begin in the tile mark their first entries (of rows that begin at the same entry the last one has entries); an entry's
  // row is the last mark up to it
  auto look_up = [&]() {
    if (job.bounds) {
      b0 = job.bounds[tile]; b1 = job.bounds[tile + 1];
    } else {
      const int2 p = find_parents(job.ptr, (uint32_t)job.nparents, t0 > 0 ? t0 - 1 : 0, t1 - 1, s_last);
      b0.x = p.x;
      b1 = make_int2(p.y, t1 < n && (uint32_t)job.ptr[p.y + 1] <= t1 ? -1 : p.y);
    }
    if (b1.x - b0.x > PS_FAR) {
      const uint32_t p = find_parent(job.ptr, b0.x, b1.x, e, live, s_mark);
      const bool first = live && (uint32_t)job.ptr[p] == e;
      __syncthreads();
      s_mark[threadIdx.x] = first ? p : 0;
    }
  };
  if constexpr (SEARCH && H > 1) look_up();   // (behind the gathers it takes more registers than these shapes have left)
  walk.first_gathers(X, xo);
  if constexpr (SEARCH) {
    if constexpr (H == 1) look_up();
    next_same = t1 < n && b1.x == b1.y;
    if (b1.x - b0.x <= PS_FAR) {
      __syncthreads();
      for (int32_t p = b0.x + 1 + (int32_t)threadIdx.x; p <= b1.x; p += PS_T) atomicMax(&s_mark[(uint32_t)job.ptr[p] - t0], (uint32_t)p);
    }
    __syncthreads();
    const uint32_t mark = s_mark[threadIdx.x];
    uint32_t last = wave_inclusive_max_dpp(mark);
    if (lane == 63) s_last[w] = last;
    __syncthreads();
    last = max(last, (uint32_t)b0.x);
#pragma unroll
    for (int q = 0; q < PS_WAVES - 1; ++q)
      if (q < w) last = max(last, s_last[q]);
    if (live) { start = mark != 0 || e == 0; r = job.ids ? job.ids[last] : (int32_t)last; }
  }
  const uint64_t sm = __ballot(start), dead = __ballot(!live);
  const auto yo = Walk::offset(r, job.ldy);
  walk.walk(X, xo, v, sm, dead, Y, yo, ADD, s_head[group], s);
  const uint32_t starts = (uint32_t)(sm >> (lane & 48)) & 0xffffu;
  if (s == 0) s_starts[group] = starts;
  const auto y_last = Walk::template of<15>(yo);
  const int32_t r_last = bcast16<15>(r);
  __syncthreads();
  const PanelRuns runs = panel_runs(s_starts);
  float *carry_head = job.carry + (int64_t)tile * 2 * job.carry_ld, *carry_tail = carry_head + job.carry_ld;
  // the group in which a run begins collects what later groups have of it
  const bool cut = starts != 0 && next_same && runs.next(group + 1) >= PS_GROUPS;   // the run goes on behind the tile
  if (starts != 0 && !(runs.fresh >> (group + 1) & 1)) {
    const int end = runs.end(group + 1);
#pragma unroll
    for (int h = 0; h < H; ++h) walk.acc[h] = panel_heads<H>(s_head, h, s, group + 1, end, walk.acc[h]);
  }
  const uint64_t full = __ballot(starts != 0 && !cut && r_last >= 0), part = __ballot(cut);
  uint64_t to[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    to[h] = full & walk.cols_ok[h];
    if (__builtin_amdgcn_inverse_ballot_w64(part & walk.cols_ok[h])) *reinterpret_cast<M *>(carry_tail + walk.c0[h]) = walk.acc[h];
  }
  walk.put(Y, y_last, to, ADD);
  const bool head_cut = !(runs.fresh & 1);   // the tile's first run began in an earlier one
  const bool single = head_cut && runs.next(0) >= PS_GROUPS;   // ... and is all that the tile holds
  if (head_cut && group == 0) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (!__builtin_amdgcn_inverse_ballot_w64(walk.cols_ok[h])) continue;
      *reinterpret_cast<M *>(carry_head + walk.c0[h]) = panel_heads<H>(s_head, h, s, 0, runs.end(0), V(0.f));
      if (single) *reinterpret_cast<M *>(carry_tail + walk.c0[h]) = V(0.f);
    }
  }
  if (job.carry_row && blockIdx.y == 0 && s == 0) {
    int32_t *cr = job.carry_row + (int64_t)tile * 2;
    if (group == 0) cr[0] = head_cut ? r : -1;
    if (single) { if (group == 0) cr[1] = r; }
    else if (starts != 0 && runs.next(group + 1) >= PS_GROUPS) cr[1] = cut ? r_last : -1;   // the group in which the last run begins
  }
}

// The pieces of rows that tile boundaries cut, in the order of the tiles (two slots a tile: reproducible).  A wavefront takes
// the run of slots of a row, if it is the run's first, and 256 columns.
__global__ __launch_bounds__(256) void panel_fixup_kernel(const int32_t *carry_row, const float *carry, int64_t carry_ld,
                                                          int64_t nslots, int64_t N, float *Y, int64_t ldy, int add) {
  const int lane = lane_id();
  const int64_t e = (int64_t)blockIdx.x * 4 + wave_id();
  if (e >= nslots) return;
  const int32_t r = carry_row[e];
  if (r < 0) return;
  if (e > 0 && carry_row[e - 1] == r) return;   // (a run never skips a slot)
  // length of the run, 64 slots per look (a 20,000-entry row leaves 80 pieces)
  int64_t len = 0;
  for (;;) {
    const int64_t j = e + len + lane;
    const uint64_t same = __ballot(j < nslots && carry_row[j] == r);
    const int run = same == ~0ull ? 64 : __ffsll((unsigned long long)~same) - 1;
    len += run;
    if (run < 64) break;
  }
  for (int64_t cb = (int64_t)blockIdx.y * 256; cb < N; cb += (int64_t)gridDim.y * 256) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    const float *p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = carry + e * carry_ld + min(cb + q * 64 + lane, N - 1);
    int64_t j = 0;
    for (; j + 8 <= len; j += 8) {   // 32 independent loads in flight, added in the order of the pieces
      float t[8][4];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) t[u][q] = p[q][(j + u) * carry_ld];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] += t[u][q];
    }
    for (; j < len; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] += p[q][j * carry_ld];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t c = cb + q * 64 + lane;
      if (c < N) {
        float *yp = Y + (int64_t)r * ldy + c;
        *yp = add ? *yp + s[q] : s[q];
      }
    }
  }
}

// ------------------------------------------------------------------ ELL
struct EllJob {
  const int32_t *col;
  const float *val;
  int64_t K, nrows;
  const float *X; int64_t ldx;
  float *Y; int64_t ldy;
  uint32_t N;
  int add;
  int64_t per_xcd;
};

// The lane groups of the kernel above over a slab: a group takes R rows and 16 / R slots of them at a time (one load of columns
// and one of values a lane, the next ones fetched early), so that a load brings pieces of four rows of X; where all four slots are
// pads it is jumped over by a scalar branch, where some are their lanes stay away.  Rows are whole: no pieces, no carries.  Bound by
// the misses of the L2s as well (N = 128: 49 M lines of 128 bytes, 5.9 TB/s), below 64 columns by the slab, which is pads to two
// thirds.  us, 8 rows a wavefront and one row of X a load -> this: 2 M rows of up to 20 slots, N = 1 / 16 / 33 / 64 / 72 / 128 459 / 471 /
// 542 / 614 / 1268 / 1005 -> 266 / 266 / 424 / 480 / 765 / 967; 250,000 rows of up to 42, N = 8 / 64 / 100 / 250 134 / 150 / 303 / 563 ->
// 82 / 116 / 200 / 448; 30,000 of up to 80, N = 4 / 64 57 / 63 -> 34 / 42; 3,000 of up to 20, N = 8 / 64 12 / 15 -> 10 / 11.  Measured
// and left: R = 2 (N = 16 319, N = 64 542), 8 (283, 532), 16 (287, 542, and 30,000 rows N = 64 119); the live slots of 64 to 512 rows put
// together in LDS and taken like a list (N = 16 469, N = 64 1462: a chain of barriers, and spills).
template <int VEC, int H, int R, bool FULL, bool WIDE>
__global__ __launch_bounds__(256) void ell_panel_kernel(EllJob job) {
  typedef PanelWalk<VEC, H, FULL, WIDE, 16 / H> Walk;
  typedef typename Walk::V V;
  typedef typename Walk::M M;
  constexpr int B = 16 / H, S = 16 / R;   // entries in flight; slots that a group takes together
  const int lane = lane_id(), s = lane & 15;
  const int64_t i0 = (((int64_t)(blockIdx.x & 7) * job.per_xcd + (blockIdx.x >> 3)) * 4 + wave_id()) * (4 * R);
  if (i0 >= job.nrows) return;
  Walk walk;
  walk.columns(blockIdx.y, job.N, s);
  const char *X = reinterpret_cast<const char *>(job.X);
  char *Y = reinterpret_cast<char *>(job.Y);
  const int64_t row0 = i0 + (lane >> 4) * R, i = row0 + (s & (R - 1));
  const bool mine = i < job.nrows;
  int64_t k = s / R;
  const int32_t *cp = job.col + k * job.nrows + i;
  const float *vp = job.val + k * job.nrows + i;
  V acc[R][H];
#pragma unroll
  for (int q = 0; q < R; ++q)
#pragma unroll
    for (int h = 0; h < H; ++h) acc[q][h] = V(0.f);
  int32_t c = mine && k < job.K ? __builtin_nontemporal_load(cp) : -1;
  float v = mine && k < job.K ? __builtin_nontemporal_load(vp) : 0.f;
  for (;;) {
    const uint64_t live = __ballot(c >= 0);
    if (live == 0) break;   // slots fill from the front
    k += S;
    cp += S * job.nrows; vp += S * job.nrows;
    const bool more = mine && k < job.K;
    const int32_t nc = more ? __builtin_nontemporal_load(cp) : -1;
    const float nv = more ? __builtin_nontemporal_load(vp) : 0.f;
    const auto xo = Walk::offset(c, job.ldx);
    static_for<0, H>([&](auto bc) {
      constexpr int q0 = decltype(bc)::value * B;
      V x[B][H];
      static_for<q0, q0 + B>([&](auto kc) {
        constexpr int q = decltype(kc)::value;
        const uint64_t m = (live >> q) & FIRST16;
        if (m) {
          const auto o = Walk::template of<q>(xo);
          if (__builtin_amdgcn_inverse_ballot_w64(spread16(m))) {
#pragma unroll
            for (int h = 0; h < H; ++h) x[q - q0][h] = *reinterpret_cast<const M *>(walk.at(X, o, h));
          }
        }
      });
      static_for<q0, q0 + B>([&](auto kc) {
        constexpr int q = decltype(kc)::value;
        const uint64_t m = (live >> q) & FIRST16;
        if (m) {
          const float t = bcast16<q>(v);
          if (__builtin_amdgcn_inverse_ballot_w64(spread16(m))) {
#pragma unroll
            for (int h = 0; h < H; ++h) acc[q & (R - 1)][h] += t * x[q - q0][h];
          }
        }
      });
    });
    c = nc; v = nv;
  }
  char *yp = Y + (uint64_t)row0 * (uint64_t)job.ldy * 4u;
  if (job.add) {   // (all is read before anything is written)
    V old[R][H];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int h = 0; h < H; ++h) {
        old[q][h] = V(0.f);
        if ((walk.cols_ok[h] >> lane & 1) && row0 + q < job.nrows) old[q][h] = *reinterpret_cast<const M *>(yp + q * job.ldy * 4 + walk.c0[h] * 4u);
      }
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int h = 0; h < H; ++h) acc[q][h] = old[q][h] + acc[q][h];
  }
#pragma unroll
  for (int q = 0; q < R; ++q)
#pragma unroll
    for (int h = 0; h < H; ++h)
      if ((walk.cols_ok[h] >> lane & 1) && row0 + q < job.nrows) *reinterpret_cast<M *>(yp + q * job.ldy * 4 + walk.c0[h] * 4u) = acc[q][h];
}

// Columns per lane and part, and parts, of the panels for `cols` columns.  Up to 64 columns one panel just wide enough.  Rows of X
// that begin at whole lines: 64, two lines a piece (262,144 rows, local columns, 5.2 M entries, N = 256, panels of 64 / 128 / 256:
// 545 / 554 / 592 us, 40 M and N = 128 2371 / 2559 / 2677; uniform, N = 512 657 / 663 / 671).  Others: every piece of a row
// touches a line more than it fills, so few and wide panels: N = 1000 2729 / 2468 / 2468, uniform, N = 500 4424 / 3740 / 3380;
// N = 100, one panel of 128 instead of two of 64: 375 -> 272.
struct PanelShape { int vec, parts; int width() const { return 16 * vec * parts; } };
static PanelShape panel_shape(int64_t cols, bool whole_lines) {
  if (cols <= 16) return {1, 1};
  if (cols <= 32) return {2, 1};
  if (cols <= 64 || whole_lines) return {4, 1};
  return {4, cols <= 128 ? 2 : 4};
}

void panel_spmm(Env &env, const us_formatted &A, const int32_t *row, const StoredRows *rows, const int32_t *col, const char *name,
                const float *X, int64_t N, int64_t ldx, float *Y, int64_t ldy, bool add) {
  const int64_t n = A.nnz, tiles = ceil_div<int64_t>(n, PS_TILE), carry_ld = ceil_div<int64_t>(N, 32) * 32;
  // A short list is bound by its launches and by the chain of loads inside a workgroup, not by lines.
  // - While all workgroups of panels of 64 columns are resident at once (512, two on a CU) these are taken whatever the lines: sixteen
  //   rows of X in flight instead of four.  Beyond 256 columns rows with pointers stop at half of that (us, panels of 64 / 256: 50,000
  //   entries of 5,000 / 2 M rows, N = 300 21.3 / 19.3, 59.6 / 54.7), lists with a row per entry, which look for nothing, at four
  //   times (50,000 of 8,000 rows, N = 1000 42.9 / 48.8).
  // - What is left of the columns beyond whole panels is one more panel of the same launch, and not a launch of its own, up to 1024
  //   workgroups; 2048 where Y is added to, which hides the idle lanes.  Rest apart -> this, us: 20,000 entries of 8,000 rows, N = 300
  //   31 -> 17, N = 1000 44 -> 27; 150,000 of 8,000 / 2 M, added, N = 300 45 -> 38, 186 -> 148; 400,000 of 200,000, added, 219 -> 193;
  //   but 1 M of 100,000, not added, 227 -> 248.
  // - Up to 1024 workgroups each finds its parents itself, some 3 us, where a launch of its own for the table of all takes 14: 50,000
  //   entries of 5,000 rows, N = 1 16.5 -> 12.0, 150,000 of 2 M 31 -> 21; beyond, where more rounds of workgroups pay for it, it depends on
  //   how many rows there are: 1 M (1,954 workgroups) of 2 M rows 47 -> 44, of 8,000, N = 64 26.5 -> 29.1.
  constexpr int64_t RESIDENT = 512;
  const bool whole_lines = (uintptr_t)X % 128 == 0 && ldx % 32 == 0;
  const bool narrow = whole_lines || tiles * ceil_div<int64_t>(N, 64) <= (N <= 256 ? RESIDENT : rows ? RESIDENT / 2 : 4 * RESIDENT);
  const int64_t workgroups = tiles * ceil_div<int64_t>(N, panel_shape(N, narrow).width());
  const bool one_launch = workgroups <= (add ? 4 : 2) * RESIDENT, table = rows && workgroups > 2 * RESIDENT;
  const size_t b_bounds = table ? Env::granule((tiles + 1) * sizeof(int2)) : 0, b_crow = Env::granule(tiles * 2 * sizeof(int32_t));
  char *ws = (char *)ensure_workspace(env, A, b_bounds + b_crow + tiles * 2 * carry_ld * sizeof(float));
  if (!env.ok()) return;
  int2 *bounds = (int2 *)ws;
  int32_t *carry_row = (int32_t *)(ws + b_bounds);
  float *carry = (float *)(ws + b_bounds + b_crow);
  if (table)
    US_LAUNCH(env, "spmm_bounds", 8.0 * tiles, tile_bounds_kernel, ceil_div<int64_t>(tiles + 1, 256), 256, rows->ptr, A.nmajor, n,
              tiles, bounds);
  const bool wide = (double)A.ncols * ldx * 4 >= 4294967296.0 || (double)A.nrows * ldy * 4 >= 4294967296.0;
  for (int64_t c = 0; c < N && env.ok();) {   // else: whole panels first, then what is left in one of the width that fits it
    const PanelShape shape = panel_shape(N - c, narrow);
    const int64_t pw = shape.width(), npanels = std::min<int64_t>(std::max<int64_t>(one_launch ? ceil_div<int64_t>(N - c, pw) : (N - c) / pw, 1), 65535);
    const int64_t cols = std::min(npanels * pw, N - c);
    PanelJob job{row, rows ? rows->ptr : nullptr, rows ? rows->row_ids : nullptr, table ? bounds : nullptr, A.nmajor, col, (const float *)A.val, (uint32_t)n,
                 X + c, ldx, Y + c, ldy, (uint32_t)cols, c == 0 ? carry_row : nullptr, carry + c, carry_ld};
    const dim3 grid((unsigned)(ceil_div<int64_t>(tiles, 8) * 8), (unsigned)npanels);
    LaunchScope ls(env, name, 12.0 * n + 4.0 * cols * (A.ncols + A.nrows));
    const bool full = cols % pw == 0;
#define US_PS_LAUNCH4(V, H, F, W, S, A) hipLaunchKernelGGL((panel_spmm_kernel<V, H, F, W, S, A>), grid, dim3(PS_T), 0, env.stream, job)
#define US_PS_LAUNCH3(V, H, F, W, S) do { if (add) US_PS_LAUNCH4(V, H, F, W, S, true); else US_PS_LAUNCH4(V, H, F, W, S, false); } while (0)
#define US_PS_LAUNCH2(V, H, F, W) do { if (rows) US_PS_LAUNCH3(V, H, F, W, true); else US_PS_LAUNCH3(V, H, F, W, false); } while (0)
#define US_PS_LAUNCH(V, H) do { if (wide) US_PS_LAUNCH2(V, H, false, true); else if (full) US_PS_LAUNCH2(V, H, true, false); else US_PS_LAUNCH2(V, H, false, false); } while (0)
    if (shape.vec == 1) US_PS_LAUNCH(1, 1);
    else if (shape.vec == 2) US_PS_LAUNCH(2, 1);
    else if (shape.parts == 1) US_PS_LAUNCH(4, 1);
    else if (shape.parts == 2) US_PS_LAUNCH(4, 2);
    else US_PS_LAUNCH(4, 4);
#undef US_PS_LAUNCH
#undef US_PS_LAUNCH2
#undef US_PS_LAUNCH3
#undef US_PS_LAUNCH4
    env.check(hipGetLastError());
    c += cols;
  }
  if (!env.ok()) return;
  LaunchScope ls(env, "spmm_rows_fixup", 8.0 * tiles);
  hipLaunchKernelGGL(panel_fixup_kernel, dim3((unsigned)ceil_div<int64_t>(tiles * 2, 4), (unsigned)std::min<int64_t>(ceil_div<int64_t>(N, 256), 65535)),
                     dim3(256), 0, env.stream, (const int32_t *)carry_row, (const float *)carry, carry_ld, tiles * 2, N, Y, ldy, add ? 1 : 0);
  env.check(hipGetLastError());
}

// Up to 64 columns one panel just wide enough, up to 128 one of 128, up to 256 one of 256 (with half as many rows a wavefront: the
// sums are in registers), beyond that panels of 128 and one for the rest.
void panel_ell_spmm(Env &env, const us_formatted &A, const float *X, int64_t N, int64_t ldx, float *Y, int64_t ldy, bool add) {
  const bool wide = (double)A.ncols * ldx * 4 >= 4294967296.0 || (double)A.nrows * ldy * 4 >= 4294967296.0;
  for (int64_t c = 0; c < N && env.ok();) {
    PanelShape shape = panel_shape(N - c, false);
    if (N > 256 && shape.parts == 4) shape.parts = 2;
    const int64_t pw = shape.width(), npanels = std::min<int64_t>(std::max<int64_t>((N - c) / pw, 1), 65535), cols = std::min(npanels * pw, N - c);
    const int64_t per_xcd = ceil_div<int64_t>(A.nrows, 8 * 16 * (shape.parts == 4 ? 2 : 4));
    const EllJob job{A.level[2].idx, (const float *)A.val, A.nmajor, A.nrows, X + c, ldx, Y + c, ldy, (uint32_t)cols, add ? 1 : 0, per_xcd};
    const dim3 grid((unsigned)(per_xcd * 8), (unsigned)npanels);
    const bool full = cols % pw == 0;
    LaunchScope ls(env, "spmm_ell", 8.0 * A.nval + 4.0 * cols * (A.ncols + A.nrows));
#define US_EP_LAUNCH2(V, H, R, F, W) hipLaunchKernelGGL((ell_panel_kernel<V, H, R, F, W>), grid, dim3(256), 0, env.stream, job)
#define US_EP_LAUNCH(V, H, R) do { if (wide) US_EP_LAUNCH2(V, H, R, false, true); else if (full) US_EP_LAUNCH2(V, H, R, true, false); else US_EP_LAUNCH2(V, H, R, false, false); } while (0)
    if (shape.vec == 1) US_EP_LAUNCH(1, 1, 4);
    else if (shape.vec == 2) US_EP_LAUNCH(2, 1, 4);
    else if (shape.parts == 1) US_EP_LAUNCH(4, 1, 4);
    else if (shape.parts == 2) US_EP_LAUNCH(4, 2, 4);
    else US_EP_LAUNCH(4, 4, 2);
#undef US_EP_LAUNCH
#undef US_EP_LAUNCH2
    env.check(hipGetLastError());
    c += cols;
  }
}

}  // namespace us
