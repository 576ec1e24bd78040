// The decompose op (Section 6): rank-in-row splits (ELL + COO hybrids), splits by the nodes of a blocked layout
// (the #sum queries of Figure 3c and of the BELL/COO case study), and the dispatch over predicates.
#include "convert_internal.h"
#include "device.h"

#include <algorithm>

namespace us {

// ------------------------------------------------------------------ decompose
// The row length of a given rank (the nearest-rank percentile) without sorting the lengths: digit by digit from the top,
// every launch counts the values of its digit among the rows whose length agrees with the digits picked so far.  The digit
// that holds the rank is picked by every workgroup of the launch that follows, for itself: 8 KB from L2 and a scan, where a
// launch of one workgroup in between takes as long as the count (2 M rows: three digits of 8 bits with such launches 66 us, two
// of 11 bits 25).  At most SEL_GRID workgroups, each adding up in LDS first:
// the lengths of a matrix crowd into a few values, and adds to the same device counter take their turns at ~20 ns each
// (a thousand workgroups: 63 us a pass on 2 M rows).
constexpr int SEL_T = 512, SEL_GRID = 256, SEL_IPT = 8, SEL_TILE = SEL_T * SEL_IPT;
constexpr int SEL_BITS = 11, SEL_BINS = 1 << SEL_BITS, SEL_PASSES = 3;   // lengths have 31 bits
struct SelectState {
  uint32_t hist[SEL_PASSES][SEL_BINS];     // zero before the first pass
  struct { uint32_t prefix, rank; } at[SEL_PASSES + 1];   // at[p]: the digits picked before pass p, and the rank among the rows they leave
};

// what pass `pass` (of `bits` bits) picks, in every thread.  If no count holds the rank (the lengths are garbage) the digit is 0.
template <int T>
__device__ __forceinline__ uint2 select_pick(const SelectState *s, int pass, int bits) {
  constexpr int PER = SEL_BINS / T;
  __shared__ uint32_t s_wave[T / 64 + 1];
  __shared__ uint2 s_pick;
  const uint32_t prefix = s->at[pass].prefix << bits, rank = s->at[pass].rank;
  uint32_t cnt[PER], sum = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) sum += cnt[k] = s->hist[pass][threadIdx.x * PER + k];
  if (threadIdx.x == 0) s_pick = make_uint2(prefix, rank);
  uint32_t total;
  uint32_t before = block_exclusive_sum<T>(sum, s_wave, &total);
#pragma unroll
  for (int k = 0; k < PER; ++k) {   // one bin of the workgroup
    if (before <= rank && rank - before < cnt[k]) s_pick = make_uint2(prefix | (threadIdx.x * PER + k), rank - before);
    before += cnt[k];
  }
  __syncthreads();
  return s_pick;
}

// prev_bits: how many the pass before this one has
__global__ __launch_bounds__(SEL_T) void select_count_kernel(const int32_t *ptr, int64_t nrows, int pass, int shift, int bits,
                                                            int prev_bits, uint32_t rank, SelectState *s) {
  __shared__ uint32_t s_hist[SEL_BINS];
  for (int i = threadIdx.x; i < SEL_BINS; i += SEL_T) s_hist[i] = 0;
  const uint2 at = pass > 0 ? select_pick<SEL_T>(s, pass - 1, prev_bits) : make_uint2(0u, rank);
  if (blockIdx.x == 0 && threadIdx.x == 0) { s->at[pass].prefix = at.x; s->at[pass].rank = at.y; }
  __syncthreads();
  const int hi = shift + bits;
  const uint32_t mask = (1u << bits) - 1u;
  for (int64_t base = (int64_t)blockIdx.x * SEL_TILE; base < nrows; base += (int64_t)gridDim.x * SEL_TILE) {
    uint32_t v[SEL_IPT];
#pragma unroll
    for (int k = 0; k < SEL_IPT; ++k) {   // all loads first
      const int64_t g = base + k * SEL_T + threadIdx.x;
      v[k] = g < nrows ? (uint32_t)(ptr[g + 1] - ptr[g]) : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int k = 0; k < SEL_IPT; ++k) {
      const int64_t g = base + k * SEL_T + threadIdx.x;
      if (g < nrows && (hi >= 32 ? 0u : v[k] >> hi) == at.x) atomicAdd(&s_hist[(v[k] >> shift) & mask], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < SEL_BINS; i += SEL_T)
    if (s_hist[i]) atomicAdd(&s->hist[pass][i], s_hist[i]);
}

// Where the entries that a cut at rank K leaves over go: ptr_b[r] = sum of max(length - K, 0) over the rows before r (the
// entries below the cut start at ptr[r] - ptr_b[r]).  A reduction per tile of rows, which also finds the longest row, a
// scan of the tiles' sums, and the prefixes, each reading the lengths from ptr (not from an array of them).
constexpr int RC_T = 256, RC_IPT = 8, RC_TILE = RC_T * RC_IPT;
__device__ __forceinline__ uint32_t beyond(int32_t len, int64_t K) { return len > K ? (uint32_t)(len - K) : 0u; }

// sel != null: K is what the last pass of the select picks, left in *K_dev for the launches that follow
__global__ __launch_bounds__(RC_T) void rank_reduce_kernel(const int32_t *ptr, int64_t nrows, int64_t K, const SelectState *sel,
                                                          int last_pass, int last_bits, int32_t *K_dev, uint2 *partial) {
  __shared__ uint32_t s_wave[RC_T / 64 + 1];
  __shared__ int32_t s_max[RC_T / 64];
  const int64_t base = (int64_t)blockIdx.x * RC_TILE;
  int32_t len[RC_IPT], most = 0;
#pragma unroll
  for (int k = 0; k < RC_IPT; ++k) {
    const int64_t g = base + k * RC_T + threadIdx.x;
    len[k] = g < nrows ? ptr[g + 1] - ptr[g] : 0;
  }
  if (sel) {
    K = (int32_t)select_pick<RC_T>(sel, last_pass, last_bits).x;
    if (blockIdx.x == 0 && threadIdx.x == 0) *K_dev = (int32_t)K;
  }
  uint32_t s = 0, total;
#pragma unroll
  for (int k = 0; k < RC_IPT; ++k) { s += beyond(len[k], K); most = max(most, len[k]); }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) most = max(most, __shfl_xor(most, d));
  if (lane_id() == 0) s_max[wave_id()] = most;
  block_exclusive_sum<RC_T>(s, s_wave, &total);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < RC_T / 64; ++w) most = max(most, s_max[w]);
    partial[blockIdx.x] = make_uint2(total, (uint32_t)most);
  }
}
__global__ __launch_bounds__(RC_T) void rank_apply_kernel(const int32_t *ptr, int64_t nrows, int64_t K, const int32_t *K_dev,
                                                         const uint2 *partial, int32_t *ptr_b) {
  __shared__ uint32_t s_wave[RC_T / 64 + 1];
  if (K_dev) K = *K_dev;
  const int64_t r0 = (int64_t)blockIdx.x * RC_TILE + (int64_t)threadIdx.x * RC_IPT;   // eight rows in a row; arrays start at 256 bytes
  int32_t p[RC_IPT + 1];
  const bool whole = r0 + RC_IPT <= nrows;
  if (whole) {
    const int4 a = *reinterpret_cast<const int4 *>(ptr + r0), b = *reinterpret_cast<const int4 *>(ptr + r0 + 4);
    p[0] = a.x; p[1] = a.y; p[2] = a.z; p[3] = a.w; p[4] = b.x; p[5] = b.y; p[6] = b.z; p[7] = b.w;
    p[8] = ptr[r0 + 8];
  } else {
#pragma unroll
    for (int k = 0; k <= RC_IPT; ++k) p[k] = r0 + k <= nrows ? ptr[r0 + k] : 0;
  }
  uint32_t v[RC_IPT], s = 0, total;
#pragma unroll
  for (int k = 0; k < RC_IPT; ++k) {
    v[k] = r0 + k < nrows ? beyond(p[k + 1] - p[k], K) : 0u;
    s += v[k];
  }
  uint32_t ex = block_exclusive_sum<RC_T>(s, s_wave, &total) + partial[blockIdx.x].x;
  int32_t o[RC_IPT];
#pragma unroll
  for (int k = 0; k < RC_IPT; ++k) { o[k] = (int32_t)ex; ex += v[k]; }
  if (whole) {
    *reinterpret_cast<int4 *>(ptr_b + r0) = make_int4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<int4 *>(ptr_b + r0 + 4) = make_int4(o[4], o[5], o[6], o[7]);
  } else {
#pragma unroll
    for (int k = 0; k < RC_IPT; ++k)
      if (r0 + k < nrows) ptr_b[r0 + k] = o[k];
  }
  if (r0 < nrows && r0 + RC_IPT >= nrows) ptr_b[nrows] = (int32_t)ex;   // (what lies behind the last row is 0)
}

// Part B alone (part A is an ELL slab built from the rows of the sorted list): entry z of it belongs to the row r with
// ptr_b[r] <= z < ptr_b[r + 1] and comes from ptr[r] + K + (z - ptr_b[r]).  Only what part B holds is moved, and the rows
// come from ptr_b, so that the sort need not write one per entry.  Bound by memory and by the chain from one search step to
// the next: 26 M entries of a list of 40 M, 2 M rows, 139 us, 4.1 TB/s (a pass over the whole list 165; tiles of 2048 steps,
// twice as many searches, 154).  A workgroup takes an equal share of
// the merged sequence of row ends and entries of part B, since either can be few: a list with one entry left over in a few
// of very many rows, or one row that holds them all.  Ends of part B are looked for by all threads at once.
constexpr int RT_T = 512, RT_IPT = 8, RT_TILE = RT_T * RT_IPT;
__global__ __launch_bounds__(RT_T) void rank_tail_kernel(const int32_t *minor, const float *val, const int32_t *ptr,
                                                        const int32_t *ptr_b, int64_t nrows, int64_t nb, int32_t K,
                                                        int32_t *br, int32_t *bc, float *bv) {
  __shared__ __align__(16) int32_t s_row[RT_TILE];   // entry of the tile -> row of the tile
  __shared__ int32_t s_from[RT_TILE];                // row of the tile -> where entry 0 of part B would come from
  __shared__ int32_t s_wave[RT_T / 64];
  const int tid = threadIdx.x;
  const int64_t diag0 = (int64_t)blockIdx.x * RT_TILE, diag1 = min(diag0 + (int64_t)RT_TILE, nrows + nb);
  // rows that end before the tile: their end, ptr_b[r + 1], is step ptr_b[r + 1] + r of the sequence
  int64_t r0 = 0, hi = nrows;
  while (r0 < hi) {
    const int64_t step = ceil_div<int64_t>(hi - r0, RT_T), r = r0 + (tid + 1) * step - 1;
    const int c = __syncthreads_count(r < hi && ptr_b[r + 1] + r < diag0);
    r0 += c * step;
    hi = min(hi, r0 + step - 1);
  }
  const int64_t z0 = diag0 - r0;
#pragma unroll
  for (int k = 0; k < RT_IPT; ++k) s_row[k * RT_T + tid] = 0;
  __syncthreads();
  int nr = 0;   // rows that end inside the tile
  for (int i = tid;; i += RT_T) {
    const int64_t r = r0 + i;
    bool ends = false;
    if (r < nrows) {
      const int64_t b0 = ptr_b[r], b1 = ptr_b[r + 1], first = max(b0, z0);
      ends = b1 + r < diag1;
      if (first < b1 && first + r < diag1) {   // then first - z0 and i are below RT_TILE
        s_row[first - z0] = i;
        s_from[i] = ptr[r] + K - (int32_t)b0;
      }
    }
    const int c = __syncthreads_count(ends);
    nr += c;
    if (c < RT_T) break;
  }
  const int nz = (int)(diag1 - diag0) - nr;
  // the row of an entry is the last one marked up to it (the first entry is marked)
  int4 *mine = reinterpret_cast<int4 *>(s_row + tid * RT_IPT);
  static_assert(RT_IPT == 8, "two int4 per thread");
  int4 a = mine[0], b = mine[1];
  a.y = max(a.x, a.y); a.z = max(a.y, a.z); a.w = max(a.z, a.w);
  b.x = max(a.w, b.x); b.y = max(b.x, b.y); b.z = max(b.y, b.z); b.w = max(b.z, b.w);
  int32_t upto = b.w;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t t = __shfl_up(upto, d);
    if (lane_id() >= d) upto = max(upto, t);
  }
  if (lane_id() == 63) s_wave[wave_id()] = upto;
  int32_t before = __shfl_up(upto, 1);
  if (lane_id() == 0) before = 0;
  __syncthreads();
  for (int w = 0; w < wave_id(); ++w) before = max(before, s_wave[w]);
  a.x = max(a.x, before); a.y = max(a.y, before); a.z = max(a.z, before); a.w = max(a.w, before);
  b.x = max(b.x, before); b.y = max(b.y, before); b.z = max(b.z, before); b.w = max(b.w, before);
  mine[0] = a; mine[1] = b;
  __syncthreads();
  int32_t row[RT_IPT], c[RT_IPT];
  float v[RT_IPT];
#pragma unroll
  for (int k = 0; k < RT_IPT; ++k) {   // all loads first
    const int p = k * RT_T + tid;
    row[k] = 0; c[k] = 0; v[k] = 0.f;
    if (p < nz) {
      const int i = s_row[p];
      const int64_t from = (int64_t)s_from[i] + z0 + p;
      row[k] = (int32_t)(r0 + i); c[k] = minor[from]; v[k] = val[from];
    }
  }
#pragma unroll
  for (int k = 0; k < RT_IPT; ++k) {
    const int p = k * RT_T + tid;
    if (p < nz) { br[z0 + p] = row[k]; bc[z0 + p] = c[k]; bv[z0 + p] = v[k]; }
  }
}

// stable split of the sorted list by rank-in-row: rank < K -> part A, else part B.  (Equal neighbours have
// been looked for before: the two copies of a coordinate may end up in different parts.)
constexpr int RSP_IPT = 4;
__global__ __launch_bounds__(256) void rank_split_kernel(const int32_t *major, const int32_t *minor, const float *val,
                                                        const int32_t *ptr, const int32_t *ptr_b, int64_t n,
                                                        int64_t K, CooLists la, CooLists lb) {
  // RSP_IPT entries per thread, each step for all of them before the next: the entry, then the two pointers of its
  // row, then the stores
  const int64_t base = (int64_t)blockIdx.x * (256 * RSP_IPT) + threadIdx.x;
  int32_t r[RSP_IPT], c[RSP_IPT], p0[RSP_IPT], pb[RSP_IPT];
  float v[RSP_IPT];
#pragma unroll
  for (int k = 0; k < RSP_IPT; ++k) {
    const int64_t i = base + k * 256;
    r[k] = i < n ? major[i] : 0; c[k] = i < n ? minor[i] : 0; v[k] = i < n ? val[i] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < RSP_IPT; ++k) {
    const bool in = base + k * 256 < n;
    p0[k] = in ? ptr[r[k]] : 0; pb[k] = in ? ptr_b[r[k]] : 0;
  }
#pragma unroll
  for (int k = 0; k < RSP_IPT; ++k) {
    const int64_t i = base + k * 256;
    if (i >= n) continue;
    const int64_t rank = i - p0[k];
    const int64_t p = rank < K ? p0[k] - pb[k] + rank : pb[k] + (rank - K);
    const CooLists &l = rank < K ? la : lb;
    l.r[p] = r[k]; l.c[p] = c[k]; l.v[p] = v[k];
  }
}

static bool row_major_family(const Plan &p) {
  return !p.swapped && (p.pattern == P_COO || p.pattern == P_CSR || p.pattern == P_DCSR || p.pattern == P_ELL);
}

static us_status decompose_rank(Env &env, const us_coo &coo, const Plan &pa, const us_format_desc &da, const Plan &pb,
                                const us_format_desc &db, const us_predicate &pred, us_formatted **oa,
                                us_formatted **ob) {
  const int64_t n = coo.nnz, nrows = coo.nrows;
  const KeySpec ks = rowcol_keyspec(coo, false);
  const bool with_ptr = sort_gives_ptr(env, n, ks, false), slab = pa.pattern == P_ELL && !pa.swapped;
  const bool need_major = !slab || !with_ptr;   // (part B beside a slab is split off by rows)
  const bool by_percentile = pred.kind == US_P_RANK_LT_PERCENTILE;
  const int64_t ntile = ceil_div<int64_t>(nrows, RC_TILE);
  {  // every temporary of the call in one allocation
    auto g = [](size_t count) { return Env::granule(4 * count); };
    env.reserve(sort_temp_bytes(env, n, ks, false) + (need_major ? 3 : 2) * g(n) + 2 * g(nrows + 1) + g(2 * ntile) +
                Env::granule(sizeof(SelectState)) + 4 * Env::granule(sizeof(Flags)));
  }
  Flags *flags = new_flags(env, false);
  int32_t *major = need_major ? env.temp<int32_t>(n) : nullptr, *minor = env.temp<int32_t>(n);
  float *val = env.temp<float>(n);
  int32_t *ptr = env.temp<int32_t>(nrows + 1), *ptr_b = env.temp<int32_t>(nrows + 1);
  uint2 *partial = env.temp<uint2>(ntile);
  SelectState *sel = by_percentile ? env.temp<SelectState>(1) : nullptr;
  if (!env.ok()) return env.status;
  SortOut so{};
  so.clear_flags = true;
  so.major = major; so.minor = minor; so.val = val;
  if (with_ptr) so.ptr = ptr;
  const bool checked = sort_coo(env, coo.row, coo.col, coo.val, n, ks, so, flags);
  if (!env.ok()) return env.status;
  if (!so.ptr_done) sorted_ptr(env, major, minor, n, nrows, ptr, !checked, flags);
  Flags h{};
  int64_t K = pred.abs;
  int npass = 0, last_bits = 0;
  if (by_percentile) {
    // nearest-rank percentile of the row lengths over all rows: the length of rank k - 1 in ascending order
    const int64_t maxlen = n < coo.ncols ? n : coo.ncols;
    int64_t k = (pred.num * nrows + pred.den - 1) / pred.den;
    if (k < 1) k = 1;
    if (k > nrows) k = nrows;
    const int total_bits = bits_for((uint64_t)maxlen) > 0 ? bits_for((uint64_t)maxlen) : 1;
    npass = ceil_div(total_bits, SEL_BITS);
    fill_u32(env, &sel->hist[0][0], (uint64_t)npass * SEL_BINS, 0u);
    const int64_t grid = std::min<int64_t>(ceil_div<int64_t>(nrows, SEL_TILE), SEL_GRID);
    for (int p = 0, left = total_bits; p < npass; ++p) {
      const int w = total_bits / npass + (p < total_bits % npass ? 1 : 0);
      left -= w;
      US_LAUNCH(env, "select_count", 4.0 * nrows, select_count_kernel, grid, SEL_T, (const int32_t *)ptr, nrows, p, left, w,
                last_bits, (uint32_t)(k - 1), sel);
      last_bits = w;
    }
  }
  // the cut K (if picked above), the size of part B and the longest row all come back in one read of the flags
  US_LAUNCH(env, "rank_reduce", 4.0 * nrows, rank_reduce_kernel, ntile, RC_T, (const int32_t *)ptr, nrows, K,
            (const SelectState *)sel, npass - 1, last_bits, &flags->scalar[2], partial);
  scan_pairs(env, partial, ntile, &flags->scalar[1], &flags->scalar[3], true);
  US_LAUNCH(env, "rank_apply", 8.0 * nrows, rank_apply_kernel, ntile, RC_T, (const int32_t *)ptr, nrows, K,
            (const int32_t *)(by_percentile ? &flags->scalar[2] : nullptr), (const uint2 *)partial, ptr_b);
  if (!read_flags(env, flags, &h)) return env.status;
  if (flag_status(h) != US_OK) return flag_status(h);
  if (by_percentile) K = h.scalar[2];
  const int64_t longest = h.scalar[3];
  const int64_t nb = h.scalar[1], na = n - nb;
  // part A as row-major ELL: its slab is built from the first min(length, K) entries of every row of the sorted
  // list (which gives the automatic width), 64 rows at a time through LDS; only part B is split off as a list.
  // Any other format of part A gets a sorted list first.
  us_formatted *ell = nullptr;
  if (slab) {
    const int64_t ell_width = pa.ell_width > 0 ? pa.ell_width : (longest < K ? longest : K);
    if (ell_width * nrows >= (1ll << 31)) return US_ERR_OVERFLOW;
    ell = new_ell_of_rows(env, da, nrows, coo.ncols, na, ell_width, K, minor, val, ptr, flags);
    if (!ell) return env.status;
  }
  CooLists la = ell ? CooLists() : alloc_lists(env, na), lb = alloc_lists(env, nb);
  us_status st = env.status;
  if (st == US_OK && ell && nb > 0) {   // (then the cut is below the longest row and fits 31 bits)
    US_LAUNCH(env, "rank_tail", 20.0 * nb + 8.0 * nrows, rank_tail_kernel, ceil_div<int64_t>(nrows + nb, RT_TILE), RT_T,
              (const int32_t *)minor, (const float *)val, (const int32_t *)ptr, (const int32_t *)ptr_b, nrows, nb, (int32_t)K,
              lb.r, lb.c, lb.v);
    st = env.status;
  } else if (st == US_OK && !ell && n > 0) {
    US_LAUNCH(env, "rank_split", 28.0 * n, rank_split_kernel, ceil_div<int64_t>(n, 256 * RSP_IPT), 256,
              (const int32_t *)major, (const int32_t *)minor, (const float *)val, (const int32_t *)ptr,
              (const int32_t *)ptr_b, n, K, la, lb);
    st = env.status;
  }
  auto finish_part = [&](const Plan &p, const us_format_desc &d, CooLists &l, int64_t cnt, us_formatted **o) {
    if (row_major_family(p)) {   // the list is already in (row, col) order: no second sort
      // the same flag block goes on (its duplicate flag may have been set by the split); sizes start from zero
      fill_u32(env, (uint32_t *)&flags->scalar[0], 4, 0u);
      if (!env.ok()) return env.status;
      Plan q = p;
      // part A as ELL of automatic width: its rows hold min(length, K) entries, so the width is known here
      if (&l == &la && q.pattern == P_ELL && q.ell_width == 0) q.ell_width = longest < K ? longest : K;
      us_status s = build_from_sorted(env, q, d, coo.nrows, coo.ncols, cnt, l.r, l.c, l.v, flags, false, o, true);
      l = CooLists();  // ownership moved
      return s;
    }
    Flags hh{};
    if (!read_flags(env, flags, &hh)) return env.status;
    if (flag_status(hh) != US_OK) return flag_status(hh);
    us_coo c{coo.nrows, coo.ncols, cnt, l.r, l.c, l.v};
    return convert_with_plan(env, c, p, d, o);
  };
  if (st == US_OK && !ell) st = finish_part(pa, da, la, na, oa);
  if (st == US_OK) st = finish_part(pb, db, lb, nb, ob);   // ends with a read of the flags: covers the slab's overflow flag too
  if (ell) {
    if (st == US_OK) *oa = ell; else free_formatted(env, ell);
  }
  env.sync();
  free_lists(env, la);
  free_lists(env, lb);
  return st;
}

// ------------------------------------------------------------------ decompose by the nodes of a blocked layout
// The #sum query of the BDIA/CSR hybrid (Figure 3c) groups by (d0/b, d1-d0), the one of the BELL/COO case
// study (Section 7.2.2) by blocks (d0/bh, d1/bw).  Such groups are exactly the nodes of the BDIA / BCSR tree, so the entries are sorted by the BDIA tuple first: a group is then a run
// of the sorted list, its count is the run length, and the entries that stay (part A) are already
// in BDIA order -- no second sort for them.
__global__ __launch_bounds__(256) void node_head_kernel(const uint64_t *key, int64_t n, int ih_bits, int32_t *head,
                                                       Flags *flags) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint64_t cur = key[i], prev = i > 0 ? key[i - 1] : ~0ull;
  if (i > 0 && cur == prev) flags->duplicate = 1;
  head[i] = (i == 0) | ((cur >> ih_bits) != (prev >> ih_bits));
}

// start[g] = first entry of run g; the slot after the last run gets n
__global__ __launch_bounds__(256) void node_start_kernel(const int32_t *head, const int32_t *pos, int64_t n,
                                                        int32_t *start) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  if (head[i]) start[pos[i]] = (int32_t)i;
  if (i == n - 1) start[pos[i] + head[i]] = (int32_t)n;
}

__global__ __launch_bounds__(256) void node_keep_kernel(const int32_t *head, const int32_t *pos, const int32_t *start,
                                                       int64_t n, int64_t thld, int32_t *keep) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int32_t g = pos[i] + head[i] - 1;
  keep[i] = (int64_t)(start[g + 1] - start[g]) >= thld ? 1 : 0;
}

// The same decision without the run tables when a node cannot hold more than `width` entries (a blocked
// diagonal piece holds at most b, a bh x bw block bh*bw): every entry counts its run by looking at most
// width - 1 neighbours to either side (cached reads), and equal neighbours are flagged on the way.
constexpr int NK_T = 256, NK_IPT = 4, NK_TILE = NK_T * NK_IPT, NK_HALO = 15;
__global__ __launch_bounds__(NK_T) void node_keep_window_kernel(const uint64_t *key, int64_t n, int ih_bits, int width,
                                                               int64_t thld, int32_t *keep, Flags *flags) {
  __shared__ uint64_t s_key[NK_TILE + 2 * NK_HALO];   // the tile's keys with width - 1 <= NK_HALO neighbours either side
  const int64_t i0 = (int64_t)blockIdx.x * NK_TILE - NK_HALO;
  for (int t = threadIdx.x; t < NK_TILE + 2 * NK_HALO; t += NK_T) {
    const int64_t i = i0 + t;
    s_key[t] = (i >= 0 && i < n) ? key[i] : 0ull;
  }
  __syncthreads();
  bool dup = false;
#pragma unroll
  for (int k = 0; k < NK_IPT; ++k) {
    const int t = NK_HALO + k * NK_T + threadIdx.x;
    const int64_t i = i0 + t;
    if (i >= n) continue;
    const uint64_t cur = s_key[t], node = cur >> ih_bits;
    dup |= i > 0 && s_key[t - 1] == cur;
    int count = 1;
    for (int d = 1; d < width && i - d >= 0 && (s_key[t - d] >> ih_bits) == node; ++d) ++count;
    for (int d = 1; d < width && i + d < n && (s_key[t + d] >> ih_bits) == node; ++d) ++count;
    keep[i] = count >= thld ? 1 : 0;
  }
  if (dup) flags->duplicate = 1;
}

__global__ __launch_bounds__(256) void node_split_kernel(const uint64_t *key, const float *val, const int32_t *keep,
                                                        const int32_t *pos_a, int64_t n, KeySpec ks, uint64_t *key_a,
                                                        float *val_a, CooLists la, CooLists lb) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint64_t k = key[i];
  const bool a = keep[i] != 0;
  const int64_t at = a ? pos_a[i] : i - pos_a[i];
  if (a && key_a) { key_a[at] = k; val_a[at] = val[i]; return; }
  const int inner = ks.ih_bits + ks.iw_bits;
  const uint64_t bk = k >> inner;
  const int32_t row = (int32_t)((bk >> ks.b_bits) * ks.bh + ((k >> ks.iw_bits) & ((1ull << ks.ih_bits) - 1)));
  const int32_t second = (int32_t)(bk & ((1ull << ks.b_bits) - 1));
  // blocked diagonal: the second component is d1 - d0 biased by nrows - 1; blocks: d1 / bw, with d1 % bw below
  const int32_t col = ks.mode == 2 ? row + second - (int32_t)(ks.a_extent - 1)
                                   : second * (int32_t)ks.bw + (int32_t)(k & ((1ull << ks.iw_bits) - 1));
  const CooLists &l = a ? la : lb;
  l.r[at] = row; l.c[at] = col; l.v[at] = val[i];
}

static us_status decompose_blocked(Env &env, const us_coo &coo, const Plan &pa, const us_format_desc &da,
                                   const Plan &pb, const us_format_desc &db, const Plan &pg, int64_t thld,
                                   us_formatted **oa, us_formatted **ob) {
  Flags *flags = new_flags(env);
  const int64_t n = coo.nnz;
  const KeySpec ks = blocked_keyspec(pg, coo.nrows, coo.ncols);
  const int inner_bits = ks.ih_bits + ks.iw_bits;
  // part A keeps the sorted order when it is stored by the very tuple the groups were cut by
  const bool direct = (pa.pattern == pg.pattern || (pa.pattern == P_BELL && pg.pattern == P_BCSR)) && pa.bh == pg.bh && pa.bw == pg.bw;
  uint64_t *skey = env.temp<uint64_t>(n);
  float *sval = env.temp<float>(n);
  int32_t *keep = env.temp<int32_t>(n), *pos_a = env.temp<int32_t>(n);
  if (!env.ok()) return env.status;
  int64_t na = 0;
  if (n > 0) {
    SortOut so{};
    so.key64 = skey; so.val = sval;
    sort_coo(env, coo.row, coo.col, coo.val, n, ks, so, flags);
    const int64_t g = ceil_div<int64_t>(n, 256);
    const int64_t width = pg.bh * pg.bw;   // the most entries a node can hold
    if (width <= 16) {
      US_LAUNCH(env, "node_keep", 12.0 * n, node_keep_window_kernel, ceil_div<int64_t>(n, NK_TILE), NK_T,
                (const uint64_t *)skey, n, inner_bits, (int)width, thld, keep, flags);
    } else {
      int32_t *head = env.temp<int32_t>(n), *pos = env.temp<int32_t>(n), *start = env.temp<int32_t>(n + 1);
      if (!env.ok()) return env.status;
      US_LAUNCH(env, "node_head", 12.0 * n, node_head_kernel, g, 256, (const uint64_t *)skey, n, inner_bits, head, flags);
      exclusive_scan_i32(env, head, pos, n, &flags->scalar[0]);
      US_LAUNCH(env, "node_start", 12.0 * n, node_start_kernel, g, 256, (const int32_t *)head, (const int32_t *)pos, n,
                start);
      US_LAUNCH(env, "node_keep", 16.0 * n, node_keep_kernel, g, 256, (const int32_t *)head, (const int32_t *)pos,
                (const int32_t *)start, n, thld, keep);
    }
    exclusive_scan_i32(env, keep, pos_a, n, &flags->scalar[1]);
    Flags h{};
    if (!read_flags(env, flags, &h)) return env.status;
    if (flag_status(h) != US_OK) return flag_status(h);
    na = h.scalar[1];
  }
  const int64_t nb = n - na;
  uint64_t *key_a = direct ? env.temp<uint64_t>(na) : nullptr;
  float *val_a = direct ? env.temp<float>(na) : nullptr;
  CooLists la = direct ? CooLists() : alloc_lists(env, na), lb = alloc_lists(env, nb);
  us_status st = env.status;
  if (st == US_OK && n > 0) {
    US_LAUNCH(env, "node_split", 20.0 * n + 12.0 * n, node_split_kernel, ceil_div<int64_t>(n, 256), 256,
              (const uint64_t *)skey, (const float *)sval, (const int32_t *)keep, (const int32_t *)pos_a, n, ks, key_a,
              val_a, la, lb);
    st = env.status;
  }
  if (st == US_OK) {
    if (direct) {
      st = emit_blocked(env, pa, da, coo.nrows, coo.ncols, ks, key_a, val_a, na, flags, oa);
    } else {
      us_coo ca{coo.nrows, coo.ncols, na, la.r, la.c, la.v};
      st = convert_with_plan(env, ca, pa, da, oa);
    }
  }
  if (st == US_OK) {
    us_coo cb{coo.nrows, coo.ncols, nb, lb.r, lb.c, lb.v};
    st = convert_with_plan(env, cb, pb, db, ob);
  }
  env.sync();
  free_lists(env, la);
  free_lists(env, lb);
  return st;
}

us_status decompose_impl(Env &env, const us_coo &coo, const us_format_desc &da, const us_format_desc &db,
                         const us_predicate &pred, us_formatted **oa, us_formatted **ob) {
  *oa = *ob = nullptr;
  us_status s = validate_coo(coo);
  if (s != US_OK) return s;
  Plan pa, pb;
  if (!match_desc(da, &pa) || !match_desc(db, &pb)) return US_ERR_UNSUPPORTED_DESC;
  if ((pa.pattern == P_ELL && pa.swapped) || (pb.pattern == P_ELL && pb.swapped)) return US_ERR_UNSUPPORTED_DESC;
  if (pred.ngroup == 2) {
    // groups that are the nodes of a blocked layout: (d0/b, d1-d0) of Figure 3c, or the blocks (d0/bh, d1/bw)
    // of the BELL/COO case study (Section 7.2.2: a threshold on the entries of each block)
    Plan pg;
    int64_t bh, bw;
    if (pred.kind != US_P_SUM_GE_ABS || !tile(pred.group[0], US_E_DIV, 0, &bh)) return US_ERR_UNSUPPORTED_DESC;
    if (aff(pred.group[1], -1, 1)) { pg.pattern = P_BDIA; pg.bh = bh; pg.bw = 1; }
    else if (tile(pred.group[1], US_E_DIV, 1, &bw)) { pg.pattern = P_BCSR; pg.bh = bh; pg.bw = bw; }
    else return US_ERR_UNSUPPORTED_DESC;
    s = decompose_blocked(env, coo, pa, da, pb, db, pg, pred.abs, oa, ob);
    if (s == US_OK && !env.ok()) s = env.status;
    if (s != US_OK) {
      if (*oa) { free_formatted(env, *oa); *oa = nullptr; }
      if (*ob) { free_formatted(env, *ob); *ob = nullptr; }
    }
    return s;
  }
  if (pred.ngroup != 1) return US_ERR_UNSUPPORTED_DESC;
  const us_expr &ge = pred.group[0];
  int gkind = aff(ge, -1, 1) ? G_DIAG : aff(ge, 1, 0) ? G_ROW : aff(ge, 0, 1) ? G_COL : -1;
  if (gkind < 0) return US_ERR_UNSUPPORTED_DESC;
  if (pred.kind == US_P_SUM_GE_ABS || pred.kind == US_P_SUM_GE_FRAC_OF_CAPACITY) {
    if (pred.kind == US_P_SUM_GE_FRAC_OF_CAPACITY && (pred.den <= 0 || pred.num < 0)) return US_ERR_SHAPE;
    s = decompose_sum(env, coo, pa, da, pb, db, pred, gkind, oa, ob);
  } else if (pred.kind == US_P_RANK_LT_ABS || pred.kind == US_P_RANK_LT_PERCENTILE) {
    if (gkind != G_ROW) return US_ERR_UNSUPPORTED_DESC;
    if (pred.kind == US_P_RANK_LT_PERCENTILE && (pred.den <= 0 || pred.num < 0 || pred.num > pred.den)) return US_ERR_SHAPE;
    if (pred.kind == US_P_RANK_LT_ABS && pred.abs < 0) return US_ERR_SHAPE;
    s = decompose_rank(env, coo, pa, da, pb, db, pred, oa, ob);
  } else {
    return US_ERR_UNSUPPORTED_DESC;
  }
  if (s == US_OK && !env.ok()) s = env.status;
  if (s != US_OK) {
    if (*oa) { free_formatted(env, *oa); *oa = nullptr; }
    if (*ob) { free_formatted(env, *ob); *ob = nullptr; }
  }
  return s;
}

}  // namespace us
