// The sum query (Section 4.1.2) over diagonals, rows or columns as a histogram, what it selects, the DIA layout
// (Devectorize/Fill/Vectorize: entries scattered into a pre-filled slab, no sort), and the decomposition
// driven by that query (Section 6, the decompose op).
#include "convert_internal.h"
#include "device.h"

namespace us {

// ------------------------------------------------------------------ Sum query (group histogram) and DIA
// Groups supported by the groupBy map of the sum query: diagonals (d1-d0), rows (d0), columns (d1).

__device__ __forceinline__ uint32_t group_bin(int gkind, uint32_t r, uint32_t c, uint32_t nrows) {
  return gkind == G_DIAG ? c - r + (nrows - 1) : (gkind == G_ROW ? r : c);
}

// One counter per group.  A matrix whose entries sit on a handful of diagonals would send
// almost every update to the same few counters, and same-address HBM atomics cost ~20 ns apiece
// on this part, so updates are combined in a small LDS hash table first (LDS takes 64 lanes
// hitting one slot in about as many cycles; electing one lane per bin with ballots beforehand was
// slower).  A workgroup walks several tiles; after each it flushes and frees the slots that stayed
// cold and keeps the hot ones, so a hot counter gets one HBM atomic per workgroup (at most GH_GRID of
// them), not one per tile.  Freeing a slot may cut a probe chain; the bin then simply takes a second
// slot, and counts add up all the same.
// Large workgroups, because the launch is short of them, and no more than are resident at once (two per CU): with 768 of
// them a third starts when the others have ended, on a half-empty part.  256 threads x 16 entries and 768 workgroups /
// 1024 x 4 and 768 / 1024 x 4 and 512, us: 14.8 M entries on seven diagonals and a few beside them 92 / 62 / 53; rows of a
// sorted list of 16.5 M entries 149 / 126 / 108; diagonals, rows, columns of 16.8 M uniformly spread entries, where every
// entry is an atomic of its own, 649, 649, 645 / 634, 634, 635 / 633, 636, 636; 41 k entries 26 / 12 / 12.  With the next tile's
// entries on their way while a tile is counted (their loads waited behind the barriers of the one before) the first is 45 -> 35.  Rows of an
// unsorted list whose first rows hold hundreds of thousands of entries and the many next ones some thousands, too few of
// a tile to stay in the table: 2039 / 2069 / 2070, bound by atomics that meet on those counters.
constexpr int GH_T = 1024, GH_IPT = 4, GH_TILE = GH_T * GH_IPT, GH_SLOTS = 1024, GH_PROBES = 8, GH_GRID = 512;
static_assert(GH_GRID <= ONE_COUNTER_GRID, "hot counters");
constexpr uint32_t GH_HOT = 64;

__global__ __launch_bounds__(GH_T) void group_hist_kernel(const int32_t *row, const int32_t *col, int64_t n,
                                                         int gkind, uint32_t nrows, uint32_t ncols, uint32_t *count,
                                                         Flags *flags) {
  __shared__ uint32_t s_key[GH_SLOTS];
  __shared__ uint32_t s_cnt[GH_SLOTS];
  for (int i = threadIdx.x; i < GH_SLOTS; i += GH_T) { s_key[i] = 0xFFFFFFFFu; s_cnt[i] = 0; }
  __syncthreads();
  bool bad = false;
  uint32_t r[GH_IPT], c[GH_IPT];
  auto load = [&](int64_t base) {
#pragma unroll
    for (int k = 0; k < GH_IPT; ++k) {
      const int64_t i = base + k * GH_T + threadIdx.x;
      r[k] = i < n ? (uint32_t)row[i] : 0u; c[k] = i < n ? (uint32_t)col[i] : 0u;
    }
  };
  const int64_t stride = (int64_t)gridDim.x * GH_TILE;
  load((int64_t)blockIdx.x * GH_TILE);
  for (int64_t base = (int64_t)blockIdx.x * GH_TILE; base < n; base += stride) {
    uint32_t bin[GH_IPT];
#pragma unroll
    for (int k = 0; k < GH_IPT; ++k) {
      bin[k] = 0xFFFFFFFFu;
      if (base + k * GH_T + threadIdx.x < n) {
        if (r[k] >= nrows || c[k] >= ncols) bad = true;
        else bin[k] = group_bin(gkind, r[k], c[k], nrows);
      }
    }
    load(base + stride);   // on its way while this tile is counted
#pragma unroll 1
    for (int k = 0; k < GH_IPT; ++k) {
      const uint32_t b = bin[k];
      if (b == 0xFFFFFFFFu) continue;
      uint32_t h = (b * 2654435761u) >> 22;
      bool done = false;
      for (int probe = 0; probe < GH_PROBES && !done; ++probe) {
        uint32_t old = s_key[h];   // a bin that is already in the table (the hot ones, soon) needs no CAS
        if (old == 0xFFFFFFFFu) old = atomicCAS(&s_key[h], 0xFFFFFFFFu, b);
        if (old == 0xFFFFFFFFu || old == b) { atomicAdd(&s_cnt[h], 1u); done = true; }
        h = (h + 1) & (GH_SLOTS - 1);
      }
      if (!done) atomicAdd(&count[b], 1u);
    }
    __syncthreads();
    const bool last = base + stride >= n;
    for (int i = threadIdx.x; i < GH_SLOTS; i += GH_T) {
      const uint32_t c = s_cnt[i];
      if (s_key[i] != 0xFFFFFFFFu && (last || c < GH_HOT)) {
        if (c) atomicAdd(&count[s_key[i]], c);
        s_key[i] = 0xFFFFFFFFu; s_cnt[i] = 0;
      }
    }
    __syncthreads();
  }
  if (bad) flags->index_range = 1;
}

// Which groups go to part A, and their numbers in order: counted per tile of groups, the tiles' counts scanned, then every
// group's number written over its count (-1: the group stays out).  The predicate is evaluated in both passes: the counts
// are read twice, and nothing in between is written (4.2 M diagonals: flags, their scan, the numbers and the offsets in
// arrays and launches of their own took 50 us, this 24).
struct GroupRule { int gkind, pkind; int64_t num, den, thr, nrows, ncols; };   // pkind < 0: every non-empty group (plain conversion)
__device__ __forceinline__ bool group_goes(const GroupRule &q, int64_t g, uint32_t cnt) {
  if (cnt == 0) return false;
  if (q.pkind < 0) return true;
  if (q.pkind == US_P_SUM_GE_ABS) return (int64_t)cnt >= q.thr;
  int64_t cap;
  if (q.gkind == G_DIAG) {
    const int64_t off = g - (q.nrows - 1);
    const int64_t hi = q.nrows < q.ncols - off ? q.nrows : q.ncols - off, lo = off < 0 ? -off : 0;
    cap = hi > lo ? hi - lo : 0;
  } else cap = q.gkind == G_ROW ? q.ncols : q.nrows;
  return q.den * (int64_t)cnt >= q.num * cap;
}

constexpr int GS_T = 256, GS_IPT = 8, GS_TILE = GS_T * GS_IPT;
// partial[t] = groups of tile t that go, entries in them
__global__ __launch_bounds__(GS_T) void group_reduce_kernel(const uint32_t *count, int64_t nbins, GroupRule q, uint2 *partial) {
  __shared__ uint32_t s_wave[GS_T / 64 + 1];
  const int64_t base = (int64_t)blockIdx.x * GS_TILE;
  uint32_t cnt[GS_IPT], go = 0, in = 0, groups, entries;
#pragma unroll
  for (int k = 0; k < GS_IPT; ++k) {
    const int64_t g = base + k * GS_T + threadIdx.x;
    cnt[k] = g < nbins ? count[g] : 0u;
  }
#pragma unroll
  for (int k = 0; k < GS_IPT; ++k)
    if (group_goes(q, base + k * GS_T + threadIdx.x, cnt[k])) { ++go; in += cnt[k]; }
  block_exclusive_sum<GS_T>(go, s_wave, &groups);
  block_exclusive_sum<GS_T>(in, s_wave, &entries);
  if (threadIdx.x == 0) partial[blockIdx.x] = make_uint2(groups, entries);
}

// off (or null): the offsets of the diagonals that go, in order
// far: where the first workgroup leaves how many of 256 pairs of neighbours in the list lie more than DIA_FAR rows apart,
// or null
constexpr uint32_t DIA_FAR = 256;
__global__ __launch_bounds__(GS_T) void group_number_kernel(uint32_t *count, int64_t nbins, GroupRule q, const uint2 *partial,
                                                           int32_t *off, const int32_t *row, int64_t n, int32_t *far) {
  __shared__ uint32_t s_wave[GS_T / 64 + 1];
  static_assert(GS_IPT == 8, "two 16-byte vectors per thread");
  const int64_t g0 = (int64_t)blockIdx.x * GS_TILE + (int64_t)threadIdx.x * GS_IPT;   // (the counts start at 256 bytes)
  const bool whole = g0 + GS_IPT <= nbins;
  uint32_t cnt[GS_IPT], go = 0, total;
  if (whole) {
    const uint4 a = *reinterpret_cast<const uint4 *>(count + g0), b = *reinterpret_cast<const uint4 *>(count + g0 + 4);
    cnt[0] = a.x; cnt[1] = a.y; cnt[2] = a.z; cnt[3] = a.w; cnt[4] = b.x; cnt[5] = b.y; cnt[6] = b.z; cnt[7] = b.w;
  } else {
#pragma unroll
    for (int k = 0; k < GS_IPT; ++k) cnt[k] = g0 + k < nbins ? count[g0 + k] : 0u;
  }
  bool goes[GS_IPT];
#pragma unroll
  for (int k = 0; k < GS_IPT; ++k) { goes[k] = group_goes(q, g0 + k, cnt[k]); go += goes[k]; }
  int32_t at = (int32_t)(block_exclusive_sum<GS_T>(go, s_wave, &total) + partial[blockIdx.x].x), id[GS_IPT];
#pragma unroll
  for (int k = 0; k < GS_IPT; ++k) {
    id[k] = -1;
    if (goes[k]) {
      if (off) off[at] = (int32_t)(g0 + k - (q.nrows - 1));
      id[k] = at++;
    }
  }
  if (whole) {
    *reinterpret_cast<int4 *>(count + g0) = make_int4(id[0], id[1], id[2], id[3]);
    *reinterpret_cast<int4 *>(count + g0 + 4) = make_int4(id[4], id[5], id[6], id[7]);
  } else {
#pragma unroll
    for (int k = 0; k < GS_IPT; ++k)
      if (g0 + k < nbins) count[g0 + k] = (uint32_t)id[k];
  }
  if (far && blockIdx.x == 0) {
    __shared__ uint32_t s_far;
    if (threadIdx.x == 0) s_far = 0;
    __syncthreads();
    const int64_t i = (int64_t)threadIdx.x * (n - 1) / 256;   // n > 1: i + 1 < n
    const uint32_t step = (uint32_t)row[i + 1] - (uint32_t)row[i];
    const uint64_t away = __ballot(step + DIA_FAR > 2 * DIA_FAR);
    if (lane_id() == 0) atomicAdd(&s_far, (uint32_t)__popcll(away));
    __syncthreads();
    if (threadIdx.x == 0) *far = (int32_t)s_far;
  }
}
// what has to be there before the entries are dealt out: the offsets in the result's own array, counters at zero
__global__ __launch_bounds__(256) void dia_begin_kernel(const int32_t *off, int64_t ndiag, int32_t *out, uint32_t *zero, int64_t nzero) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < ndiag) out[i] = off[i];
  if (i < nzero) zero[i] = 0u;
}

// One pass over the COO list that sends every entry to its part of a decomposition.
//   TO_SLAB: entries of flagged diagonals go straight into the DIA slab val[k*L + i]
//            (Devectorize/Fill/Vectorize).  A duplicate coordinate shows as fewer occupied slots
//            than entries, counted afterwards.  Occupied = not the fill pattern: the slab starts
//            out filled with DIA_EMPTY (a NaN bit pattern no computation produces) and a finishing
//            pass counts and zeroes what is left of it, which costs two streaming passes over the
//            slab instead of one more scattered byte store per entry (a byte map of marked slots,
//            the form used when an input value happens to carry that very bit pattern);
//   otherwise they are appended to list A.  Entries of unflagged groups are appended to list B.
// Appends reserve space once per workgroup (one atomic per list), so order inside a list is
// arbitrary; each part is put into canonical order by its conversion.
constexpr int SP_T = 512, SP_IPT = 16, SP_TILE = SP_T * SP_IPT;
constexpr uint32_t DIA_EMPTY = 0x7FC5A5A5u;

template <bool TO_SLAB>
__global__ __launch_bounds__(SP_T) void split_kernel(const int32_t *row, const int32_t *col, const float *val,
                                                    int64_t n, int gkind, uint32_t nrows, const int32_t *gmap,
                                                    int64_t L, int by_col, float *slab, uint8_t *slotmap,
                                                    CooLists la, CooLists lb, int32_t *cursors, Flags *flags) {
  __shared__ uint32_t s_wave[SP_T / 64 + 1];
  __shared__ int32_t s_base[2];
  const int64_t base = (int64_t)blockIdx.x * SP_TILE;
  uint32_t r[SP_IPT], c[SP_IPT];
  float v[SP_IPT];
  int32_t g[SP_IPT];
#pragma unroll
  for (int k = 0; k < SP_IPT; ++k) {
    int64_t i = base + k * SP_T + threadIdx.x;
    r[k] = c[k] = 0; v[k] = 0.f;
    if (i < n) { r[k] = (uint32_t)row[i]; c[k] = (uint32_t)col[i]; v[k] = val[i]; }
  }
  uint32_t na = 0, nb = 0;
#pragma unroll
  for (int k = 0; k < SP_IPT; ++k) {
    int64_t i = base + k * SP_T + threadIdx.x;
    g[k] = -2;  // no entry
    if (i < n) {
      g[k] = gmap[group_bin(gkind, r[k], c[k], nrows)];
      if (g[k] >= 0) ++na; else ++nb;
    }
  }
  uint32_t ta, tb;
  uint32_t pa = (!TO_SLAB && la.r) ? block_exclusive_sum<SP_T>(na, s_wave, &ta) : 0u;
  uint32_t pb = lb.r ? block_exclusive_sum<SP_T>(nb, s_wave, &tb) : 0u;
  if (threadIdx.x == 0) {
    s_base[0] = (!TO_SLAB && la.r && ta) ? atomicAdd(&cursors[0], (int32_t)ta) : 0;
    s_base[1] = (lb.r && tb) ? atomicAdd(&cursors[1], (int32_t)tb) : 0;
  }
  __syncthreads();
  pa += s_base[0]; pb += s_base[1];
#pragma unroll
  for (int k = 0; k < SP_IPT; ++k) {
    if (g[k] >= 0) {
      if (TO_SLAB) {
        int64_t slot = (int64_t)g[k] * L + (by_col ? c[k] : r[k]);
        slab[slot] = v[k];
        if (slotmap) slotmap[slot] = 1;
        else if (__float_as_uint(v[k]) == DIA_EMPTY) flags->retry = RETRY_DIA_MARKS;
      } else if (la.r) {
        la.r[pa] = (int32_t)r[k]; la.c[pa] = (int32_t)c[k]; la.v[pa] = v[k]; ++pa;
      }
    } else if (g[k] == -1 && lb.r) {
      lb.r[pb] = (int32_t)r[k]; lb.c[pb] = (int32_t)c[k]; lb.v[pb] = v[k]; ++pb;
    }
  }
}

// A slab beyond the L2s in two passes instead: the entries go to bins of 2^DB_SHIFT or more neighbouring slots first, as
// {slot inside the bin, value}, and every bin is then put together in LDS and written whole, empty slots included, while
// its occupied slots are counted in a bit map: no fill, no second look at the slab and no value that could be taken for
// an empty slot.  A bin holds as many entries as it has slots; what does not fit (only duplicates can make it so) is
// dropped, and the count of occupied slots says so.  One workgroup per CU walks its tiles and has the next tile's entries on
// their way while it writes one (without: 1200 workgroups of one tile each, whose phases follow one another, 135 -> 128 us).
// The first pass is bound by its device atomics, one per tile and bin: 14.7 M entries, 896 bins, tiles of 4096 / 8192 / 12,288
// entries 332 / 153 / 134 us; with a count of its own per workgroup first, and 256 workgroups, 144.  The second writes at
// 4.6 TB/s.
constexpr int64_t DIA_BINNED = 3 << 19;   // slots
constexpr int DB_T = 1024, DB_IPT = 12, DB_TILE = DB_T * DB_IPT, DB_BINS = 2048, DB_GRID = 256;

__global__ __launch_bounds__(DB_T) void dia_bin_kernel(const int32_t *row, const int32_t *col, const float *val, int64_t n,
                                                       uint32_t nrows, const int32_t *gmap, int64_t L, int by_col, int shift,
                                                       uint2 *rec, uint32_t *filled, CooLists lb, int32_t *cursors) {
  __shared__ uint2 s_rec[DB_TILE];
  __shared__ uint16_t s_bin[DB_TILE];
  __shared__ uint32_t s_cnt[DB_BINS];    // entries of the tile per bin, then where they start in the tile
  __shared__ uint32_t s_goff[DB_BINS];   // place of the tile's entries in the bin, minus their start in the tile
  __shared__ uint32_t s_wave[DB_T / 64 + 1];
  __shared__ int32_t s_base;
  constexpr int PER = DB_BINS / DB_T;
  const int tid = threadIdx.x;
  uint32_t r[DB_IPT], c[DB_IPT];
  float v[DB_IPT];
  auto load = [&](int64_t base) {
    const uint32_t in_tile = base < n ? (uint32_t)min(n - base, (int64_t)DB_TILE) : 0u;
    const int32_t *rows = row + base, *cols = col + base;
    const float *vals = val + base;
#pragma unroll
    for (int k = 0; k < DB_IPT; ++k) {
      const uint32_t i = k * DB_T + tid;
      r[k] = c[k] = 0; v[k] = 0.f;
      if (i < in_tile) { r[k] = (uint32_t)rows[i]; c[k] = (uint32_t)cols[i]; v[k] = vals[i]; }
    }
  };
  const int64_t stride = (int64_t)gridDim.x * DB_TILE;
  load((int64_t)blockIdx.x * DB_TILE);
  for (int64_t base = (int64_t)blockIdx.x * DB_TILE; base < n; base += stride) {
    const uint32_t in_tile = (uint32_t)min(n - base, (int64_t)DB_TILE);
    uint32_t kept = 0, rest = 0;   // bit k: entry k belongs to a flagged diagonal (r: its slot, c: its place in the bin) / to none
#pragma unroll
    for (int q = 0; q < PER; ++q) s_cnt[q * DB_T + tid] = 0;   // (last read before the barrier that the tile before was written behind)
#pragma unroll
    for (int k = 0; k < DB_IPT; ++k) {
      if (k * DB_T + tid < in_tile) {
        const int32_t g = gmap[group_bin(G_DIAG, r[k], c[k], nrows)];
        if (g >= 0) { r[k] = (uint32_t)((int64_t)g * L + (by_col ? c[k] : r[k])); kept |= 1u << k; }   // below 2^31
        else rest |= 1u << k;
      }
    }
    const uint32_t nb = __popc(rest);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < DB_IPT; ++k)
      if (kept >> k & 1u) c[k] = atomicAdd(&s_cnt[r[k] >> shift], 1u);
    uint32_t tb, ta, cnt[PER], sum = 0;
    uint32_t pb = block_exclusive_sum<DB_T>(nb, s_wave, &tb);   // (its barriers close the counts)
    if (tid == 0) s_base = lb.r && tb ? atomicAdd(&cursors[1], (int32_t)tb) : 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) { cnt[q] = s_cnt[tid * PER + q]; sum += cnt[q]; }
    uint32_t run = block_exclusive_sum<DB_T>(sum, s_wave, &ta);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t b = tid * PER + q;
      s_cnt[b] = run;
      s_goff[b] = (cnt[q] ? atomicAdd(&filled[b], cnt[q]) : 0u) - run;   // (bins past the slab's hold nothing)
      run += cnt[q];
    }
    __syncthreads();
    pb += (uint32_t)s_base;
#pragma unroll
    for (int k = 0; k < DB_IPT; ++k) {
      if (kept >> k & 1u) {
        const uint32_t b = r[k] >> shift, pos = s_cnt[b] + c[k];
        s_rec[pos] = make_uint2(r[k] & ((1u << shift) - 1u), __float_as_uint(v[k]));
        s_bin[pos] = (uint16_t)b;
      } else if ((rest >> k & 1u) && lb.r) {
        lb.r[pb] = (int32_t)r[k]; lb.c[pb] = (int32_t)c[k]; lb.v[pb] = v[k]; ++pb;
      }
    }
    __syncthreads();
    load(base + stride);   // on its way while this tile is written
    for (uint32_t i = tid; i < ta; i += DB_T) {
      const uint32_t b = s_bin[i], at = s_goff[b] + i;
      if (at < 1u << shift) rec[((size_t)b << shift) + at] = s_rec[i];
    }
  }
}

template <int SHIFT>
__global__ __launch_bounds__(DB_T) void dia_image_kernel(const uint2 *rec, const uint32_t *filled, float *slab, int64_t nslots,
                                                         int32_t *out) {
  constexpr uint32_t S = 1u << SHIFT;
  __shared__ uint32_t s_img[S];
  __shared__ uint32_t s_bits[S / 32];
  __shared__ uint32_t s_wave[DB_T / 64 + 1];
  const int tid = threadIdx.x;
  const uint32_t b = blockIdx.x, n = min(filled[b], S);
  for (uint32_t i = tid; i < S / 4; i += DB_T) reinterpret_cast<uint4 *>(s_img)[i] = make_uint4(0, 0, 0, 0);
  for (uint32_t i = tid; i < S / 32; i += DB_T) s_bits[i] = 0;
  __syncthreads();
  const uint2 *src = rec + ((size_t)b << SHIFT);
#pragma unroll 4
  for (uint32_t i = tid; i < n; i += DB_T) {
    const uint2 e = src[i];
    s_img[e.x] = e.y;
    atomicOr(&s_bits[e.x >> 5], 1u << (e.x & 31u));
  }
  __syncthreads();
  const int64_t first = (int64_t)b << SHIFT;
  float4 *dst = reinterpret_cast<float4 *>(slab + first);
  const uint32_t nv = (uint32_t)min((int64_t)S / 4, (nslots - first + 3) / 4);   // (the allocation is padded to whole vectors)
  for (uint32_t i = tid; i < nv; i += DB_T) dst[i] = reinterpret_cast<const float4 *>(s_img)[i];
  uint32_t cnt = 0, total;
  for (uint32_t i = tid; i < S / 32; i += DB_T) cnt += __popc(s_bits[i]);
  block_exclusive_sum<DB_T>(cnt, s_wave, &total);
  if (tid == 0 && total) atomicAdd(out, (int32_t)total);
}

// occupied slots of a slab that started out as DIA_EMPTY; what is still empty becomes +0.0
__global__ __launch_bounds__(256) void dia_finish_kernel(uint4 *slab4, int64_t nvec, int64_t nslots, int32_t *out) {
  __shared__ uint32_t s_wave[256 / 64 + 1];
  uint32_t cnt = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * 256) {
    uint4 w = slab4[i];
    uint32_t *e = reinterpret_cast<uint32_t *>(&w);
    bool changed = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i * 4 + k >= nslots) continue;   // the allocation is padded to whole vectors
      if (e[k] == DIA_EMPTY) { e[k] = 0u; changed = true; } else ++cnt;
    }
    if (changed) slab4[i] = w;
  }
  uint32_t total;
  block_exclusive_sum<256>(cnt, s_wave, &total);
  if (threadIdx.x == 0 && total) atomicAdd(out, (int32_t)total);
}

// number of marked slots (bytes are 0 or 1; the map is padded with zeros to a multiple of 16)
__global__ __launch_bounds__(256) void count_marks_kernel(const uint4 *m, int64_t nvec, int32_t *out) {
  __shared__ uint32_t s_wave[256 / 64 + 1];
  uint32_t cnt = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * 256) {
    uint4 w = m[i];
    cnt += __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
  }
  uint32_t total;
  block_exclusive_sum<256>(cnt, s_wave, &total);
  if (threadIdx.x == 0 && total) atomicAdd(out, (int32_t)total);
}

CooLists alloc_lists(Env &env, int64_t n) {
  CooLists l;
  l.r = env.owned<int32_t>(n); l.c = env.owned<int32_t>(n); l.v = env.owned<float>(n);
  return l;
}
void free_lists(Env &env, CooLists &l) {
  env.free_raw(l.r); env.free_raw(l.c); env.free_raw(l.v);
  l = CooLists();
}

// number[g] = position of group g among those that go to part A, or -1 (in place of the counts); off: see group_number_kernel
struct GroupMap { const int32_t *number; int32_t *off; };

// histogram of the groups, and the number of every group that goes to part A (flags->scalar[0] groups, [1] entries in them)
size_t group_temp_bytes(int64_t nbins) {
  return 2 * Env::granule(4 * (size_t)nbins) + Env::granule(8 * (size_t)ceil_div<int64_t>(nbins, GS_TILE)) +
         Env::granule(4 * (DB_BINS + 2)) + 8 * Env::granule(256);
}
static int64_t group_bins(const us_coo &coo, int gkind) {
  return gkind == G_DIAG ? coo.nrows + coo.ncols - 1 : (gkind == G_ROW ? coo.nrows : coo.ncols);
}

static GroupMap group_map(Env &env, const us_coo &coo, int gkind, int pkind, int64_t num, int64_t den, int64_t thr, Flags *flags,
                          bool slab) {
  const int64_t nbins = group_bins(coo, gkind), ntile = ceil_div<int64_t>(nbins, GS_TILE), n = coo.nnz;
  GroupMap g{};
  uint32_t *count = env.temp<uint32_t>(nbins);
  if (slab) g.off = env.temp<int32_t>(nbins);
  uint2 *partial = env.temp<uint2>(ntile);
  if (!env.ok()) return g;
  fill_u32(env, count, nbins, 0);
  if (n > 0)
    US_LAUNCH(env, "group_hist", 8.0 * n, group_hist_kernel, std::min<int64_t>(ceil_div<int64_t>(n, GH_TILE), GH_GRID), GH_T, coo.row,
              coo.col, n, gkind, (uint32_t)coo.nrows, (uint32_t)coo.ncols, count, flags);
  const GroupRule q{gkind, pkind, num, den, thr, coo.nrows, coo.ncols};
  US_LAUNCH(env, "group_reduce", 4.0 * nbins, group_reduce_kernel, ntile, GS_T, (const uint32_t *)count, nbins, q, partial);
  scan_pairs(env, partial, ntile, &flags->scalar[0], &flags->scalar[1], false);
  US_LAUNCH(env, "group_number", 8.0 * nbins, group_number_kernel, ntile, GS_T, count, nbins, q, (const uint2 *)partial, g.off,
            coo.row, n, slab && n > 1 ? &flags->scalar[2] : (int32_t *)nullptr);
  g.number = (const int32_t *)count;
  return g;
}

// DIA of the diagonals that group_map has numbered.
// If `rest` is given, the entries of the unflagged diagonals are collected into it in the same
// pass (its arrays are allocated here; the caller owns them afterwards) and *nrest is their number.
// verify_later != null: the last read of the flags (coordinates in range, no value carrying the empty pattern, as
// many occupied slots as entries) is left to the caller, who enqueues more work first and then calls
// dia_verify with *verify_later: the host then waits once for both instead of twice.
struct DiaPending { Flags *flags = nullptr; int64_t na = 0; };

static us_status dia_verify(Env &env, const DiaPending &p) {
  Flags h{};
  if (!read_flags(env, p.flags, &h)) return env.status;
  if (flag_status(h) != US_OK) return flag_status(h);
  return h.scalar[3] != p.na ? US_ERR_DUPLICATE : US_OK;
}

static us_status dia_from_flags(Env &env, const us_coo &coo, const Plan &plan, const us_format_desc &desc,
                                Flags *flags, const GroupMap &g, us_formatted **out, CooLists *rest,
                                int64_t *nrest, DiaPending *verify_later = nullptr) {
  const int64_t n = coo.nnz;
  const int64_t L = plan.swapped ? coo.ncols : coo.nrows;
  Flags h{};
  if (!read_flags(env, flags, &h)) return env.status;
  if (flag_status(h) != US_OK) return flag_status(h);
  const int64_t ndiag = h.scalar[0], na = h.scalar[1];
  if (ndiag * L >= (1ll << 31)) return US_ERR_OVERFLOW;
  us_formatted *f = new us_formatted();
  f->desc = desc; f->pattern = P_DIA; f->swapped = plan.swapped;
  f->nrows = coo.nrows; f->ncols = coo.ncols; f->nnz = na;
  f->nlevels = 2;
  f->level[0].idx = env.owned<int32_t>(ndiag); f->level[0].nidx = ndiag;
  f->level[1].size = L;
  const int64_t nslab4 = ceil_div<int64_t>(ndiag * L, 4);
  f->val = env.owned<float>(nslab4 * 4); f->nval = ndiag * L; f->nmajor = ndiag;   // whole 16-byte vectors
  // Into bins first where the slab is beyond the caches of an XCD, mostly full, and the list in no order that keeps
  // neighbouring stores together; a list sorted by rows or by diagonals writes whole lines as it is.  Seven diagonals, stores
  // and finish / bins and images, us: in random order 1.1 M entries 37 / 36, 2.1 M 54 / 40, 4.9 M 94 / 65, 14.7 M 279 / 174,
  // 40 M 676 / 514; 14.7 M sorted by rows 109 / 184, by diagonals 87 / 216.
  const int64_t nslots = ndiag * L;
  const int shift = nslots <= (int64_t)DB_BINS << 14 ? 14 : 15;
  const bool binned = nslots >= DIA_BINNED && na >= nslots / 4 && nslots <= (int64_t)DB_BINS << 15 && h.scalar[2] > 128;
  const int64_t nbins_slab = ceil_div<int64_t>(nslots, 1ll << shift);
  const bool marks = env.dia_marks && !binned;
  const int64_t nvec = ceil_div<int64_t>(nslots, 16) + 1;
  uint8_t *slotmap = marks ? (uint8_t *)env.temp<uint4>(nvec) : nullptr;
  if (binned) env.reserve(Env::granule(4 * (DB_BINS + 2)) + Env::granule(((size_t)nbins_slab << shift) * sizeof(uint2)));
  uint32_t *counters = env.temp<uint32_t>(DB_BINS + 2);   // the lists' two, then the bins'
  uint32_t *filled = counters + 2;
  int32_t *cursors = (int32_t *)counters;
  uint2 *rec = binned ? env.temp<uint2>((size_t)nbins_slab << shift) : nullptr;
  CooLists lb;
  if (rest) { *nrest = n - na; lb = alloc_lists(env, n - na); *rest = lb; }
  if (!env.ok()) { free_formatted(env, f); return env.status; }
  if (!binned) fill_u32(env, (uint32_t *)f->val, nslots, marks ? 0u : DIA_EMPTY);
  if (marks) fill_u32(env, (uint32_t *)slotmap, nvec * 4, 0u);
  const int64_t ncounters = binned ? DB_BINS + 2 : 2;
  US_LAUNCH(env, "dia_begin", 8.0 * ndiag, dia_begin_kernel, ceil_div<int64_t>(std::max(ndiag, ncounters), 256), 256,
            (const int32_t *)g.off, ndiag, f->level[0].idx, counters, ncounters);
  if (binned) {
    US_LAUNCH(env, "dia_bin", 12.0 * n + 8.0 * na + 12.0 * (rest ? n - na : 0), dia_bin_kernel, std::min<int64_t>(ceil_div<int64_t>(n, DB_TILE), DB_GRID), DB_T,
              coo.row, coo.col, coo.val, n, (uint32_t)coo.nrows, g.number, L, plan.swapped ? 1 : 0, shift, rec,
              filled, lb, cursors);
    if (shift == 14) US_LAUNCH(env, "dia_image", 8.0 * na + 4.0 * nslots, dia_image_kernel<14>, nbins_slab, DB_T, (const uint2 *)rec, (const uint32_t *)filled, f->val, nslots, &flags->scalar[3]);
    else US_LAUNCH(env, "dia_image", 8.0 * na + 4.0 * nslots, dia_image_kernel<15>, nbins_slab, DB_T, (const uint2 *)rec, (const uint32_t *)filled, f->val, nslots, &flags->scalar[3]);
  } else if (n > 0)
    US_LAUNCH(env, "dia_split_scatter", 12.0 * n + 5.0 * na + 12.0 * (rest ? n - na : 0), (split_kernel<true>),
              ceil_div<int64_t>(n, SP_TILE), SP_T, coo.row, coo.col, coo.val, n, (int)G_DIAG, (uint32_t)coo.nrows,
              g.number, L, plan.swapped ? 1 : 0, f->val, slotmap, CooLists(), lb, cursors, flags);
  if (marks)
    US_LAUNCH(env, "count_marks", 1.0 * nslots, count_marks_kernel, one_counter_grid(nvec, 256), 256, (const uint4 *)slotmap, nvec, &flags->scalar[3]);
  else if (!binned && nslab4 > 0)
    US_LAUNCH(env, "dia_finish", 4.0 * nslots, dia_finish_kernel, one_counter_grid(nslab4, 256), 256, (uint4 *)f->val, nslab4, nslots, &flags->scalar[3]);
  if (verify_later) {
    verify_later->flags = flags; verify_later->na = na;
    if (!env.ok()) { free_formatted(env, f); return env.status; }
    *out = f;
    return US_OK;
  }
  const us_status st = dia_verify(env, DiaPending{flags, na});
  if (st != US_OK) { free_formatted(env, f); return st; }
  *out = f;
  return US_OK;
}


us_status convert_dia(Env &env, const us_coo &coo, const Plan &plan, const us_format_desc &desc,
                      Flags *flags, us_formatted **out) {
  const GroupMap g = group_map(env, coo, G_DIAG, -1, 0, 1, 0, flags, true);
  if (!env.ok()) return env.status;
  return dia_from_flags(env, coo, plan, desc, flags, g, out, nullptr, nullptr);
}

us_status decompose_sum(Env &env, const us_coo &coo, const Plan &pa, const us_format_desc &da, const Plan &pb,
                        const us_format_desc &db, const us_predicate &pred, int gkind, us_formatted **oa,
                        us_formatted **ob) {
  const bool slab = gkind == G_DIAG && pa.pattern == P_DIA;
  env.reserve(group_temp_bytes(group_bins(coo, gkind)));
  Flags *flags = new_flags(env);
  if (!env.ok()) return env.status;
  const GroupMap g = group_map(env, coo, gkind, pred.kind, pred.num, pred.den, pred.abs, flags, slab);
  if (!env.ok()) return env.status;
  const int64_t n = coo.nnz;
  CooLists la, lb;
  int64_t na = 0, nb = 0;
  us_status st;
  DiaPending pending;
  if (slab) {
    // part A goes straight into the slab while part B is collected, in one pass over the input; its flags are read
    // after part B's conversion has been enqueued (and has read its own): an input that fails them (a coordinate
    // out of range reaches no slab slot and no list; a duplicate is a slot written twice) is reported then
    st = dia_from_flags(env, coo, pa, da, flags, g, oa, &lb, &nb, &pending);
  } else {
    Flags h{};
    if (!read_flags(env, flags, &h)) return env.status;
    if (flag_status(h) != US_OK) return flag_status(h);
    na = h.scalar[1]; nb = n - na;
    la = alloc_lists(env, na); lb = alloc_lists(env, nb);
    int32_t *cursors = env.temp<int32_t>(2);
    st = env.status;
    if (st == US_OK) {
      fill_u32(env, (uint32_t *)cursors, 2, 0u);
      if (n > 0)
        US_LAUNCH(env, "split", 24.0 * n, (split_kernel<false>), ceil_div<int64_t>(n, SP_TILE), SP_T, coo.row, coo.col,
                  coo.val, n, gkind, (uint32_t)coo.nrows, g.number, (int64_t)0, 0, (float *)nullptr,
                  (uint8_t *)nullptr, la, lb, cursors, flags);
      st = env.status;
    }
    if (st == US_OK) {
      us_coo ca{coo.nrows, coo.ncols, na, la.r, la.c, la.v};
      st = convert_with_plan(env, ca, pa, da, oa);
    }
  }
  if (st == US_OK) {
    us_coo cb{coo.nrows, coo.ncols, nb, lb.r, lb.c, lb.v};
    st = convert_with_plan(env, cb, pb, db, ob);
  }
  if (pending.flags) {   // part A's own verdict comes first: part B may have failed only because of what it reports
    const us_status sa = dia_verify(env, pending);
    if (sa != US_OK) st = sa;
  }
  env.sync();
  free_lists(env, la);
  free_lists(env, lb);
  return st;
}

}  // namespace us
