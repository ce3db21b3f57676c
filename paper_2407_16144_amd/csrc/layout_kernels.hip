// Kernels of lp_create (and of an engine that re-blocks its last LPs) that
// never run in a solver step: validation of device-resident input, the
// explicit transpose K^T, column slicing, the sort keys of column-sorted
// blocks and groups and the gathers that apply a sorted permutation.
// Included by engine.hip after kernels.hip (shared types from halp_types.h).

namespace halp {

// dst = src narrowed to int32 (row pointers given as int64); *bad = 1 when an
// entry is negative or above 2^31 - 1 (that entry is written as 0)
__global__ void narrow_row_ptr_kernel(const int64_t* src, int32_t* dst, int64_t n, int* bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t v = src[i];
  if (v < 0 || v > (int64_t)INT32_MAX) {
    atomicOr(bad, 1);
    dst[i] = 0;
  } else {
    dst[i] = (int32_t)v;
  }
}

// ends[k] = first and last row pointer of LP k
__global__ void row_ends_kernel(const LpInput* in, int count, int2* ends) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < count) ends[k] = make_int2(in[k].rp[0], in[k].rp[in[k].m]);
}

// Validation of device-resident LPs, `parts` workgroups each (one launch and
// one answer for all of them; one LP after the other cost a batch of 128
// 10 ms in launches and round trips).  flags[k]: 1 bad row pointers, 2
// column out of range or not increasing, 4 non-finite value, 8 non-finite
// objective or right-hand side, 16 bad bounds.
// Entries: column in range and strictly above the previous entry's unless the
// entry starts its row (found by a binary search of the row pointers: the
// last row whose start is at or before it), finite value.  The search stays
// within rp[0..m] whatever the row pointers hold; invalid row pointers have
// a flag of their own.
__global__ __launch_bounds__(kThreads) void validate_lps_kernel(const LpInput* in, int parts, int* flags) {
  const LpInput p = in[blockIdx.x / parts];
  const int64_t first = (int64_t)(blockIdx.x % parts) * kThreads + threadIdx.x, step = (int64_t)parts * kThreads;
  int bad = 0;
  if (first == 0 && (p.rp[0] != 0 || p.rp[p.m] != p.nnz)) bad |= 1;
  for (int64_t r = first; r < p.m; r += step) {
    if (p.rp[r + 1] < p.rp[r] || p.rp[r] < 0 || p.rp[r + 1] > p.nnz) bad |= 1;
    if (!isfinite(p.rhs[r])) bad |= 8;
  }
  if (p.m > 0) {
    for (int64_t e = first; e < p.nnz; e += step) {
      const int64_t c = p.ci[e];
      if (c < 0 || c >= p.n) bad |= 2;
      if (!isfinite(p.val[e])) bad |= 4;
      if (e == 0) continue;
      int64_t lo = 0, hi = p.m;
      while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if ((int64_t)p.rp[mid] <= e) lo = mid; else hi = mid - 1;
      }
      if ((int64_t)p.rp[lo] != e && c <= (int64_t)p.ci[e - 1]) bad |= 2;
    }
  }
  for (int64_t i = first; i < p.n; i += step) {
    if (!isfinite(p.c[i])) bad |= 8;
    const double a = p.lb[i], b = p.ub[i];
    if (isnan(a) || isnan(b) || a > b || a == INFINITY || b == -INFINITY) bad |= 16;
  }
  if (bad) atomicOr(flags + blockIdx.x / parts, bad);
}

// Device-resident LPs into the engine's spaces: row pointers and columns
// become space positions, and the factors are 1.
__global__ __launch_bounds__(kThreads) void load_lps_kernel(const LpInput* in, int parts, int32_t* K_rp, int32_t* K_ci,
                                                            double* K_v, double* q, double* c, double* l, double* u,
                                                            double* Dr, double* Dc) {
  const LpInput p = in[blockIdx.x / parts];
  const int64_t first = (int64_t)(blockIdx.x % parts) * kThreads + threadIdx.x, step = (int64_t)parts * kThreads;
#pragma unroll 4
  for (int64_t e = first; e < p.nnz; e += step) {
    K_ci[p.nz0 + e] = (int32_t)(p.ci[e] + p.col0);
    K_v[p.nz0 + e] = p.val[e];
  }
  for (int64_t r = first; r <= p.m; r += step) {
    K_rp[p.row0 + r] = (int32_t)(p.rp[r] + p.nz0);
    Dr[p.row0 + r] = 1.0;
    if (r < p.m) q[p.row0 + r] = p.rhs[r];
  }
  for (int64_t j = first; j <= p.n; j += step) {
    Dc[p.col0 + j] = 1.0;
    if (j < p.n) {
      c[p.col0 + j] = p.c[j];
      l[p.col0 + j] = p.lb[j];
      u[p.col0 + j] = p.ub[j];
    }
  }
}

__global__ void shift_copy_kernel(int32_t* dst, const int32_t* src, int64_t n, int64_t add) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (int32_t)(src[i] + add);
}

__global__ void iota_kernel(int32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int32_t)i;
}

// rowid[e - z0] = row, for every entry of the rows in the dual schedule
__global__ __launch_bounds__(kThreads) void row_ids_kernel(const Blk* sched, const int32_t* rp,
                                                           int64_t z0, int32_t* rowid) {
  const Blk b = sched[blockIdx.x];
  const int nrows = b.r1 - b.r0;
  const int G = (blk_kind(b) == BK_LONG) ? kThreads : group_size(nrows);
  const int lane = threadIdx.x & (G - 1);
  for (int base = 0; base < nrows; base += kThreads / G) {
    const int r = base + threadIdx.x / G;
    if (r >= nrows) continue;
    const int row = b.r0 + r;
    const int p1 = rp[row + 1];
    for (int e = rp[row] + lane; e < p1; e += G) rowid[e - z0] = row;
  }
}

// cnt[(r - r0) * kSlices + s] = entries of row r whose column lies in slice s
// of the gathered range [c0, c0 + len)
__global__ void slice_count_kernel(const int32_t* rp, const int32_t* ci, int64_t r0, int64_t nrows,
                                   int64_t c0, int64_t len, int nsl, int32_t* cnt) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrows) return;
  int32_t c[kGroupSlices];
  for (int q = 0; q < kGroupSlices; ++q) c[q] = 0;
  for (int32_t e = rp[r0 + r]; e < rp[r0 + r + 1]; ++e) {
    const int q = (int)(((int64_t)(ci[e] - c0) * nsl) / len);
    c[q] += 1;
  }
  for (int q = 0; q < nsl; ++q) cnt[r * nsl + q] = c[q];
}

// Scatter row r's entries to their slice-major positions: dst[(r - r0) *
// kSlices + s] is the first position of row r's slice-s entries.
template <class V>
__global__ void slice_scatter_kernel(const int32_t* rp, const int32_t* ci, const V* val, const double* v64,
                                     int64_t r0, int64_t nrows, int64_t c0, int64_t len, const int32_t* dst,
                                     int32_t* ci_out, V* val_out, double* v64_out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrows) return;
  int32_t d[kSlices];
  for (int q = 0; q < kSlices; ++q) d[q] = dst[r * kSlices + q];
  for (int32_t e = rp[r0 + r]; e < rp[r0 + r + 1]; ++e) {
    const int q = (int)(((int64_t)(ci[e] - c0) * kSlices) / len);
    const int32_t p = d[q]++;
    ci_out[p] = ci[e];
    val_out[p] = val[e];
    if (v64_out) v64_out[p] = v64[e];
  }
}

// cnt[g * nsl + q] += entries of group g (rows [gstart[g], gstart[g + 1]) of
// the LP) in column slice q, over the row-major tiles: counted in LDS (a tile
// has at most as many groups as rows), then added up.
__global__ __launch_bounds__(kThreads) void group_count_kernel(const Blk* tiles, const int32_t* rp, const int32_t* ci,
                                                               const int32_t* gstart, int ngroups, int64_t r0,
                                                               int64_t c0, int64_t len, int nsl, int32_t* cnt) {
  __shared__ int32_t s_rp[kMaxRows];
  __shared__ int32_t s_g[kMaxRows];  // the row's group
  __shared__ int32_t s_first[kGroupSlices + 1];
  __shared__ int32_t s_cnt[kMaxRows * kGroupSlices];
  const Blk b = tiles[blockIdx.x];
  const int nrows = b.r1 - b.r0;
  if (nrows == 0) return;
  for (int r = threadIdx.x; r < nrows; r += kThreads) {
    const int32_t row = (int32_t)(b.r0 + r - r0);
    int lo = 0, up = ngroups - 1;  // the last group that starts at or before the row
    while (lo < up) {
      const int mid = (lo + up + 1) >> 1;
      if (gstart[mid] <= row) lo = mid; else up = mid - 1;
    }
    s_rp[r] = rp[b.r0 + r];
    s_g[r] = lo;
  }
  if ((int)threadIdx.x <= nsl) s_first[threadIdx.x] = (int32_t)((threadIdx.x * len + nsl - 1) / nsl);
  __syncthreads();
  const int g0 = s_g[0], words = (s_g[nrows - 1] - g0 + 1) * nsl;
  for (int i = threadIdx.x; i < words; i += kThreads) s_cnt[i] = 0;
  __syncthreads();
#pragma unroll 4
  for (int k = threadIdx.x; k < b.pn; k += kThreads) {
    const int32_t e = b.p0 + k;
    int lo = 0, up = words > nsl ? nrows - 1 : 0;  // (one group: any row of it)
    while (lo < up) {
      const int mid = (lo + up + 1) >> 1;
      if (s_rp[mid] <= e) lo = mid; else up = mid - 1;
    }
    const int32_t c = (int32_t)(ci[e] - c0);
    int q = 0;
    for (int i = 1; i < nsl; ++i) q += c >= s_first[i];
    atomicAdd(&s_cnt[(s_g[lo] - g0) * nsl + q], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < words; i += kThreads)
    if (s_cnt[i] > 0) atomicAdd(&cnt[(int64_t)g0 * nsl + i], s_cnt[i]);
}

// Sorted groups, step 1: for every entry of the row-major tiles, its
// (group, slice) block in the high word of a 64-bit key, (column - first
// column of the slice) << rb | (row - first row of the group) in the low word,
// and its position.  Group g holds rows [gstart[g], gstart[g + 1]) of the LP.
// One thread per entry (coalesced reads and writes, its row found among the
// tile's row starts in LDS); with one thread per row and positions counted per
// (row, slice) before it, 500k x 2M took 7.9 ms here and 32 MB of counts
// through the host, instead of 0.9 ms.
__global__ __launch_bounds__(kThreads) void group_keys_kernel(const Blk* tiles, const int32_t* rp, const int32_t* ci,
                                                              const int32_t* gstart, int ngroups, int64_t r0,
                                                              int64_t z0, int64_t c0, int64_t len, int nsl, int rb,
                                                              uint64_t* key, int32_t* src) {
  __shared__ int32_t s_rp[kMaxRows];
  __shared__ int32_t s_blk[kMaxRows];  // the row's first (group, slice) block
  __shared__ int32_t s_loc[kMaxRows];  // the row in its group
  __shared__ int32_t s_first[kGroupSlices + 1];
  const Blk b = tiles[blockIdx.x];
  const int nrows = b.r1 - b.r0;
  for (int r = threadIdx.x; r < nrows; r += kThreads) {
    const int32_t row = (int32_t)(b.r0 + r - r0);
    int lo = 0, up = ngroups - 1;  // the last group that starts at or before the row
    while (lo < up) {
      const int mid = (lo + up + 1) >> 1;
      if (gstart[mid] <= row) lo = mid; else up = mid - 1;
    }
    s_rp[r] = rp[b.r0 + r];
    s_blk[r] = lo * nsl;
    s_loc[r] = row - gstart[lo];
  }
  if ((int)threadIdx.x <= nsl) s_first[threadIdx.x] = (int32_t)((threadIdx.x * len + nsl - 1) / nsl);
  __syncthreads();
  for (int k = threadIdx.x; k < b.pn; k += kThreads) {
    const int32_t e = b.p0 + k;
    int lo = 0, up = nrows - 1;
    while (lo < up) {
      const int mid = (lo + up + 1) >> 1;
      if (s_rp[mid] <= e) lo = mid; else up = mid - 1;
    }
    const int32_t c = (int32_t)(ci[e] - c0);
    int q = 0;
    for (int i = 1; i < nsl; ++i) q += c >= s_first[i];
    key[e - z0] = ((uint64_t)(uint32_t)(s_blk[lo] + q) << 32) | (((uint32_t)(c - s_first[q]) << rb) | (uint32_t)s_loc[lo]);
    src[e - z0] = e;
  }
}

// Column-sorting of plain blocks, step 1: for every entry of every block of
// the given LPs, a 64-bit sort key with the block's index in the high word
// and, in the low word, (column - b.rp_off) << rb | (row - b.r0) for a
// BK_SORTED block, the entry's index in the block for any other (so that it
// stays in place), and the entry's position.  The key arrays hold the LPs one
// after the other: position p is at p + b.gid there.
__global__ __launch_bounds__(kThreads) void block_keys_kernel(const Blk* blks, const int32_t* rp,
                                                              const int32_t* ci, uint64_t* key, int32_t* src) {
  __shared__ int32_t s_rp[kSortRowsPlain];
  const Blk b = blks[blockIdx.x];
  const uint64_t hi = (uint64_t)blockIdx.x << 32;
  const int64_t at = (int64_t)b.p0 + b.gid;
  if (blk_kind(b) == BK_SORTED) {
    // one thread per entry; its row is the last of the block's rows that
    // starts at or before it (empty rows share the next row's start), found
    // among the row starts in LDS
    const int rb = blk_rowbits(b);
    const int nrows = b.r1 - b.r0;
    for (int r = threadIdx.x; r < nrows; r += kThreads) s_rp[r] = rp[b.r0 + r];
    __syncthreads();
    for (int k = threadIdx.x; k < b.pn; k += kThreads) {
      const int32_t e = b.p0 + k;
      int lo = 0, up = nrows - 1;
      while (lo < up) {
        const int mid = (lo + up + 1) >> 1;
        if (s_rp[mid] <= e) lo = mid; else up = mid - 1;
      }
      key[at + k] = hi | (((uint32_t)(ci[e] - b.rp_off) << rb) | (uint32_t)lo);
      src[at + k] = e;
    }
  } else {
    for (int e = threadIdx.x; e < b.pn; e += kThreads) {
      key[at + e] = hi | (uint32_t)e;
      src[at + e] = b.p0 + e;
    }
  }
}

// Re-blocking of products stored in column-sorted blocks: every entry of
// the old blocks `old` (which cover the LPs' entries) gets the key of its
// place in the new blocks, where[r + b.rp_off] = (new block index, row in that
// block) of the row at space position r.  BK_SORTED entries read their row and
// column back from the packed key (the column relative to the LP's first
// column, which the new blocks share); other entries (rows that stay in a
// block of their own) keep their order.  blk_nsl(b): row bits of the new
// blocks; p + b.gid: place of position p in the key arrays.
__global__ __launch_bounds__(kThreads) void reblock_keys_kernel(const Blk* old, const int2* where, const int32_t* ci,
                                                                uint64_t* key, int32_t* src) {
  const Blk b = old[blockIdx.x];
  const int64_t at = (int64_t)b.p0 + b.gid;
  if (blk_kind(b) == BK_SORTED) {
    const int rb = blk_rowbits(b), rb_new = blk_nsl(b);
    const uint32_t rmask = (1u << rb) - 1u;
    for (int e = threadIdx.x; e < b.pn; e += kThreads) {
      const uint32_t w = (uint32_t)ci[b.p0 + e];
      const int2 t = where[b.r0 + (int64_t)(w & rmask) + b.rp_off];
      key[at + e] = ((uint64_t)(uint32_t)t.x << 32) | (((w >> rb) << rb_new) | (uint32_t)t.y);
      src[at + e] = b.p0 + e;
    }
  } else {
    const uint64_t hi = (uint64_t)(uint32_t)where[b.r0 + (int64_t)b.rp_off].x << 32;
    for (int e = threadIdx.x; e < b.pn; e += kThreads) {
      key[at + e] = hi | (uint32_t)e;
      src[at + e] = b.p0 + e;
    }
  }
}

// Step 2 (after the keys are sorted): the entries of every BK_SORTED block
// take the low words of the sorted keys as packed column indices and the FP64
// values of the entries they came from (staged in v_tmp, in the order of the
// key arrays).
__global__ __launch_bounds__(kThreads) void sorted_block_gather_kernel(const Blk* blks, const uint64_t* key,
                                                                       const int32_t* src, const double* v64,
                                                                       int32_t* ci_out, double* v_tmp) {
  const Blk b = blks[blockIdx.x];
  const int64_t at = (int64_t)b.p0 + b.gid;
  for (int e = threadIdx.x; e < b.pn; e += kThreads) {
    ci_out[b.p0 + e] = (int32_t)(uint32_t)key[at + e];
    v_tmp[at + e] = v64[src[at + e]];
  }
}

// Step 3: the staged values take their places, also as the compute type's
// (val is v64 itself where that is FP64).
template <class V>
__global__ __launch_bounds__(kThreads) void sorted_block_store_kernel(const Blk* blks, const double* v_tmp, V* val,
                                                                      double* v64) {
  const Blk b = blks[blockIdx.x];
  const int64_t at = (int64_t)b.p0 + b.gid;
  for (int e = threadIdx.x; e < b.pn; e += kThreads) {
    const double v = v_tmp[at + e];
    v64[b.p0 + e] = v;
    if constexpr (sizeof(V) != 8) val[b.p0 + e] = (V)v;
  }
}

// Sorted groups, step 2 (after the keys are sorted): off[s] = first position
// of block s, for s in [0, nseg].
__global__ void segment_offsets_kernel(const uint64_t* key, int64_t nnz, int nseg, int32_t* off) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s > nseg) return;
  int64_t lo = 0, up = nnz;
  while (lo < up) {
    const int64_t mid = (lo + up) >> 1;
    if ((int64_t)(key[mid] >> 32) < s) lo = mid + 1; else up = mid;
  }
  off[s] = (int32_t)lo;
}

// Sorted groups, step 3: entry p takes the sorted key as its packed column
// index and the FP64 value of the entry it came from.
__global__ void sorted_gather_kernel(const uint64_t* key, const int32_t* src, const double* v64, int64_t nnz,
                                     int32_t* ci_out, double* v_out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nnz) return;
  ci_out[p] = (int32_t)(uint32_t)key[p];
  v_out[p] = v64[src[p]];
}

template <class V>
__global__ void transpose_gather_kernel(const int32_t* perm, const int32_t* rowid, const V* val,
                                        int64_t z0, int64_t nnz, int32_t* kt_ci, V* kt_val) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nnz) return;
  const int32_t e = perm[p];
  kt_ci[z0 + p] = rowid[e];
  kt_val[z0 + p] = val[z0 + e];
}

// kt_rp[j] = z0 + #{sorted keys < j - c0} for space positions j in [c0, c1]
// (keys: columns relative to c0)
__global__ void transpose_rowptr_kernel(const uint32_t* keys, int64_t nnz, int64_t z0, int64_t c0,
                                        int64_t c1, int32_t* kt_rp) {
  const int64_t j = c0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j > c1) return;
  int64_t lo = 0, hi = nnz;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)keys[mid] + c0 < j) lo = mid + 1; else hi = mid;
  }
  kt_rp[j] = (int32_t)(z0 + lo);
}

template __global__ void sorted_block_store_kernel<double>(const Blk*, const double*, double*, double*);
template __global__ void sorted_block_store_kernel<float>(const Blk*, const double*, float*, double*);
template __global__ void slice_scatter_kernel<double>(const int32_t*, const int32_t*, const double*,
                                                      const double*, int64_t, int64_t, int64_t, int64_t,
                                                      const int32_t*, int32_t*, double*, double*);
template __global__ void slice_scatter_kernel<float>(const int32_t*, const int32_t*, const float*,
                                                     const double*, int64_t, int64_t, int64_t, int64_t,
                                                     const int32_t*, int32_t*, float*, double*);
template __global__ void transpose_gather_kernel<double>(const int32_t*, const int32_t*, const double*,
                                                         int64_t, int64_t, int32_t*, double*);

}  // namespace halp
