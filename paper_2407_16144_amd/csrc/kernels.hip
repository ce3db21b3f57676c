// Device kernels of the restarted Halpern PDHG solver (gfx950 / CDNA4).
//
// One solver step is two launches over fixed workgroup schedules:
//   primal_step : y-gather SpMV over the rows of the explicit K^T, fused with
//                 the primal PDHG step, box projection and Halpern blend;
//   dual_step   : xbar-gather SpMV over the rows of K, fused with the dual
//                 step, cone projection and Halpern blend; at check, eval and
//                 residual steps the last workgroup of each LP (arrival
//                 counter) reduces that LP's block partial sums in a fixed
//                 order and runs its restart / termination controller.
// Column-sorted blocks of either product run in sorted_step; the products of
// large LPs in slice kernels (sorted_group_step), whose partial sums part_step
// finishes; small LPs run all steps of a chunk in one workgroup
// (resident_steps).
// The path is bandwidth bound (about 2 flop per 12 bytes of matrix), so there
// is no MFMA: the work is coalesced entry loads, gathers, LDS staging and
// wave64 shuffle reductions.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "halp_types.h"
#include "kernels.h"

namespace halp {

// ---------------------------------------------------------------------------
// reductions (fixed order: results do not depend on scheduling)
// ---------------------------------------------------------------------------

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sum of kNS per-thread values over the block; result valid in s_out[0..kNS).
template <int TPB = kThreads>
__device__ __forceinline__ void block_sum_ns(double (&v)[kNS], double (*s_red)[kNS], double* s_out) {
#pragma unroll
  for (int s = 0; s < kNS; ++s) v[s] = wave_sum(v[s]);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int s = 0; s < kNS; ++s) s_red[wave][s] = v[s];
  }
  __syncthreads();
  if (threadIdx.x < kNS) {
    double a = s_red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < TPB / 64; ++w) a += s_red[w][threadIdx.x];
    s_out[threadIdx.x] = a;
  }
  __syncthreads();
}

template <class T>
__device__ __forceinline__ T block_sum1(T v, double (*s_red)[kNS]) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) s_red[wave][0] = (double)v;
  __syncthreads();
  T a = (T)s_red[0][0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) a += (T)s_red[w][0];
  __syncthreads();
  return a;
}

// Fixed-order sum of nb rows of kNS partials; all threads call, result in s_out.
template <int TPB = kThreads>
__device__ void sum_partials(const double* part, int nb, double (*s_red)[kNS], double* s_out) {
  double v[kNS];
#pragma unroll
  for (int s = 0; s < kNS; ++s) v[s] = 0.0;
#pragma unroll 2
  for (int b = threadIdx.x; b < nb; b += TPB) {
#pragma unroll
    for (int s = 0; s < kNS; ++s) v[s] += part[(int64_t)b * kNS + s];
  }
  block_sum_ns<TPB>(v, s_red, s_out);
}

__device__ __forceinline__ int group_size(int nrows) {
  // largest power of two G <= 64 with nrows * G <= kThreads (at least 1)
  int g = 64;
  while (g > 1 && g * nrows > kThreads) g >>= 1;
  return g;
}

// Workgroup barrier that orders LDS only: outstanding global loads (prefetched
// epilogue operands) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// block SpMV: row sums of NV gathered vectors for the rows of one block.
// rp points at the block's row pointers (rp[0..nrows], entry positions);
// the entry range [b.p0, b.p0 + b.pn) comes with the descriptor, so entry
// loads start without waiting for the row pointers.
// Stream blocks (<= NB entries, <= kMaxRows rows): entries are loaded once,
// coalesced, into registers; per gathered vector the products go to LDS and
// groups of G lanes reduce each row.  Long blocks (one row): strided loop
// with four accumulators and a block reduction.
// Result: s_rsum[a][r - b.r0].
// ---------------------------------------------------------------------------

template <class T, int NB = kPlainNB>
struct TileRegs {
  static constexpr int EPT = NB / kThreads;
  int cidx[EPT];
  T v[EPT];
  T p[EPT];      // products with a gathered vector
  int rpv = 0;   // row pointer t of the block (relative to p0), t = thread
  int rpv2 = 0;  // row pointer kThreads (thread 0, blocks of kThreads rows)
};

// Products with the step's usual gathered vector, issued before the LP
// state is read (the state only decides whether they are used).
template <class T, int NB>
__device__ __forceinline__ void spec_products(const Blk& b, const T* __restrict__ src, TileRegs<T, NB>& R) {
  if (blk_kind(b) != BK_STREAM) return;
#pragma unroll
  for (int k = 0; k < TileRegs<T, NB>::EPT; ++k) {
    const int e = (int)threadIdx.x + k * kThreads;
    if (e < b.pn) R.p[k] = R.v[k] * src[R.cidx[k]];
  }
}

// Loads a stream block's entries (coalesced) and row pointers into
// registers; independent of the step mode, so callers issue it before
// reading the LP state.  rp points at the block's first row pointer.
template <bool NT, class V>
__device__ __forceinline__ V ld_entry(const V* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <bool NT, class T, int NB>
__device__ __forceinline__ void load_tile_as(const Blk& b, const int32_t* __restrict__ rp,
                                             const int32_t* __restrict__ ci, const T* __restrict__ val,
                                             TileRegs<T, NB>& R) {
  const int t = threadIdx.x;
  const int nrows = b.r1 - b.r0;
#pragma unroll
  for (int k = 0; k < TileRegs<T, NB>::EPT; ++k) {
    const int e = t + k * kThreads;
    if (e < b.pn) {
      R.cidx[k] = ld_entry<NT>(ci + b.p0 + e);
      R.v[k] = ld_entry<NT>(val + b.p0 + e);
    }
  }
  if (t <= nrows) R.rpv = rp[t] - b.p0;
  if (nrows == kThreads && t == 0) R.rpv2 = rp[kThreads] - b.p0;
}

// Loads a stream block's entries (coalesced) and row pointers into
// registers; independent of the step mode, so callers issue it before
// reading the LP state.  rp points at the block's first row pointer.
template <class T, int NB>
__device__ __forceinline__ void load_tile(const Blk& b, const int32_t* __restrict__ rp,
                                          const int32_t* __restrict__ ci, const T* __restrict__ val,
                                          TileRegs<T, NB>& R) {
  if (blk_kind(b) != BK_STREAM) return;
  if (blk_nt(b)) load_tile_as<true, T, NB>(b, rp, ci, val, R);
  else load_tile_as<false, T, NB>(b, rp, ci, val, R);
}

// Strided partial sums of one long row (entries [p0, p0 + pn)).
template <bool NT, class T>
__device__ __forceinline__ T long_row_sum(int p0, int pn, const int32_t* __restrict__ ci,
                                          const T* __restrict__ val, const T* __restrict__ src) {
  T acc0 = (T)0, acc1 = (T)0;
  int e = threadIdx.x;
  for (; e + kThreads < pn; e += 2 * kThreads) {
    const int c0 = ld_entry<NT>(ci + p0 + e), c1 = ld_entry<NT>(ci + p0 + e + kThreads);
    const T v0 = ld_entry<NT>(val + p0 + e), v1 = ld_entry<NT>(val + p0 + e + kThreads);
    acc0 += v0 * src[c0];
    acc1 += v1 * src[c1];
  }
  if (e < pn) acc0 += ld_entry<NT>(val + p0 + e) * src[ld_entry<NT>(ci + p0 + e)];
  return acc0 + acc1;
}

// One gathered vector: row sums into out[r - b.r0] (LDS).
template <class T, int NB>
__device__ void block_spmv1(const Blk& b, const int32_t* __restrict__ ci,
                            const T* __restrict__ val, const TileRegs<T, NB>& R, const T* __restrict__ src,
                            T* s_prod, T* out, int* s_rp, double (*s_red)[kNS], T scale = (T)1,
                            bool have_products = false) {
  const int tid = threadIdx.x;
  const int nrows = b.r1 - b.r0;
  const int p0 = b.p0, pn = b.pn;
  if (blk_kind(b) == BK_LONG) {
    T t = wave_sum(blk_nt(b) ? long_row_sum<true>(p0, pn, ci, val, src) : long_row_sum<false>(p0, pn, ci, val, src));
    if ((tid & 63) == 0) s_red[tid >> 6][0] = (double)t;
    lds_barrier();
    if (tid == 0) {
      T u = (T)s_red[0][0];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) u += (T)s_red[w][0];
      out[0] = u * scale;
    }
    lds_barrier();
    return;
  }
  constexpr int EPT = TileRegs<T, NB>::EPT;
  if (tid <= nrows) s_rp[tid] = R.rpv;
  if (nrows == kThreads && tid == 0) s_rp[kThreads] = R.rpv2;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int e = tid + k * kThreads;
    if (e < pn) s_prod[e] = have_products ? R.p[k] : R.v[k] * src[R.cidx[k]];
  }
  lds_barrier();
  const int G = group_size(nrows);
  const int lane = tid & (G - 1);
  const int rpb = kThreads / G;  // rows per pass
  for (int base = 0; base < nrows; base += rpb) {
    const int r = base + tid / G;
    T acc = (T)0;
    if (r < nrows) {
      const int q1 = s_rp[r + 1];
      for (int q = s_rp[r] + lane; q < q1; q += G) acc += s_prod[q];
    }
    for (int off = G >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0 && r < nrows) out[r] = acc * scale;
  }
  lds_barrier();
}

// NV gathered vectors, one after the other over the same register tile
template <class T, int NV, int NB>
__device__ __forceinline__ void block_spmv_regs(const Blk& b,
                                                const int32_t* __restrict__ ci, const T* __restrict__ val,
                                                const TileRegs<T, NB>& R, const T* __restrict__ s0,
                                                const T* __restrict__ s1, const T* __restrict__ s2, T* s_prod,
                                                T (*s_rsum)[kMaxRows], int* s_rp, double (*s_red)[kNS],
                                                T scale0 = (T)1) {
  block_spmv1<T, NB>(b, ci, val, R, s0, s_prod, s_rsum[0], s_rp, s_red, scale0);
  if constexpr (NV > 1) block_spmv1<T, NB>(b, ci, val, R, s1, s_prod, s_rsum[1], s_rp, s_red);
  if constexpr (NV > 2) block_spmv1<T, NB>(b, ci, val, R, s2, s_prod, s_rsum[2], s_rp, s_red);
}

template <class T, int NV>
__device__ __forceinline__ void block_spmv(const Blk& b, const int32_t* __restrict__ rp,
                                           const int32_t* __restrict__ ci, const T* __restrict__ val,
                                           const T* __restrict__ s0, const T* __restrict__ s1,
                                           const T* __restrict__ s2, T* s_prod, T (*s_rsum)[kMaxRows],
                                           int* s_rp, double (*s_red)[kNS], T scale0 = (T)1) {
  TileRegs<T, kPlainNB> R;
  load_tile<T, kPlainNB>(b, rp, ci, val, R);
  block_spmv_regs<T, NV, kPlainNB>(b, ci, val, R, s0, s1, s2, s_prod, s_rsum, s_rp, s_red, scale0);
}

// ---------------------------------------------------------------------------
// step modes
// ---------------------------------------------------------------------------

// Device memory that no wave of the running kernel writes before the block has
// read it (schedules, the step counter, an LP's state, which the last of its
// blocks updates): uniform loads of it are scalar.
template <class V>
using cptr = const __attribute__((address_space(4))) V*;
// Device memory, vector loads.
template <class V>
using gptr = const __attribute__((address_space(1))) V*;

// A block's descriptor, loaded whole.
typedef int BlkWords __attribute__((ext_vector_type(8)));
__device__ __forceinline__ Blk load_blk(cptr<BlkWords> p) {
  const BlkWords w = *p;
  return Blk{w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]};
}

// Mode of step g for one LP.  Checks fall at inner counters k = C, 2C, ...
// of an epoch (k = g - kbase); the controller keeps the step index of the
// next one in next_check.
__device__ __forceinline__ int mode_of(int status, int phase, int64_t kbase, int64_t next, int64_t g) {
  if (status != ST_RUNNING) return M_SKIP;
  if (phase == PH_EVAL) return M_EVAL;
  if (phase == PH_RESID) return M_RESID;
  if (g < kbase) return M_SKIP;
  if (g == next) return M_CHECK;
  return M_NORMAL;
}
__device__ __forceinline__ int step_mode(const InstState& S, int64_t g) {
  return mode_of(S.status, S.phase, S.kbase, S.next_check, g);
}
// The same in a step kernel: the four fields are loaded together (the asm ties
// them), in one round trip instead of one per test.
__device__ __forceinline__ int step_mode(cptr<InstState> S, int64_t g) {
  int status = S->status, phase = S->phase;
  int64_t kbase = S->kbase, next = S->next_check;
  asm("" : "+s"(status), "+s"(phase), "+s"(kbase), "+s"(next));
  return mode_of(status, phase, kbase, next, g);
}

template <class T>
__device__ __forceinline__ T clampT(T v, T lo, T hi) {
  return fmin(fmax(v, lo), hi);
}

// projection of a direction onto the recession cone of [l, u]
template <class T>
__device__ __forceinline__ T rec_proj(T d, bool lf, bool uf) {
  return (lf && uf) ? (T)0 : lf ? fmax(d, (T)0) : uf ? fmin(d, (T)0) : d;
}

// ---------------------------------------------------------------------------
// primal step (rows of K^T = variables)
// ---------------------------------------------------------------------------

// The entries of one column-sorted block (a plain BK_SORTED block or one
// (group, slice) block of a sorted-group product) as a software pipeline: TPB
// threads take U entries each per batch; a batch's packed indices and values
// are loaded D batches before its gathers, and its gathers are issued one
// batch before its products are added into the LDS row sums.  Consecutive
// entries gather nearby elements of the vector, so the lanes of one gather
// share cache lines.  The row sums are FP64 LDS words whatever the compute
// type (products in the compute type; ds_add_f64 measured 1.8x faster than
// ds_add_f32 on these scattered adds), added by LDS atomics: the order of the
// additions within a row is not fixed (the last bits of a sum can differ from
// run to run).
//
// Loads start at the block's first entry rounded down to 32 entries (whole
// 128-byte lines per wave: neighbouring waves otherwise both wait for the
// line they share) and go through buffer descriptors that end with the block:
// a position past the end reads index 0 and value 0.  What lies outside the
// block is added into kSpareWords words behind the row sums (one per lane), so
// the loop has no per-entry branch.
template <class T, int TPB, int U, int D>
struct SortedStream {
  static constexpr int NS = D + 2;  // batches in registers
  static_assert(D >= 1, "a batch is loaded before it is gathered");
  static constexpr int BT = TPB * U;
  __amdgpu_buffer_rsrc_t rk, rv;
  int lo, hi, rb;
  bool nt;  // non-temporal loads
  uint32_t k[NS][U];
  T v[NS][U];

  template <int AUX>
  __device__ __forceinline__ void load_as(int i, int slot) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = (uint32_t)(i * BT + u * TPB) + threadIdx.x;
      k[slot][u] = __builtin_amdgcn_raw_buffer_load_b32(rk, (int)(e * 4u), 0, AUX);
      if constexpr (sizeof(T) == 8)
        v[slot][u] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rv, (int)(e * 8u), 0, AUX));
      else
        v[slot][u] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rv, (int)(e * 4u), 0, AUX));
    }
  }
  // the first batches, issued before anything else the block waits for
  __device__ __forceinline__ void open(const Blk& b, const int32_t* ci, const T* val) {
    lo = b.p0 & 31;
    hi = lo + b.pn;
    rb = blk_rowbits(b);
    nt = blk_nt(b);
    rk = __builtin_amdgcn_make_buffer_rsrc((void*)(ci + (b.p0 - lo)), 0, (int)((uint32_t)hi * 4u), 0x00020000);
    rv = __builtin_amdgcn_make_buffer_rsrc((void*)(val + (b.p0 - lo)), 0,
                                           (int)((uint32_t)hi * (uint32_t)sizeof(T)), 0x00020000);
    if (nt) {
#pragma unroll
      for (int d = 0; d <= D; ++d) load_as<2>(d, d);
    } else {
#pragma unroll
      for (int d = 0; d <= D; ++d) load_as<0>(d, d);
    }
  }
  // slice widths keep the byte offset of a gather below 2^32 (kSortColBits)
  __device__ __forceinline__ void gather(const T* srcb, int slot, T (&g)[U]) const {
#pragma unroll
    for (int u = 0; u < U; ++u)
      g[u] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(srcb) +
                                         (size_t)(uint32_t)((k[slot][u] >> rb) * (uint32_t)sizeof(T)));
  }
  // products with srcb (the vector from the block's first column on) added
  // into the row sums s_row[row << rs] (rs > 0: this lane's copy), which the
  // block has cleared; s_row[spare]: this lane's word for what lies outside the
  // block
  __device__ __forceinline__ void sum(const T* srcb, double* s_row, int spare, int rs = 0) {
    if (nt) sum_as<2>(srcb, s_row, spare, rs);
    else sum_as<0>(srcb, s_row, spare, rs);
  }
  template <int AUX>
  __device__ __forceinline__ void sum_as(const T* srcb, double* s_row, int spare, int rs) {
    const uint32_t rmask = (1u << rb) - 1u;
    const int nb = (hi + BT - 1) / BT;
    // positions before the block's first entry hold another block's columns
    if ((int)threadIdx.x < lo) k[0][0] = 0;
    T g[2][U];
    gather(srcb, 0, g[0]);
    constexpr int RND = NS % 2 ? 2 * NS : NS;  // batches per round: register slots repeat
    for (int i = 0; i < nb; i += RND) {
#pragma unroll
      for (int d = 0; d < RND; ++d) {
        if (i + d >= nb) break;
        gather(srcb, (d + 1) % NS, g[(d + 1) & 1]);
        load_as<AUX>(i + d + D + 1, (d + D + 1) % NS);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = (i + d) * BT + u * TPB + (int)threadIdx.x;
          const int row = (int)((k[d % NS][u] & rmask) << rs);
          atomicAdd(&s_row[e >= lo && e < hi ? row : spare], (double)(v[d % NS][u] * g[d & 1][u]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
};

// Clears the LDS row sums of a block (a barrier has to follow).
__device__ __forceinline__ void clear_rows(double* s_row, int words, int tpb) {
  for (int r = threadIdx.x; r < words; r += tpb) s_row[r] = 0.0;
}

// One variable's part of a primal step (rows of K^T): j is its space
// position, kty its row sum (K^T y, or K^T yT at an eval step, where g1 and
// g2 are K^T cy1 and K^T cy2; at a residual step the caller passes T(z) as
// xo and x0j and K^T yT as kty).  Adds the check / eval / residual terms of
// the variable to ps.  Returns xbar (eval step: nothing of use).
template <class T>
__device__ __forceinline__ T primal_row(const IterArgs<T>& A, const InstState& S, int mode, int64_t g,
                                           int64_t j, T cj, T lj, T uj, T xo, T x0j, T kty, T g1, T g2,
                                           double (&ps)[kNS]) {
  const bool resid = (mode == M_RESID);
  const bool lf = isfinite(lj), uf = isfinite(uj);
  if (mode == M_EVAL) {
    const T g0 = kty;
    A.ktyp[j] = g0;
    const double dc = A.Dc[j];
    const double r = (double)cj - (double)g0;
    const double lam = (lf && uf) ? r : lf ? fmax(r, 0.0) : uf ? fmin(r, 0.0) : 0.0;
    const double rd = (r - lam) / dc;
    ps[0] += rd * rd;
    ps[1] += (lf ? (double)lj * fmax(lam, 0.0) : 0.0) - (uf ? (double)uj * fmax(-lam, 0.0) : 0.0);
#pragma unroll
    for (int a = 1; a <= 2; ++a) {
      const double gg = (double)(a == 1 ? g1 : g2);
      double sv = 0.0, vv = 0.0;
      if (gg > 0.0) {
        if (uf) sv = (double)uj * gg; else vv = gg / dc;
      } else if (gg < 0.0) {
        if (lf) sv = (double)lj * gg; else vv = -gg / dc;
      }
      ps[2 * a] += sv;
      ps[2 * a + 1] += vv * vv;
    }
    return (T)0;
  }
  const T tau = (T)S.tau;
  const T xp = clampT<T>(xo - tau * (cj - kty), lj, uj);
  const T xb = (T)2 * xp - xo;
  const int64_t k = g - S.kbase;
  T xn, xc = xp;  // next iterate; check candidate (T(z), or the epoch average)
  if (S.avg) {
    // plain PDHG step; running sum of z^{n,0..k+1} (restarted at k = 0)
    const T xsum = (k == 0 ? xo : A.xs[j]) + xp;
    A.xs[j] = xsum;
    xn = xp;
    if (mode == M_CHECK) xc = xsum / (T)(k + 2);
  } else {
    const double w = (double)(k + 1) / (double)(k + 2);
    const T xh = S.reflect ? xb : xp;
    xn = (T)w * xh + (T)(1.0 - w) * x0j;
  }
  A.xbar[j] = xb;
  A.x[j] = xn;
  if (resid) {
    A.x0[j] = xo;
    const double d = (double)xo - (double)xp;
    ps[0] += d * d;
  } else if (mode == M_CHECK) {
    A.xT[j] = xc;
    const double d = (double)xo - (double)xp;
    const double ad = (double)xc - (double)x0j;
    const T d1 = rec_proj<T>(xp - xo, lf, uf);
    const T d2 = rec_proj<T>(xo - x0j, lf, uf);
    A.cx1[j] = d1;
    A.cx2[j] = d2;
    ps[0] += d * d;
    ps[1] += ad * ad;
    ps[2] += (double)cj * (double)xc;
    ps[3] += (double)cj * (double)d1;
    ps[4] += (double)cj * (double)d2;
    const uint8_t act = (lf && xp == lj) ? 1 : (uf && xp == uj) ? 2 : 0;
    const uint8_t was = A.actx[j];
    A.actx[j] = act;
    ps[5] += (was != 255 && was != act) ? 1.0 : 0.0;
  }
  return xb;
}

template <class T>
__global__ __launch_bounds__(kThreads) void primal_step(IterArgs<T> A, int step) {
  __shared__ T s_prod[Tile<T>::NB];
  __shared__ T s_rsum[3][kMaxRows];
  __shared__ int s_rp[kMaxRows + 1];
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];

  const Blk b = A.schedP[blockIdx.x];
  if (blk_kind(b) == BK_PAD) return;
  const int nrows = b.r1 - b.r0;
  const int t = threadIdx.x;
  const bool own = t < nrows;
  const int64_t j = (int64_t)b.r0 + (own ? t : 0);
  // entries and epilogue operands are loaded before the LP state is read,
  // so their latency overlaps the state loads (none depends on the mode)
  TileRegs<T, kPlainNB> R;
  load_tile<T, kPlainNB>(b, A.KT_rp + b.r0, A.KT_ci, A.KT_v, R);
  spec_products<T, kPlainNB>(b, A.y, R);
  T cj = 0, lj = 0, uj = 0, xo = 0, x0j = 0, kty = 0;
  if (own) {
    cj = A.c[j];
    lj = A.l[j];
    uj = A.u[j];
    xo = A.x[j];
    x0j = A.x0[j];
  }
  const InstState& S = A.st[b.inst];
  const int64_t g = *A.gbase + step;
  const int mode = step_mode(S, g);
  if (mode == M_SKIP) return;
  const bool resid = (mode == M_RESID);
  if (resid && own) {
    xo = A.xT[j];
    x0j = xo;
    kty = A.ktyp[j];
  }
  if (mode == M_EVAL) {
    block_spmv_regs<T, 3, kPlainNB>(b, A.KT_ci, A.KT_v, R, A.yT, A.cy1, A.cy2, s_prod, s_rsum, s_rp, s_red);
  } else if (!resid) {
    block_spmv1<T, kPlainNB>(b, A.KT_ci, A.KT_v, R, A.y, s_prod, s_rsum[0], s_rp, s_red, (T)1, true);
  }

  double ps[kNS];
#pragma unroll
  for (int s = 0; s < kNS; ++s) ps[s] = 0.0;
  if (own) {
    const bool eval = (mode == M_EVAL);
    primal_row<T>(A, S, mode, g, j, cj, lj, uj, xo, x0j, resid ? kty : s_rsum[0][t],
                  eval ? s_rsum[1][t] : (T)0, eval ? s_rsum[2][t] : (T)0, ps);
  }
  if (mode != M_NORMAL) {
    block_sum_ns(ps, s_red, s_out);
    if (t < kNS) A.partP[(int64_t)b.gid * kNS + t] = s_out[t];
  }
}

// Partial row sums of one column slice of a sliced row group (written to
// spart for the step kernel of the same step to add up).  dual = 1: rows of
// K gathering xbar (or xT, cx1, cx2 at an eval step); dual = 0: rows of K^T
// gathering y (or yT, cy1, cy2).
template <class T, bool dual, int NB>
__device__ __forceinline__ void slice_body(const IterArgs<T>& A, int step) {
  __shared__ T s_prod[NB];
  __shared__ T s_rsum[3][kMaxRows];
  __shared__ int s_rp[kMaxRows + 1];
  __shared__ double s_red[kThreads / 64][kNS];
  const Blk b = (dual ? A.schedDS : A.schedPS)[blockIdx.x];
  if (blk_kind(b) == BK_PAD) return;
  const int32_t* rp = (dual ? A.brpK : A.brpKT) + b.rp_off;
  const int32_t* ci = dual ? A.K_ci : A.KT_ci;
  const T* val = dual ? A.K_v : A.KT_v;
  TileRegs<T, NB> R;
  load_tile<T, NB>(b, rp, ci, val, R);
  const T* src = dual ? A.xbar : A.y;
  spec_products<T, NB>(b, src, R);
  const InstState& S = A.st[b.inst];
  const int64_t g = *A.gbase + step;
  const int mode = step_mode(S, g);
  if (mode == M_SKIP || (!dual && mode == M_RESID)) return;
  T* spart = dual ? A.spartD : A.spartP;
  const int64_t space = dual ? A.MS : A.NS;
  const int nv = mode == M_EVAL ? 3 : 1;
  if (mode == M_EVAL) {
    if (dual) block_spmv_regs<T, 3, NB>(b, ci, val, R, A.xT, A.cx1, A.cx2, s_prod, s_rsum, s_rp, s_red);
    else block_spmv_regs<T, 3, NB>(b, ci, val, R, A.yT, A.cy1, A.cy2, s_prod, s_rsum, s_rp, s_red);
  } else {
    block_spmv1<T, NB>(b, ci, val, R, src, s_prod, s_rsum[0], s_rp, s_red, (T)1, true);
  }
  const int nrows = b.r1 - b.r0;
  const int sl = blk_slice(b);
  for (int r = threadIdx.x; r < nrows; r += kThreads)
    for (int a = 0; a < nv; ++a) spart[(int64_t)(a * (dual ? A.nslD : A.nslP) + sl) * space + b.r0 + r] = s_rsum[a][r];
}

// NB: entries per slice tile (kSliceTiles lists the compiled sizes; the
// engine picks one per solver, and the tuner in the Python package times them)
template <class T, int NB>
__global__ __launch_bounds__(kThreads) void primal_slice_step(IterArgs<T> A, int step) {
  slice_body<T, false, NB>(A, step);
}

template <class T, int NB>
__global__ __launch_bounds__(kThreads) void dual_slice_step(IterArgs<T> A, int step) {
  slice_body<T, true, NB>(A, step);
}

// Row sums of one (group, slice) block of a sorted-group product, one gather
// per add (Options::group_batched = 0): each gather is guarded by its own
// bounds test and waits for the previous add.
template <class T, int TPB, int U, bool NT>
__device__ __forceinline__ void group_rows_sum(const Blk& b, const uint32_t* __restrict__ w,
                                               const T* __restrict__ val, const T* __restrict__ src,
                                               double* s_row) {
  const int rb = blk_rowbits(b);
  const uint32_t rmask = (1u << rb) - 1u;
  const T* srcb = src + b.rp_off;
  const uint32_t* kp = w + b.p0;
  const T* vp = val + b.p0;
  const int pn = b.pn;
  for (int e0 = threadIdx.x; e0 < pn; e0 += TPB * U) {
    uint32_t k[U];
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * TPB;
      if (e < pn) {
        k[u] = ld_entry<NT>(kp + e);
        v[u] = ld_entry<NT>(vp + e);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * TPB;
      if (e < pn) atomicAdd(&s_row[k[u] & rmask], (double)(v[u] * srcb[k[u] >> rb]));
    }
  }
}

// Partial row sums of one column slice of a sorted row group (written to the
// slice-partial buffer for the step kernel of the same step to add up).
// DUAL: a group of K's rows gathering xbar (xT, cx1 and cx2 one after the
// other at an eval step) into spartD; otherwise a group of K^T's rows
// gathering y (yT, cy1, cy2) into spartP.  The group's row sums sit in
// dynamic LDS (FP64 words for the rows of the largest group of the schedule).
template <class T, bool DUAL, int TPB, bool BATCHED>
__global__ __launch_bounds__(TPB) void sorted_group_step(IterArgs<T> A, int step) {
  extern __shared__ __align__(16) unsigned char group_lds[];
  double* s_row = reinterpret_cast<double*>(group_lds);
  auto sched = (cptr<BlkWords>)(DUAL ? A.schedDS : A.schedPS);
  auto gbase = (cptr<int64_t>)A.gbase;
  auto states = (cptr<InstState>)A.st;
  const int32_t* ci = DUAL ? A.K_ci : A.KT_ci;
  const T* val = DUAL ? A.K_v : A.KT_v;
  int at = step;
  asm("" : "+s"(sched), "+s"(gbase), "+s"(states), "+s"(ci), "+s"(val), "+s"(at));
  const Blk b = load_blk(sched + blockIdx.x);
  const int64_t g = *gbase + at;
  if (blk_kind(b) == BK_PAD) return;
  SortedStream<T, TPB, kGroupEntries / TPB, 1> st;
  if constexpr (BATCHED) st.open(b, ci, val);  // before the LP state is read
  const int mode = step_mode(states + b.inst, g);
  if (mode == M_SKIP || (!DUAL && mode == M_RESID)) return;
  const int nrows = b.r1 - b.r0;
  const int sl = blk_slice(b);
  const int nv = mode == M_EVAL ? 3 : 1;
  T* spart = DUAL ? A.spartD : A.spartP;
  const int64_t space = DUAL ? A.MS : A.NS;
  for (int a = 0; a < nv; ++a) {
    const T* src = DUAL ? (mode != M_EVAL ? A.xbar : a == 0 ? A.xT : a == 1 ? A.cx1 : A.cx2)
                        : (mode != M_EVAL ? A.y : a == 0 ? A.yT : a == 1 ? A.cy1 : A.cy2);
    clear_rows(s_row, nrows, TPB);
    lds_barrier();
    if constexpr (BATCHED) {
      st.sum(src + b.rp_off, s_row, nrows + (threadIdx.x & 63));
      if (a + 1 < nv) st.open(b, ci, val);
    } else if (blk_nt(b)) {
      group_rows_sum<T, TPB, 4, true>(b, reinterpret_cast<const uint32_t*>(ci), val, src, s_row);
    } else {
      group_rows_sum<T, TPB, 4, false>(b, reinterpret_cast<const uint32_t*>(ci), val, src, s_row);
    }
    lds_barrier();
    for (int r = threadIdx.x; r < nrows; r += TPB)
      spart[(int64_t)(a * (DUAL ? A.nslD : A.nslP) + sl) * space + b.r0 + r] = (T)s_row[r];
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// controller: runs once per LP per check / eval / residual step
// ---------------------------------------------------------------------------

__device__ void controller(InstState& S, const double* sp, const double* sd, int mode, int64_t g,
                           int* status_out, int inst) {
  if (mode == M_CHECK) {
    S.acc[A_DX2] = sp[0];
    S.acc[A_AX2] = sp[1];
    S.acc[A_POBJ] = sp[2];
    S.acc[A_CD1] = sp[3];
    S.acc[A_CD2] = sp[4];
    S.acc[A_DY2] = sd[0];
    S.acc[A_AY2] = sd[1];
    S.acc[A_DOBJQ] = sd[2];
    S.acc[A_QY1] = sd[3];
    S.acc[A_QY2] = sd[4];
    S.acc[A_ACTX] = sp[5];
    S.acc[A_ACTY] = sd[5];
    S.phase = PH_EVAL;
    return;
  }
  if (mode == M_RESID) {
    const double v = sp[0] / S.tau + sd[0] / S.sigma + 2.0 * sd[1];
    S.r0 = sqrt(fmax(v, 0.0));
    S.phase = PH_NORMAL;
    return;
  }
  // eval step: the check candidate is T(z^{n,k}) from the previous step
  const int64_t t = g - S.tbase;          // evaluations of T so far
  const int64_t k = (g - 1) - S.kbase;    // inner counter of the check step
  S.tbase += 1;
  S.checks += 1;
  const double vres = S.acc[A_DX2] / S.tau + S.acc[A_DY2] / S.sigma + 2.0 * sd[1];
  const double res = sqrt(fmax(vres, 0.0));
  const double rel_p = sqrt(sd[0]) / (1.0 + S.qnorm);
  const double rel_d = sqrt(sp[0]) / (1.0 + S.cnorm);
  const double pobj = S.acc[A_POBJ];
  const double dobj = S.acc[A_DOBJQ] + sp[1];
  const double gap = fabs(pobj - dobj) / (1.0 + fabs(pobj) + fabs(dobj));
  const double kkt = fmax(rel_p, fmax(rel_d, gap));
  S.kkt = kkt;
  S.rel_p = rel_p;
  S.rel_d = rel_d;
  S.rel_gap = gap;
  S.pobj = pobj;
  S.dobj = dobj;
  S.resid = res;
  S.iters = t;
  S.act_changes = (int64_t)(S.acc[A_ACTX] + S.acc[A_ACTY]);
  if (S.act_changes > 0) S.ident_iters = t;
  int st = ST_RUNNING;
  // a NaN or Inf in any reduction (fmax would pass over a NaN part)
  if (!isfinite(kkt) || !isfinite(vres) || !isfinite(rel_p) || !isfinite(rel_d) || !isfinite(gap)) {
    st = ST_NUMERICAL;
  } else if (kkt <= S.tol) {
    st = ST_OPTIMAL;
  } else {
    const double m1 = S.acc[A_QY1] - sp[2];
    const double m2 = S.acc[A_QY2] - sp[4];
    if (m1 > 0.0 && sqrt(sp[3]) <= S.eps_inf * m1) {
      st = ST_PRIMAL_INFEAS;
      S.ray = 1;
    } else if (m2 > 0.0 && sqrt(sp[5]) <= S.eps_inf * m2) {
      st = ST_PRIMAL_INFEAS;
      S.ray = 2;
    } else {
      const double c1 = S.acc[A_CD1], c2 = S.acc[A_CD2];
      if (c1 < 0.0 && sqrt(sd[2]) + sqrt(sd[3]) <= S.eps_inf * fabs(c1)) {
        st = ST_DUAL_INFEAS;
        S.ray = 1;
      } else if (c2 < 0.0 && sqrt(sd[4]) + sqrt(sd[5]) <= S.eps_inf * fabs(c2)) {
        st = ST_DUAL_INFEAS;
        S.ray = 2;
      }
    }
    if (st == ST_RUNNING && t >= S.max_iter) st = ST_ITER_LIMIT;
    if (!(kkt >= 0.9 * S.best_kkt)) {
      S.best_kkt = kkt;
      S.best_check = S.checks;
    }
    if (st == ST_RUNNING && S.stall_checks > 0 && S.checks - S.best_check >= S.stall_checks) st = ST_ITER_LIMIT;
  }
  if (st != ST_RUNNING) {
    S.status = st;
    S.phase = PH_NORMAL;
    status_out[inst] = st;
    return;
  }
  bool restart = false;
  const bool artificial = S.artificial > 0.0 && (double)k >= S.artificial * (double)t;
  if (S.restart_mode == 0 && S.avg)
    restart = (S.nrest == 0) || (kkt <= S.avg_b1 * S.kkt_anchor) ||
              (kkt <= S.avg_b2 * S.kkt_anchor && kkt > S.kkt_prev) || artificial;
  else if (S.restart_mode == 0)
    restart = (S.nrest == 0) || (res <= S.beta * S.r0) || artificial;
  else if (S.restart_mode == 1)
    restart = k >= S.fixed_len;
  S.kkt_prev = kkt;
  if (restart) {
    S.kkt_anchor = kkt;
    S.kkt_prev = INFINITY;
  }
  if (restart) {
    const double dX = sqrt(S.acc[A_AX2]), dY = sqrt(S.acc[A_AY2]);
    if (S.primal_weight && dX > 1e-10 && dY > 1e-10 && isfinite(dX) && isfinite(dY))
      S.omega = exp(0.5 * log(dY / dX) + 0.5 * log(S.omega));
    S.tau = S.eta / S.omega;
    S.sigma = S.eta * S.omega;
    S.nrest += 1;
    S.phase = PH_RESID;
    S.kbase = g + 1;
    S.next_check = g + 1 + S.C;
  } else {
    S.phase = PH_NORMAL;
    S.kbase += 1;
    S.next_check = g + S.C;
  }
}

// ---------------------------------------------------------------------------
// dual step (rows of K = constraints) + per-LP controller
// ---------------------------------------------------------------------------

// End of a check, eval or residual step: the LP's dual blocks (of both step
// kernels) count themselves in, and the last one sums the partial sums of the
// step in a fixed order and runs the controller.  Normal steps (61 of 64) do
// none of this, so the fences, which write back and drop an XCD's L2, are
// rare; a control kernel of its own cost every step its launch and a round
// trip for the LP state (1.3 us of 8.8 at 60 x 120, 4.6 us at 20k rows or more).
// Every other block has read the LP state before it counts itself in.
template <int TPB, class T>
__device__ __forceinline__ void finish_step(const IterArgs<T>& A, int inst, int mode, int64_t g,
                                            double (*s_red)[kNS], double* s_out) {
  __shared__ double s_sum[kNS];
  __shared__ int s_last;
  InstState& S = A.st[inst];
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    const int blocks = S.db1 - S.db0;
    const int last = __hip_atomic_fetch_add(A.cnt + inst, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == blocks - 1;
    if (last) {
      A.cnt[inst] = 0;
      __threadfence();
    }
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  sum_partials<TPB>(A.partP + (int64_t)S.pb0 * kNS, S.pb1 - S.pb0, s_red, s_out);
  sum_partials<TPB>(A.partD + (int64_t)S.db0 * kNS, S.db1 - S.db0, s_red, s_sum);
  if (threadIdx.x == 0) controller(S, s_out, s_sum, mode, g, A.status_out, inst);
}

// One constraint's part of a dual step (rows of K): i is its space
// position, s0 its row sum (K xbar, or K xT at an eval step, where a1 and a2
// are K cx1 and K cx2; at a residual step the caller passes T(z) as yo and
// y0i and the saved K x+ as kxpi).  Adds the check / eval / residual terms
// of the row to ps.  Returns the next y (eval step: nothing of use).
template <class T>
__device__ __forceinline__ T dual_row(const IterArgs<T>& A, const InstState& S, int mode, int64_t g,
                                         int64_t i, T qi, T yo, T y0i, T kxpi, T s0, T a1, T a2,
                                         double (&ps)[kNS]) {
  const bool resid = (mode == M_RESID);
  const bool ineq = (i - S.row0) >= S.m_eq;
  if (mode == M_EVAL) {
    A.kxp[i] = s0;
    const double dr = A.Dr[i];
    double r = ((double)s0 - (double)qi) / dr;
    if (ineq) r = fmin(r, 0.0);
    ps[0] += r * r;
    ps[1] += (double)A.dy[i] * ((double)s0 - (double)A.kxbar[i]);
#pragma unroll
    for (int a = 1; a <= 2; ++a) {
      const double av = (double)(a == 1 ? a1 : a2) / dr;
      if (ineq) {
        const double mv = fmin(av, 0.0);
        ps[2 * a + 1] += mv * mv;
      } else {
        ps[2 * a] += av * av;
      }
    }
    return (T)0;
  }
  const T sigma = (T)S.sigma;
  T yp = yo + sigma * (qi - s0);
  if (ineq) yp = fmax(yp, (T)0);
  const T yb = (T)2 * yp - yo;
  const int64_t k = g - S.kbase;
  T yn = yp, yc = yp;  // next iterate; check candidate
  if (S.avg) {
    const T ysum = (k == 0 ? yo : A.ys[i]) + yp;
    A.ys[i] = ysum;
    if (mode == M_CHECK) yc = ysum / (T)(k + 2);
  } else {
    const double w = (double)(k + 1) / (double)(k + 2);
    const T yh = S.reflect ? yb : yp;
    yn = (T)w * yh + (T)(1.0 - w) * y0i;
  }
  A.y[i] = yn;
  if (resid) {
    A.y0[i] = yo;
    const double d = (double)yo - (double)yp;
    ps[0] += d * d;
    ps[1] += d * (0.5 * ((double)kxpi - (double)s0));
  } else if (mode == M_CHECK) {
    A.yT[i] = yc;
    const T dyv = yo - yp;
    A.dy[i] = dyv;
    A.kxbar[i] = s0;
    T e1 = yp - yo, e2 = yo - y0i;
    if (ineq) {
      e1 = fmax(e1, (T)0);
      e2 = fmax(e2, (T)0);
    }
    A.cy1[i] = e1;
    A.cy2[i] = e2;
    const double ad = (double)yc - (double)y0i;
    ps[0] += (double)dyv * (double)dyv;
    ps[1] += ad * ad;
    ps[2] += (double)qi * (double)yc;
    ps[3] += (double)qi * (double)e1;
    ps[4] += (double)qi * (double)e2;
    const uint8_t act = (ineq && yp == (T)0) ? 1 : 0;
    const uint8_t was = A.acty[i];
    A.acty[i] = act;
    ps[5] += (was != 255 && was != act) ? 1.0 : 0.0;
  }
  return yn;
}

template <class T>
__global__ __launch_bounds__(kThreads) void dual_step(IterArgs<T> A, int step) {
  __shared__ T s_prod[Tile<T>::NB];
  __shared__ T s_rsum[3][kMaxRows];
  __shared__ int s_rp[kMaxRows + 1];
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];

  const Blk b = A.schedD[blockIdx.x];
  if (blk_kind(b) == BK_PAD) return;
  const int nrows = b.r1 - b.r0;
  const int t = threadIdx.x;
  const bool own = t < nrows;
  const int64_t i = (int64_t)b.r0 + (own ? t : 0);
  // entries and epilogue operands are loaded before the LP state is read
  TileRegs<T, kPlainNB> R;
  load_tile<T, kPlainNB>(b, A.K_rp + b.r0, A.K_ci, A.K_v, R);
  spec_products<T, kPlainNB>(b, A.xbar, R);
  T qi = 0, yo = 0, y0i = 0, kxpi = 0;
  if (own) {
    qi = A.q[i];
    yo = A.y[i];
    y0i = A.y0[i];
  }
  const InstState& S = A.st[b.inst];
  const int64_t g = *A.gbase + step;
  const int mode = step_mode(S, g);
  if (mode == M_SKIP) return;
  const bool resid = (mode == M_RESID);
  if (resid && own) {
    yo = A.yT[i];
    y0i = yo;
    kxpi = A.kxp[i];
  }
  if (mode == M_EVAL) {
    block_spmv_regs<T, 3, kPlainNB>(b, A.K_ci, A.K_v, R, A.xT, A.cx1, A.cx2, s_prod, s_rsum, s_rp, s_red);
  } else {
    block_spmv1<T, kPlainNB>(b, A.K_ci, A.K_v, R, A.xbar, s_prod, s_rsum[0], s_rp, s_red, (T)1, true);
  }

  double ps[kNS];
#pragma unroll
  for (int s = 0; s < kNS; ++s) ps[s] = 0.0;
  if (own) {
    const bool eval = (mode == M_EVAL);
    dual_row<T>(A, S, mode, g, i, qi, yo, y0i, kxpi, s_rsum[0][t], eval ? s_rsum[1][t] : (T)0,
                eval ? s_rsum[2][t] : (T)0, ps);
  }
  if (mode == M_NORMAL) return;

  block_sum_ns(ps, s_red, s_out);
  if (t < kNS) A.partD[(int64_t)b.gid * kNS + t] = s_out[t];
  finish_step<kThreads>(A, b.inst, mode, g, s_red, s_out);
}

// One step over a column-sorted block (BK_SORTED): a block of K^T rows
// (DUAL false, a primal step) or of K rows (a dual step).  The products with
// y (yT, cy1, cy2 at an eval step) or xbar (xT, cx1, cx2) are added into LDS
// row sums, then each thread takes the epilogue of every TPB-th row.  The
// first entries and the operands of the thread's first row are loaded before
// the LP state is read (none depends on it).
//
// Where one row holds a large part of a block's entries (blk_rep_shift > 0)
// its products would queue up at one LDS word; such a block keeps 2^shift
// copies of each row sum, lane l adding into copy l mod 2^shift.
// The row sums sit in dynamic LDS (FP64 words for the largest block of the
// schedule, and kSpareWords).
template <class T, bool DUAL, int TPB, int D>
__global__ __launch_bounds__(TPB) void sorted_step(IterArgs<T> A, int step) {
  extern __shared__ __align__(16) unsigned char sorted_lds[];
  __shared__ double s_red[TPB / 64][kNS];
  __shared__ double s_out[kNS];
  double* s_row = reinterpret_cast<double*>(sorted_lds);
  // The block starts with a chain of loads: kernel arguments, descriptor,
  // entries, gathers.  The arguments that the chain needs are tied together so
  // that they cost one round trip.
  auto sched = (cptr<BlkWords>)(DUAL ? A.schedDB : A.schedPB);
  auto gbase = (cptr<int64_t>)A.gbase;
  auto states = (cptr<InstState>)A.st;
  const int32_t* ci = DUAL ? A.K_ci : A.KT_ci;
  const T* val = DUAL ? A.K_v : A.KT_v;
  // q, y, y0 or c, l, u, x, x0
  gptr<T> v0 = (gptr<T>)(DUAL ? A.q : A.c), v1 = (gptr<T>)(DUAL ? A.y : A.l), v2 = (gptr<T>)(DUAL ? A.y0 : A.u),
          v3 = (gptr<T>)A.x, v4 = (gptr<T>)A.x0;
  int at = step;
  asm("" : "+s"(sched), "+s"(gbase), "+s"(states), "+s"(ci), "+s"(val), "+s"(v0), "+s"(v1), "+s"(v2), "+s"(v3),
      "+s"(v4), "+s"(at));
  const Blk b = load_blk(sched + blockIdx.x);
  const int64_t g = *gbase + at;
  if (blk_kind(b) == BK_PAD) return;
  const int nrows = b.r1 - b.r0;
  const int tid = threadIdx.x;
  const int64_t p0 = (int64_t)b.r0 + min(tid, nrows - 1);
  T o0 = v0[p0], o1 = v1[p0], o2 = v2[p0], o3 = 0, o4 = 0;
  if constexpr (!DUAL) {
    o3 = v3[p0];
    o4 = v4[p0];
  }
  SortedStream<T, TPB, kPlainU, D> st;
  st.open(b, ci, val);
  const int rs = blk_rep_shift(b);
  const int words = nrows << rs;
  clear_rows(s_row, words, TPB);
  const int mode = step_mode(states + b.inst, g);
  if (mode == M_SKIP) return;
  const InstState& S = A.st[b.inst];
  const bool resid = (mode == M_RESID);
  // row sum of row r (its copies added in a fixed order)
  auto row_sum = [&](int r) -> T {
    const double* w = s_row + (r << rs);
    if (rs == 0) return (T)w[0];
    double a = 0.0;
    for (int c = 0; c < (1 << rs); c += 8)  // kMinRepShift: at least 8 copies
      a += ((w[c] + w[c + 1]) + (w[c + 2] + w[c + 3])) + ((w[c + 4] + w[c + 5]) + (w[c + 6] + w[c + 7]));
    return (T)a;
  };
  const int copy = tid & ((1 << rs) - 1);
  // at an eval step first the two ray candidates (their sums are read back
  // below by the thread that stores them)
  const int np = mode == M_EVAL ? 3 : (DUAL || !resid) ? 1 : 0;
  for (int a = np; a > 0; --a) {
    const T* src = mode != M_EVAL ? (DUAL ? A.xbar : A.y)
                   : a == 3       ? (DUAL ? A.cx1 : A.cy1)
                   : a == 2       ? (DUAL ? A.cx2 : A.cy2)
                                  : (DUAL ? A.xT : A.yT);
    lds_barrier();
    st.sum(src + b.rp_off, s_row + copy, words - copy + (tid & 63), rs);
    lds_barrier();
    if (a > 1) {
      T* out = a == 3 ? (DUAL ? A.kx1 : A.kt1) : (DUAL ? A.kx2 : A.kt2);
      st.open(b, ci, val);
      for (int r = tid; r < nrows; r += TPB) out[(int64_t)b.r0 + r] = row_sum(r);
      lds_barrier();
      clear_rows(s_row, words, TPB);
    }
  }
  double ps[kNS];
#pragma unroll
  for (int s = 0; s < kNS; ++s) ps[s] = 0.0;
  for (int r = tid; r < nrows; r += TPB) {
    const int64_t i = (int64_t)b.r0 + r;
    if constexpr (DUAL) {
      if (r >= TPB) {
        o0 = A.q[i];
        o1 = A.y[i];
        o2 = A.y0[i];
      }
      T kxpi = 0, a1 = 0, a2 = 0;
      if (resid) {
        o1 = A.yT[i];
        o2 = o1;
        kxpi = A.kxp[i];
      }
      if (mode == M_EVAL) {
        a1 = A.kx1[i];
        a2 = A.kx2[i];
      }
      dual_row<T>(A, S, mode, g, i, o0, o1, o2, kxpi, row_sum(r), a1, a2, ps);
    } else {
      if (r >= TPB) {
        o0 = A.c[i];
        o1 = A.l[i];
        o2 = A.u[i];
        o3 = A.x[i];
        o4 = A.x0[i];
      }
      T kty, g1 = 0, g2 = 0;
      if (resid) {
        o3 = A.xT[i];
        o4 = o3;
        kty = A.ktyp[i];
      } else {
        kty = row_sum(r);
        if (mode == M_EVAL) {
          g1 = A.kt1[i];
          g2 = A.kt2[i];
        }
      }
      primal_row<T>(A, S, mode, g, i, o0, o1, o2, o3, o4, kty, g1, g2, ps);
    }
  }
  if (mode != M_NORMAL) {
    block_sum_ns<TPB>(ps, s_red, s_out);
    if (tid < kNS) (DUAL ? A.partD : A.partP)[(int64_t)b.gid * kNS + tid] = s_out[tid];
    if constexpr (DUAL) finish_step<TPB>(A, b.inst, mode, g, s_red, s_out);
  }
}

// The step of rows whose products a slice kernel computed (kBlkPart blocks of
// up to kPartRows rows): a row's nsl slice partial sums, added in slice order,
// then its epilogue.  Streaming work (9 vectors and the partial sums): each
// thread takes RPT rows, kThreads apart, and issues their loads together,
// before the LP state is read.  1024 variables or 512 constraints per block
// instead of 256 also leave fewer partial sums to the controller.
template <class T, bool DUAL>
__global__ __launch_bounds__(kThreads) void part_step(IterArgs<T> A, int step) {
  constexpr int RPT = kPartRows(DUAL) / kThreads;
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  const Blk b = load_blk((cptr<BlkWords>)(DUAL ? A.schedDE : A.schedPE) + blockIdx.x);
  if (blk_kind(b) == BK_PAD) return;
  const int64_t g = *(cptr<int64_t>)A.gbase + step;
  const int nrows = b.r1 - b.r0, nsl = blk_nsl(b);
  const int tid = threadIdx.x;
  const int64_t space = DUAL ? A.MS : A.NS;
  const T* spart = (DUAL ? A.spartD : A.spartP) + b.r0;
  int r[RPT];
  T o[RPT][DUAL ? 3 : 5];  // q, y, y0 or c, l, u, x, x0
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    r[k] = min(tid + k * kThreads, max(nrows - 1, 0));
    const int64_t i = (int64_t)b.r0 + r[k];
    if constexpr (DUAL) {
      o[k][0] = A.q[i];
      o[k][1] = A.y[i];
      o[k][2] = A.y0[i];
    } else {
      o[k][0] = A.c[i];
      o[k][1] = A.l[i];
      o[k][2] = A.u[i];
      o[k][3] = A.x[i];
      o[k][4] = A.x0[i];
    }
  }
  // sums of vector a's partials (a > 0: the ray candidates of an eval step),
  // added in slice order, four slices' loads in flight together
  auto sums = [&](int a, T (&acc)[RPT]) {
    const T* p = spart + (int64_t)a * (DUAL ? A.nslD : A.nslP) * space;
    if (nsl <= 2) {
      T v[2][RPT];
#pragma unroll
      for (int k = 0; k < RPT; ++k) {
        v[0][k] = p[r[k]];
        v[1][k] = nsl == 2 ? p[space + r[k]] : (T)0;
      }
#pragma unroll
      for (int k = 0; k < RPT; ++k) acc[k] = nsl == 2 ? v[0][k] + v[1][k] : v[0][k];
      return;
    }
    for (int q = 0; q < nsl; q += 4, p += 4 * space) {
      T v[4][RPT];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < RPT; ++k) v[j][k] = p[j * space + r[k]];
#pragma unroll
      for (int k = 0; k < RPT; ++k)
        acc[k] = (q == 0 ? v[0][k] : acc[k] + v[0][k]) + v[1][k] + v[2][k] + v[3][k];
    }
  };
  const int mode = step_mode((cptr<InstState>)A.st + b.inst, g);
  if (mode == M_SKIP) return;
  const InstState& S = A.st[b.inst];
  const bool resid = (mode == M_RESID);
  T s0[RPT], s1[RPT], s2[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) s0[k] = s1[k] = s2[k] = 0;
  if (DUAL || !resid) sums(0, s0);
  if (mode == M_EVAL) {
    sums(1, s1);
    sums(2, s2);
  }
  double ps[kNS];
#pragma unroll
  for (int s = 0; s < kNS; ++s) ps[s] = 0.0;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    if (tid + k * kThreads < nrows) {
      const int64_t i = (int64_t)b.r0 + r[k];
      if constexpr (DUAL) {
        T kxpi = 0;
        if (resid) {
          o[k][1] = A.yT[i];
          o[k][2] = o[k][1];
          kxpi = A.kxp[i];
        }
        dual_row<T>(A, S, mode, g, i, o[k][0], o[k][1], o[k][2], kxpi, s0[k], s1[k], s2[k], ps);
      } else {
        if (resid) {
          o[k][3] = A.xT[i];
          o[k][4] = o[k][3];
          s0[k] = A.ktyp[i];
        }
        primal_row<T>(A, S, mode, g, i, o[k][0], o[k][1], o[k][2], o[k][3], o[k][4], s0[k], s1[k], s2[k], ps);
      }
    }
  }
  if (mode != M_NORMAL) {
    block_sum_ns(ps, s_red, s_out);
    if (tid < kNS) (DUAL ? A.partD : A.partP)[(int64_t)b.gid * kNS + tid] = s_out[tid];
    if constexpr (DUAL) finish_step<kThreads>(A, b.inst, mode, g, s_red, s_out);
  }
}

// ---------------------------------------------------------------------------
// small LPs: all steps of a chunk in one workgroup
// ---------------------------------------------------------------------------

// One thread's entries of a column-sorted block, kept in registers.
template <class T, int TPB>
struct ResidentEntries {
  uint32_t k[kResEntries];
  T v[kResEntries];
  int cnt, rb, rs;
  __device__ __forceinline__ void load(const Blk& b, const int32_t* ci, const T* val) {
    const int tid = threadIdx.x;
    cnt = b.pn > tid ? (b.pn - tid + TPB - 1) / TPB : 0;
    rb = blk_rowbits(b);
    rs = blk_rep_shift(b);
#pragma unroll
    for (int u = 0; u < kResEntries; ++u) {
      k[u] = 0;
      v[u] = (T)0;
      if (u < cnt) {
        k[u] = (uint32_t)ci[b.p0 + tid + u * TPB];
        v[u] = val[b.p0 + tid + u * TPB];
      }
    }
  }
  // adds the products with src (the vector from the block's first column on)
  // into the row sums, each lane into its copy of a row's
  template <class Src>
  __device__ __forceinline__ void sum(Src src, double* s_row) const {
    const uint32_t rmask = (1u << rb) - 1u;
    const uint32_t copy = threadIdx.x & ((1u << rs) - 1u);
    T g[kResEntries];
#pragma unroll
    for (int u = 0; u < kResEntries; ++u)
      if (u < cnt) g[u] = src[k[u] >> rb];
#pragma unroll
    for (int u = 0; u < kResEntries; ++u)
      if (u < cnt) atomicAdd(&s_row[((k[u] & rmask) << rs) + copy], (double)(v[u] * g[u]));
  }
  // row r's sum (copies in a fixed order), which is cleared for the next product
  __device__ __forceinline__ T take(double* s_row, int r) const {
    double* w = s_row + (r << rs);
    double a = 0.0;
    for (int c = 0; c < (1 << rs); ++c) {
      a += w[c];
      w[c] = 0.0;
    }
    return (T)a;
  }
};

// All steps of a chunk of an LP whose K and K^T are one column-sorted block
// each of at most TPB rows and kResEntries * TPB entries: one workgroup
// per LP, one thread per row of either product.  Two kernels per iteration are
// bound by their launches and by the chain of loads that each begins with
// (arguments, descriptor, entries, gathers: 3.9 us per kernel at 60 x 120,
// for 0.1 us of work); here the entries stay in registers, the gathered
// vectors and the LP state in LDS, and a step waits for LDS only: what is in
// device memory a thread only reads back itself (x and x0 right after they are
// stored, a half step before their use).
template <class T, int TPB>
__global__ __launch_bounds__(TPB) void resident_steps(IterArgs<T> A, int steps) {
  extern __shared__ __align__(16) unsigned char resident_lds[];
  __shared__ double s_red[TPB / 64][kNS];
  __shared__ double s_p[kNS], s_d[kNS];
  __shared__ InstState s_S;
  const int tid = threadIdx.x;
  const Blk bp = A.schedR[2 * blockIdx.x], bd = A.schedR[2 * blockIdx.x + 1];
  const int n = bp.r1 - bp.r0, m = bd.r1 - bd.r0;
  const int wordsP = n << blk_rep_shift(bp), wordsD = m << blk_rep_shift(bd);
  double* s_rowP = reinterpret_cast<double*>(resident_lds);
  double* s_rowD = s_rowP + wordsP;
  T* s_xbar = reinterpret_cast<T*>(s_rowD + wordsD);
  T* s_y = s_xbar + n;
  const int64_t g0 = *A.gbase;
  const int words = (int)(sizeof(InstState) / sizeof(uint32_t));
  for (int i = tid; i < words; i += TPB)
    reinterpret_cast<uint32_t*>(&s_S)[i] = reinterpret_cast<const uint32_t*>(A.st + bp.inst)[i];
  ResidentEntries<T, TPB> eP, eD;
  eP.load(bp, A.KT_ci, A.KT_v);
  eD.load(bd, A.K_ci, A.K_v);
  int64_t j = (int64_t)bp.r0 + min(tid, n - 1), i = (int64_t)bd.r0 + min(tid, m - 1);
  const T cj = A.c[j], lj = A.l[j], uj = A.u[j], qi = A.q[i];
  T x = A.x[j], x0 = A.x0[j], y = A.y[i], y0 = A.y0[i];
  if (tid < n) s_xbar[tid] = A.xbar[j];
  if (tid < m) s_y[tid] = y;
  for (int w = tid; w < wordsP + wordsD; w += TPB) s_rowP[w] = 0.0;
  __syncthreads();
  for (int s = 0; s < steps; ++s) {
    const int64_t g = g0 + s;
    if (s_S.status != ST_RUNNING) break;
    const int mode = __builtin_amdgcn_readfirstlane(step_mode(s_S, g));
    if (mode == M_SKIP) continue;
    // addresses formed where they are used, not kept in registers for all steps
    asm volatile("" : "+v"(j), "+v"(i));
    double ps[kNS];
    T a0 = 0, a1 = 0, a2 = 0;
    // an eval step puts the vectors that it multiplies in the place of y
    // (of xbar below, which the next primal step replaces), one after the other
#pragma unroll 1
    for (int a = mode == M_EVAL ? 2 : mode == M_RESID ? -1 : 0; a >= 0; --a) {
      if (mode == M_EVAL) {
        if (tid < m) s_y[tid] = (a == 0 ? A.yT : a == 1 ? A.cy1 : A.cy2)[i];
        lds_barrier();
      }
      eP.sum(s_y, s_rowP);
      lds_barrier();
      a2 = a1;
      a1 = a0;
      if (tid < n) a0 = eP.take(s_rowP, tid);
    }
    if (mode == M_EVAL && tid < m) s_y[tid] = y;
#pragma unroll
    for (int q = 0; q < kNS; ++q) ps[q] = 0.0;
    if (tid < n) {
      if (mode == M_RESID) {
        x = A.xT[j];
        x0 = x;
        a0 = A.ktyp[j];
      }
      const T xb = primal_row<T>(A, s_S, mode, g, j, cj, lj, uj, x, x0, a0, a1, a2, ps);
      if (mode != M_EVAL) s_xbar[tid] = xb;
      x = A.x[j];
      x0 = A.x0[j];
    }
    if (mode == M_NORMAL) {
      lds_barrier();
    } else {
      block_sum_ns<TPB>(ps, s_red, s_p);
    }
#pragma unroll 1
    for (int a = mode == M_EVAL ? 2 : 0; a >= 0; --a) {
      if (mode == M_EVAL) {
        if (tid < n) s_xbar[tid] = (a == 0 ? A.xT : a == 1 ? A.cx1 : A.cx2)[j];
        lds_barrier();
      }
      eD.sum(s_xbar, s_rowD);
      lds_barrier();
      a2 = a1;
      a1 = a0;
      if (tid < m) a0 = eD.take(s_rowD, tid);
    }
#pragma unroll
    for (int q = 0; q < kNS; ++q) ps[q] = 0.0;
    if (tid < m) {
      T kxpi = 0;
      if (mode == M_RESID) {
        y = A.yT[i];
        y0 = y;
        kxpi = A.kxp[i];
      }
      const T yn = dual_row<T>(A, s_S, mode, g, i, qi, y, y0, kxpi, a0, a1, a2, ps);
      if (mode != M_EVAL) {
        s_y[tid] = yn;
        y = yn;
      }
      if (mode != M_NORMAL) {
        y = A.y[i];
        y0 = A.y0[i];
      }
    }
    if (mode == M_NORMAL) {
      lds_barrier();
    } else {
      block_sum_ns<TPB>(ps, s_red, s_d);
      __syncthreads();
      if (tid == 0) controller(s_S, s_p, s_d, mode, g, A.status_out, bp.inst);
      __syncthreads();
    }
  }
  for (int i2 = tid; i2 < words; i2 += TPB)
    reinterpret_cast<uint32_t*>(A.st + bp.inst)[i2] = reinterpret_cast<const uint32_t*>(&s_S)[i2];
}

__global__ void tick_kernel(int64_t* gbase, int64_t add) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *gbase += add;
}

// ---------------------------------------------------------------------------
// preprocessing: Ruiz / Pock-Chambolle scaling
// ---------------------------------------------------------------------------

// A pass's factors of one side's rows, from the previous pass to this one.
// The other side's pass gathers the previous ones, so K's rows, which come
// first, keep theirs apart (`held`, or two halves where the buffers at hand
// hold 32-bit words) and pass the previous ones on (`prev`); the rows of K^T
// overwrite theirs (`held`; prev null).
struct RowFactors {
  double* held;
  uint32_t *lo, *hi;
  double* prev;
  __device__ double get(int64_t r) const {
    return held ? held[r] : __hiloint2double((int)hi[r], (int)lo[r]);
  }
  __device__ void set(int64_t r, double v) const {
    if (held) {
      held[r] = v;
    } else {
      hi[r] = (uint32_t)__double2hiint(v);
      lo[r] = (uint32_t)__double2loint(v);
    }
  }
};

// One scaling pass over one side's rows: entries divided by the previous
// pass's factors (by that of the row of K, then by that of its column, on both
// sides, so that K~ and its transpose hold the same bits; none in the first
// pass), then each row's new factor, the root of its largest entry (op 0) or
// of the sum of its entries^expo (op 1), 1 for rows of zeros, and D[r] divided
// by it; op 2 divides the entries only.  Every entry is rounded after each
// division: that is how the CPU oracle defines K~, and iterates are compared
// with its over a thousand steps, where entries formed from the product of
// the factors (as close to Dr K Dc, but rounded otherwise) end 2 to 3 times
// further from it (200k x 1M, 1,030 steps, largest difference of y 6e-11 to
// 1.0e-10 for 2e-11 to 5e-11).  Bound by the gathers of the other side's
// factors and 20 bytes per entry; one kernel divides and reduces, so the
// entries are read once per pass and side, coalesced, and staged in LDS (500k
// x 2M, 30M entries: 367 us per pass and side; 775 in two kernels with a row's
// entries read by its own lanes, 317 where entries are left alone).  A thread
// divides its own entries, by the row noted for each: divided in the rows'
// loops, one after another, 128 LPs took 36.5 ms to create instead of 34.7
// (33.3 with undivided entries), one of 2.4k x 8k 2.23 instead of 2.13.
__global__ __launch_bounds__(kThreads) void row_factor_kernel(const Blk* sched, const int32_t* __restrict__ rp,
                                                              const int32_t* __restrict__ ci, double* __restrict__ val,
                                                              int op, double expo, bool first, bool transposed,
                                                              const double* __restrict__ other, RowFactors F, double* D) {
  __shared__ double s_val[kPlainNB];
  __shared__ double s_f[kMaxRows];
  __shared__ uint8_t s_row[kPlainNB];  // row of an entry in the tile
  __shared__ int s_rp[kMaxRows + 1];
  __shared__ double s_red[kThreads / 64];
  const Blk b = sched[blockIdx.x];
  const int tid = threadIdx.x;
  const int nrows = b.r1 - b.r0;
  // entry v of a row with factor f in a column with factor o
  auto divide = [&](double v, double f, double o) { return transposed ? v / o / f : v / f / o; };
  auto add = [&](double a, double v) {
    v = fabs(v);
    if (op == 0) return fmax(a, v);
    return a + (expo != 1.0 ? pow(v, expo) : v);
  };
  auto finish = [&](int64_t r, double f, double a) {
    if (!first && F.prev) F.prev[r] = f;
    if (op == 2) return;
    const double q = sqrt(a), g = q > 0.0 ? q : 1.0;
    F.set(r, g);
    D[r] = (first ? 1.0 : D[r]) / g;
  };
  if (blk_kind(b) == BK_LONG) {
    const double f = first ? 1.0 : F.get(b.r0);
    double a = 0.0;
#pragma unroll 4
    for (int k = tid; k < b.pn; k += kThreads) {
      double v = val[b.p0 + k];
      if (!first) {
        v = divide(v, f, other[ci[b.p0 + k]]);
        val[b.p0 + k] = v;
      }
      a = add(a, v);
    }
    // max or sum over the block, in fixed order
    if (op == 0) {
      for (int off = 32; off > 0; off >>= 1) a = fmax(a, __shfl_xor(a, off, 64));
    } else {
      a = wave_sum(a);
    }
    if ((tid & 63) == 0) s_red[tid >> 6] = a;
    __syncthreads();
    if (tid == 0) {
      double r = s_red[0];
      for (int w = 1; w < kThreads / 64; ++w) r = op == 0 ? fmax(r, s_red[w]) : r + s_red[w];
      finish(b.r0, f, r);
    }
    return;
  }
  for (int r = tid; r <= nrows; r += kThreads) s_rp[r] = rp[b.r0 + r] - b.p0;
  for (int r = tid; r < nrows; r += kThreads) s_f[r] = first ? 1.0 : F.get(b.r0 + r);
  constexpr int kPer = kPlainNB / kThreads;
  double v[kPer], o[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int k = tid + i * kThreads;
    if (k < b.pn) {
      v[i] = val[b.p0 + k];
      if (!first) o[i] = other[ci[b.p0 + k]];
    }
  }
  __syncthreads();
  const int L = group_size(nrows);  // lanes per row
  const int lane = tid & (L - 1);
  if (!first) {
    for (int r = tid / L; r < nrows; r += kThreads / L)
      for (int k = s_rp[r] + lane; k < s_rp[r + 1]; k += L) s_row[k] = (uint8_t)r;
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int k = tid + i * kThreads;
    if (k < b.pn) {
      if (!first) {
        v[i] = divide(v[i], s_f[s_row[k]], o[i]);
        val[b.p0 + k] = v[i];
      }
      s_val[k] = v[i];
    }
  }
  __syncthreads();
  for (int base = 0; base < nrows; base += kThreads / L) {
    const int r = base + tid / L;
    double a = 0.0;
    if (r < nrows)
      for (int k = s_rp[r] + lane; k < s_rp[r + 1]; k += L) a = add(a, s_val[k]);
    for (int off = L >> 1; off > 0; off >>= 1) {
      const double o = __shfl_xor(a, off, 64);
      a = op == 0 ? fmax(a, o) : a + o;
    }
    if (lane == 0 && r < nrows) finish((int64_t)b.r0 + r, s_f[r], a);
  }
}

__global__ void fill_kernel(double* p, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

template <class T>
__global__ void cast_kernel(const double* src, T* dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (T)src[i];
}

// Scaled vectors over the rows of the given schedules, with each block's
// sums of squares for the norms: c^2 and (D_c c)^2 in part[0..1], q^2 and
// (D_r q)^2 likewise.  (A pass of one block per LP over q, c and both factors
// took 2.8 ms at 500k x 2M; here the values are at hand.)
template <class T>
__global__ __launch_bounds__(kThreads) void scale_primal_kernel(const Blk* schedP, const double* Dc,
                                                                const double* c, const double* l,
                                                                const double* u, T* cs, T* ls, T* us, double* part) {
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  const Blk b = schedP[blockIdx.x];
  double v[kNS];
  for (int s = 0; s < kNS; ++s) v[s] = 0.0;
  if ((int)threadIdx.x < b.r1 - b.r0) {
    const int64_t j = (int64_t)b.r0 + threadIdx.x;
    const double a = c[j], sa = Dc[j] * a;
    cs[j] = (T)sa;
    ls[j] = (T)(l[j] / Dc[j]);
    us[j] = (T)(u[j] / Dc[j]);
    v[0] = a * a;
    v[1] = sa * sa;
  }
  block_sum_ns(v, s_red, s_out);
  if (threadIdx.x < kNS) part[(int64_t)blockIdx.x * kNS + threadIdx.x] = s_out[threadIdx.x];
}

template <class T>
__global__ __launch_bounds__(kThreads) void scale_dual_kernel(const Blk* schedD, const double* Dr,
                                                              const double* q, T* qs, double* part) {
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  const Blk b = schedD[blockIdx.x];
  double v[kNS];
  for (int s = 0; s < kNS; ++s) v[s] = 0.0;
  if ((int)threadIdx.x < b.r1 - b.r0) {
    const int64_t i = (int64_t)b.r0 + threadIdx.x;
    const double a = q[i], sa = Dr[i] * a;
    qs[i] = (T)sa;
    v[0] = a * a;
    v[1] = sa * sa;
  }
  block_sum_ns(v, s_red, s_out);
  if (threadIdx.x < kNS) part[(int64_t)blockIdx.x * kNS + threadIdx.x] = s_out[threadIdx.x];
}

// per-LP norms from those sums, one block per LP, fixed order: ||q||, ||c||
// (unscaled) to the state, ||D_r q||, ||D_c c|| to out[2 * block + {0,1}]
__global__ __launch_bounds__(kThreads) void inst_norms_kernel(InstState* st, const int* ids, const int4* ranges,
                                                              const double* partP, const double* partD, double* out) {
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_c[kNS], s_q[kNS];
  InstState& S = st[ids[blockIdx.x]];
  const int4 rg = ranges[blockIdx.x];
  sum_partials(partP + (int64_t)rg.x * kNS, rg.y - rg.x, s_red, s_c);
  __syncthreads();
  sum_partials(partD + (int64_t)rg.z * kNS, rg.w - rg.z, s_red, s_q);
  if (threadIdx.x == 0) {
    S.qnorm = sqrt(s_q[0]);
    S.cnorm = sqrt(s_c[0]);
    out[2 * blockIdx.x] = sqrt(s_q[1]);
    out[2 * blockIdx.x + 1] = sqrt(s_c[1]);
  }
}

// write the host-prepared states of new LPs and clear their status words
__global__ void write_states_kernel(InstState* st, int* status_out, int* cnt, const int* ids,
                                    const InstState* src, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) {
    st[ids[i]] = src[i];
    status_out[ids[i]] = src[i].status;
    cnt[ids[i]] = 0;
  }
}

// schedule ranges of live LPs after a schedule rebuild
__global__ void set_ranges_kernel(InstState* st, const int* ids, const int4* ranges, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) {
    InstState& S = st[ids[i]];
    const int4 r = ranges[i];
    S.pb0 = r.x;
    S.pb1 = r.y;
    S.db0 = r.z;
    S.db1 = r.w;
  }
}

// ---------------------------------------------------------------------------
// power iteration on K~^T K~ (per LP)
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t j) {
  uint64_t z = seed + (j + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// w = SplitMix64 uniform [-1, 1) start vector over each LP's variables, and
// the block partial of sum w^2
__global__ __launch_bounds__(kThreads) void pw_start_kernel(const Blk* schedP, const InstState* st,
                                                            uint64_t seed, double* w, double* partP) {
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  const Blk b = schedP[blockIdx.x];
  const InstState& S = st[b.inst];
  double v[kNS];
  for (int s = 0; s < kNS; ++s) v[s] = 0.0;
  const int nrows = b.r1 - b.r0;
  if ((int)threadIdx.x < nrows) {
    const int64_t j = (int64_t)b.r0 + threadIdx.x;
    const uint64_t z = splitmix64_at(seed, (uint64_t)(j - S.col0));
    const double u = (double)(z >> 11) * 0x1.0p-53 * 2.0 - 1.0;
    w[j] = u;
    v[0] = u * u;
  }
  block_sum_ns(v, s_red, s_out);
  if (threadIdx.x < kNS) partP[(int64_t)blockIdx.x * kNS + threadIdx.x] = s_out[threadIdx.x];
}

// u = pw_scale * K~ w over the rows of K (dual schedule)
__global__ __launch_bounds__(kThreads) void pw_forward_kernel(const Blk* schedD, const InstState* st,
                                                              const int32_t* rp, const int32_t* ci,
                                                              const double* val, const double* w,
                                                              double* u) {
  __shared__ double s_prod[Tile<double>::NB];
  __shared__ double s_rsum[3][kMaxRows];
  __shared__ int s_rp[kMaxRows + 1];
  __shared__ double s_red[kThreads / 64][kNS];
  const Blk b = schedD[blockIdx.x];
  const InstState& S = st[b.inst];
  if (S.pw_done) return;
  block_spmv<double, 1>(b, rp + b.r0, ci, val, w, w, w, s_prod, s_rsum, s_rp, s_red, S.pw_scale);
  const int nrows = b.r1 - b.r0;
  if ((int)threadIdx.x < nrows) u[(int64_t)b.r0 + threadIdx.x] = s_rsum[0][threadIdx.x];
}

// Ends a power iteration of one LP: the estimate sqrt(||w||) and the stop
// rule; *done counts the LPs that have stopped.
__device__ __forceinline__ void pw_update(InstState& S, double w2, int start, int min_iters, int max_iters, double rtol,
                                          int* done) {
  const double nw = sqrt(w2);
  bool stop = !(nw > 0.0);
  if (start) {
    S.pw_scale = stop ? 0.0 : 1.0 / nw;
    S.pw_iter = 0;
    S.pw_prev = -1.0;
    S.sigma_hat = 0.0;
  } else {
    S.pw_iter += 1;
    if (stop) {
      S.sigma_hat = 0.0;
    } else {
      const double s = sqrt(nw);
      S.sigma_hat = s;
      S.pw_scale = 1.0 / nw;
      stop = (S.pw_prev >= 0.0 && S.pw_iter >= min_iters && fabs(s - S.pw_prev) <= rtol * s) || S.pw_iter >= max_iters;
      if (!stop) S.pw_prev = s;
    }
  }
  if (stop) {
    S.pw_done = 1;
    atomicAdd(done, 1);
  }
}

// A block's part of ||w||^2 (every thread's v), and, FUSED, the end of the
// iteration by the last of the LP's blocks, which saves small LPs a launch per
// iteration; the device-wide fence that each block then takes is dearer than the
// launch where there are many (kPowerFuse).
struct PowerEnd {
  double* partP;
  int *cnt, *done;
  int min_iters, max_iters;
  double rtol;
};
template <bool FUSED, int TPB = kThreads>
__device__ __forceinline__ void pw_block_end(const Blk& b, InstState& S, double v, const PowerEnd& E,
                                             double (*s_red)[kNS], double* s_out) {
  __shared__ int s_last;
  double ps[kNS];
  for (int s = 0; s < kNS; ++s) ps[s] = 0.0;
  ps[0] = v;
  block_sum_ns<TPB>(ps, s_red, s_out);
  if (threadIdx.x < kNS) E.partP[(int64_t)b.gid * kNS + threadIdx.x] = s_out[threadIdx.x];
  if constexpr (FUSED) {
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence();
      const int last =
          __hip_atomic_fetch_add(E.cnt + b.inst, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == S.pb1 - S.pb0 - 1;
      if (last) {
        E.cnt[b.inst] = 0;
        __threadfence();
      }
      s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    sum_partials<TPB>(E.partP + (int64_t)S.pb0 * kNS, S.pb1 - S.pb0, s_red, s_out);
    if (threadIdx.x == 0) pw_update(S, s_out[0], 0, E.min_iters, E.max_iters, E.rtol, E.done);
  }
}

// w = K~^T u over tiles of K^T, with the partial sum w^2
template <bool FUSED>
__global__ __launch_bounds__(kThreads) void pw_backward_kernel(const Blk* schedP, InstState* st,
                                                               const int32_t* rp, const int32_t* ci,
                                                               const double* val, const double* u, double* w,
                                                               PowerEnd E) {
  __shared__ double s_prod[Tile<double>::NB];
  __shared__ double s_rsum[3][kMaxRows];
  __shared__ int s_rp[kMaxRows + 1];
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  const Blk b = schedP[blockIdx.x];
  InstState& S = st[b.inst];
  if (S.pw_done) return;
  block_spmv<double, 1>(b, rp + b.r0, ci, val, u, u, u, s_prod, s_rsum, s_rp, s_red);
  double a = 0.0;
  const int nrows = b.r1 - b.r0;
  if ((int)threadIdx.x < nrows) {
    a = s_rsum[0][threadIdx.x];
    w[(int64_t)b.r0 + threadIdx.x] = a;
  }
  pw_block_end<FUSED>(b, S, a * a, E, s_red, s_out);
}

// The same products over column-sorted blocks: out = pw_scale * K~ w (DUAL)
// or w = K~^T u.  The power iteration runs on the layouts of the steps: at
// 500k x 2M its two products took 640 us in row-major tiles and take 260 us
// in sorted groups.
template <bool DUAL, bool FUSED>
__global__ __launch_bounds__(kThreads) void pw_sorted_kernel(const Blk* sched, InstState* st, const int32_t* ci,
                                                             const double* val, const double* src, double* out,
                                                             PowerEnd E) {
  extern __shared__ __align__(16) unsigned char sorted_lds[];
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  double* s_row = reinterpret_cast<double*>(sorted_lds);
  const Blk b = sched[blockIdx.x];
  InstState& S = st[b.inst];
  if (S.pw_done) return;
  SortedStream<double, kThreads, kPlainU, kPlainD> stream;
  stream.open(b, ci, val);
  const int nrows = b.r1 - b.r0, rs = blk_rep_shift(b), words = nrows << rs;
  const int copy = threadIdx.x & ((1 << rs) - 1);
  clear_rows(s_row, words, kThreads);
  lds_barrier();
  stream.sum(src + b.rp_off, s_row + copy, words - copy + (threadIdx.x & 63), rs);
  lds_barrier();
  const double scale = DUAL ? S.pw_scale : 1.0;
  double v = 0.0;
  for (int r = threadIdx.x; r < nrows; r += kThreads) {
    double a = 0.0;
    for (int c = 0; c < (1 << rs); ++c) a += s_row[(r << rs) + c];
    a *= scale;
    out[(int64_t)b.r0 + r] = a;
    v += a * a;
  }
  if constexpr (!DUAL) pw_block_end<FUSED>(b, S, v, E, s_red, s_out);
}

// Slice partial sums of sorted groups, part[slice][row]
template <int TPB>
__global__ __launch_bounds__(TPB) void pw_group_kernel(const Blk* sched, const InstState* st, const int32_t* ci,
                                                       const double* val, const double* src, double* part,
                                                       int64_t space) {
  extern __shared__ __align__(16) unsigned char group_lds[];
  double* s_row = reinterpret_cast<double*>(group_lds);
  const Blk b = sched[blockIdx.x];
  if (st[b.inst].pw_done) return;
  SortedStream<double, TPB, kGroupEntries / TPB, 1> stream;
  stream.open(b, ci, val);
  const int nrows = b.r1 - b.r0;
  clear_rows(s_row, nrows, TPB);
  lds_barrier();
  stream.sum(src + b.rp_off, s_row, nrows + (threadIdx.x & 63));
  lds_barrier();
  for (int r = threadIdx.x; r < nrows; r += TPB) part[(int64_t)blk_slice(b) * space + b.r0 + r] = s_row[r];
}

// Rows of sorted groups from their slices' sums
template <bool DUAL, bool FUSED>
__global__ __launch_bounds__(kThreads) void pw_part_kernel(const Blk* sched, InstState* st, const double* part,
                                                           int64_t space, double* out, PowerEnd E) {
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_out[kNS];
  const Blk b = sched[blockIdx.x];
  InstState& S = st[b.inst];
  if (S.pw_done) return;
  const double scale = DUAL ? S.pw_scale : 1.0;
  const int nsl = blk_nsl(b);
  double v = 0.0;
  for (int64_t i = (int64_t)b.r0 + threadIdx.x; i < b.r1; i += kThreads) {
    double a = 0.0;
    for (int q = 0; q < nsl; ++q) a += part[(int64_t)q * space + i];
    a *= scale;
    out[i] = a;
    v += a * a;
  }
  if constexpr (!DUAL) pw_block_end<FUSED>(b, S, v, E, s_red, s_out);
}

// one block per LP: ||w|| from the partials, then pw_update
__global__ __launch_bounds__(kThreads) void pw_control_kernel(InstState* st, const int* ids, const double* partP,
                                                              int start, int min_iters, int max_iters,
                                                              double rtol, int* done) {
  __shared__ double s_red[kThreads / 64][kNS];
  __shared__ double s_sum[kNS];
  InstState& S = st[ids[blockIdx.x]];
  if (S.pw_done) return;
  sum_partials(partP + (int64_t)S.pb0 * kNS, S.pb1 - S.pb0, s_red, s_sum);
  if (threadIdx.x == 0) pw_update(S, s_sum[0], start, min_iters, max_iters, rtol, done);
}

// ---------------------------------------------------------------------------
// iterate initialisation, results, validation
// ---------------------------------------------------------------------------

template <class T>
__global__ __launch_bounds__(kThreads) void init_primal_kernel(const Blk* schedP, const T* l, const T* u,
                                                               T* x, T* x0, uint8_t* actx) {
  const Blk b = schedP[blockIdx.x];
  const int nrows = b.r1 - b.r0;
  if ((int)threadIdx.x < nrows) {
    const int64_t j = (int64_t)b.r0 + threadIdx.x;
    const T v = clampT<T>((T)0, l[j], u[j]);
    x[j] = v;
    x0[j] = v;
    actx[j] = 255;
  }
}

template <class T>
__global__ __launch_bounds__(kThreads) void init_dual_kernel(const Blk* schedD, T* y, T* y0, uint8_t* acty) {
  const Blk b = schedD[blockIdx.x];
  const int nrows = b.r1 - b.r0;
  if ((int)threadIdx.x < nrows) {
    const int64_t i = (int64_t)b.r0 + threadIdx.x;
    y[i] = (T)0;
    y0[i] = (T)0;
    acty[i] = 255;
  }
}

template <class T>
__global__ void unscale_kernel(const T* v, const double* D, int64_t off, int64_t n, double* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = D[off + i] * (double)v[off + i];
}

template <class T>
__global__ void load_point_kernel(const double* src, T* v, T* v0, int64_t off, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    v[off + i] = (T)src[i];
    v0[off + i] = (T)src[i];
  }
}

// LPs that continue from another engine's candidates, `parts` workgroups each:
// the points, and the step sizes of a given primal weight.  One launch for
// all of them: an LP at a time (four copies and six round trips) cost 48 LPs
// 5 ms of a 73 ms solve.
template <class T>
__global__ __launch_bounds__(kThreads) void take_over_kernel(const HandOver* in, int parts, InstState* st, T* x, T* x0,
                                                             T* y, T* y0) {
  const HandOver h = in[blockIdx.x / parts];
  const int64_t first = (int64_t)(blockIdx.x % parts) * kThreads + threadIdx.x, step = (int64_t)parts * kThreads;
  auto at = [&](const void* p, int64_t i) {
    return (T)(h.fp32 ? (double)((const float*)p)[i] : ((const double*)p)[i]);
  };
  for (int64_t j = first; j < h.n; j += step) x[h.col0 + j] = x0[h.col0 + j] = at(h.x, j);
  for (int64_t i = first; i < h.m; i += step) y[h.row0 + i] = y0[h.row0 + i] = at(h.y, i);
  if (first == 0 && h.omega > 0.0 && isfinite(h.omega)) {
    InstState& S = st[h.inst];
    S.omega = h.omega;
    S.tau = S.eta / h.omega;
    S.sigma = S.eta * h.omega;
  }
}

template <class T>
__global__ void copy_state_kernel(const T* src, double* dst, int64_t off, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (double)src[off + i];
}

__global__ void set_limit_status_kernel(InstState* st, int* status_out, int ninst, int code) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < ninst && st[i].status == ST_RUNNING) {
    st[i].status = code;
    status_out[i] = code;
  }
}

// ---------------------------------------------------------------------------
// explicit instantiations
// ---------------------------------------------------------------------------

template __global__ void primal_step<double>(IterArgs<double>, int);
template __global__ void primal_step<float>(IterArgs<float>, int);
template __global__ void dual_step<double>(IterArgs<double>, int);
template __global__ void dual_step<float>(IterArgs<float>, int);
template __global__ void primal_slice_step<double, 256>(IterArgs<double>, int);
template __global__ void primal_slice_step<double, 512>(IterArgs<double>, int);
template __global__ void primal_slice_step<double, 1024>(IterArgs<double>, int);
template __global__ void primal_slice_step<float, 256>(IterArgs<float>, int);
template __global__ void primal_slice_step<float, 512>(IterArgs<float>, int);
template __global__ void primal_slice_step<float, 1024>(IterArgs<float>, int);
template __global__ void dual_slice_step<double, 256>(IterArgs<double>, int);
template __global__ void dual_slice_step<double, 512>(IterArgs<double>, int);
template __global__ void dual_slice_step<double, 1024>(IterArgs<double>, int);
template __global__ void dual_slice_step<float, 256>(IterArgs<float>, int);
template __global__ void dual_slice_step<float, 512>(IterArgs<float>, int);
template __global__ void dual_slice_step<float, 1024>(IterArgs<float>, int);
template __global__ void cast_kernel<float>(const double*, float*, int64_t);
template __global__ void resident_steps<double, 256>(IterArgs<double>, int);
template __global__ void resident_steps<double, 1024>(IterArgs<double>, int);
template __global__ void resident_steps<float, 256>(IterArgs<float>, int);
template __global__ void resident_steps<float, 1024>(IterArgs<float>, int);
template __global__ void scale_primal_kernel<double>(const Blk*, const double*, const double*, const double*,
                                                     const double*, double*, double*, double*, double*);
template __global__ void scale_primal_kernel<float>(const Blk*, const double*, const double*, const double*,
                                                    const double*, float*, float*, float*, double*);
template __global__ void scale_dual_kernel<double>(const Blk*, const double*, const double*, double*, double*);
template __global__ void scale_dual_kernel<float>(const Blk*, const double*, const double*, float*, double*);
template __global__ void init_primal_kernel<double>(const Blk*, const double*, const double*, double*,
                                                    double*, uint8_t*);
template __global__ void init_primal_kernel<float>(const Blk*, const float*, const float*, float*, float*,
                                                   uint8_t*);
template __global__ void init_dual_kernel<double>(const Blk*, double*, double*, uint8_t*);
template __global__ void init_dual_kernel<float>(const Blk*, float*, float*, uint8_t*);
template __global__ void unscale_kernel<double>(const double*, const double*, int64_t, int64_t, double*);
template __global__ void unscale_kernel<float>(const float*, const double*, int64_t, int64_t, double*);
template __global__ void load_point_kernel<double>(const double*, double*, double*, int64_t, int64_t);
template __global__ void load_point_kernel<float>(const double*, float*, float*, int64_t, int64_t);
template __global__ void take_over_kernel<double>(const HandOver*, int, InstState*, double*, double*, double*, double*);
template __global__ void take_over_kernel<float>(const HandOver*, int, InstState*, float*, float*, float*, float*);
template __global__ void copy_state_kernel<double>(const double*, double*, int64_t, int64_t);
template __global__ void copy_state_kernel<float>(const float*, double*, int64_t, int64_t);

}  // namespace halp
