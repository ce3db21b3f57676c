// Host-side engine of the HIP solver.  This translation unit also holds the
// kernels (included below), so every launch resolves inside one code object.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "engine.h"
#include "kernels.hip"
#include "layout_kernels.hip"

namespace halp {

#define HIPCHECK(expr)                                                                       \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      throw Error(-3, std::string(#expr) + ": " + hipGetErrorString(e_));                    \
  } while (0)

static inline unsigned nblk(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// first-fit allocator over one space
class RangeAlloc {
 public:
  explicit RangeAlloc(int64_t cap = 0) : cap_(cap) {
    if (cap > 0) free_[0] = cap;
  }
  int64_t alloc(int64_t len) {
    if (len <= 0) return 0;
    for (auto it = free_.begin(); it != free_.end(); ++it) {
      if (it->second >= len) {
        const int64_t at = it->first, rest = it->second - len;
        free_.erase(it);
        if (rest > 0) free_[at + len] = rest;
        return at;
      }
    }
    return -1;
  }
  void release(int64_t at, int64_t len) {
    if (len <= 0) return;
    auto it = free_.emplace(at, len).first;
    auto nx = std::next(it);
    if (nx != free_.end() && it->first + it->second == nx->first) {
      it->second += nx->second;
      free_.erase(nx);
    }
    if (it != free_.begin()) {
      auto pv = std::prev(it);
      if (pv->first + pv->second == it->first) {
        pv->second += it->second;
        free_.erase(it);
      }
    }
  }
  bool can(int64_t len) const {
    if (len <= 0) return true;
    for (auto& kv : free_)
      if (kv.second >= len) return true;
    return false;
  }

 private:
  int64_t cap_;
  std::map<int64_t, int64_t> free_;
};

// ---------------------------------------------------------------------------
// device memory
//
// Every buffer of an engine comes from dalloc or, where it lives only for a
// call, from talloc.  Normally dalloc is hipMalloc;
// inside a WorkspaceScope (the allocation-free entry point) the buffers are
// carved out of `scratch`, a static device array, by a stack allocator: a
// freed block is reclaimed once every block above it is freed too (the
// engine frees its temporaries in the reverse order of their allocation).
// Carved blocks are cleared to zero on the workspace's stream, as fresh
// device memory would be.
//
// An allocation and a release of 16 MiB or more take 0.3 ms each whatever the
// size (4 GiB: 0.42 and 0.39 ms), so the engine's own buffers are one
// allocation (Engine::carve), and talloc carves its blocks out of one
// allocation per TempScope; a block that does not fit there, or is taken
// outside a scope, is a dalloc.  128 LPs of 2-8k rows, creation 67 -> 60 ms
// and release 9.9 -> 0.4 ms (221 allocations -> 9).  The engine's work on the blocks is
// ordered by its one stream, also across blocks that share an address; the
// scope's end waits for it (hipFree).
// ---------------------------------------------------------------------------

static __device__ __align__(256) char scratch[kWorkspaceBytes];

struct Workspace {
  char* base = nullptr;    // this device's copy of `scratch` (from hipGetSymbolAddress), or a TempScope's memory
  size_t size = 0, used = 0, peak = 0;
  hipStream_t stream = nullptr;
  std::vector<std::pair<size_t, bool>> blocks;  // (offset, freed) in allocation order
  std::vector<void*> extra;  // of a TempScope: blocks that did not fit its memory

  bool fits(size_t b) const { return b <= size - used; }
  char* take(size_t b) {
    char* p = base + used;
    blocks.push_back({used, false});
    used += b;
    peak = std::max(peak, used);
    return p;
  }
  bool give_back(void* p) {
    if ((char*)p < base || (char*)p >= base + size) return false;
    const size_t off = (size_t)((char*)p - base);
    for (auto& bl : blocks)
      if (bl.first == off) bl.second = true;
    while (!blocks.empty() && blocks.back().second) {
      used = blocks.back().first;
      blocks.pop_back();
    }
    return true;
  }
};
static thread_local Workspace* t_ws = nullptr;    // of the thread's WorkspaceScope
static thread_local Workspace* t_temp = nullptr;  // of the thread's TempScope

static inline size_t aligned_bytes(size_t bytes) { return (bytes + 255) & ~size_t(255); }

// Address of this device's copy of `scratch`; looked up once per device with
// that device current (the array's host-side name is not a device address).
static char* scratch_base(int device) {
  static std::mutex mu;
  static std::map<int, char*> base;
  std::lock_guard<std::mutex> lk(mu);
  auto it = base.find(device);
  if (it != base.end()) return it->second;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p)
    throw Error(-3, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
  base[device] = (char*)p;
  return (char*)p;
}

static void* ws_alloc(size_t bytes) {
  Workspace& w = *t_ws;
  const size_t b = aligned_bytes(bytes);
  if (!w.fits(b))
    throw Error(-2, "static workspace exhausted: " + std::to_string(w.used + b) + " bytes needed of " +
                        std::to_string((long long)kWorkspaceBytes));
  char* p = w.take(b);
  const hipError_t e = hipMemsetAsync(p, 0, b, w.stream);
  if (e != hipSuccess) throw Error(-3, std::string("hipMemsetAsync: ") + hipGetErrorString(e));
  return p;
}

template <class P>
static void dalloc(P** p, int64_t count) {
  *p = nullptr;
  if (count <= 0) count = 1;
  if (t_ws) {
    *p = (P*)ws_alloc(sizeof(P) * (size_t)count);
    return;
  }
  hipError_t e = hipMalloc((void**)p, sizeof(P) * (size_t)count);
  if (e != hipSuccess && t_temp && t_temp->base && t_temp->used == 0) {
    // the thread's temporary memory is not in use just now
    (void)hipGetLastError();
    (void)hipFree(t_temp->base);
    t_temp->base = nullptr;
    t_temp->size = 0;
    e = hipMalloc((void**)p, sizeof(P) * (size_t)count);
  }
  if (e != hipSuccess) throw Error(-2, std::string("device allocation failed: ") + hipGetErrorString(e));
}

// temporaries of a call (TempScope)
template <class P>
static void talloc(P** p, int64_t count) {
  const size_t b = aligned_bytes(sizeof(P) * (size_t)std::max<int64_t>(count, 1));
  if (t_temp && t_temp->fits(b)) {
    *p = (P*)t_temp->take(b);
  } else if (t_temp) {
    t_temp->extra.push_back(nullptr);
    dalloc(p, count);
    t_temp->extra.back() = (void*)*p;
  } else {
    dalloc(p, count);
  }
}

template <class P>
static void dfree(P*& p) {
  if (p && !(t_ws && t_ws->give_back((void*)p)) && !(t_temp && t_temp->give_back((void*)p))) {
    if (t_temp) {
      auto& extra = t_temp->extra;
      extra.erase(std::remove(extra.begin(), extra.end(), (void*)p), extra.end());
    }
    (void)hipFree((void*)p);
  }
  p = nullptr;
}

// While it lives, what talloc takes on this thread is freed with it at the
// latest, also where an exception passes by, and comes out of the memory that
// reserve() got.  If that cannot be had in one piece (or inside another scope or
// a WorkspaceScope) talloc allocates block by block; so it does once dalloc has
// found no memory left and taken that back.
class TempScope {
 public:
  explicit TempScope(size_t bytes = 0) {
    if (t_ws || t_temp) return;
    t_temp = &w_;
    reserve(bytes);
  }
  ~TempScope() {
    if (t_temp != &w_) return;
    t_temp = nullptr;
    for (void* p : w_.extra) (void)hipFree(p);
    (void)hipFree(w_.base);
  }
  bool reserve(size_t bytes) {
    void* p = nullptr;
    if (t_temp != &w_ || bytes == 0) return false;
    if (hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    w_.base = (char*)p;
    w_.size = bytes;
    return true;
  }
  TempScope(const TempScope&) = delete;
  TempScope& operator=(const TempScope&) = delete;

 private:
  Workspace w_;
};

WorkspaceScope::WorkspaceScope(hipStream_t stream) {
  if (t_ws) throw Error(-4, "nested use of the static workspace");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) throw Error(-3, "hipGetDevice failed");
  std::unique_ptr<Workspace> w(new Workspace());
  w->base = scratch_base(dev);
  w->size = (size_t)kWorkspaceBytes;
  w->stream = stream;
  t_ws = w.release();
}

WorkspaceScope::~WorkspaceScope() {
  delete t_ws;
  t_ws = nullptr;
}

size_t WorkspaceScope::peak() const { return t_ws ? t_ws->peak : 0; }

}  // namespace halp

#include "radix_sort.hip"

namespace halp {

// Workgroup schedule of one LP's rows: consecutive rows are packed into
// "stream" blocks of at most NB entries and kMaxRows rows; a row with more
// than NB entries gets a "long" block.  Every LP gets at least one block so
// that its controller always runs.  gid counts blocks from 0 (offset when the
// schedules of all LPs are concatenated).
static void build_blocks(const int32_t* rp, int64_t nrows, int64_t base, int inst, int NB, int max_rows,
                         std::vector<Blk>& out) {
  const size_t first = out.size();
  int64_t start = 0, acc = 0;
  auto emit = [&](int64_t a, int64_t b, int kind) {
    Blk k;
    k.r0 = (int32_t)(base + a);
    k.r1 = (int32_t)(base + b);
    k.inst = inst;
    k.meta = blk_meta(kind, 1, 0);
    k.gid = (int32_t)(out.size() - first);
    k.rp_off = 0;
    k.p0 = rp[a];
    k.pn = rp[b] - rp[a];
    out.push_back(k);
  };
  for (int64_t r = 0; r < nrows; ++r) {
    const int64_t len = (int64_t)rp[r + 1] - rp[r];
    if (len > NB) {
      if (r > start) emit(start, r, BK_STREAM);
      emit(r, r + 1, BK_LONG);
      start = r + 1;
      acc = 0;
      continue;
    }
    if (acc + len > NB || (r - start) >= max_rows) {
      if (r > start) emit(start, r, BK_STREAM);
      start = r;
      acc = 0;
    }
    acc += len;
  }
  if (nrows > start) emit(start, nrows, BK_STREAM);
  if (out.size() == first) emit(0, 0, BK_STREAM);
}

// Column-sliced schedule of one LP's rows.  cnt[r * kSlices + s] counts row
// r's entries in column slice s.  Rows are grouped (at most max_rows rows)
// so that every slice of a group holds at most NB entries (a row with more
// gets a group of its own and "long" slice blocks).  Each group has kSlices
// slice blocks in `sl` whose entries are stored group-major, then
// slice-major, then row-major starting at entry position nz0.  `grp` gets
// epilogue blocks (nsl = kSlices, part_rows rows each) that add up the
// slice partial sums.  Row pointers of slice blocks go to brp (positions from brp_base);
// dst[r * kSlices + s] receives the first position of row r's slice s.
static void build_sliced(const int32_t* cnt, int64_t nrows, int64_t base, int inst, int NB, int max_rows,
                         int part_rows, int64_t nz0,
                         int64_t brp_base, std::vector<Blk>& grp, std::vector<Blk>& sl,
                         std::vector<int32_t>& brp, std::vector<int32_t>& dst) {
  std::vector<std::pair<int64_t, int64_t>> groups;
  int64_t start = 0;
  int64_t acc[kSlices] = {0};
  auto flush = [&](int64_t e) {
    if (e > start) groups.emplace_back(start, e);
    start = e;
    for (int q = 0; q < kSlices; ++q) acc[q] = 0;
  };
  for (int64_t r = 0; r < nrows; ++r) {
    const int32_t* c = cnt + r * kSlices;
    bool big = false, over = (r - start) >= max_rows;
    for (int q = 0; q < kSlices; ++q) {
      big |= c[q] > NB;
      over |= acc[q] + c[q] > NB;
    }
    if (big) {
      flush(r);
      groups.emplace_back(r, r + 1);
      start = r + 1;
      continue;
    }
    if (over) flush(r);
    for (int q = 0; q < kSlices; ++q) acc[q] += c[q];
  }
  flush(nrows);
  if (groups.empty()) groups.emplace_back(0, 0);
  dst.assign(nrows * kSlices, 0);
  int64_t pos = nz0;
  // epilogue blocks: consecutive rows, independent of the groups
  for (int64_t a = 0; a < std::max<int64_t>(nrows, 1); a += part_rows) {
    Blk ep;
    ep.r0 = (int32_t)(base + a);
    ep.r1 = (int32_t)(base + std::min<int64_t>(a + part_rows, nrows));
    ep.inst = inst;
    ep.meta = blk_meta(BK_STREAM, kSlices, 0) | kBlkPart;
    ep.gid = (int32_t)grp.size();
    ep.rp_off = 0;
    ep.p0 = 0;
    ep.pn = 0;
    grp.push_back(ep);
  }
  for (size_t g = 0; g < groups.size(); ++g) {
    const int64_t a = groups[g].first, e = groups[g].second;
    Blk ep;
    ep.r0 = (int32_t)(base + a);
    ep.r1 = (int32_t)(base + e);
    ep.inst = inst;
    ep.gid = (int32_t)g;
    for (int q = 0; q < kSlices; ++q) {
      Blk k = ep;
      k.rp_off = (int32_t)(brp_base + (int64_t)brp.size());
      k.p0 = (int32_t)pos;
      int64_t mx = 0;
      for (int64_t r = a; r < e; ++r) {
        brp.push_back((int32_t)pos);
        dst[r * kSlices + q] = (int32_t)pos;
        pos += cnt[r * kSlices + q];
        mx = std::max<int64_t>(mx, cnt[r * kSlices + q]);
      }
      brp.push_back((int32_t)pos);
      k.pn = (int32_t)(pos - k.p0);
      k.meta = blk_meta((e - a == 1 && mx > NB) ? BK_LONG : BK_STREAM, kSlices, q);
      sl.push_back(k);
    }
  }
}

// Column-sorted blocks per product, at most, and rows per block, at least, of
// an LP that shares the launches with `live` LPs in all.  A lone LP gets one
// block per CU: more blocks only repeat the chain of loads a block starts with
// (20k x 70k: 256 blocks 16.0 us per iteration, 512 17.6, 128 19.2; 100k x
// 400k: 42.8, 45.6, 45.3), and a block of a small LP is over soon however few
// rows it has (2.4k x 8k: 16 rows or more 10.4 us, 64 or more 12.0).  In a
// batch the launches are full anyway, and fewer, larger blocks share more
// lines of the gathered vector (128 LPs: 16 blocks each 146 us, 24 151, 32
// 158, 64 173; 48 LPs: 16 blocks 56.4, 24 54.5, 32 58.8).  Engines re-block
// their running LPs as LPs finish (refine_layouts).
static void plain_shape(int64_t live, int64_t* max_blocks, int64_t* min_rows) {
  live = std::max<int64_t>(live, 1);
  *max_blocks = std::max<int64_t>(16, std::min<int64_t>(kCUs, 4 * kCUs / live));
  *min_rows = std::max<int64_t>(16, std::min<int64_t>(256, 8 * live));
}

// Entries that one sort of plain blocks takes together at most (temp_bytes).
constexpr int64_t kSortRun = 1 << 26;
// temporary memory per entry of a transpose and its radix sort
constexpr int64_t kTransposeBytes = 29;

// Most blocks of K^T over the LPs of an add for which the last block of a power
// iteration ends it itself (pw_block_end).  Up to as many row-major tiles the
// power iteration runs on those, before the layouts: its kernels are then bound
// by latency, and small LPs have more tiles than sorted blocks (creation of
// 60 x 120 1.03 ms against 1.13 on its two sorted blocks, 2.4k x 8k 1.90
// against 2.05; 100k x 400k 5.95 on tiles, 5.33 on sorted blocks).
constexpr int kPowerFuse = 512;

struct Slot {
  bool used = false;
  int64_t n = 0, m = 0, m_eq = 0, nnz = 0;
  int64_t row0 = 0, col0 = 0, nz0 = 0;
  std::vector<Blk> bP, bD;  // one block per row group (inst field = slot id, gid local)
  std::vector<Blk> bPS, bDS;  // slice blocks of sliced groups (empty when not sliced)
  int64_t brpP0 = 0, brpPn = 0, brpD0 = 0, brpDn = 0;  // ranges in the brp spaces
  int rowsP = 0, rowsD = 0;  // rows of the largest sorted group of K^T / K (0: not grouped)
  int64_t plainP = 0, plainD = 0;  // blocks K^T's / K's rows were cut into for column-sorted blocks (0: none)
  bool watched = false;
  bool reported = false;
};

template <class T>
class Engine final : public EngineBase {
 public:
  Engine(const Options& opt, hipStream_t s, int64_t cap_m, int64_t cap_n, int64_t cap_nnz, int slots)
      : opt_(opt), stream_(s), MS_(cap_m), NS_(cap_n), NZ_(cap_nnz), nslots_(slots),
        am_(cap_m), an_(cap_n), az_(cap_nnz), abK_(2 * kSlices * cap_m), abKT_(2 * kSlices * cap_n),
        slots_(slots) {
    try {
      allocate();
    } catch (...) {
      release_all();
      throw;
    }
  }
  ~Engine() override {
    if (stream_) (void)hipStreamSynchronize(stream_);
    for (hipEvent_t e : pev_) (void)hipEventDestroy(e);
    release_all();
  }

  hipStream_t stream() const override { return stream_; }
  int64_t n_of(int id) const override { return slots_.at(id).n; }
  int64_t m_of(int id) const override { return slots_.at(id).m; }
  int live() const override {
    int c = 0;
    for (auto& s : slots_) c += s.used;
    return c;
  }

  int64_t footprint(int64_t n, int64_t m, int64_t nnz) const override {
    // as allocate() sizes the spaces: per row K_rp, three FP64 and ten (twelve
    // with sorted blocks) compute-type vectors, the activity byte and the
    // slice row pointers; per variable the same for K^T's side
    const int64_t s = sizeof(T);
    const int64_t brp = opt_.slice_min_bytes >= 0 ? 2 * kSlices * 4 : 0;
    const int64_t ev = opt_.plain_sort ? 2 * s : 0;
    const int64_t per_row = 4 + 3 * 8 + 10 * s + ev + 1 + brp, per_col = 4 + 5 * 8 + 11 * s + ev + 1 + brp;
    const int64_t per_nz = 8 + 16 + (sizeof(T) == 8 ? 0 : 2 * s);
    return per_row * (m + 1) + per_col * (n + 1) + per_nz * nnz;
  }
  KernelTimes kernel_times() const override { return ktimes_; }
  bool fits(int64_t n, int64_t m, int64_t nnz) const override {
    int free_slots = 0;
    for (auto& s : slots_) free_slots += !s.used;
    return free_slots > 0 && am_.can(m + 1) && an_.can(n + 1) && az_.can(nnz);
  }
  bool fits_empty(int64_t n, int64_t m, int64_t nnz) const override {
    return nslots_ > 0 && m + 1 <= MS_ && n + 1 <= NS_ && nnz <= NZ_;
  }

  std::vector<int> add(const std::vector<Problem>& probs, bool on_device, bool partial) override;
  void set_params(const std::vector<int>& ids, double tol, int64_t max_iter,
                  int64_t stall_checks = 0) override;
  void set_params(const std::vector<int>& ids, double tol, const std::vector<int64_t>& max_iter,
                  int64_t stall_checks) override;
  std::vector<Result> results(const std::vector<int>& ids) override;
  void take_over(const EngineBase& src, const std::vector<int>& src_ids, const std::vector<int>& ids,
                 const std::vector<double>& omega) override;
  Candidate candidate(int id) const override {
    const Slot& S = slots_[id];
    return {xT + S.col0, yT + S.row0, sizeof(T) == 4};
  }
  void run(double time_limit_s) override;
  std::vector<int> advance(int chunks) override;
  void remove(const std::vector<int>& ids) override;
  Result result(int id) override;
  void solution(int id, double* x, double* y, bool to_device) override;
  void certificate(int id, double* ray, bool to_device) override;
  Norm norm(int id) const override { return {true, h_st_[id].sigma_hat, h_st_[id].pw_iter}; }
  void export_point(int id, double* x, double* y, double* omega) override;
  void stored_matrix(int id, bool transpose, int32_t* rp, int32_t* ci, double* val) override;
  void refine_layouts() override {
    HIPCHECK(hipStreamSynchronize(stream_));
    reblock_for(h_status[0]);
  }
  void import_point(int id, const double* x, const double* y, double omega) override;

 private:
  void allocate();
  size_t carve(char* base);
  void release_all();
  void release_slots(const std::vector<int>& ids);
  void rebuild_schedules();
  void pin_to_xcds(std::vector<Blk>& v, const std::vector<std::pair<int, int>>& ranges) const;
  void launch_slices(bool dual, const IterArgs<T>& A, int step);
  template <bool DUAL>
  void launch_group(unsigned g, int tpb, size_t lds, const IterArgs<T>& A, int step);
  int ldsP_ = 0, ldsD_ = 0;  // rows of the largest sorted group in the current schedules
  int tpbP_ = 256, tpbD_ = 256;  // threads per workgroup of the sorted-group kernels
  bool batchedP_ = true, batchedD_ = true;  // and whether they run the entries as a pipeline
  template <bool DUAL>
  void launch_sorted(const IterArgs<T>& A, int step);
  int ldsPB_ = 0, ldsDB_ = 0;      // LDS words of the largest column-sorted block in the current schedules
  int tpbPB_ = 256, tpbDB_ = 256;  // threads per workgroup of the column-sorted blocks' kernels
  void mark_streaming(const std::vector<int>& live, std::initializer_list<std::vector<Blk>*> lists) const;
  int scheduled_ = 0;          // LPs in the current schedules
  bool compacted_ = false;     // current schedules leave finished LPs out
  const int* finished_ = nullptr;  // status words used to leave finished LPs out (compaction)
  void launch_chunk();
  void collect_times();
  void validate_device(const std::vector<Problem>& probs, std::vector<int64_t>& nnzs);
  void load_device(const std::vector<Problem>& probs, const std::vector<int>& ids);
  void download_rows(const std::vector<int>& ids, bool dual, std::vector<std::vector<int32_t>>& out);
  void transpose_group(int64_t z0, int64_t nnz, int64_t c0, int64_t c1, const std::vector<Blk>& bD);
  int preprocess(const std::vector<int>& ids, const std::vector<Problem>& probs, const std::vector<Blk>& nP,
                 const std::vector<Blk>& nD, const std::vector<int4>& nr, std::vector<double>& norms);
  void power_iterate(const std::vector<int>& ids, int running);
  void finish_states(const std::vector<int>& ids, const std::vector<double>& norms);
  void slice_matrix(int id, bool dual);
  void need_partials(bool dual, int nsl);
  void group_sorted(int id, bool dual, const int32_t* hrp, int nsl, int64_t ngroups, int64_t cap);
  bool group_shape(int64_t nrows, int64_t width, int nsl_min, int* nsl, int64_t* ngroups, int64_t* cap) const;
  int group_lds_rows(bool dual) const;
  // An LP that resident_steps can step.  It does so where all LPs of the
  // schedule are small (the kernel of a chunk would otherwise hold up the
  // larger ones' steps) and K and K^T one column-sorted block each.  Timed
  // engines (profile) step every LP in the kernels they time.
  bool small(const Slot& S) const {
    const int64_t rows = std::min<int64_t>({(int64_t)opt_.sort_rows, kSortRowsPlain, kResRows});
    return opt_.plain_sort && opt_.profile == 0 && S.m > 0 && S.nnz > 0 && S.m <= rows && S.n <= rows &&
           S.nnz <= (int64_t)kResRows * kResEntries;
  }
  bool all_small(const std::vector<int>& ids) const {
    return std::all_of(ids.begin(), ids.end(), [&](int id) { return small(slots_[id]); });
  }
  void recut(const std::vector<int>& ids, int64_t max_blocks, int64_t min_rows, bool solo);
  // temporary memory of a sort of nnz entries into blocks: keys and positions
  // twice over and once more for the radix sort, its counts, and the values
  // (44.5 bytes per entry; lists of blocks take the rest)
  static int64_t temp_bytes(int64_t nnz) { return 45 * nnz + (1 << 14); }
  std::vector<Blk> cut_blocks(int id, bool dual, const int32_t* rp, int64_t max_blocks, int64_t min_rows, int* rb,
                              int* cb) const;
  void sort_blocks(const std::vector<int>& ids, bool dual, const std::vector<const int32_t*>& rps, int64_t max_blocks,
                   int64_t min_rows, bool reblock, int64_t max_entries);
  void reblock_for(const int* status);
  IterArgs<T> args() const;
  std::vector<InstState> states(const std::vector<int>& ids);

  Options opt_;
  hipStream_t stream_;
  int64_t MS_, NS_, NZ_;
  int nslots_;
  RangeAlloc am_, an_, az_, abK_, abKT_;
  std::vector<Slot> slots_;
  int64_t g_next_ = 0;  // index of the next step to launch

  char* mem_ = nullptr;  // the engine's buffers (carve)
  // nnz-space
  int32_t *K_ci = nullptr, *KT_ci = nullptr;
  double *K_v64 = nullptr, *KT_v64 = nullptr;
  T *K_v = nullptr, *KT_v = nullptr;
  // m-space
  int32_t* K_rp = nullptr;
  double *q_o = nullptr, *Dr = nullptr, *fm = nullptr;
  T *q = nullptr, *y = nullptr, *y0 = nullptr, *yT = nullptr, *dy = nullptr, *kxbar = nullptr,
    *kxp = nullptr, *cy1 = nullptr, *cy2 = nullptr, *ys = nullptr;
  // n-space
  int32_t* KT_rp = nullptr;
  double *c_o = nullptr, *l_o = nullptr, *u_o = nullptr, *Dc = nullptr, *fn = nullptr;
  T *c = nullptr, *l = nullptr, *u = nullptr, *x = nullptr, *x0 = nullptr, *xbar = nullptr,
    *xT = nullptr, *ktyp = nullptr, *cx1 = nullptr, *cx2 = nullptr, *xs = nullptr;
  // column-sliced layout
  int32_t *brpK = nullptr, *brpKT = nullptr;
  T *spartD = nullptr, *spartP = nullptr;  // slice partial sums, allocated on first use
  int nslD_ = 0, nslP_ = 0;                // slices they hold
  T *kt1_ = nullptr, *kt2_ = nullptr, *kx1_ = nullptr, *kx2_ = nullptr;  // sorted blocks' eval products
  uint8_t *actx = nullptr, *acty = nullptr;  // activity at the last check (two-stage diagnostics)
  Blk *d_schedPS = nullptr, *d_schedDS = nullptr;
  int64_t capPS_ = 0, capDS_ = 0, nPS_ = 0, nDS_ = 0;
  // control
  InstState* d_st = nullptr;
  int* d_status = nullptr;
  int* d_cnt = nullptr;
  int64_t* d_gbase = nullptr;
  Blk *d_schedP = nullptr, *d_schedD = nullptr, *d_schedPB = nullptr, *d_schedDB = nullptr,
      *d_schedPE = nullptr, *d_schedDE = nullptr;
  int64_t capP_ = 0, capD_ = 0, nP_ = 0, nD_ = 0;
  int64_t capPB_ = 0, capDB_ = 0, nPB_ = 0, nDB_ = 0;  // column-sorted blocks (sorted_step)
  Blk* d_schedR = nullptr;
  int64_t capR_ = 0, nR_ = 0;  // small LPs (resident_steps), two blocks each
  int tpbR_ = 256;             // threads per workgroup there
  size_t ldsR_ = 0;            // and its dynamic LDS
  int64_t capPE_ = 0, capDE_ = 0, nPE_ = 0, nDE_ = 0;  // rows of sliced products (part_step)
  int64_t cap_partP_ = 0, cap_partD_ = 0;              // blocks that partP / partD hold sums of
  double *partP = nullptr, *partD = nullptr;
  int* h_status[2] = {nullptr, nullptr};
  hipEvent_t ev_[2] = {nullptr, nullptr};
  bool ws_ = false;  // buffers come from the static workspace (no events, no pinned memory)
  bool sched_dirty_ = true;
  hipGraphExec_t gexec_ = nullptr;
  hipGraph_t graph_ = nullptr;
  std::vector<InstState> h_st_;
  int64_t chunk_count_ = 0;
  std::vector<hipEvent_t> pev_;  // 6 events per step of one chunk, reused by each timed chunk
  bool pev_pending_ = false;     // pev_ holds a timed chunk not yet added to ktimes_
  bool pev_slices_[2] = {false, false};  // the timed chunk launched primal / dual slice kernels
  double pev_size_[3] = {0, 0, 0};       // nnz, n, m of the LPs in the timed chunk's schedules
  double sched_size_[3] = {0, 0, 0};     // the same for the current schedules
  KernelTimes ktimes_;
};

// Places the engine's buffers one after the other from `base` (each on a
// 256-byte boundary); returns their size.
template <class T>
size_t Engine<T>::carve(char* base) {
  size_t at = 0;
  auto take = [&](auto** p, int64_t count) {
    *p = (std::remove_reference_t<decltype(*p)>)((uintptr_t)base + at);
    at += aligned_bytes(sizeof(**p) * (size_t)std::max<int64_t>(count, 1));
  };
  take(&K_ci, NZ_);
  take(&KT_ci, NZ_);
  take(&K_v64, NZ_);
  take(&KT_v64, NZ_);
  if (sizeof(T) == 8) {
    K_v = (T*)K_v64;
    KT_v = (T*)KT_v64;
  } else {
    take(&K_v, NZ_);
    take(&KT_v, NZ_);
  }
  take(&K_rp, MS_);
  for (double** p : {&q_o, &Dr, &fm}) take(p, MS_);
  for (T** p : {&q, &y, &y0, &yT, &dy, &kxbar, &kxp, &cy1, &cy2, &ys}) take(p, MS_);
  take(&KT_rp, NS_);
  for (double** p : {&c_o, &l_o, &u_o, &Dc, &fn}) take(p, NS_);
  for (T** p : {&c, &l, &u, &x, &x0, &xbar, &xT, &ktyp, &cx1, &cx2, &xs}) take(p, NS_);
  take(&actx, NS_);
  take(&acty, MS_);
  if (opt_.plain_sort) {
    for (T** p : {&kx1_, &kx2_}) take(p, MS_);
    for (T** p : {&kt1_, &kt2_}) take(p, NS_);
  }
  // row pointers of row-major slice tiles: only where products may be sliced
  const bool may_slice = opt_.slice_min_bytes >= 0;
  take(&brpK, may_slice ? 2 * kSlices * MS_ : 1);
  take(&brpKT, may_slice ? 2 * kSlices * NS_ : 1);
  take(&d_st, nslots_);
  take(&d_status, nslots_);
  take(&d_cnt, nslots_);
  take(&d_gbase, 1);
  return at;
}

template <class T>
void Engine<T>::allocate() {
  dalloc(&mem_, (int64_t)carve(nullptr));
  carve(mem_);
  HIPCHECK(hipMemsetAsync(d_cnt, 0, sizeof(int) * nslots_, stream_));
  HIPCHECK(hipMemsetAsync(d_status, 0, sizeof(int) * nslots_, stream_));
  HIPCHECK(hipMemsetAsync(d_st, 0, sizeof(InstState) * nslots_, stream_));
  // a zeroed state reads as running: park every slot until an LP is added
  set_limit_status_kernel<<<nblk(nslots_), 256, 0, stream_>>>(d_st, d_status, nslots_, ST_ITER_LIMIT);
  HIPCHECK(hipGetLastError());
  const int64_t gb = -(int64_t)opt_.chunk;
  HIPCHECK(hipMemcpyAsync(d_gbase, &gb, sizeof(int64_t), hipMemcpyHostToDevice, stream_));
  ws_ = t_ws != nullptr;
  for (int i = 0; i < 2; ++i) {
    if (ws_) {
      // static workspace: ordinary host memory, status reads synchronise the stream
      h_status[i] = new int[nslots_];
    } else {
      HIPCHECK(hipHostMalloc((void**)&h_status[i], sizeof(int) * nslots_, hipHostMallocDefault));
      HIPCHECK(hipEventCreateWithFlags(&ev_[i], hipEventDisableTiming));
    }
    std::memset(h_status[i], 0, sizeof(int) * nslots_);
  }
  h_st_.resize(nslots_);
  // sorted groups keep up to kSortRows row sums in dynamic LDS
  const int lds_max = (int)(sizeof(double) * (kSortRows + kSpareWords));
  for (const void* f : {(const void*)sorted_group_step<T, true, 256, true>, (const void*)sorted_group_step<T, true, 256, false>,
                        (const void*)sorted_group_step<T, true, 512, true>, (const void*)sorted_group_step<T, true, 512, false>,
                        (const void*)sorted_group_step<T, true, 1024, true>, (const void*)sorted_group_step<T, true, 1024, false>,
                        (const void*)sorted_group_step<T, false, 256, true>, (const void*)sorted_group_step<T, false, 256, false>,
                        (const void*)sorted_group_step<T, false, 512, true>, (const void*)sorted_group_step<T, false, 512, false>,
                        (const void*)sorted_group_step<T, false, 1024, true>,
                        (const void*)sorted_group_step<T, false, 1024, false>})
    HIPCHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max));
  for (const void* f : {(const void*)sorted_step<T, true, 128, 1>, (const void*)sorted_step<T, false, 128, 1>,
                        (const void*)sorted_step<T, true, 256, kPlainD>, (const void*)sorted_step<T, true, 512, kPlainD>,
                        (const void*)sorted_step<T, false, 256, kPlainD>, (const void*)sorted_step<T, false, 512, kPlainD>})
    HIPCHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(double) * (kSortWordsPlain + kSpareWords)));
  // row sums of both products with their copies, and the gathered vectors
  const int lds_res = 2 * (int)sizeof(double) * kSortWordsPlain + 2 * (int)sizeof(T) * kResRows;
  for (const void* f : {(const void*)resident_steps<T, 256>, (const void*)resident_steps<T, kResRows>})
    HIPCHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds_res));
  for (const void* f : {(const void*)pw_group_kernel<512>, (const void*)pw_group_kernel<1024>})
    HIPCHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max));
  for (const void* f : {(const void*)pw_sorted_kernel<true, false>, (const void*)pw_sorted_kernel<false, true>,
                        (const void*)pw_sorted_kernel<false, false>})
    HIPCHECK(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(double) * (kSortWordsPlain + kSpareWords)));
  HIPCHECK(hipStreamSynchronize(stream_));
}

template <class T>
void Engine<T>::release_all() {
  if (gexec_) (void)hipGraphExecDestroy(gexec_);
  if (graph_) (void)hipGraphDestroy(graph_);
  gexec_ = nullptr;
  graph_ = nullptr;
  dfree(spartD);
  dfree(spartP);
  dfree(d_schedPS);
  dfree(d_schedDS);
  dfree(d_schedP);
  dfree(d_schedD);
  dfree(d_schedPB);
  dfree(d_schedDB);
  dfree(d_schedR);
  dfree(d_schedPE);
  dfree(d_schedDE);
  dfree(partP);
  dfree(partD);
  dfree(mem_);
  for (int i = 0; i < 2; ++i) {
    if (h_status[i]) {
      if (ws_) delete[] h_status[i];
      else (void)hipHostFree(h_status[i]);
    }
    h_status[i] = nullptr;
    if (ev_[i]) (void)hipEventDestroy(ev_[i]);
    ev_[i] = nullptr;
  }
}

template <class T>
IterArgs<T> Engine<T>::args() const {
  IterArgs<T> A;
  A.K_rp = K_rp;
  A.K_ci = K_ci;
  A.K_v = K_v;
  A.KT_rp = KT_rp;
  A.KT_ci = KT_ci;
  A.KT_v = KT_v;
  A.brpK = brpK;
  A.brpKT = brpKT;
  A.spartD = spartD;
  A.spartP = spartP;
  A.nslD = nslD_;
  A.nslP = nslP_;
  A.kt1 = kt1_;
  A.kt2 = kt2_;
  A.kx1 = kx1_;
  A.kx2 = kx2_;
  A.MS = MS_;
  A.NS = NS_;
  A.c = c;
  A.l = l;
  A.u = u;
  A.Dc = Dc;
  A.x = x;
  A.x0 = x0;
  A.xbar = xbar;
  A.xT = xT;
  A.ktyp = ktyp;
  A.cx1 = cx1;
  A.cx2 = cx2;
  A.xs = xs;
  A.actx = actx;
  A.q = q;
  A.Dr = Dr;
  A.y = y;
  A.y0 = y0;
  A.yT = yT;
  A.dy = dy;
  A.kxbar = kxbar;
  A.kxp = kxp;
  A.cy1 = cy1;
  A.cy2 = cy2;
  A.ys = ys;
  A.acty = acty;
  A.st = d_st;
  A.gbase = d_gbase;
  A.cnt = d_cnt;
  A.status_out = d_status;
  A.partP = partP;
  A.partD = partD;
  A.schedP = d_schedP;
  A.schedD = d_schedD;
  A.schedPB = d_schedPB;
  A.schedDB = d_schedDB;
  A.schedPE = d_schedPE;
  A.schedDE = d_schedDE;
  A.schedR = d_schedR;
  A.schedPS = d_schedPS;
  A.schedDS = d_schedDS;
  return A;
}

// ---------------------------------------------------------------------------
// input validation and canonical CSR on the host
// ---------------------------------------------------------------------------

struct HostCSR {
  std::vector<int32_t> rp, ci;
  std::vector<double> val;
};

// At the start of a cache line: the loop over the entries is a few instructions
// long, and where it lies across lines the checks of 24 submitted LPs of 500 x
// 20,000 take 8.2 ms instead of 7.2, by the size of whatever is linked before it.
__attribute__((aligned(64))) static void validate_host(const Problem& p, HostCSR& canon, bool& use_canon) {
  const int64_t m = p.m_eq + p.m_ineq, n = p.n;
  if (n < 1 || p.m_eq < 0 || p.m_ineq < 0) throw Error(-1, "sizes must satisfy n >= 1, m_eq >= 0, m_ineq >= 0");
  if (!p.rp || (m > 0 && (!p.c || !p.rhs)) || !p.c || !p.lb || !p.ub)
    throw Error(-1, "null input pointer");
  if (p.rp[0] != 0) throw Error(-1, "row_ptr[0] must be 0");
  for (int64_t i = 0; i < m; ++i)
    if (p.rp[i + 1] < p.rp[i]) throw Error(-1, "row_ptr must be non-decreasing");
  const int64_t nnz = p.rp[m];
  if (nnz > 0 && (!p.ci || !p.val)) throw Error(-1, "null column or value array");
  bool sorted = true;
  for (int64_t i = 0; i < m; ++i) {
    for (int64_t e = p.rp[i]; e < p.rp[i + 1]; ++e) {
      const int64_t cidx = p.ci[e];
      if (cidx < 0 || cidx >= n) throw Error(-1, "column index out of range");
      if (!std::isfinite(p.val[e])) throw Error(-1, "non-finite matrix value");
      if (e > p.rp[i] && cidx <= p.ci[e - 1]) sorted = false;
    }
  }
  for (int64_t i = 0; i < m; ++i)
    if (!std::isfinite(p.rhs[i])) throw Error(-1, "non-finite right-hand side");
  for (int64_t j = 0; j < n; ++j) {
    if (!std::isfinite(p.c[j])) throw Error(-1, "non-finite objective");
    const double a = p.lb[j], b = p.ub[j];
    if (std::isnan(a) || std::isnan(b) || a > b || a == INFINITY || b == -INFINITY)
      throw Error(-1, "invalid bounds (NaN, lb > ub, lb = +inf or ub = -inf)");
  }
  use_canon = !sorted;
  if (sorted) return;
  // sort each row by column and sum duplicate entries
  canon.rp.assign(m + 1, 0);
  canon.ci.clear();
  canon.val.clear();
  std::vector<std::pair<int32_t, double>> row;
  for (int64_t i = 0; i < m; ++i) {
    row.clear();
    for (int64_t e = p.rp[i]; e < p.rp[i + 1]; ++e) row.emplace_back(p.ci[e], p.val[e]);
    std::stable_sort(row.begin(), row.end(),
                     [](const std::pair<int32_t, double>& a, const std::pair<int32_t, double>& b) {
                       return a.first < b.first;
                     });
    for (size_t k = 0; k < row.size(); ++k) {
      if (k > 0 && row[k].first == canon.ci.back()) {
        canon.val.back() += row[k].second;
      } else {
        canon.ci.push_back(row[k].first);
        canon.val.push_back(row[k].second);
      }
    }
    canon.rp[i + 1] = (int32_t)canon.ci.size();
  }
}

void validate_host_problem(const Problem& p) {
  HostCSR canon;
  bool uc = false;
  validate_host(p, canon, uc);
}

// ---------------------------------------------------------------------------
// add LPs
// ---------------------------------------------------------------------------

template <class T>
void Engine<T>::transpose_group(int64_t z0, int64_t nnz, int64_t c0, int64_t c1,
                                const std::vector<Blk>& bD) {
  if (nnz > 0) {
    Blk* d_b = nullptr;
    int32_t *rowid = nullptr, *vin = nullptr, *vout = nullptr;
    uint32_t *keys = nullptr, *kout = nullptr;
    talloc(&d_b, (int64_t)bD.size());
    talloc(&rowid, nnz);
    talloc(&keys, nnz);
    talloc(&kout, nnz);
    talloc(&vin, nnz);
    talloc(&vout, nnz);
    HIPCHECK(hipMemcpyAsync(d_b, bD.data(), sizeof(Blk) * bD.size(), hipMemcpyHostToDevice, stream_));
    row_ids_kernel<<<(unsigned)bD.size(), kThreads, 0, stream_>>>(d_b, K_rp, z0, rowid);
    iota_kernel<<<nblk(nnz), 256, 0, stream_>>>(vin, nnz);
    // keys: columns relative to the LP's first column; a stable sort keeps
    // each column's entries in row order
    shift_copy_kernel<<<nblk(nnz), 256, 0, stream_>>>((int32_t*)keys, K_ci + z0, nnz, -c0);
    HIPCHECK(hipGetLastError());
    std::vector<int> shifts;
    radix_shifts(shifts, 0, bits_for(c1 - c0));
    radix_sort_pairs<uint32_t>(keys, vin, kout, vout, nnz, shifts, stream_);
    transpose_gather_kernel<double><<<nblk(nnz), 256, 0, stream_>>>(vout, rowid, K_v64, z0, nnz, KT_ci,
                                                                     KT_v64);
    transpose_rowptr_kernel<<<nblk(c1 - c0 + 1), 256, 0, stream_>>>(kout, nnz, z0, c0, c1, KT_rp);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(stream_));
    dfree(vout);
    dfree(vin);
    dfree(kout);
    dfree(keys);
    dfree(rowid);
    dfree(d_b);
  } else {
    std::vector<int32_t> h(c1 - c0 + 1, (int32_t)z0);
    HIPCHECK(hipMemcpyAsync(KT_rp + c0, h.data(), sizeof(int32_t) * h.size(), hipMemcpyHostToDevice,
                            stream_));
    HIPCHECK(hipStreamSynchronize(stream_));
  }
}

// Checks device-resident LPs (the first one at fault throws) and reads their
// entry counts.
template <class T>
void Engine<T>::validate_device(const std::vector<Problem>& probs, std::vector<int64_t>& nnzs) {
  std::vector<LpInput> in;
  for (const Problem& p : probs)
    in.push_back({p.rp, p.ci, p.val, p.c, p.rhs, p.lb, p.ub, p.m_eq + p.m_ineq, p.n, 0, 0, 0, 0});
  if (in.empty()) return;
  LpInput* d_in = nullptr;
  int2* d_ends = nullptr;
  int* d_flags = nullptr;
  const int64_t most = (int64_t)in.size();
  talloc(&d_in, most);
  talloc(&d_ends, most);
  talloc(&d_flags, most);
  HIPCHECK(hipMemcpyAsync(d_in, in.data(), sizeof(LpInput) * in.size(), hipMemcpyHostToDevice, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  // on the null stream, after the caller's work there that may still write the inputs
  std::vector<int2> ends(in.size());
  row_ends_kernel<<<nblk(most), 256, 0, nullptr>>>(d_in, (int)most, d_ends);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipMemcpy(ends.data(), d_ends, sizeof(int2) * in.size(), hipMemcpyDeviceToHost));
  bool bad_ends = false;  // of the LP after the last of `in`
  int64_t largest = 1;
  for (size_t k = 0; k < in.size(); ++k) {
    if (ends[k].x != 0 || ends[k].y < 0) {
      bad_ends = true;
      in.resize(k);
      break;
    }
    in[k].nnz = nnzs[k] = ends[k].y;
    largest = std::max({largest, in[k].nnz, in[k].m, in[k].n});
  }
  std::vector<int> flags(in.size(), 0);
  if (!in.empty()) {
    const int parts = parts_for(largest, in.size());
    HIPCHECK(hipMemcpyAsync(d_in, in.data(), sizeof(LpInput) * in.size(), hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemsetAsync(d_flags, 0, sizeof(int) * in.size(), stream_));
    validate_lps_kernel<<<(unsigned)(in.size() * parts), kThreads, 0, stream_>>>(d_in, parts, d_flags);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipMemcpyAsync(flags.data(), d_flags, sizeof(int) * in.size(), hipMemcpyDeviceToHost, stream_));
    HIPCHECK(hipStreamSynchronize(stream_));
  }
  dfree(d_flags);
  dfree(d_ends);
  dfree(d_in);
  for (const int f : flags) {
    if (f & 1) throw Error(-1, "row_ptr must be non-decreasing from 0 to nnz");
    if (f & 2) throw Error(-1, "device CSR needs in-range, strictly increasing column indices per row");
    if (f & 4) throw Error(-1, "non-finite matrix value");
    if (f & 8) throw Error(-1, "non-finite objective or right-hand side");
    if (f & 16) throw Error(-1, "invalid bounds (NaN, lb > ub, lb = +inf or ub = -inf)");
  }
  if (bad_ends) throw Error(-1, "row_ptr must start at 0 and end at nnz >= 0");
}

// Copies device-resident LPs into their places.
template <class T>
void Engine<T>::load_device(const std::vector<Problem>& probs, const std::vector<int>& ids) {
  std::vector<LpInput> in;
  int64_t largest = 1;
  for (size_t k = 0; k < ids.size(); ++k) {
    const Problem& p = probs[k];
    const Slot& S = slots_[ids[k]];
    in.push_back({p.rp, p.ci, p.val, p.c, p.rhs, p.lb, p.ub, S.m, S.n, S.nnz, S.row0, S.col0, S.nz0});
    largest = std::max({largest, S.nnz, S.m, S.n});
  }
  LpInput* d_in = nullptr;
  talloc(&d_in, (int64_t)in.size());
  HIPCHECK(hipMemcpyAsync(d_in, in.data(), sizeof(LpInput) * in.size(), hipMemcpyHostToDevice, stream_));
  const int parts = parts_for(largest, in.size());
  load_lps_kernel<<<(unsigned)(in.size() * parts), kThreads, 0, stream_>>>(d_in, parts, K_rp, K_ci, K_v64, q_o, c_o, l_o,
                                                                          u_o, Dr, Dc);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_in);
}

// Row pointers of the LPs' K (dual) or K^T on the host, one copy per run of
// neighbouring LPs.
template <class T>
void Engine<T>::download_rows(const std::vector<int>& ids, bool dual, std::vector<std::vector<int32_t>>& out) {
  auto at = [&](size_t k) { return dual ? slots_[ids[k]].row0 : slots_[ids[k]].col0; };
  auto len = [&](size_t k) { return (dual ? slots_[ids[k]].m : slots_[ids[k]].n) + 1; };
  std::vector<int32_t> all;
  for (size_t k = 0; k < ids.size();) {
    size_t e = k + 1;
    while (e < ids.size() && at(e) == at(e - 1) + len(e - 1)) ++e;
    all.resize(at(e - 1) + len(e - 1) - at(k));
    HIPCHECK(hipMemcpyAsync(all.data(), (dual ? K_rp : KT_rp) + at(k), sizeof(int32_t) * all.size(),
                            hipMemcpyDeviceToHost, stream_));
    HIPCHECK(hipStreamSynchronize(stream_));
    for (size_t t = k; t < e; ++t)
      out[t].assign(all.begin() + (at(t) - at(k)), all.begin() + (at(t) - at(k)) + len(t));
    k = e;
  }
}

template <class T>
std::vector<int> Engine<T>::add(const std::vector<Problem>& probs_in, bool on_device, bool partial) {
  std::vector<Problem> probs(probs_in);
  constexpr int NB = Tile<T>::NB;
  std::vector<int> ids;
  HIPCHECK(hipStreamSynchronize(stream_));
  TempScope temp;
  // 1. validate and reserve
  std::vector<HostCSR> canon(probs.size());
  std::vector<char> use_canon(probs.size(), 0);
  std::vector<int64_t> nnzs(probs.size());
  if (!on_device) {
    for (size_t k = 0; k < probs.size(); ++k) {
      bool uc = false;
      validate_host(probs[k], canon[k], uc);
      use_canon[k] = uc;
      nnzs[k] = (uc ? canon[k].rp.data() : probs[k].rp)[probs[k].m_eq + probs[k].m_ineq];
    }
  } else {
    validate_device(probs, nnzs);
  }
  // the slots are given back if anything below throws
  struct Undo {
    Engine* eng;
    std::vector<int>* ids;
    ~Undo() {
      if (!ids || ids->empty()) return;
      (void)hipStreamSynchronize(eng->stream_);
      try {
        eng->release_slots(*ids);
      } catch (...) {  // no host memory for the lists of free ranges
      }
    }
  } undo{this, &ids};
  for (size_t k = 0; k < probs.size(); ++k) {
    const Problem& p = probs[k];
    const int64_t m = p.m_eq + p.m_ineq;
    int id = -1;
    for (int s = 0; s < nslots_; ++s)
      if (!slots_[s].used) {
        id = s;
        break;
      }
    if (id < 0) {
      if (partial) break;
      throw Error(-2, "no free LP slot");
    }
    const int64_t r0 = am_.alloc(m + 1);
    const int64_t c0 = r0 < 0 ? -1 : an_.alloc(p.n + 1);
    const int64_t z0 = c0 < 0 ? -1 : az_.alloc(nnzs[k]);
    if (r0 < 0 || c0 < 0 || z0 < 0 || z0 + nnzs[k] > INT32_MAX) {
      if (r0 >= 0) am_.release(r0, m + 1);
      if (c0 >= 0) an_.release(c0, p.n + 1);
      if (z0 >= 0) az_.release(z0, nnzs[k]);
      if (z0 >= 0) throw Error(-1, "more than 2^31 stored entries");
      if (partial) break;
      throw Error(-2, "not enough device memory reserved for this LP");
    }
    Slot& S = slots_[id];
    S = Slot();
    S.used = true;
    S.n = p.n;
    S.m = m;
    S.m_eq = p.m_eq;
    S.nnz = nnzs[k];
    S.row0 = r0;
    S.col0 = c0;
    S.nz0 = z0;
    ids.push_back(id);
  }

  if (ids.size() < probs.size()) {
    probs.resize(ids.size());
    canon.resize(ids.size());
    use_canon.resize(ids.size());
    nnzs.resize(ids.size());
  }
  if (ids.empty()) return ids;
  int64_t total_nz = 0, largest_nz = 0;
  for (int id : ids) {
    total_nz += slots_[id].nnz;
    largest_nz = std::max(largest_nz, slots_[id].nnz);
  }
  // the LPs' blocks are sorted together, or, where memory is short, in runs that
  // take no more than the transpose and the largest LP do
  const int64_t least = std::max(kTransposeBytes * total_nz, temp_bytes(largest_nz));
  int64_t sort_run = kSortRun;
  if (!temp.reserve(std::max(least, temp_bytes(std::min(total_nz, kSortRun))))) {
    sort_run = std::min(kSortRun, (least - temp_bytes(0)) / (temp_bytes(1) - temp_bytes(0)));
    temp.reserve(least);
  }
  // 2. upload (K values in FP64, row pointers / columns shifted to space positions)
  std::vector<std::vector<int32_t>> host_rp(probs.size());
  for (size_t k = 0; k < probs.size() && !on_device; ++k) {
    const Problem& p = probs[k];
    Slot& S = slots_[ids[k]];
    const int64_t m = S.m, n = S.n, nnz = S.nnz;
    const int32_t* rp_src = use_canon[k] ? canon[k].rp.data() : p.rp;
    const int32_t* ci_src = use_canon[k] ? canon[k].ci.data() : p.ci;
    const double* v_src = use_canon[k] ? canon[k].val.data() : p.val;
    host_rp[k].resize(m + 1);
    for (int64_t i = 0; i <= m; ++i) host_rp[k][i] = (int32_t)(rp_src[i] + S.nz0);
    HIPCHECK(hipMemcpyAsync(K_rp + S.row0, host_rp[k].data(), sizeof(int32_t) * (m + 1), hipMemcpyHostToDevice,
                            stream_));
    std::vector<int32_t> cs(nnz);
    for (int64_t e = 0; e < nnz; ++e) cs[e] = (int32_t)(ci_src[e] + S.col0);
    if (nnz) {
      HIPCHECK(hipMemcpyAsync(K_ci + S.nz0, cs.data(), sizeof(int32_t) * nnz, hipMemcpyHostToDevice, stream_));
      HIPCHECK(hipMemcpyAsync(K_v64 + S.nz0, v_src, sizeof(double) * nnz, hipMemcpyHostToDevice, stream_));
    }
    HIPCHECK(hipStreamSynchronize(stream_));
    if (m) HIPCHECK(hipMemcpyAsync(q_o + S.row0, p.rhs, sizeof(double) * m, hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(c_o + S.col0, p.c, sizeof(double) * n, hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(l_o + S.col0, p.lb, sizeof(double) * n, hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(u_o + S.col0, p.ub, sizeof(double) * n, hipMemcpyHostToDevice, stream_));
    fill_kernel<<<nblk(m + 1), 256, 0, stream_>>>(Dr + S.row0, m + 1, 1.0);
    fill_kernel<<<nblk(n + 1), 256, 0, stream_>>>(Dc + S.col0, n + 1, 1.0);
  }
  if (on_device) {
    load_device(probs, ids);
    download_rows(ids, true, host_rp);
  }
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(stream_));

  // 3. dual schedules, transpose, primal schedules
  for (size_t k = 0; k < probs.size(); ++k) {
    Slot& S = slots_[ids[k]];
    build_blocks(host_rp[k].data(), S.m, S.row0, ids[k], NB, opt_.tile_rows, S.bD);
    // host_rp holds space positions; build_blocks only uses differences
  }
  // contiguous groups transpose together
  size_t k = 0;
  while (k < probs.size()) {
    size_t e = k + 1;
    while (e < probs.size()) {
      const Slot& A = slots_[ids[e - 1]];
      const Slot& B = slots_[ids[e]];
      if (B.row0 != A.row0 + A.m + 1 || B.col0 != A.col0 + A.n + 1 || B.nz0 != A.nz0 + A.nnz) break;
      ++e;
    }
    const Slot& F = slots_[ids[k]];
    const Slot& L = slots_[ids[e - 1]];
    std::vector<Blk> bD;
    for (size_t t = k; t < e; ++t) bD.insert(bD.end(), slots_[ids[t]].bD.begin(), slots_[ids[t]].bD.end());
    transpose_group(F.nz0, L.nz0 + L.nnz - F.nz0, F.col0, L.col0 + L.n, bD);
    k = e;
  }
  std::vector<std::vector<int32_t>> host_rpT(probs.size());
  download_rows(ids, false, host_rpT);
  for (size_t t = 0; t < probs.size(); ++t) {
    Slot& S = slots_[ids[t]];
    build_blocks(host_rpT[t].data(), S.n, S.col0, ids[t], NB, opt_.tile_rows, S.bP);
  }

  // 4. temporary schedules of the new LPs, preprocessing, power iteration
  std::vector<Blk> nP, nD;
  std::vector<int4> nr;
  for (int id : ids) {
    const Slot& S = slots_[id];
    int4 r;
    r.x = (int)nP.size();
    nP.insert(nP.end(), S.bP.begin(), S.bP.end());
    r.y = (int)nP.size();
    r.z = (int)nD.size();
    nD.insert(nD.end(), S.bD.begin(), S.bD.end());
    r.w = (int)nD.size();
    nr.push_back(r);
  }
  compacted_ = false;
  std::vector<double> norms;
  int running = preprocess(ids, probs, nP, nD, nr, norms);
  if (running > 0 && nP.size() <= (size_t)kPowerFuse) {
    power_iterate(ids, running);
    running = 0;
  }
  // Layout of each product.  A product whose gathered vector would not stay
  // in one XCD's L2 is column-sliced: in sorted groups by default, in row-major
  // slice tiles with slice_sort = 0.  With sorted layouts on, a product with
  // more rows than one plain sorted block per CU holds is stored in sorted
  // groups of 1 or 2 slices (the fused step of plain blocks is the better one
  // as long as it fits: 100k x 400k, K^T in 256 plain blocks 36.5 us per
  // iteration, in 2 slices x 128 groups 40.0), unless its groups may not hold
  // more rows than a plain block either (20k x 70k with sort_rows = 256: K^T in
  // groups 20.0 us, in plain blocks 15.0).  The other products get
  // column-sorted plain blocks (plain_sort) or plain tiles.
  std::vector<int> plain[2];  // LPs whose K^T / K gets column-sorted plain blocks
  std::vector<const int32_t*> plain_rp[2];
  std::vector<std::pair<int, bool>> sliced;  // row-major slices, cut after the power iteration
  for (size_t t = 0; t < ids.size(); ++t) {
    const int id = ids[t];
    const Slot& S = slots_[id];
    for (const bool dual : {true, false}) {
      const int64_t nrows = dual ? S.m : S.n, width = dual ? S.n : S.m;
      // fewest slices that keep each slice of the gathered vector within
      // slice_min_bytes (1: the product need not be sliced)
      int nsl_min = 1;
      if (opt_.slice_min_bytes >= 0 && S.nnz > 0)
        while (nsl_min < kSlices && width * (int64_t)sizeof(T) > opt_.slice_min_bytes * nsl_min) nsl_min *= 2;
      const bool slice = nsl_min > 1;
      int nsl = 0;
      int64_t ngroups = 0, cap = 0;
      if (slice && !opt_.slice_sort) {
        sliced.push_back({id, dual});
      } else if (S.nnz > 0 && opt_.slice_sort && (slice || opt_.plain_sort) &&
                 group_shape(nrows, width, nsl_min, &nsl, &ngroups, &cap) &&
                 (slice || (nrows > kCUs * kSortRowsPlain && cap > kSortRowsPlain))) {
        group_sorted(id, dual, (dual ? host_rp[t] : host_rpT[t]).data(), nsl, ngroups, cap);
      } else if (opt_.plain_sort) {
        plain[dual].push_back(id);
        plain_rp[dual].push_back((dual ? host_rp[t] : host_rpT[t]).data());
      }
    }
  }
  int64_t maxb = 0, minr = 0;
  plain_shape(live(), &maxb, &minr);
  std::vector<int> used, single;  // single: small LPs in one block that now share their launches with larger ones
  for (int s = 0; s < nslots_; ++s)
    if (slots_[s].used) used.push_back(s);
  if (all_small(used)) {
    maxb = minr = 1;
  } else {
    for (int s : used)
      if (small(slots_[s]) && slots_[s].plainP == 1 && slots_[s].plainD == 1) single.push_back(s);
    recut(single, maxb, minr, false);
  }
  for (const bool dual : {true, false})
    sort_blocks(plain[dual], dual, plain_rp[dual], maxb, minr, false, sort_run);
  if (running > 0) power_iterate(ids, running);
  finish_states(ids, norms);
  for (auto& [id, dual] : sliced) slice_matrix(id, dual);
  sched_dirty_ = true;
  for (int id : ids) slots_[id].watched = true;
  undo.ids = nullptr;
  return ids;
}

template <class T>
int Engine<T>::preprocess(const std::vector<int>& ids, const std::vector<Problem>& probs, const std::vector<Blk>& nP,
                          const std::vector<Blk>& nD, const std::vector<int4>& nr, std::vector<double>& norms) {
  const int ni = (int)ids.size();
  // the spectral norm of every LP is given
  const bool given = std::all_of(probs.begin(), probs.end(), [](const Problem& p) { return p.norm.known; });
  Blk *d_nP = nullptr, *d_nD = nullptr;
  int* d_ids = nullptr;
  int4* d_nr = nullptr;
  double *d_pp = nullptr, *d_pd = nullptr;
  double* d_norms = nullptr;
  int* d_done = nullptr;
  InstState* d_src = nullptr;
  auto cleanup = [&]() {
    dfree(d_nP);
    dfree(d_nD);
    dfree(d_ids);
    dfree(d_nr);
    dfree(d_pd);
    dfree(d_pp);
    dfree(d_norms);
    dfree(d_done);
    dfree(d_src);
  };
  try {
    talloc(&d_nP, (int64_t)nP.size());
    talloc(&d_nD, (int64_t)nD.size());
    talloc(&d_ids, ni);
    talloc(&d_nr, ni);
    talloc(&d_pp, (int64_t)nP.size() * kNS);
    talloc(&d_pd, (int64_t)nD.size() * kNS);
    talloc(&d_norms, 2 * ni);
    talloc(&d_done, 1);
    talloc(&d_src, ni);
    HIPCHECK(hipMemcpyAsync(d_nP, nP.data(), sizeof(Blk) * nP.size(), hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(d_nD, nD.data(), sizeof(Blk) * nD.size(), hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(d_ids, ids.data(), sizeof(int) * ni, hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(d_nr, nr.data(), sizeof(int4) * ni, hipMemcpyHostToDevice, stream_));
    const unsigned gP = (unsigned)nP.size(), gD = (unsigned)nD.size();

    // scaling (Ruiz infinity-norm passes, then Pock-Chambolle): each pass
    // applies the factors of the one before and finds its own, a last one only
    // applies.  K's rows keep theirs where the dual iterates will be, those
    // that K^T gathers are in fm, the columns' in fn.
    const int passes = opt_.ruiz_iters + (opt_.pc_alpha > 0.0 ? 1 : 0);
    const bool words = sizeof(T) != sizeof(double);
    const RowFactors fr{words ? nullptr : (double*)y, words ? (uint32_t*)y : nullptr, words ? (uint32_t*)y0 : nullptr, fm};
    const RowFactors fc{fn, nullptr, nullptr, nullptr};
    for (int it = 0; it <= passes && passes > 0; ++it) {
      const int op = it == passes ? 2 : it == opt_.ruiz_iters ? 1 : 0;
      row_factor_kernel<<<gD, kThreads, 0, stream_>>>(d_nD, K_rp, K_ci, K_v64, op, op == 1 ? 2.0 - opt_.pc_alpha : 1.0,
                                                      it == 0, false, fn, fr, Dr);
      row_factor_kernel<<<gP, kThreads, 0, stream_>>>(d_nP, KT_rp, KT_ci, KT_v64, op, op == 1 ? opt_.pc_alpha : 1.0,
                                                      it == 0, true, fm, fc, Dc);
    }
    scale_primal_kernel<T><<<gP, kThreads, 0, stream_>>>(d_nP, Dc, c_o, l_o, u_o, c, l, u, d_pp);
    scale_dual_kernel<T><<<gD, kThreads, 0, stream_>>>(d_nD, Dr, q_o, q, d_pd);

    // layout constants for the norm and power kernels
    std::vector<InstState> src(ni);
    for (int k = 0; k < ni; ++k) {
      const Slot& S = slots_[ids[k]];
      InstState& s = src[k];
      std::memset(&s, 0, sizeof(InstState));
      s.row0 = S.row0;
      s.col0 = S.col0;
      s.nz0 = S.nz0;
      s.m = (int32_t)S.m;
      s.m_eq = (int32_t)S.m_eq;
      s.n = (int32_t)S.n;
      s.status = ST_ITER_LIMIT;  // parked until set_params
      s.pb0 = nr[k].x;  // of the temporary schedule
      s.pb1 = nr[k].y;
      s.pw_done = opt_.eta > 0.0 || given ? 1 : 0;
      if (given) {
        s.sigma_hat = probs[k].norm.sigma_hat;
        s.pw_iter = probs[k].norm.power_iters;
      }
    }
    HIPCHECK(hipMemcpyAsync(d_src, src.data(), sizeof(InstState) * ni, hipMemcpyHostToDevice, stream_));
    write_states_kernel<<<nblk(ni), 256, 0, stream_>>>(d_st, d_status, d_cnt, d_ids, d_src, ni);
    inst_norms_kernel<<<ni, kThreads, 0, stream_>>>(d_st, d_ids, d_nr, d_pp, d_pd, d_norms);

    // start of the power iteration on K~^T K~ (u in fm, w in fn)
    int done = ni;
    if (opt_.eta <= 0.0 && !given) {
      pw_start_kernel<<<gP, kThreads, 0, stream_>>>(d_nP, d_st, opt_.seed, fn, d_pp);
      HIPCHECK(hipMemsetAsync(d_done, 0, sizeof(int), stream_));
      pw_control_kernel<<<ni, kThreads, 0, stream_>>>(d_st, d_ids, d_pp, 1, opt_.power_min_iters, opt_.power_max_iters,
                                                      opt_.power_rtol, d_done);
      HIPCHECK(hipMemcpyAsync(&done, d_done, sizeof(int), hipMemcpyDeviceToHost, stream_));
    }
    if (sizeof(T) != 8) {
      for (int id : ids) {
        const Slot& S = slots_[id];
        if (S.nnz) {
          cast_kernel<T><<<nblk(S.nnz), 256, 0, stream_>>>(K_v64 + S.nz0, K_v + S.nz0, S.nnz);
          cast_kernel<T><<<nblk(S.nnz), 256, 0, stream_>>>(KT_v64 + S.nz0, KT_v + S.nz0, S.nnz);
        }
      }
    }
    init_primal_kernel<T><<<gP, kThreads, 0, stream_>>>(d_nP, l, u, x, x0, actx);
    init_dual_kernel<T><<<gD, kThreads, 0, stream_>>>(d_nD, y, y0, acty);
    HIPCHECK(hipGetLastError());

    norms.resize(2 * ni);
    HIPCHECK(hipMemcpyAsync(norms.data(), d_norms, sizeof(double) * 2 * ni, hipMemcpyDeviceToHost, stream_));
    HIPCHECK(hipStreamSynchronize(stream_));
    cleanup();
    return ni - done;
  } catch (...) {
    cleanup();
    throw;
  }
}

// Power iteration on K~^T K~ of new LPs over the blocks their products now
// have (u in fm, w in fn, the state as preprocess left it).
template <class T>
void Engine<T>::power_iterate(const std::vector<int>& ids, int running) {
  const int ni = (int)ids.size();
  // tiles, column-sorted blocks, rows and slice blocks of sorted groups, for K^T and K
  std::vector<Blk> tile[2], sorted[2], part[2], group[2];
  std::vector<int4> rg;
  int g = 0;
  size_t lds_sorted[2] = {0, 0}, lds_group[2] = {0, 0};
  for (int id : ids) {
    const Slot& S = slots_[id];
    const int g0 = g;
    for (const int d : {0, 1}) {
      for (Blk k : d ? S.bD : S.bP) {
        if (!d) k.gid = g++;  // its partial sum
        if (blk_kind(k) == BK_SORTED)
          lds_sorted[d] = std::max(lds_sorted[d], sizeof(double) * (((size_t)(k.r1 - k.r0) << blk_rep_shift(k)) + kSpareWords));
        (blk_part(k) ? part : blk_kind(k) == BK_SORTED ? sorted : tile)[d].push_back(k);
      }
      const std::vector<Blk>& sl = d ? S.bDS : S.bPS;
      group[d].insert(group[d].end(), sl.begin(), sl.end());
      for (const Blk& k : sl) lds_group[d] = std::max(lds_group[d], sizeof(double) * (size_t)(k.r1 - k.r0 + kSpareWords));
    }
    rg.push_back(make_int4(g0, g, 0, 0));
  }
  mark_streaming(ids, {&tile[0], &sorted[0], &group[0], &group[1], &tile[1], &sorted[1]});
  Blk* d_blk[8] = {nullptr};
  int* d_ids = nullptr;
  int4* d_rg = nullptr;
  double* d_pp = nullptr;
  int* d_done = nullptr;
  const std::vector<Blk>* lists[8] = {&tile[0], &sorted[0], &part[0], &group[0], &tile[1], &sorted[1], &part[1], &group[1]};
  for (int k = 0; k < 8; ++k) {
    talloc(&d_blk[k], (int64_t)lists[k]->size());
    if (!lists[k]->empty())
      HIPCHECK(hipMemcpyAsync(d_blk[k], lists[k]->data(), sizeof(Blk) * lists[k]->size(), hipMemcpyHostToDevice, stream_));
  }
  talloc(&d_ids, ni);
  talloc(&d_rg, ni);
  talloc(&d_pp, (int64_t)g * kNS);
  talloc(&d_done, 1);
  HIPCHECK(hipMemcpyAsync(d_ids, ids.data(), sizeof(int) * ni, hipMemcpyHostToDevice, stream_));
  HIPCHECK(hipMemcpyAsync(d_rg, rg.data(), sizeof(int4) * ni, hipMemcpyHostToDevice, stream_));
  HIPCHECK(hipMemsetAsync(d_done, 0, sizeof(int), stream_));
  set_ranges_kernel<<<nblk(ni), 256, 0, stream_>>>(d_st, d_ids, d_rg, ni);
  const bool fused = g <= kPowerFuse;
  const PowerEnd E{d_pp, d_cnt, d_done, opt_.power_min_iters, opt_.power_max_iters, opt_.power_rtol};
  auto groups = [&](int d, const double* src, double* sums, int64_t space) {
    const size_t nb = group[d].size();
    const int32_t* ci = d ? K_ci : KT_ci;
    const double* val = d ? K_v64 : KT_v64;
    if (nb <= (size_t)kCUs)
      pw_group_kernel<1024><<<(unsigned)nb, 1024, lds_group[d], stream_>>>(d_blk[3 + 4 * d], d_st, ci, val, src, sums, space);
    else
      pw_group_kernel<512><<<(unsigned)nb, 512, lds_group[d], stream_>>>(d_blk[3 + 4 * d], d_st, ci, val, src, sums, space);
  };
  const auto tile_back = fused ? pw_backward_kernel<true> : pw_backward_kernel<false>;
  const auto sorted_back = fused ? pw_sorted_kernel<false, true> : pw_sorted_kernel<false, false>;
  const auto part_back = fused ? pw_part_kernel<false, true> : pw_part_kernel<false, false>;
  // the slices' FP64 sums use the step's room for three vectors of type T
  static_assert(3 * sizeof(T) >= sizeof(double), "slice sums");
  double *sumsD = (double*)spartD, *sumsP = (double*)spartP;
  int done = 0;
  for (int it = 0; done < running && it < opt_.power_max_iters;) {
    for (int b = 0; b < 8 && it < opt_.power_max_iters; ++b, ++it) {
      if (!group[1].empty()) groups(1, fn, sumsD, MS_);
      if (!tile[1].empty())
        pw_forward_kernel<<<(unsigned)tile[1].size(), kThreads, 0, stream_>>>(d_blk[4], d_st, K_rp, K_ci, K_v64, fn, fm);
      if (!sorted[1].empty())
        pw_sorted_kernel<true, false><<<(unsigned)sorted[1].size(), kThreads, lds_sorted[1], stream_>>>(
            d_blk[5], d_st, K_ci, K_v64, fn, fm, E);
      if (!part[1].empty())
        pw_part_kernel<true, false><<<(unsigned)part[1].size(), kThreads, 0, stream_>>>(d_blk[6], d_st, sumsD, MS_, fm, E);
      if (!group[0].empty()) groups(0, fm, sumsP, NS_);
      if (!tile[0].empty())
        tile_back<<<(unsigned)tile[0].size(), kThreads, 0, stream_>>>(d_blk[0], d_st, KT_rp, KT_ci, KT_v64, fm, fn, E);
      if (!sorted[0].empty())
        sorted_back<<<(unsigned)sorted[0].size(), kThreads, lds_sorted[0], stream_>>>(d_blk[1], d_st, KT_ci, KT_v64, fm, fn, E);
      if (!part[0].empty())
        part_back<<<(unsigned)part[0].size(), kThreads, 0, stream_>>>(d_blk[2], d_st, sumsP, NS_, fn, E);
      if (!fused)
        pw_control_kernel<<<ni, kThreads, 0, stream_>>>(d_st, d_ids, d_pp, 0, opt_.power_min_iters, opt_.power_max_iters,
                                                        opt_.power_rtol, d_done);
    }
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipMemcpyAsync(&done, d_done, sizeof(int), hipMemcpyDeviceToHost, stream_));
    HIPCHECK(hipStreamSynchronize(stream_));
  }
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_done);
  dfree(d_pp);
  dfree(d_rg);
  dfree(d_ids);
  for (int k = 7; k >= 0; --k) dfree(d_blk[k]);
}

// Step size and primal weight of new LPs, which are parked until set_params.
template <class T>
void Engine<T>::finish_states(const std::vector<int>& ids, const std::vector<double>& norms) {
  const int ni = (int)ids.size();
  std::vector<InstState> cur = states(ids);
  for (int k = 0; k < ni; ++k) {
    InstState& s = cur[k];
    const double sh = s.sigma_hat;
    double eta;
    if (opt_.eta > 0.0) {
      eta = opt_.eta;
      s.sigma_hat = NAN;
    } else {
      eta = sh > 0.0 ? opt_.step_safety / sh : opt_.step_safety;
    }
    const double nq = norms[2 * k], nc = norms[2 * k + 1];
    double omega = 1.0;
    if (opt_.omega0 > 0.0) omega = opt_.omega0;
    else if (opt_.primal_weight && nc > 1e-10 && nq > 1e-10) omega = nc / nq;
    s.eta = eta;
    s.omega = omega;
    s.tau = eta / omega;
    s.sigma = eta * omega;
    s.reflect = opt_.method == 1;
    s.avg = opt_.method == 2;
    s.avg_b1 = opt_.avg_beta_sufficient;
    s.avg_b2 = opt_.avg_beta_necessary;
    s.kkt_anchor = NAN;
    s.kkt_prev = INFINITY;
    s.act_changes = 0;
    s.ident_iters = 0;
    s.C = opt_.check_every;
    s.primal_weight = opt_.primal_weight;
    s.beta = opt_.restart_beta;
    s.artificial = opt_.artificial_restart;
    s.restart_mode = opt_.restart_mode;
    s.fixed_len = opt_.fixed_restart_len;
    s.eps_inf = opt_.eps_infeas;
    s.r0 = NAN;
    s.status = ST_ITER_LIMIT;  // parked
    s.phase = PH_NORMAL;
    s.nrest = 0;
    s.checks = 0;
    s.ray = 0;
    s.iters = 0;
    s.kkt = NAN;
    s.best_kkt = INFINITY;
    s.best_check = 0;
    s.stall_checks = 0;
    h_st_[ids[k]] = s;
  }
  int* d_ids = nullptr;
  InstState* d_src = nullptr;
  talloc(&d_ids, ni);
  talloc(&d_src, ni);
  HIPCHECK(hipMemcpyAsync(d_ids, ids.data(), sizeof(int) * ni, hipMemcpyHostToDevice, stream_));
  HIPCHECK(hipMemcpyAsync(d_src, cur.data(), sizeof(InstState) * ni, hipMemcpyHostToDevice, stream_));
  write_states_kernel<<<nblk(ni), 256, 0, stream_>>>(d_st, d_status, d_cnt, d_ids, d_src, ni);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_src);
  dfree(d_ids);
}

// Reorders one LP's K (dual = true; slices over its variables) or K^T
// (slices over its constraints) into the column-sliced layout.
template <class T>
void Engine<T>::slice_matrix(int id, bool dual) {
  const int NB = opt_.slice_entries;
  Slot& S = slots_[id];
  const int64_t nrows = dual ? S.m : S.n;
  const int64_t r0 = dual ? S.row0 : S.col0;
  const int64_t c0 = dual ? S.col0 : S.row0;
  const int64_t len = dual ? S.n : S.m;
  const int32_t* rp = dual ? K_rp : KT_rp;
  int32_t* ci = dual ? K_ci : KT_ci;
  T* val = dual ? K_v : KT_v;
  double* v64 = dual ? K_v64 : KT_v64;
  if (nrows == 0 || S.nnz == 0) return;
  int32_t* d_cnt = nullptr;
  talloc(&d_cnt, nrows * kSlices);
  slice_count_kernel<<<nblk(nrows), 256, 0, stream_>>>(rp, ci, r0, nrows, c0, len, kSlices, d_cnt);
  std::vector<int32_t> cnt(nrows * kSlices);
  HIPCHECK(hipMemcpyAsync(cnt.data(), d_cnt, sizeof(int32_t) * cnt.size(), hipMemcpyDeviceToHost, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  std::vector<Blk> grp, sl;
  std::vector<int32_t> brp, dst;
  RangeAlloc& ab = dual ? abK_ : abKT_;
  // reserve the worst case first, then return what is unused
  const int64_t cap = kSlices * (2 * nrows + 1);
  const int64_t at = ab.alloc(cap);
  if (at < 0) {
    dfree(d_cnt);
    throw Error(-2, "no room for sliced row pointers");
  }
  build_sliced(cnt.data(), nrows, r0, id, NB, opt_.slice_rows, kPartRows(dual), S.nz0, at, grp, sl, brp, dst);
  if ((int64_t)brp.size() > cap) throw Error(-3, "sliced row pointer overflow");
  ab.release(at + (int64_t)brp.size(), cap - (int64_t)brp.size());
  (dual ? S.brpD0 : S.brpP0) = at;
  (dual ? S.brpDn : S.brpPn) = (int64_t)brp.size();
  int32_t* brp_d = dual ? brpK : brpKT;
  HIPCHECK(hipMemcpyAsync(brp_d + at, brp.data(), sizeof(int32_t) * brp.size(), hipMemcpyHostToDevice, stream_));
  int32_t* d_dst = nullptr;
  int32_t* ci2 = nullptr;
  T* v2 = nullptr;
  double* v642 = nullptr;
  talloc(&d_dst, nrows * kSlices);
  talloc(&ci2, S.nnz);
  talloc(&v2, S.nnz);
  if (sizeof(T) != 8) talloc(&v642, S.nnz);
  HIPCHECK(hipMemcpyAsync(d_dst, dst.data(), sizeof(int32_t) * dst.size(), hipMemcpyHostToDevice, stream_));
  // the scatter writes positions nz0..nz0+nnz; shift the temporaries by -nz0
  slice_scatter_kernel<T><<<nblk(nrows), 256, 0, stream_>>>(rp, ci, val, v64, r0, nrows, c0, len, d_dst,
                                                            ci2 - S.nz0, v2 - S.nz0,
                                                            v642 ? v642 - S.nz0 : nullptr);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipMemcpyAsync(ci + S.nz0, ci2, sizeof(int32_t) * S.nnz, hipMemcpyDeviceToDevice, stream_));
  HIPCHECK(hipMemcpyAsync(val + S.nz0, v2, sizeof(T) * S.nnz, hipMemcpyDeviceToDevice, stream_));
  if (v642) HIPCHECK(hipMemcpyAsync(v64 + S.nz0, v642, sizeof(double) * S.nnz, hipMemcpyDeviceToDevice, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_cnt);
  dfree(d_dst);
  dfree(ci2);
  dfree(v2);
  dfree(v642);
  if (dual) {
    S.bD = grp;
    S.bDS = sl;
  } else {
    S.bP = grp;
    S.bPS = sl;
  }
  need_partials(dual, kSlices);
}

// Room for the partial sums of a product of nsl slices (three vectors at an
// eval step).
template <class T>
void Engine<T>::need_partials(bool dual, int nsl) {
  T*& p = dual ? spartD : spartP;
  int& have = dual ? nslD_ : nslP_;
  if (nsl <= have) return;
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(p);
  have = 0;
  dalloc(&p, 3 * (int64_t)nsl * (dual ? MS_ : NS_));
  have = nsl;
}


// Blocks that the rows of a column-sorted product are cut into: of min_rows
// rows on average, or of the entries that min_rows rows of kLongRows entries
// have, whichever are more (us per iteration by rows alone and by entries too:
// 200 x 200k of 5000 entries a row 42.0 and 20.1, 50 x 100k of 2000 21.4 and
// 12.2, K^T of 20k x 300 15.7 and 10.8, a batch of 64 of 50 x 20k 93 and 58;
// limits of 32 to 128 entries differ by less than 10%, 256 is slower).
static int64_t plain_blocks(int64_t nrows, int64_t nnz, int64_t max_blocks, int64_t min_rows) {
  const int64_t want = std::max<int64_t>((nrows + min_rows - 1) / min_rows, nnz / (kLongRows * min_rows));
  return std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(max_blocks, nrows), want));
}

// Smaller column-sorted blocks for the LPs still running (status) when few
// are left (plain_shape for their number), so that the launches keep the
// CUs busy.  Products in sorted groups, column slices or plain tiles keep
// their layout.
template <class T>
void Engine<T>::reblock_for(const int* status) {
  std::vector<int> run;
  for (int s = 0; s < nslots_; ++s)
    if (slots_[s].used && status[s] == ST_RUNNING) run.push_back(s);
  if (run.empty()) return;
  int64_t maxb = 0, minr = 0;
  plain_shape((int64_t)run.size(), &maxb, &minr);
  recut(run, maxb, minr, all_small(run));
}

// Lays the plain sorted blocks of the LPs `ids` out anew where the shape calls
// for more of them, or (solo: all of them are small) for one block each.
template <class T>
void Engine<T>::recut(const std::vector<int>& ids, int64_t maxb, int64_t minr, bool solo) {
  if (solo) maxb = minr = 1;
  for (const bool dual : {false, true}) {
    std::vector<int> todo;
    std::vector<std::vector<int32_t>> rp;
    std::vector<const int32_t*> rps;
    int64_t largest = 0;
    for (int s : ids) {
      const Slot& S = slots_[s];
      const int64_t cur = dual ? S.plainD : S.plainP, nrows = dual ? S.m : S.n;
      if (cur == 0 || (solo ? cur == 1 : plain_blocks(nrows, S.nnz, maxb, minr) <= cur)) continue;
      todo.push_back(s);
      largest = std::max(largest, S.nnz);
      rp.emplace_back(nrows + 1);
      HIPCHECK(hipMemcpy(rp.back().data(), (dual ? K_rp : KT_rp) + (dual ? S.row0 : S.col0),
                         sizeof(int32_t) * (nrows + 1), hipMemcpyDeviceToHost));
    }
    if (todo.empty()) continue;
    for (auto& v : rp) rps.push_back(v.data());
    // the schedules are of the old blocks, also where an allocation below throws
    // with some LPs laid out anew
    sched_dirty_ = true;
    compacted_ = false;
    TempScope temp(temp_bytes(largest));
    // temporary memory for the largest of them, as a server's budget allows
    sort_blocks(todo, dual, rps, maxb, minr, true, largest);
  }
}

// Column-sorted blocks of one LP's K (dual = true) or K^T over its row pointers
// rp (space positions): rows longer than kSortedRowMax keep a block of their
// own; the other rows go to blocks of equal work, of at most min(sort_rows,
// kSortRowsPlain) rows and kSortEntries entries, whose entries are put in
// column order, each column index packed with the entry's row in the block
// (see blk_rowbits).  *rb: row bits, *cb: column bits.
template <class T>
std::vector<Blk> Engine<T>::cut_blocks(int id, bool dual, const int32_t* rp, int64_t max_blocks, int64_t min_rows,
                                       int* rb_out, int* cb_out) const {
  const Slot& S = slots_[id];
  const int64_t nrows = dual ? S.m : S.n;
  const int64_t base = dual ? S.row0 : S.col0;
  const int64_t c0 = dual ? S.col0 : S.row0;
  const int64_t width = dual ? S.n : S.m;
  std::vector<Blk> out;
  int cb = 0;
  while (((int64_t)1 << cb) < width) ++cb;
  *cb_out = cb;
  if (nrows == 0 || S.nnz == 0 || cb > kSortColBits) return out;
  // most rows per block: the packed index holds the column and the row in 32 bits
  const int64_t rows =
      std::min<int64_t>(std::min<int64_t>(opt_.sort_rows, kSortRowsPlain), (int64_t)1 << (32 - std::min(cb, 31)));
  int rb = 0;
  while (((int64_t)1 << rb) < rows) ++rb;
  *rb_out = rb;
  int64_t longest_row = 0;  // of the block being filled
  auto emit = [&](int64_t a, int64_t e, int kind) {
    Blk k;
    k.r0 = (int32_t)(base + a);
    k.r1 = (int32_t)(base + e);
    k.inst = id;
    k.gid = (int32_t)out.size();
    k.rp_off = kind == BK_SORTED ? (int32_t)c0 : 0;
    k.p0 = rp[a];
    k.pn = rp[e] - rp[a];
    // copies of the row sums where one long row gets more than 4 of 64
    // consecutive products: 8, or up to 32 while the entries are 16 times the
    // words, which have to be cleared and added up (with 32 wherever they fit: a
    // batch of 32 in blocks of 128 rows 64.2 us per iteration, so 57.1; 53.0
    // before rows this long were sorted)
    int rs = 0;
    if (kind == BK_SORTED && longest_row >= kRepRow && longest_row * 16 > k.pn &&
        ((e - a) << kMinRepShift) <= kSortWordsPlain)
      for (rs = kMinRepShift; rs < kMaxRepShift && ((e - a) << (rs + 5)) <= k.pn;) ++rs;
    k.meta = blk_meta(kind, 1, rs) | (kind == BK_SORTED ? (rb << 25) : 0);
    out.push_back(k);
    longest_row = 0;
  };
  // blocks of equal weight (entries, and kRowWeight per row for its epilogue):
  // a block ends at the row whose middle passes the next multiple of the
  // average weight
  const int64_t nblk_want = plain_blocks(nrows, S.nnz, max_blocks, min_rows);
  const double per = (double)((int64_t)S.nnz + kRowWeight * nrows) / (double)nblk_want;
  int64_t start = 0, acc = 0, cum = 0;
  double bound = per;
  for (int64_t r = 0; r < nrows; ++r) {
    const int64_t len = (int64_t)rp[r + 1] - rp[r];
    const int64_t w = len + kRowWeight;
    if (len > kSortedRowMax) {
      if (r > start) emit(start, r, BK_SORTED);
      emit(r, r + 1, BK_LONG);
      start = r + 1;
      acc = 0;
    } else {
      if (r > start && ((r - start) >= rows || acc + len > kSortEntries || (double)cum + 0.5 * (double)w > bound)) {
        emit(start, r, BK_SORTED);
        start = r;
        acc = 0;
      }
      longest_row = std::max(longest_row, len);
      acc += len;
    }
    if (r == start || start == r + 1)
      while (bound < (double)cum + 0.5 * per + (start == r + 1 ? (double)w : 0.0)) bound += per;
    cum += w;
  }
  if (nrows > start) emit(start, nrows, BK_SORTED);
  return out;
}

// Column-sorts the K (dual = true) or K^T products of the LPs `ids` into blocks
// (cut_blocks).  rps[k]: LP k's row pointers on the host.  Built on the device
// for all of them together: a 64-bit key per entry (block index, packed column
// and row) and one stable radix sort by block and column (rows of a column
// come in order), where a sort per LP spent 75 ms on a batch of 128 in kernels
// of a few microseconds.  From the row-major input (reblock false), or
// re-blocking products already in column-sorted blocks into smaller ones
// (reblock true: each entry's row and column are read back from its packed
// key).  The LPs are taken in runs of at most max_entries entries (at least
// one LP), which bounds the temporary memory.
template <class T>
void Engine<T>::sort_blocks(const std::vector<int>& ids, bool dual, const std::vector<const int32_t*>& rps,
                            int64_t max_blocks, int64_t min_rows, bool reblock, int64_t max_entries) {
  const int32_t* rpd = dual ? K_rp : KT_rp;
  int32_t* ci = dual ? K_ci : KT_ci;
  T* val = dual ? K_v : KT_v;
  double* v64 = dual ? K_v64 : KT_v64;
  size_t next = 0;
  while (next < ids.size()) {
    std::vector<int> lps;                  // of this run
    std::vector<std::vector<Blk>> blocks;  // their new blocks
    std::vector<Blk> all, sorted, old;     // for the kernels: gid holds the shift of positions into the key arrays
    std::vector<int2> where;               // reblock: each row's new block and its row in that block
    int64_t total = 0;
    int rb_min = 32, key_bits = 1;
    for (; next < ids.size(); ++next) {
      const int id = ids[next];
      const Slot& S = slots_[id];
      if (total > 0 && total + S.nnz > max_entries) break;
      int rb = 0, cb = 0;
      std::vector<Blk> out = cut_blocks(id, dual, rps[next], max_blocks, min_rows, &rb, &cb);
      if (out.empty()) continue;
      const int32_t shift = (int32_t)(total - S.nz0);
      const int64_t base = dual ? S.row0 : S.col0, nrows = dual ? S.m : S.n;
      const int first = (int)all.size();
      int32_t longest = 0;
      bool any = false;
      for (const Blk& k : out) {
        Blk d = k;
        d.gid = shift;
        all.push_back(d);
        any |= blk_kind(k) == BK_SORTED;
        if (blk_kind(k) == BK_SORTED) sorted.push_back(d);
        else longest = std::max(longest, k.pn);
      }
      if (!any) {  // nothing to sort: the blocks alone
        all.resize(first);
        Slot& W = slots_[id];
        (dual ? W.plainD : W.plainP) = 0;
        (dual ? W.bD : W.bP) = out;
        continue;
      }
      if (reblock) {
        const int32_t to_where = (int32_t)((int64_t)where.size() - base);
        for (const Blk& k : dual ? S.bD : S.bP) {
          Blk d = k;
          d.gid = shift;
          d.rp_off = to_where;
          d.meta = (k.meta & ~0xff00) | (rb << 8);
          old.push_back(d);
        }
        where.resize(where.size() + nrows);
        for (size_t bi = 0; bi < out.size(); ++bi)
          for (int32_t r = out[bi].r0; r < out[bi].r1; ++r)
            where[(int64_t)r + to_where] = make_int2(first + (int)bi, r - out[bi].r0);
      }
      rb_min = std::min(rb_min, rb);
      key_bits = std::max(key_bits, std::max(std::min(32, cb + rb), bits_for(longest)));
      total += S.nnz;
      lps.push_back(id);
      blocks.push_back(std::move(out));
    }
    if (lps.empty()) continue;
    Blk *d_all = nullptr, *d_blk = nullptr, *d_old = nullptr;
    int2* d_where = nullptr;
    int32_t *src_in = nullptr, *src_out = nullptr;
    uint64_t *key_in = nullptr, *key_out = nullptr;
    double* v_tmp = nullptr;
    const unsigned nall = (unsigned)all.size(), nseg = (unsigned)sorted.size();
    talloc(&d_all, nall);
    talloc(&d_blk, nseg);
    talloc(&key_in, total);
    talloc(&key_out, total);
    talloc(&src_in, total);
    talloc(&src_out, total);
    talloc(&v_tmp, total);
    HIPCHECK(hipMemcpyAsync(d_all, all.data(), sizeof(Blk) * nall, hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(d_blk, sorted.data(), sizeof(Blk) * nseg, hipMemcpyHostToDevice, stream_));
    if (!reblock) {
      block_keys_kernel<<<nall, kThreads, 0, stream_>>>(d_all, rpd, ci, key_in, src_in);
    } else {
      talloc(&d_old, (int64_t)old.size());
      talloc(&d_where, (int64_t)where.size());
      HIPCHECK(hipMemcpyAsync(d_old, old.data(), sizeof(Blk) * old.size(), hipMemcpyHostToDevice, stream_));
      HIPCHECK(hipMemcpyAsync(d_where, where.data(), sizeof(int2) * where.size(), hipMemcpyHostToDevice, stream_));
      reblock_keys_kernel<<<(unsigned)old.size(), kThreads, 0, stream_>>>(d_old, d_where, ci, key_in, src_in);
    }
    HIPCHECK(hipGetLastError());
    // the input is in row order within a column (entries of other blocks in
    // their own order), so a stable sort needs the column bits only
    std::vector<int> shifts;
    radix_shifts(shifts, rb_min, key_bits);
    radix_shifts(shifts, 32, 32 + bits_for((int64_t)nall - 1));
    radix_sort_pairs<uint64_t>(key_in, src_in, key_out, src_out, total, shifts, stream_);
    sorted_block_gather_kernel<<<nseg, kThreads, 0, stream_>>>(d_blk, key_out, src_out, v64, ci, v_tmp);
    sorted_block_store_kernel<T><<<nseg, kThreads, 0, stream_>>>(d_blk, v_tmp, val, v64);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(stream_));
    dfree(d_where);
    dfree(d_old);
    dfree(v_tmp);
    dfree(src_out);
    dfree(src_in);
    dfree(key_out);
    dfree(key_in);
    dfree(d_blk);
    dfree(d_all);
    for (size_t k = 0; k < lps.size(); ++k) {
      Slot& S = slots_[lps[k]];
      (dual ? S.plainD : S.plainP) = plain_blocks(dual ? S.m : S.n, S.nnz, max_blocks, min_rows);
      (dual ? S.bD : S.bP) = std::move(blocks[k]);
    }
  }
}

// Shape of a sorted-group layout for a product of nrows rows over `width`
// columns: the slice count, from nsl_min (the fewest that keep a slice of
// the gathered vector within slice_min_bytes) up to 8 for a product that
// must be sliced, else 1 or 2, and the number of row groups: the fewest that
// keep the groups' rows within *cap (the packed column index: row bits +
// column bits of a slice <= 32, Options::sort_rows and kSortRows) and leave at
// least group_blocks workgroups per product, rounded up so that every CU has
// the same number of workgroups.  Larger groups share more lines of the
// gathered vector, and more slices allow larger groups of a product with few
// rows; the slice count with the larger groups wins (a tie goes to fewer
// slices: fewer partial sums).  False when no shape fits.
template <class T>
bool Engine<T>::group_shape(int64_t nrows, int64_t width, int nsl_min, int* nsl, int64_t* ngroups, int64_t* cap) const {
  int64_t best_r = 0;
  for (int q = nsl_min; q <= (nsl_min == 1 ? 2 : kGroupSlices); q *= 2) {
    const int64_t w = (width + q - 1) / q + 1;
    int cb = 0;
    while (((int64_t)1 << cb) < w) ++cb;
    if (cb > kSortColBits) continue;
    const int64_t most = std::min<int64_t>(std::min<int64_t>(opt_.sort_rows, kSortRows), (int64_t)1 << (32 - cb));
    int64_t blocks = std::max<int64_t>((nrows + most - 1) / most * q, opt_.group_blocks);
    if (opt_.group_blocks >= kMinGroupBlocks) blocks = (blocks + kCUs - 1) / kCUs * kCUs;
    const int64_t g = std::max<int64_t>((nrows + most - 1) / most,
                                        std::min<int64_t>((blocks + q - 1) / q, (nrows + kMaxRows - 1) / kMaxRows));
    const int64_t r = (nrows + g - 1) / g;
    if (r > best_r) {
      best_r = r;
      *nsl = q;
      *ngroups = g;
      *cap = most;
    }
  }
  return best_r > 0;
}

// Rows of the largest sorted group among the live LPs' K (dual) or K^T
// products: the slice kernel's dynamic LDS holds that many row sums.
template <class T>
int Engine<T>::group_lds_rows(bool dual) const {
  int r = 0;
  for (const Slot& sl : slots_)
    if (sl.used) r = std::max(r, dual ? sl.rowsD : sl.rowsP);
  return r;
}

// Sorted groups of one LP's K (dual = true) or K^T over its row pointers hrp
// on the host (space positions): about ngroups groups of equal work (entries
// and rows), of at most cap rows and kSortEntries entries per slice on
// average, split where one slice holds most of them, each group's entries in nsl column slices, each (group, slice)
// block's entries in column order with the row of the group packed beside the
// column.  Built on the device from the row-major entries: keys, one stable
// radix sort by block and column (rows of a column come in order), values.
template <class T>
void Engine<T>::group_sorted(int id, bool dual, const int32_t* hrp, int nsl, int64_t ngroups, int64_t cap) {
  Slot& S = slots_[id];
  const int64_t nrows = dual ? S.m : S.n, r0 = dual ? S.row0 : S.col0, c0 = dual ? S.col0 : S.row0;
  const int64_t len = dual ? S.n : S.m;
  const int32_t* rp = dual ? K_rp : KT_rp;
  int32_t* ci = dual ? K_ci : KT_ci;
  T* val = dual ? K_v : KT_v;
  double* v64 = dual ? K_v64 : KT_v64;
  const int64_t nnz = S.nnz;
  if (nrows == 0 || nnz == 0) return;
  if (nsl < 1 || nsl > kGroupSlices || kGroupSlices % nsl != 0) throw Error(-3, "bad slice count");
  // a group ends at the row whose middle passes the next multiple of the
  // average work, found by bisection (the work of rows 0 .. r - 1 is
  // hrp[r] - hrp[0] + r)
  std::vector<int32_t> gstart;
  const double per = (double)(nnz + nrows) / (double)ngroups;
  const int64_t most_entries = (int64_t)kSortEntries * nsl;
  double bound = per;
  for (int64_t start = 0; start < nrows;) {
    const double cum = (double)((int64_t)hrp[start] - hrp[0] + start);
    while (bound < cum + 0.5 * per) bound += per;
    int64_t lo = start + 1, up = std::min(nrows, start + cap);  // the group's end
    while (lo < up) {
      const int64_t r = (lo + up) >> 1;
      const double mid = (double)((int64_t)hrp[r] - hrp[0] + r) + 0.5 * (double)((int64_t)hrp[r + 1] - hrp[r] + 1);
      if (mid > bound || (int64_t)hrp[r + 1] - hrp[start] > most_entries) up = r;
      else lo = r + 1;
    }
    gstart.push_back((int32_t)start);
    start = lo;
  }
  gstart.push_back((int32_t)nrows);
  const std::vector<Blk>& tiles = dual ? S.bD : S.bP;
  Blk* d_tiles = nullptr;
  talloc(&d_tiles, (int64_t)tiles.size());
  HIPCHECK(hipMemcpyAsync(d_tiles, tiles.data(), sizeof(Blk) * tiles.size(), hipMemcpyHostToDevice, stream_));
  // Where a group's entries crowd into few of its slices (a banded matrix), the
  // blocks that hold them would be few and large: a group is split while a block
  // of it holds more than 1.5 times the average of its slice's blocks (and
  // kMinSplit) and of its group's.  A block that is large because its slice is
  // (the slice's XCD has as much to do either way) or because of one long row
  // (split rows 5% slower at 500k x 1M) is left.
  const double groups0 = (double)gstart.size() - 1.0;
  double most[kGroupSlices] = {0.0};
  bool split = false;  // (a group of fewer entries is not split: nothing to count)
  for (size_t g = 0; g + 1 < gstart.size() && nsl > 1; ++g) split |= hrp[gstart[g + 1]] - hrp[gstart[g]] > kMinSplit;
  while (split) {
    const int n = (int)gstart.size() - 1;
    int32_t *d_cut = nullptr, *d_cnt = nullptr;
    talloc(&d_cut, n + 1);
    talloc(&d_cnt, (int64_t)n * nsl);
    HIPCHECK(hipMemcpyAsync(d_cut, gstart.data(), sizeof(int32_t) * gstart.size(), hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemsetAsync(d_cnt, 0, sizeof(int32_t) * n * nsl, stream_));
    group_count_kernel<<<(unsigned)tiles.size(), kThreads, 0, stream_>>>(d_tiles, rp, ci, d_cut, n, r0, c0, len, nsl, d_cnt);
    HIPCHECK(hipGetLastError());
    std::vector<int32_t> cnt((size_t)n * nsl), cut;
    HIPCHECK(hipMemcpyAsync(cnt.data(), d_cnt, sizeof(int32_t) * cnt.size(), hipMemcpyDeviceToHost, stream_));
    HIPCHECK(hipStreamSynchronize(stream_));
    dfree(d_cnt);
    dfree(d_cut);
    if (most[0] == 0.0) {
      for (size_t i = 0; i < cnt.size(); ++i) most[i % nsl] += 1.5 / groups0 * (double)cnt[i];
      for (double& v : most) v = std::max(v, (double)kMinSplit);
    }
    split = false;
    for (int g = 0; g < n; ++g) {
      const int64_t a = gstart[g], e = gstart[g + 1], total = (int64_t)hrp[e] - hrp[a];
      int64_t parts = 1;
      for (int q = 0; q < nsl; ++q) {
        const int64_t full = cnt[(size_t)g * nsl + q];
        if (2 * full * nsl > 3 * total) parts = std::max<int64_t>(parts, (int64_t)std::ceil((double)full / most[q]));
      }
      parts = std::min(parts, e - a);
      cut.push_back((int32_t)a);
      split |= parts > 1;
      // parts of equal work, of at least a row each
      for (int64_t k = 1; k < parts; ++k) {
        const double at = (double)hrp[a] + (double)a + (double)((int64_t)hrp[e] - hrp[a] + e - a) * (double)k / (double)parts;
        int64_t lo = (int64_t)cut.back() + 1, up = e - (parts - k);
        while (lo < up) {
          const int64_t r = (lo + up) >> 1;
          if ((double)hrp[r] + (double)r < at) lo = r + 1;
          else up = r;
        }
        cut.push_back((int32_t)lo);
      }
    }
    cut.push_back((int32_t)nrows);
    gstart.swap(cut);
  }
  const int ng = (int)gstart.size() - 1, nseg = ng * nsl;
  int64_t maxrows = 0;
  for (int g = 0; g < ng; ++g) maxrows = std::max<int64_t>(maxrows, gstart[g + 1] - gstart[g]);
  int rb = 0;
  while (((int64_t)1 << rb) < maxrows) ++rb;
  int32_t *d_g = nullptr, *d_off = nullptr, *src_in = nullptr, *src_out = nullptr;
  uint64_t *key_in = nullptr, *key_out = nullptr;
  double* v2 = nullptr;
  talloc(&d_g, ng + 1);
  talloc(&d_off, nseg + 1);
  talloc(&key_in, nnz);
  talloc(&key_out, nnz);
  talloc(&src_in, nnz);
  talloc(&src_out, nnz);
  talloc(&v2, nnz);
  HIPCHECK(hipMemcpyAsync(d_g, gstart.data(), sizeof(int32_t) * gstart.size(), hipMemcpyHostToDevice, stream_));
  group_keys_kernel<<<(unsigned)tiles.size(), kThreads, 0, stream_>>>(d_tiles, rp, ci, d_g, ng, r0, S.nz0, c0, len, nsl,
                                                                      rb, key_in, src_in);
  HIPCHECK(hipGetLastError());
  std::vector<int> shifts;
  radix_shifts(shifts, rb, std::min(32, bits_for((len + nsl - 1) / nsl) + rb));
  radix_shifts(shifts, 32, 32 + bits_for(nseg - 1));
  radix_sort_pairs<uint64_t>(key_in, src_in, key_out, src_out, nnz, shifts, stream_);
  segment_offsets_kernel<<<nblk(nseg + 1), 256, 0, stream_>>>(key_out, nnz, nseg, d_off);
  sorted_gather_kernel<<<nblk(nnz), 256, 0, stream_>>>(key_out, src_out, v64, nnz, ci + S.nz0, v2);
  if (sizeof(T) != 8) cast_kernel<T><<<nblk(nnz), 256, 0, stream_>>>(v2, val + S.nz0, nnz);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipMemcpyAsync(v64 + S.nz0, v2, sizeof(double) * nnz, hipMemcpyDeviceToDevice, stream_));
  std::vector<int32_t> off(nseg + 1);
  HIPCHECK(hipMemcpyAsync(off.data(), d_off, sizeof(int32_t) * off.size(), hipMemcpyDeviceToHost, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(v2);
  dfree(src_out);
  dfree(src_in);
  dfree(key_out);
  dfree(key_in);
  dfree(d_off);
  dfree(d_g);
  dfree(d_tiles);
  if (off[0] != 0 || off[nseg] != nnz) throw Error(-3, "sorted group layout does not cover the matrix");
  // step blocks (row sums from the partials) and slice blocks
  std::vector<Blk> grp, sl;
  for (int64_t a = 0; a < nrows; a += kPartRows(dual)) {
    Blk ep;
    ep.r0 = (int32_t)(r0 + a);
    ep.r1 = (int32_t)(r0 + std::min<int64_t>(a + kPartRows(dual), nrows));
    ep.inst = id;
    ep.meta = blk_meta(BK_STREAM, nsl, 0) | kBlkPart;
    ep.gid = (int32_t)grp.size();
    ep.rp_off = 0;
    ep.p0 = 0;
    ep.pn = 0;
    grp.push_back(ep);
  }
  for (int s = 0; s < nseg; ++s) {
    const int g = s / nsl, q = s % nsl;
    Blk k;
    k.r0 = (int32_t)(r0 + gstart[g]);
    k.r1 = (int32_t)(r0 + gstart[g + 1]);
    k.inst = id;
    k.gid = g;
    k.rp_off = (int32_t)(c0 + (q * len + nsl - 1) / nsl);
    k.p0 = (int32_t)(S.nz0 + off[s]);
    k.pn = off[s + 1] - off[s];
    k.meta = blk_meta(BK_STREAM, nsl, q) | (rb << 25);
    sl.push_back(k);
  }
  if (dual) {
    S.bD = grp;
    S.bDS = sl;
    S.brpD0 = 0;
    S.brpDn = 0;
    S.rowsD = (int)maxrows;
    need_partials(true, nsl);
  } else {
    S.bP = grp;
    S.bPS = sl;
    S.brpP0 = 0;
    S.brpPn = 0;
    S.rowsP = (int)maxrows;
    need_partials(false, nsl);
  }
}

template <class T>
void Engine<T>::set_params(const std::vector<int>& ids, double tol, int64_t max_iter, int64_t stall_checks) {
  set_params(ids, tol, std::vector<int64_t>(ids.size(), max_iter), stall_checks);
}

// The states of the LPs `ids`, in one copy of the slots they span.
template <class T>
std::vector<InstState> Engine<T>::states(const std::vector<int>& ids) {
  const int first = *std::min_element(ids.begin(), ids.end()), last = *std::max_element(ids.begin(), ids.end());
  std::vector<InstState> all(last - first + 1), out(ids.size());
  HIPCHECK(hipMemcpyAsync(all.data(), d_st + first, sizeof(InstState) * all.size(), hipMemcpyDeviceToHost, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  for (size_t k = 0; k < ids.size(); ++k) out[k] = all[ids[k] - first];
  return out;
}

template <class T>
void Engine<T>::set_params(const std::vector<int>& ids, double tol, const std::vector<int64_t>& max_iter,
                           int64_t stall_checks) {
  HIPCHECK(hipStreamSynchronize(stream_));
  const int ni = (int)ids.size();
  if (ni == 0) return;
  std::vector<InstState> cur = states(ids);
  for (int k = 0; k < ni; ++k) {
    InstState& s = cur[k];
    s.tol = tol;
    s.max_iter = max_iter[k];
    s.stall_checks = stall_checks;
    s.best_kkt = INFINITY;
    s.best_check = s.checks;
    if (s.status != ST_RUNNING) {
      // (re)start from the last candidate as a fresh epoch is not supported
      // for finished LPs; a parked LP starts here
      if (s.checks == 0) {
        s.status = ST_RUNNING;
        s.phase = PH_NORMAL;
        s.kbase = g_next_;
        s.tbase = g_next_;
        s.next_check = g_next_ + s.C;
      }
    }
    slots_[ids[k]].watched = true;
    slots_[ids[k]].reported = false;
  }
  TempScope temp;
  InstState* d_src = nullptr;
  int* d_ids = nullptr;
  talloc(&d_src, ni);
  talloc(&d_ids, ni);
  HIPCHECK(hipMemcpyAsync(d_src, cur.data(), sizeof(InstState) * ni, hipMemcpyHostToDevice, stream_));
  HIPCHECK(hipMemcpyAsync(d_ids, ids.data(), sizeof(int) * ni, hipMemcpyHostToDevice, stream_));
  write_states_kernel<<<nblk(ni), 256, 0, stream_>>>(d_st, d_status, d_cnt, d_ids, d_src, ni);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_src);
  dfree(d_ids);
  for (int k = 0; k < ni; ++k) h_status[0][ids[k]] = h_status[1][ids[k]] = cur[k].status;
}

// Many LPs in one schedule: each LP's blocks go to one XCD.  Workgroups are
// dispatched round-robin over the 8 XCDs, so schedule position p runs on XCD
// p % 8; LPs are assigned to 8 lanes (largest first, to the lane with the
// least work) and lane q fills positions q, q + 8, ... (padded with no-op
// blocks).  Each XCD's L2 then caches only the gathered vectors of its own
// LPs instead of every running LP's.
template <class T>
void Engine<T>::pin_to_xcds(std::vector<Blk>& v, const std::vector<std::pair<int, int>>& ranges) const {
  if (v.empty()) return;
  std::vector<int> order(ranges.size());
  std::vector<int64_t> weight(ranges.size(), 0);
  for (size_t i = 0; i < order.size(); ++i) {
    order[i] = (int)i;
    for (int p = ranges[i].first; p < ranges[i].second; ++p)
      weight[i] += v[p].pn + kRowWeight * (v[p].r1 - v[p].r0) + kBlockWeight;
  }
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return weight[a] > weight[b]; });
  std::vector<std::vector<Blk>> lane(kSlices);
  int64_t load[kSlices] = {0};
  for (int i : order) {
    int q = 0;
    for (int k = 1; k < kSlices; ++k)
      if (load[k] < load[q]) q = k;
    load[q] += weight[i];
    for (int p = ranges[i].first; p < ranges[i].second; ++p) lane[q].push_back(v[p]);
  }
  size_t len = 0;
  for (auto& l : lane) len = std::max(len, l.size());
  Blk pad{};
  pad.meta = blk_meta(BK_PAD, 1, 0);
  std::vector<Blk> out;
  out.reserve(len * kSlices);
  for (size_t r = 0; r < len; ++r)
    for (int q = 0; q < kSlices; ++q) out.push_back(r < lane[q].size() ? lane[q][r] : pad);
  v.swap(out);
}

// The vectors of a step and the matrix tiles read before the cache budget is
// used up are read normally and stay in the last-level cache from one step to
// the next; the remaining tiles are streamed with non-temporal loads, so that
// they do not evict what fits.  (A matrix pair larger than the cache read
// round-robin would otherwise evict every line before its next use.)
template <class T>
void Engine<T>::mark_streaming(const std::vector<int>& live, std::initializer_list<std::vector<Blk>*> lists) const {
  const int64_t budget = opt_.cache_budget_bytes;
  int64_t used = 0;
  for (int s : live) {
    const Slot& sl = slots_[s];
    // n-space: c, l, u, x, x0, xbar; m-space: q, y, y0; row pointers; slice partial sums
    used += (int64_t)sizeof(T) * (6 * sl.n + 3 * sl.m) + 4 * (sl.n + sl.m);
    if (!sl.bDS.empty()) used += (int64_t)sizeof(T) * blk_nsl(sl.bDS[0]) * sl.m + 4 * sl.brpDn;
    if (!sl.bPS.empty()) used += (int64_t)sizeof(T) * blk_nsl(sl.bPS[0]) * sl.n + 4 * sl.brpPn;
  }
  for (std::vector<Blk>* v : lists) {
    for (Blk& k : *v) {
      k.meta &= ~kBlkNT;
      if (blk_kind(k) == BK_PAD) continue;
      const int64_t bytes = (int64_t)k.pn * (int64_t)(sizeof(T) + 4);
      if (budget >= 0 && used + bytes > budget) k.meta |= kBlkNT;
      else used += bytes;
    }
  }
}

// Blocks that have entries.
static size_t with_entries(const std::vector<Blk>& v) {
  return (size_t)std::count_if(v.begin(), v.end(), [](const Blk& b) { return b.pn > 0; });
}

template <class T>
void Engine<T>::rebuild_schedules() {
  sched_dirty_ = true;  // until all of them are in place
  compacted_ = false;
  // P / D: tiles; PB / DB: column-sorted blocks; PE / DE: rows of sliced
  // products; PS / DS: slice blocks; R: both blocks of each small LP.  gids number an LP's step blocks of all
  // three kinds in one range.
  std::vector<Blk> P, D, PB, DB, PE, DE, PS, DS, R;
  const std::vector<Blk> none;
  std::vector<int> live;
  std::vector<int4> rg;
  std::vector<std::pair<int, int>> rP, rD, rPB, rDB;
  int gP = 0, gD = 0;
  auto append = [](std::vector<Blk>& tiles, std::vector<Blk>& sorted, std::vector<Blk>& part,
                   const std::vector<Blk>& src, int& g, std::vector<std::pair<int, int>>& rt,
                   std::vector<std::pair<int, int>>& rs) {
    const int t0 = (int)tiles.size(), s0 = (int)sorted.size();
    for (Blk k : src) {
      k.gid += g;
      (blk_part(k) ? part : blk_kind(k) == BK_SORTED ? sorted : tiles).push_back(k);
    }
    g += (int)src.size();
    rt.push_back({t0, (int)tiles.size()});
    rs.push_back({s0, (int)sorted.size()});
  };
  for (int s = 0; s < nslots_; ++s) {
    if (!slots_[s].used) continue;
    if (finished_ && finished_[s] != ST_RUNNING) continue;  // done: its blocks would only exit
    live.push_back(s);
  }
  auto one_block = [](const std::vector<Blk>& v) { return v.size() == 1 && blk_kind(v[0]) == BK_SORTED; };
  const bool solo = std::all_of(live.begin(), live.end(), [&](int s) {
    return small(slots_[s]) && one_block(slots_[s].bP) && one_block(slots_[s].bD);
  });
  for (int s : live) {
    const Slot& sl = slots_[s];
    int4 r;
    r.x = gP;
    r.z = gD;
    PS.insert(PS.end(), sl.bPS.begin(), sl.bPS.end());
    DS.insert(DS.end(), sl.bDS.begin(), sl.bDS.end());
    append(P, PB, PE, solo ? none : sl.bP, gP, rP, rPB);
    append(D, DB, DE, solo ? none : sl.bD, gD, rD, rDB);
    if (solo) {
      R.push_back(sl.bP[0]);
      R.push_back(sl.bD[0]);
    }
    r.y = gP;
    r.w = gD;
    rg.push_back(r);
  }
  for (double& v : sched_size_) v = 0.0;
  for (int s : live) {
    sched_size_[0] += (double)slots_[s].nnz;
    sched_size_[1] += (double)slots_[s].n;
    sched_size_[2] += (double)slots_[s].m;
  }
  if (opt_.xcd_pin && (int)live.size() >= kPinMinLPs) {
    pin_to_xcds(P, rP);
    pin_to_xcds(D, rD);
    pin_to_xcds(PB, rPB);
    pin_to_xcds(DB, rDB);
  }
  ldsP_ = ldsD_ = 0;
  for (int s2 : live) {
    ldsP_ = std::max(ldsP_, slots_[s2].rowsP);
    ldsD_ = std::max(ldsD_, slots_[s2].rowsD);
  }
  // threads per sorted-group workgroup: the configured count, or 1024 where
  // each CU has one workgroup (that has entries), else enough for about eight waves per CU (the
  // entries in flight are bound by the 32 KB of L1: more waves only queue)
  auto pick = [&](size_t nb) {
    if (opt_.group_threads > 0) return opt_.group_threads;
    if (nb <= (size_t)kCUs) return 1024;
    return (int64_t)kCUs * 8 * 64 / (int64_t)nb >= 512 ? 512 : 256;
  };
  tpbP_ = pick(with_entries(PS));
  tpbD_ = pick(with_entries(DS));
  // without the pipeline where many groups end before it is full (sort_rows = 32:
  // 500k x 2M 547 us per iteration against 1310, 200k x 1M 154 against 265)
  auto batched = [&](const std::vector<Blk>& v) {
    int64_t entries = 0;
    for (const Blk& k : v) entries += k.pn;
    const size_t nb = with_entries(v);
    return opt_.group_batched != 0 && !(nb > (size_t)kTinyGroups * kCUs && entries < kGroupEntries * (int64_t)nb);
  };
  batchedP_ = batched(PS);
  batchedD_ = batched(DS);
  auto words = [](const std::vector<Blk>& v) {
    int w = 1;
    for (const Blk& k : v)
      if (blk_kind(k) == BK_SORTED) w = std::max(w, (k.r1 - k.r0) << blk_rep_shift(k));
    return w;
  };
  tpbR_ = 256;
  ldsR_ = 0;
  for (size_t k = 0; k < R.size(); k += 2) {
    size_t lds = 0;
    for (const Blk& b : {R[k], R[k + 1]}) {
      lds += sizeof(double) * ((size_t)(b.r1 - b.r0) << blk_rep_shift(b)) + sizeof(T) * (size_t)(b.r1 - b.r0);
      if (b.r1 - b.r0 > 256 || b.pn > 256 * kResEntries) tpbR_ = kResRows;
    }
    ldsR_ = std::max(ldsR_, lds);
  }
  ldsPB_ = words(PB);
  ldsDB_ = words(DB);
  // threads per column-sorted block: 512 where each CU has one large block
  // (100k x 400k: 42.6 us per iteration against 43.4 with 256), else 256 (20k x
  // 70k: 16.0 against 16.3; a batch of 128: 146 against 155), and 128 with a
  // shorter pipeline for many blocks of few rows, which end before a longer one
  // is full (sort_rows = 32: a batch of 32 82.9 us per iteration against 112.5,
  // 20k x 70k 17.1 against 20.1; 4 LPs of 2.4k x 8k 11.0 against 12.2)
  auto pick_sorted = [](const std::vector<Blk>& v) {
    int64_t entries = 0;
    int rows = 0;
    for (const Blk& k : v) {
      entries += k.pn;
      rows = std::max(rows, k.r1 - k.r0);
    }
    if (v.size() > 2 * (size_t)kCUs && rows <= kTinyRows) return 128;
    return v.size() <= (size_t)kCUs && entries > 8192 * (int64_t)v.size() ? 512 : 256;
  };
  tpbPB_ = pick_sorted(PB);
  tpbDB_ = pick_sorted(DB);
  mark_streaming(live, {&P, &PB, &PS, &DS, &D, &DB});
  HIPCHECK(hipStreamSynchronize(stream_));
  // a capacity counts once its buffer exists (an allocation may throw)
  auto grow = [](auto*& d, int64_t& cap, int64_t n, int64_t words) {
    if (n <= cap) return;
    const int64_t want = std::max<int64_t>(n, 2 * cap);
    dfree(d);
    cap = 0;
    dalloc(&d, want * words);
    cap = want;
  };
  auto upload = [&](std::vector<Blk>& v, Blk*& d, int64_t& cap, int64_t& n) {
    grow(d, cap, (int64_t)v.size(), 1);
    n = (int64_t)v.size();
    if (n) HIPCHECK(hipMemcpyAsync(d, v.data(), sizeof(Blk) * n, hipMemcpyHostToDevice, stream_));
  };
  scheduled_ = (int)live.size();
  upload(P, d_schedP, capP_, nP_);
  upload(D, d_schedD, capD_, nD_);
  upload(PB, d_schedPB, capPB_, nPB_);
  upload(DB, d_schedDB, capDB_, nDB_);
  upload(R, d_schedR, capR_, nR_);
  upload(PE, d_schedPE, capPE_, nPE_);
  upload(DE, d_schedDE, capDE_, nDE_);
  upload(PS, d_schedPS, capPS_, nPS_);
  upload(DS, d_schedDS, capDS_, nDS_);
  grow(partP, cap_partP_, gP, kNS);
  grow(partD, cap_partD_, gD, kNS);
  if (!live.empty()) {
    TempScope temp;
    int* d_ids = nullptr;
    int4* d_rg = nullptr;
    talloc(&d_ids, (int64_t)live.size());
    talloc(&d_rg, (int64_t)live.size());
    HIPCHECK(hipMemcpyAsync(d_ids, live.data(), sizeof(int) * live.size(), hipMemcpyHostToDevice, stream_));
    HIPCHECK(hipMemcpyAsync(d_rg, rg.data(), sizeof(int4) * rg.size(), hipMemcpyHostToDevice, stream_));
    set_ranges_kernel<<<nblk((int64_t)live.size()), 256, 0, stream_>>>(d_st, d_ids, d_rg, (int)live.size());
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(stream_));
    dfree(d_ids);
    dfree(d_rg);
  }
  if (gexec_) {
    (void)hipGraphExecDestroy(gexec_);
    gexec_ = nullptr;
  }
  if (graph_) {
    (void)hipGraphDestroy(graph_);
    graph_ = nullptr;
  }
  sched_dirty_ = false;
}

// The sorted-group slice kernel in the configured shape (threads per
// workgroup, gather order), its dynamic LDS raised to what the groups need.
template <class T>
template <bool DUAL>
void Engine<T>::launch_group(unsigned g, int tpb, size_t lds, const IterArgs<T>& A, int step) {
  auto go = [&](auto kern, int t) { kern<<<g, t, lds, stream_>>>(A, step); };
  const bool b = DUAL ? batchedD_ : batchedP_;
  switch (tpb) {
    case 512:
      if (b) go(sorted_group_step<T, DUAL, 512, true>, 512);
      else go(sorted_group_step<T, DUAL, 512, false>, 512);
      break;
    case 1024:
      if (b) go(sorted_group_step<T, DUAL, 1024, true>, 1024);
      else go(sorted_group_step<T, DUAL, 1024, false>, 1024);
      break;
    default:
      if (b) go(sorted_group_step<T, DUAL, 256, true>, 256);
      else go(sorted_group_step<T, DUAL, 256, false>, 256);
      break;
  }
}

template <class T>
template <bool DUAL>
void Engine<T>::launch_sorted(const IterArgs<T>& A, int step) {
  const unsigned g = (unsigned)(DUAL ? nDB_ : nPB_);
  const size_t lds = sizeof(double) * (size_t)((DUAL ? ldsDB_ : ldsPB_) + kSpareWords);
  switch (DUAL ? tpbDB_ : tpbPB_) {
    case 128: sorted_step<T, DUAL, 128, 1><<<g, 128, lds, stream_>>>(A, step); break;
    case 512: sorted_step<T, DUAL, 512, kPlainD><<<g, 512, lds, stream_>>>(A, step); break;
    default: sorted_step<T, DUAL, 256, kPlainD><<<g, 256, lds, stream_>>>(A, step); break;
  }
}

template <class T>
void Engine<T>::launch_slices(bool dual, const IterArgs<T>& A, int step) {
  const unsigned g = (unsigned)(dual ? nDS_ : nPS_);
  if (opt_.slice_sort) {
    const size_t lds = sizeof(double) * (size_t)((dual ? ldsD_ : ldsP_) + kSpareWords);
    if (dual) launch_group<true>(g, dual ? tpbD_ : tpbP_, lds, A, step);
    else launch_group<false>(g, dual ? tpbD_ : tpbP_, lds, A, step);
    return;
  }
  switch (opt_.slice_entries) {
    case 256:
      if (dual) dual_slice_step<T, 256><<<g, kThreads, 0, stream_>>>(A, step);
      else primal_slice_step<T, 256><<<g, kThreads, 0, stream_>>>(A, step);
      break;
    case 1024:
      if (dual) dual_slice_step<T, 1024><<<g, kThreads, 0, stream_>>>(A, step);
      else primal_slice_step<T, 1024><<<g, kThreads, 0, stream_>>>(A, step);
      break;
    default:
      if (dual) dual_slice_step<T, 512><<<g, kThreads, 0, stream_>>>(A, step);
      else primal_slice_step<T, 512><<<g, kThreads, 0, stream_>>>(A, step);
      break;
  }
}

template <class T>
void Engine<T>::launch_chunk() {
  if (sched_dirty_ && !compacted_) rebuild_schedules();
  if (scheduled_ == 0) return;
  const IterArgs<T> A = args();
  const int CH = opt_.chunk;
  const bool prof = opt_.profile > 0 && (chunk_count_ % opt_.profile) == 0;
  ++chunk_count_;
  if (prof) {
    collect_times();  // the previous timed chunk (long finished) frees the event pool
    if ((int)pev_.size() != 6 * CH) {
      for (hipEvent_t e : pev_) (void)hipEventDestroy(e);
      pev_.assign(6 * CH, nullptr);
      for (auto& e : pev_) HIPCHECK(hipEventCreate(&e));
    }
  }
  auto enqueue = [&](bool timed) {
    tick_kernel<<<1, 1, 0, stream_>>>(d_gbase, (int64_t)CH);
    if (nR_) {
      if (tpbR_ == 256) resident_steps<T, 256><<<(unsigned)(nR_ / 2), 256, ldsR_, stream_>>>(A, CH);
      else resident_steps<T, kResRows><<<(unsigned)(nR_ / 2), kResRows, ldsR_, stream_>>>(A, CH);
    }
    for (int i = 0; i < CH; ++i) {
      hipEvent_t* e = timed ? &pev_[6 * i] : nullptr;
      if (timed) HIPCHECK(hipEventRecord(e[0], stream_));
      if (nPS_) launch_slices(false, A, i);
      if (timed) HIPCHECK(hipEventRecord(e[1], stream_));
      if (nP_) primal_step<T><<<(unsigned)nP_, kThreads, 0, stream_>>>(A, i);
      if (nPB_) launch_sorted<false>(A, i);
      if (nPE_) part_step<T, false><<<(unsigned)nPE_, kThreads, 0, stream_>>>(A, i);
      if (timed) HIPCHECK(hipEventRecord(e[2], stream_));
      if (nDS_) launch_slices(true, A, i);
      if (timed) HIPCHECK(hipEventRecord(e[3], stream_));
      if (nD_) dual_step<T><<<(unsigned)nD_, kThreads, 0, stream_>>>(A, i);
      if (nDB_) launch_sorted<true>(A, i);
      if (nDE_) part_step<T, true><<<(unsigned)nDE_, kThreads, 0, stream_>>>(A, i);
      if (timed) {
        HIPCHECK(hipEventRecord(e[4], stream_));
        HIPCHECK(hipEventRecord(e[5], stream_));  // empty pair: the events' own cost
      }
    }
  };
  if (prof) {
    enqueue(true);
    HIPCHECK(hipGetLastError());
    pev_pending_ = true;
    pev_slices_[0] = nPS_ > 0;
    pev_slices_[1] = nDS_ > 0;
    for (int q = 0; q < 3; ++q) pev_size_[q] = sched_size_[q];
  } else if (opt_.use_graph) {
    if (!gexec_) {
      HIPCHECK(hipStreamBeginCapture(stream_, hipStreamCaptureModeThreadLocal));
      enqueue(false);
      HIPCHECK(hipStreamEndCapture(stream_, &graph_));
      HIPCHECK(hipGraphInstantiate(&gexec_, graph_, nullptr, nullptr, 0));
    }
    HIPCHECK(hipGraphLaunch(gexec_, stream_));
  } else {
    enqueue(false);
    HIPCHECK(hipGetLastError());
  }
  g_next_ += CH;
}

template <class T>
void Engine<T>::collect_times() {
  if (!pev_pending_) return;
  HIPCHECK(hipEventSynchronize(pev_.back()));
  for (size_t k = 0; k + 5 < pev_.size(); k += 6) {
    float d[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < 5; ++q) HIPCHECK(hipEventElapsedTime(&d[q], pev_[k + q], pev_[k + q + 1]));
    // an event pair around a kernel that was not launched measures only the
    // events' own overhead: count it as no time
    if (pev_slices_[0]) ktimes_.primal_slice_ms += d[0];
    ktimes_.primal_ms += d[1];
    if (pev_slices_[1]) ktimes_.dual_slice_ms += d[2];
    ktimes_.dual_ms += d[3];
    ktimes_.event_pair_ms += d[4];
    ktimes_.nnz += pev_size_[0];
    ktimes_.n += pev_size_[1];
    ktimes_.m += pev_size_[2];
    ktimes_.launches += 1;
  }
  pev_pending_ = false;
}

template <class T>
void Engine<T>::run(double time_limit_s) {
  const auto t0 = std::chrono::steady_clock::now();
  if (sched_dirty_) {
    compacted_ = false;
    rebuild_schedules();
  }
  auto all_done = [&](const int* h) {
    for (int s = 0; s < nslots_; ++s)
      if (slots_[s].used && slots_[s].watched && h[s] == ST_RUNNING) return false;
    return true;
  };
  if (all_done(h_status[0]) && all_done(h_status[1])) {
    HIPCHECK(hipStreamSynchronize(stream_));
    HIPCHECK(hipMemcpy(h_status[0], d_status, sizeof(int) * nslots_, hipMemcpyDeviceToHost));
    if (all_done(h_status[0])) return;
  }
  int64_t j = 0;
  bool limit_set = false;
  double next_print = (double)opt_.verbose;
  while (true) {
    launch_chunk();
    HIPCHECK(hipMemcpyAsync(h_status[j & 1], d_status, sizeof(int) * nslots_, hipMemcpyDeviceToHost, stream_));
    if (ev_[j & 1]) HIPCHECK(hipEventRecord(ev_[j & 1], stream_));
    else HIPCHECK(hipStreamSynchronize(stream_));
    if (j >= 1) {
      if (ev_[(j - 1) & 1]) HIPCHECK(hipEventSynchronize(ev_[(j - 1) & 1]));
      if (all_done(h_status[(j - 1) & 1])) break;
      // leave finished LPs out of the schedules once half of them are done
      int running = 0;
      for (int s = 0; s < nslots_; ++s) running += slots_[s].used && h_status[(j - 1) & 1][s] == ST_RUNNING;
      if (scheduled_ > 1 && 2 * running <= scheduled_) {
        HIPCHECK(hipStreamSynchronize(stream_));
        HIPCHECK(hipMemcpy(h_status[0], d_status, sizeof(int) * nslots_, hipMemcpyDeviceToHost));
        std::memcpy(h_status[1], h_status[0], sizeof(int) * nslots_);
        finished_ = h_status[0];
        try {
          reblock_for(h_status[0]);
          rebuild_schedules();
        } catch (...) {
          finished_ = nullptr;
          throw;
        }
        finished_ = nullptr;
        sched_dirty_ = true;  // the next add / remove / solve rebuilds the full schedules
        compacted_ = true;
      }
    }
    ++j;
    if (opt_.verbose > 0) {
      const double el = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
      if (el >= next_print) {
        next_print = el + (double)opt_.verbose;
        int first = -1, running = 0, watched = 0;
        for (int s = 0; s < nslots_; ++s) {
          if (!slots_[s].used || !slots_[s].watched) continue;
          ++watched;
          if (h_status[(j - 1) & 1][s] == ST_RUNNING) {
            ++running;
            if (first < 0) first = s;
          }
        }
        if (first >= 0) {
          InstState st;
          HIPCHECK(hipMemcpy(&st, d_st + first, sizeof(InstState), hipMemcpyDeviceToHost));
          fprintf(stderr, "[halp] %.1fs step %lld: %d/%d LPs running; LP %d: iters %lld restarts %lld kkt %.3e "
                  "(p %.2e d %.2e gap %.2e) omega %.3e\n", el, (long long)g_next_, running, watched, first,
                  (long long)st.iters, (long long)st.nrest, st.kkt, st.rel_p, st.rel_d, st.rel_gap, st.omega);
          fflush(stderr);
        }
      }
    }
    if (!limit_set && time_limit_s >= 0.0) {
      const double el = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
      if (el > time_limit_s) {
        set_limit_status_kernel<<<nblk(nslots_), 256, 0, stream_>>>(d_st, d_status, nslots_, ST_TIME_LIMIT);
        limit_set = true;
      }
    }
  }
  HIPCHECK(hipStreamSynchronize(stream_));
  HIPCHECK(hipMemcpy(h_status[0], d_status, sizeof(int) * nslots_, hipMemcpyDeviceToHost));
  std::memcpy(h_status[1], h_status[0], sizeof(int) * nslots_);
  collect_times();
}

template <class T>
std::vector<int> Engine<T>::advance(int chunks) {
  for (int i = 0; i < chunks; ++i) launch_chunk();
  HIPCHECK(hipMemcpyAsync(h_status[0], d_status, sizeof(int) * nslots_, hipMemcpyDeviceToHost, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  collect_times();
  std::vector<int> done;
  for (int s = 0; s < nslots_; ++s) {
    if (slots_[s].used && slots_[s].watched && !slots_[s].reported && h_status[0][s] != ST_RUNNING) {
      slots_[s].reported = true;
      done.push_back(s);
    }
  }
  return done;
}

template <class T>
void Engine<T>::remove(const std::vector<int>& ids) {
  HIPCHECK(hipStreamSynchronize(stream_));
  release_slots(ids);
}

template <class T>
void Engine<T>::release_slots(const std::vector<int>& ids) {
  for (int id : ids) {
    Slot& S = slots_.at(id);
    if (!S.used) continue;
    am_.release(S.row0, S.m + 1);
    an_.release(S.col0, S.n + 1);
    az_.release(S.nz0, S.nnz);
    abK_.release(S.brpD0, S.brpDn);
    abKT_.release(S.brpP0, S.brpPn);
    S = Slot();
    h_status[0][id] = h_status[1][id] = 0;
  }
  sched_dirty_ = true;
  compacted_ = false;
}

template <class T>
Result Engine<T>::result(int id) {
  if (id < 0 || id >= nslots_ || !slots_[id].used) throw Error(-1, "invalid LP id");
  return results({id})[0];
}

static Result result_of(const InstState& s) {
  Result r;
  r.status = s.status;
  if (s.checks == 0 && s.status == ST_ITER_LIMIT) r.status = 0;  // parked, never run
  r.iters = s.iters;
  r.restarts = s.nrest;
  r.checks = s.checks;
  r.kkt = s.kkt;
  r.rel_p = s.rel_p;
  r.rel_d = s.rel_d;
  r.rel_gap = s.rel_gap;
  r.pobj = s.pobj;
  r.dobj = s.dobj;
  r.resid = s.resid;
  r.omega = s.omega;
  r.eta = s.eta;
  r.sigma_hat = s.sigma_hat;
  r.power_iters = s.pw_iter;
  r.ray = s.ray;
  r.active_changes = s.act_changes;
  r.ident_iters = s.ident_iters;
  return r;
}

template <class T>
std::vector<Result> Engine<T>::results(const std::vector<int>& ids) {
  std::vector<Result> out;
  if (ids.empty()) return out;
  for (const InstState& s : states(ids)) out.push_back(result_of(s));
  return out;
}

template <class T>
void Engine<T>::take_over(const EngineBase& src, const std::vector<int>& src_ids, const std::vector<int>& ids,
                          const std::vector<double>& omega) {
  std::vector<HandOver> in;
  int64_t largest = 1;
  for (size_t k = 0; k < ids.size(); ++k) {
    const Slot& S = slots_[ids[k]];
    const Candidate c = src.candidate(src_ids[k]);
    in.push_back({c.x, c.y, omega[k], S.m, S.n, S.row0, S.col0, ids[k], c.fp32});
    largest = std::max({largest, S.m, S.n});
  }
  if (in.empty()) return;
  TempScope temp;
  HandOver* d_in = nullptr;
  talloc(&d_in, (int64_t)in.size());
  HIPCHECK(hipMemcpyAsync(d_in, in.data(), sizeof(HandOver) * in.size(), hipMemcpyHostToDevice, stream_));
  const int parts = parts_for(largest, in.size());
  take_over_kernel<T><<<(unsigned)(in.size() * parts), kThreads, 0, stream_>>>(d_in, parts, d_st, x, x0, y, y0);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_in);
}

template <class T>
void Engine<T>::solution(int id, double* xo, double* yo, bool to_device) {
  if (id < 0 || id >= nslots_ || !slots_[id].used) throw Error(-1, "invalid LP id");
  const Slot& S = slots_[id];
  // the LP's part of the vectors that its creation worked in
  double *xu = fn + S.col0, *yu = fm + S.row0;
  unscale_kernel<T><<<nblk(S.n), 256, 0, stream_>>>(xT, Dc, S.col0, S.n, xu);
  if (S.m) unscale_kernel<T><<<nblk(S.m), 256, 0, stream_>>>(yT, Dr, S.row0, S.m, yu);
  HIPCHECK(hipGetLastError());
  const auto kind = to_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  if (xo) HIPCHECK(hipMemcpyAsync(xo, xu, sizeof(double) * S.n, kind, stream_));
  if (yo && S.m) HIPCHECK(hipMemcpyAsync(yo, yu, sizeof(double) * S.m, kind, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
}

template <class T>
void Engine<T>::certificate(int id, double* ray, bool to_device) {
  if (id < 0 || id >= nslots_ || !slots_[id].used) throw Error(-1, "invalid LP id");
  const Slot& S = slots_[id];
  InstState s;
  HIPCHECK(hipStreamSynchronize(stream_));
  HIPCHECK(hipMemcpy(&s, d_st + id, sizeof(InstState), hipMemcpyDeviceToHost));
  if (s.status != ST_PRIMAL_INFEAS && s.status != ST_DUAL_INFEAS)
    throw Error(-4, "no certificate: the LP was not found infeasible");
  const bool primal = s.status == ST_PRIMAL_INFEAS;
  const int64_t len = primal ? S.m : S.n;
  TempScope temp;
  double* tmp = nullptr;
  talloc(&tmp, len);
  if (primal)
    unscale_kernel<T><<<nblk(len), 256, 0, stream_>>>(s.ray == 1 ? cy1 : cy2, Dr, S.row0, len, tmp);
  else
    unscale_kernel<T><<<nblk(len), 256, 0, stream_>>>(s.ray == 1 ? cx1 : cx2, Dc, S.col0, len, tmp);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipMemcpyAsync(ray, tmp, sizeof(double) * len, to_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                          stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(tmp);
}

template <class T>
void Engine<T>::export_point(int id, double* xo, double* yo, double* omega) {
  if (id < 0 || id >= nslots_ || !slots_[id].used) throw Error(-1, "invalid LP id");
  const Slot& S = slots_[id];
  copy_state_kernel<T><<<nblk(S.n), 256, 0, stream_>>>(xT, xo, S.col0, S.n);
  if (S.m) copy_state_kernel<T><<<nblk(S.m), 256, 0, stream_>>>(yT, yo, S.row0, S.m);
  HIPCHECK(hipGetLastError());
  InstState st;
  HIPCHECK(hipMemcpyAsync(&st, d_st + id, sizeof(InstState), hipMemcpyDeviceToHost, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  *omega = st.omega;
}

template <class T>
void Engine<T>::import_point(int id, const double* xi, const double* yi, double omega) {
  if (id < 0 || id >= nslots_ || !slots_[id].used) throw Error(-1, "invalid LP id");
  const Slot& S = slots_[id];
  load_point_kernel<T><<<nblk(S.n), 256, 0, stream_>>>(xi, x, x0, S.col0, S.n);
  if (S.m) load_point_kernel<T><<<nblk(S.m), 256, 0, stream_>>>(yi, y, y0, S.row0, S.m);
  HIPCHECK(hipGetLastError());
  InstState st;
  HIPCHECK(hipMemcpyAsync(&st, d_st + id, sizeof(InstState), hipMemcpyDeviceToHost, stream_));
  HIPCHECK(hipStreamSynchronize(stream_));
  if (omega > 0.0 && std::isfinite(omega)) {  // else keep the LP's initial primal weight
    st.omega = omega;
    st.tau = st.eta / omega;
    st.sigma = st.eta * omega;
  }
  TempScope temp;
  InstState* d_src = nullptr;
  int* d_ids = nullptr;
  talloc(&d_src, 1);
  talloc(&d_ids, 1);
  HIPCHECK(hipMemcpyAsync(d_src, &st, sizeof(InstState), hipMemcpyHostToDevice, stream_));
  HIPCHECK(hipMemcpyAsync(d_ids, &id, sizeof(int), hipMemcpyHostToDevice, stream_));
  write_states_kernel<<<1, 256, 0, stream_>>>(d_st, d_status, d_cnt, d_ids, d_src, 1);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipStreamSynchronize(stream_));
  dfree(d_src);
  dfree(d_ids);
}

template <class T>
void Engine<T>::stored_matrix(int id, bool transpose, int32_t* rp, int32_t* ci, double* val) {
  if (id < 0 || id >= nslots_ || !slots_[id].used) throw Error(-1, "invalid LP id");
  const Slot& S = slots_[id];
  const std::vector<Blk>& blocks = transpose ? S.bP : S.bD;
  const std::vector<Blk>& slices = transpose ? S.bPS : S.bDS;
  bool row_order = slices.empty();
  for (const Blk& b : blocks) row_order &= blk_kind(b) != BK_SORTED && !blk_part(b);
  if (!row_order) throw Error(-4, "the product is not stored in row order (column slices or sorted layout)");
  const int64_t rows = transpose ? S.n : S.m, r0 = transpose ? S.col0 : S.row0;
  const int64_t c0 = transpose ? S.row0 : S.col0;
  HIPCHECK(hipStreamSynchronize(stream_));
  HIPCHECK(hipMemcpy(rp, (transpose ? KT_rp : K_rp) + r0, sizeof(int32_t) * (rows + 1), hipMemcpyDeviceToHost));
  if (S.nnz > 0) {
    HIPCHECK(hipMemcpy(ci, (transpose ? KT_ci : K_ci) + S.nz0, sizeof(int32_t) * S.nnz, hipMemcpyDeviceToHost));
    HIPCHECK(hipMemcpy(val, (transpose ? KT_v64 : K_v64) + S.nz0, sizeof(double) * S.nnz,
                       hipMemcpyDeviceToHost));
  }
  for (int64_t r = 0; r <= rows; ++r) rp[r] -= (int32_t)S.nz0;
  for (int64_t e = 0; e < S.nnz; ++e) ci[e] -= (int32_t)c0;
}

int narrow_row_ptr(const int64_t* src, int32_t* dst, int64_t count, hipStream_t stream) {
  if (count <= 0) return 0;
  TempScope temp;
  int* d_bad = nullptr;
  talloc(&d_bad, 1);
  HIPCHECK(hipMemsetAsync(d_bad, 0, sizeof(int), stream));
  narrow_row_ptr_kernel<<<nblk(count), 256, 0, stream>>>(src, dst, count, d_bad);
  HIPCHECK(hipGetLastError());
  int bad = 0;
  HIPCHECK(hipMemcpyAsync(&bad, d_bad, sizeof(int), hipMemcpyDeviceToHost, stream));
  HIPCHECK(hipStreamSynchronize(stream));
  dfree(d_bad);
  return bad;
}

std::unique_ptr<EngineBase> make_engine(const Options& opt, hipStream_t stream, int64_t cap_m, int64_t cap_n,
                                        int64_t cap_nnz, int max_slots) {
  if (opt.precision == 1)
    return std::unique_ptr<EngineBase>(new Engine<float>(opt, stream, cap_m, cap_n, cap_nnz, max_slots));
  return std::unique_ptr<EngineBase>(new Engine<double>(opt, stream, cap_m, cap_n, cap_nnz, max_slots));
}

}  // namespace halp
