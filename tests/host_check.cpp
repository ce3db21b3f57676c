// Checks of the engine's host code on the CPU (see hip_stub.h).  Usage:
// host_check NAME; prints "ok NAME".
#include "hip_stub.h"

#include "engine.h"
#include "halp.h"

#include <random>

#define CHECK(c)                                                                     \
  do {                                                                               \
    if (!(c)) {                                                                      \
      fprintf(stderr, "%s:%d: %s (%s)\n", __FILE__, __LINE__, #c, lp_last_error());  \
      exit(1);                                                                       \
    }                                                                                \
  } while (0)

namespace {

struct LP {
  int64_t m, n;
  std::vector<int32_t> rp{0}, ci;
  std::vector<double> val, c, rhs, lb, ub;
  // row r: `len` entries at random in columns [first(r), first(r) + span)
  LP(int64_t m_, int64_t n_, int64_t len, int64_t span, unsigned seed = 1) : m(m_), n(n_) {
    std::mt19937_64 g(seed);
    std::vector<int32_t> row;
    for (int64_t r = 0; r < m; ++r) {
      const int64_t first = m > 1 ? (n - span) * r / (m - 1) : 0;
      row.clear();
      for (int64_t k = 0; k < len; ++k) row.push_back((int32_t)(first + (int64_t)(g() % (uint64_t)span)));
      std::sort(row.begin(), row.end());
      row.erase(std::unique(row.begin(), row.end()), row.end());
      ci.insert(ci.end(), row.begin(), row.end());
      rp.push_back((int32_t)ci.size());
    }
    val.assign(ci.size(), 1.0);
    c.assign(n, 1.0);
    rhs.assign(m, 1.0);
    lb.assign(n, 0.0);
    ub.assign(n, 1.0);
  }
  lp_problem problem() const {
    return {n, m, 0, rp.data(), ci.data(), val.data(), c.data(), rhs.data(), lb.data(), ub.data()};
  }
};

lp_options options() {
  lp_options o;
  lp_default_options(&o);
  o.use_graph = 0;
  o.eta = 0.1;  // no power iteration: its kernels do nothing here
  return o;
}

// LP i reaches its tolerance in this step.
template <class T = double>
void finish(void** args, int i) {
  const auto& A = stub::arg<halp::IterArgs<T>>(args, 0);
  A.st[i].status = A.status_out[i] = halp::ST_OPTIMAL;
  A.st[i].checks = 1;
}

size_t step_kernels(size_t from) {
  return stub::count("_step<double", from) + stub::count("resident_steps", from);
}

// Memory runs out after n allocations of a server's first steps, for every n:
// the step after that, with memory again, finds every buffer it needs (a
// launch with a null schedule or sums buffer would fault a GPU).
void failed_schedule() {
  const LP a(40, 60, 5, 60), b(3000, 5000, 8, 5000);
  lp_options o = options();
  for (const int sorted : {1, 0}) {
    o.plain_sort = sorted;
    bool failed = true;
    for (long n = 0; failed; ++n) {
      stub::reset();
      lp_server* s = nullptr;
      CHECK(lp_server_create(&s, 64 << 20, 8, nullptr, &o) == LP_OK);
      int64_t t;
      lp_problem p = a.problem();
      CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
      p = b.problem();
      CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
      stub::fail_at = n;
      const int rc = lp_server_step(s, 1, nullptr);
      failed = rc != LP_OK;
      stub::fail_at = -1;
      CHECK(rc == LP_OK || rc == LP_ERR_OOM);
      stub::on_launch = [&](const stub::Launch& l, void** args) {
        if (l.name.find("step<double") == std::string::npos) return;
        const auto& A = stub::arg<halp::IterArgs<double>>(args, 0);
        CHECK(A.partP && A.partD);
        CHECK(sorted ? A.schedPB && A.schedDB : A.schedP && A.schedD);
      };
      const size_t from = stub::launches.size();
      CHECK(lp_server_step(s, 1, nullptr) == LP_OK);
      CHECK(step_kernels(from) > 0);
      stub::on_launch = nullptr;
      lp_server_destroy(s);
    }
  }
}

// Two small LPs of a server step on one CU each; a larger one joins, for which
// they are laid out anew, and memory runs out somewhere on the way.
// No later step may use the schedule of the old layout with re-laid matrices.
void failed_admission() {
  // (the small ones have more entries, so that laying them out takes the most
  // memory, K more than K^T, which comes first)
  const LP a(1000, 100, 8, 100), b(1000, 120, 8, 120), big(1100, 1100, 1, 1);
  const lp_options o = options();
  bool failed = true, relaid = false;
  for (size_t room = 0; failed; room += 4096) {
    stub::reset();
    lp_server* s = nullptr;
    CHECK(lp_server_create(&s, 64 << 20, 3, nullptr, &o) == LP_OK);
    int64_t t;
    lp_problem p = a.problem();
    CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
    p = b.problem();
    CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
    CHECK(lp_server_step(s, 1, nullptr) == LP_OK);
    CHECK(stub::count("resident_steps") == 1);
    p = big.problem();
    CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
    const size_t from = stub::launches.size();
    stub::limit = stub::bytes + room;
    const int rc = lp_server_step(s, 1, nullptr);
    failed = rc != LP_OK;
    stub::limit = SIZE_MAX;
    CHECK(rc == LP_OK || rc == LP_ERR_OOM);
    const bool cut = stub::count("reblock_keys_kernel", from) > 0;
    relaid |= failed && cut;
    const size_t then = stub::launches.size();
    CHECK(lp_server_step(s, 1, nullptr) == LP_OK);
    if (cut) CHECK(stub::count("resident_steps", then) == 0);
    CHECK(step_kernels(then) > 0);
    lp_server_destroy(s);
  }
  CHECK(relaid);  // the case that matters came up
}

// Memory runs out somewhere in the admission of an LP: its slot is free again
// (a server of two slots has the second one filled by the next step).
void failed_admission_frees_slots() {
  const LP a(40, 60, 5, 60), b(3000, 5000, 8, 5000);
  lp_options o = options();
  for (const int sorted : {1, 0}) {
    o.plain_sort = sorted;
    bool failed = true;
    size_t failures = 0;
    for (long n = 0; failed; ++n) {
      stub::reset();
      lp_server* s = nullptr;
      CHECK(lp_server_create(&s, 64 << 20, 2, nullptr, &o) == LP_OK);
      int64_t t;
      int queued = 0, live = 0;
      lp_problem p = a.problem();
      CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
      CHECK(lp_server_step(s, 1, nullptr) == LP_OK);
      CHECK(lp_server_info(s, &queued, &live, nullptr) == LP_OK && queued == 0 && live == 1);
      p = b.problem();
      CHECK(lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t) == LP_OK);
      stub::fail_at = n;
      failed = lp_server_step(s, 0, nullptr) != LP_OK;  // admission alone
      stub::fail_at = -1;
      failures += failed;
      CHECK(lp_server_info(s, &queued, &live, nullptr) == LP_OK && queued == failed && live == 2 - failed);
      int done = 0;
      CHECK(lp_server_step(s, 1, &done) == LP_OK && done == 0);
      CHECK(lp_server_info(s, &queued, &live, nullptr) == LP_OK && queued == 0 && live == 2);
      lp_server_destroy(s);
    }
    CHECK(failures > 0);
  }
}

// Memory runs out somewhere in the admission to an FP32 server's second phase:
// the LP waits for it again.
void failed_second_phase() {
  const LP a(40, 60, 5, 60), b(50, 70, 5, 70);
  lp_options o = options();
  o.precision = LP_PREC_FP32;
  bool failed = true;
  size_t failures = 0;
  for (long n = 0; failed; ++n) {
    stub::reset();
    lp_server* s = nullptr;
    CHECK(lp_server_create(&s, 64 << 20, 4, nullptr, &o) == LP_OK);
    int64_t t;
    for (const LP* lp : {&a, &b}) {
      const lp_problem p = lp->problem();
      CHECK(lp_server_submit(s, &p, 1e-9, 1000, 0.0, &t) == LP_OK);
    }
    stub::on_launch = [&](const stub::Launch& l, void** args) {
      if (l.name.find("resident_steps<float") != std::string::npos)
        for (int i = 0; i < 2; ++i) finish<float>(args, i);
    };
    int queued = 0, live = 0, done = 0;
    CHECK(lp_server_step(s, 1, &done) == LP_OK && done == 0);  // the first phase ends
    CHECK(lp_server_info(s, &queued, &live, nullptr) == LP_OK && queued == 2 && live == 0);
    stub::fail_at = n;
    failed = lp_server_step(s, 0, nullptr) != LP_OK;
    stub::fail_at = -1;
    failures += failed;
    CHECK(lp_server_info(s, &queued, &live, nullptr) == LP_OK && queued == 2 * failed && live == 2 - 2 * failed);
    CHECK(lp_server_step(s, 1, &done) == LP_OK && done == 0);
    CHECK(lp_server_info(s, &queued, &live, nullptr) == LP_OK && queued == 0 && live == 2);
    lp_server_destroy(s);
  }
  CHECK(failures > 4);
}

// The LPs of a batch still running when half have finished are laid out anew;
// memory runs out after n allocations of that, for every n.  The next solve
// starts from schedules built after the failure.
void failed_reblocking() {
  std::vector<LP> lps;
  std::vector<lp_problem> ps;
  for (int i = 0; i < 40; ++i) lps.emplace_back(1500, 2500, 6, 2500, i);
  for (const LP& lp : lps) ps.push_back(lp.problem());
  const lp_options o = options();
  bool failed = true, relaid = false;
  for (long n = 0; failed; ++n) {
    stub::reset();
    lp_batch* h = nullptr;
    CHECK(lp_batch_create(&h, (int)ps.size(), ps.data(), 0, nullptr, &o) == LP_OK);
    int steps = 0;
    size_t from = 0;
    stub::on_launch = [&](const stub::Launch& l, void** a) {
      if (l.name.find("sorted_step<double, true") == std::string::npos) return;
      if (++steps == 64) {  // all but three finish in the first chunk
        for (int i = 3; i < 40; ++i) finish(a, i);
        from = stub::launches.size();
        stub::fail_at = n;
      }
      if (steps > 64 * 40)  // the rest finish later
        for (int i = 0; i < 3; ++i) finish(a, i);
    };
    const int rc = lp_batch_solve(h, 1e-6, 1000, -1.0);
    failed = rc != LP_OK;
    stub::fail_at = -1;
    CHECK(rc == LP_OK || rc == LP_ERR_OOM);
    relaid |= failed && stub::count("reblock_keys_kernel", from) > 0;
    if (failed) {
      const size_t then = stub::launches.size();
      CHECK(lp_batch_solve(h, 1e-6, 1000, -1.0) == LP_OK);
      size_t ranges = then, step = then;
      while (ranges < stub::launches.size() && stub::launches[ranges].name != "set_ranges_kernel") ++ranges;
      while (step < stub::launches.size() && stub::launches[step].name.find("sorted_step") == std::string::npos) ++step;
      CHECK(step < stub::launches.size() && ranges < step);
    }
    lp_batch_destroy(h);
  }
  CHECK(relaid);
}

// A row limit that sorted groups cannot exceed any more than plain blocks can
// keeps unsliced products in plain blocks; without it, products of more rows
// than one plain block per CU holds go to groups.
void row_limit() {
  const LP wide(300, 70000, 200, 70000), tall(600, 530000, 900, 530000);
  for (const int rows : {64, 256, 2048, 16384}) {
    for (const LP* lp : {&wide, &tall}) {
      stub::reset();
      lp_options o = options();
      o.slice_min_bytes = -1;
      o.sort_rows = rows;
      const lp_problem p = lp->problem();
      lp_solver* s = nullptr;
      CHECK(lp_create(&s, p.n, p.m_eq, 0, p.row_ptr, p.col_idx, p.val, p.c, p.rhs, p.lb, p.ub, 0, nullptr, &o) == LP_OK);
      const bool groups = lp == &tall && rows > halp::kSortRowsPlain;
      CHECK((stub::count("group_keys_kernel") > 0) == groups);
      lp_destroy(s);
    }
  }
}

// Few long rows are cut into blocks by their entries, short ones by the rows.
void long_rows() {
  const struct {
    LP lp;
    unsigned least, most;  // workgroups of K's product
  } cases[] = {{LP(200, 50000, 2000, 50000), 180, 200},   // a row each
               {LP(2000, 7000, 24, 7000), 100, 140},      // 16 rows each
               {LP(3, 20000, 9000, 20000), 3, 3},
               {LP(64, 3000, 128, 3000), 7, 9}};          // 1024 entries each
  for (const auto& c : cases) {
    stub::reset();
    const lp_options o = options();
    const lp_problem p = c.lp.problem();
    lp_solver* s = nullptr;
    unsigned grid = 0;
    stub::on_launch = [&](const stub::Launch& l, void** a) {
      if (l.name.find("sorted_step<double, true") == 0) grid = l.grid;
      if (l.name.find("_step<double, true") != std::string::npos) finish(a, 0);
    };
    CHECK(lp_create(&s, p.n, p.m_eq, 0, p.row_ptr, p.col_idx, p.val, p.c, p.rhs, p.lb, p.ub, 0, nullptr, &o) == LP_OK);
    CHECK(lp_solve(s, 1e-6, 1000, -1.0) == LP_OK);
    CHECK(grid >= c.least && grid <= c.most);
    lp_destroy(s);
  }
}

// Groups whose entries crowd into one slice (a banded matrix) are split until no
// block is left that is large for its slice; groups of evenly spread entries,
// with one long row, or of a matrix with most entries in one slice are not.
void crowded_slices() {
  const int64_t m = 30000, n = 600000;
  LP band(m, n, 40, 4000), even(m, n, 40, n), row(m, n, 10, n), left(m, n, 40, n / 8);
  for (int64_t r = 0; r < m; ++r)  // all rows in the first slice
    for (int32_t e = left.rp[r]; e < left.rp[r + 1]; ++e) left.ci[e] -= (int32_t)((n - n / 8) * r / (m - 1));
  LP one(1, n, 500000, n);  // the long row takes the place of row 7
  const int32_t add = one.rp[1] - (row.rp[8] - row.rp[7]);
  row.ci.erase(row.ci.begin() + row.rp[7], row.ci.begin() + row.rp[8]);
  row.ci.insert(row.ci.begin() + row.rp[7], one.ci.begin(), one.ci.end());
  for (int64_t r = 8; r <= m; ++r) row.rp[r] += add;
  row.val.assign(row.ci.size(), 1.0);
  for (LP* lp : {&band, &even, &row, &left}) {
    stub::reset();
    const lp_options o = options();
    const lp_problem p = lp->problem();
    size_t counts = 0;
    std::vector<halp::Blk> blocks;
    stub::on_launch = [&](const stub::Launch& l, void** a) {
      if (l.name.find("group_count_kernel") == 0 && stub::arg<int64_t>(a, 7) == n) ++counts;
      if (l.name.find("sorted_group_step<double, true") == 0) {
        const auto& A = stub::arg<halp::IterArgs<double>>(a, 0);
        blocks.assign(A.schedDS, A.schedDS + l.grid);
      }
      if (l.name.find("part_step<double, true") != std::string::npos) finish(a, 0);
    };
    lp_solver* s = nullptr;
    CHECK(lp_create(&s, p.n, p.m_eq, 0, p.row_ptr, p.col_idx, p.val, p.c, p.rhs, p.lb, p.ub, 0, nullptr, &o) == LP_OK);
    CHECK(lp_solve(s, 1e-6, 1000, -1.0) == LP_OK);
    int64_t nnz = 0, largest = 0, rows = 0;
    for (const halp::Blk& b : blocks) {
      nnz += b.pn;
      if (halp::blk_slice(b) == 0) rows += b.r1 - b.r0;
      largest = std::max<int64_t>(largest, b.pn);
    }
    CHECK(nnz == (int64_t)lp->ci.size() && rows == m);
    CHECK(lp == &band ? counts > 1 && largest <= 1 << 14 : counts == 1 && blocks.size() <= 8 * 33);
    lp_destroy(s);
  }
  // groups that are too small to be split are not counted
  stub::reset();
  lp_options o = options();
  o.sort_rows = 256;
  const lp_problem p = band.problem();
  lp_solver* s = nullptr;
  CHECK(lp_create(&s, p.n, p.m_eq, 0, p.row_ptr, p.col_idx, p.val, p.c, p.rhs, p.lb, p.ub, 0, nullptr, &o) == LP_OK);
  CHECK(stub::count("group_keys_kernel") == 1 && stub::count("group_count_kernel") == 0);
  lp_destroy(s);
}

// Memory runs out after n allocations of a creation or a solve, for every n:
// nothing is left allocated.
void failed_creation() {
  const LP lps[] = {LP(40, 60, 5, 60), LP(3000, 5000, 8, 5000), LP(6000, 300000, 8, 300000)};
  std::vector<lp_problem> ps;
  for (const LP& lp : lps) ps.push_back(lp.problem());
  for (const int device : {0, 1}) {
    for (const int sorted : {1, 0}) {
      for (const double eta : {0.1, 0.0}) {
        for (const int precision : {LP_PREC_FP64, LP_PREC_FP32}) {
          lp_options o = options();
          o.plain_sort = o.slice_sort = sorted;
          o.eta = eta;
          o.precision = precision;
          o.power_max_iters = 8;
          bool failed = true;
          for (long n = 0; failed; ++n) {
            stub::reset();
            const size_t before = stub::bytes;
            stub::fail_at = n;
            lp_batch* h = nullptr;
            int rc = lp_batch_create(&h, 3, ps.data(), device, nullptr, &o);
            if (rc == LP_OK) rc = lp_batch_solve(h, 1e-6, 100, 0.0);
            failed = rc != LP_OK;
            CHECK(rc == LP_OK || rc == LP_ERR_OOM);
            if (h) lp_batch_destroy(h);
            CHECK(stub::bytes == before);
          }
        }
      }
    }
  }
}

// The temporary memory of a creation is in nobody's way: where there is no room
// for it beside the partial sums of sliced products, it makes room.
void least_memory_partials() {
  const LP lp(300000, 600000, 2, 600000);
  const lp_options o = options();
  const lp_problem p = lp.problem();
  lp_solver* s = nullptr;
  size_t limit = SIZE_MAX;
  for (const bool tight : {false, true}) {
    stub::reset();
    stub::limit = limit;
    CHECK(lp_create(&s, p.n, p.m_eq, 0, p.row_ptr, p.col_idx, p.val, p.c, p.rhs, p.lb, p.ub, 0, nullptr, &o) == LP_OK);
    if (!tight) {
      // the engine, the temporary memory, the partial sums of K and of K^T
      CHECK(stub::sizes.size() >= 4 && stub::sizes[1] >= 29 * lp.ci.size());
      limit = stub::sizes[0] + stub::sizes[2] + std::max(stub::sizes[1], stub::sizes[3]) + 4096;
      CHECK(limit < stub::sizes[0] + stub::sizes[1] + stub::sizes[2] + stub::sizes[3]);
    }
    lp_destroy(s);
  }
}

// A batch needs no more memory to be sorted together than its transpose and
// its largest LP need: with less than the whole sort takes it is sorted in runs.
void least_memory_batch() {
  std::vector<LP> lps;
  std::vector<lp_problem> ps;
  size_t nnz = 0, largest = 0;
  for (int i = 0; i < 20; ++i) lps.emplace_back(2000 + 10 * i, 7000, 20, 7000, i);
  for (const LP& lp : lps) {
    ps.push_back(lp.problem());
    nnz += lp.ci.size();
    largest = std::max(largest, lp.ci.size());
  }
  for (const int precision : {LP_PREC_FP64, LP_PREC_FP32}) {
    lp_options o = options();
    o.precision = precision;
    size_t limit = SIZE_MAX, sorts[2];
    for (const bool tight : {false, true}) {
      stub::reset();
      stub::limit = limit;
      lp_batch* h = nullptr;
      CHECK(lp_batch_create(&h, (int)ps.size(), ps.data(), 0, nullptr, &o) == LP_OK);
      sorts[tight] = stub::count("block_keys_kernel");
      // the engine, the temporary memory, and a little for what is small
      if (!tight) limit = stub::sizes[0] + std::max(29 * nnz, 45 * largest + (1 << 14)) + 65536;
      lp_batch_destroy(h);
    }
    CHECK(sorts[0] == 2 && sorts[1] > 2 && sorts[1] <= 8);
  }
}

// The largest admission that a server takes stays within its budget (up to the
// alignment of its buffers).
void server_budget() {
  for (const int precision : {LP_PREC_FP64, LP_PREC_FP32}) {
    for (const double polish : {0.0, 1e-3}) {
      for (const size_t budget : {4 << 20, 16 << 20, 64 << 20}) {
        lp_options o = options();
        o.precision = precision;
        o.polish_tol = polish;
        int64_t fits = 4, t;
        size_t peak = 0;
        for (int64_t not_so = 20000; not_so - fits > 1 + fits / 500;) {
          const int64_t m = (fits + not_so) / 2;
          const LP lp(m, 4 * m, 36, 4 * m);
          const lp_problem p = lp.problem();
          stub::reset();
          lp_server* s = nullptr;
          CHECK(lp_server_create(&s, (int64_t)budget, 4, nullptr, &o) == LP_OK);
          const int rc = lp_server_submit(s, &p, 1e-6, 1000, 0.0, &t);
          (rc == LP_OK ? fits : not_so) = m;
          stub::on_launch = [&](const stub::Launch&, void**) { peak = std::max(peak, stub::bytes); };
          if (rc == LP_OK) CHECK(lp_server_step(s, 1, nullptr) == LP_OK);
          lp_server_destroy(s);
        }
        CHECK(fits > 100 && peak <= budget + 16384);
      }
    }
  }
}

// Copies of the row sums of a block that one long row dominates: 8, or 16 or 32
// where the block has 16 times as many entries as they take words; none where
// no row dominates or 8 do not fit.
void copies_of_row_sums() {
  struct {
    int64_t rows, len, long_row;
    int shift;
  } const cases[] = {{1, 300, 300, 4}, {1, 600, 600, 5}, {30, 3, 255, 0}, {100, 20, 2000, 3}, {500, 3, 2000, 3},
                     {11200, 3, 500, 0}, {100, 100, 500, 0}, {40, 200, 6000, 4}};
  for (const auto& c : cases) {
    stub::reset();
    LP lp(c.rows, 20000, c.len, 20000);
    const int64_t old = lp.rp[1], add = c.long_row - old;  // row 0 gets columns 0 ..
    lp.ci.erase(lp.ci.begin(), lp.ci.begin() + old);
    std::vector<int32_t> row(c.long_row);
    for (int64_t k = 0; k < c.long_row; ++k) row[k] = (int32_t)(3 * k);
    lp.ci.insert(lp.ci.begin(), row.begin(), row.end());
    for (int64_t r = 1; r <= c.rows; ++r) lp.rp[r] += (int32_t)add;
    lp.val.assign(lp.ci.size(), 1.0);
    // (among many LPs a product gets a block per 256 rows or 16384 entries, at
    // most 25 of them)
    std::vector<lp_problem> ps(1, lp.problem());
    const LP other(1, 2000, 1, 2000);
    for (int i = 0; i < 40; ++i) ps.push_back(other.problem());
    lp_options o = options();
    int shift = -1, blocks = 0;
    stub::on_launch = [&](const stub::Launch& l, void** a) {
      if (l.name.find("sorted_step<double, true") == std::string::npos) return;
      blocks = 0;
      for (unsigned b = 0; b < l.grid; ++b) {
        const halp::Blk& k = stub::arg<halp::IterArgs<double>>(a, 0).schedDB[b];
        if (halp::blk_kind(k) != halp::BK_SORTED || k.inst != 0 || k.pn < c.long_row) continue;
        shift = halp::blk_rep_shift(k);
        blocks = 1;
      }
      for (int i = 0; i < 41; ++i) finish(a, i);
    };
    lp_batch* h = nullptr;
    CHECK(lp_batch_create(&h, (int)ps.size(), ps.data(), 0, nullptr, &o) == LP_OK);
    CHECK(lp_batch_solve(h, 1e-6, 1000, -1.0) == LP_OK);
    if (shift != c.shift) fprintf(stderr, "%ld rows, long row %ld: shift %d\n", (long)c.rows, (long)c.long_row, shift);
    CHECK(blocks == 1 && shift == c.shift);
    lp_batch_destroy(h);
  }
}

// a launch over all LPs of an add holds fewer than 2^32 threads, whatever the
// size of the largest LP, and no LP is left without a workgroup
void launches_of_many() {
  for (size_t lps : {size_t(1), size_t(3), size_t(512), size_t(262143), size_t(262144), size_t(5000000)})
    for (int64_t largest : {int64_t(1), int64_t(4096), int64_t(4097), int64_t(1) << 20, int64_t(1) << 31}) {
      const int64_t parts = halp::parts_for(largest, lps);
      CHECK(parts >= 1);
      CHECK(parts * (int64_t)lps * halp::kThreads < int64_t(1) << 32);
    }
  CHECK(halp::parts_for(int64_t(1) << 31, 1) == 2048 && halp::parts_for(4097, 512) == 2);
}

}  // namespace

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  const std::map<std::string, void (*)()> checks = {{"failed_schedule", failed_schedule},
                                                      {"failed_admission", failed_admission},
                                                      {"failed_admission_frees_slots", failed_admission_frees_slots},
                                                      {"failed_second_phase", failed_second_phase},
                                                      {"failed_reblocking", failed_reblocking},
                                                      {"row_limit", row_limit},
                                                      {"long_rows", long_rows},
                                                      {"crowded_slices", crowded_slices},
                                                      {"failed_creation", failed_creation},
                                                      {"least_memory_partials", least_memory_partials},
                                                      {"least_memory_batch", least_memory_batch},
                                                      {"server_budget", server_budget},
                                                      {"copies_of_row_sums", copies_of_row_sums},
                                                      {"launches_of_many", launches_of_many}};
  if (!checks.count(name)) return 2;
  checks.at(name)();
  printf("ok %s\n", name.c_str());
  return 0;
}
