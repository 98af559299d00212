// Host-only checks of the planner and the executor's host side, linked with
// the library; no device is touched.  Prints OK, or with an argument the default
// of "launch_evals".
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <tuple>
#include <vector>

#include "kde_runtime.h"

namespace kde {
bool lscv_queue_form(kde_ctx* c, const IterPlan& it);
}

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::printf("line %d: %s\n", __LINE__, #x);            \
      return 1;                                              \
    }                                                        \
  } while (0)

namespace {

kde_request lscv_request(int64_t n, int n_h) {
  kde_request r;
  std::memset(&r, 0, sizeof(r));
  r.x.data = &r;  // never read here
  r.x.n = n;
  r.x.dtype = KDE_F32;
  r.methods = KDE_METHOD_LSCV;
  r.stages = 2;
  r.grid.kind = KDE_GRID_PAPER;
  r.grid.n_h = n_h;
  return r;
}

// A tuned variant serves the jobs whose pass is longer than one launch; a
// shorter one keeps the options, whatever is cached for its shape.
int tuned_variant() {
  kde_ctx c;
  c.opt_autotune = 1;
  kde::TuneChoice t{};
  t.hc = 8;
  t.tj = 512;
  // every shape of 100 bandwidths
  for (int q = 0; q < 200; ++q) c.tune_cache[{q, 100}] = t;
  for (int64_t n : {2, 1000, 50'000, 282'000}) {  // up to 3.98e12 evaluations
    const kde_request r = lscv_request(n, 100);
    CHECK(kde::select_variant(&c, &r, 1) == KDE_OK);
    CHECK(c.job_hc == 16 && c.job_tj == 512);
  }
  const kde_request big = lscv_request(284'000, 100);
  CHECK(kde::select_variant(&c, &big, 1) == KDE_OK);
  CHECK(c.job_hc == 8);
  // passes that are not the dense one, and sliced ones, take it at any size
  const kde_request small = lscv_request(50'000, 100);
  for (int* opt : {&c.opt_prune, &c.opt_persistent}) {
    *opt ^= 1;
    CHECK(kde::select_variant(&c, &small, 1) == KDE_OK);
    CHECK(c.job_hc == 8);
    *opt ^= 1;
  }
  c.opt_launch_evals = 1e9;
  const kde_request r = lscv_request(50'000, 100);
  CHECK(kde::select_variant(&c, &r, 1) == KDE_OK);
  CHECK(c.job_hc == 8);
  c.job_hc = 16;
  return 0;
}

// The pass runs as one persistent launch where its evaluations exceed one
// launch's, in every variant that the device holds.
int queue_form() {
  kde_ctx c;
  for (int& b : c.queue_blocks) b = 1024;
  kde::IterPlan it;
  CHECK(!kde::lscv_queue_form(&c, it));
  it.lscv_units.resize(2);
  it.lscv_cost = {{1e9, 1e12}, {1e9, 3e12}};
  CHECK(!kde::lscv_queue_form(&c, it));
  it.lscv_cost[0].evals = 1.1e12;
  CHECK(kde::lscv_queue_form(&c, it));
  c.opt_persistent = 0;
  CHECK(!kde::lscv_queue_form(&c, it));
  return 0;
}

// A pass of few whole LSCV units is cut into exactly the units a piece of the
// planner's, costs included; one of many keeps them, over the same slots.
int whole_units() {
  using Key = std::tuple<int, int, int, int, int, int, double, double>;
  const auto keys = [](const std::vector<kde::Unit>& u, const std::vector<kde::UnitCost>& c) {
    std::vector<Key> k;
    for (size_t q = 0; q < u.size(); ++q)
      k.emplace_back(u[q].col, u[q].row, u[q].j_begin, u[q].j_end, u[q].item, u[q].chunk, c[q].pairs, c[q].evals);
    std::sort(k.begin(), k.end());
    return k;
  };
  for (const bool f64 : {false, true}) {
    kde_ctx c;
    c.prec = f64 ? KDE_PREC_FP64 : KDE_PREC_MIXED;
    for (int n : {2, 63, 64, 65, 256, 257, 511, 512, 513, 1000, 1025, 3001, 5003, 12345, 40001})
      for (int n_h : {1, 16, 17, 100, 500})
        for (int columns : {1, 3, 40, 700}) {
          if ((double)n * columns > 1e6) continue;
          const kde_request r = lscv_request(n, n_h);
          kde::ColPlan p;
          CHECK(kde::plan_column(&c, r, p).empty());
          kde::ColDesc d;
          kde::bind_column(p, (char*)4096, nullptr, nullptr, d);
          CHECK(d.lscv_piece == (p.lscv_pieces > 1 ? kde::kBJ / p.lscv_pieces : 0));
          kde::IterPlan it;
          std::vector<kde::Unit> fine;
          std::vector<kde::UnitCost> cost;
          for (int k = 0; k < columns; ++k) {
            it.cols.push_back(d);
            kde::lscv_units_of(p, k, it.lscv_units, it.lscv_cost, true);
            kde::lscv_units_of(p, k, fine, cost, false);
          }
          const size_t whole = it.lscv_units.size();
          CHECK(whole * p.lscv_pieces == fine.size());
          kde::split_lscv_units(it, f64);
          if (whole >= (f64 ? 4096u : 1024u) && fine.size() > 6144) {
            CHECK(it.lscv_units.size() == whole);
            // every slot of every item, once
            std::vector<int> seen((size_t)columns * d.n_items, 0);
            for (const kde::Unit& u : it.lscv_units)
              if (u.chunk == 0)
                for (int q = 0; q < p.lscv_pieces; ++q) ++seen[(size_t)u.col * d.n_items + u.item + q];
            for (int s : seen) CHECK(s == 1);
          } else {
            CHECK(keys(it.lscv_units, it.lscv_cost) == keys(fine, cost));
          }
          // a single column always fills the chip with its pieces
          CHECK(columns > 1 || it.lscv_units.size() == fine.size());
        }
  }
  return 0;
}

}  // namespace

int main(int argc, char**) {
  if (argc > 1) {
    std::printf("%.17g\n", kde_ctx().opt_launch_evals);
    return 0;
  }
  if (tuned_variant() || queue_form() || whole_units()) return 1;
  std::puts("OK");
  return 0;
}
