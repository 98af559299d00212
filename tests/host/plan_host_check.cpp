// Host-only checks of the planner and the executor's host side, linked with
// the library; no device is touched.  Prints OK, or with an argument the default
// of "launch_evals".
#include <cstdio>
#include <cstring>
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

}  // namespace

int main(int argc, char**) {
  if (argc > 1) {
    std::printf("%.17g\n", kde_ctx().opt_launch_evals);
    return 0;
  }
  if (tuned_variant() || queue_form()) return 1;
  std::puts("OK");
  return 0;
}
