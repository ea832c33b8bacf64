// The sizes that the workspace queries count against the plans that the
// launches build, and what the queries cost (host only; built and run by
// tests/test_plan_size.py, the device entry points replaced by stubs).
#include <sys/resource.h>

#include <chrono>
#include <cstdio>
#include <cstdlib>

#include <hip/hip_runtime.h>

#include "plan.hpp"
#include "tchol.h"

extern "C" {
#define STUB(name, ...) hipError_t name(__VA_ARGS__) { std::fprintf(stderr, "stub %s reached\n", #name); std::abort(); }
struct KArgs;
STUB(tchol_dev_launch, const KArgs*, int32_t, const int32_t*, int64_t, int, int, hipStream_t, hipEvent_t, hipEvent_t)
STUB(tchol_dev_max_grid, int, int*)
STUB(tchol_dev_compact_grid, int, int*)
STUB(tchol_dev_backward_prep, const double*, int64_t, double*, double*, int64_t, int64_t, hipStream_t)
STUB(tchol_refine_convert, const double*, int64_t, float*, int64_t, int64_t, hipStream_t)
STUB(tchol_refine_residual, const double*, int64_t, int64_t, const double*, const double*, double*, int64_t, int, int,
     double*, hipStream_t)
STUB(tchol_refine_colmax, const double*, int64_t, int64_t, int, double*, hipStream_t)
STUB(tchol_refine_axpy, double*, const double*, int64_t, hipStream_t)
STUB(tchol_b32_prepare, const int64_t*, int32_t, const float*, const float*, double*, double*, int, hipStream_t)
STUB(tchol_b32_finish, const int64_t*, int32_t, float*, float*, const double*, const double*, int, hipStream_t)
STUB(tchol_refine_diag, const double*, int64_t, int64_t, int64_t, double*, hipStream_t)
}

static int failures = 0;
#define CHECK(c, ...)                                                    \
  do {                                                                   \
    if (!(c)) {                                                          \
      std::fprintf(stderr, "check failed at line %d: %s", __LINE__, #c); \
      std::fprintf(stderr, " " __VA_ARGS__);                             \
      std::fprintf(stderr, "\n");                                        \
      ++failures;                                                        \
    }                                                                    \
  } while (0)

static void same(const char* what, bool have, const tchol::PlanSize& z, const std::shared_ptr<const tchol::Plan>& p,
                 long n, long nb) {
  CHECK(have && p, "%s n=%ld nb=%ld", what, n, nb);
  if (!have || !p) return;
  const tchol::PlanSize q = tchol::size_of(*p);
  CHECK(z.ntask == q.ntask && z.nedge == q.nedge && z.nitem == q.nitem && z.inv == q.inv,
        "%s n=%ld nb=%ld: tasks %ld %ld edges %ld %ld items %ld %ld", what, n, nb, (long)z.ntask, (long)q.ntask,
        (long)z.nedge, (long)q.nedge, (long)z.nitem, (long)q.nitem);
  CHECK(z.systems.size() == q.systems.size(), "%s n=%ld nb=%ld", what, n, nb);
  for (size_t s = 0; s < z.systems.size() && s < q.systems.size(); ++s)
    CHECK(z.systems[s].n == q.systems[s].n && z.systems[s].nb == q.systems[s].nb && z.systems[s].T == q.systems[s].T,
          "%s n=%ld nb=%ld system %zu", what, n, nb, s);
}

int main() {
  const int64_t ns[] = {1, 15, 16, 17, 64, 100, 128, 129, 257, 300, 511, 512, 513, 777, 1000, 1024, 1301, 2048, 3001, 12288,
                        12289, 14000};
  const int64_t nbs[] = {16, 48, 64, 112, 128, 144, 192, 256, 384, 448, 512};
  for (int64_t n : ns)
    for (int64_t nb : nbs) {
      if ((n + nb - 1) / nb > 130) continue;  // (building those takes long)
      tchol::PlanSize z;
      for (int32_t op : {(int32_t)TCHOL_OP_FACTOR, tchol::OP_FACTOR_INVT}) {
        bool have = tchol::factor_size(op, n, nb, &z);
        same("factor", have, z, tchol::get_plan(op, n, nb, TCHOL_POLICY_FIFO, 0), n, nb);
        have = tchol::run_factor_size(op, n, nb, &z);
        same("run factor", have, z, tchol::get_run_plan(op, n, nb, TCHOL_POLICY_FIFO, 0), n, nb);
      }
      std::vector<tchol::System> sys(1);
      sys[0].n = n;
      sys[0].nb = nb;
      for (bool inv : {false, true}) {
        bool have = tchol::merged_size(n, nb, inv, &z);
        same("merged", have, z, tchol::get_batched_plan(sys, TCHOL_POLICY_FIFO, 0, inv), n, nb);
        have = tchol::run_merged_size(n, nb, inv, &z);
        same("run merged", have, z, tchol::get_run_merged_plan(n, nb, TCHOL_POLICY_FIFO, 0, inv), n, nb);
      }
    }
  // beyond what the planner takes
  tchol::PlanSize z;
  CHECK(!tchol::factor_size(TCHOL_OP_FACTOR, 1201 * 16, 16, &z));
  CHECK(!tchol::merged_size(1201 * 16, 16, true, &z));
  CHECK(!tchol::run_factor_size(TCHOL_OP_FACTOR, 1201 * 16, 16, &z));
  CHECK(!tchol::run_merged_size(1201 * 16, 16, true, &z));
  // nothing to do is a size, not a plan
  CHECK(tchol_factor_solve_workspace_bytes(0, 128, 1) > 0);
  CHECK(tchol_factor_solve_workspace_bytes(0, 512, 0) > 0);
  CHECK(tchol_workspace_bytes(TCHOL_OP_FACTOR, 0, 128, 0) > 0);
  std::printf("plan sizes: %d failures\n", failures);

  // a workspace below what the queried plan needs stays refused, also where the
  // run plan would fit (order 16384 by tiles of 512: its merged updates save room)
  double* fake = reinterpret_cast<double*>(0x10000);
  const int32_t n1 = 16384, nb1 = 512;
  const int64_t need = tchol_batched_workspace_bytes(&n1, &nb1, 1);
  CHECK(tchol::run_merged_size(n1, nb1, false, &z));
  tchol::PlanSize q;
  CHECK(tchol::merged_size(n1, nb1, false, &q) && z.ntask < q.ntask && z.nedge < q.nedge && z.nitem < q.nitem);
  tchol_opts subst = {};
  subst.subst = 1;
  CHECK(tchol_factor_solve(fake, n1, nb1, fake, 1, fake, need - 256, nullptr, &subst) == -7);
  CHECK(tchol_factor(fake, n1, nb1, fake, 1 << 18, nullptr) == -5);

  // queries build no plan: small tiles of large orders would take seconds and gigabytes
  rusage before, after;
  getrusage(RUSAGE_SELF, &before);
  const auto t0 = std::chrono::steady_clock::now();
  for (int64_t n = 4000; n < 19200; n += 800) {
    CHECK(tchol_workspace_bytes(TCHOL_OP_FACTOR, n, 16, 0) > 0);
    CHECK(tchol_factor_solve_workspace_bytes(n, 16, 1) > 0);
  }
  const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  getrusage(RUSAGE_SELF, &after);
  CHECK(s < 5.0, "queries took %.1f s", s);
  CHECK(after.ru_maxrss - before.ru_maxrss < 64 * 1024, "queries kept %ld KB", (long)(after.ru_maxrss - before.ru_maxrss));
  std::printf("queries: %.3f s; %d failures\n", s, failures);
  return failures == 0 ? 0 : 1;
}
