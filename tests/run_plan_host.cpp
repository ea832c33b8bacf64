// The plans that ordinary launches run, checked against the tile algorithms
// they stand for (host only; built and run by tests/test_run_plans.py).
//
// Every task's reads and writes are listed on the cells it touches: the
// factorization's tiles, their inverses, the solve's inverses, the row blocks
// of B and of the intermediate y.  Replayed in program order, each access that
// conflicts with an earlier one (read after write, write after read, write
// after write) must be ordered by a path of the plan's edges.  The claim order
// must hold every work item once, after all items of its task's predecessors.
// argv[1], if given, leaves the edges into that kind of task out of the check's
// copy of the plan, which must then fail.
#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "plan.hpp"
#include "tchol.h"

using tchol::Plan;

static long failures = 0;
#define FAIL(...)                                                   \
  do {                                                              \
    if (failures++ < 20) std::fprintf(stderr, __VA_ARGS__);         \
  } while (0)

static int drop_kind = -1;

static int len_of(int kind) { return kind == TK_GEMM4 ? 4 : kind == TK_GEMM2 ? 2 : 1; }

static void check(const Plan& p, const char* what) {
  const int nt = (int)p.ntask();
  const int64_t n = p.systems[0].n;
  const int64_t fb = p.systems.front().nb, sb = p.systems.back().nb;  // the factorization's and the solve's tiles
  const int Tf = (int)((n + fb - 1) / fb), Ts = (int)((n + sb - 1) / sb), r = (int)(sb / fb);
  std::vector<std::vector<int>> succ(nt);
  std::vector<int> indeg(nt, 0);
  for (int t = 0; t < nt; ++t)
    for (int e = p.succ_off[t]; e < p.succ_off[t + 1]; ++e) {
      const int s = p.succ[e];
      if (p.kind[s] == drop_kind) continue;
      succ[t].push_back(s);
      ++indeg[s];
    }
  if (drop_kind < 0)
    for (int t = 0; t < nt; ++t)
      if (indeg[t] != p.dep0[t]) FAIL("%s n=%ld: task %d has %d predecessors, counter %d\n", what, (long)n, t, indeg[t], p.dep0[t]);
  // claim order: every item once, after the items of its predecessors
  std::vector<int64_t> first(nt, -1), last(nt, -1);
  std::vector<int> parts(nt, 0);
  for (int64_t i = 0; i < p.nitem(); ++i) {
    const int t = p.item_task[i];
    if (p.item_part[i] != parts[t]) FAIL("%s n=%ld: item %ld out of turn\n", what, (long)n, (long)i);
    ++parts[t];
    if (first[t] < 0) first[t] = i;
    last[t] = i;
  }
  for (int t = 0; t < nt; ++t) {
    if (parts[t] != p.parts[t]) FAIL("%s n=%ld: task %d has %d of %d items\n", what, (long)n, t, parts[t], p.parts[t]);
    for (int s : succ[t])
      if (last[t] >= first[s]) FAIL("%s n=%ld: task %d claimed before its predecessor %d\n", what, (long)n, s, t);
  }
  // what follows each task: the claim order is topological
  const int words = (nt + 63) / 64;
  std::vector<int> order(nt);
  for (int t = 0; t < nt; ++t) order[t] = t;
  std::sort(order.begin(), order.end(), [&](int a, int b) { return first[a] > first[b]; });
  std::vector<std::vector<uint64_t>> after(nt, std::vector<uint64_t>(words, 0));
  for (int t : order)
    for (int s : succ[t]) {
      after[t][s >> 6] |= 1ull << (s & 63);
      for (int w = 0; w < words; ++w) after[t][w] |= after[s][w];
    }
  // program order: the factorization step by step (a merged update with its last one), then the solve
  std::vector<int> prog(nt);
  for (int t = 0; t < nt; ++t) prog[t] = t;
  auto key = [&](int t) {
    const int kd = p.kind[t], k = p.tk[t];
    const bool tri_of_solve = kd == TK_TRTRI && (p.finv || !p.inv || p.op == TCHOL_OP_SOLVE || k + 1 == Tf);
    std::vector<long> q;
    if (kd == TK_BTRSV || kd == TK_BGEMV)
      q = {2, Ts - k, kd == TK_BTRSV ? 0 : 1};
    else if (kd == TK_FTRSV || kd == TK_FGEMV || tri_of_solve)
      q = {1, k, kd == TK_TRTRI ? 0 : kd == TK_FTRSV ? 1 : 2};
    else
      q = {0, k + len_of(kd) - 1, kd == TK_POTRF ? 0 : kd == TK_TRTRI ? 1 : kd == TK_TRSM ? 2 : 3};
    return q;
  };
  std::stable_sort(prog.begin(), prog.end(), [&](int a, int b) { return key(a) < key(b); });
  enum { A, I, V, Bk, S };
  typedef std::vector<std::array<int, 3>> Cells;
  std::map<std::array<int, 3>, int> writer;
  std::map<std::array<int, 3>, std::vector<int>> readers;
  auto ordered = [&](int a, int b) { return (after[a][b >> 6] >> (b & 63)) & 1; };
  auto cells = [&](Cells& c, int ti, int tk) {  // the factorization's tiles inside tile (ti, tk) of the solve
    for (int i = ti * r; i < std::min(Tf, (ti + 1) * r); ++i)
      for (int k = tk * r; k < std::min(Tf, (tk + 1) * r); ++k)
        if (i >= k) c.push_back({A, i, k});
  };
  auto strips = [&](int k) { return p.inv && std::min(sb, n - k * sb) % 16 == 0; };
  for (int t : prog) {
    const int kd = p.kind[t], i = p.ti[t], j = p.tj[t], k = p.tk[t];
    Cells rd, wr;
    switch (kd) {
      case TK_POTRF:
        wr = {{A, k, k}};
        if (p.finv) wr.push_back({I, k, 0});
        break;
      case TK_TRTRI:
        cells(rd, k, k);
        wr = {{V, k, 0}};
        if (p.inv && !p.finv) wr.push_back({I, k, 0});
        break;
      case TK_TRSM:
        if (p.inv) rd = {{I, k, 0}};
        else rd = {{A, k, k}};
        wr = {{A, i, k}};
        break;
      case TK_SYRK:
        rd = {{A, i, k}};
        wr = {{A, i, i}};
        break;
      case TK_GEMM: case TK_GEMM2: case TK_GEMM4:
        for (int q = k; q < k + len_of(kd); ++q) {
          rd.push_back({A, i, q});
          rd.push_back({A, j, q});
        }
        wr = {{A, i, j}};
        break;
      case TK_FTRSV:
        if (strips(k)) {
          rd = {{V, k, 0}, {Bk, k, 0}};
          wr = {{S, k, 0}};
        } else {
          cells(rd, k, k);
          wr = {{Bk, k, 0}};
        }
        break;
      case TK_FGEMV:
        cells(rd, i, k);
        rd.push_back({strips(k) ? S : Bk, k, 0});
        wr = {{Bk, i, 0}};
        break;
      case TK_BTRSV:
        if (strips(k)) {
          rd = {{V, k, 0}, {S, k, 0}};
        } else {
          cells(rd, k, k);
        }
        wr = {{Bk, k, 0}};
        break;
      case TK_BGEMV:
        cells(rd, k, i);
        rd.push_back({Bk, k, 0});
        wr = {{strips(i) ? S : Bk, i, 0}};
        break;
      default:
        FAIL("%s n=%ld: kind %d\n", what, (long)n, kd);
    }
    auto need = [&](int a, const char* how) {
      if (a != t && !ordered(a, t))
        FAIL("%s n=%ld nb=%ld/%ld: kind %d (%d,%d,%d) not ordered after kind %d (%d,%d,%d): %s\n", what, (long)n, (long)fb,
             (long)sb, kd, i, j, k, p.kind[a], p.ti[a], p.tj[a], p.tk[a], how);
    };
    for (auto& c : rd) {
      auto w = writer.find(c);
      if (w != writer.end()) need(w->second, "read after write");
      else if (c[0] == I || c[0] == V || c[0] == S) FAIL("%s n=%ld: kind %d reads what nothing wrote\n", what, (long)n, kd);
    }
    for (auto& c : wr) {
      auto w = writer.find(c);
      if (w != writer.end()) need(w->second, "write after write");
      for (int x : readers[c]) need(x, "write after read");
      writer[c] = t;
      readers[c].clear();
    }
    for (auto& c : rd) readers[c].push_back(t);
  }
  // every tile factored, every update applied once, every block solved
  std::map<std::array<int, 3>, int> applied;
  int potrf = 0, trsm = 0, syrk = 0, ft = 0, bt = 0, fg = 0, bg = 0;
  for (int t = 0; t < nt; ++t) {
    const int kd = p.kind[t];
    potrf += kd == TK_POTRF;
    trsm += kd == TK_TRSM;
    syrk += kd == TK_SYRK;
    ft += kd == TK_FTRSV;
    bt += kd == TK_BTRSV;
    fg += kd == TK_FGEMV;
    bg += kd == TK_BGEMV;
    if (kd == TK_GEMM || kd == TK_GEMM2 || kd == TK_GEMM4)
      for (int q = p.tk[t]; q < p.tk[t] + len_of(kd); ++q) ++applied[{p.ti[t], p.tj[t], q}];
  }
  const int pf = Tf * (Tf - 1) / 2, ps = Ts * (Ts - 1) / 2;
  if (potrf != Tf || trsm != pf || syrk != pf) FAIL("%s n=%ld: %d POTRF %d TRSM %d SYRK\n", what, (long)n, potrf, trsm, syrk);
  for (int i = 0; i < Tf; ++i)
    for (int j = 1; j < i; ++j)
      for (int q = 0; q < j; ++q)
        if (applied[{i, j, q}] != 1) FAIL("%s n=%ld: update (%d,%d,%d) %d times\n", what, (long)n, i, j, q, applied[{i, j, q}]);
  if (ft > 0 && (ft != Ts || bt != Ts || fg != ps || bg != ps)) FAIL("%s n=%ld: solve tasks\n", what, (long)n);
  // work items: the blocks that cover a task's output at the plan's sizes
  auto cdiv = [](int64_t a, int64_t b) { return (int)((a + b - 1) / b); };
  for (int t = 0; t < nt; ++t) {
    const int kd = p.kind[t], i = p.ti[t], j = p.tj[t];
    const int64_t nb = p.systems[p.sys[t]].nb, mi = std::min(nb, n - i * nb), mj = std::min(nb, n - j * nb);
    int want = -1;
    if (kd == TK_TRSM) want = cdiv(mi, p.inv ? p.split.inv_rows : p.split.trsm_rows);
    if (kd == TK_SYRK) want = cdiv(mi, p.split.syrk_b) * (cdiv(mi, p.split.syrk_b) + 1) / 2;
    if (kd == TK_GEMM) want = cdiv(mi, p.split.gemm1_m) * cdiv(mj, p.split.gemm1_n);
    if (kd == TK_GEMM2 || kd == TK_GEMM4) want = cdiv(mi, p.split.gemm_m) * cdiv(mj, p.split.gemm_n);
    if (kd == TK_FGEMV || kd == TK_BGEMV) want = cdiv(mi, p.split.gemv_rows);
    if (want >= 0 && want != p.parts[t]) FAIL("%s n=%ld: kind %d has %d items, %d cover it\n", what, (long)n, kd, p.parts[t], want);
  }
}

int main(int argc, char** argv) {
  if (argc > 1) drop_kind = std::atoi(argv[1]);
  // tiles that 128 divides (run at 128, the solve at the caller's: 1 to 4 to a side) and
  // others; one tile, ragged last tiles, orders that no 16 divides
  const int64_t sizes[][2] = {{100, 512}, {128, 128}, {500, 256}, {513, 512}, {1000, 128}, {1000, 384}, {1301, 512}, {1537, 256},
                              {1536, 384}, {1600, 512}, {300, 64}, {333, 32}, {257, 16}, {1000, 192}, {2000, 208}, {1500, 144},
                              {1408, 128}, {1409, 128}, {15000, 512}, {13000, 496}};
  int plans = 0;
  for (auto& z : sizes)
    for (int pol : {TCHOL_POLICY_LIST, TCHOL_POLICY_RANK, TCHOL_POLICY_FIFO, TCHOL_POLICY_RANDOM}) {
      if (z[0] > 4000 && pol != TCHOL_POLICY_LIST) continue;
      for (bool inv : {false, true}) {
        auto m = tchol::get_run_merged_plan(z[0], z[1], pol, 5, inv);
        auto f = tchol::get_run_plan(inv ? tchol::OP_FACTOR_INVT : TCHOL_OP_FACTOR, z[0], z[1], pol, 5);
        if (!m || !f) {
          FAIL("no plan for n=%ld nb=%ld\n", (long)z[0], (long)z[1]);
          continue;
        }
        check(*m, inv ? "merged, inverses" : "merged, substitution");
        check(*f, inv ? "factor, inverses" : "factor");
        plans += 2;
      }
    }
  // nothing to do: no merged plan to run, and a factorization without tasks
  if (tchol::get_run_merged_plan(0, 512, TCHOL_POLICY_LIST, 0, true)) FAIL("a merged plan of order 0\n");
  auto empty = tchol::get_run_plan(TCHOL_OP_FACTOR, 0, 512, TCHOL_POLICY_LIST, 0);
  if (!empty || empty->ntask() != 0) FAIL("the factorization of order 0\n");
  std::printf("run plans: %d checked, %ld failures\n", plans, failures);
  return failures == 0 ? 0 : 1;
}
