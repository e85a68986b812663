// Host check of the plan of the fused pass over B (plan_fused in libsdp): on
// devices of several sizes every cluster has a unit for each of its members,
// and the tiles cover every row and column of every dense instance once, with
// partial sums of their own.  Run by test_fused_plan_cpu.py; no GPU work.
#include <cstdio>
#include <set>
#include <vector>

#include "sdp_internal.h"

static int g_fail = 0, g_plans = 0;
#define CHECK(c)                                                             \
  do {                                                                       \
    if (!(c)) {                                                              \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c);   \
      ++g_fail;                                                              \
    }                                                                        \
  } while (0)

static InstDesc instance(int m, int nnz, int format) {
  InstDesc d{};
  d.m = m;
  d.nnz = nnz;
  d.ld = (nnz + 63) / 64 * 64;
  d.ldm = (m + 63) / 64 * 64;
  d.a_format = format;
  return d;
}

static void check(const std::vector<InstDesc> &inst, int units) {
  const FusedPlan p = plan_fused(inst, units);
  if (p.tiles.empty()) return;
  ++g_plans;
  CHECK((int)p.tiles.size() <= units);
  CHECK(p.part_first.size() == 2 * inst.size());
  std::set<int64_t> parts;
  int64_t doubles = 0;
  for (size_t i = 0; i < inst.size(); ++i) {
    const InstDesc &d = inst[i];
    int next = 0;
    int64_t groups = 0, cols = 0;
    for (const FusedTile &t : p.tiles) {
      if (t.inst != (int)i) continue;
      CHECK(d.a_format == 0 && t.row0 < t.row1 && t.row1 <= d.m);
      CHECK(t.member >= 0 && t.member < t.size && t.chunk % 64 == 0 && t.chunk <= 4096);
      CHECK((int64_t)t.member * t.chunk < d.ld);
      if (t.member == 0) {   // the members of a cluster follow one another
        CHECK(t.row0 == next && parts.insert(t.part_off).second);
        CHECK(t.part_off == p.part_first[2 * i] + groups * d.ld);
        next = t.row1;
        ++groups;
        doubles += d.ld;
        cols = 0;
      }
      CHECK(t.member * (int64_t)t.chunk == cols);
      cols += t.chunk;
      if (t.member == t.size - 1) CHECK(cols >= d.ld);
    }
    if (d.a_format == 0 && d.m > 0) {
      CHECK(next == d.m && groups == p.part_first[2 * i + 1]);
    } else {
      CHECK(groups == 0);
    }
  }
  CHECK(doubles == p.part_doubles);
}

int main() {
  const int units[] = {1, 8, 32, 38, 64, 104, 228, 256, 304};
  const int rows[] = {1, 7, 41, 301, 1000, 4000}, cols[] = {100, 4000, 4335, 9480, 31880, 61000};
  for (int u : units)
    for (int m : rows)
      for (int n : cols)
        for (int copies : {1, 3, 12, 60, 129}) {
          std::vector<InstDesc> v(copies, instance(m, n, 0));
          check(v, u);
          v.insert(v.begin() + copies / 2, instance(500, 3000, 1));   // a sparse one between
          v.push_back(instance(m + 13, n / 2 + 1, 0));
          check(v, u);
        }
  std::printf("%d plans, %d failed checks\n", g_plans, g_fail);
  return g_fail != 0;
}
