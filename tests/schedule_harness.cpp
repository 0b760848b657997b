// Host harness for the stage kernel's launch rules (csrc/schedule.h), linked
// with the library and run by tests/test_schedule_cpu.py.  Reads lines
//   f64(0/1) bs nb counters(0/1) n, then n times: knob value
// sets the knobs one call each on a new grid, the way the Python binding does
// (read the schedule, change the knob, write it back), and prints the schedule
// read at the end, then the RK stages' and the rhs's resolved ones, and whether
// the RK stages load their operands early with 1, 2 and 4 runs of planes.
//   schedule_harness runs: lines "tiles per_cu cus bs", prints plane_runs
#include <cstdio>
#include <cstring>

#include "schedule.h"
#include "wacm_internal.h"

static int32_t* knob(wacm_schedule& s, const char* name) {
  if (!strcmp(name, "wg_per_cu")) return &s.wg_per_cu;
  if (!strcmp(name, "xcd_map")) return &s.xcd_map;
  if (!strcmp(name, "prefetch")) return &s.prefetch;
  if (!strcmp(name, "nontemporal")) return &s.nontemporal;
  if (!strcmp(name, "tile_rows")) return &s.tile_rows;
  return !strcmp(name, "pen_split") ? &s.pen_split : nullptr;
}

static void show(const wacm_schedule& s) {
  printf("%d %d %d %d %d %d ", s.wg_per_cu, s.xcd_map, s.prefetch, s.nontemporal, s.tile_rows,
         s.pen_split);
}

int main(int argc, char**) {
  if (argc > 1) {
    long tiles;
    int per_cu, cus, bs;
    while (scanf("%ld %d %d %d", &tiles, &per_cu, &cus, &bs) == 4)
      printf("%d\n", wacm::plane_runs(tiles, per_cu, cus, bs));
    return 0;
  }
  int f64, bs, counters, n;
  long nb;
  while (scanf("%d %d %ld %d %d", &f64, &bs, &nb, &counters, &n) == 5) {
    wacm_grid g;
    for (int i = 0; i < n; ++i) {
      char name[32];
      int v;
      if (scanf("%31s %d", name, &v) != 2) return 2;
      wacm_schedule s;
      if (wacm_get_schedule(&g, &s)) return 3;
      if (strcmp(name, "none")) *knob(s, name) = v;
      if (wacm_set_schedule(&g, &s)) return 4;
    }
    wacm_schedule s;
    wacm_get_schedule(&g, &s);
    show(s);
    show(wacm::stage_schedule(g.sched, f64 != 0, bs, nb, counters != 0));
    show(wacm::rhs_schedule(g.sched));
    for (int runs = 1; runs <= 4; runs *= 2)
      printf("%d ", (int)wacm::early_loads(
                        wacm::stage_schedule(g.sched, f64 != 0, bs, nb, counters != 0),
                        f64 != 0, runs));
    printf("\n");
  }
  return 0;
}
