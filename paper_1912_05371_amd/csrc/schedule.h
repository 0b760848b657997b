// Which variant of the stage kernel a launch takes: what of the grid's
// schedule is left to the library (-1) is chosen here by element type and
// size.  Host code without HIP, so that the rules can be tested anywhere.
#pragma once

#include <cstdint>

#include "wacm.h"

namespace wacm {

// Resolved xcd_map of a launch that takes its items from work counters of the
// call's own (in its work buffer), not the grid's.
constexpr int XCD_OWN_COUNTERS = 3;

// Resolved prefetch of tiles that the library chose: see early_loads.
constexpr int PREFETCH_TILES = 2;

// Whether an RK step without an xcd_map of its own takes tiles from work
// counters: from 4096 blocks of 24^3 on (ms per step at 6000 blocks, static ->
// counters: FP64 9.40 -> 9.20, FP32 whole blocks 5.48 -> tiles 5.30; at 20028
// blocks FP64 31.4 -> 30.0; no gain at 2024 blocks, for 16^3, or for FP32 32^3).
inline bool large_grid(bool f64, int bs, int64_t nb) {
  return (bs == 24 || (bs == 32 && f64)) &&
         nb * (int64_t)(bs * bs * bs) >= (int64_t)4096 * 24 * 24 * 24;
}

// The RK stages' schedule.  Left to the library: tiles of 8 rows with early
// epilogue loads for FP64 blocks of 24^3 and more (ms per step, whole blocks ->
// tiles: 24^3 1.10 -> 1.07 at 603 blocks, 10.30 -> 9.40 at 6000; 32^3 8.91 ->
// 5.17 at 1520, where a whole block's 16 waves leave 128 registers and spill).
// FP32 keeps whole blocks below the size of large_grid (24^3, 2024 blocks: 1.90
// against 1.95).  A knob that is set is taken as it is, and setting one leaves
// the others' choice as it was; only the early loads go with tiles that are the
// library's (with tile_rows 8 set, prefetch -1 has always meant late for FP64).
// counters: the call has room for counters of its own.
inline wacm_schedule stage_schedule(const wacm_schedule& set, bool f64, int bs, int64_t nb,
                                    bool counters) {
  wacm_schedule s = set;
  const bool large = counters && large_grid(f64, bs, nb);
  if (s.tile_rows < 0 && s.prefetch < 0 && f64 && bs >= 24) s.prefetch = PREFETCH_TILES;
  if (s.tile_rows < 0) s.tile_rows = (f64 && bs >= 24) || large ? 8 : 0;
  if (s.xcd_map < 0) s.xcd_map = large ? XCD_OWN_COUNTERS : 1;
  return s;
}

// Whether a launch whose planes are cut into `runs` loads U^n and the
// accumulator early: as set; left to the library, early for FP32 and, in whole
// columns, for its FP64 tiles.  (Late against early with 2 runs, FP64 tiles: no
// mask 1.02 to 1.05, sphere 0.89 to 0.91, plate 0.89 to 0.96.)
inline bool early_loads(const wacm_schedule& resolved, bool f64, int runs) {
  if (resolved.prefetch == PREFETCH_TILES) return runs == 1;
  return resolved.prefetch < 0 ? !f64 : resolved.prefetch != 0;
}

// Runs of planes per tile (1, 2 or 4), for `per_cu` resident workgroups on each
// of `cus` compute units.  A workgroup marches through its planes one memory
// latency apart, so a grid of few tiles ends sooner cut along z: 64 blocks of
// 16^3, FP64, 27 -> 13 us per stage with 4 runs.  Large grids keep whole
// columns: each run reads 6 planes of its neighbours.
//   In units of a plane's latency, q workgroups that a compute unit holds
// together take p + 3 for p planes each, or 0.65 q times that where their
// traffic bounds them; the fullest unit's rounds add up.  Over 1364 measurements
// (60 to 3400 blocks of 16^3 to 32^3, both types, rhs and RK steps, without and
// with a mask) that takes 1.5% more than the best of 1, 2 and 4, and 12 of them
// are more than 1.5% (at most 6.5%) slower than whole columns; counting rounds
// of the whole chip alone: 1.8%, and 96 of them, up to 16% (498 blocks of 16^3,
// rhs, FP32: 32.2 us whole, 36.0 in 2 runs).
inline int plane_runs(int64_t tiles, int per_cu, int cus, int bs) {
  auto cost = [&](int n) {
    auto round = [](int64_t q) { return q * 0.65 > 1.0 ? q * 0.65 : q > 0 ? 1.0 : 0.0; };
    const int64_t k = (tiles * n + cus - 1) / cus;
    return ((double)bs / n + 3.0) * ((double)(k / per_cu) * round(per_cu) + round(k % per_cu));
  };
  int best = 1;
  double c = cost(1);
  for (int n = 2; n <= 4; n *= 2)
    if (const double d = cost(n); d < c) {
      c = d;
      best = n;
    }
  return best;
}

// The schedule of the rhs alone: whole blocks, statically mapped.
inline wacm_schedule rhs_schedule(const wacm_schedule& set) {
  wacm_schedule s = set;
  if (s.tile_rows < 0) s.tile_rows = 0;
  if (s.xcd_map < 0) s.xcd_map = 1;
  return s;
}

}  // namespace wacm
