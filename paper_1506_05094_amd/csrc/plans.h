// Host-side rules of the launch chains as plain functions of numbers (no device, no
// allocation), and the sizes that they share with the kernels.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

namespace srmd {

// ---- staged lists (k_list_stage and the staged step and force kernels)

constexpr int kStageSlots = 256;   // sorted slots of a unit
constexpr int kStageCells = 1600;  // cells of a unit's region at most
constexpr int kStageTest = 4;      // candidates tested together
constexpr int kRing = 32;          // list slots per lane that the builders stage in LDS

constexpr size_t kLdsBytes = 160 * 1024;    // of a compute unit
constexpr size_t kStageListStatic = 1024;   // k_list_stage's arrays of fixed size (650 bytes), rounded up

// Dynamic LDS of k_list_stage for regions of at most cap particles: their positions
// (16 bytes each), the cells' first places and the entry rings (2 bytes each).
constexpr size_t stage_list_bytes(int cap) {
  return 16 * (size_t)(cap + 1 + kStageTest) + 2 * (size_t)(kStageCells + 8) + 2 * (size_t)kRing * kStageSlots;
}

struct StagePlan {
  int cap = 0;  // particles the copy of one unit's region holds at most; 0: plain lists
  int lds = 0;  // particles the LDS of a step or force workgroup holds
};

// Large systems with the thread-per-particle list and blocks of whole units.  What a unit
// copies is its slab (about 5 x 5 cells and the layers that hold its slots) widened by the
// list radius, and a third more (over jittered lattices of 16 000 to 256 000 particles of
// both fluids no unit needed more than 1.15 times the estimate, nor did those that end one
// column and begin the next).  10 cells along every axis, so that a test without image
// arithmetic never sees a distance of half a box side.  n particles in the box L, nc cells
// in tiles of about tile_q (x, y), blocks of ppb particles.
inline StagePlan stage_plan(int n, const double *L, const int *nc, const int *tile_q, double reach, int tp, int ppb) {
  StagePlan plan;
  if (ppb % kStageSlots != 0 || nc[0] < 10 || nc[1] < 10 || nc[2] < 10 || n >= (1 << 28)) return plan;
  const double pi = 3.14159265358979323846;
  const double rho = n / (L[0] * L[1] * L[2]), a = tile_q[0] * L[0] / nc[0], b = tile_q[1] * L[1] / nc[1];
  const double layers = kStageSlots / (rho * a * b) / (L[2] / nc[2]);
  const double h = (layers + 0.6) * L[2] / nc[2];
  const double region = rho * (a * b * h + 2.0 * reach * (a * b + b * h + a * h) + pi * reach * reach * (a + b + h) +
                               4.0 / 3.0 * pi * reach * reach * reach);
  const double cells = (tile_q[0] + 4.0) * (tile_q[1] + 4.0) * (layers + 5.0);
  const int units = ppb / kStageSlots;
  // with one unit per block, what lets five blocks share a compute unit's LDS (32 000
  // bytes with the static 2.4 KB) if that is still a fifth more than the estimate
  int cap = std::max(1024, (int)std::min(1.35 * region, 1e9));
  if (tp == 1 && units == 1 && 1.2 * region <= 1850) cap = std::min(cap, 1850);
  if (units * (cap + 1.0) > 9400 || 1.3 * cells > kStageCells) return plan;
  // The list build holds cell starts and rings beside a region, so that the largest regions
  // leave it less than the step kernel's 9400 places: what fits (8946), which is still 1.28
  // times the estimate at the largest cap.
  constexpr int kMost = (int)((kLdsBytes - kStageListStatic - stage_list_bytes(0)) / 16);
  cap = std::min(cap, kMost);
  plan.cap = cap;
  plan.lds = units * (cap + 1);
  return plan;
}

// ---- run-ahead chains (large systems)

// Steps enqueued after a rebuild slot where lists last life steps on average.  A slot that is
// not due costs 7.5 us (five kernels that exit), a step that waits for the next slot 1.5 us.
// So the slots follow the life below 3 (a step at a life of 1: 60.7 us against 71.5 with 8
// slots at 16 000 particles, 101.8 against 115.2 at 64 000; at 2: 37.9 / 42.2 and 62.0 /
// 67.6; at 2.94: 33.1 / 32.5); from there the steps that wait up to 8 cost less than a second
// slot, and up to 32 the next larger count less than a third one.
constexpr int kAheadFirst = 8;  // before the life is known
inline int ahead_slots_for(double life) {
  return life <= 1.2 ? 1 : life <= 2.75 ? 2 : life <= 8.5 ? 8 : life <= 12.5 ? 12 : life <= 20.5 ? 20 : 32;
}

}  // namespace srmd
