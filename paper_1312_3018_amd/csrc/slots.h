// Multi-source (slot) engine: up to 64 BFS or SSSP queries advancing together
// over one GPU partition, joining and retiring at superstep boundaries.
#pragma once
#include <stdint.h>

#include "ms.h"

namespace tg {

enum { kSlotBfs = 0, kSlotSssp = 1 };

// Per-slot output pointer and the superstep at which the slot's root had
// level 0.  Passed by value.
struct SlotTable {
  int32_t *out[kSlots];
  int32_t join[kSlots];
};

struct SlotEngine {
  tg_partition *p = nullptr;
  int kind = kSlotBfs;
  hipStream_t s = nullptr;
  Workspace ws;       // frontier queue, touched bitmap (bits_a), flags
  DevArena arena;
  int64_t cap_n = -1;  // vertices the buffers below are for
  unsigned long long *visited = nullptr, *front[2] = {nullptr, nullptr}, *next = nullptr;
  int cur = 0;         // front[cur] holds the frontier's masks
  MsState *state = nullptr;    // device (its plan takes the place of ws.plan)
  MsState *h_state = nullptr;  // pinned copy
  // BFS levels, [n][kSlots]: one byte each (valid where `visited` has the
  // slot), or from a slot's 255th level on, until the engine is empty again,
  // int32 in `wide`
  uint8_t *lev = nullptr;
  int32_t *wide = nullptr;
  bool is_wide = false;
  int32_t *dist = nullptr;  // SSSP: [n][kSlots]
  // SSSP overflow: per vertex, the slots whose candidate for it did not fit
  // in int32; ovf_slots[0] = the slots with any such mark, [1] = scratch
  unsigned long long *ovf = nullptr, *ovf_slots = nullptr;
  unsigned long long *h_ovf = nullptr;  // pinned copies, then the counters' sums (MS_COUNTERS)
  SlotTable tab{};
  int64_t mu[kSlots] = {};      // BFS: edges of the vertices a slot has not had on a frontier
  unsigned long long busy = 0;  // slots in use
  unsigned long long alive = 0; // slots with a frontier
  int64_t step = 0;             // superstep counter (levels are step - join)
  int64_t supersteps = 0;
  bool have_queue = false;      // a frontier exists: in the queue, or (dense) in front[cur] only
  bool dense = false;
  bool joined = false;          // slots joined since the last superstep
  unsigned long long pull_edges = 0;  // SSSP: edges of the frontier
  SearchWork done;                    // since init
  unsigned long long counted[MS_COUNTERS] = {};  // the counters when last read
  bool clean = false;           // buffers hold no trace of an earlier slot
  ~SlotEngine();
  // Empty engine on `part`; buffers of an earlier run on it are kept.
  int init(tg_partition *part, int kind, hipStream_t stream);
  int free_slot() const;
  // Slots `first`.. start at the given local roots (BFS and SSSP results go
  // to tab.out).  Takes effect at the next superstep.
  int join(int first, int count, const int32_t *roots_local);
  // One superstep; `finished` gets the slots whose frontier became empty.
  // launch_step() only enqueues (so several engines can overlap on the
  // device); finish_step() waits for it.
  int superstep(unsigned long long *finished);
  int launch_step();
  int finish_step(unsigned long long *finished);
  // Release finished slots: write their levels or distances to tab.out
  // (original ids), and set in *overflow the SSSP slots among them whose true
  // distances do not all fit below INT32_MAX, the exact verdict of sssp().
  int retire(unsigned long long mask, unsigned long long *overflow);

 private:
  int widen();
  int launch_sparse(unsigned long long pulled);
  int launch_dense();
};

int slots_run_batch(tg_partition *p, int kind, const int32_t *roots, int32_t nr, int32_t *out, hipStream_t s,
                    int64_t *supersteps_out, SearchWork *work);
// Give the engine of `kind` and its buffers back.
void slots_drop(tg_partition *p, int kind);

}  // namespace tg
