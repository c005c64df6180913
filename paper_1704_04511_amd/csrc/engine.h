// Lock-step engine for many reconstructions (see engine.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <map>
#include <tuple>
#include <vector>

#include "../../include/slrx.h"
#include "kernels.h"
#include "plan.h"

namespace slrx {

// Eigen-decomposition buffers for up to `cap` problems of size n, strided.
struct EigGroup {
  int n = 0, cap = 0;
  void* mem = nullptr;  // one allocation holding every buffer below
  EighBufs bufs;        // pointers into mem, strides for problem b
  int* tree = nullptr;  // divide-and-conquer tree for n (device)
  std::vector<int> level_start, node_sizes;
  bool clear_stall = false;  // the next resident tridiagonalisation clears the give-up flag
  ~EigGroup();
};

// Table of a grouped launch (kernels.h CgSlice, WeightSlice): the device copy, a pinned
// staging copy, and the host copy it was made from (rewritten only when the problems
// of the group change).
template <class T>
struct DevTable {
  std::vector<T> host;
  T* dev = nullptr;
  T* pinned = nullptr;
  size_t cap = 0;                // entries of dev and pinned
  hipEvent_t copied = nullptr;   // the last upload from pinned has run
  bool pending = false;
  long step = 0;                 // engine step that last used it
  DevTable() = default;
  DevTable(const DevTable&) = delete;
  DevTable& operator=(const DevTable&) = delete;
  ~DevTable() {
    if (dev) (void)hipFree(dev);
    if (pinned) (void)hipHostFree(pinned);
    if (copied) (void)hipEventDestroy(copied);
  }
  // The table on the device, in order on stream s (whose launches alone read it).
  slrx_status upload(const std::vector<T>& h, hipStream_t s);
};
typedef std::tuple<int, int, int, int> WeightKey;  // N1, N2, M, part of the group

// Shared state of the batched eigen-decompositions and the grouped CG (own
// streams and events).
struct BatchEig {
  hipStream_t stream = nullptr;
  hipEvent_t ev = nullptr;       // eigenpairs ready
  hipEvent_t ev_free = nullptr;  // every reader of the group buffers has run
  hipEvent_t ev_w = nullptr;     // the grouped weight updates so far have run
  bool have_free = false;
  long step = 0;                 // engine steps so far
  std::map<int, EigGroup> groups;
  hipStream_t cg_stream = nullptr;  // grouped CG passes
  hipEvent_t ev_cg = nullptr;       // a group's CG has run
  std::map<std::pair<int, int>, DevTable<CgSlice>> cg_tables;  // by (M, n_cg)
  std::map<WeightKey, DevTable<WeightSlice>> weight_tables;
  size_t allocated() const;  // device bytes held by the groups and tables
  ~BatchEig();
};

// Device bytes the shared eigen-decomposition buffers hold per problem of Gram
// size n (an upper bound of what one more problem of that size adds).
size_t engine_problem_bytes(int n);
// Shrink the groups to at most keep[n] problems of size n (absent: none) and drop the
// tables of grouped launches that the last step did not use (all of them if nothing is
// kept), after the work that reads them has finished (synchronises the engine's streams).
slrx_status engine_trim(BatchEig& be, const std::map<int, int>& keep);

// Start a problem: masked data, initial iterate, start event, iteration 0.  columns: its
// tridiagonalisations by column launches (the repeat of a run whose resident launch gave up).
slrx_status engine_begin(slrx_plan* pl, bool columns = false);
// Enqueue one outer iteration for every given problem that has iterations
// left (no host synchronisation).
slrx_status engine_step(const std::vector<slrx_plan*>& plans, BatchEig& be);
// Forget that resident tridiagonalisations gave up: each group's next one clears its flag.
// Called when no run that met the flag goes on, or once the first of them is known.
void engine_clear_stalls(BatchEig& be);
// Wait for everything the engine has enqueued (after a failed step).
void engine_drain(BatchEig& be);
// Record the completion event of a problem whose iterations are done.
slrx_status engine_end(slrx_plan* pl);

}  // namespace slrx
