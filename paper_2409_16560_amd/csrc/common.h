// Internal helpers shared by the HIP translation units of libdsbd (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include "dsbd.h"

#define DSBD_MAX_TREE_NODES 64

#define DSBD_HIP_LAUNCH_CHECK()                      \
  do {                                               \
    hipError_t e__ = hipGetLastError();              \
    if (e__ != hipSuccess) return DSBD_ERR_HIP;      \
  } while (0)

static inline size_t dsbd_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Carves 256-byte aligned pieces out of a caller-supplied workspace.
struct WorkspaceCarver {
  char* base;
  size_t used;
  explicit WorkspaceCarver(void* p) : base(static_cast<char*>(p)), used(0) {}
  template <typename T>
  T* take(size_t count) {
    used = dsbd_align_up(used, 256);
    T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
    used += count * sizeof(T);
    return p;
  }
  size_t total() const { return dsbd_align_up(used, 256); }
};

// Tuning overrides and test hooks from the environment, read once per process (knobs.hip).
struct DsbdKnobs {
  int attn_nsplit;             // DSBD_ATTN_NSPLIT: KV splits per (tree, KV head, row block); 0 = the plan's choice
  int verify_g;                // DSBD_VERIFY_G: workgroups per prompt of the layer kernel; 0 = the plan's choice
  bool verify_trace;           // DSBD_VERIFY_TRACE: timeline of the layer kernel into the workspace ...
  int verify_trace_wg;         // ... of workgroup N - 1 when the variable holds N > 1 (else of the first)
  long long verify_sync_limit_us;   // DSBD_VERIFY_SYNC_LIMIT_US: bound of every wait of the layer kernel; 0 = default
  int verify_mute_wg;          // DSBD_VERIFY_TEST_MUTE_WG: test hook, this workgroup withholds its first post; -1 = none
  int verify_lds_slice;        // DSBD_VERIFY_LDS_SLICE: largest joint slice kept in the LDS; -1 = the plan's choice
  int warp_fast;               // DSBD_WARP_FAST: 0 = the warped rows' entries are always selected one by one, as where they crowd
  int draft_wait_us;           // DSBD_DRAFT_WAIT_US: how long a draft step's drawing workgroups wait for a chunk before they take it
                               // themselves (0: they always do); -1 = default
  int event_fence;             // DSBD_EVENT_FENCE: 1 = the library's cross-stream events keep HIP's system-scope fence; 0 = they order
                               // device work only (no cache write-back for the host's sake at every one)
};
const DsbdKnobs& dsbd_knobs();

// The base of a launch's exchange tags: a number of its own for every launch of the process, with 24 bits below it for the
// launch's exchanges (knobs.hip).
unsigned long long dsbd_launch_nonce();

// Measurement hook (timing.hip).  When timing is enabled for `kernel_id`, the launch goes through HIP's extended
// launch call, which stamps a pair of events with the kernel's own start and end on the device (what a profiler's
// kernel trace reports); a pair of hipEventRecord calls around an ordinary launch would also count the dispatch
// latency on either side (2-3 us).  Otherwise an ordinary launch.
bool dsbd_timing_events(int kernel_id, hipEvent_t* start, hipEvent_t* stop);
template <typename F, typename... Args>
inline void dsbd_launch(int kernel_id, F kernel, dim3 grid, dim3 block, unsigned int lds_bytes, hipStream_t stream,
                        Args... args) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (dsbd_timing_events(kernel_id, &e0, &e1))
    hipExtLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, e0, e1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, lds_bytes, stream, args...);
}
