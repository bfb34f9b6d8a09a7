// Internal representation behind the C ABI handles.
#pragma once
#include <stdint.h>
#include <string>
#include <vector>
#include "../../include/opara.h"
#include "kernel_args.h"

namespace opara {
// Host copy of a persistent executor's workspace (header, counters, flags, item table,
// predecessor lists, operator records in launch-queue order) and what the launch needs.
struct PersistImage {
  std::vector<unsigned char> host;
  int32_t prefix = 0;               // leading queue operators launched as ordinary kernels
  int32_t np_ops = 0, total = 0;    // operators inside the kernel, work items
  uint32_t wgs = 0, lds_bytes = 0;  // workgroups of the launch, dynamic LDS per workgroup
  bool f16 = false, tiled = false;  // tiled: some operator inside takes the 128 x 64 tile
};
}  // namespace opara

struct opara_dag {
  int32_t n = 0;
  std::vector<opara_op_desc> ops;
  std::vector<void *> ext;
  opara_limits lim{};
  // CSR adjacency over operator ids; predecessors in argument order, deduplicated.
  std::vector<int32_t> pred_off, pred, succ_off, succ;
  std::vector<int32_t> topo, tindex;
  std::vector<opara::KernelPlan> plan;          // graph executors (and the demand table)
  std::vector<opara::KernelPlan> plan_persist;  // persistent executor
  std::vector<opara_demand> dem;
  std::vector<int32_t> stream_of;   // empty until opara_assign_streams
  int32_t n_streams = 0;
  std::vector<int32_t> order;       // empty until opara_order_launch
  uint64_t order_gen = 0;           // counts the launch queues computed so far
  // Workspace image of the persistent executor as opara_run_persistent_noalloc last built it
  // (kept here so that the asynchronous upload reads memory that outlives the call).
  opara::PersistImage noalloc_image;
  uint64_t noalloc_gen = 0;         // order_gen the image belongs to, 0 = none
};

namespace opara {

struct KernelResource { const char *name; uint32_t vgprs, agprs, lds_bytes; };
extern const KernelResource kKernelResources[K_COUNT];

void set_error(const char *fmt, ...);

// What the kernels' fast_div takes for a divisor.
inline uint32_t div_magic(int64_t d) { return d > 1 ? (uint32_t)((1ull << 32) / (uint64_t)d) : 0xffffffffu; }

// One flag per entry of the opara_sync_edges list (same order): 0 = the dependency is
// implied by other ordering constraints and needs no synchronisation of its own.
int sync_keep_mask(const opara_dag *g, std::vector<uint8_t> *keep);

// Chooses the kernel, grid and arguments for operator `v`; `in[i]` are the resolved
// device pointers of its inputs.  kPlanGraph is the plan the graph executors launch and the
// demand table describes (also the starting point of the fused executor); kPlanPersistent the
// one the persistent executor runs (two contraction kernels, its own hand-over point between
// them).  Returns an opara_status.
enum { kPlanGraph = 0, kPlanPersistent = 1 };
int plan_op(const opara_op_desc &op, const void *const *in, int kind, KernelPlan *out);

// Operators of consecutive waves that the fused executor runs as one kernel, each
// the only operator of its wave; the kernel is launched in the place of the first.
struct Merge { int32_t count, ops[3]; KernelPlan plan; };
std::vector<Merge> find_merges(const opara_dag *g);
// Concatenations whose parts the element-wise operators that compute them write in place.
struct ConcatMerge { int32_t concat; std::vector<int32_t> ops; std::vector<EltArgs> args; };
std::vector<ConcatMerge> find_concat_merges(const opara_dag *g, const std::vector<Merge> &taken);

// Tile shapes of contractions that run together; only for kernels whose shape is open.
bool tile_choice_open(int kernel_id);
// The same contraction with an element-wise operator after it (KernelPlan::tail); -1: none.
int tail_kernel(int kernel_id);
void choose_tiles(KernelPlan *const *plans, int n, bool grouped);

}  // namespace opara
