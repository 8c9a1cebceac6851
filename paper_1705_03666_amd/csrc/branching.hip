// Launchers of the branching kernels (Sec. 3.1-3.2) with psi and g read from
// the staged term table; a problem-specialised instantiation compiled at run
// time is launched through the module API instead (BranchLaunch::spec).
#include <hip/hip_runtime.h>

#include "branch_kernels.hpp"
#include "pdd_kernels.hpp"

namespace pdd {

// (The launchers with blocks != nullptr only say how many of the kernel's
// blocks a compute unit holds.)
#define PDD_BLOCKS(KERNEL) \
  if (blocks != nullptr) return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, KERNEL, kBlock, 0)

template <typename R, int LAYOUT>
static hipError_t launch_branch_bvp_t(const BranchBvpLaunch& L, hipStream_t st, int* blocks) {
  switch (L.P->dim) {
    case 1:
      PDD_BLOCKS((k_branch_bvp<R, 1, LAYOUT>));
      hipLaunchKernelGGL((k_branch_bvp<R, 1, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, *L.B, L.items,
                         L.n_items, L.qhead, L.istat, L.dump_val, L.dump_segs, L.trees, (StackEntry<R>*)L.stack,
                         L.stack_entries, L.rings);
      break;
    case 2:
      PDD_BLOCKS((k_branch_bvp<R, 2, LAYOUT>));
      hipLaunchKernelGGL((k_branch_bvp<R, 2, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, *L.B, L.items,
                         L.n_items, L.qhead, L.istat, L.dump_val, L.dump_segs, L.trees, (StackEntry<R>*)L.stack,
                         L.stack_entries, L.rings);
      break;
    default:
      PDD_BLOCKS((k_branch_bvp<R, 3, LAYOUT>));
      hipLaunchKernelGGL((k_branch_bvp<R, 3, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, *L.B, L.items,
                         L.n_items, L.qhead, L.istat, L.dump_val, L.dump_segs, L.trees, (StackEntry<R>*)L.stack,
                         L.stack_entries, L.rings);
      break;
  }
  return hipGetLastError();
}

static hipError_t dispatch_bvp(const BranchBvpLaunch& L, hipStream_t st, int* blocks) {
  if (L.spec != nullptr) {
    if (blocks != nullptr) return hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(blocks, L.spec, kBlock, 0);
    // same argument list as k_branch_bvp; the parameter blocks are passed by value
    const TreeItems* items = L.items;
    int n_items = L.n_items;
    uint32_t* qhead = L.qhead;
    ItemStat* istat = L.istat;
    double* dump_val = L.dump_val;
    int64_t* dump_segs = L.dump_segs;
    int64_t trees = L.trees, stack_entries = L.stack_entries;
    void* stack = L.stack;
    double* rings = L.rings;
    void* args[] = {(void*)L.P, (void*)L.B, &items, &n_items, &qhead, &istat, &dump_val, &dump_segs,
                    &trees, &stack, &stack_entries, &rings};
    return hipModuleLaunchKernel(L.spec, (unsigned)L.grid, 1, 1, kBlock, 1, 1, 0, st, args, nullptr);
  }
  if (L.fp32) return launch_branch_bvp_t<float, RNG_QUAD24>(L, st, blocks);
  if (L.layout == RNG_QUAD24) return launch_branch_bvp_t<double, RNG_QUAD24>(L, st, blocks);
  return launch_branch_bvp_t<double, RNG_PAIR52>(L, st, blocks);
}

template <typename R, int LAYOUT>
static hipError_t launch_branch_t(const BranchLaunch& L, hipStream_t st, int* blocks) {
  switch (L.P->dim) {
    case 1:
      PDD_BLOCKS((k_branch<R, 1, LAYOUT>));
      hipLaunchKernelGGL((k_branch<R, 1, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, L.items, L.n_items,
                         L.qhead, L.istat, L.dump_val, L.dump_segs, L.trees, (StackEntry<R>*)L.stack,
                         L.stack_entries);
      break;
    case 2:
      PDD_BLOCKS((k_branch<R, 2, LAYOUT>));
      hipLaunchKernelGGL((k_branch<R, 2, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, L.items, L.n_items,
                         L.qhead, L.istat, L.dump_val, L.dump_segs, L.trees, (StackEntry<R>*)L.stack,
                         L.stack_entries);
      break;
    default:
      PDD_BLOCKS((k_branch<R, 3, LAYOUT>));
      hipLaunchKernelGGL((k_branch<R, 3, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, L.items, L.n_items,
                         L.qhead, L.istat, L.dump_val, L.dump_segs, L.trees, (StackEntry<R>*)L.stack,
                         L.stack_entries);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_branch_bvp(const BranchBvpLaunch& L, hipStream_t st) { return dispatch_bvp(L, st, nullptr); }

int branch_bvp_blocks(const BranchBvpLaunch& L) {
  int n = 0;
  return dispatch_bvp(L, nullptr, &n) == hipSuccess ? n : 0;
}

size_t branch_ring_bytes(int n_times) { return sizeof(double) * (size_t)kTreeRing * (size_t)n_times; }
size_t branch_stack_entry_bytes(bool fp32) { return fp32 ? sizeof(StackEntry<float>) : sizeof(StackEntry<double>); }
int branch_lds_depth(bool fp32) { return fp32 ? lds_depth<float>() : lds_depth<double>(); }

static hipError_t dispatch_branch(const BranchLaunch& L, hipStream_t st, int* blocks) {
  if (L.spec != nullptr) {
    if (blocks != nullptr) return hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(blocks, L.spec, kBlock, 0);
    // same argument list as k_branch; the parameter block is passed by value
    const TreeItems* items = L.items;
    int n_items = L.n_items;
    uint32_t* qhead = L.qhead;
    ItemStat* istat = L.istat;
    double* dump_val = L.dump_val;
    int64_t* dump_segs = L.dump_segs;
    int64_t trees = L.trees, stack_entries = L.stack_entries;
    void* stack = L.stack;
    void* args[] = {(void*)L.P, &items, &n_items, &qhead, &istat, &dump_val, &dump_segs, &trees, &stack,
                    &stack_entries};
    return hipModuleLaunchKernel(L.spec, (unsigned)L.grid, 1, 1, kBlock, 1, 1, 0, st, args, nullptr);
  }
  if (L.fp32) return launch_branch_t<float, RNG_QUAD24>(L, st, blocks);
  if (L.layout == RNG_QUAD24) return launch_branch_t<double, RNG_QUAD24>(L, st, blocks);
  return launch_branch_t<double, RNG_PAIR52>(L, st, blocks);
}

hipError_t launch_branch(const BranchLaunch& L, hipStream_t st) { return dispatch_branch(L, st, nullptr); }

int branch_blocks(const BranchLaunch& L) {
  int n = 0;
  return dispatch_branch(L, nullptr, &n) == hipSuccess ? n : 0;
}

}  // namespace pdd
