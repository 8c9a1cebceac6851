// Forward (value-only) instantiations of the walk kernels and the plain FP64 baseline.
#include <hip/hip_runtime.h>

#include "walk_kernels.hpp"
#include "walk_stream.hpp"

namespace pdd {

// Launches the instantiation, or (blocks != nullptr) says how many of its
// blocks a compute unit holds.
template <typename R, int DIM, int DFC, int LAYOUT, bool TERMS, bool WOS = false>
static hipError_t launch_fwd_t(const WalkLaunch& L, const StreamArgs& A, hipStream_t st, int* blocks) {
  if (blocks != nullptr)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_walk_fwd<R, DIM, DFC, LAYOUT, TERMS, WOS>, kBlock, 0);
  hipLaunchKernelGGL((k_walk_fwd<R, DIM, DFC, LAYOUT, TERMS, WOS>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, A);
  return hipGetLastError();
}

template <typename R, int DIM, int LAYOUT>
static hipError_t launch_fwd_dim(const WalkLaunch& L, const StreamArgs& A, hipStream_t st, int* blocks) {
  // walk on spheres (Laplace's equation; b = c = f = 0)
  if (L.wos) return launch_fwd_t<R, DIM, -1, LAYOUT, false, true>(L, A, st, blocks);
  if (L.dfc >= 0)
    return L.terms ? launch_fwd_t<R, DIM, 3, LAYOUT, true>(L, A, st, blocks) : launch_fwd_t<R, DIM, 3, LAYOUT, false>(L, A, st, blocks);
  return L.terms ? launch_fwd_t<R, DIM, -1, LAYOUT, true>(L, A, st, blocks) : launch_fwd_t<R, DIM, -1, LAYOUT, false>(L, A, st, blocks);
}

template <typename R, int LAYOUT>
static hipError_t launch_fwd_r(const WalkLaunch& L, const StreamArgs& A, hipStream_t st, int* blocks) {
  switch (L.P->dim) {
    case 1: return launch_fwd_dim<R, 1, LAYOUT>(L, A, st, blocks);
    case 2: return launch_fwd_dim<R, 2, LAYOUT>(L, A, st, blocks);
    default: return launch_fwd_dim<R, 3, LAYOUT>(L, A, st, blocks);
  }
}

static hipError_t dispatch_fwd(const WalkLaunch& L, hipStream_t st, int* blocks) {
  StreamArgs A{L.items, L.n_items, L.qhead, L.istat, L.dump_phi, L.dump_steps, L.dump_off, L.P->key0, L.P->key1,
               L.refill_groups};
  if (L.spec != nullptr) {
    // the same kernel compiled for the problem's terms; the parameter block
    // is passed by value
    if (blocks != nullptr) return hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(blocks, L.spec, kBlock, 0);
    void* args[] = {(void*)L.P, &A};
    return hipModuleLaunchKernel(L.spec, (unsigned)L.grid, 1, 1, kBlock, 1, 1, 0, st, args, nullptr);
  }
  if (L.fp32) return launch_fwd_r<float, RNG_QUAD24>(L, A, st, blocks);
  if (L.P->layout == RNG_QUAD24) return launch_fwd_r<double, RNG_QUAD24>(L, A, st, blocks);
  return launch_fwd_r<double, RNG_PAIR52>(L, A, st, blocks);
}

hipError_t launch_walk_fwd(const WalkLaunch& L, hipStream_t st) { return dispatch_fwd(L, st, nullptr); }

int walk_fwd_blocks(const WalkLaunch& L) {
  int n = 0;
  return dispatch_fwd(L, nullptr, &n) == hipSuccess ? n : 0;
}

template <int DIM, int DFC, int LAYOUT>
static hipError_t launch_plain_t(const PlainLaunch& L, hipStream_t st) {
  hipLaunchKernelGGL((k_walk_plain<DIM, DFC, LAYOUT>), dim3(L.grid), dim3(kBlock), 0, st, *L.P, L.node, L.n_paths,
                     L.bstat, L.dump_phi, L.dump_steps, L.dump_base);
  return hipGetLastError();
}

template <int LAYOUT>
static hipError_t launch_plain_l(const PlainLaunch& L, hipStream_t st) {
  const bool poly = L.dfc >= 0;
  switch (L.P->dim) {
    case 1: return poly ? launch_plain_t<1, 3, LAYOUT>(L, st) : launch_plain_t<1, -1, LAYOUT>(L, st);
    case 2: return poly ? launch_plain_t<2, 3, LAYOUT>(L, st) : launch_plain_t<2, -1, LAYOUT>(L, st);
    default: return poly ? launch_plain_t<3, 3, LAYOUT>(L, st) : launch_plain_t<3, -1, LAYOUT>(L, st);
  }
}

hipError_t launch_plain(const PlainLaunch& L, hipStream_t st) {
  return L.P->layout == RNG_QUAD24 ? launch_plain_l<RNG_QUAD24>(L, st) : launch_plain_l<RNG_PAIR52>(L, st);
}

}  // namespace pdd
