// Heterogeneous batch of linear problems in one persistent launch (the loops
// over interface nodes and their samples of Algorithm 3.1, across subdomains
// whose domains and data differ, as in a PDD partition): the items of every
// problem form a queue of their own, large ones first and longest first
// within a size class, and the wavefronts of one grid stream through the
// queues (stream_walk), so problems of different dimension and cost share
// the chip.
//
// The walk is k_walk_fwd's (Euler-Maruyama with the exit test, or walk on
// spheres; FP32 or FP64 stepping, FP64 sums) with the same arithmetic in the
// same order, so a path's value equals the single-problem kernel's and the
// oracle's on the same counters.  b, c, f are dense polynomials (of degree
// <= 3) here, g may have generic terms.
#include <hip/hip_runtime.h>

#include "pdd_device.hpp"
#include "pdd_kernels.hpp"
#include "walk_kernels.hpp"
#include "walk_stream.hpp"

namespace pdd {

template <typename R>
__device__ __forceinline__ Dom<R> batch_dom(const LinearParams PDD_CONST_AS* P, bool test);
template <>
__device__ __forceinline__ Dom<float> batch_dom<float>(const LinearParams PDD_CONST_AS* P, bool test) {
  Dom<float> D;
  D.kind = P->dom_kind;
  for (int k = 0; k < 3; ++k) {
    D.lo[k] = test ? P->tlof[k] : P->lof[k];
    D.hi[k] = test ? P->thif[k] : P->hif[k];
    D.ctr[k] = P->ctrf[k];
  }
  D.rad = P->radf;
  D.rad2 = test ? P->trad2f : P->rad2f;
  return D;
}
template <>
__device__ __forceinline__ Dom<double> batch_dom<double>(const LinearParams PDD_CONST_AS* P, bool test) {
  Dom<double> D;
  D.kind = P->dom_kind;
  for (int k = 0; k < 3; ++k) {
    D.lo[k] = test ? P->tlo[k] : P->lo[k];
    D.hi[k] = test ? P->thi[k] : P->hi[k];
    D.ctr[k] = P->ctr[k];
  }
  D.rad = P->rad;
  D.rad2 = test ? P->trad2 : P->rad2;
  return D;
}

template <typename R>
__device__ __forceinline__ R batch_dt(const LinearParams PDD_CONST_AS* P) {
  if constexpr (sizeof(R) == 4) return P->dtf; else return P->dt;
}
template <typename R>
__device__ __forceinline__ R batch_sdt(const LinearParams PDD_CONST_AS* P) {
  if constexpr (sizeof(R) == 4) return P->sdtf; else return P->sdt;
}

// The staged coefficient table as scalar loads (float or double copy).
template <typename R>
__device__ __forceinline__ const R PDD_CONST_AS* batch_coefs(const double* cd, const float* cf) {
  if constexpr (sizeof(R) == 4) return (const R PDD_CONST_AS*)const_table(cf);
  else return (const R PDD_CONST_AS*)const_table(cd);
}

// One problem of the batch as stream_walk's PROB: its record is read through
// scalar loads.  BCF = false is the instance for problems with b = c = f = 0
// (pure diffusion): the step has no drift, killing or source code and no
// per-step tests of the problem's flags.
template <typename R, int DIM, bool WOS, int KIND, bool BCF>
struct BatchProblem {
  static constexpr bool kWos = WOS, kFree = !BCF && !WOS, kYZ = BCF, kRoll = BCF && sizeof(R) == 8;
  static constexpr int NM = GradedLex<DIM, kMaxPolyBCF>::N;
  typedef ExitExtremes<R, DIM, KIND> Extremes;

  const LinearParams PDD_CONST_AS* P;
  const double* nodes;
  const DevFactor* fac;
  const double* cd;
  const float* cf;
  const Dom<R> D;
  const ExitTest<R, DIM, KIND> test;
  R dt, sdt;
  const uint32_t max_steps;
  const bool has_b, has_c, has_f;

  __device__ __forceinline__ BatchProblem(const LinearParams PDD_CONST_AS* p, const double* nd, const DevFactor* fa,
                                          const double* c64, const float* c32)
      : P(p), nodes(nd), fac(fa), cd(c64), cf(c32), D(batch_dom<R>(p, false)), test(batch_dom<R>(p, true)),
        dt(batch_dt<R>(p)), sdt(batch_sdt<R>(p)), max_steps((uint32_t)p->max_steps), has_b(BCF && p->has_b != 0),
        has_c(BCF && p->has_c != 0), has_f(BCF && p->has_f != 0) {
    if constexpr (sizeof(R) == 4) asm volatile("" : "+v"(dt), "+v"(sdt));
  }
  __device__ __forceinline__ void start(int node, R* x) const {
#pragma unroll
    for (int k = 0; k < DIM; ++k) x[k] = to_r<R>(nodes[(size_t)node * 3 + k]);
  }
  __device__ __forceinline__ bool inside(const R* x) const { return test.inside(x); }
  __device__ __forceinline__ R distance(const R* x) const {
    Dom<R> d = D;
    d.kind = KIND;
    return boundary_distance<R, DIM>(d, x);
  }
  __device__ __forceinline__ R g(const R* x) const {
    DevFun g;
    g.n_terms = P->g.n_terms;
    g.n_factors = P->g.n_factors;
    g.fac_off = P->g.fac_off;
    g.coef_off = P->g.coef_off;
    g.poly_deg = P->g.poly_deg;
    g.n_mono = P->g.n_mono;
    g.poly_off = P->g.poly_off;
    g.pad = 0;
    R v = (R)0;
    if (g.n_terms > 0) v = terms_sum<R, DIM>(fac, cd, cf, g, x);
    if (g.poly_deg >= 0) v += poly_rows<R, DIM>(cd, cf, g.poly_deg, g.poly_off, x);
    return v;
  }
  __device__ __forceinline__ void step(R* X, R& Y, R& Z, const R* z) const {
    R mono[NM];
    if (has_b || has_c || has_f) monomials<R, DIM, kMaxPolyBCF>(X, mono);
    const R PDD_CONST_AS* ct = batch_coefs<R>(cd, cf);
    if (has_f) Z = Z + poly_dot<R, NM>(ct + P->f.poly_off, mono) * Y * dt;
    if (has_c) Y = Y * fexp(-poly_dot<R, NM>(ct + P->c.poly_off, mono) * dt);
    if (has_b) {
      R bv[DIM];
#pragma unroll
      for (int k = 0; k < DIM; ++k)
        bv[k] = P->b[k].poly_deg >= 0 ? poly_dot<R, NM>(ct + P->b[k].poly_off, mono) : (R)0;
#pragma unroll
      for (int k = 0; k < DIM; ++k) X[k] = X[k] + bv[k] * dt + sdt * z[k];
    } else {
#pragma unroll
      for (int k = 0; k < DIM; ++k) X[k] = X[k] + sdt * z[k];
    }
  }
};

// A wavefront streams through the queue of one problem (whose dimension and
// domain kind its code is instantiated for), then goes on to the next
// problem's queue.  The wavefronts start spread over the problems by their
// share of the estimated work (BatchQueue::first_wave: the first wavefront of
// every problem), so the queues run out together and few wavefronts drain twice.
// FP32: built for six waves per SIMD (at most 80 VGPRs), so the default six
// blocks per CU are all resident.
template <typename R, int LAYOUT, bool WOS>
__global__ void __launch_bounds__(kBlock, (sizeof(R) == 4 ? 6 : 1))
k_walk_batch(const LinearParams* __restrict__ probs, int n_probs, const BatchQueue* __restrict__ queues,
             const double* __restrict__ nodes, const DevFactor* __restrict__ fac, const double* __restrict__ cd,
             const float* __restrict__ cf, const StreamArgs A) {
  constexpr int kWaves = kBlock / kWave;
  using Lds = StreamLds<R, stream_area_bytes<R, 3, LAYOUT, !WOS, !WOS && sizeof(R) == 8>()>;
  __shared__ Lds lds[kWaves];
  const int lane = (int)(threadIdx.x & (kWave - 1));
  const int wid = (int)(threadIdx.x / kWave);
  const uint32_t wave = blockIdx.x * kWaves + (uint32_t)__builtin_amdgcn_readfirstlane(wid);
  const BatchQueue PDD_CONST_AS* Q = const_table(queues);
  const uint32_t n_waves = gridDim.x * kWaves;
  int k = 0;
  while (k + 1 < n_probs && wave >= Q[k + 1].first_wave) ++k;
  for (int t = 0; t < n_probs; ++t, k = k + 1 == n_probs ? 0 : k + 1) {
    StreamArgs B = A;
    B.items = A.items + Q[k].first;
    B.n_items = Q[k].count;
    B.qhead = A.qhead + (size_t)k * kQueueStride;
    if (B.n_items == 0) continue;
    const uint32_t w0 = Q[k].first_wave, n_first = (k + 1 < n_probs ? Q[k + 1].first_wave : n_waves) - w0;
    const uint32_t first = t == 0 ? wave - w0 : n_first;
    const LinearParams PDD_CONST_AS* P = const_table(probs) + k;
    const bool box = P->dom_kind == DOM_BOX;
    // walk on spheres requires b = c = f = 0
    const bool bcf = !WOS && (P->has_b != 0 || P->has_c != 0 || P->has_f != 0);
#define PDD_BATCH_B(DIM, KIND, BCF) \
  stream_walk<R, DIM, LAYOUT>(BatchProblem<R, DIM, WOS, KIND, BCF>(P, nodes, fac, cd, cf), B, &lds[wid], lane, \
                              first, n_first)
#define PDD_BATCH(DIM)                                    \
  do {                                                    \
    if constexpr (!WOS) {                                 \
      if (bcf) {                                          \
        PDD_BATCH_B(DIM, kAnyKind, true);                 \
        break;                                            \
      }                                                   \
    }                                                     \
    if (box) PDD_BATCH_B(DIM, DOM_BOX, false);            \
    else PDD_BATCH_B(DIM, DOM_BALL, false);               \
  } while (0)
    switch (P->dim) {
      case 1: PDD_BATCH(1); break;
      case 2: PDD_BATCH(2); break;
      default: PDD_BATCH(3); break;
    }
#undef PDD_BATCH
#undef PDD_BATCH_B
  }
}

template <typename R, int LAYOUT, bool WOS>
static hipError_t launch_batch_t(const WalkBatchLaunch& L, hipStream_t st) {
  const StreamArgs A{L.items, L.n_items, L.qhead, L.istat, L.dump_phi, L.dump_steps, L.dump_off, L.key0, L.key1,
                     L.refill_groups};
  hipLaunchKernelGGL((k_walk_batch<R, LAYOUT, WOS>), dim3(L.grid), dim3(kBlock), 0, st, L.probs, L.n_probs, L.queues,
                     L.nodes, L.fac, L.cd, L.cf, A);
  return hipGetLastError();
}

template <typename R, int LAYOUT, bool WOS>
static int batch_blocks_t() {
  int n = 0;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_walk_batch<R, LAYOUT, WOS>, kBlock, 0) == hipSuccess ? n : 0;
}

int walk_batch_blocks(bool fp32, int layout, bool wos) {
  if (fp32) return wos ? batch_blocks_t<float, RNG_QUAD24, true>() : batch_blocks_t<float, RNG_QUAD24, false>();
  if (layout == RNG_QUAD24)
    return wos ? batch_blocks_t<double, RNG_QUAD24, true>() : batch_blocks_t<double, RNG_QUAD24, false>();
  return wos ? batch_blocks_t<double, RNG_PAIR52, true>() : batch_blocks_t<double, RNG_PAIR52, false>();
}

hipError_t launch_walk_batch(const WalkBatchLaunch& L, hipStream_t st) {
  if (L.fp32) return L.wos ? launch_batch_t<float, RNG_QUAD24, true>(L, st) : launch_batch_t<float, RNG_QUAD24, false>(L, st);
  if (L.layout == RNG_QUAD24)
    return L.wos ? launch_batch_t<double, RNG_QUAD24, true>(L, st) : launch_batch_t<double, RNG_QUAD24, false>(L, st);
  return L.wos ? launch_batch_t<double, RNG_PAIR52, true>(L, st) : launch_batch_t<double, RNG_PAIR52, false>(L, st);
}

}  // namespace pdd
