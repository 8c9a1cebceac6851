// Reduction, staging and fill kernels shared by all entry points, and the
// dispatch of the walk launch to its instantiation unit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pdd_device.hpp"
#include "pdd_kernels.hpp"

namespace pdd {

// ---------------------------------------------------------------------------
// Statistics of the items of one group (lane l takes entries l, l + 64, ..,
// then the lanes are merged pairwise: a fixed order), in every lane.
__device__ __forceinline__ ItemStat merge_group(const ItemStat* __restrict__ s, int64_t count, int lane) {
  double n = 0.0, m = 0.0, q = 0.0;
  int64_t st = 0, ce = 0, rd = 0;
  for (int64_t i = lane; i < count; i += kWave) {
    const ItemStat v = s[i];
    chan_merge(n, m, q, (double)v.n, v.mean, v.m2);
    st += v.steps;
    ce += v.censored;
    rd += v.redrawn;
  }
  wave_welford(n, m, q);
  ItemStat r;
  r.mean = m;
  r.m2 = q;
  r.n = (int64_t)n;
  r.steps = wave_sum(st);
  r.censored = wave_sum(ce);
  r.redrawn = wave_sum(rd);
  return r;
}

// The groups of a launch with a wavefront per group: the wavefront's first, and
// how many the launch takes at a time (group_blocks).
__device__ __forceinline__ int64_t first_group() {
  return (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
}
__device__ __forceinline__ int64_t groups() { return (int64_t)gridDim.x * (kBlock / kWave); }

// Merge the pieces' statistics into their items', one wavefront per item.
__global__ void k_merge_pieces(const ItemStat* __restrict__ pstat, const MergeJob* __restrict__ jobs, int n_jobs,
                               ItemStat* __restrict__ istat) {
  const int lane = (int)(threadIdx.x & (kWave - 1));
  for (int64_t i = first_group(); i < n_jobs; i += groups()) {
    const MergeJob J = jobs[i];
    const ItemStat r = merge_group(pstat + J.first, J.count, lane);
    if (lane == 0) istat[J.item] = r;
  }
}

// Merge item partials into per-node statistics, one wavefront per node.
__global__ void k_finalize_nodes(const ItemStat* __restrict__ istat, const int64_t* __restrict__ first,
                                 int64_t n_nodes, const CallPtrs* __restrict__ cp, int64_t out_off,
                                 unsigned long long* __restrict__ counters) {
  const int lane = (int)(threadIdx.x & (kWave - 1));
  for (int64_t i = first_group(); i < n_nodes; i += groups()) {
    const int64_t f = first[i];
    const ItemStat v = merge_group(istat + f, first[i + 1] - f, lane);
    if (lane != 0) continue;
    pdd_node_stat_dev r;
    r.mean = v.mean; r.m2 = v.m2; r.n = v.n; r.steps = v.steps; r.censored = v.censored;
    ((pdd_node_stat_dev*)cp->out + out_off)[i] = r;
    if (counters != nullptr) {
      if (v.censored) atomicAdd(&counters[0], (unsigned long long)v.censored);
      if (v.redrawn) atomicAdd(&counters[1], (unsigned long long)v.redrawn);
    }
  }
}

// Adjoint reduction: grad[k] = sum over items s (in slot order) of
// (w[node_s] / N[node_s]) * row_s[k]; one block per column, fixed tree order.
__global__ void k_finalize_grad(const double* __restrict__ igrad, int stride, int n_items,
                                const int32_t* __restrict__ slot_node, const CallPtrs* __restrict__ cp,
                                const double* __restrict__ inv_n, double* __restrict__ colsum) {
  const int col = blockIdx.x;
  const double* __restrict__ w = cp->w;
  __shared__ double part[kBlock];
  double acc = 0.0;
  for (int s = threadIdx.x; s < n_items; s += blockDim.x) {
    const int nd = slot_node[s];
    acc += (w[nd] * inv_n[nd]) * igrad[(size_t)s * stride + col];
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) colsum[col] = part[0];
}

// Per-node Jacobian: jac[i][c] = (1/N_i) * sum over the items of node i (slot
// order) of row_s[colmap[c]].  One block per node.
__global__ void k_node_jacobian(const double* __restrict__ igrad, int stride, const int64_t* __restrict__ first,
                                const double* __restrict__ inv_n, const int32_t* __restrict__ colmap, int n_cols,
                                const CallPtrs* __restrict__ cp, int64_t jac_ld) {
  const int64_t i = blockIdx.x;
  double* __restrict__ jac = cp->jac;
  for (int c = threadIdx.x; c < n_cols; c += blockDim.x) {
    const int src = colmap[c];
    double acc = 0.0;
    for (int64_t s = first[i]; s < first[i + 1]; ++s) acc += igrad[(size_t)s * stride + src];
    jac[(size_t)i * jac_ld + c] = acc * inv_n[i];
  }
}

// dst[map[k]] += src[k] for the gradient columns of one coefficient array
// (dst = the caller's array number `which` of the call block).
__global__ void k_scatter_add(const double* __restrict__ src, const int32_t* __restrict__ map, int count,
                              const CallPtrs* __restrict__ cp, int which) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  double* __restrict__ dst = cp->grad[which];
  if (k < count) dst[map ? map[k] : k] += src[k];
}

// Copy the caller's coefficient arrays into the staged FP64/FP32 tables, and
// clear the queue heads.  blockIdx.x = job, the blocks of one job share its
// entries (one block for all jobs took 25 us for a batch of 8 problems and
// 4096 nodes, a serial chain of small loads; 5 us this way).
__global__ void k_stage(const StageJob* __restrict__ jobs, int n_jobs, const int32_t* __restrict__ perm,
                        double* __restrict__ cd, float* __restrict__ cf, uint32_t* __restrict__ qhead, int n_qhead) {
  const int first = (int)(blockIdx.y * blockDim.x + threadIdx.x), stride = (int)(gridDim.y * blockDim.x);
  if (blockIdx.x == 0)
    for (int k = first; k < n_qhead; k += stride) qhead[k] = 0u;
  if ((int)blockIdx.x >= n_jobs) return;
  const StageJob J = jobs[blockIdx.x];
  if (J.dst != nullptr) {
    for (int k = first; k < J.count; k += stride) J.dst[k] = J.src[k];
    return;
  }
  for (int k = first; k < J.count; k += stride) {
    const int src = J.perm_off >= 0 ? perm[J.perm_off + k] : k;
    const double v = J.src != nullptr ? J.src[src] : 0.0;
    cd[J.dst_off + k] = v;
    cf[J.dst_off + k] = (float)v;
  }
}

// grad[k] = sum_i w_i J[i][k] (with `data`: w_i = 2 (mean_i - data_i), and
// loss = sum_i (mean_i - data_i)^2 into *loss).  A block owns kApplyCols
// columns (a 128-byte segment of every row); its threads take rows r = R t +
// row group, kApplyRows at a time so that as many loads are in flight, each
// summing its column over its rows in row order, and the row groups' partial
// sums are added in order: a fixed order, so the result is bitwise
// reproducible.  Bound by latency: 4096 x 160 takes 19 us (5.2 MB: 280 GB/s),
// with 4 rows in flight per column it took 163, and 510 with the misfit.
constexpr int kApplyBlock = 1024, kApplyCols = 16, kApplyGroups = kApplyBlock / kApplyCols, kApplyRows = 8;
__global__ void __launch_bounds__(kApplyBlock)
k_jacobian_apply(const double* __restrict__ jac, int64_t n_rows, int64_t ld, int64_t n_cols,
                 const double* __restrict__ w, const pdd_node_stat_dev* __restrict__ stats,
                 const double* __restrict__ data, double* __restrict__ grad, double* __restrict__ loss) {
  __shared__ double part[kApplyGroups][kApplyCols];
  __shared__ double lpart[kApplyGroups];
  const int c = (int)(threadIdx.x % kApplyCols), g = (int)(threadIdx.x / kApplyCols);
  const int64_t col = (int64_t)blockIdx.x * kApplyCols + c;
  const bool have = col < n_cols;
  double acc = 0.0, lacc = 0.0;
  for (int64_t r0 = g; r0 < n_rows; r0 += (int64_t)kApplyGroups * kApplyRows) {
    double wi[kApplyRows], v[kApplyRows], e[kApplyRows];
#pragma unroll
    for (int u = 0; u < kApplyRows; ++u) {
      const int64_t r = r0 + (int64_t)u * kApplyGroups;
      const bool in = r < n_rows;
      e[u] = in && data != nullptr ? stats[r].mean - data[r] : 0.0;
      wi[u] = in && data == nullptr ? w[r] : 0.0;
      v[u] = in && have ? jac[(size_t)r * ld + col] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kApplyRows; ++u) {
      if (r0 + (int64_t)u * kApplyGroups >= n_rows) break;
      lacc += e[u] * e[u];
      if (have) acc += (data != nullptr ? 2.0 * e[u] : wi[u]) * v[u];
    }
  }
  part[g][c] = acc;
  if (c == 0) lpart[g] = lacc;
  __syncthreads();
  if (g == 0 && have) {
    double s = part[0][c];
    for (int k = 1; k < kApplyGroups; ++k) s += part[k][c];
    grad[col] = s;
  }
  if (loss != nullptr && blockIdx.x == 0 && threadIdx.x == kWave) {
    double s = lpart[0];
    for (int k = 1; k < kApplyGroups; ++k) s += lpart[k];
    *loss = s;
  }
}

// Merges a second sample of node index[k] into the node's estimate: Chan's
// merge of the Welford triples, sums of the counts, and the Jacobian rows
// weighted by their path counts.  One block per merged node.
__global__ void k_merge_estimates(pdd_node_stat_dev* __restrict__ acc, double* __restrict__ acc_jac,
                                  int64_t acc_ld, const pdd_node_stat_dev* __restrict__ add,
                                  const double* __restrict__ add_jac, int64_t add_ld, int64_t n_params,
                                  const int64_t* __restrict__ index) {
  const int64_t k = blockIdx.x;
  const int64_t i = index[k];
  const pdd_node_stat_dev a = acc[i];
  const pdd_node_stat_dev b = add[k];
  const double na = (double)a.n, nb = (double)b.n;
  const double tot = na + nb;
  if (acc_jac != nullptr && add_jac != nullptr && tot > 0.0) {
    for (int64_t c = threadIdx.x; c < n_params; c += blockDim.x) {
      const double v = (na * acc_jac[(size_t)i * acc_ld + c] + nb * add_jac[(size_t)k * add_ld + c]) / tot;
      acc_jac[(size_t)i * acc_ld + c] = v;
    }
  }
  if (threadIdx.x == 0) {
    double n = na, m = a.mean, q = a.m2;
    chan_merge(n, m, q, nb, b.mean, b.m2);
    pdd_node_stat_dev r;
    r.mean = m; r.m2 = q; r.n = a.n + b.n; r.steps = a.steps + b.steps; r.censored = a.censored + b.censored;
    acc[i] = r;
  }
}

// var_i = m2_i / (n_i - 1) (0 for n_i < 2), se_i = sqrt(var_i / n_i).
__global__ void k_node_moments(const pdd_node_stat_dev* __restrict__ stats, int64_t n, double* __restrict__ var,
                               double* __restrict__ se) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const pdd_node_stat_dev s = stats[i];
  const double v = s.n > 1 ? s.m2 / (double)(s.n - 1) : 0.0;
  if (var != nullptr) var[i] = v;
  if (se != nullptr) se[i] = s.n > 0 ? sqrt(v / (double)s.n) : 0.0;
}

__global__ void k_fill_f64(double* p, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_walk_fwd(const WalkLaunch& L, hipStream_t st);
hipError_t launch_walk_adj_f32(const WalkLaunch& L, hipStream_t st);
hipError_t launch_walk_adj_f64(const WalkLaunch& L, hipStream_t st);

hipError_t launch_walk(const WalkLaunch& L, hipStream_t st) {
  if (!L.adjoint) return launch_walk_fwd(L, st);
  if (L.spec != nullptr) {
    // same argument list as k_walk_adj; the parameter block is passed by value
    const WorkItem* items = L.items;
    int n_items = L.n_items, grad_stride = L.grad_stride, refill = L.refill_groups;
    uint32_t* qhead = L.qhead;
    ItemStat* istat = L.istat;
    double* igrad = L.igrad;
    double* dump_phi = L.dump_phi;
    int64_t* dump_steps = L.dump_steps;
    const int64_t* dump_off = L.dump_off;
    void* args[] = {(void*)L.P, &items, &n_items, &qhead, &istat, &igrad, &grad_stride, &dump_phi, &dump_steps,
                    &dump_off, &refill};
    return hipModuleLaunchKernel(L.spec, (unsigned)L.grid, 1, 1, kBlock, 1, 1, 0, st, args, nullptr);
  }
  return L.fp32 ? launch_walk_adj_f32(L, st) : launch_walk_adj_f64(L, st);
}

hipError_t launch_merge_pieces(const ItemStat* pstat, const MergeJob* jobs, int n_jobs, ItemStat* istat,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_merge_pieces, dim3(group_blocks(n_jobs)), dim3(kBlock), 0, st, pstat, jobs, n_jobs, istat);
  return hipGetLastError();
}

hipError_t launch_finalize_nodes(const ItemStat* istat, const int64_t* first, int64_t n_nodes, const CallPtrs* cp,
                                 int64_t out_off, unsigned long long* counters, hipStream_t st) {
  hipLaunchKernelGGL(k_finalize_nodes, dim3(group_blocks(n_nodes)), dim3(kBlock), 0, st, istat, first, n_nodes, cp,
                     out_off, counters);
  return hipGetLastError();
}

hipError_t launch_finalize_grad(const double* igrad, int stride, int n_cols, int n_items, const int32_t* slot_node,
                                const CallPtrs* cp, const double* inv_n, double* colsum, hipStream_t st) {
  hipLaunchKernelGGL(k_finalize_grad, dim3(n_cols), dim3(kBlock), 0, st, igrad, stride, n_items, slot_node, cp,
                     inv_n, colsum);
  return hipGetLastError();
}

hipError_t launch_node_jacobian(const double* igrad, int stride, const int64_t* first, int64_t n_nodes,
                                const double* inv_n, const int32_t* colmap, int n_cols, const CallPtrs* cp,
                                int64_t jac_ld, hipStream_t st) {
  hipLaunchKernelGGL(k_node_jacobian, dim3((unsigned)n_nodes), dim3(kBlock), 0, st, igrad, stride, first, inv_n, colmap,
                     n_cols, cp, jac_ld);
  return hipGetLastError();
}

hipError_t launch_scatter_add(const double* src, const int32_t* map, int count, const CallPtrs* cp, int which,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_scatter_add, dim3((count + kBlock - 1) / kBlock), dim3(kBlock), 0, st, src, map, count, cp,
                     which);
  return hipGetLastError();
}

hipError_t launch_jacobian_apply(const double* jac, int64_t n_rows, int64_t ld, int64_t n_cols, const double* w,
                                 const void* stats, const double* data, double* grad, double* loss, hipStream_t st) {
  const int64_t blocks = (n_cols + kApplyCols - 1) / kApplyCols;
  hipLaunchKernelGGL(k_jacobian_apply, dim3((unsigned)(blocks > 0 ? blocks : 1)), dim3(kApplyBlock), 0, st, jac, n_rows,
                     ld, n_cols, w, (const pdd_node_stat_dev*)stats, data, grad, loss);
  return hipGetLastError();
}

hipError_t launch_merge_estimates(void* acc, double* acc_jac, int64_t acc_ld, const void* add, const double* add_jac,
                                  int64_t add_ld, int64_t n_params, const int64_t* index, int64_t n_add,
                                  hipStream_t st) {
  hipLaunchKernelGGL(k_merge_estimates, dim3((unsigned)n_add), dim3(kBlock), 0, st, (pdd_node_stat_dev*)acc, acc_jac,
                     acc_ld, (const pdd_node_stat_dev*)add, add_jac, add_ld, n_params, index);
  return hipGetLastError();
}

hipError_t launch_node_moments(const void* stats, int64_t n, double* var, double* se, hipStream_t st) {
  const int64_t blocks = (n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_node_moments, dim3((unsigned)(blocks > 0 ? blocks : 1)), dim3(kBlock), 0, st,
                     (const pdd_node_stat_dev*)stats, n, var, se);
  return hipGetLastError();
}

hipError_t launch_stage(const StageJob* jobs, int n_jobs, int max_count, const int32_t* perm, double* cd, float* cf,
                        uint32_t* qhead, int n_qhead, hipStream_t st) {
  const int share = std::max(1, std::min(16, (max_count + 1023) / 1024));
  hipLaunchKernelGGL(k_stage, dim3(std::max(1, n_jobs), share), dim3(kBlock), 0, st, jobs, n_jobs, perm, cd, cf, qhead,
                     n_qhead);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t st) {
  const int64_t blocks = (n + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)(blocks > 0 ? blocks : 1)), dim3(kBlock), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace pdd
