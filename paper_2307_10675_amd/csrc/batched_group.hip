// One launch of the on-chip solver over the increments of several plans.
//
// A plan of one small increment fills one of 256 CUs, and a launch per plan
// runs them one after the other; here the work list holds (plan, increment)
// pairs over all plans, heaviest first, and each workgroup reads its plan's
// arguments from memory.  7 independent 6o6e problems: 7 launches of 1.2 ms
// against one.
#include "batched_solver.hpp"

namespace ifci {

__global__ void __launch_bounds__(kBatchThreads)
    batched_group_kernel(const SolveArgs* __restrict__ jobs, const int2* __restrict__ work, int lds_bytes) {
  extern __shared__ __align__(16) char lds[];
  const int job = __builtin_amdgcn_readfirstlane(work[blockIdx.x].x);
  solve_dav_k(jobs[job], __builtin_amdgcn_readfirstlane(work[blockIdx.x].y), lds, lds_bytes);
}

__global__ void __launch_bounds__(kBatchThreads)
    batched_lobpcg_group_kernel(const SolveArgs* __restrict__ jobs, const int2* __restrict__ work, int lds_bytes) {
  extern __shared__ __align__(16) char lds[];
  const int job = __builtin_amdgcn_readfirstlane(work[blockIdx.x].x);
  solve_lobpcg_k(jobs[job], __builtin_amdgcn_readfirstlane(work[blockIdx.x].y), lds, lds_bytes);
}

hipError_t launch_batched_group(const SolveArgs* jobs, const int2* work, int count, int max_space, int lds_bytes,
                                hipStream_t st) {
  const void* fn = max_space == 3 ? (const void*)batched_lobpcg_group_kernel : (const void*)batched_group_kernel;
  const hipError_t e = allow_max_lds(fn);
  if (e != hipSuccess) return e;
  if (max_space == 3)
    hipLaunchKernelGGL(batched_lobpcg_group_kernel, dim3(count), dim3(kBatchThreads), lds_bytes, st, jobs, work,
                       lds_bytes);
  else
    hipLaunchKernelGGL(batched_group_kernel, dim3(count), dim3(kBatchThreads), lds_bytes, st, jobs, work, lds_bytes);
  return hipGetLastError();
}

}  // namespace ifci
