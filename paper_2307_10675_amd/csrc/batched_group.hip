// One launch of the on-chip solver over the increments of several plans.
//
// A plan of one small increment fills one of 256 CUs, and a launch per plan
// runs them one after the other; here the work list holds (plan, increment)
// pairs over all plans, heaviest first, and each workgroup reads its plan's
// arguments from memory.  7 independent 6o6e problems: 7 launches of 1.2 ms
// against one.
#include <cstring>

#include "batched_solver.hpp"

namespace ifci {

// 1.75 KB of the work list of a captured call per launch, as kernel arguments.
// (A call that is not captured uploads its list where it differs from the last
// one: a launch of this kernel takes 7 us, 64 plans 55 us more in 930.)
struct StoreWords {
  static constexpr int kWords = 448;
  uint32_t w[kWords];
};

__global__ void __launch_bounds__(StoreWords::kWords) store_kernel(uint32_t* __restrict__ dst, int n, StoreWords s) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = s.w[threadIdx.x];
}

hipError_t launch_store(void* dst, const void* src, int64_t bytes, hipStream_t st) {
  static_assert(sizeof(SolveArgs) % 4 == 0 && std::is_trivially_copyable<SolveArgs>::value, "stored by words");
  constexpr int64_t kBytes = 4 * StoreWords::kWords;
  StoreWords s;
  for (int64_t at = 0; at < bytes; at += kBytes) {
    const int64_t nb = bytes - at < kBytes ? bytes - at : kBytes;
    std::memcpy(s.w, (const char*)src + at, nb);
    hipLaunchKernelGGL(store_kernel, dim3(1), dim3(StoreWords::kWords), 0, st, (uint32_t*)((char*)dst + at),
                       (int)(nb / 4), s);
  }
  return hipGetLastError();
}

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
