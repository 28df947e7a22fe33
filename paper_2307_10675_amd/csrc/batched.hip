// Launches of the on-chip solver over one plan's increments, and the single
// sigma of its path.
#include "batched_solver.hpp"

namespace ifci {

__global__ void __launch_bounds__(kBatchThreads) batched_kernel(SolveArgs A, int lds_bytes) {
  extern __shared__ __align__(16) char lds[];
  if ((int)blockIdx.x < A.count) solve_dav_k(A, A.order[blockIdx.x], lds, lds_bytes);
}

__global__ void __launch_bounds__(kBatchThreads) batched_lobpcg_kernel(SolveArgs A, int lds_bytes) {
  extern __shared__ __align__(16) char lds[];
  if ((int)blockIdx.x < A.count) solve_lobpcg_k(A, A.order[blockIdx.x], lds, lds_bytes);
}

// Single sigma through the on-chip path (for checking it): full symmetric c
// in, full sigma out, both [n_det] FP64.
template <int K>
__device__ void sigma_one(const IncDev d, const double* __restrict__ ints, const int32_t* __restrict__ tables,
                          const double* __restrict__ c, double* __restrict__ sig, int precision,
                          char* lds, int lds_bytes) {
  Lds L = carve(lds, d, lds_bytes);
  const int n = d.n_str;
  load_tables(d, L, tables);
  for (int64_t i = threadIdx.x; i < d.n_sym; i += blockDim.x) {
    int a, b;
    unpack(i, &a, &b);
    const double v = c[(int64_t)a * n + b];
    L.tv[i] = (a == b) ? v : v * kSqrt2;
  }
  __syncthreads();
  const double* Vm = ints + d.int_off + int_block(d.k).V;
  if (precision == IFCI_MIXED)
    sigma_phase<float, K>(d, L, Vm, 0.0, et_waves_for<float, K>(d, L));
  else
    sigma_phase<double, K>(d, L, Vm, 0.0, et_waves_for<double, K>(d, L));
  for (int64_t i = threadIdx.x; i < d.n_sym; i += blockDim.x) {
    int a, b;
    unpack(i, &a, &b);
    const double v = (a == b) ? L.sp[i] : L.sp[i] * kRSqrt2;
    sig[(int64_t)a * n + b] = v;
    sig[(int64_t)b * n + a] = v;
  }
}

__global__ void __launch_bounds__(kBatchThreads) sigma_one_kernel(const IncDev* __restrict__ incs, int inc,
                                                                  const double* __restrict__ ints,
                                                                  const int32_t* __restrict__ tables,
                                                                  const double* c, double* sig,
                                                                  int precision, int lds_bytes) {
  extern __shared__ __align__(16) char lds[];
  const IncDev d = incs[inc];
  switch (d.k) {
    case 1: sigma_one<1>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 2: sigma_one<2>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 3: sigma_one<3>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 4: sigma_one<4>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 5: sigma_one<5>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 6: sigma_one<6>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 7: sigma_one<7>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    case 8: sigma_one<8>(d, ints, tables, c, sig, precision, lds, lds_bytes); break;
    default: break;
  }
}

// LDS the batched solver needs for an increment: the persistent part, then
// the transient part with the full FP64 vector after it or one FP32 E slice,
// whichever is larger, and the diagonal-pair weights.
static int64_t scratch_bytes(int k, int n_str, int slices) {
  const int64_t v = a16(transient_bytes(n_str)) + c64_bytes(n_str), e = slices * et_slice_bytes(k, n_str, 4);
  const int64_t w8 = wt_bytes(k, 8), w4 = wt_bytes(k, 4);
  return (v > e ? v : e) + (w8 > w4 ? w8 : w4) + 16;
}
int64_t batched_lds_bytes(int k, int n_str, int n_link) {
  return persistent_bytes(k, n_str, n_link) + scratch_bytes(k, n_str, 1);
}
// LDS that gives every wave of the workgroup its FP32 E slice, or the set-up
// of a P-space block its scratch.
int64_t batched_lds_want(int k, int n_str, int n_link) {
  const int64_t ps = a16(transient_bytes(n_str)) + ps_scratch_bytes(kPsMax, k);
  const int64_t sc = scratch_bytes(k, n_str, kBatchThreads / 64);
  return persistent_bytes(k, n_str, n_link) + (sc > ps ? sc : ps);
}

hipError_t launch_batched(const SolveArgs& A, int lds_bytes, hipStream_t st) {
  hipError_t e = allow_max_lds((const void*)batched_kernel);
  if (e == hipSuccess) e = allow_max_lds((const void*)batched_lobpcg_kernel);
  if (e != hipSuccess) return e;
  if (A.max_space == 3)
    hipLaunchKernelGGL(batched_lobpcg_kernel, dim3(A.count), dim3(kBatchThreads), lds_bytes, st, A, lds_bytes);
  else
    hipLaunchKernelGGL(batched_kernel, dim3(A.count), dim3(kBatchThreads), lds_bytes, st, A, lds_bytes);
  return hipGetLastError();
}

hipError_t launch_sigma_one(const IncDev* incs, int inc, const double* ints, const int32_t* tables,
                            const double* c, double* sig, int precision, int lds_bytes, hipStream_t st) {
  const hipError_t e = allow_max_lds((const void*)sigma_one_kernel);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sigma_one_kernel, dim3(1), dim3(kBatchThreads), lds_bytes, st, incs, inc, ints, tables,
                     c, sig, precision, lds_bytes);
  return hipGetLastError();
}

}  // namespace ifci
