// Device-wide sigma and a host-driven Davidson for one increment of any
// supported size (up to 16 active orbitals): sigma of arbitrary
// (non-symmetric) vectors, the symmetric-sector sigma of one increment, and
// the unfused per-increment path (one launch per step, the host reading the
// solver state every iteration) that the batched solvers are compared with.
// The kernel bodies live in sigma_wide.hpp and davidson_ops.hpp.
#include <algorithm>
#include <map>
#include <mutex>
#include <set>
#include <utility>

#include "davidson_ops.hpp"
#include "device_common.hpp"
#include "sigma_wide.hpp"
#include "launch.hpp"

namespace ifci {

__global__ void __launch_bounds__(256) sym_combine_kernel(IncDev d, const double* __restrict__ Sm,
                                                          double* __restrict__ sig) {
  __shared__ double tl[32][33];
  sym_combine_body(d.n_str, Sm, blockIdx.x, gridDim.x, tl, [&](int64_t i, double v) { sig[i] = v; });
}

// Shapes of the column kernels: 9 to 14 orbitals at any filling (LDS holds
// the fragments, a column and its accumulator), 16 at half filling.
bool sigma_column_supported(const IncDev& d) {
  return (d.k >= 9 && d.k <= 14) || (d.k == 16 && d.na * 2 == d.k);
}
// Shapes whose symmetric-sector product is an entry of its own.
bool sigma_sector_shape(const IncDev& d) {
  return d.na * 2 == d.k && (d.k == 10 || d.k == 12 || d.k == 14 || d.k == 16);
}

// Workspace doubles of the column path (full C of either precision, S, the
// fragment image, with 256-byte alignment of each); `parts` matrices and S.
static int64_t up32(int64_t x) { return (x + 31) / 32 * 32; }
static int64_t sigma_column_ws_doubles(const IncDev& d, int parts) {
  const int64_t n = d.n_str;
  const int64_t np = (int64_t)d.k * (d.k + 1) / 2, mt = (np + 15) / 16, ks = (np + 3) / 4;
  return parts * (up32((n + 1) * n + 16) + up32(n * n)) + up32(mt * (ks + 1) * 64) + 64;
}

// 16 orbitals have the column form for symmetric vectors only, and no room for
// E at half filling.
bool sigma_general_supported(const IncDev& d) { return !sigma_column_supported(d) || d.k <= 14; }
int64_t sigma_ws_doubles(const IncDev& d) {
  if (sigma_column_supported(d)) return sigma_column_ws_doubles(d, sigma_general_supported(d) ? 2 : 1);
  return (int64_t)d.npair * d.n_det;
}

// mode 0: c and sig full vectors, any c; mode 1: packed scaled symmetric ones.
template <typename T, int K>
static hipError_t launch_column_k(const IncDev& d, const double* V, const int32_t* ptab, const int16_t* ptabT,
                                  const double* c, double* sig, double* ws, int mode, double shift, hipStream_t st) {
  typedef ColShape<T, K> SH;
  static_assert(SH::lds <= kMaxLds, "column sigma LDS");
  const hipError_t e = allow_max_lds((const void*)sigma_column_kernel<T, K>);
  if (e != hipSuccess) return e;
  const int n = d.n_str, parts = mode == 0 ? 2 : 1;
  // workspace (256-byte aligned): full C (and its transpose), then S, then the
  // fragment image, each starting on a 256-byte boundary
  T* cf = (T*)ws;
  const int64_t cf_doubles = up32(((int64_t)(n + 1) * n + 16) * (int64_t)sizeof(T) / 8 + 1);
  const int64_t cf_step = cf_doubles * 8 / (int64_t)sizeof(T);
  double* Sm = ws + parts * cf_doubles;
  T* vfg = (T*)(ws + up32(parts * (cf_doubles + (int64_t)n * n)));
  const int nfrag = (int)(SH::vf_bytes / sizeof(T));
  hipLaunchKernelGGL((col_frag_kernel<T, K>), dim3((nfrag + 255) / 256), dim3(256), 0, st, V, shift, 2.0 * d.na,
                     vfg);
  const unsigned tiles = (unsigned)std::min<int64_t>(4096, (int64_t)((n + 31) / 32) * ((n + 31) / 32) + 1);
  if (mode == 0)
    hipLaunchKernelGGL((column_both_kernel<T>), dim3(tiles), dim3(256), 0, st, n, c, cf, cf_step);
  else
    hipLaunchKernelGGL((expand_sym_kernel<T>), dim3(std::min(2048u, tiles)), dim3(256), 0, st, d, c, cf);
  hipLaunchKernelGGL((sigma_column_kernel<T, K>), dim3(parts * n), dim3(col_threads<T>()), (unsigned)SH::lds, st, n,
                     ptab, ptabT, (const T*)cf, cf_step, (const T*)vfg, Sm, mode == 0 || column_ordered(d));
  if (mode == 0)
    hipLaunchKernelGGL(column_sum_kernel, dim3(tiles), dim3(256), 0, st, n, Sm, sig);
  else
    hipLaunchKernelGGL(sym_combine_kernel, dim3(tiles), dim3(256), 0, st, d, Sm, sig);
  return hipGetLastError();
}

template <typename T, int K>
static hipError_t launch_column_split(const IncDev& d, const double* V, const int32_t* ptab, const int16_t* ptabT,
                                      const double* c, double* sig, double* ws, double shift, hipStream_t st) {
  typedef ColSplit<T, K> SH;
  const hipError_t le = allow_max_lds((const void*)sigma_column_split_kernel<T, K>);
  if (le != hipSuccess) return le;
  const int n = d.n_str;
  auto up = [](int64_t x) { return (x + 31) / 32 * 32; };
  T* cf = (T*)ws;
  const int64_t cf_elems = (int64_t)(n + 1) * n + 16;
  const int64_t off_s = up((cf_elems * (int64_t)sizeof(T) + 7) / 8);
  double* Sm = ws + off_s;
  T* vfg = (T*)(ws + up(off_s + (int64_t)n * n));
  const int nfrag = (int)((int64_t)SH::MT * SH::KSP * 64);
  hipLaunchKernelGGL((col_frag_kernel<T, K>), dim3((nfrag + 255) / 256), dim3(256), 0, st, V, shift, 2.0 * d.na,
                     vfg);
  hipLaunchKernelGGL((expand_sym_kernel<T>), dim3(4096), dim3(256), 0, st, d, c, cf);
  hipLaunchKernelGGL((sigma_column_split_kernel<T, K>), dim3(n), dim3(split_threads<T>()), (unsigned)SH::lds, st, d,
                     ptab, ptabT, (const T*)cf, (const T*)vfg, Sm);
  hipLaunchKernelGGL(sym_combine_kernel, dim3(4096), dim3(256), 0, st, d, Sm, sig);
  return hipGetLastError();
}

hipError_t allow_max_lds(const void* fn) {
  static std::mutex mu;
  static std::set<std::pair<const void*, int>> done;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  if (done.count({fn, dev})) return hipSuccess;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
  if (e == hipSuccess) done.insert({fn, dev});
  return e;
}

static hipError_t launch_sigma_column(const IncDev& d, const double* V, const int32_t* ptab, const int16_t* ptabT,
                                      const double* c, double* sig, double* ws, int precision, int mode, double shift,
                                      hipStream_t st) {
  const bool f32 = precision == IFCI_MIXED;
  switch (d.k) {
#define IFCI_COL(K)                                                                               \
  case K: return f32 ? launch_column_k<float, K>(d, V, ptab, ptabT, c, sig, ws, mode, shift, st)  \
                     : launch_column_k<double, K>(d, V, ptab, ptabT, c, sig, ws, mode, shift, st);
    IFCI_COL(9) IFCI_COL(10) IFCI_COL(11) IFCI_COL(12) IFCI_COL(13) IFCI_COL(14)
#undef IFCI_COL
    case 16:
      if (mode == 0) return hipErrorInvalidValue;
      return f32 ? launch_column_split<float, 16>(d, V, ptab, ptabT, c, sig, ws, shift, st)
                 : launch_column_split<double, 16>(d, V, ptab, ptabT, c, sig, ws, shift, st);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------- static scratch
// E of the general product for callers that cannot allocate
// (ifci_sigma_noalloc): a fixed array of kStaticScratchDoubles doubles on
// every device the library runs on, held until the process ends.  Host code
// never uses the array's name as an address: it uses the device address
// hipGetSymbolAddress gives for the current device, looked up once per
// device.  Every call on a device shares that device's array.
static __device__ __align__(256) double scratch[kStaticScratchDoubles];

hipError_t static_scratch(double** out) {
  static std::mutex mu;
  static std::map<int, double*> addr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    double* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    it = addr.emplace(dev, p).first;
  }
  if (out) *out = it->second;
  return hipSuccess;
}

hipError_t launch_sigma_wide(const IncDev& d, const IncDev*, int, const double* ints, const int32_t* tables,
                             const double* c, double* sig, double* E, int precision, int mode, double shift,
                             hipStream_t st) {
  const double* V = ints + d.int_off + int_block(d.k).V;
  const int32_t* ptab = tables + d.pair_off;
  const int32_t* links = tables + d.link_off;
  if (sigma_column_supported(d) && (mode == 1 || sigma_general_supported(d)))
    return launch_sigma_column(d, V, ptab, (const int16_t*)(tables + d.pairT_off), c, sig, E, precision, mode, shift,
                               st);
  const int64_t tiles = (d.n_det + 63) / 64;
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 g1((unsigned)tiles), blk(kWideThreads);
  const int64_t nout = mode == 0 ? d.n_det : d.n_sym;
  const dim3 g2((unsigned)((nout + kWideThreads - 1) / kWideThreads));
  if (precision == IFCI_MIXED) {
    float* Ef = (float*)E;
    if (mode == 0) {
      hipLaunchKernelGGL((contract_kernel<float, 0>), g1, blk, 0, st, d, V, ptab, c, Ef, shift);
      hipLaunchKernelGGL((gather_full_kernel<float>), g2, blk, 0, st, d, links, Ef, sig);
    } else {
      hipLaunchKernelGGL((contract_kernel<float, 1>), g1, blk, 0, st, d, V, ptab, c, Ef, shift);
      hipLaunchKernelGGL((gather_sym_kernel<float>), g2, blk, 0, st, d, links, Ef, sig);
    }
  } else {
    if (mode == 0) {
      hipLaunchKernelGGL((contract_kernel<double, 0>), g1, blk, 0, st, d, V, ptab, c, E, shift);
      hipLaunchKernelGGL((gather_full_kernel<double>), g2, blk, 0, st, d, links, E, sig);
    } else {
      hipLaunchKernelGGL((contract_kernel<double, 1>), g1, blk, 0, st, d, V, ptab, c, E, shift);
      hipLaunchKernelGGL((gather_sym_kernel<double>), g2, blk, 0, st, d, links, E, sig);
    }
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ Davidson
// The per-increment loop: the steps of davidson_ops.hpp, one launch each,
// with the host reading the state after the residual test.

__global__ void string_energy_kernel(IncDev d, const int32_t* __restrict__ strs, const double* __restrict__ B,
                                     double* __restrict__ F) {
  string_energy_body(d, strs, B, F, blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ void __launch_bounds__(256) hdiag_kernel(IncDev d, const int32_t* __restrict__ strs,
                                                    const double* __restrict__ B, const double* __restrict__ F,
                                                    double* __restrict__ HD, double* part) {
  hdiag_body(d, strs, B, F, HD, nullptr, part + 2 * blockIdx.x, blockIdx.x, gridDim.x);
}

__global__ void init_state_kernel(DavState* S, const double* part, int nblk, double* V0, int64_t ns,
                                  double ecore, int phase) {
  __shared__ int64_t g;
  __shared__ double e0;
  if (threadIdx.x == 0) {
    double b = part[0];
    double ix = part[1];
    for (int i = 1; i < nblk; ++i)
      if (part[2 * i] < b || (part[2 * i] == b && part[2 * i + 1] < ix)) b = part[2 * i], ix = part[2 * i + 1];
    g = (int64_t)ix;
    e0 = b;
    S->E0 = b;
    S->guess = (int)ix;
    S->m = 0;
    S->phase = phase;
    S->iters = 0;
    S->status = IFCI_INC_NOT_CONVERGED;
    S->action = 0;
    S->ecore = ecore;
    S->keep = 0;
    S->plarge = 0;
    S->fresh = 1;
    S->count = 0;
    S->exhausted = 0;
    S->theta = 0.0;
    S->resid = 1e300;
  }
  for (int i = threadIdx.x; i < 256; i += blockDim.x) S->G[i] = 0.0;
  __syncthreads();
  for (int64_t i = threadIdx.x; i < ns; i += blockDim.x) V0[i] = (i == g) ? 1.0 : 0.0;
  (void)e0;
}

__global__ void __launch_bounds__(256) dots_kernel(const double* __restrict__ Vb, int64_t st, int m,
                                                   const double* __restrict__ s, int64_t ns, double* part) {
  __shared__ double red[4 * kNV];
  op_dots(Vb, st, m, s, ns, part + blockIdx.x * kNV, blockIdx.x, gridDim.x, red);
}

__global__ void __launch_bounds__(256) small_G_kernel(DavState* S, const double* part, int nblk, int mmax) {
  __shared__ SmallG sh;
  __shared__ double red[4 * kNV];
  small_G(S, part, nblk, mmax, &sh, red);
}

__global__ void __launch_bounds__(256) passA_kernel(const DavState* __restrict__ S, double* Vb, double* Sb,
                                                    int64_t st, const double* __restrict__ HD,
                                                    double* __restrict__ X, double* __restrict__ T,
                                                    int64_t ns, double* part) {
  __shared__ double red[4 * kNV];
  __shared__ double y[16];
  op_passA(S, Vb, Sb, st, HD, X, T, ns, part + blockIdx.x * kNV, blockIdx.x, gridDim.x, red, y);
}

__global__ void __launch_bounds__(256) small_A_kernel(DavState* S, const double* part, int nblk, double tol32,
                                                      double tol64, int max_iter, int evict) {
  __shared__ double v[kNV], red[4 * kNV];
  small_A(S, part, nblk, tol32, tol64, max_iter, evict, v, red);
}

__global__ void __launch_bounds__(256) switch_kernel(double* Vb, const double* X, int64_t ns) {
  op_switch(Vb, X, ns, blockIdx.x, gridDim.x);
}

__global__ void __launch_bounds__(256) small_switch_kernel(DavState* S) { small_switch(S); }

__global__ void __launch_bounds__(256) passB_kernel(const DavState* __restrict__ S, double* Vb, double* Sb, int64_t st,
                                                    double* __restrict__ T, int64_t ns, double* part) {
  __shared__ double red[4 * kNV];
  __shared__ double c[16 + kMaxSpace * kKeep];
  op_passB(S, Vb, Sb, st, T, ns, part + blockIdx.x * kNV, blockIdx.x, gridDim.x, red, c);
}

__global__ void __launch_bounds__(256) small_B_kernel(DavState* S, const double* part, int nblk) {
  __shared__ double v[kNV], red[4 * kNV];
  small_B(S, part, nblk, v, red);
}

__global__ void __launch_bounds__(256) advance_kernel(const DavState* S, double* Vb, int64_t st,
                                                      const double* __restrict__ T, int64_t ns) {
  const int m = S->m;
  const bool reorth = S->reorth != 0;
  const double inv = S->inv;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ns; i += (int64_t)gridDim.x * blockDim.x)
    Vb[(int64_t)m * st + i] = advance_value(Vb, st, T, i, m, reorth, inv, S->c2);
}

__global__ void finish_kernel(const DavState* S, double e_const, double* e_out, int32_t* status_out,
                              int32_t* iters_out, double* resid_out) {
  if (threadIdx.x != 0) return;
  if (e_out) *e_out = S->theta + S->E0 + S->ecore + e_const;
  if (status_out) *status_out = S->status;
  if (iters_out) *iters_out = S->iters;
  if (resid_out) *resid_out = S->resid;
}

static inline unsigned nblocks(int64_t n, int per) {
  int64_t b = (n + per - 1) / per;
  if (b < 1) b = 1;
  if (b > kPartBlocks) b = kPartBlocks;
  return (unsigned)b;
}

hipError_t run_plain(const PlainArgs& A, double* e_out, int32_t* status_out, int32_t* iters_out,
                     double* resid_out, hipStream_t st) {
  static_assert(sizeof(DavState) <= 4096 * 8, "state block too small");
  const IncDev& d = A.d;
  const int64_t ns = d.n_sym, sd = d.stride;
  const int mmax = A.max_space;
  double* Vb = A.dav;
  double* Sb = A.dav + mmax * sd;
  double* HD = A.dav + 2 * mmax * sd;
  double* X = HD + sd;
  double* T = A.tmp;
  double* F = A.tmp + sd;
  DavState* S = (DavState*)A.state;
  const double* B = A.ints + d.int_off;
  const int32_t* strs = A.tables + d.str_off;
  const unsigned nb = nblocks(ns, 256);
  hipError_t e;
  DavState hs;
  double ecore = 0.0;
  e = hipMemcpyAsync(&ecore, B + int_block(d.k).misc, sizeof(double), hipMemcpyDeviceToHost, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(string_energy_kernel, dim3((d.n_str + 255) / 256), dim3(256), 0, st, d, strs, B, F);
  hipLaunchKernelGGL(hdiag_kernel, dim3(nb), dim3(256), 0, st, d, strs, B, F, HD, A.part);
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  hipLaunchKernelGGL(init_state_kernel, dim3(1), dim3(256), 0, st, S, A.part, (int)nb, Vb, ns, ecore,
                     A.precision == IFCI_MIXED ? 32 : 64);
  int m = 0, phase = A.precision == IFCI_MIXED ? 32 : 64;
  double shift = 0.0;
  if ((e = hipMemcpyAsync(&hs, S, sizeof(DavState), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  shift = hs.E0;
  while (true) {
    e = launch_sigma_wide(d, A.d_inc, A.inc, A.ints, A.tables, Vb + m * sd, Sb + m * sd, A.E,
                          phase == 32 ? IFCI_MIXED : IFCI_FP64, 1, shift, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(dots_kernel, dim3(nb), dim3(256), 0, st, Vb, sd, m, Sb + m * sd, ns, A.part);
    hipLaunchKernelGGL(small_G_kernel, dim3(1), dim3(256), 0, st, S, A.part, (int)nb, mmax);
    hipLaunchKernelGGL(passA_kernel, dim3(nb), dim3(256), 0, st, S, Vb, Sb, sd, HD, X, T, ns, A.part);
    hipLaunchKernelGGL(small_A_kernel, dim3(1), dim3(256), 0, st, S, A.part, (int)nb, A.r_tol_inner, A.r_tol,
                       A.max_iter, A.evict ? 1 : 0);
    if ((e = hipMemcpyAsync(&hs, S, sizeof(DavState), hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    if (hs.action == kActDone || hs.action == kActMaxIter || hs.action == kActEvicted) break;
    if (hs.action == kActSwitch) {
      hipLaunchKernelGGL(switch_kernel, dim3(nb), dim3(256), 0, st, Vb, X, ns);
      hipLaunchKernelGGL(small_switch_kernel, dim3(1), dim3(256), 0, st, S);
      m = 0;
      phase = 64;
      continue;
    }
    hipLaunchKernelGGL(passB_kernel, dim3(nb), dim3(256), 0, st, S, Vb, Sb, sd, T, ns, A.part);
    hipLaunchKernelGGL(small_B_kernel, dim3(1), dim3(256), 0, st, S, A.part, (int)nb);
    hipLaunchKernelGGL(advance_kernel, dim3(nb), dim3(256), 0, st, S, Vb, sd, T, ns);
    m = hs.mb + 1;
  }
  hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(64), 0, st, S, A.e_const, e_out, status_out, iters_out,
                     resid_out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ vectors
__global__ void expand_kernel(IncDev d, const double* __restrict__ X, double* __restrict__ c) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d.n_det) return;
  const int n = d.n_str;
  const int a = (int)(j / n), b = (int)(j % n);
  const double v = X[packed(a, b)];
  c[j] = (a == b) ? v : v * kRSqrt2;
}

hipError_t launch_expand(const IncDev& d, const double* X, double* c, hipStream_t st) {
  hipLaunchKernelGGL(expand_kernel, dim3((unsigned)((d.n_det + 255) / 256)), dim3(256), 0, st, d, X, c);
  return hipGetLastError();
}

}  // namespace ifci
