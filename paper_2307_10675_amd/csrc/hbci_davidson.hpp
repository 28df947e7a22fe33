// Davidson of the heat-bath CI spaces: the lowest root of H over a
// flip-closed space, on flip-symmetric vectors.  Included by hbci.hip.
//
// Vectors are held over representatives (one entry for each flip pair or
// flip-invariant key, scaled by sqrt(2) for a pair, so that dot products are
// those of the full vector): half the entries of the full vector in every pass
// over the basis, and no flip in the preconditioner.  Only the operand of
// the product with H is spread to the full space, in key order (x).
//
// A step is five launches, none of which the host waits for: the small state
// (subspace matrix, coefficients, the end of the loop) lives on the device and
// is advanced by the block of a pass that ends last, from the partials of all
// blocks.  (Driven from the host a step was 13 launches and 3 read-backs: of
// a solve of a 16-orbital increment with 285020 keys 29 ms were passes and most
// of 83 ms waiting; now 22 and 11.)
#pragma once

#include "device_common.hpp"

namespace ifci {
namespace {

constexpr int kMaxM = 16;       // largest Davidson subspace
constexpr int kKeepRitz = 4;    // Ritz vectors kept at a Davidson restart
constexpr int kParts = kMaxM + 1;
constexpr int kVecBlocks = 512;   // most workgroups of a pass over the basis
constexpr int kVecThreads = 512;  // one entry a thread up to 262144 pairs: residual 15.6 -> 10.7 us at 158104 (256 threads: two rounds)
constexpr int kRowBlocks = 512;   // most workgroups of the product (1024 threads)

__host__ __device__ inline int kept_ritz(int m_max) { return m_max / 2 < kKeepRitz ? m_max / 2 : kKeepRitz; }

// The device's state of a Davidson loop.  Basis vector j is f_j times its
// stored form: a new vector is stored as the second orthogonalisation left
// it, its norm is known only after that pass, and the coefficients of every
// later pass carry f.
struct DavCtl {
  double theta, rn;
  int done;   // 0 running, 1 converged, 2 space exhausted
  int count;  // blocks of the current pass that have ended
  int large;  // largest component of y
  int m;      // basis vectors
  double y[kMaxM], yf[kMaxM];  // Ritz vector; y_j f_j
  double d[kMaxM];             // f_j^2 (V_j . t) of the pass before
  double f[kMaxM];
  double H[256];
  double Y[kMaxM * kKeepRitz];  // restart: f_l Y_lj
};

struct DavSpace {
  const int64_t* ptr;   // rows of H (representatives), columns in the full space
  const int32_t* col;
  const double* val;
  const double* diag;   // per representative
  const int32_t* pos;   // representative -> its place in the full space
  const int32_t* fpos;  // ... and its partner's
  double* x;            // full space
  double* Vb;
  double* Sb;
  double* part;
  DavCtl* ctl;
  int64_t ld, n;        // n representatives
  int64_t n_full;       // entries of x
  // the blocked form of H (below)
  const int32_t* bound;
  const int64_t* bptr;
  const uint32_t* bcol;
  const double* bval;
};

// The blocked form of H: shares of the rows (one workgroup each, about equal
// in entries) by windows of x.  An entry holds its column in the window and
// its row in the share.
constexpr int kWinBits = 13, kWin = 1 << kWinBits, kShareRows = 8192, kShares = 256;
// Spaces in blocked form: at most this many keys (64 windows; a row's piece of a
// window then still has 13 entries at 850 a row) and rows (what 256 shares of
// 8192 rows surely take, hbci_share_kernel).  The limits are those of the
// layout; what it would give past them was not measured.
constexpr int64_t kBlockMax = (int64_t)64 * kWin;
constexpr int64_t kBlockMaxRows = (int64_t)(kShareRows / 8 - 1) * kShares;
constexpr int kBlockLds = (kWin + kShareRows + 16 * kMaxM) * 8;

constexpr double kRoot2 = 1.4142135623730951, kRRoot2 = 0.70710678118654752;

__device__ __forceinline__ void spread(const DavSpace& a, int64_t q, double v) {
  const int32_t p = a.pos[q], f = a.fpos[q];
  const double t = p == f ? v : v * kRRoot2;
  a.x[p] = t;
  a.x[f] = t;
}

__device__ __forceinline__ double gather(const DavSpace& a, int64_t q) {
  const int32_t p = a.pos[q];
  const double t = a.x[p];
  return p == a.fpos[q] ? t : t * kRoot2;
}

// True in every thread of the block that comes last of a pass, whose partials
// (stored and loaded with agent scope, in an order that rests on vmcnt as
// last_block of davidson_ops.hpp explains) are then all visible.
__device__ __forceinline__ bool dav_last(DavCtl* c, int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int l = atomicAdd(&c->count, 1) == (int)gridDim.x - 1;
    if (l) c->count = 0;
    *flag = l;
  }
  __syncthreads();
  return *flag != 0;
}

// out[j] = sum over blocks of part[j][block], j < nv: one wave per row, in a fixed order
__device__ __forceinline__ void dav_totals(const double* part, int nv, int stride, int nblk, double* out) {
  const int lane = threadIdx.x & 63;
  for (int j = threadIdx.x >> 6; j < nv; j += (int)(blockDim.x >> 6)) {
    double s = 0.0;
    for (int b = lane; b < nblk; b += 64)
      s += __hip_atomic_load(part + j * stride + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s = wave_sum(s);
    if (lane == 0) out[j] = s;
  }
  __syncthreads();
}

// part[j][block] = sum over the block of v[j], j < nv <= NV
template <int NV>
__device__ __forceinline__ void dav_partials(const double (&v)[NV], int nv, double* red, double* part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const double t = wave_sum(v[j]);
    if (lane == 0) red[wave * NV + j] = t;
  }
  __syncthreads();
  if ((int)threadIdx.x < nv) {
    double t = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w * NV + threadIdx.x];
    __hip_atomic_store(part + (int)threadIdx.x * kVecBlocks + blockIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The M >= m entries b_j[i] of a basis, all loads in flight together.
template <int M>
__device__ __forceinline__ void dav_entries(const double* B, int64_t ld, int m, int64_t i, double (&b)[M]) {
#pragma unroll
  for (int j = 0; j < M; ++j) b[j] = B[(j < m ? j : 0) * ld + i];
}

__global__ void hbci_dav_start_kernel(DavSpace a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.n) a.Vb[i] = gather(a, i);
  if (i < 256) a.ctl->H[i] = 0.0;
  if (i < kMaxM) a.ctl->f[i] = 1.0;
  if (i == 0) {
    a.ctl->done = 0;
    a.ctl->count = 0;
  }
}

// Residual of the Ritz pair, the correction t into the slot of vector m, and
// the overlaps of t with the basis.
template <int M>
__global__ void __launch_bounds__(kVecThreads) hbci_dav_residual_kernel(DavSpace a, int m, double r_tol) {
  __shared__ double red[kVecThreads / 64 * (M + 1)], tot[M + 1];
  __shared__ int flag;
  DavCtl* c = a.ctl;
  if (c->done) return;
  const double theta = c->theta;
  double y[M], acc[M + 1] = {};
#pragma unroll
  for (int j = 0; j < M; ++j) y[j] = j < m ? c->yf[j] : 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * blockDim.x) {
    double v[M], s[M];
    dav_entries<M>(a.Vb, a.ld, m, i, v);
    dav_entries<M>(a.Sb, a.ld, m, i, s);
    double xi = 0.0, wi = 0.0;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      xi += y[j] * v[j];
      wi += y[j] * s[j];
    }
    const double r = wi - theta * xi;
    double den = theta - a.diag[i];
    if (fabs(den) < 1e-10) den = den < 0.0 ? -1e-10 : 1e-10;
    const double t = r / den;
    a.Vb[m * a.ld + i] = t;
    acc[M] += r * r;
#pragma unroll
    for (int j = 0; j < M; ++j) acc[j] += v[j] * t;
  }
  dav_partials(acc, M + 1, red, a.part);
  if (!dav_last(c, &flag)) return;
  dav_totals(a.part, M + 1, kVecBlocks, gridDim.x, tot);
  if ((int)threadIdx.x < m) {
    const double f = c->f[threadIdx.x];
    c->d[threadIdx.x] = f * f * tot[threadIdx.x];
  }
  if (threadIdx.x == 0) {
    const double rn = sqrt(tot[M]);
    c->rn = rn;
    if (rn <= r_tol) c->done = 1;
  }
}

// t -= sum_j d_j V_j; with LAST the second pass, which leaves the new basis
// vector and spreads it to x, else the overlaps for that pass.
template <int M, bool LAST>
__global__ void __launch_bounds__(kVecThreads) hbci_dav_orth_kernel(DavSpace a, int m) {
  constexpr int NV = LAST ? 1 : M;
  __shared__ double red[kVecThreads / 64 * NV], tot[NV];
  __shared__ int flag;
  DavCtl* c = a.ctl;
  if (c->done) return;
  double d[M], acc[NV] = {};
#pragma unroll
  for (int j = 0; j < M; ++j) d[j] = j < m ? c->d[j] : 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * blockDim.x) {
    double v[M];
    dav_entries<M>(a.Vb, a.ld, m, i, v);
    double t = a.Vb[m * a.ld + i];
#pragma unroll
    for (int j = 0; j < M; ++j) t -= d[j] * v[j];
    a.Vb[m * a.ld + i] = t;
    if constexpr (LAST) {
      acc[0] += t * t;
      spread(a, i, t);
    } else {
#pragma unroll
      for (int j = 0; j < M; ++j) acc[j] += v[j] * t;
    }
  }
  dav_partials(acc, NV, red, a.part);
  if (!dav_last(c, &flag)) return;
  dav_totals(a.part, NV, kVecBlocks, gridDim.x, tot);
  if constexpr (LAST) {
    if (threadIdx.x == 0) {
      if (!(tot[0] > 1e-28)) c->done = 2;  // the space is exhausted
      c->f[m] = 1.0 / sqrt(tot[0]);
    }
  } else if ((int)threadIdx.x < m) {
    const double f = c->f[threadIdx.x];
    c->d[threadIdx.x] = f * f * tot[threadIdx.x];
  }
}

// S_m = H V_m from the spread x, and its overlaps with the basis, for spaces
// past the limits of the blocked form (below), which is the faster one where
// both were timed (on average over a solve: 16.1 us here and 11.1 there at 10
// orbitals, 41.8 and 23.3 at 12, both at eps1 = 1 mEh; 48 and 26 at 14 and 2
// mEh; 338 and 154 at 16, 285020 keys).  One wave per row, 16 neighbouring rows in a workgroup.  Bound by
// first-level cache misses of the gathers.
__global__ void __launch_bounds__(1024, 8) hbci_dav_product_kernel(DavSpace a, int m) {
  __shared__ double red[16 * kMaxM];
  if (a.ctl->done) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double acc = 0.0;  // lane j: V_j . S_m over the wave's rows
  for (int64_t row = (int64_t)blockIdx.x * 16 + wave; row < a.n; row += (int64_t)gridDim.x * 16) {
    const int64_t end = a.ptr[row + 1];
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    // four entries per lane in flight: their columns and values, then the
    // four gathers; past the end the last entry with a zero value
    for (int64_t e = a.ptr[row] + lane; e < end; e += 256) {
      const int64_t e1 = e + 64 < end ? e + 64 : e, e2 = e + 128 < end ? e + 128 : e, e3 = e + 192 < end ? e + 192 : e;
      const int32_t c0 = __builtin_nontemporal_load(a.col + e), c1 = __builtin_nontemporal_load(a.col + e1),
                    c2 = __builtin_nontemporal_load(a.col + e2), c3 = __builtin_nontemporal_load(a.col + e3);
      const double v0 = __builtin_nontemporal_load(a.val + e), v1 = __builtin_nontemporal_load(a.val + e1),
                   v2 = __builtin_nontemporal_load(a.val + e2), v3 = __builtin_nontemporal_load(a.val + e3);
      s0 += v0 * a.x[c0];
      s1 += (e1 != e ? v1 : 0.0) * a.x[c1];
      s2 += (e2 != e ? v2 : 0.0) * a.x[c2];
      s3 += (e3 != e ? v3 : 0.0) * a.x[c3];
    }
    const double s = wave_sum((s0 + s1) + (s2 + s3));
    const int32_t p = a.pos[row];
    double w = s + a.diag[row] * a.x[p];
    if (p != a.fpos[row]) w *= kRoot2;
    if (lane == 0) a.Sb[m * a.ld + row] = w;
    if (lane <= m) acc += a.Vb[lane * a.ld + row] * w;
  }
  if (lane <= m) red[wave * kMaxM + lane] = acc;
  __syncthreads();
  if ((int)threadIdx.x <= m) {
    double t = 0.0;
    for (int w = 0; w < 16; ++w) t += red[w * kMaxM + threadIdx.x];
    a.part[(int)threadIdx.x * kRowBlocks + blockIdx.x] = t;
  }
}

// bound[b]: first row of share b.  A share holds 1 / kShares of 7/8 of the
// entries and 1/8 of the rows, so that it has at most 8 n / kShares rows, and
// at most 8/7 of its part of the entries.
__global__ void hbci_share_kernel(const int64_t* __restrict__ ptr, int64_t n, int32_t* __restrict__ bound) {
  const int b = threadIdx.x;
  if (b > kShares) return;
  // weight before row r, in units of 1 / (8 n nnz), against b / kShares
  const double nnz = (double)(ptr[n] > 0 ? ptr[n] : 1), want = (double)b / kShares;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (0.875 * ((double)ptr[mid] / nnz) + 0.125 * ((double)mid / (double)n) < want)
      lo = mid + 1;
    else
      hi = mid;
  }
  bound[b] = b == kShares ? (int32_t)n : (int32_t)lo;
}

// off[w][q]: entries of row q before window w, w <= nwin (one wave per row; its columns ascend)
__global__ void __launch_bounds__(256) hbci_win_offsets_kernel(const int64_t* __restrict__ ptr,
                                                               const int32_t* __restrict__ col, int64_t n, int nwin,
                                                               uint16_t* __restrict__ off) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); q < n; q += nw) {
    const int64_t b = ptr[q];
    const int len = (int)(ptr[q + 1] - b);
    for (int e = lane; e <= len; e += 64) {
      const int w = e < len ? col[b + e] >> kWinBits : nwin, v = e > 0 ? col[b + e - 1] >> kWinBits : -1;
      for (int u = v + 1; u <= w; ++u) off[u * n + q] = (uint16_t)e;
    }
  }
}

// bptr[share][w]: place of block (share, w); a share's blocks lie where its
// rows lie in H.  One workgroup per share, a wave per window.
__global__ void __launch_bounds__(1024) hbci_block_ptr_kernel(const int64_t* __restrict__ ptr, int64_t n, int nwin,
                                                              const int32_t* __restrict__ bound,
                                                              const uint16_t* __restrict__ off,
                                                              int64_t* __restrict__ bptr) {
  __shared__ int cnt[kBlockMax / kWin];
  const int lane = threadIdx.x & 63;
  const int r0 = bound[blockIdx.x], r1 = bound[blockIdx.x + 1];
  for (int w = threadIdx.x >> 6; w < nwin; w += 16) {
    int c = 0;
    for (int64_t q = r0 + lane; q < r1; q += 64) c += (int)off[(w + 1) * n + q] - (int)off[w * n + q];
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if (lane == 0) cnt[w] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t at = ptr[r0];
    for (int w = 0; w < nwin; ++w) {
      bptr[(int64_t)blockIdx.x * nwin + w] = at;
      at += cnt[w];
    }
    if (blockIdx.x == kShares - 1) bptr[(int64_t)kShares * nwin] = at;
  }
}

// Block (blockIdx.x, blockIdx.y) from the rows of H.  Its entries row by row
// are cut into chunks of kChunk, and a chunk is laid out with its 64 parts
// side by side: the lanes of a wave of the product then add to different rows.
// A chunk is put together in LDS and written in one piece.  (Entries written
// one by one to their places, 8 bytes of a line at a time, took 3.29 ms a step on
// average at 285020 keys.)
constexpr int kChunk = 3072, kChunkSlots = (kChunk / 64 + 1) * 65;
constexpr int kBlockFillLds = (kShareRows + 1024) * 4 + kChunkSlots * 12;

__global__ void __launch_bounds__(1024) hbci_block_fill_kernel(const int64_t* __restrict__ ptr,
                                                               const int32_t* __restrict__ col,
                                                               const double* __restrict__ val, int64_t n, int nwin,
                                                               const int32_t* __restrict__ bound,
                                                               const uint16_t* __restrict__ off,
                                                               const int64_t* __restrict__ bptr,
                                                               uint32_t* __restrict__ bcol, double* __restrict__ bval) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* sv = (double*)smem;
  uint32_t* sc = (uint32_t*)(sv + kChunkSlots);
  int* first = (int*)(sc + kChunkSlots);  // entries of the block before each row
  int* part = first + kShareRows;
  const int tid = threadIdx.x, w = blockIdx.y;
  const int r0 = bound[blockIdx.x], rows = bound[blockIdx.x + 1] - r0;
  const int64_t start = bptr[(int64_t)blockIdx.x * nwin + w];
  const uint16_t* o0 = off + (int64_t)w * n + r0;
  const uint16_t* o1 = o0 + n;
  constexpr int per = kShareRows / 1024;
  for (int i = tid; i < kShareRows; i += 1024) first[i] = i < rows ? (int)o1[i] - (int)o0[i] : 0;
  __syncthreads();
  int own = 0;
  for (int i = 0; i < per; ++i) own += first[tid * per + i];
  part[tid] = own;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int v = tid >= o ? part[tid - o] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  int sum = part[tid] - own;
  for (int i = 0; i < per; ++i) {
    const int v = first[tid * per + i];
    first[tid * per + i] = sum;
    sum += v;
  }
  __syncthreads();
  const int total = part[1023];
  for (int c0 = 0; c0 < total; c0 += kChunk) {
    const int nc = total - c0 < kChunk ? total - c0 : kChunk;
    const int S = nc >> 6, rem = nc & 63;  // parts of S + 1 entries, rem of them, then of S
    // the rows of this thread's entries (the last row that starts at or
    // before one), then all their loads in flight
    int row[kChunk / 1024];
    uint32_t c[kChunk / 1024];
    double v[kChunk / 1024];
#pragma unroll
    for (int u = 0; u < kChunk / 1024; ++u) {
      const int e = c0 + u * 1024 + tid;
      int lo = 0, hi = rows;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first[mid] <= e)
          lo = mid;
        else
          hi = mid;
      }
      row[u] = lo;
    }
#pragma unroll
    for (int u = 0; u < kChunk / 1024; ++u)
      if (u * 1024 + tid < nc) {
        const int g = row[u];
        const int64_t i = ptr[r0 + g] + o0[g] + (c0 + u * 1024 + tid - first[g]);
        c[u] = (uint32_t)col[i];
        v[u] = val[i];
      }
#pragma unroll
    for (int u = 0; u < kChunk / 1024; ++u) {
      const int e = u * 1024 + tid;
      if (e >= nc) break;
      int lane, step;
      if (nc == kChunk) {
        lane = e / (kChunk / 64);
        step = e % (kChunk / 64);
      } else if (e < rem * (S + 1)) {
        lane = e / (S + 1);
        step = e - lane * (S + 1);
      } else {
        const int d = e - rem * (S + 1), k = d / S;
        lane = rem + k;
        step = d - k * S;
      }
      sv[step * 65 + lane] = v[u];
      sc[step * 65 + lane] = (c[u] & (kWin - 1)) | (uint32_t)row[u] << kWinBits;
    }
    __syncthreads();
    for (int i = tid; i < nc; i += 1024) {
      const int at = (i >> 6) * 65 + (i & 63);
      bval[start + c0 + i] = sv[at];
      bcol[start + c0 + i] = sc[at];
    }
    __syncthreads();
  }
}

// The product from the blocked form: a workgroup takes its share of the rows
// through the windows one after the other, x of the window in LDS (loaded to
// registers while the window before is worked on) and the sums of its rows
// beside it.  Gathers and sums are LDS accesses, and what is left of global
// memory is the stream of H.  (The row form's gathers miss the first-level
// cache: the 16 rows of a chunk touch 414 lines each and 1212 together, and
// there is 32 KB.  At 285020 keys and 114.7e6 nonzeros it takes 608 us, with
// 73.7e6 line requests, of which 12e6 for H.)
__global__ void __launch_bounds__(1024) hbci_dav_block_kernel(DavSpace a, int m) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* xw = (double*)smem;
  double* sum = xw + kWin;
  double* red = sum + kShareRows;
  if (a.ctl->done) return;
  constexpr int kPer = kWin / 1024;
  const int tid = threadIdx.x;
  const int64_t r0 = a.bound[blockIdx.x];
  const int rows = a.bound[blockIdx.x + 1] - (int)r0;
  const int nwin = (int)((a.n_full + kWin - 1) / kWin);
  const int64_t* bp = a.bptr + (int64_t)blockIdx.x * nwin;
  double xr[kPer];
  auto fetch = [&](int w) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int64_t p = (int64_t)w * kWin + i * 1024 + tid;
      xr[i] = p < a.n_full ? a.x[p] : 0.0;
    }
  };
  fetch(0);
  for (int i = tid; i < rows; i += 1024) sum[i] = 0.0;
  for (int w = 0; w < nwin; ++w) {
    const int64_t p0 = bp[w], p1 = bp[w + 1];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) xw[i * 1024 + tid] = xr[i];
    __syncthreads();
    if (w + 1 < nwin) fetch(w + 1);
    // four entries of a lane follow each other in H: those of one row are summed first
    for (int64_t p = p0 + (tid >> 6) * 256 + (tid & 63); p < p1; p += 4096) {
      uint32_t c[4];
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // past the end the first entry again, with a zero value
        const int64_t i = p + u * 64 < p1 ? p + u * 64 : p;
        c[u] = __builtin_nontemporal_load(a.bcol + i);
        v[u] = __builtin_nontemporal_load(a.bval + i);
      }
      double s = v[0] * xw[c[0] & (kWin - 1)];
#pragma unroll
      for (int u = 1; u < 4; ++u) {
        const double t = (p + u * 64 < p1 ? v[u] : 0.0) * xw[c[u] & (kWin - 1)];
        if (c[u] >> kWinBits != c[u - 1] >> kWinBits) {
          lds_add(&sum[c[u - 1] >> kWinBits], s);
          s = 0.0;
        }
        s += t;
      }
      lds_add(&sum[c[3] >> kWinBits], s);
    }
  }
  __syncthreads();
  double acc[kMaxM] = {};
  for (int g = tid; g < rows; g += 1024) {
    const int64_t row = r0 + g;
    const int32_t p = a.pos[row];
    double y = sum[g] + a.diag[row] * a.x[p];
    if (p != a.fpos[row]) y *= kRoot2;
    a.Sb[m * a.ld + row] = y;
#pragma unroll
    for (int j = 0; j < kMaxM; ++j)
      if (j <= m) acc[j] += a.Vb[j * a.ld + row] * y;
  }
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int j = 0; j < kMaxM; ++j)
    if (j <= m) {
      const double t = wave_sum(acc[j]);
      if (lane == 0) red[wave * kMaxM + j] = t;
    }
  __syncthreads();
  if (tid <= m) {
    double t = 0.0;
    for (int w = 0; w < 16; ++w) t += red[w * kMaxM + tid];
    a.part[tid * kRowBlocks + blockIdx.x] = t;
  }
}

// The new column of the subspace matrix from the partials of the product,
// and its lowest pair (at m + 1 = m_max all pairs: the next launch restarts).
// A launch of its own: as the end of the product it took that kernel past 64
// VGPRs, and with them half of its waves.
__global__ void __launch_bounds__(1024) hbci_dav_subspace_kernel(DavSpace a, int nblk, int m, int m_max) {
  __shared__ double G[256], Q[256], ev[16], yv[16], tot[kMaxM], th;
  __shared__ int perm[16], large;
  DavCtl* c = a.ctl;
  if (c->done) return;
  dav_totals(a.part, m + 1, kRowBlocks, nblk, tot);
  const int n = m + 1, tid = threadIdx.x, lane = tid & 63;
  if (tid < 256) {
    double h = c->H[tid];
    const int r = tid >> 4, q = tid & 15, j = r == m ? q : r;
    if ((r == m || q == m) && r <= m && q <= m) {
      h = c->f[j] * c->f[m] * tot[j];
      c->H[tid] = h;
    }
    G[tid] = h;
  }
  if (tid < 16) yv[tid] = c->y[tid];
  __syncthreads();
  const bool restart = n == m_max;
  if (tid < 64) {
    int pn = restart ? -1 : lowest_pair(G, n, c->large, c->theta, yv, &th, yv);
    if (pn < 0) {
      jacobi_lowest(G, Q, n, &th, yv, ev, perm);
      pn = 0;
      for (int j = 1; j < n; ++j)
        if (fabs(yv[j]) > fabs(yv[pn])) pn = j;
    }
    if (lane == 0) large = pn;
  }
  __syncthreads();
  if (!restart) {
    if (tid < n) {
      c->y[tid] = yv[tid];
      c->yf[tid] = yv[tid] * c->f[tid];
    }
  } else {
    const int keep = kept_ritz(m_max);
    if (tid < n * kKeepRitz) {
      const int l = tid / kKeepRitz, j = tid % kKeepRitz;
      c->Y[tid] = j < keep ? Q[l * 16 + perm[j]] * c->f[l] : 0.0;
    }
    __syncthreads();
    if (tid < 256) c->H[tid] = ((tid >> 4) == (tid & 15) && (tid & 15) < keep) ? ev[tid & 15] : 0.0;
    if (tid < kMaxM) {
      c->f[tid] = 1.0;
      c->y[tid] = c->yf[tid] = tid == 0 ? 1.0 : 0.0;
    }
  }
  if (tid == 0) {
    c->theta = th;
    c->large = restart ? 0 : large;
    c->m = restart ? kept_ritz(m_max) : n;
  }
}

// Thick restart: the kept Ritz vectors and their products, in place.
template <int M>
__global__ void __launch_bounds__(256) hbci_dav_restart_kernel(DavSpace a, int m, int keep) {
  if (a.ctl->done) return;
  const double* Y = a.ctl->Y;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * blockDim.x) {
    double v[M], s[M];
    dav_entries<M>(a.Vb, a.ld, m, i, v);
    dav_entries<M>(a.Sb, a.ld, m, i, s);
    for (int j = 0; j < keep; ++j) {
      double cv = 0.0, cs = 0.0;
#pragma unroll
      for (int l = 0; l < M; ++l)
        if (l < m) {
          cv += Y[l * kKeepRitz + j] * v[l];
          cs += Y[l * kKeepRitz + j] * s[l];
        }
      a.Vb[j * a.ld + i] = cv;
      a.Sb[j * a.ld + i] = cs;
    }
  }
}

// x = the Ritz vector, over the full space
__global__ void __launch_bounds__(256) hbci_dav_vector_kernel(DavSpace a) {
  const int m = a.ctl->m;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * blockDim.x) {
    double xi = 0.0;
    for (int j = 0; j < m; ++j) xi += a.ctl->yf[j] * a.Vb[j * a.ld + i];
    spread(a, i, xi);
  }
}

// ------------------------------------- Davidson of a small space in one workgroup

// Spaces of up to kSmallDav determinants solve their Davidson in a single
// launch of one 1024-thread workgroup: the same iteration, with the small
// eigenproblem on one wavefront and every reduction in LDS, so a selection step
// costs one launch and one read-back.  The increments of an expansion run on
// concurrent streams, one CU each.
constexpr int64_t kSmallDav = 1024;
constexpr int kSmallThreads = 1024;

struct SmallDav {
  DavSpace s;
  int m_max, max_dav;
  double r_tol;
  double* out;  // theta, residual norm, converged (0/1)
};

// y = H x over the representatives
__device__ void small_product(const DavSpace& a, double* __restrict__ y) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int64_t row = wave; row < a.n; row += nw) {
    double s = 0.0;
    for (int64_t e = a.ptr[row] + lane; e < a.ptr[row + 1]; e += 64) s += a.val[e] * a.x[a.col[e]];
    s = wave_sum(s);
    if (lane == 0) {
      const int32_t p = a.pos[row];
      const double w = s + a.diag[row] * a.x[p];
      y[row] = p == a.fpos[row] ? w : w * kRoot2;
    }
  }
  __syncthreads();
}

// res[j] = sum over the workgroup of v[j], j < nv (v per thread, nv <= 17)
__device__ __forceinline__ void small_sums(const double (&v)[kMaxM + 1], int nv, double* red, double* res) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int j = 0; j < kMaxM + 1; ++j)
    if (j < nv) {
      const double t = wave_sum(v[j]);
      if (lane == 0) red[wave * (kMaxM + 1) + j] = t;
    }
  __syncthreads();
  if ((int)threadIdx.x < nv) {
    double t = 0.0;
    for (int w = 0; w < nw; ++w) t += red[w * (kMaxM + 1) + threadIdx.x];
    res[threadIdx.x] = t;
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kSmallThreads) hbci_dav_small_kernel(SmallDav a) {
  __shared__ double Hs[256], A[256], Q[256], ev[16], yv[16], th;
  __shared__ double red[(kSmallThreads / 64) * (kMaxM + 1)], res[kMaxM + 1];
  __shared__ int perm[16], large;
  const DavSpace& sp = a.s;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t n = sp.n, ld = sp.ld;
  double* Vb = sp.Vb;
  double* Sb = sp.Sb;
  for (int64_t i = tid; i < n; i += nt) Vb[i] = gather(sp, i);
  for (int t = tid; t < 256; t += nt) Hs[t] = 0.0;
  __syncthreads();
  small_product(sp, Sb);
  {
    double v[kMaxM + 1] = {};
    for (int64_t i = tid; i < n; i += nt) v[0] += Vb[i] * Sb[i];
    small_sums(v, 1, red, res);
  }
  if (tid == 0) {
    Hs[0] = th = res[0];
    yv[0] = 1.0;
    large = 0;
  }
  __syncthreads();
  int m = 1, conv = 0;
  double theta = res[0], rn = 1e300;
  // each thread owns its entries of every vector but x; the residual goes to the slot of vector m as the correction
  for (int it = 0;; ++it) {
    theta = th;
    double* T = Vb + m * ld;
    double d[kMaxM + 1] = {};
    {
      double r2[kMaxM + 1] = {};
      for (int64_t i = tid; i < n; i += nt) {
        double xi = 0.0, wi = 0.0;
        for (int j = 0; j < m; ++j) {
          xi += yv[j] * Vb[j * ld + i];
          wi += yv[j] * Sb[j * ld + i];
        }
        const double r = wi - theta * xi;
        double den = theta - sp.diag[i];
        if (fabs(den) < 1e-10) den = den < 0.0 ? -1e-10 : 1e-10;
        const double t = r / den;
        T[i] = t;
        r2[0] += r * r;
        for (int j = 0; j < kMaxM; ++j)
          if (j < m) d[j] += Vb[j * ld + i] * t;
      }
      small_sums(r2, 1, red, res);
    }
    rn = sqrt(res[0]);
    if (rn <= a.r_tol) conv = 1;
    if (conv || it == a.max_dav) break;
    __syncthreads();
    double t2 = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
      small_sums(d, m, red, res);
      double w[kMaxM + 1] = {};
      for (int j = 0; j < kMaxM + 1; ++j) d[j] = 0.0;
      for (int64_t i = tid; i < n; i += nt) {
        double ti = T[i];
        for (int j = 0; j < m; ++j) ti -= res[j] * Vb[j * ld + i];
        T[i] = ti;
        w[0] += ti * ti;
        for (int j = 0; j < kMaxM; ++j)
          if (j < m) d[j] += Vb[j * ld + i] * ti;
      }
      __syncthreads();
      if (pass == 1) {
        small_sums(w, 1, red, res);
        t2 = res[0];
      }
    }
    if (!(t2 > 1e-28)) break;  // the space is exhausted
    const double inv = 1.0 / sqrt(t2);
    for (int64_t i = tid; i < n; i += nt) {
      const double t = T[i] * inv;
      T[i] = t;
      spread(sp, i, t);
    }
    __syncthreads();
    small_product(sp, Sb + m * ld);
    {
      double v[kMaxM + 1] = {};
      for (int64_t i = tid; i < n; i += nt) {
        const double si = Sb[m * ld + i];
#pragma unroll
        for (int j = 0; j < kMaxM + 1; ++j)
          if (j <= m) v[j] += Vb[j * ld + i] * si;
      }
      small_sums(v, m + 1, red, res);
    }
    if (tid <= m) {
      Hs[tid * 16 + m] = res[tid];
      Hs[m * 16 + tid] = res[tid];
    }
    __syncthreads();
    ++m;
    const bool restart = m == a.m_max;
    if (tid < 64) {
      int pn = restart ? -1 : lowest_pair(Hs, m, large, th, yv, &th, yv);
      if (pn < 0) {
        for (int t = tid; t < 256; t += 64) A[t] = Hs[t];
        jacobi_lowest(A, Q, m, &th, yv, ev, perm);
        pn = 0;
        for (int j = 1; j < m; ++j)
          if (fabs(yv[j]) > fabs(yv[pn])) pn = j;
      }
      if (tid == 0) large = pn;
    }
    __syncthreads();
    if (restart) {  // thick restart, in place
      const int keep = kept_ritz(a.m_max);
      for (int64_t i = tid; i < n; i += nt) {
        double bv[kMaxM], bs[kMaxM];
        for (int l = 0; l < kMaxM; ++l)
          if (l < m) {
            bv[l] = Vb[l * ld + i];
            bs[l] = Sb[l * ld + i];
          }
        for (int j = 0; j < keep; ++j) {
          double cv = 0.0, cs = 0.0;
          for (int l = 0; l < kMaxM; ++l)
            if (l < m) {
              const double q = Q[l * 16 + perm[j]];
              cv += q * bv[l];
              cs += q * bs[l];
            }
          Vb[j * ld + i] = cv;
          Sb[j * ld + i] = cs;
        }
      }
      __syncthreads();
      if (tid < 256) Hs[tid] = ((tid >> 4) == (tid & 15) && (tid & 15) < keep) ? ev[tid & 15] : 0.0;
      if (tid < 16) yv[tid] = tid == 0 ? 1.0 : 0.0;
      if (tid == 0) large = 0;
      __syncthreads();
      m = keep;
    }
  }
  for (int64_t i = tid; i < n; i += nt) {
    double xi = 0.0;
    for (int j = 0; j < m; ++j) xi += yv[j] * Vb[j * ld + i];
    spread(sp, i, xi);
  }
  if (tid == 0) {
    a.out[0] = theta;
    a.out[1] = rn;
    a.out[2] = conv;
  }
}

}  // namespace
}  // namespace ifci
