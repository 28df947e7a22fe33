// Steps of the device-wide Davidson iteration (Davidson, J. Comput. Phys. 17,
// 87, 1975; thick restart, DGKS re-orthogonalisation), written once and used
// by the per-increment host-driven loop and by the batched solver that runs
// many increments per launch with device-side control.  Internal.
//
// Vector steps work on packed scaled symmetric vectors of length ns (entry
// (a <= b) at b (b + 1) / 2 + a, off-diagonals times sqrt 2, so plain dot
// products are those of the full vectors).  A step covers the elements
// blk * blockDim + tid + k * nblk * blockDim of one increment (256 threads)
// and writes its partial sums to part[blk][kNV]; the small steps then reduce
// the nblk partials in a fixed order, so results do not depend on how the
// blocks of a launch are scheduled.  A small step is run by one 256-thread
// block: a launch of its own, or the block of the vector step that finishes
// last (last_block).
//
// An iteration after sigma: the subspace matrix and its lowest pair (small_G),
// the Ritz vector, residual and preconditioned correction with its overlaps
// (pass A, small_A), the thick restart where one is due and the first
// orthogonalisation (pass B, small_B), and the second one with the
// normalisation, formed entry by entry where the new basis vector is needed
// (advance_value).  Each pass loads an entry of every basis vector once, all
// loads in flight together, and keeps them in registers.
#pragma once

#include "device_common.hpp"

namespace ifci {

constexpr int kNV = kMaxSpace + 2;  // values of a partial row

// Solver state of one increment (device memory, one block of 4096 doubles).
struct DavState {
  double G[256];   // Rayleigh matrix V^T H V (stride 16)
  double Q[256];   // its eigenvectors (written at a restart)
  double y[16];    // lowest Ritz vector in the subspace basis
  double cf[16];   // V^T t (first orthogonalisation pass)
  double c2[16];   // V^T t (second pass)
  double ev[16];   // Ritz values, increasing
  double theta, E0, resid, tt0, tt, inv, ecore;
  int m, phase, iters, status, restart, action, mb, reorth;
  int guess, keep, alive;
  int plarge;  // largest component of y (for the next subspace solve)
  int fresh;   // V[m] is in place (start of a stage), not to be formed from t
  int count;   // blocks of the current pass that are done (last_block)
  int exhausted;  // the last correction lay in the span of the basis: V[m] is zero
  int pad;
  int perm[16];
};

// LDS of small_G
struct SmallG {
  double g[kNV], G[256], Q[256], y[16], ev[16], theta;
  int perm[16];
};

// action codes written by the residual test (small_A)
// (kActMaxIter: out of iterations or of directions)
enum { kActContinue = 0, kActDone = 1, kActSwitch = 2, kActMaxIter = 3, kActEvicted = 4 };

constexpr int kPartBlocks = 1024;

// Partial sums are written and read past the caches of an XCD, so that the
// last block of the same launch sees those of all others.
__device__ __forceinline__ void part_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double part_load(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in every thread of the block that comes last of the nb blocks of an
// increment's pass (its partial rows, written by part_store, all visible);
// resets the counter.  Every block of the pass calls it once.  The atomics are
// relaxed, with no release and acquire between them (which would write back
// and invalidate an L2 per block): what orders them is that an agent-scope
// store of gfx950 is written through to memory and has reached it once vmcnt
// is zero, and that an agent-scope load is not served from a cache that it
// could be stale in.  So only data stored by part_store and loaded by part_load
// passes from one block to another here.
__device__ __forceinline__ bool last_block(int* count, int nb) {
  __shared__ int last;
  // each wave's stores have reached memory before its thread count passes on
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    last = atomicAdd(count, 1) == nb - 1;
    if (last) *count = 0;
  }
  __syncthreads();
  const bool l = last != 0;
  __syncthreads();
  return l;
}

// Partial sums of the first nv values of this block into part_row[0..nv).
// Ends with a barrier, so `red` (4 kNV doubles of LDS) may be reused right
// away.
__device__ inline void block_partial_row(double (&v)[kNV], int nv, double* part_row, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int j = 0; j < kNV; ++j)
    if (j < nv) {
      const double t = wave_sum(v[j]);
      if (lane == 0) red[wave * kNV + j] = t;
    }
  __syncthreads();
  if ((int)threadIdx.x < nv) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w * kNV + threadIdx.x];
    part_store(part_row + threadIdx.x, s);
  }
  __syncthreads();
}

// Sum of nblk partial rows, value j in out[j] (LDS) for j < nv, by one block of
// 256 threads: thread t adds the rows t, t + 256, ... in order, then the
// lanes and the waves in a fixed order.
__device__ inline void reduce_parts(const double* part, int nblk, int nv, double* out, double* red) {
  double acc[kNV];
#pragma unroll
  for (int j = 0; j < kNV; ++j) acc[j] = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x)
#pragma unroll
    for (int j = 0; j < kNV; ++j)
      if (j < nv) acc[j] += part_load(part + b * kNV + j);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int j = 0; j < kNV; ++j)
    if (j < nv) {
      const double t = wave_sum(acc[j]);
      if (lane == 0) red[wave * kNV + j] = t;
    }
  __syncthreads();
  if ((int)threadIdx.x < nv) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w * kNV + threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// f(std::integral_constant<int, N>) with N the number of basis vectors
// rounded up to 4, 8, 12 or 16
template <typename F>
__device__ __forceinline__ void by_count(int n, F&& f) {
  if (n <= 4)
    f(std::integral_constant<int, 4>{});
  else if (n <= 8)
    f(std::integral_constant<int, 8>{});
  else if (n <= 12)
    f(std::integral_constant<int, 12>{});
  else
    f(std::integral_constant<int, 16>{});
}
// entry i of the first n of N vectors (vector 0 again past n: its line is
// there already, and the loads need no branch)
template <int N>
__device__ __forceinline__ void load_entries(const double* B, int64_t st, int n, int64_t i, double (&v)[N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = B[(j < n ? j : 0) * st + i];
}

// ---------------------------------------------------------------- vector steps
// part_row[j] = V_j . s for j <= m
__device__ inline void op_dots(const double* __restrict__ Vb, int64_t st, int m, const double* __restrict__ s,
                               int64_t ns, double* part_row, int blk, int nblk, double* red) {
  by_count(m + 1, [&](auto nn) {
    constexpr int N = decltype(nn)::value;
    double acc[kNV];
#pragma unroll
    for (int j = 0; j < kNV; ++j) acc[j] = 0.0;
    for (int64_t i = (int64_t)blk * blockDim.x + threadIdx.x; i < ns; i += (int64_t)nblk * blockDim.x) {
      double v[N];
      load_entries<N>(Vb, st, m + 1, i, v);
      const double si = s[i];
#pragma unroll
      for (int j = 0; j < N; ++j) acc[j] += v[j] * si;
    }
    block_partial_row(acc, m + 1, part_row, red);
  });
}

// Ritz vector x = V y, residual r = S y - theta x, preconditioned
// t = r / (theta - (H_II - E0)) (denominator clamped at 1e-8); stores x and
// t; partials: r.r, t.t, then V_j . t (j <= m) from 2 on.  `ysh` is 16
// doubles of LDS.
__device__ inline void op_passA(const DavState* __restrict__ S, const double* __restrict__ Vb,
                                const double* __restrict__ Sb, int64_t st, const double* __restrict__ HD,
                                double* __restrict__ X, double* __restrict__ T, int64_t ns, double* part_row,
                                int blk, int nblk, double* red, double* ysh) {
  const int m = S->m;
  const double theta = S->theta, E0 = S->E0;
  if (threadIdx.x < 16) ysh[threadIdx.x] = (int)threadIdx.x <= m ? S->y[threadIdx.x] : 0.0;
  __syncthreads();
  by_count(m + 1, [&](auto nn) {
    constexpr int N = decltype(nn)::value;
    double acc[kNV];
#pragma unroll
    for (int j = 0; j < kNV; ++j) acc[j] = 0.0;
    for (int64_t i = (int64_t)blk * blockDim.x + threadIdx.x; i < ns; i += (int64_t)nblk * blockDim.x) {
      double v[N], sv[N];
      load_entries<N>(Vb, st, m + 1, i, v);
      load_entries<N>(Sb, st, m + 1, i, sv);
      const double hd = HD[i];
      double x = 0.0, sx = 0.0;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        x += ysh[j] * v[j];
        sx += ysh[j] * sv[j];
      }
      const double r = sx - theta * x;
      double den = theta - (hd - E0);
      if (fabs(den) < 1e-8) den = (den < 0.0) ? -1e-8 : 1e-8;
      const double t = r / den;
      acc[0] += r * r;
      acc[1] += t * t;
#pragma unroll
      for (int j = 0; j < N; ++j) acc[2 + j] += v[j] * t;
      T[i] = t;
      X[i] = x;
    }
    block_partial_row(acc, m + 3, part_row, red);
  });
}

// First orthogonalisation pass: t -= sum_{j <= mb} cf[j] V_j; partials t.t,
// then V_j . t (j <= mb) from 1 on.  At a thick restart the basis is first
// replaced entry by entry: V[k] <- sum_j Q[j][perm k] V[j] for the `keep`
// lowest Ritz vectors (mb = keep - 1), the same for S.  `sh` is 16 + kMaxSpace
// kKeep doubles of LDS.
__device__ inline void op_passB(const DavState* __restrict__ S, double* Vb, double* Sb, int64_t st,
                                double* __restrict__ T, int64_t ns, double* part_row, int blk, int nblk, double* red,
                                double* sh) {
  const int mb = S->mb, m = S->m;
  const bool restart = S->restart != 0;
  double* const csh = sh;
  double* const qsh = sh + 16;
  if (threadIdx.x < 16) csh[threadIdx.x] = (int)threadIdx.x <= mb ? S->cf[threadIdx.x] : 0.0;
  if (restart)
    for (int t = threadIdx.x; t < kMaxSpace * kKeep; t += blockDim.x) {
      const int j = t / kKeep, kk = t % kKeep;
      qsh[t] = (j <= m && kk <= mb) ? S->Q[j * 16 + S->perm[kk]] : 0.0;
    }
  __syncthreads();
  const int64_t i0 = (int64_t)blk * blockDim.x + threadIdx.x, di = (int64_t)nblk * blockDim.x;
  double acc[kNV];
#pragma unroll
  for (int j = 0; j < kNV; ++j) acc[j] = 0.0;
  if (restart) {
    by_count(m + 1, [&](auto nn) {
      constexpr int N = decltype(nn)::value;
      for (int64_t i = i0; i < ns; i += di) {
        // the kept vectors' entries, four old ones of each set at a time
        double nv[kKeep], ns2[kKeep];
#pragma unroll
        for (int kk = 0; kk < kKeep; ++kk) nv[kk] = ns2[kk] = 0.0;
#pragma unroll
        for (int j0 = 0; j0 < N; j0 += 4) {
          double v[4], sv[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t at = (j0 + j <= m ? j0 + j : 0) * st + i;
            v[j] = Vb[at];
            sv[j] = Sb[at];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int kk = 0; kk < kKeep; ++kk) {
              nv[kk] += qsh[(j0 + j) * kKeep + kk] * v[j];
              ns2[kk] += qsh[(j0 + j) * kKeep + kk] * sv[j];
            }
        }
        double t = T[i];
#pragma unroll
        for (int kk = 0; kk < kKeep; ++kk) {
          t -= csh[kk] * nv[kk];
          if (kk <= mb) {
            Vb[kk * st + i] = nv[kk];
            Sb[kk * st + i] = ns2[kk];
          }
        }
        T[i] = t;
        acc[0] += t * t;
#pragma unroll
        for (int kk = 0; kk < kKeep; ++kk) acc[1 + kk] += nv[kk] * t;
      }
    });
  } else {
    by_count(mb + 1, [&](auto nn) {
      constexpr int N = decltype(nn)::value;
      for (int64_t i = i0; i < ns; i += di) {
        double v[N];
        load_entries<N>(Vb, st, mb + 1, i, v);
        double t = T[i];
#pragma unroll
        for (int j = 0; j < N; ++j) t -= csh[j] * v[j];
        T[i] = t;
        acc[0] += t * t;
#pragma unroll
        for (int j = 0; j < N; ++j) acc[1 + j] += v[j] * t;
      }
    });
  }
  block_partial_row(acc, mb + 2, part_row, red);
}

// Start of the FP64 stage: V[0] <- x.
__device__ inline void op_switch(double* Vb, const double* X, int64_t ns, int blk, int nblk) {
  for (int64_t i = (int64_t)blk * blockDim.x + threadIdx.x; i < ns; i += (int64_t)nblk * blockDim.x) Vb[i] = X[i];
}
__device__ inline void small_switch(DavState* S) {
  for (int i = threadIdx.x; i < 256; i += blockDim.x) S->G[i] = 0.0;
  if (threadIdx.x == 0) {
    S->phase = 64;
    S->m = 0;
    S->plarge = 0;
    S->fresh = 1;
    S->exhausted = 0;
  }
}

// Entry i of the new basis vector V[m], m >= 1: the correction t after the
// second (DGKS) pass, taken when the first lost more than half its norm,
// normalised.  (m, reorth, inv and the second overlaps c2 from the state.)
__device__ __forceinline__ double advance_value(const double* Vb, int64_t st, const double* T, int64_t i, int m,
                                                bool reorth, double inv, const double* c2) {
  double t = T[i];
  if (reorth)
    for (int j = 0; j < m; ++j) t -= c2[j] * Vb[j * st + i];
  return t * inv;
}

// ---------------------------------------------------------------- small steps
// One block of 256 threads per increment; `red` is 4 kNV doubles of LDS and
// the other scratch arguments are LDS too.

// New column of the Rayleigh matrix from the partials of op_dots, then its
// lowest eigenpair (lowest_pair; a full Jacobi decomposition at a restart or
// where that does not apply); counts the iteration and decides whether the
// next orthogonalisation is preceded by a thick restart.  With a zero V[m] the
// pair is that of the basis before it.
__device__ inline void small_G(DavState* S, const double* part, int nblk, int mmax, SmallG* sh, double* red) {
  const int m = S->m, n = m + 1, lane = threadIdx.x;
  const bool exhausted = S->exhausted != 0, restart = n == mmax && !exhausted;
  sh->G[threadIdx.x] = S->G[threadIdx.x];
  if (lane < kMaxSpace) sh->y[lane] = S->y[lane];
  reduce_parts(part, nblk, n, sh->g, red);
  if (lane <= m) {
    const double v = sh->g[lane];
    sh->G[lane * 16 + m] = v;
    sh->G[m * 16 + lane] = v;
    S->G[lane * 16 + m] = v;
    S->G[m * 16 + lane] = v;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    int pn;
    if (exhausted) {
      pn = S->plarge;
      if (lane == 0) {
        sh->theta = S->theta;
        sh->y[m] = 0.0;
      }
      __builtin_amdgcn_wave_barrier();
    } else {
      pn = restart ? -1 : lowest_pair(sh->G, n, S->plarge, S->theta, sh->y, &sh->theta, sh->y);
    }
    if (pn < 0) {
      jacobi_lowest(sh->G, sh->Q, n, &sh->theta, sh->y, sh->ev, sh->perm);
      for (int i = lane; i < 256; i += 64) S->Q[i] = sh->Q[i];
      if (lane < n) {
        S->ev[lane] = sh->ev[lane];
        S->perm[lane] = sh->perm[lane];
      }
      pn = 0;
      for (int j = 1; j < n; ++j)
        if (fabs(sh->y[j]) > fabs(sh->y[pn])) pn = j;
    }
    if (lane < n) S->y[lane] = sh->y[lane];
    if (lane == 0) {
      S->theta = sh->theta;
      S->plarge = pn;
      S->restart = restart;
      S->keep = mmax / 2 < kKeep ? mmax / 2 : kKeep;
      S->iters += 1;
    }
  }
  __syncthreads();
}

// Residual test on the partials of op_passA: decides the action (continue,
// done, switch to the FP64 stage, out of iterations, evicted).  Without a
// direction left the FP32 stage passes on to the FP64 one, and that one ends.
// Where the
// iteration continues through a thick restart, the kept Ritz vectors become
// the basis (pass B writes them): their Ritz values are the diagonal of G, and
// cf is re-expressed in them.
__device__ inline void small_A(DavState* S, const double* part, int nblk, double tol32, double tol64, int max_iter,
                               int evict, double* v, double* red) {
  const int m = S->m;
  reduce_parts(part, nblk, m + 3, v, red);
  if (threadIdx.x >= 64) return;
  const double resid = sqrt(v[0]);
  const double tol = S->phase == 32 ? tol32 : tol64;
  int action = kActContinue, status = 0;
  if (evict) {
    action = kActEvicted;
    status = IFCI_INC_EVICTED;
  } else if (resid <= tol || (S->exhausted && S->phase == 32)) {
    if (S->phase == 32) {
      action = (S->iters >= max_iter) ? kActMaxIter : kActSwitch;
    } else {
      action = kActDone;
      status = IFCI_INC_DONE;
    }
  } else if (S->iters >= max_iter || S->exhausted) {
    action = kActMaxIter;
  }
  const bool restart = action == kActContinue && S->restart;
  const int keep = S->keep, j = threadIdx.x;
  if (j < 16) {
    double c = j <= m ? v[2 + j] : 0.0;
    if (restart) {
      c = 0.0;
      if (j < keep)
        for (int l = 0; l <= m; ++l) c += S->Q[l * 16 + S->perm[j]] * v[2 + l];
      S->y[j] = j == 0 ? 1.0 : 0.0;
    }
    S->cf[j] = c;
  }
  if (restart)
    for (int i = j; i < 256; i += 64) S->G[i] = ((i >> 4) == (i & 15) && (i & 15) < keep) ? S->ev[i & 15] : 0.0;
  if (j == 0) {
    S->resid = resid;
    S->tt0 = v[1];
    S->mb = restart ? keep - 1 : m;
    if (restart) S->plarge = 0;
    if (status) S->status = status;
    S->action = action;
  }
}

// Norm of the correction after the first pass, and whether a second one is
// due: it is when less than half of the squared norm is left, and the squared
// norm after it is |t|^2 - |V^T t|^2 (V orthonormal).  The second pass takes
// away rounding of the first: where it would take most of what is left, the
// correction lay in the span of the basis, no digit of the difference is sure,
// and there is no direction to go on with.
__device__ inline void small_B(DavState* S, const double* part, int nblk, double* v, double* red) {
  const int mb = S->mb;
  reduce_parts(part, nblk, mb + 2, v, red);
  if (threadIdx.x == 0) {
    double tt = v[0];
    const bool reorth = tt < 0.5 * S->tt0;
    if (reorth)
      for (int j = 0; j <= mb; ++j) tt -= v[1 + j] * v[1 + j];
    const bool exhausted = !(tt > (reorth ? 0.1 * v[0] : 0.0));
    for (int j = 0; j < 16; ++j) S->c2[j] = (j <= mb) ? v[1 + j] : 0.0;
    S->reorth = reorth && !exhausted;
    S->tt = tt;
    S->inv = exhausted ? 0.0 : 1.0 / sqrt(tt);
    S->m = mb + 1;
    S->fresh = 0;
    S->exhausted = exhausted;
  }
}

}  // namespace ifci
