// Heat-bath selected CI with a second-order Epstein-Nesbet correction for
// one increment (paper, Methods, iFCI subsection, the HBCI paragraph: the
// paper's increment solver; the method of Holmes, Tubman and Umrigar,
// J. Chem. Theory Comput. 12, 3674 (2016)).
//
// Determinants are 64-bit keys over the increment's k active orbitals: bit
// p is orbital p with spin alpha, bit 32 + p the same orbital with spin beta.
// The core's operators stand first, then alpha, then beta, each ascending, so
// the matrix elements are those of the active Hamiltonian
//   sum_pq h'_pq E_pq + 1/2 sum_pqrs (pq|rs) (E_pq E_rs - delta_qr E_ps)
// with h' the frozen-core one-electron operator (Slater-Condon rules in that
// determinant convention); the constant E_core + e_const is added only to the
// energies handed back.
//
// Device data, all in the caller's work buffer:
//  * the variational space V of a solve: keys in insertion order, and one bit
//    per determinant of the increment's full space (the reference is a closed
//    shell and every replacement keeps both electron counts, so a key is a pair
//    of string ranks: 20.7 MB of bits at 16 orbitals) with the count of bits
//    before each word.  Membership is one bit test, and the count is a
//    determinant's place in key order, the order of the full vectors and of
//    H's columns;
//  * H over V without its diagonal as CSR, one row per flip pair, extended
//    after every selection;
//  * the Davidson basis and sigma vectors, over flip pairs;
//  * the PT2 external space: a hash table key -> N_a (linear probing,
//    MurmurHash3's 64-bit finaliser);
//  * a caller's list of keys (the single steps, for checking them) in a hash
//    table key -> index: its keys may be of any electron count.
// Kernels that walk the excitations of a determinant give it one wavefront;
// the lanes share its occupied/empty orbital lists in LDS and stride over
// the flat list of its single and double replacements.  The integrals sit
// in LDS: h' (k x k) and (pq|rs) packed over pairs of orbital pairs (at
// most 9316 doubles for k = 16).
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "hbci_davidson.hpp"
#include "launch.hpp"

namespace ifci {

void set_error(const std::string& msg);

namespace {

constexpr uint64_t kEmpty = ~0ull;
constexpr int kNB = 512;        // workgroups of the vector kernels
// Waves per workgroup of the kernels that hold the integrals in LDS: at 16
// orbitals (80 KB) two workgroups fit a CU, so 16 waves each, of at most 64
// VGPRs, keep 32 waves in flight per CU.
constexpr int kWaves = 16;
enum : unsigned { kFlagDetCap = 1u, kFlagExtCap = 2u, kFlagDuplicate = 4u, kFlagNoPartner = 8u };

struct HbciCtl {
  unsigned long long n_det;  // keys in V
  unsigned long long n_ext;  // keys in the external table
  unsigned int flags;
  unsigned int pad;
  double e_core;
  long long nnz;
  unsigned long long n_rep;  // flip pairs and flip-invariant keys of V
};

__device__ __forceinline__ uint64_t hmix(uint64_t x) {
  x ^= x >> 33;
  x *= 0xff51afd7ed558ccdull;
  x ^= x >> 33;
  x *= 0xc4ceb9fe1a85ec53ull;
  x ^= x >> 33;
  return x;
}

__host__ __device__ __forceinline__ int tri2(int a, int b) { return a >= b ? (a * (a + 1) >> 1) + b : (b * (b + 1) >> 1) + a; }

__device__ __forceinline__ double G(const double* g, int p, int q, int r, int s) {
  return g[tri2(tri2(p, q), tri2(r, s))];
}

// (-1)^(occupied orbitals of s strictly between x and y)
__device__ __forceinline__ double phase(uint32_t s, int x, int y) {
  const int lo = x < y ? x : y, hi = x < y ? y : x;
  const uint32_t m = ((1u << hi) - 1u) & ~((2u << lo) - 1u);
  return (__popc(s & m) & 1) ? -1.0 : 1.0;
}

__host__ __device__ __forceinline__ uint64_t flip_key(uint64_t key) { return (key >> 32) | (key << 32); }

// A flip pair's representative: the smaller of a key and its partner.  In
// the solve path vectors are flip-symmetric (c_a = c_flip(a), and H commutes
// with the flip), so only representatives are walked: a row of H, a
// selection source or a PT2 source stands for its partner too.
__device__ __forceinline__ bool canonical(uint64_t key) { return key <= flip_key(key); }

// ---------------------------------------------------------------- hash tables

__device__ __forceinline__ int32_t ht_find(const uint64_t* keys, const int32_t* vals, uint64_t mask, uint64_t key) {
  uint64_t h = hmix(key) & mask;
  for (uint64_t n = 0; n <= mask; ++n) {
    const uint64_t kk = keys[h];
    if (kk == key) return vals[h];
    if (kk == kEmpty) return -1;
    h = (h + 1) & mask;
  }
  return -1;
}

// Slot of key, inserting it when absent (*fresh then true); -1 when the
// probe went round the whole table.  A plain load may still see EMPTY where
// another wave has just claimed the slot; the compare-and-swap settles it.
__device__ __forceinline__ int64_t ht_insert(uint64_t* keys, uint64_t mask, uint64_t key, bool* fresh) {
  uint64_t h = hmix(key) & mask;
  for (uint64_t n = 0; n <= mask; ++n) {
    uint64_t kk = keys[h];
    if (kk == kEmpty)
      kk = atomicCAS((unsigned long long*)(keys + h), (unsigned long long)kEmpty, (unsigned long long)key);
    if (kk == kEmpty) {
      *fresh = true;
      return (int64_t)h;
    }
    if (kk == key) {
      *fresh = false;
      return (int64_t)h;
    }
    h = (h + 1) & mask;
  }
  return -1;
}

struct Space {
  uint64_t* dets;
  uint64_t* keys;
  int32_t* vals;
  uint64_t mask;
  int64_t cap;
  HbciCtl* ctl;
};

__device__ __forceinline__ bool has_det(const Space& V, uint64_t key) {
  return ht_find(V.keys, V.vals, V.mask, key) >= 0;
}

__device__ __forceinline__ void add_det(const Space& V, uint64_t key) {
  bool fresh = false;
  const int64_t h = ht_insert(V.keys, V.mask, key, &fresh);
  if (h < 0) {
    atomicOr(&V.ctl->flags, kFlagDetCap);
    return;
  }
  if (!fresh) return;
  const unsigned long long idx = atomicAdd(&V.ctl->n_det, 1ull);
  if ((int64_t)idx < V.cap) {
    V.dets[idx] = key;
    V.vals[h] = (int32_t)idx;
  } else {
    V.vals[h] = -1;
    atomicOr(&V.ctl->flags, kFlagDetCap);
  }
}

// V of a solve as bits over pairs of string ranks: row ra holds the strings
// rb of the other spin in W words, pre[word] counts the bits before it.
struct Bits {
  uint64_t* w;
  int32_t* pre;
  const uint16_t* rank;  // string -> its rank among those of its electron count, in numeric order
  const uint16_t* str;   // rank -> string
  int W, n_str;
  uint64_t* dets;
  int64_t cap;
  HbciCtl* ctl;
};

__device__ __forceinline__ bool has_pair(const Bits& V, int ra, int rb) {
  return V.w[ra * V.W + (rb >> 6)] >> (rb & 63) & 1ull;
}

// place of the pair in key order, -1 when it is not in V
__device__ __forceinline__ int32_t place_of(const Bits& V, int ra, int rb) {
  const int i = ra * V.W + (rb >> 6);
  const uint64_t w = V.w[i], bit = 1ull << (rb & 63);
  return w & bit ? V.pre[i] + __popcll(w & (bit - 1ull)) : -1;
}

__device__ __forceinline__ bool has_det(const Bits& V, uint64_t key) {
  return has_pair(V, V.rank[(uint32_t)key], V.rank[(uint32_t)(key >> 32)]);
}

__device__ __forceinline__ void add_det(const Bits& V, uint64_t key) {
  const int ra = V.rank[(uint32_t)key], rb = V.rank[(uint32_t)(key >> 32)];
  unsigned long long* w = (unsigned long long*)(V.w + ra * V.W + (rb >> 6));
  const unsigned long long bit = 1ull << (rb & 63);
  if ((*w & bit) || (atomicOr(w, bit) & bit)) return;
  const unsigned long long idx = atomicAdd(&V.ctl->n_det, 1ull);
  if ((int64_t)idx < V.cap)
    V.dets[idx] = key;
  else
    atomicOr(&V.ctl->flags, kFlagDetCap);
}

// A slot of the external table: the key and its N_a side by side, so that a
// probe and the atomic update that follows touch one cache line.
struct alignas(16) ExtSlot {
  uint64_t key;
  double val;
};

// (each slot taken is listed in elist, so that the final sum visits the
// filled slots only)
__device__ __forceinline__ void ext_add(ExtSlot* et, int64_t* elist, uint64_t emask, int64_t cap, uint64_t key,
                                        double v, HbciCtl* ctl) {
  uint64_t h = hmix(key) & emask;
  for (uint64_t n = 0; n <= emask; ++n) {
    uint64_t kk = et[h].key;
    if (kk == kEmpty) {
      kk = atomicCAS((unsigned long long*)&et[h].key, (unsigned long long)kEmpty, (unsigned long long)key);
      if (kk == kEmpty) {
        const int64_t at = (int64_t)atomicAdd(&ctl->n_ext, 1ull);
        if (at < cap)
          elist[at] = (int64_t)h;
        else
          atomicOr(&ctl->flags, kFlagExtCap);
        atomicAdd(&et[h].val, v);
        return;
      }
    }
    if (kk == key) {
      atomicAdd(&et[h].val, v);
      return;
    }
    h = (h + 1) & emask;
  }
  atomicOr(&ctl->flags, kFlagExtCap);
}

// ------------------------------------------------------ integrals in LDS

struct Lds {
  double* h1;      // [k][k]
  double* g;       // packed (pq|rs)
  uint8_t* lo;     // pair decode: u = hi (hi - 1) / 2 + lo, lo < hi < 16
  uint8_t* hi;
  float* bound;    // kernels that screen: largest |(rp|wq)|, w != q, of each pair rp; then the two below
  double b_single, b_same;  // largest |H| over single and same-spin double replacements
  uint8_t* lists;  // per wave: occupied then empty orbitals of either spin (16 each), then kWaveBytes for the kernel
};

__host__ __device__ inline int packed_count(int k) {
  const int np = k * (k + 1) / 2;
  return np * (np + 1) / 2;
}

// integral buffer: h', packed (pq|rs), the pair bounds, the two other bounds
__host__ __device__ inline int bounds_at(int k) { return k * k + packed_count(k); }
__host__ __device__ inline int ints_count(int k) { return bounds_at(k) + k * (k + 1) / 2 + 2; }

// Bytes of a wave's lists: 32 of orbitals, and the string ranks of its 64
// single replacements of either spin (rows of H) or their orbital pairs (steps
// that screen).  At 16 orbitals both sizes leave two workgroups to a CU.
constexpr int kListRanks = 32 + 256, kListPairs = 32 + 128;

__host__ inline int lds_bytes_for(int k, int list, bool screen) {
  return (k * k + packed_count(k)) * 8 + 256 + (screen ? (k * (k + 1) / 2 + 3) / 4 * 16 : 0) + kWaves * list;
}

template <bool SCREEN = false>
__device__ Lds load_lds(const double* ints, int k) {
  extern __shared__ __align__(16) unsigned char smem[];
  Lds s;
  const int nint = k * k + packed_count(k), np = k * (k + 1) / 2;
  s.h1 = (double*)smem;
  s.g = s.h1 + k * k;
  s.lo = smem + nint * 8;
  s.hi = s.lo + 128;
  s.bound = (float*)(s.lo + 256);
  s.lists = s.lo + 256 + (SCREEN ? (np + 3) / 4 * 16 : 0);
  for (int t = threadIdx.x; t < nint; t += blockDim.x) s.h1[t] = ints[t];
  for (int t = threadIdx.x; t < 120; t += blockDim.x) {
    int j = 1;
    while ((j + 1) * j / 2 <= t) ++j;
    s.lo[t] = (uint8_t)(t - j * (j - 1) / 2);
    s.hi[t] = (uint8_t)j;
  }
  if (SCREEN) {
    const double* b = ints + bounds_at(k);
    for (int t = threadIdx.x; t < np; t += blockDim.x) s.bound[t] = __double2float_ru(b[t]);
    s.b_single = b[np];
    s.b_same = b[np + 1];
  }
  __syncthreads();
  return s;
}

// --------------------------------------------------------- matrix elements

__device__ double diag_val(const Lds& s, int k, uint32_t A, uint32_t B) {
  double e = 0.0;
  for (uint32_t m = A; m; m &= m - 1) {
    const int p = __builtin_ctz(m);
    e += s.h1[p * k + p];
    for (uint32_t n = A; n; n &= n - 1) {
      const int q = __builtin_ctz(n);
      e += 0.5 * (G(s.g, p, p, q, q) - G(s.g, p, q, q, p));
    }
    for (uint32_t n = B; n; n &= n - 1) e += G(s.g, p, p, __builtin_ctz(n), __builtin_ctz(n));
  }
  for (uint32_t m = B; m; m &= m - 1) {
    const int p = __builtin_ctz(m);
    e += s.h1[p * k + p];
    for (uint32_t n = B; n; n &= n - 1) {
      const int q = __builtin_ctz(n);
      e += 0.5 * (G(s.g, p, p, q, q) - G(s.g, p, q, q, p));
    }
  }
  return e;
}

// <D'|H|D> for D' = a+_r a_p D within string S (the other string O)
__device__ double single_val(const Lds& s, int k, uint32_t S, uint32_t O, int p, int r) {
  double v = s.h1[r * k + p];
  for (uint32_t m = S; m; m &= m - 1) {
    const int q = __builtin_ctz(m);
    v += G(s.g, r, p, q, q) - G(s.g, r, q, q, p);
  }
  for (uint32_t m = O; m; m &= m - 1) {
    const int q = __builtin_ctz(m);
    v += G(s.g, r, p, q, q);
  }
  return phase(S, p, r) * v;
}

// D' = a+_r a+_s a_q a_p D = a+_r a_p (a+_s a_q D) within one string S:
// <D'|H|D> = sign ((rp|sq) - (rq|sp))
__device__ __forceinline__ double double_same(const double* g, uint32_t S, int p, int q, int r, int s) {
  const uint32_t S1 = S ^ (1u << q) ^ (1u << s);
  return phase(S, q, s) * phase(S1, p, r) * (G(g, r, p, s, q) - G(g, r, q, s, p));
}

// A determinant's replacements, one flat index t over: alpha singles, beta
// singles, alpha-alpha doubles, beta-beta doubles, alpha-beta doubles.
struct Det {
  uint32_t A, B;
  int na, nb, va, vb, ca2, cb2;
  int sa, sb, daa, dbb, total;
  const uint8_t *oa, *ea, *ob, *eb;  // occupied and empty orbitals
};

__device__ __forceinline__ Det make_det(uint64_t key, int k, uint8_t* L, int lane) {
  Det d;
  d.A = (uint32_t)key;
  d.B = (uint32_t)(key >> 32);
  const uint32_t all = (1u << k) - 1u;
  __builtin_amdgcn_wave_barrier();
  if (lane < k) {
    const int below = __popc(d.A & ((1u << lane) - 1u));
    L[d.A >> lane & 1u ? below : __popc(d.A & all) + lane - below] = (uint8_t)lane;
  } else if (lane >= 32 && lane < 32 + k) {
    const int p = lane - 32;
    const int below = __popc(d.B & ((1u << p) - 1u));
    L[16 + (d.B >> p & 1u ? below : __popc(d.B & all) + p - below)] = (uint8_t)p;
  }
  __builtin_amdgcn_wave_barrier();
  d.na = __popc(d.A);
  d.nb = __popc(d.B);
  d.oa = L;
  d.ea = L + d.na;
  d.ob = L + 16;
  d.eb = L + 16 + d.nb;
  d.va = k - d.na;
  d.vb = k - d.nb;
  d.ca2 = d.va * (d.va - 1) / 2;
  d.cb2 = d.vb * (d.vb - 1) / 2;
  d.sa = d.na * d.va;
  d.sb = d.nb * d.vb;
  d.daa = d.na * (d.na - 1) / 2 * d.ca2;
  d.dbb = d.nb * (d.nb - 1) / 2 * d.cb2;
  d.total = d.sa + d.sb + d.daa + d.dbb + d.sa * d.sb;
  return d;
}

// Target key of replacement t; its matrix element into *val when VAL.
template <bool VAL>
__device__ __forceinline__ uint64_t replacement(const Det& d, int t, const Lds& s, int k, double* val) {
  uint32_t A = d.A, B = d.B;
  if (t < d.sa) {
    const int p = d.oa[t / d.va], r = d.ea[t % d.va];
    A ^= (1u << p) | (1u << r);
    if (VAL) *val = single_val(s, k, d.A, d.B, p, r);
  } else if ((t -= d.sa) < d.sb) {
    const int p = d.ob[t / d.vb], r = d.eb[t % d.vb];
    B ^= (1u << p) | (1u << r);
    if (VAL) *val = single_val(s, k, d.B, d.A, p, r);
  } else if ((t -= d.sb) < d.daa) {
    const int u = t / d.ca2, v = t - u * d.ca2;
    const int p = d.oa[s.lo[u]], q = d.oa[s.hi[u]], r = d.ea[s.lo[v]], w = d.ea[s.hi[v]];
    A ^= (1u << p) | (1u << q) | (1u << r) | (1u << w);
    if (VAL) *val = double_same(s.g, d.A, p, q, r, w);
  } else if ((t -= d.daa) < d.dbb) {
    const int u = t / d.cb2, v = t - u * d.cb2;
    const int p = d.ob[s.lo[u]], q = d.ob[s.hi[u]], r = d.eb[s.lo[v]], w = d.eb[s.hi[v]];
    B ^= (1u << p) | (1u << q) | (1u << r) | (1u << w);
    if (VAL) *val = double_same(s.g, d.B, p, q, r, w);
  } else {
    t -= d.dbb;
    const int u = t / d.sb, v = t - u * d.sb;
    const int p = d.oa[u / d.va], r = d.ea[u % d.va];
    const int q = d.ob[v / d.vb], w = d.eb[v % d.vb];
    A ^= (1u << p) | (1u << r);
    B ^= (1u << q) | (1u << w);
    if (VAL) *val = phase(d.A, p, r) * phase(d.B, q, w) * G(s.g, r, p, w, q);
  }
  return (uint64_t)A | ((uint64_t)B << 32);
}

// The string ranks of d's 64 or fewer single replacements of either spin, in
// the order of the flat list (k <= 16: at most 8 * 8), after its orbital lists.
struct Ranks {
  const uint16_t *a, *b;
  int ra, rb;
};

__device__ __forceinline__ Ranks make_ranks(const Det& d, const uint16_t* rank, uint8_t* L, int lane) {
  uint16_t* R = (uint16_t*)(L + 32);
  if (lane < d.sa) R[lane] = rank[d.A ^ (1u << d.oa[lane / d.va]) ^ (1u << d.ea[lane % d.va])];
  if (lane < d.sb) R[64 + lane] = rank[d.B ^ (1u << d.ob[lane / d.vb]) ^ (1u << d.eb[lane % d.vb])];
  __builtin_amdgcn_wave_barrier();
  return Ranks{R, R + 64, rank[d.A], rank[d.B]};
}

// Ranks of replacement t's strings.
__device__ __forceinline__ void replaced_ranks(const Det& d, const Ranks& R, int t, const Lds& s, const uint16_t* rank,
                                               float inv_sb, int* ra, int* rb) {
  const int doubles = d.sa + d.sb + d.daa + d.dbb;
  *ra = R.ra;
  *rb = R.rb;
  if (t >= doubles) {
    t -= doubles;
    const int u = (int)((t + 0.5f) * inv_sb);  // t / sb: both below 2^12, off by less than 0.5 / 64
    *ra = R.a[u];
    *rb = R.b[t - u * d.sb];
  } else if (t < d.sa) {
    *ra = R.a[t];
  } else if (t < d.sa + d.sb) {
    *rb = R.b[t - d.sa];
  } else {
    double v;
    const uint64_t key = replacement<false>(d, t, s, 0, &v);
    if (t < d.sa + d.sb + d.daa)
      *ra = rank[(uint32_t)key];
    else
      *rb = rank[(uint32_t)(key >> 32)];
  }
}

// The replacements of d that can pass |H_ai c_i| > eps, by the bounds on H:
// the single ones, the same-spin doubles, and the alpha-beta doubles of those
// single replacements of either spin whose orbital pair has an integral large
// enough.  (All bounds hold in floating point too: rounding is monotone, and
// the sums of a single replacement are given a margin.  A NaN among the
// integrals makes the bound of the single ones NaN, which excludes none; the
// others are largest values, which leave out a NaN, as the test itself does.)
struct Screen {
  int singles, same, na, nb, total;
  const uint8_t *a, *b;  // kept pairs, empty orbital << 4 | occupied
};

__device__ __forceinline__ Screen make_screen(const Det& d, const Lds& s, double c, double eps, uint8_t* L, int lane) {
  Screen S;
  const double ac = fabs(c);
  S.singles = s.b_single * ac <= eps ? 0 : d.sa + d.sb;
  S.same = s.b_same * ac > eps ? d.daa + d.dbb : 0;
  uint8_t* P = L + 32;
  const uint64_t below = (1ull << lane) - 1ull;
  auto keep = [&](int n, int nv, const uint8_t* occ, const uint8_t* emp, uint8_t* out) {
    int p = 0, r = 0;
    bool k = false;
    if (lane < n) {
      p = occ[lane / nv];
      r = emp[lane % nv];
      k = (double)s.bound[tri2(p, r)] * ac > eps;
    }
    const uint64_t m = __ballot(k);
    if (k) out[__popcll(m & below)] = (uint8_t)(r << 4 | p);
    return (int)__popcll(m);
  };
  S.na = keep(d.sa, d.va, d.oa, d.ea, P);
  S.nb = keep(d.sb, d.vb, d.ob, d.eb, P + 64);
  S.a = P;
  S.b = P + 64;
  S.total = S.singles + S.same + S.na * S.nb;
  __builtin_amdgcn_wave_barrier();
  return S;
}

// Target key and matrix element of the screened list's entry t.
__device__ __forceinline__ uint64_t screened(const Det& d, const Screen& S, int t, const Lds& s, int k, float inv_nb,
                                             double* val) {
  if (t < S.singles) return replacement<true>(d, t, s, k, val);
  t -= S.singles;
  if (t < S.same) return replacement<true>(d, d.sa + d.sb + t, s, k, val);
  t -= S.same;
  const int u = (int)((t + 0.5f) * inv_nb);
  const int x = S.a[u], y = S.b[t - u * S.nb];
  const int p = x & 15, r = x >> 4, q = y & 15, w = y >> 4;
  *val = phase(d.A, p, r) * phase(d.B, q, w) * G(s.g, r, p, w, q);
  return (uint64_t)(d.A ^ (1u << p) ^ (1u << r)) | ((uint64_t)(d.B ^ (1u << q) ^ (1u << w)) << 32);
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------ kernels

// h' and the packed (pq|rs) of the active orbitals, and the core energy.
__global__ void hbci_prep_kernel(const double* __restrict__ h, const double* __restrict__ eri, int n,
                                 const int32_t* __restrict__ act, int k, const int32_t* __restrict__ core, int nc,
                                 const double* __restrict__ e_core, double* __restrict__ ints, HbciCtl* ctl) {
  auto E4 = [&](int p, int q, int r, int s) { return eri[(((int64_t)p * n + q) * n + r) * n + s]; };
  for (int t = threadIdx.x; t < k * k; t += blockDim.x) {
    const int p = act[t / k], q = act[t % k];
    double v = h[(int64_t)p * n + q];
    for (int c = 0; c < nc; ++c) v += 2.0 * E4(p, q, core[c], core[c]) - E4(p, core[c], core[c], q);
    ints[t] = v;
  }
  const int npp = packed_count(k);
  for (int t = threadIdx.x; t < npp; t += blockDim.x) {
    int P = 0;
    while ((P + 1) * (P + 2) / 2 <= t) ++P;
    const int Q = t - P * (P + 1) / 2;
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= P) ++i;
    const int j = P - i * (i + 1) / 2;
    int a = 0;
    while ((a + 1) * (a + 2) / 2 <= Q) ++a;
    const int b = Q - a * (a + 1) / 2;
    ints[k * k + t] = E4(act[i], act[j], act[a], act[b]);
  }
  if (threadIdx.x == 0) {
    ctl->n_det = 0;
    ctl->n_ext = 0;
    ctl->flags = 0;
    ctl->e_core = *e_core;
    ctl->nnz = 0;
    ctl->n_rep = 0;
  }
}

// The bounds on H of make_screen, one workgroup of 1024 threads: a thread per
// orbital pair and third orbital, its share of the pair's bounds in LDS.  (A
// thread per pair, at the end of the kernel above, took 20 us at 10 orbitals and
// 70 at 14.)
__global__ void __launch_bounds__(1024) hbci_bounds_kernel(double* __restrict__ ints, int k) {
  constexpr int kMaxPair = kMaxAct * (kMaxAct + 1) / 2, kMaxUp = kMaxAct * (kMaxAct - 1) / 2;
  __shared__ double large[kMaxPair * kMaxAct], one[kMaxPair * kMaxAct];
  __shared__ uint8_t pi[kMaxPair], pj[kMaxPair], up[kMaxUp], uq[kMaxUp];
  __shared__ unsigned long long top[2];  // non-negative doubles order as their bits
  const double* h1 = ints;
  const double* g = ints + k * k;
  double* bound = ints + bounds_at(k);
  const int np = k * (k + 1) / 2, nd = k * (k - 1) / 2, tid = threadIdx.x;
  if (tid < 2) top[tid] = 0ull;
  if (tid < np) {
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= tid) ++i;
    pi[tid] = (uint8_t)i;
    pj[tid] = (uint8_t)(tid - i * (i + 1) / 2);
  } else if (tid >= 512 && tid - 512 < nd) {
    int p = 1;
    while ((p + 1) * p / 2 <= tid - 512) ++p;
    up[tid - 512] = (uint8_t)p;
    uq[tid - 512] = (uint8_t)(tid - 512 - p * (p - 1) / 2);
  }
  __syncthreads();
  for (int t = tid; t < np * k; t += 1024) {
    const int u = t / k, w = t - u * k, i = pi[u], j = pj[u];
    double m = 0.0;
    for (int q = 0; q < w; ++q) m = fmax(m, fabs(G(g, i, j, w, q)));
    large[t] = m;
    one[t] = 2.0 * fabs(G(g, i, j, w, w)) + fabs(G(g, i, w, w, j));
  }
  double same = 0.0;
  for (int t = tid; t < nd * nd; t += 1024) {
    const int u = t / nd, v = t - u * nd, p = up[u], q = uq[u], r = up[v], w = uq[v];
    same = fmax(same, fabs(G(g, r, p, w, q) - G(g, r, q, w, p)));
  }
  atomicMax(&top[1], (unsigned long long)__double_as_longlong(same));
  __syncthreads();
  if (tid < np) {
    double m = 0.0, s = fabs(h1[pi[tid] * k + pj[tid]]);
    for (int w = 0; w < k; ++w) {
      m = fmax(m, large[tid * k + w]);
      s += one[tid * k + w];
    }
    bound[tid] = m;
    atomicMax(&top[0], (unsigned long long)__double_as_longlong(s * (1.0 + 1e-12)));
  }
  __syncthreads();
  if (tid < 2) bound[np + tid] = __longlong_as_double((long long)top[tid]);
}

__global__ void fill_u64_kernel(uint64_t* p, int64_t n, uint64_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void fill_slots_kernel(ExtSlot* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = ExtSlot{kEmpty, 0.0};
}

__global__ void fill_f64_kernel(double* p, int64_t n, double v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// rank[s] of every string of the reference's electron count, and the string of every rank
__global__ void hbci_rank_kernel(int k, int na, uint16_t* __restrict__ rank, uint16_t* __restrict__ str) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= 1 << k || __popc(s) != na) return;
  int r = 0, i = 0;
  for (int m = s; m; m &= m - 1) {
    const int p = __builtin_ctz(m);
    int b = 1;  // p over ++i
    ++i;
    for (int j = 0; j < i; ++j) b = b * (p - j) / (j + 1);
    r += b;
  }
  rank[s] = (uint16_t)r;
  str[r] = (uint16_t)s;
}

// V := the reference (a closed shell)
__global__ void hbci_ref_kernel(uint64_t ref, Bits V) { add_det(V, ref); }

// V := the caller's keys, in order.
__global__ void hbci_load_kernel(const uint64_t* __restrict__ in, int64_t n, Space V) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t key = in[i];
    V.dets[i] = key;
    bool fresh = false;
    const int64_t h = ht_insert(V.keys, V.mask, key, &fresh);
    if (h < 0)
      atomicOr(&V.ctl->flags, kFlagDetCap);
    else if (!fresh)
      atomicOr(&V.ctl->flags, kFlagDuplicate);
    else
      V.vals[h] = (int32_t)i;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) V.ctl->n_det = (unsigned long long)n;
}

// Bits before each word, bits before each row's first flip pair, in three
// passes: rows counted (one wave each), row counts summed, words summed.
__global__ void __launch_bounds__(256) hbci_row_count_kernel(Bits V, int32_t* __restrict__ cnt) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= V.n_str) return;
  int all = 0, rep = 0;
  for (int i = lane; i < V.W; i += 64) {
    const uint64_t w = V.w[r * V.W + i];
    all += __popcll(w);
    // representatives: the strings up to r
    const int left = r + 1 - i * 64;
    rep += left >= 64 ? __popcll(w) : left > 0 ? __popcll(w & ((1ull << left) - 1ull)) : 0;
  }
  all = wave_sum_int(all);
  rep = wave_sum_int(rep);
  if (lane == 0) {
    cnt[r] = all;
    cnt[V.n_str + r] = rep;
  }
}

__global__ void __launch_bounds__(1024) hbci_row_scan_kernel(int n_str, int32_t* __restrict__ cnt, HbciCtl* ctl) {
  __shared__ int sh[1024];
  for (int half = 0; half < 2; ++half) {
    int32_t* c = cnt + half * n_str;
    const int per = (n_str + 1023) / 1024, lo = threadIdx.x * per, hi = lo + per < n_str ? lo + per : n_str;
    int own = 0;
    for (int i = lo; i < hi; ++i) own += c[i];
    sh[threadIdx.x] = own;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int v = threadIdx.x >= (unsigned)o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += v;
      __syncthreads();
    }
    int at = sh[threadIdx.x] - own;
    for (int i = lo; i < hi; ++i) {
      const int v = c[i];
      c[i] = at;
      at += v;
    }
    if (half && threadIdx.x == 1023) ctl->n_rep = (unsigned long long)sh[1023];
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) hbci_word_scan_kernel(Bits V, const int32_t* __restrict__ start) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= V.n_str) return;
  int base = start[r];
  for (int i0 = 0; i0 < V.W; i0 += 64) {
    const int i = i0 + lane;
    const int own = i < V.W ? __popcll(V.w[r * V.W + i]) : 0;
    int sum = own;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(sum, o, 64);
      if (lane >= o) sum += v;
    }
    if (i < V.W) V.pre[r * V.W + i] = base + sum - own;
    base += __shfl(sum, 63, 64);
  }
}

// Per determinant of V, by insertion: its place in key order and its flip
// pair's number, now and (for those before lo) before the selection step.
struct Order {
  int32_t* place;   // by insertion
  int32_t* pair;    // by insertion: flip pair's number
  int32_t* moved;   // old place -> new place
  int32_t* row_of;  // place -> flip pair's number; its complement for keys new in this step
  double* diag_in;  // by insertion
  // by flip pair, for its representative
  uint64_t* key;
  int32_t* pos;
  int32_t* fpos;
  int32_t* old;     // its number before the step, -1 for a new one
  double* diag;
};

// The new order after a selection step, and x (in the old order) moved to it.
__global__ void hbci_order_kernel(Bits V, int64_t lo, int64_t n, const int32_t* __restrict__ start, Order O,
                                  const double* __restrict__ x_old, double* __restrict__ x) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t key = V.dets[i];
    const int ra = V.rank[(uint32_t)key], rb = V.rank[(uint32_t)(key >> 32)];
    const int32_t p = place_of(V, ra, rb), f = place_of(V, rb, ra);
    if (f < 0) {  // V is closed under the flip
      atomicOr(&V.ctl->flags, kFlagNoPartner);
      continue;
    }
    const int32_t q = rb <= ra ? start[V.n_str + ra] + (p - start[ra]) : start[V.n_str + rb] + (f - start[rb]);
    const bool old = i < lo;
    if (rb <= ra) {
      O.key[q] = key;
      O.pos[q] = p;
      O.fpos[q] = f;
      O.old[q] = old ? O.pair[i] : -1;
      O.diag[q] = O.diag_in[i];
    }
    O.row_of[p] = old ? q : ~q;
    if (old) O.moved[O.place[i]] = p;
    x[p] = old ? x_old[O.place[i]] : 0.0;
    O.place[i] = p;
    O.pair[i] = q;
  }
}

// c_out[i] = x at the place of key i
__global__ void hbci_by_insertion_kernel(const int32_t* __restrict__ place, const double* __restrict__ x, int64_t n,
                                         double* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = x[place[i]];
}

// One selection step: every replacement a of a determinant i < n_src with
// |H_ai c_i| > eps joins V, with its flip partner.  src lists the sources and
// pos the places of their c (null: in order); in the solve path, whose
// vectors are flip-symmetric, only representatives are walked.
//
// Bound by the elements of H it forms; most determinants of a converged
// vector can pass the threshold with few of their replacements or none, which
// the bounds of make_screen show before any element is formed.
template <typename VSpace>
__global__ void __launch_bounds__(64 * kWaves, 8) hbci_select_kernel(const double* __restrict__ ints, int k,
                                                                  const uint64_t* __restrict__ src,
                                                                  const int32_t* __restrict__ pos,
                                                                  const double* __restrict__ c, int64_t n_src,
                                                                  double eps, VSpace V) {
  const Lds s = load_lds<true>(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListPairs;
  for (int64_t i = (int64_t)blockIdx.x * kWaves + wave; i < n_src; i += (int64_t)gridDim.x * kWaves) {
    const double ci = c[pos ? pos[i] : i];
    if (ci == 0.0) continue;
    const Det d = make_det(src[i], k, L, lane);
    const Screen S = make_screen(d, s, ci, eps, L, lane);
    const float inv_nb = 1.0f / (float)S.nb;
    for (int t = lane; t < S.total; t += 64) {
      double v;
      const uint64_t a = screened(d, S, t, s, k, inv_nb, &v);
      if (fabs(v * ci) > eps) {
        add_det(V, a);
        if (flip_key(a) != a) add_det(V, flip_key(a));
      }
    }
  }
}

// The diagonal of rows lo..n-1.
__global__ void __launch_bounds__(64 * kWaves) hbci_diag_kernel(const double* __restrict__ ints, int k,
                                                                const uint64_t* __restrict__ dets, int64_t lo,
                                                                int64_t n, double* __restrict__ diag) {
  const Lds s = load_lds(ints, k);
  for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    diag[i] = diag_val(s, k, (uint32_t)dets[i], (uint32_t)(dets[i] >> 32));
}

// Nonzeros of each row of H over a list of keys (replacements that land in it).
__global__ void __launch_bounds__(64 * kWaves) hbci_count_kernel(const double* __restrict__ ints, int k, const Space V,
                                                                 int64_t n, int32_t* __restrict__ cnt) {
  const Lds s = load_lds(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListRanks;
  for (int64_t a = (int64_t)blockIdx.x * kWaves + wave; a < n; a += (int64_t)gridDim.x * kWaves) {
    const Det d = make_det(V.dets[a], k, L, lane);
    int c = 0;
    for (int t = lane; t < d.total; t += 64) {
      double v;
      const uint64_t key = replacement<false>(d, t, s, k, &v);
      c += ht_find(V.keys, V.vals, V.mask, key) >= 0;
    }
    c = wave_sum_int(c);
    if (lane == 0) cnt[a] = c;
  }
}

// Exclusive prefix sum of cnt[0..n) into ptr[0..n]: blocks of 1024 rows,
// then the block totals, then the carry.
__global__ void __launch_bounds__(1024) scan_block_kernel(const int32_t* __restrict__ cnt, int64_t n,
                                                          int64_t* __restrict__ ptr, int64_t* __restrict__ bsum) {
  __shared__ int64_t sh[1024];
  const int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  sh[threadIdx.x] = i < n ? cnt[i] : 0;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int64_t v = threadIdx.x >= (unsigned)o ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += v;
    __syncthreads();
  }
  if (i < n) ptr[i + 1] = sh[threadIdx.x];
  if (threadIdx.x == 1023) bsum[blockIdx.x] = sh[1023];
}

__global__ void __launch_bounds__(1024) scan_top_kernel(int64_t* __restrict__ bsum, int64_t nb, HbciCtl* ctl) {
  __shared__ int64_t sh[1024];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int64_t own = i < nb ? bsum[i] : 0;
    sh[threadIdx.x] = own;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int64_t v = threadIdx.x >= (unsigned)o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += v;
      __syncthreads();
    }
    if (i < nb) bsum[i] = carry + sh[threadIdx.x] - own;  // exclusive
    __syncthreads();
    if (threadIdx.x == 0) carry += sh[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) ctl->nnz = carry;
}

__global__ void scan_add_kernel(int64_t* __restrict__ ptr, int64_t n, const int64_t* __restrict__ bsum) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) ptr[i + 1] += bsum[i / 1024];
  if (i == 0) ptr[0] = 0;
}

// Column indices and values of each row, in replacement order.
__global__ void __launch_bounds__(64 * kWaves) hbci_fill_kernel(const double* __restrict__ ints, int k, const Space V,
                                                                int64_t n, const int64_t* __restrict__ ptr,
                                                                int32_t* __restrict__ col, double* __restrict__ val) {
  const Lds s = load_lds(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListRanks;
  const uint64_t below = (1ull << lane) - 1ull;
  for (int64_t a = (int64_t)blockIdx.x * kWaves + wave; a < n; a += (int64_t)gridDim.x * kWaves) {
    const Det d = make_det(V.dets[a], k, L, lane);
    int64_t base = ptr[a];
    for (int t0 = 0; t0 < d.total; t0 += 64) {
      const int t = t0 + lane;
      int32_t j = -1;
      double v = 0.0;
      if (t < d.total) {
        const uint64_t key = replacement<false>(d, t, s, k, &v);
        j = ht_find(V.keys, V.vals, V.mask, key);
        if (j >= 0) replacement<true>(d, t, s, k, &v);
      }
      const uint64_t m = __ballot(j >= 0);
      if (j >= 0) {
        const int64_t at = base + __popcll(m & below);
        col[at] = j;
        val[at] = v;
      }
      base += __popcll(m);
    }
  }
}

// Rows of H by flip pair: row q is that of the pair's representative, with
// columns in the full space (places in key order).  After a selection step the
// rows of the pairs it added are formed from scratch, and each of their
// nonzeros (r, b) with b older also gives the entries that it implies in
// the old rows, which H's symmetry and its commuting with the flip fix:
// (b, r) when b is a representative, and (flip b, flip r) when r is not
// flip-invariant and flip b is a representative (for a flip-invariant r that
// entry is (flip b, r), reached from r's own nonzero (r, flip b)).
//
// Bound by the membership tests, 5792 for a row of a half-filled 16-orbital
// space of which one in seven lands in V.  The ranks of a row's single
// replacements are looked up once; an alpha-beta double, five of seven tests,
// is then two LDS reads and one bit, whose words lie on few lines for one
// replacement of the first string.  (Hash probes: count 1.35 ms and fill
// 1.74 ms a step on average at 285020 keys.)
__global__ void __launch_bounds__(64 * kWaves, 8) hbci_count_new_kernel(const double* __restrict__ ints, int k,
                                                                     const Bits V, const Order O, int64_t n_rep,
                                                                     int32_t* __restrict__ cnt,
                                                                     int32_t* __restrict__ addc) {
  const Lds s = load_lds(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListRanks;
  for (int64_t q = (int64_t)blockIdx.x * kWaves + wave; q < n_rep; q += (int64_t)gridDim.x * kWaves) {
    if (O.old[q] >= 0) continue;
    const Det d = make_det(O.key[q], k, L, lane);
    const bool self = d.A == d.B;
    const Ranks R = make_ranks(d, V.rank, L, lane);
    const float inv_sb = 1.0f / (float)d.sb;
    int c = 0;
    for (int t = lane; t < d.total; t += 64) {
      int ra, rb;
      replaced_ranks(d, R, t, s, V.rank, inv_sb, &ra, &rb);
      const int32_t j = place_of(V, ra, rb);
      if (j < 0) continue;
      ++c;
      const int32_t b = O.row_of[j];
      if (b >= 0) {
        const int add = (rb <= ra ? 1 : 0) + (!self && ra <= rb ? 1 : 0);
        if (add) atomicAdd(addc + b, add);
      }
    }
    c = wave_sum_int(c);
    if (lane == 0) cnt[q] = c;
  }
}

// cnt[q] = the old row's length plus its new entries, of the old pairs
__global__ void hbci_rowlen_kernel(const int64_t* __restrict__ ptr_old, const int32_t* __restrict__ old, int64_t n_rep,
                                   const int32_t* __restrict__ addc, int32_t* __restrict__ cnt) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n_rep; q += (int64_t)gridDim.x * blockDim.x) {
    const int32_t o = old[q];
    if (o >= 0) cnt[q] = (int32_t)(ptr_old[o + 1] - ptr_old[o]) + addc[q];
  }
}

// The new rows in full (replacement order) and their implied entries in
// the old rows, after the place of those they have (in no fixed order).  The hits of a row
// are gathered 64 at a time before their elements are formed, so that the
// lanes that form them are full.
__global__ void __launch_bounds__(64 * kWaves, 8) hbci_fill_new_kernel(const double* __restrict__ ints, int k,
                                                                    const Bits V, const Order O, int64_t n_rep,
                                                                    const int64_t* __restrict__ ptr_old,
                                                                    const int64_t* __restrict__ ptr,
                                                                    int32_t* __restrict__ used,
                                                                    int32_t* __restrict__ col,
                                                                    double* __restrict__ val) {
  const Lds s = load_lds(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListRanks;
  const uint64_t below = (1ull << lane) - 1ull;
  for (int64_t q = (int64_t)blockIdx.x * kWaves + wave; q < n_rep; q += (int64_t)gridDim.x * kWaves) {
    if (O.old[q] >= 0) continue;
    const Det d = make_det(O.key[q], k, L, lane);
    const bool self = d.A == d.B;
    const Ranks R = make_ranks(d, V.rank, L, lane);
    const float inv_sb = 1.0f / (float)d.sb;
    const int32_t r = O.pos[q], fr = O.fpos[q];
    int64_t base = ptr[q];
    // lane l holds gathered hit l: its replacement, place and order of ranks
    int have = 0, gt = 0, gj = 0, gs = 0;
    auto flush = [&](int m) {
      if (lane < m) {
        double v;
        replacement<true>(d, gt, s, k, &v);
        col[base + lane] = gj;
        val[base + lane] = v;
        const int32_t b = O.row_of[gj];
        if (b >= 0) {
          const int64_t at = ptr[b] + (ptr_old[O.old[b] + 1] - ptr_old[O.old[b]]);
          if (gs >= 0) {
            const int64_t e = at + atomicAdd(used + b, 1);
            col[e] = r;
            val[e] = v;
          }
          if (!self && gs <= 0) {
            const int64_t e = at + atomicAdd(used + b, 1);
            col[e] = fr;
            val[e] = v;
          }
        }
      }
      base += m;
    };
    for (int t0 = 0; t0 < d.total; t0 += 64) {
      const int t = t0 + lane;
      int32_t j = -1;
      int ra = 0, rb = 0;
      if (t < d.total) {
        replaced_ranks(d, R, t, s, V.rank, inv_sb, &ra, &rb);
        j = place_of(V, ra, rb);
      }
      const uint64_t m = __ballot(j >= 0);
      const int hits = __popcll(m);
      if (hits == 0) continue;
      // hit h goes to lane (have + h) mod 64; where that wraps, the full set is written between.
      // from: the lane that holds the hit for this lane, the src-th set bit of m
      const int sg = ra > rb ? 1 : (ra < rb ? -1 : 0);
      int from = -1, src = (lane - have) & 63;
      if (src < hits) {
        uint64_t mm = m;
        from = 0;
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {
          const int cnt = __popcll(mm & ((1ull << w) - 1ull));
          if (src >= cnt) {
            src -= cnt;
            mm >>= w;
            from += w;
          }
        }
      }
      const int st = __shfl(t, from & 63, 64), sj = __shfl(j, from & 63, 64), ss = __shfl(sg, from & 63, 64);
      const bool early = from >= 0 && lane >= have;  // lands before the set is full
      if (early) {
        gt = st;
        gj = sj;
        gs = ss;
      }
      have += hits;
      if (have >= 64) {
        flush(64);
        have -= 64;
        if (from >= 0 && !early) {
          gt = st;
          gj = sj;
          gs = ss;
        }
      }
    }
    flush(have);
  }
}

// Each row's entries in order of their columns: what the step added is
// sorted (bitonic, in LDS) and merged with the old row, whose columns keep
// their order at the new places.  One workgroup per row of more than LO and at
// most CAP entries.  Bound by reading and writing H once per step; in return
// the products after it find the columns of 64 lanes on few lines.
template <int NT, int LO, int CAP>
__global__ void __launch_bounds__(NT) hbci_merge_rows_kernel(const int64_t* __restrict__ ptr_old,
                                                             const int32_t* __restrict__ col_old,
                                                             const double* __restrict__ val_old,
                                                             const int32_t* __restrict__ old,
                                                             const int32_t* __restrict__ moved, int64_t n_rep,
                                                             const int64_t* __restrict__ ptr_new,
                                                             int32_t* __restrict__ col_new,
                                                             double* __restrict__ val_new) {
  constexpr int kIndex = 13;  // bits of an entry's index, CAP <= 2^13
  extern __shared__ __align__(16) unsigned char smem[];
  uint64_t* key = (uint64_t*)smem;
  int32_t* oc = (int32_t*)(key + CAP);
  const int tid = threadIdx.x;
  for (int64_t q = blockIdx.x; q < n_rep; q += gridDim.x) {
    const int64_t to = ptr_new[q], len = ptr_new[q + 1] - to;
    if (len <= LO || len > CAP) continue;
    const int32_t o = old[q];
    const int64_t b = o < 0 ? 0 : ptr_old[o];
    const int no = o < 0 ? 0 : (int)(ptr_old[o + 1] - b), m = (int)len - no;
    int P = 1;
    while (P < m) P <<= 1;
    for (int e = tid; e < no; e += NT) oc[e] = moved[col_old[b + e]];
    for (int e = tid; e < P; e += NT) key[e] = e < m ? (uint64_t)col_new[to + no + e] << kIndex | (uint64_t)e : ~0ull;
    for (int size = 2; size <= P; size <<= 1)
      for (int half = size >> 1; half > 0; half >>= 1) {
        __syncthreads();
        for (int t = tid; t < P / 2; t += NT) {
          const int i = 2 * t - (t & (half - 1)), j = i + half;
          const uint64_t x = key[i], y = key[j];
          if ((x > y) == ((i & size) == 0)) {
            key[i] = y;
            key[j] = x;
          }
        }
      }
    __syncthreads();
    double v[CAP / NT];
#pragma unroll
    for (int r = 0; r < CAP / NT; ++r) {
      const int e = tid + r * NT;
      if (e < m) v[r] = val_new[to + no + (int)(key[e] & ((1u << kIndex) - 1u))];
    }
    __syncthreads();  // all values are read before any is written
#pragma unroll
    for (int r = 0; r < CAP / NT; ++r) {
      const int e = tid + r * NT;
      if (e < m) {
        const int32_t c = (int32_t)(key[e] >> kIndex);
        int lo = 0, hi = no;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (oc[mid] < c)
            lo = mid + 1;
          else
            hi = mid;
        }
        col_new[to + e + lo] = c;
        val_new[to + e + lo] = v[r];
      }
    }
    for (int e = tid; e < no; e += NT) {
      const int32_t c = oc[e];
      const uint64_t k = (uint64_t)c << kIndex;
      int lo = 0, hi = m;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key[mid] < k)
          lo = mid + 1;
        else
          hi = mid;
      }
      col_new[to + e + lo] = c;
      val_new[to + e + lo] = val_old[b + e];
    }
    __syncthreads();
  }
}

// Rows of up to kShortRow entries take 256 threads and 12 KB of LDS each, up
// to kMidRow twice the LDS, the others (at most 5792 replacements at 16
// orbitals) 1024 threads and 96 KB, one workgroup a CU: that form for all rows
// past kShortRow took 0.90 ms a step on average at 316208 keys.
constexpr int kShortRow = 1024, kMidRow = 2048, kLongRow = 8192;

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// y = H x over a list of keys: the diagonal plus the CSR rows (one wave per row).
__global__ void __launch_bounds__(256) hbci_spmv_kernel(const int64_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                        const double* __restrict__ val, const double* __restrict__ diag,
                                                        const double* __restrict__ x, double* __restrict__ y,
                                                        int64_t n) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t a = (int64_t)blockIdx.x * (blockDim.x >> 6) + wave; a < n; a += nw) {
    double s = 0.0;
    for (int64_t e = ptr[a] + lane; e < ptr[a + 1]; e += 64) s += val[e] * x[col[e]];
    s = wave_sum(s);
    if (lane == 0) y[a] = s + diag[a] * x[a];
  }
}

// N_a += H_ai c_i for every replacement a outside V with |H_ai c_i| > eps.
// With half (flip-symmetric c, flip-closed V) src lists the representatives
// i, at places pos of c, and N is kept for representatives b only: the term (i, b) of a
// non-representative i equals (flip i, flip b), so a representative i adds
// each term to its target's representative (twice for a flip-invariant
// target, which i and flip(i) both reach); a flip-invariant i (a closed
// shell, whose replacements come in flip pairs) adds only the terms whose
// target is a representative.
template <typename VSpace>
__global__ void __launch_bounds__(64 * kWaves, 8) hbci_pt2_kernel(const double* __restrict__ ints, int k, const VSpace V,
                                                               const uint64_t* __restrict__ src,
                                                               const int32_t* __restrict__ pos,
                                                               const double* __restrict__ c, int64_t n, double eps,
                                                               int half, ExtSlot* __restrict__ et,
                                                               int64_t* __restrict__ elist, uint64_t emask,
                                                               int64_t ecap) {
  const Lds s = load_lds<true>(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListPairs;
  for (int64_t i = (int64_t)blockIdx.x * kWaves + wave; i < n; i += (int64_t)gridDim.x * kWaves) {
    const double ci = c[pos ? pos[i] : i];
    if (ci == 0.0) continue;
    const Det d = make_det(src[i], k, L, lane);
    const bool self = d.A == d.B;
    const Screen S = make_screen(d, s, ci, eps, L, lane);
    const float inv_nb = 1.0f / (float)S.nb;
    for (int t = lane; t < S.total; t += 64) {
      double v;
      uint64_t a = screened(d, S, t, s, k, inv_nb, &v);
      const double hc = v * ci;
      if (!(fabs(hc) > eps)) continue;
      double w = 1.0;
      if (half) {
        if (!canonical(a)) {
          if (self) continue;
          a = flip_key(a);
        } else if (!self && flip_key(a) == a) {
          w = 2.0;  // i and flip(i) reach the flip-invariant a with equal terms
        }
      }
      if (!has_det(V, a)) ext_add(et, elist, emask, ecap, a, w * hc, V.ctl);
    }
  }
}

// The external space of a solve as an array over pairs of string ranks
// (representatives ra >= rb), where it fits the room of the hash table: one
// addition that nothing waits for in place of a probe, an addition and, for
// a new key, a place in the list.  The pairs that no term has reached hold
// -0, which no sum of nonzero terms is.
__device__ __forceinline__ bool touched(double v) { return __double_as_longlong(v) != __double_as_longlong(-0.0); }

// hbci_pt2_kernel (half) into that array.  Bound by the additions, 8 bytes
// each at scattered places of 1.3 GB at 16 orbitals; sources in key order keep
// to the rows of the same few first strings.  (Into the hash table, with a
// counter that every new key passes: 33.2 ms at 285020 keys.)
__global__ void __launch_bounds__(64 * kWaves, 8) hbci_pt2_array_kernel(const double* __restrict__ ints, int k,
                                                                        const Bits V, const uint64_t* __restrict__ src,
                                                                        const int32_t* __restrict__ pos,
                                                                        const double* __restrict__ c, int64_t n,
                                                                        double eps, double* __restrict__ N) {
  const Lds s = load_lds<true>(ints, k);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint8_t* L = s.lists + wave * kListPairs;
  for (int64_t i = (int64_t)blockIdx.x * kWaves + wave; i < n; i += (int64_t)gridDim.x * kWaves) {
    const double ci = c[pos[i]];
    if (ci == 0.0) continue;
    const Det d = make_det(src[i], k, L, lane);
    const bool self = d.A == d.B;
    const Screen S = make_screen(d, s, ci, eps, L, lane);
    const float inv_nb = 1.0f / (float)S.nb;
    // lane l: the ranks of the strings of kept pairs l
    auto kept = [&](uint32_t str, int x) { return (int)V.rank[str ^ (1u << (x & 15)) ^ (1u << (x >> 4))]; };
    const int rank_a = lane < S.na ? kept(d.A, S.a[lane]) : 0, rank_b = lane < S.nb ? kept(d.B, S.b[lane]) : 0;
    for (int t0 = 0; t0 < S.total; t0 += 64) {
      const int t = t0 + lane, v = t - S.singles - S.same;
      const int u = v >= 0 && v < S.na * S.nb ? (int)((v + 0.5f) * inv_nb) : 0;
      int ra = __shfl(rank_a, u, 64), rb = __shfl(rank_b, v >= 0 ? (v - u * S.nb) & 63 : 0, 64);
      if (t >= S.total) continue;
      double h;
      const uint64_t a = screened(d, S, t, s, k, inv_nb, &h);
      const double hc = h * ci;
      if (!(fabs(hc) > eps)) continue;
      if (v < 0) {
        ra = V.rank[(uint32_t)a];
        rb = V.rank[(uint32_t)(a >> 32)];
      }
      double w = 1.0;
      if (rb > ra) {
        if (self) continue;
        const int x = ra;
        ra = rb;
        rb = x;
      } else if (!self && rb == ra) {
        w = 2.0;
      }
      if (!has_pair(V, ra, rb)) unsafeAtomicAdd(N + (int64_t)ra * V.n_str + rb, w * hc);
    }
  }
}

// The touched pairs of the array, listed row by row.
__global__ void __launch_bounds__(256) hbci_ext_list_kernel(const double* __restrict__ N, int n_str,
                                                            int64_t* __restrict__ elist, int64_t cap, HbciCtl* ctl) {
  __shared__ int cnt[4];
  __shared__ unsigned long long base;
  const int ra = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double* row = N + (int64_t)ra * n_str;
  int own = 0;
  for (int rb = threadIdx.x; rb <= ra; rb += 256) own += touched(row[rb]);
  own = wave_sum_int(own);
  if (lane == 0) cnt[wave] = own;
  __syncthreads();
  const int all = cnt[0] + cnt[1] + cnt[2] + cnt[3];
  if (all == 0) return;
  if (threadIdx.x == 0) {
    base = atomicAdd(&ctl->n_ext, (unsigned long long)all);
    if ((int64_t)base + all > cap) atomicOr(&ctl->flags, kFlagExtCap);
  }
  __syncthreads();
  int64_t at = (int64_t)base;
  for (int r0 = 0; r0 <= ra; r0 += 256) {
    const int rb = r0 + threadIdx.x;
    const bool t = rb <= ra && touched(row[rb]);
    const uint64_t m = __ballot(t);
    __syncthreads();
    if (lane == 0) cnt[wave] = (int)__popcll(m);
    __syncthreads();
    int64_t p = at;
    for (int w = 0; w < wave; ++w) p += cnt[w];
    p += __popcll(m & ((1ull << lane) - 1ull));
    if (t && p < cap) elist[p] = (int64_t)ra * n_str + rb;
    at += cnt[0] + cnt[1] + cnt[2] + cnt[3];
  }
}

// Sum over the workgroup; the result in thread 0.
__device__ __forceinline__ double group_sum(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
  return s;
}

// part[block] = partial sum of N_a^2 / (e - H_aa); part[kNB + block] = count
// (of the listed slots of the hash table, or places of the array N over pairs of str)
__global__ void __launch_bounds__(64 * kWaves) hbci_e2_kernel(const double* __restrict__ ints, int k,
                                                      const ExtSlot* __restrict__ et, const double* __restrict__ N,
                                                      const uint16_t* __restrict__ str, int n_str,
                                                      const int64_t* __restrict__ elist, int64_t cap,
                                                      const HbciCtl* __restrict__ ctl, double e, int half,
                                                      double* __restrict__ part) {
  const Lds s = load_lds(ints, k);
  double* red = (double*)s.lists;  // no static LDS beside the dynamic block
  const int64_t n_filled = (int64_t)ctl->n_ext < cap ? (int64_t)ctl->n_ext : cap;
  double sum = 0.0, cnt = 0.0;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_filled;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = elist[t];
    uint32_t A, B;
    double na;
    if (N) {
      A = str[p / n_str];
      B = str[p % n_str];
      na = N[p];
    } else {
      const ExtSlot sl = et[p];
      A = (uint32_t)sl.key;
      B = (uint32_t)(sl.key >> 32);
      na = sl.val;
    }
    // a representative stands for itself and its partner
    const double w = (half && A != B) ? 2.0 : 1.0;
    sum += w * (na * na / (e - diag_val(s, k, A, B)));
    cnt += w;
  }
  sum = group_sum(sum, red);
  if (threadIdx.x == 0) part[blockIdx.x] = sum;
  cnt = group_sum(cnt, red);
  if (threadIdx.x == 0) part[kNB + blockIdx.x] = cnt;
}

// ---------------------------------------------------------------- host side

int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

uint64_t pow2_at_least(int64_t x) {
  uint64_t p = 1;
  while ((int64_t)p < x) p <<= 1;
  return p;
}

struct Layout {
  int64_t ints, ctl, dav, part, bsum, dets, keys, vals, diag, cnt, addc, used, ptr[2], col[2], val[2], basis, sig, x[2],
      ext, elist;
  int64_t bound, off, bptr, rank, str, bits, pre, start, place, pair, moved, row_of, key, pos, fpos, old, rdiag;
  int64_t bytes;
  uint64_t tcap, ecap;
};

Layout layout(int k, const ifci_hbci_options& o) {
  Layout L{};
  int64_t off = 0;
  auto take = [&](int64_t b) {
    const int64_t at = off;
    off = align256(off + b);
    return at;
  };
  const int64_t D = o.max_det;
  L.tcap = pow2_at_least(2 * D);
  L.ecap = pow2_at_least(2 * o.max_ext);
  L.ints = take((int64_t)ints_count(k) * 8);
  L.ctl = take(sizeof(HbciCtl));
  L.dav = take(sizeof(DavCtl));
  L.part = take((int64_t)kNB * kParts * 8);
  L.bsum = take(((D + 1023) / 1024 + 1) * 8);
  L.dets = take(D * 8);
  L.keys = take((int64_t)L.tcap * 8);
  L.vals = take((int64_t)L.tcap * 4);
  L.diag = take(D * 8);
  L.cnt = take(D * 4);
  L.addc = take(D * 4);
  L.used = take(D * 4);
  // the bits of the widest space of k orbitals (half filled)
  int64_t strings = 1;
  for (int i = 0; i < k / 2; ++i) strings = strings * (k - i) / (i + 1);
  const int64_t words = strings * ((strings + 63) / 64);
  // of spaces in blocked form
  const int64_t bd = D < kBlockMax ? D : kBlockMax, bw = (bd + kWin - 1) / kWin;
  L.bound = take((kShares + 1) * 4);
  L.off = take((bw + 1) * (bd < kBlockMaxRows ? bd : kBlockMaxRows) * 2);
  L.bptr = take((kShares * bw + 1) * 8);
  L.rank = take(((int64_t)1 << k) * 2);
  L.str = take(strings * 2);
  L.bits = take(words * 8);
  L.pre = take(words * 4);
  L.start = take(strings * 2 * 4);
  for (int64_t* at : {&L.place, &L.pair, &L.moved, &L.row_of, &L.pos, &L.fpos, &L.old}) *at = take(D * 4);
  L.key = take(D * 8);
  L.rdiag = take(D * 8);
  // two CSR buffers: a selection step builds the new H from the old one
  for (int b = 0; b < 2; ++b) {
    L.ptr[b] = take((D + 1) * 8);
    L.col[b] = take(o.max_nnz * 4);
    L.val[b] = take(o.max_nnz * 8);
  }
  L.basis = take((int64_t)o.m_max * D * 8);
  L.sig = take((int64_t)o.m_max * D * 8);
  for (int b = 0; b < 2; ++b) L.x[b] = take(D * 8);
  L.ext = take((int64_t)L.ecap * (int64_t)sizeof(ExtSlot));
  L.elist = take(o.max_ext * 8);
  L.bytes = off;
  return L;
}

// Pinned host staging for read-backs, one per host thread.
double* staging() {
  static thread_local double* p = nullptr;
  if (!p && hipHostMalloc((void**)&p, sizeof(double) * (2 * kNB * kParts + 64)) != hipSuccess) p = nullptr;
  return p;
}

struct Run {
  HbciInc I;
  ifci_hbci_options o;
  Layout L;
  char* w;
  hipStream_t st;
  double* pin = nullptr;
  HbciCtl ctl{};
  int cur = 0;   // the CSR buffer that holds H
  int curx = 0;  // the buffer that holds x

  template <typename T>
  T* at(int64_t off) const {
    return (T*)(w + off);
  }
  Space list() const {
    return Space{at<uint64_t>(L.dets), at<uint64_t>(L.keys), at<int32_t>(L.vals), L.tcap - 1, o.max_det,
                 at<HbciCtl>(L.ctl)};
  }
  Bits bits() const {
    const int na = __builtin_popcount((uint32_t)I.ref);
    int64_t n = 1;
    for (int i = 0; i < na; ++i) n = n * (I.k - i) / (i + 1);
    return Bits{at<uint64_t>(L.bits), at<int32_t>(L.pre), at<uint16_t>(L.rank), at<uint16_t>(L.str), (int)((n + 63) / 64), (int)n,
                at<uint64_t>(L.dets), o.max_det, at<HbciCtl>(L.ctl)};
  }
  Order order() const {
    return Order{at<int32_t>(L.place), at<int32_t>(L.pair), at<int32_t>(L.moved), at<int32_t>(L.row_of),
                 at<double>(L.diag), at<uint64_t>(L.key), at<int32_t>(L.pos), at<int32_t>(L.fpos), at<int32_t>(L.old),
                 at<double>(L.rdiag)};
  }
  double* x() const { return at<double>(L.x[curx]); }
  int lds(int list, bool screen) const { return lds_bytes_for(I.k, list, screen); }
  static int blocks(int64_t n, int per, int cap) {
    const int64_t b = (n + per - 1) / per;
    return (int)(b < 1 ? 1 : (b > cap ? cap : b));
  }

  hipError_t read_ctl() {
    hipError_t e = hipMemcpyAsync(pin, at<HbciCtl>(L.ctl), sizeof(HbciCtl), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e == hipSuccess) std::memcpy(&ctl, pin, sizeof(HbciCtl));
    return e;
  }
  // sums of m rows of kNB partials, each in block order
  hipError_t read_parts(int m, double* out) {
    hipError_t e = hipMemcpyAsync(pin, at<double>(L.part), sizeof(double) * kNB * m, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return e;
    for (int j = 0; j < m; ++j) {
      double s = 0.0;
      for (int b = 0; b < kNB; ++b) s += pin[j * kNB + b];
      out[j] = s;
    }
    return hipSuccess;
  }

  // screen: with the bounds on H that selection and PT2 screen by
  hipError_t prepare(bool screen) {
    pin = staging();
    if (!pin) return hipErrorOutOfMemory;
    hipError_t e = hipSuccess;
    for (const void* fn : {(const void*)hbci_select_kernel<Space>, (const void*)hbci_select_kernel<Bits>,
                           (const void*)hbci_diag_kernel, (const void*)hbci_count_kernel, (const void*)hbci_fill_kernel,
                           (const void*)hbci_pt2_kernel<Space>, (const void*)hbci_pt2_kernel<Bits>,
                           (const void*)hbci_pt2_array_kernel,
                           (const void*)hbci_count_new_kernel, (const void*)hbci_fill_new_kernel,
                           (const void*)hbci_e2_kernel, (const void*)hbci_dav_block_kernel, (const void*)hbci_block_fill_kernel,
                           (const void*)hbci_merge_rows_kernel<1024, kMidRow, kLongRow>})
      if (e == hipSuccess) e = allow_max_lds(fn);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(hbci_prep_kernel, dim3(1), dim3(256), 0, st, I.h, I.eri, I.n_orb, I.act, I.k, I.core,
                       I.n_core, I.e_core, at<double>(L.ints), at<HbciCtl>(L.ctl));
    if (screen) hipLaunchKernelGGL(hbci_bounds_kernel, dim3(1), dim3(1024), 0, st, at<double>(L.ints), I.k);
    return hipGetLastError();
  }

  // V := the caller's list; ctl read
  hipError_t load(const uint64_t* dets, int64_t n) {
    hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks((int64_t)L.tcap, 256, 4096)), dim3(256), 0, st,
                       at<uint64_t>(L.keys), (int64_t)L.tcap, kEmpty);
    hipLaunchKernelGGL(hbci_load_kernel, dim3(blocks(n, 256, 4096)), dim3(256), 0, st, dets, n, list());
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? read_ctl() : e;
  }

  // V := the reference; ctl read
  hipError_t load_reference() {
    const Bits V = bits();
    const int64_t words = (int64_t)V.n_str * V.W;
    hipLaunchKernelGGL(hbci_rank_kernel, dim3(blocks((int64_t)1 << I.k, 256, 256)), dim3(256), 0, st, I.k,
                       __builtin_popcount((uint32_t)I.ref), at<uint16_t>(L.rank), at<uint16_t>(L.str));
    hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks(words, 256, 4096)), dim3(256), 0, st, V.w, words, (uint64_t)0);
    hipLaunchKernelGGL(hbci_ref_kernel, dim3(1), dim3(1), 0, st, I.ref, V);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? read_ctl() : e;
  }

  hipError_t diag(int64_t lo, int64_t n) {
    if (n <= lo) return hipSuccess;
    hipLaunchKernelGGL(hbci_diag_kernel, dim3(blocks(n - lo, 64 * kWaves, 2048)), dim3(64 * kWaves),
                       lds(kListRanks, false), st, at<double>(L.ints), I.k, at<uint64_t>(L.dets), lo, n,
                       at<double>(L.diag));
    return hipGetLastError();
  }

  // The places of the n keys after a step that added those from lo on, with
  // the diagonal and x brought to them; ctl read
  hipError_t reorder(int64_t lo, int64_t n) {
    hipError_t e = diag(lo, n);
    if (e != hipSuccess) return e;
    const Bits V = bits();
    int32_t* start = at<int32_t>(L.start);
    const int rows = (V.n_str + 3) / 4;
    hipLaunchKernelGGL(hbci_row_count_kernel, dim3(rows), dim3(256), 0, st, V, start);
    hipLaunchKernelGGL(hbci_row_scan_kernel, dim3(1), dim3(1024), 0, st, V.n_str, start, at<HbciCtl>(L.ctl));
    hipLaunchKernelGGL(hbci_word_scan_kernel, dim3(rows), dim3(256), 0, st, V, start);
    hipLaunchKernelGGL(hbci_order_kernel, dim3(blocks(n, 256, 4096)), dim3(256), 0, st, V, lo, n, start, order(),
                       at<double>(L.x[curx]), at<double>(L.x[curx ^ 1]));
    curx ^= 1;
    e = hipGetLastError();
    if (e == hipSuccess) e = read_ctl();
    return e;
  }

  // CSR of H over the n keys of a list; IFCI_ERR_OOM past max_nnz
  ifci_status build_h(int64_t n, hipError_t* he) {
    hipLaunchKernelGGL(hbci_count_kernel, dim3(blocks(n, kWaves, 8192)), dim3(64 * kWaves), lds(kListRanks, false), st,
                       at<double>(L.ints), I.k, list(), n, at<int32_t>(L.cnt));
    ifci_status s = scan_rows(n, L.ptr[cur], he);
    if (s != IFCI_OK) return s;
    hipLaunchKernelGGL(hbci_fill_kernel, dim3(blocks(n, kWaves, 8192)), dim3(64 * kWaves), lds(kListRanks, false), st,
                       at<double>(L.ints), I.k, list(), n, at<int64_t>(L.ptr[cur]), at<int32_t>(L.col[cur]),
                       at<double>(L.val[cur]));
    *he = hipGetLastError();
    return *he == hipSuccess ? IFCI_OK : IFCI_ERR_DEVICE;
  }

  // row offsets at ptr_off from cnt[0..n); the total checked against max_nnz
  ifci_status scan_rows(int64_t n, int64_t ptr_off, hipError_t* he) {
    const int64_t nb = (n + 1023) / 1024;
    hipLaunchKernelGGL(scan_block_kernel, dim3((unsigned)nb), dim3(1024), 0, st, at<int32_t>(L.cnt), n,
                       at<int64_t>(ptr_off), at<int64_t>(L.bsum));
    hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(1024), 0, st, at<int64_t>(L.bsum), nb, at<HbciCtl>(L.ctl));
    hipLaunchKernelGGL(scan_add_kernel, dim3(blocks(n, 256, 1 << 30)), dim3(256), 0, st, at<int64_t>(ptr_off), n,
                       at<int64_t>(L.bsum));
    *he = hipGetLastError();
    if (*he == hipSuccess) *he = read_ctl();
    if (*he != hipSuccess) return IFCI_ERR_DEVICE;
    if (ctl.nnz > o.max_nnz) {
      set_error("HBCI: H over the selected space has more nonzeros than max_nnz");
      return IFCI_ERR_OOM;
    }
    return IFCI_OK;
  }

  // H over the n_rep pairs of the new order from H before the step (none at
  // first): the new rows from scratch, the old ones copied and extended by
  // the entries the new rows imply; the result in the other buffer, which
  // becomes current.
  ifci_status extend_h(int64_t n_rep, hipError_t* he) {
    const int nxt = cur ^ 1;
    const Bits V = bits();
    const Order O = order();
    const int gb = blocks(n_rep, 256, 4096), gw = blocks(n_rep, kWaves, 8192);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(gb), dim3(256), 0, st, at<int32_t>(L.addc), n_rep, 0);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(gb), dim3(256), 0, st, at<int32_t>(L.used), n_rep, 0);
    hipLaunchKernelGGL(hbci_count_new_kernel, dim3(gw), dim3(64 * kWaves), lds(kListRanks, false), st,
                       at<double>(L.ints), I.k, V, O, n_rep, at<int32_t>(L.cnt), at<int32_t>(L.addc));
    hipLaunchKernelGGL(hbci_rowlen_kernel, dim3(gb), dim3(256), 0, st, at<int64_t>(L.ptr[cur]), O.old, n_rep,
                       at<int32_t>(L.addc), at<int32_t>(L.cnt));
    ifci_status s = scan_rows(n_rep, L.ptr[nxt], he);
    if (s != IFCI_OK) return s;
    hipLaunchKernelGGL(hbci_fill_new_kernel, dim3(gw), dim3(64 * kWaves), lds(kListRanks, false), st,
                       at<double>(L.ints), I.k, V, O, n_rep, at<int64_t>(L.ptr[cur]), at<int64_t>(L.ptr[nxt]),
                       at<int32_t>(L.used), at<int32_t>(L.col[nxt]), at<double>(L.val[nxt]));
    const int na = __builtin_popcount((uint32_t)I.ref), s1 = na * (I.k - na);
    const int longest = s1 * (s1 + 2) + na * (na - 1) / 2 * (I.k - na) * (I.k - na - 1);
    hipLaunchKernelGGL((hbci_merge_rows_kernel<256, 0, kShortRow>), dim3(blocks(n_rep, 1, 8192)), dim3(256),
                       kShortRow * 12, st, at<int64_t>(L.ptr[cur]), at<int32_t>(L.col[cur]), at<double>(L.val[cur]),
                       O.old, O.moved, n_rep, at<int64_t>(L.ptr[nxt]), at<int32_t>(L.col[nxt]),
                       at<double>(L.val[nxt]));
    if (longest > kShortRow)
      hipLaunchKernelGGL((hbci_merge_rows_kernel<256, kShortRow, kMidRow>), dim3(blocks(n_rep, 1, 8192)), dim3(256),
                         kMidRow * 12, st, at<int64_t>(L.ptr[cur]), at<int32_t>(L.col[cur]), at<double>(L.val[cur]),
                         O.old, O.moved, n_rep, at<int64_t>(L.ptr[nxt]), at<int32_t>(L.col[nxt]),
                         at<double>(L.val[nxt]));
    if (longest > kMidRow)
      hipLaunchKernelGGL((hbci_merge_rows_kernel<1024, kMidRow, kLongRow>), dim3(blocks(n_rep, 1, 8192)), dim3(1024),
                         kLongRow * 12, st, at<int64_t>(L.ptr[cur]), at<int32_t>(L.col[cur]), at<double>(L.val[cur]),
                         O.old, O.moved, n_rep, at<int64_t>(L.ptr[nxt]), at<int32_t>(L.col[nxt]),
                         at<double>(L.val[nxt]));
    *he = hipGetLastError();
    if (*he != hipSuccess) return IFCI_ERR_DEVICE;
    cur = nxt;
    return IFCI_OK;
  }

  template <int M>
  void dav_step(const DavSpace& a, int m, bool check_only) {
    const dim3 g(blocks(a.n, kVecThreads, kVecBlocks)), b(kVecThreads);
    hipLaunchKernelGGL(hbci_dav_residual_kernel<M>, g, b, 0, st, a, m, o.r_tol);
    if (check_only) return;
    hipLaunchKernelGGL((hbci_dav_orth_kernel<M, false>), g, b, 0, st, a, m);
    hipLaunchKernelGGL((hbci_dav_orth_kernel<M, true>), g, b, 0, st, a, m);
  }
  void dav_step(const DavSpace& a, int m, bool check_only) {
    if (m <= 4) dav_step<4>(a, m, check_only);
    else if (m <= 8) dav_step<8>(a, m, check_only);
    else if (m <= 12) dav_step<12>(a, m, check_only);
    else dav_step<16>(a, m, check_only);
  }
  static bool blocked(const DavSpace& a) {
    return a.n_full <= kBlockMax && a.n <= kBlockMaxRows;
  }
  // the blocked form of H, in the CSR buffer that the next step builds its H in
  void block_h(const DavSpace& a) {
    const int nwin = (int)((a.n_full + kWin - 1) / kWin);
    int32_t* bound = at<int32_t>(L.bound);
    uint16_t* off = at<uint16_t>(L.off);
    int64_t* bptr = at<int64_t>(L.bptr);
    hipLaunchKernelGGL(hbci_share_kernel, dim3(1), dim3(512), 0, st, a.ptr, a.n, bound);
    hipLaunchKernelGGL(hbci_win_offsets_kernel, dim3(blocks(a.n, 4, 8192)), dim3(256), 0, st, a.ptr, a.col, a.n, nwin,
                       off);
    hipLaunchKernelGGL(hbci_block_ptr_kernel, dim3(kShares), dim3(1024), 0, st, a.ptr, a.n, nwin, bound, off, bptr);
    hipLaunchKernelGGL(hbci_block_fill_kernel, dim3(kShares, nwin), dim3(1024), kBlockFillLds, st, a.ptr, a.col, a.val, a.n, nwin,
                       bound, off, bptr, at<uint32_t>(L.col[cur ^ 1]), at<double>(L.val[cur ^ 1]));
  }
  void dav_product(const DavSpace& a, int m) {
    const int nb = blocked(a) ? kShares : blocks(a.n, 16, kRowBlocks);
    if (blocked(a))
      hipLaunchKernelGGL(hbci_dav_block_kernel, dim3(nb), dim3(1024), kBlockLds, st, a, m);
    else
      hipLaunchKernelGGL(hbci_dav_product_kernel, dim3(nb), dim3(1024), 0, st, a, m);
    hipLaunchKernelGGL(hbci_dav_subspace_kernel, dim3(1), dim3(1024), 0, st, a, nb, m, o.m_max);
  }

  // Davidson for the lowest root over the n keys (n_rep pairs) from the unit,
  // flip-symmetric start vector in x; the Ritz vector is left in x.  The
  // steps are queued kBatch at a time between two looks at their state; those
  // after the last one do nothing.
  hipError_t davidson(int64_t n, int64_t n_rep, double* theta_out, double* res_out, bool* conv) {
    constexpr int kBatch = 4;
    const DavSpace a{at<int64_t>(L.ptr[cur]), at<int32_t>(L.col[cur]), at<double>(L.val[cur]), at<double>(L.rdiag),
                     at<int32_t>(L.pos), at<int32_t>(L.fpos), x(), at<double>(L.basis), at<double>(L.sig),
                     at<double>(L.part), at<DavCtl>(L.dav), o.max_det, n_rep, n, at<int32_t>(L.bound),
                     at<int64_t>(L.bptr), at<uint32_t>(L.col[cur ^ 1]), at<double>(L.val[cur ^ 1])};
    if (n <= kSmallDav) {
      const SmallDav s{a, o.m_max, o.max_dav, o.r_tol, at<double>(L.part)};
      hipLaunchKernelGGL(hbci_dav_small_kernel, dim3(1), dim3(kSmallThreads), 0, st, s);
      hipError_t e = hipGetLastError();
      if (e == hipSuccess) e = hipMemcpyAsync(pin, s.out, 3 * sizeof(double), hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) return e;
      *theta_out = pin[0];
      *res_out = pin[1];
      *conv = pin[2] != 0.0;
      return hipSuccess;
    }
    const auto look = [&](int* done) {
      hipError_t e = hipGetLastError();
      if (e == hipSuccess) e = hipMemcpyAsync(pin, a.ctl, 3 * sizeof(double), hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) return e;
      *theta_out = pin[0];
      *res_out = pin[1];
      std::memcpy(done, pin + 2, sizeof(int));
      return hipSuccess;
    };
    if (blocked(a)) block_h(a);
    hipLaunchKernelGGL(hbci_dav_start_kernel, dim3(blocks(n_rep, 256, 1 << 30)), dim3(256), 0, st, a);
    dav_product(a, 0);
    int m = 1, done = 0;
    for (int it = 0; it < o.max_dav && !done;) {
      for (int b = 0; b < kBatch && it < o.max_dav; ++b, ++it) {
        dav_step(a, m, false);
        dav_product(a, m);
        if (++m == o.m_max) {
          const dim3 g(blocks(n_rep, 256, kVecBlocks)), t(256);
          const int keep = kept_ritz(m);
          if (m <= 12)
            hipLaunchKernelGGL(hbci_dav_restart_kernel<12>, g, t, 0, st, a, m, keep);
          else
            hipLaunchKernelGGL(hbci_dav_restart_kernel<16>, g, t, 0, st, a, m, keep);
          m = keep;
        }
      }
      const hipError_t e = look(&done);
      if (e != hipSuccess) return e;
    }
    if (!done) {  // out of steps: the residual of the last Ritz pair
      dav_step(a, m, true);
      const hipError_t e = look(&done);
      if (e != hipSuccess) return e;
    }
    *conv = done == 1;
    hipLaunchKernelGGL(hbci_dav_vector_kernel, dim3(blocks(n_rep, 256, kVecBlocks)), dim3(256), 0, st, a);
    return hipGetLastError();
  }

  // PT2 over the n keys (src, at places pos of c), V a list or the bits
  template <typename VSpace>
  hipError_t pt2(const VSpace& V, const uint64_t* src, const int32_t* pos, int64_t n, const double* c, double e_act,
                 double eps2, bool half, double* e2, int64_t* n_ext) {
    hipLaunchKernelGGL(fill_slots_kernel, dim3(blocks((int64_t)L.ecap, 256, 4096)), dim3(256), 0, st,
                       at<ExtSlot>(L.ext), (int64_t)L.ecap);
    hipLaunchKernelGGL(hbci_pt2_kernel<VSpace>, dim3(blocks(n, kWaves, 8192)), dim3(64 * kWaves),
                       lds(kListPairs, true), st, at<double>(L.ints), I.k, V, src, pos, c, n, eps2, half ? 1 : 0,
                       at<ExtSlot>(L.ext), at<int64_t>(L.elist), L.ecap - 1, o.max_ext);
    return e2_sum(nullptr, 0, e_act, half, e2, n_ext);
  }

  // the same of a solve (half), with the external space as an array where it
  // fits the table's room: 16 bytes a slot, at least two slots per key
  hipError_t pt2_solve(const Bits& V, const Order& O, int64_t n_rep, double e_act, double* e2, int64_t* n_ext) {
    const int64_t pairs = (int64_t)V.n_str * V.n_str;
    if (pairs > 2 * (int64_t)L.ecap) return pt2(V, O.key, O.pos, n_rep, x(), e_act, o.eps2, true, e2, n_ext);
    double* N = at<double>(L.ext);
    hipLaunchKernelGGL(fill_f64_kernel, dim3(blocks(pairs, 256, 4096)), dim3(256), 0, st, N, pairs, -0.0);
    hipLaunchKernelGGL(hbci_pt2_array_kernel, dim3(blocks(n_rep, kWaves, 8192)), dim3(64 * kWaves),
                       lds(kListPairs, true), st, at<double>(L.ints), I.k, V, O.key, O.pos, x(), n_rep, o.eps2, N);
    hipLaunchKernelGGL(hbci_ext_list_kernel, dim3(V.n_str), dim3(256), 0, st, N, V.n_str, at<int64_t>(L.elist),
                       o.max_ext, at<HbciCtl>(L.ctl));
    return e2_sum(N, V.n_str, e_act, true, e2, n_ext);
  }

  hipError_t e2_sum(const double* N, int n_str, double e_act, bool half, double* e2, int64_t* n_ext) {
    hipLaunchKernelGGL(hbci_e2_kernel, dim3(kNB), dim3(64 * kWaves), lds(kListRanks, false), st, at<double>(L.ints),
                       I.k, at<ExtSlot>(L.ext), N, at<uint16_t>(L.str), n_str, at<int64_t>(L.elist), o.max_ext,
                       at<HbciCtl>(L.ctl), e_act, half ? 1 : 0, at<double>(L.part));
    hipError_t e = hipGetLastError();
    double s[2];
    if (e == hipSuccess) e = read_parts(2, s);
    if (e == hipSuccess) e = read_ctl();
    if (e != hipSuccess) return e;
    *e2 = s[0];
    *n_ext = (int64_t)std::llround(s[1]);
    return e;
  }

  template <typename VSpace>
  hipError_t select(const VSpace& V, const uint64_t* src, const int32_t* pos, int64_t n, const double* c, double eps) {
    hipLaunchKernelGGL(hbci_select_kernel<VSpace>, dim3(blocks(n, kWaves, 8192)), dim3(64 * kWaves),
                       lds(kListPairs, true), st, at<double>(L.ints), I.k, src, pos, c, n, eps, V);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? read_ctl() : e;
  }
};

ifci_status device_failure(hipError_t e, const char* where) {
  set_error(std::string(where) + ": " + hipGetErrorString(e));
  return IFCI_ERR_DEVICE;
}

ifci_status capacity_failure(unsigned flags) {
  if (flags & kFlagDetCap) set_error("HBCI: the selected space outgrew max_det");
  else if (flags & kFlagExtCap) set_error("HBCI: the PT2 external space outgrew max_ext");
  else if (flags & kFlagDuplicate) set_error("HBCI: the determinant list repeats a key");
  else set_error("HBCI: a determinant's spin-flipped partner is missing from the space");
  return (flags & (kFlagDetCap | kFlagExtCap)) ? IFCI_ERR_OOM : IFCI_ERR_ARG;
}

#define HB_TRY(expr, where)                                   \
  do {                                                        \
    hipError_t e_ = (expr);                                   \
    if (e_ != hipSuccess) return device_failure(e_, where);   \
  } while (0)

}  // namespace

int64_t hbci_work_bytes(int k, const ifci_hbci_options& o) { return layout(k, o).bytes; }

ifci_status hbci_solve(const HbciInc& I, const ifci_hbci_options& o, void* work, double* result, uint64_t* dets_out,
                       double* c_out, hipStream_t st) {
  Run R{I, o, layout(I.k, o), (char*)work, st};
  HB_TRY(R.prepare(true), "hbci prepare");
  HB_TRY(R.load_reference(), "hbci load");
  const double shift = R.ctl.e_core + I.e_const;
  int64_t n = (int64_t)R.ctl.n_det, n_rep = 0;
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  const Bits V = R.bits();
  const Order O = R.order();
  double theta = 0.0, res = 0.0;
  bool all_conv = true;
  // the places of V's keys after those from lo on were added, H over them and its lowest root
  auto solve = [&](int64_t lo, bool first) -> ifci_status {
    HB_TRY(R.reorder(lo, n), "hbci order");
    if (R.ctl.flags) return capacity_failure(R.ctl.flags);
    n_rep = (int64_t)R.ctl.n_rep;
    if (first) {  // V = {reference}: c = 1
      hipLaunchKernelGGL(fill_f64_kernel, dim3(1), dim3(64), 0, st, R.x(), n, 1.0);
      HB_TRY(hipGetLastError(), "hbci start");
    }
    hipError_t he;
    const ifci_status s = R.extend_h(n_rep, &he);
    if (s == IFCI_ERR_DEVICE) return device_failure(he, "hbci H");
    if (s != IFCI_OK) return s;
    bool cv;
    HB_TRY(R.davidson(n, n_rep, &theta, &res, &cv), "hbci davidson");
    all_conv = all_conv && cv;
    return IFCI_OK;
  };
  ifci_status s = solve(0, true);
  if (s != IFCI_OK) return s;
  int steps = 0;
  bool fixed = false;
  while (steps < o.max_iter) {
    const int64_t n_old = n;
    HB_TRY(R.select(V, O.key, O.pos, n_rep, R.x(), o.eps1), "hbci select");
    ++steps;
    if (R.ctl.flags) return capacity_failure(R.ctl.flags);
    n = (int64_t)R.ctl.n_det;
    if (n == n_old) {
      fixed = true;
      break;
    }
    if ((s = solve(n_old, false)) != IFCI_OK) return s;
  }
  double e2 = 0.0;
  int64_t n_ext = 0;
  HB_TRY(R.pt2_solve(V, O, n_rep, theta, &e2, &n_ext), "hbci pt2");
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  if (dets_out) HB_TRY(hipMemcpyAsync(dets_out, R.at<uint64_t>(R.L.dets), n * 8, hipMemcpyDeviceToDevice, st), "copy");
  if (c_out) {
    hipLaunchKernelGGL(hbci_by_insertion_kernel, dim3(Run::blocks(n, 256, 4096)), dim3(256), 0, st, O.place, R.x(), n,
                       c_out);
    HB_TRY(hipGetLastError(), "hbci");
  }
  HB_TRY(hipStreamSynchronize(st), "hbci");
  result[0] = theta + shift;
  result[1] = e2;
  result[2] = (double)n;
  result[3] = (double)steps;
  result[4] = (fixed && all_conv) ? 1.0 : 0.0;
  result[5] = res;
  result[6] = (double)n_ext;
  result[7] = (double)R.ctl.nnz;
  return IFCI_OK;
}

ifci_status hbci_sigma(const HbciInc& I, const ifci_hbci_options& o, void* work, const uint64_t* dets, int64_t n,
                       const double* c, double* sigma, hipStream_t st) {
  Run R{I, o, layout(I.k, o), (char*)work, st};
  HB_TRY(R.prepare(false), "hbci prepare");
  HB_TRY(R.load(dets, n), "hbci load");
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  HB_TRY(R.diag(0, n), "hbci diagonal");
  hipError_t he;
  ifci_status s = R.build_h(n, &he);
  if (s == IFCI_ERR_DEVICE) return device_failure(he, "hbci H");
  if (s != IFCI_OK) return s;
  hipLaunchKernelGGL(hbci_spmv_kernel, dim3(Run::blocks(n, 4, 8192)), dim3(256), 0, st, R.at<int64_t>(R.L.ptr[R.cur]),
                     R.at<int32_t>(R.L.col[R.cur]), R.at<double>(R.L.val[R.cur]), R.at<double>(R.L.diag), c, sigma, n);
  HB_TRY(hipGetLastError(), "hbci sigma");
  HB_TRY(hipStreamSynchronize(st), "hbci sigma");
  return IFCI_OK;
}

ifci_status hbci_select(const HbciInc& I, const ifci_hbci_options& o, void* work, const uint64_t* dets, int64_t n,
                        const double* c, double eps1, uint64_t* added, int64_t* n_added, hipStream_t st) {
  Run R{I, o, layout(I.k, o), (char*)work, st};
  HB_TRY(R.prepare(true), "hbci prepare");
  HB_TRY(R.load(dets, n), "hbci load");
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  HB_TRY(R.select(R.list(), R.at<uint64_t>(R.L.dets), nullptr, n, c, eps1), "hbci select");
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  const int64_t m = (int64_t)R.ctl.n_det - n;
  if (m > 0)
    HB_TRY(hipMemcpyAsync(added, R.at<uint64_t>(R.L.dets) + n, m * 8, hipMemcpyDeviceToDevice, st), "copy");
  HB_TRY(hipStreamSynchronize(st), "hbci select");
  *n_added = m;
  return IFCI_OK;
}

ifci_status hbci_pt2(const HbciInc& I, const ifci_hbci_options& o, void* work, const uint64_t* dets, int64_t n,
                     const double* c, double e_var, double eps2, double* e_pt2, int64_t* n_ext, hipStream_t st) {
  Run R{I, o, layout(I.k, o), (char*)work, st};
  HB_TRY(R.prepare(true), "hbci prepare");
  HB_TRY(R.load(dets, n), "hbci load");
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  const double shift = R.ctl.e_core + I.e_const;
  HB_TRY(R.pt2(R.list(), R.at<uint64_t>(R.L.dets), nullptr, n, c, e_var - shift, eps2, false, e_pt2, n_ext),
         "hbci pt2");
  if (R.ctl.flags) return capacity_failure(R.ctl.flags);
  return IFCI_OK;
}

}  // namespace ifci
