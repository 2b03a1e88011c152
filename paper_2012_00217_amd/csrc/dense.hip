// Small dense FP64 linear algebra of LOBPCG's Rayleigh-Ritz and
// orthonormalisation steps (paper Sec. 3.2), sizes up to a few hundred.
//
//  * Symmetric eigendecomposition by cyclic two-sided Jacobi with the
//    round-robin (tournament) pair ordering: in each round the indices are
//    split into disjoint pairs, so all rotations of a round commute and the
//    matrix splits into 2 x 2 blocks that are updated independently,
//    A_kl <- J_k^T A_kl J_l.  Sizes <= 192 run in one workgroup with the upper
//    triangle of A in LDS; larger ones run one kernel per round, ping-ponging A between two
//    buffers so the rotations of a round are computed from the unmodified
//    matrix.  A sweep ends with a count of rotations; none means converged.
//    Jacobi keeps small eigenvalues of positive semi-definite matrices to
//    high relative accuracy, which matters for the spectral fold.
//  * Cholesky with column dropping, R^T R = G, for Cholesky-QR: a column whose
//    pivot falls below tol * G_jj is linearly dependent on the earlier ones and
//    is dropped; the inverse of R on the kept columns is returned compacted.
//  * Small matrix products and the nearest-shift selection.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"

namespace mbl {
namespace {

constexpr double kRotTol = 1e-15;  // rotate when |a_pq| > tol * sqrt(|a_pp a_qq|)

// Pair k of a round: the fixed index mm - 1 (k = 0) or (round + k) mod (mm - 1), and
// (round - k) mod (mm - 1).  Both move on by one each round.
struct Pair {
  int a, b;
  bool fixed;  // a stays
  __device__ Pair() {}
  __device__ Pair(int mm, int round, int k) : fixed(k == 0) {
    a = round + k;
    b = round - k;
    if (a >= mm - 1) a -= mm - 1;
    if (b < 0) b += mm - 1;
    if (fixed) a = mm - 1;
  }
  __device__ void step(int mm) {
    const int a1 = a + 1 == mm - 1 ? 0 : a + 1;
    a = fixed ? a : a1;
    b = b + 1 == mm - 1 ? 0 : b + 1;
  }
};

__device__ inline void pair_of(int mm, int round, int k, int* p, int* q) {
  const Pair t(mm, round, k);
  *p = min(t.a, t.b);
  *q = max(t.a, t.b);
}

// 1 / sqrt(x) to about an ulp for normal x > 0: the hardware estimate (half the
// bits) and one third-order correction.
__device__ inline double rsqrt_fast(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Rotation (c, s) that annihilates a_pq:  A' = J^T A J with J_pp = J_qq = c,
// J_pq = s, J_qp = -s.  Returns false (c = 1, s = 0) when a_pq is negligible.
// p > q (swapped) gives the same rotation of the two rows as p < q.
// With d = a_qq - a_pp, b = 2 a_pq, u = |d| + hypot(d, b) (no cancellation):
// (c, s) = (u, +-b) / hypot(u, b).  Two reciprocal roots follow each other (d and b are
// first scaled by a power of two), where tan = 1 / (tau + sqrt(1 + tau^2)),
// c = 1 / sqrt(1 + tan^2) chains two roots and three divisions; every round of the
// sweep waits for this.
__device__ inline bool rotation(double app, double aqq, double apq, bool swapped, double* c,
                                double* s) {
  const bool rot = apq != 0.0 && !(fabs(apq) <= kRotTol * sqrt(fabs(app * aqq)));
  double d = aqq - app, b = 2.0 * apq;
  const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(b)));
  d = ldexp(d, e);
  b = ldexp(b, e);
  const double x = fma(d, d, b * b);
  const double u = fma(x, rsqrt_fast(x), fabs(d));
  const double q = rsqrt_fast(fma(u, u, b * b));
  const bool up = d > 0.0 || (d == 0.0 && !swapped);
  *c = rot ? u * q : 1.0;
  *s = rot ? (up ? b : -b) * q : 0.0;
  return rot;
}

// 2 x 2 block update B' = J_k^T B J_l.
__device__ inline void rot_block(double ck, double sk, double cl, double sl, double& bpp,
                                 double& bpq, double& bqp, double& bqq) {
  const double rpp = ck * bpp - sk * bqp, rpq = ck * bpq - sk * bqq;
  const double rqp = sk * bpp + ck * bqp, rqq = sk * bpq + ck * bqq;
  bpp = cl * rpp - sl * rpq;
  bpq = sl * rpp + cl * rpq;
  bqp = cl * rqp - sl * rqq;
  bqq = sl * rqp + cl * rqq;
}

// Whole Jacobi eigensolver in one workgroup (mm <= 192, even), A in LDS.  Only the
// blocks k <= l of a round are worked out, and every thread keeps its blocks
// through the whole run.  What a round costs is latency (the rotation of its pairs,
// then the update of the blocks, a barrier after each), so the eigenvectors are
// kept out of it: they need the rotations alone, row by row independently, and
// larger sizes record them (kVecRecord) for k_jacobi_vectors to apply on other CUs;
// sizes up to 48 update V in LDS beside A (kVecInline), which costs less than a second launch.
enum { kVecNone = 0, kVecInline = 1, kVecRecord = 2 };
constexpr int kMaxSweeps = 30;
constexpr int kLdsMax = 192;     // largest size in one workgroup
constexpr int kSquareMax = 136;  // largest size stored as a full square
constexpr int kInlineMax = 48;   // largest size with V beside A
constexpr int kVRows = 4;        // rows of V per thread with V beside A

// Wavefronts by what they do: rotations first, then blocks, then V (kVecInline).
struct JacobiWaves {
  int rot, blocks, vec;
  int threads() const { return 64 * (rot + blocks + vec); }
};
inline int jacobi_blocks(int mm) { return (mm / 2) * (mm / 2 + 1) / 2; }
inline JacobiWaves jacobi_waves(int mm, bool vec) {
  JacobiWaves w;
  const int np = mm / 2;
  if (mm > kSquareMax) return {0, 16, 0};
  w.rot = (np + 63) / 64;
  w.vec = vec ? (np * ((mm + kVRows - 1) / kVRows) + 63) / 64 : 0;
  w.blocks = std::min(16 - w.rot - w.vec, (jacobi_blocks(mm) + 63) / 64);
  return w;
}
inline size_t jacobi_lds_bytes(int mm, bool vec) {
  const size_t a = mm <= kSquareMax ? mm * (mm + 1) : mm * (mm + 1) / 2;
  return (a + (vec ? mm * mm : 0)) * sizeof(double) +
         (size_t)(mm / 2) * (sizeof(double2) + (mm <= kSquareMax ? 0 : sizeof(int4)));
}

struct JacobiOut {
  double* w;
  double* V;      // kVecInline
  int64_t ldv;
  double2* rec;   // kVecRecord: (c, s) of every pair of every round
  int* info;      // kVecRecord: rounds recorded, then the place of every column
};

// Block e of the list (0,0), (0,1), ..., (0,np-1), (1,1), ...: neighbouring threads
// read neighbouring columns of one row.
__device__ inline void block_of(int e, int np, int* k, int* l) {
  const int nb = np * (np + 1) / 2, g = nb - 1 - min(e, nb - 1);
  int r = (int)((sqrtf(8.0f * (float)g + 1.0f) - 1.0f) * 0.5f);
  while (r * (r + 1) / 2 > g) --r;
  while ((r + 1) * (r + 2) / 2 <= g) ++r;
  *k = np - 1 - r;
  *l = np - 1 - (g - r * (r + 1) / 2);
}

// Eigenvalues (diag(i)) in ascending order (ties by index), and where each went.
template <int VEC, class F>
__device__ __forceinline__ void jacobi_sorted(int m, const JacobiOut& o, F&& diag,
                                              const double* v, int mm) {
  for (int j = threadIdx.x; j < m; j += blockDim.x) {
    const double dj = diag(j);
    int r = 0;
    for (int i = 0; i < m; ++i) {
      const double di = diag(i);
      r += (di < dj) || (di == dj && i < j);
    }
    o.w[r] = dj;
    if constexpr (VEC == kVecRecord) o.info[1 + j] = r;
    if constexpr (VEC == kVecInline)
      for (int i = 0; i < m; ++i) o.V[(int64_t)i * o.ldv + r] = v[i * mm + j];
  }
}

// mm <= 136: A as a full square of odd stride; blocks k <= l are read once and
// written to both sides.  NB: blocks per thread.  A wavefront issues one instruction in
// about five cycles, so the rotations, the blocks and V have wavefronts of their own:
// while the first ones work out the rotations of a round the others read what they
// will update; barrier; update; barrier.  The indices of a pair move on by one each
// round.
template <int VEC, int NB>
__device__ __forceinline__ void jacobi_square(int m, const double* __restrict__ A, int64_t lda,
                                              const JacobiOut& o, const JacobiWaves& jw) {
  extern __shared__ __align__(16) double sh[];
  __shared__ int rotated[2];
  const int mm = m + (m & 1), np = mm / 2, S = mm + 1;
  double2* cs = reinterpret_cast<double2*>(sh);   // rotation of each pair
  double* a = reinterpret_cast<double*>(cs + np);
  double* v = a + mm * S;                         // kVecInline: mm x mm
  const int tid = threadIdx.x, nt = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int e = tid; e < mm * mm; e += nt) {
    const int i = e / mm, j = e - i * mm;
    const int r = min(i, j), c = max(i, j);  // symmetrised from the upper triangle
    a[i * S + j] = c < m ? A[(int64_t)r * lda + c] : 0.0;
    if constexpr (VEC == kVecInline) v[e] = (i == j) ? 1.0 : 0.0;
  }
  if (tid < 2) rotated[tid] = 0;
  __syncthreads();
  int sweep = 0;
  // runs sweeps until one does nothing: per round before(), barrier, after(), barrier
  auto sweeps = [&](auto&& begin, auto&& before, auto&& after) {
    for (; sweep < kMaxSweeps; ++sweep) {
      begin();
      for (int round = 0; round < mm - 1; ++round) {
        before();
        __syncthreads();
        after();
        __syncthreads();
      }
      const bool more = rotated[sweep & 1] != 0;
      if (tid == 0) rotated[1 - (sweep & 1)] = 0;
      __syncthreads();
      if (!more) break;
    }
  };
  if (wave < jw.rot) {
    Pair mine;
    double2* rec = o.rec + tid;
    const bool act = tid < np;
    sweeps([&] { mine = Pair(mm, 0, min(tid, np - 1)); },
           [&] {
             if (act) {
               double c, s;
               if (rotation(a[mine.a * S + mine.a], a[mine.b * S + mine.b], a[mine.a * S + mine.b],
                            mine.a > mine.b, &c, &s))
                 rotated[sweep & 1] = 1;
               cs[tid] = make_double2(c, s);
               if constexpr (VEC == kVecRecord) {
                 *rec = make_double2(c, s);
                 rec += np;
               }
             }
             mine.step(mm);
           },
           [] {});
  } else if (wave < jw.rot + jw.blocks) {
    const int nb = np * (np + 1) / 2, bt = tid - 64 * jw.rot, nbt = 64 * jw.blocks;
    int bk[NB], bl[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) block_of(bt + t * nbt, np, &bk[t], &bl[t]);
    Pair pk[NB], pl[NB];
    double x[NB][4];
    sweeps(
        [&] {
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            pk[t] = Pair(mm, 0, bk[t]);
            pl[t] = Pair(mm, 0, bl[t]);
          }
        },
        [&] {
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            if (bt + t * nbt >= nb) continue;
            const int ra = pk[t].a * S, rb = pk[t].b * S;
            x[t][0] = a[ra + pl[t].a];
            x[t][1] = a[ra + pl[t].b];
            x[t][2] = a[rb + pl[t].a];
            x[t][3] = a[rb + pl[t].b];
          }
        },
        [&] {
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            if (bt + t * nbt < nb) {
              const double2 ck = cs[bk[t]], cl = cs[bl[t]];
              rot_block(ck.x, ck.y, cl.x, cl.y, x[t][0], x[t][1], x[t][2], x[t][3]);
              const int ka = pk[t].a, kb = pk[t].b, la = pl[t].a, lb = pl[t].b;
              const bool diag = bk[t] == bl[t];  // then entries 1 and 2 are a_pq, now 0
              const double x1 = diag ? 0.0 : x[t][1], x2 = diag ? 0.0 : x[t][2];
              a[ka * S + la] = x[t][0];
              a[ka * S + lb] = x1;
              a[kb * S + la] = x2;
              a[kb * S + lb] = x[t][3];
              a[la * S + ka] = x[t][0];
              a[lb * S + ka] = x1;
              a[la * S + kb] = x2;
              a[lb * S + kb] = x[t][3];
            }
            pk[t].step(mm);
            pl[t].step(mm);
          }
        });
  } else if constexpr (VEC == kVecInline) {
    // pair vl (fastest over the lanes), rows vi, vi + vrows, ...
    const int vt = tid - 64 * (jw.rot + jw.blocks), vrows = (mm + kVRows - 1) / kVRows;
    const int vl = vt % np, vi = vt / np;
    const bool act = vi < vrows;
    Pair vp;
    double va[kVRows], vb[kVRows];
    sweeps([&] { vp = Pair(mm, 0, vl); },
           [&] {
#pragma unroll
             for (int r = 0; r < kVRows; ++r) {
               const int i = min(vi + r * vrows, mm - 1) * mm;
               va[r] = v[i + vp.a];
               vb[r] = v[i + vp.b];
             }
           },
           [&] {
             const double2 c = cs[vl];
#pragma unroll
             for (int r = 0; r < kVRows; ++r) {
               const int i = vi + r * vrows;
               if (act && i < mm) {
                 v[i * mm + vp.a] = c.x * va[r] - c.y * vb[r];
                 v[i * mm + vp.b] = c.y * va[r] + c.x * vb[r];
               }
             }
             vp.step(mm);
           });
  }
  // the sweep that ended the loop is all identity and not recorded
  if constexpr (VEC == kVecRecord)
    if (tid == 0) o.info[0] = sweep * (mm - 1);
  jacobi_sorted<VEC>(m, o, [&](int j) { return a[j * S + j]; }, v, mm);
}

// mm <= 192: the upper triangle packed (148 KB at 192), a_ij at off(i) + j, i <= j.
// Bound by LDS access here, so blocks are read only when their rotations are known,
// and a pair's indices and row offsets come from LDS with them.
template <int VEC>
__device__ __forceinline__ void jacobi_packed(int m, const double* __restrict__ A, int64_t lda,
                                              const JacobiOut& o) {
  extern __shared__ __align__(16) double sh[];
  __shared__ int rotated[2];
  constexpr int NB = 5;  // 96 * 97 / 2 blocks <= 5 * 1024
  const int mm = m + (m & 1), np = mm / 2;
  double2* cs = reinterpret_cast<double2*>(sh);   // rotation of each pair
  int4* pr = reinterpret_cast<int4*>(cs + np);    // its p < q and their row offsets
  double* a = reinterpret_cast<double*>(pr + np);
  const int tid = threadIdx.x, nt = blockDim.x;
  auto off = [&](int i) { return i * mm - ((i * (i + 1)) >> 1); };
  for (int e = tid; e < mm * mm; e += nt) {
    const int i = e / mm, j = e - i * mm;
    if (i <= j) a[off(i) + j] = j < m ? A[(int64_t)i * lda + j] : 0.0;
  }
  const int nb = np * (np + 1) / 2;
  int bk[NB], bl[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) block_of(tid + t * nt, np, &bk[t], &bl[t]);
  if (tid < 2) rotated[tid] = 0;
  __syncthreads();
  int sweep = 0;
  for (; sweep < kMaxSweeps; ++sweep) {
    int* flag = &rotated[sweep & 1];
    for (int round = 0; round < mm - 1; ++round) {
      if (tid < np) {
        const Pair t(mm, round, tid);
        const int p = min(t.a, t.b), q = max(t.a, t.b), op = off(p), oq = off(q);
        double c, s;
        if (rotation(a[op + p], a[oq + q], a[op + q], false, &c, &s)) *flag = 1;
        cs[tid] = make_double2(c, s);
        pr[tid] = make_int4(p, q, op, oq);
        if constexpr (VEC == kVecRecord)
          o.rec[((int64_t)sweep * (mm - 1) + round) * np + tid] =
              make_double2(c, t.a > t.b ? -s : s);
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        if (tid + t * nt >= nb) continue;
        const int4 P = pr[bk[t]], Q = pr[bl[t]];
        const double2 ck = cs[bk[t]], cl = cs[bl[t]];
        auto at = [&](int i, int oi, int j, int oj) { return i <= j ? oi + j : oj + i; };
        const int ipp = at(P.x, P.z, Q.x, Q.z), ipq = at(P.x, P.z, Q.y, Q.w);
        const int iqp = at(P.y, P.w, Q.x, Q.z), iqq = at(P.y, P.w, Q.y, Q.w);
        double bpp = a[ipp], bpq = a[ipq], bqp = a[iqp], bqq = a[iqq];
        rot_block(ck.x, ck.y, cl.x, cl.y, bpp, bpq, bqp, bqq);
        const bool diag = bk[t] == bl[t];
        a[ipp] = bpp;
        a[iqq] = bqq;
        a[ipq] = diag ? 0.0 : bpq;
        a[iqp] = diag ? 0.0 : bqp;
      }
      __syncthreads();
    }
    const bool more = *flag != 0;
    if (tid == 0) rotated[1 - (sweep & 1)] = 0;
    __syncthreads();
    if (!more) break;
  }
  if constexpr (VEC == kVecRecord)
    if (tid == 0) o.info[0] = sweep * (mm - 1);
  jacobi_sorted<VEC>(m, o, [&](int j) { return a[off(j) + j]; }, nullptr, mm);
}

// NB = 0: the packed form.
template <int VEC, int NB>
__device__ __forceinline__ void jacobi_body(int m, const double* __restrict__ A, int64_t lda,
                                            const JacobiOut& o, const JacobiWaves& jw) {
  if constexpr (NB == 0)
    jacobi_packed<VEC>(m, A, lda, o);
  else
    jacobi_square<VEC, NB>(m, A, lda, o, jw);
}

template <int VEC, int NB>
__global__ __launch_bounds__(1024) void k_jacobi_lds(int m, const double* __restrict__ A,
                                                     int64_t lda, JacobiOut o, JacobiWaves jw) {
  jacobi_body<VEC, NB>(m, A, lda, o, jw);
}

// Eigenvalues of many matrices, one workgroup each (EighItem).
template <int NB>
__global__ __launch_bounds__(1024) void k_jacobi_values(const double* __restrict__ A,
                                                        const EighItem* __restrict__ items,
                                                        double* __restrict__ w, JacobiWaves jw) {
  const EighItem t = items[blockIdx.x];
  JacobiOut o{};
  o.w = w + t.w_at;
  jacobi_body<kVecNone, NB>(t.dim, A + t.a_at, t.dim, o, jw);
}

// V from the recorded rotations: one wavefront applies all of them to its row of the
// identity, then stores the row in the order of the eigenvalues.  Bound by the latency of
// the records and the wavefront's issue: m = 192 takes 460 us with one row per wavefront and
// 8 rounds on their way, 790 with one round, 830 with four rows and one round, 850 with
// four rows and 8 rounds (m = 96: 181, 330, 278, 276).
constexpr int kVecRows = 1;
constexpr int kVecAhead = 8;
__global__ __launch_bounds__(64) void k_jacobi_vectors(int m, const double2* __restrict__ rec,
                                                       const int* __restrict__ info,
                                                       double* __restrict__ V, int64_t ldv) {
  __shared__ double v[kVecRows][kLdsMax];
  const int mm = m + (m & 1), np = mm / 2, lane = threadIdx.x;
  const int row0 = blockIdx.x * kVecRows;
  for (int e = lane; e < kVecRows * mm; e += 64) {
    const int r = e / mm, j = e - r * mm;
    v[r][j] = row0 + r == j ? 1.0 : 0.0;
  }
  const int rounds = info[0];
  constexpr int kL = (kLdsMax / 2 + 63) / 64;  // pairs per lane
  double2 next[kVecAhead][kL];
  auto fetch = [&](int rd0) {
#pragma unroll
    for (int d = 0; d < kVecAhead; ++d)
#pragma unroll
      for (int t = 0; t < kL; ++t) {
        const int l = lane + 64 * t;
        next[d][t] = l < np && rd0 + d < rounds ? rec[(int64_t)(rd0 + d) * np + l]
                                                : make_double2(1.0, 0.0);
      }
  };
  Pair pair[kL] = {Pair(mm, 0, min(lane, np - 1)), Pair(mm, 0, min(lane + 64, np - 1))};
  static_assert(kL == 2, "pairs per lane");
  if (rounds > 0) fetch(0);
  __syncthreads();
  for (int rd = 0; rd < rounds; rd += kVecAhead) {
    double2 cur[kVecAhead][kL];
#pragma unroll
    for (int d = 0; d < kVecAhead; ++d)
#pragma unroll
      for (int t = 0; t < kL; ++t) cur[d][t] = next[d][t];
    fetch(rd + kVecAhead);
#pragma unroll
    for (int d = 0; d < kVecAhead; ++d) {
#pragma unroll
      for (int t = 0; t < kL; ++t) {
        const double2 c = cur[d][t];
        if (lane + 64 * t < np && c.y != 0.0) {  // rounds beyond the last rotate nothing
          const int p = pair[t].a, q = pair[t].b;
#pragma unroll
          for (int r = 0; r < kVecRows; ++r) {
            const double vp = v[r][p], vq = v[r][q];
            v[r][p] = c.x * vp - c.y * vq;
            v[r][q] = c.y * vp + c.x * vq;
          }
        }
        pair[t].step(mm);
      }
      __syncthreads();  // one wavefront: orders its LDS accesses
    }
  }
  for (int e = lane; e < kVecRows * m; e += 64) {
    const int r = e / m, j = e - r * m;
    if (row0 + r < m) V[(int64_t)(row0 + r) * ldv + info[1 + j]] = v[r][j];
  }
}

// Multi-kernel Jacobi: one launch per round.
__global__ __launch_bounds__(256) void k_jacobi_round(int mm, int round,
                                                      const double* __restrict__ ain,
                                                      double* __restrict__ aout,
                                                      double* __restrict__ v,
                                                      int* __restrict__ nrot) {
  const int np = mm / 2;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nblk = (int64_t)np * np;
  if (e < nblk) {
    const int k = (int)(e / np), l = (int)(e % np);
    int pk, qk, pl, ql;
    pair_of(mm, round, k, &pk, &qk);
    pair_of(mm, round, l, &pl, &ql);
    double ck, sk, cl, sl;
    const bool rk = rotation(ain[pk * mm + pk], ain[qk * mm + qk], ain[pk * mm + qk], false, &ck, &sk);
    rotation(ain[pl * mm + pl], ain[ql * mm + ql], ain[pl * mm + ql], false, &cl, &sl);
    if (k == l && rk) atomicAdd(nrot, 1);
    double bpp = ain[pk * mm + pl], bpq = ain[pk * mm + ql], bqp = ain[qk * mm + pl],
           bqq = ain[qk * mm + ql];
    rot_block(ck, sk, cl, sl, bpp, bpq, bqp, bqq);
    if (k == l) {
      bpq = 0.0;
      bqp = 0.0;
    }
    aout[pk * mm + pl] = bpp;
    aout[pk * mm + ql] = bpq;
    aout[qk * mm + pl] = bqp;
    aout[qk * mm + ql] = bqq;
  } else if (e < nblk + (int64_t)mm * np) {
    const int64_t f = e - nblk;
    const int i = (int)(f / np), l = (int)(f % np);
    int pl, ql;
    pair_of(mm, round, l, &pl, &ql);
    double cl, sl;
    rotation(ain[pl * mm + pl], ain[ql * mm + ql], ain[pl * mm + ql], false, &cl, &sl);
    const double vp = v[i * mm + pl], vq = v[i * mm + ql];
    v[i * mm + pl] = cl * vp - sl * vq;
    v[i * mm + ql] = sl * vp + cl * vq;
  }
}

__global__ __launch_bounds__(256) void k_jacobi_init(int m, int mm, const double* __restrict__ A,
                                                     int64_t lda, double* __restrict__ a,
                                                     double* __restrict__ v) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)mm * mm) return;
  const int i = (int)(e / mm), j = (int)(e % mm);
  const int u = min(i, j), x = max(i, j);  // symmetrise from the upper triangle
  a[e] = (x < m) ? A[(int64_t)u * lda + x] : 0.0;
  v[e] = (i == j) ? 1.0 : 0.0;
}

__global__ __launch_bounds__(256) void k_jacobi_sort(int m, int mm, const double* __restrict__ a,
                                                     const double* __restrict__ v,
                                                     double* __restrict__ w,
                                                     double* __restrict__ V, int64_t ldv) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= m) return;
  const double dj = a[(int64_t)j * mm + j];
  int r = 0;
  for (int i = 0; i < m; ++i) {
    const double di = a[(int64_t)i * mm + i];
    r += (di < dj) || (di == dj && i < j);
  }
  w[r] = dj;
  for (int i = 0; i < m; ++i) V[(int64_t)i * ldv + r] = v[(int64_t)i * mm + j];
}

// Cholesky with dropping (row-oriented) and inverse of R on the kept columns.
// G: b x b (upper triangle read).  Outputs Rinv_c (b x b, ld b; column jc is
// the jc-th kept column of R^-1, other columns zero) and *count.  R and R^-1
// live in LDS when in_lds (b <= kCholLds), else in global memory (R in the
// work buffer).  R^-1 is built one row at a time from the bottom, every
// thread owning columns, so each step is parallel over the columns.
constexpr int kCholLds = 88;  // 2 b^2 doubles + the static arrays fit 160 KB of LDS

__global__ __launch_bounds__(1024) void k_chol_drop(int b, const double* __restrict__ G,
                                                    int64_t ldg, double tol, int in_lds,
                                                    double* __restrict__ Rg,
                                                    double* __restrict__ Rinv,
                                                    int* __restrict__ count) {
  extern __shared__ double shm[];
  __shared__ int keep[1024];
  __shared__ int pos[1024];
  __shared__ double row[1024];
  __shared__ double rjj;
  const int tid = threadIdx.x, nt = blockDim.x;
  double* R = in_lds ? shm : Rg;
  double* Ri = in_lds ? shm + b * b : Rinv;
  // row j of R holds row j of G until it is formed; rows not kept become zero, and so do,
  // before the inverse, the entries of R in columns not kept: the sums need no branch
  for (int e = tid; e < b * b; e += nt) {
    R[e] = e % b >= e / b ? G[(int64_t)(e / b) * ldg + e % b] : 0.0;
    Ri[e] = 0.0;
  }
  __syncthreads();
  for (int j = 0; j < b; ++j) {
    for (int l = j + tid; l < b; l += nt) {
      double g = R[j * b + l];
#pragma unroll 8
      for (int k = 0; k < j; ++k) g -= R[k * b + j] * R[k * b + l];
      row[l] = g;
    }
    __syncthreads();
    if (tid == 0) {
      const double gjj = R[j * b + j];
      const double d = row[j];
      keep[j] = (gjj > 0.0) && (d > tol * gjj) && isfinite(d);
      rjj = keep[j] ? sqrt(d) : 0.0;
    }
    __syncthreads();
    for (int l = j + tid; l < b; l += nt) R[j * b + l] = keep[j] ? row[l] / rjj : 0.0;
    __syncthreads();
  }
  if (tid == 0) {
    int c = 0;
    for (int j = 0; j < b; ++j) {
      pos[j] = c;
      c += keep[j];
    }
    *count = c;
  }
  for (int e = tid; e < b * b; e += nt)
    if (!keep[e % b]) R[e] = 0.0;
  __syncthreads();
  // row i of R^-1 (kept columns only) from the rows below it
  for (int i = b - 1; i >= 0; --i) {
    if (keep[i]) {
      const double rii = R[i * b + i];
      for (int j = i + tid; j < b; j += nt) {
        if (!keep[j]) continue;
        const int jc = pos[j];
        if (j == i) {
          Ri[i * b + jc] = 1.0 / rii;
          continue;
        }
        double s = 0.0;
#pragma unroll 8
        for (int k = i + 1; k <= j; ++k) s += R[i * b + k] * Ri[k * b + jc];
        Ri[i * b + jc] = -s / rii;
      }
    }
    __syncthreads();
  }
  if (in_lds)
    for (int e = tid; e < b * b; e += nt) Rinv[e] = Ri[e];
}

// ritz_project by one workgroup, with C, Ch and T1 in LDS.
__global__ __launch_bounds__(1024) void k_ritz_project(int m, int b, const double* __restrict__ V,
                                                       double* __restrict__ C, int64_t ldc,
                                                       double* __restrict__ Chg,
                                                       double* __restrict__ T1g) {
  extern __shared__ double shm[];
  double* Cs = shm;          // [m][b]
  double* Ch = Cs + m * b;   // [m][b]
  double* T1 = Ch + m * b;   // [b][b]
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int e = tid; e < m * b; e += nt) {
    const int i = e / b, j = e - i * b;
    const double v = V[(int64_t)i * m + j];
    Cs[e] = v;
    Ch[e] = i < b ? 0.0 : v;
    C[(int64_t)i * ldc + j] = v;
  }
  __syncthreads();
  auto gram = [&](const double* A) {  // T1 = A^T Ch
    for (int e = tid; e < b * b; e += nt) {
      const int i = e / b, j = e - i * b;
      double s = 0.0;
#pragma unroll 4
      for (int k = 0; k < m; ++k) s += A[k * b + i] * Ch[k * b + j];
      T1[e] = s;
    }
    __syncthreads();
  };
  for (int pass = 0; pass < 2; ++pass) {
    gram(Cs);
    for (int e = tid; e < m * b; e += nt) {  // Ch -= C T1
      const int i = e / b, j = e - i * b;
      double s = 0.0;
#pragma unroll 4
      for (int k = 0; k < b; ++k) s += Cs[i * b + k] * T1[k * b + j];
      Ch[e] -= s;
    }
    __syncthreads();
  }
  gram(Ch);
  for (int e = tid; e < m * b; e += nt) Chg[e] = Ch[e];
  for (int e = tid; e < b * b; e += nt) T1g[e] = T1[e];
}

// C = alpha op(A) op(B) + beta C for small row-major FP64 matrices.
__global__ __launch_bounds__(256) void k_small_gemm(int M, int N, int K, double alpha,
                                                    const double* __restrict__ A, int64_t lda,
                                                    int ta, const double* __restrict__ B,
                                                    int64_t ldb, int tb, double beta,
                                                    double* __restrict__ C, int64_t ldc) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)M * N) return;
  const int i = (int)(e / N), j = (int)(e % N);
  double s = 0.0;
  for (int k = 0; k < K; ++k) {
    const double av = ta ? A[(int64_t)k * lda + i] : A[(int64_t)i * lda + k];
    const double bv = tb ? B[(int64_t)j * ldb + k] : B[(int64_t)k * ldb + j];
    s += av * bv;
  }
  C[(int64_t)i * ldc + j] = alpha * s + (beta == 0.0 ? 0.0 : beta * C[(int64_t)i * ldc + j]);
}

__global__ __launch_bounds__(256) void k_gather_cols(int rows, int nsel, const int* __restrict__ sel,
                                                     const double* __restrict__ Z, int64_t ldz,
                                                     double* __restrict__ out, int64_t ldo) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)rows * nsel) return;
  const int i = (int)(e / nsel), j = (int)(e % nsel);
  out[(int64_t)i * ldo + j] = Z[(int64_t)i * ldz + sel[j]];
}

inline unsigned g1(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// Non-decreasing in m: a workspace for the largest size serves every smaller one, though
// the sizes to kLdsMax need more (every round's rotations, their number and the column
// order) than some above it (two copies of A and V).
size_t small_eigh_work_bytes(int m) {
  const int64_t mm = m + (m & 1), lm = std::min<int64_t>(mm, kLdsMax);
  return std::max((size_t)(3 * mm * mm) * sizeof(double),
                  (size_t)kMaxSweeps * (lm - 1) * (lm / 2) * sizeof(double2) +
                      (size_t)(lm + 1) * sizeof(int)) +
         256;
}

namespace {

template <class K, class... Args>
void launch_jacobi_lds(K kernel, int count, int mm, bool vec, hipStream_t s, Args... args) {
  const size_t shm = jacobi_lds_bytes(mm, vec);
  MBL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
  const JacobiWaves jw = jacobi_waves(mm, vec);
  hipLaunchKernelGGL(kernel, dim3(count), dim3(jw.threads()), shm, s, args..., jw);
  MBL_CHECK_LAUNCH();
}

// Blocks per thread of the square form, 0: the packed form.
template <class F>
void by_blocks(int mm, F&& f) {
  const int bt = 64 * jacobi_waves(mm, false).blocks, per = (jacobi_blocks(mm) + bt - 1) / bt;
  if (mm > kSquareMax)
    f(std::integral_constant<int, 0>{});
  else if (per <= 1)
    f(std::integral_constant<int, 1>{});
  else if (per <= 2)
    f(std::integral_constant<int, 2>{});
  else
    f(std::integral_constant<int, 3>{});
}

}  // namespace

void eigh_values(int count, int max_dim, const double* A, const EighItem* items_dev, double* w,
                 hipStream_t s) {
  if (count == 0) return;
  const int mm = max_dim + (max_dim & 1);
  if (mm > kLdsMax) fail(MBL_EINTERNAL, "eigh_values: matrix too large");
  by_blocks(mm, [&](auto nb) {
    launch_jacobi_lds(&k_jacobi_values<decltype(nb)::value>, count, mm, false, s, A, items_dev, w);
  });
}

void small_eigh(int m, const double* A, int64_t lda, double* w, double* V, int64_t ldv,
                const DevBuf& workspace, hipStream_t s) {
  PhaseTick tick(PhaseClock::SMALL, s);
  if (m <= 0) return;
  if (workspace.bytes() < small_eigh_work_bytes(m))
    fail(MBL_EINTERNAL, "small_eigh: workspace too small");
  double* work = workspace.as<double>();
  const int mm = m + (m & 1);
  const int max_sweeps = kMaxSweeps;
  if (m == 1) {
    MBL_HIP(hipMemcpyAsync(w, A, sizeof(double), hipMemcpyDeviceToDevice, s));
    if (V) {
      const double one = 1.0;
      MBL_HIP(hipMemcpyAsync(V, &one, sizeof(double), hipMemcpyHostToDevice, s));
      MBL_HIP(hipStreamSynchronize(s));
    }
    return;
  }
  if (mm <= kLdsMax) {
    JacobiOut o{};
    o.w = w;
    o.V = V;
    o.ldv = ldv;
    if (V && mm <= kInlineMax) {
      launch_jacobi_lds(&k_jacobi_lds<kVecInline, 1>, 1, mm, true, s, m, A, lda, o);
      return;
    }
    if (V) {
      o.rec = reinterpret_cast<double2*>(work);
      o.info = reinterpret_cast<int*>(o.rec + (size_t)kMaxSweeps * (mm - 1) * (mm / 2));
    }
    by_blocks(mm, [&](auto nb) {
      constexpr int NB = decltype(nb)::value;
      if (V)
        launch_jacobi_lds(&k_jacobi_lds<kVecRecord, NB>, 1, mm, false, s, m, A, lda, o);
      else
        launch_jacobi_lds(&k_jacobi_lds<kVecNone, NB>, 1, mm, false, s, m, A, lda, o);
    });
    if (V) {
      hipLaunchKernelGGL(k_jacobi_vectors, dim3((m + kVecRows - 1) / kVecRows), dim3(64), 0, s, m,
                         o.rec, o.info, V, ldv);
      MBL_CHECK_LAUNCH();
    }
    return;
  }
  if (!V) fail(MBL_EINTERNAL, "small_eigh: eigenvectors are needed above 192");
  double* a0 = work;
  double* a1 = work + (size_t)mm * mm;
  double* v = work + (size_t)2 * mm * mm;
  int* nrot = reinterpret_cast<int*>(work + (size_t)3 * mm * mm);
  hipLaunchKernelGGL(k_jacobi_init, dim3(g1((int64_t)mm * mm)), dim3(256), 0, s, m, mm, A, lda,
                     a0, v);
  MBL_CHECK_LAUNCH();
  const int np = mm / 2;
  const int64_t threads = (int64_t)np * np + (int64_t)mm * np;
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    MBL_HIP(hipMemsetAsync(nrot, 0, sizeof(int), s));
    for (int round = 0; round < mm - 1; ++round) {
      hipLaunchKernelGGL(k_jacobi_round, dim3(g1(threads)), dim3(256), 0, s, mm, round, a0, a1, v,
                         nrot);
      MBL_CHECK_LAUNCH();
      std::swap(a0, a1);
    }
    int h_nrot = 0;
    MBL_HIP(hipMemcpyAsync(&h_nrot, nrot, sizeof(int), hipMemcpyDeviceToHost, s));
    MBL_HIP(hipStreamSynchronize(s));
    if (h_nrot == 0) break;
  }
  hipLaunchKernelGGL(k_jacobi_sort, dim3(g1(m)), dim3(256), 0, s, m, mm, a0, v, w, V, ldv);
  MBL_CHECK_LAUNCH();
}

// Cholesky-with-dropping of a b x b Gram; returns the number of kept columns.
int chol_drop(int b, const double* G, int64_t ldg, double tol, double* Rinv, double* work,
              int* dcount, hipStream_t s) {
  PhaseTick tick(PhaseClock::SMALL, s);
  if (b <= 0) return 0;
  if (b > 1024) fail(MBL_EINVAL, "chol_drop: b > 1024");
  const int in_lds = b <= kCholLds;
  const size_t shm = in_lds ? (size_t)2 * b * b * sizeof(double) : 0;
  if (in_lds)
    MBL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_chol_drop),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
  // A column per thread, so few wavefronts at the many barriers; with G read ahead of the
  // row loop 18 us (b = 4 and 32 mixed, as in a solve of block 32), before 30.
  const int nt = in_lds ? (b + 63) / 64 * 64 : 1024;
  hipLaunchKernelGGL(k_chol_drop, dim3(1), dim3(nt), shm, s, b, G, ldg, tol, in_lds, work, Rinv,
                     dcount);
  MBL_CHECK_LAUNCH();
  int c = 0;
  MBL_HIP(hipMemcpyAsync(&c, dcount, sizeof(int), hipMemcpyDeviceToHost, s));
  MBL_HIP(hipStreamSynchronize(s));
  return c;
}

void small_gemm(int M, int N, int K, double alpha, const double* A, int64_t lda, bool ta,
                const double* B, int64_t ldb, bool tb, double beta, double* C, int64_t ldc,
                hipStream_t s) {
  PhaseTick tick(PhaseClock::SMALL, s);
  if ((int64_t)M * N == 0) return;
  hipLaunchKernelGGL(k_small_gemm, dim3(g1((int64_t)M * N)), dim3(256), 0, s, M, N, K, alpha, A,
                     lda, (int)ta, B, ldb, (int)tb, beta, C, ldc);
  MBL_CHECK_LAUNCH();
}

// In LDS up to 64 KB (b = 34 at m = 3b; m = 96, b = 32: one launch of 20 us, m = 12, b = 4 one
// of 5, for three copies and five products of 4 each and the gaps between them), else by the
// general products.
void ritz_project(int m, int b, const double* V, double* C, int64_t ldc, double* Ch, double* T1,
                  hipStream_t s) {
  const size_t lds = ((size_t)2 * m * b + (size_t)b * b) * sizeof(double);
  if (lds <= 64 * 1024) {
    PhaseTick tick(PhaseClock::SMALL, s);
    const int nt = std::min(1024, (m * b + 63) / 64 * 64);
    hipLaunchKernelGGL(k_ritz_project, dim3(1), dim3(nt), lds, s, m, b, V, C, ldc, Ch, T1);
    MBL_CHECK_LAUNCH();
    return;
  }
  MBL_HIP(hipMemcpy2DAsync(C, ldc * sizeof(double), V, m * sizeof(double), b * sizeof(double), m,
                           hipMemcpyDeviceToDevice, s));
  MBL_HIP(hipMemcpy2DAsync(Ch, b * sizeof(double), V, m * sizeof(double), b * sizeof(double), m,
                           hipMemcpyDeviceToDevice, s));
  MBL_HIP(hipMemsetAsync(Ch, 0, (size_t)b * b * sizeof(double), s));
  for (int pass = 0; pass < 2; ++pass) {
    small_gemm(b, b, m, 1.0, C, ldc, true, Ch, b, false, 0.0, T1, b, s);
    small_gemm(m, b, b, -1.0, C, ldc, false, T1, b, false, 1.0, Ch, b, s);
  }
  small_gemm(b, b, m, 1.0, Ch, b, true, Ch, b, false, 0.0, T1, b, s);
}

void gather_cols(int rows, int nsel, const int* sel, const double* Z, int64_t ldz, double* out,
                 int64_t ldo, hipStream_t s) {
  if ((int64_t)rows * nsel == 0) return;
  hipLaunchKernelGGL(k_gather_cols, dim3(g1((int64_t)rows * nsel)), dim3(256), 0, s, rows, nsel,
                     sel, Z, ldz, out, ldo);
  MBL_CHECK_LAUNCH();
}

}  // namespace mbl
