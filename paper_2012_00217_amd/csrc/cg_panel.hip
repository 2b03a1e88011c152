// Block Jacobi-PCG on the spectral fold with panel-major vectors, for sectors
// whose CG vectors leave the caches (paper Sec. 3.2 and 4.1).
//
// What bounds it.  Beyond the 4 MB L2 of an XCD every read costs the same: a
// plain read loop measures 32 TB/s while each XCD's working set stays within
// 4 MB and 6.9-7.1 TB/s above that, whether the data sits in the last-level
// cache or in HBM.  So only bytes that miss the L2 count, and a gather of row-major
// rows misses for every bond whose target lies outside the few thousand rows that
// an L2 holds: about 6.5 fetches of the gathered vector per apply at L = 24.
//
// Layout.  The CG vectors are kept as panels of one 16-byte vector per row
// (2 FP64 or 4 FP32 columns): panel j holds its columns of all n rows
// contiguously.  Each XCD works on panels of its own, so its L2 spans 8 to 16 times
// more rows than with whole rows shared by all XCDs, and every gather of
// consecutive rows stays a run of whole lines.
//
// Work.  The chain is cut at q = 12 sites; the rows that share the high
// configuration hi are a contiguous block (at most C(12, 6) = 924 rows, one tile).
//   * flips inside the low half stay in the block: gathered from LDS through a
//     table of byte offsets per low configuration (unused slots point at a zero
//     row, so there are no branches);
//   * a flip inside hi maps the block row for row onto another block, at one
//     offset for the whole tile: an unmasked contiguous load with a scalar base;
//   * the middle bond maps a contiguous part of the block onto part of hi ^ 1.
// Diagonal and Jacobi entries come from the two halves' energies, so no n-length
// table is read.
//
// One step: T = (H - sigma) p and |T|^2; alpha; r -= alpha (H - sigma) T and
// r.M^-1 r; beta; x += alpha p, p = M^-1 r + beta p.  x stays in the caller's
// row-major block: its update runs in the p update, which is elementwise and takes
// whole rows of all panels, and the applies read and write only what they gather.
#include <algorithm>
#include <cmath>

#include "cg_replay.h"
#include "common.h"

namespace mbl {
namespace {

constexpr int kPThreads = 256;
constexpr int kPWaves = kPThreads / 64;
constexpr int kPanelQ = 12;       // low half: blocks of at most 924 rows
constexpr int kPanelRows = 924;
constexpr int kPanelMinRows = 13312;
constexpr int kPanelMeanRows = 256;  // of a tile
constexpr int kPanelMaxHigh = 16;  // longest high half (L = 28)
constexpr int kMaxHigh = 18;       // of the apply's tiles (L = 28)

template <class T>
struct PV;
template <>
struct PV<double> {
  typedef double type __attribute__((ext_vector_type(2)));
};
template <>
struct PV<float> {
  typedef float type __attribute__((ext_vector_type(4)));
};

template <class T>
struct PanelArgs {
  const PanelTile* tiles;
  const uint4* lo_tab;   // per low configuration: LDS rows of its flips, their number
  const double* lo_E;
  const T* X;            // gathered vector
  T* Y;                  // apply1: T
  T* r;                  // apply2
  const PcgCoef* coef;   // apply2: alpha
  double* part;          // [column][tile]
  int* next;             // per XCD (32 ints apart): tiles taken so far
  int64_t n;
  double sigma, halfJ, zz4;
  PanelSched ts;
};

enum { PAN_NORM2 = 0, PAN_RUPD = 1 };

template <class T, bool kNt = false>
__device__ inline typename PV<T>::type pload(const T* base, uint32_t off) {
  const auto* p = reinterpret_cast<const typename PV<T>::type*>(reinterpret_cast<const char*>(base) + off);
  if constexpr (kNt) return __builtin_nontemporal_load(p);
  return *p;
}

// Sum over the wavefront of VE values per lane.  Lanes that differ in the low
// log2(VE) bits first share out the columns (each keeps half of its values and
// takes its partner's for those), so the rest of the butterfly carries one
// value: lane e ends with the sum of column col_of(e).
template <int VE>
__device__ inline double wave_cols(const double (&v)[VE]) {
  const int lane = threadIdx.x & 63;
  double s;
  if constexpr (VE == 4) {
    const bool h = lane & 2, l = lane & 1;
    double a = h ? v[2] : v[0], b = h ? v[3] : v[1];
    a += __shfl_xor(h ? v[0] : v[2], 2);
    b += __shfl_xor(h ? v[1] : v[3], 2);
    s = (l ? b : a) + __shfl_xor(l ? a : b, 1);
  } else {
    const bool l = lane & 1;
    s = (l ? v[1] : v[0]) + __shfl_xor(l ? v[0] : v[1], 1);
  }
#pragma unroll
  for (int off = VE; off < 64; off <<= 1) s += __shfl_xor(s, off);
  return s;  // column lane % VE
}

// One workgroup takes tiles of its XCD (in order, from a counter that the fold
// kernel before it has cleared) until none is left: the tiles in flight stay
// together in the row order, which keeps their common neighbours in the L2.  Each
// tile has its own partial sums, so the result does not depend on who took it.
//
// Bound: bytes that miss the L2, at the rate of a copy.  Measured with 64 FP32 columns at
// L = 24 (n = 2,704,156, 692 MB per vector): the tiles fetch 1.72 GB per apply1, 2.5
// times the gathered vector, in 558 us (with the 0.72 GB written 4.4 TB/s; a copy reaches
// 4.9).  In row order they fetch 2.07 GB (590 us); dealt out in a fixed stride, where
// workgroups with small tiles run ahead, 3.5 GB; the row-major gather 4.6 GB.  Fewer or
// larger workgroups in flight (4 of 256, 4 of 512 threads per CU) and blocks of q = 11 or
// 10 are slower (590 and 553, 600 and 700 us; the second apply 710 and 771, 735 and
// 852 against 662), eight loads of the high half at once give nothing.
template <class T, int EPI, int NT>
__global__ __launch_bounds__(NT) void k_panel(PanelArgs<T> a) {
  using V = typename PV<T>::type;
  constexpr int VE = 16 / (int)sizeof(T);
  __shared__ V tile[kPanelRows + 1];  // row u at tile[u + 1]; tile[0] stays zero
  __shared__ double sred[NT / 64][VE];
  __shared__ int snext;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xcd = blockIdx.x & 7;
  const int first = a.ts.first[xcd], last = a.ts.first[xcd + 1];
  int* next = a.next + xcd * 32;
  const T hj = (T)a.halfJ;
  if (tid == 0) {
    tile[0] = V(0);
    snext = first + atomicAdd(next, 1);
  }
  __syncthreads();
  int lt = __builtin_amdgcn_readfirstlane(snext);

  while (lt < last) {
    int nx = 0;
    if (tid == 0) nx = first + atomicAdd(next, 1);  // the tile after this one
    const int panel = lt / a.ts.ntiles, t = lt - panel * a.ts.ntiles;
    const int64_t pbase = (int64_t)panel * a.n * VE;
    const T* X = a.X + pbase;
    const MBL_CONST PanelTile* tp = (const MBL_CONST PanelTile*)a.tiles + t;
    const int nr = tp->nrows, row0 = tp->row0, cnt = tp->cnt, aux = tp->aux;
    const int mlo = tp->mlo, mhi = tp->mhi;
    for (int u = tid; u < nr; u += NT) tile[u + 1] = pload<T>(X, (uint32_t)(row0 + u) * 16u);
    T alpha[VE];
    if constexpr (EPI == PAN_RUPD) {
      const MBL_CONST PcgCoef* cf = (const MBL_CONST PcgCoef*)a.coef + panel * VE;
#pragma unroll
      for (int e = 0; e < VE; ++e) alpha[e] = (T)cf[e].alpha;
    }
    double red[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) red[e] = 0.0;
    const char* tb = reinterpret_cast<const char*>(tile);
    __syncthreads();
    for (int u0 = wave * 64; u0 < nr; u0 += NT) {
      // Lanes past the last row repeat it (so that loads are unconditional) and
      // store nothing.
      const int ul = u0 + lane, u = min(ul, nr - 1);
      const uint32_t vo = (uint32_t)(row0 + u) * 16u;
      const uint4 f = a.lo_tab[aux + u];
      const double El = a.lo_E[aux + u];
      V rv, vm;
      if constexpr (EPI == PAN_RUPD) rv = pload<T, true>(a.r + pbase, vo);
      // middle bond: rows [mlo, mhi) map to rows mbase + u of the block hi ^ 1
      const bool mid = u >= mlo && u < mhi;
      const bool anymid = u0 < mhi && u0 + 63 >= mlo;  // the same for the wavefront
      if (anymid)
        vm = pload<T>(X + (int64_t)tp->mbase * VE, (uint32_t)min(max(u, mlo), mhi - 1) * 16u);
      // flips inside the high half: one offset for the whole tile
      V s = V(0);
      auto batch = [&](int h, auto n_) {
        constexpr int N = decltype(n_)::value;
        V v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = pload<T>(X + (int64_t)tp->off[h + i] * VE, vo);
#pragma unroll
        for (int i = 0; i < N; ++i) s += v[i];
      };
      int h = 0;
      for (; h + 4 <= cnt; h += 4) batch(h, std::integral_constant<int, 4>{});
      if (h + 2 <= cnt) {
        batch(h, std::integral_constant<int, 2>{});
        h += 2;
      }
      if (h < cnt) batch(h, std::integral_constant<int, 1>{});
      if (anymid) {
#pragma unroll
        for (int e = 0; e < VE; ++e) s[e] += mid ? vm[e] : (T)0;
      }
      const int ndl = (int)(f.w >> 28);
      auto flip = [&](uint32_t w, int k) {
        s += *reinterpret_cast<const V*>(tb + ((w >> (10 * k)) & 1023u) * 16u);
      };
      flip(f.x, 0);
      flip(f.x, 1);
      flip(f.x, 2);
      if (__any(ndl > 3)) {
        flip(f.y, 0);
        flip(f.y, 1);
        flip(f.y, 2);
      }
      if (__any(ndl > 6)) {
        flip(f.z, 0);
        flip(f.z, 1);
        flip(f.z, 2);
      }
      if (__any(ndl > 9)) {
        flip(f.w, 0);
        flip(f.w, 1);
      }
      const V own = tile[u + 1];
      const double e0 = ((El + tp->E) + (mid ? -a.zz4 : a.zz4)) - a.sigma;
      const T ed = (T)e0;
      V y;
#pragma unroll
      for (int e = 0; e < VE; ++e) y[e] = ed * own[e] + hj * s[e];
      if constexpr (EPI == PAN_NORM2) {
        if (ul < nr) {
          __builtin_nontemporal_store(
              y, reinterpret_cast<V*>(reinterpret_cast<char*>(a.Y + pbase) + vo));
#pragma unroll
          for (int e = 0; e < VE; ++e) red[e] += (double)y[e] * (double)y[e];
        }
      } else {
        const int nd = ndl + tp->nd + (mid ? 1 : 0);
        const T dinv = (T)1 / (T)(e0 * e0 + a.halfJ * a.halfJ * (double)nd);
        if (ul < nr) {
#pragma unroll
          for (int e = 0; e < VE; ++e) {
            rv[e] = rv[e] - alpha[e] * y[e];
            red[e] += (double)rv[e] * (double)(rv[e] * dinv);
          }
          __builtin_nontemporal_store(
              rv, reinterpret_cast<V*>(reinterpret_cast<char*>(a.r + pbase) + vo));
        }
      }
    }
    const double w = wave_cols<VE>(red);
    if (lane < VE) sred[wave][lane] = w;
    if (tid == 0) snext = nx;
    __syncthreads();  // the tile's rows and sums are done with
    if (tid < VE) {
      double s = sred[0][tid];
#pragma unroll
      for (int v = 1; v < NT / 64; ++v) s += sred[v][tid];
      a.part[((int64_t)panel * VE + tid) * a.ts.ntiles + t] = s;
    }
    lt = __builtin_amdgcn_readfirstlane(snext);
  }
}

// Elementwise kernels between the row-major blocks and the panels.  A workgroup
// takes 64 rows of up to 16 panels: it reads and writes the panels in runs of 64
// rows (lane = row) and the row-major blocks in runs of whole rows, through an
// LDS tile, so that both sides move whole lines.
//   INIT: r = R, p = M^-1 r, W = 0        UPD: W += alpha p, p = M^-1 r + beta p
enum { PEL_INIT = 0, PEL_UPD = 1 };
constexpr int kEltThreads = 256;
constexpr int kEltRows = 64;
constexpr int kEltPanels = 16;

template <class T>
struct PanelElt {
  const T* R;     // INIT: right-hand side, row-major
  int64_t ldR;
  T* W;           // solution, row-major
  int64_t ldw;
  T* r;
  T* p;
  const T* jac;
  const PcgCoef* coef;
  int64_t n;
  int b, npan, vecR, vecW;
};

template <class T, int MODE>
__global__ __launch_bounds__(kEltThreads) void k_panel_elt(PanelElt<T> a) {
  using V = typename PV<T>::type;
  constexpr int VE = 16 / (int)sizeof(T);
  constexpr int PW = kEltPanels / (kEltThreads / 64);             // panels per wavefront
  constexpr int RC = kEltRows * kEltPanels / kEltThreads;  // row-major vectors per thread
  __shared__ V sm[kEltRows][kEltPanels + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * kEltRows;
  const int p0 = blockIdx.y * kEltPanels;
  const int np = min(kEltPanels, a.npan - p0);
  const int64_t prow = min(row0 + lane, a.n - 1);      // panel side: this lane's row
  const bool prow_ok = row0 + lane < a.n;
  const int rp = tid & (kEltPanels - 1), rr = tid >> 4;  // row-major side: panel, first row
  const int c0 = (p0 + rp) * VE;
  const int nc = rp < np ? min(VE, a.b - c0) : 0;        // columns of this thread's vector
  constexpr int RS = kEltThreads / kEltPanels;             // rows between its vectors
  const T dinv = (T)1 / a.jac[prow];
  V x[RC];
  if constexpr (MODE == PEL_INIT) {
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const int64_t row = row0 + rr + k * RS;
      x[k] = V(0);
      if (row < a.n && nc > 0) {
        const T* R = a.R + row * a.ldR + c0;
        T* w = a.W + row * a.ldw + c0;
        if (nc == VE && a.vecR) {
          x[k] = *reinterpret_cast<const V*>(R);
        } else {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (e < nc) x[k][e] = R[e];
        }
        if (nc == VE && a.vecW) {
          *reinterpret_cast<V*>(w) = V(0);
        } else {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (e < nc) w[e] = (T)0;
        }
      }
      sm[rr + k * RS][rp] = x[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      const int q = wave + k * (kEltThreads / 64);
      if (q >= np || !prow_ok) continue;
      const int64_t o = ((int64_t)(p0 + q) * a.n + prow) * VE;
      const V rv = sm[lane][q];
      V pv;
#pragma unroll
      for (int e = 0; e < VE; ++e) pv[e] = rv[e] * dinv;
      *reinterpret_cast<V*>(a.r + o) = rv;
      *reinterpret_cast<V*>(a.p + o) = pv;
    }
  } else {
    V rv[PW], pv[PW];
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      const int q = min(wave + k * (kEltThreads / 64), np - 1);
      const int64_t o = ((int64_t)(p0 + q) * a.n + prow) * VE;
      rv[k] = *reinterpret_cast<const V*>(a.r + o);
      pv[k] = *reinterpret_cast<const V*>(a.p + o);
    }
    const bool vec = nc == VE && a.vecW;
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const int64_t row = row0 + rr + k * RS;
      if (row < a.n && nc > 0) {
        const T* w = a.W + row * a.ldw + c0;
        if (vec) {
          x[k] = *reinterpret_cast<const V*>(w);
        } else {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (e < nc) x[k][e] = w[e];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      const int q = wave + k * (kEltThreads / 64);
      if (q >= np) continue;  // the same for the whole wavefront
      sm[lane][q] = pv[k];
      const MBL_CONST PcgCoef* cf =
          (const MBL_CONST PcgCoef*)a.coef + __builtin_amdgcn_readfirstlane((p0 + q) * VE);
#pragma unroll
      for (int e = 0; e < VE; ++e)
        if (cf[e].live) pv[k][e] = rv[k][e] * dinv + (T)cf[e].beta * pv[k][e];
      if (prow_ok) {
        const int64_t o = ((int64_t)(p0 + q) * a.n + prow) * VE;
        *reinterpret_cast<V*>(a.p + o) = pv[k];
      }
    }
    __syncthreads();
    if (nc > 0) {
      T alpha[VE];
#pragma unroll
      for (int e = 0; e < VE; ++e) alpha[e] = (T)a.coef[c0 + e].alpha;
#pragma unroll
      for (int k = 0; k < RC; ++k) {
        const int64_t row = row0 + rr + k * RS;
        if (row >= a.n) continue;
        const V po = sm[rr + k * RS][rp];
        T* w = a.W + row * a.ldw + c0;
#pragma unroll
        for (int e = 0; e < VE; ++e) x[k][e] = x[k][e] + alpha[e] * po[e];
        if (vec) {
          __builtin_nontemporal_store(x[k], reinterpret_cast<V*>(w));
        } else {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (e < nc) w[e] = x[k][e];
        }
      }
    }
  }
}

// rho = r.M^-1 r of the starting residual: partial sums [column][workgroup].
template <class T>
__global__ __launch_bounds__(kPThreads) void k_panel_rho(const T* __restrict__ r,
                                                         const T* __restrict__ jac, int64_t n,
                                                         double* __restrict__ part) {
  using V = typename PV<T>::type;
  constexpr int VE = 16 / (int)sizeof(T);
  __shared__ double sred[kPWaves][VE];
  const int panel = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double red[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) red[e] = 0.0;
  for (int64_t row = (int64_t)blockIdx.x * kPThreads + tid; row < n;
       row += (int64_t)gridDim.x * kPThreads) {
    const V rv = *reinterpret_cast<const V*>(r + ((int64_t)panel * n + row) * VE);
    const T dinv = (T)1 / jac[row];
#pragma unroll
    for (int e = 0; e < VE; ++e) red[e] += (double)rv[e] * (double)(rv[e] * dinv);
  }
  const double w = wave_cols<VE>(red);
  if (lane < VE) sred[wave][lane] = w;
  __syncthreads();
  if (tid < VE) {
    double s = sred[0][tid];
#pragma unroll
    for (int v = 1; v < kPWaves; ++v) s += sred[v][tid];
    part[((int64_t)panel * VE + tid) * gridDim.x + blockIdx.x] = s;
  }
}

// Folds the np partial sums of one column (one workgroup, fixed order), updates its
// CG coefficients and clears the tile counters for the next apply.  Columns from
// `lim` on are frozen.
enum { PFIN_INIT = 0, PFIN_ALPHA = 1, PFIN_BETA = 2 };
constexpr int kNextInts = 8 * 32;

template <int MODE>
__global__ __launch_bounds__(kPThreads) void k_panel_fin(const double* __restrict__ part, int np,
                                                         int lim, PcgCoef* __restrict__ coef,
                                                         int* __restrict__ next) {
  __shared__ double swave[kPWaves];
  const int c = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (c == 0)
    for (int i = threadIdx.x; i < kNextInts; i += kPThreads) next[i] = 0;
  const double* pc = part + (int64_t)c * np;
  double s = 0.0;
  for (int g = threadIdx.x; g < np; g += kPThreads) s += pc[g];
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) swave[wave] = s;
  __syncthreads();
  if (threadIdx.x != 0) return;
  s = swave[0];
  for (int v = 1; v < kPWaves; ++v) s += swave[v];
  PcgCoef& k = coef[c];
  if (MODE == PFIN_INIT) {
    k.rho = s;
    k.live = s > 0.0;
    k.alpha = 0.0;
    k.beta = 0.0;
    k.pap = 0.0;
  } else if (MODE == PFIN_ALPHA) {
    k.pap = s;
    k.live = k.live && c < lim && (s > 0.0);
    k.alpha = k.live ? k.rho / s : 0.0;
  } else {
    k.live = k.live && (s > 0.0);
    k.beta = k.live ? s / k.rho : 0.0;
    if (k.live) k.rho = s;
  }
}

// ---- tables ------------------------------------------------------------------

struct PanelTabArgs {
  int L, k, q, Lh;  // q low sites, Lh high sites
  double zz4;
  double h[kMaxL];
  const uint32_t* pascal;
  PanelTile* tiles;
  uint4* lo_tab;
  double* lo_E;
};

// Energy of the sites base .. base + len - 1 in configuration v (their fields and
// the ZZ terms of the bonds between them); *nd: anti-aligned bonds.
__device__ inline double half_energy(const PanelTabArgs& a, int base, int len, uint32_t v, int* nd) {
  double e = 0.0;
  int c = 0;
  for (int i = 0; i + 1 < len; ++i) {
    const bool anti = (((v >> i) ^ (v >> (i + 1))) & 1u) != 0;
    e += anti ? -a.zz4 : a.zz4;
    c += anti ? 1 : 0;
  }
  for (int i = 0; i < len; ++i) e += a.h[base + i] * (((v >> i) & 1u) ? 0.5 : -0.5);
  *nd = c;
  return e;
}

// First row of the block of hi: the rank of its up spins, which come after the
// kl up spins of the low half.
__device__ inline int block_row(const PanelTabArgs& a, const uint32_t* C, uint32_t hi, int kl) {
  int row = 0, j = 0;
  for (int p = 0; p < a.Lh; ++p)
    if ((hi >> p) & 1u) row += (int)C[(a.q + p) * kPascal + kl + ++j];
  return row;
}

// Subsets of {0 .. m - 1} with c elements and sum s, and those with a smaller sum.
constexpr int kMaxSum = 17 * 16 / 2;
struct Subsets {
  uint16_t n[kMaxHigh][kMaxHigh][kMaxSum + 1], below[kMaxHigh][kMaxHigh][kMaxSum + 1];
  constexpr Subsets() : n(), below() {
    n[0][0][0] = 1;
    for (int m = 1; m < kMaxHigh; ++m)
      for (int c = 0; c < kMaxHigh; ++c)
        for (int t = 0; t <= kMaxSum; ++t)
          n[m][c][t] = (uint16_t)(n[m - 1][c][t] +
                                  (c > 0 && t >= m - 1 ? n[m - 1][c - 1][t - (m - 1)] : 0));
    for (int m = 0; m < kMaxHigh; ++m)
      for (int c = 0; c < kMaxHigh; ++c)
        for (int t = 1; t <= kMaxSum; ++t)
          below[m][c][t] = (uint16_t)(below[m][c][t - 1] + n[m][c][t - 1]);
  }
};
__device__ const Subsets kSubsets = Subsets();

// The order in which the tiles are taken: by the up spins of hi without its lowest site,
// within that by the sum of their positions.  A flip inside that part keeps the first
// and moves the second by one, and the flips at its lower end (the middle bond, the
// lowest bond of hi) change the lowest site or go one group on: what a run of tiles
// gathers lies in the groups next to it, where in row order the flips of the highest
// sites go far.  An LRU cache of an XCD's L2 (262144 rows of 16 bytes) that sees the
// tiles in this order fetches each vector 1.46 times at L = 24, in row order 3.01.
// The card, where 256 tiles of an XCD are in flight at once, goes from 3.0 to 2.5; the two
// applies of a step at L = 26 (64 FP32 columns) from 5.45 to 5.05 ms.
//
// The two values of the lowest site follow each other, so a group of tiles is a number of
// equal pairs (where both have rows) and the first tile of a row count is a division
// (first_tile).
__device__ inline int tile_rank(const PanelTabArgs& a, const uint32_t* C, uint32_t hi) {
  auto rows = [&](int kl) { return kl < 0 || kl > a.q ? 0 : (int)C[a.q * kPascal + kl]; };
  const int m = a.Lh - 1;
  int c = __popc(hi >> 1), sum = 0, t = 0;
  for (uint32_t w = hi >> 1; w; w &= w - 1) sum += __ffs(w) - 1;
  for (int g = 0; g < c; ++g)
    t += (int)C[m * kPascal + g] * ((rows(a.k - g) > 0) + (rows(a.k - g - 1) > 0));
  const int even = rows(a.k - c) > 0, odd = rows(a.k - c - 1) > 0;
  int i = kSubsets.below[m][c][sum];
  for (int b = m - 1; b >= 0; --b)
    if ((hi >> (b + 1)) & 1u) {
      i += kSubsets.n[b][c][sum];
      --c;
      sum -= b;
    }
  return t + i * (even + odd) + ((hi & 1u) ? even : 0);
}

// One thread per low configuration and one per high configuration; a tile is one of those
// that have rows in the sector.
// blockIdx.y: the tables of the panels or of the apply.
__global__ __launch_bounds__(256) void k_panel_tables(PanelTabArgs a0, PanelTabArgs a1) {
  __shared__ uint32_t C[kPascal * kPascal];  // read in serial chains
  const PanelTabArgs& a = blockIdx.y == 0 ? a0 : a1;
  for (int i = threadIdx.x; i < kPascal * kPascal; i += 256) C[i] = a.pascal[i];
  __syncthreads();
  const uint32_t id = blockIdx.x * 256 + threadIdx.x;
  auto binom = [&](int i, int t) { return t < 0 || t > i ? 0 : (int)C[i * kPascal + t]; };
  if (id < (1u << a.q)) {
    // by (up spins, value); the flips as rows of the LDS tile (row u at u + 1,
    // the zero row at 0), 10 bits each, three to a word, and their number in the
    // top 4 bits of the last word
    const uint32_t v = id;
    const int kl = __popc(v);
    int at = 0, u = 0, j = 0;
    for (int c = 0; c < kl; ++c) at += binom(a.q, c);
    for (int p = 0; p < a.q; ++p)
      if ((v >> p) & 1u) u += binom(p, ++j);
    uint32_t w[4] = {0, 0, 0, 0};
    int m = 0;
    for (int b = 0; b + 1 < a.q; ++b) {
      if (!(((v >> b) ^ (v >> (b + 1))) & 1u)) continue;
      const int c = binom(b, __popc(v & ((1u << b) - 1u)));
      const uint32_t f = (uint32_t)(u + (((v >> b) & 1u) ? c : -c) + 1) << (10 * (m % 3));
      w[0] |= m / 3 == 0 ? f : 0u;
      w[1] |= m / 3 == 1 ? f : 0u;
      w[2] |= m / 3 == 2 ? f : 0u;
      w[3] |= m / 3 == 3 ? f : 0u;
      ++m;
    }
    a.lo_tab[at + u] = make_uint4(w[0], w[1], w[2], w[3] | ((uint32_t)m << 28));
    int nd;
    a.lo_E[at + u] = half_energy(a, 0, a.q, v, &nd);
  }
  if (id < (1u << a.Lh)) {
    const uint32_t v = id;
    const int kl = a.k - __popc(v);
    if (kl < 0 || kl > a.q) return;
    PanelTile t{};
    t.row0 = block_row(a, C, v, kl);
    t.nrows = binom(a.q, kl);
    for (int c = 0; c < kl; ++c) t.aux += binom(a.q, c);
    t.E = half_energy(a, a.q, a.Lh, v, &t.nd);
    for (int b = 0; b + 1 < a.Lh; ++b)
      if (((v >> b) ^ (v >> (b + 1))) & 1u)
        t.off[t.cnt++] = block_row(a, C, v ^ (3u << b), kl) - t.row0;
    // middle bond: even hi, the rows with the top low site up (the last
    // C(11, kl - 1)) land on the first rows of hi | 1; odd hi, the rows with that
    // site down land on the last rows of hi & ~1
    const uint32_t pv = v ^ 1u;
    const int pkl = a.k - __popc(pv), split = binom(a.q - 1, kl);
    if (pkl >= 0 && pkl <= a.q) {
      const int prow = block_row(a, C, pv, pkl);
      t.mlo = (v & 1u) ? 0 : split;
      t.mhi = (v & 1u) ? split : t.nrows;
      t.mbase = (v & 1u) ? prow + binom(a.q - 1, kl + 1) : prow - split;
    }
    a.tiles[tile_rank(a, C, v)] = t;
  }
}

// Calls f(tiles per pair, rows of the first, rows of both, pairs) for every group.
template <class F>
void tile_groups(const Ham& H, int q, F f) {
  const int m = H.L - q - 1;
  auto rows = [&](int kl) -> int64_t {
    return kl < 0 || kl > q ? 0 : H.pascal_host[q * kPascal + kl];
  };
  for (int c = 0; c <= m; ++c) {
    const int64_t even = rows(H.nup - c), odd = rows(H.nup - c - 1);
    if (even + odd == 0) continue;
    f((even > 0) + (odd > 0), even > 0 ? even : odd, even + odd,
      (int64_t)H.pascal_host[m * kPascal + c]);
  }
}

// Tiles before the first one that has `row` or more rows before it.
int first_tile(const Ham& H, const PanelTables& P, int64_t row) {
  int64_t t = 0;
  tile_groups(H, P.q, [&](int per, int64_t first, int64_t both, int64_t pairs) {
    const int64_t i = std::min(pairs, row / both), rest = row - i * both;
    t += i * per;
    row = i == pairs ? rest : 0;
    if (i < pairs && rest > 0) t += rest <= first ? 1 : per;
  });
  return (int)t;
}

// The arguments for the tables of P, for blocks of q low sites; false where the mean block
// is short.
bool plan_tables(Ham& H, PanelTables& P, int q, int mean_rows, PanelTabArgs* out, hipStream_t s) {
  const int Lh = H.L - q;
  int64_t tiles = 0;
  tile_groups(H, q, [&](int per, int64_t, int64_t, int64_t pairs) { tiles += per * pairs; });
  if (H.n < mean_rows * tiles) return false;
  P.q = q;
  P.ntiles = (int)tiles;
  const size_t nt = P.ntiles * sizeof(PanelTile), nl = (size_t)1 << q;
  H.table(P.buf, nl * (sizeof(uint4) + sizeof(double)) + nt, s);
  P.lo_tab = P.buf.as<uint4>();
  P.lo_E = reinterpret_cast<double*>(P.lo_tab + nl);
  P.tiles = reinterpret_cast<PanelTile*>(P.lo_E + nl);
  PanelTabArgs& a = *out;
  a.L = H.L;
  a.k = H.nup;
  a.q = q;
  a.Lh = Lh;
  a.zz4 = 0.25 * H.J * H.Delta;
  std::copy(H.h, H.h + kMaxL, a.h);
  a.pascal = H.pascal.as<uint32_t>();
  a.tiles = P.tiles;
  a.lo_tab = P.lo_tab;
  a.lo_E = P.lo_E;
  return true;
}

}  // namespace

void build_panel_tables(Ham& H, hipStream_t s) {
  PanelTabArgs a[2]{};
  auto fits = [&](int q, int most_high, int64_t least) {
    return H.L - q >= 2 && H.L - q <= most_high && H.n > least;
  };
  // Panels: smaller sectors are bound by launches, of which this path has as many.  The
  // upper limit: 32-bit byte offsets within a panel.
  //
  // Mean rows: sectors far from half filling have many tiles of few rows, which leave
  // most lanes of a workgroup idle.  CG against the gather kernels, 32 FP64 columns, by
  // rows per tile: 27 (L = 24, 5 up) 1373 us for 657, 105 (7 up) 3010 for 2852, 157
  // (L = 20, 6 up) 675 for 619, 194 (L = 24, 8 up; 4 columns) 1514 for 1375; 304 (L = 20,
  // 7 up) 842 for 887, 325 (L = 24, 9 up) 8006 for 10938.  Half filling has 600 to 800.
  // The apply: 35 153 for 75, 57 225 for 175, 88 (L = 24, 9 up) 419 for 365; 103 (L = 21,
  // 8 up; 64 columns) 69 for 82, 123 (L = 24, 10 up) 555 for 604.  Half filling has 150 to
  // 230.
  if (!H.col_ok && fits(kPanelQ, kPanelMaxHigh, kPanelMinRows) && H.n < (1ll << 28))
    H.panel.ok = plan_tables(H, H.panel, kPanelQ, kPanelMeanRows, &a[0], s);
  int n = H.panel.ok ? 1 : 0;
  if (fits(kTileQ, kMaxHigh, kTileMinRows))
    H.tile.ok = plan_tables(H, H.tile, kTileQ, kTileMeanRows, &a[n], s);
  if (H.tile.ok) ++n;
  if (n == 0) return;
  size_t threads = 0;
  for (int i = 0; i < n; ++i)
    threads = std::max({threads, (size_t)1 << a[i].q, (size_t)1 << a[i].Lh});
  hipLaunchKernelGGL(k_panel_tables, dim3((unsigned)((threads + 255) / 256), n), dim3(256), 0, s,
                     a[0], a[1]);
  MBL_CHECK_LAUNCH();
}

bool panel_grid_fits(int64_t tiles, int64_t panels) {
  return panels <= 65535 && tiles * panels < (1ll << 30);
}

namespace {

// Each XCD takes an eighth of the rows of all panels.  Eight workgroups per CU, as
// many as fit at once: a CG step at L = 24 (64 FP32 columns) takes 2.20, 2.01, 1.89
// and 1.88 ms with 3, 4, 6 and 8; at L = 20 (64 FP64 columns) 245, 228, 217, 217 us.
constexpr int kPanelPerCu = 8;

// Few tiles leave the card short of wavefronts: up to this number 512 threads take one.
// CG of 16 steps with 256 and 512: 256 tiles (L = 17, 32 FP32 columns) 743 and 673 us, 1024
// (L = 18, 32 FP64) 1119 and 1070, 2048 (L = 21, 8 FP64) 1691 and 1527, 4096 (L = 20, 32
// FP64) 2267 and 2184; 8192 (L = 20, 64 FP64) 3674 and 3666, (L = 24, 8 FP32) 5318 and 5370;
// at L = 24 with 64 columns the second apply takes 662 and 771.
constexpr int64_t kPanelWideTiles = 4096;

}  // namespace

PanelSched panel_sched(const Ham& H, const PanelTables& P, int npan, int slots) {
  const int64_t n = H.n;
  PanelSched t{};
  t.ntiles = P.ntiles;
  int most = 1;
  for (int x = 0; x <= 8; ++x) {
    const int64_t target = (int64_t)x * n * npan / 8;  // rows of all panels before XCD x
    const int64_t panel = target / n;
    t.first[x] = (int)(panel * t.ntiles) + first_tile(H, P, target - panel * n);
    if (x) most = std::max(most, t.first[x] - t.first[x - 1]);
  }
  t.nwg = 8 * std::min(most, slots);
  return t;
}

template <class T>
void run_pcg_panel(const Ham& H, double sigma, const T* jac, const T* R, int64_t ldr, T* W,
                   int64_t ldw, int b, int m, hipStream_t s, PcgTiming* tm, const StopCheck* stop,
                   int keep, int m_keep) {
  constexpr int VE = 16 / (int)sizeof(T);
  const PanelTables& P = H.panel;
  const int64_t n = H.n;
  const int npan = (b + VE - 1) / VE;
  const size_t vec = (size_t)n * npan * 16;
  const int nrho = (int)std::min<int64_t>((n + kPThreads - 1) / kPThreads, 64);
  DevBuf rbuf(vec, s), pbuf(vec, s), tbuf(vec, s);
  DevBuf partb((size_t)npan * VE * std::max(P.ntiles, nrho) * sizeof(double), s);
  DevBuf coefb((size_t)npan * VE * sizeof(PcgCoef), s);
  DevBuf nextb(kNextInts * sizeof(int), s);
  PcgCoef* coef = coefb.as<PcgCoef>();
  double* part = partb.as<double>();
  int* next = nextb.as<int>();
  auto al16 = [](const void* p, int64_t ld) {
    return reinterpret_cast<uintptr_t>(p) % 16 == 0 && (ld * (int64_t)sizeof(T)) % 16 == 0;
  };
  PanelElt<T> e{};
  e.R = R;
  e.ldR = ldr;
  e.W = W;
  e.ldw = ldw;
  e.r = rbuf.as<T>();
  e.p = pbuf.as<T>();
  e.jac = jac;
  e.coef = coef;
  e.n = n;
  e.b = b;
  e.npan = npan;
  e.vecR = al16(R, ldr);
  e.vecW = al16(W, ldw);
  auto elt = [&](auto mode, const PanelElt<T>& q, hipStream_t st) {
    const dim3 grid((unsigned)((n + kEltRows - 1) / kEltRows), (q.npan + kEltPanels - 1) / kEltPanels);
    hipLaunchKernelGGL((k_panel_elt<T, decltype(mode)::value>), grid, dim3(kEltThreads), 0, st, q);
    MBL_CHECK_LAUNCH();
  };
  auto fin = [&](auto mode, int cols, int np, int lim, hipStream_t st) {
    hipLaunchKernelGGL(k_panel_fin<decltype(mode)::value>, dim3(cols), dim3(kPThreads), 0, st, part,
                       np, lim, coef, next);
    MBL_CHECK_LAUNCH();
  };
  using FI = std::integral_constant<int, PFIN_INIT>;
  using FA = std::integral_constant<int, PFIN_ALPHA>;
  using FB = std::integral_constant<int, PFIN_BETA>;
  using MI = std::integral_constant<int, PEL_INIT>;
  using MU = std::integral_constant<int, PEL_UPD>;
  elt(MI{}, e, s);
  hipLaunchKernelGGL(k_panel_rho<T>, dim3(nrho, npan), dim3(kPThreads), 0, s, rbuf.as<T>(), jac, n,
                     part);
  MBL_CHECK_LAUNCH();
  fin(FI{}, npan * VE, nrho, npan * VE, s);

  // CG steps [from, to) on the leading np panels; columns from `cols` on are frozen
  auto steps = [&](int np, int cols, int from, int to) {
    const bool wide = (int64_t)np * P.ntiles <= kPanelWideTiles;
    const PanelSched ts = panel_sched(H, P, np, 32 * kPanelPerCu);
    PanelArgs<T> a1{};
    a1.tiles = P.tiles;
    a1.lo_tab = P.lo_tab;
    a1.lo_E = P.lo_E;
    a1.coef = coef;
    a1.part = part;
    a1.next = next;
    a1.n = n;
    a1.sigma = sigma;
    a1.halfJ = 0.5 * H.J;
    a1.zz4 = 0.25 * H.J * H.Delta;
    a1.ts = ts;
    PanelArgs<T> a2 = a1;
    a1.X = pbuf.as<T>();
    a1.Y = tbuf.as<T>();
    a2.X = tbuf.as<T>();
    a2.r = rbuf.as<T>();
    PanelElt<T> eu = e;
    eu.npan = np;
    eu.b = std::min(b, np * VE);
    auto apply = [&](auto epi, const PanelArgs<T>& a, hipStream_t st) {
      constexpr int E = decltype(epi)::value;
      if (wide)
        hipLaunchKernelGGL((k_panel<T, E, 512>), dim3(ts.nwg), dim3(512), 0, st, a);
      else
        hipLaunchKernelGGL((k_panel<T, E, 256>), dim3(ts.nwg), dim3(256), 0, st, a);
      MBL_CHECK_LAUNCH();
    };
    using E1 = std::integral_constant<int, PAN_NORM2>;
    using E2 = std::integral_constant<int, PAN_RUPD>;
    auto step = [&](hipStream_t st) {
      apply(E1{}, a1, st);
      fin(FA{}, np * VE, P.ntiles, cols, st);
      apply(E2{}, a2, st);
      fin(FB{}, np * VE, P.ntiles, cols, st);
      elt(MU{}, eu, st);
    };
    const int ntimed = tm ? std::min(to - from, PcgTiming::kSample) : 0;
    if (ntimed) tm->init();
    int it = from;
    for (int k = 0; k < ntimed; ++k, ++it) {
      MBL_HIP(hipEventRecord(tm->ev[4 * k + 0], s));
      apply(E1{}, a1, s);
      MBL_HIP(hipEventRecord(tm->ev[4 * k + 1], s));
      fin(FA{}, np * VE, P.ntiles, cols, s);
      MBL_HIP(hipEventRecord(tm->ev[4 * k + 2], s));
      apply(E2{}, a2, s);
      MBL_HIP(hipEventRecord(tm->ev[4 * k + 3], s));
      fin(FB{}, np * VE, P.ntiles, cols, s);
      elt(MU{}, eu, s);
    }
    const int run = replay_steps(step, it, to, s, stop) - from;
    if (ntimed) {
      // algorithmic bytes: apply1 reads p and writes T; apply2 reads T and r and
      // writes r
      const double w = (double)n * eu.b * sizeof(T);
      tm->collect(ntimed, run, 2.0 * w, 3.0 * w, s);
    }
  };
  if (keep < 0 || m_keep <= m || keep >= b) {
    steps(npan, b, 0, keep >= b ? std::max(m, m_keep) : m);
  } else {
    steps(npan, b, 0, m);
    if (keep > 0) steps((keep + VE - 1) / VE, keep, m, m_keep);
  }
}

template void run_pcg_panel<double>(const Ham&, double, const double*, const double*, int64_t,
                                    double*, int64_t, int, int, hipStream_t, PcgTiming*,
                                    const StopCheck*, int, int);
template void run_pcg_panel<float>(const Ham&, double, const float*, const float*, int64_t, float*,
                                   int64_t, int, int, hipStream_t, PcgTiming*, const StopCheck*,
                                   int, int);

}  // namespace mbl
