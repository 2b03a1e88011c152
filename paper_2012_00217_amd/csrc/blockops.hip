// Tall-skinny block kernels of LOBPCG (paper Sec. 3.2, property (ii): a block
// method turns the work into matrix-matrix operations).
//
//  * Gram products C = A^T B of n x p and n x q blocks on the matrix cores:
//    v_mfma_f64_16x16x4f64 for FP64 blocks, v_mfma_f32_16x16x4f32 with FP32
//    accumulation for FP32 blocks.  The n dimension is split over workgroups;
//    each writes an FP64 partial tile and a second kernel folds the partials
//    in split order, so the result is bitwise reproducible.
//  * Block combination Y = A C + beta Y with a small FP64 coefficient matrix
//    C (rounded to the block type) on the matrix cores: the rows of A straight into the
//    operand registers, C in LDS.
//  * Precision conversion and the counter-based random starting block.
#include <algorithm>
#include <mutex>
#include <string>
#include <type_traits>

#include "common.h"

namespace mbl {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <class T>
struct Mfma;
// Output row of element v held by lane group g = lane / 16 (column = lane % 16):
// the FP64 instruction interleaves the four lane groups row by row, the FP32
// one gives each lane group four consecutive rows.
template <>
struct Mfma<double> {
  using acc = d4;
  __device__ static acc op(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int g, int v) { return g + 4 * v; }
};
template <>
struct Mfma<float> {
  using acc = f4;
  __device__ static acc op(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int g, int v) { return 4 * g + v; }
};

// One workgroup = 4 waves = a 64 x 64 tile of C; wave (wy, wx) owns the
// 32 x 32 quadrant as 2 x 2 blocks of 16 x 16.  16 x 16 x 4 MFMA operand
// layout: lane l supplies A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16];
// it receives D[Mfma<T>::row(l / 16, v)][l % 16], v = 0..3.  For C = A^T B the MFMA A
// operand is the transpose of the block, so both operands are 4 rows x 16
// consecutive columns of the row-major blocks.
//
// The rows are consumed in slabs of 32: the workgroup stages the slab's
// 32 x 64 panels of A and B in LDS (16-byte loads, each element read from memory
// once per workgroup), and the next slab's loads are in flight while the waves
// run their 32 MFMAs on the current one.
// sym (A = B, p = q): only the tiles on and above the diagonal are formed;
// they are enumerated row by row, and a diagonal tile stages one panel.
constexpr int kSlab = 32;

template <class T>
struct GramStage {
  static constexpr int VE = 16 / (int)sizeof(T);           // elements per 16-byte load
  static constexpr int PER = kSlab * 64 / (256 * VE);       // loads per thread per panel
  static constexpr int SWZ = sizeof(T) == 8 ? 1 : 3;
  // Place of element (r, c) of a panel: the rows are 64 elements apart and their blocks
  // of 16 columns are exchanged, so that the 4 rows x 16 columns of an operand read lie
  // in different banks (A^T A, n = 184756, p = 192: FP32 96 us a call, with rows padded by
  // 16 bytes 103; FP64 161 and 168).
  __device__ static int at(int r, int c) { return r * 64 + (c ^ ((r & SWZ) << 4)); }
};

template <class T>
__device__ inline void gram_load(const T* __restrict__ X, int64_t ldx, int ncol, int col0,
                                 int64_t k, int64_t ke, T (&reg)[GramStage<T>::PER][GramStage<T>::VE]) {
  using S = GramStage<T>;
#pragma unroll
  for (int u = 0; u < S::PER; ++u) {
    const int e = (u * 256 + (int)threadIdx.x) * S::VE;  // element in the 32 x 64 panel
    const int r = e >> 6, c = e & 63;
    const int64_t row = k + r;
    const int col = col0 + c;
    if (row < ke && col + S::VE <= ncol) {
      // 16 bytes at the alignment of an element: unaligned rows take the same loads
      // (n = 184756, element by element: FP32 101 and 64 columns 72 us a call, now 44; FP64
      // 127 columns 151, now 95)
      typedef T vec_t __attribute__((ext_vector_type(GramStage<T>::VE), aligned(sizeof(T))));
      const vec_t v = *reinterpret_cast<const vec_t*>(X + row * ldx + col);
#pragma unroll
      for (int t = 0; t < S::VE; ++t) reg[u][t] = v[t];
    } else {
#pragma unroll
      for (int t = 0; t < S::VE; ++t)
        reg[u][t] = (row < ke && col + t < ncol) ? X[row * ldx + col + t] : (T)0;
    }
  }
}

template <class T>
__device__ inline void gram_store(T* __restrict__ sm, const T (&reg)[GramStage<T>::PER][GramStage<T>::VE]) {
  using S = GramStage<T>;
#pragma unroll
  for (int u = 0; u < S::PER; ++u) {
    const int e = (u * 256 + (int)threadIdx.x) * S::VE;
    const int r = e >> 6, c = e & 63;
#pragma unroll
    for (int t = 0; t < S::VE; ++t) sm[S::at(r, c) + t] = reg[u][t];
  }
}

// Bound by the waits of a slab's loads and barriers: 65 % of the time the matrix cores
// are busy.  Four workgroups per CU (FP64: launch_bounds caps the registers at 128) hold
// all 1024 workgroups of a launch at once; at 152 registers three fit, and the last
// quarter of the workgroups runs as a second round (n = 184756, a call: A^T A of 192
// columns 161 us, without the cap 219; 128 and 64 columns 72 and 80).  FP32 takes 64
// registers without a cap, and is slower with one (n = 705432, 96 and 48 columns: 130 us,
// capped 145).
template <class T>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? 4 : 1)
void k_gram(int64_t n, const T* __restrict__ A, int64_t lda, int p, const T* __restrict__ B,
            int64_t ldb, int q, int sym, int tiles, int64_t rows_per_split,
            double* __restrict__ part) {
  using M = Mfma<T>;
  using S = GramStage<T>;
  __shared__ T sa[kSlab * 64], sb[kSlab * 64];
  const int lane = threadIdx.x & 63;
  const int tiles_q = (q + 63) / 64;
  const int item = blockIdx.x % tiles;
  const int64_t split = blockIdx.x / tiles;
  int ty, tx;
  if (sym) {
    int t = item;
    ty = 0;
    while (t >= tiles_q - ty) {
      t -= tiles_q - ty;
      ++ty;
    }
    tx = ty + t;
  } else {
    ty = item / tiles_q;
    tx = item % tiles_q;
  }
  const bool same = sym && ty == tx;  // one panel serves both operands
  // The quadrant of a wavefront moves on with the split: the wavefronts of a SIMD
  // then skip below the diagonal equally often.
  const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) + (int)split) & 3;
  const int wy = wave >> 1, wx = wave & 1;
  const bool below = same && wy > wx;  // a quadrant below the diagonal: not needed
  const T* sbp = same ? sa : sb;
  const int li = lane & 15, lk = lane >> 4;
  const int64_t kb = split * rows_per_split;
  const int64_t ke = min(n, kb + rows_per_split);
  typename M::acc acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = typename M::acc{0, 0, 0, 0};
  T ra[S::PER][S::VE], rb[S::PER][S::VE];
  if (kb < ke) {
    gram_load<T>(A, lda, p, ty * 64, kb, ke, ra);
    if (!same) gram_load<T>(B, ldb, q, tx * 64, kb, ke, rb);
  }
  for (int64_t k = kb; k < ke; k += kSlab) {
    __syncthreads();  // the previous slab's MFMAs are done with the LDS panels
    gram_store<T>(sa, ra);
    if (!same) gram_store<T>(sb, rb);
    __syncthreads();
    if (k + kSlab < ke) {
      gram_load<T>(A, lda, p, ty * 64, k + kSlab, ke, ra);
      if (!same) gram_load<T>(B, ldb, q, tx * 64, k + kSlab, ke, rb);
    }
    if (below) continue;
#pragma unroll
    for (int kk = 0; kk < kSlab; kk += 4) {
      T a[2], b[2];
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        a[v] = sa[kk * 64 + S::at(lk, wy * 32 + 16 * v + li)];
        b[v] = sbp[kk * 64 + S::at(lk, wx * 32 + 16 * v + li)];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = M::op(a[i], b[j], acc[i][j]);
    }
  }
  if (below) return;
  const int c0 = ty * 64 + wy * 32, d0 = tx * 64 + wx * 32;
  double* out = part + split * p * q;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = c0 + 16 * i + M::row(lk, v);
        const int c = d0 + 16 * j + li;
        if (r < p && c < q) out[(int64_t)r * q + c] = (double)acc[i][j][v];
      }
}

// 16 consecutive elements of C per workgroup (a 128-byte line of every partial), 16
// threads each: thread g sums splits g, g + 16, ... in order, then the 16 sums are added
// in order.  One element per wavefront read 8 bytes of every line that it fetched
// (192 x 192, 170 splits: 17 us, now 7.8).
// sym: elements below the diagonal are written as the mirror of those above.
__global__ __launch_bounds__(256) void k_gram_fold(const double* __restrict__ part, int splits,
                                                   int p, int q, int sym, double scale,
                                                   double* __restrict__ C, int64_t ldc) {
  __shared__ double sm[16][17];
  const int e = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int64_t step = (int64_t)p * q, idx = (int64_t)blockIdx.x * 16 + e;
  const int64_t r = idx / q, c = idx % q;
  const bool mine = idx < step && !(sym && c < r);
  double s = 0.0;
  if (mine)
#pragma unroll 4
    for (int sp = g; sp < splits; sp += 16) s += part[sp * step + idx];
  sm[g][e] = s;
  __syncthreads();
  if (g != 0 || !mine) return;
  for (int k = 1; k < 16; ++k) s += sm[k][e];
  s *= scale;
  C[r * ldc + c] = s;
  if (sym && r < c) C[c * ldc + r] = s;
}

// Y[r, j] = sum_k A[r, k] C[k, j] + beta Y[r, j] on the matrix cores.
//
// A wavefront owns 16 rows x 16 NB columns.  The rows of A go from memory straight
// into the operand registers: the sum over k may run in any order, so lane (i, g) of the
// 16 x 4 operand takes the 16-byte piece g of a slab of its row (k = 2g, 2g + 1 in FP64,
// 4g .. 4g + 3 in FP32) and step t of the slab multiplies element t of every piece.  Four
// slabs are one group; the next group's loads (of the next tile at a row's end) are in
// flight while the group is multiplied.  C stands in LDS, rounded to T, in chunks of kc
// rows of k; when all of C fits it is loaded once and the wavefronts run over their
// tiles without a barrier.
//
// Bound by memory (378 MB) and the matrix cores (4.5 GFLOP FP64) about equally at
// n = 184756, 192 -> 64 columns: 99 us a call; a vector-unit form that stages A through
// LDS takes 207.  FP32: 65 and 114.  Full slabs are read without a mask (with one: FP64 122,
// FP32 73) and at the alignment of an element, so that unaligned rows take the same loads
// (FP32 150 -> 75: 82 us, element by element 119).
//
// Registers: FP32 with 32 columns takes 135 without the cap, and of the two workgroups of 8
// wavefronts that a CU is to hold only one fits (32 -> 32: 20.8 us, now 17.8; 96 -> 32: 34.6
// and 28.5).
template <class T>
struct CombineStage {
  static constexpr int VE = 16 / (int)sizeof(T);  // elements per 16-byte piece
  static constexpr int SL = 4 * VE;               // k per slab
  static constexpr int GK = 4 * SL;               // k per group
  // Place of C[k][c] in a chunk: the 4 rows of an operand, VE apart, go to different
  // banks.  Rows of 48 are padded, the others exchange their blocks of 16.
  static constexpr int row(int nb) { return nb == 3 ? 48 + 16 / VE : 16 * nb; }
  template <int NB>
  __device__ static int at(int k, int c) {
    if constexpr (NB == 3) {
      return k * row(NB) + c;
    } else {
      constexpr int M = (sizeof(T) == 8 ? 2 : 4) < NB ? (sizeof(T) == 8 ? 2 : 4) : NB;
      return k * row(NB) + (c ^ (((k / VE) & (M - 1)) << 4));
    }
  }
};

template <class T, int NB, int NW>
__global__ __launch_bounds__(64 * NW, NB == 2 ? 4 : 1)
void k_combine(int64_t n, const T* A, int64_t lda, int p, const double* __restrict__ Cm,
               int64_t ldc, T* Y, int64_t ldy, int q, double beta, double scale,
               const double* __restrict__ colscale, bool vec, int kc, int64_t tiles) {
  using M = Mfma<T>;
  using S = CombineStage<T>;
  constexpr int VE = S::VE, SL = S::SL, GK = S::GK, W = 16 * NB;
  extern __shared__ __align__(16) unsigned char combine_lds[];
  T* Cs = reinterpret_cast<T*>(combine_lds);  // [kc][W]
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = blockIdx.y * W;
  const int64_t stride = (int64_t)gridDim.x * NW;
  typedef T vec_t __attribute__((ext_vector_type(VE)));
  typedef T mem_t __attribute__((ext_vector_type(VE), aligned(sizeof(T))));  // in memory

  auto fetch = [&](vec_t (&reg)[4], int64_t tile, int k0) {
    const T* src = A + min(tile * 16 + li, n - 1) * lda;  // rows beyond n are not stored
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + u * SL + lk * VE;
      if (k0 + (u + 1) * SL <= p) {
        reg[u] = *reinterpret_cast<const mem_t*>(src + k);
      } else if (vec) {  // p is a multiple of VE
        const vec_t v = *reinterpret_cast<const mem_t*>(src + (k < p ? k : 0));
#pragma unroll
        for (int t = 0; t < VE; ++t) reg[u][t] = k < p ? v[t] : (T)0;
      } else {
#pragma unroll
        for (int t = 0; t < VE; ++t) {
          const T v = src[k + t < p ? k + t : 0];
          reg[u][t] = k + t < p ? v : (T)0;
        }
      }
    }
  };

  vec_t nxt[4];
  int64_t tile = (int64_t)blockIdx.x * NW + wave;
  if (p > 0) fetch(nxt, tile, 0);
  // every wavefront of the workgroup makes the same number of rounds (barriers)
  for (int64_t base = (int64_t)blockIdx.x * NW; base < tiles; base += stride, tile += stride) {
    typename M::acc acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = typename M::acc{0, 0, 0, 0};
    for (int k0 = 0; k0 < p; k0 += GK) {
      const int kl = k0 % kc;
      if (kl == 0 && (kc < p || base == (int64_t)blockIdx.x * NW)) {
        __syncthreads();  // the wavefronts are done with the chunk before
        for (int e = threadIdx.x; e < kc * W; e += 64 * NW) {
          const int k = e / W, c = e % W;
          const double cscale = colscale && c0 + c < q ? scale * colscale[c0 + c] : scale;
          Cs[S::template at<NB>(k, c)] =
              (k0 + k < p && c0 + c < q) ? (T)(Cm[(int64_t)(k0 + k) * ldc + c0 + c] * cscale) : (T)0;
        }
        __syncthreads();
      }
      vec_t cur[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
      if (k0 + GK < p)
        fetch(nxt, tile, k0 + GK);
      else
        fetch(nxt, tile + stride, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k0 + u * SL >= p) break;
#pragma unroll
        for (int t = 0; t < VE; ++t) {
          T b[NB];
#pragma unroll
          for (int j = 0; j < NB; ++j)
            b[j] = Cs[S::template at<NB>(kl + u * SL + lk * VE + t, 16 * j + li)];
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[j] = M::op(cur[u][t], b[j], acc[j]);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = tile * 16 + M::row(lk, v);
      if (row >= n) continue;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int c = c0 + 16 * j + li;
        if (c >= q) continue;
        T* y = Y + row * ldy + c;
        *y = (beta == 0.0) ? acc[j][v] : (T)(acc[j][v] + (T)beta * *y);
      }
    }
  }
}

// R = sign A - X diag(mu); A may be R.  The product is rounded before the sum, as in a
// combination with diag(-mu).
template <class T>
__global__ __launch_bounds__(256) void k_residual(int64_t n, int b, const T* A, int64_t lda, T sign,
                                                  const T* __restrict__ X, int64_t ldx,
                                                  const double* __restrict__ mu, T* R,
                                                  int64_t ldr) {
#pragma clang fp contract(off)
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * b) return;
  const int64_t r = idx / b;
  const int c = (int)(idx % b);
  const T t = X[r * ldx + c] * (T)-mu[c];
  R[r * ldr + c] = sign * A[r * lda + c] + t;
}

template <class S, class D>
__global__ __launch_bounds__(256) void k_convert(int64_t n, int b, const S* __restrict__ X,
                                                 int64_t ldx, D* __restrict__ Y, int64_t ldy) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * b) return;
  const int64_t r = idx / b;
  const int c = (int)(idx % b);
  Y[r * ldy + c] = (D)X[r * ldx + c];
}

// Diagonal preconditioner of the extreme-eigenvalue iteration (sign*H):
// W[r,c] = R[r,c] / max(|sign*E_r - mu_c|, floor), with E the diagonal of H and
// mu the current Ritz values.
__global__ __launch_bounds__(256) void k_diag_precond(int64_t n, int b, const double* __restrict__ R,
                                                      int64_t ldr, const double* __restrict__ E,
                                                      double sign, const double* __restrict__ mu,
                                                      double floor, double* __restrict__ W,
                                                      int64_t ldw) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * b) return;
  const int64_t r = idx / b;
  const int c = (int)(idx % b);
  const double d = fmax(fabs(sign * E[r] - mu[c]), floor);
  W[r * ldw + c] = R[r * ldr + c] / d;
}

// splitmix64 (Steele, Lea, Flood 2014) of a counter, then Box-Muller.
__device__ inline uint64_t splitmix64(uint64_t z) {
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

template <class T>
__global__ __launch_bounds__(256) void k_randn(int64_t n, int b, uint64_t seed, T* __restrict__ X,
                                               int64_t ldx) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * b) return;
  const uint64_t h1 = splitmix64(seed ^ splitmix64(2 * (uint64_t)idx));
  const uint64_t h2 = splitmix64(seed ^ splitmix64(2 * (uint64_t)idx + 1));
  const double u1 = ((h1 >> 11) + 1) * (1.0 / 9007199254740993.0);  // (0, 1]
  const double u2 = (h2 >> 11) * (1.0 / 9007199254740992.0);
  X[(idx / b) * ldx + idx % b] = (T)(sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
}

inline unsigned g1(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// At most 1024 workgroups, four per CU, which are resident at once.  FP64: splits down to
// 64 rows, where a short sector leaves CUs idle (n = 3432, p = q = 96: 14 splits of 256
// rows 24 us, 54 of 64 rows 18 us).  FP32: the accumulation is in FP32, so the split of
// the rows is part of the result and stays at 256 rows.
template <class T>
GramPlan gram_plan(int64_t n, int p, int q, bool same_operand) {
  GramPlan g;
  // A^T A: only the upper tiles (the Rayleigh-Ritz and Cholesky-QR Grams)
  g.sym = (same_operand && p == q) ? 1 : 0;
  const int tq = (q + 63) / 64;
  g.tiles = g.sym ? tq * (tq + 1) / 2 : ((p + 63) / 64) * tq;
  if (n == 0) {  // one split of zero rows: the kernel writes zero partials
    g.splits = 1;
    g.rows = kSlab;
  } else {
    const int64_t least = sizeof(T) == 8 ? 64 : 256;
    int64_t splits = std::max<int64_t>(1, 1024 / g.tiles);
    splits = std::min<int64_t>(splits, std::max<int64_t>(1, (n + least - 1) / least));
    int64_t rows = (n + splits - 1) / splits;
    rows = ((rows + kSlab - 1) / kSlab) * kSlab;
    g.rows = rows;
    g.splits = std::max<int64_t>(1, (n + rows - 1) / rows);
  }
  g.part_bytes = (size_t)g.splits * p * q * sizeof(double);
  return g;
}
template GramPlan gram_plan<double>(int64_t, int, int, bool);
template GramPlan gram_plan<float>(int64_t, int, int, bool);

template <class T>
void launch_gram_part(const GramPlan& g, int64_t n, const T* A, int64_t lda, int p, const T* B,
                      int64_t ldb, int q, double* C, int64_t ldc, double* part, hipStream_t s,
                      double scale) {
  if (p == 0 || q == 0) return;
  PhaseTick tick(PhaseClock::GRAM, s);
  hipLaunchKernelGGL(k_gram<T>, dim3((unsigned)(g.tiles * g.splits)), dim3(256), 0,
                     s, n, A, lda, p, B, ldb, q, g.sym, g.tiles, g.rows, part);
  MBL_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_gram_fold, dim3((unsigned)(((int64_t)p * q + 15) / 16)), dim3(256), 0, s,
                     part, (int)g.splits, p, q, g.sym, scale, C, ldc);
  MBL_CHECK_LAUNCH();
}

template <class T>
void launch_gram(int64_t n, const T* A, int64_t lda, int p, const T* B, int64_t ldb, int q,
                 double* C, int64_t ldc, hipStream_t s, double scale) {
  if (p == 0 || q == 0) return;
  const GramPlan g = gram_plan<T>(n, p, q, A == B && lda == ldb);
  DevBuf part(g.part_bytes, s);
  launch_gram_part<T>(g, n, A, lda, p, B, ldb, q, C, ldc, part.as<double>(), s, scale);
}

// ---- Gram partials in a fixed device array -------------------------------
// For callers that cannot allocate device memory (graph capture, tight
// loops): the per-split partial sums live in this file-scope array instead
// of a DevBuf.  Every k_gram launch writes each partial the fold reads, so
// nothing needs clearing between calls.  One copy per device; host code uses
// only the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double scratch[kGramScratchBytes / sizeof(double)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};
}  // namespace

double* gram_scratch() {
  int dev = 0;
  MBL_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) fail(MBL_EDEVICE, "device ordinal out of range for the Gram scratch");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch[dev] == nullptr) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr)
      fail(MBL_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch[dev] = static_cast<double*>(ptr);
  }
  return g_scratch[dev];
}

// Shapes of a combination: blocks of 16 columns per wavefront, wavefronts per workgroup.
struct CombineShape {
  int nb, nw;
};

// Wide: all 64 columns in one wavefront read A once, and 16 wavefronts share a C of up to 96
// KB (192 -> 64 columns, n = 184756, FP64, with masked loads: 122 us a call, in two blocks of
// 32 columns 135).
// Narrow: no work on absent columns, and for short sectors less C per workgroup and more
// workgroups (n = 3432, 192 -> 64, FP32: 12 us, wide 26).
//
// FP32 takes half the time a row, so what a short sector leaves idle shows (us a call, tiles
// of 16 rows on 256 CUs):
//  * up to 64 columns and 2048 tiles: one round of 8 wavefronts a workgroup (n = 24310, 192 ->
//    64: 18, narrow 23, wide 26);
//  * to 3072 tiles 3 workgroups of 4 are more even than 2 of 8 or 1 of 16 (n = 48620, 64 -> 64:
//    13.4, 16.5, 14.9), while C is short (192 -> 64: 33.7, wide 31.4);
//  * beyond one round of 16, to 6144 tiles, 8 (n = 92378, 64 -> 64: 21.1, wide 22.8);
//  * blocks of 48 columns where they are as few as blocks of 64 (n = 48620, 64 -> 36: 11.7,
//    wide 14.5; 96 -> 96: 24 and 31; n = 184756, 150 -> 75: 82 and 110).
template <class T>
CombineShape combine_shape(int64_t n, int p, int q) {
  if (q > 32 * 65535) return {4, 16};  // blocks of a grid
  if (q <= 32) return {2, 8};
  if (sizeof(T) == 4 && n > 16384) {
    const int64_t tiles = (n + 15) / 16;
    if (q <= 64 && tiles <= 2048) return {4, 8};
    if ((q + 47) / 48 == (q + 63) / 64) return {3, 16};
    if (q <= 64 && tiles <= 3072 && p <= 128) return {4, 4};
    if (q <= 64 && tiles > 4096 && tiles <= 6144) return {4, 8};
  }
  return n >= 32768 ? CombineShape{4, 16} : CombineShape{2, 8};
}

template <class T, int NB, int NW>
void launch_combine_as(int64_t n, const T* A, int64_t lda, int p, const double* C, int64_t ldc,
                       T* Y, int64_t ldy, int q, double beta, double scale, const double* colscale,
                       hipStream_t s) {
  using S = CombineStage<T>;
  constexpr size_t kLds = 96 * 1024;  // p = 192 of 64 FP64 columns in one chunk
  constexpr int W = 16 * NB;
  constexpr size_t row = S::row(NB) * sizeof(T);
  const int kc = (int)std::min<int64_t>(kLds / row / S::GK * S::GK,
                                        std::max<int64_t>(1, (p + S::GK - 1) / S::GK) * S::GK);
  const size_t lds = kc * row;
  const int64_t tiles = (n + 15) / 16;
  const int64_t cols = (q + W - 1) / W;
  // as many workgroups as are resident at once: each loads C once
  const int64_t per_cu = std::min<int64_t>(16 / NW, (160 * 1024) / (int64_t)lds);
  const int64_t grid = std::min<int64_t>((tiles + NW - 1) / NW,
                                         std::max<int64_t>(1, 256 * per_cu / cols));
  if (lds > 64 * 1024)
    MBL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_combine<T, NB, NW>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL((k_combine<T, NB, NW>), dim3((unsigned)grid, (unsigned)cols), dim3(64 * NW),
                     lds, s, n, A, lda, p, C, ldc, Y, ldy, q, beta, scale,
                     colscale, p % S::VE == 0, kc, tiles);
  MBL_CHECK_LAUNCH();
}

template <class T>
void launch_combine(int64_t n, const T* A, int64_t lda, int p, const double* C, int64_t ldc, T* Y,
                    int64_t ldy, int q, double beta, hipStream_t s, double scale,
                    const double* colscale) {
  if (n == 0 || q == 0) return;
  const CombineShape f = combine_shape<T>(n, p, q);
  auto run = [&](auto nb, auto nw) {
    launch_combine_as<T, decltype(nb)::value, decltype(nw)::value>(n, A, lda, p, C, ldc, Y, ldy, q,
                                                                   beta, scale, colscale, s);
  };
  using I2 = std::integral_constant<int, 2>;
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  using I16 = std::integral_constant<int, 16>;
  if (f.nb == 2) return run(I2{}, I8{});
  if constexpr (sizeof(T) == 4) {
    if (f.nb == 3) return run(std::integral_constant<int, 3>{}, I16{});
    if (f.nw == 4) return run(I4{}, I4{});
    if (f.nw == 8) return run(I4{}, I8{});
  }
  run(I4{}, I16{});
}

// One block of columns: a wavefront has read its 16 rows of A when it writes them, and no
// other reads them (rows read ahead beyond the end are not used).
template <class T>
bool combine_in_place(int64_t n, int p, int q) {
  return q <= 16 * combine_shape<T>(n, p, q).nb;
}
template bool combine_in_place<double>(int64_t, int, int);
template bool combine_in_place<float>(int64_t, int, int);

template <class T>
void launch_residual(int64_t n, int b, const T* A, int64_t lda, double sign, const T* X,
                     int64_t ldx, const double* mu, T* R, int64_t ldr, hipStream_t s) {
  if (n * b == 0) return;
  hipLaunchKernelGGL(k_residual<T>, dim3(g1(n * b)), dim3(256), 0, s, n, b, A, lda, (T)sign, X, ldx,
                     mu, R, ldr);
  MBL_CHECK_LAUNCH();
}

template <class S, class D>
void launch_convert(int64_t n, int b, const S* X, int64_t ldx, D* Y, int64_t ldy, hipStream_t s) {
  if (n * b == 0) return;
  hipLaunchKernelGGL((k_convert<S, D>), dim3(g1(n * b)), dim3(256), 0, s, n, b, X, ldx, Y, ldy);
  MBL_CHECK_LAUNCH();
}

void launch_diag_precond(int64_t n, int b, const double* R, int64_t ldr, const double* E,
                         double sign, const double* mu, double floor, double* W, int64_t ldw,
                         hipStream_t s) {
  if (n * b == 0) return;
  hipLaunchKernelGGL(k_diag_precond, dim3(g1(n * b)), dim3(256), 0, s, n, b, R, ldr, E, sign, mu,
                     floor, W, ldw);
  MBL_CHECK_LAUNCH();
}

template <class T>
void launch_randn(int64_t n, int b, uint64_t seed, T* X, int64_t ldx, hipStream_t s) {
  if (n * b == 0) return;
  hipLaunchKernelGGL(k_randn<T>, dim3(g1(n * b)), dim3(256), 0, s, n, b, seed, X, ldx);
  MBL_CHECK_LAUNCH();
}

template void launch_gram<double>(int64_t, const double*, int64_t, int, const double*, int64_t,
                                  int, double*, int64_t, hipStream_t, double);
template void launch_gram<float>(int64_t, const float*, int64_t, int, const float*, int64_t, int,
                                 double*, int64_t, hipStream_t, double);
template void launch_gram_part<double>(const GramPlan&, int64_t, const double*, int64_t, int,
                                       const double*, int64_t, int, double*, int64_t, double*,
                                       hipStream_t, double);
template void launch_gram_part<float>(const GramPlan&, int64_t, const float*, int64_t, int,
                                      const float*, int64_t, int, double*, int64_t, double*,
                                      hipStream_t, double);
template void launch_combine<double>(int64_t, const double*, int64_t, int, const double*, int64_t,
                                     double*, int64_t, int, double, hipStream_t, double,
                                     const double*);
template void launch_combine<float>(int64_t, const float*, int64_t, int, const double*, int64_t,
                                    float*, int64_t, int, double, hipStream_t, double,
                                    const double*);
template void launch_residual<double>(int64_t, int, const double*, int64_t, double, const double*,
                                      int64_t, const double*, double*, int64_t, hipStream_t);
template void launch_residual<float>(int64_t, int, const float*, int64_t, double, const float*,
                                     int64_t, const double*, float*, int64_t, hipStream_t);
template void launch_convert<double, float>(int64_t, int, const double*, int64_t, float*, int64_t,
                                            hipStream_t);
template void launch_convert<float, double>(int64_t, int, const float*, int64_t, double*, int64_t,
                                            hipStream_t);
template void launch_convert<double, double>(int64_t, int, const double*, int64_t, double*,
                                             int64_t, hipStream_t);
template void launch_convert<float, float>(int64_t, int, const float*, int64_t, float*, int64_t,
                                           hipStream_t);
template void launch_randn<double>(int64_t, int, uint64_t, double*, int64_t, hipStream_t);
template void launch_randn<float>(int64_t, int, uint64_t, float*, int64_t, hipStream_t);

}  // namespace mbl
