// Plain block apply Y = (H - sigma I) X by blocks of rows (paper Sec. 3.2 and 4.1).
//
// The rows that share the high configuration hi (the sites above the lowest kTileQ) are a
// contiguous block of at most 252 rows, one tile.  A workgroup takes one tile of one
// column slice of 128 to 208 bytes: it stages its rows in LDS, gathers the flips inside the
// low half from there, and the flips inside hi from the rows of another block, at one
// offset for the whole tile.  Consecutive workgroups of an XCD take consecutive tiles, in
// the order of tile_rank, so that what they gather stays in the XCD's L2.
//
// Bound by bytes that miss the L2 where the block is wide (L = 24, 128 FP32 columns: 1400
// us, k_apply 1675) and by the loads of the gathers where it is narrow: k_apply
// computes every flip target, and its ragged blocks go in 8- and 4-byte lanes and a launch
// per chunk (L = 21, 17 FP64 columns: 100 us, here 34; L = 24, 2 FP64 columns 160, here
// 38).  Tiles of q = 9 or 11 low sites: 2 to 10 % slower; slices of 80 or 272 bytes where
// the rows are whole lines: 40 and 130 %.
//
// A row of a slice is a number of 16-byte pieces.  The last piece ends with the slice,
// overlapping its neighbour where the width is odd (both write the same values), so that
// ragged and unaligned blocks take the same loads as aligned ones.
//
// The sum over the bonds runs in their order from the lowest, as in k_apply, and the
// results are the same bits.
#include <algorithm>

#include "common.h"

namespace mbl {
namespace {

// Vectors of a piece: in registers and LDS, and as they lie in memory.
template <class T, int VE>
struct TileVec {
  typedef T type __attribute__((ext_vector_type(VE)));
  typedef T mem __attribute__((ext_vector_type(VE), aligned(sizeof(T))));
};

template <class T>
struct TileArgs {
  const PanelTile* tiles;
  const uint4* lo_tab;
  const double* diag;
  const T* X;
  T* Y;
  int64_t ldx, ldy;
  double sigma, halfJ;
  int b, W, G;        // columns; columns and pieces of a slice
  uint32_t rcp;       // 2^18 / G rounded up
  PanelSched ts;
};

template <class T, int VE>
__global__ __launch_bounds__(512) void k_apply_tile(TileArgs<T> a) {
  using V = typename TileVec<T, VE>::type;
  using VM = typename TileVec<T, VE>::mem;
  extern __shared__ __align__(16) unsigned char tile_lds[];  // row u at piece (u + 1) * G
  V* tile = reinterpret_cast<V*>(tile_lds);
  const int xcd = blockIdx.x & 7;
  const int lt = a.ts.first[xcd] + (int)(blockIdx.x >> 3);
  if (lt >= a.ts.first[xcd + 1]) return;
  const int slice = lt / a.ts.ntiles, t = lt - slice * a.ts.ntiles;
  const MBL_CONST PanelTile* tp = (const MBL_CONST PanelTile*)a.tiles + t;
  const int nr = tp->nrows, row0 = tp->row0, cnt = tp->cnt, aux = tp->aux;
  const int mlo = tp->mlo, mhi = tp->mhi;
  const int G = a.G, items = nr * G, nt = blockDim.x;
  const int c0 = min(slice * a.W, a.b - a.W);
  const T* X = a.X + (int64_t)row0 * a.ldx + c0;
  T* Y = a.Y + (int64_t)row0 * a.ldy + c0;
  const T hj = (T)a.halfJ;
  auto split = [&](int it, int& u, int& g) {  // item -> row, piece
    u = (int)(((uint32_t)it * a.rcp) >> 18);
    g = it - u * G;
  };
  auto load = [](const T* base, uint32_t off) {
    return (V)*reinterpret_cast<const VM*>(reinterpret_cast<const char*>(base) + off);
  };
  for (int it = threadIdx.x; it < items; it += nt) {
    int u, g;
    split(it, u, g);
    tile[G + it] = load(X, (uint32_t)(u * (int)a.ldx + min(g * VE, a.W - VE)) * (uint32_t)sizeof(T));
  }
  if (threadIdx.x < G) tile[threadIdx.x] = V(0);
  __syncthreads();
  for (int it = threadIdx.x; it < items; it += nt) {
    int u, g;
    split(it, u, g);
    const int col = min(g * VE, a.W - VE);
    const uint32_t vo = (uint32_t)(u * (int)a.ldx + col) * (uint32_t)sizeof(T);
    const uint4 f = a.lo_tab[aux + u];
    const double d = a.diag[row0 + u];
    const bool mid = u >= mlo && u < mhi;
    V vm = V(0);
    if (mid)  // rows [mlo, mhi) map to rows mbase + u
      vm = load(a.X + (int64_t)tp->mbase * a.ldx + c0, vo);
    V s = V(0);
    const V* tg = tile + g;
    auto flip = [&](uint32_t w, int k) { s += tg[((w >> (10 * k)) & 1023u) * G]; };
    const int ndl = (int)(f.w >> 28);
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
    s += vm;
    auto high = [&](int h, auto n_) {
      constexpr int N = decltype(n_)::value;
      V v[N];
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = load(X + (int64_t)tp->off[h + i] * a.ldx, vo);
#pragma unroll
      for (int i = 0; i < N; ++i) s += v[i];
    };
    int h = 0;
    for (; h + 4 <= cnt; h += 4) high(h, std::integral_constant<int, 4>{});
    if (h + 2 <= cnt) {
      high(h, std::integral_constant<int, 2>{});
      h += 2;
    }
    if (h < cnt) high(h, std::integral_constant<int, 1>{});
    const V own = tile[G + it];
    const T ed = (T)(d - a.sigma);
    V y;
#pragma unroll
    for (int e = 0; e < VE; ++e) y[e] = __builtin_elementwise_fma(hj, (T)s[e], (T)(ed * own[e]));
    VM* dst = reinterpret_cast<VM*>(Y + (int64_t)u * a.ldy + col);
    __builtin_nontemporal_store((VM)y, dst);
  }
}

template <class T, int VE>
bool launch_tile(const Ham& H, double sigma, const T* X, int64_t ldx, T* Y, int64_t ldy, int w,
                 int nsl, hipStream_t s) {
  const PanelTables& P = H.tile;
  TileArgs<T> a{};
  a.tiles = P.tiles;
  a.lo_tab = P.lo_tab;
  a.diag = H.diag.as<double>();
  a.X = X;
  a.Y = Y;
  a.ldx = ldx;
  a.ldy = ldy;
  a.sigma = sigma;
  a.halfJ = 0.5 * H.J;
  a.b = w;
  // whole pieces a slice; the last slice ends with the block, overlapping its neighbour
  a.W = std::min(w, ((w + nsl - 1) / nsl + VE - 1) / VE * VE);
  a.G = (a.W + VE - 1) / VE;
  a.rcp = (1u << 18) / a.G + 1;  // exact for the at most 252 x 13 items of a tile
  a.ts = panel_sched(H, P, nsl, 1 << 20);  // one workgroup per tile
  if (a.ts.nwg == 8 << 20) return false;     // 32-bit thread numbers of a grid
  const int most = (int)H.pascal_host[kTileQ * kPascal + kTileQ / 2];
  const size_t lds = (size_t)(most + 1) * a.G * VE * sizeof(T);
  // Narrow slices have too few items for 512 threads (L = 24, FP64: 2 columns 59 us, with
  // 256 threads 38; 8 columns 129 and 112; 17 columns 360 and 427; 64 1403 and 1491).
  const int nt = a.G <= 4 ? 256 : 512;
  hipLaunchKernelGGL((k_apply_tile<T, VE>), dim3((unsigned)a.ts.nwg), dim3(nt), lds, s, a);
  MBL_CHECK_LAUNCH();
  return true;
}

}  // namespace

template <class T>
bool tile_apply(const Ham& H, double sigma, const T* X, int64_t ldx, T* Y, int64_t ldy, int w,
                hipStream_t s) {
  constexpr int VE = 16 / (int)sizeof(T);
  const PanelTables& P = H.tile;
  if (!P.ok || ldx > (1 << 20)) return false;  // 32-bit byte offsets within a tile's rows
  // Slices of whole 128-byte lines where the rows are whole lines, else as few as slices of
  // at most 208 bytes allow.  A slice that cuts lines fetches both ends of every row, so
  // narrow ones cost the most: n = 705432, rows of 2048 bytes 1232 us (k_apply 1540, slices of
  // 144 bytes 2450), 1280 bytes 774 (980, 1321); of 800 bytes in 4 slices 730 (834, in 6 of
  // 144 898), 320 bytes in 2 226 (307, in 3 of 112 310), 192 bytes in one 88 (216, in 2 146).
  // Slices of 256 bytes leave the L2 fewer rows (1024 bytes: 721, in 8 whole lines 711; 720
  // bytes: 690, in 4 of 192 663).
  const int64_t bytes = w * (int64_t)sizeof(T);
  const bool lines = (reinterpret_cast<uintptr_t>(X) | (uintptr_t)(ldx * (int64_t)sizeof(T)) |
                      (uintptr_t)bytes) % 128 == 0;
  int64_t nsl = lines ? bytes / 128 : std::max<int64_t>(1, (bytes + 207) / 208);
  // short sectors: narrower slices, of at least 32 bytes, until the card is filled
  while (P.ntiles * nsl < 512 && bytes >= 64 * nsl) nsl *= 2;
  if (P.ntiles * nsl >= (1ll << 30)) return false;  // tile numbers
  return w >= VE ? launch_tile<T, VE>(H, sigma, X, ldx, Y, ldy, w, (int)nsl, s)
                 : launch_tile<T, 1>(H, sigma, X, ldx, Y, ldy, w, 1, s);
}

template bool tile_apply<double>(const Ham&, double, const double*, int64_t, double*, int64_t, int,
                                 hipStream_t);
template bool tile_apply<float>(const Ham&, double, const float*, int64_t, float*, int64_t, int,
                                hipStream_t);

}  // namespace mbl
