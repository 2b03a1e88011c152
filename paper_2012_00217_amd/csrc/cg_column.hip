// Block Jacobi-PCG on the spectral fold for sectors small enough that one CG
// vector fits the LDS of a CU (paper Sec. 3.2): one workgroup runs every CG step
// of one column in one launch.
//
// What bounds the launch-per-kernel form at these sizes is latency: at n = 924 the
// five kernels of a step take 21 us of device time and 32 us with their gaps, for
// about 1 us of arithmetic.  The columns of a block CG are independent, so a
// workgroup that owns a column needs no other synchronisation than its own
// barriers (four per step): the vector being gathered (p, then T) sits in LDS, the
// other CG vectors in registers, and the neighbour lists, which are the same
// in every step, in registers too up to 4 rows per thread (n <= 4096), else they
// are read from the L2.
//
// Sums: per thread over its rows, butterfly over the wavefront, wavefronts in order.
#include <algorithm>

#include "common.h"

namespace mbl {
namespace {

constexpr int kColThreads = 1024;
constexpr int kColSlots = 16;        // most flips of one row
constexpr int kColChunk = 1024;      // CG steps per launch
constexpr int kColStopChunk = 32;    // with a stop check

// Neighbour list of each row: four times its flip targets in bond order (the byte
// offset of an FP32 entry), 16 bits each, then 4 n, where the CG kernel keeps a
// zero.  Two vectors of 8 per row, [half][row].
__global__ __launch_bounds__(256) void k_col_tab(const uint32_t* __restrict__ states, int n, int L,
                                                 const uint32_t* __restrict__ pascal,
                                                 uint16_t* __restrict__ tab) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  if (row >= n) return;
  const uint32_t s = states[row];
  int m = 0;
  auto put = [&](int v) {
    tab[((size_t)(m >> 3) * n + row) * 8 + (m & 7)] = (uint16_t)(4 * v);
    ++m;
  };
  for (int i = 0; i + 1 < L; ++i) {
    if (!(((s ^ (s >> 1)) >> i) & 1u)) continue;
    const int c = (int)pascal[i * kPascal + __popc(s & ((1u << i) - 1u))];
    const int t = row + (((s >> i) & 1u) ? c : -c);
    if (t >= 0 && t < n && m < kColSlots) put(t);
  }
  while (m < kColSlots) put(n);
}

// Ticks of the device's wall clock that a column spent in its two applies (each with its
// sum), over all launches.
struct ColClock {
  uint64_t apply[2];
};

template <class T>
struct ColArgs {
  const uint4* tab;
  const double* diag;
  const T* jac;
  const T* R;
  int64_t ldr;
  T* W;
  int64_t ldw;
  T* r;        // state between launches (and p, x of LEAN), [column][n]
  T* p;
  T* x;
  PcgCoef* coef;
  ColClock* clock;  // TIMED: per column
  int n, m, m_keep, keep;  // columns [0, keep) run m_keep steps, the others m
  double sigma, halfJ;
};

// Several problems in one launch (the fused CG of a batch): problem j owns
// workgroups [c0[j], c0[j + 1]), one per column.
constexpr int kColFuse = 8;
template <class T>
struct ColMulti {
  int np, from, count;  // this launch: steps [from, from + count)
  int flush;            // no more steps: the state reached is the result
  int c0[kColFuse + 1];
  ColArgs<T> a[kColFuse];
};
static_assert(sizeof(ColMulti<double>) <= 4096, "kernel arguments too large");

__device__ inline double block_sum(double s, double* sw) {
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = s;
  __syncthreads();
  s = sw[0];
  const int nw = blockDim.x >> 6;
  for (int v = 1; v < nw; ++v) s += sw[v];
  return s;
}

// K rows per thread: row = tid + k * blockDim.  LEAN (more rows than the registers
// hold vectors for): r and T take the registers; x, p and the diagonals are read
// and written in memory (in the L2).  TIMED: a kernel of its own, since reading the clock
// under a branch costs every call 1.4% (n = 924).
template <class T, int K, bool LEAN, bool TIMED>
__global__ __launch_bounds__(kColThreads) void k_cg_col(ColMulti<T> mm) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sw[2][kColThreads / 64];
  T* g = reinterpret_cast<T*>(smem);  // gathered vector, g[n] = 0
  constexpr bool kRegTab = K <= 4;
  int job = 0;
  while (job + 1 < mm.np && (int)blockIdx.x >= mm.c0[job + 1]) ++job;
  const ColArgs<T>& a = mm.a[job];
  const int c = (int)blockIdx.x - mm.c0[job];
  const int steps = (c < a.keep ? a.m_keep : a.m) - mm.from;
  if (steps <= 0 && mm.from > 0) return;  // this column is done
  const int count = mm.flush ? 0 : min(mm.count, steps);
  const int n = a.n, tid = threadIdx.x, nt = blockDim.x;
  const T hj = (T)a.halfJ;
  const int64_t cb = (int64_t)c * n;
  T* xc = a.x + cb;
  T* pc = a.p + cb;

  T r[K], p[LEAN ? 1 : K], x[LEAN ? 1 : K], ed[LEAN ? 1 : K], dinv[LEAN ? 1 : K];
  uint4 f0[kRegTab ? K : 1], f1[kRegTab ? K : 1];
  PcgCoef cf;
  bool live;
  double rho;
  double rho0 = 0.0;
  if (tid == 0) g[n] = (T)0;
  // The row index is recomputed from an opaque copy in every pass: kept across the
  // steps, the addresses of all rows would take more registers than there are.
  int tr = tid;
  auto renew = [&]() { asm volatile("" : "+v"(tr)); };
  auto row = [&](int k) { return tr + k * nt; };
  auto rowc = [&](int k) { return (uint32_t)min(row(k), n - 1); };
  auto edof = [&](int k) { return (T)(a.diag[rowc(k)] - a.sigma); };
  auto dinvof = [&](int k) { return (T)1 / a.jac[rowc(k)]; };
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = row(k);
    const bool ok = i < n;
    if constexpr (!LEAN) {
      ed[k] = edof(k);
      dinv[k] = dinvof(k);
    }
    if constexpr (kRegTab) {
      f0[k] = a.tab[rowc(k)];
      f1[k] = a.tab[n + rowc(k)];
    }
    T pk;
    if (mm.from == 0) {
      r[k] = ok ? a.R[(int64_t)i * a.ldr + c] : (T)0;
      pk = r[k] * (LEAN ? dinvof(k) : dinv[LEAN ? 0 : k]);
      rho0 += (double)r[k] * (double)pk;
      if constexpr (LEAN) {
        if (ok) {
          xc[i] = (T)0;
          pc[i] = pk;
        }
      } else {
        x[k] = (T)0;
      }
    } else {
      r[k] = ok ? a.r[cb + i] : (T)0;
      pk = ok ? pc[i] : (T)0;
      if constexpr (!LEAN) x[k] = ok ? xc[i] : (T)0;
    }
    if constexpr (!LEAN) p[k] = pk;
    if (ok) g[i] = pk;
  }
  if (mm.from == 0) {
    rho = block_sum(rho0, sw[1]);
    live = rho > 0.0;
  } else {
    cf = a.coef[c];
    rho = cf.rho;
    live = cf.live != 0;
  }
  __syncthreads();

  // What row k reads from memory; fetched one row ahead of its use.
  struct Row {
    uint4 u0, u1;
    T ed, jac;  // LEAN
  };
  auto fetch = [&](int k, bool second) {
    Row w;
    if constexpr (!kRegTab) {
      w.u0 = a.tab[rowc(k)];
      w.u1 = a.tab[n + rowc(k)];
    }
    if constexpr (LEAN) {
      w.ed = (T)(a.diag[rowc(k)] - a.sigma);
      if (second) w.jac = a.jac[rowc(k)];
    }
    return w;
  };
  // (H - sigma) v for row k, v gathered from LDS; own is v at the row
  auto apply = [&](int k, const Row& w, T own) {
    uint4 u0, u1;
    if constexpr (kRegTab) {
      u0 = f0[kRegTab ? k : 0];
      u1 = f1[kRegTab ? k : 0];
      // the packed lists are kept, not the addresses in them
      asm volatile("" : "+v"(u0.x), "+v"(u0.y), "+v"(u0.z), "+v"(u0.w));
      asm volatile("" : "+v"(u1.x), "+v"(u1.y), "+v"(u1.z), "+v"(u1.w));
    } else {
      u0 = w.u0;
      u1 = w.u1;
    }
    T s = (T)0;
    auto two = [&](uint32_t v) {
      s += *reinterpret_cast<const T*>(smem + (v & 0xffffu) * (sizeof(T) / 4));
      s += *reinterpret_cast<const T*>(smem + (v >> 16) * (sizeof(T) / 4));
    };
    auto more = [&](uint32_t v) { return __any((int)(v & 0xffffu) != 4 * n); };
    two(u0.x);
    two(u0.y);
    if (more(u0.z)) {
      two(u0.z);
      two(u0.w);
      if (more(u1.x)) {
        two(u1.x);
        two(u1.y);
        if (more(u1.z)) {
          two(u1.z);
          two(u1.w);
        }
      }
    }
    const T v = (LEAN ? w.ed : ed[LEAN ? 0 : k]) * own + hj * s;
    return row(k) < n ? v : (T)0;
  };

  uint64_t ticks[2] = {0, 0}, mark = 0;
  for (int it = 0; it < count; ++it) {
    T t[K];
    if constexpr (TIMED) mark = wall_clock64();
    double s = 0.0;
    renew();
    Row next = fetch(0, false);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const Row w = next;
      if (k + 1 < K) next = fetch(k + 1, false);
      t[k] = apply(k, w, LEAN ? g[rowc(k)] : p[LEAN ? 0 : k]);
      s += (double)t[k] * (double)t[k];
      if constexpr (K > 2) __builtin_amdgcn_sched_barrier(0);
    }
    const double pap = block_sum(s, sw[0]);  // every gather of p is done
    if constexpr (TIMED) {
      const uint64_t now = wall_clock64();
      ticks[0] += now - mark;
      mark = now;
    }
    live = live && pap > 0.0;
    const double alpha = live ? rho / pap : 0.0;
    const T al = (T)alpha;
    renew();
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (row(k) < n) g[row(k)] = t[k];
    __syncthreads();
    s = 0.0;
    renew();
    next = fetch(0, true);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const Row w = next;
      if (k + 1 < K) next = fetch(k + 1, true);
      const T q = apply(k, w, t[k]);
      if constexpr (!LEAN) x[k] = x[k] + al * p[k];
      r[k] = r[k] - al * q;
      t[k] = r[k] * (LEAN ? (T)1 / w.jac : dinv[LEAN ? 0 : k]);  // z
      s += (double)r[k] * (double)t[k];
      if constexpr (K > 2) __builtin_amdgcn_sched_barrier(0);
    }
    const double rz = block_sum(s, sw[1]);  // every gather of T is done
    if constexpr (TIMED) ticks[1] += wall_clock64() - mark;
    live = live && rz > 0.0;
    const T be = (T)(live ? rz / rho : 0.0);
    if (live) rho = rz;
    renew();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = row(k);
      if constexpr (LEAN) {
        if (i < n) {
          T pk = pc[i];
          xc[i] = xc[i] + al * pk;
          if (live) pk = t[k] + be * pk;
          pc[i] = pk;
          g[i] = pk;
        }
        if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      } else {
        if (live) p[k] = t[k] + be * p[k];
        if (i < n) g[i] = p[k];
      }
    }
    __syncthreads();
  }
  if constexpr (TIMED)
    if (tid == 0)
      for (int i = 0; i < 2; ++i) a.clock[c].apply[i] += ticks[i];
  const bool done = mm.flush || count == steps;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = row(k);
    if (i >= n) continue;
    if (done) {
      T v;
      if constexpr (LEAN)
        v = xc[i];
      else
        v = x[k];
      a.W[(int64_t)i * a.ldw + c] = v;
    } else {
      a.r[cb + i] = r[k];
      if constexpr (!LEAN) {
        pc[i] = p[k];
        xc[i] = x[k];
      }
    }
  }
  if (!done && tid == 0) {
    cf.rho = rho;
    cf.live = live;
    a.coef[c] = cf;
  }
}

template <class T, int K, bool LEAN>
void launch_col(const ColMulti<T>& mm, int threads, size_t lds, hipStream_t s) {
  const auto kernel = mm.a[0].clock ? &k_cg_col<T, K, LEAN, true> : &k_cg_col<T, K, LEAN, false>;
  MBL_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kernel, dim3(mm.c0[mm.np]), dim3(threads), lds, s, mm);
  MBL_CHECK_LAUNCH();
}

int column_threads(int64_t n) {
  return n <= kColThreads ? (int)((n + 63) / 64 * 64) : kColThreads;
}

// Largest sector: 13 rows per thread (L = 16), which is also what LDS holds of FP64.
constexpr int kColMaxRows = 13 * kColThreads;
static_assert((kColMaxRows + 1) * sizeof(double) <= (156 << 10) && 4 * kColMaxRows < 65536,
              "a vector fits the LDS, an entry 16 bits");

}  // namespace

void build_column_tables(Ham& H, hipStream_t s) {
  const int flips = std::min(H.L - 1, 2 * std::min(H.nup, H.L - H.nup));
  H.col_ok = flips <= kColSlots && H.n <= kColMaxRows;
  if (!H.col_ok) return;
  H.table(H.col_tab, (size_t)H.n * kColSlots * sizeof(uint16_t), s);
  hipLaunchKernelGGL(k_col_tab, dim3((unsigned)((H.n + 255) / 256)), dim3(256), 0, s,
                     H.states.as<uint32_t>(), (int)H.n, H.L, H.pascal.as<uint32_t>(),
                     H.col_tab.as<uint16_t>());
  MBL_CHECK_LAUNCH();
}

bool column_grid_fits(int64_t n, int64_t b) { return b * column_threads(n) < (1ll << 32); }

// One CG of each job, all with the same number of rows per thread, in shared launches.
template <class T>
void run_pcg_column(const std::vector<ColumnJob<T>>& jobs, hipStream_t s, PcgTiming* tm,
                    const StopCheck* stop) {
  ColMulti<T> mm{};
  mm.np = (int)jobs.size();
  if (mm.np < 1 || mm.np > kColFuse) fail(MBL_EINTERNAL, "column pcg: group size out of range");
  int most = 0;
  int64_t nmax = 0;
  std::vector<DevBuf> keepalive;
  for (const ColumnJob<T>& j : jobs) {
    most = std::max(most, j.keep > 0 ? std::max(j.m, j.m_keep) : j.m);
    nmax = std::max(nmax, j.H->n);
  }
  const int chunk = stop ? kColStopChunk : kColChunk;
  const int rows = (int)((nmax + kColThreads - 1) / kColThreads);
  const bool lean = rows > 7 && sizeof(T) == 8;
  int wg = 0;
  for (int k = 0; k < mm.np; ++k) {
    const ColumnJob<T>& j = jobs[k];
    ColArgs<T>& a = mm.a[k];
    const size_t vec = (size_t)j.H->n * j.b * sizeof(T);
    a.tab = j.H->col_tab.template as<uint4>();
    a.diag = j.H->diag.template as<double>();
    a.jac = j.jac;
    a.R = j.R;
    a.ldr = j.ldr;
    a.W = j.W;
    a.ldw = j.ldw;
    a.n = (int)j.H->n;
    a.m = j.m;
    a.m_keep = std::max(j.m, j.m_keep);
    a.keep = j.keep > 0 ? j.keep : 0;
    a.sigma = j.sigma;
    a.halfJ = 0.5 * j.H->J;
    if (most > chunk) {
      keepalive.emplace_back(vec, s);
      a.r = keepalive.back().template as<T>();
      keepalive.emplace_back((size_t)j.b * sizeof(PcgCoef), s);
      a.coef = keepalive.back().template as<PcgCoef>();
    }
    if (most > chunk || lean) {
      keepalive.emplace_back(vec, s);
      a.x = keepalive.back().template as<T>();
      keepalive.emplace_back(vec, s);
      a.p = keepalive.back().template as<T>();
    }
    mm.c0[k] = wg;
    wg += j.b;
  }
  mm.c0[mm.np] = wg;
  const size_t lds = ((size_t)nmax + 1) * sizeof(T);
  const int threads = column_threads(nmax);
  auto launch = [&]() {
    if (rows <= 1)
      launch_col<T, 1, false>(mm, threads, lds, s);
    else if (rows <= 2)
      launch_col<T, 2, false>(mm, threads, lds, s);
    else if (rows <= 4)
      launch_col<T, 4, false>(mm, threads, lds, s);
    else if (rows <= 7)
      launch_col<T, 7, false>(mm, threads, lds, s);
    else
      launch_col<T, 13, sizeof(T) == 8>(mm, threads, lds, s);
  };
  hipEvent_t ev[2] = {nullptr, nullptr};
  struct Events {
    hipEvent_t* e;
    ~Events() {
      for (int i = 0; i < 2; ++i)
        if (e[i]) (void)hipEventDestroy(e[i]);
    }
  } guard{ev};
  if (stop)
    for (int i = 0; i < 2; ++i) MBL_HIP(hipEventCreateWithFlags(&ev[i], hipEventDisableTiming));
  DevBuf clockb;
  if (tm) {  // one job: a timed call does not share launches
    clockb.reset((size_t)wg * sizeof(ColClock), s);
    MBL_HIP(hipMemsetAsync(clockb.get(), 0, clockb.bytes(), s));
    mm.a[0].clock = clockb.as<ColClock>();
  }
  int from = 0, k = 0;
  do {
    mm.from = from;
    mm.count = std::min(chunk, most - from);
    launch();
    from += mm.count;
    if (stop && from < most) {
      // wait for the launch before this one, then decide whether to go on
      MBL_HIP(hipEventRecord(ev[k & 1], s));
      if (k > 0) MBL_HIP(hipEventSynchronize(ev[(k - 1) & 1]));
      ++k;
      if (stop->triggered()) {
        mm.from = from;
        mm.flush = 1;
        launch();
        break;
      }
    }
  } while (from < most);
  if (tm) {
    std::vector<ColClock> clock(wg);
    MBL_HIP(hipMemcpyAsync(clock.data(), clockb.get(), clockb.bytes(), hipMemcpyDeviceToHost, s));
    MBL_HIP(hipStreamSynchronize(s));
    int dev = 0, khz = 0;
    MBL_HIP(hipGetDevice(&dev));
    MBL_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    // The columns run side by side: the mean of their times.  The bytes are those that the
    // gather kernels would move for the columns that ran; here they stay on the CU.
    const ColumnJob<T>& j = jobs[0];
    const double n = (double)j.H->n, nw = n * sizeof(T);
    double ticks[2] = {0, 0}, cols = 0;  // cols: CG steps summed over the columns
    for (int c = 0; c < wg; ++c) {
      for (int i = 0; i < 2; ++i) ticks[i] += (double)clock[c].apply[i];
      cols += std::min(from, c < mm.a[0].keep ? mm.a[0].m_keep : mm.a[0].m);
    }
    const double by[2] = {2.0 * nw * cols + 12.0 * n * from,
                          6.0 * nw * cols + (12.0 + sizeof(T)) * n * from};
    tm->launches_all += from;
    for (int i = 0; i < 2; ++i) {
      const double ms = ticks[i] / wg / std::max(1, khz);
      tm->launches[i] += from;
      tm->ms[i] += ms;
      tm->bytes[i] += by[i];
      tm->ms_all[i] += ms;
      tm->bytes_all[i] += by[i];
    }
  }
}

template void run_pcg_column<double>(const std::vector<ColumnJob<double>>&, hipStream_t, PcgTiming*,
                                     const StopCheck*);
template void run_pcg_column<float>(const std::vector<ColumnJob<float>>&, hipStream_t, PcgTiming*,
                                    const StopCheck*);

}  // namespace mbl
