// MBL observables of computed eigenpairs (paper Sec. 2.2) and spectrum
// slicing (Sec. 3.1, third level of concurrency: eigenvalue chunks).
//
// Entanglement entropy across the cut between sites l-1 and l.  Write a
// sector state as s = u 2^l + v (u: right part, sites l..L-1; v: left part).
// The reduced density matrix of the left part is block diagonal in the number
// of up spins kA of v; its block is M M^T with M[v][u] = psi(s).  In the
// ascending (colex) row order the rows with one fixed u are consecutive and
// list the admissible v in the same order for every u, so column u of M is a
// contiguous segment of psi starting at the row of (u, lowest v).  Each block
// is therefore a Gram matrix of contiguous segments (or of their transposes,
// whichever dimension is smaller); its eigenvalues p give
// S = -sum p ln p.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <thread>

#include "common.h"

namespace mbl {
namespace {

// G (dim x dim) from segments of psi (column j of a row-major block, stride
// ld): by_rows -> G[i][k] = sum_u psi[st[u]+i] psi[st[u]+k] (dim = a, sum over
// c segments); else G[u1][u2] = sum_v psi[st[u1]+v] psi[st[u2]+v] (dim = c).
__global__ __launch_bounds__(256) void k_seg_gram(const double* __restrict__ psi, int64_t ld,
                                                  const int64_t* __restrict__ st, int c, int a,
                                                  int by_rows, double* __restrict__ G) {
  const int dim = by_rows ? a : c;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)dim * dim) return;
  const int i = (int)(e / dim), k = (int)(e % dim);
  double s = 0.0;
  if (by_rows) {
    for (int u = 0; u < c; ++u) s += psi[(st[u] + i) * ld] * psi[(st[u] + k) * ld];
  } else {
    for (int v = 0; v < a; ++v) s += psi[(st[i] + v) * ld] * psi[(st[k] + v) * ld];
  }
  G[e] = s;
}

// One block of the reduced density matrix (the same of every vector).
struct SegBlock {
  int a, c, by_rows, dim;
  int64_t st;  // its segments' first rows
  int64_t g;   // its Gram matrix in a vector's share of G
};

// The Gram matrices of all blocks and vectors at once: blockIdx.y = block,
// blockIdx.z = vector (contiguous: psi + z n).  Entries on and above the diagonal,
// which is what the eigensolver reads.
__global__ __launch_bounds__(256) void k_seg_gram_all(const double* __restrict__ psi, int64_t n,
                                                      const SegBlock* __restrict__ blocks,
                                                      const int64_t* __restrict__ st_all,
                                                      double* __restrict__ G, int64_t gsum) {
  const SegBlock b = blocks[blockIdx.y];
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= b.dim * b.dim) return;
  const int i = e / b.dim, k = e - i * b.dim;
  if (i > k) return;
  const double* v = psi + blockIdx.z * n;
  const int64_t* st = st_all + b.st;
  double s = 0.0;
  if (b.by_rows) {
    for (int u = 0; u < b.c; ++u) s += v[st[u] + i] * v[st[u] + k];
  } else {
    const double *x = v + st[i], *y = v + st[k];
    for (int u = 0; u < b.a; ++u) s += x[u] * y[u];
  }
  G[blockIdx.z * gsum + b.g + e] = s;
}

// out[j][r] = V[r][j], 64 x 16 tiles through LDS.
__global__ __launch_bounds__(256) void k_columns(const double* __restrict__ V, int64_t ldv,
                                                 int64_t n, int nv, double* __restrict__ out) {
  __shared__ double t[16][65];
  const int64_t r0 = (int64_t)blockIdx.x * 64;
  const int c0 = blockIdx.y * 16;
  for (int e = threadIdx.x; e < 64 * 16; e += 256) {
    const int r = e >> 4, c = e & 15;
    if (r0 + r < n && c0 + c < nv) t[c][r] = V[(r0 + r) * ldv + c0 + c];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 16; e += 256) {
    const int c = e >> 6, r = e & 63;
    if (r0 + r < n && c0 + c < nv) out[(int64_t)(c0 + c) * n + r0 + r] = t[c][r];
  }
}

int64_t binom(int n, int k) {
  if (k < 0 || k > n) return 0;
  int64_t r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

// Adds the entropy of the eigenvalues p[0 .. count) of a block.
void add_entropy(const double* p, int count, double* s) {
  for (int i = 0; i < count; ++i)
    if (p[i] > 1e-300) *s -= p[i] * std::log(p[i]);
}

constexpr int kBatchDim = 192;            // blocks the one-workgroup eigensolver takes
constexpr int kBatchBits = 16;            // right parts whose segments are listed at once
constexpr size_t kBatchBytes = 256 << 20; // device memory of one chunk of vectors

// Blocks of at most 192 rows, all of them and all vectors in three launches (the
// eigensolver of one block takes a fraction of a millisecond on one CU, and there
// are L / 2 of them for every vector).  ent[kA][j] gets the share of block kA of vector j;
// done[kA]: the block was taken.
void entropy_small_blocks(const Ham& H, const double* V, int64_t ldv, int nev, int cut,
                          std::vector<std::vector<double>>& ent, std::vector<char>& done,
                          hipStream_t s) {
  const int k = H.nup, R = H.L - cut;
  if (R > kBatchBits || H.n * sizeof(double) > kBatchBytes) return;
  std::vector<SegBlock> blocks;
  std::vector<int> which(cut + 1, -1);
  int64_t gsum = 0, wsum = 0, nst = 0;
  int maxdim = 0;
  std::vector<int> kAs;
  for (int kA = std::max(0, k - R); kA <= std::min(cut, k); ++kA) {
    const int64_t a = binom(cut, kA), c = binom(R, k - kA);
    if (std::min(a, c) > kBatchDim) continue;
    SegBlock b{(int)a, (int)c, a <= c, (int)std::min(a, c), nst, gsum};
    which[kA] = (int)blocks.size();
    blocks.push_back(b);
    kAs.push_back(kA);
    nst += c;
    gsum += (int64_t)b.dim * b.dim;
    wsum += b.dim;
    maxdim = std::max(maxdim, b.dim);
  }
  if (blocks.empty()) return;
  // first row of every right pattern u, with the lowest left pattern beside it
  std::vector<int64_t> st(nst);
  std::vector<int64_t> fill(blocks.size());
  for (size_t i = 0; i < blocks.size(); ++i) fill[i] = blocks[i].st;
  for (uint32_t u = 0; u < (1u << R); ++u) {
    const int kA = k - __builtin_popcount(u);
    if (kA < 0 || kA > cut || which[kA] < 0) continue;
    int64_t row = 0;
    int j = kA;
    for (uint32_t w = u; w; w &= w - 1)
      row += H.pascal_host[(cut + __builtin_ctz(w)) * kPascal + ++j];
    st[fill[which[kA]]++] = row;
  }
  const int chunk = (int)std::max<int64_t>(
      1, std::min<int64_t>(std::min(nev, 4096),
                           (int64_t)(kBatchBytes / ((H.n + gsum + wsum) * sizeof(double)))));
  // largest blocks first
  std::vector<int> order(blocks.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
  std::stable_sort(order.begin(), order.end(),
                   [&](int x, int y) { return blocks[x].dim > blocks[y].dim; });
  std::vector<int64_t> wat(blocks.size());
  for (size_t i = 0, at = 0; i < blocks.size(); at += blocks[i].dim, ++i) wat[i] = at;
  std::vector<EighItem> items;
  for (int i : order)
    for (int j = 0; j < chunk; ++j)
      items.push_back({blocks[i].dim, j * gsum + blocks[i].g, j * wsum + wat[i]});
  // one allocation and one upload: segment rows, blocks, items | columns, G, w
  std::vector<char> up(nst * sizeof(int64_t) + blocks.size() * sizeof(SegBlock) +
                       items.size() * sizeof(EighItem));
  const size_t at_b = nst * sizeof(int64_t), at_i = at_b + blocks.size() * sizeof(SegBlock);
  std::copy_n(reinterpret_cast<const char*>(st.data()), at_b, up.data());
  std::copy_n(reinterpret_cast<const char*>(blocks.data()), at_i - at_b, up.data() + at_b);
  std::copy_n(reinterpret_cast<const char*>(items.data()), up.size() - at_i, up.data() + at_i);
  const size_t head = (up.size() + 255) / 256 * 256;
  DevBuf buf;
  try {
    buf.reset(head + (size_t)chunk * (H.n + gsum + wsum) * sizeof(double), s);
  } catch (const Error& e) {
    if (e.status != MBL_ENOMEM) throw;
    (void)hipGetLastError();
    return;  // block by block, which needs no copy of the vectors
  }
  char* base = buf.as<char>();
  double* psi = reinterpret_cast<double*>(base + head);
  double* G = psi + (size_t)chunk * H.n;
  double* w = G + (size_t)chunk * gsum;
  MBL_HIP(hipMemcpyAsync(base, up.data(), up.size(), hipMemcpyHostToDevice, s));
  std::vector<double> p((size_t)chunk * wsum);
  for (int j0 = 0; j0 < nev; j0 += chunk) {
    const int nv = std::min(chunk, nev - j0);
    hipLaunchKernelGGL(k_columns, dim3((unsigned)((H.n + 63) / 64), (nv + 15) / 16), dim3(256), 0, s,
                       V + j0, ldv, H.n, nv, psi);
    MBL_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_seg_gram_all, dim3((maxdim * maxdim + 255) / 256, blocks.size(), nv),
                       dim3(256), 0, s, psi, H.n, reinterpret_cast<SegBlock*>(base + at_b),
                       reinterpret_cast<int64_t*>(base), G, gsum);
    MBL_CHECK_LAUNCH();
    if (nv < chunk) {  // the last chunk: the items of its vectors only
      items.clear();
      for (int i : order)
        for (int j = 0; j < nv; ++j)
          items.push_back({blocks[i].dim, j * gsum + blocks[i].g, j * wsum + wat[i]});
      MBL_HIP(hipMemcpyAsync(base + at_i, items.data(), items.size() * sizeof(EighItem),
                             hipMemcpyHostToDevice, s));
    }
    eigh_values((int)blocks.size() * nv, maxdim, G, reinterpret_cast<EighItem*>(base + at_i), w, s);
    MBL_HIP(hipMemcpyAsync(p.data(), w, (size_t)nv * wsum * sizeof(double), hipMemcpyDeviceToHost, s));
    MBL_HIP(hipStreamSynchronize(s));
    for (size_t i = 0; i < blocks.size(); ++i)
      for (int j = 0; j < nv; ++j)
        add_entropy(p.data() + j * wsum + wat[i], blocks[i].dim, &ent[kAs[i]][j0 + j]);
  }
  for (int kA : kAs) done[kA] = 1;
}

}  // namespace

void entanglement_entropy(const Ham& H, const double* V, int64_t ldv, int nev, int cut, double* S,
                          hipStream_t s) {
  const int L = H.L, k = H.nup, R = L - cut;
  std::vector<std::vector<double>> ent(cut + 1, std::vector<double>(nev, 0.0));
  std::vector<char> done(cut + 1, 0);
  entropy_small_blocks(H, V, ldv, nev, cut, ent, done, s);
  for (int kA = std::max(0, k - R); kA <= std::min(cut, k); ++kA) {
    if (done[kA]) continue;
    const int a = (int)binom(cut, kA), c = (int)binom(R, k - kA);
    if (a == 0 || c == 0) continue;
    // first row of every right-part pattern u (popcount k - kA), in order
    uint64_t vmin = (kA == 0) ? 0 : ((1ull << kA) - 1);
    std::vector<uint64_t> q;
    q.reserve(c);
    for (uint64_t u = 0; u < (1ull << R); ++u)
      if (__builtin_popcountll(u) == k - kA) q.push_back((u << cut) | vmin);
    DevBuf qd(q.size() * sizeof(uint64_t), s), st(q.size() * sizeof(int64_t), s);
    MBL_HIP(hipMemcpyAsync(qd.get(), q.data(), qd.bytes(), hipMemcpyHostToDevice, s));
    rank_states(H, qd.as<uint64_t>(), (int64_t)q.size(), st.as<int64_t>(), s);
    const bool by_rows = a <= c;
    const int dim = by_rows ? a : c;
    DevBuf G((size_t)dim * dim * sizeof(double), s), w((size_t)dim * sizeof(double), s),
        Z((size_t)dim * dim * sizeof(double), s), work(small_eigh_work_bytes(dim), s);
    std::vector<double> p(dim);
    for (int j = 0; j < nev; ++j) {
      hipLaunchKernelGGL(k_seg_gram, dim3((unsigned)(((int64_t)dim * dim + 255) / 256)), dim3(256),
                         0, s, V + j, ldv, st.as<int64_t>(), c, a, (int)by_rows, G.as<double>());
      MBL_CHECK_LAUNCH();
      // only the eigenvalues are needed: blocks up to 192 take the values-only path
      double* zv = dim + (dim & 1) <= kBatchDim ? nullptr : Z.as<double>();
      small_eigh(dim, G.as<double>(), dim, w.as<double>(), zv, dim, work, s);
      MBL_HIP(hipMemcpyAsync(p.data(), w.get(), dim * sizeof(double), hipMemcpyDeviceToHost, s));
      MBL_HIP(hipStreamSynchronize(s));
      add_entropy(p.data(), dim, &ent[kA][j]);
    }
  }
  for (int j = 0; j < nev; ++j) {
    S[j] = 0.0;
    for (int kA = 0; kA <= cut; ++kA) S[j] += ent[kA][j];
  }
}

double mean_gap_ratio(const double* e, int count) {
  std::vector<double> v(e, e + count);
  std::sort(v.begin(), v.end());
  double sum = 0;
  int m = 0;
  for (int i = 0; i + 2 < count; ++i) {
    const double d1 = v[i + 1] - v[i], d2 = v[i + 2] - v[i + 1];
    const double hi = std::max(d1, d2);
    if (hi > 0) {
      sum += std::min(d1, d2) / hi;
      ++m;
    }
  }
  return m ? sum / m : NAN;
}

// Several shifts of one Hamiltonian, `conc` at a time on worker streams that
// share the handle's read-only tables.
mbl_status solve_slices(const Ham& H, int count, const double* sigmas, int nev, int b, double tol,
                        const mbl_solve_opts& o, double* evals, double* resid, int conc) {
  int dev = 0;
  MBL_HIP(hipGetDevice(&dev));
  std::atomic<int> next{0};
  std::vector<mbl_status> st(count, MBL_EINTERNAL);
  auto worker = [&]() {
    (void)hipSetDevice(dev);
    hipStream_t s;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return;
    for (int i; (i = next.fetch_add(1)) < count;) {
      try {
        st[i] = solve_interior(H, sigmas[i], nev, b, tol, o, evals + (size_t)i * nev, nullptr, 0,
                               resid ? resid + (size_t)i * nev : nullptr, nullptr, s);
      } catch (const Error& e) {
        st[i] = e.status;
      } catch (...) {
        st[i] = MBL_EINTERNAL;
      }
    }
    (void)hipStreamSynchronize(s);
    (void)hipStreamDestroy(s);
  };
  std::vector<std::thread> pool;
  for (int t = 0; t < std::max(1, std::min(conc, count)); ++t) pool.emplace_back(worker);
  for (auto& t : pool) t.join();
  for (auto x : st)
    if (x != MBL_OK) return x;
  return MBL_OK;
}

}  // namespace mbl
