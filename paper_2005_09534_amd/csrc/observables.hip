// Observables of the returned eigenpairs (main text, "Entanglement entropy
// and level statistics"): the entanglement entropy of an eigenvector for a
// bipartition of the ring into two halves, and the mean gap ratio of the
// eigenvalues.
//
// Cut x (a bit offset): the first half holds bits x .. x+h-1 (mod L), h =
// L/2, the second the other h bits in ring order.  With t = s rotated right
// by x, a = t & (2^h - 1) and b = t >> h.  A state of zero magnetisation has
// popcount(a) = n and popcount(b) = h - n, so the coefficient matrix
// psi[a][b] is block diagonal by n: block n is C(h, n) x C(h, n), and the
// blocks hold exactly the C(L, h) coefficients (Vandermonde's identity).
// The squared Schmidt coefficients are the eigenvalues of the blocks' Gram
// matrices M_n^T M_n; S_E = -sum lambda ln lambda.
//
// Device steps: scatter each (vector, cut) into its blocks (row and column
// by the colex rank of a and b among patterns of their weight); one workgroup
// a block forms its Gram matrix, takes its eigenvalues with the LDS Jacobi
// (blocks up to 128 x 128, i.e. L <= 18) and sums -lambda ln lambda; and the
// sums of a (vector, cut)'s blocks are added up.
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"
#include "jacobi_lds.h"

namespace polfed {

constexpr int kEntBlocks = 10;  // L <= 18: weights 0 .. 9

__device__ __forceinline__ int colex_rank(uint32_t pat, int bits, const int32_t *binom) {
  int r = 0, t = 0;
  for (int q = 0; q < bits; ++q)
    if ((pat >> q) & 1u) r += binom[32 * q + (++t)];
  return r;
}

// out[p][off[n] + rb * d_n + ra] = V[r][j], pair p = j * ncut + c.
__global__ void k_ent_scatter(long long n, int L, const uint32_t *states, const double *V,
                              long long ldv, int ncut, const int *cuts, const int32_t *binom,
                              const long long *off, double *out, int p0) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int p = p0 + (int)blockIdx.y;
  const int j = p / ncut, c = p % ncut;
  const int h = L / 2;
  const int x = cuts[c];
  const uint32_t full = (L >= 32) ? 0xffffffffu : ((1u << L) - 1u);
  const uint32_t s = states[r];
  const uint32_t t = x ? (((s >> x) | (s << (L - x))) & full) : s;
  const uint32_t a = t & ((1u << h) - 1u), b = t >> h;
  const int na = __popc(a);
  const int d = binom[32 * h + na];
  const int ra = colex_rank(a, h, binom), rb = colex_rank(b, L - h, binom);
  out[(size_t)blockIdx.y * n + off[na] + (size_t)rb * d + ra] = V[(size_t)r * ldv + j];
}

// The blocks of one (vector, cut) pair: block q is d x d at offset off.
struct EntBlocks {
  int count;
  int d[kEntBlocks];
  long long off[kEntBlocks];
  int slot[kEntBlocks];  // where its sum goes among the pair's count sums
};

// One workgroup a block: its Gram matrix G[i][k] = sum_b M[b][i] M[b][k] and
// that matrix's eigenvalues lambda, all in LDS, then part = -sum lambda ln
// lambda (ascending).  Blocks of every size in one launch, the largest first:
// one launch a size left most of the chip idle (L = 16, 20 vectors, 8 cuts:
// 160 workgroups of each of 9 sizes, 4.7 ms in all; 0.74 ms so), with the
// eigenvectors, which nothing needs, half of each.
__global__ __launch_bounds__(kEigThreads) void k_ent_blocks(long long n, int pairs, EntBlocks eb,
                                                            const double *M, double *part) {
  extern __shared__ double sA[];  // G: m * ld, kEigRed for reductions
  __shared__ JacobiRot rot;
  const int q = blockIdx.x / pairs, p = blockIdx.x % pairs;
  const int d = eb.d[q];
  const int m = eig_even(d), ld = eig_ld(d);
  double *red = sA + (size_t)m * ld;
  const double *Mb = M + (size_t)p * n + eb.off[q];
  for (int e = threadIdx.x; e < m * m; e += kEigThreads) {
    const int i = e / m, k = e % m;
    if (k < i) continue;
    double acc = 0.0;
    if (k < d)
      for (int b = 0; b < d; ++b) acc += Mb[(size_t)b * d + i] * Mb[(size_t)b * d + k];
    sA[i * ld + k] = acc;
    sA[k * ld + i] = acc;
  }
  __syncthreads();
  if (d <= 64)
    jacobi_sweeps<64, false>(d, sA, red, rot, kEigSweeps, nullptr);
  else
    jacobi_sweeps<128, false>(d, sA, red, rot, kEigSweeps, nullptr);
  __syncthreads();
  double *lam = red;
  for (int i = threadIdx.x; i < d; i += kEigThreads) {
    const double di = sA[i * ld + i];
    int rank = 0;
    for (int j = 0; j < d; ++j) {
      const double dj = sA[j * ld + j];
      rank += (dj < di || (dj == di && j < i)) ? 1 : 0;
    }
    lam[rank] = di;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < d; i += kEigThreads) {
    const double l = lam[i];
    lam[i] = (l > 1e-300) ? l * log(l) : 0.0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double acc = 0.0;
    for (int k = 0; k < d; ++k) acc -= lam[k];
    part[(size_t)p * eb.count + eb.slot[q]] = acc;
  }
}

// S[p] = sum of pair p's count sums, in order.
__global__ void k_ent_sum(int count, int pairs, const double *part, double *S) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= pairs) return;
  double acc = 0.0;
  for (int k = 0; k < count; ++k) acc += part[(size_t)p * count + k];
  S[p] = acc;
}

void entanglement_entropy(hipStream_t st, const Basis &bs, int nvec, const double *V,
                          long long ldv, const std::vector<int> &cuts, double *S_host,
                          DevBuf &work) {
  const int L = bs.L, h = L / 2;
  const long long n = bs.n;
  PF_REQUIRE(L >= 2 && L <= 18, "entanglement: L must be in [2, 18] (blocks up to 128 x 128)");
  const int ncut = (int)cuts.size();
  const long long npairs = (long long)nvec * ncut;
  std::vector<long long> d(h + 1), off(h + 2, 0);
  for (int k = 0; k <= h; ++k) {
    long long c = 1;
    for (int i = 1; i <= k; ++i) c = c * (h - k + i) / i;  // C(h, k)
    d[k] = c;
    off[k + 1] = off[k] + c * c;
  }
  PF_REQUIRE(off[h + 1] == n, "entanglement: block sizes do not add up to the sector");
  // pairs in chunks, each chunk's blocks, Gram matrices and eigenvalues
  // within a bounded workspace
  const long long chunk = std::max<long long>(1, std::min<long long>(npairs, 512));
  // the blocks, largest first
  EntBlocks eb;
  eb.count = h + 1;
  std::vector<int> order(h + 1);
  for (int k = 0; k <= h; ++k) order[k] = k;
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return d[x] > d[y]; });
  for (int q = 0; q <= h; ++q) {
    eb.d[q] = (int)d[order[q]];
    eb.off[q] = off[order[q]];
    eb.slot[q] = order[q];
  }
  const size_t shm = sizeof(double) * ((size_t)eig_even(eb.d[0]) * eig_ld(eb.d[0]) + kEigRed);
  PF_REQUIRE(eb.d[0] <= kLdsEigMax, "entanglement: block beyond the batched eigensolver (L <= 18)");
  PF_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_ent_blocks),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
  // workspace: S per pair, block offsets, cuts, then (256-byte aligned) the
  // sums of a chunk's blocks and n doubles for each of its pairs
  const size_t small = sizeof(double) * npairs + sizeof(long long) * (h + 2) + sizeof(int) * ncut;
  const size_t per = sizeof(double) * ((size_t)n + h + 1);
  char *ws = static_cast<char *>(work.ensure(small + per * chunk + 256));
  double *dS = reinterpret_cast<double *>(ws);
  long long *doff = reinterpret_cast<long long *>(ws + sizeof(double) * npairs);
  int *dcut = reinterpret_cast<int *>(ws + sizeof(double) * npairs + sizeof(long long) * (h + 2));
  double *part = reinterpret_cast<double *>(
      (reinterpret_cast<uintptr_t>(ws + small) + 255) & ~(uintptr_t)255);
  double *M = part + (size_t)(h + 1) * chunk;
  PF_HIP(hipMemcpyAsync(doff, off.data(), sizeof(long long) * (h + 2), hipMemcpyHostToDevice, st));
  PF_HIP(hipMemcpyAsync(dcut, cuts.data(), sizeof(int) * ncut, hipMemcpyHostToDevice, st));
  for (long long p0 = 0; p0 < npairs; p0 += chunk) {
    const int B = (int)std::min<long long>(chunk, npairs - p0);
    dim3 grid((unsigned)((n + 255) / 256), (unsigned)B);
    k_ent_scatter<<<grid, 256, 0, st>>>(n, L, bs.states.as<uint32_t>(), V, ldv, ncut, dcut,
                                        bs.binom.as<int32_t>(), doff, M, (int)p0);
    check_launch("k_ent_scatter");
    k_ent_blocks<<<(unsigned)(B * eb.count), kEigThreads, shm, st>>>(n, B, eb, M, part);
    check_launch("k_ent_blocks");
    k_ent_sum<<<(B + 255) / 256, 256, 0, st>>>(eb.count, B, part, dS + p0);
    check_launch("k_ent_sum");
  }
  PF_HIP(hipMemcpyAsync(S_host, dS, sizeof(double) * npairs, hipMemcpyDeviceToHost, st));
  PF_HIP(hipStreamSynchronize(st));
}

}  // namespace polfed

namespace polfed {

double mean_gap_ratio(const double *E, int n) {
  std::vector<double> e(E, E + n);
  std::sort(e.begin(), e.end());
  double acc = 0.0;
  for (int i = 0; i + 2 < n; ++i) {
    const double g1 = e[i + 1] - e[i], g2 = e[i + 2] - e[i + 1];
    const double lo = std::min(g1, g2), hi = std::max(g1, g2);
    acc += (hi > 0.0) ? lo / hi : 0.0;
  }
  return acc / (n - 2);
}

}  // namespace polfed
