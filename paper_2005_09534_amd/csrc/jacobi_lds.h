// Cyclic Jacobi of one symmetric matrix in one workgroup's LDS (device code
// of dense.hip and observables.hip).
#pragma once
#include "internal.h"

namespace polfed {

// Round-robin ("tournament") ordering: with m = n rounded up to even, round r
// pairs position 0 with position m-1 and k with m-1-k, where position i >= 1
// holds index 1 + (i - 1 + r) mod (m-1); over m-1 rounds every pair meets once.
__device__ __forceinline__ int rr_index(int i, int r, int m) {
  return (i == 0) ? 0 : 1 + (i - 1 + r) % (m - 1);
}

// The rotation [[c, s], [-s, c]] that annihilates a_pq != 0, d = a_qq - a_pp:
// with e = 2 a_pq and h = sqrt(d^2 + e^2), c^2 = (1 + |d|/h)/2 and s = sign(d)
// e/(2 h c), the smaller angle.  Two reciprocal square roots, one after the
// other, are the whole chain (t = 1/(|th| + sqrt(th^2 + 1)), th = d/e, and
// c = 1/sqrt(t^2 + 1) have five divisions and square roots); d and e scaled by
// a power of two, so that no square leaves the range.
__device__ __forceinline__ void jacobi_cs(double apq, double d, double &c, double &s) {
  const int ex = -ilogb(fmax(fabs(d), fabs(apq)));
  d = ldexp(d, ex);
  const double e = 2.0 * ldexp(apq, ex);
  const double rh = rsqrt(d * d + e * e);
  const double c2 = 0.5 + 0.5 * fabs(d) * rh;
  const double rc = rsqrt(c2);
  c = c2 * rc;
  s = copysign(0.5 * rh * rc, d) * e;
}

// Rotation of the indices x and y (p < q of the two).
__device__ __forceinline__ void jacobi_angle(const double *A, int n, int x, int y, int &p, int &q,
                                             double &c, double &s) {
  p = x < y ? x : y;
  q = x < y ? y : x;
  c = 1.0;
  s = 0.0;
  if (q < n) {
    const double apq = A[(size_t)p * n + q];
    if (apq != 0.0)
      jacobi_cs(apq, A[(size_t)q * n + q] - A[(size_t)p * n + p], c, s);
  }
}

// Rotation of pair k in round r, computed from the round's input matrix
// (which no thread of the round writes), so every workgroup that needs it
// gets the same (p, q, c, s).
__device__ __forceinline__ void jacobi_rotation(const double *A, int n, int m, int r, int k,
                                                int &p, int &q, double &c, double &s) {
  jacobi_angle(A, n, rr_index(k, r, m), rr_index(m - 1 - k, r, m), p, q, c, s);
}

// Largest matrix that fits (12 KB of LDS besides it), and the largest whose eigenvectors fit beside it (149 KB of 160).
constexpr int kLdsEigMax = 128;
constexpr int kLdsVecMax = 96;
constexpr int kEigThreads = 1024;
constexpr int kEigRed = kEigThreads;  // doubles of LDS for the reductions

// The rotations of a round: pair k's indices p, q as byte offsets in
// a row (8 p, 8 q) and of rows, and (c, s).
struct JacobiRot {
  int4 at[2][kLdsEigMax / 2];
  double2 cs[2][kLdsEigMax / 2];
};
__host__ __device__ constexpr int eig_even(int n) { return n + (n & 1); }
// Doubles from one row of the LDS matrices to the next: odd, so that a column's
// elements fall into different banks (n = 64: 0.9 ms with rows of 64 doubles).
__host__ __device__ constexpr int eig_ld(int n) { return eig_even(n) + 1; }

enum { kVecNone = 0, kVecLds = 1, kVecGlobal = 2 };

// Sweeps over sA (LDS) until its off-diagonal Frobenius norm is 1e-14 of the
// diagonal's or stops falling; rotations accumulate onto V.  sA is m x m (rows
// eig_ld apart), m = n rounded up to even, its last row and column zero where n
// is odd (the rotations of that index are the identity); V is n rows eig_ld
// apart (kVecLds) or n in global memory (kVecGlobal); unused with kVecNone.
// All threads.
//
// A round is two phases: the first applies the round's rotations to A (the
// blocks on and above the diagonal, each mirrored); in the second, the first
// wave works out the next round's (a serial chain) while the other waves
// apply this round's to V.  With V in global memory its loads go in one batch
// a round.  One matrix from scratch, before and after (us): n = 33 309 and 190, n =
// 64 1068 and 612, n = 96 2931 and 1602, n = 128 7090 and 6237 (LDS reads and
// writes bound it: about 30 cycles for each wave of blocks and of V places).
template <int VM>
__device__ void jacobi_sweeps(int n, double *sA, double *V, double *red, JacobiRot &rot,
                              int max_sweeps) {
  const int t = threadIdx.x;
  constexpr int nt = kEigThreads;
  const int m = eig_even(n), ld = eig_ld(n);
  const int npair = m / 2;
  char *Ac = reinterpret_cast<char *>(sA);
  auto el = [&](int byte) -> double & { return *reinterpret_cast<double *>(Ac + byte); };
  // the 2 x 2 blocks (pair k1 rows, pair k2 >= k1 columns) of this thread, and
  // its (row, pair) places of V
  constexpr int kHalf = kLdsEigMax / 2;
  constexpr int kA = (kHalf * (kHalf + 1) / 2 + nt - 1) / nt;         // 3
  constexpr int kVmax = VM == kVecLds ? kLdsVecMax : kLdsEigMax;
  constexpr int kV = (kVmax * (kVmax / 2) + nt - 64 - 1) / (nt - 64);  // 5 or 9
  int ak[kA];  // k1 | k2 << 8
#pragma unroll
  for (int u = 0; u < kA; ++u) {
    int idx = t + u * nt, k1 = 0;
    ak[u] = -1;
    if (idx < npair * (npair + 1) / 2) {
      while (idx >= npair - k1) idx -= npair - k1++;  // row k1 holds k2 = k1 .. npair - 1
      ak[u] = k1 | ((k1 + idx) << 8);
    }
  }
  int vk[kV];  // row's first element | k << 16
#pragma unroll
  for (int u = 0; u < kV; ++u) {
    const int idx = t - 64 + u * (nt - 64);
    vk[u] = (VM != kVecNone && t >= 64 && idx < n * npair)
                ? ((idx / npair) * (VM == kVecLds ? ld : n) | ((idx % npair) << 16))
                : -1;
  }
  // this thread's pair: positions t and m - 1 - t, their indices of round 0
  // (x, y; one further each round, position 0 stays at index 0)
  auto rotate = [&](int x, int y, int b) {
    if (t >= npair) return;
    const int p = x < y ? x : y, q = x < y ? y : x;
    const double apq = sA[p * ld + q];
    double c = 1.0, s = 0.0;
    if (apq != 0.0) jacobi_cs(apq, sA[q * ld + q] - sA[p * ld + p], c, s);
    rot.at[b][t] = make_int4(8 * p, 8 * q, 8 * p * ld, 8 * q * ld);
    rot.cs[b][t] = make_double2(c, s);
  };
  double prev = -1.0;
  int b = 0;
  for (int sweep = 0; sweep < max_sweeps && n > 1; ++sweep) {
    int x = rr_index(t, 0, m), y = rr_index(m - 1 - t, 0, m);
    rotate(x, y, b);
    __syncthreads();
    for (int r = 0; r < m - 1; ++r) {
      // A <- J^T A J: the blocks are disjoint, each read and written by one
      // thread
#pragma unroll
      for (int u = 0; u < kA; ++u) {
        if (ak[u] < 0) continue;
        const int k1 = ak[u] & 255, k2 = ak[u] >> 8;
        const int4 e1 = rot.at[b][k1], e2 = rot.at[b][k2];
        const double2 r1 = rot.cs[b][k1], r2 = rot.cs[b][k2];
        const double a00 = el(e1.z + e2.x), a01 = el(e1.z + e2.y);
        const double a10 = el(e1.w + e2.x), a11 = el(e1.w + e2.y);
        const double b00 = r1.x * a00 - r1.y * a10, b01 = r1.x * a01 - r1.y * a11;
        const double b10 = r1.y * a00 + r1.x * a10, b11 = r1.y * a01 + r1.x * a11;
        const double d00 = b00 * r2.x - b01 * r2.y, d01 = b00 * r2.y + b01 * r2.x;
        const double d10 = b10 * r2.x - b11 * r2.y, d11 = b10 * r2.y + b11 * r2.x;
        el(e1.z + e2.x) = d00;
        el(e1.z + e2.y) = d01;
        el(e1.w + e2.x) = d10;
        el(e1.w + e2.y) = d11;
        if (k1 != k2) {
          el(e2.z + e1.x) = d00;
          el(e2.w + e1.x) = d01;
          el(e2.z + e1.y) = d10;
          el(e2.w + e1.y) = d11;
        }
      }
      __syncthreads();
      if (t > 0 && ++x == m) x = 1;
      if (++y == m) y = 1;
      if (r + 1 < m - 1) rotate(x, y, b ^ 1);
      if (VM != kVecNone && t >= 64) {  // V <- V J (columns p, q of every row)
        double vp[kV], vq[kV];
#pragma unroll
        for (int u = 0; u < kV; ++u) {
          if (vk[u] < 0) continue;
          const int4 e = rot.at[b][vk[u] >> 16];
          if (VM == kVecGlobal && e.y == 8 * n) continue;
          const char *v = reinterpret_cast<const char *>(V + (vk[u] & 0xffff));
          vp[u] = *reinterpret_cast<const double *>(v + e.x);
          vq[u] = *reinterpret_cast<const double *>(v + e.y);
        }
#pragma unroll
        for (int u = 0; u < kV; ++u) {
          if (vk[u] < 0) continue;
          const int4 e = rot.at[b][vk[u] >> 16];
          if (VM == kVecGlobal && e.y == 8 * n) continue;
          const double2 cs = rot.cs[b][vk[u] >> 16];
          char *v = reinterpret_cast<char *>(V + (vk[u] & 0xffff));
          *reinterpret_cast<double *>(v + e.x) = cs.x * vp[u] - cs.y * vq[u];
          *reinterpret_cast<double *>(v + e.y) = cs.y * vp[u] + cs.x * vq[u];
        }
      }
      __syncthreads();
      b ^= 1;
    }
    // off-diagonal and diagonal sums of squares
    double off = 0.0, dg = 0.0;
    for (int e = t; e < m * m; e += nt) {
      const double v = sA[(e / m) * ld + e % m];
      if (e / m == e % m) dg += v * v; else off += v * v;
    }
    auto total = [&](double x) {
      red[t] = x;
      __syncthreads();
      for (int h = nt / 2; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
      }
      const double r = red[0];
      __syncthreads();
      return r;
    };
    const double o = total(off), d = total(dg);
    // stop at a relative off-diagonal norm of 1e-14, or when the rounding
    // floor is reached (no further decrease)
    if (!(o > 1e-28 * d) || o == 0.0) break;
    if (prev >= 0.0 && sweep >= 3 && o > 0.5 * prev) break;
    prev = o;
  }
}

}  // namespace polfed
