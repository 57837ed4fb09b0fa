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

// Largest matrix the kernels are built for: 64 pairs, one for each lane of a
// wave (its 132 KB and 4 KB of sums and rotations leave 24 KB of the LDS).
constexpr int kLdsEigMax = 128;
constexpr int kEigThreads = 1024;
constexpr int kEigSweeps = 40;  // at most (about 8 are usual)
constexpr int kEigRed = 2 * kLdsEigMax;  // doubles of LDS for sums and ranks

// A round's rotations (c, s), for pair k's indices in their order of
// positions: s changes its sign with the order.
struct JacobiRot {
  double2 cs[2][kLdsEigMax / 2];
};
__host__ __device__ constexpr int eig_even(int n) { return n + (n & 1); }
// Doubles from one row of the LDS matrix to the next: odd, so that a column's
// elements fall into different banks (n = 64: 0.9 ms with rows of 64 doubles).
__host__ __device__ constexpr int eig_ld(int n) { return eig_even(n) + 1; }

// Sweeps over sA (LDS) until its off-diagonal Frobenius norm is 1e-14 of the
// diagonal's or stops falling; returns the number of rounds.  sA is m x m
// (rows eig_ld apart), m = n <= NM rounded up to even, its last row and column
// zero where n is odd (the rotations of that index are the identity).  All
// threads.  Round i's rotations go to log[i m/2 .. (i + 1) m/2) as well (LOOK;
// null: nowhere).
//
// A round is two phases.  LOOK, for one matrix alone on its CU, where latency
// bounds it: all 2 x 2 blocks of A are read; then they are turned and written
// back, each mirrored, while the first wave works out the next round's
// rotations (a serial chain) from the entries that it has read and turned for
// itself.  Without LOOK, which takes half the registers, so that two
// workgroups share a CU and the LDS bounds them: all blocks of the upper
// triangle are turned, then the first wave works out the next round's.  The
// indices of a block go on by one a round in registers, so that its loads wait
// for the barrier alone.  The entropies of L = 16 take 737 us without LOOK,
// 804 mirrored too, 1093 with it, and took 1160 with the indices in LDS.
template <int NM, bool LOOK>
__device__ int jacobi_sweeps(int n, double *sA, double *red, JacobiRot &rot, int max_sweeps,
                             double2 *log) {
  const int t = threadIdx.x;
  constexpr int nt = kEigThreads;
  const int m = eig_even(n), ld = eig_ld(n);
  const int npair = m / 2;
  const int wrap = 8 * m;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  char *Ac = reinterpret_cast<char *>(sA);
  auto el = [&](int i, int j) -> double & {  // of indices times 8
    return *reinterpret_cast<double *>(
        Ac + (LOOK ? __mul24(i, ld) + j : __mul24(min(i, j), ld) + max(i, j)));
  };
  // the index (times 8) at a position in the next round: one further, position
  // 0 stays at index 0
  auto next = [&](int &x, bool moves) {
    const int y = x + 8 == wrap ? 8 : x + 8;
    x = moves ? y : x;
  };
  // waves 1 ..: the 2 x 2 blocks (pair k1 rows, pair k2 >= k1 columns) of this
  // thread and the indices of their pairs' positions
  constexpr int kHalf = NM / 2;
  constexpr int kA = (kHalf * (kHalf + 1) / 2 + nt - 64 - 1) / (nt - 64);  // 1 or 3
  int k1[kA], k2[kA], x1[kA], y1[kA], x2[kA], y2[kA];
#pragma unroll
  for (int u = 0; u < kA; ++u) {
    int idx = t - 64 + u * (nt - 64), k = 0;
    k1[u] = -1;
    k2[u] = x1[u] = y1[u] = x2[u] = y2[u] = 0;
    if (t >= 64 && idx < npair * (npair + 1) / 2) {
      while (idx >= npair - k) idx -= npair - k++;  // row k holds k2 = k .. npair - 1
      k1[u] = k;
      k2[u] = k + idx;
      x1[u] = 8 * k;
      y1[u] = 8 * (m - 1 - k);
      x2[u] = 8 * (k + idx);
      y2[u] = 8 * (m - 1 - k - idx);
    }
  }
  // wave 0: pair t of the next round is the index at its position k + 1 of now
  // (position 0 stays) with the one at m - k (position m - 1 takes position
  // 1's): the first (0) or second (1) of pairs jt and jb of now
  int jt = t + 1, jb = t - 1, st = 0, sb = 1;
  if (t == 0) {
    jt = 0;
    jb = npair > 1 ? 1 : 0;
    sb = npair > 1 ? 0 : 1;
  } else if (t == npair - 1) {
    jt = t;
    st = 1;
  }
  const bool looks = t < npair;
  if (!looks) jt = jb = 0;
  int tt = 8 * jt, tb = 8 * (m - 1 - jt), bt = 8 * jb, bb = 8 * (m - 1 - jb);
  int xr = 8 * t, yr = 8 * (m - 1 - t);  // pair t of now
  auto angle = [&](int b) {
    const double apq = el(xr, yr);
    double c = 1.0, s = 0.0;
    if (apq != 0.0) jacobi_cs(apq, el(yr, yr) - el(xr, xr), c, s);
    rot.cs[b][t] = make_double2(c, s);
  };
  if (looks) angle(0);
  // one block: its entries, and these turned and written back
  auto load = [&](int u, double (&a)[4]) {
    a[0] = el(x1[u], x2[u]);
    a[1] = el(x1[u], y2[u]);
    a[2] = el(y1[u], x2[u]);
    a[3] = el(y1[u], y2[u]);
  };
  auto turn = [&](int u, int b, const double (&a)[4]) {
    const double2 r1 = rot.cs[b][k1[u]], r2 = rot.cs[b][k2[u]];
    const double b00 = r1.x * a[0] - r1.y * a[2], b01 = r1.x * a[1] - r1.y * a[3];
    const double b10 = r1.y * a[0] + r1.x * a[2], b11 = r1.y * a[1] + r1.x * a[3];
    const double d00 = b00 * r2.x - b01 * r2.y, d01 = b00 * r2.y + b01 * r2.x;
    const double d10 = b10 * r2.x - b11 * r2.y, d11 = b10 * r2.y + b11 * r2.x;
    el(x1[u], x2[u]) = d00;
    el(x1[u], y2[u]) = d01;
    if (LOOK || k1[u] != k2[u]) el(y1[u], x2[u]) = d10;
    el(y1[u], y2[u]) = d11;
    if (LOOK && k1[u] != k2[u]) {
      el(x2[u], x1[u]) = d00;
      el(y2[u], x1[u]) = d01;
      el(x2[u], y1[u]) = d10;
      el(y2[u], y1[u]) = d11;
    }
    next(x1[u], k1[u] > 0);
    next(x2[u], k2[u] > 0);
    next(y1[u], true);
    next(y2[u], true);
  };
  __syncthreads();
  double prev = -1.0;
  int b = 0, rounds = 0;
  for (int sweep = 0; sweep < max_sweeps && n > 1; ++sweep) {
    for (int r = 0; r < m - 1; ++r) {
      // A <- J^T A J: the blocks are disjoint, each read and written by one
      // thread
      if constexpr (!LOOK) {
#pragma unroll
        for (int u = 0; u < kA; ++u) {
          if (k1[u] < 0) continue;
          double a[4];
          load(u, a);
          turn(u, b, a);
        }
        __syncthreads();
        next(xr, t > 0);
        next(yr, true);
        if (looks) angle(b ^ 1);
      } else if (wave == 0) {
        double p00 = 0, p01 = 0, p11 = 0, q00 = 0, q01 = 0, q11 = 0;
        double z00 = 0, z01 = 0, z10 = 0, z11 = 0;
        double2 r1 = make_double2(1.0, 0.0), r2 = r1;
        if (looks) {
          r1 = rot.cs[b][jt];
          r2 = rot.cs[b][jb];
          p00 = el(tt, tt);
          p01 = el(tt, tb);
          p11 = el(tb, tb);
          q00 = el(bt, bt);
          q01 = el(bt, bb);
          q11 = el(bb, bb);
          z00 = el(tt, bt);
          z01 = el(tt, bb);
          z10 = el(tb, bt);
          z11 = el(tb, bb);
        }
        __syncthreads();
        if (looks) {
          // the pair's first index turns into c first - s second, its second
          // into s first + c second
          const double f0 = st ? r1.y : r1.x, f1 = st ? r1.x : -r1.y;
          const double g0 = sb ? r2.y : r2.x, g1 = sb ? r2.x : -r2.y;
          const double axx = f0 * (f0 * p00 + f1 * p01) + f1 * (f0 * p01 + f1 * p11);
          const double ayy = g0 * (g0 * q00 + g1 * q01) + g1 * (g0 * q01 + g1 * q11);
          const double axy = f0 * (g0 * z00 + g1 * z01) + f1 * (g0 * z10 + g1 * z11);
          double c = 1.0, s = 0.0;
          if (axy != 0.0) jacobi_cs(axy, ayy - axx, c, s);
          rot.cs[b ^ 1][t] = make_double2(c, s);
          next(tt, jt > 0);
          next(bt, jb > 0);
          next(tb, true);
          next(bb, true);
        }
      } else {
        double a[kA][4];
#pragma unroll
        for (int u = 0; u < kA; ++u)
          if (k1[u] >= 0) load(u, a[u]);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kA; ++u)
          if (k1[u] >= 0) turn(u, b, a[u]);
        if (log != nullptr && wave == nt / 64 - 1 && (t & 63) < npair)
          log[(size_t)rounds * npair + (t & 63)] = rot.cs[b][t & 63];
      }
      ++rounds;
      __syncthreads();
      b ^= 1;
    }
    // off-diagonal and diagonal sums of squares
    double off = 0.0, dg = 0.0;
    for (int i = wave; i < m; i += nt / 64)
      for (int j = t & 63; j < m; j += 64) {
        const double x = sA[i * ld + j];
        if (i == j) dg += x * x; else if (i < j) off += 2.0 * (x * x);
      }
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) {
      off += __shfl_xor(off, h);
      dg += __shfl_xor(dg, h);
    }
    if ((t & 63) == 0) {
      red[t >> 6] = off;
      red[nt / 64 + (t >> 6)] = dg;
    }
    __syncthreads();
    double o = 0.0, d = 0.0;
    for (int i = 0; i < nt / 64; ++i) {
      o += red[i];
      d += red[nt / 64 + i];
    }
    __syncthreads();
    // stop at a relative off-diagonal norm of 1e-14, or when the rounding
    // floor is reached (no further decrease)
    if (!(o > 1e-28 * d) || o == 0.0) break;
    if (prev >= 0.0 && sweep >= 3 && o > 0.5 * prev) break;
    prev = o;
  }
  return rounds;
}

}  // namespace polfed
