// Dense FP64 kernels of the block-Lanczos side of POLFED.
//
// * Tall-skinny products on the matrix cores (v_mfma_f64_16x16x4f64):
//     gram   C = X^T Y   (A_j = Q_j^T U_j of eq. (Lan1), the projections
//                         Qm^T U of the full reorthogonalisation, U^T U of
//                         the QR step and U^T H~ U of Rayleigh-Ritz)
//     update Y = alpha X C + beta Y  (U - Q_{j-1} B_j^T, U - Q_j A_j,
//                         U - Qm (Qm^T U), Q = U R^{-1}, Ritz vectors Qm T)
//   The reduction of gram over rows is two-stage (per-workgroup partials,
//   then a fixed-order sum), so results are bitwise reproducible.
// * A cyclic Jacobi eigensolver (round-robin parallel ordering) for T_m and
//   the Rayleigh-Ritz matrix: one launch per round over the whole matrix,
//   double-buffered so that every workgroup derives the round's rotations
//   from an unmodified input; the host checks the off-diagonal norm between
//   sweeps.
// * Cholesky of the s x s Gram matrix for CholeskyQR.
// * Column reductions, Philox4x32-10 start vectors, and the single-vector
//   Lanczos helpers for the spectral bounds.
#include "internal.h"
#include "jacobi_lds.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace polfed {

typedef double d4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ gram --
//
// C = X^T Y on v_mfma_f64_16x16x4f64.  One MFMA step contracts 4 rows: lane l
// supplies A[i=l%16][k=l/16] and B[k=l/16][j=l%16]; the result tile holds
// D[l/16 + 4v][l%16] in component v of lane l (checked on gfx950).
//
// A wave owns 32 columns of X, as two tiles, the even and the odd ones, so
// that one 16-byte load feeds both; likewise 32 columns of Y (NB = 2 tiles) or
// 16 (NB = 1).  Of a workgroup's four waves, WM lie next to each other in X and
// WN in Y, the others share the rows of the chunk (their tiles are added in
// LDS); the next 8 rows are loaded while these are multiplied.  Bound by
// reading X where q <= 32, by MFMA at q = 64.  With 64 x 64 tiles whatever q
// was, 8-byte loads and chunks of at least 256 rows: n = 705,432, p = 480, q =
// 32 1040 us, n = 3,432, p = 104, q = 8 a call of 32 us; so 650 (4.3 TB/s) and 21.  (Four
// tiles of Y a wave, 64 registers of sums, spill.)

typedef double D2 __attribute__((ext_vector_type(2), aligned(8)));

// Two neighbouring elements of a row, zero past the last of `left`.
__device__ __forceinline__ D2 pair_load(const double *p, int left) {
  D2 v = {0.0, 0.0};
  if (left >= 2)
    v = *reinterpret_cast<const D2 *>(p);
  else if (left == 1)
    v[0] = p[0];
  return v;
}

// One operand of a wave: its lanes' columns of a row-major matrix of `cols`
// columns, as pairs (c, c + 1) or (PAIR false) singly.  Columns past the last
// one are read from within the row instead (what they give goes to rows or
// columns of the result that are not stored); of a pair that straddles the
// end, the one before it is read and its second value taken.  OFF: uint32_t
// where a lane's offset over four rows and the columns is below 4 GB (one
// address register a load), else uint64_t.
template <bool PAIR, class OFF>
struct GramSide {
  const char *base;   // of the row that comes next (scalar)
  long long step;     // bytes of four rows (scalar)
  OFF off;            // this lane's bytes: its row of the four, its column
  bool second;
  __device__ __forceinline__ GramSide() {}
  __device__ __forceinline__ GramSide(const double *M, long long ld, long long row, int cols,
                                      int c, int kk) {
    const int at = PAIR ? min(c, cols - 2) : min(c, cols - 1);
    second = PAIR && c > at;
    base = reinterpret_cast<const char *>(M + row * ld);
    step = 32 * ld;
    off = (OFF)(8 * (kk * ld + at));
  }
  __device__ __forceinline__ D2 fix(D2 v) const {
    if (PAIR && second) v[0] = v[1];
    return v;
  }
  __device__ __forceinline__ D2 at(const char *row, OFF lane) const {
    D2 v;
    if (PAIR)
      v = *reinterpret_cast<const D2 *>(row + lane);
    else
      v[0] = v[1] = *reinterpret_cast<const double *>(row + lane);
    return v;
  }
  // step s of the rows from here
  __device__ __forceinline__ D2 get(int s) const { return at(base + s * step, off); }
  // the last rows, `left` of the four: the others zero
  __device__ __forceinline__ D2 tail(int kk, int left, long long ld) const {
    D2 v = at(base, kk < left ? off : (OFF)(off - 8 * kk * ld));
    if (kk >= left) v = (D2){0.0, 0.0};
    return fix(v);
  }
};

template <int NB, int WM, int WN, bool PX, class OFF = uint32_t>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_gram(
    long long n, int p, int q, const double *X, long long ldx, const double *Y, long long ldy,
    double *part, long long rows_per_chunk, int tiles_m, int tiles_n) {
  constexpr int WK = 4 / (WM * WN);
  constexpr int RS = 2;  // steps of four rows loaded at once
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM % WN, wk = wave / (WM * WN);
  int t = blockIdx.x;
  const int tm = t % tiles_m;
  t /= tiles_m;
  const int tn = t % tiles_n;
  const int chunk = t / tiles_n;
  const long long c0 = (long long)chunk * rows_per_chunk;
  const long long c1 = (c0 + rows_per_chunk < n) ? c0 + rows_per_chunk : n;
  // this wave's rows of the chunk
  const long long per = rows_per_chunk / WK;
  const long long r0 = c0 + wk * per;
  const long long r1 = (r0 + per < c1) ? r0 + per : c1;
  const int i16 = lane & 15, kk = lane >> 4;

  const int x0 = (tm * WM + wm) * 32, y0 = (tn * WN + wn) * 16 * NB;
  d4 acc[2][NB];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < NB; ++v) acc[u][v] = (d4){0.0, 0.0, 0.0, 0.0};

  if (x0 < p && y0 < q && r0 < r1) {
    GramSide<PX, OFF> sx(X, ldx, r0, p, x0 + 2 * i16, kk);
    GramSide<(NB > 1), OFF> sy(Y, ldy, r0, q, y0 + (NB == 1 ? i16 : 2 * i16), kk);
    struct Rows {
      D2 a[RS], b[RS];
    };
    auto load = [&](Rows &w) {
#pragma unroll
      for (int s = 0; s < RS; ++s) {
        w.a[s] = sx.get(s);
        w.b[s] = sy.get(s);
      }
      sx.base += RS * sx.step;
      sy.base += RS * sy.step;
    };
    auto one = [&](D2 a, D2 b) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < NB; ++v)
          acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
    };
    auto multiply = [&](const Rows &w) {
#pragma unroll
      for (int s = 0; s < RS; ++s) one(sx.fix(w.a[s]), sy.fix(w.b[s]));
    };
    long long left = (r1 - r0) / (4 * RS);  // whole loads
    Rows cur, nxt;
    if (left > 0) load(cur);
    while (left > 0) {
      if (left > 1) load(nxt);
      multiply(cur);
      if (left == 1) break;
      if (left > 2) load(cur);
      multiply(nxt);
      left -= 2;
    }
    for (int rem = (int)((r1 - r0) % (4 * RS)); rem > 0; rem -= 4) {
      one(sx.tail(kk, rem, ldx), sy.tail(kk, rem, ldy));
      sx.base += sx.step;
      sy.base += sy.step;
    }
  }
  if constexpr (WK > 1) {  // the waves of one tile, in order
    constexpr int W1 = WM * WN;
    __shared__ d4 red[WK - 1][W1][2][NB][64];
    const int at = wave % W1;
    if (wk > 0)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < NB; ++v) red[wk - 1][at][u][v][lane] = acc[u][v];
    __syncthreads();
    if (wk > 0) return;
#pragma unroll
    for (int k = 0; k < WK - 1; ++k)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < NB; ++v) acc[u][v] += red[k][at][u][v][lane];
  }
  // partial tiles -> part[chunk][i][j] (p x q, row-major)
  double *out = part + (size_t)chunk * p * q;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < NB; ++v) {
      const int j = y0 + (NB == 1 ? i16 : 2 * i16 + v);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = x0 + 2 * (kk + 4 * c) + u;
        if (i < p && j < q) out[(size_t)i * q + j] = acc[u][v][c];
      }
    }
}

// C[i][j] = sum over chunks c of part[c][i][j]: a workgroup takes 16
// neighbouring elements (a line of every partial tile) with 16 lanes each,
// lane l adding chunks l, l + 16, ... in order, then the 16 lanes in order, so
// the result does not depend on timing.
__global__ __launch_bounds__(256) void k_gram_reduce(int p, int q, int nchunks,
                                                     const double *part, double *C,
                                                     long long ldc) {
  __shared__ double red[16][17];
  const int el = threadIdx.x & 15, g = threadIdx.x >> 4;
  const long long e = (long long)blockIdx.x * 16 + el;
  const long long pq = (long long)p * q;
  double s = 0.0;
  if (e < pq) {
#pragma unroll 8
    for (int c = g; c < nchunks; c += 16) s += part[(size_t)c * pq + e];
  }
  red[g][el] = s;
  __syncthreads();
  if (g == 0 && e < pq) {
    s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += red[k][el];
    const int i = (int)(e / q), j = (int)(e % q);
    C[(size_t)i * ldc + j] = s;
  }
}

// Tiles of the Gram product for a p x q output: a workgroup's waves along X
// and along Y (two tiles of Y a wave, one for q <= 16).
static void gram_tiles(int p, int q, int &wm, int &wn, int &tiles_m, int &tiles_n) {
  wn = q <= 32 ? 1 : 2;
  wm = p <= 32 ? 1 : (p <= 64 || wn == 2) ? 2 : 4;
  tiles_m = (p + 32 * wm - 1) / (32 * wm);
  tiles_n = (q + 32 * wn - 1) / (32 * wn);
}

// Row chunks of the Gram product for n rows and a p x q output: about four
// workgroups per CU in all, at least 64 rows a wave (four rounds of loads; n =
// 3,432, p = 104, q = 8: a call of 21 us with 64, 32 with 256), and (cap > 0) no more
// chunks than cap / (p q) partial tiles hold.
long long gram_chunks(long long n, int p, int q, int num_cu, long long cap,
                      long long &rows_per_chunk) {
  int wm, wn, tiles_m, tiles_n;
  gram_tiles(p, q, wm, wn, tiles_m, tiles_n);
  long long want = std::max<long long>(1, (4LL * num_cu) / (tiles_m * tiles_n));
  if (cap > 0) want = std::min<long long>(want, cap / ((long long)p * q));
  want = std::max<long long>(want, 1);
  const int wk = 4 / (wm * wn);
  rows_per_chunk = std::max<long long>(64 * wk, (n + want - 1) / want);
  rows_per_chunk = ((rows_per_chunk + 16 * wk - 1) / (16 * wk)) * (16 * wk);
  return std::max<long long>(1, (n + rows_per_chunk - 1) / rows_per_chunk);
}

void launch_gram_parts(hipStream_t st, long long n, int p, int q, const double *X,
                       long long ldx, const double *Y, long long ldy, double *C, long long ldc,
                       double *part, long long rows_per_chunk, long long nchunks) {
  int wm, wn, tiles_m, tiles_n;
  gram_tiles(p, q, wm, wn, tiles_m, tiles_n);
  // rows so far apart that a lane's offset passes 32 bits (there are few of
  // them): the smallest tile, with 64-bit offsets
  const bool far = 8.0 * (3.0 * (double)std::max(ldx, ldy) + std::max(p, q)) >= 4294967296.0;
  if (far) {
    tiles_m = (p + 31) / 32;
    tiles_n = (q + 15) / 16;
  }
  const unsigned nblk = (unsigned)(nchunks * tiles_m * tiles_n);
  auto go = [&](auto kernel) {
    kernel<<<nblk, 256, 0, st>>>(n, p, q, X, ldx, Y, ldy, part, rows_per_chunk, tiles_m, tiles_n);
  };
  if (far) {
    p < 2 ? go(k_gram<1, 1, 1, false, uint64_t>) : go(k_gram<1, 1, 1, true, uint64_t>);
  } else if (q <= 16) {
    if (p < 2)
      go(k_gram<1, 1, 1, false>);
    else
      wm == 1 ? go(k_gram<1, 1, 1, true>) : wm == 2 ? go(k_gram<1, 2, 1, true>) : go(k_gram<1, 4, 1, true>);
  } else if (wn == 1) {
    if (p < 2)
      go(k_gram<2, 1, 1, false>);
    else
      wm == 1 ? go(k_gram<2, 1, 1, true>) : wm == 2 ? go(k_gram<2, 2, 1, true>) : go(k_gram<2, 4, 1, true>);
  } else {
    if (p < 2)
      go(k_gram<2, 1, 2, false>);
    else
      wm == 1 ? go(k_gram<2, 1, 2, true>) : go(k_gram<2, 2, 2, true>);
  }
  check_launch("k_gram");
  const long long tot = (long long)p * q;
  k_gram_reduce<<<(unsigned)((tot + 15) / 16), 256, 0, st>>>(p, q, (int)nchunks, part, C, ldc);
  check_launch("k_gram_reduce");
}

void launch_gram(hipStream_t st, long long n, int p, int q, const double *X, long long ldx,
                 const double *Y, long long ldy, double *C, long long ldc, DevBuf &partials,
                 int num_cu) {
  if (p <= 0 || q <= 0) return;
  long long rows_per_chunk = 0;
  const long long nchunks = gram_chunks(n, p, q, num_cu, 0, rows_per_chunk);
  double *part = static_cast<double *>(partials.ensure(sizeof(double) * nchunks * p * q));
  launch_gram_parts(st, n, p, q, X, ldx, Y, ldy, C, ldc, part, rows_per_chunk, nchunks);
}

// ---------------------------------------------------------------- update --
//
// Y = alpha X C + beta Y.  A wave owns 16 rows and all q <= 64 columns (NB
// tiles of 16); the sum over k goes in blocks of KU, whose rows of C are
// staged in LDS once for the workgroup's NW waves (row stride = 16 mod 32
// doubles: the four rows of an MFMA step in different banks).  Lane l = (i =
// l%16, kk = l/16) reads X[row i][16 s + 4 kk .. + 3] of the block, so the four
// lanes of a row take a whole 128-byte line between them, and the k of MFMA
// step (s, e) is 16 s + 4 kk + e for both operands.  The next block's X is
// loaded while this one's is multiplied.  Bound by reading X, so by how many
// waves a SIMD holds: blocks of 64 left four of them (and 31 idle columns of 64
// at p = 33), blocks of 16 six to eight; with one tile of Y there is room for
// 32 (launch_update has the rule).  n = 705,432, us a launch with blocks of 64,
// 32, 16 (and, before there was any staging, with 8-byte loads of 4 k at a time
// and C from L1):
//   p =  33, q =  8:   73   51   49  (56)    p =  33, q = 64:  283  278  220  (251)
//   p =  64, q =  8:  103   81   90 (131)    p =  64, q = 32:  181  152  140  (211)
//   p = 480, q =  8:  571  540  577 (954)    p = 480, q = 32:  727  664  643 (1222)

// The wave's tiles: component v of lane l is element (l/16 + 4v, l%16).
template <int NB>
__device__ __forceinline__ void update_store(long long n, int q, double alpha, const d4 (&acc)[NB],
                                             double beta, double *Y, long long ldy,
                                             long long row0, int i16, int kk) {
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int j = u * 16 + i16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const long long row = row0 + kk + 4 * v;
      if (row < n && j < q) {
        double *y = Y + row * ldy + j;
        *y = (beta == 0.0) ? alpha * acc[u][v] : alpha * acc[u][v] + beta * (*y);
      }
    }
  }
}

template <int NB, int NW, int KU>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4))) void k_update(
    long long n, int p, int q, double alpha,
                                                    const double *X, long long ldx,
                                                    const double *C, long long ldc, double beta,
                                                    double *Y, long long ldy) {
  constexpr int kLd = NB == 1 ? 16 : (NB == 2 ? 48 : 80);
  constexpr int W = 16 * NB;
  constexpr int NS = KU / 16;
  __shared__ double sc[KU * kLd];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const long long row0 = ((long long)blockIdx.x * NW + wave) * 16;
  const int i16 = lane & 15, kk = lane >> 4;
  const long long ra = row0 + i16;
  const double *xr = X + (ra < n ? ra : 0) * ldx + 4 * kk;
  d4 acc[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) acc[u] = (d4){0.0, 0.0, 0.0, 0.0};
  D2 a[NS][2];
  auto load = [&](int k0) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        a[s][h] = pair_load(xr + k0 + 16 * s + 2 * h, p - (k0 + 16 * s + 4 * kk + 2 * h));
  };
  load(0);
  for (int k0 = 0; k0 < p; k0 += KU) {
    if (k0 > 0) __syncthreads();
    for (int e = threadIdx.x; e < KU * W; e += 64 * NW) {
      const int k = e / W, j = e % W;
      sc[k * kLd + j] = (k0 + k < p && j < q) ? C[(size_t)(k0 + k) * ldc + j] : 0.0;
    }
    __syncthreads();
    D2 b[NS][2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      b[s][0] = a[s][0];
      b[s][1] = a[s][1];
    }
    if (k0 + KU < p) load(k0 + KU);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int u = 0; u < NB; ++u)
          acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(
              b[s][e / 2][e % 2], sc[(16 * s + 4 * kk + e) * kLd + 16 * u + i16], acc[u], 0, 0, 0);
  }
  update_store<NB>(n, q, alpha, acc, beta, Y, ldy, row0, i16, kk);
}

// Sums of up to 8 terms: C straight from the caches; staging it and the barrier
// take longer than they save (n = 705,432, p = 1, a launch: q = 1 14.7 us
// against 16.5, q = 64 142 against 157).
template <int NB, int NW>
__global__ __launch_bounds__(64 * NW) void k_update_short(long long n, int p, int q, double alpha,
                                                          const double *X, long long ldx,
                                                          const double *C, long long ldc,
                                                          double beta, double *Y, long long ldy) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const long long row0 = ((long long)blockIdx.x * NW + wave) * 16;
  const int i16 = lane & 15, kk = lane >> 4;
  const long long ra = row0 + i16;
  d4 acc[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) acc[u] = (d4){0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < p; k0 += 4) {
    const int k = k0 + kk;
    const double a = (ra < n && k < p) ? X[ra * ldx + k] : 0.0;
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int j = 16 * u + i16;
      const double b = (k < p && j < q) ? C[(size_t)k * ldc + j] : 0.0;
      acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[u], 0, 0, 0);
    }
  }
  update_store<NB>(n, q, alpha, acc, beta, Y, ldy, row0, i16, kk);
}

void launch_update(hipStream_t st, long long n, int p, int q, double alpha, const double *X,
                   long long ldx, const double *C, long long ldc, double beta, double *Y,
                   long long ldy) {
  if (n <= 0 || q <= 0) return;
  if (q > 64) throw Error(POLFED_EINVAL, "update: q must be <= 64");
  if (p <= 0) {
    // Y = beta Y
    launch_update(st, n, 1, q, 0.0, X, ldx, C, ldc, beta, Y, ldy);
    return;
  }
  // eight waves share a block of C where that still gives every CU work
  const bool few = n < 65536;
  const int nw = few ? 4 : 8;
  // Blocks of k.  Many rows: 16, so that most waves share a SIMD, or 32 with one
  // tile of Y, where that is not half padding.  Few rows: there are few waves,
  // and what one has in flight counts for more; sums of up to 64 go in one block
  // where it is filled, long ones in blocks of 32 and 64 (n = 12,870, q = 32, in
  // blocks of 16, 32 and 64: p = 56 6.5, 6.3, 6.2 us; p = 80 7.4, 7.7, 8.9; p =
  // 160 11.2, 10.6, 11.8; p = 640 56.7, 48.8, 47.5).
  int ku = 16;
  if (few ? (p > 16 && p <= 32) || (p >= 128 && p < 256)
          : q <= 16 && ((p > 16 && p <= 32) || p > 48))
    ku = 32;
  else if (few && ((p > 48 && p <= 64) || p >= 256))
    ku = 64;
  const unsigned nwg = (unsigned)((n + 16 * nw - 1) / (16 * nw));
  auto go = [&](auto kernel) {
    kernel<<<nwg, 64 * nw, 0, st>>>(n, p, q, alpha, X, ldx, C, ldc, beta, Y, ldy);
  };
  auto with_nb = [&](auto nb_c) {
    constexpr int NB = decltype(nb_c)::value;
    if (p <= 8) {
      few ? go(k_update_short<NB, 4>) : go(k_update_short<NB, 8>);
      return;
    }
    if (few) {
      ku == 16 ? go(k_update<NB, 4, 16>) : ku == 32 ? go(k_update<NB, 4, 32>) : go(k_update<NB, 4, 64>);
      return;
    }
    if constexpr (NB == 1)
      if (ku == 32) return go(k_update<1, 8, 32>);
    go(k_update<NB, 8, 16>);
  };
  if (q <= 16)
    with_nb(std::integral_constant<int, 1>{});
  else if (q <= 32)
    with_nb(std::integral_constant<int, 2>{});
  else
    with_nb(std::integral_constant<int, 4>{});
  check_launch("k_update");
}

// --------------------------------------------------------- small gemm --

// The products are small and each entry is one chain of l sums, so latency
// bounds it: eight terms' loads at once, and a wave a workgroup, so that they
// spread over the chip (the products of a solve with bases of up to 90
// columns: 9.0 us each one by one, 3.9 so).
__global__ __launch_bounds__(64) void k_small_gemm(int m, int l, int k, const double *A, int lda,
                                                   const double *B, int ldb, double *C, int ldc,
                                                   int transA) {
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= m * k) return;
  const int i = e / k, j = e % k;
  const double *a = A + (transA ? (size_t)i : (size_t)i * lda), *b = B + j;
  const size_t step = transA ? lda : 1;
  double s = 0.0;
  int t = 0;
  for (; t + 8 <= l; t += 8) {
    double x[8], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      x[u] = a[(t + u) * step];
      y[u] = b[(size_t)(t + u) * ldb];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) s += x[u] * y[u];
  }
  for (; t < l; ++t) s += a[t * step] * b[(size_t)t * ldb];
  C[(size_t)i * ldc + j] = s;
}

void launch_small_gemm(hipStream_t st, int m, int l, int k, const double *A, int lda,
                       const double *B, int ldb, double *C, int ldc, int transA) {
  if (m <= 0 || k <= 0) return;
  const int tot = m * k;
  k_small_gemm<<<(tot + 63) / 64, 64, 0, st>>>(m, l, k, A, lda, B, ldb, C, ldc, transA);
  check_launch("k_small_gemm");
}

// -------------------------------------------------------------- cholesky --
//
// G = L L^T (s <= 64, one workgroup, G staged in LDS).  Writes B = L^T
// (upper triangular, the R factor of U = Q R) and Rinv = L^{-T}, so that
// Q = U Rinv.  flag[0] = 1 + index of the first pivot <= rel_tol * max
// diag(G) (0 if none).

__global__ __launch_bounds__(256) void k_chol(int s, const double *G, double *Rinv, double *B,
                                              int *flag, double rel_tol) {
  __shared__ double a[64 * 64];
  __shared__ double dmax;
  __shared__ int bad;
  const int t = threadIdx.x;
  for (int e = t; e < s * s; e += blockDim.x) a[e] = G[e];
  if (t == 0) {
    double m = 0.0;
    for (int i = 0; i < s; ++i) m = fmax(m, G[i * s + i]);
    dmax = m;
    bad = 0;
  }
  __syncthreads();
  for (int k = 0; k < s; ++k) {
    if (t == 0) {
      double d = a[k * s + k];
      if (!(d > rel_tol * dmax) && bad == 0) bad = k + 1;
      a[k * s + k] = (d > 0.0 && bad == 0) ? sqrt(d) : 1.0;
    }
    __syncthreads();
    const double lkk = a[k * s + k];
    for (int i = k + 1 + t; i < s; i += blockDim.x) a[i * s + k] /= lkk;
    __syncthreads();
    for (int e = t; e < (s - k - 1) * (s - k - 1); e += blockDim.x) {
      int i = k + 1 + e / (s - k - 1), j = k + 1 + e % (s - k - 1);
      if (j <= i) a[i * s + j] -= a[i * s + k] * a[j * s + k];
    }
    __syncthreads();
  }
  // column j of L^{-1} by forward substitution, one column per thread,
  // stored transposed: Rinv[j][i] = (L^{-1})[i][j]  (upper triangular)
  for (int j = t; j < s; j += blockDim.x) {
    double *row = Rinv + (size_t)j * s;
    for (int i = 0; i < j; ++i) row[i] = 0.0;
    row[j] = 1.0 / a[j * s + j];
    for (int i = j + 1; i < s; ++i) {
      double sum = 0.0;
      for (int k = j; k < i; ++k) sum += a[i * s + k] * row[k];
      row[i] = -sum / a[i * s + i];
    }
  }
  for (int e = t; e < s * s; e += blockDim.x) {
    int i = e / s, j = e % s;
    B[e] = (j >= i) ? a[j * s + i] : 0.0;  // L^T
  }
  if (t == 0) flag[0] = bad;
}

void launch_chol(hipStream_t st, int s, const double *G, double *Rinv, double *B, int *flag,
                 double rel_tol) {
  if (s > 64) throw Error(POLFED_EINVAL, "cholesky: s must be <= 64");
  k_chol<<<1, 256, 0, st>>>(s, G, Rinv, B, flag, rel_tol);
  check_launch("k_chol");
}

// out = in^T (s x s, row-major);  sym: in = (in + in^T)/2 in place
__global__ void k_small_transpose(int m, int k, const double *in, int ldi, double *out, int ldo) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= m * k) return;
  int i = e / k, j = e % k;
  out[(size_t)j * ldo + i] = in[(size_t)i * ldi + j];
}

__global__ void k_symmetrize(int s, double *A, int lda) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= s * s) return;
  int i = e / s, j = e % s;
  if (j <= i) return;
  double v = 0.5 * (A[(size_t)i * lda + j] + A[(size_t)j * lda + i]);
  A[(size_t)i * lda + j] = v;
  A[(size_t)j * lda + i] = v;
}

void launch_small_transpose(hipStream_t st, int m, int k, const double *in, int ldi, double *out,
                            int ldo) {
  if (m <= 0 || k <= 0) return;
  k_small_transpose<<<(m * k + 255) / 256, 256, 0, st>>>(m, k, in, ldi, out, ldo);
  check_launch("k_small_transpose");
}

void launch_symmetrize(hipStream_t st, int s, double *A, int lda) {
  if (s <= 0) return;
  k_symmetrize<<<(s * s + 255) / 256, 256, 0, st>>>(s, A, lda);
  check_launch("k_symmetrize");
}

// ---------------------------------------------------------------- jacobi --
//
// Cyclic Jacobi with the round-robin ordering of jacobi_lds.h.  A round
// computes the n/2 rotations from the current A, then applies J^T A J
// block-wise (each 2 x 2 block of rows {p1,q1} x cols {p2,q2} is owned by one
// thread) and V <- V J.  The rotation J = [[c, s], [-s, c]] on (p, q)
// annihilates a_pq with t = sign(th)/(|th| + sqrt(th^2+1)), th = (a_qq -
// a_pp)/(2 a_pq).

// One round over the whole matrix: Aout = J^T Ain J (2 x 2 blocks, one per
// thread, 16 x 16 pair-blocks per workgroup) and V <- V J in place (16 rows
// x 16 pairs per workgroup).  Workgroups [0, nta) do A tiles, the rest V.
constexpr int kJT = 16;

__global__ __launch_bounds__(256) void k_jacobi_round(int n, int r, const double *Ain,
                                                      double *Aout, double *V, int tiles_a) {
  __shared__ int sp[2][kJT], sq[2][kJT];
  __shared__ double sc[2][kJT], ss[2][kJT];
  const int m = n + (n & 1);
  const int npair = m / 2;
  const int tp = (npair + kJT - 1) / kJT;
  const int t = threadIdx.x;
  const int ty = t / kJT, tx = t % kJT;
  int blk = blockIdx.x;
  if (blk < tiles_a) {
    const int tk1 = blk / tp, tk2 = blk % tp;
    if (t < 2 * kJT) {
      const int which = t / kJT, i = t % kJT;
      const int k = (which == 0 ? tk1 : tk2) * kJT + i;
      int p = 0, q = n;
      double c = 1.0, s = 0.0;
      if (k < npair) jacobi_rotation(Ain, n, m, r, k, p, q, c, s);
      sp[which][i] = p; sq[which][i] = q; sc[which][i] = c; ss[which][i] = s;
    }
    __syncthreads();
    const int k1 = tk1 * kJT + ty, k2 = tk2 * kJT + tx;
    if (k1 >= npair || k2 >= npair) return;
    const int p1 = sp[0][ty], q1 = sq[0][ty], p2 = sp[1][tx], q2 = sq[1][tx];
    const double c1 = sc[0][ty], s1 = ss[0][ty], c2 = sc[1][tx], s2 = ss[1][tx];
    const bool q1ok = q1 < n, q2ok = q2 < n;
    const double a00 = Ain[(size_t)p1 * n + p2];
    const double a01 = q2ok ? Ain[(size_t)p1 * n + q2] : 0.0;
    const double a10 = q1ok ? Ain[(size_t)q1 * n + p2] : 0.0;
    const double a11 = (q1ok && q2ok) ? Ain[(size_t)q1 * n + q2] : 0.0;
    // rows: R1^T = [[c1, -s1], [s1, c1]]; cols: R2 = [[c2, s2], [-s2, c2]]
    const double b00 = c1 * a00 - s1 * a10, b01 = c1 * a01 - s1 * a11;
    const double b10 = s1 * a00 + c1 * a10, b11 = s1 * a01 + c1 * a11;
    Aout[(size_t)p1 * n + p2] = b00 * c2 - b01 * s2;
    if (q2ok) Aout[(size_t)p1 * n + q2] = b00 * s2 + b01 * c2;
    if (q1ok) Aout[(size_t)q1 * n + p2] = b10 * c2 - b11 * s2;
    if (q1ok && q2ok) Aout[(size_t)q1 * n + q2] = b10 * s2 + b11 * c2;
  } else {
    blk -= tiles_a;
    const int ti = blk / tp, tk = blk % tp;
    if (t < kJT) {
      const int k = tk * kJT + t;
      int p = 0, q = n;
      double c = 1.0, s = 0.0;
      if (k < npair) jacobi_rotation(Ain, n, m, r, k, p, q, c, s);
      sp[0][t] = p; sq[0][t] = q; sc[0][t] = c; ss[0][t] = s;
    }
    __syncthreads();
    const int i = ti * kJT + ty, k = tk * kJT + tx;
    if (i >= n || k >= npair) return;
    const int p = sp[0][tx], q = sq[0][tx];
    if (q >= n) return;
    const double c = sc[0][tx], s = ss[0][tx];
    const double vp = V[(size_t)i * n + p], vq = V[(size_t)i * n + q];
    V[(size_t)i * n + p] = c * vp - s * vq;
    V[(size_t)i * n + q] = s * vp + c * vq;
  }
}

// Batched cyclic Jacobi for many small symmetric matrices of one size, so that
// many Lanczos convergence checks of one batch run in a single launch.  The
// rotations, the 2 x 2 block updates and the stopping rule are those of
// sym_eig, applied to each matrix on its own: one workgroup per matrix turns
// the matrix in LDS and leaves a log of its rotations, and a second launch
// turns the rows of V, which need nothing of each other, over the whole chip
// (16 us for n = 40, 31 for n = 80).  One matrix from scratch (us): n = 33 162,
// n = 64 429, n = 96 1016, n = 128 2098; with V turned in LDS (n <= 96) or
// global memory in each round, by the one workgroup, 190, 612, 1602 and 6237.
// Latency bounds it: about 0.8 us a round of two barriers, LDS loads, two
// reciprocal square roots one after the other and LDS stores.
struct EigLog {
  int rounds;
  int rank[kLdsEigMax];  // of each index's eigenvalue
};

template <int NM>
__global__ __launch_bounds__(kEigThreads) void k_jacobi_lds(int n, const double *A, double *w,
                                                            EigLog *info, double2 *log,
                                                            size_t log_per) {
  extern __shared__ double sA[];  // m * ld, kEigRed for sums
  __shared__ JacobiRot rot;
  const int m = eig_even(n), ld = eig_ld(n);
  double *red = sA + (size_t)m * ld;
  const int t = threadIdx.x, nt = blockDim.x;
  const double *Ab = A + (size_t)blockIdx.x * n * n;
  for (int e = t; e < m * m; e += nt) {
    const int i = e / m, j = e % m;
    const bool in = i < n && j < n;
    sA[i * ld + j] = in ? Ab[(size_t)i * n + j] : 0.0;
  }
  __syncthreads();
  const int rounds =
      jacobi_sweeps<NM, true>(n, sA, red, rot, kEigSweeps, log + blockIdx.x * log_per);
  __syncthreads();
  // eigenvalues ascending (ties by index)
  double *wb = w + (size_t)blockIdx.x * n;
  EigLog &out = info[blockIdx.x];
  if (t == 0) out.rounds = rounds;
  for (int i = t; i < n; i += nt) {
    const double di = sA[i * ld + i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double dj = sA[j * ld + j];
      rank += (dj < di || (dj == di && j < i)) ? 1 : 0;
    }
    wb[rank] = di;
    out.rank[i] = rank;
  }
}

// A lane's neighbour's value: lane + 1's or lane - 1's.
template <int CTRL>
__device__ __forceinline__ double wave_shift(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Vout = V times the logged rotations, columns by rank; V null: the identity.
// One wave holds kRows rows in its lanes, a lane the columns at positions k and
// m - 1 - k of its row (indices k and m - 1 - k in round 0 and again after
// every sweep); from one round to the next a column moves on by one position,
// which is a shift of the lanes.  kAhead rounds of (c, s) are on their way.
template <int NM>
__global__ __launch_bounds__(64) void k_jacobi_rows(int n, const double *V, const EigLog *info,
                                                    const double2 *log, size_t log_per,
                                                    double *Vout) {
  constexpr int kLanes = NM / 2, kRows = 64 / kLanes, kAhead = 16;
  const int m = eig_even(n), npair = m / 2;
  const int k = threadIdx.x & (kLanes - 1);
  const int row = blockIdx.x * kRows + (int)threadIdx.x / kLanes;
  const EigLog &in = info[blockIdx.y];
  const size_t nn = (size_t)n * n;
  const double *Vb = V ? V + blockIdx.y * nn : nullptr;
  const bool holds = k < npair && row < n;
  const int cb = m - 1 - k;
  double top = 0.0, bot = 0.0;
  if (holds) {
    top = Vb ? Vb[(size_t)row * n + k] : (row == k) ? 1.0 : 0.0;
    if (cb < n) bot = Vb ? Vb[(size_t)row * n + cb] : (row == cb) ? 1.0 : 0.0;
  }
  // (a lane without a pair reads the last pair's; nothing takes its values)
  const double2 *lg = log + blockIdx.y * log_per + (k < npair ? k : npair - 1);
  const int rounds = in.rounds;
  const bool first = k == 0, last = k == npair - 1;
  auto turn = [&](double2 x) {
    const double p = x.x * top - x.y * bot, q = x.y * top + x.x * bot;
    const double pn = wave_shift<0x130>(p), qp = wave_shift<0x138>(q);
    top = first ? p : last ? q : pn;
    bot = !first ? qp : (npair > 1) ? pn : q;
  };
  double2 cs[kAhead];
  if (rounds >= kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) cs[u] = lg[(size_t)u * npair];
  }
  int r = 0;
  for (; r + kAhead <= rounds; r += kAhead) {
    // (past the end: the last round's, not used)
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const double2 x = cs[u];
      cs[u] = lg[(size_t)std::min(r + u + kAhead, rounds - 1) * npair];
      turn(x);
    }
  }
  for (; r < rounds; ++r) turn(lg[(size_t)r * npair]);
  if (!holds) return;
  double *Vo = Vout + blockIdx.y * nn + (size_t)row * n;
  Vo[in.rank[k]] = top;
  if (cb < n) Vo[in.rank[cb]] = bot;
}

bool sym_eig_batched(hipStream_t st, int n, int B, const double *A, const double *V, double *w,
                     double *Vout, DevBuf &log) {
  if (n < 1 || n > kLdsEigMax || B < 1) return false;
  const int m = eig_even(n);
  const size_t shm = sizeof(double) * ((size_t)m * eig_ld(n) + kEigRed);
  auto turn = n <= 64 ? k_jacobi_lds<64> : k_jacobi_lds<128>;
  auto rows = n <= 64 ? k_jacobi_rows<64> : k_jacobi_rows<128>;
  const int per_wave = n <= 64 ? 2 : 1;
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(turn),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  // the log of all sweeps there may be, 5.2 MB a matrix for n > 64 and 1.3 up
  // to there (one size each, so that growing matrices do not allocate anew),
  // at most 166 MB at a time
  const int mm = n <= 64 ? 64 : kLdsEigMax;
  const size_t log_per = (size_t)(mm / 2) * (mm - 1) * kEigSweeps;
  const int chunk = std::min(B, 32);
  const size_t nn = (size_t)n * n;
  EigLog *info = static_cast<EigLog *>(
      log.ensure(chunk * (sizeof(EigLog) + 16 + sizeof(double2) * log_per)));
  double2 *lg = reinterpret_cast<double2 *>(
      reinterpret_cast<char *>(info) + ((chunk * sizeof(EigLog) + 15) & ~(size_t)15));
  for (int b = 0; b < B; b += chunk) {
    const int nb = std::min(chunk, B - b);
    turn<<<nb, kEigThreads, shm, st>>>(n, A + b * nn, w + (size_t)b * n, info, lg, log_per);
    check_launch("k_jacobi_lds");
    rows<<<dim3((n + per_wave - 1) / per_wave, nb), 64, 0, st>>>(
        n, V ? V + b * nn : nullptr, info, lg, log_per, Vout + b * nn);
    check_launch("k_jacobi_rows");
  }
  return true;
}

// off-diagonal and diagonal sums of squares -> out[0], out[1] (one block)
__global__ __launch_bounds__(1024) void k_offnorm(int n, const double *A, double *out) {
  __shared__ double red[2][1024];
  const int t = threadIdx.x;
  double off = 0.0, dg = 0.0;
  for (long long e = t; e < (long long)n * n; e += blockDim.x) {
    const int i = (int)(e / n), j = (int)(e % n);
    const double v = A[e];
    if (i == j) dg += v * v; else off += v * v;
  }
  red[0][t] = off;
  red[1][t] = dg;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (t < w) {
      red[0][t] += red[0][t + w];
      red[1][t] += red[1][t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    out[0] = red[0][0];
    out[1] = red[1][0];
  }
}

__global__ void k_eye(int n, double *V) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)n * n) return;
  V[e] = ((e / n) == (e % n)) ? 1.0 : 0.0;
}

// Sort eigenvalues ascending (ties by index) and permute V's columns.
__global__ void k_eig_sort(int n, const double *A, const double *Vin, double *w, double *Vout) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const double x = A[(size_t)t * n + t];
  int rk = 0;
  for (int j = 0; j < n; ++j) {
    const double y = A[(size_t)j * n + j];
    if (y < x || (y == x && j < t)) ++rk;
  }
  w[rk] = x;
  for (int i = 0; i < n; ++i) Vout[(size_t)i * n + rk] = Vin[(size_t)i * n + t];
}

// W = blockdiag(V0, I): V0 is n0 x n0 (ld n0), W is n x n.
__global__ void k_embed_block(int n, int n0, const double *V0, double *W) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)n * n) return;
  const int i = (int)(e / n), j = (int)(e % n);
  W[e] = (i < n0 && j < n0) ? V0[(size_t)i * n0 + j] : (i == j ? 1.0 : 0.0);
}

void launch_embed_block(hipStream_t st, int n, int n0, const double *V0, double *W) {
  const long long nn = (long long)n * n;
  if (nn <= 0) return;
  k_embed_block<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(n, n0, V0, W);
  check_launch("k_embed_block");
}

void sym_eig(hipStream_t st, int n, double *A, double *w, double *V, DevBuf &work,
             const double *V0) {
  if (n <= 0) return;
  if (n > 4096) throw Error(POLFED_EINVAL, "sym_eig: n must be <= 4096");
  const size_t nn = (size_t)n * n;
  // up to 128 x 128 the matrix fits one workgroup's LDS: the same sweeps
  // and stopping rule in two launches, without a host round trip per sweep
  if (n <= kLdsEigMax && sym_eig_batched(st, n, 1, A, V0, w, V, work)) return;
  double *base = static_cast<double *>(work.ensure(sizeof(double) * (2 * nn + 4)));
  double *Vw = base;
  double *A2 = base + nn;
  double *off = base + 2 * nn;
  double *buf[2] = {A, A2};
  if (V0) {
    // warm start: A is already V0^T A_orig V0, rotations accumulate onto V0
    PF_HIP(hipMemcpyAsync(Vw, V0, sizeof(double) * nn, hipMemcpyDeviceToDevice, st));
  } else {
    k_eye<<<(unsigned)((nn + 255) / 256), 256, 0, st>>>(n, Vw);
    check_launch("k_eye");
  }
  const int m = n + (n & 1);
  const int npair = m / 2;
  const int tp = (npair + kJT - 1) / kJT;
  const int tiles_a = tp * tp;
  const int tiles_v = ((n + kJT - 1) / kJT) * tp;
  int cur = 0;
  double host[2] = {0.0, 0.0};
  double prev = -1.0;
  for (int sweep = 0; sweep < 40 && n > 1; ++sweep) {
    for (int r = 0; r < m - 1; ++r) {
      k_jacobi_round<<<tiles_a + tiles_v, 256, 0, st>>>(n, r, buf[cur], buf[cur ^ 1], Vw, tiles_a);
      cur ^= 1;
    }
    check_launch("k_jacobi_round");
    k_offnorm<<<1, 1024, 0, st>>>(n, buf[cur], off);
    check_launch("k_offnorm");
    PF_HIP(hipMemcpyAsync(host, off, 2 * sizeof(double), hipMemcpyDeviceToHost, st));
    PF_HIP(hipStreamSynchronize(st));
    // stop at a relative off-diagonal Frobenius norm of 1e-14, or when the
    // rounding floor is reached (no further decrease)
    if (!(host[0] > 1e-28 * host[1]) || host[0] == 0.0) break;
    if (prev >= 0.0 && sweep >= 3 && host[0] > 0.5 * prev) break;
    prev = host[0];
  }
  k_eig_sort<<<(n + 255) / 256, 256, 0, st>>>(n, buf[cur], Vw, w, V);
  check_launch("k_eig_sort");
}

// ------------------------------------------------------------- philox --
//
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of
// (c0,c1,c2,c3) -> (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1,
// lo(M0 c0)), with the key bumped by the Weyl constants between rounds.

struct U4 {
  uint32_t x, y, z, w;
};

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    const uint32_t hi0 = __umulhi(M0, c.x), lo0 = M0 * c.x;
    const uint32_t hi1 = __umulhi(M1, c.z), lo1 = M1 * c.z;
    c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
    k0 += W0;
    k1 += W1;
  }
  return c;
}

__global__ void k_philox_fill(long long n, int S, double *X, long long ld, uint32_t k0,
                              uint32_t k1, uint32_t sid) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * S) return;
  const long long r = e / S;
  const int c = (int)(e % S);
  U4 o = philox4x32_10(U4{(uint32_t)r, (uint32_t)(r >> 32), (uint32_t)c, sid}, k0, k1);
  const unsigned long long bits = ((unsigned long long)o.x << 21) ^ ((unsigned long long)o.y >> 11);
  const double u = (double)(bits & ((1ull << 53) - 1)) * (1.0 / 9007199254740992.0);
  X[r * ld + c] = 2.0 * u - 1.0;
}

void launch_philox_fill(hipStream_t st, long long n, int S, double *X, long long ld,
                        unsigned long long seed, unsigned stream_id) {
  long long tot = n * S;
  if (tot <= 0) return;
  k_philox_fill<<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(
      n, S, X, ld, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id);
  check_launch("k_philox_fill");
}

// ----------------------------------------------------- column reductions --
//
// Grid: nblk row-chunks x ceil(q/64) column groups; lane = column, the 4
// waves stride over the rows of the chunk; partials[blk][col] then a
// fixed-order sum.

template <int MODE>  // 0: sum x^2; 1: sum (hv - e v)^2
__global__ __launch_bounds__(256) void k_colsq(long long n, int q, const double *X,
                                               long long ldx, const double *V, long long ldv,
                                               const double *E, double *part,
                                               long long rows_per_blk) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cg = blockIdx.y;
  const int col = cg * 64 + lane;
  const long long r0 = (long long)blockIdx.x * rows_per_blk;
  long long r1 = r0 + rows_per_blk;
  if (r1 > n) r1 = n;
  double s = 0.0;
  if (col < q) {
    const double e = (MODE == 1) ? E[col] : 0.0;
    for (long long r = r0 + wave; r < r1; r += 4) {
      double x = X[r * ldx + col];
      if (MODE == 1) x -= e * V[r * ldv + col];
      s += x * x;
    }
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && col < q)
    part[(size_t)blockIdx.x * q + col] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// One wave a column: a single thread's chain of loads took 17 us over 512
// blocks; so under 8.
__global__ __launch_bounds__(64) void k_colsum_final(int q, int nblk, const double *part,
                                                     double *out, int do_sqrt) {
  const int j = blockIdx.x, lane = threadIdx.x;
  double s = 0.0;
  for (int b = lane; b < nblk; b += 64) s += part[(size_t)b * q + j];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) out[j] = do_sqrt ? sqrt(s) : s;
}

static void colsq(hipStream_t st, int mode, long long n, int q, const double *X, long long ldx,
                  const double *V, long long ldv, const double *E, double *out,
                  DevBuf &partials, int num_cu) {
  if (q <= 0) return;
  long long want = std::max<long long>(1, 2LL * num_cu / ((q + 63) / 64));
  long long rows = std::max<long long>(64, (n + want - 1) / want);
  long long nblk = std::max<long long>(1, (n + rows - 1) / rows);
  double *part = static_cast<double *>(partials.ensure(sizeof(double) * nblk * q));
  dim3 grid((unsigned)nblk, (unsigned)((q + 63) / 64));
  if (mode == 0)
    k_colsq<0><<<grid, 256, 0, st>>>(n, q, X, ldx, V, ldv, E, part, rows);
  else
    k_colsq<1><<<grid, 256, 0, st>>>(n, q, X, ldx, V, ldv, E, part, rows);
  check_launch("k_colsq");
  k_colsum_final<<<q, 64, 0, st>>>(q, (int)nblk, part, out, 1);
  check_launch("k_colsum_final");
}

void launch_colnorms(hipStream_t st, long long n, int q, const double *X, long long ldx,
                     double *out, DevBuf &partials, int num_cu) {
  colsq(st, 0, n, q, X, ldx, nullptr, 0, nullptr, out, partials, num_cu);
}

void launch_resid_norms(hipStream_t st, long long n, int q, const double *HV, long long ldhv,
                        const double *V, long long ldv, const double *E, double *out,
                        DevBuf &partials, int num_cu) {
  colsq(st, 1, n, q, HV, ldhv, V, ldv, E, out, partials, num_cu);
}

// argmax |x| per column, lowest row on ties -> f[j] = sign of that entry
__global__ __launch_bounds__(256) void k_colargmax(long long n, int q, const double *X,
                                                   long long ldx, double *pv, long long *pi,
                                                   long long rows_per_blk) {
  __shared__ double bv[4][64];
  __shared__ long long bi[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = blockIdx.y * 64 + lane;
  const long long r0 = (long long)blockIdx.x * rows_per_blk;
  long long r1 = r0 + rows_per_blk;
  if (r1 > n) r1 = n;
  double best = -1.0;
  long long bidx = -1;
  if (col < q) {
    for (long long r = r0 + wave; r < r1; r += 4) {
      const double a = fabs(X[r * ldx + col]);
      if (a > best) { best = a; bidx = r; }  // rows visited ascending: keeps lowest on ties
    }
  }
  bv[wave][lane] = best;
  bi[wave][lane] = bidx;
  __syncthreads();
  if (wave == 0 && col < q) {
    for (int w = 1; w < 4; ++w) {
      const double v = bv[w][lane];
      const long long i = bi[w][lane];
      if (v > best || (v == best && i >= 0 && (bidx < 0 || i < bidx))) { best = v; bidx = i; }
    }
    pv[(size_t)blockIdx.x * q + col] = best;
    pi[(size_t)blockIdx.x * q + col] = bidx;
  }
}

// One wave a column (a single thread took 73 us over 512 blocks).
__global__ __launch_bounds__(64) void k_sign_final(int q, int nblk, const double *pv,
                                                   const long long *pi, const double *X,
                                                   long long ldx, double *f) {
  const int j = blockIdx.x, lane = threadIdx.x;
  double best = -1.0;
  long long bidx = -1;
  auto take = [&](double v, long long i) {
    if (v > best || (v == best && i >= 0 && (bidx < 0 || i < bidx))) {
      best = v;
      bidx = i;
    }
  };
  for (int b = lane; b < nblk; b += 64) take(pv[(size_t)b * q + j], pi[(size_t)b * q + j]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double v = __shfl_xor(best, o);
    const long long i = __shfl_xor(bidx, o);
    take(v, i);
  }
  if (lane == 0) f[j] = (bidx >= 0 && X[bidx * ldx + j] < 0.0) ? -1.0 : 1.0;
}

void launch_sign_factors(hipStream_t st, long long n, int q, const double *X, long long ldx,
                         double *f, DevBuf &partials, int num_cu) {
  if (q <= 0) return;
  long long want = std::max<long long>(1, 2LL * num_cu / ((q + 63) / 64));
  long long rows = std::max<long long>(64, (n + want - 1) / want);
  long long nblk = std::max<long long>(1, (n + rows - 1) / rows);
  char *base = static_cast<char *>(partials.ensure((sizeof(double) + sizeof(long long)) * nblk * q));
  double *pv = reinterpret_cast<double *>(base);
  long long *pi = reinterpret_cast<long long *>(base + sizeof(double) * nblk * q);
  dim3 grid((unsigned)nblk, (unsigned)((q + 63) / 64));
  k_colargmax<<<grid, 256, 0, st>>>(n, q, X, ldx, pv, pi, rows);
  check_launch("k_colargmax");
  k_sign_final<<<q, 64, 0, st>>>(q, (int)nblk, pv, pi, X, ldx, f);
  check_launch("k_sign_final");
}

__global__ void k_scale_cols(long long n, int q, double *X, long long ldx, const double *f) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * q) return;
  long long r = e / q;
  int j = (int)(e % q);
  X[r * ldx + j] *= f[j];
}

void launch_scale_cols(hipStream_t st, long long n, int q, double *X, long long ldx,
                       const double *f) {
  long long tot = n * q;
  if (tot <= 0) return;
  k_scale_cols<<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(n, q, X, ldx, f);
  check_launch("k_scale_cols");
}

// out[j * n + r] = X[r * ldx + j] through a 32 x 32 LDS tile
__global__ void k_to_colmajor(long long n, int q, const double *X, long long ldx, double *out) {
  __shared__ double tile[32][33];
  const long long r0 = (long long)blockIdx.x * 32;
  const int c0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int k = ty; k < 32; k += 8) {
    const long long r = r0 + k;
    const int c = c0 + tx;
    tile[k][tx] = (r < n && c < q) ? X[r * ldx + c] : 0.0;
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int c = c0 + k;
    const long long r = r0 + tx;
    if (r < n && c < q) out[(size_t)c * n + r] = tile[tx][k];
  }
}

void launch_to_colmajor(hipStream_t st, long long n, int q, const double *X, long long ldx,
                        double *out) {
  if (n <= 0 || q <= 0) return;
  dim3 grid((unsigned)((n + 31) / 32), (unsigned)((q + 31) / 32));
  k_to_colmajor<<<grid, 256, 0, st>>>(n, q, X, ldx, out);
  check_launch("k_to_colmajor");
}

__global__ void k_gather_cols(long long n, int q, const double *X, long long ldx, const int *idx,
                              double *out, long long ldo) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * q) return;
  long long r = e / q;
  int j = (int)(e % q);
  out[r * ldo + j] = X[r * ldx + idx[j]];
}

void launch_gather_cols(hipStream_t st, long long n, int q, const double *X, long long ldx,
                        const int *idx, double *out, long long ldo) {
  long long tot = n * q;
  if (tot <= 0) return;
  k_gather_cols<<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(n, q, X, ldx, idx, out, ldo);
  check_launch("k_gather_cols");
}

__global__ void k_fill(double *x, long long count, double v) {
  long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) x[e] = v;
}

void launch_fill(hipStream_t st, double *x, long long count, double v) {
  if (count <= 0) return;
  k_fill<<<(unsigned)((count + 255) / 256), 256, 0, st>>>(x, count, v);
  check_launch("k_fill");
}

// ----------------------------------------------- single-vector Lanczos --
//
// One step of the bounds Lanczos (w = H v_k already computed):
//   alpha_k = v_k . w;  w <- w - alpha_k v_k - beta_k v_{k-1};
//   beta_{k+1} = ||w||;  v_{k+1} = w / beta_{k+1}.
// Scalars stay on the device; every block of a kernel re-reduces the same
// partial array in the same order, so all blocks agree bitwise.

constexpr int kRedThreads = 256;

__device__ double block_sum(double v, double *sh) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  for (int w = 0; w < (int)blockDim.x / 64; ++w) r += sh[w];
  __syncthreads();
  return r;
}

__device__ double sum_partials(const double *part, int nblk, double *sh, int stride = 1) {
  double s = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) s += part[(size_t)b * stride];
  return block_sum(s, sh);
}

__global__ __launch_bounds__(kRedThreads) void k_dot_partials(long long n, const double *x,
                                                              const double *y, double *part) {
  __shared__ double sh[kRedThreads / 64];
  double s = 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    s += x[i] * y[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ __launch_bounds__(kRedThreads) void k_lanczos_update(long long n, double *w,
                                                                const double *v,
                                                                const double *vprev,
                                                                const double *part, int npart, int stride,
                                                                double *alpha,
                                                                const double *beta_prev,
                                                                double *part2) {
  __shared__ double sh[kRedThreads / 64];
  const double a = sum_partials(part, npart, sh, stride);
  const double b = (vprev != nullptr) ? beta_prev[0] : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha[0] = a;
  double s = 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    double x = w[i] - a * v[i];
    if (vprev != nullptr) x -= b * vprev[i];
    w[i] = x;
    s += x * x;
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part2[blockIdx.x] = s;
}

__global__ __launch_bounds__(kRedThreads) void k_lanczos_normalize(long long n, const double *w,
                                                                   double *vnext,
                                                                   const double *part2, int nblk,
                                                                   double *beta) {
  __shared__ double sh[kRedThreads / 64];
  const double b = sqrt(sum_partials(part2, nblk, sh));
  if (blockIdx.x == 0 && threadIdx.x == 0) beta[0] = b;
  const double inv = (b > 1e-300) ? 1.0 / b : 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    vnext[i] = w[i] * inv;
}

// part[b] = sum of the b-th of gridDim.x parts of x[0], x[2], ..., x[2 count - 2].
__global__ __launch_bounds__(kRedThreads) void k_sum_chunks(int count, const double *x,
                                                            double *part) {
  __shared__ double sh[kRedThreads / 64];
  const int per = (count + gridDim.x - 1) / gridDim.x;
  const int i0 = blockIdx.x * per, i1 = min(count, i0 + per);
  double s = 0.0;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) s += x[(size_t)2 * i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

void launch_sum_chunks(hipStream_t st, int count, const double *x, double *part, int nblk) {
  k_sum_chunks<<<nblk, kRedThreads, 0, st>>>(count, x, part);
  check_launch("k_sum_chunks");
}

void launch_dot_partials(hipStream_t st, long long n, const double *x, const double *y,
                         double *part, int nblk) {
  k_dot_partials<<<nblk, kRedThreads, 0, st>>>(n, x, y, part);
  check_launch("k_dot_partials");
}

void launch_lanczos_update(hipStream_t st, long long n, double *w, const double *v,
                           const double *vprev, const double *part, int npart, int stride,
                           int nblk, double *alpha, const double *beta_prev, double *part2) {
  k_lanczos_update<<<nblk, kRedThreads, 0, st>>>(n, w, v, vprev, part, npart, stride, alpha,
                                                 beta_prev, part2);
  check_launch("k_lanczos_update");
}

void launch_lanczos_normalize(hipStream_t st, long long n, const double *w, double *vnext,
                              const double *part2, int nblk, double *beta) {
  k_lanczos_normalize<<<nblk, kRedThreads, 0, st>>>(n, w, vnext, part2, nblk, beta);
  check_launch("k_lanczos_normalize");
}

}  // namespace polfed
