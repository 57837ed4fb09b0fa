// The whole Clenshaw filter of a short chain in one launch.
//
// The columns of a block never meet in Y = P^K_sigma(H~) X, and a column of a
// short chain fits one compute unit's LDS, so one workgroup takes one column
// through all K + 1 steps with a workgroup barrier between them, instead of
// K + 1 launches whose kernels are shorter than the launches.  A step took, as
// launches of the step kernel in a graph and here (us, one MI355X):
//   L = 12, s = 4 FP64:  4.9 and 0.42 (J2 != 0: 5.8 and 0.74)
//   L = 14, s = 8 FP64:  5.0 and 1.27 (J2 != 0: 6.1 and 2.6); s = 64: 6.3 and 1.25
//   L = 16, s = 64 FP32: 8.2 and 7.5, the same for every column a CU holds
// What bounds it is the LDS gather: a row reads about L/2 + 1 neighbours at
// scattered addresses, 5 cycles a read of 64 lanes (half of it bank conflicts;
// LDS busy 82 % of the launch at L = 14, 70 % at L = 16).
//
// Rows are held in an order of their own: sorted by the number of J1 bonds
// that act on them (then J2 bonds, then row), so that the 64 rows of a
// wavefront's tile have (nearly) the same number of neighbours and no lane
// waits for another.  Neighbours come from a table of LDS byte offsets, two
// 16-bit offsets to a word, word p of a tile's lanes contiguous; a row with
// fewer neighbours than its tile points at a slot that holds zero.  J1 bonds
// come first, by ascending bit, then J2 bonds, as in the step kernel, and
// each row's operations are the step kernel's in the same order.
//
// Two forms:
// * k_resident_rows (up to 4096 rows, i.e. L <= 14): a thread owns R rows (1,
//   2 or 4) for the whole recurrence; their neighbour words, diagonal, X and
//   b_{k+2} live in its registers, b_{k+1} and the new b_k in two LDS
//   arrays that swap roles, so a step is one round of gathers and one barrier.
// * k_resident_tiles (FP32 up to 16379 rows, i.e. L = 16): the rows' registers
//   would not fit, so waves walk the tiles; b_k overwrites b_{k+2} in LDS (a
//   row's own value only), and the words, the diagonal and X stream from L2,
//   the next tile's words fetched ahead of this one's gathers.
#include <algorithm>
#include <vector>

#include "internal.h"

namespace polfed {

// -------------------------------------------------------------- table --

void build_res_table(int L, bool has_j2, int elem, ResTable &t) {
  const long long n = polfed_dim(L);
  std::vector<uint32_t> states;
  states.reserve((size_t)n);
  std::vector<int32_t> rank((size_t)1 << L, -1);
  for (uint32_t s = 0; s < (1u << L); ++s)
    if (__builtin_popcount(s) == L / 2) {
      rank[s] = (int32_t)states.size();
      states.push_back(s);
    }
  // rotations mark the antiparallel pairs (i, i + l mod L) at bit i
  const uint32_t full = (1u << L) - 1u;
  auto pairs = [&](uint32_t s, int l) { return s ^ (((s >> l) | (s << (L - l))) & full); };
  std::vector<int> c1((size_t)n), c2((size_t)n, 0);
  for (long long r = 0; r < n; ++r) {
    c1[r] = __builtin_popcount(pairs(states[r], 1));
    if (has_j2) c2[r] = __builtin_popcount(pairs(states[r], 2));
  }
  std::vector<uint16_t> perm((size_t)n), pos((size_t)n);
  for (long long r = 0; r < n; ++r) perm[r] = (uint16_t)r;
  std::stable_sort(perm.begin(), perm.end(), [&](uint16_t x, uint16_t y) {
    return c1[x] != c1[y] ? c1[x] > c1[y] : c2[x] > c2[y];
  });
  for (long long p = 0; p < n; ++p) pos[perm[p]] = (uint16_t)p;
  const int ntile = (int)((n + 63) / 64);
  std::vector<ResTile> tiles(ntile);
  std::vector<uint32_t> words;
  const uint32_t zero = (uint32_t)(n * elem);  // the slot that holds zero
  for (int q = 0; q < ntile; ++q) {
    int m1 = 0, m2 = 0;
    for (int l = 0; l < 64 && q * 64LL + l < n; ++l) {
      m1 = std::max(m1, c1[perm[q * 64 + l]]);
      m2 = std::max(m2, c2[perm[q * 64 + l]]);
    }
    tiles[q].off = (int)words.size();
    tiles[q].np1 = (short)((m1 + 1) / 2);
    tiles[q].np2 = (short)((m2 + 1) / 2);
    const int np = tiles[q].np1 + tiles[q].np2;
    words.resize(words.size() + (size_t)np * 64, zero | (zero << 16));
    uint32_t *w = words.data() + tiles[q].off;
    for (int l = 0; l < 64 && q * 64LL + l < n; ++l) {
      const uint32_t s = states[perm[q * 64 + l]];
      for (int b = 1; b <= (has_j2 ? 2 : 1); ++b) {
        int e = (b == 1) ? 0 : 2 * tiles[q].np1;
        for (uint32_t m = pairs(s, b); m; m &= m - 1) {
          const int i = __builtin_ctz(m);
          const uint32_t f = s ^ ((1u << i) | (1u << ((i + b) % L)));
          const uint32_t at = (uint32_t)pos[rank[f]] * (uint32_t)elem;
          uint32_t &d = w[(size_t)(e / 2) * 64 + l];
          d = (e & 1) ? ((d & 0xffffu) | (at << 16)) : ((d & 0xffff0000u) | at);
          ++e;
        }
      }
    }
  }
  t.n = (int)n;
  t.ntile = ntile;
  t.perm.ensure(sizeof(uint16_t) * perm.size());
  t.tiles.ensure(sizeof(ResTile) * tiles.size());
  t.words.ensure(sizeof(uint32_t) * words.size());
  PF_HIP(hipMemcpy(t.perm.p, perm.data(), sizeof(uint16_t) * perm.size(), hipMemcpyHostToDevice));
  PF_HIP(hipMemcpy(t.tiles.p, tiles.data(), sizeof(ResTile) * tiles.size(), hipMemcpyHostToDevice));
  PF_HIP(hipMemcpy(t.words.p, words.data(), sizeof(uint32_t) * words.size(), hipMemcpyHostToDevice));
}

// ------------------------------------------------------------- kernels --

// Distance of the two LDS arrays: room for the rows of the form (R rows a
// thread, 0 the tile form) and the zero slot, a constant so that it is an
// offset in the load instructions.
template <class T>
__host__ __device__ constexpr int res_stride(int R) {
  return R == 0 ? 65520 : (R * 1024 * (int)sizeof(T) + 16);
}

// The step's constants: b_k = alpha X + dscale dt b_{k+1} + w sum - b_{k+2},
// and the last step's with everything over D (its term in X always there).
template <class T>
struct ResStep {
  T alpha, dscale, w1, w2, gamma;
  bool has_x;
};

template <class T>
__device__ __forceinline__ ResStep<T> res_step(const ResItem<T> &it, double c) {
  return ResStep<T>{(T)c, T(2), it.w1, it.w2, T(-1), c != 0.0};
}
template <class T>
__device__ __forceinline__ ResStep<T> res_last(const ResItem<T> &it, double c) {
  return ResStep<T>{(T)(c * it.Dinv), (T)it.Dinv, it.w1f, it.w2f, (T)(-it.Dinv), true};
}

// Keeps a value's computation inside the loop it stands in: the unpacked
// offsets of all rows, moved out of the recurrence, would not fit the
// registers.
__device__ __forceinline__ uint32_t stay(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Adds w times the neighbours of words [C, NP) to acc, in order, CH words in
// flight at once.
template <class T, int CH, bool STAY, int NP, int C, int N>
__device__ __forceinline__ void res_gather_n(const uint32_t (&wd)[N], const char *V, T w, T &acc) {
  constexpr int M = (NP - C < CH) ? NP - C : CH;
  if constexpr (M > 0) {
    T v[2 * M];
#pragma unroll
    for (int p = 0; p < M; ++p) {
      const uint32_t x = STAY ? stay(wd[C + p]) : wd[C + p];
      v[2 * p] = *reinterpret_cast<const T *>(V + (x & 0xffffu));
      v[2 * p + 1] = *reinterpret_cast<const T *>(V + (x >> 16));
    }
#pragma unroll
    for (int p = 0; p < M; ++p) {
      acc += w * v[2 * p];
      acc += w * v[2 * p + 1];
    }
    if (STAY) __builtin_amdgcn_sched_barrier(0);
    res_gather_n<T, CH, STAY, NP, C + M>(wd, V, w, acc);
  }
}

// Words [0, np) of at most N: one straight piece of code for each number, so
// that all of a tile's loads are in flight before the first is used.
template <class T, int CH, bool STAY, int N>
__device__ __forceinline__ void res_gather(const uint32_t (&wd)[N], int np, const char *V, T w,
                                           T &acc) {
  static_assert(N <= 8, "cases below");
#define PF_RES_CASE(NP)                                                                    \
  case NP:                                                                                 \
    if constexpr (NP <= N) res_gather_n<T, CH, STAY, (NP <= N ? NP : 0), 0>(wd, V, w, acc); \
    break;
  switch (np) {
    PF_RES_CASE(1)
    PF_RES_CASE(2)
    PF_RES_CASE(3)
    PF_RES_CASE(4)
    PF_RES_CASE(5)
    PF_RES_CASE(6)
    PF_RES_CASE(7)
    PF_RES_CASE(8)
    default: break;
  }
#undef PF_RES_CASE
}

// The item and column of this workgroup.
template <class T>
__device__ __forceinline__ ResItem<T> res_item(const ResItem<T> &one, const ResItem<T> *items,
                                               int B, int &col) {
  const int b = (int)blockIdx.x;
  if (items == nullptr) {
    col = b;
    return one;
  }
  int lo = 0, hi = B - 1;
  while (lo < hi) {  // the last item with wg0 <= b
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].wg0 <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  col = b - items[lo].wg0;
  return items[lo];
}

// Steps [j0, j1) of the recurrence (0 .. K; step K writes Y); between launches
// the two blocks rest in the workgroup's scratch.
template <class T, int R, int N, bool J2>
__global__ __launch_bounds__(1024) void k_resident_rows(ResItem<T> one, const ResItem<T> *items,
                                                        int B, long long j0, long long j1) {
  extern __shared__ char s_res[];
  int col;
  const ResItem<T> it = res_item(one, items, B, col);
  if (j0 > it.K) return;
  const int n = it.n;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  constexpr int kStride = res_stride<T>(R);
  // words of a chain with many of them: fewer in flight, unpacked on use
  constexpr bool kMany = R * N * (J2 ? 2 : 1) * (int)sizeof(T) > 7 * 8;
  constexpr int CH = !kMany ? N : (R == 4 && J2 && sizeof(T) == 8) ? 2 : 4;
  const T *dtp = it.dt, *X = it.X + col;
  T *Y = it.Y + col;
  T *save = it.scratch + (size_t)col * it.scratch_per;

  uint32_t w1[R][N], w2[R][J2 ? N : 1];
  int np1[R], np2[R], p[R];
  T dt[R], x[R], own[R], old[R];
  const double c0 = it.coef[it.K - j0];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int t = __builtin_amdgcn_readfirstlane(r * nw + wave);
    p[r] = t * 64 + lane;
    const ResTile ti = it.tiles[t < it.ntile ? t : 0];
    np1[r] = __builtin_amdgcn_readfirstlane(t < it.ntile ? (int)ti.np1 : 0);
    np2[r] = __builtin_amdgcn_readfirstlane(t < it.ntile ? (int)ti.np2 : 0);
    const uint32_t *w = it.words + ti.off + lane;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      w1[r][q] = (q < np1[r]) ? w[q * 64] : 0u;
      if (J2) w2[r][q] = (q < np2[r]) ? w[(np1[r] + q) * 64] : 0u;
    }
    dt[r] = x[r] = own[r] = old[r] = T(0);
    if (p[r] < n) {
      const int row = it.perm[p[r]];
      dt[r] = dtp[row];
      x[r] = X[(size_t)row * it.ldx];
      if (j0 == 0) {
        if (it.K == 0) {
          Y[(size_t)row * it.ldy] = (T)(c0 * it.Dinv) * x[r];
        } else if (c0 != 0.0) {
          own[r] = (T)c0 * x[r];  // b_K = c_K X
        }
      } else {
        own[r] = save[p[r]];
        old[r] = save[n + p[r]];
      }
      reinterpret_cast<T *>(s_res)[p[r]] = own[r];
    }
  }
  if (threadIdx.x == 0) {
    reinterpret_cast<T *>(s_res)[n] = T(0);
    reinterpret_cast<T *>(s_res + kStride)[n] = T(0);
  }
  if (it.K == 0) return;
  const long long from = j0 == 0 ? 1 : j0, to = (j1 < it.K + 1) ? j1 : it.K + 1;
  double cn = it.coef[it.K - from];
  __syncthreads();
  // b_k of row r from the array at A
  auto row = [&](int r, const ResStep<T> &st, const char *A) {
    const T dd = st.dscale * dt[r];
    T acc = dd * own[r];
    res_gather<T, CH, kMany>(w1[r], np1[r], A, st.w1, acc);
    if constexpr (J2) res_gather<T, CH, kMany>(w2[r], np2[r], A, st.w2, acc);
    if (st.has_x) acc += st.alpha * x[r];
    acc += st.gamma * old[r];
    return acc;
  };
  auto step = [&](long long j, const char *A, char *Bn) {
    const ResStep<T> st = res_step(it, cn);
    cn = it.coef[it.K - j - 1];  // the next step's, ahead of its use
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T acc = row(r, st, A);
      old[r] = own[r];
      own[r] = acc;
      if (p[r] < n) reinterpret_cast<T *>(Bn)[p[r]] = acc;
    }
    __syncthreads();
  };
  const long long lim = (to <= it.K) ? to : it.K;
  long long j = from;
  for (; j + 1 < lim; j += 2) {
    step(j, s_res, s_res + kStride);
    step(j + 1, s_res + kStride, s_res);
  }
  const char *A = s_res;
  if (j < lim) {
    step(j, s_res, s_res + kStride);
    A = s_res + kStride;
  }
  if (to > it.K) {
    const ResStep<T> st = res_last(it, cn);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (p[r] < n) Y[(size_t)it.perm[p[r]] * it.ldy] = row(r, st, A);
  }
  if (to <= it.K) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (p[r] < n) {
        save[p[r]] = own[r];
        save[n + p[r]] = old[r];
      }
  }
}

// As k_resident_rows, for more rows than registers hold.  Scratch of a
// workgroup: b_{k+1}, b_{k+2} between launches, then the diagonal and X in
// the order of the rows here (written at j0 = 0).
template <class T, int N, bool J2>
__global__ __launch_bounds__(1024) void k_resident_tiles(ResItem<T> one, const ResItem<T> *items,
                                                         int B, long long j0, long long j1) {
  extern __shared__ char s_res[];
  int col;
  const ResItem<T> it = res_item(one, items, B, col);
  if (j0 > it.K) return;
  const int n = it.n, ntile = it.ntile;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  constexpr int kStride = res_stride<T>(0);
  const T *X = it.X + col;
  T *Y = it.Y + col;
  T *save = it.scratch + (size_t)col * it.scratch_per;
  T *dts = save + 2 * (size_t)n, *xs = dts + n;
  const double c0 = it.coef[it.K - j0];
  for (int t = wave; t < ntile; t += nw) {  // (each thread reads back what it wrote)
    const int p = t * 64 + lane;
    if (p >= n) continue;
    T own = T(0), old = T(0);
    if (j0 == 0) {
      const int row = it.perm[p];
      const T x = X[(size_t)row * it.ldx];
      dts[p] = it.dt[row];
      xs[p] = x;
      if (it.K == 0)
        Y[(size_t)row * it.ldy] = (T)(c0 * it.Dinv) * x;
      else if (c0 != 0.0)
        own = (T)c0 * x;
    } else {
      own = save[p];
      old = save[n + p];
    }
    reinterpret_cast<T *>(s_res)[p] = own;
    reinterpret_cast<T *>(s_res + kStride)[p] = old;
  }
  if (threadIdx.x == 0) {
    reinterpret_cast<T *>(s_res)[n] = T(0);
    reinterpret_cast<T *>(s_res + kStride)[n] = T(0);
  }
  if (it.K == 0) return;
  const long long from = j0 == 0 ? 1 : j0, to = (j1 < it.K + 1) ? j1 : it.K + 1;
  double cn = it.coef[it.K - from];
  // this wave's tiles are wave, wave + nw, ...: lane i keeps the offset and
  // counts of the i-th (at most 16)
  const int mine = (ntile - wave + nw - 1) / nw;
  int info_off = 0, info_np = 0;
  if (lane < mine) {
    const ResTile ti = it.tiles[wave + lane * nw];
    info_off = ti.off;
    info_np = (int)ti.np1 | ((int)ti.np2 << 16);
  }
  const uint32_t *words = it.words + lane;
  // what a tile reads from L2, asked for while the tile before it gathers
  struct Ahead {
    uint32_t w1[N], w2[J2 ? N : 1];
    int np1, np2;
    T dt, x;
  };
  auto fetch = [&](int i, bool has_x, Ahead &f) {
    if (i >= mine) return;
    const int np = __builtin_amdgcn_readlane(info_np, i);
    f.np1 = np & 0xffff;
    f.np2 = np >> 16;
    const uint32_t *w = words + __builtin_amdgcn_readlane(info_off, i);
    const int p = (wave + i * nw) * 64 + lane;
    const int q = p < n ? p : 0;
    f.dt = dts[q];
    if (has_x) f.x = xs[q];
#pragma unroll
    for (int e = 0; e < N; ++e)
      if (e < f.np1) f.w1[e] = w[e * 64];
    if constexpr (J2) {
      w += f.np1 * 64;
#pragma unroll
      for (int e = 0; e < N; ++e)
        if (e < f.np2) f.w2[e] = w[e * 64];
    }
  };
  __syncthreads();
  auto step = [&](long long j, const char *A, char *Bn) {
    const ResStep<T> st = (j < it.K) ? res_step(it, cn) : res_last(it, cn);
    if (j < it.K) cn = it.coef[it.K - j - 1];
    auto tile = [&](int i, const Ahead &f) {
      if (i >= mine) return;
      const int p = (wave + i * nw) * 64 + lane;
      const bool in = p < n;
      const int q = in ? p : n;
      const T own = reinterpret_cast<const T *>(A)[q];
      const T old = reinterpret_cast<const T *>(Bn)[q];
      const T dd = st.dscale * f.dt;
      T acc = dd * own;
      res_gather<T, N, false>(f.w1, f.np1, A, st.w1, acc);
      if constexpr (J2) res_gather<T, N, false>(f.w2, f.np2, A, st.w2, acc);
      if (st.has_x) acc += st.alpha * f.x;
      acc += st.gamma * old;
      if (in) {
        if (j < it.K)
          reinterpret_cast<T *>(Bn)[p] = acc;
        else
          Y[(size_t)it.perm[p] * it.ldy] = acc;
      }
    };
    Ahead f0, f1;
    fetch(0, st.has_x, f0);
    for (int i = 0; i < mine; i += 2) {
      fetch(i + 1, st.has_x, f1);
      tile(i, f0);
      fetch(i + 2, st.has_x, f0);
      tile(i + 1, f1);
    }
    __syncthreads();
  };
  for (long long j = from; j < to; j += 2) {
    step(j, s_res, s_res + kStride);
    if (j + 1 < to) step(j + 1, s_res + kStride, s_res);
  }
  const char *A = ((to - from) & 1) ? s_res + kStride : s_res;
  const char *Bn = ((to - from) & 1) ? s_res : s_res + kStride;
  if (to <= it.K) {
    for (int t = wave; t < ntile; t += nw) {
      const int p = t * 64 + lane;
      if (p >= n) continue;
      save[p] = reinterpret_cast<const T *>(A)[p];
      save[n + p] = reinterpret_cast<const T *>(Bn)[p];
    }
  }
}

// Single-vector Lanczos for the spectral bounds: w = H v_k, alpha_k = v_k . w,
// w -= alpha_k v_k + beta_k v_{k-1}, beta_{k+1} = ||w||, v_{k+1} = w /
// beta_{k+1}, v in LDS, the two sums over the workgroup in a fixed order.  A
// step of four launches took 14.6 us at L = 12 and 15.8 at L = 14; so 2.6 and
// 4.1 (the gathers, three barriers, a root and a division in a row).
template <int R, int N, bool J2>
__global__ __launch_bounds__(1024) void k_resident_lanczos(ResItem<double> it, const double *diag,
                                                           const double *start, int steps,
                                                           double w1c, double w2c, double *alpha,
                                                           double *beta) {
  extern __shared__ char s_res[];
  __shared__ double red[2][16];
  const int n = it.n;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  constexpr bool kMany = R * N * (J2 ? 2 : 1) > 7;
  constexpr int CH = kMany ? 2 : N;
  double *v = reinterpret_cast<double *>(s_res);
  int turn = 0;
  // sum over the workgroup; the two buffers take turns, so one barrier does
  auto total = [&](double x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    if (lane == 0) red[turn][wave] = x;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < nw; ++k) s += red[turn][k];
    turn ^= 1;
    return s;
  };
  uint32_t a1[R][N], a2[R][J2 ? N : 1];
  int np1[R], np2[R], p[R];
  double d[R], own[R], old[R];
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int t = r * nw + wave;
    p[r] = t * 64 + lane;
    const ResTile ti = it.tiles[t < it.ntile ? t : 0];
    np1[r] = __builtin_amdgcn_readfirstlane(t < it.ntile ? (int)ti.np1 : 0);
    np2[r] = __builtin_amdgcn_readfirstlane(t < it.ntile ? (int)ti.np2 : 0);
    const uint32_t *w = it.words + ti.off + lane;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      a1[r][q] = (q < np1[r]) ? w[q * 64] : 0u;
      if (J2) a2[r][q] = (q < np2[r]) ? w[(np1[r] + q) * 64] : 0u;
    }
    d[r] = own[r] = old[r] = 0.0;
    if (p[r] < n) {
      const int row = it.perm[p[r]];
      d[r] = diag[row];
      own[r] = start[row];
      s += own[r] * own[r];
    }
  }
  const double norm = sqrt(total(s));
  const double inv0 = (norm > 1e-300) ? 1.0 / norm : 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    own[r] *= inv0;
    if (p[r] < n) v[p[r]] = own[r];
  }
  if (threadIdx.x == 0) {
    v[n] = 0.0;  // the slot that holds zero
    beta[0] = 0.0;
  }
  __syncthreads();
  double b = 0.0;
  for (int k = 0; k < steps; ++k) {
    double w[R], t = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double acc = d[r] * own[r];
      res_gather<double, CH, kMany>(a1[r], np1[r], s_res, w1c, acc);
      if constexpr (J2) res_gather<double, CH, kMany>(a2[r], np2[r], s_res, w2c, acc);
      w[r] = acc;
      t += own[r] * acc;  // (rows past the end hold zero)
    }
    const double a = total(t);
    t = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      w[r] = w[r] - a * own[r] - b * old[r];
      t += w[r] * w[r];
    }
    b = sqrt(total(t));  // (every gather of v is done: two barriers since)
    if (threadIdx.x == 0) {
      alpha[k] = a;
      beta[k + 1] = b;
    }
    const double inv = (b > 1e-300) ? 1.0 / b : 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      old[r] = own[r];
      own[r] = w[r] * inv;
      if (p[r] < n) v[p[r]] = own[r];
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ launcher --

// Rows a thread owns (1, 2 or 4), 0 for the tile form, -1 where the chain
// does not fit: 16 waves of 4 rows a lane are 4096 rows (two FP64 arrays of
// 3432 rows are 55 KB of LDS); the tile form's 16-bit byte offsets end at
// 64 KB, 16379 FP32 rows (two arrays: 128 KB of the 160).
int resident_form(long long n, int elem) {
  const long long ntile = (n + 63) / 64;
  if (ntile <= 16) return 1;
  if (ntile <= 32) return 2;
  if (ntile <= 64) return 4;
  if (elem == 4 && (n + 1) * elem <= 65520) return 0;
  return -1;
}

// Steps of one launch: 16384 steps of the longest chain here (L = 16) are 0.12
// s, with J2 0.22.
constexpr long long kResSteps = 16384;

long long resident_scratch(long long n, int elem) { return 4 * n + 64 / elem; }

template <class T>
void launch_resident(hipStream_t st, const ResItem<T> &one, const ResItem<T> *items, int B,
                     int total_wg, long long Kmax, int L, bool has_j2) {
  if (total_wg <= 0) return;
  const long long n = polfed_dim(L);
  const int form = resident_form(n, (int)sizeof(T));
  const int ntile = (int)((n + 63) / 64);
  const size_t shm = (size_t)res_stride<T>(form) + (((size_t)n + 1) * sizeof(T) + 15 & ~(size_t)15);
  auto run = [&](auto kernel, int waves) {
    if (shm > 65536)
      PF_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    for (long long j = 0; j <= Kmax; j += kResSteps) {
      kernel<<<(unsigned)total_wg, 64 * waves, shm, st>>>(one, items, B, j, j + kResSteps);
      check_launch("k_resident");
    }
  };
  if (form == 1)
    has_j2 ? run(k_resident_rows<T, 1, 7, true>, ntile) : run(k_resident_rows<T, 1, 7, false>, ntile);
  else if (form == 2)
    has_j2 ? run(k_resident_rows<T, 2, 7, true>, (ntile + 1) / 2)
           : run(k_resident_rows<T, 2, 7, false>, (ntile + 1) / 2);
  else if (form == 4)
    has_j2 ? run(k_resident_rows<T, 4, 7, true>, (ntile + 3) / 4)
           : run(k_resident_rows<T, 4, 7, false>, (ntile + 3) / 4);
  else if (form == 0) {
    if constexpr (sizeof(T) == 4)
      has_j2 ? run(k_resident_tiles<T, 8, true>, 16) : run(k_resident_tiles<T, 8, false>, 16);
  } else {
    throw Error(POLFED_EINVAL, "resident filter: chain too long");
  }
}

void launch_resident_lanczos(hipStream_t st, const ResItem<double> &it, const double *diag,
                             const double *start, int steps, double w1, double w2, double *alpha,
                             double *beta, bool has_j2) {
  const int form = resident_form(it.n, (int)sizeof(double));
  const size_t shm = sizeof(double) * ((size_t)it.n + 1);
  auto run = [&](auto kernel, int waves) {
    kernel<<<1, 64 * waves, shm, st>>>(it, diag, start, steps, w1, w2, alpha, beta);
  };
  if (form == 1)
    has_j2 ? run(k_resident_lanczos<1, 7, true>, it.ntile)
           : run(k_resident_lanczos<1, 7, false>, it.ntile);
  else if (form == 2)
    has_j2 ? run(k_resident_lanczos<2, 7, true>, (it.ntile + 1) / 2)
           : run(k_resident_lanczos<2, 7, false>, (it.ntile + 1) / 2);
  else if (form == 4)
    has_j2 ? run(k_resident_lanczos<4, 7, true>, (it.ntile + 3) / 4)
           : run(k_resident_lanczos<4, 7, false>, (it.ntile + 3) / 4);
  else
    throw Error(POLFED_EINVAL, "resident Lanczos: chain too long");
  check_launch("k_resident_lanczos");
}

template void launch_resident<float>(hipStream_t, const ResItem<float> &, const ResItem<float> *,
                                     int, int, long long, int, bool);
template void launch_resident<double>(hipStream_t, const ResItem<double> &,
                                      const ResItem<double> *, int, int, long long, int, bool);

}  // namespace polfed
