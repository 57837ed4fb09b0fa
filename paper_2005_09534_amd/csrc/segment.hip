// The fused Chebyshev step of the longer chains, by segments of the basis.
//
//   out[r,:] = alpha X[r,:] + dscale dt[r] V[r,:] + sum_bonds w_l V[r',:]
//              + gamma W[r,:]
//
// Rows are ascending states, so the rows that share their bits from kSegM = 10
// up (the segment's high part H) are contiguous: C(10, k) rows, k = L/2 -
// popcount(H), in the order of their low parts.  A bond then is one of three:
//
// * both sites low: the neighbour is in the same segment, at a distance that
//   depends on the low part alone.  The segment's own values go to LDS once
//   (they are needed there anyway) and these neighbours are read from it.
// * both sites high: the same bond acts on every row of the segment or on
//   none, and the neighbour of its i-th row is the i-th row of another
//   segment: a contiguous load at an offset that is one number a segment.
// * one site low, one high (the boundary, and the bonds that wrap round):
//   some rows, and the neighbour's place in the other segment follows from
//   the low part alone.
//
// So no rank is computed in the kernel.  A record a segment holds the
// uniform offsets (read with scalar loads) and a 16-byte record a low part
// (32 with J2) the neighbours' places in their segments, as bytes: there are
// at most C(10, 5) = 252.  Bonds add up in the order of the step kernel (J1
// by ascending bit, then J2), so results are equal to its bit for bit.
//
// Blocks are slice-major: 16 bytes of a row to a slice (or the whole row where
// it is shorter), so that a wave's contiguous loads are 1 KB and an XCD's L2
// holds as many rows as it can.  A workgroup does one segment of one slice.
//
// What bounds it: at L >= 22 the traffic past the L2s, which moves at about 6
// TB/s whether the Infinity Cache has it or not (a plain read does 6.4 and 5.3
// TB/s): neighbours across the top bonds are further away than an L2 holds
// rows.  Below that, the latency of one round of loads.  A step, by the step
// kernel's tables and here (us, one MI355X; algorithmic rate here):
//   L = 16, s = 8 FP32:          5.2 and 3.5
//   L = 18, s = 16 FP64, J1-J2: 14.3 and 7.8 (3.2 TB/s)
//   L = 20, s = 4 FP64, J1-J2:  19.4 and 9.9 (2.5 TB/s)
//   L = 22, s = 32 FP32:         128 and 91  (4.0 TB/s)
//   L = 26, s = 64 FP64:        9215 and 7100 (3.0 TB/s)
// Measured slower: rows of 8 bytes (more waves for the same bytes: 1.2-1.6
// times), of 32 and 64 bytes (fewer rows in L2: 1.1-1.4 times), persistent
// workgroups (they drift apart and the rows in flight no longer are
// neighbours: L = 26 9.0 against 8.1 ms), all neighbours of a list in flight
// (registers: 4 waves a SIMD instead of 6, L = 22 99 against 91 us).
#include <algorithm>
#include <type_traits>
#include <vector>

#include "internal.h"

namespace polfed {

// -------------------------------------------------------------- tables --

static long long choose(int n, int k) {
  if (k < 0 || k > n) return 0;
  long long r = 1;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}

static int rank_of(uint32_t s) {  // colex rank among patterns of its weight
  int t = 0;
  long long r = 0;
  for (uint32_t m = s; m; m &= m - 1) r += choose(__builtin_ctz(m), ++t);
  return (int)r;
}

// Rows: 32 bytes a low part, low parts by weight, then ascending.
//   0..8   place of the J1 bond (i, i+1)'s neighbour (255 where it does not act)
//   9, 10  place of the low part with bit 0, bit 1 flipped
//   11     place of the low part with bit kSegM - 2 flipped
//   12, 13 the low part itself
//   16..23 place of the J2 bond (i, i+2)'s neighbour
static void seg_rows(std::vector<unsigned char> &rows) {
  const int M = kSegM;
  rows.assign((size_t)32 << M, 0);
  size_t at = 0;
  for (int k = 0; k <= M; ++k)
    for (uint32_t lo = 0; lo < (1u << M); ++lo) {
      if (__builtin_popcount(lo) != k) continue;
      unsigned char *b = rows.data() + 32 * at++;
      for (int l = 1; l <= 2; ++l)
        for (int i = 0; i + l < M; ++i) {
          const bool acts = ((lo >> i) ^ (lo >> (i + l))) & 1u;
          b[(l == 1 ? 0 : 16) + i] =
              acts ? (unsigned char)rank_of(lo ^ ((1u << i) | (1u << (i + l)))) : 255;
        }
      b[9] = (unsigned char)rank_of(lo ^ 1u);
      b[10] = (unsigned char)rank_of(lo ^ 2u);
      b[11] = (unsigned char)rank_of(lo ^ (1u << (M - 2)));
      b[12] = (unsigned char)(lo & 255u);
      b[13] = (unsigned char)(lo >> 8);
    }
}

// Records: kSegRec ints a segment.
//   0 its first row; 1 rows | first row record << 8; 2 J1 bonds within H |
//   J2 bonds << 8 | bits 0, 1, top, top - 1 of H << 16; 3 offset of the
//   boundary bond's neighbours; 4 first row of H with its top bit flipped; 5
//   of H with bit 0 flipped; 6 offset of the neighbours across the second J2
//   boundary bond; 7 first row of H with bit top - 1 flipped; 8.. offsets of
//   the J1 bonds within H; 32.. of the J2 bonds.
void build_seg_table(int L, SegTable &t) {
  const int M = kSegM, HB = L - M, up = L / 2;
  std::vector<int> koff(M + 2, 0);
  for (int k = 0; k <= M; ++k) koff[k + 1] = koff[k] + (int)choose(M, k);
  // first row of every high part (ascending states: high parts in order)
  std::vector<int> first((size_t)1 << HB, 0);
  long long row = 0;
  int nseg = 0;
  for (uint32_t H = 0; H < (1u << HB); ++H) {
    const int k = up - __builtin_popcount(H);
    first[H] = (int)row;
    if (k < 0 || k > M) continue;
    row += choose(M, k);
    ++nseg;
  }
  std::vector<int> rec((size_t)nseg * kSegRec, 0);
  std::vector<long long> row0(nseg + 1, 0);
  int q = 0;
  for (uint32_t H = 0; H < (1u << HB); ++H) {
    const int k = up - __builtin_popcount(H);
    if (k < 0 || k > M) continue;
    int *r = rec.data() + (size_t)q * kSegRec;
    const int b0 = H & 1, b1 = (H >> 1) & 1, bt = (H >> (HB - 1)) & 1, bs = (H >> (HB - 2)) & 1;
    int c[2] = {0, 0};
    for (int l = 1; l <= 2; ++l)
      for (int i = 0; i + l < HB; ++i)
        if (((H >> i) ^ (H >> (i + l))) & 1u)
          r[(l == 1 ? 8 : 32) + c[l - 1]++] = first[H ^ ((1u << i) | (1u << (i + l)))] - first[H];
    r[0] = first[H];
    r[1] = (int)choose(M, k) | (koff[k] << 8);
    r[2] = c[0] | (c[1] << 8) | (b0 << 16) | (b1 << 17) | (bt << 18) | (bs << 19);
    // across the top bit of the low part, the other bits keep their order:
    // low parts with it set come after the C(M-1, k) without
    const int kk = (int)choose(M - 1, k), k1 = (int)choose(M - 1, k + 1);
    r[3] = first[H ^ 1u] - first[H] + (b0 ? k1 : -kk);
    r[4] = first[H ^ (1u << (HB - 1))];
    r[5] = first[H ^ 1u];
    r[6] = first[H ^ 2u] - first[H] + (b1 ? k1 : -kk);
    r[7] = first[H ^ (1u << (HB - 2))];
    row0[q] = (long long)first[H];
    ++q;
  }
  row0[nseg] = row;
  t.nseg = nseg;
  for (int lp = 0; lp <= 3; ++lp) {  // parts of about equal numbers of rows
    int at = 0;
    for (int p = 0; p <= 1 << lp; ++p) {
      while (at < nseg && (row0[at] << lp) < row * p) ++at;
      t.seg0[lp][p] = (p == 1 << lp) ? nseg : at;
    }
  }
  std::vector<unsigned char> rows;
  seg_rows(rows);
  t.rec.ensure(sizeof(int) * rec.size());
  t.rows.ensure(rows.size());
  PF_HIP(hipMemcpy(t.rec.p, rec.data(), sizeof(int) * rec.size(), hipMemcpyHostToDevice));
  PF_HIP(hipMemcpy(t.rows.p, rows.data(), rows.size(), hipMemcpyHostToDevice));
}

// -------------------------------------------------------------- kernel --

template <class T, int VE>
__device__ __forceinline__ void piece_add(T (&acc)[VE], T w, const T (&v)[VE]) {
#pragma unroll
  for (int e = 0; e < VE; ++e) acc[e] += w * v[e];
}

// Byte i of a 16-byte record.
__device__ __forceinline__ uint32_t rec_byte(const uint4 &w, int i) {
  const uint32_t x = i < 4 ? w.x : i < 8 ? w.y : i < 12 ? w.z : w.w;
  return (x >> (8 * (i & 3))) & 255u;
}

// Global memory at a scalar base: with the base opaque to the compiler, a
// load is one instruction from (scalar base, 32-bit lane offset) instead of
// 64-bit address arithmetic in every lane.
typedef __attribute__((address_space(1))) char *Gptr;
__device__ __forceinline__ Gptr scalar_base(const void *p, long long off) {
  uintptr_t u = reinterpret_cast<uintptr_t>(p) + (uintptr_t)off;
  asm("" : "+s"(u));
  return (Gptr)u;
}

template <class T, int VE>
struct alignas(sizeof(T) * VE) Piece {
  T v[VE];
};

// (X, Y and the operand of a product are the caller's: aligned as their
// elements are, no more.  The loads are the same.)
template <class T, int VE, bool NT = false>
__device__ __forceinline__ void piece_load(Gptr base, uint32_t off, T (&v)[VE]) {
  typedef T VT __attribute__((ext_vector_type(VE), aligned(sizeof(T))));
  const __attribute__((address_space(1))) VT *at =
      (const __attribute__((address_space(1))) VT *)(base + off);
  const VT p = NT ? __builtin_nontemporal_load(at) : *at;
#pragma unroll
  for (int e = 0; e < VE; ++e) v[e] = p[e];
}
template <class T, int VE, bool NT>
__device__ __forceinline__ void piece_store(Gptr base, uint32_t off, const T (&v)[VE]) {
  typedef T VT __attribute__((ext_vector_type(VE), aligned(sizeof(T))));
  VT p;
#pragma unroll
  for (int e = 0; e < VE; ++e) p[e] = v[e];
  __attribute__((address_space(1))) VT *at = (__attribute__((address_space(1))) VT *)(base + off);
  if (NT)
    __builtin_nontemporal_store(p, at);
  else
    *at = p;
}
template <class T, int VE>
__device__ __forceinline__ void piece_lds(const char *at, T (&v)[VE]) {
  const Piece<T, VE> p = *reinterpret_cast<const Piece<T, VE> *>(at);
#pragma unroll
  for (int e = 0; e < VE; ++e) v[e] = p.v[e];
}

// A segment's record: constant memory to the compiler, read with scalar loads.
typedef const __attribute__((address_space(4))) int *Rec;
typedef int I16 __attribute__((ext_vector_type(16), aligned(4)));
typedef int I4 __attribute__((ext_vector_type(4), aligned(4)));
struct SegOffsets {
  I16 a;
  I4 b;
  __device__ __forceinline__ int operator[](int e) const { return e < 16 ? a[e & 15] : b[e & 3]; }
};
template <int N>
__device__ __forceinline__ SegOffsets seg_offsets(Rec at) {
  SegOffsets d;
  d.a = *(const __attribute__((address_space(4))) I16 *)at;
  if (N > 16) d.b = *(const __attribute__((address_space(4))) I4 *)(at + 16);
  return d;
}
typedef int I8 __attribute__((ext_vector_type(8), aligned(4)));
template <int NH, bool J2>
struct SegRecord {
  I8 h;
  SegOffsets d1, d2;
  __device__ __forceinline__ void read(const int *table, int seg) {
    const Rec rec = (Rec)(uintptr_t)(table + (size_t)seg * kSegRec);
    h = *(const __attribute__((address_space(4))) I8 *)rec;
    d1 = seg_offsets<NH>(rec + 8);
    if (J2) d2 = seg_offsets<NH - 1>(rec + 32);
  }
};

// Neighbours F .. F + C - 1 of the list d, loads only.
template <class T, int VE, int F, int C>
__device__ __forceinline__ void seg_loads(Gptr V, uint32_t vo, const SegOffsets &d,
                                          T (&h)[C > 0 ? C : 1][VE]) {
  constexpr int kPiece = VE * (int)sizeof(T);
#pragma unroll
  for (int e = 0; e < C; ++e) piece_load<T, VE>(V, vo + (uint32_t)d[F + e] * kPiece, h[e]);
}
template <class T, int VE, int C, int N>
__device__ __forceinline__ void seg_adds(T w, const T (&h)[N][VE], T (&acc)[VE]) {
#pragma unroll
  for (int e = 0; e < C; ++e) piece_add<T, VE>(acc, w, h[e]);
}

// The N bonds within the low part, kNear neighbours from LDS at a time.
constexpr int kNear = 3;
template <class T, int VE, int N>
__device__ __forceinline__ void seg_low(const char *tile, const uint4 &places, T w,
                                        T (&acc)[VE]) {
  constexpr int kPiece = VE * (int)sizeof(T);
#pragma unroll
  for (int f = 0; f < N; f += kNear) {
    T v[kNear][VE];
#pragma unroll
    for (int e = f; e < f + kNear && e < N; ++e)
      piece_lds<T, VE>(tile + rec_byte(places, e) * kPiece, v[e - f]);
#pragma unroll
    for (int e = f; e < f + kNear && e < N; ++e) piece_add<T, VE>(acc, w, v[e - f]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// In-flight neighbours of the list at once (32 registers of 16-byte pieces).
constexpr int kFly = 8;

// The J1 bonds of a row of a segment whose high part has C of its own, and
// the barrier that the segment's tile needs.
template <class T, int VE, int C>
__device__ __forceinline__ void seg_j1(Gptr V, uint32_t vo, const SegOffsets &d, const char *tile,
                                       const uint4 &ra, const T (&vb)[VE], const T (&vw)[VE], T w,
                                       T (&acc)[VE]) {
  constexpr int kPiece = VE * (int)sizeof(T);
  constexpr int C1 = C < kFly ? C : kFly, C2 = C - C1;
  T h[C1 > 0 ? C1 : 1][VE];
  seg_loads<T, VE, 0, C1>(V, vo, d, h);
  __syncthreads();
  seg_low<T, VE, kSegM - 1>(tile, ra, w, acc);
  piece_add<T, VE>(acc, w, vb);
  seg_adds<T, VE, C1>(w, h, acc);
  if constexpr (C2 > 0) {
    T g[C2][VE];
    seg_loads<T, VE, C1, C2>(V, vo, d, g);
    seg_adds<T, VE, C2>(w, g, acc);
  }
  piece_add<T, VE>(acc, w, vw);
}

template <class T, int VE, int C>
__device__ __forceinline__ void seg_j2(Gptr V, uint32_t vo, const SegOffsets &d, const char *tile,
                                       const uint4 &rb, const T (&vp)[VE], const T (&vq)[VE],
                                       const T (&vr)[VE], const T (&vs)[VE], T w, T (&acc)[VE]) {
  constexpr int kPiece = VE * (int)sizeof(T);
  constexpr int C1 = C < kFly ? C : kFly, C2 = C - C1;
  T h[C1 > 0 ? C1 : 1][VE];
  seg_loads<T, VE, 0, C1>(V, vo, d, h);
  seg_low<T, VE, kSegM - 2>(tile, rb, w, acc);
  piece_add<T, VE>(acc, w, vp);
  piece_add<T, VE>(acc, w, vq);
  seg_adds<T, VE, C1>(w, h, acc);
  if constexpr (C2 > 0) {
    T g[C2][VE];
    seg_loads<T, VE, C1, C2>(V, vo, d, g);
    seg_adds<T, VE, C2>(w, g, acc);
  }
  piece_add<T, VE>(acc, w, vr);
  piece_add<T, VE>(acc, w, vs);
}

// Cases 0 .. N of C, each with its own straight code.
template <int N, class F>
__device__ __forceinline__ void with_count(int c, F &&f) {
  if constexpr (N == 0) {
    f(std::integral_constant<int, 0>{});
  } else {
    if (c == N)
      f(std::integral_constant<int, N>{});
    else
      with_count<N - 1>(c, f);
  }
}

// One lane a piece (VE values, at most 16 bytes) of a row.  NH: the most bonds
// within a high part (L - kSegM - 1).  NT: X, W and out pass the caches by.
// DOT: this segment's sums of out^2 and out V go to a.dots as well.
template <class T, int VE, int NH, bool J2, bool NT, bool DOT>
__device__ __forceinline__ void segment_step(const SegArgs<T> &a, int slice, int seg, char *tile) {
  constexpr int kPiece = VE * (int)sizeof(T);
  SegRecord<NH, J2> r;
  r.read(a.rec, seg);
  const int tid = threadIdx.x;
  const bool has_x = a.X != nullptr, has_w = a.W != nullptr;
  const int base = r.h[0];
  const int nr = r.h[1] & 255, r0 = r.h[1] >> 8;
  const int flags = r.h[2];
  const uint32_t b0 = (flags >> 16) & 1, b1 = (flags >> 17) & 1, bt = (flags >> 18) & 1,
                 bs = (flags >> 19) & 1;
  const Gptr V = scalar_base(a.V, (long long)slice * a.vss);
  const bool in = tid < nr;
  // (lanes past the segment's end follow its first row and store nothing)
  const uint32_t i = in ? tid : 0;
  const uint32_t vo = (uint32_t)(base + i) * kPiece;  // (a slice is under 4 GB)
  T self[VE], vb[VE], vw[VE], xv[VE], wv[VE];
  piece_load<T, VE>(V, vo, self);
  const Gptr rows = scalar_base(a.rows, 32ll * r0);
  typedef uint32_t U4v __attribute__((ext_vector_type(4)));
  const U4v rav = *(const __attribute__((address_space(1))) U4v *)(rows + i * 32u);
  const uint4 ra = make_uint4(rav[0], rav[1], rav[2], rav[3]);
  uint4 rb;
  if constexpr (J2) {
    const U4v rbv = *(const __attribute__((address_space(1))) U4v *)(rows + i * 32u + 16u);
    rb = make_uint4(rbv[0], rbv[1], rbv[2], rbv[3]);
  }
  const T dt = *(const __attribute__((address_space(1))) T *)(
      scalar_base(a.dt, 0) + (uint32_t)(base + i) * (uint32_t)sizeof(T));
#pragma unroll
  for (int e = 0; e < VE; ++e) xv[e] = wv[e] = vb[e] = vw[e] = T(0);
  if (has_x)
    piece_load<T, VE, NT>(scalar_base(a.X, (long long)(slice * a.xss + (size_t)base * a.xrow)),
                          i * a.xrow, xv);
  if (has_w) piece_load<T, VE, NT>(scalar_base(a.W, (long long)slice * a.vss), vo, wv);
  {
    Piece<T, VE> p;
#pragma unroll
    for (int e = 0; e < VE; ++e) p.v[e] = in ? self[e] : T(0);
    // (place 255, past every segment's end, holds the zero of inactive bonds)
    *reinterpret_cast<Piece<T, VE> *>(tile + tid * kPiece) = p;
  }
  const uint32_t lo = ra.w & 0xffffu;
  if (((lo >> (kSegM - 1)) & 1u) != b0)
    piece_load<T, VE>(V, vo + (uint32_t)r.h[3] * kPiece, vb);
  const uint32_t f0 = rec_byte(ra, 9);
  if ((lo & 1u) != bt) piece_load<T, VE>(V, ((uint32_t)r.h[4] + f0) * kPiece, vw);
  T acc[VE];
  const T dd = a.dscale * dt;
#pragma unroll
  for (int e = 0; e < VE; ++e) acc[e] = dd * self[e];
  with_count<NH>(flags & 255, [&](auto c) {
    seg_j1<T, VE, decltype(c)::value>(V, vo, r.d1, tile, ra, vb, vw, a.w1, acc);
  });
  if constexpr (J2) {
    T vp[VE], vq[VE], vr[VE], vs[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) vp[e] = vq[e] = vr[e] = vs[e] = T(0);
    if (((lo >> (kSegM - 2)) & 1u) != b0)
      piece_load<T, VE>(V, ((uint32_t)r.h[5] + rec_byte(ra, 11)) * kPiece, vp);
    if (((lo >> (kSegM - 1)) & 1u) != b1)
      piece_load<T, VE>(V, vo + (uint32_t)r.h[6] * kPiece, vq);
    if ((lo & 1u) != bs) piece_load<T, VE>(V, ((uint32_t)r.h[7] + f0) * kPiece, vr);
    if (((lo >> 1) & 1u) != bt)
      piece_load<T, VE>(V, ((uint32_t)r.h[4] + rec_byte(ra, 10)) * kPiece, vs);
    with_count<NH - 1>((flags >> 8) & 255, [&](auto c) {
      seg_j2<T, VE, decltype(c)::value>(V, vo, r.d2, tile, rb, vp, vq, vr, vs, a.w2, acc);
    });
  }
  if (has_x) piece_add<T, VE>(acc, a.alpha, xv);
  if (has_w) piece_add<T, VE>(acc, a.gamma, wv);
  if (in)
    piece_store<T, VE, NT>(scalar_base(a.out, (long long)(slice * a.oss + (size_t)base * a.orow)),
                           i * a.orow, acc);
  if constexpr (DOT) {
    // lanes in a fixed butterfly, then the four waves in order
    __shared__ T red[4][2];
    T s0 = T(0), s1 = T(0);
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      s0 += in ? acc[e] * acc[e] : T(0);
      s1 += in ? acc[e] * self[e] : T(0);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      s0 += __shfl_xor(s0, o);
      s1 += __shfl_xor(s1, o);
    }
    if ((tid & 63) == 0) {
      red[tid >> 6][0] = s0;
      red[tid >> 6][1] = s1;
    }
    __syncthreads();
    if (tid < 2)
      a.dots[2 * ((size_t)slice * a.nseg + seg) + tid] =
          ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
  }
}

// (24 and more registers short of 128: six waves a SIMD, five with J2, hide
// the round of loads better than four with every neighbour in flight)
#define PF_SEG_KERNEL(J2, NH) \
  __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(((J2) || (NH) > 15) ? 5 : 6, 8)))

template <class T, int VE, int NH, bool J2, bool NT, bool DOT = false>
PF_SEG_KERNEL(J2, NH) void k_segment(SegArgs<T> a) {
  __shared__ __align__(16) char tile[256 * VE * (int)sizeof(T)];
  const int x = blockIdx.x & 7;
  const int part = x & ((1 << a.lparts) - 1);
  const int slice = ((int)blockIdx.y << (3 - a.lparts)) + (x >> a.lparts);
  const int seg = __builtin_amdgcn_readfirstlane(a.seg0[part] + (int)(blockIdx.x >> 3));
  if (slice >= a.nslices || seg >= a.seg0[part + 1]) return;
  segment_step<T, VE, NH, J2, NT, DOT>(a, slice, seg, tile);
}

// Global step j of the batched Clenshaw filter (members end together at step
// Kmax; one of order K_i is idle before step Kmax - K_i + 1).  A workgroup's
// member, slice and segment stand in the task list: XCD x takes the x-th of
// its eight parts.
template <class T, int VE, int NH, bool J2>
PF_SEG_KERNEL(J2, NH) void k_segment_batch(const SegItem<T> *items, const int2 *tasks, int per,
                                           const unsigned char *rows, long long j,
                                           long long Kmax) {
  __shared__ __align__(16) char tile[256 * VE * (int)sizeof(T)];
  typedef const __attribute__((address_space(4))) int *Ci;
  const Ci task = (Ci)(uintptr_t)(tasks + (size_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3));
  const int who = task[0], seg = task[1];
  if (seg < 0) return;  // (the list's parts are filled up)
  const int slice = who >> 20;
  // (read with scalar loads)
  typedef const __attribute__((address_space(4))) SegItem<T> *Item;
  const Item it = (Item)(uintptr_t)(items + (who & 0xfffff));
  const long long K = it->K, ji = j - (Kmax - K);
  if (ji < 1) return;
  const bool last = ji == K;
  typedef const __attribute__((address_space(4))) double *Cd;
  const double c = ((Cd)(uintptr_t)it->coef)[K - ji];
  const double Dinv = it->Dinv;
  SegArgs<T> a;
  a.rec = it->rec;
  a.rows = rows;
  a.dt = it->dt;
  a.V = (ji & 1) ? it->b0 : it->b1;
  a.W = ji >= 2 ? ((ji & 1) ? it->b1 : it->b0) : nullptr;
  const bool to_y = last && it->orow != 0;
  a.out = to_y ? it->Y : (ji & 1) ? it->b1 : it->b0;
  a.orow = to_y ? it->orow : (uint32_t)(VE * sizeof(T));
  a.X = (last || c != 0.0) ? it->X : nullptr;
  a.xrow = it->xrow;
  a.xss = a.vss = a.oss = it->ss;
  a.alpha = last ? (T)(c * Dinv) : (T)c;
  a.dscale = last ? (T)Dinv : T(2);
  a.w1 = last ? it->w1f : it->w1;
  a.w2 = last ? it->w2f : it->w2;
  a.gamma = last ? (T)(-Dinv) : T(-1);
  segment_step<T, VE, NH, J2, false, false>(a, slice, seg, tile);
}

// ------------------------------------------------------------ layout --

// X (n x S, row-major, leading dimension ldx) to slices of w columns, and
// beta X to the slices of `scaled` where that is not null (zero for beta = 0,
// also where X is not finite); or (UNPACK) slices to X.  A lane moves a piece of VE values, a row's lanes next to each other:
// the row-major side is coalesced, and a workgroup fills whole lines of every
// slice (10.4 M x 64 FP64: 2.1 ms for 10.7 GB).
template <class T, int VE, bool UNPACK>
__global__ __launch_bounds__(256) void k_slices(long long n, int S, int w, T *X, long long ldx,
                                                T *packed, T beta, T *scaled) {
  typedef T VT __attribute__((ext_vector_type(VE), aligned(sizeof(T))));
  const int per = S / VE;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n * per) return;
  const long long r = i / per;
  const int c = (int)(i - r * per) * VE;
  T *x = X + (size_t)r * ldx + c;
  const size_t at = (size_t)(c / w) * n * w + (size_t)r * w + c % w;
  if (UNPACK) {
    *(VT *)x = *(const VT *)(packed + at);
  } else {
    const VT v = *(const VT *)x;
    if (packed) *(VT *)(packed + at) = v;
    if (scaled) {
      VT b;
#pragma unroll
      for (int e = 0; e < VE; ++e) b[e] = beta != T(0) ? beta * v[e] : T(0);
      *(VT *)(scaled + at) = b;
    }
  }
}

// ---------------------------------------------------------- launchers --

template <class T, int VE, int NH>
static void launch_one(hipStream_t st, dim3 grid, bool has_j2, bool nt, const SegArgs<T> &a) {
  if (a.dots) {
    if constexpr (sizeof(T) == 8)
      has_j2 ? k_segment<T, VE, NH, true, false, true><<<grid, 256, 0, st>>>(a)
             : k_segment<T, VE, NH, false, false, true><<<grid, 256, 0, st>>>(a);
    else
      throw Error(POLFED_EINVAL, "segment step: sums are FP64");
    check_launch("k_segment");
    return;
  }
  if (has_j2)
    nt ? k_segment<T, VE, NH, true, true><<<grid, 256, 0, st>>>(a)
       : k_segment<T, VE, NH, true, false><<<grid, 256, 0, st>>>(a);
  else
    nt ? k_segment<T, VE, NH, false, true><<<grid, 256, 0, st>>>(a)
       : k_segment<T, VE, NH, false, false><<<grid, 256, 0, st>>>(a);
  check_launch("k_segment");
}

template <class T, int VE>
static void launch_nh(hipStream_t st, int L, dim3 grid, bool has_j2, bool nt, const SegArgs<T> &a) {
  const int nh = L - kSegM - 1;
  if (nh <= 7)
    launch_one<T, VE, 7>(st, grid, has_j2, nt, a);
  else if (nh <= 11)
    launch_one<T, VE, 11>(st, grid, has_j2, nt, a);
  else if (nh <= 15)
    launch_one<T, VE, 15>(st, grid, has_j2, nt, a);
  else
    launch_one<T, VE, 19>(st, grid, has_j2, nt, a);
}

template <class T, int VE>
static void launch_batch_nh(hipStream_t st, int L, bool has_j2, unsigned grid,
                            const SegItem<T> *items, const int2 *tasks, int per,
                            const unsigned char *rows, long long j, long long Kmax) {
  auto go = [&](auto nh) {
    constexpr int NH = decltype(nh)::value;
    if (has_j2)
      k_segment_batch<T, VE, NH, true><<<grid, 256, 0, st>>>(items, tasks, per, rows, j, Kmax);
    else
      k_segment_batch<T, VE, NH, false><<<grid, 256, 0, st>>>(items, tasks, per, rows, j, Kmax);
  };
  const int nh = L - kSegM - 1;
  if (nh <= 7)
    go(std::integral_constant<int, 7>{});
  else if (nh <= 11)
    go(std::integral_constant<int, 11>{});
  else if (nh <= 15)
    go(std::integral_constant<int, 15>{});
  else
    go(std::integral_constant<int, 19>{});
  check_launch("k_segment_batch");
}

template <class T>
void launch_segment_batch(hipStream_t st, int Lmax, bool has_j2, int S, const SegItem<T> *items,
                          const int2 *tasks, int per, const unsigned char *rows, long long j,
                          long long Kmax) {
  if (per <= 0) return;
  const int w = segment_width<T>(S);
  constexpr int F = 16 / (int)sizeof(T);
  const unsigned grid = 8u * (unsigned)per;
  if (w == F)
    launch_batch_nh<T, F>(st, Lmax, has_j2, grid, items, tasks, per, rows, j, Kmax);
  else if (w == 2)
    launch_batch_nh<T, 2>(st, Lmax, has_j2, grid, items, tasks, per, rows, j, Kmax);
  else
    launch_batch_nh<T, 1>(st, Lmax, has_j2, grid, items, tasks, per, rows, j, Kmax);
}

template <class T>
int segment_width(int S) {
  return std::min(S, 16 / (int)sizeof(T));
}

template <class T>
void launch_segment(hipStream_t st, int L, bool has_j2, int S, const SegTable &t, SegArgs<T> a) {
  const int w = segment_width<T>(S);
  const double n = (double)polfed_dim(L);
  a.nslices = S / w;
  a.nseg = t.nseg;
  a.rec = t.rec.as<int>();
  a.rows = t.rows.as<unsigned char>();
  // An XCD sweeps a slice of its own where its L2 (4 MB) holds a good part of
  // it (L = 18, s = 16 J1-J2 FP64: 8.0 us a step against 10.0 with all XCDs on
  // one slice, an eighth of the rows each); longer slices go one after the
  // other, so that the Infinity Cache holds the one that is gathered from (L
  // = 26, s = 64 FP64: 7.5 against 8.3 ms; L = 22, 11 MB a slice: equal).
  int lp = (n * w * sizeof(T) > 16e6) ? 3 : 0;
  while ((8 >> lp) > a.nslices) ++lp;
  a.lparts = lp;
  int most = 0;
  for (int p = 0; p < 1 << lp; ++p) {
    a.seg0[p] = t.seg0[lp][p];
    most = std::max(most, t.seg0[lp][p + 1] - t.seg0[lp][p]);
  }
  a.seg0[1 << lp] = t.nseg;
  const int conc = 8 >> lp;
  const dim3 grid((unsigned)(8 * most), (unsigned)((a.nslices + conc - 1) / conc));
  // X, W and out pass the caches by where the step's blocks are several times
  // the 256 MB Infinity Cache (L = 26: 7.5 against 8.1 ms); below that they
  // stay in it from step to step (L = 22, s = 32 FP32, 361 MB: 91 us a step
  // against 106; L = 20, s = 32 FP64, 190 MB: 39 against 52)
  const bool nt = 4.0 * n * S * sizeof(T) > 1e9;
  constexpr int F = 16 / (int)sizeof(T);
  if (w == F) return launch_nh<T, F>(st, L, grid, has_j2, nt, a);
  if constexpr (F >= 4)
    if (w == 2) return launch_nh<T, 2>(st, L, grid, has_j2, nt, a);
  launch_nh<T, 1>(st, L, grid, has_j2, nt, a);
}

template <class T, bool UNPACK>
static void slices(hipStream_t st, long long n, int S, T *X, long long ldx, T *packed, T beta,
                   T *scaled) {
  const int w = segment_width<T>(S);
  const long long tot = n * (S / w);
  const unsigned nwg = (unsigned)((tot + 255) / 256);
  if (w == 4 && sizeof(T) == 4)
    k_slices<T, 16 / (int)sizeof(T), UNPACK><<<nwg, 256, 0, st>>>(n, S, w, X, ldx, packed, beta, scaled);
  else if (w == 2)
    k_slices<T, 2, UNPACK><<<nwg, 256, 0, st>>>(n, S, w, X, ldx, packed, beta, scaled);
  else
    k_slices<T, 1, UNPACK><<<nwg, 256, 0, st>>>(n, S, w, X, ldx, packed, beta, scaled);
  check_launch("k_slices");
}
template <class T>
void launch_to_slices(hipStream_t st, long long n, int S, const T *X, long long ldx, T *packed,
                      T beta, T *scaled) {
  slices<T, false>(st, n, S, const_cast<T *>(X), ldx, packed, beta, scaled);
}
template <class T>
void launch_from_slices(hipStream_t st, long long n, int S, const T *packed, T *Y, long long ldy) {
  slices<T, true>(st, n, S, Y, ldy, const_cast<T *>(packed), T(0), nullptr);
}

// Every XCD's share of the members' (slice, segment) pairs: below 64 slices in
// all, an eighth of each slice's rows (the chip is not full otherwise); above,
// whole slices (an XCD's L2 then serves all gathers of a slice), the next one
// to the XCD with the fewest rows so far.
void segment_tasks(const std::vector<const SegTable *> &tables, int nslices,
                   std::vector<int2> &tasks, int &per) {
  std::vector<int2> part[8];
  const bool split = tables.size() * (size_t)nslices < 64;
  size_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (size_t i = 0; i < tables.size(); ++i)
    for (int s = 0; s < nslices; ++s) {
      const SegTable &t = *tables[i];
      const int who = (int)i | (s << 20);
      if (split) {
        for (int x = 0; x < 8; ++x)
          for (int q = t.seg0[3][x]; q < t.seg0[3][x + 1]; ++q) part[x].push_back(make_int2(who, q));
      } else {
        int x = 0;
        for (int y = 1; y < 8; ++y)
          if (load[y] < load[x]) x = y;
        load[x] += t.nseg;
        for (int q = 0; q < t.nseg; ++q) part[x].push_back(make_int2(who, q));
      }
    }
  size_t most = 0;
  for (auto &p : part) most = std::max(most, p.size());
  per = (int)most;
  tasks.clear();
  for (auto &p : part) {
    p.resize(most, make_int2(0, -1));
    tasks.insert(tasks.end(), p.begin(), p.end());
  }
}

#define PF_SEG(T)                                                                              \
  template int segment_width<T>(int);                                                          \
  template void launch_segment<T>(hipStream_t, int, bool, int, const SegTable &, SegArgs<T>);  \
  template void launch_segment_batch<T>(hipStream_t, int, bool, int, const SegItem<T> *,       \
                                        const int2 *, int, const unsigned char *, long long,   \
                                        long long);                                            \
  template void launch_to_slices<T>(hipStream_t, long long, int, const T *, long long, T *, T, \
                                    T *);                                                      \
  template void launch_from_slices<T>(hipStream_t, long long, int, const T *, T *, long long);
PF_SEG(float)
PF_SEG(double)
#undef PF_SEG

}  // namespace polfed
