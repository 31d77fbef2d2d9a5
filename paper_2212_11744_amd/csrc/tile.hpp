// Register-resident matrix algebra on the matrix cores, for state sizes up to 16.
//
// A matrix of a tuple is spread over the lanes of a wave in the layout in which the matrix
// instruction returns its results, and that layout also serves as both operands: a register that
// holds rows k of X is, read as a left operand, rows k of X transposed.  So X^T Y (mm, mv) needs
// no data movement between its operands' producers and itself, whatever chain of products the
// matrices came from: no LDS, no barrier, no lane exchange.  Left factors are therefore either
// symmetric (C, J, S, G) or kept transposed (A).
//
// Layouts (a matrix is n x n with n <= 4 NT, entries beyond n are zero; the entry of a vector is
// held by every lane that a product needs it in: the lanes of its row, in W64 those of vrow):
//   Q64  n <= 8, 4 nodes a wave: v_mfma_f64_4x4x4 works on 4 independent 4 x 4 tiles, one value per
//        lane; lane 16 i + 4 s + j holds entry (4 I + i, 4 J + j) of node s in register I NT + J.
//        Calls in FP32 use it too, with FP32 in memory: v_mfma_f32_4x4x1 on 16 nodes a wave was
//        no faster (4 of its instructions to a tile product, 16 registers to a matrix, twice the
//        code to fetch: the build of 6000 blocks at nx = 7 took 28 us).
//   W64  FP64, n <= 16, one node a wave: v_mfma_f64_16x16x4; lane 16 q + j holds entry (4 r + q, j)
//        in register r.
//   W32  FP32, n <= 16, one node a wave: v_mfma_f32_16x16x4; lane 16 q + j holds entry (4 q + r, j)
//        in register r.
// Measured on one MI355X: v_mfma_f64_4x4x4 issues every 16 cycles and v_mfma_f64_16x16x4 every 64:
// the rate of the vector FMA (they share its FP64 units: interleaved products and FMAs add up), but
// without operand traffic and with 1/16 of the registers per node, so that a combination (Lemma 7)
// takes one wave 1.7 us for 4 nodes at nx = 8 and 2.9 us for one at nx = 16, of which the inverse
// is about half.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "lqt_internal.hpp"

#define TDEV __device__ __forceinline__

namespace lqt {
namespace tile {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

TDEV int lane_id() { return threadIdx.x & 63; }

// Calls f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): lane-exchange controls
// are immediates of the instruction.
template <int I, int N, class F>
TDEV void unroll(const F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<I + 1, N>(f);
  }
}

// Value of lane L of each row of 16 lanes, in all of them.
template <int L>
TDEV double row_bcast(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const long long r = __builtin_amdgcn_update_dpp(b, b, 0x150 + L, 0xF, 0xF, true);
  return __builtin_bit_cast(double, r);
}
template <int L>
TDEV float row_bcast(float x) {
  const int b = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, 0x150 + L, 0xF, 0xF, true));
}
// Value of lane L of each group of 4 lanes, in all of them.
template <int L>
TDEV int quad_bcast_i(int x) {
  return __builtin_amdgcn_update_dpp(x, x, L * 0x55, 0xF, 0xF, true);
}
template <int L>
TDEV float quad_bcast(float x) {
  return __builtin_bit_cast(float, quad_bcast_i<L>(__builtin_bit_cast(int, x)));
}
template <int L>
TDEV double quad_bcast(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = quad_bcast_i<L>((int)b), hi = quad_bcast_i<L>((int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// 1 / x: the hardware estimate refined by Newton-Raphson steps (within about an ulp).
TDEV double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}
TDEV float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// Elimination without row exchanges is used while every multiplier (and reciprocal pivot) stays
// within this bound, and repeated with partial pivoting (invert_pivoted) otherwise.  The systems
// are I + J C with C, J positive semidefinite: on the package's workloads (nx 4 .. 16, every level
// of the trees, spans up to the whole horizon) the largest multiplier met is 1.02.
constexpr float kMaxMultiplier = 4.0f;

// ------------------------------------------------------------------------------------------
// Backends.  MR: registers per matrix, VR: per vector; row(r), col(r): the entry held in register
// r of a matrix; vrow(v): the row held in register v of a vector; rep(): true in one lane of the
// lanes that share a vector entry.
// ------------------------------------------------------------------------------------------
template <int N_, class Mem_>
struct Q64 {
  using R = double;
  using Mem = Mem_;
  static constexpr int N = N_, NT = (N + 3) / 4, MR = NT * NT, VR = NT, NODES = 4, LANES = 16;
  static constexpr bool kFull = N % 4 == 0;  // no register holds an entry beyond N
  static_assert(N <= 8, "two tiles of 4 a side at most");
  static TDEV int node() { return (lane_id() >> 2) & 3; }
  static TDEV int sub() { return ((lane_id() >> 4) << 2) | (lane_id() & 3); }
  static TDEV int row(int r) { return 4 * (r / NT) + (lane_id() >> 4); }
  static TDEV int col(int r) { return 4 * (r % NT) + (lane_id() & 3); }
  static TDEV int vrow(int v) { return 4 * v + (lane_id() >> 4); }
  static TDEV bool rep() { return (lane_id() & 3) == 0; }
  // where in a dump of the registers ([r][sub]) register r's transposed entry lies
  static TDEV int tpos(int r) {
    return ((r % NT) * NT + r / NT) * LANES + ((lane_id() & 3) << 2) + (lane_id() >> 4);
  }
  // acc += X^T Y.  UP: the tiles on and above the diagonal only.  it: tile rows of the result (the
  // others are not touched), kt: tiles of inner dimension (the rest of X and Y is zero).
  template <bool UP = false>
  static TDEV void mm(R (&acc)[MR], const R (&X)[MR], const R (&Y)[MR], int it = NT,
                      int kt = NT) {
#pragma unroll
    for (int K = 0; K < NT; ++K)
#pragma unroll
      for (int I = 0; I < NT; ++I)
#pragma unroll
        for (int J = 0; J < NT; ++J) {
          if ((UP && I > J) || I >= it || K >= kt) continue;
          acc[I * NT + J] = __builtin_amdgcn_mfma_f64_4x4x4f64(X[K * NT + I], Y[K * NT + J],
                                                               acc[I * NT + J], 0, 0, 0);
        }
  }
  // The tiles below the diagonal from those above (a product with the identity transposes).
  static TDEV void mirror(R (&M)[MR]) {
    const R eye = (lane_id() >> 4) == (lane_id() & 3) ? R(1) : R(0);
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
      for (int J = 0; J < I; ++J)
        M[I * NT + J] = __builtin_amdgcn_mfma_f64_4x4x4f64(M[J * NT + I], eye, R(0), 0, 0, 0);
  }
  // acc += X^T y
  static TDEV void mv(R (&acc)[VR], const R (&X)[MR], const R (&y)[VR]) {
#pragma unroll
    for (int K = 0; K < NT; ++K)
#pragma unroll
      for (int I = 0; I < NT; ++I)
        acc[I] = __builtin_amdgcn_mfma_f64_4x4x4f64(X[K * NT + I], y[K], acc[I], 0, 0, 0);
  }
  // M <- M^{-1} by Gauss-Jordan elimination in place, no row exchanges; returns the largest
  // multiplier of this lane's rows.  The pivot row reaches the other rows through a product with a
  // one-hot tile.
  static TDEV R invert(R (&M)[MR]) {
    const int li = lane_id() >> 4, lj = lane_id() & 3;
    R mx = R(0);  // largest multiplier
    unroll<0, N>([&](auto cc) {
      constexpr int c = decltype(cc)::value, Ic = c / 4, ic = c % 4;
      const R hot = li == ic ? R(1) : R(0);
      R p[NT], f[NT], m[NT];
#pragma unroll
      for (int J = 0; J < NT; ++J)
        p[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(hot, M[Ic * NT + J], R(0), 0, 0, 0);
#pragma unroll
      for (int I = 0; I < NT; ++I) f[I] = quad_bcast<ic>(M[I * NT + Ic]);
      const R piv = quad_bcast<ic>(p[Ic]);
      const R inv = recip(piv);
#pragma unroll
      for (int I = 0; I < NT; ++I) {
        m[I] = I == Ic && li == ic ? inv : -f[I] * inv;
        mx = fmax(mx, fabs(m[I]));
      }
      p[Ic] = lj == ic ? R(1) : p[Ic];
#pragma unroll
      for (int I = 0; I < NT; ++I)
#pragma unroll
        for (int J = 0; J < NT; ++J) {
          R base = M[I * NT + J];
          if (J == Ic) base = lj == ic ? R(0) : base;
          if (I == Ic) base = li == ic ? R(0) : base;
          M[I * NT + J] = fma(m[I], p[J], base);
        }
    });
    return mx;
  }
};

template <int N_>
struct W64 {
  using R = double;
  using Mem = double;
  static constexpr int N = N_, NT = (N + 3) / 4, MR = NT, VR = 1, NODES = 1, LANES = 64;
  static_assert(N <= 16, "one 16 x 16 tile");
  static constexpr bool kFull = N == 16;
  static TDEV int node() { return 0; }
  static TDEV int sub() { return lane_id(); }
  static TDEV int row(int r) { return 4 * r + (lane_id() >> 4); }
  static TDEV int col(int) { return lane_id() & 15; }
  static TDEV int vrow(int) { return (lane_id() & 12) + (lane_id() >> 4); }
  static TDEV bool rep() { return (lane_id() & 3) == 0; }
  static TDEV int tpos(int r) {
    const int l = lane_id();
    return ((l & 15) >> 2) * LANES + ((l & 3) << 4) + (l >> 4) + 4 * r;
  }
  template <bool UP = false>
  static TDEV void mm(R (&acc)[MR], const R (&X)[MR], const R (&Y)[MR], int = NT, int kt = NT) {
    d4 a = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < NT; ++r) a[r] = acc[r];
#pragma unroll
    for (int K = 0; K < NT; ++K) {
      if (K >= kt) break;
      a = __builtin_amdgcn_mfma_f64_16x16x4f64(X[K], Y[K], a, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < NT; ++r) acc[r] = a[r];
  }
  static TDEV void mirror(R (&)[MR]) {}
  // The 4 x 4 x 4 instruction on the same registers takes the entry of row 4 K + q of y in the lanes
  // 16 q .. (a row broadcast from lane 4 K of every 16) and returns row 4 b + i of X^T y in the
  // lanes 16 i + 4 b .., the form vectors are kept in.
  static TDEV void mv(R (&acc)[VR], const R (&X)[MR], const R (&y)[VR]) {
    unroll<0, NT>([&](auto K) {
      acc[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(X[decltype(K)::value],
                                                  row_bcast<4 * decltype(K)::value>(y[0]), acc[0],
                                                  0, 0, 0);
    });
  }
  static TDEV R invert(R (&M)[MR]) {
    const int li = lane_id() >> 4, lj = lane_id() & 15;
    R mx = R(0);  // largest multiplier
    unroll<0, N>([&](auto cc) {
      constexpr int c = decltype(cc)::value, rc = c / 4, ic = c % 4;
      const R hot = li == ic ? R(1) : R(0);
      R p = __builtin_amdgcn_mfma_f64_4x4x4f64(hot, M[rc], R(0), 0, 0, 0);
      R f[NT], m[NT];
#pragma unroll
      for (int r = 0; r < NT; ++r) f[r] = row_bcast<c>(M[r]);
      const R piv = row_bcast<c>(p);
      const R inv = recip(piv);
#pragma unroll
      for (int r = 0; r < NT; ++r) {
        m[r] = r == rc && li == ic ? inv : -f[r] * inv;
        mx = fmax(mx, fabs(m[r]));
      }
      p = lj == c ? R(1) : p;
#pragma unroll
      for (int r = 0; r < NT; ++r) {
        R base = lj == c ? R(0) : M[r];
        if (r == rc) base = li == ic ? R(0) : base;
        M[r] = fma(m[r], p, base);
      }
    });
    return mx;
  }
};

template <int N_>
struct W32 {
  using R = float;
  using Mem = float;
  static constexpr int N = N_, NT = 4, MR = 4, VR = 4, NODES = 1, LANES = 64;
  static_assert(N <= 16, "one 16 x 16 tile");
  static constexpr bool kFull = N == 16;
  static TDEV int node() { return 0; }
  static TDEV int sub() { return lane_id(); }
  static TDEV int row(int r) { return 4 * (lane_id() >> 4) + r; }
  static TDEV int col(int) { return lane_id() & 15; }
  static TDEV int vrow(int v) { return 4 * (lane_id() >> 4) + v; }
  static TDEV bool rep() { return (lane_id() & 15) == 0; }
  static TDEV int tpos(int r) {
    const int l = lane_id();
    return (l & 3) * LANES + ((l & 15) >> 2) * 16 + 4 * (l >> 4) + r;
  }
  static TDEV f4 pack(const R (&x)[MR]) { return f4{x[0], x[1], x[2], x[3]}; }
  static TDEV void mirror(R (&)[MR]) {}
  template <bool UP = false>
  static TDEV void mm(R (&acc)[MR], const R (&X)[MR], const R (&Y)[MR], int = 4, int = 4) {
    f4 a = pack(acc);
#pragma unroll
    for (int K = 0; K < 4; ++K) a = __builtin_amdgcn_mfma_f32_16x16x4f32(X[K], Y[K], a, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = a[r];
  }
  static TDEV void mv(R (&acc)[VR], const R (&X)[MR], const R (&y)[VR]) {
    f4 a = pack(acc);
#pragma unroll
    for (int K = 0; K < 4; ++K) a = __builtin_amdgcn_mfma_f32_16x16x4f32(X[K], y[K], a, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = a[r];
  }
  static TDEV R invert(R (&M)[MR]) {
    const int li = lane_id() >> 4, lj = lane_id() & 15;
    R mx = R(0);  // largest multiplier
    unroll<0, N>([&](auto cc) {
      constexpr int c = decltype(cc)::value, qc = c / 4, rc = c % 4;
      const R hot = li == qc ? R(1) : R(0);
      const f4 z = {0, 0, 0, 0};
      R p = __builtin_amdgcn_mfma_f32_16x16x4f32(hot, M[rc], z, 0, 0, 0)[0];
      R f[4], m[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) f[r] = row_bcast<c>(M[r]);
      const R piv = row_bcast<c>(p);
      const R inv = recip(piv);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        m[r] = r == rc && li == qc ? inv : -f[r] * inv;
        mx = fmaxf(mx, fabsf(m[r]));
      }
      p = lj == c ? R(1) : p;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        R base = lj == c ? R(0) : M[r];
        if (r == rc) base = li == qc ? R(0) : base;
        M[r] = fmaf(m[r], p, base);
      }
    });
    return mx;
  }
};

// The backend of state size N for a call of type Mem.
template <class Mem, int N>
struct Pick;
template <int N>
struct Pick<double, N> {
  using T = std::conditional_t<(N <= 8), Q64<(N <= 8 ? N : 1), double>, W64<N>>;
};
template <int N>
struct Pick<float, N> {
  using T = std::conditional_t<(N <= 8), Q64<(N <= 8 ? N : 1), float>, W32<N>>;
};

template <class B>
struct Mat {
  typename B::R x[B::MR];
};
template <class B>
struct Vec {
  typename B::R x[B::VR];
};

template <class B>
TDEV Mat<B> mzero() {
  Mat<B> m;
#pragma unroll
  for (int r = 0; r < B::MR; ++r) m.x[r] = 0;
  return m;
}
template <class B>
TDEV Vec<B> vzero() {
  Vec<B> v;
#pragma unroll
  for (int r = 0; r < B::VR; ++r) v.x[r] = 0;
  return v;
}
template <class B>
TDEV bool mdiag(int r) {
  return B::row(r) == B::col(r) && B::row(r) < B::N;
}
// m + I
template <class B>
TDEV Mat<B> plus_eye(const Mat<B>& a) {
  using R = typename B::R;
  Mat<B> m;
#pragma unroll
  for (int r = 0; r < B::MR; ++r) m.x[r] = a.x[r] + (mdiag<B>(r) ? R(1) : R(0));
  return m;
}
template <class B>
TDEV Mat<B> add(const Mat<B>& a, const Mat<B>& b) {
  Mat<B> m;
#pragma unroll
  for (int r = 0; r < B::MR; ++r) m.x[r] = a.x[r] + b.x[r];
  return m;
}
template <class B>
TDEV Vec<B> add(const Vec<B>& a, const Vec<B>& b) {
  Vec<B> m;
#pragma unroll
  for (int r = 0; r < B::VR; ++r) m.x[r] = a.x[r] + b.x[r];
  return m;
}
template <class B>
TDEV Mat<B> neg(const Mat<B>& a) {
  Mat<B> m;
#pragma unroll
  for (int r = 0; r < B::MR; ++r) m.x[r] = -a.x[r];
  return m;
}
template <class B>
TDEV Vec<B> neg(const Vec<B>& a) {
  Vec<B> m;
#pragma unroll
  for (int r = 0; r < B::VR; ++r) m.x[r] = -a.x[r];
  return m;
}
// acc + X^T Y, acc + X^T y
template <class B>
TDEV Mat<B> mm(Mat<B> acc, const Mat<B>& X, const Mat<B>& Y) {
  B::mm(acc.x, X.x, Y.x);
  return acc;
}
template <class B>
TDEV Vec<B> mv(Vec<B> acc, const Mat<B>& X, const Vec<B>& y) {
  B::mv(acc.x, X.x, y.x);
  return acc;
}

// X^T Y, X^T y.  A sum whose first term is much larger than the rest (base + X^T Y with X or Y a
// deviation of short blocks) adds the base last: one rounding at its magnitude instead of n.
template <class B>
TDEV Mat<B> mm0(const Mat<B>& X, const Mat<B>& Y) {
  return mm<B>(mzero<B>(), X, Y);
}
template <class B>
TDEV Vec<B> mv0(const Mat<B>& X, const Vec<B>& y) {
  return mv<B>(vzero<B>(), X, y);
}

// The symmetric part (M + M^T) / 2; the transpose is a product with the identity, which is exact.
template <class B>
TDEV Mat<B> sym(const Mat<B>& M) {
  using R = typename B::R;
  const Mat<B> T = mm<B>(mzero<B>(), M, plus_eye<B>(mzero<B>()));
  Mat<B> S;
#pragma unroll
  for (int r = 0; r < B::MR; ++r) S.x[r] = R(0.5) * (M.x[r] + T.x[r]);
  return S;
}

template <class B>
TDEV Mat<B> sym32(const Mat<B>& M) {
  if constexpr (sizeof(typename B::R) == 4)
    return sym<B>(M);
  else
    return M;
}

// Loads and stores.  at(i, j): the offset of entry (i, j); entries beyond N and nodes that are not
// live read as zero (a tuple of zeros is the identity in the A - I form) and are not written.
template <class B, class P, class F>
TDEV Mat<B> mload(bool live, const P* g, const F& at) {
  // lanes beyond N read entry N - 1 and drop it: the loads of a matrix are then one straight run
  Mat<B> m = mzero<B>();
  if (live) {
#pragma unroll
    for (int r = 0; r < B::MR; ++r) {
      const int i = B::row(r), j = B::col(r);
      const P v = g[at(min(i, B::N - 1), min(j, B::N - 1))];
      m.x[r] = i < B::N && j < B::N ? (typename B::R)v : 0;
    }
  }
  return m;
}
template <class B, class P, class F>
TDEV Vec<B> vload(bool live, const P* g, const F& at) {
  Vec<B> v = vzero<B>();
  if (live) {
#pragma unroll
    for (int r = 0; r < B::VR; ++r) {
      const int i = B::vrow(r);
      const P x = g[at(min(i, B::N - 1))];
      v.x[r] = i < B::N ? (typename B::R)x : 0;
    }
  }
  return v;
}
template <class B, class P, class F>
TDEV void mstore(bool live, const Mat<B>& m, P* g, const F& at) {
#pragma unroll
  for (int r = 0; r < B::MR; ++r) {
    const int i = B::row(r), j = B::col(r);
    if (live && i < B::N && j < B::N) g[at(i, j)] = (P)m.x[r];
  }
}
// Upper triangle only.
template <class B, class P, class F>
TDEV void ustore(bool live, const Mat<B>& m, P* g, const F& at) {
#pragma unroll
  for (int r = 0; r < B::MR; ++r) {
    const int i = B::row(r), j = B::col(r);
    if (live && i <= j && j < B::N) g[at(i, j)] = (P)m.x[r];
  }
}
template <class B, class P, class F>
TDEV void vstore(bool live, const Vec<B>& v, P* g, const F& at) {
  if (!B::rep()) return;
#pragma unroll
  for (int r = 0; r < B::VR; ++r) {
    const int i = B::vrow(r);
    if (live && i < B::N) g[at(i)] = (P)v.x[r];
  }
}

// The same in two halves, so that a load can stay in flight until its values are used: a mask or a
// conversion right after a load waits for it.  fetch reads every entry (lanes beyond N entry
// N - 1), so its address has to be valid for nodes that are not live, too.
template <class B, class P, int CNT, class F>
TDEV void fetch(P (&x)[CNT], const P* g, const F& at) {
#pragma unroll
  for (int r = 0; r < CNT; ++r) x[r] = g[at(min(B::row(r), B::N - 1), min(B::col(r), B::N - 1))];
}
template <class B, class P, int CNT, class F>
TDEV void vfetch(P (&x)[CNT], const P* g, const F& at) {
#pragma unroll
  for (int r = 0; r < CNT; ++r) x[r] = g[at(min(B::vrow(r), B::N - 1))];
}
template <class B, class P>
TDEV Mat<B> settle(const P (&x)[B::MR], bool on) {
  Mat<B> m;
#pragma unroll
  for (int r = 0; r < B::MR; ++r)
    m.x[r] = on && (B::kFull || (B::row(r) < B::N && B::col(r) < B::N)) ? (typename B::R)x[r]
                                                                             : 0;
  return m;
}
template <class B, class P>
TDEV Vec<B> vsettle(const P (&x)[B::VR], bool on) {
  Vec<B> v;
#pragma unroll
  for (int r = 0; r < B::VR; ++r)
    v.x[r] = on && (B::kFull || B::vrow(r) < B::N) ? (typename B::R)x[r] : 0;
  return v;
}

template <int N>
TDEV int pk(int i, int j) {  // packed upper index
  const int a = i < j ? i : j, b = i < j ? j : i;
  return a * N - (a * (a - 1)) / 2 + (b - a);
}

// Values of scratch (LDS) invert_pivoted needs per wave.
template <class B>
constexpr int kInvScr = B::NODES * (B::N * B::N + B::N);

// Orders this wave's LDS accesses (its lanes run together; the compiler must not reorder them).
TDEV void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// M <- M^{-1} with partial pivoting (the row of largest magnitude, the first one on ties), in
// LDS: the rare path of invert, so it is kept small rather than fast.
template <class B>
TDEV void invert_pivoted(typename B::R (&m)[B::MR], typename B::R* scr) {
  using R = typename B::R;
  constexpr int N = B::N, G = B::LANES, CNT = (N * N + G - 1) / G;
  R* a = scr + B::node() * (N * N + N);
  R* perm = a + N * N;
  const int g = B::sub();
#pragma unroll
  for (int r = 0; r < B::MR; ++r) {
    const int i = B::row(r), j = B::col(r);
    if (i < N && j < N) a[i * N + j] = m[r];
  }
  wave_fence();
  for (int c = 0; c < N; ++c) {
    int p = c;
    R best = fabs(a[c * N + c]);
    for (int i = c + 1; i < N; ++i) {
      const R v = fabs(a[i * N + c]);
      if (v > best) {
        best = v;
        p = i;
      }
    }
    wave_fence();
    if (g == 0) perm[c] = (R)p;
    for (int j = g; j < N; j += G) {
      const R t = a[c * N + j], u = a[p * N + j];
      a[c * N + j] = u;
      a[p * N + j] = t;
    }
    wave_fence();
    const R inv = R(1) / a[c * N + c];
    R t[CNT];
#pragma unroll
    for (int q = 0; q < CNT; ++q) {
      const int e = g + q * G;
      if (e < N * N) {
        const int i = e / N, j = e % N;
        const R f = a[i * N + c], x = a[c * N + j];
        t[q] = i == c ? (j == c ? inv : x * inv)
                      : (j == c ? -f * inv : fma(-f * inv, x, a[e]));
      }
    }
    wave_fence();
#pragma unroll
    for (int q = 0; q < CNT; ++q) {
      const int e = g + q * G;
      if (e < N * N) a[e] = t[q];
    }
    wave_fence();
  }
  for (int c = N - 1; c >= 0; --c) {
    const int p = (int)perm[c];
    for (int i = g; i < N; i += G) {
      const R t = a[i * N + c], u = a[i * N + p];
      a[i * N + c] = u;
      a[i * N + p] = t;
    }
    wave_fence();
  }
#pragma unroll
  for (int r = 0; r < B::MR; ++r) {
    const int i = B::row(r), j = B::col(r);
    m[r] = i < N && j < N ? a[i * N + j] : R(0);
  }
  wave_fence();
}

// M^{-1} (every node of the wave; scr: kInvScr<B> values of LDS of this wave's own).
template <class B>
TDEV Mat<B> inverse(const Mat<B>& M, typename B::R* scr) {
  using R = typename B::R;
  Mat<B> I = M;
  bool good = B::invert(I.x) <= R(kMaxMultiplier);
  // a zero pivot leaves NaNs (which the largest multiplier passes over)
#pragma unroll
  for (int r = 0; r < B::MR; ++r) good = good && I.x[r] == I.x[r];
  if (__ballot(!good) != 0ull) {
    I = M;
    invert_pivoted<B>(I.x, scr);
  }
  return I;
}

// ------------------------------------------------------------------------------------------
// Tuples.  Left operands of a combination hold A - I as it is, right operands hold its transpose:
// that is what the products below read, and a combination returns the transpose.
// ------------------------------------------------------------------------------------------
template <class B>
struct Tup {
  Mat<B> A, C, J;  // A: A - I, or its transpose
  Vec<B> b, e;
};

// A tuple in memory: value q at g[q * st].
template <class R>
struct Ref {
  R* g;
  long st;
};

template <class B>
struct RawTup {
  typename B::Mem A[B::MR], C[B::MR], J[B::MR], b[B::VR], e[B::VR];
};
template <class B, bool TRANS>
TDEV RawTup<B> tfetch(Ref<const typename B::Mem> f) {
  constexpr int N = B::N, NS = N * (N + 1) / 2, oB = N * N, oC = oB + N, oE = oC + NS, oJ = oE + N;
  const long st = f.st;
  RawTup<B> t;
  fetch<B>(t.A, f.g, [=](int i, int j) { return (TRANS ? j * N + i : i * N + j) * st; });
  fetch<B>(t.C, f.g, [=](int i, int j) { return (oC + pk<N>(i, j)) * st; });
  fetch<B>(t.J, f.g, [=](int i, int j) { return (oJ + pk<N>(i, j)) * st; });
  vfetch<B>(t.b, f.g, [=](int i) { return (oB + i) * st; });
  vfetch<B>(t.e, f.g, [=](int i) { return (oE + i) * st; });
  return t;
}
template <class B>
TDEV Tup<B> tsettle(const RawTup<B>& t, bool on) {
  return {settle<B>(t.A, on), settle<B>(t.C, on), settle<B>(t.J, on), vsettle<B>(t.b, on),
          vsettle<B>(t.e, on)};
}

template <class B, class P>
TDEV void tstore_t(bool live, const Tup<B>& t, Ref<P> f) {
  constexpr int N = B::N, NS = N * (N + 1) / 2, oB = N * N, oC = oB + N, oE = oC + NS, oJ = oE + N;
  const long st = f.st;
  mstore<B>(live, t.A, f.g, [=](int i, int j) { return (j * N + i) * st; });
  ustore<B>(live, t.C, f.g, [=](int i, int j) { return (oC + pk<N>(i, j)) * st; });
  ustore<B>(live, t.J, f.g, [=](int i, int j) { return (oJ + pk<N>(i, j)) * st; });
  vstore<B>(live, t.b, f.g, [=](int i) { return (oB + i) * st; });
  vstore<B>(live, t.e, f.g, [=](int i) { return (oE + i) * st; });
}

// Lemma 7 (Sec. IV-A): x1 (x) x2, x1 on the earlier interval (A - I as it is), x2 on the later one
// (A - I transposed); the result's A - I is transposed.  With M = I + C1 J2 and D = M^{-1} C1
// (symmetric), M^{-1} = I - D J2:
//   PJ = J2 (I + Ad1),  Yd = M^{-1} A1 - I = Ad1 - D PJ,
//   Ad = Ad2 + (I + Ad2) Yd,  C = C2 + (I + Ad2) D (I + Ad2)^T,  J = J1 + PJ + Yd^T PJ,
//   b = b2 + (I + Ad2) M^{-1} (b1 + C1 eta2),  eta = eta1 + w + Yd^T w, w = eta2 - J2 b1.
// 8 products, 5 matrix-vector products and the inverse of M^T (= I + J2 C1).  D is the product of
// the inverse with C1, never C1 + (M^{-1} - I) C1: over long intervals or under heavy terminal
// weights D is much smaller than C1, and that difference would leave it an error of eps |C1 J2|
// instead of eps (x of a point mass with Qf of 10^3, 64 blocks: 2e-9 instead of 1e-12).  Ad1 and D are
// small for short blocks, so that Yd keeps its relative precision.
template <class B>
TDEV Tup<B> combine(const Tup<B>& x1, const Tup<B>& x2, typename B::R* scr) {
  const Mat<B> N = inverse<B>(plus_eye<B>(mm0<B>(x2.J, x1.C)), scr);  // M^{-T}
  const Mat<B> D = mm0<B>(N, x1.C);
  const Mat<B> PJ = add<B>(x2.J, mm0<B>(x2.J, x1.A));
  const Mat<B> Yd = mm<B>(x1.A, neg<B>(D), PJ);
  const Mat<B> H = add<B>(D, mm0<B>(D, x2.A));
  const Vec<B> g = mv0<B>(N, add<B>(x1.b, mv0<B>(x1.C, x2.e)));
  const Vec<B> w = add<B>(x2.e, mv0<B>(x2.J, neg<B>(x1.b)));
  Tup<B> o;
  o.A = add<B>(x2.A, mm0<B>(Yd, plus_eye<B>(x2.A)));
  o.C = sym32<B>(add<B>(x2.C, add<B>(H, mm0<B>(x2.A, H))));
  o.J = sym32<B>(add<B>(x1.J, add<B>(PJ, mm0<B>(Yd, PJ))));
  o.b = add<B>(x2.b, add<B>(g, mv0<B>(x2.A, g)));
  o.e = add<B>(x1.e, add<B>(w, mv0<B>(Yd, w)));
  return o;
}

// The value recursion (Lemma 7 with a right operand A = b = C = 0, eta = v, J = S): (S, v) <- a (x)
// (S, v), a's A - I as it is; returns the closed-loop map x -> (I + P) x + q of the interval.
template <class B>
struct Map {
  Mat<B> P;
  Vec<B> q;
};
template <class B>
TDEV Map<B> fold(const Tup<B>& a, Mat<B>& S, Vec<B>& v, typename B::R* scr) {
  const Mat<B> N = inverse<B>(plus_eye<B>(mm0<B>(S, a.C)), scr);  // (I + C S)^{-T}
  const Mat<B> D = mm0<B>(N, a.C);
  const Mat<B> PS = add<B>(S, mm0<B>(S, a.A));
  Map<B> m;
  m.P = mm<B>(a.A, neg<B>(D), PS);
  m.q = mv0<B>(N, add<B>(a.b, mv0<B>(a.C, v)));
  const Vec<B> w = add<B>(v, mv0<B>(S, neg<B>(a.b)));
  S = sym32<B>(add<B>(a.J, add<B>(PS, mm0<B>(m.P, PS))));
  v = add<B>(a.e, add<B>(w, mv0<B>(m.P, w)));
  return m;
}

// acc <- acc o e (e first), acc.P held transposed, e.P as it is.
template <class B>
TDEV void map_after(Map<B>& acc, const Map<B>& e) {
  acc.q = add<B>(add<B>(acc.q, e.q), mv0<B>(acc.P, e.q));
  acc.P = add<B>(acc.P, mm0<B>(e.P, plus_eye<B>(acc.P)));
}

// x <- x + P x + q (P transposed)
template <class B>
TDEV Vec<B> map_apply(const Map<B>& m, const Vec<B>& x) {
  return add<B>(x, add<B>(mv0<B>(m.P, x), m.q));
}

}  // namespace tile
}  // namespace lqt
