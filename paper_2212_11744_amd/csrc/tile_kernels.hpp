// Kernels of the solve for 5 <= nx <= 16 on the register-resident matrices of tile.hpp: element
// build (Theorem 8), value scan and trajectory scan.  A wave works on B::NODES blocks or tree nodes
// side by side and exchanges nothing with other waves; LDS holds only the scratch of the rare
// pivoted inverse.
//
// Trees: node i of level l + 1 is the product of the wcs[l] nodes i wcs[l] .. of level l, combined
// right to left by one slot of a wave; nodes beyond the end of a level read as the identity.  Tree
// nodes are records ([batch][n][record]): tuples (NE values, element order), values (S full, v:
// nx^2 + nx), maps (P = Psi - I, q: nx^2 + nx), states (nx).
#pragma once

#include "tile.hpp"

namespace lqt {
namespace tile {

constexpr int kEltT = kEltTile;

template <int N>
constexpr int kNE = 2 * N * N + 3 * N;
template <int N>
constexpr int kVR = N * N + N;  // value and map records

// Element k of problem p (layout of include/lqt.h).
template <class R, int N>
TDEV Ref<R> elt_ref(R* elts, int p, long k, long T) {
  const long nt = (T + kEltT - 1) / kEltT;
  return {elts + ((p * nt + k / kEltT) * kNE<N>)*kEltT + ((k & 7) << 6) + ((k & 511) >> 3), kEltT};
}

// Waves of one launch are dealt to the eight XCDs in turn (workgroup w to XCD w % 8), each with its
// own L2.  Wave w takes group of slots `spread(w, run)`: runs of `run` consecutive groups, whose
// element columns share 128-byte lines, go to one XCD.  The grid is a multiple of 8 run waves.
TDEV long spread(long w, int run) {
  const long blk = 8L * run;
  return (w / blk) * blk + (w % 8) * run + (w % blk) / 8;
}
inline unsigned spread_grid(long groups, int run) {
  return (unsigned)((groups + 8L * run - 1) / (8L * run) * (8L * run));
}
// Run length for the bottom level: 16 (FP64) or 32 (FP32) element columns to a line, a column per
// 8 blocks, B::NODES nodes of wc blocks per wave.
template <class B>
constexpr int bottom_run(int wc) {
  return (int)(128 / sizeof(typename B::Mem)) * 8 / wc / B::NODES > 0
             ? (int)(128 / sizeof(typename B::Mem)) * 8 / wc / B::NODES
             : 1;
}

// ------------------------------------------------------------------------------------------
// Element build, Theorem 8 (Sec. IV-B) by RK4: with K = G J - F,
//   dAd/ds = (I + Ad) K,  db/ds = -(I + Ad)(G eta + c),  dC/ds = -((I + Ad) Lc)((I + Ad) Lc)^T,
//   deta/ds = K^T eta + J c - Q r,  dJ/ds = -Q + J K - F^T J,
// A held transposed.  The blocks of a wave are 8 apart (k % 8 fixed), so its stores of one value
// fill whole sectors of the element layout, and the waves that complete a line run on one XCD.
// Per stage and node group: 3 products with K, one each for K and the C part (two small ones), 3
// matrix-vector products: bound by the FP64 (FP32) rate of the matrix instruction.
// ------------------------------------------------------------------------------------------
// CC: F, L constant and no drift.
template <class B, bool CC>
__global__ __launch_bounds__(64, 2) void kt_build(const KProb kp, typename B::Mem* __restrict__ elts) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  const int nu = kp.nu, nn = kp.n;
  const long T = kp.T;
  const long k0 = (long)(blockIdx.x >> 3) * (8 * B::NODES) + 8 * B::node() + (blockIdx.x & 7);
  const bool live = k0 < T;
  const long k = live ? k0 : T - 1;
  int p = blockIdx.y;
  long s0 = (long)p * (2L * nn * T + 1), tk = (long)p * (T + 1) + k, kk = k;
  bool sep = false;
  if (kp.seg) {
    p = seg_find(kp.seg, kp.nseg, k);
    sep = k == kp.seg[p + 1] - 1 || k == T - 1;
    if (sep) kk = kp.seg[p];  // a separator integrates its problem's first block, discarded
    s0 = (long)p * (1 - 2L * nn);
    tk = kk;
  }
  const long pf = kp.seg ? p : 0;
  const Mem* t = (const Mem*)kp.t + tk;
  const R h = (t[1] - t[0]) / R(nn);
  const Mem* cs = (const Mem*)kp.consts + (long)p * consts_count(N, nu);
  const long sb = s0 + 2L * nn * kk;  // the block's sample 0
  auto full = [](int i, int j) { return i * N + j; };
  auto vec = [](int i) { return i; };
  const int ktu = (nu + 3) / 4;
  Mat<B> nQ = neg<B>(mload<B>(true, (const Mem*)kp.Q + (long)p * N * N, full));
  // F, G and Lc at a sample
  auto load_F = [&](long j) {
    const bool smp = !CC && kp.F_sampled;
    const Mem* g = smp ? (const Mem*)kp.F + (sb + j) * N * N : (const Mem*)kp.F + pf * N * N;
    return mload<B>(true, g, full);
  };
  auto load_L = [&](long j, Mat<B>& G, Mat<B>& Lc) {
    Lc = mzero<B>();
    if (CC || !kp.L_sampled) {
      G = mload<B>(true, cs + consts_off_G(N, nu), full);
#pragma unroll
      for (int r = 0; r < B::MR; ++r) {
        const int i = B::row(r), l = B::col(r);
        if (i < N && l < nu) Lc.x[r] = cs[consts_off_Lc(N, nu) + i * nu + l];
      }
      return;
    }
    // Lc = L W (n x nu) and its transpose; G = Lc Lc^T
    const Mem* Lj = (const Mem*)kp.L + (sb + j) * N * nu;
    const Mem* Wm = cs + consts_off_W(N, nu);
    Mat<B> LT = mzero<B>();
#pragma unroll
    for (int r = 0; r < B::MR; ++r) {
      const int i = B::row(r), l = B::col(r);
      if (i < N && l < nu)
        for (int q = 0; q < nu; ++q) Lc.x[r] = fma(Lj[i * nu + q], Wm[q * nu + l], Lc.x[r]);
      if (l < N && i < nu)
        for (int q = 0; q < nu; ++q) LT.x[r] = fma(Lj[l * nu + q], Wm[q * nu + i], LT.x[r]);
    }
    G = mm0<B>(LT, LT);
  };
  // the reference and the drift at a sample
  auto load_r = [&](long j) { return vload<B>(true, (const Mem*)kp.r + (sb + j) * N, vec); };
  auto load_c = [&](long j) {
    return !CC && kp.has_c ? vload<B>(true, (const Mem*)kp.c + (sb + j) * N, vec) : vzero<B>();
  };

  Mat<B> yA = mzero<B>(), yJ = mzero<B>(), yC = mzero<B>();
  Vec<B> yb = vzero<B>(), ye = vzero<B>();
  Mat<B> F = neg<B>(load_F(2L * nn)), G, Lc;  // -F
  load_L(2L * nn, G, Lc);
  Vec<B> qr = mv0<B>(nQ, load_r(2L * nn)), cv = load_c(2L * nn);
  // the next sample's F, r and c, loaded a stage or two before they are used
  Mat<B> Fn = F;
  Vec<B> rn, cn_ = cv;
#pragma unroll 1
  for (int m = 0; m < nn; ++m) {
    const long j1 = 2L * (nn - m);
    Mat<B> A1 = plus_eye<B>(yA), sJ = yJ, aA = yA, aJ = yJ;
    Vec<B> se = ye, ae = ye;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const R wk = (st == 0 || st == 3) ? -h / R(6) : -h / R(3);
      const R cn = st == 2 ? -h : -h / R(2);
      if (st == 1 || st == 3) {  // stage 2 reads stage 1's sample
        if (!CC && kp.F_sampled) F = neg<B>(Fn);
        if (!CC && kp.L_sampled) load_L(st == 1 ? j1 - 1 : j1 - 2, G, Lc);
        qr = mv0<B>(nQ, rn);
        cv = cn_;
      }
      if (st == 0 || st == 2) {
        const long j = st == 0 ? j1 - 1 : j1 - 2;
        if (!CC && kp.F_sampled) Fn = load_F(j);
        rn = load_r(j);
        cn_ = load_c(j);
      }
      const Mat<B> K = mm<B>(F, G, sJ);
      const Vec<B> w = mv0<B>(A1, mv<B>(cv, G, se));
      Mat<B> V = mzero<B>(), dC = mzero<B>();
      B::mm(V.x, Lc.x, A1.x, ktu);
      B::template mm<true>(dC.x, V.x, V.x, B::NT, ktu);
      Vec<B> ke = mv<B>(qr, K, se);
      if (!CC && kp.has_c) ke = mv<B>(ke, sJ, cv);
      Mat<B> kJ = nQ;
      B::template mm<true>(kJ.x, sJ.x, K.x);
      B::template mm<true>(kJ.x, F.x, sJ.x);
      B::mirror(kJ.x);
      const Mat<B> kA = mm0<B>(K, A1);
#pragma unroll
      for (int r = 0; r < B::MR; ++r) {
        yC.x[r] = fma(-wk, dC.x[r], yC.x[r]);
        aJ.x[r] = fma(wk, kJ.x[r], aJ.x[r]);
        aA.x[r] = fma(wk, kA.x[r], aA.x[r]);
        if (st < 3) {
          sJ.x[r] = fma(cn, kJ.x[r], yJ.x[r]);
          A1.x[r] = fma(cn, kA.x[r], yA.x[r]) + (mdiag<B>(r) ? R(1) : R(0));
        }
      }
#pragma unroll
      for (int r = 0; r < B::VR; ++r) {
        yb.x[r] = fma(-wk, w.x[r], yb.x[r]);
        ae.x[r] = fma(wk, ke.x[r], ae.x[r]);
        if (st < 3) se.x[r] = fma(cn, ke.x[r], ye.x[r]);
      }
    }
    yA = aA;
    yJ = aJ;
    ye = ae;
  }
  if (sep) {  // A - I = -I, b = x0 of the next problem (0 after the last), C = 0, eta = Qf rf, J = Qf
    const Mem* Qf = (const Mem*)kp.Qf + (long)p * N * N;
    const Mem* rf = (const Mem*)kp.rf + (long)p * N;
    const bool last = p + 1 >= kp.nseg;
#pragma unroll
    for (int r = 0; r < B::MR; ++r) {
      const int i = B::row(r), j = B::col(r);
      yA.x[r] = i == j ? R(-1) : R(0);
      yC.x[r] = R(0);
      if (i < N && j < N) yJ.x[r] = Qf[(i < j ? i : j) * N + (i < j ? j : i)];
    }
#pragma unroll
    for (int r = 0; r < B::VR; ++r) {
      const int i = B::vrow(r);
      R s = R(0);
      if (i < N) {
        for (int j = 0; j < N; ++j) s = fma(Qf[i * N + j], rf[j], s);
        yb.x[r] = last ? R(0) : ((const Mem*)kp.x0)[(long)(p + 1) * N + i];
      }
      ye.x[r] = s;
    }
  }
  const Tup<B> y{yA, yC, yJ, yb, ye};
  tstore_t<B>(live, y, elt_ref<Mem, N>(elts, blockIdx.y, k, T));
}

// ------------------------------------------------------------------------------------------
// Value scan (Theorem 6).
// ------------------------------------------------------------------------------------------
template <class B>
TDEV Ref<typename B::Mem> rec(typename B::Mem* r, int p, long i, long n) {
  return {r + ((long)p * n + i) * kNE<B::N>, 1};
}
template <class B>
TDEV void vrec_store(bool live, const Mat<B>& S, const Vec<B>& v, typename B::Mem* g) {
  constexpr int N = B::N;
  // symmetric: the upper entries, mirrored
  ustore<B>(live, S, g, [](int i, int j) { return i * N + j; });
  ustore<B>(live, S, g, [](int i, int j) { return j * N + i; });
  vstore<B>(live, v, g + N * N, [](int i) { return i; });
}
template <class B>
TDEV void vrec_load(bool live, Mat<B>& S, Vec<B>& v, const typename B::Mem* g) {
  constexpr int N = B::N;
  S = mload<B>(live, g, [](int i, int j) { return i * N + j; });
  v = vload<B>(live, g + N * N, [](int i) { return i; });
}

// Node i of level l + 1: the product of its wc children (elements when src_elts).
template <class B>
TDEV void t_vreduce(typename B::R* scr, int p, long i, int wc, bool src_elts,
                    const typename B::Mem* src, long n_src, typename B::Mem* dst, long n_dst) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  auto ref = [&](long j) -> Ref<const Mem> {
    if (src_elts) {
      const Ref<const Mem> f = elt_ref<const Mem, B::N>(src, p, j, n_src);
      return f;
    }
    return {src + ((long)p * n_src + j) * kNE<B::N>, 1};
  };
  const bool live = i < n_dst;
  const long j0 = i * wc;
  auto ok = [&](long j) { return live && j < n_src; };
  Tup<B> acc = tload<B, true>(ok(j0 + wc - 1), ref(j0 + wc - 1));
  Tup<B> nxt = tload<B, false>(ok(j0 + wc - 2), ref(j0 + wc - 2));
#pragma unroll 1
  for (int c = wc - 2; c >= 0; --c) {
    const Tup<B> x = nxt;
    if (c > 0) nxt = tload<B, false>(ok(j0 + c - 1), ref(j0 + c - 1));
    acc = combine<B>(x, acc, scr);
  }
  tstore_t<B>(live, acc, rec<B>(dst, p, i, n_dst));
}

template <class B>
__global__ __launch_bounds__(64) void kt_vreduce(int wc, int src_elts, int run,
                                                 const typename B::Mem* __restrict__ src, long n_src,
                                                 typename B::Mem* __restrict__ dst, long n_dst) {
  __shared__ typename B::R scr[kInvScr<B>];
  const long g = run > 1 ? spread(blockIdx.x, run) : (long)blockIdx.x;
  if (g * B::NODES >= n_dst) return;
  t_vreduce<B>(scr, blockIdx.y, g * B::NODES + B::node(), wc, src_elts, src, n_src, dst, n_dst);
}

// The terminal value (Sec. IV-D) of problem p: the value at the right end of the tree's root.
template <class B>
TDEV void t_terminal(const KProb& kp, int p, bool live, Mat<B>& S, Vec<B>& v) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  const Mem* Qf = (const Mem*)kp.Qf + (long)p * N * N;
  S = mload<B>(live, Qf, [](int i, int j) { return i < j ? i * N + j : j * N + i; });
  const Mat<B> QT = mload<B>(live, Qf, [](int i, int j) { return j * N + i; });
  v = mv0<B>(QT, vload<B>(live, (const Mem*)kp.rf + (long)p * N, [](int i) { return i; }));
}

// Values at the right ends of the children of node i of level l + 1, from the node's own (root:
// from the terminal value).
template <class B>
TDEV void t_vdown(const KProb& kp, typename B::R* scr, int p, long i, int wc, bool root,
                  const typename B::Mem* tup, long n_child, const typename B::Mem* val_in, long n_par,
                  typename B::Mem* val_out) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  const bool live = i < n_par;
  const long j0 = i * wc;
  auto ok = [&](long j) { return live && j < n_child; };
  auto ref = [&](long j) -> Ref<const Mem> {
    return {tup + ((long)p * n_child + j) * kNE<B::N>, 1};
  };
  Mat<B> S;
  Vec<B> v;
  if (root)
    t_terminal<B>(kp, p, live, S, v);
  else
    vrec_load<B>(live, S, v, val_in + ((long)p * n_par + i) * kVR<B::N>);
  Tup<B> nxt = tload<B, false>(ok(j0 + wc - 1), ref(j0 + wc - 1));
#pragma unroll 1
  for (int c = wc - 1; c >= 0; --c) {
    const long j = j0 + c;
    vrec_store<B>(ok(j), S, v, val_out + ((long)p * n_child + j) * kVR<B::N>);
    if (c == 0) break;
    const Tup<B> a = nxt;
    if (c > 1) nxt = tload<B, false>(ok(j - 1), ref(j - 1));
    fold<B>(a, S, v, scr);
  }
}

template <class B>
__global__ __launch_bounds__(64) void kt_vdown(const KProb kp, int wc,
                                               const typename B::Mem* __restrict__ tup, long n_child,
                                               const typename B::Mem* __restrict__ val_in, long n_par,
                                               typename B::Mem* __restrict__ val_out) {
  __shared__ typename B::R scr[kInvScr<B>];
  t_vdown<B>(kp, scr, blockIdx.y, (long)blockIdx.x * B::NODES + B::node(), wc, false, tup, n_child,
             val_in, n_par, val_out);
}

// The upper levels of a value tree in one workgroup per problem: levels l0 .. L reduced (the root,
// above level L, needs no product of its own), then the terminal value carried back down to the
// values at level l0.
constexpr int kMidWaves = 8;
struct MidArgs {
  int l0 = 0, L = 0;
  int wcs[kTreeMaxLevels + 2] = {};
  long n[kTreeMaxLevels + 2] = {};
  void* tup[kTreeMaxLevels + 2] = {};  // tuples (value) or maps (trajectory) of level l
  void* val[kTreeMaxLevels + 2] = {};  // values or states of level l
};

template <class B>
__global__ __launch_bounds__(64 * kMidWaves) void kt_vmid(const KProb kp, const MidArgs a) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  __shared__ R scr_all[kMidWaves][kInvScr<B>];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), p = blockIdx.y;
  R* scr = scr_all[w];
  for (int l = a.l0; l < a.L; ++l) {
    for (long g = w; g * B::NODES < a.n[l + 1]; g += kMidWaves)
      t_vreduce<B>(scr, p, g * B::NODES + B::node(), a.wcs[l], false, (const Mem*)a.tup[l], a.n[l],
                   (Mem*)a.tup[l + 1], a.n[l + 1]);
    __syncthreads();
  }
  for (int l = a.L; l >= a.l0; --l) {
    for (long g = w; g * B::NODES < a.n[l + 1]; g += kMidWaves)
      t_vdown<B>(kp, scr, p, g * B::NODES + B::node(), a.wcs[l], l == a.L, (const Mem*)a.tup[l],
                 a.n[l], (const Mem*)a.val[l + 1], a.n[l + 1], (Mem*)a.val[l]);
    __syncthreads();
  }
}

// Values of every block from the value at the right end of each level-1 node; the composed
// closed-loop map of the node's blocks (maps1) and every block's own map (bmaps) when given.
template <class B>
__global__ __launch_bounds__(64) void kt_vbottom(const KProb kp, int wc, int run,
                                                 const typename B::Mem* __restrict__ elts,
                                                 const typename B::Mem* __restrict__ val1, long n1,
                                                 typename B::Mem* __restrict__ Sout,
                                                 typename B::Mem* __restrict__ vout,
                                                 typename B::Mem* __restrict__ maps1,
                                                 typename B::Mem* __restrict__ bmaps) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  __shared__ R scr[kInvScr<B>];
  const long g = run > 1 ? spread(blockIdx.x, run) : (long)blockIdx.x;
  if (g * B::NODES >= n1) return;
  const int p = blockIdx.y;
  const long T = kp.T, i = g * B::NODES + B::node();
  const bool live = i < n1;
  const long j0 = i * wc;
  auto ok = [&](long k) { return live && k < T; };
  auto ref = [&](long k) -> Ref<const Mem> { return elt_ref<const Mem, N>(elts, p, k, T); };
  Mem* Sp = Sout + (long)p * (T + 1) * N * N;
  Mem* vp = vout + (long)p * (T + 1) * N;
  auto put = [&](bool on, long k, const Mat<B>& S, const Vec<B>& v) {
    ustore<B>(on, S, Sp + k * N * N, [](int a, int b) { return a * N + b; });
    ustore<B>(on, S, Sp + k * N * N, [](int a, int b) { return b * N + a; });
    vstore<B>(on, v, vp + k * N, [](int a) { return a; });
  };
  Mat<B> S;
  Vec<B> v;
  vrec_load<B>(live, S, v, val1 + ((long)p * n1 + i) * kVR<N>);
  if (!kp.seg) put(live && j0 + wc >= T, T, S, v);
  Map<B> acc{mzero<B>(), vzero<B>()};  // P transposed
  Tup<B> nxt = tload<B, false>(ok(j0 + wc - 1), ref(j0 + wc - 1));
#pragma unroll 1
  for (int c = wc - 1; c >= 0; --c) {
    const long k = j0 + c;
    const Tup<B> a = nxt;
    if (c > 0) nxt = tload<B, false>(ok(k - 1), ref(k - 1));
    const Map<B> m = fold<B>(a, S, v, scr);
    put(ok(k), k, S, v);
    if (bmaps) {
      Mem* b = bmaps + ((long)p * T + k) * kVR<N>;
      mstore<B>(ok(k), m.P, b, [](int x, int y) { return x * N + y; });
      vstore<B>(ok(k), m.q, b + N * N, [](int x) { return x; });
    }
    if (maps1) map_after<B>(acc, m);
  }
  if (maps1) {
    Mem* b = maps1 + ((long)p * n1 + i) * kVR<N>;
    mstore<B>(live, acc.P, b, [](int x, int y) { return y * N + x; });
    vstore<B>(live, acc.q, b + N * N, [](int x) { return x; });
  }
}

// ------------------------------------------------------------------------------------------
// Trajectory (Method 1, Sec. IV-E): maps composed up a tree, states carried down.
// ------------------------------------------------------------------------------------------
template <class B, bool TRANS>
TDEV Map<B> map_load(bool live, const typename B::Mem* g) {
  constexpr int N = B::N;
  return {mload<B>(live, g, [](int i, int j) { return TRANS ? j * N + i : i * N + j; }),
          vload<B>(live, g + N * N, [](int i) { return i; })};
}

template <class B>
TDEV void t_treduce(int p, long i, int wc, const typename B::Mem* src, long n_src,
                    typename B::Mem* dst, long n_dst) {
  constexpr int N = B::N;
  const bool live = i < n_dst;
  const long j0 = i * wc;
  auto at = [&](long j) { return src + ((long)p * n_src + j) * kVR<N>; };
  auto ok = [&](long j) { return live && j < n_src; };
  Map<B> acc = map_load<B, true>(ok(j0 + wc - 1), at(j0 + wc - 1));
#pragma unroll 1
  for (int c = wc - 2; c >= 0; --c) map_after<B>(acc, map_load<B, false>(ok(j0 + c), at(j0 + c)));
  typename B::Mem* b = dst + ((long)p * n_dst + i) * kVR<N>;
  mstore<B>(live, acc.P, b, [](int x, int y) { return y * N + x; });
  vstore<B>(live, acc.q, b + N * N, [](int x) { return x; });
}

template <class B>
__global__ __launch_bounds__(64) void kt_treduce(int wc, const typename B::Mem* __restrict__ src,
                                                 long n_src, typename B::Mem* __restrict__ dst,
                                                 long n_dst) {
  t_treduce<B>(blockIdx.y, (long)blockIdx.x * B::NODES + B::node(), wc, src, n_src, dst, n_dst);
}

template <class B>
TDEV void t_tdown(int p, long i, int wc, const typename B::Mem* maps, long n_child,
                  const typename B::Mem* x_in, long n_par, typename B::Mem* x_out) {
  constexpr int N = B::N;
  const bool live = i < n_par;
  const long j0 = i * wc;
  auto ok = [&](long j) { return live && j < n_child; };
  Vec<B> x = vload<B>(live, x_in + ((long)p * n_par + i) * N, [](int q) { return q; });
#pragma unroll 1
  for (int c = 0; c < wc; ++c) {
    const long j = j0 + c;
    vstore<B>(ok(j), x, x_out + ((long)p * n_child + j) * N, [](int q) { return q; });
    if (c + 1 < wc)
      x = map_apply<B>(map_load<B, true>(ok(j), maps + ((long)p * n_child + j) * kVR<N>), x);
  }
}

template <class B>
__global__ __launch_bounds__(64) void kt_tdown(int wc, const typename B::Mem* __restrict__ maps,
                                               long n_child,
                                               const typename B::Mem* __restrict__ x_in, long n_par,
                                               typename B::Mem* __restrict__ x_out) {
  t_tdown<B>(blockIdx.y, (long)blockIdx.x * B::NODES + B::node(), wc, maps, n_child, x_in, n_par,
             x_out);
}

// The upper levels of the trajectory tree in one workgroup per problem (see kt_vmid).
template <class B>
__global__ __launch_bounds__(64 * kMidWaves) void kt_tmid(const KProb kp, const MidArgs a) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), p = blockIdx.y;
  for (int l = a.l0; l < a.L; ++l) {
    for (long g = w; g * B::NODES < a.n[l + 1]; g += kMidWaves)
      t_treduce<B>(p, g * B::NODES + B::node(), a.wcs[l], (const Mem*)a.tup[l], a.n[l],
                   (Mem*)a.tup[l + 1], a.n[l + 1]);
    __syncthreads();
  }
  for (int l = a.L; l >= a.l0; --l) {
    // the one node above the top level starts at x0
    const Mem* xin = l == a.L ? (const Mem*)kp.x0 : (const Mem*)a.val[l + 1];
    for (long g = w; g * B::NODES < a.n[l + 1]; g += kMidWaves)
      t_tdown<B>(p, g * B::NODES + B::node(), a.wcs[l], (const Mem*)a.tup[l], a.n[l], xin,
                 a.n[l + 1], (Mem*)a.val[l]);
    __syncthreads();
  }
}

// x_k and u_k = -R^{-1} L(t_k)^T (S_k x_k - v_k) of every block of a level-1 node, from the block
// maps the value sweep kept.
template <class B>
__global__ __launch_bounds__(64) void kt_tbottom(const KProb kp, int wc,
                                                 const typename B::Mem* __restrict__ Sg,
                                                 const typename B::Mem* __restrict__ vg,
                                                 const typename B::Mem* __restrict__ x1, long n1,
                                                 typename B::Mem* __restrict__ xout,
                                                 typename B::Mem* __restrict__ uout,
                                                 const typename B::Mem* __restrict__ bmaps) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  const int p = blockIdx.y, nu = kp.nu;
  const long T = kp.T, i = (long)blockIdx.x * B::NODES + B::node();
  const bool live = i < n1;
  const long j0 = i * wc;
  auto ok = [&](long k) { return live && k < T; };
  const Mem* Sp = Sg + (long)p * (T + 1) * N * N;
  const Mem* vp = vg + (long)p * (T + 1) * N;
  Mem* xp = xout + (long)p * (T + 1) * N;
  Mem* up = uout ? uout + (long)p * (T + 1) * nu : nullptr;
  auto full = [](int a, int b) { return a * N + b; };
  auto vec = [](int a) { return a; };
  // gain transposed (n x nu) of the problem owning boundary k
  auto gain = [&](bool on, long k) {
    const int pk_ = kp.seg ? seg_find(kp.seg, kp.nseg, on ? k : 0) : p;
    const Mem* cs = (const Mem*)kp.consts + (long)pk_ * consts_count(N, nu);
    const long s = (kp.seg ? (long)pk_ * (1 - 2L * kp.n) : (long)p * (2L * kp.n * T + 1)) +
                   2L * kp.n * k;
    Mat<B> K = mzero<B>();
#pragma unroll
    for (int r = 0; r < B::MR; ++r) {
      const int a = B::row(r), l = B::col(r);
      if (!on || a >= N || l >= nu) continue;
      if (kp.L_sampled) {
        const Mem* Lk = (const Mem*)kp.L + s * N * nu;
        const Mem* Ri = cs + consts_off_Rinv(N, nu);
        for (int q = 0; q < nu; ++q) K.x[r] = fma(Ri[l * nu + q], Lk[a * nu + q], K.x[r]);
      } else {
        K.x[r] = cs[consts_off_Kc(N, nu) + l * N + a];
      }
    }
    return K;
  };
  const bool per_k = kp.L_sampled || kp.seg;
  Mat<B> Kc = mzero<B>();
  if (up && !per_k) Kc = gain(live, 0);
  auto control = [&](bool on, long k, const Vec<B>& x) {
    if (!up) return;
    if (per_k) Kc = gain(on, k);
    const Mat<B> S = mload<B>(on, Sp + k * N * N, full);
    const Vec<B> gv = mv<B>(neg<B>(vload<B>(on, vp + k * N, vec)), S, x);
    const Vec<B> u = neg<B>(mv0<B>(Kc, gv));
    if (B::rep()) {
#pragma unroll
      for (int r = 0; r < B::VR; ++r)
        if (on && B::vrow(r) < nu) up[k * nu + B::vrow(r)] = (Mem)u.x[r];
    }
  };
  Vec<B> x = vload<B>(live, x1 + ((long)p * n1 + i) * N, vec);
#pragma unroll 1
  for (int c = 0; c < wc; ++c) {
    const long k = j0 + c;
    const Map<B> m = map_load<B, true>(ok(k), bmaps + ((long)p * T + k) * kVR<N>);
    vstore<B>(ok(k), x, xp + k * N, vec);
    control(ok(k), k, x);
    x = map_apply<B>(m, x);
  }
  if (!kp.seg) {
    const bool end = live && j0 + wc >= T;
    vstore<B>(end, x, xp + T * N, vec);
    control(end, T, x);
  }
}

}  // namespace tile
}  // namespace lqt
