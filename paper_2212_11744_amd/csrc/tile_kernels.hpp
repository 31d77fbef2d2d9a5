// Kernels on the register-resident matrices of tile.hpp: element build (Theorem 8), value scan and
// trajectory scan of 5 <= nx <= 16 and of short horizons at nx = 3, 4, and the value tree over the tiles of
// the per-lane path's three-launch scan.  A wave works on B::NODES blocks or tree nodes side by side.
// The build exchanges nothing with other waves; the trees exchange dumps of registers in LDS, beside the
// scratch of the rare pivoted inverse.
//
// Trees: a slot of a wave takes c consecutive nodes of a level one after the other, and the slots of
// a workgroup (a group) are combined pairwise in LDS, so that a stage of the tree reduces c G
// nodes to one in one launch and 2 c + 2 log2 G steps up and down: a launch costs more than two
// or three steps, a step more than its arithmetic (chains of dependent matrix products), and the
// stages of a tree (T = 2^14 blocks at nx = 16: 3; nx <= 8: 2 up to 2^15) are what a short or
// middle horizon waits for.  What a sweep down needs of a stage are the left-to-right sibling
// products of its slots, one record per slot.  Records ([batch][n][record]): tuples (NE values,
// element order), values (S full, v: nx^2 + nx), maps (P = Psi - I, q: nx^2 + nx), states (nx).
#pragma once

#include "tile.hpp"
#include "tree_pairs.hpp"

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

// Problem and group of a workgroup of a launch over the groups of all problems (tree_pairs.hpp).
struct Place {
  int p;
  long g;
  bool live;
  TDEV Place(long n_grp, int batch, int run) {
    const unsigned w = (unsigned)(run > 1 ? spread(blockIdx.x, run) : (long)blockIdx.x);
    p = (int)(w / (unsigned)n_grp);
    g = w - (unsigned)p * (unsigned)n_grp;
    live = p < batch;
  }
};
// Waves and slots of a group, and the run length of the bottom stage: 16 (FP64) or 32 (FP32)
// element columns to a line, a column per 8 blocks, wc blocks per slot.
// One wave a SIMD (the steps of a group are serial, and two waves of matrix instructions on a SIMD
// wait for each other); two for nx <= 4, whose steps are short.
template <class B>
constexpr int kGroupWaves = B::N <= 4 ? 8 : 4;
template <class B>
constexpr int kGroup = kGroupWaves<B> * B::NODES;
template <class B>
constexpr int bottom_run(int wc) {
  const int run = (int)(128 / sizeof(typename B::Mem)) * 8 / (wc * kGroup<B>);
  return run > 0 ? run : 1;
}

// ------------------------------------------------------------------------------------------
// Element build, Theorem 8 (Sec. IV-B) by RK4: with K = G J - F,
//   dAd/ds = (I + Ad) K,  db/ds = -(I + Ad)(G eta + c),  dC/ds = -((I + Ad) Lc)((I + Ad) Lc)^T,
//   deta/ds = K^T eta + J c - Q r,  dJ/ds = -Q + J K - F^T J,
// A held transposed.  The blocks of a wave are 8 apart (k % 8 fixed), so its stores of one value
// fill whole sectors of the element layout, and the waves that complete a line run on one XCD; a
// horizon too short for that is taken in order, which fills its waves.
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
  const long w = blockIdx.x;
  const long k0 = T < 8 * B::NODES ? w * B::NODES + B::node()
                                   : (w >> 3) * (8 * B::NODES) + 8 * B::node() + (w & 7);
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
template <class P>
TDEV Ref<P> rec(P* r, int size, long i) {
  return {r + i * size, 1};
}
template <class B, class P>
TDEV void vrec_store(bool live, const Mat<B>& S, const Vec<B>& v, P* g) {
  constexpr int N = B::N;
  // symmetric: the upper entries, mirrored
  ustore<B>(live, S, g, [](int i, int j) { return i * N + j; });
  ustore<B>(live, S, g, [](int i, int j) { return j * N + i; });
  vstore<B>(live, v, g + N * N, [](int i) { return i; });
}
template <class B, class P>
TDEV void vrec_load(bool live, Mat<B>& S, Vec<B>& v, const P* g) {
  constexpr int N = B::N;
  S = mload<B>(live, g, [](int i, int j) { return i * N + j; });
  v = vload<B>(live, g + N * N, [](int i) { return i; });
}

// One stage of a tree: slot i takes the nodes i c .. of n_src, group g the slots g G ...
struct Stage {
  int c = 1;
  long n_src = 0, n_slot = 0, n_grp = 0;
};
// The slots of group g, and this wave's slot of them.
template <class B>
struct Here {
  int w, p;    // wave, problem
  long g, i;   // group, slot
  int cnt;     // slots of the group
  int loc;     // i within the group
  bool live;
  TDEV Here(const Stage& st, long g_, int p_) : p(p_), g(g_) {
    w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    cnt = (int)min((long)kGroup<B>, st.n_slot - g * kGroup<B>);
    loc = w * B::NODES + B::node();
    i = g * kGroup<B> + loc;
    live = loc < cnt;
  }
};

// Barrier of the workgroup for what is exchanged in LDS: loads from and stores to memory stay in
// flight (__syncthreads would wait for them: 7 instead of 3 us a round at nx = 16).
TDEV void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What the waves of a group exchange in LDS: dumps of a node's registers, so that neither side has
// entries to mask or offsets to compute.
template <class B>
constexpr int kDumpT = (3 * B::MR + 2 * B::VR) * B::LANES;
template <class B>
constexpr int kDumpV = (B::MR + B::VR) * B::LANES;  // values and maps
template <class B>
constexpr int kDumpX = B::VR * B::LANES;
// The LDS of a launch: a dump per slot that the workgroup's waves hold, then the waves' scratch of the
// pivoted inverse.  Sized by the host, with as many waves as a single small group needs (a full group's
// 41 KB would let three workgroups of one busy wave each onto a CU).
extern __shared__ double lds_raw[];
TDEV int lds_waves() { return (int)(blockDim.x >> 6); }
template <class B, int DUMP>
TDEV auto lds_slots() {
  return (typename B::R(*)[DUMP])lds_raw;
}
template <class B, int DUMP>
TDEV typename B::R* lds_scratch(int w) {
  return (typename B::R*)lds_raw + lds_waves() * B::NODES * DUMP + w * kInvScr<B>;
}
template <class B, int CNT>
TDEV void put(const typename B::R (&x)[CNT], typename B::R* g) {
#pragma unroll
  for (int r = 0; r < CNT; ++r) g[r * B::LANES] = x[r];
}
template <class B, int CNT>
TDEV void get(typename B::R (&x)[CNT], const typename B::R* g) {
#pragma unroll
  for (int r = 0; r < CNT; ++r) x[r] = g[r * B::LANES];
}
template <class B>
TDEV void get_t(Mat<B>& m, const typename B::R* node) {  // transposed
#pragma unroll
  for (int r = 0; r < B::MR; ++r) m.x[r] = node[B::tpos(r)];
}
template <class B>
TDEV void dump(const Tup<B>& t, typename B::R* node) {
  typename B::R* g = node + B::sub();
  constexpr int M = B::MR * B::LANES;
  put<B>(t.A.x, g);
  put<B>(t.C.x, g + M);
  put<B>(t.J.x, g + 2 * M);
  put<B>(t.b.x, g + 3 * M);
  put<B>(t.e.x, g + 3 * M + kDumpX<B>);
}
template <class B, bool TRANS>  // TRANS: A transposed against what was dumped
TDEV Tup<B> undump(const typename B::R* node) {
  const typename B::R* g = node + B::sub();
  constexpr int M = B::MR * B::LANES;
  Tup<B> t;
  if (TRANS)
    get_t<B>(t.A, node);
  else
    get<B>(t.A.x, g);
  get<B>(t.C.x, g + M);
  get<B>(t.J.x, g + 2 * M);
  get<B>(t.b.x, g + 3 * M);
  get<B>(t.e.x, g + 3 * M + kDumpX<B>);
  return t;
}
template <class B>
TDEV void vdump(const Mat<B>& S, const Vec<B>& v, typename B::R* node) {
  put<B>(S.x, node + B::sub());
  put<B>(v.x, node + B::MR * B::LANES + B::sub());
}
template <class B, bool TRANS = false>
TDEV void vundump(Mat<B>& S, Vec<B>& v, const typename B::R* node) {
  if (TRANS)
    get_t<B>(S, node);
  else
    get<B>(S.x, node + B::sub());
  get<B>(v.x, node + B::MR * B::LANES + B::sub());
}

// Product of the c nodes of slot i, the right one first; transposed (see Tup).
template <class B>
TDEV Tup<B> t_serial(const Here<B>& h, const Stage& st, bool src_elts, const typename B::Mem* src,
                     typename B::R* scr) {
  using Mem = typename B::Mem;
  const int c = st.c;
  const long j0 = h.i * c;
  auto ok = [&](int q) { return h.live && j0 + q < st.n_src; };
  auto ref = [&](int q) -> Ref<const Mem> {
    const long j = min(j0 + q, st.n_src - 1);
    if (src_elts) return elt_ref<const Mem, B::N>(src, h.p, j, st.n_src);
    return rec(src, kNE<B::N>, (long)h.p * st.n_src + j);
  };
  const RawTup<B> last = tfetch<B, true>(ref(c - 1));
  RawTup<B> nxt;
  if (c > 1) nxt = tfetch<B, false>(ref(c - 2));
  Tup<B> acc = tsettle<B>(last, ok(c - 1));
#pragma unroll 1
  for (int q = c - 2; q >= 0; --q) {
    const Tup<B> x = tsettle<B>(nxt, ok(q));
    if (q > 0) nxt = tfetch<B, false>(ref(q - 1));
    acc = combine<B>(x, acc, scr);
  }
  return acc;
}

// This node's pair in a round of distance s (tree_pairs.hpp).
template <class B>
struct Pair : PairPlaces {
  TDEV Pair(const Here<B>& h, int s) : PairPlaces(pair_places(h.w, B::node(), B::NODES, s, h.cnt)) {}
};

// Group product of the slots' products.  Slot loc sits at place cnt - 1 - loc of ex (the last slot
// at place 0): a round of distance s combines places 2 s q (right) and 2 s q + s (left) into the
// former, whose product until then, the right sibling of place 2 s q + s, is kept in
// sib[2 s q + s] for the sweep down.  The root has no use for the product of all of its slots.
template <class B>
TDEV void t_vup(const Here<B>& h, typename B::R (*ex)[kDumpT<B>], typename B::Mem* sib, bool root,
                typename B::R* scr) {
#pragma unroll 1
  for (int s = 1; s < h.cnt; s *= 2) {
    lds_sync();
    const Pair<B> q(h, s);
    if (!q.any) continue;
    Tup<B> acc = undump<B, false>(ex[q.r]);
    tstore_t<B>(q.on, acc, rec(sib, kNE<B::N>, q.r + s));
    if (root && 2 * s >= h.cnt) continue;
    acc = combine<B>(undump<B, true>(ex[q.r + s]), acc, scr);
    if (q.on) dump<B>(acc, ex[q.r]);
  }
  __syncthreads();
}

// The value at the right end of every slot (val, by place) from that at place 0: the reverse rounds.
template <class B>
TDEV void t_vdown(const Here<B>& h, typename B::R (*val)[kDumpV<B>], const typename B::Mem* sib,
                  typename B::R* scr) {
  int s = 1;
  while (2 * s < h.cnt) s *= 2;
  auto load = [&](int s_) {
    const Pair<B> q(h, s_);
    return tfetch<B, false>(rec(sib, kNE<B::N>, q.r + s_));
  };
  if (h.cnt > 1) {
    RawTup<B> nxt = load(s);
#pragma unroll 1
    for (; s >= 1; s /= 2) {
      const Tup<B> a = tsettle<B>(nxt, true);
      if (s > 1) nxt = load(s / 2);
      lds_sync();
      const Pair<B> q(h, s);
      if (!q.any) continue;
      Mat<B> S;
      Vec<B> v;
      vundump<B>(S, v, val[q.r]);
      fold<B>(a, S, v, scr);
      if (q.on) vdump<B>(S, v, val[q.r + s]);
    }
  }
  lds_sync();
}

// The terminal value (Sec. IV-D) of problem p: the value at the right end of the tree's root.
template <class B>
TDEV void t_terminal(const KProb& kp, int p, bool live, Mat<B>& S, Vec<B>& v) {
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  const Mem* Qf = (const Mem*)kp.Qf + (long)p * N * N;
  S = mload<B>(live, Qf, [](int i, int j) { return i < j ? i * N + j : j * N + i; });
  const Mat<B> QT = mload<B>(live, Qf, [](int i, int j) { return j * N + i; });
  v = mv0<B>(QT, vload<B>(live, (const Mem*)kp.rf + (long)p * N, [](int i) { return i; }));
}

// Place 0 of a group's values: the terminal value (root) or val_in, the group's own.
template <class B>
TDEV void t_vtop(const KProb& kp, const Here<B>& h, bool root, const typename B::Mem* val_in,
                 typename B::R (*val)[kDumpV<B>]) {
  if (h.w) return;
  const bool on = B::node() == 0;
  Mat<B> S;
  Vec<B> v;
  if (root)
    t_terminal<B>(kp, h.p, on, S, v);
  else
    vrec_load<B>(on, S, v, val_in);
  if (on) vdump<B>(S, v, val[0]);
}

// Values at the right ends of the c nodes of a slot from the slot's.
template <class B>
TDEV void t_vspread(const Here<B>& h, const Stage& st, const typename B::Mem* src,
                    const typename B::R (*val)[kDumpV<B>], typename B::Mem* val_out,
                    typename B::R* scr) {
  using Mem = typename B::Mem;
  if (h.w * B::NODES >= h.cnt) return;
  const int c = st.c;
  const long j0 = h.i * c;
  auto ok = [&](long j) { return h.live && j < st.n_src; };
  auto ref = [&](long j) -> Ref<const Mem> {
    return rec(src, kNE<B::N>, (long)h.p * st.n_src + min(j, st.n_src - 1));
  };
  RawTup<B> nxt;
  if (c > 1) nxt = tfetch<B, false>(ref(j0 + c - 1));
  Mat<B> S;
  Vec<B> v;
  vundump<B>(S, v, val[h.live ? h.cnt - 1 - h.loc : 0]);
#pragma unroll 1
  for (int q = c - 1; q >= 0; --q) {
    const long j = j0 + q;
    vrec_store<B>(ok(j), S, v, val_out + ((long)h.p * st.n_src + j) * kVR<B::N>);
    if (q == 0) break;
    const Tup<B> a = tsettle<B>(nxt, ok(j));
    if (q > 1) nxt = tfetch<B, false>(ref(j - 1));
    fold<B>(a, S, v, scr);
  }
}

// Reduction of a stage: the groups' products and their slots' sibling records (of a single group the
// records alone).
template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_vup(const Stage st, int src_elts, int batch,
                                                           int run,
                                                           const typename B::Mem* __restrict__ src,
                                                           typename B::Mem* __restrict__ sib,
                                                           typename B::Mem* __restrict__ grp) {
  constexpr int NE = kNE<B::N>;
  auto ex = lds_slots<B, kDumpT<B>>();
  const Place at(st.n_grp, batch, run);
  if (!at.live) return;
  const long g = at.g;
  const Here<B> h(st, g, at.p);
  typename B::R* scr = lds_scratch<B, kDumpT<B>>(h.w);
  if (h.w * B::NODES < h.cnt) {
    const Tup<B> acc = t_serial<B>(h, st, src_elts, src, scr);
    if (h.live) dump<B>(acc, ex[h.cnt - 1 - h.loc]);
  }
  const bool root = st.n_grp == 1;
  t_vup<B>(h, ex, sib + ((long)h.p * st.n_slot + g * kGroup<B>)*NE, root, scr);
  if (h.w == 0 && !root)
    tstore_t<B>(B::node() == 0, undump<B, false>(ex[0]), rec(grp, NE, (long)h.p * st.n_grp + g));
}

// The root stage: up, and down to the values of its nodes.
template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_vroot(const KProb kp, const Stage st,
                                                             const typename B::Mem* src,
                                                             typename B::Mem* sib,
                                                             typename B::Mem* __restrict__ val_out) {
  constexpr int NE = kNE<B::N>;
  auto ex = lds_slots<B, kDumpT<B>>();
  const Here<B> h(st, 0, blockIdx.y);
  typename B::R* scr = lds_scratch<B, kDumpT<B>>(h.w);
  if (h.w * B::NODES < h.cnt) {
    const Tup<B> acc = t_serial<B>(h, st, false, src, scr);
    if (h.live) dump<B>(acc, ex[h.cnt - 1 - h.loc]);
  }
  typename B::Mem* sb = sib + (long)h.p * st.n_slot * NE;
  t_vup<B>(h, ex, sb, true, scr);
  auto val = (typename B::R(*)[kDumpV<B>])ex[0];
  t_vtop<B>(kp, h, true, sb, val);
  t_vdown<B>(h, val, sb, scr);
  t_vspread<B>(h, st, src, val, val_out, scr);
}

// Values of a stage's nodes from those of its groups.
template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_vdown(
    const KProb kp, const Stage st, const typename B::Mem* __restrict__ src,
    const typename B::Mem* __restrict__ sib, const typename B::Mem* __restrict__ val_in,
    typename B::Mem* __restrict__ val_out) {
  auto val = lds_slots<B, kDumpV<B>>();
  const Here<B> h(st, blockIdx.x, blockIdx.y);
  typename B::R* scr = lds_scratch<B, kDumpV<B>>(h.w);
  t_vtop<B>(kp, h, st.n_grp == 1, val_in + ((long)h.p * st.n_grp + h.g) * kVR<B::N>, val);
  t_vdown<B>(h, val, sib + ((long)h.p * st.n_slot + h.g * kGroup<B>)*kNE<B::N>, scr);
  t_vspread<B>(h, st, src, val, val_out, scr);
}

// ------------------------------------------------------------------------------------------
// Trajectory (Method 1, Sec. IV-E): maps composed up a tree, states carried down.  Here the places
// of a group are its slots in time order.
// ------------------------------------------------------------------------------------------
template <class B>
struct RawMap {
  typename B::Mem P[B::MR], q[B::VR];
};
template <class B, bool TRANS>
TDEV RawMap<B> map_fetch(const typename B::Mem* g) {
  constexpr int N = B::N;
  RawMap<B> m;
  fetch<B>(m.P, g, [](int i, int j) { return TRANS ? j * N + i : i * N + j; });
  vfetch<B>(m.q, g + N * N, [](int i) { return i; });
  return m;
}
template <class B>
TDEV Map<B> map_settle(const RawMap<B>& m, bool on) {
  return {settle<B>(m.P, on), vsettle<B>(m.q, on)};
}
template <class B, class P>  // m.P transposed
TDEV void map_store_t(bool live, const Map<B>& m, P* g) {
  constexpr int N = B::N;
  mstore<B>(live, m.P, g, [](int i, int j) { return j * N + i; });
  vstore<B>(live, m.q, g + N * N, [](int i) { return i; });
}

// Values of every block of a slot from the one at its right end, and the composed closed-loop map
// of the blocks (transposed) when asked for; every block's own map in bmaps when given.
template <class B>
TDEV Map<B> t_vbottom(const KProb& kp, const Here<B>& h, int wc, const typename B::Mem* elts,
                      const typename B::R (*val)[kDumpV<B>], typename B::Mem* Sout,
                      typename B::Mem* vout, typename B::Mem* bmaps, bool compose,
                      typename B::R* scr) {
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  const long T = kp.T;
  const int p = h.p;
  const bool live = h.live;
  const long j0 = h.i * wc;
  auto ok = [&](long k) { return live && k < T; };
  auto ref = [&](long k) -> Ref<const Mem> { return elt_ref<const Mem, N>(elts, p, min(k, T - 1), T); };
  Mem* Sp = Sout + (long)p * (T + 1) * N * N;
  Mem* vp = vout + (long)p * (T + 1) * N;
  auto put = [&](bool on, long k, const Mat<B>& S, const Vec<B>& v) {
    vstore<B>(on, v, vp + k * N, [](int a) { return a; });
    ustore<B>(on, S, Sp + k * N * N, [](int a, int b) { return a * N + b; });
    ustore<B>(on, S, Sp + k * N * N, [](int a, int b) { return b * N + a; });
  };
  Mat<B> S;
  Vec<B> v;
  vundump<B>(S, v, val[live ? h.cnt - 1 - h.loc : 0]);
  if (compose) lds_sync();  // the maps take the place of the values
  Map<B> acc{mzero<B>(), vzero<B>()};  // P transposed
  if (h.w * B::NODES >= h.cnt) return acc;
  RawTup<B> nxt = tfetch<B, false>(ref(j0 + wc - 1));
  if (!kp.seg) put(live && j0 + wc >= T, T, S, v);
#pragma unroll 1
  for (int c = wc - 1; c >= 0; --c) {
    const long k = j0 + c;
    const Tup<B> a = tsettle<B>(nxt, ok(k));
    if (c > 0) nxt = tfetch<B, false>(ref(k - 1));
    const Map<B> m = fold<B>(a, S, v, scr);
    put(ok(k), k, S, v);
    if (bmaps) {
      Mem* b = bmaps + ((long)p * T + k) * kVR<N>;
      mstore<B>(ok(k), m.P, b, [](int x, int y) { return x * N + y; });
      vstore<B>(ok(k), m.q, b + N * N, [](int x) { return x; });
    }
    if (compose) map_after<B>(acc, m);
  }
  return acc;
}

// Group map: a round of distance s composes places 2 s q (earlier) and 2 s q + s into the former,
// whose map until then, the left sibling of place 2 s q + s, is kept in sib[2 s q + s].  The dumps
// hold P transposed.
template <class B>
TDEV void t_tup(const Here<B>& h, typename B::R (*ex)[kDumpV<B>], typename B::Mem* sib, bool root) {
  constexpr int VR = kVR<B::N>, N = B::N;
#pragma unroll 1
  for (int s = 1; s < h.cnt; s *= 2) {
    lds_sync();
    const Pair<B> q(h, s);
    if (!q.any) continue;
    Map<B> m, acc;
    vundump<B, true>(m.P, m.q, ex[q.r]);
    typename B::Mem* g = sib + (long)(q.r + s) * VR;
    mstore<B>(q.on, m.P, g, [](int i, int j) { return i * N + j; });
    vstore<B>(q.on, m.q, g + N * N, [](int i) { return i; });
    if (root && 2 * s >= h.cnt) continue;
    vundump<B>(acc.P, acc.q, ex[q.r + s]);
    map_after<B>(acc, m);
    if (q.on) vdump<B>(acc.P, acc.q, ex[q.r]);
  }
  __syncthreads();
}
template <class B>
TDEV void t_tgroup(const typename B::R (*ex)[kDumpV<B>], typename B::Mem* grp) {
  Map<B> m;
  vundump<B>(m.P, m.q, ex[0]);
  map_store_t<B>(B::node() == 0, m, grp);
}

// The state at the left end of every slot from that at place 0.
template <class B>
TDEV void t_tdown(const Here<B>& h, typename B::R (*xs)[kDumpX<B>], const typename B::Mem* sib) {
  int s = 1;
  while (2 * s < h.cnt) s *= 2;
  auto load = [&](int s_) {
    const Pair<B> q(h, s_);
    return map_fetch<B, true>(sib + (long)(q.r + s_) * kVR<B::N>);
  };
  if (h.cnt > 1) {
    RawMap<B> nxt = load(s);
#pragma unroll 1
    for (; s >= 1; s /= 2) {
      const Map<B> m = map_settle<B>(nxt, true);
      if (s > 1) nxt = load(s / 2);
      lds_sync();
      const Pair<B> q(h, s);
      if (!q.any) continue;
      Vec<B> x;
      get<B>(x.x, xs[q.r] + B::sub());
      x = map_apply<B>(m, x);
      if (q.on) put<B>(x.x, xs[q.r + s] + B::sub());
    }
  }
  lds_sync();
}

// Place 0 of a group's states: x0 (root) or x_in, the group's own.
template <class B>
TDEV void t_ttop(const KProb& kp, const Here<B>& h, bool root, const typename B::Mem* x_in,
                 typename B::R (*xs)[kDumpX<B>]) {
  if (h.w) return;
  const bool on = B::node() == 0;
  const typename B::Mem* g = root ? (const typename B::Mem*)kp.x0 + (long)h.p * B::N : x_in;
  const Vec<B> x = vload<B>(on, g, [](int i) { return i; });
  if (on) put<B>(x.x, xs[0] + B::sub());
}

// Composed map of a slot's c nodes into its place.
template <class B>
TDEV void t_tserial(const Here<B>& h, const Stage& st, const typename B::Mem* src,
                    typename B::R (*ex)[kDumpV<B>]) {
  const int c = st.c;
  const long j0 = h.i * c;
  auto at = [&](int q) {
    return src + ((long)h.p * st.n_src + min(j0 + q, st.n_src - 1)) * kVR<B::N>;
  };
  auto ok = [&](int q) { return h.live && j0 + q < st.n_src; };
  const RawMap<B> last = map_fetch<B, true>(at(c - 1));
  RawMap<B> nxt;
  if (c > 1) nxt = map_fetch<B, false>(at(c - 2));
  Map<B> acc = map_settle<B>(last, ok(c - 1));
#pragma unroll 1
  for (int q = c - 2; q >= 0; --q) {
    const Map<B> m = map_settle<B>(nxt, ok(q));
    if (q > 0) nxt = map_fetch<B, false>(at(q - 1));
    map_after<B>(acc, m);
  }
  if (h.live) vdump<B>(acc.P, acc.q, ex[h.loc]);
}

// States at the left ends of the c nodes of a slot from the slot's.
template <class B>
TDEV void t_tspread(const Here<B>& h, const Stage& st, const typename B::Mem* src,
                    const typename B::R (*xs)[kDumpX<B>], typename B::Mem* x_out) {
  constexpr int N = B::N;
  const int c = st.c;
  const long j0 = h.i * c;
  auto at = [&](int q) {
    return src + ((long)h.p * st.n_src + min(j0 + q, st.n_src - 1)) * kVR<N>;
  };
  Vec<B> x;
  get<B>(x.x, xs[h.live ? h.loc : 0] + B::sub());
  RawMap<B> nxt;
  if (c > 1) nxt = map_fetch<B, true>(at(0));
#pragma unroll 1
  for (int q = 0; q < c; ++q) {
    const bool on = h.live && j0 + q < st.n_src;
    vstore<B>(on, x, x_out + ((long)h.p * st.n_src + j0 + q) * N, [](int i) { return i; });
    if (q + 1 == c) break;
    const Map<B> m = map_settle<B>(nxt, on);
    if (q + 2 < c) nxt = map_fetch<B, true>(at(q + 1));
    x = map_apply<B>(m, x);
  }
}

template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_tup(const Stage st,
                                                           const typename B::Mem* __restrict__ src,
                                                           typename B::Mem* __restrict__ sib,
                                                           typename B::Mem* __restrict__ grp) {
  constexpr int VR = kVR<B::N>;
  auto ex = lds_slots<B, kDumpV<B>>();
  const Here<B> h(st, blockIdx.x, blockIdx.y);
  t_tserial<B>(h, st, src, ex);
  t_tup<B>(h, ex, sib + ((long)h.p * st.n_slot + h.g * kGroup<B>)*VR, false);
  if (h.w == 0) t_tgroup<B>(ex, grp + ((long)h.p * st.n_grp + h.g) * VR);
}

template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_troot(const KProb kp, const Stage st,
                                                             const typename B::Mem* src,
                                                             typename B::Mem* sib,
                                                             typename B::Mem* __restrict__ x_out) {
  constexpr int VR = kVR<B::N>;
  auto ex = lds_slots<B, kDumpV<B>>();
  auto xs = (typename B::R(*)[kDumpX<B>])ex[lds_waves() * B::NODES];  // after the maps
  const Here<B> h(st, 0, blockIdx.y);
  typename B::Mem* sb = sib + (long)h.p * st.n_slot * VR;
  t_tserial<B>(h, st, src, ex);
  t_tup<B>(h, ex, sb, true);
  t_ttop<B>(kp, h, true, sb, xs);
  t_tdown<B>(h, xs, sb);
  t_tspread<B>(h, st, src, xs, x_out);
}

template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_tdown(
    const KProb kp, const Stage st, const typename B::Mem* __restrict__ src,
    const typename B::Mem* __restrict__ sib, const typename B::Mem* __restrict__ x_in,
    typename B::Mem* __restrict__ x_out) {
  auto xs = lds_slots<B, kDumpX<B>>();
  const Here<B> h(st, blockIdx.x, blockIdx.y);
  t_ttop<B>(kp, h, st.n_grp == 1, x_in + ((long)h.p * st.n_grp + h.g) * B::N, xs);
  t_tdown<B>(h, xs, sib + ((long)h.p * st.n_slot + h.g * kGroup<B>)*kVR<B::N>);
  t_tspread<B>(h, st, src, xs, x_out);
}

// The bottom stage down: values of every block, and with msib the sibling maps of the slots and, of
// several groups, each group's map (grp).
template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_vbottom(
    const KProb kp, const Stage st, int run, const typename B::Mem* __restrict__ elts,
    const typename B::Mem* __restrict__ sib, const typename B::Mem* __restrict__ val_in,
    typename B::Mem* __restrict__ Sout, typename B::Mem* __restrict__ vout,
    typename B::Mem* __restrict__ msib, typename B::Mem* __restrict__ grp,
    typename B::Mem* __restrict__ bmaps) {
  constexpr int VR = kVR<B::N>;
  auto val = lds_slots<B, kDumpV<B>>();
  const Place at(st.n_grp, kp.batch, run);
  if (!at.live) return;
  const long g = at.g;
  const Here<B> h(st, g, at.p);
  typename B::R* scr = lds_scratch<B, kDumpV<B>>(h.w);
  t_vtop<B>(kp, h, st.n_grp == 1, val_in + ((long)h.p * st.n_grp + h.g) * kVR<B::N>, val);
  t_vdown<B>(h, val, sib + ((long)h.p * st.n_slot + g * kGroup<B>)*kNE<B::N>, scr);
  const Map<B> acc = t_vbottom<B>(kp, h, st.c, elts, val, Sout, vout, bmaps, msib != nullptr, scr);
  if (!msib) return;
  if (h.live) vdump<B>(acc.P, acc.q, val[h.loc]);
  const bool root = st.n_grp == 1;
  t_tup<B>(h, val, msib + ((long)h.p * st.n_slot + g * kGroup<B>)*VR, root);
  if (h.w == 0 && !root) t_tgroup<B>(val, grp + ((long)h.p * st.n_grp + g) * VR);
}

// x_k and u_k = -R^{-1} L(t_k)^T (S_k x_k - v_k) of every block of a slot, from the block maps the
// value sweep kept.
template <class B>
TDEV void t_tbottom(const KProb& kp, const Here<B>& h, int wc, const typename B::Mem* Sg,
                    const typename B::Mem* vg, const typename B::R (*xs)[kDumpX<B>],
                    typename B::Mem* xout, typename B::Mem* uout, const typename B::Mem* bmaps) {
  using R = typename B::R;
  using Mem = typename B::Mem;
  constexpr int N = B::N;
  const int nu = kp.nu;
  const long T = kp.T;
  const int p = h.p;
  const bool live = h.live;
  const long j0 = h.i * wc;
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
  // S, v and the map of a block, loaded a block ahead
  struct Raw {
    typename B::Mem S[B::MR], v[B::VR];
    RawMap<B> m;
  };
  auto load = [&](long k_) {
    const long k = min(k_, T - 1);
    Raw w;
    if (up) {
      fetch<B>(w.S, Sp + k * N * N, full);
      vfetch<B>(w.v, vp + k * N, vec);
    }
    w.m = map_fetch<B, true>(bmaps + ((long)p * T + k) * kVR<N>);
    return w;
  };
  auto control = [&](bool on, long k, const Mat<B>& S, const Vec<B>& v, const Vec<B>& x) {
    if (per_k) Kc = gain(on, k);
    const Vec<B> gv = mv<B>(neg<B>(v), S, x);
    const Vec<B> u = neg<B>(mv0<B>(Kc, gv));
    if (B::rep()) {
#pragma unroll
      for (int r = 0; r < B::VR; ++r)
        if (on && B::vrow(r) < nu) up[k * nu + B::vrow(r)] = (Mem)u.x[r];
    }
  };
  Vec<B> x;
  get<B>(x.x, xs[live ? h.loc : 0] + B::sub());
  Raw nxt = load(j0);
#pragma unroll 1
  for (int c = 0; c < wc; ++c) {
    const long k = j0 + c;
    const Raw w = nxt;
    if (c + 1 < wc) nxt = load(k + 1);
    vstore<B>(ok(k), x, xp + k * N, vec);
    if (up) control(ok(k), k, settle<B>(w.S, ok(k)), vsettle<B>(w.v, ok(k)), x);
    x = map_apply<B>(map_settle<B>(w.m, ok(k)), x);
  }
  if (!kp.seg) {
    const bool end = live && j0 + wc >= T;
    vstore<B>(end, x, xp + T * N, vec);
    if (up)
      control(end, T, mload<B>(end, Sp + T * N * N, full), vload<B>(end, vp + T * N, vec), x);
  }
}

template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_tbottom(
    const KProb kp, const Stage st, const typename B::Mem* __restrict__ Sg,
    const typename B::Mem* __restrict__ vg, const typename B::Mem* __restrict__ msib,
    const typename B::Mem* __restrict__ x_in, typename B::Mem* __restrict__ xout,
    typename B::Mem* __restrict__ uout, const typename B::Mem* __restrict__ bmaps) {
  auto xs = lds_slots<B, kDumpX<B>>();
  const Here<B> h(st, blockIdx.x, blockIdx.y);
  t_ttop<B>(kp, h, st.n_grp == 1, x_in + ((long)h.p * st.n_grp + h.g) * B::N, xs);
  t_tdown<B>(h, xs, msib + ((long)h.p * st.n_slot + h.g * kGroup<B>)*kVR<B::N>);
  if (h.w * B::NODES < h.cnt) t_tbottom<B>(kp, h, st.c, Sg, vg, xs, xout, uout, bmaps);
}

// Both scans of a horizon of one group in one launch.
template <class B>
__global__ __launch_bounds__(64 * kGroupWaves<B>, 2) void kt_small(
    const KProb kp, const Stage st, const typename B::Mem* __restrict__ elts, typename B::Mem* sib,
    typename B::Mem* msib, typename B::Mem* Sout, typename B::Mem* vout,
    typename B::Mem* __restrict__ xout, typename B::Mem* __restrict__ uout, typename B::Mem* bmaps) {
  constexpr int NE = kNE<B::N>, VR = kVR<B::N>;
  auto ex = lds_slots<B, kDumpT<B>>();
  const Here<B> h(st, 0, blockIdx.y);
  typename B::R* scr = lds_scratch<B, kDumpT<B>>(h.w);
  typename B::Mem* sb = sib + (long)h.p * st.n_slot * NE;
  typename B::Mem* mb = msib + (long)h.p * st.n_slot * VR;
  const bool any = h.w * B::NODES < h.cnt;
  if (any) {
    const Tup<B> acc = t_serial<B>(h, st, true, elts, scr);
    if (h.live) dump<B>(acc, ex[h.cnt - 1 - h.loc]);
  }
  t_vup<B>(h, ex, sb, true, scr);
  auto val = (typename B::R(*)[kDumpV<B>])ex[0];
  t_vtop<B>(kp, h, true, sb, val);
  t_vdown<B>(h, val, sb, scr);
  const Map<B> acc = t_vbottom<B>(kp, h, st.c, elts, val, Sout, vout, bmaps, true, scr);
  if (h.live) vdump<B>(acc.P, acc.q, val[h.loc]);
  t_tup<B>(h, val, mb, true);
  auto xs = (typename B::R(*)[kDumpX<B>])ex[0];
  t_ttop<B>(kp, h, true, mb, xs);
  t_tdown<B>(h, xs, mb);
  if (any) t_tbottom<B>(kp, h, st.c, Sout, vout, xs, xout, uout, bmaps);
}

}  // namespace tile
}  // namespace lqt
