// Launch sequences of the kernels of tile_kernels.hpp, shared by the sizes of the wave path (nx >= 5,
// lqt_wave.hip) and the short horizons of the small ones (lqt_tile.hip).
#pragma once

#include "tile_kernels.hpp"

namespace lqt {
namespace tile {

template <class B>
hipError_t launch_build(const KProb& kp, void* elts, hipStream_t s) {
  using Mem = typename B::Mem;
  const dim3 g((unsigned)tile_build_waves(kp.T, B::NODES), kp.batch);
  if (!kp.F_sampled && !kp.L_sampled && !kp.has_c)
    hipLaunchKernelGGL((kt_build<B, true>), g, dim3(64), 0, s, kp, (Mem*)elts);
  else
    hipLaunchKernelGGL((kt_build<B, false>), g, dim3(64), 0, s, kp, (Mem*)elts);
  return hipGetLastError();
}

inline Stage stage(int c, long n_src, long n_slot, long n_grp) { return {c, n_src, n_slot, n_grp}; }
inline Stage upper(const GTree& t, int j) { return stage(t.c[j], t.src[j], t.slot[j], t.grp[j]); }
template <class B>
Stage bottom(const GTree& t) {
  return stage(t.wc, t.T, t.n1, t.m);
}
// Threads of a stage's workgroups, and their LDS with a dump of DUMP values per slot (and the scratch
// of the pivoted inverse).
template <class B>
dim3 threads(const Stage& st) {
  const long slots = st.n_grp == 1 ? st.n_slot : kGroup<B>;
  return dim3((unsigned)(64 * ((slots + B::NODES - 1) / B::NODES)));
}
template <class B, int DUMP, bool SCR = true>
unsigned lds(const Stage& st) {
  const unsigned waves = threads<B>(st).x / 64;
  return (unsigned)sizeof(typename B::R) * waves * (B::NODES * DUMP + (SCR ? kInvScr<B> : 0));
}

// Arrays of the trees in the workspace (vtup, vval and tmap, tx): 1 sibling records of the bottom
// stage's slots, 2 its groups (if there are several), 3 + 2 j and 4 + 2 j those of upper stage j.
//
// Values at the right ends of the upper stages' nodes (vval[2]) from the nodes (vtup[2]).
template <class B>
hipError_t launch_value_tree(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.G != kGroup<B>) return hipErrorInvalidValue;
  const int nb = kp.batch;
  for (int j = 0; j + 1 < t.up; ++j) {
    const Stage st = upper(t, j);
    hipLaunchKernelGGL((kt_vup<B>), dim3((unsigned)(t.grp[j] * nb)), threads<B>(st),
                       (lds<B, kDumpT<B>>(st)), s, st, 0, nb, 1, (const Mem*)w.vtup[2 + 2 * j],
                       (Mem*)w.vtup[3 + 2 * j], (Mem*)w.vtup[4 + 2 * j]);
  }
  for (int j = t.up - 1; j >= 0; --j) {
    const Stage st = upper(t, j);
    if (j == t.up - 1)
      hipLaunchKernelGGL((kt_vroot<B>), dim3(1, nb), threads<B>(st), (lds<B, kDumpT<B>>(st)), s, kp,
                         st, (const Mem*)w.vtup[2 + 2 * j], (Mem*)w.vtup[3 + 2 * j],
                         (Mem*)w.vval[2 + 2 * j]);
    else
      hipLaunchKernelGGL((kt_vdown<B>), dim3((unsigned)t.grp[j], nb), threads<B>(st),
                         (lds<B, kDumpV<B>>(st)), s, kp, st, (const Mem*)w.vtup[2 + 2 * j],
                         (const Mem*)w.vtup[3 + 2 * j], (const Mem*)w.vval[4 + 2 * j],
                         (Mem*)w.vval[2 + 2 * j]);
  }
  return hipGetLastError();
}

// Values of every boundary; with maps also the bottom groups' maps and, if the workspace has room
// for them, every block's map.
template <class B>
hipError_t launch_value(const KProb& kp, const GTree& t, const Work& w, const void* elts, void* S,
                        void* v, bool maps, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.G != kGroup<B>) return hipErrorInvalidValue;
  const int nb = kp.batch;
  const SpreadGrid g0(t.m * nb, bottom_run<B>(t.wc));
  const Stage s0 = bottom<B>(t);
  if (t.n1 > 1)  // a single slot has no siblings
    hipLaunchKernelGGL((kt_vup<B>), dim3(g0.grid), threads<B>(s0), (lds<B, kDumpT<B>>(s0)), s, s0, 1,
                       nb, g0.run, (const Mem*)elts, (Mem*)w.vtup[1], (Mem*)w.vtup[2]);
  const hipError_t e = launch_value_tree<B>(kp, t, w, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((kt_vbottom<B>), dim3(g0.grid), threads<B>(s0), (lds<B, kDumpV<B>>(s0)), s, kp, s0,
                     g0.run, (const Mem*)elts, (const Mem*)w.vtup[1], (const Mem*)w.vval[2], (Mem*)S,
                     (Mem*)v, (Mem*)(maps ? w.tmap[1] : nullptr),
                     (Mem*)(maps ? w.tmap[2] : nullptr), (Mem*)(maps ? w.bmap : nullptr));
  return hipGetLastError();
}

// States at the left ends of the bottom groups (tx[2]) from their maps (tmap[2]).
template <class B>
hipError_t launch_traj_tree(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.G != kGroup<B>) return hipErrorInvalidValue;
  const int nb = kp.batch;
  for (int j = 0; j + 1 < t.up; ++j) {
    const Stage st = upper(t, j);
    hipLaunchKernelGGL((kt_tup<B>), dim3((unsigned)t.grp[j], nb), threads<B>(st),
                       (lds<B, kDumpV<B>, false>(st)), s, st, (const Mem*)w.tmap[2 + 2 * j],
                       (Mem*)w.tmap[3 + 2 * j], (Mem*)w.tmap[4 + 2 * j]);
  }
  for (int j = t.up - 1; j >= 0; --j) {
    const Stage st = upper(t, j);
    if (j == t.up - 1)
      hipLaunchKernelGGL((kt_troot<B>), dim3(1, nb), threads<B>(st),
                         (lds<B, kDumpV<B> + kDumpX<B>, false>(st)), s, kp, st,
                         (const Mem*)w.tmap[2 + 2 * j], (Mem*)w.tmap[3 + 2 * j],
                         (Mem*)w.tx[2 + 2 * j]);
    else
      hipLaunchKernelGGL((kt_tdown<B>), dim3((unsigned)t.grp[j], nb), threads<B>(st),
                         (lds<B, kDumpX<B>, false>(st)), s, kp, st, (const Mem*)w.tmap[2 + 2 * j],
                         (const Mem*)w.tmap[3 + 2 * j], (const Mem*)w.tx[4 + 2 * j],
                         (Mem*)w.tx[2 + 2 * j]);
  }
  return hipGetLastError();
}

template <class B>
hipError_t launch_tbottom(const KProb& kp, const GTree& t, const Work& w, const void* S,
                          const void* v, void* x, void* u, hipStream_t s) {
  using Mem = typename B::Mem;
  const Stage st = bottom<B>(t);
  hipLaunchKernelGGL((kt_tbottom<B>), dim3((unsigned)t.m, kp.batch), threads<B>(st),
                     (lds<B, kDumpX<B>, false>(st)), s, kp, st, (const Mem*)S, (const Mem*)v,
                     (const Mem*)w.tmap[1], (const Mem*)w.tx[2], (Mem*)x, (Mem*)u,
                     (const Mem*)w.bmap);
  return hipGetLastError();
}

// States at the left ends of the bottom slots (tx[1]) from those of their groups.
template <class B>
hipError_t launch_slot_states(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  using Mem = typename B::Mem;
  const Stage st = stage(1, t.n1, t.n1, t.m);
  hipLaunchKernelGGL((kt_tdown<B>), dim3((unsigned)t.m, kp.batch), threads<B>(st),
                     (lds<B, kDumpX<B>, false>(st)), s, kp, st, (const Mem*)nullptr,
                     (const Mem*)w.tmap[1], (const Mem*)w.tx[2], (Mem*)w.tx[1]);
  return hipGetLastError();
}

// Both scans of a solve whose workspace holds the block maps.
template <class B>
hipError_t launch_scans(const KProb& kp, const GTree& t, const Work& w, const void* elts, void* S,
                        void* v, void* x, void* u, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.m == 1 && t.up == 0) {
    if (t.G != kGroup<B>) return hipErrorInvalidValue;
    const Stage st = bottom<B>(t);
    hipLaunchKernelGGL((kt_small<B>), dim3(1, kp.batch), threads<B>(st), (lds<B, kDumpT<B>>(st)), s, kp,
                       st, (const Mem*)elts, (Mem*)w.vtup[1], (Mem*)w.tmap[1], (Mem*)S, (Mem*)v,
                       (Mem*)x, (Mem*)u, (Mem*)w.bmap);
    return hipGetLastError();
  }
  hipError_t e = launch_value<B>(kp, t, w, elts, S, v, true, s);
  if (e == hipSuccess) e = launch_traj_tree<B>(kp, t, w, s);
  if (e == hipSuccess) e = launch_tbottom<B>(kp, t, w, S, v, x, u, s);
  return e;
}

}  // namespace tile
}  // namespace lqt
