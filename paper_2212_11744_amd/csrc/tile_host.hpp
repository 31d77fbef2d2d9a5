// Launch sequences of the kernels of tile_kernels.hpp, shared by the sizes of the wave path (nx >= 5,
// lqt_wave.hip) and the short horizons of the small ones (lqt_tile.hip).
#pragma once

#include "tile_kernels.hpp"

namespace lqt {
namespace tile {

template <class B>
hipError_t launch_build(const KProb& kp, void* elts, hipStream_t s) {
  using Mem = typename B::Mem;
  // waves 8 g + r take the blocks 8 B::NODES g + 8 s + r; none without a block
  const long whole = kp.T / (8L * B::NODES), rest = kp.T % (8L * B::NODES);
  const dim3 g((unsigned)(8 * whole + (rest < 8 ? rest : 8)), kp.batch);
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
template <class B>
constexpr int kGroupThreads = 64 * kGroupWaves<B>;

// Arrays of the trees in the workspace (vtup, vval and tmap, tx): 1 sibling records of the bottom
// stage's slots, 2 its groups (if there are several), 3 + 2 j and 4 + 2 j those of upper stage j.
//
// Values at the right ends of the upper stages' nodes (vval[2]) from the nodes (vtup[2]).
template <class B>
hipError_t launch_value_tree(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.G != kGroup<B>) return hipErrorInvalidValue;
  const int nb = kp.batch;
  const dim3 b(kGroupThreads<B>);
  for (int j = 0; j + 1 < t.up; ++j)
    hipLaunchKernelGGL((kt_vup<B>), dim3((unsigned)(t.grp[j] * nb)), b, 0, s, upper(t, j), 0, nb, 1,
                       (const Mem*)w.vtup[2 + 2 * j], (Mem*)w.vtup[3 + 2 * j],
                       (Mem*)w.vtup[4 + 2 * j]);
  for (int j = t.up - 1; j >= 0; --j) {
    if (j == t.up - 1)
      hipLaunchKernelGGL((kt_vroot<B>), dim3(1, nb), b, 0, s, kp, upper(t, j),
                         (const Mem*)w.vtup[2 + 2 * j], (Mem*)w.vtup[3 + 2 * j],
                         (Mem*)w.vval[2 + 2 * j]);
    else
      hipLaunchKernelGGL((kt_vdown<B>), dim3((unsigned)t.grp[j], nb), b, 0, s, kp, upper(t, j),
                         (const Mem*)w.vtup[2 + 2 * j], (const Mem*)w.vtup[3 + 2 * j],
                         (const Mem*)w.vval[4 + 2 * j], (Mem*)w.vval[2 + 2 * j]);
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
  const dim3 b(kGroupThreads<B>);
  const Stage s0 = bottom<B>(t);
  hipLaunchKernelGGL((kt_vup<B>), dim3(g0.grid), b, 0, s, s0, 1, nb, g0.run, (const Mem*)elts,
                     (Mem*)w.vtup[1], (Mem*)w.vtup[2]);
  const hipError_t e = launch_value_tree<B>(kp, t, w, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((kt_vbottom<B>), dim3(g0.grid), b, 0, s, kp, s0, g0.run, (const Mem*)elts,
                     (const Mem*)w.vtup[1], (const Mem*)w.vval[2], (Mem*)S, (Mem*)v,
                     (Mem*)(maps ? w.tmap[1] : nullptr), (Mem*)(maps ? w.tmap[2] : nullptr),
                     (Mem*)(maps ? w.bmap : nullptr));
  return hipGetLastError();
}

// States at the left ends of the bottom groups (tx[2]) from their maps (tmap[2]).
template <class B>
hipError_t launch_traj_tree(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.G != kGroup<B>) return hipErrorInvalidValue;
  const int nb = kp.batch;
  const dim3 b(kGroupThreads<B>);
  for (int j = 0; j + 1 < t.up; ++j)
    hipLaunchKernelGGL((kt_tup<B>), dim3((unsigned)t.grp[j], nb), b, 0, s, upper(t, j),
                       (const Mem*)w.tmap[2 + 2 * j], (Mem*)w.tmap[3 + 2 * j],
                       (Mem*)w.tmap[4 + 2 * j]);
  for (int j = t.up - 1; j >= 0; --j) {
    if (j == t.up - 1)
      hipLaunchKernelGGL((kt_troot<B>), dim3(1, nb), b, 0, s, kp, upper(t, j),
                         (const Mem*)w.tmap[2 + 2 * j], (Mem*)w.tmap[3 + 2 * j],
                         (Mem*)w.tx[2 + 2 * j]);
    else
      hipLaunchKernelGGL((kt_tdown<B>), dim3((unsigned)t.grp[j], nb), b, 0, s, kp, upper(t, j),
                         (const Mem*)w.tmap[2 + 2 * j], (const Mem*)w.tmap[3 + 2 * j],
                         (const Mem*)w.tx[4 + 2 * j], (Mem*)w.tx[2 + 2 * j]);
  }
  return hipGetLastError();
}

template <class B>
hipError_t launch_tbottom(const KProb& kp, const GTree& t, const Work& w, const void* S,
                          const void* v, void* x, void* u, hipStream_t s) {
  using Mem = typename B::Mem;
  hipLaunchKernelGGL((kt_tbottom<B>), dim3((unsigned)t.m, kp.batch), dim3(kGroupThreads<B>), 0, s, kp,
                     bottom<B>(t), (const Mem*)S, (const Mem*)v, (const Mem*)w.tmap[1],
                     (const Mem*)w.tx[2], (Mem*)x, (Mem*)u, (const Mem*)w.bmap);
  return hipGetLastError();
}

// States at the left ends of the bottom slots (tx[1]) from those of their groups.
template <class B>
hipError_t launch_slot_states(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  using Mem = typename B::Mem;
  hipLaunchKernelGGL((kt_tdown<B>), dim3((unsigned)t.m, kp.batch), dim3(kGroupThreads<B>), 0, s, kp,
                     stage(1, t.n1, t.n1, t.m), (const Mem*)nullptr, (const Mem*)w.tmap[1],
                     (const Mem*)w.tx[2], (Mem*)w.tx[1]);
  return hipGetLastError();
}

// Both scans of a solve whose workspace holds the block maps.
template <class B>
hipError_t launch_scans(const KProb& kp, const GTree& t, const Work& w, const void* elts, void* S,
                        void* v, void* x, void* u, hipStream_t s) {
  using Mem = typename B::Mem;
  if (t.m == 1 && t.up == 0) {
    if (t.G != kGroup<B>) return hipErrorInvalidValue;
    hipLaunchKernelGGL((kt_small<B>), dim3(1, kp.batch), dim3(kGroupThreads<B>), 0, s, kp, bottom<B>(t),
                       (const Mem*)elts, (Mem*)w.vtup[1], (Mem*)w.tmap[1], (Mem*)S, (Mem*)v,
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
