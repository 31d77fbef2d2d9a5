// The kernels of tile_kernels.hpp for short horizons of the small sizes, where the per-lane path (one
// block or node a lane) leaves most of the device idle and waits for its chains: four lanes times
// four per block or node, 16 times the waves.
#include "lqt_internal.hpp"
#include "tile_host.hpp"

namespace lqt {

using Q4 = tile::Q64<4, double>;

hipError_t tile_build(const KProb& kp, int dtype, void* elts, hipStream_t s) {
  if (kp.nx == 4)
    return dtype == 0 ? tile::launch_build<Q4>(kp, elts, s)
                      : tile::launch_build<tile::Q64<4, float>>(kp, elts, s);
  if (kp.nx == 3)
    return dtype == 0 ? tile::launch_build<tile::Q64<3, double>>(kp, elts, s)
                      : tile::launch_build<tile::Q64<3, float>>(kp, elts, s);
  return hipErrorInvalidValue;
}
namespace {
template <class Mem>
hipError_t nodes_of(const KProb& kp, const GTree& t, const Work& w, hipStream_t s) {
  switch (kp.nx) {
    case 3: return tile::launch_value_tree<tile::Q64<3, Mem>>(kp, t, w, s);
    case 4: return tile::launch_value_tree<tile::Q64<4, Mem>>(kp, t, w, s);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace
hipError_t tile_nodes(const KProb& kp, int dtype, const GTree& t, const Work& w, hipStream_t s) {
  return dtype == 0 ? nodes_of<double>(kp, t, w, s) : nodes_of<float>(kp, t, w, s);
}
hipError_t tile_value(const KProb& kp, const GTree& t, const Work& w, const void* elts, void* S,
                      void* v, hipStream_t s) {
  return tile::launch_value<Q4>(kp, t, w, elts, S, v, false, s);
}
hipError_t tile_scans(const KProb& kp, const GTree& t, const Work& w, const void* elts, void* S,
                      void* v, void* x, void* u, hipStream_t s) {
  return tile::launch_scans<Q4>(kp, t, w, elts, S, v, x, u, s);
}

}  // namespace lqt
