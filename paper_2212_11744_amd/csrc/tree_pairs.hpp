// Which slots of a group a node of a wave combines in a round of the trees in tile_kernels.hpp.
// No device code, so that the rule can be checked on the host.
#pragma once

namespace lqt {
namespace tile {

struct PairPlaces {
  int r;         // the pair's places: r and r + s
  bool any, on;  // a pair in the wave, in the node
};

// Pair q = NODES wave + node of a round of distance s: places 2 s q and 2 s q + s of a group of cnt
// slots (1 <= s < cnt).  The pair is combined into place 2 s q, which other waves must not read in
// that round: a node without a pair takes the operands of its own wave's first pair, whose result is
// stored after every node of the wave has read them, and stores nothing.  A wave without a pair may
// only read (records of the sweep down): place s exists.
constexpr PairPlaces pair_places(int wave, int node, int nodes, int s, int cnt) {
  const int first = 2 * s * wave * nodes, own = first + 2 * s * node;
  const bool any = first + s < cnt, on = own + s < cnt;
  return {on ? own : any ? first : 0, any, on};
}

}  // namespace tile
}  // namespace lqt
