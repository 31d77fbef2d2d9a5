// Indices of the trees in tile_kernels.hpp: which slots of a group a node of a wave combines in a round,
// and which group a workgroup takes.  No device code, so that the rules can be checked on the host.
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

// Workgroups of one launch are dealt to the eight XCDs in turn (workgroup w to XCD w % 8), each with
// its own L2.  Workgroup w takes group `spread(w, run)` of the launch, the groups of all problems in
// order: runs of `run` consecutive groups, whose element columns share 128-byte lines, go to one XCD.
constexpr long spread(long w, int run) {
  const long blk = 8L * run;
  return (w / blk) * blk + (w % 8) * run + (w % blk) / 8;
}
// The grid is a multiple of 8 run, of all problems together (with the groups of every problem rounded
// up, the value scan of 1024 problems of 4 blocks at nx = 16 took 4.8 ms instead of 0.2); fewer groups
// than that are taken in order.
struct SpreadGrid {
  int run;
  unsigned grid;
  constexpr SpreadGrid(long groups, int run_) : run(groups >= 8L * run_ ? run_ : 1), grid(0) {
    const long blk = run > 1 ? 8L * run : 1;
    grid = (unsigned)((groups + blk - 1) / blk * blk);
  }
};

}  // namespace tile
}  // namespace lqt
