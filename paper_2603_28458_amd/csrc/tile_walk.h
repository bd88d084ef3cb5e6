// The walk of a wave over its tiles in the fused Stage 2: plain arithmetic, so that a host compiler can take the same
// lines.  constexpr functions are callable from host and device code alike.
#pragma once
#include <stdint.h>

namespace hisa {

// May the walks of a query's n_waves waves begin elsewhere than at their first tiles?  Tiles are finished in pairs of
// consecutive ones, so a walk that wraps round has to be even, and all waves have to take part: they then have as
// many tiles each.
constexpr inline __attribute__((always_inline)) bool walk_in_step(int n_tiles, int n_waves) {
  return n_tiles > 0 && n_tiles % (2 * n_waves) == 0;
}

// The tile, of such a wave's, that its walk begins at, `ticks` being what two tiles take: the same for all of them.
constexpr inline __attribute__((always_inline)) int walk_start(int n_tiles, int n_waves, uint32_t now, uint32_t ticks) {
  return (int)(now / ticks % ((uint32_t)n_tiles / (2u * (uint32_t)n_waves))) * 2;
}

// Of a wave's nj tiles, taken from tile j0 on and wrapping round, the one at place j < nj.
constexpr inline __attribute__((always_inline)) int walk_place(int j, int nj, int j0) {
  return j + j0 < nj ? j + j0 : j + j0 - nj;
}

// Tile of the query at place j of the walk of wave `wave` of n_waves (tiles are dealt round robin).  Every lane of the
// wave looks one up, also beyond the walk's end (it gets the wave's first tile), and so does a wave without any tile:
// tile 0, which every query has.  (Its own number may lie past the block list: 2 or 3 blocks of 32 keys, 4 waves.)
constexpr inline __attribute__((always_inline)) int walk_tile(int j, int nj, int j0, int wave, int n_waves) {
  return nj <= 0 ? 0 : wave + n_waves * (j < nj ? walk_place(j, nj, j0) : 0);
}

}  // namespace hisa
