// C entry points over the tile workspace's state
// (paper_1910_13874_amd/csrc/tile_state.h) for the CPU tests, which build this
// file with g++.  No device code is involved.
#include "tile_state.h"

using ged::TileState;

extern "C" {
void *ts_new() { return new TileState; }
void ts_free(void *p) { delete static_cast<TileState *>(p); }
int ts_zero(void *p) { return static_cast<TileState *>(p)->zero(); }
void ts_copy_replaced(void *p) { static_cast<TileState *>(p)->copy_replaced(); }
// bit 0: counts, bit 1: level 2, bit 2: the 16-bit copy
int ts_fit(void *p, unsigned long bytes, int gathered16) {
  const TileState::Fill f = static_cast<TileState *>(p)->fit(bytes, gathered16 != 0);
  return (f.counts ? 1 : 0) | (f.level2 ? 2 : 0) | (f.copy ? 4 : 0);
}
void ts_begin(void *p, int gathered16) { static_cast<TileState *>(p)->begin(gathered16 != 0); }
void ts_end(void *p, int gathered16) { static_cast<TileState *>(p)->end(gathered16 != 0); }
}
