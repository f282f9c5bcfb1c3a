// Load bookkeeping of the tile ring in gram_heads.hip, without device code so
// that a host program can replay it: how many slots the ring has, which loads
// each of the four waves requests for one tile, and how many of a wave's loads
// may still be outstanding when it goes on to the next tile.
#pragma once

namespace sn {

constexpr int kHWaves = 4;  // waves per workgroup of the one-workgroup-per-head Gram form

constexpr int tile_bytes(int dh) { return dh * 128; }  // d_h rows x 128 bytes

// Slots of a ring with vst bytes of start vectors beside each tile.  Two
// workgroups per compute unit with d_h 128, whose registers allow no more; four
// of at most 38 KB below: a workgroup that iterates streams nothing, and the
// others have to fill the memory pipe meanwhile.
constexpr int ring_slots(int dh, int vst) {
  const int fit = (dh == 128 ? 73728 : 38912) / (tile_bytes(dh) + vst);
  return fit < 8 ? fit : 8;
}

// 1 KB load instructions of a tile's rows that wave wv requests: d_h / 8 of
// them, dealt to all waves or, with d_h 16, one each to the first two.
constexpr int tile_loads(int dh, int wv) {
  const int all = dh / 8;
  return all >= kHWaves ? all / kHWaves : wv < all ? 1 : 0;
}

// Rows of start vectors one load instruction covers, at 128 / es columns of
// 4 bytes a row: 64 lanes take 16 bytes each (vec) or, where d or the address
// is not a multiple of that, 4 bytes.
constexpr int vector_rows_per_load(int es, bool vec) {
  const int row = 128 / es * 4, bytes = 64 * (vec ? 16 : 4);
  return bytes / row > 0 ? bytes / row : 1;
}
constexpr int vector_instructions(int es, bool vec, int heads) {
  const int r = vector_rows_per_load(es, vec);
  return (heads + r - 1) / r;
}
// Wave wv requests instructions first, first + 4, ..: waves 2 and 3, which
// multiply them, come first.
constexpr int vector_first(int wv) { return (wv + 2) & (kHWaves - 1); }
constexpr int vector_loads(int instructions, int wv) {
  return (instructions - vector_first(wv) + kHWaves - 1) / kHWaves > 0
             ? (instructions - vector_first(wv) + kHWaves - 1) / kHWaves
             : 0;
}

// Loads of a wave that may be outstanding when its part of tile i has to have
// landed: with `own` loads per tile, those of the slots - 2 tiles requested
// after tile i.
constexpr int outstanding_ahead(int slots, int own) { return (slots - 2) * own; }

}  // namespace sn
