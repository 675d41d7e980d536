// Which contractions the large-tile kernels (tj_gemm_wide.hip) take: plain host arithmetic without HIP, so that it can be compiled and
// checked on its own.  Tiles are 256 x 256; a round is one tile on each of the 256 compute units.
#pragma once
#include <algorithm>

namespace tjplan {

constexpr int kWideTile = 256, kCus = 256, kXcds = 8;

// A hidden layer's weight and input gradient, `tiles` of both (a weight gradient's tile counts once per slice), `k` the contraction of
// the input gradient.  Up to 640 the fixed part of a tile (first loads, result stores) counts too much for one block per unit; two of
// the smaller ones overlap it.  Updates in us, smaller tiles : these, of d-w-w-w: on-policy with 40 actions 128-300 at 32768 rows 301
// : 317, 128-512 at 12288 190 : 202 and at 32768 328 : 343, 128-640 at 15360 258 : 260; 256-704 at 16384 with 17 actions 251 : 246,
// 256-768 260 : 252, 256-1024 336 : 311.  Below five eighths of a round the smaller tiles spread better (256-832 at 4096, 128 tiles,
// double DQN 170 : 178, 256-1024 185 : 192; 136 tiles 183 : 188 and 203 : 201; 160 tiles 188 : 188 and 211 : 203).
inline bool wide_pair_pays(int tiles, int k) { return tiles >= kCus * 5 / 8 && k > 640; }

// A forward pass of tiles_i x tiles_j tiles whose last round is at most half full: columns whose tiles stay whole; those behind them
// are cut into halves.  XCD (column % 8) runs a column's tiles on its 32 units, so the whole columns are as many per XCD as make whole
// rounds there: one too many costs that XCD a round (3 x 96 tiles: 85 whole columns leave five XCDs with 33 tiles; acting on 24576
// observations, 200-768-768-768-18, 150 us with 85, 133 with 80; 200-640-640-640-18 132 and 119).
inline int wide_whole_columns(int tiles_i, int tiles_j)
{
    const int tiles = tiles_i * tiles_j, rest = tiles % kCus;
    if (rest == 0 || rest > kCus / 2) return tiles_j;
    return tiles / kCus * (kCus / kXcds) / tiles_i * kXcds;
}

// A forward pass of tiles_i x tiles_j tiles and contraction `k`.  Up to half a round the tiles are cut into halves, and win over the
// smaller tiles from a quarter of a round on (updates in us, smaller : these; 256-700-700-700-18 at batch 2048 155 : 143, 256-768 at
// 3000 183 : 170, at 4096 183 : 169, 256-1024 at 5000 256 : 221, at 6000 284 : 255); a quarter itself is 128 blocks either way, and
// these cost more (acting on 8192 observations, 128-512-512-512-64, 60 : 65, on 4096 with 1024 units 80 : 89).  Halves have one stage
// of loads in flight, which does not cover the reads of a long contraction from beyond the L2 (the 3136 or 5184 inputs of a pixel
// network's hidden layer; 81 : 105 for a layer of 520 units at batch 2048, updates with 640 units 426 : 446, 1024 units 467 : 485), so
// those wait until the tiles stay whole (1024 units at batch 3000, 144 tiles, 654 : 651; 2048 units, 288 tiles, 793 : 775). Halves
// behind one whole round that are more than a round themselves make it two: short contractions gain too little per tile to pay for
// that (3 x 128 tiles, acting on 32768 observations, 576 units 121 : 130, 640 130 : 137, 768 146 : 158; 4 x 96 tiles of 1024 units,
// whose halves are one round, 202 : 183).
inline bool wide_forward_pays(int tiles_i, int tiles_j, int k)
{
    const int tiles = tiles_i * tiles_j, whole = wide_whole_columns(tiles_i, tiles_j);
    const int halves = (2 * (tiles_j - whole) + kXcds - 1) / kXcds * tiles_i;   // per XCD
    if (k <= 768 && whole > 0 && tiles < 2 * kCus && halves > kCus / kXcds) return false;
    return tiles > (k > 2048 ? kCus / 2 : kCus / 4);
}

// Slices of the first and the last layer's weight gradients, `tiles` of 256 x 128 in all, for up to max_batch rows; the hidden layers
// take s.  A slice per 1024 rows, up to eight down to 256 rows: few tiles are a serial chain as long as their slice
// (256-640-640-640-18 at 1024 rows: 143 us with one slice, 134 with two, 129 with four; 1024 units at 8192 rows with 8, 16 and 21
// slices: 275, 285, 290). Past eight a multiple of eight, where that leaves three quarters of the chip at work or costs a ninth of the
// slices at most: the slice is the fastest index of the blocks, so that the tiles of one slice then run on one of the eight XCDs and
// share its rows in that L2 (updates in us, as many as fit : a multiple of eight; 32768 rows of 256-1024-1024-1024-32 563 : 543 with
// 21 : 16, on-policy 640-1024-1024-1024-18 at 9216 rows 288 : 274 with 9 : 8).  Fewer blocks cost more than that gives (on-policy
// 300-900-900-18 at 32768 rows 344 : 360 with 12 : 8, 200-640-640-640-18 at 14336 221 : 233 with 14 : 8, 128-512-512-512-18 at 14336
// 235 : 246 with 14 : 8).
inline int ends_slices(int tiles, int max_batch, int s)
{
    const int n = std::max(s, std::min(std::max(max_batch / 1024, std::min(8, max_batch / 256)), kCus / tiles));
    const int whole = n - n % kXcds;
    return n > kXcds && (whole * tiles >= kCus * 3 / 4 || 9 * whole >= 8 * n) ? whole : n;
}

}  // namespace tjplan
