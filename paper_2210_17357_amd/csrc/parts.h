// How layers are cut into tiles, and how many workgroups a tile's elements are dealt to (quantization compressor and receiver).
// Host arithmetic only.
#pragma once

#include <cstdint>

namespace lgreco {

constexpr int kTile = 32768;       // largest streaming tile in elements (256 buckets of 128); a position inside a
                                   // tile fits 15 bits (the Top-K candidate records rely on it)
constexpr int kTileMin = 8192;     // smallest: small problems get smaller tiles so that the launch still fills the chip
// Tile size: halved from kTile while there would be fewer than kTilesFill tiles (small problems
// still fill the chip); in calls with Top-K layers, from kTile / 2 to kTileMin while there would be fewer than half as
// many.  A tile of Top-K work ends with a flush of its
// histogram, whose adding up in memory (0.3 ns for every line of it and tile) the kernel waits for, and every
// later kernel has a record and a chain of loads per tile; a tile without ends with a few numbers, and short workgroups suit it.  Measured on 355 M elements: 10.8 k tiles of 32768
// took 4 % off the streaming kernels against 5.4 k of 65536; 21.7 k of 16384 cost the histogram
// pass more than it gained.  Steps, us, with kTileMin / twice that: Top-K of 17 M elements 129 / 125, 22 M 143 / 136, 28 M
// 172 / 162, 31 M 172 / 161, both families 157 / 154, 171 / 168, 200 / 191, 199 / 189, 100 densities of 26 M 181 / 170, quantization alone of 20 M
// 110 / 116, 27 M 134 / 139; with kTile / 2 / kTile: Top-K of 54 M 237 / 237, 66 M 273 / 274, both families 273 / 277, 310 / 318.
// Compressions of Top-K layers, 20 M elements 114 / 110, 26 M 95.5 / 96.4: as the profile in front of them, whose cut they share.
constexpr int kTilesFill = 2048;

// Tile size of a table of `total` elements.
inline int tile_size(int64_t total, bool topk) {
    int tile = kTile;
    while (tile > kTileMin && total / tile < (topk && tile < kTile ? kTilesFill / 2 : kTilesFill)) tile /= 2;
    return tile;
}

// The power of two of workgroups each of `n_tiles` tiles gets: tiles of `tile` elements, `total` in all, are to be cut into parts
// of `part` elements.  Every tile gets the same number, so that a workgroup finds its tile by a shift: those of a tile
// that is not full find nothing to do, at 0.2 to 0.4 ns each, where 4096 elements take 8 ns.  Where there would be more of them
// than one for 4096 elements (and a microsecond's), parts are longer, up to a whole tile: 50000 layers of 1500 elements
// compressed in 2322 us with parts of 512 elements and received in 1331 with 2048, now 395 and 291; 20000 of 1000 beside one of 67 M
// 1050 and 522, now 323 and 197; 600 of 150000 235 and 91 as before.
inline int part_shift(int64_t n_tiles, int64_t total, int64_t tile, int64_t part) {
    int s = 0;
    while ((tile >> s) > part) ++s;
    const auto bearable = [&](int q) {
        const int64_t groups = n_tiles << q, used = total / (tile >> q);
        return groups - used <= total / 4096 + 4096 && groups <= (int64_t)1 << 23;     // (a launch takes 2^32 threads)
    };
    while (s > 0 && !bearable(s)) --s;
    return s;
}

}  // namespace lgreco
