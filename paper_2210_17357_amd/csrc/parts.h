// How many workgroups a tile's elements are dealt to (quantization compressor and receiver).  Host arithmetic only.
#pragma once

#include <cstdint>

namespace lgreco {

// The power of two of workgroups each of `n_tiles` tiles gets: tiles of `tile` elements, `total` in all, are to be cut into parts
// of `part` elements.  Every tile gets the same number, so that a workgroup finds its tile by a shift: those of a tile
// that is not full find nothing to do, at 0.2 to 0.4 ns each, where 4096 elements take 8 ns.  Where there would be more of them
// than one for 4096 elements (and a microsecond's), parts are longer, up to a whole tile: 50000 layers of 1500 elements
// compressed in 2322 us with parts of 512 elements and received in 1331 with 2048, now 410 and 286; 20000 of 1000 beside one of 67 M
// 1050 and 522, now 334 and 194; 600 of 150000 235 and 91 as before.
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
