// Where the low-rank profile packs the matrices it leaves for its later passes.  Host arithmetic only.
#pragma once

#include <cstdint>

namespace lgreco {

// Whether every 32 elements of every row are a whole line of 128 bytes, and a whole number of 16-byte vectors.
inline bool whole_lines(int64_t offset, int32_t cols) { return offset % 32 == 0 && cols % 32 == 0; }
inline bool whole_vectors(int64_t offset, int32_t cols) { return offset % 4 == 0 && cols % 4 == 0; }

// Packs n matrices one behind the other, place(l, at) for each: those of whole lines first, then those of whole vectors, so
// that each keeps what its offset gave it (numel(l) 0: takes no part).  32 matrices of 2048 x 512 behind one of 3 x 4 and a gap
// that restores the offset: a step 308 -> 271 us (behind the small one, off their lines, before).
template <class Offset, class Cols, class Numel, class Place>
inline void pack_matrices(int n, Offset offset, Cols cols, Numel numel, Place place) {
    int64_t at = 0;
    for (int pass = 0; pass < 3; ++pass) {
        for (int l = 0; l < n; ++l) {
            const int kind = whole_lines(offset(l), cols(l)) ? 0 : whole_vectors(offset(l), cols(l)) ? 1 : 2;
            if (kind != pass || numel(l) == 0) continue;
            place(l, at);
            at += numel(l);
        }
    }
}

}  // namespace lgreco
