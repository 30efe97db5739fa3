// Size of the refinement's work items (Top-K, up to kMaxTopk densities).  Host arithmetic only.
#pragma once

#include <algorithm>
#include <cstdint>

namespace lgreco {

// Tiles per work item.  tiles(l): the layer's tiles, 0 where it takes no part; slots: work items aimed at; most: an
// item's largest size.  An item is part of one layer, so a layer no larger than an even share of the tiles is an item by
// itself; what is left of the slots is dealt to the larger layers, half an item of each for its last, short one, and
// counted: all items are to start at once (where the slots are as many as run at once, one or two in a hundred past
// them cost 3 us of 65 in a compression of 62 layers).  Layers that leave few slots or none would make the few large
// items longer and longer, and a launch is as long as its largest item: past three even shares, items are an even
// share and some start when the first ones end.  Step of 6 densities, us, with the smallest items that fit the
// slots however large / with this rule (and with active / 512): 292 layers of 10 M elements 158 / 124 (146), 77 M
// 321 / 311 (327); 244 layers of 18 M 147 / 141 (164), of 4.5 M 99 / 99 (121); 161 of 26 M 153 / 152 (173), 28 of 5 M
// 81 / 80 (105).  Up to 20 us of the first figures of many layers are the host's, which looked for that size; the
// figures in brackets are of kernels with one launch more.
template <class Tiles>
inline int tiles_per_item(int n_layers, Tiles tiles, int slots, int most) {
    int64_t active = 0;
    for (int l = 0; l < n_layers; ++l) active += tiles(l);
    const int64_t share = std::max<int64_t>(1, (active + slots - 1) / slots);
    if (share >= most) return most;
    int64_t small = 0, large = 0, rest = 0;
    for (int l = 0; l < n_layers; ++l) {
        const int64_t t = tiles(l);
        if (t > share) {
            ++large;
            rest += t;
        } else if (t > 0) {
            ++small;
        }
    }
    const int64_t left = slots - small - large / 2, limit = std::min<int64_t>(most, 3 * share);
    if (left <= 0) return (int)share;
    for (int64_t group = std::max(share, (rest + left / 2) / left); group <= limit; ++group) {
        int64_t items = 0;
        for (int l = 0; l < n_layers; ++l) items += (tiles(l) + (int)group - 1) / (int)group;
        if (items <= slots) return (int)group;
    }
    return (int)share;
}

}  // namespace lgreco
