// Layer-wise Top-K: radix-histogram threshold search, dropped-energy profile for several
// densities at once, and threshold-select compaction.  gfx950 / wave64.
//
// Magnitudes are compared as the fp32 bit pattern with the sign cleared (31 bits); the "coarse
// key" of an element is the top 12 bits (exponent + 4 mantissa bits).  Per call:
//   1. sample: coarse histogram of up to 8192 elements of every layer, 16384 in calls of 2^26 elements and more.
//      From it a cautious lower bound `lo` of the coarse key of the k-th largest magnitude is predicted for every layer (the
//      largest k asked for, with a margin).
//   2. main pass, ONE read of the data (fused into the quantization profile kernel when both
//      families are profiled): exact coarse histogram of every element (LDS per tile, integer
//      atomics to global); elements with key >= lo ("candidates", 10-20 % of the data) are
//      written, as bit patterns, to the tile's own slice of a candidate buffer in ballot-prefix
//      order; the energy of everything below lo is summed in registers.
//   3. refinement.  Every workgroup first scans its layer's exact histogram for itself (more than kMaxTopk densities: a
//      kernel in front does): for every requested k the coarse bin holding the k-th largest
//      magnitude and how many entries to take inside it.  If the prediction was too high for a
//      layer (lo above its lowest threshold bin) that layer alone is collected again with the
//      exact bound, so the result never depends on the sample.  Then, on the candidates only: energy below
//      each threshold bin (fp64, fixed order) and histogram of the next 10 bits inside each threshold bin.
//   4. Profile: the pick kernel sums those per layer and k, finds the sub-bin and the dropped energy; the last 9 bits
//      only for a sub-bin whose share of it is not provably negligible (see topk_pick_a_kernel).  Compression: the next
//      kernel's workgroups find the sub-bin themselves and add up the last 9 bits inside it, and the kernel that counts
//      kept entries finds in those the exact k-th magnitude and the number of equal magnitudes to keep.
//      Histogram bins carry their energy as integers (entries of one coarse bin share the
//      exponent: x^2 = m^2 2^(2(E-150)), m the 24-bit significand; sum (m^2 >> 16) is exact), so
//      nothing depends on the order of atomics.
// Compression then counts kept entries per tile from the candidates, and the last kernel sums the counts before
// its own tiles and writes values and indices in ascending index order (equal magnitudes: lowest indices first).
// A compression queued right behind a profile of the same data takes the candidates from that
// profile, whose main pass then also records where each candidate is (16 bits: position in the
// tile, sign), and reads the data no second time.
#include <cstdlib>
#include <cstring>

#include "internal.h"
#include "reduce_dev.h"
#include "topk_dev.h"
#include "work_items.h"

namespace lgreco {

struct TopkSel {
    uint32_t k, tbin, need, list;   // need: entries to take from the threshold bin; list: its number among the layer's
                                    // distinct threshold bins
    uint32_t bin_a, need_a;         // refinement level A (bits 18..9)
    uint32_t thr, ties_keep;        // exact threshold pattern; equal entries kept (compress)
};
struct TopkLayer {
    int64_t cand_base;              // first slot of this layer's region in the candidate buffer
    TopkSel sel[kMaxTopk];
};
// The same for a profile of more than kMaxTopk densities.  The requested k do not increase with j, so
// the densities whose threshold lies in one coarse bin are consecutive: list i holds the densities
// [first[i], first[i + 1]).
struct TopkMany {
    uint32_t nlists, recollect;
    uint32_t bin[LGRECO_MAX_CANDS];      // threshold bin of every list, ascending
    uint32_t first[LGRECO_MAX_CANDS + 1];
    uint32_t need[LGRECO_MAX_CANDS];     // per density: entries to take from its threshold bin
};
constexpr int kManyChunk = 8;       // lists one refinement workgroup works on at a time
constexpr int kManySplit = 4;       // refinement workgroups that share a work item's lists
constexpr int kManySlots = 32;      // workgroups that share a layer's lists in the pick
constexpr int kRefTiles = 16;       // largest tiles per refinement workgroup (fewer elements never: with
                                    // smaller tiles a workgroup takes proportionally more of them)
constexpr int kRefThreads = 1024;
constexpr int kRefSlots = 512;      // refinement workgroups the chip runs at a time (256 CUs x 2)
constexpr int kRefEnergySlots = 256;    // work items aimed at where they hold the energies of several densities (see topk_begin)
constexpr int kBinsA = 1024, kBinsB = 512;
constexpr int kSampleSegs = 512;     // sample of a layer: segments of 16 or 32 consecutive elements (see topk_begin)
constexpr int kSampleThreads = 1024;

// ------------------------------------------------------------------------ block helpers
// Suffix sums of a histogram in LDS over the block's first 256 threads: thread t owns the bins
// [t * per, (t + 1) * per) and scan[t] becomes the number of entries in its bins and all higher
// ones (scan[0] = total).  nbins <= 16 * 256.  Every thread of the block calls; the threads past
// the first 256 only join the barriers.
__device__ void block_suffix(const uint32_t* hist, int nbins, uint32_t* scan) {
    __shared__ uint32_t wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool act = tid < 256;
    const int per = (nbins + 255) / 256;
    const int lo = min(tid * per, nbins), hi = min(lo + per, nbins);
    uint32_t inc = 0;
    if (act)
        for (int b = lo; b < hi; ++b) inc += hist[b];
    for (int o = 1; o < 64; o <<= 1) {        // inclusive suffix scan inside the wavefront
        const uint32_t n = __shfl_down(inc, o, 64);
        if (lane + o < 64) inc += n;
    }
    if (act && lane == 0) wtot[wave] = inc;
    __syncthreads();
    if (act) {
        for (int w = wave + 1; w < 4; ++w) inc += wtot[w];
        scan[tid] = inc;
    }
    __syncthreads();
}

// Entries in the bins above a thread's own: thread t of NT holds the bins [t * PER, (t + 1) * PER) in
// c.  Threads past NT only join the barrier.  tot: NT / 64 words of LDS.
template <int NT, int PER>
__device__ __forceinline__ uint32_t entries_above(const uint32_t (&c)[PER], uint32_t* tot, uint32_t* mine) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t sum = 0;
#pragma unroll
    for (int b = 0; b < PER; ++b) sum += c[b];
    uint32_t inc = sum;
    for (int o = 1; o < 64; o <<= 1) {        // inclusive suffix scan inside the wavefront
        const uint32_t n = __shfl_down(inc, o, 64);
        if (lane + o < 64) inc += n;
    }
    if (tid < NT && lane == 0) tot[wave] = inc;
    __syncthreads();
    uint32_t above = inc - sum;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) above += w > wave ? tot[w] : 0u;
    *mine = sum;
    return above;
}

// For the thread that holds the entry of rank `need` from the top (above < need <= above + its own): the
// bin among its PER, the entries in all higher bins and those in the bin.
template <int PER>
__device__ __forceinline__ void find_in_own(const uint32_t (&c)[PER], uint32_t above, uint32_t need, uint32_t* bin,
                                            uint32_t* higher, uint32_t* count) {
    uint32_t run = above;
#pragma unroll
    for (int b = PER - 1; b >= 0; --b) {
        if (run < need && run + c[b] >= need) {
            *bin = (uint32_t)(threadIdx.x * PER + b);
            *higher = run;
            *count = c[b];
        }
        run += c[b];
    }
}

// The largest bin b of a histogram of 256 * PER bins in LDS with (entries in bins >= b) >= need in
// res[0] and the entries in bins > b in res[1], for every thread of the block; {0, total - hist[0]} if
// there are fewer than need entries.  The first 256 threads hold the bins; the others join the barriers.
template <int PER>
__device__ void block_kth_from_top(const uint32_t* hist, uint32_t need, uint32_t* tot, uint32_t* res) {
    const bool act = threadIdx.x < 256;
    uint32_t c[PER];
#pragma unroll
    for (int b = 0; b < PER; ++b) c[b] = act ? hist[threadIdx.x * PER + b] : 0u;
    uint32_t mine;
    const uint32_t above = entries_above<256, PER>(c, tot, &mine);
    if (act && above < need && above + mine >= need) {
        uint32_t count;
        find_in_own<PER>(c, above, need, &res[0], &res[1], &count);
    } else if (threadIdx.x == 0 && above + mine < need) {
        res[0] = 0;
        res[1] = above + mine - c[0];
    }
    __syncthreads();
}

// The same by one wavefront, whose lane t holds the bins [t * PER, (t + 1) * PER) in c; the results are uniform.
template <int PER>
__device__ __forceinline__ void wave_kth_from_top(const uint32_t (&c)[PER], uint32_t need, uint32_t* bin, uint32_t* higher) {
    const int lane = threadIdx.x & 63;
    uint32_t sum = 0;
#pragma unroll
    for (int b = 0; b < PER; ++b) sum += c[b];
    uint32_t inc = sum;
    for (int o = 1; o < 64; o <<= 1) {        // inclusive suffix scan
        const uint32_t n = __shfl_down(inc, o, 64);
        if (lane + o < 64) inc += n;
    }
    uint32_t run = inc - sum, at = 0, above = inc - c[0];          // (lane 0: what there is if nothing is found)
    const unsigned long long found = __ballot(run < need && inc >= need);
#pragma unroll
    for (int b = PER - 1; b >= 0; --b) {
        if (run < need && run + c[b] >= need) {
            at = (uint32_t)(lane * PER + b);
            above = run;
        }
        run += c[b];
    }
    const int src = found ? (int)__builtin_ctzll(found) : 0;
    *bin = (uint32_t)__builtin_amdgcn_readlane((int)at, src);
    *higher = (uint32_t)__builtin_amdgcn_readlane((int)above, src);
}

// ------------------------------------------------------------------------ kernels
__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// One workgroup of the refinement kernels: tiles [t0, t1) of a layer.  Its results lie at `item`, which counts the
// items in the order of the layers; the table itself is in the order in which they are to start (see topk_begin).
struct RefWork {
    int32_t layer, t0, t1, item;
};

// Lower bound of every layer's lowest threshold bin, one workgroup per layer: coarse histogram of a
// sample in LDS, and the bin that holds somewhat more of it than the largest k asks for.  The sample
// is 512 segments of SEG consecutive elements, spread evenly over the layer with a
// scrambled offset inside each stride, so that no row length of a matrix lines up with it; a layer
// of at most 512 SEG elements is taken whole and its bound is exact.  Every thread issues its SEG / 2 loads
// (twice that with error feedback) before it uses the first: the kernel is a memory round trip, 32 or 64 KB per
// layer, and a search of the histogram.  (A sample of 1/16 of the data in three kernels took 33 us
// on a 26 M-element model, remembering the last call's thresholds instead nothing, but a step
// whose gradient is larger or smaller than the one before then collects everything again, or up to
// half of the elements.)
template <int SEG>
__global__ __launch_bounds__(kSampleThreads) void topk_bound_kernel(const float* __restrict__ g,
                                                                    const float* __restrict__ e,
                                                                    const uint32_t* __restrict__ ks, int ntk,
                                                                    const DevLayer* __restrict__ layers,
                                                                    uint32_t* __restrict__ lo) {
    // a copy per residue of the lane, on other banks: most of a layer's elements lie in some 30 bins
    constexpr int kCopies = 4, kPitch = kHistBins + 16, kBinsPer = kHistBins / kSampleThreads;
    static_assert(kBinsPer == 4, "a thread's bins are one 128-bit read");
    __shared__ __align__(16) uint32_t s_hist[kCopies][kPitch];
    __shared__ uint32_t s_tot[kSampleThreads / 64];
    constexpr int kPer = kSampleSegs * SEG / kSampleThreads;
    const int l = blockIdx.x, tid = threadIdx.x;
    uint32_t kmax = 0;
    for (int j = 0; j < ntk; ++j) kmax = max(kmax, ks[(size_t)l * kMaxTopk + j]);
    if (kmax == 0) {
        if (tid == 0) lo[l] = 0xFFFFFFFFu;
        return;
    }
    const DevLayer L = layers[l];
    const uint32_t n = (uint32_t)L.numel;
    const bool whole = n <= (uint32_t)(kSampleSegs * SEG);
    const uint32_t stride = n / kSampleSegs;             // at least SEG unless whole
    float x[kPer], y[kPer];
    uint32_t at[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        if (whole) {
            at[q] = (uint32_t)(q * kSampleThreads + tid);
        } else {
            const uint32_t seg = (uint32_t)(q * (kSampleThreads / SEG) + tid / SEG);
            const uint32_t room = stride - SEG + 1u;
            at[q] = seg * stride + __umulhi(seg * 2654435761u, room) + (uint32_t)(tid % SEG);
        }
    }
    const float* const gl = g + L.offset;
#pragma unroll
    for (int q = 0; q < kPer; ++q) x[q] = gl[min(at[q], n - 1u)];
    if (e) {
        const float* const el = e + L.offset;
#pragma unroll
        for (int q = 0; q < kPer; ++q) y[q] = el[min(at[q], n - 1u)];
    }
#pragma unroll
    for (int h = 0; h < kCopies; ++h) *reinterpret_cast<uint4*>(&s_hist[h][kBinsPer * tid]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (at[q] < n) atomicAdd(&s_hist[tid % kCopies][mag_bits(e ? x[q] + y[q] : x[q]) >> kHistShift], 1u);
    __syncthreads();
    uint32_t want = kmax;
    if (!whole) {
        const float ns = (float)(kSampleSegs * SEG);
        const float t = (float)kmax * (ns / (float)n);   // expected sample entries above the threshold
        const float w = 1.2f * t + 5.0f * sqrtf(t) + 16.0f;      // a margin: the sample only has to be roughly right
        if (w >= ns) {
            if (tid == 0) lo[l] = 0u;
            return;
        }
        want = (uint32_t)w;
    }
    uint32_t c[kBinsPer] = {0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < kCopies; ++h) {
        const uint4 v = *reinterpret_cast<const uint4*>(&s_hist[h][kBinsPer * tid]);
        c[0] += v.x; c[1] += v.y; c[2] += v.z; c[3] += v.w;
    }
    uint32_t mine;
    const uint32_t above = entries_above<kSampleThreads, kBinsPer>(c, s_tot, &mine);
    if (above < want && above + mine >= want) {          // one thread: the sample holds at least `want` entries
        uint32_t bin, higher, count;
        find_in_own<kBinsPer>(c, above, want, &bin, &higher, &count);
        lo[l] = bin;
    }
}

struct CollectParams {
    const float* g;
    const float* e;
    const DevLayer* layers;
    const Tile* tiles;
    const uint32_t* ks;
    const TopkLayer* tl;        // KNOWN: the profile's selection records
    const uint32_t* lo;
    uint32_t* hist;
    uint32_t* cand;
    uint32_t* cand_idx;         // compress: index within the layer and sign of every candidate
    float* ef_out;              // compress: error feedback, written as x everywhere (kept entries are
                                // zeroed afterwards by the emit kernel)
    const int64_t* cand_base;
    TopkTileInfo* tinfo;
    double* base_part;
    uint32_t* cnt_b;            // KNOWN: [L x kBinsB] last 9 pattern bits inside each layer's boundary sub-bin
    // profile (no EMIT): not null = x is written here as it is formed (may be the buffer e points to:
    // every element is read once, by the lane that then writes it)
    float* x_out;
    // profile (no EMIT): where every candidate is goes to cand_idx too, as 16-bit entries (place16)
    int32_t record_idx;
};

// Main pass without quantization candidates: exact coarse histogram (HIST) and candidate
// collection.
// KNOWN (compression right behind a profile of the same data): which layers take part and what
// they keep comes from the layer records (family, slot of the chosen density in the profile's
// selection records), the bound is the 22-bit prefix the profile resolved the k-th magnitude to
// (nearly exactly the kept set qualifies), and the elements inside that boundary sub-bin are
// counted by their last 9 pattern bits (s_hist: kBinsB cells) for the exact threshold.
// TEAM (the second collection, made by the refinement kernel's workgroup for its own tiles): the
// workgroup is several teams of kThreads threads, each with a tile of its own and its own s_red; a team without
// a tile does not come here, so the barrier behind s_red and the sum of it are the caller's, who has checked that the
// layer takes part and gives the bound, team_lo.
template <bool HIST, bool EMIT, bool KNOWN = false, bool TEAM = false>
__device__ __forceinline__ void collect_tile(const CollectParams& p, const int tile, uint32_t* s_hist, double* s_red,
                                             const uint32_t team_lo = 0) {
    static_assert(!(HIST && KNOWN), "the coarse histogram is not built when the thresholds are known");
    static_assert(!TEAM || (!HIST && !KNOWN), "teams collect, nothing else");
    const Tile t = p.tiles[tile];
    const DevLayer L = p.layers[t.layer];
    uint32_t bound;
    if (KNOWN) {
        if (L.family != LGRECO_TOPK || L.slot < 0 || L.slot >= kMaxTopk) return;
        const TopkSel& S = p.tl[t.layer].sel[L.slot];
        bound = ((S.tbin << 10) | S.bin_a) << 9;
    } else {
        if (!TEAM) {
            if (p.ks[(size_t)t.layer * kMaxTopk] == 0) return;
        }
        bound = bound_of_key(TEAM ? team_lo : p.lo[t.layer]);
    }
    const float* gp = p.g + L.offset + t.pos;
    const float* ep = p.e ? p.e + L.offset + t.pos : nullptr;
    float* const eo = EMIT ? p.ef_out + L.offset + t.pos : nullptr;
    float* const xo = (!EMIT && p.x_out) ? p.x_out + L.offset + t.pos : nullptr;
    const int tid = TEAM ? (int)(threadIdx.x % kThreads) : (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (HIST || KNOWN) {
        for (int b = tid; b < (KNOWN ? kBinsB : kHistBins); b += kThreads) s_hist[b] = 0;
        __syncthreads();
    }
    const int64_t slice_off = p.cand_base[t.layer] + t.pos;
    uint32_t* const slice = p.cand + slice_off;
    uint32_t* const slice_idx = EMIT ? p.cand_idx + slice_off : nullptr;
    uint16_t* const slice_at = (!EMIT && p.record_idx) ? reinterpret_cast<uint16_t*>(p.cand_idx) + slice_off : nullptr;
    Collector col;
    uint32_t start;
    if (t.fast) {
        int c0, c1;
        wave_range(t.count / kChunk, wave, &c0, &c1);
        start = (uint32_t)c0 * kChunk;
        col.init(slice + start, slice_idx ? slice_idx + start : nullptr, bound,
                 slice_at ? slice_at + start : nullptr, (uint32_t)t.pos);
        // kGroup chunks of 512 elements at a time: all of them are loaded before the first is used (a wait for a load also
        // waits for the stores in front of it); two: 26 M elements 68 -> 65 us, four as two
        constexpr int kGroup = TEAM ? 1 : 2;
        for (int c = c0; c < c1; c += kGroup) {
            float4 ag[2 * kGroup], bg[2 * kGroup];
#pragma unroll
            for (int i = 0; i < 2 * kGroup; ++i) {
                if (c + i / 2 >= c1) continue;               // (uniform)
                ag[i] = load_stream(gp + c * kChunk + 256 * i + 4 * lane);
                if (ep) bg[i] = load_stream(ep + c * kChunk + 256 * i + 4 * lane);
            }
#pragma unroll
            for (int i = 0; i < 2 * kGroup; ++i) {
                if (c + i / 2 >= c1) continue;
                const int at = c * kChunk + 256 * i + 4 * lane;
                float4 a = ag[i];
                if (ep) { a.x += bg[i].x; a.y += bg[i].y; a.z += bg[i].z; a.w += bg[i].w; }
                if (!EMIT && xo) store_stream(xo + at, a);
                if (EMIT && KNOWN) {
                    // nearly every candidate is kept here: candidates are written as zero at once, the
                    // emit step puts the few that are not kept back
                    float4 w = a;
                    w.x = mag_bits(w.x) >= bound ? 0.0f : w.x;
                    w.y = mag_bits(w.y) >= bound ? 0.0f : w.y;
                    w.z = mag_bits(w.z) >= bound ? 0.0f : w.z;
                    w.w = mag_bits(w.w) >= bound ? 0.0f : w.w;
                    store_stream(eo + at, w);
                } else if (EMIT) {
                    store_stream(eo + at, a);
                }
                if (HIST) {
                    atomicAdd(&s_hist[mag_bits(a.x) >> kHistShift], 1u);
                    atomicAdd(&s_hist[mag_bits(a.y) >> kHistShift], 1u);
                    atomicAdd(&s_hist[mag_bits(a.z) >> kHistShift], 1u);
                    atomicAdd(&s_hist[mag_bits(a.w) >> kHistShift], 1u);
                }
                const float x[4] = {a.x, a.y, a.z, a.w};
                if (KNOWN) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t in = mag_bits(x[q]) - bound;      // below the bound: wraps to a large value
                        if (in < (uint32_t)kBinsB) atomicAdd(&s_hist[in], 1u);
                    }
                }
                col.take4(x, (uint32_t)(t.pos + at));
            }
        }
    } else {
        int b0, b1;
        wave_range((t.count + 63) / 64, wave, &b0, &b1);
        start = (uint32_t)b0 * 64;
        col.init(slice + start, slice_idx ? slice_idx + start : nullptr, bound,
                 slice_at ? slice_at + start : nullptr, (uint32_t)t.pos);
        for (int b = b0; b < b1; ++b) {
            const int i = b * 64 + lane;
            const bool valid = i < t.count;
            float x = 0.0f;
            if (valid) x = ep ? gp[i] + ep[i] : gp[i];
            if (EMIT && valid) eo[i] = (KNOWN && mag_bits(x) >= bound) ? 0.0f : x;
            if (!EMIT && valid && xo) xo[i] = x;
            if (HIST && valid) atomicAdd(&s_hist[mag_bits(x) >> kHistShift], 1u);
            if (KNOWN && valid && mag_bits(x) - bound < (uint32_t)kBinsB) atomicAdd(&s_hist[mag_bits(x) - bound], 1u);
            col.take(x, valid, (uint32_t)(t.pos + i));
        }
    }
    const double bs = wave_sum((double)col.base);
    if (lane == 0) {
        s_red[wave] = bs;
        p.tinfo[tile].cnt[wave] = col.cur;
        p.tinfo[tile].start[wave] = start;
    }
    if (TEAM) return;
    __syncthreads();
    if (tid == 0) p.base_part[tile] = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
    if (HIST) {
        uint32_t* gh = p.hist + (size_t)t.layer * kHistBins;
        for (int b = tid; b < kHistBins; b += kThreads) {
            const uint32_t c = s_hist[b];
            if (c) atomicAdd(&gh[b], c);
        }
    }
    if (KNOWN) {
        uint32_t* gh = p.cnt_b + (size_t)t.layer * kBinsB;
        for (int b = tid; b < kBinsB; b += kThreads) {
            const uint32_t c = s_hist[b];
            if (c) atomicAdd(&gh[b], c);
        }
    }
}

// Main pass of the compression when the profile's selection records are valid for the same data.
__global__ __launch_bounds__(kThreads) void topk_collect_known_kernel(CollectParams p) {
    __shared__ uint32_t s_hist[kBinsB];
    __shared__ double s_red[kThreads / 64];
    collect_tile<false, true, true>(p, (int)blockIdx.x, s_hist, s_red);
}

// The same step from the profile's candidates instead of the data (the profile recorded index and
// sign of every candidate and left x in the error-feedback buffer): every kept entry is among them,
// so the data is not read again.  One workgroup per tile, a wavefront per candidate slice: the
// candidates at or above the boundary sub-bin's lower edge are copied to the second candidate
// buffer IN ELEMENT ORDER (the profile's main pass may store a slice in another order), and the
// boundary sub-bin's entries are counted by their last 9 bits.  Order: every such candidate sets
// the bit of its element in a bitmap of the wavefront's share of the tile (at most kFilterSpan
// elements); its place in the output is the number of bits below its own.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m, uint32_t add);
constexpr int kFilterSpan = kTile / (kThreads / 64);
struct FilterParams {
    const DevLayer* layers;
    const Tile* tiles;
    const TopkLayer* tl;
    const int64_t* cand_base;
    const TopkTileInfo* tinfo;      // what the profile's main pass wrote
    const uint32_t* cand;
    const uint32_t* cand_idx;
    TopkTileInfo* tinfo_out;
    uint32_t* cand_out;
    uint32_t* cand_idx_out;
    uint32_t* cnt_b;
};
constexpr int kFilterKeep = 512;    // kept candidates a wavefront holds in LDS between the two steps
__global__ __launch_bounds__(kThreads) void topk_filter_known_kernel(FilterParams p) {
    constexpr int kWords = kFilterSpan / 32;
    static_assert(kFilterSpan <= 65536, "places inside a wavefront's share are kept in 16 bits");
    __shared__ uint32_t s_bits[kThreads / 64][kWords];
    __shared__ uint16_t s_before[kThreads / 64][kWords];
    __shared__ uint2 s_keep[kThreads / 64][kFilterKeep];
    __shared__ uint32_t s_hist[kBinsB];
    const int tile = blockIdx.x;
    const Tile t = p.tiles[tile];
    const DevLayer L = p.layers[t.layer];
    if (L.family != LGRECO_TOPK || L.slot < 0 || L.slot >= kMaxTopk) return;       // the whole workgroup
    const TopkSel& S = p.tl[t.layer].sel[L.slot];
    const uint32_t bound = ((S.tbin << 10) | S.bin_a) << 9;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t n = p.tinfo[tile].cnt[wave], start = p.tinfo[tile].start[wave];
    const int64_t off = p.cand_base[t.layer] + t.pos + start;
    const uint32_t* const pats = p.cand + off;
    const uint16_t* const idxs = reinterpret_cast<const uint16_t*>(p.cand_idx) + off;   // place16 entries
    for (int b = tid; b < kBinsB; b += kThreads) s_hist[b] = 0;
    for (int b = lane; b < kWords; b += 64) s_bits[wave][b] = 0;
    __syncthreads();
    // step 1: one read of the slice.  What passes sets its element's bit, is counted if it lies in
    // the boundary sub-bin, and is put aside in LDS (the first kFilterKeep of the wavefront).
    constexpr int kBatch = 4;                                 // pairs of loads a lane has in flight
    uint32_t kept = 0;                                        // uniform
    for (uint32_t i0 = 0; i0 < n; i0 += 64 * kBatch) {
        uint32_t pat[kBatch], ix[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const uint32_t i = i0 + 64 * q + lane;
            pat[q] = i < n ? pats[i] : 0u;
            ix[q] = i < n ? idxs[i] : 0u;
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const uint32_t rel = (ix[q] & 0x7FFFu) - start;
            const bool pass = i0 + 64 * q + lane < n && pat[q] >= bound && rel < (uint32_t)kFilterSpan;
            const unsigned long long m = __ballot(pass);
            if (pass) {
                atomicOr(&s_bits[wave][rel >> 5], 1u << (rel & 31u));
                if (pat[q] - bound < (uint32_t)kBinsB) atomicAdd(&s_hist[pat[q] - bound], 1u);
                const uint32_t at = kept + lanes_below(m, 0u);
                if (at < (uint32_t)kFilterKeep) s_keep[wave][at] = make_uint2(pat[q], ix[q]);
            }
            kept += (uint32_t)__popcll(m);
        }
    }
    __syncthreads();
    // exclusive prefix of the bitmap's population over the wavefront's words
    {
        constexpr int kPer = kWords / 64;
        uint32_t c[kPer], mine = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            c[j] = (uint32_t)__popc(s_bits[wave][lane * kPer + j]);
            mine += c[j];
        }
        uint32_t inc = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(inc, o, 64);
            if (lane >= o) inc += v;
        }
        uint32_t run = inc - mine;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            s_before[wave][lane * kPer + j] = (uint16_t)run;
            run += c[j];
        }
    }
    __syncthreads();
    // step 2: every kept candidate goes to the place its element has among the kept ones
    uint32_t* const out = p.cand_out + off;
    uint32_t* const out_idx = p.cand_idx_out + off;
    auto place = [&](const uint32_t pat, const uint32_t ix) __attribute__((always_inline)) {
        const uint32_t rel = (ix & 0x7FFFu) - start;
        const uint32_t w = rel >> 5;
        const uint32_t at = s_before[wave][w] + (uint32_t)__popc(s_bits[wave][w] & ((1u << (rel & 31u)) - 1u));
        out[at] = pat;
        out_idx[at] = ((uint32_t)t.pos + (ix & 0x7FFFu)) | ((ix & 0x8000u) << 16);   // index within the layer, sign
    };
    if (kept <= (uint32_t)kFilterKeep) {
        for (uint32_t i = lane; i < kept; i += 64) {
            const uint2 c = s_keep[wave][i];
            place(c.x, c.y);
        }
    } else {                                                  // more than LDS holds: the slice is read again
        for (uint32_t i0 = 0; i0 < n; i0 += 64 * kBatch) {
            uint32_t pat[kBatch], ix[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const uint32_t i = i0 + 64 * q + lane;
                pat[q] = i < n ? pats[i] : 0u;
                ix[q] = i < n ? idxs[i] : 0u;
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const uint32_t rel = (ix[q] & 0x7FFFu) - start;
                if (i0 + 64 * q + lane < n && pat[q] >= bound && rel < (uint32_t)kFilterSpan) place(pat[q], ix[q]);
            }
        }
    }
    if (lane == 0) {
        p.tinfo_out[tile].cnt[wave] = kept;
        p.tinfo_out[tile].start[wave] = start;
    }
    uint32_t* gh = p.cnt_b + (size_t)t.layer * kBinsB;
    for (int b = tid; b < kBinsB; b += kThreads) {
        const uint32_t c = s_hist[b];
        if (c) atomicAdd(&gh[b], c);
    }
}

template <bool HIST, bool EMIT>
__global__ __launch_bounds__(kThreads) void topk_collect_kernel(CollectParams p) {
    __shared__ uint32_t s_hist[HIST ? kHistBins : 1];
    __shared__ double s_red[kThreads / 64];
    collect_tile<HIST, EMIT>(p, (int)blockIdx.x, s_hist, s_red);
}

// The sums of the quantization profile's tile partials per layer, when the call profiles both families: further
// workgroups of the launch that resolves the threshold bins make them, which depends on the main pass only, too.
struct ScanReduce {
    const double* partials;     // null: no such workgroups
    double* errors;
    const DevLayer* layers;
    int32_t stride;
    ReduceCols cols;
};
// The bin that holds the entry of rank `need` from the top, and the entries in higher bins, by one
// thread alone (after block_suffix; need <= scan[0]).
__device__ __forceinline__ void thread_find(const uint32_t* hist, int nbins, uint32_t need, const uint32_t* scan,
                                            uint32_t* bin, uint32_t* above) {
    const int per = (nbins + 255) / 256;
    int t = 0;                                            // largest t with scan[t] >= need
    for (int step = 128; step; step >>= 1)
        if (t + step < 256 && scan[t + step] >= need) t += step;
    uint32_t running = t + 1 < 256 ? scan[t + 1] : 0u;
    int b = min((t + 1) * per, nbins) - 1;
    for (; b > t * per && running + hist[b] < need; --b) running += hist[b];
    *bin = (uint32_t)b;
    *above = running;
}

// The scan for more than kMaxTopk densities: a thread per density finds its bin.
__global__ __launch_bounds__(256) void topk_scan_many_kernel(uint32_t* __restrict__ hist,
                                                             const uint32_t* __restrict__ ks, int nk, uint32_t* lo,
                                                             TopkMany* __restrict__ many, int n_layers,
                                                             ScanReduce red) {
    static_assert(LGRECO_MAX_CANDS <= 128, "a thread per density, two wavefronts");
    __shared__ __align__(16) unsigned char s_raw[sizeof(uint32_t) * kHistBins];
    if ((int)blockIdx.x >= n_layers) {
        reduce_partials_block(red.partials, red.stride, red.cols, red.layers, red.errors, (int)blockIdx.x - n_layers,
                              reinterpret_cast<double(*)[4]>(s_raw));
        return;
    }
    uint32_t* const s_hist = reinterpret_cast<uint32_t*>(s_raw);
    __shared__ uint32_t s_scan[256], s_bin[LGRECO_MAX_CANDS], s_heads[2];
    const int l = blockIdx.x, tid = threadIdx.x;
    TopkMany& T = many[l];
    uint4* const h4 = reinterpret_cast<uint4*>(hist + (size_t)l * kHistBins);
    for (int b = tid; b < kHistBins / 4; b += 256) {
        reinterpret_cast<uint4*>(s_hist)[b] = h4[b];
        h4[b] = make_uint4(0u, 0u, 0u, 0u);               // the next call's main pass starts from zero
    }
    const uint32_t k = tid < nk ? ks[(size_t)l * nk + tid] : 0u;
    __syncthreads();
    block_suffix(s_hist, kHistBins, s_scan);
    uint32_t bin = 0, above = 0;
    if (tid < nk) {
        thread_find(s_hist, kHistBins, k, s_scan, &bin, &above);
        s_bin[tid] = bin;
    }
    __syncthreads();
    const bool head = tid < nk && (tid == 0 || s_bin[tid - 1] != bin);
    const unsigned long long m = __ballot(head);
    if (tid == 0) s_heads[0] = (uint32_t)__popcll(m);
    if (tid == 64) s_heads[1] = (uint32_t)__popcll(m);
    __syncthreads();
    if (tid < nk) T.need[tid] = k - above;
    if (head) {
        const uint32_t i = (tid < 64 ? 0u : s_heads[0]) + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        T.bin[i] = bin;
        T.first[i] = (uint32_t)tid;
    }
    if (tid == 0) {
        const uint32_t nl = s_heads[0] + s_heads[1];
        T.nlists = nl;
        T.first[nl] = (uint32_t)nk;
        // every element at or above the lowest threshold bin must be among the candidates
        const bool again = lo[l] > bin;
        T.recollect = again ? 1u : 0u;
        if (again) lo[l] = bin;
    }
}

struct RefineParams {
    TopkLayer* tl;
    const DevLayer* layers;
    const Tile* tiles;
    const TopkTileInfo* tinfo;
    const uint32_t* cand;
    const RefWork* work;              // [n_work]
    const int2* work_range;           // [L] the layer's workgroups [x, y)
    int32_t n_work;
    uint32_t* hist;                   // [L x kHistBins] exact coarse histogram
    ScanReduce red;
    const double* base_part;          // [n_tiles]
    double* below_part;               // [n_work x kMaxTopk] energy of candidates below each threshold bin
    // per-workgroup partial histograms (plain stores, summed by the pick kernel)
    unsigned long long* cell_a;       // [n_work x kMaxTopk x kBinsA] profile: packed count + energy
    // compression: a layer's counts, added up where they are (all zero between calls)
    uint32_t* cnt_a;                  // [L x kBinsA]
    uint32_t* cnt_b;                  // [L x kBinsB]
    double* errors;                   // may be null (compress)
    int32_t stride;
    int32_t ntk;
    int32_t col[kMaxTopk];
    // more than kMaxTopk densities: the layers' records, and per (work item, list of this pass), `room` lists
    // in a row, the partial histogram and the energy below the list's bin
    const TopkMany* many;
    const int64_t* cand_base;         // [L]
    const int32_t* cols;              // [nk] column of every density
    unsigned long long* cell_many;
    double* below_many;
    int32_t list0, room;              // the lists of this pass: [list0, list0 + room) of every layer
    // the second collection of a layer whose predicted bound was too high (rare): every workgroup of the first refinement kernel makes it for its own tiles before it looks at
    // their candidates (rc.ef_out not null: the compression's form, which also writes x)
    CollectParams rc;
};

// The second collection for the tiles [t0, t1) of a flagged layer, by a refinement workgroup: four
// teams of kThreads threads, a tile each per round.
static_assert(kRefThreads % kThreads == 0, "whole teams");
template <bool EMIT>
__device__ __forceinline__ void collect_again(const CollectParams& rc, int t0, int t1, uint32_t lo) {
    constexpr int kTeams = kRefThreads / kThreads;
    __shared__ double s_team_red[kTeams][kThreads / 64];
    const int team = threadIdx.x / kThreads;
    for (int first = t0; first < t1; first += kTeams) {
        const int tile = first + team;
        if (tile < t1) collect_tile<false, EMIT, false, true>(rc, tile, nullptr, s_team_red[team], lo);
        __syncthreads();
        if (tile < t1 && threadIdx.x % kThreads == 0) {
            const double* const r = s_team_red[team];
            rc.base_part[tile] = (r[0] + r[1]) + (r[2] + r[3]);
        }
        __syncthreads();                                // s_team_red is reused; the tile's records are written
    }
}

// Walks the candidates of tiles [t0, t1): one (tile, wavefront slice) pair per wavefront at a
// time, 8 loads in flight per lane; f(pattern) is called for every candidate, in a fixed order
// per thread.
template <typename F>
__device__ __forceinline__ void for_each_candidate(const RefineParams& p, int64_t cand_base, int t0, int t1, F f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int kSub = kThreads / 64;
    const int npairs = (t1 - t0) * kSub;
    for (int pr = wave; pr < npairs; pr += kRefThreads / 64) {
        const int t = t0 + pr / kSub, sub = pr % kSub;
        const uint32_t n = p.tinfo[t].cnt[sub];
        const uint32_t* __restrict__ items = p.cand + cand_base + p.tiles[t].pos + p.tinfo[t].start[sub];
        uint32_t i0 = 0;
        for (; i0 + 64 * 8 <= n; i0 += 64 * 8) {          // full batches: no range checks
            uint32_t pat[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) pat[q] = items[i0 + q * 64 + lane];
#pragma unroll
            for (int q = 0; q < 8; ++q) f(pat[q]);
        }
        if (i0 < n) {
            uint32_t pat[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t i = i0 + q * 64 + lane;
                pat[q] = i < n ? items[i] : 0xFFFFFFFFu;      // never a candidate's pattern (sign bit cleared)
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (pat[q] != 0xFFFFFFFFu) f(pat[q]);
        }
    }
}

// Level-A histogram cell of the profile: entries in the low 20 bits (a refinement workgroup sees at
// most kRefTiles * kTile = 2^19 candidates), their integer energy sum (m^2 >> 23 each, < 2^25) above.
constexpr int kPackCountBits = 20, kPackEnergyShift = 23;
static_assert((long long)kRefTiles * kTile < (1ll << kPackCountBits), "count field too narrow");
static_assert(48 - kPackEnergyShift + kPackCountBits - 1 + kPackCountBits <= 64, "energy field too narrow");

__device__ __forceinline__ unsigned long long packed_cell(uint32_t pat) {
    const unsigned long long m = (pat & 0x7FFFFFu) | ((pat >> 23) ? 0x800000u : 0u);
    return (((m * m) >> kPackEnergyShift) << kPackCountBits) | 1ull;
}

// below[j] += x^2 for every j < NTK whose threshold bin lies above the candidate's key.  The
// requested k do not increase with j, so the threshold bins do not decrease and the sets
// {key < tb[j]} are nested: walking j downwards, each comparison narrows the set of active lanes
// (a compare that writes the execution mask) and the add runs under it: two vector instructions
// per k.  The mask is restored at the end; one asm statement, so nothing else runs under it.  The
// closing s_nop keeps the wait states a DPP instruction needs after a vector write of the mask,
// should the compiler place one right behind the block.
#define LG_BELOW_STEP(J) "v_cmpx_gt_u32 vcc, %[t" #J "], %[key]\n\tv_fmac_f32 %[b" #J "], %[x], %[x]\n\t"
#define LG_BELOW_ASM(STEPS)                                                                          \
    asm volatile("s_mov_b64 %[save], exec\n\t" STEPS "s_mov_b64 exec, %[save]\n\ts_nop 3"            \
                 : [b0] "+v"(b[0]), [b1] "+v"(b[1]), [b2] "+v"(b[2]), [b3] "+v"(b[3]), [b4] "+v"(b[4]), \
                   [b5] "+v"(b[5]), [b6] "+v"(b[6]), [b7] "+v"(b[7]), [save] "=&s"(save)              \
                 : [key] "v"(key), [x] "v"(x), [t0] "s"(tb[0]), [t1] "s"(tb[1]), [t2] "s"(tb[2]),      \
                   [t3] "s"(tb[3]), [t4] "s"(tb[4]), [t5] "s"(tb[5]), [t6] "s"(tb[6]), [t7] "s"(tb[7]) \
                 : "vcc")
template <int NTK>
__device__ __forceinline__ void below_chain(float (&b)[kMaxTopk], const uint32_t (&tb)[kMaxTopk], uint32_t key,
                                            float x) {
    static_assert(kMaxTopk == 8 && NTK >= 1 && NTK <= 8, "written out for 8");
    unsigned long long save;
    if constexpr (NTK == 1) LG_BELOW_ASM(LG_BELOW_STEP(0));
    if constexpr (NTK == 2) LG_BELOW_ASM(LG_BELOW_STEP(1) LG_BELOW_STEP(0));
    if constexpr (NTK == 3) LG_BELOW_ASM(LG_BELOW_STEP(2) LG_BELOW_STEP(1) LG_BELOW_STEP(0));
    if constexpr (NTK == 4) LG_BELOW_ASM(LG_BELOW_STEP(3) LG_BELOW_STEP(2) LG_BELOW_STEP(1) LG_BELOW_STEP(0));
    if constexpr (NTK == 5)
        LG_BELOW_ASM(LG_BELOW_STEP(4) LG_BELOW_STEP(3) LG_BELOW_STEP(2) LG_BELOW_STEP(1) LG_BELOW_STEP(0));
    if constexpr (NTK == 6)
        LG_BELOW_ASM(LG_BELOW_STEP(5) LG_BELOW_STEP(4) LG_BELOW_STEP(3) LG_BELOW_STEP(2) LG_BELOW_STEP(1)
                         LG_BELOW_STEP(0));
    if constexpr (NTK == 7)
        LG_BELOW_ASM(LG_BELOW_STEP(6) LG_BELOW_STEP(5) LG_BELOW_STEP(4) LG_BELOW_STEP(3) LG_BELOW_STEP(2)
                         LG_BELOW_STEP(1) LG_BELOW_STEP(0));
    if constexpr (NTK == 8)
        LG_BELOW_ASM(LG_BELOW_STEP(7) LG_BELOW_STEP(6) LG_BELOW_STEP(5) LG_BELOW_STEP(4) LG_BELOW_STEP(3)
                         LG_BELOW_STEP(2) LG_BELOW_STEP(1) LG_BELOW_STEP(0));
}
#undef LG_BELOW_ASM
#undef LG_BELOW_STEP

// Threshold bins, and refinement level A over the candidates of a run of tiles.  Every workgroup finds its layer's
// threshold bins for itself in the exact histogram (16 KB from the caches; a kernel of its own for them, a workgroup
// per layer, took 5-6 us and its launch), the layer's first leaves them in the record.  NTK > 0 (profile, NTK = number of
// requested k): per list (distinct threshold bin) a histogram of bits 18..9 whose cells pack count
// and integer energy into one 64-bit LDS atomic, and per requested k the energy of the candidates
// below its threshold bin (fp32 per lane - a lane sees some tens of candidates - fp64 from the
// wavefront up).  NTK = 0 (compress): counts only.  Which list a candidate belongs to comes from a
// table over the 4096 coarse keys the workgroup builds first.  Partial histograms with energies go to global
// memory with plain stores; the compression's counts (few cells of a layer are not zero) are added to the layer's.
__host__ __device__ constexpr size_t refine_a_lds(int ntk, bool energy) {
    return (size_t)ntk * kBinsA * (energy ? 8 : 4) + kHistBins;
}
template <int NTK>
__global__ __launch_bounds__(kRefThreads, 8) void topk_refine_a_kernel(RefineParams p) {
    constexpr bool ENERGY = NTK > 0;
    constexpr int kN = ENERGY ? NTK : 1, kPer = kHistBins / kRefThreads;
    extern __shared__ unsigned char refine_smem[];
    __shared__ double s_red[kRefThreads / 64][kMaxTopk];
    __shared__ uint32_t s_tot[kRefThreads / 64], s_bin[kMaxTopk], s_higher[kMaxTopk];
    const int tid = threadIdx.x;
    if (ENERGY && (int)blockIdx.x >= p.n_work) {
        reduce_partials_block(p.red.partials, p.red.stride, p.red.cols, p.red.layers, p.red.errors,
                              (int)blockIdx.x - p.n_work, reinterpret_cast<double(*)[4]>(refine_smem));
        return;
    }
    const RefWork w = p.work[blockIdx.x];
    const int l = w.layer;
    static_assert(kPer == 4, "a thread's bins are one 128-bit load");
    const uint4 h = reinterpret_cast<const uint4*>(p.hist + (size_t)l * kHistBins)[tid];
    uint32_t kk[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) kk[j] = p.rc.ks[(size_t)l * kMaxTopk + j];
    const uint32_t used = p.rc.lo[l];
    const int64_t cand_base = p.cand_base[l];
    const bool first_item = w.item == p.work_range[l].x;
    unsigned long long* const s_cell = reinterpret_cast<unsigned long long*>(refine_smem);   // ENERGY
    uint32_t* const s_cnt = reinterpret_cast<uint32_t*>(refine_smem);                        // !ENERGY
    uint8_t* const s_tab = refine_smem + (size_t)kN * kBinsA * (ENERGY ? 8 : 4);
#pragma unroll
    for (int j = 0; j < kN; ++j) {
        if (ENERGY) s_cell[j * kBinsA + tid] = 0; else s_cnt[tid] = 0;
    }
    if (tid < kMaxTopk) s_bin[tid] = s_higher[tid] = 0u;
    // threshold bin of every k: one suffix scan of the histogram serves all of them
    {
        const uint32_t c[kPer] = {h.x, h.y, h.z, h.w};
        uint32_t mine;
        const uint32_t above = entries_above<kRefThreads, kPer>(c, s_tot, &mine);
#pragma unroll
        for (int j = 0; j < kN; ++j)
            if (above < kk[j] && above + mine >= kk[j]) {
                uint32_t count;
                find_in_own<kPer>(c, above, kk[j], &s_bin[j], &s_higher[j], &count);
            }
    }
    __syncthreads();
    // workgroup-uniform.  The k do not increase, so the bins do not decrease and a bin that is not the one before
    // it opens a list.
    uint32_t tb[kMaxTopk], list[kMaxTopk], nlists = 0;
#pragma unroll
    for (int j = 0; j < kMaxTopk; ++j) {
        tb[j] = j < kN ? __builtin_amdgcn_readfirstlane(s_bin[j]) : 0u;
        if (j < kN && (j == 0 || tb[j] != tb[j - 1])) ++nlists;
        list[j] = nlists - 1u;
    }
    if (first_item && tid < kMaxTopk) {
        TopkSel S{};
#pragma unroll
        for (int j = 0; j < kN; ++j)
            if (tid == j) {
                S.k = kk[j];
                S.list = list[j];
            }
        if (tid < kN) {
            S.tbin = s_bin[tid];
            S.need = S.k - s_higher[tid];
        }
        p.tl[l].sel[tid] = S;
        if (tid == 0) p.tl[l].cand_base = cand_base;
    }
    // every element at or above the lowest threshold bin must be among the candidates
    if (used > tb[0]) {
        if (ENERGY) collect_again<false>(p.rc, w.t0, w.t1, tb[0]);
        else collect_again<true>(p.rc, w.t0, w.t1, tb[0]);
    }
    for (uint32_t key = tid; key < (uint32_t)kHistBins; key += kRefThreads) {
        uint32_t hit = 0;               // 1 + number of the list whose bin the key is
#pragma unroll
        for (int j = 0; j < kN; ++j) hit = key == tb[j] ? list[j] + 1u : hit;
        s_tab[key] = (uint8_t)hit;
    }
    __syncthreads();
    float below[kMaxTopk];
#pragma unroll
    for (int j = 0; j < kMaxTopk; ++j) below[j] = 0.0f;
    for_each_candidate(p, cand_base, w.t0, w.t1, [&](uint32_t pat) {
        const uint32_t key = pat >> kHistShift;
        const uint32_t hit = s_tab[key];
        if constexpr (ENERGY) below_chain<NTK>(below, tb, key, __uint_as_float(pat));
        if (hit) {
            const uint32_t b = (hit - 1) * kBinsA + ((pat >> 9) & (kBinsA - 1));
            if (ENERGY) atomicAdd(&s_cell[b], packed_cell(pat));
            else atomicAdd(&s_cnt[b], 1u);
        }
    });
    if (ENERGY) {
#pragma unroll
        for (int j = 0; j < kMaxTopk; ++j) {
            if (j < kN) {
                const double s = wave_sum((double)below[j]);
                if ((tid & 63) == 0) s_red[tid >> 6][j] = s;
            }
        }
    }
    __syncthreads();
    if (ENERGY && tid < kN) {
        double s = 0.0;
        for (int wv = 0; wv < kRefThreads / 64; ++wv) s += s_red[wv][tid];
        p.below_part[(size_t)w.item * kMaxTopk + tid] = s;
    }
    if (ENERGY) {
        unsigned long long* const gc = p.cell_a + (size_t)w.item * kMaxTopk * kBinsA;
        for (int i = tid; i < (int)nlists * kBinsA; i += kRefThreads) gc[i] = s_cell[i];
    } else {
        static_assert(kBinsA == kRefThreads, "a thread per cell");
        const uint32_t c = s_cnt[tid];
        if (c) atomicAdd(&p.cnt_a[(size_t)l * kBinsA + tid], c);
    }
}

// A thread's share (of 256) of a layer's energy below the collection bound, tiles tile, tile + 256, ... before `end`, in
// that order with four loads in flight.
__device__ __forceinline__ double base_energy(const RefineParams& p, int tile, int end) {
    double part = 0.0;
    for (int tt = tile; tt < end; tt += 4 * 256) {
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = tt + q * 256 < end ? p.base_part[tt + q * 256] : 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) part += v[q];
    }
    return part;
}

// Profile: one workgroup per (layer, requested k): sub-bin of level A holding the k-th magnitude, and
// the dropped energy.  Everything outside the boundary sub-bin is
// summed exactly (integer energies).  Inside it the dropped entries are the `drop` smallest of
// `cnt` entries whose integer energies lie in [e_lo, e_hi] and sum to S, so their sum lies in
//     [ max(drop * e_lo, S - keep * e_hi),  drop * S / cnt ]
// (the kept ones are the largest: their mean is at least the overall mean, and none exceeds e_hi).
// The midpoint is taken when half the interval is within 1e-5 of the layer's error - for data
// without clusters the sub-bin holds a vanishing share of the dropped energy and this is always so.
// Otherwise (a constant or clipped layer, quantised values) the workgroup resolves the sub-bin
// exactly: it histograms the last 9 pattern bits of the layer's candidates that fall into the
// sub-bin - every cell is one fp32 value, so its energy is count * value^2 - and sums the `drop`
// smallest.  The deviation from the exact dropped energy is therefore at most 1e-5 relative from
// this step (plus 1.2e-7 from the truncated integer energies and the fp32 sums below the bound).
constexpr double kInsideTolerance = 1e-5;
// The midpoint for the sub-bin `prefix` (pattern >> 9) with `cnt` entries of summed integer energy `sum`, `need_a`
// of them kept, in *inside; false if it is not good enough.
__device__ __forceinline__ bool dropped_inside(uint32_t prefix, uint32_t cnt, uint32_t need_a, unsigned long long sum_e,
                                               int sh, double outside, double* inside) {
    const uint32_t edge = prefix << 9;
    const double e_lo = (double)(packed_cell(edge) >> kPackCountBits);
    const double e_hi = (double)(packed_cell(edge | 0x1FFu) >> kPackCountBits);
    const double sum = (double)sum_e;
    const double drop = (double)(cnt - need_a), keep = (double)need_a;
    const double lower = fmax(drop * e_lo, sum - keep * e_hi);
    const double upper = drop * (sum / (double)cnt);
    *inside = 0.5 * (lower + upper);
    const double half = 0.5 * (upper - lower);
    return !(ldexp(half, sh) > kInsideTolerance * (outside + ldexp(*inside, sh)));
}

// Shift from integer energy units of a coarse bin to x^2.
__device__ __forceinline__ int energy_shift(uint32_t tbin) {
    const uint32_t ex = tbin >> (23 - kHistShift);
    return 2 * ((int)(ex ? ex : 1u) - 150) + kPackEnergyShift;
}

// The rare exact route: histogram of the last 9 bits of a layer's candidates inside the sub-bin
// `prefix`.  s_hist holds kBinsB cells; the whole workgroup calls.
template <int NT>
__device__ void count_sub_bin(const RefineParams& p, int l, int64_t cand_base, uint32_t prefix, uint32_t* s_hist) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int b = tid; b < kBinsB; b += NT) s_hist[b] = 0;
    __syncthreads();
    const DevLayer L = p.layers[l];
    constexpr int kSub = kThreads / 64;
    const int npairs = (L.tile_end - L.tile_begin) * kSub;
    for (int pr = wave; pr < npairs; pr += NT / 64) {
        const int tt = L.tile_begin + pr / kSub, sub = pr % kSub;
        const uint32_t n = p.tinfo[tt].cnt[sub];
        const uint32_t* __restrict__ items = p.cand + cand_base + p.tiles[tt].pos + p.tinfo[tt].start[sub];
        for (uint32_t i = lane; i < n; i += 64) {
            const uint32_t pat = items[i];
            if ((pat >> 9) == prefix) atomicAdd(&s_hist[pat & (kBinsB - 1)], 1u);
        }
    }
    __syncthreads();
}

template <int kPickThreads>
__global__ __launch_bounds__(kPickThreads) void topk_pick_a_kernel(RefineParams p) {
    __shared__ uint32_t s_hist[kBinsA];
    __shared__ unsigned long long s_en[kBinsA];
    __shared__ uint32_t s_tot[4];
    __shared__ uint32_t s_res[2];
    __shared__ unsigned long long s_e;
    __shared__ double s_sum[kPickThreads / 64];
    __shared__ double s_outside;        // error without the boundary sub-bin's dropped part
    __shared__ uint32_t s_exact[3];     // [0] resolve the sub-bin exactly, [1] its prefix (pattern >> 9), [2] entries kept in it
    const int l = blockIdx.x / p.ntk, j = blockIdx.x % p.ntk;      // the grid holds L x ntk workgroups
    TopkLayer& T = p.tl[l];
    if (p.rc.ks[(size_t)l * kMaxTopk + j] == 0) return;
    const TopkSel S = T.sel[j];
    const int2 wr = p.work_range[l];
    const int tid = threadIdx.x, t = tid & 255, grp = tid >> 8;
    if (j == 0)                          // the next call's main pass starts from zero
        for (int b = tid; b < kHistBins / 4; b += kPickThreads)
            reinterpret_cast<uint4*>(p.hist + (size_t)l * kHistBins)[b] = make_uint4(0u, 0u, 0u, 0u);
    if (kPickThreads > 256)
        for (int b = tid; b < kBinsA; b += kPickThreads) {
            s_hist[b] = 0;
            s_en[b] = 0;
        }
    if (tid == 0) {
        s_e = 0;
        s_exact[0] = 0;
    }
    // energy below the collection bound (tile partials) and of the candidates below the threshold bin (workgroup
    // partials), both summed in a fixed order (per thread, then a fixed tree): the first of them are asked for here, beside
    // the partial histograms, and added up behind those
    const int tile0 = p.layers[l].tile_begin + t, tile1 = p.layers[l].tile_end;
    double part = 0.0, base[4] = {0.0, 0.0, 0.0, 0.0}, low = 0.0;
    if (tid < 256) {
#pragma unroll
        for (int q = 0; q < 4; ++q) base[q] = tile0 + q * 256 < tile1 ? p.base_part[tile0 + q * 256] : 0.0;
        if (wr.x + tid < wr.y) low = p.below_part[(size_t)(wr.x + tid) * kMaxTopk + j];
    }
    if (kPickThreads > 256) __syncthreads();
    // sum the layer's workgroup partials of this k's list: 4 bins per thread as 16-byte loads (two
    // pairs of packed cells), the workgroups dealt round-robin to the thread groups,
    // integer LDS atomics join them (order does not matter).  The loop is a chain of memory round
    // trips with a fixed number of loads in flight: wide loads halve its length.
    {
        uint32_t c[4] = {0, 0, 0, 0};
        unsigned long long e[4] = {0, 0, 0, 0};
        static_assert(kBinsA == 1024, "written out for 1024 cells and 256 threads per group");
        const size_t off = (size_t)S.list * kBinsA;
#pragma unroll(kPickThreads == 256 ? 8 : 4)
        for (int wg = wr.x + grp; wg < wr.y; wg += kPickThreads / 256) {
            const size_t i = (size_t)wg * kMaxTopk * kBinsA + off;
            const ulonglong2 v0 = *reinterpret_cast<const ulonglong2*>(p.cell_a + i + 2 * t);
            const ulonglong2 v1 = *reinterpret_cast<const ulonglong2*>(p.cell_a + i + 512 + 2 * t);
            const unsigned long long v[4] = {v0.x, v0.y, v1.x, v1.y};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] += (uint32_t)(v[q] & ((1ull << kPackCountBits) - 1));
                e[q] += v[q] >> kPackCountBits;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cell = (q >> 1) * 512 + 2 * t + (q & 1);
            if (kPickThreads == 256) {                       // a thread's own cells
                s_hist[cell] = c[q];
                s_en[cell] = e[q];
            } else {
                if (c[q]) atomicAdd(&s_hist[cell], c[q]);
                if (e[q]) atomicAdd(&s_en[cell], e[q]);
            }
        }
    }
    if (tid < 256) {
#pragma unroll
        for (int q = 0; q < 4; ++q) part += base[q];
        if (tile0 + 4 * 256 < tile1) part += base_energy(p, tile0 + 4 * 256, tile1);
        part += low;
        for (int wg = wr.x + 256 + tid; wg < wr.y; wg += 256) part += p.below_part[(size_t)wg * kMaxTopk + j];
    }
    __syncthreads();
    block_kth_from_top<kBinsA / 256>(s_hist, S.need, s_tot, s_res);
    const uint32_t bin_a = s_res[0];
    {
        unsigned long long e = 0;
        for (uint32_t b = tid; b < bin_a; b += kPickThreads) e += s_en[b];
        if (e) atomicAdd(&s_e, e);
        if (tid < 256) {
            const double w = wave_sum(part);                 // xor tree inside the wavefront
            if ((tid & 63) == 0) s_sum[tid >> 6] = w;
        }
        __syncthreads();
    }
    const int sh = energy_shift(S.tbin);
    if (tid == 0) {
        const uint32_t need_a = S.need - s_res[1];
        T.sel[j].bin_a = bin_a;
        T.sel[j].need_a = need_a;
        const uint32_t cnt = s_hist[bin_a];
        const double outside = ((s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3])) + ldexp((double)s_e, sh);
        double inside = 0.0;      // dropped part of the sub-bin, in integer-energy units
        const bool exact = cnt > need_a && !dropped_inside((S.tbin << 10) | bin_a, cnt, need_a, s_en[bin_a], sh,
                                                           outside, &inside);
        if (exact) {
            s_outside = outside;
            s_exact[1] = (S.tbin << 10) | bin_a;
            s_exact[2] = need_a;
            s_exact[0] = 1;
        } else {
            p.errors[(size_t)l * p.stride + p.col[j]] = outside + ldexp(inside, sh);
        }
    }
    __syncthreads();
    if (!s_exact[0]) return;                                  // workgroup-uniform
    const uint32_t prefix = s_exact[1], need_a = s_exact[2];
    count_sub_bin<kPickThreads>(p, l, T.cand_base, prefix, s_hist);
    block_kth_from_top<kBinsB / 256>(s_hist, need_a, s_tot, s_res);
    const uint32_t thr_b = s_res[0], keep_at_thr = need_a - s_res[1];
    // dropped inside the sub-bin: every pattern below the threshold pattern, and the entries equal
    // to it that are not kept; a thread's cells in index order, then a fixed tree
    double mine = 0.0;
    for (uint32_t b = tid; b < (uint32_t)kBinsB; b += kPickThreads) {
        const uint32_t c = s_hist[b];
        const uint32_t n_drop = b < thr_b ? c : (b == thr_b ? c - keep_at_thr : 0u);
        const double v = (double)__uint_as_float((prefix << 9) | b);
        mine += (double)n_drop * (v * v);
    }
    const double w = wave_sum(mine);
    __syncthreads();                                          // s_sum was read by thread 0 above
    if ((tid & 63) == 0) s_sum[tid >> 6] = w;
    __syncthreads();
    if (tid == 0) {
        double inside = 0.0;
        for (int q = 0; q < kPickThreads / 64; ++q) inside += s_sum[q];
        p.errors[(size_t)l * p.stride + p.col[j]] = s_outside + inside;
    }
}

// ---- more than kMaxTopk densities
// All of them are resolved at once on the candidates collected once.  What is shared between densities is worked
// out once per list (distinct threshold bin; 100 densities between 0.1 % and 10 % have about 25), and the lists
// are dealt to workgroups in chunks of 8, as many as keep two workgroups on a compute unit.  The partial histograms go
// where those of up to 8 densities do, 14 lists or more per work item; what does not fit (many layers with many
// lists each) takes further passes of these two kernels.  In groups of 8
// densities, each with its own upload, scan, refinement and pick, the 100 densities of a 26 M-element
// model took 13 times 80 us, nearly all of it the latency of short kernels.

// As topk_refine_a_kernel with energies, for the chunks blockIdx.y, blockIdx.y + gridDim.y, ... of the pass's lists.  A
// layer whose predicted bound was too high (flagged by the scan; usually none) is collected again first, by the
// workgroups with blockIdx.y = 0, which then take all of the chunks.
__global__ __launch_bounds__(kRefThreads, 8) void topk_refine_many_kernel(RefineParams p) {
    extern __shared__ unsigned char refine_smem[];
    __shared__ double s_red[kRefThreads / 64][kManyChunk];
    const RefWork w = p.work[blockIdx.x];
    const TopkMany& T = p.many[w.layer];
    const int64_t cand_base = p.cand_base[w.layer];
    const int end = min((int)T.nlists, p.list0 + p.room), tid = threadIdx.x;
    int split = (int)blockIdx.y, splits = (int)gridDim.y;
    if (T.recollect) {                  // workgroup-uniform
        if (split) return;
        splits = 1;
        if (p.list0 == 0) collect_again<false>(p.rc, w.t0, w.t1, p.rc.lo[w.layer]);
    }
    unsigned long long* const s_cell = reinterpret_cast<unsigned long long*>(refine_smem);
    uint8_t* const s_tab = refine_smem + (size_t)kManyChunk * kBinsA * 8;
    for (int c0 = p.list0 + split * kManyChunk; c0 < end; c0 += splits * kManyChunk) {
        const int n = min(kManyChunk, end - c0);
        for (int i = tid; i < n * kBinsA; i += kRefThreads) s_cell[i] = 0;
        uint32_t lb[kManyChunk];                        // ascending; past the end nothing lies above
#pragma unroll
        for (int j = 0; j < kManyChunk; ++j) lb[j] = __builtin_amdgcn_readfirstlane(j < n ? T.bin[c0 + j] : 0xFFFFFFFFu);
        for (uint32_t key = tid; key < (uint32_t)kHistBins; key += kRefThreads) {
            uint32_t hit = 0;
#pragma unroll
            for (int j = 0; j < kManyChunk; ++j) hit = key == lb[j] ? (uint32_t)(j + 1) : hit;
            s_tab[key] = (uint8_t)hit;
        }
        __syncthreads();
        float below[kManyChunk];
#pragma unroll
        for (int j = 0; j < kManyChunk; ++j) below[j] = 0.0f;
        for_each_candidate(p, cand_base, w.t0, w.t1, [&](uint32_t pat) {
            const uint32_t key = pat >> kHistShift;
            const uint32_t hit = s_tab[key];
            below_chain<kManyChunk>(below, lb, key, __uint_as_float(pat));
            if (hit) atomicAdd(&s_cell[(hit - 1) * kBinsA + ((pat >> 9) & (kBinsA - 1))], packed_cell(pat));
        });
#pragma unroll
        for (int j = 0; j < kManyChunk; ++j) {
            const double s = wave_sum((double)below[j]);
            if ((tid & 63) == 0) s_red[tid >> 6][j] = s;
        }
        __syncthreads();
        const size_t out = (size_t)w.item * p.room + (c0 - p.list0);
        if (tid < n) {
            double s = 0.0;
            for (int wv = 0; wv < kRefThreads / 64; ++wv) s += s_red[wv][tid];
            p.below_many[out + tid] = s;
        }
        ulonglong2* const gc = reinterpret_cast<ulonglong2*>(p.cell_many + out * kBinsA);
        for (int i = tid; i < n * kBinsA / 2; i += kRefThreads) gc[i] = reinterpret_cast<const ulonglong2*>(s_cell)[i];
        __syncthreads();                                // the cells are cleared for the next chunk
    }
}

// A workgroup takes the lists blockIdx.y, blockIdx.y + gridDim.y, ... of a layer's in this pass: the list's histogram over the
// layer's work items, then a thread per density for what topk_pick_a_kernel's thread 0 does.
__global__ __launch_bounds__(256) void topk_pick_many_kernel(RefineParams p) {
    __shared__ uint32_t s_hist[kBinsA];
    __shared__ unsigned long long s_en[kBinsA];
    __shared__ uint32_t s_scan[256];
    __shared__ unsigned long long s_pre[256];       // energy of the cells before thread t's four
    __shared__ unsigned long long s_wave[4];
    __shared__ double s_sum[4];
    __shared__ uint32_t s_open;                     // one density that still has to be resolved exactly, plus 1
    __shared__ uint32_t s_prefix;
    const int l = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TopkMany& T = p.many[l];
    const int end = min((int)T.nlists, p.list0 + p.room);
    if (p.list0 + (int)blockIdx.y >= end) return;
    const int2 wr = p.work_range[l];
    const double base = base_energy(p, p.layers[l].tile_begin + (int)(threadIdx.x & 255), p.layers[l].tile_end);
    for (int li = p.list0 + (int)blockIdx.y; li < end; li += (int)gridDim.y) {
        const uint32_t tbin = T.bin[li], first = T.first[li], count = T.first[li + 1] - first;
        double part = base;
        for (int wg = wr.x + tid; wg < wr.y; wg += 256) part += p.below_many[(size_t)wg * p.room + (li - p.list0)];
        // cells 4 t .. 4 t + 3
        uint32_t c[4] = {0, 0, 0, 0};
        unsigned long long e[4] = {0, 0, 0, 0};
#pragma unroll 8
        for (int wg = wr.x; wg < wr.y; ++wg) {
            const ulonglong2* const v2 = reinterpret_cast<const ulonglong2*>(p.cell_many + ((size_t)wg * p.room + (li - p.list0)) * kBinsA + 4 * tid);
            const ulonglong2 v0 = v2[0], v1 = v2[1];
            const unsigned long long v[4] = {v0.x, v0.y, v1.x, v1.y};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] += (uint32_t)(v[q] & ((1ull << kPackCountBits) - 1));
                e[q] += v[q] >> kPackCountBits;
            }
        }
        __syncthreads();                            // the previous list is done with the tables
        unsigned long long mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s_hist[4 * tid + q] = c[q];
            s_en[4 * tid + q] = e[q];
            mine += e[q];
        }
        unsigned long long inc = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long n = __shfl_up(inc, o, 64);
            if (lane >= o) inc += n;
        }
        if (lane == 63) s_wave[wave] = inc;
        const double ws = wave_sum(part);
        if (lane == 0) s_sum[wave] = ws;
        if (tid == 0) s_open = 0;
        __syncthreads();
        for (int w = 0; w < wave; ++w) inc += s_wave[w];
        s_pre[tid] = inc - mine;
        block_suffix(s_hist, kBinsA, s_scan);
        const double under = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
        const int sh = energy_shift(tbin);
        bool open = false;
        uint32_t prefix = 0, need_a = 0;
        double outside = 0.0;
        if ((uint32_t)tid < count) {
            uint32_t bin_a, above;
            thread_find(s_hist, kBinsA, T.need[first + tid], s_scan, &bin_a, &above);
            need_a = T.need[first + tid] - above;
            unsigned long long en = s_pre[bin_a >> 2];
            for (uint32_t b = bin_a & ~3u; b < bin_a; ++b) en += s_en[b];
            outside = under + ldexp((double)en, sh);
            prefix = (tbin << 10) | bin_a;
            const uint32_t cnt = s_hist[bin_a];
            double inside = 0.0;
            open = cnt > need_a && !dropped_inside(prefix, cnt, need_a, s_en[bin_a], sh, outside, &inside);
            if (!open) p.errors[(size_t)l * p.stride + p.cols[first + tid]] = outside + ldexp(inside, sh);
        }
        // densities that need it are resolved exactly, those of one sub-bin together
        for (;;) {
            if (open) s_open = (uint32_t)tid + 1u;
            __syncthreads();
            const uint32_t who = s_open;
            if (!who) break;                        // workgroup-uniform
            if (who == (uint32_t)tid + 1u) s_prefix = prefix;
            __syncthreads();
            const uint32_t now = s_prefix;
            count_sub_bin<256>(p, l, p.cand_base[l], now, s_hist);
            block_suffix(s_hist, kBinsB, s_scan);
            if (tid == 0) s_open = 0;
            if (open && prefix == now) {
                uint32_t thr_b, above;
                thread_find(s_hist, kBinsB, need_a, s_scan, &thr_b, &above);
                double inside = 0.0;
                for (uint32_t b = 0; b <= thr_b; ++b) {
                    const uint32_t n_drop = b < thr_b ? s_hist[b] : s_hist[b] - (need_a - above);
                    const double v = (double)__uint_as_float((prefix << 9) | b);
                    inside += (double)n_drop * (v * v);
                }
                p.errors[(size_t)l * p.stride + p.cols[first + tid]] = outside + inside;
                open = false;
            }
            __syncthreads();
        }
    }
}

// Refinement level B (compression, one density): the level-A sub-bin that holds the k-th magnitude, found by every
// workgroup for itself in the layer's counts, and the counts of bits 8..0 of the candidates inside it.  (In
// a kernel of its own between the two levels, a workgroup per layer, that search cost a launch; see topk_count_kernel.)
__global__ __launch_bounds__(kRefThreads) void topk_refine_b_kernel(RefineParams p) {
    __shared__ uint32_t s_cnt[kBinsB], s_tot[kRefThreads / 64], s_res[2];
    const RefWork w = p.work[blockIdx.x];
    TopkLayer& T = p.tl[w.layer];
    const int tid = threadIdx.x;
    const uint32_t c[1] = {p.cnt_a[(size_t)w.layer * kBinsA + tid]};
    const uint32_t need = T.sel[0].need, tbin = T.sel[0].tbin;
    const int64_t cand_base = T.cand_base;
    if (tid < kBinsB) s_cnt[tid] = 0;
    uint32_t mine;
    const uint32_t above = entries_above<kRefThreads, 1>(c, s_tot, &mine);      // (one barrier)
    if (above < need && above + mine >= need) {          // one thread: the bin holds at least `need` entries
        s_res[0] = (uint32_t)tid;
        s_res[1] = above;
    } else if (tid == 0 && above + mine < need) {
        s_res[0] = 0;
        s_res[1] = above + mine - c[0];
    }
    __syncthreads();
    const uint32_t prefix = (tbin << 10) | s_res[0];
    if (w.item == p.work_range[w.layer].x) {
        static_assert(kHistBins == 4 * kRefThreads, "a 128-bit store a thread");
        reinterpret_cast<uint4*>(p.hist + (size_t)w.layer * kHistBins)[tid] = make_uint4(0u, 0u, 0u, 0u);   // for the next call
        if (tid == 0) {
            T.sel[0].bin_a = s_res[0];
            T.sel[0].need_a = need - s_res[1];
        }
    }
    for_each_candidate(p, cand_base, w.t0, w.t1, [&](uint32_t pat) {
        if ((pat >> 9) == prefix) atomicAdd(&s_cnt[pat & (kBinsB - 1)], 1u);
    });
    __syncthreads();
    if (tid < kBinsB && s_cnt[tid]) atomicAdd(&p.cnt_b[(size_t)w.layer * kBinsB + tid], s_cnt[tid]);
}

// ---------------------------------------------------------------- compression kernels
// The compressor keeps the collector's partition: wavefront w of a tile owns the same contiguous
// element range it collected candidates from, so everything below is per wavefront and needs no
// workgroup barrier.

// Both kernels below are chains of dependent loads (tile -> layer record -> a few tens of
// candidates per wavefront), so a workgroup takes kSliceBatch consecutive tiles and every
// wavefront walks its slice of each of them side by side: the loads of one level are in flight
// together and the chain's latency is paid once per batch.
constexpr int kSliceBatch = 4;

// per (tile, wavefront): entries above the threshold, entries equal to it (from its candidates)
// ks: the k asked for; KNOWN: the layer records say which layers take part and which selection record counts.
// The exact threshold and the number of entries equal to it that are kept come from the layer's counts inside the
// boundary sub-bin: wavefront q of every workgroup finds them for the batch's tile q, and the one with a layer's first
// tile leaves them in its record.  (A kernel of its own in front of this one, a workgroup per layer, took 4-5 us and
// its launch; 2 KB a wavefront from the caches and six exchanges between lanes cost a fraction of that.)
static_assert(kSliceBatch == kThreads / 64, "a wavefront per tile of a batch");
template <bool KNOWN>
__global__ __launch_bounds__(kThreads) void topk_count_kernel(const Tile* __restrict__ tiles, int n_tiles,
                                                               const DevLayer* __restrict__ layers,
                                                               const uint32_t* __restrict__ ks, TopkLayer* tl,
                                                               const uint32_t* __restrict__ cnt_b,
                                                               const TopkTileInfo* __restrict__ tinfo,
                                                               const uint32_t* __restrict__ cand,
                                                               uint2* __restrict__ wavecnt) {
    __shared__ uint32_t s_thr[kSliceBatch];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = blockIdx.x * kSliceBatch;
    const Tile own = tiles[min(first + wave, n_tiles - 1)];
    const uint4* const own_cnt = reinterpret_cast<const uint4*>(cnt_b + (size_t)own.layer * kBinsB) + 2 * lane;
    const uint4 c0 = own_cnt[0], c1 = own_cnt[1];
    const uint32_t* items[kSliceBatch];
    uint32_t n[kSliceBatch], thr[kSliceBatch], gt[kSliceBatch], eq[kSliceBatch];
    bool active[kSliceBatch];
    uint32_t nmax = 0;
    // every load of a level is unconditional (indices clamped to the table), so that the levels
    // of the batch's chains are issued together
    int64_t pos[kSliceBatch], base[kSliceBatch];
    int layer[kSliceBatch];
    uint32_t start[kSliceBatch], k[kSliceBatch];
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        const int ti = min(first + q, n_tiles - 1);
        layer[q] = tiles[ti].layer;
        pos[q] = tiles[ti].pos;
        n[q] = tinfo[ti].cnt[wave];
        start[q] = tinfo[ti].start[wave];
    }
    int slot[kSliceBatch];
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        slot[q] = 0;
        if (KNOWN) {
            const DevLayer& L = layers[layer[q]];
            k[q] = (L.family == LGRECO_TOPK && L.slot >= 0 && L.slot < kMaxTopk) ? 1u : 0u;
            slot[q] = k[q] ? L.slot : 0;
        }
    }
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        const TopkLayer& T = tl[layer[q]];
        if (!KNOWN) k[q] = ks[(size_t)layer[q] * kMaxTopk];
        base[q] = T.cand_base;
    }
    {
        int own_slot = 0;
        bool own_on = first + wave < n_tiles;
        if (KNOWN) {
            const DevLayer& L = layers[own.layer];
            own_on = own_on && L.family == LGRECO_TOPK && L.slot >= 0 && L.slot < kMaxTopk;
            own_slot = own_on ? L.slot : 0;
        }
        TopkSel& S = tl[own.layer].sel[own_slot];
        const uint32_t need_a = S.need_a, prefix = (S.tbin << 10) | S.bin_a;
        if (!KNOWN) own_on = own_on && ks[(size_t)own.layer * kMaxTopk] != 0;
        static_assert(kBinsB == 64 * 8, "8 cells a lane");
        const uint32_t c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
        uint32_t bin, higher;
        wave_kth_from_top<8>(c, need_a, &bin, &higher);
        const uint32_t own_thr = (prefix << 9) | bin;
        if (lane == 0) {
            s_thr[wave] = own_thr;
            if (own_on && own.pos == 0) {
                S.thr = own_thr;
                S.ties_keep = need_a - higher;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) thr[q] = s_thr[q];
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        // a layer that is not compressed with Top-K has k = 0 (and neither candidates nor a record)
        active[q] = first + q < n_tiles && k[q] != 0;
        n[q] = active[q] ? n[q] : 0u;
        items[q] = active[q] ? cand + base[q] + pos[q] + start[q] : cand;
        gt[q] = eq[q] = 0;
        nmax = max(nmax, n[q]);
    }
    for (uint32_t i = lane; i < nmax; i += 64) {
        uint32_t pat[kSliceBatch];
#pragma unroll
        for (int q = 0; q < kSliceBatch; ++q) pat[q] = i < n[q] ? items[q][i] : 0xFFFFFFFFu;   // never a pattern
#pragma unroll
        for (int q = 0; q < kSliceBatch; ++q) {
            gt[q] += (pat[q] != 0xFFFFFFFFu) & (pat[q] > thr[q]);
            eq[q] += pat[q] == thr[q];
        }
    }
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        for (int o = 1; o < 64; o <<= 1) {
            gt[q] += __shfl_xor(gt[q], o, 64);
            eq[q] += __shfl_xor(eq[q], o, 64);
        }
        if (lane == 0 && active[q])
            wavecnt[(size_t)(first + q) * (kThreads / 64) + wave] = make_uint2(gt[q], eq[q]);
    }
}

__device__ __forceinline__ uint32_t lanes_below(unsigned long long m, uint32_t add) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, add));
}

// Counts of every run of kRunTiles tiles (by tile number; runs that reach past a layer's end are not looked at):
// one workgroup per run.  Both counts travel in one 64-bit word, (entries above the threshold) << 32 | entries equal
// to it (each stays below 2^31: a layer has fewer elements than that).
constexpr int kRunTiles = 1024;
__global__ __launch_bounds__(kThreads) void topk_runs_kernel(const uint2* __restrict__ wavecnt, int n_tiles,
                                                             unsigned long long* __restrict__ runs) {
    __shared__ unsigned long long s_sum[kThreads / 64];
    const int first = blockIdx.x * kRunTiles, n_pairs = min(kRunTiles, n_tiles - first) * (kThreads / 64 / 2);
    const uint4* const pairs = reinterpret_cast<const uint4*>(wavecnt + (size_t)first * (kThreads / 64));
    unsigned long long sum = 0;
#pragma unroll
    for (int u = 0; u < kRunTiles * (kThreads / 64 / 2) / kThreads; ++u) {
        const int i = (int)threadIdx.x + u * kThreads;
        const uint4 v = i < n_pairs ? pairs[i] : make_uint4(0u, 0u, 0u, 0u);
        sum += ((unsigned long long)(v.x + v.z) << 32) + (v.y + v.w);
    }
    for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) runs[blockIdx.x] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

// Kept values and indices in ascending index order, from the candidates alone (every kept entry
// is a candidate, and a wavefront's candidates are stored in element order); the error feedback,
// already written as x everywhere by the collection pass, is zeroed at the kept entries (KNOWN:
// written as zero at every candidate by that pass, and set back to x at those not kept).
// Where a wavefront's entries go is the sum of the counts of all wavefronts before it in the layer: the
// workgroup adds up those before its first tile (of the largest layer of a 355 M-element model 50 KB at most,
// 8 128-bit loads in flight per thread) and walks its own 16.  As a kernel of its own, a
// workgroup per layer, that prefix took 4-5 us and its launch; 18 beside a kernel that fills the chip.
// The counts of a layer that the thresholds came from are cleared by the workgroup with its first tile.
// `runs` (not null where a layer has more than kTilesInRuns tiles): the whole runs of tiles before its first come as
// their sums, so that what a workgroup reads stays bounded.
template <bool KNOWN>
__global__ __launch_bounds__(kThreads) void topk_emit_kernel(float* __restrict__ e,
                                                              const DevLayer* __restrict__ layers,
                                                              const Tile* __restrict__ tiles, int n_tiles,
                                                              const TopkLayer* __restrict__ tl,
                                                              const TopkTileInfo* __restrict__ tinfo,
                                                              const uint32_t* __restrict__ cand,
                                                              const uint32_t* __restrict__ cand_idx,
                                                              const uint2* __restrict__ wavecnt,
                                                              const unsigned long long* __restrict__ runs,
                                                              uint32_t* __restrict__ cnt_a, uint32_t* __restrict__ cnt_b,
                                                              uint8_t* __restrict__ payload, int x_in_e) {
    // x_in_e (KNOWN only): the main pass left the buffer as it was (x everywhere), so the kept
    // entries are zeroed here, as without KNOWN, and nothing is put back
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = blockIdx.x * kSliceBatch;
    struct Slice {
        const uint32_t* pats;
        const uint32_t* idxs;
        float* ef;
        float* values;
        uint32_t* indices;
        uint32_t n, thr, ties_keep, out, eq_seen;
        bool eq_all, eq_none;
    } S[kSliceBatch];
    uint32_t nmax = 0;
    // every load of a level is unconditional (indices clamped to the tables; the count arrays
    // cover every tile), so that the levels of the batch's chains are issued together
    int64_t pos[kSliceBatch];
    int layer[kSliceBatch];
    uint32_t start[kSliceBatch];
    uint2 cnt[kSliceBatch], before[kSliceBatch];
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        const int ti = min(first + q, n_tiles - 1);
        const size_t slot = (size_t)ti * (kThreads / 64) + wave;
        layer[q] = tiles[ti].layer;
        pos[q] = tiles[ti].pos;
        S[q].n = tinfo[ti].cnt[wave];
        start[q] = tinfo[ti].start[wave];
        cnt[q] = wavecnt[slot];
    }
    constexpr int kWaves = kThreads / 64, kBatch = 8;
    static_assert(kWaves % 2 == 0, "a tile's counts are read in pairs");
    __shared__ unsigned long long s_before[kWaves];
    unsigned long long sum = 0;                          // (entries above the threshold) << 32 | entries equal to it
    {
        const int begin = layers[layer[0]].tile_begin;
        const uint4* const pairs = reinterpret_cast<const uint4*>(wavecnt + (size_t)begin * kWaves);
        int n_pairs = (first - begin) * (kWaves / 2), head = n_pairs, skip = 0;       // pairs in front of the whole runs, in them
        if (runs) {
            const int r0 = (begin + kRunTiles - 1) / kRunTiles, r1 = first / kRunTiles;
            if (r0 < r1) {
                head = (r0 * kRunTiles - begin) * (kWaves / 2);
                skip = (r1 - r0) * kRunTiles * (kWaves / 2);
                n_pairs -= skip;
                for (int r = r0 + (int)threadIdx.x; r < r1; r += kThreads) sum += runs[r];
            }
        }
        for (int i = (int)threadIdx.x; i < n_pairs; i += kBatch * kThreads) {
            uint4 v[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int j = i + u * kThreads;
                v[u] = j < n_pairs ? pairs[j < head ? j : j + skip] : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) sum += ((unsigned long long)(v[u].x + v[u].z) << 32) + (v[u].y + v[u].w);
        }
        for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) s_before[wave] = sum;
        __syncthreads();
        sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += s_before[w];
    }
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        const uint2* const c = wavecnt + (size_t)min(first + q, n_tiles - 1) * kWaves;
        if (q > 0 && layer[q] != layer[q - 1]) sum = 0;  // the layer begins with this tile
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w == wave) before[q] = make_uint2((uint32_t)(sum >> 32), (uint32_t)sum);
            sum += ((unsigned long long)c[w].x << 32) + c[w].y;
        }
    }
#pragma unroll
    for (int q = 0; q < kSliceBatch; ++q) {
        const DevLayer& L = layers[layer[q]];
        const TopkLayer& T = tl[layer[q]];
        const bool active = first + q < n_tiles && L.family == LGRECO_TOPK &&
                            (!KNOWN || (L.slot >= 0 && L.slot < kMaxTopk));
        const int64_t off = active ? T.cand_base + pos[q] + start[q] : 0;
        const TopkSel& Sel = T.sel[(KNOWN && active) ? L.slot : 0];
        const uint32_t keep_eq = Sel.ties_keep;
        S[q].pats = cand + off;
        S[q].idxs = cand_idx + off;
        S[q].ef = e + L.offset;
        S[q].values = reinterpret_cast<float*>(payload + L.payload);
        S[q].indices = reinterpret_cast<uint32_t*>(payload + L.payload) + Sel.k;
        S[q].n = active ? S[q].n : 0u;
        S[q].thr = Sel.thr;
        S[q].ties_keep = keep_eq;
        // equal entries: global rank r (in index order) is kept iff r < ties_keep
        S[q].eq_all = before[q].y + cnt[q].y <= keep_eq;
        S[q].eq_none = before[q].y >= keep_eq;
        S[q].out = before[q].x + min(before[q].y, keep_eq);
        S[q].eq_seen = before[q].y;
        nmax = max(nmax, S[q].n);
        if (active && pos[q] == 0) {                         // (uniform; the count kernel was the last to read them)
            uint32_t* const b = cnt_b + (size_t)layer[q] * kBinsB;
            for (int i = (int)threadIdx.x; i < kBinsB; i += kThreads) b[i] = 0u;
            if (!KNOWN) {
                uint32_t* const a = cnt_a + (size_t)layer[q] * kBinsA;
                for (int i = (int)threadIdx.x; i < kBinsA; i += kThreads) a[i] = 0u;
            }
        }
    }
    for (uint32_t i0 = 0; i0 < nmax; i0 += 64) {
        const uint32_t i = i0 + lane;
        uint32_t pat[kSliceBatch], ix[kSliceBatch];
#pragma unroll
        for (int q = 0; q < kSliceBatch; ++q) {
            const bool ok = i < S[q].n;
            pat[q] = ok ? S[q].pats[i] : 0u;
            ix[q] = ok ? S[q].idxs[i] : 0u;
        }
#pragma unroll
        for (int q = 0; q < kSliceBatch; ++q) {
            if (i0 >= S[q].n) continue;                      // wavefront-uniform
            const bool ok = i < S[q].n;
            bool keep = ok && pat[q] > S[q].thr;
            const bool eq = ok && pat[q] == S[q].thr;
            if (S[q].eq_all) {
                keep = keep || eq;
            } else if (!S[q].eq_none) {
                const unsigned long long bq = __ballot(eq);
                if (eq) keep = S[q].eq_seen + lanes_below(bq, 0u) < S[q].ties_keep;
                S[q].eq_seen += (uint32_t)__popcll(bq);
            }
            const unsigned long long kq = __ballot(keep);
            if (keep) {
                const uint32_t pos = S[q].out + lanes_below(kq, 0u);
                S[q].values[pos] = __uint_as_float(pat[q] | (ix[q] & 0x80000000u));
                S[q].indices[pos] = ix[q] & 0x7FFFFFFFu;
                if (!KNOWN || x_in_e) S[q].ef[ix[q] & 0x7FFFFFFFu] = 0.0f;
            } else if (KNOWN && !x_in_e && ok) {
                // the main pass wrote zero for every candidate: the ones that are not kept get x back
                S[q].ef[ix[q] & 0x7FFFFFFFu] = __uint_as_float(pat[q] | (ix[q] & 0x80000000u));
            }
            S[q].out += (uint32_t)__popcll(kq);
        }
    }
}

// ------------------------------------------------------------------------ host side
#define TK_CHECK(expr)                     \
    do {                                   \
        hipError_t _e = (expr);            \
        if (_e != hipSuccess) return _e;   \
    } while (0)

// Partial histograms (and the energies beside them) of a call with more than kMaxTopk densities that the
// refinement's buffer holds, in (work item, list) pairs; at least 7 per work item.  The buffers behind it (what is kept
// of a profile's candidates, x = g + e of the low-rank layers) are written after the refinement that reads these, if at all.
constexpr size_t kManyBytes = sizeof(unsigned long long) * kBinsA + sizeof(double);
static size_t many_capacity(const TopkScratch* t) { return t->ref_bytes / kManyBytes; }

hipError_t topk_scratch_create(TopkScratch* t, int64_t max_elems, int max_layers, int max_tiles, int max_cands) {
    t->max_elems = max_elems;
    t->max_layers = max_layers;
    t->max_tiles = max_tiles;
    TK_CHECK(hipMalloc(&t->d_hist, sizeof(uint32_t) * (size_t)max_layers * kHistBins));
    // Between calls the exact histogram is all zero: cleared here once, and by the last kernel that
    // follows the search of every call for the layers that call counted.  hist_clean is false only after a call that failed midway.
    TK_CHECK(hipMemset(t->d_hist, 0, sizeof(uint32_t) * (size_t)max_layers * kHistBins));
    t->hist_clean = true;
    TK_CHECK(hipMalloc(&t->d_tl, sizeof(TopkLayer) * (size_t)max_layers));
    // counts of a compression: all zero between calls (the emit kernel clears them), counts_clean as above
    const size_t counts = (size_t)max_layers * (kBinsA + kBinsB);
    TK_CHECK(hipMalloc(&t->d_cnt_a, sizeof(uint32_t) * counts));
    TK_CHECK(hipMemset(t->d_cnt_a, 0, sizeof(uint32_t) * counts));
    t->d_cnt_b = t->d_cnt_a + (size_t)max_layers * kBinsA;
    t->counts_clean = true;
    TK_CHECK(hipMalloc(&t->d_cand, sizeof(uint32_t) * (size_t)max_elems));
    TK_CHECK(hipMalloc(&t->d_cand_idx, sizeof(uint32_t) * (size_t)max_elems));
    TK_CHECK(hipMalloc(&t->d_tinfo_kept, sizeof(TopkTileInfo) * (size_t)max_tiles));
    TK_CHECK(hipMalloc(&t->d_lo, sizeof(uint32_t) * (size_t)max_layers));
    TK_CHECK(hipMalloc(&t->d_tilecnt, sizeof(uint2) * (size_t)max_tiles * (kThreads / 64)));
    TK_CHECK(hipMalloc(&t->d_runs, sizeof(unsigned long long) * (size_t)(max_tiles / kRunTiles + 1)));
    TK_CHECK(hipMalloc(&t->d_tinfo, sizeof(TopkTileInfo) * (size_t)max_tiles));
    TK_CHECK(hipMalloc(&t->d_base_part, sizeof(double) * (size_t)max_tiles));
    t->max_work = (int)(max_elems / ((int64_t)kRefTiles * kTile)) + 2 * max_layers + 2 + 2 * kRefSlots;   // see topk_begin
    TK_CHECK(hipMalloc(&t->d_below_part, sizeof(double) * (size_t)t->max_work * kMaxTopk));
    // The refinement's partial histograms, then what is kept of a profile's candidates.  A handle that may be asked for
    // more densities than kMaxTopk uses both for a list of each in every work item (see topk_begin for their number) where
    // that fits with at most 112 KB a work item in the first part; what does not fit takes further passes.
    const size_t kept = (sizeof(uint32_t) * (size_t)max_elems + 255) / 256 * 256, part = (size_t)t->max_work * kMaxTopk * kBinsA;
    size_t ref = part * sizeof(unsigned long long);
    if (max_cands > (int)kMaxTopk) {
        const size_t items = (size_t)std::max<int64_t>(2 * kRefSlots / kManySplit, max_elems / ((int64_t)kRefTiles * kTile)) + 2 * (size_t)max_layers + 2;
        const size_t want = items * (size_t)max_cands * kManyBytes, most = part * 14;
        if (want > 2 * kept + ref) ref = std::min((want - 2 * kept + 255) / 256 * 256, most);
    }
    t->ref_bytes = ref + 2 * kept;
    TK_CHECK(hipMalloc(&t->d_ref, t->ref_bytes));
    t->d_kept = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(t->d_ref) + ref);
    t->d_kept_idx = t->d_kept + kept / sizeof(uint32_t);
    if (max_cands > (int)kMaxTopk) TK_CHECK(hipMalloc(&t->d_many, sizeof(TopkMany) * (size_t)max_layers));
    // control block layout (every part a multiple of 16 bytes)
    const size_t o_k = 0;
    const size_t o_base = o_k + sizeof(uint32_t) * (size_t)max_layers * kMaxTopk;
    const size_t o_range = o_base + (sizeof(int64_t) * (size_t)max_layers + 15) / 16 * 16;
    const size_t o_work = o_range + (sizeof(int2) * (size_t)max_layers + 15) / 16 * 16;
    const size_t o_many = o_work + sizeof(RefWork) * (size_t)t->max_work;
    const size_t many_words = max_cands > kMaxTopk ? (size_t)max_layers * max_cands + max_cands : 0;    // columns, k
    t->ctl_bytes = o_many + sizeof(uint32_t) * many_words;
    t->ctl_off[0] = o_k; t->ctl_off[1] = o_base; t->ctl_off[2] = o_range; t->ctl_off[3] = o_work;
    t->ctl_off[4] = o_many;
    TK_CHECK(hipHostMalloc(&t->h_ctl, t->ctl_bytes, hipHostMallocDefault));
    TK_CHECK(hipEventCreateWithFlags(&t->ctl_copied, hipEventDisableTiming));
    std::memset(t->h_ctl, 0, t->ctl_bytes);
    for (int i = 0; i < 2; ++i) {
        TK_CHECK(hipMalloc(&t->d_ctl[i], t->ctl_bytes));
        t->h_ctl_last[i] = static_cast<uint8_t*>(std::malloc(t->ctl_bytes));
        if (!t->h_ctl_last[i]) return hipErrorOutOfMemory;
        t->ctl_last_bytes[i] = 0;
    }
    t->many_last_bytes = 0;
    t->h_k = reinterpret_cast<uint32_t*>(t->h_ctl + o_k);
    t->h_many = reinterpret_cast<uint32_t*>(t->h_ctl + o_many);
    t->h_cand_base = reinterpret_cast<int64_t*>(t->h_ctl + o_base);
    t->h_work_range = t->h_ctl + o_range;
    t->h_work = t->h_ctl + o_work;
    return hipSuccess;
}

void topk_scratch_destroy(TopkScratch* t) {
    (void)hipFree(t->d_hist);
    (void)hipFree(t->d_tl);
    (void)hipFree(t->d_cnt_a);
    (void)hipFree(t->d_cand);
    (void)hipFree(t->d_cand_idx);
    (void)hipFree(t->d_tinfo_kept);
    (void)hipFree(t->d_lo);
    (void)hipFree(t->d_tilecnt);
    (void)hipFree(t->d_runs);
    (void)hipFree(t->d_tinfo);
    (void)hipFree(t->d_base_part);
    (void)hipFree(t->d_below_part);
    (void)hipFree(t->d_ref);
    (void)hipFree(t->d_many);
    for (int i = 0; i < 2; ++i) {
        (void)hipFree(t->d_ctl[i]);
        std::free(t->h_ctl_last[i]);
    }
    (void)hipHostFree(t->h_ctl);
    if (t->ctl_copied) (void)hipEventDestroy(t->ctl_copied);
    *t = TopkScratch{};
}

// The pinned control block may be written again once the last upload that was queued from it has
// executed (a call may return, and a stream may be busy, with that copy still pending).
static hipError_t ctl_writable(TopkScratch* t) {
    if (t->ctl_pending) {
        TK_CHECK(hipEventSynchronize(t->ctl_copied));
        t->ctl_pending = false;
    }
    return hipSuccess;
}

// One upload of the control block up to the last work item, skipped when this slot's device copy
// already holds the same bytes.
static hipError_t upload_ctl(TopkScratch* t, int slot, hipStream_t s) {
    uint8_t* const d = t->d_ctl[slot];
    t->d_k = reinterpret_cast<uint32_t*>(d + t->ctl_off[0]);
    t->d_cand_base = reinterpret_cast<int64_t*>(d + t->ctl_off[1]);
    t->d_work_range = d + t->ctl_off[2];
    t->d_work = d + t->ctl_off[3];
    t->d_many_in = reinterpret_cast<uint32_t*>(d + t->ctl_off[4]);
    const size_t used = t->ctl_off[3] + sizeof(RefWork) * (size_t)std::max(t->n_work, 1);
    const bool differs = used != t->ctl_last_bytes[slot] || std::memcmp(t->h_ctl, t->h_ctl_last[slot], used) != 0;
    if (differs) {
        TK_CHECK(hipMemcpyAsync(d, t->h_ctl, used, hipMemcpyHostToDevice, s));
        // the copy reads the pinned block when it executes: the next writer waits for this event
        TK_CHECK(hipEventRecord(t->ctl_copied, s));
        t->ctl_pending = true;
        std::memcpy(t->h_ctl_last[slot], t->h_ctl, used);
        t->ctl_last_bytes[slot] = used;
    }
    return hipSuccess;
}

hipError_t topk_densities(TopkScratch* t, const int32_t* cols, int nk, const int64_t* sizes, int P, int L, hipStream_t s) {
    // (the last upload from this part of the pinned block is over: topk_begin waited for it)
    uint32_t* const ks = t->h_many + nk;
    for (int j = 0; j < nk; ++j) t->h_many[j] = (uint32_t)cols[j];
    bool ordered = true;
    for (int l = 0; l < L; ++l) {
        const int64_t* const z = sizes + (size_t)l * P;
        uint32_t* const k = ks + (size_t)l * nk;
        for (int j = 0; j < nk; ++j) k[j] = (uint32_t)(z[cols[j]] >> 3);
        for (int j = 1; j < nk; ++j) ordered &= k[j] != 0 && k[j] <= k[j - 1];
    }
    if (!ordered) return hipErrorInvalidValue;
    const size_t used = sizeof(uint32_t) * ((size_t)nk + (size_t)L * nk), off = t->ctl_off[4];
    if (used != t->many_last_bytes || std::memcmp(t->h_many, t->h_ctl_last[0] + off, used) != 0) {
        t->many_last_bytes = 0;
        TK_CHECK(hipMemcpyAsync(t->d_ctl[0] + off, t->h_many, used, hipMemcpyHostToDevice, s));
        TK_CHECK(hipEventRecord(t->ctl_copied, s));
        t->ctl_pending = true;
        std::memcpy(t->h_ctl_last[0] + off, t->h_many, used);
        t->many_last_bytes = used;
    }
    return hipSuccess;
}

// Upload the requested k per (layer, candidate) (0 = layer inactive) and predict the collection bound
// of every layer from a sample.
hipError_t topk_begin(TopkScratch* t, const float* g, const float* e, const DevLayer* d_layers,
                      const DevLayer* h_layers, const Tile* d_tiles, int L, int n_tiles, int tile_elems,
                      const uint32_t* ks, int ntk, int slot, Timing* tm, hipStream_t s, int nk_many) {
    (void)n_tiles;
    (void)d_tiles;
    // Tiles per work item of the refinement kernels: 2^19 elements, fewer when that would leave part of the chip
    // without a work item (see work_items.h).  An item's time has a fixed part
    // (its chain of loads, the partial histograms it clears and writes), and items past the slots start when
    // the first ones end.  The compression's partial histograms are counts of one density, 4 KB, and its items fill
    // the chip, two workgroups to a compute unit, as do those of a profile of one density.  A profile's of several are 8 KB a
    // density, 31 MB in 650 items of 6 densities,
    // which the pick reads again: one workgroup to a compute unit.  Refinement and pick, us, with items for 1024 slots, as many
    // as before (650 and 620), for 512, 256 and 128: profile of 26 M elements in 161 layers 51, 38, 32, 30, 44; of 5 M
    // in 28 34, 34, 26, 22, 21; compression of the 26 M (both levels) 27, 27, 23, 28, 41.
    int group = kRefTiles * (kTile / tile_elems);
    {
        const auto tiles_of = [&](int l) { return ks[(size_t)l * kMaxTopk] ? h_layers[l].tile_end - h_layers[l].tile_begin : 0; };
        if (nk_many) {
            // (more than kMaxTopk densities: kManySplit workgroups share an item's lists; aiming at one round of items
            // takes 55 us instead of 44, a workgroup walks its candidates for several chunks of lists)
            int64_t active = 0;
            for (int l = 0; l < L; ++l) active += tiles_of(l);
            group = (int)std::max<int64_t>(1, std::min<int64_t>(group, active * kManySplit / kRefSlots));
        } else {
            group = tiles_per_item(L, tiles_of, ntk > 1 ? kRefEnergySlots : kRefSlots, group);
        }
    }
    TK_CHECK(ctl_writable(t));
    t->nk_many = nk_many;
    int64_t base = 0;
    RefWork* const work = (RefWork*)t->h_work;
    int2* const wrange = (int2*)t->h_work_range;
    int nw = 0, max_items = 0;
    // (place[z]: items of z tiles, then where the next of them goes)
    int place[kRefTiles * (kTile / kTileMin) + 1] = {};
    for (int l = 0; l < L; ++l) {
        for (int j = 0; j < kMaxTopk; ++j) t->h_k[(size_t)l * kMaxTopk + j] = ks[(size_t)l * kMaxTopk + j];
        // the refinement relies on this order: an active layer asks for ntk values of k, none larger
        // than the one before it
        if (ks[(size_t)l * kMaxTopk])
            for (int j = 1; j < ntk; ++j)
                if (ks[(size_t)l * kMaxTopk + j] == 0 || ks[(size_t)l * kMaxTopk + j] > ks[(size_t)l * kMaxTopk + j - 1])
                    return hipErrorInvalidValue;
        t->h_cand_base[l] = base;
        wrange[l].x = nw;
        if (ks[(size_t)l * kMaxTopk]) {
            base += h_layers[l].numel;
            const int tiles = h_layers[l].tile_end - h_layers[l].tile_begin, full = tiles / group, rest = tiles % group;
            place[group] += full;
            if (rest) ++place[rest];
            nw += full + (rest > 0);
        }
        wrange[l].y = nw;
        max_items = std::max(max_items, wrange[l].y - wrange[l].x);
    }
    if (nw > t->max_work) return hipErrorInvalidValue;                   // cannot happen: see max_work
    // Items past those that start at once: the largest first, so that what is left when the first ones end is small and
    // the launch does not end with a few full ones (355 M elements in 292 layers, 1163 items: 89 -> 78 us).  By counting: there are
    // up to two a layer (a compression of 25000 layers with std::stable_sort 1696 us).
    const bool by_size = nw > kRefSlots;
    for (int z = group, at = 0; z > 0; --z) {
        const int count = place[z];
        place[z] = at;
        at += count;
    }
    for (int l = 0; l < L; ++l) {
        for (int i = wrange[l].x, t0 = h_layers[l].tile_begin; i < wrange[l].y; ++i, t0 += group) {
            const int t1 = std::min(h_layers[l].tile_end, t0 + group);
            work[by_size ? place[t1 - t0]++ : i] = RefWork{l, t0, t1, i};
        }
    }
    t->n_work = nw;
    t->max_items = max_items;
    t->cand_has_idx = false;
    TK_CHECK(upload_ctl(t, slot, s));
    Section sec(tm, "topk_sample");
    // (a kernel of the previous call, behind the last that reads it, left the exact histogram cleared)
    if (!t->hist_clean) {
        const size_t n = (size_t)t->max_layers * kHistBins;
        hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)std::min<size_t>((n + 255) / 256, 2048)), dim3(256), 0, s,
                           t->d_hist, n, 0u);
        TK_CHECK(hipGetLastError());
    }
    t->hist_clean = false;
    // A sample of half the size costs 2 to 3 us less (26 M elements in 161 layers 11.2 -> 9.1 us, 5 M in 28 10.0 -> 8.0), and
    // its wider margin lets half a per cent more elements through as candidates of 10 %: of 355 M elements that costs 6 us more than it gives.
    // In between both are within 1 % of each other wherever the line is drawn (292 layers, step of 6 densities, us, half / whole:
    // 21 M 182 / 183, 46 M 242 / 242, 77 M 320 / 319, 97 M 390 / 387, 138 M 483 / 482, 209 M 695 / 689; 28 layers of 164 M 535 / 531).
    if (base >= (int64_t)1 << 26)
        hipLaunchKernelGGL(topk_bound_kernel<32>, dim3(L), dim3(kSampleThreads), 0, s, g, e, (const uint32_t*)t->d_k, ntk,
                           d_layers, t->d_lo);
    else
        hipLaunchKernelGGL(topk_bound_kernel<16>, dim3(L), dim3(kSampleThreads), 0, s, g, e, (const uint32_t*)t->d_k, ntk,
                           d_layers, t->d_lo);
    return hipGetLastError();
}

static CollectParams collect_params(TopkScratch* t, const float* g, const float* e, const DevLayer* d_layers,
                                    const Tile* d_tiles) {
    CollectParams p{};
    p.g = g;
    p.e = e;
    p.layers = d_layers;
    p.tiles = d_tiles;
    p.ks = t->d_k;
    p.tl = (const TopkLayer*)t->d_tl;
    p.lo = t->d_lo;
    p.hist = t->d_hist;
    p.cand = t->d_cand;
    p.cand_idx = t->d_cand_idx;
    p.cand_base = t->d_cand_base;
    p.tinfo = (TopkTileInfo*)t->d_tinfo;
    p.base_part = t->d_base_part;
    return p;
}

// main pass without quantization candidates: histogram + collection in one read.  ef_out != null
// (compress): also records index and sign of every candidate and writes x to the error feedback.
hipError_t topk_collect(TopkScratch* t, const float* g, const float* e, float* ef_out, const DevLayer* d_layers,
                        const Tile* d_tiles, int n_tiles, hipStream_t s, Section* sec, float* x_out) {
    if (n_tiles <= 0) return hipSuccess;
    CollectParams p = collect_params(t, g, e, d_layers, d_tiles);
    p.ef_out = ef_out;
    p.x_out = ef_out ? nullptr : x_out;        // profile only: x is left where the compression will look for it
    // ... and that compression works from the candidates, so it needs their indices and signs
    p.record_idx = p.x_out ? 1 : 0;
    t->cand_has_idx = p.record_idx != 0;
    if (ef_out)
        launch_timed(sec, true, true, topk_collect_kernel<true, true>, dim3(n_tiles), dim3(kThreads), 0, s, p);
    else
        launch_timed(sec, true, true, topk_collect_kernel<true, false>, dim3(n_tiles), dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

// The counts of a compression are all zero, for it to add to; the emit kernel's launch makes them so again.
static hipError_t take_counts(TopkScratch* t, hipStream_t s) {
    if (!t->counts_clean) {
        const size_t n = (size_t)t->max_layers * (kBinsA + kBinsB);
        hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)std::min<size_t>((n + 255) / 256, 2048)), dim3(256), 0, s, t->d_cnt_a,
                           n, 0u);
        TK_CHECK(hipGetLastError());
    }
    t->counts_clean = false;
    return hipSuccess;
}

hipError_t topk_resolve(TopkScratch* t, const float* g, const float* e, float* ef_out, const DevLayer* d_layers,
                        const Tile* d_tiles, int L, int ntk, const int* col, double* d_errors, int stride, Timing* tm,
                        hipStream_t s, const QuantReduce* quant) {
    if (t->n_work <= 0) {
        t->hist_clean = true;
        return hipSuccess;
    }
    ScanReduce red{};
    if (quant) {
        red.partials = quant->partials;
        red.errors = quant->errors;
        red.layers = d_layers;
        red.stride = quant->stride;
        red.cols.n = std::min(quant->ncols, (int)kMaxQuant);
        for (int i = 0; i < red.cols.n; ++i) red.cols.col[i] = quant->cols[i];
    }
    if (t->nk_many) {
        Section sec(tm, "topk_scan");
        hipLaunchKernelGGL(topk_scan_many_kernel, dim3(quant ? 2 * L : L), dim3(256), 0, s, t->d_hist,
                           (const uint32_t*)t->d_many_in + t->nk_many, t->nk_many, t->d_lo, (TopkMany*)t->d_many, L, red);
        TK_CHECK(hipGetLastError());
        t->hist_clean = true;
    }
    // the pick kernel's workgroups: small ones, so that all of them run at once, unless a layer has
    // so many partial histograms to sum that its workgroup alone would outlast the rest
    const bool wide_pick = t->max_items > 64;
    RefineParams p{};
    p.tl = (TopkLayer*)t->d_tl;
    p.layers = d_layers;
    p.tiles = d_tiles;
    p.tinfo = (const TopkTileInfo*)t->d_tinfo;
    p.cand = t->d_cand;
    p.work = (const RefWork*)t->d_work;
    p.work_range = (const int2*)t->d_work_range;
    p.n_work = t->n_work;
    p.hist = t->d_hist;
    p.red = red;
    p.cand_base = t->d_cand_base;
    p.base_part = t->d_base_part;
    p.below_part = t->d_below_part;
    p.cell_a = reinterpret_cast<unsigned long long*>(t->d_ref);
    p.cnt_a = t->d_cnt_a;
    p.cnt_b = t->d_cnt_b;
    p.errors = d_errors;
    p.stride = stride;
    p.ntk = ntk;
    for (int j = 0; j < ntk; ++j) p.col[j] = col ? col[j] : 0;
    // Layers whose predicted bound was too high (none in the usual call) are collected a second time with the exact
    // bound, by the first refinement kernel's workgroups, each for its own tiles.  That reads x = g + e again; in
    // a compression e already holds x, so g is not added.
    p.rc = collect_params(t, ef_out ? ef_out : g, ef_out ? nullptr : e, d_layers, d_tiles);
    p.rc.ef_out = ef_out;
    p.rc.record_idx = (!ef_out && t->cand_has_idx) ? 1 : 0;
    Section sec(tm, "topk_refine");
    if (t->nk_many) {
        p.many = (const TopkMany*)t->d_many;
        p.cols = (const int32_t*)t->d_many_in;
        p.room = (int)std::min<size_t>((size_t)t->nk_many, many_capacity(t) / t->n_work);
        p.cell_many = reinterpret_cast<unsigned long long*>(t->d_ref);
        p.below_many = reinterpret_cast<double*>(p.cell_many + (size_t)t->n_work * p.room * kBinsA);
        static bool configured_many = false;
        const size_t lds = refine_a_lds(kManyChunk, true);
        if (!configured_many) {
            TK_CHECK(hipFuncSetAttribute((const void*)topk_refine_many_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)lds));
            configured_many = true;
        }
        for (p.list0 = 0; p.list0 < t->nk_many; p.list0 += p.room) {
            // (a pass after the first finds nothing to do unless the layers have that many lists: small grids.  100
            // densities of a 26 M-element model, about 25 lists, when the buffer held 73: 3 of a run's 245 us)
            hipLaunchKernelGGL(topk_refine_many_kernel, dim3(t->n_work, p.list0 ? 1 : kManySplit), dim3(kRefThreads), lds, s, p);
            TK_CHECK(hipGetLastError());
            hipLaunchKernelGGL(topk_pick_many_kernel, dim3(L, p.list0 ? 4 : kManySlots), dim3(256), 0, s, p);
            TK_CHECK(hipGetLastError());
        }
        return hipSuccess;
    }
    if (d_errors) {       // profile: level A gives the dropped energy, no exact threshold is needed
        const size_t lds = refine_a_lds(ntk, true);
        static bool configured[kMaxTopk + 1] = {};   // the dynamic LDS limit is raised once per variant
#define LG_REFINE_A(N)                                                                                   \
    case N:                                                                                              \
        if (!configured[N]) {                                                                            \
            TK_CHECK(hipFuncSetAttribute((const void*)topk_refine_a_kernel<N>,                           \
                                         hipFuncAttributeMaxDynamicSharedMemorySize,                      \
                                         (int)refine_a_lds(kMaxTopk, true)));                            \
            configured[N] = true;                                                                        \
        }                                                                                                \
        hipLaunchKernelGGL(topk_refine_a_kernel<N>, dim3(t->n_work + (quant ? L : 0)), dim3(kRefThreads), lds, s, p); \
        break;
        switch (ntk) {
            LG_REFINE_A(1) LG_REFINE_A(2) LG_REFINE_A(3) LG_REFINE_A(4)
            LG_REFINE_A(5) LG_REFINE_A(6) LG_REFINE_A(7) LG_REFINE_A(8)
            default: return hipErrorInvalidValue;
        }
#undef LG_REFINE_A
        TK_CHECK(hipGetLastError());
        if (wide_pick) hipLaunchKernelGGL((topk_pick_a_kernel<512>), dim3(L * ntk), dim3(512), 0, s, p);
        else hipLaunchKernelGGL((topk_pick_a_kernel<256>), dim3(L * ntk), dim3(256), 0, s, p);
        TK_CHECK(hipGetLastError());
        t->hist_clean = true;
        return hipSuccess;
    }
    if (ntk != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(topk_refine_a_kernel<0>, dim3(t->n_work), dim3(kRefThreads), refine_a_lds(ntk, false), s, p);
    TK_CHECK(hipGetLastError());
    hipLaunchKernelGGL(topk_refine_b_kernel, dim3(t->n_work), dim3(kRefThreads), 0, s, p);
    TK_CHECK(hipGetLastError());
    t->hist_clean = true;
    return hipSuccess;
}

// Sums over runs of tiles for the emission, where some layer has so many tiles that every workgroup's own sum costs
// more than this launch: emission of 1 % of one layer of 9155 tiles (300 M elements) 104 us without, 106 with; of 30518
// tiles 495 without, 426 with; of 65536 tiles 1107 and 968.
constexpr int kTilesInRuns = 10240;
static hipError_t sum_runs(TopkScratch* t, int n_tiles, int layer_tiles, hipStream_t s, const unsigned long long** runs) {
    *runs = nullptr;
    if (layer_tiles <= kTilesInRuns) return hipSuccess;
    hipLaunchKernelGGL(topk_runs_kernel, dim3((n_tiles + kRunTiles - 1) / kRunTiles), dim3(kThreads), 0, s,
                       (const uint2*)t->d_tilecnt, n_tiles, t->d_runs);
    *runs = t->d_runs;
    return hipGetLastError();
}

// x_in_e: g is the error-feedback buffer itself, which already holds x = fl32(g + e) (nothing is added)
hipError_t topk_compress(TopkScratch* t, const float* g, float* e, const DevLayer* d_layers,
                         const DevLayer* h_layers, const Tile* d_tiles, int L, int n_tiles, int tile_elems,
                         int layer_tiles, uint8_t* payload, Timing* tm, hipStream_t s, bool x_in_e) {
    std::vector<uint32_t> ks((size_t)L * kMaxTopk, 0u);
    for (int l = 0; l < L; ++l)
        if (h_layers[l].family == LGRECO_TOPK) ks[(size_t)l * kMaxTopk] = (uint32_t)h_layers[l].iparam;
    const float* const e_in = x_in_e ? nullptr : e;
    TK_CHECK(topk_begin(t, g, e_in, d_layers, h_layers, d_tiles, L, n_tiles, tile_elems, ks.data(), 1, 1, tm, s, 0));
    {
        Section sec(tm, "topk_collect", true);
        TK_CHECK(topk_collect(t, g, e_in, e, d_layers, d_tiles, n_tiles, s, &sec));
    }
    TK_CHECK(take_counts(t, s));
    TK_CHECK(topk_resolve(t, g, e_in, e, d_layers, d_tiles, L, 1, nullptr, nullptr, 0, tm, s, nullptr));
    {
        Section sec(tm, "topk_count");
        hipLaunchKernelGGL(topk_count_kernel<false>, dim3((n_tiles + kSliceBatch - 1) / kSliceBatch), dim3(kThreads), 0,
                           s, d_tiles, n_tiles, d_layers, (const uint32_t*)t->d_k, (TopkLayer*)t->d_tl, (const uint32_t*)t->d_cnt_b,
                           (const TopkTileInfo*)t->d_tinfo, (const uint32_t*)t->d_cand, (uint2*)t->d_tilecnt);
        TK_CHECK(hipGetLastError());
    }
    {
        Section sec(tm, "topk_emit");
        const unsigned long long* runs;
        TK_CHECK(sum_runs(t, n_tiles, layer_tiles, s, &runs));
        hipLaunchKernelGGL(topk_emit_kernel<false>, dim3((n_tiles + kSliceBatch - 1) / kSliceBatch), dim3(kThreads), 0, s, e,
                           d_layers, d_tiles, n_tiles, (const TopkLayer*)t->d_tl,
                           (const TopkTileInfo*)t->d_tinfo, (const uint32_t*)t->d_cand,
                           (const uint32_t*)t->d_cand_idx, (const uint2*)t->d_tilecnt, runs,
                           t->d_cnt_a, t->d_cnt_b, payload, 0);
        TK_CHECK(hipGetLastError());
        t->counts_clean = true;
    }
    return hipSuccess;
}

// Compression of the Top-K layers right behind a profile of the same data (the one-call entry
// point): the layer records the solver kernel wrote say which layers take part and which of the
// profile's selection records (threshold bin, sub-bin, entries to take) applies, so nothing is
// sampled, no histogram is built and nothing depends on the host knowing the assignment.
// x_in_e (the profile left x in the error-feedback buffer and recorded where its candidates are):
// what lies at or above the sub-bin's lower edge is taken from the profile's candidates, the
// sub-bin's entries counted by their last 9 bits, and the data is not read at all.  Otherwise one
// pass over g and e writes x to the error feedback and collects the same set.  Then the exact
// threshold, the per-wavefront counts and the ordered emit, as in topk_compress.
hipError_t topk_compress_known(TopkScratch* t, const float* g, float* e, const DevLayer* d_layers,
                               const Tile* d_tiles, int L, int n_tiles, int layer_tiles, uint8_t* payload, Timing* tm,
                               hipStream_t s, bool x_in_e) {
    if (n_tiles <= 0) return hipSuccess;
    // the profile's control block (slot 0) holds every layer's candidate region
    uint8_t* const d = t->d_ctl[0];
    CollectParams p{};
    p.g = g;
    p.e = e;
    p.ef_out = e;
    p.layers = d_layers;
    p.tiles = d_tiles;
    p.tl = (const TopkLayer*)t->d_tl;
    p.cand = t->d_cand;
    p.cand_idx = t->d_cand_idx;
    p.cand_base = reinterpret_cast<const int64_t*>(d + t->ctl_off[1]);
    p.tinfo = (TopkTileInfo*)t->d_tinfo;
    p.base_part = t->d_base_part;
    p.cnt_b = t->d_cnt_b;
    const TopkTileInfo* tinfo = (const TopkTileInfo*)t->d_tinfo;
    const uint32_t* cand = t->d_cand;
    const uint32_t* cand_idx = t->d_cand_idx;
    if (x_in_e && !t->cand_has_idx) return hipErrorInvalidValue;
    TK_CHECK(take_counts(t, s));
    if (x_in_e) {
        // the profile recorded where its candidates are: what is kept is taken from them
        FilterParams f{};
        f.layers = d_layers;
        f.tiles = d_tiles;
        f.tl = p.tl;
        f.cand_base = p.cand_base;
        f.tinfo = tinfo;
        f.cand = cand;
        f.cand_idx = cand_idx;
        f.tinfo_out = (TopkTileInfo*)t->d_tinfo_kept;
        f.cand_out = t->d_kept;
        f.cand_idx_out = t->d_kept_idx;
        f.cnt_b = t->d_cnt_b;
        Section sec(tm, "topk_filter", true);
        launch_timed(&sec, true, true, topk_filter_known_kernel, dim3(n_tiles), dim3(kThreads), 0, s, f);
        TK_CHECK(hipGetLastError());
        tinfo = f.tinfo_out;
        cand = f.cand_out;
        cand_idx = f.cand_idx_out;
    } else {
        Section sec(tm, "topk_collect", true);
        launch_timed(&sec, true, true, topk_collect_known_kernel, dim3(n_tiles), dim3(kThreads), 0, s, p);
        TK_CHECK(hipGetLastError());
    }
    {
        Section sec(tm, "topk_count");
        hipLaunchKernelGGL(topk_count_kernel<true>, dim3((n_tiles + kSliceBatch - 1) / kSliceBatch), dim3(kThreads), 0,
                           s, d_tiles, n_tiles, d_layers, (const uint32_t*)nullptr, (TopkLayer*)t->d_tl, (const uint32_t*)t->d_cnt_b,
                           tinfo, cand,
                           (uint2*)t->d_tilecnt);
        TK_CHECK(hipGetLastError());
    }
    {
        Section sec(tm, "topk_emit");
        const unsigned long long* runs;
        TK_CHECK(sum_runs(t, n_tiles, layer_tiles, s, &runs));
        hipLaunchKernelGGL(topk_emit_kernel<true>, dim3((n_tiles + kSliceBatch - 1) / kSliceBatch), dim3(kThreads), 0, s, e,
                           d_layers, d_tiles, n_tiles, (const TopkLayer*)t->d_tl, tinfo, cand, cand_idx,
                           (const uint2*)t->d_tilecnt, runs,
                           t->d_cnt_a, t->d_cnt_b, payload, x_in_e ? 1 : 0);
        TK_CHECK(hipGetLastError());
        t->counts_clean = true;
    }
    return hipSuccess;
}

}  // namespace lgreco
