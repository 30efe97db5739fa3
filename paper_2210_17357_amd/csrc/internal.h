// Interfaces between the translation units of liblgreco.so (host side).
#pragma once

#include <algorithm>
#include <cstring>
#include <vector>

#include <hip/hip_ext.h>

#include "common.h"

namespace lgreco {

// Optional per-kernel timing.  A Section covers the work enqueued during its lifetime with two HIP
// events of the call's stream.  A main-kernel section (the level-1 sections a benchmark keeps on
// inside its timed region) puts its events on the kernels themselves: launch_timed below hands
// the start event to the section's first kernel and the stop event to its last one, and
// hipExtLaunchKernelGGL takes the kernel's own begin and end timestamps, so the figure is the
// kernels' time without launch gaps.  The other sections record their events as separate stream
// operations.  Either way a timed kernel leaves about 5 us of the stream idle on either side
// (measured), which is why a call kind can be timed every n-th call only.
struct Timing {
    static constexpr int kMaxSections = 32;
    int level = 0;          // 0 off, 1 main kernels, 2 every section
    int every = 1;          // only every `every`-th call of this kind is timed
    int64_t calls = 0;      // calls of this kind since the level was set
    bool active = false;    // the call in progress is one of the timed ones
    bool ready = false;
    hipStream_t stream = nullptr;
    hipEvent_t ev[2 * kMaxSections]{};
    const char* name[kMaxSections]{};
    int n = 0;
    // Read-out: the events of the last call are turned into milliseconds once ("harvested"), at a
    // moment when the host has nothing better to do, and added to the totals since the level was set.
    bool harvested = true;
    float ms[kMaxSections]{};
    static constexpr int kMaxNames = 48;
    const char* total_name[kMaxNames]{};
    double total_ms[kMaxNames]{};
    int64_t total_count[kMaxNames]{};
    int n_totals = 0;
    // A phase bracket: two recorded events around everything a call (or a part of it) queues,
    // kept at level 1 like the main kernels.  Opened and closed by hand because one phase can
    // span two functions (the compression whose first kernel is queued behind the solver).
    int open_phase(const char* nm) {
        if (!(active && level >= 1 && ready && n < kMaxSections)) return -1;
        const int idx = n++;
        name[idx] = nm;
        (void)hipEventRecord(ev[2 * idx], stream);
        return idx;
    }
    void close_phase(int idx) {
        if (idx >= 0) (void)hipEventRecord(ev[2 * idx + 1], stream);
    }
    void add_total(const char* nm, double v) {
        int i = 0;
        while (i < n_totals && total_name[i] != nm && std::strcmp(total_name[i], nm) != 0) ++i;
        if (i == n_totals) {
            if (n_totals == kMaxNames) return;
            total_name[n_totals++] = nm;
            total_ms[i] = 0.0;
            total_count[i] = 0;
        }
        total_ms[i] += v;
        total_count[i] += 1;
    }
};
struct Section {
    Timing* t;
    int idx = -1;
    bool on_kernels = false;            // events are bound to kernels, not recorded
    bool start_taken = false, stop_taken = false;
    Section(Timing* tt, const char* name, bool main_kernel = false) : t(tt) {
        if (t && t->active && t->level >= (main_kernel ? 1 : 2) && t->ready && t->n < Timing::kMaxSections) {
            idx = t->n++;
            t->name[idx] = name;
            on_kernels = main_kernel;
            if (!on_kernels) (void)hipEventRecord(t->ev[2 * idx], t->stream);
        }
    }
    ~Section() {
        if (idx < 0) return;
        if (!on_kernels) {
            (void)hipEventRecord(t->ev[2 * idx + 1], t->stream);
        } else if (!start_taken && !stop_taken) {
            // nothing was launched inside: an empty bracket
            (void)hipEventRecord(t->ev[2 * idx], t->stream);
            (void)hipEventRecord(t->ev[2 * idx + 1], t->stream);
        } else if (!stop_taken) {
            (void)hipEventRecord(t->ev[2 * idx + 1], t->stream);
        }
    }
    hipEvent_t start_event() {
        if (idx < 0 || !on_kernels || start_taken) return nullptr;
        start_taken = true;
        return t->ev[2 * idx];
    }
    hipEvent_t stop_event() {
        if (idx < 0 || !on_kernels) return nullptr;
        stop_taken = true;
        return t->ev[2 * idx + 1];
    }
    Section(const Section&) = delete;
    Section& operator=(const Section&) = delete;
};

// Kernel launch inside a main-kernel section (sec may be null = plain launch): `first` / `last`
// say whether this is the section's first / last kernel.
template <typename... P, typename... A>
inline void launch_timed(Section* sec, bool first, bool last, void (*kernel)(P...), dim3 grid, dim3 block,
                         size_t lds, hipStream_t s, A&&... args) {
    static_assert(sizeof...(P) == sizeof...(A), "one argument per kernel parameter");
    hipEvent_t a = (sec && first) ? sec->start_event() : nullptr;
    hipEvent_t b = (sec && last) ? sec->stop_event() : nullptr;
    if (a || b)
        hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)lds, s, a, b, 0u, static_cast<P>(args)...);
    else
        hipLaunchKernelGGL(kernel, grid, block, lds, s, static_cast<P>(args)...);
}

// ---- quant.hip
// sec (may be null): the main-kernel section the launch belongs to
hipError_t launch_quant_profile(const QuantParams& p, int n_tiles, bool hist, hipStream_t s, Section* sec);
hipError_t launch_reduce_partials(const double* partials, int stride, const int* cols, int ncols,
                                  const DevLayer* layers, int n_layers, double* errors, hipStream_t s);
hipError_t launch_quant_compress(const float* g, float* e, const DevLayer* layers, const Tile* tiles, int n_tiles,
                                 int tile_elems, int64_t quantized, int64_t total, uint8_t* payload, bool stochastic,
                                 uint64_t seed, hipStream_t s, Section* sec, size_t lds_pad = 0);   // lds_pad: LDS bytes requested and not used

// ---- dp.hip
struct DpEntry {            // one usable candidate of a layer (equal bins merged by the host)
    int32_t bin;
    int32_t cand;
    int64_t size;
};
// Layer groups swept side by side (dp_group_kernel) and joined pairwise (dp_conv_kernel): a
// complete binary tree in heap order, node 0 the whole table, leaves G-1 .. 2G-2 the groups in
// layer order, the left child of a node holding the lower layers.
struct DpGroups {
    int32_t G = 0;                // in: 0 = let launch_dp decide, 1 = off, 2 / 4 / 8 = forced; out: groups used (0 / 1: none)
    int32_t stride = 0;           // cells per node array (set by launch_dp, > D)
    uint32_t* nodes = nullptr;    // [(2G-1) x stride] smallest size of a node's layers per exact bin sum (null: groups off)
    int32_t* range = nullptr;     // [G x 2] swept layers [begin, end) of every group, written by the group sweeps
    int32_t* flag = nullptr;      // [1] written by dp_trace_kernel: 1 = it gave up, the sequential kernel behind it solves
};
struct DpParams {
    const DpEntry* entries;   // [L x max_count] swept layers only, in candidate order
    const int32_t* count;     // [L] entries per swept layer
    uint8_t* pd;              // [L x pd_stride] entry index per cell
    int32_t* choice;          // [L] candidate index per swept layer
    int64_t* result;          // [0] status (0 ok, 1 infeasible), [1] swept size, [2] final bin sum
    int32_t L, D;
    int32_t pad;              // set by launch_dp: cells of infinity in front of the LDS row
    int32_t pd_stride;        // set by launch_dp: bytes per PD row, a multiple of 4 and >= D + 2
    int32_t bt_lds;           // set by launch_dp: back-trace tables live in LDS behind the row
    int32_t max_count;        // largest entry count of a swept layer = row stride of `entries`
    // The input block (count | entries) as the host wrote it in pinned memory and its place in
    // device memory: the kernel's first step copies it over (in_vec 16-byte words), which saves
    // the separate copy operation and the wait between it and the kernel.  Null: nothing to copy.
    const uint4* host_in;
    uint4* dev_in;
    int32_t in_vec;
    // Written to result[7] as the kernel's last store (after a system-scope fence): the host
    // may poll the pinned result block for it instead of waiting for the stream.
    int64_t seq;
    DpGroups groups;
    // The traced-back assignment starts from the best cell among 0 .. min(D, e_limit) of the last
    // row (the strict budget looks at fewer cells than the table has; negative: none, no
    // assignment fits).
    int32_t e_limit = 0x7FFFFFFF;
};
// narrow: 32-bit costs (sum of the layers' largest sizes < 2^30)
// max_bin: largest bin in entries
// sec (may be null): the section's last kernel, and its first one too when `first_in_section`
hipError_t launch_dp(const DpParams& p, bool narrow, int max_bin, hipStream_t s, Section* sec,
                     bool first_in_section);

// ---- solve.hip: the whole solve from the error table as one kernel
constexpr int kSolveMaxLayers = 1024;
constexpr int kSolveMaxLP = 16384;      // table entries (layers x candidates)
constexpr int kSolveMaxEntries = 4096;  // entries left after dropping unusable and beaten candidates (more: status 4)
// Optional last step: the per-layer records the compression kernels read (family, parameter, payload
// offset), so that a compression queued right behind the solver needs nothing from the host.  The
// tables hold, per (layer, candidate), what the host would compute for that choice.  If the solve
// fails or the layout does not fit `capacity`, every record gets family -1 (no compression kernel
// touches such a layer) and result[8] stays 0; otherwise result[8] = 1.
struct SolveApply {
    DevLayer* layers;             // null: off
    const int32_t* iparam;        // [L x P] bits / k / rank
    const int32_t* family;        // [P]
    const int32_t* topk_slot;     // [P] position of a Top-K candidate in the profile's selection records, else -1
    int64_t capacity;             // bytes the payload buffer holds
};
struct SolveParams {
    const double* errors;         // [L x P], device memory or the host's pinned memory as the device addresses it
    const int64_t* sizes;         // [L x P]; the layers' largest sizes sum to less than 2^30
    const uint8_t* order;         // [L x P] per layer its candidates in order of size, lowest index first among equals
                                  // (null: sorted by the kernel, at most 4096 table entries)
    double* errors_host;          // [L x P] the host's pinned copy of the error table, written here (may be null)
    int32_t L, P, D;
    int32_t default_cand;         // E_max = sum of this candidate's errors ...
    int32_t have_e_max;           // ... unless the caller gives it
    double e_max;
    int32_t e_limit;              // the bins of an accepted assignment sum to at most min(D, e_limit)
    int32_t last_resort;          // 1: the caller has nothing to fall back to (at most 4096 table entries, 64 candidates)
    int32_t check_sizes;          // 1: reject (status 3) sizes this path's 32-bit costs cannot hold
    int32_t* choice;              // out [L] candidate per layer, -1 when not solved
    int64_t* result;              // out [16]: [0] status (0 ok, 1 infeasible, 2 inconsistent, 3 invalid input, 4 not
                                  //      taken here: more than kSolveMaxEntries candidates left, or rows that do not fit
                                  //      beside them, see last_resort), [1] size and [2] bins of the layers that were not fixed at
                                  //      bin 0, [3] ticks, [5] L, [6] bit pattern of E_max, [8] records written, [9] 0,
                                  //      [10] / [11] check words over choice / error table, [4], [15] and, last, [7] seq
    int64_t seq;
    uint8_t* pd;                  // device memory, L x (D + 1) bytes: arg-min table where LDS does not hold it
    SolveApply apply;
};
hipError_t launch_solve(const SolveParams& p, hipStream_t s, Section* sec);

// ---- topk.hip
struct TopkScratch {
    uint32_t* d_hist = nullptr;       // [max_layers x kHistBins] exact coarse histogram
    void* d_tl = nullptr;             // per-layer selection records
    uint32_t* d_cnt_a = nullptr;      // [max_layers x 1024] counts of a compression inside the threshold bin, and
    uint32_t* d_cnt_b = nullptr;      // [max_layers x 512] inside the boundary sub-bin
    bool counts_clean = false;        // both are all zero (the last kernel of a compression clears them)
    uint32_t* d_cand = nullptr;       // bit patterns of the candidates, tile i at its own first element
    uint32_t* d_cand_idx = nullptr;   // compress: index within the layer (+ sign bit) of every candidate; a profile that
                                      // records where its candidates are uses it for 16-bit entries (place in tile, sign)
    bool cand_has_idx = false;        // the current call's profile recorded d_cand_idx too
    // compression from the profile's candidates: what is kept of them, in element order (behind the partial histograms)
    uint32_t* d_kept = nullptr;
    uint32_t* d_kept_idx = nullptr;
    void* d_tinfo_kept = nullptr;
    uint32_t* d_k = nullptr;          // [max_layers x kMaxTopk] requested k (0 = layer inactive)
    uint32_t* d_lo = nullptr;         // [max_layers] lowest coarse key collected as a candidate
    bool hist_clean = false;          // the exact histogram is all zero (a kernel behind the search of every call clears it)
    int64_t* d_cand_base = nullptr;   // [max_layers] first candidate slot of every layer
    void* d_tilecnt = nullptr;        // per tile (above, equal) counts (compress)
    unsigned long long* d_runs = nullptr;   // ... and their sums over runs of tiles
    void* d_tinfo = nullptr;          // per tile, per wavefront: candidates written and where
    double* d_base_part = nullptr;    // per tile energy below the collection bound
    double* d_below_part = nullptr;   // refinement partial sums
    void* d_ref = nullptr;            // per-workgroup refinement histograms (counts, integer energies)
    size_t ref_bytes = 0;             // with d_kept and d_kept_idx behind them
    // control block, one upload per call and none when it repeats the last one:
    // [k | cand_base | work_range | work], then [many], uploaded on its own; the pointers above and below are views into it
    // (two device copies: profile calls and compress calls alternate and each repeats itself)
    uint8_t* d_ctl[2] = {nullptr, nullptr};
    uint8_t* h_ctl = nullptr;         // pinned
    hipEvent_t ctl_copied = nullptr;  // recorded behind every upload from h_ctl
    bool ctl_pending = false;         // an upload was queued since h_ctl was last known to be free
    uint8_t* h_ctl_last[2] = {nullptr, nullptr};    // what each d_ctl holds
    size_t ctl_bytes = 0, ctl_last_bytes[2] = {0, 0}, many_last_bytes = 0;
    size_t ctl_off[5] = {};           // byte offsets of k, cand_base, work_range, work, many
    // more than kMaxTopk densities in one profile
    uint32_t* h_many = nullptr;       // (in the control block) column of every density, then k per (layer, density)
    uint32_t* d_many_in = nullptr;
    int nk_many = 0;                  // densities of the current call, 0: at most kMaxTopk
    void* d_many = nullptr;           // per-layer records
    void* d_work = nullptr;           // refinement work table and per-layer ranges
    void* d_work_range = nullptr;
    void* h_work = nullptr;
    void* h_work_range = nullptr;
    int max_work = 0, n_work = 0;
    int max_items = 0;          // most work items of one layer in the current call
    uint32_t* h_k = nullptr;
    int64_t* h_cand_base = nullptr;
    int64_t max_elems = 0;
    int max_layers = 0, max_tiles = 0;
};
hipError_t topk_scratch_create(TopkScratch* t, int64_t max_elems, int max_layers, int max_tiles, int max_cands);
void topk_scratch_destroy(TopkScratch* t);
// Upload k per (layer, candidate), sample the data and predict every layer's collection bound.
// nk_many: more than kMaxTopk densities, so many (ks holds the largest alone); topk_densities brings them.
hipError_t topk_begin(TopkScratch* t, const float* g, const float* e, const DevLayer* d_layers,
                      const DevLayer* h_layers, const Tile* d_tiles, int L, int n_tiles, int tile_elems,
                      const uint32_t* ks, int ntk, int slot, Timing* tm, hipStream_t s, int nk_many);
// More than kMaxTopk densities: upload their columns, the largest density first, and k per (layer, density) from the
// size table (8 k bytes).  What comes before topk_resolve does not need them: the host works them out while it runs.
hipError_t topk_densities(TopkScratch* t, const int32_t* cols, int nk, const int64_t* sizes, int P, int L, hipStream_t s);
// main pass (exact coarse histogram + candidate collection) when no quantization candidate shares
// the read; otherwise the quantization profile kernel does the same work
hipError_t topk_collect(TopkScratch* t, const float* g, const float* e, float* ef_out, const DevLayer* d_layers,
                        const Tile* d_tiles, int n_tiles, hipStream_t s, Section* sec, float* x_out = nullptr);
// quant (may be null): the quantization profile's per-tile partial sums, reduced per layer by extra
// workgroups of a launch that depends on the main pass only, instead of a kernel of their own
struct QuantReduce {
    const double* partials;
    double* errors;
    int stride;
    const int* cols;
    int ncols;
};
// Behind the main pass: threshold bins from the histogram (layers whose predicted bound was too high are
// collected again with the exact one), then the refinement on the candidates.  Profile: the dropped energy to d_errors.
// Compression (d_errors null, one density; ef_out holds x): the boundary sub-bin and its counts, which the exact threshold follows from.
hipError_t topk_resolve(TopkScratch* t, const float* g, const float* e, float* ef_out, const DevLayer* d_layers,
                        const Tile* d_tiles, int L, int ntk, const int* col, double* d_errors, int stride, Timing* tm,
                        hipStream_t s, const QuantReduce* quant);
// layer_tiles: tiles of the largest layer
hipError_t topk_compress(TopkScratch* t, const float* g, float* e, const DevLayer* d_layers,
                         const DevLayer* h_layers, const Tile* d_tiles, int L, int n_tiles, int tile_elems,
                         int layer_tiles, uint8_t* payload, Timing* tm, hipStream_t s, bool x_in_e = false);

// Top-K layers of a compression queued right behind a profile of the same data and the solver
// kernel that wrote the layer records (family, k, payload offset, slot of the chosen density in
// the profile's selection records): nothing here needs the host to know the assignment.
hipError_t topk_compress_known(TopkScratch* t, const float* g, float* e, const DevLayer* d_layers,
                               const Tile* d_tiles, int L, int n_tiles, int layer_tiles, uint8_t* payload, Timing* tm,
                               hipStream_t s, bool x_in_e = false);

// ---- lowrank.hip
struct LowrankScratch {
    void* host = nullptr;        // work tables and scratch buffers (grown on demand)
    int64_t max_elems = 0;
    int max_layers = 0, r_max = 0, power_iters = 1;
};
hipError_t lowrank_scratch_create(LowrankScratch* t, int64_t max_elems, int max_layers, int r_max,
                                  int power_iters);
void lowrank_scratch_destroy(LowrankScratch* t);
// x: room for the layers' elements, where g + e is left (e not null) for the passes behind the first and for a
// compression that follows on the same data
hipError_t lowrank_profile(LowrankScratch* t, const float* g, const float* e, const DevLayer* d_layers,
                           const DevLayer* h_layers, int L, const float* q0, int r_max, const int* rank,
                           const int* col, int nlr, double* d_errors, int stride, float* x, Timing* tm, hipStream_t s);
hipError_t lowrank_compress(LowrankScratch* t, const float* g, float* e, const DevLayer* d_layers,
                            const DevLayer* h_layers, int L, float* q, int r_max, uint8_t* payload, Timing* tm,
                            hipStream_t s);
// low-rank layers of a compression queued right behind a profile of the same data (see topk_compress_known)
hipError_t lowrank_compress_known(LowrankScratch* t, const float* g, float* e, const DevLayer* d_layers, float* q,
                                  int r_max, uint8_t* payload, const float* x, Timing* tm, hipStream_t s,
                                  bool e_is_zero = false);   // e_is_zero: e holds zeros on entry (the caller's promise) and is not read
// receiver side: out (+)= Phat Q^T from the payload
hipError_t lowrank_decompress(LowrankScratch* t, const DevLayer* h_layers, int L, int r_max, const uint8_t* payload,
                              float* out, bool accumulate, Timing* tm, hipStream_t s);

// ---- decode.hip: receiver side of quantization and Top-K, gradient accumulation
hipError_t launch_accumulate(float* acc, const float* g, int64_t n, bool reset, hipStream_t s, Section* sec);
// quantized: elements of the quantized layers, of total
hipError_t launch_decode(const uint8_t* payload, const DevLayer* layers, const Tile* tiles, int n_tiles, int tile_elems,
                         int64_t quantized, int64_t total, float* out, bool accumulate, bool any_topk, Timing* tm, hipStream_t s);

}  // namespace lgreco
