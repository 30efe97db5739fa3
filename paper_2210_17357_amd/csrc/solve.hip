// Algorithm 1 from the error table to the traced-back assignment as one kernel of one workgroup:
// E_max, bins, the layers' candidate lists, the dynamic program and its back-trace, and (for a
// compression queued behind it) the layer records the compression kernels read.  gfx950 / wave64.
//
// What Algorithm 1 returns is the assignment that is first in the order (sum of sizes, sum of bins,
// c_L, ..., c_1) among those whose bins sum to at most D: strict '<' over candidates in index
// order, lowest e among equal minima at the end.  The sweep below fills only those cells of the
// table an assignment of the smallest total size can pass through:
//   * a feasible assignment gives an upper bound UB of the total size;
//   * for any multiplier v >= 0 the layers [0, l) cost at least F_v(l) - v e when their bins sum to
//     e, F_v(l) = sum of min_c (size + v bin) over them, and the layers from l on at least
//     S_v(l) - v (D - e) with S_v(l) the same sum over those.  A cell (l, e) where the two add up to
//     more than UB lies on no assignment of the smallest size.  With one of the two multipliers
//     at the value v* where the relaxed assignment just fits and the other on either side of it,
//     the test is linear in e and leaves one interval of e per layer boundary;
//   * a candidate whose reduced cost size + v* bin - min_c (..) lifts the relaxed bound above UB, or
//     that leads from no cell of one interval into the next, is dropped; a layer left with one
//     candidate only shifts the row and takes no step of the sweep.
// Every assignment of the smallest size keeps all its cells and candidates (the tests drop what is
// strictly worse, with a margin for rounding), so minima, ties and tie-breaks along them are those
// of the full table.  Measured on tables of the profiled models: intervals of 20 to 500 of 1000 to
// 10000 bins, 10 to 80 layers of up to 300 left to sweep, 2 to 4 candidates each: the full sweep's
// work divided by 5 (few layers) to 5000 (49 or 100 candidates per layer).
//
// One workgroup, because every step needs the step before it: what bounds this kernel is the
// chain of LDS round trips and barriers, not their number of operations.  So the order of the candidates comes with the
// table into LDS (read from device or host memory list by list it was a round trip for every group of lists: 11 of 53 us on
// 163 layers of 49 candidates, now 2.6), sums over the block that do not depend on each other share a barrier, and
// sums and minima over a wavefront move in registers.  Whole kernel, before and after: 163 x 49 candidates in 10000 bins 53 ->
// 43 us, 292 x 13 in 4000 54 -> 51, 161 x 6 in 1000 25 -> 22, 62 x 7 in 1000 22.3 -> 20.6, 16 x 7 in 50 12.6 -> 11.3.
// (A reciprocal and a test in place of the bins' divisions: nothing gained, 1 us lost on the 292 layers.)
#include "internal.h"

namespace lgreco {

namespace {

constexpr int kThreadsS = 1024;
constexpr int kWavesS = kThreadsS / 64;
constexpr int kMaxLayersS = kSolveMaxLayers;
constexpr int kMaxT = kSolveMaxEntries;
constexpr uint32_t kUnusable = 0xFFFFu;      // bin of a candidate whose error exceeds the budget (bins are at most 16384)
constexpr uint32_t kInfS = 1u << 30;
constexpr int kMaxRow = 17 * kThreadsS;      // cells of a row: at least LGRECO_MAX_BINS + 1
constexpr int kRowCells = 4096;              // past this many bins intervals are worked out in any case
constexpr size_t kRegionBytes = (size_t)kSolveMaxLP * 6;      // LDS: the table's bins and sizes, later see Relax and Core

// ---- wavefront scans and reductions on DPP (no LDS round trips)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or0(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = dpp_or0<CTRL, ROWS>((uint32_t)b), hi = dpp_or0<CTRL, ROWS>((uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_or0(unsigned long long b) {
    const uint32_t lo = dpp_or0<CTRL, ROWS>((uint32_t)b), hi = dpp_or0<CTRL, ROWS>((uint32_t)(b >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
// inclusive sum over the lanes up to this one: row_shr 1, 2, 4, 8, then the rows' totals carried on
template <typename T>
__device__ __forceinline__ T wave_scan(T v) {
    v += dpp_or0<0x111, 0xF>(v);
    v += dpp_or0<0x112, 0xF>(v);
    v += dpp_or0<0x114, 0xF>(v);
    v += dpp_or0<0x118, 0xF>(v);
    v += dpp_or0<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
    v += dpp_or0<0x143, 0xC>(v);      // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, ((uint64_t)lane_u32((uint32_t)(b >> 32), lane) << 32) | lane_u32((uint32_t)b, lane));
}
__device__ __forceinline__ uint32_t wave_total(uint32_t v) { return lane_u32(wave_scan(v), 63); }
__device__ __forceinline__ double wave_total(double v) { return lane_f64(wave_scan(v), 63); }
__device__ __forceinline__ unsigned long long wave_total(unsigned long long v) {
    v = wave_scan(v);
    return ((unsigned long long)lane_u32((uint32_t)(v >> 32), 63) << 32) | lane_u32((uint32_t)v, 63);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, dpp_or0<0x111, 0xF>(v));
    v = max(v, dpp_or0<0x112, 0xF>(v));
    v = max(v, dpp_or0<0x114, 0xF>(v));
    v = max(v, dpp_or0<0x118, 0xF>(v));
    v = max(v, dpp_or0<0x142, 0xA>(v));
    v = max(v, dpp_or0<0x143, 0xC>(v));
    return lane_u32(v, 63);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) { return ~wave_max_u32(~v); }

// value CTRL lanes below inside the row of 16 (row_shr), all ones where there is none
template <int CTRL>
__device__ __forceinline__ uint32_t min16(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, 0xF, 0xF, false);
}
// smallest value of the lanes below this one (all ones for lane 0)
__device__ __forceinline__ uint32_t wave_min_before(uint32_t v) {
    uint32_t m = v;
    m = min(m, min16<0x111>(m));
    m = min(m, min16<0x112>(m));
    m = min(m, min16<0x114>(m));
    m = min(m, min16<0x118>(m));
    m = min(m, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)m, 0x142, 0xA, 0xF, false));
    m = min(m, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)m, 0x143, 0xC, 0xF, false));
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)m, 0x138, 0xF, 0xF, false);      // wave_shr:1
}

// Exclusive sum over the block, one value per thread; *total = sum of all.  Two barriers.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* s_tmp, uint32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t inc = wave_scan(v);
    __syncthreads();
    if (lane == 63) s_tmp[wave] = inc;
    __syncthreads();
    const uint32_t t = wave_scan(lane < kWavesS ? s_tmp[lane] : 0u);
    *total = lane_u32(t, kWavesS - 1);
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
    return inc - v + (w ? lane_u32(t, (int)w - 1) : 0u);
}

// The same for two values, through a table nothing else uses: one barrier.
__device__ __forceinline__ void block_scan2(uint32_t a, uint32_t b, uint32_t (*s_tmp)[kWavesS], uint32_t* before_a,
                                            uint32_t* before_b, uint32_t* total_a, uint32_t* total_b) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ia = wave_scan(a), ib = wave_scan(b);
    if (lane == 63) {
        s_tmp[0][wave] = ia;
        s_tmp[1][wave] = ib;
    }
    __syncthreads();
    const uint32_t ta = wave_scan(lane < kWavesS ? s_tmp[0][lane] : 0u), tb = wave_scan(lane < kWavesS ? s_tmp[1][lane] : 0u);
    *total_a = lane_u32(ta, kWavesS - 1);
    *total_b = lane_u32(tb, kWavesS - 1);
    *before_a = ia - a + (wave ? lane_u32(ta, wave - 1) : 0u);
    *before_b = ib - b + (wave ? lane_u32(tb, wave - 1) : 0u);
}

struct alignas(16) Lds {
    union {
        double def[kMaxLayersS];             // the default candidate's errors, until E_max is known
        int32_t first[kMaxLayersS];          // first entry of a swept layer, by layer (-1: not swept)
    };
    // entries of the swept layers, layer after layer, largest bin first (hence smallest size first)
    union {
        uint32_t size[kMaxT];
        uint8_t order[kSolveMaxLP];          // before that: the table's candidates in order of size
    };
    uint16_t bin[kMaxT];
    uint16_t of[kMaxT];                      // swept layer of an entry
    uint8_t cand[kMaxT];
    int32_t off[kMaxLayersS + 1];            // first entry of every swept layer
    union {
        struct {
            int32_t lo[kMaxLayersS + 1], hi[kMaxLayersS + 1];   // interval of e at every layer boundary
        };
        uint64_t list[kMaxLayersS];          // before that: candidates kept, one word of bits per layer (two where P > 64)
    };
    uint16_t layer[kMaxLayersS];             // swept layer -> layer
    uint8_t pick[kMaxLayersS];               // core layer -> picked survivor
    uint8_t mixed[kMaxLayersS];              // 1: the layer's list is not in order of bins and sizes
    uint8_t chosen[kMaxLayersS];             // candidate per layer; 255: none
    uint64_t keep[kMaxT / 64];               // one bit per entry: hull vertices, then survivors
    uint32_t before[kMaxT / 64];             // bits of `keep` set in front of every word
    uint32_t tmp[kWavesS], tmp2[2][2][kWavesS];
    double tmp_d[kWavesS];
    unsigned long long worst;                // sum of the layers' largest sizes
    unsigned long long chk_err, chk_choice;
    unsigned long long best;                 // smallest total and its cell
    unsigned long long sums;                 // of the assignment: bins << 32 | sizes
    double total_star;
    double emax;
    uint32_t ub;
    int32_t flags;                           // 1: a layer without usable candidate, 2: invalid input, 4 and up: inconsistent
    uint32_t acc[4];
    uint32_t facts[4];                       // of the core layers: furthest shift down and up, longest list, sum of their largest sizes
};
// what the region holds while the intervals are worked out ...
struct Relax {
    double slope[kMaxT];                     // hull vertices: size saved per bin on the way to the next larger bin
    double star[kMaxLayersS];                // relaxed minimum of every swept layer at v*
    double prefix[kMaxLayersS];              // their running sum
    uint32_t hist[1024];
    uint16_t vertex[kMaxT];                  // entry of every hull vertex
    uint16_t hoff[kMaxLayersS + 1];          // first hull vertex of every swept layer
    uint8_t pick[kWavesS][kMaxLayersS];      // one assignment per wavefront
};
// ... and, in front of the rows, during the sweep: one record per core layer, and its survivors in
// candidate order, in groups of four (filled up with entries that never win)
struct Core {
    int32_t step;                            // cells from the first cell of the row before to this row's first cell
    int32_t lo;                              // the row's first cell
    uint32_t shape;                          // cells of this row | survivors << 16
    int32_t trace;                           // place of the row's first arg-min byte
};

// number of bits of s.keep set in front of position t
__device__ __forceinline__ uint32_t bits_before(const Lds& s, int t) {
    return s.before[t >> 6] + (uint32_t)__popcll(s.keep[t >> 6] & ((1ull << (t & 63)) - 1ull));
}
// s.before from s.keep over n positions: the first wavefront; barriers on both sides are the caller's
__device__ __forceinline__ void count_bits(Lds& s, int n) {
    const int lane = threadIdx.x & 63;
    const uint32_t c = lane * 64 < n ? (uint32_t)__popcll(s.keep[lane]) : 0u;
    s.before[lane] = wave_scan(c) - c;
}

// Relaxed choice of swept layer i at multiplier v: the hull vertex whose way on to the next larger bin
// saves no more than v per bin, the last such in the list (slopes rise along it).  Returns the entry.
__device__ __forceinline__ int relaxed_pick(const Relax& r, int i, double v) {
    int a = r.hoff[i], b = r.hoff[i + 1];        // slope[a] <= v (the first vertex has slope 0), slope[b] beyond
    while (b - a > 1) {
        const int m = (a + b) >> 1;
        const bool ok = r.slope[m] <= v;
        a = ok ? m : a;
        b = ok ? b : m;
    }
    return r.vertex[a];
}
__device__ __forceinline__ double relaxed_value(const Lds& s, const Relax& r, int i, double v) {
    const int k = relaxed_pick(r, i, v);
    return __builtin_fma(v, (double)s.bin[k], (double)s.size[k]);
}

// Sweep of the core layers.  Row j covers the cells [lo, hi] of core layer j (bins summed over the core
// layers so far).  The first NT threads take KMAX cells each, NT apart; the other wavefronts only join
// the barriers.  What bounds it is the number of instructions issued per layer: 7 cycles each for a
// wavefront that has a SIMD to itself, 4 each in turn for wavefronts that share one, with two LDS round
// trips and a barrier beside them.  So:
//   * a row lies between cells of infinity as wide as any entry's shift reaches, and an entry's address
//     is worked out once for all cells of a thread (with every shifted read clamped into the row, a compare
//     and two selects per entry and a byte stored per cell, 10000 cells took 4.2 us a layer; now 1.2);
//   * PACK: the position among the survivors rides in the low `bits` bits of the costs (the caller has
//     checked that they stay below 2^30), so a minimum of two entries is one instruction;
//   * rows of up to 1024 cells go to 256 or 512 threads (512 x 2 cells: 0.26 us a layer of 4 entries; 256 x 4
//     0.28, 1024 x 1 0.29), wider ones to all 1024, where 4 wavefronts share a SIMD;
//   * nothing but the row is waited for: records and survivors are fetched ahead.
// TWO: two row buffers and one barrier per layer, else one buffer and two barriers.
// Arg-mins (position among the survivors): bytes, rows back to back; WORDS: a 32-bit word per layer and
// thread, `bits` bits per cell.
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ uint32_t lds_address(const uint32_t* p) { return (uint32_t)(size_t)(const lds_u32*)p; }
__device__ __forceinline__ uint32_t lds_load(uint32_t byte) { return *(const lds_u32*)(size_t)byte; }
__device__ __forceinline__ uint32_t lds_byte(uint32_t byte) {
    return *(const __attribute__((address_space(3))) uint8_t*)(size_t)byte;
}
__device__ __forceinline__ void lds_store(uint32_t byte, uint32_t v) { *(lds_u32*)(size_t)byte = v; }
__device__ __forceinline__ void lds_store_byte(uint32_t byte, uint32_t v) {
    *(__attribute__((address_space(3))) uint8_t*)(size_t)byte = (uint8_t)v;
}
constexpr uint32_t kInfPacked = 1u << 30;
struct Sweep {
    const Core* core;
    const uint2* ent;
    uint32_t* buffer;                        // front cells of infinity, the row, infinity up to `cells` (twice)
    uint8_t* pd;
    int front, cells, n_core, bits;
};
template <int NT, int KMAX, bool TWO, bool PACK, bool WORDS, bool LDS_PD>
__device__ __forceinline__ const uint32_t* sweep(const Sweep& p) {
    static_assert(!WORDS || (PACK && !LDS_PD), "words go to device memory");
    constexpr uint32_t kInf = PACK ? kInfPacked : kInfS;
    const int tid = threadIdx.x, n_core = p.n_core, bits = p.bits;
    const uint32_t places = (1u << bits) - 1u;
    for (int i = tid; i < (TWO ? 2 : 1) * p.cells; i += kThreadsS)
        p.buffer[i] = i == p.front ? 0u : kInf;          // the row in front of the first layer is the single cell 0
    uint32_t* const row0 = p.buffer + p.front;
    uint32_t* const row1 = TWO ? row0 + p.cells : row0;
    if (NT < kThreadsS && tid >= NT) {                   // (whole wavefronts)
        __syncthreads();
        for (int j = 0; j < n_core; ++j) {
            if (!TWO) __syncthreads();
            __syncthreads();
        }
        return n_core & 1 ? row1 : row0;
    }
    uint32_t cur = lds_address(row0) + 4u * (uint32_t)tid, nxt = lds_address(row1) + 4u * (uint32_t)tid;
    const uint32_t* shape_at = &p.core[0].shape;
    uint32_t shape1 = *shape_at;
    const uint4* list = reinterpret_cast<const uint4*>(p.ent);       // two entries each
    uint4 e1 = list[0], f1 = list[1];
    uint8_t* out = p.pd + (WORDS ? 4 : 1) * tid;
    uint32_t out_lds = LDS_PD ? lds_address(reinterpret_cast<const uint32_t*>(p.pd)) + (uint32_t)tid : 0u;
    __syncthreads();
    for (int j = 0; j < n_core; ++j) {
        const uint32_t shape = (uint32_t)__builtin_amdgcn_readfirstlane((int)shape1);
        const int nw = (int)(shape & 0xFFFFu), n = (int)(shape >> 16);
        const uint4 e0 = e1, f0 = f1;
        uint32_t nv[KMAX], na[KMAX];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) { nv[k] = kInf; na[k] = 255u; }
        // two entries at a time (a list is filled up with entries that never win)
        auto relax = [&](const uint4 e, int c) __attribute__((always_inline)) {
            const uint32_t x[2] = {e.x, e.z}, z[2] = {e.y, e.w};
            uint32_t t[2][KMAX];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t f = cur + x[u];
#pragma unroll
                for (int k = 0; k < KMAX; ++k) t[u][k] = lds_load(f + 4 * k * NT);
            }
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                if (PACK) {
                    nv[k] = min(nv[k], min(t[0][k] + z[0], t[1][k] + z[1]));
                } else {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const uint32_t v = t[u][k] + z[u];
                        const bool lt = v < nv[k];
                        nv[k] = lt ? v : nv[k];
                        na[k] = lt ? (uint32_t)(c + u) : na[k];
                    }
                }
            }
        };
        relax(e0, 0);
        if (n > 2) relax(f0, 2);
        for (int c = 4; c < n; c += 2) relax(list[c >> 1], c);
        list += ((n + 3) & ~3) >> 1;
        shape_at += sizeof(Core) / sizeof(uint32_t);     // (past the last record: the first entries)
        shape1 = *shape_at;
        e1 = list[0];
        f1 = list[1];
        if (!TWO) __syncthreads();
        uint32_t word = 0;
        // Cells behind the row (sums of bins above the interval) are not stopped from taking part: what they
        // hold are totals of assignments all the same, and none of the smallest size has such a sum.
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            lds_store(nxt + 4 * k * NT, PACK ? nv[k] & ~places : nv[k]);
            const uint32_t place = PACK ? nv[k] : na[k];  // (bytes: the reader takes the low bits)
            if (WORDS) word |= (place & places) << (bits * k);
            else if (LDS_PD) lds_store_byte(out_lds + k * NT, place);      // (behind the row: overwritten by the next one's, or slack)
            else if (tid + k * NT < nw) out[k * NT] = (uint8_t)place;
        }
        if (WORDS) *reinterpret_cast<uint32_t*>(out) = word;
        __syncthreads();
        if (TWO) { const uint32_t x = cur; cur = nxt; nxt = x; }
        out += WORDS ? 4 * NT : nw;
        out_lds += (uint32_t)nw;
    }
    return n_core & 1 ? row1 : row0;
}

// Where survivors, rows and margins do not fit LDS together (tables whose candidates all stay and whose bins reach
// far) and the caller has no other solver (SolveParams::last_resort): layer records and one row, no wider than the
// widest interval, with a cell of infinity on either side into which every shifted read is clamped.  The
// candidates are taken from the lists (Lds) and their bits of `keep`: lane k of every wavefront holds the k-th of a
// layer in candidate order, so that a list has at most 64.  Arg-mins: candidates.  K cells per thread.
// cand_bits: the candidate rides in that many low bits of the costs (0: beside them).  Bound by the instructions
// issued, per entry and cell an address, its clamp, a read, a sum and a minimum (or a compare and two selects):
// 628 layers of 6 candidates, 6656 bins: 1.8 ms; 256 of 16, 16380 bins: 2.7 ms.  Callers that do have another solver
// take it: on 60 layers of 40 candidates, 10000 bins, the layer groups of dp.hip take 0.87 ms with this kernel's
// attempt in front, a clamped sweep 2.1.
__device__ __forceinline__ int clamp_i32(int v, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(lo), "v"(hi));
    return r;
}
template <int K, bool PACK>
__device__ __forceinline__ const uint32_t* sweep_lists(const Lds& s, const Core* core, uint32_t* buffer, uint8_t* pd, int n_core,
                                                       int cand_bits) {
    const uint32_t cands = (1u << cand_bits) - 1u;
    constexpr int NT = kThreadsS;
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t* const cur = buffer + 1;
    static_assert(kInfS == kInfPacked, "one infinity");
    if (tid == 0) { cur[-1] = kInfS; cur[0] = 0; cur[1] = kInfS; }
    uint8_t* out = pd + tid;
    const int row_at = __builtin_amdgcn_readfirstlane((int)lds_address(cur));
    int w_front = 1, lo_front = 0;
    __syncthreads();
    for (int j = 0; j < n_core; ++j) {
        const int nw = __builtin_amdgcn_readfirstlane((int)(core[j].shape & 0xFFFFu));
        const int lo = __builtin_amdgcn_readfirstlane(core[j].lo), i = s.lo[j];
        const int first = __builtin_amdgcn_readfirstlane(s.off[i]), count = __builtin_amdgcn_readfirstlane(s.off[i + 1]) - first;
        // this lane's entry of the list, then the one whose rank among the layer's candidates it is
        const int at = first + min(lane, count - 1);
        const bool kept = lane < count && ((s.keep[at >> 6] >> (at & 63)) & 1);
        const unsigned long long m = __ballot(kept);
        const int cand = s.cand[at];
        int rank = 0;
        for (unsigned long long w = m; w; w &= w - 1) rank += (int)lane_u32((uint32_t)cand, (int)__builtin_ctzll(w)) < cand ? 1 : 0;
        const int n = (int)__popcll(m), to = 4 * (kept ? rank : 63);           // (with 64 kept nobody is sent to 63 beside its owner)
        const uint32_t bin_cand = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)((uint32_t)s.bin[at] << 8 | (uint32_t)cand));
        const uint32_t size = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(PACK ? s.size[at] << cand_bits | (uint32_t)cand : s.size[at]));
        const int behind = row_at + 4 * w_front, from = row_at + 4 * (tid + lo - lo_front);
        uint32_t nv[K], na[K];
#pragma unroll
        for (int k = 0; k < K; ++k) { nv[k] = kInfS; na[k] = 255u; }
        for (int c = 0; c < n; ++c) {
            const uint32_t bc = lane_u32(bin_cand, c), z = lane_u32(size, c), cd = bc & 255u;
            const int f = from - 4 * (int)(bc >> 8);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t v = lds_load((uint32_t)clamp_i32(f + 4 * k * NT, row_at - 4, behind)) + z;
                if (PACK) {
                    nv[k] = min(nv[k], v);
                } else {
                    const bool lt = v < nv[k];
                    nv[k] = lt ? v : nv[k];
                    na[k] = lt ? cd : na[k];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int t = tid + k * NT;
            if (t <= nw) cur[t] = t < nw ? (PACK ? nv[k] & ~cands : nv[k]) : kInfS;
            if (t < nw) out[k * NT] = (uint8_t)(PACK ? nv[k] & cands : na[k]);
        }
        __syncthreads();
        out += nw;
        w_front = nw;
        lo_front = lo;
    }
    return cur;
}

// Threads and cells a thread for rows of up to w_max cells.
struct SweepShape {
    int threads, per;
    bool two;
};
__device__ __forceinline__ SweepShape sweep_shape(int w_max) {
    if (w_max <= 1024) return w_max <= 256 ? SweepShape{256, 1, true} : SweepShape{512, w_max <= 512 ? 1 : 2, true};
    const int k = (w_max + kThreadsS - 1) / kThreadsS;
    return SweepShape{kThreadsS, k <= 2 ? 2 : k <= 4 ? 4 : k <= 6 ? 6 : k <= 8 ? 8 : k <= 10 ? 10 : k <= 13 ? 13 : 17, false};
}
template <bool PACK, bool WORDS, bool LDS_PD>
__device__ __forceinline__ const uint32_t* sweep_shaped(SweepShape f, const Sweep& p) {
    if constexpr (!WORDS) {
        if (f.threads == 256) return sweep<256, 1, true, PACK, WORDS, LDS_PD>(p);
        if (f.threads == 512) {
            if (f.per == 1) return sweep<512, 1, true, PACK, WORDS, LDS_PD>(p);
            return sweep<512, 2, true, PACK, WORDS, LDS_PD>(p);
        }
    }
    switch (f.per) {
        case 2: return sweep<1024, 2, false, PACK, WORDS, LDS_PD>(p);
        case 4: return sweep<1024, 4, false, PACK, WORDS, LDS_PD>(p);
        case 6: return sweep<1024, 6, false, PACK, WORDS, LDS_PD>(p);
        case 8: return sweep<1024, 8, false, PACK, WORDS, LDS_PD>(p);
        case 10: return sweep<1024, 10, false, PACK, WORDS, LDS_PD>(p);
        case 13: return sweep<1024, 13, false, PACK, WORDS, LDS_PD>(p);
        default: return sweep<1024, 17, false, PACK, WORDS, LDS_PD>(p);
    }
}

// NE: table entries per thread (L x P <= NE x 1024).  LAST: with the last resort (SolveParams::last_resort).  It is left out
// where a caller has another solver: in one kernel with the rest its code cost a solve 0.2 to 1.9 us.
template <int NE, bool LAST>
__global__ __launch_bounds__(kThreadsS) void solve_kernel(SolveParams p) {
    extern __shared__ __align__(16) unsigned char solve_smem[];
    Lds& s = *reinterpret_cast<Lds*>(solve_smem);
    unsigned char* const region = solve_smem + sizeof(Lds);
    uint16_t* const t_bin = reinterpret_cast<uint16_t*>(region + sizeof(uint32_t) * NE * kThreadsS);
    uint32_t* const t_size = reinterpret_cast<uint32_t*>(region);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = p.L, P = p.P, LP = L * P;
    const int D = min(p.D, p.e_limit);                   // bins an assignment may use
    const uint64_t t_begin = wall_clock64();

    // ---- the table: errors in registers (and on to the host's copy), sizes to LDS
    double err[NE];
    if (tid == 0) {
        s.flags = 0;
        s.chk_err = 0;
        s.chk_choice = 0;
        s.worst = 0;
        s.best = ~0ull;
        s.sums = 0;
        s.ub = kInfS;
    }
    if (tid < 4) s.acc[tid] = s.facts[tid] = 0;
    bool bad = false;
    unsigned long long chk = 0;
    int64_t sz[NE];
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int i = tid + q * kThreadsS;
        err[q] = i < LP ? p.errors[i] : 0.0;
        sz[q] = i < LP ? p.sizes[i] : 0;
    }
    if (tid < L) s.def[tid] = p.have_e_max ? 0.0 : p.errors[(size_t)tid * P + p.default_cand];
    // (the table of the order is allocated in whole 16-byte words)
    if (p.order && 16 * tid < LP) reinterpret_cast<uint4*>(s.order)[tid] = reinterpret_cast<const uint4*>(p.order)[tid];
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int i = tid + q * kThreadsS;
        if (i < LP) {
            if (p.errors_host) p.errors_host[i] = err[q];
            chk += __builtin_bit_cast(unsigned long long, err[q]) * (unsigned long long)(i + 1);
            bad |= !(err[q] == err[q]);
            bad |= p.check_sizes && (sz[q] < 0 || sz[q] >= (int64_t)kInfS);
            t_size[i] = (uint32_t)sz[q];
        }
    }
    __syncthreads();
    // E_max: summed in layer order by one thread (bit-identical to the host's loop), LDS reads in
    // batches ahead of the dependent adds; the other wavefronts add up the check word meanwhile
    if (tid == 0) {
        double sum = p.e_max;
        if (!p.have_e_max) {
            sum = 0.0;
            int l = 0;
            for (; l + 32 <= L; l += 32) {
                double v[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) v[u] = s.def[l + u];
#pragma unroll
                for (int u = 0; u < 32; ++u) sum += v[u];
            }
            for (; l < L; ++l) sum += s.def[l];
        }
        s.emax = sum;
        if (!(sum == sum)) bad = true;
    }
    if (p.errors_host) {
        chk = wave_total(chk);
        if (lane == 0) atomicAdd(&s.chk_err, chk);
    }
    if (p.check_sizes) {                                 // a caller whose table the host has not seen
        uint32_t big = 0;
        if (tid < L)
            for (int c = 0; c < P; ++c) big = max(big, t_size[tid * P + c]);
        const double part = wave_total((double)big);     // whole numbers below 2^42: exact
        if (lane == 0) atomicAdd(&s.worst, (unsigned long long)part);
        __syncthreads();
        bad |= s.worst >= (unsigned long long)kInfS;
    }
    if (bad) atomicOr(&s.flags, 2);
    __syncthreads();

    // ---- bins
    const double e_max = s.emax, Dd = (double)p.D;
#pragma unroll
    for (int q = 0; q < NE; ++q) {
        const int i = tid + q * kThreadsS;
        if (q * kThreadsS < LP && i < LP) {
            double e = err[q];
            if (e < 0.0) e = 0.0;
            uint32_t b = kUnusable;
            if (e_max > 0.0) {
                const double f = floor((e * Dd) / e_max);
                if (f <= Dd) b = (uint32_t)f;
            } else if (e <= 0.0) {
                b = 0;
            }
            if ((int)b > D) b = kUnusable;               // (fits no assignment under a tighter budget)
            t_bin[i] = (uint16_t)b;
        }
    }
    __syncthreads();
    // ---- candidates in order of size (lowest index first among equals): the caller's table, or sorted here
    if (!p.order) {
        for (int i = tid; i < LP; i += kThreadsS) {
            const int l = i / P, head = l * P;
            const uint32_t z = t_size[i];
            int rank = 0;
            for (int o = head; o < head + P; ++o) rank += t_size[o] < z || (t_size[o] == z && o < i) ? 1 : 0;
            s.order[head + rank] = (uint8_t)(i - head);
        }
        __syncthreads();
    }
    // ---- candidates worth keeping: not those another one of the layer beats in bin and size (equal
    // bins: the smallest size stays, the lowest index among equals).  In order of size a candidate
    // stays if its bin lies below all bins in front of it, and if the next one that does so has a
    // larger size.  A group of 16 lanes (P <= 16) or a wavefront (two candidates a lane) takes a
    // layer.
    auto slot_of = [&](int l, int rank) -> int {         // table position of the candidate at this rank
        return l * P + (int)s.order[l * P + rank];
    };
    const int words = P > 64 ? 2 : 1;                    // (P > 64: at most 252 layers)
    if (P <= 16) {
        for (int l0 = 4 * wave; l0 < L; l0 += 4 * kWavesS) {
            const int l = l0 + (lane >> 4), rank = lane & 15;
            const bool in = l < L && rank < P;
            const int i = in ? slot_of(l, rank) : 0;
            const uint32_t b = in ? t_bin[i] : kUnusable, z = in ? t_size[i] : 0u;
            // smallest bin in front, inside the row of 16 lanes
            uint32_t m = min16<0x111>(b);
            m = min(m, min16<0x111>(m));
            m = min(m, min16<0x112>(m));
            m = min(m, min16<0x114>(m));
            m = min(m, min16<0x118>(m));
            const bool k0 = b < min(m, kUnusable);
            const uint32_t row = (uint32_t)(__ballot(k0) >> (lane & 48)) & 0xFFFFu;
            const uint32_t up = row >> (rank + 1);
            const uint32_t zn = (uint32_t)__shfl((int)z, up ? lane + 1 + (int)__builtin_ctz(up) : lane, 64);
            const bool k = k0 && !(up && zn == z);
            const unsigned long long kept = __ballot(k), moved = __ballot(in && i != l * P + rank);
            if (rank == 0 && l < L) {
                s.list[l] = (kept >> (lane & 48)) & 0xFFFFull;
                s.mixed[l] = ((moved >> (lane & 48)) & 0xFFFFull) ? 1 : 0;
            }
        }
    } else {
        for (int l = wave; l < L; l += kWavesS) {
            if (words == 1) {
                const bool in = lane < P;
                const int i = in ? slot_of(l, lane) : 0;
                const uint32_t b = in ? t_bin[i] : kUnusable, z = in ? t_size[i] : 0u;
                const bool k = b < min(wave_min_before(b), kUnusable);
                const unsigned long long low = __ballot(k);
                const uint64_t up = lane < 63 ? low >> (lane + 1) : 0ull;
                const uint32_t zn = (uint32_t)__shfl((int)z, up ? lane + 1 + (int)__builtin_ctzll(up) : lane, 64);
                const unsigned long long kept = __ballot(k && !(up && zn == z)), moved = __ballot(in && i != l * P + lane);
                if (lane == 0) {
                    s.list[l] = kept;
                    s.mixed[l] = moved ? 1 : 0;
                }
                continue;
            }
            const bool in0 = lane < P, in1 = 64 + lane < P;
            const int i0 = in0 ? slot_of(l, lane) : 0, i1 = in1 ? slot_of(l, 64 + lane) : 0;
            const uint32_t b0 = in0 ? t_bin[i0] : kUnusable, b1 = in1 ? t_bin[i1] : kUnusable;
            const uint32_t z0 = in0 ? t_size[i0] : 0u, z1 = in1 ? t_size[i1] : 0u;
            const uint32_t m0 = wave_min_before(b0);
            const uint32_t first = min(lane_u32(m0, 63), lane_u32(b0, 63));      // smallest of the first 64
            const uint32_t m1 = min(wave_min_before(b1), first);
            const unsigned long long k0 = __ballot(b0 < min(m0, kUnusable)), k1 = __ballot(b1 < min(m1, kUnusable));
            const uint64_t up0 = lane < 63 ? k0 >> (lane + 1) : 0ull, up1 = lane < 63 ? k1 >> (lane + 1) : 0ull;
            const uint32_t head1 = k1 ? lane_u32(z1, (int)__builtin_ctzll(k1)) : 0u;
            const uint32_t n0 = (uint32_t)__shfl((int)z0, up0 ? lane + 1 + (int)__builtin_ctzll(up0) : lane, 64);
            const uint32_t n1 = (uint32_t)__shfl((int)z1, up1 ? lane + 1 + (int)__builtin_ctzll(up1) : lane, 64);
            const bool beaten0 = up0 ? n0 == z0 : (k1 && head1 == z0);
            const bool beaten1 = up1 && n1 == z1;
            const unsigned long long kept0 = __ballot(((k0 >> lane) & 1) && !beaten0);
            const unsigned long long kept1 = __ballot(((k1 >> lane) & 1) && !beaten1);
            const unsigned long long moved = __ballot((in0 && i0 != l * P + lane) || (in1 && i1 != l * P + 64 + lane));
            if (lane == 0) {
                s.list[2 * l] = kept0;
                s.list[2 * l + 1] = kept1;
                s.mixed[l] = moved ? 1 : 0;
            }
        }
    }
    __syncthreads();
    // ---- the layers left to sweep and their entries
    uint32_t cnt = 0, first_cand = 255;
    if (tid < L) {
        const uint64_t b0 = s.list[words * tid], b1 = words == 2 ? s.list[2 * tid + 1] : 0ull;
        cnt = (uint32_t)(__popcll(b0) + __popcll(b1));
        if (cnt) first_cand = (uint32_t)(slot_of(tid, b0 ? (int)__builtin_ctzll(b0) : 64 + (int)__builtin_ctzll(b1)) - tid * P);
        else atomicOr(&s.flags, 1);
    }
    const bool fixed = tid < L && cnt == 1 && t_bin[tid * P + first_cand] == 0;
    const bool swept = tid < L && cnt > 0 && !fixed;
    uint32_t both;
    const uint32_t before = block_scan(swept ? (1u << 20) + cnt : 0u, s.tmp, &both);   // (both sums fit their halves)
    const uint32_t slot = before >> 20, off = before & 0xFFFFFu;
    const int n = (int)(both >> 20), T = (int)(both & 0xFFFFFu);
    if (tid < L) {
        s.chosen[tid] = fixed ? (uint8_t)first_cand : (uint8_t)255;
    }
    if (swept) {
        s.layer[slot] = (uint16_t)tid;
        s.off[slot] = (int32_t)off;
    }
    if (tid == 0) s.off[n] = T;
    int status = 0;
    const int flags = s.flags;                           // (the scans' barriers stand in front)
    if (flags & 2) status = 3;
    else if ((flags & 1) || D < 0) status = 1;
    else if (T > kMaxT) status = 4;                      // more entries than LDS holds: not taken here
    if (tid < L) s.first[tid] = swept && status == 0 ? (int32_t)(off | (slot << 16)) : -1;      // (off: at most T <= 4096)
    __syncthreads();
    // entries in order of size, that is largest bin first
    if (status == 0) {
        auto put = [&](int l, int rank, uint32_t f, uint32_t place) __attribute__((always_inline)) {
            const int i = slot_of(l, rank);
            const uint32_t at = (f & 0xFFFFu) + place;
            s.bin[at] = t_bin[i];
            s.cand[at] = (uint8_t)(i - l * P);
            s.of[at] = (uint16_t)(f >> 16);
        };
        if (P <= 16) {
            for (int l0 = 4 * wave; l0 < L; l0 += 4 * kWavesS) {
                const int l = l0 + (lane >> 4), rank = lane & 15;
                if (l >= L || s.first[l] < 0) continue;
                const uint32_t m = (uint32_t)s.list[l];
                if ((m >> rank) & 1) put(l, rank, (uint32_t)s.first[l], (uint32_t)__popc(m & ((1u << rank) - 1)));
            }
        } else {
            for (int l = wave; l < L; l += kWavesS) {
                if (s.first[l] < 0) continue;            // uniform
                const uint64_t m0 = s.list[words * l], m1 = words == 2 ? s.list[2 * l + 1] : 0ull, below = (1ull << lane) - 1;
                const uint32_t f = (uint32_t)s.first[l];
                if ((m0 >> lane) & 1) put(l, lane, f, (uint32_t)__popcll(m0 & below));
                if ((m1 >> lane) & 1) put(l, 64 + lane, f, (uint32_t)(__popcll(m0) + __popcll(m1 & below)));
            }
        }
    }
    __syncthreads();
    if (status == 0) {                                   // the sizes take the place of the order
#pragma unroll
        for (int q = 0; q < kMaxT / kThreadsS; ++q) {
            const int t = tid + q * kThreadsS;
            if (q * kThreadsS < T && t < T) s.size[t] = t_size[(int)s.layer[s.of[t]] * P + (int)s.cand[t]];
        }
    }
    __syncthreads();                                     // from here on the table's region is free

    uint64_t t_sweep = t_begin;
    int64_t total_bins = 0, total_size = 0;              // of the swept layers
    if (status == 0 && n > 0) {
        // ---- the cells and candidates that matter.  The full sweep of a small table costs less than
        // finding them: about 0.15 us a layer and 0.02 us an entry and 1024 cells, against some 10 us.
        const int rows_full = (D + kThreadsS) / kThreadsS;          // cells of a full row per thread
        const bool reduce = n > 1 && (n * 8 + T * rows_full > 500 || D >= kRowCells);
        Relax& r = *reinterpret_cast<Relax*>(region);
        double v_star = 0.0, ub_star = 0.0;
        if (reduce) {
            // ---- lower convex hull of every layer's (bin, size) points.  A point on or above the line
            // between its neighbours goes (compared exactly, as products of differences below 2^45)
            // until none does: two or three rounds on lists that are nearly convex.  A group of 16
            // lanes or a wavefront takes a layer; neighbours come from the bits of those left.
            for (int w = tid; w < kMaxT / 64; w += kThreadsS) s.keep[w] = 0;
            __syncthreads();
            auto above = [&](uint32_t bp, uint32_t sp, uint32_t b, uint32_t z, uint32_t bn, uint32_t sn) -> bool {
                // previous point: larger bin, smaller size; next: smaller bin, larger size
                const double d1b = (double)(int)(bp - b), d1s = (double)(int)(z - sp);
                const double d2b = (double)(int)(b - bn), d2s = (double)(int)(sn - z);
                return d2s * d1b <= d1s * d2b;           // the way down is no steeper than the way on
            };
            if (P <= 16) {
                for (int i0 = 4 * wave; i0 < n; i0 += 4 * kWavesS) {
                    const int i = i0 + (lane >> 4), rank = lane & 15, row = lane & 48;
                    const int first = i < n ? s.off[i] : 0, c_n = i < n ? s.off[i + 1] - first : 0;
                    const uint32_t b = rank < c_n ? s.bin[first + rank] : 0u, z = rank < c_n ? s.size[first + rank] : 0u;
                    uint32_t m = (1u << c_n) - 1u;
                    for (;;) {
                        const uint32_t lo = m & ((1u << rank) - 1u), hi = m >> (rank + 1);
                        const int pr = row + (lo ? 31 - (int)__builtin_clz(lo) : rank);
                        const int nx = row + (hi ? rank + 1 + (int)__builtin_ctz(hi) : rank);
                        const uint32_t bp = (uint32_t)__shfl((int)b, pr, 64), sp = (uint32_t)__shfl((int)z, pr, 64);
                        const uint32_t bn = (uint32_t)__shfl((int)b, nx, 64), sn = (uint32_t)__shfl((int)z, nx, 64);
                        const bool gone = ((m >> rank) & 1) && lo && hi && above(bp, sp, b, z, bn, sn);
                        const unsigned long long g = __ballot(gone);
                        if (!g) break;
                        m &= ~(uint32_t)(g >> row);
                    }
                    if (rank == 0 && c_n > 0) {
                        const int sh = first & 63;
                        atomicOr((unsigned long long*)&s.keep[first >> 6], (unsigned long long)m << sh);
                        if (sh + c_n > 64) atomicOr((unsigned long long*)&s.keep[(first >> 6) + 1], (unsigned long long)m >> (64 - sh));
                    }
                }
            } else {
                for (int i = wave; i < n; i += kWavesS) {
                    const int first = s.off[i], c_n = s.off[i + 1] - first;
                    unsigned long long m = 0, m_next = 0;
                    const bool two = c_n > 64;
                    const uint32_t b = lane < c_n ? s.bin[first + lane] : 0u, z = lane < c_n ? s.size[first + lane] : 0u;
                    m = c_n >= 64 ? ~0ull : (1ull << c_n) - 1ull;
                    uint32_t b2 = 0, z2 = 0;
                    if (two) {
                        b2 = 64 + lane < c_n ? s.bin[first + 64 + lane] : 0u;
                        z2 = 64 + lane < c_n ? s.size[first + 64 + lane] : 0u;
                        m_next = c_n >= 128 ? ~0ull : (1ull << (c_n - 64)) - 1ull;
                    }
                    for (;;) {
                        const unsigned long long below = (1ull << lane) - 1ull;
                        const unsigned long long lo = m & below, hi = lane < 63 ? m >> (lane + 1) : 0ull;
                        const int pr = lo ? 63 - (int)__builtin_clzll(lo) : lane;
                        const int nx = hi ? lane + 1 + (int)__builtin_ctzll(hi) : lane;
                        const uint32_t bp = (uint32_t)__shfl((int)b, pr, 64), sp = (uint32_t)__shfl((int)z, pr, 64);
                        uint32_t bn = (uint32_t)__shfl((int)b, nx, 64), sn = (uint32_t)__shfl((int)z, nx, 64);
                        bool has_next = hi != 0;
                        if (two && !has_next && m_next) {
                            const int f = (int)__builtin_ctzll(m_next);
                            bn = lane_u32(b2, f);
                            sn = lane_u32(z2, f);
                            has_next = true;
                        }
                        const bool gone = ((m >> lane) & 1) && lo && has_next && above(bp, sp, b, z, bn, sn);
                        unsigned long long g = __ballot(gone), g2 = 0;
                        if (two) {
                            const unsigned long long lo2 = m_next & below, hi2 = lane < 63 ? m_next >> (lane + 1) : 0ull;
                            const int pr2 = lo2 ? 63 - (int)__builtin_clzll(lo2) : lane;
                            const int nx2 = hi2 ? lane + 1 + (int)__builtin_ctzll(hi2) : lane;
                            uint32_t bq = (uint32_t)__shfl((int)b2, pr2, 64), sq = (uint32_t)__shfl((int)z2, pr2, 64);
                            const uint32_t bm = (uint32_t)__shfl((int)b2, nx2, 64), sm = (uint32_t)__shfl((int)z2, nx2, 64);
                            if (!lo2) {                   // its neighbour is the last one left of the first 64 (entry 0 always is)
                                const int f = 63 - (int)__builtin_clzll(m);
                                bq = lane_u32(b, f);
                                sq = lane_u32(z, f);
                            }
                            g2 = __ballot(((m_next >> lane) & 1) && hi2 && above(bq, sq, b2, z2, bm, sm));
                        }
                        if (!(g | g2)) break;
                        m &= ~g;
                        m_next &= ~g2;
                    }
                    if (lane < 2) {
                        const unsigned long long mm = lane ? m_next : m;
                        const int at = first + 64 * lane, sh = at & 63;
                        if (mm) {
                            atomicOr((unsigned long long*)&s.keep[at >> 6], mm << sh);
                            if (sh && (mm >> (64 - sh))) atomicOr((unsigned long long*)&s.keep[(at >> 6) + 1], mm >> (64 - sh));
                        }
                    }
                }
            }
            r.hist[tid] = 0;
            __syncthreads();
            if (wave == 0) count_bits(s, (T + 63) & ~63);
            __syncthreads();
            // the vertices side by side, each with its slope towards the vertex in front of it (none: 0)
            {
                uint32_t bins_down = 0;
#pragma unroll
                for (int q = 0; q < kMaxT / kThreadsS; ++q) {
                    const int t = tid + q * kThreadsS;
                    if (q * kThreadsS < T && t < T && ((s.keep[t >> 6] >> (t & 63)) & 1)) {
                        const int head = s.off[s.of[t]];
                        double slope = 0.0;
                        if (t > head) {
                            int w = t >> 6;
                            uint64_t m = s.keep[w] & ((1ull << (t & 63)) - 1ull);
                            while (!m) m = s.keep[--w];                       // ends: the list's first entry is a vertex
                            const int f = 64 * w + 63 - (int)__builtin_clzll(m);
                            slope = ((double)s.size[t] - (double)s.size[f]) / ((double)s.bin[f] - (double)s.bin[t]);
                        }
                        const uint32_t at = bits_before(s, t);
                        r.slope[at] = slope;
                        r.vertex[at] = (uint16_t)t;
                    }
                }
                if (tid < n) {
                    r.hoff[tid] = (uint16_t)bits_before(s, s.off[tid]);
                    bins_down = s.bin[s.off[tid + 1] - 1];           // the layer's smallest bin
                }
                uint32_t all;
                const uint32_t nh = s.before[(T - 1) >> 6] + (uint32_t)__popcll(s.keep[(T - 1) >> 6]);
                if (tid == 0) r.hoff[n] = (uint16_t)nh;
                (void)block_scan(bins_down, s.tmp, &all);
                if (tid == 0) s.acc[0] = all;
            }
            __syncthreads();
            const uint32_t bins_min = s.acc[0];
            if (bins_min > (uint32_t)D) status = 1;      // not even the smallest bins fit
            const int nh = r.hoff[n];
            // ---- v*: the multiplier at which the relaxed bins come down to the budget.  Starting from the
            // smallest bins, an edge of the hull is taken where its slope exceeds v: bins per slope
            // in a histogram over the slope's pattern (5 bits of mantissa, then 10 more inside the
            // bucket where the sum from above passes the room)
            if (status == 0) {
                uint32_t room = (uint32_t)D - bins_min, bucket = 0;
                for (int round = 0; round < 2; ++round) {
                    if (round) {
                        r.hist[tid] = 0;
                        __syncthreads();
                    }
#pragma unroll
                    for (int q = 0; q < kMaxT / kThreadsS; ++q) {
                        const int h = tid + q * kThreadsS;
                        if (q * kThreadsS < nh && h < nh && r.slope[h] > 0.0) {
                            const uint32_t bits = __float_as_uint((float)r.slope[h]);
                            const int k1 = max(0, min(1023, (int)(bits >> 18) - (126 << 5)));
                            const uint32_t db = (uint32_t)s.bin[r.vertex[h - 1]] - (uint32_t)s.bin[r.vertex[h]];
                            if (round == 0) atomicAdd(&r.hist[k1], db);
                            else if ((uint32_t)k1 == bucket) atomicAdd(&r.hist[(bits >> 8) & 1023u], db);
                        }
                    }
                    __syncthreads();
                    const uint32_t own = r.hist[1023 - tid];
                    uint32_t all;
                    const uint32_t above = block_scan(own, s.tmp, &all);       // bins of the steeper buckets
                    if (tid == 0) s.acc[1] = 0;
                    __syncthreads();
                    if (above <= room && above + own > room) {
                        s.acc[1] = 1024u - (uint32_t)tid;                      // bucket + 1
                        s.acc[2] = above;
                    }
                    __syncthreads();
                    if (s.acc[1] == 0) {                 // everything fits (first round): v* at the bottom
                        v_star = 1.0 / 1024.0;
                        break;
                    }
                    if (round == 0) {
                        bucket = s.acc[1] - 1;
                        room -= s.acc[2];
                        v_star = (double)__uint_as_float((bucket + (126u << 5) + 1) << 18);
                    } else {
                        v_star = (double)__uint_as_float(((bucket + (126u << 5)) << 18) + (s.acc[1] << 8));
                    }
                    __syncthreads();
                }
                // ---- UB: sixteen relaxed assignments from v* upwards (the last one at the smallest
                // bins), each with its four largest savings that still fit taken on top
                {
                    const double w = (double)wave;
                    const double v = wave == kWavesS - 1 ? 1e300 : v_star * (1.0 + 0.04 * w + 0.015 * w * w);
                    uint8_t* const pick = r.pick[wave];
                    uint32_t sb = 0, ss = 0;
                    for (int i = lane; i < n; i += 64) {
                        const int k = relaxed_pick(r, i, v);
                        pick[i] = (uint8_t)(k - s.off[i]);
                        sb += s.bin[k];
                        ss += s.size[k];
                    }
                    sb = wave_total(sb);
                    ss = wave_total(ss);
                    for (int it = 0; it < 4 && sb <= (uint32_t)D; ++it) {
                        const uint32_t room_w = (uint32_t)D - sb;
                        uint32_t gain = 0, cost = 0;
                        int gi = 0, gk = 0;
                        for (int i = lane; i < n; i += 64) {
                            // sizes fall as bins rise: the largest bin that fits saves most
                            const int b = s.off[i], k = b + pick[i];
                            const uint32_t limit = (uint32_t)s.bin[k] + room_w;
                            int x = b - 1, y = k;                              // bin[y] fits, bin[x] does not
                            while (y - x > 1) {
                                const int m = (x + y) >> 1;
                                const bool ok = s.bin[m] <= limit;
                                y = ok ? m : y;
                                x = ok ? x : m;
                            }
                            const uint32_t g = s.size[k] - s.size[y];
                            if (g > gain) {
                                gain = g;
                                cost = (uint32_t)s.bin[y] - (uint32_t)s.bin[k];
                                gi = i;
                                gk = y - b;
                            }
                        }
                        const uint32_t top = wave_max_u32(gain);
                        if (top == 0) break;
                        const int who = (int)__builtin_ctzll(__ballot(gain == top));
                        if (lane == who) pick[gi] = (uint8_t)gk;
                        sb += lane_u32(cost, who);
                        ss -= top;
                    }
                    if (lane == 0 && sb <= (uint32_t)D) atomicMin(&s.ub, ss);
                }
                // ---- intervals: one multiplier per wavefront, values around v* (v* itself for all layers first)
                {
                    const double m = tid < n ? relaxed_value(s, r, tid, v_star) : 0.0;
                    const double inc = wave_scan(m);
                    if (lane == 63) s.tmp_d[wave] = inc;
                    for (int i = tid; i <= n; i += kThreadsS) {
                        s.lo[i] = 0;
                        s.hi[i] = i == 0 ? 0 : D;
                    }
                    __syncthreads();
                    double front = 0.0, total = 0.0;
                    for (int w = 0; w < kWavesS; ++w) {
                        front += w < wave ? s.tmp_d[w] : 0.0;
                        total += s.tmp_d[w];
                    }
                    if (tid < n) {
                        r.star[tid] = m;
                        r.prefix[tid] = front + inc;
                    }
                    if (tid == 0) s.total_star = total;
                }
                double v = v_star;
                if (wave >= 1 && wave <= 12) {
                    const double d = 1.0 / (double)(2 << ((wave - 1) >> 1));        // 1/2 .. 1/64 either way
                    v *= (wave & 1) ? 1.0 + d : 1.0 - d;
                } else if (wave > 12) {
                    v *= wave == 13 ? 4.0 : wave == 14 ? 0.25 : 16.0;
                }
                double tot = 0.0, val[4] = {0.0, 0.0, 0.0, 0.0};        // (the first 256 layers' values are kept)
                if (wave > 0) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int i = lane + 64 * u;
                        if (64 * u < n && i < n) val[u] = relaxed_value(s, r, i, v);
                        tot += val[u];
                    }
                    for (int i = lane + 256; i < n; i += 64) tot += relaxed_value(s, r, i, v);
                }
                tot = wave_total(tot);
                __syncthreads();
                const double tot_star = s.total_star;
                // sizes are whole numbers: half a unit, and more where v D is so large that the fp64
                // sums of up to 1024 terms round by more, keeps every cell that is not strictly worse
                const double ub = (double)s.ub + 0.5 + 1e-12 * (v + v_star) * (double)D;
                ub_star = (double)s.ub + 0.5 + 2e-12 * v_star * (double)D;
                if (wave > 0) {
                    const double dv = v_star - v, inv = 1.0 / dv;
                    double carry = 0.0;
                    auto bound = [&](int i, double value) __attribute__((always_inline)) {
                        const double fv = wave_scan(value) + carry;
                        carry = lane_f64(fv, 63);
                        if (i < n) {
                            const double fs = r.prefix[i];
                            // layers up to i bounded with v, the rest with v*:  dv e <= a
                            const double a = (ub - fv - (tot_star - fs) + v_star * (double)D) * inv;
                            // layers up to i bounded with v*, the rest with v: -dv e <= b
                            const double b = -(ub - fs - (tot - fv) + v * (double)D) * inv;
                            const double up = fmin(fmax(floor(dv > 0.0 ? a : b), -1.0), (double)D);
                            const double dn = fmax(fmin(ceil(dv > 0.0 ? b : a), (double)D + 1.0), 0.0);
                            atomicMin(&s.hi[i + 1], (int)up);
                            atomicMax(&s.lo[i + 1], (int)dn);
                        }
                    };
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (64 * u < n) bound(lane + 64 * u, val[u]);
                    for (int i0 = 256; i0 < n; i0 += 64)
                        bound(i0 + lane, i0 + lane < n ? relaxed_value(s, r, i0 + lane, v) : 0.0);
                }
            }
        } else {
            for (int i = tid; i <= n; i += kThreadsS) {
                s.lo[i] = 0;
                s.hi[i] = i == 0 ? 0 : D;
            }
        }
        __syncthreads();
        // ---- candidates that can lie on an assignment of the smallest size
        if (status == 0) {
#pragma unroll
            for (int q = 0; q < kMaxT / kThreadsS; ++q) {
                const int t = tid + q * kThreadsS;
                if (q * kThreadsS >= T) continue;        // uniform
                bool k = t < T;
                if (k && reduce) {
                    const int i = s.of[t], bk = s.bin[t];
                    const double c = __builtin_fma(v_star, (double)bk, (double)s.size[t]);
                    k = c <= ub_star - (s.total_star - v_star * (double)D) + r.star[i] &&
                        s.lo[i] + bk <= s.hi[i + 1] && s.hi[i] + bk >= s.lo[i + 1];
                }
                const unsigned long long m = __ballot(k);
                if (lane == 0) s.keep[t >> 6] = m;
            }
            __syncthreads();
            if (wave == 0) count_bits(s, (T + 63) & ~63);
            if (tid == 0) s.acc[2] = 0;
            __syncthreads();
            // ---- layers with one candidate left shift the row: they are taken out of the sweep
            const bool on = tid < n;
            const int e0 = on ? s.off[tid] : 0, e1 = on ? s.off[tid + 1] : 0;
            int left = 0, only = e0;
            if (on) {
                uint32_t a = bits_before(s, e0);
                const uint32_t b = e1 < T ? bits_before(s, e1)
                                          : s.before[(T - 1) >> 6] + (uint32_t)__popcll(s.keep[(T - 1) >> 6]);
                left = (int)(b - a);
                if (left == 1) {
                    uint64_t w = s.keep[e0 >> 6] >> (e0 & 63);
                    while (!w) {                          // the one bit lies in a later word of the list
                        only = (only | 63) + 1;
                        w = s.keep[only >> 6];
                    }
                    only += (int)__builtin_ctzll(w);
                }
                if (left == 0) atomicOr(&s.flags, 4);
            }
            const bool single = on && left == 1, core = on && left > 1;
            uint32_t both_c, shift_all, cells, before_c, sh, unused, unused_total;
            block_scan2(core ? (1u << 20) + (((uint32_t)left + 3u) & ~3u) : 0u, single ? (uint32_t)s.bin[only] : 0u, s.tmp2[0],
                        &before_c, &sh, &both_c, &shift_all);
            const uint32_t j = before_c >> 20, ce = before_c & 0xFFFFFu, ents = both_c & 0xFFFFFu;
            {
                const uint32_t part = wave_total(single ? s.size[only] : 0u);
                if (lane == 0 && part) atomicAdd(&s.acc[2], part);
            }
            // cells of the core layer's row: bins summed over the core layers alone
            const int my_lo = on ? max(0, s.lo[tid + 1] - (int)sh) : 0, my_hi = on ? s.hi[tid + 1] - (int)sh : 0;
            const uint32_t w = core ? (uint32_t)max(my_hi - my_lo + 1, 0) : 0u;
            uint32_t cell0;
            block_scan2(w, 0u, s.tmp2[1], &cell0, &unused, &cells, &unused_total);
            const int n_core = (int)(both_c >> 20);
            {
                const uint32_t wm = wave_max_u32(w), lm = wave_max_u32(core ? (uint32_t)left : 0u);
                const uint32_t top = wave_total(core ? s.size[e1 - 1] : 0u);       // (a list's last entry is its largest)
                if (lane == 0 && wm) {
                    atomicMax(&s.acc[3], wm);
                    atomicMax(&s.facts[2], lm);
                    atomicAdd(&s.facts[3], top);
                }
                if (core && my_hi < my_lo) atomicOr(&s.flags, 8);
            }
            Core* const rec = reinterpret_cast<Core*>(region);
            uint2* const ent = reinterpret_cast<uint2*>(region + sizeof(Core) * (size_t)max(n_core, 1));
            uint8_t* const ent_cand = reinterpret_cast<uint8_t*>(ent + ents + 64);
            if (on) s.first[tid] = core ? (int32_t)(ce | (j << 16)) : -1;      // (under 2^13 survivors, padding included)
            if (core) {
                s.lo[j] = tid;                            // core layer -> swept layer (every interval has been read)
                s.hi[j] = (int32_t)ce;                    // ... and its first survivor
                rec[j] = Core{0, my_lo, w | ((uint32_t)left << 16), (int32_t)cell0};
            }
            __syncthreads();
            // positions ride in the costs' low bits where they fit
            int bits = 32 - __builtin_clz(max(s.facts[2], 2u) - 1);
            if (((unsigned long long)s.facts[3] << bits) >= kInfPacked) bits = 0;
            uint32_t down = 0, up = 0;                    // how far shifts reach
            if (tid < n_core) {
                const Core c = rec[tid];
                const int step = c.lo - (tid ? rec[tid - 1].lo : 0);
                rec[tid].step = step;
                // entries that never win fill the lists up
                for (int u = (int)(c.shape >> 16); u & 3; ++u) ent[s.hi[tid] + u] = make_uint2(0u, kInfPacked);
                if (tid == n_core - 1) {
                    s.acc[0] = (uint32_t)c.lo;            // the last row's first cell and width
                    s.acc[1] = c.shape & 0xFFFFu;
                }
            }
#pragma unroll
            for (int q = 0; q < kMaxT / kThreadsS; ++q) {
                const int t = tid + q * kThreadsS;
                if (q * kThreadsS < T && t < T && ((s.keep[t >> 6] >> (t & 63)) & 1)) {
                    const int i = s.of[t];
                    if (s.first[i] >= 0) {
                        uint32_t rank = 0;
                        if (s.mixed[s.layer[i]] == 0) {
                            rank = bits_before(s, t) - bits_before(s, s.off[i]);
                        } else {
                            const uint32_t cd = s.cand[t];
                            for (int k = s.off[i]; k < s.off[i + 1]; ++k)
                                rank += ((s.keep[k >> 6] >> (k & 63)) & 1) && s.cand[k] < cd ? 1u : 0u;
                        }
                        const int q0 = s.first[i] >> 16;
                        const Core c = rec[q0];
                        const int lo_front = q0 ? rec[q0 - 1].lo : 0;
                        const int w_front = q0 ? (int)(rec[q0 - 1].shape & 0xFFFFu) : 1;
                        // where a cell's row index comes from in the row in front, in bytes
                        const int d = c.lo - lo_front - (int)s.bin[t], at = (s.first[i] & 0xFFFF) + (int)rank;
                        uint2 x = make_uint2((uint32_t)(4 * d), (s.size[t] << bits) | (bits ? rank : 0u));
                        if (d >= w_front || d <= -(int)(c.shape & 0xFFFFu)) {     // leads from no cell of the row in front into this one
                            x = make_uint2(0u, kInfPacked);
                        } else {
                            down = max(down, (uint32_t)max(-d, 0));
                            up = max(up, (uint32_t)max(d, 0));
                        }
                        ent[at] = x;
                        ent_cand[at] = s.cand[t];
                    }
                }
            }
            down = wave_max_u32(down);
            up = wave_max_u32(up);
            if (lane == 0 && (down | up)) {
                atomicMax(&s.facts[0], down);
                atomicMax(&s.facts[1], up);
            }
            __syncthreads();
            const int w_max = (int)s.acc[3];
            const SweepShape form = sweep_shape(w_max);
            const int row_cells = form.threads * form.per;
            // rows behind the survivors (and the words a wavefront reads past the last list), then the
            // arg-min bytes where they fit
            const size_t at_row = sizeof(Core) * (size_t)max(n_core, 1) + sizeof(uint2) * ((size_t)ents + 64) + ((size_t)ents + 15) / 16 * 16;
            Sweep sw{rec, ent, reinterpret_cast<uint32_t*>(region + at_row), p.pd, (int)s.facts[0],
                     (int)(s.facts[0] + s.facts[1]) + row_cells, n_core, 0};
            size_t row_bytes = sizeof(uint32_t) * (size_t)sw.cells * (form.two ? 2 : 1);
            const bool lists = at_row + row_bytes > kRegionBytes;
            const bool pd_lds = !lists && at_row + row_bytes + cells + (size_t)row_cells <= kRegionBytes;
            if (pd_lds) sw.pd = region + at_row + row_bytes;
            sw.bits = bits;
            // (lists long enough that the positions do not fit the costs or a word are swept with bytes)
            const bool words = !lists && !pd_lds && bits && s.facts[2] <= 64 && form.threads == kThreadsS && form.per * bits <= 32 &&
                               ((size_t)p.pd & 3) == 0 && (size_t)n_core * 4 * kThreadsS <= (size_t)L * (size_t)(p.D + 1);
            if (s.flags & 4) {
                status = 2;
            } else if ((s.flags & 8) || (int)shift_all > D) {        // a layer no bin sum can reach
                status = reduce ? 2 : 1;
            } else if (lists && !(LAST && P <= 64)) {
                status = 4;
            } else {
                const uint32_t* last = sw.buffer;
                const int cand_bits = 32 - __builtin_clz(P - 1);                       // (lists: P is at least 2)
                const bool pack_cand = ((unsigned long long)s.facts[3] << cand_bits) < kInfPacked;
                const int row_bits = LAST && lists ? (pack_cand ? cand_bits : 0) : bits;
                if (n_core == 0) {
                    if (tid == 0) sw.buffer[0] = 0;
                    __syncthreads();
                } else if (LAST && lists) {      // (the row takes the survivors' place)
                    uint32_t* const buffer = reinterpret_cast<uint32_t*>(ent);
                    if constexpr (LAST) {
                        if (w_max < 6 * kThreadsS)
                            last = pack_cand ? sweep_lists<6, true>(s, rec, buffer, p.pd, n_core, cand_bits)
                                             : sweep_lists<6, false>(s, rec, buffer, p.pd, n_core, 0);
                        else if (w_max < 10 * kThreadsS)
                            last = pack_cand ? sweep_lists<10, true>(s, rec, buffer, p.pd, n_core, cand_bits)
                                             : sweep_lists<10, false>(s, rec, buffer, p.pd, n_core, 0);
                        else
                            last = pack_cand ? sweep_lists<kMaxRow / kThreadsS, true>(s, rec, buffer, p.pd, n_core, cand_bits)
                                             : sweep_lists<kMaxRow / kThreadsS, false>(s, rec, buffer, p.pd, n_core, 0);
                    }
                } else if (words) {
                    last = sweep_shaped<true, true, false>(form, sw);
                } else if (bits) {
                    last = pd_lds ? sweep_shaped<true, false, true>(form, sw) : sweep_shaped<true, false, false>(form, sw);
                } else {
                    last = pd_lds ? sweep_shaped<false, false, true>(form, sw) : sweep_shaped<false, false, false>(form, sw);
                }
                // smallest total, lowest cell among equals, inside the budget
                const int base = n_core ? (int)s.acc[0] : 0, top = n_core ? base + (int)s.acc[1] - 1 : 0;
                uint32_t low = kInfS, cell = ~0u;            // (cells in rising order: the first of equals stays)
                for (int e = base + tid; e <= min(top, D - (int)shift_all); e += kThreadsS) {
                    const uint32_t raw = last[e - base], v = raw >= kInfS ? kInfS : raw >> row_bits;
                    if (v < low) {
                        low = v;
                        cell = (uint32_t)e;
                    }
                }
                if ((tid & ~63) <= top - base) {
                    const uint32_t v = wave_min_u32(low), e = wave_min_u32(low == v ? cell : ~0u);
                    if (lane == 0) atomicMin(&s.best, ((unsigned long long)v << 32) | e);
                }
                if (tid == 0) t_sweep = wall_clock64();
                __syncthreads();
                const unsigned long long b = s.best;
                if ((uint32_t)(b >> 32) >= kInfS) {
                    status = reduce ? 2 : 1;
                } else {
                    // ---- back-trace: one arg-min byte per core layer is the chain; records and survivors'
                    // bins are fetched ahead of it.  A byte that cannot be is caught by the sums below
                    // (LDS reads stay in range by themselves; the walk in device memory is clamped).
                    if (LAST && lists && wave == 0) {
                        int t = (int)(uint32_t)b - base;
                        for (int j = n_core - 1; j >= 0; --j) {
                            const int a = min(max(rec[j].trace + t, 0), (int)cells - 1), i = s.lo[j];
                            const uint32_t cd = (uint32_t)__builtin_amdgcn_readfirstlane((int)p.pd[a]);
                            const int first = s.off[i], k0 = first + lane;       // (a list holds a candidate once)
                            const unsigned long long m = __ballot(k0 < s.off[i + 1] && s.cand[min(k0, kMaxT - 1)] == cd);
                            if (!m) break;                // (the sums below differ)
                            const int k = first + (int)__builtin_ctzll(m);
                            if (lane == 0) s.hi[j] = k;
                            t += rec[j].step - (int)s.bin[k];
                        }
                        if (lane == 0 && t != 0) atomicOr(&s.flags, 16);
                    } else if (wave == 0 && n_core > 0) {
                        // (in places of the rows: the sum of bins less the row's first; in front of the first layer 0)
                        int t = (int)(uint32_t)b - base;
                        const uint32_t pd_at = lds_address(reinterpret_cast<const uint32_t*>(region)) + (uint32_t)(at_row + row_bytes);
                        const uint32_t places = bits ? (1u << bits) - 1u : 255u;
                        // 64 layers at a time, lane i holding what layer q0 + i needs
                        for (int q0 = (n_core - 1) & ~63; q0 >= 0; q0 -= 64) {
                            const int mine = min(q0 + lane, n_core - 1);
                            const uint32_t trace = (uint32_t)rec[mine].trace, head = (uint32_t)s.hi[mine];
                            uint32_t picked = 0;
                            const int top = min(63, n_core - 1 - q0);
                            uint32_t b1 = ent[(int)lane_u32(head, top) + lane].x;
                            auto walk = [&](auto place) __attribute__((always_inline)) {
#pragma unroll 4
                                for (int i = top; i >= 0; --i) {
                                    const uint32_t b0 = b1;
                                    b1 = ent[(int)lane_u32(head, max(i - 1, 0)) + lane].x;
                                    const uint32_t kk = place(i);
                                    picked = lane == i ? kk : picked;
                                    t += (int)lane_u32(b0, (int)(kk & 63u)) >> 2;
                                }
                            };
                            if (s.facts[2] > 64) {        // longer lists than a wavefront holds
                                for (int i = top; i >= 0; --i) {
                                    const int a = min(max((int)lane_u32(trace, i) + t, 0), (int)cells - 1);
                                    const uint32_t kk = (uint32_t)__builtin_amdgcn_readfirstlane((int)sw.pd[a]) & places;
                                    picked = lane == i ? kk : picked;
                                    t += __builtin_amdgcn_readfirstlane((int)ent[(int)lane_u32(head, i) + (int)min(kk, 127u)].x) >> 2;
                                }
                            } else if (pd_lds) {
                                walk([&](int i) __attribute__((always_inline)) {
                                    return (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_byte(pd_at + lane_u32(trace, i) + (uint32_t)t)) & places;
                                });
                            } else if (words) {
                                walk([&](int i) __attribute__((always_inline)) {
                                    const int a = min(max(t, 0), row_cells - 1);
                                    const uint32_t w = reinterpret_cast<const uint32_t*>(p.pd)[(q0 + i) * kThreadsS + (a & (kThreadsS - 1))];
                                    return ((uint32_t)__builtin_amdgcn_readfirstlane((int)w) >> (bits * (a / kThreadsS))) & places;
                                });
                            } else {
                                walk([&](int i) __attribute__((always_inline)) {
                                    const int a = min(max((int)lane_u32(trace, i) + t, 0), (int)cells - 1);
                                    return (uint32_t)__builtin_amdgcn_readfirstlane((int)p.pd[a]) & places;
                                });
                            }
                            if (lane <= top) s.pick[q0 + lane] = (uint8_t)picked;
                        }
                        if (lane == 0 && t != 0) atomicOr(&s.flags, 16);
                    }
                    __syncthreads();
                    // the assignment, and what it adds up to
                    uint32_t pb = 0, pz = 0;
                    if (single) {
                        pb = s.bin[only];
                        pz = s.size[only];
                        s.chosen[s.layer[tid]] = s.cand[only];
                    }
                    if (LAST && lists && tid < n_core) {  // (the walk left the entries)
                        const int at = min(s.hi[tid], kMaxT - 1);
                        pb += s.bin[at];
                        pz += s.size[at];
                        s.chosen[s.layer[s.lo[tid]]] = s.cand[at];
                    } else if (tid < n_core) {
                        const int at = s.hi[tid] + min((int)s.pick[tid], (int)(rec[tid].shape >> 16) - 1);
                        const uint2 x = ent[at];
                        pb += (uint32_t)(rec[tid].step - ((int)x.x >> 2));
                        pz += x.y >> bits;
                        s.chosen[s.layer[s.lo[tid]]] = ent_cand[at];
                    }
                    const uint32_t wb = wave_total(pb), wz = wave_total(pz);
                    if (lane == 0 && (wb | wz)) atomicAdd(&s.sums, ((unsigned long long)wb << 32) | wz);
                    __syncthreads();
                    const uint32_t tb = (uint32_t)(s.sums >> 32), tz = (uint32_t)s.sums;
                    total_bins = tb;
                    total_size = tz;
                    if ((s.flags & 16) || tb != (uint32_t)b + shift_all || tz != (uint32_t)(b >> 32) + s.acc[2]) status = 2;
                }
            }
        }
    }
    __syncthreads();

    // ---- the compression's layer records: one thread per layer, payload offsets from a running sum of
    // the chosen sizes rounded up to 16 bytes
    const int c = tid < L ? (int)s.chosen[tid] : 0;
    int64_t applied = 0;
    if (p.apply.layers) {
        const SolveApply& A = p.apply;
        bool ok = status == 0;
        const bool mine = tid < L;
        const int cc = c < P ? c : 0;
        if (mine && c >= P) atomicOr(&s.flags, 32);
        int64_t raw = 0;
        int32_t fam = 0, ipar = 0, tslot = -1;
        if (mine && ok) {                                // the table reads of the chosen column go out together
            raw = p.sizes[(size_t)tid * P + cc];
            fam = A.family[cc];
            tslot = A.topk_slot[cc];
            ipar = A.iparam[(size_t)tid * P + cc];
        }
        // (sizes in units of 16 bytes: the total of a table with 32-bit costs fits 32 bits)
        uint32_t all16;
        const uint32_t off16 = block_scan(mine && ok ? (uint32_t)((raw + 15) >> 4) : 0u, s.tmp, &all16);
        ok = ok && !(s.flags & 32) && (int64_t)all16 * 16 <= A.capacity;
        if (mine) {
            if (ok) {
                A.layers[tid].payload = (int64_t)off16 * 16;
                A.layers[tid].family = fam;
                A.layers[tid].iparam = ipar;
                A.layers[tid].slot = tslot;
            } else {
                A.layers[tid].family = -1;
            }
        }
        applied = ok ? 1 : 0;
    }
    // ---- hand-over.  The result block lies in the host's pinned memory and the host may be polling it.
    // What the host relies on does not depend on the order in which stores arrive there: the
    // block's slots go out as ONE store of the first wavefront (lane i holds slot i; each 64-byte
    // half carries a copy of the launch's sequence number), error table and assignment are covered
    // by check words in it, and slot 7, which the host polls, follows behind a system-scope fence.
    unsigned long long cs = 0;
    if (tid < L) {
        const int32_t out = status == 0 ? c : -1;
        p.choice[tid] = out;
        cs = (unsigned long long)(uint32_t)(out + 1) * (unsigned long long)(tid + 1);
    }
    cs = wave_total(cs);
    if (lane == 0 && cs) atomicAdd(&s.chk_choice, cs);
    __syncthreads();
    if (wave == 0) {
        const uint64_t t_s = ((uint64_t)lane_u32((uint32_t)(t_sweep >> 32), 0) << 32) | lane_u32((uint32_t)t_sweep, 0);
        const uint64_t ticks_sweep = t_s - t_begin, ticks_rest = wall_clock64() - t_s;
        int64_t v = 0;
        bool mine = true;
        switch (lane) {
            case 0: v = status; break;
            case 1: v = status == 0 ? total_size : 0; break;
            case 2: v = status == 0 ? total_bins : 0; break;
            // ticks of the constant-rate (100 MHz) counter: up to the end of the sweep, and from there
            case 3: v = (int64_t)((ticks_sweep & 0xFFFFFFFFull) | (ticks_rest << 32)); break;
            case 4: v = p.seq; break;
            case 5: v = L; break;
            case 6: v = (int64_t)__builtin_bit_cast(uint64_t, e_max); break;
            case 8: v = applied; break;
            case 9: v = 0; break;                        // swept in one piece
            case 10: v = (int64_t)s.chk_choice; break;
            case 11: v = (int64_t)s.chk_err; break;
            case 15: v = p.seq; break;
            default: mine = false;
        }
        if (mine) p.result[lane] = v;
        __threadfence_system();
        if (tid == 0) p.result[7] = p.seq;
    }
}

}  // namespace

hipError_t launch_solve(const SolveParams& p, hipStream_t s, Section* sec) {
    if (p.L < 1 || p.L > kSolveMaxLayers || p.P < 1 || p.P > LGRECO_MAX_CANDS || p.L * p.P > kSolveMaxLP)
        return hipErrorInvalidValue;
    const size_t lds = sizeof(Lds) + kRegionBytes;
    static_assert(sizeof(Lds) % 16 == 0 && sizeof(Lds) + kRegionBytes <= 160 * 1024, "LDS of one compute unit");
    static_assert(kRegionBytes >= sizeof(Relax), "the intervals' tables fit");
    static_assert(kMaxRow > LGRECO_MAX_BINS, "a thread's cells cover the widest row");
    static_assert(kRegionBytes >= sizeof(Core) * kSolveMaxLayers + sizeof(uint32_t) * (LGRECO_MAX_BINS + 3),
                  "records and the widest row always fit");
    static bool configured = false;
    if (!configured) {
        for (const void* k : {(const void*)solve_kernel<4, false>, (const void*)solve_kernel<16, false>, (const void*)solve_kernel<4, true>}) {
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        configured = true;
    }
    const bool small = p.L * p.P <= 4 * kThreadsS;
    if (p.last_resort && !small) return hipErrorInvalidValue;
    if (p.last_resort) launch_timed(sec, true, true, solve_kernel<4, true>, dim3(1), dim3(kThreadsS), lds, s, p);
    else if (small) launch_timed(sec, true, true, solve_kernel<4, false>, dim3(1), dim3(kThreadsS), lds, s, p);
    else launch_timed(sec, true, true, solve_kernel<16, false>, dim3(1), dim3(kThreadsS), lds, s, p);
    return hipGetLastError();
}

}  // namespace lgreco
