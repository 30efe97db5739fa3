// PowerSGD-style low rank: one power-iteration step per layer on the matrix pipes, fp32 products and sums, for gfx950.
//
//   P = X Q0            X = g + e viewed as [m x n] row-major, Q0 [n x 64] warm start
//   Phat = orth(P)      Gram-Schmidt on the columns, done in coefficient space: G = P^T P in
//                       fp64, one wavefront per layer runs the column-by-column elimination
//                       on the 64 x 64 Gram matrix (lane j owns column j; this is exactly the
//                       Gram-Schmidt recurrence on the inner products), inverts the triangular
//                       factor and Phat = P T.  A column whose squared norm after projection is
//                       0 or below 1e-10 x its squared norm before projection becomes zero.
//   Q = X^T Phat
//   error_r = ||X||^2 - sum_{j<r} ||q_j||^2    (Phat orthonormal, Q = X^T Phat, and the factors
//                       of rank r are the leading columns of the rank-64 run, so one run yields
//                       every rank's error)
//   compress: payload Phat[:, :r], Q[:, :r];  e' = X - Phat[:, :r] Q[:, :r]^T
//
// The reconstruction uses v_mfma_f32_32x32x2f32 (fp32 in, fp32 accumulate), the two contractions the bf16
// instruction on values cut in three (see split8).  Operand layout of the former, lane l of 64:
//   A (32 x 2): A[i = l % 32][k = l / 32];   B (2 x 32): B[k = l / 32][j = l % 32]
//   D (32 x 32): register v (0..15) holds D[8 (v / 4) + 4 (l / 32) + v % 4][l % 32]
#include <cstring>
#include <type_traits>

#include "internal.h"
#include "pack.h"

namespace lgreco {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kLrCols = 64;       // columns computed per layer (r_max <= 64)
constexpr int kLrBM = 128;        // rows (GEMM1) / columns (GEMM2) per workgroup
constexpr int kLrBK = 32;         // contraction chunk staged in LDS
constexpr int kLrGramSpan = 128;  // rows per Gram partial (one workgroup)
constexpr int kLrQChunk = 64;     // Q rows per workgroup in the split-K reduction
constexpr int kLrPSplit = 512;    // columns contracted per workgroup in P = X Q0

struct LrLayer {
    int64_t offset;     // into g / e
    int64_t x_off;      // into LrParams::x
    int64_t q_off;      // into q0 / q (stride r_max)
    int64_t p_off;      // into the P scratch (rows x 64)
    int64_t qs_off;     // into the Q scratch (cols x 64)
    int64_t part_off;   // into the split-K partial buffer (splits x cols x 64)
    int64_t payload;    // byte offset of the payload (compress)
    int32_t rows, cols;
    int32_t rank;       // columns written out (64 when profiling)
    int32_t splits, ksplit;         // split of the row contraction of Q = X^T Phat
    int32_t psplits, pksplit;       // split of the column contraction of P = X Q0
    int64_t ppart_off;              // into the P partial buffer (psplits x rows x 64) when psplits > 1
    int32_t gram_begin, gram_end;   // Gram partial range
    int32_t rt_begin, rt_end;       // row-tile range (||X||^2 partials)
    int32_t qc_begin, qc_end;       // Q-chunk range (column-norm partials)
    int32_t index;      // index in the caller's layer table
    int32_t lines;      // every row piece of 32 elements is a whole line (see lr_ef_kernel)
};
struct LrTile {
    int32_t layer, a0, split, pad;
};

struct LrParams {
    const float* g;
    const float* e;          // may be null
    // x = g + e, left there by the first contraction where there is an e for everything that reads the matrix after it
    // (e null, from_x set): a pass over one buffer instead of two.
    float* x;
    int32_t from_x;
    float* e_out;            // compress: error feedback (same buffer as e)
    const float* q0;         // warm start (stride r_max)
    float* q_out;            // compress: new Q (stride r_max), same buffer as q0
    int32_t r_max;
    const LrLayer* layers;
    const LrTile* row_tiles;   // 128-row tiles (orthogonalisation)
    const LrTile* p_tiles;     // (128-row tile, column split) of P = X Q0
    const LrTile* ef_tiles;    // (32 rows, 128 columns) of the reconstruction
    const LrTile* col_tiles;
    const LrTile* gram_tiles;
    const LrTile* q_chunks;
    float* P;                // scratch [sum rows x 64]
    float* Q;                // scratch [sum cols x 64]
    float* part;             // split-K partials of Q
    float* ppart;            // split-K partials of P
    double* gram_part;       // [gram tiles x 64 x 64]
    double* T;               // [layers x 64 x 64]
    double* xnorm_part;      // [row tiles]
    double* qnorm_part;      // [q chunks x 64]
    uint8_t* payload;
    double* errors;          // [L x stride]
    int32_t stride;
    int32_t nrank;
    int32_t rank[LGRECO_MAX_CANDS];
    int32_t col[LGRECO_MAX_CANDS];
    int32_t accumulate;      // decode: add the image to the output instead of replacing it
    int32_t q_from_scratch;  // P = X Q reads the previous step's Q instead of the warm start
    int32_t e_is_zero;       // compression: e is null because the caller promised zeros; x = fl32(g + 0) all the same
    int32_t n_ef_tiles, n_row_tiles;     // KNOWN: workgroups behind the first n_ef_tiles fill payload and warm start
    const DevLayer* dev_layers;   // KNOWN kernels: the caller's layer records (family, rank, payload offset) on the device
};

// An address as a scalar base and a lane's byte offset, the form that costs no vector instructions.  Rows as wide as
// kLrWide, whose offsets do not fit, take the paths of a matrix's edges.
constexpr int kLrWide = 1 << 26;
template <typename T>
__device__ __forceinline__ T* at_bytes(T* base, uint32_t offset) {
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type byte;
    auto p = (__attribute__((address_space(1))) byte*)reinterpret_cast<byte*>(base);
    asm("" : "+s"(p));                                       // (uniform; not to be folded into the lane's part)
    return (T*)(p + offset);
}

// ------------------------------------------------------------------ fp32 products from bf16 pieces
// An fp32 value is the sum of three bf16 values, exactly: its upper 16 bits (cut off, so that nothing overflows), the
// rounded upper bits of the rest, and what is left (8 bits at most).  The second reaches 2^-7 of the value's leading power
// of two and the third 2^-16.  Of the nine products of two such sums all but that of the two third pieces, 2^-32 of the
// whole at most, are formed on v_mfma_f32_32x32x16_bf16 (products exact, fp32 accumulate).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
struct Split8 { bf16x8 piece[3]; };                          // 8 values: largest pieces first
__device__ __forceinline__ Split8 split8(const float* x) {
    union { uint32_t w[4]; bf16x8 v; } h, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t u0 = __float_as_uint(x[2 * i]), u1 = __float_as_uint(x[2 * i + 1]);
        h.w[i] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
        const float r0 = x[2 * i] - __uint_as_float(u0 & 0xFFFF0000u), r1 = x[2 * i + 1] - __uint_as_float(u1 & 0xFFFF0000u);
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        m.w[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{r0, r1}, bf16x2));
        const float l0 = r0 - __uint_as_float(m.w[i] << 16), l1 = r1 - __uint_as_float(m.w[i] & 0xFFFF0000u);
        l.w[i] = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);
    }
    return Split8{{h.v, m.v, l.v}};
}
// c + a b over a chunk of 32: two operands of 16 each a side; b(s, piece) is the second's.  The products of the first
// pieces go to c itself, the others are added up from zero and then to c by a vector addition: the instruction rounds
// to nearest where c is the larger part and cuts c off where the products are, by up to an ulp of what it gives.
// So a product alone is as good as one rounded to fp32 (262144 of them: 1.0 x 2^-24 at most, 0.43 in the mean square, as with the
// fp32 instruction; without the products of second with third pieces and with everything added to c 4.5 and 0.70), and a sum, with five roundings
// a chunk where the fp32 instruction has 32, better: of 16 to 512 normal terms 0.15 to 0.27 x 2^-24 of the sum of magnitudes in
// the mean square against 0.42 to 0.54, of 512 terms of one sign 2.1 to 2.4 against 5.0 to 5.7.
template <typename B>
__device__ __forceinline__ f32x16 mfma_split(const Split8 (&a)[2], B b, f32x16 c) {
    f32x16 t = {0};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const bf16x8 h = b(s, 0), m = b(s, 1), l = b(s, 2);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[1], l, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[2], m, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[0], l, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[2], h, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[1], m, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[0], m, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[1], h, t, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s].piece[0], h, c, 0, 0, 0);
    }
    return c + t;
}

// Values below 2^-110 lose bits: what they leave for the third piece falls below bf16's subnormals.  That is less than 2^-133,
// nothing beside values of the same sum some 2^30 times as large, but all that counts where there are none.  So a
// wavefront that has met no value as large as below forms its sums once more (where all are zero, if its operands are not: below 2^-134
// nothing is left for the first piece either), from the fp32
// values on the fp32 instruction, two rows of the contraction a step (a compression of 67 M elements around 1e-33: 962 us instead
// of 437, from 1e-25 up 437; of zeros, which are read once more to see that they are, 459).  Rows of values below 2^-110 that share a wavefront with larger ones keep what is left of their
// values above 2^-133.
constexpr float kLrHeldQ0 = 0x1p-100f;          // Q0
constexpr float kLrHeldP = 0x1p-91f;            // P = X Q0 over the largest of Q0: 512 values of X lose at most 2^-124 of it, 2^-33 of this
constexpr float kLrHeldQ = 0x1p-90f;            // Q = X^T Phat: K values of X lose at most 2^-133 sqrt(K), 2^-30 of this where K < 2^26
__device__ __forceinline__ float largest(f32x16 a, f32x16 b) {
    float v = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) v = fmaxf(fmaxf(fabsf(a[i]), fabsf(b[i])), v);
    return v;
}
// Whether one of the wavefront's values is not zero; bits(i), i < count: this lane's, or several together.
__device__ __forceinline__ uint32_t bits_of(float4 v) {
    return __float_as_uint(v.x) | __float_as_uint(v.y) | __float_as_uint(v.z) | __float_as_uint(v.w);
}
template <typename Bits>
__device__ __forceinline__ bool any_value(int count, Bits bits) {
    for (int i = 0; i < count; i += 8) {
        uint32_t all = 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) all |= bits(min(i + u, count - 1));
        if (__any((all << 1) != 0)) return true;
    }
    return false;
}
// left(k), right(k, 0) and right(k, 1): this lane's values of the operands at k
template <typename Left, typename Right>
__device__ __forceinline__ void mfma_plain(int kbeg, int kend, int half, Left left, Right right, f32x16& c0, f32x16& c1) {
    c0 = f32x16{0};
    c1 = f32x16{0};
    for (int k = kbeg; k < kend; k += 2) {
        const int kk = min(k + half, kend - 1);
        const float a = k + half < kend ? left(kk) : 0.0f;
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a, right(kk, 0), c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a, right(kk, 1), c1, 0, 0, 0);
    }
}

// The matrix as everything behind the first contraction reads it.
__device__ __forceinline__ const float* matrix_of(const LrParams& p, const LrLayer& L) {
    return p.from_x ? p.x + L.x_off : p.g + L.offset;
}

// ------------------------------------------------------------------ P = X Q0 (and ||X||^2)
// One workgroup: 128 rows x 64 columns of P over one column range of X, 32 columns at a time; wavefront w owns rows
// 32w .. 32w+31.  Bound by HBM where there is an e (g and e in, x out).  A wavefront's loads take 8 rows of 128 bytes each (g and e past the caches
// where those are whole lines), x leaves in the same pieces, and the operand (a lane holds a row) is formed through the wavefront's own LDS rows, which no other
// wavefront touches; the 32 x 64 chunk of Q0, shared by the four, is staged as pieces between two barriers.
// Rows are 36 words apart, 16 lanes of a 128-bit read on different banks.  Products on the bf16 matrix pipe (see split8).
// 67 M elements of 66 matrices: 167 -> 160 us, 5.0 TB/s of g, e and x (a bare read and write in this shape 148); without e 98 -> 86
// (79 with six products, all added to the accumulator), where the fp32 instruction's alone took 70; 73 M elements of odd widths: a step 698 -> 678.  Three wavefronts on a SIMD with e: at four
// registers spill (167 us).  A lane loading and storing 16 consecutive elements of its own row, 64 pieces of lines an instruction: 190;
// 16 rows of 64 bytes an instruction, the operand's own layout: 175 to 250 for the bare read and write.
// HAS_E: x = g + e is formed here and written to LrParams::x, for the caches: the passes behind read it.
constexpr int kLrXPitch = kLrBK + 4;
template <bool HAS_E>
__global__ __launch_bounds__(256, HAS_E ? 3 : 4) void lr_gemm1_kernel(LrParams p) {
    __shared__ __align__(16) float Xs[4][32][kLrXPitch];
    __shared__ __align__(16) bf16x8 Qs[kLrBK / 8][3][kLrCols];       // [8 rows][piece][column]
    __shared__ double s_red[4];
    __shared__ float s_qmax[4];
    const LrTile tile = p.p_tiles[blockIdx.x];
    const LrLayer L = p.layers[tile.layer];
    const int m = L.rows, n = L.cols, row0 = tile.a0;
    const int kbeg = tile.split * L.pksplit, kend = min(n, kbeg + L.pksplit);
    const float* __restrict__ g = (HAS_E ? p.g + L.offset : matrix_of(p, L)) + (int64_t)row0 * n;
    // (x may take the place of e: read before it is written, by the same lane)
    const float* e = HAS_E ? p.e + L.offset + (int64_t)row0 * n : nullptr;
    float* const xo = HAS_E ? p.x + L.x_off + (int64_t)row0 * n : nullptr;
    // first power-iteration step: the caller's warm start (row stride r_max); later steps: the Q
    // of the previous step in the scratch buffer (row stride 64)
    const bool qscr = p.q_from_scratch != 0;
    const float* __restrict__ q = qscr ? p.Q + L.qs_off : p.q0 + L.q_off;
    const int qstride = qscr ? kLrCols : p.r_max;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int half = lane >> 5, bj = lane & 31;
    // this lane's share of a chunk: rows 8 s + lane / 8 of the wavefront's, columns lc .. lc + 3.  Rows past the end
    // read the last one; nothing of theirs is written, summed or stored.
    const int lc = 4 * (lane & 7);
    uint32_t at[4];                                      // (below 2^31, as the layer's size is)
    bool row_ok[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int r = 32 * wave + 8 * s + (lane >> 3);
        row_ok[s] = row0 + r < m;
        at[s] = (uint32_t)min(r, m - 1 - row0) * (uint32_t)n + (uint32_t)lc;
    }
    const int nchunks = (kend - kbeg + kLrBK - 1) / kLrBK;
    f32x16 acc0 = {0}, acc1 = {0};
    float xsq = 0.0f, qmax = 0.0f;
    // (two copies of the loop: of a choice at each access the compiler makes one, without the hint)
    const auto span = [&](auto whole_lines) __attribute__((always_inline)) {
        constexpr bool lines = decltype(whole_lines)::value;
        float4 xg[4], xe[HAS_E ? 4 : 1];
        float qr[8];
        // issue the loads of one chunk (their values are first used after the MFMAs of the chunk
        // that is being multiplied)
        auto fetch = [&](int k0) __attribute__((always_inline)) {
            const float* const gk = g + k0;
            const float* const ek = HAS_E ? e + k0 : nullptr;
            if (k0 + kLrBK <= kend) {                        // uniform
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    xg[s] = HAS_E && lines ? load_stream(gk + at[s]) : load4_any(gk + at[s]);
                    if (HAS_E) xe[s] = lines ? load_stream(ek + at[s]) : load4_any(ek + at[s]);
                }
            } else {
                const int left = kend - k0 - lc;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float* const gs = gk + at[s];
                    xg[s] = make_float4(left > 0 ? gs[0] : 0.f, left > 1 ? gs[1] : 0.f, left > 2 ? gs[2] : 0.f, left > 3 ? gs[3] : 0.f);
                    if (HAS_E) {
                        const float* const es = ek + at[s];
                        xe[s] = make_float4(left > 0 ? es[0] : 0.f, left > 1 ? es[1] : 0.f, left > 2 ? es[2] : 0.f, left > 3 ? es[3] : 0.f);
                    }
                }
            }
            // Q0: this wavefront's 8 rows of the chunk, a column a lane; zero past the range and the columns there are
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = k0 + 8 * wave + u;
                qr[u] = k < kend && lane < qstride ? q[(int64_t)k * qstride + lane] : 0.0f;
            }
        };
        // take the fetched chunk into use: x = g + e, ||x||^2, x to memory and LDS, Q0 rows to LDS
        auto commit = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                float4 v = xg[s];
                if (HAS_E) { v.x += xe[s].x; v.y += xe[s].y; v.z += xe[s].z; v.w += xe[s].w; }
                if (HAS_E && row_ok[s]) {
                    float* const xs = xo + k0 + at[s];
                    const int left = kend - k0 - lc;
                    if (k0 + kLrBK <= kend) {                // uniform
                        store4_any(xs, v);
                    } else {
                        if (left > 0) xs[0] = v.x;
                        if (left > 1) xs[1] = v.y;
                        if (left > 2) xs[2] = v.z;
                        if (left > 3) xs[3] = v.w;
                    }
                }
                *reinterpret_cast<float4*>(&Xs[wave][8 * s + (lane >> 3)][lc]) = v;
                if (row_ok[s]) {
                    xsq = __builtin_fmaf(v.x, v.x, xsq);
                    xsq = __builtin_fmaf(v.y, v.y, xsq);
                    xsq = __builtin_fmaf(v.z, v.z, xsq);
                    xsq = __builtin_fmaf(v.w, v.w, xsq);
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) qmax = fmaxf(qmax, fabsf(qr[u]));
            const Split8 b = split8(qr);
#pragma unroll
            for (int t = 0; t < 3; ++t) Qs[wave][t][lane] = b.piece[t];
        };
        fetch(kbeg);
        for (int c = 0; c < nchunks; ++c) {
            const int k0 = kbeg + c * kLrBK;
            commit(k0);
            __syncthreads();
            if (c + 1 < nchunks) fetch(k0 + kLrBK);
            Split8 a[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float4 lo = *reinterpret_cast<const float4*>(&Xs[wave][bj][16 * s + 8 * half]);
                const float4 hi = *reinterpret_cast<const float4*>(&Xs[wave][bj][16 * s + 8 * half + 4]);
                const float row[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                a[s] = split8(row);
            }
            acc0 = mfma_split(a, [&](int s, int t) { return Qs[2 * s + half][t][bj]; }, acc0);
            acc1 = mfma_split(a, [&](int s, int t) { return Qs[2 * s + half][t][32 + bj]; }, acc1);
            __syncthreads();                                 // (the rows of Q0 are written again)
        }
    };
    if (HAS_E && L.lines) span(std::true_type());
    else span(std::false_type());
    const double s = wave_sum((double)xsq);
    for (int o = 32; o > 0; o >>= 1) qmax = fmaxf(qmax, __shfl_xor(qmax, o, 64));
    if (lane == 0) {
        s_red[wave] = s;
        s_qmax[wave] = qmax;
    }
    __syncthreads();                                         // (also: what the wavefront has written to xo, for its other lanes)
    if (tid == 0) p.xnorm_part[blockIdx.x] = s_red[0] + s_red[1] + s_red[2] + s_red[3];
    qmax = fmaxf(fmaxf(s_qmax[0], s_qmax[1]), fmaxf(s_qmax[2], s_qmax[3]));
    const float most = largest(acc0, acc1);
    const bool held = qmax >= kLrHeldQ0 && __any(most >= kLrHeldP * qmax);
    const float* const x = HAS_E ? xo : g;
    const auto some = [&] {
        if (kend - kbeg < 4)
            return any_value(32, [&](int i) {
                return __float_as_uint(x[(int64_t)min(32 * wave + i, m - 1 - row0) * n + min(kbeg + lane, kend - 1)]);
            });
        const int id = __lane_id();                          // (found anew: kept through the loop the register spills others)
        return any_value(4 * ((kend - kbeg + 31) / 32), [&](int i) {         // 8 rows of 32 columns at a time
            const int r = min(32 * wave + 8 * (i & 3) + (id >> 3), m - 1 - row0);
            return bits_of(load4_any(x + (int64_t)r * n + min(kbeg + 32 * (i >> 2) + 4 * (id & 7), kend - 4)));
        });
    };
    if (!held && row0 + 32 * wave < m && (__any(most > 0.0f) || (qmax > 0.0f && some()))) {      // (uniform)
        const float* const row = x + (int64_t)min(32 * wave + bj, m - 1 - row0) * n;
        mfma_plain(kbeg, kend, half, [&](int k) { return row[k]; },
                   [&](int k, int c) { return 32 * c + bj < qstride ? q[(int64_t)k * qstride + 32 * c + bj] : 0.0f; }, acc0, acc1);
    }
    float* __restrict__ P = L.psplits > 1 ? p.ppart + L.ppart_off + (int64_t)tile.split * m * kLrCols
                                          : p.P + L.p_off;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int orow = row0 + 32 * wave + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (orow < m) {
            P[(int64_t)orow * kLrCols + bj] = acc0[v];
            P[(int64_t)orow * kLrCols + 32 + bj] = acc1[v];
        }
    }
}

// ------------------------------------------------------------------ partial Gram matrices
// G = P^T P over a span of rows, accumulated in fp64 on v_mfma_f64_16x16x4f64.  Operand layout of
// that instruction, lane l of 64:  A (16 x 4): A[i = l % 16][k = l / 16];  B (4 x 16):
// B[k = l / 16][j = l % 16];  D (16 x 16): register v (0..3) holds D[4 v + l / 16][l % 16].
// With A = P^T and B = P both operands of a 4-row step are values P[row0 + l / 16][16 b + l % 16] of the
// same lane.  The instruction takes a SIMD 64 cycles and bounds the kernel, so only the 10 blocks of 16 x 16 on
// and above the diagonal are computed (nothing below it is ever read), dealt to the four wavefronts so
// that none has more than three and each finishes its own: nothing is added up across wavefronts.
// The span goes through LDS once; where P was computed in column splits their sum is formed on the way
// in (split order) and written to P.  LDS word 16 (b ^ (row & 3)) + c of a row holds column 16 b + c: the four rows
// of a step lie on different banks.  On 106 k rows of 66 layers: 21 us, of which the products are 12 (30 with spans of
// 256 rows, whose registers and LDS leave two workgroups on a compute unit; 24 with 64 rows, and the sum of the
// partials behind it 10 instead of 6).
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <int... AB>
struct GramBlocks {                          // row block, column block; ...
    static constexpr int n = sizeof...(AB) / 2;
    static constexpr int ab[sizeof...(AB)] = {AB...};
    __device__ static constexpr int a(int i) { return ab[2 * i]; }
    __device__ static constexpr int b(int i) { return ab[2 * i + 1]; }
    __device__ static constexpr bool uses(int v) { return ((AB == v) || ...); }
};

__global__ __launch_bounds__(256, 4) void lr_gram_kernel(LrParams p) {
    __shared__ float Ps[kLrGramSpan][kLrCols];
    const LrTile tile = p.gram_tiles[blockIdx.x];
    const LrLayer L = p.layers[tile.layer];
    const int row0 = tile.a0, nrows = min(kLrGramSpan, L.rows - row0);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    float* __restrict__ P = p.P + L.p_off + (int64_t)row0 * kLrCols;
    constexpr int kPer = kLrGramSpan * kLrCols / 4 / 256;
    const int filled = nrows * (kLrCols / 4);
    float4 v[kPer];
    if (L.psplits > 1) {
        const float* __restrict__ part = p.ppart + L.ppart_off + (int64_t)row0 * kLrCols;
        const int64_t stride = (int64_t)L.rows * kLrCols;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int f = tid + 256 * q;
            v[q] = f < filled ? *reinterpret_cast<const float4*>(part + 4 * f) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int sp = 1; sp < L.psplits; ++sp) {
            const float* __restrict__ src = part + sp * stride;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int f = tid + 256 * q;
                const float4 w = f < filled ? *reinterpret_cast<const float4*>(src + 4 * f) : make_float4(0.f, 0.f, 0.f, 0.f);
                v[q].x += w.x; v[q].y += w.y; v[q].z += w.z; v[q].w += w.w;
            }
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int f = tid + 256 * q;
            if (f < filled) *reinterpret_cast<float4*>(P + 4 * f) = v[q];
        }
    } else {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int f = tid + 256 * q;
            v[q] = f < filled ? *reinterpret_cast<const float4*>(P + 4 * f) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int f = tid + 256 * q, r = f >> 4, b = (f >> 2) & 3;
        *reinterpret_cast<float4*>(&Ps[r][16 * (b ^ (r & 3)) + 4 * (f & 3)]) = v[q];
    }
    __syncthreads();
    const int lr = lane >> 4, lc = lane & 15;
    double* __restrict__ out = p.gram_part + (size_t)blockIdx.x * kLrCols * kLrCols;
    const int steps = (nrows + 3) / 4;
    // N blocks (ai[n], bi[n]) of the matrix; the lane's row of a step is 4 st + lr, and lr is also its low bits
    auto run = [&](auto pairs) __attribute__((always_inline)) {
        constexpr int N = decltype(pairs)::n;
        f64x4 acc[N];
#pragma unroll
        for (int n = 0; n < N; ++n) acc[n] = f64x4{0.0, 0.0, 0.0, 0.0};
        for (int st = 0; st < steps; ++st) {
            const float* const row = Ps[4 * st + lr];
            double x[4];
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (pairs.uses(b)) x[b] = (double)row[16 * (b ^ lr) + lc];
#pragma unroll
            for (int n = 0; n < N; ++n)
                acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[pairs.a(n)], x[pairs.b(n)], acc[n], 0, 0, 0);
        }
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int u = 0; u < 4; ++u) out[(16 * pairs.a(n) + 4 * u + lr) * kLrCols + 16 * pairs.b(n) + lc] = acc[n][u];
    };
    if (wave == 0) run(GramBlocks<0, 0, 0, 1, 1, 1>{});
    else if (wave == 1) run(GramBlocks<2, 2, 2, 3, 3, 3>{});
    else if (wave == 2) run(GramBlocks<0, 2, 0, 3>{});
    else run(GramBlocks<1, 2, 1, 3>{});
}

// ------------------------------------------------------------------ Gram-Schmidt coefficients
__device__ __forceinline__ double lane_value(double v, int lane) {      // v of a given lane, as a scalar
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// G = sum of a layer's Gram partials, left in the layer's first partial: 64 workgroups per layer of many
// rows, a row of the matrix each, its four wavefronts a quarter of the partials with eight loads in flight
// (added per quarter in partial order, then the quarters in order).  A layer of up to kLrFewPartials partials is
// summed by the kernel that eliminates.
constexpr int kLrFewPartials = 4;
__global__ __launch_bounds__(256) void lr_gram_reduce_kernel(LrParams p) {
    __shared__ double s_q[4][kLrCols];
    const LrLayer L = p.layers[blockIdx.y];
    const int n = L.gram_end - L.gram_begin;
    if (n <= kLrFewPartials) return;
    const int k = blockIdx.x, j = threadIdx.x & 63, w = threadIdx.x >> 6;
    double* const first = p.gram_part + (size_t)L.gram_begin * kLrCols * kLrCols + k * kLrCols + j;
    const int per = (n + 3) / 4, c1 = min(n, (w + 1) * per);
    double s = 0.0;
    if ((k >> 4) <= (j >> 4)) {                          // on and above the diagonal blocks
        int c = w * per;
        for (; c + 8 <= c1; c += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = first[(size_t)(c + u) * kLrCols * kLrCols];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; c < c1; ++c) s += first[(size_t)c * kLrCols * kLrCols];
    }
    s_q[w][j] = s;
    __syncthreads();
    if (w == 0) *first = ((s_q[0][j] + s_q[1][j]) + s_q[2][j]) + s_q[3][j];
}

// One workgroup per layer, the matrix in registers: wavefront w, lane j hold x[m] = element (k = 8 m + w, j).
// Gram-Schmidt on the inner products is the elimination G = U^T D U (U unit upper triangular): step i
// subtracts G[i][k] / d_i times row i from every row k > i.  The same row operations turn the identity into
// U^-T, whose column i starts at step i, just when column i of G is used up: it takes its place.  At
// the end T = U^-1 D^-1/2, so that Phat = P T.  A step is a chain of an LDS round trip (the row is published
// by its owner), a reciprocal and an update, then a barrier; square roots wait for the end, where all 64 are
// taken at once.  (Cholesky with the square root and the division inside the chain, back substitution behind it: 42 us.)
constexpr int kLrOrthThreads = 512;
__global__ __launch_bounds__(kLrOrthThreads) void lr_orth_kernel(LrParams p) {
    __shared__ double X[kLrCols][kLrCols + 1];           // row i as it is when step i uses it
    __shared__ double diag0[kLrCols], scale[kLrCols];
    constexpr int kWaves = kLrOrthThreads / 64, kRows = kLrCols / kWaves;
    const LrLayer L = p.layers[blockIdx.x];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), j = tid & 63;
    double x[kRows];
    {
        const int n = L.gram_end - L.gram_begin;
        const double* __restrict__ src = p.gram_part + (size_t)L.gram_begin * kLrCols * kLrCols + w * kLrCols + j;
        double v[kLrFewPartials][kRows];                 // (all of them in flight together)
#pragma unroll
        for (int c = 0; c < kLrFewPartials; ++c)
#pragma unroll
            for (int m = 0; m < kRows; ++m) {
                v[c][m] = 0.0;
                if ((c == 0 || (c < n && n <= kLrFewPartials)) && ((kWaves * m + w) >> 4) <= (j >> 4))
                    v[c][m] = src[((size_t)c * kLrCols + kWaves * m) * kLrCols];
            }
#pragma unroll
        for (int m = 0; m < kRows; ++m) {
            x[m] = v[0][m];
#pragma unroll
            for (int c = 1; c < kLrFewPartials; ++c) x[m] += v[c][m];
        }
    }
#pragma unroll
    for (int m = 0; m < kRows; ++m)
        if (kWaves * m + w == j) diag0[j] = x[m];          // squared norms before any projection
    if (w == 0) X[0][j] = x[0];
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < kRows; ++mb) {
        for (int wi = 0; wi < kWaves; ++wi) {
            const int i = kWaves * mb + wi;
            const double row = X[i][j], d = X[i][i], d0 = diag0[i];
            const bool ok = d > 0.0 && d >= 1e-10 * d0;
            // 1 / d: the hardware's approximation and two Newton steps
            double inv = __builtin_amdgcn_rcp(d);
            inv = __builtin_fma(__builtin_fma(-d, inv, 1.0), inv, inv);
            inv = __builtin_fma(__builtin_fma(-d, inv, 1.0), inv, inv);
            if (!ok) inv = 0.0;                              // a column in the span of those before it becomes zero
            const bool here = j == i;
            const double rj = (here ? 1.0 : row) * inv;
#pragma unroll
            for (int m = mb; m < kRows; ++m) {
                if (m == mb && w <= wi) continue;            // rows up to i are done (uniform)
                const double f = lane_value(row, kWaves * m + w);
                x[m] = __builtin_fma(-f, rj, here ? 0.0 : x[m]);
                // the next row goes out as soon as it is ready
                if (m <= mb + 1 && kWaves * m + w == i + 1) X[i + 1][j] = x[m];
            }
            __syncthreads();
        }
    }
    if (w == 0) {
        const double d = X[j][j];
        scale[j] = (d > 0.0 && d >= 1e-10 * diag0[j]) ? 1.0 / sqrt(d) : 0.0;
    }
    __syncthreads();
    double* __restrict__ T = p.T + (size_t)blockIdx.x * kLrCols * kLrCols;
    const double sj = scale[j];
#pragma unroll
    for (int m = 0; m < kRows; ++m) {
        const int r = kWaves * m + w;
        T[r * kLrCols + j] = r < j ? X[j][r] * sj : (r == j ? sj : 0.0);
    }
}

// ------------------------------------------------------------------ Phat = P T
// fp64 MFMA on the transposes, Phat^T = T^T P^T: a wavefront takes 32 rows of P, 16 per operand, all of their loads
// issued before anything else (and before any store, so the update is in place), against T in LDS.  The contraction
// index of step (q, u) is 16 q + 4 (lane / 16) + u, so that a lane's four values of a q are one 128-bit load of its row,
// and operand place i of block b is column 16 b + 4 (i % 4) + i / 4, so that its four results are one 128-bit store.
// T is upper triangular: column block b needs only q <= b.  What bounds it is the matrix pipe (40 steps of 64
// cycles per 16 rows, 10 us of it on 106 k rows); every value of T fetched from LDS serves two of them.  106 k rows of
// 66 layers: 21 us (23 with 64 rows a wavefront, two wavefronts on a SIMD, and a 4-byte store per result).
__global__ __launch_bounds__(256, 4) void lr_apply_kernel(LrParams p) {
    __shared__ double Tl[kLrCols][kLrCols + 4];     // padded: rows four apart half the banks apart
    const LrTile tile = p.gram_tiles[blockIdx.x];          // one workgroup per span of kLrGramSpan rows
    const LrLayer L = p.layers[tile.layer];
    float* __restrict__ P = p.P + L.p_off;
    const double* __restrict__ T = p.T + (size_t)tile.layer * kLrCols * kLrCols;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int lr = lane >> 4, lc = lane & 15;
    constexpr int kGroups = kLrGramSpan / 64;                // 16-row groups of a wavefront
    const int row0 = tile.a0 + 16 * kGroups * wave;
    double2 t[kLrCols * kLrCols / 2 / 256];
#pragma unroll
    for (int q = 0; q < kLrCols * kLrCols / 2 / 256; ++q) t[q] = reinterpret_cast<const double2*>(T)[tid + 256 * q];
    float4 a[kGroups][4];                                        // [16-row group][q]
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        const int row = row0 + 16 * g + lc;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            a[g][q] = row < L.rows ? *reinterpret_cast<const float4*>(P + (int64_t)row * kLrCols + 16 * q + 4 * lr)
                                   : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int q = 0; q < kLrCols * kLrCols / 2 / 256; ++q) {
        const int f = tid + 256 * q;
        *reinterpret_cast<double2*>(&Tl[f >> 5][2 * (f & 31)]) = t[q];
    }
    float* pay = p.payload ? reinterpret_cast<float*>(p.payload + L.payload) : nullptr;
    __syncthreads();
    if (row0 >= L.rows) return;                            // (behind the only barrier)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        f64x4 acc[kGroups];
#pragma unroll
        for (int g = 0; g < kGroups; ++g) acc[g] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q <= b; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double tv = Tl[16 * q + 4 * lr + u][16 * b + 4 * (lc & 3) + (lc >> 2)];
#pragma unroll
                for (int g = 0; g < kGroups; ++g) {
                    const float av = u == 0 ? a[g][q].x : u == 1 ? a[g][q].y : u == 2 ? a[g][q].z : a[g][q].w;
                    acc[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(tv, (double)av, acc[g], 0, 0, 0);
                }
            }
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int row = row0 + 16 * g + lc, col = 16 * b + 4 * lr;
            if (row < L.rows) {
                const float4 v = make_float4((float)acc[g][0], (float)acc[g][1], (float)acc[g][2], (float)acc[g][3]);
                *reinterpret_cast<float4*>(P + (int64_t)row * kLrCols + col) = v;
                if (pay) {
                    float* const dst = pay + (int64_t)row * L.rank + col;
                    if (col + 4 <= L.rank) {
                        store4_any(dst, v);
                    } else {
                        if (col < L.rank) dst[0] = v.x;
                        if (col + 1 < L.rank) dst[1] = v.y;
                        if (col + 2 < L.rank) dst[2] = v.z;
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------------ Q partials = X^T Phat
// One workgroup: 128 columns of X (rows of Q) over one range of its rows, 32 rows at a time; wavefront w owns columns
// 32 w .. 32 w + 31, whose rows a lane loads straight in the layout of the instruction (two rows of 128 bytes an
// instruction), a chunk ahead; the rows of Phat, shared by the four, go through LDS as pieces (two buffers, one barrier a chunk).
// Products on the bf16 matrix pipe (see split8 and mfma_split): 67 M elements 83 us in a step (with six products, all added
// to the accumulator, 76); the reads of X are 42 of it at HBM's rate, the products 28, and vector instructions overlap both in part.
// Its error against 64 bits is below that of the fp32 instructions at every length (see mfma_split).  Splits of one
// range are neighbours, so that workgroups that run together read whole rows.
__global__ __launch_bounds__(256, 4) void lr_gemm2_kernel(LrParams p) {
    __shared__ __align__(16) bf16x8 Ps[2][kLrBK / 8][3][kLrCols];       // [8 rows][piece][column]
    const LrTile tile = p.col_tiles[blockIdx.x];
    const LrLayer L = p.layers[tile.layer];
    const int m = L.rows, n = L.cols, col0 = tile.a0;
    const int kbeg = tile.split * L.ksplit, kend = min(m, kbeg + L.ksplit);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int half = lane >> 5, bj = lane & 31;
    // columns past the matrix read its last one; their rows of Q are not written
    const float* __restrict__ X = matrix_of(p, L);
    const int col = min(col0 + 32 * wave + bj, n - 1);
    const uint32_t at_x = 4u * ((uint32_t)(8 * half) * (uint32_t)n + (uint32_t)col);
    const float* __restrict__ P = p.P + L.p_off;

    float xr[16], pr[8];
    auto fetch = [&](int k0) __attribute__((always_inline)) {
        if (k0 + kLrBK <= kend && n < kLrWide) {             // uniform: nearly every chunk
            const float* const x0 = X + (int64_t)k0 * n;
#pragma unroll
            for (int u = 0; u < 16; ++u) xr[u] = *at_bytes(x0 + (int64_t)((u & 7) + 2 * (u & 8)) * n, at_x);
            const float* const p0 = P + (int64_t)(k0 + 8 * wave) * kLrCols;
#pragma unroll
            for (int u = 0; u < 8; ++u) pr[u] = *at_bytes(p0 + u * kLrCols, 4u * (uint32_t)lane);
        } else {                                             // rows past the range count as zero
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int k = k0 + 8 * half + (u & 7) + 2 * (u & 8);
                xr[u] = X[(int64_t)min(k, kend - 1) * n + col];
                if (k >= kend) xr[u] = 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = k0 + 8 * wave + u;
                pr[u] = P[(int64_t)min(k, kend - 1) * kLrCols + lane];
                if (k >= kend) pr[u] = 0.0f;
            }
        }
    };
    Split8 a[2];
    auto take = [&](int buf) __attribute__((always_inline)) {
        a[0] = split8(xr);
        a[1] = split8(xr + 8);
        const Split8 b = split8(pr);
#pragma unroll
        for (int q = 0; q < 3; ++q) Ps[buf][wave][q][lane] = b.piece[q];
    };

    f32x16 acc0 = {0}, acc1 = {0};
    const int nchunks = (kend - kbeg + kLrBK - 1) / kLrBK;
    fetch(kbeg);
    for (int c = 0; c < nchunks; ++c) {
        const int buf = c & 1;
        take(buf);
        if (c + 1 < nchunks) fetch(kbeg + (c + 1) * kLrBK);
        __syncthreads();                                     // (the buffer's last readers were done before the barrier in between)
        acc0 = mfma_split(a, [&](int s, int t) { return Ps[buf][2 * s + half][t][bj]; }, acc0);
        acc1 = mfma_split(a, [&](int s, int t) { return Ps[buf][2 * s + half][t][32 + bj]; }, acc1);
    }
    const float most = largest(acc0, acc1);
    const auto some = [&] {
        return any_value((kend - kbeg + 3) / 4, [&](int i) {                 // 4 rows at a time
                   return bits_of(load4_any(P + (int64_t)min(kbeg + 4 * i + (lane >> 4), kend - 1) * kLrCols + 4 * (lane & 15)));
               }) &&
               any_value((kend - kbeg + 1) / 2, [&](int i) {
                   return __float_as_uint(X[(int64_t)min(kbeg + 2 * i + half, kend - 1) * n + col]);
               });
    };
    if (!__any(most >= kLrHeldQ) && (__any(most > 0.0f) || some()))        // (uniform)
        mfma_plain(kbeg, kend, half, [&](int k) { return X[(int64_t)k * n + col]; },
                   [&](int k, int c) { return P[(int64_t)k * kLrCols + 32 * c + bj]; }, acc0, acc1);
    float* __restrict__ out = p.part + L.part_off + (int64_t)tile.split * n * kLrCols;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int oc = col0 + 32 * wave + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (oc < n) {
            out[(int64_t)oc * kLrCols + bj] = acc0[v];
            out[(int64_t)oc * kLrCols + 32 + bj] = acc1[v];
        }
    }
}

// ------------------------------------------------------------------ Q = sum of partials, norms
__global__ __launch_bounds__(256) void lr_qreduce_kernel(LrParams p) {
    __shared__ double s_n[4][kLrCols];
    __shared__ float s_p[4][kLrCols];
    const LrTile tile = p.q_chunks[blockIdx.x];
    const LrLayer L = p.layers[tile.layer];
    const int n = L.cols, c0 = tile.a0, nc = min(tile.split, n - c0);    // tile.split = rows of this chunk
    const float* __restrict__ part = p.part + L.part_off;
    float* __restrict__ Q = p.Q + L.qs_off;
    const int tid = threadIdx.x, j = tid & 63, grp = tid >> 6;
    float* pay = nullptr;
    if (p.payload) pay = reinterpret_cast<float*>(p.payload + L.payload) + (int64_t)L.rows * L.rank;
    double norm = 0.0;
    auto emit = [&](int r, float s) {
        const int64_t idx = (int64_t)(c0 + r) * kLrCols + j;
        Q[idx] = s;
        norm = __builtin_fma((double)s, (double)s, norm);
        if (p.payload && j < L.rank) {
            pay[(int64_t)(c0 + r) * L.rank + j] = s;
            p.q_out[L.q_off + (int64_t)(c0 + r) * p.r_max + j] = s;
        }
    };
    // sum of partials [sp0, sp1) of one element in partial order, the loads eight deep
    auto sum_partials = [&](int64_t idx, int sp0, int sp1) {
        const int64_t stride = (int64_t)n * kLrCols;
        float s = 0.0f;
        int sp = sp0;
        for (; sp + 8 <= sp1; sp += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(sp + u) * stride + idx];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; sp < sp1; ++sp) s += part[(int64_t)sp * stride + idx];
        return s;
    };
    if (L.splits <= 4) {
        // few partials: one thread per (row, column), rows strided over the 4 wavefronts
        // (four rows per pass: their up to 16 loads are in flight together)
        const int64_t stride = (int64_t)n * kLrCols;
        for (int r = grp; r < nc; r += 16) {
            float v[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int rr = r + 4 * u;
                const int64_t idx = (int64_t)(c0 + rr) * kLrCols + j;
#pragma unroll
                for (int sp = 0; sp < 4; ++sp)
                    v[u][sp] = (rr < nc && sp < L.splits) ? part[(int64_t)sp * stride + idx] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int rr = r + 4 * u;
                if (rr < nc) {
                    float s = 0.0f;
#pragma unroll
                    for (int sp = 0; sp < 4; ++sp)
                        if (sp < L.splits) s += v[u][sp];
                    emit(rr, s);
                }
            }
        }
    } else {
        // many partials: the 4 wavefronts share one row, each sums a contiguous quarter of the
        // partials, and wavefront 0 adds the four sums in order
        const int per = (L.splits + 3) / 4;
        const int sp0 = grp * per, sp1 = min(L.splits, sp0 + per);
        for (int r = 0; r < nc; ++r) {
            const int64_t idx = (int64_t)(c0 + r) * kLrCols + j;
            s_p[grp][j] = sum_partials(idx, sp0, sp1);
            __syncthreads();
            if (grp == 0) emit(r, ((s_p[0][j] + s_p[1][j]) + s_p[2][j]) + s_p[3][j]);
            __syncthreads();
        }
    }
    s_n[grp][j] = norm;
    __syncthreads();
    if (tid < kLrCols)
        p.qnorm_part[(size_t)blockIdx.x * kLrCols + tid] = s_n[0][tid] + s_n[1][tid] + s_n[2][tid] + s_n[3][tid];
}

// ------------------------------------------------------------------ errors of every rank
// One workgroup per layer; the four wavefronts split the partial sums (column norms of Q per
// chunk, ||X||^2 per tile) into contiguous quarters that are added in a fixed order.
__global__ __launch_bounds__(256) void lr_errors_kernel(LrParams p) {
    __shared__ double s_q[4][kLrCols];
    __shared__ double s_x[4];
    const LrLayer L = p.layers[blockIdx.x];
    const int j = threadIdx.x & 63, w = threadIdx.x >> 6;
    {
        const int n = L.qc_end - L.qc_begin, per = (n + 3) / 4;
        const int c0 = L.qc_begin + min(n, w * per), c1 = L.qc_begin + min(n, (w + 1) * per);
        double qn = 0.0;
#pragma unroll 8
        for (int c = c0; c < c1; ++c) qn += p.qnorm_part[(size_t)c * kLrCols + j];
        s_q[w][j] = qn;
    }
    {
        const int n = L.rt_end - L.rt_begin, per = (n + 3) / 4;
        const int t0 = L.rt_begin + min(n, w * per), t1 = L.rt_begin + min(n, (w + 1) * per);
        double xn = 0.0;
        for (int t = t0 + j; t < t1; t += 64) xn += p.xnorm_part[t];
        xn = wave_sum(xn);
        if (j == 0) s_x[w] = xn;
    }
    __syncthreads();
    if (w != 0) return;
    const double qn = ((s_q[0][j] + s_q[1][j]) + s_q[2][j]) + s_q[3][j];
    const double xn = ((s_x[0] + s_x[1]) + s_x[2]) + s_x[3];
    // inclusive prefix over columns, in column order
    double pre = qn;
    for (int o = 1; o < 64; o <<= 1) {
        const double v = __shfl_up(pre, o, 64);
        if (j >= o) pre += v;
    }
    for (int c = 0; c < p.nrank; ++c)
        if (j == p.rank[c] - 1) p.errors[(size_t)L.index * p.stride + p.col[c]] = fmax(xn - pre, 0.0);
}

// Payload and warm-start update of a layer from the profile's scratch (KNOWN, see lr_ef_kernel): the first `rank`
// columns of Phat (row tiles, block < n_row_tiles) and of Q (its chunks after them); Q also replaces the first `rank`
// columns of the layer's warm start.  Nothing waits for them: workgroups of the reconstruction's launch make them (in
// front of it, as a launch of their own, they took 14 us of a step of 67 M elements).
__device__ __forceinline__ void emit_known(const LrParams& p, int block) {
    const bool is_p = block < p.n_row_tiles;
    const LrTile tile = is_p ? p.row_tiles[block] : p.q_chunks[block - p.n_row_tiles];
    const LrLayer L = p.layers[tile.layer];
    const DevLayer& dl = p.dev_layers[L.index];
    if (dl.family != LGRECO_LOWRANK || dl.iparam < 1 || dl.iparam > kLrCols) return;
    const int r = dl.iparam;
    float* const pay = reinterpret_cast<float*>(p.payload + dl.payload);
    const int tid = threadIdx.x;
    if (is_p) {
        const float* __restrict__ P = p.P + L.p_off;
        const int nr = min(kLrBM, L.rows - tile.a0);
        for (int f = tid; f < nr * r; f += 256) {
            const int rr = f / r, c = f - rr * r;
            pay[(int64_t)(tile.a0 + rr) * r + c] = P[(int64_t)(tile.a0 + rr) * kLrCols + c];
        }
    } else {
        const float* __restrict__ Q = p.Q + L.qs_off;
        float* const payq = pay + (int64_t)L.rows * r;
        const int nr = min(tile.split, L.cols - tile.a0);      // tile.split = rows of this chunk
        for (int f = tid; f < nr * r; f += 256) {
            const int rr = f / r, c = f - rr * r;
            const float v = Q[(int64_t)(tile.a0 + rr) * kLrCols + c];
            payq[(int64_t)(tile.a0 + rr) * r + c] = v;
            p.q_out[L.q_off + (int64_t)(tile.a0 + rr) * p.r_max + c] = v;
        }
    }
}

// ------------------------------------------------------------------ e' = X - Phat Q^T
// DECODE (receiver side): the factors come from the payload (row stride = rank) and the product
// is written, or added, to the output buffer instead of being subtracted from x.
// KNOWN (compression right behind a profile of the same data): the factors are the leading columns
// of the profile's rank-64 run, still in its scratch; whether the layer takes part and its rank
// come from the layer records the solver kernel wrote.
//
// Bound by HBM: x once in, e' once out.  A wavefront makes one tile of 32 x 32 and is over, a workgroup four of them
// side by side, 512 bytes of 32 rows: short wavefronts in the order of the addresses keep the chip in a narrow window of
// memory (a bare read and write of 67 M elements in this shape 84 us; 100 with workgroups that walk 512 columns of
// 128 rows, 32 at a time, as here before; 105 with 128 rows of 32 columns).  The factors come from the caches straight in the layout of the
// instruction; 16 consecutive workgroups run on one XCD and share their rows of them in its L2.  x is loaded and e' stored in the accumulator's
// layout (two rows of 128 bytes an instruction), past the caches where those are whole lines: e' left in them as it is written out
// costs the next call's first pass 30 us.  Four wavefronts on a SIMD or more (at three as many bytes are in flight as the latency covers, at six registers spill).
// 67 M elements of 97 layers: compression 125 -> 98 us, behind a profile 120 -> 113, receiver 124 -> 103 a call (adding; 79 -> 62
// replacing); 73 M elements of odd widths: a step 818 -> 700 with lr_gemm2_kernel's part (47), receiver 178 -> 133.
constexpr int kLrEfRows = 32, kLrEfCols = 128;
enum { kLrEfEdge, kLrEfPieces, kLrEfLines };
template <bool DECODE, bool KNOWN = false>
__global__ __launch_bounds__(256, 4) void lr_ef_kernel(LrParams p) {
    if (KNOWN && (int)blockIdx.x >= p.n_ef_tiles) {
        emit_known(p, (int)blockIdx.x - p.n_ef_tiles);
        return;
    }
    // (workgroups are dealt to the eight XCDs in turn)
    int which = (int)blockIdx.x;
    if (which < p.n_ef_tiles / 128 * 128) which = which / 128 * 128 + which % 8 * 16 + which % 128 / 8;
    const LrTile tile = p.ef_tiles[which];
    const LrLayer L = p.layers[tile.layer];
    int r = L.rank;
    if (KNOWN) {
        const DevLayer& dl = p.dev_layers[L.index];
        if (dl.family != LGRECO_LOWRANK || dl.iparam < 1 || dl.iparam > kLrCols) return;
        r = dl.iparam;
    }
    const int m = L.rows, n = L.cols;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, bj = lane & 31;
    const int row0 = tile.a0, c0 = tile.split + 32 * wave;
    if (c0 >= n) return;
    // (the buffer written may be the one read: every element is read, then written, by the same lane)
    const float* const g = DECODE ? (p.accumulate ? p.e_out + L.offset : nullptr) : matrix_of(p, L);
    float* const e = p.e_out + L.offset;
    const float* __restrict__ P =
        DECODE ? reinterpret_cast<const float*>(p.payload + L.payload) : p.P + L.p_off;
    const float* __restrict__ Q = DECODE ? P + (int64_t)m * r : p.Q + L.qs_off;
    const int stride = DECODE ? r : kLrCols;

    // Operands: step (i, u) contracts the columns 8 i + u and 8 i + 4 + u of the factors, so that a lane's values of an
    // i are one 128-bit load (in a payload moved back to the row's end), zero from the rank on.
    const float* const pa = P + (int64_t)row0 * stride;
    const float* const pb = Q + (int64_t)c0 * stride;
    const int at_a = min(bj, m - 1 - row0) * stride, at_b = min(bj, n - 1 - c0) * stride;
    f32x16 acc = {0};
    const auto fetch = [&](auto& a, auto& b, int first) __attribute__((always_inline)) {
        constexpr int N = sizeof(a) / sizeof(a[0]);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = 8 * (first + i) + 4 * half;
            if (DECODE && r < 4) {                           // (uniform) rows shorter than a load
                const float* const ra = pa + at_a;
                const float* const rb = pb + at_b;
                a[i] = make_float4(ra[0], r > 1 ? ra[1] : 0.f, r > 2 ? ra[2] : 0.f, 0.f);
                b[i] = make_float4(rb[0], r > 1 ? rb[1] : 0.f, r > 2 ? rb[2] : 0.f, 0.f);
                continue;
            }
            const int from = DECODE ? min(k, r - 4) : k;     // (not negative)
            a[i] = load4_any(at_bytes(pa, 4u * (uint32_t)(at_a + from)));
            b[i] = load4_any(at_bytes(pb, 4u * (uint32_t)(at_b + from)));
        }
    };
    const auto mask = [&](auto& a, auto& b, int first) __attribute__((always_inline)) {
        constexpr int N = sizeof(a) / sizeof(a[0]);
        if (8 * (first + N) <= r) return;                    // (uniform)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = 8 * (first + i) + 4 * half, shift = DECODE && r >= 4 ? max(k - (r - 4), 0) : 0;
            const auto behind = [&](float4 v) {
                if (DECODE)
                    v = shift == 0 ? v : shift == 1 ? make_float4(v.y, v.z, v.w, 0.f) : shift == 2 ? make_float4(v.z, v.w, 0.f, 0.f)
                                                  : make_float4(v.w, 0.f, 0.f, 0.f);
                return make_float4(k < r ? v.x : 0.f, k + 1 < r ? v.y : 0.f, k + 2 < r ? v.z : 0.f, k + 3 < r ? v.w : 0.f);
            };
            a[i] = behind(a[i]);
            b[i] = behind(b[i]);
        }
    };
    const auto multiply = [&](const auto& a, const auto& b) __attribute__((always_inline)) {
        constexpr int N = sizeof(a) / sizeof(a[0]);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].x, b[i].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].y, b[i].y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].z, b[i].z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i].w, b[i].w, acc, 0, 0, 0);
        }
    };
    // element v of the accumulator: row 8 (v / 4) + 4 half + v % 4 of the tile, column bj
    const auto row_of = [](int v) { return 8 * (v >> 2) + (v & 3); };
    const auto finish = [&](auto groups, auto where, int first) __attribute__((always_inline)) {
        constexpr bool full = decltype(where)::value != kLrEfEdge, lines = decltype(where)::value == kLrEfLines;
        float4 a[decltype(groups)::value], b[decltype(groups)::value];
        fetch(a, b, first);
        asm volatile("" ::: "memory");                       // (the order of the loads)
        // scalar row starts and one 32-bit offset per lane; at an edge the last row and column in place of what lies past
        // them
        const uint32_t at_v = 16u * (uint32_t)half * (uint32_t)n + 4u * (uint32_t)bj;
        const auto at = [&](auto* base, int v) __attribute__((always_inline)) {
            if constexpr (full) return at_bytes(base + (int64_t)(row0 + row_of(v)) * n + c0, at_v);
            else return base + (int64_t)min(row0 + row_of(v) + 4 * half, m - 1) * n + min(c0 + bj, n - 1);
        };
        float x[16];
        if (DECODE && g == nullptr) {
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = 0.0f;
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (lines) x[v] = __builtin_nontemporal_load(at(g, v));
                else x[v] = *at(g, v);
            }
        }
        asm volatile("" ::: "memory");
        mask(a, b, first);
        multiply(a, b);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            // zeros that are not read are still added (a gradient of -0 becomes the +0 the sum with
            // a stored zero gives: every bit as without the promise)
            const float xv = !DECODE && p.e_is_zero ? x[v] + 0.0f : x[v];
            const float o = DECODE ? xv + acc[v] : xv - acc[v];
            if constexpr (lines) __builtin_nontemporal_store(o, at(e, v));
            else if (full || (row0 + row_of(v) + 4 * half < m && c0 + bj < n)) *at(e, v) = o;
        }
    };
    const auto run = [&](auto where) __attribute__((always_inline)) {
        if (r > 32) {
            {
                float4 a[4], b[4];
                fetch(a, b, 0);
                multiply(a, b);
            }
            finish(std::integral_constant<int, 4>(), where, 4);
        } else if (r > 16) {
            finish(std::integral_constant<int, 4>(), where, 0);
        } else if (r > 8) {
            finish(std::integral_constant<int, 2>(), where, 0);
        } else {
            finish(std::integral_constant<int, 1>(), where, 0);
        }
    };
    // Whole lines pass by the caches; pieces of lines don't, since their other half is the next wavefront's.
    if (row0 + 32 > m || c0 + 32 > n || n >= kLrWide) run(std::integral_constant<int, kLrEfEdge>());
    else if (L.lines) run(std::integral_constant<int, kLrEfLines>());
    else run(std::integral_constant<int, kLrEfPieces>());
}

// ------------------------------------------------------------------------ host side
#define LR_CHECK(expr)                     \
    do {                                   \
        hipError_t _e = (expr);            \
        if (_e != hipSuccess) return _e;   \
    } while (0)

// Work tables and scratch are kept per kind of call (profile, compress, decompress): the three
// alternate in a training loop and each repeats its own layer table, so nothing is rebuilt.
constexpr int kLrSlots = 3;
enum { kLrSlotProfile = 0, kLrSlotCompress = 1, kLrSlotDecode = 2 };

struct LrHost {
    std::vector<LrLayer> layers;
    std::vector<LrTile> row_tiles, p_tiles, ef_tiles, col_tiles, gram_tiles, q_chunks;
    std::vector<int64_t> sig;       // signature of the layer table the tables were built for
    bool many_partials = false;     // some layer has more Gram partials than the elimination sums itself
    // device copies
    LrLayer* d_layers = nullptr;
    LrTile* d_tiles = nullptr;      // the four tile tables back to back
    size_t cap_layers = 0, cap_tiles = 0, cap_p = 0, cap_q = 0, cap_part = 0, cap_ppart = 0, cap_T = 0,
           cap_xn = 0, cap_qn = 0;
    float* P = nullptr;
    float* Q = nullptr;
    float* part = nullptr;          // partials of Q, and before them of the Gram matrices: those are used up when Q is computed
    float* ppart = nullptr;
    double* T = nullptr;
    double* xn = nullptr;
    double* qn = nullptr;
};

static hipError_t grow(void** ptr, size_t* cap, size_t need) {
    if (need <= *cap) return hipSuccess;
    if (*ptr) LR_CHECK(hipFree(*ptr));
    *ptr = nullptr;
    *cap = 0;
    LR_CHECK(hipMalloc(ptr, need));
    *cap = need;
    return hipSuccess;
}

hipError_t lowrank_scratch_create(LowrankScratch* t, int64_t max_elems, int max_layers, int r_max,
                                  int power_iters) {
    t->power_iters = power_iters;
    t->max_elems = max_elems;
    t->max_layers = max_layers;
    t->r_max = r_max;
    t->host = new LrHost[kLrSlots]();
    return hipSuccess;
}

void lowrank_scratch_destroy(LowrankScratch* t) {
    LrHost* all = (LrHost*)t->host;
    if (all) {
        for (int i = 0; i < kLrSlots; ++i) {
            LrHost* H = &all[i];
            (void)hipFree(H->d_layers);
            (void)hipFree(H->d_tiles);
            (void)hipFree(H->P);
            (void)hipFree(H->Q);
            (void)hipFree(H->part);
            (void)hipFree(H->ppart);
            (void)hipFree(H->T);
            (void)hipFree(H->xn);
            (void)hipFree(H->qn);
        }
        delete[] all;
    }
    *t = LowrankScratch{};
}

// Build the work tables for the layers with rank[l] > 0 and upload them.  Scratch buffers grow on
// demand (allocation happens only when a larger layer table arrives).
static hipError_t lr_prepare(LowrankScratch* t, int slot, const DevLayer* hl, int L, const int* rank, int r_max,
                             bool tables_only, hipStream_t s) {
    LrHost* H = &((LrHost*)t->host)[slot];
    std::vector<int64_t> sig;
    sig.reserve((size_t)L * 5 + 1);
    sig.push_back(r_max);
    for (int l = 0; l < L; ++l) {
        sig.push_back(hl[l].offset);
        sig.push_back(hl[l].rows);
        sig.push_back(hl[l].cols);
        sig.push_back(rank[l]);
        sig.push_back(hl[l].payload);
    }
    if (sig == H->sig) return hipSuccess;
    H->layers.clear();
    H->row_tiles.clear();
    H->p_tiles.clear();
    H->ef_tiles.clear();
    H->col_tiles.clear();
    H->gram_tiles.clear();
    H->q_chunks.clear();
    H->many_partials = false;
    // x: in the place of the error feedback when compressing; packed after a profile
    std::vector<int64_t> x_off((size_t)L, 0);
    pack_matrices(L, [&](int l) { return hl[l].offset; }, [&](int l) { return hl[l].cols; },
                  [&](int l) { return rank[l] > 0 ? (int64_t)hl[l].rows * hl[l].cols : 0; },
                  [&](int l, int64_t at) { x_off[l] = at; });
    int64_t p_off = 0, q_off = 0, part_off = 0, ppart_off = 0;
    for (int l = 0; l < L; ++l) {
        if (rank[l] <= 0) continue;
        LrLayer a{};
        a.offset = hl[l].offset;
        a.x_off = slot == kLrSlotProfile ? x_off[l] : a.offset;
        a.q_off = hl[l].q_offset;
        a.rows = hl[l].rows;
        a.cols = hl[l].cols;
        a.rank = rank[l];
        a.payload = hl[l].payload;
        a.index = l;
        a.p_off = p_off;
        a.qs_off = q_off;
        a.part_off = part_off;
        // split the contraction over rows so that every column tile gets enough workgroups
        const int col_tiles = (a.cols + kLrBM - 1) / kLrBM;
        int splits = 1;
        while (splits < 64 && (int64_t)a.rows / (splits * 2) >= 512 && col_tiles * splits < 256) splits *= 2;
        a.ksplit = ((a.rows + splits - 1) / splits + kLrBK - 1) / kLrBK * kLrBK;
        a.splits = (a.rows + a.ksplit - 1) / a.ksplit;
        const int li = (int)H->layers.size();
        // P = X Q0: equal work units of at most kLrPSplit contracted columns
        a.psplits = (a.cols + kLrPSplit - 1) / kLrPSplit;
        a.pksplit = ((a.cols + a.psplits - 1) / a.psplits + kLrBK - 1) / kLrBK * kLrBK;
        a.psplits = (a.cols + a.pksplit - 1) / a.pksplit;
        a.ppart_off = ppart_off;
        if (a.psplits > 1) ppart_off += (int64_t)a.psplits * a.rows * kLrCols;
        a.rt_begin = (int)H->p_tiles.size();            // ||X||^2 partials: one per P tile
        for (int r0 = 0; r0 < a.rows; r0 += kLrBM) {
            H->row_tiles.push_back(LrTile{li, r0, 0, 0});
            for (int sp = 0; sp < a.psplits; ++sp) H->p_tiles.push_back(LrTile{li, r0, sp, 0});
        }
        a.rt_end = (int)H->p_tiles.size();
        a.lines = whole_lines(a.offset, a.cols) ? 1 : 0;         // (and x_off as well, see pack_matrices)
        for (int r0 = 0; r0 < a.rows; r0 += kLrEfRows)
            for (int c0 = 0; c0 < a.cols; c0 += kLrEfCols) H->ef_tiles.push_back(LrTile{li, r0, c0, 0});
        for (int sp = 0; sp < a.splits; ++sp)
            for (int c0 = 0; c0 < a.cols; c0 += kLrBM) H->col_tiles.push_back(LrTile{li, c0, sp, 0});
        a.gram_begin = (int)H->gram_tiles.size();
        for (int r0 = 0; r0 < a.rows; r0 += kLrGramSpan) H->gram_tiles.push_back(LrTile{li, r0, 0, 0});
        a.gram_end = (int)H->gram_tiles.size();
        H->many_partials = H->many_partials || a.gram_end - a.gram_begin > kLrFewPartials;
        a.qc_begin = (int)H->q_chunks.size();
        {
            // rows per chunk: fewer when many split-K partials have to be summed per row
            const int qrows = a.splits <= 4 ? kLrQChunk : std::max(2, kLrQChunk / a.splits * 2);
            for (int c0 = 0; c0 < a.cols; c0 += qrows) H->q_chunks.push_back(LrTile{li, c0, qrows, 0});
        }
        a.qc_end = (int)H->q_chunks.size();
        p_off += (int64_t)a.rows * kLrCols;
        q_off += (int64_t)a.cols * kLrCols;
        part_off += (int64_t)a.splits * a.cols * kLrCols;
        H->layers.push_back(a);
    }
    const size_t nl = H->layers.size();
    const size_t nt = H->row_tiles.size() + H->p_tiles.size() + H->ef_tiles.size() + H->col_tiles.size() +
                      H->gram_tiles.size() + H->q_chunks.size();
    LR_CHECK(grow((void**)&H->d_layers, &H->cap_layers, sizeof(LrLayer) * std::max<size_t>(nl, 1)));
    LR_CHECK(grow((void**)&H->d_tiles, &H->cap_tiles, sizeof(LrTile) * std::max<size_t>(nt, 1)));
    if (tables_only) { p_off = q_off = part_off = ppart_off = 0; }
    LR_CHECK(grow((void**)&H->P, &H->cap_p, sizeof(float) * std::max<int64_t>(p_off, 1)));
    LR_CHECK(grow((void**)&H->Q, &H->cap_q, sizeof(float) * std::max<int64_t>(q_off, 1)));
    const size_t gram = tables_only ? 0 : sizeof(double) * kLrCols * kLrCols * H->gram_tiles.size();
    LR_CHECK(grow((void**)&H->part, &H->cap_part, std::max(sizeof(float) * std::max<int64_t>(part_off, 1), gram)));
    LR_CHECK(grow((void**)&H->ppart, &H->cap_ppart, sizeof(float) * std::max<int64_t>(ppart_off, 1)));
    LR_CHECK(grow((void**)&H->T, &H->cap_T,
                  sizeof(double) * kLrCols * kLrCols * (tables_only ? 1 : std::max<size_t>(nl, 1))));
    LR_CHECK(grow((void**)&H->xn, &H->cap_xn, sizeof(double) * std::max<size_t>(H->p_tiles.size(), 1)));
    LR_CHECK(grow((void**)&H->qn, &H->cap_qn, sizeof(double) * kLrCols * std::max<size_t>(H->q_chunks.size(), 1)));
    if (nl) {
        LR_CHECK(hipMemcpyAsync(H->d_layers, H->layers.data(), sizeof(LrLayer) * nl, hipMemcpyHostToDevice, s));
        size_t o = 0;
        for (auto* v : {&H->row_tiles, &H->p_tiles, &H->ef_tiles, &H->col_tiles, &H->gram_tiles, &H->q_chunks}) {
            if (!v->empty())
                LR_CHECK(hipMemcpyAsync(H->d_tiles + o, v->data(), sizeof(LrTile) * v->size(),
                                        hipMemcpyHostToDevice, s));
            o += v->size();
        }
        LR_CHECK(hipStreamSynchronize(s));
    }
    H->sig = std::move(sig);
    return hipSuccess;
}

static void lr_fill_params(LrHost* H, LrParams* p) {
    p->layers = H->d_layers;
    p->row_tiles = H->d_tiles;
    p->p_tiles = p->row_tiles + H->row_tiles.size();
    p->ef_tiles = p->p_tiles + H->p_tiles.size();
    p->col_tiles = p->ef_tiles + H->ef_tiles.size();
    p->gram_tiles = p->col_tiles + H->col_tiles.size();
    p->q_chunks = p->gram_tiles + H->gram_tiles.size();
    p->P = H->P;
    p->Q = H->Q;
    p->part = H->part;
    p->ppart = H->ppart;
    p->gram_part = reinterpret_cast<double*>(H->part);
    p->T = H->T;
    p->xnorm_part = H->xn;
    p->qnorm_part = H->qn;
    p->n_ef_tiles = (int)H->ef_tiles.size();
}

// `iters` power-iteration steps: P = X Q, Phat = orth(P), Q = X^T Phat, Q feeding the next step.
static hipError_t lr_factorize(LrHost* H, LrParams p, int iters, Timing* tm, hipStream_t s) {
  for (int it = 0; it < iters; ++it) {
    p.q_from_scratch = it > 0 ? 1 : 0;
    const bool x_out = p.e != nullptr;
    {
        Section sec(tm, "lowrank_gemm_p", true);
        const dim3 grid((unsigned)H->p_tiles.size()), block(256);
        if (x_out) launch_timed(&sec, true, true, lr_gemm1_kernel<true>, grid, block, 0, s, p);
        else launch_timed(&sec, true, true, lr_gemm1_kernel<false>, grid, block, 0, s, p);
        LR_CHECK(hipGetLastError());
    }
    if (x_out) {                                  // from here on x is read in one piece
        p.e = nullptr;
        p.from_x = 1;
    }
    {
        Section sec(tm, "lowrank_orth");
        hipLaunchKernelGGL(lr_gram_kernel, dim3((unsigned)H->gram_tiles.size()), dim3(256), 0, s, p);
        LR_CHECK(hipGetLastError());
        if (H->many_partials) {
            hipLaunchKernelGGL(lr_gram_reduce_kernel, dim3(kLrCols, (unsigned)H->layers.size()), dim3(256), 0, s, p);
            LR_CHECK(hipGetLastError());
        }
        hipLaunchKernelGGL(lr_orth_kernel, dim3((unsigned)H->layers.size()), dim3(kLrOrthThreads), 0, s, p);
        LR_CHECK(hipGetLastError());
        hipLaunchKernelGGL(lr_apply_kernel, dim3((unsigned)H->gram_tiles.size()), dim3(256), 0, s, p);
        LR_CHECK(hipGetLastError());
    }
    {
        Section sec(tm, "lowrank_gemm_q", true);
        launch_timed(&sec, true, true, lr_gemm2_kernel, dim3((unsigned)H->col_tiles.size()), dim3(256), 0, s, p);
        LR_CHECK(hipGetLastError());
    }
    {
        Section sec(tm, "lowrank_q_reduce");
        hipLaunchKernelGGL(lr_qreduce_kernel, dim3((unsigned)H->q_chunks.size()), dim3(256), 0, s, p);
        LR_CHECK(hipGetLastError());
    }
  }
    return hipSuccess;
}

hipError_t lowrank_profile(LowrankScratch* t, const float* g, const float* e, const DevLayer* d_layers,
                           const DevLayer* h_layers, int L, const float* q0, int r_max, const int* rank,
                           const int* col, int nlr, double* d_errors, int stride, float* x, Timing* tm,
                           hipStream_t s) {
    (void)d_layers;
    LrHost* H = &((LrHost*)t->host)[kLrSlotProfile];
    std::vector<int> ranks(L, kLrCols);
    std::vector<DevLayer> hl(h_layers, h_layers + L);
    for (auto& d : hl) d.payload = 0;                 // not part of the profile's signature
    LR_CHECK(lr_prepare(t, kLrSlotProfile, hl.data(), L, ranks.data(), r_max, false, s));
    if (H->layers.empty()) return hipSuccess;
    LrParams p{};
    lr_fill_params(H, &p);
    p.g = g;
    p.e = e;
    p.q0 = q0;
    p.r_max = r_max;
    p.errors = d_errors;
    p.stride = stride;
    p.nrank = nlr;
    for (int c = 0; c < nlr; ++c) { p.rank[c] = rank[c]; p.col[c] = col[c]; }
    p.x = e ? x : nullptr;
    LR_CHECK(lr_factorize(H, p, t->power_iters, tm, s));
    Section sec(tm, "lowrank_errors");
    hipLaunchKernelGGL(lr_errors_kernel, dim3((unsigned)H->layers.size()), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t lowrank_compress(LowrankScratch* t, const float* g, float* e, const DevLayer* d_layers,
                            const DevLayer* h_layers, int L, float* q, int r_max, uint8_t* payload, Timing* tm,
                            hipStream_t s) {
    (void)d_layers;
    LrHost* H = &((LrHost*)t->host)[kLrSlotCompress];
    std::vector<int> ranks(L, 0);
    for (int l = 0; l < L; ++l)
        if (h_layers[l].family == LGRECO_LOWRANK) ranks[l] = h_layers[l].iparam;
    LR_CHECK(lr_prepare(t, kLrSlotCompress, h_layers, L, ranks.data(), r_max, false, s));
    if (H->layers.empty()) return hipSuccess;
    LrParams p{};
    lr_fill_params(H, &p);
    p.g = g;
    p.e = e;
    p.e_out = e;
    p.x = e;                          // the error feedback becomes x, then what is left of it
    p.q0 = q;
    p.q_out = q;
    p.r_max = r_max;
    p.payload = payload;
    LR_CHECK(lr_factorize(H, p, t->power_iters, tm, s));
    p.e = nullptr;
    p.from_x = 1;
    Section sec(tm, "lowrank_ef", true);
    launch_timed(&sec, true, true, lr_ef_kernel<false>, dim3((unsigned)H->ef_tiles.size()), dim3(256), 0, s, p);
    return hipGetLastError();
}

// Low-rank layers of a compression queued right behind a profile of the same data and the solver
// kernel that wrote the layer records: the profile's rank-64 factors are still in its scratch and
// every rank's factors are their leading columns, so nothing is contracted again.  Uses the
// profile's work tables (all layers); needs nothing from the host.
hipError_t lowrank_compress_known(LowrankScratch* t, const float* g, float* e, const DevLayer* d_layers, float* q,
                                  int r_max, uint8_t* payload, const float* x, Timing* tm, hipStream_t s,
                                  bool e_is_zero) {
    LrHost* H = &((LrHost*)t->host)[kLrSlotProfile];
    if (H->layers.empty()) return hipSuccess;
    LrParams p{};
    lr_fill_params(H, &p);
    p.g = g;
    p.x = const_cast<float*>(x);
    p.from_x = e_is_zero ? 0 : 1;        // promised zeros: x is g, and the zeros are not fetched
    p.e_is_zero = e_is_zero ? 1 : 0;
    p.e_out = e;
    p.q0 = q;
    p.q_out = q;
    p.r_max = r_max;
    p.payload = payload;
    p.dev_layers = d_layers;
    p.n_row_tiles = (int)H->row_tiles.size();
    Section sec(tm, "lowrank_ef", true);
    launch_timed(&sec, true, true, lr_ef_kernel<false, true>,
                 dim3((unsigned)(H->ef_tiles.size() + H->row_tiles.size() + H->q_chunks.size())), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t lowrank_decompress(LowrankScratch* t, const DevLayer* h_layers, int L, int r_max, const uint8_t* payload,
                              float* out, bool accumulate, Timing* tm, hipStream_t s) {
    LrHost* H = &((LrHost*)t->host)[kLrSlotDecode];
    std::vector<int> ranks(L, 0);
    for (int l = 0; l < L; ++l)
        if (h_layers[l].family == LGRECO_LOWRANK) ranks[l] = h_layers[l].iparam;
    LR_CHECK(lr_prepare(t, kLrSlotDecode, h_layers, L, ranks.data(), r_max, true, s));
    if (H->layers.empty()) return hipSuccess;
    LrParams p{};
    lr_fill_params(H, &p);
    p.e_out = out;
    p.payload = const_cast<uint8_t*>(payload);
    p.accumulate = accumulate ? 1 : 0;
    p.r_max = r_max;
    Section sec(tm, "lowrank_decode", true);
    launch_timed(&sec, true, true, lr_ef_kernel<true>, dim3((unsigned)H->ef_tiles.size()), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace lgreco
