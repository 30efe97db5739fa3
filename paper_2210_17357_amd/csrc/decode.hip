// Receiver side of the codec for bucketed quantization and Top-K: payload -> dense fp32 image,
// written or added to an output buffer (the step after compression in the paper's pipeline, where
// a worker sums the gradients it received).  gfx950 / wave64.
//
// Quantization payload of a layer: (min, unit) fp32 pairs of all buckets, then every bucket's codes
// as an LSB-first bit stream padded to a byte.  A full bucket of 128 codes takes 16 b bytes, and a
// group of 4 consecutive codes lies in two words:
//   xhat = fma(code, unit, min)        (the same single rounding as the sender)
// Top-K payload: values[k] then indices[k]; the image is zero except at the indices.
#include <algorithm>

#include "internal.h"

namespace lgreco {

struct DecodeParams {
    const uint8_t* payload;
    const DevLayer* layers;
    const Tile* tiles;
    float* out;
    int32_t accumulate;
    int32_t part_shift;        // a tile's workgroups, as a power of two
    int32_t part_elems;        // elements of a workgroup
};

// Bound by HBM, a stream of code words, one of the output's old values and one of its new ones.  A thread takes
// 4 consecutive elements, so that a wavefront's accesses of the output are whole lines, and their 4 * bits
// code bits from the one or two aligned words that hold them (a bucket starts on a word: 16 * bits bytes behind
// payloads aligned to 16 and 8 bytes a bucket).  A workgroup is over after kDecodePart elements, two
// rounds: short workgroups keep the chip's accesses in a narrow window of memory (see quant_compress_kernel).  Ragged ends
// take an element per thread.  Adding 355 M elements of 4 bits to the output: 480 us, 6.3 TB/s (one round
// 487, four 528, two with both rounds' loads ahead 492; 578 with tiles of 32768 and four rounds ahead).
constexpr int kDecodePart = 2048;

template <bool ACCUMULATE>
__global__ __launch_bounds__(kThreads) void quant_decode_kernel(DecodeParams p) {
    const Tile t = p.tiles[blockIdx.x >> p.part_shift];
    const int part = (int)(blockIdx.x & ((1u << p.part_shift) - 1u));
    const DevLayer L = p.layers[t.layer];
    if (L.family != LGRECO_QUANT) return;
    const int bits = L.iparam;
    const int64_t nb_layer = (L.numel + kBucket - 1) / kBucket, bucket0 = t.pos / kBucket;   // (tiles start on a bucket)
    const uint8_t* const lp = p.payload + L.payload;
    const float2* const meta = reinterpret_cast<const float2*>(lp) + bucket0;
    const uint8_t* const codes = lp + 8 * nb_layer + bucket0 * (kBucket / 8) * bits;
    float* const out = p.out + L.offset + t.pos;
    const int tid = threadIdx.x;

    if (t.fast) {                                        // full buckets only
        const uint32_t* const words = reinterpret_cast<const uint32_t*>(codes);
        const int nq = min(t.count, (part + 1) * p.part_elems) / 4;
        const auto decode = [&](int q, uint32_t w0, uint32_t w1, float2 mu, float4 old) {
            const uint32_t v = __builtin_amdgcn_alignbit(w1, w0, (uint32_t)(4 * bits * q) & 31u);
            float4 x;
            x.x = __builtin_fmaf((float)__builtin_amdgcn_ubfe(v, 0, bits), mu.y, mu.x);
            x.y = __builtin_fmaf((float)__builtin_amdgcn_ubfe(v, bits, bits), mu.y, mu.x);
            x.z = __builtin_fmaf((float)__builtin_amdgcn_ubfe(v, 2 * bits, bits), mu.y, mu.x);
            x.w = __builtin_fmaf((float)__builtin_amdgcn_ubfe(v, 3 * bits, bits), mu.y, mu.x);
            if (ACCUMULATE) { x.x += old.x; x.y += old.y; x.z += old.z; x.w += old.w; }
            store_stream(out + 4 * q, x);
        };
        // the word that holds the first and the word that holds the last of a thread's bits
        const auto word0 = [&](int q) { return words[(uint32_t)(4 * bits * q) >> 5]; };
        const auto word1 = [&](int q) { return words[(uint32_t)(4 * bits * (q + 1) - 1) >> 5]; };
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int q = part * p.part_elems / 4 + tid; q < nq; q += kThreads)
            decode(q, word0(q), word1(q), meta[q / (kBucket / 4)], ACCUMULATE ? load_stream(out + 4 * q) : zero);
        return;
    }
    if (part) return;                                    // (less than a chunk)
    // a code lies in one byte or two; a short bucket's stream ends with the byte of its last code
    const auto low = [&](int i) { return (uint32_t)codes[(uint32_t)(bits * i) >> 3]; };
    const auto high = [&](int i) { return (uint32_t)codes[(uint32_t)(bits * i + bits - 1) >> 3]; };
    const auto decode = [&](int i, uint32_t lo, uint32_t hi, float2 mu, float old) {
        const uint32_t code = __builtin_amdgcn_ubfe(lo | hi << 8, (uint32_t)(bits * i) & 7u, bits);
        const float x = __builtin_fmaf((float)code, mu.y, mu.x);
        out[i] = ACCUMULATE ? old + x : x;
    };
    for (int i = tid; i < t.count; i += kThreads) decode(i, low(i), high(i), meta[i / kBucket], ACCUMULATE ? out[i] : 0.0f);
}

// Top-K, first kernel (only when the image replaces the output): zero the layer.
__global__ __launch_bounds__(kThreads) void topk_decode_zero_kernel(DecodeParams p) {
    const Tile t = p.tiles[blockIdx.x];
    const DevLayer L = p.layers[t.layer];
    if (L.family != LGRECO_TOPK) return;
    float* const out = p.out + L.offset + t.pos;
    if (t.fast) {
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int v = threadIdx.x; v < t.count / 4; v += kThreads) store_stream(out + 4 * v, z);
    } else {
        for (int i = threadIdx.x; i < t.count; i += kThreads) out[i] = 0.0f;
    }
}

// Top-K, second kernel: scatter.  The k entries of a layer are dealt to its tiles in proportion
// to the tiles' element ranges; indices are distinct, so plain read-modify-writes do not collide.
__global__ __launch_bounds__(kThreads) void topk_decode_scatter_kernel(DecodeParams p) {
    const Tile t = p.tiles[blockIdx.x];
    const DevLayer L = p.layers[t.layer];
    if (L.family != LGRECO_TOPK) return;
    const int64_t k = L.iparam;
    const int64_t e0 = k * t.pos / L.numel, e1 = k * (t.pos + t.count) / L.numel;
    const float* const values = reinterpret_cast<const float*>(p.payload + L.payload);
    const uint32_t* const indices = reinterpret_cast<const uint32_t*>(p.payload + L.payload) + k;
    float* const out = p.out + L.offset;
    for (int64_t i = e0 + threadIdx.x; i < e1; i += kThreads) {
        const uint32_t ix = indices[i];
        if ((int64_t)ix < L.numel) out[ix] = p.accumulate ? out[ix] + values[i] : values[i];
    }
}

// Gradient accumulation between two runs of the algorithm (section "Implementation": per-layer
// gradients are accumulated in auxiliary buffers in between runs).  acc = g or acc += g, fp32.  Bound by HBM; a
// thread takes 4 elements and is done (see quant_compress_kernel), beyond 2^30 elements as often as it takes: 355 M
// elements added 937 -> 673 us a call, copied 588 -> 449 (against 4096 workgroups that stride).
__global__ __launch_bounds__(kThreads) void accumulate_kernel(float* __restrict__ acc, const float* __restrict__ g,
                                                              int64_t n, int reset) {
    const int64_t n4 = n / 4;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t v = (int64_t)blockIdx.x * kThreads + threadIdx.x; v < n4; v += stride) {
        float4 a = load_stream(g + 4 * v);
        if (!reset) {
            const float4 o = load_stream(acc + 4 * v);
            a.x += o.x; a.y += o.y; a.z += o.z; a.w += o.w;
        }
        store_stream(acc + 4 * v, a);
    }
    if (blockIdx.x == 0 && threadIdx.x < n - 4 * n4) {
        const int64_t i = 4 * n4 + threadIdx.x;
        acc[i] = reset ? g[i] : acc[i] + g[i];
    }
}

hipError_t launch_accumulate(float* acc, const float* g, int64_t n, bool reset, hipStream_t s, Section* sec) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n / 4 + kThreads - 1) / kThreads + 1, 1 << 20);
    launch_timed(sec, true, true, accumulate_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, acc, g, n, reset ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_decode(const uint8_t* payload, const DevLayer* layers, const Tile* tiles, int n_tiles, int tile_elems,
                         int64_t quantized, int64_t total, float* out, bool accumulate, bool any_topk, Timing* tm, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    DecodeParams p{payload, layers, tiles, out, accumulate ? 1 : 0, 0, 0};
    if (quantized > 0) {
        // longer ones where most of the workgroups would only find that their layer is another family's (see
        // launch_quant_compress)
        DecodeParams q = p;
        q.part_shift = part_shift(n_tiles, total, tile_elems, 4 * quantized >= 3 * total ? kDecodePart : 4 * kDecodePart);
        q.part_elems = tile_elems >> q.part_shift;
        const dim3 grid((unsigned)n_tiles << q.part_shift);
        Section sec(tm, "quant_decode", true);
        if (accumulate) launch_timed(&sec, true, true, quant_decode_kernel<true>, grid, dim3(kThreads), 0, s, q);
        else launch_timed(&sec, true, true, quant_decode_kernel<false>, grid, dim3(kThreads), 0, s, q);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (any_topk) {
        Section sec(tm, "topk_decode", true);
        if (!accumulate) {
            launch_timed(&sec, true, false, topk_decode_zero_kernel, dim3(n_tiles), dim3(kThreads), 0, s, p);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        launch_timed(&sec, true, true, topk_decode_scatter_kernel, dim3(n_tiles), dim3(kThreads), 0, s, p);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lgreco
