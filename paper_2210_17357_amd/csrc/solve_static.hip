// lgreco_solve_static: the solver for callers that cannot allocate (code under HIP graph capture,
// tight serving loops, harnesses that forbid hipMalloc).  Same kernels as lgreco_profile_solve's
// device-side route (solve.hip), with every intermediate table in one file-scope
// device array instead of a handle's allocations.  Inputs and outputs are the caller's device
// buffers; nothing is copied to or from the host and the call does not wait.
#include "internal.h"

// The arg-min table of solves whose intervals do not fit LDS, then the result block.  One copy per
// GPU the library runs on, held until the process ends.  In host code this name is a stand-in,
// not an address: the address on the current device comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[LGRECO_STATIC_MAX_PD_BYTES + 256];

namespace lgreco {
namespace {

constexpr int kStaticMaxLP = 4096;                              // table entries
constexpr int kStaticMaxP = 16;
constexpr size_t kStaticPdBytes = LGRECO_STATIC_MAX_PD_BYTES;   // arg-min table, one byte per cell
constexpr size_t kOffResult = kStaticPdBytes;                   // int64 [16] (+ pad)
static_assert(kOffResult + 256 == sizeof(scratch), "the array above is declared with this size");
static_assert(kStaticMaxLP <= kSolveMaxEntries, "such a table never has too many entries for the kernel");
static_assert(kStaticMaxP <= 64, "nor too long a list for its last resort");

constexpr int kMaxDevices = 64;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

// Totals of the assignment the solver kernel left in choice (status 0), or each layer's minimum-error
// candidate (status 1, no assignment fits: totals 0): one workgroup.
__global__ __launch_bounds__(kSolveMaxLayers) void static_gather_kernel(
    const double* __restrict__ errors, const int64_t* __restrict__ sizes, int L, int P,
    const int64_t* __restrict__ solved, int32_t* __restrict__ choice, int64_t* __restrict__ out) {
    __shared__ double s_err[kSolveMaxLayers];
    __shared__ int64_t s_size[kSolveMaxLayers];
    const int tid = threadIdx.x;
    const int64_t status = solved[0];
    if (status == 1 && tid < L) {
        int best = 0;
        for (int c = 1; c < P; ++c)
            if (errors[(size_t)tid * P + c] < errors[(size_t)tid * P + best]) best = c;
        choice[tid] = best;
    }
    if (status == 0 && tid < L) {
        const int c = choice[tid];
        s_err[tid] = errors[(size_t)tid * P + c];
        s_size[tid] = sizes[(size_t)tid * P + c];
    }
    __syncthreads();
    if (tid == 0) {
        // totals in layer order, as the host route sums them
        double terr = 0.0;
        int64_t tsize = 0;
        if (status == 0)
            for (int l = 0; l < L; ++l) {
                terr += s_err[l];
                tsize += s_size[l];
            }
        out[0] = status;
        out[1] = tsize;
        out[2] = (int64_t)__builtin_bit_cast(uint64_t, terr);
        out[3] = solved[6];                                    // bit pattern of E_max
    }
}

}  // namespace
}  // namespace lgreco

using namespace lgreco;

extern "C" int lgreco_solve_static(const double* d_errors, const int64_t* d_sizes, int32_t L, int32_t P,
                                   int32_t default_cand, int32_t n_bins, int32_t* d_choice, int64_t* d_result,
                                   void* stream) {
    if (!d_errors || !d_sizes || !d_choice || !d_result || L <= 0 || P <= 0) return LGRECO_EINVAL;
    if (default_cand < 0 || default_cand >= P || n_bins < 1) return LGRECO_EINVAL;
    if ((uintptr_t)d_errors % 16 || (uintptr_t)d_sizes % 16) return LGRECO_EINVAL;
    // the stated maximum: what the scratch array and the device-side list building hold
    if (L > kSolveMaxLayers || P > kStaticMaxP || (int64_t)L * P > kStaticMaxLP || n_bins > LGRECO_MAX_BINS)
        return LGRECO_ENOSPACE;
    const size_t pd_stride = ((size_t)n_bins + 1 + 3) & ~(size_t)3;
    if ((size_t)L * pd_stride > kStaticPdBytes) return LGRECO_ENOSPACE;

    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LGRECO_EHIP;
    if (!g_scratch_ptr[dev]) {
        // once per device, with that device current: each GPU holds its own copy at its own address
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LGRECO_EHIP;
        g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
    }
    unsigned char* const base = g_scratch_ptr[dev];
    int64_t* const result = reinterpret_cast<int64_t*>(base + kOffResult);

    hipStream_t s = (hipStream_t)stream;
    // Nothing in the scratch has to start at zero: the solver writes every arg-min cell its back-trace
    // reads, and the gather step reads what the solver wrote.
    SolveParams sp{};
    sp.errors = d_errors;
    sp.sizes = d_sizes;
    sp.L = L;
    sp.P = P;
    sp.D = n_bins;
    sp.default_cand = default_cand;
    sp.e_limit = n_bins;
    sp.check_sizes = 1;
    sp.last_resort = 1;
    sp.choice = d_choice;
    sp.result = result;
    sp.seq = 1;
    sp.pd = base;
    if (launch_solve(sp, s, nullptr) != hipSuccess) return LGRECO_EHIP;
    hipLaunchKernelGGL(static_gather_kernel, dim3(1), dim3(kSolveMaxLayers), 0, s, d_errors, d_sizes, (int)L, (int)P,
                       (const int64_t*)result, d_choice, d_result);
    return hipGetLastError() == hipSuccess ? LGRECO_OK : LGRECO_EHIP;
}
