// C ABI of libe0m4: argument validation and dispatch.  Every check happens on
// the host before anything is enqueued, so an error return means no kernel ran.
#include <string.h>

#include <atomic>

#include "e0m4_device.h"
#include "e0m4_host.h"

namespace e0m4 {

namespace {

thread_local char g_hip_error[256] = "";

// Diagnostic knobs belong to the calling thread: a size query and the call it sizes, made from one thread,
// always see the same values, and a thread that never sets a knob always gets the built-in heuristics.
const char* const kKnobNames[] = {      // in the order of Knob
    "gemv_waves",                 // wavefronts per workgroup of the small-M kernel (4, 8 or 16)
    "gemv_workgroups",            // target number of workgroups of the small-M kernel
    // the matrix-core small-batch kernels: 1 neither; 2 activations staged in LDS always read from there; 3 their wavefront sums
    // reduced per row block; 4 plain matmuls on dequantised operands wherever that can run, 5 never; 6 staged also for groups of
    // 64 and 32 wherever that can run; 7 plain matmuls on exact codes without staging wherever that can run, 8 never; 9 as 6, and
    // X block by block wherever that can run
    "gemv_mfma",
    "gemv_xreg",                  // M = 1 kernel, a wavefront's activations in registers: 2 never
    "gemm_variant",               // 1: small-tile kernel; pipelined kernel with tiles of 2: 256 x 256, 3: 128 x 128, 4: 64 x 256, 5: 128 x 256, 6: 64 x 128, 7: that with K quarters
    "gemm_splits",                // force the number of K splits of the pipelined GEMM kernel
    "gemm_sk",                    // even scheduling of the 256 x 256 tiles over the compute units: 1 whenever the last round is partly filled, 2 never
    "gemm_panel",                 // row tiles per panel of the pipelined GEMM's tile numbering (0: the default, -1: whole columns)
    "gemm_split_order",           // work items of a K-split launch: 1 by tile, 2 by split (0: by the length of a split)
};
static_assert(sizeof(kKnobNames) / sizeof(kKnobNames[0]) == (size_t)Knob::count, "a name for each");

// Scratch of e0m4_matmul_static: the split-K partial sums that e0m4_matmul keeps in the caller's workspace.
// Every GPU the library runs on holds its own copy of the array, at its own address, until the process ends.
constexpr size_t kStaticScratchBytes = E0M4_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device, looked up once per device (in host code the array's
// name is only a handle for this lookup, never an address a kernel may use).
constexpr int kMaxTrackedDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxTrackedDevices];

int static_scratch(void** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return record_hip_error(e);
    if (dev >= 0 && dev < kMaxTrackedDevices) {
        void* known = g_scratch_ptr[dev].load(std::memory_order_acquire);
        if (known) {
            *out = known;
            return E0M4_OK;
        }
    }
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return record_hip_error(e);
    if (!ptr) return record_hip_error(hipErrorInvalidSymbol);
    if (dev >= 0 && dev < kMaxTrackedDevices) g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    *out = ptr;
    return E0M4_OK;
}

__global__ void zero_fill_kernel(half_t* y, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) y[i] = (half_t)0.f;
}

bool group_ok(int group) { return group == 32 || group == 64 || group == 128; }
// The small-batch kernel that stages X in LDS, for plain matmuls (gemv_mfma 1: off; 6 and 9: also for groups of 64 and 32 wherever
// it can run, which by default it does where it pays).
bool use_gemv_mfma(int64_t M, int64_t N, int64_t K, int group)
{
    const int k = knob(Knob::gemv_mfma);
    if (k == 1 || !gemv_mfma_supported(M, N, K, group)) return false;
    return group == 128 || k == 6 || k == 9 || gemv_mfma_groups_pay(M, N, K, group);
}
// M <= kGemvMaxM rows take the vector decode kernel, whose time grows with M, unless the matrix-core GEMM
// (64 x 256 tile, time nearly independent of M) is faster: measured crossover at about M * N * K = 3.8e8
// (27392 x 4096 from M = 4 on, 4096 x 13696 from M = 7 on, never for 4096 x 4096).
bool small_m_on_vector(int64_t M, int64_t N, int64_t K)
{
    if (M > kGemvMaxM) return false;
    if (M < 2 || !gemm_pipe_supported(K) || N > (int64_t)1 << 24) return true;
    return (double)M * (double)N * (double)K < 3.8e8;
}
// 17 <= M <= kChunkedMaxM on small weights: the small-batch matrix-core kernel on equal chunks of at most 16 rows,
// dealt to the y dimension of one launch (the chunks of a workgroup's row blocks follow each other on a compute unit
// or run side by side on the same XCD: the weights come from HBM once), instead of the GEMM, whose 64 x 256 tile with
// its split along K costs 12 - 20 us whatever M is.  The launch takes about as long as one chunk times the rounds its
// workgroups make on the 256 compute units (staging a chunk of X costs a workgroup more than its weights do):
// 4608 x 4096 (144 workgroups) 7.3 us at M = 16, 11.9 at M = 32 and 12.1 at M = 48 (two rounds; GEMM 15.2 and 16.4),
// 17.0 at M = 64 (three; GEMM 17.6); 4096 x 4096 (256 workgroups) 10.8 at M = 32 (GEMM 14.8), 15.0 at M = 48 (16.1),
// 19.1 at M = 64 (four rounds; GEMM 17.1).  So: two rounds at most, or three on small weights.  Not when a chunk of X
// needs phases along K.
constexpr int64_t kChunkRows = 16, kChunkedMaxM = 64, kChunked8MaxM = 32;
int row_chunks(int64_t M) { return (int)((M + kChunkRows - 1) / kChunkRows); }
int64_t rows_per_chunk(int64_t M) { return (M + row_chunks(M) - 1) / row_chunks(M); }
bool small_batch_in_chunks(const Fusion& f, int64_t M, int64_t N, int64_t K, int group, WholeRowsPlan* plan = nullptr)
{
    if (M <= kChunkRows || M > kChunkedMaxM || knob(Knob::gemv_mfma) == 1 || (double)N * (double)K > 7e7) return false;
    WholeRowsPlan p;
    if (!gemv_mfma_whole_rows(f, rows_per_chunk(M), N, K, group, &p)) return false;
    if (plan) *plan = p;
    const int64_t rounds = (row_chunks(M) * p.workgroups + 255) / 256;
    return rounds <= 2 || (rounds == 3 && (double)N * (double)K <= 2e7);
}
// Any of the GEMM's knobs is set: it keeps the calls that are its own without the kernel below.
bool gemm_steered()
{
    return knob(Knob::gemm_variant) || knob(Knob::gemm_splits) || knob(Knob::gemm_sk) || knob(Knob::gemm_panel) || knob(Knob::gemm_split_order);
}
// The small-batch kernel with dequantised weight operands, for plain matmuls.  It rounds every weight to 16 bits before the
// product, as the GEMM does; the kernels above work on the codes' exact values and apply scale and bias in fp32.  So it never
// takes a call from one of those, only, where it is the faster one, from the GEMM -- and, at 3 <= M <= 16 in groups of 32 and
// 64, what use_gemv_mfma leaves.  gemv_mfma 4 forces it wherever it can run (2 <= M <= 128), 1 and 5 switch it off.
bool use_gemv_dq(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    const int k = knob(Knob::gemv_mfma);
    if (k == 1 || k == 5 || !gemv_dq_supported(M, N, K, group)) return false;
    return k == 4 || gemv_dq_pays(M, N, K, group, format);
}
// The same for fused calls that would be the GEMM's, with an rms-norm alone or without operators.
bool use_gemv_dq_fused(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    const int k = knob(Knob::gemv_mfma);
    if (k == 1 || k == 5 || !gemv_dq_supported(M, N, K, group)) return false;
    return k == 4 || gemv_dq_beats_gemm(M, N, K, group, format);
}
bool use_gemv_dq4(int64_t M, int64_t N, int64_t K, int group)
{
    if (M < 2) return false;
    if (knob(Knob::gemv_mfma) != 4) {
        if (use_gemv_mfma(M, N, K, group) || small_batch_in_chunks(Fusion{}, M, N, K, group)) return false;
        const bool fits = M <= kGemvMaxM || (M <= 16 && M * (k_blocks(K) * 256 + 16) <= 140 * 1024);
        if (group != 128 && M >= 3 && fits) return use_gemv_dq(M, N, K, group, kDqFormatFp16);
        // what is left is the GEMM's, with its limit of 2^24 columns
        if (gemm_steered() || small_m_on_vector(M, N, K) || N > (int64_t)1 << 24) return false;
    }
    return use_gemv_dq(M, N, K, group, kDqFormatFp16);
}
// (whether such calls have no workspace to bring)
bool dq4_free(int64_t M, int64_t N, int64_t K, int group)
{
    return knob(Knob::gemv_mfma) == 4 || gemv_dq_free(M, N, K, group, kDqFormatFp16);
}
// bfloat16 of up to eight rows: the small-batch kernel, which multiplies the codes' exact values as the vector kernel does but
// whose time hardly grows with the rows (27392 x 5120 at M = 5 32 -> 18.3 us; M = 2 21.5 -> 18.4).  Its time over the vector kernel's:
//   Groups of 64 and 32 from three rows on (2560 x 2048 at M = 2 4.4 us there and 4.8 here, at M = 3 5.6 and 4.8), 0.37 - 1.02 on 1 100
//     calls (rows of up to 1024 weights to 1.07, of 512 at four rows to 1.12).  But 1.03 - 1.21 with K in phases on one row block per
//     workgroup and up to twelve work items (of 512 weights) per row, at three and four rows (2704 x 5120 in groups of 32 at M = 3
//     6.8 and 8.2); and 0.97 - 1.17 at three rows with up to four work items per row where a workgroup of several row blocks has up
//     to four or eight to twelve in all, which the vector kernel's wavefronts divide evenly (16000 x 1536 6.9 and 7.6, 7368 x 2048 5.6
//     and 6.3).
//   Two rows in groups of 128 on 117 problems: 0.79 - 0.93 with more than six work items per row, and with five or six where
//     workgroups have one row block each; else 0.95 - 1.15 (2560 x 2048 4.2 and 4.6, 7680 x 2560 5.8 and 6.4), but 0.79 - 1.04 with more
//     than five row blocks per workgroup and more than three work items.
// (gemv_mfma 1: the vector kernel, 6: this one from two rows on)
bool use_gemv_mfma_bf16(int64_t M, int64_t N, int64_t K, int group)
{
    const int k = knob(Knob::gemv_mfma);
    if (M > kGemvMaxM || k == 1 || !gemv_mfma_supported(M, N, K, group)) return false;
    if (k == 6 || (M > 2 && group == 128)) return true;
    const int64_t items = (k_blocks(K) + 3) / 4, rb = (row_blocks(N) + 255) / 256;
    if (M > 2) {
        if (M <= 4 && rb == 1 && items <= 12 && !gemv_mfma_whole_rows(Fusion{}, M, N, K, group)) return false;
        return M > 3 || items > 4 || rb == 1 || rb * items > 12 || (rb * items > 4 && rb * items < 8);
    }
    return group == 128 && (items > 6 || (items > 4 && rb == 1) || (items > 3 && rb > 5));
}
// The kernel of use_gemv_dq on exact codes, which multiplies unrounded weights, for plain matmuls (gemv_mfma 7 forces it wherever it
// can run; any other value but 0 leaves its calls to the kernels that have them otherwise).
bool use_gemv_exact(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    const int k = knob(Knob::gemv_mfma);
    if ((k != 0 && k != 7) || !gemv_exact_supported(M, N, K, group, format)) return false;
    if (k == 7) return true;
    if (gemm_steered() || N > (int64_t)1 << 24) return false;
    if (format == kDqFormatBf16) return gemv_exact_pays_bf16(M, N, K);
    WholeRowsPlan p;
    return small_batch_in_chunks(Fusion{}, M, N, K, group, &p) && gemv_exact_pays_chunks(M, row_chunks(M), p);
}
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Shape rules shared by all entry points.
int check_shape(int64_t N, int64_t K, int group)
{
    if (!group_ok(group)) return E0M4_ERR_GROUP;
    if (N < 0 || K < 0 || (K % kCodesPerChunk) != 0 || (K % group) != 0) return E0M4_ERR_SHAPE;
    if (N > (int64_t)1 << 31 || K > (int64_t)1 << 20) return E0M4_ERR_SHAPE;   // 32-bit offsets in the kernels
    return E0M4_OK;
}

}  // namespace

int record_hip_error(hipError_t e)
{
    if (e == hipSuccess) return E0M4_OK;
    strncpy(g_hip_error, hipGetErrorString(e), sizeof(g_hip_error) - 1);
    g_hip_error[sizeof(g_hip_error) - 1] = 0;
    return E0M4_ERR_HIP;
}

int check_launch() { return record_hip_error(hipGetLastError()); }

__thread int g_knobs[(int)Knob::count] = {};

}  // namespace e0m4

using namespace e0m4;

extern "C" {

int e0m4_abi_version(void) { return E0M4_ABI_VERSION; }

const char* e0m4_strerror(int code)
{
    switch (code) {
        case E0M4_OK: return "ok";
        case E0M4_ERR_NULL: return "a required pointer is NULL";
        case E0M4_ERR_SHAPE: return "bad shape: sizes must be >= 0 and within their limits, K a multiple of 32 and of the group size";
        case E0M4_ERR_GROUP: return "unsupported group size (supported: 32, 64, 128)";
        case E0M4_ERR_ALIGN: return "a data pointer is not 16-byte aligned";
        case E0M4_ERR_WORKSPACE: return "workspace is smaller than e0m4_workspace_bytes()";
        case E0M4_ERR_HIP: return "HIP launch failed (see e0m4_last_hip_error)";
        default: return "unknown error code";
    }
}

const char* e0m4_last_hip_error(void) { return g_hip_error; }

size_t e0m4_codes_bytes(int64_t N, int64_t K, int group)
{
    if (check_shape(N, K, group) != E0M4_OK) return 0;
    return (size_t)row_blocks(N) * (size_t)k_blocks(K) * (size_t)block_bytes(group);
}

size_t e0m4_params_elems(int64_t N, int64_t K, int group)
{
    if (check_shape(N, K, group) != E0M4_OK) return 0;
    return (size_t)N * (size_t)(K / group);
}

size_t e0m4_workspace_bytes(int64_t M, int64_t N, int64_t K, int group)
{
    if (check_shape(N, K, group) != E0M4_OK || M <= 0 || N == 0 || K == 0) return 0;             // invalid or empty: nothing runs
    if (use_gemv_exact(M, N, K, group, kDqFormatFp16)) return 0;
    if (small_m_on_vector(M, N, K)) return 0;           // the small-M kernels need none
    if (use_gemv_dq4(M, N, K, group) && dq4_free(M, N, K, group)) return 0;
    if (use_gemv_mfma(M, N, K, group) || small_batch_in_chunks(Fusion{}, M, N, K, group)) return 0;
    return gemm_workspace_bytes(M, N, K);       // partial tiles of the split-K GEMM, if it splits
}

// Fused matmul: the normalised copy of X (GEMM path with rms-norm) comes first in the workspace,
// rounded up to 256 bytes, then the partial sums of the split along K.
static size_t norm_bytes(int64_t M, int64_t K) { return ((size_t)M * (size_t)K * 2 + 255) & ~(size_t)255; }

// Which kernel family serves a fused matmul.
enum FusedPath {
    kFusedNone = -1,
    kFusedVector,                                       // the decode kernel, everything in one launch
    kFusedGemm,                                         // (an rms-norm is a launch of its own before it)
    kFusedSmallBatch,                                   // the small-batch kernel on the matrix cores, everything in one launch
    kFusedChunks,                                       // that kernel on chunks of rows
    kFusedTiles,                                        // the same sums with all rows in a workgroup (an rms-norm is a launch before it)
    kFusedExact,                                        // no operators: the kernel on exact codes
    kFusedDq,                                           // an rms-norm alone or nothing, as for the GEMM: the kernel with dequantised operands
};
// An rms-norm alone (a projection into q, k and v, or to the vocabulary) and calls without operators may go where the plain call
// goes.  Calls with a residual or the gated product keep the GEMM and its order of the sums, though the kernel with dequantised
// operands would be faster: a stack of blocks amplifies the rounding of a residual stream that is summed in another order.
static bool as_plain(const Fusion& f) { return !f.residual && !f.swiglu; }
// (`may_tiles`: the question is whether a call of the chunks goes in tiles)
static FusedPath fused_path(const Fusion& f, int64_t M, int64_t N, int64_t K, int group, bool may_tiles, TilesPlan* tiles = nullptr)
{
    if (!f.any() && use_gemv_exact(M, N, K, group, kDqFormatFp16)) return kFusedExact;
    // (groups of 64 and 32 from three rows on: 1.1 - 2 x the vector kernel and the GEMM there, 10 - 25 % slower than the
    // vector kernel at two rows)
    const int k = knob(Knob::gemv_mfma);
    if (k != 1 && gemv_mfma_fused_supported(f, M, N, K, group) && (group == 128 || M >= 3 || k == 6 || k == 9)) return kFusedSmallBatch;
    if (small_batch_in_chunks(f, M, N, K, group)) {
        TilesPlan p;
        const bool can = may_tiles && f.any() && group == 128 && (k == 0 || k == 7) && gemv_tiles_plan(f, M, row_chunks(M), N, K, &p) &&
                         gemv_tiles_supported(p, M, K);
        if (!can || (k == 0 && !gemv_tiles_pays(f, p, M, row_chunks(M)))) return kFusedChunks;
        if (tiles) *tiles = p;
        return kFusedTiles;
    }
    if (small_m_on_vector(M, N, K) && gemv_fused_supported(f, M, N, K)) return kFusedVector;
    return as_plain(f) && !gemm_steered() && N <= (int64_t)1 << 24 && use_gemv_dq_fused(M, N, K, group, kDqFormatFp16) ? kFusedDq : kFusedGemm;
}

// The workspace that a call has to bring: the normalised X, the GEMM's partial sums behind it.  (Calls of the kernel with
// dequantised operands have the same to bring as when they were the GEMM's; calls in tiles may do without, in chunks: `best`.)
static size_t fused_bytes(int64_t M, int64_t N, int64_t K, int group, bool normed, int epilogue, bool best)
{
    if (check_shape(N, K, group) != E0M4_OK || M <= 0 || N == 0 || K == 0) return 0;
    if (epilogue != E0M4_EPILOGUE_NONE && epilogue != E0M4_EPILOGUE_SWIGLU) return 0;
    Fusion f;
    f.swiglu = epilogue == E0M4_EPILOGUE_SWIGLU;
    f.residual = &f;                                    // (a call without a residual needs no more than one with it)
    if (best && normed) f.gamma = &f;                   // (which of the kernels without a need is the fastest depends on the rms-norm)
    const FusedPath path = fused_path(f, M, N, K, group, best && normed);
    if (best && path == kFusedTiles && normed) return norm_bytes(M, K);
    if (path != kFusedGemm) return 0;                   // (with a residual it is never the kernel with dequantised operands)
    return (normed ? norm_bytes(M, K) : 0) + gemm_workspace_bytes(M, N, K, f.swiglu, true);
}

size_t e0m4_fused_workspace_bytes(int64_t M, int64_t N, int64_t K, int group, int with_rmsnorm, int epilogue)
{
    return fused_bytes(M, N, K, group, with_rmsnorm != 0, epilogue, false);
}

size_t e0m4_fused_workspace_best_bytes(int64_t M, int64_t N, int64_t K, int group, int with_rmsnorm, int epilogue)
{
    return fused_bytes(M, N, K, group, with_rmsnorm != 0, epilogue, true);
}

int e0m4_set_knob(const char* name, int value)
{
    if (!name) return E0M4_ERR_NULL;
    for (int k = 0; k < (int)Knob::count; ++k)
        if (strcmp(kKnobNames[k], name) == 0) {
            g_knobs[k] = value;
            return E0M4_OK;
        }
    return E0M4_ERR_SHAPE;
}

int e0m4_quantize(const void* W, int64_t N, int64_t K, int group, void* codes, void* scales, void* bias, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !bias) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(bias)) return E0M4_ERR_ALIGN;
    return launch_quantize(W, N, K, group, codes, scales, bias, nullptr, nullptr, true, kFormatE0M4, (hipStream_t)stream);
}

int e0m4_encode(const void* W, int64_t N, int64_t K, int group, const void* scales, const void* bias, void* codes,
                void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !bias) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(bias)) return E0M4_ERR_ALIGN;
    return launch_quantize(W, N, K, group, codes, nullptr, nullptr, scales, bias, false, kFormatE0M4, (hipStream_t)stream);
}

int e0m4_dequant(const void* codes, const void* scales, const void* bias, int64_t N, int64_t K, int group, void* W_out,
                 void* stream)
{
    (void)scales; (void)bias;                   // the packed buffer carries its own copy of the parameters
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W_out || !codes) return E0M4_ERR_NULL;
    if (!aligned16(W_out) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    return launch_dequant(codes, N, K, group, W_out, kFormatE0M4, (hipStream_t)stream);
}

int e0m4_int4_quantize(const void* W, int64_t N, int64_t K, int group, void* codes, void* scales, void* zeros,
                       void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !zeros) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(zeros)) return E0M4_ERR_ALIGN;
    return launch_quantize(W, N, K, group, codes, scales, zeros, nullptr, nullptr, true, kFormatInt4, (hipStream_t)stream);
}

int e0m4_int4_dequant(const void* codes, int64_t N, int64_t K, int group, void* W_out, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W_out || !codes) return E0M4_ERR_NULL;
    if (!aligned16(W_out) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    return launch_dequant(codes, N, K, group, W_out, kFormatInt4, (hipStream_t)stream);
}

int e0m4_int4_gemv(const void* X, const void* codes, int64_t N, int64_t K, int group, void* Y, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0) return E0M4_OK;
    if (!Y) return E0M4_ERR_NULL;
    if (!aligned16(Y)) return E0M4_ERR_ALIGN;
    if (K == 0) {                                   // empty contraction: Y = 0
        hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           static_cast<half_t*>(Y), N);
        return check_launch();
    }
    if (!X || !codes) return E0M4_ERR_NULL;
    if (!aligned16(X) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    return launch_gemv_int4(X, codes, N, K, group, Y, (hipStream_t)stream);
}

int e0m4_unpack_codes(const void* codes, int64_t N, int64_t K, int group, void* out, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!codes || !out) return E0M4_ERR_NULL;
    if (!aligned16(codes) || !aligned16(out)) return E0M4_ERR_ALIGN;
    return launch_unpack(codes, N, K, group, out, (hipStream_t)stream);
}

// the workspace of a plain call that the GEMM would have otherwise, by the GEMM's rules: refused also where nobody uses it
static int check_workspace(size_t need, const void* workspace, size_t bytes)
{
    if (bytes > 0 && (!workspace || !aligned16(workspace))) return workspace ? E0M4_ERR_ALIGN : E0M4_ERR_NULL;
    return bytes < need ? E0M4_ERR_WORKSPACE : E0M4_OK;
}

int e0m4_matmul(const void* X, int64_t M, const void* codes, const void* scales, const void* bias, int64_t N, int64_t K,
                int group, void* Y, void* workspace, size_t workspace_bytes, void* stream)
{
    (void)scales; (void)bias;
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (M < 0 || M > (int64_t)1 << 31) return E0M4_ERR_SHAPE;
    if (M == 0 || N == 0) return E0M4_OK;
    if (!Y) return E0M4_ERR_NULL;
    if (!aligned16(Y)) return E0M4_ERR_ALIGN;
    if (K == 0) {                                   // empty contraction: Y = 0
        const int64_t total = M * N;
        hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           static_cast<half_t*>(Y), total);
        return check_launch();
    }
    if (!X || !codes) return E0M4_ERR_NULL;
    if (!aligned16(X) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    if (use_gemv_exact(M, N, K, group, kDqFormatFp16))
        return launch_gemv_exact(X, M, codes, N, K, kDqFormatFp16, Y, (hipStream_t)stream);
    if (use_gemv_dq4(M, N, K, group)) {
        if (!dq4_free(M, N, K, group)) rc = check_workspace(e0m4_workspace_bytes(M, N, K, group), workspace, workspace_bytes);
        return rc != E0M4_OK ? rc : launch_gemv_dq(X, M, codes, N, K, group, kDqFormatFp16, Y, (hipStream_t)stream);
    }
    if (use_gemv_mfma(M, N, K, group)) return launch_gemv_mfma(X, M, codes, N, K, Y, (hipStream_t)stream, 1, group);
    if (small_m_on_vector(M, N, K)) return launch_gemv(X, M, codes, N, K, group, Y, (hipStream_t)stream);
    if (small_batch_in_chunks(Fusion{}, M, N, K, group))
        return launch_gemv_mfma(X, M, codes, N, K, Y, (hipStream_t)stream, row_chunks(M), group);
    if (N > (int64_t)1 << 24) return E0M4_ERR_SHAPE;    // the GEMM epilogue forms 32-bit offsets of up to 256 rows of Y
    if (workspace_bytes > 0 && (!workspace || !aligned16(workspace))) return workspace ? E0M4_ERR_ALIGN : E0M4_ERR_NULL;
    return launch_gemm(X, M, codes, N, K, group, Y, workspace, workspace_bytes, (hipStream_t)stream);
}

int e0m4_matmul_static(const void* X, int64_t M, const void* codes, int64_t N, int64_t K, int group, void* Y, void* stream)
{
    // the shape decides the scratch size before anything else is looked at; nothing is allocated anywhere below
    const size_t need = e0m4_workspace_bytes(M, N, K, group);
    if (need > kStaticScratchBytes) return E0M4_ERR_WORKSPACE;
    void* ws = nullptr;
    if (need > 0) {
        const int rc = static_scratch(&ws);
        if (rc != E0M4_OK) return rc;
    }
    return e0m4_matmul(X, M, codes, nullptr, nullptr, N, K, group, Y, ws, need, stream);
}

// (`best`: a workspace of e0m4_fused_workspace_best_bytes may be written, else one of e0m4_fused_workspace_bytes)
static int matmul_fused(const void* X, int64_t M, const void* rms_gamma, float rms_eps, const void* codes, int64_t N, int64_t K,
                        int group, int epilogue, const void* residual, void* Y, void* workspace, size_t workspace_bytes, bool best,
                        void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (M < 0 || M > (int64_t)1 << 31) return E0M4_ERR_SHAPE;
    if (epilogue != E0M4_EPILOGUE_NONE && epilogue != E0M4_EPILOGUE_SWIGLU) return E0M4_ERR_SHAPE;
    Fusion f;
    f.gamma = rms_gamma;
    f.eps = rms_eps;
    f.residual = residual;
    f.swiglu = epilogue == E0M4_EPILOGUE_SWIGLU;
    // the gated epilogue pairs weight row j with row N/2 + j: the halves must be whole pairs of 16-row blocks
    if (f.swiglu && (N % (4 * kBlockRows)) != 0) return E0M4_ERR_SHAPE;
    if (M == 0 || N == 0) return E0M4_OK;
    if (K == 0) return E0M4_ERR_SHAPE;                  // nothing to normalise or to gate
    if (!X || !codes || !Y) return E0M4_ERR_NULL;
    if (!aligned16(X) || !aligned16(codes) || !aligned16(Y) || (rms_gamma && !aligned16(rms_gamma)) ||
        (residual && !aligned16(residual)))
        return E0M4_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    TilesPlan tiles;
    FusedPath path = fused_path(f, M, N, K, group, best || !rms_gamma, &tiles);
    const size_t nb = rms_gamma ? norm_bytes(M, K) : 0;
    // (chunks need no workspace: calls without one stay there)
    if (path == kFusedTiles && nb > 0 && (!workspace || !aligned16(workspace) || workspace_bytes < nb)) path = kFusedChunks;
    if (path == kFusedSmallBatch) return launch_gemv_mfma_fused(f, X, M, codes, N, K, Y, st, 1, group);
    if (path == kFusedVector) return launch_gemv_fused(f, X, M, codes, N, K, group, Y, st);
    if (path == kFusedExact) return launch_gemv_exact(X, M, codes, N, K, kDqFormatFp16, Y, st);
    if (path == kFusedChunks) return launch_gemv_mfma_fused(f, X, M, codes, N, K, Y, st, row_chunks(M), group);      // rows are independent
    if (N > (int64_t)1 << 24) return E0M4_ERR_SHAPE;    // 32-bit offsets in the GEMM epilogue
    const size_t need = path == kFusedTiles ? 0 : nb + gemm_workspace_bytes(M, N, K, f.swiglu, true);
    if (need > 0) {
        if (!workspace) return E0M4_ERR_NULL;
        if (!aligned16(workspace)) return E0M4_ERR_ALIGN;
        if (workspace_bytes < need) return E0M4_ERR_WORKSPACE;
    }
    const void* x = X;
    if (rms_gamma) {
        rc = launch_rmsnorm(X, M, K, rms_gamma, rms_eps, workspace, st, path == kFusedTiles ? tiles.waves : 4);
        if (rc != E0M4_OK) return rc;
        x = workspace;
        f.gamma = nullptr;
    }
    if (path == kFusedTiles) return launch_gemv_tiles(f, tiles, x, M, codes, N, K, Y, st);
    if (path == kFusedDq) return launch_gemv_dq(x, M, codes, N, K, group, kDqFormatFp16, Y, st);
    return launch_gemm_fused(f, x, M, codes, N, K, group, Y, static_cast<char*>(workspace) + nb,
                             workspace_bytes - nb, st);
}

int e0m4_matmul_fused(const void* X, int64_t M, const void* rms_gamma, float rms_eps, const void* codes, int64_t N,
                      int64_t K, int group, int epilogue, const void* residual, void* Y, void* workspace,
                      size_t workspace_bytes, void* stream)
{
    return matmul_fused(X, M, rms_gamma, rms_eps, codes, N, K, group, epilogue, residual, Y, workspace, workspace_bytes, false, stream);
}

int e0m4_matmul_fused_best(const void* X, int64_t M, const void* rms_gamma, float rms_eps, const void* codes, int64_t N,
                           int64_t K, int group, int epilogue, const void* residual, void* Y, void* workspace,
                           size_t workspace_bytes, void* stream)
{
    return matmul_fused(X, M, rms_gamma, rms_eps, codes, N, K, group, epilogue, residual, Y, workspace, workspace_bytes, true, stream);
}

// ---- E0M3: the 3-bit member of the family, stored in 4-bit slots ---------------------------------------
int e0m3_quantize(const void* W, int64_t N, int64_t K, int group, void* codes, void* scales, void* bias, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !bias) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(bias)) return E0M4_ERR_ALIGN;
    return launch_quantize(W, N, K, group, codes, scales, bias, nullptr, nullptr, true, kFormatE0M3, (hipStream_t)stream);
}

int e0m3_unpack_codes(const void* codes, int64_t N, int64_t K, int group, void* out, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!codes || !out) return E0M4_ERR_NULL;
    if (!aligned16(codes) || !aligned16(out)) return E0M4_ERR_ALIGN;
    return launch_unpack(codes, N, K, group, out, (hipStream_t)stream, 1);
}

// ---- E0M4 on bfloat16 ----------------------------------------------------------------------------------
int e0m4_bf16_quantize(const void* W, int64_t N, int64_t K, int group, void* codes, void* scales, void* bias,
                       void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !bias) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(bias)) return E0M4_ERR_ALIGN;
    return launch_quantize(W, N, K, group, codes, scales, bias, nullptr, nullptr, true, kFormatBf16, (hipStream_t)stream);
}

int e0m4_bf16_encode(const void* W, int64_t N, int64_t K, int group, const void* scales, const void* bias, void* codes,
                     void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !bias) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(bias)) return E0M4_ERR_ALIGN;
    return launch_quantize(W, N, K, group, codes, nullptr, nullptr, scales, bias, false, kFormatBf16, (hipStream_t)stream);
}

int e0m4_bf16_dequant(const void* codes, int64_t N, int64_t K, int group, void* W_out, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W_out || !codes) return E0M4_ERR_NULL;
    if (!aligned16(W_out) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    return launch_dequant(codes, N, K, group, W_out, kFormatBf16, (hipStream_t)stream);
}

int e0m4_bf16_matmul(const void* X, int64_t M, const void* codes, int64_t N, int64_t K, int group, void* Y, void* stream)
{
    int rc = check_shape(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (M < 0 || M > (int64_t)1 << 31) return E0M4_ERR_SHAPE;
    if (M == 0 || N == 0) return E0M4_OK;
    if (!Y) return E0M4_ERR_NULL;
    if (!aligned16(Y)) return E0M4_ERR_ALIGN;
    if (K == 0) {                                   // empty contraction: Y = +0 (the same bits in both formats)
        const int64_t total = M * N;
        hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           static_cast<half_t*>(Y), total);
        return check_launch();
    }
    if (!X || !codes) return E0M4_ERR_NULL;
    if (!aligned16(X) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    if (use_gemv_exact(M, N, K, group, kDqFormatBf16))
        return launch_gemv_exact(X, M, codes, N, K, kDqFormatBf16, Y, (hipStream_t)stream);
    if ((knob(Knob::gemv_mfma) == 4 || !gemm_steered()) && use_gemv_dq(M, N, K, group, kDqFormatBf16))
        return launch_gemv_dq(X, M, codes, N, K, group, kDqFormatBf16, Y, (hipStream_t)stream);
    if (use_gemv_mfma_bf16(M, N, K, group)) return launch_gemv_mfma_bf16(X, M, codes, N, K, group, Y, (hipStream_t)stream);
    if (M <= kGemvMaxM) return launch_gemv_bf16(X, M, codes, N, K, group, Y, (hipStream_t)stream);
    if (N > (int64_t)1 << 24) return E0M4_ERR_SHAPE;    // 32-bit offsets in the GEMM epilogue
    return launch_gemm_bf16(X, M, codes, N, K, group, Y, (hipStream_t)stream);
}

// ---- E0M8: the 8-bit member of the format family ------------------------------------------------------
static int check_shape8(int64_t N, int64_t K, int group)
{
    if (group != 64 && group != 128) return E0M4_ERR_GROUP;
    if (N < 0 || K < 0 || (K % 16) != 0 || (K % group) != 0) return E0M4_ERR_SHAPE;
    if (N > (int64_t)1 << 31 || K > (int64_t)1 << 19) return E0M4_ERR_SHAPE;   // 2K 4-bit slots within the K limit
    return E0M4_OK;
}

size_t e0m8_codes_bytes(int64_t N, int64_t K, int group)
{
    if (check_shape8(N, K, group) != E0M4_OK) return 0;
    return (size_t)row_blocks(N) * (size_t)k_blocks(2 * K) * (size_t)block_bytes(128);
}

int e0m8_quantize(const void* W, int64_t N, int64_t K, int group, void* codes, void* scales, void* bias, void* stream)
{
    int rc = check_shape8(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!W || !codes || !scales || !bias) return E0M4_ERR_NULL;
    if (!aligned16(W) || !aligned16(codes) || !aligned16(scales) || !aligned16(bias)) return E0M4_ERR_ALIGN;
    return launch_quantize8(W, N, K, group, codes, scales, bias, (hipStream_t)stream);
}

int e0m8_dequant(const void* codes, int64_t N, int64_t K, int group, void* W_out, void* stream)
{
    int rc = check_shape8(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!codes || !W_out) return E0M4_ERR_NULL;
    if (!aligned16(codes) || !aligned16(W_out)) return E0M4_ERR_ALIGN;
    return launch_dequant8(codes, N, K, W_out, nullptr, (hipStream_t)stream);
}

int e0m8_unpack_codes(const void* codes, int64_t N, int64_t K, int group, void* out, void* stream)
{
    int rc = check_shape8(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (N == 0 || K == 0) return E0M4_OK;
    if (!codes || !out) return E0M4_ERR_NULL;
    if (!aligned16(codes) || !aligned16(out)) return E0M4_ERR_ALIGN;
    return launch_dequant8(codes, N, K, nullptr, out, (hipStream_t)stream);
}

// The pipelined GEMM serves M > 8 when K is a multiple of 128 (its K slices come in pairs).
static bool e0m8_use_mfma_decode(int64_t M, int64_t N, int64_t K)
{
    return knob(Knob::gemv_mfma) != 1 && gemv_mfma8_supported(M, N, K);
}

// The 8-bit form of small_batch_in_chunks.  Twice the weight bytes per launch: the two launches only win on
// small weights with short rows (2048 x 2048: 9 against 11 us, 8192 x 1024: 10 against 10.7; 4096 x 4096 equal,
// 512 x 4096 and larger weights 5 - 20 % slower).
static bool small_batch8_in_chunks(const Fusion& f, int64_t M, int64_t N, int64_t K)
{
    return M > kChunkRows && M <= kChunked8MaxM && knob(Knob::gemv_mfma) != 1 && K <= 2048 && (double)N * (double)K <= 1e7 &&
           gemv_mfma8_whole_rows(f, rows_per_chunk(M), N, K);
}

// the GEMM's calls, of which the kernel with dequantised operands takes those where it pays
static bool e0m8_gemm_or_dq(int64_t M, int64_t N, int64_t K)
{
    return !e0m8_use_mfma_decode(M, N, K) && !small_batch8_in_chunks(Fusion{}, M, N, K) && !small_m_on_vector(M, N, K) &&
           gemm_pipe_supported(K) && N <= (int64_t)1 << 24;
}
static bool e0m8_use_gemv_dq(int64_t M, int64_t N, int64_t K)
{
    return (knob(Knob::gemv_mfma) == 4 || (e0m8_gemm_or_dq(M, N, K) && !gemm_steered())) && use_gemv_dq(M, N, K, 128, kDqFormatE8);
}
static bool e0m8_use_gemm(int64_t M, int64_t N, int64_t K) { return e0m8_gemm_or_dq(M, N, K) && !e0m8_use_gemv_dq(M, N, K); }
static bool e0m8_dq_free(int64_t M, int64_t N, int64_t K) { return knob(Knob::gemv_mfma) == 4 || gemv_dq_free(M, N, K, 128, kDqFormatE8); }

size_t e0m8_workspace_bytes(int64_t M, int64_t N, int64_t K, int group)
{
    if (check_shape8(N, K, group) != E0M4_OK || M <= 0 || N == 0 || K == 0) return 0;
    if (!e0m8_gemm_or_dq(M, N, K) || (e0m8_use_gemv_dq(M, N, K) && e0m8_dq_free(M, N, K))) return 0;
    return gemm_pipe_workspace_bytes(M, N, K, false, true);
}

int e0m8_matmul(const void* X, int64_t M, const void* codes, int64_t N, int64_t K, int group, void* Y, void* workspace,
                size_t workspace_bytes, void* stream)
{
    int rc = check_shape8(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (M < 0 || M > (int64_t)1 << 31) return E0M4_ERR_SHAPE;
    if (M == 0 || N == 0) return E0M4_OK;
    if (!Y) return E0M4_ERR_NULL;
    if (!aligned16(Y)) return E0M4_ERR_ALIGN;
    if (K == 0) {
        const int64_t total = M * N;
        hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                           static_cast<half_t*>(Y), total);
        return check_launch();
    }
    if (!X || !codes) return E0M4_ERR_NULL;
    if (!aligned16(X) || !aligned16(codes)) return E0M4_ERR_ALIGN;
    if (e0m8_use_gemv_dq(M, N, K)) {
        if (!e0m8_dq_free(M, N, K)) rc = check_workspace(e0m8_workspace_bytes(M, N, K, group), workspace, workspace_bytes);
        if (rc != E0M4_OK) return rc;
        return launch_gemv_dq(X, M, codes, N, K, 128, kDqFormatE8, Y, (hipStream_t)stream);
    }
    if (e0m8_use_mfma_decode(M, N, K)) return launch_gemv_mfma8(X, M, codes, N, K, Y, (hipStream_t)stream);
    if (small_batch8_in_chunks(Fusion{}, M, N, K))
        return launch_gemv_mfma8(X, M, codes, N, K, Y, (hipStream_t)stream, row_chunks(M));
    if (e0m8_use_gemm(M, N, K)) {
        if (workspace_bytes > 0 && (!workspace || !aligned16(workspace))) return workspace ? E0M4_ERR_ALIGN : E0M4_ERR_NULL;
        return launch_gemm_pipe8(X, M, codes, N, K, Y, workspace, workspace_bytes, (hipStream_t)stream);
    }
    if (M > kGemvMaxM && ((N % 8) != 0)) return E0M4_ERR_SHAPE;    // row chunks of Y must stay 16-byte aligned
    // otherwise up to 8 rows of X per launch of the decode kernel
    for (int64_t m0 = 0; m0 < M; m0 += kGemvMaxM) {
        const int64_t rows = M - m0 < kGemvMaxM ? M - m0 : kGemvMaxM;
        rc = launch_gemv8(static_cast<const half_t*>(X) + m0 * K, rows, codes, N, K, static_cast<half_t*>(Y) + m0 * N,
                          (hipStream_t)stream);
        if (rc != E0M4_OK) return rc;
    }
    return E0M4_OK;
}

// Fused matmul on 8-bit codes (the GEMM kernels need K % 128 == 0).
static FusedPath fused_path8(const Fusion& f, int64_t M, int64_t N, int64_t K)
{
    if (knob(Knob::gemv_mfma) != 1 && gemv_mfma8_fused_supported(f, M, N, K)) return kFusedSmallBatch;
    if (small_batch8_in_chunks(f, M, N, K)) return kFusedChunks;
    if (small_m_on_vector(M, N, K) && gemv_fused_supported(f, M, N, 2 * K)) return kFusedVector;
    if (!gemm_pipe_supported(K) || N > (int64_t)1 << 24) return kFusedNone;
    return as_plain(f) && !gemm_steered() && use_gemv_dq_fused(M, N, K, 128, kDqFormatE8) ? kFusedDq : kFusedGemm;
}

size_t e0m8_fused_workspace_bytes(int64_t M, int64_t N, int64_t K, int group, int with_rmsnorm, int epilogue)
{
    if (check_shape8(N, K, group) != E0M4_OK || M <= 0 || N == 0 || K == 0) return 0;
    if (epilogue != E0M4_EPILOGUE_NONE && epilogue != E0M4_EPILOGUE_SWIGLU) return 0;
    Fusion f;
    f.swiglu = epilogue == E0M4_EPILOGUE_SWIGLU;
    f.residual = &f;                                    // (as in e0m4_fused_workspace_bytes)
    if (fused_path8(f, M, N, K) != kFusedGemm) return 0;
    return (with_rmsnorm ? norm_bytes(M, K) : 0) + gemm_pipe_workspace_bytes(M, N, K, f.swiglu, true);
}

int e0m8_matmul_fused(const void* X, int64_t M, const void* rms_gamma, float rms_eps, const void* codes, int64_t N,
                      int64_t K, int group, int epilogue, const void* residual, void* Y, void* workspace,
                      size_t workspace_bytes, void* stream)
{
    int rc = check_shape8(N, K, group);
    if (rc != E0M4_OK) return rc;
    if (M < 0 || M > (int64_t)1 << 31) return E0M4_ERR_SHAPE;
    if (epilogue != E0M4_EPILOGUE_NONE && epilogue != E0M4_EPILOGUE_SWIGLU) return E0M4_ERR_SHAPE;
    Fusion f;
    f.gamma = rms_gamma;
    f.eps = rms_eps;
    f.residual = residual;
    f.swiglu = epilogue == E0M4_EPILOGUE_SWIGLU;
    if (f.swiglu && (N % (4 * kBlockRows)) != 0) return E0M4_ERR_SHAPE;
    if (M == 0 || N == 0) return E0M4_OK;
    if (K == 0) return E0M4_ERR_SHAPE;
    if (!X || !codes || !Y) return E0M4_ERR_NULL;
    if (!aligned16(X) || !aligned16(codes) || !aligned16(Y) || (rms_gamma && !aligned16(rms_gamma)) ||
        (residual && !aligned16(residual)))
        return E0M4_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const FusedPath path = fused_path8(f, M, N, K);
    if (path == kFusedSmallBatch) return launch_gemv_mfma8_fused(f, X, M, codes, N, K, Y, st);
    if (path == kFusedVector) return launch_gemv8_fused(f, X, M, codes, N, K, Y, st);
    if (path == kFusedChunks) return launch_gemv_mfma8_fused(f, X, M, codes, N, K, Y, st, row_chunks(M));
    if (path == kFusedNone) return E0M4_ERR_SHAPE;      // larger M needs K % 128 == 0 (GEMM kernels)
    const size_t nb = rms_gamma ? norm_bytes(M, K) : 0;
    const size_t need = nb + gemm_pipe_workspace_bytes(M, N, K, f.swiglu, true);
    if (need > 0) {
        if (!workspace) return E0M4_ERR_NULL;
        if (!aligned16(workspace)) return E0M4_ERR_ALIGN;
        if (workspace_bytes < need) return E0M4_ERR_WORKSPACE;
    }
    const void* x = X;
    if (rms_gamma) {
        rc = launch_rmsnorm(X, M, K, rms_gamma, rms_eps, workspace, st);
        if (rc != E0M4_OK) return rc;
        x = workspace;
        f.gamma = nullptr;
    }
    if (path == kFusedDq) return launch_gemv_dq(x, M, codes, N, K, 128, kDqFormatE8, Y, st);
    return launch_gemm_pipe8_fused(f, x, M, codes, N, K, Y, static_cast<char*>(workspace) + nb, workspace_bytes - nb, st);
}

int e0m4_kv_append(void* cache, int64_t max_seq, int64_t row_elems, const void* new_rows, int64_t n_new,
                   int64_t new_ld, const void* position_ids, void* stream)
{
    if (max_seq < 0 || row_elems < 0 || n_new < 0 || (row_elems % 8) != 0 || (new_ld % 8) != 0 || new_ld < row_elems)
        return E0M4_ERR_SHAPE;
    if (row_elems > (int64_t)1 << 31 || max_seq > (int64_t)1 << 40 || n_new > (int64_t)1 << 31) return E0M4_ERR_SHAPE;
    if (n_new == 0 || row_elems == 0 || max_seq == 0) return E0M4_OK;
    if (!cache || !new_rows || !position_ids) return E0M4_ERR_NULL;
    if (!aligned16(cache) || !aligned16(new_rows) || (reinterpret_cast<uintptr_t>(position_ids) & 7u) != 0)
        return E0M4_ERR_ALIGN;
    return launch_kv_append(cache, max_seq, row_elems, new_rows, n_new, new_ld, position_ids, (hipStream_t)stream);
}

}  // extern "C"
