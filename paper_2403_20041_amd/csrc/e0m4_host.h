// Host-side internals of libe0m4: launcher prototypes shared between the C-ABI
// file and the kernel files.  Not installed; the public interface is e0m4.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "e0m4.h"

namespace e0m4 {

// Records hipGetLastError(); returns E0M4_OK or E0M4_ERR_HIP.
int check_launch();
int record_hip_error(hipError_t e);

// Raises a kernel's dynamic LDS limit, once per device (it is an attribute of the function on the current
// device).  `done` is the caller's own mask of devices that have it; safe to call from several threads.
inline int allow_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return record_hip_error(e);
    const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;        // devices beyond 64 are not remembered
    if (done.load(std::memory_order_acquire) & bit) return E0M4_OK;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return record_hip_error(e);
    done.fetch_or(bit, std::memory_order_release);
    return E0M4_OK;
}

// Tuning knobs of the calling thread (0 = use the heuristic), by index: a plan asks for dozens of them, and compared by name they
// were half of its time.  Names and meanings stand at kKnobNames.
enum class Knob { gemv_waves, gemv_workgroups, gemv_mfma, gemv_xreg, gemm_variant, gemm_splits, gemm_sk, gemm_panel, gemm_split_order, count };
extern __thread int g_knobs[(int)Knob::count];
inline int knob(Knob k) { return g_knobs[(int)k]; }

// Operators folded into a matmul (e0m4_matmul_fused).  All-zero is the plain matmul.
struct Fusion {
    const void* gamma = nullptr;        // [K] fp16 rms-norm weight applied to the rows of X, or null
    float eps = 0.f;                    // rms-norm epsilon
    const void* residual = nullptr;     // [M, N_out] fp16 added to the result, or null
    bool swiglu = false;                // Y[m, j] = silu(a[m, j]) * a[m, N/2 + j], N_out = N/2
    bool any() const { return gamma || residual || swiglu; }
};

struct GemvFusion;
// Device view of `f` for the decode kernels (defined in e0m4_gemv.hip).
GemvFusion make_gemv_fusion(const Fusion& f, int64_t N, int64_t K, int group);

// `format`: 0 E0M4, 1 the INT4 comparison format, 2 E0M3 (codes stored as the E0M4 codes of the same values),
// 3 E0M4 on bfloat16 (W, scales and bias are bfloat16 bit patterns).
enum { kFormatE0M4 = 0, kFormatInt4 = 1, kFormatE0M3 = 2, kFormatBf16 = 3 };
int launch_quantize(const void* W, int64_t N, int64_t K, int group, void* packed, void* scales, void* bias,
                    const void* scales_in, const void* bias_in, bool fit, int format, hipStream_t stream);
int launch_dequant(const void* packed, int64_t N, int64_t K, int group, void* W_out, int format, hipStream_t stream);
// codes_u8[n,k] = stored 4-bit code >> shift (shift 1 for 3-bit codes, which are stored doubled)
int launch_unpack(const void* packed, int64_t N, int64_t K, int group, void* out, hipStream_t stream, int shift = 0);

// Small-M path (M <= kGemvMaxM).
constexpr int kGemvMaxM = 8;
int launch_gemv(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                hipStream_t stream);
// With fused operators.  gemv_fused_supported: false when the gated epilogue meets activations that do
// not fit the LDS in one piece (the caller then takes the GEMM path).
bool gemv_fused_supported(const Fusion& f, int64_t M, int64_t N, int64_t K);
int launch_gemv_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group,
                      void* Y, hipStream_t stream);
// Small-batch path on the matrix cores: 2 <= M <= 16 at group 128, 8 at group 64, 4 at group 32.
bool gemv_mfma_supported(int64_t M, int64_t N, int64_t K, int group);
// ... and, for groups of 64 and 32, whether the plain matmul takes it rather than the kernel with dequantised operands
bool gemv_mfma_groups_pay(int64_t M, int64_t N, int64_t K, int group);
// `chunks` > 1: M (17 ... 64) rows in that many equal chunks of at most 16 rows, dealt to the y dimension of one launch
int launch_gemv_mfma(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y, hipStream_t stream,
                     int chunks = 1, int group = 128);
// 4-bit codes on bfloat16, the same sizes
int launch_gemv_mfma_bf16(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y, hipStream_t stream);
bool gemv_mfma_fused_supported(const Fusion& f, int64_t M, int64_t N, int64_t K, int group);
// ... and all M rows of X fit the LDS at once (no phases along K)
struct WholeRowsPlan {
    int64_t workgroups;
    int row_blocks;                                     // of a workgroup (pairs of them with the gated product), at most
    int resident;                                       // workgroups of a plain call that a compute unit holds at once
    int items, waves;                                   // work items per row block
    bool x_in_registers;
};
bool gemv_mfma_whole_rows(const Fusion& f, int64_t M, int64_t N, int64_t K, int group, WholeRowsPlan* plan = nullptr);
bool gemv_mfma8_whole_rows(const Fusion& f, int64_t M, int64_t N, int64_t K);
int launch_gemv_mfma_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                           hipStream_t stream, int chunks = 1, int group = 128);
// Its plain and residual calls with one or two row blocks per workgroup, where X block by block is the faster way, to the same bits
// (e0m4_gemv_items.hip).  The plan is that kernel's: wavefronts and work items per phase give the order of the sums.
struct ItemsPlan {
    int64_t grid;
    int rb_base, rb_rem;
    int waves, items_ph;
    bool phased;                                        // X does not fit that kernel's LDS at once
    bool e8;                                            // 8-bit codes (group 128, K in 4-bit slots, two per code)
};
bool gemv_items_supported(const ItemsPlan& p, int64_t M, int64_t N, int64_t K, int group);
bool gemv_items_pays(const ItemsPlan& p, int64_t M, int group, bool fused);
int launch_gemv_items(const ItemsPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                      const void* residual, hipStream_t stream);
// Fused calls of 17 to 64 rows with all rows in a workgroup, to the bits of that kernel on chunks of rows (e0m4_gemv_tiles.hip).
struct TilesPlan {
    int64_t grid;
    int rb_base, rb_rem;                                // even deal of row blocks, or of pairs
    int slots, waves, items;                            // row blocks of a workgroup, at most; wavefronts and work items of the order
    bool x_in_registers;                                // in that kernel
};
bool gemv_tiles_plan(const Fusion& f, int64_t M, int chunks, int64_t N, int64_t K, TilesPlan* plan);
bool gemv_tiles_supported(const TilesPlan& p, int64_t M, int64_t K);
bool gemv_tiles_pays(const Fusion& f, const TilesPlan& p, int64_t M, int chunks);
int launch_gemv_tiles(const Fusion& f, const TilesPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                      hipStream_t stream);
// Small-batch path with the weight operand dequantised in registers: 2 <= M <= 128, any group (e0m4_gemv_dq.hip).
// (`beats_gemm`: it is expected to be the faster one; `free`: plain calls that need no workspace, the others as much as the GEMM;
// `pays`: plain calls that it has)
enum DqFormat { kDqFormatFp16 = 0, kDqFormatE8 = 1, kDqFormatBf16 = 2 };     // 4-bit codes, 8-bit codes, 4-bit codes on bfloat16
bool gemv_dq_supported(int64_t M, int64_t N, int64_t K, int group);
bool gemv_dq_pays(int64_t M, int64_t N, int64_t K, int group, DqFormat format);
bool gemv_dq_beats_gemm(int64_t M, int64_t N, int64_t K, int group, DqFormat format);
bool gemv_dq_free(int64_t M, int64_t N, int64_t K, int group, DqFormat format);
int launch_gemv_dq(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, DqFormat format, void* Y,
                   hipStream_t stream);
// The same kernel on exact code values (4-bit codes, groups of 128; bfloat16 of up to 8 rows, fp16 of 17 to 64).
// (`pays`: it is expected to beat the kernels that have the call otherwise: the small-batch kernel, fp16 in `chunks` launches of
// `plan` side by side)
bool gemv_exact_supported(int64_t M, int64_t N, int64_t K, int group, DqFormat format);
bool gemv_exact_pays_bf16(int64_t M, int64_t N, int64_t K);
bool gemv_exact_pays_chunks(int64_t M, int chunks, const WholeRowsPlan& plan);
int launch_gemv_exact(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, DqFormat format, void* Y, hipStream_t stream);
// INT4 twin of the M = 1 kernel: same layout and work decomposition, codes turned into numbers with
// integer-to-float conversion instructions.
int launch_gemv_int4(const void* X, const void* packed, int64_t N, int64_t K, int group, void* Y, hipStream_t stream);

// E0M4 on bfloat16: decode kernel (M <= 8) and small-tile MFMA kernel (any M); no workspace.
int launch_gemv_bf16(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                     hipStream_t stream);
int launch_gemm_bf16(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                     hipStream_t stream);

// MFMA path.
int launch_gemm(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                void* workspace, size_t workspace_bytes, hipStream_t stream);
size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K, bool swiglu = false, bool fused = false);
// The same with the epilogue operators of `f` (residual add, gated product of the two halves of N);
// rms-norm is not applied here: X must already be normalised.
int launch_gemm_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group,
                      void* Y, void* workspace, size_t workspace_bytes, hipStream_t stream);
int launch_gemm_pipe_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group,
                           void* Y, void* workspace, size_t workspace_bytes, hipStream_t stream);
// Row-wise rms-norm of X [M, K] into X_out (fp16): the prologue of e0m4_matmul_fused for the GEMM path.
// (`waves` per row, which give the order of its sum of squares: 4 or 8)
int launch_rmsnorm(const void* X, int64_t M, int64_t K, const void* gamma, float eps, void* X_out, hipStream_t stream, int waves = 4);
// Software-pipelined 256 x 256 tile kernel (needs K % 128 == 0).  Problems with too few tiles to
// fill the chip are split along K; the fp32 partial sums ([splits][M][N]) live in the caller's
// workspace of gemm_pipe_workspace_bytes() bytes and a second kernel adds them.
bool gemm_pipe_supported(int64_t K);
size_t gemm_pipe_workspace_bytes(int64_t M, int64_t N, int64_t K, bool swiglu = false, bool fused = false);
int launch_gemm_pipe(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                     void* workspace, size_t workspace_bytes, hipStream_t stream);
// The bfloat16 member on the same kernel, whole tiles only (no workspace); `pays`: enough tiles to fill the chip that way.
bool gemm_pipe_bf16_pays(int64_t M, int64_t N, int64_t K);
int launch_gemm_pipe_bf16(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                          hipStream_t stream);

// 8-bit format (E0M8): offline side and decode kernel.
int launch_quantize8(const void* W, int64_t N, int64_t K, int group, void* packed, void* scales, void* bias,
                     hipStream_t stream);
int launch_dequant8(const void* packed, int64_t N, int64_t K, void* W_out, void* codes_out, hipStream_t stream);
int launch_gemm_pipe8(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y, void* workspace,
                      size_t workspace_bytes, hipStream_t stream);
bool gemv_mfma8_supported(int64_t M, int64_t N, int64_t K);
int launch_gemv_mfma8(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y, hipStream_t stream,
                      int chunks = 1);
int launch_gemv8_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                       hipStream_t stream);
bool gemv_mfma8_fused_supported(const Fusion& f, int64_t M, int64_t N, int64_t K);
int launch_gemv_mfma8_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                            hipStream_t stream, int chunks = 1);
int launch_gemm_pipe8_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                            void* workspace, size_t workspace_bytes, hipStream_t stream);
int launch_gemv8(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y, hipStream_t stream);

// In-place KV-cache append: cache[position_ids[i], :] = src[i, :row_elems], src rows src_ld elements apart.
int launch_kv_append(void* cache, int64_t max_seq, int64_t row_elems, const void* src, int64_t n_new, int64_t src_ld,
                     const void* position_ids, hipStream_t stream);

}  // namespace e0m4
