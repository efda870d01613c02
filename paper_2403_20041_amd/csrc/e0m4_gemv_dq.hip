// Small-batch path with the weight operand dequantised in registers: Y[M,N] = X[M,K] * dequant(packed)^T for
// 2 <= M <= 128, any group size, 4-bit codes on fp16 or bfloat16 activations and 8-bit codes on fp16.  Paper: section
// "Operator and lagging optimizations" (vector-matrix product of the decoding stage, bound by memory bandwidth) with
// the dequantisation of section "E0M4 FP4 quantization" fused in registers.
//
// A workgroup of eight wavefronts owns a few consecutive row blocks (16 weight rows) over all of K.  The wavefronts are
// WR groups of WK: a group has up to R of the row blocks, and wavefront number w of a group takes the k blocks w,
// w + WK, ...  Nothing is shared between wavefronts before their sums are added at the end, so the loop over K has no
// barrier: each brings in its own part of X.  MFMA number i of a k block takes word i of every lane's chunk: lane
// (n = l%16, q = l/16) supplies the weights of row n, k = 32q + 8i .. 32q + 8i + 7, dequantised to the bits that the
// dequant entry points produce, and the activations of row l%16 of a tile of 16 rows of X at the same k.  One dequantised
// operand serves MT tiles of X, and one set of activation registers R row blocks.
//
// What bounds it: the weights come from memory and X (2 M K bytes, of which every workgroup needs all) from L2, and what a
// wavefront waits for, dequantises and multiplies does not overlap well with eight wavefronts on a compute unit.  27392 x 4096 at M =
// 45 takes 26 us; without X 24, without X and the dequantisation 23, the weights alone 16.  X as the matrix core takes it, 16 rows
// at a stride of 2 K bytes per load, comes at 13 bytes per clock and compute unit (4096 x 13696 at M = 16: 21.7 us), so whole rows
// of a k block are loaded and turned around in LDS.  From nine rows on they go there without a register in between, one k block
// ahead: 4096 x 4096 at M = 16, 24, 45 and 64 6.7 -> 6.2, 8.6 -> 7.2, 11.1 -> 8.8 and 12.3 -> 10.0 us (bfloat16); two and four k blocks
// of X in flight were 0 - 10 % slower than one, as were three and four of weights.  Up to eight rows, which are one or two loads
// per k block, registers in between are 2 - 8 % faster.  An operand is dequantised by 15 vector instructions (bfloat16: 19), so one
// should serve many rows.
// The GEMM and this kernel at 4096 x 4096, 27392 x 4096, 4096 x 13696 (us): bfloat16 at M = 16 23.5 and 5.7, 28.2 and 19.6, 70 and 13.0;
// groups of 64 at M = 16 10.7 and 5.5, 25.9 and 19.5, 17.9 and 13.2; 8-bit codes at M = 45 13.3 and 10.0, 32.3 and 35.4 (not used), 24.2 and
// 28.1 (gemv_dq_free).
//
// Every weight is rounded to 16 bits before the product, as it is in the GEMM, but in the instances on exact codes (EX below),
// which apply scale and bias in fp32 as e0m4_gemv.hip and e0m4_gemv_mfma.hip do.  Calls of those two go to EX instances only.
#include "e0m4_device.h"
#include "e0m4_host.h"

#include <algorithm>
#include <type_traits>

namespace e0m4 {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kDqWaves = 8;
constexpr int kDqThreads = kDqWaves * 64;
// Row blocks per wavefront, for so many tiles of X: as many as the registers hold (exact codes keep a k block's sums beside the
// others), but not more than five.  Five in place of two groups of wavefronts of three: 20000 x 3072 at M = 32 15.2 -> 14.0 us; seven and
// eight in place of two groups of four 32768 x 2048 17.6 and 21.9.
constexpr int dq_max_r(int MT, bool exact) { return exact ? (MT == 4 ? 3 : 4) : MT == 4 ? 4 : 5; }
// row blocks per workgroup (so that two wavefronts at least share a row block)
constexpr int kDqMaxSlots = 16;
constexpr int kDqMaxM = 64;                     // rows of X per workgroup
constexpr int kDqMaxGroups = 4;                 // of wavefronts with row blocks of their own
constexpr int kDqMaxParts = 2;
constexpr int kTargetWorkgroups = 256;          // one workgroup per compute unit

// k blocks of weights that a wavefront has under way (a round of the loop)
constexpr int dq_weights_ahead(int R) { return R == 1 ? 4 : 2; }

struct DqPlan {
    int64_t grid;
    int rb_base, rb_rem;                        // even deal of row blocks
    int parts;                                  // of the rows of X
    int wr, r;                                  // groups of wavefronts, row blocks per group
};

template <int N, int I = 0, typename F>
__device__ inline void for_each_of(F&& f)               // f(0), ..., f(N - 1), the numbers as constants
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        for_each_of<N, I + 1>(f);
    }
}

__device__ inline half2_t dq_pair(half2_t w1, half2_t bias2, half2_t scale2)
{
    return (w1 - bias2) * scale2;               // difference exact, product rounded once
}

// XE: loads of X per tile and k block.  A load brings a quarter of the tile's rows (8-bit codes: half); calls of up to 4 and 8
// rows make one and two of them, the other rows of the tile stay what LDS held and so do their sums, which nobody stores.
// Groups of 32 at 4096 x 4096: M = 3 6.0 -> 5.3 us with one load for four, M = 8 6.1 -> 5.5 with two.
// EX (4-bit codes, groups of 128, i.e. one group per k block): the codes' exact values 2 + c/8 are multiplied, not rounded
// weights, and scale and bias are applied to the sums of a k block in fp32, as in the kernels of e0m4_gemv.hip and
// e0m4_gemv_mfma.hip.  The sum of a k block's activations that the bias multiplies comes from MFMAs of the same X operands
// with an all-ones weight operand, once for all row blocks.  28 vector instructions per weight operand and 8 per tile of X,
// where the dequantisation takes 60 (bfloat16 76).
template <DqFormat FMT, int MT, int R, int XE, bool EX>
__global__ __launch_bounds__(kDqThreads, 2) void gemv_dq_kernel(const half_t* __restrict__ X, const uint4* __restrict__ packed,
                                                                half_t* __restrict__ Y, int m_total, uint32_t N32, uint32_t K32,
                                                                int rb_base, int rb_rem, int wk_shift, int group_shift)
{
    static_assert(!EX || FMT != kDqFormatE8, "exact codes: 4 bits");
    constexpr int NP = FMT == kDqFormatE8 ? 2 : 4;            // pieces of X (and MFMAs) per k block
    static_assert(XE == NP || (XE < NP && MT == 1), "a part of the rows: of a single tile");
    constexpr int BLK = NP * 32;                        // weights of a row per k block
    constexpr int DW = dq_weights_ahead(R);
    constexpr bool kFew = XE < NP;                      // X through registers, XD k blocks ahead
    constexpr int XD = 2;
    static_assert(DW >= XD, "a round of the loop is DW k blocks");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int64_t N = N32;
    const int K = (int)K32;
    // (more than 64 rows: equal parts of them in the y dimension of the grid)
    const int m_part = (m_total + (int)gridDim.y - 1) / (int)gridDim.y, m0 = (int)blockIdx.y * m_part;
    const int M = min(m_part, m_total - m0);
    X += (int64_t)m0 * K;
    Y += (int64_t)m0 * N;
    const int nkb = (K + BLK - 1) / BLK;
    const int pw = kBlockRows << (7 - group_shift);     // parameter words per k block (8-bit codes: 16)
    const uint32_t rb_stride = (uint32_t)nkb * (uint32_t)(kBlockCodeBytes + 4 * pw);

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n_l = lane & 15, g_l = lane >> 4;         // weight row and chunk of this lane; also (row of X, k-group)
    const int wk_n = 1 << wk_shift;                     // wavefronts per group
    const int wr = wave >> wk_shift, wk = wave & (wk_n - 1);
    const uint32_t fmask = EX && FMT == kDqFormatBf16 ? frac_mask_bf16_vgpr() : frac_mask_vgpr();
    const int64_t rb0 = (int64_t)blockIdx.x * rb_base + min((int)blockIdx.x, rb_rem);
    const int n_rb = rb_base + ((int)blockIdx.x < rb_rem ? 1 : 0);
    const char* wg_base = reinterpret_cast<const char*>(packed) + (size_t)rb0 * rb_stride;
    uint32_t rb_off[R];                                 // this group's row blocks (beyond the last: that one again, its sums are not used)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t s = (uint32_t)min(wr * R + r, n_rb - 1);
        rb_off[r] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(s * rb_stride));
    }
    const uint32_t code_voff = lane * 16;
    const uint32_t param_voff = (uint32_t)nkb * kBlockCodeBytes + 4 * (((g_l * kCodesPerChunk) >> group_shift) * kBlockRows + n_l);
    const uint32_t pb = 4 * pw;
    // X on its way to the matrix core: load number e of a tile brings RPI whole rows of the k block, 16 bytes per lane, to a piece
    // of LDS of the wavefront's own, where lane l's come to lie at 16 l; the wavefront reads them back as operands.  (row, piece)
    // lies at row * RB + 16 * (piece ^ swizzle(row)), by the choice of the piece that a lane loads: the 16 rows of an operand read
    // fall into 16 different bank groups.
    constexpr int PPR = NP * 4, RPI = 64 / PPR, RB = PPR * 16;
    unsigned char* xl = smem + wave * (MT * 16 * RB);
    auto swizzle = [](int row) -> int { return FMT == kDqFormatE8 ? (row >> 1) & 7 : row & 15; };
    // A last k block that K does not fill (groups of 32 and 64): instead of chunks of X that do not exist the block's first
    // is read, and zeroed before use; their codes and parameters are stored as zeros.  (Groups of 128 and blocks of 64 fill every block:
    // without the code for it calls of 3 to 8 rows on rows of up to 1024 weights are 2 % faster.)
    constexpr bool kTail = !EX && FMT != kDqFormatE8;
    const int tail_kb = (K % BLK) != 0 ? nkb - 1 : -1;
    const bool none = (nkb - 1) * BLK + g_l * (NP * 8) >= K;
    uint32_t x_voff[MT][XE], x_back[XE];
    uint32_t x_rd[NP];
#pragma unroll
    for (int e = 0; e < XE; ++e) {
        const int row = e * RPI + lane / PPR, j = (lane % PPR) ^ swizzle(row);
#pragma unroll
        for (int i = 0; i < MT; ++i) x_voff[i][e] = ((uint32_t)min(16 * i + row, M - 1) * K32 + (uint32_t)(j * 8)) * 2;
        x_back[e] = (nkb - 1) * BLK + j * 8 < K ? 0u : (uint32_t)((j / NP) * NP * 16);
    }
#pragma unroll
    for (int e = 0; e < NP; ++e) x_rd[e] = (uint32_t)(n_l * RB + (((g_l * NP + e) ^ swizzle(n_l)) << 4));

    u32x4 c[DW][R];
    uint32_t pwd[DW][R];
    u32x4 xr[kFew ? XD : 1][XE];
    // (a k block beyond the last is requested through a resource of no bytes: zeros, without an access to memory)
    auto load_w = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(wg_base, kb < nkb);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            c[d][r] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)code_voff, (int)(rb_off[r] + (uint32_t)kb * kBlockCodeBytes), 0);
            pwd[d][r] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)param_voff, (int)(rb_off[r] + (uint32_t)kb * pb), 0);
        }
    };
    auto load_x = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(X, kb < nkb);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < XE; ++e) {
                const uint32_t voff = kTail && kb == tail_kb ? x_voff[i][e] - x_back[e] : x_voff[i][e];
                if constexpr (kFew) xr[d][e] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voff, kb * RB, 0);
                else load_to_lds_b128(rsrc, xl + (i * 16 + e * RPI) * RB, voff, (uint32_t)kb * RB);
            }
    };
    // (in the order of use: a wait for one request is a wait for all before it)
#pragma unroll
    for (int d = 0; d < DW; ++d) {
        if (d < (kFew ? XD : 1)) load_x(wk + d * wk_n, d);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        load_w(wk + d * wk_n, d);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }

    // the weight operand of MFMA p: word p of the chunk (8-bit codes: words 2p and 2p + 1)
    auto dequant = [&](const u32x4& cc, uint32_t pw1, int p) -> half8_t {
        if (FMT == kDqFormatBf16) {
            // w1 * scale - bias * scale in one fp32 fused multiply-add per weight (both products and their difference
            // are exact: 5, 4 and 8 significant bits), then the one rounding to bfloat16
            const float sf = __builtin_bit_cast(float, pw1 << 16);
            const float nb = -__builtin_bit_cast(float, pw1 & 0xFFFF0000u) * sf;
            const half2_t q[4] = {w1_pair<0>(cc[p], fmask), w1_pair<1>(cc[p], fmask), w1_pair<2>(cc[p], fmask), w1_pair<3>(cc[p], fmask)};
            bf16x2_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const floatx2 f = {__builtin_fmaf((float)q[e][0], sf, nb), __builtin_fmaf((float)q[e][1], sf, nb)};
                o[e] = __builtin_convertvector(f, bf16x2_t);
            }
            return *reinterpret_cast<const half8_t*>(o);
        }
        const half_t sc = param_scale(pw1), bi = param_bias(pw1);
        const half2_t s2 = {sc, sc}, b2 = {bi, bi};
        half2_t o[4];
        if (FMT == kDqFormatE8) {
            const uint32_t m8 = fmask | (fmask >> 4);   // 0x03FC03FC: eight fraction bits of both halves
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t w8 = cc[2 * (p & 1) + h];
                o[2 * h] = dq_pair(__builtin_bit_cast(half2_t, (w8 & m8) | kExpBits2), b2, s2);
                o[2 * h + 1] = dq_pair(__builtin_bit_cast(half2_t, (__builtin_amdgcn_alignbit(w8, w8, 8) & m8) | kExpBits2), b2, s2);
            }
        } else {
            o[0] = dq_pair(w1_pair<0>(cc[p], fmask), b2, s2);
            o[1] = dq_pair(w1_pair<1>(cc[p], fmask), b2, s2);
            o[2] = dq_pair(w1_pair<2>(cc[p], fmask), b2, s2);
            o[3] = dq_pair(w1_pair<3>(cc[p], fmask), b2, s2);
        }
        return *reinterpret_cast<const half8_t*>(o);
    };

    // word p of the chunk as eight exact code values
    auto codes = [&](const u32x4& cc, int p) -> half8_t {
        uint32_t o[4];
        if (FMT == kDqFormatBf16) {
            o[0] = ((cc[p] >> 3) & fmask) | kExpBits2;
            o[1] = ((cc[p] << 1) & fmask) | kExpBits2;
            o[2] = ((cc[p] >> 7) & fmask) | kExpBits2;
            o[3] = (__builtin_amdgcn_alignbit(cc[p], cc[p], 11) & fmask) | kExpBits2;
        } else {
            o[0] = w1_pair_bits<0>(cc[p], fmask);
            o[1] = w1_pair_bits<1>(cc[p], fmask);
            o[2] = w1_pair_bits<2>(cc[p], fmask);
            o[3] = w1_pair_bits<3>(cc[p], fmask);
        }
        return *reinterpret_cast<const half8_t*>(o);
    };
    auto mfma = [](const half8_t& a, const half8_t& b, const floatx4& v) -> floatx4 {
        if constexpr (FMT == kDqFormatBf16)
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), v, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, v, 0, 0, 0);
    };
    const half_t one = FMT == kDqFormatBf16 ? __builtin_bit_cast(half_t, (uint16_t)0x3F80) : (half_t)1.f;
    const half8_t ones8 = {one, one, one, one, one, one, one, one};

    floatx4 acc[R][MT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[r][i] = floatx4{0.f, 0.f, 0.f, 0.f};

    // One k block (number u of a round).  Its X goes from LDS to registers, whereupon this wavefront's next block's is requested into
    // the same place; its weights' registers are requested again for DW of this wavefront's blocks on.
    // (REST: one of the blocks after the last whole round, whose own requests for weights nobody uses and the compiler may leave out)
    auto block = [&](auto rest_c, int kb, auto u_c) {
        constexpr int u = decltype(u_c)::value;
        if constexpr (kFew) {
#pragma unroll
            for (int e = 0; e < XE; ++e) *reinterpret_cast<u32x4*>(xl + e * (RPI * RB) + lane * 16) = xr[u % XD][e];
            load_x(kb + XD * wk_n, u % XD);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // read back by the wavefront that wrote it
            __builtin_amdgcn_wave_barrier();
        } else {
            // (behind this block's X, requested in the block before, come only that block's weights; behind the first block's all
            // of the prologue's)
            if (u == 0 && kb < wk_n) wait_loads<DW * 2 * R>();
            else wait_loads<(decltype(rest_c)::value && u > 0) ? 0 : 2 * R>();
        }
        half8_t xa[NP][MT];
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int i = 0; i < MT; ++i) xa[p][i] = *reinterpret_cast<const half8_t*>(xl + i * (16 * RB) + x_rd[p]);
        if constexpr (!kFew) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // read before it is written again
            __builtin_amdgcn_sched_barrier(0);
            // (after the last whole round not beyond the last block: also zeros are written to LDS, 128 KB of them by eight wavefronts with
            // four tiles.  4496 x 896 at M = 62 5.6 -> 5.3 us, bfloat16 15280 x 512 at M = 49 6.9 -> 6.1.  Within whole rounds the compiler would
            // wait for all requests where the two ways meet.)
            if (!decltype(rest_c)::value || kb + wk_n < nkb) load_x(kb + wk_n, 0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        if (kTail && kb == tail_kb && none) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int i = 0; i < MT; ++i) xa[p][i] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
        }
        if constexpr (EX) {
            floatx4 sx[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) sx[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int i = 0; i < MT; ++i) sx[i] = mfma(xa[p][i], ones8, sx[i]);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                floatx4 a[MT];
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const half8_t w = codes(c[u % DW][r], p);
#pragma unroll
                    for (int i = 0; i < MT; ++i) a[i] = mfma(xa[p][i], w, p == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : a[i]);
                }
                const uint32_t pw1 = pwd[u % DW][r];
                const float sc = FMT == kDqFormatBf16 ? __builtin_bit_cast(float, pw1 << 16) : (float)param_scale(pw1);
                const float bi = FMT == kDqFormatBf16 ? __builtin_bit_cast(float, pw1 & 0xFFFF0000u) : (float)param_bias(pw1);
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[r][i][e] += sc * (a[i][e] - bi * sx[i][e]);
            }
        } else
#pragma unroll
        for (int p = 0; p < NP; ++p) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const half8_t w = dequant(c[u % DW][r], pwd[u % DW][r], p);
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[r][i] = mfma(xa[p][i], w, acc[r][i]);
            }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        load_w(kb + DW * wk_n, u % DW);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                // X is read before the next block's is written
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);              // (or blocks are mixed, and registers spilled)
    };
    int kb = wk;
    for (; kb + (DW - 1) * wk_n < nkb; kb += DW * wk_n) {
        for_each_of<DW>([&](auto u_c) { block(std::false_type{}, kb + decltype(u_c)::value * wk_n, u_c); });
    }
    for_each_of<DW - 1>([&](auto u_c) {
        if (kb + decltype(u_c)::value * wk_n < nkb) block(std::true_type{}, kb + decltype(u_c)::value * wk_n, u_c);
    });

    // The wavefronts' sums, added in wavefront order: lane l holds rows 4 (l/16) .. + 3 of every tile, weight row l%16
    floatx4* red = reinterpret_cast<floatx4*>(smem);    // [wavefronts][R][MT][64]
    wait_loads<0>();                                    // (what was requested beyond the last block has arrived)
    __syncthreads();                                    // every wavefront has finished with its X
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < MT; ++i) red[((wave * R + r) * MT + i) * 64 + lane] = acc[r][i];
    __syncthreads();
    for (int idx = t; idx < n_rb * MT * 64; idx += kDqThreads) {
        const int s = idx / (MT * 64), i = (idx / 64) % MT, l = idx % 64;
        const floatx4* src = red + ((((s / R) << wk_shift) * R + s % R) * MT + i) * 64 + l;
        floatx4 v = src[0];
        for (int w = 1; w < wk_n; ++w) v += src[w * R * MT * 64];
        const int64_t col = (rb0 + s) * kBlockRows + (l & 15);
        if (col >= N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = 16 * i + 4 * (l >> 4) + e;
            if (m >= M) continue;
            if (FMT == kDqFormatBf16) reinterpret_cast<__bf16*>(Y)[(int64_t)m * N + col] = (__bf16)v[e];
            else Y[(int64_t)m * N + col] = (half_t)v[e];
        }
    }
}

// One workgroup per compute unit where the row blocks allow it (its eight wavefronts fill the unit's registers): with more
// than 256 x 16 of them, as few whole rounds as possible.  (`nkb`: k blocks of a row; without it the plan's size only)
// Rows shorter than a group of wavefronts has members are shared among more groups: 18848 x 512 (five row blocks per workgroup, four k
// blocks) in bfloat16 at M = 45 6.6 us with four of eight wavefronts at work, 5.8 with all; at M = 16 4.8 and 4.1.  (Exact codes of up to
// eight rows not with two row blocks, of which most workgroups then have one: 4816 x 384 at M = 5 3.2 us in one group, 3.4 in two; with X
// straight to LDS, 7888 x 256 at M = 9, 3.8 and 3.6.)
bool make_dq_plan(int64_t M, int64_t N, int64_t K, DqPlan& p, bool exact = false, int64_t nkb = kDqWaves)
{
    if (M < 2 || M > kDqMaxParts * kDqMaxM || N <= 0 || K <= 0) return false;
    p.parts = M > kDqMaxM ? kDqMaxParts : 1;
    const int64_t nrb = row_blocks(N);
    int target = knob(Knob::gemv_workgroups);
    if (target <= 0) target = kTargetWorkgroups;
    const int64_t rounds = (nrb + target * kDqMaxSlots - 1) / (target * kDqMaxSlots);
    const int64_t most = (nrb + target * rounds - 1) / (target * rounds);
    p.grid = (nrb + most - 1) / most;
    p.rb_base = (int)(nrb / p.grid);
    p.rb_rem = (int)(nrb % p.grid);
    p.wr = 1;
    const int max_r = dq_max_r((int)(((M + p.parts - 1) / p.parts + 15) / 16), exact);
    const int fewest = exact && M <= 8 ? 3 : 2;             // row blocks to be shared by groups
    while (p.wr * max_r < most || (most >= fewest && p.wr < kDqMaxGroups && p.wr * 2 <= most && p.wr * 2 * nkb <= kDqWaves)) p.wr *= 2;
    p.r = (int)((most + p.wr - 1) / p.wr);
    return true;
}

template <DqFormat FMT, int MT, int R, int XE, bool EX>
int launch_dq(const DqPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K,
              int group, void* Y, hipStream_t stream)
{
    constexpr int lds = std::max(kDqWaves * R * MT * 64 * 16, kDqWaves * MT * 16 * (FMT == kDqFormatE8 ? 128 : 256));
    static std::atomic<uint64_t> lds_allowed{0};
    const int arc = allow_dynamic_lds(reinterpret_cast<const void*>(&gemv_dq_kernel<FMT, MT, R, XE, EX>), lds, lds_allowed);
    if (arc != E0M4_OK) return arc;
    int wk_shift = 0;                                   // log2 of the wavefronts in a group
    while ((p.wr << (wk_shift + 1)) <= kDqWaves) ++wk_shift;
    const int group_shift = FMT == kDqFormatE8 || group == 128 ? 7 : group == 64 ? 6 : 5;
    hipLaunchKernelGGL((gemv_dq_kernel<FMT, MT, R, XE, EX>), dim3((unsigned)p.grid, (unsigned)p.parts), dim3(kDqThreads), lds, stream,
                       static_cast<const half_t*>(X), static_cast<const uint4*>(packed), static_cast<half_t*>(Y), (int)M,
                       (uint32_t)N, (uint32_t)K, p.rb_base, p.rb_rem, wk_shift, group_shift);
    return check_launch();
}

template <DqFormat FMT, int MT, int R, int XE, bool EX>
int launch_dq_at_r(const DqPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K,
                   int group, void* Y, hipStream_t stream)
{
    if (p.r == R) return launch_dq<FMT, MT, R, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
    if constexpr (R < dq_max_r(MT, EX)) return launch_dq_at_r<FMT, MT, R + 1, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
    return E0M4_ERR_SHAPE;
}

template <DqFormat FMT, int MT, int XE, bool EX>
int launch_dq_r(const DqPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K,
                int group, void* Y, hipStream_t stream)
{
    return launch_dq_at_r<FMT, MT, 1, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
}

template <DqFormat FMT, bool EX = false>
int launch_dq_m(const DqPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K,
                int group, void* Y, hipStream_t stream)
{
    constexpr int XE = FMT == kDqFormatE8 ? 2 : 4;
    // (calls of up to eight rows: fp16 with rounded weights, bfloat16 with exact codes)
    if constexpr (EX == (FMT == kDqFormatBf16) && FMT != kDqFormatE8) {
        if (M <= 4) return launch_dq_r<FMT, 1, 1, EX>(p, X, M, packed, N, K, group, Y, stream);
        if (M <= 8) return launch_dq_r<FMT, 1, 2, EX>(p, X, M, packed, N, K, group, Y, stream);
    }
    if constexpr (!(EX && FMT == kDqFormatBf16)) {
        const int64_t tiles = ((M + p.parts - 1) / p.parts + 15) / 16;
        if constexpr (!EX) {
            if (tiles == 1) return launch_dq_r<FMT, 1, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
        }
        switch (tiles) {
            case 2: return launch_dq_r<FMT, 2, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
            case 3: return launch_dq_r<FMT, 3, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
            case 4: return launch_dq_r<FMT, 4, XE, EX>(p, X, M, packed, N, K, group, Y, stream);
            default: break;
        }
    }
    return E0M4_ERR_SHAPE;
}

}  // namespace


bool gemv_dq_supported(int64_t M, int64_t N, int64_t K, int group)
{
    DqPlan p;
    return (group == 32 || group == 64 || group == 128) && make_dq_plan(M, N, K, p);
}

// Where this kernel is faster than the GEMM, which rounds the weights as it does.  (The callers keep the calls of the kernels
// that multiply unrounded weights away from here, faster or not; the instances on exact codes are chosen below.)  The other
// side's time over this kernel's, with cold weights:
//   bfloat16: up to 64 rows always (1.0 - 5.4: the GEMM has whole tiles only).  65 to 128 rows in two parts, where a workgroup has one
//     row block or two; on 248 calls with one row block and rows of 1024 weights and more 1.0 - 4.5, from 512 on 0.84 - 1.7; with two on
//     4096 and more 1.2 - 1.7, from 1024 on 0.94 - 1.25, from 512 on, since there are 64 x 128 tiles, 0.77 - 0.84 (8192 x 512 at M = 128 6.5
//     us and here 8.3); with more 0.5 - 1.3.  At M = 100 4096 x 4096 24.0 and 17.2, 4096 x 13696 71 and 43, but 32768 x 2048 (8 row blocks)
//     21.6 and 35.4, 27392 x 4096 36 and 56.
//   On the shortest rows most wavefronts have no k block of their own, and many rows of X cost the others time: M = 64, 16384 x
//     128 4.5 us against 5.0; in two parts M = 128, 8192 x 256 5.3 against 7.9.
//   Groups of 32 and 64 up to 16 rows: always (1.3 - 3.1, the vector kernel's calls among them).
//   17 to 64 rows: gemv_dq_beats_gemm, but plain calls within the lines of gemv_dq_free stay here whatever the GEMM has become.
//   (gemv_dq_free: calls that need no workspace.  Callers of the others, up to 64 rows, bring the GEMM's; those lines stay
//   where they are, so that a size that was asked for once is enough for good.)
bool gemv_dq_free(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    if (format == kDqFormatBf16 || M > kDqMaxM) return format == kDqFormatBf16;
    if (M > 16) return (double)N * (double)K <= (format == kDqFormatE8 ? 1e8 : 7e7) && (M <= 48 || (K >= 256 && K <= 9216));
    return format == kDqFormatFp16 && group != 128;
}
// fp16, on 1130 calls with 640 to 260 000 columns and 256 to 14 000 weights a row, by the row blocks that a compute unit has: every
// workgroup reads all of X, and beyond sixteen row blocks of its own the workgroups come in rounds.  The GEMM's time over this kernel's:
//   4-bit codes.  17 to 32 rows: 1.1 - 1.8 up to six row blocks, 1.0 - 1.3 up to twelve, up to 24 on rows of 1024 weights and more 0.97 -
//   1.2; on shorter ones 0.79 - 0.94 (65984 x 512 at M = 22 10.8 and 13.5 us), beyond 24 0.6 - 0.92 (201088 x 384 at M = 22 0.62).
//   33 to 48 rows: 1.0 - 2.0 up to six, 0.84 - 0.93 with seven and eight (the last of two groups of wavefronts is half empty), 1.09 - 1.14
//   with nine and ten, beyond 0.6 - 0.96 (209792 x 1152 at M = 38 48.5 and 71.3).  49 to 64 rows: 1.0 - 1.4 up to four, with three and
//   four on rows of 640 weights and fewer 0.85 - 0.95; 0.75 - 1.25 with five and six (where the GEMM's tiles are just more than the
//   compute units it is the slower one), beyond 0.55 - 1.0 (59328 x 1280 at M = 64 19.3 and 25.6).  The longest rows, of which a workgroup
//   reads all of X: 0.9 - 1.0.
//   8-bit codes.  17 to 32 rows: 0.96 - 1.5 up to twenty, on rows of 384 weights beyond thirteen and on all beyond twenty 0.82 - 1.05; 33 to
//   48: 1.0 - 1.3 up to four, and up to ten on rows of 1024 weights and more, else 0.7 - 0.96; 49 to 64: 1.0 - 1.4 up to four, beyond 0.7 -
//   1.1 (78720 x 1280 at M = 53 31.2 and 40.9).
//   Up to sixteen rows: groups of 32 and 64, up to 60 row blocks (1.04 - 1.9).
bool gemv_dq_beats_gemm(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    DqPlan p;
    if (M < 3 || M > kDqMaxM || !make_dq_plan(M, N, K, p)) return false;
    if (M <= 16) return format == kDqFormatFp16 && group != 128;
    const int64_t rb = (row_blocks(N) + kTargetWorkgroups - 1) / kTargetWorkgroups;
    if (format == kDqFormatE8) {
        if (M <= 32) return rb <= 13 || (rb <= 20 && K >= 512);
        if (M <= 48) return (rb <= 4 || (rb <= 10 && K >= 1024)) && K <= 8192;
        return rb <= 4 && K >= 256 && K <= 6144;
    }
    if (M <= 32) return rb <= 6 || (rb <= 12 && K >= 768) || (rb <= 24 && K >= 1024);
    if (M <= 48) return (rb <= 6 || (rb >= 9 && rb <= 10 && K >= 512)) && K <= 12800;
    return rb <= 4 && K >= (rb <= 2 ? 256 : 768) && K <= 7680;
}
bool gemv_dq_pays(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    DqPlan p;
    if (M < 3 || !make_dq_plan(M, N, K, p)) return false;
    if (format == kDqFormatBf16)
        return M > kGemvMaxM && N <= (int64_t)1 << 24 &&
               (M <= 48 || (M <= kDqMaxM ? K >= 256 : K >= 512 && (double)N * (double)K <= 7e7 && p.wr * p.r <= 2));
    return gemv_dq_free(M, N, K, group, format) || (M > 16 && gemv_dq_beats_gemm(M, N, K, group, format));
}

// (the row counts of the calls below; the kernel is not compiled for others)
bool gemv_exact_supported(int64_t M, int64_t N, int64_t K, int group, DqFormat format)
{
    DqPlan p;
    const bool rows = format == kDqFormatBf16 ? M <= 8 : format == kDqFormatFp16 && M > 16 && M <= kDqMaxM;
    return rows && group == 128 && make_dq_plan(M, N, K, p, true);
}

// Where exact codes are faster than the kernels of unrounded weights that have the call otherwise (us, cold weights, the other and
// this one).  Calls of kernels that round the weights are not taken, though some would gain (27392 x 4096 at M = 24 27.6 and 22.2):
// against the dequantised weights they would be further off.  Plain calls only: a form with fused operators is not built (a
// residual call of 4096 x 4096 at M = 45 would go from 18.9 to 14.3 us).  Errors against float64 on the unrounded weights are those
// of the other kernels (fp16 2.072e-4 on both sides, bfloat16 1.656e-3).
//   bfloat16, 3 to 8 rows: the staging kernel (4608 x 4096 at M = 5 6.0 and 5.8, 4096 x 13696 at M = 8 13.9 and 10.2), but not where
//     row blocks do not fill the wavefronts' (27392 x 4096, seven of eight: 15.1 and 16.0), nor where a wavefront walks three or four
//     row blocks that lie almost a multiple of 16 KiB apart, on the same few memory channels: rows of 1920, 3840, 5760 and 7680
//     weights, 16384 of them at M = 5 7.0 and 7.8, 9.6 and 11.9, 14.0 and 15.1, 17.6 and 19.0 (of 1792 and 2048 6.9 and 6.5, 7.0
//     and 6.75; of 9600 as fast); with three 12288 x 3840 8.3 and 9.4, but x 7680 15.2 and 14.7; with two never slower.
constexpr int64_t kChannelBytes = 16 * 1024;
bool gemv_exact_pays_bf16(int64_t M, int64_t N, int64_t K)
{
    DqPlan p;
    if (M < 3 || !gemv_exact_supported(M, N, K, 128, kDqFormatBf16) || !make_dq_plan(M, N, K, p, true)) return false;
    const int64_t beyond = k_blocks(K) * block_bytes(128) % kChannelBytes, off = std::min(beyond, kChannelBytes - beyond);
    if (p.r >= 3 && off <= 64 * p.r) return false;
    return p.wr * p.r == p.rb_base + (p.rb_rem > 0 ? 1 : 0);
}

//   fp16, 17 to 64 rows: the staging kernel in chunks of equal rows, by the workgroups of all chunks (this kernel's time over its on
//     1 400 calls of 17 to 64 rows, 480 to 9 000 x 1536 to 12 000).
//     More than one row block per workgroup: 0.55 - 0.98 (4608 x 4096 at M = 24 11.6 and 8.9).
//     A compute unit for each workgroup of a chunk: 1.02 - 1.79 (840 x 4096 at M = 59 6.3 and 11.3); but two chunks with five to
//       seven work items for eight wavefronts 0.92 - 0.98 beyond 28 rows and, with most units taken, beyond 24 (1904 x 3328 at M =
//       28 6.4 and 6.0).
//     Two of them on a compute unit at once: with two chunks 0.85 - 0.92, with more 1.04 - 1.17 (1816 x 2688 at M = 35 6.7 and 7.6).
//     Else 0.51 - 1.02 (2376 x 1920 at M = 64 11.0 and 7.3; 1056 x 5120 at M = 49, eight workgroups beyond a round, 1.11), but with four
//       chunks in two rounds whose wavefronts each stage their own X (as many work items as wavefronts) 1.00 - 1.18 (2040 x 4096 at
//       M = 51 9.8 and 11.5).
//     These lines were drawn before X came straight to LDS.  Since then, on 500 calls: more than one row block 0.44 - 1.0, two chunks of
//     more than a round 0.50 - 1.0, three and four of fewer than eight work items 0.41 - 1.0; but of the calls that the lines leave to chunks
//     those of two with a compute unit each take 0.74 - 1.0 (1856 x 4736 at M = 27 8.4 and 6.5), of three 0.83 - 1.2, of four 0.90 - 1.27,
//     and four with eight work items 0.78 - 0.87 (1864 x 4096 at M = 56 11.2 and 8.8).  The lines stand: calls beyond them keep the order
//     of their sums.
bool gemv_exact_pays_chunks(int64_t M, int chunks, const WholeRowsPlan& plan)
{
    if (plan.row_blocks > 1) return true;
    const int64_t wgs = plan.workgroups * chunks;
    if (wgs <= kTargetWorkgroups)
        return chunks == 2 && plan.items > 4 && plan.items < 8 && (M > 28 || (M > 24 && wgs > kTargetWorkgroups * 3 / 4));
    if (chunks == 2) return true;
    if (wgs <= kTargetWorkgroups * plan.resident) return false;
    return !(chunks == 4 && plan.x_in_registers && plan.items == plan.waves && wgs <= 2 * kTargetWorkgroups);
}

int launch_gemv_exact(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, DqFormat format, void* Y, hipStream_t stream)
{
    DqPlan p;
    if (!gemv_exact_supported(M, N, K, 128, format) || !make_dq_plan(M, N, K, p, true, k_blocks(K))) return E0M4_ERR_SHAPE;
    if (format == kDqFormatBf16) return launch_dq_m<kDqFormatBf16, true>(p, X, M, packed, N, K, 128, Y, stream);
    return launch_dq_m<kDqFormatFp16, true>(p, X, M, packed, N, K, 128, Y, stream);
}

int launch_gemv_dq(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, DqFormat format, void* Y,
                   hipStream_t stream)
{
    DqPlan p;
    const int64_t nkb = k_blocks(format == kDqFormatE8 ? 2 * K : K);
    if (!gemv_dq_supported(M, N, K, group) || !make_dq_plan(M, N, K, p, false, nkb)) return E0M4_ERR_SHAPE;
    switch (format) {
        case kDqFormatBf16: return launch_dq_m<kDqFormatBf16>(p, X, M, packed, N, K, group, Y, stream);
        case kDqFormatE8: return launch_dq_m<kDqFormatE8>(p, X, M, packed, N, K, group, Y, stream);
        default: return launch_dq_m<kDqFormatFp16>(p, X, M, packed, N, K, group, Y, stream);
    }
}

}  // namespace e0m4
