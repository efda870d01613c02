// Fused calls of 17 to 64 rows in groups of 128: Y = epilogue(X * dequant(packed)^T) with the gated product and the residual of
// e0m4_matmul_fused, X normalised before.  Paper: section "Operator and lagging optimizations" (vector-matrix product with its
// element-wise neighbours fused) with the dequantisation of section "E0M4 FP4 quantization" fused in registers.
//
// The same products and sums, in the same order, as gemv_mfma_kernel (e0m4_gemv_mfma.hip) on chunks of sixteen rows, to the bit:
// exact code values on v_mfma_f32_16x16x32_f16 with the two kinds of code pairs apart, the group's affine map per k block, a
// running sum per wavefront of that kernel over its work items of four k blocks, the wavefronts' sums added in their order.  There a
// chunk is a workgroup of its own (in y), stages its X behind a barrier and forms the weight operands for itself; here a workgroup
// owns its row blocks for all rows, each operand serves MT tiles of X, and X comes block by block as in gemv_dq_kernel
// (e0m4_gemv_dq.hip): whole rows of a k block straight to a piece of LDS of the wavefront's own, one block ahead.  An rms-norm is a
// launch before this one, with as many threads per row as that kernel has, whose order of sums it keeps.
//
// What bounds it: X from L2 and the start of a launch (4096 x 4096 at M = 45: 256 workgroups read 369 KB of X each for 35 KB of
// weights).  Chunks and this kernel with its norm (us): 4608 x 4096 with norm at M = 45 20.8 -> 13.4, 4096 x 4096 with a residual
// 16.5 -> 9.7, gated 22016 x 3072 with norm at M = 30 32.2 -> 19.2.  Where it is not the faster one: gemv_tiles_pays.
#include "e0m4_device.h"
#include "e0m4_host.h"

#include <algorithm>

namespace e0m4 {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileWaves = 8;
constexpr int kTileThreads = kTileWaves * 64;
constexpr int kTileBlocks = 4;                  // k blocks of 128 per work item
constexpr int kTileXBytes = 16 * kBlockK * 2;   // sixteen rows of a k block
constexpr int kMaxTiles = 4;
constexpr int max_slots(int MT) { return MT == 2 ? 8 : MT == 3 ? 4 : 3; }       // row blocks of a workgroup (registers)

// MT: tiles of sixteen rows.  R: row blocks per workgroup.  inner, outer: 30 and 1 where the other kernel keeps the activations'
// operands and sums in registers, and 30 times a sum is rounded before it is subtracted; 1 and 30 where it is not (one fused
// multiply-add with the sum).
template <int MT, int R>
__global__ __launch_bounds__(kTileThreads, 2) void gemv_tiles_kernel(const half_t* __restrict__ X, const uint4* __restrict__ packed,
                                                                     half_t* Y, const half_t* residual, int M, uint32_t N32,
                                                                     uint32_t K32, int rb_base, int rb_rem, uint32_t half_bytes,
                                                                     float outer, float inner)
{
    constexpr int DW = 2;                               // k blocks of weights under way
    constexpr int ROWB = kBlockK * 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const bool gated = half_bytes != 0;
    const int64_t n_out = gated ? N32 / 2 : N32;
    const int nkb = (int)(K32 / kBlockK), items = (nkb + kTileBlocks - 1) / kTileBlocks;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n_l = lane & 15, g_l = lane >> 4;         // weight row and chunk of this lane; also (row of X, k-group)
    const uint32_t fmask = frac_mask_vgpr(), fmask_low = frac_mask_low_vgpr();
    const uint32_t rb_stride = (uint32_t)nkb * block_bytes(128);
    const int64_t rb0 = (int64_t)blockIdx.x * rb_base + min((int)blockIdx.x, rb_rem);
    const int n_rb = (rb_base + ((int)blockIdx.x < rb_rem ? 1 : 0)) << (gated ? 1 : 0);     // (the deal is of pairs)
    const char* base = reinterpret_cast<const char*>(packed) + (size_t)rb0 * rb_stride;
    uint32_t rb_off[R];                                 // (beyond the last: that one again, its sums are not used)
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const uint32_t sl = (uint32_t)min(s, n_rb - 1);
        rb_off[s] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(gated ? (sl >> 1) * rb_stride + (sl & 1) * half_bytes : sl * rb_stride));
    }
    const uint32_t param_voff = (uint32_t)nkb * kBlockCodeBytes + 4 * n_l;

    // X: load number e of a tile brings rows 4 e .. 4 e + 3 of the k block; lane l's 16 bytes come to lie at 16 l.  Piece p of a row
    // is at 16 (p ^ row): the sixteen rows of an operand read fall into sixteen different bank groups.
    unsigned char* xl = smem + wave * (MT * kTileXBytes);
    uint32_t x_voff[MT][4], x_rd[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = 4 * e + (lane >> 4), piece = (lane & 15) ^ row;
#pragma unroll
        for (int i = 0; i < MT; ++i) x_voff[i][e] = ((uint32_t)min(16 * i + row, M - 1) * K32 + (uint32_t)(piece * 8)) * 2;
        x_rd[e] = (uint32_t)(n_l * ROWB + (((g_l * 4 + e) ^ n_l) << 4));
    }
    // (a k block beyond the last is requested through a resource of no bytes: zeros, without an access to memory)
    u32x4 c[DW][R];
    uint32_t pw[DW][R];
    auto load_w = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(base, kb < nkb);
#pragma unroll
        for (int s = 0; s < R; ++s) {
            c[d][s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, (int)(rb_off[s] + (uint32_t)kb * kBlockCodeBytes), 0);
            pw[d][s] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)param_voff, (int)(rb_off[s] + (uint32_t)kb * (4 * kBlockRows)), 0);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load_x = [&](int kb) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(X, kb < nkb);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) load_to_lds_b128(rsrc, xl + (i * 4 + e) * 1024, x_voff[i][e], (uint32_t)kb * ROWB);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // (in the order of use: a wait for one request is a wait for all before it)
    load_x(wave * kTileBlocks);
    load_w(wave * kTileBlocks, 0);
    load_w(wave * kTileBlocks + 1, 1);

    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    const half_t one = (half_t)1.f;
    const half8_t ones8 = {one, one, one, one, one, one, one, one};
    auto mfma = [](const half8_t& a, const half8_t& b, const floatx4& v) -> floatx4 {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, v, 0, 0, 0);
    };
    floatx4 ysum[R][MT];
#pragma unroll
    for (int s = 0; s < R; ++s)
#pragma unroll
        for (int i = 0; i < MT; ++i) ysum[s][i] = zero4;
    for (int item = wave; item < items; item += kTileWaves) {
        const int on = item + kTileWaves;               // this wavefront's next work item
#pragma unroll
        for (int j = 0; j < kTileBlocks; ++j) {
            const int kb = item * kTileBlocks + j, d = j % DW;
            // (behind this block's X, requested in the block before, come only that block's weights)
            wait_loads<2 * R>();
            half8_t xh[2][MT], xs[2][MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                half8_t v[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) v[w] = *reinterpret_cast<const half8_t*>(xl + i * kTileXBytes + x_rd[w]);
#pragma unroll
                for (int wp = 0; wp < 2; ++wp) {
                    const half8_t a = v[2 * wp], b = v[2 * wp + 1];
                    xh[wp][i] = half8_t{a[0], a[1], a[6], a[7], b[0], b[1], b[6], b[7]};
                    xs[wp][i] = half8_t{a[2], a[3], a[4], a[5], b[2], b[3], b[4], b[5]};
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // read before it is written again
            __builtin_amdgcn_sched_barrier(0);
            load_x(j + 1 < kTileBlocks ? kb + 1 : on * kTileBlocks);
            if (kb < nkb) {                             // (the last item may reach beyond K)
                floatx4 sx[MT], sx30[MT];               // (the second times `outer`)
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    floatx4 sh = zero4, sl = zero4;
#pragma unroll
                    for (int wp = 0; wp < 2; ++wp) {
                        sh = mfma(xh[wp][i], ones8, sh);
                        sl = mfma(xs[wp][i], ones8, sl);
                    }
                    sx[i] = sh + sl;
                    sx30[i] = inner * sl;
                }
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    half2_t p[4][4];
#pragma unroll
                    for (int w = 0; w < 4; ++w) w1_pairs_mixed(c[d][s][w], fmask, fmask_low, p[w]);
                    const float sc = (float)param_scale(pw[d][s]);
                    const float bi = (float)param_bias(pw[d][s]);
                    floatx4 acc_h[MT], acc_l[MT];
#pragma unroll
                    for (int wp = 0; wp < 2; ++wp) {
                        const half2_t* w0 = p[2 * wp];
                        const half2_t* w1 = p[2 * wp + 1];
                        const half8_t wh = {w0[0][0], w0[0][1], w0[3][0], w0[3][1], w1[0][0], w1[0][1], w1[3][0], w1[3][1]};
                        const half8_t wl = {w0[1][0], w0[1][1], w0[2][0], w0[2][1], w1[1][0], w1[1][1], w1[2][0], w1[2][1]};
#pragma unroll
                        for (int i = 0; i < MT; ++i) {
                            acc_h[i] = mfma(xh[wp][i], wh, wp == 0 ? zero4 : acc_h[i]);
                            acc_l[i] = mfma(xs[wp][i], wl, wp == 0 ? zero4 : acc_l[i]);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float a = __builtin_fmaf(16.f, acc_l[i][r], acc_h[i][r]);
                            a = __builtin_fmaf(-outer, sx30[i][r], a);
                            a = __builtin_fmaf(-bi, sx[i][r], a);
                            ysum[s][i][r] = __builtin_fmaf(sc, a, ysum[s][i][r]);
                        }
                }
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            load_w(j + DW < kTileBlocks ? kb + DW : on * kTileBlocks + j + DW - kTileBlocks, d);
        }
    }

    // The sums of the order's wavefronts in their order: the work items i of row block s that wavefront v has there are those with
    // (s * items + i) % 8 = v; here they are wavefront (v - s * items) % 8's.
    floatx4* red = reinterpret_cast<floatx4*>(smem);    // [wavefronts][R][MT][64]
    wait_loads<0>();                                    // (what was requested beyond the last block has arrived)
    __syncthreads();                                    // every wavefront has finished with its X
#pragma unroll
    for (int s = 0; s < R; ++s)
#pragma unroll
        for (int i = 0; i < MT; ++i) red[((wave * R + s) * MT + i) * 64 + lane] = ysum[s][i];
    __syncthreads();
    auto sum_of = [&](int sl, int i, int l) -> floatx4 {
        floatx4 y = zero4;
#pragma unroll
        for (int v = 0; v < kTileWaves; ++v) y += red[((((v - sl * items) & (kTileWaves - 1)) * R + sl) * MT + i) * 64 + l];
        return y;
    };
    const int units = n_rb >> (gated ? 1 : 0);
    for (int idx = t; idx < units * MT * 64; idx += kTileThreads) {
        const int u = idx / (MT * 64), i = (idx / 64) % MT, l = idx % 64;
        const int64_t col = (rb0 + u) * kBlockRows + (l & 15);
        floatx4 y = sum_of(gated ? 2 * u : u, i, l);
        if (gated) {
            const floatx4 up = sum_of(2 * u + 1, i, l);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = silu_f32(y[e]) * up[e];
        }
        if (col >= n_out) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = 16 * i + 4 * (l >> 4) + e;
            if (m >= M) continue;
            if (residual) y[e] += (float)residual[(int64_t)m * n_out + col];
            Y[(int64_t)m * n_out + col] = (half_t)y[e];
        }
    }
}

template <int MT, int R>
int launch_tiles(const Fusion& f, const TilesPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                 hipStream_t stream)
{
    constexpr int lds = std::max(kTileWaves * MT * kTileXBytes, kTileWaves * R * MT * 1024);
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    static std::atomic<uint64_t> lds_allowed{0};
    const int arc = allow_dynamic_lds(reinterpret_cast<const void*>(&gemv_tiles_kernel<MT, R>), lds, lds_allowed);
    if (arc != E0M4_OK) return arc;
    hipLaunchKernelGGL((gemv_tiles_kernel<MT, R>), dim3((unsigned)p.grid), dim3(kTileThreads), lds, stream,
                       static_cast<const half_t*>(X), static_cast<const uint4*>(packed), static_cast<half_t*>(Y),
                       static_cast<const half_t*>(f.residual), (int)M, (uint32_t)N, (uint32_t)K, p.rb_base, p.rb_rem,
                       f.swiglu ? (uint32_t)gated_half_bytes(N, K, 128) : 0u, p.x_in_registers ? 1.f : 30.f,
                       p.x_in_registers ? 30.f : 1.f);
    return check_launch();
}

template <int MT, int R = 1>
int launch_tiles_m(const Fusion& f, const TilesPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                   hipStream_t stream)
{
    if (p.slots == R) return launch_tiles<MT, R>(f, p, X, M, packed, N, K, Y, stream);
    if constexpr (R < max_slots(MT)) return launch_tiles_m<MT, R + 1>(f, p, X, M, packed, N, K, Y, stream);
    return E0M4_ERR_SHAPE;
}

}  // namespace

// (the plan is that of a chunk in e0m4_gemv_mfma.hip)
bool gemv_tiles_supported(const TilesPlan& p, int64_t M, int64_t K)
{
    if (M <= 16 || M > 16 * kMaxTiles || K <= 0 || K % kBlockK != 0 || p.rb_base < 1) return false;
    return p.waves == kTileWaves && p.slots <= max_slots((int)((M + 15) / 16));
}

// Where it is faster than chunks, on 800 calls of 64 to 20 000 columns: 1.15 - 2.4 where chunks need more than a compute unit each.
// Else, with an rms-norm, which they do in every workgroup: two chunks 1.03 - 1.6 and, without the gated product, three 1.0 - 1.3, but
// three with eight work items to a row, of which each of the chunk kernel's wavefronts has one, 0.93 - 0.96 (192 x 3968 at M = 36 9.1 and 9.7
// us), four 0.89 - 1.02 (384 x 2816 at M = 51 9.8 and 10.6 us) and three with the gated product 0.86 - 1.04.  With the gated product
// alone two chunks 1.0 - 1.22, but 0.83 - 0.99 with eight work items (2944 x 3968 at M = 22 7.2 and 7.9), 0.94 - 1.02 on rows of one or
// two, 0.96 - 0.98 on rows of four in sixteen workgroups, and 0.88 - 1.09 at 17 to 20 rows of up to seven (512 x 3072 at M = 17 6.1 and 6.9);
// with a residual alone 0.66 - 1.03 (960 x 2176 at M = 37 5.5 and 6.2).
bool gemv_tiles_pays(const Fusion& f, const TilesPlan& p, int64_t M, int chunks)
{
    if (p.grid * chunks > 256) return true;
    if (f.gamma) return chunks == 2 || (chunks == 3 && !f.swiglu && p.items != kTileWaves);
    return f.swiglu && chunks == 2 && (p.items > kTileWaves || (p.items >= 4 && p.items < kTileWaves && M > 20 && (p.items > 4 || p.grid > 16)));
}

int launch_gemv_tiles(const Fusion& f, const TilesPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                      hipStream_t stream)
{
    if (!gemv_tiles_supported(p, M, K)) return E0M4_ERR_SHAPE;
    switch ((M + 15) / 16) {
        case 2: return launch_tiles_m<2>(f, p, X, M, packed, N, K, Y, stream);
        case 3: return launch_tiles_m<3>(f, p, X, M, packed, N, K, Y, stream);
        default: return launch_tiles_m<4>(f, p, X, M, packed, N, K, Y, stream);
    }
}

}  // namespace e0m4
