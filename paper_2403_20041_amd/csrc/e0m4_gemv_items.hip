// Small batch on long rows: Y[M,N] = X[M,K] * dequant(packed)^T (+ residual) for 2 <= M <= 16, groups of 128, where M rows of X
// exceed the LDS and every workgroup has one row block (16 weight rows).  Paper: section "Operator and lagging optimizations"
// (vector-matrix product of the decoding stage, bound by memory bandwidth) with the dequantisation of section "E0M4 FP4
// quantization" fused in registers.
//
// The same products and sums, in the same order, as gemv_mfma_kernel (e0m4_gemv_mfma.hip) walking K in phases, to the bit:
// exact code values on v_mfma_f32_16x16x32_f16 with the two kinds of code pairs apart, the group's affine map per k block, one
// sum per work item of four k blocks; the items of one place in all phases are added first, then the places.  What differs is
// how X comes in.  There a phase stages 128 KiB of X behind two barriers, with half of the wavefronts idle, since a phase is
// eight items long and there are sixteen of them.  Here nothing is shared before the end and no barrier stands in the loop: a
// wavefront takes the items w, w + 8, ..., loads the rows of X of its own k blocks two ahead and turns them into operand order
// in a piece of LDS of its own, and parks an item's sums in LDS.
//
// What bounds it: X from L2 (every workgroup needs all 2 M K bytes: at M = 16 512 KiB for 136 KiB of weights).  With a
// residual, in phases and here (us): 2048 x 16384 at M = 16 19.8 -> 11.6, at M = 6 13.1 -> 9.5; 4096 x 13696 20.2 -> 14.5 and
// 14.7 -> 11.1; 4096 x 24576 30.0 -> 22.7 and, at M = 8, 22.0 -> 17.1.
#include "e0m4_device.h"
#include "e0m4_host.h"

#include <algorithm>

namespace e0m4 {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kItemWaves = 8;
constexpr int kItemThreads = kItemWaves * 64;
constexpr int kItemBlocks = 4;                  // k blocks of 128 per work item
constexpr int kMaxItems = 96;                   // their sums (1 KiB each) and the wavefronts' X (4 KiB each) share the LDS
constexpr int kItemXBytes = 16 * kBlockK * 2;   // sixteen rows of a k block

// XE: loads of X per k block, four rows each (calls of up to 4 and 8 rows make one and two; the other rows of the tile stay
// what LDS held, and so do their sums, which nobody stores)
template <int XE>
__global__ __launch_bounds__(kItemThreads, 2) void gemv_items_kernel(const half_t* __restrict__ X, const uint4* __restrict__ packed,
                                                                     half_t* __restrict__ Y, const half_t* __restrict__ residual,
                                                                     int M, uint32_t N32, uint32_t K32, int items_ph)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int64_t N = N32;
    const int nkb = (int)(K32 / kBlockK), items = (nkb + kItemBlocks - 1) / kItemBlocks;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n_l = lane & 15, g_l = lane >> 4;         // weight row and chunk of this lane; also (row of X, k-group)
    const uint32_t fmask = frac_mask_vgpr(), fmask_low = frac_mask_low_vgpr();
    unsigned char* xl = smem + wave * kItemXBytes;
    float* red = reinterpret_cast<float*>(smem + kItemWaves * kItemXBytes);     // [items][16 m][16 n]
    const char* base = reinterpret_cast<const char*>(packed) + (size_t)blockIdx.x * ((size_t)nkb * block_bytes(128));

    // X: load number e brings rows 4 e .. 4 e + 3 of the k block, 16 bytes per lane.  A piece of eight activations (of one code
    // word) is two halves, those of the pairs that read 2 + c/8 and those that read 2 + c/128; unit u = 4 q + 2 (w / 2) + half
    // of a row lies at 16 (u ^ row): the sixteen rows of an operand read fall into sixteen different bank groups.
    const int x_a = lane >> 4, x_q = (lane >> 2) & 3, x_w = lane & 3;
    uint32_t x_voff[XE], x_wr[XE][2], x_rd[2][2];
#pragma unroll
    for (int e = 0; e < XE; ++e) {
        const int row = 4 * e + x_a;
        x_voff[e] = ((uint32_t)min(row, M - 1) * K32 + (uint32_t)((lane & 15) * 8)) * 2;
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)
            x_wr[e][hl] = (uint32_t)(row * kBlockK * 2 + (((x_q * 4 + (x_w >> 1) * 2 + hl) ^ row) << 4) + ((x_w & 1) << 3));
    }
#pragma unroll
    for (int wp = 0; wp < 2; ++wp)
#pragma unroll
        for (int hl = 0; hl < 2; ++hl) x_rd[wp][hl] = (uint32_t)(n_l * kBlockK * 2 + (((g_l * 4 + wp * 2 + hl) ^ n_l) << 4));

    // (a k block beyond the last is requested through a resource of no bytes: zeros, without an access to memory)
    auto rsrc_if = [](const void* p, bool in) -> __amdgpu_buffer_rsrc_t {
        const uint64_t a = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
        void* q = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
        return __builtin_amdgcn_make_buffer_rsrc(q, 0, __builtin_amdgcn_readfirstlane(in ? 0x7fffffff : 0), 0x00020000);
    };
    u32x4 c[kItemBlocks], xr[2][XE];
    uint32_t pw[kItemBlocks];
    const uint32_t param_voff = (uint32_t)nkb * kBlockCodeBytes + 4 * n_l;
    auto load_w = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(base, kb < nkb);
        c[d] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, kb * kBlockCodeBytes, 0);
        pw[d] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)param_voff, kb * (4 * kBlockRows), 0);
    };
    auto load_x = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(X, kb < nkb);
#pragma unroll
        for (int e = 0; e < XE; ++e) xr[d][e] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)x_voff[e], kb * (kBlockK * 2), 0);
    };
    // (in the order of use: a wait for one request is a wait for all before it)
#pragma unroll
    for (int j = 0; j < kItemBlocks; ++j) {
        if (j < 2) load_x(wave * kItemBlocks + j, j);
        load_w(wave * kItemBlocks + j, j);
    }

    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    const half_t one = (half_t)1.f;
    const half8_t ones8 = {one, one, one, one, one, one, one, one};
    auto mfma = [](const half8_t& a, const half8_t& b, const floatx4& v) -> floatx4 { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, v, 0, 0, 0); };
    for (int item = wave; item < items; item += kItemWaves) {
        floatx4 ysum = zero4;
#pragma unroll
        for (int j = 0; j < kItemBlocks; ++j) {
            const int kb = item * kItemBlocks + j;
#pragma unroll
            for (int e = 0; e < XE; ++e) {
                const half8_t v = __builtin_bit_cast(half8_t, xr[j & 1][e]);
                *reinterpret_cast<half4_t*>(xl + x_wr[e][0]) = half4_t{v[0], v[1], v[6], v[7]};
                *reinterpret_cast<half4_t*>(xl + x_wr[e][1]) = half4_t{v[2], v[3], v[4], v[5]};
            }
            load_x(j < 2 ? kb + 2 : kb - 2 + kItemWaves * kItemBlocks, j & 1);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // read back by the wavefront that wrote it
            __builtin_amdgcn_wave_barrier();
            half8_t xh[2], xs[2];
#pragma unroll
            for (int wp = 0; wp < 2; ++wp) {
                xh[wp] = *reinterpret_cast<const half8_t*>(xl + x_rd[wp][0]);
                xs[wp] = *reinterpret_cast<const half8_t*>(xl + x_rd[wp][1]);
            }
            half2_t p[4][4];
#pragma unroll
            for (int w = 0; w < 4; ++w) w1_pairs_mixed(c[j][w], fmask, fmask_low, p[w]);
            const float sc = (float)param_scale(pw[j]);
            const float bi = (float)param_bias(pw[j]);
            load_w(kb + kItemWaves * kItemBlocks, j);
            floatx4 acc_h = zero4, acc_l = zero4, sh = zero4, sl = zero4;
#pragma unroll
            for (int wp = 0; wp < 2; ++wp) {
                const half2_t* w0 = p[2 * wp];
                const half2_t* w1 = p[2 * wp + 1];
                const half8_t wh = {w0[0][0], w0[0][1], w0[3][0], w0[3][1], w1[0][0], w1[0][1], w1[3][0], w1[3][1]};
                const half8_t wl = {w0[1][0], w0[1][1], w0[2][0], w0[2][1], w1[1][0], w1[1][1], w1[2][0], w1[2][1]};
                acc_h = mfma(xh[wp], wh, acc_h);
                acc_l = mfma(xs[wp], wl, acc_l);
                sh = mfma(xh[wp], ones8, sh);
                sl = mfma(xs[wp], ones8, sl);
            }
            const floatx4 sx = sh + sl, sx30 = 30.f * sl;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ysum[r] += sc * ((acc_h[r] + 16.f * acc_l[r] - sx30[r]) - bi * sx[r]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();            // X is read before the next block's is written
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(item * 16 + 4 * g_l + r) * kBlockRows + n_l] = ysum[r];
    }
    __syncthreads();
    if (t < 16 * kBlockRows) {
        const int m = t >> 4;
        const int64_t col = (int64_t)blockIdx.x * kBlockRows + (t & 15);
        float s = 0.f;
        for (int i = 0; i < min(items_ph, items); ++i) {
            float cell = red[i * (16 * kBlockRows) + t];
            for (int g = i + items_ph; g < items; g += items_ph) cell += red[g * (16 * kBlockRows) + t];
            s += cell;
        }
        if (m < M && col < N) {
            if (residual) s += (float)residual[(int64_t)m * N + col];
            Y[(int64_t)m * N + col] = (half_t)s;
        }
    }
}

template <int XE>
int launch_items(const half_t* X, int64_t M, const uint4* packed, int64_t N, int64_t K, int items_ph, half_t* Y, const half_t* residual,
                 hipStream_t stream)
{
    const int items = (int)((K / kBlockK + kItemBlocks - 1) / kItemBlocks);
    const int lds = kItemWaves * kItemXBytes + items * 16 * kBlockRows * (int)sizeof(float);
    static std::atomic<uint64_t> lds_allowed{0};
    const int arc = allow_dynamic_lds(reinterpret_cast<const void*>(&gemv_items_kernel<XE>),
                                      kItemWaves * kItemXBytes + kMaxItems * 16 * kBlockRows * (int)sizeof(float), lds_allowed);
    if (arc != E0M4_OK) return arc;
    hipLaunchKernelGGL(gemv_items_kernel<XE>, dim3((unsigned)row_blocks(N)), dim3(kItemThreads), lds, stream, X, packed, Y, residual,
                       (int)M, (uint32_t)N, (uint32_t)K, items_ph);
    return check_launch();
}

}  // namespace

// `items_ph`: work items per phase of the order of the sums, `waves` the wavefronts of that order: an item per wavefront and
// phase at most, or a wavefront's items of a phase would be one sum.
bool gemv_items_supported(int64_t M, int64_t K, int items_ph, int waves)
{
    return M >= 2 && M <= 16 && K > 0 && K % kBlockK == 0 && items_ph > 0 && items_ph <= waves &&
           (K / kBlockK + kItemBlocks - 1) / kItemBlocks <= kMaxItems;
}

int launch_gemv_items(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int items_ph, int waves, void* Y,
                      const void* residual, hipStream_t stream)
{
    if (!gemv_items_supported(M, K, items_ph, waves) || N <= 0) return E0M4_ERR_SHAPE;
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    const half_t* r = static_cast<const half_t*>(residual);
    if (M <= 4) return launch_items<1>(x, M, c, N, K, items_ph, y, r, stream);
    if (M <= 8) return launch_items<2>(x, M, c, N, K, items_ph, y, r, stream);
    return launch_items<4>(x, M, c, N, K, items_ph, y, r, stream);
}

}  // namespace e0m4
