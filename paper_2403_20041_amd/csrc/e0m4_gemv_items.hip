// Small batch with X taken block by block: Y[M,N] = X[M,K] * dequant(packed)^T (+ residual) for few rows of X (16, 8 and 4 with
// groups of 128, 64 and 32) and one or two row blocks (of 16 weight rows) per workgroup.  Paper: section "Operator and lagging
// optimizations" (vector-matrix product of the decoding stage, bound by memory bandwidth) with the dequantisation of section
// "E0M4 FP4 quantization" fused in registers.
//
// The same products and sums, in the same order, as gemv_mfma_kernel (e0m4_gemv_mfma.hip), to the bit: exact code values on
// v_mfma_f32_16x16x32_f16 with the two kinds of code pairs apart, the group's affine map per k block, one running sum per
// wavefront of that kernel and phase of K ("unit": of the work items of four k blocks r, r + W, ... of phase p, for every row
// block), the phases' sums of a wavefront added first, then the wavefronts'.  What differs is how X comes in.  There a
// workgroup stages M rows of X, or as much of K as fits the LDS, behind barriers, a piece of work that does not shrink with
// the row blocks that share it.  Here nothing is shared before the end and no barrier stands in the loop: a wavefront takes the
// units w, w + 8, ..., loads the rows of X of its own k blocks two ahead, turns them into operand order in a piece of LDS of its
// own and parks a unit's sums in LDS.
//
// What bounds it: X from L2 (every workgroup needs all 2 M K bytes: at M = 16 and K = 16384 512 KiB for 136 KiB of weights).
// With a residual and cold weights, X staged and here (us): 4096 x 13696 at M = 16 20.1 -> 14.7, at M = 8 15.2 -> 11.7; 2048 x 16384
// 19.4 -> 14.8 and 13.9 -> 11.6 (with the weights in the last-level cache 11.0 at M = 16); two row blocks: 5120 x 13696 26.7 -> 18.3,
// 5120 x 5120 13.5 -> 9.7; groups of 64 at M = 8: 5120 x 13696 21.2 -> 15.5, 5120 x 5120 11.3 -> 8.5; 8-bit codes: 4096 x 4096 at M =
// 16 9.1 -> 7.3, at M = 8 7.4 -> 6.6, 4096 x 13696 at M = 16 23.2 -> 18.9.  Where it is not the faster one: gemv_items_pays.
#include "e0m4_device.h"
#include "e0m4_host.h"

#include <algorithm>

namespace e0m4 {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kItemWaves = 8;
constexpr int kItemThreads = kItemWaves * 64;
constexpr int kItemBlocks = 4;                  // k blocks of 128 per work item
constexpr int kMaxSums = 96;                    // of units and row blocks: 1 KiB each, beside the wavefronts' X (4 KiB each)
constexpr int kZeroBytes = 64;                  // several groups per block: the zeros of a k-group that is not the row's
constexpr int kItemXBytes = 16 * kBlockK * 2;   // sixteen rows of a k block (8-bit codes: half of that)

// XE: loads of X per k block, four rows each (calls of up to 4 and 8 rows make one and two; the other rows of the tile stay
// what LDS held, and so do their sums, which nobody stores; 8-bit codes: eight rows a load).  R: row blocks per workgroup.
// GS: groups per k block; a row of X is then GS rows of the MFMA, with zeros for the k-groups of the other groups.  E8: 8-bit codes,
// k blocks of 64 weights, a single kind of code slot.  `residual` may be Y: neither is declared free of aliases.
template <int XE, int R, int GS, bool E8>
__global__ __launch_bounds__(kItemThreads, 2) void gemv_items_kernel(const half_t* __restrict__ X, const uint4* __restrict__ packed,
                                                                     half_t* Y, const half_t* residual,
                                                                     int M, uint32_t N32, uint32_t K32, int rb_base, int rb_rem,
                                                                     int order_waves, int items_ph)
{
    static_assert(!E8 || GS == 1, "8-bit codes: a parameter word per block");
    constexpr int SLOT = 16 / GS;
    constexpr int BLK = E8 ? kBlockK / 2 : kBlockK, ROWB = BLK * 2;     // weights of a row per k block, bytes of X
    constexpr int PPR = ROWB / 16, RPI = 64 / PPR;                      // 16-byte pieces per row, rows per load
    constexpr uint32_t kFirstX = GS > 1 ? kZeroBytes : 0;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int64_t N = N32;
    const int nkb = (int)(K32 / BLK), items = (nkb + kItemBlocks - 1) / kItemBlocks;
    const int n_ph = (items + items_ph - 1) / items_ph, items_end = items - (n_ph - 1) * items_ph;
    const int units_ph = min(order_waves, items_ph);
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n_l = lane & 15, g_l = lane >> 4;         // weight row and chunk of this lane; also (row of X, k-group)
    const uint32_t fmask = frac_mask_vgpr(), fmask_low = frac_mask_low_vgpr();
    unsigned char* xl = smem + kFirstX + wave * kItemXBytes;
    float* red = reinterpret_cast<float*>(smem + kFirstX + kItemWaves * kItemXBytes);   // [units][R][16 m][16 n]
    const uint32_t rb_stride = (uint32_t)nkb * block_bytes(128 / GS);
    const int64_t rb0 = (int64_t)blockIdx.x * rb_base + min((int)blockIdx.x, rb_rem);
    const int n_rb = rb_base + ((int)blockIdx.x < rb_rem ? 1 : 0);
    const char* base = reinterpret_cast<const char*>(packed) + (size_t)rb0 * rb_stride;
    const uint32_t rb_next = n_rb > 1 ? rb_stride : 0;  // (no second row block: the first again, its sums are not used)

    // X: load number e brings rows 4 e .. 4 e + 3 of the k block, 16 bytes per lane.  A piece of eight activations (of one code
    // word) is two halves, those of the pairs that read 2 + c/8 and those that read 2 + c/128; unit u = 4 q + 2 (w / 2) + half
    // of a row lies at 16 (u ^ row): the sixteen rows of an operand read fall into sixteen different bank groups.
    // (8-bit codes: a piece is a unit, at 16 (u ^ row / 2))
    const int x_a = lane / PPR, x_j = lane % PPR, x_q = (lane >> 2) & 3, x_w = lane & 3;
    uint32_t x_voff[XE], x_wr[XE][2], x_rd[2][2];
#pragma unroll
    for (int e = 0; e < XE; ++e) {
        const int row = RPI * e + x_a;
        x_voff[e] = ((uint32_t)min(row, M - 1) * K32 + (uint32_t)(x_j * 8)) * 2;
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)
            x_wr[e][hl] = (uint32_t)(row * ROWB) + (uint32_t)(E8 ? (x_j ^ ((row >> 1) & 7)) << 4
                                                                 : (((x_q * 4 + (x_w >> 1) * 2 + hl) ^ row) << 4) + ((x_w & 1) << 3));
    }
#pragma unroll
    for (int wp = 0; wp < 2; ++wp)
#pragma unroll
        for (int hl = 0; hl < 2; ++hl) {
            const int row = n_l % SLOT;
            const bool own = GS == 1 || n_l / SLOT == g_l * GS / 4;
            if (E8) x_rd[wp][hl] = (uint32_t)(wave * kItemXBytes + row * ROWB + (((g_l * 2 + wp) ^ ((row >> 1) & 7)) << 4));
            else x_rd[wp][hl] = own ? kFirstX + (uint32_t)(wave * kItemXBytes + row * ROWB + (((g_l * 4 + wp * 2 + hl) ^ row) << 4)) : 0u;
        }
    if (GS > 1) {                                       // (every wavefront before its own reads, with the same zeros)
        if (lane < kZeroBytes / 4) reinterpret_cast<uint32_t*>(smem)[lane] = 0;
    }

    // (a k block beyond the last is requested through a resource of no bytes: zeros, without an access to memory)
    u32x4 c[kItemBlocks][R], xr[2][XE];
    uint32_t pw[kItemBlocks][R];
    const uint32_t param_voff = (uint32_t)nkb * kBlockCodeBytes + 4 * ((g_l * GS / 4) * kBlockRows + n_l);
    auto load_w = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(base, kb < nkb);
#pragma unroll
        for (int s = 0; s < R; ++s) {
            c[d][s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, (int)(s * rb_next + (uint32_t)kb * kBlockCodeBytes), 0);
            pw[d][s] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)param_voff,
                                                            (int)(s * rb_next + (uint32_t)kb * (4 * kBlockRows * GS)), 0);
        }
    };
    auto load_x = [&](int kb, int d) {
        const __amdgpu_buffer_rsrc_t rsrc = rsrc_if(X, kb < nkb);
#pragma unroll
        for (int e = 0; e < XE; ++e) xr[d][e] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)x_voff[e], kb * ROWB, 0);
    };
    // Units in the order u = p * units_ph + r, dealt round the wavefronts; where that gives a wavefront the same units of every
    // phase, `turn` on from phase to phase, the number of units with one item more than the others.  Item i of phase p is item
    // p * items_ph + i of all.  Past the last unit (in a last phase of fewer items than units_ph, too) the item is one without
    // k blocks.
    struct Place {
        int ph, r, i;
    };
    auto items_of = [&](int p) -> int { return p == n_ph - 1 ? items_end : items_ph; };
    auto there = [&](const Place& q) -> bool { return q.ph < n_ph && q.r < items_of(q.ph); };
    auto item_of = [&](const Place& q) -> int { return there(q) ? q.ph * items_ph + q.i : items; };
    const int turn = units_ph % kItemWaves == 0 ? items_ph % order_waves : 0;
    auto settle = [&](Place q) -> Place {
        while (q.r >= units_ph) {
            q.r -= units_ph;
            if (units_ph % kItemWaves == 0) q.r = (q.r - turn) & (kItemWaves - 1);
            ++q.ph;
        }
        q.i = q.r;
        return q;
    };
    auto after = [&](Place q) -> Place {
        if (q.i + order_waves < items_of(q.ph)) {
            q.i += order_waves;
            return q;
        }
        q.r += kItemWaves;
        return settle(q);
    };
    Place at = settle(Place{0, wave, 0});
    // (in the order of use: a wait for one request is a wait for all before it)
#pragma unroll
    for (int j = 0; j < kItemBlocks; ++j) {
        if (j < 2) load_x(item_of(at) * kItemBlocks + j, j);
        load_w(item_of(at) * kItemBlocks + j, j);
    }

    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
    const half_t one = (half_t)1.f;
    const half8_t ones8 = {one, one, one, one, one, one, one, one};
    auto mfma = [](const half8_t& a, const half8_t& b, const floatx4& v) -> floatx4 {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, v, 0, 0, 0);
    };
    floatx4 ysum[R];
#pragma unroll
    for (int s = 0; s < R; ++s) ysum[s] = zero4;
    while (there(at)) {
        const Place next = after(at);
        const int kb_at = item_of(at) * kItemBlocks, kb_next = item_of(next) * kItemBlocks;
#pragma unroll
        for (int j = 0; j < kItemBlocks; ++j) {
#pragma unroll
            for (int e = 0; e < XE; ++e) {
                const half8_t v = __builtin_bit_cast(half8_t, xr[j & 1][e]);
                if (E8) {
                    *reinterpret_cast<half8_t*>(xl + x_wr[e][0]) = v;
                    continue;
                }
                *reinterpret_cast<half4_t*>(xl + x_wr[e][0]) = half4_t{v[0], v[1], v[6], v[7]};
                *reinterpret_cast<half4_t*>(xl + x_wr[e][1]) = half4_t{v[2], v[3], v[4], v[5]};
            }
            load_x(j < 2 ? kb_at + j + 2 : kb_next + j - 2, j & 1);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // read back by the wavefront that wrote it
            __builtin_amdgcn_wave_barrier();
            half8_t xh[2], xs[2];
#pragma unroll
            for (int wp = 0; wp < 2; ++wp) {
                xh[wp] = *reinterpret_cast<const half8_t*>(smem + x_rd[wp][0]);
                xs[wp] = E8 ? xh[wp] : *reinterpret_cast<const half8_t*>(smem + x_rd[wp][1]);
            }
            floatx4 sh = zero4, sl = zero4;
#pragma unroll
            for (int wp = 0; wp < 2; ++wp) {
                sh = mfma(xh[wp], ones8, sh);
                if (!E8) sl = mfma(xs[wp], ones8, sl);
            }
            const floatx4 sx = sh + sl, sx30 = 30.f * sl;
#pragma unroll
            for (int s = 0; s < R; ++s) {
                half2_t p[4][4];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    if (E8) {                               // (w1_0, w1_1) and, after the rotation, (w1_2, w1_3)
                        const uint32_t m8 = fmask | fmask_low, word = c[j][s][w];
                        p[w][0] = __builtin_bit_cast(half2_t, (word & m8) | kExpBits2);
                        p[w][1] = __builtin_bit_cast(half2_t, (__builtin_amdgcn_alignbit(word, word, 8) & m8) | kExpBits2);
                    } else {
                        w1_pairs_mixed(c[j][s][w], fmask, fmask_low, p[w]);
                    }
                }
                const float sc = (float)param_scale(pw[j][s]);
                const float bi = (float)param_bias(pw[j][s]);
                floatx4 acc_h = zero4, acc_l = zero4;
#pragma unroll
                for (int wp = 0; wp < 2; ++wp) {
                    const half2_t* w0 = p[2 * wp];
                    const half2_t* w1 = p[2 * wp + 1];
                    if (E8) {
                        const half8_t w8 = {w0[0][0], w0[0][1], w0[1][0], w0[1][1], w1[0][0], w1[0][1], w1[1][0], w1[1][1]};
                        acc_h = mfma(xh[wp], w8, acc_h);
                        continue;
                    }
                    const half8_t wh = {w0[0][0], w0[0][1], w0[3][0], w0[3][1], w1[0][0], w1[0][1], w1[3][0], w1[3][1]};
                    const half8_t wl = {w0[1][0], w0[1][1], w0[2][0], w0[2][1], w1[1][0], w1[1][1], w1[2][0], w1[2][1]};
                    acc_h = mfma(xh[wp], wh, acc_h);
                    acc_l = mfma(xs[wp], wl, acc_l);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    ysum[s][r] += sc * ((acc_h[r] + 16.f * acc_l[r] - sx30[r]) - bi * sx[r]);
            }
            load_w(kb_next + j, j);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();            // X is read before the next block's is written
        }
        if (next.ph != at.ph || next.r != at.r) {       // the unit is complete
#pragma unroll
            for (int s = 0; s < R; ++s) {
#pragma unroll
                for (int r = 0; r < 4; ++r) red[(((at.ph * units_ph + at.r) * R + s) * 16 + 4 * g_l + r) * kBlockRows + n_l] = ysum[s][r];
                ysum[s] = zero4;
            }
        }
        at = next;
    }
    // The sums of all phases per wavefront of the order, then (in LDS that X has left) the wavefronts' in their order: the items i
    // of row block s that wavefront v has are those with (s * items of the phase + i) % W = v, the first of them r below.  (In one
    // pass over both, each sum a chain of dependent reads, 2048 x 16384 at M = 16 took 2.8 us longer.)
    __syncthreads();
    float* cells = reinterpret_cast<float*>(smem + kFirstX);        // [W][R][16 m][16 n]
    for (int c0 = wave >> 2; c0 < order_waves * R; c0 += kItemWaves / 4) {
        const int v = c0 / R, s = c0 % R, at_cell = t & 255;
        const int r_all = (v - s * items_ph) & (order_waves - 1), r_end = (v - s * items_end) & (order_waves - 1);
        float cell = 0.f;
        if (r_all < items_ph)
            for (int p = 0; p < n_ph - 1; ++p) cell += red[((p * units_ph + r_all) * R + s) * (16 * kBlockRows) + at_cell];
        if (r_end < items_end) cell += red[(((n_ph - 1) * units_ph + r_end) * R + s) * (16 * kBlockRows) + at_cell];
        cells[c0 * (16 * kBlockRows) + at_cell] = cell;
    }
    __syncthreads();
    const int s = t >> 8, m = (t >> 4) & 15;
    if (s < n_rb) {
        const int64_t col = (rb0 + s) * kBlockRows + (t & 15);
        float y = 0.f;
        for (int v0 = 0; v0 < order_waves; v0 += 8) {
            float cell[8][GS];
#pragma unroll
            for (int v = 0; v < 8; ++v)
#pragma unroll
                for (int gg = 0; gg < GS; ++gg)
                    cell[v][gg] = cells[(((v0 + v) * R + s) * 16 + min(m + SLOT * gg, 15)) * kBlockRows + (t & 15)];
#pragma unroll
            for (int v = 0; v < 8; ++v)
#pragma unroll
                for (int gg = 0; gg < GS; ++gg) y += cell[v][gg];
        }
        if (m < M && col < N) {
            if (residual) y += (float)residual[(int64_t)m * N + col];
            Y[(int64_t)m * N + col] = (half_t)y;
        }
    }
}

static_assert(kItemWaves * kItemXBytes >= 16 * 2 * 16 * kBlockRows * (int)sizeof(float), "the wavefronts' sums take the place of X");

// (K in 4-bit slots, two per 8-bit code)
int order_units(int64_t K, int items_ph, int waves)
{
    const int items = (int)((K / kBlockK + kItemBlocks - 1) / kItemBlocks), n_ph = (items + items_ph - 1) / items_ph;
    return n_ph * std::min(waves, items_ph);
}

template <int XE, int R, int GS, bool E8 = false>
int launch_items(const ItemsPlan& p, const half_t* X, int64_t M, const uint4* packed, int64_t N, int64_t K, half_t* Y,
                 const half_t* residual, hipStream_t stream)
{
    constexpr int kFixed = (GS > 1 ? kZeroBytes : 0) + kItemWaves * kItemXBytes, kSum = 16 * kBlockRows * (int)sizeof(float);
    const int lds = kFixed + order_units(K, p.items_ph, p.waves) * R * kSum;
    static std::atomic<uint64_t> lds_allowed{0};
    const int arc = allow_dynamic_lds(reinterpret_cast<const void*>(&gemv_items_kernel<XE, R, GS, E8>), kFixed + kMaxSums * kSum,
                                      lds_allowed);
    if (arc != E0M4_OK) return arc;
    hipLaunchKernelGGL((gemv_items_kernel<XE, R, GS, E8>), dim3((unsigned)p.grid), dim3(kItemThreads), lds, stream, X, packed, Y, residual,
                       (int)M, (uint32_t)N, (uint32_t)(E8 ? K / 2 : K), p.rb_base, p.rb_rem, p.waves, p.items_ph);
    return check_launch();
}

template <int R>
int launch_items_m(const ItemsPlan& p, const half_t* x, int64_t M, const uint4* c, int64_t N, int64_t K, int group, half_t* y,
                   const half_t* r, hipStream_t stream)
{
    if (p.e8) {
        if (M <= 8) return launch_items<1, R, 1, true>(p, x, M, c, N, K, y, r, stream);
        return launch_items<2, R, 1, true>(p, x, M, c, N, K, y, r, stream);
    }
    if (group == 32) return launch_items<1, R, 4>(p, x, M, c, N, K, y, r, stream);
    if (group == 64) {
        if (M <= 4) return launch_items<1, R, 2>(p, x, M, c, N, K, y, r, stream);
        return launch_items<2, R, 2>(p, x, M, c, N, K, y, r, stream);
    }
    if (M <= 4) return launch_items<1, R, 1>(p, x, M, c, N, K, y, r, stream);
    if (M <= 8) return launch_items<2, R, 1>(p, x, M, c, N, K, y, r, stream);
    return launch_items<4, R, 1>(p, x, M, c, N, K, y, r, stream);
}

}  // namespace

bool gemv_items_supported(const ItemsPlan& p, int64_t M, int64_t N, int64_t K, int group)
{
    if (M < 2 || M > 16 * group / 128 || N <= 0 || K <= 0 || K % kBlockK != 0) return false;
    if (p.items_ph <= 0 || (p.waves != 8 && p.waves != 16)) return false;
    const int most = p.rb_base + (p.rb_rem > 0 ? 1 : 0);
    return p.rb_base >= 1 && most <= 2 && order_units(K, p.items_ph, p.waves) * most <= kMaxSums;
}

// Where it is the faster one, by the plan (cold weights, this kernel's time over the staging kernel's; `fused`: the staging kernel
// would run in its instance for fused operators, 0.3 - 0.5 us slower than the one for plain calls; measured on 90 random problems per
// format and row count).  From three rows on:
//   K in phases: 0.57 - 0.95.  But 8-bit codes with two row blocks and sixteen wavefronts lie between 0.84 and 1.12, above one where
//     workgroups leave a good part of the compute units idle (4416 x 12416 at M = 9 1.10).
//   Whole rows, one row block: 0.68 - 0.97 with eight wavefronts.  With sixteen, X is staged in half the time: 4-bit codes 0.94 -
//     1.08 at three rows (fused 0.90 - 1.00) and 0.90 - 0.98 at four; 8-bit codes plain 0.96 - 1.17 up to six rows, 0.91 - 1.03 from
//     eight on, fused 0.89 - 1.03 from six on and, where three quarters of the compute units have a workgroup, from three (0.92 -
//     1.03; 4096 x 13696 at M = 3 15.6 and 15.3 us, but 2048 x 16384 12.7 and 14.1).
//   Whole rows, two row blocks share what is staged: fused 0.80 - 1.05 with eight wavefronts (0.94 on average), plain 1.0 - 1.15
//     (5120 x 5120 at M = 4 7.1 and 7.4 us, 8-bit at M = 12 10.1 and 11.2), but 0.88 - 0.98 where X is too large for sixteen
//     wavefronts' sums beside it, and with thirteen rows or more in 4-bit codes; with sixteen wavefronts 1.0 - 1.15.
// Groups of 64 and 32: plain calls with two row blocks 0.97 - 1.12, everything else 0.67 - 0.98.
constexpr int64_t kBusyGrid8 = 192;
bool gemv_items_pays(const ItemsPlan& p, int64_t M, int group, bool fused)
{
    const bool two = p.rb_base + (p.rb_rem > 0 ? 1 : 0) > 1;
    if (group == 128 && M < 3) return false;
    if (p.phased) return !(p.e8 && two && p.waves == 16) || p.grid >= kBusyGrid8;
    if (!two && p.waves == 16) return p.e8 ? (fused ? M >= 6 || p.grid >= kBusyGrid8 : M >= 8) : M >= (fused ? 3 : 4);
    if (!two) return true;
    return p.waves == 8 && (fused || p.items_ph > 16 || (!p.e8 && M > 12));
}

int launch_gemv_items(const ItemsPlan& p, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                      const void* residual, hipStream_t stream)
{
    if (!gemv_items_supported(p, M, N, K, group)) return E0M4_ERR_SHAPE;
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    const half_t* r = static_cast<const half_t*>(residual);
    return p.rb_base + (p.rb_rem > 0 ? 1 : 0) == 1 ? launch_items_m<1>(p, x, M, c, N, K, group, y, r, stream)
                                                   : launch_items_m<2>(p, x, M, c, N, K, group, y, r, stream);
}

}  // namespace e0m4
