// Software-pipelined tile of the prefill GEMM (paper: section "Operator and lagging optimizations",
// matrix-matrix product; dequantisation of section "E0M4 FP4 quantization" fused in registers), built
// for 256 x 256 outputs and, with four wavefronts side by side, for 128 x 256, 64 x 256, 128 x 128 (two workgroups
// per compute unit) and 64 x 128 outputs (four); shortest() below chooses.  The description is that of the large tile.
//
// Eight wavefronts (2 x 4, two per SIMD) share the tile, 128 x 64 outputs and 128 fp32 accumulator
// registers per lane each, which leaves two wavefronts per SIMD at most: little but a wavefront's own
// instruction stream can hide latency.  The stream is therefore laid out by hand, per K slice of 64
// (= 4 MFMA sub-steps of 16):
//   - activations: global -> LDS ring of four stages, without a register in between, requested two and a half
//     slices ahead -> 16-byte fragments, read one sub-step ahead of their use;
//   - weights: never touch LDS.  Lane (n = l%32, h = l/32) reads the 16-byte chunk of row n with
//     k = 32h..32h+31 of the slice (three slices ahead), and word s of that chunk is dequantised
//     (shift, mask-or exponent, minus bias, times scale; packed fp16, bit-identical to
//     e0m4_dequant) one sub-step ahead of MFMA number s, whose K set is {8s..8s+7} u
//     {32+8s..32+8s+7}; the activation fragment of the same MFMA is piece 4h+s of the row.
//   - one barrier per slice, placed after sub-step 1: before it a wavefront waits for its own requests of slice
//     kt+1, whose fragment reads start in sub-step 3; behind it the stage of slice kt-1 is free for slice kt+3.
// Through registers the activations could be requested one slice ahead, and the weights too: less than a memory latency
// where a wavefront has a SIMD to itself.  Time of a pair of slices (K = 8192 against 2048), then and now: 64 x 256 tiles on
// 64, 256 and 512 workgroups 1.24 -> 0.85, 1.82 -> 1.47 and 2.56 -> 2.41 us; 128 x 256 tiles on 64, 256 and 512 1.43 -> 1.15, 1.95 ->
// 1.86 and 3.62 -> 3.54; 256 x 256 tiles on 256 3.53 -> 3.39.  With all compute units at work the clock that the chip holds
// is the bound: the same launch on zero operands takes 0.56 of the time, without the dequantisation 0.86 of it, with
// activation fragments that are read once 0.94, with neither 0.68 (128 x 256 tiles).  A wavefront that owns all 256 rows of the
// large tile (accumulators in the AGPRs, each weight dequantised once) gains 3 % per pair and loses 3 us per tile.
// The LDS tile is 128-byte rows whose eight 16-byte pieces are XOR-swizzled with (row / 2) % 8: the
// LDS of gfx950 serves a 16-byte-per-lane read 16 lanes (256 bytes, two rows of the tile) at a time,
// so 16 consecutive rows have to land in 16 different 16-byte bank groups (swizzling with row % 8, the
// right choice for 128-byte-wide LDS, costs 40 % more LDS cycles here, all of them bank conflicts).
#include "e0m4_device.h"
#include "e0m4_host.h"

#include <algorithm>
#include <type_traits>

namespace e0m4 {

namespace {

constexpr int BK = 64;
constexpr int kRowBytes = BK * 2;
constexpr int kStages = 4;
constexpr int kNumXcd = 8;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ inline half2_t dequant_pair(half2_t w1, half2_t bias2, half2_t scale2)
{
    return (w1 - bias2) * scale2;                       // difference exact, product rounded once
}

// bfloat16 member (BF): X, the embedded parameters and Y are bfloat16; the same packed codes.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ inline T out_value(float v)                 // one rounding to the output type (nearest even)
{
    return (T)v;
}

// WGM x WGN wavefronts share the tile.  Built as 2 x 4 (two per SIMD, 128 x 64 each): against 2 x 2
// (one per SIMD, 128 x 128 each) that doubles the instruction issue capacity and lets one wavefront's
// waits hide behind the other's MFMAs, for twice the activation fragment traffic; 2 x 2 (accumulators in
// the 256 AGPRs, one wavefront per SIMD, 17 registers spilled) was measured 3-9 % slower on every shape.
//
// FUSED adds the operators of e0m4_matmul_fused that belong to the epilogue (paper: section "Operator and
// lagging optimizations", element-wise operators fused into their neighbours).  With the gated
// epilogue a tile covers 128 output columns: the first operand block of a wavefront holds 32 gate rows
// o .. o+31 and its second the up rows N/2 + o .. N/2 + o+31, so that a lane finds the gate and the up
// value of an output element in the same register of its two accumulator blocks and writes
// silu(gate) * up.  The residual is added before the one rounding.  It may be Y, so neither is declared free of
// aliases.
struct PipeFusion {
    const half_t* residual;
    int swiglu;
    int panel;                                          // row tiles per panel of the tile numbering (0: one panel)
    int split_major;                                    // work items ordered by K split first, then by tile
    int64_t n_half;                                     // N / 2 (gated epilogue)
};

// Even scheduling of the tiles over the compute units ("stream-K").  When the tile count is not a multiple of
// the number of compute units, the last, partly filled round would leave units idle for the length of a whole
// tile.  With `enabled`, the launch has exactly one workgroup per compute unit, and each workgroup runs
//   - `rounds_dp` whole tiles (tile r * grid + position), written out directly, then
//   - its share of the remaining `rem_tiles` tiles: those tiles' K ranges, in pairs of K slices, laid end to end
//     are `rem_tiles * pairs` units, of which the workgroup at position p owns [p * U / grid, (p + 1) * U / grid):
//     at most the tail of one tile and the head of the next.
// A tile that several workgroups share is finished by whichever of them arrives last: every sharer stores its
// fp32 partial sums to a slab of the workspace (slabs of the sharers of a tile are consecutive, in K order) with
// write-through stores, one thread orders them ahead of the counter (release fence) and adds one to the tile's
// counter; the one that brings the counter to the number of sharers reads all slabs back (acquire, device-coherent
// loads), adds them in K order -- a fixed order, whoever does it -- and writes the tile.  Nobody waits for anybody,
// so a workgroup that is never scheduled next to the others cannot stall them.  The counters are zeroed by a small
// kernel before the launch.  The shared-out tiles are numbered row by row (see the kernel).
struct SkArgs {
    int enabled;
    int rounds_dp;                                      // whole tiles per workgroup
    int rem_tiles;                                      // tiles shared out in K ranges, after rounds_dp * grid whole tiles
    int pairs;                                          // K / 128: pairs of K slices per tile
    unsigned int* counters;                             // [rem_tiles], zero on entry
    float* slabs;                                       // [grid + rem_tiles][BM * BN] fp32
};

//
// The tile is BM x BN: 256 x 256 with 2 x 4 wavefronts; 128 x 256 with 1 x 4 wavefronts (the same 128 x 64 per
// wavefront, two independent workgroups per compute unit); 64 x 256 with 1 x 4 wavefronts, where the taller tiles
// would compute many rows that do not exist or leave compute units without a tile; 128 x 128 and 64 x 128 with 1 x 4
// wavefronts of 32 columns (TN = 1), which take half of those wavefronts' registers and time per slice, where tiles are few.  Gated,
// such wavefronts alternate: an even one holds the gate's columns, the next one the same columns of the up projection, and
// hands its sums over in LDS. 
//
// SHORT: M leaves 64 rows or fewer in the last row tile of 128.  Those tiles are computed in two of their four 32-row blocks
// (one block would take as long: below that the dequantisation is all there is to do) and are numbered last on every XCD, so
// that they fill the gaps at the end.  In instances of its own: another form of the K loop beside it costs the usual one 2 %
// (1024 rows, two 6B blocks 899 -> 916 us).  It takes as many tiles as compute units, or nobody waits for the whole ones (7424 x
// 2688 at M = 700, 174 tiles, 38.0 and 40.3 us), and six row tiles at most.  Short over whole with this tile forced, 3 to 13 row
// tiles with 20 and 60 rows left, 4-bit 27392 x 4096 and 32768 x 2048 gated and 15360 x 5120, bfloat16 27392 x 4096 and 11008 x
// 4096, 8-bit 22016 x 3072: up to six row tiles 0.81 - 1.00, the least where the last round of workgroups is nearly empty (gated
// 27392 x 4096 at M = 316 97.6 -> 84.7 us, bfloat16 95.3 -> 84.1, gated 32768 x 2048 in groups of 32 57.5 -> 50.6, 15360 x 5120 at
// M = 572 116 -> 101; at six row tiles 0.97 - 1.00, but 0.87 and 0.90 with 258 and 516 tiles); beyond, 0.90 - 1.02: 4-bit codes still
// gain (27392 x 4096 at M = 828 177 -> 173), 8-bit codes and bfloat16 of fewer columns lose (22016 x 3072 at M = 788 128.6 -> 131.1,
// 11008 x 4096 93.9 -> 95.0).
//
// E8 selects the 8-bit format E0M8 (e0m8_pack.hip; G is then 128, the group of its 4-bit slots): a K slice
// of 64 is one block, a lane reads two 16-byte chunks of 16 weights per slice, and MFMA number s takes
// words 2(s%2) and 2(s%2)+1 of chunk s/2, each of which one mask-or (and one more after a rotation) turns
// into four binade values.  DEPTH: slices of codes in registers, where it is not the default.
template <int G, int WGM, int WGN, bool FUSED, int BM, int BN, bool E8 = false, bool BF = false, int KS = 1, bool SHORT = false, int DEPTH = 0>
__global__ __launch_bounds__(64 * WGM * WGN * KS, 2) void gemm_pipe_kernel(const half_t* __restrict__ X, int64_t M,
                                                             const uint4* __restrict__ packed, int64_t N, int64_t K,
                                                             half_t* Y, int m_tiles, int n_tiles,
                                                             int splits, float* __restrict__ partial, PipeFusion fu,
                                                             SkArgs sk)
{
    constexpr int kThreads = 64 * WGM * WGN;            // per K part
    constexpr int kStageBytes = BM * kRowBytes;
    // Slices of weights in registers (8-bit codes: twice the registers per slice), stages of activations in LDS, and how many
    // slices ahead those are requested.
    constexpr int PD = DEPTH > 0 ? DEPTH : E8 && BM > 64 ? 2 : 4, S = kStages, L = S - 1;
    constexpr int TM = BM / (32 * WGM), TN = BN / (32 * WGN);      // 32x32 MFMA blocks per wavefront
    constexpr int RP = kThreads / 8;                    // rows covered by one activation loader pass
    constexpr int PA = BM / RP;                         // activation loader passes
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    // Work items are (tile, K split) pairs, the splits of a tile adjacent -- or, with split_major, all tiles of one
    // split before those of the next, so that the workgroups running together on an XCD are on the same K range of
    // neighbouring tiles and share operands in its L2; each XCD takes a contiguous run.
    // (even scheduling exists in the instance the launcher uses it with; elsewhere the segment loop below folds away)
    static_assert(!BF || (!FUSED && !E8), "the bfloat16 member has the plain 4-bit kernel only");
    static_assert(!SHORT || (WGM == 1 && BM == 128 && KS == 1), "short last row tiles: of 128 rows");
    static_assert(KS == 1 || BM == 64, "K parts inside a workgroup: tiles of 64 rows");
    static_assert(!FUSED || KS == 1 || TN == 2, "the exchange of gated sums between wavefronts has no place for more than one K part");
    constexpr bool kSk = !FUSED && !E8 && !BF && BM == 256 && BN == 256;
    const bool sk_on = kSk && sk.enabled;
    const int total = m_tiles * n_tiles * splits;
    const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
    int item = (blockIdx.x % kNumXcd) * per_xcd + blockIdx.x / kNumXcd;
    int tiles_m = m_tiles;                              // row tiles of the numbering
    if (SHORT) {                                        // (splits == 1, two row tiles at least)
        const int full = (m_tiles - 1) * n_tiles, pf = (full + kNumXcd - 1) / kNumXcd, pr = (n_tiles + kNumXcd - 1) / kNumXcd;
        const int xcd = blockIdx.x % kNumXcd, j = blockIdx.x / kNumXcd;
        item = j < pf ? xcd * pf + j : full + xcd * pr + (j - pf);
        if (j < pf ? item >= full : item >= total) return;
        tiles_m = m_tiles - 1;
    }
    if (!sk_on && item >= total) return;
    const int KT_all = (int)(K / BK);
    // Even scheduling: this workgroup's position (consecutive positions on one XCD: they share weight rows in
    // its L2), its range of units among the shared-out tiles, and the one or two K ranges that makes.
    // (Quotients are computed on the vector unit: every one of them goes through readfirstlane, or the segment
    // loop below, its trip count included, counts as divergent and every buffer load turns into a per-lane loop.
    // All of this fits 32 bits: at most 255 shared-out tiles of at most 8192 pairs, times 256 positions.)
    const uint32_t sk_grid = gridDim.x;
    const uint32_t sk_pos = (blockIdx.x % kNumXcd) * (sk_grid / kNumXcd) + blockIdx.x / kNumXcd;
    const uint32_t sk_pairs = (uint32_t)sk.pairs;
    const uint32_t sk_units = (uint32_t)sk.rem_tiles * sk_pairs;
    // (fewer units than workgroups, which only a forced launch has: the first sk_units positions take one each, so
    // that the sharers of a tile are always consecutive positions with a share each)
    const uint32_t sk_div = sk_units < sk_grid ? (sk_units > 0 ? sk_units : 1u) : sk_grid;
    auto sk_begin = [&](uint32_t pos) -> uint32_t {     // first unit of the workgroup at `pos`
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(sk_units * (pos < sk_div ? pos : sk_div) / sk_div));
    };
    const uint32_t sk_u0 = sk_on ? sk_begin(sk_pos) : 0u, sk_u1 = sk_on ? sk_begin(sk_pos + 1) : 0u;
    const uint32_t sk_t0 = sk_u1 > sk_u0 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(sk_u0 / sk_pairs)) : 0u;  // its first tile
    int sk_segs = 0;
    if (sk_u1 > sk_u0) sk_segs = sk_u1 > (sk_t0 + 1) * sk_pairs ? 2 : 1;
    const int n_segments = sk_on ? sk.rounds_dp + sk_segs : 1;
    // the position whose range holds `unit`
    auto sk_pos_of = [&](uint32_t unit) -> int {
        uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)(unit * sk_div / sk_units));
        while (sk_begin(g + 1) <= unit) ++g;
        while (sk_begin(g) > unit) --g;
        return (int)g;
    };
    // the work item of a launch without even scheduling
    const int all_tiles = m_tiles * n_tiles;
    const int plain_tile = __builtin_amdgcn_readfirstlane(fu.split_major ? item % all_tiles : item / splits);
    const int plain_split = __builtin_amdgcn_readfirstlane(fu.split_major ? item / all_tiles : item % splits);
    // (KS > 1: no K split of the launch; the workgroup's wavefronts take a part of K each)
    const int part = KS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads) : 0;
    const int k_part = KS > 1 ? part : plain_split, k_parts = KS > 1 ? KS : splits;
    const int plain_kb = __builtin_amdgcn_readfirstlane(2 * (int)((int64_t)(KT_all / 2) * k_part / k_parts));
    const int plain_ke = __builtin_amdgcn_readfirstlane(2 * (int)((int64_t)(KT_all / 2) * (k_part + 1) / k_parts));
  for (int seg = 0; seg < n_segments; ++seg) {
    if (seg > 0) __syncthreads();                       // every wavefront has left the previous segment's LDS stages
    // what this segment computes: a tile, a range of its K slices, and where the sums go
    //   out_mode 0: the whole K range, results to Y (with the fused epilogue, if any)
    //   out_mode 1: one of `splits` K ranges, fp32 sums to slab `split` of the [splits][M][N] workspace
    //   out_mode 2: a shared-out K range (see SkArgs), fp32 sums to this sharer's slab; the last sharer finishes the tile
    int seg_tile, seg_kb, seg_ke, out_mode, seg_split = 0, sk_rt = 0, sk_first = 0, sk_sharers = 1;
    if (!sk_on) {
        seg_tile = plain_tile;
        seg_split = plain_split;
        seg_kb = plain_kb;
        seg_ke = plain_ke;
        out_mode = splits > 1 ? 1 : 0;
    } else if (seg < sk.rounds_dp) {
        seg_tile = seg * (int)sk_grid + (int)sk_pos;
        seg_kb = 0;
        seg_ke = KT_all;
        out_mode = 0;
    } else {
        sk_rt = (int)sk_t0 + (seg - sk.rounds_dp);      // the range's first tile, then its second
        const uint32_t t_lo = (uint32_t)sk_rt * sk_pairs, t_hi = t_lo + sk_pairs;
        const uint32_t lo = sk_u0 > t_lo ? sk_u0 : t_lo, hi = sk_u1 < t_hi ? sk_u1 : t_hi;
        // Which tile is shared-out tile number sk_rt: the shared tiles are the last rem_tiles of the column-by-column
        // numbering (the tail of column c0 from row tile m_start on, then whole columns); they are taken row by row
        // instead, so that the workgroups of one XCD, whose ranges are consecutive, are on tiles of the same rows of
        // X at nearly the same K (consecutive tiles start 'units per workgroup' apart): the activations, four
        // times the bytes of the weights, are then shared through that XCD's L2.
        const uint32_t first_shared = (uint32_t)sk.rounds_dp * sk_grid, mt = (uint32_t)m_tiles;
        const uint32_t c0 = first_shared / mt, m_start = first_shared - c0 * mt;
        const uint32_t w_full = (uint32_t)n_tiles - 1 - c0;         // columns after c0: shared in every row tile
        const uint32_t head = m_start * w_full;                     // shared tiles of the row tiles above m_start
        uint32_t tm, tn;
        if ((uint32_t)sk_rt < head) {
            tm = (uint32_t)sk_rt / w_full;
            tn = c0 + 1 + ((uint32_t)sk_rt - tm * w_full);
        } else {
            const uint32_t r = (uint32_t)sk_rt - head, q = r / (w_full + 1);
            tm = m_start + q;
            tn = c0 + (r - q * (w_full + 1));
        }
        seg_tile = (int)(tn * mt + tm);
        seg_kb = 2 * (int)(lo - t_lo);
        seg_ke = 2 * (int)(hi - t_lo);
        sk_first = sk_pos_of(t_lo);
        sk_sharers = sk_pos_of(t_hi - 1) - sk_first + 1;
        out_mode = sk_sharers > 1 ? 2 : 0;
    }
    // (quotients and remainders are computed on the vector unit; move them to scalar registers, or
    // everything derived from them, the K loop counter included, is treated as divergent and every
    // buffer load below turns into a per-lane loop)
    const int tile = __builtin_amdgcn_readfirstlane(seg_tile);
    const int split = __builtin_amdgcn_readfirstlane(seg_split);
    out_mode = __builtin_amdgcn_readfirstlane(out_mode);
    // (Not with even scheduling, whose shared-out tiles have a numbering of their own: measured, panels under it gain
    // or lose 2 %, 4 % lost on 2048 x 5120 x 13696.)
    // Tiles are numbered down the rows of a panel of `panel` row tiles, column after column, panel after panel: the
    // workgroups that run together on an XCD (consecutive numbers) then cover a block of panel x (their number / panel)
    // tiles and share both operands through its L2, instead of one or two whole columns of tiles.
    int tile_m = tile % tiles_m, tile_n = tile / tiles_m;
    if (SHORT && tile >= tiles_m * n_tiles) {          // (a column of the last row tile)
        tile_m = tiles_m;
        tile_n = tile - tiles_m * n_tiles;
    } else if (!sk_on && fu.panel > 0 && fu.panel < tiles_m) {
        const int per_panel = fu.panel * n_tiles, pn = tile / per_panel;
        const int rows_p = min(fu.panel, tiles_m - pn * fu.panel), t_in = tile - pn * per_panel;
        tile_m = pn * fu.panel + t_in % rows_p;
        tile_n = t_in / rows_p;
    }
    const int64_t m0 = (int64_t)__builtin_amdgcn_readfirstlane(tile_m) * BM;
    const bool gated = FUSED && fu.swiglu;
    // first column of the tile: of the weight rows, or of the output (= of the gate rows) when gated
    const int64_t n0 = (int64_t)__builtin_amdgcn_readfirstlane(tile_n) * (gated ? BN / 2 : BN);

    // (the thread number is made opaque to the optimiser in every segment: what is derived from it -- loader
    // offsets, epilogue rows and masks -- is then computed where it is used, not ahead of the segment loop, where it
    // would hold registers through the K loop)
    int t = KS > 1 ? (int)threadIdx.x % kThreads : (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const uint32_t fmask = frac_mask_vgpr();
    const PackedLayout<G> lay(E8 ? 2 * K : K);
    const int64_t nrb = row_blocks(N);
    const int wm = (wave / WGN) * (BM / WGM), wn = (wave % WGN) * (BN / WGN);
    // this segment's K slices [kt_begin, kt_end): whole pairs of slices (K % 128 == 0 is required by the launcher)
    const int kt_begin = __builtin_amdgcn_readfirstlane(seg_kb);
    const int kt_end = __builtin_amdgcn_readfirstlane(seg_ke);

    // ---- activation loader: 8 lanes cover one 128-byte row slice; pass p handles row RP*p + t/8.
    // Rows beyond M are clamped (their products are never stored).
    // Global reads are buffer loads: a wavefront-uniform resource (base of this tile's data, in
    // scalar registers), a scalar offset that advances with the K slice, and a 32-bit per-lane
    // offset that never changes -- no vector address arithmetic inside the K loop.
    const int a_row = t >> 3, a_piece = (t & 7) ^ ((a_row >> 1) & 7);
    const half_t* a_base = X + m0 * K;
    uint32_t a_pass_off[PA];
#pragma unroll
    for (int p = 0; p < PA; ++p)
        a_pass_off[p] = (uint32_t)((min((int64_t)(a_row + RP * p), M - 1 - m0) * K + a_piece * 8) * 2);
    // LDS position of this wavefront's eight rows (pass p adds RP rows); lane l fills the 16 bytes at 16 l
    const uint32_t a_lds_off = (uint32_t)(wave * 8 * kRowBytes);

    // ---- weight loader: operand block j of this wavefront covers rows n0 + wn + 32j .. +31
    const int b_h = lane >> 5, b_r = lane & 15;
    const int64_t rb_tile = n0 / kBlockRows;            // first row block of the tile (exists: n0 < N)
    const uint4* b_codes = packed + lay.code_index(rb_tile, 0);
    const uint32_t* b_params = reinterpret_cast<const uint32_t*>(packed) + lay.param_index(rb_tile, 0);
    const uint32_t rb_stride = (uint32_t)lay.nkb * block_bytes(G);
    uint32_t b_code_off[TN], b_param_off[TN];           // row blocks beyond N are clamped (never stored)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        int64_t rb = min(rb_tile + wn / kBlockRows + 2 * j + ((lane >> 4) & 1), nrb - 1) - rb_tile;
        if (gated) {                                    // block 0: gate rows, block 1: the up rows, N/2 further
            const int64_t nrbh = fu.n_half / kBlockRows;    // (TN = 1: those of an odd wavefront)
            rb = min(rb_tile + (TN == 2 ? wave % WGN : wave >> 1) * 2 + ((lane >> 4) & 1), nrbh - 1) - rb_tile + (TN == 2 ? j : wave & 1) * nrbh;
        }
        // 4-bit: chunk b_h of the slice; 8-bit: chunks 2 b_h and 2 b_h + 1 of the block (the second 256 bytes on)
        b_code_off[j] = (uint32_t)rb * rb_stride + (uint32_t)((E8 ? 2 * b_h : b_h) * kBlockRows + b_r) * 16;
        b_param_off[j] = (uint32_t)rb * rb_stride + (uint32_t)b_r * 4 + (G == 32 ? b_h * 64 : 0);
    }

    // ---- fragment read position: row wm + 32i + l%32 (32i rows = immediate 4096 i), piece 4h + s
    uint32_t frag_off[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
        frag_off[s] = (uint32_t)((wm + (lane & 31)) * kRowBytes + (((4 * b_h + s) ^ ((lane >> 1) & 7)) << 4));

    constexpr int NCH = E8 ? 2 : 1;                     // 16-byte chunks per lane, slice and operand block
    u32x4 bset[PD][TN][NCH];
    uint32_t pwset[PD][TN];
    half8_t fa[2][TM], fb[2][TN];

    // (slices beyond the range are requested through a resource of no bytes: the number of requests stays, memory is not read)
    auto load_a = [&](auto pa_c, int kt, uint32_t stage_off) {
        const __amdgpu_buffer_rsrc_t a_rsrc = rsrc_if(a_base, kt < kt_end);
        const uint32_t k0 = (uint32_t)kt * BK;
#pragma unroll
        for (int p = 0; p < decltype(pa_c)::value; ++p)
            load_to_lds_b128(a_rsrc, smem + stage_off + a_lds_off + p * RP * kRowBytes, a_pass_off[p], k0 * 2);
    };
    auto load_b = [&](int kt, int set) {
        const __amdgpu_buffer_rsrc_t b_code_rsrc = rsrc_if(b_codes, kt < kt_end), b_param_rsrc = rsrc_if(b_params, kt < kt_end);
        const uint32_t k0 = (uint32_t)kt * BK;
        // chunk (k0/32) of the row block's codes starts (k0/32)*256 bytes in; the parameter words of
        // group k0/G start (k0/G)*64 bytes into the row block's parameters
        // (8-bit: the slice is block k0/64 of 1 KiB with 16 parameter words)
        const int code_soff = E8 ? (int)((k0 / BK) * kBlockCodeBytes) : (int)((k0 / kCodesPerChunk) * (kBlockRows * 16));
        const int param_soff = E8 ? (int)((k0 / BK) * (kBlockRows * 4)) : (int)((k0 / G) * (kBlockRows * 4));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int c = 0; c < NCH; ++c)
                bset[set][j][c] = __builtin_amdgcn_raw_buffer_load_b128(b_code_rsrc, (int)b_code_off[j] + c * kBlockRows * 16,
                                                                        code_soff, 0);
            pwset[set][j] = __builtin_amdgcn_raw_buffer_load_b32(b_param_rsrc, (int)b_param_off[j], param_soff, 0);
        }
    };
    auto read_frags = [&](auto tm_c, uint32_t stage_off, int s, half8_t (&dst)[TM]) {
        const unsigned char* base = smem + stage_off + frag_off[s];
#pragma unroll
        for (int i = 0; i < decltype(tm_c)::value; ++i) dst[i] = *reinterpret_cast<const half8_t*>(base + i * 32 * kRowBytes);
    };
    auto dequant_frags = [&](int set, int s, half8_t (&dst)[TN]) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const half_t sc = param_scale(pwset[set][j]), bi = param_bias(pwset[set][j]);
            const half2_t s2 = {sc, sc}, b2 = {bi, bi};
            half2_t o[4];
            if (E8) {
                const uint32_t m8 = fmask | (fmask >> 4);       // 0x03FC03FC: eight fraction bits of both halves
#pragma unroll
                for (int h2 = 0; h2 < 2; ++h2) {
                    const uint32_t w8 = bset[set][j][(s >> 1) * (NCH - 1)][2 * (s & 1) + h2];
                    const uint32_t lo = (w8 & m8) | kExpBits2;
                    const uint32_t hi = (__builtin_amdgcn_alignbit(w8, w8, 8) & m8) | kExpBits2;
                    o[2 * h2] = dequant_pair(__builtin_bit_cast(half2_t, lo), b2, s2);
                    o[2 * h2 + 1] = dequant_pair(__builtin_bit_cast(half2_t, hi), b2, s2);
                }
                dst[j] = *reinterpret_cast<const half8_t*>(o);
                continue;
            }
            const uint32_t word = bset[set][j][0][s];
            if (BF) {
                // bfloat16 member: the parameter word holds bfloat16 scale and bias; w1 * scale - bias * scale in one
                // fp32 fused multiply-add per weight (both products and their difference are exact: 5, 4 and 8
                // significant bits), then the one rounding to bfloat16 -- the bits e0m4_bf16_dequant produces
                const float sf = __builtin_bit_cast(float, pwset[set][j] << 16);
                const float nb = -__builtin_bit_cast(float, pwset[set][j] & 0xFFFF0000u) * sf;
                const half2_t q[4] = {w1_pair<0>(word, fmask), w1_pair<1>(word, fmask), w1_pair<2>(word, fmask),
                                      w1_pair<3>(word, fmask)};
                bf16x2_t ob[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const floatx2 f = {__builtin_fmaf((float)q[p][0], sf, nb), __builtin_fmaf((float)q[p][1], sf, nb)};
                    ob[p] = __builtin_convertvector(f, bf16x2_t);
                }
                dst[j] = *reinterpret_cast<const half8_t*>(ob);
                continue;
            }
            o[0] = dequant_pair(w1_pair<0>(word, fmask), b2, s2);
            o[1] = dequant_pair(w1_pair<1>(word, fmask), b2, s2);
            o[2] = dequant_pair(w1_pair<2>(word, fmask), b2, s2);
            o[3] = dequant_pair(w1_pair<3>(word, fmask), b2, s2);
            dst[j] = *reinterpret_cast<const half8_t*>(o);
        }
    };

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    auto mfma_block = [&](auto tm_c, const half8_t (&a)[TM], const half8_t (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < decltype(tm_c)::value; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = BF ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[i]),
                                                                         __builtin_bit_cast(bf16x8_t, b[j]), acc[i][j], 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], b[j], acc[i][j], 0, 0, 0);
    };

    // Instruction order inside one sub-step: after every MFMA a few of the vector instructions that
    // prepare the next sub-step's operands, so that a single wavefront keeps the matrix pipe busy
    // (an MFMA of this shape occupies it for 32 cycles, its issue only for 4).
    auto interleave = [&](auto tm_c, auto vmem) {
        constexpr int TMX = decltype(tm_c)::value, kMfma = TMX * TN;
#pragma unroll
        for (int i = 0; i < kMfma; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // one MFMA
            if (i < TMX) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);      // one LDS fragment read
            __builtin_amdgcn_sched_group_barrier(0x002, TMX >= 4 ? 5 : 9, 0);       // vector ALU
            if (i < decltype(vmem)::value) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // global load
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using ITN2 = std::integral_constant<int, (1 + NCH) * TN>;      // loads issued by load_b

    // The K range on TMX of the wavefront's TM row blocks (all of them, but in a last row tile)
    auto k_loop = [&](auto tm_c) {
        using IPA = std::integral_constant<int, SHORT ? decltype(tm_c)::value * 32 / RP : PA>;
        constexpr int PAX = IPA::value, NB = ITN2::value;
        // One K slice.  On entry: stage `cur` holds slice kt; fa[0], fb[0] hold its sub-step 0 operands;
        // bset[set] holds its codes; the next PD - 1 slices' codes and the next L - 1 slices' activations are in flight.
        // (REST: one of the range's last two slices, which request nothing)
        auto step = [&](auto rest_c, int kt, int set, uint32_t cur, uint32_t nxt, uint32_t last) {
            constexpr bool REST = decltype(rest_c)::value;
            // sub-step 0: operands of sub-step 1
            read_frags(tm_c, cur, 1, fa[1]);
            dequant_frags(set, 1, fb[1]);
            mfma_block(tm_c, fa[0], fb[0]);
            interleave(tm_c, I0{});
            __builtin_amdgcn_sched_barrier(0);
            // sub-step 1: operands of sub-step 2
            read_frags(tm_c, cur, 2, fa[0]);
            dequant_frags(set, 2, fb[0]);
            mfma_block(tm_c, fa[1], fb[1]);
            interleave(tm_c, I0{});
            __builtin_amdgcn_sched_barrier(0);
            wait_loads<REST ? 0 : (L - 1) * NB + (L - 2) * PAX>();
            __builtin_amdgcn_s_barrier();   // slice kt+1 is complete in stage `nxt`, and nobody reads slice kt-1 any more
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            // sub-step 2: operands of sub-step 3 (last use of this slice's codes); activations into the stage of slice kt-1
            read_frags(tm_c, cur, 3, fa[1]);
            dequant_frags(set, 3, fb[1]);
            if (!REST) load_a(IPA{}, kt + L, last);
            mfma_block(tm_c, fa[0], fb[0]);
            interleave(tm_c, I0{});
            __builtin_amdgcn_sched_barrier(0);
            // sub-step 3: operands of the next slice's sub-step 0; this slice's code registers are free,
            // so the codes of slice kt+PD are requested into them
            if (!REST) load_b(kt + PD, set);
            read_frags(tm_c, nxt, 0, fa[0]);
            dequant_frags((set + 1) % PD, 0, fb[0]);
            mfma_block(tm_c, fa[1], fb[1]);
            interleave(tm_c, ITN2{});
            __builtin_amdgcn_sched_barrier(0);
        };

        // ---- prologue
        const uint32_t ring = (uint32_t)part * S * kStageBytes;
        // (in the order that the loop keeps up: slice kt requests activations L slices on, then codes PD slices on)
#pragma unroll
        for (int d = -(PD > L ? PD : L); d < 0; ++d) {
            if (d + L >= 0) load_a(IPA{}, kt_begin + d + L, ring + (d + L) * kStageBytes);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            if (d + PD >= 0) load_b(kt_begin + d + PD, d + PD);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_loads<(L - 1) * PAX + (PD < L ? PD : L) * NB>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_frags(tm_c, ring, 0, fa[0]);
        dequant_frags(0, 0, fb[0]);

        uint32_t so[S];                                     // stages of slices kt, kt + 1, ..., kt - 1
#pragma unroll
        for (int i = 0; i < S; ++i) so[i] = ring + i * kStageBytes;
        auto advance_ring = [&]() {                         // by two slices
            uint32_t tmp[S];
#pragma unroll
            for (int i = 0; i < S; ++i) tmp[i] = so[(i + 2) % S];
#pragma unroll
            for (int i = 0; i < S; ++i) so[i] = tmp[i];
        };
        // (K ranges are whole pairs of slices)
        int kt = kt_begin;
        for (; kt + PD <= kt_end; kt += PD) {
#pragma unroll
            for (int d = 0; d < PD; d += 2) {
                step(std::false_type{}, kt + d, d, so[0], so[1], so[S - 1]);
                step(std::false_type{}, kt + d + 1, d + 1, so[1], so[2], so[0]);
                advance_ring();
            }
        }
        if (PD == 4 && kt < kt_end) {
            step(std::true_type{}, kt, 0, so[0], so[1], so[S - 1]);
            step(std::true_type{}, kt + 1, 1, so[1], so[2], so[0]);
        }
        // (what was requested beyond the range has arrived before the stages are used otherwise)
        wait_loads<0>();
    };
    if constexpr (SHORT) {
        static_assert(PA * RP == TM * 32, "a loader pass is whole row blocks");
        if (M - m0 > 64) k_loop(std::integral_constant<int, TM>{});
        else k_loop(std::integral_constant<int, 2>{});
    } else {
        k_loop(std::integral_constant<int, TM>{});
    }
    if (KS > 1) {
        // The parts' sums are added to the first's, in the order of K, through LDS.  Parts of one pair of slices fewer wait at the
        // barriers of two steps more.
        if (kt_end - kt_begin < 2 * ((KT_all / 2 + KS - 1) / KS)) {
            __syncthreads();
            __syncthreads();
        }
        __syncthreads();                                // every wavefront has left the K loop's stages
        floatx4* sums = reinterpret_cast<floatx4*>(smem);
        constexpr int kPart = TM * TN * 4 * kThreads;
        if (part > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        sums[(part - 1) * kPart + ((i * TN + j) * 4 + q) * kThreads + t] =
                            floatx4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int s = 0; s < KS - 1; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const floatx4 v = sums[s * kPart + ((i * TN + j) * 4 + q) * kThreads + t];
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
                        }
        }
    }

    // accumulator layout of a 32x32 block: register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32
    // (n32 is made opaque to the optimiser here, after the K loop: otherwise the products of n32 with the row
    // numbers of the epilogue, invariant across the segment loop, are computed before it and held in registers
    // through the K loop: a hundred registers more, and spills in the large tile)
    uint32_t n32 = (uint32_t)N;
    asm volatile("" : "+s"(n32));
    // (KS > 1: the first part's wavefronts write the rows; gated with TN = 1, the odd wavefronts have none of their own)
    const int rows_left = KS > 1 && part > 0 ? 0 : (int)min((int64_t)BM, M - m0), cols_left = (int)min((int64_t)BN, N - n0);
    const int rows_mine = TN == 1 && gated && (wave & 1) ? 0 : rows_left;
    const int row0 = wm + 4 * (lane >> 5), col0 = wn + (lane & 31);
    const uint32_t off0 = (uint32_t)row0 * n32 + (uint32_t)col0;
    auto store_tile = [&](auto* __restrict__ dst) {     // dst: element (m0, n0) of a row-major [M, N] array
        using out_t = std::remove_reference_t<decltype(*dst)>;
        if (rows_left >= BM && cols_left >= BN) {       // a whole tile (uniform): stores without per-element masks
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int dr = 32 * i + 8 * (r >> 2) + (r & 3);
                        dst[off0 + (uint32_t)dr * n32 + 32 * j] = out_value<out_t>(acc[i][j][r]);
                    }
            return;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (col0 + 32 * j < cols_left) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int dr = 32 * i + 8 * (r >> 2) + (r & 3);
                        if (row0 + dr < rows_left) dst[off0 + (uint32_t)dr * n32 + 32 * j] = out_value<out_t>(acc[i][j][r]);
                    }
            }
        }
    };
    // Results to Y in whole 16-byte pieces of its rows, for row lengths that are a multiple of 8: the accumulators hold
    // single elements of 32 different columns, so a wavefront turns 4 KiB of them at a time around in a piece of LDS of its
    // own (the K loop's stages are free by then) and reads back eight neighbouring columns per lane.  The residual comes in
    // the same way, the next piece's while this one's is used.  Element by element, the residual's loads -- one 2-byte load
    // and one 2-byte store after the other, each masked by itself -- were a serial
    // chain of 128 round trips to memory: 2048 x 5120 x 5120 with a residual (160 large tiles) 198 us, now 144; gated 2048 x
    // 27392 x 5120 538 -> 514.  Whole tiles without a residual are stored element by element: nothing waits for those stores,
    // and turning the sums around costs 0.3 - 0.5 us at the end of a launch (1024 x 8192 x 256 10.9 us, element by element 10.5);
    // tiles that the matrix ends in need a mask per element there (1000 x 4096 x 512 10.4 us, in pieces 9.8).
    constexpr uint32_t kTurnBytes = 32 * (32 + 4) * 4;  // per wavefront: 32 x 32 or 16 x 64 sums, rows padded by 16 bytes
    static_assert(kTurnBytes >= 16 * (64 + 4) * 4 && kTurnBytes * WGM * WGN <= (uint32_t)kStages * kStageBytes, "fits the stages");
    // COLS: columns of the wavefront's results (64, or 32 gated); value(i, r, j): accumulator register r of block i (j)
    auto write_rows = [&](auto cols_c, auto value, auto* dst, const half_t* res, uint32_t ld, int wcol, int cols_valid) {
        using out_t = std::remove_reference_t<decltype(*dst)>;
        typedef out_t out8_t __attribute__((ext_vector_type(8)));
        constexpr int COLS = decltype(cols_c)::value, ROWS = 1024 / COLS, kChunks = TM * 32 / ROWS;
        constexpr int PPR = COLS / 8, RPP = 64 / PPR;   // 16-byte pieces per row, rows per pass (two passes per chunk)
        constexpr int kStride = COLS + 4, NJ = COLS / 32, NR = 16 / NJ;
        float* turn = reinterpret_cast<float*>(smem + (part * WGM * WGN + wave) * kTurnBytes);
        const int prow = lane / PPR, pcol = (lane % PPR) * 8;
        const bool col_ok = wcol + pcol < cols_valid;
        const uint32_t o0 = (uint32_t)(wm + prow) * ld + (uint32_t)(wcol + pcol);
        const int my_rows = col_ok ? rows_mine - wm - prow : 0;     // rows from this lane's first on that exist
        half8_t rs[2][2];
        auto load_res = [&](int ch) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int dr = ch * ROWS + p * RPP;
                rs[ch & 1][p] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
                if (dr < my_rows) rs[ch & 1][p] = *reinterpret_cast<const half8_t*>(res + (o0 + (uint32_t)dr * ld));
            }
        };
        __syncthreads();                                // every wavefront has left the K loop's stages
        if (res) load_res(0);
#pragma unroll
        for (int ch = 0; ch < kChunks; ++ch) {
            if (res && ch + 1 < kChunks) load_res(ch + 1);
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int rr = 0; rr < NR; ++rr)
                    turn[(8 * (rr >> 2) + 4 * (lane >> 5) + (rr & 3)) * kStride + 32 * j + (lane & 31)] =
                        value(ch * ROWS / 32, (ch * ROWS % 32) / 2 + rr, j);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int dr = ch * ROWS + p * RPP;
                const float* src = turn + (p * RPP + prow) * kStride + pcol;
                floatx4 lo = *reinterpret_cast<const floatx4*>(src), hi = *reinterpret_cast<const floatx4*>(src + 4);
                if (res) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        lo[e] += (float)rs[ch & 1][p][e];
                        hi[e] += (float)rs[ch & 1][p][4 + e];
                    }
                }
                out8_t o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] = out_value<out_t>(lo[e]);
                    o[4 + e] = out_value<out_t>(hi[e]);
                }
                if (dr < my_rows) *reinterpret_cast<out8_t*>(dst + (o0 + (uint32_t)dr * ld)) = o;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();            // the piece of LDS is read before it is written again
        }
    };
    // A shared-out K range (even scheduling): this sharer's sums go to its slab, in the order the registers hold
    // them (16 bytes per lane and store, a wavefront's stores contiguous); the sharer that arrives last adds all
    // slabs of the tile in K order and goes on to write the tile like an unshared one.
    if (kSk && out_mode == 2) {
        constexpr uint32_t kSlabStep = kThreads * 16;   // bytes between consecutive register quads of a lane
        constexpr int kCoherent = 17;                   // sc0 | sc1: written through to memory, read from memory
        uint32_t lane_off = (uint32_t)t * 16;
        asm volatile("" : "+v"(lane_off));              // (opaque, like n32: the slab offsets stay here)
        const __amdgpu_buffer_rsrc_t my_slab = make_rsrc(sk.slabs + (size_t)((int)sk_pos + sk_rt) * (size_t)(BM * BN));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const floatx4 f = {acc[i][j][4 * q4], acc[i][j][4 * q4 + 1], acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f), my_slab,
                                                           (int)(lane_off + ((i * TN + j) * 4 + q4) * kSlabStep), 0, kCoherent);
                }
        // The slab is in memory before the counter moves: every thread waits for its own stores, and after the
        // barrier one thread orders them, at device scope, ahead of its addition to the counter.  (One fence per
        // workgroup: a device-scope release writes back the XCD's whole L2, and two thousand of those, one per
        // wavefront, took longer than the tiles they shared out.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                                // (also: every wavefront has left the K loop's LDS stages)
        if (t == 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const unsigned int before = __hip_atomic_fetch_add(sk.counters + sk_rt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *reinterpret_cast<volatile int*>(smem) = before + 1 == (unsigned int)sk_sharers ? 1 : 0;
        }
        __syncthreads();
        const int last = __builtin_amdgcn_readfirstlane(*reinterpret_cast<volatile int*>(smem));
        if (!last) continue;
        // (acquire at device scope: nothing this XCD's caches may still hold of these slabs from an earlier launch is
        // used; the loads below are device-coherent besides)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        // The last sharer: the tile's slabs (its own among them) added in K order, a quarter of the registers at a
        // time -- the accumulators are not needed any more, and this way the code shares nothing with the other
        // epilogues.  The loads are device-coherent: the other sharers ran on other XCDs, whose L2 this one cannot see.
        half_t* yt = Y + m0 * N + n0;
        // (one of the wavefront's TM row blocks at a time: two at a time measured twice as slow)
        constexpr int kAtOnce = 1;
#pragma unroll 1
        for (int i0 = 0; i0 < TM; i0 += kAtOnce) {
            floatx4 sum[kAtOnce * TN * 4];
#pragma unroll
            for (int v = 0; v < kAtOnce * TN * 4; ++v) sum[v] = floatx4{0.f, 0.f, 0.f, 0.f};
            const int quad0 = __builtin_amdgcn_readfirstlane(i0 * TN * 4 * (int)kSlabStep);
            for (int sh = 0; sh < sk_sharers; ++sh) {
                const __amdgpu_buffer_rsrc_t slab = make_rsrc(sk.slabs + (size_t)(sk_first + sk_rt + sh) * (size_t)(BM * BN));
#pragma unroll
                for (int v = 0; v < kAtOnce * TN * 4; ++v) {
                    const u32x4 d = __builtin_amdgcn_raw_buffer_load_b128(slab, (int)(lane_off + v * kSlabStep), quad0, kCoherent);
                    sum[v] += __builtin_bit_cast(floatx4, d);
                }
            }
#pragma unroll
            for (int a = 0; a < kAtOnce; ++a)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int dr = 32 * (i0 + a) + 8 * q4 + e;
                            if (col0 + 32 * j < cols_left && row0 + dr < rows_left)
                                yt[off0 + (uint32_t)dr * n32 + 32 * j] = (half_t)sum[(a * TN + j) * 4 + q4][e];
                        }
        }
        continue;
    }
    // Split K in a fixed number of ranges: this work item's fp32 partial sums go to slab `split` of the workspace
    // (row-major [splits][M][N]); a second kernel adds the slabs in split order and rounds to fp16.
    if (FUSED) {
        static_assert(!FUSED || TN == 2 || (TN == 1 && WGM == 1), "the gated epilogue pairs operand blocks of a wavefront, or two wavefronts");
        if (gated) {
            const int ocols_left = (int)min((int64_t)(BN / 2), fu.n_half - n0);
            const int wcol = (TN == 2 ? wave % WGN : wave >> 1) * 32, ocol = wcol + (lane & 31);
            if (ocol < ocols_left) {
                if (out_mode == 1) {                    // partial sums keep the [M, N] layout of the weight rows
                    float* __restrict__ pg = partial + ((size_t)split * (size_t)M + (size_t)m0) * (size_t)N + (size_t)n0;
                    float* __restrict__ pu = pg + fu.n_half;
                    const uint32_t o0 = (uint32_t)row0 * n32 + (uint32_t)ocol;
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int dr = 32 * i + 8 * (r >> 2) + (r & 3);
                            if (row0 + dr < rows_left) {
                                if constexpr (TN == 2) {
                                    pg[o0 + (uint32_t)dr * n32] = acc[i][0][r];
                                    pu[o0 + (uint32_t)dr * n32] = acc[i][1][r];
                                } else {
                                    (wave & 1 ? pu : pg)[o0 + (uint32_t)dr * n32] = acc[i][0][r];
                                }
                            }
                        }
                }
            }
            if (out_mode != 1) {
                uint32_t nh32 = (uint32_t)fu.n_half;    // (a multiple of 32)
                asm volatile("" : "+s"(nh32));          // (opaque, like n32)
                if constexpr (TN == 1) {                // the up sums of an odd wavefront to the even one before it
                    floatx4* sums = reinterpret_cast<floatx4*>(smem) + (wave >> 1) * (TM * 4 * 64) + lane;
                    __syncthreads();                    // every wavefront has left the K loop's stages
                    if (wave & 1) {
#pragma unroll
                        for (int i = 0; i < TM; ++i)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                sums[(i * 4 + q) * 64] = floatx4{acc[i][0][4 * q], acc[i][0][4 * q + 1], acc[i][0][4 * q + 2], acc[i][0][4 * q + 3]};
                    }
                    __syncthreads();
                    if (!(wave & 1)) {
#pragma unroll
                        for (int i = 0; i < TM; ++i)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const floatx4 up = sums[(i * 4 + q) * 64];
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[i][0][4 * q + e] = silu_f32(acc[i][0][4 * q + e]) * up[e];
                            }
                    }
                    write_rows(std::integral_constant<int, 32>{}, [&](int i, int r, int) { return acc[i][0][r]; }, Y + m0 * fu.n_half + n0,
                               fu.residual ? fu.residual + m0 * fu.n_half + n0 : nullptr, nh32, wcol, ocols_left);
                } else
                write_rows(std::integral_constant<int, 32>{},
                           [&](int i, int r, int) { return silu_f32(acc[i][0][r]) * acc[i][1][r]; },
                           Y + m0 * fu.n_half + n0, fu.residual ? fu.residual + m0 * fu.n_half + n0 : nullptr, nh32,
                           wcol, ocols_left);
            }
            continue;
        }
        if (out_mode != 1 && fu.residual && (n32 & 7u) != 0) {
            const half_t* rt = fu.residual + m0 * N + n0;
            half_t* yt = Y + m0 * N + n0;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (col0 + 32 * j < cols_left) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int dr = 32 * i + 8 * (r >> 2) + (r & 3);
                            const uint32_t o = off0 + (uint32_t)dr * n32 + 32 * j;
                            if (row0 + dr < rows_left) yt[o] = (half_t)(acc[i][j][r] + (float)rt[o]);
                        }
                }
            }
            continue;
        }
    }
    using out_t = std::conditional_t<BF, __bf16, half_t>;
    out_t* yt = reinterpret_cast<out_t*>(Y) + m0 * N + n0;
    if (out_mode == 1)
        store_tile(partial + ((size_t)split * (size_t)M + (size_t)m0) * (size_t)N + (size_t)n0);
    else if ((n32 & 7u) == 0 && (KS > 1 || (FUSED && fu.residual) || M - m0 < BM || N - n0 < BN))
        write_rows(std::integral_constant<int, TN * 32>{}, [&](int i, int r, int j) { return acc[i][j][r]; }, yt,
                   FUSED && fu.residual ? fu.residual + m0 * N + n0 : nullptr, n32, wn, cols_left);
    else
        store_tile(yt);
  }
}

// The same with the fused epilogue: element i of the output is (m, j) with j < n_out; its sums are at
// [m, j] of the slabs (and, gated, [m, n_half + j]), whose rows are N long.
// V consecutive elements per thread (V = 4 needs n_out, N and N/2 to be multiples of 4).
template <int V>
__global__ __launch_bounds__(256) void splitk_reduce_fused_kernel(const float* __restrict__ partial, int splits,
                                                                  int64_t M, int64_t N, int64_t n_out,
                                                                  half_t* Y, PipeFusion fu)
{
    typedef float fvec __attribute__((ext_vector_type(V)));
    typedef _Float16 hvec __attribute__((ext_vector_type(V)));
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (i >= M * n_out) return;
    const int64_t m = i / n_out, j = i - m * n_out;
    const size_t slab = (size_t)M * (size_t)N;
    const float* __restrict__ src = partial + (size_t)m * (size_t)N + (size_t)j;
    fvec v = *reinterpret_cast<const fvec*>(src);
    for (int s = 1; s < splits; ++s) v += *reinterpret_cast<const fvec*>(src + (size_t)s * slab);
    if (fu.swiglu) {
        fvec up = *reinterpret_cast<const fvec*>(src + fu.n_half);
        for (int s = 1; s < splits; ++s) up += *reinterpret_cast<const fvec*>(src + (size_t)s * slab + fu.n_half);
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = silu_f32(v[e]) * up[e];
    }
    if (fu.residual) {
        const hvec r = *reinterpret_cast<const hvec*>(fu.residual + i);
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] += (float)r[e];
    }
    *reinterpret_cast<hvec*>(Y + i) = __builtin_convertvector(v, hvec);
}

// Y[i] = fp16(sum over splits, in split order, of partial[s][i]); V elements per thread.
template <int V>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int64_t count,
                                                            half_t* __restrict__ Y)
{
    typedef float fvec __attribute__((ext_vector_type(V)));
    typedef _Float16 hvec __attribute__((ext_vector_type(V)));
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (i >= count) return;
    fvec sum = *reinterpret_cast<const fvec*>(partial + i);
    for (int s = 1; s < splits; ++s) sum += *reinterpret_cast<const fvec*>(partial + (size_t)s * count + i);
    *reinterpret_cast<hvec*>(Y + i) = __builtin_convertvector(sum, hvec);
}

// K splits: none when the tiles alone give every compute unit work, else the number the estimate below puts ahead,
// up to kMaxSplits, each split keeping at least kMinPairsPerSplit pairs of K slices.
constexpr int kComputeUnits = 256;
constexpr int kMinPairsPerSplit = 4;
constexpr int kMaxSplits = 8;

// The tile a problem gets (gemm_variant 2, 3, 4, 5, 6 force the 256 x 256, 128 x 128, 64 x 256, 128 x 256 and 64 x 128 tile) and
// whether the large tile runs with even scheduling (SkArgs; gemm_sk 1 forces it whenever the last round is partly
// filled, 2 forbids it) are decided by an estimate of the launch's duration.  Up to 64 rows only the tiles of 64 rows
// make sense.  The 128 x 256 tile has the large tile's wavefront (128 x 64, 3.75 vector instructions per MFMA) in workgroups
// of four, two to a compute unit, that start and finish independently: it pads fewer rows than the large tile,
// dequantises half as often as the flat one and leaves a shorter tail (354 x 13056 x 10368: 111 us against 138 and
// 146; 2048 x 27392 x 4096: 397 against 421 with even scheduling).  The tiles of 128 columns have wavefronts of half the width
// (64 x 32 and 128 x 32, an operand of X read for every MFMA): twice as many workgroups where tiles are few, each with half the
// work per slice, so that fewer splits do or none (317 x 2560 x 2048 on 64 x 256 tiles in splits 16.9 us, on 64 x 128 tiles unsplit 12.9;
// 1024 x 4096 x 4096 on 128 x 256 in two splits 45.7, on 128 x 128 unsplit 39.7; 64 x 4096 x 13696 in eight splits 27.3 and 19.1).
//
// The estimate counts rounds: the work items (tiles times K splits) run `cap` at a time (one 256 x 256 tile per
// compute unit, two of the others, four of the smallest), a full round takes  pairs-of-K-slices * a(1) + b  and the last, partly filled
// one  pairs * a(fill) + b  with a() piecewise linear in the fill -- a compute unit is slower the more of them run
// (one round of 160 large tiles with K = 5120 takes 112 us, one of 256 tiles 152 us, whether the workgroups read
// different tiles or all the same one: it is not the memory side), which is why filling idle units buys much less
// than their number suggests; a() has a step where the first compute units get a second workgroup, at half fill (at a quarter for the
// 64 x 128 tile: gated 297 x 6656 x 6656, 260 such tiles, 50.7 us, on 128 x 256 tiles 41.1).
// A K split adds its reduction kernel (a fixed part and one per MB of partial sums), and the number of splits is the
// one with the shortest estimate; even scheduling runs its whole rounds like whole tiles and the shared-out rest on
// every unit at the full rate, and adds the slabs' cost, of which the part per sharer of a tile is serial (the last
// arriver reads them all).
// The constants are a least-squares fit (logarithm of the ratio to the measurement, rms 5.1 %) to 12893 timings of 608
// problems -- M = 17 .. 8192, N = 1024 .. 20480, K = 1024 .. 14336, groups of 128, random ones and the layer shapes of 6B and 14B models --
// on two cards, each timed with the five tiles, one to eight K splits, and with even scheduling, on weights out of cache.  Choosing by
// the estimate costs 0.6 % over always choosing the measured best on the one card and 1.4 - 2.1 % on the other (geometric means), where
// split launches on tiles of 128 columns take up to 28 % longer than on the first; up to 64 rows 6 %, above 384 0.5 %.  Without the tiles of 128
// columns the best would be 2.3 - 4.0 % slower (up to 64 rows 11 - 16 %).  tune_gemm_estimate.py of the Python package times and fits in
// this way.
struct PipeTile {
    int bm, bn;
};
constexpr PipeTile kFlatTile{64, 256}, kMidTile{128, 128}, kBigTile{256, 256}, kHalfTile{128, 256}, kNarrowTile{64, 128};
constexpr int kFlatOnlyMaxM = 64;

// The gated product's epilogue takes longer than the plain one, the exchange of gate and up sums between wavefronts of 128-column tiles
// longest: 1.4 and 2.4 us for every workgroup that a compute unit has, on tiles of 256 columns 0.6 - 1.6.  On 498 gated calls of 65 to 900 rows
// and 256 to 5000 weights a row the choice among whole tiles costs 0.2 - 0.6 % over the best, without these costs 3.6 - 4.1 %
// (683 x 9408 x 384 in 8-bit codes 14.5 us on 64 x 128 tiles, 11.8 on 64 x 256).
struct TileCost {
    double lo[4];                                       // us per pair of K slices at fill 0, 1/8, 1/4, 1/2 of a round ...
    double past;                                        // ... just above 1/4 ...
    double hi[3];                                       // ... and just above 1/2, at 3/4 and 1
    double b;                                           // us per round: prologue and epilogue of a work item
    int cap;                                            // work items per round
    double gated;                                       // us more per workgroup of a compute unit for the gated product's epilogue
};
constexpr TileCost kFlatCost{{0.821, 0.866, 0.887, 1.113}, 0.887, {1.604, 1.867, 1.868}, 3.74, 2 * kComputeUnits, 1.0};
constexpr TileCost kHalfCost{{1.114, 1.174, 1.222, 1.713}, 1.222, {2.513, 2.919, 3.212}, 6.07, 2 * kComputeUnits, 0.6};
constexpr TileCost kBigCost{{2.008, 2.046, 2.094, 2.227}, 2.094, {2.220, 2.730, 3.313}, 7.35, kComputeUnits, 1.6};
constexpr TileCost kNarrowCost{{0.505, 0.549, 0.628, 1.162}, 0.847, {1.393, 1.858, 2.078}, 3.33, 4 * kComputeUnits, 1.35};
constexpr TileCost kMidCost{{0.683, 0.726, 0.761, 0.988}, 0.761, {1.391, 1.660, 1.840}, 4.29, 2 * kComputeUnits, 2.4};
constexpr double kReduceUs = 4.23, kReduceUsPerMB = 0.211;      // reduction kernel of a K split
constexpr double kSkUs = 39.1, kSkUsPerSharer = 0.86;           // even scheduling: slabs, and the serial part per sharer
// 8-bit codes, twice the registers per slice and twice the bytes: 128-row tiles request codes two slices ahead instead of four, and those of
// 128 columns, a wavefront to a SIMD, wait for them.  A fit of their own to 13181 timings of 622 problems (rms 6.7 %): the choice
// costs 1.0 - 2.4 % over the best, by the costs of 4-bit codes 2.4 - 4.2 % (gated 192 x 11712 x 7808, 184 tiles of 128 x 128, 79.8 us, on
// 64 x 256 tiles 61.9).
constexpr TileCost kFlatCost8{{0.789, 0.877, 0.917, 1.203}, 0.917, {1.773, 2.006, 2.045}, 4.88, 2 * kComputeUnits, 0.9};
constexpr TileCost kHalfCost8{{1.266, 1.351, 1.392, 1.898}, 1.392, {2.739, 3.236, 3.436}, 5.85, 2 * kComputeUnits, 0.8};
constexpr TileCost kBigCost8{{2.225, 2.287, 2.356, 2.515}, 2.356, {2.499, 2.965, 3.553}, 5.99, kComputeUnits, 2.6};
constexpr TileCost kNarrowCost8{{0.518, 0.598, 0.698, 1.326}, 1.053, {1.570, 2.062, 2.250}, 3.75, 4 * kComputeUnits, 1.35};
constexpr TileCost kMidCost8{{0.988, 1.134, 1.163, 1.244}, 1.163, {1.487, 1.892, 1.981}, 4.21, 2 * kComputeUnits, 2.2};
constexpr double kReduceUs8 = 4.42, kReduceUsPerMB8 = 0.245;
struct Estimate {
    TileCost flat, half, big, narrow, mid;
    double reduce_us, reduce_us_per_mb, sk_us, sk_us_per_sharer;
    bool all_tiles;                                     // with the tiles of 128 columns, and a short last row tile counted as such
    int short_rounds = 1 << 20;                         // rounds of a launch up to which a short row of tiles counts less than a whole one
    bool gated = false;                                 // for a call with the gated product
};
constexpr Estimate kNow{kFlatCost, kHalfCost, kBigCost, kNarrowCost, kMidCost, kReduceUs, kReduceUsPerMB, kSkUs, kSkUsPerSharer, true};
constexpr Estimate kNow8{kFlatCost8, kHalfCost8, kBigCost8, kNarrowCost8, kMidCost8, kReduceUs8, kReduceUsPerMB8, kSkUs, kSkUsPerSharer, true, 2};
// The workspace that callers are asked for, and with it the most K splits that a launch may have, come from an estimate with
// constants that stay as they are, whatever becomes of the kernel: a size once asked for is enough for good.  Calls of up to 64 rows
// with a residual or the gated product have exactly its number of splits: with another one their sums, and the residual streams that
// they feed, would be rounded otherwise.
constexpr Estimate kSizes{{{0.809, 1.173, 1.302, 1.456}, 1.302, {1.601, 2.034, 1.971}, 4.39, 2 * kComputeUnits, 0.0},
                          {{1.427, 1.531, 1.573, 1.894}, 1.573, {2.592, 3.118, 3.411}, 5.92, 2 * kComputeUnits, 0.0},
                          {{2.052, 2.302, 2.454, 2.523}, 2.454, {2.445, 2.908, 3.461}, 9.34, kComputeUnits, 0.0},
                          kNarrowCost, kMidCost,        // (not among its tiles)
                          4.87, 0.176, 34.7, 0.68, false};
// Those calls choose between the two tiles of 64 rows only, by costs of their own: on 240 calls in 4- and 8-bit codes 0.3 - 1.0 % over the
// better tile on two cards, with the costs above 0.15 - 1.8 %; on 202 gated ones in whole tiles, of 128 weights a row and more, 0.06 - 0.3 %, without the
// gated costs 3.5 - 4.2 % (39 x 36096 x 128 7.2 us on 64 x 128 tiles, 5.8 on 64 x 256).
constexpr Estimate kFewFused{{{0.800, 0.868, 0.905, 1.150}, 0.905, {1.662, 1.908, 2.013}, 2.99, 2 * kComputeUnits, 1.0}, kHalfCost, kBigCost,
                             {{0.551, 0.515, 0.747, 1.243}, 0.747, {1.388, 1.925, 2.255}, 2.73, 4 * kComputeUnits, 1.35}, kMidCost,
                             4.38, 0.184, kSkUs, kSkUsPerSharer, true};
constexpr int kSplitMajorMinPairs = 16;
constexpr int kSkMinTiles = 128;                        // fewer tiles: the fixed K split (the fit holds no such launch)

double rounds_us(const TileCost& c, int64_t items, double pairs_per_item)
{
    const int64_t full = items / c.cap, rem = items % c.cap;
    double t = (double)full * (pairs_per_item * c.hi[2] + c.b);
    if (rem > 0) {
        const double fill = (double)rem / (double)c.cap;
        double a;
        if (fill <= 0.125) a = c.lo[0] + (c.lo[1] - c.lo[0]) * fill * 8.0;
        else if (fill <= 0.25) a = c.lo[1] + (c.lo[2] - c.lo[1]) * (fill - 0.125) * 8.0;
        else if (fill <= 0.5) a = c.past + (c.lo[3] - c.past) * (fill - 0.25) * 4.0;
        else if (fill <= 0.75) a = c.hi[0] + (c.hi[1] - c.hi[0]) * (fill - 0.5) * 4.0;
        else a = c.hi[1] + (c.hi[2] - c.hi[1]) * (fill - 0.75) * 4.0;
        t += pairs_per_item * a + c.b;
    }
    return t;
}

// `tiles` whole tiles (splits = 1), or each in `splits` K ranges followed by the reduction kernel
double split_launch_us(const Estimate& e, const TileCost& c, int64_t tiles, int splits, int64_t M, int64_t N, int64_t K)
{
    double us = rounds_us(c, tiles * splits, (double)(K / (2 * BK)) / splits);
    if (splits > 1) us += e.reduce_us + e.reduce_us_per_mb * (double)splits * (double)M * (double)N * 4e-6;
    else if (e.gated) us += c.gated * (double)(tiles / c.cap * (c.cap / kComputeUnits) + (tiles % c.cap + kComputeUnits - 1) / kComputeUnits);
    return us;
}

const TileCost& cost_of(const Estimate& e, const PipeTile& t)
{
    if (t.bn == 128) return t.bm == 64 ? e.narrow : e.mid;
    return t.bm == 64 ? e.flat : t.bm == 256 ? e.big : e.half;
}

// The number of K splits of a launch with the tile `t`, at most `most` (gemm_splits forces one).  Which number pays depends on the
// tile count as much as on K: 1024 x 4096 x 4096 on 128 tiles of 128 x 256 takes 56 us unsplit, 44.6 in two splits
// (one work item per compute unit) and 53 in four; 256 x 4096 x 13696 on 32 such tiles 177, 95, 55 and 41 us in one,
// two, four and eight.
int choose_splits(const Estimate& e, const PipeTile& t, int64_t tiles, int64_t M, int64_t N, int64_t K, int64_t most)
{
    const int forced = knob(Knob::gemm_splits);
    const int64_t pairs = K / (2 * BK);
    if (forced > 0) return (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(forced, pairs), kMaxSplits));   // tests: down to one pair per split
    // every compute unit already has a tile (of the smallest, two): the partial sums and their reduction cost more than further
    // workgroups per unit gain
    const TileCost& c = cost_of(e, t);
    if (tiles >= std::max(kComputeUnits, c.cap / 2) || tiles <= 0) return 1;
    const int max_splits = (int)std::min<int64_t>(std::min<int64_t>(pairs / kMinPairsPerSplit, kMaxSplits), most);
    int best = 1;
    // (a tie is the whole tiles': 2048 x 5120 x 13696 on large tiles 267 us, in three splits, which the estimate puts 0.3 % ahead, 272)
    double best_us = split_launch_us(e, c, tiles, 1, M, N, K) / (e.all_tiles ? 1.01 : 1.0);
    for (int sp = 2; sp <= max_splits; ++sp) {
        const double us = split_launch_us(e, c, tiles, sp, M, N, K);
        if (us < best_us) {
            best_us = us;
            best = sp;
        }
    }
    return best;
}

// (gated calls have as many: halves of bn / 2 columns of the N / 2, and N is even)
int64_t pipe_tiles(const PipeTile& t, int64_t M, int64_t N) { return ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

constexpr int64_t kShortMaxTiles = 6;                   // row tiles of a launch with a short last one (see the kernel)
bool short_last(const PipeTile& t, int64_t M, int64_t tiles, int splits)
{
    const int64_t m_tiles = (M + t.bm - 1) / t.bm;
    return t.bm == 128 && t.bn == 256 && splits == 1 && m_tiles > 1 && m_tiles <= kShortMaxTiles && tiles >= kComputeUnits &&
           M % t.bm != 0 && M % t.bm <= 64;
}

// whole tiles (a short last row tile counts as 0.6, but more tiles than compute units stay more: the first of them have two workgroups,
// whatever the last one's rows; gated 288 x 23296 x 640, 273 tiles, 18.3 us, on 64 x 256 tiles 14.7.  8-bit codes of more than two rounds
// are bound by the codes, which a short tile reads as a whole one does: gated 142 x 200192 x 1920, 1564 tiles, 207 us, on 64 x 256 tiles
// 182; on 114 calls with such a row the choice costs 1.3 % over the best whole tiles, 1.7 % without this line), or `splits` K ranges of
// each and the reduction kernel
double tile_launch_us(const Estimate& e, const PipeTile& t, int splits, int64_t M, int64_t N, int64_t K)
{
    int64_t tiles = pipe_tiles(t, M, N);
    if (e.all_tiles && short_last(t, M, tiles, splits) && tiles <= (int64_t)e.short_rounds * cost_of(e, t).cap) {
        const int64_t less = tiles - tiles / ((M + t.bm - 1) / t.bm) * 2 / 5;
        tiles = tiles > kComputeUnits ? std::max<int64_t>(less, kComputeUnits + 1) : less;
    }
    return split_launch_us(e, cost_of(e, t), tiles, splits, M, N, K);
}

// even scheduling of `tiles` large tiles, of which `rem` are shared out
double sk_launch_us(const Estimate& e, int64_t tiles, int64_t rem, int64_t pairs)
{
    const double sharers = std::min<double>((double)kComputeUnits / (double)rem + 1.0, (double)pairs);
    const double whole_rounds = (double)(tiles / kComputeUnits) * ((double)pairs * e.big.hi[2] + e.big.b);
    return whole_rounds + (double)rem * (double)pairs / kComputeUnits * e.big.hi[2] + e.big.b + e.sk_us + e.sk_us_per_sharer * sharers;
}

constexpr size_t kSkCounterBytes = 1024;                // 255 counters at most, then the slabs (16-byte aligned)
struct SkPlan {
    bool on;
    int rounds_dp, rem_tiles, pairs;
    size_t workspace_bytes;
    double us;                                          // estimated duration of the launch when on
};

// With M = 2048, G = 128: N = 27392, K = 5120 (856 tiles) 547 -> 525 us; N = 5120, K = 13696 (160 tiles) 293 -> 275 us;
// but N = 5120, K = 5120 (160 tiles) 113 -> 133 us and N = 15360, K = 5120 (480 tiles) 286 -> 316 us.  (Shared tiles
// taken row by row, see the kernel; column by column the first two were 525 and 284.)
SkPlan sk_plan(const Estimate& e, const PipeTile& t, int64_t tiles, int64_t K, size_t room)
{
    SkPlan p{false, 0, 0, 0, 0, 0.0};
    const int forced = knob(Knob::gemm_sk);
    if (room == 0 || forced == 2 || t.bm != 256 || tiles <= 0) return p;
    p.rounds_dp = (int)(tiles / kComputeUnits);
    p.rem_tiles = (int)(tiles % kComputeUnits);
    p.pairs = (int)(K / (2 * BK));
    if (p.rem_tiles == 0 || tiles > 0x3fffffffLL || p.pairs > 8192) return p;      // (the kernel's unit arithmetic is 32-bit)
    p.us = sk_launch_us(e, tiles, p.rem_tiles, p.pairs);
    if (forced != 1) {
        if (tiles < kSkMinTiles) return p;
        if (p.us >= rounds_us(e.big, tiles, (double)p.pairs)) return p;
    }
    p.workspace_bytes = kSkCounterBytes + (size_t)(kComputeUnits + p.rem_tiles) * (size_t)t.bm * t.bn * sizeof(float);
    p.on = p.workspace_bytes <= room;
    return p;
}

// Whole flat tiles (the bfloat16 member: no workspace, hence no K split) that leave compute units with one workgroup of four
// wavefronts or none run as workgroups of eight, whose halves take one half of K each and add their sums in LDS: two
// wavefronts per SIMD hide each other's waits.  M = 700: 4096 x 13696 (176 tiles) 151 -> 114 us, 4608 x 4096 (198) 50 -> 42;
// M = 100: 27392 x 4096 (214) 54 -> 44, 4096 x 4096 (32) 46 -> 35.  With more tiles than compute units there are two
// workgroups per unit anyway, and two of the larger ones do not fit: M = 700, 27392 x 4096 (1177) 205 -> 219.
// On shorter rows the longer start and the exchange of the sums cost more than they give: M = 512, N = 8192 (256 tiles) at K =
// 256 8.8 us against 7.5, at 768 12.6 against 12.5, at 1024 15.1 against 14.9, but at 1536 19.0 against 20.2.
constexpr int64_t kHalvesMinK = 18 * BK;
bool k_halves(const PipeTile& t, int64_t M, int64_t N, int64_t K)
{
    return t.bm == 64 && t.bn == 256 && K >= kHalvesMinK && ((M + 63) / 64) * ((N + 255) / 256) <= kComputeUnits;
}
// (whatever the number of tiles: a compute unit has two wavefronts per SIMD or none.  As fitted to the cases above, when activations came
// through registers; on 163 calls the launches take 0.87 of it now, and on 195 the choice of a tile costs 1.1 % over the best)
constexpr double kHalvesUsPerPair = 1.1;                // us per pair of K slices of the whole K

// Fused calls of up to 64 rows in four K splits, to the same bits without partial sums in memory: workgroups of eight wavefronts on
// 64 x 128 tiles, a pair of wavefronts to a quarter of K each, whose sums are added in LDS in the order of the splits.  One
// workgroup fits a compute unit, so there have to be nearly as many tiles as units, and not more.  Against the splits, gated, at M = 20, 33, 45
// and 64 (us): 27392 x 4096 30.5, 33.4, 33.9, 36.9 -> 29.3, 30.2, 29.9, 30.7; 32768 x 2048 25.7, 25.0, 26.7, 30.8 -> 17.8, 22.2, 22.6, 22.8;
// 30720 x 11008 66.0, 67.5, 69.5, 72.8 -> 64.4, 65.8, 66.6, 66.9.  With fewer tiles 64 x 128 tiles in splits are the
// better ones (128 tiles, 16384 x 2048 at M = 64 18.5 and 16.8), with more the second round (288 tiles, 36864 x 3072, 1.2 - 1.35 x the splits' time).
// Rows of Y that are no multiple of 8 long are written by a quarter of the wavefronts element by element (27356 x 4096 at M = 45 33.5
// -> 36.5), and 8-bit codes gain nothing up to 48 rows (27392 x 4096 at M = 30 37.1 and 38.2): both keep the splits.
// gemm_variant 7 takes these tiles whatever their number.
constexpr int64_t kQuartersMinTiles = 160;
bool k_quarters(int splits, int64_t M, int64_t N)
{
    const int64_t tiles = pipe_tiles(kNarrowTile, M, N);
    const int v = knob(Knob::gemm_variant);
    return splits == 4 && N % 8 == 0 && (v == 7 || (v == 0 && tiles >= kQuartersMinTiles && tiles <= kComputeUnits));
}

size_t partial_bytes(int splits, int64_t M, int64_t N) { return (size_t)splits * (size_t)M * (size_t)N * sizeof(float); }

PipeTile tile_of(int bm, int bn)
{
    if (bm == 64) return bn == 128 ? kNarrowTile : kFlatTile;
    return bm == 256 ? kBigTile : bn == 256 ? kHalfTile : kMidTile;
}

struct PipePlan {
    PipeTile tile;
    int splits;
    SkPlan sk;
    size_t room;                                        // workspace that the call has to bring
    bool quarters;                                      // four K parts in each workgroup
    size_t bytes(int64_t M, int64_t N) const { return sk.on ? sk.workspace_bytes : splits > 1 ? partial_bytes(splits, M, N) : 0; }
};

// What a call's launch is: whole tiles without a workspace, else at most `splits` K splits (`exactly`: that many), the even
// scheduling in `sk_room` bytes or not at all (0).
struct PipeRules {
    bool whole_tiles, exactly;
    int64_t splits;
    size_t sk_room;
};

// The tile with the shortest estimate, up to 64 rows one of 64 rows.
PipePlan shortest(const Estimate& e, int64_t M, int64_t N, int64_t K, const PipeRules& r)
{
    auto splits_of = [&](const PipeTile& t) -> int {
        if (r.whole_tiles) return 1;
        if (r.exactly && knob(Knob::gemm_splits) == 0) return (int)r.splits;
        return choose_splits(e, t, pipe_tiles(t, M, N), M, N, K, r.splits);
    };
    auto plan_of = [&](const PipeTile& t) -> PipePlan {
        PipePlan p{t, 1, sk_plan(e, t, pipe_tiles(t, M, N), K, r.sk_room), 0, false};
        if (!p.sk.on) p.splits = splits_of(t);
        return p;
    };
    switch (knob(Knob::gemm_variant)) {
        case 2: return plan_of(kBigTile);
        case 3: return plan_of(kMidTile);
        case 4: return plan_of(kFlatTile);
        case 5: return plan_of(kHalfTile);
        case 6: return plan_of(kNarrowTile);
        default: break;
    }
    if (N <= 0 || K < 2 * BK) return plan_of(kFlatTile);
    PipeTile best = kFlatTile;
    double best_us = r.whole_tiles && k_halves(kFlatTile, M, N, K) ? (double)(K / (2 * BK)) * kHalvesUsPerPair + e.flat.b
                                                                   : tile_launch_us(e, kFlatTile, splits_of(kFlatTile), M, N, K);
    auto consider = [&](const PipeTile& t) {
        const double us = tile_launch_us(e, t, splits_of(t), M, N, K);
        if (us < best_us) {
            best = t;
            best_us = us;
        }
    };
    if (e.all_tiles) consider(kNarrowTile);
    if (M > kFlatOnlyMaxM) {
        if (e.all_tiles) consider(kMidTile);
        consider(kHalfTile);
        consider(kBigTile);
        const SkPlan sk = sk_plan(e, kBigTile, pipe_tiles(kBigTile, M, N), K, r.sk_room);
        if (sk.on && sk.us < best_us) best = kBigTile;
    }
    return plan_of(best);
}

// (fused matmuls and the 8-bit format have whole tiles or the fixed K split, `sk` false.  With a knob set a launch has what it asks
// for, and the room for it.)
size_t pipe_room(int64_t M, int64_t N, int64_t K, bool sk, PipePlan* plan)
{
    const bool steered = (knob(Knob::gemm_variant) && knob(Knob::gemm_variant) != 7) || knob(Knob::gemm_splits) || knob(Knob::gemm_sk);
    const PipePlan p = shortest(steered ? kNow : kSizes, M, N, K, PipeRules{false, false, kMaxSplits, sk ? ~(size_t)0 : 0});
    if (plan) *plan = p;
    return p.bytes(M, N);
}

PipePlan pipe_plan(const Fusion& f, int64_t M, int64_t N, int64_t K, bool fused, bool e8)
{
    PipePlan p;
    const bool sk = !fused && !e8;
    const size_t room = pipe_room(M, N, K, sk, &p);
    const bool steered = (knob(Knob::gemm_variant) && knob(Knob::gemm_variant) != 7) || knob(Knob::gemm_splits) || knob(Knob::gemm_sk);
    if (!steered) {
        const bool exactly = fused && M <= kFlatOnlyMaxM && (f.residual || f.swiglu);
        Estimate e = exactly ? kFewFused : e8 ? kNow8 : kNow;
        e.gated = f.swiglu;
        p = shortest(e, M, N, K, PipeRules{false, exactly, exactly ? p.splits : std::max<int64_t>(1, (int64_t)(room / partial_bytes(1, M, N))),
                                           sk ? room : 0});
    }
    if (fused && !e8 && M <= kFlatOnlyMaxM && k_quarters(p.splits, M, N)) {
        p.tile = kNarrowTile;
        p.splits = 1;
        p.quarters = true;
    }
    p.room = room;
    return p;
}

__global__ void zero_u32_kernel(unsigned int* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

template <int G, int WGM, int WGN, bool FUSED, int BM, int BN, bool E8 = false, bool BF = false, int KS = 1>
int launch_pipe(const half_t* x, int64_t M, const uint4* c, int64_t N, int64_t K, half_t* y, void* workspace,
                size_t workspace_bytes, hipStream_t stream, const Fusion& f, const PipePlan& plan)
{
    PipeFusion fu;
    fu.residual = static_cast<const half_t*>(f.residual);
    fu.swiglu = f.swiglu ? 1 : 0;
    // Panels of four row tiles (two of the large tile): 2 to 7 % faster than whole columns of tiles from M = 2048 on (2048 x 27392 x 5120 on
    // 128 x 256 tiles: 504 -> 488 us, 2048 x 32768 x 2048: 269 -> 251; on 64 x 256 tiles 601 -> 569 and 318 -> 285; on
    // the large tile 550 -> 541 and 270 -> 254); heights of 2 to 6 tiles of 128 rows measured alike.
    // gemm_panel forces a height, -1 whole columns.
    const int panel_knob = knob(Knob::gemm_panel);
    fu.panel = panel_knob > 0 ? panel_knob : panel_knob < 0 ? 0 : BM == 256 ? 2 : 4;
    fu.split_major = 0;
    fu.n_half = N / 2;
    const PipeTile shape = tile_of(BM, BN);
    const int64_t m_tiles = (M + BM - 1) / BM;
    const int64_t tiles = pipe_tiles(shape, M, N), n_tiles = tiles / m_tiles;
    const SkPlan& skp = plan.sk;
    const int splits = plan.splits;
    if (tiles * splits > 0x3fffffffLL) return E0M4_ERR_SHAPE;
    // Long K ranges gain from the order by split (1024 x 4096 x 13696 in four splits 122 -> 116 us, 512 x 2048 x 16384
    // in eight 46.9 -> 44.6), short ones lose (128 x 4608 x 4096 in eight splits of four pairs 19.6 -> 21.6, 1024 x 4608
    // x 4096 in three of ten or eleven 56.9 -> 58.5); gemm_split_order 1 forces the order by tile, 2 the order by split.
    const int order_knob = knob(Knob::gemm_split_order);
    fu.split_major = splits > 1 && (order_knob == 2 || (order_knob == 0 && K / (2 * BK) / splits >= kSplitMajorMinPairs)) ? 1 : 0;
    const int total = (int)(tiles * splits);
    const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
    float* partial = nullptr;
    if (plan.room > 0 && (workspace == nullptr || workspace_bytes < plan.room)) return E0M4_ERR_WORKSPACE;
    if (splits > 1) partial = static_cast<float*>(workspace);
    SkArgs sk{0, 0, 0, 0, nullptr, nullptr};
    unsigned grid = (unsigned)(per_xcd * kNumXcd);
    const bool last_short = short_last(shape, M, tiles, splits);
    if (last_short) grid = (unsigned)((((m_tiles - 1) * n_tiles + kNumXcd - 1) / kNumXcd + (n_tiles + kNumXcd - 1) / kNumXcd) * kNumXcd);
    if (skp.on) {
        sk.enabled = 1;
        sk.rounds_dp = skp.rounds_dp;
        sk.rem_tiles = skp.rem_tiles;
        sk.pairs = skp.pairs;
        sk.counters = static_cast<unsigned int*>(workspace);
        sk.slabs = reinterpret_cast<float*>(static_cast<char*>(workspace) + kSkCounterBytes);
        grid = kComputeUnits;
        hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(256), 0, stream, sk.counters, skp.rem_tiles);
        const int zrc = check_launch();
        if (zrc != E0M4_OK) return zrc;
    }
    // 128 KiB for the large tile: above the default limit.  (KS > 1: as many rings; the other parts' sums, afterwards.)
    constexpr size_t lds = std::max((size_t)KS * kStages * BM * kRowBytes, (size_t)(KS - 1) * BM * BN * sizeof(float));
    constexpr int per_unit = KS > 1 || BM == 256 ? 1 : BM == 64 && BN == 128 ? 4 : 2;      // as TileCost::cap counts on
    static_assert(lds * per_unit <= 160 * 1024, "LDS of a compute unit");
    auto launch = [&](auto kernel, std::atomic<uint64_t>& lds_allowed) -> int {
        const int arc = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)lds, lds_allowed);
        if (arc != E0M4_OK) return arc;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * WGM * WGN * KS), lds, stream, x, M, c, N, K, y, (int)m_tiles, (int)n_tiles, splits,
                           partial, fu, sk);
        return check_launch();
    };
    if constexpr (BM == 128 && BN == 256) {
        static std::atomic<uint64_t> lds_allowed{0};
        if (last_short) return launch(&gemm_pipe_kernel<G, WGM, WGN, FUSED, BM, BN, E8, BF, KS, true>, lds_allowed);
    }
    static std::atomic<uint64_t> lds_allowed{0};
    int rc = E0M4_OK;
    // 8-bit codes of up to 64 rows in splits that make a work item per compute unit or fewer: codes two slices ahead instead of four,
    // a shorter start (gated 16384 x 2048 at M = 20 and 64 20.6 -> 18.4 and 24.0 -> 21.9 us, 8192 x 8192 28.7 -> 26.2; with more items the
    // longer lead is the better one, 22016 x 3072 at M = 50 28.5 and 30.1).  Above 64 rows, on 40 calls against the kernel that had two slices
    // ahead everywhere, these tiles take 0.64 - 0.98 of its time on rows of 1536 weights and more; on rows of up to 768 with more tiles than compute units
    // 1.02 - 1.07, but there other tiles are chosen and the calls take 0.75 - 1.04.
    bool two_ahead = false;
    if constexpr (E8 && FUSED && BM == 64 && BN == 256) {
        static std::atomic<uint64_t> allowed{0};
        two_ahead = M <= kFlatOnlyMaxM && splits > 1 && total <= kComputeUnits;
        if (two_ahead) rc = launch(&gemm_pipe_kernel<G, WGM, WGN, FUSED, BM, BN, E8, BF, KS, false, 2>, allowed);
    }
    if (!two_ahead) rc = launch(&gemm_pipe_kernel<G, WGM, WGN, FUSED, BM, BN, E8, BF, KS>, lds_allowed);
    if (rc != E0M4_OK || splits == 1) return rc;
    if (FUSED) {
        const int64_t n_out = f.swiglu ? N / 2 : N;
        if (n_out % 4 == 0 && N % 8 == 0)
            hipLaunchKernelGGL(splitk_reduce_fused_kernel<4>, dim3((unsigned)((M * n_out / 4 + 255) / 256)), dim3(256), 0,
                               stream, partial, splits, M, N, n_out, y, fu);
        else
            hipLaunchKernelGGL(splitk_reduce_fused_kernel<1>, dim3((unsigned)((M * n_out + 255) / 256)), dim3(256), 0,
                               stream, partial, splits, M, N, n_out, y, fu);
        return check_launch();
    }
    const int64_t count = M * N;
    if (count % 4 == 0)                                 // slabs stay 16-byte aligned
        hipLaunchKernelGGL(splitk_reduce_kernel<4>, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, stream,
                           partial, splits, count, y);
    else
        hipLaunchKernelGGL(splitk_reduce_kernel<1>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream,
                           partial, splits, count, y);
    return check_launch();
}

}  // namespace

bool gemm_pipe_supported(int64_t K) { return K >= 128 && (K % (2 * BK)) == 0; }

size_t gemm_pipe_workspace_bytes(int64_t M, int64_t N, int64_t K, bool swiglu, bool fused)
{
    if (M <= 0 || N <= 0 || !gemm_pipe_supported(K)) return 0;
    PipePlan p;
    const size_t room = pipe_room(M, N, K, !fused && !swiglu, &p);
    if (!swiglu || N % 2 == 0) return room;
    // (such calls are refused; their size is that of splits of whole pairs of columns)
    const int splits = choose_splits(kSizes, p.tile, pipe_tiles(p.tile, M, N - 1), M, N, K, kMaxSplits);
    return splits > 1 ? partial_bytes(splits, M, N) : 0;
}

namespace {

// the kernel instance of a tile
template <int G, bool FUSED, bool E8 = false, bool BF = false>
int launch_pipe_as(const PipePlan& p, const half_t* x, int64_t M, const uint4* c, int64_t N, int64_t K, half_t* y,
                   void* workspace, size_t workspace_bytes, hipStream_t stream, const Fusion& f)
{
    const PipeTile& t = p.tile;
    if constexpr (BF) {
        if (k_halves(t, M, N, K))
            return launch_pipe<G, 1, 4, FUSED, 64, 256, E8, BF, 2>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
    }
    if constexpr (FUSED && !E8) {
        if (p.quarters) return launch_pipe<G, 1, 2, FUSED, 64, 128, E8, BF, 4>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
    }
    if (t.bm == 64 && t.bn == 128)
        return launch_pipe<G, 1, 4, FUSED, 64, 128, E8, BF>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
    if (t.bm == 64)
        return launch_pipe<G, 1, 4, FUSED, 64, 256, E8, BF>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
    if (t.bm == 128 && t.bn == 256)
        return launch_pipe<G, 1, 4, FUSED, 128, 256, E8, BF>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
    if (t.bm == 128)
        return launch_pipe<G, 1, 4, FUSED, 128, 128, E8, BF>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
    return launch_pipe<G, 2, 4, FUSED, 256, 256, E8, BF>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f, p);
}

template <int G, bool FUSED>
int launch_pipe_tile(const half_t* x, int64_t M, const uint4* c, int64_t N, int64_t K, half_t* y, void* workspace,
                     size_t workspace_bytes, hipStream_t stream, const Fusion& f)
{
    return launch_pipe_as<G, FUSED>(pipe_plan(f, M, N, K, FUSED, false), x, M, c, N, K, y, workspace, workspace_bytes, stream, f);
}

}  // namespace

// 8-bit format: same tiles, K splits and workspace as the 4-bit problem of the same M, N, K.
int launch_gemm_pipe8(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y, void* workspace,
                      size_t workspace_bytes, hipStream_t stream)
{
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    return launch_pipe_as<128, false, true>(pipe_plan(Fusion{}, M, N, K, false, true), x, M, c, N, K, y, workspace, workspace_bytes, stream,
                                            Fusion{});
}

int launch_gemm_pipe8_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, void* Y,
                            void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    if (f.swiglu && (N % (2 * kBlockRows) != 0 || gated_half_bytes(N, 2 * K, 128) > kMaxHalfBytes)) return E0M4_ERR_SHAPE;
    return launch_pipe_as<128, true, true>(pipe_plan(f, M, N, K, true, true), x, M, c, N, K, y, workspace, workspace_bytes, stream, f);
}

int launch_gemm_pipe(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                     void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    switch (group) {
        case 32: return launch_pipe_tile<32, false>(x, M, c, N, K, y, workspace, workspace_bytes, stream, Fusion{});
        case 64: return launch_pipe_tile<64, false>(x, M, c, N, K, y, workspace, workspace_bytes, stream, Fusion{});
        case 128: return launch_pipe_tile<128, false>(x, M, c, N, K, y, workspace, workspace_bytes, stream, Fusion{});
        default: return E0M4_ERR_GROUP;
    }
}

namespace {
// Whole tiles only (no workspace to split K into); the tile by the same estimate as for fp16, whose timings those of
// this member follow, flat tiles as K halves where k_halves says so.  Before the tiles of 128 columns and now: M = 700, 4608 x 4096 39.6
// and 32.7 us, 4096 x 13696 108 and 92; M = 1024, 4096 x 13696 (256 flat tiles in halves) 128 and 112; M = 100, 27392 x 4096 43 and 34.
template <int G>
int launch_pipe_bf16(const half_t* x, int64_t M, const uint4* c, int64_t N, int64_t K, half_t* y, hipStream_t stream)
{
    const PipePlan p = shortest(kNow, M, N, K, PipeRules{true, false, 1, 0});
    return launch_pipe_as<G, false, false, true>(p, x, M, c, N, K, y, nullptr, 0, stream, Fusion{});
}
}  // namespace

// bfloat16 member (X, parameters and Y bfloat16): whole tiles only, so no workspace.  At least as fast as the caller's
// 128 x 128-tile kernel on every measured shape (1.3 - 2.2 x at M = 512 ... 2048, 1.8 x at M = 64 and 128).
bool gemm_pipe_bf16_pays(int64_t M, int64_t N, int64_t K)
{
    (void)M;
    return gemm_pipe_supported(K) && N <= (int64_t)1 << 24;
}

int launch_gemm_pipe_bf16(const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group, void* Y,
                          hipStream_t stream)
{
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    switch (group) {
        case 32: return launch_pipe_bf16<32>(x, M, c, N, K, y, stream);
        case 64: return launch_pipe_bf16<64>(x, M, c, N, K, y, stream);
        case 128: return launch_pipe_bf16<128>(x, M, c, N, K, y, stream);
        default: return E0M4_ERR_GROUP;
    }
}

// With the epilogue operators of e0m4_matmul_fused (rms-norm is applied to X before this call).  The
// gated epilogue needs N/2 to be whole pairs of row blocks and the halves less than 2 GiB apart.
int launch_gemm_pipe_fused(const Fusion& f, const void* X, int64_t M, const void* packed, int64_t N, int64_t K, int group,
                           void* Y, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    const half_t* x = static_cast<const half_t*>(X);
    const uint4* c = static_cast<const uint4*>(packed);
    half_t* y = static_cast<half_t*>(Y);
    if (f.swiglu) {
        if (N % (2 * kBlockRows) != 0 || gated_half_bytes(N, K, group) > kMaxHalfBytes) return E0M4_ERR_SHAPE;
    }
    switch (group) {
        case 32: return launch_pipe_tile<32, true>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f);
        case 64: return launch_pipe_tile<64, true>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f);
        case 128: return launch_pipe_tile<128, true>(x, M, c, N, K, y, workspace, workspace_bytes, stream, f);
        default: return E0M4_ERR_GROUP;
    }
}

}  // namespace e0m4
