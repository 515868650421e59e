// Grouped (mixture-of-experts) launch of the CTA-tile kernels, for experts with more rows than the decode kernels
// take in one pass.  Same body as tile_kernel, same build flags as the small tiles; what differs is how a CTA finds
// its tile: the rows per expert are only known on the device, so the grid covers an upper bound of row tiles and
// every CTA locates its (expert, row tile) by a prefix scan over the experts' row-tile counts.
// What such a launch spends beyond a plain GEMM is work on rows that are not there and CUs that wait: the last row tile of an expert
// runs with a body of 32, 64 or 96 rows if no more are left (8 experts x 250 rows, 4096 x 28672, 128 x 256 tiles: 593 -> 552 us), and
// tiles are numbered over the row tiles there are (128 experts x 62 rows, 4096 x 3072 and 1536 x 4096, 64 x 128 tiles: 585 -> 463 us).
#include "tm_w4_tile_impl.h"

namespace tmw4 {

namespace {

template <int TM, int TN, int NW, int GPU, int KW, int FMT = kFmtInt4>
__global__ __launch_bounds__(NW * 64) void tile_grouped_kernel(GroupedParams gp)
{
    constexpr int BM = TM * 16, PD = 2;
    // The experts' row tiles: 64 experts per step, an inclusive scan of their row-tile counts across the wave.
    const int lane = threadIdx.x & 63;
    struct Step {
        int a, z, cnt, incl;                        // rows [a, z) of the lane's expert, its row tiles, the sum up to it
    };
    auto scan = [&](int base) {
        const int e = base + lane;
        Step s{0, 0, 0, 0};
        if (e < gp.experts) {
            s.a = gp.offsets[e];
            s.z = gp.offsets[e + 1];
        }
        s.a = min(max(s.a, 0), gp.total_rows);      // rows are clamped to the buffers whatever the offsets hold
        s.z = max(min(s.z, gp.total_rows), s.a);
        s.cnt = (s.z - s.a + BM - 1) / BM;
        s.incl = s.cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(s.incl, d);
            if (lane >= d) s.incl += t;
        }
        return s;
    };
    Step at = scan(0);
    int row_tiles = __builtin_amdgcn_readlane(at.incl, 63);
    for (int base = 64; base < gp.experts; base += 64) row_tiles += __builtin_amdgcn_readlane(scan(base).incl, 63);
    // Same XCD-aware numbering as tile_kernel, over the row tiles there are and not over the grid's upper bound: that one's
    // surplus would fall to some XCDs and leave the others more CTAs than CUs (8 experts of 4096 x 2560, 44 rows each, 64 x 128
    // tiles: 180 CTAs, of which one XCD had 33).
    row_tiles = min(row_tiles, gp.mtiles);
    const int tiles = row_tiles * gp.tiles_n;
    const int chunk = (tiles + 7) / 8;
    const int b = blockIdx.x;
    const int logical = (b % 8) * chunk + b / 8;
    if (b / 8 >= chunk || logical >= tiles) return;
    const int panel_tiles = kPanelN * row_tiles;
    const int panel = logical / panel_tiles;
    const int within = logical % panel_tiles;
    const int pw = min(kPanelN, gp.tiles_n - panel * kPanelN);
    const int tile_n = panel * kPanelN + within % pw;
    int want = within / pw;                         // row tile, counted over all experts in order

    // row tile -> (expert, its row tile)
    int expert0 = 0;
    for (int base = 0;;) {
        const int total = __builtin_amdgcn_readlane(at.incl, 63);
        if (want < total) break;
        want -= total;
        base += 64;
        if (base >= gp.experts) return;             // (not reached: want is below the sum)
        at = scan(base);
        expert0 = base;
    }
    const int src = __builtin_ctzll(__ballot(at.cnt > 0 && at.incl - at.cnt <= want && want < at.incl));      // exactly one lane
    const int r0 = __builtin_amdgcn_readlane(at.a, src), r1 = __builtin_amdgcn_readlane(at.z, src);
    const int tile_m = want - __builtin_amdgcn_readlane(at.incl - at.cnt, src);
    const uint64_t wptr = gp.table[2 * (expert0 + src)], szptr = gp.table[2 * (expert0 + src) + 1];

    GemmParams p{};
    p.X = gp.X + (size_t)r0 * gp.K;
    p.ldy = gp.act ? gp.N / 2 : gp.N;
    p.act = gp.act;
    p.epi = gp.act;
    p.Y = gp.Y + (size_t)r0 * p.ldy;
    p.W = (const u32x4*)wptr;
    p.SZ = (const uint32_t*)szptr;
    p.M = r1 - r0;
    p.K = gp.K;
    p.N = gp.N;
    p.KU = gp.KU;
    p.NT = gp.NT;
    p.G = gp.G;
    p.split = 1;
    p.ku_per_split = gp.KU;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = gp.tiles_n;
    using Lds = TileLds<TM, TN, NW, KW, 1>;
    __shared__ __attribute__((aligned(16))) unsigned char smem0[Lds::kFirst];
    __shared__ __attribute__((aligned(16))) unsigned char smem1[Lds::kXsBytes];
    const int m0 = tile_m * BM, left = p.M - m0;
    // The last row tile of an expert: a body of as many rows as are left, in steps of 32.  The tallest body comes first in the code:
    // behind a shorter one it was given two more registers (64 x 128, 4-bit, groups of 128: 130 instead of 128, three CTAs per CU
    // instead of four; int8 in groups of 32: 170 instead of 168, two instead of three).
    if (TM == 2 || left > 16 * TM - 32) {
        tile_body<TM, TN, NW, GPU, KW, PD, 1, FMT, TM == 2>(p, m0, tile_m, tile_n, 0, smem0, smem1);
        return;
    }
    if constexpr (TM > 6) {
        if (left > 64) {
            tile_body<6, TN, NW, GPU, KW, PD, 1, FMT>(p, m0, tile_m, tile_n, 0, smem0, smem1);
            return;
        }
    }
    if constexpr (TM > 4) {
        if (left > 32) {
            tile_body<4, TN, NW, GPU, KW, PD, 1, FMT>(p, m0, tile_m, tile_n, 0, smem0, smem1);
            return;
        }
    }
    if constexpr (TM > 2) tile_body<2, TN, NW, GPU, KW, PD, 1, FMT>(p, m0, tile_m, tile_n, 0, smem0, smem1);
}

template <int TM, int TN, int KW, int FMT = kFmtInt4>
hipError_t launch_grouped_shape(GroupedParams gp, int experts, int group, hipStream_t stream)
{
    constexpr int BM = TM * 16, BN = 4 * TN * 16;
    constexpr int SPU = FMT == kFmtInt4 ? 4 : 2;                             // MFMA steps per packed unit
    if ((gp.KU * SPU) % KW) return hipErrorInvalidValue;                     // whole stages
    if ((uint64_t)gp.total_rows * (uint64_t)gp.K >= (1ull << 31)) return hipErrorInvalidValue;   // 32-bit X offsets
    gp.tiles_n = (gp.N + BN - 1) / BN;
    // every expert with rows adds at most one partly filled row tile
    gp.mtiles = gp.total_rows / BM + (gp.total_rows < experts ? gp.total_rows : experts);
    const long tiles = (long)gp.mtiles * gp.tiles_n;
    if (tiles <= 0 || tiles > (1l << 30)) return hipErrorInvalidValue;
    dim3 grid((unsigned)(((tiles + 7) / 8) * 8)), block(256);
    switch (group) {
        case 128: hipLaunchKernelGGL((tile_grouped_kernel<TM, TN, 4, 1, KW, FMT>), grid, block, 0, stream, gp); break;
        case 64: hipLaunchKernelGGL((tile_grouped_kernel<TM, TN, 4, 2, KW, FMT>), grid, block, 0, stream, gp); break;
        case 32: hipLaunchKernelGGL((tile_grouped_kernel<TM, TN, 4, 4, KW, FMT>), grid, block, 0, stream, gp); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_grouped(const GroupedParams& gp, int variant, int experts, int group, hipStream_t stream)
{
    if (experts <= 0) return hipErrorInvalidValue;
    switch (variant) {
        case kTile64x128: return launch_grouped_shape<4, 2, 4>(gp, experts, group, stream);
        case kTile32x128: return launch_grouped_shape<2, 2, 4>(gp, experts, group, stream);
        case kTile128x256: return launch_grouped_shape<8, 4, 2>(gp, experts, group, stream);
        default: return hipErrorInvalidValue;
    }
}

// The 8-bit formats (integer codes, FP8 E4M3): the same two tile shapes.
hipError_t launch_tile_grouped_8bit(const GroupedParams& gp, int variant, int experts, int group, bool fp8, hipStream_t stream)
{
    if (experts <= 0) return hipErrorInvalidValue;
    switch (variant) {
        case kTile32x128:
            return fp8 ? launch_grouped_shape<2, 2, 4, kFmtFp8>(gp, experts, group, stream)
                       : launch_grouped_shape<2, 2, 4, kFmtInt8>(gp, experts, group, stream);
        case kTile64x128:
            return fp8 ? launch_grouped_shape<4, 2, 4, kFmtFp8>(gp, experts, group, stream)
                       : launch_grouped_shape<4, 2, 4, kFmtInt8>(gp, experts, group, stream);
        case kTile128x256:
            return fp8 ? launch_grouped_shape<8, 4, 2, kFmtFp8>(gp, experts, group, stream)
                       : launch_grouped_shape<8, 4, 2, kFmtInt8>(gp, experts, group, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tmw4
