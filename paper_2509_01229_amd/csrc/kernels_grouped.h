// Grouped (mixture-of-experts) launches of the per-block device functions.
// (part of liquidgemm.hip: included there, inside namespace lqq)
#pragma once

// ------------------------------------------------------------------------------------
// Grouped launches (mixture-of-experts layers, Sec. 7.3): one launch runs the same per-block
// code over several experts that share N, K and the group size.  Expert i of the launch
// owns rows row_off[i] .. row_off[i] + rows[i] - 1 of X / Y and the expert[i]-th weight
// blob.  The table travels by value in the kernel arguments (no device copy, nothing to
// allocate), which bounds a call to 64 experts.
// ------------------------------------------------------------------------------------
constexpr int kMaxExperts = 64;
struct GroupTable {
    int count;
    int block_end[kMaxExperts];  // running total of blocks up to and including entry i
    int expert[kMaxExperts];
    int row_off[kMaxExperts];
    int rows[kMaxExperts];
};
struct GroupedPtrs {
    const int8_t *X;
    const float *sx;
    const u32x4 *Wp;
    const uint8_t *gp;
    const float *sw;
    __half *Y;
    int32_t *ACC;
    size_t w_stride;   // u32x4 elements between the packed codes of consecutive experts
    size_t gp_stride;  // bytes between their group parameters
};

template <int NW, int UU, bool G128>
__global__ __launch_bounds__(NW * 64) void w4a8_stream16_grouped_kernel(const GroupTable g, const GroupedPtrs p,
                                                                        int N, int K, int groups)
{
    const int i = blockIdx.x / groups, gx = blockIdx.x % groups;
    const int e = g.expert[i], r0 = g.row_off[i];
    stream16_block<2, NW, UU, G128, true>(Place{gx, groups, 0, 1, nullptr}, g.rows[i], N, K, p.X + (size_t)r0 * K, p.sx + r0,
                                    p.Wp + e * p.w_stride, p.gp + e * p.gp_stride, p.sw + (size_t)e * N,
                                    p.Y ? p.Y + (size_t)r0 * N : nullptr, p.ACC ? p.ACC + (size_t)r0 * N : nullptr,
                                    nullptr);
}

// The entry that block `lid` belongs to: one lane per entry compares, instead of a walk through the
// table (one dependent scalar load after the other, which a short block of a late entry waits for).  The lanes hold the
// rest of their entries by then, so that nothing else is loaded once the entry is known (tiles of 64 experts: 256 rows each on 1408 x 2048
// 67.0 / 63.9 us, 16 of 60 rows on 4096 x 2560 24.3 / 23.3).
static_assert(kMaxExperts == 64, "one lane per entry");
struct GroupEntry {
    int first, expert, row_off, rows;  // (first: the entry's first block)
};
__device__ __forceinline__ GroupEntry entry_of(const GroupTable &g, int lid)
{
    const int lane = threadIdx.x & 63;
    const int end = g.block_end[lane], expert = g.expert[lane], row_off = g.row_off[lane], rows = g.rows[lane];
    const int i = __popcll(__ballot(lane < g.count - 1 && lid >= end));
    return GroupEntry{i ? __builtin_amdgcn_readlane(end, i - 1) : 0, __builtin_amdgcn_readlane(expert, i),
                      __builtin_amdgcn_readlane(row_off, i), __builtin_amdgcn_readlane(rows, i)};
}

// block_end counts row tiles x column groups of every entry.  As in w4a8_panel_kernel each XCD gets a
// run of blocks, in which the row tiles of one column group are neighbours.
template <int F, int MF, bool G128, bool ONCE>
__global__ __launch_bounds__(512) void w4a8_panel_grouped_kernel(const GroupTable g, const GroupedPtrs p, int N, int K)
{
    const int total = g.block_end[g.count - 1];
    const int xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
    const int lid = xcd * per + min(xcd, rem) + (int)(blockIdx.x >> 3);
    const GroupEntry en = entry_of(g, lid);
    const int local = lid - en.first, M = en.rows, e = en.expert, r0 = en.row_off;
    const int blocks_m = (M + 32 * MF - 1) / (32 * MF), groups = (N / 32 + F - 1) / F;
    const int gx = blocks_m == 1 ? local : (int)((unsigned)local / (unsigned)blocks_m);
    panel_block<F, 8, MF, G128, ONCE>(Place{gx, groups, 0, 1, nullptr}, local - gx * blocks_m, M, N, K,
                                p.X + (size_t)r0 * K, p.sx + r0, p.Wp + e * p.w_stride, p.gp + e * p.gp_stride,
                                p.sw + (size_t)e * N, p.Y ? p.Y + (size_t)r0 * N : nullptr,
                                p.ACC ? p.ACC + (size_t)r0 * N : nullptr, nullptr, 0);
}

// TM = rows per row tile (128, or 64: twice the blocks for launches that would leave CUs idle)
template <bool G128, int KG, int TM = 128>
__global__ __launch_bounds__(256 * KG, KG == 1 ? 2 : 1) void w4a8_duo_grouped_kernel(const GroupTable g,
                                                                                     const GroupedPtrs p, int N,
                                                                                     int K)
{
    const GroupEntry en = entry_of(g, (int)blockIdx.x);
    const int local = (int)blockIdx.x - en.first, M = en.rows, e = en.expert, r0 = en.row_off;
    // row tiles of one column block are neighbours, so they meet on the expert's W columns
    const int blocks_m = (M + TM - 1) / TM;
    const int bm = local % blocks_m, bn = local / blocks_m;
    duo_block<G128, KG, TM>(Place{0, 1, 0, 1, nullptr}, bm, bn, M, N, K, p.X + (size_t)r0 * K, p.sx + r0,
                            p.Wp + e * p.w_stride, p.gp + e * p.gp_stride, p.sw + (size_t)e * N,
                            p.Y ? p.Y + (size_t)r0 * N : nullptr, p.ACC ? p.ACC + (size_t)r0 * N : nullptr,
                            nullptr);
}

// The direct-to-LDS form of the tiles for launches with more blocks than CUs (one k group per
// block, two blocks per CU).
template <bool G128>
__global__ __launch_bounds__(256, 2) void w4a8_duo_dl_grouped_kernel(const GroupTable g, const GroupedPtrs p, int N,
                                                                     int K)
{
    const GroupEntry en = entry_of(g, (int)blockIdx.x);
    const int local = (int)blockIdx.x - en.first, M = en.rows, e = en.expert, r0 = en.row_off;
    const int blocks_m = (M + 127) >> 7;
    const int bm = local % blocks_m, bn = local / blocks_m;
    const Place pl{0, 1, 0, 1, nullptr};
    const int8_t *X = p.X + (size_t)r0 * K;
    const float *sx = p.sx + r0, *sw = p.sw + (size_t)e * N;
    const u32x4 *Wp = p.Wp + e * p.w_stride;
    const uint8_t *gp = p.gp + e * p.gp_stride;
    __half *Y = p.Y ? p.Y + (size_t)r0 * N : nullptr;
    int32_t *ACC = p.ACC ? p.ACC + (size_t)r0 * N : nullptr;
    const int left = M - 128 * bm;  // block-uniform
    if (left <= 64)
        duo_dl_tile<G128, 2>(pl, bm, bn, M, N, K, X, sx, Wp, gp, sw, Y, ACC, nullptr);
    else if (left <= 96)
        duo_dl_tile<G128, 3>(pl, bm, bn, M, N, K, X, sx, Wp, gp, sw, Y, ACC, nullptr);
    else
        duo_dl_tile<G128, 4>(pl, bm, bn, M, N, K, X, sx, Wp, gp, sw, Y, ACC, nullptr);
}

// The 256-row tiles (one wave per SIMD, see kernels_tiled_solo16.h) of all experts of a launch as
// one persistent stream: resident blocks walk the tiles of every expert, with 256 x 256 tiles (KG = 1)
// prefetching across the boundaries between them.  block_end counts 256 x 256 / KG tiles here.
template <int KG>
struct SoloGrouped {
    const GroupedPtrs &p;
    int N, K, blocks_n, total;
    int end, expert, row_off, rows;  // this lane's entry: nothing is loaded when a tile is looked up, in the middle of the stage loop
    __device__ __forceinline__ SoloGrouped(const GroupTable &g, const GroupedPtrs &ptrs, int n, int k, int tn)
        : p(ptrs), N(n), K(k), blocks_n((n + tn - 1) / tn), total(g.block_end[g.count - 1])
    {
        const int lane = threadIdx.x & 63;
        end = lane < g.count ? g.block_end[lane] : 0x7fffffff;
        expert = g.expert[lane], row_off = g.row_off[lane], rows = g.rows[lane];
        asm volatile("" : "+v"(end), "+v"(expert), "+v"(row_off), "+v"(rows));  // (here, and not at each use)
    }
    __device__ __forceinline__ int slices() const { return 1; }
    __device__ __forceinline__ int tiles() const { return total; }
    __device__ __forceinline__ SoloTile tile(int lid, int G) const
    {
        lid = solo_xcd_order(lid, total, G);
        const int i = __popcll(__ballot(lid >= end));
        const int local = lid - (i ? __builtin_amdgcn_readlane(end, i - 1) : 0);
        const int M = __builtin_amdgcn_readlane(rows, i), e = __builtin_amdgcn_readlane(expert, i);
        const int r0 = __builtin_amdgcn_readlane(row_off, i);
        int bm, bn;
        solo_coords<KG>(local, (M + 255) / 256, blocks_n, bm, bn);
        return SoloTile{M,
                        bm,
                        bn,
                        0,
                        p.X + (size_t)r0 * K,
                        p.sx + r0,
                        p.Wp + e * p.w_stride,
                        p.gp + e * p.gp_stride,
                        p.sw + (size_t)e * N,
                        p.Y ? p.Y + (size_t)r0 * N : nullptr,
                        p.ACC ? p.ACC + (size_t)r0 * N : nullptr};
    }
};
template <bool G128, int KG>
__global__ __launch_bounds__(256, 1) void w4a8_solo_grouped_kernel(const GroupTable g, const GroupedPtrs p, int N, int K)
{
    solo16_body<G128, KG>(SoloGrouped<KG>(g, p, N, K, 256 / KG), N, K);
}
