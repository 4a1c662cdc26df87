// gfx950 kernels and the C-ABI dispatcher of the LiquidQuant W4A8 GEMM.
//
// Three kernel families share the packed layout of lqq_layout.h and the dequantisation of
// lqq_device.h (paper Sec. 5.3):
//
//   stream16 (M <= 16): the memory-bound regime of the paper's cost model (Sec. 3.2,
//           T_LD dominates).  A block owns F tiles of 32 output channels; its NW waves
//           split K between them (in-block split-K), stream the packed weights straight
//           from HBM into registers with one 16-byte load per lane, dequantise, feed the
//           16-row MFMA, and reduce their INT32 partials through LDS -- integer sums, so the
//           result does not depend on the order.  Optional grid-level split-K through a workspace.
//
//   panel   (17 rows to a few hundred): the same split of K between the waves of a block, with
//           32, 64 or 128 rows and 32 to 128 channels per block on the 32-row MFMA and X passed
//           through LDS a wave at a time.
//
//   tiled   (larger M): the compute-bound regime (T_DQ + T_MMA dominates).  A block owns
//           128 rows of X and 256 output channels; the X tile is staged in LDS (double
//           buffered) and shared by the waves, each wave keeps its own 64 channels'
//           weights in registers (global -> VGPR, never through LDS: the dequantised
//           operand is consumed by the MFMA of the same wave, which is the point of the
//           paper's implicit fine-grained pipeline, Sec. 5.1) and reuses every dequantised
//           fragment for 4 MFMAs.  Three forms: `duo` (X staged through registers, two k
//           groups per block for grids of at most one block per CU), `duo_dl` (X straight
//           into LDS, deeper pipeline, grids that fill the chip) and `duo_pt` (duo_dl with
//           resident blocks walking several tiles as one stream of stages).
//
// All compute Y = X W^T with the weights on the B operand of the INT8 MFMA, so that a lane
// ends up with 2 adjacent output channels of one row (the tile interleave of the layout)
// and a half-wave writes a full 128-byte line of FP16.
//
// Every kernel here must compile without scratch memory (the build checks it): register
// spills next to the divergent single-thread sections of the split-K protocol are not
// something to rely on.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "lqq_common.h"
#include "lqq_device.h"

namespace lqq {

// Clears the ticket area at the head of a workspace (a fill kernel rather than a memset, so
// that it can be captured in a HIP graph like everything else here).
__global__ __launch_bounds__(256) void workspace_init_kernel(unsigned int *tickets, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) tickets[i] = 0u;
}

// ------------------------------------------------------------------------------------
// Layout hook: packed -> INT8 [N,K] with the kernels' own unpack + Eq. 12 path.
// One wave per 1 KiB chunk (32 channels x 64 k).
// ------------------------------------------------------------------------------------
template <bool G128>
__global__ __launch_bounds__(256) void dequant_dump_kernel(const u32x4 *__restrict__ Wp,
                                                           const uint8_t *__restrict__ gp, int N, int K,
                                                           int8_t *__restrict__ Wd)
{
    const int lane = threadIdx.x & 63;
    const int j = lane & 31, kb = lane >> 5;
    const int chunks_per_tile = K >> 6;
    const int t = blockIdx.y;
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= chunks_per_tile) return;
    const u32x4 p = Wp[((size_t)t * chunks_per_tile + c) * 64 + lane];
    UnitParams<G128> up;
    up.load(gp, (size_t)t * (K >> 7) + (c >> 1), j);
    uint32_t s2, a4;
    up.get(c & 1, s2, a4);
    v4i lo, hi;
    dequant_chunk(p, s2, a4, lo, hi);
    int8_t *row = Wd + (size_t)channel_of(t, j) * K + (size_t)c * 64 + 16 * kb;
    *reinterpret_cast<v4i *>(row) = lo;
    *reinterpret_cast<v4i *>(row + 32) = hi;
}

// ------------------------------------------------------------------------------------
// Epilogue of one accumulator element (Sec. 4: first-level dequantisation; Sec. 5.3).
// ------------------------------------------------------------------------------------
__device__ __forceinline__ __half scale_to_half(int acc, float sx, float sw)
{
    return __float2half_rn((float)acc * sx * sw);
}

#include "kernels_common.h"
#include "kernels_stream.h"
#include "kernels_panel.h"
#include "kernels_tiled.h"
#include "kernels_tiled_dl.h"
#include "kernels_tiled_pt.h"
#include "kernels_tiled_solo.h"
#include "kernels_tiled_solo16.h"
#include "kernels_reference.h"
#include "kernels_grouped.h"

// ------------------------------------------------------------------------------------
// Variant table and dispatcher
// ------------------------------------------------------------------------------------
struct Args {
    int M, N, K, group;
    const int8_t *X;
    const float *sx;
    const u32x4 *Wp;
    const uint8_t *gp;
    const float *sw;
    __half *Y;
    int32_t *ACC;
    hipStream_t stream;
    void *ws;
    size_t ws_bytes;
    size_t *query = nullptr;  // set: store the workspace bytes the launch would use and launch nothing
};

typedef int (*LaunchFn)(const Args &);

// Kernels that need more than the default 48 KiB of dynamic LDS must be told so once per
// device; the grant is remembered, so the launch path of a short kernel pays one map lookup
// instead of a runtime call.
static int allow_lds_once(const void *kernel, size_t bytes)
{
    struct Grant {
        int dev;
        const void *kernel;
        size_t bytes;
    };
    static std::mutex mu;
    static Grant granted[512];  // (device, kernel) pairs seen so far; no heap
    static int count = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return fail(LQ_ERR_HIP, "hipGetDevice failed");
    std::lock_guard<std::mutex> lock(mu);
    Grant *g = nullptr;
    for (int i = 0; i < count && !g; ++i)
        if (granted[i].dev == dev && granted[i].kernel == kernel) g = &granted[i];
    if (g && g->bytes >= bytes) return LQ_OK;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess)
        return fail(LQ_ERR_HIP, "hipFuncSetAttribute(%zu bytes of LDS): %s", bytes, hipGetErrorString(e));
    if (!g && count < 512) g = &granted[count++];
    if (g) *g = Grant{dev, kernel, bytes};  // a full table only means asking again next time
    return LQ_OK;
}
template <class Kernel>
static int allow_lds(Kernel kernel, size_t bytes)
{
    if (bytes <= 48 * 1024) return LQ_OK;
    return allow_lds_once(reinterpret_cast<const void *>(kernel), bytes);
}

constexpr long long kAssumedCUs = 256;  // the shape rules of the dispatcher are written for the MI355X

// Grid-level split of K for the 16-row kernel, each wave keeping at least two units of 128 k.
static int stream_split(int N, int K, int F, int NW)
{
    const int groups = N / (32 * F), units = K / 128;
    // Measured on MI355X: the exchange of partial tiles through memory costs about 3 us, so
    // K is split across blocks only when N alone leaves most CUs without a block.
    int s = groups > 128 ? 1 : (groups > 64 ? 2 : 4);
    s = std::min(s, units / (2 * NW));
    return std::max(1, s);
}

template <int F, int NW, int SPLIT, int UU = 1>
static int launch_stream16(const Args &a)
{
    if (a.M > 16) return fail(LQ_ERR_INVALID, "stream16 variants handle M <= 16, got %d", a.M);
    if ((a.N / 32) % F != 0) return fail(LQ_ERR_INVALID, "N/32 not a multiple of F=%d", F);
    const int groups = a.N / (32 * F);
    int S = SPLIT ? SPLIT : stream_split(a.N, a.K, F, NW);
    // the deep-prefetch form (small shapes) keeps whole K in one block unless N gives very few
    if (!SPLIT && UU == 4) S = groups <= 64 ? 2 : 1;
    if ((a.K / 128) % UU != 0) return fail(LQ_ERR_INVALID, "K/128 not a multiple of UU=%d", UU);
    S = std::min(S, a.K / (128 * UU));
    if (S > 1 && groups > kMaxTicketGroups) S = 1;
    size_t need = S > 1 ? kTicketBytes + (size_t)S * (a.N / 32) * 8 * 64 * sizeof(int32_t) : 0;
    if (a.query) return *a.query = need, LQ_OK;
    if (need > 0 && (!a.ws || a.ws_bytes < need)) {
        if (SPLIT)
            return fail(LQ_ERR_WORKSPACE, "split-K needs %zu bytes of workspace, got %zu", need,
                        a.ws ? a.ws_bytes : 0);
        S = 1;
        need = 0;
    }
    const dim3 grid(groups, S), block(NW * 64);
    size_t lds_bytes = (size_t)NW * F * 8 * 64 * sizeof(int);
    // Two tiles in four waves: with groups of 64 the registers let five blocks on a CU (four with 128), which is ahead where five
    // hold them all (15 x 76416 x 9472 75.4 / 67.8 us) and behind where a few are left for a round of their own; four at a time, by the LDS
    // that they ask for, are more even there (more than 5 to 6 blocks a CU 0.99 of the time to K = 4352, 0.97 to 6400, 0.95 beyond; 4 x 93056 x
    // 9728 86.1 / 79.2 us).
    if (NW == 4 && groups > 5 * kAssumedCUs && groups <= 6 * kAssumedCUs) lds_bytes = std::max<size_t>(lds_bytes, 36 << 10);
    unsigned int *tickets = static_cast<unsigned int *>(a.ws);
    int32_t *partials = a.ws ? reinterpret_cast<int32_t *>(static_cast<char *>(a.ws) + kTicketBytes) : nullptr;
    if (a.group == 128) {
        if (int rc = allow_lds(&w4a8_stream16_kernel<F, NW, UU, true>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_stream16_kernel<F, NW, UU, true>), grid, block, lds_bytes, a.stream, a.M, a.N,
                           a.K, S, a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, partials, tickets);
    } else {
        if (int rc = allow_lds(&w4a8_stream16_kernel<F, NW, UU, false>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_stream16_kernel<F, NW, UU, false>), grid, block, lds_bytes, a.stream, a.M, a.N,
                           a.K, S, a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, partials, tickets);
    }
    return LQ_OK;
}

// The 16-row kernel with half a tile per block.
template <int NW, int D, int SPLIT>
static int launch_stream16_half(const Args &a)
{
    if (a.M > 16) return fail(LQ_ERR_INVALID, "stream16 variants handle M <= 16, got %d", a.M);
    const int groups = a.N / 16;
    const int S = groups > kMaxTicketGroups ? 1 : std::min(SPLIT, a.K / 128);
    const size_t need = S > 1 ? kTicketBytes + (size_t)S * groups * 4 * 64 * sizeof(int32_t) : 0;
    if (a.query) return *a.query = need, LQ_OK;
    if (need > 0 && (!a.ws || a.ws_bytes < need))
        return fail(LQ_ERR_WORKSPACE, "split-K needs %zu bytes of workspace, got %zu", need, a.ws ? a.ws_bytes : 0);
    unsigned int *tickets = static_cast<unsigned int *>(a.ws);
    int32_t *partials = a.ws ? reinterpret_cast<int32_t *>(static_cast<char *>(a.ws) + kTicketBytes) : nullptr;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(groups, S), dim3(NW * 64), 0, a.stream, a.M, a.N, a.K, S, a.X, a.sx, a.Wp, a.gp, a.sw,
                           a.Y, a.ACC, partials, tickets);
        return (int)LQ_OK;
    };
    return a.group == 128 ? go(&w4a8_stream16_half_kernel<NW, D, true>) : go(&w4a8_stream16_half_kernel<NW, D, false>);
}

// Panel kernel: 32 MF rows x 32 F channels per block, S slices of K across blocks, NW waves per
// block (two per SIMD while the accumulators leave room for that, i.e. up to 64 rows).
static long long panel_blocks(int M, int N, int F, int MF)
{
    return (long long)((M + 32 * MF - 1) / (32 * MF)) * ((N / 32 + F - 1) / F);
}
static size_t panel_ws_bytes(int blocks, int F, int MF, int S)
{
    return S <= 1 ? 0 : kTicketBytes + (size_t)blocks * S * F * MF * 1024 * sizeof(int32_t);
}
static size_t workspace_limit(const Args &a)  // (a query names its limit, if it has one, in ws_bytes)
{
    return a.query ? (a.ws_bytes ? a.ws_bytes : SIZE_MAX) : a.ws ? a.ws_bytes : 0;
}
template <int F, int NW, int MF>
static int launch_panel(const Args &a, int S)
{
    const int blocks_m = (a.M + 32 * MF - 1) / (32 * MF), blocks_n = (a.N / 32 + F - 1) / F;
    S = std::max(1, std::min({S, a.K / 128, kMaxPanelSlices}));
    if (S > 1 && blocks_m * blocks_n > kMaxTicketGroups) S = 1;
    const size_t need = panel_ws_bytes(blocks_m * blocks_n, F, MF, S);
    if (a.query) return *a.query = need, LQ_OK;
    if (need > 0 && (!a.ws || a.ws_bytes < need))
        return fail(LQ_ERR_WORKSPACE, "split-K needs %zu bytes of workspace, got %zu", need, a.ws ? a.ws_bytes : 0);
    const dim3 grid((unsigned)(blocks_m * blocks_n * S)), block(NW * 64);
    const size_t lds_bytes = panel_lds_bytes(F, NW, MF, (a.K / 128 + S - 1) / S);
    unsigned int *tickets = static_cast<unsigned int *>(a.ws);
    int32_t *partials = a.ws ? reinterpret_cast<int32_t *>(static_cast<char *>(a.ws) + kTicketBytes) : nullptr;
    auto go = [&](auto kernel) {
        if (int rc = allow_lds(kernel, lds_bytes)) return rc;
        hipLaunchKernelGGL(kernel, grid, block, lds_bytes, a.stream, a.M, a.N, a.K, S, a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC,
                           partials, tickets);
        return (int)LQ_OK;
    };
    if (blocks_m == 1)
        return a.group == 128 ? go(&w4a8_panel_kernel<F, NW, MF, true, true>) : go(&w4a8_panel_kernel<F, NW, MF, false, true>);
    return a.group == 128 ? go(&w4a8_panel_kernel<F, NW, MF, true, false>) : go(&w4a8_panel_kernel<F, NW, MF, false, false>);
}
struct PanelForm {
    int F, NW, MF;
    int (*launch)(const Args &, int S);
};
static const PanelForm kPanelForms[] = {
    {1, 8, 1, &launch_panel<1, 8, 1>}, {2, 8, 1, &launch_panel<2, 8, 1>}, {4, 8, 1, &launch_panel<4, 8, 1>},
    {1, 8, 2, &launch_panel<1, 8, 2>}, {2, 8, 2, &launch_panel<2, 8, 2>}, {3, 8, 2, &launch_panel<3, 8, 2>},
    {4, 8, 2, &launch_panel<4, 8, 2>}, {3, 4, 4, &launch_panel<3, 4, 4>}, {4, 4, 4, &launch_panel<4, 4, 4>},
    {2, 4, 4, &launch_panel<2, 4, 4>}, {3, 8, 1, &launch_panel<3, 8, 1>},  // (the last two not in choose_panel's fit)
};
constexpr int kFittedPanelForms = 9;
static const PanelForm &panel_form(int F, int MF)
{
    for (const PanelForm &f : kPanelForms)
        if (f.F == F && f.MF == MF) return f;
    return kPanelForms[0];
}
struct PanelChoice {
    const PanelForm *form = nullptr;  // null: no form takes the shape
    int S = 1;
    double us = 1e30;
};
// The form and the number of K slices for a shape.  The time of a form is linear in what it does,
// fitted to 14 row counts (17 to 512) x 17 weight shapes (1024 to 28672 channels and k) x all forms
// and 1 to 4 slices of the panel kernel with one set of W registers, 8 % rms.  Audited with the present kernel on 2200 calls of 17 to 512
// rows (channels from 1024, k from 2048, to 28672 each, weights from HBM): the form it picks is 0.5 % behind the best one at 17..32 rows, 0.8 %
// at 33..64, 1.4 to 2.0 % above (geometric means; 24 % at worst).  The fit itself never picks 32 x 64 and 128 x 128, the best in 7 and 4 % of
// them; the exceptions behind it and panel_instead_of_few_tiles do.
//   2.26 us of launch and first loads
//   + 0.61 us per accumulator tile (32 x 32) of a block: the sum over the waves and the epilogue
//   + 9.8 ns per KB of X and 19.1 ns per KB of W that a CU takes in (X comes from L2; W is also dequantised)
//   + 75 ns per MB of packed weights, streamed from HBM once
//   + with K slices 1.33 us for the exchange and 0.85 us per 1024 (block, accumulator tile) pairs of its volume
// Beyond 64 rows, no more than two rounds of blocks were fitted (more never paid); 128-row panels
// with K slices were never among the best, nor slices that leave a wave less than two units (1024 x
// 4096 at 45 rows: 5.8 us with one slice, 6.2 / 6.4 / 6.7 with two, three, four).
static PanelChoice choose_panel(int M, int N, int K, size_t ws_limit)
{
    PanelChoice best;
    for (int i = 0; i < kFittedPanelForms; ++i) {
        const PanelForm &f = kPanelForms[i];
        const long long blocks = panel_blocks(M, N, f.F, f.MF);
        const int tiles = f.F * f.MF;
        for (int S = 1; S <= 4 && S <= K / 128; ++S) {
            if (S > 1 && (f.MF == 4 || K / 128 < 2 * f.NW * S || blocks * S > 2 * kAssumedCUs ||
                          panel_ws_bytes((int)blocks, f.F, f.MF, S) > ws_limit)) break;
            if (M > 64 && blocks * S > 2 * kAssumedCUs) break;
            const double rounds = (double)((blocks * S + kAssumedCUs - 1) / kAssumedCUs);
            const int units = (K / 128 + S - 1) / S, walked = (units + f.NW - 1) / f.NW * f.NW;
            const double x_kb = rounds * walked * 4.096 * f.MF, w_kb = rounds * walked * 2.048 * f.F;
            const double us = 2.26 + 0.611 * rounds * tiles + 0.00983 * x_kb + 0.0191 * w_kb + 0.0753 * (0.5e-6 * N * K) +
                              (S > 1 ? 1.33 + 0.00085 * (double)(blocks * S * tiles) : 0.0);
            if (us < best.us) best = PanelChoice{&f, S, us};
        }
    }
    // Exceptions.  For launches of several rounds, which the fit prices alike whatever stays on a CU: 32 x 128 panels, one
    // on a CU, run a round at a time: beyond one round 32 x 64 panels, two on a CU, are ahead (136 x 11520 x 2048 15.9 / 13.1 us,
    // 390 such calls 1.05 / 0.91 of what the form with one set of W registers took).  32 x 32 panels of more than two rounds are
    // behind them while a wave has no second unit (24 x 24064 x 256 5.5 / 5.2, 5.0 of that form; K = 512 5.7 / 5.4, 768 6.1 / 6.0,
    // 1024 6.2 / 6.5).
    if (!best.form || best.form->MF != 1) return best;
    const int F = best.form->F;
    const long long blocks = panel_blocks(M, N, F, 1);
    if (best.S == 1 && ((F == 4 && blocks > kAssumedCUs) || (F == 1 && blocks > 2 * kAssumedCUs && K <= 768)))
        best.form = &panel_form(2, 1);
    // From 5200 random calls (17 to 512 rows, N from 1024, K from 2048, to 28672 each), these against the fit's choice: with one row
    // tile, panels of 96 channels where they are less than a round in place of 128 channels (0.91: more of the CUs work), also
    // of 128 with slices in more than one round of blocks (20 x 20608 x 14336 37.2 / 30.0 us, 0.90); two slices of 64 channels for
    // four of 128 up to K = 40960 (0.92 to 28672, 0.96 beyond; 0.98 to 49152, behind from there on: 88 x 2432 x 124928 64.7 /
    // 73.2 us); two of 32 for four of 64 (with several row tiles 0.85 to K = 12288, 0.96 to 20480, behind beyond; with one from 3072
    // channels on 0.93); with several row tiles up to K = 8192 one slice of 32 for two (0.96).
    if (K < 2048 || N < 1024) return best;
    if (M <= 32 && F == 4 && best.S == 1 && blocks <= kAssumedCUs && panel_blocks(M, N, 3, 1) < kAssumedCUs)
        best.form = &panel_form(3, 1);
    else if (F == 4 && best.S == 4) {
        if (K <= 40960) best.form = &panel_form(2, 1), best.S = 2;
    } else if (M <= 32 && F == 4 && best.S > 1 && blocks * best.S > kAssumedCUs)
        best.form = &panel_form(3, 1), best.S = 1;
    else if (F == 2 && best.S == 4 && K <= 20480 && (M > 32 || N >= 3072))
        best.form = &panel_form(1, 1), best.S = 2;
    else if (M > 32 && F == 1 && best.S == 2 && K <= 8192)
        best.S = 1;
    return best;
}
// 17..64 rows: the form that choose_panel picks
static int launch_panel_auto(const Args &a)
{
    const PanelChoice c = choose_panel(a.M, a.N, a.K, workspace_limit(a));
    return c.form->launch(a, c.S);
}
template <int F, int NW, int MF, int SPLIT>
static int launch_panel_named(const Args &a)
{
    return launch_panel<F, NW, MF>(a, SPLIT);
}

// Grid-level split of K for the duo kernel with two k groups per block (grids of at most
// one block per CU).  Measured: a slice costs about as much in partial-tile exchange
// (128 KiB per tile and slice, added up by the last block) as half a 256-k unit costs in
// matrix work, which puts the best slice count near 0.75 * sqrt(K / 256); more slices than
// CUs per tile would only queue up.
static int duo_split(int M, int N, int K)
{
    const int tiles = ((M + 127) / 128) * ((N + 255) / 256);
    if (tiles > 128 || tiles > kMaxTicketGroups) return 1;
    const int units = K / 256;
    int s = (int)(0.75 * std::sqrt((double)units) + 0.5);
    s = std::min(std::min(s, 256 / tiles), std::min(units / 2, 8));
    return std::max(1, s);
}
static size_t duo_ws_bytes(int M, int N, int S, int tm = 128)
{
    if (S <= 1) return 0;
    const size_t tiles = (size_t)((M + tm - 1) / tm) * ((N + 255) / 256);
    return kTicketBytes + tiles * S * 4 * 32 * 256 * sizeof(int32_t);  // a tile's slot has the full size whatever its height
}

template <int SPLIT, int KG, int TM = 128>
static int launch_duo_as(const Args &a, int S)
{
    constexpr int WM = TM;
    const int blocks_n = (a.N + 255) / 256, blocks_m = (a.M + WM - 1) / WM;
    if ((long long)a.M * a.K >= (1ll << 32))
        return fail(LQ_ERR_INVALID, "M * K = %lld is beyond the 2^32 - 1 bytes of X one call addresses; split the batch",
                    (long long)a.M * a.K);
    S = std::min(S, a.K / (256 * KG));  // every k group of every slice gets at least one unit
    if (blocks_n * blocks_m * 8 > kMaxTicketGroups || S < 1) S = 1;  // one ticket per (tile, wave of the block)
    size_t need = duo_ws_bytes(a.M, a.N, S, TM);
    if (a.query) return *a.query = need, LQ_OK;
    if (need > 0 && (!a.ws || a.ws_bytes < need)) {
        if (SPLIT)
            return fail(LQ_ERR_WORKSPACE, "split-K needs %zu bytes of workspace, got %zu", need,
                        a.ws ? a.ws_bytes : 0);
        S = 1;
        need = 0;
    }
    // KG groups x 2 stages of X; the in-block reduction reuses them and needs 64 KiB
    const size_t lds_bytes = KG == 1 ? 2 * (size_t)128 * kTilePitch
                                     : std::max<size_t>(KG * 2 * (size_t)128 * kTilePitch, 64 * 1024);
    const dim3 grid((unsigned)(blocks_n * blocks_m), (unsigned)S), block(256 * KG);
    unsigned int *tickets = static_cast<unsigned int *>(a.ws);
    int32_t *partials = a.ws ? reinterpret_cast<int32_t *>(static_cast<char *>(a.ws) + kTicketBytes) : nullptr;
    if constexpr (KG == 2 && TM == 128) {
      // one row tile of 65..96 rows: the kernel that computes three of its four row fragments
      if (a.M > 64 && a.M <= 96) {
        constexpr int KG3 = 2;
        if (a.group == 128) {
            if (int rc = allow_lds(w4a8_duo_kernel<true, KG3, 128, true>, lds_bytes)) return rc;
            hipLaunchKernelGGL((w4a8_duo_kernel<true, KG3, 128, true>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K,
                               a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, partials, tickets);
        } else {
            if (int rc = allow_lds(w4a8_duo_kernel<false, KG3, 128, true>, lds_bytes)) return rc;
            hipLaunchKernelGGL((w4a8_duo_kernel<false, KG3, 128, true>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K,
                               a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, partials, tickets);
        }
        return LQ_OK;
      }
    }
    if (a.group == 128) {
        if (int rc = allow_lds(w4a8_duo_kernel<true, KG, TM>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_duo_kernel<true, KG, TM>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K, a.X,
                           a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, partials, tickets);
    } else {
        if (int rc = allow_lds(w4a8_duo_kernel<false, KG, TM>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_duo_kernel<false, KG, TM>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K, a.X,
                           a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, partials, tickets);
    }
    return LQ_OK;
}

// KGSEL: 0 = choose from the grid size, 1 / 2 = fixed number of k groups per block.
template <int SPLIT, int KGSEL>
static int launch_duo(const Args &a)
{
    const int tiles = ((a.M + 127) / 128) * ((a.N + 255) / 256);
    int kg = KGSEL, S = SPLIT;
    if (!kg) kg = (tiles * std::max(1, SPLIT) <= 256 && a.K >= 512) ? 2 : 1;
    if (a.K < 512) kg = 1;
    if (!S) S = kg == 2 ? duo_split(a.M, a.N, a.K) : 1;
    return kg == 2 ? launch_duo_as<SPLIT, 2>(a, S) : launch_duo_as<SPLIT, 1>(a, S);
}

// The direct-to-LDS form of the kernel (one k group per block; for grids that fill the chip).
template <int SPLIT>
static int launch_duo_dl(const Args &a)
{
    const int blocks_n = (a.N + 255) / 256, blocks_m = (a.M + 127) / 128;
    if ((long long)a.M * a.K >= (1ll << 32))
        return fail(LQ_ERR_INVALID, "M * K = %lld is beyond the 2^32 - 1 bytes of X one call addresses; split the batch",
                    (long long)a.M * a.K);
    int S = std::min(std::max(1, SPLIT), a.K / 256);
    if (blocks_n * blocks_m > kMaxTicketGroups) S = 1;
    const size_t need = duo_ws_bytes(a.M, a.N, S);
    if (a.query) return *a.query = need, LQ_OK;
    if (need > 0 && (!a.ws || a.ws_bytes < need))
        return fail(LQ_ERR_WORKSPACE, "split-K needs %zu bytes of workspace, got %zu", need, a.ws ? a.ws_bytes : 0);
    const size_t lds_bytes = 4 * (size_t)128 * 128;
    const dim3 grid((unsigned)(blocks_n * blocks_m), (unsigned)S), block(256);
    unsigned int *tickets = static_cast<unsigned int *>(a.ws);
    int32_t *partials = a.ws ? reinterpret_cast<int32_t *>(static_cast<char *>(a.ws) + kTicketBytes) : nullptr;
    if (a.group == 128) {
        if (int rc = allow_lds(w4a8_duo_dl_kernel<true>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_duo_dl_kernel<true>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K, a.X, a.sx,
                           a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, partials, tickets);
    } else {
        if (int rc = allow_lds(w4a8_duo_dl_kernel<false>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_duo_dl_kernel<false>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K, a.X, a.sx,
                           a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, partials, tickets);
    }
    return LQ_OK;
}

// Compute units of the current device (the grid of the persistent kernels), asked once per device.
static int cu_count()
{
    static std::mutex mu;
    static int cached[64];  // 0 = not asked yet
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    std::lock_guard<std::mutex> lock(mu);
    if (cached[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
        cached[dev] = cus;
    }
    return cached[dev];
}

// The persistent form of the direct-to-LDS kernel: one block per resident slot (two per CU),
// each walking its share of the tiles as one stream of stages.  Needs K % 512 == 0.
static bool duo_pt_fits(int M, int N, int K)
{
    // (a ragged last row tile of at most 64 rows is better off with the two-fragment path of
    // the one-tile-per-block kernels)
    return K % 512 == 0 && (M % 128 == 0 || M % 128 > 64);
}
static int launch_duo_pt(const Args &a)
{
    if (a.query) return LQ_OK;  // no workspace
    if (a.K % 512 != 0) return fail(LQ_ERR_INVALID, "the persistent tiled variant needs K %% 512 == 0, got %d", a.K);
    const int blocks_n = (a.N + 255) / 256, blocks_m = (a.M + 127) / 128;
    if ((long long)a.M * a.K >= (1ll << 32))
        return fail(LQ_ERR_INVALID, "M * K = %lld is beyond the 2^32 - 1 bytes of X one call addresses; split the batch",
                    (long long)a.M * a.K);
    const int cus = cu_count();
    const int grid = std::min(blocks_m * blocks_n, 2 * std::max(cus, 1));
    const size_t lds_bytes = 4 * (size_t)128 * 128;
    if (a.group == 128) {
        if (int rc = allow_lds(w4a8_duo_pt_kernel<true>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_duo_pt_kernel<true>), dim3((unsigned)grid), dim3(256), lds_bytes, a.stream, a.M, a.N,
                           a.K, a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n);
    } else {
        if (int rc = allow_lds(w4a8_duo_pt_kernel<false>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_duo_pt_kernel<false>), dim3((unsigned)grid), dim3(256), lds_bytes, a.stream, a.M, a.N,
                           a.K, a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n);
    }
    return LQ_OK;
}

// Persistent 256 x 256 tiles, one wave per SIMD (see kernels_tiled_solo.h); KG = 2: 256 x 128
// tiles with the four waves as two k groups.  Needs K % 512 == 0 (the 16x16x64 forms without K
// slices: K % 256 == 0).
// K slices across blocks for outputs with fewer tiles than CUs: every slice a multiple of 512 k,
// tiles * slices at most the CUs (one round), the partial sums of a slice as an INT32 matrix of
// its own in the workspace and a second, streaming kernel that adds them up.  Unlike the ticket
// scheme of the 128-row kernels nothing here is serial -- but the partial matrices are 4 S M N
// bytes written and read once, which is why this pays for long K only.  Returns 1 for no split.
static int solo_split(int tiles, int K, int cus)
{
    const int units = K / 512;
    int best = 1;
    for (int s = 2; s <= 4 && s <= units && tiles * s <= cus; ++s)  // (more than four: measured behind the 128-row tiles)
        if (units % s == 0) best = s;
    return best;
}
static size_t solo_ws_bytes(int M, int N, int S)
{
    return S <= 1 ? 0 : kTicketBytes + (size_t)S * M * N * sizeof(int32_t);
}
// SPLIT: 0 = no K slices, -1 = as many as solo_split gives and the workspace holds, n = exactly n
template <int KG, int SPLIT = 0, bool SHAPE16 = false>
static int launch_solo_pt(const Args &a)
{
    // (the 16x16x64 forms without K slices also take K % 512 == 256: two added stages of zero weights)
    if (a.K % 512 != 0 && !(SHAPE16 && SPLIT <= 0))
        return fail(LQ_ERR_INVALID, "this 256-row tile variant needs K %% 512 == 0, got %d", a.K);
    constexpr int TN = 256 / KG;
    const int blocks_n = (a.N + TN - 1) / TN, blocks_m = (a.M + 255) / 256;
    if ((long long)a.M * a.K >= (1ll << 32))
        return fail(LQ_ERR_INVALID, "M * K = %lld is beyond the 2^32 - 1 bytes of X one call addresses; split the batch",
                    (long long)a.M * a.K);
    if (a.N > (1 << 26))  // (a row's lane offsets are 32-bit byte offsets)
        return fail(LQ_ERR_INVALID, "the 256-row tile variants take N up to 2^26, got %d", a.N);
    const int cus = std::max(cu_count(), 1);
    int S = 1;
    if (SPLIT > 0) {
        S = SPLIT;
        if ((a.K / 512) % S != 0)
            return fail(LQ_ERR_INVALID, "%d K slices need K %% %d == 0, got %d", S, 512 * S, a.K);
    } else if (SPLIT < 0) {
        S = a.K % 512 != 0 ? 1 : solo_split(blocks_m * blocks_n, a.K, a.query ? (int)kAssumedCUs : cus);
        // (a workspace too small for them: the largest number of slices it holds)
        // (a query names its limit, if it has one, in ws_bytes)
        auto too_large = [&](int s) {
            const size_t need = solo_ws_bytes(a.M, a.N, s);
            return a.query ? a.ws_bytes > 0 && a.ws_bytes < need : !a.ws || a.ws_bytes < need;
        };
        while (S > 1 && too_large(S)) {
            do --S; while (S > 1 && (a.K / 512) % S != 0);
        }
    }
    const size_t need = solo_ws_bytes(a.M, a.N, S);
    if (a.query) return *a.query = need, LQ_OK;
    if (need > 0 && (!a.ws || a.ws_bytes < need))
        return fail(LQ_ERR_WORKSPACE, "%d K slices need %zu bytes of workspace, got %zu", S, need, a.ws ? a.ws_bytes : 0);
    int32_t *partials = S > 1 ? reinterpret_cast<int32_t *>(static_cast<char *>(a.ws) + kTicketBytes) : nullptr;
    const int grid = std::min(blocks_m * blocks_n * S, cus);
    const size_t lds_bytes = 4 * (size_t)256 * 128 + 4 * 1024;  // X stages; two copies of both scales
    __half *Y = S > 1 ? nullptr : a.Y;
    int32_t *ACC = S > 1 ? partials : a.ACC;
    if constexpr (SHAPE16) {
        if (a.group == 128) {
            if (int rc = allow_lds(w4a8_solo16_pt_kernel<true, KG>, lds_bytes)) return rc;
            hipLaunchKernelGGL((w4a8_solo16_pt_kernel<true, KG>), dim3((unsigned)grid), dim3(256), lds_bytes, a.stream, a.M,
                               a.N, a.K, blocks_m, blocks_n, S, a.X, a.Wp, a.gp, a.sx, a.sw, Y, ACC);
        } else {
            if (int rc = allow_lds(w4a8_solo16_pt_kernel<false, KG>, lds_bytes)) return rc;
            hipLaunchKernelGGL((w4a8_solo16_pt_kernel<false, KG>), dim3((unsigned)grid), dim3(256), lds_bytes, a.stream, a.M,
                               a.N, a.K, blocks_m, blocks_n, S, a.X, a.Wp, a.gp, a.sx, a.sw, Y, ACC);
        }
    } else if (a.group == 128) {
        if (int rc = allow_lds(w4a8_solo_pt_kernel<true, KG>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_solo_pt_kernel<true, KG>), dim3((unsigned)grid), dim3(256), lds_bytes, a.stream, a.M,
                           a.N, a.K, a.X, a.sx, a.Wp, a.gp, a.sw, Y, ACC, blocks_m, blocks_n, S);
    } else {
        if (int rc = allow_lds(w4a8_solo_pt_kernel<false, KG>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_solo_pt_kernel<false, KG>), dim3((unsigned)grid), dim3(256), lds_bytes, a.stream, a.M,
                           a.N, a.K, a.X, a.sx, a.Wp, a.gp, a.sw, Y, ACC, blocks_m, blocks_n, S);
    }
    if (S > 1) {
        const size_t quads = (size_t)a.M * a.N / 4;
        hipLaunchKernelGGL(splitk_finish_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, a.stream, partials,
                           S, a.M, a.N, a.sx, a.sw, a.Y, a.ACC);
    }
    return LQ_OK;
}

// the explicit producer / consumer form (measured only, never dispatched)
static int launch_excp(const Args &a)
{
    if (a.query) return LQ_OK;  // no workspace
    const int blocks_n = (a.N + 255) / 256, blocks_m = (a.M + 127) / 128;
    if ((long long)a.M * a.K >= (1ll << 32))
        return fail(LQ_ERR_INVALID, "M * K = %lld is beyond the 2^32 - 1 bytes of X one call addresses; split the batch",
                    (long long)a.M * a.K);
    const size_t lds_bytes = 2 * (size_t)128 * kTilePitch + 2 * (size_t)32 * 1024;
    const dim3 grid((unsigned)(blocks_n * blocks_m)), block(512);
    if (a.group == 128) {
        if (int rc = allow_lds(w4a8_excp_kernel<true>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_excp_kernel<true>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K, a.X, a.sx, a.Wp,
                           a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n);
    } else {
        if (int rc = allow_lds(w4a8_excp_kernel<false>, lds_bytes)) return rc;
        hipLaunchKernelGGL((w4a8_excp_kernel<false>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K, a.X, a.sx, a.Wp,
                           a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n);
    }
    return LQ_OK;
}

// The tiled kernel with the overflow-safe widened dequantisation in place of LiquidQuant's
// (the dequantisation half of the paper's ablation, Sec. 7.3; measured only, never dispatched).
static int launch_duo_widened(const Args &a)
{
    if (a.query) return LQ_OK;  // no workspace
    const int blocks_n = (a.N + 255) / 256, blocks_m = (a.M + 127) / 128;
    const size_t lds_bytes = 2 * (size_t)128 * kTilePitch;
    const dim3 grid((unsigned)(blocks_n * blocks_m), 1u), block(256);
    if (a.group == 128)
        hipLaunchKernelGGL((w4a8_duo_kernel<true, 1, 128, false, 1>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K,
                           a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, nullptr, nullptr);
    else
        hipLaunchKernelGGL((w4a8_duo_kernel<false, 1, 128, false, 1>), grid, block, lds_bytes, a.stream, a.M, a.N, a.K,
                           a.X, a.sx, a.Wp, a.gp, a.sw, a.Y, a.ACC, blocks_m, blocks_n, nullptr, nullptr);
    return LQ_OK;
}

// The same kernel on a grid of 64-row tiles (two row fragments per wave, two k groups per
// block): twice the tiles for a given M, half the partial-tile volume per slice.
static int duo64_split(int M, int N, int K)
{
    const int tiles = ((M + 63) / 64) * ((N + 255) / 256);
    const int units = K / 256;
    int s = (int)(0.6 * std::sqrt((double)units) + 0.5);  // minimum of the fitted cost below
    // with few tiles the exchange of a slice is cheap (few blocks share the memory system)
    s = std::max(s, tiles <= 40 ? 4 : tiles <= 64 ? 3 : 1);
    s = std::min(std::min(s, 256 / std::max(1, tiles)), std::min(units / 2, 8));
    return std::max(1, s);
}
template <int SPLIT>
static int launch_duo64(const Args &a)
{
    if (a.K < 512) return fail(LQ_ERR_INVALID, "the 64-row tiled variant needs K >= 512");
    return launch_duo_as<SPLIT, 2, 64>(a, SPLIT ? SPLIT : duo64_split(a.M, a.N, a.K));
}

// Which tile height for a problem with few tiles.  Fitted to measurements of both forms with
// two k groups per block (microseconds; u = 256-k units per k group, S = K slices):
//   128-row tiles: 13.9 + 1.95 u + 2.3 (S - 1)       64-row tiles: 8.1 + 1.76 u + c (S - 1),
//   c = 0.8 + 1.6 * blocks / 256 (a slice costs less when few blocks exchange at once)
static double duo_us(int M, int N, int K)
{
    const int s = duo_split(M, N, K), units = K / 256;
    return 13.9 + 1.95 * units / (2.0 * s) + 2.3 * (s - 1);
}
static double duo64_us(int M, int N, int K)
{
    const int t64 = ((M + 63) / 64) * ((N + 255) / 256), s = duo64_split(M, N, K), units = K / 256;
    return 8.1 + 1.76 * units / (2.0 * s) + (0.8 + 1.6 * t64 * s / 256.0) * (s - 1);
}
static bool prefer_64_row_tiles(int M, int N, int K)
{
    const int bn = (N + 255) / 256;
    const int t128 = ((M + 127) / 128) * bn, t64 = ((M + 63) / 64) * bn;
    if (K < 512 || t64 > 256 || t128 > 256) return false;
    const double est128 = duo_us(M, N, K), est64 = duo64_us(M, N, K);
    return est64 < est128;
}

// Where the dispatcher arrives at duo_m64 or duo_m128 it runs a panel form instead if that is estimated to
// be faster (a null form: it is not).  The estimate of the tiles is 2.5 us below its terms (the fits above
// include more launch time) and low by up to half for some shapes, by 18 % on average; with a factor of
// 1.15 the choice was 0.8 % from the better of both over 128 shapes of 96 to 512 rows (256 x 8192 x 8192:
// 27.2 against 30.6 us, 128 x 4096 x 11008: 15.8 against 21.2, 192 x 5120 x 5120: 12.8 against 18.3); the panel kernel is
// 4 to 8 % faster since, and over 1300 calls of 65 to 512 rows what runs is 4 to 6 % behind the best form or tile.  With
// more rows and more than 64 tiles of 128 x 256 the tiles stay ahead (384 x 6144 x 2048: 12.9 against 14.8 us,
// 1024 x 3072 x 3072: 17.5 against 18.9; with 64 tiles 500 x 4096 x 4096: 18.6 against 15.3).
static double few_tiles_us(int M, int N, int K);

// Where that estimate leaves a batch of 33 to 512 rows on duo_m64 or duo_m128, both sides are estimated once more, from 5200
// random calls (N from 1024, K from 2048, to 28672 each, weights from HBM), each form by itself: the panels' time without K slices is
// linear in their rounds, the units that a wave walks in each, how far the first round fills the CUs, and the packed weights
// (4 to 7 % rms, 11 % for 32 x 64); the tiles' in the same and in the volume of their slices (5 and 8 %).  With panels that have to
// win by 5 %, 594 of 892 such calls leave the tiles, at 0.87 of their time; 21 of them lose more than 2 %, one more than 8.  (104 x
// 16000 x 2304 18.3 / 11.7 us on 128 x 64 panels, 36 x 22464 x 6912 28.0 / 20.9 on 64 x 96, 312 x 6400 x 4096 21.0 / 14.0 on 64 x
// 128, 256 x 10240 x 8192 35.0 / 29.5 on 128 x 96.)  8300 calls on 10240 to 12672 channels with K up to 8192 and 12000 of 64 rows on
// 28672 and more, which kept the tiles for a time, take 0.81 and 0.84 of their time on the panels; of the former one loses 4 %, of the latter none.
static PanelChoice panel_instead_of_few_tiles(int M, int N, int K, bool rows64)
{
    struct Cost {
        int F, MF;
        double fixed, round, unit, fill, mb;
    };
    static const Cost kCosts[] = {
        {2, 1, 1.391, 1.239, 0.683, 0.346, 0.099}, {3, 1, 1.556, 2.466, 1.006, 0.093, 0.092}, {4, 1, 0.744, 3.720, 1.253, 0.101, 0.096},
        {2, 2, 1.068, 2.347, 1.029, 0.121, 0.089}, {3, 2, 0.461, 4.470, 1.263, 0.232, 0.081}, {4, 2, 0.371, 4.939, 1.509, 0.351, 0.076},
        {2, 4, 1.045, 4.068, 0.815, 0.131, 0.088}, {3, 4, 0.000, 8.265, 1.014, 0.271, 0.056}, {4, 4, 0.000, 9.031, 1.183, 0.524, 0.033},
    };
    PanelChoice best;
    if (M <= 32 || M > 512 || N < 1024 || K < 2048) return best;
    const double mb = 0.5e-6 * N * K;
    for (const Cost &c : kCosts) {
        const PanelForm &f = panel_form(c.F, c.MF);
        const long long blocks = panel_blocks(M, N, c.F, c.MF);
        const bool two = c.F == 2 && c.MF == 1;  // (two 32 x 64 panels fit a CU)
        if (c.F > 2 && c.MF == 4 && K < 2816) continue;  // (0.97 there, a seventh of them behind)
        if (blocks > (two ? 4 : K <= 8192 ? 2 : 1) * kAssumedCUs) continue;  // (a second round with longer K: 0.98, a quarter of them behind)
        const double fill = (double)blocks / kAssumedCUs, units = (K / 128 + f.NW - 1) / f.NW;
        const double rounds = two ? std::max(fill, 1.0) : std::ceil(fill);
        const double us = c.fixed + rounds * (c.round + c.unit * units) + c.fill * std::min(fill, 1.0) * units + c.mb * mb;
        if (us < best.us) best = PanelChoice{&f, 1, us};
    }
    const int bn = (N + 255) / 256, tiles = rows64 ? (M + 63) / 64 * bn : (M + 127) / 128 * bn;
    const int S = rows64 ? duo64_split(M, N, K) : duo_split(M, N, K);
    const double fill = (double)tiles * S / kAssumedCUs, k = K / 1024.0 / S, volume = (S - 1) * (double)tiles / kAssumedCUs;
    const double us = rows64 ? std::ceil(fill) * (7.394 + 2.299 * k) + 1.778 * std::min(fill, 1.0) * k + 7.466 * volume + 0.063 * mb
                             : std::ceil(fill) * (9.415 + 3.473 * k) + 3.654 * std::min(fill, 1.0) * k + 11.112 * volume + 0.023 * mb;
    return best.us < 0.95 * us ? best : PanelChoice{};
}
static PanelChoice panel_instead_of_tiles(const Args &a, bool rows64)
{
    if (a.M <= 256 || (long long)((a.M + 127) / 128) * ((a.N + 255) / 256) <= 64) {
        const PanelChoice c = choose_panel(a.M, a.N, a.K, workspace_limit(a));
        if (c.form && c.us < 1.15 * few_tiles_us(a.M, a.N, a.K)) return c;
    }
    return panel_instead_of_few_tiles(a.M, a.N, a.K, rows64);
}

struct Variant {
    const char *name;
    LaunchFn fn;
    int max_m;      // 0 = unlimited
    int tiles_div;  // N/32 must be a multiple of this
    int chunks_div; // K/64 must be a multiple of this
    int min_k = 256;
};

// stream_m32, stream_m64, stream_f*, stream_x*, stream_m64x*: panel forms for up to 32 and 64 rows
// (the names of the kernels they took the place of).  panel_f<F>_m<rows>[_s<S>]: F tiles
// and 32, 64 or 128 rows per block.  duo_m64, duo_m128: few 64- or 128-row tiles, K split over blocks (the
// dispatcher runs a panel form in their place where that is faster).  stream16_f<F>_w<NW>[_s<S>]: F tiles per block, NW waves splitting the block's K slice,
// S grid-level K slices (chosen from the shape when not named); _u4 = four 128-k units per
// pipeline step; stream16_h_w<NW>_d<D>: half a tile per block, D units per step (in_place_of_stream16); g2 = two k groups per block.
static const Variant kVariants[] = {
    // --- dispatched (select_variant) ---
    {"stream16_f1_w16_s1", &launch_stream16<1, 16, 1>, 16, 1, 1},
    {"stream16_f1_w8_u4", &launch_stream16<1, 8, 0, 4>, 16, 1, 8},
    {"stream16_f1_w8", &launch_stream16<1, 8, 0>, 16, 1, 1},
    {"stream16_f2_w8", &launch_stream16<2, 8, 0>, 16, 2, 1},
    {"stream16_f2_w16_s1", &launch_stream16<2, 16, 1>, 16, 2, 1},
    {"stream16_f2_w4", &launch_stream16<2, 4, 0>, 16, 2, 1},
    {"stream16_h_w8_d2", &launch_stream16_half<8, 2, 1>, 16, 1, 1},
    {"stream16_h_w8_d3", &launch_stream16_half<8, 3, 1>, 16, 1, 1},
    {"stream16_h_w8_d4", &launch_stream16_half<8, 4, 1>, 16, 1, 1},
    {"stream16_h_w16_d3", &launch_stream16_half<16, 3, 1>, 16, 1, 1},
    {"stream16_h_w16_d4", &launch_stream16_half<16, 4, 1>, 16, 1, 1},
    {"stream16_h_w8_d2_s2", &launch_stream16_half<8, 2, 2>, 16, 1, 1},
    {"stream16_h_w8_d3_s2", &launch_stream16_half<8, 3, 2>, 16, 1, 1},
    {"stream16_h_w8_d4_s2", &launch_stream16_half<8, 4, 2>, 16, 1, 1},
    {"panel_f1_m32", &launch_panel_named<1, 8, 1, 1>, 0, 1, 1},
    {"stream_m32", &launch_panel_auto, 32, 2, 1},
    {"stream_m64", &launch_panel_auto, 64, 2, 1},
    {"duo_m64", &launch_duo64<0>, 0, 1, 1, 512},
    {"duo_m128", &launch_duo<0, 0>, 0, 1, 1},
    {"duo_dl_m128", &launch_duo_dl<0>, 0, 1, 1},
    {"duo_pt_m128", &launch_duo_pt, 0, 1, 8, 512},
    {"solo16_pt_m256", &launch_solo_pt<1, 0, true>, 0, 1, 4},
    {"solo16_g2_m256", &launch_solo_pt<2, 0, true>, 0, 1, 4},
    {"solo16_g2_sk_m256", &launch_solo_pt<2, -1, true>, 0, 1, 8, 512},
    // --- the 256-row tile kernels on the 32x32x32 MFMA (what the 16x16x64 forms are measured against) ---
    {"solo_pt_m256", &launch_solo_pt<1>, 0, 1, 8, 512},
    {"solo_g2_m256", &launch_solo_pt<2>, 0, 1, 8, 512},
    // --- the same kernels with a named number of K slices: the split paths at sizes where the
    //     dispatcher would not split (parity tests) ---
    {"stream16_f2_w8_s2", &launch_stream16<2, 8, 2>, 16, 2, 1},
    {"stream16_f1_w8_u4_s2", &launch_stream16<1, 8, 2, 4>, 16, 1, 8},
    {"stream_f2_w8_s2", &launch_panel_named<2, 8, 1, 2>, 32, 2, 1},
    {"stream_x_f1_w8_s2", &launch_panel_named<1, 8, 1, 2>, 32, 1, 1},
    {"stream_m64x_f1_w8_s2", &launch_panel_named<1, 8, 2, 2>, 64, 1, 1},
    {"stream_m64x_f2_w8_s4", &launch_panel_named<2, 8, 2, 4>, 64, 2, 1},
    {"panel_f4_m32_s2", &launch_panel_named<4, 8, 1, 2>, 0, 1, 1},
    {"panel_f3_m64_s2", &launch_panel_named<3, 8, 2, 2>, 0, 1, 1},
    {"panel_f4_m64_s3", &launch_panel_named<4, 8, 2, 3>, 0, 1, 1},
    {"duo_m64_s2", &launch_duo64<2>, 0, 1, 1, 512},
    // (... and the panel forms without slices)
    {"panel_f1_m64", &launch_panel_named<1, 8, 2, 1>, 0, 1, 1},
    {"panel_f2_m32", &launch_panel_named<2, 8, 1, 1>, 0, 1, 1},
    {"panel_f4_m64", &launch_panel_named<4, 8, 2, 1>, 0, 1, 1},
    {"panel_f3_m128", &launch_panel_named<3, 4, 4, 1>, 0, 1, 1},
    {"panel_f4_m128", &launch_panel_named<4, 4, 4, 1>, 0, 1, 1},
    {"duo_m128_s1", &launch_duo<1, 1>, 0, 1, 1},
    {"duo_m128_s2", &launch_duo<2, 1>, 0, 1, 1},
    {"duo_m128_g2_s2", &launch_duo<2, 2>, 0, 1, 1},
    {"duo_dl_m128_s2", &launch_duo_dl<2>, 0, 1, 1},
    {"solo16_pt_m256_s2", &launch_solo_pt<1, 2, true>, 256, 1, 16, 1024},
    {"solo16_g2_m256_s4", &launch_solo_pt<2, 4, true>, 256, 1, 32, 2048},
    // --- ablation forms (Sec. 7.3), measured by the benchmark, never dispatched ---
    {"excp_m128", &launch_excp, 0, 1, 1},
    {"widened_dq_m128", &launch_duo_widened, 0, 1, 1},
    // (panel forms that were added last: indices are part of the interface)
    {"panel_f3_m32", &launch_panel_named<3, 8, 1, 1>, 0, 1, 1},
    {"panel_f2_m128", &launch_panel_named<2, 4, 4, 1>, 0, 1, 1},
};
constexpr int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));

static bool variant_supports(int v, int M, int N, int K)
{
    const Variant &x = kVariants[v];
    return (x.max_m == 0 || M <= x.max_m) && (N / 32) % x.tiles_div == 0 && (K / 64) % x.chunks_div == 0 &&
           K >= x.min_k;
}

static int find_variant(const char *name)
{
    for (int i = 0; i < kNumVariants; ++i)
        if (!strcmp(kVariants[i].name, name)) return i;
    return -1;
}

static bool is_64_row_tiles(int variant) { return kVariants[variant].fn == &launch_duo64<0>; }
static bool is_few_tiles(int variant) { return is_64_row_tiles(variant) || kVariants[variant].fn == &launch_duo<0, 0>; }

// The 256-row tiles with one wave per SIMD (solo16_pt_m256: 256 x 256; solo16_g2_m256: 256 x 128
// with two k groups per block) against the 128 x 256 tiles with two waves per SIMD.  Half the
// dequantisation per MFMA makes their stage loop shorter -- per 128 x 256 of output and 1024 k,
// 6.0 us (256 x 256) and 7.0 us (256 x 128) against 7.1 to 7.4 us measured on N = K = 8192 --
// but they run one block per CU, in whole rounds, and rows past M in a 256-row tile are lost.
// Costs in units of one 128 x 256 tile's time on a CU, from the numbers of tiles of each form;
// returns 1 for 256 x 256, 2 for 256 x 128, 0 for neither.
struct TiledCosts {
    double duo, solo, g2;
    double best() const { return std::min(duo, std::min(solo, g2)); }
};
// (pt_ok: the persistent form of the 128-row tiles can run the shape)
static TiledCosts tiled_costs(long long t128, long long t256, long long t2, int K, bool pt_ok)
{
    // (K % 512 == 256: the 16x16x64 forms of the 256-row tiles run two added stages of zero weights,
    // the persistent form of the 128-row tiles does not take the shape -- pt_ok is false then)
    // No form's cost is proportional to its tiles while these leave CUs idle or half occupied (a
    // partly filled chip clocks higher).  Fitted to measurements on K = 8192 (us / 64, so that a
    // round of 256 128-row tiles, one per CU, costs about 1):
    //   128-row tiles, K slices across blocks up to 128 tiles:  29.6 / 38.7 / 44 us at 64 / 96 / 128
    //   ... 129..256 tiles, persistent form (one block per CU): 50.6 / 57.3 / 63.5 at 160 / 192 / 256
    //       (one tile per block: 56 / 60 / 67)
    //   ... 257..512 tiles (a second resident block on some CUs): 85 / 95 / 102 / 111 / 116 at 270 / 320 / 384 / 448 / 512
    //   ... beyond: whole rounds of 512 at 2 each, the rest as above
    //   256 x 256 tiles, one round: 84 / 93 / 107 at 160 / 192 / 256 tiles; more: whole rounds at 2 * 0.86
    //   256 x 128 tiles, one round of more than half the CUs: 45.8 / 49 / 56 / 61.5 at 144 / 160 / 192 / 256
    //       (at 128 tiles equal to the 128-row tiles; their tiles are separate, a second round costs a tenth more)
    // one round of up to 512 tiles (or the rest after whole rounds of 512: 4096 + 40 rows on 8192 x 8192,
    // 1056 tiles, took 259 us against 235 us of 4096 rows)
    auto part = [](long long t) {
        const double fill = (double)t / kAssumedCUs;
        return t == 0 ? 0.0 : 2 * t <= kAssumedCUs ? 0.24 + 0.90 * fill : t <= kAssumedCUs ? 0.47 + 0.52 * fill : 0.80 + 0.51 * fill;
    };
    const double fill = (double)t128 / kAssumedCUs;
    const double duo = t128 <= kAssumedCUs && 2 * t128 > kAssumedCUs && !pt_ok
                           ? 0.60 + 0.45 * fill
                           : 2.0 * (t128 / (2 * kAssumedCUs)) + part(t128 % (2 * kAssumedCUs));
    const double short_k = K >= 4096 ? 1.0 : 1.06;  // (their longer epilogue weighs more)
    // (those were measured with the 32x32x32 MFMA; on the 16x16x64 one the 256 x 256 tiles take 8 % less)
    const double solo = (t256 <= kAssumedCUs ? 0.734 + 0.94 * t256 / kAssumedCUs
                                             : 2.0 * ((t256 + kAssumedCUs - 1) / kAssumedCUs) * 0.86) * short_k * 0.92;
    // (... and the 256 x 128 tiles 1 to 5 % less, most on a full round: 57.4 against 60.4 us at 256 tiles,
    // 48.8 against 50.5 at 192, 28.3 against 28.5 at 172 tiles with K = 4096)
    const double g2 = 16 * t2 > 8.5 * kAssumedCUs && t2 <= kAssumedCUs
                          ? (0.406 + 0.56 * t2 / kAssumedCUs) * short_k * (1.0 - 0.05 * t2 / kAssumedCUs)
                          : 1e30;
    return TiledCosts{duo, solo, g2};
}
static TiledCosts tiled_costs(int M, int N, int K)
{
    const long long bm256 = (M + 255) / 256;
    return tiled_costs((long long)((M + 127) / 128) * ((N + 255) / 256), bm256 * ((N + 255) / 256),
                       bm256 * ((N + 127) / 128), K, K % 512 == 0);
}
static double few_tiles_us(int M, int N, int K)
{
    const int bn = (N + 255) / 256, t128 = ((M + 127) / 128) * bn, t64 = ((M + 63) / 64) * bn;
    const TiledCosts c = tiled_costs(M, N, K);
    const double round_us = 60.0 * K / 8192;
    double us = std::min(c.solo, c.g2) * round_us + 4;
    if (t128 > 128) us = std::min(us, c.duo * round_us + 4);
    else us = std::min(us, duo_us(M, N, K));
    if (t128 <= 128 && t64 <= 256) us = std::min(us, duo64_us(M, N, K));
    return us - 2.5;
}
static int solo_form_of(const TiledCosts &c)
{
    if (c.solo < c.duo && c.solo <= c.g2) return 1;
    if (c.g2 < c.duo) return 2;
    return 0;
}
static int solo_form_for(long long t128, long long t256, long long t2, int K)
{
    return solo_form_of(tiled_costs(t128, t256, t2, K, false));
}
static int solo_form_that_pays(int M, int N, int K) { return solo_form_of(tiled_costs(M, N, K)); }

// Shape -> kernel.  Up to 16 rows the 16-row kernel, up to 64 the panels while N alone does not fill the
// chip with tiles, then tiles of 256, 128 or 64 rows by cost; where these are few (duo_m64, duo_m128) the
// dispatcher compares a panel form once more (panel_instead_of_tiles).
static int select_variant(int M, int N, int K)
{
    if (M <= 16) {
        // Measured over 36 weight shapes (N, K from 2048 to 28672) at 1, 8 and 16 rows.
        const int tiles = N / 32;
        if (tiles <= 256) {
            // one tile per block.  Short K is bound by launch and first-load latency: sixteen
            // waves per block take one or two units of 128 k each ...
            if (K <= 4096) return find_variant("stream16_f1_w16_s1");
            if (K <= 8192 && K % 512 == 0) {
                // ... up to 8192, all of a wave's loads (512 k) in flight at once; from 9 rows
                // K slices across blocks while N leaves room for them, else sixteen waves again
                if (M <= 8) return find_variant("stream16_f1_w8_u4");
                return find_variant(tiles <= 128 ? "stream16_f1_w8" : "stream16_f1_w16_s1");
            }
            // 129..256 tiles and long K (no room for K slices across blocks): up to 8 rows, sixteen
            // waves per block split K (21.5 instead of 26 us on 8192 x 28672, 12.4 / 17.8 on
            // 6144 x 16384); above, two tiles per block and two K slices (23.3 / 25.9, 14.8 / 15.7)
            if (tiles > 128 && M <= 8 && K >= 12288) return find_variant("stream16_f1_w16_s1");
            if (tiles > 128 && M > 8 && K >= 16384) return find_variant("stream16_f2_w8");
            // otherwise 2 or 4 K slices across blocks
            return find_variant("stream16_f1_w8");
        }
        // up to 512 tiles with short K: sixteen waves again (8.1 instead of 9.1 us on 16384 x 4096)
        if (tiles <= 512 && K <= 4096) return find_variant(M <= 8 ? "stream16_f1_w16_s1" : "stream16_f2_w16_s1");
        if (N / 64 >= 384) return find_variant(K <= 2048 ? "stream16_f2_w8" : "stream16_f2_w4");
        return find_variant("stream16_f2_w8");
    }
    if (M <= 32) return find_variant("stream_m32");
    // up to 64 rows the panels, unless N alone fills the chip with 128 x 256 tiles.  (48 rows and more on
    // 129..256 tiles of 32 channels with very long K arrive at duo_m64 / duo_m128 below, where the estimates
    // pick a panel again: 26.2 against 31.2 us on the tiles for 48 x 6144 x 28672, 31.6 / 35.2 for 64 x 8192 x 28672.)
    if (M <= 64 && N / 32 <= 512 && !(M >= 48 && N / 32 > 128 && N / 32 <= 256 && K >= 24576))
        return find_variant("stream_m64");
    // 256-row tiles with one wave per SIMD where their whole rounds come out ahead
    if (const int form = solo_form_that_pays(M, N, K)) return find_variant(form == 1 ? "solo16_pt_m256" : "solo16_g2_m256");
    // ... and, with very long K and row tiles that are nearly full, their 256 x 128 form with K
    // slices across blocks where tiles x slices come to one round of at least three quarters of the
    // CUs (256 x 8192 x 28672: 65 against 70 us; 512 rows: 114 against 121; 256 x 6144 x 16384: 37
    // against 40; shorter K or emptier rounds: equal or behind -- the partial sums are a matrix per slice)
    if (K >= 16384 && K % 512 == 0 && (M % 256 == 0 || M % 256 > 192)) {
        const long long t2 = (long long)((M + 255) / 256) * ((N + 127) / 128);
        if (t2 <= kAssumedCUs / 2) {
            const int slices = solo_split((int)t2, K, (int)kAssumedCUs);
            if (slices > 1 && 4 * t2 * slices >= 3 * kAssumedCUs) return find_variant("solo16_g2_sk_m256");
        }
    }
    // more 128 x 256 tiles than CUs (blocks of one k group): the deeper memory pipeline of the
    // direct-to-LDS form pays (3 to 6 % measured from 320 tiles up, 1 to 5 % at 264..288); with
    // one tile per CU or fewer, the two k groups per block of the other form do
    // (from two tiles per resident slot on and with whole 512-k units, its persistent form:
    // one pipeline fill per block instead of per tile, 1 to 2 % measured)
    const int tiles128 = ((M + 127) / 128) * ((N + 255) / 256);
    if (tiles128 > 256) return find_variant(duo_pt_fits(M, N, K) ? "duo_pt_m128" : "duo_dl_m128");
    // more than half a round of them (no room for K slices across blocks): the persistent form again,
    // one block per CU -- 50.6 against 56.1 us on 640 x 8192 x 8192, 28.0 against 31.1 on 384 x 11008 x 4096
    // (also with a ragged last row tile of at most 64 rows: 47.8 against 50.9 us on 576 x 8192 x 8192)
    if (tiles128 > 128 && K % 512 == 0) return find_variant("duo_pt_m128");
    // few tiles: a grid of 64-row tiles can fill the chip with half the split-K exchange
    return find_variant(prefer_64_row_tiles(M, N, K) ? "duo_m64" : "duo_m128");
}

// Up to 16 rows: the form that runs where select_variant names a stream16 variant of whole tiles (null: that variant itself).
// From 8000 random calls (N 1024..28672, K 2048..28672, groups of 64 and 128, 1 to 16 rows, weights from HBM), all forms of each timed in
// turn; the figures are times against what ran before (geometric means).  What decides: how evenly the blocks fill 256
// CUs, and how many bytes a CU has in flight (64 to 128 KB; sixteen waves of one tile, or panels two units ahead, hold
// most).  Half tiles do where all of a wave's units are in flight at once: 32 units of K in two passes of two, 48 of three,
// 64 of four.  Fewer than 32 tiles keep the rules of an audit of their own (N from 64).
static const char *form_up_to_16_rows(int M, int N, int K)
{
    const int tiles = N / 32;
    const bool some = tiles >= 32;  // (N >= 1024)
    if (tiles <= 128) {
        // 256 instead of 128 blocks at N = 4096 and no K slices: at 4 rows 4096 x 4096 5.3 / 4.5 us, 4096 x 11008 8.9 / 7.2, 1024 x
        // 4096 5.1 / 4.0.  Shorter K keeps whole tiles: a wave of half tiles issues four units' loads whatever there is (K =
        // 256 3.0 / 3.4, 1536 3.60 / 3.64, 2048 3.76 / 3.67).  X is read twice as often, so from 13 rows long K keeps whole tiles too.
        if (K < 2048) return nullptr;
        const int few = K <= 49152 ? 8 : 7;  // (beyond 8 rows are behind, 1.01 over 64 calls, 7 rows 0.95)
        if (K <= 4096) return "stream16_h_w8_d2";
        if (K <= 6144) return "stream16_h_w8_d3";
        // two units a pass in four passes against four in two: 0.97 up to 4 rows, 0.98 up to 8, equal above
        if (K <= 8192) return tiles <= 64 && M > 12 ? "stream16_h_w8_d2_s2" : M <= 8 && some ? "stream16_h_w8_d2" : "stream16_h_w8_d4";
        if (tiles <= 64) {
            // two slices of K fill the CUs (2048 x 14336 at 4 rows 8.3 / 7.2; one slice 7.6), with up to 16 tiles for up to 10 rows (320 x
            // 12544 at 12 rows 6.9 / 7.3); up to 4 rows and K = 12288 one slice is ahead (0.90 to 0.96)
            const int most = tiles <= 16 ? 10 : 12;
            if (K <= 12288) return M <= 4 && some ? "stream16_h_w8_d2" : M <= most ? "stream16_h_w8_d3_s2" : nullptr;
            if (K <= 16384) return M <= most ? "stream16_h_w8_d4_s2" : nullptr;
            return (M <= 4 && K <= 20480) || (M <= few && some) ? "stream16_h_w8_d2_s2" : nullptr;  // (beyond 20480: 0.88 / 0.93 up to 4 / 8 rows)
        }
        if (K <= 16384) {
            if (M <= 4 && K <= 10240) return "stream16_h_w8_d2";  // (0.96; beyond equal to three units in sixteen waves)
            return M > 12 ? nullptr : K <= 12288 ? "stream16_h_w16_d3" : "stream16_h_w16_d4";
        }
        return M <= few ? "stream16_h_w8_d2" : nullptr;  // (0.78 / 0.85 up to 4 / 8 rows)
    }
    if (tiles <= 256) {
        // one block a CU or less: up to 8 rows sixteen waves of one tile (K 4352..5888 0.91 / 0.93 up to 4 / 8 rows, 6400..8192 0.96 /
        // 0.92, 8448..12032 0.94 / 0.96: 32-row panels 1.06 / 1.03 of it at 8448, 1.07 / 1.05 at 8960), above 32-row panels (K 5376..6144 0.97, 16640..24576 0.95), but not for 9 and 10 rows where
        // all sixteen waves' loads are in flight at once (7360 x 7168 at 9 rows 1.03 to 1.07 of the time on panels)
        if (M <= 8) {
            if (K <= 4096 || K >= 12288) return nullptr;
            // ... but half tiles where their passes are full or nearly so: two of three units for 46 to 48 units (0.96 / 0.97 up to 4
            // / 8 rows; 44 units 1.02 / 1.04), up to 4 rows two of four for 62 to 64 (0.97; 56 to 60 units 1.03 to 1.04)
            if (K > 5632 && K <= 6144) return "stream16_h_w8_d3";
            return M <= 4 && K > 7680 && K <= 8192 ? "stream16_h_w8_d4" : "stream16_f1_w16_s1";
        }
        if (K > 24576) return nullptr;  // (0.98, at 28672 behind)
        if (K > 16384 || (K > 8192 && K < 12288)) return "panel_f1_m32";
        return K >= 5376 && M >= (K <= 8192 && K % 512 == 0 ? 11 : 9) ? "panel_f1_m32" : nullptr;
    }
    if (tiles <= 384) {
        // half tiles where K is close below 4096 or 6144 (4 x 11008 x 4096 8.1 / 7.25 us; K = 3072 0.97, 2816 1.01; at 5 to 8 rows
        // from 3584 on), else panels of 32 x 64 (K to 6144 0.96, to 12288 0.95, beyond 0.88 to 0.97; above 28672 0.90 over 948 calls, but 13 of
        // them more than 4 % behind, at worst 6 x 11776 x 73728 87 / 103 us)
        if (K <= 4096) return (M <= 4 && K >= 3072) || (M <= 8 && K >= 3584) ? "stream16_h_w8_d2" : nullptr;
        if (M <= 4 && K >= 4864 && K <= 8192) return K <= 6144 ? "stream16_h_w8_d3" : "stream16_h_w8_d4";
        return "panel_f2_m32";
    }
    if (tiles <= 512) {
        // up to 224 blocks of two tiles the same panels (0.94 to 0.98); with more these are between 0.97 and 1.25 of the time, from one
        // machine to another, and one tile a block is ahead for few rows (0.97)
        if (K <= 4096) return nullptr;
        if (tiles <= 448) return "panel_f2_m32";
        return M <= 4 && K <= 12288 ? "stream16_f1_w8" : nullptr;
    }
    if (K < 2048) return nullptr;
    if (tiles <= 768) {
        // blocks of two tiles are two on some CUs and one on others (257..384 of them); one tile a block is at most three on
        // every CU: 0.80 to 0.86 for K to 6144, beyond with sixteen waves 0.82 to 0.85 up to 8 rows; with more, 0.87 to K = 8192, panels
        // of 32 x 32 0.86 to 0.88 and two slices of K 0.83 to 0.86 (12 x 24192 x 11776 33.2 / 29.1 us)
        if (K <= 6144) return "stream16_f1_w8";
        if (M <= 8 || K <= 8192) return "stream16_f1_w16_s1";
        return K <= 16384 ? "panel_f1_m32" : "stream16_f2_w8_s2";
    }
    if (tiles <= 896) {
        // (0.92 and 0.94; 0.96 to 0.98: 16 x 28672 x 8192 25.3 / 24.6 us; from 9 rows on K = 2048, which has eight waves a block before
        // it, 1.02 on panels)
        if (M <= 8 && K <= 4096) return "stream16_f1_w8";
        return K <= 2048 ? nullptr : "panel_f2_m32";
    }
    return nullptr;
}
static int in_place_of_stream16(int variant, const Args &a)
{
    const char *name = form_up_to_16_rows(a.M, a.N, a.K);
    if (!name) return variant;
    const int other = find_variant(name);
    Args query = a;
    size_t need = 0;
    query.query = &need;
    if (kVariants[other].fn(query) || need > workspace_limit(a)) return variant;
    return other;
}

// A batch whose 256 x 256 tiles are whole rounds plus a few rows (4096 + 40 rows on 8192 x 8192)
// is better run as two launches over consecutive rows: the row blocks that fill whole rounds with
// the 256 x 256 tiles, and the rest with whatever the dispatcher picks for it -- 226 us against
// 259 us of the best single kernel there.  Also with a larger rest, unless the rest would run on
// 256 x 256 tiles itself (then the one persistent launch over all tiles is 1 to 5 % ahead of two):
// 1536 + 512 rows on the 70B qkv projection 143 against 150 us, 2048 + 1024 on 8192 x 8192 157
// against 162, 1024 + 256 on 28672 x 8192 240 against 255, 2048 + 512 on 8192 x 8192 143 against
// 156 and on 8192 x 28672 423 against 513, 3072 + 512 on 5120 x 13824 201 against 245, 4096 + 1024
// on 4096 x 4096 78 against 84 (4096 + 1904 on 4096 x 4096 and 4096 + 1024 on 8192 x 8192: equal).
// Same cost units as solo_form_for; a second launch is charged 5 us
// (2048 + 100 rows on 8192 x 4096: 55.7 + 16.2 us against 78.4 us of the best single kernel; 1024 + 30 rows on
// 16384 x 4096: 56 + 11.3 against 79.7).  Returns
// the rows of the first piece (M if the batch stays whole).
static int rows_of_first_launch(int M, int N, int K)
{
    if (M <= 256) return M;
    const int bm = (M + 255) / 256, bn = (N + 255) / 256;
    double best = tiled_costs(M, N, K).best() * 0.97;  // (a split has to win by 3 %)
    const double second_launch = 5.0 / (8.0 * K / 1024.0);  // (a unit is 64 us at K = 8192)
    const double short_k = K >= 4096 ? 1.0 : 1.06;
    int rows = M;
    for (int rounds = 1; rounds <= 8; ++rounds) {
        const int rb = (int)(kAssumedCUs * rounds / bn);  // row blocks whose tiles fill `rounds` rounds
        if (rb >= bm) break;
        if (rb < 1) continue;
        const TiledCosts rest = tiled_costs(M - 256 * rb, N, K);
        // (a larger rest not where it would be 256 x 256 tiles again: the one persistent launch
        // over all of them is 1 to 5 % ahead of two)
        if (M - 256 * rb > 256 && solo_form_of(rest) == 1) continue;
        const double c = rounds * 2.0 * 0.86 * 0.92 * short_k + rest.best() + second_launch;
        if (c < best) best = c, rows = 256 * rb;
    }
    return rows;
}

static int check_device_args(const Args &a)
{
    if (a.M < 0 || !shape_ok(a.N, a.K, a.group))
        return fail(LQ_ERR_INVALID,
                    "bad shape M=%d N=%d K=%d group=%d (need M>=0, N%%64==0, K%%256==0, group 64|128, K<=131072)",
                    a.M, a.N, a.K, a.group);
    if (a.M == 0) return LQ_OK;  // nothing to read or write; pointers may be null
    if (!a.Y && !a.ACC) return fail(LQ_ERR_INVALID, "no output pointer");
    if (!a.X || !a.Wp || !a.gp) return fail(LQ_ERR_INVALID, "null input pointer");
    if (a.Y && (!a.sx || !a.sw)) return fail(LQ_ERR_INVALID, "null scale pointer");
    const uintptr_t bits = (uintptr_t)a.X | (uintptr_t)a.Wp | (uintptr_t)a.gp | (uintptr_t)a.sx |
                           (uintptr_t)a.sw | (uintptr_t)a.Y | (uintptr_t)a.ACC;
    if (bits & 15) return fail(LQ_ERR_ALIGN, "device pointers must be 16-byte aligned");
    return LQ_OK;
}

static void panel_name(const PanelChoice &c, char *text, size_t text_bytes)
{
    const int n = snprintf(text, text_bytes, "panel_f%d_m%d", c.form->F, 32 * c.form->MF);
    if (c.S > 1 && (size_t)n < text_bytes) snprintf(text + n, text_bytes - n, "_s%d", c.S);
}

static int run_rows(int variant, const Args &a)
{
    const bool dispatched = variant < 0;
    if (dispatched) variant = select_variant(a.M, a.N, a.K);
    if (variant < 0 || variant >= kNumVariants) return fail(LQ_ERR_INVALID, "unknown variant %d", variant);
    if (!variant_supports(variant, a.M, a.N, a.K))
        return fail(LQ_ERR_INVALID, "variant %s cannot run M=%d N=%d K=%d", kVariants[variant].name, a.M, a.N,
                    a.K);
    (void)hipGetLastError();
    // The tiled kernels address X with 32-bit byte offsets.  A batch with M * K >= 2^32 is
    // run as consecutive row chunks (multiples of 256 rows, so every chunk keeps the
    // alignment and the tile grid of a call of its own) on the same stream; rows are
    // independent, so the result is that of one launch.
    const long long rows_max = ((1ll << 32) - 1) / a.K / 256 * 256;
    size_t need_max = 0;
    int ran = variant;  // (for the error below)
    PanelChoice ran_panel;
    for (long long r0 = 0; r0 < a.M; r0 += rows_max) {
        Args c = a;
        size_t need = 0;
        if (a.query) c.query = &need;
        c.M = (int)std::min<long long>(rows_max, a.M - r0);
        c.X = a.X + r0 * a.K;
        if (a.sx) c.sx = a.sx + r0;
        if (a.Y) c.Y = a.Y + r0 * a.N;
        if (a.ACC) c.ACC = a.ACC + r0 * a.N;
        const int runs = dispatched && a.M <= 16 ? in_place_of_stream16(variant, c) : variant;
        const PanelChoice panel = dispatched && is_few_tiles(variant) ? panel_instead_of_tiles(c, is_64_row_tiles(variant)) : PanelChoice{};
        if (int rc = panel.form ? panel.form->launch(c, panel.S) : kVariants[runs].fn(c)) return rc;
        ran = runs, ran_panel = panel;
        need_max = std::max(need_max, need);
    }
    if (a.query) return *a.query = need_max, LQ_OK;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        char panel[32];
        if (ran_panel.form) panel_name(ran_panel, panel, sizeof(panel));
        return fail(LQ_ERR_HIP, "launch of %s failed: %s", ran_panel.form ? panel : kVariants[ran].name, hipGetErrorString(e));
    }
    return LQ_OK;
}

static int run(int variant, const Args &a)
{
    if (int rc = check_device_args(a)) return rc;
    if (a.M == 0) return LQ_OK;
    const int first = variant < 0 ? rows_of_first_launch(a.M, a.N, a.K) : a.M;
    if (first == a.M) return run_rows(variant, a);
    // two launches on the same stream (rows are independent); a workspace serves both in turn
    Args head = a, rest = a;
    size_t need_head = 0, need_rest = 0;
    if (a.query) head.query = &need_head, rest.query = &need_rest;
    head.M = first;
    rest.M = a.M - first;
    rest.X = a.X + (size_t)first * a.K;
    if (a.sx) rest.sx = a.sx + first;
    if (a.Y) rest.Y = a.Y + (size_t)first * a.N;
    if (a.ACC) rest.ACC = a.ACC + (size_t)first * a.N;
    if (int rc = run_rows(find_variant("solo16_pt_m256"), head)) return rc;
    if (int rc = run_rows(-1, rest)) return rc;
    if (a.query) *a.query = std::max(need_head, need_rest);
    return LQ_OK;
}

// The name of the kernel that a launch over the given rows runs (with all K slices), to `text`.
static void launch_name(int variant, int M, int N, int K, char *text, size_t text_bytes)
{
    Args a{};
    size_t unused = 0;
    a.M = M, a.N = N, a.K = K, a.query = &unused;
    const bool dispatched = variant < 0;
    if (dispatched) variant = select_variant(M, N, K);
    if (dispatched && M <= 16) {
        const int runs = in_place_of_stream16(variant, a);
        if (runs != variant) {
            snprintf(text, text_bytes, "%s[as %s]", kVariants[variant].name, kVariants[runs].name);
            return;
        }
    }
    PanelChoice panel{};
    if (kVariants[variant].fn == &launch_panel_auto) panel = choose_panel(M, N, K, workspace_limit(a));
    else if (dispatched && is_few_tiles(variant)) panel = panel_instead_of_tiles(a, is_64_row_tiles(variant));
    if (panel.form)
        panel_name(panel, text, text_bytes);
    else
        snprintf(text, text_bytes, "%s", kVariants[variant].name);
}

// ------------------------------------------------------------------------------------
// Grouped GEMM: experts are sorted by their number of rows into the three kernel families
// (16-row stream kernel, 32- or 64-row panels, tiles); large experts on up to two kinds of 256-row tiles
// and what these leave over.  Each kernel that is needed gets one launch over all of its experts, or
// ranges of their rows; at most five in all.
// ------------------------------------------------------------------------------------
struct GroupedArgs {
    int E, N, K, group;
    const int *row_offsets;  // host, E + 1
    GroupedPtrs p;
    hipStream_t stream;
    char *text = nullptr;  // set: append the launches to it and launch nothing
    size_t text_bytes = 0;
};

template <class Kernel, class... A>
static int grouped_launch(const GroupedArgs &a, const char *name, Kernel kernel, dim3 grid, dim3 block, size_t lds,
                          const GroupTable &t, A... more)
{
    if (a.text) {
        int rows = 0;
        for (int i = 0; i < t.count; ++i) rows += t.rows[i];
        const size_t at = strlen(a.text);
        const char *as = strchr(name, '[');  // ("<kernel>[as <form>]")
        snprintf(a.text + at, a.text_bytes - at, "%s%.*s[%d experts, %d rows%s%s", at ? "+" : "",
                 (int)(as ? as - name : (ptrdiff_t)strlen(name)), name, t.count, rows, as ? ", " : "", as ? as + 1 : "]");
        return LQ_OK;
    }
    if (int rc = allow_lds(kernel, lds)) return rc;
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel, grid, block, lds, a.stream, t, a.p, a.N, a.K, more...);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LQ_ERR_HIP, "launch of %s failed: %s", name, hipGetErrorString(e));
    return LQ_OK;
}

// The experts of more than 32 rows (or row ranges of them) as 128- or 64-row tiles: one launch.
static int grouped_tiles_run(const GroupedArgs &a, GroupTable &big)
{
    const bool g128 = a.group == 128;
    const int blocks_n = (a.N + 255) / 256;
    long long big_blocks = 0, big_blocks64 = 0;
    for (int i = 0; i < big.count; ++i) {
        big_blocks += (long long)((big.rows[i] + 127) / 128) * blocks_n;
        big_blocks64 += (long long)((big.rows[i] + 63) / 64) * blocks_n;
        if (big_blocks > 0x7fffffff) return fail(LQ_ERR_INVALID, "grouped GEMM too large for one launch");
        big.block_end[i] = (int)big_blocks;
    }
    if (big_blocks64 <= 256 && big_blocks64 > big_blocks && a.K >= 512) {
        // few blocks and experts of more than 64 rows: a grid of 64-row tiles has up to twice the
        // blocks, still at most one per CU (8 experts of 72 rows on 4096 x 14336: 128 -> 256 blocks)
        long long end = 0;
        for (int i = 0; i < big.count; ++i) {
            end += (long long)((big.rows[i] + 63) / 64) * blocks_n;
            big.block_end[i] = (int)end;
        }
        const dim3 grid((unsigned)big_blocks64);
        const size_t lds2 = std::max<size_t>(4 * (size_t)128 * kTilePitch, 64 * 1024);
        return g128 ? grouped_launch(a, "duo_m64", w4a8_duo_grouped_kernel<true, 2, 64>, grid, dim3(512), lds2, big)
                    : grouped_launch(a, "duo_m64", w4a8_duo_grouped_kernel<false, 2, 64>, grid, dim3(512), lds2, big);
    }
    const dim3 grid((unsigned)big_blocks);
    // as for single GEMMs: two k groups per block while the grid gives at most one block per CU
    const bool kg2 = big_blocks <= 256 && a.K >= 512;
    const size_t lds1 = 2 * (size_t)128 * kTilePitch;
    const size_t lds2 = std::max<size_t>(2 * lds1, 64 * 1024);
    // more blocks than CUs: the direct-to-LDS form, as for single GEMMs (its X offsets have 32
    // bits) -- unless the experts are so small that most tiles have two row fragments, which
    // the other form runs with a deeper W pipeline (8 experts of 58..71 rows: 63 against 67 us;
    // of 128 rows: 91 against 79; of about 1000: 531 against 513)
    bool dl = !kg2 && a.K >= 512;
    long long big_rows = 0;
    for (int i = 0; i < big.count; ++i) {
        dl = dl && (long long)big.rows[i] * a.K < (1ll << 32);
        big_rows += big.rows[i];
    }
    dl = dl && big_rows > 96ll * big.count;
    if (dl)
        return g128 ? grouped_launch(a, "duo_dl_m128", w4a8_duo_dl_grouped_kernel<true>, grid, dim3(256), 4 * (size_t)128 * 128, big)
                    : grouped_launch(a, "duo_dl_m128", w4a8_duo_dl_grouped_kernel<false>, grid, dim3(256), 4 * (size_t)128 * 128, big);
    if (kg2)
        return g128 ? grouped_launch(a, "duo_m128_g2", w4a8_duo_grouped_kernel<true, 2>, grid, dim3(512), lds2, big)
                    : grouped_launch(a, "duo_m128_g2", w4a8_duo_grouped_kernel<false, 2>, grid, dim3(512), lds2, big);
    return g128 ? grouped_launch(a, "duo_m128", w4a8_duo_grouped_kernel<true, 1>, grid, dim3(256), lds1, big)
                : grouped_launch(a, "duo_m128", w4a8_duo_grouped_kernel<false, 1>, grid, dim3(256), lds1, big);
}

// Experts (or what they leave over) of up to 128 rows as panels: one launch for all of them.
// 32-row panels of 64 channels that are half a round of blocks or less run on 32 channels a block instead where K is long: a CU takes in
// weights at some 60 KB per us, however few others do (25000 calls of 1 to 16 experts, 8 to 128 blocks of 64 channels: 0.79 of the time with K above
// 8448, 0.83 from 4352 on and none slower but by noise; at K = 3072 0.95 and one call in five slower, at 2048 1.01; from 129 blocks on, where
// 32 channels make more than one round, 1.03 to 1.19).  27 rows on 4096 x 14336, what eight experts of some 750 leave over: 17.3 -> 13.3 us.
template <int F, int MF>
static int grouped_panel_run(const GroupedArgs &a, GroupTable &t)
{
    const int groups = (a.N / 32 + F - 1) / F;
    long long blocks = 0;
    for (int i = 0; i < t.count; ++i) {
        blocks += (long long)((t.rows[i] + 32 * MF - 1) / (32 * MF)) * groups;
        if (blocks > 0x7fffffff) return fail(LQ_ERR_INVALID, "grouped GEMM too large for one launch");
        t.block_end[i] = (int)blocks;
    }
    if constexpr (F == 2)
        if (a.K > 4096 && 2 * blocks <= kAssumedCUs) return grouped_panel_run<1, 1>(a, t);
    const size_t lds = panel_lds_bytes(F, 8, MF, a.K / 128);
    static_assert((F <= 2 && MF == 1) || (F == 4 && MF == 2), "the names below");
    const dim3 grid((unsigned)blocks);
    auto go = [&](auto kernel) {
        return grouped_launch(a, F == 1 ? "panel_f2_m32[as panel_f1_m32]" : MF == 1 ? "panel_f2_m32" : "panel_f4_m64", kernel, grid,
                              dim3(512), lds, t);
    };
    if (blocks == (long long)t.count * groups)  // one row tile each
        return a.group == 128 ? go(&w4a8_panel_grouped_kernel<F, MF, true, true>)
                              : go(&w4a8_panel_grouped_kernel<F, MF, false, true>);
    return a.group == 128 ? go(&w4a8_panel_grouped_kernel<F, MF, true, false>)
                          : go(&w4a8_panel_grouped_kernel<F, MF, false, false>);
}

// Up to 128 rows of each expert (experts of 33 to 128 rows, and what larger ones leave over): 32-row
// panels, 64-row panels of 128 channels or tiles, whichever a fitted cost (us) finds cheapest.  The panels' is fitted to 12000
// calls of 1 to 64 experts of up to 128 rows (N 128 to 16384, K 256 to 14336) with the present panel kernel, 6 % rms; the tiles' to
// 8 to 128 rows of 1 to 16 experts on five weight shapes (2816 x 2048 to 4096 x 14336), and is off by 19 % over those
// 12000, hence the 10 % that panels have to win by.  So picked, 4600 such calls are 0.9 % behind the best of the three and none
// is more than 3 % behind tiles alone (48 % ahead of them): a few experts are few tiles, and the tiles of a grouped launch have no
// K slices across blocks (us on tiles / as picked: one expert of 128 rows on 4096 x 14336 55.8 / 19.4, two of 64 on
// 14336 x 4096 20.0 / 19.7; eight of 64 there stay on tiles, 60 against 69).  32-row panels are priced as of 64 channels; where
// grouped_panel_run takes 32 a block they run in about 0.8 of that, so tiles are taken a little too often there.
static double grouped_panel_us(const GroupTable &t, int N, int K, int F, int MF)
{
    long long blocks = 0;
    for (int i = 0; i < t.count; ++i) blocks += panel_blocks(t.rows[i], N, F, MF);
    const double fill = (double)blocks / kAssumedCUs, k = K / 1024.0, mb = 0.5e-6 * N * K * t.count;
    return MF == 1 ? 2.91 + (0.6 * std::ceil(fill) + 0.4 * std::max(fill, 1.0)) * (1.25 + 0.715 * k) + 0.30 * std::min(fill, 1.0) * k + 0.088 * mb
                   : 1.42 + std::ceil(fill) * (4.72 + 1.666 * k) + 0.136 * mb;  // (one block on a CU)
}
// ... as 128- or 64-row tiles, also of experts of more rows (the last line: the rounds of a single GEMM, 6 % off
// on 264 to 3584 tiles with K from 2048 to 14336)
static double grouped_tiles_us(const GroupTable &t, int N, int K)
{
    long long tiles[2] = {0, 0}, b64 = 0;  // 128-row tiles with up to 64 and with more rows; 64-row tiles
    const int bn = (N + 255) / 256;
    bool few_rows = true;
    for (int i = 0; i < t.count; ++i) {
        const int last = t.rows[i] % 128;
        tiles[1] += (long long)(t.rows[i] / 128 + (last > 64)) * bn;
        tiles[0] += last > 0 && last <= 64 ? bn : 0;
        b64 += (long long)((t.rows[i] + 63) / 64) * bn;
        few_rows = few_rows && t.rows[i] <= 128;
    }
    if (b64 <= kAssumedCUs) tiles[0] = b64, tiles[1] = 0;
    const long long all = tiles[0] + tiles[1];
    const double k = K / 1024.0, mb = 0.5e-6 * N * K * t.count;
    if (all <= kAssumedCUs || few_rows)
        return 8.24 + k * (all <= kAssumedCUs ? 2.365 : 5.378) + k * (2.033 * tiles[0] + 4.451 * tiles[1]) / kAssumedCUs + 0.061 * mb;
    return 9 + 0.95 * 64.0 * K / 8192 * tiled_costs(all, 0, 0, K, true).duo;
}
static double grouped_few_rows_us(const GroupTable &t, int N, int K)
{
    return t.count == 0 ? 0.0 : std::min({grouped_panel_us(t, N, K, 2, 1), grouped_panel_us(t, N, K, 4, 2), grouped_tiles_us(t, N, K)});
}
// (t: every entry at most 128 rows; mid: entries of at most 32 rows, which run as 32-row panels, in the
// same launch where t does too; either may be empty)
static int grouped_few_rows_run(const GroupedArgs &a, GroupTable &t, GroupTable &mid)
{
    int most = 0;
    for (int i = 0; i < t.count; ++i) most = std::max(most, t.rows[i]);
    const double p32 = grouped_panel_us(t, a.N, a.K, 2, 1), p64 = grouped_panel_us(t, a.N, a.K, 4, 2);
    const double tiles = 0.90 * grouped_tiles_us(t, a.N, a.K);  // (panels have to win by 10 %: the tiles' estimate is off by up to that and more)
    const bool as_p32 = most <= 32 || (p32 <= p64 && p32 <= tiles);
    for (int i = 0; as_p32 && i < t.count; ++i) {
        const int k = mid.count++;
        mid.expert[k] = t.expert[i], mid.row_off[k] = t.row_off[i], mid.rows[k] = t.rows[i];
    }
    if (mid.count)
        if (int rc = grouped_panel_run<2, 1>(a, mid)) return rc;
    if (as_p32) return LQ_OK;
    return p64 <= tiles ? grouped_panel_run<4, 2>(a, t) : grouped_tiles_run(a, t);
}

// 256 x 256 / KG tiles of the one-wave-per-SIMD kernel, all entries of the table in one launch
template <int KG>
static int grouped_solo_run(const GroupedArgs &a, const GroupTable &t)
{
    const dim3 grid((unsigned)std::min(t.block_end[t.count - 1], std::max(cu_count(), 1)));
    const size_t lds = 4 * (size_t)256 * 128 + 4 * 1024;
    const char *name = KG == 1 ? "solo16_pt_m256" : "solo16_g2_m256";
    return a.group == 128 ? grouped_launch(a, name, w4a8_solo_grouped_kernel<true, KG>, grid, dim3(256), lds, t)
                          : grouped_launch(a, name, w4a8_solo_grouped_kernel<false, KG>, grid, dim3(256), lds, t);
}
// The larger experts' row blocks of 256: time (us) of 256 x 256 and of 256 x 128 tiles, from 65
// calls on five weight shapes (2816 x 2048 to 4096 x 14336; 4 to 64 row blocks).  A round that leaves CUs
// idle takes 62 % of a full one plus its part of the rest (the others clock higher): 1.06 rounds of 256 x 256
// tiles with K = 14336 took 275 us, 1.5 rounds 287, two 323.  Hence the rows that fill whole rounds go to
// 256 x 256 tiles, a last round of up to about half to 256 x 128 tiles: 24 row blocks on 4096 x 14336
// 274 us (287 on 256 x 256 tiles alone, 281 on 256 x 128, 347 on 128-row tiles), 20 on 14336 x 4096 226 / 237 / 263
// / 259, 16 of 256 rows on 8192 x 5120 128 on 256 x 256 tiles / 152 / 143, eight of 129..256 on 4096 x 14336 92 on
// 256 x 128 / 124 / 110.
static double rounds_us(long long tiles, double round)
{
    const double part = (double)(tiles % kAssumedCUs) / kAssumedCUs;
    return round * ((double)(tiles / kAssumedCUs) + (part > 0 ? 0.62 + 0.30 * part : 0.0));
}
static double grouped_solo_us(long long t256, int K) { return t256 ? 6 + rounds_us(t256, 6 + 11.1 * K / 1024) : 0.0; }
static double grouped_g2_us(long long t2, int K) { return t2 ? 3 + rounds_us(t2, 9 + 5.8 * K / 1024) : 0.0; }
static int grouped_run(const GroupedArgs &a)
{
    // Up to 32 rows: as one launch of 32-row panels if any expert has more than 16 rows or K is long (8
    // experts of 10..24 rows: 45.8 against 52.9 us in two launches on 14336 x 4096, 64 experts of 7..25 rows
    // on 1408 x 2048 25.2 / 29.5; 16 of 3..15 rows on 3072 x 8192 36.2 / 37.9) -- unless the experts of up to
    // 16 rows alone are more than nine rounds of blocks with short K: a panel costs more than a 16-row block
    // there, and nothing is idle in either launch (64 experts on 4096 x 1536, 60 of them up to 16 rows: 54.5
    // us in one launch, 44.9 in two; 36 of them: 54.5 / 52.8; on 2816 x 2048 52 of them, 8.9 rounds: 43.2 / 45.6).
    // 33..64 rows, if no expert has more: 64-row panels of 128 channels for all experts where these
    // are one round of blocks (8 experts of 36..55 rows on 4096 x 14336: 44.9 / 59.0 us, 17..35 rows:
    // 42.4 / 93.3; with 3.5 rounds on 14336 x 4096 64.5 / 50.9), else 32-row panels for all where at
    // least half of them have no more than 32 rows and the second row tiles of the others are less than two
    // rounds of blocks (0.9 rounds, 16 experts of 24..36 rows on 3072 x 8192: 52.5 / 67.0 us; 1.9, 64 experts of
    // 17..40 on 2048 x 1536: 36.3 / 39.3; 2.0, 32 of 16..39 on 4096 x 2560: 50.2 / 47.7; 5.2, 64 of 20..47 on
    // 2816 x 2048: 59.9 / 52.5).
    int used = 0, upto16 = 0, upto32 = 0, most = 0, most32 = 0;
    for (int e = 0; e < a.E; ++e) {
        const int rows = a.row_offsets[e + 1] - a.row_offsets[e];
        if (rows == 0) continue;
        ++used;
        most = std::max(most, rows);
        if (rows <= 16) ++upto16;
        if (rows <= 32) ++upto32, most32 = std::max(most32, rows);
    }
    const long long panel_groups = a.N / 64;  // blocks of a 32-row panel's row tile
    const bool up_to_64 = most > 32 && most <= 64;
    const bool panel64 = up_to_64 && (long long)used * ((a.N / 32 + 3) / 4) <= kAssumedCUs;
    const bool panels_for_all = panel64 || (up_to_64 && 2 * upto32 >= used && (used - upto32) * panel_groups < 2 * kAssumedCUs);
    const int panel_max = panels_for_all ? 64 : 32;
    const bool split16 = !panels_for_all && a.K < 4096 && upto16 * panel_groups > 9 * kAssumedCUs;
    // panels also for the experts of up to 16 rows: as above, or where they are so few blocks that they run on 32 channels
    // (grouped_panel_run; 7254 calls of 1 to 8 experts with K from 4352 to 7936 0.77 of the time: 16 experts of 12 rows on 512 x 5120 11.3 / 8.8 us)
    const bool panels16 = panels_for_all || most32 > 16 || a.K >= 8192 || (a.K > 4096 && 2 * upto16 * panel_groups <= kAssumedCUs);
    const int stream16_max = panels16 && !split16 ? 0 : 16;
    GroupTable small{}, mid{}, big{};
    for (int e = 0; e < a.E; ++e) {
        const int r0 = a.row_offsets[e], rows = a.row_offsets[e + 1] - r0;
        if (rows == 0) continue;
        GroupTable &t = rows > panel_max ? big : rows > stream16_max ? mid : small;
        const int i = t.count++;
        t.expert[i] = e, t.row_off[i] = r0, t.rows[i] = rows;
    }
    const bool g128 = a.group == 128;
    const int groups = a.N / 64;  // stream kernels: two tiles of 32 channels per block
    if (small.count) {
        const dim3 grid((unsigned)(small.count * groups));
        // four waves per block once the grid alone gives every CU several blocks
        const bool w4 = (long long)small.count * groups >= 384 * 2;
        const size_t lds = (size_t)(w4 ? 4 : 8) * 2 * 8 * 64 * sizeof(int);
        int rc;
        if (w4)
            rc = g128 ? grouped_launch(a, "stream16_f2_w4", w4a8_stream16_grouped_kernel<4, 1, true>, grid, dim3(256), lds, small, groups)
                      : grouped_launch(a, "stream16_f2_w4", w4a8_stream16_grouped_kernel<4, 1, false>, grid, dim3(256), lds, small, groups);
        else
            rc = g128 ? grouped_launch(a, "stream16_f2_w8", w4a8_stream16_grouped_kernel<8, 1, true>, grid, dim3(512), lds, small, groups)
                      : grouped_launch(a, "stream16_f2_w8", w4a8_stream16_grouped_kernel<8, 1, false>, grid, dim3(512), lds, small, groups);
        if (rc) return rc;
    }
    if (mid.count && (panel64 || !big.count)) {
        const int rc = panel64 ? grouped_panel_run<4, 2>(a, mid) : grouped_panel_run<2, 1>(a, mid);
        if (rc) return rc;
    }
    if (!big.count) return LQ_OK;
    // The larger experts: whole 256-row blocks of them (and a last block of more than 128 rows) on the
    // one-wave-per-SIMD tiles where these pay, what is left of each expert (at most 128 rows) as panels
    // or tiles in a launch of its own; everything on 128- or 64-row tiles otherwise.
    const int blocks_n = (a.N + 255) / 256, blocks_n2 = (a.N + 127) / 128;
    GroupTable rest{};
    long long row_blocks = 0, main_t128 = 0;
    bool fits = a.N <= (1 << 26);
    for (int i = 0; i < big.count; ++i) {
        const int rows = big.rows[i], tail = rows % 256;
        const int rows_rest = tail > 0 && tail <= 128 ? tail : 0, rows_main = rows - rows_rest;
        fits = fits && (long long)rows * a.K < (1ll << 32);
        row_blocks += (rows_main + 255) / 256;
        main_t128 += (long long)((rows_main + 127) / 128) * blocks_n;
        if (row_blocks * blocks_n > 0x7fffffff) return fail(LQ_ERR_INVALID, "grouped GEMM too large for one launch");
        if (rows_rest) {
            const int k = rest.count++;
            rest.expert[k] = big.expert[i], rest.row_off[k] = big.row_off[i] + rows_main, rest.rows[k] = rows_rest;
        }
    }
    if (row_blocks == 0) return grouped_few_rows_run(a, rest, mid);
    // What the rule of single GEMMs picks -- 256 x 256 tiles for all row blocks (first = row_blocks) or 128-row tiles for
    // everything (first = -1) -- or, where it is estimated to be enough faster, another split: `first` row blocks on
    // 256 x 256 tiles and the others on 256 x 128.  Enough is what a replay of the rule over 16000 timed calls (1 to 64 experts, N 128
    // to 16384, K 256 to 14336) showed it to be: the 128-row tiles' estimate is 45 % too low at K = 512 and 20 % at 1024 against the
    // 256-row tiles' (two experts of 3650 rows on 15936 x 512: 90 us on 256 x 256 tiles, 121 on 128-row ones), except where K % 512
    // == 256 adds two stages to the latter; two kinds of 256-row tiles in turn, one of them in part of a round, were equal to 128-row tiles on average
    // (94 calls) and need 18 %.  1540 calls leave the single GEMMs' rule, at 0.865 of its time; 7 of them lose more than 10 %.
    const double rest_us = grouped_few_rows_us(rest, a.N, a.K), tiles_us = grouped_tiles_us(big, a.N, a.K);
    const bool solo_by_rule = fits && solo_form_for(main_t128, row_blocks * blocks_n, 0, a.K) == 1;
    long long first = solo_by_rule ? row_blocks : -1;
    const double rule_us = solo_by_rule ? grouped_solo_us(row_blocks * blocks_n, a.K) + rest_us : tiles_us;
    double best_us = 1e30;
    auto consider = [&](long long rb, double us, double margin) {
        if (us < margin * rule_us && us < best_us) best_us = us, first = rb;
    };
    if (solo_by_rule) consider(-1, tiles_us, a.K % 512 == 0 ? std::min(0.95, 0.50 + 0.22 * a.K / 1024) : 0.95);
    const long long rounds = row_blocks * blocks_n / kAssumedCUs;
    for (const long long rb : {0ll, (rounds - 1) * kAssumedCUs / blocks_n, rounds * kAssumedCUs / blocks_n, row_blocks}) {
        if (!fits || rb < 0 || (row_blocks - rb) * blocks_n2 > 0x7fffffff) continue;
        const bool two_kinds = rb > 0 && rb < row_blocks;
        consider(rb, grouped_solo_us(rb * blocks_n, a.K) + grouped_g2_us((row_blocks - rb) * blocks_n2, a.K) + rest_us,
                 solo_by_rule ? 0.95 : two_kinds ? 0.82 : rb == row_blocks ? 0.90 : 0.95);
    }
    if (first < 0) {
        if (mid.count)
            if (int rc = grouped_panel_run<2, 1>(a, mid)) return rc;
        return grouped_tiles_run(a, big);
    }
    GroupTable solo{}, g2{};
    long long left = first;
    int solo_tiles = 0, g2_tiles = 0;
    for (int i = 0; i < big.count; ++i) {
        const int tail = big.rows[i] % 256, rows_main = big.rows[i] - (tail <= 128 ? tail : 0);
        const int rb = (rows_main + 255) / 256, rb1 = (int)std::min<long long>(rb, left), rows1 = std::min(rows_main, 256 * rb1);
        left -= rb1;
        if (rows1) {
            const int k = solo.count++;
            solo.expert[k] = big.expert[i], solo.row_off[k] = big.row_off[i], solo.rows[k] = rows1;
            solo.block_end[k] = solo_tiles += rb1 * blocks_n;
        }
        if (rows1 < rows_main) {
            const int k = g2.count++;
            g2.expert[k] = big.expert[i], g2.row_off[k] = big.row_off[i] + rows1, g2.rows[k] = rows_main - rows1;
            g2.block_end[k] = g2_tiles += (rb - rb1) * blocks_n2;
        }
    }
    if (solo.count)
        if (int rc = grouped_solo_run<1>(a, solo)) return rc;
    if (g2.count)
        if (int rc = grouped_solo_run<2>(a, g2)) return rc;
    return rest.count || mid.count ? grouped_few_rows_run(a, rest, mid) : LQ_OK;
}

static int check_grouped_shape(int E, const int *row_offsets, int N, int K, int group)
{
    if (E < 1 || E > kMaxExperts) return fail(LQ_ERR_INVALID, "E=%d out of range (1..%d)", E, kMaxExperts);
    if (!shape_ok(N, K, group))
        return fail(LQ_ERR_INVALID, "bad shape N=%d K=%d group=%d (need N%%64==0, K%%256==0, group 64|128, K<=131072)",
                    N, K, group);
    if (!row_offsets || row_offsets[0] != 0) return fail(LQ_ERR_INVALID, "row_offsets must start at 0");
    for (int e = 0; e < E; ++e) {
        if (row_offsets[e + 1] < row_offsets[e]) return fail(LQ_ERR_INVALID, "row_offsets must not decrease");
        // the kernels address an expert's rows of X with 32-bit byte offsets
        if ((long long)(row_offsets[e + 1] - row_offsets[e]) * K >= (1ll << 32))
            return fail(LQ_ERR_INVALID, "expert %d has rows * K >= 2^32 bytes of X; split it into two experts", e);
    }
    return LQ_OK;
}

// ------------------------------------------------------------------------------------
// Built-in split-K workspace for callers that cannot allocate (w4a8_gemm_static): tickets
// followed by partial tiles, laid out exactly like a caller's workspace.  Zero when the code
// object is loaded; the kernels leave the tickets zero after every call.  The array's name
// is only a host-side handle: its address on the current device comes from the runtime.
// ------------------------------------------------------------------------------------
constexpr size_t kStaticScratchBytes = kTicketBytes + ((size_t)32 << 20);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;

static int static_scratch_ptr(void **out)
{
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(LQ_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(LQ_ERR_INVALID, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(LQ_ERR_HIP, "hipGetSymbolAddress(built-in workspace): %s", hipGetErrorString(e));
        addr[dev] = p;
    }
    *out = addr[dev];
    return LQ_OK;
}

}  // namespace lqq

using namespace lqq;

extern "C" {

size_t w4a8_gemm_workspace_size(int M, int N, int K, int group)
{
    if (M <= 0 || !shape_ok(N, K, group)) return 0;
    // Enough for the dispatcher, for any variant that can run a shape of fewer than 192 tiles of
    // 128 x 256 (tiled kernels and panels split K only there, into at most 8 slices) and for the variants of
    // up to 64 rows (panels of at most 4 slices; the 16-row kernels take up to 16 and exchange 8 values per
    // lane and tile).
    const int tiles = ((M + 127) / 128) * ((N + 255) / 256);
    size_t need = tiles >= 192 ? 0 : std::max(duo_ws_bytes(M, N, 8), duo_ws_bytes(M, N, 8, 64));
    if (M <= 64) need = std::max(need, panel_ws_bytes(N / 32 + 3, 1, 2, 4));
    if (M <= 16) need = std::max(need, kTicketBytes + (size_t)16 * (N / 32) * 8 * 64 * sizeof(int32_t));
    if (K % 512 == 0) {
        // the 256-row tiles with K slices: a whole INT32 matrix per slice, at most one round of blocks
        // (up to 256 rows also the variants with a named number of slices)
        const long long t256 = (long long)((M + 255) / 256) * ((N + 255) / 256);
        const int s = M <= 256 ? 4 : (int)std::min<long long>(4, kAssumedCUs / t256);
        need = std::max(need, solo_ws_bytes(M, N, s));
    }
    return need;
}

int w4a8_workspace_init(void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!workspace || workspace_bytes == 0) return LQ_OK;
    if ((uintptr_t)workspace & 15) return fail(LQ_ERR_ALIGN, "device pointers must be 16-byte aligned");
    const int n = (int)(std::min(workspace_bytes, kTicketBytes) / sizeof(unsigned int));
    if (n == 0) return LQ_OK;
    (void)hipGetLastError();
    hipLaunchKernelGGL(workspace_init_kernel, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<unsigned int *>(workspace), n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LQ_ERR_HIP, "workspace init launch failed: %s", hipGetErrorString(e));
    return LQ_OK;
}

int w4a8_gemm(int M, int N, int K, int group, const int8_t *X, const float *act_scales,
              const void *W_packed, const uint8_t *gparams, const float *w_scales, uint16_t *Y,
              void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!Y && M != 0) return fail(LQ_ERR_INVALID, "null Y");
    const Args a{M, N, K, group, X, act_scales, static_cast<const u32x4 *>(W_packed), gparams, w_scales,
                 reinterpret_cast<__half *>(Y), nullptr, static_cast<hipStream_t>(hip_stream), workspace, workspace_bytes};
    return run(-1, a);
}

int w4a8_gemm_static(int M, int N, int K, int group, const int8_t *X, const float *act_scales,
                     const void *W_packed, const uint8_t *gparams, const float *w_scales, uint16_t *Y,
                     void *hip_stream)
{
    if (!Y && M != 0) return fail(LQ_ERR_INVALID, "null Y");
    Args a{M, N, K, group, X, act_scales, static_cast<const u32x4 *>(W_packed), gparams, w_scales,
           reinterpret_cast<__half *>(Y), nullptr, static_cast<hipStream_t>(hip_stream), nullptr, 0};
    // what the dispatcher's kernel for this shape would use of a workspace (nothing is launched;
    // a launcher that can make do with fewer K slices is told how much there is)
    size_t need = 0;
    a.query = &need;
    a.ws_bytes = kStaticScratchBytes;
    if (int rc = run(-1, a)) return rc;
    a.query = nullptr;
    a.ws_bytes = 0;
    if (M == 0) return LQ_OK;
    if (need > kStaticScratchBytes)
        return fail(LQ_ERR_WORKSPACE,
                    "M=%d N=%d K=%d needs %zu bytes of split-K workspace, the built-in one holds %zu: "
                    "use w4a8_gemm with a workspace of the caller",
                    M, N, K, need, kStaticScratchBytes);
    if (need > 0) {
        if (int rc = static_scratch_ptr(&a.ws)) return rc;
        a.ws_bytes = kStaticScratchBytes;
    }
    return run(-1, a);
}

int w4a8_gemm_i32(int M, int N, int K, int group, const int8_t *X, const void *W_packed,
                  const uint8_t *gparams, int32_t *ACC, void *workspace, size_t workspace_bytes,
                  void *hip_stream)
{
    if (!ACC && M != 0) return fail(LQ_ERR_INVALID, "null ACC");
    const Args a{M, N, K, group, X, nullptr, static_cast<const u32x4 *>(W_packed), gparams, nullptr,
                 nullptr, ACC, static_cast<hipStream_t>(hip_stream), workspace, workspace_bytes};
    return run(-1, a);
}

int w4a8_gemm_variant(int variant, int M, int N, int K, int group, const int8_t *X,
                      const float *act_scales, const void *W_packed, const uint8_t *gparams,
                      const float *w_scales, uint16_t *Y, int32_t *ACC, void *workspace,
                      size_t workspace_bytes, void *hip_stream)
{
    if (variant < -1 || variant >= kNumVariants) return fail(LQ_ERR_INVALID, "unknown variant %d", variant);
    const Args a{M, N, K, group, X, act_scales, static_cast<const u32x4 *>(W_packed), gparams, w_scales,
                 reinterpret_cast<__half *>(Y), ACC, static_cast<hipStream_t>(hip_stream), workspace, workspace_bytes};
    return run(variant, a);
}

int w4a8_variant_count(void) { return kNumVariants; }

const char *w4a8_variant_name(int variant)
{
    return (variant >= 0 && variant < kNumVariants) ? kVariants[variant].name : nullptr;
}

int w4a8_variant_supports(int variant, int M, int N, int K, int group)
{
    if (variant < 0 || variant >= kNumVariants || M < 0 || !shape_ok(N, K, group)) return 0;
    return variant_supports(variant, M, N, K) ? 1 : 0;
}

int w4a8_select_variant(int M, int N, int K, int group)
{
    if (M < 0 || !shape_ok(N, K, group)) return fail(LQ_ERR_INVALID, "bad shape");
    return select_variant(M, N, K);
}

int w4a8_select_plan(int M, int N, int K, int group, int *rows_first, int *variant_rest)
{
    if (M < 0 || !shape_ok(N, K, group) || !rows_first || !variant_rest) return fail(LQ_ERR_INVALID, "bad shape");
    const int first = M > 0 ? rows_of_first_launch(M, N, K) : M;
    *rows_first = first;
    *variant_rest = first == M ? -1 : select_variant(M - first, N, K);
    return first == M ? select_variant(M, N, K) : find_variant("solo16_pt_m256");
}

int w4a8_describe_launch(int variant, int M, int N, int K, int group, char *text, size_t text_bytes,
                         size_t *workspace_bytes)
{
    if (variant < -1 || variant >= kNumVariants) return fail(LQ_ERR_INVALID, "unknown variant %d", variant);
    if (M < 0 || !shape_ok(N, K, group)) return fail(LQ_ERR_INVALID, "bad shape");
    if (variant >= 0 && !variant_supports(variant, M, N, K))
        return fail(LQ_ERR_INVALID, "variant %s cannot run M=%d N=%d K=%d", kVariants[variant].name, M, N, K);
    size_t need[2] = {0, 0};
    char words[160] = "";
    if (M > 0) {
        const int first = variant < 0 ? rows_of_first_launch(M, N, K) : M;
        char name[64];
        Args a{};
        a.M = first, a.N = N, a.K = K, a.group = group, a.query = &need[0];
        if (int rc = run_rows(first == M ? variant : find_variant("solo16_pt_m256"), a)) return rc;
        launch_name(first == M ? variant : -1, M - (first == M ? 0 : first), N, K, name, sizeof(name));
        if (first == M) {
            snprintf(words, sizeof(words), "%s", name);
        } else {
            a.M = M - first, a.query = &need[1];
            if (int rc = run_rows(-1, a)) return rc;
            snprintf(words, sizeof(words), "solo16_pt_m256[%d rows]+%s[%d rows]", first, name, M - first);
        }
    }
    if (workspace_bytes) *workspace_bytes = std::max(need[0], need[1]);
    if (text && text_bytes) snprintf(text, text_bytes, "%s", words);
    return LQ_OK;
}

int w4a8_dequant_dump(const void *W_packed, const uint8_t *gparams, int N, int K, int group,
                      int8_t *Wd, void *hip_stream)
{
    if (!shape_ok(N, K, group)) return fail(LQ_ERR_INVALID, "bad shape N=%d K=%d group=%d", N, K, group);
    if (!W_packed || !gparams || !Wd) return fail(LQ_ERR_INVALID, "null pointer");
    if (((uintptr_t)W_packed | (uintptr_t)gparams | (uintptr_t)Wd) & 15)
        return fail(LQ_ERR_ALIGN, "device pointers must be 16-byte aligned");
    const dim3 grid((unsigned)((K / 64 + 3) / 4), (unsigned)(N / 32)), block(256);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    (void)hipGetLastError();
    if (group == 128)
        hipLaunchKernelGGL(dequant_dump_kernel<true>, grid, block, 0, st,
                           static_cast<const u32x4 *>(W_packed), gparams, N, K, Wd);
    else
        hipLaunchKernelGGL(dequant_dump_kernel<false>, grid, block, 0, st,
                           static_cast<const u32x4 *>(W_packed), gparams, N, K, Wd);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LQ_ERR_HIP, "dequant_dump launch failed: %s", hipGetErrorString(e));
    return LQ_OK;
}

int w4a8_grouped_gemm(int E, const int *row_offsets, int N, int K, int group, const int8_t *X,
                      const float *act_scales, const void *W_packed, const uint8_t *gparams,
                      const float *w_scales, uint16_t *Y, int32_t *ACC, void *hip_stream)
{
    if (int rc = check_grouped_shape(E, row_offsets, N, K, group)) return rc;
    if (row_offsets[E] == 0) return LQ_OK;
    if (!Y && !ACC) return fail(LQ_ERR_INVALID, "no output pointer");
    if (!X || !W_packed || !gparams) return fail(LQ_ERR_INVALID, "null input pointer");
    if (Y && (!act_scales || !w_scales)) return fail(LQ_ERR_INVALID, "null scale pointer");
    const uintptr_t bits = (uintptr_t)X | (uintptr_t)W_packed | (uintptr_t)gparams | (uintptr_t)act_scales |
                           (uintptr_t)w_scales | (uintptr_t)Y | (uintptr_t)ACC;
    if (bits & 15) return fail(LQ_ERR_ALIGN, "device pointers must be 16-byte aligned");
    GroupedArgs a{};
    a.E = E, a.N = N, a.K = K, a.group = group, a.row_offsets = row_offsets;
    a.p = GroupedPtrs{X, act_scales, static_cast<const u32x4 *>(W_packed), gparams, w_scales,
                      reinterpret_cast<__half *>(Y), ACC, (size_t)N * K / 32, (size_t)2 * N * K / group};
    a.stream = static_cast<hipStream_t>(hip_stream);
    return grouped_run(a);
}

int w4a8_describe_grouped(int E, const int *row_offsets, int N, int K, int group, char *text, size_t text_bytes)
{
    if (int rc = check_grouped_shape(E, row_offsets, N, K, group)) return rc;
    char words[320] = "";
    GroupedArgs a{};
    a.E = E, a.N = N, a.K = K, a.group = group, a.row_offsets = row_offsets;
    a.text = words, a.text_bytes = sizeof(words);
    if (row_offsets[E] > 0)
        if (int rc = grouped_run(a)) return rc;
    if (text && text_bytes) snprintf(text, text_bytes, "%s", words);
    return LQ_OK;
}

int w8a8_gemm(int M, int N, int K, const int8_t *X, const float *act_scales, const void *W8_packed,
              const float *w_scales, uint16_t *Y, int32_t *ACC, void *hip_stream)
{
    if (M < 0 || !shape_ok(N, K, 64))
        return fail(LQ_ERR_INVALID, "bad shape M=%d N=%d K=%d (need M>=0, N%%64==0, K%%256==0, K<=131072)", M, N, K);
    if (M == 0) return LQ_OK;
    if (!Y && !ACC) return fail(LQ_ERR_INVALID, "no output pointer");
    if (!X || !W8_packed) return fail(LQ_ERR_INVALID, "null input pointer");
    if (Y && (!act_scales || !w_scales)) return fail(LQ_ERR_INVALID, "null scale pointer");
    if (((uintptr_t)X | (uintptr_t)W8_packed | (uintptr_t)act_scales | (uintptr_t)w_scales | (uintptr_t)Y |
         (uintptr_t)ACC) & 15)
        return fail(LQ_ERR_ALIGN, "device pointers must be 16-byte aligned");
    if ((long long)M * K >= (1ll << 32))
        return fail(LQ_ERR_INVALID, "M * K = %lld is beyond the 2^32 - 1 bytes of X one call addresses; split the batch",
                    (long long)M * K);
    const int blocks_n = (N + 255) / 256, blocks_m = (M + 127) / 128;
    const size_t lds_bytes = 4 * (size_t)128 * 128;
    if (int rc = allow_lds(w8a8_kernel, lds_bytes)) return rc;
    (void)hipGetLastError();
    hipLaunchKernelGGL(w8a8_kernel, dim3((unsigned)(blocks_n * blocks_m)), dim3(256), lds_bytes,
                       static_cast<hipStream_t>(hip_stream), M, N, K, X, act_scales,
                       static_cast<const u32x4 *>(W8_packed), w_scales, reinterpret_cast<__half *>(Y), ACC,
                       blocks_m, blocks_n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LQ_ERR_HIP, "w8a8 launch failed: %s", hipGetErrorString(e));
    return LQ_OK;
}

}  // extern "C"
