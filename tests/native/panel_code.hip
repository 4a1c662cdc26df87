// The panel kernel of 32 rows x 32 channels alone, for both group sizes, to look at the code that is made of it.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lqq_common.h"
#include "lqq_device.h"

namespace lqq {
__device__ __forceinline__ __half scale_to_half(int acc, float sx, float sw) { return __float2half_rn((float)acc * sx * sw); }
#include "kernels_common.h"
#include "kernels_panel.h"

#define PANEL(G128)                                                                                                      \
    template __global__ void w4a8_panel_kernel<1, 8, 1, G128, true>(                                                      \
        int, int, int, int, const int8_t *, const float *, const u32x4 *, const uint8_t *, const float *, __half *,       \
        int32_t *, int32_t *, unsigned int *);
PANEL(true)
PANEL(false)

// 32 x 32, one unit a wave: at 67 registers three blocks fit a CU, and its LDS has to let them
static_assert(3 * panel_lds_bytes(1, 8, 1, 8) <= 160 * 1024);
// every form fits, with one unit a wave and with more
template <int F, int NW, int MF>
constexpr bool fits = panel_lds_bytes(F, NW, MF, 1) <= 160 * 1024 && panel_lds_bytes(F, NW, MF, 1024) <= 160 * 1024 &&
                      panel_lds_bytes(F, NW, MF, 1) >= (size_t)NW * (F % 2 == 0 ? 2 : 1) * MF * 4096;
static_assert(fits<1, 8, 1> && fits<2, 8, 1> && fits<4, 8, 1> && fits<1, 8, 2> && fits<2, 8, 2> && fits<3, 8, 2> &&
              fits<4, 8, 2> && fits<3, 4, 4> && fits<4, 4, 4> && fits<3, 8, 1> && fits<2, 4, 4>);
}  // namespace lqq
