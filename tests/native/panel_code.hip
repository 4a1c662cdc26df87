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
        int, int, int, const int8_t *, const float *, const u32x4 *, const uint8_t *, const float *, __half *, int32_t *, \
        int32_t *, unsigned int *, int, int, int);
PANEL(true)
PANEL(false)
}  // namespace lqq
