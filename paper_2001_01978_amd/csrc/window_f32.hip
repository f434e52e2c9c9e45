// FP32 instantiation of the windowed product (window_impl.h).
#include "window_impl.h"

namespace pd {
hipError_t window_product_f32(const WinPlan &plan, int omega, int n, const float *d, const float *V,
                              const float *x, float *y, hipStream_t s) {
    return win::launch_product<float>(plan, omega, n, d, V, x, y, s);
}
}  // namespace pd
