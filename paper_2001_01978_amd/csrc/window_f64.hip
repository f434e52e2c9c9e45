// FP64 instantiation of the windowed product (window_impl.h).
#include "window_impl.h"

namespace pd {
hipError_t window_product_f64(const WinPlan &plan, int omega, int n, const double *d, const double *V,
                              const double *x, double *y, hipStream_t s) {
    return win::launch_product<double>(plan, omega, n, d, V, x, y, s);
}
}  // namespace pd
