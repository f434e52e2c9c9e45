// Stands in for the kernel's row code: one row of y = H x, hop by hop.
#pragma once
#include <cstdint>

namespace pd {
namespace sigma_detail {
template <typename T>
int x_resource(const T *, int64_t) { return 0; }

template <typename R, typename T, int NN, bool COMP, bool BUF, int MAP, bool ALL>
T sigma_row(int64_t row, int64_t, int omega, int ks, const R *Ct, const T *Vs, const T *ds, T, const T *x, R *, int,
            int) {
    R rem = (R)row;
    uint64_t s = 0;
    T diag = 0;
    for (int p = omega - 1, k = NN; p >= 0; --p)
        if (k > 0 && Ct[p * ks + k] <= rem) {
            rem -= Ct[p * ks + k--];
            s |= 1ull << p;
            diag += ds[p];
        }
    T y = diag * x[row];
    for (int o = 0; o < omega; ++o)
        for (int e = 0; e < omega; ++e) {
            if (!((s >> o) & 1) || ((s >> e) & 1)) continue;
            const uint64_t t = (s ^ (1ull << o)) | (1ull << e);
            R r = 0;
            for (int p = 0, k = 0; p < omega; ++p)
                if ((t >> p) & 1) r += Ct[p * ks + ++k];
            y += Vs[o * omega + e] * x[r];
        }
    return y;
}
}  // namespace sigma_detail
}  // namespace pd
