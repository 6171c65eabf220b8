// Matrix-core x pass, complex128 (xpass.hpp).
#include "xpass.hpp"

namespace vie {

bool p3_mx_fits(int es, int n) {
    switch (n) {
#define CASE(n_) \
    case n_: return (es == 8 ? p3_mx_lds<float, n_>() : p3_mx_lds<double, n_>()) <= 160 * 1024;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

template <>
bool launch_p3_mx<double>(C<double>* A, const C<double>* U, const P3Params& p, const C<double>* tw, hipStream_t s) {
    if (2 * p.Nx > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                                                          \
    case n_:                                                                              \
        if constexpr (p3_mx_lds<double, n_>() <= 160 * 1024 && !p3_mx_left_out(16, n_)) { \
            launch_p3_mx_n<double, n_, X_N>(A, U, nullptr, p, tw, {}, {}, s);             \
            return true;                                                                  \
        }                                                                                 \
        return false;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

}  // namespace vie
