// Matrix-core x pass of the curl operator, complex128 (xpass.hpp).  In complex64
// the raw curl product is needed only where the J-M sums have no kernel of
// their own, at lengths that this one does not take either.
#include "xpass.hpp"

namespace vie {

bool launch_p3_mx_curl(double2* A, const double2* U, const P3Params& p, const double2* tw, hipStream_t s) {
    if (2 * p.Nx > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                                                          \
    case n_:                                                                              \
        if constexpr (n_ <= 256) {                                                        \
            launch_p3_mx_n<double, n_, X_K>(A, U, nullptr, p, tw, {}, {}, s);             \
            return true;                                                                  \
        }                                                                                 \
        return false;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

}  // namespace vie
