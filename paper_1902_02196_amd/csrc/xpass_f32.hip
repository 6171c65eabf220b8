// Matrix-core x pass, complex64 (xpass.hpp).
#include "xpass.hpp"

namespace vie {

template <>
bool launch_p3_mx<float>(C<float>* A, const C<float>* U, const P3Params& p, const C<float>* tw, hipStream_t s) {
    if (!p3_mx_fits(8, p.plan.n) || 2 * p.Nx > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                          \
    case n_:                                             \
        launch_p3_mx_n<float, n_, X_N>(A, U, nullptr, p, tw, {}, {}, s);    \
        return true;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

}  // namespace vie
