// Matrix-core x pass of the curl operator, both precisions (xpass.hpp).
#include "xpass.hpp"

namespace vie {

template <typename R>
static bool launch_k(C<R>* A, const C<R>* U, const P3Params& p, const C<R>* tw, hipStream_t s) {
    if (!p3_mx_fits((int)sizeof(C<R>), p.plan.n) || 2 * p.Nx > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                                                \
    case n_:                                                                   \
        if constexpr (p3_mx_lds<R, n_>() <= 160 * 1024)                        \
            launch_p3_mx_n<R, n_, X_K>(A, U, nullptr, p, tw, {}, {}, s);       \
        return true;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

template <>
bool launch_p3_mx_curl<float>(C<float>* A, const C<float>* U, const P3Params& p, const C<float>* tw, hipStream_t s) {
    return launch_k<float>(A, U, p, tw, s);
}
template <>
bool launch_p3_mx_curl<double>(C<double>* A, const C<double>* U, const P3Params& p, const C<double>* tw,
                               hipStream_t s) {
    return launch_k<double>(A, U, p, tw, s);
}

}  // namespace vie
