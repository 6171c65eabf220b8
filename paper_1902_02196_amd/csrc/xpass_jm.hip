// Matrix-core x pass of the J-M product, both precisions (xpass.hpp).
#include "xpass.hpp"

namespace vie {

// lengths it takes: those whose 48 rows fit LDS and that are not left to the
// 24-row kernel
template <typename R, int N> constexpr bool jm_fits() {
    return !p3_jm_rows24((int)sizeof(C<R>), N) && p3_mx_lds<R, N>(2) <= 160 * 1024;
}

bool p3_mx_jm_fits(int es, int n) {
    switch (n) {
#define CASE(n_) \
    case n_: return es == 8 ? jm_fits<float, n_>() : jm_fits<double, n_>();
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

template <typename R>
static bool launch_jm(C<R>* A, const C<R>* UN, const C<R>* UK, const P3Params& p, const C<R>* tw, C<R> kj, C<R> km,
                      hipStream_t s) {
    if (!p3_mx_jm_fits((int)sizeof(C<R>), p.plan.n) || 2 * p.Nx > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                                                    \
    case n_:                                                                       \
        if constexpr (jm_fits<R, n_>())                                            \
            launch_p3_mx_n<R, n_, X_JM>(A, UN, UK, p, tw, kj, km, s);              \
        return true;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

template <>
bool launch_p3_mx_jm<float>(C<float>* A, const C<float>* UN, const C<float>* UK, const P3Params& p,
                            const C<float>* tw, C<float> kj, C<float> km, hipStream_t s) {
    return launch_jm<float>(A, UN, UK, p, tw, kj, km, s);
}
template <>
bool launch_p3_mx_jm<double>(C<double>* A, const C<double>* UN, const C<double>* UK, const P3Params& p,
                             const C<double>* tw, C<double> kj, C<double> km, hipStream_t s) {
    return launch_jm<double>(A, UN, UK, p, tw, kj, km, s);
}

}  // namespace vie
