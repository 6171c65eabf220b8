// Strided passes of the fft_mix.hpp lengths, complex128 (strided_mix.hpp).
#include "strided_mix.hpp"

namespace vie {

bool strided_mix_fits(int es, int n) {
    switch (n) {
#define CASE(n_) \
    case n_: return (es == 8 ? mix_lds<float, n_, 16>() : mix_lds<double, n_, 8>()) <= 160 * 1024;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}


template <>
bool launch_strided_mix<double>(bool fwd, bool epi, const C<double>* in, C<double>* out, const StridedPass& p,
                               long long n_o2, long long n_o1, const C<double>* tw, const Epilogue<double>& ep,
                               hipStream_t s) {
    if (!strided_mix_fits(16, p.plan.n) || 2 * (fwd ? p.n_in : p.n_out) > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                                                                        \
    case n_:                                                                                           \
        if (fwd) launch_strided_mix_n<double, true, false, n_, 8>(in, out, p, n_o2, n_o1, tw, ep, s);   \
        else if (epi) launch_strided_mix_n<double, false, true, n_, 8>(in, out, p, n_o2, n_o1, tw, ep, s); \
        else launch_strided_mix_n<double, false, false, n_, 8>(in, out, p, n_o2, n_o1, tw, ep, s);      \
        return true;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

}  // namespace vie
