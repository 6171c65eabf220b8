// Strided passes of the fft_mix.hpp lengths, complex64 (strided_mix.hpp).
#include "strided_mix.hpp"

namespace vie {

template <>
bool launch_strided_mix<float>(bool fwd, bool epi, const C<float>* in, C<float>* out, const StridedPass& p,
                               long long n_o2, long long n_o1, const C<float>* tw, const Epilogue<float>& ep,
                               hipStream_t s) {
    if (!strided_mix_fits(8, p.plan.n) || 2 * (fwd ? p.n_in : p.n_out) > p.plan.n) return false;
    switch (p.plan.n) {
#define CASE(n_)                                                                                        \
    case n_:                                                                                           \
        if (fwd) launch_strided_mix_n<float, true, false, n_, 16>(in, out, p, n_o2, n_o1, tw, ep, s);   \
        else if (epi) launch_strided_mix_n<float, false, true, n_, 16>(in, out, p, n_o2, n_o1, tw, ep, s); \
        else launch_strided_mix_n<float, false, false, n_, 16>(in, out, p, n_o2, n_o1, tw, ep, s);      \
        return true;
        VIE_MIX_LENGTHS(CASE)
#undef CASE
        default: return false;
    }
}

}  // namespace vie
