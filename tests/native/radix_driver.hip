// Host run of the register DFTs of csrc/fft_mix.hpp:
//   radix RAD FWD HALF <largest error against the definition, double>
//   length N <rms error of a zero-padded forward and a cropped inverse
//   transform in float, with the radices of mix_radices and with those of the
//   run-time plan>
// Inputs that a half-zero butterfly must not read are NaN.
#include <hip/hip_runtime.h>

#undef __device__
#define __device__ __attribute__((device)) __attribute__((host))
#include "fft_mix.hpp"

#include <complex>
#include <cstdio>
#include <random>
#include <vector>

using namespace vie;
using cd = std::complex<double>;

template <bool FWD, int RAD, bool HALF>
static void one_radix() {
    double2 v[RAD];
    cd x[RAD];
    for (int i = 0; i < RAD; ++i) {
        const bool zero = HALF && 2 * i >= RAD;
        x[i] = zero ? cd(0, 0) : cd(std::sin(3 * i + 1.0), std::cos(5 * i * i + 0.3));
        v[i] = zero ? make_double2(NAN, NAN) : make_double2(x[i].real(), x[i].imag());
    }
    dft_mix<double, FWD, RAD, HALF>(v);
    double e = 0;
    for (int k = 0; k < RAD; ++k) {
        cd s = 0;
        for (int i = 0; i < RAD; ++i) s += x[i] * std::polar(1.0, (FWD ? -2 : 2) * M_PI * ((i * k) % RAD) / RAD);
        const double d = std::abs(s - cd(v[k].x, v[k].y));
        if (!(d <= e)) e = d;   // NaN stays
    }
    std::printf("radix %d %d %d %.3e\n", RAD, FWD, HALF, e);
}

template <bool FWD>
static void butterfly(float2* v, int rad, bool half) {
    switch (rad) {
#define CASE(r_)                                                    \
    case r_:                                                        \
        if (half && r_ % 2 == 0) dft_mix<float, FWD, r_, true>(v);  \
        else dft_mix<float, FWD, r_, false>(v);                     \
        break;
        CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(8) CASE(9) CASE(10) CASE(12) CASE(15) CASE(16)
#undef CASE
    }
}

template <bool FWD>
static std::vector<float2> transform(std::vector<float2> x, const std::vector<int>& radices,
                                     const std::vector<float2>& tw) {
    const int n = (int)x.size();
    int Ns = 1;
    for (int r : radices) {
        std::vector<float2> y(n);
        const int nb = n / r;
        for (int j = 0; j < nb; ++j) {
            const int k = j % Ns;
            float2 v[16];
            for (int i = 0; i < r; ++i) v[i] = x[j + i * nb];
            if (Ns > 1)
                for (int i = 1; i < r; ++i) {
                    const float2 w = tw[i * k * (n / (Ns * r))];
                    v[i] = FWD ? cmul(w, v[i]) : cmulc(w, v[i]);
                }
            butterfly<FWD>(v, r, FWD && Ns == 1);
            for (int i = 0; i < r; ++i) y[(j - k) * r + k + i * Ns] = v[i];
        }
        x.swap(y);
        Ns *= r;
    }
    return x;
}

static double error(int n, const std::vector<int>& radices) {
    std::mt19937 g(7);
    std::normal_distribution<double> N;
    std::vector<float2> tw(n);
    std::vector<cd> W(n);
    for (int m = 0; m < n; ++m) {
        W[m] = std::polar(1.0, -2 * M_PI * m / n);
        tw[m] = make_float2((float)W[m].real(), (float)W[m].imag());
    }
    double num = 0, den = 0;
    for (int t = 0; t < 60; ++t) {
        std::vector<float2> x(n), z(n);
        for (int i = 0; i < n; ++i) {
            x[i] = 2 * i < n ? make_float2((float)N(g), (float)N(g)) : make_float2(0, 0);
            z[i] = make_float2((float)N(g), (float)N(g));
        }
        const auto f = transform<true>(x, radices, tw);
        const auto b = transform<false>(z, radices, tw);
        for (int k = 0; k < n; ++k) {
            cd s = 0, q = 0;
            for (int i = 0; i < n; ++i) {
                s += cd(x[i].x, x[i].y) * W[(long long)i * k % n];
                q += cd(z[i].x, z[i].y) * std::conj(W[(long long)i * k % n]);
            }
            num += std::norm(cd(f[k].x, f[k].y) - s);
            den += std::norm(s);
            if (2 * k < n) {
                num += 2 * std::norm(cd(b[k].x, b[k].y) - q);
                den += 2 * std::norm(q);
            }
        }
    }
    return std::sqrt(num / den);
}

int main() {
#define BOTH(r_)                   \
    one_radix<true, r_, false>();  \
    one_radix<false, r_, false>();
#define HALF(r_)                  \
    BOTH(r_)                      \
    one_radix<true, r_, true>();  \
    one_radix<false, r_, true>();
    HALF(2) BOTH(3) HALF(4) BOTH(5) HALF(6) HALF(8) BOTH(9) HALF(10) HALF(12) BOTH(15) HALF(16)
#define LENGTH(n_)                                                                  \
    {                                                                               \
        std::vector<int> mix, plan;                                                 \
        for (int i = 0; i < 3; ++i)                                                 \
            if (mix_radices(n_).r[i]) mix.push_back(mix_radices(n_).r[i]);          \
        int m = n_;                                                                 \
        for (int r : {16, 8, 4, 2, 3, 5})                                           \
            while (m % r == 0) plan.push_back(r), m /= r;                           \
        std::printf("length %d %.4e %.4e\n", n_, error(n_, mix), error(n_, plan)); \
    }
    VIE_MIX_LENGTHS(LENGTH)
    return 0;
}
