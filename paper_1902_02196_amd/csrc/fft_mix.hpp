// Register DFTs of the composite radices 6, 9, 10, 12 and 15, and the radix
// sequences of every length the wave-owned transforms are compiled for: all
// even lengths 8 ... 256 made of 2, 3 and 5 (whatever vie_set_grid picks for
// up to 128 voxels), and 320, 384, 512.
#pragma once

#include "fft.hpp"

namespace vie {

constexpr double kPi = 3.14159265358979323846264338327950288;

// cos and sin of 2 pi m / n at compile time: reduced to [0, pi/4] and summed
// from their Taylor series, the last terms first
constexpr double taylor_cos(double x) {
    double s = 1;
    for (int k = 13; k > 0; --k) s = 1 - x * x / ((2 * k - 1) * (2 * k)) * s;
    return s;
}
constexpr double taylor_sin(double x) {
    double s = 1;
    for (int k = 13; k > 0; --k) s = 1 - x * x / ((2 * k) * (2 * k + 1)) * s;
    return x * s;
}
// octant o of the angle and the remainder in units of a full turn / (8 n)
constexpr double turn_cos(int m, int n) {
    m %= n;
    const int o = 8 * m / n;
    const double r = kPi * (8 * m - o * n) / (4.0 * n);         // in [0, pi/4)
    const double q = kPi * (n - (8 * m - o * n)) / (4.0 * n);   // pi/4 - r
    switch (o) {
        case 0: return taylor_cos(r);
        case 1: return taylor_sin(q);
        case 2: return -taylor_sin(r);
        case 3: return -taylor_cos(q);
        case 4: return -taylor_cos(r);
        case 5: return -taylor_sin(q);
        case 6: return taylor_sin(r);
        default: return taylor_cos(q);
    }
}
// sin(2 pi m / n) = cos(2 pi (4 m + 3 n) / (4 n))
constexpr double turn_sin(int m, int n) { return turn_cos(4 * (m % n) + 3 * n, 4 * n); }

// v[n], n = B n1 + n2: length-A DFTs over n1, twiddles W^(n2 k1), length-B
// DFTs over n2, output k1 + A k2 (radix 9, whose factors have one in common).
template <typename R, bool FWD, int A, int B>
__device__ __forceinline__ void dft_ab(C<R>* v) {
    C<R> t[A * B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
        C<R> u[A];
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) u[n1] = v[B * n1 + n2];
        dft_r<R, FWD, A>(u);
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) {
            const R c = R(turn_cos(n2 * k1, A * B)), s = R((FWD ? -1 : 1) * turn_sin(n2 * k1, A * B));
            t[k1 * B + n2] = n2 * k1 == 0 ? u[k1] : cmul(u[k1], mk<R>(c, s));
        }
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        dft_r<R, FWD, B>(t + k1 * B);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = t[k1 * B + k2];
    }
}

// Length-A DFT (A = 2 or 4) of A / 2 inputs, u[s] or u[s] and u[s + 1 mod 4];
// the others are zero and not read.
template <typename R, bool FWD, int A>
__device__ __forceinline__ void dft_run(C<R>* u, int s) {
    if constexpr (A == 2) {
        const C<R> x = u[s];
        u[0] = x;
        u[1] = s ? mk<R>(-x.x, -x.y) : x;
    } else {
        static_assert(A == 4, "a run of half the inputs");
        const C<R> a = u[s], b = u[(s + 1) & 3];
        const C<R> p = cadd(a, b), m = csub(a, b);
        // W^(s k) (a + W^k b)
        if (s == 0) {
            const C<R> d = mul_mi<FWD>(b);
            u[0] = p, u[2] = m, u[1] = cadd(a, d), u[3] = csub(a, d);
        } else if (s == 2) {
            const C<R> d = mul_mi<FWD>(b);
            u[0] = p, u[2] = m, u[1] = mk<R>(-a.x - d.x, -a.y - d.y), u[3] = csub(d, a);
        } else if (s == 3) {
            const C<R> d = mul_mi<FWD>(a);
            u[0] = p, u[2] = csub(b, a), u[1] = csub(b, d), u[3] = cadd(b, d);
        } else {
            const C<R> d = mul_mi<FWD>(a);
            u[0] = p, u[2] = csub(b, a), u[1] = csub(d, b), u[3] = mk<R>(-b.x - d.x, -b.y - d.y);
        }
    }
}

// Inverse of a modulo m
constexpr int inv_mod(int a, int m) {
    for (int x = 1; x < m; ++x)
        if (a % m * x % m == 1) return x;
    return 1;
}

// A and B without a common factor: input n = (B n1 + A n2) mod A B, length-A
// DFTs over n1 and length-B DFTs over n2, output k with k = k1 mod A and
// k = k2 mod B (Good's prime factor algorithm).  No twiddles between the two:
// their roundings, the same for every element and in all three axes, made a
// complex64 product's error up to a third larger (20^3 1.57e-7 of the result
// with radices 8 and 5, 2.07e-7 with a radix of 10 with twiddles).
// HALF: v[n] = 0 for n >= A B / 2 (A even); those inputs are not read.
template <typename R, bool FWD, int A, int B, bool HALF>
__device__ __forceinline__ void dft_pfa(C<R>* v) {
    constexpr int N = A * B, EA = B * inv_mod(B, A), EB = A * inv_mod(A, B);
    C<R> t[N];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
        C<R> u[A];
        int s = 0;   // first of the run of inputs below N / 2
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) {
            const int n = (B * n1 + A * n2) % N, before = (B * (n1 + A - 1) + A * n2) % N;
            if (!HALF || 2 * n < N) u[n1] = v[n];
            if (2 * n < N && 2 * before >= N) s = n1;
        }
        if constexpr (HALF) dft_run<R, FWD, A>(u, s);
        else dft_r<R, FWD, A>(u);
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) t[k1 * B + n2] = u[k1];
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        dft_r<R, FWD, B>(t + k1 * B);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) v[(k1 * EA + k2 * EB) % N] = t[k1 * B + k2];
    }
}

template <typename R, bool FWD, int RAD, bool HALF>
__device__ __forceinline__ void dft_mix(C<R>* v) {
    if constexpr (RAD == 6) dft_pfa<R, FWD, 2, 3, HALF>(v);
    else if constexpr (RAD == 9) dft_ab<R, FWD, 3, 3>(v);
    else if constexpr (RAD == 10) dft_pfa<R, FWD, 2, 5, HALF>(v);
    else if constexpr (RAD == 12) dft_pfa<R, FWD, 4, 3, HALF>(v);
    else if constexpr (RAD == 15) dft_pfa<R, FWD, 3, 5, false>(v);
    else if constexpr (HALF) dft_r_halfin<R, FWD, RAD>(v);
    else dft_r<R, FWD, RAD>(v);
}

// radix sequence of a length (up to three passes, 0 past the last).  An even
// radix first lets a zero-padded transform skip its zero half, an even one
// last lets a cropped inverse skip the half that is dropped; lengths that are
// no power of two start with a radix that is no multiple of 8, so that the
// first pass's stores, RAD elements apart, spread over the LDS banks; but 40 is
// 8 x 5, whose twiddles' roundings add up to less than those of 10 x 4 (error
// of a complex64 product at 20^3 1.58e-7, 1.80e-7; x pass 9.4 us, 10.2).
struct MixRadices {
    int r[3];
};
constexpr MixRadices mix_radices(int n) {
    switch (n) {
        case 8: return {{8, 0, 0}};
        case 10: return {{10, 0, 0}};
        case 12: return {{12, 0, 0}};
        case 16: return {{16, 0, 0}};
        case 18: return {{6, 3, 0}};
        case 20: return {{10, 2, 0}};
        case 24: return {{6, 4, 0}};
        case 30: return {{10, 3, 0}};
        case 32: return {{8, 4, 0}};
        case 36: return {{6, 6, 0}};
        case 40: return {{8, 5, 0}};
        case 48: return {{6, 8, 0}};
        case 50: return {{10, 5, 0}};
        case 54: return {{6, 9, 0}};
        case 60: return {{10, 6, 0}};
        case 64: return {{8, 8, 0}};
        case 72: return {{12, 6, 0}};
        case 80: return {{10, 8, 0}};
        case 90: return {{10, 9, 0}};
        case 96: return {{12, 8, 0}};
        case 100: return {{10, 10, 0}};
        case 108: return {{12, 9, 0}};
        case 120: return {{12, 10, 0}};
        case 128: return {{16, 8, 0}};
        case 144: return {{12, 12, 0}};
        case 150: return {{10, 15, 0}};
        case 160: return {{10, 16, 0}};
        case 162: return {{6, 3, 9}};
        case 180: return {{12, 15, 0}};
        case 192: return {{12, 16, 0}};
        case 200: return {{10, 4, 5}};
        case 216: return {{6, 6, 6}};
        case 240: return {{15, 16, 0}};
        case 250: return {{10, 5, 5}};
        case 256: return {{16, 16, 0}};
        case 320: return {{5, 8, 8}};
        case 384: return {{6, 8, 8}};
        case 512: return {{8, 8, 8}};
        default: return {{0, 0, 0}};
    }
}
constexpr bool mix_supported(int n) { return mix_radices(n).r[0] != 0; }

#define VIE_MIX_LENGTHS(X)                                                                                  \
    X(8) X(10) X(12) X(16) X(18) X(20) X(24) X(30) X(32) X(36) X(40) X(48) X(50) X(54) X(60) X(64) X(72)   \
    X(80) X(90) X(96) X(100) X(108) X(120) X(128) X(144) X(150) X(160) X(162) X(180) X(192) X(200) X(216)  \
    X(240) X(250) X(256) X(320) X(384) X(512)

}  // namespace vie
