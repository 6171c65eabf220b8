// Strided FFT passes (Sec. IV-A) for the lengths of fft_mix.hpp: T pencils
// (consecutive x) per workgroup, work items (butterfly j, pencil t) with t
// fastest.  The first pass reads its inputs from global memory straight into
// the butterflies and the last one stores from them, T contiguous elements at
// a time, so that a two-pass length goes through LDS once, with one barrier.
// Forward transforms are zero-padded (n_in <= N / 2), inverse ones cropped
// (n_out <= N / 2).
//
// Bound by memory: 64^3 complex64 z, y, inverse y and inverse z with its
// epilogue 15, 28, 27 and 29 us (3.7 to 5.7 TB/s); 96 x 128 x 128 with four
// vectors 378, 755, 692 and 384, where staging the tile in LDS first and last
// took 463, 925, 1065 and 634; lengths that had only the run-time kernel (72 x
// 61 x 85 with three, 180 along z) 96 and 124 against 246 and 273.  Tiles of 128 bytes: half of that costs 20 to 40% (partial lines),
// twice leaves fewer workgroups and gained nothing.  Plain instead of
// streaming loads of the input save 8 us of the y pass at 64^3 and cost the
// x pass 8, whose operator then leaves the Infinity Cache.
#pragma once

#include <mutex>

#include "fft_mix.hpp"
#include "kernels.hpp"
#include "passes.hpp"
#include "vie.h"

namespace vie {

// the radices of fft_mix.hpp, except that with the pencils fastest in LDS a
// radix of 16 may come first: more loads in flight per work item.  us of the z,
// y, inverse y and inverse z passes, three complex64 vectors, 16 first against
// 12 or 10: 80 (40^3, four vectors) 19, 39, 34, 19 against 19, 40, 36, 24; 96
// (64 x 48 x 48) 26, 42, 42, 24 against 28, 42, 46, 33; 160 (64 x 80 x 80) 82,
// 162, 148 against 92, 188, 170 (its inverse z is staged); 192 (64 x 96 x 96)
// 113, 227, 208, 138 against 115, 229, 211, 151.
// 8 to 16 take two passes where one radix would do: with a whole pencil per
// work item a workgroup of 64 had 8 or 16 of them, and the epilogue, which
// loads and stores three values per output, waited on each in turn (64 x 64 x
// 8, four vectors: inverse z pass 20 us in one pass, 10 in two; complex128 76
// and 24, 33 in the staged kernel).
constexpr MixRadices strided_radices(int n) {
    switch (n) {
        case 8: return {{4, 2, 0}};
        case 10: return {{2, 5, 0}};
        case 12: return {{4, 3, 0}};
        case 16: return {{4, 4, 0}};
        case 80: return {{16, 5, 0}};
        case 96: return {{16, 6, 0}};
        case 160: return {{16, 10, 0}};
        case 192: return {{16, 12, 0}};
        default: return mix_radices(n);
    }
}
template <int N, int S>
struct MixShape {
    static constexpr int RAD = S < 3 ? strided_radices(N).r[S < 3 ? S : 2] : 0;
    static constexpr int NS = MixShape<N, S - 1>::NS * MixShape<N, S - 1>::RAD;
    static constexpr bool LAST = S == 2 || strided_radices(N).r[S < 2 ? S + 1 : 2] == 0;
};
template <int N>
struct MixShape<N, 0> {
    static constexpr int RAD = strided_radices(N).r[0], NS = 1;
    static constexpr bool LAST = strided_radices(N).r[1] == 0;
};

// Work items of a workgroup: the count (64 ... 256) whose rounds over the
// butterflies of all passes leave the fewest idle, the larger one of equals
constexpr int mix_cost(int n, int T, int nt) {
    int c = 0;
    for (int s = 0; s < 3; ++s) {
        const int r = strided_radices(n).r[s];
        if (r) c += (n / r * T + nt - 1) / nt * r;
    }
    return c * nt;
}
constexpr int mix_threads(int n, int T) {
    int best = 64;
    for (int nt = 128; nt <= 256; nt += 64)
        if (mix_cost(n, T, nt) <= mix_cost(n, T, best)) best = nt;
    return best;
}

// element k of pencil t in LDS: an odd pitch spreads the butterflies of a pass
template <int T> constexpr int mix_pitch() { return T + 1; }
template <typename R, int N, int T> constexpr size_t mix_lds() {
    return MixShape<N, 0>::LAST ? 0 : (size_t)N * mix_pitch<T>() * sizeof(C<R>);
}

template <typename R, bool FWD, int N, int T, int NT, int S, typename Load, typename Pre, typename Store>
__device__ __forceinline__ void mix_passes(C<R>* buf, const C<R>* __restrict__ tw, int tid, Load load,
                                           Pre pre, Store store) {
    using P = MixShape<N, S>;
    constexpr int RAD = P::RAD, NS = P::NS, nb = N / RAD, TP = mix_pitch<T>();
    constexpr int WORK = nb * T, ROUNDS = (WORK + NT - 1) / NT;
    constexpr bool FIRST = S == 0, LAST = P::LAST, MIDDLE = !FIRST && !LAST;
    C<R> v[MIDDLE ? ROUNDS : 1][RAD];
    decltype(pre(0, 0)) ex[LAST ? RAD : 1];   // what the outputs will be combined with
    auto prefetch = [&](int q) {
        const int w = tid + q * NT, j = w / T, t = w - j * T, k = j % NS, c0 = (j - k) * RAD + k;
        if (WORK % NT != 0 && w >= WORK) return;
#pragma unroll
        for (int i = 0; i < RAD; ++i)
            if (FWD || 2 * i * NS < N) ex[i] = pre(c0 + i * NS, t);
    };
    auto butterfly = [&](int q, C<R>* v) {
        const int w = tid + q * NT, j = w / T, t = w - j * T, k = j % NS;
        if (WORK % NT != 0 && w >= WORK) return;
        if constexpr (FIRST) {
#pragma unroll
            for (int i = 0; i < RAD; ++i) {
                if (!FWD || 2 * i * nb < N) v[i] = load(j + i * nb, t);   // beyond: the zero padding
                else if (RAD % 2) v[i] = mk<R>(0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < RAD; ++i) v[i] = buf[(j + i * nb) * TP + t];
#pragma unroll
            for (int i = 1; i < RAD; ++i) {
                const C<R> u = tw[i * k * (N / (NS * RAD))];
                v[i] = FWD ? cmul(u, v[i]) : cmulc(u, v[i]);
            }
        }
        dft_mix<R, FWD, RAD, FIRST && FWD && RAD % 2 == 0>(v);
    };
    auto put = [&](int q, C<R>* v) {
        const int w = tid + q * NT, j = w / T, t = w - j * T, k = j % NS, c0 = (j - k) * RAD + k;
        if (WORK % NT != 0 && w >= WORK) return;
        if constexpr (LAST) {
#pragma unroll
            for (int i = 0; i < RAD; ++i)
                if (FWD || 2 * i * NS < N) store(c0 + i * NS, t, v[i], ex[i]);   // beyond: cropped
        } else {
#pragma unroll
            for (int i = 0; i < RAD; ++i) buf[(c0 + i * NS) * TP + t] = v[i];
        }
    };
    if constexpr (MIDDLE) {   // in place: all inputs are read before any output is written
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) butterfly(q, v[q]);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) put(q, v[q]);
    } else {
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            if constexpr (LAST) prefetch(q);
            butterfly(q, v[0]);
            put(q, v[0]);
        }
    }
    if constexpr (!LAST) {
        __syncthreads();
        mix_passes<R, FWD, N, T, NT, S + 1>(buf, tw, tid, load, pre, store);
    }
}

template <typename R, bool FWD, bool EPI, int N, int T>
__global__ void __launch_bounds__(mix_threads(N, T)) k_strided_mix(const C<R>* in, C<R>* out, StridedPass p,
                                                                   const C<R>* __restrict__ tw, Epilogue<R> ep) {
    constexpr int NT = mix_threads(N, T);
    extern __shared__ unsigned char smem_raw[];
    C<R>* buf = reinterpret_cast<C<R>*>(smem_raw);
    // (tile, row, component array) in XCD-contiguous order, tiles fastest
    const unsigned gx = gridDim.x, gy = gridDim.y, gz = gridDim.z;
    const unsigned lid = xcd_contiguous(blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z), gx * gy * gz);
    const unsigned bx = lid % gx, by = (lid / gx) % gy, bz = lid / gx / gy;
    const int t0 = bx * T, tw_n = min(T, p.n_inner - t0);
    const long long o2 = by;
    const int o1 = bz, rr = o1 / p.nc, cc = o1 - p.nc * rr;
    const C<R>* src = in + rr * p.in_s1 + cc * p.in_sc + o2 * p.in_s2 + t0;
    const long long obase = rr * p.out_s1 + cc * p.out_sc;
    C<R>* dst = out + obase + o2 * p.out_s2 + t0;
    const int l = p.nc == 12 ? (cc & 3) : 0;
    const int n_in = p.n_in, n_out = p.n_out;
    auto load = [&](int k, int t) {
        return k < n_in && t < tw_n ? stream_load(&src[k * p.in_sk + t]) : mk<R>(0, 0);   // last read of the input
    };
    // the epilogue's operands are fetched ahead of the last pass, so that their
    // latency runs beside its LDS reads and butterflies
    struct Operands { C<R> b, a, x; };
    const bool has_a = EPI && (ep.a || ep.a_const != R(0));
    auto pre = [&](int k, int t) {
        Operands o{};
        if (EPI && k < n_out && t < tw_n) {
            const long long v = o2 * p.out_s2 + k * p.out_sk + t0 + t;   // voxel
            o.b = ep.b ? ep.b[v] : mk<R>(ep.b_const, 0);
            if (has_a) {
                o.a = ep.a ? ep.a[v] : mk<R>(ep.a_const, 0);
                o.x = ep.x[obase + v];
            }
        }
        return o;
    };
    auto store = [&](int k, int t, C<R> w, const Operands& o) {
        if (k < n_out && t < tw_n) {
            if (EPI) {
                const long long e = obase + o2 * p.out_s2 + k * p.out_sk + t0 + t;   // element
                C<R> y = cscale(cmul(o.b, w), ep.gb[l]);
                if (has_a) y = cadd(y, cscale(cmul(o.a, o.x), ep.ga[l]));
                if (ep.rhs) y = cadd(y, ep.rhs[e]);
                w = y;
            }
            dst[k * p.out_sk + t] = w;
        }
    };
    mix_passes<R, FWD, N, T, NT, 0>(buf, tw, threadIdx.x, load, pre, store);
}

template <typename R, bool FWD, bool EPI, int N, int T>
void launch_strided_mix_n(const C<R>* in, C<R>* out, const StridedPass& p, long long n_o2, long long n_o1,
                          const C<R>* tw, const Epilogue<R>& ep, hipStream_t s) {
    constexpr size_t lds = mix_lds<R, N, T>();
    static std::once_flag once;
    std::call_once(once, [&] {
        (void)hipFuncSetAttribute((const void*)k_strided_mix<R, FWD, EPI, N, T>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        (void)hipGetLastError();
    });
    dim3 grid((p.n_inner + T - 1) / T, (unsigned)n_o2, (unsigned)n_o1);
    VIE_REQUIRE((unsigned long long)grid.x * grid.y * grid.z < (1ULL << 32), VIE_EINVAL,
                "strided pass grid above 2^32 workgroups");
    timed_launch(k_strided_mix<R, FWD, EPI, N, T>, grid, dim3(mix_threads(N, T)), (unsigned)lds, s, in, out, p, tw,
                 ep);
    VIE_HIP(hipGetLastError());
}

}  // namespace vie
