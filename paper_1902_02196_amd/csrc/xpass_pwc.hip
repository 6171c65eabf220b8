// x pass of the PWC basis (3 unknowns per voxel, the pulse functions), both
// precisions: the row transforms of xpass.hpp around the 3 x 3 block of each
// frequency.  That block couples only the three components of one sibling at
// one frequency, so a wavefront that owns whole siblings needs nobody else:
// one wavefront per workgroup, 3 SB rows of N in LDS, no workgroup barrier.
// The block comes from the 6 tensors of the pulse functions (unique entries
// u = 10 pq, ll = 11), one lane per frequency, shared by the SB siblings.
#include "xpass.hpp"

namespace vie {

template <typename R, int N, int SB>
__global__ void __launch_bounds__(64) k_p3_pwc_wave(C<R>* __restrict__ A, const C<R>* __restrict__ U, P3Params p,
                                                    const C<R>* __restrict__ tw) {
    constexpr int RW = 3 * SB, PARTS = 4 / SB, OX = N / 2 + 1, ITERS = (N + 63) / 64;
    using L = RowLayout<R, N>;
    extern __shared__ unsigned char smem_raw[];
    C<R>* buf = reinterpret_cast<C<R>*>(smem_raw);
    const int lane = threadIdx.x, Nx = p.Nx, s_c = (int)p.s_c;
    // item -> (octant row, right-hand side, part of its siblings), the items
    // of one operator row on one XCD
    const int K = PARTS * p.nrhs, q0 = blockIdx.x >> 3;
    const int row = (q0 / K) * 8 + (blockIdx.x & 7);
    const int kk = q0 - (q0 / K) * K, r = kk / PARTS, part = kk - r * PARTS;
    const int oz = row / p.Oy, oy = row - oz * p.Oy;
    const bool has_y = oy > 0 && 2 * oy < p.My, has_z = oz > 0 && 2 * oz < p.Mz;
    if (row >= p.Oy * p.Oz || (SB < 4 && part * SB >= 2 && !has_z) || (SB == 1 && (part & 1) && !has_y)) return;
    const C<R>* Ur = U + (long long)row * 60 * OX;
    const long long base = (long long)r * p.s_r + (long long)oz * p.s_z + (long long)oy * p.s_y;
    const long long ystep = (long long)(p.My - 2 * oy) * p.s_y, zstep = (long long)(p.Mz - 2 * oz) * p.s_z;
    // row t = 3 sb + c: offset, whether its sibling exists, sign bit
    auto at = [&](int t, bool& ok, unsigned& sgn) {
        const int sb = t / 3, c = t - 3 * sb, g = part * SB + sb, sy = g & 1, sz = g >> 1;
        ok = (!sy || has_y) && (!sz || has_z);
        sgn = ((((sz ? kFoldZ : 0u) ^ (sy ? kFoldY : 0u)) >> (4 * c)) & 1u) << 31;
        return base + (sy ? ystep : 0) + (sz ? zstep : 0) + (long long)c * s_c;
    };
    auto load = [&](int t, auto body) {
        bool ok;
        unsigned s;
        const C<R>* src = A + at(t, ok, s);
        body([=](int c) { return ok && c < Nx ? flip_sign(src[c], s) : mk<R>(0, 0); });
    };
    auto store = [&](int t, auto body) {
        bool ok;
        unsigned s;
        C<R>* dst = A + at(t, ok, s);
        body([=](int c, C<R> v) { if (ok && c < Nx) dst[c] = flip_sign(v, s); });
    };
    RowInputs<R, N, RW> in;
    Twiddles<R, N> w;
    in.fetch(0, lane, load);
    row_pass<R, true, N, RW, 0>(buf, w, &in, 0, lane, store);
    w.fetch(tw, lane);
    auto fetch = [&](int i, C<R>* u) {
        const int xi = i * 64 + lane, ox = 2 * xi > N ? (xi < N ? N - xi : 0) : xi;
#pragma unroll
        for (int k = 0; k < 6; ++k) u[k] = Ur[10 * k * OX + ox];
    };
    C<R> u[6];
    fetch(0, u);
    if constexpr (!PassShape<N, 0>::LAST) row_passes<R, true, N, RW, 1>(buf, w, &in, 0, lane, store);
#pragma unroll 1
    for (int i = 0; i < ITERS; ++i) {
        C<R> v[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = u[k];
        if (i + 1 < ITERS) fetch(i + 1, u);
        const int xi = i * 64 + lane;
        if (xi < N) {
            const unsigned sx = 2 * xi > N ? 0x80000000u : 0u;
            C<R>* col = buf + L::col(xi);
#pragma unroll
            for (int sb = 0; sb < SB; ++sb) {
                C<R> x[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    x[c] = col[(3 * sb + c) * L::RB];
                    if ((kFoldX >> (4 * c)) & 1) x[c] = flip_sign(x[c], sx);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    C<R> y = mk<R>(0, 0);
#pragma unroll
                    for (int d = 0; d < 3; ++d) cfma(y, v[pq_index(c, d)], x[d]);
                    if ((kFoldX >> (4 * c)) & 1) y = flip_sign(y, sx);
                    col[(3 * sb + c) * L::RB] = y;
                }
            }
        }
    }
    wave_sync();
    row_pass<R, false, N, RW, 0>(buf, w, &in, 0, lane, store);
    w.fetch(tw, lane);
    if constexpr (!PassShape<N, 0>::LAST) row_passes<R, false, N, RW, 1>(buf, w, &in, 0, lane, store);
}

// Siblings per wavefront: two, which fill the lanes of a pass better than one
// and leave twice as many wavefronts as four (64^3 complex64: 22.6 us with
// two, 27 with one or four); one from length 320, where the rows of two no
// longer leave registers for enough wavefronts (160 x 64 x 64 60 us against
// 73).  Before, with the twelve rows of a z, y octant spread over a workgroup
// of 256 threads: 16^3 5.9 -> 4.1 us, 48^3 19.7 -> 14.6, 64^3 23.8 -> 22.6
// (four vectors 74.8 -> 65.6), 192 x 64 x 64 94 -> 67; complex128 48^3 26.9 ->
// 22.1, 64^3 37.0 -> 35.7, 256 x 64 x 64 328 -> 207.  That kernel stays at 256
// (128 x 64 x 64: 40.5 us against 48.8, four vectors in complex128 364 against
// 429).  What bounds this one at 64^3: the transforms' arithmetic, about 13 us
// at the vector units' rate, and 63 MB of memory traffic, 12 us.
//
// Thin grids (few octant rows) wait for one workgroup from end to end: there
// one sibling per wavefront is taken at 96, 160 and 192, and the workgroup of a
// whole row at 128.  As the bits differ, the rows alone decide, not the number
// of vectors.  us, one / eight vectors, against two siblings: 96 5.8 / 6.3
// against 6.6 / 7.1 at 25 rows, 5.7 / 9.2 against 6.6 / 8.7 at 81; 160 7.9 / 8.2
// against 10.1 / 10.7 at 25, complex128 8.5 / 18.1 against 11.0 / 16.4 at 81; 192
// 8.6 / 12.3 against 12.9 / 15.6 at 81, 9.6 / 27.3 against 13.7 / 27.8 at 289; 128
// 6.4 / 8.7 against 7.4 / 10.1 at 81, 7.2 / 17.5 against 8.3 / 17.2 at 289.
template <typename R, int N> constexpr int pwc_siblings() { return N < 320 ? 2 : 1; }
template <int N> constexpr int pwc_thin_rows() { return N == 128 || N == 192 ? 300 : N == 96 || N == 160 ? 40 : 0; }

template <typename R, int N, int SB = pwc_siblings<R, N>()>
static void launch_n(C<R>* A, const C<R>* U, const P3Params& p, const C<R>* tw, hipStream_t s) {
    constexpr size_t lds = (size_t)3 * SB * RowLayout<R, N>::RB * sizeof(C<R>);
    static_assert(lds <= 64 * 1024, "within the LDS a kernel has without asking");
    const long long nblk = ((long long)p.Oy * p.Oz + 7) / 8 * 8 * (4 / SB) * (long long)p.nrhs;
    VIE_REQUIRE(nblk < (1LL << 31), -1, "x pass: too many workgroups");
    timed_launch(k_p3_pwc_wave<R, N, SB>, dim3((unsigned)nblk), dim3(64), (unsigned)lds, s, A, U, p, tw);
    VIE_HIP(hipGetLastError());
}

template <typename R>
void launch_p3_pwc(C<R>* A, const C<R>* U, const P3Params& p, const C<R>* tw, hipStream_t s) {
    VIE_REQUIRE(2 * p.Nx <= p.plan.n, -1, "x pass: fft length below 2 Nx");
    switch (p.plan.n) {
#define CASE(n_)                                                                                \
    case n_:                                                                                   \
        if constexpr (n_ == 256) return launch_p3_pwc_rows<R, n_>(A, U, p, tw, s);             \
        if constexpr (pwc_thin_rows<n_>() > 0)                                                 \
            if (p.Oy * p.Oz <= pwc_thin_rows<n_>()) {                                          \
                if constexpr (n_ == 128) return launch_p3_pwc_rows<R, n_>(A, U, p, tw, s);     \
                else return launch_n<R, n_, 1>(A, U, p, tw, s);                                \
            }                                                                                  \
        return launch_n<R, n_>(A, U, p, tw, s);
        VIE_P3_LENGTHS(CASE)
#undef CASE
        default: break;
    }
    throw Error(-1, "the PWC x pass needs an fft length along x of 8, 16, 32, 64, 96, 128, 160, 192, 256, "
                            "320, 384 or 512");
}

template void launch_p3_pwc<float>(C<float>*, const C<float>*, const P3Params&, const C<float>*, hipStream_t);
template void launch_p3_pwc<double>(C<double>*, const C<double>*, const P3Params&, const C<double>*, hipStream_t);

}  // namespace vie
