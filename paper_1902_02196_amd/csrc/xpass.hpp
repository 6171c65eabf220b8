// x pass on the matrix cores (Sec. IV-A): forward FFT along x of the 12
// component rows of a pencil, the 12 x 12 block product with the
// octant-folded operator at every frequency, inverse FFT, crop; in place on
// the [R][Mz][My][12][Nx] buffer.
//
// One workgroup holds the two y siblings (xi_y, M_y - xi_y) of one z sibling
// of one octant row, for one right-hand side: 24 rows of N in LDS.  With the
// x fold (xi, N - xi) four vectors then share the operator block of an octant
// frequency up to signs, which is what a 4 x 4 matrix instruction wants: the
// rows of a matrix block are the four scalar bases of one field component,
// its columns the four (x fold, y sibling) vectors.
//
//   complex64   v_mfma_f32_4x4x1_16b: 16 frequencies per instruction, one
//               input unknown (q, l') each; 144 instructions per 16
//               frequencies and 4 vectors
//   complex128  v_mfma_f64_4x4x4_4b: 4 frequencies, the four l' of one q;
//               36 instructions per 4 frequencies and 4 vectors
//
// Both are exact products accumulated in the precision of the data, as the
// fused multiply-adds of the other variants are.  The product leaves the
// vector units to the transforms: with one fused multiply-add per entry it
// was 19 of the 43 million vector instructions of a launch at 64^3.
//
// Each wavefront transforms its own rows (24 / NW of them) from end to end,
// so that the passes of a transform need no workgroup barrier; the first pass
// reads global memory straight into its butterflies, the last one stores from
// them.  Two barriers remain, around the product, which mixes the rows.
//
// What bounds it (64^3 complex64, 105-110 us for 333 MB): no single unit.
// Every lane's operator load is an L1 access of its own (65 of 79 million); the
// L1's address and data units are busy 71% and 85% of the time, the vector
// units 46%, the matrix cores 17%, LDS 28%, memory runs at 3.1 TB/s; without
// the operator loads 65 us, without the product 48.  Tried and no faster: the
// loads along the frequencies and a lane exchange through LDS (L1 accesses 79
// -> 33 million, LDS 28 -> 45%: 110-116 us), four siblings per workgroup (half
// the operator loads, but workgroups too large to overlap: 125 us), a
// persistent kernel that prefetches the next rows (its loads queue behind its
// stores: 172 us), operator values ahead of the last forward pass (117 us).
// Against the variants before it: 16^3 complex64 9.0 -> 8.3 us, 64^3 level
// with the best of them (2, the siblings of a row in a workgroup), 48^3 84 ->
// 57, 96 x 128 x 128 with four vectors 3504 -> 3090; complex128 16^3 19.8 -> 9.2, 32^3 92 -> 25, 64^3 294 -> 210; the lengths
// that had only the run-time kernel 72 x 61 x 85 with three vectors 2593 ->
// 601, complex128 45 x 50 x 37 with two 710 -> 107.
//
// The curl operator K takes the same tiles: 30 tensors instead of 60, one
// field component of the input fewer per output component.  Complex128 64^3,
// two vectors, the whole magnetic-field product: 3059 -> 1648 us with the
// strided passes (the staged kernel before it held a workgroup per CU and ran
// its length's plan).  The J-M pass holds both coefficient sets of a row (48
// rows) and applies N and K to each in one visit; p3_jm_rows24 states where
// it does not run.
#pragma once

#include <mutex>

#include "fft_mix.hpp"
#include "kernels.hpp"
#include "vie.h"

namespace vie {

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

// order LDS accesses of one wavefront (its instructions complete in order;
// this keeps the compiler from moving them across)
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// flip the sign of both parts where bit 31 of s is set
__device__ __forceinline__ float2 flip_sign(float2 v, unsigned s) {
    v.x = __uint_as_float(__float_as_uint(v.x) ^ s);
    v.y = __uint_as_float(__float_as_uint(v.y) ^ s);
    return v;
}
__device__ __forceinline__ double2 flip_sign(double2 v, unsigned s) {
    const unsigned long long f = (unsigned long long)s << 32;
    v.x = __longlong_as_double(__double_as_longlong(v.x) ^ f);
    v.y = __longlong_as_double(__double_as_longlong(v.y) ^ f);
    return v;
}

// LDS layout of groups of 12 rows of N (one group per sibling): rows of a
// power of two are padded by one element every 16, others to an odd pitch;
// every second group is offset so that the two y siblings of a column fall on
// opposite halves of the banks
template <typename R, int N>
struct RowLayout {
    static constexpr bool PAD = (N & (N - 1)) == 0 && N >= 16;
    static constexpr int RB = PAD ? N + N / 16 : (N | 1);
    static constexpr int BANKS = 256 / (int)sizeof(C<R>);   // elements per sweep of the 64 banks
    static constexpr int SD = (BANKS / 2 + BANKS - 12 * RB % BANKS) % BANKS;
    static constexpr int PAIR = 24 * RB + SD;               // two groups
    // row t of the workgroup (12 consecutive rows per group)
    static __device__ __forceinline__ int row(int t) {
        const int g = t / 12;
        return t * RB + (g & 1) * SD + (g >> 1) * (PAIR - 24 * RB);
    }
    static __device__ __forceinline__ int col(int c) { return PAD ? c + (c >> 4) : c; }
};

// radix and span of pass S
template <int N, int S>
struct PassShape {
    static constexpr int RAD = S < 3 ? mix_radices(N).r[S < 3 ? S : 2] : 0;
    static constexpr int NS = PassShape<N, S - 1>::NS * PassShape<N, S - 1>::RAD;
    static constexpr bool LAST = RAD > 0 && (S == 2 || mix_radices(N).r[S < 2 ? S + 1 : 2] == 0);
};
template <int N>
struct PassShape<N, 0> {
    static constexpr int RAD = mix_radices(N).r[0], NS = 1;
    static constexpr bool LAST = mix_radices(N).r[1] == 0;
};

// Twiddles of a lane's butterflies in the second and third pass: the same for
// all rows and for both directions (conjugated), so they are fetched ahead of
// the pass that needs them.
template <typename R, int N>
struct Twiddles {
    static constexpr int R1 = PassShape<N, 1>::RAD, R2 = PassShape<N, 2>::RAD;
    C<R> w1[R1 > 0 ? R1 : 1], w2[R2 > 0 ? R2 : 1];

    __device__ __forceinline__ void fetch(const C<R>* __restrict__ tw, int lane) {
        if constexpr (R1 > 0) {
            constexpr int nb = N / R1, NS = PassShape<N, 1>::NS;
            const int k = lane % nb % NS;
#pragma unroll
            for (int i = 1; i < R1; ++i) w1[i] = tw[i * k * (N / (NS * R1))];
        }
        if constexpr (R2 > 0) {
            constexpr int nb = N / R2, NS = PassShape<N, 2>::NS;
            const int k = lane % nb % NS;
#pragma unroll
            for (int i = 1; i < R2; ++i) w2[i] = tw[i * k * (N / (NS * R2))];
        }
    }
};

// Butterflies of the rows [t0, t0 + RW) of one wavefront in pass S: butterfly j
// of a row sits in lane lr nb + j, a round covers RPR whole rows, so a pass
// may work in place.
template <int N, int RW, int S>
struct PassMap {
    static constexpr int RAD = PassShape<N, S>::RAD, NS = PassShape<N, S>::NS, nb = N / RAD;
    static_assert(nb <= 64, "one row per round at least");
    static constexpr int RPR = 64 / nb, ROUNDS = (RW + RPR - 1) / RPR;
    int lr, j, c0;
    __device__ __forceinline__ PassMap(int lane) {
        lr = lane / nb;
        j = lane - lr * nb;
        const int k = j % NS;
        c0 = (j - k) * RAD + k;
    }
    __device__ __forceinline__ bool act(int q) const { return lr < RPR && q * RPR + lr < RW; }
    __device__ __forceinline__ int row(int q) const { return q * RPR + lr; }
};

// Inputs of the first forward pass, fetched from global memory into the
// registers of its butterflies (the zero padding of a row is not read)
template <typename R, int N, int RW>
struct RowInputs {
    using P = PassMap<N, RW, 0>;
    static constexpr int CNT = (P::RAD + 1) / 2;   // inputs below N / 2
    C<R> v[P::ROUNDS][CNT];

    template <typename Load>
    __device__ __forceinline__ void fetch(int t0, int lane, Load load) {
        const P m(lane);
#pragma unroll
        for (int q = 0; q < P::ROUNDS; ++q)
            if (m.act(q)) {
                load(t0 + m.row(q), [&](auto get) {
#pragma unroll
                    for (int i = 0; i < CNT; ++i) v[q][i] = get(m.j + i * P::nb);
                });
            }
    }
};

// Pass S of the transform of rows [t0, t0 + RW), all in one wavefront.  The
// first forward pass takes its inputs from `in`, the last inverse pass hands
// its outputs to store(row, column, value); all else is LDS.
template <typename R, bool FWD, int N, int RW, int S, typename Store>
__device__ __forceinline__ void row_pass(C<R>* buf, const Twiddles<R, N>& tw, const RowInputs<R, N, RW>* in, int t0,
                                         int lane, Store store) {
    using L = RowLayout<R, N>;
    using P = PassMap<N, RW, S>;
    constexpr int RAD = P::RAD, NS = P::NS, nb = P::nb;
    constexpr bool GIN = FWD && S == 0, GOUT = !FWD && PassShape<N, S>::LAST;
    constexpr bool HIN = GIN && RAD % 2 == 0;
    const P m(lane);
#pragma unroll
    for (int q = 0; q < P::ROUNDS; ++q) {
        const int t = t0 + m.row(q);
        if (m.act(q)) {
            C<R> v[RAD];
            if constexpr (GIN) {
                constexpr int CNT = RowInputs<R, N, RW>::CNT;
#pragma unroll
                for (int i = 0; i < RAD; ++i) {
                    if (i < CNT) v[i] = in->v[q][i];
                    else if (!HIN) v[i] = mk<R>(0, 0);
                }
            } else {
                const C<R>* src = buf + L::row(t) + L::col(m.j);
#pragma unroll
                for (int i = 0; i < RAD; ++i) v[i] = src[i * nb + (L::PAD ? (i * nb) >> 4 : 0)];
            }
            if constexpr (S > 0) {
#pragma unroll
                for (int i = 1; i < RAD; ++i) {
                    const C<R> w = S == 1 ? tw.w1[i] : tw.w2[i];
                    v[i] = FWD ? cmul(w, v[i]) : cmulc(w, v[i]);
                }
            }
            dft_mix<R, FWD, RAD, HIN>(v);
            if constexpr (GOUT) {
                store(t, [&](auto put) {
#pragma unroll
                    for (int i = 0; i < RAD; ++i)
                        if (2 * i * NS < N) put(m.c0 + i * NS, v[i]);   // beyond: cropped
                });
            } else {
                C<R>* dst = buf + L::row(t) + L::col(m.c0);
#pragma unroll
                for (int i = 0; i < RAD; ++i) dst[i * NS + (L::PAD ? (i * NS) >> 4 : 0)] = v[i];
            }
        }
    }
    wave_sync();
}

// passes S, S + 1, ... of the transform
template <typename R, bool FWD, int N, int RW, int S, typename Store>
__device__ __forceinline__ void row_passes(C<R>* buf, const Twiddles<R, N>& tw, const RowInputs<R, N, RW>* in, int t0,
                                           int lane, Store store) {
    if constexpr (PassShape<N, S>::RAD > 0) {
        row_pass<R, FWD, N, RW, S>(buf, tw, in, t0, lane, store);
        if constexpr (!PassShape<N, S>::LAST) row_passes<R, FWD, N, RW, S + 1>(buf, tw, in, t0, lane, store);
    }
}

// signs of the component rows under the folds: bit a set where the sibling's
// value enters with the opposite sign
constexpr unsigned kFoldX = fold_mask(1, 0, 0), kFoldY = fold_mask(0, 1, 0), kFoldZ = fold_mask(0, 0, 1);

// curl operator K^{(p,l),(q,l')} = levi(p, k, q) Q_k^{ll'} (zero for p = q):
// dyad index and sign of the block (p, q)
constexpr int curl_k(int p, int q) { return 3 - p - q; }
constexpr bool curl_neg(int p, int q) { return levi(p, 3 - p - q, q) < 0; }

// One tile of octant frequencies in complex64: 16 frequencies (block b =
// lane / 4), row or column lane % 4.  Column (fx, sy) reads and writes its
// own column xi of its own sibling's rows.
template <int N>
struct Tile32 {
    using L = RowLayout<float, N>;
    static constexpr int COUNT = 16, OX = N / 2 + 1, TILES = (OX + COUNT - 1) / COUNT;
    // operator values of ND dyads: column l', dyad, row lane % 4
    template <int ND> struct Op {
        float2 a[4][ND];
        __device__ __forceinline__ void load(const float2* __restrict__ U, int tile, int lane, int lp) {
            const int ox = min(tile * COUNT + (lane >> 2), OX - 1), i = lane & 3;
            const int lo = min(i, lp), hi = max(i, lp);
            const int off = (lo * (9 - lo) / 2 + (hi - lo)) * OX + ox;   // ll_index(i + 1, lp + 1)
#pragma unroll
            for (int d = 0; d < ND; ++d) a[lp][d] = U[10 * d * OX + off];
        }
        __device__ __forceinline__ void load(const float2* __restrict__ U, int tile, int lane) {
#pragma unroll
            for (int lp = 0; lp < 4; ++lp) load(U, tile, lane, lp);
        }
        // exchanged pulse / linear pairs: column l' = 1, rows l > 1
        __device__ __forceinline__ void fix(int lane) {
            const unsigned sa = (lane & 3) ? 0x80000000u : 0u;
#pragma unroll
            for (int d = 0; d < ND; ++d) a[0][d] = flip_sign(a[0][d], sa);
        }
    };
    struct Acc { mfma_f4 r[3], i[3]; };

    bool ok;
    int off;       // of the column in the rows of a pair of siblings
    unsigned sx;   // x fold

    __device__ __forceinline__ Tile32(int tile, int lane, int ny_sib) {
        const int ox = tile * COUNT + (lane >> 2), fx = (lane >> 1) & 1, sy = lane & 1;
        // the folded column exists strictly between 0 and N / 2
        ok = ox < OX && (!fx || (ox > 0 && 2 * ox < N)) && sy < ny_sib;
        const int oxc = ok ? ox : 0;
        off = (sy && ok ? L::row(12) : 0) + L::col(fx && ok ? N - oxc : oxc);
        sx = (unsigned)fx << 31;
    }
    static __device__ __forceinline__ void clear(Acc& y) {
#pragma unroll
        for (int p = 0; p < 3; ++p) y.r[p] = y.i[p] = mfma_f4{0, 0, 0, 0};
    }
    // y *= f
    static __device__ __forceinline__ void scale(Acc& y, float2 f) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float2 v = cmul(make_float2(y.r[p][i], y.i[p][i]), f);
                y.r[p][i] = v.x;
                y.i[p][i] = v.y;
            }
    }
    // y += the part of N x or K x from the inputs of scalar basis l' = lp + 1,
    // x the column of rows at buf
    template <bool CURL, int ND>
    __device__ __forceinline__ void accumulate(Acc& y, const Op<ND>& op, const float2* buf, int lp) const {
        const float2* col = buf + off;
        float2 x[3], nx[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            x[q] = col[(4 * q + lp) * L::RB];
            if ((kFoldX >> (4 * q + lp)) & 1) x[q] = flip_sign(x[q], sx);
            nx[q] = make_float2(-x[q].x, -x[q].y);
        }
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                if (CURL && p == q) continue;
                const float2 v = op.a[lp][CURL ? curl_k(p, q) : pq_index(p, q)];
                const bool neg = CURL && curl_neg(p, q);
                const float2 u = neg ? nx[q] : x[q], w = neg ? x[q] : nx[q];
                y.r[p] = __builtin_amdgcn_mfma_f32_4x4x1f32(v.x, u.x, y.r[p], 0, 0, 0);
                y.i[p] = __builtin_amdgcn_mfma_f32_4x4x1f32(v.x, u.y, y.i[p], 0, 0, 0);
                y.r[p] = __builtin_amdgcn_mfma_f32_4x4x1f32(v.y, w.y, y.r[p], 0, 0, 0);
                y.i[p] = __builtin_amdgcn_mfma_f32_4x4x1f32(v.y, u.x, y.i[p], 0, 0, 0);
            }
    }
    template <bool CURL, int ND>
    __device__ __forceinline__ void accumulate(Acc& y, const Op<ND>& op, const float2* buf) const {
#pragma unroll
        for (int lp = 0; lp < 4; ++lp) accumulate<CURL>(y, op, buf, lp);
    }
    // y0 += N x0 and y1 += N x1 (or K), the operator fetched column by column:
    // with all of it in registers the two sums would spill
    template <bool CURL, int ND>
    __device__ __forceinline__ void accumulate2(Acc& y0, Acc& y1, const float2* __restrict__ U, int tile, int lane,
                                                const float2* x0, const float2* x1) const {
        Op<ND> op;
#pragma unroll
        for (int lp = 0; lp < 4; ++lp) {
            if (lp % 2 == 0) __builtin_amdgcn_sched_barrier(0);   // loads of two columns in flight
            op.load(U, tile, lane, lp);
            if (lp == 0) op.fix(lane);
            accumulate<CURL>(y0, op, x0, lp);
            accumulate<CURL>(y1, op, x1, lp);
        }
    }
    // ODD: the operator itself changes sign under the x fold (the curl)
    template <bool ODD>
    __device__ __forceinline__ void store(const Acc& y, float2* buf) const {
        if (!ok) return;
        float2* col = buf + off;
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float2 v = make_float2(y.r[p][i], y.i[p][i]);
                if ((((kFoldX >> (4 * p + i)) & 1) != 0) != ODD) v = flip_sign(v, sx);
                col[(4 * p + i) * L::RB] = v;
            }
    }
};

// The same in complex128: 4 frequencies (block (lane / 4) % 4), row or column
// lane % 4, the four l' of an input component at lane / 16; the output row of
// a column sits at lane / 16.
template <int N>
struct Tile64 {
    using L = RowLayout<double, N>;
    static constexpr int COUNT = 4, OX = N / 2 + 1, TILES = (OX + COUNT - 1) / COUNT;
    template <int ND> struct Op {
        double2 a[ND];
        __device__ __forceinline__ void load(const double2* __restrict__ U, int tile, int lane) {
            const int ox = min(tile * COUNT + ((lane >> 2) & 3), OX - 1), i = lane & 3, lp = lane >> 4;
            const int lo = min(i, lp), hi = max(i, lp);
            const int off = (lo * (9 - lo) / 2 + (hi - lo)) * OX + ox;   // ll_index(i + 1, lp + 1)
#pragma unroll
            for (int d = 0; d < ND; ++d) a[d] = U[10 * d * OX + off];
        }
        __device__ __forceinline__ void fix(int lane) {   // exchanged pulse / linear pairs
            const unsigned sa = lane < 16 && (lane & 3) ? 0x80000000u : 0u;
#pragma unroll
            for (int d = 0; d < ND; ++d) a[d] = flip_sign(a[d], sa);
        }
    };
    struct Acc { double r[3], i[3]; };

    bool ok;
    int off, l;
    unsigned sx;

    __device__ __forceinline__ Tile64(int tile, int lane, int ny_sib) {
        const int ox = tile * COUNT + ((lane >> 2) & 3), fx = (lane >> 1) & 1, sy = lane & 1;
        l = lane >> 4;
        ok = ox < OX && (!fx || (ox > 0 && 2 * ox < N)) && sy < ny_sib;
        const int oxc = ok ? ox : 0;
        off = (sy && ok ? L::row(12) : 0) + L::col(fx && ok ? N - oxc : oxc) + l * L::RB;
        sx = (unsigned)fx << 31;
    }
    static __device__ __forceinline__ void clear(Acc& y) {
#pragma unroll
        for (int p = 0; p < 3; ++p) y.r[p] = y.i[p] = 0;
    }
    static __device__ __forceinline__ void scale(Acc& y, double2 f) {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const double2 v = cmul(make_double2(y.r[p], y.i[p]), f);
            y.r[p] = v.x;
            y.i[p] = v.y;
        }
    }
    template <bool CURL, int ND>
    __device__ __forceinline__ void accumulate(Acc& y, const Op<ND>& op, const double2* buf) const {
        const double2* col = buf + off;
        double2 x[3], nx[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            x[q] = flip_sign(col[4 * q * L::RB], ((kFoldX >> (4 * q + l)) & 1) ? sx : 0u);
            nx[q] = make_double2(-x[q].x, -x[q].y);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                if (CURL && p == q) continue;
                const double2 v = op.a[CURL ? curl_k(p, q) : pq_index(p, q)];
                const bool neg = CURL && curl_neg(p, q);
                const double2 u = neg ? nx[q] : x[q], w = neg ? x[q] : nx[q];
                y.r[p] = __builtin_amdgcn_mfma_f64_4x4x4f64(v.x, u.x, y.r[p], 0, 0, 0);
                y.i[p] = __builtin_amdgcn_mfma_f64_4x4x4f64(v.x, u.y, y.i[p], 0, 0, 0);
                y.r[p] = __builtin_amdgcn_mfma_f64_4x4x4f64(v.y, w.y, y.r[p], 0, 0, 0);
                y.i[p] = __builtin_amdgcn_mfma_f64_4x4x4f64(v.y, u.x, y.i[p], 0, 0, 0);
            }
    }
    template <bool CURL, int ND>
    __device__ __forceinline__ void accumulate2(Acc& y0, Acc& y1, const double2* __restrict__ U, int tile, int lane,
                                                const double2* x0, const double2* x1) const {
        Op<ND> op;
        op.load(U, tile, lane);
        op.fix(lane);
        accumulate<CURL>(y0, op, x0);
        accumulate<CURL>(y1, op, x1);
    }
    template <bool ODD>
    __device__ __forceinline__ void store(const Acc& y, double2* buf) const {
        if (!ok) return;
        double2* col = buf + off;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const bool f = (((kFoldX >> (4 * p + l)) & 1) != 0) != ODD;
            col[4 * p * L::RB] = flip_sign(make_double2(y.r[p], y.i[p]), f ? sx : 0u);
        }
    }
};

template <typename R, int N> struct TileOf;
template <int N> struct TileOf<float, N> { using type = Tile32<N>; };
template <int N> struct TileOf<double, N> { using type = Tile64<N>; };

// Products of the x pass: N (60 tensors), K (30), or the coupled J-M sums
//   s_j = N x_j + kj K x_m,  s_m = N x_m + km K x_j
// over the two halves of a vector pair (rows of the second pair of siblings)
enum XOp { X_N = 0, X_K = 1, X_JM = 2 };

// where the rows of one workgroup's item live: the two y siblings of one z
// sibling of an octant row, for one right-hand side (or both halves of one)
template <typename R>
struct XItem {
    bool valid;
    int row, ny_sib;
    unsigned mz;
    int sz;
    long long off, ystep, hstep;   // of row 0, from one y sibling or one half to the other

    __device__ __forceinline__ XItem(const P3Params& p, int q, int xcd, int halves) {
        // item -> (octant row, right-hand side, z sibling); the 2 nrhs items
        // of one operator row are dealt to one XCD and share its L2
        const int K = 2 * p.nrhs;
        row = (q / K) * 8 + xcd;
        const int kk = q - (q / K) * K, r = kk >> 1;
        sz = kk & 1;
        const int oz = row / p.Oy, oy = row - oz * p.Oy;
        ny_sib = (oy == 0 || 2 * oy == p.My) ? 1 : 2;
        valid = row < p.Oy * p.Oz && !(sz && (oz == 0 || 2 * oz == p.Mz));
        mz = sz ? kFoldZ : 0u;
        off = (long long)(halves * r) * p.s_r + (long long)(sz ? p.Mz - oz : oz) * p.s_z + (long long)oy * p.s_y;
        ystep = (long long)(p.My - 2 * oy) * p.s_y;
        hstep = p.s_r;
    }
    // row t = 24 h + 12 sy + c: offset, whether it exists, sign bit (odd: of
    // the outputs of an operator that itself changes sign under each fold)
    __device__ __forceinline__ long long at(int t, int s_c, bool odd, bool& ok, unsigned& sgn) const {
        const int g = t / 12, c = t - 12 * g, sy = g & 1, h = g >> 1;
        ok = sy < ny_sib;
        sgn = ((((mz ^ (sy ? kFoldY : 0u)) >> c) ^ (odd ? sy ^ sz : 0)) & 1u) << 31;
        return off + (sy ? ystep : 0) + (h ? hstep : 0) + c * s_c;
    }
};

// U: the 60 N tensors (X_N, X_JM) or the 30 curl tensors (X_K); UK: the curl
// tensors of X_JM
template <typename R, int N, int NW, int OP>
__global__ void __launch_bounds__(64 * NW, 3) k_p3_mx(C<R>* __restrict__ A, const C<R>* __restrict__ U,
                                                      const C<R>* __restrict__ UK, P3Params p,
                                                      const C<R>* __restrict__ tw, C<R> kj, C<R> km) {
    constexpr int H = OP == X_JM ? 2 : 1, RW = 24 * H / NW, OX = N / 2 + 1;
    static_assert(24 * H % NW == 0, "whole rows per wavefront");
    using T = typename TileOf<R, N>::type;
    using L = RowLayout<R, N>;
    extern __shared__ unsigned char smem_raw[];
    C<R>* buf = reinterpret_cast<C<R>*>(smem_raw);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = wave * RW, Nx = p.Nx, s_c = (int)p.s_c;
    const XItem<R> it(p, blockIdx.x >> 3, blockIdx.x & 7, H);
    if (!it.valid) return;   // uniform over the workgroup
    const C<R>* Ur = U + (long long)it.row * (OP == X_K ? 30 : 60) * OX;
    auto load = [&](int t, auto body) {
        bool ok;
        unsigned s;
        const C<R>* src = A + it.at(t, s_c, false, ok, s);
        body([=](int c) { return ok && c < Nx ? flip_sign(src[c], s) : mk<R>(0, 0); });
    };
    auto store = [&](int t, auto body) {
        bool ok;
        unsigned s;
        C<R>* dst = A + it.at(t, s_c, OP == X_K, ok, s);
        body([=](int c, C<R> v) { if (ok && c < Nx) dst[c] = flip_sign(v, s); });
    };
    RowInputs<R, N, RW> in;
    Twiddles<R, N> w;
    [[maybe_unused]] typename T::template Op<OP == X_K ? 3 : 6> op;
    in.fetch(t0, lane, load);
    row_pass<R, true, N, RW, 0>(buf, w, &in, t0, lane, store);
    w.fetch(tw, lane);
    if constexpr (!PassShape<N, 0>::LAST) row_passes<R, true, N, RW, 1>(buf, w, &in, t0, lane, store);
    if (OP != X_JM && wave < T::TILES) op.load(Ur, wave, lane);
    __syncthreads();
    for (int i = wave; i < T::TILES; i += NW) {
        const T tile(i, lane, it.ny_sib);
        if constexpr (OP == X_JM) {
            // K's sign under the folds of this column, into its factors
            const unsigned s = (((lane >> 1) ^ lane ^ it.sz) & 1u) << 31;
            typename T::Acc yj, ym;
            T::clear(yj);
            T::clear(ym);
            tile.template accumulate2<true, 3>(yj, ym, UK + (long long)it.row * 30 * OX, i, lane, buf + L::PAIR, buf);
            T::scale(yj, flip_sign(kj, s));
            T::scale(ym, flip_sign(km, s));
            tile.template accumulate2<false, 6>(yj, ym, Ur, i, lane, buf, buf + L::PAIR);
            tile.template store<false>(yj, buf);
            tile.template store<false>(ym, buf + L::PAIR);
        } else {
            typename T::Acc y;
            T::clear(y);
            op.fix(lane);
            tile.template accumulate<OP == X_K>(y, op, buf);
            tile.template store<OP == X_K>(y, buf);
            if (i + NW < T::TILES) op.load(Ur, i + NW, lane);
        }
    }
    __syncthreads();
    row_pass<R, false, N, RW, 0>(buf, w, &in, t0, lane, store);
    w.fetch(tw, lane);
    if constexpr (!PassShape<N, 0>::LAST) row_passes<R, false, N, RW, 1>(buf, w, &in, t0, lane, store);
}

// Wavefronts of a workgroup: 3 (8 rows each) or 4 (6 rows each), the count
// whose transforms leave the fewest lanes idle; the product's rounds are not
// counted.  us in complex64 with 3 / 4 wavefronts (N / 2 x 64 x 64, one vector),
// the choice first: 64 65 / 71, 72 74 / 83, 96 95 / 102, 128 104 / 121, 144 139 /
// 163, 180 192 / 233, 192 205 / 247; 4 at 90 84 (95), 100 99 (112), 108 111 (116),
// 120 112 (115), 150 165 (166).  It misses 80 (4: 79, 3: 77) and 160 (4: 194, 3:
// 174), and where LDS holds few workgroups (N / 2 x 48 x 48): 320 288 / 252, 384
// 320 / 285, 512 655 / 557, with 6 wavefronts 469.  From 160 up in complex128
// LDS leaves so few that 6 are taken (192: 966 us against 1137 at 96^3); below,
// they lose (64^3 262 us to 207).
template <int N, int NW, int S>
constexpr int lane_rounds() {
    if constexpr (S < 3 && PassShape<N, S < 3 ? S : 0>::RAD > 0) {
        using P = PassMap<N, 24 / NW, S>;
        return NW * P::ROUNDS * P::RAD + (PassShape<N, S>::LAST ? 0 : lane_rounds<N, NW, S + 1>());
    } else {
        return 0;
    }
}
template <typename R, int N>
constexpr int p3_mx_waves() {
    if (sizeof(R) == 8 && N >= 160) return 6;
    return lane_rounds<N, 4, 0>() < lane_rounds<N, 3, 0>() ? 4 : 3;
}

// The J-M pass keeps 48 rows, so that fewer workgroups fit: 4 wavefronts (12
// rows each), more in complex128 where LDS holds one or two workgroups (64^3:
// 360 us with 4 against 553 with 6 in complex64; complex128 48^3 263 with 4
// against 216 with 8, 72 x 61 x 85 1468 against 868 with 12).
template <typename R, int N>
constexpr int p3_mx_jm_waves() {
    return sizeof(R) == 4 || N <= 64 ? 4 : N <= 100 ? 8 : 12;
}

template <typename R, int N> constexpr size_t p3_mx_lds(int halves = 1) {
    return (size_t)halves * RowLayout<R, N>::PAIR * sizeof(C<R>);
}

template <typename R, int N, int OP, int NW = OP == X_JM ? p3_mx_jm_waves<R, N>() : p3_mx_waves<R, N>()>
void launch_p3_mx_n(C<R>* A, const C<R>* U, const C<R>* UK, const P3Params& p, const C<R>* tw, C<R> kj, C<R> km,
                    hipStream_t s) {
    const size_t lds = p3_mx_lds<R, N>(OP == X_JM ? 2 : 1);
    const long long nblk = ((long long)p.Oy * p.Oz + 7) / 8 * 8 * 2LL * p.nrhs;
    VIE_REQUIRE(nblk < (1LL << 31), VIE_EINVAL, "x pass: too many workgroups");
    static std::once_flag once;
    std::call_once(once, [&] {
        (void)hipFuncSetAttribute((const void*)k_p3_mx<R, N, NW, OP>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        (void)hipGetLastError();
    });
    timed_launch(k_p3_mx<R, N, NW, OP>, dim3((unsigned)nblk), dim3(64 * NW), (unsigned)lds, s, A, U, UK, p, tw, kj,
                 km);
    VIE_HIP(hipGetLastError());
}

}  // namespace vie
