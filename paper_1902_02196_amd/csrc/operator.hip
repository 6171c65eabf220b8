// Operator set-up (Sec. III-C, IV-A): assembly of the 60 unique
// Toeplitz-defining block tensors on the device, circulant embedding with the
// reflection signs of the PWL bases, forward FFT, octant extraction.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "assembly.hpp"
#include "fft.hpp"
#include "kernels.hpp"
#include "vie.h"

namespace vie {

// ---------------------------------------------------------------------------
// host: axis kernels in closed form
// ---------------------------------------------------------------------------
// measure kinds: 0 '1', 1 't/D', 2 'D(1)', 3 'D(t/D)'
static AxisKernel axis_kernel(int kt, int kb, double D) {
    AxisKernel k{};
    auto set = [&](double* c, double a0, double a1, double a2, double a3) { c[0] = a0; c[1] = a1; c[2] = a2; c[3] = a3; };
    const double D2 = D * D;
    switch (kt * 4 + kb) {
        case 0:  // (1,1): D - |w|
            set(k.left, D, 1, 0, 0); set(k.right, D, -1, 0, 0); break;
        case 4:  // (t,1): w (D - |w|) / (2D)
            set(k.left, 0, 0.5, 0.5 / D, 0); set(k.right, 0, 0.5, -0.5 / D, 0); break;
        case 1:  // (1,t): -w (D - |w|) / (2D)
            set(k.left, 0, -0.5, -0.5 / D, 0); set(k.right, 0, -0.5, 0.5 / D, 0); break;
        case 5:  // (t,t): (D^3 - 3 D^2 |w| + 2 |w|^3) / (12 D^2)
            set(k.left, D / 12, 0.25, 0, -1.0 / (6 * D2)); set(k.right, D / 12, -0.25, 0, 1.0 / (6 * D2)); break;
        case 8:  // (D1,1): +1 left, -1 right
            set(k.left, 1, 0, 0, 0); set(k.right, -1, 0, 0, 0); break;
        case 9:  // (D1,t)
            set(k.left, -0.5, -1 / D, 0, 0); set(k.right, -0.5, 1 / D, 0, 0); break;
        case 2:  // (1,D1)
            set(k.left, -1, 0, 0, 0); set(k.right, 1, 0, 0, 0); break;
        case 6:  // (t,D1)
            set(k.left, -0.5, -1 / D, 0, 0); set(k.right, -0.5, 1 / D, 0, 0); break;
        case 10:  // (D1,D1): 2 delta_0 - delta_{-D} - delta_{D}
            k.pts[0] = -1; k.pts[1] = 2; k.pts[2] = -1; break;
        case 12:  // (Dt,1): 1/2 - |w|/D
            set(k.left, 0.5, 1 / D, 0, 0); set(k.right, 0.5, -1 / D, 0, 0); break;
        case 3:  // (1,Dt)
            set(k.left, 0.5, 1 / D, 0, 0); set(k.right, 0.5, -1 / D, 0, 0); break;
        case 13:  // (Dt,t)
            set(k.left, 0.25, 0, -0.5 / D2, 0); set(k.right, -0.25, 0, 0.5 / D2, 0); break;
        case 7:  // (t,Dt)
            set(k.left, -0.25, 0, 0.5 / D2, 0); set(k.right, 0.25, 0, -0.5 / D2, 0); break;
        case 11:  // (D1,Dt)
            set(k.left, 1 / D, 0, 0, 0); set(k.right, -1 / D, 0, 0, 0); k.pts[0] = -0.5; k.pts[2] = 0.5; break;
        case 14:  // (Dt,D1)
            set(k.left, -1 / D, 0, 0, 0); set(k.right, 1 / D, 0, 0, 0); k.pts[0] = 0.5; k.pts[2] = -0.5; break;
        case 15:  // (Dt,Dt): -|w|/D^2, 1/4 delta_{-D} + 1/2 delta_0 + 1/4 delta_D
            set(k.left, 0, 1 / D2, 0, 0); set(k.right, 0, -1 / D2, 0, 0);
            k.pts[0] = 0.25; k.pts[1] = 0.5; k.pts[2] = 0.25; break;
    }
    return k;
}

static void gauss_legendre01(int n, double* x, double* w) {
    // roots of P_n by Newton from the usual cosine guesses, weights
    // 2 / ((1 - z^2) P_n'(z)^2); mapped from [-1, 1] to [0, 1]
    for (int i = 0; i < n; ++i) {
        double z = std::cos(M_PI * (i + 0.75) / (n + 0.5)), pp = 1.0;
        for (int it = 0; it < 100; ++it) {
            double p1 = 1.0, p2 = 0.0;
            for (int j = 1; j <= n; ++j) {
                const double p3 = p2;
                p2 = p1;
                p1 = ((2.0 * j - 1.0) * z * p2 - (j - 1.0) * p3) / j;
            }
            pp = n * (z * p1 - p2) / (z * z - 1.0);
            const double dz = p1 / pp;
            z -= dz;
            if (std::fabs(dz) < 1e-15) {
                // refresh the derivative at the converged root
                p1 = 1.0; p2 = 0.0;
                for (int j = 1; j <= n; ++j) {
                    const double p3 = p2;
                    p2 = p1;
                    p1 = ((2.0 * j - 1.0) * z * p2 - (j - 1.0) * p3) / j;
                }
                pp = n * (z * p1 - p2) / (z * z - 1.0);
                break;
            }
        }
        x[i] = 0.5 * (1.0 - z);
        w[i] = 1.0 / ((1.0 - z * z) * pp * pp);
    }
}

AssemblyTables build_assembly_tables(const double D[3], double k0) {
    AssemblyTables T{};
    for (int ax = 0; ax < 3; ++ax)
        for (int kt = 0; kt < 4; ++kt)
            for (int kb = 0; kb < 4; ++kb) T.ker[ax * 16 + kt * 4 + kb] = axis_kernel(kt, kb, D[ax]);
    const double dv = D[0] * D[1] * D[2];
    T.gram[0] = dv;
    T.gram[1] = T.gram[2] = T.gram[3] = dv / 12;
    for (int pq = 0; pq < 6; ++pq) {
        static const int P[6] = {0, 0, 0, 1, 1, 2}, Q[6] = {0, 1, 2, 1, 2, 2};
        static const int L[10] = {1, 1, 1, 1, 2, 2, 2, 3, 3, 4}, LP[10] = {1, 2, 3, 4, 2, 3, 4, 3, 4, 4};
        for (int ll = 0; ll < 10; ++ll) {
            const int p = P[pq], q = Q[pq], l = L[ll], lp = LP[ll];
            EntryTerms& e = T.ent[pq * 10 + ll];
            e.nterm = 0;
            int kt[3], kb[3];
            for (int ax = 0; ax < 3; ++ax) {
                kt[ax] = (l == ax + 2) ? 1 : 0;
                kb[ax] = (lp == ax + 2) ? 1 : 0;
            }
            if (p == q && k0 != 0.0) {
                e.coef[e.nterm] = k0 * k0;
                for (int ax = 0; ax < 3; ++ax) e.ker[e.nterm][ax] = ax * 16 + kt[ax] * 4 + kb[ax];
                e.nterm++;
            }
            int ct[3] = {kt[0], kt[1], kt[2]}, cb[3] = {kb[0], kb[1], kb[2]};
            ct[p] += 2;
            cb[q] += 2;
            e.coef[e.nterm] = -1.0;
            for (int ax = 0; ax < 3; ++ax) e.ker[e.nterm][ax] = ax * 16 + ct[ax] * 4 + cb[ax];
            e.nterm++;
            e.gram_l = (p == q && l == lp) ? l - 1 : -1;
        }
    }
    for (int n = 1; n <= kMaxGauss; ++n) gauss_legendre01(n, T.gl_x[n], T.gl_w[n]);
    T.D[0] = D[0]; T.D[1] = D[1]; T.D[2] = D[2];
    T.k0 = k0;
    T.order_near = 14;
    T.order_duffy = 12;
    T.nent = 60;
    return T;
}

// the 30 unique tensors of the curl operator: entry 10 k + ll is
// Q_k^{ll'}(d) = <N^l, S D_k N^{l'}> (l <= l'), one term, no Gram part
AssemblyTables build_curl_tables(const double D[3], double k0) {
    AssemblyTables T = build_assembly_tables(D, k0);
    static const int L[10] = {1, 1, 1, 1, 2, 2, 2, 3, 3, 4}, LP[10] = {1, 2, 3, 4, 2, 3, 4, 3, 4, 4};
    for (int k = 0; k < 3; ++k)
        for (int ll = 0; ll < 10; ++ll) {
            EntryTerms& e = T.ent[10 * k + ll];
            e.nterm = 1;
            e.coef[0] = 1.0;
            for (int ax = 0; ax < 3; ++ax) {
                const int kt = (L[ll] == ax + 2) ? 1 : 0;
                const int kb = ((LP[ll] == ax + 2) ? 1 : 0) + (ax == k ? 2 : 0);
                e.ker[0][ax] = ax * 16 + kt * 4 + kb;
            }
            e.gram_l = -1;
        }
    T.nent = 30;
    return T;
}

// ---------------------------------------------------------------------------
// device: integration
// ---------------------------------------------------------------------------
__host__ __device__ __forceinline__ double horner(const double* c, double w) { return ((c[3] * w + c[2]) * w + c[1]) * w + c[0]; }

// slot: 0 = density on [-D,0], 1 = density on [0,D], 2/3/4 = point at -D/0/+D
__host__ __device__ __forceinline__ bool slot_used(const AxisKernel& k, int slot) {
    if (slot == 0) return k.left[0] != 0 || k.left[1] != 0 || k.left[2] != 0 || k.left[3] != 0;
    if (slot == 1) return k.right[0] != 0 || k.right[1] != 0 || k.right[2] != 0 || k.right[3] != 0;
    return k.pts[slot - 2] != 0;
}

__host__ __device__ __forceinline__ double slot_value(const AxisKernel& k, int slot, double w) {
    if (slot == 0) return horner(k.left, w);
    if (slot == 1) return horner(k.right, w);
    return k.pts[slot - 2];
}

__host__ __device__ __forceinline__ double2 green(double r, double k0) {
    double s, c;
    sincos(k0 * r, &s, &c);
    const double a = 1.0 / (4.0 * M_PI * r);
    return make_double2(c * a, -s * a);
}

// Work item tid's share (points tid, tid + nthr, ...) of the quadrature of
// one geometry: a density or point-mass slot per axis at offset d.
__device__ double2 integrate_geometry(const AssemblyTables& T, const AxisKernel* kx[3], const int slot[3],
                                      const int d[3], int order_far, int tid, int nthr) {
    const double* D = T.D;
    // singular corner: w* = -d Delta, touching when each axis reaches it
    bool touch = true;
    for (int i = 0; i < 3; ++i) {
        const int s = slot[i];
        bool ti;
        if (s == 0) ti = (d[i] == 0 || d[i] == 1);
        else if (s == 1) ti = (d[i] == 0);
        else if (s == 2) ti = (d[i] == 1);
        else if (s == 3) ti = (d[i] == 0);
        else ti = (d[i] == -1);
        touch = touch && ti;
    }
    int dens[3], nd = 0, pt_axis = -1;
    for (int i = 0; i < 3; ++i) {
        if (slot[i] <= 1) dens[nd++] = i;
        else pt_axis = i;
    }
    double off[3] = {d[0] * D[0], d[1] * D[1], d[2] * D[2]};
    double base[3], wfix = 1.0;
    if (pt_axis >= 0) {
        base[pt_axis] = (slot[pt_axis] - 3) * D[pt_axis];
        wfix = kx[pt_axis]->pts[slot[pt_axis] - 2];
    }
    double2 acc = make_double2(0, 0);
    if (!touch) {
        const int n = order_far;
        const double* gx = T.gl_x[n];
        const double* gw = T.gl_w[n];
        double lo[3];
        for (int i = 0; i < 3; ++i) lo[i] = (slot[i] == 0) ? -D[i] : 0.0;
        if (nd == 3) {
            for (int q = tid; q < n * n * n; q += nthr) {
                const int a = q / (n * n), b = (q / n) % n, c = q % n;
                const double wx = lo[0] + D[0] * gx[a];
                const double fx = slot_value(*kx[0], slot[0], wx) * gw[a] * D[0];
                const double rx = off[0] + wx;
                const double wy = lo[1] + D[1] * gx[b];
                const double fy = fx * slot_value(*kx[1], slot[1], wy) * gw[b] * D[1];
                const double ry = off[1] + wy;
                const double wz = lo[2] + D[2] * gx[c];
                const double f = fy * slot_value(*kx[2], slot[2], wz) * gw[c] * D[2];
                const double rz = off[2] + wz;
                const double2 g = green(sqrt(rx * rx + ry * ry + rz * rz), T.k0);
                acc.x += f * g.x;
                acc.y += f * g.y;
            }
        } else {
            const int i0 = dens[0], i1 = dens[1];
            const double rp = off[pt_axis] + base[pt_axis];
            for (int q = tid; q < n * n; q += nthr) {
                const int a = q / n, b = q % n;
                const double w0 = lo[i0] + D[i0] * gx[a];
                const double f0 = slot_value(*kx[i0], slot[i0], w0) * gw[a] * D[i0] * wfix;
                const double r0 = off[i0] + w0;
                const double w1 = lo[i1] + D[i1] * gx[b];
                const double f = f0 * slot_value(*kx[i1], slot[i1], w1) * gw[b] * D[i1];
                const double r1 = off[i1] + w1;
                const double2 g = green(sqrt(r0 * r0 + r1 * r1 + rp * rp), T.k0);
                acc.x += f * g.x;
                acc.y += f * g.y;
            }
        }
        return acc;
    }
    // Duffy: the singular point is a corner of the box.  Map the box to the
    // unit cube (square) with that corner at the origin and split it into
    // pyramids (triangles) with apex there: on the piece whose far face is
    // xi_k = 1, xi_k = s and xi_j = s t_j, Jacobian s^(dim-1).
    const int n = T.order_duffy;
    const double* gx = T.gl_x[n];
    const double* gw = T.gl_w[n];
    double corner[3], ext[3];
    for (int i = 0; i < 3; ++i) {
        corner[i] = -off[i];                     // w* = -d Delta
        if (slot[i] <= 1) {
            const double lo = (slot[i] == 0) ? -D[i] : 0.0;
            ext[i] = (corner[i] == lo) ? D[i] : -D[i];
        }
    }
    if (nd == 3) {
        const double jac0 = D[0] * D[1] * D[2];
        for (int k = 0; k < 3; ++k) {
            for (int q = tid; q < n * n * n; q += nthr) {
                const int a = q / (n * n), b = (q / n) % n, c = q % n;
                const double s = gx[a], st1 = s * gx[b], st2 = s * gx[c];
                double rr = 0, f = gw[a] * gw[b] * gw[c] * s * s * jac0;
                for (int i = 0; i < 3; ++i) {
                    // xi_k = s, the next axis s t1, the one after s t2
                    const double xi = i == k ? s : (i == (k + 1) % 3 ? st1 : st2);
                    const double w = corner[i] + ext[i] * xi;
                    const double ri = off[i] + w;
                    rr += ri * ri;
                    f *= slot_value(*kx[i], slot[i], w);
                }
                const double2 g = green(sqrt(rr), T.k0);
                acc.x += f * g.x;
                acc.y += f * g.y;
            }
        }
    } else {
        const int i0 = dens[0], i1 = dens[1];
        const double jac0 = D[i0] * D[i1] * wfix;
        for (int k = 0; k < 2; ++k) {
            for (int q = tid; q < n * n; q += nthr) {
                const int a = q / n, b = q % n;
                const double s = gx[a], t = gx[b];
                const double xi0 = (k == 0) ? s : s * t;
                const double xi1 = (k == 0) ? s * t : s;
                const double w0 = corner[i0] + ext[i0] * xi0;
                const double w1 = corner[i1] + ext[i1] * xi1;
                const double r0 = off[i0] + w0, r1 = off[i1] + w1;
                const double f = gw[a] * gw[b] * s * jac0 * slot_value(*kx[i0], slot[i0], w0) *
                                 slot_value(*kx[i1], slot[i1], w1);
                const double2 g = green(sqrt(r0 * r0 + r1 * r1), T.k0);
                acc.x += f * g.x;
                acc.y += f * g.y;
            }
        }
    }
    return acc;
}

__host__ __device__ __forceinline__ int far_order(int dinf, int near) {
    if (dinf <= 2) return near;
    if (dinf <= 4) return 9;
    if (dinf <= 8) return 7;
    if (dinf <= 16) return 5;
    return 4;
}

// Gauss order bands of far_order for offsets beyond the singular corner
static const int kBandLo[kFarBands] = {2, 3, 5, 9, 17};
static const int kBandHi[kFarBands] = {2, 4, 8, 16, 1 << 30};

FarTables build_far_tables(const AssemblyTables& T) {
    FarTables F{};
    for (int b = 0; b < kFarBands; ++b) {
        FarBand& B = F.band[b];
        B.dlo = kBandLo[b];
        B.dhi = kBandHi[b];
        B.n = far_order(B.dlo, T.order_near);
        B.P = 2 * B.n + 3;
        const double* gx = T.gl_x[B.n];
        const double* gw = T.gl_w[B.n];
        for (int i = 0; i < B.P; ++i) B.ispt[i] = i >= 2 * B.n;
        for (int ax = 0; ax < 3; ++ax) {
            const double D = T.D[ax];
            for (int a = 0; a < B.n; ++a) {
                B.w[ax][a] = -D + D * gx[a];
                B.w[ax][B.n + a] = D * gx[a];
            }
            for (int m = 0; m < 3; ++m) B.w[ax][2 * B.n + m] = (m - 1) * D;
            for (int k = 0; k < 16; ++k) {
                const AxisKernel& K = T.ker[ax * 16 + k];
                for (int a = 0; a < B.n; ++a) {
                    B.W[ax][k][a] = horner(K.left, B.w[ax][a]) * gw[a] * D;
                    B.W[ax][k][B.n + a] = horner(K.right, B.w[ax][B.n + a]) * gw[a] * D;
                }
                for (int m = 0; m < 3; ++m) B.W[ax][k][2 * B.n + m] = K.pts[m];
            }
        }
    }
    F.nterm = 0;
    F.npair = 0;
    F.nent = T.nent;
    for (int e = 0; e < T.nent; ++e) {
        const EntryTerms& E = T.ent[e];
        F.ent_first[e] = F.nterm;
        F.ent_count[e] = E.nterm;
        for (int t = 0; t < E.nterm; ++t) {
            const int ky = E.ker[t][1] % 16, kz = E.ker[t][2] % 16;
            int p = 0;
            while (p < F.npair && !(F.pair_ky[p] == ky && F.pair_kz[p] == kz)) ++p;
            if (p == F.npair) {
                F.pair_ky[p] = ky;
                F.pair_kz[p] = kz;
                ++F.npair;
            }
            F.term_kx[F.nterm] = E.ker[t][0] % 16;
            F.term_pair[F.nterm] = p;
            F.term_coef[F.nterm] = E.coef[t];
            ++F.nterm;
        }
    }
    return F;
}

// Weights and points of one lane, fixed for the launch: of its z kernel (tid %
// 16), of its (ky, kz) pair, and the points (y, z) of a slab it evaluates
// with how many of the two are point values (2 bits each).
template <int P>
struct FarLane {
    static constexpr int RG = (P * P + 63) / 64;
    static_assert(RG <= 16, "flags of a lane in 32 bits");
    double wz[P], wy[P], gy[RG], gz[RG], ryz[RG];
    unsigned npt = 0;
    int tid, kzp;

    __device__ __forceinline__ FarLane(const FarTables& F, const FarBand& B, int lane) : tid(lane) {
        const int kz = tid & 15, p = min(tid, F.npair - 1), ky = F.pair_ky[p];
        kzp = F.pair_kz[p];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            wz[k] = B.W[2][kz][k];
            wy[k] = B.W[1][ky][k];
        }
#pragma unroll
        for (int u = 0; u < RG; ++u) {
            const int idx = min(tid + 64 * u, P * P - 1), j = idx / P, k = idx - j * P;
            gy[u] = B.w[1][j];
            gz[u] = B.w[2][k];
            npt |= (unsigned)(B.ispt[j] + B.ispt[k]) << (2 * u);
        }
    }
    // squared distances in y and z at offset (y0, z0)
    __device__ __forceinline__ void place(double y0, double z0) {
#pragma unroll
        for (int u = 0; u < RG; ++u) {
            const double ry = y0 + gy[u], rz = z0 + gz[u];
            ryz[u] = ry * ry + rz * rz;
        }
    }
    // the (y, z) slab of Green's values at x distance rx; pi: 1 at a point value of x
    __device__ __forceinline__ void slab(double2* g, double rx, int pi, double k0) const {
#pragma unroll
        for (int u = 0; u < RG; ++u) {
            const int idx = tid + 64 * u;
            if (idx < P * P)
                g[idx] = pi + (int)((npt >> (2 * u)) & 3) <= 1 ? green(sqrt(rx * rx + ryz[u]), k0)
                                                                : make_double2(0, 0);
        }
    }
    // z contraction of a slab for the 16 kernels
    __device__ __forceinline__ void contract_z(double2* t1, const double2* g) const {
        for (int idx = tid; idx < P * 16; idx += 64) {
            const int j = idx >> 4;   // kernel idx % 16 = tid % 16
            double2 a = make_double2(0, 0);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double2 v = g[j * P + k];
                a.x += wz[k] * v.x;
                a.y += wz[k] * v.y;
            }
            t1[idx] = a;
        }
    }
    // y contraction for the (ky, kz) pairs in use
    __device__ __forceinline__ void contract_y(double2* t2, const double2* t1, const FarTables& F,
                                               const FarBand& B) const {
        if (tid < F.npair) {
            double2 a = make_double2(0, 0);
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const double2 u = t1[j * 16 + kzp];
                a.x += wy[j] * u.x;
                a.y += wy[j] * u.y;
            }
            t2[tid] = a;
        }
        for (int p = tid + 64; p < F.npair; p += 64) {
            const double* w2 = B.W[1][F.pair_ky[p]];
            const int kz = F.pair_kz[p];
            double2 a = make_double2(0, 0);
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const double2 u = t1[j * 16 + kz];
                a.x += w2[j] * u.x;
                a.y += w2[j] * u.y;
            }
            t2[p] = a;
        }
    }
};

// Near bands: one workgroup of W wavefronts per offset (grid-stride over the
// offsets of the cube that holds the band, those below the band skipped);
// wavefront w takes the x abscissae w, w + W, ...  Per x abscissa: the (y, z)
// slab of Green's values, the z contraction for all 16 kernel pairs, the y
// contraction for the (ky, kz) pairs in use, and the x accumulation of every
// (entry, term) sum; the wavefronts' sums are added in order at the end.
// W = 4: 19, 98 and 604 offsets leave most of the chip idle and wait on one
// wavefront's serial chain (214, 80 and 46 us; one wavefront each 576,
// 326 and 199).
template <int P, int W>
__global__ void __launch_bounds__(64 * W) k_assemble_far(double2* __restrict__ out, const FarTables* __restrict__ Fg,
                                                         int b, double Dx, double Dy, double Dz, double k0, int Nx,
                                                         int Ny, int Nz, int cx, int cy, int cz) {
    __shared__ double2 slab_[W][P * P];
    __shared__ double2 t1_[W][P * 16];
    __shared__ double2 t2_[W][kFarTerms];
    const FarTables& F = *Fg;
    const FarBand& B = F.band[b];
    const int tid = threadIdx.x & 63, w = threadIdx.x >> 6;
    double2* slab = slab_[w];
    double2* t1 = t1_[w];
    double2* t2 = t2_[w];
    const long long V = (long long)Nx * Ny * Nz;
    const int nterm = F.nterm;
    FarLane<P> lane(F, B, tid);
    // offsets of the band lie in the cube [0, cx) x [0, cy) x [0, cz)
    const long long ncube = (long long)cx * cy * cz;
    for (long long q = blockIdx.x; q < ncube; q += gridDim.x) {
        const int d0 = int(q % cx), d1 = int((q / cx) % cy), d2 = int(q / ((long long)cx * cy));
        const long long v = ((long long)d2 * Ny + d1) * Nx + d0;
        const int dinf = max(d0, max(d1, d2));
        if (dinf < B.dlo || dinf > B.dhi) continue;   // uniform over the workgroup
        lane.place(d1 * Dy, d2 * Dz);
        double2 s0 = make_double2(0, 0), s1 = make_double2(0, 0);   // terms tid, tid + 64
        // every wavefront runs every round (barriers); one past the last
        // abscissa has nothing to add
        for (int i0 = 0; i0 < P; i0 += W) {
            const int i = i0 + w;
            const bool act = i < P;
            if (act) lane.slab(slab, d0 * Dx + B.w[0][i], B.ispt[i], k0);
            __syncthreads();
            if (act) lane.contract_z(t1, slab);
            __syncthreads();
            if (act) lane.contract_y(t2, t1, F, B);
            __syncthreads();
            if (act && tid < nterm) {
                const double wx = B.W[0][F.term_kx[tid]][i];
                const double2 u = t2[F.term_pair[tid]];
                s0.x += wx * u.x;
                s0.y += wx * u.y;
            }
            if (act && tid + 64 < nterm) {
                const double wx = B.W[0][F.term_kx[tid + 64]][i];
                const double2 u = t2[F.term_pair[tid + 64]];
                s1.x += wx * u.x;
                s1.y += wx * u.y;
            }
            __syncthreads();
        }
        // combine the terms of each entry (t2 reused for the term sums)
        if (tid < nterm) t2[tid] = s0;
        if (tid + 64 < nterm) t2[tid + 64] = s1;
        __syncthreads();
        if (w == 0 && tid < F.nent) {
            double2 a = make_double2(0, 0);
            for (int t = F.ent_first[tid]; t < F.ent_first[tid] + F.ent_count[tid]; ++t)
                for (int u = 0; u < W; ++u) {
                    a.x += F.term_coef[t] * t2_[u][t].x;
                    a.y += F.term_coef[t] * t2_[u][t].y;
                }
            out[(long long)tid * V + v] = a;
        }
        __syncthreads();
    }
}

// Far bands: one wavefront per run of up to T offsets along x.  Neighbouring
// offsets share their x abscissae, the Gauss points of the cell between two of
// them and the lattice points, so each plane x = const is evaluated and
// contracted in y and z once and added to the two (cell) or three (lattice)
// offsets it belongs to: n + 1 planes per offset of a long run instead of
// 2 n + 3.  Bound by the FP64 Green's function (sqrt, sincos, division) of a
// plane's points: 1.39 ms at 48^3 with all planes per offset and the weights
// reloaded each time, 1.06 with the weights in registers, 0.59 so (64^3: 2.6 ->
// 1.35).
template <int P>
__global__ void __launch_bounds__(64) k_assemble_far_rows(double2* __restrict__ out,
                                                          const FarTables* __restrict__ Fg, int b, double Dx,
                                                          double Dy, double Dz, double k0, int Nx, int Ny, int Nz,
                                                          int cx, int cy, int cz, int T) {
    constexpr int n = (P - 3) / 2;
    __shared__ double2 slab[P * P];
    __shared__ double2 t1[P * 16];
    __shared__ double2 t2[kFarTerms];
    __shared__ double wx[16 * P];
    const FarTables& F = *Fg;
    const FarBand& B = F.band[b];
    const int tid = threadIdx.x;
    const long long V = (long long)Nx * Ny * Nz;
    const int nterm = F.nterm;
    FarLane<P> lane(F, B, tid);
    for (int idx = tid; idx < 16 * P; idx += 64) wx[idx] = B.W[0][idx / P][idx % P];
    const double* wt[2];
    int pr[2];
    bool has[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {   // terms tid, tid + 64
        const int t = min(tid + 64 * h, nterm - 1);
        has[h] = tid + 64 * h < nterm;
        wt[h] = wx + F.term_kx[t] * P;
        pr[h] = F.term_pair[t];
    }
    const int nch = (cx + T - 1) / T;
    const long long nrun = (long long)nch * cy * cz;
    for (long long q = blockIdx.x; q < nrun; q += gridDim.x) {
        const int ch = int(q % nch), d1 = int((q / nch) % cy), d2 = int(q / ((long long)nch * cy));
        // the band's offsets of a row: all of it, or those from dlo on
        const int x0 = (max(d1, d2) >= B.dlo ? 0 : B.dlo) + ch * T, x1 = min(x0 + T, cx);
        if (x0 >= x1) continue;   // uniform over the workgroup
        lane.place(d1 * Dy, d2 * Dz);
        double2 s[3][2];   // sums of the offsets c - 1, c, c + 1
#pragma unroll
        for (int k = 0; k < 3; ++k) s[k][0] = s[k][1] = make_double2(0, 0);
        for (int c = x0 - 1; c <= x1; ++c) {
            // the lattice plane x = c, then the Gauss planes of the cell [c, c + 1]
            for (int a = -1; a < (c < x1 ? n : 0); ++a) {
                lane.slab(slab, c * Dx + (a < 0 ? 0.0 : B.w[0][n + a]), a < 0, k0);
                __syncthreads();
                lane.contract_z(t1, slab);
                __syncthreads();
                lane.contract_y(t2, t1, F, B);
                __syncthreads();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double2 u = t2[pr[h]];
                    auto add = [&](double2& acc, double w) {
                        acc.x += w * u.x;
                        acc.y += w * u.y;
                    };
                    if (a < 0) {
                        add(s[0][h], wt[h][2 * n + 2]);
                        add(s[1][h], wt[h][2 * n + 1]);
                        add(s[2][h], wt[h][2 * n]);
                    } else {
                        add(s[1][h], wt[h][n + a]);
                        add(s[2][h], wt[h][a]);
                    }
                }
                __syncthreads();
                if (a < 0 && c > x0) {   // offset c - 1 is complete: combine the terms of each entry
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (has[h]) t2[tid + 64 * h] = s[0][h];
                    __syncthreads();
                    if (tid < F.nent) {
                        double2 r = make_double2(0, 0);
                        for (int t = F.ent_first[tid]; t < F.ent_first[tid] + F.ent_count[tid]; ++t) {
                            r.x += F.term_coef[t] * t2[t].x;
                            r.y += F.term_coef[t] * t2[t].y;
                        }
                        out[(long long)tid * V + ((long long)d2 * Ny + d1) * Nx + (c - 1)] = r;
                    }
                    __syncthreads();
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s[0][h] = s[1][h];
                s[1][h] = s[2][h];
                s[2][h] = make_double2(0, 0);
            }
        }
    }
}

// Entry-by-entry assembly of the offsets at the singular corner, d in
// {0, 1}^3 (those may touch the singular point; Duffy rules): one workgroup
// per (entry, offset), the quadrature points of every geometry dealt to its
// work items and their partial sums added in a fixed order.  Bound by the
// FP64 Green's function (sqrt, sincos) of up to 40k points per entry and
// offset: 0.36 ms on any grid; one work item per (entry, offset) ran the
// points in series for 75 ms, most of a 64^3 set-up.
constexpr int kNearThreads = 256;

__global__ void __launch_bounds__(kNearThreads) k_assemble_near(double2* __restrict__ out,
                                                                const AssemblyTables* __restrict__ Tg, int Nx, int Ny,
                                                                int Nz) {
    const AssemblyTables& T = *Tg;
    const long long V = (long long)Nx * Ny * Nz;
    const int e = blockIdx.x, c = blockIdx.y, tid = threadIdx.x;
    const int d[3] = {c & 1, (c >> 1) & 1, c >> 2};
    if (d[0] >= Nx || d[1] >= Ny || d[2] >= Nz) return;   // uniform over the workgroup
    const int nfar = far_order(max(d[0], max(d[1], d[2])), T.order_near);
    const EntryTerms& E = T.ent[e];
    double2 acc = make_double2(0, 0);
    for (int t = 0; t < E.nterm; ++t) {
        const AxisKernel* kx[3] = {&T.ker[E.ker[t][0]], &T.ker[E.ker[t][1]], &T.ker[E.ker[t][2]]};
        double2 part = make_double2(0, 0);
        int slot[3];
        for (slot[0] = 0; slot[0] < 5; ++slot[0]) {
            if (!slot_used(*kx[0], slot[0])) continue;
            for (slot[1] = 0; slot[1] < 5; ++slot[1]) {
                if (!slot_used(*kx[1], slot[1])) continue;
                for (slot[2] = 0; slot[2] < 5; ++slot[2]) {
                    if (!slot_used(*kx[2], slot[2])) continue;
                    const int npt = (slot[0] >= 2) + (slot[1] >= 2) + (slot[2] >= 2);
                    if (npt > 1) continue;  // does not occur for these measures
                    const double2 g = integrate_geometry(T, kx, slot, d, nfar, tid, kNearThreads);
                    part.x += g.x;
                    part.y += g.y;
                }
            }
        }
        acc.x += E.coef[t] * part.x;
        acc.y += E.coef[t] * part.y;
    }
    __shared__ double2 sum[kNearThreads];
    sum[tid] = acc;
    __syncthreads();
    for (int h = kNearThreads / 2; h > 0; h /= 2) {
        if (tid < h) {
            sum[tid].x += sum[tid + h].x;
            sum[tid].y += sum[tid + h].y;
        }
        __syncthreads();
    }
    if (tid == 0) {
        double2 v = sum[0];
        if (c == 0 && E.gram_l >= 0) v.x += T.gram[E.gram_l];
        out[(long long)e * V + ((long long)d[2] * Ny + d[1]) * Nx + d[0]] = v;
    }
}

// One axis of the operator spectra (Sec. IV-A): every pencil of the N
// offsets d >= 0 along the axis is extended to the circulant of length M in
// LDS (index j -> offset j for j < N, M - j with the entry's reflection sign
// for j > M - N, otherwise zero), transformed, and only its octant half
// xi <= M / 2 is kept, since C^(M - xi) = sign C^(xi).  With the mirror taken
// per axis the three passes move 60 V values each way instead of 60 full
// circulants of 8 V, and the entries of a chunk share one launch: 0.67 ms at
// 48^3 in 27 launches, against 3.6 ms for the whole circulants in 300.
//
// Pencil (e, o, t): element k at in + e in_e + o in_o + k in_k + t; ROWS:
// the pencils are contiguous rows (t counts rows, in_k = 1) and row t of
// entry e goes to U[(t nent + e0 + e)][O].  Bound by LDS latency: two ping-pong
// buffers of `tile` pencils per workgroup, the run-time radix plan.
struct SpecPass {
    FftPlan plan;
    int N, O;              // input offsets, kept outputs
    int tile, pitch;       // pencils per workgroup, LDS pitch
    int n_inner;           // extent of t
    long long in_e, in_o, in_k, out_e, out_o, out_k;
    unsigned long long neg;   // bit e set: the entry's reflection sign is -1
    int e0, nent;          // first entry of the chunk, entries in all
};
constexpr int kSpecThreads = 128;

template <bool ROWS>
__global__ void __launch_bounds__(kSpecThreads) k_spectrum_axis(const double2* __restrict__ in,
                                                                double2* __restrict__ out, float2* __restrict__ out64,
                                                                SpecPass p, const double2* __restrict__ tw) {
    extern __shared__ unsigned char smem_raw[];
    const int M = p.plan.n, tile = p.tile, pitch = p.pitch;
    double2* buf0 = reinterpret_cast<double2*>(smem_raw);
    double2* buf1 = buf0 + (ROWS ? tile : M) * pitch;
    const int tid = threadIdx.x;
    const int e = blockIdx.z;
    const long long o = blockIdx.y, t0 = (long long)blockIdx.x * tile;
    const int nt = (int)min((long long)tile, p.n_inner - t0);
    const double sg = (p.neg >> (p.e0 + e)) & 1 ? -1.0 : 1.0;
    const double2* src = in + e * p.in_e + o * p.in_o;
    for (int idx = tid; idx < M * tile; idx += kSpecThreads) {
        const int k = ROWS ? idx % M : idx / tile, t = ROWS ? idx / M : idx % tile;
        double2 v = make_double2(0, 0);
        if (t < nt && (k < p.N || k > M - p.N)) {
            const int d = k < p.N ? k : M - k;
            const double s = k < p.N ? 1.0 : sg;
            const double2 u = ROWS ? src[(t0 + t) * p.N + d] : src[d * p.in_k + t0 + t];
            v = make_double2(s * u.x, s * u.y);
        }
        buf0[ROWS ? t * pitch + k : k * pitch + t] = v;
    }
    __syncthreads();
    const double2* res = fft_lds<double, true, ROWS>(buf0, buf1, p.plan, tile, ROWS ? pitch : 1, ROWS ? 1 : pitch, tw,
                                                     tid, kSpecThreads);
    if (ROWS) {
        for (int idx = tid; idx < p.O * nt; idx += kSpecThreads) {
            const int t = idx / p.O, k = idx - t * p.O;
            const double2 v = res[t * pitch + k];
            const long long dst = ((t0 + t) * p.nent + p.e0 + e) * p.O + k;
            out[dst] = v;
            if (out64) out64[dst] = make_float2((float)v.x, (float)v.y);
        }
    } else {
        double2* dst = out + e * p.out_e + o * p.out_o + t0;
        for (int idx = tid; idx < p.O * tile; idx += kSpecThreads) {
            const int k = idx / tile, t = idx - k * tile;
            if (t < nt) dst[k * p.out_k + t] = res[k * pitch + t];
        }
    }
}

// ---------------------------------------------------------------------------
// host entry points
// ---------------------------------------------------------------------------
void assemble_blocks(double2* out, const AssemblyTables& T, int Nx, int Ny, int Nz, hipStream_t s) {
    const FarTables F = build_far_tables(T);
    VIE_REQUIRE(F.nterm <= kFarTerms && F.npair <= kFarTerms, -1, "assembly: term table overflow");
    struct Tables {   // released after the drain below, on every way out
        AssemblyTables* T = nullptr;
        FarTables* F = nullptr;
        ~Tables() {
            if (T) (void)hipFree(T);
            if (F) (void)hipFree(F);
        }
    } dev;
    const StreamDrain drain(s);
    VIE_HIP(hipMalloc(&dev.T, sizeof(AssemblyTables)));
    VIE_HIP(hipMalloc(&dev.F, sizeof(FarTables)));
    AssemblyTables* const dT = dev.T;
    FarTables* const dF = dev.F;
    VIE_HIP(hipMemcpyAsync(dT, &T, sizeof(AssemblyTables), hipMemcpyHostToDevice, s));
    VIE_HIP(hipMemcpyAsync(dF, &F, sizeof(FarTables), hipMemcpyHostToDevice, s));
    const long long V = (long long)Nx * Ny * Nz;
    hipLaunchKernelGGL(k_assemble_near, dim3(T.nent, 8), dim3(kNearThreads), 0, s, out, dT, Nx, Ny, Nz);
    VIE_HIP(hipGetLastError());
    const int dmax = std::max(Nx, std::max(Ny, Nz)) - 1;
    for (int b = 0; b < kFarBands; ++b) {
        const FarBand& B = F.band[b];
        if (B.dlo > dmax) break;
        // offsets in the band: the cube of edge min(dhi, dmax) + 1 minus the one of edge dlo
        const int hi = std::min(B.dhi, dmax) + 1;
        const int cx = std::min(hi, Nx), cy = std::min(hi, Ny), cz = std::min(hi, Nz);
        const long long cnt = (long long)cx * cy * cz -
                              (long long)std::min(B.dlo, Nx) * std::min(B.dlo, Ny) * std::min(B.dlo, Nz);
        const unsigned grid = (unsigned)std::max<long long>(1, std::min<long long>(cnt, 1 << 16));
        const double* D = T.D;
#define FAR_CASE(P_, W_)                                                                                         \
    case P_:                                                                                                     \
        hipLaunchKernelGGL((k_assemble_far<P_, W_>), dim3(grid), dim3(64 * W_), 0, s, out, dF, b, D[0], D[1],    \
                           D[2], T.k0, Nx, Ny, Nz, cx, cy, cz);                                                  \
        break;
        // runs as long as leaves 8192 of them (12 wavefronts per CU fill the
        // chip with 3072), at most 16
        const int run = (int)std::max<long long>(1, std::min<long long>(cnt / 8192, 16));
        const long long runs = (long long)((cx + run - 1) / run) * cy * cz;
#define FAR_ROWS(P_)                                                                                             \
    case P_:                                                                                                     \
        hipLaunchKernelGGL(k_assemble_far_rows<P_>, dim3((unsigned)std::min<long long>(runs, 1 << 16)), dim3(64), \
                           0, s, out, dF, b, D[0], D[1], D[2], T.k0, Nx, Ny, Nz, cx, cy, cz, run);               \
        break;
        switch (B.P) {
            FAR_CASE(31, 4)
            FAR_CASE(21, 4)
            FAR_CASE(17, 4)
            FAR_ROWS(13)
            FAR_ROWS(11)
            default: throw Error(-1, "assembly: unsupported Gauss order band");
        }
#undef FAR_CASE
#undef FAR_ROWS
        VIE_HIP(hipGetLastError());
    }
    VIE_HIP(hipStreamSynchronize(s));
}

// reflection sign of unique entry e along an axis (same for its whole orbit)
int unique_refl_sign(int e, int axis) {
    static const int P[6] = {0, 0, 0, 1, 1, 2}, Q[6] = {0, 1, 2, 1, 2, 2};
    static const int L[10] = {1, 1, 1, 1, 2, 2, 2, 3, 3, 4}, LP[10] = {1, 2, 3, 4, 2, 3, 4, 3, 4, 4};
    const int pq = e / 10, ll = e % 10;
    const int a = 4 * P[pq] + L[ll] - 1, b = 4 * Q[pq] + LP[ll] - 1;
    return refl_sign(axis, a) * refl_sign(axis, b);
}

// reflection sign of curl tensor e = 10 k + ll along an axis: the linear
// functions along the axis change sign, and d_k g is odd along k, so
// K(.., -d_i, ..) = -sigma_i(a) sigma_i(b) K(.., d_i, ..)
int curl_refl_sign(int e, int axis) {
    static const int L[10] = {1, 1, 1, 1, 2, 2, 2, 3, 3, 4}, LP[10] = {1, 2, 3, 4, 2, 3, 4, 3, 4, 4};
    const int k = e / 10, ll = e % 10;
    int s = 1;
    if (L[ll] == axis + 2) s = -s;
    if (LP[ll] == axis + 2) s = -s;
    if (k == axis) s = -s;
    return s;
}

// values of scratch one entry needs between its passes: [Oz][Ny][Nx] after
// z, [Oz][Oy][Nx] after y
static long long spectrum_values(const int N[3], const int M[3]) {
    const long long Oz = M[2] / 2 + 1, Oy = M[1] / 2 + 1;
    return Oz * N[1] * N[0] + Oz * Oy * N[0];
}

// Scratch of the spectra: chunks of entries go through the three passes
// together, about 7 in 16 V values (a quarter of what a complex128 product
// will need), all of them where that is below 8 MiB (small grids, where the
// launches count), at least one.
size_t spectra_scratch_bytes(const int N[3], const int M[3]) {
    const long long per = spectrum_values(N, M), V = (long long)N[0] * N[1] * N[2];
    const long long most = std::max<long long>(16 * V, (8LL << 20) / (long long)sizeof(double2));
    return (size_t)std::max(per, std::min(60 * per, most / per * per)) * sizeof(double2);
}

void operator_spectra(double2* U128, float2* U64, const double2* T, double2* scratch, size_t scratch_bytes,
                      const int N[3], const int M[3], const FftPlan plans[3], const double2* const tw[3],
                      hipStream_t s, bool curl) {
    const long long V = (long long)N[0] * N[1] * N[2], per = spectrum_values(N, M);
    const int Ox = M[0] / 2 + 1, Oy = M[1] / 2 + 1, Oz = M[2] / 2 + 1;
    const int nent = curl ? 30 : 60;
    const int chunk = (int)std::min<long long>(nent, (long long)(scratch_bytes / sizeof(double2)) / per);
    VIE_REQUIRE(chunk >= 1, VIE_EINVAL, "operator spectra: scratch below one entry");
    SpecPass ps[3];
    for (int ax = 0; ax < 3; ++ax) {
        SpecPass& p = ps[ax];
        p = SpecPass{};
        p.plan = plans[ax];
        p.N = N[ax];
        p.O = M[ax] / 2 + 1;
        p.nent = nent;
        // up to 8 pencils (whole 128-byte lines) in 64 KiB of LDS, one at the longest lengths
        p.tile = std::max(1, std::min(8, (int)(64 * 1024 / (2 * sizeof(double2) * M[ax]))));
        p.pitch = ax == 0 ? M[ax] + 1 : p.tile;
        for (int e = 0; e < nent; ++e)
            if ((curl ? curl_refl_sign(e, ax) : unique_refl_sign(e, ax)) < 0) p.neg |= 1ULL << e;
    }
    // z: [e][Nz][Ny Nx] -> [e][Oz][Ny Nx]
    ps[2].n_inner = N[0] * N[1];
    ps[2].in_e = V;
    ps[2].in_k = ps[2].out_k = (long long)N[0] * N[1];
    ps[2].out_e = (long long)Oz * N[1] * N[0];
    // y: [e][Oz][Ny][Nx] -> [e][Oz][Oy][Nx]
    ps[1].n_inner = N[0];
    ps[1].in_e = ps[2].out_e;
    ps[1].in_o = (long long)N[1] * N[0];
    ps[1].in_k = ps[1].out_k = N[0];
    ps[1].out_e = (long long)Oz * Oy * N[0];
    ps[1].out_o = (long long)Oy * N[0];
    // x: rows [e][Oz Oy][Nx] -> U[Oz Oy][nent][Ox]
    ps[0].n_inner = Oz * Oy;
    ps[0].in_e = ps[1].out_e;
    auto lds = [](const SpecPass& p, bool rows) {
        return 2 * (size_t)(rows ? p.tile : p.plan.n) * p.pitch * sizeof(double2);
    };
    static std::once_flag once;
    std::call_once(once, [] {
        (void)hipFuncSetAttribute((const void*)k_spectrum_axis<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  160 * 1024);
        (void)hipFuncSetAttribute((const void*)k_spectrum_axis<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  160 * 1024);
        (void)hipGetLastError();
    });
    double2* A = scratch;
    double2* B = scratch + (long long)chunk * ps[2].out_e;
    for (int e0 = 0; e0 < nent; e0 += chunk) {
        const unsigned ne = (unsigned)std::min(chunk, nent - e0);
        for (auto& p : ps) p.e0 = e0;
        auto tiles = [](const SpecPass& p) { return (unsigned)((p.n_inner + p.tile - 1) / p.tile); };
        hipLaunchKernelGGL(k_spectrum_axis<false>, dim3(tiles(ps[2]), 1, ne), dim3(kSpecThreads), lds(ps[2], false), s,
                           T + e0 * V, A, (float2*)nullptr, ps[2], tw[2]);
        VIE_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_spectrum_axis<false>, dim3(tiles(ps[1]), (unsigned)Oz, ne), dim3(kSpecThreads),
                           lds(ps[1], false), s, A, B, (float2*)nullptr, ps[1], tw[1]);
        VIE_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_spectrum_axis<true>, dim3(tiles(ps[0]), 1, ne), dim3(kSpecThreads), lds(ps[0], true), s,
                           B, U128, U64, ps[0], tw[0]);
        VIE_HIP(hipGetLastError());
    }
}

}  // namespace vie
