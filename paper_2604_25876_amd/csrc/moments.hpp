// Moment observables of a field (Sec. 5): centre of mass (eq. CoM), RMS
// radius (eq. RMS radius), the inertia tensors U, V, W (eqs. U, V, W inertia
// tensor), the isospin-0 quadrupole (eq. Q tensor) and the D-term (eq. D-term
// with the static stress tensor of eq. Stress tensor).
//
// Two passes over the interior I, FP64 arithmetic from the stored field: pass 1 sums the
// charge density b, its first moments and the energy density, and fixes the centre X_c on the
// device; pass 2 sums the tensor densities in the frame r = x - X_c.  Per-block partial sums
// are reduced in a fixed order, so the result is deterministic.
//
// A thread takes two neighbouring sites of a row and reads their 13-point stars in pairs: 11
// accesses a component where two sites one by one take 26.  The vector memory unit spends 16
// cycles on an access of a wave whatever its width up to 16 bytes, which is what bounded the
// passes (52 accesses a site: 101 us a pass on 151^3 double for 110 MB of field).
//
// The traces of the printed formulas are evaluated in the vector form of
// su(2): with X = x0 + i x.tau, Tr(XY) = 2 (x0 y0 - x.y) and a commutator
// [X, Y] = i (-2 x cross y).tau, so Tr([X, Z][Y, W]) = -8 (x cross z).(y cross w).
// L_k = U^dagger d_k U has scalar part s_k = phi . a_k and vector part
// l_k = phi0 a_k - a_k^0 phi + phi cross a_k (3-vector parts); T_j =
// (i/2) U^dagger [tau^j, U] is pure with vector t_j = -phi0 (e_j cross phi)
// - |phi|^2 e_j + phi_j phi.  With the Gram matrices G = (l_m . l_p), S = tr G,
// Mx = (l_k . t_i) the densities are
//   U_ij: 2 (1 + S) t_i.t_j - 2 (Mx^T Mx)_ij
//   K    = 2 (G - s s^T) + 2 (S G - G^2)   (the stress tensor without its delta_ij part)
//   V   = R K R^T, R v = r cross v
//   W_ij: -2 (R N)_ji, N = (1 + S) Mx - G Mx
//   D   : r.K.r - |r|^2 tr K / 3
// Quantities use the printed (un-halved) normalisation of the Lagrangian.
#pragma once

#include <hip/hip_runtime.h>

namespace skyr {

constexpr int MOM_THREADS = 256;
constexpr int MOM_MAX_BLOCKS = 1024;
constexpr int MOM_NACC = 32;  // partial-sum slots per block (pass 2 uses 28)
constexpr int MOM_PASS_CENTRE = 1;
constexpr int MOM_PASS_TENSORS = 2;

// device result record: {B, E, X[3], R, U[9], V[9], W[9], Q[9], D}
constexpr int MOM_OUT_DOUBLES = 43;

struct MomArgs {
    const void* phi;
    int n0, n1, n2;
    double h;
    double* partials;      // [gridDim.x][MOM_NACC]
    double* centre;        // 5 doubles: sum b, X_c, sum of the energy density (pass 1)
    double* out;           // MOM_OUT_DOUBLES
    double m, m_y, m_z, m_w, c6;  // couplings of the energy
};

template <int PASS> struct MomAcc {
    static constexpr int N = PASS == MOM_PASS_CENTRE ? 5 : 28;
    static constexpr int WAVES = PASS == MOM_PASS_CENTRE ? 3 : 2;  // per SIMD, as the registers allow
    static constexpr int MAX_BLOCKS = WAVES * 256;                 // one round of the chip
    static_assert(MAX_BLOCKS <= MOM_MAX_BLOCKS, "partial records");
};

// two neighbouring elements of a row, at the alignment of one
template <typename T> struct MomPair {
    typedef T type __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};

// The field p, its first differences d (Sec. 3: (f(-2) - 8 f(-1) + 8 f(+1) - f(+2)) / 12h) and, in
// pass 1, phi . Lap phi (five-point second differences) at sites c and c + 1 of every component.
template <typename T, bool LAP>
__device__ __forceinline__ void mom_stars(const T* c, long long sx, long long sy, long long N3, double inv12h,
                                          double inv12h2, double (&p)[2][4], double (&d)[2][3][4], double (&pl)[2])
{
    typedef typename MomPair<T>::type pair;
    pl[0] = pl[1] = 0.0;
#pragma unroll
    for (int A = 0; A < 4; ++A, c += N3) {
        const auto at = [&](long long o) { return *(const pair*)(c + o); };
        const pair z0 = at(-2), z1 = at(0), z2 = at(2);
        const pair y0 = at(-2 * sy), y1 = at(-sy), y2 = at(sy), y3 = at(2 * sy);
        const pair x0 = at(-2 * sx), x1 = at(-sx), x2 = at(sx), x3 = at(2 * sx);
        const T z[6] = {z0[0], z0[1], z1[0], z1[1], z2[0], z2[1]};
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const double q = (double)z[2 + s];
            const double am2 = (double)x0[s], am1 = (double)x1[s], ap1 = (double)x2[s], ap2 = (double)x3[s];
            const double bm2 = (double)y0[s], bm1 = (double)y1[s], bp1 = (double)y2[s], bp2 = (double)y3[s];
            const double cm2 = (double)z[s], cm1 = (double)z[s + 1], cp1 = (double)z[s + 3], cp2 = (double)z[s + 4];
            p[s][A] = q;
            d[s][0][A] = (am2 - 8.0 * am1 + 8.0 * ap1 - ap2) * inv12h;
            d[s][1][A] = (bm2 - 8.0 * bm1 + 8.0 * bp1 - bp2) * inv12h;
            d[s][2][A] = (cm2 - 8.0 * cm1 + 8.0 * cp1 - cp2) * inv12h;
            if constexpr (LAP) {
                const double s1 = ((ap1 + am1) + (bp1 + bm1)) + (cp1 + cm1);
                const double s2 = ((ap2 + am2) + (bp2 + bm2)) + (cp2 + cm2);
                pl[s] += q * ((16.0 * s1 - s2 - 90.0 * q) * inv12h2);
            }
        }
        // formed here: moved to their uses, they would keep all four components' neighbours in
        // registers (230 of them, two waves a SIMD)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            asm volatile("" : "+v"(d[s][0][A]), "+v"(d[s][1][A]), "+v"(d[s][2][A]));
            if constexpr (LAP) asm volatile("" : "+v"(pl[s]));
        }
    }
}

template <typename T, int PASS>
__global__ __launch_bounds__(MOM_THREADS, MomAcc<PASS>::WAVES) void moments_kernel(MomArgs a)
{
    constexpr int NA = MomAcc<PASS>::N;
    const T* __restrict__ phi = (const T*)a.phi;
    const int n0 = a.n0, n1 = a.n1, n2 = a.n2;
    const long long sy = n2, sx = (long long)n1 * n2, N3 = n0 * sx;
    // pairs of sites of I: the second site of a row's last pair lies outside I when I has an odd
    // number of columns (its star is still within the arrays: the rows of I are not the last ones)
    const unsigned ni1 = n1 - 4, ni2 = n2 - 4, np2 = (ni2 + 1) / 2;
    const unsigned pairs = (unsigned)(n0 - 4) * ni1 * np2;
    const double h = a.h, inv12h = 1.0 / (12.0 * h), inv12h2 = 1.0 / (12.0 * h * h);
    const double cb0 = 0.5 * (n0 - 1), cb1 = 0.5 * (n1 - 1), cb2 = 0.5 * (n2 - 1);
    double Xc0 = 0.0, Xc1 = 0.0, Xc2 = 0.0;
    if constexpr (PASS == MOM_PASS_TENSORS) {
        Xc0 = a.centre[1];
        Xc1 = a.centre[2];
        Xc2 = a.centre[3];
    }
    double acc[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) acc[k] = 0.0;

    // The blocks of an XCD (block i runs on XCD i mod 8) walk an eighth of I together, so that the
    // five planes their stars span stay in its L2; in steps of the whole grid, every XCD read the
    // planes around 17 others' (151^3 double: 87 us a pass against 58 us).
    const unsigned xcd = blockIdx.x % 8, in_xcd = (gridDim.x + 7 - xcd) / 8;
    const unsigned share = (pairs + 7) / 8, begin = min(xcd * share, pairs), end = min(begin + share, pairs);
    for (unsigned q = begin + (blockIdx.x / 8) * MOM_THREADS + threadIdx.x; q < end; q += in_xcd * MOM_THREADS) {
        const unsigned yx = q / np2;
        const int z0 = 2 + 2 * (int)(q - yx * np2);
        const int x = 2 + (int)(yx / ni1);
        const int y = 2 + (int)(yx - (unsigned)(x - 2) * ni1);
        double p2[2][4], d2[2][3][4], pl[2];
        mom_stars<T, PASS == MOM_PASS_CENTRE>(phi + (x * sx + y * sy + z0), sx, sy, N3, inv12h, inv12h2, p2, d2, pl);
#pragma unroll
      for (int site = 0; site < 2; ++site) {
        const int z = z0 + site;
        if (z > n2 - 3) break;
        const double(&p)[4] = p2[site];
        const double(&d)[3][4] = d2[site];
        const double det = det4(p, d[0], d[1], d[2]);
        const double b = -det * (1.0 / (2.0 * M_PI * M_PI));
        const double X0 = (x - cb0) * h, X1 = (y - cb1) * h, X2 = (z - cb2) * h;
        if constexpr (PASS == MOM_PASS_CENTRE) {
            acc[0] += b;
            acc[1] += X0 * b;
            acc[2] += X1 * b;
            acc[3] += X2 * b;
            // the energy density of E_h (Sec. 2.1, halved) and its optional terms
            const double gxx = dot4(d[0], d[0]), gyy = dot4(d[1], d[1]), gzz = dot4(d[2], d[2]);
            const double gxy = dot4(d[0], d[1]), gxz = dot4(d[0], d[2]), gyz = dot4(d[1], d[2]);
            const double e4 = 0.5 * (gxx * gyy + gxx * gzz + gyy * gzz - gxy * gxy - gxz * gxz - gyz * gyz);
            const double u = 1.0 - p[0];
            const double V = a.m * a.m * u + 0.5 * a.m_y * a.m_y * (1.0 - p[0] * p[0]) + 0.5 * a.m_z * a.m_z * u * u +
                             0.25 * a.m_w * a.m_w * (u * u) * (u * u);
            acc[4] += (e4 - 0.5 * pl[site]) + (V + 0.5 * a.c6 * det * det);
        } else {
            const double r[3] = {X0 - Xc0, X1 - Xc1, X2 - Xc2};
            // charge moments: xx yy zz xy xz yz
            acc[0] += r[0] * r[0] * b;
            acc[1] += r[1] * r[1] * b;
            acc[2] += r[2] * r[2] * b;
            acc[3] += r[0] * r[1] * b;
            acc[4] += r[0] * r[2] * b;
            acc[5] += r[1] * r[2] * b;
            // currents
            const double p0 = p[0], p1 = p[1], p2 = p[2], p3 = p[3];
            double sk[3], l[3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double* e = d[k];
                sk[k] = p0 * e[0] + p1 * e[1] + p2 * e[2] + p3 * e[3];
                l[k][0] = p0 * e[1] - e[0] * p1 + (p2 * e[3] - p3 * e[2]);
                l[k][1] = p0 * e[2] - e[0] * p2 + (p3 * e[1] - p1 * e[3]);
                l[k][2] = p0 * e[3] - e[0] * p3 + (p1 * e[2] - p2 * e[1]);
            }
            const double pv2 = p1 * p1 + p2 * p2 + p3 * p3;
            const double t[3][3] = {{p1 * p1 - pv2, p0 * p3 + p1 * p2, p1 * p3 - p0 * p2},
                                    {p1 * p2 - p0 * p3, p2 * p2 - pv2, p0 * p1 + p2 * p3},
                                    {p0 * p2 + p1 * p3, p2 * p3 - p0 * p1, p3 * p3 - pv2}};
            // symmetric matrices by their six entries xx yy zz xy xz yz: sym(i, j) is the index
            constexpr int iu[6] = {0, 1, 2, 0, 0, 1}, ju[6] = {0, 1, 2, 1, 2, 2};
            const auto sym = [](int i, int j) { return i == j ? i : i + j + 2; };
            double G[6], Mx[3][3];
#pragma unroll
            for (int e = 0; e < 6; ++e)
                G[e] = l[iu[e]][0] * l[ju[e]][0] + l[iu[e]][1] * l[ju[e]][1] + l[iu[e]][2] * l[ju[e]][2];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 3; ++j) Mx[i][j] = l[i][0] * t[j][0] + l[i][1] * t[j][1] + l[i][2] * t[j][2];
            const double S = G[0] + G[1] + G[2];
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const int i = iu[e], j = ju[e];
                const double tt = t[i][0] * t[j][0] + t[i][1] * t[j][1] + t[i][2] * t[j][2];
                const double mm = Mx[0][i] * Mx[0][j] + Mx[1][i] * Mx[1][j] + Mx[2][i] * Mx[2][j];
                acc[6 + e] += 2.0 * (1.0 + S) * tt - 2.0 * mm;
            }
            // N = (1 + S) Mx - G Mx; W_ij = -2 (r cross N_i)_j with N_i the column i of N
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                double N[3];
#pragma unroll
                for (int m = 0; m < 3; ++m)
                    N[m] = (1.0 + S) * Mx[m][i] -
                           (G[sym(m, 0)] * Mx[0][i] + G[sym(m, 1)] * Mx[1][i] + G[sym(m, 2)] * Mx[2][i]);
                acc[18 + 3 * i + 0] += -2.0 * (r[1] * N[2] - r[2] * N[1]);
                acc[18 + 3 * i + 1] += -2.0 * (r[2] * N[0] - r[0] * N[2]);
                acc[18 + 3 * i + 2] += -2.0 * (r[0] * N[1] - r[1] * N[0]);
            }
            // K = 2 (G - s s^T) + 2 (S G - G^2)
            double K[6];
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const int i = iu[e], j = ju[e];
                const double gg = G[sym(i, 0)] * G[sym(0, j)] + G[sym(i, 1)] * G[sym(1, j)] + G[sym(i, 2)] * G[sym(2, j)];
                K[e] = 2.0 * (G[e] - sk[i] * sk[j]) + 2.0 * (S * G[e] - gg);
            }
            // V = R K R^T with R v = r cross v: the columns of K, then the rows of R K, crossed with r
            double RK[3][3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                RK[0][j] = r[1] * K[sym(2, j)] - r[2] * K[sym(1, j)];
                RK[1][j] = r[2] * K[sym(0, j)] - r[0] * K[sym(2, j)];
                RK[2][j] = r[0] * K[sym(1, j)] - r[1] * K[sym(0, j)];
            }
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                const int i = iu[e], j = ju[e], j1 = (j + 1) % 3, j2 = (j + 2) % 3;
                acc[12 + e] += r[j1] * RK[i][j2] - r[j2] * RK[i][j1];
            }
            // D-term moment: r.K.r - |r|^2 tr K / 3
            double rKr = 0.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) rKr += r[i] * (K[sym(i, 0)] * r[0] + K[sym(i, 1)] * r[1] + K[sym(i, 2)] * r[2]);
            const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
            acc[27] += rKr - r2 * (K[0] + K[1] + K[2]) * (1.0 / 3.0);
        }
      }
    }

    // fixed-order block reduction: the lanes of a wave, then the four waves in order
    __shared__ double red[MOM_THREADS / 64][NA];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        const double v = wave_total<false>(acc[k]);
        if (lane == 0) red[wave][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < NA) {
        const int k = threadIdx.x;
        double v = 0.0;
        for (int w = 0; w < MOM_THREADS / 64; ++w) v += red[w][k];
        a.partials[(size_t)blockIdx.x * MOM_NACC + k] = v;
    }
}

// sum of slot k over nblocks records, thread t taking blocks t, t + 256, ...
// then a fixed tree; every thread returns the total
__device__ static double mom_reduce_slot(const double* __restrict__ part, int nblocks, int k, double* red)
{
    const int t = threadIdx.x;
    double s = 0.0;
    for (int b = t; b < nblocks; b += MOM_THREADS) s += part[(size_t)b * MOM_NACC + k];
    red[t] = s;
    __syncthreads();
    for (int w = MOM_THREADS / 2; w > 0; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    const double total = red[0];
    __syncthreads();
    return total;
}

// sum of slot k over nblocks records by one wave: lane t takes records t, t + 64, ... in order,
// then the lanes in the fixed order of wave_total; every lane returns the total
__device__ static double mom_wave_slot(const double* __restrict__ part, int nblocks, int k)
{
    double s = 0.0;
    for (int b = threadIdx.x & 63; b < nblocks; b += 64) s += part[(size_t)b * MOM_NACC + k];
    return wave_total<false>(s);
}

// one wave per slot (a block-wide tree per slot, one slot after the other, took 39 us for the 28
// tensor slots)
constexpr int MOM_FINISH_THREADS = 1024;

__global__ __launch_bounds__(MOM_FINISH_THREADS) void moments_centre_kernel(MomArgs a, int nblocks)
{
    constexpr int N = MomAcc<MOM_PASS_CENTRE>::N;
    __shared__ double s[N];
    const int wave = threadIdx.x >> 6;
    if (wave < N) {
        const double v = mom_wave_slot(a.partials, nblocks, wave);
        if ((threadIdx.x & 63) == 0) s[wave] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.centre[0] = s[0];
        a.centre[1] = s[1] / s[0];
        a.centre[2] = s[2] / s[0];
        a.centre[3] = s[3] / s[0];
        a.centre[4] = s[4];
    }
}

__global__ __launch_bounds__(MOM_FINISH_THREADS) void moments_finish_kernel(MomArgs a, int nblocks)
{
    constexpr int N = MomAcc<MOM_PASS_TENSORS>::N, WAVES = MOM_FINISH_THREADS / 64;
    __shared__ double s[N];
    for (int k = threadIdx.x >> 6; k < N; k += WAVES) {
        const double v = mom_wave_slot(a.partials, nblocks, k);
        if ((threadIdx.x & 63) == 0) s[k] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double h3 = a.h * a.h * a.h;
    const double B = h3 * a.centre[0];
    const double E = 2.0 * h3 * a.centre[4];  // printed normalisation
    double* o = a.out;
    o[0] = B;
    o[1] = E;
    o[2] = a.centre[1];
    o[3] = a.centre[2];
    o[4] = a.centre[3];
    const int iu[6] = {0, 1, 2, 0, 0, 1}, ju[6] = {0, 1, 2, 1, 2, 2};
    double Mom[3][3];
    for (int e = 0; e < 6; ++e) Mom[iu[e]][ju[e]] = Mom[ju[e]][iu[e]] = h3 * s[e];
    const double trM = Mom[0][0] + Mom[1][1] + Mom[2][2];
    o[5] = sqrt(trM / B);
    double* U = o + 6;
    double* V = o + 15;
    double* W = o + 24;
    double* Q = o + 33;
    for (int e = 0; e < 6; ++e) {
        const int i = iu[e], j = ju[e];
        U[3 * i + j] = U[3 * j + i] = h3 * s[6 + e];
        V[3 * i + j] = V[3 * j + i] = h3 * s[12 + e];
    }
    for (int e = 0; e < 9; ++e) W[e] = h3 * s[18 + e];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) Q[3 * i + j] = 0.5 * (3.0 * Mom[i][j] - (i == j ? trM : 0.0));
    o[42] = -(2.0 * E / 5.0) * h3 * s[27];
}

// kinetic energy: per-block sums of |v|^2 over I (slot 0 of the partial records)
template <typename T>
__global__ __launch_bounds__(MOM_THREADS) void kinetic_kernel(const T* __restrict__ vel, int n0, int n1, int n2,
                                                              double* __restrict__ partials)
{
    const size_t sy = (size_t)n2, sx = (size_t)n1 * n2, N3 = (size_t)n0 * sx;
    const int ni1 = n1 - 4, ni2 = n2 - 4;
    const long long nI = (long long)(n0 - 4) * ni1 * ni2;
    double acc = 0.0;
    for (long long q = (long long)blockIdx.x * MOM_THREADS + threadIdx.x; q < nI;
         q += (long long)gridDim.x * MOM_THREADS) {
        const int z = 2 + (int)(q % ni2);
        const long long yx = q / ni2;
        const int y = 2 + (int)(yx % ni1);
        const int x = 2 + (int)(yx / ni1);
        const size_t s = (size_t)x * sx + (size_t)y * sy + (size_t)z;
#pragma unroll
        for (int A = 0; A < 4; ++A) {
            const double v = (double)vel[(size_t)A * N3 + s];
            acc += v * v;
        }
    }
    __shared__ double red[MOM_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double v = 0.0;
        for (int w = 0; w < MOM_THREADS / 64; ++w) v += red[w];
        partials[(size_t)blockIdx.x * MOM_NACC] = v;
    }
}

__global__ __launch_bounds__(MOM_THREADS) void kinetic_finish_kernel(const double* __restrict__ partials, int nblocks,
                                                                     double h, double* __restrict__ out)
{
    __shared__ double red[MOM_THREADS];
    const double s = mom_reduce_slot(partials, nblocks, 0, red);
    if (threadIdx.x == 0) out[0] = 0.5 * h * h * h * s;
}

}  // namespace skyr
