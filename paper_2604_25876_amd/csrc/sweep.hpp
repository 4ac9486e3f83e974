// sweep.hpp -- fused per-step sweep of the arrested Newton flow for gfx950.
//
// One launch evaluates, for every interior site of one field, the discrete
// energy density, the exact gradient of the discrete energy E_h (Sec. 2.1
// energy, Sec. 3 stencils), its tangent projection (Sec. 3, eq. Newton_flow)
// and either the kick-drift-renormalise update (Sec. 3) or a gradient output,
// plus FP64 per-block partial sums of E2, E4, E0, B and the largest |F|^2.
//
// The gradient is -Lap phi (with boundary terms) - sum_i D_i Q_i + V'(phi0) e0, where
// Q_i = S a_i - sum_j G_ij a_j is the flux of the quartic term at the sites of I (zero
// elsewhere).  Two stencil passes: the flux needs phi within two sites, the divergence
// needs the flux within two sites.
//
// Work decomposition (2.5D march along x):
//   * a tile is OY rows (y) x OZ columns (z) of output sites; tiles in z start on a
//     128-byte line when that costs no extra tile;
//   * the block's waves have two roles.  Interior waves hold one output site per lane
//     and do everything there: the derivatives, the Laplacian, the three fluxes, the
//     x-divergence by pushes into a register ring of five gradient accumulators, the
//     y/z-divergence from LDS and the update.  Halo waves hold the flux positions
//     around the tile (two rows above and below, two columns left and right), where
//     only one flux component is ever read (Q_y on the y-halo, Q_z on the z-halo), and
//     compute just that one;
//   * x-neighbours live in per-lane register rings of five phi planes; the march is
//     unrolled five planes deep so that every ring slot is a fixed register;
//   * y- and z-neighbours go through LDS: phi planes (with the frame of sites only the halo
//     positions read, loaded by the halo lanes) and planes of Q_y and Q_z, each
//     double-buffered by plane parity, so one block barrier per plane suffices;
//   * x is cut into slabs; a launch has one block per (slab, tile) item, so that the
//     blocks of neighbouring tiles march through the same planes together and read the
//     phi lines of their shared halo from L2 once; on fields larger than the last-level cache
//     the velocity read and the outputs are streamed past the caches (non-temporal) so that
//     they do not displace those lines.
// Stencils are evaluated in the scaled form 8 (f[+1] - f[-1]) - (f[+2] - f[-2]) =
// 12 h D f (and 16 (...) - (...) = 12 h^2 L f); the constant factors are folded into
// the weights of the final sums.  Energy, charge and force sums are accumulated in
// double.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/skyr.h"
#include "cut.hpp"
#include "shapes.hpp"

#include <type_traits>

namespace skyr {

// partial-sum slots per thread block (doubles)
constexpr int NPART = 8;
enum : int { P_E2 = 0, P_E4 = 1, P_E0 = 2, P_B = 3, P_F2 = 4, P_POW = 5, P_E6 = 6 };
constexpr int NRED = 7;  // slots in use

// Control block of one flow, in device memory at the start of the workspace.
struct Ctl {
    int32_t cur;          // field buffer holding phi_k: 0 = phi, 1 = phi_alt
    int32_t redo;         // this sweep re-runs phi_k with v_k = 0
    int32_t done;         // 1: no further sweep does any work
    int32_t status;       // 0 running, 1 converged, 2 step target reached, 3 non-finite
    int64_t steps;        // accepted steps
    int64_t target;       // stop when steps reaches this
    int64_t arrests;
    int64_t redo_sweeps;
    int64_t sweeps;
    int32_t renorm64_every;
    int32_t nblocks;      // number of partial-sum blocks of the sweep
    int32_t flow_mode;    // skyr_flow_mode
    int32_t restore;      // after convergence: the next sweep over phi_k rewrites v_k (RESTORE_*)
    int32_t ticket;       // blocks of the running sweep that have finished (zero between sweeps)
    int32_t hold;         // timing sweeps: the sweep takes no decision (the state stays as it is)
    double E_prev;
    double E;
    double P;             // power h^3 sum F_k . v_k of the last sweep (arrest rule POWER)
    double unused_[1];
    double max_force;
    double tol;
    double h3;
    double pad[4];
};
static_assert(sizeof(Ctl) <= 256, "control block must fit its 256-byte slot");

enum : int { MODE_STEP = 0, MODE_GRAD = 1 };

// Cache policy of a step sweep's accesses that are used once per sweep (the velocity read, the
// outputs written); the host chooses it by the bytes of the fields (stream_policy in skyr.hip).
// A template parameter of the kernels: as a branch around the accesses it split the plane's one
// block of code and cost 10% (128^3 float) to 20% (256^3 double).
enum : int {
    STREAM_NONE = 0,    // plain accesses: the fields stay in the last-level cache between sweeps
    STREAM_STORES = 1,  // non-temporal outputs
    STREAM_ALL = 2      // non-temporal outputs and velocity reads
};

// The converging sweep over phi_k has already written v_k + dt F_k over v_k.  The sweep
// after it recomputes F_k from phi_k (the same arithmetic, so the same F_k) and writes
// v_k back: v - dt F_k, or exactly zero when v_k was zero (an arrest at step k, a redo
// sweep, or the gradient flow).  No field is written by that sweep.
enum : int { RESTORE_NONE = 0, RESTORE_UNKICK = 1, RESTORE_ZERO = 2 };

struct SweepArgs {
    const void* phi0;  // field buffer 0 (phi)
    void* phi1;        // field buffer 1 (phi_alt); MODE_GRAD: unused
    void* vel;         // MODE_STEP: velocity, updated in place
    void* grad;        // MODE_GRAD: nullable gradient output
    double* partials;  // [nblocks][NPART]
    Ctl* ctl;          // MODE_STEP: control block
    int n0, n1, n2;        // extent of the stored array (the whole lattice, or a padded block)
    // elements from one component of the field to the next: n0 n1 n2 for component-major
    // arrays; the row length when the components of a row follow each other (the row of
    // n2 elements then holding all four, each in its own quarter)
    long long cstride;
    int zlo, zhi;          // the columns of a row a load may touch: z is clamped into [zlo, zhi]
    // In array coordinates: I, the sites the energy sums over and the flux lives on (the
    // lattice's interior: [2, n-3] per axis for a whole lattice), and the output region, the
    // sites this launch updates (a box within I; all of I for a whole lattice).
    int ilo[3], ihi[3];
    int olo[3], ohi[3];
    int tiles_z, tiles_y;  // output tiles of the (y, z) plane
    int zstart;            // z of the first tile's first column (at most olo[2]; below it for line-aligned tiles)
    int xchunk;            // planes per slab (the work order's outer unit)
    int units, per_block;  // batched sweeps (instead of xchunk): units of planes, and units of one block
    int unit_len;          // planes of a unit (a tile that was set: one slab each), 0 for units of one length
    int projected;     // MODE_GRAD: write g - (g.phi) phi instead of g
    int baryon;        // accumulate the baryon density
    double h, dt;
    double m, m_y, m_z, m_w;  // potential masses
    double c6;                // sextic (BPS-Skyrme) coefficient
    int gradient_flow;        // MODE_STEP: phi += dt F, no velocity
    int stream;               // STREAM_*: chooses the step kernel (host only)
};

// stencil coefficients (Sec. 3)
//   D f  = ( 2/3 (f[+1] - f[-1]) - 1/12 (f[+2] - f[-2]) ) / h
//   L f  = ( 4/3 (f[+1] + f[-1]) - 1/12 (f[+2] + f[-2]) - 5/2 f ) / h^2
//        = ( 4/3 ((f[+1] - f) + (f[-1] - f)) - 1/12 ((f[+2] - f) + (f[-2] - f)) ) / h^2
template <typename T> struct Coef {
    static constexpr T c1 = T(2.0 / 3.0);
    static constexpr T c2 = T(-1.0 / 12.0);
    static constexpr T d1 = T(4.0 / 3.0);
    static constexpr T d2 = T(-1.0 / 12.0);
    static constexpr T d0 = T(-5.0 / 2.0);
};

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// 1/sqrt(s) for s near 1 (a renormalisation): the hardware reciprocal square root,
// without the denormal rescaling rsqrtf wraps around it
__device__ __forceinline__ float rnorm(float s) { return __builtin_amdgcn_rsqf(s); }
__device__ __forceinline__ double rnorm(double s) { return 1.0 / sqrt(s); }

// Field access by a 32-bit byte offset from a base that is uniform over the block: the
// offset stays in one VGPR and the base in SGPRs (no 64-bit address arithmetic per
// access).  Kernel arguments are known to be global, uniform pointers; pointers read
// from a batch's job table are made so explicitly (uniform_ptr, global address space).
#define SKYR_GLOBAL __attribute__((address_space(1)))
template <typename T> using gptr = SKYR_GLOBAL T*;
template <bool GLOBAL, typename T> using fptr = std::conditional_t<GLOBAL, gptr<T>, T*>;

template <typename T> __device__ __forceinline__ T ldb(const T* base, unsigned off)
{
    return *(const T*)((const char*)base + off);
}
template <typename T> __device__ __forceinline__ void stb(T* base, unsigned off, T v)
{
    *(T*)((char*)base + off) = v;
}
template <typename T> __device__ __forceinline__ T ldb(gptr<const T> base, unsigned off)
{
    return *(gptr<const T>)((SKYR_GLOBAL const char*)base + off);
}
// The accesses used once per sweep (the velocity read, the outputs written), by cache policy.
template <int STREAM, typename T> __device__ __forceinline__ T ld_once(gptr<const T> base, unsigned off)
{
    const gptr<const T> p = (gptr<const T>)((SKYR_GLOBAL const char*)base + off);
    if constexpr (STREAM >= STREAM_ALL) return __builtin_nontemporal_load(p);
    return *p;
}
template <int STREAM, typename T> __device__ __forceinline__ void st_once(gptr<T> base, unsigned off, T v)
{
    const gptr<T> p = (gptr<T>)((SKYR_GLOBAL char*)base + off);
    if constexpr (STREAM >= STREAM_STORES)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// a pointer that is the same in every lane, made visibly uniform (held in SGPRs)
template <typename P> __device__ __forceinline__ P uniform_ptr(P p)
{
    const unsigned long long u = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return (P)(((unsigned long long)hi << 32) | lo);
}

// max of two non-negative values (or NaN): for floats the unsigned order of the bit
// patterns is the numeric order, and a NaN pattern exceeds +inf
__device__ __forceinline__ float fmax_nonneg(float a, float b)
{
    return __uint_as_float(max(__float_as_uint(a), __float_as_uint(b)));
}
__device__ __forceinline__ double fmax_nonneg(double a, double b) { return fmax(a, b); }

template <typename T> __device__ __forceinline__ T dot4(const T* a, const T* b)
{
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + a[3] * b[3];
}

// det[c0 c1 c2 c3] of four column 4-vectors (expansion by 2x2 minors)
template <typename T> __device__ __forceinline__ T det4(const T* c0, const T* c1, const T* c2, const T* c3)
{
    // minors of columns (c0, c1) and (c2, c3) over row pairs
    const T m01 = c0[0] * c1[1] - c0[1] * c1[0];
    const T m02 = c0[0] * c1[2] - c0[2] * c1[0];
    const T m03 = c0[0] * c1[3] - c0[3] * c1[0];
    const T m12 = c0[1] * c1[2] - c0[2] * c1[1];
    const T m13 = c0[1] * c1[3] - c0[3] * c1[1];
    const T m23 = c0[2] * c1[3] - c0[3] * c1[2];
    const T n01 = c2[0] * c3[1] - c2[1] * c3[0];
    const T n02 = c2[0] * c3[2] - c2[2] * c3[0];
    const T n03 = c2[0] * c3[3] - c2[3] * c3[0];
    const T n12 = c2[1] * c3[2] - c2[2] * c3[1];
    const T n13 = c2[1] * c3[3] - c2[3] * c3[1];
    const T n23 = c2[2] * c3[3] - c2[3] * c3[2];
    return m01 * n23 - m02 * n13 + m03 * n12 + m12 * n03 - m13 * n02 + m23 * n01;
}

// det[c0 c1 c2 c3] and its derivatives with respect to each column (det is linear in
// every column; the derivative with respect to column k is the cofactor vector),
// from the 2x2 minors m of columns (c0, c1) and n of columns (c2, c3):
//   det = m01 n23 - m02 n13 + m03 n12 + m12 n03 - m13 n02 + m23 n01
template <typename T>
__device__ __forceinline__ T det4_cofactors(const T* c0, const T* c1, const T* c2, const T* c3, T* d0, T* d1, T* d2,
                                            T* d3)
{
    const T m01 = c0[0] * c1[1] - c0[1] * c1[0], m02 = c0[0] * c1[2] - c0[2] * c1[0];
    const T m03 = c0[0] * c1[3] - c0[3] * c1[0], m12 = c0[1] * c1[2] - c0[2] * c1[1];
    const T m13 = c0[1] * c1[3] - c0[3] * c1[1], m23 = c0[2] * c1[3] - c0[3] * c1[2];
    const T n01 = c2[0] * c3[1] - c2[1] * c3[0], n02 = c2[0] * c3[2] - c2[2] * c3[0];
    const T n03 = c2[0] * c3[3] - c2[3] * c3[0], n12 = c2[1] * c3[2] - c2[2] * c3[1];
    const T n13 = c2[1] * c3[3] - c2[3] * c3[1], n23 = c2[2] * c3[3] - c2[3] * c3[2];
    // d det / d m_ab and d det / d n_ab are the complementary minors with the signs above
    const T M01 = n23, M02 = -n13, M03 = n12, M12 = n03, M13 = -n02, M23 = n01;
    const T N23 = m01, N13 = -m02, N12 = m03, N03 = m12, N02 = -m13, N01 = m23;
    // m_ab = c0_a c1_b - c0_b c1_a:  d/dc0_a = c1_b (and -c1_a for d/dc0_b); d/dc1 likewise
    d0[0] = M01 * c1[1] + M02 * c1[2] + M03 * c1[3];
    d0[1] = -M01 * c1[0] + M12 * c1[2] + M13 * c1[3];
    d0[2] = -M02 * c1[0] - M12 * c1[1] + M23 * c1[3];
    d0[3] = -M03 * c1[0] - M13 * c1[1] - M23 * c1[2];
    d1[0] = -M01 * c0[1] - M02 * c0[2] - M03 * c0[3];
    d1[1] = M01 * c0[0] - M12 * c0[2] - M13 * c0[3];
    d1[2] = M02 * c0[0] + M12 * c0[1] - M23 * c0[3];
    d1[3] = M03 * c0[0] + M13 * c0[1] + M23 * c0[2];
    d2[0] = N01 * c3[1] + N02 * c3[2] + N03 * c3[3];
    d2[1] = -N01 * c3[0] + N12 * c3[2] + N13 * c3[3];
    d2[2] = -N02 * c3[0] - N12 * c3[1] + N23 * c3[3];
    d2[3] = -N03 * c3[0] - N13 * c3[1] - N23 * c3[2];
    d3[0] = -N01 * c2[1] - N02 * c2[2] - N03 * c2[3];
    d3[1] = N01 * c2[0] - N12 * c2[2] - N13 * c2[3];
    d3[2] = N02 * c2[0] + N12 * c2[1] - N23 * c2[3];
    d3[3] = N03 * c2[0] + N13 * c2[1] + N23 * c2[2];
    return m01 * n23 - m02 * n13 + m03 * n12 + m12 * n03 - m13 * n02 + m23 * n01;
}

// fused multiply-add in the field type
__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

// A plane of N sites of four components in LDS.  Every access moves 16 bytes per lane with
// neighbouring lanes 16 bytes apart: one for a float site; two for a double site, whose
// component pairs lie in two arrays.  (Whole 32-byte records put the lanes of one access 32
// bytes apart, on half of the banks: 53% of the LDS cycles of the double sweep were conflicts.)
template <typename T, int N> struct SitePlane;
template <int N> struct SitePlane<float, N> {
    float4 s[N];
    __device__ __forceinline__ void ld(int i, float (&o)[4]) const
    {
        const float4 t = s[i];
        o[0] = t.x, o[1] = t.y, o[2] = t.z, o[3] = t.w;
    }
    __device__ __forceinline__ void st(int i, const float (&v)[4]) { s[i] = make_float4(v[0], v[1], v[2], v[3]); }
};
template <int N> struct SitePlane<double, N> {
    double2 s[2][N];
    __device__ __forceinline__ void ld(int i, double (&o)[4]) const
    {
        const double2 a = s[0][i], b = s[1][i];
        o[0] = a.x, o[1] = a.y, o[2] = b.x, o[3] = b.y;
    }
    __device__ __forceinline__ void st(int i, const double (&v)[4])
    {
        s[0][i] = make_double2(v[0], v[1]);
        s[1][i] = make_double2(v[2], v[3]);
    }
};

// Tile geometry of a shape: NWI interior waves of 64 / OZ rows of OZ lanes, NWH halo
// waves whose lanes hold HPT halo positions each.
template <int NWI_, int NWH_, int HPT_, int OZ_> struct Geo {
    static constexpr int NWI = NWI_, NWH = NWH_, HPT = HPT_, OZ = OZ_;
    static constexpr int NW = NWI + NWH;
    static constexpr int THREADS = NW * 64;
    static constexpr int RPW = 64 / OZ;
    static constexpr int OY = NWI * RPW;
    // halo positions: rows -2, -1, OY, OY+1 over the OZ columns (they supply Q_y), then
    // columns -2, -1, OZ, OZ+1 of the OY rows (they supply Q_z)
    static constexpr int NHALO = 4 * OZ + 4 * OY;
    // frame: the phi sites only halo positions read (rows -4, -3, OY+2, OY+3 over the
    // columns; columns -4, -3, OZ+2, OZ+3 over the rows; the sixteen corner sites of the
    // halo rows and columns)
    static constexpr int NFRAME = 4 * OZ + 4 * OY + 16;
    static constexpr int PW = OZ + 8, PH = OY + 8;  // phi plane: rows -4 .. OY+3, columns -4 .. OZ+3
    static constexpr int QW = OZ + 4, QH = OY + 4;  // flux plane: rows -2 .. OY+1, columns -2 .. OZ+1
    static constexpr int PPLANE = PH * PW, QPLANE = QH * QW;
    static_assert(64 % OZ == 0, "an interior wave covers whole rows");
    static constexpr int FPT = (NFRAME + NWH * 64 - 1) / (NWH * 64);  // frame sites per halo lane
    static_assert(NWH * 64 * HPT >= NHALO, "every halo position has a lane");
};

// A batched sweep keeps a field's sums per unit of planes; records of energy density, largest
// |F|^2 and power, at most MAX_UNITS of them from one block.  On a tile that was set a unit is a slab,
// and the sums are formed in the order of the single-field sweep: its records, bit for bit.
enum : int { U_E = 0, U_F2 = 1, U_POW = 2, UNIT_REC = 4 };

template <typename T, class G> struct SweepSmem {
    SitePlane<T, G::PPLANE> phi[2];     // [plane parity]
    SitePlane<T, 2 * G::QPLANE> q[2];   // [plane parity]: sites of Q_y, then those of Q_z
    double red[G::NW][NPART];
    double unit[MAX_UNITS - 1][G::NWI][3];  // batched sweeps: the waves' sums over the units before the last
    int unit_end[MAX_UNITS];                // and the ends of the block's units, in planes from its first
    int units_ended[G::NWI];
    int last;  // this block is the last of its field to finish the sweep
};

// EXT: 0 the plain variant (pion-mass potential, kick-drift update); 1 adds the extra
// potentials (m_y, m_z, m_w) and the gradient flow; 2 also the sextic term.  The levels
// are separate kernels so that each carries only the registers it needs.
enum : int { EXT_NONE = 0, EXT_POT = 1, EXT_SEXTIC = 2 };

// Waves per SIMD that a kernel leaves registers for: those of the blocks its shape has on a CU
// (shapes.hpp).  At 131 registers, three more than that allows, the second float shape had one block
// on a CU instead of two: 40 x 5 x 20000 sites 156 us a sweep against 120, 300 x 12 x 1500 97 against 80.
// The sextic kernels need more and have one block a CU in every shape.
template <typename T, class G, int EXT> constexpr int waves_per_simd()
{
    int blocks = 1;
    const auto look = [&](const Shape& s) {
        if (s.nwi == G::NWI && s.nwh == G::NWH && s.hpt == G::HPT && s.cols == G::OZ) blocks = s.per_cu;
    };
    if (EXT != EXT_SEXTIC) {
        if (sizeof(T) == 8)
            for (const Shape& s : kShapesF64) look(s);
        else
            for (const Shape& s : kShapesF32) look(s);
    }
    return blocks * G::NW / 4;
}

// Per-launch constants.  With a^ = 12 h a (the scaled first difference), G^ = (12 h)^2 G,
// Q^ = (12 h)^3 Q and L^ = 12 h^2 Lap, the scaled gradient g^ = K g, K = (12 h)^4, is
//   g^ = lapw (L^ phi - boundary terms) - sum_i (8 (Q^_i[+1] - Q^_i[-1]) - (Q^_i[+2] - Q^_i[-2]))
//        + K V'(phi0) e0 + (sextic local term),
// and F = F^ / K with F^ = (g^.phi) phi - g^.
template <typename T> struct SweepConst {
    T lapw;                  // -K / (12 h^2) = -1728 h^2
    T ke2, ke4;              // e2 = ke2 phi.L^phi, e4 = ke4 (G^ quadratic form)
    T dt, dtK;               // dt and dt / K
    T m2, my2, mz2, mw2;     // potential energy density (unscaled)
    T m2K, my2K, mz2K, mw2K; // the same masses times K (scaled slope)
    T c6e, c6q;              // sextic: e6 = c6e det^2, flux and local weight c6q det (det of phi, a^_i)
    T invK;                  // gradient output
    double dinvK, dinvK2, dinv12h3;  // unscale the power, |F|^2 and charge-density sums
    bool more_pot, sextic, grad_flow;

    __device__ __forceinline__ void init(const SweepArgs& a, bool step_mode)
    {
        const double h = a.h, s = 12.0 * h, K = s * s * s * s;
        lapw = T(-1728.0 * h * h);
        ke2 = T(-1.0 / (24.0 * h * h));
        ke4 = T(0.5 / K);
        dt = T(a.dt);
        dtK = T(a.dt / K);
        m2 = T(a.m * a.m);
        my2 = T(a.m_y * a.m_y);
        mz2 = T(a.m_z * a.m_z);
        mw2 = T(a.m_w * a.m_w);
        m2K = T(K * a.m * a.m);
        my2K = T(K * a.m_y * a.m_y);
        mz2K = T(K * a.m_z * a.m_z);
        mw2K = T(K * a.m_w * a.m_w);
        c6e = T(0.5 * a.c6 / (K * s * s));
        c6q = T(a.c6 / (s * s));
        invK = T(1.0 / K);
        dinvK = 1.0 / K;
        dinvK2 = 1.0 / (K * K);
        dinv12h3 = 1.0 / (s * s * s);
        more_pot = a.m_y != 0.0 || a.m_z != 0.0 || a.m_w != 0.0;
        sextic = a.c6 != 0.0;
        grad_flow = step_mode && a.gradient_flow != 0;
    }
};

// v of another lane, by cross-lane moves of the vector unit (the shuffles of a butterfly went
// through LDS, six dependent round trips a sum)
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// The last stages of a wave's sums: the lanes 16 and 32 away (a swap of two copies' rows or halves
// leaves one's in one copy and the other's in the other).  (With these stages first the block ends took
// longer: 40^3 double 5800 us for 300 steps against 5760.)
template <bool MAX> __device__ __forceinline__ double wave_rows(double v)
{
    const auto halves = [&](auto swap) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const auto lo = swap((unsigned)u), hi = swap((unsigned)(u >> 32));
        const double x = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]);
        const double y = __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
        return MAX ? fmax(x, y) : x + y;
    };
    v = halves([](unsigned u) { return __builtin_amdgcn_permlane16_swap(u, u, false, false); });
    return halves([](unsigned u) { return __builtin_amdgcn_permlane32_swap(u, u, false, false); });
}
// The sum (maximum) of v over the wave, in every lane, in a fixed order: lanes 1 and 2 away, then (the
// sums of all lanes of a quad being equal) the mirrored lanes of 8 and 16, then 16 and 32 away.
template <bool MAX> __device__ __forceinline__ double wave_total(double v)
{
    const auto add = [](double a, double b) { return MAX ? fmax(a, b) : a + b; };
    v = add(v, dpp_f64<0xb1>(v));   // quad lanes 1, 0, 3, 2
    v = add(v, dpp_f64<0x4e>(v));   // quad lanes 2, 3, 0, 1
    v = add(v, dpp_f64<0x141>(v));  // mirrored in 8 lanes
    v = add(v, dpp_f64<0x140>(v));  // mirrored in 16 lanes
    return wave_rows<MAX>(v);
}

// a and b summed over the wave (two sums for little more than one), every lane ending with both: a in
// the even lanes, b in the odd ones from the first stage on, every later stage an even number of lanes
// away.  The row is turned by 4 and by 8 lanes where wave_total mirrors it: quad 1 then adds quads 0 and
// 1, and to them quads 2 and 3, as wave_total does, so that a sum is the same from either.
__device__ __forceinline__ void wave_totals(double& a, double& b)
{
    const bool odd = threadIdx.x & 1;
    double v = (odd ? b : a) + dpp_f64<0xb1>(odd ? a : b);
    v += dpp_f64<0x4e>(v);
    v += dpp_f64<0x124>(v);
    v += dpp_f64<0x128>(v);
    const unsigned long long w = __builtin_bit_cast(unsigned long long, wave_rows<false>(v));
    const auto lane = [&](int i) {
        return __builtin_bit_cast(double, ((unsigned long long)__builtin_amdgcn_readlane((unsigned)(w >> 32), i) << 32) |
                                              (unsigned)__builtin_amdgcn_readlane((unsigned)w, i));
    };
    a = lane(4);
    b = lane(5);
}
// the largest of the non-negative v over the wave, in every lane
__device__ __forceinline__ double wave_most(double v) { return wave_total<true>(v); }
__device__ __forceinline__ float wave_most(float v)
{
    const auto other = [](float x, auto dpp) { return __builtin_bit_cast(float, dpp(__builtin_bit_cast(int, x))); };
    v = fmaxf(v, other(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0xb1, 0xf, 0xf, true); }));
    v = fmaxf(v, other(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0x4e, 0xf, 0xf, true); }));
    v = fmaxf(v, other(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true); }));
    v = fmaxf(v, other(v, [](int x) { return __builtin_amdgcn_mov_dpp(x, 0x140, 0xf, 0xf, true); }));
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = fmaxf(__builtin_bit_cast(float, (unsigned)p[0]), __builtin_bit_cast(float, (unsigned)p[1]));
    const unsigned t = __builtin_bit_cast(unsigned, v);
    const auto q = __builtin_amdgcn_permlane32_swap(t, t, false, false);
    return fmaxf(__builtin_bit_cast(float, (unsigned)q[0]), __builtin_bit_cast(float, (unsigned)q[1]));
}

// One item of a field's work: output planes [xa, xe) of tile (ty, tz).
struct Segment {
    int ty, tz, xa, xe;
};

// The work of a field is cut into items, one (slab, tile) pair each (slabs of xchunk
// planes along x), numbered slab by slab and tile by tile within a slab.  Logical block
// b of nb takes items b, b + nb, ...; a launch normally has one block per item, so that
// the blocks of neighbouring tiles march through the same planes at the same time and
// the phi lines of their shared halo are read from L2 once.
__device__ __forceinline__ Segment item_segment(int item, int tiles, int tiles_z, int x0, int nx, int xchunk)
{
    const int slab = item / tiles, tile = item - slab * tiles;
    Segment s;
    s.ty = tile / tiles_z;
    s.tz = tile - s.ty * tiles_z;
    s.xa = x0 + slab * xchunk;
    s.xe = x0 + min(nx, (slab + 1) * xchunk);
    return s;
}

// Fields, flags and sums shared by the two roles.
template <typename T, bool FROM_TABLE> struct SweepCommon {
    // global-memory pointers, uniform over the block
    gptr<const T> pin[4];
    gptr<T> pout[4];
    gptr<T> vel[4];
    gptr<T> gout[4];
    long long cs;        // bytes from one component to the next (set and read by the printed form alone)
    int n0, n1, n2;
    int zlo, zhi;        // the columns of a row a load may touch
    int ilo[3], ihi[3];  // I in array coordinates
    int olo1, olo2, ohi1, ohi2;  // the output region in y and z
    unsigned plane_b;  // bytes per x-plane of one component
    bool redo, renorm64, projected, baryon, has_grad;
    int restore;       // RESTORE_*: this sweep only rewrites the velocity

    __device__ __forceinline__ void load(unsigned off, int x, T (&dst)[4]) const
    {
        const unsigned base = (unsigned)clampi(x, 0, n0 - 1) * plane_b;
#pragma unroll
        for (int A = 0; A < 4; ++A) dst[A] = ldb(pin[A], base + off);
    }
    // component A of an array with component 0 at base: formed on the scalar unit where it is used
    // and kept there (see formp.hpp)
    template <typename P> __device__ __forceinline__ P comp(P base, int A) const
    {
        long long c = cs;
        asm volatile("" : "+s"(c));
        unsigned long long u = (unsigned long long)base + (unsigned long long)(A * c);
        asm volatile("" : "+s"(u));
        return (P)u;
    }
    __device__ __forceinline__ unsigned site_off(int y, int z) const
    {
        return (unsigned)(clampi(y, 0, n1 - 1) * n2 + clampi(z, zlo, zhi)) * (unsigned)sizeof(T);
    }
};

// --------------------------------------------------------------- interior role
// One output site per lane: row, col of the tile.
template <typename T, class G, int MODE, bool FROM_TABLE, int EXT, int STREAM> struct Interior {
    using Smem = SweepSmem<T, G>;
    Smem& sm;
    const SweepConst<T>& k;
    const SweepCommon<T, FROM_TABLE>& cm;
    int row, col;
    // LDS index of the site two rows above the own one in a phi plane and in a flux plane: every
    // neighbour then lies at a non-negative constant offset, which the access itself adds
    int pidx, qidx;
    static constexpr int PO = 2 * G::PW, QO = 2 * G::QW;  // the own site from there
    unsigned off;      // byte offset of the own site within a plane
    int xa, xe;
    bool out;          // the own site is in the output region (in y and z)
    bool in_i;         // the own site is in I (in y and z); the flux there is not zero
    // uniform over the wave: it has an output site within two sites of a y face / of a z face of I
    bool wave_y_near, wave_z_near;
    unsigned outside;  // bit d: the y/z neighbour d (O_* below) lies outside I
    enum : unsigned { O_YP1 = 1, O_YM1 = 2, O_YP2 = 4, O_YM2 = 8, O_ZP1 = 16, O_ZM1 = 32, O_ZP2 = 64, O_ZM2 = 128 };

    T ring[5][4];  // phi of planes j-2 .. j+2 (slot = plane offset + 2 + step, mod 5)
    T acc[5][4];   // scaled gradient accumulators of planes j-2 .. j+2 (same slots)
    T nxt[4];      // prefetched phi(j+3)
    T vnxt[4];     // prefetched velocity of plane j-1

    double pe2 = 0.0, pe4 = 0.0, pe0 = 0.0, pe6 = 0.0, pb_sum = 0.0;
    T elate[2] = {T(0), T(0)};  // batched sweeps: the energy density of planes j-1, j-2
    double pp = 0.0;  // scaled power F^ . v of the incoming velocity
    T pf2 = T(0);     // largest scaled |F^|^2

    __device__ __forceinline__ Interior(Smem& s, const SweepConst<T>& kk, const SweepCommon<T, FROM_TABLE>& c, int tid)
        : sm(s), k(kk), cm(c)
    {
        row = tid / G::OZ;
        col = tid - row * G::OZ;
        pidx = (row + 2) * G::PW + col + 4;
        qidx = row * G::QW + col + 2;
    }

    __device__ __forceinline__ T potential(T p0) const
    {
        const T u = T(1) - p0;
        T v = k.m2 * u;
        if constexpr (EXT) {
            if (k.more_pot)
                v += T(0.5) * k.my2 * (T(1) - p0 * p0) + T(0.5) * k.mz2 * u * u + T(0.25) * k.mw2 * (u * u) * (u * u);
        }
        return v;
    }
    // K dV/dphi0
    __device__ __forceinline__ T slopeK(T p0) const
    {
        const T u = T(1) - p0;
        T d = -k.m2K;
        if constexpr (EXT) {
            if (k.more_pot) d -= k.my2K * p0 + k.mz2K * u + k.mw2K * u * u * u;
        }
        return d;
    }

    __device__ __forceinline__ void setup(const Segment& s, int tiles_z_start)
    {
        const int y0 = cm.olo1 + s.ty * G::OY, z0 = tiles_z_start + s.tz * G::OZ;
        const int y = y0 + row, z = z0 + col;
        const int ly = cm.ilo[1], hy = cm.ihi[1], lz = cm.ilo[2], hz = cm.ihi[2];
        out = (y <= cm.ohi1) && (z >= cm.olo2) && (z <= cm.ohi2);
        in_i = (y >= ly) && (y <= hy) && (z >= lz) && (z <= hz);
        outside = (y + 1 > hy ? O_YP1 : 0u) | (y - 1 < ly ? O_YM1 : 0u) | (y + 2 > hy ? O_YP2 : 0u) |
                  (y - 2 < ly ? O_YM2 : 0u) | (z + 1 > hz ? O_ZP1 : 0u) | (z - 1 < lz ? O_ZM1 : 0u) |
                  (z + 2 > hz ? O_ZP2 : 0u) | (z - 2 < lz ? O_ZM2 : 0u);
        wave_y_near = __builtin_amdgcn_ballot_w64(out && (outside & (O_YP1 | O_YM1 | O_YP2 | O_YM2))) != 0;
        wave_z_near = __builtin_amdgcn_ballot_w64(out && (outside & (O_ZP1 | O_ZM1 | O_ZP2 | O_ZM2))) != 0;
        off = cm.site_off(y, z);
        xa = s.xa;
        xe = s.xe;
    }

    // The terms of Lap phi whose neighbour lies outside I, from the neighbours read for the
    // derivatives.  Every axis is a branch of its own, taken only by waves with a site within two
    // of a face of that axis: the tiles at the z faces run the z terms on every plane and are the
    // last blocks of a launch to end, so they must not pay for the other axes as well (four
    // selects and two sums per component against sixteen and ten).  Measured: the double sweep
    // of 256^3 505 -> 482 us, of 40^3 50.2 -> 47.4; the float one of 96^3 with the sextic term 55 -> 52.
    template <int SM2, int SM1, int S0, int SP1, int SP2>
    __device__ __forceinline__ void boundary_terms(int j, bool x_near, const T (&Ym2)[4], const T (&Ym1)[4],
                                                   const T (&Yp1)[4], const T (&Yp2)[4], const T (&Zm2)[4],
                                                   const T (&Zm1)[4], const T (&Zp1)[4], const T (&Zp2)[4])
    {
        const auto pick = [](bool c, T v) { return c ? v : T(0); };
        T o1[4], o2[4];  // sums of the outside first / second neighbours
#pragma unroll
        for (int A = 0; A < 4; ++A) o1[A] = o2[A] = T(0);
        if (x_near) {
            const int lx = cm.ilo[0], hx = cm.ihi[0];
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                o1[A] = pick(j + 1 > hx, ring[SP1][A]) + pick(j - 1 < lx, ring[SM1][A]);
                o2[A] = pick(j + 2 > hx, ring[SP2][A]) + pick(j - 2 < lx, ring[SM2][A]);
            }
        }
        if (wave_y_near) {
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                o1[A] = (o1[A] + pick(outside & O_YP1, Yp1[A])) + pick(outside & O_YM1, Ym1[A]);
                o2[A] = (o2[A] + pick(outside & O_YP2, Yp2[A])) + pick(outside & O_YM2, Ym2[A]);
            }
        }
        if (wave_z_near) {
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                o1[A] = (o1[A] + pick(outside & O_ZP1, Zp1[A])) + pick(outside & O_ZM1, Zm1[A]);
                o2[A] = (o2[A] + pick(outside & O_ZP2, Zp2[A])) + pick(outside & O_ZM2, Zm2[A]);
            }
        }
        // + 1/2 the outside terms of Lap phi: 12 h^2 x that is 8 o1 - o2 / 2, and L^ enters the
        // scaled gradient with weight lapw < 0 and the opposite sign (zero at sites without such
        // neighbours, and unused outside the output region)
#pragma unroll
        for (int A = 0; A < 4; ++A) acc[S0][A] = fmaT(k.lapw, fmaT(T(0.5), o2[A], T(-8) * o1[A]), acc[S0][A]);
    }

    template <int U> __device__ __forceinline__ void step(int j, int pb)
    {
        constexpr int SM2 = U % 5, SM1 = (U + 1) % 5, S0 = (U + 2) % 5, SP1 = (U + 3) % 5, SP2 = (U + 4) % 5;
        const int qb = pb ^ 1;
        // Opaque to the optimiser from here on: the LDS and global addresses and the x-stencil
        // arithmetic of this plane are then formed within it, not carried over from an
        // earlier plane in registers across the barriers.
        asm volatile("" : "+v"(pidx), "+v"(qidx), "+v"(off));
#pragma unroll
        for (int sl = 0; sl < 5; ++sl)
            asm volatile("" : "+v"(ring[sl][0]), "+v"(ring[sl][1]), "+v"(ring[sl][2]), "+v"(ring[sl][3]));
        // stage phi(j+1) into the other phi buffer (its last reads, of phi(j-1), came before
        // the last barrier), then prefetch
        sm.phi[qb].st(pidx + PO, ring[SP1]);
        // the velocity of output plane j-2 was prefetched one plane earlier; the velocity of
        // plane j-1 is loaded now, before the prefetch of phi(j+3) (loads complete in order)
        T vcur[4];
        if constexpr (MODE == MODE_STEP) {
            const unsigned vb = (unsigned)clampi(j - 1, 0, cm.n0 - 1) * cm.plane_b;
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                vcur[A] = vnxt[A];
                vnxt[A] = ld_once<STREAM>((gptr<const T>)cm.vel[A], vb + off);
            }
        }
#pragma unroll
        for (int A = 0; A < 4; ++A) ring[SP2][A] = nxt[A];
        cm.load(off, j + 3, nxt);
        if constexpr (MODE == MODE_STEP) {
            if (cm.redo) {  // a redo sweep starts from zero velocity
#pragma unroll
                for (int A = 0; A < 4; ++A) vcur[A] = T(0);
            }
        }
        const bool j_in = (j >= cm.ilo[0]) && (j <= cm.ihi[0]);
        const bool j_out = (j >= xa) && (j < xe);

        const auto& P = sm.phi[pb];
        T c[4], ax[4], ay[4], az[4];
        T Ym2[4], Ym1[4], Yp1[4], Yp2[4], Zm2[4], Zm1[4], Zp1[4], Zp2[4];
        P.ld(pidx + (PO - 2 * G::PW), Ym2);
        P.ld(pidx + (PO - G::PW), Ym1);
        P.ld(pidx + (PO + G::PW), Yp1);
        P.ld(pidx + (PO + 2 * G::PW), Yp2);
        P.ld(pidx + (PO - 2), Zm2);
        P.ld(pidx + (PO - 1), Zm1);
        P.ld(pidx + (PO + 1), Zp1);
        P.ld(pidx + (PO + 2), Zp2);
        T cl = T(0);
#pragma unroll
        for (int A = 0; A < 4; ++A) {
            const T cc = ring[S0][A];
            const T xm2 = ring[SM2][A], xm1 = ring[SM1][A], xp1 = ring[SP1][A], xp2 = ring[SP2][A];
            const T ym2 = Ym2[A], ym1 = Ym1[A], yp1 = Yp1[A], yp2 = Yp2[A];
            const T zm2 = Zm2[A], zm1 = Zm1[A], zp1 = Zp1[A], zp2 = Zp2[A];
            c[A] = cc;
            ax[A] = fmaT(T(8), xp1 - xm1, xm2 - xp2);
            ay[A] = fmaT(T(8), yp1 - ym1, ym2 - yp2);
            az[A] = fmaT(T(8), zp1 - zm1, zm2 - zp2);
            // (formed on every plane of the march: beside the output planes it reaches no
            // accumulator that is read)
            T lap;  // 12 h^2 Lap phi
            if constexpr (sizeof(T) == 4) {
                // differences from the centre: no cancellation of O(1) terms in single precision
                const T s1 = ((xp1 - cc) + (xm1 - cc)) + ((yp1 - cc) + (ym1 - cc)) + ((zp1 - cc) + (zm1 - cc));
                const T s2 = ((xp2 - cc) + (xm2 - cc)) + ((yp2 - cc) + (ym2 - cc)) + ((zp2 - cc) + (zm2 - cc));
                lap = fmaT(T(16), s1, -s2);
            } else {
                const T s1 = ((xp1 + xm1) + (yp1 + ym1)) + (zp1 + zm1);
                const T s2 = ((xp2 + xm2) + (yp2 + ym2)) + (zp2 + zm2);
                lap = fmaT(T(-90), cc, fmaT(T(16), s1, -s2));
            }
            cl = fmaT(cc, lap, cl);
            acc[S0][A] = fmaT(k.lapw, lap, acc[S0][A]);
        }
        // The E2 part of the gradient is -1/2 (Lap phi + Lap(1_I phi)): the terms of Lap phi
        // whose neighbour lies outside I count half.  Only sites within two of a face of I
        // have such terms; a wave none of whose sites has one skips this.
        const bool x_near = (j <= cm.ilo[0] + 1) || (j >= cm.ihi[0] - 1);
        if (j_out && (x_near || wave_y_near || wave_z_near))
            boundary_terms<SM2, SM1, S0, SP1, SP2>(j, x_near, Ym2, Ym1, Yp1, Yp2, Zm2, Zm1, Zp1, Zp2);

        const T gxx = dot4(ax, ax), gyy = dot4(ay, ay), gzz = dot4(az, az);
        const T gxy = dot4(ax, ay), gxz = dot4(ax, az), gyz = dot4(ay, az);
        const bool valid = in_i && j_in;
        // the flux vanishes outside I: zero the Gram entries it is built from
        const T fxx = valid ? gxx : T(0), fyy = valid ? gyy : T(0), fzz = valid ? gzz : T(0);
        const T fxy = valid ? gxy : T(0), fxz = valid ? gxz : T(0), fyz = valid ? gyz : T(0);
        const T sx = fyy + fzz, sy = fxx + fzz, sz = fxx + fyy;
        T qx[4], qy[4], qz[4];
#pragma unroll
        for (int A = 0; A < 4; ++A) {
            qx[A] = fmaT(sx, ax[A], -fmaT(fxy, ay[A], fxz * az[A]));
            qy[A] = fmaT(sy, ay[A], -fmaT(fxy, ax[A], fyz * az[A]));
            qz[A] = fmaT(sz, az[A], -fmaT(fxz, ax[A], fyz * ay[A]));
        }
        T e6 = T(0);
        if constexpr (EXT == EXT_SEXTIC) {
            if (k.sextic) {
                // e6 = c6 det^2 / 2, det = det[phi, a_x, a_y, a_z]: flux c6 det ddet/da_i (zero
                // outside I) and the local term c6 det ddet/dphi
                T C0[4], C1[4], C2[4], C3[4];
                const T det = det4_cofactors(c, ax, ay, az, C0, C1, C2, C3);
                const T dv = valid ? k.c6q * det : T(0);
#pragma unroll
                for (int A = 0; A < 4; ++A) {
                    qx[A] = fmaT(dv, C1[A], qx[A]);
                    qy[A] = fmaT(dv, C2[A], qy[A]);
                    qz[A] = fmaT(dv, C3[A], qz[A]);
                    acc[S0][A] = fmaT(dv, C0[A], acc[S0][A]);
                }
                e6 = k.c6e * det * det;
            }
        }
        sm.q[pb].st(qidx + QO, qy);
        sm.q[pb].st(qidx + (QO + G::QPLANE), qz);
#pragma unroll
        for (int A = 0; A < 4; ++A) {
            // x-divergence pushed to the accumulators of planes j-2 .. j+2
            acc[SM1][A] = fmaT(T(-8), qx[A], acc[SM1][A]);
            acc[SP1][A] = fmaT(T(8), qx[A], acc[SP1][A]);
            acc[SM2][A] += qx[A];
            acc[SP2][A] -= qx[A];
        }
        T ecur = T(0);
        if (out && j_out) {
            const T e2 = k.ke2 * cl;
            const T quartic = gxx * gyy + gxx * gzz + gyy * gzz - gxy * gxy - gxz * gxz - gyz * gyz;
            const T e4 = k.ke4 * quartic;
            const T e0 = potential(c[0]);
            if constexpr (MODE == MODE_STEP) {
                // The flow needs the total energy only.  In single precision it is written out which of
                // the two products is rounded: left to the compiler it changed with the code around it,
                // and with it the energy of a field by some 1e-10.
                const T e24 = sizeof(T) == 4 ? fmaT(k.ke4, quartic, e2) : e2 + e4;
                if constexpr (FROM_TABLE) ecur = e24 + e0 + e6;
                else pe2 += (double)(e24 + e0 + e6);
            } else {
                pe2 += (double)e2;
                pe4 += (double)e4;
                pe0 += (double)e0;
                pe6 += (double)e6;
                if (cm.baryon) pb_sum += (double)det4(c, ax, ay, az);
            }
        }

        // y- and z-divergence of the flux of plane j-1 (written before the last barrier)
        if (j - 1 >= xa && j - 1 < xe) {
            const auto& F = sm.q[qb];
            T ym2[4], ym1[4], yp1[4], yp2[4], zm2[4], zm1[4], zp1[4], zp2[4];
            F.ld(qidx + (QO - 2 * G::QW), ym2);
            F.ld(qidx + (QO - G::QW), ym1);
            F.ld(qidx + (QO + G::QW), yp1);
            F.ld(qidx + (QO + 2 * G::QW), yp2);
            F.ld(qidx + (QO + G::QPLANE - 2), zm2);
            F.ld(qidx + (QO + G::QPLANE - 1), zm1);
            F.ld(qidx + (QO + G::QPLANE + 1), zp1);
            F.ld(qidx + (QO + G::QPLANE + 2), zp2);
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                const T t = (ym1[A] - yp1[A]) + (zm1[A] - zp1[A]);
                const T u = (yp2[A] - ym2[A]) + (zp2[A] - zm2[A]);
                acc[SM1][A] = fmaT(T(8), t, acc[SM1][A]) + u;
            }
        }

        // output plane j-2 is complete
        if (j - 2 >= xa && j - 2 < xe && out) {
            const unsigned base = (unsigned)(j - 2) * cm.plane_b + off;
            T g[4], p[4], f[4];
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                g[A] = acc[SM2][A];
                p[A] = ring[SM2][A];
            }
            g[0] += slopeK(p[0]);
            const T gp = dot4(g, p);
#pragma unroll
            for (int A = 0; A < 4; ++A) f[A] = fmaT(gp, p[A], -g[A]);  // F^ = (g^.phi) phi - g^
            pf2 = fmax_nonneg(pf2, dot4(f, f));
            if constexpr (MODE == MODE_STEP) {
                if constexpr (FROM_TABLE) pe2 += (double)elate[1];
                pp += (double)dot4(f, vcur);  // the product in the field precision, the sum in double
                if (cm.restore) {
#pragma unroll
                    for (int A = 0; A < 4; ++A)
                        st_once<STREAM>(cm.vel[A], base, cm.restore == RESTORE_ZERO ? T(0) : fmaT(-k.dtK, f[A], vcur[A]));
                } else {
                    T v[4], q[4], pn[4];
#pragma unroll
                    for (int A = 0; A < 4; ++A) {
                        if constexpr (EXT) {
                            v[A] = k.grad_flow ? T(0) : fmaT(k.dtK, f[A], vcur[A]);
                            q[A] = k.grad_flow ? fmaT(k.dtK, f[A], p[A]) : fmaT(k.dt, v[A], p[A]);
                        } else {
                            v[A] = fmaT(k.dtK, f[A], vcur[A]);
                            q[A] = fmaT(k.dt, v[A], p[A]);
                        }
                    }
                    if (cm.renorm64) {
                        const double s2 = (double)q[0] * q[0] + (double)q[1] * q[1] + (double)q[2] * q[2] +
                                          (double)q[3] * q[3];
                        const double inv = 1.0 / sqrt(s2);
#pragma unroll
                        for (int A = 0; A < 4; ++A) pn[A] = T((double)q[A] * inv);
                    } else {
                        const T inv = rnorm(dot4(q, q));
#pragma unroll
                        for (int A = 0; A < 4; ++A) pn[A] = q[A] * inv;
                    }
#pragma unroll
                    for (int A = 0; A < 4; ++A) {
                        st_once<STREAM>(cm.pout[A], base, pn[A]);
                        st_once<STREAM>(cm.vel[A], base, v[A]);
                    }
                }
            } else {
                if (cm.has_grad) {
#pragma unroll
                    for (int A = 0; A < 4; ++A) st_once<STREAM>(cm.gout[A], base, (cm.projected ? -f[A] : g[A]) * k.invK);
                }
            }
        }
#pragma unroll
        for (int A = 0; A < 4; ++A) acc[SM2][A] = T(0);  // the slot starts plane j+3
        if constexpr (FROM_TABLE) {
            elate[1] = elate[0];
            elate[0] = ecur;
        }
        __syncthreads();
    }

    // A block of a batched sweep marches through one or more units of planes and keeps the sums of
    // each apart, so that a field's sums do not depend on how its planes are cut into blocks: when
    // every unit but the last has ended, before step k units + 4, the wave's sums go to shared memory
    // and start anew.  `ev` is the next such step or the end of the march, and all that the march
    // itself looks at.  (The energy of a plane is added two planes late, with its force, so that a
    // unit ends once.)  It costs 0.5% of the march at 16 planes a unit.
    __device__ __forceinline__ bool at_event(int st, int& ev)
    {
        if constexpr (FROM_TABLE) {
            int last = xe;  // (formed here, not kept through the march)
            asm volatile("" : "+s"(last));
            if (st >= last - xa + 4) return true;
            const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            const int u = __builtin_amdgcn_readfirstlane(sm.units_ended[wave]);
            double e = pe2, p = pp * k.dinvK;
            wave_totals(e, p);
            const T f = wave_most(pf2);
            if ((threadIdx.x & 63) == 0) {
                sm.unit[u][wave][U_E] = e;
                sm.unit[u][wave][U_F2] = (double)f * k.dinvK2;
                sm.unit[u][wave][U_POW] = p;
                sm.units_ended[wave] = u + 1;
            }
            pe2 = pp = 0.0;
            pf2 = T(0);
            ev = next_event(u + 1);
            return false;
        } else {
            return true;
        }
    }
    // the step before which unit k has ended, or the end of the march for the last
    __device__ __forceinline__ int next_event(int k) const
    {
        return __builtin_amdgcn_readfirstlane(sm.unit_end[k]) + 4;
    }

    // the march over one segment
    __device__ __forceinline__ void march()
    {
#pragma unroll
        for (int s = 0; s < 5; ++s)
#pragma unroll
            for (int A = 0; A < 4; ++A) acc[s][A] = T(0);
        // The march is unrolled five planes deep and leaves the group at its last plane: rounding it
        // up to whole groups cost two planes in the mean, 12% of a 16-plane slab (40^3 double, two
        // 18-plane slabs: 47 -> 43.5 us).
        const int js = xa - 2;  // first flux plane; ring slots 0 .. 3 hold planes js-2 .. js+1
        cm.load(off, js - 2, ring[0]);
        cm.load(off, js - 1, ring[1]);
        cm.load(off, js, ring[2]);
        cm.load(off, js + 1, ring[3]);
        cm.load(off, js + 2, nxt);
        if constexpr (MODE == MODE_STEP) {
            const unsigned vb = (unsigned)clampi(js - 2, 0, cm.n0 - 1) * cm.plane_b;
#pragma unroll
            for (int A = 0; A < 4; ++A) vnxt[A] = ld_once<STREAM>((gptr<const T>)cm.vel[A], vb + off);
        }
        sm.phi[0].st(pidx + PO, ring[2]);
        __syncthreads();
        const int nst = (xe - xa) + 4;
        int ev = FROM_TABLE ? next_event(0) : nst;
        for (int st = 0;; st += 5) {
            const int j = js + st, pb = st & 1;
            step<0>(j, pb);
            if (st + 1 >= ev && at_event(st + 1, ev)) break;
            step<1>(j + 1, pb ^ 1);
            if (st + 2 >= ev && at_event(st + 2, ev)) break;
            step<2>(j + 2, pb);
            if (st + 3 >= ev && at_event(st + 3, ev)) break;
            step<3>(j + 3, pb ^ 1);
            if (st + 4 >= ev && at_event(st + 4, ev)) break;
            step<4>(j + 4, pb);
            if (st + 5 >= ev && at_event(st + 5, ev)) break;
        }
    }
};

// ------------------------------------------------------------------ halo role
// HPT halo positions per lane; each supplies one flux component: Q_y on the y-halo
// rows, Q_z on the z-halo columns.
template <typename T, class G, bool FROM_TABLE, int EXT> struct Halo {
    using Smem = SweepSmem<T, G>;
    static constexpr int HPT = G::HPT;
    Smem& sm;
    const SweepConst<T>& k;
    const SweepCommon<T, FROM_TABLE>& cm;
    int pos[HPT];        // halo position index (>= NHALO: none)
    int pidx[HPT];       // LDS index in a phi plane of the site two rows above
    int qidx[HPT];       // LDS index of the supplied flux (Q_y or Q_z plane, component 0)
    unsigned off[HPT];
    bool active[HPT], is_y[HPT], vyz[HPT];
    int hr[HPT], hc[HPT];  // tile-relative row and column
    static constexpr int FPT = G::FPT;
    bool floader[FPT];     // frame sites of this lane
    int fr[FPT], fc[FPT];  // their tile-relative rows and columns
    int fidx[FPT];         // LDS index in a phi plane
    unsigned foff[FPT];    // byte offset in the current segment
    int xa, xe;
    T ring[HPT][5][4];
    T nxt[HPT][4];
    T fnxt[FPT][4];        // prefetched frame sites of phi(j+2)

    __device__ __forceinline__ Halo(Smem& s, const SweepConst<T>& kk, const SweepCommon<T, FROM_TABLE>& c, int u)
        : sm(s), k(kk), cm(c)
    {
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            const int p = u + i * G::NWH * 64;
            active[i] = p < G::NHALO;
            const int pp = active[i] ? p : 0;
            int r, cc;
            bool yh;
            if (pp < 4 * G::OZ) {
                const int q = pp / G::OZ;
                r = q < 2 ? q - 2 : G::OY + q - 2;
                cc = pp - q * G::OZ;
                yh = true;
            } else {
                const int g = pp - 4 * G::OZ, q = g & 3;
                r = g >> 2;
                cc = q < 2 ? q - 2 : G::OZ + q - 2;
                yh = false;
            }
            hr[i] = r;
            hc[i] = cc;
            is_y[i] = yh;
            pidx[i] = (r + 2) * G::PW + cc + 4;
            qidx[i] = (yh ? 0 : G::QPLANE) + (r + 2) * G::QW + cc + 2;
        }
#pragma unroll
        for (int i = 0; i < FPT; ++i) {
            const int f0 = u + i * G::NWH * 64;
            floader[i] = f0 < G::NFRAME;
            const int f = floader[i] ? f0 : 0;
            int r, cc;
            if (f < 4 * G::OZ) {
                const int q = f / G::OZ;
                r = q < 2 ? q - 4 : G::OY + q;
                cc = f - q * G::OZ;
            } else if (f < 4 * G::OZ + 4 * G::OY) {
                const int g = f - 4 * G::OZ, q = g & 3;
                r = g >> 2;
                cc = q < 2 ? q - 4 : G::OZ + q;
            } else {
                const int g = f - 4 * G::OZ - 4 * G::OY, qr = g >> 2, qc = g & 3;
                r = qr < 2 ? qr - 2 : G::OY + qr - 2;
                cc = qc < 2 ? qc - 2 : G::OZ + qc - 2;
            }
            fr[i] = r;
            fc[i] = cc;
            fidx[i] = (r + 4) * G::PW + cc + 4;
        }
    }

    __device__ __forceinline__ void setup(const Segment& s, int tiles_z_start)
    {
        const int y0 = cm.olo1 + s.ty * G::OY, z0 = tiles_z_start + s.tz * G::OZ;
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            const int y = y0 + hr[i], z = z0 + hc[i];
            vyz[i] = (y >= cm.ilo[1]) && (y <= cm.ihi[1]) && (z >= cm.ilo[2]) && (z <= cm.ihi[2]);
            off[i] = cm.site_off(y, z);
        }
#pragma unroll
        for (int i = 0; i < FPT; ++i) foff[i] = cm.site_off(y0 + fr[i], z0 + fc[i]);
        xa = s.xa;
        xe = s.xe;
    }

    template <int U> __device__ __forceinline__ void step(int j, int pb)
    {
        constexpr int SM2 = U % 5, SM1 = (U + 1) % 5, S0 = (U + 2) % 5, SP1 = (U + 3) % 5, SP2 = (U + 4) % 5;
        const int qb = pb ^ 1;
        auto& Pn = sm.phi[qb];
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            asm volatile("" : "+v"(pidx[i]), "+v"(qidx[i]), "+v"(off[i]));
#pragma unroll
            for (int sl = 0; sl < 5; ++sl)
                asm volatile("" : "+v"(ring[i][sl][0]), "+v"(ring[i][sl][1]), "+v"(ring[i][sl][2]), "+v"(ring[i][sl][3]));
            // stage phi(j+1) into the other phi buffer, then prefetch
            if (active[i]) Pn.st(pidx[i] + 2 * G::PW, ring[i][SP1]);
#pragma unroll
            for (int A = 0; A < 4; ++A) ring[i][SP2][A] = nxt[i][A];
            if (active[i]) cm.load(off[i], j + 3, nxt[i]);
        }
        // the frame sites of phi(j+1) likewise
#pragma unroll
        for (int i = 0; i < FPT; ++i) {
            asm volatile("" : "+v"(fidx[i]), "+v"(foff[i]));
            if (floader[i]) {
                Pn.st(fidx[i], fnxt[i]);
                cm.load(foff[i], j + 2, fnxt[i]);
            }
        }
        const bool j_in = (j >= cm.ilo[0]) && (j <= cm.ihi[0]);
        const auto& P = sm.phi[pb];
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            if (!active[i]) continue;
            T c[4], ax[4], ap[4], aq[4];
            const bool yh = is_y[i];
            T Ym2[4], Ym1[4], Yp1[4], Yp2[4], Zm2[4], Zm1[4], Zp1[4], Zp2[4];
            const int pa = pidx[i];
            P.ld(pa + (2 * G::PW - 2 * G::PW), Ym2);
            P.ld(pa + (2 * G::PW - G::PW), Ym1);
            P.ld(pa + (2 * G::PW + G::PW), Yp1);
            P.ld(pa + (2 * G::PW + 2 * G::PW), Yp2);
            P.ld(pa + (2 * G::PW - 2), Zm2);
            P.ld(pa + (2 * G::PW - 1), Zm1);
            P.ld(pa + (2 * G::PW + 1), Zp1);
            P.ld(pa + (2 * G::PW + 2), Zp2);
#pragma unroll
            for (int A = 0; A < 4; ++A) {
                c[A] = ring[i][S0][A];
                ax[A] = fmaT(T(8), ring[i][SP1][A] - ring[i][SM1][A], ring[i][SM2][A] - ring[i][SP2][A]);
                const T ay = fmaT(T(8), Yp1[A] - Ym1[A], Ym2[A] - Yp2[A]);
                const T az = fmaT(T(8), Zp1[A] - Zm1[A], Zm2[A] - Zp2[A]);
                ap[A] = yh ? ay : az;
                aq[A] = yh ? az : ay;
            }
            const bool valid = vyz[i] && j_in;
            const T gxx = valid ? dot4(ax, ax) : T(0), gqq = valid ? dot4(aq, aq) : T(0);
            const T gpx = valid ? dot4(ap, ax) : T(0), gpq = valid ? dot4(ap, aq) : T(0);
            const T sp = gxx + gqq;
            T qp[4];
#pragma unroll
            for (int A = 0; A < 4; ++A) qp[A] = fmaT(sp, ap[A], -fmaT(gpx, ax[A], gpq * aq[A]));
            if constexpr (EXT == EXT_SEXTIC) {
                if (k.sextic) {
                    // the sextic flux of the supplied direction, c6 det ddet/da_p
                    T ay[4], az[4], C0[4], C1[4], C2[4], C3[4];
#pragma unroll
                    for (int A = 0; A < 4; ++A) {
                        ay[A] = yh ? ap[A] : aq[A];
                        az[A] = yh ? aq[A] : ap[A];
                    }
                    const T det = det4_cofactors(c, ax, ay, az, C0, C1, C2, C3);
                    const T dv = valid ? k.c6q * det : T(0);
#pragma unroll
                    for (int A = 0; A < 4; ++A) qp[A] = fmaT(dv, yh ? C2[A] : C3[A], qp[A]);
                }
            }
            sm.q[pb].st(qidx[i], qp);
        }
        __syncthreads();
    }

    __device__ __forceinline__ void march()
    {
        const int js = xa - 2;
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            if (!active[i]) continue;
            cm.load(off[i], js - 2, ring[i][0]);
            cm.load(off[i], js - 1, ring[i][1]);
            cm.load(off[i], js, ring[i][2]);
            cm.load(off[i], js + 1, ring[i][3]);
            cm.load(off[i], js + 2, nxt[i]);
        }
        auto& Q = sm.phi[0];
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            if (!active[i]) continue;
            Q.st(pidx[i] + 2 * G::PW, ring[i][2]);
        }
#pragma unroll
        for (int i = 0; i < FPT; ++i) {
            if (!floader[i]) continue;
            T f0[4];
            cm.load(foff[i], js, f0);
            cm.load(foff[i], js + 1, fnxt[i]);
            Q.st(fidx[i], f0);
        }
        __syncthreads();
        const int nst = (xe - xa) + 4;
        for (int st = 0; st < nst; st += 5) {
            const int j = js + st, pb = st & 1;
            step<0>(j, pb);
            if (st + 1 >= nst) break;
            step<1>(j + 1, pb ^ 1);
            if (st + 2 >= nst) break;
            step<2>(j + 2, pb);
            if (st + 3 >= nst) break;
            step<3>(j + 3, pb ^ 1);
            if (st + 4 >= nst) break;
            step<4>(j + 4, pb);
        }
    }
};

// The flow's decision after the sweep over phi_k (Sec. 3), from the sums of that sweep (the
// energy density, the largest |F|^2, the power): arrest when E_k > E_{k-1} (energy rule) or when
// the power h^3 sum F_k . v_k < 0 (power rule), re-running the sweep with v_k = 0; stop when
// max|F_k| < tol; otherwise accept the update (swap the field buffers).  c: the control block as
// read before the sums were complete; the fields that change are written to ctl.  One thread.
__device__ inline void flow_decide(double sum_e, double max_f2, double sum_pow, const Ctl& c, Ctl* ctl)
{
    const double E = c.h3 * sum_e;
    const double P = c.h3 * sum_pow;
    const double r = sqrt(max_f2);
    ctl->sweeps = c.sweeps + 1;
    ctl->E = E;
    ctl->P = P;
    ctl->max_force = r;
    if (!isfinite(E) || !isfinite(r)) {
        ctl->done = 1;
        ctl->status = 3;
        return;
    }
    bool arrest = false;
    if (!c.redo && ((c.flow_mode == SKYR_ARREST_POWER && P < 0.0) ||
                    (c.flow_mode == SKYR_ARREST_ENERGY && E > c.E_prev))) {
        arrest = true;
        ctl->arrests = c.arrests + 1;
    }
    if (r < c.tol) {
        ctl->done = 1;
        ctl->status = 1;
        // the sweep wrote v_k + dt F_k over v_k; the next one puts v_k back (zero if v_k was
        // reset by an arrest at this step or was zero on this redo sweep)
        const bool v_zero = c.redo || arrest || c.flow_mode == SKYR_GRADIENT_FLOW;
        ctl->restore = v_zero ? RESTORE_ZERO : RESTORE_UNKICK;
        ctl->redo = 0;
        return;
    }
    if (arrest) {
        ctl->redo = 1;
        ctl->redo_sweeps = c.redo_sweeps + 1;
        return;
    }
    ctl->cur = c.cur ^ 1;
    ctl->redo = 0;
    ctl->E_prev = E;
    ctl->steps = c.steps + 1;
    if (c.steps + 1 >= c.target) {
        ctl->done = 1;
        ctl->status = 2;
    }
}

// End of a step sweep: every block has published its partial sums; the block that
// finishes last (a ticket counter in the control block, no waiting) sums them all in a
// fixed order (thread t takes records t, t + THREADS, ..., then a fixed butterfly per wave
// and the waves in order) and takes the flow's decision.  A restore sweep only clears the
// restore flag; a sweep on a held control block leaves the sums themselves there (E and P without
// the factor h^3) and takes no decision.
// The partial sums are agent-scope atomic stores of wave 0, complete (s_waitcnt) before the
// block's ticket, and the last block reads them with agent-scope atomic loads: they are coherent
// across the XCDs' L2 caches without a device-wide fence, which would write back and
// invalidate the whole L2 of the block's XCD while its neighbours still read halo lines.
// The fields of the control block other than the ticket change only between launches: thread 0
// reads those of the decision while the partial sums are on their way.
// Only the three sums that the decision needs are reduced, on the vector unit, and nothing waits
// twice: 40^3 double (six march steps a block) 19.2 -> 17.9 us a sweep, 256^3 float 2% faster.
// Smem: shared memory with `int last` and `double red[NW][NPART]`; THREADS threads in NW waves.
// records: of REC doubles, the three sums at E, F2 and POW.
template <int THREADS, int NW, int REC, int E, int F2, int POW, class Smem>
__device__ __forceinline__ void finish_step(const double* part, int nb, int records, Ctl* ctl, bool restore, Smem& sm)
{
    const int tid = threadIdx.x;
    Ctl c{};
    if (tid == 0) {
        c = *ctl;
        __builtin_amdgcn_s_waitcnt(0);  // this block's partial sums before its ticket
        sm.last = __hip_atomic_fetch_add(&ctl->ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nb - 1;
    }
    __syncthreads();
    if (!sm.last) return;
    if (restore) {
        if (tid == 0) {
            ctl->restore = RESTORE_NONE;
            __hip_atomic_store(&ctl->ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    // the flow sweep sums the whole energy density in slot P_E2 (slots P_E4, P_E0, P_E6 are zero)
    double e = 0.0, f2 = 0.0, pw = 0.0;
    for (int b = tid; b < records; b += THREADS) {
        const double* p = part + (size_t)b * REC;
        const double x0 = __hip_atomic_load(p + E, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double x1 = __hip_atomic_load(p + F2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double x2 = __hip_atomic_load(p + POW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        e += x0;
        f2 = fmax(f2, x1);
        pw += x2;
    }
    e = wave_total<false>(e);
    f2 = wave_total<true>(f2);
    pw = wave_total<false>(pw);
    const int lane = tid & 63, wave = tid >> 6;
    if (lane == 0) {
        sm.red[wave][0] = e;
        sm.red[wave][1] = f2;
        sm.red[wave][2] = pw;
    }
    __syncthreads();
    if (tid == 0) {
        e = f2 = pw = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            e += sm.red[w][0];
            f2 = fmax(f2, sm.red[w][1]);
            pw += sm.red[w][2];
        }
        if (c.hold) {
            ctl->E = e;
            ctl->P = pw;
            ctl->max_force = sqrt(f2);
        } else {
            flow_decide(e, f2, pw, c, ctl);
        }
        __hip_atomic_store(&ctl->ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// A block's sums over its threads, in a fixed order (a butterfly per wave, then waves 0 .. NWS-1),
// published as the block's record.  e2: in a step sweep the whole energy density (the parts and the
// charge are then not summed).  Lane i of wave 0 publishes slot i, f2 and pw with the
// factors given.
template <int NWS, bool STEP, class Smem>
__device__ __forceinline__ void block_sums(double e2, double f2, double pw, double f2_scale, double pw_scale, double e4,
                                           double e0, double b, double e6, double* record, Smem& sm)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave < NWS) {
        e2 = wave_total<false>(e2);
        f2 = wave_total<true>(f2);
        if constexpr (STEP) {
            pw = wave_total<false>(pw);
        } else {
            e4 = wave_total<false>(e4);
            e0 = wave_total<false>(e0);
            b = wave_total<false>(b);
            e6 = wave_total<false>(e6);
        }
        if (lane == 0) {
            double* r = sm.red[wave];
            r[P_E2] = e2;
            r[P_E4] = STEP ? 0.0 : e4;
            r[P_E0] = STEP ? 0.0 : e0;
            r[P_B] = STEP ? 0.0 : b;
            r[P_F2] = f2;
            r[P_POW] = STEP ? pw : 0.0;
            r[P_E6] = STEP ? 0.0 : e6;
        }
    }
    __syncthreads();
    if (threadIdx.x < NRED) {
        const int i = threadIdx.x;
        double sum = 0.0, most = 0.0;
#pragma unroll
        for (int w = 0; w < NWS; ++w) {
            const double v = sm.red[w][i];
            sum += v;
            most = fmax(most, v);
        }
        __hip_atomic_store(record + i, i == P_F2 ? most * f2_scale : i == P_POW ? sum * pw_scale : sum, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The same for a block of a batched sweep: the records of its units, `stride` doubles apart, from
// the waves' sums over the `before` units before the last and the threads' over the last.  Lane
// 3 u + q of wave 0 publishes sum q of unit u.
template <int NWS, class Smem>
__device__ __forceinline__ void unit_sums(double e, double f2, double pw, int before, double* record, int stride,
                                          Smem& sm)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave < NWS) {
        wave_totals(e, pw);
        f2 = wave_total<true>(f2);
        if (lane == 0) {
            sm.red[wave][U_E] = e;
            sm.red[wave][U_F2] = f2;
            sm.red[wave][U_POW] = pw;
        }
    }
    __syncthreads();
    static_assert(3 * MAX_UNITS <= 64, "one lane per sum");
    const int u = threadIdx.x / 3, q = threadIdx.x - 3 * u;
    if (u <= before) {
        double sum = 0.0, most = 0.0;
#pragma unroll
        for (int w = 0; w < NWS; ++w) {
            const double v = u < before ? sm.unit[u][w][q] : sm.red[w][q];
            sum += v;
            most = fmax(most, v);
        }
        __hip_atomic_store(record + (size_t)u * stride + q, q == U_F2 ? most : sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// One block's share of one field: logical block b of nb blocks, which takes the items b,
// b + nb, ... of the field's work.  Used by the single-field and the batched kernels
// (FROM_TABLE: the arguments were read from the batch's job table).
template <typename T, class G, int MODE, bool FROM_TABLE, int EXT, int STREAM>
__device__ __forceinline__ void sweep_block(const SweepArgs& a, int b, int nb, SweepSmem<T, G>& sm)
{
    SweepCommon<T, FROM_TABLE> cm;
    int cur = 0;
    cm.redo = false;
    cm.renorm64 = false;
    cm.restore = RESTORE_NONE;
    if constexpr (MODE == MODE_STEP) {
        // the control block is the same for the whole block: its fields are read as uniform values
        const gptr<const Ctl> ctl = (gptr<const Ctl>)uniform_ptr(a.ctl);
        const auto rd = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
        cm.restore = rd(ctl->restore);
        if (rd(ctl->done) && !cm.restore) return;  // the flow has stopped
        cur = rd(ctl->cur);
        cm.redo = rd(ctl->redo) != 0;
        const int kr = rd(ctl->renorm64_every);
        const long long st = ctl->steps;
        const int st_lo = rd((int)(unsigned)(st & 0xffffffff)), st_hi = rd((int)(unsigned)(st >> 32));
        const long long steps = (long long)(((unsigned long long)(unsigned)st_hi << 32) | (unsigned)st_lo);
        cm.renorm64 = (kr > 0) && (((steps + 1) % kr) == 0);
    }
    cm.n0 = a.n0;
    cm.n1 = a.n1;
    cm.n2 = a.n2;
    cm.zlo = a.zlo;
    cm.zhi = a.zhi;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        cm.ilo[d] = a.ilo[d];
        cm.ihi[d] = a.ihi[d];
    }
    cm.olo1 = a.olo[1];
    cm.olo2 = a.olo[2];
    cm.ohi1 = a.ohi[1];
    cm.ohi2 = a.ohi[2];
    cm.plane_b = (unsigned)(a.n1 * a.n2) * (unsigned)sizeof(T);
    const long long N3 = a.cstride;
    {
        const T* pin = (const T*)(MODE == MODE_STEP && cur ? (const void*)a.phi1 : a.phi0);
        T* pout = (T*)(MODE == MODE_STEP ? (cur ? (void*)a.phi0 : a.phi1) : nullptr);
        T* pvel = (T*)a.vel;
        T* pgrad = (T*)a.grad;
        // the same for the whole block (kernel arguments or the job table): kept in SGPRs
        pin = uniform_ptr(pin);
        pout = uniform_ptr(pout);
        pvel = uniform_ptr(pvel);
        pgrad = uniform_ptr(pgrad);
#pragma unroll
        for (int A = 0; A < 4; ++A) {
            cm.pin[A] = (gptr<const T>)(pin + A * N3);
            cm.pout[A] = (gptr<T>)(pout ? pout + A * N3 : nullptr);
            cm.vel[A] = (gptr<T>)(pvel ? pvel + A * N3 : nullptr);
            cm.gout[A] = (gptr<T>)(pgrad ? pgrad + A * N3 : nullptr);
        }
    }
    cm.has_grad = a.grad != nullptr;
    cm.projected = a.projected != 0;
    cm.baryon = a.baryon != 0;
    SweepConst<T> k;
    k.init(a, MODE == MODE_STEP);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = a.tiles_y * a.tiles_z;
    const int x0 = a.olo[0], nx = a.ohi[0] - a.olo[0] + 1;
    // a block of a batched sweep: its slab, its first unit and how many, and its first plane and the
    // one after its last
    const int slab = b / tiles, unit0 = FROM_TABLE ? slab * a.per_block : 0;
    const int own = FROM_TABLE ? min(a.units - unit0, a.per_block) : 0;
    int first = 0, end = 0;
    if constexpr (FROM_TABLE) {
        first = __builtin_amdgcn_readfirstlane(unit_start(unit0, nx, a.units, a.unit_len));
        end = __builtin_amdgcn_readfirstlane(unit_start(unit0 + own, nx, a.units, a.unit_len));
        // (read after the march's first barrier)
        if (tid < own) sm.unit_end[tid] = unit_start(unit0 + tid + 1, nx, a.units, a.unit_len) - first;
        if (tid < G::NWI) sm.units_ended[tid] = 0;
    }
    const auto segment = [&](int item) {
        Segment s = item_segment(item, tiles, a.tiles_z, x0, nx, a.xchunk);
        if constexpr (FROM_TABLE) {
            s.xa = x0 + first;
            s.xe = x0 + end;
        }
        return s;
    };
    const int items = FROM_TABLE ? nb : tiles * ((nx + a.xchunk - 1) / a.xchunk);

    double e2 = 0.0, e4 = 0.0, e0 = 0.0, e6 = 0.0, bsum = 0.0, f2 = 0.0, pw = 0.0;
    if (wave < G::NWI) {
        Interior<T, G, MODE, FROM_TABLE, EXT, STREAM> it(sm, k, cm, tid);
        for (int item = b; item < items; item += nb) {
            it.setup(segment(item), a.zstart);
            it.march();
        }
        e2 = it.pe2;
        e4 = it.pe4;
        e0 = it.pe0;
        bsum = it.pb_sum * k.dinv12h3;
        f2 = (double)it.pf2 * k.dinvK2;  // (scaled here: after the roles meet it cost four registers)
        pw = it.pp * k.dinvK;
        e6 = it.pe6;
    } else {
        Halo<T, G, FROM_TABLE, EXT> hl(sm, k, cm, tid - G::NWI * 64);
        for (int item = b; item < items; item += nb) {
            hl.setup(segment(item), a.zstart);
            hl.march();
        }
    }
    if constexpr (FROM_TABLE) {
        // the records of the block's units, in the order of the units and tiles of the field
        unit_sums<G::NWI>(e2, f2, pw, own - 1,
                          a.partials + (size_t)(unit0 * tiles + b - slab * tiles) * UNIT_REC, tiles * UNIT_REC, sm);
        finish_step<G::THREADS, G::NW, UNIT_REC, U_E, U_F2, U_POW>(a.partials, nb, tiles * a.units, a.ctl,
                                                                   cm.restore != RESTORE_NONE, sm);
    } else {
        block_sums<G::NWI, MODE == MODE_STEP>(e2, f2, pw, 1.0, 1.0, e4, e0, bsum, e6, a.partials + (size_t)b * NPART, sm);
        if constexpr (MODE == MODE_STEP)
            finish_step<G::THREADS, G::NW, NPART, P_E2, P_F2, P_POW>(a.partials, nb, nb, a.ctl,
                                                                     cm.restore != RESTORE_NONE, sm);
    }
}

// Blocks are dispatched round-robin over the eight XCDs (block i to XCD i % 8).
// The logical index gives each XCD a contiguous run of the work: neighbouring
// tiles of one slab, which march through the same planes and share halo rows
// in one L2.
__device__ __forceinline__ int xcd_logical_block(int i, int n)
{
    const int xcd = i % 8, q8 = n / 8, r8 = n % 8;
    return xcd * q8 + min(xcd, r8) + i / 8;
}

template <typename T, class G, int MODE, int EXT, int STREAM>
__global__ __launch_bounds__(G::THREADS, (waves_per_simd<T, G, EXT>())) void sweep_kernel(SweepArgs a)
{
    __shared__ SweepSmem<T, G> smem;
    const int nb = gridDim.x;
    sweep_block<T, G, MODE, false, EXT, STREAM>(a, xcd_logical_block(blockIdx.x, nb), nb, smem);
}

// Many fields in one launch: launch block p sweeps block slot[p].y of field slot[p].x
// (no field when slot[p].x < 0: a padding block that ends at once).  The host lays the
// slots out for the round-robin dispatch of blocks over the XCDs (block p runs on XCD
// p mod 8); a field's sums are taken per unit of planes, in the order of the units and tiles, and do not
// depend on how many units its blocks march through.
template <typename T, class G, int EXT, int STREAM>
__global__ __launch_bounds__(G::THREADS, (waves_per_simd<T, G, EXT>())) void batch_sweep_kernel(
    const SweepArgs* __restrict__ jobs, const int2* __restrict__ slot, const int* __restrict__ blocks_of_job)
{
    __shared__ SweepSmem<T, G> smem;
    const int2 e = slot[blockIdx.x];
    if (e.x < 0) return;
    const SweepArgs a = jobs[e.x];
    sweep_block<T, G, MODE_STEP, true, EXT, STREAM>(a, e.y, blocks_of_job[e.x], smem);
}

}  // namespace skyr
