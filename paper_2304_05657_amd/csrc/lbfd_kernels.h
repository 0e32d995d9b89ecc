#pragma once
// lbfd_kernels.h -- templates of the fused coupled step for gfx950: pull-scheme lattice-Boltzmann streaming
// with boundary conditions, finite-difference advection-diffusion-reaction
// of T and Y_k with ghost nodes, source Xi, central-moment collision, and
// explicit Euler update -- one thread per cell, one kernel per step.
//
// Method: Hosseini & Thevenin, arXiv:2304.05657, Secs. II-III.  The step
// order (all terms at level n) and the readings of the paper's silent or
// garbled passages are those stated in include/lbfd.h and the design notes.
//
// Storage (structure of arrays, x fastest):
//   populations  pop[i][cell]   post-collision values g*_i of the previous
//                               level; FP64: g itself, mixed: g/(w_i cs^2)
//   scalars      sc[0][cell] = T, sc[1+k][cell] = Y_k
//   outlet       post-streaming values of the populations that enter
//                through an outflow face, per face cell (double)
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "lbfd_internal.h"
#include "lbfd_math.h"

#include <type_traits>

namespace lbfd {

constexpr double kCs2 = 1.0 / 3.0;

// ---------------------------------------------------------------- lattice
template <int Q>
struct Lat {
    static constexpr int D = (Q == 9) ? 2 : 3;
    __host__ __device__ static constexpr int cx(int i) { return i % 3 - 1; }
    __host__ __device__ static constexpr int cy(int i) { return (i / 3) % 3 - 1; }
    __host__ __device__ static constexpr int cz(int i) { return Q == 9 ? 0 : i / 9 - 1; }
    __host__ __device__ static constexpr int c(int i, int d) { return d == 0 ? cx(i) : d == 1 ? cy(i) : cz(i); }
    __host__ __device__ static constexpr double w(int i)
    {
        // textbook weights by |c|^2
        return Q == 9 ? (cx(i) * cx(i) + cy(i) * cy(i) == 0   ? 4.0 / 9.0
                         : cx(i) * cx(i) + cy(i) * cy(i) == 1 ? 1.0 / 9.0
                                                              : 1.0 / 36.0)
                      : (cx(i) * cx(i) + cy(i) * cy(i) + cz(i) * cz(i) == 0   ? 8.0 / 27.0
                         : cx(i) * cx(i) + cy(i) * cy(i) + cz(i) * cz(i) == 1 ? 2.0 / 27.0
                         : cx(i) * cx(i) + cy(i) * cy(i) + cz(i) * cz(i) == 2 ? 1.0 / 54.0
                                                                              : 1.0 / 216.0);
    }
};

// ------------------------------------------------------------- precision
template <int PREC> struct Prec;
template <> struct Prec<LBFD_FP64> { using calc = double; using pop = double; using scal = double; };
template <> struct Prec<LBFD_MIXED_FP32> { using calc = float; using pop = float; using scal = float; };
template <> struct Prec<LBFD_MIXED_FP16> { using calc = float; using pop = __half; using scal = float; };

// Loads and stores at a 32-bit byte offset from a uniform base pointer
// (base in scalar registers, one 32-bit offset register per access; every
// buffer is below 4 GiB, checked at init).
template <class T>
__device__ __forceinline__ T ldo(const void *base, uint32_t byte_off)
{
    return *(const T *)((const char *)base + byte_off);
}
template <class T>
__device__ __forceinline__ void sto(void *base, uint32_t byte_off, T v)
{
    *(T *)((char *)base + byte_off) = v;
}

// A uniform base address in scalar registers that steps from plane to plane
// of a field (one field of a structure of arrays after another).  step() and
// the empty asm keep the planes' addresses from being formed all at once: left
// to itself the compiler holds the 27 populations' 64-bit bases (three times
// over, for the interior, boundary and curved-wall pulls) in scalar registers,
// spills them into vector lanes -- 850 of the 7,200 vector instructions of the
// 3-D FP64 step -- and, in one instantiation, gave a spilled base's register to
// another value before it was stored.
template <class T> struct PlanePtr {
    typedef __attribute__((address_space(1))) T G;
    G *p;
    __device__ __forceinline__ PlanePtr(const void *base, long long planes, long long N)
        : p((G *)base + planes * N)
    {
        asm volatile("" : "+s"(p));
    }
    __device__ __forceinline__ void step(long long n)
    {
        p += n;
        asm volatile("" : "+s"(p));
    }
    // the element at a 32-bit byte offset
    __device__ __forceinline__ G *at(uint32_t byte_off) const
    {
        return (G *)((__attribute__((address_space(1))) char *)p + byte_off);
    }
};
template <bool STREAM, class G>
__device__ __forceinline__ auto load_global(const G *p)
{
    if constexpr (STREAM)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

// Populations in 3-D pass through L2 without displacing the scalars, whose
// stencil rows and planes are read again: each population is read by one cell
// and written once, so its loads and stores are marked nontemporal.  In half
// precision a wave's 128 bytes of a direction, shifted by a cell, share their
// lines with the neighbouring tile and the mark costs more than it gives:
// 256 x 256 x 128 packing, FP64, 1888 -> 1847 us a step; 256 x 128 x 128 with
// 9 species, FP64, 1404 -> 1378 us; 161 x 99 x 83, half, 179 -> 184 us.
template <int Q, int PREC> constexpr bool pop_stream() { return Q == 27 && PREC != LBFD_MIXED_FP16; }
// Populations: FP64 stores g; mixed stores g / (w_i cs^2) (deviation from
// the lattice weights, scaled to comparable magnitude across directions).
template <int Q, int PREC, int I>
__device__ __forceinline__ typename Prec<PREC>::calc pop_load(const void *base, long long N, uint32_t idx)
{
    using T = typename Prec<PREC>::pop;
    const char *b = (const char *)base + (size_t)I * (size_t)N * sizeof(T);
    const uint32_t off = idx * (uint32_t)sizeof(T);
    if constexpr (PREC == LBFD_FP64) {
        return ldo<double>(b, off);
    } else if constexpr (PREC == LBFD_MIXED_FP32) {
        constexpr float s = (float)(Lat<Q>::w(I) * kCs2);
        return ldo<float>(b, off) * s;
    } else {
        constexpr float s = (float)(Lat<Q>::w(I) * kCs2);
        return __half2float(ldo<__half>(b, off)) * s;
    }
}

template <int Q, int PREC, int I>
__device__ __forceinline__ void pop_store(void *base, long long N, uint32_t idx, typename Prec<PREC>::calc v)
{
    using T = typename Prec<PREC>::pop;
    char *b = (char *)base + (size_t)I * (size_t)N * sizeof(T);
    const uint32_t off = idx * (uint32_t)sizeof(T);
    if constexpr (PREC == LBFD_FP64) {
        sto<double>(b, off, v);
    } else if constexpr (PREC == LBFD_MIXED_FP32) {
        constexpr float s = (float)(1.0 / (Lat<Q>::w(I) * kCs2));
        sto<float>(b, off, v * s);
    } else {
        constexpr float s = (float)(1.0 / (Lat<Q>::w(I) * kCs2));
        sto<__half>(b, off, __float2half_rn(v * s));
    }
}

// Population I of a cell stored at q, scaled (pop_store on a plane).
template <int Q, int PREC, int I>
__device__ __forceinline__ void plane_store(__attribute__((address_space(1))) typename Prec<PREC>::pop *q,
                                            typename Prec<PREC>::calc v)
{
    using T = typename Prec<PREC>::pop;
    constexpr float s = (float)(1.0 / (Lat<Q>::w(I) * kCs2));
    if constexpr (PREC == LBFD_MIXED_FP16)
        *(__attribute__((address_space(1))) unsigned short *)q = __builtin_bit_cast(unsigned short, __float2half_rn(v * s));
    else if constexpr (pop_stream<Q, PREC>())
        __builtin_nontemporal_store(PREC == LBFD_FP64 ? (T)v : (T)(v * s), q);
    else
        *q = PREC == LBFD_FP64 ? (T)v : (T)(v * s);
}

// compile-time loop
template <int B, int E, class F>
__device__ __forceinline__ void sfor(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        sfor<B + 1, E>(f);
    }
}

// ------------------------------------------------------------- geometry
struct Nb {
    int kind;
    int face;
    long long idx;
    double Tw;
};

__device__ __forceinline__ int wrapc(int v, int n)
{
    if ((unsigned)v < (unsigned)n) return v;
    int r = v % n;
    return r < 0 ? r + n : r;
}

// What sits at (x, y, z): periodic faces wrap; outside any other face the
// point is that face (walls before inflow before outflow, lower axis and
// face first); inside, the mask decides.
__device__ __forceinline__ Nb classify(const KParams &P, int x, int y, int z)
{
    int q[3] = {x, y, z};
    const int n[3] = {P.nx, P.ny, P.nz};
    int best_face = -1, best_rank = 99;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        if ((unsigned)q[d] >= (unsigned)n[d]) {
            int f = 2 * d + (q[d] >= n[d] ? 1 : 0);
            int kind = P.face[f];
            if (kind == LBFD_FACE_PERIODIC) {
                q[d] = wrapc(q[d], n[d]);
            } else {
                int rank = (kind == LBFD_FACE_WALL || kind == LBFD_FACE_WALL_ADIABATIC) ? 0
                         : kind == LBFD_FACE_INFLOW ? 1 : 2;
                if (rank < best_rank) {
                    best_rank = rank;
                    best_face = f;
                }
            }
        }
    }
    Nb r;
    r.idx = 0;
    r.Tw = 0.0;
    r.face = best_face;
    if (best_face >= 0) {
        int kind = P.face[best_face];
        r.kind = kind == LBFD_FACE_WALL ? kIso : kind == LBFD_FACE_WALL_ADIABATIC ? kAdia
               : kind == LBFD_FACE_INFLOW ? kInflow : kOutflow;
        r.Tw = P.face_T[best_face];
        return r;
    }
    r.idx = ((long long)q[2] * P.ny + q[1]) * P.nx + q[0];
    uint8_t m = P.mask[r.idx];
    r.kind = m == LBFD_FLUID ? kFluid : m == LBFD_SOLID_ISOTHERMAL ? kIso : kAdia;
    if (r.kind == kIso) r.Tw = P.wall_T[r.idx];
    return r;
}

__device__ __forceinline__ long long outlet_index(const KParams &P, int face, int i, int Q, int y, int z)
{
    return ((long long)((face & 1) * Q + i) * P.nz + z) * P.ny + y;
}

// c_I . u_in for population I of fluid cell (x, y, z) entering through an
// inflow face (Eq. 31): an x face carries a per-cell inlet profile, indexed
// by the entering cell's (y, z); other faces the uniform inflow velocity.
// (A source beyond an x inflow face and another non-periodic face is the
// wall's, or the x face's: walls rank first, then the lower axis.)
__device__ __forceinline__ double inflow_cu_c(const KParams &P, int cx, int cy, int cz, int x, int y, int z)
{
    const int f = (cx == 1 && x == 0 && P.face[0] == LBFD_FACE_INFLOW)               ? 0
                  : (cx == -1 && x == P.nx - 1 && P.face[1] == LBFD_FACE_INFLOW) ? 1
                                                                                 : -1;
    if (f >= 0) {
        const long long s = (long long)P.ny * P.nz;
        const double *u = P.inflow_u + 3 * s * f + (long long)z * P.ny + y;
        return cx * u[0] + cy * u[s] + cz * u[2 * s];
    }
    return cx * P.u_in[0] + cy * P.u_in[1] + cz * P.u_in[2];
}

template <int Q, int I>
__device__ __forceinline__ double inflow_cu(const KParams &P, int x, int y, int z)
{
    using L = Lat<Q>;
    return inflow_cu_c(P, L::cx(I), L::cy(I), L::cz(I), x, y, z);
}

// ------------------------------------------------------------ scalars
template <int NSP, class C>
struct Pt {
    C T, rho;
    C Y[NSP];
};

template <int NSP, class C>
__device__ __forceinline__ C density(const KParams &P, C T, const C *Y)
{
    C s = 0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) s += Y[k] * (C)P.invW[k];
    return (C)P.T_ref_over_W_ref * rcp(T * s);
}

// The density over its constant factor T_ref / W_ref.
template <int NSP, class C>
__device__ __forceinline__ C density_rcp(const KParams &P, C T, const C *Y)
{
    C s = 0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) s += Y[k] * (C)P.invW[k];
    return rcp(T * s);
}

template <int NSP, int PREC>
__device__ __forceinline__ void load_point(const KParams &P, long long idx, Pt<NSP, typename Prec<PREC>::calc> &o)
{
    using S = typename Prec<PREC>::scal;
    const char *sc = (const char *)P.sc_in;
    const size_t fstride = (size_t)P.N * sizeof(S);
    const uint32_t off = (uint32_t)idx * (uint32_t)sizeof(S);
    o.T = ldo<S>(sc, off);
#pragma unroll
    for (int k = 0; k < NSP; ++k) o.Y[k] = ldo<S>(sc + (size_t)(1 + k) * fstride, off);
    o.rho = density<NSP>(P, o.T, o.Y);
}

// Population I or its opposite (same lattice weight, hence the same scale
// in the mixed forms) of cell idx, the direction chosen per lane.
template <int Q, int PREC, int I>
__device__ __forceinline__ typename Prec<PREC>::calc pop_load_pair(const void *base, long long N, bool opp,
                                                                   uint32_t idx)
{
    using T = typename Prec<PREC>::pop;
    constexpr int OPP = Q - 1 - I;
    static_assert(Lat<Q>::w(I) == Lat<Q>::w(OPP), "opposite directions share a weight");
    const size_t dir = opp ? (size_t)OPP : (size_t)I;
    const char *b = (const char *)base + dir * (size_t)N * sizeof(T);
    const uint32_t off = idx * (uint32_t)sizeof(T);
    if constexpr (PREC == LBFD_FP64) {
        return ldo<double>(b, off);
    } else if constexpr (PREC == LBFD_MIXED_FP32) {
        constexpr float s = (float)(Lat<Q>::w(I) * kCs2);
        return ldo<float>(b, off) * s;
    } else {
        constexpr float s = (float)(Lat<Q>::w(I) * kCs2);
        return __half2float(ldo<__half>(b, off)) * s;
    }
}

// Values (T, Y_k, rho) at a listed image point, reconstructed for this
// level by image_kernel.
template <int NSP, class C>
__device__ __forceinline__ void image_value(const KParams &P, int li, Pt<NSP, C> &o)
{
    const C *v = (const C *)P.img_val + li;
    o.T = v[0];
#pragma unroll
    for (int k = 0; k < NSP; ++k) o.Y[k] = v[(1 + k) * P.n_img];
    o.rho = v[(1 + NSP) * P.n_img];
}

// fourth-order central first and second derivatives (Sec. II.D)
template <class C>
__device__ __forceinline__ C d1(C a, C b, C c, C d, C e)
{
    return ((a - (C)8 * b) + ((C)8 * d - e)) * (C)(1.0 / 12.0);
}
template <class C>
__device__ __forceinline__ C d2(C a, C b, C c, C d, C e)
{
    return ((C)16 * (b + d) - (a + e) - (C)30 * c) * (C)(1.0 / 12.0);
}

// WENO3 convective derivative (Jiang-Shu weights, eps = 1e-6): for u >= 0
// the face values at i+1/2 and i-1/2 are reconstructed from the left; for
// u < 0 the stencil is mirrored and the result negated, which is the
// right-biased reconstruction.  At a face between b and c reconstructed
// from the side of b (a the far upwind point) the value is
// q1 + w0 (q0 - q1), q0 = 3b/2 - a/2, q1 = (b+c)/2, with the normalised
// weight w0 = e1^2 / (e1^2 + 2 e0^2), e0 = eps + (b-a)^2,
// e1 = eps + (c-b)^2; both faces share one division.
template <class C>
__device__ __forceinline__ C weno3(C m2, C m1, C c0, C p1, C p2, C u)
{
    const bool neg = u < (C)0;
    const C A = neg ? p2 : m2, B = neg ? p1 : m1, E = neg ? m1 : p1;
    const C eps = (C)1e-6;
    const C dA = B - A, dB = c0 - B, dE = E - c0;
    const C eA = eps + dA * dA, eB = eps + dB * dB, eE = eps + dE * dE;
    const C eA2 = eA * eA, eB2 = eB * eB, eE2 = eE * eE;
    const C den_p = eE2 + (C)2 * eB2;  // face i+1/2: e0 = eB, e1 = eE
    const C den_m = eB2 + (C)2 * eA2;  // face i-1/2: e0 = eA, e1 = eB
    const C inv = rcp(den_p * den_m);
    const C w_p = eE2 * den_m * inv, w_m = eB2 * den_p * inv;
    const C q0p = (C)1.5 * c0 - (C)0.5 * B, q1p = (C)0.5 * (c0 + E);
    const C q0m = (C)1.5 * B - (C)0.5 * A, q1m = (C)0.5 * (B + c0);
    const C conv = (q1p + w_p * (q0p - q1p)) - (q1m + w_m * (q0m - q1m));
    return neg ? -conv : conv;
}

// The three finite-difference operators of one scalar along one axis from
// its five stencil values, written on the forward differences
// D0 = m1 - m2, D1 = c0 - m1, D2 = p1 - c0, D3 = p2 - p1:
//   D1 (4th order) = (7 (D1 + D2) - (D0 + D3)) / 12,
//   D2 (4th order) = (15 (D2 - D1) - (D3 - D0)) / 12,
//   conv2 = twice the WENO3 convective derivative of weno3() (the caller
//   folds the 1/2 into u): with (a, b, c) = (D0, D1, D2) for u >= 0 and
//   (D3, D2, D1) for u < 0 (the mirrored stencil, whose negation cancels the
//   sign of its differences), conv2 = (b + c) + w+ (b - c) - w- (a - b),
//   w+ = eC^2 / (eC^2 + 2 eB^2), w- = eB^2 / (eB^2 + 2 eA^2), eX = eps + X^2,
//   both weights from one reciprocal; next to walls (near) the centred
//   difference b + c.
template <class C>
__device__ __forceinline__ void axis5(C m2, C m1, C c0, C p1, C p2, C u, bool near, C &d1o, C &d2o, C &conv2)
{
    const C D0 = m1 - m2, D1 = c0 - m1, D2 = p1 - c0, D3 = p2 - p1;
    const C s12 = D1 + D2;
    d1o = ((C)7 * s12 - (D0 + D3)) * (C)(1.0 / 12.0);
    d2o = ((C)15 * (D2 - D1) - (D3 - D0)) * (C)(1.0 / 12.0);
    const bool neg = u < (C)0;
    const C a = neg ? D3 : D0, b = neg ? D2 : D1, c = neg ? D1 : D2;
    const C eps = (C)1e-6;
    const C eA = eps + a * a, eB = eps + b * b, eC = eps + c * c;
    const C eA2 = eA * eA, eB2 = eB * eB, eC2 = eC * eC;
    const C den_p = eC2 + (C)2 * eB2, den_m = eB2 + (C)2 * eA2;
    const C inv = rcp(den_p * den_m);
    const C X = (eC2 * (b - c)) * den_m - (eB2 * (a - b)) * den_p;
    conv2 = near ? s12 : s12 + X * inv;
}

// ------------------------------------------------------------ chemistry
// Arrhenius source over one step in double precision (per reaction
// r = A dt T^b exp(-Ta/T) prod Y_react; species nu_k r, temperature q r):
// one explicit Euler step, or, with chem_substeps_max > 1, N sub-steps
// with N = ceil(max_j k_j / 0.1) capped at chem_substeps_max; a sub-step
// that would consume a mass fraction below zero is scaled down.
// The rate coefficient A dt T^b exp(-Ta/T) is formed from ln T and 1/T
// shared by every reaction as (A dt) exp(b ln T - Ta / T), one exponential
// per reaction (with b = 0 it is A dt exp(-Ta / T)).
__device__ __forceinline__ double rate_coeff_l(const ChemRx &r, double lnT, double invT, const double *tab)
{
    return r.adt * exp_tab(r.b * lnT - r.ta * invT, tab);
}

// The same coefficient divided by the sub-step count N, with ln(A dt) and
// ln N moved into the exponent: exp(b ln T - Ta/T + ln(A dt) - ln N), formed
// in units of ln 2 / 256 (lnNs = ln N 256/ln 2).  Each operation takes one
// per-reaction constant: an instruction reads at most one scalar register
// operand.
__device__ __forceinline__ double rate_coeff_sub(const ChemRx &r, double lnT, double invT, double lnNs,
                                                 const double *tab)
{
    return exp_scaled_tab(fma(r.bs, lnT, fma(-r.tas, invT, -lnNs)) + r.lnadts, tab);
}

// Returns the number of sub-steps taken.  NR: the largest reactant count
// of a reaction (slots past a reaction's own count multiply by 1).
template <int NSP, bool LE = false, int NR = 4>
__device__ __forceinline__ int chemistry(const KParams &P, const double *tab, const double *ltab, double T,
                                         const double (&Y)[NSP],
                                         double &srcT, double (&srcY)[NSP])
{
    // ln T is needed only when a temperature exponent is not zero
    const bool anyb = P.chem_anyb != 0;
    int nsub = 1;
    if (P.chem_substeps_max > 1) {
        const double lnT = anyb ? log(T) : 0.0, invT = rcp(T);
        double kmax = 0.0;
        for (int j = 0; j < P.n_rx; ++j) kmax = fmax(kmax, rate_coeff_l(P.rxk[j], lnT, invT, tab));
        double want = ceil(kmax / 0.1);
        nsub = want < 1.0 ? 1 : want > (double)P.chem_substeps_max ? P.chem_substeps_max : (int)want;
    }
    const double lnNs = nsub == 1 ? 0.0 : log((double)nsub) * 0x1.71547652b82fep+8;  // ln N 256/ln 2
    double dT = 0.0, dY[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) dY[k] = 0.0;
    for (int s = 0; s < nsub; ++s) {
        const double Tc = T + dT;
        // Yc[NSP] = 1 is the factor of the unused reactant slots
        double Yc[NSP + 1];
#pragma unroll
        for (int k = 0; k < NSP; ++k) Yc[k] = Y[k] + dY[k];
        Yc[NSP] = 1.0;
        double incT = 0.0, incY[NSP];
#pragma unroll
        for (int k = 0; k < NSP; ++k) incY[k] = 0.0;
        const double lnTc = anyb ? log_tab(Tc, ltab) : 0.0, invTc = rcp(Tc);
        // one reaction's progress over the sub-step and its increments;
        // the reactant indices are the same for every lane, so Yc is
        // indexed through the register file (no private memory).  The four
        // reactant slots are all multiplied in (the unused ones index the
        // constant 1): a fixed count lets the four indices arrive in one
        // scalar load ahead of the products instead of one dependent load
        // per reactant
        auto apply = [&](const ChemRx &r, double k) {
            double rr = k;
#pragma unroll
            for (int m = 0; m < NR; ++m) rr *= Yc[r.react[m]];
#pragma unroll
            for (int k2 = 0; k2 < NSP; ++k2) incY[k2] += r.nu[k2] * rr;
            incT += r.q * rr;
        };
        // reactions four at a time: the four exponentials are independent
        // and interleave, the increments follow in reaction order
        int j = 0;
        for (; j + 4 <= P.n_rx; j += 4) {
            double k4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) k4[u] = rate_coeff_sub(P.rxk[j + u], lnTc, invTc, lnNs, tab);
#pragma unroll
            for (int u = 0; u < 4; ++u) apply(P.rxk[j + u], k4[u]);
        }
        for (; j < P.n_rx; ++j) apply(P.rxk[j], rate_coeff_sub(P.rxk[j], lnTc, invTc, lnNs, tab));
        if constexpr (LE) {
            // q_over_cp is the rise at c_p,ref: divide by c_p(Y) / c_p,ref
            // at the sub-step's composition (Eq. 7: omega_T / (rho c_p))
            double cpm = 0.0;
#pragma unroll
            for (int k = 0; k < NSP; ++k) cpm += Yc[k] * P.cpk[k];
            incT *= rcp(cpm);
        }
        // positivity limiter: scale the sub-step so that no mass fraction
        // is consumed below zero (1, i.e. plain Euler, otherwise)
        double lam = 1.0;
#pragma unroll
        for (int k = 0; k < NSP; ++k)
            if (incY[k] < 0.0 && Yc[k] + incY[k] < 0.0) lam = fmin(lam, fmax(Yc[k], 0.0) * rcp(-incY[k]));
        dT = fma(lam, incT, dT);
#pragma unroll
        for (int k = 0; k < NSP; ++k) dY[k] = fma(lam, incY[k], dY[k]);
    }
    srcT = dT;
#pragma unroll
    for (int k = 0; k < NSP; ++k) srcY[k] = dY[k];
    return nsub;
}

// ------------------------------------------------- central-moment transform
// Central moments about u (Sec. II.C, Eq. 21) of the 3 x 3 (x 3) cube of
// populations, one axis at a time.  Along a line with velocities -1, 0, 1
// holding (a, b, d): m0 = a+b+d, m1 = (d-a) - u m0,
// m2 = (a+d) + 2u(a-d) + u^2 m0.  Moment (p, q, r) lands at p + 3q + 9r.
template <class C>
__device__ __forceinline__ void cm_fwd_line(C &a, C &b, C &d, C u)
{
    C m0 = a + b + d;
    C m1 = (d - a) - u * m0;
    C m2 = (a + d) + (C)2 * u * (a - d) + u * u * m0;
    a = m0;
    b = m1;
    d = m2;
}

// exact inverse of cm_fwd_line
template <class C>
__device__ __forceinline__ void cm_inv_line(C &a, C &b, C &d, C u)
{
    C m0 = a, m1 = b, m2 = d;
    C uu = u * u;
    a = (C)0.5 * (m0 * (uu - u) + m1 * ((C)2 * u - (C)1) + m2);
    b = m0 * ((C)1 - uu) - (C)2 * u * m1 - m2;
    d = (C)0.5 * (m0 * (uu + u) + m1 * ((C)2 * u + (C)1) + m2);
}

template <int Q, class C>
__device__ __forceinline__ void central_fwd(C (&h)[Q], const C (&u)[3])
{
#pragma unroll
    for (int l = 0; l < Q / 3; ++l) cm_fwd_line(h[3 * l], h[3 * l + 1], h[3 * l + 2], u[0]);
#pragma unroll
    for (int zp = 0; zp < Q / 9; ++zp)
#pragma unroll
        for (int p = 0; p < 3; ++p) cm_fwd_line(h[9 * zp + p], h[9 * zp + p + 3], h[9 * zp + p + 6], u[1]);
    if constexpr (Q == 27) {
#pragma unroll
        for (int r = 0; r < 9; ++r) cm_fwd_line(h[r], h[r + 9], h[r + 18], u[2]);
    }
}

template <int Q, class C>
__device__ __forceinline__ void central_inv(C (&h)[Q], const C (&u)[3])
{
    if constexpr (Q == 27) {
#pragma unroll
        for (int r = 0; r < 9; ++r) cm_inv_line(h[r], h[r + 9], h[r + 18], u[2]);
    }
#pragma unroll
    for (int zp = 0; zp < Q / 9; ++zp)
#pragma unroll
        for (int p = 0; p < 3; ++p) cm_inv_line(h[9 * zp + p], h[9 * zp + p + 3], h[9 * zp + p + 6], u[1]);
#pragma unroll
    for (int l = 0; l < Q / 3; ++l) cm_inv_line(h[3 * l], h[3 * l + 1], h[3 * l + 2], u[0]);
}

// Relax toward the Maxwellian central moments at temperature cs^2: orders
// 0-1 kept, order 2 at 1/tau, order 3 at omega3, higher at omega4.
template <int Q, class C>
__device__ __forceinline__ void relax(C (&k)[Q], C om2, C om3, C om4)
{
    sfor<0, Q>([&](auto J) {
        constexpr int j = decltype(J)::value;
        constexpr int p = j % 3, q = (j / 3) % 3, r = (Q == 27) ? j / 9 : 0;
        constexpr int order = p + q + r;
        if constexpr (order >= 2) {
            constexpr bool odd = (p == 1) || (q == 1) || (r == 1);
            constexpr int n2 = (p == 2) + (q == 2) + (r == 2);
            constexpr double tgt = odd ? 0.0 : (n2 == 1 ? kCs2 : n2 == 2 ? kCs2 * kCs2 : kCs2 * kCs2 * kCs2);
            C om = order == 2 ? om2 : order == 3 ? om3 : om4;
            k[j] = k[j] - om * (k[j] - (C)tgt);
        }
    });
}

// Relaxation with the orders >= 4 taken as cumulants (the cumulant form of
// the collision, Sec. II.C).  For the unit-mass, zero-mean shifted
// distribution the cumulants of orders 2 and 3 are the central moments;
// those of orders 4-6 on the 3 x 3 (x 3) cube follow from the
// moment-cumulant relation, kappa_a = sum over the set partitions of a's
// index positions into blocks of two or more of the product of the blocks'
// cumulants (first-order blocks vanish), expanded here by hand:
//   order 4: C_xxyy = k_xxyy - k_xx k_yy - 2 k_xy^2,
//            C_xxyz = k_xxyz - k_xx k_yz - 2 k_xy k_xz;
//   order 5: C_xxyyz = k_xxyyz - k_xx k_yyz - k_yy k_xxz - 2 k_xz k_xyy
//                      - 2 k_yz k_xxy - 4 k_xy k_xyz;
//   order 6: C_xxyyzz = k_xxyyzz - (pair x 4-block: 15 terms)
//                       - (two triples: 10) - (three pairs: 15),
// and the inverse with the relaxed cumulants and the post-collision
// orders 2, 3.  Cumulants of order >= 4 relax at om4 toward 0 (those of the
// Maxwellian); orders 2, 3 as in relax().
template <int Q, class C>
__device__ __forceinline__ void relax_cumulants(C (&k)[Q], C om2, C om3, C om4)
{
    auto K = [&](int p, int q, int r) -> C & { return k[p + 3 * q + 9 * r]; };
    const C keep = (C)1 - om4;
    if constexpr (Q == 9) {
        const C c22 = K(2, 2, 0) - K(2, 0, 0) * K(0, 2, 0) - (C)2 * K(1, 1, 0) * K(1, 1, 0);
        relax<Q>(k, om2, om3, (C)0);
        K(2, 2, 0) = keep * c22 + K(2, 0, 0) * K(0, 2, 0) + (C)2 * K(1, 1, 0) * K(1, 1, 0);
    } else {
        // pre-collision second and third orders
        const C a = K(2, 0, 0), b = K(0, 2, 0), c = K(0, 0, 2);          // xx, yy, zz
        const C xy = K(1, 1, 0), xz = K(1, 0, 1), yz = K(0, 1, 1);
        const C xxy = K(2, 1, 0), xxz = K(2, 0, 1), xyy = K(1, 2, 0), yyz = K(0, 2, 1);
        const C xzz = K(1, 0, 2), yzz = K(0, 1, 2), xyz = K(1, 1, 1);
        // pre-collision cumulants of orders 4, 5, 6
        const C c220 = K(2, 2, 0) - a * b - (C)2 * xy * xy;
        const C c202 = K(2, 0, 2) - a * c - (C)2 * xz * xz;
        const C c022 = K(0, 2, 2) - b * c - (C)2 * yz * yz;
        const C c211 = K(2, 1, 1) - a * yz - (C)2 * xy * xz;
        const C c121 = K(1, 2, 1) - b * xz - (C)2 * xy * yz;
        const C c112 = K(1, 1, 2) - c * xy - (C)2 * xz * yz;
        const C c221 = K(2, 2, 1) - a * yyz - b * xxz - (C)2 * xz * xyy - (C)2 * yz * xxy - (C)4 * xy * xyz;
        const C c212 = K(2, 1, 2) - a * yzz - c * xxy - (C)2 * xy * xzz - (C)2 * yz * xxz - (C)4 * xz * xyz;
        const C c122 = K(1, 2, 2) - b * xzz - c * xyy - (C)2 * xy * yzz - (C)2 * xz * yyz - (C)4 * yz * xyz;
        const C s42 = a * c022 + b * c202 + c * c220 + (C)4 * (xy * c112 + xz * c121 + yz * c211);
        const C s33 = (C)2 * (xxy * yzz + xxz * yyz + xyy * xzz) + (C)4 * xyz * xyz;
        const C s222 = a * b * c + (C)2 * (a * yz * yz + b * xz * xz + c * xy * xy) + (C)8 * xy * xz * yz;
        const C c222 = K(2, 2, 2) - s42 - s33 - s222;
        relax<Q>(k, om2, om3, (C)0);
        // post-collision second and third orders, relaxed cumulants
        const C A = K(2, 0, 0), B = K(0, 2, 0), Cc = K(0, 0, 2);
        const C XY = K(1, 1, 0), XZ = K(1, 0, 1), YZ = K(0, 1, 1);
        const C XXY = K(2, 1, 0), XXZ = K(2, 0, 1), XYY = K(1, 2, 0), YYZ = K(0, 2, 1);
        const C XZZ = K(1, 0, 2), YZZ = K(0, 1, 2), XYZ = K(1, 1, 1);
        const C d220 = keep * c220, d202 = keep * c202, d022 = keep * c022;
        const C d211 = keep * c211, d121 = keep * c121, d112 = keep * c112;
        K(2, 2, 0) = d220 + A * B + (C)2 * XY * XY;
        K(2, 0, 2) = d202 + A * Cc + (C)2 * XZ * XZ;
        K(0, 2, 2) = d022 + B * Cc + (C)2 * YZ * YZ;
        K(2, 1, 1) = d211 + A * YZ + (C)2 * XY * XZ;
        K(1, 2, 1) = d121 + B * XZ + (C)2 * XY * YZ;
        K(1, 1, 2) = d112 + Cc * XY + (C)2 * XZ * YZ;
        K(2, 2, 1) = keep * c221 + A * YYZ + B * XXZ + (C)2 * XZ * XYY + (C)2 * YZ * XXY + (C)4 * XY * XYZ;
        K(2, 1, 2) = keep * c212 + A * YZZ + Cc * XXY + (C)2 * XY * XZZ + (C)2 * YZ * XXZ + (C)4 * XZ * XYZ;
        K(1, 2, 2) = keep * c122 + B * XZZ + Cc * XYY + (C)2 * XY * YZZ + (C)2 * XZ * YYZ + (C)4 * YZ * XYZ;
        const C S42 = A * d022 + B * d202 + Cc * d220 + (C)4 * (XY * d112 + XZ * d121 + YZ * d211);
        const C S33 = (C)2 * (XXY * YZZ + XXZ * YYZ + XYY * XZZ) + (C)4 * XYZ * XYZ;
        const C S222 = A * B * Cc + (C)2 * (A * YZ * YZ + B * XZ * XZ + Cc * XY * XY) + (C)8 * XY * XZ * YZ;
        K(2, 2, 2) = keep * c222 + S42 + S33 + S222;
    }
}

// ------------------------------------------------------------ reductions
__device__ __forceinline__ void diag_combine(double (&a)[kNDiag], const double *b)
{
    a[kSumG] += b[kSumG];
    a[kSumXi] += b[kSumXi];
    a[kMomX] += b[kMomX];
    a[kMomY] += b[kMomY];
    a[kMomZ] += b[kMomZ];
    a[kMaxY] = fmax(a[kMaxY], b[kMaxY]);
    a[kNonfinite] += b[kNonfinite];
    a[kTheta] += b[kTheta];
    if (b[kHrrMax] > a[kHrrMax] || (b[kHrrMax] == a[kHrrMax] && b[kHrrIdx] < a[kHrrIdx])) {
        a[kHrrMax] = b[kHrrMax];
        a[kHrrIdx] = b[kHrrIdx];
    }
    a[kWallQ] += b[kWallQ];
    a[kFuel] += b[kFuel];
    a[kFuelMass] += b[kFuelMass];
}

__device__ __forceinline__ void diag_identity(double (&a)[kNDiag])
{
#pragma unroll
    for (int s = 0; s < kNDiag; ++s) a[s] = 0.0;
    a[kHrrMax] = -INFINITY;
    a[kHrrIdx] = 1e300;
}

// Block reduction (wave64 butterflies, then the waves in order) of the
// per-thread diagnostics; thread 0 writes the block's partial.
__device__ __forceinline__ void block_reduce_diag(double (&a)[kNDiag], double *out)
{
    __shared__ double red[kBlock / 64][kNDiag];
    const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        double b[kNDiag];
#pragma unroll
        for (int s = 0; s < kNDiag; ++s) b[s] = __shfl_xor(a[s], off, 64);
        diag_combine(a, b);
    }
    if (lane == 0)
#pragma unroll
        for (int s = 0; s < kNDiag; ++s) red[wave][s] = a[s];
    __syncthreads();
    if (tid == 0) {
        const int nw = (blockDim.x * blockDim.y * blockDim.z + 63) / 64;
        for (int w = 1; w < nw; ++w) diag_combine(a, red[w]);
#pragma unroll
        for (int s = 0; s < kNDiag; ++s) out[s] = a[s];
    }
}

// ------------------------------------------------------------ step kernel
// Everything after the finite differences, for one fluid cell: Arrhenius
// source, Lambda (Eq. 6), Euler update, P_h (Eq. 13a), source Xi_i (Eq. 9),
// central-moment collision (Eqs. 14, 19, 21), diagnostics, stores.
// diffT, diffY already carry the factor alpha.
template <int Q, int NSP, int PREC, int MODE, bool LE = false, class Pops>
__device__ __forceinline__ void finish_cell(const KParams &P, long long idx, Pops &&g,
                                            const Pt<NSP, typename Prec<PREC>::calc> &ctr,
                                            const typename Prec<PREC>::calc (&u)[3],
                                            const typename Prec<PREC>::calc (&m)[3], typename Prec<PREC>::calc sg,
                                            typename Prec<PREC>::calc inv_rc, typename Prec<PREC>::calc diffT,
                                            const typename Prec<PREC>::calc (&diffY)[NSP],
                                            typename Prec<PREC>::calc CT, const typename Prec<PREC>::calc (&CY)[NSP],
                                            const typename Prec<PREC>::calc (&grad)[3], double wallq,
                                            double (&acc)[kNDiag])
{
    using L = Lat<Q>;
    using C = typename Prec<PREC>::calc;
    using S = typename Prec<PREC>::scal;
    constexpr bool DIAG = mode_reduces(MODE);
    const C rho = ctr.rho;
    // Arrhenius source (double): computed here, or read back from this
    // step's output scalars where the chemistry launch left it
    double srcT, srcY[NSP];
    if constexpr (chem_pass(NSP)) {
        const char *so = (const char *)P.sc_out;
        const size_t fstride = (size_t)P.N * sizeof(S);
        const uint32_t off = (uint32_t)idx * (uint32_t)sizeof(S);
        srcT = (double)ldo<S>(so, off);
#pragma unroll
        for (int k = 0; k < NSP; ++k) srcY[k] = (double)ldo<S>(so + (size_t)(1 + k) * fstride, off);
    } else {
        double Yd[NSP];
#pragma unroll
        for (int k = 0; k < NSP; ++k) Yd[k] = (double)ctr.Y[k];
        chemistry<NSP, LE>(P, kExp2Tab, kLogTab, (double)ctr.T, Yd, srcT, srcY);
    }

    // material derivatives, Lambda (Eq. 6), Euler update, P_h (Eq. 13a)
    const C DtT = diffT + (C)srcT;
    C DtY[NSP], invW = 0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) {
        DtY[k] = diffY[k] + (C)srcY[k];
        invW += ctr.Y[k] * (C)P.invW[k];
    }
    const C Wm = rcp(invW);
    C Lam = DtT * rcp(ctr.T);
#pragma unroll
    for (int k = 0; k < NSP; ++k) Lam += (Wm * (C)P.invW[k]) * DtY[k];
    const C Tn = ctr.T - CT + DtT;
    C Yn[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) Yn[k] = ctr.Y[k] - CY[k] + DtY[k];
    const C Ph = sg + (C)0.5 * rho * (C)kCs2 * Lam;

    if constexpr (MODE == kModeFields) {
        if (P.f_rho) P.f_rho[idx] = (double)rho;
        if (P.f_u)
#pragma unroll
            for (int d = 0; d < L::D; ++d) P.f_u[d * P.N + idx] = (double)u[d];
        if (P.f_Ph) P.f_Ph[idx] = (double)Ph;
        if (P.f_T) P.f_T[idx] = (double)ctr.T;
        if (P.f_Y)
#pragma unroll
            for (int k = 0; k < NSP; ++k) P.f_Y[k * P.N + idx] = (double)ctr.Y[k];
        return;
    }

    // the scalars' stores go out here, so that they need not be held through
    // the collision
    if constexpr (mode_advances(MODE)) {
        const uint32_t off = (uint32_t)idx * (uint32_t)sizeof(S);
        if constexpr (L::D == 3) {
            PlanePtr<S> ps(P.sc_out, 0, P.N);
            *ps.at(off) = (S)Tn;
#pragma unroll
            for (int k = 0; k < NSP; ++k) {
                ps.step(P.N);
                *ps.at(off) = (S)Yn[k];
            }
        } else {
            char *so = (char *)P.sc_out;
            const size_t fstride = (size_t)P.N * sizeof(S);
            sto<S>(so, off, (S)Tn);
#pragma unroll
            for (int k = 0; k < NSP; ++k) sto<S>(so + (size_t)(1 + k) * fstride, off, (S)Yn[k]);
        }
    }
    bool bad = false;
    if constexpr (DIAG) {
        bad = !isfinite((double)ctr.T);
#pragma unroll
        for (int k = 0; k < NSP; ++k) bad |= !isfinite((double)ctr.Y[k]);
        // (a sum with a term that is not finite is not finite; the terms are
        // looked at only where it is not, which it also is on overflow)
        if (__any(!isfinite((double)sg))) sfor<0, Q>([&](auto I) { bad |= !isfinite((double)g(I)); });
    }

    // source Xi_i (Eq. 9) and pre-conditioned populations (Eq. 19)
    const C uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    C xi[Q], h[Q], pi = 0, sxi = 0;
    const C half_inv = (C)0.5 * inv_rc;
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr C wi = (C)L::w(i);
        const C cu = (C)L::cx(i) * u[0] + (C)L::cy(i) * u[1] + (C)L::cz(i) * u[2];
        const C feq_r = wi * ((C)1 + (C)3 * cu + (C)4.5 * cu * cu - (C)1.5 * uu);
        const C proj = ((C)L::cx(i) - u[0]) * grad[0] + ((C)L::cy(i) - u[1]) * grad[1] +
                       ((C)L::cz(i) - u[2]) * grad[2];
        xi[i] = (C)kCs2 * (feq_r - wi) * proj + wi * rho * (C)kCs2 * Lam;
        sxi += xi[i];
        // (3-D: which product is rounded is stated, so that populations held in
        // registers or in LDS give the same bits)
        if constexpr (L::D == 3)
            h[i] = fma(g(I), inv_rc, xi[i] * half_inv);
        else
            h[i] = g(I) * inv_rc + xi[i] * half_inv;
        pi += h[i];
    });
    // unit-mass shift, central-moment relaxation, shift back (Eq. 14)
    const C sh = (C)1 - pi;
    sfor<0, Q>([&](auto I) { h[decltype(I)::value] += (C)L::w(decltype(I)::value) * sh; });
    central_fwd<Q>(h, u);
    if (P.collision == LBFD_CUMULANTS)
        relax_cumulants<Q>(h, (C)P.omega2, (C)P.omega3, (C)P.omega4);
    else
        relax<Q>(h, (C)P.omega2, (C)P.omega3, (C)P.omega4);
    central_inv<Q>(h, u);
    const C rc = rho * (C)kCs2;
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        h[i] = rc * (h[i] - (C)L::w(i) * sh) + (C)0.5 * xi[i];
    });

    if constexpr (DIAG) {
        if (bad) {
            acc[kNonfinite] = 1.0;
        } else {
            double sy = 0.0;
#pragma unroll
            for (int k = 0; k < NSP; ++k) sy += (double)ctr.Y[k];
            acc[kSumG] = (double)sg;
            acc[kSumXi] = (double)sxi;
            acc[kMomX] = (double)m[0] * 3.0;
            acc[kMomY] = (double)m[1] * 3.0;
            acc[kMomZ] = (double)m[2] * 3.0;
            acc[kMaxY] = fabs(sy - 1.0);
            acc[kTheta] = ((double)ctr.T - P.T_u) / (P.T_b - P.T_u);
            acc[kHrrMax] = srcT;
            acc[kHrrIdx] = (double)idx;
            acc[kWallQ] = wallq;
            acc[kFuel] = -srcY[0];
            acc[kFuelMass] = -srcY[0] * (double)ctr.rho;
        }
    }

    if constexpr (mode_advances(MODE)) {
        if constexpr (L::D == 3) {
            using T = typename Prec<PREC>::pop;
            PlanePtr<T> pl(P.pop_out, 0, P.N);
            sfor<0, Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                plane_store<Q, PREC, i>(pl.at((uint32_t)idx * (uint32_t)sizeof(T)), h[i]);
                pl.step(P.N);
            });
        } else {
            sfor<0, Q>(
                [&](auto I) { pop_store<Q, PREC, decltype(I)::value>(P.pop_out, P.N, idx, h[decltype(I)::value]); });
        }
    }
}

// ------------------------------------------------------------ tiles
// The pull of one cell of a tile.  The rows of the neighbour lines
// are the same for a wave (its lanes differ in x only), so an interior wave
// loads each population at a scalar base plus one of three lane offsets.
// Where the wave holds a boundary cell, a lane whose source is no fluid cell
// takes its own cell's opposite population by selecting the address (no
// branch and no wait between the loads); inlet, outlet and interpolated
// walls, which few waves hold, follow in passes of their own.
// m: the momentum sums (3-D).  In the mixed forms an interior cell's sum takes the
// stored value and its scale in one fused multiply-add, a boundary cell's the
// scaled population (one factor per lane and lattice weight tells them apart).
template <int Q, int PREC, bool CW>
__device__ __forceinline__ void tile_pull(const KParams &P, int x, int y, int z, long long tb, bool bnd,
                                          unsigned long long pcode, typename Prec<PREC>::calc (&g)[Q],
                                          typename Prec<PREC>::calc (&m)[3])
{
    using C = typename Prec<PREC>::calc;
    using T = typename Prec<PREC>::pop;
    using L = Lat<Q>;
    constexpr bool kStream = pop_stream<Q, PREC>() && !CW;  // (curved walls read them again)
    using R = std::conditional_t<PREC == LBFD_MIXED_FP16, unsigned short, T>;  // as loaded
    // wrapped neighbour coordinates (a wrapped source beyond a face that is
    // not periodic is never read: its code is not kPullFluid), as byte offsets
    // in a population's plane: three along the lane's row, nine rows
    constexpr uint32_t kB = sizeof(T);
    const uint32_t xs[3] = {kB * (uint32_t)(x == 0 ? P.nx - 1 : x - 1), kB * (uint32_t)x,
                            kB * (uint32_t)(x == P.nx - 1 ? 0 : x + 1)};
    const int ys[3] = {y == 0 ? P.ny - 1 : y - 1, y, y == P.ny - 1 ? 0 : y + 1};
    const int zs[3] = {z == 0 ? P.nz - 1 : z - 1, z, z == P.nz - 1 ? 0 : z + 1};
    uint32_t rows[3];  // (2-D)
#pragma unroll
    for (int k = 0; k < 3; ++k) rows[k] = (uint32_t)(ys[k] * P.nx) * kB;
    auto off = [&](int ox, int oy, int oz) -> uint32_t {
        if constexpr (L::D == 2) return rows[1 + oy] + xs[1 + ox];
        return (uint32_t)((zs[1 + oz] * P.ny + ys[1 + oy]) * P.nx) * kB + xs[1 + ox];
    };
    const uint32_t own = off(0, 0, 0);
    auto raw = [](R v) -> C {
        if constexpr (PREC == LBFD_MIXED_FP16)
            return __half2float(__builtin_bit_cast(__half, v));
        else
            return v;
    };
    auto scale = [](auto I) -> C {
        return PREC == LBFD_FP64 ? (C)1 : (C)(float)(L::w(decltype(I)::value) * kCs2);
    };
    auto widen = [&](R v, auto I) -> C {
        if constexpr (PREC == LBFD_FP64)
            return v;
        else
            return raw(v) * scale(I);
    };
    // sum of c v s over the populations (v with its scale s)
    auto momentum = [&](auto &&v, auto &&sc) {
        if constexpr (L::D == 2) return;
        m[0] = m[1] = m[2] = 0;
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            auto add = [&](C &acc, auto sign) {
                if constexpr (PREC == LBFD_FP64)
                    acc += (C)decltype(sign)::value * v(I);
                else
                    acc = fma(v(I), (C)decltype(sign)::value * sc(I), acc);
            };
            if constexpr (L::cx(i) != 0) add(m[0], std::integral_constant<int, L::cx(i)>{});
            if constexpr (L::cy(i) != 0) add(m[1], std::integral_constant<int, L::cy(i)>{});
            if constexpr (L::cz(i) != 0) add(m[2], std::integral_constant<int, L::cz(i)>{});
        });
    };
    C v[Q];
    if (!__any(bnd)) {
        PlanePtr<const R> pl(P.pop_in, 0, P.N);
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (L::D == 2)
                // (one offset for the lane, the shift in the scalar base)
                v[i] = raw(*((const R *)P.pop_in + i * P.N - (L::cy(i) * P.nx + L::cx(i)) + own / kB));
            else
                v[i] = raw(load_global<kStream>(pl.at(off(-L::cx(i), -L::cy(i), -L::cz(i)))));
            g[i] = PREC == LBFD_FP64 ? v[i] : v[i] * scale(I);
            pl.step(P.N);
        });
        momentum([&](auto I) { return v[decltype(I)::value]; }, scale);
        return;
    }
    {
        PlanePtr<const R> pl(P.pop_in, 0, P.N), po(P.pop_in, Q - 1, P.N);  // directions i and opposite
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            const auto *src = pl.at(off(-L::cx(i), -L::cy(i), -L::cz(i))), *opp = po.at(own);
            if constexpr (L::D == 2) {
                // both, so that the loads need not wait for the code
                const R a = load_global<kStream>(src), b = load_global<kStream>(opp);
                v[i] = raw(decode_pull_kind(pcode, i) == kPullFluid ? a : b);
            } else {
                v[i] = raw(load_global<kStream>(decode_pull_kind(pcode, i) == kPullFluid ? src : opp));
            }
            g[i] = PREC == LBFD_FP64 ? v[i] : v[i] * scale(I);
            pl.step(P.N);
            po.step(-P.N);
        });
    }
    if (__any((pcode & 0xaaaaaaaaaaaaaaaaull) != 0)) {
        // inlets (Eq. 31: + 2 w_I rho_in c_I.u_in; an x face carries the
        // per-cell profile indexed by the cell's (y, z), the same for a wave)
        // and outlets (the value kept in the outlet buffer)
        const long long s3 = (long long)P.ny * P.nz, o = (long long)z * P.ny + y;
        const bool in0 = x == 0 && P.face[0] == LBFD_FACE_INFLOW, in1 = x == P.nx - 1 && P.face[1] == LBFD_FACE_INFLOW;
        double p0[3], p1[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            p0[d] = P.inflow_u[d * s3 + o];
            p1[d] = P.inflow_u[(3 + d) * s3 + o];
        }
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i != (Q - 1) / 2) {
                constexpr int cx = L::cx(i), cy = L::cy(i), cz = L::cz(i);
                const int kind = decode_pull_kind(pcode, i);
                const bool inflow = kind == kPullInflow;
                if (__any(inflow)) {
                    const double cu0 = cx * p0[0] + cy * p0[1] + cz * p0[2], cu1 = cx * p1[0] + cy * p1[1] + cz * p1[2];
                    double cu = cx * P.u_in[0] + cy * P.u_in[1] + cz * P.u_in[2];
                    if constexpr (cx == 1) cu = in0 ? cu0 : cu;
                    if constexpr (cx == -1) cu = in1 ? cu1 : cu;
                    g[i] = inflow ? g[i] + (C)(2.0 * L::w(i) * P.rho_in * cu) : g[i];
                }
                if constexpr (cx != 0) {
                    const bool outlet = kind == kPullOutlet;
                    if (__any(outlet)) {
                        const C ov = (C)P.outlet[outlet_index(P, cx < 0 ? 1 : 0, i, Q, y, z)];
                        g[i] = outlet ? ov : g[i];
                    }
                }
            }
        });
    }
    if constexpr (CW) {
        // linearly interpolated bounce-back (post-collision form) for a
        // wall met at the fraction q of the link toward it (direction OPP).
        // Bound by the latency of its loads, which depend on one another:
        // hence every direction's q first, then the populations of nine
        // directions, in flight together.  (One direction after the other
        // the pass waited 26 times for a q and then for the populations: 160 x
        // 128 x 96 packing, FP64 / single / half, 683 / 545 / 511 us a step;
        // now 479 / 434 / 408.)
        if (P.bq != nullptr && __any((pcode & ~(pcode >> 1) & 0x5555555555555555ull) != 0)) {
            const uint32_t tq = (uint32_t)tb * (uint32_t)sizeof(float);
            float qs[Q];
            {
                PlanePtr<const float> pq(P.bq, 0, P.n_boundary);
                sfor<0, Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    qs[i] = __builtin_nanf("");
                    if constexpr (i != (Q - 1) / 2) qs[i] = *pq.at(tq);
                    pq.step(P.n_boundary);
                });
            }
            PlanePtr<const R> pl(P.pop_in, 0, P.N), po(P.pop_in, Q - 1, P.N);
            sfor<0, Q / 9>([&](auto B) {
                constexpr int b = 9 * decltype(B)::value;
                R vfar[9], vown[9];
                // q < 1/2: the far node r + c_I is the pull source of
                // direction OPP (when it is a fluid cell)
                auto interp = [&](auto I) -> bool {
                    constexpr int i = decltype(I)::value;
                    return decode_pull_kind(pcode, i) == kPullBounce && qs[i] == qs[i];
                };
                auto use_far = [&](auto I) -> bool {
                    constexpr int i = decltype(I)::value;
                    return interp(I) && qs[i] < 0.5f && decode_pull_kind(pcode, Q - 1 - i) == kPullFluid;
                };
                sfor<b, b + 9>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    vfar[i - b] = vown[i - b] = R();
                    if constexpr (i != (Q - 1) / 2) {
                        if (__any(interp(I))) {
                            vfar[i - b] = *po.at(use_far(I) ? off(L::cx(i), L::cy(i), L::cz(i)) : own);
                            vown[i - b] = *pl.at(own);
                        }
                    }
                    pl.step(P.N);
                    po.step(-P.N);
                });
                sfor<b, b + 9>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if constexpr (i != (Q - 1) / 2) {
                        asm("" : "+v"(qs[i]));  // (the lane masks formed again, not kept in scalars)
                        if (__any(interp(I))) {
                            const C q2 = (C)2 * (C)qs[i];  // weights in the arithmetic precision
                            const bool far_half = use_far(I), near_wall = interp(I) && !(qs[i] < 0.5f);
                            const C gfar = widen(vfar[i - b], I), gown = widen(vown[i - b], I);
                            const C lo = q2 * g[i] + ((C)1 - q2) * gfar;
                            const C iq = (C)1 / (near_wall ? q2 : (C)1);
                            const C hi = g[i] * iq + (q2 - (C)1) * iq * gown;
                            g[i] = far_half ? lo : near_wall ? hi : g[i];
                        }
                    }
                });
            });
        }
    }
    if constexpr (PREC == LBFD_FP64) {
        momentum([&](auto I) { return g[decltype(I)::value]; }, scale);
    } else {
        if constexpr (L::D == 2) return;
        // one factor per squared speed
        constexpr int kMid = (Q - 1) / 2, kEdge = L::D == 3 ? 9 : 0;
        const C f[4] = {bnd ? (C)1 : scale(std::integral_constant<int, kMid>{}),
                        bnd ? (C)1 : scale(std::integral_constant<int, kMid - 1>{}),
                        bnd ? (C)1 : scale(std::integral_constant<int, kEdge>{}),
                        bnd ? (C)1 : scale(std::integral_constant<int, 0>{})};
        sfor<0, Q>([&](auto I) { v[decltype(I)::value] = bnd ? g[decltype(I)::value] : v[decltype(I)::value]; });
        momentum([&](auto I) { return v[decltype(I)::value]; },
                 [&](auto I) {
                     constexpr int i = decltype(I)::value;
                     return f[L::cx(i) * L::cx(i) + L::cy(i) * L::cy(i) + L::cz(i) * L::cz(i)];
                 });
    }
}

// The lowest kind bit of the slots (five bits each) whose kind is kInflow.
__device__ __forceinline__ unsigned inflow_slots(unsigned s20)
{
    static_assert(kInflow == 3 && kOutflow == 4, "the only kind with its two low bits set");
    return s20 & (s20 >> 1) & 0x8421u;
}

// Ghosts behind isothermal walls among the stencil points m = -2, -1, 1, 2
// of a cell along axis d (Dirichlet 2 phi_B - phi(I) for T, the density ghost
// reconstructed from its wall value; Sec. III.B): T(j) and R(j) hold the image
// values and receive the ghosts, wall_density(j, Tw) is the density at the
// wall with the composition of slot j.  The two points of a side share their
// wall, the first non-fluid point from the cell (the kinds of both slots are
// its kind when it is the first neighbour), hence one wall temperature a side.
// c: the cell's coordinate along the axis of n cells; off: the points' cell
// offsets along the wrapped axis.
template <bool DIAG, class C, class FT, class FR, class FD, class FQ>
__device__ __forceinline__ void iso_ghosts(const KParams &P, int d, int c, int n, long long idx, const int (&off)[4],
                                           unsigned s20, FT &&T, FR &&R, FD &&wall_density, FQ &&heat, double &wallq)
{
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int j1 = side ? 2 : 1, j2 = side ? 3 : 0;
        const int k1 = (int)(s20 >> (5 * j1)) & 7, k2 = (int)(s20 >> (5 * j2)) & 7;
        const bool iso1 = k1 == kIso, iso2 = k2 == kIso;
        if (__any(iso2)) {
            const bool second = k1 == kFluid;
            const int mw = (side ? 1 : -1) * (second ? 2 : 1);
            const bool out = (unsigned)(c + mw) >= (unsigned)n && !((P.periodic_bits >> (2 * d + side)) & 1u);
            const double *tw = out ? P.face_Td + (2 * d + side) : P.wall_T + (idx + off[second ? j2 : j1]);
            const C Tw = (C)*(iso2 ? tw : P.face_Td);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int j = q ? j2 : j1;
                const bool iso = q ? iso2 : iso1;
                const C rb = wall_density(j, Tw);
                R(j) = iso ? (C)2 * rb - R(j) : R(j);
                T(j) = iso ? (C)2 * Tw - T(j) : T(j);
            }
            if constexpr (DIAG) {
                const double q = heat(Tw);
                wallq += iso1 ? q : 0.0;
            }
        }
    }
}

// The stencil points m = -2, -1, 1, 2 of one cell of a 3-D tile along axis d
// (T, rho, Y_k), ghosts included; near: some point lies behind a wall.  A
// ghost's image is a cell of the same line (the point itself, the cell, a
// first neighbour), so boundary lanes select their four cells and the loads
// are those of interior lanes; ghost values are formed by selection where a
// lane of the wave has one on this axis.
// d1r: the density's first derivative (d1).  An interior cell leaves the
// constant factor of the first point's density to the difference that takes
// it (one rounding less); the select keeps that form beside the boundary
// cells' formed densities.
template <int NSP, int PREC, bool DIAG, bool CW>
__device__ __forceinline__ void tile_stencil(const KParams &P, int d, int x, int y, int z, long long idx,
                                             long long tb, bool bnd, unsigned long long scode,
                                             const Pt<NSP, typename Prec<PREC>::calc> &ctr,
                                             Pt<NSP, typename Prec<PREC>::calc> (&pv)[4], bool &near,
                                             typename Prec<PREC>::calc &d1r, double &wallq)
{
    using C = typename Prec<PREC>::calc;
    const int c = d == 0 ? x : d == 1 ? y : z, n = d == 0 ? P.nx : d == 1 ? P.ny : P.nz;
    const int stride = d == 0 ? 1 : d == 1 ? P.nx : P.nx * P.ny;
    int off[4];  // cell offsets of m = -2, -1, 1, 2 along the (wrapped) axis
#pragma unroll
    for (int j = 0; j < 4; ++j) off[j] = (wrap_once(c + slot_offset(j), n) - c) * stride;
    const unsigned s20 = (unsigned)(scode >> (20 * d)) & 0xfffffu;  // this axis' four slots of five bits
    int at[4] = {off[0], off[1], off[2], off[3]};
    if (__any(s20 != 0)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // the two bits of the image: self, cell, mirror, same
            const bool b0 = (s20 >> (5 * j + 3)) & 1u, b1 = (s20 >> (5 * j + 4)) & 1u;
            const int same = off[j < 2 ? 1 : 2], mirror = off[j < 2 ? 2 : 1];
            const int lo = b0 ? 0 : off[j], hi = b0 ? same : mirror;
            at[j] = b1 ? hi : lo;
        }
    }
    using S = typename Prec<PREC>::scal;
    static_assert(std::is_same_v<S, C>, "image points and cells hold the same type");
    const unsigned kinds = s20 & 0x39ce7u;  // the kinds of the four slots
    near = kinds != 0;
    // ghosts with an image point of their own take its values in place of the
    // mirror cell's: the lane's address and plane stride are selected, so that
    // the points' loads stay in flight together (with a pass of loads a slot,
    // one after the other, the images of 160 x 128 x 96 added 133 us in FP64 and
    // 120 in half beside their reconstruction; now some 30)
    int li[4] = {-1, -1, -1, -1};
    bool images = false;
    if constexpr (CW) {
        if (P.bimg != nullptr && __any(near)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) li[j] = near ? P.bimg[(d * 4 + j) * P.n_boundary + tb] : -1;
            images = __any(li[0] >= 0 || li[1] >= 0 || li[2] >= 0 || li[3] >= 0);
        }
    }
    if (images) {
        const S *img = (const S *)P.img_val;
        const S *q[4];
        uint32_t step[4];  // in elements (n_img < 2^31)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            q[j] = li[j] >= 0 ? img + li[j] : (const S *)P.sc_in + (idx + at[j]);
            step[j] = (uint32_t)(li[j] >= 0 ? P.n_img : P.N);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) pv[j].T = *q[j];
#pragma unroll
        for (int k = 0; k < NSP; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                q[j] += step[j];
                pv[j].Y[k] = *q[j];
            }
        C ri[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) ri[j] = img[(1 + NSP) * P.n_img + (li[j] >= 0 ? li[j] : 0)];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const C r = density<NSP>(P, pv[j].T, pv[j].Y);
            pv[j].rho = li[j] >= 0 ? ri[j] : r;
        }
    } else {
        uint32_t bo[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) bo[j] = (uint32_t)((int)idx + at[j]) * (uint32_t)sizeof(S);
        PlanePtr<const S> pl(P.sc_in, 0, P.N);
#pragma unroll
        for (int j = 0; j < 4; ++j) pv[j].T = *pl.at(bo[j]);
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            pl.step(P.N);
#pragma unroll
            for (int j = 0; j < 4; ++j) pv[j].Y[k] = *pl.at(bo[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) pv[j].rho = density<NSP>(P, pv[j].T, pv[j].Y);
    }
    const C r0 = density_rcp<NSP>(P, pv[0].T, pv[0].Y);
    if (__any(near)) {
        iso_ghosts<DIAG, C>(
            P, d, c, n, idx, off, s20, [&](int j) -> C & { return pv[j].T; }, [&](int j) -> C & { return pv[j].rho; },
            [&](int j, C Tw) -> C { return density<NSP>(P, Tw, pv[j].Y); },
            [&](C Tw) -> double {
                return 2.0 * P.alpha * (double)density<NSP>(P, Tw, ctr.Y) * ((double)ctr.T - (double)Tw);
            },
            wallq);
        if (__any(inflow_slots(s20) != 0)) {
            // Dirichlet ghosts of T, Y_k and rho at the inlet
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool in = ((s20 >> (5 * j)) & 7u) == (unsigned)kInflow;
                pv[j].rho = in ? (C)2 * (C)P.rho_in - pv[j].rho : pv[j].rho;
                pv[j].T = in ? (C)2 * (C)P.T_in - pv[j].T : pv[j].T;
#pragma unroll
                for (int k = 0; k < NSP; ++k)
                    pv[j].Y[k] = in ? (C)2 * (C)P.Y_in[k] - pv[j].Y[k] : pv[j].Y[k];
            }
        }
    }
    const C f0 = bnd ? (C)1 : (C)P.T_ref_over_W_ref, ra = bnd ? pv[0].rho : r0;
    const C lo = fma(f0, ra, -((C)8 * pv[1].rho)), hi = (C)8 * pv[2].rho - pv[3].rho;
    d1r = (lo + hi) * (C)(1.0 / 12.0);
}

// 2-D: the populations entering through outflow face f at face cell idx
// (Eq. 32): g_i(r) <- g_i(r-n)(cs - u.n) + g_i(r)(1 - cs + u.n) with the
// post-streaming values and velocity of this level; pc: the cell's pull code
// (whose outlet kinds imply a fluid inner neighbour; without one there may be
// no inner cell at all: a box of one cell in x).
template <int Q, int PREC>
__device__ __forceinline__ void outlet_2d(const KParams &P, int f, int x, int y, long long idx, unsigned long long pc,
                                          typename Prec<PREC>::calc ux, const typename Prec<PREC>::calc (&g)[Q])
{
    using L = Lat<Q>;
    using C = typename Prec<PREC>::calc;
    // (in half precision by selection: 2048 x 512 burner 36.5 us a step, behind
    // the branch 36.9; in FP64 the branch is the faster, 256 x 64 8.0 and 8.4)
    if constexpr (PREC != LBFD_MIXED_FP16)
        if (!pulls_outlet(pc)) return;
    const int sign = f ? 1 : -1;
    const long long in = pulls_outlet(pc) ? idx - sign : idx;
    const unsigned long long pci = P.code[in] == kCodeBoundary ? P.cell_code[in].x : 0;
    const C cs = (C)0.57735026918962576451;
    const C un = (C)sign * ux;
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (L::cx(i) != 0) {
            if (L::cx(i) == -sign && decode_pull_kind(pc, i) == kPullOutlet) {
                // the inner cell's source is a neighbour inside the box along x
                const int kind = decode_pull_kind(pci, i);
                const bool fluid = kind == kPullFluid;
                const uint32_t src = (uint32_t)cell_at(x, y, 0, 0, -L::cy(i), 0, P.nx, P.ny, 1);
                C G = pop_load_pair<Q, PREC, i>(P.pop_in, P.N, !fluid, fluid ? src : (uint32_t)in);
                if (kind == kPullInflow)
                    G += (C)(2.0 * L::w(i) * P.rho_in *
                             (L::cx(i) * P.u_in[0] + L::cy(i) * P.u_in[1] + L::cz(i) * P.u_in[2]));
                P.outlet[outlet_index(P, f, i, Q, y, 0)] = (double)(G * (cs - un) + g[i] * ((C)1 - cs + un));
            }
        }
    });
}

// Tile of one 256-thread block: 16 x 16 cells in 2-D (a wave 16 x 4), 64 x 2 x 2
// in 3-D (a wave one row); THIN, for boxes that would leave most of such a
// tile's lanes outside: 64 x 4, and 8 x 8 x 4 (a wave 8 x 8).
template <int D, bool THIN> struct TileShape {
    static constexpr int X = D == 2 ? (THIN ? kThinX2 : kTileX2) : (THIN ? kThinX3 : kTileX3),
                         Y = D == 2 ? (THIN ? kThinY2 : kTileY2) : (THIN ? kThinY3 : kTileY3),
                         Z = D == 2 ? 1 : (THIN ? kThinZ3 : kTileZ3);
    static_assert(X * Y * Z == kBlock, "a thread a cell");
};

// One tile (bx, by, bz) of the step: its threads work on every fluid cell.  A
// boundary cell (some pull source or finite-difference point is no in-box
// fluid cell) differs from an interior one in its addresses and in ghost
// values, both selected per lane from the cell's two 64-bit codes under
// wave-uniform conditions (some lane of the wave is a boundary cell), so that
// the cache lines that interior and boundary cells share are fetched and
// written once and no list of boundary cells, with its chain of dependent
// loads, is walked.  Interior tiles and listed boundary cells apart moved 53 GB
// a step on a 512 x 256 x 256 packing with 9 species, 2.6 times what the cells
// need; in 2-D the list's chain was most of a small box's step (channel of
// 256 x 64, FP64: 11.7 -> 8.6 us; 70 x 37: 16.0 -> 10.6 us).
// 2-D tiles are 16 x 16 because the near-wall work is a wave's when any of its
// lanes has it, and because a square halo is smaller (400 points, 544 around
// 64 x 4): a burner of 2048 x 512 with cylinders every 64 cells issues 1160
// vector instructions a wave against 1596 (FP64), 63 us a step against 75
// (tiles and a list 64; the step with diagnostics 86, 106; a field read 46,
// 67), in half precision 1103 against 1520, 40 us against 50 (40; 64, 67; 32).
// Waves of 8 x 8 cells issue 2 % fewer and take as long.  The kernel then moves
// 211 MB in FP64 (273 MB before), 3.4 TB/s; in half precision it is bound by
// its instructions.
// (tx, ty, tz): the thread's place in the tile, in 3-D ty and tz the same for
// a wave (THIN: tz);
// slot: the block's row of the diagnostics partials.
// CW: boundary cells apply the curved-wall treatments when listed: the
// interpolated bounce-back of P.bq and the Shepard image points of P.bimg (a
// separate instantiation, so that contexts without them keep the registers
// of plain bounce-back and axis-mirror ghosts).
template <int Q, int NSP, int PREC, int MODE, bool CW = false, bool LE = false, bool THIN = false>
__device__ __forceinline__ void step_block(const KParams &P, int bx, int by, int bz, int tx, int ty, int tz,
                                           long long slot)
{
    using L = Lat<Q>;
    using C = typename Prec<PREC>::calc;
    using S = typename Prec<PREC>::scal;
    constexpr int D = L::D;
    constexpr bool DIAG = mode_reduces(MODE);
    using TS = TileShape<D, THIN>;
    const int x = bx * TS::X + tx, y = by * TS::Y + ty, z = bz * TS::Z + tz;
    const bool inbox = x < P.nx && y < P.ny && z < P.nz;
    const long long idx = inbox ? ((long long)z * P.ny + y) * P.nx + x : 0;
    const int code = inbox ? (int)P.code[idx] : (int)kCodeSolid;
    const bool active = code != kCodeSolid, bnd = code == kCodeBoundary;
    double acc[kNDiag];
    if constexpr (DIAG) diag_identity(acc);

    // 2-D: T, Y_k and rho of the tile's cells and a 2-cell halo staged
    // once in LDS (field-major planes of 20 x 20 points, THIN 68 x 8); every finite-
    // difference point and ghost image is then an LDS read.  Points across a
    // periodic face wrap; a point beyond an inflow face holds the ghost itself
    // (Dirichlet T, Y_k, rho), which depends on the point alone; others beyond
    // the box hold the nearest in-box point's values and are never read.
    constexpr int kTX = TS::X, kTY = TS::Y, kHX = kTX + 4, kHY = kTY + 4, kNP = kHX * kHY;
    constexpr bool TILE = D == 2;
    __shared__ C tile[TILE ? (NSP + 2) * kNP : 1];
    C g[Q], m[3] = {0, 0, 0};
    long long tb = 0;  // the cell's place in the curved-wall tables
    unsigned long long pcode = 0, scode = 0;
    auto load_codes = [&] {
        if (bnd) {
            const ulonglong2 cc = P.cell_code[idx];
            pcode = cc.x;
            scode = cc.y;
            if constexpr (CW) tb = P.bslot[idx];
        }
    };
    if constexpr (TILE) {
        // the staging loads go out first, every thread's (at most three)
        // points before any is stored, so that they are in flight together
        // with the cell's codes and pulls
        const int tid = tx + kTX * ty;
        const int gx0 = bx * kTX - 2, gy0 = by * kTY - 2;
        const bool edge = gx0 < 0 || gy0 < 0 || gx0 + kHX > P.nx || gy0 + kHY > P.ny;  // the same for the block
        constexpr int kRounds = (kNP + kBlock - 1) / kBlock;
        Pt<NSP, C> pt[kRounds];
        bool in[kRounds];
        // coordinate v of an axis of n cells between faces f and f + 1, moved
        // into the box; dist: how far beyond an inflow face it was (0: not)
        auto inside = [&](int v, int n, int f, int &dist) -> int {
            const int lo = P.face[f], hi = P.face[f + 1];
            dist = v < 0 && lo == LBFD_FACE_INFLOW ? -v : v >= n && hi == LBFD_FACE_INFLOW ? v - n + 1 : 0;
            if (v < 0) v = lo == LBFD_FACE_PERIODIC ? v + n : lo == LBFD_FACE_INFLOW ? dist - 1 : 0;
            if (v >= n) v = hi == LBFD_FACE_PERIODIC && v - n < 2 ? v - n : hi == LBFD_FACE_INFLOW ? n - dist : n - 1;
            return min(max(v, 0), n - 1);
        };
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int i = tid + r * kBlock;
            int gx = gx0 + i % kHX, gy = gy0 + i / kHX;
            in[r] = false;
            if (edge) {
                const int sx = gx < 0 ? -1 : 1, sy = gy < 0 ? -1 : 1;
                int dx, dy;
                gx = inside(gx, P.nx, 0, dx);
                gy = inside(gy, P.ny, 2, dy);
                in[r] = dx == 1 || dx == 2 || dy == 1 || dy == 2;
                // the second ghost's image is the mirror cell where that is
                // fluid, else the face cell
                if (dx == 2 && P.code[(long long)gy * P.nx + gx] == kCodeSolid) gx = min(max(gx + sx, 0), P.nx - 1);
                if (dy == 2 && P.code[(long long)gy * P.nx + gx] == kCodeSolid) gy = min(max(gy + sy, 0), P.ny - 1);
            }
            if (kNP % kBlock == 0 || r + 1 < kRounds || i < kNP)
                load_point<NSP, PREC>(P, (long long)gy * P.nx + gx, pt[r]);
        }
        load_codes();
        if (active) tile_pull<Q, PREC, CW>(P, x, y, z, tb, bnd, pcode, g, m);
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int i = tid + r * kBlock;
            if (edge && __any(in[r])) {
                pt[r].T = in[r] ? (C)2 * (C)P.T_in - pt[r].T : pt[r].T;
                pt[r].rho = in[r] ? (C)2 * (C)P.rho_in - pt[r].rho : pt[r].rho;
#pragma unroll
                for (int k = 0; k < NSP; ++k) pt[r].Y[k] = in[r] ? (C)2 * (C)P.Y_in[k] - pt[r].Y[k] : pt[r].Y[k];
            }
            if (i < kNP) {
                tile[i] = pt[r].T;
                tile[kNP + i] = pt[r].rho;
#pragma unroll
                for (int k = 0; k < NSP; ++k) tile[(2 + k) * kNP + i] = pt[r].Y[k];
            }
        }
        __syncthreads();
    } else {
        load_codes();
    }
    const int ic = (ty + 2) * kHX + tx + 2;  // the cell's place in the LDS tile

    if (active) {
        // streaming with boundary conditions (2-D: issued above)
        if constexpr (!TILE) tile_pull<Q, PREC, CW>(P, x, y, z, tb, bnd, pcode, g, m);
        Pt<NSP, C> ctr;
        if constexpr (TILE) {
            ctr.T = tile[ic];
            ctr.rho = tile[kNP + ic];
#pragma unroll
            for (int k = 0; k < NSP; ++k) ctr.Y[k] = tile[(2 + k) * kNP + ic];
        } else {
            load_point<NSP, PREC>(P, idx, ctr);
        }
        const C rho = ctr.rho;

        // moments: sum g and sum c g (Eq. 13; in 3-D formed with the pull)
        C sg = 0;
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            sg += g[i];
            if constexpr (D == 2) {
                if constexpr (L::cx(i) == 1) m[0] += g[i];
                if constexpr (L::cx(i) == -1) m[0] -= g[i];
                if constexpr (L::cy(i) == 1) m[1] += g[i];
                if constexpr (L::cy(i) == -1) m[1] -= g[i];
            }
        });
        // 3-D: the populations wait in LDS while the stencils are evaluated
        // where their registers make the difference.  FP64 with more than 4
        // species: with them two waves a SIMD spill 34 registers, which moved 1
        // GB of the 4.1 GB of a step on 256 x 128 x 128 through memory (1046 ->
        // 889 us).  Mixed with up to 4: 148 -> 122 registers, four waves for
        // three (161 x 99 x 83, half: 139 -> 123 us).  FP64 with up to 4 would
        // stay at two waves, mixed with more at three (154 us either way).
        constexpr bool STASH = D == 3 && (PREC == LBFD_FP64) == (NSP > 4) && MODE != kModeFields;
        __shared__ C pops[STASH ? Q * kBlock : 1];
        if constexpr (STASH) {
            sfor<0, Q>([&](auto I) { pops[decltype(I)::value * kBlock + threadIdx.x] = g[decltype(I)::value]; });
            asm volatile("" ::: "memory");
        }
        const C inv_rho = rcp(rho);
        const C inv_rc = (C)3 * inv_rho;  // 1 / (rho cs^2)
        const C u[3] = {m[0] * inv_rc, m[1] * inv_rc, m[2] * inv_rc};
        if constexpr (D == 2 && mode_advances(MODE)) {
            // (here, while few values are live)
#pragma unroll
            for (int f = 0; f < 2; ++f)
                if (P.face[f] == LBFD_FACE_OUTFLOW && x == (f ? P.nx - 1 : 0))
                    outlet_2d<Q, PREC>(P, f, x, y, idx, pcode, u[0], g);
        }

        // finite differences per axis with ghost nodes (Sec. II.D, III.B);
        // one axis at a time, one scalar at a time, to bound register use
        C diffT = 0, CT = 0, grad[3] = {0, 0, 0};
        C diffY[NSP], CY[NSP];
#pragma unroll
        for (int k = 0; k < NSP; ++k) diffY[k] = CY[k] = 0;
        double wallq = 0.0;
        // mixture-averaged transport (Sec. II.A, Eq. 2 and Eq. 7): the cell's
        // 1/W, c_p and their reciprocals; div V_c summed over the axes
        C Mc = 0, cpc = 0, divVc = 0;
        if constexpr (LE) {
#pragma unroll
            for (int k = 0; k < NSP; ++k) {
                Mc += ctr.Y[k] * (C)P.invW[k];
                cpc += ctr.Y[k] * (C)P.cpk[k];
            }
        }
        const C inv_M = LE ? rcp(Mc) : (C)0, inv_cp = LE ? rcp(cpc) : (C)0;
        auto axis_terms = [&](auto &&val, C d1r, bool near, C ud) {
            // val(f, m): field f (0 = T, 2 + k = Y_k) at offset m = -2..2;
            // d1r: the derivative of rho
            const C uh = (C)0.5 * ud;  // the conv2 values are twice the derivatives
            C t1, t2;
            {
                C tc;
                axis5(val(0, -2), val(0, -1), ctr.T, val(0, 1), val(0, 2), ud, near, t1, t2, tc);
                if constexpr (!LE) diffT += t2 + d1r * t1 * inv_rho;
                CT += uh * tc;
            }
            C cY[NSP], sumc = 0, y1[NSP], y2[NSP];
#pragma unroll
            for (int k = 0; k < NSP; ++k) {
                axis5(val(2 + k, -2), val(2 + k, -1), ctr.Y[k], val(2 + k, 1), val(2 + k, 2), ud, near, y1[k], y2[k],
                      cY[k]);
                if constexpr (!LE) diffY[k] += y2[k] + d1r * y1[k] * inv_rho;
                sumc += cY[k];
            }
            if constexpr (LE) {
                // along this axis, in units of alpha: d ln W = l1, d2 ln W = l2
                // (from 1/W = sum Y_k / W_k, linear in Y_k), G_k = (W_k/W) dX_k
                // = dY_k + Y_k l1, V_c = sum D_k G_k, and sum_k c_pk Y_k V_k
                C M1 = 0, M2 = 0, cp1 = 0;
#pragma unroll
                for (int k = 0; k < NSP; ++k) {
                    M1 += y1[k] * (C)P.invW[k];
                    M2 += y2[k] * (C)P.invW[k];
                    cp1 += y1[k] * (C)P.cpk[k];
                }
                const C l1 = -M1 * inv_M;
                const C l2 = l1 * l1 - M2 * inv_M;
                const C rr = d1r * inv_rho;
                C Vc = 0, H = 0;
#pragma unroll
                for (int k = 0; k < NSP; ++k) {
                    const C Dk = (C)P.dk[k];
                    const C G = y1[k] + ctr.Y[k] * l1;
                    const C dG = y2[k] + y1[k] * l1 + ctr.Y[k] * l2;
                    diffY[k] += Dk * (dG + rr * G);
                    Vc += Dk * G;
                    divVc += Dk * dG;
                    H -= (C)P.cpk[k] * Dk * G;
                }
                H += cpc * Vc;
#pragma unroll
                for (int k = 0; k < NSP; ++k) diffY[k] -= Vc * (y1[k] + ctr.Y[k] * rr);
                diffT += t2 + (rr + cp1 * inv_cp) * t1 - H * inv_cp * t1;
            }
            // mass-conserving correction of the convection (Eq. 26)
#pragma unroll
            for (int k = 0; k < NSP; ++k) CY[k] += uh * (cY[k] - ctr.Y[k] * sumc);
        };
#pragma unroll 1
        for (int d = 0; d < D; ++d) {
            const C ud = d == 0 ? u[0] : d == 1 ? u[1] : u[2];
            C d1r;
            if constexpr (TILE) {
                // the points' (or their images') places in the tile
                const int sd = d == 0 ? 1 : kHX;
                const unsigned s20 = (unsigned)(scode >> (20 * d)) & 0xfffffu;
                int li[4] = {ic - 2 * sd, ic - sd, ic + sd, ic + 2 * sd};
                const unsigned kinds = s20 & 0x39ce7u;
                const bool near = kinds != 0;
                if (__any(near)) {
                    const int self[4] = {li[0], li[1], li[2], li[3]};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        // the two bits of the image: self, cell, mirror, same;
                        // beyond an inflow face the point holds the ghost
                        const bool b0 = (s20 >> (5 * j + 3)) & 1u, b1 = (s20 >> (5 * j + 4)) & 1u;
                        const bool inf = ((s20 >> (5 * j)) & 3u) == 3u;
                        const int same = self[j < 2 ? 1 : 2], mirror = self[j < 2 ? 2 : 1];
                        const int lo = b0 ? ic : self[j], hi = b0 ? same : mirror;
                        li[j] = inf ? self[j] : b1 ? hi : lo;
                    }
                }
                C Tv[4], rv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    Tv[j] = tile[li[j]];
                    rv[j] = tile[kNP + li[j]];
                }
                C Yv[CW ? 4 : 1][NSP];  // (image points: values of their own)
                if constexpr (CW) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int k = 0; k < NSP; ++k) Yv[j][k] = tile[(2 + k) * kNP + li[j]];
                }
                if (__any(near)) {
                    if constexpr (CW) {
                        if (P.bimg != nullptr) {
                            int im[4];
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                im[j] = near ? P.bimg[(d * 4 + j) * P.n_boundary + tb] : -1;
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                asm volatile("" ::: "memory");  // (a slot's values at a time: registers)
                                if (__any(im[j] >= 0)) {
                                    Pt<NSP, C> iv;
                                    image_value<NSP>(P, im[j] >= 0 ? im[j] : 0, iv);
                                    Tv[j] = im[j] >= 0 ? iv.T : Tv[j];
                                    rv[j] = im[j] >= 0 ? iv.rho : rv[j];
#pragma unroll
                                    for (int k = 0; k < NSP; ++k) Yv[j][k] = im[j] >= 0 ? iv.Y[k] : Yv[j][k];
                                }
                            }
                        }
                    }
                    const int c = d == 0 ? x : y, n = d == 0 ? P.nx : P.ny, stride = d == 0 ? 1 : P.nx;
                    int off[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) off[j] = (wrap_once(c + slot_offset(j), n) - c) * stride;
                    iso_ghosts<DIAG, C>(
                        P, d, c, n, idx, off, s20, [&](int j) -> C & { return Tv[j]; },
                        [&](int j) -> C & { return rv[j]; },
                        [&](int j, C Tw) -> C {
                            C Yj[NSP];
#pragma unroll
                            for (int k = 0; k < NSP; ++k) {
                                if constexpr (CW)
                                    Yj[k] = Yv[j][k];
                                else
                                    Yj[k] = tile[(2 + k) * kNP + li[j]];
                            }
                            return density<NSP>(P, Tw, Yj);
                        },
                        [&](C Tw) -> double {
                            return 2.0 * P.alpha * (double)density<NSP>(P, Tw, ctr.Y) * ((double)ctr.T - (double)Tw);
                        },
                        wallq);
                }
                d1r = d1(rv[0], rv[1], rho, rv[2], rv[3]);
                axis_terms(
                    [&](int f, int mm) -> C {
                        const int j = mm < 0 ? mm + 2 : mm + 1;
                        if (f == 0) return Tv[j];
                        if constexpr (CW)
                            return Yv[j][f - 2];
                        else
                            return tile[f * kNP + li[j]];
                    },
                    d1r, near, ud);
            } else {
                // 3-D: the four points' T and Y, read once for their densities
                // and kept for the finite differences; behind a wall a point
                // is the ghost formed from its image (Sec. III.B)
                Pt<NSP, C> pv[4];
                bool near = false;
                tile_stencil<NSP, PREC, DIAG, CW>(P, d, x, y, z, idx, tb, bnd, scode, ctr, pv, near, d1r, wallq);
                axis_terms(
                    [&](int f, int m) -> C {
                        const int j = m < 0 ? m + 2 : m + 1;
                        return f == 0 ? pv[j].T : pv[j].Y[f - 2];
                    },
                    d1r, near, ud);
            }
            grad[0] = d == 0 ? d1r : grad[0];
            grad[1] = d == 1 ? d1r : grad[1];
            grad[2] = d == 2 ? d1r : grad[2];
        }
        if constexpr (LE) {
#pragma unroll
            for (int k = 0; k < NSP; ++k) diffY[k] -= ctr.Y[k] * divVc;
        }
        const C alpha = (C)P.alpha;
        diffT *= alpha;
#pragma unroll
        for (int k = 0; k < NSP; ++k) diffY[k] *= alpha;

        auto pop = [&](auto I) -> C {
            if constexpr (STASH)
                return pops[decltype(I)::value * kBlock + threadIdx.x];
            else
                return g[decltype(I)::value];
        };
        if constexpr (STASH) asm volatile("" ::: "memory");
        finish_cell<Q, NSP, PREC, MODE, LE>(P, idx, pop, ctr, u, m, sg, inv_rc, diffT, diffY, CT, CY, grad, wallq, acc);

        if constexpr (D == 3 && mode_advances(MODE)) {
            // 3-D: outlet cells hand their outward normal velocity to
            // outlet_kernel, which applies the same update (keeps the nine
            // extra gathers out of this kernel's registers)
#pragma unroll
            for (int f = 0; f < 2; ++f)
                if (P.face[f] == LBFD_FACE_OUTFLOW && x == (f ? P.nx - 1 : 0))
                    P.outlet_un[(long long)f * P.ny * P.nz + (long long)z * P.ny + y] = (double)(f ? u[0] : -u[0]);
        }
    } else if constexpr (MODE == kModeFields) {
        // solid cells: their stored T and Y, no flow
        if (inbox) {
            if (P.f_rho) P.f_rho[idx] = 0.0;
            if (P.f_u)
#pragma unroll
                for (int d = 0; d < D; ++d) P.f_u[d * P.N + idx] = 0.0;
            if (P.f_Ph) P.f_Ph[idx] = 0.0;
            if (P.f_T) P.f_T[idx] = (double)((const S *)P.sc_in)[idx];
            if (P.f_Y)
#pragma unroll
                for (int k = 0; k < NSP; ++k)
                    P.f_Y[k * P.N + idx] = (double)((const S *)P.sc_in)[(1 + k) * P.N + idx];
        }
    }

    if constexpr (DIAG) block_reduce_diag(acc, P.partials + slot * kNDiag);
}

// Minimum waves per SIMD asked of the register allocator for a step
// kernel (measured on MI355X).  2-D with up to 4 species: three waves
// (168 VGPRs) in FP64 and four (128) in the mixed forms, there also with the
// diagnostics (2048 x 512, half: 70 us free, 64 us at four; one more wave
// than these spills: FP64 64 -> 70 us, half 41 -> 45 us a step).
// 3-D FP64: two waves (256 VGPRs), also with the diagnostics (256 x 256 x 128,
// 4 species: 2476 -> 1664 us with the 27 finiteness tests behind that of their
// sum, which had kept it at one wave; 9 species, spilling 37: 1402 free, 1223).
// 3-D mixed: four waves (128) with up to 4 species, there also for the fields
// (104 -> 99 us; 9 species spill: 117 -> 147), three (168) with more.
// Curved walls and mixture-averaged transport (CW, LE): the 2-D steps with up
// to 4 species, with and without the diagnostics, take the same budgets (at
// most two registers spill; 1024 x 512 burner with links, image points and
// mixture transport, step with the diagnostics, free / budget: FP64 87 / 82 us,
// single 69 / 67, half 70 / 66).  Otherwise the allocator is left free (1): for
// the other launches with diagnostics or fields (MODE != kModeStep), which run
// once per check or read, and for CW and LE in 3-D, with 9 species and in the
// launches that only evaluate a level.  Of those the 2-D FP64 fields launch with
// both once returned wrong velocities at the three-wave budget (spilling) and
// exact ones without it; the assembly check of the build finds no one-sided
// copy in it, so they stay without.  (test_gpu_modes.py runs every
// instantiation of this table against the oracle.)
template <int Q, int NSP, int PREC, int MODE = kModeStep, bool CWLE = false> struct StepWaves {
    static constexpr int value = CWLE ? (Q == 9 && NSP <= 4 && mode_advances(MODE) ? (PREC == LBFD_FP64 ? 3 : 4) : 1)
                                 : (Q == 9 && NSP <= 4 && PREC != LBFD_FP64 && MODE == kModeStepDiag) ? 4
                                 : (Q == 27 && PREC == LBFD_FP64 && MODE == kModeStepDiag) ? 2
                                 : (Q == 27 && NSP <= 4 && PREC != LBFD_FP64 && MODE == kModeFields) ? 4
                                 : MODE != kModeStep                    ? 1
                                 : (Q == 9 && NSP <= 4)                 ? (PREC == LBFD_FP64 ? 3 : 4)
                                 : Q == 27                              ? (PREC == LBFD_FP64 ? 2 : NSP <= 4 ? 4 : 3)
                                                                        : 1;
};

// The step, a tile a block.  Consecutive blocks go to the 8 XCDs in turn, so
// the tiles are renumbered to give each XCD one contiguous band of the box.
template <int Q, int NSP, int PREC, int MODE, bool CW = false, bool LE = false, bool THIN = false>
__global__ void __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(StepWaves<Q, NSP, PREC, MODE, CW || LE>::value))) step_kernel(const KParams P)
{
    using TS = TileShape<Lat<Q>::D, THIN>;
    const long long t = (long long)blockIdx.x;
    const long long n = P.nblocks, q = n >> 3;
    const int xcd = (int)(t & 7), r = (int)(n & 7);
    const long long tile = xcd * q + (xcd < r ? xcd : r) + (t >> 3);
    int bx, by, bz;
    if constexpr (Lat<Q>::D == 3) {
        // bands of tile_band tiles in y, each marched in z, so that the
        // planes a stencil reads again are still in the XCD's L2
        const int per = P.tiles_x * P.tile_band * P.tiles_z;
        const int band = (int)tile / per, in = (int)tile - band * per;
        const int rows = min(P.tile_band, P.tiles_y - band * P.tile_band) * P.tiles_x;
        bz = in / rows;
        const int row = in - bz * rows;
        by = band * P.tile_band + row / P.tiles_x;
        bx = row % P.tiles_x;
    } else {
        bx = (int)(tile % P.tiles_x);
        by = (int)(tile / P.tiles_x);
        bz = 0;
    }
    const int tx = (int)threadIdx.x % TS::X;
    // 3-D: a wave is one row of the tile, its y and z are scalars (THIN: its z)
    const int trow = (int)threadIdx.x / TS::X;
    if constexpr (Lat<Q>::D == 2) {
        step_block<Q, NSP, PREC, MODE, CW, LE, THIN>(P, bx, by, bz, tx, trow, 0, tile);
    } else {
        const int row = THIN ? trow : __builtin_amdgcn_readfirstlane(trow);
        step_block<Q, NSP, PREC, MODE, CW, LE, THIN>(P, bx, by, bz, tx, row % TS::Y,
                                                     THIN ? __builtin_amdgcn_readfirstlane(row / TS::Y) : row / TS::Y,
                                                     tile);
    }
}

// ------------------------------------------------------------ image points
// Shepard reconstruction at the image points of curved-wall ghost nodes
// (Sec. III.B) for the current level: T, rho, Y_k averaged over the listed
// fluid nodes within four cells with the normalised inverse-square-distance
// weights -- a sparse matrix-vector product, one row per image point.  The
// distinct nodes of all rows (the support) are first packed, once each, into
// records of (T, rho, Y_k) (support_kernel), so that a row entry is one
// contiguous record read rather than 1 + N_sp scattered loads and a density
// evaluation.  LPP lanes share a row (chosen at set-up from the mean row
// length), stride over its entries and combine their sums with a butterfly
// inside the group; the result is written before the step launches read it.
template <int NSP, int PREC>
__global__ void __launch_bounds__(kBlock) support_kernel(const KParams P)
{
    using C = typename Prec<PREC>::calc;
    const long long s = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (s >= P.n_sup) return;
    Pt<NSP, C> pt;
    load_point<NSP, PREC>(P, P.sup_idx[s], pt);
    double *rec = P.sup_val + s * (2 + NSP);
    rec[0] = (double)pt.T;
    rec[1] = (double)pt.rho;
#pragma unroll
    for (int k = 0; k < NSP; ++k) rec[2 + k] = (double)pt.Y[k];
}

template <int NSP, int PREC, int LPP>
__global__ void __launch_bounds__(kBlock) image_kernel(const KParams P)
{
    using C = typename Prec<PREC>::calc;
    const long long k = ((long long)blockIdx.x * kBlock + threadIdx.x) / LPP;
    const int lane = (int)threadIdx.x % LPP;
    const bool live = k < P.n_img;  // every lane stays for the butterfly
    const int2 r = live ? P.img_rng[k] : make_int2(0, 0);
    C acc[2 + NSP];
#pragma unroll
    for (int f = 0; f < 2 + NSP; ++f) acc[f] = 0;
#pragma unroll 2
    for (int e = r.x + lane; e < r.x + r.y; e += LPP) {
        const double *rec = P.sup_val + (long long)P.img_idx[e] * (2 + NSP);
        const C w = (C)P.img_w[e];
#pragma unroll
        for (int f = 0; f < 2 + NSP; ++f) acc[f] += w * (C)rec[f];
    }
#pragma unroll
    for (int f = 0; f < 2 + NSP; ++f) {
        C v = acc[f];
#pragma unroll
        for (int o = LPP / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        // (T, Y_k, rho: the order of the scalars' planes)
        const int o = f == 0 ? 0 : f == 1 ? 1 + NSP : f - 1;
        if (live && lane == 0) ((C *)P.img_val)[(size_t)o * P.n_img + k] = v;
    }
}

template <int NSP, int PREC>
hipError_t launch_images(const KParams &kp, hipStream_t s)
{
    support_kernel<NSP, PREC><<<dim3((unsigned)((kp.n_sup + kBlock - 1) / kBlock)), dim3(kBlock), 0, s>>>(kp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int lpp = kp.img_lpp;
    const unsigned nb = (unsigned)((kp.n_img * lpp + kBlock - 1) / kBlock);
    if (lpp == 16)
        image_kernel<NSP, PREC, 16><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
    else if (lpp == 32)
        image_kernel<NSP, PREC, 32><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
    else
        image_kernel<NSP, PREC, 64><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
    return hipGetLastError();
}

// ------------------------------------------------------------ chemistry launch
// Mechanisms of many species (chem_pass): the FP64 Arrhenius source of every
// fluid cell as a launch of its own ahead of the step, one thread per fluid
// cell, written into this step's output scalars (the slots of T and Y_k),
// where the cell's step thread reads it back before overwriting them with
// the cell's new state.  The sub-stepped source then runs at the occupancy
// of its own registers, not of the step's populations and stencils; the
// exponential's table is staged in LDS.  In the mixed forms the stored
// source is rounded to single precision, as the step kernel rounds it when
// it adds it.
//
// A wave takes as long as its lane with the most sub-steps, and the counts
// are bimodal (cold gas 1, burning gas up to the cap), so the cells are
// ordered first (chem_order_kernel): those whose previous source took at
// most kChemLight sub-steps from the front of chem_order, the others from
// the back, runs of the fluid-cell list kept in list order within a wave (31
// sub-steps a lane on a 256 x 128 x 128 front where the cells take 29 and list
// order 50).  The launch starts at the back: the long waves first, so that it
// does not end on a few of them (2001 -> 1925 us; 133 x 97 x 75, single: 505 ->
// 474).
// The previous step's count only decides where a cell goes; every cell's
// source is computed alike wherever it lands, so the results do not depend
// on the order (which the atomics make vary from run to run).
constexpr int kChemChunk = 16;  // fluid-list positions per thread of the ordering

template <int NSP>
__global__ void __launch_bounds__(kBlock) chem_order_kernel(const KParams P)
{
    __shared__ int cnt[2], base[2];
    if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
    __syncthreads();
    const long long n = P.n_fluid;
    const long long t0 = (long long)blockIdx.x * kBlock * kChemChunk;
    const int lane = (int)(threadIdx.x & 63);
    const unsigned long long below = (1ull << lane) - 1ull;
    // this block's light and heavy cells
    int nh = 0, nl = 0;
    for (int r = 0; r < kChemChunk; ++r) {
        const long long t = t0 + (long long)r * kBlock + threadIdx.x;
        if (t < n) {
            const bool h = P.chem_heavy[P.fluid[t]] != 0;
            nh += h;
            nl += !h;
        }
    }
    atomicAdd(&cnt[0], nl);
    atomicAdd(&cnt[1], nh);
    __syncthreads();
    if (threadIdx.x == 0) {
        base[0] = atomicAdd(&P.chem_count[0], cnt[0]);
        base[1] = atomicAdd(&P.chem_count[1], cnt[1]);
        cnt[0] = cnt[1] = 0;
    }
    __syncthreads();
    // places: per round and wave one run per class, in list order
    for (int r = 0; r < kChemChunk; ++r) {
        const long long t = t0 + (long long)r * kBlock + threadIdx.x;
        const bool valid = t < n;
        const int idx = valid ? P.fluid[t] : 0;
        const bool h = valid && P.chem_heavy[idx] != 0;
        const bool l = valid && !h;
        const unsigned long long bh = __ballot(h), bl = __ballot(l);
        int wh = 0, wl = 0;
        if (lane == 0) {
            wh = atomicAdd(&cnt[1], __popcll(bh));
            wl = atomicAdd(&cnt[0], __popcll(bl));
        }
        wh = __shfl(wh, 0, 64);
        wl = __shfl(wl, 0, 64);
        // (the counts of both passes agree, so every place is in [0, n))
        const long long ph = n - 1 - (base[1] + wh + __popcll(bh & below));
        const long long pl = base[0] + wl + __popcll(bl & below);
        if (h && ph >= 0) P.chem_order[ph] = idx;
        if (l && pl < n) P.chem_order[pl] = idx;
    }
}

// The ordering's two counters, cleared ahead of it (a kernel, so that a
// captured step records no memset node).
template <int NSP>
__global__ void chem_count_clear_kernel(int *count)
{
    if (threadIdx.x < 2) count[threadIdx.x] = 0;
}

template <int NSP, int PREC, bool LE, int NR>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) chem_kernel(const KParams P)
{
    using S = typename Prec<PREC>::scal;
    __shared__ double tab[kExpTabN], ltab[2 * kLogTabN];
    for (int i = (int)threadIdx.x; i < kExpTabN; i += (int)blockDim.x) tab[i] = kExp2Tab[i];
    for (int i = (int)threadIdx.x; i < 2 * kLogTabN; i += (int)blockDim.x) ltab[i] = kLogTab[i];
    __syncthreads();
    const long long t = P.n_fluid - 1 - ((long long)blockIdx.x * kBlock + threadIdx.x);
    if (t < 0) return;
    const long long idx = P.chem_order[t];
    const char *si = (const char *)P.sc_in;
    char *so = (char *)P.sc_out;
    const size_t fstride = (size_t)P.N * sizeof(S);
    const uint32_t off = (uint32_t)idx * (uint32_t)sizeof(S);
    double Y[NSP], srcT, srcY[NSP];
    const double T = (double)ldo<S>(si, off);
#pragma unroll
    for (int k = 0; k < NSP; ++k) Y[k] = (double)ldo<S>(si + (size_t)(1 + k) * fstride, off);
    const int nsub = chemistry<NSP, LE, NR>(P, tab, ltab, T, Y, srcT, srcY);
    P.chem_heavy[idx] = nsub > kChemLight;
    sto<S>(so, off, (S)srcT);
#pragma unroll
    for (int k = 0; k < NSP; ++k) sto<S>(so + (size_t)(1 + k) * fstride, off, (S)srcY[k]);
}

template <int NSP, int PREC>
hipError_t launch_chem(const KParams &kp, hipStream_t s)
{
    const unsigned nb = (unsigned)((kp.n_fluid + kBlock - 1) / kBlock);
    if (nb == 0) return hipSuccess;
    const long long per = (long long)kBlock * kChemChunk;
    chem_count_clear_kernel<NSP><<<dim3(1), dim3(64), 0, s>>>(kp.chem_count);
    chem_order_kernel<NSP><<<dim3((unsigned)((kp.n_fluid + per - 1) / per)), dim3(kBlock), 0, s>>>(kp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the kernel specialised to the mechanism's structure when one was
    // compiled for this context (unity-Lewis transport)
    if (kp.chem_jit != nullptr && kp.transport != LBFD_MIXTURE_AVERAGED)
        return launch_chem_jit(kp, nb, sizeof(typename Prec<PREC>::scal), s);
    // mechanisms of at most two reactants per reaction skip the two
    // constant-1 slots
    const bool two = kp.chem_nreact <= 2;
    if (kp.transport == LBFD_MIXTURE_AVERAGED) {
        if (two)
            chem_kernel<NSP, PREC, true, 2><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
        else
            chem_kernel<NSP, PREC, true, 4><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
    } else {
        if (two)
            chem_kernel<NSP, PREC, false, 2><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
        else
            chem_kernel<NSP, PREC, false, 4><<<dim3(nb), dim3(kBlock), 0, s>>>(kp);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------ outlet
// Outlet (Eq. 32): for every fluid cell of an outflow face whose inner
// neighbour is fluid, the populations entering through the face become
// g_i(r) <- g_i(r-n)(cs - u.n) + g_i(r)(1 - cs + u.n), with the
// post-streaming values g_i(r) (the outlet buffer, read by this step) and
// g_i(r-n) (pulled again from the buffer this step read), and u.n of this
// level (written by the step).  Runs after it; used for D3Q27 (D2Q9 applies
// the update in the step).
// A thread per face cell; it is bound by the latency of its loads, so both
// cells' sources come from their pull codes -- the face cell's name the
// populations the outlet sets, the inner cell's where its own are pulled from
// -- and the nine gathers are in flight together.  (With the sources
// classified anew, which copied the launch parameters to scratch memory, 50 us
// on a 256 x 128 face and 36 us on 99 x 83; now 17 and 10 us.)
template <int Q, int PREC>
__global__ void __launch_bounds__(kBlock) outlet_kernel(const KParams P)
{
    using L = Lat<Q>;
    using C = typename Prec<PREC>::calc;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nf = (long long)P.ny * P.nz;
    if (t >= 2 * nf) return;
    const int f = (int)(t / nf);
    const int y = (int)((t % nf) % P.ny), z = (int)((t % nf) / P.ny);
    if ((f ? P.face[1] : P.face[0]) != LBFD_FACE_OUTFLOW) return;
    const int x = f ? P.nx - 1 : 0, sign = f ? 1 : -1;
    const long long idx = ((long long)z * P.ny + y) * P.nx + x;
    if (P.code[idx] != kCodeBoundary) return;  // (a fluid cell next to this face is a boundary cell)
    const unsigned long long pc = P.cell_code[idx].x;
    if (!pulls_outlet(pc)) return;  // (else the inner neighbour is fluid)
    const long long in = idx - sign;
    const unsigned long long pci = P.code[in] == kCodeBoundary ? P.cell_code[in].x : 0;
    const C cs = (C)0.57735026918962576451;
    const C un = (C)P.outlet_un[t];
    C G[Q];
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (L::cx(i) != 0) {
            if (L::cx(i) == -sign) {
                // the inner cell's source: a neighbour inside the box along x
                const int kind = decode_pull_kind(pci, i);
                const uint32_t src = (uint32_t)cell_at(x, y, z, 0, -L::cy(i), -L::cz(i), P.nx, P.ny, P.nz);
                const bool fluid = kind == kPullFluid;
                G[i] = pop_load_pair<Q, PREC, i>(P.pop_in, P.N, !fluid, fluid ? src : (uint32_t)in);
                if (kind == kPullInflow)
                    G[i] += (C)(2.0 * L::w(i) * P.rho_in *
                                (L::cx(i) * P.u_in[0] + L::cy(i) * P.u_in[1] + L::cz(i) * P.u_in[2]));
            }
        }
    });
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (L::cx(i) != 0) {
            if (L::cx(i) == -sign && decode_pull_kind(pc, i) == kPullOutlet) {
                double &S = P.outlet[outlet_index(P, f, i, Q, y, z)];
                S = (double)(G[i] * (cs - un) + (C)S * ((C)1 - cs + un));
            }
        }
    });
}

// ------------------------------------------------------------ init kernel
// g^0 = w (P_h0 - rho cs^2) + cs^2 f^eq(rho, u0) (Eq. 12), scattered into
// the post-collision buffer so that the first gather returns it (inverse
// of the pull, the inlet and the bounce-back rules); populations entering
// through an outlet are written to the outlet buffer.
template <int Q, int NSP, int PREC>
__global__ void __launch_bounds__(kBlock) init_kernel(const KParams P, const double *u0, const double *Ph0)
{
    using L = Lat<Q>;
    using S = typename Prec<PREC>::scal;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z = blockIdx.z * blockDim.z + threadIdx.z;
    if (x >= P.nx || y >= P.ny || z >= P.nz) return;
    const long long idx = ((long long)z * P.ny + y) * P.nx + x;
    if (P.mask[idx] != LBFD_FLUID) return;
    const S *sc = (const S *)P.sc_in;
    double T = (double)sc[idx], Y[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) Y[k] = (double)sc[(1 + k) * P.N + idx];
    const double rho = density<NSP>(P, T, Y);
    double u[3] = {0.0, 0.0, 0.0};
    if (u0)
        for (int d = 0; d < L::D; ++d) u[d] = u0[d * P.N + idx];
    const double ph = Ph0 ? Ph0[idx] : 0.0;
    const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int opp = Q - 1 - i;
        const double cu = L::cx(i) * u[0] + L::cy(i) * u[1] + L::cz(i) * u[2];
        const double feq = L::w(i) * rho * (1.0 + cu / kCs2 + cu * cu / (2.0 * kCs2 * kCs2) - uu / (2.0 * kCs2));
        const double g0 = L::w(i) * (ph - rho * kCs2) + kCs2 * feq;
        using C = typename Prec<PREC>::calc;
        if constexpr (i == (Q - 1) / 2) {
            pop_store<Q, PREC, i>(P.pop_out, P.N, idx, (C)g0);
        } else {
            Nb s = classify(P, x - L::cx(i), y - L::cy(i), z - L::cz(i));
            if (s.kind == kFluid) {
                pop_store<Q, PREC, i>(P.pop_out, P.N, s.idx, (C)g0);
            } else if (s.kind == kInflow) {
                const double ci = inflow_cu<Q, i>(P, x, y, z);
                pop_store<Q, PREC, opp>(P.pop_out, P.N, idx, (C)(g0 - 2.0 * L::w(i) * P.rho_in * ci));
            } else if (s.kind == kOutflow) {
                const int sign = (s.face & 1) ? 1 : -1;
                Nb in = classify(P, x - sign, y, z);
                if (in.kind == kFluid)
                    P.outlet[outlet_index(P, s.face, i, Q, y, z)] = g0;
                else
                    pop_store<Q, PREC, opp>(P.pop_out, P.N, idx, (C)g0);
            } else {
                pop_store<Q, PREC, opp>(P.pop_out, P.N, idx, (C)g0);
            }
        }
    });
}

// ------------------------------------------------------------ launchers
// Instantiated once per configuration in inst/*.hip (explicit
// instantiation), declared extern in the dispatcher.
// One step: the tiles in one launch on the context stream, then for D3Q27
// the outlet update.
template <int Q, int NSP, int PREC, int MODE, bool LE>
hipError_t launch_tiles_t(const KParams &kp, hipStream_t s)
{
    // boundary cells with curved-wall links or image points
    const dim3 grid((unsigned)kp.nblocks), block(kBlock);
    if (kp.bq != nullptr || kp.bimg != nullptr)
        step_kernel<Q, NSP, PREC, MODE, true, LE><<<grid, block, 0, s>>>(kp);
    else if (kp.thin)
        step_kernel<Q, NSP, PREC, MODE, false, LE, true><<<grid, block, 0, s>>>(kp);
    else
        step_kernel<Q, NSP, PREC, MODE, false, LE><<<grid, block, 0, s>>>(kp);
    return hipGetLastError();
}

template <int Q, int NSP, int PREC, int MODE>
hipError_t launch_parts(const KParams &kp, const Streams &st)
{
    // st.part 0: every launch; 1: the tiles (and the image points they read);
    // 2: the outlet; 3: the chemistry launch only
    hipError_t e = hipSuccess;
    if constexpr (chem_pass(NSP)) {
        if ((st.part == 0 || st.part == 3) && (e = launch_chem<NSP, PREC>(kp, st.main)) != hipSuccess)
            return e;
    }
    if (st.part == 3) return hipSuccess;
    if (st.part != 2) {
        if (kp.bimg != nullptr && kp.n_img > 0)
            if ((e = launch_images<NSP, PREC>(kp, st.main)) != hipSuccess) return e;
        // the mixture-averaged transport is a separate instantiation, so that
        // unity-Lewis steps keep their registers
        e = kp.transport == LBFD_MIXTURE_AVERAGED ? launch_tiles_t<Q, NSP, PREC, MODE, true>(kp, st.main)
                                                  : launch_tiles_t<Q, NSP, PREC, MODE, false>(kp, st.main);
        if (e != hipSuccess) return e;
    }
    if constexpr (Lat<Q>::D == 3 && mode_advances(MODE)) {
        if (st.part != 1 && kp.n_boundary > 0 &&
            (kp.face[0] == LBFD_FACE_OUTFLOW || kp.face[1] == LBFD_FACE_OUTFLOW)) {
            // small blocks: the launch is one round of loads on few threads
            const unsigned no = (unsigned)((2LL * kp.ny * kp.nz + 63) / 64);
            outlet_kernel<Q, PREC><<<dim3(no), dim3(64), 0, st.main>>>(kp);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

template <int Q, int NSP, int PREC>
hipError_t launch_step_t(int mode, const KParams &kp, const Streams &st)
{
    switch (mode) {
    case kModeStep: return launch_parts<Q, NSP, PREC, kModeStep>(kp, st);
    case kModeStepDiag: return launch_parts<Q, NSP, PREC, kModeStepDiag>(kp, st);
    case kModeDiag: return launch_parts<Q, NSP, PREC, kModeDiag>(kp, st);
    default: return launch_parts<Q, NSP, PREC, kModeFields>(kp, st);
    }
}

template <int Q, int NSP, int PREC>
hipError_t launch_init_t(const KParams &kp, const double *u0, const double *Ph0, dim3 grid, dim3 block,
                         hipStream_t s)
{
    init_kernel<Q, NSP, PREC><<<grid, block, 0, s>>>(kp, u0, Ph0);
    return hipGetLastError();
}

// (lattice, species, precision) combinations built into the library
#define LBFD_FOR_CONFIGS(X) \
    X(9, 2, 0) X(9, 4, 0) X(9, 9, 0) X(27, 2, 0) X(27, 4, 0) X(27, 9, 0) \
    X(9, 2, 1) X(9, 4, 1) X(9, 9, 1) X(27, 2, 1) X(27, 4, 1) X(27, 9, 1) \
    X(9, 4, 2) X(27, 4, 2) X(27, 9, 2)

#define LBFD_INSTANTIATE(q, n, p) \
    template hipError_t launch_step_t<q, n, p>(int, const KParams &, const Streams &); \
    template hipError_t launch_init_t<q, n, p>(const KParams &, const double *, const double *, dim3, dim3, \
                                               hipStream_t);

}  // namespace lbfd
