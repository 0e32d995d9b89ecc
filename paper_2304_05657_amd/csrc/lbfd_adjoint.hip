// lbfd_adjoint.hip -- derivatives of the FP64 coupled step.
//
// The objective is J = sum_{n = 0}^{N-1} w_n q(s^n), w_n = 1 inside the
// chosen window of levels, with q either the wall heat flux (the sum over
// fluid cells and axis sides whose first neighbour is an isothermal wall of
// 2 alpha rho(T_w, Y)(T - T_w)) or the flame position
// nx - sum_cells (T - T_u)/(T_b - T_u) nx / n_fluid, and the state
// s^n = (post-collision populations read by step n, T^n, Y^n).
// With s^{n+1} = F(s^n; theta), theta = (wall temperatures, A_j, Ta_j), the
// adjoint recursion is lambda^N = 0,
//   lambda^n = (dF/ds^n)^T lambda^{n+1} + (dq/ds^n)^T,
//   dJ/dtheta = sum_n (dF/dtheta)^T lambda^{n+1} + dq^n/dtheta.
// One thread per fluid cell c gathers the cell's inputs (pull sources, the
// finite-difference stencil's scalars, ghost wall temperatures; at interior
// cells plain offsets, elsewhere from the cell's codes) and runs the cell's
// update forward in FP64, then backward: the reverse of every operation,
// hand-derived, from the adjoint of the cell's outputs to those of its inputs,
// in two kernels (cell_vjp_collision, cell_vjp_stencil).  The Arrhenius source
// is reversed sub-step by sub-step, each sub-step's state recomputed from the
// cell's (chem_vjp): a single step in the first of the two, sub-steps in a
// kernel between them (cell_vjp_chem).
// Each pulled population is read by exactly one cell, so its adjoint is
// stored; each stencil slot's share of a scalar's adjoint is stored per slot
// and gathered by the slot's cell in a last kernel; the wall temperatures'
// adjoints are added atomically.  Steps are recomputed from checkpoints taken
// every K steps (host side, lbfd_api.hip).
//
// tangent_kernel evaluates the same update in dual numbers with a given
// tangent of every input (the Jacobian-vector product of one step); the
// identity <J dx, lambda> = <dx, J^T lambda> between the two checks the
// reverse sweep.  Both evaluate the forward step's formulas in the general
// geometry path; rate coefficients are formed as in the step's chemistry
// (A dt exp(b ln T - Ta/T) with the step's exponential).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbfd_kernels.h"

namespace lbfd {

// ----------------------------------------------------------- dual numbers
// Value and N tangents.
template <int N>
struct DualN {
    double v;
    double d[N];
    __device__ DualN() : v(0.0)
    {
        for (int i = 0; i < N; ++i) d[i] = 0.0;
    }
    __device__ DualN(double x) : v(x)
    {
        for (int i = 0; i < N; ++i) d[i] = 0.0;
    }
    __device__ explicit operator double() const { return v; }
    __device__ DualN &operator+=(const DualN &b)
    {
        v += b.v;
        for (int i = 0; i < N; ++i) d[i] += b.d[i];
        return *this;
    }
    __device__ DualN &operator-=(const DualN &b)
    {
        v -= b.v;
        for (int i = 0; i < N; ++i) d[i] -= b.d[i];
        return *this;
    }
    __device__ DualN &operator*=(const DualN &b)
    {
        for (int i = 0; i < N; ++i) d[i] = d[i] * b.v + v * b.d[i];
        v *= b.v;
        return *this;
    }
};
using Dual = DualN<1>;

template <int N> __device__ inline DualN<N> operator+(DualN<N> a, const DualN<N> &b) { return a += b; }
template <int N> __device__ inline DualN<N> operator-(DualN<N> a, const DualN<N> &b) { return a -= b; }
template <int N> __device__ inline DualN<N> operator*(DualN<N> a, const DualN<N> &b) { return a *= b; }
template <int N> __device__ inline DualN<N> operator-(const DualN<N> &a)
{
    DualN<N> r(-a.v);
    for (int i = 0; i < N; ++i) r.d[i] = -a.d[i];
    return r;
}
// (divisions, not a reciprocal: with b.v subnormal, 1 / b.v overflows and a
// zero numerator would give 0 * inf)
template <int N> __device__ inline DualN<N> operator/(const DualN<N> &a, const DualN<N> &b)
{
    const double q = a.v / b.v;
    DualN<N> r(q);
    for (int i = 0; i < N; ++i) r.d[i] = (a.d[i] - q * b.d[i]) / b.v;
    return r;
}
// f(a) with f(a.v) = fv and f'(a.v) = fd
template <int N> __device__ inline DualN<N> chain(const DualN<N> &a, double fv, double fd)
{
    DualN<N> r(fv);
    for (int i = 0; i < N; ++i) r.d[i] = fd * a.d[i];
    return r;
}
template <int N> __device__ inline DualN<N> rcp(const DualN<N> &a)
{
    const double r = rcp(a.v);
    return chain(a, r, -r * r);
}
template <int N> __device__ inline bool operator<(const DualN<N> &a, const DualN<N> &b) { return a.v < b.v; }
template <int N> __device__ inline bool operator>(const DualN<N> &a, const DualN<N> &b) { return a.v > b.v; }
template <int N> __device__ inline bool operator>=(const DualN<N> &a, const DualN<N> &b) { return a.v >= b.v; }
template <int N> __device__ inline bool operator<=(const DualN<N> &a, const DualN<N> &b) { return a.v <= b.v; }
// the exponential of the forward chemistry (exp_tab; tab: its table, in
// LDS or constant memory)
template <int N> __device__ inline DualN<N> dexp(const DualN<N> &a, const double *tab)
{
    const double e = exp_tab(a.v, tab);
    return chain(a, e, e);
}
__device__ inline double dexp(double a, const double *tab) { return exp_tab(a, tab); }
template <int N> __device__ inline DualN<N> dlog(const DualN<N> &a) { return chain(a, log(a.v), rcp(a.v)); }
__device__ inline double dlog(double a) { return log(a); }
template <int N> __device__ inline double val(const DualN<N> &a) { return a.v; }
__device__ inline double val(double a) { return a; }

// ------------------------------------------------------------ cell inputs
// Stencil slots: 0 = the cell, 1 + 4 d + j for axis d < D and
// m = -2, -1, 1, 2 (j = 0 .. 3).
template <int Q> constexpr int n_slots() { return 1 + 4 * Lat<Q>::D; }

// A ghost's image is a fluid slot: the cell for a first neighbour; the
// cell or one of the axis's two first neighbours (slots img_lo, img_hi) for
// a second neighbour.
constexpr bool second_nb(int s) { return s > 0 && ((s - 1) % 4 == 0 || (s - 1) % 4 == 3); }
constexpr int img_lo(int s) { return second_nb(s) ? s - (s - 1) % 4 + 1 : 0; }
constexpr int img_hi(int s) { return second_nb(s) ? s - (s - 1) % 4 + 2 : 0; }

template <int Q, int NSP>
struct CellIn {
    static constexpr int S = n_slots<Q>();
    double g[Q];          // pulled populations (with the inlet correction)
    int tdir[Q], tcell[Q];  // population entry each pull read
    int cell[S];          // fluid slot: its cell; ghost slot: -1
    int kind[S];          // kFluid or the kind of the wall behind the ghost
    int img[S];           // ghost slot: slot of its image point
    double Tw[S];         // ghost slot: wall temperature
    int wall[S];          // ghost slot behind an isothermal in-box solid: its cell, else -1
};

// (the tangent's; the reverse sweep reads the cell's codes instead)
template <int Q, int NSP>
__device__ void gather_inputs(const KParams &P, int x, int y, int z, long long idx, CellIn<Q, NSP> &in)
{
    using L = Lat<Q>;
    constexpr int D = L::D;
    const double *pop = (const double *)P.pop_in;
    if (P.code[idx] == kCodeInterior) {
        // every pull source and stencil point is an in-box fluid cell
        const long long st[3] = {1, P.nx, (long long)P.nx * P.ny};
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            in.tdir[i] = i;
            in.tcell[i] = (int)(idx - (L::cx(i) * st[0] + L::cy(i) * st[1] + L::cz(i) * st[2]));
            in.g[i] = pop[(long long)i * P.N + in.tcell[i]];
        }
#pragma unroll
        for (int s = 0; s < n_slots<Q>(); ++s) {
            const int d = s == 0 ? 0 : (s - 1) / 4, j = s == 0 ? 0 : (s - 1) % 4;
            const int mm = j == 0 ? -2 : j == 1 ? -1 : j == 2 ? 1 : 2;
            in.cell[s] = (int)(s == 0 ? idx : idx + mm * st[d]);
            in.kind[s] = kFluid;
            in.img[s] = -1;
            in.Tw[s] = 0.0;
            in.wall[s] = -1;
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int cx = i % 3 - 1, cy = (i / 3) % 3 - 1, cz = Q == 9 ? 0 : i / 9 - 1;
        const int opp = Q - 1 - i;
        double corr = 0.0;
        if (cx == 0 && cy == 0 && cz == 0) {
            in.tdir[i] = i;
            in.tcell[i] = (int)idx;
        } else {
            const Nb s = classify(P, x - cx, y - cy, z - cz);
            const bool fl = s.kind == kFluid;
            in.tdir[i] = fl ? i : opp;
            in.tcell[i] = fl ? (int)s.idx : (int)idx;
            if (s.kind == kInflow) corr = 2.0 * L::w(i) * P.rho_in * inflow_cu_c(P, cx, cy, cz, x, y, z);
        }
        in.g[i] = pop[(long long)in.tdir[i] * P.N + in.tcell[i]] + corr;
    }
    auto load = [&](int s, long long c) {
        in.cell[s] = (int)c;
        in.kind[s] = kFluid;
        in.img[s] = -1;
        in.Tw[s] = 0.0;
        in.wall[s] = -1;
    };
    auto ghost_slot = [&](int s, const Nb &w, int image) {
        in.cell[s] = -1;
        in.kind[s] = w.kind;
        in.img[s] = image;
        in.Tw[s] = w.Tw;
        in.wall[s] = (w.kind == kIso && w.face < 0) ? (int)w.idx : -1;
    };
    load(0, idx);
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
        for (int sg = -1; sg <= 1; sg += 2) {
            const int j1 = sg < 0 ? 1 : 2, j2 = sg < 0 ? 0 : 3;
            const int s1 = 1 + 4 * d + j1, s2 = 1 + 4 * d + j2, sm = 1 + 4 * d + (sg < 0 ? 2 : 1);
            const int ox = d == 0, oy = d == 1, oz = d == 2;
            const Nb c1 = classify(P, x + sg * ox, y + sg * oy, z + sg * oz);
            if (c1.kind != kFluid) {
                const Nb cm = classify(P, x - sg * ox, y - sg * oy, z - sg * oz);
                ghost_slot(s1, c1, 0);
                ghost_slot(s2, c1, cm.kind == kFluid ? sm : 0);
            } else {
                load(s1, c1.idx);
                const Nb c2 = classify(P, x + 2 * sg * ox, y + 2 * sg * oy, z + 2 * sg * oz);
                if (c2.kind != kFluid)
                    ghost_slot(s2, c2, s1);
                else
                    load(s2, c2.idx);
            }
        }
    }
}

// T and Y of the fluid slots (read from the state; 0 at ghost slots).
template <int Q, int NSP>
__device__ __forceinline__ void slot_scalars(const KParams &P, const CellIn<Q, NSP> &in, double (&T)[n_slots<Q>()],
                                             double (&Y)[n_slots<Q>()][NSP])
{
    const double *sc = (const double *)P.sc_in;
#pragma unroll
    for (int s = 0; s < n_slots<Q>(); ++s) {
        const bool fl = in.kind[s] == kFluid;
        const long long c = fl ? in.cell[s] : in.cell[0];
        T[s] = fl ? sc[c] : 0.0;
#pragma unroll
        for (int k = 0; k < NSP; ++k) Y[s][k] = fl ? sc[(1 + k) * P.N + c] : 0.0;
    }
}

// Input slot numbering of the tangent: [0, Q) pulls; then S x (1 + NSP)
// stencil scalars (T, Y_k); then S ghost wall temperatures; then
// (A_j, Ta_j) per reaction.
template <int Q, int NSP>
struct Slots {
    static constexpr int S = n_slots<Q>();
    static constexpr int pull = 0;
    static constexpr int scal = Q;
    static constexpr int wall = Q + S * (1 + NSP);
    static constexpr int param = wall + S;
};

template <int NSP, class A>
__device__ A density_a(const KParams &P, A T, const A (&Y)[NSP])
{
    A s = 0.0;
    for (int k = 0; k < NSP; ++k) s += Y[k] * A(P.invW[k]);
    return A(P.T_ref_over_W_ref) / (T * s);
}

// Arrhenius source of one cell over the step in the number type A (the
// forward chemistry's sub-stepping, rate coefficients and limiter): from
// the cell's T0, Y0 and the reactions' (A_j, Ta_j) = par(j) to (srcT, srcY).
// The sub-step count and the limiter's choice follow the values.
template <int NSP, class A, class Par>
__device__ void chem_source(const KParams &P, const double *tab, const A &T0, const A (&Y0)[NSP], Par par, A &srcT,
                            A (&srcY)[NSP])
{
    const bool anyb = P.chem_anyb != 0;
    int nsub = 1;
    if (P.chem_substeps_max > 1) {
        const double lnT = anyb ? log(val(T0)) : 0.0, invT = rcp(val(T0));
        double kmax = 0.0;
        for (int j = 0; j < P.n_rx; ++j) kmax = fmax(kmax, rate_coeff_l(P.rxk[j], lnT, invT, tab));
        const double want = ceil(kmax / 0.1);
        nsub = want < 1.0 ? 1 : want > (double)P.chem_substeps_max ? P.chem_substeps_max : (int)want;
    }
    const double inv_nsub = nsub == 1 ? 1.0 : rcp((double)nsub);
    A dT = 0.0, dY[NSP];
    for (int k = 0; k < NSP; ++k) dY[k] = 0.0;
    for (int s = 0; s < nsub; ++s) {
        const A Tc = T0 + dT;
        A Yc[NSP], incT = 0.0, incY[NSP];
        for (int k = 0; k < NSP; ++k) {
            Yc[k] = Y0[k] + dY[k];
            incY[k] = 0.0;
        }
        const A lnTc = anyb ? dlog(Tc) : A(0.0), invTc = rcp(Tc);
        for (int j = 0; j < P.n_rx; ++j) {
            const lbfd_reaction &r = P.rx[j];
            A Aj, Taj;
            par(j, Aj, Taj);
            A rr = Aj * A(P.dt_phys) * dexp(A(r.b) * lnTc - Taj * invTc, tab) * A(inv_nsub);
            // four reactant factors, Y of the reactant or 1 (react[m] = NSP)
#pragma unroll
            for (int mm = 0; mm < 4; ++mm) {
                const int sp = P.rxk[j].react[mm];
                A f = 1.0;
#pragma unroll
                for (int k = 0; k < NSP; ++k) f = sp == k ? Yc[k] : f;
                rr *= f;
            }
            for (int k = 0; k < NSP; ++k) incY[k] += A(r.nu_mass[k]) * rr;
            incT += A(r.q_over_cp) * rr;
        }
        // positivity limiter (value-based choice, differentiable scale)
        A lam = 1.0;
        for (int k = 0; k < NSP; ++k)
            if (val(incY[k]) < 0.0 && val(Yc[k] + incY[k]) < 0.0) {
                const A l = (val(Yc[k]) > 0.0 ? Yc[k] : A(0.0)) / (-incY[k]);
                if (val(l) < val(lam)) lam = l;
            }
        dT += lam * incT;
        for (int k = 0; k < NSP; ++k) dY[k] += lam * incY[k];
    }
    srcT = dT;
    for (int k = 0; k < NSP; ++k) srcY[k] = dY[k];
}

// One sub-step of chem_source in FP64 from the state (Tc, Yc): the
// increments, the limiter's scale lam and the species that set it (kstar,
// -1 when lam = 1), with the same arithmetic as chem_source.
template <int NSP>
__device__ __forceinline__ void chem_substep(const KParams &P, const double *tab, bool anyb, double inv_nsub,
                                             double Tc, const double (&Yc)[NSP], double &incT, double (&incY)[NSP],
                                             double &lam, int &kstar)
{
    const double lnTc = anyb ? log(Tc) : 0.0, invTc = rcp(Tc);
    incT = 0.0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) incY[k] = 0.0;
    for (int j = 0; j < P.n_rx; ++j) {
        const lbfd_reaction &r = P.rx[j];
        double rr = r.A * P.dt_phys * dexp(r.b * lnTc - r.Ta * invTc, tab) * inv_nsub;
#pragma unroll
        for (int mm = 0; mm < 4; ++mm) {
            const int sp = P.rxk[j].react[mm];
            double f = 1.0;
#pragma unroll
            for (int k = 0; k < NSP; ++k) f = sp == k ? Yc[k] : f;
            rr *= f;
        }
#pragma unroll
        for (int k = 0; k < NSP; ++k) incY[k] += r.nu_mass[k] * rr;
        incT += r.q_over_cp * rr;
    }
    lam = 1.0;
    kstar = -1;
#pragma unroll
    for (int k = 0; k < NSP; ++k)
        if (incY[k] < 0.0 && Yc[k] + incY[k] < 0.0) {
            const double l = (Yc[k] > 0.0 ? Yc[k] : 0.0) / (-incY[k]);
            if (l < lam) {
                lam = l;
                kstar = k;
            }
        }
}

// Reverse of chem_source (FP64): given ls, the adjoint of (srcT, srcY),
// adds ls^T d src / d (T0, Y0) to aT0, aY0 and ls^T d src / d (A_j, Ta_j) to
// the thread's copies of lam_param[2 j], lam_param[2 j + 1] (LDS).  The sub-steps are reversed
// from the last; the state of each is recomputed from (T0, Y0), so the cost
// grows with the square of the sub-step count (one sub-step: one forward
// and one reverse evaluation).
constexpr int kParamCopies = 16;
template <int NSP>
__device__ void chem_vjp(const KParams &P, const double *tab, double T0, const double (&Y0)[NSP],
                         const double (&ls)[1 + NSP], double &aT0, double (&aY0)[NSP], double *lam_param)
{
    const bool anyb = P.chem_anyb != 0;
    int nsub = 1;
    if (P.chem_substeps_max > 1) {
        const double lnT = anyb ? log(T0) : 0.0, invT = rcp(T0);
        double kmax = 0.0;
        for (int j = 0; j < P.n_rx; ++j) kmax = fmax(kmax, rate_coeff_l(P.rxk[j], lnT, invT, tab));
        const double want = ceil(kmax / 0.1);
        nsub = want < 1.0 ? 1 : want > (double)P.chem_substeps_max ? P.chem_substeps_max : (int)want;
    }
    const double inv_nsub = nsub == 1 ? 1.0 : rcp((double)nsub);
    // adjoint of the accumulated increments (dT, dY) after sub-step s
    double LdT = ls[0], LdY[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) LdY[k] = ls[1 + k];
    for (int s = nsub - 1; s >= 0; --s) {
        double dT = 0.0, dY[NSP];
#pragma unroll
        for (int k = 0; k < NSP; ++k) dY[k] = 0.0;
        double Yc[NSP], incT, incY[NSP], lam;
        int kstar;
        for (int t = 0; t < s; ++t) {
#pragma unroll
            for (int k = 0; k < NSP; ++k) Yc[k] = Y0[k] + dY[k];
            chem_substep<NSP>(P, tab, anyb, inv_nsub, T0 + dT, Yc, incT, incY, lam, kstar);
            dT += lam * incT;
#pragma unroll
            for (int k = 0; k < NSP; ++k) dY[k] += lam * incY[k];
        }
        const double Tc = T0 + dT;
#pragma unroll
        for (int k = 0; k < NSP; ++k) Yc[k] = Y0[k] + dY[k];
        chem_substep<NSP>(P, tab, anyb, inv_nsub, Tc, Yc, incT, incY, lam, kstar);
        // (dT, dY) += lam (incT, incY)
        double llam = LdT * incT, lincY[NSP], lYc[NSP];
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            llam += LdY[k] * incY[k];
            lincY[k] = lam * LdY[k];
            lYc[k] = 0.0;
        }
        const double lincT = lam * LdT;
        // lam = Yc_k / (-incY_k) for the limiting species k (0 if Yc_k <= 0)
#pragma unroll
        for (int k = 0; k < NSP; ++k)
            if (k == kstar && Yc[k] > 0.0) {
                lYc[k] += llam / (-incY[k]);
                lincY[k] += llam * Yc[k] / (incY[k] * incY[k]);
            }
        // the rates rr_j = A_j dt exp(b_j ln Tc - Ta_j / Tc) / nsub prod_m F_jm
        const double lnTc = anyb ? log(Tc) : 0.0, invTc = rcp(Tc);
        double lTc = 0.0;
        for (int j = 0; j < P.n_rx; ++j) {
            const lbfd_reaction &r = P.rx[j];
            const double e = dexp(r.b * lnTc - r.Ta * invTc, tab);
            const double base = r.A * P.dt_phys * e * inv_nsub;
            double F[4];
            int sp[4];
#pragma unroll
            for (int mm = 0; mm < 4; ++mm) {
                sp[mm] = P.rxk[j].react[mm];
                double f = 1.0;
#pragma unroll
                for (int k = 0; k < NSP; ++k) f = sp[mm] == k ? Yc[k] : f;
                F[mm] = f;
            }
            const double pr = F[0] * F[1] * F[2] * F[3];
            const double rr = base * pr;
            double lrr = r.q_over_cp * lincT;
#pragma unroll
            for (int k = 0; k < NSP; ++k) lrr += r.nu_mass[k] * lincY[k];
            lTc += lrr * rr * (r.b * invTc + r.Ta * invTc * invTc);
            // (copies by lane: on one address the compiler adds the lanes one
            // after the other in a loop, 6 of 69 us of a 2-D level)
            double *lp = lam_param + 2 * j * kParamCopies + (threadIdx.x & (kParamCopies - 1));
            atomicAdd(lp, lrr * P.dt_phys * e * inv_nsub * pr);
            atomicAdd(lp + kParamCopies, -lrr * rr * invTc);
            // each factor: the product of the other three
            const double other[4] = {F[1] * F[2] * F[3], F[0] * F[2] * F[3], F[0] * F[1] * F[3], F[0] * F[1] * F[2]};
#pragma unroll
            for (int mm = 0; mm < 4; ++mm) {
                const double g = lrr * base * other[mm];
#pragma unroll
                for (int k = 0; k < NSP; ++k) lYc[k] += sp[mm] == k ? g : 0.0;
            }
        }
        // Tc = T0 + dT, Yc = Y0 + dY
        aT0 += lTc;
        LdT += lTc;
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            aY0[k] += lYc[k];
            LdY[k] += lYc[k];
        }
    }
}

// The cell's update in dual numbers with the tangent tan[slot] of every
// input slot (Slots numbering): outputs out[0..Q) = g*, out[Q] = T^{n+1},
// out[Q+1+k] = Y_k^{n+1}; *qc = the cell's wall-heat-flux contribution at
// level n.
template <int Q, int NSP>
__device__ void cell_eval(const KParams &P, const CellIn<Q, NSP> &in, const double *tan, Dual (&out)[Q + 1 + NSP],
                          Dual &qc)
{
    using A = Dual;
    using L = Lat<Q>;
    using S = Slots<Q, NSP>;
    constexpr int D = L::D;
    auto mk = [&](double v, int slot) -> A {
        A r(v);
        r.d[0] = tan[slot];
        return r;
    };
    A g[Q];
    for (int i = 0; i < Q; ++i) g[i] = mk(in.g[i], S::pull + i);
    constexpr int NSL = n_slots<Q>();
    double Tv[NSL], Yv[NSL][NSP];
    slot_scalars<Q, NSP>(P, in, Tv, Yv);
    A T[NSL], Y[NSL][NSP], R[NSL], Tw[NSL];
    for (int s = 0; s < NSL; ++s) {
        Tw[s] = mk(in.Tw[s], S::wall + s);
        if (in.kind[s] == kFluid) {
            T[s] = mk(Tv[s], S::scal + s * (1 + NSP));
            A Ys[NSP];
            for (int k = 0; k < NSP; ++k) {
                Y[s][k] = mk(Yv[s][k], S::scal + s * (1 + NSP) + 1 + k);
                Ys[k] = Y[s][k];
            }
            R[s] = density_a<NSP>(P, T[s], Ys);
        }
    }
    // ghosts (Sec. III.B): images are fluid slots
    for (int s = 0; s < NSL; ++s) {
        if (in.kind[s] == kFluid) continue;
        const int im = in.img[s];
        if (in.kind[s] == kIso) {
            T[s] = A(2.0) * Tw[s] - T[im];
            A Ys[NSP];
            for (int k = 0; k < NSP; ++k) {
                Y[s][k] = Y[im][k];
                Ys[k] = Y[im][k];
            }
            R[s] = A(2.0) * density_a<NSP>(P, Tw[s], Ys) - R[im];
        } else if (in.kind[s] == kInflow) {
            T[s] = A(2.0 * P.T_in) - T[im];
            for (int k = 0; k < NSP; ++k) Y[s][k] = A(2.0 * P.Y_in[k]) - Y[im][k];
            R[s] = A(2.0 * P.rho_in) - R[im];
        } else {
            T[s] = T[im];
            for (int k = 0; k < NSP; ++k) Y[s][k] = Y[im][k];
            R[s] = R[im];
        }
    }
    const A rho = R[0];
    A m[3] = {0.0, 0.0, 0.0};
    for (int i = 0; i < Q; ++i) {
        m[0] += A((double)L::cx(i)) * g[i];
        m[1] += A((double)L::cy(i)) * g[i];
        m[2] += A((double)L::cz(i)) * g[i];
    }
    const A inv_rc = A(1.0) / (rho * A(kCs2));
    const A u[3] = {m[0] * inv_rc, m[1] * inv_rc, m[2] * inv_rc};
    const A inv_rho = A(1.0) / rho;
    A diffT = 0.0, CT = 0.0, grad[3] = {0.0, 0.0, 0.0}, diffY[NSP], CY[NSP];
    for (int k = 0; k < NSP; ++k) diffY[k] = CY[k] = 0.0;
    qc = 0.0;
    for (int d = 0; d < D; ++d) {
        const int sl[5] = {1 + 4 * d, 2 + 4 * d, 0, 3 + 4 * d, 4 + 4 * d};
        bool near = false;
        for (int j = 0; j < 5; ++j) near |= in.kind[sl[j]] != kFluid;
        // wall heat flux through the first-neighbour walls
        for (int j = 1; j <= 3; j += 2)
            if (in.kind[sl[j]] == kIso) {
                A Yc[NSP];
                for (int k = 0; k < NSP; ++k) Yc[k] = Y[0][k];
                qc += A(2.0 * P.alpha) * density_a<NSP>(P, Tw[sl[j]], Yc) * (T[0] - Tw[sl[j]]);
            }
        const A ud = u[d];
        const A d1r = d1(R[sl[0]], R[sl[1]], R[sl[2]], R[sl[3]], R[sl[4]]);
        {
            const A a = T[sl[0]], b = T[sl[1]], c = T[sl[2]], e = T[sl[3]], f = T[sl[4]];
            diffT += d2(a, b, c, e, f) + d1r * d1(a, b, c, e, f) * inv_rho;
            CT += ud * (near ? A(0.5) * (e - b) : weno3(a, b, c, e, f, ud));
        }
        A cY[NSP], sumc = 0.0;
        for (int k = 0; k < NSP; ++k) {
            const A a = Y[sl[0]][k], b = Y[sl[1]][k], c = Y[sl[2]][k], e = Y[sl[3]][k], f = Y[sl[4]][k];
            diffY[k] += d2(a, b, c, e, f) + d1r * d1(a, b, c, e, f) * inv_rho;
            cY[k] = near ? A(0.5) * (e - b) : weno3(a, b, c, e, f, ud);
            sumc += cY[k];
        }
        for (int k = 0; k < NSP; ++k) CY[k] += ud * (cY[k] - Y[0][k] * sumc);
        grad[d] = d1r;
    }
    const A alpha = A(P.alpha);
    diffT *= alpha;
    for (int k = 0; k < NSP; ++k) diffY[k] *= alpha;

    A srcT, srcY[NSP], Y0[NSP];
    for (int k = 0; k < NSP; ++k) Y0[k] = Y[0][k];
    chem_source<NSP>(
        P, kExp2Tab, T[0], Y0,
        [&](int j, A &Aj, A &Taj) {
            Aj = mk(P.rx[j].A, S::param + 2 * j);
            Taj = mk(P.rx[j].Ta, S::param + 2 * j + 1);
        },
        srcT, srcY);

    const A DtT = diffT + srcT;
    A DtY[NSP], invW = 0.0;
    for (int k = 0; k < NSP; ++k) {
        DtY[k] = diffY[k] + srcY[k];
        invW += Y[0][k] * A(P.invW[k]);
    }
    const A Wm = A(1.0) / invW;
    A Lam = DtT / T[0];
    for (int k = 0; k < NSP; ++k) Lam += (Wm * A(P.invW[k])) * DtY[k];
    out[Q] = T[0] - CT + DtT;
    for (int k = 0; k < NSP; ++k) out[Q + 1 + k] = Y[0][k] - CY[k] + DtY[k];

    const A uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    A xi[Q], h[Q], pi = 0.0;
    const A half_inv = A(0.5) * inv_rc;
    for (int i = 0; i < Q; ++i) {
        const A wi = A(L::w(i));
        const A cu = A((double)L::cx(i)) * u[0] + A((double)L::cy(i)) * u[1] + A((double)L::cz(i)) * u[2];
        const A feq_r = wi * (A(1.0) + A(3.0) * cu + A(4.5) * cu * cu - A(1.5) * uu);
        const A proj = (A((double)L::cx(i)) - u[0]) * grad[0] + (A((double)L::cy(i)) - u[1]) * grad[1] +
                       (A((double)L::cz(i)) - u[2]) * grad[2];
        xi[i] = A(kCs2) * (feq_r - wi) * proj + wi * rho * A(kCs2) * Lam;
        h[i] = g[i] * inv_rc + xi[i] * half_inv;
        pi += h[i];
    }
    const A sh = A(1.0) - pi;
    for (int i = 0; i < Q; ++i) h[i] += A(L::w(i)) * sh;
    central_fwd<Q>(h, u);
    relax<Q>(h, A(P.omega2), A(P.omega3), A(P.omega4));
    central_inv<Q>(h, u);
    const A rc = rho * A(kCs2);
    for (int i = 0; i < Q; ++i) out[i] = rc * (h[i] - A(L::w(i)) * sh) + A(0.5) * xi[i];
}

// ------------------------------------------------------- the reverse sweep
// Reverse of cm_fwd_line at the input (a, b, d): (la, lb, ld) holds the
// adjoints of (m0, m1, m2) and receives those of (a, b, d); returns the
// contribution to the adjoint of u.
__device__ __forceinline__ double cm_fwd_line_adj(double a, double b, double d, double u, double &la, double &lb,
                                                  double &ld)
{
    const double m0 = a + b + d;
    const double l0 = la, l1 = lb, l2 = ld;
    la = l0 - (1.0 + u) * l1 + (1.0 + u) * (1.0 + u) * l2;
    lb = l0 - u * l1 + u * u * l2;
    ld = l0 + (1.0 - u) * l1 + (1.0 - u) * (1.0 - u) * l2;
    return -m0 * l1 + (2.0 * (a - d) + 2.0 * u * m0) * l2;
}

// Reverse of cm_inv_line at the input moments (m0, m1, m2).
__device__ __forceinline__ double cm_inv_line_adj(double m0, double m1, double m2, double u, double &la, double &lb,
                                                  double &ld)
{
    const double uu = u * u;
    const double A = la, B = lb, E = ld;
    la = 0.5 * (uu - u) * A + (1.0 - uu) * B + 0.5 * (uu + u) * E;
    lb = 0.5 * (2.0 * u - 1.0) * A - 2.0 * u * B + 0.5 * (2.0 * u + 1.0) * E;
    ld = 0.5 * A - B + 0.5 * E;
    (void)m2;
    return 0.5 * (m0 * (2.0 * u - 1.0) + 2.0 * m1) * A - 2.0 * (u * m0 + m1) * B +
           0.5 * (m0 * (2.0 * u + 1.0) + 2.0 * m1) * E;
}

// Reverse of relax(): the orders >= 2 were scaled by (1 - omega).
template <int Q>
__device__ __forceinline__ void relax_adj(double (&lk)[Q], double om2, double om3, double om4)
{
    sfor<0, Q>([&](auto J) {
        constexpr int j = decltype(J)::value;
        constexpr int p = j % 3, q = (j / 3) % 3, r = (Q == 27) ? j / 9 : 0;
        constexpr int order = p + q + r;
        if constexpr (order >= 2) lk[j] *= 1.0 - (order == 2 ? om2 : order == 3 ? om3 : om4);
    });
}

// Reverse of weno3(m2, m1, c0, p1, p2, u) for the adjoint lam of its
// result: adds the adjoints of the five stencil values to l[0..5) (u
// enters through its sign only).
__device__ __forceinline__ void weno3_adj(double m2, double m1, double c0, double p1, double p2, double u, double lam,
                                          double (&l)[5])
{
    const bool neg = u < 0.0;
    const double A = neg ? p2 : m2, B = neg ? p1 : m1, E = neg ? m1 : p1;
    const double eps = 1e-6;
    const double dA = B - A, dB = c0 - B, dE = E - c0;
    const double eA = eps + dA * dA, eB = eps + dB * dB, eE = eps + dE * dE;
    const double eA2 = eA * eA, eB2 = eB * eB, eE2 = eE * eE;
    const double den_p = eE2 + 2.0 * eB2, den_m = eB2 + 2.0 * eA2;
    const double ip = rcp(den_p), im = rcp(den_m);
    const double w_p = eE2 * ip, w_m = eB2 * im;
    const double q0p = 1.5 * c0 - 0.5 * B, q1p = 0.5 * (c0 + E);
    const double q0m = 1.5 * B - 0.5 * A, q1m = 0.5 * (B + c0);
    const double L = neg ? -lam : lam;
    const double lq1p = L * (1.0 - w_p), lq0p = L * w_p, lw_p = L * (q0p - q1p);
    const double lq1m = -L * (1.0 - w_m), lq0m = -L * w_m, lw_m = -L * (q0m - q1m);
    const double leE2 = lw_p * 2.0 * eB2 * ip * ip;
    const double leB2 = -lw_p * 2.0 * eE2 * ip * ip + lw_m * 2.0 * eA2 * im * im;
    const double leA2 = -lw_m * 2.0 * eB2 * im * im;
    const double ldA = leA2 * 4.0 * eA * dA, ldB = leB2 * 4.0 * eB * dB, ldE = leE2 * 4.0 * eE * dE;
    const double lA = -ldA - 0.5 * lq0m;
    const double lB = ldA - ldB - 0.5 * lq0p + 1.5 * lq0m + 0.5 * lq1m;
    const double lC = ldB - ldE + 1.5 * lq0p + 0.5 * lq1p + 0.5 * lq1m;
    const double lE = ldE + 0.5 * lq1p;
    // selects on the values, not on the destination (an indexed store would
    // put l in scratch memory)
    l[0] += neg ? 0.0 : lA;
    l[1] += neg ? lE : lB;
    l[2] += lC;
    l[3] += neg ? lB : lE;
    l[4] += neg ? lA : 0.0;
}

// The backward step runs as two kernels per level.  The first
// (adjoint_collision_kernel) evaluates the cell's update forward and reverses
// the collision, the moments and the velocity's part of the convection: it
// finishes the adjoints of the pulled populations and leaves, per cell, the
// few adjoints the rest needs (AdjMid).  The second (adjoint_stencil_kernel)
// reverses the finite-difference stencils, the ghosts and densities, and
// leaves the stencil scalars' adjoints for the gather.  Split so that each
// kernel's live values fit the registers: what a kernel spills goes through
// memory for every lane.  Measured a level, 1024 x 256 (D2Q9): 63, 43 and 16 us
// for the collision, the stencils and the gather, 126, 147 and 90 MB that they
// must move (29, 34, 21 us at a copy's rate; the gather's reads are partly in
// the caches); 72 x 56 x 40 (D3Q27): 100, 59, 18 us.  Two waves a SIMD in D2Q9
// and for the stencils (three spill: 127 and 88 us), one for the D3Q27
// collision (two spill 395 registers: 209 us).

// Fields of the per-cell state between the two kernels, [field][N]:
// lDtT, lDtY_k (adjoints of the increments Dt), lgrad_d (of d1 rho), u_d,
// aT0, aY0_k (partial adjoints of the cell's own T, Y), lR0 (of its rho).
template <int D, int NSP>
struct AdjMid {
    static constexpr int ls = 0, lgrad = 1 + NSP, u = lgrad + D, aT0 = u + D, aY0 = aT0 + 1,
                         lR0 = aY0 + NSP, n = lR0 + 1;
};

// Where the reverse sweep puts the adjoints of a cell's inputs.
struct AdjOut {
    const double *lo_pop;  // [Q][N] adjoint of the populations the step writes
    const double *lo_sc;   // [1+NSP][N] adjoint of the scalars the step writes
    double *lam_pop;    // [Q][N]: stored (every entry is pulled by one cell)
    double *lam_sc;     // [1+NSP][N]: the cell's own share, completed by the gather
    double *dwallT;     // [N]: accumulated atomically
    double *lam_param;  // [2 n_rx][kParamCopies] in LDS: accumulated atomically
    double *mid;        // [AdjMid::n][N]
    double *nb;         // [S - 1][1+NSP][N]: what each stencil slot's cell receives
};

// Entry of plane k ([planes][N]) at a cell's byte offset: a scalar base and a
// 32-bit offset (N < 2^29), not an address in two registers for each plane.
template <class T>
__device__ __forceinline__ T &plane_at(T *base, long long N, int k, uint32_t off)
{
    return *(T *)((std::conditional_t<std::is_const_v<T>, const char, char> *)(base + (long long)k * N) + off);
}

// A cell as the reverse sweep reads it: its coordinates and codes (boundary
// cells; an interior cell's codes are 0 and its coordinates are not needed).
struct AdjCell {
    long long idx;
    int x, y, z;
    bool bnd;
    unsigned long long pcode, scode;
};

// The fluid cell of a thread; false when there is none.
__device__ __forceinline__ bool adj_cell(const KParams &P, AdjCell &c)
{
    c.idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c.idx >= P.N) return false;
    const int code = P.code[c.idx];
    c.bnd = code == kCodeBoundary;
    c.x = c.y = c.z = 0;
    c.pcode = c.scode = 0;
    if (c.bnd) {
        const unsigned i = (unsigned)c.idx, row = i / (unsigned)P.nx;  // (N < 2^29)
        c.x = (int)(i - row * (unsigned)P.nx);
        c.z = (int)(row / (unsigned)P.ny);
        c.y = (int)(row - (unsigned)c.z * (unsigned)P.ny);
        const ulonglong2 cc = P.cell_code[c.idx];
        c.pcode = cc.x;
        c.scode = cc.y;
    }
    return code != kCodeSolid;
}

// The cell offsets of the neighbours at -1, 0, 1 along each axis (wrapped).
struct AdjNb {
    int x[3], y[3], z[3];
};
__device__ __forceinline__ AdjNb adj_neighbours(const KParams &P, const AdjCell &c)
{
    const int sy = P.nx, sz = P.nx * P.ny;
    AdjNb o = {{-1, 0, 1}, {-sy, 0, sy}, {-sz, 0, sz}};
    if (c.bnd) {
        o.x[0] = c.x == 0 ? P.nx - 1 : -1;
        o.x[2] = c.x == P.nx - 1 ? 1 - P.nx : 1;
        o.y[0] = (c.y == 0 ? P.ny - 1 : -1) * sy;
        o.y[2] = (c.y == P.ny - 1 ? 1 - P.ny : 1) * sy;
        o.z[0] = (c.z == 0 ? P.nz - 1 : -1) * sz;
        o.z[2] = (c.z == P.nz - 1 ? 1 - P.nz : 1) * sz;
    }
    return o;
}

// f(I, population entry that the cell's population I is pulled from) for
// every I: the neighbour's entry, or behind a wall or an inlet the cell's own
// opposite one.
template <int Q, class T, class F>
__device__ __forceinline__ void pull_entries(const KParams &P, const AdjCell &c, T *pop, F &&f)
{
    using L = Lat<Q>;
    const uint32_t own = (uint32_t)c.idx * 8u;
    if (!__any(c.bnd)) {
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            const long long shift = (L::cz(i) * (long long)P.ny + L::cy(i)) * P.nx + L::cx(i);
            f(I, plane_at(pop - shift, P.N, i, own));
        });
        return;
    }
    const AdjNb o = adj_neighbours(P, c);
    sfor<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        const uint32_t src = own + 8u * (uint32_t)(o.x[1 - L::cx(i)] + o.y[1 - L::cy(i)] + o.z[1 - L::cz(i)]);
        const bool fl = decode_pull_kind(c.pcode, i) == kPullFluid;
        f(I, *(fl ? &plane_at(pop, P.N, i, src) : &plane_at(pop, P.N, Q - 1 - i, own)));
    });
}

// sum_d c_d v_d over the axes with c_d != 0 (a product with a constant zero is
// not dropped by itself)
template <int Q, int I>
__device__ __forceinline__ double dot_c(const double (&v)[3])
{
    using L = Lat<Q>;
    double r = 0.0;
    if constexpr (L::cx(I) != 0) r = L::cx(I) * v[0];
    if constexpr (L::cy(I) != 0) r = L::cx(I) != 0 ? r + L::cy(I) * v[1] : L::cy(I) * v[1];
    if constexpr (L::cz(I) != 0) r = L::cx(I) != 0 || L::cy(I) != 0 ? r + L::cz(I) * v[2] : L::cz(I) * v[2];
    return r;
}
// v_d += c_d a
template <int Q, int I>
__device__ __forceinline__ void add_c(double (&v)[3], double a)
{
    using L = Lat<Q>;
    if constexpr (L::cx(I) != 0) v[0] += L::cx(I) * a;
    if constexpr (L::cy(I) != 0) v[1] += L::cy(I) * a;
    if constexpr (L::cz(I) != 0) v[2] += L::cz(I) * a;
}

// One axis of a cell's stencil: T, Y, rho and sum_k Y_k / W_k at the points
// m = -2, -1, 1, 2, a ghost formed from its image; the kinds and images of
// the four slots (s20) and the points' cell offsets along the wrapped axis.
// The points are read here, axis by axis, rather than all at once: every slot
// held through the cell's evaluation took 182 registers in 3-D.
template <int NSP>
struct AdjAxis {
    double T[4], Y[4][NSP], R[4], Sw[4];
    double Tw[2];       // wall temperature behind the isothermal ghosts of side 0, 1
    int wall[2];        // that wall's cell when it is an in-box solid, else -1
    unsigned s20;
    __device__ __forceinline__ int kind(int j) const { return (int)(s20 >> (5 * j)) & 7; }
    __device__ __forceinline__ int image(int j) const { return (int)(s20 >> (5 * j + 3)) & 3; }
    __device__ __forceinline__ bool near() const { return (s20 & 0x39ce7u) != 0; }
};

template <int NSP>
__device__ __forceinline__ void load_axis(const KParams &P, const AdjCell &c, int d, AdjAxis<NSP> &A)
{
    const double *sc = (const double *)P.sc_in;
    const double c0 = P.T_ref_over_W_ref;
    const int stride = d == 0 ? 1 : d == 1 ? P.nx : P.nx * P.ny;
    const int x = d == 0 ? c.x : d == 1 ? c.y : c.z, n = d == 0 ? P.nx : d == 1 ? P.ny : P.nz;
    A.s20 = (unsigned)(c.scode >> (20 * d)) & 0xfffffu;
    int off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) off[j] = slot_offset(j) * stride;
    if (c.bnd) {
#pragma unroll
        for (int j = 0; j < 4; ++j) off[j] = (wrap_once(x + slot_offset(j), n) - x) * stride;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // the value point, or the ghost's image: the point itself, the cell,
        // the first neighbour on the other side, on the same side
        static_assert(kImgSelf == 0 && kImgCell == 1 && kImgMirror == 2 && kImgSame == 3);
        const bool b0 = A.image(j) & 1, b1 = A.image(j) & 2;
        const int same = off[j < 2 ? 1 : 2], mirror = off[j < 2 ? 2 : 1];
        const int lo = b0 ? 0 : off[j], hi = b0 ? same : mirror;
        const int at = b1 ? hi : lo;
        const uint32_t p = (uint32_t)((int)c.idx + at) * 8u;
        A.T[j] = plane_at(sc, P.N, 0, p);
        double sw = 0.0;
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            A.Y[j][k] = plane_at(sc, P.N, 1 + k, p);
            sw += A.Y[j][k] * P.invW[k];
        }
        A.Sw[j] = sw;
        A.R[j] = c0 * rcp(A.T[j] * sw);
    }
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int j1 = side ? 2 : 1, j2 = side ? 3 : 0;
        A.Tw[side] = 0.0;
        A.wall[side] = -1;
        if (A.kind(j2) == kIso) {
            // the two points of a side share their wall, the first non-fluid
            // point from the cell
            const bool second = A.kind(j1) == kFluid;
            const int mw = (side ? 1 : -1) * (second ? 2 : 1);
            const bool out = (unsigned)(x + mw) >= (unsigned)n && !((P.periodic_bits >> (2 * d + side)) & 1u);
            const int w = (int)c.idx + off[second ? j2 : j1];
            A.wall[side] = out ? -1 : w;
            A.Tw[side] = out ? P.face_Td[2 * d + side] : P.wall_T[w];
        }
    }
    if (A.near()) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kd = A.kind(j);
            if (kd == kIso) {
                const double Tw = A.Tw[j < 2 ? 0 : 1];
                A.T[j] = 2.0 * Tw - A.T[j];
                A.R[j] = 2.0 * (c0 * rcp(Tw * A.Sw[j])) - A.R[j];
            } else if (kd == kInflow) {
                A.T[j] = 2.0 * P.T_in - A.T[j];
#pragma unroll
                for (int k = 0; k < NSP; ++k) A.Y[j][k] = 2.0 * P.Y_in[k] - A.Y[j][k];
                A.R[j] = 2.0 * P.rho_in - A.R[j];
            }
        }
    }
}

// First half: the cell's update forward in FP64, then the reverse of the
// collision (central moments and their transforms, the forcing Xi, the
// equilibrium), of the scalars' increments up to Dt, of the convection's
// dependence on u and of the moments (u = m / (rho cs2)).  From the adjoint
// of the outputs (g*, T^{n+1}, Y^{n+1}; read from out) and the weight wT0 of
// the cell's own T (the flame position's linear term): the adjoints of the
// pulled populations (stored) and the cell's AdjMid.
// hxs (D3Q27): [Q][kBlock] doubles of LDS for the moments' input between the
// forward and the reverse half, which together with the relaxed moments, the
// adjoints and a transform's passes would not fit the registers.
// SUB: the source is sub-stepped and reversed by adjoint_chem_kernel.
template <int Q, int NSP, bool SUB>
__device__ __forceinline__ void cell_vjp_collision(const KParams &P, const AdjCell &c, double wT0, const double *tab,
                                                   const AdjOut &out, double *hxs)
{
    using L = Lat<Q>;
    using M = AdjMid<Lat<Q>::D, NSP>;
    constexpr int D = L::D, NS = 1 + NSP;

    // ------------------------------------------------ forward (values)
    const double *pop = (const double *)P.pop_in;
    const double *sc = (const double *)P.sc_in;
    const uint32_t self = (uint32_t)c.idx * 8u;
    double g[Q];
    pull_entries<Q>(P, c, pop, [&](auto I, const double &v) { g[decltype(I)::value] = v; });
    if (c.pcode & 0xaaaaaaaaaaaaaaaaull) {
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i != (Q - 1) / 2) {
                if (decode_pull_kind(c.pcode, i) == kPullInflow)
                    g[i] += 2.0 * L::w(i) * P.rho_in * inflow_cu_c(P, L::cx(i), L::cy(i), L::cz(i), c.x, c.y, c.z);
            }
        });
    }
    double T0 = plane_at(sc, P.N, 0, self), Y0[NSP], invWs = 0.0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) {
        Y0[k] = plane_at(sc, P.N, 1 + k, self);
        invWs += Y0[k] * P.invW[k];
    }
    const double rho = P.T_ref_over_W_ref * rcp(T0 * invWs);
    double m[3] = {0.0, 0.0, 0.0};
    sfor<0, Q>([&](auto I) { add_c<Q, decltype(I)::value>(m, g[decltype(I)::value]); });
    const double inv_rc = rcp(rho * kCs2), inv_rho = rcp(rho);
    double u[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = m[d] * inv_rc;
    // the scalars' outputs are T' = T0 - CT + DtT, Y' = Y0 - CY + DtY with
    // CT = sum_d u_d cT_d, CY_k = sum_d u_d (cY_k - Y0_k sumc): the adjoints of
    // the convection's u (luc) and of Y0 through sumc (us) are linear in the
    // outputs' and are formed with the axis
    double lsc[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) lsc[k] = plane_at(out.lo_sc, P.N, k, self);
    double diffT = 0.0, grad[3] = {0.0, 0.0, 0.0}, diffY[NSP], luc[3] = {0.0, 0.0, 0.0}, us = 0.0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) diffY[k] = 0.0;
#pragma unroll 1
    for (int d = 0; d < D; ++d) {
        const double ud = d == 0 ? u[0] : d == 1 ? u[1] : u[2];
        AdjAxis<NSP> A;
        load_axis<NSP>(P, c, d, A);
        const bool near = A.near();
        const double d1r = d1(A.R[0], A.R[1], rho, A.R[2], A.R[3]);
        double l = 0.0, sumc = 0.0, cY[NSP];
        {
            diffT += d2(A.T[0], A.T[1], T0, A.T[2], A.T[3]) + d1r * d1(A.T[0], A.T[1], T0, A.T[2], A.T[3]) * inv_rho;
            const double cT = near ? 0.5 * (A.T[2] - A.T[1]) : weno3(A.T[0], A.T[1], T0, A.T[2], A.T[3], ud);
            l -= lsc[0] * cT;
        }
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            const double p = A.Y[0][k], b = A.Y[1][k], e = A.Y[2][k], f = A.Y[3][k];
            diffY[k] += d2(p, b, Y0[k], e, f) + d1r * d1(p, b, Y0[k], e, f) * inv_rho;
            cY[k] = near ? 0.5 * (e - b) : weno3(p, b, Y0[k], e, f, ud);
            sumc += cY[k];
        }
#pragma unroll
        for (int k = 0; k < NSP; ++k) l -= lsc[1 + k] * (cY[k] - Y0[k] * sumc);
        us += ud * sumc;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            grad[a] = a == d ? d1r : grad[a];
            luc[a] = a == d ? l : luc[a];
        }
    }
    diffT *= P.alpha;
#pragma unroll
    for (int k = 0; k < NSP; ++k) diffY[k] *= P.alpha;
    double srcT, srcY[NSP];
    chem_source<NSP>(
        P, tab, T0, Y0,
        [&](int j, double &Aj, double &Taj) {
            Aj = P.rx[j].A;
            Taj = P.rx[j].Ta;
        },
        srcT, srcY);
    const double DtT = diffT + srcT;
    double DtY[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) DtY[k] = diffY[k] + srcY[k];
    const double Wm = rcp(invWs);
    const double inv_T0 = rcp(T0);
    double Lam = DtT * inv_T0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) Lam += (Wm * P.invW[k]) * DtY[k];

    // xi_i = cs2 (feq_i - w_i) proj_i + w_i rho cs2 Lam, feq_i and proj_i
    // from u and grad (recomputed in the reverse)
    struct Feq {
        double feq, proj, cu;
    };
    auto feq_of = [](auto I, const double (&u)[3], const double (&grad)[3], double uu, double ug) -> Feq {
        constexpr int i = decltype(I)::value;
        const double cu = dot_c<Q, i>(u);
        return {L::w(i) * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu), dot_c<Q, i>(grad) - ug, cu};
    };
    const double half_inv = 0.5 * inv_rc;
    double hx[Q], pi = 0.0;
    {
        const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
        const double ug = u[0] * grad[0] + u[1] * grad[1] + u[2] * grad[2];
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            const Feq f = feq_of(I, u, grad, uu, ug);
            const double xi = kCs2 * (f.feq - L::w(i)) * f.proj + L::w(i) * rho * kCs2 * Lam;
            hx[i] = g[i] * inv_rc + xi * half_inv;
            pi += hx[i];
        });
    }
    const double sh = 1.0 - pi;
#pragma unroll
    for (int i = 0; i < Q; ++i) hx[i] += L::w(i) * sh;
    // the relaxed central moments (the passes' inputs are recomputed in the
    // reverse)
    double kr[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) kr[i] = hx[i];
    if constexpr (Q == 27) {
#pragma unroll
        for (int i = 0; i < Q; ++i) hxs[i * kBlock + threadIdx.x] = hx[i];
    }
    auto hx_at = [&](int i) -> double {
        if constexpr (Q == 27)
            return hxs[i * kBlock + threadIdx.x];
        else
            return hx[i];
    };
    central_fwd<Q>(kr, u);
    relax<Q>(kr, P.omega2, P.omega3, P.omega4);
    const double rc = rho * kCs2;

    // ------------------------------------------------------ reverse
    double lu[3], lrho = 0.0, linv_rc = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) lu[d] = luc[d];

    // out_i = rc (h3_i - w_i sh) + xi_i / 2, h3 = central_inv(kr); the passes
    // in x and y plane by plane
    double lh[Q], lrc = 0.0, lsh = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) lh[i] = plane_at(out.lo_pop, P.N, i, self);
    {
        double(&iz)[Q] = kr;  // in place: the z pass's input is its output's transform
        if constexpr (Q == 27) {
#pragma unroll
            for (int r = 0; r < 9; ++r) cm_inv_line(iz[r], iz[r + 9], iz[r + 18], u[2]);
        }
#pragma unroll
        for (int zp = 0; zp < Q / 9; ++zp) {
            const int o = 9 * zp;
            double iy[9];
#pragma unroll
            for (int p = 0; p < 9; ++p) iy[p] = iz[o + p];
#pragma unroll
            for (int p = 0; p < 3; ++p) cm_inv_line(iy[p], iy[p + 3], iy[p + 6], u[1]);
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                double h3[3] = {iy[3 * l], iy[3 * l + 1], iy[3 * l + 2]};
                cm_inv_line(h3[0], h3[1], h3[2], u[0]);
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int i = o + 3 * l + q;
                    lrc += lh[i] * (h3[q] - L::w(i) * sh);
                    lh[i] *= rc;
                    lsh -= L::w(i) * lh[i];
                }
                lu[0] += cm_inv_line_adj(iy[3 * l], iy[3 * l + 1], iy[3 * l + 2], u[0], lh[o + 3 * l],
                                         lh[o + 3 * l + 1], lh[o + 3 * l + 2]);
            }
#pragma unroll
            for (int p = 0; p < 3; ++p)
                lu[1] += cm_inv_line_adj(iz[o + p], iz[o + p + 3], iz[o + p + 6], u[1], lh[o + p], lh[o + p + 3],
                                         lh[o + p + 6]);
        }
        if constexpr (Q == 27) {
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                cm_fwd_line(iz[r], iz[r + 9], iz[r + 18], u[2]);
                lu[2] += cm_inv_line_adj(iz[r], iz[r + 9], iz[r + 18], u[2], lh[r], lh[r + 9], lh[r + 18]);
            }
        }
    }
    relax_adj<Q>(lh, P.omega2, P.omega3, P.omega4);
    // central_fwd, reversed
    if constexpr (Q == 27) {
        double hz[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) hz[i] = hx_at(i);
#pragma unroll
        for (int l = 0; l < Q / 3; ++l) cm_fwd_line(hz[3 * l], hz[3 * l + 1], hz[3 * l + 2], u[0]);
#pragma unroll
        for (int zp = 0; zp < Q / 9; ++zp)
#pragma unroll
            for (int p = 0; p < 3; ++p) cm_fwd_line(hz[9 * zp + p], hz[9 * zp + p + 3], hz[9 * zp + p + 6], u[1]);
#pragma unroll
        for (int r = 0; r < 9; ++r)
            lu[2] += cm_fwd_line_adj(hz[r], hz[r + 9], hz[r + 18], u[2], lh[r], lh[r + 9], lh[r + 18]);
    }
#pragma unroll
    for (int zp = 0; zp < Q / 9; ++zp) {
        // (the plane's input read again, not kept)
        if constexpr (Q == 27) asm volatile("" ::: "memory");
        const int o = 9 * zp;
        double hp[9], hy[9];
#pragma unroll
        for (int p = 0; p < 9; ++p) hy[p] = hp[p] = hx_at(o + p);
#pragma unroll
        for (int l = 0; l < 3; ++l) cm_fwd_line(hy[3 * l], hy[3 * l + 1], hy[3 * l + 2], u[0]);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            lu[1] += cm_fwd_line_adj(hy[p], hy[p + 3], hy[p + 6], u[1], lh[o + p], lh[o + p + 3], lh[o + p + 6]);
#pragma unroll
        for (int l = 0; l < 3; ++l)
            lu[0] += cm_fwd_line_adj(hp[3 * l], hp[3 * l + 1], hp[3 * l + 2], u[0], lh[o + 3 * l], lh[o + 3 * l + 1],
                                     lh[o + 3 * l + 2]);
    }
    // hx = h0 + w sh, sh = 1 - sum h0
#pragma unroll
    for (int i = 0; i < Q; ++i) lsh += L::w(i) * lh[i];
    // (from here the outputs' adjoints are read again and the equilibrium's
    // terms formed again: kept from above they would be 100 more values)
    asm volatile("" : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(grad[0]), "+v"(grad[1]), "+v"(grad[2])::"memory");
    double ag[Q];
    double lLam = 0.0, lgrad[3] = {0.0, 0.0, 0.0}, luu = 0.0;
    {
        const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
        const double ug = u[0] * grad[0] + u[1] * grad[1] + u[2] * grad[2];
        double lug = 0.0;
        sfor<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            constexpr double wi = L::w(i);
            const double lh0 = lh[i] - lsh;
            const Feq f = feq_of(I, u, grad, uu, ug);
            // h0 = g inv_rc + xi inv_rc / 2 = hx - w sh
            ag[i] = inv_rc * lh0;
            const double lxi = 0.5 * plane_at(out.lo_pop, P.N, i, self) + half_inv * lh0;
            linv_rc += lh0 * (rc * (hx_at(i) - wi * sh));
            // xi = cs2 (feq - w) proj + w rho cs2 Lam
            const double lfeq = kCs2 * f.proj * lxi;
            const double lproj = kCs2 * (f.feq - wi) * lxi;
            lLam += wi * lxi;
            // proj = sum_d c_d grad_d - sum_d u_d grad_d
            add_c<Q, i>(lgrad, lproj);
            lug -= lproj;
            // feq = w (1 + 3 cu + 9/2 cu^2 - 3/2 uu)
            add_c<Q, i>(lu, wi * (3.0 + 9.0 * f.cu) * lfeq);
            luu -= 1.5 * wi * lfeq;
        });
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lgrad[d] += lug * u[d];
            lu[d] += lug * grad[d] + 2.0 * u[d] * luu;
        }
        lrho += kCs2 * Lam * lLam;
        lLam *= rho * kCs2;
    }
    lrho += kCs2 * lrc;

    // (the scalars and their outputs' adjoints, too, are read again)
    asm volatile("" ::: "memory");
    T0 = plane_at(sc, P.N, 0, self);
#pragma unroll
    for (int k = 0; k < NSP; ++k) Y0[k] = plane_at(sc, P.N, 1 + k, self);
#pragma unroll
    for (int k = 0; k < NS; ++k) lsc[k] = plane_at(out.lo_sc, P.N, k, self);
    // scalar outputs: T' = T0 - CT + DtT, Y' = Y0 - CY + DtY
    double aT0 = lsc[0] + wT0, aY0[NSP];
    double lDtT = lsc[0], lDtY[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) {
        aY0[k] = lsc[1 + k] + lsc[1 + k] * us;
        lDtY[k] = lsc[1 + k];
    }
    // Lam = DtT / T0 + sum_k Wm / W_k DtY_k, Wm = 1 / sum_k Y0_k / W_k
    lDtT += lLam * inv_T0;
    aT0 -= lLam * DtT * inv_T0 * inv_T0;
    double lWm = 0.0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) {
        lDtY[k] += lLam * Wm * P.invW[k];
        lWm += lLam * P.invW[k] * DtY[k];
    }
    const double linvWs = -lWm * Wm * Wm;
#pragma unroll
    for (int k = 0; k < NSP; ++k) aY0[k] += linvWs * P.invW[k];
    // u = m / (rho cs2)
    double lm[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lm[d] = lu[d] * inv_rc;
        linv_rc += lu[d] * m[d];
    }
    sfor<0, Q>([&](auto I) { ag[decltype(I)::value] += dot_c<Q, decltype(I)::value>(lm); });
    lrho -= linv_rc * inv_rc * inv_rho;

    // pull streaming reads every population entry at most once (the source
    // cell's, or the cell's own opposite entry behind a wall)
    {
        AdjCell c2 = c;  // (the entries computed again, not kept)
        asm volatile("" : "+v"(c2.idx));
        pull_entries<Q>(P, c2, out.lam_pop, [&](auto I, double &v) { v = ag[decltype(I)::value]; });
    }
    // the source, reversed (with sub-steps by adjoint_chem_kernel)
    if constexpr (!SUB) {
        double ls[NS];
        ls[0] = lDtT;
#pragma unroll
        for (int k = 0; k < NSP; ++k) ls[1 + k] = lDtY[k];
        chem_vjp<NSP>(P, tab, T0, Y0, ls, aT0, aY0, out.lam_param);
    }
    auto mid = [&](int k) -> double & { return plane_at(out.mid, P.N, k, self); };
    mid(M::ls) = lDtT;
#pragma unroll
    for (int k = 0; k < NSP; ++k) mid(M::ls + 1 + k) = lDtY[k];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        mid(M::lgrad + d) = lgrad[d];
        mid(M::u + d) = u[d];
    }
    mid(M::aT0) = aT0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) mid(M::aY0 + k) = aY0[k];
    mid(M::lR0) = lrho;
}

// The source's reverse where it is sub-stepped, from the cell's AdjMid and into
// its aT0, aY0.
template <int Q, int NSP>
__device__ __forceinline__ void cell_vjp_chem(const KParams &P, const AdjCell &c, const double *tab, const AdjOut &out)
{
    using M = AdjMid<Lat<Q>::D, NSP>;
    const uint32_t self = (uint32_t)c.idx * 8u;
    const double *sc = (const double *)P.sc_in;
    auto mid = [&](int k) -> double & { return plane_at(out.mid, P.N, k, self); };
    double Y0[NSP], ls[1 + NSP], aT0 = mid(M::aT0), aY0[NSP];
    const double T0 = plane_at(sc, P.N, 0, self);
#pragma unroll
    for (int k = 0; k < NSP; ++k) {
        Y0[k] = plane_at(sc, P.N, 1 + k, self);
        aY0[k] = mid(M::aY0 + k);
    }
#pragma unroll
    for (int k = 0; k < 1 + NSP; ++k) ls[k] = mid(M::ls + k);
    chem_vjp<NSP>(P, tab, T0, Y0, ls, aT0, aY0, out.lam_param);
    mid(M::aT0) = aT0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) mid(M::aY0 + k) = aY0[k];
}

// Second half: the reverse of the finite-difference stencils (diffusion,
// the convection's dependence on the stencil values, d1 rho), the ghosts
// and densities and the wall-heat-flux term (weight wq), from the cell's
// AdjMid: the adjoints of the stencil's T, Y for the gather, field by field,
// and of the wall temperatures (atomically).
template <int Q, int NSP>
__device__ __forceinline__ void cell_vjp_stencil(const KParams &P, const AdjCell &c, double wq, const AdjOut &out)
{
    using L = Lat<Q>;
    using M = AdjMid<Lat<Q>::D, NSP>;
    constexpr int D = L::D, NS = 1 + NSP;
    constexpr double c1[5] = {1.0 / 12.0, -8.0 / 12.0, 0.0, 8.0 / 12.0, -1.0 / 12.0};
    constexpr double c2[5] = {-1.0 / 12.0, 16.0 / 12.0, -30.0 / 12.0, 16.0 / 12.0, -1.0 / 12.0};
    const double c0 = P.T_ref_over_W_ref;
    const uint32_t self = (uint32_t)c.idx * 8u;
    const double *sc = (const double *)P.sc_in;
    auto mid = [&](int k) -> double { return plane_at(out.mid, P.N, k, self); };
    double ls[NS];
#pragma unroll
    for (int o = 0; o < NS; ++o) ls[o] = mid(M::ls + o);
    double aT0 = mid(M::aT0), aY0[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) aY0[k] = mid(M::aY0 + k);
    double lR0 = mid(M::lR0);
    const double lCT = -plane_at(out.lo_sc, P.N, 0, self);
    double lCY[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) lCY[k] = -plane_at(out.lo_sc, P.N, 1 + k, self);

    double Y0[NSP], Sw0 = 0.0;
    const double T0 = plane_at(sc, P.N, 0, self);
#pragma unroll
    for (int k = 0; k < NSP; ++k) {
        Y0[k] = plane_at(sc, P.N, 1 + k, self);
        Sw0 += Y0[k] * P.invW[k];
    }
    const double rho = c0 * rcp(T0 * Sw0), inv_rho = rcp(rho);
    const double ldT = P.alpha * ls[0];
    double ldY[NSP];
#pragma unroll
    for (int k = 0; k < NSP; ++k) ldY[k] = P.alpha * ls[1 + k];
    double linv_rho = 0.0;

    // the axes, reversed; each axis's four slots finished and scattered
#pragma unroll 1
    for (int d = 0; d < D; ++d) {
        AdjAxis<NSP> A;
        load_axis<NSP>(P, c, d, A);
        const double ud = mid(M::u + d);
        const bool near = A.near();
        // adjoints of the stencil's values of one field at a time (index 2:
        // the cell, accumulated into aT0, aY0, lR0), the density's first
        double aTw[2] = {0.0, 0.0};
        // wall heat flux q += 2 alpha rho(Tw, Y0) (T0 - Tw), rho(Tw, Y0) = c0 / (Tw Sw0)
#pragma unroll
        for (int side = 0; side < 2; ++side)
            if (A.kind(side ? 2 : 1) == kIso && wq != 0.0) {
                const double Tw = A.Tw[side], rw = c0 * rcp(Tw * Sw0), f = 2.0 * P.alpha * wq;
                aT0 += f * rw;
                aTw[side] += f * (-rw * rcp(Tw) * (T0 - Tw) - rw);
                const double rwS = rw * rcp(Sw0);
#pragma unroll
                for (int k = 0; k < NSP; ++k) aY0[k] += f * (T0 - Tw) * (-rwS * P.invW[k]);
            }
        const double d1r = d1(A.R[0], A.R[1], rho, A.R[2], A.R[3]);
        // diffusion: d2(phi) + d1r d1(phi) / rho, through d1r = d1(R) and rho
        const double dT1 = d1(A.T[0], A.T[1], T0, A.T[2], A.T[3]);
        double s1 = ldT * dT1, lsumc = 0.0;
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            s1 += ldY[k] * d1(A.Y[0][k], A.Y[1][k], Y0[k], A.Y[2][k], A.Y[3][k]);
            lsumc -= lCY[k] * ud * Y0[k];
        }
        linv_rho += d1r * s1;
        const double ld1r = mid(M::lgrad + d) + s1 * inv_rho;
        double lR[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) lR[j] = ld1r * c1[j];
        // Adjoint of a field with the adjoint ld of its diffusion and lc of its
        // convection's derivative
        const double e1 = d1r * inv_rho;
        auto field = [&](double m2, double m1, double v0, double p1, double p2, double ld, double lc, double (&l)[5]) {
#pragma unroll
            for (int j = 0; j < 5; ++j) l[j] = ld * (c2[j] + e1 * c1[j]);
            if (near) {
                l[3] += 0.5 * lc;
                l[1] -= 0.5 * lc;
            } else {
                weno3_adj(m2, m1, v0, p1, p2, ud, lc, l);
            }
        };
        // Ghosts of this axis onto their images (the cell, index 2, or a first
        // neighbour, index 1 or 3): slot j's value is s v(image) + constant, s
        // = -1 behind Dirichlet walls (T, R; Y at inlets).  add: what the image
        // receives beyond s l[a]
        auto onto_images = [&](double (&l)[5], bool species, auto &&add) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int kd = A.kind(j), a = j < 2 ? j : j + 1, side = j < 2 ? 0 : 1, im = A.image(j);
                const int li = im == kImgCell ? 2 : (im == kImgSame) == (side == 0) ? 1 : 3;
                const bool odd = kd == kInflow || (kd == kIso && !species);
                double gv = odd ? -l[a] : l[a];
                if (kd == kIso) gv += add(j, side, a);
                if (kd == kFluid) gv = 0.0;
                l[1] += li == 1 ? gv : 0.0;
                l[3] += li == 3 ? gv : 0.0;
                l[2] += li == 2 ? gv : 0.0;
            }
        };
        // Densities at isothermal ghosts: R = 2 c0 / (Tw Sw) - R(image), onto
        // Tw and the image's Y (f[j] invW_k)
        double f[4] = {0.0, 0.0, 0.0, 0.0};
        if (near) {
            onto_images(lR, false, [&](int j, int side, int a) -> double {
                const double Tw = A.Tw[side], rw = c0 * rcp(Tw * A.Sw[j]);
                aTw[side] -= 2.0 * lR[a] * rw * rcp(Tw);
                f[j] = -2.0 * lR[a] * rw * rcp(A.Sw[j]);
                return 0.0;
            });
        }
        // what each slot's cell receives, stored for the gather (0 at ghost
        // slots): with the densities R = c0 / (T Sw) onto T and Y
        const int nb = 4 * d * NS;
        {
            double l[5];
            field(A.T[0], A.T[1], T0, A.T[2], A.T[3], ldT, lCT * ud, l);
            if (near)
                onto_images(l, false, [&](int, int side, int a) -> double {
                    aTw[side] += 2.0 * l[a];
                    return 0.0;
                });
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int a = j < 2 ? j : j + 1;
                plane_at(out.nb, P.N, nb + j * NS, self) =
                    A.kind(j) == kFluid ? l[a] - lR[a] * (A.R[j] * rcp(A.T[j])) : 0.0;
            }
            aT0 += l[2];
        }
        if (near) {
#pragma unroll
            for (int side = 0; side < 2; ++side)
                if (A.wall[side] >= 0) atomicAdd(&out.dwallT[A.wall[side]], aTw[side]);
        }
        double rS[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) rS[j] = A.R[j] * rcp(A.Sw[j]) * lR[j < 2 ? j : j + 1];
#pragma unroll
        for (int k = 0; k < NSP; ++k) {
            double l[5];
            field(A.Y[0][k], A.Y[1][k], Y0[k], A.Y[2][k], A.Y[3][k], ldY[k], lCY[k] * ud + lsumc, l);
            if (near) onto_images(l, true, [&](int j, int, int) -> double { return f[j] * P.invW[k]; });
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int a = j < 2 ? j : j + 1;
                plane_at(out.nb, P.N, nb + j * NS + 1 + k, self) = A.kind(j) == kFluid ? l[a] - rS[j] * P.invW[k] : 0.0;
            }
            aY0[k] += l[2];
        }
        lR0 += lR[2];
    }

    // inv_rho = 1 / rho; the cell's own slot
    lR0 -= linv_rho * inv_rho * inv_rho;
    const double rT0 = rho * rcp(T0), rS0 = rho * rcp(Sw0);
    plane_at(out.lam_sc, P.N, 0, self) = aT0 - lR0 * rT0;
#pragma unroll
    for (int k = 0; k < NSP; ++k) plane_at(out.lam_sc, P.N, 1 + k, self) = aY0[k] - lR0 * rS0 * P.invW[k];
}

struct AdjParams {
    KParams k;              // pop_in / sc_in: the state of level n
    const double *lam_pop_next;  // [Q][N] adjoint of the populations written by step n
    const double *lam_sc_next;   // [1+NSP][N]
    double *lam_pop;        // [Q][N] adjoint of level n (stored at every fluid cell's entries)
    double *lam_sc;         // [1+NSP][N] (stored at every fluid cell)
    double *dwallT;         // [N] dJ/d wall_T (accumulated)
    double *dparam;         // [2 n_rx]: dJ/dA_j, dJ/dTa_j (accumulated)
    double *mid;            // [AdjMid::n][N] between the first two kernels
    double *nb;             // [S - 1][1+NSP][N] from the stencil kernel to the gather
    int obj_kind;           // LBFD_OBJ_*
    double obj_w;           // weight of this level's q (flame position: times dq/dT of a cell)
};

// The block's sums of dJ/d(A, Ta), summed over their copies, onto the result.
__device__ __forceinline__ void add_params(const KParams &P, const double *red, double *dparam)
{
    for (int j = threadIdx.x; j < 2 * P.n_rx; j += blockDim.x) {
        double v = 0.0;
        for (int q = 0; q < kParamCopies; ++q) v += red[j * kParamCopies + q];
        if (v != 0.0) atomicAdd(&dparam[j], v);
    }
}

template <int Q, int NSP, bool SUB>
__global__ void __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(Q == 27 ? 1 : 2))) adjoint_collision_kernel(const AdjParams AP)
{
    const KParams &P = AP.k;
    __shared__ double red[SUB ? 1 : 2 * LBFD_MAX_REACTIONS * kParamCopies];
    __shared__ double tab[kExpTabN];
    __shared__ double hxs[Q == 27 ? Q * kBlock : 1];
    if constexpr (!SUB)
        for (int j = threadIdx.x; j < 2 * P.n_rx * kParamCopies; j += blockDim.x) red[j] = 0.0;
    for (int j = threadIdx.x; j < kExpTabN; j += blockDim.x) tab[j] = kExp2Tab[j];
    __syncthreads();
    AdjCell c;
    if (adj_cell(P, c)) {
        const double wT0 = AP.obj_kind == LBFD_OBJ_FLAME_POSITION ? AP.obj_w : 0.0;
        AdjOut o{AP.lam_pop_next, AP.lam_sc_next, AP.lam_pop, AP.lam_sc, AP.dwallT, red, AP.mid, AP.nb};
        cell_vjp_collision<Q, NSP, SUB>(P, c, wT0, tab, o, hxs);
    }
    if constexpr (!SUB) {
        __syncthreads();
        add_params(P, red, AP.dparam);
    }
}

// The sub-stepped source's reverse is a serial chain a cell that grows with the
// square of its sub-steps and needs few registers: a kernel of its own runs it
// at four waves a SIMD (126 registers), where the collision kernel's one or two
// left its latency open.  Four levels of 72 x 56 x 40, up to 64 sub-steps: 27.7
// ms with it in the collision kernel, 15.0; ten of 512 x 128 22.7 and 18.8.  A
// single sub-step stays there (its reads and writes of the cell's state would
// cost more than it).
template <int Q, int NSP>
__global__ void __launch_bounds__(kBlock) adjoint_chem_kernel(const AdjParams AP)
{
    const KParams &P = AP.k;
    __shared__ double red[2 * LBFD_MAX_REACTIONS * kParamCopies];
    __shared__ double tab[kExpTabN];
    for (int j = threadIdx.x; j < 2 * P.n_rx * kParamCopies; j += blockDim.x) red[j] = 0.0;
    for (int j = threadIdx.x; j < kExpTabN; j += blockDim.x) tab[j] = kExp2Tab[j];
    __syncthreads();
    AdjCell c;
    if (adj_cell(P, c)) {
        AdjOut o{AP.lam_pop_next, AP.lam_sc_next, AP.lam_pop, AP.lam_sc, AP.dwallT, red, AP.mid, AP.nb};
        cell_vjp_chem<Q, NSP>(P, c, tab, o);
    }
    __syncthreads();
    add_params(P, red, AP.dparam);
}

template <int Q, int NSP>
__global__ void __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(2))) adjoint_stencil_kernel(const AdjParams AP)
{
    const KParams &P = AP.k;
    AdjCell c;
    if (!adj_cell(P, c)) return;
    const double wq = AP.obj_kind == LBFD_OBJ_WALL_HEAT_FLUX ? AP.obj_w : 0.0;
    AdjOut o{AP.lam_pop_next, AP.lam_sc_next, AP.lam_pop, AP.lam_sc, AP.dwallT, nullptr, AP.mid, AP.nb};
    cell_vjp_stencil<Q, NSP>(P, c, wq, o);
}

// The stencil scalars' adjoints: each fluid cell adds to its own share (in
// lam_sc) what the cells whose stencils hold it stored for it, slot by slot
// in a fixed order (so the sums do not depend on scheduling).  The cell
// whose slot s (offset m along axis d) is this cell sits at -m along d;
// at a wall or outside the box nothing is added, and a ghost slot stored 0.
template <int Q, int NSP>
__global__ void __launch_bounds__(kBlock) adjoint_gather_kernel(const AdjParams AP)
{
    constexpr int S = n_slots<Q>(), NS = 1 + NSP;
    const KParams &P = AP.k;
    AdjCell c;
    if (!adj_cell(P, c)) return;
    const uint32_t self = (uint32_t)c.idx * 8u;
    const int st[3] = {1, P.nx, P.nx * P.ny};
    double acc[NS];
#pragma unroll
    for (int v = 0; v < NS; ++v) acc[v] = plane_at(AP.lam_sc, P.N, v, self);
#pragma unroll
    for (int s = 1; s < S; ++s) {
        // (the slot of the opposite offset holds the source cell's kind; a
        // fluid cell behind a first-neighbour wall, whose slot carries the
        // wall's kind, stored 0)
        const int d = (s - 1) / 4, j = (s - 1) % 4, mm = slot_offset(j);
        const bool ok = decode_kind(c.scode, d, 3 - j) == kFluid;
        int o = -mm * st[d];
        if (c.bnd) {
            const int x = d == 0 ? c.x : d == 1 ? c.y : c.z, n = d == 0 ? P.nx : d == 1 ? P.ny : P.nz;
            o = (wrap_once(x - mm, n) - x) * st[d];
        }
        const uint32_t src = (uint32_t)((int)c.idx + (ok ? o : 0)) * 8u;
#pragma unroll
        for (int v = 0; v < NS; ++v) {
            const double b = plane_at(AP.nb, P.N, (s - 1) * NS + v, src);
            acc[v] += ok ? b : 0.0;
        }
    }
#pragma unroll
    for (int v = 0; v < NS; ++v) plane_at(AP.lam_sc, P.N, v, self) = acc[v];
}

struct TanParams {
    KParams k;               // pop_in / sc_in: the state of level n
    const double *dpop;      // [Q][N] tangent of the populations read by the step
    const double *dsc;       // [1+NSP][N] tangent of T, Y
    const double *dwallT;    // [N] tangent of the wall temperatures
    const double *dparam;    // [2 n_rx] tangents of A_j, Ta_j
    double *dpop_out;        // [Q][N] tangent of the populations written (fluid cells)
    double *dsc_out;         // [1+NSP][N] tangent of T, Y written (fluid cells)
    double *dq;              // tangent of this level's q (accumulated)
    int obj_kind;
    double obj_w;            // flame position: dq/dT of a cell
};

template <int Q, int NSP>
__global__ void __launch_bounds__(kBlock) tangent_kernel(const TanParams TP)
{
    using S = Slots<Q, NSP>;
    const KParams &P = TP.k;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= P.N || P.mask[idx] != LBFD_FLUID) return;
    const int x = (int)(idx % P.nx), y = (int)((idx / P.nx) % P.ny), z = (int)(idx / ((long long)P.nx * P.ny));
    CellIn<Q, NSP> in;
    gather_inputs<Q, NSP>(P, x, y, z, idx, in);
    double tan[S::param + 2 * LBFD_MAX_REACTIONS];
    for (int i = 0; i < Q; ++i) tan[S::pull + i] = TP.dpop[(long long)in.tdir[i] * P.N + in.tcell[i]];
    for (int s = 0; s < S::S; ++s) {
        const bool fl = in.kind[s] == kFluid;
        for (int v = 0; v < 1 + NSP; ++v)
            tan[S::scal + s * (1 + NSP) + v] = fl ? TP.dsc[(long long)v * P.N + in.cell[s]] : 0.0;
        tan[S::wall + s] = (in.kind[s] == kIso && in.wall[s] >= 0) ? TP.dwallT[in.wall[s]] : 0.0;
    }
    for (int j = 0; j < 2 * P.n_rx; ++j) tan[S::param + j] = TP.dparam[j];
    Dual out[Q + 1 + NSP], qc;
    cell_eval<Q, NSP>(P, in, tan, out, qc);
    for (int i = 0; i < Q; ++i) TP.dpop_out[(long long)i * P.N + idx] = out[i].d[0];
    for (int k = 0; k < 1 + NSP; ++k) TP.dsc_out[(long long)k * P.N + idx] = out[Q + k].d[0];
    const double dq = TP.obj_kind == LBFD_OBJ_WALL_HEAT_FLUX ? qc.d[0] : TP.obj_w * tan[S::scal];
    if (dq != 0.0) atomicAdd(TP.dq, dq);
}

template <int Q, int NSP>
void launch_collision(const AdjParams &ap, unsigned nb, hipStream_t s)
{
    if (ap.k.chem_substeps_max > 1 && ap.k.n_rx > 0) {
        adjoint_collision_kernel<Q, NSP, true><<<nb, kBlock, 0, s>>>(ap);
        adjoint_chem_kernel<Q, NSP><<<nb, kBlock, 0, s>>>(ap);
    } else {
        adjoint_collision_kernel<Q, NSP, false><<<nb, kBlock, 0, s>>>(ap);
    }
}

bool adjoint_supported(int Q, int nsp) { return (Q == 9 && nsp == 4) || (Q == 27 && nsp == 4); }

int adjoint_mid_fields(int Q, int nsp)
{
    if (nsp != 4) return 0;
    const int mid = Q == 9 ? AdjMid<2, 4>::n : Q == 27 ? AdjMid<3, 4>::n : 0;
    const int nb = Q == 9 ? (n_slots<9>() - 1) * 5 : Q == 27 ? (n_slots<27>() - 1) * 5 : 0;
    return mid + nb;
}

hipError_t launch_adjoint(int Q, int nsp, const KParams &kp, const double *lam_pop_next, const double *lam_sc_next,
                          double *lam_pop, double *lam_sc, double *dwallT, double *dparam, double *mid, int obj_kind,
                          double obj_w, hipStream_t s)
{
    AdjParams ap;
    ap.k = kp;
    ap.lam_pop_next = lam_pop_next;
    ap.lam_sc_next = lam_sc_next;
    ap.lam_pop = lam_pop;
    ap.lam_sc = lam_sc;
    ap.dwallT = dwallT;
    ap.dparam = dparam;
    ap.mid = mid;
    ap.nb = mid + (size_t)(Q == 9 ? AdjMid<2, 4>::n : AdjMid<3, 4>::n) * kp.N;
    ap.obj_kind = obj_kind;
    ap.obj_w = obj_w;
    const unsigned nb = (unsigned)((kp.N + kBlock - 1) / kBlock);
    if (Q == 9 && nsp == 4) {
        launch_collision<9, 4>(ap, nb, s);
        adjoint_stencil_kernel<9, 4><<<nb, kBlock, 0, s>>>(ap);
        adjoint_gather_kernel<9, 4><<<nb, kBlock, 0, s>>>(ap);
    } else if (Q == 27 && nsp == 4) {
        launch_collision<27, 4>(ap, nb, s);
        adjoint_stencil_kernel<27, 4><<<nb, kBlock, 0, s>>>(ap);
        adjoint_gather_kernel<27, 4><<<nb, kBlock, 0, s>>>(ap);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_tangent(int Q, int nsp, const KParams &kp, const double *dpop, const double *dsc,
                          const double *dwallT, const double *dparam, double *dpop_out, double *dsc_out, double *dq,
                          int obj_kind, double obj_w, hipStream_t s)
{
    TanParams tp;
    tp.k = kp;
    tp.dpop = dpop;
    tp.dsc = dsc;
    tp.dwallT = dwallT;
    tp.dparam = dparam;
    tp.dpop_out = dpop_out;
    tp.dsc_out = dsc_out;
    tp.dq = dq;
    tp.obj_kind = obj_kind;
    tp.obj_w = obj_w;
    const unsigned nb = (unsigned)((kp.N + kBlock - 1) / kBlock);
    if (Q == 9 && nsp == 4)
        tangent_kernel<9, 4><<<nb, kBlock, 0, s>>>(tp);
    else if (Q == 27 && nsp == 4)
        tangent_kernel<27, 4><<<nb, kBlock, 0, s>>>(tp);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

__global__ void fill_kernel(double *dst, int n, double v)
{
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) dst[i] = v;
}

hipError_t launch_fill(double *dst, int n, double v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    fill_kernel<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(dst, n, v);
    return hipGetLastError();
}

}  // namespace lbfd
