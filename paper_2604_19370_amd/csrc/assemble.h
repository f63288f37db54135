// assemble.h -- Gauss-quadrature right-hand side of one substep: the kernels.
//
// Weak forms eq. (varPR_wildfire) and eq. (varCN), with F of the generic
// equation at the start of Section 3 evaluated explicitly from the state S
// entering the substep:
//   R_ij = sum_e sum_q w|J| [ S v - alpha (C_diff d_eS d_ev + C_adv bbar_e d_eS v
//                                           - [e=x] C_react S v)
//                             + beta (f v - C_nld S^3 grad S . grad v) ]
//   f = -C_adv (b - bbar).grad S + C_forcing - C_rad S^4
//       + [S > T_ig and fuel > thr] C_ign S exp(-T_act/S)
// and, for the first substep of a step, the fuel right-hand side of the
// compute_rhs listing (Section 7): fuel v (1 - tau rate [ign] S exp(-T_act/S)).
// A forced step adds to f a source sampled at the quadrature points (the
// forcing of the manufactured-solution study, Section 6.1); that is a
// separate compile-time variant, the unforced kernels do not test for it.
// Steps assemble the same quantities in increment form, R - A_impl S (A_impl
// the substep's implicit Kronecker operator): the right-hand side carries only
// the O(tau) change of the state, and is exactly zero where nothing happens.
//
// Schedule: one wavefront owns a strip of 64 element columns (lane = element
// column ey, the strip's first p lanes are halo) and marches along x over a
// tile of element rows.  Per step it takes one new coefficient row of S
// (loaded p+1 rows ahead, coalesced; the fuel's rows only where elements are
// hot), contracts it in y (the y half of the sum factorisation, reused by the
// p+1 elements that share the row; neighbouring columns arrive by DPP rotates),
// finishes the x half, evaluates the pointwise terms at the (p+1)^2 points and
// accumulates the x half of the test-function contraction into per-row
// accumulators.  When a dof row is complete its y contraction is gathered from
// the p neighbouring lanes and stored.  In the stacked variant a workgroup's
// four wavefronts take four consecutive tiles of one strip; the p dof rows
// where two of its tiles meet are summed in two parts (the upper tile's
// elements, then the lower one's) that meet in LDS, so only the first tile
// re-evaluates the p elements above it (in the unstacked variant every tile
// does).  Every dof is summed by one lane, or two parts by two fixed lanes,
// in a fixed order: no atomics, deterministic.  The right-hand sides are
// stored non-temporally (streamed out of L2): the sweep that reads them next
// runs on every XCD.
//
// The marching loop is unrolled by p+1, so the rolling windows (coefficient
// rows, accumulators, pending loads) are renamed, not copied.  The quadrature
// weights are folded into the test functions' values.  The ignition indicator needs S > T_ig somewhere in
// the element; S is a convex combination of the element's coefficients
// (B-splines are non-negative and sum to one), so where no coefficient of any
// element of the wavefront's row exceeds T_ig (less a rounding margin) the
// Arrhenius term is zero and the fuel terms that only it feeds are skipped.
// In increment form an element whose coefficients all equal the
// ambient fixed point (where c_react T + c_forcing - c_rad T^4 = 0) has no
// gradient and no net source, so it contributes nothing; where that holds for
// every element of the wavefront's row, the row's pointwise terms and test
// contractions are skipped too.
#pragma once
#include "dpp.h"
#include "iga_internal.h"

namespace iga {

template <typename T> struct AsmParams {
    const T *S, *F;
    T *R, *RF;
    const T *wx, *wy;   // (b_y(x) - bbar_y) at x-points, (b_x(y) - bbar_x) at y-points
    // integrand  a0 v + ax v_x + ay v_y in element coordinates, S_x and S_y the
    // scaled derivatives of element_values(); every constant carries the
    // element's area and its derivatives' scale:
    //   a0 = cs S + (cx + bcax wy) S_x + (cy + bcay wx) S_y + frc + rad S^4 + ign arr
    //   ax = (dx + nldx S^3) S_x,  ay = (dy + nldy S^3) S_y
    // fuel: af = F (cf - rate arr)
    T cs, frc, rad, cx, cy, bcax, bcay, dx, dy, nldx, nldy, ign, cf, rate;
    T t_ig, t_skip, fthr, t_act;
    // increment form: an element whose coefficients all equal t_fix (the
    // ambient fixed point) contributes nothing, and is skipped when amb != 0
    T t_fix;
    int amb;
    int fuel_all;       // fuel right-hand side nonzero without ignition (direct form)
    int nel_x, nel_y, Nx, Ny, rows, nstrips, ntiles, ngroups;   // rows: dof rows per tile
    int stack;   // tiles of a workgroup share halos (else each evaluates its own);
                 // the kernels are compiled for one or the other
    // source samples src[(ex*Q + qx) * nel_y*Q + ey*Q + qy] (forced variant),
    // weighted by src_w = beta * area
    const T *src;
    T src_w;
};

template <int N> struct Ic {
    static constexpr int value = N;
};

// read-only device data seen through the constant address space (loads the
// compiler may issue as scalar loads where the address is uniform)
template <typename T> using CT = const __attribute__((address_space(4))) T;
template <typename T> __device__ __forceinline__ CT<T> *as_const(const T *p)
{
    return (CT<T> *)p;
}

// a pointer read from memory, known to point to device memory: through it the
// compiler issues global accesses, which do not count as LDS ones (flat ones do,
// and every wait for LDS data waits for them too)
template <typename T> __device__ __forceinline__ T *as_global(T *p)
{
    auto g = (__attribute__((address_space(1))) T *)p;
    asm("" : "+s"(g));   // (or the two casts cancel)
    return (T *)g;
}

// ---------------------------------------------------------------------------
// One element in the uniform basis
// ---------------------------------------------------------------------------
// Splines with open knots and splines with the uniform knots continued past
// both ends are the same functions on the domain.  In the uniform basis every
// element has the same p+1 functions, so all tables are compile-time constants
// (no registers, loads or per-element cases); only the first and last p-1
// coefficients differ from the open-knot ones (to_uniform).  t in [-1/2, 1/2]
// is the element coordinate, g the Gauss nodes, w their weights (sum 1).
__host__ __device__ constexpr double gauss_t(int Q, int q)
{
    if (Q == 2) return q == 0 ? -0.28867513459481288 : 0.28867513459481288;
    if (Q == 3) return q == 0 ? -0.38729833462074169 : q == 1 ? 0.0 : 0.38729833462074169;
    const double inner = 0.16999052179242813, outer = 0.43056815579702629;
    return q == 0 ? -outer : q == 1 ? -inner : q == 2 ? inner : outer;
}
__host__ __device__ constexpr double gauss_w(int Q, int q)
{
    if (Q == 2) return 0.5;
    if (Q == 3) return q == 1 ? 4.0 / 9.0 : 5.0 / 18.0;
    return (q == 1 || q == 2) ? 0.32607257743127307 : 0.17392742256872693;
}
// value of function a at t
__host__ __device__ constexpr double bval(int P, int a, double t)
{
    const double l = 0.5 - t, r = 0.5 + t;
    if (P == 1) return a == 0 ? l : r;
    if (P == 2) return a == 0 ? 0.5 * l * l : a == 1 ? 0.75 - t * t : 0.5 * r * r;
    if (a == 0) return l * l * l / 6.0;
    if (a == 3) return r * r * r / 6.0;
    const double x = a == 1 ? r : l;   // functions 1 and 2 mirror each other
    return (3.0 * x * x * x - 6.0 * x * x + 4.0) / 6.0;
}
// derivatives are taken as DSCALE d/dt (twice the derivative for p = 2, whose
// middle point then needs no arithmetic)
template <int P> struct DScale {
    static constexpr double value = P == 2 ? 2.0 : 1.0;
};
__host__ __device__ constexpr double bder(int P, int a, double t)
{
    const double l = 0.5 - t, r = 0.5 + t;
    if (P == 1) return a == 0 ? -1.0 : 1.0;
    if (P == 2) return a == 0 ? -2.0 * l : a == 1 ? -4.0 * t : 2.0 * r;
    if (a == 0) return -0.5 * l * l;
    if (a == 3) return 0.5 * r * r;
    return a == 1 ? 1.5 * r * r - 2.0 * r : 2.0 * l - 1.5 * l * l;
}
// test side: the Gauss weight times function value / scaled derivative
template <int P> __host__ __device__ constexpr double tval(int a, int q)
{
    return gauss_w(P + 1, q) * bval(P, a, gauss_t(P + 1, q));
}
template <int P> __host__ __device__ constexpr double tder(int a, int q)
{
    return gauss_w(P + 1, q) * bder(P, a, gauss_t(P + 1, q));
}

// Values v and scaled derivatives d at the p+1 points of the spline with
// coefficients c, from its expansion about the element's middle: symmetric
// points share the even and the odd part (p = 2: 9 operations for both where
// the two tables take 18; p = 3: 25 for 32).  d may be left unused.
template <typename T>
__device__ __forceinline__ void element_values(const T (&c)[2], T (&v)[2], T (&d)[2])
{
    const T s = c[1] - c[0];
    v[0] = T(0.5 + gauss_t(2, 0)) * s + c[0];
    v[1] = T(0.5 + gauss_t(2, 1)) * s + c[0];
    d[0] = d[1] = s;
}
template <typename T>
__device__ __forceinline__ void element_values(const T (&c)[3], T (&v)[3], T (&d)[3])
{
    constexpr double g = gauss_t(3, 2);
    const T s = c[2] - c[0];                          // 2 S'(0)
    const T e = (c[2] + c[0]) - T(2) * c[1];          // S''
    const T m = T(0.125 + 0.5 * g * g) * e + c[1];
    v[0] = T(-0.5 * g) * s + m;
    v[1] = T(0.125) * e + c[1];
    v[2] = T(0.5 * g) * s + m;
    d[0] = T(-2.0 * g) * e + s;
    d[1] = s;
    d[2] = T(2.0 * g) * e + s;
}
template <typename T>
__device__ __forceinline__ void element_values(const T (&c)[4], T (&v)[4], T (&d)[4])
{
    const T p = c[1] + c[2], o = c[0] + c[3], m = c[2] - c[1], f = c[3] - c[0], b = o - p;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double g = gauss_t(4, 2 + k);
        const T even = T(1.0 / 48 + 0.25 * g * g) * o + T(23.0 / 48 - 0.25 * g * g) * p;
        const T a = T(g / 8 + g * g * g / 6), q = T(5 * g / 8 - g * g * g / 2);
        v[2 + k] = a * f + (q * m + even);
        v[1 - k] = -a * f + (-q * m + even);
        const T de = T(0.125 + 0.5 * g * g) * f + T(0.625 - 1.5 * g * g) * m;
        d[2 + k] = T(0.5 * g) * b + de;
        d[1 - k] = T(-0.5 * g) * b + de;
    }
}

// Element e of n: the open-knot coefficients c of its functions become the
// uniform ones (u_0 = 2 c_0 - c_1 for p = 2; u_1 = (3 c_1 - c_2) / 2,
// u_0 = 6 c_0 - 4 u_1 - u_2 for p = 3; mirrored at the other end), by knot
// insertion.  Only e = 0, 1, n-2, n-1 change.
template <typename T, int P>
__device__ __forceinline__ void to_uniform(T (&c)[P + 1], int e, int n)
{
    if constexpr (P == 2) {
        c[0] = e == 0 ? T(2) * c[0] - c[1] : c[0];
        c[2] = e == n - 1 ? T(2) * c[2] - c[1] : c[2];
    }
    if constexpr (P == 3) {
        c[1] = e == 0 ? T(1.5) * c[1] - T(0.5) * c[2] : c[1];
        c[0] = e == 0 ? T(6) * c[0] - T(4) * c[1] - c[2]
                      : e == 1 ? T(1.5) * c[0] - T(0.5) * c[1] : c[0];
        c[2] = e == n - 1 ? T(1.5) * c[2] - T(0.5) * c[1] : c[2];
        c[3] = e == n - 1 ? T(6) * c[3] - T(4) * c[2] - c[1]
                          : e == n - 2 ? T(1.5) * c[3] - T(0.5) * c[2] : c[3];
    }
}
// its transpose: what the element's uniform test functions collected, for the
// open-knot ones
template <typename T, int P>
__device__ __forceinline__ void from_uniform(T (&r)[P + 1], int e, int n)
{
    if constexpr (P == 2) {
        const T r0 = r[0], r2 = r[2];
        r[1] = e == 0 ? r[1] - r0 : r[1];
        r[0] = e == 0 ? T(2) * r0 : r0;
        r[1] = e == n - 1 ? r[1] - r2 : r[1];
        r[2] = e == n - 1 ? T(2) * r2 : r2;
    }
    if constexpr (P == 3) {
        auto end = [](T &a, T &b, T &c, bool first, bool second) {   // a: outermost
            const T b1 = first ? b - T(4) * a : b;
            c = first ? c - a - T(0.5) * b1 : c;
            b = first ? T(1.5) * b1 : second ? b - T(0.5) * a : b;
            a = first ? T(6) * a : second ? T(1.5) * a : a;
        };
        end(r[0], r[1], r[2], e == 0, e == 1);
        end(r[3], r[2], r[1], e == n - 1, e == n - 2);
    }
}

// The work of one wavefront: dof rows [X0, X1) of strip `strip` (and the
// elements of those rows).
//   halo: also evaluate the p elements above the tile, so that its first p
//         dof rows are complete (the first tile of a workgroup);
//   hold: those p rows get the contributions of the tile's own elements only
//         and go to hd[2][P][64] (T, fuel) for the workgroup to finish;
//   tail: march p more steps without elements, and put the contributions of
//         the tile's last elements to the p rows below it into tl[2][P][64].
//   lf:   this lane's fuel accumulators [Q][Q], 256 lanes apart (LDS)
//   ap:   the same record as a, in constant memory: constants that need not
//         stay in scalar registers are read from it where they are used
//
// Bound by VALU issue at 4096^2 (S3 in FP32: 9 tenths of its time by instruction
// count), by latency on small meshes.  Per element and step (p = 2): 9
// operations for the y half of the new row, 48 for the values and gradient at
// the points, 90 pointwise, 76 for the x half of the test contraction and about
// 20 for the finished row.  The fuel enters only where the ignition terms are
// evaluated (LDS accumulators, y contraction formed there), and its rows are
// requested only there: loaded ahead with every row of S they cost a quarter of
// the launch's reads and 8 registers (unstacked steps: 4096^2 FP32 465 -> 454 us,
// together with the points' exponentials side by side 1500^2 cubic in double
// 422 -> 400).  Constants of the points in vector registers (double, p <= 2):
// 4096^2 1126 -> 1116 us a step.  Against tables per element and column in registers
// (p = 2: 36 of them), which this replaced: FP32 108-120 registers for 152-168
// (4 wavefronts per SIMD for 3), double 237-253 (the test functions' values
// among them) for 340 (2 for 1).  p = 3 takes 168-189 in FP32 (2 wavefronts) and
// 325-362 in double (1, and 45-93 scalar registers spilled to vector lanes).  Both
// assemblies of a Strang step, best tiles: FP32 4096^2 155 + 140 -> 109 + 101 us,
// 1024^2 24.0 + 22.8 -> 19.2 + 17.1, cubic 4096^2 399 + 347 -> 284 + 260; direct
// form in double 4096^2 578 + 408 -> 415 + 250, cubic 1562 + 946 -> 1527 + 830.
template <typename T, int P, bool FUEL, bool SRC = false>
__device__ __forceinline__ void assemble_body(const AsmParams<T> &a, CT<AsmParams<T>> *ap,
                                              const int strip, const int X0,
                                              const int X1, const bool halo, const bool hold, const bool tail,
                                              T *__restrict__ hd, T *__restrict__ tl,
                                              T *__restrict__ lf)
{
    constexpr int Q = P + 1;
    const int lane = threadIdx.x & 63;
    const int J0 = strip * (64 - P);
    const int ey = J0 - P + lane;
    const bool eyok = ey >= 0 && ey < a.nel_y;
    // some lane's element touches the first or last functions in y
    const bool yedge = P > 1 && (strip == 0 || J0 - P + 63 >= a.nel_y - 2);
    const int Ny = a.Ny;
    const int colA = J0 - P + lane, colB = colA + 64;
    const bool okA = colA >= 0 && colA < Ny, okB = lane < P && colB < Ny;

    T kx[Q];   // coefficient of S_x in a0, by y point
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) kx[qy] = eyok ? a.wy[(size_t)ey * Q + qy] : T(0);

    // Raw coefficients of row `row` for columns colA (and colB for the halo).
    // Every lane loads, from its column clamped into the mesh (lanes without
    // a halo column repeat their own); columns outside the mesh are zeroed
    // where the values are consumed, so no lane mask surrounds the loads.
    // Rows from min(X1, nel_x) + p on only feed elements that are not
    // evaluated: the last row that is needed is loaded in their place.
    const int rlast = min(X1, a.nel_x) + P - 1;
    const unsigned offA = (unsigned)min(max(colA, 0), Ny - 1) * (unsigned)sizeof(T);
    const unsigned offB = okB ? (unsigned)colB * (unsigned)sizeof(T) : offA;
    auto fetch = [&](const T *field, int row, T &c0, T &c1) {
        const char *p = reinterpret_cast<const char *>(field) + (size_t)min(row, rlast) * Ny * sizeof(T);
        c0 = *reinterpret_cast<const T *>(p + offA);
        c1 = *reinterpret_cast<const T *>(p + offB);
    };
    // the p+1 coefficients of the lane's element in one row
    auto element_row = [&](T c0, T c1, T(&cb)[Q]) {
        c0 = okA ? c0 : T(0);
        c1 = okB ? c1 : T(0);
        cb[0] = c0;
        cb[1] = lane_ahead<1>(c0, c1, lane);
        if constexpr (Q > 2) cb[2] = lane_ahead<2>(c0, c1, lane);
        if constexpr (Q > 3) cb[3] = lane_ahead<3>(c0, c1, lane);
        if (yedge) {
            int e = ey;   // (its comparisons are made here, not kept as masks)
            asm volatile("" : "+v"(e));
            to_uniform<T, P>(cb, e, a.nel_y);
        }
    };
    // y half of the sum factorisation of one fetched row, the largest
    // coefficient of the row within the lane's element, and whether all of
    // them equal the ambient fixed point (both hold for the function itself:
    // the uniform functions are non-negative and sum to one too)
    auto ytransform = [&](T c0, T c1, T(&v)[Q], T(&d)[Q], T &mx, bool &am) {
        T cb[Q];
        element_row(c0, c1, cb);
        // (compare and select, not fmax: the inputs need no canonicalising,
        // and a NaN coefficient leaves a NaN right-hand side either way)
        mx = cb[0];
        am = cb[0] == a.t_fix;
#pragma unroll
        for (int b = 1; b < Q; ++b) {
            mx = cb[b] > mx ? cb[b] : mx;
            am = am & (cb[b] == a.t_fix);
        }
        element_values(cb, v, d);
    };

    const int E0 = halo ? X0 - P : X0;       // first element row marched
    const int K = X1 - E0 + (tail ? P : 0);   // marching steps
    // rings indexed by (step + i) mod Q
    T tv[Q][Q], td[Q][Q], rmx[Q];
    // raw fuel coefficients, followed while elements are hot: fuel says whether
    // this step's rows are here (pf: the newest).  The first rows of a tile are
    // requested in any case: a tile that is hot from its first step would wait
    // for them
    T rf0[Q], rf1[Q], pf0, pf1;
    bool fuel = true;
    bool ram[Q];
    T acc0[Q][Q], acc1[Q][Q];
    T pc0[Q], pc1[Q];
    // live[s]: the dof row in slot s has received the contribution of an
    // evaluated element (wavefront-uniform); a row without one is exactly zero.
    // burnt[s]: the same for its fuel accumulators
    bool live[Q], burnt[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        live[i] = burnt[i] = false;
#pragma unroll
        for (int q = 0; q < Q; ++q) acc0[i][q] = acc1[i][q] = T(0);
    }
    // window rows E0 .. E0+P-1 (slots 0 .. P-1) and the pending rows (step
    // k consumes row E0 + P + k from slot k mod Q), all requested before the
    // window rows are transformed, so that their latencies overlap
    T wc0[P], wc1[P];
#pragma unroll
    for (int s = 0; s < P; ++s) fetch(a.S, E0 + s, wc0[s], wc1[s]);
#pragma unroll
    for (int s = 0; s < Q; ++s) fetch(a.S, E0 + P + s, pc0[s], pc1[s]);
#pragma unroll
    for (int s = 0; s < P; ++s) fetch(a.F, E0 + s, rf0[s], rf1[s]);
    fetch(a.F, E0 + P, pf0, pf1);
    rf0[P] = rf1[P] = T(0);
#pragma unroll
    for (int s = 0; s < P; ++s) ytransform(wc0[s], wc1[s], tv[s], td[s], rmx[s], ram[s]);
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) kx[qy] = a.bcax * kx[qy] + a.cx;
    // rows of the ring in the uniform basis (to_uniform along x; the rows'
    // maxima and ambient marks stay those of the open-knot rows, which bound
    // the same function): ring row i <- ca i + cb j + cc k
    auto mix_rows = [&](int i, T ca, int j, T cb, int k, T cc) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            tv[i][q] = ca * tv[i][q] + cb * tv[j][q] + cc * tv[k][q];
            td[i][q] = ca * td[i][q] + cb * td[j][q] + cc * td[k][q];
        }
    };
    if constexpr (P == 2) {
        if (E0 == 0) mix_rows(0, T(2), 1, T(-1), 1, T(0));
    }
    if constexpr (P == 3) {
        if (E0 == 0) {
            mix_rows(1, T(1.5), 2, T(-0.5), 2, T(0));
            mix_rows(0, T(6), 1, T(-4), 2, T(-1));
        } else if (E0 == 1) {
            mix_rows(0, T(1.5), 1, T(-0.5), 1, T(0));
        } else if (E0 == a.nel_x - 1) {
            mix_rows(2, T(1.5), 1, T(-0.5), 1, T(0));   // row Nx - 2 is in the window
        }
    }
    // transpose on the accumulated rows: row i += c row j, row i *= c
    auto fuel_at = [&](int s, int q) -> T & { return lf[(s * Q + q) * 256]; };
    auto add_row = [&](int i, int j, T c) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            acc0[i][q] += c * acc0[j][q];
            acc1[i][q] += c * acc1[j][q];
            if (FUEL && burnt[j]) fuel_at(i, q) = (burnt[i] ? fuel_at(i, q) : T(0)) + c * fuel_at(j, q);
        }
        burnt[i] = burnt[i] || burnt[j];
    };
    auto scale_row = [&](int i, T c) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            acc0[i][q] *= c;
            acc1[i][q] *= c;
            if (FUEL && burnt[i]) fuel_at(i, q) *= c;
        }
    };

    const T t_skip = a.t_skip;
    // Constants of the points.  Double: beside the basis values they do not fit
    // the scalar registers (40 to 300 were spilled into vector lanes); p <= 2
    // has vector registers left within its occupancy, p = 3 has not and reads
    // them every step.
    struct Point {
        T rad, cs, frc, nldx, nldy, dx, dy, bcay, cy;
    };
    auto point_constants = [](CT<AsmParams<T>> *cp) {
        return Point{cp->rad, cp->cs, cp->frc, cp->nldx, cp->nldy, cp->dx, cp->dy, cp->bcay, cp->cy};
    };
    constexpr bool held = sizeof(T) == 8 && P < 3;
    Point kheld = point_constants(ap);
    if constexpr (held)
        asm volatile("" : "+v"(kheld.rad), "+v"(kheld.cs), "+v"(kheld.frc), "+v"(kheld.nldx), "+v"(kheld.nldy),
                          "+v"(kheld.dx), "+v"(kheld.dy), "+v"(kheld.bcay), "+v"(kheld.cy));
    // The test functions at the points: immediates, except in double, where
    // forming one in scalar registers takes two instructions of its own each
    // time.  p = 2 has vector registers for one of each mirrored pair
    // (FP64 steps: 4096^2 1107 -> 1067 us, 1024^2 128.6 -> 126.2).
    constexpr bool held_tests = held && P == 2;
    constexpr int NH = (Q * Q + 1) / 2;
    T tvh[NH], tdh[NH];
    if constexpr (held_tests) {
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            tvh[i] = T(tval<P>(i / Q, i % Q));
            tdh[i] = T(tder<P>(i / Q, i % Q));
            asm volatile("" : "+v"(tvh[i]));
            if (tder<P>(i / Q, i % Q) != 0.0) asm volatile("" : "+v"(tdh[i]));
        }
    }
    auto testv = [&](int i, int q) -> T {
        const int k = i * Q + q;
        if constexpr (held_tests) return k < NH ? tvh[k] : tvh[Q * Q - 1 - k];
        return T(tval<P>(i, q));
    };
    auto testd = [&](int i, int q) -> T {
        const int k = i * Q + q;
        if constexpr (held_tests) return k < NH ? tdh[k] : -tdh[Q * Q - 1 - k];
        return T(tder<P>(i, q));
    };
    auto step = [&](auto phase, int n) {
        constexpr int ph = decltype(phase)::value;
        constexpr int snew = (ph + P) % Q;   // slot of the new coefficient row / dof row ex+P
        constexpr int sp1 = (ph + P + Q - 1) % Q, sp2 = (ph + P + 2 * Q - 2) % Q;   // rows ex+P-1, ex+P-2
        const int ex = E0 + n;
        ytransform(pc0[ph], pc1[ph], tv[snew], td[snew], rmx[snew], ram[snew]);
        rf0[snew] = pf0;
        rf1[snew] = pf1;
        fetch(a.S, ex + P + Q, pc0[ph], pc1[ph]);
        if constexpr (P == 2) {
            if (ex == a.nel_x - 1) mix_rows(snew, T(2), sp1, T(-1), sp1, T(0));
        }
        if constexpr (P == 3) {
            if (ex == a.nel_x - 2) mix_rows(snew, T(1.5), sp1, T(-0.5), sp1, T(0));
            if (ex == a.nel_x - 1) mix_rows(snew, T(6), sp1, T(-4), sp2, T(-1));
        }
        // an element whose coefficients all sit at the ambient fixed point
        // has no gradient, no net source and no ignition: in increment form
        // it contributes exactly nothing (the skip is wavefront-uniform)
        bool eam = ram[0];
#pragma unroll
        for (int s = 1; s < Q; ++s) eam = eam & ram[s];
        const bool quiet = !SRC && a.amb && __all(!eyok || eam);
        burnt[snew] = false;
        if (ex < a.nel_x && ex < X1 && !quiet) {
            CT<AsmParams<T>> *cp = ap;
            if constexpr (sizeof(T) == 8) asm volatile("" : "+s"(cp));
            const Point k = held ? kheld : point_constants(cp);
            T ky[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) ky[q] = k.bcay * as_const(a.wx)[(size_t)ex * Q + q] + k.cy;
            T emx = rmx[0];
#pragma unroll
            for (int s = 1; s < Q; ++s) emx = rmx[s] > emx ? rmx[s] : emx;
            const bool hot = (FUEL && a.fuel_all) || __any(emx > t_skip);
            if (hot) {
                if (!fuel) {   // (used after the terms below)
#pragma unroll
                    for (int i = 0; i < Q; ++i) fetch(a.F, ex + i, rf0[(ph + i) % Q], rf1[(ph + i) % Q]);
                }
                fetch(a.F, ex + P + 1, pf0, pf1);
            }
            fuel = hot;
            // linear, loss, forcing, wind and T^3-diffusion terms; the first
            // contribution to the fresh dof row (slot snew) is assigned
#pragma unroll
            for (int qy = 0; qy < Q; ++qy) {
                T cv[Q], cd[Q], S[Q], Sx[Q], Sy[Q], un[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    cv[i] = tv[(ph + i) % Q][qy];
                    cd[i] = td[(ph + i) % Q][qy];
                }
                element_values(cv, S, Sx);
                element_values(cd, Sy, un);
#pragma unroll
                for (int qx = 0; qx < Q; ++qx) {
                    // chains ordered so that no instruction reads two scalar operands
                    const T s = S[qx], s3 = s * s * s;
                    T a0 = (k.rad * s3 + k.cs) * s + k.frc;
                    a0 += kx[qy] * Sx[qx];
                    a0 += ky[qx] * Sy[qx];
                    if constexpr (SRC) {
                        if (eyok)
                            a0 += a.src_w * a.src[((size_t)ex * Q + qx) * ((size_t)a.nel_y * Q) +
                                                  (size_t)ey * Q + qy];
                    }
                    const T ax = (k.nldx * s3 + k.dx) * Sx[qx];
                    const T ay = (k.nldy * s3 + k.dy) * Sy[qx];
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        const int si = (ph + i) % Q;
                        const double d = tder<P>(i, qx);
                        if (i == P && qx == 0) {
                            acc0[si][qy] = a0 * testv(i, qx);
                            acc1[si][qy] = ay * testv(i, qx);
                        } else {
                            acc0[si][qy] += a0 * testv(i, qx);
                            acc1[si][qy] += ay * testv(i, qx);
                        }
                        if (d != 0.0) acc0[si][qy] += ax * testd(i, qx);
                    }
                }
            }
            if (hot) {
                // ignition source and fuel terms (S re-evaluated); its constants
                // are read here
                CT<AsmParams<T>> *hp = ap;
                asm volatile("" : "+s"(hp));
                const T t_ig = hp->t_ig, fthr = hp->fthr, t_act = hp->t_act, ign = hp->ign,
                        cff = hp->cf, rate = hp->rate;
                T fb[Q][Q];   // fuel coefficients of the element's rows
                {
                    T f0[Q], f1[Q];
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        f0[i] = rf0[(ph + i) % Q];
                        f1[i] = rf1[(ph + i) % Q];
                    }
                    if (P > 1 && (ex < P || ex >= a.nel_x - P)) {
                        to_uniform<T, P>(f0, ex, a.nel_x);
                        to_uniform<T, P>(f1, ex, a.nel_x);
                    }
#pragma unroll
                    for (int i = 0; i < Q; ++i) element_row(f0[i], f1[i], fb[i]);
                }
#pragma unroll
                for (int qy = 0; qy < Q; ++qy) {
                    T cv[Q], cf[Q], S[Q], F[Q], arr[Q], un[Q], fa[Q];
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        const int si = (ph + i) % Q;
                        cv[i] = tv[si][qy];
                        cf[i] = T(0);
#pragma unroll
                        for (int b = 0; b < Q; ++b)
                            cf[i] += fb[i][b] * T(bval(P, b, gauss_t(Q, qy)));
                        if (FUEL) fa[i] = burnt[si] ? fuel_at(si, qy) : T(0);
                    }
                    element_values(cv, S, un);
                    bool lit = false;
#pragma unroll
                    for (int qx = 0; qx < Q; ++qx) {
                        F[qx] = T(0);
#pragma unroll
                        for (int i = 0; i < Q; ++i) F[qx] += T(bval(P, i, gauss_t(Q, qx))) * cf[i];
                        arr[qx] = T(0);
                        lit = lit | ((S[qx] > t_ig) & (F[qx] > fthr));
                    }
                    // the points side by side: their chains (division,
                    // exponential) are far longer than they are wide
                    if (__any(lit)) {
#pragma unroll
                        for (int qx = 0; qx < Q; ++qx) {
                            const T v = S[qx] * exp(-t_act / S[qx]);
                            arr[qx] = ((S[qx] > t_ig) & (F[qx] > fthr)) ? v : T(0);
                        }
                    }
#pragma unroll
                    for (int qx = 0; qx < Q; ++qx) {
                        const T a0 = ign * arr[qx];
                        const T af = F[qx] * (cff - rate * arr[qx]);
#pragma unroll
                        for (int i = 0; i < Q; ++i) {
                            acc0[(ph + i) % Q][qy] += a0 * T(tval<P>(i, qx));
                            if (FUEL) fa[i] += af * T(tval<P>(i, qx));
                        }
                    }
                    if (FUEL) {
#pragma unroll
                        for (int i = 0; i < Q; ++i) fuel_at((ph + i) % Q, qy) = fa[i];
                    }
                }
#pragma unroll
                for (int s = 0; s < Q; ++s) burnt[s] = true;
            }
#pragma unroll
            for (int s = 0; s < Q; ++s) live[s] = true;
        } else {
#pragma unroll
            for (int q = 0; q < Q; ++q) acc0[snew][q] = acc1[snew][q] = T(0);
            live[snew] = fuel = false;
        }
        // rows of the open-knot test functions at the ends of x (from_uniform,
        // on sums that are linear in the elements: partial ones of a tile too)
        constexpr int s1 = (ph + 1) % Q, s2 = (ph + 2) % Q;
        if constexpr (P == 2) {
            if (ex == 0) {
                add_row(s1, ph, T(-1));
                scale_row(ph, T(2));
            }
            if (ex == a.nel_x - 1) {
                add_row(s1, s2, T(-1));
                scale_row(s2, T(2));
            }
        }
        if constexpr (P == 3) {
            constexpr int s3 = (ph + 3) % Q;
            if (ex == 0) {
                add_row(s1, ph, T(-4));
                add_row(s2, ph, T(-1));
                scale_row(ph, T(6));
            }
            if (ex == 1) {
                add_row(s1, ph, T(-0.5));
                scale_row(ph, T(1.5));
            }
            if (ex == a.nel_x - 1) {
                add_row(s2, s3, T(-4));
                add_row(s1, s3, T(-1));
                scale_row(s3, T(6));
                add_row(s1, s2, T(-0.5));
                scale_row(s2, T(1.5));
            }
        }
        if (ex >= X0) {
            // dof row ex (slot ph) is complete: y half of the test
            // contraction, gather from the p lanes to the left.  A row that no
            // evaluated element reached stores zero (what the contraction of
            // its zero accumulators gives, +0, without evaluating it).
            auto finish = [&](T(&pb)[Q]) {
                if (yedge) {
                    int e = ey;
                    asm volatile("" : "+v"(e));
                    from_uniform<T, P>(pb, e, a.nel_y);
                }
                T r = pb[0] + lane_behind<1>(pb[1]);
                if constexpr (Q > 2) r += lane_behind<2>(pb[2]);
                if constexpr (Q > 3) r += lane_behind<3>(pb[3]);
                return r;
            };
            T r = T(0), rf = T(0);
            if (live[ph]) {
                T pb[Q];
#pragma unroll
                for (int b = 0; b < Q; ++b) {
                    T s = T(0);
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        s += acc0[ph][q] * testv(b, q);
                        if (tder<P>(b, q) != 0.0) s += acc1[ph][q] * testd(b, q);
                    }
                    pb[b] = eyok ? s : T(0);
                }
                r = finish(pb);
                if (FUEL && burnt[ph]) {
#pragma unroll
                    for (int b = 0; b < Q; ++b) {
                        T s = T(0);
#pragma unroll
                        for (int q = 0; q < Q; ++q) s += fuel_at(ph, q) * T(tval<P>(b, q));
                        pb[b] = eyok ? s : T(0);
                    }
                    rf = finish(pb);
                }
            }
            const int hi = ex - X0, ti = ex - X1;
            if (hold && hi < P) {
                hd[hi * 64 + lane] = r;
                if (FUEL) hd[(P + hi) * 64 + lane] = rf;
            } else if (ti >= 0) {
                tl[ti * 64 + lane] = r;
                if (FUEL) tl[(P + ti) * 64 + lane] = rf;
            } else if (lane >= P && colA < Ny) {
                __builtin_nontemporal_store(r, &a.R[(size_t)ex * Ny + colA]);
                if (FUEL) __builtin_nontemporal_store(rf, &a.RF[(size_t)ex * Ny + colA]);
            }
        }
    };

    // one copy of the step per ring phase (not a second set for the last
    // steps): the code of a launch has to stay in the instruction cache
    for (int n = 0; n < K; n += Q) {
        step(Ic<0>{}, n);
        if (n + 1 < K) step(Ic<1>{}, n + 1);
        if constexpr (Q > 2) {
            if (n + 2 < K) step(Ic<2>{}, n + 2);
        }
        if constexpr (Q > 3) {
            if (n + 3 < K) step(Ic<3>{}, n + 3);
        }
    }
}

// The work of workgroup `grp`: four wavefronts on four consecutive tiles of
// dof rows of one strip.  Stacked (a.stack): only the first evaluates the p
// elements above its tile (the halo); each later wavefront leaves its first
// p dof rows with its own elements' contributions in LDS, its predecessor
// adds the contributions of its last elements to the same rows, and after
// the barrier the later wavefront stores predecessor + own, in that order
// (deterministic, no atomics).  The first tile is p rows shorter than the
// others, so that the four wavefronts march the same number of elements; a
// group covers 4 rows - p dof rows, and a tile shorter than p rows evaluates
// its own halo.  Unstacked: the four wavefronts take neighbouring strips of
// one tile row, every tile evaluates its own halo and no wavefront waits for
// another (better where few wavefronts fit per SIMD).
template <typename T, int P, bool FUEL, bool SRC, bool STK>
__device__ __forceinline__ void assemble_group(const AsmParams<T> &a, CT<AsmParams<T>> *ap, const int grp)
{
    constexpr int G = 4;   // wavefronts per workgroup
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // fuel accumulators: [row slot][point][lane of the workgroup]
    __shared__ T fuel_acc[FUEL ? (P + 1) * (P + 1) * 64 * G : 1];
    T *lf = fuel_acc + (FUEL ? threadIdx.x : 0);
    if constexpr (!STK) {
        // independent wavefronts: four neighbouring strips of one tile row
        const int gw = grp * G + w;
        if (gw >= a.nstrips * a.ntiles) return;
        const int X0 = (gw / a.nstrips) * a.rows;
        assemble_body<T, P, FUEL, SRC>(a, ap, gw % a.nstrips, X0, min(X0 + a.rows, a.Nx), X0 > 0, false,
                                       false, nullptr, nullptr, lf);
    } else {
        __shared__ T part[2][G][2 * P * 64];   // [head, tail][wavefront][(T, fuel) x row x lane]
        const int strip = grp % a.nstrips;
        const int base = (grp / a.nstrips) * (G * a.rows - P);
        // dof rows of the tile of wavefront ww (the first is p rows shorter)
        auto first = [&](int ww) { return min(base + (ww == 0 ? 0 : ww * a.rows - P), a.Nx); };
        auto last = [&](int ww) { return min(base + (ww + 1) * a.rows - P, a.Nx); };
        auto holds = [&](int ww) { return ww > 0 && ww < G && first(ww) > 0 && last(ww) - first(ww) >= P; };
        const int X0 = first(w), X1 = last(w);
        const bool live = X1 > X0;
        const bool hold = holds(w);
        const bool halo = live && X0 > 0 && !hold;
        const bool tail = live && holds(w + 1);
        if (live)
            assemble_body<T, P, FUEL, SRC>(a, ap, strip, X0, X1, halo, hold, tail, part[0][w], part[1][w], lf);
        __syncthreads();
        if (hold) {
            const int lane = threadIdx.x & 63;
            const int colA = strip * (64 - P) - P + lane;
            if (lane >= P && colA < a.Ny) {
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const size_t o = (size_t)(X0 + i) * a.Ny + colA;
                    __builtin_nontemporal_store(part[1][w - 1][i * 64 + lane] + part[0][w][i * 64 + lane], &a.R[o]);
                    if (FUEL)
                        __builtin_nontemporal_store(part[1][w - 1][(P + i) * 64 + lane] + part[0][w][(P + i) * 64 + lane], &a.RF[o]);
                }
            }
        }
    }
}

template <typename T, int P, bool FUEL, bool SRC, bool STK>
__global__ __launch_bounds__(256)
void k_assemble(AsmParams<T> a)
{
    // the record is the only argument: the kernel's argument segment
    assemble_group<T, P, FUEL, SRC, STK>(a, (CT<AsmParams<T>> *)__builtin_amdgcn_kernarg_segment_ptr(),
                                         blockIdx.x);
}

// Batched launch over the members of an ensemble: workgroup b does workgroup
// info[b].y of member info[b].x (x < 0: no work).
template <typename T, int P, bool FUEL, bool STK>
__global__ __launch_bounds__(256)
void k_assemble_batch(const AsmParams<T> *__restrict__ prms, const int2 *__restrict__ info)
{
    const int2 wi = info[blockIdx.x];
    if (wi.x < 0) return;   // the whole workgroup
    // read once, before any store: read where it is used, the record is fetched
    // again after every store that might have changed it (with global accesses,
    // both assemblies of 16 cubic 2048^2 members in FP32: 1509 + 1145 -> 1022 + 920 us;
    // with the fuel accumulators in registers, before they moved to LDS, 1216 + 1181)
    AsmParams<T> a = prms[wi.x];
    a.S = as_global(a.S);
    a.F = as_global(a.F);
    a.R = as_global(a.R);
    a.RF = as_global(a.RF);
    a.wx = as_global(a.wx);
    a.wy = as_global(a.wy);
    assemble_group<T, P, FUEL, false, STK>(a, as_const(prms + wi.x), wi.y);
}

// The compiled kernel of degree P: unforced or forced (SRC), stacked or not,
// one plan or a batch (never forced).
template <typename T, int P, bool FUEL>
static const void *asm_kernel_t(bool src, bool stk, bool batch)
{
    if (batch)
        return stk ? reinterpret_cast<const void *>(k_assemble_batch<T, P, FUEL, true>)
                   : reinterpret_cast<const void *>(k_assemble_batch<T, P, FUEL, false>);
    if (src)
        return stk ? reinterpret_cast<const void *>(k_assemble<T, P, FUEL, true, true>)
                   : reinterpret_cast<const void *>(k_assemble<T, P, FUEL, true, false>);
    return stk ? reinterpret_cast<const void *>(k_assemble<T, P, FUEL, false, true>)
               : reinterpret_cast<const void *>(k_assemble<T, P, FUEL, false, false>);
}
template <typename T, int P> static const void *asm_kernel(bool fuel, bool src, bool stk, bool batch)
{
    return fuel ? asm_kernel_t<T, P, true>(src, stk, batch) : asm_kernel_t<T, P, false>(src, stk, batch);
}

// one translation unit per precision and degree (assemble_f1.hip, ..)
const void *asm_kernel_f1(bool fuel, bool src, bool stk, bool batch);
const void *asm_kernel_f2(bool fuel, bool src, bool stk, bool batch);
const void *asm_kernel_f3(bool fuel, bool src, bool stk, bool batch);
const void *asm_kernel_d1(bool fuel, bool src, bool stk, bool batch);
const void *asm_kernel_d2(bool fuel, bool src, bool stk, bool batch);
const void *asm_kernel_d3(bool fuel, bool src, bool stk, bool batch);

}  // namespace iga
