// assemble.hip -- launch of the right-hand-side kernels (assemble.h), and the
// non-finite detector.
#include <cmath>
#include <limits>

#include "assemble.h"

namespace iga {

static const void *pick_asm(const iga_plan *pl, bool fuel, bool src, bool stk, bool batch)
{
    if (pl->fp32) {
        if (pl->P == 1) return asm_kernel_f1(fuel, src, stk, batch);
        if (pl->P == 2) return asm_kernel_f2(fuel, src, stk, batch);
        if (pl->P == 3) return asm_kernel_f3(fuel, src, stk, batch);
    } else {
        if (pl->P == 1) return asm_kernel_d1(fuel, src, stk, batch);
        if (pl->P == 2) return asm_kernel_d2(fuel, src, stk, batch);
        if (pl->P == 3) return asm_kernel_d3(fuel, src, stk, batch);
    }
    return nullptr;
}

// The ambient fixed point: the temperature c > 0 at which the source of a
// constant field vanishes, c_react c + c_forcing - c_rad c^4 = 0 (the
// ambient temperature of the generic equation at the start of Section 3;
// 300 K with the default coefficients).  Newton from the radiative root.
static bool ambient_fixed_point(const iga_coeffs &c, double &out)
{
    auto g = [&](double t) { return c.c_react * t + c.c_forcing - c.c_rad * t * t * t * t; };
    double t;
    if (c.c_rad > 0 && c.c_forcing > 0) t = std::pow(c.c_forcing / c.c_rad, 0.25);
    else if (c.c_rad == 0 && c.c_react != 0) t = -c.c_forcing / c.c_react;
    else return false;
    for (int it = 0; it < 60 && std::isfinite(t) && t > 0; ++it) {
        const double d = c.c_react - 4.0 * c.c_rad * t * t * t;
        if (d == 0) return false;
        const double step = g(t) / d;
        t -= step;
        if (std::fabs(step) <= 1e-15 * std::fabs(t)) break;
    }
    if (!std::isfinite(t) || !(t > 0)) return false;
    out = t;
    return true;
}

template <typename T>
static void make_params(const iga_plan *pl, int substep, const void *S, const void *F, void *R,
                        void *RF, AsmParams<T> &a, bool delta, const void *src = nullptr)
{
    const iga_plan_desc &d = pl->d;
    const int P = pl->P;
    std::memset(&a, 0, sizeof a);
    a.S = static_cast<const T *>(S);
    a.F = static_cast<const T *>(F);
    a.R = static_cast<T *>(R);
    a.RF = static_cast<T *>(RF);
    a.wx = pl->asm_wx.as<T>();
    a.wy = pl->asm_wy.as<T>();
    // weights of the explicit (kx_e, ky_e) and implicit (kx_i, ky_i) parts of
    // the linear operator in this substep, and of F (beta)
    double kx_e = 0, ky_e = 0, kx_i = 0, ky_i = 0, beta;
    if (d.scheme == IGA_PR) {
        // substep 0: x implicit, L2 (y) explicit; substep 1: y implicit, L1 (x) explicit
        const double h = 0.5 * d.dt;
        if (substep == 0) { ky_e = h; kx_i = h; }
        else { kx_e = h; ky_i = h; }
        beta = h;
    } else if (d.scheme == IGA_EXPLICIT) {
        // eq. (linear): every term at T^n with weight tau; implicit part M (x) M
        kx_e = ky_e = d.dt;
        beta = d.dt;
    } else {
        // S1 / S3: Crank-Nicolson on L1 over tau/2 (explicit and implicit halves)
        kx_e = kx_i = 0.25 * d.dt;
        beta = 0.5 * d.dt;
    }
    const double react = d.c.c_react;
    double cs, kx, ky, cf;
    if (delta) {
        // increment form: R - (implicit operator) S
        kx = kx_e + kx_i;
        ky = ky_e + ky_i;
        cs = kx * react;
        cf = 0.0;
    } else {
        kx = kx_e;
        ky = ky_e;
        cs = 1.0 + kx * react;
        cf = 1.0;
    }
    // element area, and the scale of element_values()' derivatives per unit of
    // length, folded into the constants
    const double area = pl->X.h * pl->Y.h, ds = P == 2 ? DScale<2>::value : DScale<1>::value;
    const double ix = 1.0 / (ds * pl->X.h), iy = 1.0 / (ds * pl->Y.h);
    a.cs = (T)(cs * area);
    a.frc = (T)(beta * d.c.c_forcing * area);
    a.rad = (T)(-beta * d.c.c_rad * area);
    a.cx = (T)(-kx * d.c.c_adv * d.wind.bbar_x * area * ix);
    a.cy = (T)(-ky * d.c.c_adv * d.wind.bbar_y * area * iy);
    a.bcax = (T)(-beta * d.c.c_adv * area * ix);
    a.bcay = (T)(-beta * d.c.c_adv * area * iy);
    a.dx = (T)(-kx * d.c.c_diff * area * ix * ix);
    a.dy = (T)(-ky * d.c.c_diff * area * iy * iy);
    a.nldx = (T)(-beta * d.c.c_nld * area * ix * ix);
    a.nldy = (T)(-beta * d.c.c_nld * area * iy * iy);
    a.ign = (T)(beta * d.c.c_ign * area);
    a.cf = (T)(cf * area);
    a.rate = (T)(d.dt * d.c.fuel_rate * area);
    a.src_w = (T)(beta * area);
    a.src = static_cast<const T *>(src);
    a.t_ig = (T)d.c.t_ig;
    // S exceeds the largest coefficient of its element by at most a few
    // roundings of the basis contraction; skip only well below T_ig
    a.t_skip = (T)(d.c.t_ig - 1e-4 * std::fabs(d.c.t_ig));
    a.fthr = (T)d.c.fuel_thr;
    a.t_act = (T)d.c.t_act;
    // Increment form, no sampled source: elements whose coefficients all equal
    // the fixed point in the state's precision are skipped, provided the
    // source left at that rounded value, over a step, is far below the
    // state's resolution there (and the point is below the ignition cut).
    a.amb = 0;
    a.t_fix = T(0);
    double tfix;
    if (delta && !src && ambient_fixed_point(d.c, tfix)) {
        // the float nearest to it first: an ambient state is given in few
        // digits (300 K), where Newton in double may end an ulp beside it
        for (const T tf : {(T)(float)tfix, (T)tfix}) {
            const double t = (double)tf;
            const double gres = d.c.c_react * t + d.c.c_forcing - d.c.c_rad * t * t * t * t;
            const double ulp = std::ldexp(t, -std::numeric_limits<T>::digits);
            if (std::fabs(gres) * d.dt <= 1e-3 * ulp && tf < a.t_skip) {
                a.amb = 1;
                a.t_fix = tf;
                break;
            }
        }
    }
    a.fuel_all = cf != 0.0;
    a.nel_x = d.nel_x;
    a.nel_y = d.nel_y;
    a.Nx = pl->Nx;
    a.Ny = pl->Ny;
    a.rows = pl->asm_rows;
    a.nstrips = (pl->Ny + (64 - P) - 1) / (64 - P);
    a.stack = pl->asm_stack;
    a.ntiles = (pl->Nx + a.rows - 1) / a.rows;
    a.ngroups = (pl->Nx + 4 * a.rows - P - 1) / (4 * a.rows - P);
}

double assembly_work(const iga_plan *pl)
{
    return (double)((pl->Ny + (64 - pl->P) - 1) / (64 - pl->P)) * pl->Nx;
}

// Default tile height.  Small launches leave most of the chip idle, and a
// launch lasts as long as one wavefront marches its tile and halo: the smallest
// tiles (p + 1 rows) are fastest (a 64^2 p = 2 FP64 step: 73 us at 3 rows, 78 at
// 4, 85 at 5).  Large launches are bound by VALU issue and want few halo rows.
// Between, the best height of a sweep of steps over 64^2 .. 4096^2 grows like the
// square root of the launch (best heights at 1024^2, 2048^2, 4096^2: FP32 p = 2
// 5, 6, 11 and p = 3 5, 8, 18; FP64 p = 2 5, 7, 18 and p = 3 6, 12, 24); heights
// next to it cost a few per cent.  Where one more row lets all workgroups be on
// the chip at once it is taken (512^2 p = 3 FP64: 297 workgroups of 4 rows 166 us a
// step, 234 of 5 rows 153).
int default_assembly_rows(const iga_plan *pl, double work)
{
    const int P = pl->P;
    const double f = pl->fp32 ? (P == 3 ? 30 : 45) : P == 1 ? 45 : P == 2 ? 29 : 22;
    const int rows = std::max(P + 1, (int)std::lround(std::sqrt(work) / f));
    // resident workgroups of four wavefronts per compute unit, by registers
    const double resident = 256.0 * (pl->fp32 ? (P == 1 ? 8 : P == 2 ? 4 : 2) : (P == 1 ? 3 : P == 2 ? 2 : 1));
    return rows + (work / (4 * rows) > resident && work / (4 * (rows + 1)) <= resident);
}

// Tiles share halos within a workgroup except in the largest launches, where
// the halos are a small part and wavefronts that do not wait for each other fill
// the chip better (steps at 3000^2 / 4096^2, stacked to unstacked: FP32 p = 2 284 to
// 294 / 489 to 485 us, FP64 p = 2 643 to 645 / 1142 to 1123).
int default_assembly_stacking(double work) { return work < 2e5; }

// workgroups of one assembly launch: four tiles of one strip each (stacked),
// or four wavefronts on neighbouring strips of a tile row
template <typename T> static int asm_groups(const AsmParams<T> &a)
{
    return a.stack ? a.nstrips * a.ngroups : (a.nstrips * a.ntiles + 3) / 4;
}

template <typename T>
static iga_status launch_t(const iga_plan *pl, int substep, const void *S, const void *F, void *R,
                           void *RF, const void *src, bool delta, hipStream_t s)
{
    AsmParams<T> a;
    make_params<T>(pl, substep, S, F, R, RF, a, delta, src);
    const int blocks = asm_groups(a);
    const void *fn = pick_asm(pl, RF != nullptr, src != nullptr, a.stack != 0, false);
    if (!fn) return fail(IGA_EUNSUPPORTED, "degree not compiled");
    void *args[] = {&a};
    IGA_HIP(hipLaunchKernel(fn, dim3(blocks), dim3(256), args, 0, s));
    return IGA_OK;
}

iga_status launch_assemble(const iga_plan *pl, int substep, const void *S, const void *F, void *R,
                           void *RF, bool delta, hipStream_t s, const void *src)
{
    return pl->fp32 ? launch_t<float>(pl, substep, S, F, R, RF, src, delta, s)
                    : launch_t<double>(pl, substep, S, F, R, RF, src, delta, s);
}

template <typename T>
static iga_status batch_t(const std::vector<iga_plan *> &pls, const std::vector<AsmArgs> &args,
                          BatchLaunch &out)
{
    const int P = pls[0]->P;
    const bool fuel = args[0].RF != nullptr;
    std::vector<AsmParams<T>> prms(pls.size());
    std::vector<int2> info;
    for (size_t m = 0; m < pls.size(); ++m) {
        if (pls[m]->P != P || pls[m]->fp32 != pls[0]->fp32 || (args[m].RF != nullptr) != fuel ||
            pls[m]->asm_stack != pls[0]->asm_stack)
            return fail(IGA_EINVAL,
                        "assembly batch: members differ in degree, precision, fuel or tile stacking");
        make_params<T>(pls[m], args[m].substep, args[m].T, args[m].fuel, args[m].R, args[m].RF,
                       prms[m], true);
        const int groups = asm_groups(prms[m]);
        for (int g = 0; g < groups; ++g) info.push_back(int2{(int)m, g});
    }
    const void *fn = pick_asm(pls[0], fuel, false, pls[0]->asm_stack != 0, true);
    if (!fn) return fail(IGA_EUNSUPPORTED, "degree not compiled");
    out.fn = fn;
    out.nblk = (int)info.size();
    out.njobs = 1;
    out.block = 256;
    out.lds = 0;
    IGA_HIP(out.prm.alloc(prms.size() * sizeof(AsmParams<T>)));
    IGA_HIP(out.info.alloc(info.size() * sizeof(int2)));
    IGA_HIP(hipMemcpy(out.prm.ptr, prms.data(), prms.size() * sizeof(AsmParams<T>),
                      hipMemcpyHostToDevice));
    IGA_HIP(hipMemcpy(out.info.ptr, info.data(), info.size() * sizeof(int2), hipMemcpyHostToDevice));
    return IGA_OK;
}

iga_status build_assemble_batch(const std::vector<iga_plan *> &pls, const std::vector<AsmArgs> &args,
                                BatchLaunch &out)
{
    if (pls.empty() || args.size() != pls.size()) return fail(IGA_EINVAL, "assembly batch: members");
    return pls[0]->fp32 ? batch_t<float>(pls, args, out) : batch_t<double>(pls, args, out);
}

// ---------------------------------------------------------------------------
// non-finite detector (iga_run with check_every > 0)
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_nonfinite(const T *a, const T *b, size_t n, int *flag)
{
    int bad = 0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        bad |= (!isfinite(a[i]) || !isfinite(b[i])) ? 1 : 0;
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

iga_status launch_nonfinite(const iga_plan *pl, const void *T_, const void *F, int *flag,
                            hipStream_t s)
{
    const size_t n = pl->ndof;
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 2048);
    if (pl->fp32)
        hipLaunchKernelGGL(k_nonfinite<float>, dim3(blocks), dim3(256), 0, s,
                           static_cast<const float *>(T_), static_cast<const float *>(F), n, flag);
    else
        hipLaunchKernelGGL(k_nonfinite<double>, dim3(blocks), dim3(256), 0, s,
                           static_cast<const double *>(T_), static_cast<const double *>(F), n, flag);
    IGA_HIP(hipGetLastError());
    return IGA_OK;
}

}  // namespace iga
