// sweep_line.hip -- tables and launch of the line-per-lane solves (sweep_line.h).
#include <cmath>
#include <new>

#include "sweep_line.h"

namespace iga {

static const void *pick_line(const iga_plan *pl, bool diry, bool band, bool batch)
{
    if (pl->fp32) {
        if (pl->P == 1) return line_kernel_f1(diry, band, batch);
        if (pl->P == 2) return line_kernel_f2(diry, band, batch);
        if (pl->P == 3) return line_kernel_f3(diry, band, batch);
    } else {
        if (pl->P == 1) return line_kernel_d1(diry, band, batch);
        if (pl->P == 2) return line_kernel_d2(diry, band, batch);
        if (pl->P == 3) return line_kernel_d3(diry, band, batch);
    }
    return nullptr;
}

// halo rows, wavefronts, own rows and LDS bytes of a tile and its edge tables
struct LineShape {
    int HL, NW, own, lds[2];   // [BAND]
};
template <typename T, int P> static LineShape shape_of()
{
    using S = LineTile<T, P, true>;
    constexpr int edge = LineEdge<T, P>::N * 8;
    static_assert(S::BYTES + edge + LineBand<P>::N * 8 <= 160 * 1024, "a tile fits in LDS");
    return LineShape{S::HL, S::NW, S::OWN, {LineTile<T, P, false>::BYTES + edge, S::BYTES + edge + LineBand<P>::N * 8}};
}
static LineShape line_shape(const iga_plan *pl)
{
    if (pl->fp32) return pl->P == 1 ? shape_of<float, 1>() : pl->P == 2 ? shape_of<float, 2>() : shape_of<float, 3>();
    return pl->P == 1 ? shape_of<double, 1>() : pl->P == 2 ? shape_of<double, 2>() : shape_of<double, 3>();
}

static int line_row_size(int P) { return (3 * P + 2) & ~1; }   // LineRow

// Reversed factorisation A = V W of a banded operator (V unit upper, W lower),
// Gaussian elimination from the last row up: rows [V(r, r+1+j), j < P;
// W(r, r-j), j <= P].
static std::vector<double> reversed_rows(const std::vector<double> &band, int N, int P)
{
    const int W = 2 * P + 1, RS = 2 * P + 1;
    std::vector<double> a(band), f((size_t)N * RS, 0.0);
    for (int k = N - 1; k >= 0; --k) {
        double *ak = &a[(size_t)k * W];   // final: columns k-P .. k
        for (int j = 0; j <= P; ++j)
            if (k - j >= 0) f[(size_t)k * RS + P + j] = ak[P - j];
        for (int i = 1; i <= P && k - i >= 0; ++i) {
            double *ai = &a[(size_t)(k - i) * W];   // row k - i, column k at P + i
            const double v = ai[P + i] / ak[P];
            f[(size_t)(k - i) * RS + (i - 1)] = v;
            for (int j = 1; j <= P; ++j) {           // column k - j of both rows
                const int c = P + i - j;
                if (k - j >= 0 && c >= 0) ai[c] -= v * ak[P - j];
            }
        }
    }
    return f;
}

// Host view of one operator for the tables.
struct LineHostOp {
    const OpHost *o = nullptr;
    std::vector<double> rev;
    int N = 0, P = 0;
    // row r of the forward factors: L (P), 1/U, U/U_rr (P); nullptr outside the line
    const double *fwd(int r) const
    {
        return r < 0 || r >= N ? nullptr : &o->rows[(size_t)row_of(r, o->K0, o->NK, o->nrows) * (2 * P + 2)];
    }
    const double *back(int r) const { return r < 0 || r >= N ? nullptr : &rev[(size_t)r * (2 * P + 1)]; }
};

// py, pc of LineConst for a chunk whose last row is e: the 2P unknowns
// x(e-P+1) .. x(e+P) from the rows of U above the cut and of W below it.
static bool meet(const LineHostOp &h, int e, double *py, double *pc)
{
    const int P = h.P, n = 2 * P;
    std::fill(py, py + P * P, 0.0);
    std::fill(pc, pc + P * P, 0.0);
    if (e + 1 >= h.N) return true;   // nothing after the chunk
    double A[6][12] = {};            // [2P][2P | right-hand sides]
    for (int q = 0; q < n; ++q) {
        const int r = e - P + 1 + q;
        A[q][q] = 1.0;
        if (r <= e) {
            const double *f = h.fwd(r);
            for (int j = 0; j < P && q + 1 + j < n; ++j) A[q][q + 1 + j] = f[P + 1 + j];
            A[q][n + q] = f[P];
        } else if (r < h.N) {
            const double *b = h.back(r);
            for (int j = 0; j <= P; ++j) A[q][q - j] = b[P + j];
            A[q][n + q] = 1.0;
        }
    }
    for (int k = 0; k < n; ++k) {
        int piv = k;
        for (int i = k + 1; i < n; ++i)
            if (std::fabs(A[i][k]) > std::fabs(A[piv][k])) piv = i;
        if (!(std::fabs(A[piv][k]) > 0)) return false;
        for (int c = 0; c < 2 * n; ++c) std::swap(A[k][c], A[piv][c]);
        for (int i = 0; i < n; ++i) {
            if (i == k) continue;
            const double f = A[i][k] / A[k][k];
            if (f != 0)
                for (int c = k; c < 2 * n; ++c) A[i][c] -= f * A[k][c];
        }
    }
    for (int j = 0; j < P; ++j)
        for (int i = 0; i < P; ++i) {
            py[j * P + i] = A[P + j][n + P - 1 - i] / A[P + j][P + j];   // y(e-i)
            pc[j * P + i] = A[P + j][n + P + i] / A[P + j][P + j];       // c(e+1+i)
        }
    return true;
}

// Canonical constants of an operator, as LineConst<P> lays them out.
static bool canonical(const LineHostOp &h, std::vector<double> &k)
{
    const int P = h.P, rc = h.N / 2;
    const double *f = h.fwd(rc), *b = h.back(rc);
    k.assign(f, f + 2 * P + 1);
    k.insert(k.end(), b, b + P);
    k.resize((size_t)(3 * P + 1) + 2 * P * P);
    return meet(h, rc, &k[3 * P + 1], &k[3 * P + 1 + P * P]);
}

// Line-per-lane solves of direction dir.  Used by the steps (out of place);
// iga_line_solve keeps the direction's windowed or exact schedule.
// IGA_EUNSUPPORTED if an operator decays too slowly for the compiled halo, has
// long edges, or the lines are shorter than 4p + 1.
static iga_status build_line(iga_plan *pl, int dir)
{
    const int N = dir ? pl->Ny : pl->Nx, P = pl->P, RS = 2 * P + 2, LROW = line_row_size(P);
    const LineShape sh = line_shape(pl);
    const double tol = std::ldexp(1.0, pl->fp32 ? -30 : -55);
    const int ntiles = (N + sh.own - 1) / sh.own;
    // the kernel looks D's rows up as the first 2P, the interior one and the last
    // 2P (LineBand), which are 4P + 1 different rows only from here on
    if (N < 4 * P + 1) return fail(IGA_EUNSUPPORTED, "lines too short for the line-per-lane solves");
    LineHostOp h[NOPS];
    int K0 = 0, NK = N;   // rows [K0, NK) are canonical in both factorisations of every operator
    std::vector<double> consts[NOPS];
    for (int op = 0; op < NOPS; ++op) {
        if (op_dir(op) != dir) continue;
        LineHostOp &q = h[op];
        q.o = &pl->op_host[op];
        q.N = N;
        q.P = P;
        q.rev = reversed_rows(pl->op_band[op], N, P);
        int b0, bn;
        interior_range(q.rev, N, 2 * P + 1, 1e-15, b0, bn);
        K0 = std::max(K0, std::max(q.o->K0, b0));
        NK = std::min(NK, std::min(q.o->NK, bn));
        // decay of the two eliminations: L downwards, V upwards
        std::vector<double> lv((size_t)N * RS, 0.0);
        for (int r = 0; r < N; ++r) {
            std::copy(q.fwd(r), q.fwd(r) + P, &lv[(size_t)r * RS]);
            std::copy(q.back(r), q.back(r) + P, &lv[(size_t)r * RS + P + 1]);
        }
        OpHost t;
        interior_range(lv, N, RS, 1e-15, t.K0, t.NK);
        t.rows = compress_rows(lv, N, RS, t.K0, t.NK);
        t.nrows = (int)(t.rows.size() / RS);
        if (compute_warmup(t, N, P, tol, sh.HL) <= 0 || !canonical(q, consts[op]))
            return fail(IGA_EUNSUPPORTED, "the operators decay too slowly for the line-per-lane halo");
    }
    // (the middle row is in every interior range: K0 <= N/2 < NK)
    const BandHost &bd = pl->band_host[dir ? BAND_BY : BAND_BX];
    const int nrows = K0 + 1 + (N - NK) + 1;   // edge rows, the canonical one, zeros
    if (nrows > 1024) return fail(IGA_EUNSUPPORTED, "the operators' edges are too long");
    // D's own rows are the first and last 2P
    if (dir && (bd.K0 > 2 * P || bd.NK < N - 2 * P)) return fail(IGA_EUNSUPPORTED, "no uniform interior");
    // tiles whose rows are all canonical and inside the line
    auto interior = [&](int t) {
        const int a = t * sh.own - sh.HL - P, e = (t + 1) * sh.own + sh.HL + P;
        return a >= K0 && e <= NK && a >= 2 * P && e <= N - 2 * P;
    };
    int lo = 0, hi = ntiles;
    while (lo < ntiles && !interior(lo)) ++lo;
    while (hi > lo && !interior(hi - 1)) --hi;
    const int nedge = lo + ntiles - hi;
    // one buffer for the direction's tables, each 16-byte aligned: edge rows and
    // meeting matrices of A and M, edge rows of D
    LineGeom geom{lo, hi, K0, NK, nrows, {0, 0, 0, 0, 0}};
    std::vector<double> all;
    auto add = [&](int which, const std::vector<double> &t) {
        all.resize((all.size() + 1) & ~size_t(1), 0.0);
        geom.off[which] = all.size();
        all.insert(all.end(), t.begin(), t.end());
    };
    for (int op = 0; op < NOPS; ++op) {
        if (op_dir(op) != dir) continue;
        const int first = (op == OP_MX || op == OP_MY) ? 2 : 0;
        std::vector<double> t((size_t)nrows * LROW, 0.0);
        auto put = [&](int i, int r) {
            const double *f = h[op].fwd(r), *b = h[op].back(r);
            std::copy(f, f + 2 * P + 1, &t[(size_t)i * LROW]);
            std::copy(b, b + P, &t[(size_t)i * LROW + 2 * P + 1]);
        };
        for (int r = 0; r <= K0; ++r) put(r, r);
        for (int r = NK; r < N; ++r) put(K0 + 1 + r - NK, r);
        add(first, t);
        t.assign((size_t)std::max(1, nedge) * sh.NW * 2 * P * P, 0.0);
        for (int i = 0; i < nedge; ++i)
            for (int w = 0; w < sh.NW; ++w) {
                const int tile = i < lo ? i : hi + (i - lo);
                double *p = &t[((size_t)i * sh.NW + w) * 2 * P * P];
                if (!meet(h[op], tile * sh.own + (w + 1) * LINE_MM - 1, p, p + P * P))
                    return fail(IGA_EUNSUPPORTED, "singular operator at a chunk's end");
            }
        add(first + 1, t);
    }
    if (dir) {
        const int LB = (2 * P + 2) & ~1;   // LineBand
        std::vector<double> t((size_t)(4 * P + 1) * LB, 0.0);
        for (int i = 0; i <= 4 * P; ++i) {
            const int r = i < 2 * P ? i : i == 2 * P ? N / 2 : N - 4 * P - 1 + i;
            const double *row = &bd.rows[(size_t)row_of(r, bd.K0, bd.NK, bd.nrows) * RS];
            std::copy(row, row + 2 * P + 1, &t[(size_t)i * LB]);
        }
        add(4, t);
    }
    DevBuf tab;   // moved into the plan when it is on the device
    IGA_HIP(tab.alloc(all.size() * sizeof(double)));
    IGA_HIP(hipMemcpy(tab.ptr, all.data(), all.size() * sizeof(double), hipMemcpyHostToDevice));
    // the sweeps write a second pair of right-hand sides
    if (!pl->scratch_r2.ptr) {
        DevBuf r2, rf2;
        IGA_HIP(r2.alloc(pl->ndof * pl->wsize));
        IGA_HIP(rf2.alloc(pl->ndof * pl->wsize));
        pl->scratch_r2 = std::move(r2);
        pl->scratch_rf2 = std::move(rf2);
    }
    for (int band = 0; band <= dir; ++band)
        for (int batch = 0; batch < 2; ++batch)
            IGA_HIP(hipFuncSetAttribute(pick_line(pl, dir == 1, band != 0, batch != 0),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    for (int op = 0; op < NOPS; ++op)
        if (op_dir(op) == dir) pl->line_const[op] = std::move(consts[op]);
    if (dir) {
        const double *row = &bd.rows[(size_t)row_of(N / 2, bd.K0, bd.NK, bd.nrows) * RS];
        pl->line_d.assign(row, row + 2 * P + 1);
    }
    pl->line_tab[dir] = std::move(tab);
    pl->line_geom[dir] = geom;
    return IGA_OK;
}

// The tables depend on the operators alone: built once after a factorisation,
// whatever schedules come and go beneath (ensembles and the autotuners lay the
// solves over one schedule after another).
iga_status choose_line_schedule(iga_plan *pl, int dir)
{
    int &state = pl->line_state[dir];
    if (state < 0) return fail(IGA_EUNSUPPORTED, "no line-per-lane solves for these operators");
    if (!state) {
        const iga_status st = build_line(pl, dir);
        if (st == IGA_EUNSUPPORTED) state = -1;
        if (st) return st;
        state = 1;
    }
    pl->sched[dir].line = 1;
    return IGA_OK;
}

// out of place: single solves (along y with a base field or not), or, alone in
// its launch, Strang's middle substep along y
bool line_jobs_ok(const iga_plan *pl, int dir, const SweepJob *jobs, int njobs)
{
    if (!pl->sched[dir].line || njobs < 1 || njobs > LMAXJOBS) return false;
    for (int i = 0; i < njobs; ++i) {
        const SweepJob &j = jobs[i];
        if (j.src == j.dst || (dir == 0 && j.base)) return false;
        const bool single = j.op0 >= 0 && op_dir(j.op0) == dir && j.band < 0 && j.op1 < 0;
        const bool middle = dir == 1 && njobs == 1 && j.op0 < 0 && j.band == BAND_BY && j.op1 == OP_AY &&
                            !j.base && j.add_after;
        if (!single && !middle) return false;
    }
    return true;
}

// parameters of a launch
struct LineLaunch {
    const void *fn = nullptr;
    int blocks = 0, block = 0;
    size_t lds = 0;
};
template <int P>
static LineLaunch fill(const iga_plan *pl, int dir, const SweepJob *jobs, int njobs, LineParams<P> &prm, bool batch)
{
    static_assert(sizeof(LineConst<P>) == (3 * P + 1 + 2 * P * P) * sizeof(double), "LineConst layout");
    const LineShape sh = line_shape(pl);
    const LineGeom &g = pl->line_geom[dir];
    const bool band = jobs[0].op0 < 0;
    std::memset(&prm, 0, sizeof prm);
    for (int i = 0; i < njobs; ++i) {
        const SweepJob &j = jobs[i];
        LineJob<P> &q = prm.jobs[i];
        const int op = band ? j.op1 : j.op0;
        q.src = j.src;
        q.base = j.base;
        q.dst = j.dst;
        q.zero_skip = j.zero_skip && j.base && j.base == j.dst;
        std::memcpy(&q.a.k, pl->line_const[op].data(), sizeof q.a.k);
        const double *tab = pl->line_tab[dir].as<double>();
        const int first = (op == OP_MX || op == OP_MY) ? 2 : 0;
        q.a.rows = tab + g.off[first];
        q.a.meet = tab + g.off[first + 1];
        if (band) {
            std::memcpy(q.d, pl->line_d.data(), sizeof q.d);
            q.dend = tab + g.off[4];
        }
    }
    prm.N = dir ? pl->Ny : pl->Nx;
    prm.nlines = dir ? pl->Nx : pl->Ny;
    prm.ld = pl->Ny;
    prm.ntiles = (prm.N + sh.own - 1) / sh.own;
    prm.lo = g.lo;
    prm.hi = g.hi;
    prm.K0 = g.K0;
    prm.NK = g.NK;
    prm.nrows = g.nrows;
    prm.njobs = njobs;
    return LineLaunch{pick_line(pl, dir == 1, band, batch), (prm.nlines + 63) / 64 * prm.ntiles, sh.NW * 64,
                      (size_t)sh.lds[band]};
}

template <int P>
static iga_status launch_p(const iga_plan *pl, int dir, const SweepJob *jobs, int njobs, hipStream_t s)
{
    LineParams<P> prm;
    const LineLaunch q = fill<P>(pl, dir, jobs, njobs, prm, false);
    void *args[] = {&prm};
    IGA_HIP(hipLaunchKernel(q.fn, dim3(q.blocks, njobs), dim3(q.block), args, q.lds, s));
    return IGA_OK;
}

iga_status launch_line(const iga_plan *pl, int dir, const SweepJob *jobs, int njobs, hipStream_t s)
{
    if (pl->P == 1) return launch_p<1>(pl, dir, jobs, njobs, s);
    if (pl->P == 2) return launch_p<2>(pl, dir, jobs, njobs, s);
    return launch_p<3>(pl, dir, jobs, njobs, s);
}

// one batched launch over the members listed in `who`
template <int P>
static iga_status batch_p(const std::vector<iga_plan *> &pls, const std::vector<int> &who, int dir,
                          const std::vector<std::vector<SweepJob>> &jobs, BatchLaunch &out)
{
    std::vector<LineParams<P>> prms(who.size());
    std::vector<int4> info;
    int maxjobs = 1;
    for (size_t i = 0; i < who.size(); ++i) {
        const std::vector<SweepJob> &j = jobs[who[i]];
        const LineLaunch q = fill<P>(pls[who[i]], dir, j.data(), (int)j.size(), prms[i], true);
        for (int b = 0; b < q.blocks; ++b) info.push_back(int4{(int)i, b, q.blocks, 0});
        maxjobs = std::max(maxjobs, (int)j.size());
        out.fn = q.fn;
        out.block = q.block;
        out.lds = q.lds;
    }
    out.nblk = (int)info.size();
    out.njobs = maxjobs;
    IGA_HIP(out.prm.alloc(prms.size() * sizeof prms[0]));
    IGA_HIP(out.info.alloc(info.size() * sizeof info[0]));
    IGA_HIP(hipMemcpy(out.prm.ptr, prms.data(), prms.size() * sizeof prms[0], hipMemcpyHostToDevice));
    IGA_HIP(hipMemcpy(out.info.ptr, info.data(), info.size() * sizeof info[0], hipMemcpyHostToDevice));
    return IGA_OK;
}

iga_status build_line_batch(const std::vector<iga_plan *> &pls, const std::vector<int> &who, int dir,
                            const std::vector<std::vector<SweepJob>> &jobs, BatchLaunch &out)
{
    const int P = pls[who[0]]->P;
    if (P == 1) return batch_p<1>(pls, who, dir, jobs, out);
    if (P == 2) return batch_p<2>(pls, who, dir, jobs, out);
    return batch_p<3>(pls, who, dir, jobs, out);
}

}  // namespace iga
