// sweep_line.h -- line solves with one line per lane.
//
// Section 4's directional solves are independent banded systems per line.  Here
// a workgroup owns 64 lines, one per lane, and NW chunks of MM rows of them, one
// per wavefront.  All lanes stand on the same row, so the factor coefficients
// are wavefront-uniform: none is held per lane, and away from the line ends all
// are scalar constants of the operator.
//
// Twisted elimination.  Forward elimination (A = L U) is restarted from a zero
// state HL rows before the chunk and run to the chunk's end; the HL rows after
// the chunk are eliminated backwards, with the reversed factorisation
// (A = V W, V unit upper), also from a zero state.  Both recurrences contract
// geometrically, so the restarts change the result by less than 2^-55 of the
// state (double) or 2^-30 (float; the plan checks its operators).  The two
// states meet behind the chunk: the P unknowns there follow from P forward and
// P backward states (constant P x P matrices), and back substitution runs over
// the chunk alone.  Each halo row so costs P multiply-adds and nothing is kept
// of it.
//
// All arithmetic is in double, for float state too: the fields are read and
// written in float, and the result is the double solve of the float data,
// rounded once; a base field is then added in float, as the other solves do.
// (An FP32 solve refined once with a double residual, which this replaces in the
// steps, costs four substitutions for two and does not get nearer: the vector
// units do double multiply-adds at the rate of unpacked float ones.)
//
// Strang's middle substep, T** = A^{-1} B T* = T* + A^{-1} D T* with D = B - A, is
// the same solve with D T* formed from the tile as it is read (BAND), in a
// launch of its own: fused with the solve before it (as T + A^{-1} (2 R + D T) -
// M^{-1} R, two operators over two tiles) it took 22 us at 1024^2 and 107 us at
// 4096^2 in FP32, 313 us in double, for lack of registers and LDS for a second
// workgroup; the two launches take 10 + 12, 55 + 44 and 118 + 102 us.
//
// Data.  The rows of the workgroup's chunks and their halos are a tile in LDS,
// filled by DMA (every load in flight at once, no registers): x-lines row by
// row, y-lines as the runs of consecutive columns they are in memory, which is
// where they are transposed.  The wavefronts share the tile, so the halo rows of
// neighbouring chunks are loaded once.  Results of y-lines go back through
// the tile to be written as runs.  (Read by each lane
// from its own line instead, 16 bytes at a time, y-lines were bound by the
// vector cache: 64 lines an instruction, 102 us for the fused 4096^2 job.)
//
// Bound by latency on small meshes (1024^2: 289 workgroups, about one per
// compute unit: fill, eliminate, write), by memory on large ones.  Against the
// windowed and chunk-scan solves in the steps: 4096^2 FP32, x 50 -> 36 us (one
// field; 3.7 TB/s of the 4.7 a copy reaches), y 104-113 -> 65 us (T with the
// fuel's zero check); double, x 270 -> 77, y 196 -> 115 (T alone); cubic 1500^2
// double x 119 -> 20, y 111 -> 21; 64^2 double x 11.8 -> 6.9, y 11.2 -> 8.4.
#pragma once
#include "sweep_kernels.h"

namespace iga {

// halo rows
template <typename T, int P> struct LineHalo;
template <> struct LineHalo<float, 1> { static constexpr int value = 20; };
template <> struct LineHalo<float, 2> { static constexpr int value = 28; };
template <> struct LineHalo<float, 3> { static constexpr int value = 40; };
template <> struct LineHalo<double, 1> { static constexpr int value = 32; };
template <> struct LineHalo<double, 2> { static constexpr int value = 48; };
template <> struct LineHalo<double, 3> { static constexpr int value = 72; };

// Wavefronts (chunks of MM rows) per workgroup.  Other workgroups beside it in
// LDS load while it solves: five, four and three share a compute unit in float
// (29, 35, 43 KB), two in double for p <= 2 (67, 77 KB).  For p = 3 in double no
// number of wavefronts leaves room for a second one (the halo rows alone take
// 72 KB); six share the halos of one workgroup (131 KB).
constexpr int LINE_MM = 16;
template <typename T, int P> struct LineWaves;
template <> struct LineWaves<float, 1> { static constexpr int value = 4; };
template <> struct LineWaves<float, 2> { static constexpr int value = 4; };
template <> struct LineWaves<float, 3> { static constexpr int value = 4; };
template <> struct LineWaves<double, 1> { static constexpr int value = 4; };
template <> struct LineWaves<double, 2> { static constexpr int value = 3; };
template <> struct LineWaves<double, 3> { static constexpr int value = 6; };

// Tile: the rows of NW chunks and their halos, with PD = P more rows on each side
// for the band D (BAND).  y-lines take an odd row stride, so that the lanes'
// elements of one row lie in different banks.
template <typename T, int P, bool BAND> struct LineTile {
    static constexpr int HL = LineHalo<T, P>::value, NW = LineWaves<T, P>::value;
    static constexpr int OWN = NW * LINE_MM;
    static constexpr int PD = BAND ? P : 0, ROWS = OWN + 2 * (HL + PD), LD = ROWS | 1;
    static constexpr int BYTES = (64 * LD * (int)sizeof(T) + 15) & ~15;
};

// Coefficients of one operator: of the canonical interior, and per row for
// workgroups whose tile leaves it.  A row of the table holds L(r, r-1-j) (P),
// 1/U(r,r), U(r, r+1+j)/U(r,r) (P), V(r, r+1+j) (P), padded to LROW; line rows
// [0, K0) and [NK, N) have their own, the others share row K0, the last row
// (zeros) stands for rows outside the line.  py, pc (P x P each, per edge chunk):
//   x(e+1+j) = sum_i py[j][i] y(e-i) + pc[j][i] c(e+1+i)
// with e the chunk's last row, y the forward and c the backward states.
template <int P> struct LineConst {
    double l[P], ui, u[P], v[P], py[P][P], pc[P][P];
};
template <int P> struct LineRow {
    static constexpr int value = (3 * P + 2) & ~1;   // even: 16-byte reads
};

template <int P> struct LineBand {
    static constexpr int value = (2 * P + 2) & ~1, N = (4 * P + 1) * value;   // LBAND, table size
};

template <int P> struct LineOp {
    LineConst<P> k;
    const double *rows, *meet;   // edge rows [nrows][LROW], py and pc of each edge chunk
};
template <int P> struct LineJob {
    const void *src, *base;   // base: y-lines, not BAND; or NULL
    void *dst;
    int zero_skip;   // y-lines with dst == base: an all-zero window is left alone
    LineOp<P> a;
    double d[2 * P + 1];   // BAND: canonical row of D,
    const double *dend;    // and [4P+1][LBAND]: its rows [0, 2P), that one, [N-2P, N)
};
constexpr int LMAXJOBS = 2;
template <int P> struct LineParams {
    LineJob<P> jobs[LMAXJOBS];
    int N, nlines;      // rows per line, lines
    int ld;             // row stride of the field (Ny)
    int ntiles;         // tiles per line (of LineTile::OWN rows)
    int lo, hi;         // tiles [0, lo) and [hi, ntiles) use the edge tables
    int K0, NK, nrows;  // edge rows
    int njobs;
};

using LineTab = const __attribute__((address_space(4))) double *;

// Edge tables of one operator in LDS, in the order the passes use them, so that
// a wavefront reads them at compile-time offsets from its own base:
//   L(r, r-1-j) (P) of rows R0 - HL .. R0 + OWN - 1
//   1/U(r,r), U(r, r+1+j)/U(r,r) (P+1) of rows R0 .. R0 + OWN - 1
//   V(r, r+1+j) (P) of rows R0 .. R0 + OWN + HL - 1
template <typename T, int P> struct LineEdge {
    using S = LineTile<T, P, false>;
    static constexpr int L = 0, U = L + (S::HL + S::OWN) * P, V = U + S::OWN * (P + 1),
                         N = (V + (S::OWN + S::HL) * P + 1) & ~1;
};
template <typename T, int P>
__device__ __forceinline__ void line_edges(double *tab, const double *rows, int R0, int N, int K0, int NK, int nrows)
{
    using E = LineEdge<T, P>;
    constexpr int HL = E::S::HL;
    // all loads, then all stores: one latency, not one per round (a 64^2 FP64
    // x sweep 7.2 -> 6.9 us)
    constexpr int NT = E::S::NW * 64, IT = (E::N + NT - 1) / NT;
    double v[IT];
#pragma unroll
    for (int n = 0; n < IT; ++n) {
        const int i = min(n * NT + (int)threadIdx.x, E::N - 1);
        int r, c;
        if (i < E::U) {
            r = R0 - HL + i / P;
            c = i % P;
        } else if (i < E::V) {
            r = R0 + (i - E::U) / (P + 1);
            c = P + (i - E::U) % (P + 1);
        } else {
            r = R0 + (i - E::V) / P;
            c = 2 * P + 1 + (i - E::V) % P;
        }
        const int k = r < 0 || r >= N ? nrows - 1 : min(r, K0) + max(0, r - NK + 1);
        v[n] = rows[k * LineRow<P>::value + c];
    }
#pragma unroll
    for (int n = 0; n < IT; ++n) {
        const int i = n * NT + (int)threadIdx.x;
        if (i < E::N) tab[i] = v[n];
    }
}

// Nothing moves across every K-th row: bounds what is read ahead from LDS, and
// so the registers.
template <int K> __device__ __forceinline__ void line_fence(int i)
{
    if ((i + 1) % K == 0) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    }
}

// One operator's elimination.  EDGE: l, u, v point at this wavefront's rows of
// the edge tables (l at its lower halo's first row, u at its chunk's, v at the
// row after its chunk), otherwise all rows are canonical.
template <int P, int HL, int MM, bool EDGE> struct LineSolve {
    const LineConst<P> &k;
    const double *l, *u, *v;
    double s[P], c[P], y[MM];

    __device__ __forceinline__ LineSolve(const LineConst<P> &k_, const double *l_, const double *u_, const double *v_)
        : k(k_), l(l_), u(u_), v(v_)
    {
        clear();
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j < P; ++j) s[j] = c[j] = 0.0;
    }
    // forward elimination of row i, counted from the lower halo's first
    __device__ __forceinline__ double fwd(double b, int i)
    {
#pragma unroll
        for (int j = P - 1; j >= 0; --j) b -= (EDGE ? l[i * P + j] : k.l[j]) * s[j];
#pragma unroll
        for (int j = P - 1; j > 0; --j) s[j] = s[j - 1];
        return s[0] = b;
    }
    // backward elimination of row i after the chunk
    __device__ __forceinline__ void back(double b, int i)
    {
#pragma unroll
        for (int j = P - 1; j >= 0; --j) b -= (EDGE ? v[i * P + j] : k.v[j]) * c[j];
#pragma unroll
        for (int j = P - 1; j > 0; --j) c[j] = c[j - 1];
        c[0] = b;
    }
    // the states are formed here, not where they are used next
    __device__ __forceinline__ void pin()
    {
#pragma unroll
        for (int j = 0; j < P; ++j) asm volatile("" : "+v"(s[j]), "+v"(c[j]));
    }
    // the chunk's solution, from its forward values y and the states at its
    // end, into y; meet: py, pc of an edge chunk
    __device__ __forceinline__ void finish(LineTab meet)
    {
        double x[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            x[j] = 0.0;
#pragma unroll
            for (int i = 0; i < P; ++i) {
                x[j] += (EDGE ? meet[j * P + i] : k.py[j][i]) * s[i];
                x[j] += (EDGE ? meet[P * P + j * P + i] : k.pc[j][i]) * c[i];
            }
        }
#pragma unroll
        for (int i = MM - 1; i >= 0; --i) {
            const double *t = u + i * (P + 1);
            double z = y[i] * (EDGE ? t[0] : k.ui);
#pragma unroll
            for (int j = P - 1; j >= 0; --j) z -= (EDGE ? t[1 + j] : k.u[j]) * x[j];
#pragma unroll
            for (int j = P - 1; j > 0; --j) x[j] = x[j - 1];
            x[0] = z;
            y[i] = z;
            if (EDGE && i % 8 == 0) {
                asm volatile("" : "+v"(x[0]));
                line_fence<1>(0);
            }
        }
    }
};

// Fill the tile with rows [row0, row0 + ROWS) of the workgroup's lines, lines
// clamped into the field and (EDGE) rows into the line: x-lines [row][64],
// y-lines [64][LD].  An instruction moves 64 words from a uniform address plus
// a per-lane offset that no instruction changes (of a row of 64 x-lines, of one
// y-line's run of columns), so that issuing it costs a few scalar operations.
// The data are visible after the next barrier.
template <typename T, int ROWS, int LD, int NW, bool DIRY, bool EDGE>
__device__ __forceinline__ void line_fill(T *tile, const T *src, int line0, int nlines, int row0, int N, int ld)
{
    typedef __attribute__((address_space(1))) const void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    constexpr int D = sizeof(T) / 4;   // words per element
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const char *g = reinterpret_cast<const char *>(src);
    unsigned *l = reinterpret_cast<unsigned *>(tile);
    if constexpr (!DIRY) {
        unsigned off[D];
#pragma unroll
        for (int h = 0; h < D; ++h) off[h] = min(h * 64 + lane, (unsigned)(min(64, nlines - line0) * D - 1)) * 4u;
        const size_t ldb = (size_t)ld * sizeof(T);
        g += (size_t)line0 * sizeof(T);
        const char *p = g + (ptrdiff_t)(row0 + wave) * (ptrdiff_t)ldb;
        const size_t step = NW * ldb;
#pragma unroll 4
        for (int k = wave; k < ROWS; k += NW, p += step) {
            if (EDGE) p = g + (size_t)min(max(row0 + k, 0), N - 1) * ldb;
#pragma unroll
            for (int h = 0; h < D; ++h)
                __builtin_amdgcn_global_load_lds((gvoid *)(p + off[h]), (lvoid *)(l + (k * D + h) * 64), 4, 0, 0);
        }
    } else {
        constexpr int NP = (ROWS * D + 63) / 64;   // pieces of a line
        unsigned off[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int w = j * 64 + (int)lane;
            off[j] = EDGE ? (unsigned)(min(max(row0 + w / D, 0), N - 1) * D + (D == 2 ? w & 1 : 0)) * 4u
                          : (unsigned)w * 4u;
        }
        const size_t ldb = (size_t)ld * sizeof(T);
        if (!EDGE) g += (ptrdiff_t)row0 * (ptrdiff_t)sizeof(T);
        const char *p = g + (size_t)min(line0 + wave, nlines - 1) * ldb;
        const size_t step = NW * ldb;
#pragma unroll 2
        for (int k = wave; k < 64; k += NW) {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                lvoid *to = (lvoid *)(l + k * LD * D + j * 64);
                if ((j + 1) * 64 <= ROWS * D || (int)lane < ROWS * D - j * 64)
                    __builtin_amdgcn_global_load_lds((gvoid *)(p + off[j]), to, 4, 0, 0);
            }
            if (line0 + k + NW < nlines) p += step;   // lines past the last repeat one
        }
    }
}

__device__ __forceinline__ unsigned line_bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ unsigned line_bits(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (unsigned)b | (unsigned)(b >> 32);
}

template <typename T, int P, bool DIRY, bool BAND, bool EDGE>
__device__ __forceinline__ void line_tile(const LineParams<P> &prm, const LineJob<P> &job, T *tile, double *tab,
                                          int line0, int tidx, int edge)
{
    using S = LineTile<T, P, BAND>;
    using E = LineEdge<T, P>;
    constexpr int HL = S::HL, PD = S::PD, NW = S::NW, MM = LINE_MM, W = 2 * P + 1, K = EDGE ? (BAND ? 4 : 8) : 16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = prm.N, ld = prm.ld;
    const int R0 = tidx * S::OWN;       // first own row of the tile
    const int r0 = R0 + wave * MM;      // this wavefront's chunk
    line_fill<T, S::ROWS, S::LD, NW, DIRY, EDGE>(tile, static_cast<const T *>(job.src), line0, prm.nlines,
                                                 R0 - HL - PD, N, ld);
    if constexpr (EDGE) line_edges<T, P>(tab, job.a.rows, R0, N, prm.K0, prm.NK, prm.nrows);
    double *dtab = tab + E::N;   // D's edge rows
    if constexpr (EDGE && BAND) {
        for (int i = threadIdx.x; i < LineBand<P>::N; i += NW * 64) dtab[i] = job.dend[i];
    }
    // results of y-lines are written as runs of MM columns, LPI lines per
    // instruction: lane -> (line, column) of the wavefront's block
    constexpr int LPI = 64 / MM;
    const int sl = lane / MM, sc = lane % MM;
    const int col = r0 + sc;
    const unsigned vo = ((unsigned)sl * (unsigned)ld + (unsigned)col) * (unsigned)sizeof(T);
    auto at_store = [&](const void *f, int k) {
        return reinterpret_cast<T *>(const_cast<char *>(static_cast<const char *>(f)) +
                                     (size_t)(line0 + k * LPI) * ld * sizeof(T) + vo);
    };
    auto ok = [&](int k) { return (!EDGE || col < N) && line0 + k * LPI + sl < prm.nlines; };
    // the base field's values in the order of the stores: by edge tiles (all there
    // is on small meshes, where a launch is one chain of latencies) requested with
    // the tile, by interior ones before the back substitution (with the tile they
    // cost more than they hid: 4096^2 FP32 68 -> 75 us for the T and fuel jobs).
    // y-lines of 64^2 FP64 10.3 -> 8.7 us, 1024^2 FP64 12.9 -> 11.2
    T bs[MM];
    auto request = [&](bool want) {
        if constexpr (DIRY && !BAND) {
#pragma unroll
            for (int k = 0; k < MM; ++k) bs[k] = want && ok(k) ? *at_store(job.base, k) : T(0);
        }
    };
    if (EDGE) request(job.base);
    __syncthreads();
    // tile row wave*MM + i (line row r0 - HL - PD + i) of this lane's line
    const int tb = DIRY ? lane * S::LD + wave * MM : wave * MM * 64 + lane;
    constexpr int ts = DIRY ? 1 : 64;
    auto at = [&](int i) -> T { return tile[tb + i * ts]; };
    const LineTab meet = (LineTab)job.a.meet + (size_t)(EDGE ? edge * NW + wave : 0) * 2 * P * P;
    LineSolve<P, HL, MM, EDGE> a(job.a.k, tab + E::L + wave * MM * P, tab + E::U + wave * MM * (P + 1),
                                 tab + E::V + (wave + 1) * MM * P);
    unsigned nz = 0;
    double w[W];   // BAND: the field at rows r - P .. r + P of the current row r
    auto dband = [&](int r) {
        const double *t = job.d;
        if constexpr (EDGE)
            t = dtab + (min(max(r, 0), 2 * P) + max(0, min(r, N - 1) - (N - 2 * P) + 1)) * LineBand<P>::value;
        double q = 0.0;
#pragma unroll
        for (int j = 0; j < W; ++j) q += (EDGE ? t[j] : job.d[j]) * w[j];
        return q;
    };
    auto pin = [&] {
        a.pin();
        if (DIRY && !BAND) asm volatile("" : "+v"(nz));
    };
    // forward over the lower halo and the chunk
    if constexpr (BAND) {
#pragma unroll
        for (int j = 0; j < W - 1; ++j) w[j + 1] = (double)at(j);
    }
#pragma unroll
    for (int i = 0; i < HL + MM; ++i) {
        double b;
        if constexpr (BAND) {
#pragma unroll
            for (int j = 0; j < W - 1; ++j) w[j] = w[j + 1];
            w[W - 1] = (double)at(i + 2 * P);
            b = dband(r0 - HL + i);
        } else {
            const T v = at(i);
            if (DIRY) nz |= line_bits(v);
            b = (double)v;
        }
        const double y = a.fwd(b, i);
        if (i >= HL) a.y[i - HL] = y;
        if (i % K == K - 1) pin();
        line_fence<K>(i);
    }
    // backward over the upper halo
    if constexpr (BAND) {
#pragma unroll
        for (int j = 0; j < W - 1; ++j) w[j] = (double)at(MM + 2 * HL + j);
    }
#pragma unroll
    for (int i = HL - 1; i >= 0; --i) {
        double b;
        if constexpr (BAND) {
#pragma unroll
            for (int j = W - 1; j > 0; --j) w[j] = w[j - 1];
            w[0] = (double)at(HL + MM + i);
            b = dband(r0 + MM + i);
        } else {
            const T v = at(HL + MM + i);
            if (DIRY) nz |= line_bits(v);
            b = (double)v;
        }
        a.back(b, i);
        if (i % K == 0) {
            pin();
            line_fence<1>(0);
        }
    }
    if constexpr (BAND) {
        a.finish(meet);
#pragma unroll
        for (int i = 0; i < MM; ++i) a.y[i] += (double)at(P + HL + i);
    }
    if constexpr (!DIRY) {
        if (!BAND) a.finish(meet);
        T *d = static_cast<T *>(job.dst) + line0 + lane;
        if (line0 + lane < prm.nlines) {
#pragma unroll
            for (int i = 0; i < MM; ++i)
                if (!EDGE || r0 + i < N) d[(size_t)(r0 + i) * ld] = (T)a.y[i];
        }
    } else {
        // the solve of zero data is exactly zero, and dst == base holds its sum
        const bool skip = !BAND && job.zero_skip && !__any(nz != 0);
        if (!EDGE) request(job.base && !skip);
        if (!BAND) a.finish(meet);
        __syncthreads();   // every wavefront has read its rows of the tile
        if (skip) return;
        constexpr int LB = MM | 1;
        T *blk = tile + wave * 64 * LB;
#pragma unroll
        for (int i = 0; i < MM; ++i) blk[lane * LB + i] = (T)a.y[i];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < MM; ++k) {
            const T v = blk[(k * LPI + sl) * LB + sc] + (BAND ? T(0) : bs[k]);
            if (ok(k)) *at_store(job.dst, k) = v;
        }
    }
}

// One workgroup: block blk of job jobi.  Edge tiles take the first blocks (they
// take longest); the interior tiles follow, consecutive tiles of 64 lines on
// one XCD.
template <typename T, int P, bool DIRY, bool BAND>
__device__ __forceinline__ void line_body(const LineParams<P> &prm, int blk, int nblk, int jobi)
{
    extern __shared__ __align__(16) unsigned char smem[];
    T *tile = reinterpret_cast<T *>(smem);
    double *tab = reinterpret_cast<double *>(smem + LineTile<T, P, BAND>::BYTES);
    const int ngrp = (prm.nlines + 63) / 64;
    const int nedge = prm.lo + prm.ntiles - prm.hi, nint = prm.hi - prm.lo;
    const int e0 = ngrp * nedge;
    const LineJob<P> &job = prm.jobs[jobi];
    if (blk < e0) {
        const int grp = blk / nedge, edge = blk - grp * nedge;
        const int t = edge < prm.lo ? edge : prm.hi + (edge - prm.lo);
        line_tile<T, P, DIRY, BAND, true>(prm, job, tile, tab, grp * 64, t, edge);
    } else {
        const int b = xcd_remap(blk - e0, nblk - e0);
        const int grp = b / nint;
        line_tile<T, P, DIRY, BAND, false>(prm, job, tile, tab, grp * 64, prm.lo + (b - grp * nint), 0);
    }
}

template <typename T, int P, bool DIRY, bool BAND>
__global__ __launch_bounds__((LineWaves<T, P>::value * 64)) void k_line(LineParams<P> prm)
{
    line_body<T, P, DIRY, BAND>(prm, blockIdx.x, gridDim.x, blockIdx.y);
}

// ensembles: block b is block info[b].y of member info[b].x, whose launch
// alone would have info[b].z blocks
template <typename T, int P, bool DIRY, bool BAND>
__global__ __launch_bounds__((LineWaves<T, P>::value * 64)) void k_line_batch(
    const LineParams<P> *__restrict__ prms, const int4 *__restrict__ info)
{
    const int4 bi = info[blockIdx.x];
    const LineParams<P> &prm = prms[bi.x];
    if ((int)blockIdx.y >= prm.njobs) return;
    line_body<T, P, DIRY, BAND>(prm, bi.y, bi.z, blockIdx.y);
}

// the compiled kernel (BAND: y-lines only)
template <typename T, int P> static const void *line_kernel(bool diry, bool band, bool batch)
{
    if (!diry)
        return batch ? reinterpret_cast<const void *>(k_line_batch<T, P, false, false>)
                     : reinterpret_cast<const void *>(k_line<T, P, false, false>);
    if (!band)
        return batch ? reinterpret_cast<const void *>(k_line_batch<T, P, true, false>)
                     : reinterpret_cast<const void *>(k_line<T, P, true, false>);
    return batch ? reinterpret_cast<const void *>(k_line_batch<T, P, true, true>)
                 : reinterpret_cast<const void *>(k_line<T, P, true, true>);
}

// one translation unit per precision and degree
const void *line_kernel_f1(bool diry, bool band, bool batch);
const void *line_kernel_f2(bool diry, bool band, bool batch);
const void *line_kernel_f3(bool diry, bool band, bool batch);
const void *line_kernel_d1(bool diry, bool band, bool batch);
const void *line_kernel_d2(bool diry, bool band, bool batch);
const void *line_kernel_d3(bool diry, bool band, bool batch);

}  // namespace iga
