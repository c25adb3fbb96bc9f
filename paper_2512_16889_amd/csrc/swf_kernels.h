// Kernel templates of the SWF solver (included by the per-size instantiation
// files and by swf_reduce.hip).
//
// One RK4 stage of the scattered-wave equation (eq. (scatDirac) of arXiv
// 2512.16889 multiplied by gamma^0),
//     k = IFFT[-i H0(k) FFT y_i] - i (A_0 + alpha^j A_j)(t_i) (y_i + psi_b(t_i)),
// H0(k) = alpha.k + beta.  Spectral derivatives along different axes commute,
// so the kinetic term is a sum over axes,
//     IFFT[-i H0 FFT y] = -i sum_j alpha^j D_j y - i beta y,
//     D_j y = IFFT_j[k_j FFT_j y]   (a one-dimensional transform along axis j),
// and in the Dirac representation every alpha^j is a signed permutation of
// the four components: (alpha^1 y)_q = y_{3-q}, (alpha^2 y)_q = -+i y_{3-q}
// (- for even q), (alpha^3 y)_q = +-y_{q^2} (+ for q = 0, 2).  A stage is
// therefore split into passes over the spinor-of-arrays state that never mix
// components inside a transform:
//   * column passes (axes y, z): one component per block; D_j of the component
//     alpha^j takes, written (y) or added (z) into the G buffer at the
//     component it lands on, G = alpha^2 D_y y + alpha^3 D_z y;
//   * one row pass (axis x): D_x of the component alpha^1 takes, then the
//     stage epilogue (beta and trivial-axis terms, the source, the RK4
//     update, the absorber) for the thread's own component.
// Per RK4 step this reads and writes 36 state arrays in 3D (24 in 2D, 12 in
// 1D).  The other row and column kernels (forward / inverse transforms of a
// whole state, the full right-hand side) serve the t_in observables, the
// operator test hook and the Breit-Wheeler partial-integration route.
#pragma once
#include "swf_dev.h"

namespace swf {

// Row-pass modes.
// ROW_SRC writes the source term -i V(t) (y + psi_b(t)) of the RK4 stage
// `stage` alone, in x space (no transform).
enum { ROW_FWD = 0, ROW_STAGE = 1, ROW_INV = 2, ROW_RHS = 3, ROW_FWDPH = 4, ROW_SRC = 5, ROW_NMODES = 6 };
// Column-pass modes.
enum { COL_FWD = 0, COL_INV = 1, COL_H0 = 2 };

struct PassArgs {
    const SolveDev* solves;
    const TermDev* terms;
    const void* rtab;      // real tables (field profiles, masks)
    const void* ctab;      // complex tables (phases, twiddles)
    const int2* items;     // (solve, tile) per block
    const int* step;       // device step counter
    double t_out, dt;
    int stage;             // RK4 stage 0..3 (ROW_STAGE, ROW_SRC)
    int src, dst;          // buffer roles
    int h0row;             // 1: the row pass also applies -i H0 / N (dim == 1)
    int expo;              // 1: the k-space multiply (COL_H0, h0row) is exp(-i H0 tau) / N instead
    double tau;            //    of -i H0 / N: the free evolution over tau (interaction picture)
    double t_explicit;     // time of ROW_RHS
    long long ph2;         // ROW_FWDPH: complex offset of exp(i k_j x_j) tables
    int nitems;            // work items of this launch
    int rev;               // stepping passes: the items in reverse order
    int step_add;          // steps enqueued since the device counter was last advanced
    const void* consts;    // StageConst per solve and stage of the current step (nst each)
    int nst;               // stages of the stepper
    int nsteps;            // line_kernel: RK4 steps per launch
};

// ------------------------------------------------------------------ tile variants
// A stepping column pass is instantiated for several tile widths (W adjacent
// x-columns per block, T threads per line); the host times them on the actual
// problem (autotuner) and keeps the fastest.
template <int N, int T, class P = FftPlan<N>> constexpr bool plan_ok() {
    if (T < 1 || N % T) return false;
    for (int j = 0; j < P::NR; ++j)
        if ((N / P::R[j]) % T || (N / T) % P::R[j]) return false;
    return true;
}
constexpr int NVAR = 3;       // tile variants of the stepping column passes
constexpr int imax(int a, int b) { return a > b ? a : b; }
constexpr int imin(int a, int b) { return a < b ? a : b; }

// Tile of the row kernel (inverse along the only axis, right-hand side, source):
// the default plan, T threads per x-line, up to 256 threads per block.
template <class R, int N> struct RowVar {
    using PL = FftPlan<N>;
    static constexpr int T = PL::T;
    static constexpr int ROWS = imax(1, 256 / T);
    static constexpr int THREADS = T * ROWS;
    using Lay = RowLay<N>;
    static constexpr size_t BYTES = (size_t)ROWS * Lay::STRIDE * sizeof(cpx<R>);
    static_assert(plan_ok<N, T, PL>(), "row tile violates the FFT plan constraints");
};

// Tile of the last-axis pass with four components in each thread: as much of a
// 128-byte line of columns as 512 threads hold.
template <class R, int N> struct ColVar {
    using PL = SmallPlan<N>;
    static constexpr int T = PL::T;
    static constexpr int W = imax(1, imin(128 / (int)sizeof(cpx<R>), 512 / T));
    static constexpr int THREADS = T * W;
    static constexpr size_t BYTES = (size_t)N * W * sizeof(cpx<R>);
    static_assert(plan_ok<N, T, PL>(), "column tile violates the FFT plan constraints");
};

// ------------------------------------------------------------------ row pass
// Global-address-space views of the state arrays (their pointers come from the
// solve descriptors, so the compiler cannot infer the address space itself and
// would otherwise emit flat memory instructions).
template <class T> using gptr = T __attribute__((address_space(1)))*;
template <class T> __device__ __forceinline__ gptr<T> glob(T* p) { return (gptr<T>)p; }
// complex numbers cross the global address space as native clang vectors
template <class R> using nv2 = R __attribute__((ext_vector_type(2)));
template <class C> __device__ __forceinline__ C gload(gptr<const nv2<decltype(C::x)>> p, long long i) {
    const nv2<decltype(C::x)> v = p[i];
    return cmake<C>(v.x, v.y);
}
template <class C> __device__ __forceinline__ void gstore(gptr<nv2<decltype(C::x)>> p, long long i, C c) {
    nv2<decltype(C::x)> v;
    v.x = c.x;
    v.y = c.y;
    p[i] = v;
}
// streaming (non-temporal) load and store: the stepping passes read and write
// each line once per launch, so caching it mostly evicts other data (the column
// tiles cover whole 128-byte lines).
template <class C> __device__ __forceinline__ C gload_nt(gptr<const nv2<decltype(C::x)>> p, long long i) {
    const nv2<decltype(C::x)> v = __builtin_nontemporal_load(&p[i]);
    return cmake<C>(v.x, v.y);
}
template <class C> __device__ __forceinline__ void gstore_nt(gptr<nv2<decltype(C::x)>> p, long long i, C c) {
    nv2<decltype(C::x)> v;
    v.x = c.x;
    v.y = c.y;
    __builtin_nontemporal_store(v, &p[i]);
}
template <class R> __device__ __forceinline__ gptr<const nv2<R>> cview(const void* p) {
    return (gptr<const nv2<R>>)(reinterpret_cast<const nv2<R>*>(p));
}
template <class R> __device__ __forceinline__ gptr<nv2<R>> wview(void* p) {
    return (gptr<nv2<R>>)(reinterpret_cast<nv2<R>*>(p));
}

template <class R, int N, int MODE>
__global__ void __launch_bounds__((RowVar<R, N>::THREADS)) row_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = RowVar<R, N>;
    constexpr int T = VC::T;
    constexpr int ROWS = VC::ROWS;
    constexpr int E = N / T;
    using Lay = typename VC::Lay;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* lds = reinterpret_cast<C*>(smem_raw);
    __shared__ R sh_fyz[ROWS][MAX_TERMS];
    __shared__ int sh_mu[MAX_TERMS];
    __shared__ long long sh_tab[MAX_TERMS];
    __shared__ C sh_wc[4];
    __shared__ C sh_phyz[ROWS];
    __shared__ C tw[N];

    const int tid = threadIdx.x;
    const int t = tid % T;
    const int line = tid / T;
    const int2 it = a.items[blockIdx.x];
    const SolveDev* __restrict__ S = a.solves + it.x;
    const int nrows = S->nrows;
    const int row = it.y * ROWS + line;
    const bool act = row < nrows;
    const int rowc = act ? row : 0;
    const long long base = (long long)rowc * N;
    const long long ns = S->nsites;
    // twiddle table in LDS: the first twiddle read comes after the first
    // exchange's barriers, so no extra barrier is needed here
    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    gptr<const R> rtab = glob(reinterpret_cast<const R*>(a.rtab));
    for (int i = tid; i < N; i += VC::THREADS) tw[i] = gload<C>(ctab, S->tw[0] + i);
    const int n0 = S->n[0], n1 = S->n[1];
    const int yy = rowc % n1, zz = rowc / n1;

    auto load = [&](int role, C (&w)[4][E]) {
        gptr<const nv2<R>> p = cview<R>(S->buf[role]) + base + t;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < E; ++m) w[q][m] = gload_nt<C>(p, q * ns + T * m);
    };
    auto store = [&](int role, const C (&w)[4][E]) {
        if (!act) return;
        gptr<nv2<R>> p = wview<R>(S->buf[role]) + base + t;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < E; ++m) gstore_nt<C>(p, q * ns + T * m, w[q][m]);
    };

    C v[4][E];
    if constexpr (MODE == ROW_SRC) {
        // no kinetic term: the epilogue below adds the source to zero
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < E; ++m) v[q][m] = cmake<C>((R)0, (R)0);
    } else {
        // ---- inverse transform of the k-space buffer (optionally after -i H0 / N)
        load(BUF_T, v);
        if (a.h0row) {
            const R Ky = (R)S->kap[1], Kz = (R)S->kap[2], s = (R)S->inv_n;
            const double dk = S->dk[0];
            if (a.expo) {
#pragma unroll
                for (int m = 0; m < E; ++m)
                    apply_expo(v[0][m], v[1][m], v[2][m], v[3][m], dk * kindex(t + T * m, N), S->kap[1], S->kap[2],
                               a.tau, S->inv_n);
            } else {
#pragma unroll
                for (int m = 0; m < E; ++m) {
                    const R Kx = (R)(dk * kindex(t + T * m, N));
                    apply_h0(v[0][m], v[1][m], v[2][m], v[3][m], Kx, Ky, Kz, s);
                }
            }
        }
        fft_line<C, N, T, +1, 4, Lay, typename VC::PL>(v, lds, t, line, tw);
    }
    if constexpr (MODE == ROW_INV) {
        store(a.dst, v);
        return;
    } else {
        // ---- stage epilogue: k = K - i V(t_i) (y_i + psi_b(t_i))
        double ts;
        if constexpr (MODE == ROW_RHS) {
            ts = a.t_explicit;
        } else {
            const double cst = a.stage == 0 ? 0.0 : (a.stage == 3 ? 1.0 : 0.5);
            ts = a.t_out - (double)(*a.step + a.step_add) * a.dt - cst * a.dt;
        }
        const int nterm = S->nterm;
        for (int j = t; j < nterm; j += T) {
            const TermDev tm = a.terms[S->term0 + j];
            const double coef = tm.amp * profile_t(tm.ft_type, tm.c, tm.w, tm.k, tm.phi, ts);
            sh_fyz[line][j] = (R)coef * rtab[tm.tab + n0 + yy] * rtab[tm.tab + n0 + n1 + zz];
            if (line == 0) {
                sh_mu[j] = tm.mu;
                sh_tab[j] = tm.tab;
            }
        }
        for (int q = tid; q < 4; q += VC::THREADS) {
            double sn, cs;
            sincos(-S->E * ts, &sn, &cs);
            const double wr = S->w[2 * q], wi = S->w[2 * q + 1];
            sh_wc[q] = cmake<C>((R)(wr * cs - wi * sn), (R)(wr * sn + wi * cs));
        }
        if (t == 0) sh_phyz[line] = cmul(gload<C>(ctab, S->ph + n0 + yy), gload<C>(ctab, S->ph + n0 + n1 + zz));
        {
            // state loads are independent of the barrier below: issue them first
            C yi[4][E];
            load(a.src, yi);
            __syncthreads();
            // field A_mu on this line's points
            R A[4][E];
#pragma unroll
            for (int mu = 0; mu < 4; ++mu)
#pragma unroll
                for (int m = 0; m < E; ++m) A[mu][m] = (R)0;
#pragma unroll
            for (int j = 0; j < MAX_TERMS; ++j) {
                if (j < nterm) {
                    const R fyz = sh_fyz[line][j];
                    gptr<const R> tab = rtab + sh_tab[j] + t;
                    const int mu = sh_mu[j];
#pragma unroll
                    for (int m = 0; m < E; ++m) {
                        const R f = fyz * tab[T * m];
                        A[0][m] += mu == 0 ? f : (R)0;
                        A[1][m] += mu == 1 ? f : (R)0;
                        A[2][m] += mu == 2 ? f : (R)0;
                        A[3][m] += mu == 3 ? f : (R)0;
                    }
                }
            }
            const long long phx = S->ph + t;
            const C wc[4] = {sh_wc[0], sh_wc[1], sh_wc[2], sh_wc[3]};
            const C phyz = sh_phyz[line];
#pragma unroll
            for (int m = 0; m < E; ++m) {
                const C ph = cmul(gload<C>(ctab, phx + T * m), phyz);
                C sv[4], vs[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) sv[q] = cadd(yi[q][m], cmul(wc[q], ph));
                apply_pot(sv, vs, A[0][m], A[1][m], A[2][m], A[3][m]);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q][m] = cadd(v[q][m], cmul_mi(vs[q]));   // v = k
            }
            store(a.dst, v);
        }
    }
}

// ------------------------------------------------------------------ column pass
// Forward transform along the last axis, -i H0 / N or the free evolution, and back
// (the whole state of a column in a thread group: the multiply mixes components).
template <class R, int N, int AXIS>
__global__ void __launch_bounds__((ColVar<R, N>::THREADS)) col_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = ColVar<R, N>;
    constexpr int T = VC::T;
    constexpr int W = VC::W;
    constexpr int E = N / T;
    using Lay = ColLay<N, W>;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* lds = reinterpret_cast<C*>(smem_raw);
    __shared__ C tw[N];

    const int tid = threadIdx.x;
    const int xl = tid % W;
    const int t = tid / W;

    // One tile = W adjacent columns of one solve at one fixed other-axis index.
    const int2 it = a.items[blockIdx.x];
    const SolveDev* __restrict__ S = a.solves + it.x;
    const int n0 = S->n[0], n1 = S->n[1];
    const int ntx = (n0 + W - 1) / W;
    const int other = it.y / ntx;
    const int x = (it.y % ntx) * W + xl;
    const bool act = x < n0;
    const long long stride = AXIS == 1 ? (long long)n0 : (long long)n0 * n1;
    const long long obase = AXIS == 1 ? (long long)other * n0 * n1 : (long long)other * n0;
    const long long base = obase + (act ? x : 0) + (long long)t * stride;
    const long long ns = S->nsites;

    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    for (int i = tid; i < N; i += VC::THREADS) tw[i] = gload<C>(ctab, S->tw[AXIS] + i);

    C v[4][E];
    {
        gptr<const nv2<R>> p = cview<R>(S->buf[a.dst]) + base;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < E; ++m) v[q][m] = gload<C>(p, q * ns + (long long)(T * m) * stride);
    }
    fft_line<C, N, T, -1, 4, Lay, typename VC::PL>(v, lds, t, xl, tw);
    const double kx = S->dk[0] * kindex(act ? x : 0, n0);
#pragma unroll
    for (int m = 0; m < E; ++m) {
        const int idx = t + T * m;
        double ky, kz;
        if constexpr (AXIS == 1) {
            ky = S->dk[1] * kindex(idx, N);
            kz = S->kap[2];
        } else {
            ky = S->dk[1] * kindex(other, n1);
            kz = S->dk[2] * kindex(idx, N);
        }
        if (a.expo) apply_expo(v[0][m], v[1][m], v[2][m], v[3][m], kx, ky, kz, a.tau, S->inv_n);
        else apply_h0(v[0][m], v[1][m], v[2][m], v[3][m], (R)kx, (R)ky, (R)kz, (R)S->inv_n);
    }
    fft_line<C, N, T, +1, 4, Lay, typename VC::PL>(v, lds, t, xl, tw);
    if (act) {
        gptr<nv2<R>> p = wview<R>(S->buf[a.dst]) + base;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int m = 0; m < E; ++m) gstore<C>(p, q * ns + (long long)(T * m) * stride, v[q][m]);
    }
}

// ------------------------------------------------------------------ stepping passes
// Source component and phase of the alpha^j entries (Dirac representation):
// (alpha^1 y)_q = y_{3-q}; (alpha^2 y)_q = (-i for even q, +i for odd q) y_{3-q};
// (alpha^3 y)_q = (+1 for q = 0, 2; -1 for q = 1, 3) y_{q^2}; beta = diag(1, 1, -1, -1).
template <class C> __device__ __forceinline__ C alpha2_phase(int q, C v) { return (q & 1) ? cmul_i(v) : cmul_mi(v); }
template <class C> __device__ __forceinline__ C alpha3_phase(int q, C v) { return (q & 1) ? cmake<C>(-v.x, -v.y) : v; }

// Values that are the same for a whole workgroup are read through the constant
// address space, as scalar loads.
template <class T> using sptr = const T __attribute__((address_space(4)))*;
template <class T> __device__ __forceinline__ sptr<T> uni(const T* p) { return (sptr<T>)p; }

// A uniform address the compiler has to keep in scalar registers (it otherwise
// folds the lane's offset into a chain of 64-bit vector addresses, two registers
// each).
__device__ __forceinline__ gptr<const char> scalar_base(gptr<const char> p) {
    asm("" : "+s"(p));
    return p;
}
// A complex number at a uniform base plus a byte offset of 32 bits.
template <class C, bool NT = true> __device__ __forceinline__ C gload_at(gptr<const char> base, unsigned off) {
    using V2 = nv2<decltype(C::x)>;
    V2 v;
    if constexpr (NT) v = __builtin_nontemporal_load((gptr<const V2>)(base + off));
    else v = *(gptr<const V2>)(base + off);
    return cmake<C>(v.x, v.y);
}
template <bool NT = true, class C> __device__ __forceinline__ void gstore_at(gptr<char> base, unsigned off, C c) {
    using V2 = nv2<decltype(C::x)>;
    V2 v;
    v.x = c.x;
    v.y = c.y;
    if constexpr (NT) __builtin_nontemporal_store(v, (gptr<V2>)(base + off));
    else *(gptr<V2>)(base + off) = v;
}

// Column derivative pass: a block transforms the component alpha^j takes for
// output component q of one tile along axis j = AXIS (y or z), multiplies by
// k_j / n_j, transforms back, and writes (ACCUM = 0) or adds (ACCUM = 1) the
// result, with alpha^j's phase, into component q of the G buffer (a.dst).  a.src: the stage input.  One component per thread: E
// points of the transform in registers, exchanged through LDS: as real and
// imaginary parts in turn where whole numbers would leave a compute unit room
// for one workgroup (SPLIT), so that one's loads cover another's transform.
//   v0, v1, v2: 1, 2, 4 lines of 128 bytes along x per tile, at most what 1024
//   threads and the LDS allow (512 points in single precision: one line; 512 in
//   double, 256 in single, 768 and 1024 in either: two).
// The four components of a tile are neighbouring blocks along y; along z a
// sweep over the tiles takes one component (blockIdx.y) after the other: y / z
// 2.87 / 5.19 ms with neighbouring components, 3.02 / 5.04 component after
// component (8 x 320^3 in single precision), 1.47 / 2.48 and 1.58 / 2.44 ms
// (4 x 256^3 in double).
// What bounds it: the access pattern, rows of a tile's width at the stride of
// the axis.  More lines per row help while several tiles fit a compute unit:
// 31 x 128^3 in single precision, y / z: 4.9 / 5.0 TB/s with one line, 6.1 / 5.8
// with four; 64 x 512^2 in double 5.1 with one, 5.5 with two; 768 points and
// more only fit one (28 x 768^2 in double 4.8 TB/s, two lines 4.0).  The 768-
// and 1024-point passes ran at 3.2 / 3.9 TB/s in double and 2.7 / 3.4 in single
// precision as one persistent workgroup per compute unit with the default plans.
template <class R, int N, int V> struct CdVar {
    static constexpr int LINE = 128 / sizeof(cpx<R>);   // columns per 128-byte line
    using PL = ColPlan<N>;
    static constexpr int T = PL::T;
    static constexpr int E = N / T;
    static constexpr size_t TAB = N * sizeof(cpx<R>) + (sizeof(R) == 4 ? N * sizeof(R) : 0);
    // widest power-of-two tile whose exchange buffer fits the LDS with the tables
    static constexpr int WFIT = (int)((163840 - TAB) / (N * sizeof(R)));
    static constexpr int WMAX = WFIT >= 64 ? 64 : (WFIT >= 32 ? 32 : (WFIT >= 16 ? 16 : 8));
    // (short lines: at least a wave per tile)
    static constexpr int W = imin(imin(imax(LINE << V, 64 / T), 1024 / T), WMAX);
    static constexpr int THREADS = T * W;
    static constexpr bool SPLIT = 2 * (N * W * sizeof(cpx<R>) + TAB) > 163840;
    static constexpr int XB = SPLIT ? sizeof(R) : sizeof(cpx<R>);
    static constexpr size_t XCH = (size_t)N * W * XB;
    static constexpr size_t BYTES = XCH + TAB;
    // the z pass's partial sums: loaded ahead of the transforms, or after them
    // where they would cost a workgroup's worth of registers (320 points in single
    // precision, two lines: 4.9 TB/s against 4.1)
    static constexpr bool LATE = sizeof(R) == 4 && E >= 20;
    // waves per SIMD the compiler is asked to fit, where it would otherwise end a
    // few registers above what the LDS has room for: 8 points a thread (512 points
    // in double, two lines: 66 registers leave one workgroup a compute unit and
    // 3.9 TB/s, 64 leave two and 5.3), and the longest lines
    static constexpr int FIT = (int)(163840 / BYTES) * imax(1, THREADS / 64) / 4;
    template <int ACCUM> static constexpr int waves() {
        return E <= 8 ? (ACCUM ? 1 : imax(1, imin(8, FIT)))
             : sizeof(R) == 8 ? (E >= 24 && !ACCUM ? 2 : 1) : E >= 24 ? (ACCUM ? 2 : 4) : 1;
    }
    static_assert(plan_ok<N, T, PL>(), "column derivative variant violates the FFT plan constraints");
};

template <class R, int N, int V, int AXIS, int ACCUM>
__global__ void __launch_bounds__((CdVar<R, N, V>::THREADS))
__attribute__((amdgpu_waves_per_eu(CdVar<R, N, V>::template waves<ACCUM>(), 8))) col_d_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = CdVar<R, N, V>;
    constexpr int T = VC::T;
    constexpr int W = VC::W;
    constexpr int E = VC::E;
    using PL = typename VC::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw + VC::XCH);
    R* kt = reinterpret_cast<R*>(tw + N);

    const int tid = threadIdx.x;
    const int xl = tid % W;
    const int t = tid / W;
    const int block = a.rev ? a.nitems - 1 - (int)blockIdx.x : (int)blockIdx.x;
    const int q = AXIS == 1 ? block & 3 : (int)blockIdx.y;   // output component
    const int src = AXIS == 1 ? 3 - q : (q ^ 2);    // the component alpha^j takes
    const unsigned long long item = *(sptr<unsigned long long>)(a.items + (AXIS == 1 ? block >> 2 : block));
    const int solve = (int)(unsigned)item, ty = (int)(item >> 32);
    const sptr<SolveDev> S = uni(a.solves + solve);
    const int n0 = S->n[0], n1 = S->n[1];
    const int ntx = (n0 + W - 1) / W;
    const long long ns = S->nsites;
    const unsigned stride = AXIS == 1 ? (unsigned)n0 : (unsigned)n0 * (unsigned)n1;
    // One tile = W adjacent columns of one solve at one fixed other-axis index;
    // thread (t, x) holds points t + T m of column x, at a 32-bit offset from
    // uniform addresses.
    const int other = __builtin_amdgcn_readfirstlane(ty / ntx), x0 = (ty - other * ntx) * W;
    const bool act = x0 + xl < n0;
    const long long base = x0 + (AXIS == 1 ? (long long)other * n0 * n1 : (long long)other * n0);
    const unsigned off = (unsigned)(t * stride + (act ? xl : 0)) * (unsigned)sizeof(C);
    gptr<const char> ps = (gptr<const char>)(cview<R>(S->buf[a.src]) + (base + src * ns));
    gptr<const char> pd = (gptr<const char>)(cview<R>(S->buf[a.dst]) + (base + q * ns));
    const long long step = (long long)T * stride * (long long)sizeof(C);   // from a thread's point to its next

    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    gptr<const R> rtab = glob(reinterpret_cast<const R*>(a.rtab));
    for (int i = tid; i < N; i += VC::THREADS) {
        tw[i] = gload<C>(ctab, S->twp[AXIS] + i);
        if constexpr (sizeof(R) == 4) kt[i] = rtab[S->kt[AXIS] + i];
    }
    C v[E], g[E];
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = gload_at<C>(scalar_base(ps + m * step), off);
    if constexpr (ACCUM && !VC::LATE) {
#pragma unroll
        for (int m = 0; m < E; ++m) g[m] = gload_at<C>(scalar_base(pd + m * step), off);
    }
    if constexpr (T * W <= 64) __syncthreads();   // the tables (else the first exchange's barriers come before their use)
    unsigned char* col = smem_raw + xl * VC::XB;
    fft_col<C, N, -1, W, VC::SPLIT, PL>(v, col, t, tw);
    const double kscale = S->dk[AXIS] / (double)N, td = (double)t;
#pragma unroll
    for (int m = 0; m < E; ++m) {
        // k / n (numpy order; E is even, so the sign of k follows from m)
        C w;
        if constexpr (sizeof(R) == 4) w = cscale(v[m], kt[t + T * m]);
        else w = cscale(v[m], (R)(kscale * (td + (double)(T * m - (m < E / 2 ? 0 : N)))));
        v[m] = AXIS == 1 ? alpha2_phase(q, w) : alpha3_phase(q, w);
    }
    fft_col<C, N, +1, W, VC::SPLIT, PL>(v, col, t, tw);
    if constexpr (ACCUM && VC::LATE) {
#pragma unroll
        for (int m = 0; m < E; ++m) g[m] = gload_at<C>(scalar_base(pd + m * step), off);
    }
    if (act) {
#pragma unroll
        for (int m = 0; m < E; ++m) gstore_at((gptr<char>)scalar_base(pd + m * step), off, ACCUM ? cadd(g[m], v[m]) : v[m]);
    }
}

// Row (x) stage pass: the RK4 stage STAGE.  T threads hold one spinor component
// of a grid line (E = N/T points each), 4T a line.  A thread transforms
// component 3 - q along x, multiplies by k_x / n_0 and transforms back, which
// gives (alpha^1 D_x y)_q, leaves it in LDS, and finishes whole sites (all
// four components of the sites t + T m, m = q, q + 4, ...), reading the stage
// input there again from the cache, so that the field and phase work is done
// once per site:
//     k_q = -i [alpha^1 D_x y + G + (beta y) + sum over trivial axes kappa_j (alpha^j y)
//               + (A_0 + alpha^j A_j)(y + psi_b)]_q,
// the RK4 update with the accumulator written once, and the absorber at the
// last stage.  STAGE 4..9 are the six stages of the fixed-step Dormand-Prince
// 5(4) stepper instead: the stage writes its slope k_s and the next stage input
// y + h sum_{j<=s} a_{s+1,j} k_j (reading the earlier slopes), the last one the
// step y + h sum_j b_j k_j.
//
// Every component line lies within one wave (T divides 64 in the default
// plans), so the transforms run without a barrier: the waves of a compute unit
// drift apart and one's loads cover another's arithmetic.
// The exchanges move real and imaginary parts one after the other (SPLIT): half
// the LDS, so that three or four waves per SIMD fit for every length (1024
// points in double: 0.59 ms against 0.63 ms unsplit, 9 x 1024^2, stage 1; the
// shorter lengths differ by 2% at most either way).  Blocks of 256 threads: 128
// were up to 9% slower (256 points in single precision) and at most 2% faster.
//
// What bounds it: HBM.  A kernel that only reads and writes the same lines of
// the same arrays takes 1.04 / 0.59 ms for stages 1 / 0 on 64 x 512^2 in double
// (5.2 / 5.5 TB/s), this pass 1.00 / 0.56 ms; 8 x 320^3 in single precision 7.7
// against 8.0 ms.  With barriers between the exchanges, the field selected by
// component per term and site, and the time factors formed per workgroup, the
// same stages took 0.99 / 0.67 ms and 9.1 ms, 9 x 1024^2 in double 0.82 ms
// (now 0.59) and 192 x 192 x 256 x 4 in double 3.7 ms (now 2.2).
template <class R, int N> struct RdVar {
    using PL = StepPlan<N>;
    static constexpr int T = PL::T;
    static constexpr int E = N / T;
    static constexpr int LT = 4 * T;          // threads of a grid line
    static constexpr bool WLINE = LT <= 64;   // a line within one wave
    static constexpr int ROWS = imax(1, 256 / LT);
    static constexpr int THREADS = LT * ROWS;
    static constexpr int SITES = E / 4;       // sites a thread finishes
    static constexpr int STRIDE = xch_stride<N, PL, sizeof(R)>();   // reals of a component line
    static constexpr size_t XCH = ((size_t)4 * ROWS * STRIDE * sizeof(R) + 15) / 16 * 16;
    // exchange buffer, twiddles and (single precision) the derivative's factors
    static constexpr size_t BYTES = XCH + N * sizeof(cpx<R>) + (sizeof(R) == 4 ? N * sizeof(R) : 0);
    // waves per SIMD the compiler is asked to fit: what the LDS of a compute
    // unit allows, and what the points and a prefetched site leave registers for
    static constexpr int BLOCKS_PER_CU = (int)(163840 / BYTES);
    static constexpr int WAVES = imax(1, imin(sizeof(R) == 4 ? (E >= 20 ? 3 : 4) : (E >= 16 ? 2 : 3), BLOCKS_PER_CU * imax(1, THREADS / 64) / 4));
    static_assert(plan_ok<N, T, PL>(), "row derivative pass violates the FFT plan constraints");
    static_assert(64 % T == 0 && E % 4 == 0, "a component line within one wave, whole sites per thread");
};

// (V: the tile variant, of which this pass has one; profiles name the kernel by it)
template <class R, int N, int V, int STAGE>
__global__ void __launch_bounds__((RdVar<R, N>::THREADS))
__attribute__((amdgpu_waves_per_eu(RdVar<R, N>::WAVES, 8))) row_d_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = RdVar<R, N>;
    constexpr int T = VC::T;
    constexpr int E = VC::E;
    constexpr int ROWS = VC::ROWS;
    constexpr int LT = VC::LT;
    constexpr int SITES = VC::SITES;
    using PL = typename VC::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw + VC::XCH);
    R* kt = reinterpret_cast<R*>(tw + N);

    const int tid = threadIdx.x;
    const int t = tid % T;
    // (uniform over the wave where a line, or a component line, takes whole waves)
    const int q = T == 64 ? __builtin_amdgcn_readfirstlane(tid / T % 4) : tid / T % 4;
    const int line = LT >= 64 ? __builtin_amdgcn_readfirstlane(tid / LT) : tid / LT;
    const unsigned long long item =
        *(sptr<unsigned long long>)(a.items + (a.rev ? a.nitems - 1 - (int)blockIdx.x : (int)blockIdx.x));
    const int solve = (int)(unsigned)item, ty = (int)(item >> 32);
    const sptr<SolveDev> S = uni(a.solves + solve);
    const int row0 = ty * ROWS;
    const bool act = row0 + line < S->nrows;
    const int linec = act ? line : 0;       // a line beyond the last one repeats the tile's first
    const long long ns = S->nsites;
    const long long tile0 = (long long)row0 * N;
    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    gptr<const R> rtab = glob(reinterpret_cast<const R*>(a.rtab));

    // STAGE 0..3: classical RK4 stages; 4..9: Dormand-Prince stages 0..5
    constexpr bool DP = STAGE >= 4;
    constexpr int DS = DP ? STAGE - 4 : 0;
    constexpr bool FIRST = STAGE == 0 || STAGE == 4, LAST = STAGE == 3 || STAGE == 9;
    gptr<const nv2<R>> pin = cview<R>(S->buf[FIRST ? BUF_Y : BUF_YS]) + tile0;
    for (int i = tid; i < N; i += VC::THREADS) {
        tw[i] = gload<C>(ctab, S->twp[0] + i);
        if constexpr (sizeof(R) == 4) kt[i] = rtab[S->kt[0] + i];
    }
    // the component alpha^1 takes (read again, as whole sites, by the epilogue)
    C v[E];
    {
        gptr<const nv2<R>> p = pin + (3 - q) * ns + (linec * N + t);
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = gload<C>(p, T * m);
    }
    __syncthreads();
    R* xl = reinterpret_cast<R*>(smem_raw) + 4 * line * VC::STRIDE;   // this line's exchange buffer
    R* xch = xl + q * VC::STRIDE;                                     // this component's part of it
    fft_row<C, N, -1, true, PL>(v, xch, t, tw);
    // k_x / n_0 (numpy order; E is even, so the sign of k follows from m)
    if constexpr (sizeof(R) == 4) {
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = cscale(v[m], kt[t + T * m]);
    } else {
        const double kscale = S->dk[0] / (double)N, td = (double)t;
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = cscale(v[m], (R)(kscale * (td + (double)(T * m - (m < E / 2 ? 0 : N)))));
    }

    // ---- stage epilogue: the thread's sites t + T (q + 4 j), one at a time, the
    // next one's operands in flight
    gptr<const char> by[4], bg[4], bo[4];
    gptr<char> w0[4], w1[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const long long o = c * ns + tile0;
        by[c] = (gptr<const char>)(pin + c * ns);
        bg[c] = (gptr<const char>)(cview<R>(S->buf[BUF_T]) + o);
        bo[c] = (gptr<const char>)(cview<R>(S->buf[STAGE == 3 ? BUF_ACC : BUF_Y]) + o);
        w0[c] = (gptr<char>)(wview<R>(S->buf[LAST ? BUF_Y : BUF_YS]) + o);
        w1[c] = (gptr<char>)(wview<R>(S->buf[DP ? dp5_kbuf(DS < 5 ? DS : 0) : BUF_ACC]) + o);
    }
    const int dim = S->dim, nterm = S->nterm, mus = S->mus;
    const int site0 = t + T * q;
    const unsigned off0 = (unsigned)(linec * N + site0) * (unsigned)sizeof(C);
    struct Ops { C y[4], g[4], o[4]; };
    auto load = [&](Ops& p, int j) {
        const unsigned off = off0 + (unsigned)(4 * T * j * (int)sizeof(C));
#pragma unroll
        for (int c = 0; c < 4; ++c) p.y[c] = gload_at<C>(by[c], off);
        if (dim >= 2) {
#pragma unroll
            for (int c = 0; c < 4; ++c) p.g[c] = gload_at<C>(bg[c], off);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) p.g[c] = cmake<C>((R)0, (R)0);
        }
        if constexpr (!FIRST) {
#pragma unroll
            for (int c = 0; c < 4; ++c) p.o[c] = gload_at<C>(bo[c], off);
        }
    };

    fft_row<C, N, +1, true, PL>(v, xch, t, tw);

    Ops ops[2];
    load(ops[0], 0);
    // ---- from one component per thread to whole sites
    C d[SITES][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (h && !VC::WLINE) __syncthreads();
        else wave_lds_order();
#pragma unroll
        for (int m = 0; m < E; ++m) xch[t + T * m] = h ? v[m].y : v[m].x;
        if constexpr (VC::WLINE) wave_lds_order();
        else __syncthreads();
#pragma unroll
        for (int j = 0; j < SITES; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) (h ? d[j][c].y : d[j][c].x) = xl[c * VC::STRIDE + site0 + 4 * T * j];
    }

    const R h = (R)(-a.dt);
    const R h2 = (R)(-0.5 * a.dt), h6 = (R)(-a.dt / 6.0), third = (R)(1.0 / 3.0);
    const R hk = (R)(-a.dt * dp5_a(DS + 1, DS));   // h a_{s+1,s} for the stage's own slope
    const sptr<StageConst<R>> K = uni(reinterpret_cast<const StageConst<R>*>(a.consts) + (long long)solve * a.nst + (DP ? DS : STAGE));
    const int n0 = N, n1 = S->n[1];
    const int row = row0 + linec;
    const int yy = row % n1, zz = row / n1;
    const C phyz = cmul(gload<C>(ctab, S->ph + n0 + yy), gload<C>(ctab, S->ph + n0 + n1 + zz));
    const long long mask = S->mask;
    const R myz = (LAST && mask >= 0) ? rtab[mask + n0 + yy] * rtab[mask + n0 + n1 + zz] : (R)1;
#pragma unroll
    for (int j = 0; j < SITES; ++j) {
        const int idx = site0 + 4 * T * j;
        const unsigned off = off0 + (unsigned)(4 * T * j * (int)sizeof(C));
        // field A_mu and background phase at the site
        R A[4] = {(R)0, (R)0, (R)0, (R)0};
        for (int jt = 0; jt < nterm; ++jt) {
            const sptr<TermDev> tm = uni(a.terms + S->term0 + jt);
            gptr<const R> tab = rtab + tm->tab;
            const R f = K->coef[jt] * tab[n0 + yy] * tab[n0 + n1 + zz] * tab[idx];
            const int mu = tm->mu;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (mu == u) A[u] += f;
        }
        const C ph = cmul(gload<C>(ctab, S->ph + idx), phyz);
        if (j + 1 < SITES) load(ops[(j + 1) & 1], j + 1);
        const Ops& p = ops[j & 1];
        // u = alpha^1 D_x y + G + beta y + kappa terms + (A_0 + alpha^j A_j)(y + psi_b)
        C u[4], s[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const C w = cadd(d[j][c], p.g[c]);
            u[c] = c < 2 ? cadd(w, p.y[c]) : csub(w, p.y[c]);
            s[c] = cadd(p.y[c], cmul(cmake<C>(K->w[2 * c], K->w[2 * c + 1]), ph));
        }
        if (dim < 3) {
            const R ky = (R)S->kap[1], kz = (R)S->kap[2];   // zero on non-trivial axes
#pragma unroll
            for (int c = 0; c < 4; ++c)
                u[c] = cadd(u[c], cadd(cscale(alpha2_phase(c, p.y[3 - c]), ky), cscale(alpha3_phase(c, p.y[c ^ 2]), kz)));
        }
        // only the components some term has (the bits are the same for the whole workgroup)
#pragma unroll
        for (int mu = 0; mu < 4; ++mu)
            if (mus & (1 << mu)) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const C b = mu == 0 ? s[c] : mu == 1 ? s[3 - c] : mu == 2 ? alpha2_phase(c, s[3 - c]) : alpha3_phase(c, s[c ^ 2]);
                    u[c] = cadd(u[c], cscale(b, A[mu]));
                }
            }
        // classical RK4 with the accumulator written once: with the stage
        // inputs y_2 = y + h/2 k1, y_3 = y + h/2 k2, y_4 = y + h k3,
        //   y_{n+1} = (y_2 + 2 y_3 - y)/3 + y_4/3 + h/6 k4,
        // so stage 1 stores acc = (y_2 + 2 y_3 - y)/3 and stage 3 finishes
        const R mk = (LAST && mask >= 0) ? rtab[mask + idx] * myz : (R)1;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const C k = cmul_mi(u[c]);
            C o0, o1;
            if constexpr (DP) {
                // Dormand-Prince: y_{s+1} = y + h sum_{j<=s} a_{s+1,j} k_j (row 6: the step)
                C acc = DS == 0 ? p.y[c] : p.o[c];
#pragma unroll
                for (int i = 0; i < DS; ++i)
                    if (dp5_a(DS + 1, i) != 0.0)
                        acc = cadd(acc, cscale(gload_at<C>((gptr<const char>)(cview<R>(S->buf[dp5_kbuf(i)]) + (c * ns + tile0)), off),
                                               (R)(-a.dt * dp5_a(DS + 1, i))));
                o0 = cadd(acc, cscale(k, hk));
                if constexpr (LAST) o0 = cscale(o0, mk);
                o1 = k;
            } else if constexpr (STAGE == 0) {
                o0 = cadd(p.y[c], cscale(k, h2));                                                 // y_2
            } else if constexpr (STAGE == 1) {
                o0 = cadd(p.o[c], cscale(k, h2));                                                 // y_3
                o1 = cscale(csub(cadd(p.y[c], cscale(o0, (R)2)), p.o[c]), third);
            } else if constexpr (STAGE == 2) {
                o0 = cadd(p.o[c], cscale(k, h));                                                  // y_4
            } else {
                o0 = cscale(cadd(cadd(p.o[c], cscale(p.y[c], third)), cscale(k, h6)), mk);
            }
            if (act) {
                if constexpr (STAGE == 1 || (DP && DS < 5)) gstore_at(w1[c], off, o1);
                gstore_at(w0[c], off, o0);
            }
        }
    }
}

// ------------------------------------------------------------------ whole-state transforms
// Transforms of a state along one axis that mix no components: one component
// per group of threads, with the row pass's lines and exchanges or the column
// pass's tiles (one component per blockIdx.y).  They read a state once and write
// it once, which is what bounds them where the state is large; a single small
// state is bound by the launch, so more threads a line help there too.
// PH: times exp(i k.x) before the transform (tables at a.ph2).  NT: past the caches.
//
// Measured, one 320^3 state in single precision: x 0.36 ms (5.8 TB/s; 0.46 with
// all four components in each thread and barriers), y 0.37, z 0.42 ms (5.0 TB/s;
// 0.42 on average); 16 x 256 x 192 in double, x inverse 17 us (25), forward 20 (19).
template <class R, int N, int DIR, bool PH, bool NT>
__global__ void __launch_bounds__((RdVar<R, N>::THREADS)) row_t_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = RdVar<R, N>;
    constexpr int T = VC::T;
    constexpr int E = VC::E;
    using PL = typename VC::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw + VC::XCH);
    const int tid = threadIdx.x;
    const int t = tid % T, q = tid / T % 4, line = tid / VC::LT;
    const unsigned long long item = *(sptr<unsigned long long>)(a.items + blockIdx.x);
    const sptr<SolveDev> S = uni(a.solves + (int)(unsigned)item);
    const int row0 = (int)(item >> 32) * VC::ROWS;
    const bool act = row0 + line < S->nrows;
    const int row = row0 + (act ? line : 0);
    const long long at = q * S->nsites + (long long)row * N + t;
    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    for (int i = tid; i < N; i += VC::THREADS) tw[i] = gload<C>(ctab, S->twp[0] + i);
    C v[E];
    {
        gptr<const nv2<R>> p = cview<R>(S->buf[a.src]) + at;
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = NT ? gload_nt<C>(p, T * m) : gload<C>(p, T * m);
    }
    if constexpr (PH) {
        const int n1 = S->n[1];
        const C pyz = cmul(gload<C>(ctab, a.ph2 + N + row % n1), gload<C>(ctab, a.ph2 + N + n1 + row / n1));
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = cmul(v[m], cmul(gload<C>(ctab, a.ph2 + t + T * m), pyz));
    }
    __syncthreads();   // the twiddles
    fft_row<C, N, DIR, true, PL>(v, reinterpret_cast<R*>(smem_raw) + (4 * line + q) * VC::STRIDE, t, tw);
    if (act) {
        gptr<nv2<R>> p = wview<R>(S->buf[a.dst]) + at;
#pragma unroll
        for (int m = 0; m < E; ++m) NT ? gstore_nt<C>(p, T * m, v[m]) : gstore<C>(p, T * m, v[m]);
    }
}

// Along z tiles of two lines up to 512 points (320^3 in
// single precision 0.42 ms, one line 0.45); along y one, since a single (2+1)D
// state has few tiles (256 x 192 in double 5.1 us, two lines 5.7; 320^3 0.37 either way).
constexpr int col_t_tile(int axis, int n) { return axis == 2 && n <= 512 ? 1 : 0; }
template <class R, int N, int AXIS, int DIR>
__global__ void __launch_bounds__((CdVar<R, N, col_t_tile(AXIS, N)>::THREADS)) col_t_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = CdVar<R, N, col_t_tile(AXIS, N)>;
    constexpr int T = VC::T;
    constexpr int W = VC::W;
    constexpr int E = VC::E;
    using PL = typename VC::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw + VC::XCH);
    const int tid = threadIdx.x, xl = tid % W, t = tid / W;
    const unsigned long long item = *(sptr<unsigned long long>)(a.items + blockIdx.x);
    const int ty = (int)(item >> 32);
    const sptr<SolveDev> S = uni(a.solves + (int)(unsigned)item);
    const int n0 = S->n[0], n1 = S->n[1];
    const int ntx = (n0 + W - 1) / W;
    const unsigned stride = AXIS == 1 ? (unsigned)n0 : (unsigned)n0 * (unsigned)n1;
    const int other = __builtin_amdgcn_readfirstlane(ty / ntx), x0 = (ty - other * ntx) * W;
    const bool act = x0 + xl < n0;
    const long long base = x0 + (AXIS == 1 ? (long long)other * n0 * n1 : (long long)other * n0);
    const unsigned off = (unsigned)(t * stride + (act ? xl : 0)) * (unsigned)sizeof(C);
    gptr<const char> pd = (gptr<const char>)(cview<R>(S->buf[a.dst]) + (base + (int)blockIdx.y * S->nsites));
    const long long step = (long long)T * stride * (long long)sizeof(C);
    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    for (int i = tid; i < N; i += VC::THREADS) tw[i] = gload<C>(ctab, S->twp[AXIS] + i);
    C v[E];
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = gload_at<C>(scalar_base(pd + m * step), off);
    if constexpr (T * W <= 64) __syncthreads();   // the twiddles
    fft_col<C, N, DIR, W, VC::SPLIT, PL>(v, smem_raw + xl * VC::XB, t, tw);
    if (act) {
#pragma unroll
        for (int m = 0; m < E; ++m) gstore_at((gptr<char>)scalar_base(pd + m * step), off, v[m]);
    }
}

// Forward transform along the last axis, -i H0 / N or the free evolution, and
// back: one component per group of threads for the transforms, whole sites (a
// quarter of them a thread) for the multiply, which mixes components; real and
// imaginary parts cross the LDS one after the other.
//
// With all four components in each thread (col_kernel) a batch of 50 MB in
// double leaves one wave per SIMD, which waits for its own loads, sincos and
// barriers.  Microseconds here and there, 256 columns x N, 3072 / N solves, in
// double / single precision:  32: 15 / 12 (29 / 14), 64: 24 / 15 (34 / 18),
// 80: 26 / 18 (126 / 32), 160: 37 / 34 (70 / 37), 192: 31 / 22 (40 / 27),
// 320: 56 / 36 (73 / 38), 384 in double: 37 (47).  No better, and left to
// col_kernel: powers of two from 128 (double 31 (29) at 128 and 46 (45) at 256
// points, single precision 28 (21) at 128: the other plan is already at 8 points
// a thread), 384 in single precision (42 (32): 1024 threads of 24 points), and
// what does not fit a workgroup with whole 128-byte lines.
template <class R, int N> struct HdVar {
    using CV = CdVar<R, N, 0>;
    static constexpr int T = CV::T, W = CV::W, E = CV::E;
    static constexpr int THREADS = 4 * T * W;
    static constexpr size_t COMP = (size_t)N * W * sizeof(R);
    static constexpr size_t BYTES = 4 * COMP + N * sizeof(cpx<R>);
    static constexpr bool FITS = THREADS <= 1024 && BYTES <= 163840 && E % 4 == 0 &&
                                 ((N & (N - 1)) == 0 ? N <= 64 : THREADS <= 512 || E <= 20);
};

template <class R, int N, int AXIS>
__global__ void __launch_bounds__((HdVar<R, N>::THREADS)) col_h0_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = HdVar<R, N>;
    constexpr int T = VC::T;
    constexpr int W = VC::W;
    constexpr int E = VC::E;
    constexpr int SITES = E / 4;
    using PL = typename VC::CV::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* tw = reinterpret_cast<C*>(smem_raw + 4 * VC::COMP);
    const int tid = threadIdx.x, xl = tid % W, t = tid / W % T, q = tid / (W * T);
    const unsigned long long item = *(sptr<unsigned long long>)(a.items + blockIdx.x);
    const int ty = (int)(item >> 32);
    const sptr<SolveDev> S = uni(a.solves + (int)(unsigned)item);
    const int n0 = S->n[0], n1 = S->n[1];
    const int ntx = (n0 + W - 1) / W;
    const unsigned stride = AXIS == 1 ? (unsigned)n0 : (unsigned)n0 * (unsigned)n1;
    const int other = __builtin_amdgcn_readfirstlane(ty / ntx), x0 = (ty - other * ntx) * W;
    const bool act = x0 + xl < n0;
    const int x = act ? x0 + xl : x0;
    gptr<nv2<R>> p = wview<R>(S->buf[a.dst]) + (x + (AXIS == 1 ? (long long)other * n0 * n1 : (long long)other * n0) +
                                              q * S->nsites + (long long)t * stride);
    const long long step = (long long)T * stride;
    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    for (int i = tid; i < N; i += VC::THREADS) tw[i] = gload<C>(ctab, S->twp[AXIS] + i);
    C v[E];
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = gload<C>(p, m * step);
    if constexpr (T * W <= 64) __syncthreads();   // the twiddles
    unsigned char* col = smem_raw + q * VC::COMP + xl * sizeof(R);
    fft_col<C, N, -1, W, true, PL>(v, col, t, tw);
    // ---- to whole sites t + T (q + 4 j), the multiply, and back to components
    R* xs = reinterpret_cast<R*>(smem_raw) + t * W + xl;
    constexpr int COMP = N * W, LINE = T * W;
    C d[SITES][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
#pragma unroll
        for (int m = 0; m < E; ++m) xs[q * COMP + m * LINE] = h ? v[m].y : v[m].x;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SITES; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) (h ? d[j][c].y : d[j][c].x) = xs[c * COMP + (q + 4 * j) * LINE];
    }
    const double kx = S->dk[0] * kindex(x, n0);
#pragma unroll
    for (int j = 0; j < SITES; ++j) {
        const int idx = t + T * (q + 4 * j);
        const double ky = S->dk[1] * (AXIS == 1 ? kindex(idx, N) : kindex(other, n1));
        const double kz = AXIS == 1 ? S->kap[2] : S->dk[2] * kindex(idx, N);
        if (a.expo) apply_expo(d[j][0], d[j][1], d[j][2], d[j][3], kx, ky, kz, a.tau, S->inv_n);
        else apply_h0(d[j][0], d[j][1], d[j][2], d[j][3], (R)kx, (R)ky, (R)kz, (R)S->inv_n);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SITES; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) xs[c * COMP + (q + 4 * j) * LINE] = h ? d[j][c].y : d[j][c].x;
        __syncthreads();
#pragma unroll
        for (int m = 0; m < E; ++m) (h ? v[m].y : v[m].x) = xs[q * COMP + m * LINE];
    }
    fft_col<C, N, +1, W, true, PL>(v, col, t, tw);
    if (act) {
#pragma unroll
        for (int m = 0; m < E; ++m) gstore<C>(p, m * step, v[m]);
    }
}

// ------------------------------------------------------------------ 1D whole-loop kernel
// A (1+1)D solve is one line of at most 1024 points: its whole state fits on
// one compute unit.  line_kernel runs a.nsteps complete RK4 steps of one solve
// per workgroup without leaving the chip.  4T threads, as in the row pass: a
// group of T transforms one component (E = N/T points each, within one wave, so
// without a barrier), and every thread finishes whole sites t + T (q + 4 j),
// whose state, stage input and RK4 sum it keeps in registers, with the
// background phase, the absorber mask and the profiles of the first
// LINE_TERMS field terms (further terms' profiles are staged in LDS).  A stage
// costs two workgroup barriers: the stage inputs go through LDS to the component
// groups, the derivatives back to the sites.  The update is the classical
// y_{n+1} = y + h/6 (k1 + 2 k2 + 2 k3 + k4) with h = -dt, accumulated stage by
// stage.  The time factors of LINE_BLOCK steps are evaluated at once, in double,
// one per thread, and kept in LDS.  Only the final state is written to the Y array.
//
// What bounds it: one workgroup's latency, LDS first (1024 points in double:
// about 270 16-byte accesses a thread and stage, 8 cycles each for every one of
// four waves, against 1500 vector instructions of 4 cycles).  In double, 1024
// points take 33 us a step and 512 points 16.6 us (47 and 34 us with all four
// components in each thread, radix 4 and a barrier per exchange and component
// pair); 1024 points over eight waves, whose exchanges then need barriers, 37 us.
constexpr int LINE_TERMS = 4;    // field terms whose profiles a thread keeps in registers
constexpr int LINE_BLOCK = 16;   // steps whose time factors are formed together
template <class R, int N> struct LineVar {
    using PL = StepPlan<N>;
    static constexpr int T = PL::T;
    static constexpr int E = N / T;
    static constexpr int THREADS = 4 * T;
    static constexpr int SITES = E / 4;
    static constexpr bool WLINE = THREADS <= 64;
    static constexpr int STRIDE = xch_stride<N, PL, sizeof(cpx<R>)>();   // points of a component line
    static constexpr size_t XCH = (size_t)4 * STRIDE * sizeof(cpx<R>);
    static constexpr size_t IN = (size_t)4 * N * sizeof(cpx<R>);
    // dynamic LDS without profiles: exchange, stage input, twiddles, derivative
    // factors (single precision), time factors (the host adds N reals per term
    // beyond LINE_TERMS)
    static constexpr size_t BASE_BYTES = XCH + IN + N * sizeof(cpx<R>) + (sizeof(R) == 4 ? N * sizeof(R) : 0) +
                                         LINE_BLOCK * 3 * sizeof(StageConst<R>);
    static_assert(plan_ok<N, T, PL>() && E % 4 == 0, "whole sites per thread");
};

// A zero the compiler cannot see through.
__device__ __forceinline__ int opaque_zero() {
    int z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

template <class R, int N>
__global__ void __launch_bounds__((LineVar<R, N>::THREADS)) line_kernel(PassArgs a) {
    using C = cpx<R>;
    using VC = LineVar<R, N>;
    constexpr int T = VC::T;
    constexpr int E = VC::E;
    constexpr int SITES = VC::SITES;
    constexpr int STRIDE = VC::STRIDE;
    using PL = typename VC::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* xch = reinterpret_cast<C*>(smem_raw);
    C* yin = reinterpret_cast<C*>(smem_raw + VC::XCH);
    C* tw = reinterpret_cast<C*>(smem_raw + VC::XCH + VC::IN);
    StageConst<R>* tc = reinterpret_cast<StageConst<R>*>(tw + N);   // [step of the block][node 0, 1/2, 1]
    R* kt = reinterpret_cast<R*>(tc + LINE_BLOCK * 3);
    R* fxl = kt + (sizeof(R) == 4 ? N : 0);                         // profiles of the terms beyond LINE_TERMS

    const int tid = threadIdx.x;
    const int t = tid % T;
    const int q = T == 64 ? __builtin_amdgcn_readfirstlane(tid / T) : tid / T;
    const int solve = (int)*(sptr<unsigned>)(a.items + blockIdx.x);
    const sptr<SolveDev> S = uni(a.solves + solve);
    gptr<const nv2<R>> ctab = cview<R>(a.ctab);
    gptr<const R> rtab = glob(reinterpret_cast<const R*>(a.rtab));
    const int nterm = S->nterm, mus = S->mus;
    const long long mk = S->mask;
    for (int i = tid; i < N; i += VC::THREADS) {
        tw[i] = gload<C>(ctab, S->twp[0] + i);
        if constexpr (sizeof(R) == 4) kt[i] = rtab[S->kt[0] + i];
    }
    const int site0 = t + T * q;
    // trivial axes (index 0 of each): constant factors of the tables
    C ph[SITES];
    R msk[SITES], fx0[SITES], fx1[SITES], fx2[SITES], fx3[SITES];
    int mu0, mu1, mu2, mu3;
    static_assert(LINE_TERMS == 4, "fx0 .. fx3");
    {
        const C phyz = cmul(gload<C>(ctab, S->ph + N), gload<C>(ctab, S->ph + N + 1));
        const R myz = mk >= 0 ? rtab[mk + N] * rtab[mk + N + 1] : (R)1;
#pragma unroll
        for (int j = 0; j < SITES; ++j) {
            const int i = site0 + 4 * T * j;
            ph[j] = cmul(gload<C>(ctab, S->ph + i), phyz);
            msk[j] = mk >= 0 ? rtab[mk + i] * myz : (R)1;
        }
        auto term = [&](int k, int& m, R (&f)[SITES]) {
            m = -1;
#pragma unroll
            for (int j = 0; j < SITES; ++j) f[j] = (R)0;
            if (k < nterm) {
                const sptr<TermDev> tm = uni(a.terms + S->term0 + k);
                gptr<const R> tab = rtab + tm->tab;
                const R fyz = tab[N] * tab[N + 1];
                m = tm->mu;
#pragma unroll
                for (int j = 0; j < SITES; ++j) f[j] = tab[site0 + 4 * T * j] * fyz;
            }
        };
        // (written out: a loop over them is unrolled too late for registers)
        term(0, mu0, fx0);
        term(1, mu1, fx1);
        term(2, mu2, fx2);
        term(3, mu3, fx3);
        for (int k = LINE_TERMS; k < nterm; ++k) {
            gptr<const R> tab = rtab + uni(a.terms + S->term0 + k)->tab;
            const R fyz = tab[N] * tab[N + 1];
            for (int i = tid; i < N; i += VC::THREADS) fxl[(k - LINE_TERMS) * N + i] = tab[i] * fyz;
        }
    }
    gptr<nv2<R>> py = wview<R>(S->buf[BUF_Y]) + site0;
    C y[SITES][4];
#pragma unroll
    for (int j = 0; j < SITES; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) y[j][c] = gload<C>((gptr<const nv2<R>>)py, c * (long long)N + 4 * T * j);

    const R Ky = (R)S->kap[1], Kz = (R)S->kap[2];
    const double kscale = S->dk[0] / (double)N;
    const double dt = a.dt;
    const R h = (R)(-dt), h2 = (R)(-0.5 * dt), h3 = (R)(-dt / 3.0), h6 = (R)(-dt / 6.0);
    const int n_first = *a.step + a.step_add;
    C* xq = xch + q * STRIDE;

    // k = -i [alpha^1 D_x y + beta y + kappa terms + (A_0 + alpha^j A_j)(y + psi_b)] at the thread's
    // sites; tcs: the stage's time factors
    auto rhs = [&](const C (&yst)[SITES][4], C (&k)[SITES][4], const StageConst<R>* tcs) {
#pragma unroll
        for (int j = 0; j < SITES; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) yin[c * N + site0 + 4 * T * j] = yst[j][c];
        xch_order<VC::WLINE>();
        C v[E];
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = yin[(3 - q) * N + t + T * m];
        fft_row<C, N, -1, false, PL>(v, xq, t, tw);
        // (an opaque zero: the factors are formed here, not kept in registers over the time loop)
        const double td = (double)(t + opaque_zero());
#pragma unroll
        for (int m = 0; m < E; ++m) {
            if constexpr (sizeof(R) == 4) v[m] = cscale(v[m], kt[t + T * m]);
            else v[m] = cscale(v[m], (R)(kscale * (td + (double)(T * m - (m < E / 2 ? 0 : N)))));
        }
        fft_row<C, N, +1, false, PL>(v, xq, t, tw);
        wave_lds_order();
#pragma unroll
        for (int m = 0; m < E; ++m) xq[t + T * m] = v[m];
        // field and source at the sites: independent of the derivative, ahead of the barrier
        R A[4][SITES];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < SITES; ++j) A[u][j] = (R)0;
        auto add = [&](int m, R coef, const R (&f)[SITES]) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (m == u) {
#pragma unroll
                    for (int j = 0; j < SITES; ++j) A[u][j] += coef * f[j];
                }
        };
        if (nterm > 0) add(mu0, tcs->coef[0], fx0);
        if (nterm > 1) add(mu1, tcs->coef[1], fx1);
        if (nterm > 2) add(mu2, tcs->coef[2], fx2);
        if (nterm > 3) add(mu3, tcs->coef[3], fx3);
        for (int i = LINE_TERMS; i < nterm; ++i) {
            R f[SITES];
#pragma unroll
            for (int j = 0; j < SITES; ++j) f[j] = fxl[(i - LINE_TERMS) * N + site0 + 4 * T * j];
            add(uni(a.terms + S->term0 + i)->mu, tcs->coef[i], f);
        }
        C wc[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) wc[c] = cmake<C>(tcs->w[2 * c], tcs->w[2 * c + 1]);
        C u[SITES][4];
#pragma unroll
        for (int j = 0; j < SITES; ++j) {
            // (the stage input again from LDS: not held in registers over the transforms)
            C yi[4], s[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) yi[c] = yin[c * N + site0 + 4 * T * j];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                s[c] = cadd(yi[c], cmul(wc[c], ph[j]));
                u[j][c] = cadd(cscale(yi[c], c < 2 ? (R)1 : (R)-1),
                               cadd(cscale(alpha2_phase(c, yi[3 - c]), Ky), cscale(alpha3_phase(c, yi[c ^ 2]), Kz)));
            }
            // only the components some term has
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (mus & (1 << m)) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const C b = m == 0 ? s[c] : m == 1 ? s[3 - c] : m == 2 ? alpha2_phase(c, s[3 - c]) : alpha3_phase(c, s[c ^ 2]);
                        u[j][c] = cadd(u[j][c], cscale(b, A[m][j]));
                    }
                }
        }
        xch_order<VC::WLINE>();
#pragma unroll
        for (int j = 0; j < SITES; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) k[j][c] = cmul_mi(cadd(xch[c * STRIDE + site0 + 4 * T * j], u[j][c]));
    };

#pragma unroll 1
    for (int n0 = 0; n0 < a.nsteps; n0 += LINE_BLOCK) {
        // the time factors of the next LINE_BLOCK steps (the last stage of the
        // block before has been left by every thread once they are all here)
        __syncthreads();
        constexpr int SLOTS = 4 + MAX_TERMS;
        for (int i = tid; i < LINE_BLOCK * 3 * SLOTS; i += VC::THREADS) {
            const int slot = i % SLOTS, node = i / SLOTS % 3, n = n0 + i / SLOTS / 3;
            const double tn = a.t_out - (double)(n_first + n) * dt;
            const double ts = node == 0 ? tn : node == 1 ? tn - 0.5 * dt : tn - dt;
            StageConst<R>* K = tc + i / SLOTS;
            if (slot < 4) {
                double sn, cs;
                sincos(-S->E * ts, &sn, &cs);
                const double wr = S->w[2 * slot], wi = S->w[2 * slot + 1];
                K->w[2 * slot] = (R)(wr * cs - wi * sn);
                K->w[2 * slot + 1] = (R)(wr * sn + wi * cs);
            } else if (slot - 4 < nterm) {
                const TermDev tm = a.terms[S->term0 + slot - 4];
                K->coef[slot - 4] = (R)(tm.amp * profile_t(tm.ft_type, tm.c, tm.w, tm.k, tm.phi, ts));
            }
        }
        __syncthreads();
        const int nb = a.nsteps - n0 < LINE_BLOCK ? a.nsteps - n0 : LINE_BLOCK;
#pragma unroll 1
        for (int n = 0; n < nb; ++n) {
            // stage 1 at t_n, stages 2 and 3 at t_n + h/2, stage 4 at t_n + h, then the
            // absorber: one copy of the stage's code, which otherwise does not fit the
            // instruction cache
            C yi[SITES][4], acc[SITES][4];
#pragma unroll
            for (int j = 0; j < SITES; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) yi[j][c] = acc[j][c] = y[j][c];
#pragma unroll 1
            for (int st = 0; st < 4; ++st) {
                const R ha = st == 0 || st == 3 ? h6 : h3, hn = st < 2 ? h2 : h;
                C k[SITES][4];
                rhs(yi, k, tc + 3 * n + (st + 1) / 2);
#pragma unroll
                for (int j = 0; j < SITES; ++j)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        acc[j][c] = cadd(acc[j][c], cscale(k[j][c], ha));
                        yi[j][c] = cadd(y[j][c], cscale(k[j][c], hn));
                    }
            }
#pragma unroll
            for (int j = 0; j < SITES; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) y[j][c] = cscale(acc[j][c], msk[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < SITES; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) gstore<C>(py, c * (long long)N + 4 * T * j, y[j][c]);
}

// Kernel table of one (precision, N) instantiation.
struct RowVariant { const void* stage[4]; const void* dp5[6]; int threads, rows; size_t lds; };   // RK4 / Dormand-Prince stages
struct CdVariant { const void* fn[2]; int threads, w; size_t lds; };   // [axis - 1]: y writes G, z adds to it
struct ColVariant { const void* fn[2]; int threads, w; size_t lds; };   // [axis - 1]
struct StepRadices { int n, r[8]; };   // a plan's radices
struct SizeKernels {
    StepRadices row_plan, col_plan;   // of the stepping passes (their twiddle tables' order)
    RowVariant row;                // the stage row pass
    CdVariant cd[NVAR];            // the stepping column passes, by variant
    const void* row_t[3][2];       // whole-state transforms along x: forward, forward with a phase, inverse; cached or streaming
    const void* col_t[2][2];       // along y, z: forward, inverse
    int col_tv[2];                 // and the stepping variant whose tiles these have
    const void* row_other[ROW_NMODES];  // whole-state row modes that mix components
    int row0_threads, row0_rows;
    size_t row0_lds;
    ColVariant col;                // last axis with -i H0 or the free evolution
    const void* line;              // 1D whole-loop kernel
    int line_threads;
    size_t line_lds;               // its dynamic LDS without the profiles of terms beyond LINE_TERMS
};

template <class R, int N>
RowVariant make_row_variant() {
    using VC = RdVar<R, N>;
    return RowVariant{{(const void*)row_d_kernel<R, N, 0, 0>, (const void*)row_d_kernel<R, N, 0, 1>,
                       (const void*)row_d_kernel<R, N, 0, 2>, (const void*)row_d_kernel<R, N, 0, 3>},
                      {(const void*)row_d_kernel<R, N, 0, 4>, (const void*)row_d_kernel<R, N, 0, 5>,
                       (const void*)row_d_kernel<R, N, 0, 6>, (const void*)row_d_kernel<R, N, 0, 7>,
                       (const void*)row_d_kernel<R, N, 0, 8>, (const void*)row_d_kernel<R, N, 0, 9>},
                      VC::THREADS, VC::ROWS, VC::BYTES};
}
template <class R, int N, int V>
CdVariant make_cd_variant() {
    using VC = CdVar<R, N, V>;
    CdVariant c;
    c.fn[0] = (const void*)col_d_kernel<R, N, V, 1, 0>;
    c.fn[1] = (const void*)col_d_kernel<R, N, V, 2, 1>;
    c.threads = VC::THREADS;
    c.w = VC::W;
    c.lds = VC::BYTES;
    return c;
}
template <class R, int N>
ColVariant make_col_variant() {
    ColVariant c;
    if constexpr (HdVar<R, N>::FITS) {
        using VC = HdVar<R, N>;
        c.fn[0] = (const void*)col_h0_kernel<R, N, 1>;
        c.fn[1] = (const void*)col_h0_kernel<R, N, 2>;
        c.threads = VC::THREADS;
        c.w = VC::W;
        c.lds = VC::BYTES;
    } else {
        using VC = ColVar<R, N>;
        c.fn[0] = (const void*)col_kernel<R, N, 1>;
        c.fn[1] = (const void*)col_kernel<R, N, 2>;
        c.threads = VC::THREADS;
        c.w = VC::W;
        c.lds = VC::BYTES;
    }
    return c;
}

template <class P> StepRadices radices() {
    StepRadices s;
    s.n = P::NR;
    for (int j = 0; j < P::NR; ++j) s.r[j] = P::R[j];
    return s;
}
template <class R, int N>
SizeKernels make_size_kernels() {
    SizeKernels k;
    k.row_plan = radices<StepPlan<N>>();
    k.col_plan = radices<ColPlan<N>>();
    k.row = make_row_variant<R, N>();
    // (a width that T or the LDS caps is the narrower variant's kernel again)
    k.cd[0] = make_cd_variant<R, N, 0>();
    if constexpr (CdVar<R, N, 1>::W == CdVar<R, N, 0>::W) k.cd[1] = k.cd[0];
    else k.cd[1] = make_cd_variant<R, N, 1>();
    if constexpr (CdVar<R, N, 2>::W == CdVar<R, N, 1>::W) k.cd[2] = k.cd[1];
    else k.cd[2] = make_cd_variant<R, N, 2>();
    k.col = make_col_variant<R, N>();
    k.row_t[0][0] = (const void*)row_t_kernel<R, N, -1, false, false>;
    k.row_t[0][1] = (const void*)row_t_kernel<R, N, -1, false, true>;
    k.row_t[1][0] = (const void*)row_t_kernel<R, N, -1, true, false>;
    k.row_t[1][1] = (const void*)row_t_kernel<R, N, -1, true, true>;
    k.row_t[2][0] = (const void*)row_t_kernel<R, N, +1, false, false>;
    k.row_t[2][1] = (const void*)row_t_kernel<R, N, +1, false, true>;
    k.col_t[0][0] = (const void*)col_t_kernel<R, N, 1, -1>;
    k.col_t[0][1] = (const void*)col_t_kernel<R, N, 1, +1>;
    k.col_t[1][0] = (const void*)col_t_kernel<R, N, 2, -1>;
    k.col_t[1][1] = (const void*)col_t_kernel<R, N, 2, +1>;
    k.col_tv[0] = col_t_tile(1, N);
    k.col_tv[1] = col_t_tile(2, N);
    k.row_other[ROW_FWD] = k.row_other[ROW_FWDPH] = nullptr;
    k.row_other[ROW_STAGE] = nullptr;
    k.row_other[ROW_INV] = (const void*)row_kernel<R, N, ROW_INV>;
    k.row_other[ROW_RHS] = (const void*)row_kernel<R, N, ROW_RHS>;
    k.row_other[ROW_SRC] = (const void*)row_kernel<R, N, ROW_SRC>;
    k.row0_threads = RowVar<R, N>::THREADS;
    k.row0_rows = RowVar<R, N>::ROWS;
    k.row0_lds = RowVar<R, N>::BYTES;
    k.line = (const void*)line_kernel<R, N>;
    k.line_threads = LineVar<R, N>::THREADS;
    k.line_lds = LineVar<R, N>::BASE_BYTES;
    return k;
}

}  // namespace swf
