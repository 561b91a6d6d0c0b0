// Element form of the fine operator: y = (K + lambda M) v by sum
// factorisation over the elements instead of a product with the assembled
// rows.  The operator is that of the fine-level assembly (tensor basis, p + 2
// Gauss points per direction, trilinear geometry, identity rows and columns at
// the constrained nodes), evaluated from the element corners:
//
//  1. element_kernel: a block gathers v on a few elements, takes it to the
//     quadrature points one direction at a time (z, y, x), multiplies by the
//     geometric factors, which each thread forms from the element's trilinear
//     coefficients, and goes back the same way.  The (p + 1)^3 results of each
//     element go to the element vector ev.
//  2. element_node_kernel: every node adds its entries of ev in ascending
//     element order (no atomics: bitwise reproducible) and runs the fused row
//     epilogue of the product (smoother step, residual, dot partials).
//
// Why: the assembled rows hold (p + 2)^3 nonzeros of 10 to 12 bytes per node,
// read once per product: 4.4 GB at 32^3, p = 4, 0.62 ms at the rate of a plain
// read stream and 0.94 ms measured.  The element form reads the element map,
// the corners and the vectors (about 0.15 GB there).  Its first kernel takes
// 60 us there in FP64 and 36 us in FP32 (990 vector instructions per wave, half
// of the vector ALUs' time in FP64 at three waves per SIMD, 83 % of it in FP32
// at five; with full tables instead of the even and odd parts 91 and 40 us:
// the tables then spilled from the scalar registers), the second 20 to 28 us
// (its vectors at about 6 TB/s).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>

#include "kernels.h"
#include "row_epilogue.h"

namespace giamg {

namespace {

constexpr int NODE_THREADS = 256;

// Rows (and columns) of an element's matrix in the dense form: (p + 1)^3 to whole tiles of 16.
constexpr int dense_rows(int p) { return ((p + 1) * (p + 1) * (p + 1) + 15) / 16 * 16; }
// Where entry (i, j) of an nlp x nlp element matrix lies in its tiles: column
// step t, row tile r, lane 16 g + row, column b of the lane's KB.
template <typename T>
__host__ __device__ constexpr int element_tile(int nlp, int i, int j) {
    const int kb = 16 / (int)sizeof(T);
    const int t = j / (4 * kb), g = j / kb % 4, b = j % kb;
    return ((t * (nlp / 16) + i / 16) * 64 + g * 16 + i % 16) * kb + b;
}

// 120 bytes: the launch's own arguments (the grid's size) follow in the same 64 bytes as
// the last ones; eight bytes more cost 0.2 us a launch (a third line of arguments).
template <typename T>
struct ElemArgs {
    int64_t ne = 0;
    const int32_t* map = nullptr;    // [ne][nl] node of each local position, -1 constrained
    const T* v = nullptr;
    T* ev = nullptr;                 // [ne][nl]
    const T* coef = nullptr;         // [elem_coefs][ne] trilinear coefficients
    const T* tabs = nullptr;         // 1-D tables (element_tables)
    T lambda = 0, ps = 1, pt = -1;   // pair transform of the inner positions (element_tables)
    int k = 1;                       // columns of v ([n][k]) and ev ([ne][nl][k])
    int e0 = 0;                      // UNIT: first element of this launch
    const int* stop = nullptr;
    const int* run = nullptr;        // when set and zero, nothing to do
    const double* vnz = nullptr;     // when set and zero, v is +0: nothing to do
    double* mat = nullptr;           // UNIT: element matrices in tiles
    float* mat32 = nullptr;
};

static_assert(sizeof(ElemArgs<double>) <= 120, "kernel arguments of element_kernel");

// Every multiply-add is written out, so each instance of the kernel gives the
// same bits (see the contract pragma at each function).
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double recip(double d) {
    // reciprocal estimate and two Newton steps (1 ulp)
    double r = __builtin_amdgcn_rcp(d);
    r = mad(mad(-d, r, 1.0), r, r);
    return mad(mad(-d, r, 1.0), r, r);
}
__device__ __forceinline__ float recip(float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    return mad(mad(-d, r, 1.0f), r, r);
}

// Thread counts and elements per block.  The quadrature step takes (p + 2)^2
// lanes per element: narrow blocks are the whole waves one element needs (or
// several elements in one wave), wide blocks fill 256 threads with elements.
// Wide where that fills more lanes (p = 3, 4, 5, 7, 8) and the mesh has a wide
// block for every CU.  Measured with the full tables (product, FP64, wide /
// narrow): 32^3 p = 4 116 / 155 us, 12^3 p = 7 51 / 75, 13^3 p = 5 23 / 29; with
// fewer elements 8^3 p = 4 16 / 13; 40^3 p = 2 49 / 45.
constexpr int64_t ELEM_WIDE_LANES = 65536;   // 256 lanes on each of 256 CUs
constexpr bool elem_wide_pays(int p) { return p == 3 || p == 4 || p == 5 || p == 7 || p == 8; }
template <int P>
constexpr int elem_threads(bool wide) {
    constexpr int q2 = (P + 2) * (P + 2);
    return wide ? 256 : (q2 + 63) / 64 * 64;
}
template <int P>
constexpr int elem_per_block(bool wide) { return elem_threads<P>(wide) / ((P + 2) * (P + 2)); }

// 1-D contractions in even and odd parts.  A line of N nodal values u becomes
// N / 2 pairs (e, o) of position k and its mirror N - 1 - k (and the middle
// value, which is even); the values at the Gauss points q and Q - 1 - q are
// then (even part) +- (odd part), and likewise for the derivative, whose even
// part comes from the odd coefficients.  This halves the multiply-adds of both
// tables, and one q's entries (2 N numbers: Le, Lo, De, Do) are all a step
// needs at a time, so they stay in scalar registers.
template <typename T, int N>
struct Line {
    static constexpr int H = (N + 1) / 2, O = N / 2;
    T e[H], o[O > 0 ? O : 1];
};
template <typename T, int N>
__device__ __forceinline__ void to_parity(const T* u, Line<T, N>& l, T ps, T pt) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        const T a = u[k], b = u[N - 1 - k];
        if (k == 0) {
            l.e[0] = a + b;
            l.o[0] = a - b;
        } else {
            l.e[k] = mad(ps, b, a);
            l.o[k] = mad(pt, b, ps * a);
        }
    }
    if constexpr (N % 2) l.e[N / 2] = u[N / 2];
}
template <typename T, int N>
__device__ __forceinline__ void from_parity(const Line<T, N>& l, T* u, T ps, T pt) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < N / 2; ++k) {
        if (k == 0) {
            u[0] = l.e[0] + l.o[0];
            u[N - 1] = l.e[0] - l.o[0];
        } else {
            u[k] = mad(ps, l.o[k], l.e[k]);
            u[N - 1 - k] = mad(pt, l.o[k], ps * l.e[k]);
        }
    }
    if constexpr (N % 2) u[N / 2] = l.e[N / 2];
}
// The table entries of one Gauss point pair: [H] Le, [O] Lo, [H] De, [O] Do.
// In the constant address space: uniform loads into scalar registers.
template <typename T>
using const_ptr = const T __attribute__((address_space(4)))*;
template <typename T, int N>
struct Rec {
    const_ptr<T> p;
    __device__ __forceinline__ T le(int k) const { return p[k]; }
    __device__ __forceinline__ T lo(int k) const { return p[(N + 1) / 2 + k]; }
    __device__ __forceinline__ T de(int k) const { return p[N + k]; }
    __device__ __forceinline__ T dod(int k) const { return p[N + (N + 1) / 2 + k]; }
};
template <typename T, int N>
__device__ __forceinline__ T even_l(const Rec<T, N>& r, const Line<T, N>& l) {
    T s = r.le(0) * l.e[0];
#pragma unroll
    for (int k = 1; k < (N + 1) / 2; ++k) s = mad(r.le(k), l.e[k], s);
    return s;
}
template <typename T, int N>
__device__ __forceinline__ T odd_l(const Rec<T, N>& r, const Line<T, N>& l) {
    T s = r.lo(0) * l.o[0];
#pragma unroll
    for (int k = 1; k < N / 2; ++k) s = mad(r.lo(k), l.o[k], s);
    return s;
}
template <typename T, int N>   // derivative: even in q
__device__ __forceinline__ T even_d(const Rec<T, N>& r, const Line<T, N>& l) {
    T s = r.dod(0) * l.o[0];
#pragma unroll
    for (int k = 1; k < N / 2; ++k) s = mad(r.dod(k), l.o[k], s);
    return s;
}
template <typename T, int N>   // derivative: odd in q
__device__ __forceinline__ T odd_d(const Rec<T, N>& r, const Line<T, N>& l) {
    T s = r.de(0) * l.e[0];
#pragma unroll
    for (int k = 1; k < (N + 1) / 2; ++k) s = mad(r.de(k), l.e[k], s);
    return s;
}
// Transposes: a Gauss pair's even and odd parts into the coefficients.
template <typename T, int N>
__device__ __forceinline__ void add_l(const Rec<T, N>& r, T ev, T od, Line<T, N>& l) {
#pragma unroll
    for (int k = 0; k < (N + 1) / 2; ++k) l.e[k] = mad(r.le(k), ev, l.e[k]);
#pragma unroll
    for (int k = 0; k < N / 2; ++k) l.o[k] = mad(r.lo(k), od, l.o[k]);
}
template <typename T, int N>
__device__ __forceinline__ void add_d(const Rec<T, N>& r, T ev, T od, Line<T, N>& l) {
#pragma unroll
    for (int k = 0; k < (N + 1) / 2; ++k) l.e[k] = mad(r.de(k), od, l.e[k]);
#pragma unroll
    for (int k = 0; k < N / 2; ++k) l.o[k] = mad(r.dod(k), ev, l.o[k]);
}
template <typename T, int N>
__device__ __forceinline__ void clear(Line<T, N>& l) {
#pragma unroll
    for (int k = 0; k < (N + 1) / 2; ++k) l.e[k] = T(0);
#pragma unroll
    for (int k = 0; k < N / 2; ++k) l.o[k] = T(0);
}
// The same pointer, opaque to the compiler: the table entries of one step are
// loaded again in the next instead of being held (and spilled) across it.
template <typename T>
__device__ __forceinline__ const_ptr<T> fresh(const T* p) {
    asm volatile("" : "+s"(p));
    return (const_ptr<T>)(uintptr_t)p;
}

// A block of NT threads works on V elements side by side.  COLS: block vectors
// of a.k columns, the V elements are (element, column) pairs, column fastest.
// UNIT (FP64, a.k = nl): the columns are the element's unit vectors and the
// results, the columns of its matrix, go to the tiles of both precisions
// (element_tile) instead of ev.
template <typename T, int P, int NT, int V, bool COLS, bool UNIT = false>
__global__ void __launch_bounds__(NT) element_kernel(ElemArgs<T> a) {
#pragma clang fp contract(off)
    if (a.run != nullptr && *a.run == 0) return;
    if (a.vnz != nullptr && *a.vnz == 0.0) return;
    const int done = a.stop != nullptr ? *a.stop : 0;   // looked at once the loads are under way
    constexpr int N = P + 1, Q = P + 2, N2 = N * N, NL = N2 * N, Q2 = Q * Q;
    constexpr int H = (Q + 1) / 2;                 // Gauss pairs, the middle point one of its own
    static_assert(V * Q2 <= NT, "block shape");
    constexpr int LINES = NT / V, CITER = (NL + LINES - 1) / LINES;   // COLS: nodal values per thread
    constexpr int ITER = (V * NL + NT - 1) / NT;
    constexpr int UNROLL = 2 * N * H * (int)sizeof(T) <= 240 ? H : 1;   // one step's tables in 60 scalar registers
    // one region, element fastest: nodal values [i][j][k], then [2][qz][i][j],
    // then [3][i][qy][qz], and back; every step has at most one line per
    // thread, reads it, waits, and writes its results over the others' inputs
    __shared__ T sh[V * 3 * N * Q2];
    const int tid = threadIdx.x;
    const int v = tid % V, line = tid / V;
    const int64_t first = (UNIT ? (int64_t)a.e0 * a.k : 0) + xcd_block(blockIdx.x, gridDim.x) * V;   // element, or pair
    const int64_t total = COLS ? a.ne * a.k : a.ne;
    const int64_t mine = min(first + v, total - 1);
    const int64_t e = COLS ? (total <= (int64_t)UINT32_MAX ? (uint32_t)mine / (uint32_t)a.k : mine / a.k) : mine;
    const int64_t col0 = COLS ? mine - e * a.k : 0;
    const int cnt = (int)min((int64_t)V, total - first) * NL;
    const T ps = a.ps, pt = a.pt;
    // gather
    if constexpr (COLS) {
        const int32_t* __restrict__ map = a.map + e * NL;
        const T* __restrict__ vec = a.v + col0;
        int32_t g[CITER];
        T x[CITER];
        if constexpr (UNIT) {
#pragma unroll
            for (int it = 0; it < CITER; ++it) {
                g[it] = 0;
                x[it] = line + it * LINES == (int)col0 ? T(1) : T(0);
            }
        } else {
#pragma unroll
            for (int it = 0; it < CITER; ++it) g[it] = map[min(line + it * LINES, NL - 1)];
#pragma unroll
            for (int it = 0; it < CITER; ++it) x[it] = vec[(int64_t)max(g[it], 0) * a.k];
        }
#pragma unroll
        for (int it = 0; it < CITER; ++it) {
            const int loc = line + it * LINES;
            if (line < LINES && loc < NL) sh[loc * V + v] = g[it] >= 0 ? x[it] : T(0);
        }
    } else {
        const int32_t* __restrict__ map = a.map + first * NL;
        const T* __restrict__ vec = a.v;
        int32_t g[ITER];
        T x[ITER];
#pragma unroll
        for (int it = 0; it < ITER; ++it) g[it] = map[min(tid + it * NT, cnt - 1)];
#pragma unroll
        for (int it = 0; it < ITER; ++it) x[it] = vec[max(g[it], 0)];
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int t = tid + it * NT;
            if (t < V * NL) sh[(t % NL) * V + t / NL] = g[it] >= 0 ? x[it] : T(0);
        }
    }
    T c[elem_coefs<T>()];   // the element's geometry, used at the quadrature points
#pragma unroll
    for (int m = 0; m < elem_coefs<T>(); ++m) c[m] = a.coef[m * a.ne + e];
    __syncthreads();
    if (done) return;
    // z: nodal lines to Gauss points, values and derivatives
    {
        const const_ptr<T> tab = fresh(a.tabs);
        T u[N];
        Line<T, N> l;
        if (line < N2) {
#pragma unroll
            for (int k = 0; k < N; ++k) u[k] = sh[(line * N + k) * V + v];
        }
        to_parity<T, N>(u, l, ps, pt);
        __syncthreads();
        if (line < N2) {
#pragma unroll UNROLL
            for (int q = 0; q < H; ++q) {
                const Rec<T, N> r{tab + q * 2 * N};
                const T ve = even_l(r, l), vo = odd_l(r, l), de = even_d(r, l), dd = odd_d(r, l);
                sh[(q * N2 + line) * V + v] = ve + vo;
                sh[((Q + q) * N2 + line) * V + v] = de + dd;
                if (Q % 2 == 0 || q < H - 1) {
                    sh[((Q - 1 - q) * N2 + line) * V + v] = ve - vo;
                    sh[((2 * Q - 1 - q) * N2 + line) * V + v] = de - dd;
                }
            }
        }
    }
    __syncthreads();
    // y: lines (qz, i)
    const int li = line % N, lq = line / N;
    {
        const const_ptr<T> tab = fresh(a.tabs);
        T u[N];
        Line<T, N> l0, l1;
        if (line < N * Q) {
#pragma unroll
            for (int j = 0; j < N; ++j) u[j] = sh[(line * N + j) * V + v];
            to_parity<T, N>(u, l0, ps, pt);
#pragma unroll
            for (int j = 0; j < N; ++j) u[j] = sh[(Q * N2 + line * N + j) * V + v];
            to_parity<T, N>(u, l1, ps, pt);
        }
        __syncthreads();
        if (line < N * Q) {
            T* out = sh + (li * Q2 + lq) * V + v;
#pragma unroll UNROLL
            for (int q = 0; q < H; ++q) {
                const Rec<T, N> r{tab + q * 2 * N};
                const T ve = even_l(r, l0), vo = odd_l(r, l0), de = even_d(r, l0), dd = odd_d(r, l0);
                const T ze = even_l(r, l1), zo = odd_l(r, l1);
                out[q * Q * V] = ve + vo;
                out[(N * Q2 + q * Q) * V] = de + dd;
                out[(2 * N * Q2 + q * Q) * V] = ze + zo;
                if (Q % 2 == 0 || q < H - 1) {
                    out[(Q - 1 - q) * Q * V] = ve - vo;
                    out[(N * Q2 + (Q - 1 - q) * Q) * V] = de - dd;
                    out[(2 * N * Q2 + (Q - 1 - q) * Q) * V] = ze - zo;
                }
            }
        }
    }
    __syncthreads();
    // x, the quadrature points of one x line per thread, and x back
    if (line < Q2) {
        const const_ptr<T> tab = fresh(a.tabs);
        const const_ptr<T> gq = tab + 2 * N * H, wq = gq + Q;
        const T* __restrict__ lgq = a.tabs + 2 * N * H;   // per lane
        const T eta = lgq[line / Q], zeta = lgq[line % Q];
        const T wyz = lgq[Q + line / Q] * lgq[Q + line % Q];
        // Columns of the Jacobian: ax = dx/dxi is fixed on the line, b = dx/deta
        // and d = dx/dzeta are linear in xi.  gx = b x d, gy = d x ax,
        // gz = ax x b are the reference gradients times the determinant.
        T ax[3], b0[3], b1[3], d0[3], d1[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            // c: xi, eta, zeta, xi eta, xi zeta, eta zeta, xi eta zeta
            ax[m] = mad(mad(c[18 + m], eta, c[12 + m]), zeta, mad(c[9 + m], eta, c[m]));
            b0[m] = mad(c[15 + m], zeta, c[3 + m]);
            b1[m] = mad(c[18 + m], zeta, c[9 + m]);
            d0[m] = mad(c[15 + m], eta, c[6 + m]);
            d1[m] = mad(c[18 + m], eta, c[12 + m]);
        }
        T g0[3], g1[3], g2[3], y0[3], y1[3], z0[3], z1[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const int m1 = (m + 1) % 3, m2 = (m + 2) % 3;
            g0[m] = mad(b0[m1], d0[m2], -(b0[m2] * d0[m1]));
            g1[m] = mad(b0[m1], d1[m2], -(b0[m2] * d1[m1])) + mad(b1[m1], d0[m2], -(b1[m2] * d0[m1]));
            g2[m] = mad(b1[m1], d1[m2], -(b1[m2] * d1[m1]));
            y0[m] = mad(d0[m1], ax[m2], -(d0[m2] * ax[m1]));
            y1[m] = mad(d1[m1], ax[m2], -(d1[m2] * ax[m1]));
            z0[m] = mad(ax[m1], b0[m2], -(ax[m2] * b0[m1]));
            z1[m] = mad(ax[m1], b1[m2], -(ax[m2] * b1[m1]));
        }
        const T t0 = mad(ax[2], g0[2], mad(ax[1], g0[1], ax[0] * g0[0]));
        const T t1 = mad(ax[2], g1[2], mad(ax[1], g1[1], ax[0] * g1[0]));
        const T t2 = mad(ax[2], g2[2], mad(ax[1], g2[1], ax[0] * g2[0]));
        T* col = sh + line * V + v;
        Line<T, N> u0, u1, u2, o0, o1, o2;
        {
            T u[N];
#pragma unroll
            for (int i = 0; i < N; ++i) u[i] = col[i * Q2 * V];
            to_parity<T, N>(u, u0, ps, pt);
#pragma unroll
            for (int i = 0; i < N; ++i) u[i] = col[(N + i) * Q2 * V];
            to_parity<T, N>(u, u1, ps, pt);
#pragma unroll
            for (int i = 0; i < N; ++i) u[i] = col[(2 * N + i) * Q2 * V];
            to_parity<T, N>(u, u2, ps, pt);
        }
        clear(o0);
        clear(o1);
        clear(o2);
#pragma unroll UNROLL
        for (int q = 0; q < H; ++q) {
            const Rec<T, N> r{tab + q * 2 * N};
            const T xi = gq[q], w = wq[q] * wyz;
            // FP32: h and lambda h^3 of the scaled element (exact: powers of two)
            T ws = w, mass = a.lambda;
            if constexpr (elem_coefs<T>() > ELEM_COEF) {
                ws = w * c[ELEM_COEF];
                mass = c[ELEM_COEF + 1];
            }
            const bool pair = Q % 2 == 0 || q < H - 1;
            const T ve = even_l(r, u0), vo = odd_l(r, u0);
            const T xe = even_d(r, u0), xo = odd_d(r, u0);
            const T ye = even_l(r, u1), yo = odd_l(r, u1);
            const T ze = even_l(r, u2), zo = odd_l(r, u2);
            const T te = mad(t2, xi * xi, t0), to = t1 * xi;
            T ge[3], go[3];
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                ge[m] = mad(g2[m], xi * xi, g0[m]);
                go[m] = g1[m] * xi;
            }
            T f[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && !pair) {
                    f[1][0] = f[1][1] = f[1][2] = f[1][3] = T(0);
                    continue;
                }
                const T x = h == 0 ? xi : -xi;
                T gx[3], gy[3], gz[3], W[3];
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    gx[m] = h == 0 ? ge[m] + go[m] : ge[m] - go[m];
                    gy[m] = mad(y1[m], x, y0[m]);
                    gz[m] = mad(z1[m], x, z0[m]);
                }
                const T det = h == 0 ? te + to : te - to;
                const T ux = h == 0 ? xe + xo : xe - xo, uy = h == 0 ? ye + yo : ye - yo;
                const T uz = h == 0 ? ze + zo : ze - zo, val = h == 0 ? ve + vo : ve - vo;
                const T s = ws * recip(det);
#pragma unroll
                for (int m = 0; m < 3; ++m) W[m] = s * mad(gz[m], uz, mad(gy[m], uy, gx[m] * ux));
                f[h][0] = mad(gx[2], W[2], mad(gx[1], W[1], gx[0] * W[0]));
                f[h][1] = mad(gy[2], W[2], mad(gy[1], W[1], gy[0] * W[0]));
                f[h][2] = mad(gz[2], W[2], mad(gz[1], W[1], gz[0] * W[0]));
                f[h][3] = (mass * w) * (det * val);
            }
            add_d(r, f[0][0] + f[1][0], f[0][0] - f[1][0], o0);
            add_l(r, f[0][3] + f[1][3], f[0][3] - f[1][3], o0);
            add_l(r, f[0][1] + f[1][1], f[0][1] - f[1][1], o1);
            add_l(r, f[0][2] + f[1][2], f[0][2] - f[1][2], o2);
        }
        {
            T u[N];
            from_parity<T, N>(o0, u, ps, pt);
#pragma unroll
            for (int i = 0; i < N; ++i) col[i * Q2 * V] = u[i];
            from_parity<T, N>(o1, u, ps, pt);
#pragma unroll
            for (int i = 0; i < N; ++i) col[(N + i) * Q2 * V] = u[i];
            from_parity<T, N>(o2, u, ps, pt);
#pragma unroll
            for (int i = 0; i < N; ++i) col[(2 * N + i) * Q2 * V] = u[i];
        }
    }
    __syncthreads();
    // y back
    {
        const const_ptr<T> tab = fresh(a.tabs);
        Line<T, N> l0, l1;
        clear(l0);
        clear(l1);
        if (line < N * Q) {
            const T* in = sh + (li * Q2 + lq) * V + v;
#pragma unroll UNROLL
            for (int q = 0; q < H; ++q) {
                const Rec<T, N> r{tab + q * 2 * N};
                const bool pair = Q % 2 == 0 || q < H - 1;
                const T a0 = in[q * Q * V], a1 = in[(N * Q2 + q * Q) * V], a2 = in[(2 * N * Q2 + q * Q) * V];
                const T b0 = pair ? in[(Q - 1 - q) * Q * V] : T(0);
                const T b1 = pair ? in[(N * Q2 + (Q - 1 - q) * Q) * V] : T(0);
                const T b2 = pair ? in[(2 * N * Q2 + (Q - 1 - q) * Q) * V] : T(0);
                add_l(r, a0 + b0, a0 - b0, l0);
                add_d(r, a1 + b1, a1 - b1, l0);
                add_l(r, a2 + b2, a2 - b2, l1);
            }
        }
        __syncthreads();
        if (line < N * Q) {
            T u[N];
            from_parity<T, N>(l0, u, ps, pt);
#pragma unroll
            for (int j = 0; j < N; ++j) sh[(line * N + j) * V + v] = u[j];
            from_parity<T, N>(l1, u, ps, pt);
#pragma unroll
            for (int j = 0; j < N; ++j) sh[(Q * N2 + line * N + j) * V + v] = u[j];
        }
    }
    __syncthreads();
    // z back
    {
        const const_ptr<T> tab = fresh(a.tabs);
        Line<T, N> l;
        clear(l);
        if (line < N2) {
#pragma unroll UNROLL
            for (int q = 0; q < H; ++q) {
                const Rec<T, N> r{tab + q * 2 * N};
                const bool pair = Q % 2 == 0 || q < H - 1;
                const T a0 = sh[(q * N2 + line) * V + v], a1 = sh[((Q + q) * N2 + line) * V + v];
                const T b0 = pair ? sh[((Q - 1 - q) * N2 + line) * V + v] : T(0);
                const T b1 = pair ? sh[((2 * Q - 1 - q) * N2 + line) * V + v] : T(0);
                add_l(r, a0 + b0, a0 - b0, l);
                add_d(r, a1 + b1, a1 - b1, l);
            }
        }
        __syncthreads();
        if (line < N2) {
            T u[N];
            from_parity<T, N>(l, u, ps, pt);
#pragma unroll
            for (int k = 0; k < N; ++k) sh[(line * N + k) * V + v] = u[k];
        }
    }
    __syncthreads();
    if constexpr (UNIT) {
        constexpr int NLP = dense_rows(P);
#pragma unroll
        for (int it = 0; it < CITER; ++it) {
            const int loc = line + it * LINES;
            if (line < LINES && loc < NL && first + v < total) {
                const T x = sh[loc * V + v];
                a.mat[e * NLP * NLP + element_tile<double>(NLP, loc, (int)col0)] = x;
                if (a.mat32 != nullptr)
                    a.mat32[e * NLP * NLP + element_tile<float>(NLP, loc, (int)col0)] = (float)x;
            }
        }
    } else if constexpr (COLS) {
        T* __restrict__ ev = a.ev + e * NL * a.k + col0;
#pragma unroll
        for (int it = 0; it < CITER; ++it) {
            const int loc = line + it * LINES;
            if (line < LINES && loc < NL && first + v < total) ev[(int64_t)loc * a.k] = sh[loc * V + v];
        }
    } else {
        T* __restrict__ ev = a.ev + first * NL;
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int t = tid + it * NT;
            if (t < cnt) ev[t] = sh[(t % NL) * V + t / NL];
        }
    }
}

// One thread per node: its entries of ev in ascending element order, then the
// row epilogue.  A node without entries is constrained (identity row).
template <typename T, int MODE>
__global__ void __launch_bounds__(NODE_THREADS) element_node_kernel(SpmvArgs<T> a, const int32_t* __restrict__ ptr,
                                                                    const int32_t* __restrict__ ent,
                                                                    const T* __restrict__ ev) {
    constexpr int U = 4;   // entries under way: a vertex has 8, most nodes one or two
    const int done = a.stop != nullptr ? *a.stop : 0;
    const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
    const int64_t row = lb * NODE_THREADS + threadIdx.x;
    double dot = 0.0, dot2 = 0.0;
    if (row < a.n) {
        RowIn<T> in{};
        epilogue_load<T, MODE>(a, row, in);
        T y = 0;
        bool product = true;
        if constexpr (MODE == SPMV_RINIT) product = !(a.vnz != nullptr && *a.vnz == 0.0);
        if (product) {
            const int32_t s = ptr[row], e = ptr[row + 1];
            for (int32_t j = s; j < e; j += U) {
                int32_t at[U];
                T x[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j + u < e) at[u] = ent[j + u];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j + u < e) x[u] = ev[at[u]];
#pragma unroll
                for (int u = 0; u < U; ++u) y = j + u < e ? y + x[u] : y;
            }
            if (s == e) y = a.v[row];
        }
        if (!done) epilogue_store<T, MODE>(a, row, y, in, dot, dot2);
    }
    if constexpr (has_partials<MODE>()) {
        __shared__ double red[2 * NODE_THREADS / WAVE];
        block_sum_to0<NODE_THREADS, n_partials<T, MODE>()>(red, threadIdx.x, dot, dot2);
        if (threadIdx.x == 0 && !done) {
            a.partial[lb] = dot;
            if (n_partials<T, MODE>() == 2) a.partial[a.nblk + lb] = dot2;
        }
    }
}

template <typename T, int P, bool WIDE>
void launch_element_kernel(const ElemArgs<T>& a, hipEvent_t ev_start, hipStream_t s) {
    constexpr int EPB = elem_per_block<P>(WIDE), NT = elem_threads<P>(WIDE);
    const dim3 grid((unsigned)((a.ne + EPB - 1) / EPB)), block(NT);
    if (ev_start != nullptr)
        hipExtLaunchKernelGGL((element_kernel<T, P, NT, EPB, false>), grid, block, 0, s, ev_start, nullptr, 0, a);
    else
        element_kernel<T, P, NT, EPB, false><<<grid, block, 0, s>>>(a);
}

template <typename T, int P>
void launch_element_columns(const ElemArgs<T>& a, hipStream_t s) {
    constexpr int NT = P <= 9 ? 256 : 192, V = NT / ((P + 2) * (P + 2));
    const int64_t pairs = a.ne * a.k;
    element_kernel<T, P, NT, V, true><<<(unsigned)((pairs + V - 1) / V), NT, 0, s>>>(a);
}

template <typename T>
void launch_element_order(int p, const ElemArgs<T>& a, hipEvent_t ev_start, hipStream_t s) {
#define GIAMG_ELEM(P)                                                                              \
    case P:                                                                                        \
        if constexpr (elem_wide_pays(P)) {                                                         \
            if (a.ne * (P + 2) * (P + 2) >= ELEM_WIDE_LANES) {                                     \
                launch_element_kernel<T, P, true>(a, ev_start, s);                                 \
                break;                                                                             \
            }                                                                                      \
        }                                                                                          \
        launch_element_kernel<T, P, false>(a, ev_start, s);                                        \
        break;
    switch (p) {
        GIAMG_ELEM(2) GIAMG_ELEM(3) GIAMG_ELEM(4) GIAMG_ELEM(5) GIAMG_ELEM(6)
        GIAMG_ELEM(7) GIAMG_ELEM(8) GIAMG_ELEM(9) GIAMG_ELEM(10)
        default: throw Error(GIAMG_EINVAL, "element form of an unsupported order");
    }
#undef GIAMG_ELEM
    GIAMG_HIP(hipGetLastError());
}

template <typename T>
void launch_element_block_order(int p, const ElemArgs<T>& a, hipStream_t s) {
    if (a.k == 1) {
        launch_element_order<T>(p, a, nullptr, s);
        return;
    }
#define GIAMG_ELEM(P) \
    case P: launch_element_columns<T, P>(a, s); break;
    switch (p) {
        GIAMG_ELEM(5) GIAMG_ELEM(6) GIAMG_ELEM(7) GIAMG_ELEM(8) GIAMG_ELEM(9) GIAMG_ELEM(10)
        default: throw Error(GIAMG_EINVAL, "element form of an unsupported order");
    }
#undef GIAMG_ELEM
    GIAMG_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// Dense form of the block products (p <= 4): an element's matrix, stored once,
// times its nodal values of 16 columns by matrix instructions.  The matrix is
// cut into tiles of 16 rows and four lane groups of KB columns, in the order the
// instruction's left operand wants: lane 16 g + r of a tile holds row r and
// columns KB g .. KB g + KB - 1 in one 16-byte load (KB = 2 in FP64, 4 in FP32),
// and instruction b of the tile sums over the columns KB g + b of the four
// groups.  The right operand's lane 16 g + c holds column c of the same nodes.
// RS: waves that share the rows of one element and 16 columns (few columns);
// the block's four waves cover 4 / RS tiles of 16 columns.  Every result is the
// same sum in the same order whatever k, so a column's bits do not depend on it.
// With RS = 1 the waves share the matrix through LDS in chunks of 16 KB, the next
// one on its way from memory meanwhile; with RS > 1 each wave reads its own rows.
//
// Measured at k = 64: 20^3 p = 3 (0.26 GB of FP64 matrices and as much of results)
// 113 us FP64 and 69 us FP32, 16^3 p = 4 194 and 108 us; every wave reading the
// whole matrix by itself 139, 89 and 215 us.  The CSR block products, which
// gather a row of the block vector per nonzero group, take 319, 143-185, about
// 580 and 260 us (their epilogues included; the node step below adds 55 to 170).
// At k = 8, 11^3 p = 4 FP64 (170 MB of matrices): 30 us, the CSR form 240.
// ---------------------------------------------------------------------------
template <typename T> struct Mfma;
template <> struct Mfma<double> {
    typedef double vec __attribute__((ext_vector_type(4)));
    typedef double load __attribute__((ext_vector_type(2)));
    static constexpr int KB = 2;
    static __device__ __forceinline__ vec mul(double x, double y, vec c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int i) { return g + 4 * i; }   // of result register i
};
template <> struct Mfma<float> {
    typedef float vec __attribute__((ext_vector_type(4)));
    typedef float load __attribute__((ext_vector_type(4)));
    static constexpr int KB = 4;
    static __device__ __forceinline__ vec mul(float x, float y, vec c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int i) { return 4 * g + i; }
};

template <typename T, int P, int RS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) element_dense_kernel(ElemArgs<T> a, const T* __restrict__ mats) {
    if (a.run != nullptr && *a.run == 0) return;
    typedef Mfma<T> M;
    constexpr int NL = (P + 1) * (P + 1) * (P + 1), NLP = dense_rows(P), KB = M::KB;
    constexpr int RT = NLP / 16, TK = NLP / (4 * KB), RPW = RT / RS;
    static_assert(RT % RS == 0 && 4 % RS == 0, "row tiles per wave");
    const int lane = threadIdx.x % WAVE, w = threadIdx.x / WAVE;
    const int c = lane % 16, g = lane / 16, r0 = (w % RS) * RPW;
    const int64_t e = xcd_block(blockIdx.x, gridDim.x);
    const int c0 = ((int)blockIdx.y * (4 / RS) + w / RS) * 16;
    if (RS > 1 && c0 >= a.k) return;   // a whole wave without columns
    const int32_t* __restrict__ map = a.map + e * NL;
    const T* __restrict__ vec = a.v + min(c0 + c, a.k - 1);
    const typename M::load* __restrict__ tiles =
        reinterpret_cast<const typename M::load*>(mats + e * NLP * NLP) + r0 * WAVE + lane;
    // RS > 1: this step's tiles and the next one's; RS == 1: the block's next
    // chunk of TS steps, one 16-byte piece of it per thread and register
    constexpr int TS = TK < 16 / RT ? TK : 16 / RT, PIECES = TS * RT * WAVE / 256;
    typename M::load m[2][RS > 1 ? RPW : 1], next[RS > 1 ? 1 : PIECES];
    __shared__ typename M::load chunk[RS > 1 ? 1 : 2][RS > 1 ? 1 : TS * RT * WAVE];
    if constexpr (RS > 1) {
#pragma unroll
        for (int r = 0; r < RPW; ++r) m[0][r] = tiles[r * WAVE];
    } else {
#pragma unroll
        for (int u = 0; u < PIECES; ++u) next[u] = tiles[(int)threadIdx.x - lane + u * 256];
    }
    T x[TK][KB];
    int32_t node[TK][KB];
#pragma unroll
    for (int t = 0; t < TK; ++t)
#pragma unroll
        for (int b = 0; b < KB; ++b) node[t][b] = map[min((4 * t + g) * KB + b, NL - 1)];
#pragma unroll
    for (int t = 0; t < TK; ++t)
#pragma unroll
        for (int b = 0; b < KB; ++b) x[t][b] = vec[(int64_t)max(node[t][b], 0) * a.k];
#pragma unroll
    for (int t = 0; t < TK; ++t)
#pragma unroll
        for (int b = 0; b < KB; ++b)   // constrained nodes and padding: zero
            if (node[t][b] < 0 || (4 * t + g) * KB + b >= NL) x[t][b] = T(0);
    typename M::vec acc[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) acc[r] = typename M::vec{0, 0, 0, 0};
    if constexpr (RS > 1) {
#pragma unroll
        for (int t = 0; t < TK; ++t) {
            if (t + 1 < TK) {
#pragma unroll
                for (int r = 0; r < RPW; ++r) m[(t + 1) & 1][r] = tiles[((t + 1) * RT + r) * WAVE];
            }
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int r = 0; r < RPW; ++r) acc[r] = M::mul(m[t & 1][r][b], x[t][b], acc[r]);
        }
    } else {
#pragma unroll
        for (int t0 = 0; t0 < TK; t0 += TS) {
            typename M::load* buf = chunk[(t0 / TS) & 1];
#pragma unroll
            for (int u = 0; u < PIECES; ++u) buf[threadIdx.x + u * 256] = next[u];
            __syncthreads();   // also: the buffer of the step after next is free
            if (t0 + TS < TK) {
#pragma unroll
                for (int u = 0; u < PIECES; ++u)
                    next[u] = tiles[(int)threadIdx.x - lane + (t0 + TS) * RT * WAVE + u * 256];
            }
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                typename M::load s[RPW];
#pragma unroll
                for (int r = 0; r < RPW; ++r) s[r] = buf[(t * RT + r) * WAVE + lane];
#pragma unroll
                for (int b = 0; b < KB; ++b)
#pragma unroll
                    for (int r = 0; r < RPW; ++r) acc[r] = M::mul(s[r][b], x[t0 + t][b], acc[r]);
            }
        }
    }
    if (c0 + c < a.k) {
        T* __restrict__ ev = a.ev + e * NL * a.k + c0 + c;
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = (r0 + r) * 16 + M::row(g, i);
                if (row < NL) ev[(int64_t)row * a.k] = acc[r][i];
            }
    }
}

template <typename T, int P, int RS>
void launch_dense(const ElemArgs<T>& a, const T* mats, hipStream_t s) {
    const dim3 grid((unsigned)a.ne, (unsigned)((a.k + 64 / RS - 1) / (64 / RS)));
    element_dense_kernel<T, P, RS><<<grid, 256, 0, s>>>(a, mats);
}

template <typename T>
void launch_dense_order(int p, const ElemArgs<T>& a, const T* mats, hipStream_t s) {
#define GIAMG_DENSE(P)                                                          \
    case P:                                                                     \
        if (a.k <= 16 && dense_rows(P) >= 64) launch_dense<T, P, dense_rows(P) >= 64 ? 4 : 2>(a, mats, s); \
        else if (a.k <= 32) launch_dense<T, P, 2>(a, mats, s);                  \
        else launch_dense<T, P, 1>(a, mats, s);                                 \
        break;
    switch (p) {
        GIAMG_DENSE(2) GIAMG_DENSE(3) GIAMG_DENSE(4)
        default: throw Error(GIAMG_EINVAL, "dense element form of an unsupported order");
    }
#undef GIAMG_DENSE
    GIAMG_HIP(hipGetLastError());
}

// In launches of at most UNIT_BLOCKS blocks (a launch holds less than 2^32 threads;
// one for all pairs would pass that from 9.9 M elements of order 2 on).
constexpr int64_t UNIT_BLOCKS = 1 << 16;
template <int P>
void launch_unit(ElemArgs<double> a, hipStream_t s) {
    constexpr int NT = 256, V = NT / ((P + 2) * (P + 2));
    const int64_t step = UNIT_BLOCKS * V / a.k;   // elements
    for (int64_t e = 0; e < a.ne; e += step) {
        a.e0 = (int)e;   // a last block that runs on into the next launch's pairs writes the same values
        const int64_t blocks = (std::min(step, a.ne - e) * a.k + V - 1) / V;
        element_kernel<double, P, NT, V, true, true><<<(unsigned)blocks, NT, 0, s>>>(a);
    }
}

// The node step over k columns: one thread per node and VW columns, which it
// loads and stores as one vector (16 bytes, or 1 column where k or a pointer
// does not allow it).  Bound by its vectors: the FP32 Chebyshev step of 20^3
// p = 3 at k = 64 moves 0.48 GB in 81 us (5.9 TB/s); with one column per thread,
// 165 us, the dependent loads of the node lists bound it.
template <typename T, int VW>
struct alignas(VW * sizeof(T)) ColVec {
    T c[VW];
};
template <typename T, int MODE, int VW>
__global__ void __launch_bounds__(NODE_THREADS) element_node_block_kernel(SpmmArgs<T> a,
                                                                          const int32_t* __restrict__ ptr,
                                                                          const int32_t* __restrict__ ent,
                                                                          const T* __restrict__ ev) {
#pragma clang fp contract(off)
    if (a.run != nullptr && *a.run == 0) return;
    typedef ColVec<T, VW> Vec;
    const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
    const int64_t idx = lb * NODE_THREADS + threadIdx.x;
    const int kv = a.k / VW;
    if (idx >= a.n * kv) return;
    const int64_t row = idx <= (int64_t)UINT32_MAX ? (uint32_t)idx / (uint32_t)kv : idx / kv;
    const int cv = (int)(idx - row * kv);
    const int32_t s = ptr[row], e = ptr[row + 1];
    // row-local operands, loaded ahead of the sum
    Vec f, r, v, x, y;
    T dinv = 0;
    auto at = [&](const T* p) { return reinterpret_cast<const Vec*>(p)[idx]; };
    auto put = [&](T* p, const Vec& u) { reinterpret_cast<Vec*>(p)[idx] = u; };
    if constexpr (MODE == SPMV_RESID || MODE == SPMV_CHEB_INIT || MODE == SPMV_JACOBI) f = at(a.f);
    if constexpr (MODE == SPMV_CHEB_INIT || MODE == SPMV_CHEB_STEP || MODE == SPMV_JACOBI) dinv = a.dinv[row];
    if constexpr (MODE == SPMV_CHEB_STEP || MODE == SPMV_JACOBI) v = at(a.v);
    if constexpr (MODE == SPMV_CHEB_STEP) {
        r = at(a.r);
        if (!(a.flags & CHEB_ASSIGN)) x = at(a.x);
    }
    const Vec* __restrict__ el = reinterpret_cast<const Vec*>(ev) + cv;
#pragma unroll
    for (int i = 0; i < VW; ++i) y.c[i] = T(0);
    for (int32_t j = s; j < e; ++j) {
        const Vec t = el[(int64_t)ent[j] * kv];
#pragma unroll
        for (int i = 0; i < VW; ++i) y.c[i] += t.c[i];
    }
    if (s == e) y = at(a.v);   // constrained: identity row
    Vec o, o2;
#pragma unroll
    for (int i = 0; i < VW; ++i) {
        if constexpr (MODE == SPMV_PLAIN) {
            o.c[i] = y.c[i];
        } else if constexpr (MODE == SPMV_RESID) {
            o.c[i] = f.c[i] - y.c[i];
        } else if constexpr (MODE == SPMV_CHEB_INIT) {
            o2.c[i] = dinv * (f.c[i] - y.c[i]);
            o.c[i] = o2.c[i] * a.inv_theta;
        } else if constexpr (MODE == SPMV_CHEB_STEP) {
            r.c[i] = mad(-dinv, y.c[i], r.c[i]);
            o.c[i] = mad(a.c1, v.c[i], a.c2 * r.c[i]);
            const T inc = (a.flags & CHEB_LAST) ? v.c[i] + o.c[i] : v.c[i];
            x.c[i] = ((a.flags & CHEB_ASSIGN) ? T(0) : x.c[i]) + inc;
        } else if constexpr (MODE == SPMV_JACOBI) {
            o.c[i] = mad(a.omega * dinv, f.c[i] - y.c[i], v.c[i]);
        }
    }
    put(a.y, o);
    if constexpr (MODE == SPMV_CHEB_INIT) put(a.r, o2);
    if constexpr (MODE == SPMV_CHEB_STEP) {
        put(a.r, r);
        put(a.x, x);
    }
}

template <typename T, int MODE>
void launch_node_block(const SpmmArgs<T>& a, const ElementForm& E, const T* ev, hipStream_t s) {
    constexpr int VW = 16 / (int)sizeof(T);
    uintptr_t bits = 0;
    for (const void* p : {(const void*)a.v, (const void*)a.y, (const void*)a.f, (const void*)a.r, (const void*)a.x,
                          (const void*)ev})
        bits |= reinterpret_cast<uintptr_t>(p);
    const int vw = a.k % VW == 0 && bits % 16 == 0 ? VW : 1;
    const unsigned grid = (unsigned)((a.n * (a.k / vw) + NODE_THREADS - 1) / NODE_THREADS);
    if (vw == VW)
        element_node_block_kernel<T, MODE, VW><<<grid, NODE_THREADS, 0, s>>>(a, E.nptr.get(), E.nent.get(), ev);
    else
        element_node_block_kernel<T, MODE, 1><<<grid, NODE_THREADS, 0, s>>>(a, E.nptr.get(), E.nent.get(), ev);
}

// ---------------------------------------------------------------------------
// Transfers between the fine level and the next order q (M = q + 1 coarse nodes per
// axis): contraction of an element's values with the 1-D interpolation along one
// axis after the other.  A block takes V elements, each thread a line at a time.
// The rows of P hold 8 entries on average at p = 4; the element form reads no entry
// but the maps and the vectors.  32^3 p = 4, FP64: P 47 -> 23 us (map, coarse values, x
// read and written: 55 MB; bound by its chain of three passes and the scattered
// update of x), R 42 -> 14 + 8 us (its node step adds a coarse node's elements);
// 13^3 p = 5 to order 3: 25 -> 6 and 26 -> 10 us.
// ---------------------------------------------------------------------------
template <typename T>
struct XferArgs {
    int64_t ne = 0;
    int M = 0;
    const int32_t* own = nullptr;
    const int32_t* cmap = nullptr;
    const T* i1 = nullptr;           // [p + 1][M]
    const T* v = nullptr;
    T* y = nullptr;                  // R: element results [ne][M^3]; P: the fine vector
    const int* stop = nullptr;
};
constexpr int XFER_THREADS = 256;
template <int P> constexpr int xfer_elems() { return XFER_THREADS / ((P + 1) * (P + 1)); }

template <typename T, int P>
__global__ void __launch_bounds__(XFER_THREADS) element_restrict_kernel(XferArgs<T> a) {
#pragma clang fp contract(off)
    constexpr int N = P + 1, N2 = N * N, N3 = N2 * N, V = xfer_elems<P>(), ITER = (V * N3 + XFER_THREADS - 1) / XFER_THREADS;
    __shared__ T s0[V * N3], s1[V * N2 * P], si[N * P];
    const int done = a.stop != nullptr ? *a.stop : 0;
    const int tid = threadIdx.x, M = a.M;
    const int64_t first = xcd_block(blockIdx.x, gridDim.x) * V;
    const int cnt = (int)min((int64_t)V, a.ne - first);
    const int32_t* __restrict__ own = a.own + first * N3;
    int32_t g[ITER];
    T x[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it) g[it] = own[min(tid + it * XFER_THREADS, cnt * N3 - 1)];
#pragma unroll
    for (int it = 0; it < ITER; ++it) x[it] = a.v[max(g[it], 0)];
    if (tid < N * M) si[tid] = a.i1[tid];
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int t = tid + it * XFER_THREADS;
        if (t < V * N3) s0[t] = g[it] >= 0 ? x[it] : T(0);
    }
    __syncthreads();
    if (done) return;
    if (tid < cnt * N2) {   // z: [i][j][k] -> [i][j][c]
        T l[N];
#pragma unroll
        for (int k = 0; k < N; ++k) l[k] = s0[tid * N + k];
        for (int c = 0; c < M; ++c) {
            T r = 0;
#pragma unroll
            for (int k = 0; k < N; ++k) r = mad(si[k * M + c], l[k], r);
            s1[tid * M + c] = r;
        }
    }
    __syncthreads();
    const unsigned m = M, m2 = m * m;
    for (unsigned t = tid; t < cnt * N * m; t += XFER_THREADS) {   // y: -> [i][b][c]
        const unsigned vi = t / m, c = t - vi * m;
        T l[N];
#pragma unroll
        for (int j = 0; j < N; ++j) l[j] = s1[(vi * N + j) * m + c];
        for (unsigned b = 0; b < m; ++b) {
            T r = 0;
#pragma unroll
            for (int j = 0; j < N; ++j) r = mad(si[j * m + b], l[j], r);
            s0[vi * m2 + b * m + c] = r;
        }
    }
    __syncthreads();
    for (unsigned t = tid; t < cnt * m2; t += XFER_THREADS) {      // x: -> [a][b][c]
        const unsigned e = t / m2, bc = t - e * m2;
        T l[N];
#pragma unroll
        for (int i = 0; i < N; ++i) l[i] = s0[(e * N + i) * m2 + bc];
        T* out = a.y + (first + e) * m2 * m + bc;
        for (unsigned q = 0; q < m; ++q) {
            T r = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) r = mad(si[i * m + q], l[i], r);
            out[q * m2] = r;
        }
    }
}

template <typename T, int P>
__global__ void __launch_bounds__(XFER_THREADS) element_prolong_kernel(XferArgs<T> a) {
#pragma clang fp contract(off)
    constexpr int N = P + 1, N2 = N * N, N3 = N2 * N, V = xfer_elems<P>(), ITER = (V * N3 + XFER_THREADS - 1) / XFER_THREADS;
    __shared__ T s0[V * N2 * P], s1[V * N3], si[N * P];
    const int done = a.stop != nullptr ? *a.stop : 0;
    const int tid = threadIdx.x;
    const unsigned m = a.M, m2 = m * m, m3 = m2 * m;
    const int64_t first = xcd_block(blockIdx.x, gridDim.x) * V;
    const int cnt = (int)min((int64_t)V, a.ne - first);
    const int32_t* __restrict__ own = a.own + first * N3;
    const int32_t* __restrict__ cmap = a.cmap + first * m3;
    int32_t g[ITER];
    T y[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it) g[it] = own[min(tid + it * XFER_THREADS, cnt * N3 - 1)];
    if (tid < N * (int)m) si[tid] = a.i1[tid];
    for (unsigned t = tid; t < cnt * m3; t += XFER_THREADS) {
        const int32_t c = cmap[t];
        s0[t] = c >= 0 ? a.v[c] : T(0);
    }
#pragma unroll
    for (int it = 0; it < ITER; ++it) y[it] = a.y[max(g[it], 0)];
    __syncthreads();
    if (done) return;
    for (unsigned t = tid; t < cnt * m2; t += XFER_THREADS) {      // x: [a][b][c] -> [i][b][c]
        const unsigned e = t / m2, bc = t - e * m2;
        T r[N];
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = 0;
        for (unsigned q = 0; q < m; ++q) {
            const T c = s0[e * m3 + q * m2 + bc];
#pragma unroll
            for (int i = 0; i < N; ++i) r[i] = mad(si[i * m + q], c, r[i]);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) s1[(e * N + i) * m2 + bc] = r[i];
    }
    __syncthreads();
    for (unsigned t = tid; t < cnt * N * m; t += XFER_THREADS) {   // y: -> [i][j][c]
        const unsigned vi = t / m, c = t - vi * m;
        T r[N];
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = 0;
        for (unsigned b = 0; b < m; ++b) {
            const T w = s1[vi * m2 + b * m + c];
#pragma unroll
            for (int j = 0; j < N; ++j) r[j] = mad(si[j * m + b], w, r[j]);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) s0[(vi * N + j) * m + c] = r[j];
    }
    __syncthreads();
    if (tid < cnt * N2) {                                          // z: -> [i][j][k]
        T r[N];
#pragma unroll
        for (int k = 0; k < N; ++k) r[k] = 0;
        for (unsigned c = 0; c < m; ++c) {
            const T w = s0[tid * m + c];
#pragma unroll
            for (int k = 0; k < N; ++k) r[k] = mad(si[k * m + c], w, r[k]);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) s1[tid * N + k] = r[k];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int t = tid + it * XFER_THREADS;
        if (t < cnt * N3 && g[it] >= 0) a.y[g[it]] = y[it] + s1[t];
    }
}

__global__ void transfer_own_kernel(int64_t m, const int32_t* __restrict__ map, const int32_t* __restrict__ nptr,
                                    const int32_t* __restrict__ nent, int32_t* __restrict__ own) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = map[t];
        own[t] = g >= 0 && nent[nptr[g]] == t ? g : -1;
    }
}

// Whether every row of P is what the node's first element gives: as many entries
// as that element has coarse nodes with a nonzero weight (P's row is the union over
// the node's elements, first occurrence kept), and no element lists a coarse node twice.
__global__ void transfer_rows_kernel(int64_t m, int N, int M, const int32_t* __restrict__ own,
                                     const int32_t* __restrict__ cmap, const double* __restrict__ i1,
                                     const int64_t* __restrict__ rp, int* bad) {
    const int M3 = M * M * M;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t g = own[t];
        if (g < 0) continue;
        const int64_t e = t / (N * N * N);
        const int loc = (int)(t - e * (N * N * N)), i = loc / (N * N), j = loc / N % N, k = loc % N;
        int count = 0;
        for (int c = 0; c < M3; ++c)
            count += i1[i * M + c / (M * M)] != 0.0 && i1[j * M + c / M % M] != 0.0 && i1[k * M + c % M] != 0.0 &&
                     cmap[e * M3 + c] >= 0;
        if (count != rp[g + 1] - rp[g]) *bad = 1;
    }
}
__global__ void transfer_twice_kernel(int64_t mc, int M3, const int32_t* __restrict__ cmap, int* bad) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < mc; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t c = cmap[t];
        if (c < 0) continue;
        for (int64_t u = t / M3 * M3; u < t; ++u)
            if (cmap[u] == c) *bad = 1;
    }
}

template <typename T, int MODE>
void launch_node_lists(const SpmvArgs<T>& a, const int32_t* nptr, const int32_t* nent, const T* ev, hipStream_t s) {
    const dim3 grid((unsigned)a.nblk), block(NODE_THREADS);
    if (a.ev_stop != nullptr)
        hipExtLaunchKernelGGL((element_node_kernel<T, MODE>), grid, block, 0, s, nullptr, a.ev_stop, 0, a, nptr, nent,
                              ev);
    else
        element_node_kernel<T, MODE><<<grid, block, 0, s>>>(a, nptr, nent, ev);
}
template <typename T, int MODE>
void launch_node_kernel(const SpmvArgs<T>& a, const ElementForm& E, const T* ev, hipStream_t s) {
    launch_node_lists<T, MODE>(a, E.nptr.get(), E.nent.get(), ev, s);
}

template <typename T> const T* form_coef(const ElementForm& E);
template <> const double* form_coef<double>(const ElementForm& E) { return E.coef.get(); }
template <> const float* form_coef<float>(const ElementForm& E) { return E.coef32.get(); }
template <typename T> const T* form_tabs(const ElementForm& E);
template <> const double* form_tabs<double>(const ElementForm& E) { return E.tabs.get(); }
template <> const float* form_tabs<float>(const ElementForm& E) { return E.tabs32.get(); }

// Entries per node (free nodes only) by atomic counts, then placed by atomic
// counters and sorted ascending per node, which removes the atomics' order.
__global__ void node_count_kernel(int64_t m, const int32_t* __restrict__ map, int32_t* __restrict__ counts) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        if (map[i] >= 0) atomicAdd(counts + map[i], 1);
}
__global__ void node_place_kernel(int64_t m, const int32_t* __restrict__ map, const int32_t* __restrict__ ptr,
                                  int32_t* __restrict__ fill, int32_t* __restrict__ ent) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        if (map[i] >= 0) ent[ptr[map[i]] + atomicAdd(fill + map[i], 1)] = (int32_t)i;
}
__global__ void node_sort_kernel(int64_t n, const int32_t* __restrict__ ptr, int32_t* __restrict__ ent) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const int32_t s = ptr[r], e = ptr[r + 1];
        for (int32_t i = s + 1; i < e; ++i) {
            const int32_t x = ent[i];
            int32_t j = i;
            for (; j > s && ent[j - 1] > x; --j) ent[j] = ent[j - 1];
            ent[j] = x;
        }
    }
}

unsigned setup_grid(int64_t m) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((m + 255) / 256, 65536)); }

}  // namespace

int64_t element_blocks(int64_t n) { return (n + NODE_THREADS - 1) / NODE_THREADS; }

template <typename T>
void launch_element_product(int mode, const SpmvArgs<T>& args, hipStream_t s) {
    SpmvArgs<T> a = args;
    const ElementForm& E = *a.elem;
    a.nblk = element_blocks(a.n);
    ElemArgs<T> e;
    e.ne = E.ne; e.map = E.map.get(); e.v = a.v; e.ev = reinterpret_cast<T*>(E.ev.get());
    e.coef = form_coef<T>(E); e.tabs = form_tabs<T>(E); e.lambda = (T)E.lambda;
    e.ps = (T)E.ps; e.pt = (T)E.pt;
    e.stop = a.stop;
    e.vnz = mode == SPMV_RINIT ? a.vnz : nullptr;
    if (e.coef == nullptr || e.tabs == nullptr) throw Error(GIAMG_EINVAL, "element form without this precision");
    launch_element_order<T>(E.order, e, a.ev_start, s);
    switch (mode) {
        case SPMV_PLAIN: launch_node_kernel<T, SPMV_PLAIN>(a, E, e.ev, s); break;
        case SPMV_RESID: launch_node_kernel<T, SPMV_RESID>(a, E, e.ev, s); break;
        case SPMV_CHEB_INIT: launch_node_kernel<T, SPMV_CHEB_INIT>(a, E, e.ev, s); break;
        case SPMV_CHEB_STEP: launch_node_kernel<T, SPMV_CHEB_STEP>(a, E, e.ev, s); break;
        case SPMV_JACOBI: launch_node_kernel<T, SPMV_JACOBI>(a, E, e.ev, s); break;
        case SPMV_DOT: launch_node_kernel<T, SPMV_DOT>(a, E, e.ev, s); break;
        case SPMV_DINV: launch_node_kernel<T, SPMV_DINV>(a, E, e.ev, s); break;
        case SPMV_RINIT: launch_node_kernel<T, SPMV_RINIT>(a, E, e.ev, s); break;
        case SPMV_CHEB_DOT: launch_node_kernel<T, SPMV_CHEB_DOT>(a, E, e.ev, s); break;
        case SPMV_JACOBI_DOT: launch_node_kernel<T, SPMV_JACOBI_DOT>(a, E, e.ev, s); break;
        default: throw Error(GIAMG_EINVAL, "unknown product mode of the element form");
    }
    GIAMG_HIP(hipGetLastError());
}
template <typename T>
void launch_transfer(int mode, const SpmvArgs<T>& args, hipStream_t s) {
    SpmvArgs<T> a = args;
    const TransferForm& X = *a.xfer;
    const bool down = mode != SPMV_ADD;
    XferArgs<T> x;
    x.ne = X.ne; x.M = X.q + 1; x.own = X.own.get(); x.cmap = X.cmap.get();
    if constexpr (sizeof(T) == 8) x.i1 = X.i1.get(); else x.i1 = X.i132.get();
    x.v = a.v; x.y = down ? reinterpret_cast<T*>(X.ev) : a.y; x.stop = a.stop;
    if (x.i1 == nullptr) throw Error(GIAMG_EINVAL, "transfer form without this precision");
    const hipEvent_t end = down ? nullptr : a.ev_stop;
#define GIAMG_XFER(P)                                                                                     \
    case P: {                                                                                             \
        const dim3 grid((unsigned)((X.ne + xfer_elems<P>() - 1) / xfer_elems<P>())), block(XFER_THREADS); \
        auto* k = down ? element_restrict_kernel<T, P> : element_prolong_kernel<T, P>;                    \
        if (a.ev_start != nullptr)                                                                        \
            hipExtLaunchKernelGGL(k, grid, block, 0, s, a.ev_start, end, 0, x);                           \
        else                                                                                              \
            k<<<grid, block, 0, s>>>(x);                                                                  \
        break;                                                                                            \
    }
    switch (X.p) {
        GIAMG_XFER(2) GIAMG_XFER(3) GIAMG_XFER(4) GIAMG_XFER(5) GIAMG_XFER(6)
        GIAMG_XFER(7) GIAMG_XFER(8) GIAMG_XFER(9) GIAMG_XFER(10)
        default: throw Error(GIAMG_EINVAL, "transfer form of an unsupported order");
    }
#undef GIAMG_XFER
    if (down) {   // every coarse node has entries, so the node step never looks at v
        a.nblk = element_blocks(a.n);
        switch (mode) {
            case SPMV_PLAIN: launch_node_lists<T, SPMV_PLAIN>(a, X.nptr.get(), X.nent.get(), x.y, s); break;
            case SPMV_RCHEB0: launch_node_lists<T, SPMV_RCHEB0>(a, X.nptr.get(), X.nent.get(), x.y, s); break;
            default: throw Error(GIAMG_EINVAL, "unknown product mode of the transfer form");
        }
    }
    GIAMG_HIP(hipGetLastError());
}
template void launch_transfer<double>(int, const SpmvArgs<double>&, hipStream_t);
template void launch_transfer<float>(int, const SpmvArgs<float>&, hipStream_t);

template <typename T>
void launch_element_block(int mode, const SpmmArgs<T>& a, const ElementForm& E, double* ev, hipStream_t s) {
    ElemArgs<T> e;
    e.ne = E.ne; e.map = E.map.get(); e.v = a.v; e.ev = reinterpret_cast<T*>(ev);
    e.coef = form_coef<T>(E); e.tabs = form_tabs<T>(E); e.lambda = (T)E.lambda;
    e.ps = (T)E.ps; e.pt = (T)E.pt;
    e.k = a.k; e.run = a.run;
    if (e.coef == nullptr || e.tabs == nullptr) throw Error(GIAMG_EINVAL, "element form without this precision");
    if (E.mat.get() != nullptr) {
        const T* mats = nullptr;
        if constexpr (sizeof(T) == 8) mats = E.mat.get(); else mats = E.mat32.get();
        launch_dense_order<T>(E.order, e, mats, s);
    } else {
        launch_element_block_order<T>(E.order, e, s);
    }
    switch (mode) {
        case SPMV_PLAIN: launch_node_block<T, SPMV_PLAIN>(a, E, e.ev, s); break;
        case SPMV_RESID: launch_node_block<T, SPMV_RESID>(a, E, e.ev, s); break;
        case SPMV_CHEB_INIT: launch_node_block<T, SPMV_CHEB_INIT>(a, E, e.ev, s); break;
        case SPMV_CHEB_STEP: launch_node_block<T, SPMV_CHEB_STEP>(a, E, e.ev, s); break;
        case SPMV_JACOBI: launch_node_block<T, SPMV_JACOBI>(a, E, e.ev, s); break;
        default: throw Error(GIAMG_EINVAL, "unknown block product mode of the element form");
    }
    GIAMG_HIP(hipGetLastError());
}
template void launch_element_block<double>(int, const SpmmArgs<double>&, const ElementForm&, double*, hipStream_t);
template void launch_element_block<float>(int, const SpmmArgs<float>&, const ElementForm&, double*, hipStream_t);

template void launch_element_product<double>(int, const SpmvArgs<double>&, hipStream_t);
template void launch_element_product<float>(int, const SpmvArgs<float>&, hipStream_t);

void build_element_matrices(ElementForm& E, bool mixed, hipStream_t s) {
    if (E.mat.get() != nullptr) return;
    GIAMG_REQUIRE(E.order >= 2 && E.order <= 4, "dense element form of an unsupported order");
    const int64_t nl = (E.order + 1) * (E.order + 1) * (E.order + 1), nlp = dense_rows(E.order);
    DevBuf<double> mat((size_t)(E.ne * nlp * nlp));
    DevBuf<float> mat32;
    GIAMG_HIP(hipMemsetAsync(mat.get(), 0, mat.n * sizeof(double), s));   // padding
    if (mixed) {
        mat32.alloc(mat.n);
        GIAMG_HIP(hipMemsetAsync(mat32.get(), 0, mat32.n * sizeof(float), s));
    }
    ElemArgs<double> a;
    a.ne = E.ne; a.map = E.map.get(); a.coef = E.coef.get(); a.tabs = E.tabs.get(); a.lambda = E.lambda;
    a.ps = E.ps; a.pt = E.pt;
    a.k = (int)nl; a.mat = mat.get(); a.mat32 = mat32.get();
    switch (E.order) {
        case 2: launch_unit<2>(a, s); break;
        case 3: launch_unit<3>(a, s); break;
        default: launch_unit<4>(a, s); break;
    }
    GIAMG_HIP(hipGetLastError());
    GIAMG_HIP(hipStreamSynchronize(s));
    E.mat = std::move(mat);
    E.mat32 = std::move(mat32);
}

// Per node its entries of map[m], ascending.
static void build_node_lists(const int32_t* map, int64_t m, int64_t n, DevBuf<int32_t>& nptr, DevBuf<int32_t>& nent,
                      hipStream_t s) {
    DevBuf<int32_t> counts((size_t)n);
    GIAMG_HIP(hipMemsetAsync(counts.get(), 0, n * sizeof(int32_t), s));
    node_count_kernel<<<setup_grid(m), 256, 0, s>>>(m, map, counts.get());
    GIAMG_HIP(hipGetLastError());
    std::vector<int32_t> hc((size_t)n), ptr((size_t)n + 1, 0);
    GIAMG_HIP(hipMemcpyAsync(hc.data(), counts.get(), n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    GIAMG_HIP(hipStreamSynchronize(s));
    for (int64_t i = 0; i < n; ++i) ptr[i + 1] = ptr[i] + hc[i];
    nptr.alloc((size_t)n + 1);
    nent.alloc((size_t)std::max<int32_t>(ptr[n], 1));
    GIAMG_HIP(hipMemcpyAsync(nptr.get(), ptr.data(), ptr.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    GIAMG_HIP(hipMemsetAsync(counts.get(), 0, n * sizeof(int32_t), s));
    node_place_kernel<<<setup_grid(m), 256, 0, s>>>(m, map, nptr.get(), counts.get(), nent.get());
    node_sort_kernel<<<setup_grid(n), 256, 0, s>>>(n, nptr.get(), nent.get());
    GIAMG_HIP(hipGetLastError());
    GIAMG_HIP(hipStreamSynchronize(s));   // the host arrays go out of scope
}

// Coefficients of x = sum over the corners of X_c (1 +- xi)(1 +- eta)(1 +- zeta) / 8; corner
// c = 4 i + 2 j + k; xi, eta, zeta, xi eta, xi zeta, eta zeta, xi eta zeta, three axes each.
static void trilinear_coefs(const double* corners, double* coef) {
    const int sub[7] = {4, 2, 1, 6, 5, 3, 7};
    for (int t = 0; t < 7; ++t)
        for (int r = 0; r < 3; ++r) {
            double v = 0.0;
            for (int c = 0; c < 8; ++c) {
                const int low = __builtin_popcount(sub[t] & ~c) & 1;   // one minus sign per -1 side
                v += (low ? -1.0 : 1.0) * corners[c * 3 + r];
            }
            coef[3 * t + r] = 0.125 * v;
        }
}
// Exponent of the power of two that an element is scaled by in FP32: its largest coefficient's.
static int element_exponent(const double* coef) {
    double m = 0.0;
    for (int i = 0; i < ELEM_COEF; ++i) m = std::max(m, std::fabs(coef[i]));
    return m > 0.0 ? std::ilogb(m) : 0;
}

bool fp32_geometry(const std::vector<double>& corners, int64_t ne, int p, double lambda) {
    std::vector<double> g, w;
    gauss_points(p + 2, g, w);
    const double at[3] = {g.front(), 0.0, g.back()};
    std::atomic<bool> ok{true};
    parallel_for(ne, 1 << 14, [&](int64_t b, int64_t en) {   // 50 ns an element; threads cost 50 us
        bool good = true;
        for (int64_t e = b; e < en && good; ++e) {
            double c[ELEM_COEF];
            trilinear_coefs(corners.data() + (size_t)e * 24, c);
            const int ex = element_exponent(c);
            good = std::abs(ex) <= 64 && std::ldexp(lambda, 3 * ex) <= 0x1p100;
            if (!good) break;
            const double scale = std::ldexp(1.0, -ex);
            for (double& v : c) v *= scale;
            auto norm = [&](int m) { return std::sqrt(c[m] * c[m] + c[m + 1] * c[m + 1] + c[m + 2] * c[m + 2]); };
            auto det = [](const double* x, const double* y, const double* z) {
                return x[0] * (y[1] * z[2] - y[2] * z[1]) + x[1] * (y[2] * z[0] - y[0] * z[2]) +
                       x[2] * (y[0] * z[1] - y[1] * z[0]);
            };
            // Bounds from the middle, which most elements pass: the columns change by at most
            // v, so the determinant by at most the product of l + v less that of l.
            const double xy = norm(9), xz = norm(12), yz = norm(15), xyz = norm(18);
            const double l[3] = {norm(0), norm(3), norm(6)};
            const double v[3] = {xy + xz + xyz, xy + yz + xyz, xz + yz + xyz};
            const double most = (l[0] + v[0]) * (l[1] + v[1]) * (l[2] + v[2]);
            if (std::min({l[0] - v[0], l[1] - v[1], l[2] - v[2]}) >= 0x1p-20 &&
                det(c, c + 3, c + 6) - (most - l[0] * l[1] * l[2]) >= 0x1p-10 * most)
                continue;
            for (int q = 0; q < 27 && good; ++q) {
                const double xi = at[q / 9], eta = at[q / 3 % 3], zeta = at[q % 3];
                double J[3][3], len[3];   // columns dx/dxi, dx/deta, dx/dzeta
                for (int m = 0; m < 3; ++m) {
                    J[0][m] = c[m] + c[9 + m] * eta + c[12 + m] * zeta + c[18 + m] * eta * zeta;
                    J[1][m] = c[3 + m] + c[9 + m] * xi + c[15 + m] * zeta + c[18 + m] * xi * zeta;
                    J[2][m] = c[6 + m] + c[12 + m] * xi + c[15 + m] * eta + c[18 + m] * xi * eta;
                }
                for (int d = 0; d < 3; ++d)
                    len[d] = std::sqrt(J[d][0] * J[d][0] + J[d][1] * J[d][1] + J[d][2] * J[d][2]);
                good = std::min({len[0], len[1], len[2]}) >= 0x1p-20 &&
                       det(J[0], J[1], J[2]) >= 0x1p-10 * len[0] * len[1] * len[2];
            }
        }
        if (!good) ok = false;
    });
    return ok;
}

void build_element_form(ElementForm& E, const std::vector<double>& corners, const int32_t* l2g, int64_t ne, int p,
                        int64_t n, double lambda, const std::vector<uint8_t>& cons, int basis, bool mixed,
                        hipStream_t s) {
    const int n1 = p + 1, nq = p + 2;
    const int64_t m = ne * n1 * n1 * n1;
    E.order = p;
    E.ne = ne;
    E.lambda = lambda;
    // Local positions of the kernel: the nodal basis keeps its order (position k
    // mirrors N - 1 - k).  The modal basis puts its two vertex modes at the ends
    // and its bubbles (even bubble m = 2, 4, ... at k, odd one at N - 1 - k)
    // inside: they are even or odd by themselves, so the pair transform of the
    // inner positions is the identity there (ps = 0, pt = 1).
    std::vector<int> pos(n1);   // position -> 1-D basis index
    for (int k = 0; k < n1; ++k) pos[k] = k;
    if (basis == GIAMG_BASIS_MODAL) {
        pos[0] = 0;
        pos[n1 - 1] = 1;
        for (int k = 1; 2 * k <= p; ++k) pos[k] = 2 * k;
        for (int k = 1; 2 * k + 1 <= p; ++k) pos[n1 - 1 - k] = 2 * k + 1;
        E.ps = 0.0;
        E.pt = 1.0;
    }
    std::vector<int32_t> map((size_t)m);
    parallel_for(ne, 1 << 10, [&](int64_t b, int64_t en) {
        for (int64_t e = b; e < en; ++e) {
            const int32_t* g = l2g + e * n1 * n1 * n1;
            int32_t* o = map.data() + e * n1 * n1 * n1;
            for (int i = 0; i < n1; ++i)
                for (int j = 0; j < n1; ++j)
                    for (int k = 0; k < n1; ++k) {
                        const int32_t node = g[(pos[i] * n1 + pos[j]) * n1 + pos[k]];
                        o[(i * n1 + j) * n1 + k] = cons[node] ? -1 : node;
                    }
        }
    });
    E.map.alloc(m);
    GIAMG_HIP(hipMemcpyAsync(E.map.get(), map.data(), m * sizeof(int32_t), hipMemcpyHostToDevice, s));
    std::vector<double> coef((size_t)ELEM_COEF * ne);
    std::vector<float> coef32(mixed ? (size_t)elem_coefs<float>() * ne : 0);
    parallel_for(ne, 1 << 12, [&](int64_t b, int64_t en) {
        for (int64_t e = b; e < en; ++e) {
            double c[ELEM_COEF];
            trilinear_coefs(corners.data() + (size_t)e * 24, c);
            for (int m = 0; m < ELEM_COEF; ++m) coef[(size_t)m * ne + e] = c[m];
            if (!mixed) continue;
            const int ex = element_exponent(c);
            const double scale = std::ldexp(1.0, -ex);
            for (int m = 0; m < ELEM_COEF; ++m) coef32[(size_t)m * ne + e] = (float)(c[m] * scale);
            coef32[(size_t)ELEM_COEF * ne + e] = (float)std::ldexp(1.0, ex);
            coef32[(size_t)(ELEM_COEF + 1) * ne + e] = (float)std::ldexp(lambda, 3 * ex);
        }
    });
    E.coef.alloc(coef.size());
    GIAMG_HIP(hipMemcpyAsync(E.coef.get(), coef.data(), coef.size() * sizeof(double), hipMemcpyHostToDevice, s));
    std::vector<double> L, D, g, w;
    reference_tables(p, basis, L, D, g, w);
    // per Gauss pair q, Q - 1 - q: even and odd parts of the values (Le from the
    // even, Lo from the odd coefficients) and derivatives (De: odd in q, Do: even)
    std::vector<double> tabs;
    const int hq = (nq + 1) / 2, hn = (n1 + 1) / 2, on = n1 / 2;
    auto part = [&](const std::vector<double>& M, int k, int q, double parity, double mirror) {
        const bool pairs = basis != GIAMG_BASIS_MODAL || k == 0;
        auto sym = [&](int i) {   // average of the two points' values with the part's symmetry in q
            return 0.5 * (M[i * nq + q] + mirror * M[i * nq + nq - 1 - q]);
        };
        if (k == n1 - 1 - k) return sym(pos[k]);
        if (!pairs) return sym(parity > 0 ? pos[k] : pos[n1 - 1 - k]);
        return 0.5 * (sym(pos[k]) + parity * sym(pos[n1 - 1 - k]));
    };
    for (int q = 0; q < hq; ++q) {
        for (int k = 0; k < hn; ++k) tabs.push_back(part(L, k, q, 1.0, 1.0));
        for (int k = 0; k < on; ++k) tabs.push_back(part(L, k, q, -1.0, -1.0));
        for (int k = 0; k < hn; ++k) tabs.push_back(part(D, k, q, 1.0, -1.0));
        for (int k = 0; k < on; ++k) tabs.push_back(part(D, k, q, -1.0, 1.0));
    }
    for (const auto* v : {&g, &w}) tabs.insert(tabs.end(), v->begin(), v->end());
    GIAMG_REQUIRE((int)tabs.size() == 2 * n1 * hq + 2 * nq, "unexpected size of the 1-D tables");
    E.tabs.alloc(tabs.size());
    GIAMG_HIP(hipMemcpyAsync(E.tabs.get(), tabs.data(), tabs.size() * sizeof(double), hipMemcpyHostToDevice, s));
    if (mixed) {
        E.coef32.alloc(coef32.size());
        GIAMG_HIP(hipMemcpyAsync(E.coef32.get(), coef32.data(), coef32.size() * sizeof(float), hipMemcpyHostToDevice, s));
        E.tabs32.alloc(tabs.size());
        launch_convert<double, float>((int64_t)tabs.size(), E.tabs.get(), E.tabs32.get(), s);
    }
    build_node_lists(E.map.get(), m, n, E.nptr, E.nent, s);
}

bool build_transfer_form(TransferForm& X, const ElementForm& E, const DevCSR& P, const std::vector<int32_t>& coarse_l2g,
                         int q, bool mixed, hipStream_t s) {
    const int p = E.order, N = p + 1, M = q + 1;
    const int64_t m = E.ne * N * N * N, mc = E.ne * M * M * M;
    GIAMG_REQUIRE(q >= 1 && q < p && (int64_t)coarse_l2g.size() == mc, "transfer form of unexpected sizes");
    std::vector<double> xp, xq, w, i1;
    gll_points(p, xp, w);
    gll_points(q, xq, w);
    for (int i = 0; i < N; ++i)
        for (int c = 0; c < M; ++c) {
            const double v = lagrange_value(xq, c, xp[i]);
            i1.push_back(std::fabs(v) <= 1e-12 ? 0.0 : v);   // the structural zeros of p_transfer_maps
        }
    X.p = p;
    X.ne = E.ne;
    X.ev = E.ev.get();
    X.own.alloc((size_t)m);
    X.cmap.alloc((size_t)mc);
    X.i1.alloc(i1.size());
    transfer_own_kernel<<<setup_grid(m), 256, 0, s>>>(m, E.map.get(), E.nptr.get(), E.nent.get(), X.own.get());
    GIAMG_HIP(hipGetLastError());
    GIAMG_HIP(hipMemcpyAsync(X.cmap.get(), coarse_l2g.data(), mc * sizeof(int32_t), hipMemcpyHostToDevice, s));
    GIAMG_HIP(hipMemcpyAsync(X.i1.get(), i1.data(), i1.size() * sizeof(double), hipMemcpyHostToDevice, s));
    if (mixed) {
        X.i132.alloc(i1.size());
        launch_convert<double, float>((int64_t)i1.size(), X.i1.get(), X.i132.get(), s);
    }
    DevBuf<int> bad(1);
    GIAMG_HIP(hipMemsetAsync(bad.get(), 0, sizeof(int), s));
    transfer_rows_kernel<<<setup_grid(m), 256, 0, s>>>(m, N, M, X.own.get(), X.cmap.get(), X.i1.get(), P.rp.get(),
                                                       bad.get());
    transfer_twice_kernel<<<setup_grid(mc), 256, 0, s>>>(mc, M * M * M, X.cmap.get(), bad.get());
    GIAMG_HIP(hipGetLastError());
    int hbad = 0;
    GIAMG_HIP(hipMemcpyAsync(&hbad, bad.get(), sizeof(int), hipMemcpyDeviceToHost, s));
    GIAMG_HIP(hipStreamSynchronize(s));   // also: the host arrays go out of scope
    if (hbad) return false;
    build_node_lists(X.cmap.get(), mc, P.ncols, X.nptr, X.nent, s);
    X.q = q;
    return true;
}

}  // namespace giamg
