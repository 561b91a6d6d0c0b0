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
// read stream.  The element form reads the element map, the corners and the
// vectors (about 0.15 GB there) and is bound by the vector ALUs and LDS.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "row_epilogue.h"

namespace giamg {

namespace {

constexpr int NODE_THREADS = 256;

template <typename T>
struct ElemArgs {
    int64_t ne = 0;
    const int32_t* map = nullptr;    // [ne][nl] node of each local position, -1 constrained
    const T* v = nullptr;
    T* ev = nullptr;                 // [ne][nl]
    const T* coef = nullptr;         // [ELEM_COEF][ne] trilinear coefficients
    const T* tabs = nullptr;         // L [n1][nq], D [n1][nq], Gauss points [nq], weights [nq]
    T lambda = 0;
    const int* stop = nullptr;
    const double* vnz = nullptr;     // when set and zero, v is +0: nothing to do
};

__device__ __forceinline__ double recip(double d) {
    // reciprocal estimate and two Newton steps (1 ulp)
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
}
__device__ __forceinline__ float recip(float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    return __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
}

// Thread counts and elements per block.  The quadrature step takes (p + 2)^2
// lanes per element: narrow blocks are the whole waves one element needs (or
// several elements in one wave), wide blocks fill 256 threads with elements.
// Wide where that fills more lanes (p = 3, 4, 5, 7, 8) and the mesh has a wide
// block for every CU; measured (product of the fine operator, FP64, wide /
// narrow): 32^3 p = 4 115.6 / 154.6 us, 12^3 p = 7 51.2 / 74.8, 13^3 p = 5
// 23.1 / 28.7; with fewer elements 8^3 p = 4 16.3 / 13.2; 40^3 p = 2 48.8 / 44.8.
constexpr int64_t ELEM_WIDE_LANES = 65536;   // 256 lanes on each of 256 CUs
constexpr bool elem_wide_pays(int p) { return p == 3 || p == 4 || p == 5 || p == 7 || p == 8; }
template <int P>
constexpr int elem_threads(bool wide) {
    constexpr int q2 = (P + 2) * (P + 2);
    return wide ? 256 : (q2 + 63) / 64 * 64;
}
template <int P>
constexpr int elem_per_block(bool wide) { return elem_threads<P>(wide) / ((P + 2) * (P + 2)); }

template <typename T, int P, bool WIDE>
__global__ void __launch_bounds__(elem_threads<P>(WIDE)) element_kernel(ElemArgs<T> a) {
    if (a.stop != nullptr && *a.stop != 0) return;
    if (a.vnz != nullptr && *a.vnz == 0.0) return;
    constexpr int N = P + 1, Q = P + 2, N2 = N * N, NL = N2 * N, Q2 = Q * Q;
    constexpr int NT = elem_threads<P>(WIDE), EPB = elem_per_block<P>(WIDE);
    constexpr int SA = 2 * Q * N2;     // [2][qz][i][j]
    constexpr int SB = 3 * N * Q2;     // [3][i][qy][qz]; first and last the element's nodal values
    constexpr int ITER = (EPB * NL + NT - 1) / NT;
    __shared__ T sA[EPB * SA];
    __shared__ T sB[EPB * SB];
    const int tid = threadIdx.x;
    const int64_t e0 = xcd_block(blockIdx.x, gridDim.x) * EPB;
    const int cnt = (int)min((int64_t)EPB, a.ne - e0) * NL;
    const T* __restrict__ L = a.tabs;
    const T* __restrict__ D = a.tabs + N * Q;
    const T* __restrict__ gq = a.tabs + 2 * N * Q;
    const T* __restrict__ wq = gq + Q;
    // gather
    {
        const int32_t* __restrict__ map = a.map + e0 * NL;
        const T* __restrict__ v = a.v;
        int32_t g[ITER];
        T x[ITER];
#pragma unroll
        for (int it = 0; it < ITER; ++it) g[it] = map[min(tid + it * NT, cnt - 1)];
#pragma unroll
        for (int it = 0; it < ITER; ++it) x[it] = v[max(g[it], 0)];
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            const int t = tid + it * NT;
            if (t < EPB * NL) sB[(t / NL) * SB + t % NL] = g[it] >= 0 ? x[it] : T(0);
        }
    }
    __syncthreads();
    // z: nodal lines to Gauss points, values and derivatives
    for (int t = tid; t < EPB * N2; t += NT) {
        const int el = t / N2, ij = t % N2;
        T u[N];
#pragma unroll
        for (int k = 0; k < N; ++k) u[k] = sB[el * SB + ij * N + k];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            T s0 = L[q] * u[0], s1 = D[q] * u[0];
#pragma unroll
            for (int k = 1; k < N; ++k) {
                s0 += L[k * Q + q] * u[k];
                s1 += D[k * Q + q] * u[k];
            }
            sA[el * SA + q * N2 + ij] = s0;
            sA[el * SA + (Q + q) * N2 + ij] = s1;
        }
    }
    __syncthreads();
    // y
    for (int t = tid; t < EPB * N * Q; t += NT) {
        const int el = t / (N * Q), r = t % (N * Q), qz = r / N, i = r % N;
        T a0[N], a1[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            a0[j] = sA[el * SA + r * N + j];
            a1[j] = sA[el * SA + Q * N2 + r * N + j];
        }
        T* out = sB + el * SB + i * Q2 + qz;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            T s0 = L[q] * a0[0], s1 = D[q] * a0[0], s2 = L[q] * a1[0];
#pragma unroll
            for (int j = 1; j < N; ++j) {
                s0 += L[j * Q + q] * a0[j];
                s1 += D[j * Q + q] * a0[j];
                s2 += L[j * Q + q] * a1[j];
            }
            out[q * Q] = s0;
            out[N * Q2 + q * Q] = s1;
            out[2 * N * Q2 + q * Q] = s2;
        }
    }
    __syncthreads();
    // x, the quadrature points of one x line per thread, and x back
    if (tid < EPB * Q2) {
        const int el = tid / Q2, r = tid % Q2;
        const int64_t e = min(e0 + el, a.ne - 1);
        T c[ELEM_COEF];
#pragma unroll
        for (int m = 0; m < ELEM_COEF; ++m) c[m] = a.coef[m * a.ne + e];
        const T eta = gq[r / Q], zeta = gq[r % Q];
        const T wyz = wq[r / Q] * wq[r % Q];
        // columns of the Jacobian: dx/dxi is fixed on the line, the others are linear in xi
        T ax[3], b0[3], b1[3], d0[3], d1[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            // c: xi, eta, zeta, xi eta, xi zeta, eta zeta, xi eta zeta
            ax[m] = c[m] + c[9 + m] * eta + (c[12 + m] + c[18 + m] * eta) * zeta;
            b0[m] = c[3 + m] + c[15 + m] * zeta;
            b1[m] = c[9 + m] + c[18 + m] * zeta;
            d0[m] = c[6 + m] + c[15 + m] * eta;
            d1[m] = c[12 + m] + c[18 + m] * eta;
        }
        T* col = sB + el * SB + r;
        T u0[N], u1[N], u2[N], o0[N], o1[N], o2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            u0[i] = col[i * Q2];
            u1[i] = col[(N + i) * Q2];
            u2[i] = col[(2 * N + i) * Q2];
            o0[i] = o1[i] = o2[i] = T(0);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            T val = L[q] * u0[0], ux = D[q] * u0[0], uy = L[q] * u1[0], uz = L[q] * u2[0];
#pragma unroll
            for (int i = 1; i < N; ++i) {
                val += L[i * Q + q] * u0[i];
                ux += D[i * Q + q] * u0[i];
                uy += L[i * Q + q] * u1[i];
                uz += L[i * Q + q] * u2[i];
            }
            const T xi = gq[q];
            T b[3], d[3], gx[3], gy[3], gz[3], V[3];
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                b[m] = b0[m] + b1[m] * xi;
                d[m] = d0[m] + d1[m] * xi;
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const int m1 = (m + 1) % 3, m2 = (m + 2) % 3;
                gx[m] = b[m1] * d[m2] - b[m2] * d[m1];
                gy[m] = d[m1] * ax[m2] - d[m2] * ax[m1];
                gz[m] = ax[m1] * b[m2] - ax[m2] * b[m1];
            }
            const T det = ax[0] * gx[0] + ax[1] * gx[1] + ax[2] * gx[2];
            const T w = wq[q] * wyz;
            const T s = w * recip(det);
#pragma unroll
            for (int m = 0; m < 3; ++m) V[m] = s * (gx[m] * ux + gy[m] * uy + gz[m] * uz);
            const T fx = gx[0] * V[0] + gx[1] * V[1] + gx[2] * V[2];
            const T fy = gy[0] * V[0] + gy[1] * V[1] + gy[2] * V[2];
            const T fz = gz[0] * V[0] + gz[1] * V[1] + gz[2] * V[2];
            const T fm = a.lambda * w * det * val;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                o0[i] += D[i * Q + q] * fx;
                o0[i] += L[i * Q + q] * fm;
                o1[i] += L[i * Q + q] * fy;
                o2[i] += L[i * Q + q] * fz;
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            col[i * Q2] = o0[i];
            col[(N + i) * Q2] = o1[i];
            col[(2 * N + i) * Q2] = o2[i];
        }
    }
    __syncthreads();
    // y back
    for (int t = tid; t < EPB * N * Q; t += NT) {
        const int el = t / (N * Q), r = t % (N * Q), qz = r / N, i = r % N;
        const T* in = sB + el * SB + i * Q2 + qz;
        T c0[Q], c1[Q], c2[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            c0[q] = in[q * Q];
            c1[q] = in[N * Q2 + q * Q];
            c2[q] = in[2 * N * Q2 + q * Q];
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            T s0 = L[j * Q] * c0[0], s1 = L[j * Q] * c2[0];
            s0 += D[j * Q] * c1[0];
#pragma unroll
            for (int q = 1; q < Q; ++q) {
                s0 += L[j * Q + q] * c0[q];
                s0 += D[j * Q + q] * c1[q];
                s1 += L[j * Q + q] * c2[q];
            }
            sA[el * SA + r * N + j] = s0;
            sA[el * SA + Q * N2 + r * N + j] = s1;
        }
    }
    __syncthreads();
    // z back
    for (int t = tid; t < EPB * N2; t += NT) {
        const int el = t / N2, ij = t % N2;
        T d0[Q], d1[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            d0[q] = sA[el * SA + q * N2 + ij];
            d1[q] = sA[el * SA + (Q + q) * N2 + ij];
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            T s = L[k * Q] * d0[0];
            s += D[k * Q] * d1[0];
#pragma unroll
            for (int q = 1; q < Q; ++q) {
                s += L[k * Q + q] * d0[q];
                s += D[k * Q + q] * d1[q];
            }
            sB[el * SB + ij * N + k] = s;
        }
    }
    __syncthreads();
    T* __restrict__ ev = a.ev + e0 * NL;
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        const int t = tid + it * NT;
        if (t < cnt) ev[t] = sB[(t / NL) * SB + t % NL];
    }
}

// One thread per node: its entries of ev in ascending element order, then the
// row epilogue.  A node without entries is constrained (identity row).
template <typename T, int MODE>
__global__ void __launch_bounds__(NODE_THREADS) element_node_kernel(SpmvArgs<T> a, const int32_t* __restrict__ ptr,
                                                                    const int32_t* __restrict__ ent,
                                                                    const T* __restrict__ ev) {
    if (a.stop != nullptr && *a.stop != 0) return;
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
            for (int32_t j = s; j < e; ++j) y += ev[ent[j]];
            if (s == e) y = a.v[row];
        }
        epilogue_store<T, MODE>(a, row, y, in, dot, dot2);
    }
    if constexpr (has_partials<MODE>()) {
        __shared__ double red[2 * NODE_THREADS / WAVE];
        block_sum_to0<NODE_THREADS, n_partials<MODE>()>(red, threadIdx.x, dot, dot2);
        if (threadIdx.x == 0) {
            a.partial[lb] = dot;
            if (MODE == SPMV_RINIT) a.partial[a.nblk + lb] = dot2;
        }
    }
}

template <typename T, int P, bool WIDE>
void launch_element_kernel(const ElemArgs<T>& a, hipEvent_t ev_start, hipStream_t s) {
    constexpr int EPB = elem_per_block<P>(WIDE);
    const dim3 grid((unsigned)((a.ne + EPB - 1) / EPB)), block(elem_threads<P>(WIDE));
    if (ev_start != nullptr)
        hipExtLaunchKernelGGL((element_kernel<T, P, WIDE>), grid, block, 0, s, ev_start, nullptr, 0, a);
    else
        element_kernel<T, P, WIDE><<<grid, block, 0, s>>>(a);
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

template <typename T, int MODE>
void launch_node_kernel(const SpmvArgs<T>& a, const ElementForm& E, const T* ev, hipStream_t s) {
    const dim3 grid((unsigned)a.nblk), block(NODE_THREADS);
    if (a.ev_stop != nullptr)
        hipExtLaunchKernelGGL((element_node_kernel<T, MODE>), grid, block, 0, s, nullptr, a.ev_stop, 0, a,
                              E.nptr.get(), E.nent.get(), ev);
    else
        element_node_kernel<T, MODE><<<grid, block, 0, s>>>(a, E.nptr.get(), E.nent.get(), ev);
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
        default: throw Error(GIAMG_EINVAL, "unknown product mode of the element form");
    }
    GIAMG_HIP(hipGetLastError());
}
template void launch_element_product<double>(int, const SpmvArgs<double>&, hipStream_t);
template void launch_element_product<float>(int, const SpmvArgs<float>&, hipStream_t);

void build_element_form(ElementForm& E, const std::vector<double>& corners, const int32_t* l2g, int64_t ne, int p,
                        int64_t n, double lambda, const std::vector<uint8_t>& cons, int basis, bool mixed,
                        hipStream_t s) {
    const int n1 = p + 1, nq = p + 2;
    const int64_t m = ne * n1 * n1 * n1;
    E.order = p;
    E.ne = ne;
    E.lambda = lambda;
    std::vector<int32_t> map((size_t)m);
    parallel_for(m, 1 << 16, [&](int64_t b, int64_t e) {
        for (int64_t i = b; i < e; ++i) map[i] = cons[l2g[i]] ? -1 : l2g[i];
    });
    E.map.alloc(m);
    GIAMG_HIP(hipMemcpyAsync(E.map.get(), map.data(), m * sizeof(int32_t), hipMemcpyHostToDevice, s));
    // x = sum over the corners of X_c (1 +- xi)(1 +- eta)(1 +- zeta) / 8; corner c = 4 i + 2 j + k
    std::vector<double> coef((size_t)ELEM_COEF * ne);
    const int sub[7] = {4, 2, 1, 6, 5, 3, 7};   // xi, eta, zeta, xi eta, xi zeta, eta zeta, xi eta zeta
    parallel_for(ne, 1 << 12, [&](int64_t b, int64_t en) {
        for (int64_t e = b; e < en; ++e)
            for (int t = 0; t < 7; ++t)
                for (int r = 0; r < 3; ++r) {
                    double v = 0.0;
                    for (int c = 0; c < 8; ++c) {
                        const int low = __builtin_popcount(sub[t] & ~c) & 1;   // one minus sign per -1 side
                        v += (low ? -1.0 : 1.0) * corners[(size_t)e * 24 + c * 3 + r];
                    }
                    coef[(size_t)(3 * t + r) * ne + e] = 0.125 * v;
                }
    });
    E.coef.alloc(coef.size());
    GIAMG_HIP(hipMemcpyAsync(E.coef.get(), coef.data(), coef.size() * sizeof(double), hipMemcpyHostToDevice, s));
    std::vector<double> L, D, g, w;
    reference_tables(p, basis, L, D, g, w);
    std::vector<double> tabs(L);
    for (const auto* v : {&D, &g, &w}) tabs.insert(tabs.end(), v->begin(), v->end());
    GIAMG_REQUIRE((int)tabs.size() == 2 * n1 * nq + 2 * nq, "unexpected size of the 1-D tables");
    E.tabs.alloc(tabs.size());
    GIAMG_HIP(hipMemcpyAsync(E.tabs.get(), tabs.data(), tabs.size() * sizeof(double), hipMemcpyHostToDevice, s));
    if (mixed) {
        E.coef32.alloc(coef.size());
        launch_convert<double, float>((int64_t)coef.size(), E.coef.get(), E.coef32.get(), s);
        E.tabs32.alloc(tabs.size());
        launch_convert<double, float>((int64_t)tabs.size(), E.tabs.get(), E.tabs32.get(), s);
    }
    // node -> entries
    DevBuf<int32_t> counts((size_t)n);
    GIAMG_HIP(hipMemsetAsync(counts.get(), 0, n * sizeof(int32_t), s));
    node_count_kernel<<<setup_grid(m), 256, 0, s>>>(m, E.map.get(), counts.get());
    GIAMG_HIP(hipGetLastError());
    std::vector<int32_t> hc((size_t)n), ptr((size_t)n + 1, 0);
    GIAMG_HIP(hipMemcpyAsync(hc.data(), counts.get(), n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    GIAMG_HIP(hipStreamSynchronize(s));
    for (int64_t i = 0; i < n; ++i) ptr[i + 1] = ptr[i] + hc[i];
    E.nptr.alloc((size_t)n + 1);
    E.nent.alloc((size_t)std::max<int32_t>(ptr[n], 1));
    GIAMG_HIP(hipMemcpyAsync(E.nptr.get(), ptr.data(), ptr.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    GIAMG_HIP(hipMemsetAsync(counts.get(), 0, n * sizeof(int32_t), s));
    node_place_kernel<<<setup_grid(m), 256, 0, s>>>(m, E.map.get(), E.nptr.get(), counts.get(), E.nent.get());
    node_sort_kernel<<<setup_grid(n), 256, 0, s>>>(n, E.nptr.get(), E.nent.get());
    GIAMG_HIP(hipGetLastError());
    E.ev.alloc((size_t)m);
    GIAMG_HIP(hipStreamSynchronize(s));   // the host arrays go out of scope
}

}  // namespace giamg
