// Row epilogues and fixed-order block sums shared by the product kernels
// (device code, internal).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace giamg {

constexpr int WAVE = 64;

// Row sums of groups of L lanes (L = 16, 4 or 1, each group inside one
// 16-lane DPP row): the same butterfly as group_sum<L> -- step k adds the
// value of the lane that differs in bit k, own value first -- done with DPP
// row rotations instead of LDS permutes.  After the step for bit 8 (4, 2)
// every value repeats with period 8 (4, 2) inside the group, so rotating by
// 4 (2, 1) reads exactly the xor partner's value: the sums are the
// butterfly's bit for bit.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                                 0xF, 0xF, false));
}
template <int L, typename T>
__device__ __forceinline__ T row_group_sum(T v) {
    static_assert(L == 16 || L == 4 || L == 1, "row groups of 16, 4 or 1 lanes");
    if constexpr (L == 16) {
        v += dpp_move<0x128>(v);   // row_ror:8  (xor 8)
        v += dpp_move<0x124>(v);   // row_ror:4  (xor 4 on period-8 values)
        v += dpp_move<0x122>(v);   // row_ror:2
        v += dpp_move<0x121>(v);   // row_ror:1
    } else if constexpr (L == 4) {
        v += dpp_move<0x4E>(v);    // quad_perm [2,3,0,1]  (xor 2)
        v += dpp_move<0xB1>(v);    // quad_perm [1,0,3,2]  (xor 1)
    }
    return v;
}

// Row-local operands of an epilogue, loaded before the row sum is known.
template <typename T>
struct RowIn {
    T f, dinv, r, x, v, y;
    double dr, drold;
};

template <typename T, int MODE>
__device__ __forceinline__ void epilogue_load(const SpmvArgs<T>& a, int64_t row, RowIn<T>& in) {
    constexpr bool cheb = MODE == SPMV_CHEB_STEP || MODE == SPMV_CHEB_DOT;
    constexpr bool jacobi = MODE == SPMV_JACOBI || MODE == SPMV_JACOBI_DOT;
    if constexpr (MODE == SPMV_RESID || MODE == SPMV_CHEB_INIT || jacobi || MODE == SPMV_RINIT)
        in.f = a.f[row];
    if constexpr (MODE == SPMV_CHEB_INIT || cheb || jacobi || MODE == SPMV_DINV || MODE == SPMV_RCHEB0)
        in.dinv = a.dinv[row];
    if constexpr (cheb) {
        in.r = a.r[row];
        in.x = (a.flags & CHEB_ASSIGN) ? T(0) : a.x[row];
    }
    if constexpr (cheb || jacobi || MODE == SPMV_DOT)
        in.v = a.v[row];
    if constexpr (MODE == SPMV_CHEB_DOT || MODE == SPMV_JACOBI_DOT) {
        in.dr = a.dot_r[row];
        if constexpr (sizeof(T) == 4) in.drold = a.dot_rold[row];
    }
    if constexpr (MODE == SPMV_ADD) in.y = a.y[row];
}

// Row epilogue: y is (A v)_row.  `dot` collects this row's share of a block
// partial (DOT: v.y; RINIT: f.f in dot, y.y in dot2; CHEB_DOT, JACOBI_DOT:
// dot_r . result and, in FP32, dot_rold . result).
template <typename T, int MODE>
__device__ __forceinline__ void epilogue_store(const SpmvArgs<T>& a, int64_t row, T y,
                                               const RowIn<T>& in, double& dot, double& dot2) {
    if constexpr (MODE == SPMV_PLAIN) {
        a.y[row] = y;
    } else if constexpr (MODE == SPMV_RESID) {
        a.y[row] = in.f - y;
    } else if constexpr (MODE == SPMV_ADD) {
        a.y[row] = in.y + y;
    } else if constexpr (MODE == SPMV_CHEB_INIT) {
        const T res = in.dinv * (in.f - y);
        a.r[row] = res;
        a.y[row] = res * a.inv_theta;
    } else if constexpr (MODE == SPMV_CHEB_STEP || MODE == SPMV_CHEB_DOT) {
        const T rr = in.r - in.dinv * y;
        const T dn = a.c1 * in.v + a.c2 * rr;
        a.r[row] = rr;
        a.y[row] = dn;
        const T inc = (a.flags & CHEB_LAST) ? in.v + dn : in.v;
        const T xn = in.x + inc;
        a.x[row] = xn;
        if constexpr (MODE == SPMV_CHEB_DOT) {
            dot += in.dr * (double)xn;
            if constexpr (sizeof(T) == 4) dot2 += in.drold * (double)xn;
        }
    } else if constexpr (MODE == SPMV_RCHEB0) {
        a.y[row] = y;
        const T res = in.dinv * y;
        a.r[row] = res;
        a.x[row] = res * a.inv_theta;
    } else if constexpr (MODE == SPMV_JACOBI || MODE == SPMV_JACOBI_DOT) {
        const T xn = in.v + a.omega * in.dinv * (in.f - y);
        a.y[row] = xn;
        if constexpr (MODE == SPMV_JACOBI_DOT) {
            dot += in.dr * (double)xn;
            if constexpr (sizeof(T) == 4) dot2 += in.drold * (double)xn;
        }
    } else if constexpr (MODE == SPMV_DOT) {
        a.y[row] = y;
        dot += (double)in.v * (double)y;
    } else if constexpr (MODE == SPMV_DINV) {
        a.y[row] = in.dinv * y;
    } else if constexpr (MODE == SPMV_RINIT) {
        const T ri = in.f - y;
        a.y[row] = ri;
        dot += (double)in.f * (double)in.f;
        dot2 += (double)ri * (double)ri;
    }
}

template <int MODE>
constexpr bool has_partials() {
    return MODE == SPMV_DOT || MODE == SPMV_RINIT || MODE == SPMV_CHEB_DOT || MODE == SPMV_JACOBI_DOT;
}

// Butterfly sum over the lanes of a wave with partners 32, 16, 8, 4, 2, 1 in
// that order (the order of group_sum<WAVE>): the two steps across 16-lane
// rows by LDS permutes, the four inside each row by DPP rotations
// (row_group_sum<16>).  Every lane ends with the same bits as
// group_sum<WAVE> gives.
__device__ __forceinline__ double wave_butterfly(double v) {
    v += __shfl_xor(v, 32, WAVE);
    v += __shfl_xor(v, 16, WAVE);
    return row_group_sum<16>(v);
}

// Fixed-order block sums of NV (1 or 2) values per thread, valid in thread 0
// only: each wave adds its lanes by the butterfly above, then thread 0 adds
// the waves' sums in wave order.  One barrier; red holds 2 * NT / WAVE
// doubles and may be reused after a further barrier.
template <int NT, int NV>
__device__ __forceinline__ void block_sum_to0(double* red, int tid, double& a, double& b) {
    static_assert(NV == 1 || NV == 2, "one or two sums");
    constexpr int NW = NT / WAVE;
    a = wave_butterfly(a);
    if constexpr (NV == 2) b = wave_butterfly(b);
    if (tid % WAVE == 0) {
        red[tid / WAVE] = a;
        if constexpr (NV == 2) red[NW + tid / WAVE] = b;
    }
    __syncthreads();
    if (tid == 0) {
        a = red[0];
        if constexpr (NV == 2) b = red[NW];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            a += red[w];
            if constexpr (NV == 2) b += red[NW + w];
        }
    }
}

template <typename T, int MODE>
constexpr int n_partials() {
    return MODE == SPMV_RINIT || (sizeof(T) == 4 && (MODE == SPMV_CHEB_DOT || MODE == SPMV_JACOBI_DOT)) ? 2 : 1;
}

// Row-local tail of a block product: acc = (A v)[row][col].
template <typename T, int MODE>
__device__ __forceinline__ void spmm_epilogue(const SpmmArgs<T>& a, int64_t row, int64_t col, T acc) {
    const int64_t idx = row * a.k + col;
    if constexpr (MODE == SPMV_PLAIN) {
        a.y[idx] = acc;
    } else if constexpr (MODE == SPMV_RESID) {
        a.y[idx] = a.f[idx] - acc;
    } else if constexpr (MODE == SPMV_ADD) {
        a.y[idx] += acc;
    } else if constexpr (MODE == SPMV_CHEB_INIT) {
        const T res = a.dinv[row] * (a.f[idx] - acc);
        a.r[idx] = res;
        a.y[idx] = res * a.inv_theta;
    } else if constexpr (MODE == SPMV_CHEB_STEP) {
        const T rr = a.r[idx] - a.dinv[row] * acc;
        const T dold = a.v[idx];
        const T dn = a.c1 * dold + a.c2 * rr;
        a.r[idx] = rr;
        a.y[idx] = dn;
        const T inc = (a.flags & CHEB_LAST) ? dold + dn : dold;
        a.x[idx] = ((a.flags & CHEB_ASSIGN) ? T(0) : a.x[idx]) + inc;
    } else if constexpr (MODE == SPMV_JACOBI) {
        a.y[idx] = a.v[idx] + a.omega * a.dinv[row] * (a.f[idx] - acc);
    }
}

}  // namespace giamg
