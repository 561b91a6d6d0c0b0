// Dense inverse of the coarsest operator on the device (setup).
//
// Symmetric block sweeps: sweeping block k of a symmetric matrix M replaces
//   M_kk by -D,  M_ik by M_ik D,  M_ij by M_ij - M_ik D M_kj,   D = M_kk^-1,
// and keeps it symmetric; after all blocks M = -A^-1.  No pivoting: the pivots
// are those of the Cholesky factorisation, positive for an SPD matrix.  Only the
// lower triangle of 64 x 64 tiles is kept up to date, so the result is exactly
// symmetric.  A sweep is two launches: every block of the first inverts the
// diagonal tile for itself (in registers, 64 pivots of one barrier each) and
// forms its tile of the panel M_ik D; the second updates one tile per block.
// Both multiply by FP64 matrix instructions.  n = 1331: 1.3 ms where the host's
// Cholesky factorisation and solves took 86; bound by the chain of n / 64 pivot
// tiles up to a few thousand rows, by the n^3 multiply-adds above.  Largest error
// against extended precision, relative to the largest entry, device and host:
// 1331 rows 3.8e-15 and 2.6e-15, 729 rows of one pinned node 0.97e-14 and 2.3e-14.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace giamg {
namespace {

constexpr int TB = 64;            // tile
constexpr int TLD = TB + 2;       // its LDS rows: 16 rows of one column fall into distinct banks
constexpr int DENSE_THREADS = 256;
using f64x4 = __attribute__((ext_vector_type(4))) double;

__global__ void dense_scatter_kernel(int64_t n, const int64_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                     const double* __restrict__ val, double* __restrict__ m) {
    for (int64_t r = blockIdx.x; r < n; r += gridDim.x)
        for (int64_t j = rp[r] + threadIdx.x; j < rp[r + 1]; j += blockDim.x) m[r * n + ci[j]] = val[j];
}

// acc += the 16 x 64 strip of rows 16 w .. 16 w + 15 of A B (BT: of A B^T), A and B
// tiles in LDS; lane 16 g + c of acc[t][i] holds row 16 w + g + 4 i, column 16 t + c.
template <bool BT>
__device__ __forceinline__ void strip_product(const double* A, const double* B, int w, int lane, f64x4 (&acc)[4]) {
    const int g = lane / 16, c = lane % 16;
#pragma unroll 4
    for (int k = 0; k < TB; k += 4) {
        const double a = A[(16 * w + c) * TLD + k + g];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double b = BT ? B[(16 * t + c) * TLD + k + g] : B[(k + g) * TLD + 16 * t + c];
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[t], 0, 0, 0);
        }
    }
}

// Tile i of the panel of block k: rows of tile i, columns of tile k, zero past n,
// from the lower triangle (M_ki transposed above the diagonal).
__device__ __forceinline__ void load_panel(const double* m, int64_t n, int i, int k, double* sh) {
    const int64_t r0 = (int64_t)(i > k ? i : k) * TB, c0 = (int64_t)(i > k ? k : i) * TB;
    for (int t = threadIdx.x; t < TB * TB; t += DENSE_THREADS) {
        const int r = t / TB, c = t % TB;
        const double v = r0 + r < n && c0 + c < n ? m[(r0 + r) * n + c0 + c] : 0.0;
        sh[i > k ? r * TLD + c : c * TLD + r] = v;
    }
}

// Block i: D = M_kk^-1; P_i = M_ik and W_i = P_i D to pan and wid ([tiles][64][64]),
// W_i also in M_ik's place; block k leaves D in wid.  *bad is set at a pivot that
// is not positive.
__global__ void __launch_bounds__(DENSE_THREADS) dense_panel_kernel(int64_t n, int k, double* __restrict__ m,
                                                                    double* __restrict__ pan,
                                                                    double* __restrict__ wid, int* bad) {
    __shared__ double sa[TB * TLD], sd[TB * TLD], piv[2][TB];
    const int tid = threadIdx.x, i = blockIdx.x;
    const int tr = tid / 16 * 4, tc = tid % 16 * 4;   // this thread's 4 x 4 entries of M_kk
    const int64_t k0 = (int64_t)k * TB;
    double s[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int64_t r = k0 + max(tr + a, tc + b), c = k0 + min(tr + a, tc + b);
            s[a][b] = r < n ? m[r * n + c] : r == c ? 1.0 : 0.0;   // the last tile: identity past n
        }
    if (i != k) load_panel(m, n, i, k, sa);
    bool fail = false;
    for (int p0 = 0; p0 < TB; p0 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // pivot p: column p is in the registers of the threads tc == p0
            const int p = p0 + q;
            double* pv = piv[q & 1];
            if (tc == p0) {
#pragma unroll
                for (int a = 0; a < 4; ++a) pv[tr + a] = s[a][q];
            }
            __syncthreads();
            const double d = pv[p], inv = 1.0 / d;
            fail = fail || !(d > 0.0);
            double u[4], v[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                u[a] = pv[tr + a];
                v[a] = pv[tc + a] * inv;
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const bool row = tr + a == p, col = tc + b == p;
                    const double in = __builtin_fma(-u[a], v[b], s[a][b]);
                    s[a][b] = row && col ? -inv : row ? v[b] : col ? u[a] * inv : in;
                }
        }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) sd[(tr + a) * TLD + tc + b] = -s[a][b];
    __syncthreads();
    double* const pt = pan + (int64_t)i * TB * TB;
    double* const wt = wid + (int64_t)i * TB * TB;
    if (i == k) {
        if (tid == 0 && fail) *bad = 1;
        for (int t = tid; t < TB * TB; t += DENSE_THREADS) wt[t] = sd[t / TB * TLD + t % TB];
        return;
    }
    const int lane = tid % 64, w = tid / 64, g = lane / 16, c = lane % 16;
    f64x4 acc[4] = {};
    strip_product<false>(sa, sd, w, lane, acc);
    for (int t = tid; t < TB * TB; t += DENSE_THREADS) pt[t] = sa[t / TB * TLD + t % TB];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 16 * w + g + 4 * q, col = 16 * t + c;
            wt[row * TB + col] = acc[t][q];
            const int64_t r = (int64_t)i * TB + row, cc = k0 + col;
            if (r < n && cc < n) m[i > k ? r * n + cc : cc * n + r] = acc[t][q];
        }
}

// Tile (i, j), i >= j, of the update: M_ij -= P_i W_j^T; tile (k, k) becomes -D.
__global__ void __launch_bounds__(DENSE_THREADS) dense_update_kernel(int64_t n, int k, double* __restrict__ m,
                                                                     const double* __restrict__ pan,
                                                                     const double* __restrict__ wid) {
    __shared__ double sp[TB * TLD], sw[TB * TLD];
    const int i = blockIdx.x, j = blockIdx.y, tid = threadIdx.x;
    if (j > i || (i == k) != (j == k)) return;
    const int64_t r0 = (int64_t)i * TB, c0 = (int64_t)j * TB;
    if (i == k) {
        for (int t = tid; t < TB * TB; t += DENSE_THREADS) {
            const int64_t r = r0 + t / TB, c = c0 + t % TB;
            if (r < n && c < n) m[r * n + c] = -wid[(int64_t)k * TB * TB + t];
        }
        return;
    }
    for (int t = tid; t < TB * TB; t += DENSE_THREADS) {
        sp[t / TB * TLD + t % TB] = -pan[(int64_t)i * TB * TB + t];
        sw[t / TB * TLD + t % TB] = wid[(int64_t)j * TB * TB + t];
    }
    const int lane = tid % 64, w = tid / 64, g = lane / 16, c = lane % 16;
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = r0 + 16 * w + g + 4 * q, cc = c0 + 16 * t + c;
            acc[t][q] = r < n && cc < n ? m[r * n + cc] : 0.0;
        }
    __syncthreads();
    strip_product<true>(sp, sw, w, lane, acc);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = r0 + 16 * w + g + 4 * q, cc = c0 + 16 * t + c;
            if (r < n && cc < n) m[r * n + cc] = acc[t][q];
        }
}

// m = -m, the lower triangle mirrored.
__global__ void dense_mirror_kernel(int64_t n, double* __restrict__ m) {
    const int64_t r = blockIdx.x;
    for (int64_t c = threadIdx.x; c <= r; c += blockDim.x) {
        const double v = -m[r * n + c];
        m[r * n + c] = v;
        m[c * n + r] = v;
    }
}

}  // namespace

bool spd_inverse_device(const DevCSR& A, DevBuf<double>& inv, hipStream_t s) {
    const int64_t n = A.nrows;
    const int tiles = (int)((n + TB - 1) / TB);
    inv.alloc(n * n);
    DevBuf<double> pan((size_t)tiles * TB * TB), wid((size_t)tiles * TB * TB);
    DevBuf<int> bad(1);
    GIAMG_HIP(hipMemsetAsync(inv.get(), 0, (size_t)(n * n) * sizeof(double), s));
    GIAMG_HIP(hipMemsetAsync(bad.get(), 0, sizeof(int), s));
    dense_scatter_kernel<<<(unsigned)std::min<int64_t>(n, 65536), 64, 0, s>>>(n, A.rp.get(), A.ci.get(), A.val.get(),
                                                                            inv.get());
    for (int k = 0; k < tiles; ++k) {
        dense_panel_kernel<<<tiles, DENSE_THREADS, 0, s>>>(n, k, inv.get(), pan.get(), wid.get(), bad.get());
        dense_update_kernel<<<dim3(tiles, tiles), DENSE_THREADS, 0, s>>>(n, k, inv.get(), pan.get(), wid.get());
    }
    dense_mirror_kernel<<<(unsigned)n, 256, 0, s>>>(n, inv.get());
    GIAMG_HIP(hipGetLastError());
    int hbad = 0;
    GIAMG_HIP(hipMemcpyAsync(&hbad, bad.get(), sizeof(int), hipMemcpyDeviceToHost, s));
    GIAMG_HIP(hipStreamSynchronize(s));
    return hbad == 0;
}

}  // namespace giamg
