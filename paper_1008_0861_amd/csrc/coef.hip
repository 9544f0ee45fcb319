// Face coefficients of one sweep direction (section 2): at the face between
// cell c and c + e_d,
//     b_f     = (b_c + b_{c+e_d}) / 2      (arithmetic mean, not renormalised)
//     chi_f   = chi_par, or the harmonic mean of the two cells' chi (a per-cell
//               field, or chi_par (U / T_ref)^p of a state U, section 3.3)
//     alpha_f = dt (chi_perp + (chi_f - chi_perp) b_d,f^2) / h_d^2
//     beta_t  = dt (chi_f - chi_perp) b_d,f b_t,f / (h_d h_t)
// A wall face (c on the last plane) gets zeros, except with T = 0 walls:
// there the entry holds the wall coefficients of the line (the right wall's
// alpha in alpha, the left wall's in beta1), each from its own cell's b and
// chi, since the wall face has no second cell.
// Computed in FP64 and rounded once to the grid's type.  With a constant or
// per-cell chi they depend on dt, b and chi only and a step loop computes
// them once; with chi(T) they are recomputed from each sweep's input.
#include <algorithm>

#include "asd_device.h"
#include "asd_launch.h"

namespace asd {

// chi of one cell: the per-cell field (index i), chi_par (U / T_ref)^p of the
// state (index o in the sweep-input layout), or chi_par
template <typename T>
__device__ __forceinline__ double coef_cell_chi(const CoefParams<T>& C, int i, int o) {
    if (C.U) return C.chi_par * pow((double)C.U[o] / C.chi_tref, C.chi_exp);
    if (C.chi) return (double)C.chi[i];
    return C.chi_par;
}

// The coefficients of the face after cell xyz (index i), chi0 and chi1 the
// chi of its two cells (unused with a constant chi): alpha, beta1, beta2.
struct FaceCoef {
    double a, b1, b2;
};
template <typename T>
__device__ __forceinline__ FaceCoef face_coef(const CoefParams<T>& C, int i, int j, bool wall, double chi0, double chi1) {
    FaceCoef f{0.0, 0.0, 0.0};
    if (!wall) {
        double bf[3] = {0.0, 0.0, 0.0};
        for (int q = 0; q < C.ndim; ++q) bf[q] = 0.5 * ((double)C.b[q][i] + (double)C.b[q][j]);
        double chif = C.chi_par;
        if (C.U || C.chi) chif = (chi0 + chi1) != 0.0 ? 2.0 * chi0 * chi1 / (chi0 + chi1) : 0.0;
        const double dpar = chif - C.chi_perp;
        f.a = C.cnn * (C.chi_perp + dpar * bf[C.d] * bf[C.d]);
        f.b1 = C.ct1 * dpar * bf[C.d] * bf[C.t1];
        if (C.ndim == 3) f.b2 = C.ct2 * dpar * bf[C.d] * bf[C.t2];
    } else if (C.dirichlet) {
        // right wall from cell i (last of its line), left wall from cell j (first)
        const double bi = (double)C.b[C.d][i], bj = (double)C.b[C.d][j];
        f.a = C.cnn * (C.chi_perp + (chi0 - C.chi_perp) * bi * bi);
        f.b1 = C.cnn * (C.chi_perp + (chi1 - C.chi_perp) * bj * bj);
    }
    return f;
}

// One thread per cell: the x sweep, whose output has the input's layout, and
// the other sweeps of small and thin grids (coef_by_cells), written to the
// output layout directly.
template <typename T, bool X>
__global__ void __launch_bounds__(256) coef_cell_kernel(CoefParams<T> C) {
    const int nx = C.n[0], ny = C.n[1], nz = C.n[2];
    const int N = nx * ny * nz;
    // 64-bit loop index: the stride would overflow int near N = 2^31 (each i < N fits an int)
    for (int64_t i64 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i64 < N; i64 += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)i64, x = i % nx;
        int j, o, oj;  // the next cell, and both in the output layout
        bool last;
        if constexpr (X) {
            last = x + 1 == nx;
            o = i;
            oj = j = last ? i - x : i + 1;
        } else {
            const int c[3] = {x, (i / nx) % ny, i / (nx * ny)};
            const int back = C.n[C.d] - 1, st = C.d == 1 ? nx : nx * ny;
            last = c[C.d] == back;
            o = x * C.so[0] + c[1] * C.so[1] + c[2] * C.so[2];
            j = last ? i - back * st : i + st;
            oj = last ? o - back : o + 1;
        }
        const FaceCoef f = face_coef<T>(C, i, j, last && !C.periodic, coef_cell_chi<T>(C, i, o), coef_cell_chi<T>(C, j, oj));
        C.alpha[o] = (T)f.a;
        C.beta1[o] = (T)f.b1;
        if (C.ndim == 3) C.beta2[o] = (T)f.b2;
    }
}

// y and z sweeps: the output has the sweep axis (t) fastest, the input x.  A
// block takes a 32 x 32 tile of the (t, x) plane at one coordinate of the
// third axis: it reads b (and chi) along x and writes through LDS along t (a
// thread per cell writing the output layout directly takes one cache line per
// 4 or 8 bytes: 256^3 FP32 616 us per axis on average, now 170; 4096^2 163 and
// 112).  A state U is in the output layout:
// it is read along t, with the tile's next t, through the same LDS.
template <typename T>
__global__ void __launch_bounds__(256) coef_t_kernel(CoefParams<T> C) {
    constexpr int W = 32;
    __shared__ double tile[3][W][W + 1];  // [output array][t][x]
    __shared__ double chi_u[W + 1][W + 1];  // [t, and the next][x]
    const int d = C.d, w = C.ndim == 3 ? 3 - d : 2;  // the third axis (2-D: z, of length 1)
    const int nx = C.n[0], nt = C.n[d];
    const int st = d == 1 ? nx : nx * C.n[1], sw = d == 1 ? nx * C.n[1] : nx;
    const int tilesx = (nx + W - 1) / W, tilest = (nt + W - 1) / W;
    int b = blockIdx.x;
    const int x0 = (b % tilesx) * W;
    b /= tilesx;
    const int t0 = (b % tilest) * W, zw = b / tilest;
    const int lx = threadIdx.x & 31, ly = threadIdx.x >> 5;
    const int ob = C.so[0] * x0 + (C.ndim == 3 ? C.so[w] * zw : 0);  // output offset of (x0, t = 0)
    if (C.U) {
        for (int r = ly; r < W; r += 8)         // x0 + r
            for (int q = lx; q <= W; q += 32) {  // t0 + q, wrapping past the line's end
                const int t = t0 + q < nt ? t0 + q : (t0 + q == nt ? 0 : nt - 1);
                if (x0 + r < nx)
                    chi_u[q][r] = C.chi_par * pow((double)C.U[ob + C.so[0] * r + t] / C.chi_tref, C.chi_exp);
            }
        __syncthreads();
    }
    for (int r = ly; r < W; r += 8) {
        const int x = x0 + lx, t = t0 + r;
        if (x < nx && t < nt) {
            const bool last = t + 1 == nt;
            const int i = x + t * st + zw * sw, j = last ? x + zw * sw : i + st;
            const double c0 = C.U ? chi_u[r][lx] : C.chi ? (double)C.chi[i] : C.chi_par;
            const double c1 = C.U ? chi_u[r + 1][lx] : C.chi ? (double)C.chi[j] : C.chi_par;
            const FaceCoef f = face_coef<T>(C, i, j, last && !C.periodic, c0, c1);
            tile[0][r][lx] = f.a;
            tile[1][r][lx] = f.b1;
            tile[2][r][lx] = f.b2;
        }
    }
    __syncthreads();
    for (int r = ly; r < W; r += 8) {
        const int t = t0 + lx;
        if (x0 + r < nx && t < nt) {
            const int o = ob + C.so[0] * r + t;
            C.alpha[o] = (T)tile[0][lx][r];
            C.beta1[o] = (T)tile[1][lx][r];
            if (C.ndim == 3) C.beta2[o] = (T)tile[2][lx][r];
        }
    }
}

// The y and z sweeps' tiles need enough of them to fill the chip, more so with
// chi(T), whose power takes longest.  us per one-step call that computes the
// coefficients, cells / tiles: 256^2 FP32 15.1 / 16.1, 400^2 21.2 / 21.0, 64^3
// with a per-cell chi 36.5 / 39.0, 80^3 67.7 / 54.8; chi(T), us per step: 256^2
// 17.6 / 24.9, 600^2 39.1 / 41.7, 64^3 45.3 / 54.4, 80^3 81.2 / 78.8.  Short lines
// and chi(T), 300 x 300 x 4: 86 / 124, x 12 FP32 157 / 173, FP64 235 / 211; rows
// shorter than half a tile, 8 x 400 x 400: 159 / 315.  (A thread per cell of a row
// in chunks of 256 idles on short rows in the x sweep: 64 x 300 x 300 FP32 329,
// 294 by cells.)
static bool coef_by_cells(int es, int ndim, int d, const int n[3], bool of_T) {
    const int64_t N = (int64_t)n[0] * n[1] * n[2];
    return d == 0 || N <= (of_T ? 1 << 19 : ndim == 3 ? 1 << 18 : 1 << 17) || n[0] < 16 || (of_T && n[d] <= 48 / es);
}

template <typename T>
hipError_t launch_coef(const CoefParams<T>& C, hipStream_t st) {
    if (C.so[C.d] != 1) return hipErrorInvalidValue;  // the sweep's input layout: its axis fastest
    if (C.d == 0 && (C.so[1] != C.n[0] || (C.ndim == 3 && C.so[2] != C.n[0] * C.n[1]))) return hipErrorInvalidValue;
    if (coef_by_cells((int)sizeof(T), C.ndim, C.d, C.n, C.U != nullptr)) {
        const int64_t nb = std::min<int64_t>(((int64_t)C.n[0] * C.n[1] * C.n[2] + 255) / 256, 16384);
        if (C.d == 0) hipLaunchKernelGGL((coef_cell_kernel<T, true>), dim3((unsigned)nb), dim3(256), 0, st, C);
        else hipLaunchKernelGGL((coef_cell_kernel<T, false>), dim3((unsigned)nb), dim3(256), 0, st, C);
    } else {
        const int w = C.ndim == 3 ? 3 - C.d : 2;
        const int64_t nb = (int64_t)((C.n[0] + 31) / 32) * ((C.n[C.d] + 31) / 32) * C.n[w];
        hipLaunchKernelGGL(coef_t_kernel<T>, dim3((unsigned)nb), dim3(256), 0, st, C);
    }
    return hipGetLastError();
}

template hipError_t launch_coef<float>(const CoefParams<float>&, hipStream_t);
template hipError_t launch_coef<double>(const CoefParams<double>&, hipStream_t);

}  // namespace asd
