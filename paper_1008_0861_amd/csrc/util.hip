// Small kernels of libasd: the 2-D transpose between the two state layouts,
// a standalone FP64 reduction of a state, fills and copies.
#include "asd_device.h"
#include "asd_launch.h"

namespace asd {

// 2-D transpose: in [ny][nx] -> out [nx][ny].  A block takes a 64 x 64 tile
// through LDS (a padded row: conflict-free both ways).  A wave loads and
// stores 64 consecutive elements: whole cache lines where the rows of that
// side start on them; elsewhere neighbouring tiles share each row's edge lines.
// A thread's sixteen loads are all in flight before the first is used.
template <typename T>
__global__ void __launch_bounds__(256) transpose_kernel(const T* __restrict__ in, T* __restrict__ out, int nx, int ny) {
    constexpr int W = 64, R = 16;
    __shared__ T tile[W][W + 1];
    const int tilesx = (nx + W - 1) / W;
    int b = blockIdx.x;
    // neighbouring tiles on one XCD (they share lines at ragged edges)
    if ((gridDim.x & 7) == 0) b = (b & 7) * (gridDim.x >> 3) + (b >> 3);
    const int x0 = (b % tilesx) * W, y0 = (b / tilesx) * W;
    const int lx = threadIdx.x & 63, ly = threadIdx.x >> 6;
    T v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int x = min(x0 + lx, nx - 1), y = min(y0 + ly + 4 * r, ny - 1);
        v[r] = in[(int64_t)y * nx + x];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) tile[ly + 4 * r][lx] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int x = x0 + ly + 4 * r, y = y0 + lx;
        if (x < nx && y < ny) out[(int64_t)x * ny + y] = tile[lx][ly + 4 * r];
    }
}

template <typename T>
hipError_t launch_transpose(const T* in, T* out, int nx, int ny, hipStream_t st) {
    const int64_t nb = (int64_t)((nx + 63) / 64) * ((ny + 63) / 64);
    hipLaunchKernelGGL(transpose_kernel<T>, dim3((unsigned)nb), dim3(256), 0, st, in, out, nx, ny);
    return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(256) reduce_kernel(const T* __restrict__ x, int64_t N, ReduceParams R) {
    // partials only; a later launch folds them
    constexpr int U = 8;  // loads in flight per thread
    double s4[U] = {}, mn = __builtin_huge_val(), mx = -__builtin_huge_val();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i0 < N; i0 += U * stride) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = x[i0 + u * stride < N ? i0 + u * stride : i0];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s4[u] += i0 + u * stride < N ? (double)v[u] : 0.0;
            mn = fmin(mn, (double)v[u]);
            mx = fmax(mx, (double)v[u]);
        }
    }
    const double s = ((s4[0] + s4[1]) + (s4[2] + s4[3])) + ((s4[4] + s4[5]) + (s4[6] + s4[7]));
    block_partials(R.partials, s, mn, mx);
}

__global__ void __launch_bounds__(1024) fold_kernel(FoldParams f) { fold_partials(f); }

hipError_t launch_fold(const FoldParams& f, hipStream_t st) {
    if (f.count < 1) return hipSuccess;
    hipLaunchKernelGGL(fold_kernel, dim3(f.count), dim3(f.nblocks > 1024 ? 1024 : 256), 0, st, f);
    return hipGetLastError();
}

int reduce_num_blocks(int64_t N) {
    int64_t nb = (N + 256 * 8 - 1) / (256 * 8);
    if (nb < 1) nb = 1;
    if (nb > 1024) nb = 1024;
    return (int)nb;
}

template <typename T>
hipError_t launch_reduce(const T* x, int64_t N, const ReduceParams& R, int nblocks, hipStream_t st) {
    hipLaunchKernelGGL(reduce_kernel<T>, dim3(nblocks), dim3(256), 0, st, x, N, R);
    return hipGetLastError();
}

__global__ void fill_u32_kernel(unsigned* p, unsigned v, int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void fill_f64_kernel(double* p, double v, int64_t n) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
hipError_t launch_fill_u32(unsigned* p, unsigned v, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}
hipError_t launch_fill_f64(double* p, double v, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

// Plain streaming copy (also the calibration kernel for HBM byte counters).
template <typename T>
__global__ void __launch_bounds__(256) copy_kernel(const T* __restrict__ in, T* __restrict__ out, int64_t N) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = in[i];
}
template <typename T>
hipError_t launch_copy(const T* in, T* out, int64_t N, hipStream_t st) {
    int64_t nb = (N + 255) / 256;
    if (nb > 8192) nb = 8192;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(copy_kernel<T>, dim3((unsigned)nb), dim3(256), 0, st, in, out, N);
    return hipGetLastError();
}

// Streaming copy for the practical bandwidth ceiling: 16-byte accesses,
// each thread keeps kWideUnroll loads in flight before its stores, and the
// block's accesses of one round are contiguous (coalesced).  nvec 16-byte
// vectors; the caller copies any remainder.
static constexpr int kWideUnroll = 4;
__global__ void __launch_bounds__(256) copy_wide_kernel(const float4* __restrict__ in, float4* __restrict__ out,
                                                        int64_t nvec) {
    const int64_t base = (int64_t)blockIdx.x * (256 * kWideUnroll) + threadIdx.x;
    float4 v[kWideUnroll];
#pragma unroll
    for (int j = 0; j < kWideUnroll; ++j) {
        const int64_t i = base + j * 256;
        if (i < nvec) v[j] = in[i];
    }
#pragma unroll
    for (int j = 0; j < kWideUnroll; ++j) {
        const int64_t i = base + j * 256;
        if (i < nvec) out[i] = v[j];
    }
}
hipError_t launch_copy_wide(const void* in, void* out, size_t nbytes, hipStream_t st) {
    const int64_t nvec = (int64_t)(nbytes / 16);
    if (nvec > 0) {
        const int64_t nb = (nvec + 256 * kWideUnroll - 1) / (256 * kWideUnroll);
        if (nb > INT32_MAX) return hipErrorInvalidValue;
        hipLaunchKernelGGL(copy_wide_kernel, dim3((unsigned)nb), dim3(256), 0, st, (const float4*)in, (float4*)out,
                           nvec);
    }
    const int64_t tail = (int64_t)(nbytes - 16 * (size_t)nvec) / 4;  // nbytes is a multiple of 4
    if (tail > 0)
        hipLaunchKernelGGL(copy_kernel<float>, dim3(1), dim3(256), 0, st, (const float*)in + 4 * nvec,
                           (float*)out + 4 * nvec, tail);
    return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(256) axpy_kernel(T* __restrict__ y, const T* __restrict__ x, T a, int64_t N) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] += a * x[i];
}
template <typename T>
hipError_t launch_axpy(T* y, const T* x, T a, int64_t N, hipStream_t st) {
    int64_t nb = (N + 255) / 256;
    if (nb > 8192) nb = 8192;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(axpy_kernel<T>, dim3((unsigned)nb), dim3(256), 0, st, y, x, a, N);
    return hipGetLastError();
}

#define ASD_INST(T)                                                                          \
    template hipError_t launch_transpose<T>(const T*, T*, int, int, hipStream_t);             \
    template hipError_t launch_reduce<T>(const T*, int64_t, const ReduceParams&, int, hipStream_t); \
    template hipError_t launch_copy<T>(const T*, T*, int64_t, hipStream_t);                  \
    template hipError_t launch_axpy<T>(T*, const T*, T, int64_t, hipStream_t);
ASD_INST(float)
ASD_INST(double)
#undef ASD_INST

}  // namespace asd
