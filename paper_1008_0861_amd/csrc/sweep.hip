// One directional sweep of the split semi-implicit scheme (section 2,
// Eqs. xup / yup): kernel wrappers and launchers.  Two variants of the tile
// body compute the same sweep: face slots (sweep_tile.h: faces evaluated
// while the tile is staged, 8-byte LDS slots) and cell slots
// (sweep_cell.h: 16-byte cell slots, faces evaluated in the solve); the
// description of the method and of its gfx950 mapping is in those files.
#include "sweep_cell.h"
#include "sweep_tile.h"

namespace asd {

// The parameters every wave needs before its first global load arrive as
// leading scalar arguments, which the build preloads into scalar registers
// at wave launch (gfx950 kernel-argument preloading, at most 14 dwords): the
// wave then issues its loads without first waiting on a scalar load of the
// argument block.  The remaining fields are read from P as usual; the
// leading arguments override the copies of those fields in P.
//   packed: bits 0-3 log2(64 wpl), 4-7 log2(lpw), 8 periodic, 9 solve only,
//           10-14 LDS pad, 15 aligned tile layout, 16 log2(io).
template <typename T, int NDIM, int MMAX, int LIMC, bool EXT, bool TW>
__device__ __forceinline__ void sweep_block(const T* U, const T* alpha, const T* beta1, int n, int nt1, int si_t1,
                                            int si_t2, int nb1, int nblk, int packed, int row1,
                                            const SweepParams<T>& Pk) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    SweepParams<T> P = Pk;
    P.U = U;
    P.alpha = alpha;
    P.beta1 = beta1;
    P.n = n;
    P.nt1 = nt1;
    P.si_t1 = si_t1;
    P.si_t2 = si_t2;
    P.spl_log2 = packed & 15;
    P.wpl = 1 << (P.spl_log2 - 6);
    P.lpw_log2 = (packed >> 4) & 15;
    P.lpw = 1 << P.lpw_log2;
    P.periodic = (packed >> 8) & 1;
    P.rhs_mode = TW ? 0 : (packed >> 9) & 1;
    P.lds.pad = (packed >> 10) & 31;
    P.lds.aligned = (packed >> 15) & 1;
    P.io_log2 = TW ? 0 : (packed >> 16) & 1;
    P.lds.row1 = row1;
    // XCD-aware block order: consecutive logical blocks on the same XCD so
    // that halo lines and the partial lines of a transposed store are shared
    // through that XCD's L2.
    int blk = blockIdx.x;
    if ((nblk & 7) == 0) blk = (blk & 7) * (nblk >> 3) + (blk >> 3);
    const int l2 = blk / nb1;
    const int l1_0 = (blk - l2 * nb1) * P.lpw;
    double lsum;
    T lmin, lmax;
    sweep_tile<T, NDIM, MMAX, LIMC, EXT, false, 64, TW>(P, l1_0, l2, smem_raw, lsum, lmin, lmax);
    // FP64 energy / min / max partials (folded by a later launch)
    if (P.red.partials) block_partials<T>(P.red.partials, lsum, lmin, lmax);
}

template <typename T, int NDIM, int MMAX, int LIMC, bool EXT>
__global__ void __launch_bounds__((SweepBounds<T, MMAX>::max_threads))
    sweep_kernel(const T* U, const T* alpha, const T* beta1, int n, int nt1, int si_t1, int si_t2, int nb1,
                 int nblk, int packed, int row1, SweepParams<T> Pk) {
    sweep_block<T, NDIM, MMAX, LIMC, EXT, false>(U, alpha, beta1, n, nt1, si_t1, si_t2, nb1, nblk, packed, row1, Pk);
}

// The 4-step scheme's two solves of a direction in one launch: one pass over
// memory instead of two (256^3 FP32: 427 -> 305 us per step, 293 with 8
// lines per workgroup).
template <typename T, int NDIM, int MMAX, int LIMC, bool EXT>
__global__ void __launch_bounds__((sweep_twice_max_threads((int)sizeof(T), MMAX)))
    sweep_twice_kernel(const T* U, const T* alpha, const T* beta1, int n, int nt1, int si_t1, int si_t2, int nb1,
                       int nblk, int packed, int row1, SweepParams<T> Pk) {
    sweep_block<T, NDIM, MMAX, LIMC, EXT, true>(U, alpha, beta1, n, nt1, si_t1, si_t2, nb1, nblk, packed, row1, Pk);
}

// The cell-slot variant: the same leading arguments (io is always 1).
template <typename T, int NDIM, int MMAX, int LIMC, bool EXT>
__global__ void __launch_bounds__((SweepCellBounds<T, MMAX>::max_threads))
    sweep_cell_kernel(const T* U, const T* alpha, const T* beta1, int n, int nt1, int si_t1, int si_t2, int nb1,
                      int nblk, int packed, int row1, SweepParams<T> Pk) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    SweepParams<T> P = Pk;
    P.U = U;
    P.alpha = alpha;
    P.beta1 = beta1;
    P.n = n;
    P.nt1 = nt1;
    P.si_t1 = si_t1;
    P.si_t2 = si_t2;
    P.spl_log2 = packed & 15;
    P.wpl = 1 << (P.spl_log2 - 6);
    P.lpw_log2 = (packed >> 4) & 15;
    P.lpw = 1 << P.lpw_log2;
    P.periodic = (packed >> 8) & 1;
    P.rhs_mode = (packed >> 9) & 1;
    P.lds.pad = (packed >> 10) & 31;
    P.lds.aligned = (packed >> 15) & 1;
    P.io_log2 = 0;
    P.lds.row1 = row1;
    int blk = blockIdx.x;
    if ((nblk & 7) == 0) blk = (blk & 7) * (nblk >> 3) + (blk >> 3);
    const int l2 = blk / nb1;
    const int l1_0 = (blk - l2 * nb1) * P.lpw;
    double lsum;
    T lmin, lmax;
    cell::sweep_tile<T, NDIM, MMAX, LIMC, EXT>(P, l1_0, l2, smem_raw, lsum, lmin, lmax);
    if (P.red.partials) block_partials<T>(P.red.partials, lsum, lmin, lmax);
}

// Van Leer, minmod and MC get straight-line instantiations of their own; the
// linear mean reads the limiter at run time.  T = 0 walls, a source or a
// second output take the EXT instantiations, van Leer's or the run-time one.
// (A limiter read at run time costs several branches per face: 1403 x 937
// FP32 MC 386 us per 10 steps, 345 straight-line; 129^2 FP64 with walls and a
// source, van Leer, 1492 and 1389 us per 100 steps.)
template <typename T, int NDIM>
hipError_t launch_sweep_dim(const SweepParams<T>& P, int mmax, dim3 grid, dim3 block, size_t lds, hipStream_t st,
                            int variant) {
    // T = 0 walls, a source or a second output take the EXT instantiation
    const bool ext = P.dirichlet || P.Q || P.out2;
    const bool cellv = variant == SWEEP_CELL_SLOTS;
    if (P.lpw != (1 << P.lpw_log2) || P.spl_log2 < 6 || 64 * P.wpl != (1 << P.spl_log2) || P.spl_log2 > 15 || P.lpw_log2 > 15 ||
        P.lds.pad < 0 || P.lds.pad > 31 || P.io_log2 < 0 || P.io_log2 > 1 || (cellv && P.io_log2 != 0) ||
        (variant != SWEEP_FACE_SLOTS && !cellv) || (int)block.x != (P.lpw << (P.spl_log2 + P.io_log2)) ||
        (int)block.x > (cellv ? sweep_cell_max_threads((int)sizeof(T), mmax) : sweep_max_threads((int)sizeof(T), mmax)))
        return hipErrorInvalidValue;
    // the kernel's leading (preloaded) arguments; P.rhs_mode holds 0 or SWEEP_SOLVE_ONLY
    const int nb1 = (P.nt1 + P.lpw - 1) / P.lpw;
    const int packed = P.spl_log2 | (P.lpw_log2 << 4) | ((P.periodic != 0) << 8) | ((P.rhs_mode != 0) << 9) |
                       (P.lds.pad << 10) | ((P.lds.aligned != 0) << 15) | ((P.io_log2 & 1) << 16);
#define ASD_SWEEP_ARGS P.U, P.alpha, P.beta1, P.n, P.nt1, P.si_t1, P.si_t2, nb1, (int)grid.x, packed, P.lds.row1, P
#define ASD_SWEEP_LAUNCH(KERNEL, MM)                                                                          \
    do {                                                                                                      \
        if (ext && P.limiter == LIM_VANLEER)                                                                  \
            hipLaunchKernelGGL((KERNEL<T, NDIM, MM, LIM_VANLEER, true>), grid, block, lds, st, ASD_SWEEP_ARGS); \
        else if (ext)                                                                                         \
            hipLaunchKernelGGL((KERNEL<T, NDIM, MM, -1, true>), grid, block, lds, st, ASD_SWEEP_ARGS);        \
        else if (P.limiter == LIM_VANLEER)                                                                    \
            hipLaunchKernelGGL((KERNEL<T, NDIM, MM, LIM_VANLEER, false>), grid, block, lds, st, ASD_SWEEP_ARGS); \
        else if (P.limiter == LIM_MINMOD)                                                                     \
            hipLaunchKernelGGL((KERNEL<T, NDIM, MM, LIM_MINMOD, false>), grid, block, lds, st, ASD_SWEEP_ARGS); \
        else if (P.limiter == LIM_MC)                                                                         \
            hipLaunchKernelGGL((KERNEL<T, NDIM, MM, LIM_MC, false>), grid, block, lds, st, ASD_SWEEP_ARGS);   \
        else                                                                                                  \
            hipLaunchKernelGGL((KERNEL<T, NDIM, MM, -1, false>), grid, block, lds, st, ASD_SWEEP_ARGS);       \
    } while (0)
#define ASD_SWEEP_CASE(MM)                                      \
    case MM:                                                    \
        if (cellv) ASD_SWEEP_LAUNCH(sweep_cell_kernel, MM);     \
        else ASD_SWEEP_LAUNCH(sweep_kernel, MM);                \
        return hipGetLastError();
    switch (mmax) {
        ASD_SWEEP_CASE(1)
        ASD_SWEEP_CASE(2)
        ASD_SWEEP_CASE(4)
        ASD_SWEEP_CASE(8)
        ASD_SWEEP_CASE(16)
        default: return hipErrorInvalidValue;
    }
#undef ASD_SWEEP_CASE
#undef ASD_SWEEP_LAUNCH
#undef ASD_SWEEP_ARGS
}

// One instantiation for everything but van Leer without walls and source.
template <typename T, int NDIM>
hipError_t launch_sweep_twice(const SweepParams<T>& P, int mmax, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (P.lpw != (1 << P.lpw_log2) || P.lpw_log2 > 15 || P.lds.pad < 0 || P.lds.pad > 31 || P.io_log2 != 0 ||
        P.spl_log2 < 6 || P.spl_log2 > 15 || 64 * P.wpl != (1 << P.spl_log2) || P.rhs_mode != 0 ||
        (int)block.x != (P.lpw << P.spl_log2) || (int)block.x > sweep_twice_max_threads((int)sizeof(T), mmax))
        return hipErrorInvalidValue;
    const bool general = P.dirichlet || P.Q || P.out2 || P.limiter != LIM_VANLEER;
    const int nb1 = (P.nt1 + P.lpw - 1) / P.lpw;
    const int packed = P.spl_log2 | (P.lpw_log2 << 4) | ((P.periodic != 0) << 8) | (P.lds.pad << 10) |
                       ((P.lds.aligned != 0) << 15);
#define ASD_TWICE_ARGS grid, block, lds, st, P.U, P.alpha, P.beta1, P.n, P.nt1, P.si_t1, P.si_t2, nb1, (int)grid.x, packed, P.lds.row1, P
#define ASD_TWICE_CASE(MM)                                                                                     \
    case MM:                                                                                                   \
        if (general) hipLaunchKernelGGL((sweep_twice_kernel<T, NDIM, MM, -1, true>), ASD_TWICE_ARGS);          \
        else hipLaunchKernelGGL((sweep_twice_kernel<T, NDIM, MM, LIM_VANLEER, false>), ASD_TWICE_ARGS);        \
        return hipGetLastError();
    switch (mmax) {
        ASD_TWICE_CASE(1)
        ASD_TWICE_CASE(2)
        ASD_TWICE_CASE(4)
        ASD_TWICE_CASE(8)
        ASD_TWICE_CASE(16)
        default: return hipErrorInvalidValue;
    }
#undef ASD_TWICE_CASE
#undef ASD_TWICE_ARGS
}

// Raise the dynamic-LDS limit of every sweep instantiation to the gfx950
// maximum.  Called once per process, before any launch or stream capture.
template <typename T, int NDIM, int LIMC, bool EXT>
static hipError_t set_attrs_lim(int bytes) {
    const void* fns[] = {(const void*)sweep_kernel<T, NDIM, 1, LIMC, EXT>, (const void*)sweep_kernel<T, NDIM, 2, LIMC, EXT>,
                         (const void*)sweep_kernel<T, NDIM, 4, LIMC, EXT>, (const void*)sweep_kernel<T, NDIM, 8, LIMC, EXT>,
                         (const void*)sweep_kernel<T, NDIM, 16, LIMC, EXT>,
                         (const void*)sweep_cell_kernel<T, NDIM, 1, LIMC, EXT>,
                         (const void*)sweep_cell_kernel<T, NDIM, 2, LIMC, EXT>,
                         (const void*)sweep_cell_kernel<T, NDIM, 4, LIMC, EXT>,
                         (const void*)sweep_cell_kernel<T, NDIM, 8, LIMC, EXT>,
                         (const void*)sweep_cell_kernel<T, NDIM, 16, LIMC, EXT>};
    for (const void* f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <typename T, int NDIM>
hipError_t set_attrs_dim(int bytes) {
    hipError_t e = set_attrs_lim<T, NDIM, LIM_VANLEER, false>(bytes);
    if (e == hipSuccess) e = set_attrs_lim<T, NDIM, LIM_MINMOD, false>(bytes);
    if (e == hipSuccess) e = set_attrs_lim<T, NDIM, LIM_MC, false>(bytes);
    if (e == hipSuccess) e = set_attrs_lim<T, NDIM, -1, false>(bytes);
    if (e == hipSuccess) e = set_attrs_lim<T, NDIM, LIM_VANLEER, true>(bytes);
    if (e == hipSuccess) e = set_attrs_lim<T, NDIM, -1, true>(bytes);
    return e;
}
template <typename T, int NDIM>
hipError_t set_attrs_twice(int bytes) {
    const void* fns[] = {(const void*)sweep_twice_kernel<T, NDIM, 1, LIM_VANLEER, false>,
                         (const void*)sweep_twice_kernel<T, NDIM, 2, LIM_VANLEER, false>,
                         (const void*)sweep_twice_kernel<T, NDIM, 4, LIM_VANLEER, false>,
                         (const void*)sweep_twice_kernel<T, NDIM, 8, LIM_VANLEER, false>,
                         (const void*)sweep_twice_kernel<T, NDIM, 16, LIM_VANLEER, false>,
                         (const void*)sweep_twice_kernel<T, NDIM, 1, -1, true>,
                         (const void*)sweep_twice_kernel<T, NDIM, 2, -1, true>,
                         (const void*)sweep_twice_kernel<T, NDIM, 4, -1, true>,
                         (const void*)sweep_twice_kernel<T, NDIM, 8, -1, true>,
                         (const void*)sweep_twice_kernel<T, NDIM, 16, -1, true>};
    for (const void* f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// One object per (type, dimension, kernel family) compiles its kernels; the
// first also holds the entry points that choose between them.
#define ASD_SWEEP_MAIN(PRE, T, ND)                                                                              \
    PRE template hipError_t launch_sweep_dim<T, ND>(const SweepParams<T>&, int, dim3, dim3, size_t, hipStream_t, \
                                                    int);                                                       \
    PRE template hipError_t set_attrs_dim<T, ND>(int);
#define ASD_SWEEP_TWICE(PRE, T, ND)                                                                             \
    PRE template hipError_t launch_sweep_twice<T, ND>(const SweepParams<T>&, int, dim3, dim3, size_t, hipStream_t); \
    PRE template hipError_t set_attrs_twice<T, ND>(int);
#if ASD_PART == 0
ASD_SWEEP_MAIN(, float, 2)
ASD_SWEEP_MAIN(extern, float, 3)
ASD_SWEEP_MAIN(extern, double, 2)
ASD_SWEEP_MAIN(extern, double, 3)
ASD_SWEEP_TWICE(extern, float, 2)
ASD_SWEEP_TWICE(extern, float, 3)
ASD_SWEEP_TWICE(extern, double, 2)
ASD_SWEEP_TWICE(extern, double, 3)

template <typename T>
static hipError_t set_attrs_type(int bytes) {
    hipError_t e = set_attrs_dim<T, 2>(bytes);
    if (e == hipSuccess) e = set_attrs_dim<T, 3>(bytes);
    if (e == hipSuccess) e = set_attrs_twice<T, 2>(bytes);
    if (e == hipSuccess) e = set_attrs_twice<T, 3>(bytes);
    return e;
}
hipError_t sweep_set_lds_limits(int bytes) {
    hipError_t e = set_attrs_type<float>(bytes);
    return e == hipSuccess ? set_attrs_type<double>(bytes) : e;
}

template <typename T>
hipError_t launch_sweep(const SweepParams<T>& P, int ndim, int mmax, dim3 grid, dim3 block, size_t lds,
                        hipStream_t st, int variant, bool twice) {
    if (twice) {
        if (variant != SWEEP_FACE_SLOTS) return hipErrorInvalidValue;
        if (ndim == 2) return launch_sweep_twice<T, 2>(P, mmax, grid, block, lds, st);
        return launch_sweep_twice<T, 3>(P, mmax, grid, block, lds, st);
    }
    if (ndim == 2) return launch_sweep_dim<T, 2>(P, mmax, grid, block, lds, st, variant);
    return launch_sweep_dim<T, 3>(P, mmax, grid, block, lds, st, variant);
}

template hipError_t launch_sweep<float>(const SweepParams<float>&, int, int, dim3, dim3, size_t, hipStream_t, int, bool);
template hipError_t launch_sweep<double>(const SweepParams<double>&, int, int, dim3, dim3, size_t, hipStream_t, int,
                                         bool);
#elif ASD_PART == 1
ASD_SWEEP_MAIN(, float, 3)
#elif ASD_PART == 2
ASD_SWEEP_MAIN(, double, 2)
#elif ASD_PART == 3
ASD_SWEEP_MAIN(, double, 3)
#elif ASD_PART == 4
ASD_SWEEP_TWICE(, float, 2)
#elif ASD_PART == 5
ASD_SWEEP_TWICE(, float, 3)
#elif ASD_PART == 6
ASD_SWEEP_TWICE(, double, 2)
#else
ASD_SWEEP_TWICE(, double, 3)
#endif

}  // namespace asd
