// Explicit limited step (the time-step-limited baseline of sections 1 and
// 3): forward Euler of the same conservative operator, every face from T^n:
//
//   T^{n+1}_c = T^n_c + sum_d [ alpha_{c+1/2}(T_{c+e} - T_c) - alpha_{c-1/2}(T_c - T_{c-e})
//                               + F_{c+1/2} - F_{c-1/2} ]
//
// with alpha_f and F_f defined exactly as in the semi-implicit sweep (plus
// dt Q with a source).  T = 0 walls stage odd ghosts (-U, with the cell's b
// and chi) in the halo, so a wall face takes the normal flux
// alpha_w (-U_c - U_c) and a transverse flux that vanishes (the limited
// difference of a cell and its odd ghost is zero).
//
// gfx950 mapping: each wave owns a small block of cells, one column per
// lane (2-D: a band of rows; 3-D: rows of consecutive planes), loads it with a one-cell
// halo, and evaluates every face once (lane shifts across columns,
// registers across rows and planes).  No LDS staging.
#include <algorithm>

#include "asd_device.h"
#include "asd_launch.h"

namespace asd {

// What a kernel instantiation reads (MODE): a constant chi, a per-cell chi or
// chi(T), and with EX_EXTRA also T = 0 walls and a source, told apart at run
// time.  Every limiter has its own instantiations too: tests of the mode or the
// limiter inside a wave's block keep its loads and faces waiting for one
// another (256^3 FP32, us per step: minmod 271-312 with both read at run time,
// 110 straight-line; van Leer with walls 159 and 112).
enum : int { EX_CHI_CONST = 0, EX_CHI_CELL = 1, EX_CHI_OF_T = 2, EX_EXTRA = 4 };
template <int MODE>
struct ExMode {
    static constexpr int chi = MODE & 3;
    static constexpr bool extra = (MODE & EX_EXTRA) != 0;
};

// Neighbour coordinate with the boundary rule, in 32 bits (periodic wraps,
// walls clamp; the odd ghost's sign is applied by the caller).
__device__ __forceinline__ int nb_coord32(int c, int n, bool periodic) {
    if (c < 0) return periodic ? n - 1 : 0;
    if (c >= n) return periodic ? 0 : n - 1;
    return c;
}

// 2-D: one wave streams down a band of ExStream::TY rows of 64 columns
// (lane = column).  Lanes 0 and 63 hold the halo columns, so a wave updates
// the 62 columns between them; the row above and the row below the band
// are halo rows.  All loads of the band are issued first, in row order, so
// the first rows are updated while the later ones are still arriving.
// Every face is evaluated once: a cell's left x face is its left lane's
// right x face (a lane shift), its lower y face the upper y face of the
// previous row (kept in a register).  No LDS and no barrier (except the
// block's final reduction).
struct ExStream {
    static constexpr int COLS = 62;  // updated columns per wave
    static constexpr int TY = 4;     // rows per wave
    static constexpr int WAVES = 4;  // waves per block
};

// from_right: the value of lane+1 (the column to the right); from_left: that
// of lane-1.  The edge lanes receive values they never use.
template <typename T>
__device__ __forceinline__ T from_right(T v) { return __shfl_down(v, 1, 64); }
template <typename T>
__device__ __forceinline__ T from_left(T v) { return __shfl_up(v, 1, 64); }

template <typename T, int LIM, int MODE>
__global__ void __launch_bounds__(256) explicit_stream2d_kernel(ExplicitParams<T> P) {
    constexpr int TY = ExStream::TY, NR = TY + 2;  // rows y0-1 .. y0+TY
    const int nx = P.n[0], ny = P.n[1];
    const int lane = threadIdx.x & 63;
    // XCD-aware block order (the grid is a multiple of 8 blocks): bands that
    // share halo rows run on one XCD and share its L2
    const int blk = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int wave = blk * ExStream::WAVES + (threadIdx.x >> 6);
    const int ncb = (nx + ExStream::COLS - 1) / ExStream::COLS;
    const int nrb = (ny + TY - 1) / TY;
    double lsum = 0.0;
    T lmin = T(__builtin_huge_val()), lmax = T(-__builtin_huge_val());
    if (wave < ncb * nrb) {  // wave-uniform
        const int cb = wave % ncb, rb = wave / ncb;
        const int x = cb * ExStream::COLS - 1 + lane;  // this lane's column (halo lanes may lie outside)
        const int y0 = rb * TY;
        const bool periodic = P.periodic != 0;
        const bool dir = ExMode<MODE>::extra && P.dirichlet != 0;
        const bool has_q = ExMode<MODE>::extra && P.Q != nullptr;
        constexpr int lim = LIM;
        constexpr bool pchi = ExMode<MODE>::chi != EX_CHI_CONST;
        const int xc = nb_coord32(x, nx, periodic);
        const bool xout = xc != x;
        // the band's rows: state (odd ghosts negated), b and chi
        T u[NR], bx[NR], by[NR], ch[NR], q[TY];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int y = y0 - 1 + r;
            const int yc = nb_coord32(y, ny, periodic);
            const unsigned c = (unsigned)xc + (unsigned)yc * (unsigned)nx;
            const T v = P.U[c];
            // odd ghost: one sign flip per axis on which the cell lies outside
            u[r] = dir && (xout != (yc != y)) ? -v : v;
            bx[r] = P.b[0][c];
            by[r] = P.b[1][c];
            ch[r] = ExMode<MODE>::chi == EX_CHI_CELL ? P.chi[c] : P.chi_par;
            // chi(T): the cell's value from T^n, in FP64 (section 3.3)
            if (ExMode<MODE>::chi == EX_CHI_OF_T) ch[r] = (T)((double)P.chi_par * pow((double)v / P.chi_tref, P.chi_exp));
            if (r >= 1 && r <= TY && has_q) q[r - 1] = P.Q[c];
        }
        const T cn0 = P.cn[0], cn1 = P.cn[1], ct01 = P.ct[0][1], ct10 = P.ct[1][0];
        const T chi_par = P.chi_par, chi_perp = P.chi_perp;
        auto face = [&](T u0, T u1, T bn0, T bn1, T bt0, T bt1, T c0, T c1, T s0, T s1, T cn, T ct) {
            // face between cells 0 and 1 along the normal axis: bn = normal
            // component of b, bt = transverse component, s = transverse slopes
            const T bnf = T(0.5) * (bn0 + bn1);
            const T chif = pchi ? harmonic<T>(c0, c1) : chi_par;
            const T dpar = chif - chi_perp;
            const T alpha = cn * (chi_perp + dpar * bnf * bnf);
            const T btf = T(0.5) * (bt0 + bt1);
            // (written as fma: every instantiation rounds alike)
            return fma(dpar * bnf, ct * btf * limit2<T>(lim, s1, s0), alpha * (u1 - u0));
        };
        // slopes along x of a row (lane shifts), along y of a row (registers)
        auto slope_x = [&](T uc) { return cell_slope<T>(lim, from_left(uc), uc, from_right(uc)); };
        const bool xwall = !periodic && !dir && (x < 0 || x + 1 > nx - 1);  // this lane's right x face
        const bool out_col = lane >= 1 && lane <= ExStream::COLS && x < nx;
        // upper y face of row y0-1 (the lower face of the first row)
        T sx_prev = slope_x(u[0]);
        T sx_cur = slope_x(u[1]);
        T fy_low;
        {
            const bool ywall = !periodic && !dir && (y0 - 1 < 0 || y0 > ny - 1);
            fy_low = ywall ? T(0) : face(u[0], u[1], by[0], by[1], bx[0], bx[1], ch[0], ch[1], sx_prev, sx_cur, cn1, ct10);
        }
#pragma unroll
        for (int r = 1; r <= TY; ++r) {
            const int y = y0 - 1 + r;
            // x faces of row r: this lane's right face, and its left face from the left lane
            const T sy = cell_slope<T>(lim, u[r - 1], u[r], u[r + 1]);
            T fxr = face(u[r], from_right(u[r]), bx[r], from_right(bx[r]), by[r], from_right(by[r]), ch[r],
                         from_right(ch[r]), sy, from_right(sy), cn0, ct01);
            fxr = xwall ? T(0) : fxr;
            const T fxl = from_left(fxr);
            // upper y face of row r
            const T sx_next = slope_x(u[r + 1]);
            const bool ywall = !periodic && !dir && (y < 0 || y + 1 > ny - 1);
            T fyh = face(u[r], u[r + 1], by[r], by[r + 1], bx[r], bx[r + 1], ch[r], ch[r + 1], sx_cur, sx_next,
                         cn1, ct10);
            fyh = ywall ? T(0) : fyh;
            T acc = T(0);
            acc += -fxl;
            acc += fxr;
            acc += -fy_low;
            acc += fyh;
            if (out_col && y < ny) {
                const T uc = u[r];
                const T un = has_q ? (uc + P.dtq * q[r - 1]) + acc : uc + acc;
                P.out[(unsigned)x + (unsigned)y * (unsigned)nx] = un;
                lsum += (double)un;
                lmin = un < lmin ? un : lmin;
                lmax = un > lmax ? un : lmax;
            }
            fy_low = fyh;
            sx_cur = sx_next;
        }
    }
    if (P.red.partials) block_partials<T>(P.red.partials, lsum, lmin, lmax);
}

// 3-D: the same scheme as the 2-D streaming kernel, marching along z.  A wave
// owns 62 columns x TY rows of P.planes consecutive planes (lane = column)
// and keeps the state, b and slopes of the current plane in registers; each
// step loads the next plane (TY + 2 rows), evaluates every face of the current
// plane once (x faces by a lane shift, y faces between rows, z faces between
// planes, the lower ones kept from the step before) and updates its cells.
// No LDS and no barrier apart from the final reduction.
//
// What bounds it: vector instructions (about 31 per face and 9 per slope) and
// the L2 requests of the halo rows.  Marching loads each plane once per wave,
// (TY + 2) / TY values per cell and field, where a 2 x 2 block of rows and
// planes loads 4, and evaluates 3.25 faces and 4 slopes per cell instead of
// 4 and 8 (TY = 4).  256^3, us per step without energies: FP32 110, 2 x 2
// blocks with every option read at run time 140; FP64 245 and 330.
struct ExStream3 {
    static constexpr int COLS = 62;
    static constexpr int WAVES = 4;
};
// Rows per wave (TY): 4 in FP32 on grids of 2^21 cells and more (us per step
// with 4 and 2 rows: 256^3 107-113 and 111, 200^3 51 and 62, 140^3 23.6 and
// 24.5), 2 on smaller ones (100^3 12.1 and 10.9, 256 x 30 x 256 17.9 and 17.2)
// and in FP64, for the registers.
template <typename T>
static int explicit_rows(const int n[3]) {
    return sizeof(T) == 4 && (int64_t)n[0] * n[1] * n[2] >= (1 << 21) ? 4 : 2;
}
// Planes per wave: long marches load fewer halo planes, short ones leave
// more waves; the longest of 2 ... 32 that leaves 12 waves per CU.  With chi(T)
// the power of every loaded cell is most of the work, and the time is that of
// the SIMD with the most waves: the march with the least of waves per SIMD times
// loaded planes (one wave alone counts for 1.4, it hides little of its latency).
// us per step, chi(T): 80^3 FP64 43.7 with 2 planes, 39.7 with 4, 45.6 with 8;
// 100^3 FP64 59.7, 58.8, 68.6, 54.9 with 6; 200^3 FP32 182 with 8, 210 with 16.
template <typename T>
static int explicit_planes(const int n[3], bool of_T) {
    using S = ExStream3;
    const int ty = explicit_rows<T>(n);
    const int64_t cols = (int64_t)((n[0] + S::COLS - 1) / S::COLS) * ((n[1] + ty - 1) / ty);
    auto waves = [&](int p) { return cols * ((n[2] + p - 1) / p); };
    int p = 32;
    if (of_T) {
        auto cost = [&](int q) {
            const int64_t k = (waves(q) + 1023) / 1024;
            return (double)(q + 2) * (k == 1 ? 1.4 : (double)k);
        };
        for (int q = 31; q >= 1; --q)
            if (cost(q) < cost(p)) p = q;
    } else {
        while (p > 2 && waves(p) < 12 * 256) p /= 2;
    }
    return p;
}

// One plane of a wave's rows and their halo rows.
template <typename T, int NR>
struct ExPlane {
    T u[NR], bx[NR], by[NR], bz[NR], ch[NR];
    T sx[NR], sy[NR];  // limited slopes along x, and along y (inner rows)
};

template <typename T, int LIM, int MODE, int TY>
__global__ void __launch_bounds__(256) explicit_stream3d_kernel(ExplicitParams<T> P) {
    using S = ExStream3;
    constexpr int NR = TY + 2;
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int lane = threadIdx.x & 63;
    const int blk = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);  // XCD-aware order
    // wave-uniform (readfirstlane): the row and plane arithmetic stays scalar
    const int wave = blk * S::WAVES + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ncb = (nx + S::COLS - 1) / S::COLS, nrb = (ny + TY - 1) / TY, nzb = (nz + P.planes - 1) / P.planes;
    double lsum = 0.0;
    T lmin = T(__builtin_huge_val()), lmax = T(-__builtin_huge_val());
    if (wave < ncb * nrb * nzb) {  // wave-uniform
        const int cb = wave % ncb, rb = (wave / ncb) % nrb, zb = wave / (ncb * nrb);
        const int x = cb * S::COLS - 1 + lane;
        const int y0 = rb * TY, z0 = zb * P.planes;
        const int z1 = min(z0 + P.planes, nz);
        const bool periodic = P.periodic != 0;
        const bool dir = ExMode<MODE>::extra && P.dirichlet != 0;
        const bool has_q = ExMode<MODE>::extra && P.Q != nullptr;
        constexpr int lim = LIM;
        constexpr bool pchi = ExMode<MODE>::chi != EX_CHI_CONST;
        const int xc = nb_coord32(x, nx, periodic);
        const bool xout = xc != x;
        const unsigned sy = (unsigned)nx, sz = (unsigned)nx * (unsigned)ny;
        using Plane = ExPlane<T, NR>;
        // plane z of the wave's rows y0-1 .. y0+TY, all loads before any use
        auto load = [&](int z, Plane& p) {
            const int zc = nb_coord32(z, nz, periodic);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int y = y0 - 1 + r;
                // (rows past ny, in the last block, are clamped to a valid one and not stored)
                const int yc = nb_coord32(y, ny, periodic);
                const unsigned c = (unsigned)xc + (unsigned)yc * sy + (unsigned)zc * sz;
                const T v = P.U[c];
                // odd ghost: one sign flip per axis on which the cell lies outside
                const int nout = (int)xout + (int)(yc != y) + (int)(zc != z);
                p.u[r] = dir && (nout & 1) ? -v : v;
                p.bx[r] = P.b[0][c];
                p.by[r] = P.b[1][c];
                p.bz[r] = P.b[2][c];
                // (chi(T): T^n, until chi_of_T)
                p.ch[r] = ExMode<MODE>::chi == EX_CHI_CELL ? P.chi[c] : ExMode<MODE>::chi == EX_CHI_OF_T ? v : P.chi_par;
            }
        };
        // chi(T): the cells' values from T^n, in FP64 (section 3.3)
        auto chi_of_T = [&](Plane& p) {
            if constexpr (ExMode<MODE>::chi == EX_CHI_OF_T) {
#pragma unroll
                for (int r = 0; r < NR; ++r) p.ch[r] = (T)((double)P.chi_par * pow((double)p.ch[r] / P.chi_tref, P.chi_exp));
            }
        };
        auto slopes = [&](Plane& p) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                p.sx[r] = cell_slope<T>(lim, from_left(p.u[r]), p.u[r], from_right(p.u[r]));
                p.sy[r] = (r >= 1 && r <= TY) ? cell_slope<T>(lim, p.u[r - 1], p.u[r], p.u[r + 1]) : T(0);
            }
        };
        const T chi_par = P.chi_par, chi_perp = P.chi_perp;
        // face between cells 0 and 1 along the normal axis n; a and b are the
        // two transverse axes in increasing order (components ta, tb of b,
        // limited slopes sa, sb)
        auto face = [&](T u0, T u1, T bn0, T bn1, T ta0, T ta1, T tb0, T tb1, T c0, T c1, T sa0, T sa1, T sb0,
                        T sb1, T cn, T cta, T ctb) {
            const T bnf = T(0.5) * (bn0 + bn1);
            const T chif = pchi ? harmonic<T>(c0, c1) : chi_par;
            const T dpar = chif - chi_perp;
            const T alpha = cn * (chi_perp + dpar * bnf * bnf);
            T tr = T(0);
            tr += cta * (T(0.5) * (ta0 + ta1)) * limit2<T>(lim, sa1, sa0);
            tr += ctb * (T(0.5) * (tb0 + tb1)) * limit2<T>(lim, sb1, sb0);
            // (written as fma: every instantiation rounds alike)
            return fma(dpar * bnf, tr, alpha * (u1 - u0));
        };
        const bool xwall = !periodic && !dir && (x < 0 || x + 1 > nx - 1);
        const bool out_col = lane >= 1 && lane <= S::COLS && x < nx;
        auto zfaces = [&](int z, const Plane& a, const Plane& b, T (&f)[TY]) {  // between planes z and z + 1
            const bool zwall = !periodic && !dir && (z < 0 || z + 1 > nz - 1);
#pragma unroll
            for (int r = 1; r <= TY; ++r) {
                const T v = face(a.u[r], b.u[r], a.bz[r], b.bz[r], a.bx[r], b.bx[r], a.by[r], b.by[r], a.ch[r], b.ch[r],
                                 a.sx[r], b.sx[r], a.sy[r], b.sy[r], P.cn[2], P.ct[2][0], P.ct[2][1]);
                f[r - 1] = zwall ? T(0) : v;
            }
        };
        T up[NR];     // the state of the plane below
        Plane C;      // the current plane
        T fz_lo[TY];  // its lower z faces
        {
            Plane B;
            load(z0 - 1, B);
            load(z0, C);
            slopes(B);
            slopes(C);
            chi_of_T(B);
            chi_of_T(C);
            zfaces(z0 - 1, B, C, fz_lo);
#pragma unroll
            for (int r = 0; r < NR; ++r) up[r] = B.u[r];
        }
#pragma unroll 1
        for (int z = z0; z < z1; ++z) {
            Plane N;
            load(z + 1, N);
            T q[TY];
            if (has_q) {
#pragma unroll
                for (int r = 1; r <= TY; ++r)
                    q[r - 1] = P.Q[(unsigned)xc + (unsigned)min(y0 - 1 + r, ny - 1) * sy + (unsigned)z * sz];
            }
            slopes(N);
            T szs[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) szs[r] = cell_slope<T>(lim, up[r], C.u[r], N.u[r]);
            // y faces of this plane, rows r and r+1, r = 0 .. TY
            T fy[TY + 1];
#pragma unroll
            for (int r = 0; r <= TY; ++r) {
                const int y = y0 - 1 + r;
                const bool ywall = !periodic && !dir && (y < 0 || y + 1 > ny - 1);
                const T f = face(C.u[r], C.u[r + 1], C.by[r], C.by[r + 1], C.bx[r], C.bx[r + 1], C.bz[r], C.bz[r + 1],
                                 C.ch[r], C.ch[r + 1], C.sx[r], C.sx[r + 1], szs[r], szs[r + 1], P.cn[1], P.ct[1][0],
                                 P.ct[1][2]);
                fy[r] = ywall ? T(0) : f;
            }
            chi_of_T(N);
            T fz_hi[TY];
            zfaces(z, C, N, fz_hi);
#pragma unroll
            for (int r = 1; r <= TY; ++r) {
                const int y = y0 - 1 + r;
                T fxr = face(C.u[r], from_right(C.u[r]), C.bx[r], from_right(C.bx[r]), C.by[r], from_right(C.by[r]),
                             C.bz[r], from_right(C.bz[r]), C.ch[r], pchi ? from_right(C.ch[r]) : C.ch[r], C.sy[r],
                             from_right(C.sy[r]), szs[r], from_right(szs[r]), P.cn[0], P.ct[0][1], P.ct[0][2]);
                fxr = xwall ? T(0) : fxr;
                const T fxl = from_left(fxr);
                T acc = T(0);
                acc += -fxl;
                acc += fxr;
                acc += -fy[r - 1];
                acc += fy[r];
                acc += -fz_lo[r - 1];
                acc += fz_hi[r - 1];
                if (out_col && y < ny) {
                    const T uc = C.u[r];
                    const T un = has_q ? (uc + P.dtq * q[r - 1]) + acc : uc + acc;
                    P.out[(unsigned)x + (unsigned)y * sy + (unsigned)z * sz] = un;
                    lsum += (double)un;
                    lmin = un < lmin ? un : lmin;
                    lmax = un > lmax ? un : lmax;
                }
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) up[r] = C.u[r];
#pragma unroll
            for (int r = 0; r < TY; ++r) fz_lo[r] = fz_hi[r];
            C = N;
        }
    }
    if (P.red.partials) block_partials<T>(P.red.partials, lsum, lmin, lmax);
}

// Blocks of an explicit launch: a multiple of 8 for the XCD-aware order.
template <typename T>
static int explicit_blocks_t(int ndim, const int n[3], bool of_T) {
    int waves, per_block;
    if (ndim == 2) {
        waves = ((n[0] + ExStream::COLS - 1) / ExStream::COLS) * ((n[1] + ExStream::TY - 1) / ExStream::TY);
        per_block = ExStream::WAVES;
    } else {
        using S = ExStream3;
        const int pl = explicit_planes<T>(n, of_T), ty = explicit_rows<T>(n);
        waves = ((n[0] + S::COLS - 1) / S::COLS) * ((n[1] + ty - 1) / ty) * ((n[2] + pl - 1) / pl);
        per_block = S::WAVES;
    }
    const int blocks = (waves + per_block - 1) / per_block;
    return (blocks + 7) & ~7;
}

// The larger of the two precisions' block counts (sizes the reduction
// scratch), with and without chi(T).
int explicit_num_blocks(int ndim, const int n[3]) {
    int most = 0;
    for (bool of_T : {false, true}) {
        most = std::max(most, explicit_blocks_t<float>(ndim, n, of_T));
        most = std::max(most, explicit_blocks_t<double>(ndim, n, of_T));
    }
    return most;
}

template <typename T, int LIM, int MODE>
static void launch_instance(const ExplicitParams<T>& P, int ndim, int nb, hipStream_t st) {
    constexpr int MOST = sizeof(T) == 4 ? 4 : 2;  // rows of the 3-D instantiations: 2, and 4 in FP32
    if (ndim == 2)
        hipLaunchKernelGGL((explicit_stream2d_kernel<T, LIM, MODE>), dim3(nb), dim3(64 * ExStream::WAVES), 0, st, P);
    else if (explicit_rows<T>(P.n) == MOST)
        hipLaunchKernelGGL((explicit_stream3d_kernel<T, LIM, MODE, MOST>), dim3(nb), dim3(64 * ExStream3::WAVES), 0, st, P);
    else
        hipLaunchKernelGGL((explicit_stream3d_kernel<T, LIM, MODE, 2>), dim3(nb), dim3(64 * ExStream3::WAVES), 0, st, P);
}
template <typename T, int LIM, int CHI>
static void launch_mode(const ExplicitParams<T>& P, int ndim, int nb, hipStream_t st) {
    if (P.dirichlet || P.Q) launch_instance<T, LIM, CHI | EX_EXTRA>(P, ndim, nb, st);
    else launch_instance<T, LIM, CHI>(P, ndim, nb, st);
}
template <typename T, int LIM>
static void launch_limiter(const ExplicitParams<T>& P, int ndim, int nb, hipStream_t st) {
    if (P.chi_exp != 0.0) launch_mode<T, LIM, EX_CHI_OF_T>(P, ndim, nb, st);
    else if (P.chi) launch_mode<T, LIM, EX_CHI_CELL>(P, ndim, nb, st);
    else launch_mode<T, LIM, EX_CHI_CONST>(P, ndim, nb, st);
}

template <typename T>
hipError_t launch_explicit(const ExplicitParams<T>& Pin, int ndim, hipStream_t st, int* nblocks_out) {
    ExplicitParams<T> P = Pin;
    const bool of_T = P.chi_exp != 0.0;
    P.planes = ndim == 3 ? explicit_planes<T>(P.n, of_T) : 1;
    const int nb = explicit_blocks_t<T>(ndim, P.n, of_T);
    if (nblocks_out) *nblocks_out = nb;
    switch (P.limiter) {
        case LIM_VANLEER: launch_limiter<T, LIM_VANLEER>(P, ndim, nb, st); break;
        case LIM_MINMOD: launch_limiter<T, LIM_MINMOD>(P, ndim, nb, st); break;
        case LIM_MC: launch_limiter<T, LIM_MC>(P, ndim, nb, st); break;
        case LIM_LINEAR: launch_limiter<T, LIM_LINEAR>(P, ndim, nb, st); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template hipError_t launch_explicit<float>(const ExplicitParams<float>&, int, hipStream_t, int*);
template hipError_t launch_explicit<double>(const ExplicitParams<double>&, int, hipStream_t, int*);

}  // namespace asd
