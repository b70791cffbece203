// Geometric multigrid for (L_h - k2) u = f with u = 0 on the boundary, the
// solver behind Solve_Wakefield (WAND-PIC, Sec. II item 4 and Sec. VII.A).
// L_h is the 5-point Laplacian of Sec. VII.B eq. (33); psi, Ez and Bz use
// k2 = 0 (eqs. (12)-(14)), B_perp uses k2 = n* / (1+psi) (eq. (18)).
//
// One V(nu1, nu2) cycle over levels N, N/2, ..., 2:
//   * levels with N > 64 run two fused tile kernels per level:
//       down: load a tile plus halo into LDS, nu1 red-black Gauss-Seidel sweeps,
//             write the smoothed tile, residual, full-weighting restriction;
//       up:   load a tile plus halo, add the bilinear prolongation of the coarse
//             correction, nu2 sweeps, write the tile;
//     the halo (2 nu + 2 nodes) makes the tile result identical to a global
//     red-black sweep, so every node array is read and written once per pass;
//   * the levels N <= 64 of a Helmholtz cycle, and whole grids that small, run in
//     registers inside one workgroup per right-hand side, down to the 2x2-cell grid,
//     which is solved exactly;
//   * a Poisson cycle ends on the level below the finest (64^2 .. 2048^2) with an exact
//     sine-transform solve; to a tolerance, grids up to 2048^2 take that solve on the
//     finest level itself and no V-cycles at all (direct_poisson).
// Two right-hand sides with one operator (Ez, Bz and Bx, By) share each pass.
// All reductions (residual norms) have a fixed order: results are bitwise
// reproducible.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <type_traits>

#include "wq_common.h"

namespace wq {
namespace {

// Kernel names for the per-kernel timing; formatted only when it is on.
template <class... A>
void prof_name(const wandqs_ctx* c, char* nm, size_t n, const char* fmt, A... a) {
    if (c->prof.on) std::snprintf(nm, n, fmt, a...);
    else nm[0] = 0;
}

#ifndef WQ_SMALL_TILE_MAX
#define WQ_SMALL_TILE_MAX 256
#endif
constexpr int kThreads = 256;  // norm and reduction kernels
// Helmholtz levels with h^2 n0 > kOmegaH2N0 smooth with plain Gauss-Seidel:
// where the diagonal shift h^2 k2 (k2 ~ n0 in the plasma) is no longer small,
// over-relaxation slows the cycle (measured).
constexpr double kOmegaH2N0 = 0.125;
// Pre-smoothing on the levels kFullPreLevels and more below the finest (the
// coarse kernel's levels included when it lies that deep) is one sweep: a
// second sweep there cost more time than the extra V-cycles it saved
// (measured).  The finer levels and every post-smoothing keep nu_pre, nu_post.
constexpr int kFullPreLevels = 2;
// In the tolerance mode the Helmholtz V-cycles visit the levels of at most 64^2
// with two cycles of a sweep fewer each way (at least one), two V(1, 1) instead of
// one V(1, 2) by default; nu_post = 1 keeps its one cycle.  A further cycle there
// costs about 4 us inside the launch and takes B_perp from 8.8 to 6.1 V-cycles per
// solve at 256^2, from 7.6 to 6.2 at 512^2 and from 6.2 to 5.4 at 1024^2 (slices of
// 477 -> 402, 763 -> 722 and 1065 -> 1032 us; V(1, 2) twice 415, 740, 1043; three
// V(1, 1) with two pre-sweeps on every tile level 432, 723, 1056).  Fixed mode
// keeps the single cycle its callers count.
constexpr int kCoarseCycles = 2;
// Tile kernels: 32 x 32 owned nodes with 512 threads, or 16 x 16 with 256
// threads on the levels N <= WQ_SMALL_TILE_MAX (more workgroups and a shorter
// chain of dependent LDS phases per workgroup where the grid is small).
// 64 x 64 with 1024 threads on the levels N >= WQ_BIG_TILE_MIN (the finest
// level of the large grids: a quarter of the halo re-reads of 32 x 32 tiles).
#ifndef WQ_BIG_TILE_MIN
#define WQ_BIG_TILE_MIN 1024
#endif
template <int T>
constexpr int tile_threads() { return T >= 64 ? 1024 : (T >= 32 ? 512 : 256); }
int tile_for(const wandqs_ctx* c, int N) {
    return N <= c->small_tile_max ? 16 : (N >= (WQ_BIG_TILE_MIN) ? 64 : 32);
}

// Deterministic block sum of NV values; the result is valid in thread 0.
template <int NV, int NT>
__device__ void block_sum(double (&v)[NV], double* red) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] += __shfl_xor(v[k], off, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k) red[wave * NV + k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double s = 0.0;
            for (int w = 0; w < NT / 64; ++w) s += red[w * NV + k];
            v[k] = s;
        }
    }
}

// ------------------------------------------------------------ tile engine --
//
// A tile kernel holds an EX x EY block of nodes whose node (0, 0) is global
// node (ex0, ey0), ex0 even.  The iterate u lives in LDS; each thread owns
// KP horizontal node pairs (x = 2p, 2p+1 of a row) and keeps their f and the
// Gauss-Seidel diagonal D = 4 + h^2 k2 (and 1/D) in registers.  In a pair the
// two nodes have opposite colours, so every thread updates exactly one node of
// each of its pairs in every half sweep.
// Fused multiply-add, written out so that every tile kernel rounds the same
// way whatever the compiler shares between sweeps.
__device__ __forceinline__ double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Value select (not an address select, so register arrays stay in registers).
template <typename T>
__device__ __forceinline__ T pick(int j, T a, T b) { return j ? b : a; }

template <int R, bool HELM, int EX, int EY, int NT>
struct TileShape {
    static constexpr int PW = EX / 2;
    static constexpr int NP = PW * EY;
    static constexpr int KP = (NP + NT - 1) / NT;
    static constexpr int EN = EX * EY;
    static_assert(EX % 2 == 0, "tile width must be even");
};

// E is the element type of the iterate, f and the sweep arithmetic (double, or
// float for the inner cycles of the mixed form); k2 is always read as double
// and D = 4 + h^2 k2, 1/D are formed in double before rounding to E.
template <typename E, int R, bool HELM, int EX, int EY, int KP, int NT>
__device__ __forceinline__ void tile_load(E (*su)[EX * EY], E (&fr)[R][KP][2], E (&Dr)[KP][2],
                                          E (&iDr)[KP][2], const E* const* u, const E* const* f,
                                          const double* k2, int pitch, int ex0, int ey0, int N,
                                          double h2) {
    constexpr int PW = EX / 2, NP = PW * EY;
    // Every load and LDS store is unconditional, so that the loads are all in
    // flight at once (the compiler waits for a load moved behind a
    // lane-dependent branch before the branch ends): the threads past the
    // tile redo the last pair (the same values to the same slots), the
    // indices are clamped into the grid and the values outside it masked by a
    // product with 0 (every value loaded is finite).
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int p = min((int)threadIdx.x + k * NT, NP - 1);
        const int ly = p / PW, px = p - ly * PW;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lx = 2 * px + j;
            const int gx = ex0 + lx, gy = ey0 + ly;
            const bool in = gx >= 0 && gx <= N && gy >= 0 && gy <= N;
            const size_t g = (size_t)min(max(gy, 0), N) * pitch + min(max(gx, 0), N);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const E* ur = u[r] ? u[r] : f[r];
                const E uv = ur[g] * E(in && u[r] ? 1 : 0);
                su[r][ly * EX + lx] = uv;
                fr[r][k][j] = f[r][g] * E(in ? 1 : 0);
            }
            const double D = fmad(h2, HELM ? k2[g] * (in ? 1.0 : 0.0) : 0.0, 4.0);
            Dr[k][j] = (E)D;
            iDr[k][j] = HELM ? (E)(1.0 / D) : E(0.25);
        }
    }
}

// Over-relaxed red-black update of one node: with g = (sum of the 4
// neighbours - h^2 f) / D, the node's own equation solved for it,
// u <- u + om (g - u).  Every smoothing kernel forms it with these three
// fused operations, so they all give the same bits.
template <typename E>
__device__ __forceinline__ E sor_update(E u, E nb, E fv, E iD, E h2, E om) {
    return fmad(om, fmad(fmad(-h2, fv, nb), iD, -u), u);
}

// One red-black half sweep (sor_update) on the nodes of colour `color`
// ((gx + gy) % 2) that have all four neighbours in the tile and lie inside the
// domain.
template <typename E, int R, bool HELM, int EX, int EY, int KP, int NT>
__device__ __forceinline__ void tile_sweep(E (*su)[EX * EY], const E (&fr)[R][KP][2],
                                           const E (&iDr)[KP][2], int ex0, int ey0, int N, E h2,
                                           E om, int color) {
    constexpr int PW = EX / 2, NP = PW * EY;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int p = threadIdx.x + k * NT;
        const int ly = p / PW, px = p - ly * PW;
        const int gy = ey0 + ly;
        const int j = (gy + color) & 1;  // ex0 is even
        const int lx = 2 * px + j;
        const int gx = ex0 + lx;
        if (p < NP && lx >= 1 && lx <= EX - 2 && ly >= 1 && ly <= EY - 2 && gx >= 1 &&
            gx <= N - 1 && gy >= 1 && gy <= N - 1) {
            const int l = ly * EX + lx;
            const E id = pick(j, iDr[k][0], iDr[k][1]);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const E fv = pick(j, fr[r][k][0], fr[r][k][1]);
                const E nb = su[r][l - 1] + su[r][l + 1] + su[r][l - EX] + su[r][l + EX];
                su[r][l] = sor_update(su[r][l], nb, fv, id, h2, om);
            }
        }
    }
}

template <typename E>
struct DownArgs {
    int N;
    double h;
    int pitch, pitch_c;
    const E* u_in[2];  // nullptr: zero initial guess
    const E* f[2];
    const double* k2;
    E* u_out[2];
    E* f_c[2];
    double* norm_part;  // (double only) nullptr or [3R][nblk]: sums r^2, f^2, u^2 of the incoming u
    int nblk;
    double omega;  // relaxation factor of the smoothing sweeps
};

// Down pass of one level: nu1 sweeps on the tile, write the smoothed tile,
// residual, full-weighting restriction onto the coarse tile.  Halo: 2 nu + 2
// nodes on the low side (the residual at x0 - 1 needs the smoothed u at x0 - 2),
// 2 nu + 2 on the high side (one more than needed, to keep the width even).
template <typename E, int R, bool HELM, int NU, int T>
__global__ __launch_bounds__(tile_threads<T>()) void k_mg_down(DownArgs<E> a) {
    constexpr int NT = tile_threads<T>();
    constexpr int HL = 2 * NU + 2, HH = 2 * NU + 2;
    constexpr int EX = T + HL + HH, EY = EX;
    using S = TileShape<R, HELM, EX, EY, NT>;
    constexpr int PW = S::PW, NP = S::NP, KP = S::KP, EN = S::EN;
    __shared__ E su[R][EN];
    __shared__ double red[(NT / 64) * 3 * R];

    const int tid = threadIdx.x;
    const int N = a.N;
    int bx, by, z;  // z: right-hand side of a split launch (R = 1, one per z)
    tile_rhs_of_block(bx, by, z);
    const int x0 = bx * T, y0 = by * T;
    const int ex0 = x0 - HL, ey0 = y0 - HL;
    const E h2 = (E)(a.h * a.h), ih2 = (E)(1.0 / (a.h * a.h));
    const E om = (E)a.omega;

    E fr[R][KP][2], Dr[KP][2], iDr[KP][2];
    tile_load<E, R, HELM, EX, EY, KP, NT>(su, fr, Dr, iDr, a.u_in + z, a.f + z, a.k2, a.pitch, ex0, ey0, N,
                                      a.h * a.h);
    __syncthreads();

    auto residual = [&](int r, int k, int j, int l) {
        const E u0 = su[r][l];
        const E nb = su[r][l - 1] + su[r][l + 1] + su[r][l - EX] + su[r][l + EX];
        const E D = pick(j, Dr[k][0], Dr[k][1]);
        const E fv = pick(j, fr[r][k][0], fr[r][k][1]);
        return fmad(-fmad(-D, u0, nb), ih2, fv);
    };

    if (a.norm_part) {  // residual of the incoming iterate on the owned interior nodes
        double acc[3 * R];
#pragma unroll
        for (int q = 0; q < 3 * R; ++q) acc[q] = 0.0;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const int p = tid + k * NT;
            const int ly = p / PW, px = p - ly * PW;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int lx = 2 * px + j;
                const int gx = ex0 + lx, gy = ey0 + ly;
                if (p < NP && lx >= HL && lx < HL + T && ly >= HL && ly < HL + T && gx >= 1 &&
                    gx <= N - 1 && gy >= 1 && gy <= N - 1) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double rr = residual(r, k, j, ly * EX + lx);
                        const double fv = pick(j, fr[r][k][0], fr[r][k][1]);
                        const double uv = su[r][ly * EX + lx];
                        acc[3 * r] += rr * rr;
                        acc[3 * r + 1] += fv * fv;
                        acc[3 * r + 2] += uv * uv;
                    }
                }
            }
        }
        block_sum<3 * R, NT>(acc, red);
        if (tid == 0) {
            const int b = by * gridDim.x + bx;
#pragma unroll
            for (int q = 0; q < 3 * R; ++q) a.norm_part[(3 * z + q) * a.nblk + b] = acc[q];
        }
    }

    for (int s = 0; s < NU; ++s)
        for (int color = 0; color < 2; ++color) {
            tile_sweep<E, R, HELM, EX, EY, KP, NT>(su, fr, iDr, ex0, ey0, N, h2, om, color);
            __syncthreads();
        }

    // write the owned nodes; residual on [x0-1, x0+T-1]^2 into registers
    E rr[R][KP][2];
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int p = tid + k * NT;
        const int ly = p / PW, px = p - ly * PW;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lx = 2 * px + j;
            const int gx = ex0 + lx, gy = ey0 + ly;
            const int l = ly * EX + lx;
            if (p < NP && lx >= HL && lx < HL + T && ly >= HL && ly < HL + T && gx <= N - 1 &&
                gy <= N - 1)
#pragma unroll
                for (int r = 0; r < R; ++r) a.u_out[r + z][(size_t)gy * a.pitch + gx] = su[r][l];
            const bool interior = p < NP && lx >= HL - 1 && lx <= HL + T - 1 && ly >= HL - 1 &&
                                  ly <= HL + T - 1 && gx >= 1 && gx <= N - 1 && gy >= 1 &&
                                  gy <= N - 1;
#pragma unroll
            for (int r = 0; r < R; ++r) rr[r][k][j] = interior ? residual(r, k, j, l) : E(0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KP; ++k) {  // the residual replaces u in LDS
        const int p = tid + k * NT;
        const int ly = p / PW, px = p - ly * PW;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lx = 2 * px + j;
            if (p < NP && lx >= HL - 1 && lx <= HL + T - 1 && ly >= HL - 1 && ly <= HL + T - 1)
#pragma unroll
                for (int r = 0; r < R; ++r) su[r][ly * EX + lx] = rr[r][k][j];
        }
    }
    __syncthreads();

    // full weighting onto coarse nodes x0/2 .. x0/2 + T/2 - 1 (< N/2)
    const int Nc = N / 2;
    for (int i = tid; i < (T / 2) * (T / 2); i += NT) {
        const int oy = i / (T / 2), ox = i - oy * (T / 2);
        const int I = x0 / 2 + ox, J = y0 / 2 + oy;
        if (I > Nc - 1 || J > Nc - 1) continue;
        const bool interior = I >= 1 && J >= 1;
        const int l = (2 * J - ey0) * EX + (2 * I - ex0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            E v = E(0);
            if (interior) {
                const E* q = su[r];
                v = (E(4) * q[l] + E(2) * (q[l - 1] + q[l + 1] + q[l - EX] + q[l + EX]) +
                     (q[l - EX - 1] + q[l - EX + 1] + q[l + EX - 1] + q[l + EX + 1])) *
                    E(1.0 / 16.0);
            }
            a.f_c[r + z][(size_t)J * a.pitch_c + I] = v;
        }
    }
}

template <typename E>
struct UpArgs {
    int N;
    double h;
    int pitch, pitch_c;
    const E* u_mid[2];
    const E* e_c[2];
    const E* f[2];
    const double* k2;
    E* u_out[2];
    double omega;
    // (register tiles, double only) nullptr or [3R][nblk]: sums r^2, f^2, u^2
    // of the corrected, smoothed u on the owned nodes (halo 2 nu + 2)
    double* norm_part;
    int nblk;
    // (float, finest level of the mixed form) nullptr, or the FP64 iterates
    // that the result corrects in place (u += e) instead of being stored
    double* corr[2];
};

// Up pass of one level: u += bilinear prolongation of the coarse correction on
// the whole tile (halo 2 nu), nu2 sweeps, write the owned nodes.
template <typename E, int R, bool HELM, int NU, int T>
__global__ __launch_bounds__(tile_threads<T>()) void k_mg_up(UpArgs<E> a) {
    constexpr int NT = tile_threads<T>();
    constexpr int H = 2 * NU;
    constexpr int EX = T + 2 * H, EY = EX;
    using S = TileShape<R, HELM, EX, EY, NT>;
    constexpr int PW = S::PW, NP = S::NP, KP = S::KP, EN = S::EN;
    constexpr int CX = EX / 2 + 1, CY = EY / 2 + 1;
    __shared__ E su[R][EN];
    __shared__ E se[R][CX * CY];

    const int tid = threadIdx.x;
    const int N = a.N, Nc = N / 2;
    int bx, by, z;  // z: right-hand side of a split launch (R = 1, one per z)
    tile_rhs_of_block(bx, by, z);
    const int x0 = bx * T, y0 = by * T;
    const int ex0 = x0 - H, ey0 = y0 - H;  // even
    const int cx0 = ex0 / 2, cy0 = ey0 / 2;
    const E h2 = (E)(a.h * a.h);
    const E om = (E)a.omega;

    E fr[R][KP][2], Dr[KP][2], iDr[KP][2];
    tile_load<E, R, HELM, EX, EY, KP, NT>(su, fr, Dr, iDr, a.u_mid + z, a.f + z, a.k2, a.pitch, ex0, ey0, N,
                                      a.h * a.h);
    // the coarse correction, loaded as the tile (threads past the end redo
    // the last node)
#pragma unroll
    for (int q = 0; q < (CX * CY + NT - 1) / NT; ++q) {
        const int i = min(tid + q * NT, CX * CY - 1);
        const int cy = i / CX, cx = i - cy * CX;
        const int I = cx0 + cx, J = cy0 + cy;
        const bool in = I >= 0 && I <= Nc && J >= 0 && J <= Nc;
        const size_t g = (size_t)min(max(J, 0), Nc) * a.pitch_c + min(max(I, 0), Nc);
#pragma unroll
        for (int r = 0; r < R; ++r) se[r][i] = a.e_c[r + z][g] * E(in ? 1 : 0);
    }
    __syncthreads();

#pragma unroll
    for (int k = 0; k < KP; ++k) {  // each thread corrects the nodes of its own pairs
        const int p = tid + k * NT;
        const int ly = p / PW, px = p - ly * PW;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lx = 2 * px + j;
            const int gx = ex0 + lx, gy = ey0 + ly;
            if (p >= NP || gx < 1 || gx > N - 1 || gy < 1 || gy > N - 1) continue;
            const int c = ((gy >> 1) - cy0) * CX + (gx >> 1) - cx0;
            const bool ox = gx & 1, oy = gy & 1;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const E* e = se[r];
                E v;
                if (!ox && !oy) v = e[c];
                else if (ox && !oy) v = E(0.5) * (e[c] + e[c + 1]);
                else if (!ox && oy) v = E(0.5) * (e[c] + e[c + CX]);
                else v = E(0.25) * (e[c] + e[c + 1] + e[c + CX] + e[c + CX + 1]);
                su[r][ly * EX + lx] += v;
            }
        }
    }
    __syncthreads();

    for (int s = 0; s < NU; ++s)
        for (int color = 0; color < 2; ++color) {
            tile_sweep<E, R, HELM, EX, EY, KP, NT>(su, fr, iDr, ex0, ey0, N, h2, om, color);
            __syncthreads();
        }

#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int p = tid + k * NT;
        const int ly = p / PW, px = p - ly * PW;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int lx = 2 * px + j;
            const int gx = ex0 + lx, gy = ey0 + ly;
            if (p < NP && lx >= H && lx < H + T && ly >= H && ly < H + T && gx <= N - 1 &&
                gy <= N - 1)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const size_t g = (size_t)gy * a.pitch + gx;
                    if (a.corr[0]) a.corr[r + z][g] += (double)su[r][ly * EX + lx];
                    else a.u_out[r + z][g] = su[r][ly * EX + lx];
                }
        }
    }
}

// ------------------------------------------------------- register tiles --
//
// Tile kernels for the large levels with the iterate held in registers.  A
// workgroup of NW wavefronts holds a 128-column x 4 NW-row block of nodes
// whose node (0, 0) is global node (ex0, ey0), both even: lane l of wavefront
// w holds the node pair (2l, 2l + 1) of the rows 4w .. 4w + 3.  The colour of
// element j of row k is (j + k) % 2, so in a half sweep every lane updates one
// node per row, with no divergence.  Horizontal neighbours come from the next
// lane by DPP wave shifts, vertical ones from the lane's own rows; the rows at
// wavefront boundaries go through LDS once per half sweep.  The arithmetic and
// its order are those of the LDS tile kernels above: both give the same bits.
#ifndef WQ_REG_ROWS
#define WQ_REG_ROWS 4
#endif
constexpr int kRegRows = WQ_REG_ROWS;  // rows per wavefront (even)
#ifndef WQ_REG_WAVES
#define WQ_REG_WAVES 8
#endif
#ifndef WQ_REG_TILE_MIN
#define WQ_REG_TILE_MIN 512
#endif
constexpr int kRegWaves = WQ_REG_WAVES;
static_assert(kRegWaves * kRegRows >= 32, "register tiles need at least 32 rows");

// DPP wave shifts by one lane: lane i reads lane i - 1 (wave_shr:1) or lane
// i + 1 (wave_shl:1); the lane past the end of the wavefront reads 0.
constexpr int kFromLeft = 0x138, kFromRight = 0x130;
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <typename E> struct Pair2;
template <> struct Pair2<double> { using T = double2; };
template <> struct Pair2<float> { using T = float2; };

// Geometry of a register tile with halo HL: owned TX x TY nodes (K rows per
// wavefront).
template <int HL, int NW, int K = kRegRows>
struct RegShape {
    static constexpr int ROWS = K * NW;
    static constexpr int TX = 128 - 2 * HL, TY = ROWS - 2 * HL;
    static_assert(TY > 0 && HL % 2 == 0, "register tile shape");
};

// Loads the lane's pairs of u (nullptr: 0), f and the Gauss-Seidel diagonal:
// D = 4 + h^2 k2 and 1/D formed in double, rounded to E.  Nodes outside
// [0, N]^2 read 0 (D = 4).
template <typename E, int R, bool HELM, int K>
__device__ __forceinline__ void reg_load(E (&u)[R][K][2], E (&f)[R][K][2], E (&D)[K][2],
                                         E (&iD)[K][2], const E* const* uin, const E* const* fin,
                                         const double* k2, int pitch, int gx, int gy0, int N,
                                         double h2) {
    using V2 = typename Pair2<E>::T;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int gy = gy0 + k;
        const bool in = gy >= 0 && gy <= N && gx >= 0 && gx <= N;
        const bool in1 = in && gx + 1 <= N;  // gx + 1 <= pitch - 1: the load stays in the row
        // every row's loads issued without a lane-dependent branch (a node
        // past the grid loads node 0 and is masked by a product with 0: the
        // values are finite), so that the rows' loads are in flight together
        const size_t g = in ? (size_t)gy * pitch + gx : 0;
        const E m0 = in ? E(1) : E(0), m1 = in1 ? E(1) : E(0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            V2 uv{E(0), E(0)};
            if (uin[r]) uv = *reinterpret_cast<const V2*>(uin[r] + g);  // uniform
            const V2 fv = *reinterpret_cast<const V2*>(fin[r] + g);
            u[r][k][0] = uv.x * m0;
            u[r][k][1] = uv.y * m1;
            f[r][k][0] = fv.x * m0;
            f[r][k][1] = fv.y * m1;
        }
        double q0 = 0.0, q1 = 0.0;
        if (HELM) {
            const double2 kv = *reinterpret_cast<const double2*>(k2 + g);
            q0 = kv.x * (double)m0;
            q1 = kv.y * (double)m1;
        }
        const double D0 = fmad(h2, q0, 4.0), D1 = fmad(h2, q1, 4.0);
        D[k][0] = (E)D0;
        D[k][1] = (E)D1;
        iD[k][0] = HELM ? (E)(1.0 / D0) : E(0.25);
        iD[k][1] = HELM ? (E)(1.0 / D1) : E(0.25);
    }
}

// Rows 0 and K-1 of every wavefront into buffer b; after a barrier each
// wavefront reads the row above its row 0 and the row below its row K-1
// (0 past the tile).
template <typename E, int R, int K, int NW>
struct RegExchange {
    using V2 = typename Pair2<E>::T;
    V2 (*xb)[R][NW][2][64];
    __device__ __forceinline__ void put(int b, const E (&v)[R][K][2], int w, int lane) const {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            xb[b][r][w][0][lane] = V2{v[r][0][0], v[r][0][1]};
            xb[b][r][w][1][lane] = V2{v[r][K - 1][0], v[r][K - 1][1]};
        }
    }
    __device__ __forceinline__ void get(int b, V2 (&up)[R], V2 (&dn)[R], int w, int lane) const {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            up[r] = w > 0 ? xb[b][r][w - 1][1][lane] : V2{E(0), E(0)};
            dn[r] = w < NW - 1 ? xb[b][r][w + 1][0][lane] : V2{E(0), E(0)};
        }
    }
};

template <typename V2>
__device__ __forceinline__ auto el(const V2& v, int j) { return j ? v.y : v.x; }

// One red-black half sweep of colour c over the lane's rows; upd[k][j] marks
// the nodes inside the tile's update region and the domain interior.
template <typename E, int R, bool HELM, int K>
__device__ __forceinline__ void reg_half_sweep(E (&u)[R][K][2], const E (&f)[R][K][2],
                                               const E (&iD)[K][2], const bool (&upd)[K][2],
                                               const typename Pair2<E>::T (&up)[R],
                                               const typename Pair2<E>::T (&dn)[R], E h2, E om,
                                               int c) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            if (((c + k) & 1) != jj) continue;  // element jj of row k has colour c
            const int j = jj;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                E left, right;
                if (j == 0) {
                    left = lane_shift<kFromLeft>(u[r][k][1]);
                    right = u[r][k][1];
                } else {
                    left = u[r][k][0];
                    right = lane_shift<kFromRight>(u[r][k][0]);
                }
                const E upv = k == 0 ? el(up[r], j) : u[r][k - 1][j];
                const E dnv = k == K - 1 ? el(dn[r], j) : u[r][k + 1][j];
                const E nb = left + right + upv + dnv;
                const E nv = sor_update(u[r][k][j], nb, f[r][k][j], iD[k][j], h2, om);
                u[r][k][j] = upd[k][j] ? nv : u[r][k][j];
            }
        }
    }
}

// Residual f - A u of every node of the lane's rows (0 outside the domain
// interior); up/dn are the rows across the wavefront boundaries.
template <typename E, int R, int K>
__device__ __forceinline__ void reg_residual(E (&rr)[R][K][2], const E (&u)[R][K][2],
                                             const E (&f)[R][K][2], const E (&D)[K][2],
                                             const bool (&dom)[K][2],
                                             const typename Pair2<E>::T (&up)[R],
                                             const typename Pair2<E>::T (&dn)[R], E ih2) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const E l0 = lane_shift<kFromLeft>(u[r][k][1]);
            const E r1 = lane_shift<kFromRight>(u[r][k][0]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const E left = j == 0 ? l0 : u[r][k][0];
                const E right = j == 0 ? u[r][k][1] : r1;
                const E upv = k == 0 ? el(up[r], j) : u[r][k - 1][j];
                const E dnv = k == K - 1 ? el(dn[r], j) : u[r][k + 1][j];
                const E nb = left + right + upv + dnv;
                const E v = fmad(-fmad(-D[k][j], u[r][k][j], nb), ih2, f[r][k][j]);
                rr[r][k][j] = dom[k][j] ? v : E(0);
            }
        }
}

// Down pass with register tiles: the same steps as k_mg_down.
template <typename E, int R, bool HELM, int NU, int NW>
__global__ __launch_bounds__(64 * NW) void k_mg_down_reg(DownArgs<E> a) {
    constexpr int K = kRegRows;
    constexpr int HL = 2 * NU + 2;
    using S = RegShape<HL, NW>;
    constexpr int TX = S::TX, TY = S::TY, ROWS = S::ROWS;
    using V2 = typename Pair2<E>::T;
    __shared__ V2 xb[2][R][NW][2][64];
    __shared__ double red[NW * 3 * R];
    const RegExchange<E, R, K, NW> xc{xb};

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int N = a.N;
    int bx, by, z;  // z: right-hand side of a split launch (R = 1, one per z)
    tile_rhs_of_block(bx, by, z);
    const int x0 = bx * TX, y0 = by * TY;
    const int ex0 = x0 - HL, ey0 = y0 - HL;
    const int gx = ex0 + 2 * lane, gy0 = ey0 + w * K;
    const E h2 = (E)(a.h * a.h), ih2 = (E)(1.0 / (a.h * a.h));
    const E om = (E)a.omega;

    E u[R][K][2], f[R][K][2], D[K][2], iD[K][2];
    reg_load<E, R, HELM, K>(u, f, D, iD, a.u_in + z, a.f + z, a.k2, a.pitch, gx, gy0, N, a.h * a.h);

    bool upd[K][2], dom[K][2], own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int Y = w * K + k, gy = gy0 + k;
        own[k] = Y >= HL && Y < HL + TY;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int X = 2 * lane + j;
            dom[k][j] = gx + j >= 1 && gx + j <= N - 1 && gy >= 1 && gy <= N - 1;
            upd[k][j] = dom[k][j] && X >= 1 && X <= 126 && Y >= 1 && Y <= ROWS - 2;
        }
    }
    const bool own_x = 2 * lane >= HL && 2 * lane < HL + TX;

    V2 up[R], dn[R];
    int buf = 0;
    xc.put(buf, u, w, lane);
    __syncthreads();
    xc.get(buf, up, dn, w, lane);

    if (a.norm_part) {  // residual of the incoming iterate on the owned interior nodes
        E rr[R][K][2];
        reg_residual<E, R, K>(rr, u, f, D, dom, up, dn, ih2);
        double acc[3 * R];
#pragma unroll
        for (int q = 0; q < 3 * R; ++q) acc[q] = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (own[k] && own_x && dom[k][j])
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double rv = rr[r][k][j];
                        const double fv = f[r][k][j];
                        const double uv = u[r][k][j];
                        acc[3 * r] += rv * rv;
                        acc[3 * r + 1] += fv * fv;
                        acc[3 * r + 2] += uv * uv;
                    }
        block_sum<3 * R, 64 * NW>(acc, red);
        if (threadIdx.x == 0) {
            const int b = by * gridDim.x + bx;
#pragma unroll
            for (int q = 0; q < 3 * R; ++q) a.norm_part[(3 * z + q) * a.nblk + b] = acc[q];
        }
    }

#pragma unroll
    for (int q = 0; q < 2 * NU; ++q) {
        if (q > 0) {
            buf ^= 1;
            xc.put(buf, u, w, lane);
            __syncthreads();
            xc.get(buf, up, dn, w, lane);
        }
        reg_half_sweep<E, R, HELM, K>(u, f, iD, upd, up, dn, h2, om, q & 1);
    }

    // the smoothed owned nodes
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int gy = gy0 + k;
        if (own[k] && own_x && gx <= N - 1 && gy <= N - 1)
#pragma unroll
            for (int r = 0; r < R; ++r)
                *reinterpret_cast<V2*>(a.u_out[r + z] + (size_t)gy * a.pitch + gx) =
                    V2{u[r][k][0], u[r][k][1]};
    }

    // residual of the smoothed iterate, then full weighting onto the coarse
    // nodes (x0/2 + i, y0/2 + m) owned by this tile
    buf ^= 1;
    xc.put(buf, u, w, lane);
    __syncthreads();
    xc.get(buf, up, dn, w, lane);
    E rr[R][K][2];
    reg_residual<E, R, K>(rr, u, f, D, dom, up, dn, ih2);
    buf ^= 1;
    xc.put(buf, rr, w, lane);
    __syncthreads();
    xc.get(buf, up, dn, w, lane);

    const int Nc = N / 2;
    const int I = ex0 / 2 + lane;
#pragma unroll
    for (int k = 0; k < K; k += 2) {
        const int J = (gy0 + k) / 2;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const E am = k == 0 ? up[r].y : rr[r][k - 1][1];  // row k-1, odd column
            const E a0 = k == 0 ? up[r].x : rr[r][k - 1][0];
            const E sl = lane_shift<kFromLeft>(rr[r][k][1]);
            const E sm = lane_shift<kFromLeft>(am);
            const E sp = lane_shift<kFromLeft>(rr[r][k + 1][1]);
            if (own[k] && own_x && I <= Nc - 1 && J <= Nc - 1) {
                E v = E(0);
                if (I >= 1 && J >= 1)
                    v = (E(4) * rr[r][k][0] +
                         E(2) * (sl + rr[r][k][1] + a0 + rr[r][k + 1][0]) +
                         (sm + am + sp + rr[r][k + 1][1])) *
                        E(1.0 / 16.0);
                a.f_c[r + z][(size_t)J * a.pitch_c + I] = v;
            }
        }
    }
}

// Up pass with register tiles: the same steps as k_mg_up.  NORM: the tiles
// carry a halo of 2 nu + 2, so that the residual of the result is exact on the
// owned nodes, and its norms go to a.norm_part (the last cycle of a batch).
template <typename E, int R, bool HELM, int NU, int NW, bool NORM>
__global__ __launch_bounds__(64 * NW) void k_mg_up_reg(UpArgs<E> a) {
    constexpr int K = kRegRows;
    constexpr int H = NORM ? 2 * NU + 2 : 2 * NU;
    using S = RegShape<H, NW>;
    constexpr int TX = S::TX, TY = S::TY, ROWS = S::ROWS;
    using V2 = typename Pair2<E>::T;
    __shared__ V2 xb[2][R][NW][2][64];
    const RegExchange<E, R, K, NW> xc{xb};

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int N = a.N, Nc = N / 2;
    int bx, by, z;  // z: right-hand side of a split launch (R = 1, one per z)
    tile_rhs_of_block(bx, by, z);
    const int x0 = bx * TX, y0 = by * TY;
    const int ex0 = x0 - H, ey0 = y0 - H;
    const int gx = ex0 + 2 * lane, gy0 = ey0 + w * K;
    const E h2 = (E)(a.h * a.h);
    const E om = (E)a.omega;

    E u[R][K][2], f[R][K][2], D[K][2], iD[K][2];
    reg_load<E, R, HELM, K>(u, f, D, iD, a.u_mid + z, a.f + z, a.k2, a.pitch, gx, gy0, N, a.h * a.h);

    // coarse correction at (I, J0 + m) and (I + 1, J0 + m), m = 0 .. K/2
    constexpr int KC = K / 2 + 1;
    const int I = ex0 / 2 + lane, J0 = gy0 / 2;
    E eL[R][KC], eR[R][KC];
#pragma unroll
    for (int m = 0; m < KC; ++m) {
        const int J = J0 + m;
        const bool inJ = J >= 0 && J <= Nc;
        const bool inL = inJ && I >= 0 && I <= Nc, inR = inJ && I + 1 >= 0 && I + 1 <= Nc;
        // indices clamped into the coarse grid, values masked after (no load
        // behind a lane-dependent branch)
        const size_t row = (size_t)min(max(J, 0), Nc) * a.pitch_c;
        const int iL = min(max(I, 0), Nc), iR = min(max(I + 1, 0), Nc);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            eL[r][m] = a.e_c[r + z][row + iL] * (inL ? E(1) : E(0));
            eR[r][m] = a.e_c[r + z][row + iR] * (inR ? E(1) : E(0));
        }
    }

    bool upd[K][2], own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int Y = w * K + k, gy = gy0 + k;
        own[k] = Y >= H && Y < H + TY;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int X = 2 * lane + j;
            const bool dom = gx + j >= 1 && gx + j <= N - 1 && gy >= 1 && gy <= N - 1;
            upd[k][j] = dom && X >= 1 && X <= 126 && Y >= 1 && Y <= ROWS - 2;
            // u += bilinear prolongation (gy even: row J0 + k/2; odd: between it and the next)
            const int m = k / 2;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                E v;
                if (!(k & 1)) v = j == 0 ? eL[r][m] : E(0.5) * (eL[r][m] + eR[r][m]);
                else if (j == 0) v = E(0.5) * (eL[r][m] + eL[r][m + 1]);
                else v = E(0.25) * (eL[r][m] + eR[r][m] + eL[r][m + 1] + eR[r][m + 1]);
                if (dom) u[r][k][j] += v;
            }
        }
    }
    const bool own_x = 2 * lane >= H && 2 * lane < H + TX;

    V2 up[R], dn[R];
#pragma unroll
    for (int q = 0; q < 2 * NU; ++q) {
        xc.put(q & 1, u, w, lane);
        __syncthreads();
        xc.get(q & 1, up, dn, w, lane);
        reg_half_sweep<E, R, HELM, K>(u, f, iD, upd, up, dn, h2, om, q & 1);
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int gy = gy0 + k;
        if (own[k] && own_x && gx <= N - 1 && gy <= N - 1)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const size_t g = (size_t)gy * a.pitch + gx;
                if (a.corr[0]) {
                    double2* p = reinterpret_cast<double2*>(a.corr[r + z] + g);
                    double2 o = *p;
                    o.x += (double)u[r][k][0];
                    o.y += (double)u[r][k][1];
                    *p = o;
                } else {
                    *reinterpret_cast<V2*>(a.u_out[r + z] + g) = V2{u[r][k][0], u[r][k][1]};
                }
            }
    }

    if (NORM) {  // residual norms of the result on the owned interior nodes
        __shared__ double red[NW * 3 * R];
        bool dom[K][2];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                dom[k][j] = gx + j >= 1 && gx + j <= N - 1 && gy0 + k >= 1 && gy0 + k <= N - 1;
        const int qb = 2 * NU;  // exchange buffer not used by the last sweep
        xc.put(qb & 1, u, w, lane);
        __syncthreads();
        xc.get(qb & 1, up, dn, w, lane);
        E rr[R][K][2];
        reg_residual<E, R, K>(rr, u, f, D, dom, up, dn, (E)(1.0 / (a.h * a.h)));
        double acc[3 * R];
#pragma unroll
        for (int q = 0; q < 3 * R; ++q) acc[q] = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (own[k] && own_x && dom[k][j])
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double rv = rr[r][k][j];
                        const double fv = f[r][k][j];
                        const double uv = u[r][k][j];
                        acc[3 * r] += rv * rv;
                        acc[3 * r + 1] += fv * fv;
                        acc[3 * r + 2] += uv * uv;
                    }
        block_sum<3 * R, 64 * NW>(acc, red);
        if (threadIdx.x == 0) {
            const int b = by * gridDim.x + bx;
#pragma unroll
            for (int q = 0; q < 3 * R; ++q) a.norm_part[(3 * z + q) * a.nblk + b] = acc[q];
        }
    }
}

// Up pass of one V-cycle fused with the down pass of the next, on the finest
// level (register tiles, FP64, one right-hand side per workgroup): the tile of
// the smoothed iterate of the last down pass is corrected by the prolonged
// coarse correction and post-smoothed (the up pass), the residual norms of that
// iterate are recorded (those the next down pass would record), then it is
// pre-smoothed, written, and its residual restricted (the down pass).  The
// arithmetic and its order are those of the two passes, so the result has the
// same bits; the iterate between them never goes to memory.  Halo: 2 NU2 + 2
// NU1 + 2 nodes.
template <typename E>
struct FuseArgs {
    int N;
    double h;
    int pitch, pitch_c;
    const E* u_mid[2];  // smoothed iterate of the previous down pass
    const E* e_c[2];    // coarse correction
    const E* f[2];
    const double* k2;
    E* u_out[2];        // smoothed iterate of this pass's down part
    E* f_c[2];          // restricted residual
    double omega;
    double* norm_part;  // [3R][nblk]: sums r^2, f^2, u^2 of the up part's result (or null)
    int nblk;
};

template <typename E, int R, bool HELM, int NU1, int NU2, int NW, int K>
__global__ __launch_bounds__(64 * NW) void k_mg_updown_reg(FuseArgs<E> a) {
    constexpr int HL = 2 * NU2 + 2 * NU1 + 2;
    using S = RegShape<HL, NW, K>;
    constexpr int TX = S::TX, TY = S::TY, ROWS = S::ROWS;
    using V2 = typename Pair2<E>::T;
    __shared__ V2 xb[2][R][NW][2][64];
    __shared__ double red[NW * 3 * R];
    const RegExchange<E, R, K, NW> xc{xb};

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int N = a.N, Nc = N / 2;
    int bx, by, z;  // z: right-hand side of a split launch (R = 1, one per z)
    tile_rhs_of_block(bx, by, z);
    const int x0 = bx * TX, y0 = by * TY;
    const int ex0 = x0 - HL, ey0 = y0 - HL;
    const int gx = ex0 + 2 * lane, gy0 = ey0 + w * K;
    const E h2 = (E)(a.h * a.h), ih2 = (E)(1.0 / (a.h * a.h));
    const E om = (E)a.omega;

    E u[R][K][2], f[R][K][2], D[K][2], iD[K][2];
    reg_load<E, R, HELM, K>(u, f, D, iD, a.u_mid + z, a.f + z, a.k2, a.pitch, gx, gy0, N, a.h * a.h);

    // up part: coarse correction at (I, J0 + m) and (I + 1, J0 + m)
    constexpr int KC = K / 2 + 1;
    const int I = ex0 / 2 + lane, J0 = gy0 / 2;
    E eL[R][KC], eR[R][KC];
#pragma unroll
    for (int m = 0; m < KC; ++m) {
        const int J = J0 + m;
        const bool inJ = J >= 0 && J <= Nc;
        const bool inL = inJ && I >= 0 && I <= Nc, inR = inJ && I + 1 >= 0 && I + 1 <= Nc;
        // indices clamped into the coarse grid, values masked after (no load
        // behind a lane-dependent branch)
        const size_t row = (size_t)min(max(J, 0), Nc) * a.pitch_c;
        const int iL = min(max(I, 0), Nc), iR = min(max(I + 1, 0), Nc);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            eL[r][m] = a.e_c[r + z][row + iL] * (inL ? E(1) : E(0));
            eR[r][m] = a.e_c[r + z][row + iR] * (inR ? E(1) : E(0));
        }
    }
    bool upd[K][2], dom[K][2], own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int Y = w * K + k, gy = gy0 + k;
        own[k] = Y >= HL && Y < HL + TY;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int X = 2 * lane + j;
            dom[k][j] = gx + j >= 1 && gx + j <= N - 1 && gy >= 1 && gy <= N - 1;
            upd[k][j] = dom[k][j] && X >= 1 && X <= 126 && Y >= 1 && Y <= ROWS - 2;
            const int m = k / 2;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                E v;
                if (!(k & 1)) v = j == 0 ? eL[r][m] : E(0.5) * (eL[r][m] + eR[r][m]);
                else if (j == 0) v = E(0.5) * (eL[r][m] + eL[r][m + 1]);
                else v = E(0.25) * (eL[r][m] + eR[r][m] + eL[r][m + 1] + eR[r][m + 1]);
                if (dom[k][j]) u[r][k][j] += v;
            }
        }
    }
    const bool own_x = 2 * lane >= HL && 2 * lane < HL + TX;

    V2 up[R], dn[R];
    int buf = 0;
#pragma unroll
    for (int q = 0; q < 2 * NU2; ++q) {
        xc.put(buf, u, w, lane);
        __syncthreads();
        xc.get(buf, up, dn, w, lane);
        buf ^= 1;
        reg_half_sweep<E, R, HELM, K>(u, f, iD, upd, up, dn, h2, om, q & 1);
    }

    // the norms of the up part's result (the next cycle's incoming iterate)
    xc.put(buf, u, w, lane);
    __syncthreads();
    xc.get(buf, up, dn, w, lane);
    buf ^= 1;
    if (a.norm_part) {
        E rr[R][K][2];
        reg_residual<E, R, K>(rr, u, f, D, dom, up, dn, ih2);
        double acc[3 * R];
#pragma unroll
        for (int q = 0; q < 3 * R; ++q) acc[q] = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (own[k] && own_x && dom[k][j])
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double rv = rr[r][k][j];
                        const double fv = f[r][k][j];
                        const double uv = u[r][k][j];
                        acc[3 * r] += rv * rv;
                        acc[3 * r + 1] += fv * fv;
                        acc[3 * r + 2] += uv * uv;
                    }
        block_sum<3 * R, 64 * NW>(acc, red);
        if (threadIdx.x == 0) {
            const int b = by * gridDim.x + bx;
#pragma unroll
            for (int q = 0; q < 3 * R; ++q) a.norm_part[(3 * z + q) * a.nblk + b] = acc[q];
        }
    }

    // down part: pre-smoothing (the first half sweep uses the exchange above)
#pragma unroll
    for (int q = 0; q < 2 * NU1; ++q) {
        if (q > 0) {
            xc.put(buf, u, w, lane);
            __syncthreads();
            xc.get(buf, up, dn, w, lane);
            buf ^= 1;
        }
        reg_half_sweep<E, R, HELM, K>(u, f, iD, upd, up, dn, h2, om, q & 1);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int gy = gy0 + k;
        if (own[k] && own_x && gx <= N - 1 && gy <= N - 1)
#pragma unroll
            for (int r = 0; r < R; ++r)
                *reinterpret_cast<V2*>(a.u_out[r + z] + (size_t)gy * a.pitch + gx) =
                    V2{u[r][k][0], u[r][k][1]};
    }
    xc.put(buf, u, w, lane);
    __syncthreads();
    xc.get(buf, up, dn, w, lane);
    buf ^= 1;
    E rr[R][K][2];
    reg_residual<E, R, K>(rr, u, f, D, dom, up, dn, ih2);
    xc.put(buf, rr, w, lane);
    __syncthreads();
    xc.get(buf, up, dn, w, lane);
    const int Ic = ex0 / 2 + lane;
#pragma unroll
    for (int k = 0; k < K; k += 2) {
        const int J = (gy0 + k) / 2;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const E am = k == 0 ? up[r].y : rr[r][k - 1][1];  // row k-1, odd column
            const E a0 = k == 0 ? up[r].x : rr[r][k - 1][0];
            const E sl = lane_shift<kFromLeft>(rr[r][k][1]);
            const E sm = lane_shift<kFromLeft>(am);
            const E sp = lane_shift<kFromLeft>(rr[r][k + 1][1]);
            if (own[k] && own_x && Ic <= Nc - 1 && J <= Nc - 1) {
                E v = E(0);
                if (Ic >= 1 && J >= 1)
                    v = (E(4) * rr[r][k][0] +
                         E(2) * (sl + rr[r][k][1] + a0 + rr[r][k + 1][0]) +
                         (sm + am + sp + rr[r][k + 1][1])) *
                        E(1.0 / 16.0);
                a.f_c[r + z][(size_t)J * a.pitch_c + Ic] = v;
            }
        }
    }
}


// ---------------------------------------------------------------- coarse --
//
// The levels of at most 64^2 cells of the Helmholtz V-cycle, and whole solves on
// grids that small, in one workgroup per right-hand side with the iterate in
// registers.  The 64^2 level lies across kCoarseWaves wavefronts (lane = column,
// 64 / kCoarseWaves rows each); the levels below run in the first wavefront
// alone, 64 / n row groups side by side, with no workgroup barrier.  The grid's
// boundary column and row 0 lie in the layout and are held at 0 by a zero 1/D;
// those at n read as 0 past the end.
//
// A lane's rows come in pairs (2m, 2m + 1), one red node ((x + y) even) and one
// black each, held as two arrays: with p = x mod 2 the red node of pair m lies
// in row 2m + p, the black one in row 2m + 1 - p.  A node's left and right
// neighbours are then the other colour's entry m of the neighbouring lanes (DPP
// wave shifts), its vertical ones the lane's own entry m and m + 1 or m - 1:
// every half sweep updates one node per lane and pair, with no divergence and
// no LDS but the row that crosses to the next wavefront or group.
//
// What bounds it is the serial chain of half sweeps and transfers of one
// workgroup per right-hand side, and its loads: 12.0 us for a launch of one V(1, 2)
// in float, 14.8 in double, 15.4 and 20.0 with two V(1, 1) (every level in LDS with a
// workgroup barrier per half sweep and one cycle per launch: 22.2 and 28.3).  Four
// wavefronts: with eight the double form spills (19.7 us for one cycle, float 12.1).
constexpr int kCoarseWaves = 4;
static_assert(kCoarseMax == 64, "the coarse kernel holds levels up to 64 cells a side");

// Level of n <= 32 cells in one wavefront: G groups of ROWS rows, NP row pairs
// per lane (lanes past G n idle).  Offsets of its LDS arrays: E, the correction
// it hands to the next finer level ((n + 1)^2); F, its right-hand side (n^2);
// T, its 1/D and D in the lane layout (entry (2 m + colour) 64 + lane).
template <int n>
struct CoarseLevel {
    static constexpr int G = n >= 16 ? 64 / n : (n == 8 ? 4 : 2);
    static constexpr int ROWS = n / G, NP = ROWS / 2;
};
template <int n0>
constexpr int coarse_threads() { return n0 == 64 ? 64 * kCoarseWaves : 64; }
template <int n0>
constexpr int coarse_rows() {
    if constexpr (n0 == 64) return 64 / kCoarseWaves;
    else return CoarseLevel<n0>::ROWS;
}
constexpr int coarse_off_E(int n) {  // levels 32, 16, 8, 4, 2
    int o = 0;
    for (int k = 32; k > n; k /= 2) o += (k + 1) * (k + 1);
    return o;
}
constexpr int coarse_off_F(int n) {
    int o = 0;
    for (int k = 32; k > n; k /= 2) o += k * k;
    return o;
}
constexpr int coarse_off_T(int n) {  // levels 32, 16, 8, 4: NP = 8, 2, 1, 1
    return n == 32 ? 0 : n == 16 ? 1024 : n == 8 ? 1280 : n == 4 ? 1408 : 1536;
}

constexpr int kCoarseT = coarse_off_T(2);
static_assert(kCoarseT < kCoarseTab, "room for the tables");

// The node of an entry of the T tables: its level, row and column, and whether
// it is an interior one (the rest: boundary, idle lanes).
struct CoarseSlot {
    int n, x, y;
    bool in;
};
__device__ __forceinline__ CoarseSlot coarse_slot(int i) {
    const int n = i >= coarse_off_T(4) ? 4 : i >= coarse_off_T(8) ? 8 : i >= coarse_off_T(16) ? 16 : 32;
    const int rows = n == 32 ? 16 : n == 16 ? 4 : 2, groups = n == 32 ? 2 : n == 4 ? 2 : 4;
    const int e = i - (n == 32 ? 0 : n == 16 ? coarse_off_T(16) : n == 8 ? coarse_off_T(8) : coarse_off_T(4));
    const int lane = e & 63, m = e >> 7, colour = (e >> 6) & 1;
    CoarseSlot c;
    c.n = n;
    c.x = lane & (n - 1);
    const int g = lane / n;
    c.y = g * rows + 2 * m + ((lane & 1) ^ colour);
    c.in = g < groups && c.x > 0 && c.y > 0;
    return c;
}

template <typename C>
struct CoarseLds {
    C E[coarse_off_E(1)];
    C F[coarse_off_F(1)];
    C id[kCoarseT], D[kCoarseT];
    C edge[2][kCoarseWaves + 2][64];  // rows across the wavefronts of the 64^2 level
    double red[kCoarseWaves][3];
};

template <typename E>
struct CoarseArgs {
    double h;  // of the top level
    int pitch;
    const E* f[2];
    const E* u_init[2];  // nullptr: zero initial guess
    CoarseTabs tab;  // Helmholtz: what k_coarse_k2 made of k2
    E* u_out[2];
    int ncycles, inner;  // ncycles times inner V-cycles
    int nu1, nu2;
    double omega;       // relaxation factor of the levels with h^2 <= h2max (Helmholtz)
    double h2max;       // coarser Helmholtz levels relax with factor 1
    double* norm_part;  // nullptr, or the sums of r^2, f^2, u^2 before each of the ncycles and after
    size_t norm_stride;  // the last ([3 r + q] of slots norm_stride apart)
};

// the tables in the type of the sweeps
template <typename C> __device__ __forceinline__ const C* coarse_tab(const double* d, const float* f);
template <> __device__ __forceinline__ const double* coarse_tab<double>(const double* d, const float*) { return d; }
template <> __device__ __forceinline__ const float* coarse_tab<float>(const double*, const float* f) { return f; }

// One half sweep: the nodes s (sor_update) from the other colour o.  q: the
// node's second vertical neighbour is entry m + 1, else m - 1; e: that of the
// lane's last or first pair, from the next wavefront or group.
template <typename C, int NP>
__device__ __forceinline__ void coarse_half(C (&s)[NP], const C (&f)[NP], const C (&id)[NP],
                                            const C (&o)[NP], C e, bool q, C h2, C om) {
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        const C hi = m + 1 < NP ? o[m + 1 < NP ? m + 1 : m] : e, lo = m > 0 ? o[m > 0 ? m - 1 : 0] : e;
        const C nb = lane_shift<kFromLeft>(o[m]) + lane_shift<kFromRight>(o[m]) + o[m] + (q ? hi : lo);
        s[m] = sor_update(s[m], nb, f[m], id[m], h2, om);
    }
}

// The same neighbours' residual f - A u; in, in0: the lane's nodes (its first
// entry) are interior ones, 0 elsewhere.
template <typename C, int NP>
__device__ __forceinline__ void coarse_resid(C (&r)[NP], const C (&u)[NP], const C (&f)[NP],
                                             const C (&D)[NP], const C (&o)[NP], C e, bool q, C ih2,
                                             bool in, bool in0) {
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        const C hi = m + 1 < NP ? o[m + 1 < NP ? m + 1 : m] : e, lo = m > 0 ? o[m > 0 ? m - 1 : 0] : e;
        const C nb = lane_shift<kFromLeft>(o[m]) + lane_shift<kFromRight>(o[m]) + o[m] + (q ? hi : lo);
        const C v = fmad(-fmad(-D[m], u[m], nb), ih2, f[m]);
        r[m] = (m > 0 ? in : in0) ? v : C(0);
    }
}

// Full weighting of the residual: fine row 2J = row 2m of the lane's pair, at
// the even columns.  An odd lane hands its three rows' weighted sum to its even
// neighbours; e: the row 2m - 1 of the lane's first pair.  Entry m, to be used
// on the even lanes.
template <typename C, int NP>
__device__ __forceinline__ void coarse_restrict(C (&v)[NP], const C (&rR)[NP], const C (&rB)[NP], C e,
                                                bool p) {
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        const C below = m > 0 ? (p ? rR[m > 0 ? m - 1 : 0] : rB[m > 0 ? m - 1 : 0]) : e;
        const C s = C(2) * rB[m] + rR[m] + below;
        v[m] = (C(4) * rR[m] + C(2) * (rB[m] + below) + lane_shift<kFromLeft>(s) +
                lane_shift<kFromRight>(s)) * C(1.0 / 16.0);
    }
}

// u += bilinear interpolation of the coarse correction E ((nc + 1)^2, zero
// boundary): column I = x / 2 (the mean with I + 1 at odd x), coarse rows J0 ..
// J0 + NP.
template <typename C, int NP>
__device__ __forceinline__ void coarse_prolong(C (&uR)[NP], C (&uB)[NP], const C* E, int lde, int x,
                                               int J0, bool p) {
    C c[NP + 1];
    const C* q = E + J0 * lde + (x >> 1);
#pragma unroll
    for (int m = 0; m <= NP; ++m) c[m] = C(0.5) * (q[m * lde] + q[m * lde + (p ? 1 : 0)]);
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        const C odd = C(0.5) * (c[m] + c[m + 1]);
        uR[m] += p ? odd : c[m];
        uB[m] += p ? c[m] : odd;
    }
}

// A level of n <= 32 cells in the calling wavefront.
template <typename C, int n, bool HELM>
struct CoarseWave {
    using L = CoarseLevel<n>;
    static constexpr int NP = L::NP, G = L::G;
    CoarseLds<C>& lds;
    int lane, x, g;
    bool p;
    C h2, om;
    double h;
    __device__ __forceinline__ CoarseWave(CoarseLds<C>& l, double h_, double omega, double h2max)
        : lds(l), lane(threadIdx.x & 63), x(lane & (n - 1)), g(lane / n), p(lane & 1), h(h_) {
        h2 = (C)(h * h);
        om = (C)(h * h > h2max ? 1.0 : omega);
    }
    __device__ __forceinline__ int row(int m, int colour) const {
        return g * L::ROWS + 2 * m + ((p ? 1 : 0) ^ colour);
    }
    // entry from the neighbouring row group (0 past the last one)
    __device__ __forceinline__ C edge(const C (&o)[NP], bool q) const {
        const C t = q ? o[0] : o[NP - 1];
        const C r = __shfl(t, (q ? lane + n : lane - n) & 63, 64);
        return q && g == G - 1 ? C(0) : r;
    }
    __device__ __forceinline__ void table(const C* T, int colour, C (&v)[NP]) const {
#pragma unroll
        for (int m = 0; m < NP; ++m) v[m] = T[coarse_off_T(n) + (2 * m + colour) * 64 + lane];
    }
    __device__ __forceinline__ void smooth(C (&uR)[NP], C (&uB)[NP], const C (&fR)[NP], const C (&fB)[NP],
                                           int nu) const {
        C iR[NP], iB[NP];
        table(lds.id, 0, iR);
        table(lds.id, 1, iB);
        for (int s = 0; s < nu; ++s) {
            coarse_half<C, NP>(uR, fR, iR, uB, edge(uB, p), p, h2, om);
            coarse_half<C, NP>(uB, fB, iB, uR, edge(uR, !p), !p, h2, om);
        }
    }
    __device__ __forceinline__ void load_f(C (&fR)[NP], C (&fB)[NP]) const {
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            fR[m] = g < G ? lds.F[coarse_off_F(n) + min(row(m, 0), n - 1) * n + x] : C(0);
            fB[m] = g < G ? lds.F[coarse_off_F(n) + min(row(m, 1), n - 1) * n + x] : C(0);
        }
    }
    // the correction into E for the next finer level
    __device__ __forceinline__ void store_E(const C (&uR)[NP], const C (&uB)[NP]) const {
        if (g < G)
#pragma unroll
            for (int m = 0; m < NP; ++m) {
                lds.E[coarse_off_E(n) + row(m, 0) * (n + 1) + x] = uR[m];
                lds.E[coarse_off_E(n) + row(m, 1) * (n + 1) + x] = uB[m];
            }
    }
    // V-cycle of this level and those below on u
    __device__ __forceinline__ void cycle(C (&uR)[NP], C (&uB)[NP], const C (&fR)[NP], const C (&fB)[NP],
                                          int nu1, int nu2, double omega, double h2max, double k2_two) const {
        constexpr int nc = n / 2;
        smooth(uR, uB, fR, fB, nu1);
        C rR[NP], rB[NP];
        {
            C dR[NP], dB[NP];
            table(lds.D, 0, dR);
            table(lds.D, 1, dB);
            const C ih2 = (C)(1.0 / (h * h));
            const bool in = x > 0 && g < G;
            coarse_resid<C, NP>(rR, uR, fR, dR, uB, edge(uB, p), p, ih2, in, in && (g > 0 || p));
            coarse_resid<C, NP>(rB, uB, fB, dB, uR, edge(uR, !p), !p, ih2, in, in && (g > 0 || !p));
        }
        C t[NP], v[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) t[m] = p ? rR[m] : rB[m];
        const C below = __shfl(t[NP - 1], (lane - n) & 63, 64);  // (row -1: only of coarse row 0)
        coarse_restrict<C, NP>(v, rR, rB, below, p);
        if constexpr (n == 4) {
            // 2 x 2 cells: one unknown, four zero neighbours, solved in double.  (The
            // cycle has to end exactly: four over-relaxed sweeps on the 8-cell level
            // in place of the levels below it take 1.2 us less a launch of two cycles, but
            // where k2 is close to 0 they leave 0.7 of the worst error and a cycle
            // then gains 8 instead of 30.)
            const double f2 = (double)__shfl(v[0], 4 + 2, 64), H = 2.0 * h;
            if (lane == 0) lds.E[coarse_off_E(2) + 4] = (C)(-f2 / (4.0 / (H * H) + k2_two));
            wave_sync();
        } else {
            if (!p && g < G)
#pragma unroll
                for (int m = 0; m < NP; ++m) {
                    const int J = g * (L::ROWS / 2) + m;
                    lds.F[coarse_off_F(nc) + J * nc + x / 2] = x > 0 && J > 0 ? v[m] : C(0);
                }
            wave_sync();
            const CoarseWave<C, nc, HELM> lc(lds, 2.0 * h, omega, h2max);
            constexpr int NC = CoarseLevel<nc>::NP;
            C cR[NC], cB[NC], gR[NC], gB[NC];
#pragma unroll
            for (int m = 0; m < NC; ++m) cR[m] = cB[m] = C(0);
            lc.load_f(gR, gB);
            lc.cycle(cR, cB, gR, gB, nu1, nu2, omega, h2max, k2_two);
            lc.store_E(cR, cB);
            wave_sync();
        }
        coarse_prolong<C, NP>(uR, uB, lds.E + coarse_off_E(nc), nc + 1, x, min(g, G - 1) * (L::ROWS / 2), p);
        if (g >= G)
#pragma unroll
            for (int m = 0; m < NP; ++m) uR[m] = uB[m] = C(0);
        smooth(uR, uB, fR, fB, nu2);
    }
};

// n0: cells a side of the top level.  E is the type of the arrays in memory, C
// that of the sweeps: float where the result only corrects a finer FP64 level
// (whose residual and smoothing set the fixed point), double elsewhere.
template <typename E, typename C, bool HELM, int n0>
__global__ __launch_bounds__(coarse_threads<n0>()) void k_mg_coarse(CoarseArgs<E> a) {
    constexpr int ROWS = coarse_rows<n0>(), NP = ROWS / 2, NT = coarse_threads<n0>();
    __shared__ CoarseLds<C> lds;
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x = n0 == 64 ? lane : lane & (n0 - 1), g = n0 == 64 ? w : lane / n0;
    const bool p = lane & 1, live = n0 >= 16 || g < CoarseLevel<n0 == 64 ? 32 : n0>::G;
    const C h2 = (C)(a.h * a.h), ih2 = (C)(1.0 / (a.h * a.h));
    const C om = (C)(a.h * a.h > a.h2max ? 1.0 : a.omega);
    // the top level's nodes (row y of entry m): every load unconditional, from
    // clamped indices, and masked after
    C uR[NP], uB[NP], fR[NP], fB[NP], iR[NP], iB[NP], dR[NP], dB[NP];
    const bool has_u = a.u_init[r] != nullptr;
    const E* ui = has_u ? a.u_init[r] : a.f[r];
    const C* top_D = coarse_tab<C>(a.tab.D, a.tab.Df);
    const C* top_id = coarse_tab<C>(a.tab.id, a.tab.idf);
    const auto load = [&](int m, int colour, C& u, C& f, C& id, C& D) {
        const int y = min(g * ROWS + 2 * m + ((p ? 1 : 0) ^ colour), n0 - 1);
        const size_t i = (size_t)y * a.pitch + x;
        const bool in = live && x > 0 && y > 0;
        u = (C)ui[i] * C(in && has_u ? 1 : 0);
        f = (C)a.f[r][i] * C(in ? 1 : 0);
        if (HELM) {
            const int k = y * (n0 + 1) + x;
            id = top_id[k] * C(in ? 1 : 0);
            D = top_D[k];
        } else {
            id = in ? C(0.25) : C(0);
            D = C(4);
        }
    };
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        load(m, 0, uR[m], fR[m], iR[m], dR[m]);
        load(m, 1, uB[m], fB[m], iB[m], dB[m]);
    }
    // 1/D and D of the levels in one wavefront, in their lane layout
    {
        constexpr int T0 = n0 == 64 ? 0 : coarse_off_T(n0), IT = (kCoarseT - T0) / NT;
        static_assert((kCoarseT - T0) % NT == 0, "whole trips");
        const C* tid_ = coarse_tab<C>(a.tab.Tid, a.tab.Tidf) + T0;
        const C* tD = coarse_tab<C>(a.tab.TD, a.tab.TDf) + T0;
        C vi[IT], vD[IT];
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const int i = tid + q * NT;
            if (HELM) {
                vi[q] = tid_[i];
                vD[q] = tD[i];
            } else {
                vi[q] = C(coarse_slot(T0 + i).in ? 0.25 : 0.0);
                vD[q] = C(4);
            }
        }
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            lds.id[T0 + tid + q * NT] = vi[q];
            lds.D[T0 + tid + q * NT] = vD[q];
        }
    }
    const double k2_two = HELM ? a.tab.TD[kCoarseT] : 0.0;  // node (1, 1) of the 2-cell level
    for (int i = tid; i < coarse_off_E(1); i += NT) lds.E[i] = C(0);
    if constexpr (n0 == 64)
        for (int i = tid; i < 2 * 64; i += NT)  // past the first and last wavefront
            lds.edge[i >> 6][0][i & 63] = lds.edge[i >> 6][kCoarseWaves + 1][i & 63] = C(0);
    if constexpr (n0 == 64) __syncthreads();
    else wave_sync();

    int buf = 0;
    // the row across the boundary to the next wavefront (64^2) or group
    const auto edge = [&](const C (&o)[NP], bool q) -> C {
        if constexpr (n0 == 64) {
            lds.edge[buf][w + 1][lane] = q ? o[0] : o[NP - 1];
            __syncthreads();
            const C e = lds.edge[buf][q ? w + 2 : w][lane];
            buf ^= 1;
            return e;
        } else {
            const C t = q ? o[0] : o[NP - 1];
            const C e = __shfl(t, (q ? lane + n0 : lane - n0) & 63, 64);
            return q && g == CoarseLevel<n0>::G - 1 ? C(0) : e;
        }
    };
    const auto residual = [&](C (&rR)[NP], C (&rB)[NP]) {
        const bool in = x > 0 && live;
        coarse_resid<C, NP>(rR, uR, fR, dR, uB, edge(uB, p), p, ih2, in, in && (g > 0 || p));
        coarse_resid<C, NP>(rB, uB, fB, dB, uR, edge(uR, !p), !p, ih2, in, in && (g > 0 || !p));
    };
    const auto norms = [&](int slot) {
        C rR[NP], rB[NP];
        residual(rR, rB);
        double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            s[0] += (double)rR[m] * rR[m] + (double)rB[m] * rB[m];
            s[1] += (double)fR[m] * fR[m] + (double)fB[m] * fB[m];
            s[2] += (double)uR[m] * uR[m] + (double)uB[m] * uB[m];
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
            for (int q = 0; q < 3; ++q) s[q] += __shfl_xor(s[q], d, 64);
        if constexpr (n0 == 64) {
            if (lane == 0)
#pragma unroll
                for (int q = 0; q < 3; ++q) lds.red[w][q] = s[q];
            __syncthreads();
            if (tid < 3) {
                double t = 0.0;
                for (int k = 0; k < kCoarseWaves; ++k) t += lds.red[k][tid];
                a.norm_part[slot * a.norm_stride + 3 * r + tid] = t;
            }
        } else if (lane < 3) {
            a.norm_part[slot * a.norm_stride + 3 * r + lane] = lane == 0 ? s[0] : lane == 1 ? s[1] : s[2];
        }
    };
    const auto smooth = [&](int nu) {
        for (int k = 0; k < nu; ++k) {
            coarse_half<C, NP>(uR, fR, iR, uB, edge(uB, p), p, h2, om);
            coarse_half<C, NP>(uB, fB, iB, uR, edge(uR, !p), !p, h2, om);
        }
    };
    for (int cyc = 0; cyc < a.ncycles; ++cyc) {
        if (a.norm_part) norms(cyc);
        for (int k = 0; k < a.inner; ++k) {
            if constexpr (n0 < 64) {
                const CoarseWave<C, n0, false> top(lds, a.h, a.omega, a.h2max);
                top.cycle(uR, uB, fR, fB, a.nu1, a.nu2, a.omega, a.h2max, k2_two);
            } else {
                smooth(a.nu1);
                C rR[NP], rB[NP], t[NP], v[NP];
                residual(rR, rB);
#pragma unroll
                for (int m = 0; m < NP; ++m) t[m] = p ? rR[m] : rB[m];
                const C below = edge(t, false);  // row -1 of the first wavefront: 0
                coarse_restrict<C, NP>(v, rR, rB, below, p);
                if (!p)
#pragma unroll
                    for (int m = 0; m < NP; ++m) {
                        const int J = w * NP + m;
                        lds.F[J * 32 + x / 2] = x > 0 && J > 0 ? v[m] : C(0);
                    }
                __syncthreads();
                if (w == 0) {
                    const CoarseWave<C, 32, HELM> lc(lds, 2.0 * a.h, a.omega, a.h2max);
                    constexpr int NC = CoarseLevel<32>::NP;
                    C cR[NC], cB[NC], gR[NC], gB[NC];
#pragma unroll
                    for (int m = 0; m < NC; ++m) cR[m] = cB[m] = C(0);
                    lc.load_f(gR, gB);
                    lc.cycle(cR, cB, gR, gB, a.nu1, a.nu2, a.omega, a.h2max, k2_two);
                    lc.store_E(cR, cB);
                }
                __syncthreads();
                coarse_prolong<C, NP>(uR, uB, lds.E, 33, x, w * NP, p);
                smooth(a.nu2);
            }
        }
    }
    if (a.norm_part) norms(a.ncycles);
    if (live)
#pragma unroll
        for (int m = 0; m < NP; ++m) {
            const int y = g * ROWS + 2 * m;
            a.u_out[r][(size_t)(y + (p ? 1 : 0)) * a.pitch + x] = (E)uR[m];
            a.u_out[r][(size_t)(y + (p ? 0 : 1)) * a.pitch + x] = (E)uB[m];
        }
}

// Exact solve of the Poisson problem on the 64^2 coarse level (u = 0 on the
// boundary).  The 2-D sine transform diagonalises the 5-point operator of
// eq. (33): with S_jk = sin(pi (j+1)(k+1) / 64) (S S = 32 I) and the
// eigenvalues lambda_kl = -(4/H^2) (sin^2(pi (k+1)/128) + sin^2(pi (l+1)/128)),
// u = S (M o (S f S)) S with M = 1 / (32^2 lambda).  The four products run on
// fp32 MFMA (v_mfma_f32_16x16x4_f32), 16 wavefronts with one 16 x 16 output
// tile each; the 63 interior rows and columns are padded to 64 with zeros.
// Like the V-cycle coarse kernel below a finer level, the coarse correction
// is computed in float.
constexpr int kDstN = 64;
constexpr int kDstLd = 68;  // LDS row stride of the 64 x 64 matrices
typedef float dst_v4f __attribute__((ext_vector_type(4)));

template <typename E>
struct DstArgs {
    int pitch;
    const E* f[2];
    E* u_out[2];
    const float* S;
    const float* M;
};

// D = A B for 64 x 64 matrices in LDS: A row-major, B given transposed (Bt[j][k]
// = B[k][j]).  Wavefront w computes the tile rows 16 (w / 4) .., columns
// 16 (w % 4) ..; lane l feeds A[i0 + l % 16][4 s + l / 16] and
// Bt[j0 + l % 16][4 s + l / 16] at step s and holds D[i0 + 4 (l / 16) + q][j0 + l % 16].
__device__ __forceinline__ dst_v4f dst_tile(const float* A, const float* Bt) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i0 = 16 * (w >> 2), j0 = 16 * (w & 3);
    const float* a = A + (i0 + (lane & 15)) * kDstLd + (lane >> 4);
    const float* b = Bt + (j0 + (lane & 15)) * kDstLd + (lane >> 4);
    dst_v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kDstN / 4; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[4 * s], b[4 * s], acc, 0, 0, 0);
    return acc;
}

template <typename E>
__global__ __launch_bounds__(1024) void k_coarse_dst(DstArgs<E> a) {
    __shared__ float sS[kDstN * kDstLd];
    __shared__ float sX[kDstN * kDstLd];
    __shared__ float sY[kDstN * kDstLd];
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int i0 = 16 * (w >> 2), j0 = 16 * (w & 3);
    const int ti = i0 + 4 * (lane >> 4), tj = j0 + (lane & 15);  // this lane's outputs: rows ti + q, column tj
    float mv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) mv[q] = a.M[(ti + q) * kDstN + tj];
    // S (symmetric, so also S^T) and f^T: sX[x][y] = f(node y + 1, x + 1); every
    // load is issued before the first store, so their latencies overlap
    {
        constexpr int kIt = kDstN * kDstN / 1024;
        float sv[kIt], fv[kIt];
#pragma unroll
        for (int t = 0; t < kIt; ++t) {
            const int i = tid + t * 1024, y = i >> 6, x = i & 63;
            sv[t] = a.S[i];
            fv[t] = (x < kDstN - 1 && y < kDstN - 1) ? (float)a.f[r][(size_t)(y + 1) * a.pitch + x + 1]
                                                     : 0.f;
        }
#pragma unroll
        for (int t = 0; t < kIt; ++t) {
            const int i = tid + t * 1024, y = i >> 6, x = i & 63;
            sS[y * kDstLd + x] = sv[t];
            sX[x * kDstLd + y] = fv[t];
        }
    }
    __syncthreads();
    dst_v4f d = dst_tile(sS, sX);  // Y = S F
#pragma unroll
    for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd + tj] = d[q];
    __syncthreads();
    d = dst_tile(sY, sS);  // X = M o (Y S), stored transposed for the next product
    __syncthreads();       // every read of the operands is done before sX is rewritten
#pragma unroll
    for (int q = 0; q < 4; ++q) sX[tj * kDstLd + ti + q] = mv[q] * d[q];
    __syncthreads();
    d = dst_tile(sS, sX);  // Y = S X
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd + tj] = d[q];
    __syncthreads();
    d = dst_tile(sY, sS);  // U = Y S
#pragma unroll
    for (int q = 0; q < 4; ++q) sX[(ti + q) * kDstLd + tj] = d[q];
    __syncthreads();
    for (int i = tid; i < (kDstN + 1) * (kDstN + 1); i += 1024) {
        const int y = i / (kDstN + 1), x = i - y * (kDstN + 1);
        const bool in = x >= 1 && x <= kDstN - 1 && y >= 1 && y <= kDstN - 1;
        a.u_out[r][(size_t)y * a.pitch + x] = (E)(in ? sX[(y - 1) * kDstLd + x - 1] : 0.f);
    }
}

// FP64 form of the exact 64^2 coarse Poisson solve, for the mixed form, whose
// coarsest-grid solve stays in FP64 while its V-cycle levels run in FP32.
// The products run on FP64 MFMA (v_mfma_f64_16x16x4_f64: one 16 x 16 output
// tile per wavefront, lane l feeding A[i0 + l % 16][4 s + l / 16] and
// Bt[j0 + l % 16][4 s + l / 16] and holding D[i0 + 4 (l / 16) + q][j0 + l % 16],
// the layout of the FP32 instruction).  Plain FP64 fused multiply-adds from LDS
// were LDS-bound here: a wavefront's read of one shared row element costs a
// full LDS pass.
typedef double dst_v4d __attribute__((ext_vector_type(4)));
constexpr int kDstLd64 = kDstN + 4;  // LDS row stride (doubles) of the 64 x 64 operands

// 16 x 16 tile (rows 0..15 of A, columns j0.. of B) of A B for an inner
// dimension n: A row-major with stride LDA, B given transposed (Bt[j][k] =
// B[k][j]) with stride LDB.
template <int n, int LDA, int LDB>
__device__ __forceinline__ dst_v4d tile64(const double* A, const double* Bt, int j0) {
    const int lane = threadIdx.x & 63;
    const double* pa = A + (lane & 15) * LDA + (lane >> 4);
    const double* pb = Bt + (j0 + (lane & 15)) * LDB + (lane >> 4);
    dst_v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int s = 0; s < n / 4; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[4 * s], pb[4 * s], acc, 0, 0, 0);
    return acc;
}

// The 64^2 exact solve in FP64 (grids of 128^2): one workgroup of 16
// wavefronts per right-hand side, u = S (M o (S F S)) S as four products in
// LDS, as in k_coarse_dst.
template <typename E>
struct DstArgs64 {
    int pitch;
    const E* f[2];
    E* u_out[2];
    const double* S;
    const double* M;
};

template <typename E>
__global__ __launch_bounds__(1024) void k_coarse_dst64(DstArgs64<E> a) {
    __shared__ double sS[kDstN * kDstLd64];
    __shared__ double sX[kDstN * kDstLd64];
    __shared__ double sY[kDstN * kDstLd64];
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int i0 = 16 * (w >> 2), j0 = 16 * (w & 3);
    const int ti = i0 + 4 * (lane >> 4), tj = j0 + (lane & 15);
    double mv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) mv[q] = a.M[(ti + q) * kDstN + tj];
    constexpr int kIt = kDstN * kDstN / 1024;
    {   // S and F^T: sX[x][y] = f(node y + 1, x + 1); unconditional loads first
        double sv[kIt], fv[kIt];
#pragma unroll
        for (int t = 0; t < kIt; ++t) {
            const int i = tid + t * 1024, y = i >> 6, x = i & (kDstN - 1);
            const bool in = x < kDstN - 1 && y < kDstN - 1;
            sv[t] = a.S[i];
            const double v = (double)a.f[r][in ? (size_t)(y + 1) * a.pitch + x + 1 : 0];
            fv[t] = in ? v : 0.0;
        }
#pragma unroll
        for (int t = 0; t < kIt; ++t) {
            const int i = tid + t * 1024, y = i >> 6, x = i & (kDstN - 1);
            sS[y * kDstLd64 + x] = sv[t];
            sX[x * kDstLd64 + y] = fv[t];
        }
    }
    __syncthreads();
    dst_v4d d = tile64<kDstN, kDstLd64, kDstLd64>(sS + i0 * kDstLd64, sX, j0);  // Y = S F
#pragma unroll
    for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd64 + tj] = d[q];
    __syncthreads();
    d = tile64<kDstN, kDstLd64, kDstLd64>(sY + i0 * kDstLd64, sS, j0);  // X = M o (Y S), stored transposed
    __syncthreads();  // every read of the operands is done before sX is rewritten
#pragma unroll
    for (int q = 0; q < 4; ++q) sX[tj * kDstLd64 + ti + q] = mv[q] * d[q];
    __syncthreads();
    d = tile64<kDstN, kDstLd64, kDstLd64>(sS + i0 * kDstLd64, sX, j0);  // Y = S X
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd64 + tj] = d[q];
    __syncthreads();
    d = tile64<kDstN, kDstLd64, kDstLd64>(sY + i0 * kDstLd64, sS, j0);  // U = Y S
#pragma unroll
    for (int q = 0; q < 4; ++q) sX[(ti + q) * kDstLd64 + tj] = d[q];
    __syncthreads();
    for (int i = tid; i < (kDstN + 1) * (kDstN + 1); i += 1024) {
        const int y = i / (kDstN + 1), x = i - y * (kDstN + 1);
        const bool in = x >= 1 && x <= kDstN - 1 && y >= 1 && y <= kDstN - 1;
        a.u_out[r][(size_t)y * a.pitch + x] = (E)(in ? sX[(y - 1) * kDstLd64 + x - 1] : 0.0);
    }
}

// Whole Poisson solves on grids of n^2 <= 64^2 in one workgroup per right-hand
// side: `iters` iterations u += L_h^-1 (f - L_h u), the exact solve by the four
// products of k_coarse_dst64 (the tables of a smaller grid are padded with
// zeros), and the norms of every iterate.  A thread keeps f and u of the four
// nodes of its product tile in registers; u's neighbours come through LDS.
// Bound by the chain of four products and two residuals of one workgroup: 21 us
// for one iteration (what a slice's guess needs) where 5 V-cycles took 58; 16 of
// these solves in 8 slices at 64^2: 2.83 -> 1.82 ms.
struct Poisson64Args {
    int n, pitch;
    double ih2;
    const double* f[2];
    double* u[2];
    const double* S;
    const double* M;
    int iters;
    double* norm_part;  // the sums of r^2, f^2, u^2 before each iteration and after the last
    size_t norm_stride;
};

__global__ __launch_bounds__(1024) void k_poisson64(Poisson64Args a) {
    __shared__ double sS[kDstN * kDstLd64];
    __shared__ double sX[kDstN * kDstLd64];
    __shared__ double sY[kDstN * kDstLd64];
    __shared__ double red[16][3];
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int i0 = 16 * (w >> 2), j0 = 16 * (w & 3);
    const int ti = i0 + 4 * (lane >> 4), tj = j0 + (lane & 15);  // node (x, y) = (tj + 1, ti + q + 1)
    const int last = a.n - 2;                                    // the last interior index
    double mv[4], f[4], u[4];
    {
        double sv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = tj <= last && ti + q <= last;
            const size_t g = in ? (size_t)(ti + q + 1) * a.pitch + tj + 1 : 0;
            mv[q] = a.M[(ti + q) * kDstN + tj];
            sv[q] = a.S[tid + q * 1024];
            f[q] = a.f[r][g] * (in ? 1.0 : 0.0);
            u[q] = a.u[r][g] * (in ? 1.0 : 0.0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = tid + q * 1024;
            sS[(i >> 6) * kDstLd64 + (i & 63)] = sv[q];
        }
    }
    for (int it = 0;; ++it) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd64 + tj] = u[q];
        __syncthreads();
        double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int y = ti + q, i = y * kDstLd64 + tj;
            const bool in = tj <= last && y <= last;
            const double l = tj > 0 ? sY[i - 1] : 0.0, h = tj < last ? sY[i + 1] : 0.0;
            const double d = y > 0 ? sY[i - kDstLd64] : 0.0, t = y < last ? sY[i + kDstLd64] : 0.0;
            const double v = in ? f[q] - (l + h + d + t - 4.0 * u[q]) * a.ih2 : 0.0;
            sX[tj * kDstLd64 + y] = v;
            s[0] += v * v;
            s[1] += f[q] * f[q];
            s[2] += u[q] * u[q];
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
            for (int q = 0; q < 3; ++q) s[q] += __shfl_xor(s[q], d, 64);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < 3; ++q) red[w][q] = s[q];
        __syncthreads();
        if (tid < 3) {
            double t = 0.0;
            for (int k = 0; k < 16; ++k) t += red[k][tid];
            a.norm_part[it * a.norm_stride + 3 * r + tid] = t;
        }
        if (it == a.iters) break;
        dst_v4d d = tile64<kDstN, kDstLd64, kDstLd64>(sS + i0 * kDstLd64, sX, j0);  // Y = S F
#pragma unroll
        for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd64 + tj] = d[q];
        __syncthreads();
        d = tile64<kDstN, kDstLd64, kDstLd64>(sY + i0 * kDstLd64, sS, j0);  // X = M o (Y S), stored transposed
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) sX[tj * kDstLd64 + ti + q] = mv[q] * d[q];
        __syncthreads();
        d = tile64<kDstN, kDstLd64, kDstLd64>(sS + i0 * kDstLd64, sX, j0);  // Y = S X
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) sY[(ti + q) * kDstLd64 + tj] = d[q];
        __syncthreads();
        d = tile64<kDstN, kDstLd64, kDstLd64>(sY + i0 * kDstLd64, sS, j0);  // U = Y S
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] += d[q];
        __syncthreads();  // every read of sY and red is done before they are rewritten
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (tj <= last && ti + q <= last) a.u[r][(size_t)(ti + q + 1) * a.pitch + tj + 1] = u[q];
}

// Tables of the exact coarse Poisson solve on an n^2 level of spacing H:
// S_jk = sin(pi (j+1)(k+1) / n) (the argument reduced exactly modulo 2 pi),
// M_jk = 1 / ((n/2)^2 lambda_jk), lambda_jk = -(4/H^2)(sin^2(pi (j+1)/2n) +
// sin^2(pi (k+1)/2n)), the eigenvalue of the 5-point operator for the sine
// mode (j+1, k+1); the rows and columns from n-1 on are zero (n <= 64 = the
// tables' stride).  Float and (when S64 is set) double copies.
__global__ void k_dst_tables(int n, double H, float* S, float* M, double* S64, double* M64) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kDstN * kDstN) return;
    const int jj = i / kDstN, kk = i - jj * kDstN;
    const bool in = jj < n - 1 && kk < n - 1;
    const double pi = 3.14159265358979323846;
    double sv = 0.0, mv = 0.0;
    if (in) {
        const int m = ((jj + 1) * (kk + 1)) % (2 * n);
        sv = sin(pi * (double)m / (double)n);
        const double sj = sin(pi * (jj + 1) / (2.0 * n));
        const double sk = sin(pi * (kk + 1) / (2.0 * n));
        const double lambda = -(4.0 / (H * H)) * (sj * sj + sk * sk);
        mv = 1.0 / ((n / 2.0) * (n / 2.0) * lambda);
    }
    S[i] = (float)sv;
    M[i] = (float)mv;
    if (S64) {
        S64[i] = sv;
        M64[i] = mv;
    }
}

// The coarse kernel's tables from k2 on its top level (N <= 64, pitched), the
// coarser levels by full weighting: D = 4 + h^2 k2 and 1/D on the top level
// (dense [N+1]^2) and, in their lane layout, on the levels of at most 32 cells
// (T; entry kCoarseT of TD: k2 at the one node of the 2-cell level).  One block.
constexpr int kK2Threads = 1024;
__global__ __launch_bounds__(kK2Threads) void k_coarse_k2(int N, int pitch, double h,
                                                          const double* __restrict__ k2top,
                                                          CoarseTabs t) {
    // every level in LDS: the top level's loads in batches of kB per thread,
    // the restrictions from LDS, the three outputs written once
    __shared__ double sk[65 * 65 + coarse_off_E(1)];
    constexpr int kB = 8;
    const int tid = threadIdx.x;
    const int nt = (N + 1) * (N + 1);
    for (int base = 0; base < nt; base += kB * kK2Threads) {
        double v[kB];
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const int i = base + b * kK2Threads + tid;
            const int y = i / (N + 1), x = i - y * (N + 1);
            const bool ok = i < nt && x != 0 && y != 0 && x != N && y != N;
            v[b] = ok ? k2top[(size_t)y * pitch + x] : 0.0;
        }
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const int i = base + b * kK2Threads + tid;
            if (i < nt) sk[i] = v[b];
        }
    }
    __syncthreads();
    int off = 0;
    for (int nf = N; nf > 2; nf /= 2) {
        const int nc = nf / 2, w = nf + 1;
        const double* kf = sk + off;
        double* kc = sk + off + (nf + 1) * (nf + 1);
        for (int i = tid; i < (nc + 1) * (nc + 1); i += kK2Threads) {
            const int J = i / (nc + 1), I = i - J * (nc + 1);
            double v = 0.0;
            if (I >= 1 && J >= 1 && I <= nc - 1 && J <= nc - 1) {
                const int c = (2 * J) * w + 2 * I;
                v = (4.0 * kf[c] + 2.0 * (kf[c - 1] + kf[c + 1] + kf[c - w] + kf[c + w]) +
                     (kf[c - w - 1] + kf[c - w + 1] + kf[c + w - 1] + kf[c + w + 1])) *
                    (1.0 / 16.0);
            }
            kc[i] = v;
        }
        __syncthreads();
        off += (nf + 1) * (nf + 1);
    }
    const auto put = [](double k2, double h2, double in, double& D, double& id, float& Df, float& idf) {
        const double Dd = fmad(h2, k2, 4.0);
        const float Ds = 4.f + (float)h2 * (float)k2;
        D = Dd;
        id = in / Dd;
        Df = Ds;
        idf = (float)in / Ds;
    };
    for (int i = tid; i < (N + 1) * (N + 1); i += kK2Threads)
        put(sk[i], h * h, 1.0, t.D[i], t.id[i], t.Df[i], t.idf[i]);
    for (int i = tid; i < kCoarseT; i += kK2Threads) {
        const CoarseSlot c = coarse_slot(i);
        if (c.n > N) continue;  // a level above the top one
        int o = 0;
        for (int n = N; n > c.n; n /= 2) o += (n + 1) * (n + 1);
        const double hl = h * (double)(N / c.n);
        put(sk[o + min(c.y, c.n) * (c.n + 1) + c.x], hl * hl, c.in ? 1.0 : 0.0, t.TD[i], t.Tid[i],
            t.TDf[i], t.Tidf[i]);
    }
    if (tid == 0) t.TD[kCoarseT] = sk[off + 4];  // off: the 2-cell level
}

// Residual norms of the current iterate, one partial sum per interior row and
// right-hand side (one wavefront a row, four rows a workgroup; blockIdx.y the
// right-hand side).  With r_out set (mixed form), the FP64 residual is also
// stored, rounded to float, as the right-hand side of the FP32 error equation
// (boundary 0).  HBM-bound on the large grids: the loads of four node pairs a
// lane are in flight together (one node a thread and trip, a branch around
// each, measured 10.9 us for two right-hand sides at 512^2).
template <bool HELM>
__global__ __launch_bounds__(kThreads) void k_resnorm(int N, double ih2, int pitch, const double* u0,
                                                      const double* u1, const double* f0,
                                                      const double* f1, const double* k2,
                                                      double* part, int nblk, float* r0, float* r1) {
    constexpr int CH = 4;
    int bx, r;
    tile_of_block(bx, r);
    const int lane = threadIdx.x & 63, row = bx * (kThreads / 64) + (threadIdx.x >> 6) + 1;
    if (row > N - 1) return;
    const size_t g0 = (size_t)row * pitch;
    const double* u = (r ? u1 : u0) + g0;
    const double* f = (r ? f1 : f0) + g0;
    float* ro = r ? r1 : r0;
    double s[3] = {0.0, 0.0, 0.0};
    for (int m0 = 0; m0 < N / 2; m0 += 64 * CH) {
        double2 c[CH], up[CH], dn[CH], fv[CH], kv[CH];
        double lf[CH], rt[CH];
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int j = 2 * min(m0 + lane + 64 * q, N / 2 - 1);
            c[q] = *reinterpret_cast<const double2*>(u + j);
            up[q] = *reinterpret_cast<const double2*>(u + j - pitch);
            dn[q] = *reinterpret_cast<const double2*>(u + j + pitch);
            fv[q] = *reinterpret_cast<const double2*>(f + j);
            if (HELM) kv[q] = *reinterpret_cast<const double2*>(k2 + g0 + j);
            lf[q] = u[max(j - 1, 0)];
            rt[q] = u[j + 2];
        }
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int j = 2 * (m0 + lane + 64 * q);
            if (j >= N) continue;
            const bool in = j > 0;  // node 0 is a boundary node
            double a0 = (lf[q] + c[q].y + up[q].x + dn[q].x - 4.0 * c[q].x) * ih2;
            double a1 = (c[q].x + rt[q] + up[q].y + dn[q].y - 4.0 * c[q].y) * ih2;
            if (HELM) {
                a0 -= kv[q].x * c[q].x;
                a1 -= kv[q].y * c[q].y;
            }
            const double v0 = in ? fv[q].x - a0 : 0.0, v1 = fv[q].y - a1;
            const double w = in ? 1.0 : 0.0;
            s[0] += v0 * v0 + v1 * v1;
            s[1] += w * fv[q].x * fv[q].x + fv[q].y * fv[q].y;
            s[2] += w * c[q].x * c[q].x + c[q].y * c[q].y;
            if (ro) *reinterpret_cast<float2*>(ro + g0 + j) = float2{(float)v0, (float)v1};
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
        for (int q = 0; q < 3; ++q) s[q] += __shfl_xor(s[q], d, 64);
    if (lane < 3)
        part[(size_t)(3 * r + lane) * nblk + row - 1] = lane == 0 ? s[0] : lane == 1 ? s[1] : s[2];
}

// The norms of a batch of V-cycles to the host: one workgroup per slot and
// sum adds the slot's per-tile partials (in a fixed order) and writes the sum
// into the host's coherent pinned array dst; the last workgroup to finish
// (device-scope counter, which it resets) then copies the flags word and
// publishes the sequence number with a system-scope release, after which the
// host reads the sums.  Slot up_slot has nblk_up tiles, the slots in
// [fuse_lo, fuse_hi) nblk_fuse (fused passes), the others nblk.
__global__ __launch_bounds__(kThreads) void k_reduce_publish(
    const double* part, int stride, int nblk, int s0, int nvec, int up_slot, int nblk_up,
    int fuse_lo, int fuse_hi, int nblk_fuse, double* dst, const int32_t* __restrict__ flags,
    int32_t* dst_flags, uint32_t* dst_seq, uint32_t seq, uint32_t* count) {
    __shared__ double red[kThreads / 64];
    const int s = s0 + blockIdx.x / nvec, k = blockIdx.x % nvec;
    if (s == up_slot) nblk = nblk_up;
    if (s >= fuse_lo && s < fuse_hi) nblk = nblk_fuse;  // written by fused up-and-down passes
    const double* p = part + (size_t)s * stride + (size_t)k * nblk;
    double acc[1] = {0.0};
    for (int b = threadIdx.x; b < nblk; b += kThreads) acc[0] += p[b];
    block_sum<1, kThreads>(acc, red);
    if (threadIdx.x == 0) {
        dst[s * kNormVec + k] = acc[0];
        __threadfence_system();
        if (atomicAdd(count, 1u) == gridDim.x - 1) {
            *count = 0;
            *dst_flags = *flags;
            __threadfence_system();
            __hip_atomic_store(dst_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Full weighting of a fine node array onto the interior coarse nodes (boundary 0).
__global__ void k_restrict_fw(const double* fine, int pf, double* coarse, int pc, int Nc) {
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    const int J = blockIdx.y;
    if (I > Nc) return;
    double v = 0.0;
    if (I >= 1 && J >= 1 && I <= Nc - 1 && J <= Nc - 1) {
        const size_t c = (size_t)(2 * J) * pf + 2 * I;
        v = (4.0 * fine[c] + 2.0 * (fine[c - 1] + fine[c + 1] + fine[c - pf] + fine[c + pf]) +
             (fine[c - pf - 1] + fine[c - pf + 1] + fine[c + pf - 1] + fine[c + pf + 1])) *
            (1.0 / 16.0);
    }
    coarse[(size_t)J * pc + I] = v;
}

// Full weighting over LC levels in one launch (the same sums, level by level, as
// k_restrict_fw).  A workgroup owns kChainB^2 nodes of the last level and what
// lies above them; it loads the fine nodes that those depend on, (2^LC (kChainB +
// 1) - 1)^2, and keeps every level in LDS.  Launches of their own took 4.1 us a
// level, 8.8 us at 256^2 and 16.4 at 1024^2; now 4.0 and 6.7.
constexpr int kChainB = 4, kChainMax = 4;
template <int LC>
constexpr int chain_threads() { return LC >= 3 ? 1024 : 256; }
struct ChainArgs {
    const double* fine;
    int N, pitch;
    double* coarse[kChainMax];
    int pc[kChainMax];
};
template <int LC>
constexpr int chain_edge(int l) { return (1 << (LC - l)) * (kChainB + 1) - 1; }
template <int LC>
constexpr int chain_off(int l) {
    int o = 0;
    for (int k = 0; k < l; ++k) o += chain_edge<LC>(k) * chain_edge<LC>(k);
    return o;
}
template <int LC>
__global__ __launch_bounds__(chain_threads<LC>()) void k_restrict_chain(ChainArgs a) {
    constexpr int NT = chain_threads<LC>();
    __shared__ double v[chain_off<LC>(LC)];
    const int I0 = blockIdx.x * kChainB, J0 = blockIdx.y * kChainB;
    {
        constexpr int m = chain_edge<LC>(0), s = 1 << LC;
        const int x0 = s * I0 - (s - 1), y0 = s * J0 - (s - 1);
        constexpr int IT = (m * m + NT - 1) / NT;  // loads all in flight together
        double t[IT];
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const int i = min((int)threadIdx.x + q * NT, m * m - 1);
            const int y = y0 + i / m, x = x0 + i % m;
            const bool in = x >= 0 && x <= a.N && y >= 0 && y <= a.N;
            t[q] = a.fine[(size_t)min(max(y, 0), a.N) * a.pitch + min(max(x, 0), a.N)] * (in ? 1.0 : 0.0);
        }
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const int i = threadIdx.x + q * NT;
            if (i < m * m) v[i] = t[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int l = 1; l <= LC; ++l) {
        const int m = chain_edge<LC>(l), mf = chain_edge<LC>(l - 1), s = 1 << (LC - l), n = a.N >> l;
        const double* f = v + chain_off<LC>(l - 1);
        for (int i = threadIdx.x; i < m * m; i += NT) {
            const int j = i / m, k = i - j * m;
            const int I = s * I0 - (s - 1) + k, J = s * J0 - (s - 1) + j;
            double t = 0.0;
            if (I >= 1 && J >= 1 && I <= n - 1 && J <= n - 1) {
                const int c = (2 * j + 1) * mf + 2 * k + 1;
                t = (4.0 * f[c] + 2.0 * (f[c - 1] + f[c + 1] + f[c - mf] + f[c + mf]) +
                     (f[c - mf - 1] + f[c - mf + 1] + f[c + mf - 1] + f[c + mf + 1])) *
                    (1.0 / 16.0);
            }
            if (l < LC) v[chain_off<LC>(l) + i] = t;
            if (k >= s - 1 && j >= s - 1 && k < s * (kChainB + 1) - 1 && j < s * (kChainB + 1) - 1 &&
                I <= n && J <= n)
                a.coarse[l - 1][(size_t)J * a.pc[l - 1] + I] = t;
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------- dispatch --

template <typename E, int R, bool HELM, int T>
void launch_down_t(const DownArgs<E>& a, int nu, dim3 grid, hipStream_t s, const ProfScope& ps) {
    constexpr int NT = tile_threads<T>();
    switch (nu) {
        case 1: WQ_KLAUNCH(ps, (k_mg_down<E, R, HELM, 1, T>), grid, dim3(NT), 0, s, a); break;
        case 2: WQ_KLAUNCH(ps, (k_mg_down<E, R, HELM, 2, T>), grid, dim3(NT), 0, s, a); break;
        default: WQ_KLAUNCH(ps, (k_mg_down<E, R, HELM, 3, T>), grid, dim3(NT), 0, s, a); break;
    }
}

template <typename E, int R, bool HELM, int T>
void launch_up_t(const UpArgs<E>& a, int nu, dim3 grid, hipStream_t s, const ProfScope& ps) {
    constexpr int NT = tile_threads<T>();
    switch (nu) {
        case 1: WQ_KLAUNCH(ps, (k_mg_up<E, R, HELM, 1, T>), grid, dim3(NT), 0, s, a); break;
        case 2: WQ_KLAUNCH(ps, (k_mg_up<E, R, HELM, 2, T>), grid, dim3(NT), 0, s, a); break;
        default: WQ_KLAUNCH(ps, (k_mg_up<E, R, HELM, 3, T>), grid, dim3(NT), 0, s, a); break;
    }
}

template <typename E, int R, bool HELM>
void launch_down(const DownArgs<E>& a, int nu, dim3 grid, hipStream_t s, const ProfScope& ps, int T) {
    if (T == 16) launch_down_t<E, R, HELM, 16>(a, nu, grid, s, ps);
    else if (T == 64) launch_down_t<E, R, HELM, 64>(a, nu, grid, s, ps);
    else launch_down_t<E, R, HELM, 32>(a, nu, grid, s, ps);
}

template <typename E, int R, bool HELM>
void launch_up(const UpArgs<E>& a, int nu, dim3 grid, hipStream_t s, const ProfScope& ps, int T) {
    if (T == 16) launch_up_t<E, R, HELM, 16>(a, nu, grid, s, ps);
    else if (T == 64) launch_up_t<E, R, HELM, 64>(a, nu, grid, s, ps);
    else launch_up_t<E, R, HELM, 32>(a, nu, grid, s, ps);
}

template <typename E>
void down(int R, bool helm, const DownArgs<E>& a, int nu, dim3 g, hipStream_t s, const ProfScope& ps, int T) {
    if (R == 1) helm ? launch_down<E, 1, true>(a, nu, g, s, ps, T) : launch_down<E, 1, false>(a, nu, g, s, ps, T);
    else helm ? launch_down<E, 2, true>(a, nu, g, s, ps, T) : launch_down<E, 2, false>(a, nu, g, s, ps, T);
}

template <typename E>
void up(int R, bool helm, const UpArgs<E>& a, int nu, dim3 g, hipStream_t s, const ProfScope& ps, int T) {
    if (R == 1) helm ? launch_up<E, 1, true>(a, nu, g, s, ps, T) : launch_up<E, 1, false>(a, nu, g, s, ps, T);
    else helm ? launch_up<E, 2, true>(a, nu, g, s, ps, T) : launch_up<E, 2, false>(a, nu, g, s, ps, T);
}

// Tiles of a level's down or up pass: register tiles on the levels
// N >= c->reg_tile_min, LDS tiles of edge tile_for(N) below.  TX x TY owned
// nodes per workgroup.  split (register tiles) and split_lds (LDS tiles): two
// right-hand sides run as separate workgroups of one launch (grid z), not both
// in each workgroup.
struct PassGeom {
    bool reg, split, split_lds;
    int TX, TY;
    dim3 grid;
};
// The finest level takes register tiles from top_tile_min up already in FP64:
// its up pass then records the norms of the result and fuses with the next
// cycle's down pass (fuse_shape).
bool top_tiles(const wandqs_ctx* c) {
    return c->N >= c->top_tile_min && c->cfg.precision != WANDQS_MIXED;
}
PassGeom pass_geom(const wandqs_ctx* c, int N, int nu, bool down, bool norm = false) {
    PassGeom g{};
    g.reg = N >= c->reg_tile_min || (N == c->N && top_tiles(c));
    g.split = c->reg_split;
    g.split_lds = c->lds_split;
    if (g.reg) {
        const int halo = down || norm ? 2 * nu + 2 : 2 * nu;
        g.TX = 128 - 2 * halo;
        g.TY = kRegRows * kRegWaves - 2 * halo;
    } else {
        g.TX = g.TY = tile_for(c, N);
    }
    g.grid = dim3((N + g.TX - 1) / g.TX, (N + g.TY - 1) / g.TY);
    return g;
}

template <typename E, int R, bool HELM>
void launch_down_reg(const DownArgs<E>& a, int nu, dim3 grid, hipStream_t s, const ProfScope& ps) {
    constexpr int NW = kRegWaves;
    switch (nu) {
        case 1: WQ_KLAUNCH(ps, (k_mg_down_reg<E, R, HELM, 1, NW>), grid, dim3(64 * NW), 0, s, a); break;
        case 2: WQ_KLAUNCH(ps, (k_mg_down_reg<E, R, HELM, 2, NW>), grid, dim3(64 * NW), 0, s, a); break;
        default: WQ_KLAUNCH(ps, (k_mg_down_reg<E, R, HELM, 3, NW>), grid, dim3(64 * NW), 0, s, a); break;
    }
}

template <typename E, int R, bool HELM>
void launch_up_reg(const UpArgs<E>& a, int nu, dim3 grid, hipStream_t s, const ProfScope& ps) {
    constexpr int NW = kRegWaves;
    if (a.norm_part) {
        switch (nu) {
            case 1: WQ_KLAUNCH(ps, (k_mg_up_reg<E, R, HELM, 1, NW, true>), grid, dim3(64 * NW), 0, s, a); break;
            case 2: WQ_KLAUNCH(ps, (k_mg_up_reg<E, R, HELM, 2, NW, true>), grid, dim3(64 * NW), 0, s, a); break;
            default: WQ_KLAUNCH(ps, (k_mg_up_reg<E, R, HELM, 3, NW, true>), grid, dim3(64 * NW), 0, s, a); break;
        }
        return;
    }
    switch (nu) {
        case 1: WQ_KLAUNCH(ps, (k_mg_up_reg<E, R, HELM, 1, NW, false>), grid, dim3(64 * NW), 0, s, a); break;
        case 2: WQ_KLAUNCH(ps, (k_mg_up_reg<E, R, HELM, 2, NW, false>), grid, dim3(64 * NW), 0, s, a); break;
        default: WQ_KLAUNCH(ps, (k_mg_up_reg<E, R, HELM, 3, NW, false>), grid, dim3(64 * NW), 0, s, a); break;
    }
}

template <typename E>
void down_pass(int R, bool helm, const DownArgs<E>& a, int nu, const PassGeom& g, hipStream_t s,
               const ProfScope& ps) {
    if (!g.reg) {
        if (g.split_lds) return down<E>(1, helm, a, nu, dim3(g.grid.x, g.grid.y, R), s, ps, g.TX);
        return down<E>(R, helm, a, nu, g.grid, s, ps, g.TX);
    }
    if (R == 1 || g.split) {
        const dim3 gz(g.grid.x, g.grid.y, R);
        helm ? launch_down_reg<E, 1, true>(a, nu, gz, s, ps) : launch_down_reg<E, 1, false>(a, nu, gz, s, ps);
    } else {
        helm ? launch_down_reg<E, 2, true>(a, nu, g.grid, s, ps) : launch_down_reg<E, 2, false>(a, nu, g.grid, s, ps);
    }
}

template <typename E>
void up_pass(int R, bool helm, const UpArgs<E>& a, int nu, const PassGeom& g, hipStream_t s,
             const ProfScope& ps) {
    if (!g.reg) {
        if (g.split_lds) return up<E>(1, helm, a, nu, dim3(g.grid.x, g.grid.y, R), s, ps, g.TX);
        return up<E>(R, helm, a, nu, g.grid, s, ps, g.TX);
    }
    if (R == 1 || g.split) {
        const dim3 gz(g.grid.x, g.grid.y, R);
        helm ? launch_up_reg<E, 1, true>(a, nu, gz, s, ps) : launch_up_reg<E, 1, false>(a, nu, gz, s, ps);
    } else {
        helm ? launch_up_reg<E, 2, true>(a, nu, g.grid, s, ps) : launch_up_reg<E, 2, false>(a, nu, g.grid, s, ps);
    }
}

const char* type_name(double) { return "double"; }
const char* type_name(float) { return "float"; }

// Arrays of one solve: level 0 (u, f, k2) and the per-level buffers of type E.
// Geometry of the fused level-0 up-and-down launch (halo 2 nu_post + 2 nu_pre
// + 2), and whether a solve can use it: FP64 register tiles with one
// right-hand side per workgroup, equal pre- and post-sweep counts of 1 or 2.
bool fuse_possible(const wandqs_ctx* c) {
    const int nu = c->cfg.nu_pre;
    return c->mg_fuse && c->lc > 0 && (c->N >= c->reg_tile_min || top_tiles(c)) && c->reg_split &&
           nu == c->cfg.nu_post && nu >= 1 && nu <= 2 && c->lev[0].um2[0] != nullptr;
}
// Wavefronts and rows per wavefront of a fused tile (its halo: 10 rows on either
// side at two sweeps).  At 1024^2 (one right-hand side a workgroup, 2 in all)
// 8 x 8 took 30 us, 12 x 4 34, 8 x 4 51: the halo's share counts.  At 512^2 8 x 8
// leaves half the chip idle: 13.7 us, 12 x 4 11.3, 8 x 4 16.0.  At 256^2 the time
// of one tile counts: 8 x 8 13.1, 12 x 4 10.6, 8 x 4 9.2 (separate passes 13.1,
// and 4.3 for the residual norms of the result).
struct FuseShape {
    int waves, rows;
};
FuseShape fuse_shape(int N) {
    return N >= 1024 ? FuseShape{8, 8} : N >= 512 ? FuseShape{12, 4} : FuseShape{8, 4};
}
dim3 fuse_grid(const wandqs_ctx* c, int R) {
    const FuseShape f = fuse_shape(c->N);
    const int hl = 4 * c->cfg.nu_pre + 2;
    const int TX = 128 - 2 * hl, TY = f.rows * f.waves - 2 * hl, N = c->N;
    return dim3((N + TX - 1) / TX, (N + TY - 1) / TY, R);
}
template <int NW, int K>
void launch_updown_shape(const FuseArgs<double>& a, bool helm, int nu, dim3 grid, hipStream_t s,
                         const ProfScope& ps) {
    const dim3 blk(64 * NW);
    if (helm) {
        if (nu == 1) WQ_KLAUNCH(ps, (k_mg_updown_reg<double, 1, true, 1, 1, NW, K>), grid, blk, 0, s, a);
        else WQ_KLAUNCH(ps, (k_mg_updown_reg<double, 1, true, 2, 2, NW, K>), grid, blk, 0, s, a);
    } else {
        if (nu == 1) WQ_KLAUNCH(ps, (k_mg_updown_reg<double, 1, false, 1, 1, NW, K>), grid, blk, 0, s, a);
        else WQ_KLAUNCH(ps, (k_mg_updown_reg<double, 1, false, 2, 2, NW, K>), grid, blk, 0, s, a);
    }
}
void launch_updown_reg(const FuseArgs<double>& a, bool helm, int nu, dim3 grid, hipStream_t s,
                       const ProfScope& ps) {
    const FuseShape f = fuse_shape(a.N);
    if (f.rows == 8) launch_updown_shape<8, 8>(a, helm, nu, grid, s, ps);
    else if (f.waves == 12) launch_updown_shape<12, 4>(a, helm, nu, grid, s, ps);
    else launch_updown_shape<8, 4>(a, helm, nu, grid, s, ps);
}

// Level-0 fusion state of one cycle inside a batch (FP64 only).
struct FuseCtl {
    bool skip_down0 = false;  // the level-0 down pass ran fused into the previous cycle
    bool fuse_up0 = false;    // the level-0 up pass fuses with the next cycle's down pass
    int next_slot = -1;       // norm slot of the next cycle's incoming iterate (-1: none)
    int cur = 0;              // level-0 pre-smoothed iterate in um (0) or um2 (1)
};

template <typename E>
struct Hier {
    E* u0[2];
    E* f0[2];
    const double* k2;
};

template <typename E> E* lev_u(wq::Level& L, int r);
template <> double* lev_u<double>(wq::Level& L, int r) { return L.u[r]; }
template <> float* lev_u<float>(wq::Level& L, int r) { return L.u32[r]; }
template <typename E> E* lev_um(wq::Level& L, int r);
template <> double* lev_um<double>(wq::Level& L, int r) { return L.um[r]; }
template <> float* lev_um<float>(wq::Level& L, int r) { return L.um32[r]; }
template <typename E> E* lev_f(wq::Level& L, int r);
template <> double* lev_f<double>(wq::Level& L, int r) { return L.f[r]; }
template <> float* lev_f<float>(wq::Level& L, int r) { return L.f32[r]; }

int nu_pre_at(const wandqs_ctx* c, int l) { return l >= kFullPreLevels ? 1 : c->cfg.nu_pre; }

// The arguments of k_mg_coarse that do not depend on the launch (top level: lev[lc]).
template <typename E>
void coarse_args(wandqs_ctx* c, CoarseArgs<E>& a, bool helm) {
    const wq::Level& L = c->lev[c->lc];
    a.h = L.h;
    a.pitch = L.pitch;
    a.tab = c->ctab;
    a.omega = helm ? c->cfg.mg_omega_helm : c->cfg.mg_omega;
    a.h2max = helm ? kOmegaH2N0 / c->cfg.n0 : std::numeric_limits<double>::infinity();
    a.nu2 = c->cfg.nu_post;
}

// ncycles (times inner) V-cycles of a whole solve on a grid of at most 64^2 in
// one launch; slot >= 0: the norms before each of them and after the last go to
// the slots from it on, one partial each.
void whole_cycles(wandqs_ctx* c, int R, bool helm, const Hier<double>& hz, int ncycles, int inner,
                  int slot) {
    CoarseArgs<double> a{};
    coarse_args(c, a, helm);
    for (int r = 0; r < R; ++r) {
        a.f[r] = hz.f0[r];
        a.u_init[r] = hz.u0[r];
        a.u_out[r] = hz.u0[r];
    }
    a.ncycles = ncycles;
    a.inner = inner;
    a.nu1 = nu_pre_at(c, 0);
    a.norm_stride = (size_t)kNormVec * c->max_tiles;
    a.norm_part = slot >= 0 ? c->norm_part + slot * a.norm_stride : nullptr;
    const double nodes = (double)(c->N + 1) * (c->N + 1);
    char nm[64];
    prof_name(c, nm, sizeof nm, "k_mg_coarse<double, double, %s, %d>", helm ? "true" : "false", c->N);
    ProfScope ps(c, nm, nodes * (24.0 * R + (helm ? 16.0 : 0.0)));
#define WQ_WHOLE(n)                                                                                  \
    do {                                                                                             \
        const dim3 b(coarse_threads<n>());                                              \
        if (helm) WQ_KLAUNCH(ps, (k_mg_coarse<double, double, true, n>), dim3(R), b, 0, c->stream, a); \
        else WQ_KLAUNCH(ps, (k_mg_coarse<double, double, false, n>), dim3(R), b, 0, c->stream, a);   \
    } while (0)
    switch (c->N) {
        case 8: WQ_WHOLE(8); break;
        case 16: WQ_WHOLE(16); break;
        case 32: WQ_WHOLE(32); break;
        default: WQ_WHOLE(64); break;
    }
#undef WQ_WHOLE
}

// `iters` iterations with the exact solve on a grid of at most 64^2, in one launch;
// the norms go to the slots from `slot` on, as in whole_cycles.
void whole_direct(wandqs_ctx* c, int R, const Hier<double>& hz, int iters, int slot) {
    const wq::Level& L = c->lev[0];
    Poisson64Args a{};
    a.n = L.N;
    a.pitch = L.pitch;
    a.ih2 = 1.0 / (L.h * L.h);
    for (int r = 0; r < R; ++r) {
        a.f[r] = hz.f0[r];
        a.u[r] = hz.u0[r];
    }
    a.S = c->dst_S64;
    a.M = c->dst_M64;
    a.iters = iters;
    a.norm_stride = (size_t)kNormVec * c->max_tiles;
    a.norm_part = c->norm_part + slot * a.norm_stride;
    const double nodes = (double)(c->N + 1) * (c->N + 1);
    ProfScope ps(c, "k_poisson64", nodes * 24.0 * R + 2.0 * 8.0 * kDstN * kDstN);
    WQ_KLAUNCH(ps, k_poisson64, dim3(R), dim3(1024), 0, c->stream, a);
}

// One V-cycle on levels 0..L (grids above 64^2).  zero_guess: the level-0 iterate starts from 0.
// norm_slot >= 0 (double only) records the residual of the incoming iterate.
template <typename E>
void vcycle(wandqs_ctx* c, int R, bool helm, const Hier<E>& hz, bool zero_guess, int norm_slot,
            int up_norm_slot = -1, double* const* corr = nullptr, const FuseCtl* fz = nullptr) {
    hipStream_t s = c->stream;
    const int lc = c->lc;
    const double eb = sizeof(E);
    auto U = [&](int l, int r) { return l == 0 ? hz.u0[r] : lev_u<E>(c->lev[l], r); };
    auto F = [&](int l, int r) { return l == 0 ? hz.f0[r] : lev_f<E>(c->lev[l], r); };
    auto K = [&](int l) { return l == 0 ? hz.k2 : (const double*)c->lev[l].k2; };
    // Poisson: the V-cycle ends with the exact fast-sine-transform solve on
    // level 1 when that is 128^2 .. 2048^2
    const bool fst = !helm && fst_used(c);
    const int lb = fst ? 1 : lc;
    // relaxation factor of the smoothing sweeps: the Helmholtz levels whose
    // diagonal shift is no longer small (h^2 n0 > 1/8) relax with factor 1
    const double om = helm ? c->cfg.mg_omega_helm : c->cfg.mg_omega;
    const double h2max = helm ? kOmegaH2N0 / c->cfg.n0 : std::numeric_limits<double>::infinity();
    auto omega_of = [&](double h) { return h * h > h2max ? 1.0 : om; };
    // the level-0 pre-smoothed iterate (the fused passes alternate two buffers)
    auto um0 = [&](int r) -> E* {
        if (fz && fz->cur) return reinterpret_cast<E*>(c->lev[0].um2[r]);
        return lev_um<E>(c->lev[0], r);
    };
    for (int l = 0; l < lb; ++l) {
        if (l == 0 && fz && fz->skip_down0) continue;
        wq::Level& L = c->lev[l];
        DownArgs<E> a{};
        a.omega = omega_of(L.h);
        a.N = L.N;
        a.h = L.h;
        a.pitch = L.pitch;
        a.pitch_c = c->lev[l + 1].pitch;
        for (int r = 0; r < R; ++r) {
            a.u_in[r] = (l == 0 && !zero_guess) ? hz.u0[r] : nullptr;
            a.f[r] = F(l, r);
            a.u_out[r] = l == 0 ? um0(r) : lev_um<E>(L, r);
            a.f_c[r] = F(l + 1, r);
        }
        a.k2 = helm ? K(l) : nullptr;
        const int nu = nu_pre_at(c, l);
        const PassGeom g = pass_geom(c, L.N, nu, true);
        a.nblk = g.grid.x * g.grid.y;
        a.norm_part = (l == 0 && norm_slot >= 0)
                          ? c->norm_part + (size_t)norm_slot * kNormVec * c->max_tiles
                          : nullptr;
        // algorithmic bytes per owned node: u (when read), f, k2, smoothed u, coarse f
        const double nodes = (double)L.N * L.N;
        char nm[64];
        if (g.reg)
            prof_name(c, nm, sizeof nm, "k_mg_down_reg<%s, %d, %s, %d, %d>@%d", type_name(E()), g.split ? 1 : R,
                          helm ? "true" : "false", nu, kRegWaves, L.N);
        else
            prof_name(c, nm, sizeof nm, "k_mg_down<%s, %d, %s, %d, %d>@%d", type_name(E()), g.split_lds ? 1 : R,
                          helm ? "true" : "false", nu, g.TX, L.N);
        ProfScope ps(c, nm, nodes * ((a.u_in[0] ? eb * R : 0.0) + eb * R + (helm ? 8.0 : 0.0) +
                                     eb * R + eb * R / 4));
        down_pass<E>(R, helm, a, nu, g, s, ps);
    }
    // the mixed form's inner cycles (E = float) solve their coarsest grid in FP64
    constexpr bool coarse64 = std::is_same<E, float>::value;
    if (fst) {
        const E* fo[2] = {F(1, 0), R > 1 ? F(1, 1) : nullptr};
        E* uo[2] = {U(1, 0), R > 1 ? U(1, 1) : nullptr};
        fst_solve<E>(c, R, fo, uo);
    } else {
        wq::Level& L = c->lev[lc];  // 64^2
        const double nodes = (double)(L.N + 1) * (L.N + 1);
        char nm[64];
        if (!helm && coarse64) {  // exact Poisson coarse solve, FP64
            DstArgs64<E> d{};
            d.pitch = L.pitch;
            for (int r = 0; r < R; ++r) {
                d.f[r] = F(lc, r);
                d.u_out[r] = U(lc, r);
            }
            d.S = c->dst_S64;
            d.M = c->dst_M64;
            ProfScope ps(c, "k_coarse_dst64<float>", nodes * 2.0 * eb * R + 2.0 * 8.0 * kDstN * kDstN);
            WQ_KLAUNCH(ps, k_coarse_dst64<E>, dim3(R), dim3(1024), 0, s, d);
        } else if (!helm) {  // exact Poisson coarse solve
            DstArgs<E> d{};
            d.pitch = L.pitch;
            for (int r = 0; r < R; ++r) {
                d.f[r] = F(lc, r);
                d.u_out[r] = U(lc, r);
            }
            d.S = c->dst_S;
            d.M = c->dst_M;
            prof_name(c, nm, sizeof nm, "k_coarse_dst<%s>", type_name(E()));
            ProfScope ps(c, nm, nodes * 2.0 * eb * R + 2.0 * 4.0 * kDstN * kDstN);
            WQ_KLAUNCH(ps, k_coarse_dst<E>, dim3(R), dim3(1024), 0, s, d);
        } else {
            // float sweeps, as they only correct a finer FP64 level; double in
            // the mixed form's inner cycles, whose finer levels are in float
            using CT = typename std::conditional<coarse64, double, float>::type;
            CoarseArgs<E> a{};
            coarse_args(c, a, helm);
            for (int r = 0; r < R; ++r) {
                a.f[r] = F(lc, r);
                a.u_out[r] = U(lc, r);
            }
            a.ncycles = 1;
            a.inner = 1;
            a.nu1 = nu_pre_at(c, lc);
            if (c->cfg.mg_rtol > 0.0 && a.nu2 >= 2) {
                a.inner = kCoarseCycles;
                a.nu1 = std::max(1, a.nu1 - 1);
                --a.nu2;
            }
            prof_name(c, nm, sizeof nm, "k_mg_coarse<%s, %s, true, 64>", type_name(E()), type_name(CT()));
            ProfScope ps(c, nm, nodes * (2.0 * eb * R + 2.0 * sizeof(CT)));
            WQ_KLAUNCH(ps, (k_mg_coarse<E, CT, true, 64>), dim3(R), dim3(coarse_threads<64>()), 0, s, a);
        }
    }
    for (int l = lb - 1; l >= 0; --l) {
        wq::Level& L = c->lev[l];
        if constexpr (std::is_same<E, double>::value) {
            if (l == 0 && fz && fz->fuse_up0) {
                // up pass fused with the next cycle's down pass: into the other
                // buffer, recording the norms of the next cycle's incoming iterate
                FuseArgs<double> a{};
                a.N = L.N;
                a.h = L.h;
                a.pitch = L.pitch;
                a.pitch_c = c->lev[1].pitch;
                a.omega = omega_of(L.h);
                for (int r = 0; r < R; ++r) {
                    a.u_mid[r] = um0(r);
                    a.e_c[r] = U(1, r);
                    a.f[r] = F(0, r);
                    a.u_out[r] = fz->cur ? L.um[r] : L.um2[r];
                    a.f_c[r] = F(1, r);
                }
                a.k2 = helm ? K(0) : nullptr;
                const dim3 g = fuse_grid(c, R);
                a.nblk = g.x * g.y;
                if (fz->next_slot >= 0)
                    a.norm_part = c->norm_part + (size_t)fz->next_slot * kNormVec * c->max_tiles;
                const double nodes = (double)L.N * L.N;
                char nm[64];
                prof_name(c, nm, sizeof nm, "k_mg_updown_reg<double, 1, %s, %d, %d, %d, %d>@%d",
                          helm ? "true" : "false", c->cfg.nu_pre, c->cfg.nu_post, fuse_shape(L.N).waves,
                          fuse_shape(L.N).rows, L.N);
                // per owned node and right-hand side: smoothed u, 1/4 coarse e,
                // f, new smoothed u, 1/4 coarse f; k2 once
                ProfScope ps(c, nm, nodes * (R * (8.0 + 2.0 + 8.0 + 8.0 + 2.0) + (helm ? 8.0 : 0.0)));
                launch_updown_reg(a, helm, c->cfg.nu_pre, g, s, ps);
                continue;
            }
        }
        UpArgs<E> a{};
        a.omega = omega_of(L.h);
        a.N = L.N;
        a.h = L.h;
        a.pitch = L.pitch;
        a.pitch_c = c->lev[l + 1].pitch;
        for (int r = 0; r < R; ++r) {
            a.u_mid[r] = l == 0 ? um0(r) : lev_um<E>(L, r);
            a.e_c[r] = U(l + 1, r);
            a.f[r] = F(l, r);
            a.u_out[r] = U(l, r);
        }
        a.k2 = helm ? K(l) : nullptr;
        // per owned node: smoothed u, coarse correction (1/4), f, k2, corrected u
        const double nodes = (double)L.N * L.N;
        char nm[64];
        // the finest up pass of a batch's last cycle records the result's norms
        const bool unorm = l == 0 && up_norm_slot >= 0;
        if (l == 0 && corr)
            for (int r = 0; r < R; ++r) a.corr[r] = corr[r];
        const PassGeom g = pass_geom(c, L.N, c->cfg.nu_post, false, unorm);
        if (unorm) {
            a.norm_part = c->norm_part + (size_t)up_norm_slot * kNormVec * c->max_tiles;
            a.nblk = g.grid.x * g.grid.y;
        }
        if (g.reg)
            prof_name(c, nm, sizeof nm, "k_mg_up_reg<%s, %d, %s, %d, %d, %s>@%d", type_name(E()),
                      g.split ? 1 : R, helm ? "true" : "false", c->cfg.nu_post, kRegWaves,
                      unorm ? "true" : "false", L.N);
        else
            prof_name(c, nm, sizeof nm, "k_mg_up<%s, %d, %s, %d, %d>@%d", type_name(E()), g.split_lds ? 1 : R,
                          helm ? "true" : "false", c->cfg.nu_post, g.TX, L.N);
        ProfScope ps(c, nm, nodes * (eb * R + eb * R / 4 + eb * R + (helm ? 8.0 : 0.0) + eb * R));
        up_pass<E>(R, helm, a, c->cfg.nu_post, g, s, ps);
    }
}

// FP64 residual norms of the level-0 iterate into `slot` (one partial per
// interior row); with r32 set the residual is also stored in float (the mixed
// form's defect).
void resnorm(wandqs_ctx* c, int R, bool helm, const Hier<double>& hz, int slot,
             float* const* r32) {
    const wq::Level& L = c->lev[0];
    const dim3 g((L.N - 1 + kThreads / 64 - 1) / (kThreads / 64), R);
    double* part = c->norm_part + (size_t)slot * kNormVec * c->max_tiles;
    const double ih2 = 1.0 / (L.h * L.h);
    float* o0 = r32 ? r32[0] : nullptr;
    float* o1 = (r32 && R > 1) ? r32[1] : nullptr;
    char nm[56];
    prof_name(c, nm, sizeof nm, "k_resnorm<%s>%s", helm ? "true" : "false", r32 ? "+defect" : "");
    ProfScope ps(c, nm, (double)L.N * L.N * (16.0 * R + (helm ? 8.0 : 0.0) + (r32 ? 4.0 * R : 0.0)));
    if (helm)
        WQ_KLAUNCH(ps, k_resnorm<true>, g, dim3(kThreads), 0, c->stream, L.N, ih2, L.pitch, hz.u0[0],
                   hz.u0[1], hz.f0[0], hz.f0[1], hz.k2, part, L.N - 1, o0, o1);
    else
        WQ_KLAUNCH(ps, k_resnorm<false>, g, dim3(kThreads), 0, c->stream, L.N, ih2, L.pitch, hz.u0[0],
                   hz.u0[1], hz.f0[0], hz.f0[1], hz.k2, part, L.N - 1, o0, o1);
}

// One outer iteration of the mixed form: defect r = f - A u in FP64 (stored in
// float, norms recorded in `slot`), `inner` FP32 V-cycles on A e = r from e = 0,
// then u += e in FP64.
void mixed_iteration(wandqs_ctx* c, int R, bool helm, const Hier<double>& hz, int slot) {
    wq::Level& L0 = c->lev[0];
    Hier<float> hf{{L0.u32[0], L0.u32[1]}, {L0.f32[0], L0.f32[1]}, hz.k2};
    resnorm(c, R, helm, hz, slot, hf.f0);
    const int inner = c->cfg.mg_inner_cycles > 0 ? c->cfg.mg_inner_cycles : 1;
    // the last inner cycle's finest up pass adds its result to the FP64
    // iterate (u += e) itself
    double* const corr[2] = {hz.u0[0], R > 1 ? hz.u0[1] : nullptr};
    for (int i = 0; i < inner; ++i)
        vcycle<float>(c, R, helm, hf, i == 0, -1, -1, i == inner - 1 ? corr : nullptr);
}

}  // namespace

#ifndef WQ_TOP_TILE_MIN
#define WQ_TOP_TILE_MIN 128
#endif
int reg_tile_min_default() { return WQ_REG_TILE_MIN; }
int top_tile_min_default() { return WQ_TOP_TILE_MIN; }
int small_tile_max_default() { return WQ_SMALL_TILE_MAX; }

wandqs_status make_dst_tables(wandqs_ctx* c) {
    hipLaunchKernelGGL(k_dst_tables, dim3(kDstN * kDstN / 256), dim3(256), 0, c->stream,
                       c->lev[c->lc].N, c->lev[c->lc].h, c->dst_S, c->dst_M, c->dst_S64, c->dst_M64);
    WQ_LAUNCH_CHECK();
    return make_fst_tables(c);
}


// Launches one cycle, body() on c->stream, as a HIP graph: the graph of `key`
// is captured on c->cap_stream and instantiated at its first use and replayed
// after.  With graphs off, with the per-kernel timing on (its events belong to
// direct launches), or when a capture fails (graphs then stay off for the
// context), body() launches directly.
template <class F>
hipError_t run_cycle(wandqs_ctx* c, const CycleKey& key, F&& body) {
    if (c->graphs_on && !c->prof.on && hipPeekAtLastError() == hipSuccess) {
        for (const CycleGraph& g : c->graphs)
            if (g.key == key) return hipGraphLaunch(g.exec, c->stream);
        if ((int)c->graphs.size() < kMaxGraphs) {
            hipGraphExec_t ex = nullptr;
            bool ok = c->cap_stream ||
                      hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking) == hipSuccess;
            if (!ok) c->cap_stream = nullptr;
            ok = ok && hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed) == hipSuccess;
            if (ok) {
                const hipStream_t s0 = c->stream;
                c->stream = c->cap_stream;
                body();
                c->stream = s0;
                const bool launched = hipGetLastError() == hipSuccess;
                hipGraph_t g = nullptr;
                ok = hipStreamEndCapture(c->cap_stream, &g) == hipSuccess && launched && g &&
                     hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) == hipSuccess;
                if (g) (void)hipGraphDestroy(g);
            }
            if (ok) {
                c->graphs.push_back(CycleGraph{key, ex});
                return hipGraphLaunch(ex, c->stream);
            }
            if (ex) (void)hipGraphExecDestroy(ex);
            (void)hipGetLastError();
            c->graphs_on = false;
        }
    }
    body();
    return hipSuccess;
}

// Waits until the device has published sequence number seq (k_reduce_publish): a
// bounded spin on the coherent host word, then a stream synchronisation,
// which also reports a failed kernel.
wandqs_status wait_published(wandqs_ctx* c, const uint32_t* h_seq, uint32_t seq) {
    const auto t0 = std::chrono::steady_clock::now();
    for (long it = 0;; ++it) {
        if (__atomic_load_n(h_seq, __ATOMIC_ACQUIRE) == seq) return WANDQS_OK;
        if ((it & 1023) == 1023 &&
            std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(200))
            break;
        __builtin_ia32_pause();
    }
    WQ_HIP(hipStreamSynchronize(c->stream));
    if (__atomic_load_n(h_seq, __ATOMIC_ACQUIRE) == seq) return WANDQS_OK;
    c->err = "residual norms were not published by the device";
    return WANDQS_E_HIP;
}

// Poisson solves in tolerance mode on grids up to 2048^2 iterate
// u += L_h^-1 (f - L_h u) with the exact sine-transform solve on the finest
// level itself (fst.hip; up to 64^2 k_poisson64) in FP64, in both precision forms: the correction's
// rounding (1e-14 .. 3e-13 of it) is the only error an iteration leaves, so from
// an extrapolated guess one iteration reaches the rounding floor and from zero
// two do, where the V-cycles that end with the same solve one level down took 5
// to 7.  The three
// solves of a slice at 1024^2: 130 instead of 446 us (kernel time), at 256^2
// 46 instead of 310 us.
// A caller that allows fewer than kDirectMinCycles cycles counts V-cycles (and
// may want the WANDQS_E_NOCONV they end with), so it keeps them; with that many
// the V-cycles (a factor 10 and more per cycle) converge as well.  Fixed mode
// (mg_rtol <= 0) is a number of V-cycles by definition.
constexpr int kDirectMinCycles = 16;
bool direct_poisson(const wandqs_ctx* c, bool helm) {
    return !helm && c->cfg.mg_rtol > 0.0 && c->cfg.mg_max_cycles >= kDirectMinCycles &&
           (c->fst_top_tw != nullptr || c->lc == 0);
}

// Solve with the context's stop rule.  Tolerance mode (mg_rtol > 0) runs a batch
// of V-cycles sized by the previous slice's count for this solve, reads the
// residual norms back once per batch and adds batches sized by its gain until every
// right-hand side meets ||r|| <= rtol ||f|| + atol sqrt(n) or reaches the
// rounding floor: either ||r|| <= kFloorBE eps (8/h^2 ||u|| + ||f||) (the
// residual is at the size that rounding in forming it leaves), or a cycle no
// longer halves ||r|| once ||r|| <= 1e-9 max(||f||, ||r_0||), r_0 the initial
// residual.
// Fixed mode runs mg_max_cycles cycles without any host synchronisation.
wandqs_status helm_levels(wandqs_ctx* c, const double* k2) {
    hipStream_t s = c->stream;
    {  // k2 on the tile levels 1..lc: the last kChainMax of them in one launch
        const int l0 = std::max(0, c->lc - kChainMax);
        for (int l = 1; l <= l0; ++l) {
            const wq::Level& F = c->lev[l - 1];
            const wq::Level& C = c->lev[l];
            const double* src = l == 1 ? k2 : F.k2;
            ProfScope ps(c, "k_restrict_fw", 8.0 * ((double)(F.N + 1) * (F.N + 1) + (double)(C.N + 1) * (C.N + 1)));
            WQ_KLAUNCH(ps, k_restrict_fw, dim3((C.N + 1 + 127) / 128, C.N + 1), dim3(128), 0, s,
                               src, F.pitch, C.k2, C.pitch, C.N);
        }
        if (c->lc > 0) {
            const wq::Level& F = c->lev[l0];
            ChainArgs a{};
            a.fine = l0 == 0 ? k2 : F.k2;
            a.N = F.N;
            a.pitch = F.pitch;
            double bytes = 8.0 * (F.N + 1) * (F.N + 1);
            for (int l = l0 + 1; l <= c->lc; ++l) {
                a.coarse[l - l0 - 1] = c->lev[l].k2;
                a.pc[l - l0 - 1] = c->lev[l].pitch;
                bytes += 8.0 * (c->lev[l].N + 1) * (c->lev[l].N + 1);
            }
            const int nb = (c->lev[c->lc].N + kChainB) / kChainB;
            ProfScope ps(c, "k_restrict_chain", bytes);
            switch (c->lc - l0) {
                case 1: WQ_KLAUNCH(ps, k_restrict_chain<1>, dim3(nb, nb), dim3(chain_threads<1>()), 0, s, a); break;
                case 2: WQ_KLAUNCH(ps, k_restrict_chain<2>, dim3(nb, nb), dim3(chain_threads<2>()), 0, s, a); break;
                case 3: WQ_KLAUNCH(ps, k_restrict_chain<3>, dim3(nb, nb), dim3(chain_threads<3>()), 0, s, a); break;
                default: WQ_KLAUNCH(ps, k_restrict_chain<4>, dim3(nb, nb), dim3(chain_threads<4>()), 0, s, a); break;
            }
        }
        // k2 of the coarse-kernel levels, once per solve
        const wq::Level& T = c->lev[c->lc];
        const double* top = c->lc == 0 ? k2 : T.k2;
        ProfScope ps(c, "k_coarse_k2", 32.0 * (T.N + 1) * (T.N + 1) + 24.0 * kCoarseT);
        WQ_KLAUNCH(ps, k_coarse_k2, dim3(1), dim3(kK2Threads), 0, s, T.N, T.pitch, T.h, top,
                           c->ctab);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

wandqs_status mg_solve(wandqs_ctx* c, int kind, int R, bool helm, double* const u[2],
                       double* const f[2], const double* k2, SolveResult* res,
                       const std::function<wandqs_status()>& ahead, bool k2_levels_ready) {
    hipStream_t s = c->stream;
    Hier<double> hz{{u[0], R > 1 ? u[1] : nullptr}, {f[0], R > 1 ? f[1] : nullptr}, k2};
    // grids of at most 64^2 run whole in the coarse kernel, in double in both
    // forms (a mixed iteration is then its inner cycles)
    const bool whole = c->lc == 0;
    const bool mixed = c->cfg.precision == WANDQS_MIXED && !whole;
    const int inner = c->cfg.precision == WANDQS_MIXED ? std::max(1, c->cfg.mg_inner_cycles) : 1;
    const bool direct = direct_poisson(c, helm);
    if (helm && !k2_levels_ready) {
        const wandqs_status st = helm_levels(c, k2);
        if (st != WANDQS_OK) return st;
    }
    // one "cycle" is a V-cycle (FP64) or an outer defect-correction iteration
    // (mixed) that records its residual norms in `slot` (FP64: -1, none)
    hipError_t gerr = hipSuccess;
    // upslot >= 0 (FP64, register tiles on level 0): the cycle's finest up pass
    // records the norms of its result in slot upslot
    auto cycle = [&](int slot, int upslot, const FuseCtl& fz) {
        const int fk = (fz.skip_down0 ? 1 : 0) | (fz.fuse_up0 ? 2 : 0) | (fz.cur ? 4 : 0) |
                       (direct ? 8 : 0);
        const CycleKey key{{hz.u0[0], hz.u0[1], hz.f0[0], hz.f0[1], hz.k2}, R, helm, mixed, slot,
                           upslot, fk};
        const hipError_t e = run_cycle(c, key, [&] {
            if (direct)
                fst_top_iteration(c, R, hz.f0, hz.u0, c->norm_part + (size_t)slot * kNormVec * c->max_tiles);
            else if (mixed) mixed_iteration(c, R, helm, hz, slot);
            else vcycle<double>(c, R, helm, hz, false, slot, upslot, nullptr, &fz);
        });
        if (gerr == hipSuccess) gerr = e;
    };
    auto graph_check = [&]() -> wandqs_status {
        if (gerr == hipSuccess) return WANDQS_OK;
        c->err = std::string("hipGraphLaunch: ") + hipGetErrorString(gerr);
        return WANDQS_E_HIP;
    };
    const int maxc = c->cfg.mg_max_cycles;
    if (!(c->cfg.mg_rtol > 0.0)) {
        if (whole) whole_cycles(c, R, helm, hz, maxc, inner, -1);
        const bool fuse = !mixed && fuse_possible(c);
        for (int k = 0, cur = 0; k < maxc && !whole; ++k) {
            FuseCtl fz;
            fz.skip_down0 = fuse && k > 0;
            fz.fuse_up0 = fuse && k < maxc - 1;
            fz.cur = cur;
            cycle(mixed ? 0 : -1, -1, fz);
            if (fz.fuse_up0) cur ^= 1;
        }
        if (graph_check() != WANDQS_OK) return WANDQS_E_HIP;
        WQ_LAUNCH_CHECK();
        if (res) *res = SolveResult{maxc, {-1.0, -1.0}};
        return ahead ? ahead() : WANDQS_OK;
    }
    const int N = c->N;
    const double atol = c->cfg.mg_atol * std::sqrt((double)(N - 1) * (N - 1));
    // partial sums of the norms per slot
    // (the V-cycles' down passes: one per level-0 tile; resnorm and the sine
    // transform solve: one per interior row; whole solves in one workgroup: one)
    const dim3 g = pass_geom(c, N, nu_pre_at(c, 0), true).grid;
    const int nblk = whole ? 1 : mixed || direct ? N - 1 : g.x * g.y;
    // the batch's last cycle records the final norms in its finest up pass
    // (register tiles, FP64) instead of a separate residual pass
    const PassGeom gu = pass_geom(c, N, c->cfg.nu_post, false, true);
    const bool up_norms = !mixed && !direct && !whole && gu.reg;
    const int nblk_up = up_norms ? (int)(gu.grid.x * gu.grid.y) : whole ? 1 : N - 1;
    // inside a batch, each cycle's level-0 up pass but the last fuses with the
    // next cycle's down pass; their norm slots have the fused launch's tiles
    const bool fuse = !mixed && up_norms && fuse_possible(c);
    const dim3 fg = fuse_grid(c, R);
    const int nblk_fuse = fg.x * fg.y;
    int cur = 0;
    int done = 0, more = 1;
    int pred = c->pred[kind] < 1 ? 1 : c->pred[kind];
    double* hr = c->h_pin;  // [kMaxSlots][kNormVec] + flags
    constexpr int V = kNormVec;
    const double a_norm = 8.0 / (c->lev[0].h * c->lev[0].h);  // ||L_h||_2 bound
    const double eps = std::numeric_limits<double>::epsilon();
    while (true) {
        int b = done == 0 ? pred : more;
        if (done + b > maxc) b = maxc - done;
        if (whole && direct) whole_direct(c, R, hz, b, done);
        else if (whole) whole_cycles(c, R, helm, hz, b, inner, done);
        for (int k = 0; k < b && !whole; ++k) {
            const int cyc = done + k;
            FuseCtl fz;
            fz.skip_down0 = fuse && k > 0;
            fz.fuse_up0 = fuse && k < b - 1;
            fz.next_slot = cyc + 1;
            fz.cur = cur;
            cycle(cyc, up_norms && k == b - 1 ? cyc + 1 : -1, fz);
            if (fz.fuse_up0) cur ^= 1;
        }
        if (!whole && !up_norms) resnorm(c, R, helm, hz, done + b, nullptr);
        const int s0 = done == 0 ? 0 : done + 1;
        const int ns = done + b + 1 - s0;
        if (graph_check() != WANDQS_OK) return WANDQS_E_HIP;
        WQ_LAUNCH_CHECK();
        int32_t* h_flags = reinterpret_cast<int32_t*>(hr + V * kMaxSlots);
        uint32_t* h_seq = reinterpret_cast<uint32_t*>(hr + V * kMaxSlots + 1);
        const uint32_t seq = ++c->pub_seq;
        {
            ProfScope ps(c, "k_reduce_publish", 8.0 * ns * 3 * R * (nblk + 1));
            WQ_KLAUNCH(ps, k_reduce_publish, dim3(ns * 3 * R), dim3(kThreads), 0, s,
                       c->norm_part, V * c->max_tiles, nblk, s0, 3 * R, done + b, nblk_up, fuse ? done + 1 : 0, fuse ? done + b : 0, nblk_fuse, hr, c->flags,
                       h_flags, h_seq, seq, c->pub_count);
        }
        WQ_LAUNCH_CHECK();
        // behind the first batch: the caller's follow-up work, on the device
        // while the host waits for the norms
        const bool first = done == 0;
        if (first && ahead) {
            const wandqs_status st = ahead();
            if (st != WANDQS_OK) return st;
        }
        if (wait_published(c, h_seq, seq) != WANDQS_OK) return WANDQS_E_HIP;
        done += b;
        const int32_t fl = __atomic_load_n(h_flags, __ATOMIC_ACQUIRE);
        // first cycle count at which every rhs satisfies the stop rule
        int need = -1;
        for (int k = 0; k <= done && need < 0; ++k) {
            bool all = true;
            for (int r = 0; r < R; ++r) {
                const double rr = std::sqrt(hr[V * k + 3 * r]);
                const double ff = std::sqrt(hr[V * k + 3 * r + 1]);
                const double uu = std::sqrt(hr[V * k + 3 * r + 2]);
                // relative to ||f||; for f = 0 (solution 0) relative to ||r_0||
                const double ref = ff > 0 ? ff : std::sqrt(hr[3 * r]);
                bool ok = std::isfinite(rr) && (rr <= c->cfg.mg_rtol * ref + atol ||
                                                rr <= kFloorBE * eps * (a_norm * uu + ff));
                if (!ok && k >= 2) {
                    const double rp = std::sqrt(hr[V * (k - 1) + 3 * r]);
                    const double scale = std::max(ff, std::sqrt(hr[3 * r]));
                    ok = std::isfinite(rr) && rr > 0.5 * rp && rr <= 1e-9 * scale;
                }
                all = all && ok;
            }
            if (all) need = k;
        }
        if (need >= 0 || done >= maxc || (fl & 1)) {
            if (res) {
                res->cycles = done;
                for (int r = 0; r < R; ++r) {
                    const double rr = std::sqrt(hr[V * done + 3 * r]);
                    const double ff = std::sqrt(hr[V * done + 3 * r + 1]);
                    res->rel[r] = ff > 0 ? rr / ff : rr;
                }
            }
            if (fl & 1) {
                c->err = "1 + psi <= 0 where plasma is present";
                return WANDQS_E_NONPHYS;
            }
            if (need < 0) {
                static const char* names[kPredKinds] = {"psi", "Ez/Bz", "B_perp", "user",
                                                        "psi adjoint", "Ez/Bz adjoint",
                                                        "B_perp adjoint", "user"};
                c->err = std::string("multigrid did not converge within mg_max_cycles (") +
                         names[kind & (kPredKinds - 1)] + " solve, ||r||/||f|| = " +
                         std::to_string(res ? res->rel[0] : -1.0) + ")";
                return WANDQS_E_NOCONV;
            }
            c->pred[kind] = need < 1 ? 1 : need;
            // further cycles ran after the follow-up work: it reads the final
            // iterate only when enqueued again
            if (!first && ahead) return ahead();
            return WANDQS_OK;
        }
        // the next batch: the cycles that the last one's gain leaves to do for the
        // right-hand side that is furthest off, rounded down and one fewer (later
        // cycles gain more than the first).  Single cycles cost a norm check each:
        // the slice behind a restored state, whose own solve predicts none, took
        // eight batches at 64^2, now four or five.
        more = 1;
        for (int r = 0; r < R; ++r) {
            const double rr = std::sqrt(hr[V * done + 3 * r]), rp = std::sqrt(hr[V * (done - 1) + 3 * r]);
            const double ff = std::sqrt(hr[V * done + 3 * r + 1]), uu = std::sqrt(hr[V * done + 3 * r + 2]);
            const double goal = std::max(c->cfg.mg_rtol * (ff > 0 ? ff : std::sqrt(hr[3 * r])) + atol,
                                         kFloorBE * eps * (a_norm * uu + ff));
            const double left = std::log(goal / rr) / std::log(rr / rp);
            if (rr > goal && left >= more + 2.0 && left < maxc) more = (int)left - 1;
        }
    }
}

}  // namespace wq

