// Multigrid on a non-uniform transverse grid (Sec. VII.B): lap u + M u = J on
// a tensor grid x_0 < ... < x_N, y_0 < ... < y_N with u = 0 on the boundary.
//
// Along x at an interior node i (h- = x_i - x_{i-1}, h+ = x_{i+1} - x_i,
// ha = h+ + h-, hb = h+ - h-): Dxx u = 2 (h+ u_{i-1} - ha u_i + h- u_{i+1}) /
// (h- h+ ha) and the three-point derivative dx u = h-/(ha h+) (u_{i+1} - u_i)
// + h+/(ha h-) (u_i - u_{i-1}).  Since Dxx u = u_xx + (hb/3) u_xxx + O(h^2),
// the third-order terms are removed with eq. (36), which gives the discrete
// equation L u = R J with
//   L u = Dxx u + Dyy u + (1/3)[hb_x dx(Dyy u) + hb_y dy(Dxx u)]
//         + (1/3)(hb_x dx + hb_y dy)(M u) + M u,
//   R J = J + (1/3)(hb_x dx + hb_y dy) J,
// a nine-point, non-symmetric operator (the 5-point Laplacian plus M on a
// uniform grid).
//
// The solver: V-cycles smoothing by alternating zebra line relaxation (x-lines
// of odd then even rows, y-lines of odd then even columns, one such step before and
// one after the coarse correction, on the levels of N <= 64 (nu + 1) / 2 of them for
// nu_pre and nu_post: cells of aspect ratio up to 3 defeat point smoothers, and a
// line step smooths like two of their sweeps); coarse grids keep every other node
// and rediscretise L; the prolongation interpolates linearly in the coordinates and the restriction
// is its transpose weighted by the control volumes (x_{i+1} - x_{i-1})/2 per
// direction, for the residual and for M.  Levels of N <= 64 run in one
// workgroup in LDS down to the single interior node of the 2-cell grid.  The
// stop rule is the context's (mg_rtol, mg_atol, the rounding floor with
// 2 max |d| as the size of L, d the coefficient of u_ij in its own equation),
// except that a cycle counts as stagnating only when it reduces ||r|| by less
// than 10% once ||r|| <= 1e-9 ||R J||.
//
// With a_k, b_k the Dxx and Dyy weights of a node's index and g_k, h_k the dx
// and dy weights times hb/3 (k = -1, 0, 1), L u needs per column only
//   S = Dyy u + M u,  V = u + sum_k h_k u(., j+k),  W = sum_k h_k (M u)(., j+k):
//   L u = S + W + sum_k (g_k S(i+k, .) + a_k V(i+k, .)),
// so a wavefront along x forms it from three rows with two pairs of lane
// shifts.  Per-level 1-D tables (host-made, one copy per call): for every index
// a_k and g_k (6 arrays); for the restriction to the next level, three weights
// per coarse index; for the prolongation from it, two per fine index.
//
// Line solves: holding the other lines, L restricted to a line is tridiagonal
// and depends on the grid and M alone, so its factors are made once per call
// (k_nu_factor: the pivots are a serial chain, one thread per line) and every
// relaxation is two first-order recurrences, y_t = (r_t - sub_t y_{t-1}) ib_t and
// x_t = y_t + ga_t x_{t+1}, which one wavefront runs as scans of affine maps: each
// lane a chunk of the line, the chunks' maps composed across the lanes by DPP.
// The factors (be = -sub ib, ib, ga) lie in the fields of the earlier slices,
// which a solve gives up anyway.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <limits>
#include <vector>

#include "wq_common.h"

namespace wq {
namespace {

constexpr int kNuCoarse = 64;
static_assert(kCoarseMax == kNuCoarse, "the coarse workgroup's LDS holds levels up to 64 cells");
constexpr int kNuThreads = 1024;
constexpr int kNuLdsNodes = 65 * 65 + 33 * 33 + 17 * 17 + 9 * 9 + 5 * 5 + 3 * 3;
constexpr int kNuLines = 4;  // lines per workgroup of the line kernels

// doubles of one level's tables: cx, cy [6][n+1]; rx, ry [n/2+1][3] (restriction
// to the next level); px, py [n+1][2] (prolongation from the next level)
constexpr int nu_level_doubles(int n) { return 2 * (6 * (n + 1) + 3 * (n / 2 + 1) + 2 * (n + 1)); }
constexpr int nu_chain_doubles(int n) { return n < 2 ? 0 : nu_level_doubles(n) + nu_chain_doubles(n / 2); }

struct NuTabs {
    const double *cx, *cy, *rx, *ry, *px, *py;
};
__host__ __device__ inline NuTabs nu_tabs_at(const double* b, int n) {
    NuTabs t;
    t.cx = b;
    t.cy = t.cx + 6 * (n + 1);
    t.rx = t.cy + 6 * (n + 1);
    t.ry = t.rx + 3 * (n / 2 + 1);
    t.px = t.ry + 3 * (n / 2 + 1);
    t.py = t.px + 2 * (n + 1);
    return t;
}

// The factors of one level and direction, in the layout of the lanes that read
// them: line-major; within a line of n > 64 cells unknown t at (t % per) 64 + t /
// per, per = n / 64; of n <= 64 at t, and ga at n - 1 - t (the backward scan runs
// over reversed lanes).  Unknown n - 1 (past the end) holds zeros.
struct NuFac {
    double *be, *ib, *ga;
};

__device__ __forceinline__ double nu_shift_up(double v) {  // lane i reads lane i - 1 (0 at lane 0)
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x138, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x138, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double nu_shift_down(double v) {  // lane i reads lane i + 1 (0 at lane 63)
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x130, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x130, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// DPP move that leaves `old` in the lanes without a source.
template <int CTRL, int ROWS>
__device__ __forceinline__ double nu_dpp(double old, double v) {
    const unsigned long long o = (unsigned long long)__double_as_longlong(old);
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)o, (int)(unsigned)b, CTRL, ROWS, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(o >> 32), (int)(unsigned)(b >> 32), CTRL, ROWS, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Inclusive scan of the affine maps y -> A y + B over segments of n lanes (n a
// power of two from 4): afterwards B is the value after the lane's own map of a
// chain that starts at 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ void nu_scan_step(double& A, double& B, bool in) {
    const double Ap = nu_dpp<CTRL, ROWS>(1.0, A), Bp = nu_dpp<CTRL, ROWS>(0.0, B);
    B = __builtin_fma(A, in ? Bp : 0.0, B);
    A *= in ? Ap : 1.0;
}
template <int n>
__device__ __forceinline__ void nu_scan(double& A, double& B, int seg) {
    nu_scan_step<0x111, 0xF>(A, B, n >= 16 || seg >= 1);  // row_shr:1, 2, 4, 8 (rows of 16 lanes)
    nu_scan_step<0x112, 0xF>(A, B, n >= 16 || seg >= 2);
    if constexpr (n >= 8) nu_scan_step<0x114, 0xF>(A, B, n >= 16 || seg >= 4);
    if constexpr (n >= 16) nu_scan_step<0x118, 0xF>(A, B, true);
    if constexpr (n >= 32) nu_scan_step<0x142, 0xA>(A, B, true);  // row_bcast:15 into rows 1 and 3
    if constexpr (n >= 64) nu_scan_step<0x143, 0xC>(A, B, true);  // row_bcast:31 into rows 2 and 3
}

// Coefficients of one row (or, mirrored, of one column) of the tables.
struct NuRow {
    double b0, b1, b2, h0, h1, h2;
    __device__ __forceinline__ NuRow(const double* c, int n, int j)
        : b0(c[j]), b1(c[(n + 1) + j]), b2(c[2 * (n + 1) + j]), h0(c[3 * (n + 1) + j]),
          h1(c[4 * (n + 1) + j]), h2(c[5 * (n + 1) + j]) {}
};

// S, V and W of a column from its three rows.
template <bool HELM>
__device__ __forceinline__ void nu_svw(const NuRow& r, double u0, double u1, double u2, double m0,
                                       double m1, double m2, double& S, double& V, double& W) {
    const double q1 = HELM ? m1 * u1 : 0.0;
    S = r.b0 * u0 + r.b1 * u1 + r.b2 * u2 + q1;
    V = u1 + (r.h0 * u0 + r.h1 * u1 + r.h2 * u2);
    W = HELM ? r.h0 * (m0 * u0) + r.h1 * q1 + r.h2 * (m2 * u2) : 0.0;
}
// L u of a lane's column from its own and its neighbours' S and V (x: the
// coefficients of its column).
__device__ __forceinline__ double nu_Lu(const NuRow& x, double S, double V, double W) {
    return S + W + (x.h0 * nu_shift_up(S) + x.h1 * S + x.h2 * nu_shift_down(S)) +
           (x.b0 * nu_shift_up(V) + x.b1 * V + x.b2 * nu_shift_down(V));
}
__device__ __forceinline__ double nu_diag(double m, const NuRow& x, const NuRow& y) {
    return x.b1 + y.b1 + (x.h1 * y.b1 + y.h1 * x.b1) + (x.h1 + y.h1) * m + m;
}

// Dense [N+1][N+1] to the padded layout, boundary nodes included (J's
// boundary values enter R J at the nodes next to it).
__global__ void k_nu_copy_in(int N, int pitch, const double* __restrict__ src, double* __restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (i > N) return;
    dst[(size_t)j * pitch + i] = src[(size_t)j * (N + 1) + i];
}

// R J on the interior nodes (boundary 0) and u = 0 on the boundary.
__global__ void k_nu_rhs(int N, int pitch, const double* __restrict__ J, const double* cx,
                         const double* cy, double* __restrict__ F, double* __restrict__ u) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (i > N) return;
    const size_t g = (size_t)j * pitch + i;
    if (i == 0 || j == 0 || i == N || j == N) {
        F[g] = 0.0;
        u[g] = 0.0;
        return;
    }
    const NuRow x(cx, N, i), y(cy, N, j);
    F[g] = J[g] + (x.h0 * J[g - 1] + x.h1 * J[g] + x.h2 * J[g + 1] + y.h0 * J[g - pitch] +
                   y.h1 * J[g] + y.h2 * J[g + pitch]);
}

// The factors of every line of every level: blockIdx.y = 2 level + direction,
// 16 lines per workgroup (x-lines of rows, y-lines of columns).  For an x-line
// the coefficients of u(i-1, j), u(i, j), u(i+1, j) are
//   a_k (1 + h_0) + g_k (b_0 + M(i+k, j)) and, on the diagonal, d,
// mirrored for a y-line.  Tiles of 256 unknowns: all threads form the
// coefficients in LDS, 16 lanes run the pivots' serial chain in place (one
// reciprocal a step: v_rcp_f64 and two Newton steps), all threads write the
// factors out in their layout.  Bound by the chain, 1023 steps at 1024^2: 148 us
// for all levels, once per solve (one thread a line, storing from the chain:
// 424 us).
constexpr int kFacLines = 16, kFacTile = 256, kFacLd = kFacLines + 1;
struct NuFactorArgs {
    int n[kMaxLevels], pitch[kMaxLevels];
    const double* M[kMaxLevels];  // null: M = 0
    NuTabs t[kMaxLevels];
    NuFac f[kMaxLevels][2];
};
__global__ __launch_bounds__(256) void k_nu_factor(NuFactorArgs a) {
    __shared__ double sa[kFacTile * kFacLd], sd[kFacTile * kFacLd], sc[kFacTile * kFacLd];
    const int l = blockIdx.y >> 1, dir = blockIdx.y & 1;
    const int n = a.n[l], line0 = blockIdx.x * kFacLines, tid = threadIdx.x;
    if (line0 > n - 1) return;  // the whole workgroup
    const double* M = a.M[l];
    const size_t pitch = a.pitch[l], step = dir ? pitch : 1, across = dir ? 1 : pitch;
    const double* ct = dir ? a.t[l].cy : a.t[l].cx;  // along the line
    const double* co = dir ? a.t[l].cx : a.t[l].cy;  // across it
    const NuFac f = a.f[l][dir];
    const int per = n > 64 ? n / 64 : 1;
    double ga = 0.0;
    for (int t0 = 0; t0 < n; t0 += kFacTile) {
        const int T = min(kFacTile, n - t0);
        // dir 0: neighbouring threads along the line, dir 1: across (coalesced M)
        for (int k = tid; k < T * kFacLines; k += 256) {
            const int t = dir ? k / kFacLines : k % T, q = dir ? k % kFacLines : k / T;
            const int i = min(t0 + t + 1, n - 1), line = min(max(line0 + q, 1), n - 1);
            const NuRow x(ct, n, i), o(co, n, line);
            const size_t g = (size_t)line * across + (size_t)i * step;
            const double ml = M ? M[g - step] : 0.0, mc = M ? M[g] : 0.0, mr = M ? M[g + step] : 0.0;
            const double fy = 1.0 + o.h1;
            const bool last = t0 + t >= n - 1;  // past the end: factors 0
            sa[t * kFacLd + q] = t0 + t == 0 || last ? 0.0 : x.b0 * fy + x.h0 * (o.b1 + ml);
            sc[t * kFacLd + q] = t0 + t >= n - 2 ? 0.0 : x.b2 * fy + x.h2 * (o.b1 + mr);
            sd[t * kFacLd + q] = nu_diag(mc, x, o);
        }
        __syncthreads();
        if (tid < kFacLines) {
#pragma unroll 8
            for (int t = 0; t < T; ++t) {
                const int e = t * kFacLd + tid;
                const double sub = sa[e], sup = sc[e];
                const double p = __builtin_fma(sub, ga, sd[e]);  // d - sub (sup ib)_{t-1}
                double ib = __builtin_amdgcn_rcp(p);
                ib = __builtin_fma(__builtin_fma(-p, ib, 1.0), ib, ib);
                ib = __builtin_fma(__builtin_fma(-p, ib, 1.0), ib, ib);
                ga = -sup * ib;
                sa[e] = -sub * ib;
                sd[e] = t0 + t < n - 1 ? ib : 0.0;
                sc[e] = ga;
            }
        }
        __syncthreads();
        const int tp = T / per > 0 ? T / per : 1;  // lanes of the layout in this tile
        for (int k = tid; k < T * kFacLines; k += 256) {
            const int q = k / T, r = k % T;
            const int t = n > 64 ? (r % tp) * per + r / tp : r;
            const int line = line0 + q;
            if (line < 1 || line > n - 1) continue;
            const size_t base = (size_t)line * n;
            const int tt = t0 + t;
            const size_t o = base + (n > 64 ? (tt % per) * 64 + tt / per : tt);
            f.be[o] = sa[t * kFacLd + q];
            f.ib[o] = sd[t * kFacLd + q];
            f.ga[n > 64 ? o : base + n - 1 - tt] = sc[t * kFacLd + q];
        }
        __syncthreads();
    }
}

__device__ __forceinline__ int nu_pad(int t) { return t + (t >> 4); }

// One line of 64 PER cells by the calling wavefront: R (padded, LDS) holds the
// residual by unknown and receives T^-1 r.
template <int PER>
__device__ __forceinline__ void nu_line_solve(double* R, const NuFac& f, size_t base) {
    const int lane = threadIdx.x & 63;
    double be[PER], y[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) be[q] = f.be[base + q * 64 + lane];
#pragma unroll
    for (int q = 0; q < PER; ++q) y[q] = f.ib[base + q * 64 + lane] * R[nu_pad(lane * PER + q)];
    double A = 1.0, B = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        B = __builtin_fma(be[q], B, y[q]);
        A *= be[q];
    }
    nu_scan<64>(A, B, lane);
    double c = nu_shift_up(B);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c = __builtin_fma(be[q], c, y[q]);
        y[q] = c;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) be[q] = f.ga[base + q * 64 + lane];
    A = 1.0;
    B = 0.0;
#pragma unroll
    for (int q = PER - 1; q >= 0; --q) {
        B = __builtin_fma(be[q], B, y[q]);
        A *= be[q];
    }
    A = __shfl(A, 63 - lane, 64);
    B = __shfl(B, 63 - lane, 64);
    nu_scan<64>(A, B, lane);
    c = __shfl(nu_shift_up(B), 63 - lane, 64);
#pragma unroll
    for (int q = PER - 1; q >= 0; --q) {
        c = __builtin_fma(be[q], c, y[q]);
        R[nu_pad(lane * PER + q)] = c;
    }
}

// One zebra half step: the x-lines of every other row (DIR 0) or the y-lines of
// every other column (DIR 1), u += T^-1 (R J - L u), kNuLines lines per
// workgroup.  All wavefronts form the residual in coalesced order and hand it to
// the solve, one wavefront a line, through LDS: DIR 0, 62 nodes of a row a
// wavefront and step (the outer two lanes only feed their neighbours); DIR 1,
// the block's 9 columns, 7 rows of 9 nodes a wavefront and step, so that each
// row is read in one piece.  512 lines at 1024^2 leave two solving wavefronts a
// CU, and the kernel is bound by the latency of its loads and of the chain, so
// up to 16 wavefronts a workgroup share the residual: at 1024^2 with M 14.1 us for
// the x-lines and 27.4 us for the y-lines (9-column pieces of the rows), 7.8 /
// 13.7 at 512^2.  With parallel cyclic reduction (ten barrier-separated steps
// with two divisions each, one 512-thread workgroup a line, each y-line reading
// its column by itself) the averages over the levels were 9.2 / 20.7 us, now 8.0
// / 14.1; four wavefronts a workgroup measured 11.5 / 20.5.
template <int PER>
constexpr int nu_line_waves() { return PER <= 16 ? 16 : 8; }
template <int DIR, int PER, bool HELM>
__global__ __launch_bounds__(64 * nu_line_waves<PER>()) void k_nu_line(
    int n, int pitch, int par, double* u, const double* __restrict__ F, const double* __restrict__ M,
    const double* __restrict__ cx, const double* __restrict__ cy, NuFac fac) {
    extern __shared__ double sh[];
    constexpr int LD = 64 * PER + 4 * PER;  // padded line
    constexpr int NW = nu_line_waves<PER>(), NT = 64 * NW;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // lines first, first + 2, .. of this workgroup; neighbouring workgroups on one
    // XCD, whose L2 then serves the rows (DIR 1: the 128-byte lines) they share
    int bx, by;
    tile_of_block(bx, by);
    const int first = 2 * kNuLines * bx + (par ? 1 : 2);
    if (threadIdx.x < kNuLines) sh[threadIdx.x * LD + nu_pad(n - 1)] = 0.0;
    if (DIR == 0) {
        constexpr int G = NW / kNuLines;  // wavefronts a line
        const int k = w % kNuLines, j = first + 2 * k;
        if (j <= n - 1) {
            const NuRow y(cy, n, j);
            const size_t g0 = (size_t)j * pitch;
            constexpr int IT = ((64 * PER - 1 + 61) / 62 + G - 1) / G;
#pragma unroll
            for (int c0 = 0; c0 < IT; ++c0) {
                const int c = w / kNuLines + G * c0;
                const int i = min(62 * c + lane, n);
                const size_t g = g0 + i;
                const double u0 = u[g - pitch], u1 = u[g], u2 = u[g + pitch], f = F[g];
                const NuRow x(cx, n, i);
                double S, V, W;
                nu_svw<HELM>(y, u0, u1, u2, HELM ? M[g - pitch] : 0.0, HELM ? M[g] : 0.0,
                             HELM ? M[g + pitch] : 0.0, S, V, W);
                const double r = f - nu_Lu(x, S, V, W);
                if (lane >= 1 && lane <= 62 && 62 * c + lane <= n - 1) sh[k * LD + nu_pad(i - 1)] = r;
            }
        }
    } else {
        const int s = first - 1;  // columns s .. s + 8
        const int cc = lane % 9, rr = lane / 9;
        const int i = min(s + cc, n);
        const NuRow x(cx, n, i);
        constexpr int STEP = 7 * NW, IT = (64 * PER - 1 + STEP - 1) / STEP;
#pragma unroll 5
        for (int c = 0; c < IT; ++c) {
            const int jr = 1 + c * STEP + 7 * w + rr, j = min(jr, n - 1);
            const NuRow y(cy, n, j);
            const size_t g = (size_t)j * pitch + i;
            const double u0 = u[g - pitch], u1 = u[g], u2 = u[g + pitch], f = F[g];
            double S, V, W;
            nu_svw<HELM>(y, u0, u1, u2, HELM ? M[g - pitch] : 0.0, HELM ? M[g] : 0.0,
                         HELM ? M[g + pitch] : 0.0, S, V, W);
            const double r = f - nu_Lu(x, S, V, W);
            if ((cc & 1) && rr < 7 && jr <= n - 1) sh[(cc >> 1) * LD + nu_pad(j - 1)] = r;
        }
    }
    __syncthreads();
    if (w < kNuLines && first + 2 * w <= n - 1)
        nu_line_solve<PER>(sh + w * LD, fac, (size_t)(first + 2 * w) * n);
    __syncthreads();
    if (DIR == 0) {
#pragma unroll 4
        for (int e = threadIdx.x; e < kNuLines * 64 * PER; e += NT) {
            const int k = e / (64 * PER), t = e % (64 * PER), j = first + 2 * k;
            if (t < n - 1 && j <= n - 1) u[(size_t)j * pitch + 1 + t] += sh[k * LD + nu_pad(t)];
        }
    } else {
        const int k = threadIdx.x % kNuLines, i = first + 2 * k;
        if (i <= n - 1)
#pragma unroll 4
            for (int t = threadIdx.x / kNuLines; t < n - 1; t += NT / kNuLines)
                u[(size_t)(t + 1) * pitch + i] += sh[k * LD + nu_pad(t)];
    }
}

// Coarse right-hand side = weighted restriction of the fine residual; the
// coarse correction starts at zero.  One wavefront per coarse row and 30 coarse
// columns: the residual of its three fine rows from five rows of u (no
// intermediate array).
template <bool HELM>
__global__ __launch_bounds__(256) void k_nu_restrict(int nc, int pf, const double* __restrict__ uf,
                                                     const double* __restrict__ Ff,
                                                     const double* __restrict__ Mf, NuTabs t, int pc,
                                                     double* __restrict__ Fc, double* __restrict__ uc) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int J = blockIdx.y * 4 + w + 1, n = 2 * nc;
    if (J > nc - 1) return;
    const int i = min(60 * (int)blockIdx.x + lane, n);
    const NuRow x(t.cx, n, i);
    const size_t g = (size_t)(2 * J) * pf + i;
    double u[5], m[5], f[3];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        u[k] = uf[g + (ptrdiff_t)(k - 2) * pf];
        m[k] = HELM ? Mf[g + (ptrdiff_t)(k - 2) * pf] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) f[k] = Ff[g + (ptrdiff_t)(k - 1) * pf];
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const NuRow y(t.cy, n, 2 * J - 1 + k);
        double S, V, W;
        nu_svw<HELM>(y, u[k], u[k + 1], u[k + 2], m[k], m[k + 1], m[k + 2], S, V, W);
        v += t.ry[3 * J + k] * (f[k] - nu_Lu(x, S, V, W));
    }
    const double vl = nu_shift_up(v), vr = nu_shift_down(v);
    const int I = 30 * blockIdx.x + lane / 2;
    if (!(lane & 1) && lane >= 2 && lane <= 60 && I <= nc - 1) {
        const double* rx = t.rx + 3 * I;
        const size_t c = (size_t)J * pc + I;
        Fc[c] = rx[0] * vl + rx[1] * v + rx[2] * vr;
        uc[c] = 0.0;
    }
}

// The same weighted restriction of a node array (M), interior coarse nodes.
__global__ void k_nu_restrict_plain(int nc, int pf, const double* __restrict__ vf, const double* rx,
                                    const double* ry, int pc, double* __restrict__ vc) {
    const int I = blockIdx.x * blockDim.x + threadIdx.x, J = blockIdx.y;
    if (I > nc) return;
    double s = 0.0;
    if (I >= 1 && J >= 1 && I <= nc - 1 && J <= nc - 1)
        for (int sy = -1; sy <= 1; ++sy)
            for (int sx = -1; sx <= 1; ++sx)
                s += rx[3 * I + sx + 1] * ry[3 * J + sy + 1] * vf[(size_t)(2 * J + sy) * pf + 2 * I + sx];
    vc[(size_t)J * pc + I] = s;
}

// u_fine += prolongation of the coarse correction (interior fine nodes): at
// an odd fine index the weights of coarse I = i/2 and I + 1 are px[2i], px[2i+1].
__device__ __forceinline__ double prolong_at(const double* e, int pc, int i, int j, const double* px,
                                             const double* py) {
    const int ox = i & 1, oy = j & 1;
    const double* q = e + (size_t)(j >> 1) * pc + (i >> 1);
    const double wx0 = ox ? px[2 * i] : 1.0, wx1 = ox ? px[2 * i + 1] : 0.0;
    const double wy0 = oy ? py[2 * j] : 1.0, wy1 = oy ? py[2 * j + 1] : 0.0;
    // (at an even index the second node is the first again, with weight 0)
    return wy0 * (wx0 * q[0] + wx1 * q[ox]) + wy1 * (wx0 * q[oy * pc] + wx1 * q[oy * pc + ox]);
}

__global__ void k_nu_prolong(int nf, int pf, double* __restrict__ uf, int pc, const double* uc,
                             const double* px, const double* py) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y + 1;
    if (i < 1 || i > nf - 1) return;
    uf[(size_t)j * pf + i] += prolong_at(uc, pc, i, j, px, py);
}

// One alternating zebra line step of an n-cell level in LDS: a line lies on n
// neighbouring lanes, one unknown each.
template <int n, bool HELM>
__device__ __forceinline__ void nu_lds_lines(double* U, const double* F, const double* M, const NuTabs& t,
                                             const NuFac* fac) {
    constexpr int W = n + 1, ITEMS = n / 2 * n, IT = (ITEMS + kNuThreads - 1) / kNuThreads;
    static_assert(ITEMS % kNuThreads == 0 || ITEMS < kNuThreads, "whole trips or one");
    const int seg = threadIdx.x & (n - 1);
    const bool on = (int)(threadIdx.x & ~63) < ITEMS;  // (whole wavefronts)
    // the factors of the next half step load while this one runs
    double be[IT], ib[IT], ga[IT];
    const auto fetch = [&](int half) {
        const NuFac& f = fac[half >> 1];
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const int line = 2 * ((threadIdx.x + q * kNuThreads) / n) + ((half & 1) ? 2 : 1);
            const size_t k = (size_t)min(line, n - 1) * n + seg;
            be[q] = f.be[k];
            ib[q] = f.ib[k];
            ga[q] = f.ga[k];
        }
    };
    if (on) fetch(0);
    // lane seg holds node seg + 1 of its line (seg = n - 1: the boundary node n,
    // where S and V vanish, as they do left of node 1), so that the neighbours
    // along the line come by lane shifts; L is symmetric under an exchange of x
    // and y, so a y-line runs the same formula with the tables exchanged
    const NuRow ax(t.cx, n, seg + 1), ay(t.cy, n, seg + 1);
#pragma unroll 1
    for (int half = 0; half < 4; ++half) {
        const int dir = half >> 1;
        if (on) {
            double B[IT], G[IT];
            const int along = dir ? W : 1, across = dir ? 1 : W;
            const NuRow& x = dir ? ay : ax;
#pragma unroll
            for (int q = 0; q < IT; ++q) {
                const int line = 2 * ((threadIdx.x + q * kNuThreads) / n) + ((half & 1) ? 2 : 1);
                const int ln = min(line, n - 1), l = ln * across + (seg + 1) * along;
                const NuRow y(dir ? t.cx : t.cy, n, ln);
                double S, V, Wv;
                nu_svw<HELM>(y, U[l - across], U[l], U[l + across], HELM ? M[l - across] : 0.0,
                             HELM ? M[l] : 0.0, HELM ? M[l + across] : 0.0, S, V, Wv);
                double A = be[q];
                B[q] = ib[q] * (F[l] - nu_Lu(x, S, V, Wv));  // (ib = 0 past the end)
                nu_scan<n>(A, B[q], seg);
                G[q] = ga[q];
            }
            if (half < 3) fetch(half + 1);
            const int rev = (threadIdx.x & 63 & ~(n - 1)) + n - 1 - seg;
#pragma unroll
            for (int q = 0; q < IT; ++q) B[q] = __shfl(B[q], rev, 64);
#pragma unroll
            for (int q = 0; q < IT; ++q) {
                const int line = 2 * ((threadIdx.x + q * kNuThreads) / n) + ((half & 1) ? 2 : 1);
                nu_scan<n>(G[q], B[q], seg);
                // lane seg holds unknown n - 1 - seg: node n - seg
                if (line <= n - 1 && seg > 0) U[dir ? (n - seg) * W + line : line * W + n - seg] += B[q];
            }
        }
        __syncthreads();
    }
}

// The V-cycle from level n0 (<= kNuCoarse) down to 2 cells in one workgroup,
// in LDS: u (the initial iterate), F and M of level n0 come from global memory
// (pitch), u goes back.  tab: the tables of the levels from n0 on, one after the
// other; fac[q]: the factors of chain level q; pre, post: line steps on each level
// before and after the coarse correction.
struct NuChain {
    NuFac f[6][2];
    int pre, post;
};
template <bool HELM, int n>
__device__ void nu_chain_level(double* U, double* F, double* M, const double* tab, const NuChain& ch, int q) {
    constexpr int W = n + 1, nc = n / 2, Wc = nc + 1;
    const NuTabs t = nu_tabs_at(tab, n);
    const int tid = threadIdx.x;
    if constexpr (n == 2) {  // one interior node (1, 1)
        if (tid == 0) U[4] = F[4] / nu_diag(HELM ? M[4] : 0.0, NuRow(t.cx, 2, 1), NuRow(t.cy, 2, 1));
        __syncthreads();
    } else {
        for (int k = 0; k < ch.pre; ++k) nu_lds_lines<n, HELM>(U, F, M, t, ch.f[q]);
        double *Uc = U + W * W, *Fc = F + W * W;
        // one coarse row per n lanes, lane = fine column (as k_nu_restrict): the
        // coarse boundary is 0
        const int x_ = tid & (n - 1);
        const NuRow x(t.cx, n, x_);
        for (int J = tid / n; J <= nc; J += kNuThreads / n) {
            double s = 0.0;
            const int Jc = min(max(J, 1), nc - 1);
            double u[5], m[5], v = 0.0;
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                u[k] = U[(2 * Jc - 2 + k) * W + x_];
                m[k] = HELM ? M[(2 * Jc - 2 + k) * W + x_] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int j = 2 * Jc - 1 + k;
                const NuRow y(t.cy, n, j);
                double S, V, Wv;
                nu_svw<HELM>(y, u[k], u[k + 1], u[k + 2], m[k], m[k + 1], m[k + 2], S, V, Wv);
                v += t.ry[3 * Jc + k] * (F[j * W + x_] - nu_Lu(x, S, V, Wv));
            }
            const double vl = nu_shift_up(v), vr = nu_shift_down(v);
            const int I = x_ / 2;
            if (!(x_ & 1)) {
                if (I > 0 && J > 0 && J < nc) s = t.rx[3 * I] * vl + t.rx[3 * I + 1] * v + t.rx[3 * I + 2] * vr;
                Fc[J * Wc + I] = s;
                Uc[J * Wc + I] = 0.0;
            }
            if (x_ == 0) Fc[J * Wc + nc] = Uc[J * Wc + nc] = 0.0;
        }
        __syncthreads();
        nu_chain_level<HELM, nc>(Uc, Fc, HELM ? M + W * W : M, tab + nu_level_doubles(n), ch, q + 1);
        for (int k = tid; k < (n - 1) * (n - 1); k += kNuThreads) {
            const int i = 1 + k % (n - 1), j = 1 + k / (n - 1);
            U[j * W + i] += prolong_at(Uc, Wc, i, j, t.px, t.py);
        }
        __syncthreads();
        for (int k = 0; k < ch.post; ++k) nu_lds_lines<n, HELM>(U, F, M, t, ch.f[q]);
    }
}

template <int n0, bool HELM>
__global__ __launch_bounds__(kNuThreads) void k_nu_coarse(int pitch, double* ug,
                                                          const double* __restrict__ Fg,
                                                          const double* __restrict__ Mg,
                                                          const double* __restrict__ tab, NuChain ch) {
    __shared__ double U[kNuLdsNodes], F[kNuLdsNodes], M[HELM ? kNuLdsNodes : 1];
    __shared__ double T[nu_chain_doubles(64)];
    const int tid = threadIdx.x;
    constexpr int m = n0 + 1;
#pragma unroll
    for (int k0 = 0; k0 < m * m; k0 += kNuThreads) {
        const int k = min(k0 + tid, m * m - 1);
        const size_t g = (size_t)(k / m) * pitch + k % m;
        U[k] = ug[g];
        F[k] = Fg[g];
        if (HELM) M[k] = Mg[g];
    }
#pragma unroll
    for (int k0 = 0; k0 < nu_chain_doubles(n0); k0 += kNuThreads) {
        const int k = min(k0 + tid, nu_chain_doubles(n0) - 1);
        T[k] = tab[k];
    }
    __syncthreads();
    if (HELM) {  // M of the coarser levels, boundary 0
        double* Mf = M;
        const double* tb = T;
        for (int n = n0; n > 2; n /= 2) {
            const int nc = n / 2, Wc = nc + 1, W = n + 1;
            const NuTabs t = nu_tabs_at(tb, n);
            double* Mc = Mf + W * W;
            for (int k = tid; k < Wc * Wc; k += kNuThreads) {
                const int I = k % Wc, J = k / Wc;
                double s = 0.0;
                if (I >= 1 && J >= 1 && I <= nc - 1 && J <= nc - 1)
                    for (int sy = -1; sy <= 1; ++sy)
                        for (int sx = -1; sx <= 1; ++sx)
                            s += t.rx[3 * I + sx + 1] * t.ry[3 * J + sy + 1] * Mf[(2 * J + sy) * W + 2 * I + sx];
                Mc[k] = s;
            }
            __syncthreads();
            Mf = Mc;
            tb += nu_level_doubles(n);
        }
    }
    nu_chain_level<HELM, n0>(U, F, M, T, ch, 0);
    for (int k = tid; k < m * m; k += kNuThreads) ug[(size_t)(k / m) * pitch + k % m] = U[k];
}

// Per interior row: sum of F^2 (MODE 0) or of r^2 (MODE 1), sum of u^2, max |d|
// (MODE 0).  One workgroup a row, its wavefronts taking turns at 62 nodes.
template <int MODE, bool HELM>
__global__ __launch_bounds__(256) void k_nu_norm(int n, int pitch, const double* __restrict__ u,
                                                 const double* __restrict__ F,
                                                 const double* __restrict__ M, const double* __restrict__ cx,
                                                 const double* __restrict__ cy, double* __restrict__ part) {
    __shared__ double red[4][3];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int j = blockIdx.x + 1;
    const NuRow y(cy, n, j);
    const size_t g0 = (size_t)j * pitch;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int c = w; 62 * c < n - 1; c += 4) {
        const int i = min(62 * c + lane, n);
        const size_t g = g0 + i;
        const NuRow x(cx, n, i);
        const double u1 = u[g], f = F[g], m1 = HELM ? M[g] : 0.0;
        double v = f;
        if (MODE == 1) {
            double S, V, W;
            nu_svw<HELM>(y, u[g - pitch], u1, u[g + pitch], HELM ? M[g - pitch] : 0.0, m1,
                         HELM ? M[g + pitch] : 0.0, S, V, W);
            v = f - nu_Lu(x, S, V, W);
        }
        const bool in = lane >= 1 && lane <= 62 && 62 * c + lane <= n - 1;
        s0 += in ? v * v : 0.0;
        s1 += in ? u1 * u1 : 0.0;
        if (MODE == 0) s2 = in ? fmax(s2, fabs(nu_diag(m1, x, y))) : s2;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        s0 += __shfl_xor(s0, d, 64);
        s1 += __shfl_xor(s1, d, 64);
        s2 = fmax(s2, __shfl_xor(s2, d, 64));
    }
    if (lane < 3) red[w][lane] = lane == 0 ? s0 : lane == 1 ? s1 : s2;
    __syncthreads();
    if (threadIdx.x < 3) {
        const int k = threadIdx.x;
        part[(size_t)3 * (j - 1) + k] = k < 2 ? ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k]
                                              : fmax(fmax(red[0][2], red[1][2]), fmax(red[2][2], red[3][2]));
    }
}

// The rows' sums into the host's coherent pinned array, then (seq != 0) the
// sequence number that tells the host so.
constexpr int kNormT = 256;
__global__ __launch_bounds__(kNormT) void k_nu_norm_fin(int rows, const double* __restrict__ part,
                                                        double* out, uint32_t* dst_seq, uint32_t seq) {
    __shared__ double red[3][kNormT];
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int r = threadIdx.x; r < rows; r += kNormT) {
        s0 += part[3 * (size_t)r];
        s1 += part[3 * (size_t)r + 1];
        s2 = fmax(s2, part[3 * (size_t)r + 2]);
    }
    red[0][threadIdx.x] = s0;
    red[1][threadIdx.x] = s1;
    red[2][threadIdx.x] = s2;
    __syncthreads();
    for (int w = kNormT / 2; w >= 1; w >>= 1) {
        if (threadIdx.x < w) {
            red[0][threadIdx.x] += red[0][threadIdx.x + w];
            red[1][threadIdx.x] += red[1][threadIdx.x + w];
            red[2][threadIdx.x] = fmax(red[2][threadIdx.x], red[2][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) out[k] = red[k][0];
        if (seq) {
            __threadfence_system();
            __hip_atomic_store(dst_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// The restricted M of the levels below 64 cells: offset of level n <= 32.
size_t coarse_m_off(int n) {
    size_t o = 0;
    for (int k = 32; k > n; k /= 2) o += (size_t)(k + 1) * (k + 1);
    return o;
}

dim3 rows(int n, int t) { return dim3((n + 1 + t - 1) / t, n + 1); }

// Dxx weights and hb/3 times the dx weights of every index, 6 arrays of N + 1.
void axis_tabs(const std::vector<double>& X, double* t) {
    const int N = (int)X.size() - 1, W = N + 1;
    for (int k = 0; k < 6; ++k) t[k * W] = t[k * W + N] = 0.0;
    for (int i = 1; i < N; ++i) {
        const double hm = X[i] - X[i - 1], hp = X[i + 1] - X[i], ha = hm + hp, hb3 = (hp - hm) / 3.0;
        t[i] = 2.0 / (hm * ha);
        t[W + i] = -2.0 / (hm * hp);
        t[2 * W + i] = 2.0 / (hp * ha);
        t[3 * W + i] = hb3 * (-hp / (ha * hm));
        t[4 * W + i] = hb3 * (-hm / (ha * hp) + hp / (ha * hm));
        t[5 * W + i] = hb3 * (hm / (ha * hp));
    }
}

// restriction weights of coarse index I (fine 2I - 1, 2I, 2I + 1) and
// prolongation weights of fine index i (coarse i/2 and i/2 + 1)
void transfer_tabs(const std::vector<double>& X, double* r, double* p) {
    const int N = (int)X.size() - 1, Nc = N / 2;
    auto pw = [&](int f, bool right) {  // odd fine f: weight of its left / right coarse node
        const double lo = X[f - 1], hi = X[f + 1];
        return right ? (X[f] - lo) / (hi - lo) : (hi - X[f]) / (hi - lo);
    };
    std::fill(r, r + 3 * (size_t)(Nc + 1), 0.0);
    for (int I = 1; I < Nc; ++I) {
        const double Vc = 0.5 * (X[2 * I + 2] - X[2 * I - 2]);
        for (int s = -1; s <= 1; ++s) {
            const int f = 2 * I + s;
            const double Vf = 0.5 * (X[f + 1] - X[f - 1]);
            const double P = s == 0 ? 1.0 : pw(f, s < 0);
            r[3 * (size_t)I + s + 1] = P * Vf / Vc;
        }
    }
    std::fill(p, p + 2 * (size_t)(N + 1), 0.0);
    for (int f = 1; f < N; f += 2) {
        p[2 * (size_t)f] = pw(f, false);
        p[2 * (size_t)f + 1] = pw(f, true);
    }
}

}  // namespace

size_t nu_table_doubles(int N) {
    size_t s = 0;
    for (int n = N; n >= 2; n /= 2) s += nu_level_doubles(n);
    return s;
}

}  // namespace wq

using namespace wq;

extern "C" wandqs_status wandqs_nu_mg_solve(wandqs_ctx* c, const double* h_x, const double* h_y,
                                            const double* d_M, const double* d_J, double* d_u,
                                            int32_t* h_cycles, double* h_rel) {
    if (!c || !h_x || !h_y || !d_J || !d_u) return WANDQS_E_INVALID;
    const int N = c->N;
    for (int i = 0; i < N; ++i)
        if (!(h_x[i + 1] > h_x[i]) || !(h_y[i + 1] > h_y[i])) {
            c->err = "grid coordinates must increase";
            return WANDQS_E_INVALID;
        }
    hipStream_t s = c->stream;
    // tables of every level
    const int nlev = c->nlev;
    std::vector<std::vector<double>> X(nlev), Y(nlev);
    X[0].assign(h_x, h_x + N + 1);
    Y[0].assign(h_y, h_y + N + 1);
    for (int l = 1; l < nlev; ++l)
        for (size_t i = 0; i < X[l - 1].size(); i += 2) {
            X[l].push_back(X[l - 1][i]);
            Y[l].push_back(Y[l - 1][i]);
        }
    std::vector<double> host(nu_table_doubles(N));
    std::vector<NuTabs> tabs(nlev);
    {
        size_t o = 0;
        for (int l = 0; l < nlev; ++l) {
            const int n = N >> l;
            const NuTabs h = nu_tabs_at(host.data() + o, n);
            tabs[l] = nu_tabs_at(c->nu_tab + o, n);
            axis_tabs(X[l], const_cast<double*>(h.cx));
            axis_tabs(Y[l], const_cast<double*>(h.cy));
            if (l + 1 < nlev) {
                transfer_tabs(X[l], const_cast<double*>(h.rx), const_cast<double*>(h.px));
                transfer_tabs(Y[l], const_cast<double*>(h.ry), const_cast<double*>(h.py));
            }
            o += nu_level_doubles(n);
        }
    }
    WQ_HIP(hipMemcpyAsync(c->nu_tab, host.data(), sizeof(double) * host.size(), hipMemcpyHostToDevice, s));
    // level arrays: u, F, M (level 0: the field, f and k2 scratch; J in the
    // j_z scratch, which every slice rewrites whole: the multigrid's own
    // scratch arrays keep zero boundary values that its passes rely on)
    const int lc = c->lc;
    const bool helm = d_M != nullptr;
    auto U = [&](int l) { return l == 0 ? c->fields[0] : c->lev[l].u[0]; };
    auto Fa = [&](int l) { return c->lev[l].f[0]; };
    auto Ma = [&](int l) { return c->lev[l].k2; };
    Level& L0 = c->lev[0];
    double* Jp = c->jz;
    wandqs_status st;
    {
        {
            ProfScope ps(c, "k_nu_copy_in", (double)(N + 1) * (N + 1) * 16.0);
            WQ_KLAUNCH(ps, k_nu_copy_in, rows(N, 128), dim3(128), 0, s, N, L0.pitch, d_J, Jp);
        }
        WQ_LAUNCH_CHECK();
        double* du[1] = {U(0)};
        if ((st = unpack_fields(c, d_u, 1, du)) != WANDQS_OK) return st;
        double* dm[1] = {Ma(0)};
        if (helm && (st = unpack_fields(c, d_M, 1, dm)) != WANDQS_OK) return st;
    }
    c->tape_ok = false;  // the level arrays are the slice's scratch
    c->n_guess = 0;      // and the line factors take the place of the earlier slices' fields
    NuFactorArgs fa{};
    NuFac fac[kMaxLevels][2];
    const size_t cap = (size_t)(N + 1) * L0.pitch;
    double* pool[15];
    for (int q = 0; q < 5; ++q) {
        pool[q] = c->fields_prev[q];
        pool[5 + q] = c->fields_prev2[q];
        pool[10 + q] = c->fields_prev3[q];
    }
    static_assert(kGuessMax > 3, "three earlier generations of the fields");
    int used = 0;
    {
        size_t at = 0;
        const int nf = nlev - 1;  // every level but the 2-cell one
        for (int l = 0; l < nf; ++l) {
            const size_t n = N >> l;
            fa.n[l] = (int)n;
            fa.pitch[l] = l <= lc ? c->lev[l].pitch : 0;
            fa.t[l] = tabs[l];
            for (int d = 0; d < 2; ++d)
                for (double** f : {&fac[l][d].be, &fac[l][d].ib, &fac[l][d].ga}) {
                    if (at + n * n > cap) {
                        at = 0;
                        ++used;
                    }
                    if (used >= 15) {
                        c->err = "internal: line factors overflow";
                        return WANDQS_E_INVALID;
                    }
                    *f = pool[used] + at;
                    at += n * n;
                }
            fa.f[l][0] = fac[l][0];
            fa.f[l][1] = fac[l][1];
        }
        ++used;
    }
    {
        ProfScope ps(c, "k_nu_rhs", (double)(N + 1) * (N + 1) * 24.0);
        WQ_KLAUNCH(ps, k_nu_rhs, rows(N, 128), dim3(128), 0, s, N, L0.pitch, Jp, tabs[0].cx,
                   tabs[0].cy, Fa(0), U(0));
    }
    // M on every level; those below lc, which the coarse workgroup makes again
    // for itself in LDS, in its scratch for the factors alone
    for (int l = 1; helm && l < nlev - 1; ++l) {
        const int n = N >> l;
        double* dst = l <= lc ? Ma(l) : c->nu_coarse_m + coarse_m_off(n);
        const double* src = l - 1 <= lc ? Ma(l - 1) : c->nu_coarse_m + coarse_m_off(2 * n);
        const int ps = l - 1 <= lc ? c->lev[l - 1].pitch : 2 * n + 1, pd = l <= lc ? c->lev[l].pitch : n + 1;
        ProfScope ps_(c, "k_nu_restrict_plain", (double)(2 * n + 1) * (2 * n + 1) * 8.0 + (double)(n + 1) * (n + 1) * 8.0);
        WQ_KLAUNCH(ps_, k_nu_restrict_plain, rows(n, 128), dim3(128), 0, s, n, ps, src, tabs[l - 1].rx,
                   tabs[l - 1].ry, pd, dst);
    }
    for (int l = 0; l < nlev - 1; ++l) {
        const int n = N >> l;
        fa.M[l] = !helm ? nullptr : l <= lc ? Ma(l) : c->nu_coarse_m + coarse_m_off(n);
        if (l > lc) fa.pitch[l] = n + 1;
    }
    {
        ProfScope ps(c, "k_nu_factor", (double)(N + 1) * (N + 1) * 8.0 * (helm ? 8.0 : 6.0));
        WQ_KLAUNCH(ps, k_nu_factor, dim3((N + kFacLines - 1) / kFacLines, 2 * (nlev - 1)), dim3(256), 0, s, fa);
    }
    NuChain ch{};
    ch.pre = (c->cfg.nu_pre + 1) / 2;
    ch.post = (c->cfg.nu_post + 1) / 2;
    for (int q = 0; lc + q < nlev - 1 && q < 6; ++q)
        for (int d = 0; d < 2; ++d) ch.f[q][d] = fac[lc + q][d];
    double* hn = c->h_pin + kMaxSlots * kNormVec + 16;  // [F^2, u^2, max d, -, r^2, u^2, -]
    uint32_t* h_seq = reinterpret_cast<uint32_t*>(c->h_pin + kMaxSlots * kNormVec + 1);
    // the norms; wait: the host waits for them (published by the kernel)
    auto norms = [&](int mode, double* out, bool wait) -> wandqs_status {
        {
            ProfScope ps(c, "k_nu_norm", (double)(N + 1) * (N + 1) * ((mode ? 16.0 : 16.0) + (helm ? 8.0 : 0.0)));
            const dim3 g(N - 1), b(256);
#define WQ_NU_NORM(MODE, H) WQ_KLAUNCH(ps, (k_nu_norm<MODE, H>), g, b, 0, s, N, L0.pitch, U(0), Fa(0), Ma(0), tabs[0].cx, tabs[0].cy, c->nu_part)
            if (mode == 0) { if (helm) WQ_NU_NORM(0, true); else WQ_NU_NORM(0, false); }
            else { if (helm) WQ_NU_NORM(1, true); else WQ_NU_NORM(1, false); }
#undef WQ_NU_NORM
        }
        const uint32_t seq = wait ? ++c->pub_seq : 0;
        {
            ProfScope ps(c, "k_nu_norm_fin", 24.0 * (N - 1));
            WQ_KLAUNCH(ps, k_nu_norm_fin, dim3(1), dim3(kNormT), 0, s, N - 1, c->nu_part, out, h_seq, seq);
        }
        WQ_LAUNCH_CHECK();
        return wait ? wait_published(c, h_seq, seq) : WANDQS_OK;
    };
    // one smoothing step on a tile level: x-lines of odd and even rows, then
    // y-lines of odd and even columns (alternating zebra line relaxation)
    auto line_step = [&](int l) {
        const Level& Fl = c->lev[l];
        const int per = Fl.N / 64;
        const size_t lds = sizeof(double) * kNuLines * (size_t)(68 * per);
        const dim3 g(Fl.N / (2 * kNuLines));
        for (int dir = 0; dir < 2; ++dir)
            for (int par = 1; par >= 0; --par) {
                char nm[32];
                if (c->prof.on) std::snprintf(nm, sizeof nm, "k_nu_line<%d, %d, %s>", dir, per, helm ? "true" : "false");
                else nm[0] = 0;
                ProfScope ps(c, nm, (double)(Fl.N + 1) * (Fl.N + 1) * (24.0 + (helm ? 8.0 : 0.0)));
#define WQ_NU_LINE(D, P, H)                                                                          \
    WQ_KLAUNCH(ps, (k_nu_line<D, P, H>), g, dim3(64 * nu_line_waves<P>()), lds, s, Fl.N, Fl.pitch, par, U(l), Fa(l), Ma(l), tabs[l].cx, \
               tabs[l].cy, fac[l][D])
#define WQ_NU_LINE_P(P)                                                        \
    case P:                                                                    \
        if (dir == 0) { if (helm) WQ_NU_LINE(0, P, true); else WQ_NU_LINE(0, P, false); } \
        else { if (helm) WQ_NU_LINE(1, P, true); else WQ_NU_LINE(1, P, false); }          \
        break;
                switch (per) {
                    WQ_NU_LINE_P(2)
                    WQ_NU_LINE_P(4)
                    WQ_NU_LINE_P(8)
                    WQ_NU_LINE_P(16)
                    WQ_NU_LINE_P(32)
                    WQ_NU_LINE_P(64)
                }
#undef WQ_NU_LINE_P
#undef WQ_NU_LINE
            }
    };
    auto vcycle = [&]() -> wandqs_status {
        for (int l = 0; l < lc; ++l) {
            const Level &Fl = c->lev[l], &Cl = c->lev[l + 1];
            line_step(l);  // one alternating line step smooths like several point sweeps
            ProfScope ps(c, "k_nu_restrict", (double)(Fl.N + 1) * (Fl.N + 1) * (16.0 + (helm ? 8.0 : 0.0)) + (double)(Cl.N + 1) * (Cl.N + 1) * 16.0);
            const dim3 g((Cl.N - 1 + 29) / 30, (Cl.N - 1 + 3) / 4), b(256);
            if (helm)
                WQ_KLAUNCH(ps, k_nu_restrict<true>, g, b, 0, s, Cl.N, Fl.pitch, U(l), Fa(l), Ma(l), tabs[l],
                           Cl.pitch, Fa(l + 1), U(l + 1));
            else
                WQ_KLAUNCH(ps, k_nu_restrict<false>, g, b, 0, s, Cl.N, Fl.pitch, U(l), Fa(l), Ma(l), tabs[l],
                           Cl.pitch, Fa(l + 1), U(l + 1));
        }
        {
            const Level& Cl = c->lev[lc];
            ProfScope ps(c, "k_nu_coarse", (double)(Cl.N + 1) * (Cl.N + 1) * (24.0 + (helm ? 8.0 : 0.0)));
#define WQ_NU_COARSE(n)                                                                                     \
    case n:                                                                                                 \
        if (helm) WQ_KLAUNCH(ps, (k_nu_coarse<n, true>), dim3(1), dim3(kNuThreads), 0, s, Cl.pitch, U(lc),   \
                             Fa(lc), Ma(lc), tabs[lc].cx, ch);                                              \
        else WQ_KLAUNCH(ps, (k_nu_coarse<n, false>), dim3(1), dim3(kNuThreads), 0, s, Cl.pitch, U(lc),       \
                        Fa(lc), Ma(lc), tabs[lc].cx, ch);                                                   \
        break;
            switch (Cl.N) {
                WQ_NU_COARSE(64)
                WQ_NU_COARSE(32)
                WQ_NU_COARSE(16)
                WQ_NU_COARSE(8)
            }
#undef WQ_NU_COARSE
        }
        for (int l = lc - 1; l >= 0; --l) {
            const Level &Fl = c->lev[l], &Cl = c->lev[l + 1];
            {
                ProfScope ps(c, "k_nu_prolong", (double)(Fl.N + 1) * (Fl.N + 1) * 16.0 + (double)(Cl.N + 1) * (Cl.N + 1) * 8.0);
                WQ_KLAUNCH(ps, k_nu_prolong, dim3((Fl.N + 1 + 255) / 256, Fl.N - 1), dim3(256), 0, s, Fl.N,
                           Fl.pitch, U(l), Cl.pitch, U(l + 1), tabs[l].px, tabs[l].py);
            }
            line_step(l);
        }
        WQ_LAUNCH_CHECK();
        return WANDQS_OK;
    };
    if (lc > 0) {
        // the largest level's lines in LDS (above 64 KiB only at 2048^2 and 4096^2)
        const int per = N / 64, bytes = (int)(sizeof(double) * kNuLines * (size_t)(68 * per));
        if (bytes > 65536) {
            const void* k[8] = {(const void*)k_nu_line<0, 32, false>, (const void*)k_nu_line<0, 32, true>,
                                (const void*)k_nu_line<1, 32, false>, (const void*)k_nu_line<1, 32, true>,
                                (const void*)k_nu_line<0, 64, false>, (const void*)k_nu_line<0, 64, true>,
                                (const void*)k_nu_line<1, 64, false>, (const void*)k_nu_line<1, 64, true>};
            for (int q = 0; q < 8; ++q)
                WQ_HIP(hipFuncSetAttribute(k[q], hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
        }
    }
    if ((st = norms(0, hn, false)) != WANDQS_OK || (st = norms(1, hn + 4, true)) != WANDQS_OK) return st;
    const double fn = std::sqrt(hn[0]), amax = hn[2];
    double rn = std::sqrt(hn[4]), rprev = rn;
    const double tol = c->cfg.mg_rtol * (fn > 0 ? fn : rn) + c->cfg.mg_atol * std::sqrt((double)(N - 1) * (N - 1));
    const double scale = fn > 0 ? fn : rn;
    const double floor_be = kFloorBE * std::numeric_limits<double>::epsilon();
    bool done = rn <= tol;
    int cyc = 0;
    while (!done && cyc < c->cfg.mg_max_cycles) {
        if ((st = vcycle()) != WANDQS_OK) return st;
        ++cyc;
        if ((st = norms(1, hn + 4, true)) != WANDQS_OK) return st;
        rprev = rn;
        rn = std::sqrt(hn[4]);
        const double un = std::sqrt(hn[5]);
        done = rn <= tol || rn <= floor_be * (2.0 * amax * un + fn) ||
               (cyc >= 2 && rn > 0.9 * rprev && rn <= 1e-9 * scale);
    }
    if ((st = pack_fields(c, c->fields, 1, d_u)) != WANDQS_OK) return st;
    // no infinities or NaN stay in the arrays lent to the factors (their
    // padding is read and masked by a product with 0 once they hold fields again):
    // a cycle with undefined factors leaves an undefined residual; without a cycle
    // nothing has told of them
    for (int q = 0; q < used && !(cyc > 0 && std::isfinite(rn)); ++q)
        if ((st = fill_f64(c, pool[q], cap, 0.0)) != WANDQS_OK) return st;
    WQ_HIP(hipStreamSynchronize(s));
    if (h_cycles) *h_cycles = cyc;
    if (h_rel) *h_rel = fn > 0 ? rn / fn : rn;
    if (!(done && std::isfinite(rn))) {
        c->err = "non-uniform multigrid did not converge";
        return WANDQS_E_NOCONV;
    }
    return WANDQS_OK;
}
