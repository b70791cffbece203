// Node-array kernels of one slice: the right-hand sides of the Ez and Bz
// Poisson equations (WAND-PIC Sec. III.B eqs. (13)-(14)), the longitudinal
// current with the frozen driver, the B_perp Helmholtz system (eqs. (18)-(19),
// rows 4-5 of eq. (30) with the laser envelope absent), probes and layout
// conversion between the padded internal arrays and the dense interface arrays.
#include <algorithm>
#include <cmath>

#include "wq_common.h"

namespace wq {
namespace {

// f_Ez = -(D_x jx + D_y jy), f_Bz = D_x jy - D_y jx on the interior nodes.
__global__ void k_rhs_EB(int N, double h, int pitch, const double* __restrict__ jx,
                         const double* __restrict__ jy, double* __restrict__ fE,
                         double* __restrict__ fB) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (a > N) return;
    const size_t g = (size_t)b * pitch + a;
    double e = 0.0, m = 0.0;
    if (a >= 1 && b >= 1 && a <= N - 1 && b <= N - 1) {
        const double i2h = 1.0 / (2.0 * h);
        const double dxjx = (jx[g + 1] - jx[g - 1]) * i2h;
        const double dyjy = (jy[g + pitch] - jy[g - pitch]) * i2h;
        const double dxjy = (jy[g + 1] - jy[g - 1]) * i2h;
        const double dyjx = (jx[g + pitch] - jx[g - pitch]) * i2h;
        e = -(dxjx + dyjy);
        m = dxjy - dyjx;
    }
    fE[g] = e;
    fB[g] = m;
}

// Driver density at node (a, b) = (x, y).  Radial-bin membership comes from the
// node map built on the host, so bin edges are decided exactly once.
__device__ double beam_density(const BeamSet& B, double x, double y, size_t node, double xi) {
    if (xi < 0.0) return 0.0;
    double s = 0.0;
    for (int k = 0; k < B.n; ++k) {
        const double lz = (xi - B.xc[k]) * (xi - B.xc[k]) / (B.sz[k] * B.sz[k]);
        if (B.kind[k] == 0) {
            const double rx = x - B.x0[k], ry = y - B.y0[k];
            const double r2 = rx * rx + ry * ry;
            s += B.amp[k] * exp(-r2 / (B.sr[k] * B.sr[k]) - lz);
        } else {
            const int kb = B.bmap[k][node];
            if (kb >= 0) s += B.bins[k][kb] * exp(-lz);
        }
    }
    return s;
}

// Node (a, b) inside the disc of radius r around (x0, y0); every operation
// rounded separately so that host and device agree on the edge.
__device__ bool in_disc(double L, double h, int a, int b, double x0, double y0, double r) {
#pragma clang fp contract(off)
    const double rx = (-L + a * h) - x0, ry = (-L + b * h) - y0;
    return rx * rx + ry * ry <= r * r;
}

// Current of the driver macroparticles (time loop) at a node and slice
// position xi: the fixed-point deposit planes interpolated linearly in xi
// (zero outside them).
struct DriverPlanes {
    const unsigned long long* p;  // nullptr: no driver particles in this sweep
    int nz;
    double xi0, dz;
    size_t plane;  // words per plane
};

__device__ __forceinline__ double driver_current(const DriverPlanes& D, size_t i, double xi) {
    if (!D.p) return 0.0;
    const double t = (xi - D.xi0) / D.dz;
    const int m = (int)floor(t);
    if (m < 0 || m > D.nz - 2) return 0.0;
    const double a = t - m;
    constexpr double kUnfix = 1.0 / 1099511627776.0;  // one unit of the planes: 2^-40
    const double v0 = (double)(long long)D.p[(size_t)m * D.plane + i] * kUnfix;
    const double v1 = (double)(long long)D.p[(size_t)(m + 1) * D.plane + i] * kUnfix;
    return (1.0 - a) * v0 + a * v1;
}

// Total j_z on every node: plasma n*<p_z>/g = G/g - n* with G = n*<gamma> =
// [n*(1 + g^2 + a2/2) + g^2 (Txx + Tyy)]/(2g) (eq. (9) and the gamma of Sec.
// III.A, <p_perp^2> = g^2 <V^2>, a2 = |A-hat|^2 of a laser envelope or 0 when
// a2 is null), plus the frozen drivers' density at xi (luminal beam current)
// and the driver macroparticles' current (time loop).
__global__ void k_jz(int N, double L, double h, int pitch, const double* __restrict__ n,
                     const double* __restrict__ txx, const double* __restrict__ tyy,
                     const double* __restrict__ psi, const double* __restrict__ a2,
                     const double* __restrict__ st, BeamSet beams, DriverPlanes drv,
                     double* __restrict__ jz, double* __restrict__ k2,
                     int32_t* __restrict__ flags) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (a > N) return;
    const size_t i = (size_t)b * pitch + a;
    // every load unconditional and the plasma term selected after (a load
    // behind the n* > 0 branch would be waited for inside it)
    const double ni = n[i], g = 1.0 + psi[i], tt = txx[i] + tyy[i];
    const double q = a2 ? 0.5 * a2[i] : 0.0;
    if (ni > 0.0 && !(g > 0.0)) atomicOr(flags, 1);
    const double G = (ni * (1.0 + g * g + q) + g * g * tt) / (2.0 * g);
    const double v = ni > 0.0 ? G / g - ni : 0.0;
    jz[i] = v + beam_density(beams, -L + a * h, -L + b * h, (size_t)b * (N + 1) + a, st[0]) +
            driver_current(drv, i, st[0]);
    // k2 = n* / g of the B_perp Helmholtz system (eqs. (18)-(19)) on the
    // interior nodes (it reads neither E_z nor B_z)
    const bool interior = a >= 1 && b >= 1 && a <= N - 1 && b <= N - 1;
    k2[i] = interior && ni > 0.0 ? ni / g : 0.0;
}

// The B_perp right-hand sides on the interior nodes (k_jz writes k2 = n* / g):
//   f_Bx = D_y(j_z - Tyy) - D_x Txy + (jx Bz - jy Ez)/g + (G/g^2 - Tyy/g) psi_y - (Txy/g) psi_x
//          - n* D_y(a2/4)/g^2
//   f_By = D_x(Txx - j_z) + D_y Txy + (jy Bz + jx Ez)/g - (G/g^2 - Txx/g) psi_x + (Txy/g) psi_y
//          + n* D_x(a2/4)/g^2
// (G as in k_jz; the a2 terms are the ponderomotive part of S, present when a2
// is not null).
__global__ void k_assemble(int N, double h, int pitch, const double* __restrict__ n,
                           const double* __restrict__ jx, const double* __restrict__ jy,
                           const double* __restrict__ txx, const double* __restrict__ txy,
                           const double* __restrict__ tyy, const double* __restrict__ psi,
                           const double* __restrict__ Ez, const double* __restrict__ Bz,
                           const double* __restrict__ jz, const double* __restrict__ a2,
                           double* __restrict__ fBx, double* __restrict__ fBy) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (a > N) return;
    const size_t i = (size_t)b * pitch + a;
    double fx = 0.0, fy = 0.0;
    if (a >= 1 && b >= 1 && a <= N - 1 && b <= N - 1) {
        const double i2h = 1.0 / (2.0 * h);
        const size_t e = i + 1, w = i - 1, nn = i + pitch, s = i - pitch;
        const double g = 1.0 + psi[i];
        const double psx = (psi[e] - psi[w]) * i2h, psy = (psi[nn] - psi[s]) * i2h;
        fx = ((jz[nn] - tyy[nn]) - (jz[s] - tyy[s])) * i2h - (txy[e] - txy[w]) * i2h;
        fy = ((txx[e] - jz[e]) - (txx[w] - jz[w])) * i2h + (txy[nn] - txy[s]) * i2h;
        if (n[i] > 0.0) {
            const double q = a2 ? 0.5 * a2[i] : 0.0;
            const double G = (n[i] * (1.0 + g * g + q) + g * g * (txx[i] + tyy[i])) / (2.0 * g);
            fx += (jx[i] * Bz[i] - jy[i] * Ez[i]) / g + (G / (g * g) - tyy[i] / g) * psy -
                  (txy[i] / g) * psx;
            fy += (jy[i] * Bz[i] + jx[i] * Ez[i]) / g - (G / (g * g) - txx[i] / g) * psx +
                  (txy[i] / g) * psy;
            if (a2) {
                fx -= n[i] * (0.25 * ((a2[nn] - a2[s]) * i2h)) / (g * g);
                fy += n[i] * (0.25 * ((a2[e] - a2[w]) * i2h)) / (g * g);
            }
        }
    }
    fBx[i] = fx;
    fBy[i] = fy;
}

// Probe k adds the mean of its field over its disc (fixed summation order, one
// block).  The nodes looked at are the W x H ones from (a0, b0) on, the disc's
// bounding box: over the whole grid the serial chain of trips took 29 us at 256^2
// for a disc of a tenth of the box, now 5 us.
constexpr int kProbeThreads = 1024;
__global__ __launch_bounds__(kProbeThreads) void k_probe(int a0, int b0, int W, int H, double L, double h,
                                                         int pitch, const double* __restrict__ F, double x0,
                                                         double y0, double rmax, double scale,
                                                         double* __restrict__ acc) {
    constexpr int NW = kProbeThreads / 64;
    __shared__ double red[2][NW];
    double s = 0.0, cnt = 0.0;
    for (int i = threadIdx.x; i < W * H; i += kProbeThreads) {
        const int b = b0 + i / W, a = a0 + i % W;
        if (in_disc(L, h, a, b, x0, y0, rmax)) {
            s += F[(size_t)b * pitch + a];
            cnt += 1.0;
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        s += __shfl_xor(s, off, 64);
        cnt += __shfl_xor(cnt, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = s;
        red[1][threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double S = 0.0, C = 0.0;
        for (int w = 0; w < NW; ++w) {
            S += red[0][w];
            C += red[1][w];
        }
        if (C > 0) *acc += scale * S / C;
    }
}

// Adjoint seed of a probe: Fb += w on the interior nodes of its disc (the
// boundary values are fixed, their adjoints never propagate).
__global__ void k_probe_seed(int N, double L, double h, int pitch, double x0, double y0,
                             double rmax, double w, double* __restrict__ Fb) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = blockIdx.y;
    if (a < 1 || a > N - 1 || b < 1 || b > N - 1) return;
    if (in_disc(L, h, a, b, x0, y0, rmax)) Fb[(size_t)b * pitch + a] += w;
}

// Dense [N+1][N+1] interface arrays <-> padded node arrays, one of them per
// blockIdx.z: a call's arrays in one launch (each launch of its own cost 4 us on
// small grids).
constexpr int kMaxNodeArrays = 9;
struct NodeArrays {
    const double* src[kMaxNodeArrays];
    double* dst[kMaxNodeArrays];
};

__global__ void k_pack(int N, int pitch, NodeArrays p) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = blockIdx.y, k = blockIdx.z;
    if (a > N) return;
    p.dst[k][(size_t)b * (N + 1) + a] = p.src[k][(size_t)b * pitch + a];
}

__global__ void k_unpack(int N, int pitch, NodeArrays p) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int b = blockIdx.y, k = blockIdx.z;
    if (a > N) return;
    const bool bnd = a == 0 || b == 0 || a == N || b == N;
    p.dst[k][(size_t)b * pitch + a] = bnd ? 0.0 : p.src[k][(size_t)b * (N + 1) + a];
}

// Initial guesses for the five solves of this slice: the fields u of the last
// slice (at xi_0), extrapolated to xi through the slices before (p1 at xi_1,
// p2 at xi_2, p3 at xi_3) -- order 0: u; order m: the Lagrange polynomial of
// degree m through u, p1, ..., pm.  The guess goes to `out` (the oldest
// array, which the host then rotates into the field's place).
struct FieldPtrs {
    const double* u[5];
    const double* p1[5];
    const double* p2[5];
    const double* p3[5];
    double* out[5];
};

// The first LINEAR fields extrapolate through the last two slices only (weight
// w[0] of p1): the exact solve of psi, E_z and B_z reaches the rounding floor in
// one iteration from there as well, and their older history need not be read (at
// 1024^2 35.4 -> 26.9 us; from u itself some slices took two).  Steps of many times a
// workload's own bring second iterations, never a third: a slice of 1082 instead of
// 1061 us at 1024^2 with ten times the step (1.8 instead of 1.1 iterations for E_z and
// B_z), 393 and 394 at 256^2 with ten times, 372 and 383 with five.  Every load of a
// node is issued before the first is used.
template <int ORDER, int LINEAR>
__device__ __forceinline__ void extrapolate_node(const FieldPtrs& f, size_t g, const double* w) {
    double u[5], p[5][3];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        u[k] = f.u[k][g];
        if (ORDER >= 1) p[k][0] = f.p1[k][g];
        if (k >= LINEAR) {
            if (ORDER >= 2) p[k][1] = f.p2[k][g];
            if (ORDER >= 3) p[k][2] = f.p3[k][g];
        }
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        double v = u[k];
        if (k < LINEAR) {
            if (ORDER >= 1) v = u[k] + w[0] * (p[k][0] - u[k]);
        } else {
            if (ORDER == 1) v = u[k] + w[1] * (p[k][0] - u[k]);
            if (ORDER == 2) v = u[k] + (w[1] * (p[k][0] - u[k]) + w[2] * (p[k][1] - u[k]));
            if (ORDER == 3)
                v = u[k] + (w[1] * (p[k][0] - u[k]) + w[2] * (p[k][1] - u[k]) + w[3] * (p[k][2] - u[k]));
        }
        f.out[k][g] = v;
    }
}

// Every workgroup forms the Lagrange weights w[m] of p_m relative to u (w[0]: of p1
// in the linear form) for itself (thread m; a launch for them alone cost 4 us a slice): the order drops while two
// of the points coincide.
constexpr int kExtraThreads = 128;
template <int LINEAR>
__global__ __launch_bounds__(kExtraThreads) void k_extrapolate(int N, int pitch, const double* __restrict__ st,
                                                               int order, FieldPtrs f) {
    __shared__ double w[4];
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const double x[4] = {st[2], st[3], st[4], st[5]};
    const auto differ = [&x](int n) {  // points 0 .. n are all different
        bool ok = true;
#pragma unroll
        for (int i = 1; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < i; ++j) ok = ok && (i > n || x[i] != x[j]);
        return ok;
    };
    while (order > 0 && !differ(order)) --order;
    if (threadIdx.x < 4) {
        const int i = max((int)threadIdx.x, 1), deg = threadIdx.x == 0 ? 1 : order;
        const double xi = st[0], xm = st[2 + i];
        double l = 1.0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j <= deg && j != i) l *= (xi - x[j]) / (xm - x[j]);
        w[threadIdx.x] = l;
    }
    __syncthreads();
    if (a > N) return;
    const size_t g = (size_t)blockIdx.y * pitch + a;
    if (order >= 3) extrapolate_node<3, LINEAR>(f, g, w);
    else if (order == 2) extrapolate_node<2, LINEAR>(f, g, w);
    else if (order == 1) extrapolate_node<1, LINEAR>(f, g, w);
    else extrapolate_node<0, LINEAR>(f, g, w);
}

__global__ void k_fill(double* p, size_t n, double v) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

dim3 node_grid(int N) { return dim3((N + 1 + 127) / 128, N + 1); }

}  // namespace

wandqs_status rhs_EB(wandqs_ctx* c) {
    const Level& L0 = c->lev[0];
    {
        ProfScope ps(c, "k_rhs_EB", (double)(c->N + 1) * (c->N + 1) * 32.0);
        WQ_KLAUNCH(ps, k_rhs_EB, node_grid(c->N), dim3(128), 0, c->stream, c->N, c->h, L0.pitch,
                           c->mom[1], c->mom[2], L0.f[0], L0.f[1]);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

wandqs_status plasma_jz(wandqs_ctx* c) {
    const Level& L0 = c->lev[0];
    {
        const DriverPlanes drv{c->drv_active ? c->drv_planes : nullptr, c->drv_nz, c->cfg.driver_xi0,
                               c->cfg.driver_dz, (size_t)(c->N + 1) * L0.pitch};
        ProfScope ps(c, "k_jz", (double)(c->N + 1) * (c->N + 1) * 48.0);
        WQ_KLAUNCH(ps, k_jz, node_grid(c->N), dim3(128), 0, c->stream, c->N, c->L, c->h, L0.pitch,
                           c->mom[0], c->mom[3], c->mom[5], c->fields[0],
                           c->las_on ? c->las_a2 : nullptr, c->st, c->beamset, drv, c->jz, L0.k2,
                           c->flags);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

// jz_ready: plasma_jz has run already (it does not read E_z or B_z).
wandqs_status assemble(wandqs_ctx* c, bool jz_ready) {
    const Level& L0 = c->lev[0];
    if (!jz_ready) {
        const wandqs_status s = plasma_jz(c);
        if (s != WANDQS_OK) return s;
    }
    {
        ProfScope ps(c, "k_assemble", (double)(c->N + 1) * (c->N + 1) * 96.0);
        WQ_KLAUNCH(ps, k_assemble, node_grid(c->N), dim3(128), 0, c->stream, c->N, c->h, L0.pitch,
                           c->mom[0], c->mom[1], c->mom[2], c->mom[3], c->mom[4], c->mom[5],
                           c->fields[0], c->fields[1], c->fields[2], c->jz,
                           c->las_on ? c->las_a2 : nullptr, L0.f[0], L0.f[1]);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

wandqs_status probes_accumulate(wandqs_ctx* c, int64_t slice) {
    for (size_t k = 0; k < c->probes.size(); ++k) {
        const wandqs_probe& p = c->probes[k];
        if (slice < p.slice_begin || slice >= p.slice_end) continue;
        const double scale = 1.0 / (double)(p.slice_end - p.slice_begin);
        // nodes lo .. hi along an axis hold every node within r_max of x (and one more a side)
        const auto range = [c](double x, double r, int& lo, int& n) {
            const auto clamped = [c](double v) { return !(v > 0.0) ? 0 : v < c->N ? (int)v : c->N; };
            lo = clamped(std::floor((x - r + c->L) / c->h) - 1.0);
            n = std::max(clamped(std::ceil((x + r + c->L) / c->h) + 1.0) - lo + 1, 1);
        };
        int a0, b0, W, H;
        range(p.x0, p.r_max, a0, W);
        range(p.y0, p.r_max, b0, H);
        {
            ProfScope ps(c, "k_probe", (double)W * H * 8.0);
            WQ_KLAUNCH(ps, k_probe, dim3(1), dim3(kProbeThreads), 0, c->stream, a0, b0, W, H, c->L, c->h,
                               c->lev[0].pitch, c->fields[p.field], p.x0, p.y0, p.r_max, scale,
                               c->probe_acc + k);
        }
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

wandqs_status probe_seed(wandqs_ctx* c, int k, double w, double* const* Fb) {
    const wandqs_probe& p = c->probes[k];
    {
        ProfScope ps(c, "k_probe_seed", (double)(c->N + 1) * (c->N + 1) * 16.0);
        WQ_KLAUNCH(ps, k_probe_seed, node_grid(c->N), dim3(128), 0, c->stream, c->N, c->L, c->h,
                           c->lev[0].pitch, p.x0, p.y0, p.r_max, w, Fb[p.field]);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

wandqs_status pack_fields(wandqs_ctx* c, double* const* src, int n, double* dst) {
    const size_t nn = (size_t)(c->N + 1) * (c->N + 1);
    NodeArrays p{};
    for (int k = 0; k < n; ++k) {
        p.src[k] = src[k];
        p.dst[k] = dst + k * nn;
    }
    dim3 g = node_grid(c->N);
    g.z = n;
    {
        ProfScope ps(c, "k_pack", (double)nn * 16.0 * n);
        WQ_KLAUNCH(ps, k_pack, g, dim3(128), 0, c->stream, c->N, c->lev[0].pitch, p);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

namespace {
wandqs_status unpack(wandqs_ctx* c, int n, const NodeArrays& p) {
    dim3 g = node_grid(c->N);
    g.z = n;
    {
        ProfScope ps(c, "k_unpack", (double)(c->N + 1) * (c->N + 1) * 16.0 * n);
        WQ_KLAUNCH(ps, k_unpack, g, dim3(128), 0, c->stream, c->N, c->lev[0].pitch, p);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}
}  // namespace

wandqs_status unpack_fields(wandqs_ctx* c, const double* src, int n, double* const* dst) {
    const size_t nn = (size_t)(c->N + 1) * (c->N + 1);
    NodeArrays p{};
    for (int k = 0; k < n; ++k) {
        p.src[k] = src + k * nn;
        p.dst[k] = dst[k];
    }
    return unpack(c, n, p);
}

wandqs_status unpack_solve(wandqs_ctx* c, int nrhs, const double* f, const double* u, const double* k2) {
    const size_t nn = (size_t)(c->N + 1) * (c->N + 1);
    NodeArrays p{};
    int n = 0;
    for (int r = 0; r < nrhs; ++r) {
        p.src[n] = f + r * nn;
        p.dst[n++] = c->lev[0].f[r];
        p.src[n] = u + r * nn;
        p.dst[n++] = c->fields[r];
    }
    if (k2) {
        p.src[n] = k2;
        p.dst[n++] = c->lev[0].k2;
    }
    return unpack(c, n, p);
}

wandqs_status extrapolate_guess(wandqs_ctx* c, int order) {
    FieldPtrs f;
    double* const* oldest = kGuessMax > 3 ? c->fields_prev3 : c->fields_prev2;
    for (int k = 0; k < 5; ++k) {
        f.u[k] = c->fields[k];
        f.p1[k] = c->fields_prev[k];
        f.p2[k] = c->fields_prev2[k];
        f.p3[k] = kGuessMax > 3 ? c->fields_prev3[k] : c->fields_prev2[k];
        f.out[k] = oldest[k];
    }
    order = order < 0 ? 0 : (order > kGuessMax - 1 ? kGuessMax - 1 : order);
    {
        const bool lin = direct_poisson(c, false);
        ProfScope ps(c, "k_extrapolate", (double)(c->N + 1) * (c->N + 1) * 8.0 * (lin ? 3 * (std::min(order, 1) + 2) + 2 * (order + 2) : 5 * (order + 2)));
        if (lin)
            WQ_KLAUNCH(ps, k_extrapolate<3>, node_grid(c->N), dim3(kExtraThreads), 0, c->stream, c->N,
                       c->lev[0].pitch, c->st, order, f);
        else
            WQ_KLAUNCH(ps, k_extrapolate<0>, node_grid(c->N), dim3(kExtraThreads), 0, c->stream, c->N,
                       c->lev[0].pitch, c->st, order, f);
    }
    WQ_LAUNCH_CHECK();
    for (int k = 0; k < 5; ++k) {  // oldest <- ... <- prev <- u <- guess
        double* g = oldest[k];
        if (kGuessMax > 3) c->fields_prev3[k] = c->fields_prev2[k];
        c->fields_prev2[k] = c->fields_prev[k];
        c->fields_prev[k] = c->fields[k];
        c->fields[k] = g;
    }
    return WANDQS_OK;
}

wandqs_status copy_d2d(wandqs_ctx* c, void* dst, const void* src, size_t bytes) {
    WQ_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, c->stream));
    return WANDQS_OK;
}

wandqs_status fill_f64(wandqs_ctx* c, double* p, size_t n, double v) {
    if (n == 0) return WANDQS_OK;
    {
        ProfScope ps(c, "k_fill", 8.0 * n);
        WQ_KLAUNCH(ps, k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, p, n, v);
    }
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

}  // namespace wq
