// Exact Poisson solve by fast sine transforms, FP64, of eqs. (12)-(15), Sec.
// III.B (the five-point operator of Sec. VII.B on a uniform grid): on the
// finest level as the whole solve (TOP: iterations u += L_h^-1 (f - L_h u) of
// the tolerance mode), and on the level just below the finest as the
// coarse-grid correction of the Poisson V-cycles (fixed-cycle mode, grids
// above 2048^2).
//
// With zero Dirichlet values the five-point Laplacian of an n x n-cell level
// of spacing H has the eigenvectors sin(pi i k / n) sin(pi j l / n) (1 <= k, l
// <= n - 1) and the eigenvalues -(4 / H^2) (sin^2(pi k / 2n) + sin^2(pi l / 2n)),
// so u = (2/n)^2 S (S f S ./ lambda) S with the sine matrix S.
//
// The sine transform X_k = sum_{j=1}^{n-1} x_j sin(pi j k / n) of one real row
// comes from the real DFT Y of length n of
//     y_j = sin(pi j / n) (x_j + x_{n-j}) + (x_j - x_{n-j}) / 2   (x_0 = x_n = 0):
// the symmetric part x_j + x_{n-j}, weighted by sin(pi j / n), turns
// cos(2 pi j k / n) into a difference of odd-frequency sines and the
// antisymmetric part gives the even-frequency ones, so
//     X_2k = -Im Y_k,   X_2k+1 = X_2k-1 + Re Y_k   (X_1 = Re Y_0 / 2),
// the odd coefficients a prefix sum.  Y comes from one complex FFT of length
// n/2 of z_m = y_2m + i y_2m+1 (Y_k = E_k + W_n^k O_k, E and O the transforms
// of the even and odd samples, from Z_k and conj(Z_{n/2-k})).
//
// One wavefront transforms one row: a Stockham (self-sorting) radix-4 FFT
// (one radix-2 stage last for an odd power of two) whose stages exchange
// through LDS (one pad slot per 16 doubles) with no workgroup barrier, since a
// wavefront's LDS operations complete in order.  Three launches; T1 and T2 are
// stored transposed, so that every pass reads whole rows and only the writes
// of the first two are scattered (two or four rows per workgroup, written together):
//   x: row g of f -> column g of T1 (T1[k-1][g-1] = coefficient k);
//   y: row k-1 of T1 -> transform, divide by lambda, transform back ->
//      column k-1 of T2 (T2[j-1][k-1], j the y-node);
//   x inverse: row j-1 of T2 -> row j of u.
// A first form with two rows packed into one complex FFT of length 2n (the
// odd extensions; 256 threads and a barrier per stage) measured 9.7 / 6.6 /
// 5.3 us for the y / x inverse / x passes at n = 512, this one 7.5 / 5.4 /
// 5.4.  TOP at n = 1024, averaged over one and two right-hand sides: x 16.1,
// y 20.0, x inverse 11.7 us (2.3, 1.3 and 3.2 TB/s of its bytes; the transposed
// writes and, in y, the registers bound the first two); at n = 512 6.3 / 7.1 /
// 4.7.  With two LDS buffers per wavefront and the table's entries kept in scratch
// they took 23.6 / 23.2 / 13.2 and 6.8 / 7.3 / 4.8; y at n = 1024 without the bound
// of two wavefronts per SIMD (17 registers spilled) 21.4.
#include <cstdio>

#include "wq_common.h"

namespace wq {
namespace {

template <typename E>
struct FstArgs {
    int pitch;  // row stride of f and u
    int ld;     // row stride of T1 and T2
    const E* f[2];
    double* t1[2];
    double* t2[2];
    E* u[2];
    const double2* tw;  // exp(-2 pi i m / 2n), m < 2n
    const double* s2;   // sin^2(pi k / (2n)), k <= n
    double lam;         // -4 / H^2
    double scale;       // (2 / n)^2
    // TOP (the whole solve on the finest level): 1 / H^2 and the norm sums of
    // the incoming iterate, [3 r + q][nblk] with one entry per row
    double ih2;
    double* norm_part;
    int nblk;
};

// In-register DFT of length R (2 or 4), natural order in and out.
template <int R>
__device__ __forceinline__ void dft(double (&re)[R], double (&im)[R]) {
    static_assert(R == 2 || R == 4, "radix");
    if constexpr (R == 2) {
        const double ar = re[0], ai = im[0];
        re[0] = ar + re[1];
        im[0] = ai + im[1];
        re[1] = ar - re[1];
        im[1] = ai - im[1];
    } else {
        // X_q = sum_s x_s (-i)^(s q)
        const double s0r = re[0] + re[2], s0i = im[0] + im[2];
        const double d0r = re[0] - re[2], d0i = im[0] - im[2];
        const double s1r = re[1] + re[3], s1i = im[1] + im[3];
        const double d1r = re[1] - re[3], d1i = im[1] - im[3];
        re[0] = s0r + s1r;
        im[0] = s0i + s1i;
        re[2] = s0r - s1r;
        im[2] = s0i - s1i;
        re[1] = d0r + d1i;  // d0 - i d1
        im[1] = d0i - d1r;
        re[3] = d0r - d1i;  // d0 + i d1
        im[3] = d0i + d1r;
    }
}

// LDS slot of element i of a padded buffer
__device__ __forceinline__ int pidx(int i) { return i + (i >> 4); }

__device__ __forceinline__ double2 ld2(const double* p) { return *reinterpret_cast<const double2*>(p); }

// TOP, x pass: the residual f - L_h u of one row (u and f point at it) into V
// (padded; V[0] = 0) and the lane's sums of r^2, f^2, u^2 over its nodes.
// Lane l takes the pairs (2m, 2m + 1), m = l + 64 q, in batches whose loads are
// all in flight together (row starts are 64-byte aligned: 16-byte loads).
template <int PER>
__device__ __forceinline__ void residual_row(const double* u, const double* f, int pitch, double ih2,
                                             double* V, double (&s)[3]) {
    constexpr int CH = PER < 4 ? PER : 4;
    const int lane = threadIdx.x & 63;
    s[0] = s[1] = s[2] = 0.0;
#pragma unroll
    for (int q0 = 0; q0 < PER; q0 += CH) {
        double2 c[CH], up[CH], dn[CH], fv[CH];
        double lf[CH], rt[CH];
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int j = 2 * (lane + 64 * (q0 + q));
            c[q] = ld2(u + j);
            up[q] = ld2(u + j - pitch);
            dn[q] = ld2(u + j + pitch);
            fv[q] = ld2(f + j);
            lf[q] = u[max(j - 1, 0)];
            rt[q] = u[j + 2];
        }
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int j = 2 * (lane + 64 * (q0 + q));
            const double in = j > 0 ? 1.0 : 0.0;  // node 0 is a boundary node
            const double r0 = in * (fv[q].x - (lf[q] + c[q].y + up[q].x + dn[q].x - 4.0 * c[q].x) * ih2);
            const double r1 = fv[q].y - (c[q].x + rt[q] + up[q].y + dn[q].y - 4.0 * c[q].y) * ih2;
            V[pidx(j)] = r0;
            V[pidx(j + 1)] = r1;
            s[0] += r0 * r0 + r1 * r1;
            s[1] += in * fv[q].x * fv[q].x + fv[q].y * fv[q].y;
            s[2] += in * c[q].x * c[q].x + c[q].y * c[q].y;
        }
    }
}

// Twiddle W_L^m (m < L) from the table of W_L^m, m < L / 2 (W_L^(m + L/2) = -W_L^m).
template <int L>
__device__ __forceinline__ double2 twiddle(const double2* tw, int m) {
    if (m < L / 2) return tw[m];
    const double2 v = tw[m - L / 2];
    return double2{-v.x, -v.y};
}

template <int LOGN>
struct FstSize {
    static constexpr int n = 1 << LOGN;
    static constexpr int H = n / 2;                 // complex FFT length
    static constexpr int PER = H / 64;              // Y coefficients per lane (chunk)
    static constexpr int NB = (H / 4 + 63) / 64;    // first-stage butterflies per lane
    static constexpr int LP = H + H / 16;           // padded FFT buffer
    static_assert(PER >= 1, "n >= 128");
};

// One radix-R Stockham stage of the length-H FFT run by one wavefront:
// butterfly j (lane + 64 b) takes X[j + s H / R] (s < R; src(t, b, s) gives
// input t) times W_(NS R)^(k s), k = j mod NS, and puts its DFT at
// (j - k) R + k + q NS.  The twiddles W_(NS R)^(k s) = W_n^(2 k s H / (NS R))
// come from the LDS table T of W_n^m, m < H.
// Every input is read before the first output is written, so that a stage may
// work in place (half the LDS of two buffers, twice the wavefronts in flight).
template <int H, int R, int NS, class Src>
__device__ __forceinline__ void wstage(const Src& src, double* yr, double* yi, const double2* T) {
    constexpr int NBF = H / R, NBL = (NBF + 63) / 64;
    double vr[NBL][R], vi[NBL][R];
#pragma unroll
    for (int b = 0; b < NBL; ++b) {
        const int j = min((int)(threadIdx.x & 63) + 64 * b, NBF - 1);
        const int k = j & (NS - 1);
#pragma unroll
        for (int s = 0; s < R; ++s) {
            const double2 x = src(j + s * (H / R), b, s);
            if (NS > 1 && s > 0) {
                const double2 w = twiddle<2 * H>(T, 2 * (k * s * (H / (NS * R))));
                vr[b][s] = x.x * w.x - x.y * w.y;
                vi[b][s] = x.x * w.y + x.y * w.x;
            } else {
                vr[b][s] = x.x;
                vi[b][s] = x.y;
            }
        }
        dft<R>(vr[b], vi[b]);
    }
    wave_sync();
#pragma unroll
    for (int b = 0; b < NBL; ++b) {
        const int j = (threadIdx.x & 63) + 64 * b;
        if (NBF % 64 != 0 && j >= NBF) break;
        const int k = j & (NS - 1), base = (j - k) * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            yr[pidx(base + q * NS)] = vr[b][q];
            yi[pidx(base + q * NS)] = vi[b][q];
        }
    }
}

template <int H, int NS, class Src>
__device__ __forceinline__ void wfft(const Src& src, double* yr, double* yi, const double2* T) {
    constexpr int R = H / NS >= 4 ? 4 : H / NS;
    wstage<H, R, NS>(src, yr, yi, T);
    wave_sync();
    if constexpr (NS * R < H) {
        const auto lds = [yr, yi](int t, int, int) { return double2{yr[pidx(t)], yi[pidx(t)]}; };
        wfft<H, NS * R>(lds, yr, yi, T);
    }
}

// Sine transform of the row x (get(j) = x_j for j in 1 .. n-1, called with
// clamped indices only) by the lane: xe[q] = X_2k, xo[q] = X_2k+1 for
// k = lane PER + q.  sn[b][s][e] = sin(pi j / n) of the lane's sample
// j = 2m + e (m = the first-stage input of butterfly b, leg s), loaded by the
// caller.  buf: 2 LP doubles of LDS (get may read it: its loads come first).
// STORE: the lane's entries tvr + i tvi of the LDS table T (T[lane + 64 q]) are
// stored once the row's loads are issued, so that both sets of loads overlap.
template <int LOGN, bool STORE, class Get>
__device__ __forceinline__ void wdst(const Get& get, const double (&sn)[FstSize<LOGN>::NB][4][2],
                                     double* buf, double2* T, const double (&tvr)[FstSize<LOGN>::PER],
                                     const double (&tvi)[FstSize<LOGN>::PER],
                                     double (&xe)[FstSize<LOGN>::PER], double (&xo)[FstSize<LOGN>::PER]) {
    using F = FstSize<LOGN>;
    constexpr int n = F::n, H = F::H, NB = F::NB, PER = F::PER, LP = F::LP;
    const int lane = threadIdx.x & 63;
    // first-stage inputs z_m, m = min(lane + 64 b, H/4 - 1) + s H/4; every load
    // issued before any is used (indices clamped, zero ends masked after)
    double xa[NB][4][2], xb[NB][4][2];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int m = min(lane + 64 * b, H / 4 - 1) + s * (H / 4);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int j = 2 * m + e;  // 0 .. n-1; n - j in 1 .. n
                xa[b][s][e] = get(max(j, 1)) * (j >= 1 ? 1.0 : 0.0);
                xb[b][s][e] = get(min(n - j, n - 1)) * (j >= 1 ? 1.0 : 0.0);
            }
        }
    if (STORE)
#pragma unroll
        for (int q = 0; q < PER; ++q) T[lane + 64 * q] = double2{tvr[q], tvi[q]};
    wave_sync();
    double2 z[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            double y[2];
#pragma unroll
            for (int e = 0; e < 2; ++e)
                y[e] = sn[b][s][e] * (xa[b][s][e] + xb[b][s][e]) + 0.5 * (xa[b][s][e] - xb[b][s][e]);
            z[b][s] = double2{y[0], y[1]};
        }
    double *zr = buf, *zi = buf + LP;
    wfft<H, 1>([&](int, int b, int s) { return z[b][s]; }, zr, zi, T);
    // Y_k over the lane's chunk, then the prefix sum of Re Y (Re Y_0 halved)
    double rs[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int k = lane * PER + q, km = (H - k) & (H - 1);
        const double ar = zr[pidx(k)], ai = zi[pidx(k)], br = zr[pidx(km)], bi = zi[pidx(km)];
        const double er = 0.5 * (ar + br), ei = 0.5 * (ai - bi);
        const double orr = 0.5 * (ai + bi), oi = -0.5 * (ar - br);
        const double2 w = T[k];
        const double yr = er + w.x * orr - w.y * oi, yi = ei + w.x * oi + w.y * orr;
        xe[q] = -yi;
        rs[q] = (k == 0 ? 0.5 : 1.0) * yr;
    }
    double run = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        run += rs[q];
        rs[q] = run;
    }
    double incl = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double t = __shfl_up(incl, d, 64);
        incl += lane >= d ? t : 0.0;
    }
    const double excl = incl - run;
#pragma unroll
    for (int q = 0; q < PER; ++q) xo[q] = excl + rs[q];
    wave_sync();  // the caller may overwrite buf next
}

// MODE 0: x pass; MODE 1: y pass; MODE 2: x inverse (see above).  A
// workgroup holds RW wavefronts, wavefront w transforming row RW b + w
// (0-based interior; b the block) of right-hand side r; a wavefront past the
// last row transforms the last row again and writes nothing.  With RW > 1 the
// transposed writes of MODE 0 and 1 go through LDS, RW consecutive rows'
// values of one coefficient written together.
// TOP (E = double): the level is the finest one and the pass belongs to a
// whole Poisson solve: the x pass transforms the residual f - L_h u of the
// incoming iterate, formed row by row in LDS, and records its norms; the
// inverse x pass adds the correction to u.
template <typename E, int LOGN, int MODE, int RW, bool TOP>
__global__ __launch_bounds__(64 * RW, (LOGN == 10 ? 2 : 1)) void k_fst(FstArgs<E> a) {
    using F = FstSize<LOGN>;
    constexpr int n = F::n, H = F::H, NB = F::NB, PER = F::PER, LP = F::LP;
    __shared__ double bufs[RW][2 * LP];
    __shared__ double2 T[H];
    int pb, r;
    tile_of_block(pb, r);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool live = pb * RW + w < n - 1;
    const int p = live ? pb * RW + w : n - 2;
    double* buf = bufs[w];
    // tables: W_n^m (m < H) = W_2n^2m into LDS; the lane's sin(pi j / n) =
    // -Im W_2n^j; for MODE 1 its sin^2(pi l / 2n) and that of k = p + 1
    double tvr[PER], tvi[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        tvr[q] = a.tw[2 * (lane + 64 * q)].x;
        tvi[q] = a.tw[2 * (lane + 64 * q)].y;
    }
    double sn[NB][4][2];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int m = min(lane + 64 * b, H / 4 - 1) + s * (H / 4);
                sn[b][s][e] = -a.tw[2 * m + e].y;
            }
    double s2e[MODE == 1 ? PER : 1], s2o[MODE == 1 ? PER : 1], s2k = 0.0;
    if constexpr (MODE == 1) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            s2e[q] = a.s2[2 * k];
            s2o[q] = a.s2[2 * k + 1];
        }
        s2k = a.s2[p + 1];
    }
    const size_t ld = a.ld;
    double xe[PER], xo[PER];
    if constexpr (MODE == 0 && TOP) {
        double* V = buf;
        double s[3];
        residual_row<PER>(a.u[r] + (size_t)(p + 1) * a.pitch, a.f[r] + (size_t)(p + 1) * a.pitch,
                          a.pitch, a.ih2, V, s);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
            for (int q = 0; q < 3; ++q) s[q] += __shfl_xor(s[q], d, 64);
        if (lane < 3 && live)
            a.norm_part[(size_t)(3 * r + lane) * a.nblk + p] = lane == 0 ? s[0] : lane == 1 ? s[1] : s[2];
#pragma unroll
        for (int q = 0; q < PER; ++q) T[lane + 64 * q] = double2{tvr[q], tvi[q]};
        wave_sync();
        const auto get = [=](int j) { return V[pidx(j)]; };
        wdst<LOGN, false>(get, sn, buf, T, tvr, tvi, xe, xo);
    } else if (MODE == 0) {
        const E* row = a.f[r] + (size_t)(p + 1) * a.pitch;
        const auto get = [=](int j) { return (double)row[j]; };
        wdst<LOGN, true>(get, sn, buf, T, tvr, tvi, xe, xo);
    } else {
        const double* row = (MODE == 1 ? a.t1 : a.t2)[r] + (size_t)p * ld - 1;
        const auto get = [=](int j) { return row[j]; };
        wdst<LOGN, true>(get, sn, buf, T, tvr, tvi, xe, xo);
    }
    if constexpr (MODE == 1) {
        // coefficient (k, l) over its eigenvalue, into LDS by l (V[0] = 0),
        // then transformed back along y
        double* V = buf;
        const double lam = a.lam, lk = lam * s2k;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            V[pidx(2 * k)] = k == 0 ? 0.0 : xe[q] / (lk + lam * s2e[q]);
            V[pidx(2 * k + 1)] = xo[q] / (lk + lam * s2o[q]);
        }
        wave_sync();
        const auto get = [=](int j) { return V[pidx(j)]; };
        wdst<LOGN, false>(get, sn, buf, T, tvr, tvi, xe, xo);
    }
    if (MODE < 2 && RW == 1) {
        // coefficient c (1 .. n-1) of this row to T[c - 1][p]
        double* Tt = (MODE == 0 ? a.t1 : a.t2)[r] + p;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int c = 2 * (lane * PER + q);
            if (c >= 1) Tt[(size_t)(c - 1) * ld] = xe[q];
            Tt[(size_t)c * ld] = xo[q];
        }
    } else if (MODE < 2) {
        // the RW rows' coefficients through LDS: T[c - 1][RW b .. RW b + RW - 1]
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            buf[pidx(2 * k)] = xe[q];
            buf[pidx(2 * k + 1)] = xo[q];
        }
        __syncthreads();
        double* Tt = (MODE == 0 ? a.t1 : a.t2)[r] + pb * RW;
        for (int i = threadIdx.x; i < (n - 1) * RW; i += 64 * RW) {
            const int c = 1 + i / RW, ww = i % RW;
            if (pb * RW + ww < n - 1) Tt[(size_t)(c - 1) * ld + ww] = bufs[ww][pidx(c)];
        }
    } else if constexpr (TOP) {
        // u += scale X through LDS: coalesced pairs, as residual_row
        double* V = buf;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            V[pidx(2 * k)] = k == 0 ? 0.0 : xe[q];
            V[pidx(2 * k + 1)] = xo[q];
        }
        wave_sync();
        const double sc = a.scale;
        double* row = a.u[r] + (size_t)(p + 1) * a.pitch;
        double2 uv[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) uv[q] = ld2(row + 2 * (lane + 64 * q));
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int j = 2 * (lane + 64 * q);
            uv[q].x += sc * V[pidx(j)];
            uv[q].y += sc * V[pidx(j + 1)];
            *reinterpret_cast<double2*>(row + j) = uv[q];
        }
    } else {
        E* u = a.u[r];
        E* row = u + (size_t)(p + 1) * a.pitch;
        const double sc = a.scale;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int c = 2 * (lane * PER + q);
            row[c] = c == 0 ? E(0) : (E)(sc * xe[q]);
            row[c + 1] = (E)(sc * xo[q]);
        }
        if (lane == 63) row[n] = E(0);
        if (p == 0)
            for (int x = lane; x <= n; x += 64) {
                u[x] = E(0);
                u[(size_t)n * a.pitch + x] = E(0);
            }
    }
}

// Rows per workgroup of the x and y passes, whose transposed writes then go
// out in 16-byte pieces: TOP at n = 512 measured 6.3 / 7.1 us with 2 rows, 6.9 /
// 7.6 with 1 and 8.2 / 7.8 with 4; at n = 1024, where the writes count more, 4
// rows 16.1 / 21.4, 2 rows 18.0 / 24.2; at n = 2048 the x and y passes below a
// finest level of 4096^2 37.6 / 64.2 with 4 rows, 43.1 / 74.0 with 2 and 62.4 /
// 82.4 with 1 (the same bits in every case)
#ifndef WQ_FST_ROWS
#define WQ_FST_ROWS 2
#endif

template <typename E, int LOGN, bool TOP>
void launch_fst(wandqs_ctx* c, const FstArgs<E>& a, int R, const char* tname) {
    constexpr int n = 1 << LOGN;
    constexpr int RW = LOGN >= 10 ? 2 * WQ_FST_ROWS : WQ_FST_ROWS;
    const dim3 g(n - 1, R), gw((n - 1 + RW - 1) / RW, R);
    const double nodes = (double)(n - 1) * (n - 1) * R;
    const double eb = sizeof(E);
    char nm[64];
    {
        std::snprintf(nm, sizeof nm, "k_fst<%s, x>@%d", tname, n);
        ProfScope ps(c, nm, nodes * (eb + 8.0 + (TOP ? 8.0 : 0.0)));
        WQ_KLAUNCH(ps, (k_fst<E, LOGN, 0, RW, TOP>), gw, dim3(64 * RW), 0, c->stream, a);
    }
    {
        std::snprintf(nm, sizeof nm, "k_fst<%s, y>@%d", tname, n);
        ProfScope ps(c, nm, nodes * 16.0);
        WQ_KLAUNCH(ps, (k_fst<E, LOGN, 1, RW, TOP>), gw, dim3(64 * RW), 0, c->stream, a);
    }
    {
        std::snprintf(nm, sizeof nm, "k_fst<%s, xinv>@%d", tname, n);
        ProfScope ps(c, nm, nodes * (8.0 + eb + (TOP ? 8.0 : 0.0)));
        WQ_KLAUNCH(ps, (k_fst<E, LOGN, 2, 1, TOP>), g, dim3(64), 0, c->stream, a);
    }
}

// ------------------------------------------------- laser envelope planes --

// One iteration u += (L_h - kbar)^-1 (f - (L_h - k) u) of a laser envelope plane
// (complex, (re, im) pairs): L_h - kbar with a constant kbar = kr - i gam is
// diagonal under the sine transform, eigenvalue lambda_kl - kr + i gam.  The
// passes are those of k_fst on the real and the imaginary part of a row, one
// wavefront each: T1 and T2 hold (re, im) pairs, so that the transposed writes
// of the x and y passes go out in 32-byte pieces (two rows per workgroup), and
// the y pass exchanges the parts' coefficients through LDS for the complex
// division.  At 512^2 x 7.1, y 9.8, x inverse 5.8 us (2.4, 0.85 and 2.2 TB/s of
// its bytes; the two transforms of the y pass and its scattered writes bound
// that one).  A plane of a pulse with the plasma behind its front (512^2) takes
// 6 of these instead of 9.4 V-cycles of 95 us: its time step of 20 planes 31.2
// -> 15.5 ms.
struct LasFstArgs {
    int pitch, ld;
    const double2* f;
    const double2* k;
    double2* u;
    double* t1;
    double* t2;
    const double2* tw;
    const double* s2;
    double lam, scale, ih2;
    double kr, gam;
};

template <int LOGN, int MODE>
constexpr int las_rows() { return MODE < 2 && LOGN <= 10 ? 2 : 1; }

template <int LOGN, int MODE>
__global__ __launch_bounds__((128 * las_rows<LOGN, MODE>())) void k_las_fst(LasFstArgs a) {
    using F = FstSize<LOGN>;
    constexpr int n = F::n, H = F::H, NB = F::NB, PER = F::PER, LP = F::LP;
    constexpr int RW = las_rows<LOGN, MODE>();
    __shared__ double bufs[2 * RW][2 * LP];
    __shared__ double2 T[H];
    int pb, r0;
    tile_of_block(pb, r0);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, part = w & 1, t = threadIdx.x & 127;
    const bool live = pb * RW + (w >> 1) < n - 1;
    const int p = live ? pb * RW + (w >> 1) : n - 2;
    double* buf = bufs[w];
    double *V0 = bufs[w & ~1], *V1 = bufs[w | 1];  // the row's real and imaginary part
    double tvr[PER], tvi[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        tvr[q] = a.tw[2 * (lane + 64 * q)].x;
        tvi[q] = a.tw[2 * (lane + 64 * q)].y;
    }
    double sn[NB][4][2];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int m = min(lane + 64 * b, H / 4 - 1) + s * (H / 4);
                sn[b][s][e] = -a.tw[2 * m + e].y;
            }
    const size_t ld = a.ld;
    double xe[PER], xo[PER];
    if constexpr (MODE == 0) {
        // the row's residual, node j = t + 128 q (node 0 is a boundary node)
        const size_t g0 = (size_t)(p + 1) * a.pitch;
        const double2 *u = a.u + g0, *f = a.f + g0, *k = a.k + g0;
        constexpr int Q = n / 128, CH = Q < 2 ? Q : 2;
#pragma unroll
        for (int q0 = 0; q0 < Q; q0 += CH) {
            double2 c[CH], l[CH], r[CH], up[CH], dn[CH], fv[CH], kv[CH];
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                const int j = t + 128 * (q0 + q);
                c[q] = u[j];
                l[q] = u[max(j - 1, 0)];
                r[q] = u[j + 1];
                up[q] = u[j - a.pitch];
                dn[q] = u[j + a.pitch];
                fv[q] = f[j];
                kv[q] = k[j];
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                const int j = t + 128 * (q0 + q);
                const double in = j > 0 ? 1.0 : 0.0;
                const double lx = a.ih2 * (l[q].x + r[q].x + up[q].x + dn[q].x - 4.0 * c[q].x);
                const double ly = a.ih2 * (l[q].y + r[q].y + up[q].y + dn[q].y - 4.0 * c[q].y);
                V0[pidx(j)] = in * (fv[q].x - (lx - (kv[q].x * c[q].x - kv[q].y * c[q].y)));
                V1[pidx(j)] = in * (fv[q].y - (ly - (kv[q].x * c[q].y + kv[q].y * c[q].x)));
            }
        }
        __syncthreads();
        const auto get = [=](int j) { return buf[pidx(j)]; };
        wdst<LOGN, true>(get, sn, buf, T, tvr, tvi, xe, xo);
    } else {
        const double* row = (MODE == 1 ? a.t1 : a.t2) + 2 * ((size_t)p * ld - 1) + part;
        const auto get = [=](int j) { return row[2 * j]; };
        wdst<LOGN, true>(get, sn, buf, T, tvr, tvi, xe, xo);
    }
    if constexpr (MODE == 1) {
        // coefficient (k, l) over its eigenvalue er + i gam, then back along y
        const double lk = a.lam * a.s2[p + 1] - a.kr;
        const double sg = part ? -a.gam : a.gam;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            buf[pidx(2 * k)] = xe[q];
            buf[pidx(2 * k + 1)] = xo[q];
        }
        __syncthreads();
        const double* o = bufs[w ^ 1];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            const double e0 = lk + a.lam * a.s2[2 * k], e1 = lk + a.lam * a.s2[2 * k + 1];
            xe[q] = k == 0 ? 0.0 : (xe[q] * e0 + sg * o[pidx(2 * k)]) / (e0 * e0 + sg * sg);
            xo[q] = (xo[q] * e1 + sg * o[pidx(2 * k + 1)]) / (e1 * e1 + sg * sg);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = lane * PER + q;
            buf[pidx(2 * k)] = xe[q];
            buf[pidx(2 * k + 1)] = xo[q];
        }
        wave_sync();
        const auto get = [=](int j) { return buf[pidx(j)]; };
        wdst<LOGN, false>(get, sn, buf, T, tvr, tvi, xe, xo);
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int k = lane * PER + q;
        buf[pidx(2 * k)] = k == 0 ? 0.0 : xe[q];
        buf[pidx(2 * k + 1)] = xo[q];
    }
    __syncthreads();
    if constexpr (MODE < 2) {
        // coefficient c (1 .. n-1) of the workgroup's rows: T[c - 1][row] = (re, im)
        double* Tt = (MODE == 0 ? a.t1 : a.t2) + 2 * (size_t)(pb * RW);
        for (int i = threadIdx.x; i < (n - 1) * 2 * RW; i += 128 * RW) {
            const int c = 1 + i / (2 * RW), ww = i % (2 * RW);
            if (pb * RW + (ww >> 1) < n - 1) Tt[2 * (size_t)(c - 1) * ld + ww] = bufs[ww][pidx(c)];
        }
    } else {
        double2* row = a.u + (size_t)(p + 1) * a.pitch;
        constexpr int Q = n / 128;
        double2 uv[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) uv[q] = row[t + 128 * q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j = t + 128 * q;
            uv[q].x += a.scale * V0[pidx(j)];
            uv[q].y += a.scale * V1[pidx(j)];
            row[j] = uv[q];
        }
    }
}

template <int LOGN>
void launch_las_fst(wandqs_ctx* c, const LasFstArgs& a) {
    constexpr int n = 1 << LOGN, RW = las_rows<LOGN, 0>();
    const double nodes = (double)(n - 1) * (n - 1);
    const dim3 gw((n - 1 + RW - 1) / RW);
    {
        ProfScope ps(c, "k_las_fst<x>", nodes * 64.0);
        WQ_KLAUNCH(ps, (k_las_fst<LOGN, 0>), gw, dim3(128 * RW), 0, c->stream, a);
    }
    {
        ProfScope ps(c, "k_las_fst<y>", nodes * 32.0);
        WQ_KLAUNCH(ps, (k_las_fst<LOGN, 1>), gw, dim3(128 * RW), 0, c->stream, a);
    }
    {
        ProfScope ps(c, "k_las_fst<xinv>", nodes * 48.0);
        WQ_KLAUNCH(ps, (k_las_fst<LOGN, 2>), dim3(n - 1), dim3(128), 0, c->stream, a);
    }
}

__global__ void k_fst_tables(int L, double2* tw, double* s2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < L) {
        double sv, cv;
        sincospi(-2.0 * i / L, &sv, &cv);
        tw[i] = double2{cv, sv};
    }
    if (i <= L / 2) {
        const double s = sinpi((double)i / L);  // sin(pi k / (2n)), L = 2n
        s2[i] = s * s;
    }
}

}  // namespace

bool fst_used(const wandqs_ctx* c) {
    return c->lc >= 2 && c->lev[1].N >= kFstMinN && c->lev[1].N <= kFstMaxN;
}

size_t fst_ld(const wandqs_ctx* c) { return (size_t)c->lev[1].N + 8; }

bool fst_top_used(const wandqs_ctx* c) { return c->N >= kFstMinN && c->N <= kFstMaxN; }

wandqs_status make_fst_tables(wandqs_ctx* c) {
    const auto make = [c](int n, double2* tw, double* s2) {
        const int L = 2 * n;
        hipLaunchKernelGGL(k_fst_tables, dim3(L / 256 + 1), dim3(256), 0, c->stream, L, tw, s2);
    };
    if (fst_used(c)) make(c->lev[1].N, c->fst_tw, c->fst_s2);
    if (c->fst_top_tw) make(c->N, c->fst_top_tw, c->fst_top_s2);
    WQ_LAUNCH_CHECK();
    return WANDQS_OK;
}

void fst_top_iteration(wandqs_ctx* c, int R, const double* const* f, double* const* u,
                       double* norm_part) {
    const Level& L0 = c->lev[0];
    FstArgs<double> a{};
    a.pitch = L0.pitch;
    a.ld = L0.N + 8;
    for (int r = 0; r < R; ++r) {
        a.f[r] = f[r];
        a.u[r] = u[r];
        a.t1[r] = c->fst_t1[r];
        a.t2[r] = c->fst_t2[r];
    }
    a.tw = c->fst_top_tw;
    a.s2 = c->fst_top_s2;
    a.lam = -4.0 / (L0.h * L0.h);
    a.scale = (2.0 / L0.N) * (2.0 / L0.N);
    a.ih2 = 1.0 / (L0.h * L0.h);
    a.norm_part = norm_part;
    a.nblk = L0.N - 1;
    switch (L0.N) {
        case 128: launch_fst<double, 7, true>(c, a, R, "top"); break;
        case 256: launch_fst<double, 8, true>(c, a, R, "top"); break;
        case 512: launch_fst<double, 9, true>(c, a, R, "top"); break;
        case 1024: launch_fst<double, 10, true>(c, a, R, "top"); break;
        default: launch_fst<double, 11, true>(c, a, R, "top"); break;
    }
}

void las_fst_iteration(wandqs_ctx* c, const double2* f, const double2* k, double2* u, double kr, double gam) {
    const Level& L0 = c->lev[0];
    LasFstArgs a{};
    a.pitch = L0.pitch;
    a.ld = L0.N + 8;
    a.f = f;
    a.k = k;
    a.u = u;
    a.t1 = c->fst_t1[0];  // the two right-hand sides' arrays, contiguous
    a.t2 = c->fst_t2[0];
    a.tw = c->fst_top_tw;
    a.s2 = c->fst_top_s2;
    a.lam = -4.0 / (L0.h * L0.h);
    a.scale = (2.0 / L0.N) * (2.0 / L0.N);
    a.ih2 = 1.0 / (L0.h * L0.h);
    a.kr = kr;
    a.gam = gam;
    switch (L0.N) {
        case 128: launch_las_fst<7>(c, a); break;
        case 256: launch_las_fst<8>(c, a); break;
        case 512: launch_las_fst<9>(c, a); break;
        case 1024: launch_las_fst<10>(c, a); break;
        default: launch_las_fst<11>(c, a); break;
    }
}

template <typename E>
void fst_solve(wandqs_ctx* c, int R, const E* const* f, E* const* u) {
    const Level& L1 = c->lev[1];
    FstArgs<E> a{};
    a.pitch = L1.pitch;
    a.ld = (int)fst_ld(c);
    for (int r = 0; r < R; ++r) {
        a.f[r] = f[r];
        a.u[r] = u[r];
        a.t1[r] = c->fst_t1[r];
        a.t2[r] = c->fst_t2[r];
    }
    a.tw = c->fst_tw;
    a.s2 = c->fst_s2;
    a.lam = -4.0 / (L1.h * L1.h);
    a.scale = (2.0 / L1.N) * (2.0 / L1.N);
    const char* tn = sizeof(E) == 8 ? "double" : "float";
    switch (L1.N) {
        case 128: launch_fst<E, 7, false>(c, a, R, tn); break;
        case 256: launch_fst<E, 8, false>(c, a, R, tn); break;
        case 512: launch_fst<E, 9, false>(c, a, R, tn); break;
        case 1024: launch_fst<E, 10, false>(c, a, R, tn); break;
        default: launch_fst<E, 11, false>(c, a, R, tn); break;
    }
}

template void fst_solve<double>(wandqs_ctx*, int, const double* const*, double* const*);
template void fst_solve<float>(wandqs_ctx*, int, const float* const*, float* const*);

}  // namespace wq
