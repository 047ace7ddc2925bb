// gfx950 FP64 particle loader: drifting Maxwell-Juttner momenta by the method
// of Melzani et al., "Apar-T" (arXiv:1308.5892), Sect. 4.3 and App. D, with
// co-located pairs (Sect. 2.1) and the relativistic Harris sheet (App. C).
//
// The p_y marginal (App. D, eq. distr_y) is tabulated as an inverse CDF in
// FP64 on the device: Gauss-Legendre integrals over a fine grid, a block scan,
// and a safeguarded Newton solve for each quantile.  Each pair then draws its
// position and two momenta from a counter-based Philox4x64-10 stream.
#include <hip/hip_runtime.h>

#include "pic_internal.h"

namespace pic {

// ------------------------------------------------------------ Philox4x64-10

// Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as easy as 1, 2, 3"
// (SC'11): ten rounds; each multiplies counter words 0 and 2 by fixed odd
// constants, swaps halves and xors in words 1 and 3 and the round key; the key
// advances by two Weyl increments between rounds.
__device__ inline void philox4x64_10(uint64_t ctr[4], uint64_t k0, uint64_t k1)
{
    constexpr uint64_t kMulA = 0xD2E7470EE14C6C93ull, kMulB = 0xCA5A826395121157ull;
    constexpr uint64_t kWeylA = 0x9E3779B97F4A7C15ull, kWeylB = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t hA = __umul64hi(kMulA, ctr[0]), lA = kMulA * ctr[0];
        const uint64_t hB = __umul64hi(kMulB, ctr[2]), lB = kMulB * ctr[2];
        const uint64_t w0 = hB ^ ctr[1] ^ k0, w2 = hA ^ ctr[3] ^ k1;
        ctr[0] = w0; ctr[1] = lB; ctr[2] = w2; ctr[3] = lA;
        k0 += kWeylA;
        k1 += kWeylB;
    }
}

__device__ inline double unit53(uint64_t w) { return (double)(w >> 11) * (1.0 / 9007199254740992.0); }

// ------------------------------------------------- p_y marginal and its table

struct MJShape {
    double mu, G, beta0;   // 1/theta, Gamma0, beta0
};

// App. D, eq. distr_y without its constant factor, scaled by exp(mu) so that it
// is O(1) at the drift momentum y = Gamma0 beta0.
__device__ inline double py_density(double y, const MJShape &m)
{
    const double gy = sqrt(1.0 + y * y);
    return (1.0 + m.mu * m.G * gy) * exp(m.mu - m.mu * m.G * (gy - m.beta0 * y));
}

// five-point Gauss-Legendre integral of the density over [a, b]
__device__ inline double py_integral(double a, double b, const MJShape &m)
{
    const double x1 = 0.5384693101056831, x2 = 0.9061798459386640;
    const double w0 = 0.5688888888888889, w1 = 0.4786286704993665, w2 = 0.2369268850561891;
    const double c = 0.5 * (a + b), h = 0.5 * (b - a);
    return h * (w0 * py_density(c, m) + w1 * (py_density(c - h * x1, m) + py_density(c + h * x1, m)) +
                w2 * (py_density(c - h * x2, m) + py_density(c + h * x2, m)));
}

// Up to two populations' tables are built by the same launches (blockIdx.y).
struct MJTable {
    MJShape m;
    double ylo, yhi, h;
    double *cum, *tab;
};
struct MJTables {
    MJTable t[2];
};

// The integral of each of the M intervals and its prefix sum, compensated
// (Kahan) and always in the same order, so that a table does not depend on the
// launch: within chunks of kMjChunk intervals, then over the chunks' totals.
// cum[i + 1] gets the sum over interval i's chunk up to i, cum[M + 1 + c] the
// total of chunk c; mj_offsets_kernel adds the chunks before.  (One block that
// read all 65536 intervals with a stride and had one thread for the 1024 totals
// took 190 us per table, half of the time of a small load; these two take 26.)
__global__ void __launch_bounds__(kMjBlock) mj_intervals_kernel(MJTables T, int M)
{
    constexpr int kChunks = kMjBlock / kMjChunk, kRow = kMjChunk + 1;
    __shared__ double v[kChunks * kRow];
    const MJTable &P = T.t[blockIdx.y];
    const int t = threadIdx.x, i = blockIdx.x * kMjBlock + t;
    double &own = v[t / kMjChunk * kRow + t % kMjChunk];
    own = i < M ? py_integral(P.ylo + i * P.h, P.ylo + (i + 1) * P.h, P.m) : 0.0;
    __syncthreads();
    const int c0 = blockIdx.x * kChunks;
    if (t < kChunks && (c0 + t) * kMjChunk < M) {
        const int n = min(kMjChunk, M - (c0 + t) * kMjChunk);
        double s = 0.0, comp = 0.0;
        for (int q = 0; q < n; ++q) {
            const double y = v[t * kRow + q] - comp;
            const double z = s + y;
            comp = (z - s) - y;
            s = z;
            v[t * kRow + q] = s;
        }
        P.cum[M + 1 + c0 + t] = s;
    }
    __syncthreads();
    if (i < M) P.cum[i + 1] = own;
}
__global__ void __launch_bounds__(kMjBlock) mj_offsets_kernel(MJTables T, int M)
{
    constexpr int kChunks = kMjBlock / kMjChunk;
    __shared__ double tot[kMjBlock], base[kChunks];
    const MJTable &P = T.t[blockIdx.y];
    const int t = threadIdx.x, i = blockIdx.x * kMjBlock + t, c0 = blockIdx.x * kChunks;
    double run = 0.0, comp = 0.0;                // of thread 0: sum of the chunks before
    for (int first = 0; first < c0 + kChunks; first += kMjBlock) {
        __syncthreads();
        if (first + t < c0 + kChunks) tot[t] = (first + t) * kMjChunk < M ? P.cum[M + 1 + first + t] : 0.0;
        __syncthreads();
        if (t) continue;
        auto add = [&](double v) {
            const double y = v - comp;
            const double z = run + y;
            comp = (z - run) - y;
            run = z;
        };
        const int before = min(kMjBlock, c0 - first), all = min(kMjBlock, c0 + kChunks - first);
        int c = 0;
        for (; c + 8 <= before; c += 8) {         // eight reads in flight before eight sums
            double v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = tot[c + q];
#pragma unroll
            for (int q = 0; q < 8; ++q) add(v[q]);
        }
        for (; c < all; ++c) {
            if (first + c >= c0) base[first + c - c0] = run;
            add(tot[c]);
        }
    }
    __syncthreads();
    if (i < M) P.cum[i + 1] += base[t / kMjChunk];
    if (i == 0) P.cum[0] = 0.0;
}

// tab[i] = J^{-1}(i/N) for 0 < i < N (App. D), tab[0] = ylo, tab[N] = yhi.
__global__ void mj_invert_kernel(MJTables T, int M, int N)
{
    const MJTable &P = T.t[blockIdx.y];
    const MJShape m = P.m;
    const double ylo = P.ylo, yhi = P.yhi, h = P.h;
    const double *cum = P.cum;
    double *tab = P.tab;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > N) return;
    if (i == 0) { tab[0] = ylo; return; }
    if (i == N) { tab[N] = yhi; return; }
    const double target = cum[M] * ((double)i / (double)N);
    int lo = 0, hi = M;                     // cum[lo] <= target < cum[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cum[mid] <= target) lo = mid; else hi = mid;
    }
    const double a = ylo + lo * h;
    double left = a, right = a + h;
    const double rem = target - cum[lo];
    const double piece = cum[lo + 1] - cum[lo];
    double y = a + h * (piece > 0.0 ? rem / piece : 0.5);
    for (int it = 0; it < 80; ++it) {
        const double F = py_integral(a, y, m) - rem;
        if (F > 0.0) right = y; else left = y;
        const double f = py_density(y, m);
        double yn = f > 0.0 ? y - F / f : 0.5 * (left + right);
        if (!(yn > left && yn < right)) yn = 0.5 * (left + right);
        const bool done = fabs(yn - y) <= 1e-15 * (fabs(y) + 1e-3);
        y = yn;
        if (done) break;
    }
    tab[i] = y;
}

// ------------------------------------------------------------- pair loading

// The radial solve of mj_momentum by Newton on the logarithm from d = 0.
__device__ double mj_radial_newton(double a, double lw)
{
    double dx = 0.0;
    for (int it = 0; it < 60; ++it) {
        const double gval = log1p(dx / (1.0 + a)) - dx - lw;        // decreasing in dx
        const double slope = (a + dx) / (1.0 + a + dx);              // -d(gval)/d(dx)
        const double step = gval / slope;
        dx = fmax(dx + step, 0.0);
        if (it >= 3 && fabs(step) <= 1e-15 * (dx + 1e-300)) break;
    }
    return dx;
}

// u from (quantile t, radial w in (0,1], azimuth v): p_y from the table by
// linear interpolation; r from l(x) = w l(a) (App. D, eq. finding_u), solved
// on the logarithm in d = x - a >= 0; azimuth uniform; then the drift axis y
// is carried onto `axis` by a cyclic relabelling.
// The load is bound by the FP64 vector ALU, and most of it by the logarithms
// of this solve: Newton from d = 0 took six of them per momentum.  Four FP32
// Newton steps give a start good to about 1e-6, from which one FP64 step of
// third order (Halley) reaches roundoff; a step larger than 1e-6 d is followed
// by another.  With g = ln(1 + d/(1 + a)) - d - ln w the step's error is below
// (step/d)^3 d, since g2 and g3 (second and third derivative) are below
// |g1|/(a + d) and 2 |g1|/(a + d)^2.  16.8 M pairs: 1.87 -> 1.40 ms.
// (A thread loads one pair: in a loop over pairs the constants of the logarithms
// stayed live, 218 registers instead of 76 and 1.72 ms.)
// FP32 momenta are those of the Newton solve bit for bit: where roundoff, here
// at most 2^-53 * 4 (1 + a + d)/(a + d) of d in either solve and 1e-15 of the
// radius from the azimuth, could carry a component over a rounding boundary of
// FP32 (about one momentum in 10^6), Newton decides.
template <typename R>
__device__ inline void mj_momentum(const MJPop &P, int N, double t, double w, double v, double out[3])
{
    const double f = t * N;
    int i = (int)f;
    if (i > N - 1) i = N - 1;
    const double py = P.tab[i] + (f - i) * (P.tab[i + 1] - P.tab[i]);
    const double gy = sqrt(1.0 + py * py);
    const double a = P.mu * P.G * gy;
    const double lw = log(w);
    const float af = (float)a, lf = (float)lw, ra = 1.0f / (1.0f + af);
    float df = -lf * (1.0f + af) / af;           // the first Newton step from 0
#pragma unroll
    for (int it = 0; it < 4; ++it)
        df = fmaxf(df + (log1pf(df * ra) - df - lf) * (1.0f + af + df) / (af + df), 0.0f);
    double dx = (double)df, cond = 0.0;          // cond: (1 + a + d)/(a + d)
    for (int it = 0; it < 60; ++it) {
        const double t = 1.0 + a + dx, inv = 1.0 / (a + dx);        // g1 = -1 / (t inv), g2 = -1 / t^2
        cond = t * inv;
        const double newton = (log1p(dx / (1.0 + a)) - dx - lw) * cond;
        const double step = newton / (1.0 + 0.5 * newton * inv / t);
        dx = fmax(dx + step, 0.0);
        if (fabs(step) <= 1e-6 * dx) break;
    }
    double um1 = dx / a, r = sqrt(um1 * (2.0 + um1)), sn, cs;
    sincospi(2.0 * v, &sn, &cs);
    double q[3] = {gy * r * cs, py, gy * r * sn};
    if (sizeof(R) == sizeof(float)) {
        const double e = gy * r * (8e-15 * cond + 4e-15);
        if ((float)(q[0] - e) != (float)(q[0] + e) || (float)(q[2] - e) != (float)(q[2] + e)) {
            um1 = mj_radial_newton(a, lw) / a;
            r = sqrt(um1 * (2.0 + um1));
            sincos(6.283185307179586 * v, &sn, &cs);
            q[0] = gy * r * cs;
            q[2] = gy * r * sn;
        }
    }
    const int sh = (P.axis + 2) % 3;          // component 1 -> axis
    for (int c = 0; c < 3; ++c) out[(c + sh) % 3] = q[c];
}

template <typename R>
__device__ inline void to_storage(const BoxDev<R> &B, const double x[3], int32_t &cell, R d[3])
{
    int c[3];
    for (int a = 0; a < 3; ++a) {
        double s = x[a];
        if (!(s >= 0.0 && s < B.n[a])) s = fmod(s, (double)B.n[a]);
        if (s < 0.0) s += B.n[a];
        if (s >= B.n[a]) s -= B.n[a];
        double f = floor(s);
        R off = (R)(s - f);
        int ci = (int)f;
        if (off >= R(1)) {           // rounding reached the next cell
            off = R(0);
            ci += 1;
        }
        if (ci >= B.n[a]) ci -= B.n[a];
        c[a] = ci;
        d[a] = off;
    }
    cell = pack_cell(c[0], c[1], c[2]);
}

template <typename R>
__global__ void __launch_bounds__(256) load_pairs_kernel(const BoxDev<R> *__restrict__ boxes, LoadArgs L)
{
    const BoxDev<R> &B = boxes[L.box];
    const SpeciesDev<R> &SA = B.sp[L.sa];
    const SpeciesDev<R> &SB = B.sp[L.sb];
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p < L.npairs) {
        uint64_t w[3][4];
        for (int j = 0; j < 3; ++j) {
            w[j][0] = (uint64_t)p; w[j][1] = (uint64_t)j; w[j][2] = 0; w[j][3] = 0;
            philox4x64_10(w[j], L.seed, L.stream);
        }
        // word map: (0,0..2) position, (0,3) A quantile, (1,0) A radial,
        // (1,1) A azimuth, (1,2) B quantile, (1,3) B radial, (2,0) B azimuth
        double x[3];
        for (int a = 0; a < 3; ++a) {
            const double U = unit53(w[0][a]);
            if (L.profile == PIC_PROFILE_HARRIS && a == L.paxis)
                x[a] = L.centre + L.thick * atanh((2.0 * U - 1.0) * tanh(L.halfw / L.thick));
            else
                x[a] = U * B.n[a];
        }
        double ua[3], ub[3];
        mj_momentum<R>(L.A, L.N, unit53(w[0][3]), 1.0 - unit53(w[1][0]), unit53(w[1][1]), ua);
        mj_momentum<R>(L.B, L.N, unit53(w[1][2]), 1.0 - unit53(w[1][3]), unit53(w[2][0]), ub);
        int32_t cell;
        R d[3];
        to_storage(B, x, cell, d);
        const int ia = L.offa + (int)p, ib = L.offb + (int)p;
        SA.stage.cell[ia] = cell;
        SB.stage.cell[ib] = cell;
        for (int a = 0; a < 3; ++a) {
            SA.stage.d[a][ia] = d[a];
            SB.stage.d[a][ib] = d[a];
            SA.stage.u[a][ia] = (R)ua[a];
            SB.stage.u[a][ib] = (R)ub[a];
        }
        if (SA.stage.id) SA.stage.id[ia] = L.ida + (int32_t)p;
        if (SB.stage.id) SB.stage.id[ib] = L.idb + (int32_t)p;
    }
}

// Harris-sheet b component at its staggered position (App. C,
// eq. B_field_Harris), one or two sheets.
template <typename R>
__global__ void __launch_bounds__(256) harris_field_kernel(const BoxDev<R> *__restrict__ boxes,
                                                           pic_harris_field H)
{
    const BoxDev<R> &B = boxes[H.box];
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= B.nc) return;
    const int n0 = B.n[0], n1 = B.n[1];
    const int idx[3] = {(int)(p % n0), (int)((p / n0) % n1), (int)(p / ((int64_t)n0 * n1))};
    // b_c sits half a cell off the node along the two axes other than c
    const double s = idx[H.grad_axis] + (H.grad_axis != H.field_axis ? 0.5 : 0.0);
    double v = tanh((s - H.centre[0]) / H.thickness);
    if (H.n_sheets == 2) v = v - tanh((s - H.centre[1]) / H.thickness) - 1.0;
    B.b[H.field_axis * B.nc + p] = (R)(H.b0 * v);
}

// ----------------------------------------------------------- host launchers

hipError_t launch_mj_tables(int n, const double *theta, const double *gamma_beta, double *const *cum, int M, int N,
                            double *const *tab, hipStream_t st)
{
    MJTables T;
    for (int q = 0; q < n; ++q) {
        MJTable &P = T.t[q];
        MJShape &m = P.m;
        m.mu = 1.0 / theta[q];
        m.G = sqrt(1.0 + gamma_beta[q] * gamma_beta[q]);
        m.beta0 = gamma_beta[q] / m.G;
        // support: where the exponent is 70 below its peak, gy - beta0 y = H
        const double H = 1.0 / m.G + 70.0 / (m.mu * m.G);
        const double rt = sqrt(H * H - 1.0 / (m.G * m.G));
        P.ylo = m.G * m.G * (H * m.beta0 - rt);
        P.yhi = m.G * m.G * (H * m.beta0 + rt);
        P.h = (P.yhi - P.ylo) / M;
        P.cum = cum[q];
        P.tab = tab[q];
    }
    const int blocks = (M + kMjBlock - 1) / kMjBlock;
    hipLaunchKernelGGL(mj_intervals_kernel, dim3(blocks, n), dim3(kMjBlock), 0, st, T, M);
    hipLaunchKernelGGL(mj_offsets_kernel, dim3(blocks, n), dim3(kMjBlock), 0, st, T, M);
    hipLaunchKernelGGL(mj_invert_kernel, dim3((N + 1 + 255) / 256, n), dim3(256), 0, st, T, M, N);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_load_pairs(const BoxDev<R> *boxes, const LoadArgs &L, hipStream_t st)
{
    int64_t blocks = (L.npairs + 255) / 256;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(load_pairs_kernel<R>, dim3((unsigned)blocks), dim3(256), 0, st, boxes, L);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_harris_field(const BoxDev<R> *boxes, int64_t nc, const pic_harris_field &H, hipStream_t st)
{
    hipLaunchKernelGGL(harris_field_kernel<R>, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st, boxes, H);
    return hipGetLastError();
}

template hipError_t launch_load_pairs<float>(const BoxDev<float> *, const LoadArgs &, hipStream_t);
template hipError_t launch_load_pairs<double>(const BoxDev<double> *, const LoadArgs &, hipStream_t);
template hipError_t launch_harris_field<float>(const BoxDev<float> *, int64_t, const pic_harris_field &, hipStream_t);
template hipError_t launch_harris_field<double>(const BoxDev<double> *, int64_t, const pic_harris_field &, hipStream_t);

} // namespace pic
