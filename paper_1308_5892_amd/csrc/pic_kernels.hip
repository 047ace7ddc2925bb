// gfx950 kernels of the PIC hot path: fused gather + Boris push + deposit per
// spatial tile, Yee field updates, counting-sort repack and FP64 diagnostics.
//
// Paper: Melzani et al., "Apar-T" (arXiv:1308.5892), App. A.  The readings of
// the paper used here (cyclic node averaging, standard Boris rotation,
// splitting of cell-crossing moves at node planes) are stated where they are
// used.  Every kernel is templated on the storage/arithmetic type R: float is
// the production form (int64 fixed-point current), double the FP64 form.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <limits>

#include "pic_internal.h"

namespace pic {

// ------------------------------------------------------------ arithmetic

__device__ inline float fast_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ inline double fast_rsqrt(double x) { return 1.0 / sqrt(x); }
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double fast_rcp(double x) { return 1.0 / x; }

template <typename R> __device__ inline R qscale_bits();
template <> __device__ inline float qscale_bits<float>() { return 2147483648.0f; }  // 2^31
template <> __device__ inline double qscale_bits<double>() { return 1.0; }

// FP32 form: a value already scaled by 2^31 rounded to the nearest integer,
// ties upward, in one conversion (|value| < 2^31 since every face value of one
// move is below one cell volume)
__device__ inline int quantize(float v)
{
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ inline double quantize(double v) { return v; }

__device__ inline void atomic_add_lds(long long *p, long long v)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}
__device__ inline void atomic_add_lds(double *p, double v) { atomicAdd(p, v); }
__device__ inline void atomic_add_global(long long *p, long long v)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}
__device__ inline void atomic_add_global(double *p, double v) { atomicAdd(p, v); }

// Relativistic Boris step (App. A.3.3, eq. mover) with hk = k h / 2:
// half electric kick, rotation about b with t = hk B / gamma^t and
// s = 2 t / (1 + t^2) (READING: the printed rotation is garbled; this is the
// rotation that solves the implicit mover equation), half electric kick.
template <typename R>
__device__ inline void boris(R hk, const R E[3], const R Bf[3], R u[3])
{
    R um0 = u[0] + hk * E[0], um1 = u[1] + hk * E[1], um2 = u[2] + hk * E[2];
    R ig = fast_rsqrt(R(1) + um0 * um0 + um1 * um1 + um2 * um2);
    R f = hk * ig;
    R t0 = f * Bf[0], t1 = f * Bf[1], t2 = f * Bf[2];
    R sf = R(2) * fast_rcp(R(1) + t0 * t0 + t1 * t1 + t2 * t2);
    R s0 = sf * t0, s1 = sf * t1, s2 = sf * t2;
    R v0 = um0 + (um1 * t2 - um2 * t1);
    R v1 = um1 + (um2 * t0 - um0 * t2);
    R v2 = um2 + (um0 * t1 - um1 * t0);
    u[0] = um0 + (v1 * s2 - v2 * s1) + hk * E[0];
    u[1] = um1 + (v2 * s0 - v0 * s2) + hk * E[1];
    u[2] = um2 + (v0 * s1 - v1 * s0) + hk * E[2];
}

// ------------------------------------------------------ global-memory reads

template <typename R>
__device__ inline R fld(const PIC_GLOBAL R *F, const BoxDev<R> &B, int c, int i, int j, int k)
{
    i = wrap_idx(i, B.n[0]);
    j = wrap_idx(j, B.n[1]);
    k = wrap_idx(k, B.n[2]);
    return F[c * B.nc + i + (int64_t)B.n[0] * (j + (int64_t)B.n[1] * k)];
}

// Fourth-order field solver (App. A.3.2, last paragraph; App. B, third item;
// READING: the paper prints no stencil): Faraday's law takes the staggered
// fourth-order difference along each axis, (9/8)(f[+1/2] - f[-1/2]) -
// (1/24)(f[+3/2] - f[-3/2]); Ampere's law keeps the second-order curl, so the
// second-order divergence of e still changes only by the charge-conserving
// current (Gauss's law as with Yee).  d4_e: that difference along axis a of
// component f of e at the point half a cell above (i,j,k) along a.
template <typename R>
__device__ inline R d4_e(const BoxDev<R> &B, int f, int i, int j, int k, int a)
{
    const int o0 = a == 0, o1 = a == 1, o2 = a == 2;
    const R near = fld(B.e, B, f, i + o0, j + o1, k + o2) - fld(B.e, B, f, i, j, k);
    const R far = fld(B.e, B, f, i + 2 * o0, j + 2 * o1, k + 2 * o2) - fld(B.e, B, f, i - o0, j - o1, k - o2);
    return R(9.0 / 8.0) * near - R(1.0 / 24.0) * far;
}

// (curl e)_c of the fourth-order solver at the b_c position of cell (i,j,k)
template <typename R>
__device__ inline R curl4_e(const BoxDev<R> &B, int c, int i, int j, int k)
{
    if (c == 0) return d4_e(B, 2, i, j, k, 1) - d4_e(B, 1, i, j, k, 2);
    if (c == 1) return d4_e(B, 0, i, j, k, 2) - d4_e(B, 2, i, j, k, 0);
    return d4_e(B, 1, i, j, k, 0) - d4_e(B, 0, i, j, k, 1);
}

// b^t = b^{t-dt/2} - (dt/2) curl e^t at the b_c position of cell (i,j,k).
// F4: 1 the fourth-order curl, 0 Yee's, -1 as the box says (the push kernel
// is compiled for one solver, so its loop carries only that one's code).
template <typename R, int F4 = -1>
__device__ inline R bt_global(const BoxDev<R> &B, int c, int i, int j, int k, R hdt)
{
    if (F4 == 1 || (F4 < 0 && B.faraday4)) return fld(B.b, B, c, i, j, k) - hdt * curl4_e(B, c, i, j, k);
    const PIC_GLOBAL R *e = B.e;
    R curl;
    if (c == 0)
        curl = (fld(e, B, 2, i, j + 1, k) - fld(e, B, 2, i, j, k)) - (fld(e, B, 1, i, j, k + 1) - fld(e, B, 1, i, j, k));
    else if (c == 1)
        curl = (fld(e, B, 0, i, j, k + 1) - fld(e, B, 0, i, j, k)) - (fld(e, B, 2, i + 1, j, k) - fld(e, B, 2, i, j, k));
    else
        curl = (fld(e, B, 1, i + 1, j, k) - fld(e, B, 1, i, j, k)) - (fld(e, B, 0, i, j + 1, k) - fld(e, B, 0, i, j, k));
    return fld(B.b, B, c, i, j, k) - hdt * curl;
}

// Node-averaged field values (App. A.3.3; READING: e_c averaged over the two
// edges along c that meet at the node, b_c over the four faces normal to c).
// The tile set-up forms the same sums in the same order from its LDS copy.
template <typename R>
__device__ inline R node_avg2(R a, R b) { return R(0.5) * (a + b); }
template <typename R>
__device__ inline R node_avg4(R a, R b, R c, R d) { return R(0.25) * (a + b + c + d); }

// Component c (0-2: e, 3-5: b^t) at node (i,j,k), read from HBM.
template <typename R, int F4 = -1>
__device__ inline R node_value_global(const BoxDev<R> &B, int c, int i, int j, int k, R hdt)
{
    switch (c) {
    case 0: return node_avg2(fld(B.e, B, 0, i - 1, j, k), fld(B.e, B, 0, i, j, k));
    case 1: return node_avg2(fld(B.e, B, 1, i, j - 1, k), fld(B.e, B, 1, i, j, k));
    case 2: return node_avg2(fld(B.e, B, 2, i, j, k - 1), fld(B.e, B, 2, i, j, k));
    case 3: return node_avg4(bt_global<R, F4>(B, 0, i, j, k, hdt), bt_global<R, F4>(B, 0, i, j - 1, k, hdt),
                             bt_global<R, F4>(B, 0, i, j - 1, k - 1, hdt), bt_global<R, F4>(B, 0, i, j, k - 1, hdt));
    case 4: return node_avg4(bt_global<R, F4>(B, 1, i, j, k, hdt), bt_global<R, F4>(B, 1, i, j, k - 1, hdt),
                             bt_global<R, F4>(B, 1, i - 1, j, k - 1, hdt), bt_global<R, F4>(B, 1, i - 1, j, k, hdt));
    default: return node_avg4(bt_global<R, F4>(B, 2, i, j, k, hdt), bt_global<R, F4>(B, 2, i - 1, j, k, hdt),
                              bt_global<R, F4>(B, 2, i - 1, j - 1, k, hdt), bt_global<R, F4>(B, 2, i, j - 1, k, hdt));
    }
}

// The trilinear interpolant of the eight node values of a cell, f[q] at node
// (q & 1, (q >> 1) & 1, q >> 2), written as c0 + c1 x + c2 y + c3 z + c4 xy +
// c5 yz + c6 zx + c7 xyz in the in-cell offsets: its coefficients, and its
// value at d, nested as c0 + x (c1 + y (c4 + z c7) + z c6) + y (c2 + z c5) +
// z c3 (seven multiply-adds, no products of the offsets).  The tile path and
// the HBM path both use these two, so the fields a particle sees do not
// depend on the path it takes.
template <typename R, typename P>
__device__ inline void trilinear_coef(const R f[8], P cf)
{
    const R ax = f[1] - f[0], ay = f[2] - f[0], az = f[4] - f[0];
    const R axy = (f[3] - f[2]) - ax, ayz = (f[6] - f[4]) - ay, azx = (f[5] - f[1]) - az;
    cf[0] = f[0];
    cf[1] = ax;
    cf[2] = ay;
    cf[3] = az;
    cf[4] = axy;
    cf[5] = ayz;
    cf[6] = azx;
    cf[7] = ((f[7] - f[6]) - (f[5] - f[4])) - axy;
}
template <typename R, typename P>
__device__ inline R trilinear_eval(P k8, const R d[3])
{
    const R t = fma(d[2], k8[7], k8[4]);
    const R u = fma(d[2], k8[6], fma(d[1], t, k8[1]));
    const R v = fma(d[2], k8[5], k8[2]);
    return fma(d[2], k8[3], fma(d[1], v, fma(d[0], u, k8[0])));
}

// e^t and b^t at (cell, d) from HBM: the node values, the interpolant's
// coefficients and its value, as the tile path computes them.
template <typename R, int F4 = -1>
__device__ inline void gather_global(const BoxDev<R> &B, int ix, int iy, int iz, const R d[3], R hdt,
                                     R E[3], R Bf[3])
{
    if constexpr (sizeof(R) == 8) {
        // the component loop stays rolled (each pass inlines eight node
        // values); in the FP64 form, at three waves per SIMD, its results are
        // selected into registers, since an array indexed by the loop counter
        // would live in scratch there
        R o[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
        for (int c = 0; c < 6; ++c) {
            R f[8], cf[8];
            for (int q = 0; q < 8; ++q)
                f[q] = node_value_global<R, F4>(B, c, ix + (q & 1), iy + ((q >> 1) & 1), iz + (q >> 2), hdt);
            trilinear_coef(f, cf);
            const R v = trilinear_eval(cf, d);
#pragma unroll
            for (int k = 0; k < 6; ++k) o[k] = c == k ? v : o[k];
        }
        E[0] = o[0]; E[1] = o[1]; E[2] = o[2];
        Bf[0] = o[3]; Bf[1] = o[4]; Bf[2] = o[5];
    } else {
        for (int c = 0; c < 6; ++c) {
            R f[8], cf[8];
            for (int q = 0; q < 8; ++q)
                f[q] = node_value_global<R, F4>(B, c, ix + (q & 1), iy + ((q >> 1) & 1), iz + (q >> 2), hdt);
            trilinear_coef(f, cf);
            const R v = trilinear_eval(cf, d);
            if (c < 3) E[c] = v;
            else Bf[c - 3] = v;
        }
    }
}

// ------------------------------------------------------------ slot claims

// Number of lanes below this one whose bit is set in the wave mask m.
__device__ inline int lane_rank(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Wave-aggregated claim of one slot per pending lane in the counter of its
// target segment: one atomic per distinct target in the wave.
__device__ inline int claim_slot(PIC_GLOBAL int32_t *cnt, int target, bool pending)
{
    int slot = -1;
    uint64_t m;
    while ((m = __ballot(pending)) != 0ull) {
        const int leader = __ffsll((unsigned long long)m) - 1;
        const int tgt = __shfl(target, leader);
        const bool mine = pending && target == tgt;
        const uint64_t mm = __ballot(mine);
        int base = 0;
        if (__lane_id() == leader) base = atomicAdd(&cnt[tgt], (int)__popcll(mm));
        base = __shfl(base, leader);
        if (mine) {
            slot = base + lane_rank(mm);
            pending = false;
        }
    }
    return slot;
}

// Element i of a 4-byte particle array (packed cells, ids) as a 32-bit byte
// offset from the array's (wave-uniform) base: slot counts stay below 2^29, so
// the offset fits and the access is one scalar base plus one vector offset.
template <typename T>
__device__ inline PIC_GLOBAL T &slot_ref(PIC_GLOBAL T *base, int i)
{
    return *reinterpret_cast<PIC_GLOBAL T *>(reinterpret_cast<PIC_GLOBAL char *>(base) +
                                             (uint32_t)i * (uint32_t)sizeof(T));
}

// Store a particle at slot `at` of copy P.  wide: the slot is in the overflow
// region or stages a leaver, and takes the packed cell; otherwise it is in
// the ranges of the cell's tile and takes the tile-local code.
template <bool NARROW = false, typename R>
__device__ inline void write_particle(const PBuf<R> &P, int at, bool wide, int32_t cell, int code, const R d[3],
                                      const R u[3], int32_t id)
{
    const PSlot<R> s = slot_at<NARROW>(P, at);
    if (wide) slot_ref(P.cell, at) = cell;
    else s.code() = (uint8_t)code;
    s.d(0) = d[0]; s.d(1) = d[1]; s.d(2) = d[2];
    s.u(0) = u[0]; s.u(1) = u[1]; s.u(2) = u[2];
    if (P.id) slot_ref(P.id, at) = id;
}

// Slot of copy `dst` for position `pos` of the B range of tile `tgt`, or of the
// overflow region when the segment is full; -1 (and the LOST flag) when both are.
template <typename R>
__device__ inline int b_range_slot(const BoxDev<R> &B, const SpeciesDev<R> &S, int dst, int tgt, int pos,
                                   PIC_GLOBAL uint32_t *flags)
{
    if (pos < S.seg_cap[dst][tgt]) return S.seg_start[dst][tgt] + pos;
    const int o = atomicAdd(&S.nb[dst][B.ntiles], 1);
    if (o >= S.ovf_cap) {
        atomicOr(flags, PIC_FLAG_LOST);
        return -1;
    }
    return S.seg_start[dst][B.ntiles] + o;
}

// Store a particle into the B range of tile `tgt` of copy `dst` (or the
// overflow region); slots are claimed with one atomic per distinct target in
// the wave.  Every lane of the wave must call it.
template <typename R>
__device__ inline void store_particle(const BoxDev<R> &B, const SpeciesDev<R> &S, int dst, int tgt, bool valid,
                                      int32_t cell, const R d[3], const R u[3], int32_t id,
                                      PIC_GLOBAL uint32_t *flags)
{
    const int slot = claim_slot(S.nb[dst], tgt, valid);
    if (!valid) return;
    const int at = b_range_slot(B, S, dst, tgt, S.bs[dst][tgt] + slot, flags);
    if (at >= 0) write_particle(S.buf[dst], at, at >= S.slots - S.ovf_cap, cell, local_code(B, cell), d, u, id);
}

// Offset of x in its cell, x - floor(x), kept below 1: an x a hair below a
// node plane, whose difference would round up to 1, stays in the lower cell
// at the largest offset below 1 (one v_fract_f32, which clamps so).
__device__ inline float offset_in_cell(float x) { return __builtin_amdgcn_fractf(x); }
__device__ inline double offset_in_cell(double x) { return fmin(x - floor(x), 1.0 - 0x1p-53); }

// New cell and offset after the move x1 = d + D (home-cell frame), wrapped.
template <typename R>
__device__ inline int32_t advance_cell(const BoxDev<R> &B, int ix, int iy, int iz, const R x1[3], R dn[3])
{
    int c[3] = {ix, iy, iz};
    for (int a = 0; a < 3; ++a) {
        const int f = (int)floor(x1[a]);      // -1, 0 or 1: x1 lies in (-1, 2)
        dn[a] = offset_in_cell(x1[a]);
        int ci = c[a] + f;
        if (ci < 0) ci += B.n[a];
        else if (ci >= B.n[a]) ci -= B.n[a];
        c[a] = ci;
    }
    return pack_cell(c[0], c[1], c[2]);
}

// ------------------------------------------------- fused per-tile push kernel

template <typename R>
struct TileGeom {
    int o[3], ext[3];
    int NX, NY, NN;      // node region (ext+1)^3, origin o
    int JX, JY, JN;      // J / raw-e region (ext+3)^3, origin o-1
    int BX, BY, BN;      // raw-b region (ext+2)^3, origin o-1
};

// Geometry of tile T.  The LDS regions are laid out for the full tile shape
// (1 << tshift per axis; ext only limits which cells hold particles), so with
// FIX = 1 (every tile 4x4x4) all their strides are compile-time constants.
template <typename R, int FIX = 0>
__device__ inline TileGeom<R> tile_geom(const BoxDev<R> &B, int T)
{
    TileGeom<R> g;
    const int sx = FIX ? 2 : B.tshift[0], sy = FIX ? 2 : B.tshift[1], sz = FIX ? 2 : B.tshift[2];
    const int tx = T % B.ntile[0];
    const int r = T / B.ntile[0];
    const int ty = r % B.ntile[1], tz = r / B.ntile[1];
    g.o[0] = tx << sx;
    g.o[1] = ty << sy;
    g.o[2] = tz << sz;
    const int t0 = 1 << sx, t1 = 1 << sy, t2 = 1 << sz;
    g.ext[0] = min(t0, B.n[0] - g.o[0]);
    g.ext[1] = min(t1, B.n[1] - g.o[1]);
    g.ext[2] = min(t2, B.n[2] - g.o[2]);
    g.NX = t0 + 1; g.NY = t1 + 1; g.NN = g.NX * g.NY * (t2 + 1);
    g.JX = t0 + 3; g.JY = t1 + 3; g.JN = g.JX * g.JY * (t2 + 3);
    g.BX = t0 + 2; g.BY = t1 + 2; g.BN = g.BX * g.BY * (t2 + 2);
    return g;
}

// Per-wave queue of unfinished moves (LDS ring buffer): a move that crosses
// node planes deposits its first piece at once and waits here for the rest;
// the wave deposits the next piece of 64 queued moves at a time and puts back
// those that still have pieces left.  An entry holds the start of the next
// piece and the end of the move (home-cell frame), the LDS index of the home
// cell with the species sign, and the meta word of the move (move_meta).
// FP32 form: two waves' worth of entries, so that a put after a drain always
// fits.  FP64 form: one wave's worth (a wave drains before a put that would
// not fit), which keeps a 4x4x4 block within the LDS of three blocks per CU.
template <typename R> struct QCap { static constexpr int value = 128; };
template <> struct QCap<double> { static constexpr int value = 64; };
constexpr int kWaves = kBlock / 64;

template <typename R>
__host__ __device__ inline size_t queue_bytes(int waves)
{
    return (size_t)waves * QCap<R>::value * (sizeof(int32_t) + 6 * sizeof(R));
}

// Values per cell in the gather's coefficient table: 8 per field component,
// and 16 bytes more, so that a record is an odd number of 16-byte units and the
// 16-byte reads of lanes in different cells start on different LDS banks: 52
// values in FP32, 50 in FP64, whose push the LDS bounds (busy for 0.81 of it;
// with 52 values there too, half the banks served all reads: 0.958 against
// 0.932 ms, 33.5 M particles).  (A coefficient-major table, one dword per lane
// per read, ran the push 43 % slower.)
template <typename R>
constexpr int kCoef = 48 + 16 / (int)sizeof(R);

// Strides of the tile current in LDS, (t + 3)^3 points per component.  4x4x4
// tiles: rows of 7 and planes of 52, with which the points of the 64 cells, at
// equal moves, lie more evenly over the 32 banks of 8 bytes that the adds use than
// with planes of 49 (sum over the banks of the square of their load 152 against
// 160, 16 cells of an x-z plane 16 against 24).  Push with planes of 52
// against 49: 33.5 M thermal particles 500 against 510 us, in FP64 895 against
// 916; over 200 steps after 20, two beams 575 against 606, Harris sheet 411
// against 422 (over 20 steps after 5, while the clock still falls, 624 against
// 651 and 442 against 450).  Planes of 60 are as fast and take more room; rows of
// 8 with planes of 60 were slower for beams (694 us over 20 steps: the rows of a
// plane then share banks).
struct CurrentGrid {
    int x, xy, n;
    __host__ __device__ constexpr CurrentGrid(int t0, int t1, int t2)
        : x(t0 == 4 && t1 == 4 && t2 == 4 ? 7 : t0 + 3), xy(t0 == 4 && t1 == 4 && t2 == 4 ? 52 : (t0 + 3) * (t1 + 3)),
          n(xy * (t2 + 3))
    {
    }
};

// LDS of one push block for tiles of t0 x t1 x t2 cells, three regions:
//   [coef]   the gather's coefficient table (kCoef<R> values per cell);
//   [stage]  the piece queues during the particle loop, the staged raw e and
//            b (tile plus halo) during set-up;
//   [union]  the node fields during set-up, the tile current afterwards.
struct TileLds {
    size_t coef, stage, uni;
    __host__ __device__ size_t total() const { return coef + stage + uni; }
};

template <typename R>
__host__ __device__ inline TileLds tile_lds(int t0, int t1, int t2, int waves = kWaves)
{
    const size_t nc = (size_t)t0 * t1 * t2;
    const size_t nn = (size_t)(t0 + 1) * (t1 + 1) * (t2 + 1);
    const size_t jn = (size_t)(t0 + 3) * (t1 + 3) * (t2 + 3);
    const size_t bn = (size_t)(t0 + 2) * (t1 + 2) * (t2 + 2);
    const size_t raw = 3 * (jn + bn) * sizeof(R), q = queue_bytes<R>(waves);
    const size_t nodes = 6 * nn * sizeof(R);
    const size_t jb = 3 * (size_t)CurrentGrid(t0, t1, t2).n * sizeof(typename JType<R>::T);
    TileLds L;
    L.coef = (nc * kCoef<R> * sizeof(R) + 15) & ~size_t(15);
    L.stage = ((raw > q ? raw : q) + 15) & ~size_t(15);
    L.uni = ((nodes > jb ? nodes : jb) + 15) & ~size_t(15);
    return L;
}

// q / m for 0 <= q < 4096 and 1 <= m <= 16, with mul = 65536 / m + 1: the
// rounding error q (mul - 65536/m) / 65536 < 1/16 never reaches the next
// integer because q/m is at least 1/m below it.
__device__ inline int div_small(int q, int mul) { return (int)(__umul24((unsigned)q, (unsigned)mul) >> 16); }

// v wrapped into [0, n) for v in [-n, 2n) (one correction step)
__device__ inline int wrap1(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// The twelve fluxes of one piece (start offset s in its cell, displacement
// dd), eq. current_dep (App. A.3.4) with the sign and scale of the species,
// rounded to the fixed-point current: per component a, the four faces around
// the cell's a-edge, f = 0 at the cell, 1 one step along b2, 2 one step along
// b1, 3 both (b1, b2 the two other axes in cyclic order).  With
// m = s + dd/2 and K = dd_b1 dd_b2 / 12 the weights are (1-m1)(1-m2)+K,
// (1-m1)m2-K, m1(1-m2)-K and m1 m2+K; they sum to one, so the f = 0 value is
// the rounded total minus the other three rounded values, and a piece moves
// exactly its charge.  add(a, f, q) receives each rounded value.
template <typename R, typename Add>
__device__ inline void piece_fluxes(const R s[3], const R dd[3], R scale, Add &&add)
{
    const R m[3] = {s[0] + R(0.5) * dd[0], s[1] + R(0.5) * dd[1], s[2] + R(0.5) * dd[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int b1 = a == 2 ? 0 : a + 1, b2 = a == 0 ? 2 : a - 1;
        const R PK = m[b1] * m[b2] + dd[b1] * dd[b2] * R(1.0 / 12.0);
        const R F = scale * dd[a];
        const R t11 = F * PK, t01 = fma(F, m[b2], -t11), t10 = fma(F, m[b1], -t11);
        const auto q11 = quantize(t11), q01 = quantize(t01), q10 = quantize(t10);
        const auto q00 = quantize(F) - q01 - q10 - q11;
        add(a, 0, q00);
        add(a, 1, q01);
        add(a, 2, q10);
        add(a, 3, q11);
    }
}

// The fluxes of one piece added to the LDS tile current at jl[cb + off[a][f]].
template <typename R>
__device__ inline void deposit_piece(typename JType<R>::T *jl, int cb, const int (&off)[3][4], const R s[3],
                                     const R dd[3], R scale)
{
    piece_fluxes(s, dd, scale, [&](int a, int f, auto q) { atomic_add_lds(&jl[cb + off[a][f]], q); });
}

template <typename R>
__device__ inline R sel3(int i, R a0, R a1, R a2) { return i == 0 ? a0 : (i == 1 ? a1 : a2); }

// Node planes crossed by the move d -> x1 = d + D in the home-cell frame
// (|D| < 1: at most one per axis): direction per axis and the crossing
// parameter lambda in (0, 1] (2 where no plane is crossed).
template <typename R>
__device__ inline void move_crossings(const R d[3], const R D[3], R x1[3], int dir[3], R lam[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        x1[a] = d[a] + D[a];
        dir[a] = (int)floor(x1[a]);       // -1, 0 or 1, since x1 lies in (-1, 2)
        lam[a] = dir[a] != 0 ? ((dir[a] > 0 ? R(1) : R(0)) - d[a]) * fast_rcp(D[a]) : R(2);
    }
}

// Conducting wall on axis w (App. A.4): when the move d -> d + D (home-cell
// frame; cw = home cell index along w, nw = cells along w) leaves the box
// through a wall, the move is cut where it meets the wall: D1 takes it there,
// P = d + D1 is that point as the deposit computes it, D2 takes the rest
// mirrored back into the box along w, and u_w changes sign.  Returns whether
// the move hit the wall.
template <typename R>
__device__ inline bool wall_hit(int w, int cw, int nw, const R d[3], const R D[3], R D1[3], R P[3], R D2[3],
                                R u[3])
{
    const R xw = d[w] + D[w];
    const bool lo = cw == 0 && xw < R(0), hi = cw == nw - 1 && xw >= R(1);
    if (!lo && !hi) return false;
    const R plane = hi ? R(1) : R(0);
    const R l = (plane - d[w]) / D[w];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        D1[a] = a == w ? plane - d[w] : l * D[a];
        asm volatile("" : "+v"(D1[a]));
        P[a] = d[a] + D1[a];
    }
    R xr = R(2) * plane - xw;                    // the mirrored end along w
    if (xr >= R(1)) xr = R(1) - R(1) / R(1 << 23);  // a move ending exactly on the upper wall
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        D2[a] = (a == w ? xr : d[a] + D[a]) - P[a];
        asm volatile("" : "+v"(D2[a]));
    }
    u[w] = -u[w];
    return true;
}

// The mirrored rest of a wall move starts at P (home-cell frame), which lies
// in a neighbouring cell along each other axis that the first piece crossed.
// Rebase it onto that cell: s = the cell's offset from the home cell (0 along
// the wall axis, where P is on a face of the home cell), P in [0, 1) of it.
template <typename R>
__device__ inline void wall_rest_start(int w, R P[3], int s[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        s[a] = a == w ? 0 : (P[a] < R(0) ? -1 : (P[a] >= R(1) ? 1 : 0));
        R v = P[a] - R(s[a]);
        if (v >= R(1)) v = R(1) - R(0.5) * std::numeric_limits<R>::epsilon();   // -tiny + 1 rounded up
        if (a != w) P[a] = v;
    }
}

__device__ inline float clamp01(float v) { return __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f); }
__device__ inline double clamp01(double v) { return fmin(fmax(v, 0.0), 1.0); }

// First breakpoint of a move d -> d + D: where its first crossing axis ax
// meets its plane (parameter l).  That coordinate is the plane itself; no
// other plane is crossed before it, so every other coordinate lies in the
// closed home cell [0, 1] (clamped there against rounding).  A plane crossed
// at the same parameter is left at the plane: its own piece then has length
// zero.
template <typename R>
__device__ inline void first_breakpoint(const R d[3], const R D[3], const int dir[3], int ax, R l, R q[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const R c = clamp01(fma(l, D[a], d[a]));
        q[a] = a == ax ? (dir[a] > 0 ? R(1) : R(0)) : c;
    }
}

// Meta word of a queued move: per axis a the crossing direction + 1 (bits 8a,
// 8a + 1), next piece k (bits 2-3), crossings nb (4-5), the crossing axes in
// order o0, o1, o2 (10-15), the tile current's index of the home cell (18-30; at
// most 1064, in 8x8x8 tiles) and the sign of the species (31).
constexpr int kMetaK = 2, kMetaNb = 4, kMetaO = 10, kMetaJ = 18;
__device__ inline int move_meta(int k, int nb, int o0, int o1, int o2, const int dir[3])
{
    return (k << kMetaK) | (nb << kMetaNb) | (o0 << kMetaO) | (o1 << (kMetaO + 2)) | (o2 << (kMetaO + 4)) |
           (dir[0] + 1) | ((dir[1] + 1) << 8) | ((dir[2] + 1) << 16);
}
__device__ inline int meta_k(int meta) { return (meta >> kMetaK) & 3; }
__device__ inline int meta_nb(int meta) { return (meta >> kMetaNb) & 3; }
__device__ inline int meta_axis(int meta, int i) { return (meta >> (kMetaO + 2 * i)) & 3; }
__device__ inline int meta_dir(int meta, int a) { return ((meta >> (8 * a)) & 3) - 1; }

// Piece k of a queued move (0 <= k <= nb crossings), from its start ps (the
// previous breakpoint; home-cell frame) towards the move's end x1.  The piece
// lies in the cell offset `offc` from the home cell: the directions of the
// crossings before it (axes o_0 .. o_{k-1} of the meta word).  Its end pe is
// x1 for the last piece; otherwise the point where axis o_k meets its plane,
// reached along the rest of the move, with every other coordinate clamped
// into the piece's cell (against rounding).  Every later breakpoint of a
// move is computed this way from the one before, on the tile path and on
// the HBM path alike, so consecutive pieces share their breakpoints exactly
// and the last piece ends exactly at the particle's new position.  Returns
// the piece's start in its cell (sv) and displacement (dd).
template <typename R>
__device__ inline void chain_piece(const R ps[3], const R x1[3], int meta, int k, R pe[3], int offc[3], R sv[3],
                                   R dd[3])
{
    const int nb = meta_nb(meta);
    int crossed = 0;
    if (k > 0) crossed |= 1 << meta_axis(meta, 0);
    if (k > 1) crossed |= 1 << meta_axis(meta, 1);
    if (k > 2) crossed |= 1 << meta_axis(meta, 2);
#pragma unroll
    for (int a = 0; a < 3; ++a) offc[a] = (crossed >> a) & 1 ? meta_dir(meta, a) : 0;
    if (k < nb) {
        const int ax = meta_axis(meta, k);
        const R Dp[3] = {x1[0] - ps[0], x1[1] - ps[1], x1[2] - ps[2]};
        const R plane = meta_dir(meta, ax) > 0 ? R(1) : R(0);
        // the parameter of the crossing along the rest of the move; a rest
        // that no longer moves along the axis (0 * inf) gives 0
        R l = (plane - sel3(ax, ps[0], ps[1], ps[2])) * fast_rcp(sel3(ax, Dp[0], Dp[1], Dp[2]));
        l = fmin(fmax(l, R(0)), R(1));
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const R lo = R(offc[a]);
            const R v = fmin(fmax(fma(l, Dp[a], ps[a]), lo), lo + R(1));
            pe[a] = a == ax ? plane : v;
        }
    } else {
        pe[0] = x1[0]; pe[1] = x1[1]; pe[2] = x1[2];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        sv[a] = ps[a] - R(offc[a]);
        dd[a] = pe[a] - ps[a];
    }
}

// The pieces k, k+1, ..., nb of a queued move, from breakpoint ps to the
// move's end x1 (see chain_piece), as the queue deposits them.
// add(a, ox, oy, oz, q): rounded flux q of component a at node (cell + o).
template <typename R, typename Add>
__device__ inline void deposit_chain(const R ps0[3], const R x1[3], int meta, int k, R scale, Add &&add)
{
    const int nb = meta_nb(meta);
    R ps[3] = {ps0[0], ps0[1], ps0[2]};
    for (; k <= nb; ++k) {
        R pe[3], sv[3], dd[3];
        int offc[3];
        chain_piece(ps, x1, meta, k, pe, offc, sv, dd);
        piece_fluxes(sv, dd, scale, [&](int a, int f, auto q) {
            const int b1 = a == 2 ? 0 : a + 1, b2 = a == 0 ? 2 : a - 1;
            int o[3] = {offc[0], offc[1], offc[2]};
            if (f & 1) o[b2] += 1;
            if (f & 2) o[b1] += 1;
            add(a, o[0], o[1], o[2], q);
        });
        ps[0] = pe[0]; ps[1] = pe[1]; ps[2] = pe[2];
    }
}

// Crossings of the move d -> d + D, their order and the meta word (next piece
// k), as the push computes them.
template <typename R>
__device__ inline int move_order(const R d[3], const R D[3], int k, R x1[3], int dir[3], R lam[3], int &o0,
                                 R &l0)
{
    move_crossings(d, D, x1, dir, lam);
    const int nb = (dir[0] != 0) + (dir[1] != 0) + (dir[2] != 0);
    int q0 = 0, q1 = 1, q2 = 2;
    R m0 = lam[0], m1 = lam[1], m2 = lam[2];
    if (m1 < m0) { R t = m0; m0 = m1; m1 = t; int q = q0; q0 = q1; q1 = q; }
    if (m2 < m1) { R t = m1; m1 = m2; m2 = t; int q = q1; q1 = q2; q2 = q; }
    if (m1 < m0) { R t = m0; m0 = m1; m1 = t; int q = q0; q0 = q1; q1 = q; }
    o0 = q0;
    l0 = m0;
    return move_meta(k, nb, q0, q1, q2, dir);
}

// Charge-conserving deposit of the straight move d -> d + D from the start
// cell (d in [0,1)^3, |D| < 1), for the particles that take the HBM path.
// READING (the paper defers cell-crossing moves to references not given): the
// move is cut at each node plane it crosses, in order of the crossing
// parameter, and each piece deposits its fluxes (eq. current_dep, App. A.3.4)
// in its own cell.  The first breakpoint comes from d and the crossing
// parameter, the later ones from chain_piece, the fluxes from piece_fluxes:
// exactly as the tile path computes them (its first piece at once, the
// others from the queue), so a move deposits the same integers whichever
// path it takes.  add(a, ox, oy, oz, q): rounded flux q of component a at
// node (start cell + o).
template <typename R, typename Add>
__device__ inline void deposit_move(const R d[3], const R D[3], R scale, Add &&add)
{
    R x1[3], lam[3], l0;
    int dir[3], o0;
    const int meta = move_order(d, D, 1, x1, dir, lam, o0, l0);
    const int nb = meta_nb(meta);
    R p1[3];
    if (nb == 0) {
        p1[0] = x1[0]; p1[1] = x1[1]; p1[2] = x1[2];
    } else {
        first_breakpoint(d, D, dir, o0, l0, p1);
    }
    const R dd[3] = {p1[0] - d[0], p1[1] - d[1], p1[2] - d[2]};
    piece_fluxes(d, dd, scale, [&](int a, int f, auto q) {
        const int b1 = a == 2 ? 0 : a + 1, b2 = a == 0 ? 2 : a - 1;
        int o[3] = {0, 0, 0};
        if (f & 1) o[b2] += 1;
        if (f & 2) o[b1] += 1;
        add(a, o[0], o[1], o[2], q);
    });
    if (nb > 0) deposit_chain(p1, x1, meta, 1, scale, add);
}

// The whole move d -> d + D as one chain from its start (the mirrored rest of
// a move through a conducting wall, queued from its first piece).
template <typename R, typename Add>
__device__ inline void deposit_rest(const R d[3], const R D[3], R scale, Add &&add)
{
    R x1[3], lam[3], l0;
    int dir[3], o0;
    const int meta = move_order(d, D, 0, x1, dir, lam, o0, l0);
    deposit_chain(d, x1, meta, 0, scale, add);
}

// The Boris step, the non-finite check and the displacement D = dt u / gamma
// of the move, shared by the tile and HBM paths.  D stays the rounded product
// (opaque to the compiler, so that no multiply-add fuses it into d + D): the
// move's end x1 = d + D and its crossings must come out identical wherever
// they are computed.
template <typename R>
__device__ inline void boris_move(R hk, const R E[3], const R Bf[3], R u[3], R dt, bool valid,
                                  PIC_GLOBAL uint32_t *flags, R D[3])
{
    boris(hk, E, Bf, u);
    // one test catches NaN and infinity (and |u| beyond 1e15)
    R u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const bool bad = !(u2 < R(1e30));
    if (__builtin_expect(__ballot(bad) != 0, 0)) {     // wave-uniform: the fix-up costs nothing otherwise
        if (bad) {
            if (valid) atomicOr(flags, PIC_FLAG_NONFINITE);
            u[0] = u[1] = u[2] = R(0);
            u2 = R(0);
        }
    }
    const R ig = dt * fast_rsqrt(R(1) + u2);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        D[a] = ig * u[a];
        asm volatile("" : "+v"(D[a]));
    }
}

// Tile one step away from tile T in direction code = (dx+1) + 3(dy+1) + 9(dz+1).
template <typename R>
__device__ inline int neighbor_tile(const BoxDev<R> &B, const TileGeom<R> &g, int code)
{
    int t = 0, mul = 1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int dl = code % 3 - 1;
        code /= 3;
        int ta = (g.o[a] >> B.tshift[a]) + dl;
        ta = ta < 0 ? ta + B.ntile[a] : (ta >= B.ntile[a] ? ta - B.ntile[a] : ta);
        t += ta * mul;
        mul *= B.ntile[a];
    }
    return t;
}

// Cells just outside tile g along each axis (wrapped into the box).
struct TileRim {
    int lo[3], hi[3];
};

template <typename R>
__device__ inline TileRim tile_rim(const BoxDev<R> &B, const TileGeom<R> &g)
{
    TileRim r;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.lo[a] = g.o[a] == 0 ? B.n[a] - 1 : g.o[a] - 1;
        r.hi[a] = g.o[a] + g.ext[a] == B.n[a] ? 0 : g.o[a] + g.ext[a];
    }
    return r;
}

// Direction code of a particle in cell c relative to tile g: 13 if it is
// inside g, (dx+1) + 3(dy+1) + 9(dz+1) for a cell in the layer around g (the
// adjacent tile in that direction is then the particle's tile, since a cell
// one step outside a tile lies in the next tile along that axis), or -1
// otherwise.  A pure function of the stored cell, so that the push and the
// hand-over of the leavers classify a particle the same way.
template <typename R>
__device__ inline int move_bin(const TileGeom<R> &g, const TileRim &rim, const int c[3])
{
    int code = 0, mul = 1;
    bool bad = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int dl = (unsigned)(c[a] - g.o[a]) < (unsigned)g.ext[a] ? 0
                       : (c[a] == rim.lo[a] ? -1 : (c[a] == rim.hi[a] ? 1 : 2));
        bad |= dl == 2;
        code += (dl + 1) * mul;
        mul *= 3;
    }
    return bad ? -1 : code;
}

// Cell coordinates of a 4x4x4 tile as bytes of one word (axis a in byte a), so
// that one instruction works on the three axes: the dot product with byte
// weights turns them into a table index, and adding a packed move shifts all
// three.  A moved particle's coordinate c lies in [-1, ext]; its word P holds
// c + 4 per byte.
__device__ inline uint32_t udot4(uint32_t a, uint32_t b) { return __builtin_amdgcn_udot4(a, b, 0u, false); }
constexpr uint32_t kOnes = 0x010101u, kThrees = 0x030303u, kFours = 0x040404u;

// Where the moved particles of a tile go: per axis t = 0, 1 or 2 (the tile
// below, the same, the tile above) and q, the coordinate in that tile.  In a
// regular tile (4x4x4, full tiles around it, more than one tile per axis)
// these are the bits of P; in a partial tile, at the box's lower edge when its
// last tile is partial, or on an axis that one tile spans, the axis decides.
struct TileMove {
    bool regular;
    int ext[3], low[3];              // cells of the tile; coordinate of cell -1 in its tile
    bool span[3];
    template <typename R>
    __device__ void init(const BoxDev<R> &B, const TileGeom<R> &g)
    {
        regular = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            ext[a] = g.ext[a];
            span[a] = B.ntile[a] == 1;
            low[a] = g.o[a] == 0 ? (B.n[a] - 1) & 3 : 3;
            regular = regular && ext[a] == 4 && !span[a] && low[a] == 3;
        }
    }
    __device__ void to(uint32_t P, uint32_t &t, uint32_t &q) const
    {
        if (regular) {
            t = (P >> 2) & kThrees;
            q = P & kThrees;
            return;
        }
        t = q = 0u;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int c = (int)((P >> (8 * a)) & 255u) - 4;
            const bool up = c == ext[a], dn = c < 0;
            t |= (uint32_t)(span[a] ? 1 : (up ? 2 : (dn ? 0 : 1))) << (8 * a);
            q |= (uint32_t)(up ? 0 : (dn ? low[a] : c)) << (8 * a);
        }
    }
};
// A staged leaver's byte: c + 1 of the three axes in base 6 (the tile grown by
// one cell, 216 codes), and back (exact for every code below 216).
__device__ inline uint32_t leaver_code(uint32_t P) { return udot4(P, 0x240601u) - 3u * 43u; }
__device__ inline uint32_t leaver_cell(uint32_t c)
{
    const uint32_t z = (c * 57u) >> 11, r = c - 36u * z, y = (r * 43u) >> 8, x = r - 6u * y;
    return (x | (y << 8) | (z << 16)) + kThrees;
}

template <typename R> struct PushWaves { static constexpr int value = 4; };
template <> struct PushWaves<double> { static constexpr int value = 3; };

// Grid index of the point (o - 1) + (i, j, k) around tile g, wrapped periodically.
template <typename R>
struct TileGrid {
    int o[3], n[3];
    int64_t n0, n01;
    __device__ TileGrid(const BoxDev<R> &B, const TileGeom<R> &g)
    {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            o[a] = g.o[a] - 1;
            n[a] = B.n[a];
        }
        n0 = n[0];
        n01 = (int64_t)n[0] * n[1];
    }
    __device__ int64_t operator()(int i, int j, int k) const
    {
        const int gi = wrap1(o[0] + i, n[0]), gj = wrap1(o[1] + j, n[1]), gk = wrap1(o[2] + k, n[2]);
        if ((unsigned)gi >= (unsigned)n[0] || (unsigned)gj >= (unsigned)n[1] || (unsigned)gk >= (unsigned)n[2])
            return wrap_idx(o[0] + i, n[0]) + n0 * wrap_idx(o[1] + j, n[1]) +   // boxes narrower than the halo
                   n01 * wrap_idx(o[2] + k, n[2]);
        return gi + n0 * gj + n01 * gk;
    }
};

// Set-up of a tile by one block: the trilinear coefficients of e^t and b^t of
// every cell, from the staged e^t and b^{t-dt/2} of the tile and its halo
// (raw e in re, raw b in rb, node fields in node; ends with every thread past
// its last read of node).  STEP: also write b^{t+dt/2} of the tile's cells.
// staged() is called by every thread once the raw fields are staged and says
// whether the tile has particles; without any the set-up ends after b, and
// its result is passed on.
template <typename R, int FIX, int WALLS, int F4, bool STEP, int NT, typename Staged>
__device__ __forceinline__ bool tile_coefs(const BoxDev<R> &B, const TileGeom<R> &g, const TileGrid<R> &gidx, R dt,
                                           R *coef, R *re, R *rb, R *node, Staged &&staged)
{
    const int tid = threadIdx.x;
    // region indices are decoded by multiply-shift (edges of at most 11 and
    // fewer than 2^11 points: exact)
    const int mJX = 65536 / g.JX + 1, mJY = 65536 / g.JY + 1;
    const int mBX = 65536 / g.BX + 1, mBY = 65536 / g.BY + 1;
    const int mNX = 65536 / g.NX + 1, mNY = 65536 / g.NY + 1;
    const int JX = g.JX, JXY = g.JX * g.JY, BX = g.BX, BXY = g.BX * g.BY;
    const int NX = g.NX, NXY = g.NX * g.NY;
    const int tsx = FIX ? 2 : B.tshift[0], tsxy = FIX ? 4 : B.tshift[0] + B.tshift[1];

    // 1. stage e^t and b^{t-dt/2} of the tile and its halo
    for (int q = tid; q < g.JN; q += NT) {
        const int jk = div_small(q, mJX), i = q - jk * JX;
        const int k = div_small(jk, mJY), j = jk - k * g.JY;
        const int64_t gp = gidx(i, j, k);
#pragma unroll
        for (int c = 0; c < 3; ++c) re[c * g.JN + q] = B.e[c * B.nc + gp];
    }
    for (int q = tid; q < g.BN; q += NT) {
        const int jk = div_small(q, mBX), i = q - jk * BX;
        const int k = div_small(jk, mBY), j = jk - k * g.BY;
        const int64_t gp = gidx(i, j, k);
#pragma unroll
        for (int c = 0; c < 3; ++c) rb[c * g.BN + q] = B.b[c * B.nc + gp];
    }
    __syncthreads();
    const bool any = staged();

    // 2. b^t = b^{t-dt/2} - (dt/2) curl e^t (App. A.3.1 item 1), in place;
    //    and for the tile's own cells the full step b^{t+dt/2} = b^{t-dt/2} -
    //    dt curl e^t (App. A.3.1 items 1 and 4 together), written to the other
    //    b buffer, so that no separate b update is launched: every cell
    //    belongs to one tile, and no block reads that buffer in this launch
    const R hdt = R(0.5) * dt;
    // raw-b point (i, j, k) is a cell of this tile
    auto own = [&](int i, int j, int k) {
        return (unsigned)(i - 1) < (unsigned)g.ext[0] && (unsigned)(j - 1) < (unsigned)g.ext[1] &&
               (unsigned)(k - 1) < (unsigned)g.ext[2];
    };
    // the new b of own raw-b point (i, j, k), the normal component zero on a
    // conducting wall (App. A.4)
    auto put_b = [&](int i, int j, int k, const R bnew[3]) {
        const int gi = g.o[0] - 1 + i, gj = g.o[1] - 1 + j, gk = g.o[2] - 1 + k;
        const int64_t gp = gi + gidx.n0 * gj + gidx.n01 * gk;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const bool wall0 = WALLS && B.wall == c && (c == 0 ? gi : (c == 1 ? gj : gk)) == 0;
            B.bn[c * B.nc + gp] = wall0 ? R(0) : bnew[c];
        }
    };
    if (F4) {
        // the fourth-order curl reaches two cells out, past the staged halo:
        // b^t from HBM, exactly as the HBM path forms it (staging the wider e
        // instead changed the push by 0.2 %)
        for (int q = tid; q < g.BN; q += NT) {
            const int jk = div_small(q, mBX), i = q - jk * BX;
            const int k = div_small(jk, mBY), j = jk - k * g.BY;
            const int gi = g.o[0] - 1 + i, gj = g.o[1] - 1 + j, gk = g.o[2] - 1 + k;
            if (STEP && own(i, j, k)) {
                R bnew[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const R cu = curl4_e(B, c, gi, gj, gk);
                    bnew[c] = rb[c * g.BN + q] - dt * cu;
                    rb[c * g.BN + q] = rb[c * g.BN + q] - hdt * cu;
                }
                put_b(i, j, k, bnew);
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) rb[c * g.BN + q] = bt_global<R, 1>(B, c, gi, gj, gk, hdt);
            }
        }
    } else {
        const R *ex = re, *ey = re + g.JN, *ez = re + 2 * g.JN;
        for (int q = tid; q < g.BN; q += NT) {
            const int jk = div_small(q, mBX), i = q - jk * BX;
            const int k = div_small(jk, mBY), j = jk - k * g.BY;
            const int p = i + JX * j + JXY * k;
            const R cu[3] = {(ez[p + JX] - ez[p]) - (ey[p + JXY] - ey[p]),
                             (ex[p + JXY] - ex[p]) - (ez[p + 1] - ez[p]),
                             (ey[p + 1] - ey[p]) - (ex[p + JX] - ex[p])};
            const R bo[3] = {rb[q], rb[g.BN + q], rb[2 * g.BN + q]};
            rb[q] = bo[0] - hdt * cu[0];
            rb[g.BN + q] = bo[1] - hdt * cu[1];
            rb[2 * g.BN + q] = bo[2] - hdt * cu[2];
            if (STEP && own(i, j, k)) {
                const R bnew[3] = {bo[0] - dt * cu[0], bo[1] - dt * cu[1], bo[2] - dt * cu[2]};
                put_b(i, j, k, bnew);
            }
        }
    }
    if (!any) return false;
    __syncthreads();

    // 3. node fields on the (ext+1)^3 nodes of the tile (App. A.3.3)
    {
        const R *ex = re, *ey = re + g.JN, *ez = re + 2 * g.JN;
        const R *bx = rb, *by = rb + g.BN, *bz = rb + 2 * g.BN;
        for (int q = tid; q < g.NN; q += NT) {
            const int jk = div_small(q, mNX), i = q - jk * NX;
            const int k = div_small(jk, mNY), j = jk - k * g.NY;
            // raw coordinates of node (i,j,k) are (i+1, j+1, k+1)
            const int pe = (i + 1) + JX * (j + 1) + JXY * (k + 1);
            const int pb = (i + 1) + BX * (j + 1) + BXY * (k + 1);
            node[q] = node_avg2(ex[pe - 1], ex[pe]);
            node[g.NN + q] = node_avg2(ey[pe - JX], ey[pe]);
            node[2 * g.NN + q] = node_avg2(ez[pe - JXY], ez[pe]);
            node[3 * g.NN + q] = node_avg4(bx[pb], bx[pb - BX], bx[pb - BX - BXY], bx[pb - BXY]);
            node[4 * g.NN + q] = node_avg4(by[pb], by[pb - BXY], by[pb - 1 - BXY], by[pb - 1]);
            node[5 * g.NN + q] = node_avg4(bz[pb], bz[pb - 1], bz[pb - 1 - BX], bz[pb - BX]);
        }
    }
    __syncthreads();

    // 4. per cell and component, the trilinear interpolant of the eight node
    //    values as c0 + c1 x + c2 y + c3 z + c4 xy + c5 yz + c6 zx + c7 xyz in
    //    the in-cell offsets (the same polynomial, 8 instead of 16 operations
    //    per component at the particle)
    {
        const int ncell = g.ext[0] * g.ext[1] * g.ext[2];
        const int mEX = 65536 / g.ext[0] + 1, mEY = 65536 / g.ext[1] + 1;
        for (int q = tid; q < ncell; q += NT) {
            const int jk = div_small(q, mEX), i = q - jk * g.ext[0];
            const int k = div_small(jk, mEY), j = jk - k * g.ext[1];
            R *cf = coef + kCoef<R> * (i | (j << tsx) | (k << tsxy));
            const int m = i + NX * j + NXY * k;
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                const R *F = node + c * g.NN + m;
                const R f[8] = {F[0], F[1], F[NX], F[1 + NX], F[NXY], F[1 + NXY], F[NX + NXY], F[1 + NX + NXY]};
                trilinear_coef(f, cf + 8 * c);
            }
        }
    }
    __syncthreads();
    return true;
}

// Overflow sweep: same physics, fields from HBM, current by global atomics.
template <typename R, int WALLS, int F4, int NT>
__device__ void push_overflow(const BoxDev<R> &B, int kblk, const StepConst<R> &C)
{
    using JT = typename JType<R>::T;
    const R hdt = R(0.5) * C.dt;
    for (int s = 0; s < C.nsp; ++s) {
        const SpeciesDev<R> &S = B.sp[s];
        const TileRanges rg = overflow_range(B, S, C.cur);
        const int n = rg.n;
        const int start = rg.start;
        const PBuf<R> &P = S.buf[C.cur];
        const R hk = R(0.5) * C.kq[s] * C.dt;
        const R scale = -C.qs[s] * qscale_bits<R>();
        for (int pb = kblk * NT; pb < n; pb += NT * kOvfBlocks) {
            const int p = pb + (int)threadIdx.x;
            const bool valid = p < n;
            const int idx = start + (valid ? p : 0);
            int32_t cell = 0, id = 0;
            R d[3] = {R(0.5), R(0.5), R(0.5)}, u[3] = {R(0), R(0), R(0)};
            if (valid) {
                cell = P.cell[idx];
                const PSlot<R> ps = slot_at(P, idx);
                for (int a = 0; a < 3; ++a) { d[a] = ps.d(a); u[a] = ps.u(a); }
                if (P.id) id = P.id[idx];
            }
            const int ix = cell_x(cell), iy = cell_y(cell), iz = cell_z(cell);
            R E[3], Bf[3];
            if (valid) gather_global<R, F4>(B, ix, iy, iz, d, hdt, E, Bf);
            else for (int a = 0; a < 3; ++a) { E[a] = R(0); Bf[a] = R(0); }
            R D[3];
            boris_move(hk, E, Bf, u, C.dt, valid, C.flags, D);
            // a move through a conducting wall (App. A.4): deposit up to the
            // wall, then the mirrored rest; the particle ends at P2 + D2
            R D1[3], P2[3], D2[3];
            const bool hitw = WALLS && B.wall >= 0 && valid &&
                              wall_hit(B.wall, B.wall == 0 ? ix : (B.wall == 1 ? iy : iz), B.n[B.wall], d, D, D1, P2,
                                       D2, u);
            if (valid) {
                JT *J = B.J;
                auto put_j = [&](int a, int ox, int oy, int oz, JT q) {
                    if (q == JT(0)) return;
                    const int i = wrap_idx(ix + ox, B.n[0]), j = wrap_idx(iy + oy, B.n[1]),
                              k = wrap_idx(iz + oz, B.n[2]);
                    atomic_add_global(&J[a * B.nc + i + (int64_t)B.n[0] * (j + (int64_t)B.n[1] * k)], q);
                };
                if (hitw) {
                    deposit_move(d, D1, scale, put_j);
                    R Q2[3] = {P2[0], P2[1], P2[2]};
                    int s2[3];
                    wall_rest_start(B.wall, Q2, s2);
                    deposit_rest(Q2, D2, scale, [&](int a, int ox, int oy, int oz, JT q) {
                        put_j(a, s2[0] + ox, s2[1] + oy, s2[2] + oz, q);
                    });
                } else {
                    deposit_move(d, D, scale, put_j);
                }
            }
            R x1[3] = {d[0] + D[0], d[1] + D[1], d[2] + D[2]}, dn[3];
            if (hitw)
                for (int a = 0; a < 3; ++a) x1[a] = P2[a] + D2[a];
            const int32_t nc = advance_cell(B, ix, iy, iz, x1, dn);
            store_particle(B, S, C.cur ^ 1, tile_of(B, nc), valid, nc, dn, u, id, C.flags);
        }
    }
}

// The push of one work item by a block of NT threads.  FIX: 0 tiles of any
// shape, 1 all tiles 4x4x4 and every particle copy below 4 GiB (32-bit slot
// addresses), 2 all tiles 4x4x4.
template <typename R, int FIX, int WALLS, int F4, int NT>
__device__ __forceinline__ void push_block(const BoxDev<R> *__restrict__ boxes, const Item *__restrict__ items,
                                           const StepConst<R> &C)
{
    using JT = typename JType<R>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    const Item it = items[blockIdx.x];
    if (it.box < 0) return;                       // padding of the push order
    const BoxDev<R> &B = boxes[it.box];
    if (it.tile < 0) {
        push_overflow<R, WALLS, F4, NT>(B, -1 - it.tile, C);
        return;
    }
    const int T = it.tile;
    const int tid = threadIdx.x;
    const TileGeom<R> g = tile_geom<R, FIX>(B, T);
    const TileRim rim = tile_rim(B, g);
    // 4x4x4 tiles take the packed loop, except those on a conducting wall and
    // the FP64 form with walls, whose 168 registers do not hold both loops: with
    // the packed one in it the kernel had 272 B of scratch per lane and took 390
    // us on 64^3 cells with 16 pairs per cell, with the general loop alone 292
    constexpr bool kPacked = FIX != 0 && !(WALLS != 0 && sizeof(R) == 8);
    bool packed = kPacked;
    if (WALLS) {
#pragma unroll
        for (int a = 0; a < 3; ++a) packed = packed && !(B.wall == a && (g.o[a] == 0 || g.o[a] + g.ext[a] == B.n[a]));
    }
    TileMove mv;
    mv.init(B, g);
    // per axis: box edge length, whether the tile touches the box edge (only
    // then can a move wrap), and whether one tile spans the box
    int bn[3];
    bool edge[3], span[3];
    bool fastbin = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        bn[a] = B.n[a];
        edge[a] = g.o[a] == 0 || g.o[a] + g.ext[a] >= bn[a];
        span[a] = B.ntile[a] == 1;
        // with two tiles along an axis the cells on both sides of a tile are
        // the same cells, and a partial tile at the box's far end has its
        // own extent: move_bin's rule decides there
        fastbin &= B.ntile[a] != 2 && g.ext[a] == 4;
    }
    // LDS: per-cell trilinear coefficients | piece queues | union of {raw e,
    // raw b, node fields} (set-up) and the tile current (particle loop)
    const int tsx = FIX ? 2 : B.tshift[0], tsxy = FIX ? 4 : B.tshift[0] + B.tshift[1];
    const int tsz = FIX ? 2 : B.tshift[2];
    constexpr int kWaves = NT / 64;
    const TileLds lds = FIX ? tile_lds<R>(4, 4, 4, kWaves)
                            : tile_lds<R>(1 << B.tshift[0], 1 << B.tshift[1], 1 << B.tshift[2], kWaves);
    R *coef = reinterpret_cast<R *>(smem);
    unsigned char *qmem = smem + lds.coef;
    unsigned char *uni = qmem + lds.stage;
    R *re = reinterpret_cast<R *>(qmem);          // raw e, 3 x JN, origin o-1 (set-up)
    R *rb = re + 3 * g.JN;                        // raw b, 3 x BN, origin o-1 (set-up)
    R *node = reinterpret_cast<R *>(uni);         // node fields, 6 x NN, origin o (set-up)
    JT *jl = reinterpret_cast<JT *>(uni);         // J, 3 x JN, origin o-1 (particle loop)

    // re-binning counters: per species the stayers (from the front of the
    // tile's new A range), the leavers (staged from the back) and the leavers
    // per neighbour direction
    __shared__ int sh_cnt[2][kMaxSpecies];        // [0] stayers, [1] leavers
    __shared__ int sh_bin[kMaxSpecies][27], sh_base[kMaxSpecies][27];
    // hand-over targets per (species, direction): first slot of the claimed
    // part of the target tile's segment, and the segment's end
    __shared__ int sh_tseg[kMaxSpecies][27], sh_tend[kMaxSpecies][27];
    // hand-over sources per species: the arrays of copy cur^1, and the slot
    // of leaver q of the block's combined leaver range is q + sh_loff[s]
    __shared__ PBuf<R> sh_q[kMaxSpecies];
    __shared__ int sh_loff[kMaxSpecies], sh_lend[kMaxSpecies];
    // per species the tile's ranges in copy cur (start, na, bs, n) and its
    // segment start in copy cur^1, read here, while the fields are staged,
    // instead of at the start of each species' loop and in the hand-over
    __shared__ int sh_rng[kMaxSpecies][5];
    if (tid < 2 * kMaxSpecies) (&sh_cnt[0][0])[tid] = 0;
    if (tid < kMaxSpecies * 27) (&sh_bin[0][0])[tid] = 0;
    if (tid < C.nsp) {
        const TileRanges r = tile_ranges(B.sp[tid], C.cur, T);
        sh_rng[tid][0] = r.start;
        sh_rng[tid][1] = r.na;
        sh_rng[tid][2] = r.bs;
        sh_rng[tid][3] = r.n;
        sh_rng[tid][4] = B.sp[tid].seg_start[C.cur ^ 1][T];
    }

    const TileGrid<R> grid(B, g);
    // strides of the tile current
    const CurrentGrid cg = FIX ? CurrentGrid(4, 4, 4) : CurrentGrid(1 << B.tshift[0], 1 << B.tshift[1], 1 << B.tshift[2]);
    const int JX = cg.x, JXY = cg.xy;
    const R hdt = R(0.5) * C.dt;

    // the particle loops load each lane's next particle one iteration ahead
    // (lanes past the end load the tile's last particle again and are masked
    // out of every store, claim and deposit by `valid`); the tile's first
    // particles are loaded during the set-up, once the ranges are known, so
    // that their HBM latency is covered by the rest of it
    int32_t nx_code = 0, nx_id = 0;
    R nx_d[3] = {R(0.5), R(0.5), R(0.5)}, nx_u[3] = {R(0), R(0), R(0)};
    auto fetch_particle = [&](const PBuf<R> &P, const TileRanges &src, int q) {
        const int at = src.slot(min(q, src.n - 1));
        const PSlot<R> ps = slot_at<FIX == 1>(P, at);
        nx_code = ps.code();
        nx_d[0] = ps.d(0); nx_d[1] = ps.d(1); nx_d[2] = ps.d(2);
        nx_u[0] = ps.u(0); nx_u[1] = ps.u(1); nx_u[2] = ps.u(2);
        if (P.id) nx_id = slot_ref(P.id, at);
    };
    auto ranges = [&](int s) {
        TileRanges r;
        r.start = __builtin_amdgcn_readfirstlane(sh_rng[s][0]);
        r.na = __builtin_amdgcn_readfirstlane(sh_rng[s][1]);
        r.bs = __builtin_amdgcn_readfirstlane(sh_rng[s][2]);
        r.n = __builtin_amdgcn_readfirstlane(sh_rng[s][3]);
        return r;
    };
    // the next species after s that has particles in the tile, C.nsp if none
    auto next_species = [&](int s) {
        do ++s;
        while (s < C.nsp && __builtin_amdgcn_readfirstlane(sh_rng[s][3]) <= 0);
        return s;
    };
    int s0 = 0;
    const bool any = tile_coefs<R, FIX, WALLS, F4, true, NT>(B, g, grid, C.dt, coef, re, rb, node, [&]() {
        s0 = next_species(-1);
        if (s0 < C.nsp) fetch_particle(B.sp[s0].buf[C.cur], ranges(s0), tid);
        return s0 < C.nsp;
    });
    // a tile without particles has written its b and hands nothing over (na of
    // the other copy is zero already): two thirds of the tiles of a 796 x 632 x 4
    // Harris sheet, whose push takes 0.515 ms with this and 0.548 without
    if (!any) return;
    for (int q = tid; q < 3 * cg.n; q += NT) jl[q] = JT(0);
    __syncthreads();

    // 5. particles of every species: gather, push, move, deposit, re-bin
    // uniform index offsets of the twelve faces of a piece (see deposit_piece)
    int joff[3][4];
    {
        const int S[3] = {1, JX, JXY};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int b1 = a == 2 ? 0 : a + 1, b2 = a == 0 ? 2 : a - 1;
            joff[a][0] = a * cg.n;
            joff[a][1] = a * cg.n + S[b2];
            joff[a][2] = a * cg.n + S[b1];
            joff[a][3] = a * cg.n + S[b1] + S[b2];
        }
    }
    // this wave's queue of unfinished moves: meta word (move_meta), start of
    // the next piece and end of the move
    const int wave = tid >> 6, lane = __lane_id();
    constexpr int kQCap = QCap<R>::value;
    int32_t *qmeta = reinterpret_cast<int32_t *>(qmem) + wave * kQCap;
    R *qval = reinterpret_cast<R *>(qmem + kWaves * kQCap * sizeof(int32_t)) + wave * 6 * kQCap;
    int qhead = 0, qcount = 0;                    // wave-uniform
    auto put = [&](bool has, int32_t meta, const R ps[3], const R x1[3]) {
        const uint64_t mh = __ballot(has);
        if (has) {
            const int pos = (qhead + qcount + lane_rank(mh)) & (kQCap - 1);
            qmeta[pos] = meta;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                qval[a * kQCap + pos] = ps[a];
                qval[(3 + a) * kQCap + pos] = x1[a];
            }
        }
        qcount += (int)__popcll(mh);
    };
    // deposit the next piece of up to 64 queued moves (whole wave); moves with
    // pieces left go back into the queue
    auto drain = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int nq = min(qcount, 64);
        int32_t meta = 0;
        R ps[3] = {R(0), R(0), R(0)}, x1[3] = {R(0), R(0), R(0)};
        if (lane < nq) {
            const int e = (qhead + lane) & (kQCap - 1);
            meta = qmeta[e];
#pragma unroll
            for (int a = 0; a < 3; ++a) { ps[a] = qval[a * kQCap + e]; x1[a] = qval[(3 + a) * kQCap + e]; }
        }
        qhead = (qhead + nq) & (kQCap - 1);
        qcount -= nq;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int k = meta_k(meta), nb = meta_nb(meta);
        bool more = false;
        R pe[3] = {x1[0], x1[1], x1[2]};
        if (lane < nq) {
            int offc[3];
            R sv[3], dd[3];
            chain_piece(ps, x1, meta, k, pe, offc, sv, dd);
            const int cb = ((meta >> kMetaJ) & 8191) + offc[0] + __mul24(JX, offc[1]) + __mul24(JXY, offc[2]);
            const R sc = meta < 0 ? -qscale_bits<R>() : qscale_bits<R>();
            deposit_piece<R>(jl, cb, joff, sv, dd, sc);
            more = k < nb;
        }
        put(more, meta + (1 << kMetaK), pe, x1);
    };
    // Particle loop of 4x4x4 tiles.  What bounds it: on the 64^3 thermal box
    // (33.5 M particles) the vector ALU, the LDS and HBM are each busy for
    // 0.67-0.75 of the launch, so it is written for few instructions and for
    // no wait that the data does not force (0.540 ms with the general loop,
    // 0.510 ms with this one, 0.500 with CurrentGrid's planes; 430 -> 376 VALU
    // instructions per 64 particles):
    // - cells, moves and bins are packed words (TileMove), every particle of
    //   the tile's ranges goes to the tile or to one next to it, and no lane
    //   takes a path of its own;
    // - every iteration issues the same loads and stores, none behind a branch
    //   (idle lanes store to the buffer's spare slots): the wait for the next
    //   particle's loads then leaves this iteration's stores in flight.  Behind
    //   a branch the compiler has to wait for all of them;
    // - the buffers' addresses and the species' constants are read where the
    //   species changes, and the first particles of the next species are
    //   loaded one iteration ahead like any others.
    auto packed_loop = [&]() {
        int s = s0;
        if (s >= C.nsp) return;
        TileRanges src = ranges(s), nsrc = src;
        PBuf<R> P = B.sp[s].buf[C.cur], Q = B.sp[s].buf[C.cur ^ 1];
        R hk = R(0.5) * C.kq[s] * C.dt, scale = -C.qs[s] * qscale_bits<R>();
        int32_t sgnbit = scale < R(0) ? (int32_t)0x80000000 : 0;
        int dst_start = __builtin_amdgcn_readfirstlane(sh_rng[s][4]), spare = B.sp[s].slots;
        const R dt = C.dt;
        // the first particles are waited for here: a wait at the loop's top
        // that also covers the entry could not leave stores in flight
#pragma unroll
        for (int a = 0; a < 3; ++a) asm volatile("" : "+v"(nx_d[a]), "+v"(nx_u[a]));
        asm volatile("" : "+v"(nx_code), "+v"(nx_id));
        for (int pb = 0;;) {
            const bool valid = pb + tid < src.n;
            const uint32_t code = (uint32_t)nx_code & 63u;
            const int id = nx_id;
            const R d[3] = {nx_d[0], nx_d[1], nx_d[2]};
            R u[3] = {nx_u[0], nx_u[1], nx_u[2]};
            int ns = s, npb = pb + NT;
            if (npb >= src.n) {
                ns = next_species(s);
                npb = 0;
                if (ns < C.nsp) {
                    nsrc = ranges(ns);
                    P = B.sp[ns].buf[C.cur];
                }
            }
            // past the last chunk every lane reloads the last particle
            fetch_particle(P, nsrc, ns < C.nsp ? npb + tid : nsrc.n);

            // gather, Boris step, move
            const uint32_t pc = __umul24(code, 0x1041u) & kThrees;
            const R *cf = coef + __umul24(kCoef<R>, code);
            R E[3], Bf[3], D[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) E[c] = trilinear_eval(cf + 8 * c, d);
#pragma unroll
            for (int c = 0; c < 3; ++c) Bf[c] = trilinear_eval(cf + 24 + 8 * c, d);
            boris_move(hk, E, Bf, u, dt, valid, C.flags, D);

            // node planes crossed (move_crossings): floor of the end is the
            // crossing direction, its positive part the plane
            R x1[3], fl[3], pl[3], lam[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                x1[a] = d[a] + D[a];
                fl[a] = floor(x1[a]);
                pl[a] = clamp01(fl[a]);
                lam[a] = fl[a] != R(0) ? (pl[a] - d[a]) * fast_rcp(D[a]) : R(2);
            }
            const int F = (int)fma(fl[2], R(65536), fma(fl[1], R(256), fl[0]));
            const bool cross = F != 0;
            const uint32_t Pw = pc + kFours + (uint32_t)F;
            uint32_t t, q;
            mv.to(Pw, t, q);

            // re-binning: lanes 0 and 1 claim the wave's stayer and leaver slots
            const bool stay = valid && t == kOnes, lv = valid && t != kOnes;
            const uint64_t ms = __ballot(stay), ml = __ballot(lv);
            int claimed = 0;
            if (lane < 2) claimed = atomicAdd(&sh_cnt[lane][s], lane ? (int)__popcll(ml) : (int)__popcll(ms));
            if (lv) atomicAdd(&sh_bin[s][udot4(t, 0x090301u)], 1);

            // deposit: the first piece at once, the rest of the move queued;
            // the crossings in (stable) increasing order of their parameter
            const bool c10 = lam[1] < lam[0], c20 = lam[2] < lam[0], c21 = lam[2] < lam[1];
            const bool f2 = c20 && c21;
            const R l0 = f2 ? lam[2] : (c10 ? lam[1] : lam[0]);
            const int jb = (int)udot4(pc, 1u | ((uint32_t)cg.x << 8) | ((uint32_t)cg.xy << 16)) + 1 + cg.x + cg.xy;
            R p1[3] = {x1[0], x1[1], x1[2]};
            if (cross) {
                const R q0 = clamp01(fma(l0, D[0], d[0])), q1 = clamp01(fma(l0, D[1], d[1])),
                        q2 = clamp01(fma(l0, D[2], d[2]));
                p1[0] = f2 || c10 ? q0 : pl[0];
                p1[1] = !f2 && c10 ? pl[1] : q1;
                p1[2] = f2 ? pl[2] : q2;
            }
            if (valid) {
                const R dd[3] = {p1[0] - d[0], p1[1] - d[1], p1[2] - d[2]};
                deposit_piece<R>(jl, jb, joff, d, dd, scale);
            }

            // store: stayers from the front of the tile's segment, leavers from
            // the back of its first n slots, idle lanes to the spare slots
            {
                const int fb = dst_start + __builtin_amdgcn_readlane(claimed, 0);
                const int bb = dst_start + src.n - 1 - __builtin_amdgcn_readlane(claimed, 1);
                int at = stay ? fb + lane_rank(ms) : bb - lane_rank(ml);
                at = valid ? at : spare + lane;
                const PSlot<R> ps = slot_at<FIX == 1>(Q, at);
                ps.code() = (uint8_t)(stay ? udot4(q, 0x100401u) : leaver_code(Pw));
#pragma unroll
                for (int a = 0; a < 3; ++a) ps.d(a) = offset_in_cell(x1[a]);
#pragma unroll
                for (int a = 0; a < 3; ++a) ps.u(a) = u[a];
                if (Q.id) slot_ref(Q.id, at) = id;
            }

            if (kQCap < 128) {
                const int cnt = (int)__popcll(__ballot(valid && cross));
                while (qcount + cnt > kQCap) drain();
            }
            {
                const uint32_t Fw = kOnes + (uint32_t)F;
                const int nb = 3 - __popc(Fw & kOnes);
                const int o012 = c10 ? (c20 ? (c21 ? 2 | (1 << 2) : 1 | (2 << 2)) | (0 << 4) : 1 | (2 << 4))
                                     : (c21 ? (c20 ? 2 | (1 << 4) : (2 << 2) | (1 << 4)) : (1 << 2) | (2 << 4));
                put(valid && cross, (int)Fw | (1 << kMetaK) | (nb << kMetaNb) | (o012 << kMetaO) | (jb << kMetaJ) | sgnbit,
                    p1, x1);
            }
            while (qcount >= 64) drain();

            if (ns >= C.nsp) break;
            if (ns != s) {
                s = ns;
                src = nsrc;
                Q = B.sp[s].buf[C.cur ^ 1];
                hk = R(0.5) * C.kq[s] * C.dt;
                scale = -C.qs[s] * qscale_bits<R>();
                sgnbit = scale < R(0) ? (int32_t)0x80000000 : 0;
                dst_start = __builtin_amdgcn_readfirstlane(sh_rng[s][4]);
                spare = B.sp[s].slots;
            }
            pb = npb;
        }
    };
    if constexpr (kPacked) {
        if (packed) packed_loop();
    }
    // the general loop: other tile shapes, tiles on a conducting wall
    if constexpr (FIX == 0 || WALLS != 0)
    if (!packed)
    for (int s = 0; s < C.nsp; ++s) {
        const SpeciesDev<R> &S = B.sp[s];
        const PBuf<R> &P = S.buf[C.cur];
        const TileRanges src = ranges(s);
        const int n = src.n;
        const R hk = R(0.5) * C.kq[s] * C.dt;
        const R scale = -C.qs[s] * qscale_bits<R>();
        const int32_t sgnbit = scale < R(0) ? (int32_t)0x80000000 : 0;
        const int dst = C.cur ^ 1;
        const int dst_start = __builtin_amdgcn_readfirstlane(sh_rng[s][4]);
        const int ovf0 = S.slots - S.ovf_cap;           // first slot of the overflow region
        auto fetch = [&](int q) { fetch_particle(P, src, q); };
        if (n > 0 && s != s0) fetch(tid);                // the first species: loaded during the set-up
        for (int pb = 0; pb < n; pb += NT) {
            const int p = pb + tid;
            const bool valid = p < n;
            const int code = nx_code, id = nx_id;
            R d[3] = {nx_d[0], nx_d[1], nx_d[2]}, u[3] = {nx_u[0], nx_u[1], nx_u[2]};
            if (pb + NT < n) fetch(p + NT);
            const int lx = code & ((1 << tsx) - 1), ly = (code >> tsx) & ((1 << (tsxy - tsx)) - 1), lz = code >> tsxy;
            const int ix = g.o[0] + lx, iy = g.o[1] + ly, iz = g.o[2] + lz;
            // a particle of the tile's ranges has its cell in the tile; a code
            // past a partial tile's extent would index the tile's LDS out of
            // range, so it takes the HBM path instead
            const bool inside = (unsigned)lx < (unsigned)g.ext[0] && (unsigned)ly < (unsigned)g.ext[1] &&
                                (unsigned)lz < (unsigned)g.ext[2];
            // gather: the cell's trilinear interpolant at the in-cell offset
            R E[3] = {R(0), R(0), R(0)}, Bf[3] = {R(0), R(0), R(0)};
            if (!inside) {
                gather_global<R, F4>(B, ix, iy, iz, d, hdt, E, Bf);
            } else {
                const R *cf = coef + __umul24(kCoef<R>, lx | (ly << tsx) | (lz << tsxy));
                R F[6];
#pragma unroll
                for (int c = 0; c < 6; ++c) F[c] = trilinear_eval(cf + 8 * c, d);
                E[0] = F[0]; E[1] = F[1]; E[2] = F[2];
                Bf[0] = F[3]; Bf[1] = F[4]; Bf[2] = F[5];
            }
            R D[3];
            boris_move(hk, E, Bf, u, C.dt, valid, C.flags, D);

            // node planes crossed by the move (end x1 in the home-cell frame)
            R x1[3], lam[3];
            int dir[3];
            move_crossings(d, D, x1, dir, lam);
            // conducting walls (App. A.4): a move through a wall ends at the
            // mirrored point P2 + D2; its deposit is the piece d -> d + D1
            // (below) and the queued move P2 -> P2 + D2
            bool hitw = false;
            R P2[3], D2[3], D1[3];
            if (WALLS && B.wall >= 0) {
                const int w = B.wall;
                hitw = valid && wall_hit(w, w == 0 ? ix : (w == 1 ? iy : iz), B.n[w], d, D, D1, P2, D2, u);
                if (hitw) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        x1[a] = P2[a] + D2[a];
                        dir[a] = x1[a] < R(0) ? -1 : (x1[a] >= R(1) ? 1 : 0);
                    }
                }
            }

            // new cell and offset, re-binning target, and the slot claims:
            // one returning LDS atomic for the stayers' block of slots and one
            // for the leavers' staging slots, each by the lowest lane of its
            // group, plus a per-direction count for each leaver
            // (the periodic wrap only where a lane may cross the box edge: in
            // a tile on the edge, or when a lane came from outside its tile)
            const bool anyout = __ballot(valid && !inside) != 0;
            int cn[3] = {ix, iy, iz}, lc[3] = {lx, ly, lz};
            R dn[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int f = dir[a];                 // floor(x1)
                dn[a] = offset_in_cell(x1[a]);
                lc[a] += f;
                int ci = cn[a] + f;
                if (edge[a] || anyout) ci = ci < 0 ? ci + bn[a] : (ci >= bn[a] ? ci - bn[a] : ci);
                cn[a] = ci;
            }
            const int32_t ncell = pack_cell(cn[0], cn[1], cn[2]);
            const int ncode = (cn[0] & ((1 << tsx) - 1)) | ((cn[1] & ((1 << (tsxy - tsx)) - 1)) << tsx) |
                              ((cn[2] & ((1 << tsz) - 1)) << tsxy);
            const int tn = tile_of(B, ncell);
            // re-binning: stayers take the next slots at the front of the
            // tile's new A range, leavers into an adjacent tile are staged from
            // the back (both claimed with one LDS atomic per wave); anything
            // else claims its target's B range with a global atomic
            int bin;
            if (FIX && fastbin && !anyout) {
                // every valid lane started in this full 4x4x4 tile and moved at
                // most one cell per axis: its direction code from the local
                // cell, (lc + 4) >> 2 = 0, 1, 2 for lc = -1, 0..3, 4, and 1 on
                // an axis that one tile spans (it wraps into the same tile);
                // the same code as move_bin's
                int code = 0;
#pragma unroll
                for (int a = 0; a < 3; ++a) code += ((span[a] ? 4 : lc[a] + 4) >> 2) * (a == 0 ? 1 : (a == 1 ? 3 : 9));
                bin = valid ? code : -1;
            } else {
                bin = valid ? move_bin(g, rim, cn) : -1;
            }
            const bool stay = bin == 13, lv = bin >= 0 && bin != 13;
            const uint64_t ms = __ballot(stay), ml = __ballot(lv);
            const int sl = ms ? __ffsll((unsigned long long)ms) - 1 : 0;
            const int ll = ml ? __ffsll((unsigned long long)ml) - 1 : 0;
            int fb = 0, bb = 0;
            if (stay && lane == sl) fb = atomicAdd(&sh_cnt[0][s], (int)__popcll(ms));
            if (lv && lane == ll) bb = atomicAdd(&sh_cnt[1][s], (int)__popcll(ml));
            if (lv) atomicAdd(&sh_bin[s][bin], 1);
            fb = __builtin_amdgcn_readlane(fb, sl);
            bb = __builtin_amdgcn_readlane(bb, ll);
            int at = -1;
            if (stay) {
                at = dst_start + fb + lane_rank(ms);
            } else if (lv) {
                at = dst_start + n - 1 - (bb + lane_rank(ml));
            } else if (valid) {
                const int slot = atomicAdd(&S.nb[dst][tn], 1);
                at = b_range_slot(B, S, dst, tn, S.bs[dst][tn] + slot, C.flags);
            }
            if (at >= 0) write_particle<FIX == 1>(S.buf[dst], at, lv || at >= ovf0, ncell, ncode, dn, u, id);

            // deposit: the first piece (in the home cell) at once, the move
            // into the wave's queue for its later pieces; the crossings in
            // increasing order of their parameter (axes o0, o1, o2)
            if (WALLS && hitw) {
#pragma unroll
                for (int a = 0; a < 3; ++a) D[a] = D1[a];
                move_crossings(d, D, x1, dir, lam);
            }
            const int nb = (dir[0] != 0) + (dir[1] != 0) + (dir[2] != 0);
            int o0 = 0, o1 = 1, o2 = 2;
            R l0 = lam[0], l1 = lam[1], l2 = lam[2];
            if (l1 < l0) { R t = l0; l0 = l1; l1 = t; int q = o0; o0 = o1; o1 = q; }
            if (l2 < l1) { R t = l1; l1 = l2; l2 = t; int q = o1; o1 = o2; o2 = q; }
            if (l1 < l0) { R t = l0; l0 = l1; l1 = t; int q = o0; o0 = o1; o1 = q; }
            const int jb = (lx + 1) + __mul24(JX, ly + 1) + __mul24(JXY, lz + 1);
            R p1[3];
            if (nb == 0) {
                p1[0] = x1[0]; p1[1] = x1[1]; p1[2] = x1[2];
            } else {
                first_breakpoint(d, D, dir, o0, l0, p1);
            }
            if (valid && inside) {
                const R dd[3] = {p1[0] - d[0], p1[1] - d[1], p1[2] - d[2]};
                deposit_piece<R>(jl, jb, joff, d, dd, scale);
            } else if (valid) {
                PIC_GLOBAL JT *J = B.J;
                deposit_move(d, D, scale, [&](int a, int ox, int oy, int oz, JT q) {
                    if (q == JT(0)) return;
                    const int i = wrap_idx(ix + ox, B.n[0]), j = wrap_idx(iy + oy, B.n[1]),
                              k = wrap_idx(iz + oz, B.n[2]);
                    atomic_add_global(&J[a * B.nc + i + (int64_t)B.n[0] * (j + (int64_t)B.n[1] * k)], q);
                });
            }
            if (kQCap < 128) {
                const int cnt = (int)__popcll(__ballot(valid && inside && nb > 0));
                while (qcount + cnt > kQCap) drain();
            }
            put(valid && inside && nb > 0, move_meta(1, nb, o0, o1, o2, dir) | (jb << kMetaJ) | sgnbit, p1, x1);
            while (qcount >= 64) drain();
            if (WALLS && B.wall >= 0 && __ballot(hitw)) {
                // the mirrored rest of the moves that hit a wall: a whole move
                // from its first piece (next piece 0) through the queue
                R y1[3], lb[3];
                int db[3], s2[3];
                wall_rest_start(B.wall, P2, s2);
                move_crossings(P2, D2, y1, db, lb);
                const int nb2 = (db[0] != 0) + (db[1] != 0) + (db[2] != 0);
                int q0 = 0, q1 = 1, q2 = 2;
                R m0 = lb[0], m1 = lb[1], m2 = lb[2];
                if (m1 < m0) { R t = m0; m0 = m1; m1 = t; int q = q0; q0 = q1; q1 = q; }
                if (m2 < m1) { R t = m1; m1 = m2; m2 = t; int q = q1; q1 = q2; q2 = q; }
                if (m1 < m0) { R t = m0; m0 = m1; m1 = t; int q = q0; q0 = q1; q1 = q; }
                const int jb2 = jb + s2[0] + __mul24(JX, s2[1]) + __mul24(JXY, s2[2]);
                if (kQCap < 128) {
                    const int cnt = (int)__popcll(__ballot(hitw && inside));
                    while (qcount + cnt > kQCap) drain();
                }
                put(hitw && inside, move_meta(0, nb2, q0, q1, q2, db) | (jb2 << kMetaJ) | sgnbit, P2, y1);
                if (hitw && !inside) {
                    PIC_GLOBAL JT *J = B.J;
                    deposit_rest(P2, D2, scale, [&](int a, int ox, int oy, int oz, JT q) {
                        if (q == JT(0)) return;
                        const int i = wrap_idx(ix + s2[0] + ox, B.n[0]), j = wrap_idx(iy + s2[1] + oy, B.n[1]),
                                  k = wrap_idx(iz + s2[2] + oz, B.n[2]);
                        atomic_add_global(&J[a * B.nc + i + (int64_t)B.n[0] * (j + (int64_t)B.n[1] * k)], q);
                    });
                }
                while (qcount >= 64) drain();
            }
        }
    }
    // 7a. every wave is past its particle loops, so the leaver counts per
    //     (species, direction) are final: claim their slots in the adjacent
    //     tiles' B ranges now, one global atomic each; the replies come back
    //     while the queues drain and the current is flushed
    __syncthreads();
    const int dst = C.cur ^ 1;
    int claim = 0, ctile = 0;
    const bool claimer = tid < C.nsp * 27;
    const int cs = claimer ? tid / 27 : 0, ck = claimer ? tid - 27 * cs : 0;
    const int ccnt = claimer ? sh_bin[cs][ck] : 0;
    int tbs = 0, tseg = 0, tcap = 0;
    if (ccnt > 0) {
        ctile = neighbor_tile(B, g, ck);
        claim = atomicAdd(&B.sp[cs].nb[dst][ctile], ccnt);
        // the target's layout, read while the queues drain
        const SpeciesDev<R> &S = B.sp[cs];
        tbs = S.bs[dst][ctile];
        tseg = S.seg_start[dst][ctile];
        tcap = S.seg_cap[dst][ctile];
    }
    if (tid < C.nsp) {
        const SpeciesDev<R> &S = B.sp[tid];
        S.na[dst][T] = sh_cnt[0][tid];
        // staged leavers of species tid: slots [first, first + nl) of copy cur^1
        const int nl = sh_cnt[1][tid];
        int before = 0;                                       // leavers of the species before it
        for (int s = 0; s < tid; ++s) before += sh_cnt[1][s];
        sh_q[tid] = S.buf[dst];
        sh_loff[tid] = sh_rng[tid][4] + sh_rng[tid][3] - nl - before;
        sh_lend[tid] = before + nl;
    }
    __syncthreads();
    // the staged leavers of all species form one range [0, ntot); a thread
    // loads up to kHand of them before it stores any, so that their HBM round
    // trips overlap instead of following each other.  The first batch is
    // loaded here: its round trips overlap the claims' replies, the drains
    // and the flush.
    constexpr int kHand = 4;
    const int ntot = C.nsp > 0 ? sh_lend[C.nsp - 1] : 0;
    int hsp[kHand], hcell[kHand], hid[kHand];
    R hd[kHand][3], hu[kHand][3];
    auto load_leavers = [&](int q0) {
#pragma unroll
        for (int h = 0; h < kHand; ++h) {
            const int q = q0 + h * NT;
            hsp[h] = -1;
            if (q < ntot) {
                int s = 0;
#pragma unroll
                for (int r = 0; r + 1 < kMaxSpecies; ++r) s += (r + 1 < C.nsp && q >= sh_lend[r]) ? 1 : 0;
                const PBuf<R> &Q = sh_q[s];
                const int from = q + sh_loff[s];
                const PSlot<R> ps = slot_at<FIX == 1>(Q, from);
                if (kPacked && (!WALLS || packed)) hcell[h] = ps.code();
                else hcell[h] = slot_ref(Q.cell, from);
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    hd[h][a] = ps.d(a);
                    hu[h][a] = ps.u(a);
                }
                hid[h] = Q.id ? slot_ref(Q.id, from) : 0;
                hsp[h] = s;
            }
        }
    };
    load_leavers(tid);
    while (qcount > 0) drain();
    __syncthreads();

    // 6. flush the tile current to HBM (integer sums: order-independent)
    const int mJX = 65536 / g.JX + 1, mJY = 65536 / g.JY + 1;
    for (int q = tid; q < g.JN; q += NT) {
        const int jk = div_small(q, mJX), i = q - jk * g.JX;
        const int k = div_small(jk, mJY), j = jk - k * g.JY;
        const JT *at = jl + i + JX * j + JXY * k;
        const JT v0 = at[0], v1 = at[cg.n], v2 = at[2 * cg.n];
        if (v0 != JT(0) || v1 != JT(0) || v2 != JT(0)) {
            const int64_t gp = grid(i, j, k);
            if (v0 != JT(0)) atomic_add_global(&B.J[gp], v0);
            if (v1 != JT(0)) atomic_add_global(&B.J[B.nc + gp], v1);
            if (v2 != JT(0)) atomic_add_global(&B.J[2 * B.nc + gp], v2);
        }
    }

    // 7b. hand the staged leavers over: the claimed positions and the target
    //     segments go to LDS, so that the copies below read no layout from HBM
    if (claimer) {
        if (ccnt > 0) {
            sh_base[cs][ck] = tbs + claim;                    // position in the target's segment
            sh_tseg[cs][ck] = tseg;
            sh_tend[cs][ck] = tcap;
        }
        sh_bin[cs][ck] = 0;                                   // now the rank counter
    }
    __syncthreads();
    // 7c. store each loaded leaver at its claimed slot, then load the next
    //     batch (tiles with more than kHand * NT leavers)
    for (int q0 = tid; q0 < ntot; q0 += kHand * NT) {
        if (q0 != tid) load_leavers(q0);
#pragma unroll
        for (int h = 0; h < kHand; ++h) {
            const int s = hsp[h];
            if (s < 0) continue;
            // the same bin as at staging, and the code in the new tile
            int k, code;
            if (kPacked && (!WALLS || packed)) {
                uint32_t t, q;
                mv.to(leaver_cell((uint32_t)hcell[h]), t, q);
                k = (int)udot4(t, 0x090301u);
                code = (int)udot4(q, 0x100401u);
            } else {
                const int c3[3] = {cell_x(hcell[h]), cell_y(hcell[h]), cell_z(hcell[h])};
                k = move_bin(g, rim, c3);
                code = local_code(B, hcell[h]);
            }
            const int pos = sh_base[s][k] + atomicAdd(&sh_bin[s][k], 1);
            const bool wide = pos >= sh_tend[s][k];
            int at;
            if (!wide) {
                at = sh_tseg[s][k] + pos;
            } else {                                    // the target segment is full: overflow region
                if (kPacked && (!WALLS || packed)) {        // its particles keep the packed cell
                    int o[3];
                    tile_origin(B, neighbor_tile(B, g, k), o);
                    hcell[h] = pack_cell(o[0] + (code & 3), o[1] + ((code >> 2) & 3), o[2] + (code >> 4));
                }
                const SpeciesDev<R> &S = B.sp[s];
                const int o = atomicAdd(&S.nb[dst][B.ntiles], 1);
                if (o >= S.ovf_cap) {
                    atomicOr(C.flags, PIC_FLAG_LOST);
                    at = -1;
                } else {
                    at = S.seg_start[dst][B.ntiles] + o;
                }
            }
            if (at >= 0) write_particle<FIX == 1>(sh_q[s], at, wide, hcell[h], code, hd[h], hu[h], hid[h]);
        }
    }
}

// FP32 form: four waves per SIMD (at most 128 VGPRs), the occupancy that
// hides the latency of the LDS gather and of the particle loads best on
// gfx950.  FP64 form: three (at most 168 VGPRs; with its 64-entry queues a
// 4x4x4 block's LDS allows three blocks per CU as well).
template <typename R, int FIX, int WALLS, int F4>
__global__ void __launch_bounds__(kBlock, PushWaves<R>::value) push_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                           const Item *__restrict__ items, StepConst<R> C)
{
    push_block<R, FIX, WALLS, F4, kBlock>(boxes, items, C);
}

// 4x4x4 tiles and a particle copy of 4 GiB or more (125 M particles of a species
// at the default headroom, 64 M in the FP64 form): 64-bit slot addresses.
// 128^3 cells, 64 pairs per cell: 3.86 ms; 4.14 with the kernel for tiles of any
// shape.  (32-bit addresses, where they reach: 64^3, 64 pairs 480 us, with these
// 483; FP64 866 and 873.)
template <typename R, int WALLS, int F4>
__global__ void __launch_bounds__(kBlock, PushWaves<R>::value) far_push_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                               const Item *__restrict__ items,
                                                                               StepConst<R> C)
{
    push_block<R, 2, WALLS, F4, kBlock>(boxes, items, C);
}

// Launches that leave CUs idle take more threads per tile (wide_threads): the
// time of such a launch is one tile's chain of set-up, iterations and hand-over,
// and a wave then makes fewer iterations.  Step time with 256 / 512 / 1024
// threads: 16^3 cells at 8 pairs per cell 23.0 / 20.5 / 19.2 us, at 256 221 / 156 /
// 146; 24^3 at 64 (216 tiles) 70.1 / 52.9 / 50.2; 32^3 at 64 (512 tiles) 87.8 / 82.2 / -;
// FP64 24^3 at 16 40.2 / 35.8 / 37.4.
template <typename R, int F4, int NT>
__global__ void __launch_bounds__(NT) wide_push_kernel(const BoxDev<R> *__restrict__ boxes,
                                                       const Item *__restrict__ items, StepConst<R> C)
{
    push_block<R, 1, 0, F4, NT>(boxes, items, C);
}

// ------------------------------------------------------------- Yee updates

// Between two pushes: copy `old` (just read, written by the next push) gets,
// for tile t, empty A and B ranges with B starting after the particles that
// the tile now holds in copy old ^ 1, and an empty overflow region.
template <typename R>
__device__ inline void next_layout(const BoxDev<R> &B, int nsp, int old, int t)
{
    for (int s = 0; s < nsp; ++s) {
        const SpeciesDev<R> &S = B.sp[s];
        if (t < B.ntiles) {
            S.bs[old][t] = tile_ranges(S, old ^ 1, t).n;
            S.na[old][t] = 0;
        }
        S.nb[old][t] = 0;
    }
}

// Overflow watch, by one whole block: fill of the fullest overflow region
// after a push, over every box and species of copy `copy` (the one just
// written), in thousandths of the smaller of its capacity and kOvfBlocks *
// 1024 particles (the load its sweep blocks take in four rounds).
template <typename R>
__device__ void overflow_watch_block(const BoxDev<R> *__restrict__ boxes, int nboxes, int nsp, int copy,
                                     const Watch &out)
{
    __shared__ unsigned int best;

    if (threadIdx.x == 0) best = 0;
    __syncthreads();
    unsigned int m = 0;
    for (int b = threadIdx.x; b < nboxes; b += kBlock) {
        const BoxDev<R> &B = boxes[b];
        for (int s = 0; s < nsp; ++s) {
            const SpeciesDev<R> &S = B.sp[s];
            const long long c = S.nb[copy][B.ntiles];
            const long long cap = min((long long)S.ovf_cap, (long long)kOvfBlocks * 1024);
            const unsigned int f = (unsigned int)min(1000LL, c * 1000LL / max(1LL, cap));
            m = max(m, f);
        }
    }
    atomicMax(&best, m);
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(out.slot, ((uint64_t)out.step << 32) | best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Book-keeping after a push, by the first field kernel that follows it: the
// tile descriptors of copy `old` (the one just read) for the next push, and
// in the grid's last block the overflow watch of copy old ^ 1 (the one just
// written); the whole last block reaches the watch's barriers.
template <typename R>
__device__ inline void after_push(const BoxDev<R> *__restrict__ boxes, const BoxDev<R> &B, int64_t p, int nsp,
                                  int old, int nboxes, Watch watch)
{
    if (p < B.ntiles) next_layout(B, nsp, old, (int)p);
    if (p == 0) next_layout(B, nsp, old, B.ntiles);
    if (watch.slot && blockIdx.x == gridDim.x - 1) overflow_watch_block(boxes, nboxes, nsp, old ^ 1, watch);
}

// Coordinates of cell p of a box with edges n0, n1 (p < n0 n1 n2 <= 2^32, so
// 32-bit divisions are exact).
__device__ inline void cell_coords(int64_t p, int n0, int n1, int &i, int &j, int &k)
{
    const uint32_t q = (uint32_t)p, r = q / (uint32_t)n0;
    i = (int)(q - r * (uint32_t)n0);
    k = (int)(r / (uint32_t)n1);
    j = (int)(r - (uint32_t)k * (uint32_t)n1);
}

// b <- b - h curl e (App. A.3.2), in place.  The steps advance b inside the
// push (its set-up writes b^{t+dt/2} of each tile's cells); this kernel makes
// the half step of the start (h = -dt/2).
template <typename R>
__global__ void __launch_bounds__(kBlock) advance_b_kernel(const BoxDev<R> *__restrict__ boxes,
                                                           const CellBlock *__restrict__ blocks, R h)
{
    const CellBlock cb = blocks[blockIdx.x];
    const BoxDev<R> &B = boxes[cb.box];
    const int64_t p = (int64_t)cb.first + threadIdx.x;
    if (p >= B.nc) return;
    const int n0 = B.n[0], n1 = B.n[1], n2 = B.n[2];
    int i, j, k;
    cell_coords(p, n0, n1, i, j, k);
    const int64_t sx = (i + 1 < n0) ? 1 : 1 - n0;
    const int64_t sy = (j + 1 < n1) ? n0 : (int64_t)n0 * (1 - n1);
    const int64_t sz = (k + 1 < n2) ? (int64_t)n0 * n1 : (int64_t)n0 * n1 * (1 - n2);
    const R *ex = B.e, *ey = B.e + B.nc, *ez = B.e + 2 * B.nc;
    R cx, cy, cz;
    if (B.faraday4) {
        cx = curl4_e(B, 0, i, j, k);
        cy = curl4_e(B, 1, i, j, k);
        cz = curl4_e(B, 2, i, j, k);
    } else {
        cx = (ez[p + sy] - ez[p]) - (ey[p + sz] - ey[p]);
        cy = (ex[p + sz] - ex[p]) - (ez[p + sx] - ez[p]);
        cz = (ey[p + sx] - ey[p]) - (ex[p + sy] - ex[p]);
    }
    B.b[p] -= h * cx;
    B.b[B.nc + p] -= h * cy;
    B.b[2 * B.nc + p] -= h * cz;
    if (B.wall >= 0 && (B.wall == 0 ? i : (B.wall == 1 ? j : k)) == 0)
        B.b[B.wall * B.nc + p] = R(0);           // normal b on a conducting wall (App. A.4)
}

// e <- e + dt curl b + alpha0 J (App. A.3.2 and A.2, eq. max2bis); J <- 0;
// and the book-keeping after the push (after_push).
template <typename R>
__global__ void __launch_bounds__(kBlock) advance_e_kernel(const BoxDev<R> *__restrict__ boxes,
                                                           const CellBlock *__restrict__ blocks, R dt, int nsp,
                                                           int old, int nboxes, Watch watch)
{
    using JT = typename JType<R>::T;
    const CellBlock cb = blocks[blockIdx.x];
    const BoxDev<R> &B = boxes[cb.box];
    const int64_t p = (int64_t)cb.first + threadIdx.x;
    after_push(boxes, B, p, nsp, old, nboxes, watch);
    if (p >= B.nc) return;
    const int n0 = B.n[0], n1 = B.n[1], n2 = B.n[2];
    int i, j, k;
    cell_coords(p, n0, n1, i, j, k);
    const int64_t sx = (i > 0) ? 1 : 1 - n0;
    const int64_t sy = (j > 0) ? n0 : (int64_t)n0 * (1 - n1);
    const int64_t sz = (k > 0) ? (int64_t)n0 * n1 : (int64_t)n0 * n1 * (1 - n2);
    const R *bx = B.b, *by = B.b + B.nc, *bz = B.b + 2 * B.nc;
    const R cx = (bz[p] - bz[p - sy]) - (by[p] - by[p - sz]);
    const R cy = (bx[p] - bx[p - sz]) - (bz[p] - bz[p - sx]);
    const R cz = (by[p] - by[p - sx]) - (bx[p] - bx[p - sy]);
    JT *J = B.J;
    const double a = B.alpha0 / (double)qscale_bits<R>();
    const R jx = (R)(a * (double)J[p]), jy = (R)(a * (double)J[B.nc + p]), jz = (R)(a * (double)J[2 * B.nc + p]);
    B.e[p] += dt * cx + jx;
    B.e[B.nc + p] += dt * cy + jy;
    B.e[2 * B.nc + p] += dt * cz + jz;
    if (B.wall >= 0 && (B.wall == 0 ? i : (B.wall == 1 ? j : k)) == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c)              // tangential e on a conducting wall (App. A.4)
            if (c != B.wall) B.e[c * B.nc + p] = R(0);
    }
    J[p] = JT(0);
    J[B.nc + p] = JT(0);
    J[2 * B.nc + p] = JT(0);
}

// Sum over the 27 values around cell (i,j,k) of one periodic grid with the
// smoothing weights of App. A.3.4 scaled to integers: 8 for the cell itself,
// 4 per face neighbour, 2 per edge neighbour, 1 per corner neighbour (the
// paper's 1, 1/2, 1/4, 1/8 times 8; they add up to 64).
template <typename T>
__device__ inline T smooth27(const PIC_GLOBAL T *f, const int n[3], int i, int j, int k)
{
    T acc = T(0);
#pragma unroll
    for (int dk = -1; dk <= 1; ++dk) {
        const int64_t kk = wrap1(k + dk, n[2]);
#pragma unroll
        for (int dj = -1; dj <= 1; ++dj) {
            const int64_t row = (int64_t)n[0] * (wrap1(j + dj, n[1]) + (int64_t)n[1] * kk);
#pragma unroll
            for (int di = -1; di <= 1; ++di) {
                const int w = 8 >> ((di != 0) + (dj != 0) + (dk != 0));
                acc += T(w) * f[row + wrap1(i + di, n[0])];
            }
        }
    }
    return acc;
}

// e <- e + dt curl b + alpha0 S J with S the 27-point smoothing of App. A.3.4
// (integer weights in the FP32 form, so the smoothed current stays exact and
// order-independent until its one conversion); J is cleared afterwards by
// clear_current_kernel, since every cell reads its neighbours' J here.
template <typename R>
__global__ void __launch_bounds__(kBlock) advance_e_smoothed_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                    const CellBlock *__restrict__ blocks, R dt,
                                                                    int nsp, int old, int nboxes,
                                                                    Watch watch)
{
    using JT = typename JType<R>::T;
    const CellBlock cb = blocks[blockIdx.x];
    const BoxDev<R> &B = boxes[cb.box];
    const int64_t p = (int64_t)cb.first + threadIdx.x;
    after_push(boxes, B, p, nsp, old, nboxes, watch);
    if (p >= B.nc) return;
    const int n0 = B.n[0], n1 = B.n[1], n2 = B.n[2];
    int i, j, k;
    cell_coords(p, n0, n1, i, j, k);
    const int64_t sx = (i > 0) ? 1 : 1 - n0;
    const int64_t sy = (j > 0) ? n0 : (int64_t)n0 * (1 - n1);
    const int64_t sz = (k > 0) ? (int64_t)n0 * n1 : (int64_t)n0 * n1 * (1 - n2);
    const R *bx = B.b, *by = B.b + B.nc, *bz = B.b + 2 * B.nc;
    const R cx = (bz[p] - bz[p - sy]) - (by[p] - by[p - sz]);
    const R cy = (bx[p] - bx[p - sz]) - (bz[p] - bz[p - sx]);
    const R cz = (by[p] - by[p - sx]) - (bx[p] - bx[p - sy]);
    const double a = B.alpha0 / (double)qscale_bits<R>() / 64.0;
    const R cur[3] = {cx, cy, cz};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const JT s = smooth27<JT>(B.J + c * B.nc, B.n, i, j, k);
        B.e[c * B.nc + p] += dt * cur[c] + (R)(a * (double)s);
    }
}

template <typename R>
__global__ void __launch_bounds__(kBlock) clear_current_kernel(const BoxDev<R> *__restrict__ boxes,
                                                               const CellBlock *__restrict__ blocks)
{
    using JT = typename JType<R>::T;
    const CellBlock cb = blocks[blockIdx.x];
    const BoxDev<R> &B = boxes[cb.box];
    const int64_t p = (int64_t)cb.first + threadIdx.x;
    if (p >= B.nc) return;
    B.J[p] = JT(0);
    B.J[B.nc + p] = JT(0);
    B.J[2 * B.nc + p] = JT(0);
}

// ------------------------------------------------------ counting-sort repack

// Tile counts for the repack: a tile's ranges hold only particles of that
// tile, so they count as a whole; overflow particles one by one.
template <typename R>
__global__ void __launch_bounds__(kBlock) repack_count_kernel(const BoxDev<R> *__restrict__ boxes,
                                                              const Item *__restrict__ items, int nsp, int cur)
{
    const Item it = items[blockIdx.x];
    const BoxDev<R> &B = boxes[it.box];
    for (int s = 0; s < nsp; ++s) {
        const SpeciesDev<R> &S = B.sp[s];
        int first, stride;
        const TileRanges r = item_range(B, S, cur, it.tile, first, stride);
        if (it.tile >= 0) {
            if (threadIdx.x == 0 && r.n > 0) atomicAdd(&S.tcount[it.tile], r.n);
        } else {
            for (int p = first; p < r.n; p += stride) atomicAdd(&S.tcount[tile_of(B, S.buf[cur].cell[r.slot(p)])], 1);
        }
    }
}

// Staged particles: counted in nb of the copy to be written (zero between
// steps), where the layout kernel finds them; a particle's place in its tile
// is kept in that copy's packed-cell array (no slot of it is in use yet) for
// the scatter, which then claims nothing.  One block per chunk of particles
// (stage_chunk) counts them per tile in LDS and claims each tile's places with
// one global atomic; boxes of more than kCountTiles tiles, where few particles
// of a chunk share a tile, take one global atomic per particle (33.5 M
// particles in 4096 tiles: 0.12 ms against 2.2).
template <typename R>
__global__ void __launch_bounds__(kStageBlock) repack_count_stage_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                         const StageItem *__restrict__ items, int dst)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int *cnt = reinterpret_cast<int *>(smem);
    const StageItem it = items[blockIdx.x];
    const BoxDev<R> &B = boxes[it.box];
    const SpeciesDev<R> &S = B.sp[it.species];
    PIC_GLOBAL int32_t *cell = S.stage.cell, *place = S.buf[dst].cell, *nb = S.nb[dst];
    const int nt = B.ntiles;
    if (nt > kCountTiles) {
        for (int p = it.first + threadIdx.x; p < it.last; p += kStageBlock)
            place[p] = atomicAdd(&nb[tile_of(B, cell[p])], 1);
        return;
    }
    for (int t = threadIdx.x; t < nt; t += kStageBlock) cnt[t] = 0;
    __syncthreads();
    for (int p = it.first + threadIdx.x; p < it.last; p += kStageBlock) atomicAdd(&cnt[tile_of(B, cell[p])], 1);
    __syncthreads();
    for (int t = threadIdx.x; t < nt; t += kStageBlock)
        if (cnt[t]) cnt[t] = atomicAdd(&nb[t], cnt[t]);
    __syncthreads();
    for (int p = it.first + threadIdx.x; p < it.last; p += kStageBlock)
        place[p] = atomicAdd(&cnt[tile_of(B, cell[p])], 1);
}

// One block per (box, species): new segment layout from the tile counts.
// Free slots: up to 32 for every tile, the rest shared in proportion to
// (count + 1).  (All in proportion, an empty tile got none and every particle
// that entered it took the overflow region's slow path: at the edges of a
// Harris sheet, 796 x 632 x 4 cells, 7300 of 15.7 M particles after 60 steps
// and a push of 0.99 ms against 0.53.)  The overflow region is the
// fixed tail of the arrays.
// The block takes as many neighbouring tiles as it has threads at a time, in
// order, and loads the next ones' counts while it adds up the capacities of
// these: 64000 tiles 69 us (350 with a run of tiles per thread, whose loads wait
// for one another, and 510 with one more count in them).  1024 threads, where
// boxes are small 256 (repack of 200 boxes of 8 tiles 44 and 46 us).
constexpr int kLayoutBlock = 1024;
template <typename R>
__global__ void __launch_bounds__(kLayoutBlock) repack_layout_kernel(const BoxDev<R> *__restrict__ boxes, int nsp,
                                                                     int dst, uint32_t *flags)
{
    constexpr int kW = kLayoutBlock / 64;
    __shared__ int part[2][kW];
    const int NT = blockDim.x;
    const int box = blockIdx.x / nsp, s = blockIdx.x % nsp;
    const BoxDev<R> &B = boxes[box];
    const SpeciesDev<R> &S = B.sp[s];
    PIC_GLOBAL int32_t *tcount = S.tcount, *nb = S.nb[dst], *na = S.na[dst], *bs = S.bs[dst];
    PIC_GLOBAL int32_t *seg_start = S.seg_start[dst], *seg_cap = S.seg_cap[dst];
    const int nt = B.ntiles, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // a tile's particles: binned ones in tcount, staged ones in nb; all of them
    // and the slots below are fewer than 2^31
    int mine = 0;
#pragma unroll 4
    for (int t = tid; t < nt; t += NT) mine += tcount[t] + nb[t];
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if (tid < 2 * kW) (&part[0][0])[tid] = 0;          // of waves that a small block has not
    __syncthreads();
    if (lane == 0) part[1][wave] = mine;
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int w = 0; w < kW; ++w) sum += part[1][w];
    const long long total = sum, region = (long long)S.slots - S.ovf_cap;
    if (total > region) {                              // uniform: the whole block leaves
        // the counts still start from zero at the next repack
        for (int t = tid; t < nt; t += NT) tcount[t] = nb[t] = 0;
        if (tid == 0) atomicOr((PIC_GLOBAL uint32_t *)flags, PIC_FLAG_LOST);
        return;
    }
    // the same slack for every tile first (up to the 32 slots per tile that
    // the arrays hold for it), the rest in proportion
    const long long slack = min(32LL, (region - total) / nt);
    const long long freeslots = region - total - slack * nt;
    const long long den = total + nt;
    int run = 0;
    int binned = tid < nt ? tcount[tid] : 0, staged = tid < nt ? nb[tid] : 0;
    int *sums = part[0];
    for (int first = 0; first < nt; first += NT) {
        const int t = first + tid, next = t + NT, here = staged;
        const long long c = binned + staged;
        if (next < nt) {
            binned = tcount[next];
            staged = nb[next];
        }
        const int cap = t < nt ? (int)(c + slack + (freeslots * (c + 1)) / den) : 0;
        int end = cap;                                 // of the capacities up to this tile's
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(end, off);
            if (lane >= off) end += v;
        }
        // (two sets of wave sums, so that one barrier per pass separates writing
        // a set from the reads of the pass before the last; the total used set 1)
        if (lane == 63) sums[wave] = end;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kW; ++w) {
            const int v = sums[w];
            before += w < wave ? v : 0;
            all += v;
        }
        if (t < nt) {
            seg_start[t] = run + before + end - cap;
            seg_cap[t] = cap;
            // the staged particles are the A range, the binned ones follow as B
            na[t] = bs[t] = here;
            nb[t] = 0;
            tcount[t] = 0;
        }
        run += all;
        sums = sums == part[0] ? part[1] : part[0];
    }
    if (tid == 0) {
        seg_start[nt] = S.slots - S.ovf_cap;
        seg_cap[nt] = S.ovf_cap;
        nb[nt] = 0;
    }
}

template <typename R>
__global__ void __launch_bounds__(kBlock) repack_scatter_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                const Item *__restrict__ items, int nsp, int cur,
                                                                uint32_t *flags)
{
    const Item it = items[blockIdx.x];
    const BoxDev<R> &B = boxes[it.box];
    int o[3] = {0, 0, 0};                               // origin of the tile (tile items)
    if (it.tile >= 0) tile_origin(B, it.tile, o);
    for (int s = 0; s < nsp; ++s) {
        const SpeciesDev<R> &S = B.sp[s];
        int first, stride;
        const TileRanges r = item_range(B, S, cur, it.tile, first, stride);
        const int n = r.n;
        const PBuf<R> &P = S.buf[cur];
        // wave-uniform trip count so that the ballots in store_particle see every lane
        const int trips = n > first - (int)threadIdx.x ? (n - (first - (int)threadIdx.x) + stride - 1) / stride : 0;
        for (int tr = 0; tr < trips; ++tr) {
            const int p = first + tr * stride;
            const bool valid = p < n;
            int32_t cell = 0, id = 0;
            R d[3] = {R(0), R(0), R(0)}, u[3] = {R(0), R(0), R(0)};
            if (valid) {
                const int idx = r.slot(p);
                const PSlot<R> ps = slot_at(P, idx);
                cell = it.tile >= 0 ? local_cell(B, o, ps.code()) : P.cell[idx];
                for (int a = 0; a < 3; ++a) { d[a] = ps.d(a); u[a] = ps.u(a); }
                if (P.id) id = P.id[idx];
            }
            store_particle(B, S, cur ^ 1, tile_of(B, cell), valid, cell, d, u, id, (PIC_GLOBAL uint32_t *)flags);
        }
    }
}

// `split` blocks per chunk, one particle per thread: the blocks that run
// together then write neighbouring places of the tiles (one block per chunk
// took 5.7 ms for 33.5 M particles, this 2.9: 4-byte stores scattered over
// every tile).
template <typename R>
__global__ void __launch_bounds__(kStageBlock) repack_scatter_stage_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                           const StageItem *__restrict__ items, int split,
                                                                           int dst)
{
    const StageItem it = items[blockIdx.x / split];
    const BoxDev<R> &B = boxes[it.box];
    const SpeciesDev<R> &S = B.sp[it.species];
    const int p = it.first + (int)(blockIdx.x % split) * kStageBlock + threadIdx.x;
    if (p >= it.last) return;
    const int32_t cell = S.stage.cell[p];
    const int t = tile_of(B, cell), rank = S.buf[dst].cell[p];
    if (rank >= S.seg_cap[dst][t]) return;               // only where the layout found no room (flagged there)
    R d[3], u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) { d[a] = S.stage.d[a][p]; u[a] = S.stage.u[a][p]; }
    write_particle(S.buf[dst], S.seg_start[dst][t] + rank, false, cell, local_code(B, cell), d, u,
                   S.stage.id ? S.stage.id[p] : 0);
}

// Backward half step (App. A.3.1): u^t -> u^{t-dt/2} in e^t, b^t, of the
// particles just binned from a load (the A ranges of copy C.cur ^ 1) of the
// species in the box's mask.  One block per tile, with the push's set-up and
// gather, so each node value is formed once per tile instead of 48 times per
// particle from HBM (33.5 M particles: 0.28 ms; gathered
// per particle in the scatter, 81 ms together with its slot claims).
template <typename R, int F4>
__global__ void __launch_bounds__(kBlock) half_step_kernel(const BoxDev<R> *__restrict__ boxes,
                                                           const Item *__restrict__ items,
                                                           const uint32_t *__restrict__ half, StepConst<R> C)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const Item it = items[blockIdx.x];
    if (it.tile < 0) return;
    const BoxDev<R> &B = boxes[it.box];
    const uint32_t mask = half[it.box];
    const int dst = C.cur ^ 1;
    bool any = false;
    for (int s = 0; s < C.nsp; ++s) any = any || ((mask >> s) & 1u && B.sp[s].na[dst][it.tile] > 0);
    if (!any) return;
    const TileGeom<R> g = tile_geom<R>(B, it.tile);
    const TileLds lds = tile_lds<R>(1 << B.tshift[0], 1 << B.tshift[1], 1 << B.tshift[2]);
    R *coef = reinterpret_cast<R *>(smem);
    R *re = reinterpret_cast<R *>(smem + lds.coef);
    R *node = reinterpret_cast<R *>(smem + lds.coef + lds.stage);
    tile_coefs<R, 0, 0, F4, false, kBlock>(B, g, TileGrid<R>(B, g), C.dt, coef, re, re + 3 * g.JN, node, []() { return true; });
    for (int s = 0; s < C.nsp; ++s) {
        if (!((mask >> s) & 1u)) continue;
        const SpeciesDev<R> &S = B.sp[s];
        const int n = S.na[dst][it.tile], start = S.seg_start[dst][it.tile];
        for (int p = threadIdx.x; p < n; p += kBlock) {
            const PSlot<R> ps = slot_at(S.buf[dst], start + p);
            const R d[3] = {ps.d(0), ps.d(1), ps.d(2)};
            R u[3] = {ps.u(0), ps.u(1), ps.u(2)}, E[3], Bf[3];
            const R *cf = coef + kCoef<R> * (int)ps.code();
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                E[c] = trilinear_eval(cf + 8 * c, d);
                Bf[c] = trilinear_eval(cf + 24 + 8 * c, d);
            }
            boris(R(-0.25) * C.kq[s] * C.dt, E, Bf, u);
#pragma unroll
            for (int a = 0; a < 3; ++a) ps.u(a) = u[a];
        }
    }
}

// After a repack into copy 1-old: clear the counters of copy `old` (all tiles
// and the overflow entry) and give it the new segment layout too.
template <typename R>
__global__ void __launch_bounds__(kBlock) clear_counts_kernel(const BoxDev<R> *__restrict__ boxes, int nboxes,
                                                              int nsp, int old)
{
    const int box = blockIdx.y;
    if (box >= nboxes) return;
    const BoxDev<R> &B = boxes[box];
    for (int t = blockIdx.x * kBlock + threadIdx.x; t <= B.ntiles; t += gridDim.x * kBlock)
        for (int s = 0; s < nsp; ++s) {
            const SpeciesDev<R> &S = B.sp[s];
            S.seg_start[old][t] = S.seg_start[old ^ 1][t];
            S.seg_cap[old][t] = S.seg_cap[old ^ 1][t];
            S.bs[old][t] = t < B.ntiles ? tile_ranges(S, old ^ 1, t).n : 0;
            S.na[old][t] = 0;
            S.nb[old][t] = 0;
        }
}

// -------------------------------------------------------------- diagnostics

__device__ inline double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    return v;
}

// Histogram bin of a particle with gamma - 1 = g: that of the FP64 logarithm.
// An FP32 logarithm decides it unless it falls within its error of an edge
// (relative error 2^-21 of the logarithm and of its operands, taken four
// times; every lane near an edge, beyond FP32's range, or with bins finer than
// that takes the FP64 one): a quarter of the kernel's FP64 work.
__device__ inline int gamma_bin(double g, double lo, double hi, int bins)
{
    const float l = 0.30102999566398120f * __builtin_amdgcn_logf((float)g), scale = (float)(bins / (hi - lo));
    const float x = (l - (float)lo) * scale, f = floorf(x);
    const float err = 2e-6f * (scale * (fabsf(l) + fabsf((float)lo) + 1.0f) + fabsf(x));
    int bin = (int)f;
    if (!(g > 1e-30 && g < 1e30 && x - f > err && f + 1.0f - x > err)) {
        const double v = log10(g > 1e-300 ? g : 1e-300);
        bin = (int)floor((v - lo) / (hi - lo) * bins);
    }
    return bin < 0 ? 0 : (bin >= bins ? bins - 1 : bin);
}

// Per-particle diagnostics of one box (items of that box only): gamma^t from
// u^- = u^{t-dt/2} + (k dt/2) E(x^t) (READING: the mover's own gamma^t), the
// k = 0 momentum, the gamma-1 histogram and the CIC charge density.  A block
// takes every gridDim.x-th item.  A tile item stages the node-averaged e of its
// (t+1)^3 nodes in LDS once and sums its charge there (one global atomic per
// node); the overflow items gather from HBM and add to the global charge
// directly.  The six sums per species and the histogram stay in LDS until the
// block ends: their global atomics all meet on a few addresses, where each
// takes about 8 ns.  One set per tile and species took 3.19 ms on a box of 31442
// tiles (15.7 M particles), this 0.35; 0.64 and 0.46 ms on one of 4096 (33.5 M),
// where the FP64 arithmetic and the LDS atomics of the charge bound it now.
constexpr int kDiagNodes = 9 * 9 * 9;   // nodes of the largest tile (8^3 cells)
constexpr int kDiagHist = 512;          // histograms up to this many bins are summed in LDS
constexpr int kDiagBlocks = 2048;       // at most, eight per CU
template <typename R>
__global__ void __launch_bounds__(kBlock) diag_particles_kernel(const BoxDev<R> *__restrict__ boxes,
                                                                const Item *__restrict__ items, int nitems,
                                                                StepConst<R> C, DiagBuf out)
{
    extern __shared__ unsigned shist[];             // [species][bins]
    __shared__ R sE[3 * kDiagNodes];
    __shared__ double srho[kDiagNodes];
    __shared__ double sacc[kBlock / 64][6 * kMaxSpecies];
    const R hdt = R(0.5) * C.dt;
    const int tid = threadIdx.x, wave = tid >> 6;
    const bool lhist = C.hist_bins > 0 && C.hist_bins <= kDiagHist;
    if (lhist)
        for (int q = tid; q < C.nsp * C.hist_bins; q += kBlock) shist[q] = 0u;
    if (tid < kBlock / 64 * 6 * kMaxSpecies) (&sacc[0][0])[tid] = 0.0;
    __syncthreads();
    for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
        const Item it = items[item];
        const BoxDev<R> &B = boxes[it.box];
        const bool in_tile = it.tile >= 0;
        TileGeom<R> g{};
        if (in_tile) {
            int n = 0;
            for (int s = 0; s < C.nsp; ++s) n += tile_ranges(B.sp[s], C.cur, it.tile).n;
            if (n == 0) continue;
            g = tile_geom<R>(B, it.tile);
            // node-averaged e (App. A.3.3)
            for (int q = tid; q < g.NN; q += kBlock) {
                const int i = g.o[0] + q % g.NX, j = g.o[1] + (q / g.NX) % g.NY, k = g.o[2] + q / (g.NX * g.NY);
                sE[q] = node_value_global(B, 0, i, j, k, R(0));
                sE[g.NN + q] = node_value_global(B, 1, i, j, k, R(0));
                sE[2 * g.NN + q] = node_value_global(B, 2, i, j, k, R(0));
                srho[q] = 0.0;
            }
            __syncthreads();
        }
        for (int s = 0; s < C.nsp; ++s) {
            const SpeciesDev<R> &S = B.sp[s];
            int first, stride;
            const TileRanges r = item_range(B, S, C.cur, it.tile, first, stride);
            const PBuf<R> P = S.buf[C.cur];
            const double q = (double)C.qs[s] * B.alpha0, hk = 0.5 * (double)C.kq[s] * (double)C.dt;
            double acc[6] = {0, 0, 0, 0, 0, 0};
            for (int p = first; p < r.n; p += stride) {
                const int idx = r.slot(p);
                const PSlot<R> ps = slot_at(P, idx);
                const int32_t cell = in_tile ? local_cell(B, g.o, ps.code()) : P.cell[idx];
                const int ix = cell_x(cell), iy = cell_y(cell), iz = cell_z(cell);
                const R d[3] = {ps.d(0), ps.d(1), ps.d(2)}, u[3] = {ps.u(0), ps.u(1), ps.u(2)};
                R E[3];
                int nb = 0;
                if (in_tile) {
                    // the cell's trilinear interpolant, as the push evaluates it
                    nb = (ix - g.o[0]) + g.NX * ((iy - g.o[1]) + g.NY * (iz - g.o[2]));
                    for (int c = 0; c < 3; ++c) {
                        const R *F = sE + c * g.NN + nb;
                        const int NX = g.NX, NXY = g.NX * g.NY;
                        const R f[8] = {F[0],   F[1],       F[NX],       F[1 + NX],
                                        F[NXY], F[1 + NXY], F[NX + NXY], F[1 + NX + NXY]};
                        R cf[8];
                        trilinear_coef(f, cf);
                        E[c] = trilinear_eval(cf, d);
                    }
                } else {
                    R Bf[3];
                    gather_global(B, ix, iy, iz, d, hdt, E, Bf);
                }
                double um[3];
                for (int a = 0; a < 3; ++a) um[a] = (double)u[a] + hk * (double)E[a];
                const double gm1 = sqrt(1.0 + um[0] * um[0] + um[1] * um[1] + um[2] * um[2]) - 1.0;
                acc[0] += (double)C.mass[s] * gm1;
                acc[1] += um[0]; acc[2] += um[1]; acc[3] += um[2];
                acc[4] += 1.0;
                acc[5] += gm1;
                if (C.hist_bins > 0) {
                    const int bin = s * C.hist_bins + gamma_bin(gm1, C.hist_lo, C.hist_hi, C.hist_bins);
                    if (lhist) atomicAdd(&shist[bin], 1u);
                    else atomicAdd(reinterpret_cast<unsigned long long *>(&out.hist[bin]), 1ull);
                }
                for (int kk = 0; kk < 2; ++kk)
                    for (int jj = 0; jj < 2; ++jj)
                        for (int ii = 0; ii < 2; ++ii) {
                            const double w = (ii ? (double)d[0] : 1.0 - (double)d[0]) *
                                             (jj ? (double)d[1] : 1.0 - (double)d[1]) *
                                             (kk ? (double)d[2] : 1.0 - (double)d[2]);
                            if (in_tile) {
                                atomicAdd(&srho[nb + ii + g.NX * (jj + g.NY * kk)], q * w);
                            } else {
                                const int i = wrap_idx(ix + ii, B.n[0]), j = wrap_idx(iy + jj, B.n[1]),
                                          k = wrap_idx(iz + kk, B.n[2]);
                                atomicAdd(&out.rho[i + (int64_t)B.n[0] * (j + (int64_t)B.n[1] * k)], q * w);
                            }
                        }
            }
            if (r.n > 0)
                for (int k = 0; k < 6; ++k) {
                    const double v = wave_sum(acc[k]);
                    if (__lane_id() == 0) sacc[wave][6 * s + k] += v;
                }
        }
        if (in_tile) {
            __syncthreads();
            for (int q = tid; q < g.NN; q += kBlock)
                if (srho[q] != 0.0) {
                    const int i = wrap_idx(g.o[0] + q % g.NX, B.n[0]), j = wrap_idx(g.o[1] + (q / g.NX) % g.NY, B.n[1]),
                              k = wrap_idx(g.o[2] + q / (g.NX * g.NY), B.n[2]);
                    atomicAdd(&out.rho[i + (int64_t)B.n[0] * (j + (int64_t)B.n[1] * k)], srho[q]);
                }
            __syncthreads();                            // before the next tile's nodes
        }
    }
    __syncthreads();
    if (tid < 6 * C.nsp) {
        double t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t += sacc[w][tid];
        if (t != 0.0) atomicAdd(out.copy(blockIdx.x) + kAccSp + tid, t);
    }
    if (lhist)
        for (int q = tid; q < C.nsp * C.hist_bins; q += kBlock)
            if (shist[q])
                atomicAdd(reinterpret_cast<unsigned long long *>(&out.hist[q]), (unsigned long long)shist[q]);
}

// Largest of values that are not negative, by their bits: NaN is above infinity
// and stays.
__device__ inline double max_pos(double a, double b)
{
    return __longlong_as_double(max(__double_as_longlong(a), __double_as_longlong(b)));
}
__device__ inline void atomic_max_pos(double *p, double v)
{
    atomicMax(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__double_as_longlong(v));
}

// Field energies (e^t, b^t) and the Gauss-law residual div e - rho at the nodes.
// The largest residual passes over a node where it is NaN (the sum of squares,
// NaN then, tells), but is NaN itself where all 64 nodes of a wave are: a field
// that is NaN throughout does not look like one that obeys Gauss's law.
// A few blocks stride over the cells, so that the sums' atomics stay few (one
// block per 256 cells: 0.14 ms on 64^3 cells and 1.03 ms on 796 x 632 x 4).
constexpr int kDiagFieldBlocks = 1024;
template <typename R>
__global__ void __launch_bounds__(kBlock) diag_fields_kernel(const BoxDev<R> *__restrict__ boxes, int box,
                                                             R dt, int filter, DiagBuf out)
{
    __shared__ double red[kBlock / 64][8];
    const BoxDev<R> &B = boxes[box];
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};             // [6]: the largest residual, [7]: the sum of squares
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < B.nc; p += (int64_t)gridDim.x * kBlock) {
        const int n0 = B.n[0], n1 = B.n[1];
        int i, j, k;
        cell_coords(p, n0, n1, i, j, k);
        for (int c = 0; c < 3; ++c) {
            const double ec = (double)B.e[c * B.nc + p];
            const double bc = (double)bt_global(B, c, i, j, k, R(0.5) * dt);
            v[c] += 0.5 * ec * ec;
            v[3 + c] += 0.5 * bc * bc;
        }
        const double div = (double)fld(B.e, B, 0, i, j, k) - (double)fld(B.e, B, 0, i - 1, j, k) +
                           (double)fld(B.e, B, 1, i, j, k) - (double)fld(B.e, B, 1, i, j - 1, k) +
                           (double)fld(B.e, B, 2, i, j, k) - (double)fld(B.e, B, 2, i, j, k - 1);
        // with a smoothed current the conserved charge is the smoothed one
        const double rho = filter ? smooth27<double>(out.rho, B.n, i, j, k) / 64.0 : out.rho[p];
        const bool on_wall = B.wall >= 0 && (B.wall == 0 ? i : (B.wall == 1 ? j : k)) == 0;
        const double r = on_wall ? 0.0 : div - rho;   // a wall plane carries the conductor's surface charge
        v[7] += r * r;
        const bool nan = r != r, keep = __ballot(nan) == ~0ull;
        v[6] = max_pos(v[6], nan && !keep ? 0.0 : fabs(r));
    }
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        double t = v[q];
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_down(t, off);
            t = q == 6 ? max_pos(t, o) : t + o;
        }
        if (__lane_id() == 0) red[wave][q] = t;
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        const int q = threadIdx.x;
        double t = red[0][q];
        for (int w = 1; w < kBlock / 64; ++w) t = q == 6 ? max_pos(t, red[w][q]) : t + red[w][q];
        double *dst = (double *)(out.copy(blockIdx.x) + kAccField + q);
        if (q == 6) atomic_max_pos(dst, t);
        else atomicAdd(dst, t);
    }
}

// The last diagnostics kernel: the copies of the accumulators added up, and
// the overflow counts and the error flag word put behind them (over the charge
// density, which is no longer needed), so that one copy brings all to the host.
template <typename R>
__global__ void __launch_bounds__(64) diag_collect_kernel(const BoxDev<R> *__restrict__ boxes, int box, StepConst<R> C,
                                                          DiagBuf out)
{
    const BoxDev<R> &B = boxes[box];
    const int q = threadIdx.x;
    if (q < kAccLen) {
        double t = out.acc[q];
        for (int r = 1; r < out.copies; ++r) t = q == kAccField + 6 ? max_pos(t, out.copy(r)[q]) : t + out.copy(r)[q];
        out.acc[q] = t;
    }
    if (q < kMaxSpecies) out.rho[q] = q < C.nsp ? (double)B.sp[q].nb[C.cur][B.ntiles] : 0.0;
    if (q == kMaxSpecies) out.rho[q] = (double)*C.flags;
}

// ----------------------------------------------------------- host launchers

template <typename R>
size_t push_lds_bytes(int t0, int t1, int t2) { return tile_lds<R>(t0, t1, t2).total(); }
template <typename R>
size_t wide_lds_bytes(int threads) { return tile_lds<R>(4, 4, 4, threads / 64).total(); }

template <typename R>
hipError_t launch_push(const BoxDev<R> *boxes, const Item *items, int nitems, size_t lds, const StepConst<R> &C,
                       int fix, int walls, int faraday4, int wide, hipStream_t st)
{
    // dynamic LDS beyond 64 KiB has to be allowed per kernel; where a launch
    // needs it the limit goes to the largest at once, so that no thread lowers it
    // for another
    static size_t raised[13] = {65536, 65536, 65536, 65536, 65536, 65536, 65536, 65536, 65536, 65536, 65536, 65536, 65536};
    auto go = [&](auto kern, int v, int threads = kBlock) -> hipError_t {
        if (lds > raised[v]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
            if (e != hipSuccess) return e;
            raised[v] = kMaxLds;
        }
        hipLaunchKernelGGL(kern, dim3(nitems), dim3(threads), lds, st, boxes, items, C);
        return hipGetLastError();
    };
    if constexpr (sizeof(R) == 4) {
        if (wide == 1024) return faraday4 ? go(wide_push_kernel<R, 1, 1024>, 9, 1024) : go(wide_push_kernel<R, 0, 1024>, 8, 1024);
    }
    if (wide) return faraday4 ? go(wide_push_kernel<R, 1, 512>, 7, 512) : go(wide_push_kernel<R, 0, 512>, 6, 512);
    // walls and the fourth-order solver are never combined (pic_plan refuses it)
    if (fix == 2) {
        if (walls) return go(far_push_kernel<R, 1, 0>, 11);
        return faraday4 ? go(far_push_kernel<R, 0, 1>, 12) : go(far_push_kernel<R, 0, 0>, 10);
    }
    if (walls) return fix ? go(push_kernel<R, 1, 1, 0>, 3) : go(push_kernel<R, 0, 1, 0>, 2);
    if (faraday4) return fix ? go(push_kernel<R, 1, 0, 1>, 5) : go(push_kernel<R, 0, 0, 1>, 4);
    return fix ? go(push_kernel<R, 1, 0, 0>, 1) : go(push_kernel<R, 0, 0, 0>, 0);
}

template <typename R>
hipError_t launch_fields(const BoxDev<R> *boxes, const CellBlock *blocks, int nblocks, R dt, int nsp, int filter,
                         int clear_copy, int nboxes, Watch watch, hipStream_t st)
{
    if (filter) {
        hipLaunchKernelGGL(advance_e_smoothed_kernel<R>, dim3(nblocks), dim3(kBlock), 0, st, boxes, blocks, dt, nsp,
                           clear_copy, nboxes, watch);
        hipLaunchKernelGGL(clear_current_kernel<R>, dim3(nblocks), dim3(kBlock), 0, st, boxes, blocks);
    } else {
        hipLaunchKernelGGL(advance_e_kernel<R>, dim3(nblocks), dim3(kBlock), 0, st, boxes, blocks, dt, nsp,
                           clear_copy, nboxes, watch);
    }
    return hipGetLastError();
}

template <typename R>
hipError_t launch_advance_b(const BoxDev<R> *boxes, const CellBlock *blocks, int nblocks, R h, hipStream_t st)
{
    hipLaunchKernelGGL(advance_b_kernel<R>, dim3(nblocks), dim3(kBlock), 0, st, boxes, blocks, h);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_repack(const BoxDev<R> *boxes, int nboxes, const Item *items, int nitems,
                         const StageItem *sitems, int nsitems, int split, const uint32_t *half, size_t lds, int faraday4,
                         const StepConst<R> &C, hipStream_t st)
{
    const int dst = C.cur ^ 1;
    if (nsitems)
        hipLaunchKernelGGL(repack_count_stage_kernel<R>, dim3(nsitems), dim3(kStageBlock), kCountTiles * sizeof(int), st,
                           boxes, sitems, dst);
    if (nitems) hipLaunchKernelGGL(repack_count_kernel<R>, dim3(nitems), dim3(kBlock), 0, st, boxes, items, C.nsp, C.cur);
    const int lthreads = nitems > (256 + kOvfBlocks) * nboxes ? kLayoutBlock : 256;   // by the boxes' mean
    hipLaunchKernelGGL(repack_layout_kernel<R>, dim3(nboxes * C.nsp), dim3(lthreads), 0, st, boxes, C.nsp, dst, C.flags);
    if (nsitems)
        hipLaunchKernelGGL(repack_scatter_stage_kernel<R>, dim3(nsitems * split), dim3(kStageBlock), 0, st, boxes, sitems,
                           split, dst);
    if (half) {
        // before the binned particles follow the staged ones into the tiles
        auto go = [&](auto kern) -> hipError_t {
            // the same limit in every call, so that contexts of different tile
            // shapes in several threads do not lower it for each other
            if (lds > 65536) {
                const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
                if (e != hipSuccess) return e;
            }
            hipLaunchKernelGGL(kern, dim3(nitems), dim3(kBlock), lds, st, boxes, items, half, C);
            return hipGetLastError();
        };
        const hipError_t e = faraday4 ? go(half_step_kernel<R, 1>) : go(half_step_kernel<R, 0>);
        if (e != hipSuccess) return e;
    }
    if (nitems) hipLaunchKernelGGL(repack_scatter_kernel<R>, dim3(nitems), dim3(kBlock), 0, st, boxes, items, C.nsp, C.cur,
                                   C.flags);
    hipLaunchKernelGGL(clear_counts_kernel<R>, dim3(64, nboxes), dim3(kBlock), 0, st, boxes, nboxes, C.nsp, C.cur);
    return hipGetLastError();
}

// zero n 8-byte words (a kernel rather than a memset, so that a caller may
// capture the diagnostics into a graph)
// (a plain pointer parameter: an address-space qualifier on a kernel
// parameter would give the device symbol another name than the host's)
__global__ void __launch_bounds__(kBlock) zero_words_kernel(uint64_t *__restrict__ p, int64_t n)
{
    PIC_GLOBAL uint64_t *q = (PIC_GLOBAL uint64_t *)p;
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < n; t += (int64_t)gridDim.x * kBlock) q[t] = 0;
}

hipError_t launch_zero(void *p, int64_t words, hipStream_t st)
{
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)std::min<int64_t>(1024, (words + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, st, (uint64_t *)p, words);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_diag(const BoxDev<R> *boxes, int box, int64_t nc, const Item *items, int nitems,
                       const StepConst<R> &C, const DiagBuf &out, int hist_len, hipStream_t st)
{
    // the accumulators, the charge density and the histogram start from zero
    // (they follow each other in memory)
    PIC_GLOBAL double *first = out.copy(out.copies - 1);
    const int64_t words = (PIC_GLOBAL double *)out.hist + hist_len - first;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)std::min<int64_t>(1024, (words + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, st, (uint64_t *)first, words);
    const size_t lhist = C.hist_bins <= kDiagHist ? (size_t)C.nsp * C.hist_bins * sizeof(unsigned) : 0;
    if (nitems)
        hipLaunchKernelGGL(diag_particles_kernel<R>, dim3(std::min(nitems, kDiagBlocks)), dim3(kBlock), lhist, st, boxes,
                           items, nitems, C, out);
    const int nb = (int)std::min<int64_t>(kDiagFieldBlocks, (nc + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(diag_fields_kernel<R>, dim3(nb), dim3(kBlock), 0, st, boxes, box, C.dt, C.filter, out);
    hipLaunchKernelGGL(diag_collect_kernel<R>, dim3(1), dim3(64), 0, st, boxes, box, C, out);
    return hipGetLastError();
}

// The diagnostics' own scratch for callers that cannot allocate device
// memory: one array per GPU, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in for
// the symbol); it uses the device address that hipGetSymbolAddress returns,
// taken once per device with that device current.
static __device__ __align__(256) unsigned char scratch[kDiagScratchBytes];

constexpr int kMaxDevices = 64;
static void *scratch_ptr[kMaxDevices];

hipError_t diag_scratch_setup()
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (scratch_ptr[dev]) return hipSuccess;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_ptr[dev] = p;
    return hipSuccess;
}

void *diag_scratch()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return scratch_ptr[dev];
}

// ------------------------------------------------- field Fourier spectra

// Value of field f (0: e^t, 1: b^t = b^{t-dt/2} - (dt/2) curl e^t), component
// c, at grid point (x[0], x[1], x[2]).
template <typename R>
__device__ inline double field_at(const BoxDev<R> &B, int f, int c, const int x[3], R hdt)
{
    if (f == 0) return (double)B.e[c * B.nc + x[0] + (int64_t)B.n[0] * (x[1] + (int64_t)B.n[1] * x[2])];
    return (double)bt_global(B, c, x[0], x[1], x[2], hdt);
}

// Plane spectra (Sect. 3.2.2): the two DFTs are matrix products of the field
// with a table of twiddle factors, in FP64 on the matrix cores
// (v_mfma_f64_16x16x4: lane l holds A[l & 15][l >> 4], B[l >> 4][l & 15] and
// D[(l >> 4) + 4 r][l & 15], r = 0..3).  The field is real, so only
// m1 <= N1 / 2 is formed; the rest follows from PS(-m1, -m2) = PS(m1, m2).
// Scratch: the field, [plane][i2][i1], in the box's charge array, where the
// result goes at the end; tmp, [plane][i2][m1] complex, and behind it the
// partial powers in the current's array (3 nc words; the two take at most
// 3 N2 NP (N1 / 2 + 1)), which the last kernel clears again.
// (One thread per output that formed b^t anew for every term of its sum took
// 5.9 + 1.0 ms for 796 x 632 cells and 4 planes, these four kernels 0.31.)
typedef double Mfma4 __attribute__((ext_vector_type(4)));
__device__ inline Mfma4 mfma16(double a, double b, Mfma4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// exp(-2 pi i q / n) for every q < n, in LDS
__device__ inline void twiddle_table(double2 *w, int n)
{
    for (int q = threadIdx.x; q < n; q += kBlock) {
        double sn, cs;
        sincospi(-2.0 * q / n, &sn, &cs);
        w[q] = make_double2(cs, sn);
    }
    __syncthreads();
}

template <typename R>
__global__ void __launch_bounds__(kBlock) spectrum_field_kernel(const BoxDev<R> *__restrict__ boxes, int box, int f,
                                                                int c, int a1, int a2, int an, R hdt,
                                                                double *__restrict__ out)
{
    const BoxDev<R> &B = boxes[box];
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= B.nc) return;
    int x[3];
    cell_coords(p, B.n[0], B.n[1], x[0], x[1], x[2]);
    const int i1 = a1 == 0 ? x[0] : x[1], i2 = a2 == 1 ? x[1] : x[2], ip = an == 0 ? x[0] : (an == 1 ? x[1] : x[2]);
    const int N1 = a1 == 0 ? B.n[0] : B.n[1], N2 = a2 == 1 ? B.n[1] : B.n[2];
    out[i1 + (int64_t)N1 * (i2 + (int64_t)N2 * ip)] = field_at(B, f, c, x, hdt);
}

// tmp[r][m1] = sum_i f[r][i] exp(-2 pi i m1 i / N1) over the rows r of all
// planes: a block takes 128 rows (32 per wave, so that each twiddle factor read
// feeds two products) and 16 modes; value(r, i) is f[r][i].
template <typename Value>
__device__ inline void spectrum_rows(int64_t rows, int N1, int nm, double2 *__restrict__ tmp, Value &&value)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *w = reinterpret_cast<double2 *>(smem);
    twiddle_table(w, N1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lo = lane & 15, hi = lane >> 4;
    const int64_t r0 = ((int64_t)blockIdx.x * (kBlock / 64) + wave) * 32;
    const int m0 = blockIdx.y * 16, m = min(m0 + lo, N1 - 1);
    const int64_t ra = min(r0 + lo, rows - 1), rb = min(r0 + 16 + lo, rows - 1);
    Mfma4 re[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}}, im[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    const int step = (int)((int64_t)4 * m % N1);
    int k = (int)((int64_t)hi * m % N1);                    // (m i) mod N1
    auto add = [&](double va, double vb) {
        const double2 t = w[k];
        re[0] = mfma16(va, t.x, re[0]);
        im[0] = mfma16(va, t.y, im[0]);
        re[1] = mfma16(vb, t.x, re[1]);
        im[1] = mfma16(vb, t.y, im[1]);
        k += step;
        if (k >= N1) k -= N1;
    };
    int i = hi;
#pragma unroll 4
    for (; i - hi + 4 <= N1; i += 4) add(value(ra, i), value(rb, i));
    if (N1 & 3) add(i < N1 ? value(ra, i) : 0.0, i < N1 ? value(rb, i) : 0.0);
    if (m0 + lo >= nm) return;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = r0 + 16 * h + hi + 4 * q;
            if (r < rows) tmp[r * nm + m0 + lo] = make_double2(re[h][q], im[h][q]);
        }
}

__global__ void __launch_bounds__(kBlock) spectrum_rows_kernel(const double *__restrict__ f, int64_t rows, int N1, int nm,
                                                               double2 *__restrict__ tmp)
{
    spectrum_rows(rows, N1, nm, tmp, [&](int64_t r, int i) { return f[r * N1 + i]; });
}

// The same straight from the grid, without a pass that writes the field first,
// for short rows: up to kShortRow[f] values, where that is faster.  One block
// column takes all modes, so each value is read once, but b^t takes five reads
// with wrapped indices that only the loads in flight of one row cover (rows of
// 31: e 8.0 us against 3.4 + 5.8, b 17.6 against 4.1 + 5.7; of 4: b 3.8 against
// 2.3 + 4.0).
constexpr int kShortRow[2] = {31, 8};
template <typename R>
__global__ void __launch_bounds__(kBlock) spectrum_rows_small_kernel(const BoxDev<R> *__restrict__ boxes, int box, int f,
                                                                     int c, int a1, int a2, int an, R hdt, int64_t rows,
                                                                     int nm, double2 *__restrict__ tmp)
{
    const BoxDev<R> &B = boxes[box];
    const int N1 = a1 == 0 ? B.n[0] : B.n[1], N2 = a2 == 1 ? B.n[1] : B.n[2];
    spectrum_rows(rows, N1, nm, tmp, [&](int64_t r, int i) {
        const int p = (int)((uint32_t)r / (uint32_t)N2), i2 = (int)((uint32_t)r - (uint32_t)p * (uint32_t)N2);
        const int x[3] = {a1 == 0 ? i : p, a1 == 1 ? i : (a2 == 1 ? i2 : p), a2 == 2 ? i2 : p};
        return field_at(B, f, c, x, hdt);
    });
}

// part[chunk][m2][m1] = sum over the planes of the chunk of
// |sum_i tmp[p][i][m1] exp(-2 pi i m2 i / N2)|^2: a wave takes 16 x 16 modes
// of one chunk of planes (blockIdx.y; few modes leave the chip idle otherwise).
// SPLIT: the four waves of a block take a quarter of the sum over i each, where
// there are so few tiles of modes that a wave's chain of products is the time
// (1 x 1 x 256 cells 8 us, without 22).
template <bool SPLIT>
__global__ void __launch_bounds__(kBlock) spectrum_cols_kernel(const double2 *__restrict__ tmp, int N2, int NP, int nm,
                                                               int per, double *__restrict__ part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double2 *w = reinterpret_cast<double2 *>(smem);
    twiddle_table(w, N2);
    constexpr int kW = kBlock / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lo = lane & 15, hi = lane >> 4;
    const int tm = (nm + 15) / 16, tile = SPLIT ? blockIdx.x : blockIdx.x * kW + wave;
    if (tile >= tm * ((N2 + 15) / 16)) return;
    const int m1 = tile % tm * 16 + lo, a0 = tile / tm * 16, m2 = min(a0 + lo, N2 - 1), mc = min(m1, nm - 1);
    // groups of four i: all, or this wave's quarter
    const int groups = (N2 + 3) / 4, g0 = SPLIT ? groups * wave / kW : 0, g1 = SPLIT ? groups * (wave + 1) / kW : groups;
    const int step = (int)((int64_t)4 * m2 % N2), k0 = (int)((int64_t)(4 * g0 + hi) * m2 % N2);
    double2 *sum = w + N2;                                  // SPLIT: [wave][q][lane], after the twiddle factors
    double pw[4] = {0.0, 0.0, 0.0, 0.0};
    const int p1 = min(NP, (int)(blockIdx.y + 1) * per);
    for (int p = blockIdx.y * per; p < p1; ++p) {
        const double2 *src = tmp + (int64_t)p * N2 * nm + mc;
        Mfma4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
        int k = k0;
        auto add = [&](double2 v) {
            const double2 t = w[k];
            re = mfma16(t.x, v.x, re);
            im = mfma16(t.x, v.y, im);
            re = mfma16(-t.y, v.y, re);
            im = mfma16(t.y, v.x, im);
            k += step;
            if (k >= N2) k -= N2;
        };
        int i = 4 * g0 + hi;
        const int full = min(4 * g1, N2 & ~3);
#pragma unroll 4
        for (; i - hi < full; i += 4) add(src[(int64_t)i * nm]);
        if (i - hi < 4 * g1) add(i < N2 ? src[(int64_t)i * nm] : make_double2(0.0, 0.0));
        if (SPLIT) {
            // wave q adds up the quarters of the rows hi + 4 q
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[(wave * 4 + q) * 64 + lane] = make_double2(re[q], im[q]);
            __syncthreads();
            double x = 0.0, y = 0.0;
#pragma unroll
            for (int v = 0; v < kW; ++v) {
                const double2 z = sum[(v * 4 + wave) * 64 + lane];
                x += z.x;
                y += z.y;
            }
            pw[0] += x * x + y * y;
            __syncthreads();
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) pw[q] += re[q] * re[q] + im[q] * im[q];
        }
    }
    if (m1 >= nm) return;
#pragma unroll
    for (int q = 0; q < (SPLIT ? 1 : 4); ++q) {
        const int r = a0 + hi + 4 * (SPLIT ? wave : q);
        if (r < N2) part[((int64_t)blockIdx.y * N2 + r) * nm + m1] = pw[q];
    }
}
static_assert(kBlock / 64 == 4, "a wave of a split block takes the rows of one register of the product");

// ps[m1 + N1 m2]: the chunks added in order, the modes above N1 / 2 by symmetry;
// every word of the scratch is cleared, a partial power by the one thread that
// reads it.
__global__ void __launch_bounds__(kBlock) spectrum_sum_kernel(double2 *__restrict__ tmp, int64_t ntmp,
                                                              double *__restrict__ part, int N1, int N2, int nm, int chunks,
                                                              double *__restrict__ ps)
{
    const int64_t first = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
    const int64_t modes = (int64_t)N2 * nm;
    for (int64_t t = first; t < modes; t += stride) {
        const int m1 = (int)(t % nm), m2 = (int)(t / nm);
        double v = 0.0;
#pragma unroll 8
        for (int c = 0; c < chunks; ++c) v += part[c * modes + t];
        for (int c = 0; c < chunks; ++c) part[c * modes + t] = 0.0;
        ps[m1 + (int64_t)N1 * m2] = v;
        if (m1 > 0 && N1 - m1 >= nm) ps[N1 - m1 + (int64_t)N1 * (m2 ? N2 - m2 : 0)] = v;
    }
    for (int64_t t = first; t < ntmp; t += stride) tmp[t] = make_double2(0.0, 0.0);
}

template <typename R>
hipError_t launch_spectrum(const BoxDev<R> *boxes, int box, const int n[3], int f, int c, int an, R hdt,
                           double *scratch, double *ps, hipStream_t st)
{
    const int a1 = an == 0 ? 1 : 0, a2 = an == 2 ? 1 : 2;
    const int N1 = n[a1], N2 = n[a2], NP = n[an], nm = N1 / 2 + 1;
    const int64_t nc = (int64_t)N1 * N2 * NP, rows = (int64_t)N2 * NP;
    double *field = ps;
    double2 *tmp = reinterpret_cast<double2 *>(scratch);
    const auto blocks = [](int64_t work) { return dim3((unsigned)((work + kBlock - 1) / kBlock)); };
    const dim3 rgrid((unsigned)((rows + 127) / 128), (nm + 15) / 16);
    if (N1 <= kShortRow[f]) {
        hipLaunchKernelGGL(spectrum_rows_small_kernel<R>, rgrid, dim3(kBlock), N1 * sizeof(double2), st, boxes, box, f, c, a1,
                           a2, an, hdt, rows, nm, tmp);
    } else {
        hipLaunchKernelGGL(spectrum_field_kernel<R>, blocks(nc), dim3(kBlock), 0, st, boxes, box, f, c, a1, a2, an, hdt,
                           field);
        hipLaunchKernelGGL(spectrum_rows_kernel, rgrid, dim3(kBlock), N1 * sizeof(double2), st, (const double *)field, rows,
                           N1, nm, tmp);
    }
    // the planes in chunks, so that about 2048 waves run
    const int tiles = (nm + 15) / 16 * ((N2 + 15) / 16);
    const int chunks0 = std::min(NP, std::max(1, 2048 / tiles)), per = (NP + chunks0 - 1) / chunks0;
    const int chunks = (NP + per - 1) / per;
    double *part = scratch + 2 * rows * nm;
    // split blocks where there is less than a wave per SIMD otherwise and the
    // quarters are longer than the adding up (four products)
    if ((int64_t)tiles * chunks <= 1024 && N2 >= 64)
        hipLaunchKernelGGL(spectrum_cols_kernel<true>, dim3(tiles, chunks), dim3(kBlock),
                           (N2 + 4 * kBlock) * sizeof(double2), st, (const double2 *)tmp, N2, NP, nm, per, part);
    else
        hipLaunchKernelGGL(spectrum_cols_kernel<false>, dim3((tiles + kBlock / 64 - 1) / (kBlock / 64), chunks), dim3(kBlock),
                           N2 * sizeof(double2), st, (const double2 *)tmp, N2, NP, nm, per, part);
    // the scratch is the current of the box, which the next push expects cleared
    const int64_t work = std::max(rows * nm, (int64_t)N2 * nm);
    hipLaunchKernelGGL(spectrum_sum_kernel, blocks(std::min<int64_t>(work, 1024 * kBlock)), dim3(kBlock), 0, st, tmp, rows * nm,
                       part, N1, N2, nm, chunks, ps);
    return hipGetLastError();
}

#define PIC_INSTANTIATE(R)                                                                                     \
    template size_t push_lds_bytes<R>(int, int, int);                                                         \
    template hipError_t launch_push<R>(const BoxDev<R> *, const Item *, int, size_t, const StepConst<R> &,   \
                                       int, int, int, int, hipStream_t);                                      \
    template size_t wide_lds_bytes<R>(int);                                                                    \
    template hipError_t launch_fields<R>(const BoxDev<R> *, const CellBlock *, int, R, int, int, int, int,     \
                                         Watch, hipStream_t);                                                        \
    template hipError_t launch_advance_b<R>(const BoxDev<R> *, const CellBlock *, int, R, hipStream_t);       \
    template hipError_t launch_repack<R>(const BoxDev<R> *, int, const Item *, int, const StageItem *, int,    \
                                         int, const uint32_t *, size_t, int, const StepConst<R> &, hipStream_t); \
    template hipError_t launch_diag<R>(const BoxDev<R> *, int, int64_t, const Item *, int,                    \
                                       const StepConst<R> &, const DiagBuf &, int, hipStream_t);              \
    template hipError_t launch_spectrum<R>(const BoxDev<R> *, int, const int[3], int, int, int, R, double *,   \
                                           double *, hipStream_t);

PIC_INSTANTIATE(float)
PIC_INSTANTIATE(double)

} // namespace pic
