// gfx950 kernels behind the host copies of pic.h: particles are converted to and
// from the caller's FP64 layout and put in order, and fields converted from it,
// on the GPU, so that a copy carries exactly what the caller's arrays hold and
// the host touches every value once.
#include <hip/hip_runtime.h>

#include "pic_internal.h"

namespace pic {

// ------------------------------------------------------------------ fields

// A field of a box with walls from FP64: on the wall plane (index 0 along the
// wall axis) the components that the conductor forbids become zero, tangential e
// and normal b (App. A.4).
template <typename R>
__global__ void __launch_bounds__(kBlock) fields_in_kernel(const double *__restrict__ src, int n0, int n1, int64_t nc,
                                                           int wall, int is_b, R *__restrict__ dst)
{
    for (int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x; q < 3 * nc; q += (int64_t)gridDim.x * kBlock) {
        const int c = (int)(q / nc);
        const uint32_t p = (uint32_t)(q - c * nc), r = p / (uint32_t)n0;   // nc <= 2^32
        const uint32_t i = wall == 0 ? p - r * (uint32_t)n0 : (wall == 1 ? r % (uint32_t)n1 : r / (uint32_t)n1);
        dst[q] = i == 0 && (is_b ? c == wall : c != wall) ? R(0) : (R)src[q];
    }
}

static unsigned grid_for(int64_t n) { return (unsigned)(n < (int64_t)2048 * kBlock ? (n + kBlock - 1) / kBlock : 2048); }

template <typename R>
hipError_t launch_fields_in(const double *src, const int n[3], int wall, int is_b, R *dst, hipStream_t st)
{
    const int64_t nc = (int64_t)n[0] * n[1] * n[2];
    hipLaunchKernelGGL(fields_in_kernel<R>, dim3(grid_for(3 * nc)), dim3(kBlock), 0, st, src, n[0], n[1], nc, wall, is_b,
                       dst);
    return hipGetLastError();
}

// --------------------------------------------------------------- particles

// First output place of every tile (in tile order) into tcount[0..ntiles], that
// of the overflow region last; info[0]: the particles of the species; info[1]
// is cleared (bad ids).  One block; it reads the tiles' counts twice.
template <typename R>
__global__ void __launch_bounds__(1024) particle_offsets_kernel(const BoxDev<R> *__restrict__ boxes, int box, int s,
                                                                int cur, int32_t *__restrict__ info)
{
    __shared__ int part[1024];
    const BoxDev<R> &B = boxes[box];
    const SpeciesDev<R> &S = B.sp[s];
    const int tid = threadIdx.x, per = (B.ntiles + 1023) / 1024;
    const int t0 = min(B.ntiles, tid * per), t1 = min(B.ntiles, t0 + per);
    int mine = 0;
    for (int t = t0; t < t1; ++t) mine += tile_ranges(S, cur, t).n;
    part[tid] = mine;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int v = tid >= off ? part[tid - off] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    int run = part[tid] - mine;
    for (int t = t0; t < t1; ++t) {
        S.tcount[t] = run;
        run += tile_ranges(S, cur, t).n;
    }
    if (tid == 1023) {
        S.tcount[B.ntiles] = part[1023];
        info[0] = part[1023] + overflow_range(B, S, cur).n;
        info[1] = 0;
    }
}

// Whether the ids are 0 .. total - 1, each once (info[1] stays zero): then an
// id is its own place in the output's order.
template <typename R>
__global__ void __launch_bounds__(kBlock) particle_ids_kernel(const BoxDev<R> *__restrict__ boxes,
                                                              const Item *__restrict__ items, int s, int cur, int total,
                                                              uint32_t *__restrict__ seen, int32_t *__restrict__ info)
{
    const Item it = items[blockIdx.x];
    const BoxDev<R> &B = boxes[it.box];
    const SpeciesDev<R> &S = B.sp[s];
    int first, stride;
    const TileRanges r = item_range(B, S, cur, it.tile, first, stride);
    for (int p = first; p < r.n; p += stride) {
        const int32_t id = S.buf[cur].id[r.slot(p)];
        const uint32_t bit = 1u << (id & 31);
        if (id < 0 || id >= total || (atomicOr(&seen[id >> 5], bit) & bit)) info[1] = 1;
    }
}

// The particles whose place in the output lies in [lo, hi): absolute position
// and momentum in FP64, and the id.  Places: the id (by_id) or tile order.
template <typename R>
__global__ void __launch_bounds__(kBlock) particles_out_kernel(const BoxDev<R> *__restrict__ boxes,
                                                               const Item *__restrict__ items, int s, int cur, int by_id,
                                                               int lo, int hi, double *__restrict__ x,
                                                               double *__restrict__ u, int32_t *__restrict__ ids)
{
    const Item it = items[blockIdx.x];
    const BoxDev<R> &B = boxes[it.box];
    const SpeciesDev<R> &S = B.sp[s];
    const PBuf<R> P = S.buf[cur];
    int first, stride, o[3] = {0, 0, 0};
    const TileRanges r = item_range(B, S, cur, it.tile, first, stride);
    if (it.tile >= 0) tile_origin(B, it.tile, o);
    const int base = S.tcount[it.tile >= 0 ? it.tile : B.ntiles];
    for (int p = first; p < r.n; p += stride) {
        const int idx = r.slot(p);
        const int32_t id = P.id ? P.id[idx] : 0;
        const int at = by_id ? id : base + p;
        if (at < lo || at >= hi) continue;
        const PSlot<R> ps = slot_at(P, idx);
        const int32_t cell = it.tile >= 0 ? local_cell(B, o, ps.code()) : P.cell[idx];
        const int c[3] = {cell_x(cell), cell_y(cell), cell_z(cell)};
        const int64_t q = 3 * (int64_t)(at - lo);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            x[q + a] = (double)c[a] + (double)ps.d(a);
            u[q + a] = (double)ps.u(a);
        }
        ids[at - lo] = id;
    }
}

// Particles [lo, lo + n) of the stage from the caller's values: positions
// wrapped into the box, cell and in-cell offset in the storage format; without
// ids given (ids == nullptr), the particle's number.
template <typename R>
__global__ void __launch_bounds__(kBlock) particles_in_kernel(const BoxDev<R> *__restrict__ boxes, int box, int s, int lo,
                                                              int n, const double *__restrict__ x,
                                                              const double *__restrict__ u, int own_ids)
{
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    const BoxDev<R> &B = boxes[box];
    const SpeciesDev<R> &S = B.sp[s];
    int c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int N = B.n[a];
        double v = x[3 * (int64_t)p + a];
        if (!(v >= 0.0 && v < N)) {
            v = fmod(v, (double)N);
            if (v < 0) v += N;
            if (v >= N) v -= N;
        }
        const double f = floor(v);
        R off = (R)(v - f);
        int ci = (int)f;
        if (off >= R(1)) { off = R(0); ci += 1; }
        if (ci >= N) ci -= N;
        c[a] = ci;
        S.stage.d[a][lo + p] = off;
        S.stage.u[a][lo + p] = (R)u[3 * (int64_t)p + a];
    }
    S.stage.cell[lo + p] = pack_cell(c[0], c[1], c[2]);
    if (own_ids && S.stage.id) S.stage.id[lo + p] = lo + p;
}

template <typename R>
hipError_t launch_particle_offsets(const BoxDev<R> *boxes, int box, int s, int cur, int32_t *info, hipStream_t st)
{
    hipLaunchKernelGGL(particle_offsets_kernel<R>, dim3(1), dim3(1024), 0, st, boxes, box, s, cur, info);
    return hipGetLastError();
}
template <typename R>
hipError_t launch_particle_ids(const BoxDev<R> *boxes, const Item *items, int nitems, int s, int cur, int total,
                               uint32_t *seen, int32_t *info, hipStream_t st)
{
    hipLaunchKernelGGL(particle_ids_kernel<R>, dim3(nitems), dim3(kBlock), 0, st, boxes, items, s, cur, total, seen, info);
    return hipGetLastError();
}
template <typename R>
hipError_t launch_particles_out(const BoxDev<R> *boxes, const Item *items, int nitems, int s, int cur, int by_id, int lo,
                                int hi, double *x, double *u, int32_t *ids, hipStream_t st)
{
    hipLaunchKernelGGL(particles_out_kernel<R>, dim3(nitems), dim3(kBlock), 0, st, boxes, items, s, cur, by_id, lo, hi, x,
                       u, ids);
    return hipGetLastError();
}
template <typename R>
hipError_t launch_particles_in(const BoxDev<R> *boxes, int box, int s, int lo, int n, const double *x, const double *u,
                               int own_ids, hipStream_t st)
{
    hipLaunchKernelGGL(particles_in_kernel<R>, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, boxes, box, s, lo, n,
                       x, u, own_ids);
    return hipGetLastError();
}

#define PIC_INSTANTIATE_IO(R)                                                                                         \
    template hipError_t launch_fields_in<R>(const double *, const int[3], int, int, R *, hipStream_t);               \
    template hipError_t launch_particle_offsets<R>(const BoxDev<R> *, int, int, int, int32_t *, hipStream_t);        \
    template hipError_t launch_particle_ids<R>(const BoxDev<R> *, const Item *, int, int, int, int, uint32_t *,      \
                                               int32_t *, hipStream_t);                                              \
    template hipError_t launch_particles_out<R>(const BoxDev<R> *, const Item *, int, int, int, int, int, int,       \
                                                double *, double *, int32_t *, hipStream_t);                         \
    template hipError_t launch_particles_in<R>(const BoxDev<R> *, int, int, int, int, const double *, const double *, \
                                               int, hipStream_t);
PIC_INSTANTIATE_IO(float)
PIC_INSTANTIATE_IO(double)

} // namespace pic
