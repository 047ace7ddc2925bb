// Internal device-side layout of the gfx950 PIC library (not part of the ABI).
//
// Particles of one (box, species) live in slots binned by spatial tile (PBuf).
// Two copies of them alternate between steps: the push reads copy
// `cur` and writes every particle straight into the segment of its new tile in
// copy `cur ^ 1`, so the binning is refreshed every step at no extra traffic.
// Tile T owns the slots [seg_start[c][T], seg_start[c][T] + seg_cap[c][T]) of
// copy c and holds two ranges of particles there, all with their cell in T:
//   A = [0, na[c][T])                the tile's own particles that stayed,
//   B = [bs[c][T], bs[c][T] + nb[c][T])  particles that entered from elsewhere.
// The block that pushes tile T writes A from the front with an LDS counter and
// stages its leavers at the back of [0, n_src); at the end it hands them to
// the neighbouring tiles' B ranges, one global atomic per neighbour.  bs of the
// next step is the current particle count of the tile, set between steps.
// The last segment (index ntiles) is an overflow region (count nb[c][ntiles])
// for particles whose target range is full; it is swept by the slow path
// (fields read from HBM, current added with global atomics).  A counting-sort
// repack recomputes the segment layout from the actual counts.
//
// Stored particle state: the cell (a one-byte code local to the tile, or packed
// as ix | iy << 11 | iz << 22), in-cell offset d in [0, 1) per axis, and u =
// gamma v / c.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pic.h"

// Device pointers into the arena are global-memory pointers; saying so in the
// descriptor types lets the compiler emit global_* instead of flat_* memory
// instructions for every access through them.  The qualifier only exists in
// the device compilation of files with kernels; the host (and the host-only
// API file, which defines PIC_HOST_ONLY_TU) sees plain pointers of the same size.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(PIC_HOST_ONLY_TU)
#define PIC_GLOBAL __attribute__((address_space(1)))
#else
#define PIC_GLOBAL
#endif

namespace pic {

constexpr int kMaxSpecies = PIC_MAX_SPECIES;
constexpr int kOvfBlocks = 16;     // blocks per box sweeping the overflow region
constexpr int kBlock = 256;        // threads per block of the particle kernels
// threads per block of the push where tiles are few (0: kBlock): up to two tiles
// per CU, and up to one in the FP32 form (wide_push_kernel has the times)
constexpr int kWideTiles = 512;
template <typename R>
constexpr int wide_threads(int tiles)
{
    return tiles > kWideTiles ? 0 : (tiles <= kWideTiles / 2 && sizeof(R) == 4 ? 1024 : 512);
}
constexpr int kQBits = 31;         // fractional bits of the fixed-point current
// LDS one workgroup may allocate on gfx950 (160 KiB per CU, minus the push
// kernel's static counters and tables)
constexpr size_t kMaxLds = 160 * 1024 - 2176;

__host__ __device__ inline int32_t pack_cell(int ix, int iy, int iz)
{
    return (int32_t)((uint32_t)ix | ((uint32_t)iy << 11) | ((uint32_t)iz << 22));
}
__host__ __device__ inline int cell_x(int32_t c) { return (int)((uint32_t)c & 2047u); }
__host__ __device__ inline int cell_y(int32_t c) { return (int)(((uint32_t)c >> 11) & 2047u); }
__host__ __device__ inline int cell_z(int32_t c) { return (int)((uint32_t)c >> 22); }

// A particle in a tile's ranges keeps its cell as a one-byte code local to
// the tile, x | y << tx | z << (tx + ty) (tile edges 2^tx, 2^ty, 2^tz, at most
// 256 cells; tiles start at multiples of their edges, so the code is the low
// bits of the cell's coordinates).  The overflow region, whose particles
// belong to any tile, keeps the packed cell; so do the leavers that the push's
// general loop stages for the hand-over (its loop for 4x4x4 tiles stages a
// one-byte code of the tile grown by one cell).
//
// d, u and the code of a copy are kept in groups of slots: six rows of values
// (d x, y, z, u x, y, z), then the codes.  A block that walks a tile's segment
// then reads one stream and writes one, instead of seven of each: a
// copy-shaped kernel with the push's block order moves 33.5 M particles in
// 0.319 ms this way and in 0.384-0.424 ms with one array per value (5.3
// against 4.0-4.4 TB/s), and a slot is one address with constant offsets.
// 128 slots in FP32 (3200 B, whole 128-B lines); 64 in FP64 (3136 B), where the
// rows of 128 slots would lie past a load's constant offset.
template <typename R>
struct PBuf {                      // one copy of the particle arrays
    static constexpr int kSlots = sizeof(R) == 4 ? 128 : 64, kShift = sizeof(R) == 4 ? 7 : 6;
    static constexpr int kRow = kSlots * (int)sizeof(R);
    static constexpr int kGroup = 6 * kRow + kSlots;
    PIC_GLOBAL uint8_t *rec;       // the groups
    PIC_GLOBAL int32_t *cell;      // packed cell (overflow region, staged leavers)
    PIC_GLOBAL int32_t *id;        // nullptr without PIC_TRACK_IDS
    static constexpr int kSpare = 64;   // slots after the last one that idle lanes may write
    __host__ __device__ static size_t bytes(size_t slots)
    {
        return (slots + kSpare + kSlots - 1) / kSlots * (size_t)kGroup;
    }
};

// One slot of a copy: the address of its d x (the other five values are whole
// rows further on) and of its code.
template <typename R>
struct PSlot {
    PIC_GLOBAL uint8_t *row, *lc;
    __host__ __device__ PIC_GLOBAL R &d(int a) const
    {
        return *reinterpret_cast<PIC_GLOBAL R *>(row + a * PBuf<R>::kRow);
    }
    __host__ __device__ PIC_GLOBAL R &u(int a) const { return d(3 + a); }
    __host__ __device__ PIC_GLOBAL uint8_t &code() const { return *lc; }
};

// Slot i of copy P.  NARROW: the copy is smaller than 4 GiB, so that a slot is
// a 32-bit byte offset from a (wave-uniform) base, formed with 24-bit
// multiplies (slots / 64 < 2^23).
template <bool NARROW = false, typename R>
__host__ __device__ inline PSlot<R> slot_at(const PBuf<R> &P, int i)
{
    constexpr uint32_t G = PBuf<R>::kGroup;
    PSlot<R> s;
    const uint32_t l = (uint32_t)i & (PBuf<R>::kSlots - 1), g = (uint32_t)i >> PBuf<R>::kShift;
#ifdef __HIP_DEVICE_COMPILE__
    if (NARROW) {
        const uint32_t at = __umul24(g, G) + l;
        s.row = P.rec + (uint32_t)(at + l * (uint32_t)(sizeof(R) - 1));
        s.lc = P.rec + at + 6 * PBuf<R>::kRow;
        return s;
    }
#endif
    PIC_GLOBAL uint8_t *at = P.rec + (uint64_t)g * G + l;
    s.row = at + l * (uint32_t)(sizeof(R) - 1);
    s.lc = at + 6 * PBuf<R>::kRow;
    return s;
}

template <typename R>
struct PStage {                    // particles loaded or set and not yet binned
    PIC_GLOBAL int32_t *cell;
    PIC_GLOBAL R *d[3];
    PIC_GLOBAL R *u[3];
    PIC_GLOBAL int32_t *id;        // nullptr without PIC_TRACK_IDS
};

template <typename R>
struct SpeciesDev {
    PBuf<R> buf[2];
    PStage<R> stage;
    PIC_GLOBAL int32_t *seg_start[2];   // ntiles + 1 per copy (last: overflow region)
    PIC_GLOBAL int32_t *seg_cap[2];     // ntiles + 1 per copy
    PIC_GLOBAL int32_t *na[2];          // ntiles + 1 per copy: A-range count
    PIC_GLOBAL int32_t *nb[2];          // ntiles + 1 per copy: B-range count (overflow count last)
    PIC_GLOBAL int32_t *bs[2];          // ntiles + 1 per copy: B-range start
    PIC_GLOBAL int32_t *tcount;         // ntiles + 1, repack scratch
    int32_t slots;                 // length of each array
    int32_t ovf_cap;               // slots reserved for the overflow region
};

// J type: int64 fixed point (2^-31 cell volumes) for FP32, double for FP64.
template <typename R> struct JType;
template <> struct JType<float> { using T = long long; };
template <> struct JType<double> { using T = double; };

template <typename R>
struct BoxDev {
    int32_t n[3];
    int32_t tshift[3];             // log2 of the tile edge per axis
    int32_t ntile[3];
    int32_t ntiles;
    int64_t nc;
    PIC_GLOBAL R *e;               // 3 * nc, e^t
    PIC_GLOBAL R *b;               // 3 * nc, b^{t-dt/2}
    PIC_GLOBAL R *bn;              // 3 * nc, the other b buffer: the push writes b^{t+dt/2} there
    PIC_GLOBAL typename JType<R>::T *J;   // 3 * nc, current of the step in flight
    PIC_GLOBAL double *rho;        // nc, diagnostic charge density
    PIC_GLOBAL double *acc;        // diagnostic accumulators (kAccLen doubles, the other copies before them)
    PIC_GLOBAL int64_t *hist;      // n_species * hist_bins
    double alpha0;                 // 2 / (n_x^2 rho0)
    int32_t wall;                  // axis with conducting walls, -1: periodic
    int32_t faraday4;              // fourth-order curl of e in Faraday's law
    SpeciesDev<R> sp[kMaxSpecies];
};

// per-launch constants of the particle kernels
template <typename R>
struct StepConst {
    R dt;
    int32_t nsp;
    R kq[kMaxSpecies];             // (q/e)(m_e/m)
    R qs[kMaxSpecies];             // sgn(q)
    R mass[kMaxSpecies];           // m/m_e
    PIC_GLOBAL uint32_t *flags;    // device error flag word
    int32_t cur;                   // copy read this step
    int32_t hist_bins;
    double hist_lo, hist_hi;
    int32_t filter;                // smooth the current (and the Gauss charge)
};

// diagnostic accumulator layout per box
constexpr int kAccField = 0;       // [0..2] sum e^2/2, [3..5] sum (b^t)^2/2, [6] gauss max, [7] gauss sum sq
constexpr int kAccSp = 8;          // then per species 6: K, P[3], count, sum(gamma-1)
constexpr int kAccLen = kAccSp + 6 * kMaxSpecies;
constexpr int kAccCopies = 16;     // blocks add to one of these many copies, so that fewer meet on an address

// work item of the particle kernels: box, and tile (>= 0) or -1-k for overflow
// block k; box -1 is an idle item (padding of the push order)
struct Item {
    int32_t box;
    int32_t tile;
};

__device__ inline int wrap_idx(int i, int n)
{
    int r = i % n;
    return r < 0 ? r + n : r;
}

template <typename R>
__device__ inline int tile_of(const BoxDev<R> &B, int32_t c)
{
    // tile counts are below 2^11, so 24-bit multiplies are exact
    const unsigned ty = (unsigned)(cell_y(c) >> B.tshift[1]), tz = (unsigned)(cell_z(c) >> B.tshift[2]);
    return (cell_x(c) >> B.tshift[0]) +
           (int)__umul24((unsigned)B.ntile[0], ty + __umul24((unsigned)B.ntile[1], tz));
}

// Tile-local code of a cell (the low bits of its coordinates) and its inverse
// for a tile with origin o.
template <typename R>
__device__ inline int local_code(const BoxDev<R> &B, int32_t c)
{
    const int sx = B.tshift[0], sy = B.tshift[1];
    return (cell_x(c) & ((1 << sx) - 1)) | ((cell_y(c) & ((1 << sy) - 1)) << sx) |
           ((cell_z(c) & ((1 << B.tshift[2]) - 1)) << (sx + sy));
}

template <typename R>
__host__ __device__ inline int32_t local_cell(const BoxDev<R> &B, const int o[3], int code)
{
    const int sx = B.tshift[0], sy = B.tshift[1];
    return pack_cell(o[0] + (code & ((1 << sx) - 1)), o[1] + ((code >> sx) & ((1 << sy) - 1)), o[2] + (code >> (sx + sy)));
}

// Origin cell of tile T.
template <typename R>
__host__ __device__ inline void tile_origin(const BoxDev<R> &B, int T, int o[3])
{
    const int r = T / B.ntile[0];
    o[0] = (T - r * B.ntile[0]) << B.tshift[0];
    o[1] = (r % B.ntile[1]) << B.tshift[1];
    o[2] = (r / B.ntile[1]) << B.tshift[2];
}

// The particles of tile T in copy c: the A range then the clamped B range.
struct TileRanges {
    int start, na, bs, n;
    __device__ int slot(int q) const { return start + (q < na ? q : bs + (q - na)); }
};

template <typename R>
__device__ inline TileRanges tile_ranges(const SpeciesDev<R> &S, int c, int T)
{
    TileRanges r;
    r.start = S.seg_start[c][T];
    r.na = S.na[c][T];
    r.bs = S.bs[c][T];
    r.n = r.na + max(0, min(S.nb[c][T], S.seg_cap[c][T] - r.bs));
    return r;
}

// The overflow region of copy c as a range.
template <typename R>
__device__ inline TileRanges overflow_range(const BoxDev<R> &B, const SpeciesDev<R> &S, int c)
{
    TileRanges r;
    r.start = S.seg_start[c][B.ntiles];
    r.na = min(S.nb[c][B.ntiles], S.ovf_cap);
    r.bs = 0;
    r.n = r.na;
    return r;
}

// The particles of a work item in copy c: a tile's A and B ranges (one block
// striding), or the overflow region (kOvfBlocks blocks striding).
template <typename R>
__device__ inline TileRanges item_range(const BoxDev<R> &B, const SpeciesDev<R> &S, int c, int tile, int &first,
                                        int &stride)
{
    if (tile >= 0) {
        first = threadIdx.x;
        stride = kBlock;
        return tile_ranges(S, c, tile);
    }
    first = (-1 - tile) * kBlock + threadIdx.x;
    stride = kBlock * kOvfBlocks;
    return overflow_range(B, S, c);
}

// cell blocks of the field kernels: (box, first cell) of kBlock cells
struct CellBlock {
    int32_t box;
    int32_t first;
};

// stage item: particles [first, last) of the stage of (box, species), the
// chunk of one block.  A chunk holds 16 particles per tile of the box, so that
// counting them per tile in LDS saves most of the global atomics, within
// [4096, 65536]: enough blocks for a small load, and the LDS table of
// kCountTiles tiles (64 KB) never larger than the chunk.  4096 in boxes of more
// tiles, whose blocks have no table to fill (256,000 particles in 64000 tiles:
// counted in 14 us, 137 in chunks of 65536, which are four blocks).
struct StageItem {
    int32_t box, species, first, last;
};
constexpr int kStageBlock = 1024;      // threads per block of the stage kernels
constexpr int kCountTiles = 16384;
inline int stage_chunk(int ntiles)
{
    if (ntiles > kCountTiles) return 4096;
    const int64_t n = ((int64_t)16 * ntiles + 1023) / 1024 * 1024;
    return (int)(n < 4096 ? 4096 : (n > 65536 ? 65536 : n));
}

// one drifting Maxwell-Juttner population of a load
struct MJPop {
    double mu, G, beta0;
    int axis;
    const PIC_GLOBAL double *tab;
};

struct LoadArgs {
    int32_t box, sa, sb;
    int64_t npairs;
    int32_t offa, offb;        // first stage slot of each species
    int32_t ida, idb;          // first particle id of each species
    int32_t profile, paxis;
    double centre, thick, halfw;
    uint64_t seed, stream;
    int N;                     // table intervals
    MJPop A, B;
};

// Where the diagnostics sum: kAccLen accumulators, the charge density (one
// value per cell) and the gamma-1 histogram (n_species x bins).  pic_diag
// points it into the arena, pic_diag_noalloc into the library's static
// scratch.
struct DiagBuf {
    PIC_GLOBAL double *acc;        // copy 0; copy r lies r * kAccLen before it
    PIC_GLOBAL double *rho;        // right behind acc
    PIC_GLOBAL int64_t *hist;      // behind rho
    int copies;
    __host__ __device__ PIC_GLOBAL double *copy(unsigned block) const
    {
        return acc - (int64_t)(block % (unsigned)copies) * kAccLen;
    }
};
static_assert(kAccLen * sizeof(double) % 256 == 0, "rho follows acc in 256-byte aligned buffers");

// size of the static scratch of pic_diag_noalloc (per GPU)
constexpr size_t kDiagScratchBytes = size_t(32) << 20;

// Where a step's overflow watch goes: 8 bytes of coherent host memory, the
// step's number in the upper half and the fill in the lower, stored at once, so
// that the host can tell a step's report from an older one by itself.
struct Watch {
    uint64_t *slot;
    uint32_t step;
};

// launchers (pic_kernels.hip, pic_loader.hip)
template <typename R> size_t push_lds_bytes(int t0, int t1, int t2);
template <typename R> size_t wide_lds_bytes(int threads);   // of a wide_push_kernel block (4x4x4 tiles)
template <typename R>
hipError_t launch_push(const BoxDev<R> *boxes, const Item *items, int nitems, size_t lds, const StepConst<R> &C,
                       int fix, int walls, int faraday4, int wide, hipStream_t st);
template <typename R>
hipError_t launch_fields(const BoxDev<R> *boxes, const CellBlock *blocks, int nblocks, R dt, int nsp, int filter,
                         int clear_copy, int nboxes, Watch watch, hipStream_t st);
template <typename R>
hipError_t launch_advance_b(const BoxDev<R> *boxes, const CellBlock *blocks, int nblocks, R h, hipStream_t st);
template <typename R>
hipError_t launch_repack(const BoxDev<R> *boxes, int nboxes, const Item *items, int nitems,
                         const StageItem *sitems, int nsitems, int split, const uint32_t *half, size_t lds, int faraday4,
                         const StepConst<R> &C, hipStream_t st);
template <typename R>
hipError_t launch_diag(const BoxDev<R> *boxes, int box, int64_t nc, const Item *items, int nitems,
                       const StepConst<R> &C, const DiagBuf &out, int hist_len, hipStream_t st);
// copies to and from the host (pic_io.hip)
template <typename R>
hipError_t launch_fields_in(const double *src, const int n[3], int wall, int is_b, R *dst, hipStream_t st);
template <typename R>
hipError_t launch_particle_offsets(const BoxDev<R> *boxes, int box, int s, int cur, int32_t *info, hipStream_t st);
template <typename R>
hipError_t launch_particle_ids(const BoxDev<R> *boxes, const Item *items, int nitems, int s, int cur, int total,
                               uint32_t *seen, int32_t *info, hipStream_t st);
template <typename R>
hipError_t launch_particles_out(const BoxDev<R> *boxes, const Item *items, int nitems, int s, int cur, int by_id, int lo,
                                int hi, double *x, double *u, int32_t *ids, hipStream_t st);
template <typename R>
hipError_t launch_particles_in(const BoxDev<R> *boxes, int box, int s, int lo, int n, const double *x, const double *u,
                               int own_ids, hipStream_t st);
hipError_t launch_zero(void *p, int64_t words, hipStream_t st);   // 8-byte words
// device address of the static diagnostics scratch of the current device:
// set up once per device (pic_init), then read
hipError_t diag_scratch_setup();
void *diag_scratch();
constexpr int kMjBlock = 1024;          // intervals per block of the table's prefix sum
constexpr int kMjChunk = 64;            // intervals per compensated sum
hipError_t launch_mj_tables(int n, const double *theta, const double *gamma_beta, double *const *cum, int M, int N,
                            double *const *tab, hipStream_t st);
template <typename R> hipError_t launch_load_pairs(const BoxDev<R> *boxes, const LoadArgs &L, hipStream_t st);
template <typename R>
hipError_t launch_harris_field(const BoxDev<R> *boxes, int64_t nc, const pic_harris_field &H, hipStream_t st);
template <typename R>
hipError_t launch_spectrum(const BoxDev<R> *boxes, int box, const int n[3], int f, int c, int an, R hdt,
                           double *scratch, double *ps, hipStream_t st);

} // namespace pic
