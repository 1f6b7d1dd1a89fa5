// HIP kernels of the blur-zone consumers of the extrapolated reference maps (Lin, Derr &
// Rycroft, arXiv 2104.00095):
//   k_blur_heaviside  per grid cell inside some solid's box: phi_m = phi0_m(xi_m) on the
//                     cells the solid labels 0..L, the smoothed Heaviside of eq. (sm_heavi),
//                     and the multi-body modified Heaviside of eq. (mod_heaviside),
//                     H = max(1 - sum_m (1 - H_eps(phi_m)), 0);
//   k_blur_stress     per cell face with a cell inside some solid's box (SI "Stress
//                     calculations"): for each solid whose difference stencil is labelled,
//                     grad xi by centred differences at the face, F = (grad xi)^{-1},
//                     B = F F^T, tau_m = G_m (B - tr(B)/3 I), the weight 1 - H_eps(phi_m)
//                     at the face's xi; the blend T (sum of weights S <= 1) or T / S.
// Tiles are 8^3 cells of the grid; the solids that can touch one come from a list built on
// the host (boxes dilated by one cell), visited in ascending order, so every sum runs in the
// same order as in any other implementation.  Each consumer runs in three launches: a fill
// writes the result every cell or face of a box takes when no solid covers its stencil
// (H = 1, zero stress); a scan, a wave per tile, lists the tiles where a candidate labels
// (0..L) a cell (dilated by one cell for the faces' stencils); the full kernel, a block per
// listed tile, then finds the covered cells or faces by bit operations on the label rows and
// computes those, packed, over the fill's values.
// Periodic axes (SI "Test cases"): a box holds the solid's unwrapped map and may run past
// the grid's end; grid cell g lies at box coordinate (g - lo) mod n there.  A tile meets
// such a box in up to two images per axis (offset by 0 or n); within an image tile and
// stencil are contiguous in box coordinates, so differences never join the two ends of a box
// that spans the axis.  Stencil gathers of FP64 fields over the thin blur zones: bandwidth
// and latency work, no MFMA.
#include "rmx_blur.h"
#include "rmx_device.h"
#include "rmx_weight.h"

namespace rmx {
namespace {
using namespace dev;

typedef const RMX_CONST_AS BlurDev BlurDevC;

__device__ __forceinline__ BlurDevC* blur_solid(const BlurBatch& b, int m) {
    return (BlurDevC*)(b.solids + m);
}

__device__ __forceinline__ ShapeR blur_shape(BlurDevC* s) {
    ShapeR r;
    r.kind = s->kind;
    r.c0 = s->centre[0]; r.c1 = s->centre[1]; r.c2 = s->centre[2];
    r.e0 = s->semi[0]; r.e1 = s->semi[1]; r.e2 = s->semi[2];
    r.r00 = s->rot[0]; r.r01 = s->rot[1]; r.r02 = s->rot[2];
    r.r10 = s->rot[3]; r.r11 = s->rot[4]; r.r12 = s->rot[5];
    r.r20 = s->rot[6]; r.r21 = s->rot[7]; r.r22 = s->rot[8];
    return r;
}

// The first cell of tile t in grid coordinates.
__device__ __forceinline__ void tile_origin(const BlurBatch& b, int t, int o[3]) {
    o[0] = t % b.tiles[0] * kBlurTX;
    o[1] = t / b.tiles[0] % b.tiles[1] * kBlurTY;
    o[2] = t / (b.tiles[0] * b.tiles[1]) * kBlurTZ;
}

// Image i (bit a: offset by n along a periodic axis a) of a tile with origin o in the solid's
// box: d, the box coordinates of the tile's first cell.  False where the tile, dilated by
// `h` cells, misses the box, or the image does not exist.
__device__ __forceinline__ bool tile_image(const BlurBatch& b, BlurDevC* s, const int o[3], int i,
                                           int h, int d[3]) {
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool moved = (i >> a) & 1;
        d[a] = o[a] - s->lo[a] + (moved ? b.grid[a] : 0);
        ok = ok && !(moved && !b.periodic[a]) && d[a] + 8 + h > 0 && d[a] - h < s->ext[a];
    }
    return ok;
}

// Covered cells (label 0..L) of row (y, z) of the tile dilated by h cells, as bits; d as
// above.  The 12 columns from d[0] - h on are read, the caller keeps what it needs.
__device__ __forceinline__ unsigned cover_row(BlurDevC* s, const int d[3], int h, int y, int z) {
    const int e0 = s->ext[0], e1 = s->ext[1], e2 = s->ext[2];
    const int gy = d[1] - h + y, gz = d[2] - h + z, ox = d[0] - h;
    if ((unsigned)gy >= (unsigned)e1 || (unsigned)gz >= (unsigned)e2 || ox >= e0) return 0u;
    const RowBits r = label_row_bits(s->labels, e0 * e1 * e2, (gz * e1 + gy) * e0 + ox, ox, e0,
                                     s->L);
    return r.data | r.target;
}

// The columns of a tile that lie in the grid.
__device__ __forceinline__ unsigned grid_columns(const BlurBatch& b, const int o[3]) {
    return b.grid[0] - o[0] >= kBlurTX ? 0xFFu : (1u << (b.grid[0] - o[0])) - 1u;
}

// ------------------------------------------------------------------------------------
// The scan: does a candidate label any cell of the tile, dilated by one cell for the
// stress (a face's difference stencil reaches one cell beyond its owner's tile)?  A wave
// takes a tile, one or two label rows per lane (16-byte loads); a block appends its tiles
// with one atomic.  Bound by the chain of dependent loads to a tile's labels, so every tile
// is a wave of its own.  One 256^3 box: 21 us (H) and 28 us (stress); a thread per cell
// and candidate, bytes at a time, took 63 and 97 us, four tiles per wave in turn 22 and 34 us.
// ------------------------------------------------------------------------------------
template <bool STRESS>
__device__ __forceinline__ bool tile_covered(const BlurBatch& b, int t) {
    constexpr int h = STRESS ? 1 : 0, D = 8 + 2 * h;
    const int lane = threadIdx.x & 63;
    const int e0 = load_const(b.tile_start + t), e1 = load_const(b.tile_start + t + 1);
    int o[3];
    tile_origin(b, t, o);
    const int images = b.periodic[0] || b.periodic[1] || b.periodic[2] ? 8 : 1;
    for (int e = e0; e < e1; ++e) {
        BlurDevC* s = blur_solid(b, load_const(b.tile_list + e));
        for (int i = 0; i < images; ++i) {
            int d[3];
            if (!tile_image(b, s, o, i, h, d)) continue;   // uniform
            unsigned bits = 0u;
#pragma unroll
            for (int r = lane; r < D * D; r += 64) bits |= cover_row(s, d, h, r % D, r / D);
            if (__ballot((bits & ((1u << D) - 1u)) != 0u)) return true;
        }
    }
    return false;
}

template <bool STRESS>
__global__ __launch_bounds__(256) void k_blur_scan(BlurBatch b) {
    __shared__ int s_tile[4];
    const int lane = threadIdx.x & 63, wid = uniform_int(threadIdx.x >> 6);
    const int i = blockIdx.x * 4 + wid;
    int t = -1;
    if (i < b.n_active) {   // uniform
        t = load_const(b.active + i);
        if (!tile_covered<STRESS>(b, t)) t = -1;
    }
    if (lane == 0) s_tile[wid] = t;
    __syncthreads();
    if (threadIdx.x < 64) {   // (lanes 0..3 hold the block's tiles)
        t = lane < 4 ? s_tile[lane & 3] : -1;
        const unsigned long long m = __ballot(t >= 0);
        int base = 0;
        if (lane == 0 && m) base = atomicAdd(b.n_covered, __popcll(m));
        base = uniform_int(base);
        if (t >= 0) b.covered[base + __popcll(m & ((1ull << lane) - 1ull))] = t;
    }
}

// ------------------------------------------------------------------------------------
// The fill: what a cell or face with no covered stencil takes (H = 1 on a cell inside some
// box; zero stress on a face with a cell inside some box), over every box.  Regions that
// overlap are written more than once, with the same value.  A region (a solid's cells, or
// its faces along an axis: ext_a + 1 of them along a, at most n on a periodic axis) is cut
// into units, a wave each: 8192 consecutive values where the region spans whole planes of
// the array (16-byte stores), else 16 rows along x of one plane.  Bound by the stores where
// planes are whole: 2.4 GB of stress zeros of one 256^3 box 418 us (5.8 TB/s; a row along x
// per wave 469 us).  The runs bypass the caches, since they hold nothing of use to the next
// kernel: through the caches 434 us (426 against 415 on arrays written for the first time, 436
// against 421 on four sets of arrays in turn), and the stress kernel behind it 107 us against 100.
// The rows of small boxes go through the caches (127 us for 376 MB on 40 boxes; bypassing them
// 235: a row's ends share cache lines with cells outside the box).
// ------------------------------------------------------------------------------------
__device__ __forceinline__ int fill_extent(const BlurBatch& b, BlurDevC* s, int a, int ax) {
    const int e = s->ext[ax] + (ax == a ? 1 : 0);
    return b.periodic[ax] && e > b.grid[ax] ? b.grid[ax] : e;
}

__device__ __forceinline__ int find_solid_by_unit(const BlurBatch& b, int64_t u) {
    const BlurDev* s = b.solids;
    return wave_search(b.n_solids, u, [s](int i) { return (int64_t)load_global(&s[i].unit0); });
}

// n values v from p on, by a wave: 16-byte stores, single ones at unaligned ends.
__device__ __forceinline__ void fill_run(double* p, int64_t n, double v, int lane) {
    if (n <= 0) return;
    if ((reinterpret_cast<uintptr_t>(p) & 15u) != 0) {
        if (lane == 0) p[0] = v;
        ++p;
        --n;
    }
    typedef double Two __attribute__((ext_vector_type(2)));
    Two* q = reinterpret_cast<Two*>(p);
    for (int64_t i = lane; i < n / 2; i += 64) __builtin_nontemporal_store(Two{v, v}, q + i);
    if ((n & 1) && lane == 0) p[n - 1] = v;
}

template <bool STRESS>
__device__ __forceinline__ void fill_unit(const BlurBatch& b, int64_t u, int lane) {
    const int m = find_solid_by_unit(b, u);
    BlurDevC* s = blur_solid(b, m);
    int64_t r = u - s->unit0;
    int a = 0;
    if (STRESS) {
        a = r >= s->units[0] + s->units[1] ? 2 : (r >= s->units[0] ? 1 : 0);
        r -= (a > 0 ? s->units[0] : 0) + (a > 1 ? s->units[1] : 0);
    }
    const int comps = STRESS ? 6 : 1;
    const int per = (int)(s->units[a] / comps);   // units per component
    const int c = (int)r / per;
    int q = (int)r - c * per;
    const int fa = STRESS ? a : 3;   // (3: cells)
    const int64_t n0 = b.grid[0] + (fa == 0 && !b.periodic[0]),
                  n1 = b.grid[1] + (fa == 1 && !b.periodic[1]),
                  n2 = b.grid[2] + (fa == 2 && !b.periodic[2]);
    const int E0 = fill_extent(b, s, fa, 0), E1 = fill_extent(b, s, fa, 1),
              E2 = fill_extent(b, s, fa, 2);
    double* out = (STRESS ? b.tau[a] : b.H) + (int64_t)c * (n0 * n1 * n2);
    const double v = STRESS ? 0.0 : 1.0;
    if (fill_planes(E0, E1, (int)n0, (int)n1)) {   // (lo is 0 there, or wraps onto itself)
        const int64_t plane = n0 * n1, total = plane * E2, i0 = (int64_t)q * kFillRun;
        const int64_t i1 = i0 + kFillRun < total ? i0 + kFillRun : total;
        const int64_t start = (int64_t)s->lo[2] * plane, end = plane * n2;
        // planes past the end of a periodic axis wrap to its first
        const int64_t p0 = start + i0, p1 = start + i1;
        fill_run(out + p0, (p1 < end ? p1 : end) - p0, v, lane);
        const int64_t w0 = p0 > end ? p0 - end : 0;
        fill_run(out + w0, p1 - end - w0, v, lane);
        return;
    }
    const int chunks = (E1 + kFillRows - 1) / kFillRows;
    const int z = q / chunks, y0 = (q - z * chunks) * kFillRows;
    int gz = s->lo[2] + z;
    if (b.periodic[2] && gz >= b.grid[2]) gz -= b.grid[2];
    const int ny = E1 - y0 < kFillRows ? E1 - y0 : kFillRows;
    for (int x = lane; x < E0; x += 64) {
        int gx = s->lo[0] + x, gy = s->lo[1] + y0;
        if (b.periodic[0] && gx >= b.grid[0]) gx -= b.grid[0];
        if (b.periodic[1] && gy >= b.grid[1]) gy -= b.grid[1];
        double* p = out + ((int64_t)gz * n1 + gy) * n0 + gx;
        if (!b.periodic[1]) {   // a loop of its own: 125 boxes of 22^3 cells 70 us against 73
            for (int y = 0; y < ny; ++y, p += n0) *p = v;
            continue;
        }
        for (int y = 0; y < ny; ++y) {
            *p = v;
            p += n0;
            if (++gy == b.grid[1]) {   // uniform
                gy = 0;
                p -= n1 * n0;
            }
        }
    }
}

template <bool STRESS>
__global__ __launch_bounds__(256) void k_blur_fill(BlurBatch b) {
    const int lane = threadIdx.x & 63;
    int64_t u = (int64_t)blockIdx.x * 4 + uniform_int(threadIdx.x >> 6);
    for (; u < b.fill_units; u += (int64_t)gridDim.x * 4) fill_unit<STRESS>(b, u, lane);
}

// Blocks of the full kernels: they stride over the covered tiles.
constexpr int kBlurFullBlocks = 4096;

// Bits of a tile's 64 rows (row r = 8 z + y per lane, `bits` its columns) as a list of cell
// numbers x + 8 r, by one wave; returns their number.
__device__ __forceinline__ int list_cells(unsigned bits, int lane, uint16_t* list) {
    const unsigned long long lt = (1ull << lane) - 1ull;
    int n = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const unsigned long long m = __ballot((bits >> x) & 1u);
        if ((bits >> x) & 1u) list[n + __popcll(m & lt)] = (uint16_t)(8 * lane + x);
        n += __popcll(m);
    }
    return n;
}

// ------------------------------------------------------------------------------------
// Modified Heaviside (and phi_m).  Spheres: a distance costs less than finding the covered
// cells first, so each thread takes two cells of the tile and visits the candidates.
// Otherwise the covered cells of a tile are listed by one wave; the certificates decide most
// weights; the cells they leave are listed again, so that the exact distances (a bisection)
// run in full waves.  256 threads a tile: the chain of the distance binds, and its rounds over a
// tile count (with 128 threads 50 us instead of 47 for 40 ellipsoids, 62 instead of 48 for phi of
// a 128^3 box; 512 threads, with phi: the call 100 us against 90 on the 40, 73 against 79 on the
// box).  Measured: 40 ellipsoids 95 -> 47 us without phi (81 with a bisection of each
// point), 49 with phi (28 bytes of scratch); one sphere in 256^3 16.6 -> 15.6 us with phi (the
// listed form took 27 us there).
__global__ __launch_bounds__(256) void k_blur_heaviside_spheres(BlurBatch b) {
    const int tid = threadIdx.x;
    const int images = b.periodic[0] || b.periodic[1] || b.periodic[2] ? 8 : 1;
    const int n_tiles = load_const(b.n_covered);
    const XcdRange rg = xcd_range(n_tiles);   // neighbouring tiles share cache lines
    for (int k = rg.begin; k < rg.end; k += rg.stride) {
        const int t = load_const(b.covered + k);
        const int e0 = load_const(b.tile_start + t), e1 = load_const(b.tile_start + t + 1);
        int o[3];
        tile_origin(b, t, o);
        const int x = tid % 8, y = tid / 8 % 8, z = tid / 64;   // and z + 4
        const bool in_row = o[0] + x < b.grid[0] && o[1] + y < b.grid[1];
        double acc[2] = {0.0, 0.0};
        bool any[2] = {false, false};
        for (int e = e0; e < e1; ++e) {
            BlurDevC* s = blur_solid(b, load_const(b.tile_list + e));
            const int nxy = s->ext[0] * s->ext[1];
            const int64_t nc = (int64_t)nxy * s->ext[2];
            for (int i = 0; i < images; ++i) {
                int d[3];
                if (!tile_image(b, s, o, i, 0, d)) continue;   // uniform
                const bool in_box = in_row && (unsigned)(d[0] + x) < (unsigned)s->ext[0] &&
                                    (unsigned)(d[1] + y) < (unsigned)s->ext[1];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int zz = z + 4 * h;
                    if (!in_box || o[2] + zz >= b.grid[2] ||
                        (unsigned)(d[2] + zz) >= (unsigned)s->ext[2])
                        continue;
                    const int c = (d[2] + zz) * nxy + (d[1] + y) * s->ext[0] + d[0] + x;
                    const int lab = load_global(s->labels + c);
                    if (lab < 0 || lab > s->L) continue;
                    const double p = phi0_sphere(blur_shape(s), load_global(s->xi + c),
                                                 load_global(s->xi + nc + c),
                                                 load_global(s->xi + 2 * nc + c));
                    if (s->phi) s->phi[c] = p;
                    acc[h] += 1.0 - heaviside_eps(p, b.eps);
                    any[h] = true;
                }
            }
        }
        if (!b.H) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!any[h]) continue;   // the fill's value
            const double r = 1.0 - acc[h];
            b.H[((int64_t)(o[2] + z + 4 * h) * b.grid[1] + o[1] + y) * b.grid[0] + o[0] + x] =
                r > 0.0 ? r : 0.0;
        }
    }
}

constexpr int kHeavisideThreads = 256;

__global__ __launch_bounds__(kHeavisideThreads, 4) void k_blur_heaviside(BlurBatch b) {
    __shared__ double s_acc[kBlurTileCells];
    __shared__ uint16_t s_list[kBlurTileCells], s_left[kBlurTileCells];
    __shared__ unsigned s_any[64];   // covered columns of each row, over all solids
    __shared__ int s_n, s_m;
    const int tid = threadIdx.x, lane = tid & 63, wid = uniform_int(tid >> 6);
    const int images = b.periodic[0] || b.periodic[1] || b.periodic[2] ? 8 : 1;
    const int n_tiles = load_const(b.n_covered);
    const XcdRange rg = xcd_range(n_tiles);   // neighbouring tiles share cache lines
    for (int k = rg.begin; k < rg.end; k += rg.stride) {
        const int t = load_const(b.covered + k);
        const int e0 = load_const(b.tile_start + t), e1 = load_const(b.tile_start + t + 1);
        int o[3];
        tile_origin(b, t, o);
        for (int q = tid; q < kBlurTileCells; q += kHeavisideThreads) s_acc[q] = 0.0;
        if (tid < 64) s_any[tid] = 0u;
        __syncthreads();
        for (int e = e0; e < e1; ++e) {
            BlurDevC* s = blur_solid(b, load_const(b.tile_list + e));
            const int nx = s->ext[0], nxy = nx * s->ext[1];
            const int64_t nc = (int64_t)nxy * s->ext[2];
            const double* xi = s->xi;
            double* phi = s->phi;
            for (int i = 0; i < images; ++i) {
                int d[3];
                if (!tile_image(b, s, o, i, 0, d)) continue;   // uniform
                if (wid == 0) {
                    const int y = lane % 8, z = lane / 8;
                    unsigned bits = 0u;
                    if (o[1] + y < b.grid[1] && o[2] + z < b.grid[2])
                        bits = cover_row(s, d, 0, y, z) & grid_columns(b, o);
                    s_any[lane] |= bits;
                    const int n = list_cells(bits, lane, s_list);
                    if (lane == 0) {
                        s_n = n;
                        s_m = 0;
                    }
                }
                __syncthreads();
                const int n = s_n;
                const int origin = d[2] * nxy + d[1] * nx + d[0];
                for (int j0 = 0; j0 < n; j0 += kHeavisideThreads) {   // uniform
                    const int j = j0 + tid;
                    bool left = false;
                    int q = 0;
                    if (j < n) {
                        q = s_list[j];
                        const int c = origin + (q >> 6) * nxy + ((q >> 3) & 7) * nx + (q & 7);
                        const double x0 = load_global(xi + c), x1 = load_global(xi + nc + c),
                                     x2 = load_global(xi + 2 * nc + c);
                        double w;
                        left = phi || !weight_certain(blur_shape(s), x0, x1, x2, b.eps, &w);
                        if (!left) s_acc[q] += w;
                    }
                    const unsigned long long m = __ballot(left);
                    int base = 0;
                    if (lane == 0 && m) base = atomicAdd(&s_m, __popcll(m));
                    base = uniform_int(base);
                    if (left) s_left[base + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)q;
                }
                __syncthreads();
                const int nleft = s_m;
                for (int j = tid; j < nleft; j += kHeavisideThreads) {
                    const int q = s_left[j];
                    const int c = origin + (q >> 6) * nxy + ((q >> 3) & 7) * nx + (q & 7);
                    const double p = phi0(blur_shape(s), load_global(xi + c),
                                          load_global(xi + nc + c),
                                          load_global(xi + 2 * nc + c));
                    if (phi) phi[c] = p;
                    s_acc[q] += 1.0 - heaviside_eps(p, b.eps);
                }
                __syncthreads();   // the lists are free
            }
        }
        if (b.H) {
            for (int q = tid; q < kBlurTileCells; q += kHeavisideThreads) {
                if (!((s_any[q >> 3] >> (q & 7)) & 1u)) continue;   // the fill's value
                const double r = 1.0 - s_acc[q];
                b.H[((int64_t)(o[2] + (q >> 6)) * b.grid[1] + o[1] + ((q >> 3) & 7)) * b.grid[0] +
                    o[0] + (q & 7)] = r > 0.0 ? r : 0.0;
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------
// Solid stress at faces.
// ------------------------------------------------------------------------------------
constexpr int kHaloSpan = kBlurTX + 2;                            // a tile with a halo of 1
constexpr int kHaloCells = kHaloSpan * kHaloSpan * kHaloSpan;     // 1000

// The weight 1 - H_eps(phi0) of a solid at x.
template <bool kSpheres>
__device__ __forceinline__ double face_weight(BlurDevC* s, double x0, double x1, double x2,
                                              double eps) {
    if constexpr (kSpheres)
        return 1.0 - heaviside_eps(phi0_sphere(blur_shape(s), x0, x1, x2), eps);
    else
        return weight_at(blur_shape(s), x0, x1, x2, eps);
}

// a / b from r = 1 / b to rounding: the quotient and one residual correction (none where an
// infinity or a zero divisor makes it undefined).
__device__ __forceinline__ double quotient(double a, double b, double r) {
    const double q = a * r, c = fma(fma(-b, q, a), r, q);
    return c == c ? c : q;
}

// Faces of a tile row (y, z) along axis a whose whole difference stencil is covered, as bits
// (bit x: the face between cell x and the one before it along a): the two cells, and their
// neighbours across both other axes.  rows: the covered columns of the dilated tile's rows.
__device__ __forceinline__ unsigned face_bits(const unsigned* rows, int a, int y, int z) {
    constexpr int S = kHaloSpan;
    const unsigned* r = rows + (z + 1) * S + y + 1;
    unsigned v;
    if (a == 0) {
        auto pair = [&](int q) { return r[q] & (r[q] << 1); };
        v = pair(0) & pair(-1) & pair(1) & pair(-S) & pair(S);
    } else {
        const int sa = a == 1 ? 1 : S, st = a == 1 ? S : 1;
        auto pair = [&](int q) { return r[q] & r[q - sa]; };
        const unsigned p = pair(0);
        v = p & (p << 1) & (p >> 1) & pair(-st) & pair(st);
    }
    return (v >> 1) & 0xFFu;
}

// A block per covered tile and solid: the covered columns of the dilated tile's rows as
// bits, the faces whose stencil is covered listed by three waves (an axis each), xi of the
// covered cells of the dilated tile staged in LDS once for the three axes, then the listed
// faces in full waves.  Tiles that one solid covers (nearly all) store the stress directly;
// where several do, they add up in tau in ascending order, and the sums with
// S > 1 are divided at the end.  Bound by instructions and by the latency of each tile's
// chain (labels, list, xi, faces).  Measured: 40 ellipsoids in 128x128x256 420 -> 120 us,
// one sphere in 256^3 159 -> 98 us (before: an 8^3 tile's faces on all threads, ten label
// bytes and thirty xi loads per face, the bisection of the distance in sparse waves).
template <bool kSpheres>
__global__ __launch_bounds__(256, 3) void k_blur_stress(BlurBatch b) {
    constexpr int S = kHaloSpan, S2 = kHaloSpan * kHaloSpan;
    __shared__ double s_xi[3][kHaloCells];
    __shared__ unsigned s_rows[S2];
    __shared__ uint16_t s_list[3][kBlurTileCells];
    __shared__ int s_n[3];
    __shared__ double s_sum[3][kBlurTileCells];   // S of each face, where several solids cover
    __shared__ double s_w[3 * kBlurTileCells];    // the listed faces' weights
    const int images = b.periodic[0] || b.periodic[1] || b.periodic[2] ? 8 : 1;
    const int n_tiles = load_const(b.n_covered);
    int64_t nf[3];
    int64_t f0[3], f1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        f0[a] = b.grid[0] + (a == 0 && !b.periodic[0]);
        f1[a] = b.grid[1] + (a == 1 && !b.periodic[1]);
        nf[a] = f0[a] * f1[a] * (b.grid[2] + (a == 2 && !b.periodic[2]));
    }
    const XcdRange rg = xcd_range(n_tiles);   // neighbouring tiles share cache lines
    for (int k = rg.begin; k < rg.end; k += rg.stride) {
        const int t = load_const(b.covered + k);
        const int e0 = load_const(b.tile_start + t), e1 = load_const(b.tile_start + t + 1);
        int o[3];
        tile_origin(b, t, o);
        // whether more than one solid can add to a face of the tile
        // (thread indices re-derived: their math is not kept live across tiles and solids)
        const int tid0 = opaque_lane_value(threadIdx.x);
        bool many = false;
        if (e1 - e0 > 1) {   // uniform
            int covering = 0;
            for (int e = e0; e < e1; ++e) {
                BlurDevC* s = blur_solid(b, load_const(b.tile_list + e));
                unsigned bits = 0u;
                for (int i = 0; i < images; ++i) {
                    int d[3];
                    if (tile_image(b, s, o, i, 1, d) && tid0 < S2)
                        bits |= cover_row(s, d, 1, tid0 % S, tid0 / S);
                }
                covering += __syncthreads_or((bits & ((1u << S) - 1u)) != 0u) ? 1 : 0;
            }
            many = covering > 1;
        }
        if (many)
            for (int q = tid0; q < 3 * kBlurTileCells; q += 256) (&s_sum[0][0])[q] = -1.0;   // none
        for (int e = e0; e < e1; ++e) {
            BlurDevC* s = blur_solid(b, load_const(b.tile_list + e));
            const int nx = s->ext[0], nxy = nx * s->ext[1];
            const int64_t nc = (int64_t)nxy * s->ext[2];
            const double* xi = s->xi;
            const double G = s->G;
            for (int i = 0; i < images; ++i) {
                int d[3];
                if (!tile_image(b, s, o, i, 1, d)) continue;   // uniform
                const int tid = opaque_lane_value(threadIdx.x);
                const int lane = tid & 63, wid = uniform_int(tid >> 6);
                __syncthreads();   // the LDS is free
                if (tid < S2) s_rows[tid] = cover_row(s, d, 1, tid % S, tid / S) & ((1u << S) - 1u);
                __syncthreads();
                // xi of the covered cells: every load before the first store
                const int origin = (d[2] - 1) * nxy + (d[1] - 1) * nx + d[0] - 1;
                constexpr int kH = (kHaloCells + 255) / 256;
                double v[kH][3];
                unsigned on = 0u;
#pragma unroll
                for (int h = 0; h < kH; ++h) {
                    const int q = tid + 256 * h;
                    const int x = q % S, y = q / S % S, z = q / S2;
                    if (q < kHaloCells && ((s_rows[z * S + y] >> x) & 1u)) {
                        const int c = origin + z * nxy + y * nx + x;
                        on |= 1u << h;
                        v[h][0] = load_global(xi + c);
                        v[h][1] = load_global(xi + nc + c);
                        v[h][2] = load_global(xi + 2 * nc + c);
                    }
                }
                if (wid < 3) {
                    const int y = lane % 8, z = lane / 8;
                    unsigned bits = 0u;
                    if (o[1] + y < b.grid[1] && o[2] + z < b.grid[2])
                        bits = face_bits(s_rows, wid, y, z) & grid_columns(b, o);
                    const int n = list_cells(bits, lane, s_list[wid]);
                    if (lane == 0) s_n[wid] = n;
                }
#pragma unroll
                for (int h = 0; h < kH; ++h)
                    if ((on >> h) & 1u)
#pragma unroll
                        for (int c = 0; c < 3; ++c) s_xi[c][tid + 256 * h] = v[h][c];
                __syncthreads();
                const int na = s_n[0], nb = s_n[1], n = na + nb + s_n[2];
                // the weights first (each read by the thread that wrote it): with the distance
                // and the stress in one loop the registers do not suffice
                for (int j = tid; j < n; j += 256) {
                    const int a = j < na ? 0 : (j < na + nb ? 1 : 2);
                    const int q = s_list[a][j - (a > 0 ? na : 0) - (a > 1 ? nb : 0)];
                    const int r = (((q >> 6) + 1) * S + ((q >> 3) & 7) + 1) * S + (q & 7) + 1;
                    const int sa = a == 0 ? 1 : (a == 1 ? S : S2);
                    s_w[j] = face_weight<kSpheres>(
                        s, (s_xi[0][r - sa] + s_xi[0][r]) * 0.5,
                        (s_xi[1][r - sa] + s_xi[1][r]) * 0.5,
                        (s_xi[2][r - sa] + s_xi[2][r]) * 0.5, b.eps);
                }
                for (int j = tid; j < n; j += 256) {
                    const int a = j < na ? 0 : (j < na + nb ? 1 : 2);
                    const int q = s_list[a][j - (a > 0 ? na : 0) - (a > 1 ? nb : 0)];
                    const int x = q & 7, y = (q >> 3) & 7, z = q >> 6;
                    const int r = ((z + 1) * S + y + 1) * S + x + 1;
                    // strides of the face's axis, then of the other two in order
                    const int sa = a == 0 ? 1 : (a == 1 ? S : S2), s1 = a == 0 ? S : 1,
                              s2 = a == 2 ? S : S2;
                    const double w = s_w[j];
                    // J = grad xi: differences across the face, and the mean of the centred
                    // differences of its two cells along the other axes
                    double J[3][3];
                    const double hx = a == 0 ? b.h[0] : 4.0 * b.h[0],
                                 hy = a == 1 ? b.h[1] : 4.0 * b.h[1],
                                 hz = a == 2 ? b.h[2] : 4.0 * b.h[2];
                    const double rx = a == 0 ? b.rh[0] : 0.25 * b.rh[0],
                                 ry = a == 1 ? b.rh[1] : 0.25 * b.rh[1],
                                 rz = a == 2 ? b.rh[2] : 0.25 * b.rh[2];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const double* f = s_xi[c] + r;
                        const double A = f[0] - f[-sa];
                        const double P = (f[s1 - sa] - f[-s1 - sa]) + (f[s1] - f[-s1]);
                        const double Q = (f[s2 - sa] - f[-s2 - sa]) + (f[s2] - f[-s2]);
                        J[c][0] = quotient(a == 0 ? A : P, hx, rx);
                        J[c][1] = quotient(a == 0 ? P : (a == 1 ? A : Q), hy, ry);
                        J[c][2] = quotient(a == 2 ? A : Q, hz, rz);
                    }
                    // F = J^{-1} by cofactors
                    const double c00 = J[1][1] * J[2][2] - J[1][2] * J[2][1];
                    const double c01 = J[1][2] * J[2][0] - J[1][0] * J[2][2];
                    const double c02 = J[1][0] * J[2][1] - J[1][1] * J[2][0];
                    const double det = (J[0][0] * c00 + J[0][1] * c01) + J[0][2] * c02;
                    const double rd = 1.0 / det;
                    double F[3][3];
                    F[0][0] = c00;
                    F[1][0] = c01;
                    F[2][0] = c02;
                    F[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
                    F[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
                    F[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
                    F[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
                    F[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
                    F[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
#pragma unroll
                    for (int c = 0; c < 3; ++c)
#pragma unroll
                        for (int g = 0; g < 3; ++g) F[c][g] = quotient(F[c][g], det, rd);
                    auto dot = [&](int c, int g) {
                        return (F[c][0] * F[g][0] + F[c][1] * F[g][1]) + F[c][2] * F[g][2];
                    };
                    const double xx = dot(0, 0), yy = dot(1, 1), zz = dot(2, 2);
                    const double xy = dot(0, 1), xz = dot(0, 2), yz = dot(1, 2);
                    const double tr3 = ((xx + yy) + zz) / 3.0;
                    const double tau[6] = {G * (xx - tr3), G * (yy - tr3), G * (zz - tr3),
                                           G * xy, G * xz, G * yz};
                    double* out = a == 0 ? b.tau[0] : (a == 1 ? b.tau[1] : b.tau[2]);
                    const int64_t pf = a == 0 ? nf[0] : (a == 1 ? nf[1] : nf[2]);
                    const int64_t p0 = a == 0 ? f0[0] : b.grid[0], p1 = a == 1 ? f1[1] : b.grid[1];
                    out += ((int64_t)(o[2] + z) * p1 + o[1] + y) * p0 + o[0] + x;
                    if (many) {   // uniform
                        const double sum = s_sum[a][q];
                        s_sum[a][q] = sum == -1.0 ? w : sum + w;
#pragma unroll
                        for (int c = 0; c < 6; ++c)
                            out[c * pf] = sum == -1.0 ? w * tau[c] : out[c * pf] + w * tau[c];
                    } else {
                        double v[6];
#pragma unroll
                        for (int c = 0; c < 6; ++c) v[c] = w * tau[c];
                        if (w > 1.0)   // by rounding, close to phi = -eps
#pragma unroll
                            for (int c = 0; c < 6; ++c) v[c] = v[c] / w;
#pragma unroll
                        for (int c = 0; c < 6; ++c) out[c * pf] = v[c];
                    }
                }
            }
        }
        if (many) {
            __syncthreads();
            for (int j = tid0; j < 3 * kBlurTileCells; j += 256) {
                const int a = j / kBlurTileCells, q = j % kBlurTileCells;
                const double sum = s_sum[a][q];
                if (!(sum > 1.0)) continue;
                const int64_t p0 = a == 0 ? f0[0] : b.grid[0], p1 = a == 1 ? f1[1] : b.grid[1];
                const int64_t pf = a == 0 ? nf[0] : (a == 1 ? nf[1] : nf[2]);
                double* out = (a == 0 ? b.tau[0] : (a == 1 ? b.tau[1] : b.tau[2])) +
                              ((int64_t)(o[2] + (q >> 6)) * p1 + o[1] + ((q >> 3) & 7)) * p0 +
                              o[0] + (q & 7);
#pragma unroll
                for (int c = 0; c < 6; ++c) out[c * pf] = out[c * pf] / sum;
            }
        }
    }
}

}  // namespace

hipError_t launch_blur_heaviside(const BlurBatch& b, hipStream_t st) {
    if (b.n_active <= 0) return hipSuccess;
    hipError_t e;
    if (b.H) {
        hipLaunchKernelGGL(k_blur_fill<false>, dim3(b.fill_blocks), dim3(256), 0, st, b);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_blur_scan<false>, dim3((b.n_active + 3) / 4), dim3(256), 0, st, b);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int g = b.n_active < kBlurFullBlocks ? b.n_active : kBlurFullBlocks;
    if (b.spheres)
        hipLaunchKernelGGL(k_blur_heaviside_spheres, dim3(g), dim3(256), 0, st, b);
    else
        hipLaunchKernelGGL(k_blur_heaviside, dim3(g), dim3(kHeavisideThreads), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_blur_stress(const BlurBatch& b, hipStream_t st) {
    if (b.n_active <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_blur_fill<true>, dim3(b.fill_blocks), dim3(256), 0, st, b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_blur_scan<true>, dim3((b.n_active + 3) / 4), dim3(256), 0, st, b);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int g = b.n_active < kBlurFullBlocks ? b.n_active : kBlurFullBlocks;
    if (b.spheres)
        hipLaunchKernelGGL(k_blur_stress<true>, dim3(g), dim3(256), 0, st, b);
    else
        hipLaunchKernelGGL(k_blur_stress<false>, dim3(g), dim3(256), 0, st, b);
    return hipGetLastError();
}

}  // namespace rmx
