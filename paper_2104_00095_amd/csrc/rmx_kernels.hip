// HIP kernels of the reference-map band extrapolation (Lin, Derr & Rycroft, arXiv
// 2104.00095, section "Extrapolation of xi(x,t)"; SI "Weighting scheme for weighted least
// squares-based extrapolation", eq. (weight)).  One call is a chain of L + 3 launches,
// each covering every solid of the batch:
//   k_classify  streams xi once (coalesced) and packs the interior predicate
//               phi0(xi) < 0 into a 1-bit mask (wave ballots); zeroes the call's counters.
//   k_label     per 16 x 16-row tile: L bit-parallel dilations in LDS, each on the rows
//               still able to reach the tile, give the layers (first dilation reaching a
//               cell = its layer), written as int8 labels; the tile counts its interior
//               and band cells, detects a band truncated by a box face, and lists the 8^3
//               bricks holding cells of each layer (64 buckets per layer).
//   k_normal    sums the tile counts per solid; copies each layer's bucketed brick list
//               into a dense list with its count; per listed brick of layers
//               1..normal_layers, evaluates phi0(xi) once per needed cell (LDS) and forms
//               the normals of the brick's cells of that layer by central differences, from
//               the field before any write.
//   k_extrap    one launch per layer, ascending: a block stages a listed brick with a
//               halo of r_s (12^3 cells: the labels as row bits, then xi where a fit reads
//               it) in LDS; a group of 4, 8 or 16 lanes per cell of the layer (as many as
//               keep the brick's cells in one pass) gathers the (2r+1)^3 box from LDS,
//               accumulates the 4x4 normal-equation moments, reduces them by DPP moves,
//               decides degeneracy by the pivots where they are far from 0 and by an exact
//               integer determinant elsewhere, solves in FP64 and writes xi_e.
// The work is bandwidth- and latency-bound, with 4x4 systems per cell: no MFMA.
#include "rmx_device.h"

namespace rmx {
namespace {
using namespace dev;

// ------------------------------------------------------------------------------------
// Classification of mask words [wb, we) of solid d by the 4 waves of the block: each wave
// streams its 4 consecutive 64-cell row segments, ballot-packs the interior predicate
// and writes one mask word per segment (the wave's words in one store).  Cells past the
// row end (x >= n0) are never interior.
//
// Sphere: the components are read in turn, each only where the decision is still open,
// which leaves it unchanged: the test is ((dx*dx + dy*dy) + dz*dz) < R*R, and in
// round-to-nearest a sum of non-negative terms is never below any of its partial sums,
// so dx*dx >= R*R, or dx*dx + dy*dy >= R*R, already means "not interior" (a non-finite
// component fails its test as well, as in the full predicate).  The running sum is all a
// lane keeps, so a wave issues each component's 4 loads at once.  Ellipsoid: the body
// coordinates need all three components, read together.
// ------------------------------------------------------------------------------------
constexpr int kWaveWords = kChunkWords / 4;   // 4 segments per wave
constexpr int kSegE = 4;                       // ellipsoid: segments per batch

__device__ __forceinline__ void classify_sphere(DevSolidC* dp, const ShapeR& sh, int wb,
                                                int we) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const int wave = uniform_int(threadIdx.x >> 6);
    const int n0 = dp->n0, W = dp->W;
    const int64_t ncell = dp->ncell;
    const double* __restrict__ xi = dp->xi;
    unsigned long long* __restrict__ mask = dp->mask;
    const double T = sh.e0 * sh.e0;
    const int w0 = wb + wave * kWaveWords;
    if (w0 >= we) return;
    int row = w0 / W, wx = w0 - row * W;
    int32_t c[kWaveWords];
    double p[kWaveWords];
#pragma unroll
    for (int u = 0; u < kWaveWords; ++u) {
        const int x = wx * 64 + lane;
        c[u] = (w0 + u < we && x < n0) ? row * n0 + x : -1;
        p[u] = __builtin_nan("");
        if (c[u] >= 0) p[u] = xi[c[u]];
        if (++wx == W) {
            wx = 0;
            ++row;
        }
    }
#pragma unroll
    for (int u = 0; u < kWaveWords; ++u) {
        const double dx = p[u] - sh.c0;
        p[u] = dx * dx;
    }
#pragma unroll
    for (int u = 0; u < kWaveWords; ++u) {
        double v = __builtin_nan("");
        if (p[u] < T) v = xi[ncell + c[u]];
        const double dy = v - sh.c1;
        p[u] = p[u] + dy * dy;
    }
    unsigned long long mw = 0ull;   // lane u keeps mask word u
#pragma unroll
    for (int u = 0; u < kWaveWords; ++u) {
        double v = __builtin_nan("");
        if (p[u] < T) v = xi[2 * ncell + c[u]];
        const double dz = v - sh.c2;
        const unsigned long long m = __ballot((p[u] + dz * dz) < T);
        if (lane == u) mw = m;
    }
    if (lane < kWaveWords && w0 + lane < we) mask[w0 + lane] = mw;   // one store
}

__device__ __forceinline__ void classify_ellipsoid(DevSolidC* dp, const ShapeR& sh, int wb,
                                                   int we) {
    const int lane = threadIdx.x & 63;
    const int wave = uniform_int(threadIdx.x >> 6);
    const int n0 = dp->n0, W = dp->W;
    const int64_t ncell = dp->ncell;
    const double* __restrict__ xi = dp->xi;
    unsigned long long* __restrict__ mask = dp->mask;
    const int first = wb + wave * kWaveWords;
    // (semi-axes far from 1: reciprocals might leave the range)
    const bool usual = near_one(sh.e0) && near_one(sh.e1) && near_one(sh.e2);
    const double r0 = 1.0 / sh.e0, r1 = 1.0 / sh.e1, r2 = 1.0 / sh.e2;
#pragma unroll 1
    for (int it = 0; it < kWaveWords; it += kSegE) {
        const int w0 = first + it;
        if (w0 >= we) break;
        int row = w0 / W, wx = w0 - row * W;
        double v0[kSegE], v1[kSegE], v2[kSegE];
#pragma unroll
        for (int u = 0; u < kSegE; ++u) {
            const int x = wx * 64 + lane;
            v0[u] = v1[u] = v2[u] = __builtin_nan("");
            if (w0 + u < we && x < n0) {
                const int64_t c = (int64_t)row * n0 + x;
                v0[u] = __builtin_nontemporal_load(xi + c);
                v1[u] = __builtin_nontemporal_load(xi + ncell + c);
                v2[u] = __builtin_nontemporal_load(xi + 2 * ncell + c);
            }
            if (++wx == W) {
                wx = 0;
                ++row;
            }
        }
#pragma unroll
        for (int u = 0; u < kSegE; ++u) {
            // the form with reciprocals is within 1e-14 of the one with quotients: it decides
            // all but the points within 1e-9 of the surface (and those that are not finite);
            // 40 ellipsoids 22 -> 18 us, bound by the reads from there on
            double y0, y1, y2;
            body(sh, v0[u], v1[u], v2[u], y0, y1, y2);
            const double q0 = y0 * r0, q1 = y1 * r1, q2 = y2 * r2;
            const double F = (q0 * q0 + q1 * q1) + q2 * q2;
            bool in = usual && F < 1.0 - 1e-9;
            if (!(in || (usual && F > 1.0 + 1e-9))) in = interior(sh, v0[u], v1[u], v2[u]);
            const unsigned long long m = __ballot(in);
            if (lane == 0 && w0 + u < we) mask[w0 + u] = m;
        }
    }
}

__device__ __forceinline__ void classify_words(DevSolidC* dp, int wb, int we) {
    const ShapeR sh = load_shape(dp);
    if (sh.kind == 1)
        classify_sphere(dp, sh, wb, we);
    else
        classify_ellipsoid(dp, sh, wb, we);
}

// A block owns a chunk of kChunkWords mask words of one solid.  Block 0 also zeroes the
// call's statistics and brick counters, which nothing else touches before the labels.
__global__ __launch_bounds__(256) void k_classify(Batch b) {
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < b.n_solids * kStatWords; i += 256) b.stats[i] = 0ull;
        for (int i = threadIdx.x; i < kMaxLayers * kBuckets; i += 256) b.bcount[i] = 0;
        const int nctl = (int)(sizeof(BandCtl) / sizeof(int));
        for (int i = threadIdx.x; i < nctl; i += 256) reinterpret_cast<int*>(b.band)[i] = 0;
    }
    for (int chunk = blockIdx.x; chunk < b.n_chunks; chunk += gridDim.x) {
        const int s = find_solid_by_chunk(b.solids, b.n_solids, chunk);
        DevSolidC* dp = const_solid(b.solids, s);
        const int nwords = dp->n1 * dp->n2 * dp->W;
        const int first = (chunk - dp->chunk_base) * kChunkWords;
        classify_words(dp, first, min(first + kChunkWords, nwords));
    }
}

// ------------------------------------------------------------------------------------
// Labels of one tile of 16 (y) x 16 (z) rows x tile_w 64-cell words (x), by a block of
// 512 threads: threads i and i + 256 own row (tj, tk) = (i % 16, i / 16) of the tile, the
// first the low half of its words, the second the high half (with one word, the first
// all of it).  The region in LDS carries a halo of L rows in y and z and
// one word on each side in x where the box continues (L <= 16 < 64), so after L dilations
// through face neighbours (64-bit shifts and ORs) the tile is exact; dilation l is formed
// only on the rows within L - l of the tile, the only ones later dilations read.  Counts
// go to LDS by atomics, one wave appends the tile's bricks with one round of global
// atomics for all layers, and the labels go through an LDS transpose: whole 128-byte rows
// per store instruction in full-width tiles, aligned 4-byte words elsewhere.
// ------------------------------------------------------------------------------------
constexpr int kLabelThreads = 512;
constexpr int kRowsPerThread =      // region rows per thread at most: (16 + 2 * 16)^2 rows
    ((kTileJ + 2 * kMaxLayers) * (kTileK + 2 * kMaxLayers) + kLabelThreads - 1) / kLabelThreads;

// Label bytes of the 8 cells at bits 8g..8g+7 of a row word: the layer (bit planes
// p0..p4 hold its bits) where the cell was reached, 0xFF where not.  Bit q of a plane's
// nibble goes to bit 8q + k of a 32-bit half by one product (the partial products of
// nibble * (1 + 2^7 + 2^14 + 2^21) never overlap, and the shift by the plane k is folded
// into the constants); a cell not reached has no plane bit.  NP planes are read: layers
// below 2^NP.
template <int NP>
__device__ __forceinline__ unsigned long long label_word(
    unsigned long long p0, unsigned long long p1, unsigned long long p2, unsigned long long p3,
    unsigned long long p4, unsigned long long reached, int sh8) {
    const unsigned long long pl[5] = {p0, p1, p2, p3, p4};
    uint32_t lo = 0u, hi = 0u;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const uint32_t b = (uint32_t)(pl[k] >> sh8) & 255u;
        lo |= ((b & 15u) * (0x00204081u << k)) & (0x01010101u << k);
        hi |= ((b >> 4) * (0x00204081u << k)) & (0x01010101u << k);
    }
    const uint32_t u = (uint32_t)(~reached >> sh8) & 255u;
    lo |= (((u & 15u) * 0x00204081u) & 0x01010101u) * 0xFFu;
    hi |= (((u >> 4) * 0x00204081u) & 0x01010101u) * 0xFFu;
    return ((unsigned long long)hi << 32) | lo;
}

// The sum over the wave (every lane active): DPP sums within each row of 16 lanes (every
// lane of a row ends with the row's sum), then the four rows' sums read out.
__device__ __forceinline__ int wave_sum(int v) {
    v += dpp_i<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_i<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_i<0x141>(v);   // row_half_mirror
    v += dpp_i<0x140>(v);   // row_mirror
    return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
           (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}

template <int N>
struct IntC {
    static constexpr int value = N;
};

// Brick r of a tile's layer-l flags (r = brick row pair * 8 * MAXTW + 8 w + g).
template <int MAXTW>
__device__ __forceinline__ bool brick_flag(const unsigned int* s_bmask, int l, int r) {
    return (s_bmask[(l - 1) * 4 + r / (8 * MAXTW)] >> (r % (8 * MAXTW))) & 1u;
}

// Bytes value(r, x) of the cells of a tile (row r = tk * kTileJ + tj, column x of the nx
// from the tile's first column xs) into dst, a box array, by the whole block; quad(r, x)
// gives the four bytes x..x+3 of row r at once.  The tile's bytes form runs: one per plane
// when it spans whole box rows (its rows of a plane are contiguous), else one per row.
// Thread i takes aligned 4-byte slot i of the runs' slots: one word store where the slot
// lies inside one row of its run, byte stores at a run's ends and across two rows.
template <typename F, typename Q>
__device__ __forceinline__ void store_tile_bytes(int8_t* dst, DevSolidC* d, int xs, int nx,
                                                 int j0, int k0, F value, Q quad) {
    const int n0 = d->n0, n1 = d->n1, n2 = d->n2;
    const int nj = min(kTileJ, n1 - j0), nk = min(kTileK, n2 - k0);
    const bool whole = xs == 0 && nx == n0;
    const int len = whole ? nj * n0 : nx;   // bytes per run
    const int nrun = whole ? nk : nk * nj;
    const int U = (len + 3) / 4 + 1;        // aligned slots a run touches, at most
    for (int i = threadIdx.x; i < nrun * U; i += blockDim.x) {
        const int u = i / U, slot = i - u * U;
        const int tk = whole ? u : u / nj, tj0 = whole ? 0 : u - (u / nj) * nj;
        int8_t* run = dst + ((int64_t)(k0 + tk) * n1 + (j0 + tj0)) * n0 + xs;
        const int q0 = 4 * slot - (int)(reinterpret_cast<uintptr_t>(run) & 3u);
        if (q0 >= len) continue;
        const int qs = q0 < 0 ? 0 : q0;
        const int tj = whole ? qs / n0 : 0;   // row within the run, and column
        int r = tk * kTileJ + tj0 + tj, x = qs - tj * (whole ? n0 : 0);
        if (q0 >= 0 && q0 + 4 <= len && x + 4 <= nx) {
            *reinterpret_cast<uint32_t*>(run + q0) = quad(r, x);
            continue;
        }
        for (int q = qs; q < q0 + 4 && q < len; ++q) {
            run[q] = (int8_t)value(r, x);
            if (++x == nx) {
                x = 0;
                ++r;
            }
        }
    }
}

// Labels of a tile with no layer cell: -1 everywhere (and decision 0).  Whole-width tiles
// with 16-byte aligned rows store 16-byte chunks, consecutive threads on consecutive
// chunks of a row; other tiles go through the block's word stores.
template <int MAXTW>
__device__ __forceinline__ void label_tile_empty(DevSolidC* d, int wx0, int tw, int j0,
                                                 int k0) {
    const int tid = threadIdx.x;
    const int n0 = d->n0, n1 = d->n1, n2 = d->n2;
    const int xs = wx0 * 64, nx = min(64 * tw, n0 - xs);
    const bool wide = nx == 64 * MAXTW && (n0 & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(d->labels) & 15) == 0 &&
                      (!d->decisions || (reinterpret_cast<uintptr_t>(d->decisions) & 15) == 0);
    if (wide) {
        constexpr int CPR = 4 * MAXTW;   // 16-byte chunks per row
        const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u), zero = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int h = 0; h < 256 * CPR / kLabelThreads; ++h) {
            const int c = tid + kLabelThreads * h;
            const int row = c / CPR, off = c % CPR;
            const int jj = j0 + row % kTileJ, kk = k0 + row / kTileJ;
            if (jj < n1 && kk < n2) {
                const int64_t o = ((int64_t)kk * n1 + jj) * n0 + xs + 16 * off;
                *reinterpret_cast<uint4*>(d->labels + o) = ones;
                if (d->decisions) *reinterpret_cast<uint4*>(d->decisions + o) = zero;
            }
        }
        return;
    }
    store_tile_bytes(d->labels, d, xs, nx, j0, k0, [](int, int) { return 0xFFu; },
                     [](int, int) { return 0xFFFFFFFFu; });
    if (d->decisions)
        store_tile_bytes(d->decisions, d, xs, nx, j0, k0, [](int, int) { return 0u; },
                         [](int, int) { return 0u; });
}

// i / n for 0 <= i < 4096 and n >= 1, from inv = 1.0f / n: (i + 1/2) / n is at least 1 / 2n
// from a whole number, far above its rounding.
__device__ __forceinline__ int quotient_by(int i, float inv) {
    return (int)(((float)i + 0.5f) * inv);
}

// Word w of a row's words c, dilated by one cell along x.
template <int MW>
__device__ __forceinline__ unsigned long long x_dilated(const unsigned long long* c, int w) {
    const unsigned long long left = w > 0 ? c[w - 1] : 0ull;
    const unsigned long long right = w < MW - 1 ? c[w + 1] : 0ull;
    return c[w] | (c[w] << 1) | (c[w] >> 1) | (left >> 63) | (right << 63);
}

// The OR of word idx over a row and its eight neighbour rows (stride RS, planes RS * RJ).
__device__ __forceinline__ unsigned long long cube_rows(const unsigned long long* A, int idx,
                                                        int RS, int RJ) {
    unsigned long long v = 0ull;
#pragma unroll
    for (int dk = -1; dk <= 1; ++dk)
#pragma unroll
        for (int dj = -1; dj <= 1; ++dj) v |= A[idx + dj * RS + dk * RS * RJ];
    return v;
}

template <int MAXTW>
__global__ __launch_bounds__(kLabelThreads) void k_label(Batch b) {
    constexpr int FPL = 4 * 8 * MAXTW;   // brick flags per layer: 2 (y) x 2 (z) x 8 per word
    constexpr int MW = MAXTW + 2;        // region words per row at most
    constexpr int WPH = MAXTW > 1 ? MAXTW / 2 : 1;   // row words per owning thread
    HIP_DYNAMIC_SHARED(double, lds_d)
    unsigned long long* lds = reinterpret_cast<unsigned long long*>(lds_d);
    __shared__ int s_cnt[kLT];
    __shared__ int s_trunc;
    __shared__ unsigned int s_bmask[kMaxLayers * 4];   // bricks holding layer-l cells:
                                                        // [l-1][2 x 2 brick rows], bit 8w + g

    const int t = blockIdx.x;
    const int s = load_const(b.tile_solid + t);
    DevSolidC* d = const_solid(b.solids, s);
    unsigned long long* st = b.stats + (int64_t)s * kStatWords;
    const int tid = threadIdx.x;
    const int n0 = d->n0, n1 = d->n1, n2 = d->n2, W = d->W, L = d->L;
    const int lt = t - d->tile_base;
    const int txi = lt % d->ntx;
    const int tyi = (lt / d->ntx) % d->ty;
    const int tzi = lt / (d->ntx * d->ty);
    const int wx0 = txi * MAXTW, tw = min(MAXTW, W - wx0);
    const int xr0 = max(0, wx0 - 1), xr1 = min(W, wx0 + tw + 1);
    const int RW = xr1 - xr0;
    const int RS = RW | 1;   // row stride in words: odd, so that rows fall on distinct banks
    const int j0 = tyi * kTileJ, k0 = tzi * kTileK;
    const int RJ = kTileJ + 2 * L, RK = kTileK + 2 * L;
    const int R = RJ * RK;
    unsigned long long* A = lds;
    unsigned long long* B = lds + (size_t)RS * R;
    const unsigned long long tail = (n0 & 63) ? ((1ull << (n0 & 63)) - 1ull) : ~0ull;
    const unsigned long long* __restrict__ mask = d->mask;

    for (int q = tid; q < L * 4; q += kLabelThreads) s_bmask[q] = 0u;
    if (tid < kLT) s_cnt[tid] = 0;
    if (tid == 0) s_trunc = 0;
    // The mask rows of the region (rows outside the box: empty).  Every load of the
    // thread is issued into registers before the first LDS store, so they overlap instead
    // of each waiting for the previous one.
    unsigned long long mv[kRowsPerThread][MW];
    unsigned long long any = 0ull;
    const float inv_rj = 1.0f / (float)RJ;
#pragma unroll
    for (int q = 0; q < kRowsPerThread; ++q) {
        const int rr = tid + kLabelThreads * q;
        const int rk = quotient_by(rr, inv_rj), rj = rr - rk * RJ;
        const int jj = j0 - L + rj, kk = k0 - L + rk;
        const bool ok = rr < R && jj >= 0 && jj < n1 && kk >= 0 && kk < n2;
        const int64_t base = ok ? ((int64_t)kk * n1 + jj) * W + xr0 : 0;
#pragma unroll
        for (int w = 0; w < MW; ++w) {
            mv[q][w] = (ok && w < RW) ? mask[base + w] : 0ull;
            any |= mv[q][w];
        }
    }
    // A tile whose whole region holds no interior cell has no layer cell either: its
    // labels are all -1 (decisions 0), its counts 0, and it lists no brick.
    if (!__syncthreads_or(any != 0ull)) {
        if (tid <= L) b.tile_cnt[(int64_t)t * kLT + tid] = 0;
        label_tile_empty<MAXTW>(d, wx0, tw, j0, k0);
        return;
    }
#pragma unroll
    for (int q = 0; q < kRowsPerThread; ++q) {
        const int rr = tid + kLabelThreads * q;
        if (rr < R) {
#pragma unroll
            for (int w = 0; w < MW; ++w)
                if (w < RW) A[rr * RS + w] = b.adj26 ? x_dilated<MW>(mv[q], w) : mv[q][w];
        }
    }
    __syncthreads();

    const int row = tid & 255, wb = (tid >> 8) * WPH;   // the row; its first owned word
    const int tj = row % kTileJ, tk = row / kTileJ;
    const int jrow = j0 + tj, krow = k0 + tk;
    const bool row_ok = jrow < n1 && krow < n2;
    const int my = ((tk + L) * RJ + (tj + L)) * RS + (wx0 - xr0) + wb;
    // owned words wb + w, w < WPH (none past the tile)
    unsigned long long prev[WPH], p0[WPH], p1[WPH], p2[WPH], p3[WPH], p4[WPH];
    int cnt0 = 0;
    bool trunc = false;
#pragma unroll
    for (int w = 0; w < WPH; ++w) {
        prev[w] = 0ull;
        if (row_ok && wb + w < tw)   // (the 26-neighbour form keeps dilated rows in A)
            prev[w] = b.adj26 ? load_global(mask + ((int64_t)krow * n1 + jrow) * W + wx0 + wb + w)
                              : A[my + w];
        p0[w] = p1[w] = p2[w] = p3[w] = p4[w] = 0ull;
        cnt0 += __popcll(prev[w]);
        // An interior cell closer than L to a box face that is no grid wall: the band
        // would leave the box (reported; the solid's band is then not fitted).
        if (prev[w]) {
            const int x0 = (wx0 + wb + w) * 64;
            if (!d->wall_lo[0] && x0 < L) {
                const int nb = min(64, L - x0);
                trunc |= (prev[w] & (nb == 64 ? ~0ull : ((1ull << nb) - 1ull))) != 0ull;
            }
            if (!d->wall_hi[0] && x0 + 63 >= n0 - L) {
                const int f = max(0, n0 - L - x0);
                trunc |= (prev[w] & (~0ull << f)) != 0ull;
            }
            trunc |= (!d->wall_lo[1] && jrow < L) || (!d->wall_hi[1] && jrow >= n1 - L) ||
                     (!d->wall_lo[2] && krow < L) || (!d->wall_hi[2] && krow >= n2 - L);
        }
    }
    // counts: wave sums, then one LDS atomic per wave
    const int lane = tid & 63;
    cnt0 = wave_sum(cnt0);
    if (lane == 0 && cnt0) atomicAdd(&s_cnt[0], cnt0);
    if (trunc) s_trunc = 1;

    const int by2 = (tk >> 3) * 2 + (tj >> 3);   // which of the tile's 2 x 2 brick rows
    for (int l = 1; l <= L; ++l) {
        // One dilation step through face neighbours (or, with the 26-neighbour adjacency,
        // through every cell of the 3^3 cube), A -> B, over the rows that can still reach
        // the tile: D_l is needed only within L - l rows of it, i.e. on region rows
        // [l, RJ - l) x [l, RK - l) (their neighbours lie inside the region).  The cube's
        // dilation is the x-dilated rows' OR over 3 x 3 rows, so its form keeps the rows
        // x-dilated: 9 LDS reads per word (25 of the plain rows took 42 us on three ragged
        // boxes, this 37 us), and forms D_l itself for the tile's rows only.
        const unsigned long long* __restrict__ Ar = A;
        unsigned long long* __restrict__ Br = B;
        const int SJ = RJ - 2 * l, S = b.adj26 && l == L ? 0 : SJ * (RK - 2 * l);
        const float inv_sj = 1.0f / (float)SJ;
        for (int i = tid; i < S; i += kLabelThreads) {
            const int ik = quotient_by(i, inv_sj), rk = l + ik, rj = l + i - ik * SJ;
            const int jj = j0 - L + rj, kk = k0 - L + rk;
            const bool rok = jj >= 0 && jj < n1 && kk >= 0 && kk < n2;
            const int base = (rk * RJ + rj) * RS;
            unsigned long long c[MW];
            if (!b.adj26) {
#pragma unroll
                for (int w = 0; w < MW; ++w) c[w] = w < RW ? Ar[base + w] : 0ull;
#pragma unroll
                for (int w = 0; w < MW; ++w) {
                    if (w >= RW) break;
                    const int idx = base + w;
                    const unsigned long long v = x_dilated<MW>(c, w) | Ar[idx - RS] |
                                                 Ar[idx + RS] | Ar[idx - RS * RJ] |
                                                 Ar[idx + RS * RJ];
                    const unsigned long long vm = !rok ? 0ull : (xr0 + w == W - 1 ? tail : ~0ull);
                    Br[idx] = v & vm;
                }
            } else {
#pragma unroll
                for (int w = 0; w < MW; ++w) {
                    const unsigned long long vm = !rok ? 0ull : (xr0 + w == W - 1 ? tail : ~0ull);
                    c[w] = w < RW ? cube_rows(Ar, base + w, RS, RJ) & vm : 0ull;
                }
#pragma unroll
                for (int w = 0; w < MW; ++w)
                    if (w < RW) Br[base + w] = x_dilated<MW>(c, w);
            }
        }
        unsigned long long dcube[WPH];
        if (b.adj26) {
#pragma unroll
            for (int w = 0; w < WPH; ++w)
                dcube[w] = row_ok && wb + w < tw ? cube_rows(Ar, my + w, RS, RJ) &
                                                       (wx0 + wb + w == W - 1 ? tail : ~0ull)
                                                 : 0ull;
        }
        __syncthreads();
        unsigned long long* tmp = A;
        A = B;
        B = tmp;
        int cnt = 0;
        unsigned int fl = 0u;   // bricks of this row holding a layer-l cell: bit 8w + g
#pragma unroll
        for (int w = 0; w < WPH; ++w) {
            const unsigned long long dl =
                b.adj26 ? dcube[w] : (row_ok && wb + w < tw ? A[my + w] : 0ull);
            const unsigned long long nw = dl & ~prev[w];
            prev[w] = dl;
            if (l & 1) p0[w] |= nw;
            if (l & 2) p1[w] |= nw;
            if (l & 4) p2[w] |= nw;
            if (l & 8) p3[w] |= nw;
            if (l & 16) p4[w] |= nw;
            cnt += __popcll(nw);
#pragma unroll
            for (int g = 0; g < 8; ++g)
                if ((nw >> (8 * g)) & 255ull) fl |= 1u << ((wb + w) * 8 + g);
        }
        // Wave sums of the counts; the flags ORed over the lanes of each brick row pair (a
        // wave's lanes share tk >> 3, lane bit 3 is tj >> 3): then lane 0's LDS atomics.
        cnt = wave_sum(cnt);
        fl |= dpp_i<0xB1>((int)fl);    // quad_perm [1,0,3,2]
        fl |= dpp_i<0x4E>((int)fl);    // quad_perm [2,3,0,1]
        fl |= dpp_i<0x141>((int)fl);   // row_half_mirror: the OR over each 8 lanes
        const unsigned int f0 = (unsigned)(__builtin_amdgcn_readlane((int)fl, 0) |
                                           __builtin_amdgcn_readlane((int)fl, 16) |
                                           __builtin_amdgcn_readlane((int)fl, 32) |
                                           __builtin_amdgcn_readlane((int)fl, 48));
        const unsigned int f1 = (unsigned)(__builtin_amdgcn_readlane((int)fl, 8) |
                                           __builtin_amdgcn_readlane((int)fl, 24) |
                                           __builtin_amdgcn_readlane((int)fl, 40) |
                                           __builtin_amdgcn_readlane((int)fl, 56));
        if (lane == 0) {
            if (cnt) atomicAdd(&s_cnt[l], cnt);
            if (f0) atomicOr(&s_bmask[(l - 1) * 4 + (by2 & ~1)], f0);
            if (f1) atomicOr(&s_bmask[(l - 1) * 4 + (by2 | 1)], f1);
        }
    }
    __syncthreads();   // counts, flags and the last step complete; A/B free
    if (tid <= L) b.tile_cnt[(int64_t)t * kLT + tid] = s_cnt[tid];
    if (tid == 0 && s_trunc) atomicOr(st + ST_FLAGS, FLAG_TRUNCATED);

    // Bricks holding cells of each layer, appended to the layer's list in this tile's
    // bucket: wave 0 counts every layer, reserves all layers' slots with one round of
    // atomics, and writes the entries last, when they have returned.  A brick lies in exactly
    // one tile, so a tile lists at most FPL bricks per layer and its bucket never overflows.
    const int bk = t % kBuckets;
    int mybase = 0;
    if (tid < 64) {   // (lane == tid)
        int mytot = 0;   // lane l - 1: bricks of layer l
        for (int l = 1; l <= L; ++l) {
            int tot = 0;
            for (int f0 = 0; f0 < FPL; f0 += 64)
                tot += __popcll(__ballot(f0 + lane < FPL && brick_flag<MAXTW>(s_bmask, l, f0 + lane)));
            if (lane == l - 1) mytot = tot;
        }
        if (lane < L && mytot > 0) mybase = atomicAdd(b.bcount + lane * kBuckets + bk, mytot);
    }

    // Labels: byte = layer where the cell was reached, 0xFF where not.  Each thread forms
    // its row's label words in LDS; full-width tiles with aligned rows then store whole
    // 128-byte rows per store instruction, other tiles go through the block's word stores.
    constexpr int TS = 8 * MAXTW + 1;   // padded row stride: rows on distinct banks
    unsigned long long* T = lds;         // [256 rows][TS] label words
    {
        // the planes the layers 1..L use (L uniform: one branch per tile)
        auto fill = [&](auto np) {
            constexpr int NP = decltype(np)::value;
#pragma unroll
            for (int w = 0; w < WPH; ++w) {
                if (wb + w >= MAXTW) break;   // (the second thread of a one-word row)
#pragma unroll
                for (int g = 0; g < 8; ++g)
                    T[row * TS + (wb + w) * 8 + g] =
                        label_word<NP>(p0[w], p1[w], p2[w], p3[w], p4[w], prev[w], 8 * g);
            }
        };
        if (L < 8)
            fill(IntC<3>{});
        else
            fill(IntC<5>{});
    }
    __syncthreads();
    const bool full = tw == MAXTW && (wx0 + MAXTW) * 64 <= n0 && (n0 & 7) == 0 &&
                      (reinterpret_cast<uintptr_t>(d->labels) & 7) == 0 &&
                      (!d->decisions || (reinterpret_cast<uintptr_t>(d->decisions) & 7) == 0);
    if (full) {   // uniform
        constexpr int CPR = 8 * MAXTW;   // 8-byte chunks per tile row
#pragma unroll
        for (int h = 0; h < 256 * CPR / kLabelThreads; ++h) {
            const int ch = tid + kLabelThreads * h;
            const int row = ch / CPR, off = ch % CPR;   // row = tk * 16 + tj
            const int rj = j0 + row % kTileJ, rk = k0 + row / kTileJ;
            if (rj < n1 && rk < n2) {
                const int64_t o = ((int64_t)rk * n1 + rj) * n0 + wx0 * 64 + 8 * off;
                reinterpret_cast<unsigned long long*>(d->labels + o)[0] = T[row * TS + off];
                if (d->decisions) reinterpret_cast<unsigned long long*>(d->decisions + o)[0] = 0ull;
            }
        }
    } else {
        const int xs = wx0 * 64, nx = min(64 * tw, n0 - xs);
        const uint8_t* Tb = reinterpret_cast<const uint8_t*>(T);
        const uint32_t* Tw = reinterpret_cast<const uint32_t*>(T);
        // four bytes of a row from the two aligned words holding them (a row's padding word
        // lies past its last byte)
        auto quad = [&](int r, int x) {
            const int o = r * TS * 8 + x;
            const unsigned long long two =
                ((unsigned long long)Tw[(o >> 2) + 1] << 32) | Tw[o >> 2];
            return (uint32_t)(two >> (8 * (o & 3)));
        };
        store_tile_bytes(d->labels, d, xs, nx, j0, k0,
                         [&](int r, int x) { return (uint32_t)Tb[r * TS * 8 + x]; }, quad);
        if (d->decisions)
            store_tile_bytes(d->decisions, d, xs, nx, j0, k0, [](int, int) { return 0u; },
                             [](int, int) { return 0u; });
    }
    if (tid < 64) {
        const int64_t base0 = bucket_base(bk, b.n_tiles, b.tile_w);
        const int64_t cap = bucket_base(bk + 1, b.n_tiles, b.tile_w) - base0;
        for (int l = 1; l <= L; ++l) {
            const int lbase = __shfl(mybase, l - 1, 64);
            int run = 0;
            for (int f0 = 0; f0 < FPL; f0 += 64) {
                const int r = f0 + lane;
                const bool f = r < FPL && brick_flag<MAXTW>(s_bmask, l, r);
                const unsigned long long bal = __ballot(f);
                if (f) {
                    const int pos = lbase + run + __popcll(bal & ((1ull << lane) - 1ull));
                    const int yz = r / (8 * MAXTW), xb = r % (8 * MAXTW);
                    const int bx = wx0 * 8 + xb, by = 2 * tyi + (yz & 1), bz = 2 * tzi + (yz >> 1);
                    if (pos < cap)
                        b.blist[(int64_t)(l - 1) * b.blist_cap + base0 + pos] =
                            ((unsigned long long)s << 32) |
                            (unsigned long long)(bx | (by << 10) | (bz << 20));
                    else
                        atomicOr(st + ST_FLAGS, FLAG_OVERFLOW);
                }
                run += __popcll(bal);
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// Extrapolation of the layer-l cells of one brick, staged in LDS.
// ------------------------------------------------------------------------------------
// The weights of the radius-2 offsets: entry (|dx| * 3 + |dy|) * 3 + |dz| is
// 2^-(|dx|+|dy|+|dz|) / |(dx rho_x, dy rho_y, dz rho_z)| (eq. (weight) with the spacings of
// the axes); d == nullptr or equal spacings: the same over |d|.
constexpr int kRlen = 27;

__device__ __forceinline__ double rlen_entry(DevSolidC* d, int e) {
    const int ax = e / 9, ay = (e / 3) % 3, az = e % 3;
    if (e == 0) return 0.0;
    const double r = d == nullptr || !d->aniso
                         ? c_rlen[ax * ax + ay * ay + az * az]
                         : 1.0 / norm3((double)ax * d->rho[0], (double)ay * d->rho[1],
                                       (double)az * d->rho[2]);
    return ldexp(r, -(ax + ay + az));
}

// Row sums over the five offsets dx = -2..2 for a 5-bit set of them, with the weights
// w = 2^-|dx|: sum w, sum w dx, sum w dx^2.
constexpr int kRowSets = 32;
struct RowSums {
    double s0, s1, s2;
};
struct RowSumTable {
    RowSums v[kRowSets];
};
constexpr RowSumTable make_row_sums() {
    RowSumTable t{};
    for (int e = 0; e < kRowSets; ++e)
        for (int u = 0; u < 5; ++u) {
            const int dx = u - 2, ad = dx < 0 ? -dx : dx;
            const double w = ((e >> u) & 1) / (double)(1 << ad);
            t.v[e].s0 += w;
            t.v[e].s1 += w * dx;
            t.v[e].s2 += w * dx * dx;
        }
    return t;
}
static __constant__ RowSumTable c_row_sums = make_row_sums();

// Tables of the fits in LDS: the weights (of the solid in `tab`, -1: equal spacings) and
// the row sums.
struct FitTables {
    double* rlen;       // [kRlen]
    RowSums* rows;      // [kRowSets]
};

__device__ __forceinline__ void fill_fit_tables(const FitTables& t) {
    const int tid = threadIdx.x;
    if (tid < kRlen) t.rlen[tid] = rlen_entry(nullptr, tid);
    if (tid < 3 * kRowSets)
        reinterpret_cast<double*>(t.rows)[tid] = reinterpret_cast<const double*>(&c_row_sums)[tid];
}

// LDS of a staged brick (brick_lds_bytes).
template <typename T>
struct BrickLds {
    T* sx;                       // [3][span_cells<T>()] xi - A of the staged cells
    unsigned long long* target;  // [8] cells of the layer in plane y = 2 + i of the region:
                                 // bit 8 k + j is column 2 + j of z = 2 + k
    unsigned* rows;              // [144] the staged rows as the gathers read them
    int* ctl;                    // [0..2] the first datum of the rows of wave 0, 1, 2,
                                 // [3..5] their staged cells, [6] cells listed, [7] a cell
                                 // is left open
    uint16_t* slots;             // [span_cells<T>()] code of each staged cell, | kCellNeeded
    uint16_t* cells;             // [512] the layer's cells
};
template <typename T>
__device__ __forceinline__ BrickLds<T> brick_lds(unsigned char* lds) {
    BrickLds<T> b;
    b.sx = reinterpret_cast<T*>(lds);
    b.target = reinterpret_cast<unsigned long long*>(b.sx + 3 * span_cells<T>());
    b.rows = reinterpret_cast<unsigned*>(b.target + kBrick);
    b.ctl = reinterpret_cast<int*>(b.rows + kBrickSpan * kBrickSpan);
    b.slots = reinterpret_cast<uint16_t*>(b.ctl + 8);
    b.cells = b.slots + span_cells<T>();
    return b;
}
constexpr unsigned kCellNeeded = 0x8000u;   // a staged cell that carries data
constexpr unsigned kCellOpen = 0x8000u;     // a listed cell that its first fit left open

// A staged row as the gathers read it: bits 0..11 the columns that carry data, above them
// the staged place of its column 0 (which itself need not be staged), plus 16.
__device__ __forceinline__ int row_place(unsigned info) { return (int)(info >> 12) - 16; }

// A cell of the 12^3 region in the block's lists: column, row, plane.
__device__ __forceinline__ unsigned cell_code(int x, int y, int z) {
    return (unsigned)(x | (y << 4) | (z << 8));
}
__device__ __forceinline__ int code_x(unsigned c) { return (int)(c & 15u); }
__device__ __forceinline__ int code_y(unsigned c) { return (int)((c >> 4) & 15u); }
__device__ __forceinline__ int code_z(unsigned c) { return (int)((c >> 8) & 15u); }

// The 25 lines (dy, dz) of the radius-2 box, i = 5 (dz + 2) + dy + 2, i / 5 without a division.
__device__ __forceinline__ int line_dz(int i) { return ((i * 13) >> 6) - 2; }
__device__ __forceinline__ int line_dy(int i, int dz) { return i - 5 * dz - 12; }
// The staged row of line i of the cell on staged row `row`.
__device__ __forceinline__ int line_row(int i, int row) {
    return row + i + (kBrickSpan - 5) * ((i * 13) >> 6) - 2 * kBrickSpan - 2;
}

// The columns of line (dy, dz) within radius r (1 or 2), as a 5-bit set.
__device__ __forceinline__ unsigned line_columns(int r, int dy, int dz) {
    return r == kBrickHalo ? 31u : (abs(dy) < 2 && abs(dz) < 2 ? 14u : 0u);
}

// Sums over a cell's data of radius r = 2 (or 1), plain weights w = 2^-(|dx|+|dy|+|dz|).  A lane
// takes every nl-th line of the box around the cell at column x of staged row `row`.  The
// staged values are xi - A for the brick's anchor A, 0 where the cell carries no data, so a
// line's sums over dx need no selection, and the normal matrix depends only on which of its
// five cells carry data: five bits of the row, looked up.  Powers of two scale exactly, so
// factoring the line's weight out changes no rounding, and the matrix is exact.
template <typename T>
__device__ __forceinline__ void gather_plain(const T* __restrict__ sx,
                                             const unsigned* __restrict__ rows,
                                             const RowSums* __restrict__ row_sums, int x,
                                             int row, int r, int lq, int nl, Moments<T>& acc) {
    const T we = r == kBrickHalo ? T(0.25) : T(0);   // the weight of dx = -2 and 2
    unsigned info = rows[line_row(lq, row)];
#pragma unroll 1
    for (int i = lq; i < 25; i += nl) {
        const int dz = line_dz(i), dy = line_dy(i, dz);
        const unsigned bits = (info >> (x - 2)) & line_columns(r, dy, dz);
        const T* p = sx + (row_place(info) + x - 2);
        info = rows[line_row(min(i + nl, 24), row)];   // the next line's, read ahead
        if (bits == 0u) continue;   // no data: the line adds zeros
        const RowSums rs = row_sums[bits];
        const T fy = (T)dy, fz = (T)dz;
        const T w = (T)ldexp(1.0, -(abs(dy) + abs(dz))), wy = fy * w, wz = fz * w;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T* v = p + c * span_cells<T>();
            const T a0 = v[0], a1 = v[1], a2 = v[2], a3 = v[3], a4 = v[4];
            const T t0 = fma(we, a4, fma(T(0.5), a3, a2 + fma(T(0.5), a1, we * a0)));
            const T t1 = fma(T(2) * we, a4, fma(T(0.5), a3, fma(T(-0.5), a1, T(-2) * we * a0)));
            acc.r[c] = fma(w, t0, acc.r[c]);
            acc.r[3 + c] = fma(w, t1, acc.r[3 + c]);
            acc.r[6 + c] = fma(wy, t0, acc.r[6 + c]);
            acc.r[9 + c] = fma(wz, t0, acc.r[9 + c]);
        }
        const T s0 = (T)rs.s0, s1 = (T)rs.s1, s2 = (T)rs.s2;
        acc.m[0] = fma(w, s0, acc.m[0]);
        acc.m[1] = fma(w, s1, acc.m[1]);
        acc.m[2] = fma(wy, s0, acc.m[2]);
        acc.m[3] = fma(wz, s0, acc.m[3]);
        acc.m[4] = fma(w, s2, acc.m[4]);
        acc.m[5] = fma(wy, s1, acc.m[5]);
        acc.m[6] = fma(wz, s1, acc.m[6]);
        acc.m[7] = fma(fy * wy, s0, acc.m[7]);
        acc.m[8] = fma(fz * wy, s0, acc.m[8]);
        acc.m[9] = fma(fz * wz, s0, acc.m[9]);
    }
}

// Adds the offsets dx of a 5-bit set on line (dy, dz) to the integer sums g (as in Moments).
__device__ __forceinline__ void add_offsets(int* g, unsigned set, int dy, int dz) {
    const int ends = __builtin_popcount(set & 17u), mids = __builtin_popcount(set & 10u);
    const int n = __builtin_popcount(set), nxx = mids + 4 * ends;
    const int nx = (__builtin_popcount(set & 24u) + __builtin_popcount(set & 16u)) -
                   (__builtin_popcount(set & 3u) + __builtin_popcount(set & 1u));
    const int ny = mul24(dy, n), nz = mul24(dz, n);
    g[0] += n + (nxx << 16);
    g[1] += nx + (mul24(dy, nx) << 16);
    g[2] += ny + (mul24(dz, nx) << 16);
    g[3] += nz + (mul24(dy, ny) << 16);
    g[4] += mul24(dy, nz) + (mul24(dz, nz) << 16);
}

// The same with the normal factor: 2^-(|dx|+|dy|+|dz|) (x_e - x_d).n / |x_e - x_d| where that
// is positive; the sign is decided on (dx gx + dy gy) + dz gz, in that order, without
// contraction.  In FP64 the weights stay unnormalised (all of a cell's weights share the
// factor rgn = 1/|g|, which cancels in the fit); the FP32 sums take them normalised.
template <typename T>
__device__ __forceinline__ void gather_normal(const T* __restrict__ sx,
                                              const unsigned* __restrict__ rows,
                                              const double* __restrict__ rlen, int x, int row,
                                              double g0, double g1, double g2, double rgn, int r,
                                              int lq, int nl, Moments<T>& acc) {
    unsigned info = rows[line_row(lq, row)];
#pragma unroll 1
    for (int i = lq; i < 25; i += nl) {
        const int dz = line_dz(i), dy = line_dy(i, dz);
        const unsigned bits = (info >> (x - 2)) & line_columns(r, dy, dz);
        const T* p = sx + (row_place(info) + x - 2);
        info = rows[line_row(min(i + nl, 24), row)];   // the next line's, read ahead
        if (bits == 0u) continue;   // no data: the line adds zeros
        const int rowi = abs(dy) * 3 + abs(dz);
        T w[5];
        unsigned pos = 0u;   // the offsets of positive weight
        {
#pragma clang fp contract(off)
            const double ry = (double)dy * g1, rz = (double)dz * g2;
            const double cw[3] = {rlen[rowi], rlen[9 + rowi], rlen[18 + rowi]};
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                const int dx = u - 2;
                const double dot = ((double)dx * g0 + ry) + rz;
                const bool e = ((bits >> u) & 1u) && dot < 0.0;
                double ww = -dot * cw[abs(dx)];
                if (sizeof(T) == 4) ww = ww * rgn;
                w[u] = e ? (T)ww : T(0);
                pos |= e ? 1u << u : 0u;
            }
        }
        const T fy = (T)dy, fz = (T)dz;
        T s0 = T(0), s1 = T(0), s2 = T(0);
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            s0 += w[u];
            if (u != 2) {
                const T wx = (T)(u - 2) * w[u];
                s1 += wx;
                s2 = fma((T)(u - 2), wx, s2);
            }
        }
        acc.m[0] += s0;
        acc.m[1] += s1;
        acc.m[2] = fma(fy, s0, acc.m[2]);
        acc.m[3] = fma(fz, s0, acc.m[3]);
        acc.m[4] += s2;
        acc.m[5] = fma(fy, s1, acc.m[5]);
        acc.m[6] = fma(fz, s1, acc.m[6]);
        acc.m[7] = fma(fy * fy, s0, acc.m[7]);
        acc.m[8] = fma(fy * fz, s0, acc.m[8]);
        acc.m[9] = fma(fz * fz, s0, acc.m[9]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T* v = p + c * span_cells<T>();
            T t0 = T(0), t1 = T(0);
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                t0 = fma(w[u], v[u], t0);
                if (u != 2) t1 = fma((T)(u - 2) * w[u], v[u], t1);
            }
            acc.r[c] += t0;
            acc.r[3 + c] += t1;
            acc.r[6 + c] = fma(fy, t0, acc.r[6 + c]);
            acc.r[9 + c] = fma(fz, t0, acc.r[9 + c]);
        }
        if (sizeof(T) == 4) add_offsets(acc.g, pos, dy, dz);
    }
}

// The exact rank of a staged cell's data: the integer Gram matrix of their offsets (with the
// normal, of those of positive weight, decided as in gather_normal).
__device__ __forceinline__ bool staged_full_rank(const unsigned* rows, int x, int row, int r,
                                                 bool has_normal, double g0, double g1,
                                                 double g2, int lq, int sh) {
    int g[5] = {0, 0, 0, 0, 0};
#pragma unroll 1
    for (int i = lq; i < 25; i += 1 << sh) {
        const int dz = line_dz(i), dy = line_dy(i, dz);
        unsigned set = (rows[line_row(i, row)] >> (x - 2)) & line_columns(r, dy, dz);
        if (has_normal) {
#pragma clang fp contract(off)
            const double ry = (double)dy * g1, rz = (double)dz * g2;
#pragma unroll
            for (int u = 0; u < 5; ++u)
                if (!(((double)(u - 2) * g0 + ry) + rz < 0.0)) set &= ~(1u << u);
        }
        add_offsets(g, set, dy, dz);
    }
    reduce_values<5>(g, sh);
    return det_gram(g) > 0;
}

// What the fits need of the call.
struct FitArgs {
    const DevSolid* solids;
    unsigned long long* stats;
    int normal_layers, r_s, r_max;
};
// A list entry: the solid and the brick's place.
__device__ __forceinline__ int entry_solid(unsigned long long pk) { return (int)(pk >> 32); }
__device__ __forceinline__ int entry_x(unsigned long long pk) { return (int)(pk & 1023ull); }
__device__ __forceinline__ int entry_y(unsigned long long pk) { return (int)((pk >> 10) & 1023ull); }
__device__ __forceinline__ int entry_z(unsigned long long pk) { return (int)((pk >> 20) & 1023ull); }

// What a fit needs of its brick: the box index of the region's cell 0 (which may lie outside
// the box), the row and plane strides, the cells of the box, and the anchor.
struct BrickCtx {
    int ox, oy, oz, origin, n0, n01;
    int64_t nc;
    double A[3];
};
__device__ __forceinline__ int brick_cell(const BrickCtx& c, unsigned q) {
    return c.origin + code_z(q) * c.n01 + code_y(q) * c.n0 + code_x(q);
}

// The open cells of a brick's list.  Where they were fitted from the staged data (`staged`),
// the exact rank test on the staged rows comes first: a cell whose data have full rank keeps
// its value.  The others take the radii from there to r_max with eq. (weight), then F1 (normal factor
// dropped) at r_max, then F2 (kernel-weighted mean) at r_max, gathered from global memory, each
// radius accepted by the exact rank test.  Out of line after the other cells, so that its
// registers are not the fits'; the arguments, which a call passes in vector registers, are made
// uniform again (the descriptor's fields are then scalar loads).  8192 cells of a plate that go
// through every radius and both fallbacks: 297 -> 66 us, 180 of them atomics of a cell each.
template <typename T>
static __device__ __noinline__ void fit_open_cells(FitArgs args, unsigned long long pk_, int l_,
                                                   unsigned char* lds, int sh_, bool staged_,
                                                   double A0_, double A1_, double A2_) {
    const FitArgs b = {uniform_ptr(args.solids), uniform_ptr(args.stats),
                       uniform_int(args.normal_layers), uniform_int(args.r_s),
                       uniform_int(args.r_max)};
    const unsigned long long pk = uniform_word(pk_);
    const int l = uniform_int(l_), sh = uniform_int(sh_);
    const bool staged = uniform_int(staged_);
    const BrickLds<T> B = brick_lds<T>(lds);
    const uint16_t* cells = B.cells;
    const int total = uniform_int(B.ctl[6]);
    const bool nrm = l <= b.normal_layers;
    DevSolidC* d = const_solid(b.solids, entry_solid(pk));
    unsigned long long* st = b.stats + (int64_t)entry_solid(pk) * kStatWords;
    const int ox = kBrick * entry_x(pk) - kBrickHalo, oy = kBrick * entry_y(pk) - kBrickHalo,
              oz = kBrick * entry_z(pk) - kBrickHalo;
    const int lq = threadIdx.x & ((1 << sh) - 1);
    const int64_t nc = d->ncell;
    CellCtx cx;
    cx.n0 = d->n0;
    cx.n1 = d->n1;
    cx.n2 = d->n2;
    cx.le = l;
    cx.ncell = nc;
    cx.xi = d->xi;
    cx.labels = d->labels;
    cx.a0 = uniform_double(A0_);
    cx.a1 = uniform_double(A1_);
    cx.a2 = uniform_double(A2_);
    cx.rho = d->aniso ? (const double*)d->rho : nullptr;
    int tally = 0;   // grown, F1 and F2 cells, ten bits each (an atomic per cell takes 12 ns)
    for (int ci = threadIdx.x >> sh; ci < total; ci += 256 >> sh) {
        const unsigned q = cells[ci];
        if (!(q & kCellOpen)) {   // (the same in every lane of the cell)
            tally += lq == 0 && kBrickHalo > b.r_s;   // fitted at the staged radius
            continue;
        }
        cx.i = ox + code_x(q);
        cx.j = oy + code_y(q);
        cx.k = oz + code_z(q);
        const int32_t cell = (cx.k * cx.n1 + cx.j) * cx.n0 + cx.i;
        cx.g0 = nrm ? load_global(d->normals + cell) : 0.0;
        cx.g1 = nrm ? load_global(d->normals + nc + cell) : 0.0;
        cx.g2 = nrm ? load_global(d->normals + 2 * nc + cell) : 0.0;
        const bool has_normal = cx.g0 != 0.0 || cx.g1 != 0.0 || cx.g2 != 0.0;
        const int dec = nrm && !has_normal ? kDecNoNormal : 0;
        if (staged &&
            staged_full_rank(B.rows, code_x(q), code_z(q) * kBrickSpan + code_y(q), kBrickHalo,
                             has_normal, cx.g0, cx.g1, cx.g2, lq, sh)) {
            if (lq == 0 && d->decisions) d->decisions[cell] = (int8_t)(kBrickHalo + dec);
            tally += lq == 0 && kBrickHalo > b.r_s;
            continue;
        }
        cx.rgn = !has_normal ? 0.0
                 : d->aniso  ? rlen_scaled((const double*)d->irho, cx.g0, cx.g1, cx.g2)
                             : 1.0 / norm3(cx.g0, cx.g1, cx.g2);
        int code = -1;
        double res = 0.0;
        const int comp = min(lq & 3, 2);   // lanes 0..2 of the cell solve and store one each
        for (int r = staged ? kBrickHalo + 1 : b.r_s; code < 0; ++r) {   // r_max + 1: F1, + 2: F2
            const bool f1 = r == b.r_max + 1, f2 = r > b.r_max + 1;
            if (f1 && !has_normal) continue;
            Moments<T> acc;
            zero(acc);
            gather_any<T>(cx, min(r, b.r_max), has_normal && r <= b.r_max, lq, 1 << sh, acc);
            reduce_lanes(acc, sh);
            double R[4];
#pragma unroll
            for (int p = 0; p < 4; ++p)
                R[p] = (double)(comp == 0 ? acc.r[3 * p]
                                          : comp == 1 ? acc.r[3 * p + 1] : acc.r[3 * p + 2]);
            if (f2) {
                res = R[0] / (double)acc.m[0];
                code = kDecF2;
            } else if (det_gram(acc.g) > 0) {
                double M[10];
#pragma unroll
                for (int p = 0; p < 10; ++p) M[p] = (double)acc.m[p];
                res = solve_intercept<T>(M, R[0], R[1], R[2], R[3]).value;
                code = f1 ? kDecF1 : r;
            }
        }
        if (lq < 3)
            d->xi[comp * nc + cell] = (comp == 0 ? cx.a0 : (comp == 1 ? cx.a1 : cx.a2)) + res;
        if (lq == 0) {
            if (d->decisions) d->decisions[cell] = (int8_t)(code + dec);
            tally += (code > b.r_s) + ((code == kDecF1) << 10) + ((code == kDecF2) << 20);
        }
    }
    // (the F codes are larger than any radius; a brick has at most 512 cells)
    tally = wave_sum(tally);
    if ((threadIdx.x & 63) == 0 && tally) {
        atomicAdd(st + ST_GROWN, (unsigned long long)(tally & 1023));
        if ((tally >> 10) & 1023) atomicAdd(st + ST_F1, (unsigned long long)((tally >> 10) & 1023));
        if (tally >> 20) atomicAdd(st + ST_F2, (unsigned long long)(tally >> 20));
    }
}

// The open cells of the list moved to its front, as a list of their own, by one wave.
template <typename T>
static __device__ __noinline__ void keep_open_cells(unsigned char* lds) {
    const BrickLds<T> B = brick_lds<T>(lds);
    const int total = uniform_int(B.ctl[6]), lane = threadIdx.x & 63;
    int n = 0;
    if (threadIdx.x < 64) {
        for (int i = 0; i < total; i += 64) {
            const unsigned q = i + lane < total ? B.cells[i + lane] : 0u;
            const unsigned long long m = __ballot((q & kCellOpen) != 0u);
            if (q & kCellOpen)   // (no place is written before it is read)
                B.cells[n + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(q & ~kCellOpen);
            n += __popcll(m);
        }
    }
    __syncthreads();   // (the others have read ctl[6])
    if (threadIdx.x == 0) B.ctl[6] = n;
    __syncthreads();
}

// The fits of the listed layer-l cells of a staged brick at radius r, 2^sh lanes per cell; a cell whose data may not have full rank is left open (flagged in the list, and
// ctl[7] set).  Values are relative to the brick's anchor A: xi_e = A + the fitted intercept.
// (fn0, fn1, fn2): the normal of the group's first cell, loaded while the brick was staged.
//
// The rank is certain where the elimination's pivots are: the plain weights' matrix is exact,
// and so is, to rounding, the FP64 matrix with the normal factor.  The FP32 one is not, so
// it carries the exact integer Gram matrix of the offsets beside it.
template <typename T, bool kAny>
__device__ __forceinline__ void fit_cells(DevSolidC* d, bool nrm, const BrickCtx& cx, int total,
                                          int sh, int r, const BrickLds<T>& B,
                                          const FitTables& tab, double fn0, double fn1,
                                          double fn2) {
    double* xi = d->xi;
    int8_t* decisions = d->decisions;
    const double* normals = d->normals;
    const int nl = 1 << sh;
    const int grp = threadIdx.x >> sh, lq = threadIdx.x & (nl - 1);
    for (int ci = grp; ci < total; ci += 256 >> sh) {
        const unsigned q = B.cells[ci];
        const int x = code_x(q), row = code_z(q) * kBrickSpan + code_y(q);
        const int cell = brick_cell(cx, q);
        double g0 = fn0, g1 = fn1, g2 = fn2;
        if (nrm && ci != grp) {
            g0 = load_global(normals + cell);
            g1 = load_global(normals + cx.nc + cell);
            g2 = load_global(normals + 2 * cx.nc + cell);
        }
        const bool has_normal = nrm && (g0 != 0.0 || g1 != 0.0 || g2 != 0.0);
        Moments<T> acc;
        zero(acc);
        bool full = true;   // the data have full rank, where the pivots do not tell
        if (has_normal) {
            // the physical gradient is g / rho up to a common factor (1 / h)
            double rgn = 0.0;
            if (sizeof(T) == 4)
                rgn = d->aniso ? rlen_scaled((const double*)d->irho, g0, g1, g2)
                               : 1.0 / norm3(g0, g1, g2);
            gather_normal<T>(B.sx, B.rows, tab.rlen, x, row, g0, g1, g2, rgn, r, lq, nl, acc);
            if (sizeof(T) == 4) {
                reduce_values<5>(acc.g, sh);
                full = det_gram(acc.g) > 0;
            }
        } else {
            gather_plain<T>(B.sx, B.rows, tab.rows, x, row, r, lq, nl, acc);
        }
        reduce_values<10>(acc.m, sh);
        reduce_values<12>(acc.r, sh);
        // lanes 0..2 of the group solve and store a component each
        const int comp = min(lq & 3, 2);
        double M[10], R[4];
#pragma unroll
        for (int p = 0; p < 10; ++p) M[p] = (double)acc.m[p];
#pragma unroll
        for (int p = 0; p < 4; ++p)
            R[p] = (double)(comp == 0 ? acc.r[3 * p]
                                      : comp == 1 ? acc.r[3 * p + 1] : acc.r[3 * p + 2]);
        const Intercept f = solve_intercept<T>(M, R[0], R[1], R[2], R[3]);
        if (lq < 3)
            xi[comp * cx.nc + cell] = (comp == 0 ? cx.A[0] : (comp == 1 ? cx.A[1] : cx.A[2])) +
                                      f.value;
        if (!(sizeof(T) == 4 && has_normal)) full = f.certain;
        if (kAny && r < kBrickHalo && !full)   // (the same in every lane of the cell)
            full = staged_full_rank(B.rows, x, row, r, has_normal, g0, g1, g2, lq, sh);
        if (lq == 0) {
            if (full) {
                if (decisions)
                    decisions[cell] = (int8_t)(r + (nrm && !has_normal ? kDecNoNormal : 0));
            } else {
                B.cells[ci] = (uint16_t)(q | kCellOpen);
                B.ctl[7] = 1;
            }
        }
    }
}

// A brick is bound by the latency of its dependent loads and by the instructions of its
// fits, not by bandwidth.  It takes two round trips: the labels (one 16-byte load per row),
// then xi of the cells that some fit reads -- the data within radius 2 of a cell of the
// layer, about 250 of the region's 1728 -- with the normals of the groups' first cells.
// Staged are, row by row, the columns from the first to the last within radius 2 of a cell
// of the layer (about 650 cells; 0 where they carry no data), so that a gather reads five
// consecutive places of a row and the block's LDS leaves room for four blocks per CU.  A
// brick whose columns exceed the staged places (layers around solids of a few cells; not
// in FP32, whose places hold the whole region) is staged and fitted in two halves along z,
// whose columns always fit, by the same code: a copy of its own for the few blocks that have
// such a brick is fetched cold (8 ellipsoids on 64 x 64 x 96: fits 52 -> 29 us).
//
// Of a block's 13 us on a 256^3 sphere (layers past the normal's; wall-clock stamps) the
// gathers take 2.6 (4.2 with the normal factor), the labels' round trip 1.0, xi's 1.2, the
// lists of rows and cells 2.0, the reduction and solve 1.1.  Staging all 1728 cells with
// their labels as bytes (1 round trip, 41 MB a launch), moments summed per datum and a rank
// test on every cell took 22: a layer's launch went 23.4 -> 15 us there and 38 -> 25 us on a
// suspension of 40 ellipsoids.  Measured slower: the rows of a brick along the axis that
// gives its gathers the fewest lines (fewer lines, but 0.6 us more to transpose the bits:
// call 144 -> 161 us), and a row's xi loaded by the thread that owns the row, without the
// list of staged cells (three round trips instead of one: 144 -> 158 us).
//
// part: 0 the whole brick, 1 and 2 its halves.  Returns the part to do next, 0 for none.
// kAny: for any r_s (else r_s is the staged radius, 2, and the kernel holds no other code).  A
// smaller r_s is fitted from the staged data first; with a larger one every cell is gathered from
// global memory.  Call of 40 ellipsoids with r_s = 1, a third of whose cells grow to 2: 238 us
// (588 with both radii from global memory), with r_s = 3: 547 us (880 before gather_any's rows).
template <typename T, bool kAny>
__device__ __forceinline__ int extrap_brick(const FitArgs& b, unsigned long long pk, int l,
                                            unsigned char* lds, const FitTables& tables, int& tab,
                                            int part) {
    constexpr int S = kBrickSpan, S2 = kBrickSpan * kBrickSpan;
    const int s = entry_solid(pk);
    DevSolidC* d = const_solid(b.solids, s);
    const int want = d->aniso ? s : -1;   // the weight table this brick needs
    const BrickLds<T> B = brick_lds<T>(lds);
    // re-derived per brick: the staging index math is not kept live across bricks
    const int tid = opaque_lane_value(threadIdx.x);
    const int lane = tid & 63, wid = uniform_int(tid >> 6);
    const unsigned long long lt = (1ull << lane) - 1ull;
    const int n1 = d->n1, n2 = d->n2;
    BrickCtx cx;
    cx.n0 = d->n0;
    cx.n01 = cx.n0 * n1;
    cx.nc = d->ncell;
    cx.ox = kBrick * entry_x(pk) - kBrickHalo;
    cx.oy = kBrick * entry_y(pk) - kBrickHalo;
    cx.oz = kBrick * entry_z(pk) - kBrickHalo;
    cx.origin = cx.oz * cx.n01 + cx.oy * cx.n0 + cx.ox;
    const double* xi = d->xi;
    // Waves 0..2, a row per thread (threads past the last: empty rows).
    const int ry = tid % S, rz = tid / S;
    unsigned data = 0u;
    if (wid < 3) {
        RowBits rb = {0u, 0u};
        if (tid < S2 && (unsigned)(cx.oy + ry) < (unsigned)n1 &&
            (unsigned)(cx.oz + rz) < (unsigned)n2)
            rb = label_row_bits(d->labels, (int)cx.nc, cx.origin + rz * cx.n01 + ry * cx.n0,
                                cx.ox, cx.n0, l);
        data = rb.data;
        const int yc = ry - kBrickHalo, zc = rz - kBrickHalo;
        if ((unsigned)yc < (unsigned)kBrick && (unsigned)zc < (unsigned)kBrick)
            reinterpret_cast<uint8_t*>(B.target)[yc * kBrick + zc] =
                part == 0 || zc / (kBrick / 2) == part - 1 ? (uint8_t)(rb.target >> kBrickHalo) : 0;
        // the first datum of the wave's rows
        const unsigned long long m = __ballot(data != 0u);
        if (m ? lane == __builtin_ctzll(m) : lane == 0)
            B.ctl[wid] = m ? (int)cell_code(__builtin_ctz(data), ry, rz) : -1;
    }
    if (want != tab) {   // uniform: the table's owner is the same in every thread
        if (tid < kRlen) tables.rlen[tid] = rlen_entry(d, tid);
        tab = want;
    }
    __syncthreads();
    int width = 0, lo = 0, place = 0;
    unsigned near = 0u;
    if (wid < 3) {
        // The columns within radius 2 of a cell of the layer: the planes y within 2 (the
        // nearest one twice where one would lie outside), their rows z within 2, then two
        // columns to each side.
        if (tid < S2) {
            const int yc = ry - kBrickHalo, zs = 8 * (rz - 2 * kBrickHalo);
            unsigned long long t = 0ull;
#pragma unroll
            for (int dy = -2; dy <= 2; ++dy) t |= B.target[min(max(yc + dy, 0), kBrick - 1)];
            t = (zs >= 0 ? t >> zs : t << -zs) & 0xFFFFFFFFFFull;   // five rows
            t |= t >> 32;
            near = (unsigned)(t | t >> 8 | t >> 16 | t >> 24) & 255u;
            near <<= kBrickHalo;
            near |= (near << 1) | (near >> 1) | (near << 2) | (near >> 2);
            lo = near ? __builtin_ctz(near) : 0;
            width = near ? 32 - __builtin_clz(near) - lo : 0;
        }
        // the row's place among the wave's rows: a prefix sum of the widths, bit by bit
        int total = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned long long m = __ballot((width >> i) & 1);
            place += __popcll(m & lt) << i;
            total += __popcll(m) << i;
        }
        if (lane == 0) B.ctl[3 + wid] = total;
    } else {
        // the layer's cells, listed by wave 3: a row of the brick per lane, a column at a time
        const int y = lane / kBrick, z = lane % kBrick;
        const unsigned mine = reinterpret_cast<const uint8_t*>(B.target)[lane];
        int total = 0;
#pragma unroll
        for (int x = 0; x < kBrick; ++x) {
            const unsigned long long m = __ballot((mine >> x) & 1u);
            if ((mine >> x) & 1u)
                B.cells[total + __popcll(m & lt)] =
                    (uint16_t)cell_code(kBrickHalo + x, kBrickHalo + y, kBrickHalo + z);
            total += __popcll(m);
        }
        if (lane == 0) {
            B.ctl[6] = total;
            B.ctl[7] = 0;
        }
    }
    __syncthreads();
    int total = uniform_int(B.ctl[6]);
    const int span0 = uniform_int(B.ctl[3]), span1 = uniform_int(B.ctl[4]);
    const int span = span0 + span1 + uniform_int(B.ctl[5]);
    const bool staged = !kAny || b.r_s == kBrickHalo || (b.r_s < kBrickHalo && b.r_max >= kBrickHalo);
    if (sizeof(T) == 8 && staged && span > span_cells<T>()) {   // uniform: does not fit
        __syncthreads();   // the LDS is free for the first half
        return 1;
    }
    // log2 of the lanes per cell: as many as keep every cell of the brick in one pass
    int sh = total <= 256 / 16 ? 4 : (total <= 256 / 8 ? 3 : 2);
    // The brick's anchor A: xi of the first cell of the region (in row order) that carries
    // data for layer l; one exists, since every layer-l cell has a neighbour in layer l - 1.
    // Staged values are xi - A: the fit is invariant to the shift, and the offsets are small
    // (the region spans 12 cells), which keeps the moments accurate and lets the
    // reduced-precision form hold them in FP32.
    int qa = uniform_int(B.ctl[0]);
    if (qa < 0) qa = uniform_int(B.ctl[1]);
    if (qa < 0) qa = uniform_int(B.ctl[2]);
    const int ca = qa < 0 ? 0 : brick_cell(cx, (unsigned)qa);
    const double a0 = load_global(xi + ca), a1 = load_global(xi + cx.nc + ca),
                 a2 = load_global(xi + 2 * cx.nc + ca);
    const bool nrm = l <= b.normal_layers;
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
    if (nrm && staged && total > 0) {
        const int cell = brick_cell(cx, B.cells[min(tid >> sh, total - 1)]);
        g0 = load_global(d->normals + cell);
        g1 = load_global(d->normals + cx.nc + cell);
        g2 = load_global(d->normals + 2 * cx.nc + cell);
    }
    if (tid < S2 && staged) {
        place += (wid > 0 ? span0 : 0) + (wid > 1 ? span1 : 0);
        B.rows[tid] = data | (unsigned)(place - lo + 16) << 12;
        const unsigned needed = data & near;
        const unsigned code = cell_code(lo, ry, rz);
        for (int j = 0; j < width; ++j)
            B.slots[place + j] =
                (uint16_t)((code + j) | (((needed >> (lo + j)) & 1u) ? kCellNeeded : 0u));
    }
    __syncthreads();
    if (staged) {
        // Every load of the thread is issued before its first use, so they cost one round
        // trip; a cell that is not needed loads the anchor's (no load waits on a branch).
        constexpr int kH = (span_cells<T>() + 255) / 256;
        unsigned on = 0u;   // bit h: cell h of the thread is needed
        double v0[kH], v1[kH], v2[kH];
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            if (256 * h < span) {   // uniform
                const int i = tid + 256 * h;
                const unsigned q = i < span ? B.slots[i] : 0u;
                const bool n = (q & kCellNeeded) != 0u;
                on |= n ? 1u << h : 0u;
                const int c = n ? brick_cell(cx, q) : ca;
                v0[h] = load_global(xi + c);
                v1[h] = load_global(xi + cx.nc + c);
                v2[h] = load_global(xi + 2 * cx.nc + c);
            }
        }
        cx.A[0] = uniform_double(a0);
        cx.A[1] = uniform_double(a1);
        cx.A[2] = uniform_double(a2);
#pragma unroll
        for (int h = 0; h < kH; ++h) {
            const int i = tid + 256 * h;
            if (i < span) {
                const bool n = (on >> h) & 1u;
                B.sx[i] = n ? (T)(v0[h] - cx.A[0]) : T(0);
                B.sx[span_cells<T>() + i] = n ? (T)(v1[h] - cx.A[1]) : T(0);
                B.sx[2 * span_cells<T>() + i] = n ? (T)(v2[h] - cx.A[2]) : T(0);
            }
        }
        __syncthreads();
        if (kAny && b.r_s < kBrickHalo) {   // radius 1 first: the cells it settles leave the list
            fit_cells<T, true>(d, nrm, cx, total, sh, 1, B, tables, g0, g1, g2);
            __syncthreads();
            keep_open_cells<T>(lds);
            total = uniform_int(B.ctl[6]);
            sh = total <= 256 / 16 ? 4 : (total <= 256 / 8 ? 3 : 2);
            if (nrm && total > 0) {
                const int cell = brick_cell(cx, B.cells[min(tid >> sh, total - 1)]);
                g0 = load_global(d->normals + cell);
                g1 = load_global(d->normals + cx.nc + cell);
                g2 = load_global(d->normals + 2 * cx.nc + cell);
            }
        }
        fit_cells<T, false>(d, nrm, cx, total, sh, kBrickHalo, B, tables, g0, g1, g2);
    } else {   // (only kAny) every cell is gathered from global memory
        cx.A[0] = uniform_double(a0);
        cx.A[1] = uniform_double(a1);
        cx.A[2] = uniform_double(a2);
        for (int ci = tid; ci < total; ci += 256) B.cells[ci] |= (uint16_t)kCellOpen;
        if (tid == 0) B.ctl[7] = 1;
    }
    __syncthreads();   // the list's flags; the rest of the LDS is free for the next brick
    if (uniform_int(B.ctl[7])) {
        fit_open_cells<T>(b, pk, l, lds, sh, staged, cx.A[0], cx.A[1], cx.A[2]);
        __syncthreads();
    }
    return part == 1 ? 2 : 0;
}

// ------------------------------------------------------------------------------------
// Brick lists: the bucket counts of layers l0..l0+nl-1 form one prefix in LDS
// (s_pref[0..nl*kBuckets]); entry e of the concatenation is found by bisection.  The
// normal kernel walks the bucketed lists this way and copies them into dense per-layer
// lists for the fits.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ int list_prefix(const Batch& b, int l0, int nl, int* s_pref,
                                           int* s_wave) {
    const int n = nl * kBuckets;   // <= 1024: four counts per thread
    int v[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // the four loads first
        const int i = threadIdx.x * 4 + q;
        v[q] = i < n ? b.bcount[(l0 - 1) * kBuckets + i] : 0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = threadIdx.x * 4 + q;
        if (i < n) {
            const int bk = i % kBuckets;
            const int64_t cap = bucket_base(bk + 1, b.n_tiles, b.tile_w) -
                                bucket_base(bk, b.n_tiles, b.tile_w);
            // entries past a bucket's capacity were never written (reported as overflow)
            v[q] = (int)min((int64_t)v[q], cap);
        }
        sum += v[q];
    }
    int excl, total;
    block_scan<4>(sum, excl, total, s_wave);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = threadIdx.x * 4 + q;
        if (i < n) s_pref[i] = excl;
        excl += v[q];
    }
    if (threadIdx.x == 0) s_pref[n] = total;
    __syncthreads();
    return total;
}

// Entry e of the concatenated lists: its layer and list entry.
__device__ __forceinline__ unsigned long long list_entry(const Batch& b, int l0, int nl,
                                                         const int* s_pref, int e, int* layer) {
    int lo = 0, hi = nl * kBuckets - 1;   // last i with s_pref[i] <= e
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_pref[mid] <= e) lo = mid; else hi = mid - 1;
    }
    const int li = lo / kBuckets, bk = lo % kBuckets;
    *layer = l0 + li;
    return b.blist[(int64_t)(l0 - 1 + li) * b.blist_cap + bucket_base(bk, b.n_tiles, b.tile_w) +
                   (e - s_pref[lo])];
}

// ------------------------------------------------------------------------------------
// Per-solid statistics from the tile counts, then the normals of the listed bricks of
// layers 1..normal_layers.
// ------------------------------------------------------------------------------------
constexpr int kNSpan = kBrick + 2;                        // brick with a halo of 1
constexpr int kNCells = kNSpan * kNSpan * kNSpan;         // 1000

// The flagged cells of the region as a list (in any order): cells tid + 256 h, by
// ballots.  Returns their number; a block's barrier at the end.
__device__ __forceinline__ int flagged_cells(int tid, const unsigned char* s_flag,
                                             uint16_t* s_list, int* s_wave) {
    const int lane = tid & 63, wid = tid >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    unsigned long long bal[4];
    int wsum = 0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int q = tid + 256 * h;
        bal[h] = __ballot(q < kNCells && s_flag[q]);
        wsum += __popcll(bal[h]);
    }
    if (lane == 0) s_wave[wid] = wsum;
    __syncthreads();
    int pos = 0, total = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = s_wave[i];
        if (i < wid) pos += t;
        total += t;
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int q = tid + 256 * h;
        if ((bal[h] >> lane) & 1ull) s_list[pos + __popcll(bal[h] & lt)] = (uint16_t)q;
        pos += __popcll(bal[h]);
    }
    __syncthreads();
    return total;
}

template <bool kSpheres>
__device__ __forceinline__ void normal_brick(DevSolidC* d, unsigned long long* st, int l,
                                             int bx, int by, int bz, double* s_phi,
                                             unsigned char* s_flag, int8_t* s_lab,
                                             uint16_t* s_list, int* s_wave) {
    // re-derived per brick: the index math is not kept live across bricks
    const int tid = opaque_lane_value(threadIdx.x);
    const int n0 = d->n0, n1 = d->n1, n2 = d->n2;
    const int64_t nc = d->ncell;
    const int ox = kBrick * bx - 1, oy = kBrick * by - 1, oz = kBrick * bz - 1;
    for (int q = tid; q < kNCells; q += 256) s_flag[q] = 0;
    const int8_t* __restrict__ labels = d->labels;
    int8_t lv[2];   // both label loads issued before the LDS stores
    bool inb[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int q = tid + 256 * h;
        const int x = q % kBrick, y = (q / kBrick) % kBrick, z = q / (kBrick * kBrick);
        const int gx = ox + 1 + x, gy = oy + 1 + y, gz = oz + 1 + z;
        inb[h] = gx < n0 && gy < n1 && gz < n2;
        lv[h] = load_global(labels + (inb[h] ? ((int64_t)gz * n1 + gy) * n0 + gx : 0));
    }
    s_lab[tid] = inb[0] ? lv[0] : (int8_t)-1;
    s_lab[tid + 256] = inb[1] ? lv[1] : (int8_t)-1;
    __syncthreads();
    if (load_const(st + ST_FLAGS) & FLAG_TRUNCATED) return;   // uniform: no fit follows
    // a cell of layer l needs phi0 at itself and at its six face neighbours
    for (int q = tid; q < kBrick * kBrick * kBrick; q += 256) {
        if (s_lab[q] != l) continue;
        const int x = q % kBrick, y = (q / kBrick) % kBrick, z = q / (kBrick * kBrick);
        const int r = ((z + 1) * kNSpan + (y + 1)) * kNSpan + (x + 1);
        s_flag[r] = 1;
        s_flag[r - 1] = 1;
        s_flag[r + 1] = 1;
        s_flag[r - kNSpan] = 1;
        s_flag[r + kNSpan] = 1;
        s_flag[r - kNSpan * kNSpan] = 1;
        s_flag[r + kNSpan * kNSpan] = 1;
    }
    __syncthreads();
    const int total = flagged_cells(tid, s_flag, s_list, s_wave);
    // phi0 of each needed cell once (defined: inside the box with a finite xi)
    const ShapeR sh = load_shape(d);
    const double* __restrict__ f = d->xi_normal;
    for (int i = tid; i < total; i += 256) {
        const int r = s_list[i];
        const int x = r % kNSpan, y = (r / kNSpan) % kNSpan, z = r / (kNSpan * kNSpan);
        const int gx = ox + x, gy = oy + y, gz = oz + z;
        const bool in = (unsigned)gx < (unsigned)n0 && (unsigned)gy < (unsigned)n1 &&
                        (unsigned)gz < (unsigned)n2;
        const int64_t c = in ? ((int64_t)gz * n1 + gy) * n0 + gx : 0;
        const double x0 = load_global(f + c), x1 = load_global(f + nc + c),
                     x2 = load_global(f + 2 * nc + c);
        const bool def = in && finite3(x0, x1, x2);
        double ph = 0.0;
        if (def) {
            if constexpr (kSpheres)
                ph = phi0_sphere(sh, x0, x1, x2);
            else
                ph = phi0(sh, x0, x1, x2);
        }
        s_phi[r] = ph;
        s_flag[r] = def ? 3 : 1;
    }
    __syncthreads();
    // central differences where both neighbours are defined, else one-sided with the cell
    // itself (forward first), else 0
    int nzero = 0;
    for (int q = tid; q < kBrick * kBrick * kBrick; q += 256) {
        if (s_lab[q] != l) continue;
        const int x = q % kBrick, y = (q / kBrick) % kBrick, z = q / (kBrick * kBrick);
        const int r = ((z + 1) * kNSpan + (y + 1)) * kNSpan + (x + 1);
        const int step[3] = {1, kNSpan, kNSpan * kNSpan};
        const bool d0 = s_flag[r] == 3;
        double g[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int rp = r + step[a], rm = r - step[a];
            const bool dp = s_flag[rp] == 3, dm = s_flag[rm] == 3;
            double ga;
            if (dp && dm) ga = 0.5 * (s_phi[rp] - s_phi[rm]);
            else if (dp && d0) ga = s_phi[rp] - s_phi[r];
            else if (dm && d0) ga = s_phi[r] - s_phi[rm];
            else ga = 0.0;
            g[a] = ga;
        }
        const int64_t cell = ((int64_t)(oz + 1 + z) * n1 + (oy + 1 + y)) * n0 + (ox + 1 + x);
        d->normals[cell] = g[0];
        d->normals[nc + cell] = g[1];
        d->normals[2 * nc + cell] = g[2];
        nzero += (g[0] == 0.0 && g[1] == 0.0 && g[2] == 0.0);
    }
    if (nzero) atomicAdd(st + ST_NONORMAL, (unsigned long long)nzero);   // rare
}

// Per-solid interior and band counts, the sums of the solids' tile counts, into the
// statistics (blocks b, b + gridDim.x, ... take solids b, ...).
__device__ __forceinline__ void solid_counts(const Batch& b, unsigned long long* s_acc) {
    const int tid = threadIdx.x;
    for (int s = blockIdx.x; s < b.n_solids; s += gridDim.x) {
        const DevSolid* d = b.solids + s;
        if (tid < kLT) s_acc[tid] = 0ull;
        __syncthreads();
        // (a count is at most the box's cells, below 2^31: 32-bit sums)
        int acc[kLT];
#pragma unroll
        for (int l = 0; l < kLT; ++l) acc[l] = 0;
        const int L = d->L;
        for (int t = d->tile_base + tid; t < d->tile_base + d->n_tiles; t += 256) {
            // every count of the tile loaded at once (entries past L hold no count of
            // this call and are dropped)
            int v[kLT];
#pragma unroll
            for (int l = 0; l < kLT; ++l) v[l] = b.tile_cnt[(int64_t)t * kLT + l];
#pragma unroll
            for (int l = 0; l < kLT; ++l) acc[l] += l <= L ? v[l] : 0;
        }
        // wave sums first (DPP row sums and four lane reads): one LDS atomic per wave and
        // count
#pragma unroll
        for (int l = 0; l < kLT; ++l) {
            if (l <= L) {   // uniform
                const int v = wave_sum(acc[l]);
                if ((tid & 63) == 0 && v) atomicAdd(&s_acc[l], (unsigned long long)(unsigned)v);
            }
        }
        __syncthreads();
        if (tid < kLT) b.stats[(int64_t)s * kStatWords + tid] = s_acc[tid];
        __syncthreads();
    }
}

// Four waves per SIMD (at most 128 registers, none spilled): the blocks go through their
// bricks' distances one at a time (bound by that chain: 6 of the 9 us of a brick), so resident
// waves hide it.  The entry of a block's next brick is on its way while one is done.  40
// ellipsoids 68 -> 36 us, one 128^3 ellipsoid 24 -> 14 us, 3 small solids 32 -> 15 us.  (Both
// layers of a brick at once, sharing phi0: 71 against 55 us at the time, as a brick's chain
// grows to two rounds and the blocks' shares are less even.)  A call whose solids are all
// spheres takes the sphere-only form (kSpheres), which holds no bisection and keeps more
// blocks resident.
template <bool kSpheres>
__global__ __launch_bounds__(256, kSpheres ? 8 : 4) void k_normal(Batch b) {
    __shared__ int s_wave[4];
    __shared__ int s_pref[kMaxLayers * kBuckets + 1];
    __shared__ unsigned long long s_acc[kLT];
    __shared__ double s_phi[kNCells];
    __shared__ unsigned char s_flag[kNCells];
    __shared__ int8_t s_lab[kBrick * kBrick * kBrick];
    __shared__ uint16_t s_list[kNCells];
    const int tid = threadIdx.x;
    solid_counts(b, s_acc);
    // Dense per-layer brick lists for the fits: entry e of the bucketed lists of layers
    // 1..Lmax goes to its rank within its layer (bucket order), and each layer's count to
    // dcount.  The prefix over all layers also serves the normals' layers 1..nl.
    const int tot = list_prefix(b, 1, b.Lmax, s_pref, s_wave);
    if (blockIdx.x == 0 && tid < b.Lmax)
        b.dcount[tid] = s_pref[(tid + 1) * kBuckets] - s_pref[tid * kBuckets];
    for (int e = blockIdx.x * 256 + tid; e < tot; e += gridDim.x * 256) {
        int layer = 1;
        const unsigned long long pk = list_entry(b, 1, b.Lmax, s_pref, e, &layer);
        const int64_t i = e - s_pref[(layer - 1) * kBuckets];
        if (i < b.dlist_cap) b.dlist[(int64_t)(layer - 1) * b.dlist_cap + i] = pk;
    }
    const int nl = b.normal_layers;
    if (nl <= 0) return;
    const int total = s_pref[nl * kBuckets];
    const XcdRange rg = xcd_range(total);
    int l_next = 0;   // (the next brick's entry is on its way while this one is done)
    unsigned long long next = 0ull;
    if (rg.begin < rg.end) next = list_entry(b, 1, nl, s_pref, rg.begin, &l_next);
    for (int e = rg.begin; e < rg.end; e += rg.stride) {
        const unsigned pk = (unsigned)uniform_int((int)next);
        const int s = uniform_int((int)(next >> 32)), l = uniform_int(l_next);
        if (e + rg.stride < rg.end) next = list_entry(b, 1, nl, s_pref, e + rg.stride, &l_next);
        normal_brick<kSpheres>(const_solid(b.solids, s), b.stats + (int64_t)s * kStatWords, l,
                               entry_x(pk), entry_y(pk), entry_z(pk), s_phi, s_flag, s_lab,
                               s_list, s_wave);
        __syncthreads();   // the LDS is reused by the next brick
    }
}

// One launch per layer over the layer's dense brick list (built by the normal kernel):
// the blocks of each XCD stride over a contiguous range of it, so neighbouring bricks,
// whose halos overlap, share one L2.
template <typename T, bool kAny>
__global__ __launch_bounds__(256, 4) void k_extrap(Batch b, int l) {
    HIP_DYNAMIC_SHARED(double, lds_d)
    unsigned char* lds = reinterpret_cast<unsigned char*>(lds_d);
    __shared__ double s_rlen[kRlen];
    __shared__ RowSums s_rows[kRowSets];
    const unsigned long long* dl = b.dlist + (int64_t)(l - 1) * b.dlist_cap;
    const int count = (int)min((int64_t)load_const(b.dcount + l - 1), b.dlist_cap);
    const FitTables tables = {s_rlen, s_rows};   // (read after the first brick's barriers)
    fill_fit_tables(tables);
    int tab = -1;   // the loaded weights: equal spacings
    const FitArgs args = {b.solids, b.stats, b.normal_layers, b.r_s, b.r_max};
    const XcdRange rg = xcd_range(count);
    int part = 0;   // (a brick that does not fit comes round again in halves)
    for (int e = rg.begin; e < rg.end;) {
        const unsigned long long pk = load_const(dl + e);
        const unsigned long long* st = b.stats + (int64_t)entry_solid(pk) * kStatWords;
        if (!(load_const(st + ST_FLAGS) & FLAG_TRUNCATED))   // uniform: the block skips
            part = extrap_brick<T, kAny>(args, pk, l, lds, tables, tab, part);
        if (part == 0) e += rg.stride;
    }
}

// ------------------------------------------------------------------------------------
// Persistent band launch: the normals and the fits of every layer of the whole batch in
// ONE launch, over the compacted brick lists.  Work items are bricks: phase 0 the bricks
// of layers 1..normal_layers (normals), phase l the bricks of layer l (fits).  Each phase
// is split into kQueues contiguous slices, one queue each, in proportion to the blocks of
// queue x (blocks b with b % kQueues == x): neighbouring bricks, whose halos overlap, are
// then mostly fitted on one XCD (the hardware deals blocks to the XCDs round-robin).  A
// block takes items of its current phase from its own queue, then from any queue with
// items left, and moves to the next phase only once every queue of its phase is
// exhausted.  An item of phase p > 0 waits until every item of phase p - 1 is complete
// (layers in ascending order, "Extrapolation of xi"; the normals are taken from the field
// before any fit writes).  A block publishes its finished items of a phase (one release,
// one count) when it leaves the phase, before it can wait; it acquires once per phase it
// enters, and polls without ordering: an ordered poll would invalidate the XCD's L2 on
// every read.  Since no block reaches phase p before all items of phase p - 1 were
// handed out, each to a block that is running, the lowest unfinished phase always has
// its items in blocks that do not wait: no deadlock, whatever the residency.  Every wait
// is bounded: past the bound the call's error flag is set, the item is skipped (still
// counted), and every wave reaches the end.
// ------------------------------------------------------------------------------------
constexpr int kQueues = kXcds;
constexpr int kBandSpin = 1 << 20;   // polls of a bounded wait (each an acquire load and a
                                     // short sleep: about a second in all)

// Shared memory of the band kernel, carved from its dynamic LDS (no static LDS: the
// block's whole state lies in its own allocation).
struct BandLds {
    unsigned char* work;   // a brick's fit staging, or a brick's normal scratch
    double* s_phi;
    unsigned char* s_flag;
    int8_t* s_lab;
    uint16_t* s_list;
    int* s_pref;           // [kMaxLayers * kBuckets + 1]
    int* s_wave;           // [4]
    int* s_ctl;            // [4]: ticket, wait result
    FitTables tables;      // the fits' weights [kRlen] and row sums [kRowSets]
    unsigned long long* s_acc;  // [kLT]
};

__host__ __device__ constexpr size_t band_small_bytes() {
    return sizeof(int) * (kMaxLayers * kBuckets + 1 + 4 + 4) + sizeof(double) * kRlen +
           sizeof(RowSums) * kRowSets + sizeof(unsigned long long) * kLT + 64;
}

__device__ __forceinline__ BandLds band_lds(unsigned char* lds, size_t work_bytes) {
    BandLds L;
    L.work = lds;
    L.s_phi = reinterpret_cast<double*>(lds);
    L.s_flag = lds + sizeof(double) * kNCells;
    L.s_lab = reinterpret_cast<int8_t*>(L.s_flag + kNCells);
    L.s_list = reinterpret_cast<uint16_t*>(lds + sizeof(double) * kNCells + kNCells +
                                           kBrick * kBrick * kBrick);
    unsigned char* sm = lds + ((work_bytes + 15) & ~size_t(15));
    L.tables.rlen = reinterpret_cast<double*>(sm);
    L.tables.rows = reinterpret_cast<RowSums*>(L.tables.rlen + kRlen);
    L.s_acc = reinterpret_cast<unsigned long long*>(L.tables.rows + kRowSets);
    L.s_pref = reinterpret_cast<int*>(L.s_acc + kLT);
    L.s_wave = L.s_pref + kMaxLayers * kBuckets + 1;
    L.s_ctl = L.s_wave + 4;
    return L;
}

// Items of phase p (0: bricks of layers 1..nl; p >= 1: bricks of layer p).
__device__ __forceinline__ int phase_items(const int* s_pref, int p, int nl) {
    return p == 0 ? s_pref[nl * kBuckets] : s_pref[p * kBuckets] - s_pref[(p - 1) * kBuckets];
}

// Slice [lo, hi) of a phase's n items held by queue x of nq, over G blocks.
__device__ __forceinline__ void queue_slice(int n, int G, int nq, int x, int* lo, int* hi) {
    int before = 0;   // blocks of the queues before x
    for (int y = 0; y < x; ++y) before += (G - y + nq - 1) / nq;
    const int mine = (G - x + nq - 1) / nq;
    *lo = (int)((int64_t)n * before / G);
    *hi = (int)((int64_t)n * (before + mine) / G);
}

// Wave 0 of a block: the next item of the block's phase *ph (advanced past exhausted
// phases); returns its index within the phase, or -1 once every phase is exhausted.
__device__ int band_take(BandCtl* ctl, const int* s_pref, int nl, int Lmax, int q, int nq,
                         int* ph) {
    const int lane = threadIdx.x;
    const int G = gridDim.x;
    for (; *ph <= Lmax; ++*ph) {
        const int p = *ph;
        const int n = phase_items(s_pref, p, nl);
        int lo, hi;
        queue_slice(n, G, nq, q, &lo, &hi);
        int t = 0;
        if (lane == 0) t = atomicAdd(&ctl->taken[p][q], 1);
        t = __shfl(t, 0);
        if (t < hi - lo) return lo + t;
        // the other queues: lane i < nq - 1 looks at queue (q + 1 + i) % nq
        for (;;) {
            const int x = (q + 1 + lane) % nq;
            int xlo = 0, xhi = 0, left = 0;
            if (lane < nq - 1) {
                queue_slice(n, G, nq, x, &xlo, &xhi);
                left = __hip_atomic_load(&ctl->taken[p][x], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) < xhi - xlo;
            }
            const unsigned long long m = __ballot(left);
            if (m == 0ull) break;   // phase exhausted
            const int src = __ffsll((long long)m) - 1;
            int u = 0;
            if (lane == src) u = atomicAdd(&ctl->taken[p][x], 1);
            u = __shfl(u, src);
            const int ulo = __shfl(xlo, src), uhi = __shfl(xhi, src);
            if (u < uhi - ulo) return ulo + u;
        }
    }
    return -1;
}

template <typename T, bool kAny>
__global__ __launch_bounds__(256, 3) void k_band(Batch b, int work_bytes) {
    HIP_DYNAMIC_SHARED(double, lds_d)
    const BandLds L = band_lds(reinterpret_cast<unsigned char*>(lds_d), (size_t)work_bytes);
    BandCtl* ctl = b.band;
    const int tid = threadIdx.x;
    fill_fit_tables(L.tables);
    int tab = -1;   // the loaded weights: equal spacings
    solid_counts(b, L.s_acc);
    list_prefix(b, 1, b.Lmax, L.s_pref, L.s_wave);   // (ends with a barrier)
    const int nl = b.normal_layers;
    const int nq = gridDim.x < kQueues ? (int)gridDim.x : kQueues;
    const int q = blockIdx.x % nq;
    int ph = 0, err = 0;
    int ready = 0;              // phases before this one are complete and acquired
    int pend = 0, pend_ph = 0;  // items of phase pend_ph done here and not yet published
    for (;;) {
        if (tid < 64) {
            int p = ph;
            const int it = band_take(ctl, L.s_pref, nl, b.Lmax, q, nq, &p);
            if (tid == 0) {
                L.s_ctl[0] = it;
                L.s_ctl[2] = p;
            }
        }
        __syncthreads();
        const int item = L.s_ctl[0];
        const int p = L.s_ctl[2];
        __syncthreads();   // (s_ctl is rewritten by the next take)
        ph = p;
        // publish this block's finished items of an earlier phase before anything waits:
        // every thread's stores (one release), then their count
        if (pend > 0 && (item < 0 || p != pend_ph)) {
            __threadfence();
            __syncthreads();
            if (tid == 0) atomicAdd(&ctl->done[pend_ph], pend);
            pend = 0;
        }
        if (item < 0) break;   // every phase is exhausted
        bool run = !err;
        if (p > ready) {
            // wait until every item of phase p - 1 is complete (polled without ordering,
            // then one acquire for the whole block)
            if (tid == 0) {
                const int need = phase_items(L.s_pref, p - 1, nl);
                int ok = 1, spins = 0;
                while (__hip_atomic_load(&ctl->done[p - 1], __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) < need) {
                    if (++spins > kBandSpin ||
                        __hip_atomic_load(&ctl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        atomicOr(&ctl->err, 1);
                        ok = 0;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(4);
                }
                L.s_ctl[1] = ok;
            }
            __syncthreads();
            const int ok = L.s_ctl[1];
            run = run && ok;
            err = !ok || err;
            // every thread: its later loads see what the finished items stored
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (ok) ready = p;
        }
        if (run) {
            const int e = p == 0 ? item : L.s_pref[(p - 1) * kBuckets] + item;
            int layer = 1;
            const unsigned long long pk = list_entry(b, 1, b.Lmax, L.s_pref, e, &layer);
            const int s = uniform_int((int)(pk >> 32));
            const unsigned place = (unsigned)uniform_int((int)pk);
            const unsigned long long pk_uniform = ((unsigned long long)s << 32) | place;
            const int bx = entry_x(place), by = entry_y(place), bz = entry_z(place);
            layer = uniform_int(layer);
            unsigned long long* st = b.stats + (int64_t)s * kStatWords;
            if (!(st[ST_FLAGS] & FLAG_TRUNCATED)) {   // uniform: no fit follows a truncation
                if (p == 0)
                    normal_brick<false>(const_solid(b.solids, s), st, layer, bx, by, bz, L.s_phi,
                                        L.s_flag, L.s_lab, L.s_list, L.s_wave);
                else
                    for (int part = 0;;) {
                        part = extrap_brick<T, kAny>(
                            {b.solids, b.stats, b.normal_layers, b.r_s, b.r_max}, pk_uniform, p,
                            L.work, L.tables, tab, part);
                        if (part == 0) break;
                    }
            }
        }
        ++pend;   // (a skipped item counts too)
        pend_ph = p;
        __syncthreads();   // the item's LDS is free for the next one
    }
    if (err && tid == 0)
        for (int s = 0; s < b.n_solids; ++s)
            atomicOr(b.stats + (int64_t)s * kStatWords + ST_FLAGS, FLAG_TIMEOUT);
}

}  // namespace

// ------------------------------------------------------------------------------------
// Launchers.
// ------------------------------------------------------------------------------------
hipError_t launch_classify(const Batch& b, hipStream_t st) {
    const int grid = b.n_chunks < 8192 ? b.n_chunks : 8192;
    hipLaunchKernelGGL(k_classify, dim3(grid), dim3(256), 0, st, b);
    return hipGetLastError();
}

size_t label_lds_bytes(int Lmax, int tile_w, int Wmax) {
    const int RJ = kTileJ + 2 * Lmax, RK = kTileK + 2 * Lmax;
    const int RW = tile_w + 2 < Wmax ? tile_w + 2 : Wmax;
    const size_t region = sizeof(unsigned long long) * 2 * (size_t)(RW | 1) * RJ * RK;
    const size_t rows = (size_t)256 * 8 * (8 * tile_w + 1);   // transposed labels of a tile
    return region > rows ? region : rows;
}

hipError_t launch_label(const Batch& b, size_t lds, hipStream_t st) {
    if (b.tile_w == 1)
        hipLaunchKernelGGL(k_label<1>, dim3(b.n_tiles), dim3(kLabelThreads), lds, st, b);
    else if (b.tile_w == 2)
        hipLaunchKernelGGL(k_label<2>, dim3(b.n_tiles), dim3(kLabelThreads), lds, st, b);
    else if (b.tile_w == 4)
        hipLaunchKernelGGL(k_label<4>, dim3(b.n_tiles), dim3(kLabelThreads), lds, st, b);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

int normal_blocks_per_cu(bool spheres) {
    static const int n[2] = {[] {
                                 int v = 0;
                                 if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                         &v, k_normal<false>, 256, 0) != hipSuccess || v < 1)
                                     v = 4;
                                 return v;
                             }(),
                             [] {
                                 int v = 0;
                                 if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                         &v, k_normal<true>, 256, 0) != hipSuccess || v < 1)
                                     v = 4;
                                 return v;
                             }()};
    return n[spheres ? 1 : 0];
}

hipError_t launch_normal(const Batch& b, int blocks, hipStream_t st) {
    if (b.spheres)
        hipLaunchKernelGGL(k_normal<true>, dim3(blocks), dim3(256), 0, st, b);
    else
        hipLaunchKernelGGL(k_normal<false>, dim3(blocks), dim3(256), 0, st, b);
    return hipGetLastError();
}

size_t band_lds_bytes(int precision) {
    const size_t normal = sizeof(double) * kNCells + kNCells + kBrick * kBrick * kBrick +
                          sizeof(uint16_t) * kNCells;
    const size_t fit = brick_lds_bytes(precision);
    const size_t work = fit > normal ? fit : normal;
    return ((work + 15) & ~size_t(15)) + band_small_bytes();
}

// Blocks per CU of the persistent launch: one, when one fits.  Each block releases (an L2
// write-back of its XCD) when it leaves a phase and acquires (an L2 invalidation) when it
// enters one; with more blocks per CU these operations thrash the L2 more than the added
// residency hides latency (with the fits of before the row bits, a 256^3 sphere's launch took
// 384 us with one block per CU and 790 with three; the call takes 416 us now).
int band_blocks_per_cu(int precision) {
    static const int n[2] = {
        [] {
            int v = 0, w = 0;
            const size_t lds = band_lds_bytes(0);
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k_band<double, false>, 256,
                                                                lds) == hipSuccess &&
                           hipOccupancyMaxActiveBlocksPerMultiprocessor(&w, k_band<double, true>,
                                                                        256, lds) == hipSuccess &&
                           v >= 1 && w >= 1
                       ? 1
                       : 0;
        }(),
        [] {
            int v = 0, w = 0;
            const size_t lds = band_lds_bytes(1);
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k_band<float, false>, 256,
                                                                lds) == hipSuccess &&
                           hipOccupancyMaxActiveBlocksPerMultiprocessor(&w, k_band<float, true>,
                                                                        256, lds) == hipSuccess &&
                           v >= 1 && w >= 1
                       ? 1
                       : 0;
        }()};
    return n[precision == 1 ? 1 : 0];
}

// Forms of the fits: for r_s equal to the staged radius, and (kAny) for any r_s.
hipError_t launch_band(const Batch& b, int precision, int blocks, hipStream_t st) {
    const size_t lds = band_lds_bytes(precision);
    const int work = (int)(lds - band_small_bytes());
    const bool any = b.r_s != kBrickHalo;
    const auto k_band_form = precision == 1 ? (any ? k_band<float, true> : k_band<float, false>)
                                            : (any ? k_band<double, true> : k_band<double, false>);
    hipLaunchKernelGGL(k_band_form, dim3(blocks), dim3(256), lds, st, b, work);
    return hipGetLastError();
}

hipError_t launch_extrap(const Batch& b, int layer, int precision, int blocks,
                         hipStream_t st) {
    const size_t lds = brick_lds_bytes(precision);
    const bool any = b.r_s != kBrickHalo;
    const auto form = precision == 1 ? (any ? k_extrap<float, true> : k_extrap<float, false>)
                                     : (any ? k_extrap<double, true> : k_extrap<double, false>);
    hipLaunchKernelGGL(form, dim3(blocks), dim3(256), lds, st, b, layer);
    return hipGetLastError();
}

}  // namespace rmx
