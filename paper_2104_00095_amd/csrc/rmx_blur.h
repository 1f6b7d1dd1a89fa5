// Device tables and launchers of the blur-zone consumers of the extrapolated reference
// maps (Lin, Derr & Rycroft, arXiv 2104.00095: "Blurred interface method and monolithic
// governing equations", eq. (sm_heavi); SI "Stress calculations", eq. (mod_heaviside)).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace rmx {

// Tiles of 8^3 grid cells.  (A wider tile lists more candidate solids for every cell.)
constexpr int kBlurTX = 8, kBlurTY = 8, kBlurTZ = 8;
constexpr int kBlurTileCells = kBlurTX * kBlurTY * kBlurTZ;

// Units of the fill (a wave each): consecutive values of a region that spans whole planes of
// its array, or rows along x of one plane.
constexpr int kFillRun = 8192, kFillRows = 16;
__host__ __device__ inline bool fill_planes(int E0, int E1, int n0, int n1) {
    return E0 == n0 && E1 == n1;
}
// Blocks of the fill (four units at a time), which stride over the units: a launch takes fewer
// than 2^32 threads, and the units are not bounded by the arrays' sizes (a thin box has one per
// 16 rows, and boxes may overlap).
constexpr int kFillBlocksPerCu = 256;
inline int fill_blocks(int64_t units, int cus) {
    const int64_t most = (int64_t)kFillBlocksPerCu * (cus > 1 ? cus : 1);
    const int64_t blocks = (units + 3) / 4;
    return (int)(blocks < most ? blocks : most);
}

// One solid: its box in the grid, phi0, and its fields (from an extrapolation call).
struct BlurDev {
    int32_t lo[3], ext[3];
    int32_t L, kind;
    double centre[3], semi[3], rot[9];   // a sphere: semi = R (three times), rot = I
    const double* xi;                    // [3][e2][e1][e0]
    const int8_t* labels;                // [e2][e1][e0]
    double* phi;                         // [e2][e1][e0] or null
    double G;                            // shear modulus
    int64_t unit0;                       // first unit of the solid in the fill
    int64_t units[3];                    // its units: of its cells ([0]), or of its faces per axis
};

struct BlurBatch {
    const BlurDev* solids;
    int32_t n_solids;
    int32_t grid[3];
    int32_t periodic[3];         // 1: the grid wraps along the axis (n faces, not n + 1)
    int32_t tiles[3];            // tiles along x, y, z
    int32_t n_active;
    int32_t spheres;             // every solid is a sphere: the full kernels' sphere-only form
    const int32_t* tile_start;   // [tiles + 1]: candidate solids of each tile (CSR)
    const int32_t* tile_list;    // ascending solid indices (boxes dilated by one cell)
    const int32_t* active;       // tiles with a candidate
    int32_t* n_covered;          // tiles of `active` with a covered cell (zeroed per call)
    int32_t* covered;            // [n_active]: those tiles, in the order the scan found them
    int64_t fill_units;          // units of the fill, all solids
    int32_t fill_blocks;         // blocks that stride over them
    double eps;
    double h[3], rh[3];          // spacing of each axis, and 1 / spacing
    double* H;                   // [n2][n1][n0] or null
    double* tau[3];              // [6][n2 + f2][n1 + f1][n0 + f0] or null, f_b = 1 if b == a
                                 // and axis a is walled, else 0
};

hipError_t launch_blur_heaviside(const BlurBatch& b, hipStream_t st);
hipError_t launch_blur_stress(const BlurBatch& b, hipStream_t st);

}  // namespace rmx
