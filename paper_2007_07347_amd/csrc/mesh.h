// Host-side mesh builder of the solver library: raw polygons -> per-cell slot
// arrays in the library's (optionally RCM) order.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/sdugks.h"

namespace sdg {

constexpr int32_t kEmptySlot = INT32_MIN;   // padding slot of a cell with fewer faces than D

struct BcEntry {
    int32_t type;
    double rho, u, v;        // SYMMETRY: (u, v) = unit outward normal of the tag's line
};

// Everything the device needs, in the library's cell order.  Per-slot arrays
// are structure-of-arrays [D][nc]: slot s of cell c at index s*nc + c.
struct MeshBuild {
    int32_t nc = 0;        // cells
    int32_t D = 0;         // slots per cell (max polygon degree)
    int32_t n_faces = 0;   // faces after periodic gluing
    int32_t n_bfaces = 0;  // boundary (non-periodic) faces
    int32_t n_singular = 0;
    double h_min = 0, dt = 0, tau = 0;
    std::vector<int32_t> perm;    // internal index -> caller index
    std::vector<int32_t> iperm;   // caller index -> internal index
    // per cell, internal order
    std::vector<double> area, cx, cy;
    std::vector<double> ainv;     // [3][nc]: (A^-1)_xx, (A^-1)_xy, (A^-1)_yy of the LSQ normal matrix
    // per slot
    std::vector<int32_t> nbr;     // >= 0 neighbour cell; < 0: -(1 + boundary face); kEmptySlot
    std::vector<double> lnx, lny; // scaled outward normal l*n of the face, seen from this cell
    std::vector<double> rsx, rsy; // face midpoint minus this cell's centroid
    std::vector<double> rox, roy; // face midpoint (in the neighbour's frame) minus the neighbour's centroid
    std::vector<double> wx, wy;   // least-squares weight A^-1 d of the stencil point behind the slot
    std::vector<int32_t> fid;     // face behind the slot (both cells of an interior face share it); -1 empty
    // boundary faces
    std::vector<int32_t> bf_cell, bf_tag;
    std::vector<BcEntry> bcs;
    // Tiles of the fused step (empty when the two-kernel step is used).  Tile t
    // owns the contiguous internal cells [g0, g0 + nt); its local cells are
    // those, then the n1 cells of its first halo ring, then the n2 of its
    // second.  Per-tile tables, padded to the largest tile (PL = nl_max local
    // cells, PA = na_max cells of tile + first ring, PT = nt_max tile cells,
    // PF = nf_max face records):
    //   lgid [n_tiles][PL]          internal id of every local cell;
    //   ladj [n_tiles][D][PA]       neighbour behind each slot of a tile or
    //                               first-ring cell: local index >= 0, -1 empty,
    //                               -2 - tag for a boundary face of that tag;
    //   lfc  [n_tiles][D][PT]       face of each slot of a tile cell: record
    //                               index * 2, + 1 if the record is stored as
    //                               seen from the other cell; -1 empty;
    //   frec [n_tiles][3][PF][2]    one record per face of the tile's cells, as
    //                               seen from the first tile cell that has it:
    //                               rows l n, r_self, r_other of (x, y).  A face
    //                               between two tile cells is stored once; the
    //                               other cell's view is (-l n, r_other, r_self),
    //                               the exact mirror the per-slot arrays hold.
    //   fcell [n_tiles][PF]         its two cells: local index of the first, and in
    //                               the upper 16 bits the local index of the
    //                               second or -2 - tag (as ladj);
    //   lw   [n_tiles][D][PA][2]    least-squares weight (x, y) behind each slot
    //                               of a tile or first-ring cell.
    int32_t tile_T = 0, n_tiles = 0, nl_max = 0, na_max = 0, nt_max = 0, nf_max = 0;
    std::vector<int32_t> tile_hdr;   // [n_tiles][8]: g0, nt, n1, n2, faces, 0...
    std::vector<int32_t> lgid;
    std::vector<int16_t> ladj;
    std::vector<int16_t> lfc;
    std::vector<int32_t> fcell;
    std::vector<double> frec;
    std::vector<double> lw;
    // Structured step (tensor-product quad meshes; cart == true): the cells
    // are (i, j), 0 <= i < nx, 0 <= j < ny, with corners (xs[i], ys[j]) ..
    // (xs[i+1], ys[j+1]); the internal order is row by row.  Per
    // column i, col[i][kCartVals]: width, offsets of its left and right face
    // midpoints from its centre, least-squares weights of its left and right
    // stencil points (neighbour centre, periodic image, or the wall face
    // midpoint), inverse width; per row the same in y.  Boundary-condition
    // entry of every boundary face of the four sides (-1 where periodic):
    // side[0..nx) bottom, [nx..2nx) top, [2nx..2nx+ny) left, then right.
    bool cart = false;
    int32_t nx = 0, ny = 0, per_x = 0, per_y = 0;
    std::vector<double> col, row;
    std::vector<int32_t> side;
};

// Nominal tiles of the structured step, as sdugks_tiling reports them (a unit of
// work for callers that size by tiles; the step itself cuts a mesh by its size,
// cart_plan.h): 16 x 14 cells for FP32 deviations, 16 x 7 otherwise.  Length of a
// per-column / per-row record.
constexpr int32_t kCartTX = 16, kCartTY = 14;
__host__ __device__ constexpr int32_t cart_tile_rows(int precision)
{
    return precision == SDUGKS_FP32DEV ? kCartTY : kCartTY / 2;
}
constexpr int32_t kCartVals = 8;   // width, left offset, right offset, left weight, right weight, 1/width, pad, pad
// Columns a wave of the marching step writes: its lanes less two halo columns
// on either side.
constexpr int32_t kCartCols = 60;

// Accelerator complex dies of an MI355X, each with its own L2: the fused step
// gives each a contiguous range of tiles.
constexpr int32_t kXcds = 8;
// Workgroups of a batched launch with room for cap_tiles tiles (a multiple of
// kXcds, so each XCD has the same number of tile slots).
inline int32_t batch_grid(int32_t cap_tiles) { return (cap_tiles + kXcds - 1) / kXcds * kXcds; }
// The single-instance fused step launches one workgroup per tile; workgroup b
// runs on XCD b % kXcds, so XCD x gets n / kXcds tiles, one more if
// x < n % kXcds, and takes the contiguous range that starts here.
__host__ __device__ inline int32_t xcd_range_start(int32_t n, int32_t x)
{
    return x * (n / kXcds) + (x < n % kXcds ? x : n % kXcds);
}
// Boundary-condition entries the fused step keeps in LDS (more: two-kernel step).
constexpr int32_t kMaxTileBcs = 64;
// LDS bytes of one workgroup of the fused step (elem: bytes of its arithmetic):
// W of the tile cells in FP64, the boundary table, slopes and carried-back
// fbar+ of every tile or first-ring cell, fbar+ of every local cell or the
// fluxes of the faces.
inline size_t tile_lds_bytes(int32_t nl_max, int32_t na_max, int32_t nt_max, int32_t nf_max, int32_t n_bc, size_t elem = 8)
{
    const size_t last = std::max(9 * (size_t)nl_max, 8 * (size_t)nf_max);
    return (3 * (size_t)nt_max + 1) / 2 * 16 + 32 * (size_t)n_bc + (27 * (size_t)na_max + last) * elem;
}
constexpr size_t kTileLdsLimit = 64 * 1024;
// Threads of the fused step by default, on tiles of 64 cells; with a number of
// threads given, tiles hold at most a quarter as many cells and every local cell
// and face has a thread of its own.
constexpr int32_t kDefaultBlock = 128, kDefaultTile = 64;

// Returns SDUGKS_OK or an error code with a message in err.
int build_mesh(const sdugks_mesh *mesh, const sdugks_bc *bc, int32_t n_bc, const sdugks_params *prm,
               MeshBuild &out, std::string &err);

}  // namespace sdg
