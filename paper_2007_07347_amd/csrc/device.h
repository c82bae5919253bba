// Device-side data of one solver instance and the launchers of its kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <tuple>
#include <utility>

#include "mesh.h"

namespace sdg {

struct DevBC {
    int32_t type;
    double rho, u, v;
};

// Mesh and constants of one instance, as seen by the kernels.  All per-cell
// arrays are pitched: entry (row r, cell c) at r*np + c.
struct DevMesh {
    int32_t nc, np, D, n_bfaces, n_bc;
    const int32_t *nbr;                 // [D][np]
    // two-kernel step only (the fused step reads per-tile face records):
    const double2 *ln;                  // [D][np] scaled outward normal (x, y)
    const double2 *rs;                  // [D][np] midpoint - own centroid
    const double2 *ro;                  // [D][np] midpoint image - neighbour centroid
    const double *ainv;                 // [3][np] inverse LSQ normal matrix
    const double *dtv;                  // [np] dt / V
    const double *area;                 // [np]
    const int32_t *bf_tag;              // [n_bfaces]
    const DevBC *bcs;                   // [n_bc]
    double a, b, c1, lam, dt;           // (2tau-dt)/2tau, dt/2tau, 2tau/(2tau+dt), dt/tau, dt
    double inv1l;                       // 1 / (1 + dt/tau)
    // face step: reconstruction time, and the coefficients of the face
    // distribution f_face = fc1 (fbar + fb feq_f); (dt, b, c1) for the paper's
    // scheme, (dt/2, dt/4tau, 2tau/(2tau+dt/2)) for the original one
    double dtr, fb, fc1;
    int32_t scheme;                     // 0 the paper's scheme, 1 the original one
    double rho0;                        // offset of the deviation form: f = w_i rho0 + stored value
};

// State buffers of one step: read (in) and write (out).  f is FP64 ([9][np]
// doubles) or, in the deviation form, f - w_i rho0 in FP32 (f32 / fo32).
struct DevState {
    const double *f, *W, *G;            // [9][np], [3][np], [3][np]
    double *fo, *Wo, *Go;
    const float *f32;
    float *fo32;
};

// Tiles of the fused step (see MeshBuild): headers [n_tiles][8] (g0, nt, n1,
// n2, faces), the padded per-tile tables lgid [PL], ladj [D][PA], lfc [D][PT], the
// cells of every face fcell [PF], the
// face records [3][PF] (rows l n, r_self, r_other of (x, y) pairs) and the
// least-squares weights lw [D][PA] ((x, y) pairs), with PL = nl_max,
// PA = na_max, PT = nt_max, PF = nf_max.
struct DevTiles {
    int32_t n_tiles, nl_max, na_max, nt_max, nf_max;
    const int32_t *hdr;
    const int32_t *lgid;
    const int16_t *ladj;
    const int16_t *lfc;
    const int32_t *fcell;
    const double2 *fr, *lw;             // FP64 form
    const float2 *fr32, *lw32;          // deviation form
};

// Structured step (tensor-product quad meshes): grid, periodic flags, how the
// march cuts it (strips of columns, segments of rows: so many of one cell more
// than the rest), per-column and per-row records and the boundary-condition
// entry of every boundary face of the four sides (bottom [nx], top [nx], left
// [ny], right [ny]; -1 on periodic sides).
struct DevCart {
    int32_t nx, ny, per_x, per_y;
    int32_t strips, strip_w, strip_more, segs, seg_h, seg_more;
    uint32_t inv_segs;                  // 2^32 / segs, rounded down
    const double *col;                  // [nx][kCartVals]
    const void *row;                    // [ny] CartRow of the step's arithmetic
    const int32_t *side;
};

// A row's record in the step's arithmetic: offsets of its lower and upper face
// from its centre, least-squares weights of the points below and above, height
// times the factor of the face distribution, 1 / height.
template <typename R>
struct CartRow {
    R hb, ht, wb, wt, c;
    double ih;
};

// Boxes of the structured step's form with several steps per launch: box
// columns (a power of two up to 64) and threads (one per box cell), steps K
// after which a box that does not hold the whole axis is spent, boxes per axis.
struct CartBlock {
    int32_t log_bx, threads, K, nbx, nby;
};

// One member of a batched launch: its mesh, tiles (or structured grid), both
// ping-pong buffers and the buffer index it reads at parity 0.
struct BatchInst {
    DevMesh m;
    DevTiles t;
    DevCart c;
    CartBlock b;
    void *f[2];
    double *W[2];
    double *G[2];
    int32_t parity0, lagged;
};

// Device-side batch table: the members, and for every tile slot of the
// launch grid its member and the tile's index inside that member (member -1
// for the slots past the live tiles).
struct BatchTable {
    const BatchInst *inst;
    const int2 *tmap;
};

// Plain boundary faces for the face-flux diagnostic, in the caller's order of
// its non-periodic boundary edges: the adjacent cell, the face's slot and tag,
// the cell's least-squares stencil (neighbour >= 0, -2 - tag for a boundary
// point, -1 empty) with its weights, and the face's scaled normal l n and
// midpoint offset r_self.  out [n][4]: mass flux, x- and y-momentum flux
// leaving the fluid, face density; sum [3]: the fluxes summed over one tag.
struct DevBnd {
    int32_t n;
    const int4 *hdr;                    // [n]: cell, slot, tag, 0
    const int32_t *nb;                  // [n][D]
    const double2 *w;                   // [n][D]
    const double2 *geo;                 // [n][2]: l n, r_self
    double *out;
    double *sum;
};

struct DevScratch {
    double *fbp;                        // [9][np] fbar+ at the cell centres
    double *sg;                         // [18][np] its least-squares gradient (x rows 0..8, y rows 9..17)
};

// Where a step launcher puts its kernels: on its stream, or, given a chain,
// as the next nodes of a graph under construction (each node depending on the
// previous one).  Graphs are built node by node rather than by stream
// capture, so that another thread's allocations or synchronous copies can
// never invalidate them.
struct GraphChain {
    hipGraph_t graph = nullptr;
    hipGraphNode_t last = nullptr;
};

template <typename Tup, size_t... I>
inline void kernel_arg_ptrs(Tup &t, void **p, std::index_sequence<I...>)
{
    ((p[I] = (void *)&std::get<I>(t)), ...);
}

// Launch fn<<<grid, blk, lds, st>>>(args...), or append it to the chain.
template <typename... P, typename... A>
inline hipError_t emit(void (*fn)(P...), dim3 grid, dim3 blk, size_t lds, hipStream_t st, GraphChain *gc,
                       A &&...args)
{
    std::tuple<P...> vals(std::forward<A>(args)...);
    void *ptrs[sizeof...(P) > 0 ? sizeof...(P) : 1];
    kernel_arg_ptrs(vals, ptrs, std::index_sequence_for<P...>{});
    if (!gc) return hipLaunchKernel(reinterpret_cast<const void *>(fn), grid, blk, ptrs, lds, st);
    hipKernelNodeParams kp{};
    kp.func = reinterpret_cast<void *>(fn);
    kp.gridDim = grid;
    kp.blockDim = blk;
    kp.sharedMemBytes = (unsigned)lds;
    kp.kernelParams = ptrs;
    kp.extra = nullptr;
    hipGraphNode_t node = nullptr;
    const hipError_t e = hipGraphAddKernelNode(&node, gc->graph, gc->last ? &gc->last : nullptr, gc->last ? 1 : 0, &kp);
    if (e == hipSuccess) gc->last = node;
    return e;
}

// Launchers (stream-ordered, no synchronisation).  Return the hipError_t of the launch.
hipError_t launch_grad(const DevMesh &m, const DevState &s, const DevScratch &x, hipStream_t st,
                       GraphChain *gc = nullptr);
hipError_t launch_flux_update(const DevMesh &m, const DevState &s, const DevScratch &x, int lagged, hipStream_t st,
                              GraphChain *gc = nullptr);
// Threads and LDS of one tile in a workgroup that has one or two.
struct TileShare {
    int32_t threads, bytes;
};
// Fused one-kernel step over tiles (D <= 4 slots per cell), workgroups of `block`
// threads with `per` of them to a tile (block or half of it).
// mode: 0 FP64; 1 FP32 storage of f - w_i rho0, FP32 face arithmetic; 2 FP32
// storage of f - feq(W), FP64 arithmetic.
hipError_t launch_step_tiled(const DevMesh &m, const DevTiles &t, const DevState &s, int lagged, int mode,
                             int block, int per, hipStream_t st, GraphChain *gc = nullptr);
size_t step_tiled_lds_bytes(const DevTiles &t, int mode, int n_bc);
// More local cells or faces than threads (never more than twice as many, nor
// more cells of tile and first ring than threads).
inline bool step_tiled_two(const DevTiles &t, int block) { return t.nl_max > block || t.nf_max > block; }
inline bool step_tiled_fits(const DevTiles &t, int block)
{
    return t.na_max <= block && t.nl_max <= 2 * block && t.nf_max <= 2 * block;
}
// Threads of the fused step where the caller leaves them to the library: four
// waves a tile while all tiles are on the chip at once (three per CU in FP64:
// a 45,000-cell mesh took 8.0 us a step where two waves took 8.3), two beyond (a
// 200,000-cell mesh with FP32 deviations takes 13.6 us, with four waves 17.1).
inline int step_tiled_block(const DevTiles &t, int64_t n_tiles)
{
    return n_tiles <= 768 && !step_tiled_two(t, 256) ? 256 : 128;
}
// Threads per tile of a workgroup whose threads the caller gives: half of them,
// and two tiles at a time, beyond as many tiles as the chip takes at once, where
// half the waves do more with a tile (figures: Place in step_tiled.hip).
inline int step_tiled_per(const DevTiles &t, int block, int64_t n_tiles)
{
    return block > 64 && n_tiles > 768 * 256 / block && step_tiled_fits(t, block / 2) ? block / 2 : block;
}
// Structured step of a tensor-product quad mesh, marching form (a wave per
// segment of a strip of columns), and below its batched form (members of one
// mode).
hipError_t launch_step_cart(const DevMesh &m, const DevCart &c, const DevState &s, int lagged, int mode,
                            hipStream_t st, GraphChain *gc = nullptr);
// The same, `steps` steps at once (at most B.K unless one box holds the mesh).
hipError_t launch_step_block(const DevMesh &m, const DevCart &c, const DevState &s, const CartBlock &B, int lagged,
                             int mode, int steps, hipStream_t st, GraphChain *gc = nullptr);
size_t step_block_lds_bytes(int threads, int mode, int n_bc);
inline bool block_wraps(const DevCart &c, const CartBlock &B)
{
    return c.per_x && B.nbx == 1 && c.nx <= (1 << B.log_bx);
}
// The batched form: members whose boxes have the same number of threads and
// which all wrap rows inside a box or all do not.
hipError_t launch_step_batch_block(const BatchTable &tab, bool wrap, int threads, int mode, int steps, int parity,
                                   int cap_tiles, size_t lds, hipStream_t st, GraphChain *gc = nullptr);
// LDS of a wave of the march: W and f of its last kRing rows, and besides (the
// launch's dynamic LDS) the boundary table and nine values for each row of a segment
// and the two on either side of it, for both columns outside the walls where
// one strip holds both.
constexpr int kRing = 3;
constexpr size_t kBcBytes = 4 * sizeof(double);
constexpr size_t march_ring_bytes(int mode)
{
    return (size_t)kRing * 64 * (3 * sizeof(double) + 9 * (mode == SDUGKS_FP64 ? sizeof(double) : sizeof(float)));
}
inline size_t march_lds_bytes(const DevCart &c, int n_bc, int mode)
{
    const size_t rows = c.seg_h + (c.seg_more > 0) + 4, value = mode == SDUGKS_FP32DEV ? sizeof(float) : sizeof(double);
    return n_bc * kBcBytes + (c.per_x ? 0 : (c.strips == 1 ? 2 : 1) * rows * 9 * value);
}
// Waves of the march on a CU at once: two on each of its four SIMDs, the most that
// the registers allow, where the LDS (160 KB, allocated in units of 1280 bytes) holds them.
inline int march_waves_per_cu(size_t lds)
{
    const int fit = (int)(160 * 1024 / ((lds + 1279) / 1280 * 1280));
    return fit < 8 ? (fit < 1 ? 1 : fit) : 8;
}
// Workgroups of a structured instance cut into strips and segments.
inline int32_t cart_groups(const DevCart &c) { return c.strips * c.segs; }
hipError_t launch_step_batch_cart(const BatchTable &tab, int mode, int parity, int cap_tiles, size_t lds,
                                  hipStream_t st, GraphChain *gc = nullptr);
// Batched fused step over the tiles of all members (same D class and mode).
hipError_t launch_step_batch(const BatchTable &tab, int D, int mode, bool two, int parity, int cap_tiles, size_t lds_tile,
                             int block, int per, hipStream_t st, GraphChain *gc = nullptr);
// Deterministic reductions of the residual / mass / finiteness check: writes
// out4 = {sum |u-u_snap|^2, sum |u_snap|^2, sum V rho, count of non-finite}.
// snap = [2][np] (U, V); update_snap re-snapshots.
hipError_t launch_reduce(const DevMesh &m, const double *W, double *snap, int update_snap, double *partials,
                         double *out4, hipStream_t st);
// Boundary face fluxes on the state s (mode: the storage of f, as for the
// step), then their sums over the faces of `tag` (all when tag < 0).
hipError_t launch_boundary_flux(const DevMesh &m, const DevState &s, const DevBnd &q, int mode, int tag, hipStream_t st);
// One member of a batched residual: its cells, current W, areas, snapshot
// (re-snapshotted) and its own partial sums.
struct ReduceJob {
    int32_t nc, np;
    const double *W;
    const double *area;
    double *snap;
    double *partials;
};
// Residuals of n members at once: out [n][4] as launch_reduce's out4 each.
hipError_t launch_reduce_batch(const ReduceJob *jobs, int n, double *out, hipStream_t st);
// Residuals of n members without any allocation: the per-member results
// [n][4] go to the file-scope scratch array of noalloc.hip (at most
// kNoAllocMaxMembers members), the job table travels in the kernel arguments
// (kNoAllocPack members per launch).
constexpr int kNoAllocMaxMembers = 1024;
constexpr int kNoAllocPack = 32;
constexpr int kNoAllocMaxDevices = 64;
struct ReducePack {
    ReduceJob jobs[kNoAllocPack];
};
// The device address of this device's scratch array ([kNoAllocMaxMembers][4]
// doubles), looked up once per device.
hipError_t noalloc_scratch(int device, double **out);
hipError_t launch_reduce_packs(const ReduceJob *jobs, int n, double *out, hipStream_t st);
// f = feq of the macros m3 = [3][np] (rho, u, v) (FP64 f, or with f32 the
// FP32 deviation from w_i rho0, or zero -- the non-equilibrium part -- when
// rho0 < 0), W, G = 0 and the residual snapshot.
hipError_t launch_set_equilibrium(int nc, int np, const double *m3, double *f, float *f32, double rho0, double *W,
                                  double *G, double *snap, hipStream_t st);
// State between the caller's cell order (cell-major arrays, n cells from c0 on)
// and the internal rows: macros or W, G ([n][3]) or f ([n][9]) out, W, G or f in.
// kGetF and kPutF need the W that goes with f; kPutRows3 also sets the residual's
// snapshot where snap is given.
enum StateMove { kGetMacros, kGetRows3, kPutRows3, kGetF, kPutF };
struct StateLayout {
    int32_t np, mode;
    const int32_t *iperm;               // [nc] internal index of a caller's cell, NULL where the orders agree
    double rho0, k;                     // k: dt / (2 tau) of the original scheme's variable, else 0
};
hipError_t launch_state_io(StateMove move, const StateLayout &l, int c0, int n, const double *W, void *rows, double *snap,
                           double *host_order, hipStream_t st);
// The same f (as stored) and W in every cell, G = 0, snapshot = its velocity.
hipError_t launch_set_uniform(int nc, int np, const double *f9, const double *W3, double *f, float *f32, double *W,
                              double *G, double *snap, hipStream_t st);
// y = 1 / x as the steps form it of their densities.
hipError_t launch_reciprocal(int n, const double *x, double *y, hipStream_t st);
// The buffer index (bit k) that each of n members of a batch table reads at parity 0;
// the bits travel in the kernel arguments.
constexpr int kParityPack = 1024;
struct ParityPack {
    uint32_t bits[kParityPack / 32];
};
hipError_t launch_set_parity(BatchInst *inst, int n, const ParityPack &p, hipStream_t st);
// *p = NaN, p pointing at a double (bytes 8) or a float (bytes 4): failure injection.
hipError_t launch_poke_nan(void *p, int bytes, hipStream_t st);

constexpr int kReduceBlocks = 256;

}  // namespace sdg
