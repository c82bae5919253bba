// Structured step, several steps per launch, for meshes that are too small to
// fill the chip: there a launch costs a fixed time (its start, the load of the
// state and the chain of phases), about 3 us, against 1.5 to 2.5 us for a step
// whose state is on the chip.  A workgroup holds a box of cells, one thread
// per cell with f and W in registers, and advances it `steps` steps; per step
// the cells within two of the box's edge lose their meaning (a step reads two
// rings of neighbours), so a box of B cells along an axis writes the B - 4 K
// in its middle after K steps, more where it ends at a wall.  A mesh that fits
// one box loses none and takes all steps of a call in one launch.
//
// A row of the box lies in one wave, so neighbours along x are read by wave
// shifts (by lane permutation where a periodic mesh wraps inside the box),
// neighbours along y through LDS: fbar+, then the upper sides, then the fluxes
// through the lower faces, with one barrier each.  The arithmetic is that of
// the marching step (cart_math.h), expression by expression: the results are
// the same bits.
//
// What bounds it is the latency of a step's chain (three barriers, wave shifts,
// one cell per lane).  us per step against one workgroup per tile and launch:
// 4 x 32 cells FP64 6.9 -> 2.2, 48 x 48 FP64 8.0 -> 3.2, 101 x 101 FP32
// deviations 8.1 -> 3.4, 256 x 256 10.3 -> 6.3, FP64 10.8 -> 7.3.  With the march
// instead 256 x 256 takes 9.7 and 10.6; 512 x 512 15.3 against 16.3 (FP32
// deviations), where the two meet.
#include <cstdint>
#include <type_traits>
#include <utility>

#include "cart_math.h"
#include "device.h"
#include "mesh.h"
#include "step_common.h"

namespace sdg {

namespace {

// Slots of the boundary states below and above the mesh: two rows of at most 64 cells.
constexpr int kGhosts = 128;

// Boxes along one axis: cells [a, b) are written by box `t`, whose first cell
// is `o` (outside the mesh: ghost cells or, periodic, wrapped ones).
struct Span {
    int o, a, b;
};
__device__ __forceinline__ Span span(int n, bool per, int B, int pad, int K, int boxes, int t)
{
    if (boxes == 1 && (per ? n <= B : n + 2 * pad <= B)) return {per ? 0 : -pad, 0, n};
    const int T = B - 4 * K;
    if (per) return {t * T - 2 * K, t * T, t * T + T < n ? t * T + T : n};
    const int first = B - pad - 2 * K, a = t == 0 ? 0 : first + (t - 1) * T;
    return {t == 0 ? -pad : a - 2 * K, a, t == boxes - 1 ? n : first + t * T};
}

// Values of the cells to the right and left (lane + 1, lane - 1, or the lanes
// given where rows wrap).
template <bool WRAP>
struct Lanes {
    int next4, prev4;                   // byte indices of the lanes (WRAP)
    __device__ __forceinline__ int perm(int at, int v) const { return __builtin_amdgcn_ds_bpermute(at, v); }
    template <int CTRL>
    __device__ __forceinline__ int move(int at, int v) const
    {
        if constexpr (WRAP) return perm(at, v);
        else return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
    }
    template <int CTRL>
    __device__ __forceinline__ float get(int at, float v) const { return __int_as_float(move<CTRL>(at, __float_as_int(v))); }
    template <int CTRL>
    __device__ __forceinline__ double get(int at, double v) const
    {
        return __hiloint2double(move<CTRL>(at, __double2hiint(v)), move<CTRL>(at, __double2loint(v)));
    }
    template <typename R>
    __device__ __forceinline__ R next(R v) const { return get<0x130>(next4, v); }
    template <typename R>
    __device__ __forceinline__ R prev(R v) const { return get<0x138>(prev4, v); }
};

template <typename T>
__device__ __forceinline__ T ld(const T *base, size_t i) { return gin(base)[i]; }

// `steps` steps of box t of an instance by the whole workgroup (NT = B.threads
// threads (LDS offsets are then constants), at least as many as boundary entries); LDS: see step_block_lds_bytes.
template <int PM, bool WRAP, int NT>
__device__ __forceinline__ void block_steps(const DevMesh &m, const DevCart &cg, const DevState &s, const CartBlock &B,
                                            int lagged, int steps, int t)
{
    using R = Arith<PM>;
    using V = Stored<PM>;
    extern __shared__ double smem[];
    const int bx = 1 << B.log_bx, by = NT >> B.log_bx;
    constexpr int NG = NT + kGhosts;
    R *const sfb = reinterpret_cast<R *>(smem);          // [9][NG] fbar+; below and above the mesh
    R *const sup = sfb + 9 * NG;                         // [5][NT] upper sides
    R *const sfl = sup + 5 * NT;                         // [6][NT] fluxes through the lower faces
    const int nx = cg.nx, ny = cg.ny;
    const size_t np = (size_t)m.np;
    const int tid = (int)threadIdx.x;
    const int ix = tid & (bx - 1), iy = tid >> B.log_bx;
    const int ty = t / B.nbx, tx = t - ty * B.nbx;
    const Span sx = span(nx, cg.per_x, bx, 1, B.K, B.nbx, tx), sy = span(ny, cg.per_y, by, 0, B.K, B.nby, ty);
    const int gi = sx.o + ix, gj = sy.o + iy;            // this thread's cell, before wrapping
    const bool wrap_y = cg.per_y && B.nby == 1 && ny <= by;
    // clamped or wrapped into the mesh for reading
    int ci = gi, cj = gj;
    if (cg.per_x) { ci = ci < 0 ? ci + nx : (ci >= nx ? ci - nx : ci); ci = ci >= nx ? nx - 1 : ci; }
    else ci = ci < 0 ? 0 : (ci >= nx ? nx - 1 : ci);
    if (cg.per_y) { cj = cj < 0 ? cj + ny : (cj >= ny ? cj - ny : cj); cj = cj >= ny ? ny - 1 : cj; }
    else cj = cj >= ny ? ny - 1 : cj;
    const size_t g = (size_t)(uint32_t)cj * (uint32_t)nx + (uint32_t)ci;
    const bool out = gi >= sx.a && gi < sx.b && gj >= sy.a && gj < sy.b;
    // state
    double W[3], G[3] = {0.0, 0.0, 0.0};
    V f[9];
#pragma unroll
    for (int i = 0; i < 3; i++) W[i] = ld(s.W, i * np + g);
#pragma unroll
    for (int i = 0; i < 9; i++) {
        if constexpr (PM == SDUGKS_FP64) f[i] = ld(s.f, i * np + g);
        else f[i] = ld(s.f32, i * np + g);
    }
    if (lagged)
        for (int i = 0; i < 3; i++) G[i] = ld(s.G, i * np + g);
    // walls of this cell: columns 0 and nx - 1, rows 0 and ny - 1; the thread
    // left of column 0 computes the wall face there
    const bool ghost_l = !cg.per_x && gi == -1, wall_l = !cg.per_x && gi == 0, wall_r = !cg.per_x && gi == nx - 1;
    const bool wall_b = !cg.per_y && gj == 0, wall_t = !cg.per_y && gj == ny - 1;
    const bool any_x = __any(wall_l || wall_r || ghost_l), any_b = __any(wall_b), any_t = __any(wall_t);
    // their boundary entries, 8 bits each (a structured mesh has at most 64), and the table in LDS
    int tags = 0;
    if (wall_l || wall_r) tags |= gin(cg.side)[2 * nx + (wall_l ? 0 : ny) + cj];
    if (wall_b) tags |= gin(cg.side)[ci] << 8;
    if (wall_t) tags |= gin(cg.side)[nx + ci] << 16;
    WallBC *const bcs = reinterpret_cast<WallBC *>(sfl + 6 * NT);
    if (tid < m.n_bc) {
        const DevBC b = gin(m.bcs)[tid];
        bcs[tid] = {(double)b.type, b.rho, b.u, b.v};
    }
    __syncthreads();
    // records
    const gmem<double> *const col = gin(cg.col) + (size_t)ci * kCartVals;
    const gmem<CartRow<R>> *const row = gin((const CartRow<R> *)cg.row) + cj;
    const Factors<PM> c(m);
    const R hl = (R)col[1], hr = (R)col[2], wl = (R)col[3], wr = (R)col[4];
    const R Cy = (R)col[0] * c.c1;
    const R hb = row->hb, ht = row->ht, wb = row->wb, wt = row->wt;
    const R Cx = row->c;
    const double dtv = (m.dt * col[5]) * row->ih;
    // neighbours: lanes along x, LDS slots along y
    Lanes<WRAP> ln{0, 0};
    if constexpr (WRAP) {
        const int lane = tid & 63, base = lane - ix;
        ln.next4 = 4 * (base + (ix + 1 >= nx ? 0 : ix + 1));
        ln.prev4 = 4 * (base + (ix == 0 ? nx - 1 : (ix < nx ? ix - 1 : ix)));
    }
    const int up = wrap_y && iy + 1 == ny ? ix : (iy + 1 < by ? tid + bx : tid);
    const int dn = iy > 0 ? tid - bx : (wrap_y ? (ny - 1) * bx + ix : tid);
    const int upb = wall_t ? NT + bx + ix : up, dnb = wall_b ? NT + ix : dn;     // of fbar+

    for (int n = 0; n < steps; n++) {
        R fb[9];
        cell_plus<PM>(m, c, W[0], W[1], W[2], f, fb);
#pragma unroll
        for (int i = 0; i < 9; i++) sfb[i * NG + tid] = fb[i];
        // boundary states below and above the mesh, beside the cells
        if (any_b || any_t) {
            R df[9];
            if (wall_b) {
                wall_diff<PM>(m, bcs[(tags >> 8) & 255], W[0], W[1], W[2], df);
#pragma unroll
                for (int i = 0; i < 9; i++) sfb[i * NG + NT + ix] = fb[i] + df[i];
            }
            if (wall_t) {
                wall_diff<PM>(m, bcs[tags >> 16], W[0], W[1], W[2], df);
#pragma unroll
                for (int i = 0; i < 9; i++) sfb[i * NG + NT + bx + ix] = fb[i] + df[i];
            }
        }
        // slopes along x
        R gx[9], gy[9], dl[3], dr[3];
        {
            R fg[9];
#pragma unroll
            for (int i = 0; i < 9; i++) fg[i] = 0;
            if (any_x) {
                wall_diff<PM>(m, bcs[tags & 255], W[0], W[1], W[2], fg);
#pragma unroll
                for (int i = 0; i < 9; i++) fg[i] = fb[i] + fg[i];
            }
#pragma unroll
            for (int i = 0; i < 9; i++) {
                const R dn_ = ln.next(fb[i]) - fb[i];
                const R dp = wall_r ? fg[i] - fb[i] : dn_;
                const R dq = ln.prev(dn_);
                const R dm = wall_l ? fb[i] - fg[i] : dq;
                gx[i] = slope(wl, wr, dm, dp);
                for (int e = 0; e < 3; e++) {
                    if (i == cP[0][e]) dl[e] = dm;
                    if (i == cN[0][e]) dr[e] = dp;
                }
            }
        }
        __syncthreads();
        // and along y
        R db[3], dt[3];
        {
#pragma unroll
            for (int i = 0; i < 9; i++) {
                const R dm = fb[i] - sfb[i * NG + dnb], dp = sfb[i * NG + upb] - fb[i];
                gy[i] = slope(wb, wt, dm, dp);
                for (int e = 0; e < 3; e++) {
                    if (i == cP[1][e]) db[e] = dm;
                    if (i == cN[1][e]) dt[e] = dp;
                }
            }
        }
        R bkx[9], bky[9];
        carried<0>(c.dt, fb, gx, gy, bkx);
        carried<1>(c.dt, fb, gx, gy, bky);
        Side<R> lower, upper;
        sides<1>(c.dt, hb, ht, bky, gy, lower, upper);
#pragma unroll
        for (int e = 0; e < 3; e++) sup[e * NT + tid] = upper.c[e];
        sup[3 * NT + tid] = upper.s;
        sup[4 * NT + tid] = upper.d;
        // x faces
        Outflow acc;
        {
            Side<R> left, right;
            sides<0>(c.dt, hl, hr, bkx, gx, left, right);
            Side<R> nb{{ln.next(left.c[0]), ln.next(left.c[1]), ln.next(left.c[2])}, ln.next(left.s), ln.next(left.d)};
            if (any_x) {
#pragma unroll
                for (int e = 0; e < 3; e++) {
                    const R v = ln.next(entering<0, true>(c.dt, bkx, gx, e) - dl[e]);
                    right.c[e] = ghost_l ? v : right.c[e];
                    nb.c[e] = wall_r ? entering<0, false>(c.dt, bkx, gx, e) + dr[e] : nb.c[e];
                }
                right.s = ghost_l ? nb.s : right.s;
                right.d = ghost_l ? nb.d : right.d;
                nb.s = wall_r ? right.s : nb.s;
                nb.d = wall_r ? right.d : nb.d;
            }
            R pr[3], nr[3], pl[3], nl[3];
            face_flux<PM>(m, right, nb, Cx, Cx * c.k1, Cx * c.k5, pr, nr);
#pragma unroll
            for (int e = 0; e < 3; e++) { pl[e] = ln.prev(pr[e]); nl[e] = ln.prev(nr[e]); }
            outflow_x<0>(acc, pr, nr, pl, nl);
        }
        __syncthreads();
        // y faces: each thread the one below its cell
        Side<R> top{{sup[dn], sup[NT + dn], sup[2 * NT + dn]}, sup[3 * NT + dn], sup[4 * NT + dn]};
#pragma unroll
        for (int e = 0; e < 3; e++) top.c[e] = wall_b ? entering<1, true>(c.dt, bky, gy, e) - db[e] : top.c[e];
        top.s = wall_b ? lower.s : top.s;
        top.d = wall_b ? lower.d : top.d;
        R p[3], q[3];
        face_flux<PM>(m, top, lower, Cy, Cy * c.k1, Cy * c.k5, p, q);
#pragma unroll
        for (int e = 0; e < 3; e++) { sfl[e * NT + tid] = p[e]; sfl[(3 + e) * NT + tid] = q[e]; }
        outflow_below(acc, p, q);
        R pw[3], qw[3];
        if (any_t) {
            // the face between the last row and the upper wall
            const Side<R> in{{entering<1, false>(c.dt, bky, gy, 0) + dt[0], entering<1, false>(c.dt, bky, gy, 1) + dt[1],
                              entering<1, false>(c.dt, bky, gy, 2) + dt[2]},
                             upper.s, upper.d};
            face_flux<PM>(m, upper, in, Cy, Cy * c.k1, Cy * c.k5, pw, qw);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 3; e++) { p[e] = sfl[e * NT + up]; q[e] = sfl[(3 + e) * NT + up]; }
        if (any_t) {
#pragma unroll
            for (int e = 0; e < 3; e++) { p[e] = wall_t ? pw[e] : p[e]; q[e] = wall_t ? qw[e] : q[e]; }
        }
        outflow_above(acc, p, q);
        double Wn[3];
        V v[9];
        cell_update<PM>(m, lagged, dtv, W[0], W[1], W[2], acc, f, G, Wn[0], Wn[1], Wn[2], v);
#pragma unroll
        for (int i = 0; i < 3; i++) W[i] = Wn[i];
#pragma unroll
        for (int i = 0; i < 9; i++) f[i] = v[i];
    }
    if (!out) return;
#pragma unroll
    for (int i = 0; i < 3; i++) gout(s.Wo)[i * np + g] = W[i];
#pragma unroll
    for (int i = 0; i < 9; i++) {
        if constexpr (PM == SDUGKS_FP64) gout(s.fo)[i * np + g] = f[i];
        else gout(s.fo32)[i * np + g] = f[i];
    }
    if (lagged)
        for (int i = 0; i < 3; i++) gout(s.Go)[i * np + g] = G[i];
}

template <int PM, bool WRAP, int NT>
__global__ void __launch_bounds__(NT) k_step_block(DevMesh m, DevCart c, DevState s, CartBlock B, int lagged, int steps)
{
    const int x = (int)(blockIdx.x % kXcds);
    const int t = xcd_range_start((int)gridDim.x, x) + (int)(blockIdx.x / kXcds);
    block_steps<PM, WRAP, NT>(m, c, s, B, lagged, steps, t);
}

// Batched form: as the batched general step, the slot map gives each workgroup
// its member and box.
template <int PM, bool WRAP, int NT>
__global__ void __launch_bounds__(NT) k_step_batch_block(BatchTable tab, int steps, int parity)
{
    const int x = (int)(blockIdx.x % kXcds);
    const int per = (int)gridDim.x / kXcds;
    const unsigned long long slot = reinterpret_cast<const unsigned long long *>(tab.tmap)[x * per + (int)(blockIdx.x / kXcds)];
    const int member = (int)(unsigned)slot, box = (int)(unsigned)(slot >> 32);
    if (member < 0) return;
    const BatchInst &in = tab.inst[member];
    const DevMesh m = in.m;
    const DevCart cg = in.c;
    const CartBlock B = in.b;
    block_steps<PM, WRAP, NT>(m, cg, batch_state(in, parity), B, in.lagged, steps, box);
}

}  // namespace

size_t step_block_lds_bytes(int threads, int mode, int n_bc)
{
        // fbar+ of the cells and the boundary states, upper sides, fluxes
    return (20 * (size_t)threads + 9 * kGhosts) * (mode == SDUGKS_FP32DEV ? sizeof(float) : sizeof(double)) +
           n_bc * sizeof(WallBC);
}

hipError_t launch_step_block(const DevMesh &m, const DevCart &c, const DevState &s, const CartBlock &B, int lagged,
                             int mode, int steps, hipStream_t st, GraphChain *gc)
{
    const dim3 grid((unsigned)(B.nbx * B.nby)), blk((unsigned)B.threads);
    const size_t lds = step_block_lds_bytes(B.threads, mode, m.n_bc);
    const bool wrap = block_wraps(c, B);
#define SDG_NT(PP, WW, NN) emit(&k_step_block<PP, WW, NN>, grid, blk, lds, st, gc, m, c, s, B, lagged, steps)
#define SDG_BLOCK(PP, WW) \
    return B.threads == 128 ? SDG_NT(PP, WW, 128) : (B.threads == 256 ? SDG_NT(PP, WW, 256) : SDG_NT(PP, WW, 512))
    if (mode == SDUGKS_FP32DEV) { if (wrap) SDG_BLOCK(SDUGKS_FP32DEV, true); SDG_BLOCK(SDUGKS_FP32DEV, false); }
    if (mode == SDUGKS_FP32NEQ) { if (wrap) SDG_BLOCK(SDUGKS_FP32NEQ, true); SDG_BLOCK(SDUGKS_FP32NEQ, false); }
    if (wrap) SDG_BLOCK(SDUGKS_FP64, true);
    SDG_BLOCK(SDUGKS_FP64, false);
#undef SDG_BLOCK
#undef SDG_NT
}

hipError_t launch_step_batch_block(const BatchTable &tab, bool wrap, int threads, int mode, int steps, int parity,
                                   int cap_tiles, size_t lds, hipStream_t st, GraphChain *gc)
{
    const dim3 grid((unsigned)batch_grid(cap_tiles)), blk((unsigned)threads);
#define SDG_NT(PP, WW, NN) emit(&k_step_batch_block<PP, WW, NN>, grid, blk, lds, st, gc, tab, steps, parity)
#define SDG_BLOCK(PP, WW) \
    return threads == 128 ? SDG_NT(PP, WW, 128) : (threads == 256 ? SDG_NT(PP, WW, 256) : SDG_NT(PP, WW, 512))
    if (mode == SDUGKS_FP32DEV) { if (wrap) SDG_BLOCK(SDUGKS_FP32DEV, true); SDG_BLOCK(SDUGKS_FP32DEV, false); }
    if (mode == SDUGKS_FP32NEQ) { if (wrap) SDG_BLOCK(SDUGKS_FP32NEQ, true); SDG_BLOCK(SDUGKS_FP32NEQ, false); }
    if (wrap) SDG_BLOCK(SDUGKS_FP64, true);
    SDG_BLOCK(SDUGKS_FP64, false);
#undef SDG_BLOCK
#undef SDG_NT
}

}  // namespace sdg
