// Structured sDUGKS time step (Zhong et al., arXiv:2007.07347, Section II,
// the eleven-step summary) for tensor-product quad meshes: the cells are the
// rectangles of two coordinate arrays, stored row by row, so every face is
// normal to x or to y, each cell's least-squares stencil is its four face
// neighbours (or the wall face midpoints), and nothing about the geometry needs
// a table beyond one record per column and per row.
//
// One wave takes a strip of up to 60 columns (one lane per column, two halo
// columns on either side) and marches along a segment of its rows.  A lane
// keeps what the rows behind it still need in registers (their W and f in the
// wave's own LDS) and reads its left and right neighbours by wave shifts, so no
// wave waits for another and no value is computed twice but those of the halo
// columns and of the two rows before and after the segment.  When row k arrives:
//
//   fbar+ of row k = a f + b feq(W) (Eq. fbarplus), after which the loads of
//     row k + 1 are issued into the same registers;
//   row k - 1: the least-squares slopes (the LLSR normal equations, diagonal on
//     this stencil), the reconstruction at the foot points of its four faces
//     (Eq. fbpsource), the fluxes of its x faces and of the y face below it
//     (Eqs. f_t_n+1, MesoFlux);
//   row k - 2: with the flux of the face above it, W^{n+1} (Eq. MacroUpdate),
//     feq^{n+1} and f^{n+1} (Eq. fn+1).
//
// A face shared by two strips or segments is evaluated by both from identical
// operands, so the flux that leaves one cell enters the other exactly.
// Boundary faces follow Section III as in the general step: velocities entering
// the fluid take the boundary state's fbar+ carried to the foot point with the
// adjacent cell's slopes, the others the adjacent cell's reconstruction; the
// boundary state is a least-squares point at the face midpoint.  The lane (or
// row) outside a wall stands for the boundary state.
//
// What bounds it is memory: with the arithmetic left out the same accesses take
// 29.0 of 33.3 us on 1024 x 1024 cells in FP32 deviations and 43.7 of 47.2 in
// FP64 (12 values in and out per cell, each array a stream of some 240 bytes per
// wave and row), and three waves on a SIMD instead of two, requests of two rows
// ahead, or cache lines touched before they are requested change nothing or cost
// 5 to 20 %; so do non-temporal stores.  Before it, one workgroup per 16 x 14 or
// 16 x 7 cells with their halo in LDS: 52.8 and 86.7 us, 1430 lane instructions
// per cell against 550; now 31.5 and 44.7 (2048 x 2048 cells 129 and 227, FP64 reading
// and writing 1.04 GB at 4.6 TB/s).
#include <cstdint>
#include <type_traits>
#include <utility>

#include "cart_math.h"
#include "d2q9.h"
#include "device.h"
#include "mesh.h"
#include "step_common.h"

namespace sdg {

namespace {

// A value every lane reads alike, through the constant cache (tables that no
// kernel writes).
template <typename T>
__device__ __forceinline__ T ld_uniform(const T *p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(4))) T *)p;
#else
    return *p;
#endif
}

// N rows of a pitched array at one cell: `base` points at the wave's mesh row
// in the first of them (a scalar), `off` is the lane's byte offset in the row.
// The base steps from row to row in scalar registers; kept opaque, or the
// compiler holds N pointers per array across the whole march and spills them
// (and so is the offset, or its widened copy is held and added by every lane).
template <typename T>
__device__ __forceinline__ void opaque(T *&p, uint32_t &off)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(p), "+v"(off));
#endif
}
template <int N, typename T>
__device__ __forceinline__ void ld_rows(const T *base, size_t pitch, uint32_t off, T *v)
{
    const gmem<char> *p = (const gmem<char> *)gin(base);
#pragma unroll
    for (int i = 0; i < N; i++) {
        opaque(p, off);
        v[i] = *(const gmem<T> *)(p + off);
        p += pitch * sizeof(T);
    }
}
template <int N, typename T>
__device__ __forceinline__ void st_rows(T *base, size_t pitch, uint32_t off, const T *v)
{
    gmem<char> *p = (gmem<char> *)gout(base);
#pragma unroll
    for (int i = 0; i < N; i++) {
        opaque(p, off);
        *(gmem<T> *)(p + off) = v[i];
        p += pitch * sizeof(T);
    }
}

// The value of the next lane (column + 1) or of the previous one.
template <int CTRL>
__device__ __forceinline__ float shift(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double shift(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
constexpr int kNext = 0x130, kPrev = 0x138;   // wave_shl:1, wave_shr:1
template <int CTRL, typename R>
__device__ __forceinline__ Side<R> shift(const Side<R> &v)
{
    return {{shift<CTRL>(v.c[0]), shift<CTRL>(v.c[1]), shift<CTRL>(v.c[2])}, shift<CTRL>(v.s), shift<CTRL>(v.d)};
}

template <int PM>
struct Ring {
    double W[kRing][3][64];
    Stored<PM> f[kRing][9][64];
};
static_assert(sizeof(Ring<SDUGKS_FP64>) == march_ring_bytes(SDUGKS_FP64) &&
                  sizeof(Ring<SDUGKS_FP32DEV>) == march_ring_bytes(SDUGKS_FP32DEV) && sizeof(WallBC) == kBcBytes,
              "the march's LDS as the planner counts it");

// One time step of rows [j0, j1) of the columns [i0, i0 + w), w <= 60, by one
// wave, from the lowest row up or (DOWN) from the highest down.  Where
// neighbouring segments march in opposite directions, both come to the rows they
// share at the same time and the second finds them in L2 (1024 x 1024 cells, FP32
// deviations: 86 MB read per step against 115, 63 being the state).  Marching
// down, march row k is mesh row j0 + j1 - 1 - k; the code below follows march rows.
template <int PM, bool DOWN>
struct March {
    using R = Arith<PM>;
    using V = Stored<PM>;

    const DevMesh &m;
    const DevCart &cg;
    const DevState &s;
    const int lagged, j0, j1;
    size_t np;
    int cc;
    int kend, klow, khigh;              // march rows below kend are read; those outside the walls (far away where periodic)
    bool out, wall_r, ghost_l, ghost_r, at_l, at_r, edge;
    uint32_t offv, offw;                // byte offsets of this lane's column in a row of f, of W
    const Factors<PM> c;
    R hl, hr, wl, wr, Cy, Cy1, Cy5;
    double icol;
    // requested: W and f of the next row
    double W[3];
    V fv[9];
    const WallBC *const bcs;
    // W and f of the last kRing rows, [row % kRing][value][lane]: the wave's own LDS
    double *const lw;
    V *const lf;
    // fbar+ of the boundary states in the columns outside the walls less the cell's: rows of
    // the march, nine values each, for the left column and then the right
    R *const lx;

    __device__ __forceinline__ March(const DevMesh &m_, const DevCart &c_, const DevState &s_, int lagged_, int i0,
                                     int w, int j0_, int j1_, Ring<PM> &ring, const WallBC *bcs_, R *lx_)
        : m(m_), cg(c_), s(s_), lagged(lagged_), j0(j0_), j1(j1_), c(m_), bcs(bcs_), lw(ring.W[0][0] + (threadIdx.x & 63)),
          lf(ring.f[0][0] + (threadIdx.x & 63)), lx(lx_)
    {
        const int nx = cg.nx;
        np = (size_t)m.np;
        const int lane = (int)(threadIdx.x & 63);
        const int ci = i0 - 2 + (lane < w + 3 ? lane : w + 3);          // this lane's column, before wrapping
        if (cg.per_x) {
            cc = ci < 0 ? ci + nx : (ci >= nx ? ci - nx : ci);
        } else {
            cc = ci < 0 ? 0 : (ci >= nx ? nx - 1 : ci);
        }
        out = lane >= 2 && lane < w + 2;                // this lane's cells are written
        // the columns outside the walls hold boundary states; whether the strip has one
        at_l = !cg.per_x && i0 <= 1;
        at_r = !cg.per_x && i0 + w + 1 >= nx;
        edge = at_l || at_r;
        ghost_l = at_l && ci == -1;
        ghost_r = at_r && ci == nx;
        wall_r = !cg.per_x && ci == nx - 1;
        offv = (uint32_t)cc * (uint32_t)sizeof(V);
        offw = (uint32_t)cc * 8u;
        const gmem<double> *const col = gin(cg.col) + (size_t)cc * kCartVals;
        hl = (R)col[1];
        hr = (R)col[2];
        wl = (R)col[3];
        wr = (R)col[4];
        icol = m.dt * col[5];
        Cy = (R)col[0] * c.c1;
        Cy1 = Cy * c.k1;
        Cy5 = Cy * c.k5;
    }

    __device__ __forceinline__ size_t at(int row) const { return (size_t)(uint32_t)row * (uint32_t)cg.nx; }
    // mesh row of march row k: wrapped where periodic, else that inside the wall
    __device__ __forceinline__ int mesh_row(int k) const
    {
        const int j = DOWN ? j0 + j1 - 1 - k : k;
        if (cg.per_y) return j < 0 ? j + cg.ny : (j >= cg.ny ? j - cg.ny : j);
        return j < 0 ? 0 : (j >= cg.ny ? cg.ny - 1 : j);
    }
    __device__ __forceinline__ CartRow<R> record(int row) const { return ld_uniform((const CartRow<R> *)cg.row + row); }
    __device__ __forceinline__ void request(int row)
    {
        const size_t g = at(row);
        ld_rows<3>(s.W + g, np, offw, W);
        if constexpr (PM == SDUGKS_FP64) ld_rows<9>(s.f + g, np, offv, fv);
        else ld_rows<9>(s.f32 + g, np, offv, fv);
    }
    // Wait for the requested row here, before the update's stores are issued:
    // the counter of outstanding accesses is in order, so a wait at the next
    // row's first use would wait for those stores too.
    __device__ __forceinline__ void settle()
    {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
        for (int i = 0; i < 3; i++) asm volatile("" : "+v"(W[i]));
#pragma unroll
        for (int i = 0; i < 9; i++) asm volatile("" : "+v"(fv[i]));
#endif
    }
    // The boundary states' part in the columns outside the walls, one lane per row from row k on:
    // in the march it took every lane of the strip a fifth of the row's time.
    __device__ __forceinline__ void columns(int k, int rows) const
    {
        for (int n = (int)(threadIdx.x & 63); n < rows; n += 64) {
            int j = DOWN ? j0 + j1 - 1 - (k + n) : k + n;
            if (cg.per_y) j = j < 0 ? j + cg.ny : j % cg.ny;
            else j = j < 0 ? 0 : (j >= cg.ny ? cg.ny - 1 : j);
            const gmem<double> *const Wj = gin(s.W) + at(j);
            auto column = [&](int i, int tags, R *to) {
                R df[9];
                wall_diff<PM>(m, bcs[gin(cg.side)[tags + j]], Wj[i], Wj[np + i], Wj[2 * np + i], df);
#pragma unroll
                for (int e = 0; e < 9; e++) to[n * 9 + e] = df[e];
            };
            if (at_l) column(0, 2 * cg.nx, lx);
            if (at_r) column(cg.nx - 1, 2 * cg.nx + cg.ny, lx + (at_l ? rows * 9 : 0));
        }
    }
    // fbar+ of row k, requested before; the cells outside the walls read the cell inside and hold the boundary state
    __device__ __forceinline__ void arrive(int k, R fb[9]) const
    {
        cell_plus<PM>(m, c, W[0], W[1], W[2], fv, fb);
        if (k == klow || k == khigh) {
            const int tag = gin(cg.side)[((k == klow) != DOWN ? 0 : cg.nx) + cc];
            R df[9];
            wall_diff<PM>(m, bcs[tag], W[0], W[1], W[2], df);
#pragma unroll
            for (int i = 0; i < 9; i++) fb[i] += df[i];
        } else if (edge && (ghost_l || ghost_r)) {
#pragma unroll
            for (int i = 0; i < 9; i++) fb[i] += wx[i];
        }
    }
    // W and f of the row in ring slot t, put there when it arrived
    __device__ __forceinline__ void keep(int t) const
    {
#pragma unroll
        for (int i = 0; i < 3; i++) lw[(t * 3 + i) * 64] = W[i];
#pragma unroll
        for (int i = 0; i < 9; i++) lf[(t * 9 + i) * 64] = fv[i];
    }
    __device__ __forceinline__ void kept(int t, double Wp[3], V fo[9]) const
    {
#pragma unroll
        for (int i = 0; i < 3; i++) Wp[i] = lw[(t * 3 + i) * 64];
#pragma unroll
        for (int i = 0; i < 9; i++) fo[i] = lf[(t * 9 + i) * 64];
    }

    // State of the march between rows.
    R fbp[9], dyp[9];                   // of row k - 1: fbar+, and its differences to row k - 2
    Side<R> top;                        // of row k - 2: its side towards row k - 1,
    R px[3], nx[3], py[3], ny[3];       // the fluxes through its upper x face and the y face to row k - 3
    double ip;                          // and 1 / height
    CartRow<R> rq;                      // record of row k - 1
    int t, row;                         // ring slot of row k, its index (wrapped, or inside the wall)
    const R *wx;                        // the part above of row k in this lane's column, where it is outside

    // Row k arrives.
    template <bool UPDATE>
    __device__ __forceinline__ void step(int k)
    {
        const int q = k - 1, next = mesh_row(k + 1);
        const CartRow<R> rk = record(row);
        R fb[9], dy[9];
        arrive(k, fb);
        keep(t);
        t = t == kRing - 1 ? 0 : t + 1;     // now of rows k + 1 and k - 2
        if (k + 1 < kend) request(next);
#pragma unroll
        for (int i = 0; i < 9; i++) dy[i] = DOWN ? fbp[i] - fb[i] : fb[i] - fbp[i];
        const bool wall_t = q == khigh - 1;
        if (UPDATE || (q >= j0 - 1 && q > klow)) {
            const R hb = uniform(rq.hb), ht = uniform(rq.ht), wb = uniform(rq.wb), wt = uniform(rq.wt), Cx = uniform(rq.c);
            R gx[9], gy[9], bx[9], by[9], dr[3], dl[3];
#pragma unroll
            for (int i = 0; i < 9; i++) {
                const R dp = shift<kNext>(fbp[i]) - fbp[i];
                const R dm = shift<kPrev>(dp);
                gx[i] = slope(wl, wr, dm, dp);
                gy[i] = DOWN ? slope(wb, wt, dy[i], dyp[i]) : slope(wb, wt, dyp[i], dy[i]);
                // of the velocities entering on the left and on the right
                for (int e = 0; e < 3; e++) {
                    if (i == cP[0][e]) dl[e] = dm;
                    if (i == cN[0][e]) dr[e] = dp;
                }
            }
            carried<0>(c.dt, fbp, gx, gy, bx);
            carried<1>(c.dt, fbp, gx, gy, by);
            Side<R> lower, upper;
            sides<1>(c.dt, hb, ht, by, gy, lower, upper);
            if (UPDATE || q >= j0) {
                // the x faces (of no use for the row after the segment)
                Side<R> left, right;
                sides<0>(c.dt, hl, hr, bx, gx, left, right);
                Side<R> beside = shift<kNext>(left);
                if (edge) {
#pragma unroll
                    for (int e = 0; e < 3; e++) {
                        const R v = shift<kNext>(entering<0, true>(c.dt, bx, gx, e) - dl[e]);
                        right.c[e] = ghost_l ? v : right.c[e];
                        beside.c[e] = wall_r ? entering<0, false>(c.dt, bx, gx, e) + dr[e] : beside.c[e];
                    }
                    right.s = ghost_l ? beside.s : right.s;
                    right.d = ghost_l ? beside.d : right.d;
                    beside.s = wall_r ? right.s : beside.s;
                    beside.d = wall_r ? right.d : beside.d;
                }
                R pr[3], nr[3];
                face_flux<PM>(m, right, beside, Cx, Cx * c.k1, Cx * c.k5, pr, nr);
                if (!UPDATE && q == klow + 1) {
#pragma unroll
                    for (int e = 0; e < 3; e++)
                        top.c[e] = DOWN ? entering<1, false>(c.dt, by, gy, e) + dyp[cN[1][e]]
                                        : entering<1, true>(c.dt, by, gy, e) - dyp[cP[1][e]];
                    top.s = DOWN ? upper.s : lower.s;
                    top.d = DOWN ? upper.d : lower.d;
                }
                R p[3], n[3];
                if constexpr (DOWN) face_flux<PM>(m, upper, top, Cy, Cy1, Cy5, p, n);
                else face_flux<PM>(m, top, lower, Cy, Cy1, Cy5, p, n);
                if constexpr (UPDATE) update(q - 1, p, n);
#pragma unroll
                for (int e = 0; e < 3; e++) { px[e] = pr[e]; nx[e] = nr[e]; py[e] = p[e]; ny[e] = n[e]; }
            }
            top = DOWN ? lower : upper;
            if (wall_t) {
                // the row outside the wall ends the march: its side
                R in[3];
#pragma unroll
                for (int e = 0; e < 3; e++)
                    in[e] = DOWN ? entering<1, true>(c.dt, by, gy, e) - dy[cP[1][e]]
                                 : entering<1, false>(c.dt, by, gy, e) + dy[cN[1][e]];
                fb[0] = in[0]; fb[1] = in[1]; fb[2] = in[2];
            }
        }
        if constexpr (!UPDATE) settle();
#pragma unroll
        for (int i = 0; i < 9; i++) { fbp[i] = fb[i]; dyp[i] = dy[i]; }
        ip = rq.ih;
        wx += 9;
        rq = rk;
        row = next;
    }

    // March row j, pu and nu the fluxes through the face to the next.
    __device__ __forceinline__ void update(int j, const R pu[3], const R nu[3])
    {
        const size_t g = at(DOWN ? j0 + j1 - 1 - j : j);
        R pl[3], nl[3];
#pragma unroll
        for (int e = 0; e < 3; e++) { pl[e] = shift<kPrev>(px[e]); nl[e] = shift<kPrev>(nx[e]); }
        Outflow acc;
        outflow_x<0>(acc, px, nx, pl, nl);
        outflow_below(acc, DOWN ? pu : py, DOWN ? nu : ny);
        outflow_above(acc, DOWN ? py : pu, DOWN ? ny : nu);
        const double dtv = icol * ip;
        double Wp[3], G[3] = {0.0, 0.0, 0.0}, Wn[3];
        V fo[9], v[9];
        kept(t, Wp, fo);
        if (lagged) {
            ld_rows<3>(s.G + g, np, offw, G);
#if defined(__HIP_DEVICE_COMPILE__)
            // waited for here, or all that was requested is waited for in either mode
            asm volatile("" : "+v"(G[0]), "+v"(G[1]), "+v"(G[2]));
#endif
        }
        cell_update<PM>(m, lagged, dtv, Wp[0], Wp[1], Wp[2], acc, fo, G, Wn[0], Wn[1], Wn[2], v);
        settle();
        if (out) {
            st_rows<3>(s.Wo + g, np, offw, Wn);
            if constexpr (PM == SDUGKS_FP64) st_rows<9>(s.fo + g, np, offv, v);
            else st_rows<9>(s.fo32 + g, np, offv, v);
            if (lagged) st_rows<3>(s.Go + g, np, offw, G);
        }
    }

    __device__ __forceinline__ void run()
    {
        const bool per_y = cg.per_y != 0;
        klow = per_y ? INT32_MIN / 2 : (DOWN ? j0 + j1 - 1 - cg.ny : -1);
        khigh = per_y ? INT32_MAX / 2 : (DOWN ? j0 + j1 : cg.ny);
        int k = j0 - 2 > klow ? j0 - 2 : klow;
        kend = j1 + 2 < khigh + 1 ? j1 + 2 : khigh + 1;
        row = mesh_row(k);
        t = 0;
#pragma unroll
        for (int i = 0; i < 9; i++) { fbp[i] = 0; dyp[i] = 0; }
        top = {};
        for (int e = 0; e < 3; e++) px[e] = nx[e] = py[e] = ny[e] = 0;
        request(row);
        wx = lx + (at_l && ghost_r ? (kend - k) * 9 : 0);
        if (edge) columns(k, kend - k);
        __syncthreads();
        rq = record(row);
        for (; k <= j0 + 1; k++) step<false>(k);
        for (; k < kend; k++) step<true>(k);
        if (khigh == j1) {
            // the face between the last row and the wall
            const Side<R> in{{fbp[0], fbp[1], fbp[2]}, top.s, top.d};
            R p[3], n[3];
            if constexpr (DOWN) face_flux<PM>(m, in, top, Cy, Cy1, Cy5, p, n);
            else face_flux<PM>(m, top, in, Cy, Cy1, Cy5, p, n);
            t = t == kRing - 1 ? 0 : t + 1;
            update(j1 - 1, p, n);
        }
    }
};

// Unit u of an instance: units run along y inside a strip (a unit's halo rows
// are then its neighbours' rows), strips of nearly equal width.
template <int PM>
__device__ __forceinline__ void march_unit(const DevMesh &m, const DevCart &cg, const DevState &s, int lagged, int u)
{
    // [n_bc] boundary entries, then the columns outside the walls
    extern __shared__ WallBC bcs[];
    static_assert(kMaxTileBcs <= 64, "one thread per boundary entry");
    if ((int)threadIdx.x < m.n_bc) {
        const DevBC b = gin(m.bcs)[threadIdx.x];
        bcs[threadIdx.x] = {(double)b.type, b.rho, b.u, b.v};
    }
    __syncthreads();
    // strip u / segs (the estimate from the rounded inverse is at most one too small) and segment u % segs
    int strip = (int)(((uint64_t)(uint32_t)u * cg.inv_segs) >> 32), seg = u - strip * cg.segs;
    if (seg >= cg.segs) { strip++; seg -= cg.segs; }
    const int i0 = strip * cg.strip_w + (strip < cg.strip_more ? strip : cg.strip_more);
    const int j0 = seg * cg.seg_h + (seg < cg.seg_more ? seg : cg.seg_more);
    __shared__ Ring<PM> ring;
    const int w = strip + 1 < cg.strips ? cg.strip_w + (strip < cg.strip_more) : cg.nx - i0;
    const int j1 = j0 + cg.seg_h + (seg < cg.seg_more);
    Arith<PM> *const lx = (Arith<PM> *)(bcs + m.n_bc);
    // Every other segment downwards while the state, in and out, is little more than
    // the memory-side cache's 256 MB.  us a step, upwards all against every other
    // downwards, by cells an edge: FP64 800 32.3 / 29.2, 1024 45.7 / 43.3, 1152 53.3 /
    // 51.0, 1280 (315 MB) 77.6 / 77.3, 1448 (403 MB) 100 / 105; FP32 deviations 1024 31.3 /
    // 30.7, 1448 (252 MB) 50.1 / 50.1, 1600 76.0 / 76.0, 1792 (385 MB) 95.7 / 97.4, 2560 199 /
    // 200; FP32NEQ the same up to 1024 and 2 to 8 % slower beyond.
    constexpr int most = (int)(((size_t)320 << 20) / (2 * (3 * sizeof(double) + 9 * sizeof(Stored<PM>))));
    if (PM != SDUGKS_FP32NEQ && (seg & 1) && m.nc <= most)
        March<PM, true>(m, cg, s, lagged, i0, w, j0, j1, ring, bcs, lx).run();
    else
        March<PM, false>(m, cg, s, lagged, i0, w, j0, j1, ring, bcs, lx).run();
}

// The units of an instance, one per workgroup (so that the dispatcher evens
// out their lengths wave by wave: on the 64-cavity batch 103 us a step against
// 106 and 110 with two and four waves per workgroup), XCD by XCD in contiguous
// ranges.
template <int PM>
__global__ void __launch_bounds__(64, 2) k_step_cart(DevMesh m, DevCart c, DevState s, int lagged)
{
    const int x = (int)(blockIdx.x % kXcds);
    const int t = xcd_range_start((int)gridDim.x, x) + (int)(blockIdx.x / kXcds);
    march_unit<PM>(m, c, s, lagged, t);
}

// Batched structured step: as the batched general step, the slot map gives
// each workgroup its member and its unit there.
template <int PM>
__global__ void __launch_bounds__(64, 2) k_step_batch_cart(BatchTable tab, int parity)
{
    const int x = (int)(blockIdx.x % kXcds);
    const int per = (int)gridDim.x / kXcds;
    const unsigned long long slot = reinterpret_cast<const unsigned long long *>(tab.tmap)[x * per + (int)(blockIdx.x / kXcds)];
    const int member = (int)(unsigned)slot, unit = (int)(unsigned)(slot >> 32);
    if (member < 0) return;
    const BatchInst &in = tab.inst[member];
    const DevMesh m = in.m;
    const DevCart cg = in.c;
    march_unit<PM>(m, cg, batch_state(in, parity), in.lagged, unit);
}

}  // namespace

hipError_t launch_step_cart(const DevMesh &m, const DevCart &c, const DevState &s, int lagged, int mode,
                            hipStream_t st, GraphChain *gc)
{
    const dim3 grid((unsigned)cart_groups(c)), blk(64);
    const size_t lds = march_lds_bytes(c, m.n_bc, mode);
    if (mode == SDUGKS_FP32DEV) return emit(&k_step_cart<SDUGKS_FP32DEV>, grid, blk, lds, st, gc, m, c, s, lagged);
    if (mode == SDUGKS_FP32NEQ) return emit(&k_step_cart<SDUGKS_FP32NEQ>, grid, blk, lds, st, gc, m, c, s, lagged);
    return emit(&k_step_cart<SDUGKS_FP64>, grid, blk, lds, st, gc, m, c, s, lagged);
}

hipError_t launch_step_batch_cart(const BatchTable &tab, int mode, int parity, int cap_tiles, size_t lds,
                                  hipStream_t st, GraphChain *gc)
{
    const dim3 grid((unsigned)batch_grid(cap_tiles)), blk(64);
    if (mode == SDUGKS_FP32DEV) return emit(&k_step_batch_cart<SDUGKS_FP32DEV>, grid, blk, lds, st, gc, tab, parity);
    if (mode == SDUGKS_FP32NEQ) return emit(&k_step_batch_cart<SDUGKS_FP32NEQ>, grid, blk, lds, st, gc, tab, parity);
    return emit(&k_step_batch_cart<SDUGKS_FP64>, grid, blk, lds, st, gc, tab, parity);
}

}  // namespace sdg
