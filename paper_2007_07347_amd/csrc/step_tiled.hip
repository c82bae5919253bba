// Fused sDUGKS time step (Zhong et al., arXiv:2007.07347, Section II, the
// eleven-step summary) in one kernel for any mesh of triangles and quads: one
// workgroup per tile of cells.  A thread takes one cell of the tile or its first
// halo ring and, where there are more of them than threads, another of the
// second ring and a second face: two waves for a tile of 64 cells keep their
// lanes busier than four, and twice as many tiles fit a CU.
//
//   phase 1  fbar+ = a f + b feq(W) (Eq. fbarplus) of the tile and its two
//            halo rings into LDS; halo values are recomputed by every tile that
//            needs them instead of being stored to memory;
//   phase 2  least-squares slopes of fbar+ (the LLSR normal equations solved
//            through precomputed weights A^-1 d; boundary states are points at
//            the face midpoints) for the tile and its first ring, into LDS with
//            fbar+;
//   phase 3  one lane per face of the tile's cells: the upwind value of every
//            velocity at the foot point (Eq. fbpsource), fbar+_i + (r - e_i dt).g_i
//            with r from the upwind cell's centre to the face (one offset: fbar+
//            carried back first and then to the face is rounded once more in
//            between, which shows in FP32); face macros and equilibrium,
//            f at the face (Eq. f_t_n+1) and its mesoscopic fluxes (Eq. MesoFlux)
//            into LDS, over fbar+;
//   phase 4  one lane per tile cell: the fluxes of its faces summed in FP64 in the
//            order of its slots, W^{n+1} (Eq. MacroUpdate), feq^{n+1}, f^{n+1}
//            (Eq. fn+1), from the state the lane read in phase 1.
//
// Velocities are taken by opposite pairs: of each pair one leaves a face's
// first cell and the other its second, so a pair needs one reconstruction from
// each cell, at indices that the sign of e.n selects.
//
// Three forms share the code (template parameter PM), all with FP64 density
// and momentum, their update and the flux sums:
//   PM = 0  f stored and computed in FP64;
//   PM = 1  the deviation f - w_i rho0 stored in FP32 with FP32 face records
//           and least-squares weights, fbar+, slopes and face fluxes computed in
//           FP32 on deviations (the constant parts cancel exactly: sum_i w_i e_i
//           = 0 and the scaled normals of a closed cell sum to zero);
//   PM = 2  the non-equilibrium part f - feq(W) stored in FP32 (FP32 tables),
//           every operation in FP64: f = feq(W) + stored part on load, and
//           f^{n+1} - feq(W^{n+1}) rounded to FP32 on store.
//
// Every global input of the later phases is requested at kernel start, so its
// latency overlaps phase 1.  Each XCD sweeps a contiguous range of bisection
// tiles, those with boundary faces first, so the halo cells a tile reads are
// mostly L2 hits and the slower tiles start earliest.  A face shared by two
// tiles is evaluated by both, perhaps from opposite sides: exchanging the cells
// and the sign of n exchanges the operands of commutative operations only, so
// the flux that leaves one cell enters the other exactly.
//
// What bounds it: up to about 100,000 cells the chain of one tile (two dependent
// loads, three barriers, the phases), 5 to 6 us besides the launch; beyond,
// instruction issue and the tables' bytes.  Against four lanes per cell that
// evaluated each face from both of its cells: 200,000 triangles in FP32
// deviations 19.1 -> 13.6 us a step, 45,000 cells of a hybrid mesh in FP64
// 9.8 -> 8.1; tighter register limits that spill took 22 to 38 us.  fbar+ carried
// back in phase 2 rather than one offset per face: 13.6 and 8.7.
#include <type_traits>
#include <utility>

#include "cart_math.h"
#include "d2q9.h"
#include "device.h"
#include "mesh.h"
#include "step_common.h"

namespace sdg {

namespace {

// Opposite velocities: pair k is cPair[k][0] and cPair[k][1].
constexpr int cPair[4][2] = {{1, 3}, {2, 4}, {5, 7}, {6, 8}};

// One time step of tile t of one instance by the threads of its place (B of them,
// smem its LDS), whose results are written where live.  TWO: more local cells or
// faces than threads, so threads take second ones.
template <int D, int PM, bool TWO>
__device__ __forceinline__ void step_tile(const DevMesh &m, const DevTiles &tl, const DevState &s, int lagged, int t,
                                          int tid, int B, double *smem, bool live)
{
    using R = Arith<PM>;                        // arithmetic of fbar+, slopes, faces
    using V = Stored<PM>;
    using T = typename std::conditional<PM == SDUGKS_FP64, double, float>::type;    // tables
    using T2 = typename std::conditional<PM == SDUGKS_FP64, double2, float2>::type;
    struct R3 {
        R b, x, y;
    };
    const int P = tl.nl_max, PA = tl.na_max, PT = tl.nt_max, PF = tl.nf_max;
    const size_t np = (size_t)m.np;
    // LDS: W of the tile cells [3][PT] (faces on a boundary need it), the
    // boundary table [n_bc]; then fbar+ and the slopes (x, y) [PA][9] of the tile and
    // its first ring, cell by cell, and fbar+ [P][9], whose place the fluxes
    // [8][PF] take in phase 3
    double *const sW = smem;
    WallBC *const sbc = reinterpret_cast<WallBC *>(sW + 3 * PT + (PT & 1));
    R3 *const sr = reinterpret_cast<R3 *>(sbc + m.n_bc);
    R *const sfb = reinterpret_cast<R *>(sr + 9 * PA);
    R *const sphi = sfb;
    const Factors<PM> c(m);

    // ---- requests of all phases: the local cell id; what needs nothing loaded
    // first; then the state at the cell id.  Indices are clamped with the tables'
    // pitches, not the tile's own counts: every padded entry is a valid filler
    // (cell 0, no neighbour, zero weight, empty face), so no request waits for
    // the tile header, whose counts only mask what lanes without work read.
    // element i of a table (its base a scalar, the offset 32 bits)
    auto ld = [](const auto *base, int i) {
        using E = std::remove_const_t<std::remove_pointer_t<decltype(base)>>;
        return *(const gmem<E> *)((const gmem<char> *)gin(base) + (uint32_t)i * (uint32_t)sizeof(E));
    };
    const int *const lgid = tl.lgid + (size_t)t * P;
    const unsigned g1 = (unsigned)ld(lgid, tid < P ? tid : 0);
    const int t2 = B + tid < P ? B + tid : 0;
    const unsigned g2 = TWO ? (unsigned)ld(lgid, t2) : 0u;
    const int ta = tid < PA ? tid : 0, tt = tid < PT ? tid : 0;
    const int16_t *const ladj = tl.ladj + (size_t)t * D * PA, *const lfc = tl.lfc + (size_t)t * D * PT;
    const T2 *lw, *fr;
    if constexpr (PM == SDUGKS_FP64) {
        lw = tl.lw + (size_t)t * D * PA;
        fr = tl.fr + (size_t)t * PF * 3;
    } else {
        lw = tl.lw32 + (size_t)t * D * PA;
        fr = tl.fr32 + (size_t)t * PF * 3;
    }
    int la[D], code[D];
    T2 w[D];
#pragma unroll
    for (int sl = 0; sl < D; sl++) {
        la[sl] = ld(ladj, sl * PA + ta);
        w[sl] = ld(lw, sl * PA + ta);
        code[sl] = ld(lfc, sl * PT + tt);
    }
    struct Face {
        int cells;
        T2 ln, ra, rb;
    };
    auto face_of = [&](int f) {
        const int k = f < PF ? f : 0;
        return Face{ld(tl.fcell + (size_t)t * PF, k), ld(fr, k), ld(fr, PF + k), ld(fr, 2 * PF + k)};
    };
    const Face face1 = face_of(tid);
    Face face2 = face1;
    if constexpr (TWO) face2 = face_of(B + tid);
    const bool pb = tid < m.n_bc;
    const DevBC bcl = gin(m.bcs)[pb ? tid : 0];
    __builtin_amdgcn_sched_barrier(0);
    const double r = gin(s.W)[g1], mu = gin(s.W)[np + g1], mv = gin(s.W)[2 * np + g1];
    V fv[9];
#pragma unroll
    for (int i = 0; i < 9; i++) {
        if constexpr (PM == SDUGKS_FP64) fv[i] = gin(s.f)[(size_t)i * np + g1];
        else fv[i] = gin(s.f32)[(size_t)i * np + g1];
    }
    double W2[3] = {1.0, 0.0, 0.0};
    V fv2[9];
#pragma unroll
    for (int i = 0; i < 9; i++) fv2[i] = 0;
    if constexpr (TWO) {
        for (int k = 0; k < 3; k++) W2[k] = gin(s.W)[k * np + g2];
#pragma unroll
        for (int i = 0; i < 9; i++) {
            if constexpr (PM == SDUGKS_FP64) fv2[i] = gin(s.f)[(size_t)i * np + g2];
            else fv2[i] = gin(s.f32)[(size_t)i * np + g2];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // the tile header: counts of tile, first-ring and second-ring cells and faces
    const gmem<int> *const hd = gin(tl.hdr + 8 * t);
    const int nt = hd[1], na = nt + hd[2], nl = na + hd[3], nf = hd[4];
    const bool p1 = tid < nl, p2 = tid < na, p4 = tid < nt;
    const double dtv = gin(m.dtv)[p4 ? g1 : 0];

    // ---- phase 1
    if (pb) sbc[tid] = {(double)bcl.type, bcl.rho, bcl.u, bcl.v};
    if (p4) {
        sW[tid] = r;
        sW[PT + tid] = mu;
        sW[2 * PT + tid] = mv;
    }
    R fb[9];
    if (p1) {
        cell_plus<PM>(m, c, r, mu, mv, fv, fb);
#pragma unroll
        for (int i = 0; i < 9; i++) sfb[tid * 9 + i] = fb[i];
    }
    if (TWO && B + tid < nl) {
        R fb2[9];
        cell_plus<PM>(m, c, W2[0], W2[1], W2[2], fv2, fb2);
#pragma unroll
        for (int i = 0; i < 9; i++) sfb[t2 * 9 + i] = fb2[i];
    }
    __syncthreads();

    // ---- phase 2
    if (p2) {
        R gx[9], gy[9];
#pragma unroll
        for (int i = 0; i < 9; i++) { gx[i] = 0; gy[i] = 0; }
        // neighbours first, without a branch (an empty slot or a boundary point
        // reads the cell itself, whose difference is zero), so that all reads are
        // in flight together; then the few boundary points
        bool wall = false;
#pragma unroll
        for (int sl = 0; sl < D; sl++) {
            const int nb = la[sl] >= 0 ? la[sl] : tid;
            const R wx = (R)w[sl].x, wy = (R)w[sl].y;
            wall = wall || la[sl] < -1;
#pragma unroll
            for (int i = 0; i < 9; i++) {
                const R df = sfb[nb * 9 + i] - fb[i];
                gx[i] = fma_(wx, df, gx[i]);
                gy[i] = fma_(wy, df, gy[i]);
            }
        }
        if (wall) {
#pragma unroll
            for (int sl = 0; sl < D; sl++) {
                if (la[sl] >= -1) continue;
                R df[9];
                wall_diff<PM>(m, sbc[-2 - la[sl]], r, mu, mv, df);
#pragma unroll
                for (int i = 0; i < 9; i++) { gx[i] = fma_((R)w[sl].x, df[i], gx[i]); gy[i] = fma_((R)w[sl].y, df[i], gy[i]); }
            }
        }
#pragma unroll
        for (int i = 0; i < 9; i++) sr[tid * 9 + i] = R3{fb[i], gx[i], gy[i]};
    }
    __syncthreads();

    // ---- phase 3
    auto face_fluxes = [&](int f, const Face &face) {
        const int c0 = face.cells & 0xffff, c1 = face.cells >> 16;      // c1 < 0: boundary entry -2 - c1
        const R lx = (R)face.ln.x, ly = (R)face.ln.y, ax = (R)face.ra.x, ay = (R)face.ra.y;
        const bool inner = c1 >= 0;
        const int c2 = inner ? c1 : c0;
        const R bx = inner ? (R)face.rb.x : ax, by = inner ? (R)face.rb.y : ay;
        auto at = [&](int cell, R x, R y, int i) {
            const R3 v = sr[cell * 9 + i];
            return fma_(y, v.y, fma_(x, v.x, v.b));
        };
        const R f0 = (R)0.5 * (at(c0, ax, ay, 0) + at(c2, bx, by, 0));
        R fp[4], fm[4], sn[4];
        bool special = !inner;
        static_for<4>([&](auto K) {
            constexpr int k = K, p = cPair[k][0], q = cPair[k][1];
            sn[k] = cdot<cEx[p], cEy[p]>(lx, ly);
            special = special || sn[k] == (R)0;
            // of the pair, out leaves the first cell and in, its opposite, the second
            const bool up = sn[k] > (R)0;
            const int io = up ? p : q;
            const R ds = up ? c.dt : -c.dt;
            const R out = at(c0, ax - cmul<cEx[p]>(ds), ay - cmul<cEy[p]>(ds), io);
            const R in = at(c2, bx + cmul<cEx[p]>(ds), by + cmul<cEy[p]>(ds), p + q - io);
            fp[k] = up ? out : in;
            fm[k] = up ? in : out;
        });
        if (special) {
            if (!inner) {
                // entering through a boundary: the boundary state's fbar+ carried to the
                // foot point; leaving or along it: the cell's own value
                R df[9];
                wall_diff<PM>(m, sbc[-2 - c1], sW[c0], sW[PT + c0], sW[2 * PT + c0], df);
                static_for<4>([&](auto K) {
                    constexpr int k = K, p = cPair[k][0], q = cPair[k][1];
                    auto back = [&](R dt, int i) {
                        const R3 v = sr[c0 * 9 + i];
                        return fma_(-dt, cdot<cEx[p], cEy[p]>(v.x, v.y), v.b + df[i]);
                    };
                    const R ip = back(c.dt, p), iq = back(-c.dt, q);
                    fm[k] = sn[k] > (R)0 ? iq : fm[k];
                    fp[k] = sn[k] < (R)0 ? ip : fp[k];
                });
            } else {
                // along the face: the mean of both sides
                static_for<4>([&](auto K) {
                    constexpr int k = K, p = cPair[k][0], q = cPair[k][1];
                    const R dx = cmul<cEx[p]>(c.dt), dy = cmul<cEy[p]>(c.dt);
                    const R mp = (R)0.5 * (at(c0, ax - dx, ay - dy, p) + at(c2, bx - dx, by - dy, p));
                    const R mq = (R)0.5 * (at(c0, ax + dx, ay + dy, q) + at(c2, bx + dx, by + dy, q));
                    fp[k] = sn[k] == (R)0 ? mp : fp[k];
                    fm[k] = sn[k] == (R)0 ? mq : fm[k];
                });
            }
        }
        // face macros (deviations in DEV: rho_f = rho0 + sum, momentum unchanged)
        const R rsum = f0 + (((fp[0] + fm[0]) + (fp[1] + fm[1])) + ((fp[2] + fm[2]) + (fp[3] + fm[3])));
        const R d2 = fp[2] - fm[2], d3 = fp[3] - fm[3];
        const R mx = (fp[0] - fm[0]) + (d2 - d3), my = (fp[1] - fm[1]) + (d2 + d3);
        const R rf = PM == SDUGKS_FP32DEV ? (R)m.rho0 + rsum : rsum;
        R irf;
        if constexpr (PM == SDUGKS_FP32DEV) irf = (R)1 / rf;
        else irf = recip(rf);
        const R uf = mx * irf, vf = my * irf;
        const R B = fma_((R)-1.5, fma_(mx, uf, my * vf), rsum);
        const R k1 = c.c1 * c.k1, k5 = c.c1 * c.k5;
        // fluxes along n of the pair (p, q): e_q = -e_p
        auto flux = [&](int k, R K, R dm, R du) {
            const R S = fma_((R)4.5 * dm, du, B);
            sphi[(2 * k) * PF + f] = sn[k] * fma_(K, fma_((R)3, dm, S), c.c1 * fp[k]);
            sphi[(2 * k + 1) * PF + f] = -sn[k] * fma_(K, fma_((R)-3, dm, S), c.c1 * fm[k]);
        };
        flux(0, k1, mx, uf);
        flux(1, k1, my, vf);
        flux(2, k5, mx + my, uf + vf);
        flux(3, k5, my - mx, vf - uf);
    };
    if (tid < nf) face_fluxes(tid, face1);
    if (TWO && B + tid < nf) face_fluxes(B + tid, face2);
    __syncthreads();

    // ---- phase 4
    if (!p4 || !live) return;
    Outflow o;
#pragma unroll
    for (int i = 0; i < 9; i++) o.F[i] = 0.0;
#pragma unroll
    for (int sl = 0; sl < D; sl++) {
        if (code[sl] < 0) continue;
        const R *const ph = sphi + (code[sl] >> 1);
        const double sign = (code[sl] & 1) ? -1.0 : 1.0;        // the record as seen from the other cell
        static_for<8>([&](auto I) {
            constexpr int i = cPair[I / 2][I % 2];
            o.F[i] = fma_(sign, (double)ph[I * PF], o.F[i]);
        });
    }
    double G[3] = {0.0, 0.0, 0.0}, Wn[3];
    if (lagged)
        for (int k = 0; k < 3; k++) G[k] = gin(s.G)[k * np + g1];
    V v[9];
    cell_update<PM>(m, lagged, dtv, r, mu, mv, o, fv, G, Wn[0], Wn[1], Wn[2], v);
#pragma unroll
    for (int k = 0; k < 3; k++) gout(s.Wo)[k * np + g1] = Wn[k];
#pragma unroll
    for (int i = 0; i < 9; i++) {
        if constexpr (PM == SDUGKS_FP64) gout(s.fo)[(size_t)i * np + g1] = v[i];
        else gout(s.fo32)[(size_t)i * np + g1] = v[i];
    }
    if (lagged)
        for (int k = 0; k < 3; k++) gout(s.Go)[k * np + g1] = G[k];
}

// Waves on a SIMD that the registers are bound to allow.
template <int PM, bool TWO>
constexpr int kTiledWaves = PM == SDUGKS_FP32DEV ? 4 : (TWO ? 2 : 3);

// A workgroup's tiles: one, or (PAIR) two side by side on half of its threads each
// and on LDS of their own, which go through the barriers together.  Two tiles
// on 256 threads do what one on 128 does: 1024 x 1024 quads in tiles of 64, 32
// and 16 cells on 256, 128 and 128 threads take 129, 129 and 146 us a step in FP64
// (one tile per workgroup 176, 166 and 266), 200,000 triangles 22.7, 23.3 and 27.5.
template <bool PAIR>
struct Place {
    int sub = 0, tid;                   // which of them this thread works on, its index there
    double *smem;
    __device__ __forceinline__ explicit Place(const TileShare &sh)
    {
        extern __shared__ double lds[];
        tid = (int)threadIdx.x;
        smem = lds;
        if constexpr (PAIR) {
            sub = __builtin_amdgcn_readfirstlane(tid >= sh.threads ? 1 : 0);
            tid -= sub * sh.threads;
            smem += sub * (sh.bytes / 8);
        }
    }
};

// The tiles of this block, XCD by XCD in contiguous ranges (xcd_range_start).  They
// follow from the block index and the grid size alone, so the first requests
// wait for nothing but the table pointers.  Past the last tile the second place
// repeats it and writes nothing.
template <int D, int PM, bool TWO, bool PAIR>
__global__ void __launch_bounds__(256, (kTiledWaves<PM, TWO>)) k_step_tiled(DevMesh m, DevTiles tl, DevState s, int lagged, TileShare sh)
{
    const Place<PAIR> at(sh);
    const int x = (int)(blockIdx.x % kXcds);
    const int u = xcd_range_start((int)gridDim.x, x) + (int)(blockIdx.x / kXcds);
    const int t = PAIR ? 2 * u + at.sub : u;
    const bool live = !PAIR || t < tl.n_tiles;
    step_tile<D, PM, TWO>(m, tl, s, lagged, live ? t : tl.n_tiles - 1, at.tid, PAIR ? sh.threads : (int)blockDim.x, at.smem, live);
}

// Batched step: the tiles of all instances form one sequence; the grid covers
// a fixed capacity and each block reads its members and local tiles from the
// device map (one load each; member -1 past the live tiles), so the table can
// change between launches of a captured graph.  parity selects each
// instance's ping-pong buffers: it reads buffer (parity0 ^ parity).  Global
// memory is reached through global-address-space pointers (gin, gout in
// step_tile): the members' pointers come from their records, not from
// kernel arguments.  per: slots of an XCD, the live ones at their start.
template <int D, int PM, bool TWO, bool PAIR>
__global__ void __launch_bounds__(256, (kTiledWaves<PM, TWO>)) k_step_batch(BatchTable tab, int parity, TileShare sh, int per)
{
    // a slot's (member, tile) as one 8-byte load, so that the tile index
    // does not wait for the exit test on the member
    const Place<PAIR> at(sh);
    const unsigned long long *const map = reinterpret_cast<const unsigned long long *>(tab.tmap) + (int)(blockIdx.x % kXcds) * per;
    const int j = (PAIR ? 2 : 1) * (int)(blockIdx.x / kXcds);
    unsigned long long slot = map[j];
    bool live = true;
    if (PAIR && at.sub) {
        // a place past the live tiles goes along with the workgroup's first, writing nothing
        const unsigned long long second = j + 1 < per ? map[j + 1] : ~0ull;
        live = (int)(unsigned)second >= 0;
        slot = live ? second : slot;
    }
    const int member = (int)(unsigned)slot, tile = (int)(unsigned)(slot >> 32);
    // the member's record copied once: its fields are then requested together
    // (no address depends on another field) and stay in scalar registers
    // across the barriers instead of being reloaded from memory.  A workgroup past
    // the live tiles (member -1) leaves without stepping (the compiler may
    // take that exit before the record is requested).
    const BatchInst &in = tab.inst[member < 0 ? 0 : member];
    const DevMesh m = in.m;
    const DevTiles tl = in.t;
    if (member < 0) return;
    step_tile<D, PM, TWO>(m, tl, batch_state(in, parity), in.lagged, tile, at.tid, PAIR ? sh.threads : (int)blockDim.x, at.smem, live);
}

}  // namespace

size_t step_tiled_lds_bytes(const DevTiles &t, int mode, int n_bc)
{
    return tile_lds_bytes(t.nl_max, t.na_max, t.nt_max, t.nf_max, n_bc, mode == 1 ? sizeof(float) : sizeof(double));
}

// LDS of a place: the next one begins on a boundary of 16 bytes.
static TileShare tile_share(int threads, size_t lds) { return {threads, (int32_t)((lds + 15) / 16 * 16)}; }

// mode: 0 FP64, 1 FP32 deviation with FP32 face arithmetic, 2 FP32
// storage of f - feq(W) with FP64 arithmetic (the SDUGKS_FP64 / FP32DEV / FP32NEQ values)
hipError_t launch_step_tiled(const DevMesh &m, const DevTiles &t, const DevState &s, int lagged, int mode,
                             int block, int per, hipStream_t st, GraphChain *gc)
{
    const TileShare sh = tile_share(per, step_tiled_lds_bytes(t, mode, m.n_bc));
    const int tiles = block / per;
    const size_t lds = (size_t)tiles * sh.bytes;
    const dim3 grid((unsigned)((t.n_tiles + tiles - 1) / tiles)), blk(block);
    const bool two = step_tiled_two(t, per);
#define SDG_K(...) emit(&k_step_tiled<__VA_ARGS__>, grid, blk, lds, st, gc, m, t, s, lagged, sh)
#define SDG_TILED(DD, PP) \
    return tiles == 2 ? (two ? SDG_K(DD, PP, true, true) : SDG_K(DD, PP, false, true)) \
                      : (two ? SDG_K(DD, PP, true, false) : SDG_K(DD, PP, false, false))
    if (m.D <= 3) {
        if (mode == 1) SDG_TILED(3, 1);
        if (mode == 2) SDG_TILED(3, 2);
        SDG_TILED(3, 0);
    }
    if (mode == 1) SDG_TILED(4, 1);
    if (mode == 2) SDG_TILED(4, 2);
    SDG_TILED(4, 0);
#undef SDG_TILED
#undef SDG_K
}

hipError_t launch_step_batch(const BatchTable &tab, int D, int mode, bool two, int parity, int cap_tiles, size_t lds_tile,
                             int block, int per, hipStream_t st, GraphChain *gc)
{
    const TileShare sh = tile_share(per, lds_tile);
    const int tiles = block / per, slots = batch_grid(cap_tiles) / kXcds;
    const size_t lds = (size_t)tiles * sh.bytes;
    const dim3 grid((unsigned)(kXcds * ((slots + tiles - 1) / tiles))), blk(block);
#define SDG_K(...) emit(&k_step_batch<__VA_ARGS__>, grid, blk, lds, st, gc, tab, parity, sh, slots)
#define SDG_BATCH(DD, PP) \
    return tiles == 2 ? (two ? SDG_K(DD, PP, true, true) : SDG_K(DD, PP, false, true)) \
                      : (two ? SDG_K(DD, PP, true, false) : SDG_K(DD, PP, false, false))
    if (D <= 3) {
        if (mode == 1) SDG_BATCH(3, 1);
        if (mode == 2) SDG_BATCH(3, 2);
        SDG_BATCH(3, 0);
    }
    if (mode == 1) SDG_BATCH(4, 1);
    if (mode == 2) SDG_BATCH(4, 2);
    SDG_BATCH(4, 0);
#undef SDG_BATCH
#undef SDG_K
}

}  // namespace sdg
