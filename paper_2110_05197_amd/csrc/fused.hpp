// fused.hpp -- one-pass step: each block owns a TX x TY column of nodes and
// marches it through a chunk of TZ planes (D3Q19), or a row of TX nodes
// through a chunk of rows (D2Q9, the box seen as nx x 1 x ny).  The stencil
// inputs (colour-gradient densities / pseudopotential) of a plane are
// computed from its populations as they are loaded (two planes ahead of the
// collision), for the tile and a one-node halo ring, into a four-plane LDS
// ring; a tile node's populations wait one iteration in the thread's LDS slot
// and are collided from registers.  Only the halo ring's populations are read
// twice (by this block and by its neighbour), so HBM traffic stays near one
// read and one write of every population per step; no density field is
// written.  The solo and the batched kernels share the column body.
//
// Any nx (the last column in x is masked when TX does not divide it), any nz;
// ny % TY == 0, or, in the columns of their own for such boxes, the last row of
// columns masked as well.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"
#include "launch.hpp"

namespace mclbm {

// Stencil-field values of one node from its populations (the same values the
// density-field pass stores).
template <int MODEL, int NF, class C, class M, class FT>
__device__ __forceinline__ void field_values(const HP<C, M> &H, const M (&dr)[2], FT (&v)[NF])
{
    if constexpr (MODEL == CG) {
        v[0] = (FT)dr[0];
        v[1] = (FT)dr[1];
        v[2] = (FT)colour_field(H, dr[0], dr[1]);
    } else if constexpr (MODEL == SC_MP) {
        v[0] = (FT)pseudo_potential(H, H.rho0[0] + dr[0]);
    } else {
        v[0] = (FT)dr[0];
        v[1] = (FT)dr[1];
    }
}

// Collision of one node from the stencil values of its neighbours
// (v[field][direction], field_values order) and, for SC multiphase, its own
// pseudopotential; c holds its populations, dr and j their moments.
template <class L, int MODEL, int CONS, int NF, int K, class C, class M>
__device__ __forceinline__ void collide_values(const HP<C, M> &H, C (&c)[K][L::Q], const M (&dr)[2], const M (&j)[3],
                                               const C (&v)[NF][L::Q], C psi)
{
    if constexpr (MODEL == CG) {
        C gR[3], gB[3], gN[3];
        stencil_sum<L>(v[0], gR);
        stencil_sum<L>(v[1], gB);
        stencil_sum<L>(v[NF - 1], gN);
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) { gR[dd] *= C(3); gB[dd] *= C(3); gN[dd] *= C(3); }
        const C F0[3] = {C(0), C(0), C(0)};
        cg_collide<L, C, M, false, CONS>(H, c, dr, j, gR, gB, gN, F0);
    } else if constexpr (MODEL == SC_MP) {
        C s3[3];
        stencil_sum<L>(v[0], s3);
        const M rho = H.rho0[0] + dr[0];
        const M irho = rcp(rho);
        C F[3], u[3];
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) {
            F[dd] = -H.G * psi * s3[dd];
            u[dd] = (C)((j[dd] + M(0.5) * (M)F[dd]) * irho);
        }
        sc_collide_component<L, C, M>(c[0], H.om[0], dr[0], rho, u, F, H.rho0[0], H.corrM[0], H.shiftM[0]);
    } else {
        C sR[3], sB[3];
        stencil_sum<L>(v[0], sR);
        stencil_sum<L>(v[NF - 1], sB);
        const M rR = H.rho0[0] + dr[0], rB = H.rho0[1] + dr[1];
        const M ir = rcp(rR + rB);
        C FR[3], FB[3], u[3];
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) {
            FR[dd] = -H.xpref * (C)rR * sB[dd];
            FB[dd] = -H.xpref * (C)rB * sR[dd];
            u[dd] = (C)((j[dd] + M(0.5) * ((M)FR[dd] + (M)FB[dd])) * ir);
        }
        sc_collide_component<L, C, M>(c[0], H.om[0], dr[0], rR, u, FR, H.rho0[0], H.corrM[0], H.shiftM[0]);
        sc_collide_component<L, C, M>(c[K - 1], H.om[1], dr[1], rB, u, FB, H.rho0[1], H.corrM[1], H.shiftM[1]);
    }
}

// Block index -> tile, keeping runs of consecutive tiles on one XCD (blocks
// are dealt round-robin to the 8 XCDs, each with its own L2).
__device__ __forceinline__ int xcd_tile(int b, int nblocks)
{
    if (nblocks % 8) return b;
    return (b % 8) * (nblocks / 8) + b / 8;
}

// Whether a lattice has velocities along y (D2Q9Z has none: its tile rows
// need no halo rows).
template <class L>
constexpr bool uses_y()
{
    for (int i = 0; i < L::Q; ++i)
        if (L::cy[i] != 0) return true;
    return false;
}
template <class L, int TY>
constexpr int ring_rows() { return uses_y<L>() ? TY + 2 : TY; }

template <class L, int MODEL, int TX, int TY, class FT>
constexpr int fused_ring_bytes()
{
    return (4 * NField<MODEL>::n * (TX + 2) * ring_rows<L, TY>() * (int)sizeof(FT) + 15) / 16 * 16;
}
template <int PR, int MODEL, int TX, int TY, class L = D3Q19>
constexpr int fused_lds_bytes()
{
    return fused_ring_bytes<L, MODEL, TX, TY, typename Prec<PR>::F>()
           + NComp<MODEL>::n * L::Q * TX * TY * (int)sizeof(typename Prec<PR>::C);
}

// Spreading the loads of plane z+2 over the collision of plane z: vector
// instructions between two loads, 0 = all loads first.  One block fills a
// compute unit, its waves run in step from barrier to barrier, and 38 loads in
// a row from each of them reach memory as one burst per plane.  256^3 FP32
// colour gradient, ms per step, first 1.082, every 6 instructions 1.11,
// 14 1.06, 20 1.07, 22 1.14 (64-bit addressing, whose address arithmetic
// spaces the loads a little by itself: 1.115); SC multiphase 0.488 first,
// 0.470 every 14; 256^3 FP16 storage 0.658 first, 0.61 every 30.  Not where
// registers are short or the arithmetic is FP64 (128^3 FP64 0.293 first,
// 0.302 every 12; mixed 256^3 1.12 and 1.20), nor for the two-component
// Shan-Chen model (0.597 and 0.600 at 128 x 128 x 512), nor the 2-D rows (two
// blocks a compute unit, 18 loads; 4096^2 FP32 0.494 and 0.490).
template <int PR, int MODEL, bool YH>
constexpr int kLoadSpacing = !YH ? 0 : PR == 1 && MODEL != SC_MC ? 14 : PR == 3 && MODEL == CG ? 30 : 0;

// Kernels that read through 64-bit pointers although their stores are buffer
// accesses: the address arithmetic between the loads keeps them from leaving
// in one burst where kLoadSpacing does not.  4096^2 FP32 rows: 0.480 ms,
// 0.494 with buffer loads; mixed columns, 96 x 96 x 384 with walls and
// outflow: 0.348 and 0.383, 256^3 1.12 and 1.15.
template <int PR, bool YH> constexpr bool kPointerLoads = (PR == 1 && !YH) || (PR == 2 && YH);

// The type of a column's node indices (N < 2^31).  With 32-bit indices the
// pointer loads hold a zero-extended copy beside each offset: mixed-precision
// columns, at the 256 registers an eight-wave block allows, then spill 12-47 of
// them with the mass-keeping collision on periodic boxes, where 64-bit ones spill
// 0-4 (0.68-0.84 of the time), 96-wide ones 3 instead of none (0.94-1.0), and boxes
// in the other precisions take 0-3 % longer.  The plain mixed colour gradient on 64-wide
// periodic columns is the exception: it spills 4-25 with 32-bit indices and is 2-13 %
// faster for them (256^3 1116 us and 1204, 213 x 136 x 197 0.89 and 1.01 of the time
// through plain pointers), for the order its loads then leave in.
template <int PR, int MODEL, int TX, bool PERIODIC, int CONS>
using ColumnIndex = std::conditional_t<PR == 2 && MODEL == CG && TX == 64 && PERIODIC && CONS == kConsNever, unsigned, long long>;

// One block's work: the TX x TY column at (x0, y0), planes [z0, z1).  An
// EDGE column is the last one in x when TX does not divide nx: its first
// w = nx - x0 threads hold nodes, the others only take part in the barriers,
// and its +x halo is the column at x0 + w.  L is the lattice of the
// arithmetic, LA the one that places neighbours: both D3Q19, or D2Q9 and
// D2Q9Z for a 2-D box seen as nx x 1 x ny (TY = 1, halo columns only), so
// that a 2-D node's arithmetic is the two-pass kernels', operation for
// operation.  CONS: whether the collision keeps each colour's node mass
// (kConsNever / kConsAsked / kConsAlways, see cg_collide): the batched
// kernels ask each simulation, the solo launches choose a kernel.
template <int PR, int MODEL, int TX, int TY, bool PERIODIC, int EDGE = 0, class L = D3Q19, class LA = L,
          int CONS = kConsShared<PR>, bool FAR = false, bool SPREAD = true>
__device__ __forceinline__ void fused_column(const KParams &P, const void *srcp, void *dstp, unsigned *flag, int x0,
                                             int y0, int z0, int z1, unsigned char *smem)
{
    using S = typename Prec<PR>::S;
    using C = typename Prec<PR>::C;
    using M = typename Prec<PR>::M;
    using FT = typename Prec<PR>::F;
    constexpr int Q = L::Q;
    constexpr int K = NComp<MODEL>::n;
    constexpr int NF = NField<MODEL>::n;
    static_assert(LA::Q == L::Q, "one velocity set");
    constexpr bool YH = uses_y<LA>();   // halo rows y0-1 and y0+TY
    constexpr int RY = YH ? 1 : 0;      // ring row of tile row 0
    constexpr int HX = TX + 2, HY = ring_rows<LA, TY>(), PL = HX * HY, NT = TX * TY, NH = PL - NT;
    static_assert(NH <= NT, "halo ring larger than the block");
    // Dynamic LDS: a four-plane ring of stencil values (planes z-1, z, z+1
    // are read while plane z+2 is written), then each thread's private slot
    // holding the populations of plane z+1 (laid out [population][thread] so
    // that a wavefront's accesses are contiguous).
    FT (*lds)[NF][PL] = reinterpret_cast<FT (*)[NF][PL]>(smem);
    C *pop = reinterpret_cast<C *>(smem + fused_ring_bytes<LA, MODEL, TX, TY, FT>());

    const int nx = P.nx, ny = P.ny, nz = P.nz;
    const Pops<L, K, S, FAR || kPointerLoads<PR, YH>> src(srcp, P);
    const Pops<L, K, S, FAR> dst(dstp, P);
    const HP<C, M> H = make_hp<C, M>(P);
    const int tid = threadIdx.x;
    const int lx = tid % TX, ly = tid / TX;
    const int x = x0 + lx, y = y0 + ly;
    const int my_slot = (ly + RY) * HX + (lx + 1);
    const int w = EDGE ? min(TX, nx - x0) : TX;        // nodes per row of this column
    const int h = EDGE == 2 ? min(TY, ny - y0) : TY;   // rows of this column
    const bool act = (!EDGE || lx < w) && (EDGE != 2 || ly < h);

    // halo ring node of this thread: rows y0-1 and y0+h (when the lattice
    // has y velocities), then columns x0-1 and x0+w
    constexpr int NR = YH ? 2 * HX : 0;
    int hx = 0, hy = 0;
    if (YH && tid < HX) { hx = tid - 1; hy = -1; }
    else if (YH && tid < NR) { hx = tid - HX - 1; hy = h; }
    else if (tid < NR + TY) { hx = -1; hy = tid - NR; }
    else { hx = w; hy = tid - NR - TY; }
    const bool has_h = tid < NH && hx <= w && (EDGE != 2 || hy <= h);
    const int h_slot = (hy + RY) * HX + (hx + 1);
    const int hgx = stencil_coord(x0 + hx, nx, P.bc[0]);
    const int hgy = stencil_coord(y0 + hy, ny, P.bc[1]);
    using Idx = ColumnIndex<PR, MODEL, TX, PERIODIC, CONS>;
    const Idx n_xy = (Idx)x + (Idx)nx * (Idx)y;
    const Idx h_xy = (Idx)hgx + (Idx)nx * (Idx)hgy;
    const Idx sxy = (Idx)nx * (Idx)ny;
    auto ring = [&](int p) { return (p - z0 + 1) & 3; };

    bool bad = false;
    // stencil values of one node of plane p from its populations
    auto put = [&](int p, int slot, const C (&gv)[K][Q], M (&drv)[2], M (&jv)[3], bool interior) {
        node_moments<L, K>(gv, drv, jv);
        FT v[NF];
        field_values<MODEL, NF>(H, drv, v);
#pragma unroll
        for (int a = 0; a < NF; ++a) lds[ring(p)][a][slot] = v[a];
        if (interior && p >= z0 && p < z1) {
            const M r = H.rho0[0] + drv[0] + (K == 2 ? H.rho0[1] + drv[1] : M(0));
            bad = bad || node_bad(r, jv[0] + jv[1] + jv[2]);
        }
    };
    auto zoff = [&](int p) { return sxy * (Idx)stencil_coord(p, nz, P.bc[2]); };

    C c[K][Q];                  // populations of plane z (plane z+1's wait in LDS)
    M drc[2], jc[3], drn[2], jn[3];
    {
        // prologue: stencil values of planes z0-1, z0, z0+1; populations of z0, z0+1
        C tmp[K][Q];
        M d2[2], j2[3];
        if (act) {
            load_node(src, n_xy + zoff(z0 - 1), tmp);
            put(z0 - 1, my_slot, tmp, d2, j2, true);
            load_node(src, n_xy + zoff(z0), c);
            put(z0, my_slot, c, drc, jc, true);
            load_node(src, n_xy + zoff(z0 + 1), tmp);
            put(z0 + 1, my_slot, tmp, drn, jn, true);
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int i = 0; i < Q; ++i) pop[(k * Q + i) * NT + tid] = tmp[k][i];
        }
        if (has_h)
            for (int p = z0 - 1; p <= z0 + 1; ++p) {
                load_node(src, h_xy + zoff(p), tmp);
                put(p, h_slot, tmp, d2, j2, false);
            }
    }
    __syncthreads();

    for (int z = z0; z < z1; ++z) {
        // 1. issue the loads of plane z+2 (consumed after the collision): the
        // halo ring's here; the tile's here too, or spread over the collision
        // (kLoadSpacing).  Raised wave priority lets them leave before the
        // SIMD's other waves take the issue slots for their arithmetic: 2-D
        // rows 4096^2 FP32 0.489 -> 0.480 ms, buffer loads at 256^3 FP32 1.155
        // -> 1.085 ms, 64-bit addressed columns on ragged rows 234 x 80 x 119
        // FP32 0.223 -> 0.217.  In the other precisions it is worth -2 to +4 %
        // (150 boxes of nine shapes; one component in mixed precision and FP16
        // storage gains most, 192^3 295 -> 284 us; FP64 within 1 %), but periodic
        // mixed two-component Shan-Chen boxes lose 1-7 % (160^3 316 -> 334 us).
        constexpr bool raised = !(PR == 2 && MODEL == SC_MC);
        constexpr int spacing = FAR || !SPREAD ? 0 : kLoadSpacing<PR, MODEL, YH>;
        const bool ahead = z + 2 <= z1;
        RawNode<L, K, S, C> dr_, hr_;
        if constexpr (raised) __builtin_amdgcn_s_setprio(3);
        if (ahead) {
            if (spacing == 0 && act) dr_.load(src, n_xy + zoff(z + 2));
            if (has_h) hr_.load(src, h_xy + zoff(z + 2));
        }
        if constexpr (raised) __builtin_amdgcn_s_setprio(0);

        // 2. collide plane z with the stencil values of planes z-1, z, z+1
        if (act) {
            if constexpr (spacing > 0) dr_.load(src, ahead ? (unsigned)(n_xy + zoff(z + 2)) : kNoNode);
            C v[NF][Q];
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const int s = ring(z + LA::cz[i]);
                const int o = my_slot + LA::cy[i] * HX + LA::cx[i];
#pragma unroll
                for (int a = 0; a < NF; ++a) v[a][i] = (C)lds[s][a][o];
            }
#pragma unroll
            for (int a = 0; a < NF; ++a) v[a][0] = C(0);

            collide_values<L, MODEL, CONS>(H, c, drc, jc, v, MODEL == SC_MP ? (C)lds[ring(z)][0][my_slot] : C(0));
            const unsigned n = (unsigned)(n_xy + sxy * (Idx)z);
            // populations that stay on their x (cx = 0) land on whole cache
            // lines and are never read again in this step: stream them past
            // the cache; the x-shifted ones share lines with the neighbouring
            // tile's stores and go through L2
            if constexpr (PERIODIC) push_store_periodic<LA, true>(P, dst, x, y, z, n, c);
            else push_store_general<LA, true>(P, dst, x, y, z, n, c);
            // the order asked of the scheduler: one load, then `spacing`
            // vector instructions of the collision, and so on
            if constexpr (spacing > 0) {
#pragma unroll
                for (int q = 0; q < RawNode<L, K, S, C>::KA * Q; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, spacing, 0);
                }
            }
        }

        // 3. stencil values of plane z+2
        M drd[2], jd[3];
        C d[K][Q];
        dr_.get(d);
        if (ahead) {
            if (act) put(z + 2, my_slot, d, drd, jd, true);
            if (has_h) {
                C hh[K][Q];
                hr_.get(hh);
                M dh[2], jh[3];
                put(z + 2, h_slot, hh, dh, jh, false);
            }
        }
        // 4. rotate through this thread's LDS slot: z+1 -> z, z+2 -> z+1
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                C *sl = &pop[(k * Q + i) * NT + tid];
                c[k][i] = *sl;
                *sl = d[k][i];
            }
        __syncthreads();  // plane z+2 complete; plane z-1's slot is free
        drc[0] = drn[0]; drc[1] = drn[1];
        jc[0] = jn[0]; jc[1] = jn[1]; jc[2] = jn[2];
        drn[0] = drd[0]; drn[1] = drd[1];
        jn[0] = jd[0]; jn[1] = jd[1]; jn[2] = jd[2];
    }
    const unsigned long long any = __ballot(bad);
    if (any != 0ull && (tid & 63) == 0) atomicOr(flag, 1u);
}

// The columns of a launch in x: all full (TX divides nx), the last one an edge
// column, or one edge column only (nx < TX; a kernel of its own holds a single
// column body: 27 x 32 x 230 mixed 0.0385 -> 0.0362 ms).
// Or, for boxes whose rows no column height divides, the last column in x and in
// y edge columns of both kinds (near addressing, loads not spread: such boxes'
// rows are seldom line-aligned).
constexpr int kColsFull = 0, kColsRagged = 1, kColsNarrow = 2, kColsOdd = 3;
template <int PR, int MODEL, int TX, int TY, bool PERIODIC, int COLS, class L, class LA, bool CONS, bool FAR>
__global__ __launch_bounds__(TX *TY) void k_fused(KParams P, const void *src, void *dst, unsigned *flag, int TZ,
                                                  int tiles_x, int tiles_y)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int bx = t % tiles_x, by = (t / tiles_x) % tiles_y, bz = t / (tiles_x * tiles_y);
    const int x0 = bx * TX, y0 = by * TY, z0 = bz * TZ, z1 = min(z0 + TZ, P.nz);
    constexpr int cons = CONS ? kConsAlways : kConsNever;
    if constexpr (COLS == kColsOdd) {
        if (bx == tiles_x - 1 || by == tiles_y - 1) {
            fused_column<PR, MODEL, TX, TY, PERIODIC, 2, L, LA, cons, FAR, false>(P, src, dst, flag, x0, y0, z0, z1, smem);
            return;
        }
    } else if constexpr (COLS != kColsFull) {
        if (COLS == kColsNarrow || bx == tiles_x - 1) {
            fused_column<PR, MODEL, TX, TY, PERIODIC, 1, L, LA, cons, FAR>(P, src, dst, flag, x0, y0, z0, z1, smem);
            return;
        }
    }
    fused_column<PR, MODEL, TX, TY, PERIODIC, 0, L, LA, cons, FAR, COLS != kColsOdd>(P, src, dst, flag, x0, y0, z0, z1, smem);
}

// Batched one-pass step: the blocks of all eligible simulations of a group
// (D3Q19, ny a multiple of the column height) in one launch per kind; a
// block finds its simulation in the descriptor array (one-pass block ranges),
// skips it unless it is running and of the launch's kind (all faces periodic
// or not; nx a multiple of 64 or not; 96-wide columns or not), and processes
// one column of that simulation.  EDGE launches take the simulations whose nx
// is not a multiple of 64 and run every column through the masked column body
// (the last column in x holds nx mod 64 nodes; a full column computes the same
// as unmasked); WIDE launches take those on 96 x 4 columns.
// The per-node arithmetic is the solo kernels', so a batched simulation
// evolves bitwise as it would alone.  Columns: 64-wide rows (at 16
// or 32 nodes the rows of the x-shifted pushes split cache lines between
// neighbouring blocks and the step runs at half speed), 8 rows (4 in FP64 and
// in mixed precision, whose FP64 sums need the registers).  One kernel per
// kind keeps a single column body per kernel: with two inlined the
// mixed-precision kernel needed 270 registers (one wave per SIMD) and ran no
// faster than the batched two-pass kernels.
constexpr int kBatchTX = 64;
constexpr int batch_ty(int precision) { return precision == 0 || precision == 2 ? 4 : 8; }
// As in the solo kernel, a simulation whose nx 96 divides and 64 does not
// takes 96 x 4 columns (kernels of their own, WIDE): no lane idles where a
// 64-wide split would leave half of its last column empty.  Not FP64, nor the
// mixed-precision colour gradient: a six-wave block allows 256 registers a
// lane, and their batched columns (which ask each simulation whether to keep
// colour mass) need more (FP64 about 400, mixed 290).
constexpr int kBatchWideTX = 96, kBatchWideTY = 4;
constexpr bool batch_wide_kernel(int precision, int model)
{
    return precision != 0 && !(precision == 2 && model == CG);
}
constexpr bool batch_wide(int precision, int model, int nx, int ny)
{
    return batch_wide_kernel(precision, model) && nx % kBatchWideTX == 0 && nx % kBatchTX != 0
           && ny % kBatchWideTY == 0;
}
constexpr int batch_tile_tx(int precision, int model, int nx, int ny)
{
    return batch_wide(precision, model, nx, ny) ? kBatchWideTX : kBatchTX;
}
constexpr int batch_tile_ty(int precision, int model, int nx, int ny)
{
    return batch_wide(precision, model, nx, ny) ? kBatchWideTY : batch_ty(precision);
}
// which kernels a group launches: all-periodic sims and others, each with nx
// a multiple of 64 or not (EDGE), or on 96 x 4 columns (WIDE)
constexpr int kFusedPeriodic = 1, kFusedBounded = 2, kFusedPeriodicEdge = 4, kFusedBoundedEdge = 8;
constexpr int kFusedPeriodicWide = 16, kFusedBoundedWide = 32;
constexpr int kFusedFar = 6;   // the same kinds, 64-bit addressing: bits 6 .. 11
constexpr int fused_kind(bool periodic, bool edge, bool wide, bool far)
{
    const int k = wide ? (periodic ? kFusedPeriodicWide : kFusedBoundedWide)
                  : edge ? (periodic ? kFusedPeriodicEdge : kFusedBoundedEdge) : (periodic ? kFusedPeriodic : kFusedBounded);
    return far ? k << kFusedFar : k;
}

__device__ __forceinline__ int find_sim_fused(const SimDesc *D, int n, long long b)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (D[mid].fblock0 <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

constexpr int kb_tx(bool wide) { return wide ? kBatchWideTX : kBatchTX; }
constexpr int kb_ty(int precision, bool wide) { return wide ? kBatchWideTY : batch_ty(precision); }

template <int PR, int MODEL, bool PERIODIC, bool EDGE, bool WIDE = false, bool FAR = false>
__global__ __launch_bounds__(kb_tx(WIDE) * kb_ty(PR, WIDE)) void kb_fused(SimDesc *D, int nsims)
{
    static_assert(!(WIDE && EDGE) && !(WIDE && !batch_wide_kernel(PR, MODEL)), "96-wide columns: full columns");
    constexpr int TX = kb_tx(WIDE), TY = kb_ty(PR, WIDE);
    extern __shared__ __align__(16) unsigned char smem[];
    const int s = find_sim_fused(D, nsims, blockIdx.x);
    const SimDesc &d = D[s];
    if (d.state != 0 || (d.P.far_rows != 0) != FAR) return;
    if ((d.P.bc[0] == 0 && d.P.bc[1] == 0 && d.P.bc[2] == 0) != PERIODIC) return;
    if (batch_wide(PR, MODEL, d.P.nx, d.P.ny) != WIDE) return;
    if (!WIDE && (d.P.nx % kBatchTX != 0) != EDGE) return;
    const long long b = blockIdx.x - d.fblock0;
    const int tiles_x = (d.P.nx + TX - 1) / TX, tiles_y = d.P.ny / TY;
    const int bx = (int)(b % tiles_x), by = (int)((b / tiles_x) % tiles_y), bz = (int)(b / ((long long)tiles_x * tiles_y));
    const int x0 = bx * TX, y0 = by * TY, z0 = bz * d.ftz, z1 = min(z0 + d.ftz, d.P.nz);
    unsigned *flag = global_ptr<unsigned>(d.flag);
    fused_column<PR, MODEL, TX, TY, PERIODIC, EDGE ? 1 : 0, D3Q19, D3Q19, kConsShared<PR>, FAR>(
        d.P, global_ptr<char>(d.f[d.cur]), global_ptr<char>(d.f[d.cur ^ 1]), flag, x0, y0, z0, z1, smem);
}

// Planes per column of the batched simulations of a group.  A column
// advances one plane at a time and starts with three planes of loads, and
// the blocks run in rounds of `resident` (the blocks the chip holds at
// once), so the time of a step goes as rounds * (planes per chunk + 3).  The
// chunk length is searched for the least such cost (ties: fewer blocks);
// each simulation then balances its chunks over its nz.
inline int batch_fused_tz(int nz, int group_tz)
{
    const int chunks = (nz + group_tz - 1) / group_tz;
    return (nz + chunks - 1) / chunks;
}

// cols[s], nz[s]: columns per plane and planes of the group's one-pass sims
inline int batch_group_tz(const long long *cols, const int *nz, int n, long long resident)
{
    int best = 1;
    long long best_cost = -1, best_blocks = 0;
    for (int tz = 1; tz <= 64; ++tz) {
        long long blocks = 0;
        int longest = 0;
        for (int s = 0; s < n; ++s) {
            const int t = batch_fused_tz(nz[s], tz);
            blocks += cols[s] * ((nz[s] + t - 1) / t);
            longest = std::max(longest, t);
        }
        const long long rounds = (blocks + resident - 1) / std::max<long long>(1, resident);
        const long long cost = rounds * (longest + 3);
        if (best_cost < 0 || cost < best_cost || (cost == best_cost && blocks < best_blocks)) {
            best = tz;
            best_cost = cost;
            best_blocks = blocks;
        }
    }
    return best;
}

// Classes of one-pass steps that always address through pointers (column_pointers
// has the times), which need no kernels with buffer accesses: rows of D2Q9 (flat),
// 96-wide columns or others.
constexpr bool always_pointers(int precision, int model, bool periodic, bool flat, bool wide)
{
    if (precision == 3) return !periodic || (!flat && wide && model == SC_MC);
    if (flat) return (precision == 1 && model != SC_MP) || (precision == 2 && model == CG && !periodic);
    return precision == 1 && periodic && model != CG && wide;
}
// The same of the batched kernels (batch_column_pointers).
constexpr bool batch_always_pointers(int precision, int model, bool periodic, bool edge, bool wide)
{
    if (periodic && wide && model == CG && (precision == 1 || precision == 3)) return true;
    if (periodic && edge && model == SC_MP && precision == 1) return true;
    return always_pointers(precision, model, periodic, false, wide);
}

// Blocks a compute unit holds of the batched one-pass kernels of one column
// width: the fewest over periodic or not, edge columns or not, near and FAR.
template <int PR, int MODEL, bool WIDE>
int batch_fused_per_cu()
{
    constexpr int lds = fused_lds_bytes<PR, MODEL, kb_tx(WIDE), kb_ty(PR, WIDE)>();
    constexpr bool EDGE = !WIDE;
    constexpr bool PF = batch_always_pointers(PR, MODEL, true, false, WIDE), BF = batch_always_pointers(PR, MODEL, false, false, WIDE);
    constexpr bool PE = batch_always_pointers(PR, MODEL, true, EDGE, WIDE), BE = batch_always_pointers(PR, MODEL, false, EDGE, WIDE);
    const void *fns[8] = {
        (const void *)kb_fused<PR, MODEL, true, false, WIDE, PF>, (const void *)kb_fused<PR, MODEL, false, false, WIDE, BF>,
        (const void *)kb_fused<PR, MODEL, true, false, WIDE, true>, (const void *)kb_fused<PR, MODEL, false, false, WIDE, true>,
        (const void *)kb_fused<PR, MODEL, true, EDGE, WIDE, PE>, (const void *)kb_fused<PR, MODEL, false, EDGE, WIDE, BE>,
        (const void *)kb_fused<PR, MODEL, true, EDGE, WIDE, true>, (const void *)kb_fused<PR, MODEL, false, EDGE, WIDE, true>};
    int per_cu = 1 << 30;
    for (int i = 0; i < (EDGE ? 8 : 4); ++i) {
        int b = 0;
        (void)hipFuncSetAttribute(fns[i], hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, fns[i], kb_tx(WIDE) * kb_ty(PR, WIDE), lds) != hipSuccess) return 0;
        per_cu = std::min(per_cu, b);
    }
    return std::max(1, per_cu);
}

// Blocks of kb_fused<PR, MODEL, ...> the device holds at once (the smallest
// over the kinds).
template <int PR, int MODEL>
long long batch_fused_resident()
{
    int dev = 0, cus = 0, per_cu = batch_fused_per_cu<PR, MODEL, false>();
    if constexpr (batch_wide_kernel(PR, MODEL)) per_cu = std::min(per_cu, batch_fused_per_cu<PR, MODEL, true>());
    if (per_cu == 0 || hipGetDevice(&dev) != hipSuccess
        || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 256;
    return (long long)per_cu * std::max(1, cus);
}

// kinds: the fused_kind() bits of the simulations present.  Every launch
// covers the group's whole one-pass block range; a block whose simulation is
// of another kind returns at once.
template <int PR, int MODEL, bool PERIODIC, bool EDGE, bool WIDE, bool FAR>
void launch_batch_kind(SimDesc *D, int n, long long fblocks, int kinds, hipStream_t s)
{
    if constexpr (FAR || !batch_always_pointers(PR, MODEL, PERIODIC, EDGE, WIDE)) {
        if (!(kinds & fused_kind(PERIODIC, EDGE, WIDE, FAR))) return;
        constexpr int TX = kb_tx(WIDE), TY = kb_ty(PR, WIDE), lds = fused_lds_bytes<PR, MODEL, TX, TY>();
        static bool attr_set = false;
        if (!attr_set) {
            (void)hipFuncSetAttribute((const void *)kb_fused<PR, MODEL, PERIODIC, EDGE, WIDE, FAR>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            attr_set = true;
        }
        hipLaunchKernelGGL((kb_fused<PR, MODEL, PERIODIC, EDGE, WIDE, FAR>), dim3((unsigned)fblocks), dim3(TX * TY), lds, s, D, n);
    }
}
template <int PR, int MODEL, bool FAR>
void launch_batch_kinds(SimDesc *D, int n, long long fblocks, int kinds, hipStream_t s)
{
    launch_batch_kind<PR, MODEL, true, false, false, FAR>(D, n, fblocks, kinds, s);
    launch_batch_kind<PR, MODEL, false, false, false, FAR>(D, n, fblocks, kinds, s);
    launch_batch_kind<PR, MODEL, true, true, false, FAR>(D, n, fblocks, kinds, s);
    launch_batch_kind<PR, MODEL, false, true, false, FAR>(D, n, fblocks, kinds, s);
    if constexpr (batch_wide_kernel(PR, MODEL)) {
        launch_batch_kind<PR, MODEL, true, false, true, FAR>(D, n, fblocks, kinds, s);
        launch_batch_kind<PR, MODEL, false, false, true, FAR>(D, n, fblocks, kinds, s);
    }
}
template <int PR, int MODEL>
void launch_batch_fused(SimDesc *D, int n, long long fblocks, int kinds, hipStream_t s)
{
    launch_batch_kinds<PR, MODEL, false>(D, n, fblocks, kinds, s);
    if (kinds >> kFusedFar) launch_batch_kinds<PR, MODEL, true>(D, n, fblocks, kinds, s);
}

// One-pass kernels that keep 64-bit addressing below the 4 GB line too
// (KParams::far_rows), from sweeps of 1800 random boxes stepped both ways; t is
// the time through buffers over the time through pointers (10 % quantile,
// median, 90 % quantile).
// - FP16 storage with walls or outflow: t 0.99, 1.02, 1.06 on D3Q19, 1.01, 1.02,
//   1.06 on D2Q9 (periodic 0.87, 0.95, 1.00 and 0.93, 0.95, 0.98).
// - D2Q9: mixed colour gradient with walls or outflow, t 1.07, 1.09, 1.11
//   (periodic 0.94, 0.96, 0.98), and FP32 with two components, t 0.99, 1.005, 1.02,
//   up to 1.17 (one component 0.99, 0.99, 1.00; FP64 0.96, 0.99, 1.01).
// - D3Q19 on 96-wide columns, periodic: the Shan-Chen models in FP32, t 1.00, 1.03,
//   1.05, the two-component one in FP16 storage too (1.01, 1.04, 1.08).
// - D3Q19 FP32 on 96-wide columns with walls or outflow, two components, from 2^19
//   nodes: colour gradient t 1.00, 1.02, 1.04, Shan-Chen 1.00, 1.05, 1.07 (fewer nodes
//   0.95-1.03; one component 0.98, 1.00, 1.01; the colour gradient periodic 0.92, 0.985,
//   1.005; 96 x 96 x 384 319 us, 309 through pointers).
// - D3Q19 FP32 colour gradient, periodic, more than one column and rows off the
//   cache lines, from 2^22 nodes: t 0.98, 1.02, 1.06 (178 x 192 x 140 434 and 473 us;
//   fewer nodes 0.93, 0.98, 1.04, every other FP32 box 0.90, 0.97, 1.01).
// - D3Q19 mixed colour gradient, periodic, more than one column and rows off the
//   cache lines: with the mass-keeping collision t 0.97, 1.01, 1.05, without 1.06 at
//   the median (the other models 0.95, 0.98, 1.01).
// - D3Q19 FP64, two components, from 11 * 2^20 nodes: t 0.97, 1.07, 1.15 (8 to
//   11 * 2^20 nodes 0.95, 0.98, 1.03, fewer 0.90, 0.94, 0.98); not the colour
//   gradient on ragged rows with walls (0.90, 0.94, 0.96 at any size).
inline bool column_pointers(const KParams &P, bool flat, int precision, int model)
{
    const bool periodic = P.bc[0] == 0 && P.bc[1] == 0 && P.bc[2] == 0;
    const bool wide = P.nx % 96 == 0 && P.nx % 64 != 0;
    if (always_pointers(precision, model, periodic, flat, wide)) return true;
    if (flat || precision == 3) return false;
    const bool off_lines = P.nx > 64 && P.nx % 32 != 0;
    if (precision == 1) {
        if (!periodic) return wide && model != SC_MP && P.N >= 1 << 19;
        return model == CG && off_lines && P.N >= 1 << 22;
    }
    if (precision == 2) return model == CG && periodic && off_lines;
    return model != SC_MP && P.N >= 11LL << 20 && (periodic || model != CG || P.nx % 64 == 0);
}

// The same for a batched one-pass step, whose launches hold several simulations.
// Periodic, of 1-8 equal boxes: also the colour gradient on 96-wide columns, in FP32
// (70 batches, t 0.98, 1.025, 1.045) and FP16 storage (1.00, 1.07, 1.12), and FP32 SC
// multiphase with edge columns (50 batches, 1.00, 1.035, 1.06; whole ones 0.99).
inline bool batch_column_pointers(const KParams &P, int precision, int model)
{
    const bool periodic = P.bc[0] == 0 && P.bc[1] == 0 && P.bc[2] == 0;
    const bool wide = batch_wide(precision, model, P.nx, P.ny);
    return batch_always_pointers(precision, model, periodic, !wide && P.nx % kBatchTX != 0, wide)
           || column_pointers(P, false, precision, model);
}

// A box's columns (D3Q19) on the one-pass kernel, planned once per simulation.
struct FusedShape {
    int tx, ty, tz;
    bool ragged;   // the last column in x is an edge column
    bool odd;      // the last column in x and in y may be (no column height divides ny)
};

// What a one-pass step of this shape does beyond its nodes' work, as a factor:
// idle lanes of edge columns, three planes of loads per chunk before the march
// starts, compute units (256 on MI355X, one block each) left idle.
inline double fused_overhead(const KParams &P, const FusedShape &sh)
{
    const long long tiles_x = (P.nx + sh.tx - 1) / sh.tx, tiles_y = (P.ny + sh.ty - 1) / sh.ty;
    const long long chunks = (P.nz + sh.tz - 1) / sh.tz, blocks = tiles_x * tiles_y * chunks;
    const double lanes = (double)(tiles_x * sh.tx) * (double)(tiles_y * sh.ty) / ((double)P.nx * P.ny);
    const double fill = (double)((blocks + 255) / 256 * 256) / (double)blocks;
    return lanes * fill * (sh.tz + 3) / sh.tz;
}

// z-chunks: at most one block per compute unit -- more resident blocks per XCD
// overflow its L2 and the halo re-reads miss, and a grid just above 256 blocks
// runs a second, nearly empty round.  Where that leaves units idle, the chunk
// length with the least rounds * (planes + 3) instead, if that promises a tenth
// less than one round: 170 boxes of 130 to 232 blocks in one round, both ways,
// promised 0.66-0.9, took 0.72-1.0 of the time (median 0.86; 247 x 192 x 201 FP64
// 1.04), promised more, 0.84-1.22 (median 0.99).  FP32 boxes of 200 blocks and more
// gain nothing at 0.83-0.91 either (200^3 1.05, 309 x 160 x 193 1.12, 262 x 320 x 112
// 0.91), FP16 storage gains what is promised (median 0.92 at 0.79-0.98).
inline void fused_chunks(const KParams &P, FusedShape &sh, int precision)
{
    const long long txy = (long long)((P.nx + sh.tx - 1) / sh.tx) * ((P.ny + sh.ty - 1) / sh.ty);
    const long long tiles_z = std::max<long long>(1, 256 / txy);
    sh.tz = (int)((P.nz + tiles_z - 1) / tiles_z);
    const long long blocks = txy * ((P.nz + sh.tz - 1) / sh.tz), plain = sh.tz + 3;
    if (blocks >= (precision == 1 ? 200 : 256) || txy * P.nz < 256) return;
    // the most chunks of every number of rounds, until the planes that the
    // columns cannot do without leave no less cost (about sqrt(nz) steps)
    long long best = plain, tz = sh.tz;
    for (long long rounds = 1; 256 * (best - 3 * rounds) > txy * P.nz; ++rounds) {
        const long long chunks = std::min<long long>(P.nz, 256 * rounds / txy), t = (P.nz + chunks - 1) / chunks;
        const long long cost = (txy * ((P.nz + t - 1) / t) + 255) / 256 * (t + 3);
        if (cost < best) {
            best = cost;
            tz = t;
        }
        if (chunks == P.nz) break;
    }
    if (precision == 3 || 10 * best <= 9 * plain) sh.tz = (int)tz;
}

// Tile choice: 64-wide rows (narrower rows split the x-shifted pushes' cache
// lines between blocks), the last column masked when 64 does not divide nx;
// TY = 8 when ny allows, else 4; TZ planes per block.  FP64 (wide) tiles are
// 4 rows: half the threads, so that each wave may hold its double-precision
// planes in up to 512 registers and the LDS slot of plane z+1 stays at the
// FP32 size.  Where 96 divides nx and 64 does not (nx = 96, 288, ...), the
// columns are 96 x 4 instead (six waves, no lane idle), in place of 64-wide
// columns whose last one would leave a third of its lanes or more idle.
inline bool fused_shape(const KParams &P, FusedShape &sh, int precision)
{
    const bool wide = precision == 0;
    sh.tx = 64;
    sh.ragged = P.nx % 64 != 0;
    if (!wide && P.nx % 96 == 0 && P.nx % 64 != 0 && P.ny % 4 == 0) {
        sh.tx = 96;
        sh.ty = 4;
        sh.ragged = false;
    } else if (!wide && P.ny % 8 == 0) sh.ty = 8;
    else if (P.ny % 4 == 0) sh.ty = 4;
    else return false;
    sh.odd = false;
    fused_chunks(P, sh, precision);
    return true;
}

// Automatic choice between the one-pass and the two-pass kernels on D3Q19,
// where both exist: two-pass where the one-pass shape's overhead is past a line.
// The lines come from 1900 random boxes of 24 to 350 nodes a side in every
// precision and model, a third of them periodic, stepped both ways.  Median
// one-pass over two-pass time at an overhead of 1.15-1.3, 1.3-1.5 and 2-3:
//   FP64 CG 0.87, 1.03, 1.45       mixed CG 0.92, 1.02, 1.43
//   FP32 CG 0.84, 1.07, 1.23       FP32 SC_MP 0.87, 1.11, 1.32
//   FP32 SC_MC 1.04, 0.9-1.1, 1.32  mixed SC_MP 1.02, 1.12, 1.36
//   FP16 CG 0.96, 1.03, 1.13       FP16 SC_MP 1.5, 1.5, 1.5
// and of the mass-keeping collision alike.  FP64 with two components breaks even
// at 1.45 with walls and 1.6 periodic (110 x 104 x 117 CG, 1.58: 245 us and 279), FP32
// with two components, periodic, at 1.62 where one population buffer fits the
// Infinity Cache and both do not (52 x 216 x 124 CG, 1.58: 112 and 151), 64 x 4
// columns below FP64, which hold half the waves of 64 x 8 ones, under 1.3, 96-wide
// ones at 1.35-1.45 for the colour gradient and 1.2 else.  One box in 25 is left the
// choice that takes more than 5 % longer, by 37 % at most (FP16 boxes of 10^5 nodes
// among them, 10 to 20 us either way).  Up to 2^13 nodes a step takes 6-12 us either
// way.
inline double one_pass_line(const KParams &P, const FusedShape &sh, int precision, int model)
{
    const bool periodic = P.bc[0] == 0 && P.bc[1] == 0 && P.bc[2] == 0;
    const bool low = precision != 0 && sh.tx == 64 && sh.ty == 4;
    if (precision == 3 ? low || model == SC_MP : low && model == SC_MP) return 1.1;
    if (low) return 1.25;
    if (sh.tx == 96) return precision != 3 && model == CG ? 1.47 : 1.2;
    // bytes of both population buffers, against the 256 MB Infinity Cache
    const double state = 76.0 * (model == SC_MP ? 1 : 2) * (precision == 0 ? 8 : precision == 3 ? 2 : 4) / 2.0 * (double)P.N;
    if (precision == 0) return !periodic ? (model == SC_MP ? 1.4 : 1.45) : model == SC_MP && state < 0x1p28 ? 1.35 : 1.6;
    if (model == SC_MP) return periodic ? 1.35 : 1.25;
    if (precision == 1 && periodic && state > 0x1p28 && state < 0x1p29) return 1.62;
    return periodic ? 1.45 : 1.4;
}
inline bool d3_prefers_two_pass(const KParams &P, int precision, int model)
{
    FusedShape sh;
    if (P.N <= 1 << 13 || !fused_shape(P, sh, precision)) return false;
    return fused_overhead(P, sh) > one_pass_line(P, sh, precision, model);
}

// The automatic choice for D3Q19 boxes whose ny 4 does not divide: one-pass
// columns with edge columns in y too where they have little to spare (128 x 126
// x 128, overhead 1.2: FP32 0.212 -> 0.161 ms, FP64 0.418 -> 0.302; 40 random boxes
// under 1.3: 0.75-1.03 of the two-pass time; FP16 storage 0.81-1.11, its one
// multiphase box 1.4).
constexpr int odd_column_height(bool wide) { return wide ? 4 : 8; }
inline bool fused_odd_shape(const KParams &P, FusedShape &sh, int precision)
{
    sh.tx = 64;
    sh.ty = odd_column_height(precision == 0);
    sh.ragged = true;
    sh.odd = true;
    fused_chunks(P, sh, precision);
    return P.ny % 4 != 0 && !P.far && !P.conserve && P.N >= (1 << 18) && fused_overhead(P, sh) < 1.3;
}

// One launch of k_fused; the dynamic-LDS limit is raised once per kernel and
// process.
template <int PR, int MODEL, int TX, int TY, bool PERIODIC, int COLS, class L, class LA, bool CONS, bool FAR>
void launch_fused_one(const KParams &P, const void *src, void *dst, unsigned *flag, int tz, int tiles_x, int tiles_y,
                      hipStream_t s)
{
    constexpr int lds = fused_lds_bytes<PR, MODEL, TX, TY, LA>();
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_fused<PR, MODEL, TX, TY, PERIODIC, COLS, L, LA, CONS, FAR>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    const dim3 grid(tiles_x * tiles_y * ((P.nz + tz - 1) / tz)), block(TX * TY);
    hipLaunchKernelGGL((k_fused<PR, MODEL, TX, TY, PERIODIC, COLS, L, LA, CONS, FAR>), grid, block, lds, s, P, src, dst,
                       flag, tz, tiles_x, tiles_y);
}
template <int PR, int MODEL, int TX, int TY, bool PERIODIC, int COLS, class L, class LA, bool CONS>
void launch_fused_far(const KParams &P, const void *src, void *dst, unsigned *flag, int tz, int tiles_x, int tiles_y,
                      hipStream_t s)
{
    if constexpr (!always_pointers(PR, MODEL, PERIODIC, std::is_same_v<L, D2Q9>, TX == 96)) {
        if (!P.far_rows) {
            launch_fused_one<PR, MODEL, TX, TY, PERIODIC, COLS, L, LA, CONS, false>(P, src, dst, flag, tz, tiles_x, tiles_y, s);
            return;
        }
    }
    launch_fused_one<PR, MODEL, TX, TY, PERIODIC, COLS, L, LA, CONS, true>(P, src, dst, flag, tz, tiles_x, tiles_y, s);
}
template <int PR, int MODEL, int TX, int TY, int COLS, class L, class LA, bool CONS>
void launch_fused_bc(const KParams &P, const void *src, void *dst, unsigned *flag, int tz, int tiles_x, int tiles_y,
                     hipStream_t s)
{
    if (P.bc[0] == 0 && P.bc[1] == 0 && P.bc[2] == 0)
        launch_fused_far<PR, MODEL, TX, TY, true, COLS, L, LA, CONS>(P, src, dst, flag, tz, tiles_x, tiles_y, s);
    else
        launch_fused_far<PR, MODEL, TX, TY, false, COLS, L, LA, CONS>(P, src, dst, flag, tz, tiles_x, tiles_y, s);
}
template <int PR, int MODEL, int TX, int TY, int COLS, bool CONS>
void launch_fused_kernel(const KParams &P, const void *src, void *dst, unsigned *flag, int tz, hipStream_t s)
{
    launch_fused_bc<PR, MODEL, TX, TY, COLS, D3Q19, D3Q19, CONS>(P, src, dst, flag, tz, (P.nx + TX - 1) / TX, P.ny / TY, s);
}

// The mass-keeping collision has kernels of its own, so that the default
// step carries none of it.
template <int PR, int MODEL, int TX, int TY, int COLS>
void launch_fused_shape(const KParams &P, const void *src, void *dst, unsigned *flag, int tz, hipStream_t s)
{
    if constexpr (kConserveRest<PR> && MODEL == CG) {
        if (P.conserve) {
            launch_fused_kernel<PR, MODEL, TX, TY, COLS, true>(P, src, dst, flag, tz, s);
            return;
        }
    }
    launch_fused_kernel<PR, MODEL, TX, TY, COLS, false>(P, src, dst, flag, tz, s);
}

template <int PR, int MODEL, int TY>
void launch_fused_cols(const KParams &P, const FusedShape &sh, const void *src, void *dst, unsigned *flag, hipStream_t s)
{
    if (sh.odd) {
        if constexpr (TY == odd_column_height(PR == 0)) {
            const int tiles_x = (P.nx + 63) / 64, tiles_y = (P.ny + TY - 1) / TY;
            if (P.bc[0] == 0 && P.bc[1] == 0 && P.bc[2] == 0)
                launch_fused_one<PR, MODEL, 64, TY, true, kColsOdd, D3Q19, D3Q19, false, false>(
                    P, src, dst, flag, sh.tz, tiles_x, tiles_y, s);
            else
                launch_fused_one<PR, MODEL, 64, TY, false, kColsOdd, D3Q19, D3Q19, false, false>(
                    P, src, dst, flag, sh.tz, tiles_x, tiles_y, s);
        }
    } else if (!sh.ragged) launch_fused_shape<PR, MODEL, 64, TY, kColsFull>(P, src, dst, flag, sh.tz, s);
    else if (P.nx > 64) launch_fused_shape<PR, MODEL, 64, TY, kColsRagged>(P, src, dst, flag, sh.tz, s);
    else launch_fused_shape<PR, MODEL, 64, TY, kColsNarrow>(P, src, dst, flag, sh.tz, s);
}

template <int PR, int MODEL>
void launch_fused(const KParams &P, const FusedShape &sh, const void *src, void *dst, unsigned *flag, hipStream_t s)
{
    if constexpr (PR != 0) {
        if (sh.tx == 96) {
            launch_fused_shape<PR, MODEL, 96, 4, kColsFull>(P, src, dst, flag, sh.tz, s);
            return;
        }
    }
    if (sh.ty == 4) launch_fused_cols<PR, MODEL, 4>(P, sh, src, dst, flag, s);
    else if constexpr (PR != 0) launch_fused_cols<PR, MODEL, 8>(P, sh, src, dst, flag, s);
}

// D2Q9 one-pass step: the 2-D box as nx x 1 x ny (neighbours placed by
// D2Q9Z, arithmetic in D2Q9), rows of
// 256 nodes marching along y, the last row segment masked when 256 does not
// divide nx.  Chunks of at least 8 rows, about two blocks per compute unit.
constexpr int k2dTX = 256;

inline KParams as_marching_2d(const KParams &P)
{
    KParams Q = P;
    Q.ny = 1;
    Q.nz = P.ny;
    Q.bc[1] = 0;
    Q.bc[2] = P.bc[1];
    return Q;
}

// Automatic choice on D2Q9: rows from 2^19 nodes on (fewer step on tiles), where
// their segments leave few lanes idle.  One-pass over two-pass time, 160 boxes of
// 2^19 to 2^21 nodes: up to 128 wide 1.2-70, above 1.5 lanes per node (258 to 340
// wide) 0.97-1.6, under that 0.7-1.3.
inline bool rows_preferred(const KParams &P)
{
    return P.N >= 1LL << 19 && 2LL * ((P.nx + k2dTX - 1) / k2dTX * k2dTX) <= 3LL * P.nx;
}

// Row segments and rows per block of the 2-D launch (Q: the box as
// nx x 1 x ny).
inline void fused2d_rows(const KParams &Q, int &tiles_x, int &tz)
{
    tiles_x = (Q.nx + k2dTX - 1) / k2dTX;
    const int tiles_z = std::max(1, std::min(512 / tiles_x, Q.nz / 8));
    tz = (Q.nz + tiles_z - 1) / tiles_z;
}

template <int PR, int MODEL, int COLS, bool CONS>
void launch_fused2d_shape(const KParams &Q, const void *src, void *dst, unsigned *flag, hipStream_t s)
{
    int tiles_x = 0, tz = 0;
    fused2d_rows(Q, tiles_x, tz);
    launch_fused_bc<PR, MODEL, k2dTX, 1, COLS, D2Q9, D2Q9Z, CONS>(Q, src, dst, flag, tz, tiles_x, 1, s);
}

template <int PR, int MODEL>
void launch_fused2d(const KParams &P, const void *src, void *dst, unsigned *flag, hipStream_t s)
{
    const KParams Q = as_marching_2d(P);
    if constexpr (kConserveRest<PR> && MODEL == CG) {
        if (P.conserve) {
            if (Q.nx % k2dTX) launch_fused2d_shape<PR, MODEL, kColsRagged, true>(Q, src, dst, flag, s);
            else launch_fused2d_shape<PR, MODEL, kColsFull, true>(Q, src, dst, flag, s);
            return;
        }
    }
    if (Q.nx % k2dTX) launch_fused2d_shape<PR, MODEL, kColsRagged, false>(Q, src, dst, flag, s);
    else launch_fused2d_shape<PR, MODEL, kColsFull, false>(Q, src, dst, flag, s);
}

}  // namespace mclbm
