// tile2d.hpp -- D2Q9 steps of boxes too small to march (fused.hpp's rows): one
// launch per step, or per two steps, over tiles, one node per thread.  Such a
// box is bound by launches and by the latency of one node's step, not by
// bandwidth (its state stays in cache), so the two passes' separate launches
// and the density field's trip through memory are what there is to save.
// Per-node arithmetic and results are the two-pass kernels', bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include "fused.hpp"

namespace mclbm {

// One step: a block owns a TX x TY tile.  Every thread loads its node, the
// first threads also the ring of nodes around the tile; their stencil values
// meet in LDS, then the tile's nodes collide and push.
template <int PR, int MODEL, int TX, int TY, bool PERIODIC>
__global__ __launch_bounds__(TX *TY) void k_tile2d(KParams P, const void *srcp, void *dstp, unsigned *flag)
{
    using L = D2Q9;
    using C = typename Prec<PR>::C;
    using M = typename Prec<PR>::M;
    using FT = typename Prec<PR>::F;
    using S = typename Prec<PR>::S;
    constexpr int K = NComp<MODEL>::n, NF = NField<MODEL>::n, Q = L::Q, NT = TX * TY, HX = TX + 2, PL = HX * (TY + 2);
    __shared__ FT fld[NF][PL];
    const Pops<L, K, S, false> src(srcp, P), dst(dstp, P);
    const HP<C, M> H = make_hp<C, M>(P);
    const int tid = (int)threadIdx.x, lx = tid % TX, ly = tid / TX;
    const int x0 = (int)blockIdx.x * TX, y0 = (int)blockIdx.y * TY;
    const int w = min(TX, P.nx - x0), h = min(TY, P.ny - y0);   // nodes of this tile
    const bool act = lx < w && ly < h;
    const int x = x0 + lx, y = y0 + ly;
    const unsigned n = (unsigned)x + (unsigned)P.nx * (unsigned)y;
    const int slot = (ly + 1) * HX + lx + 1;
    C c[K][Q];
    M dr[2], j[3];
    bool bad = false;
    // ring node r: the rows above and below (corners included), then the columns
    const int ring = 2 * (w + 2) + 2 * h;
    if (act) load_node(src, n, c);
    for (int r = tid; r < ring; r += NT) {
        int rx, ry;
        if (r < 2 * (w + 2)) {
            ry = r < w + 2 ? -1 : h;
            rx = (r < w + 2 ? r : r - (w + 2)) - 1;
        } else {
            const int q = r - 2 * (w + 2);
            rx = q < h ? -1 : w;
            ry = q < h ? q : q - h;
        }
        const unsigned m = (unsigned)stencil_coord(x0 + rx, P.nx, P.bc[0])
                           + (unsigned)P.nx * (unsigned)stencil_coord(y0 + ry, P.ny, P.bc[1]);
        C g[K][Q];
        M d2[2], j2[3];
        load_node(src, m, g);
        node_moments<L, K>(g, d2, j2);
        FT v[NF];
        field_values<MODEL, NF>(H, d2, v);
#pragma unroll
        for (int a = 0; a < NF; ++a) fld[a][(ry + 1) * HX + rx + 1] = v[a];
    }
    if (act) {
        node_moments<L, K>(c, dr, j);
        FT v[NF];
        field_values<MODEL, NF>(H, dr, v);
#pragma unroll
        for (int a = 0; a < NF; ++a) fld[a][slot] = v[a];
        bad = node_bad(H.rho0[0] + dr[0] + (K == 2 ? H.rho0[1] + dr[1] : M(0)), j[0] + j[1] + j[2]);
    }
    __syncthreads();
    if (act) {
        C v[NF][Q];
#pragma unroll
        for (int a = 0; a < NF; ++a) {
            v[a][0] = C(0);
#pragma unroll
            for (int i = 1; i < Q; ++i) v[a][i] = (C)fld[a][slot + L::cy[i] * HX + L::cx[i]];
        }
        collide_values<L, MODEL, kConsShared<PR>>(H, c, dr, j, v, MODEL == SC_MP ? (C)fld[0][slot] : C(0));
        push_store<L, PERIODIC>(P, dst, x, y, 0, n, c);
    }
    flag_if_bad(flag, bad);
}

// Two steps of an all-periodic box: a block steps a TX x TY tile of nodes with
// three rings around it, (TX + 6) x (TY + 6) threads.  The first step is
// computed for the tile and two rings (the third supplies their stencil
// values), its populations stream through LDS, the second step for the tile,
// which pushes to memory.  The outer rings' first step is computed by several
// blocks alike.
template <int PR, int MODEL, int TX, int TY>
__global__ __launch_bounds__((TX + 6) * (TY + 6)) void k_tile2d_two(KParams P, const void *srcp, void *dstp, unsigned *flag)
{
    using L = D2Q9;
    using C = typename Prec<PR>::C;
    using M = typename Prec<PR>::M;
    using FT = typename Prec<PR>::F;
    using S = typename Prec<PR>::S;
    constexpr int K = NComp<MODEL>::n, NF = NField<MODEL>::n, Q = L::Q, RX = TX + 6, RY = TY + 6, NT = RX * RY;
    __shared__ FT fld[NF][NT];
    __shared__ S pop[K][Q][NT];   // in storage precision, as between two launches
    const Pops<L, K, S, false> src(srcp, P), dst(dstp, P);
    const HP<C, M> H = make_hp<C, M>(P);
    const int t = (int)threadIdx.x, rx = t % RX, ry = t / RX;
    const int x0 = (int)blockIdx.x * TX, y0 = (int)blockIdx.y * TY;
    // the node, wrapped (a box may be smaller than the region)
    const int x = (x0 + rx - 3 + 4 * P.nx) % P.nx, y = (y0 + ry - 3 + 4 * P.ny) % P.ny;
    const unsigned n = (unsigned)x + (unsigned)P.nx * (unsigned)y;
    // distance from the region's edge, and whether the node is this tile's
    const int edge = min(min(rx, RX - 1 - rx), min(ry, RY - 1 - ry));
    const bool mine = edge >= 3 && x0 + rx - 3 < P.nx && y0 + ry - 3 < P.ny;
    C c[K][Q];
    M dr[2], j[3];
    bool bad = false;
    auto moments = [&]() {
        node_moments<L, K>(c, dr, j);
        FT v[NF];
        field_values<MODEL, NF>(H, dr, v);
#pragma unroll
        for (int a = 0; a < NF; ++a) fld[a][t] = v[a];
        if (mine) bad = bad || node_bad(H.rho0[0] + dr[0] + (K == 2 ? H.rho0[1] + dr[1] : M(0)), j[0] + j[1] + j[2]);
    };
    auto collide = [&]() {
        C v[NF][Q];
#pragma unroll
        for (int a = 0; a < NF; ++a) {
            v[a][0] = C(0);
#pragma unroll
            for (int i = 1; i < Q; ++i) v[a][i] = (C)fld[a][t + L::cy[i] * RX + L::cx[i]];
        }
        collide_values<L, MODEL, kConsShared<PR>>(H, c, dr, j, v, MODEL == SC_MP ? (C)fld[0][t] : C(0));
    };
    load_node(src, n, c);
    moments();
    __syncthreads();
    if (edge >= 1) {
        collide();
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i) pop[k][i][t] = (S)c[k][i];
    }
    __syncthreads();
    if (edge >= 2) {
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < Q; ++i) c[k][i] = (C)pop[k][i][t - L::cy[i] * RX - L::cx[i]];
        moments();
    }
    __syncthreads();
    if (mine) {
        collide();
        push_store_periodic<L, false>(P, dst, x, y, 0, n, c);
    }
    flag_if_bad(flag, bad);
}

// Shapes (FP32 / FP64 colour gradient, us per step; two-pass launches first).
// One step: 64 x 8 tiles, whole rows of a wave: 600^2 17.4 -> 14.9, 711 x 701
// 23.3 -> 20.8, 300^2 with walls 11.8 -> 9.2 (16 x 4 tiles 28.3, 40, 10.3);
// 16 x 4 where that leaves most compute units idle (100 x 75 with walls 8.1 ->
// 5.5, 64 x 8 6.2).
// Two steps, the box periodic: 8 x 8 tiles where there are few (64^2 FP64 8.2
// -> 3.3, 128^2 7.0 -> 3.4 / 8.6 -> 4.5; 16 x 16: 4.3, 3.9 / 5.0), then
// 10 x 10 (256^2 FP32 9.1 -> 5.4; 8 x 8 5.6, 16 x 16 6.3), in FP64, whose
// blocks step more slowly, 16 x 16 (256^2 13.2 -> 6.3, 8 x 8 7.3; 400^2 18.3 ->
// 11.6).  Beyond, the rings' extra work (threefold at 8 x 8) outweighs the
// launch saved: 400^2 FP64 12.6 with one step a launch, 600^2 FP32 14.9
// against 18.
constexpr long long kTile2dFew = 1 << 14;
constexpr long long kTile2dSmall = 1 << 15;
template <int PR> constexpr int kTile2dLarge = PR == 0 ? 16 : 10;
template <int PR> constexpr long long kTile2dTwoNodes = PR == 0 ? 1 << 18 : 1 << 17;

// Thin boxes leave most of a tile's lanes without a node (4 x 44370 FP64 with
// walls on 64 x 8 tiles: 72.6 us, two-pass launches 18.4).  Lanes per row of
// TX-wide tiles, over the box (idle rows cost little: 82271 x 2 FP32 8.9 us,
// two-pass 12.0):
inline long long tile2d_lanes(const KParams &P, int tx) { return (P.nx + tx - 1LL) / tx * tx * P.ny; }
// 64 x 8 tiles up to 2.2 lanes per node (nx = 28: 12.0 and 11.7 two-pass; 31:
// 12.7 and 14.8; 15 and 20 wide boxes 1.06-1.5 times the two-pass time), or
// where all fit the chip at once (20 x 1888: 5.3 and 7.3).
inline bool tile2d_wide(const KParams &P)
{
    const long long lanes = tile2d_lanes(P, 64);
    return 5 * lanes <= 11 * P.N || lanes <= 1 << 17;
}
// 16 x 4 tiles up to 2^16 lanes (4 x 1041: 5.5 and 7.0; 2 x 10665, 170000
// lanes, 8.0 and 6.8; 10 x 4885, 78000, 9.9 and 9.0).
inline bool tile2d_narrow(const KParams &P) { return tile2d_lanes(P, 16) <= 1 << 16; }
// Two steps: the tiles' nodes, idle ones among them, within a quarter more than
// the most nodes (6 x 11636: 6.1 and 7.9; 2 x 37184, fivefold: 18.0 and 8.2), on
// 8 x 8 tiles twice as many (2 x 11358: 5.5 and 6.0; 3 x 8620 FP64 9.1 and 7.6).
template <int PR>
bool tile2d_two(const KParams &P)
{
    const int T = P.N <= kTile2dSmall ? 8 : kTile2dLarge<PR>;
    const long long nodes = tile2d_lanes(P, T) / P.ny * ((P.ny + T - 1LL) / T * T);
    return P.bc[0] == 0 && P.bc[1] == 0 && P.N <= kTile2dTwoNodes<PR>
           && (T == 8 ? nodes <= 2 * kTile2dSmall : 4 * nodes <= 5 * kTile2dTwoNodes<PR>);
}

// Launches the tile kernels take over from the two passes.
template <int PR>
int tile2d_steps(const KParams &P)
{
    if (P.N >= 1LL << 19) return 0;   // rows, or two-pass launches
    return (tile2d_wide(P) || tile2d_narrow(P) ? kTileOne : 0) | (tile2d_two<PR>(P) ? kTileTwo : 0);
}

template <int PR, int MODEL, int T>
void launch_tile2d_two(const KParams &P, const void *src, void *dst, unsigned *flag, hipStream_t s)
{
    hipLaunchKernelGGL((k_tile2d_two<PR, MODEL, T, T>), dim3((P.nx + T - 1) / T, (P.ny + T - 1) / T),
                       dim3((T + 6) * (T + 6)), 0, s, P, src, dst, flag);
}

template <int PR, int MODEL, int TX, int TY>
void launch_tile2d_one(const KParams &P, const void *src, void *dst, unsigned *flag, hipStream_t s)
{
    const dim3 grid((P.nx + TX - 1) / TX, (P.ny + TY - 1) / TY), block(TX * TY);
    if (P.bc[0] == 0 && P.bc[1] == 0)
        hipLaunchKernelGGL((k_tile2d<PR, MODEL, TX, TY, true>), grid, block, 0, s, P, src, dst, flag);
    else
        hipLaunchKernelGGL((k_tile2d<PR, MODEL, TX, TY, false>), grid, block, 0, s, P, src, dst, flag);
}

template <int PR, int MODEL>
void launch_tile2d(const KParams &P, const void *src, void *dst, unsigned *flag, int steps, hipStream_t s)
{
    if (steps == 2) {
        if (P.N <= kTile2dSmall) launch_tile2d_two<PR, MODEL, 8>(P, src, dst, flag, s);
        else launch_tile2d_two<PR, MODEL, kTile2dLarge<PR>>(P, src, dst, flag, s);
        return;
    }
    if (tile2d_narrow(P) && (P.N <= kTile2dFew || !tile2d_wide(P))) launch_tile2d_one<PR, MODEL, 16, 4>(P, src, dst, flag, s);
    else launch_tile2d_one<PR, MODEL, 64, 8>(P, src, dst, flag, s);
}

}  // namespace mclbm
