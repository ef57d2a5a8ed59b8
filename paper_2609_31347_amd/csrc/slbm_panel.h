// Fused sweeps with register-resident nodes (gfx950): several time steps of a
// panel of the grid per launch.
#pragma once
#include "slbm_kernels.h"

namespace slbm {

// A workgroup of kPanelWaves waves owns a region of 64 columns x (waves x R)
// rows: lane = column, each lane keeps R consecutive rows of its column in
// registers (populations, source term, relaxation), wave w the rows w R ..
// w R + R - 1.  A sweep moves populations between columns with whole-wave lane
// shifts, between a lane's rows by register names, and only the six
// populations that cross the wave's top and bottom rows go through LDS (two
// copies by sweep parity, one barrier per sweep).  Of the region, a halo of
// `halo` nodes on every side is recomputed; the rest is written back after
// `steps` <= halo sweeps.
//
// Panels of 32 columns (WC; R = 2) hold two row blocks per wave, one in each
// half: their neighbours' rows come from LDS as between waves, and the lane
// shifts that cross the halves bring values to the outermost columns only, which
// are halo.  Their region, 32 x 32, is the LDS tiles' with a third of the LDS
// accesses and no index arithmetic: a launch of 8 steps at 256^2 takes 8.6 us
// against 10.3, of which about 3.4 are the launch and 2.4 the loads.  Their first
// sweep may be a residual check (CHECK): the wave sums follow the last sweep.
//
// The arithmetic per node is the single-step kernels' own (collide_bulk,
// adj_collide_bulk), so a launch of k sweeps equals k single sweeps bit for
// bit.
//
// What bounds it: a launch costs about 3 us (launch gap, one round trip for
// the loads, the stores' drain), 1 us per row of a lane (all planes of 64
// columns x R rows per wave come through one compute unit at about 34 B/ns)
// and 0.18 us per row and sweep (46 VALU instructions per node-step at two
// waves per SIMD).  The LDS tiles (one node per thread, 16 LDS accesses per
// node-step) need a quarter of the region per compute unit for the same time,
// so on grids of more nodes than 16 x 16 tiles can cover in one round of
// workgroups the panels win.  us per primal step, before (strips or two rounds
// of tiles) / panel: 300^2 2.24 / 1.57, 371^2 2.60 / 1.65, 501 x 333 2.64 /
// 1.78, 448^2 2.76 / 1.88, 512^2 2.87 / 2.18, 600^2 3.27 / 2.47; from 700^2 the
// wave pipeline is faster (3.21 against 3.37).
//
// Plates (k_sweep_plate): four more waves run the boundary nodes, one per lane
// with its record, closure values and relaxation in registers.  In a sweep the
// bulk waves pull and collide all their nodes as above, the lanes of boundary
// nodes put the pulled populations into LDS, the boundary waves apply the node
// map, and those lanes take the result back (two more barriers, only in tiles
// that have boundary nodes).  The closure values of cut links (primal) and the
// node's own slots of them (adjoint) stay with the boundary lane; ghost slots
// in HBM are read at the start and written at the end of a launch.  What the
// lanes of outside nodes compute is never read: every link between a domain
// node and an outside node is a cut link.  The handover's LDS writes (a full
// instruction for the few lanes of a row) make a sweep of a rim tile about
// twice an inner tile's; the workgroups' order starts the rim tiles first, so
// that inner tiles fill the time a compute unit has left.  Against LDS tiles,
// us per primal step: 384 x 231 3.16 -> 2.57, 512 x 308 (E field) 3.65 -> 2.65,
// 1000 x 600 (E field) 9.95 -> 5.81.  Packing the boundary nodes inside the bulk
// waves instead (no barriers) took 4.6 at 512 x 308; handing them over before
// the bulk rows are collided, so that both run at once, the same time.
constexpr int kPanelWaves = 8;
constexpr int kPanelBlock = 64 * kPanelWaves;

struct PanelArgs {
    const double* __restrict__ src;
    double* __restrict__ dst;
    const double* __restrict__ g;     // primal: forcing; adjoint: r
    const double* __restrict__ E;     // E plane or null
    const Status* __restrict__ status;
    int32_t nx, ny;
    int64_t N;
    double k11, ks, kd, nu, scale;
    int32_t halo, steps, tiles_x;
    // launches whose first sweep is a residual check: the state of the last check, sums by workgroup
    double* __restrict__ snap;
    double* __restrict__ partial;
    // plates
    const int32_t* __restrict__ code;
    const BNode* __restrict__ bnodes;
    double E0;
    // launch plan of the shape (k_panel_plan): by place in the plan, per slot (cell,
    // cut | dirichlet << 8 | written << 16) and 32 coefficient planes of kPanelCap
    // (kPanelStride words in all); by workgroup, its boundary nodes
    const int2* __restrict__ plan;
    const double* __restrict__ plan_coef;
    const int32_t* __restrict__ plan_n;
    const int32_t* __restrict__ tiles;    // tile of each workgroup
    int32_t rims;                         // tiles with boundary nodes: the first of every XCD's run
};

// Boundary nodes that a workgroup takes (plates): kPanelBWaves waves, one node per lane.
constexpr int kPanelBWaves = 4;
constexpr int kPanelCap = 64 * kPanelBWaves;
// Words of a tile's coefficient planes in the plan: not a power of two (64 KiB
// apart the adjoint's steps of 32-column panels took 4 % longer, the primal's 1.5 %
// less: 360 x 216 2.23 and 2.27 us, 2.14 and 2.30 so).
constexpr int kPanelStride = 32 * kPanelCap + 544;
constexpr int kPlateBlock = 64 * (kPanelWaves + kPanelBWaves);

// Edge rows: 2 parities x waves x 6 populations x 64 columns.
constexpr int kPanelEdge = 2 * kPanelWaves * 6 * 64;

__device__ __forceinline__ int panel_slot(int e) { return (e % kPanelBWaves) * 64 + e / kPanelBWaves; }

// The bulk waves of a tile.  MASKED: io holds 8 doubles per boundary slot,
// cnt the boundary nodes per wave, nbt the tile's.
template <bool MASKED, bool EFIELD, bool ADJ, int R, int WC, bool CHECK = false>
__device__ __forceinline__ void panel_tile(const PanelArgs& a, int tile, double* edge, double2* io, int* cnt, int nbt)
{
    constexpr int HW = 64 / WC, W = kPanelWaves * HW;    // row blocks per wave, in all
    // planes pulled from the row below (A: none, x - 1, x + 1) and above (B: none, x + 1, x - 1)
    constexpr int A0 = ADJ ? 3 : 1, A1 = ADJ ? 6 : 4, A2 = ADJ ? 7 : 5;
    constexpr int B0 = ADJ ? 1 : 3, B1 = ADJ ? 4 : 6, B2 = ADJ ? 5 : 7;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, h = a.halo;
    const int64_t N = a.N;
    constexpr int RY = W * R;
    const int x0 = (tile % a.tiles_x) * (WC - 2 * h) - h, y0 = (tile / a.tiles_x) * (RY - 2 * h) - h;
    const int col = lane % WC, v = w * HW + lane / WC;   // column and row block of this lane
    const int x = wrapi(x0 + col, nx);
    const bool colin = col >= h && col < WC - h && x0 + col < nx;      // columns this tile writes
    double o[R][8], c0[R], c1[R], rk11[R], rks[R];
    int64_t cell[R];
    int cd[R], bs[R];
    double s0[CHECK ? R : 1], s1[CHECK ? R : 1], num = 0.0, den = 0.0;
    bool own[CHECK ? R : 1];
    {
        int y = wrapi(y0 + v * R, ny);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t n = (int64_t)y * nx + x;
            cell[r] = n;
            cd[r] = MASKED ? ldg(a.code + n) : 0;
#pragma unroll
            for (int q = 0; q < 8; ++q) o[r][q] = ldg(a.src + q * N + n);
            c0[r] = ldg(a.g + n);
            c1[r] = ldg(a.g + N + n);
            if (EFIELD) rk11[r] = ldg(a.E + n);
            if (CHECK) {
                const int ry = v * R + r;
                own[r] = colin && ry >= h && ry < RY - h && y0 + ry < ny;
                s0[r] = own[r] ? ldg(a.snap + n) : 0.0;
                s1[r] = own[r] ? ldg(a.snap + N + n) : 0.0;
            }
            y = y + 1 == ny ? 0 : y + 1;
        }
    }
    auto publish = [&](int par) {
        double* e = edge + (size_t)(par * W + v) * 6 * WC + col;
        e[0] = o[R - 1][A0];
        e[WC] = o[R - 1][A1];
        e[2 * WC] = o[R - 1][A2];
        e[3 * WC] = o[0][B0];
        e[4 * WC] = o[0][B1];
        e[5 * WC] = o[0][B2];
    };
    publish(0);
    uint32_t rowb = 0;                                   // rows with boundary nodes
    if (MASKED && nbt) {
        const uint64_t below = __lanemask_lt();
        int nbw = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t b = __ballot(cd[r] > 0);
            bs[r] = nbw + __popcll(b & below);
            nbw += __popcll(b);
            if (b) rowb |= 1u << r;
        }
        if (lane == 0) cnt[w] = nbw;
        __syncthreads();
        int base = 0;
        for (int k = 0; k < w; ++k) base += cnt[k];
#pragma unroll
        for (int r = 0; r < R; ++r) bs[r] = panel_slot(base + bs[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        c0[r] = (ADJ ? a.scale : 0.25) * c0[r];
        c1[r] = (ADJ ? a.scale : 0.25) * c1[r];
        if (EFIELD) {
            const Relax<double> rl = relax_from_E<double>(rk11[r], a.nu, false);
            rk11[r] = rl.k11;
            rks[r] = rl.ks;
        }
    }
    const int lm = max(col - 1, 0), lp = min(col + 1, WC - 1);
    for (int s = 1; s <= a.steps; ++s) {
        __syncthreads();
        const int m = h - (a.steps - s);                 // this sweep computes rows [m, RY - m)
        if ((w + 1) * HW * R <= m || w * HW * R >= RY - m) {
            if (MASKED && nbt) {
                __syncthreads();
                __syncthreads();
            }
            continue;
        }
        const double* eb = edge + (size_t)(((s - 1) & 1) * W + max(v - 1, 0)) * 6 * WC;
        const double* ea = edge + ((size_t)(((s - 1) & 1) * W + min(v + 1, W - 1)) * 6 + 3) * WC;
        const double la[3] = {eb[col], eb[WC + lm], eb[2 * WC + lp]};
        const double lb[3] = {ea[col], ea[WC + lp], ea[2 * WC + lm]};
        auto row = [&](int r, const double (&A)[3], const double (&B)[3]) {
            double f[8];
            f[0] = ADJ ? lane_down(o[r][0]) : lane_up(o[r][0]);
            f[2] = ADJ ? lane_up(o[r][2]) : lane_down(o[r][2]);
            f[A0] = A[0];
            f[A1] = A[1];
            f[A2] = A[2];
            f[B0] = B[0];
            f[B1] = B[1];
            f[B2] = B[2];
            if (MASKED && ((rowb >> r) & 1u)) {
                if (cd[r] > 0) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) io[q * kPanelCap + bs[r]] = make_double2(f[2 * q], f[2 * q + 1]);
                }
            }
            const double k11 = EFIELD ? rk11[r] : a.k11, ks = EFIELD ? rks[r] : a.ks, kd = EFIELD ? rk11[r] : a.kd;
            double d0, d1;
            if (CHECK && ADJ) {
                d0 = (f[0] - f[2]) + (f[4] - f[5]) + (f[7] - f[6]);
                d1 = (f[1] - f[3]) + (f[4] + f[5]) - (f[6] + f[7]);
            }
            if (!ADJ) collide_bulk(f, c0[r], c1[r], k11, ks, kd, d0, d1);
            else adj_collide_bulk(f, c0[r], c1[r], k11, ks, kd);
            if (CHECK && s == 1 && own[r]) {
                num += (d0 - s0[r]) * (d0 - s0[r]) + (d1 - s1[r]) * (d1 - s1[r]);
                den += d0 * d0 + d1 * d1;
                stg(a.snap + cell[r], d0);
                stg(a.snap + N + cell[r], d1);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) o[r][q] = f[q];
        };
        // rows 1 .. R - 1 first (row R - 1 reads the edge above), row 0 last:
        // the edges' LDS latency is covered by the rows that need none
        const double sb[3] = {o[1][B0], lane_down(o[1][B1]), lane_up(o[1][B2])};
        double ca[3] = {o[0][A0], lane_up(o[0][A1]), lane_down(o[0][A2])};
#pragma unroll
        for (int r = 1; r < R; ++r) {
            const double na[3] = {o[r][A0], lane_up(o[r][A1]), lane_down(o[r][A2])};
            if (r < R - 1) {
                const double b[3] = {o[r + 1][B0], lane_down(o[r + 1][B1]), lane_up(o[r + 1][B2])};
                row(r, ca, b);
            } else {
                row(r, ca, lb);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) ca[k] = na[k];
        }
        row(0, la, sb);
        if (MASKED && nbt) {
            __syncthreads();
            __syncthreads();
            // two rows' reads in flight at a time
#pragma unroll
            for (int r0 = 0; r0 < R; r0 += 2)
                if ((rowb >> r0) & 3u) {
                    double2 t[2][4];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (r0 + k < R && cd[r0 + k] > 0) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) t[k][q] = io[q * kPanelCap + bs[r0 + k]];
                        }
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (r0 + k < R) {
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                o[r0 + k][2 * q] = cd[r0 + k] > 0 ? t[k][q].x : o[r0 + k][2 * q];
                                o[r0 + k][2 * q + 1] = cd[r0 + k] > 0 ? t[k][q].y : o[r0 + k][2 * q + 1];
                            }
                        }
                }
        }
        if (s < a.steps) publish(s & 1);
    }
    if (CHECK) block_sum2_tile<kPanelBlock>(num, den, a.partial + 2 * (int64_t)tile);
    if (!colin) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int ry = v * R + r;
        if (ry < h || ry >= RY - h || y0 + ry >= ny) continue;
        if (MASKED && cd[r] < 0) continue;
#pragma unroll
        for (int q = 0; q < 8; ++q) stg(a.dst + q * N + cell[r], o[r][q]);
    }
}


// The boundary waves of a plate tile: wave b, lane j runs entry 4 j + b of the
// tile's list, with its record, closure values and relaxation in registers.
template <bool EFIELD, bool ADJ>
__device__ __forceinline__ void panel_boundary(const PanelArgs& a, int place, int b, double2* io, int nbt)
{
    const int lane = threadIdx.x & 63, nx = a.nx;
    const int64_t N = a.N;
    const int slot = 64 * b + lane;
    const bool on = kPanelBWaves * lane + b < nbt;
    const int64_t at = (int64_t)place * kPanelCap + (on ? slot : 0);   // a tile with boundary nodes has slot 0
    const int2 en = a.plan[at];
    BNode bn;
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int j = 0; j < (ADJ ? 3 : 4); ++j)
            bn.coef[q][j] = ldg(a.plan_coef + (int64_t)place * kPanelStride + (4 * q + j) * kPanelCap + (on ? slot : 0));
    const int64_t cell = en.x;
    bn.cut = (uint32_t)en.y & 0xffu;
    bn.dirichlet = ((uint32_t)en.y >> 8) & 0xffu;
    const bool written = on && (en.y >> 16);
    double st[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        // primal: the ghost slot of the cut link (inside the box: domain nodes
        // do not lie on its edge); adjoint: the node's own slot
        st[q] = ldg(a.src + q * N + (ADJ ? cell : cell - ((bn.cut >> q) & 1u ? cx(q) + cy(q) * nx : 0)));
        if (!((bn.cut >> q) & 1u)) st[q] = 0.0;
    }
    double gg[2] = {ldg(a.g + cell), ldg(a.g + N + cell)};
    if (ADJ) {
        gg[0] = a.scale * gg[0];
        gg[1] = a.scale * gg[1];
    }
    const Relax<double> rl = relax_from_E<double>(EFIELD ? ldg(a.E + cell) : a.E0, a.nu, true);
    __syncthreads();
    for (int s = 1; s <= a.steps; ++s) {
        __syncthreads();
        __syncthreads();
        if (on) {
            double f[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double2 v = io[q * kPanelCap + slot];
                f[2 * q] = v.x;
                f[2 * q + 1] = v.y;
            }
            if (!ADJ) {
                double fC[8], mb[5];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if ((bn.cut >> q) & 1u) f[q] = st[q];
                node_map<double>(f, gg, rl, &bn, true, fC, st, mb);
#pragma unroll
                for (int q = 0; q < 4; ++q) io[q * kPanelCap + slot] = make_double2(fC[2 * q], fC[2 * q + 1]);
            } else {
                double out[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)              // the populations of outside nodes are zero
                    if ((bn.cut >> opp(q)) & 1u) f[q] = 0.0;
                adj_boundary(f, st, &bn, rl, gg[0], gg[1], out);
#pragma unroll
                for (int q = 0; q < 4; ++q) io[q * kPanelCap + slot] = make_double2(out[2 * q], out[2 * q + 1]);
#pragma unroll
                for (int q = 0; q < 8; ++q) st[q] = ((bn.cut >> q) & 1u) ? out[q] : 0.0;
            }
        }
        __syncthreads();
    }
    if (!ADJ && written) {
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if ((bn.cut >> q) & 1u) stg(a.dst + q * N + cell - (cx(q) + cy(q) * nx), st[q]);
    }
}

template <bool EFIELD, bool ADJ, int R, int WC, bool CHECK>
__global__ __launch_bounds__(kPanelBlock) void k_sweep_panel(PanelArgs a)
{
    if (a.status->stop) return;
    __shared__ __align__(16) double edge[kPanelEdge];
    panel_tile<false, EFIELD, ADJ, R, WC, CHECK>(a, xcd_order(blockIdx.x, gridDim.x), edge, nullptr, nullptr, 0);
}

template <bool EFIELD, bool ADJ, int R, int WC>
__global__ __launch_bounds__(kPlateBlock) void k_sweep_plate(PanelArgs a)
{
    if (a.status->stop) return;
    extern __shared__ __align__(16) double lds[];        // edge rows, then 8 doubles per boundary slot
    __shared__ int cnt[kPanelWaves];
    const int wg = xcd_order(blockIdx.x, gridDim.x);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = a.tiles[wg];
    const int nbt = a.plan_n[wg];
    double2* io = reinterpret_cast<double2*>(lds + kPanelEdge);
    if (w < kPanelWaves) panel_tile<true, EFIELD, ADJ, R, WC>(a, tile, lds, io, cnt, nbt);
    else if (nbt) panel_boundary<EFIELD, ADJ>(a, xcd_order(blockIdx.x, a.rims), w - kPanelWaves, io, nbt);
}

// Launch plan of a plate's panels (grid: that of the sweeps): the boundary nodes
// of every region in region order, spread over the boundary waves, with their
// records in planes, so that a boundary wave loads consecutive words.
__global__ __launch_bounds__(kPanelBlock) void k_panel_plan(PanelArgs a, int R, int cols, int2* plan, double* coef, int32_t* plan_n)
{
    const int b = blockIdx.x, wg = xcd_order(b, gridDim.x), tile = a.tiles[wg], lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int place = xcd_order(b, a.rims);
    const bool rim = b / kXcds < a.rims / kXcds + (b % kXcds < a.rims % kXcds ? 1 : 0);
    const int h = a.halo, HW = 64 / cols, RY = kPanelWaves * HW * R;
    const int x0 = (tile % a.tiles_x) * (cols - 2 * h) - h, y0 = (tile / a.tiles_x) * (RY - 2 * h) - h;
    const int col = lane % cols, row0 = (w * HW + lane / cols) * R;
    const int x = wrapi(x0 + col, a.nx);
    const bool colin = col >= h && col < cols - h && x0 + col < a.nx;
    __shared__ int cnt[kPanelWaves];
    int mine = 0;
    for (int r = 0; r < R; ++r) mine += __popcll(__ballot(a.code[(int64_t)wrapi(y0 + row0 + r, a.ny) * a.nx + x] > 0));
    if (lane == 0) cnt[w] = mine;
    __syncthreads();
    int at = 0, total = 0;
    for (int v = 0; v < kPanelWaves; ++v) {
        if (v < w) at += cnt[v];
        total += cnt[v];
    }
    for (int r = 0; r < R; ++r) {
        const int ry = row0 + r;
        const int64_t n = (int64_t)wrapi(y0 + ry, a.ny) * a.nx + x;
        const int code = a.code[n];
        const uint64_t b = __ballot(code > 0);
        const int e = at + __popcll(b & __lanemask_lt());
        const bool wr = colin && ry >= h && ry < RY - h && y0 + ry < a.ny;
        if (code > 0 && rim && e < kPanelCap) {
            const BNode& bn = a.bnodes[code - 1];
            const int s = panel_slot(e);
            plan[(int64_t)place * kPanelCap + s] = make_int2((int)n, (int)(bn.cut | bn.dirichlet << 8 | (wr ? 1u << 16 : 0u)));
            for (int k = 0; k < 32; ++k) coef[(int64_t)place * kPanelStride + k * kPanelCap + s] = bn.coef[k / 4][k % 4];
        }
        at += __popcll(b);
    }
    if (threadIdx.x == 0) plan_n[wg] = rim ? min(total, kPanelCap) : 0;
}

}  // namespace slbm
