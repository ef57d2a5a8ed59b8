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
// 1.78, 448^2 2.76 / 1.88, 512^2 2.87 / 2.18, 600^2 3.27 / 2.47, 700^2 3.62 /
// 3.23; 800^2 4.14 / 4.25 (no gain: strips stay).
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
};

// Edge rows: 2 parities x waves x 6 populations x 64 columns.
constexpr int kPanelEdge = 2 * kPanelWaves * 6 * 64;

template <bool EFIELD, bool ADJ, int R>
__device__ __forceinline__ void panel_tile(const PanelArgs& a, int tile, double* edge)
{
    constexpr int W = kPanelWaves;
    // planes pulled from the row below (A: none, x - 1, x + 1) and above (B: none, x + 1, x - 1)
    constexpr int A0 = ADJ ? 3 : 1, A1 = ADJ ? 6 : 4, A2 = ADJ ? 7 : 5;
    constexpr int B0 = ADJ ? 1 : 3, B1 = ADJ ? 4 : 6, B2 = ADJ ? 5 : 7;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, h = a.halo;
    const int64_t N = a.N;
    constexpr int RY = W * R;
    const int x0 = (tile % a.tiles_x) * (64 - 2 * h) - h, y0 = (tile / a.tiles_x) * (RY - 2 * h) - h;
    const int x = wrapi(x0 + lane, nx);
    const bool colin = lane >= h && lane < 64 - h && x0 + lane < nx;   // columns this tile writes
    double o[R][8], c0[R], c1[R], rk11[R], rks[R];
    int64_t cell[R];
    {
        int y = wrapi(y0 + w * R, ny);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t n = (int64_t)y * nx + x;
            cell[r] = n;
#pragma unroll
            for (int q = 0; q < 8; ++q) o[r][q] = ldg(a.src + q * N + n);
            c0[r] = ldg(a.g + n);
            c1[r] = ldg(a.g + N + n);
            if (EFIELD) rk11[r] = ldg(a.E + n);
            y = y + 1 == ny ? 0 : y + 1;
        }
    }
    auto publish = [&](int par) {
        double* e = edge + (size_t)(par * W + w) * 6 * 64 + lane;
        e[0] = o[R - 1][A0];
        e[64] = o[R - 1][A1];
        e[128] = o[R - 1][A2];
        e[192] = o[0][B0];
        e[256] = o[0][B1];
        e[320] = o[0][B2];
    };
    publish(0);
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
    const int lm = max(lane - 1, 0), lp = min(lane + 1, 63);
    for (int s = 1; s <= a.steps; ++s) {
        __syncthreads();
        const int m = h - (a.steps - s);                 // this sweep computes rows [m, RY - m)
        if (w * R + R <= m || w * R >= RY - m) continue;
        const double* eb = edge + (size_t)(((s - 1) & 1) * W + max(w - 1, 0)) * 6 * 64;
        const double* ea = edge + ((size_t)(((s - 1) & 1) * W + min(w + 1, W - 1)) * 6 + 3) * 64;
        const double la[3] = {eb[lane], eb[64 + lm], eb[128 + lp]};
        const double lb[3] = {ea[lane], ea[64 + lp], ea[128 + lm]};
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
            const double k11 = EFIELD ? rk11[r] : a.k11, ks = EFIELD ? rks[r] : a.ks, kd = EFIELD ? rk11[r] : a.kd;
            if (!ADJ) {
                double d0, d1;
                collide_bulk(f, c0[r], c1[r], k11, ks, kd, d0, d1);
            } else {
                adj_collide_bulk(f, c0[r], c1[r], k11, ks, kd);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) o[r][q] = f[q];
        };
        // rows 1 .. R - 1 first (row R - 1 reads the edge above), row 0 last:
        // the edges' LDS latency is covered by the rows that need none
        if (R > 1) {
            const double sb[3] = {o[1][B0], lane_down(o[1][B1]), lane_up(o[1][B2])};
            double ca[3] = {o[0][A0], lane_up(o[0][A1]), lane_down(o[0][A2])};
#pragma unroll
            for (int r = 1; r < R; ++r) {
                const double na[3] = {o[r][A0], lane_up(o[r][A1]), lane_down(o[r][A2])};
                if (r < R - 1) {
                    const int t = r + 1 < R ? r + 1 : r;
                    const double b[3] = {o[t][B0], lane_down(o[t][B1]), lane_up(o[t][B2])};
                    row(r, ca, b);
                } else {
                    row(r, ca, lb);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) ca[k] = na[k];
            }
            row(0, la, sb);
        } else {
            row(0, la, lb);
        }
        if (s < a.steps) publish(s & 1);
    }
    if (!colin) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int ry = w * R + r;
        if (ry < h || ry >= RY - h || y0 + ry >= ny) continue;
#pragma unroll
        for (int q = 0; q < 8; ++q) stg(a.dst + q * N + cell[r], o[r][q]);
    }
}

template <bool EFIELD, bool ADJ, int R>
__global__ __launch_bounds__(kPanelBlock) void k_sweep_panel(PanelArgs a)
{
    if (a.status->stop) return;
    __shared__ __align__(16) double edge[kPanelEdge];
    panel_tile<EFIELD, ADJ, R>(a, xcd_order(blockIdx.x, gridDim.x), edge);
}

}  // namespace slbm
