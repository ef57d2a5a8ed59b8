// Fused sweeps of large periodic, uniform-material grids (gfx950): a strip's
// pipeline of time levels spread over the waves of a workgroup.
#pragma once
#include "slbm_kernels.h"

namespace slbm {

// T = L S time steps per launch.  A workgroup of S waves owns a strip of 128
// columns (two adjacent columns per lane; 128 - 2 T of them written) and H
// output rows.  Wave s runs levels s L + 1 .. (s + 1) L of the pipeline that
// k_sweep_tb runs in one wave: a row enters level 0 once per iteration, level k
// computes step t + k - 1 of the row k behind it from the register histories of
// level k - 1.  The first wave loads rows from HBM (one iteration ahead), each
// wave hands its last level's rows and their forcing to the next one through
// LDS (two buffers, one barrier per iteration), the last wave stores.
//
// One wave's registers hold 8 levels of one column, and 8 steps per launch
// leave large grids bound by HBM (2048^2: 604 MB at least in 152 us, 4.0 TB/s
// of a copy's 5.0 - 5.4).  With S = 8 waves of L = 2 levels (205 VGPRs, two
// waves per SIMD, 140 KiB of LDS: one workgroup per compute unit) a launch does
// 16 steps for those bytes: 2048^2 215 us, 13.4 us per step against 19.0, now
// bound by FP64 issue at the clock that the power leaves it (1.3 - 1.5 GHz; the
// vector units issue in 80 - 85 % of its cycles).  Hence what saves
// instructions counts: loops by role and no branch around a row's work (copies
// where paths join: 15.6 -> 15.0 us), 4 rows per trip (the histories' registers
// come round: no copies) and waves that idle until their first useful row
// (-> 13.6).  L = 3, S = 4 in two workgroups per compute unit takes the same
// there (13.9) but 8 % more at 1024^2, and spills for odd nx; L = 2,
// S = 4 is bound by HBM again (18.1).  Half of the waves shifted by half a row,
// to compute while the others use LDS, was slower (two barriers per row).

// One level: row y of step t + k from the histories of the rows y - 1 (p2) and
// y (p1) and the incoming row y + 1 (o), which becomes the result.
template <bool ADJ>
__device__ __forceinline__ void pipe_level(double (&p2)[2][3], double (&p1a)[2][3], double (&p1b)[2][2],
                                           const double (&gh)[2][2], double (&o)[2][8], const TBArgs& a)
{
    constexpr int A0 = ADJ ? 3 : 1, A1 = ADJ ? 6 : 4, A2 = ADJ ? 7 : 5;   // planes pulled from row y-1
    double f[2][8];
    // x - 1 of column 0 is column 1 of the lane before, x + 1 of column 1 column 0 of the lane after
    if (!ADJ) {
        f[0][0] = lane_up(p1b[1][0]);
        f[1][0] = p1b[0][0];
        f[0][2] = p1b[1][1];
        f[1][2] = lane_down(p1b[0][1]);
        f[0][4] = lane_up(p2[1][1]);
        f[1][4] = p2[0][1];
        f[0][5] = p2[1][2];
        f[1][5] = lane_down(p2[0][2]);
        f[0][6] = o[1][6];
        f[1][6] = lane_down(o[0][6]);
        f[0][7] = lane_up(o[1][7]);
        f[1][7] = o[0][7];
    } else {
        f[0][0] = p1b[1][0];
        f[1][0] = lane_down(p1b[0][0]);
        f[0][2] = lane_up(p1b[1][1]);
        f[1][2] = p1b[0][1];
        f[0][6] = lane_up(p2[1][1]);
        f[1][6] = p2[0][1];
        f[0][7] = p2[1][2];
        f[1][7] = lane_down(p2[0][2]);
        f[0][4] = o[1][4];
        f[1][4] = lane_down(o[0][4]);
        f[0][5] = lane_up(o[1][5]);
        f[1][5] = o[0][5];
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        f[c][A0] = p2[c][0];
        f[c][ADJ ? 1 : 3] = o[c][ADJ ? 1 : 3];
        p2[c][0] = p1a[c][0];
        p2[c][1] = p1a[c][1];
        p2[c][2] = p1a[c][2];
        p1a[c][0] = o[c][A0];
        p1a[c][1] = o[c][A1];
        p1a[c][2] = o[c][A2];
        p1b[c][0] = o[c][0];
        p1b[c][1] = o[c][2];
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        if (!ADJ) {
            double d0, d1;
            collide_bulk(f[c], gh[c][0], gh[c][1], a.k11, a.ks, a.kd, d0, d1);
        } else {
            adj_collide_bulk(f[c], gh[c][0], gh[c][1], a.k11, a.ks, a.kd);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) o[c][q] = f[c][q];
    }
}

typedef double pair_t __attribute__((ext_vector_type(2)));
constexpr int kPipeCols = 128;
constexpr int kPipeRow = 10 * kPipeCols;              // a handed-over row: 8 populations, 2 forcings
template <int S>
constexpr size_t pipe_lds_bytes() { return (size_t)(S - 1) * 2 * kPipeRow * sizeof(double); }

// Barrier that orders LDS only: the prefetched rows stay in flight.
__device__ __forceinline__ void pipe_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// EVEN: nx is even, so a lane's two columns are one 16-byte aligned pair.
template <int L, int S, bool ADJ, bool EVEN>
__global__ __launch_bounds__(64 * S) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sweep_pipe(TBArgs a)
{
    if (a.status->stop) return;
    extern __shared__ __align__(16) double lds[];
    constexpr int T = L * S, V = kPipeCols - 2 * T;
    constexpr int XOFF = V % 16 == 0 ? T : 0;         // strips start on 128-byte lines (when a row does)
    const int wg = xcd_order(blockIdx.x, gridDim.x);
    const int sx = wg % a.strips, sy = wg / a.strips;
    const int lane = threadIdx.x & 63;
    const int stage = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny;
    const int64_t N = a.N;
    const int xs = sx * V - T + XOFF + 2 * lane;      // unwrapped first column of this lane
    const int xa = wrapi(xs, nx), xb = xa + 1 == nx ? 0 : xa + 1;
    const bool out_a = 2 * lane >= T && 2 * lane < kPipeCols - T && xs < nx + XOFF;
    const bool out_b = 2 * lane >= T && 2 * lane < kPipeCols - T && xs + 1 < nx + XOFF;
    const int y0 = sy * a.H, y1 = min(y0 + a.H, ny);
    const int rows = y1 - y0;
    double p2[L][2][3], p1a[L][2][3], p1b[L][2][2], gh[L][2][2];
#pragma unroll
    for (int k = 0; k < L; ++k)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            p2[k][c][0] = p2[k][c][1] = p2[k][c][2] = 0.0;
            p1a[k][c][0] = p1a[k][c][1] = p1a[k][c][2] = 0.0;
            p1b[k][c][0] = p1b[k][c][1] = 0.0;
            gh[k][c][0] = gh[k][c][1] = 0.0;
        }
    const double gsc = ADJ ? a.scale : 0.25;
    auto load = [&](int row, double (&v)[2][8], double (&g)[2][2]) {
        const int64_t base = (int64_t)row * nx;
        auto pair = [&](const double* p, double& u, double& w) {
            if (EVEN) {
                const pair_t t = *(const __attribute__((address_space(1))) pair_t*)(p + base + xa);
                u = t.x;
                w = t.y;
            } else {
                u = ldg(p + base + xa);
                w = ldg(p + base + xb);
            }
        };
#pragma unroll
        for (int q = 0; q < 8; ++q) pair(a.src + q * N, v[0][q], v[1][q]);
        pair(a.g, g[0][0], g[1][0]);
        pair(a.g + N, g[0][1], g[1][1]);
    };
    // Stage s takes input row y0 - T + it - s (L + 1) in iteration it; its first
    // useful one is y0 - T + s L, its last y1 - 1 + T - s L.  It only joins the
    // barriers before and after these.  The rows are rounded up to whole trips of
    // the loop: a row past the last is computed from valid buffers and not stored.
    const int first = stage * (2 * L + 1), trips = (rows + 2 * T - stage * 2 * L + 3) / 4;
    const int after = rows + 2 * T + S + 2 - first - 4 * trips;
    const double* in0 = lds + (size_t)((stage - 1) * 2 + (~first & 1)) * kPipeRow + 2 * lane;   // first read
    const double* in1 = lds + (size_t)((stage - 1) * 2 + (first & 1)) * kPipeRow + 2 * lane;
    double* out0 = lds + (size_t)(stage * 2 + (first & 1)) * kPipeRow + 2 * lane;
    double* out1 = lds + (size_t)(stage * 2 + (~first & 1)) * kPipeRow + 2 * lane;
    for (int it = 0; it < first; ++it) pipe_barrier();
    auto levels = [&](double (&o)[2][8], const double (&g)[2][2], double (&go)[2][2]) {
#pragma unroll
        for (int k = 0; k < L; ++k) pipe_level<ADJ>(p2[k], p1a[k], p1b[k], gh[k], o, a);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                go[c][j] = gh[L - 1][c][j];
#pragma unroll
                for (int k = L - 1; k > 0; --k) gh[k][c][j] = gh[k - 1][c][j];
                gh[0][c][j] = g[c][j];
            }
    };
    auto take = [&](int par, double (&o)[2][8], double (&g)[2][2]) {
        const double* p = par ? in1 : in0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double2 t = *reinterpret_cast<const double2*>(p + q * kPipeCols);
            o[0][q] = t.x;
            o[1][q] = t.y;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double2 t = *reinterpret_cast<const double2*>(p + (8 + j) * kPipeCols);
            g[0][j] = t.x;
            g[1][j] = t.y;
        }
    };
    auto give = [&](int par, const double (&o)[2][8], const double (&g)[2][2]) {
        double* p = par ? out1 : out0;
#pragma unroll
        for (int q = 0; q < 8; ++q) *reinterpret_cast<double2*>(p + q * kPipeCols) = make_double2(o[0][q], o[1][q]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *reinterpret_cast<double2*>(p + (8 + j) * kPipeCols) = make_double2(g[0][j], g[1][j]);
    };
    // one loop per role, four rows per trip
    if (stage == 0) {
        double nv[2][8], ng[2][2];                    // the next row
        int rw = wrapi(y0 - T, ny);                   // its index
        load(rw, nv, ng);
        auto step = [&](int par) {
            double o[2][8], g[2][2], go[2][2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int q = 0; q < 8; ++q) o[c][q] = nv[c][q];
                g[c][0] = gsc * ng[c][0];
                g[c][1] = gsc * ng[c][1];
            }
            rw = rw + 1 == ny ? 0 : rw + 1;
            load(rw, nv, ng);
            levels(o, g, go);
            give(par, o, go);
            pipe_barrier();
        };
        for (int it = 0; it < trips; ++it) {
            step(0);
            step(1);
            step(0);
            step(1);
        }
    } else if (stage < S - 1) {
        auto step = [&](int par) {
            double o[2][8], g[2][2], go[2][2];
            take(par, o, g);
            levels(o, g, go);
            give(par, o, go);
            pipe_barrier();
        };
        for (int it = 0; it < trips; ++it) {
            step(0);
            step(1);
            step(0);
            step(1);
        }
    } else {
        int yo = y0 - T + (S - 1) * L - L;            // the row that this iteration completes
        auto step = [&](int par) {
            double o[2][8], g[2][2], go[2][2];
            take(par, o, g);
            levels(o, g, go);
            if (yo >= y0 && yo < y1) {
                const int64_t base = (int64_t)yo * nx;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    double* d = a.dst + q * N + base;
                    if (EVEN) {
                        if (out_a) *(__attribute__((address_space(1))) pair_t*)(d + xa) = pair_t{o[0][q], o[1][q]};
                    } else {
                        if (out_a) stg(d + xa, o[0][q]);
                        if (out_b) stg(d + xb, o[1][q]);
                    }
                }
            }
            ++yo;
            pipe_barrier();
        };
        for (int it = 0; it < trips; ++it) {
            step(0);
            step(1);
            step(0);
            step(1);
        }
    }
    for (int it = 0; it < after; ++it) pipe_barrier();
}

}  // namespace slbm
