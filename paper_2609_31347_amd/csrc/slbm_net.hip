// Convolution kernels of the learned warm start (gfx950): 3x3 convolutions as
// implicit GEMMs on MFMA (bf16 inputs, FP32 accumulation), their backward
// passes, a masked MSE and Adam.  See include/solid_lbm_net.h.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "solid_lbm_net.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx8 __attribute__((ext_vector_type(8)));

// FP32 -> bfloat16, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// K of the packed weights: rounded up to the 16 of one bf16 MFMA k-slice.
__host__ __device__ inline int kpad(int K) { return (K + 15) / 16 * 16; }

// A workgroup's pixels: kTileY rows x kTileX columns of one image.
constexpr int kTileX = 32, kTileY = 4, kTilePix = kTileX * kTileY;
constexpr int64_t kCus = 256;                // compute units of an MI355X
constexpr size_t kStageMax = 136 * 1024;     // LDS bytes for the staged input region

// Staged input region of a tile for dilation dil: the tile's pixels and their
// 3x3 taps, zero outside the image, channels of a pixel together.  A pixel
// takes an odd number of words (channels rounded up to even, plus 2): lanes
// that run over pixels or over channels both spread over the LDS banks.
__host__ __device__ inline int region_w(int dil) { return kTileX + 2 * dil; }
__host__ __device__ inline int region_h(int dil) { return kTileY + 2 * dil; }
__host__ __device__ inline int pix_halves(int Cin) { return ((Cin + 1) / 2 | 1) * 2; }
inline size_t region_bytes(int Cin, int64_t dil)
{
    const int64_t px = (kTileX + 2 * dil) * (kTileY + 2 * dil);
    return px > 65536 ? SIZE_MAX : (size_t)px * pix_halves(Cin) * sizeof(uint16_t);
}

// Copies the region of tile (tx, ty) of one image xb [Cin][H][W] to LDS.
// Threads run over the region's pixels (coalesced rows), two channels at once
// (one 4-byte LDS write).
__device__ __forceinline__ void stage_region(const uint16_t* __restrict__ xb, uint16_t* __restrict__ xs, int Cin, int H,
                                             int W, int dil, int tx, int ty)
{
    const int rw = region_w(dil), np = rw * region_h(dil), ph = pix_halves(Cin), HW = H * W;
    const int y0 = ty * kTileY - dil, x0 = tx * kTileX - dil;
    for (int p = threadIdx.x; p < np; p += blockDim.x) {
        const int ry = p / rw, y = y0 + ry, x = x0 + p - ry * rw;
        const bool in = y >= 0 && y < H && x >= 0 && x < W;
        const uint16_t* src = xb + (in ? (int64_t)y * W + x : 0);
        uint32_t* dst = reinterpret_cast<uint32_t*>(xs + (size_t)p * ph);
#pragma unroll 8
        for (int c = 0; c < Cin; c += 2) {
            const uint32_t lo = in ? src[(int64_t)c * HW] : 0u;
            const uint32_t hi = in && c + 1 < Cin ? src[(int64_t)(c + 1) * HW] : 0u;
            dst[c / 2] = lo | hi << 16;
        }
    }
}

// 3x3 convolution as an implicit GEMM on gfx950's v_mfma_f32_32x32x16_bf16:
// one wave = 32 output channels x 32 pixels, the packed weights (A, rows =
// output channels) in LDS.  The B operand (the input at the 3x3 offsets, columns
// = pixels) comes from one of two places.
// STAGE: a workgroup's pixels are a tile of 4 x 32 (a wave a row of it) whose
// input region is copied into LDS first; element k lies at the pixel's place plus
// an offset that a table in LDS holds, and the region's zero rim stands for the
// padding, so a gathered element is one add and one read.
// Otherwise they are 128 consecutive pixels of the image, and every element is
// read from memory (through the L1), with its division and bounds tests.
// The copy of the region is what bounds the first, its instructions the second:
// see fwd_staged.  Operand lanes: row / column =
// lane % 32, k = 8 (lane / 32) + j, j < 8; result register r of lane l holds
// row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
template <bool STAGE>
__global__ __launch_bounds__(256) void k_conv_fwd(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                                 const float* __restrict__ bias, float* __restrict__ y,
                                                 uint16_t* __restrict__ yb, int Cin, int Cout, int H, int W,
                                                 int Kp, int relu, int dil, int ntx, int wide)
{
    extern __shared__ __align__(16) uint16_t smem[];
    const int wp = Kp + 8;                     // row of weights in LDS: 8 rows start on different banks
    uint16_t* wl = smem;                       // [32][wp] weights
    int* off = reinterpret_cast<int*>(wl + 32 * wp);        // [Kp] offsets of k in the region (STAGE)
    uint16_t* xs = reinterpret_cast<uint16_t*>(off + Kp);   // the region
    const int HW = H * W, K = Cin * 9;
    const int tx = blockIdx.x % ntx, ty = blockIdx.x / ntx, b = blockIdx.y;
    const uint16_t* xb = x + (int64_t)b * Cin * HW;
    const int rw = region_w(dil), ph = pix_halves(Cin);
    for (int i = threadIdx.x; i < 4 * Kp; i += 256) {       // 32 Kp halves, 8 at a time
        const int row = i / (Kp / 8), c = i - row * (Kp / 8);
        shortx8 v;
        if (wide) v = *reinterpret_cast<const shortx8*>(w + row * Kp + 8 * c);
        else
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (short)w[row * Kp + 8 * c + j];
        *reinterpret_cast<shortx8*>(wl + row * wp + 8 * c) = v;
    }
    if (STAGE) {
        for (int k = threadIdx.x; k < Kp; k += 256) {
            const int kk = k < K ? k : 0;                   // padding columns multiply zero weights by a staged value
            const int ci = kk / 9, tap = kk - ci * 9;
            off[k] = ((tap / 3) * dil * rw + (tap % 3) * dil) * ph + ci;
        }
        stage_region(xb, xs, Cin, H, W, dil, tx, ty);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, col = lane & 31, kq = (lane >> 5) * 8;
    const int wv = threadIdx.x >> 6;
    const int64_t q = (int64_t)blockIdx.x * kTilePix + 32 * wv + col;
    const bool pv = STAGE ? ty * kTileY + wv < H && tx * kTileX + col < W : q < HW;
    const int py = STAGE ? ty * kTileY + wv : pv ? (int)q / W : 0;
    const int px = STAGE ? tx * kTileX + col : pv ? (int)q - py * W : 0;
    const uint16_t* xp = xs + (size_t)(wv * rw + col) * ph;
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    for (int kb = 0; kb < Kp; kb += 16) {
        const shortx8 av = *reinterpret_cast<const shortx8*>(wl + col * wp + kb + kq);
        shortx8 bv;
        if (STAGE) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const short v = (short)xp[off[kb + kq + j]];
                bv[j] = kb + kq + j < K ? v : (short)0;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = kb + kq + j;
                short v = 0;
                if (pv && k < K) {
                    const int ci = k / 9, tap = k - ci * 9;
                    const int yy = py + (tap / 3 - 1) * dil, xx = px + (tap % 3 - 1) * dil;
                    if (yy >= 0 && yy < H && xx >= 0 && xx < W) v = (short)xb[(int64_t)ci * HW + yy * W + xx];
                }
                bv[j] = v;
            }
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                      acc, 0, 0, 0);
    }
    if (!pv) return;
    const int p = py * W + px;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int co = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (co < Cout) {
            float v = acc[r] + (bias ? bias[co] : 0.0f);
            if (relu) v = v > 0.0f ? v : 0.0f;
            const int64_t o = ((int64_t)b * Cout + co) * HW + p;
            y[o] = v;
            if (yb) yb[o] = f2bf(v);
        }
    }
}

// Whether k_conv_fwd stages: a workgroup of 4 waves takes `lds` bytes of LDS, so
// 160 KiB / lds of them run on a compute unit.  It does while all tiles run at
// once, and beyond that while the copied regions hold at most 4 times the
// image's pixels.  us, 32 -> 32 channels, from memory / staged (with a switch in one
// kernel; by itself either form takes 1 - 2 us less): 32 images of 64 x
// 39, dilation 1 36 / 18, 4 36 / 25, 8 (one workgroup of 84 KiB per compute unit,
// 640 tiles) 36 / 82; one image of them, dilation 8, 26 / 20; 64 images of 128 x
// 77, dilation 1 165 / 93, 4 164 / 152, 8 163 / 482; 32 images of 20 x 200 (2.5 and
// 6 times the pixels), dilation 1 45 / 34, 4 45 / 59; 64 images of 10 x 256,
// dilation 1 (5.1 times) 53 / 71.
inline bool fwd_staged(int64_t B, int64_t H, int64_t W, int64_t dil, size_t lds)
{
    if (lds > 160 * 1024) return false;
    const int64_t tiles = (W + kTileX - 1) / kTileX * ((H + kTileY - 1) / kTileY);
    const int64_t at_once = kCus * std::min<int64_t>(8, 160 * 1024 / (int64_t)lds);
    return B * tiles <= at_once || (kTileX + 2 * dil) * (kTileY + 2 * dil) * tiles <= 4 * H * W;
}

// Weight gradient as a GEMM on the FP32 MFMA v_mfma_f32_32x32x2_f32:
// dw[co][k] = sum over pixels of dz[co][pixel] x~[k][pixel], x~ the input at
// tap k's offset (im2col, bf16 values, exact in FP32).  A workgroup of 16
// waves owns 32 columns k; wave v takes the pixel pairs v, v + 16, ... (A:
// rows co = lane % 32, pixel 2 t + lane / 32; B: column k = lane % 32, same
// pixel), and the 16 partial 32 x 32 blocks are summed in a fixed order in
// LDS: deterministic, no scratch memory.  db[co] = sum of dz (workgroup 0).
__global__ __launch_bounds__(1024) void k_conv_bwd_w(const float* __restrict__ dz, const uint16_t* __restrict__ x,
                                                    float* __restrict__ dw, float* __restrict__ db, int B, int Cin,
                                                    int Cout, int H, int W, int dil)
{
    __shared__ float part[16][16][64];        // [wave][register][lane]
    __shared__ float bsum[16][64];
    const int HW = H * W, K = Cin * 9;
    const int kb = blockIdx.x * 32;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
    // this lane's column k: input channel and tap offset (fixed for the loop)
    const int kk = kb + row;
    const bool kval = kk < K;
    const int ci = kval ? kk / 9 : 0, tap = kval ? kk - ci * 9 : 0;
    const int oy = (tap / 3 - 1) * dil, ox = (tap % 3 - 1) * dil;
    const bool cval = row < Cout;
    const int64_t npair = ((int64_t)B * HW + 1) / 2, P = (int64_t)B * HW;
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    float s = 0.0f;
    for (int64_t t = wv; t < npair; t += 16) {
        const int64_t pix = 2 * t + half;
        float av = 0.0f, bv = 0.0f;
        if (pix < P) {
            const int bb = (int)(pix / HW), p = (int)(pix - (int64_t)bb * HW);
            if (cval) av = dz[((int64_t)bb * Cout + row) * HW + p];
            if (kval) {
                const int py = p / W, px = p - py * W, yy = py + oy, xx = px + ox;
                if (yy >= 0 && yy < H && xx >= 0 && xx < W) bv = bf2f(x[((int64_t)bb * Cin + ci) * HW + yy * W + xx]);
            }
        }
        s += av;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wv][r][lane] = acc[r];
    bsum[wv][lane] = s;
    __syncthreads();
    {
        const int r = threadIdx.x >> 6, l = threadIdx.x & 63;   // one output element per thread
        float v = 0.0f;
        for (int q = 0; q < 16; ++q) v += part[q][r][l];
        const int co = 8 * (r >> 2) + 4 * (l >> 5) + (r & 3), k = kb + (l & 31);
        if (co < Cout && k < K) dw[(int64_t)co * K + k] = v;
    }
    if (blockIdx.x == 0 && db && threadIdx.x < 32 && threadIdx.x < Cout) {
        float v = 0.0f;
        for (int q = 0; q < 16; ++q) v += bsum[q][threadIdx.x] + bsum[q][threadIdx.x + 32];
        db[threadIdx.x] = v;
    }
}

// The same weight gradient over many workgroups: the pixels are split into
// nsplit runs of tiles of kTileY x kTileX pixels; a workgroup keeps its 32 x
// (9 Cin) block of sums in MFMA registers over its run and writes it to the
// workspace, and k_conv_bwd_w_sum adds the runs in a fixed order
// (deterministic).  dz of a tile ([pixel][channel], rows of 33 words) and the
// input region are staged in LDS.  Columns are ordered (tap, ci): a wave owns
// 32 of them, nb = ceil(9 Cin / 32) waves cover all, and with few columns
// `parts` groups of nb waves share the tile's pixels.  FP32 products and sums
// as k_conv_bwd_w.  32 -> 32 channels on 32 images of 64 x 39: 2.06 ms with one
// workgroup per 32 columns (9 of 256 compute units), 48 us here plus 5 us for
// the sum (the FP32 MFMAs alone take about 15 us).
constexpr int kBwdRow = 33;                   // words of a staged dz pixel
// Pixels that the unsplit kernel still does in less time (us, unsplit / split: 32
// channels, 100 pixels 8.4 / 14.1, 256 8.9 / 15.0, 520 14.8 / 18.9, 676 18.7 /
// 15.2; 7 channels, 256 8.8 / 11.3, 400 11.8 / 11.1).
inline int64_t bwd_few(int Cin) { return Cin > 16 ? 576 : 384; }

struct BwdSplit {
    int nb, parts, ntx, nty, run, nsplit;     // see above; run = tiles per workgroup
    size_t lds, words;                        // LDS bytes; FP32 words of workspace
};

// Split of a layer; false if it does not take this path.
inline bool bwd_split(int64_t B, int Cin, int64_t H, int64_t W, int64_t dil, BwdSplit* s)
{
    if (Cin > 56) return false;               // 16 waves of 32 columns
    const size_t xbytes = region_bytes(Cin, dil);
    if (xbytes > kStageMax) return false;
    s->nb = (9 * Cin + 31) / 32;
    s->parts = s->nb <= 2 ? 4 : s->nb <= 4 ? 2 : 1;
    s->ntx = (int)((W + kTileX - 1) / kTileX);
    s->nty = (int)((H + kTileY - 1) / kTileY);
    const int64_t tiles = (int64_t)s->ntx * s->nty * B;
    if (tiles > INT32_MAX) return false;
    s->run = (int)((tiles + kCus - 1) / kCus);   // one workgroup per compute unit
    s->nsplit = (int)((tiles + s->run - 1) / s->run);
    s->lds = (size_t)kTilePix * kBwdRow * sizeof(float) + xbytes;
    s->words = (size_t)s->nsplit * s->parts * (s->nb * 32 + 1) * 32;
    return true;
}

__global__ __launch_bounds__(1024) void k_conv_bwd_w_split(const float* __restrict__ dz, const uint16_t* __restrict__ x,
                                                          float* __restrict__ ws, int B, int Cin, int Cout, int H,
                                                          int W, int dil, int nb, int parts, int ntx, int nty, int run)
{
    extern __shared__ __align__(16) uint16_t smem[];
    float* zs = reinterpret_cast<float*>(smem);
    uint16_t* xs = smem + kTilePix * kBwdRow * 2;
    const int HW = H * W, K = Cin * 9;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
    const int cb = wv % nb, part = wv / nb;
    const int rw = region_w(dil), ph = pix_halves(Cin);
    const int c = cb * 32 + row;                            // column (tap, ci) of this lane's B operand
    const int tap = c < K ? c / Cin : 0, ci = c < K ? c - tap * Cin : 0;
    const int xoff = ((tap / 3) * dil * rw + (tap % 3) * dil) * ph + ci;
    const int per = kTilePix / 2 / parts;                    // pixel pairs of this part
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    float s = 0.0f;
    const int tiles = ntx * nty * B, t0 = blockIdx.x * run, t1 = min(t0 + run, tiles);
    for (int t = t0; t < t1; ++t) {
        const int b = t / (ntx * nty), tt = t - b * (ntx * nty), ty = tt / ntx, tx = tt - ty * ntx;
        __syncthreads();
        stage_region(x + (int64_t)b * Cin * HW, xs, Cin, H, W, dil, tx, ty);
        for (int i = threadIdx.x; i < 32 * kTilePix; i += blockDim.x) {
            const int co = i / kTilePix, p = i - co * kTilePix;
            const int yy = ty * kTileY + p / kTileX, xx = tx * kTileX + p % kTileX;
            const bool in = co < Cout && yy < H && xx < W;
            zs[p * kBwdRow + co] = in ? dz[((int64_t)b * Cout + co) * HW + yy * W + xx] : 0.0f;
        }
        __syncthreads();
        // pixels outside the image have no part, not even that of a zero dz: their taps reach back into the image,
        // and an Inf or NaN there times zero would be a NaN
        const int cols = W - tx * kTileX, end = min((part + 1) * per, (H - ty * kTileY) * (kTileX / 2));
        auto pairs = [&](auto ragged) {
            for (int j = part * per; j < end; j += 8) {             // 8 pairs of one row of the tile
                const int p = 2 * j + half, left = cols - p % kTileX;
                if (decltype(ragged)::value && 2 * j % kTileX >= cols) continue;
                const float* za = zs + p * kBwdRow + row;
                const uint16_t* xa = xs + ((p / kTileX) * rw + p % kTileX) * ph + xoff;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float av = za[2 * u * kBwdRow];
                    const float bv = !decltype(ragged)::value || 2 * u < left ? bf2f(xa[2 * u * ph]) : 0.0f;
                    s += av;
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bv, acc, 0, 0, 0);
                }
            }
        };
        if (cols >= kTileX) pairs(std::false_type());
        else pairs(std::true_type());
    }
    // [split][co][column], then one more column: the sums of dz
    float* out = ws + (size_t)(blockIdx.x * parts + part) * (nb * 32 + 1) * 32;
#pragma unroll
    for (int r = 0; r < 16; ++r) out[(8 * (r >> 2) + 4 * half + (r & 3)) * (nb * 32) + c] = acc[r];
    s += __shfl_xor(s, 32);
    if (cb == 0 && half == 0) out[nb * 32 * 32 + row] = s;
}

// Sums the nsplit partial blocks: 32 consecutive elements per workgroup, 8
// threads per element over the splits, then those 8 in order.
__global__ __launch_bounds__(256) void k_conv_bwd_w_sum(const float* __restrict__ ws, float* __restrict__ dw,
                                                       float* __restrict__ db, int nsplit, int nb, int Cin, int Cout)
{
    const int cols = nb * 32, block = (cols + 1) * 32;
    const int e = blockIdx.x * 32 + (threadIdx.x & 31), part = threadIdx.x >> 5;
    float v = 0.0f;
    if (e < block) {
#pragma unroll 8
        for (int s = part; s < nsplit; s += 8) v += ws[(size_t)s * block + e];
    }
    __shared__ float red[8][32];
    red[part][threadIdx.x & 31] = v;
    __syncthreads();
    if (part || e >= block) return;
    v = red[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < 8; ++q) v += red[q][threadIdx.x];
    if (e < cols * 32) {
        const int co = e / cols, c = e - co * cols, tap = c / Cin, ci = c - tap * Cin;
        if (co < Cout && c < 9 * Cin) dw[(int64_t)co * Cin * 9 + ci * 9 + tap] = v;
    } else if (db && e - cols * 32 < Cout) {
        db[e - cols * 32] = v;
    }
}

__global__ void k_act_bwd(const float* __restrict__ dy, const float* __restrict__ y, float* __restrict__ dz,
                          uint16_t* __restrict__ dzb, int64_t n, int relu)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = relu ? (y[i] > 0.0f ? dy[i] : 0.0f) : dy[i];
    if (dz) dz[i] = v;
    if (dzb) dzb[i] = f2bf(v);
}

__global__ void k_pack(const float* __restrict__ w32, uint16_t* __restrict__ wp, uint16_t* __restrict__ wt,
                       int Cin, int Cout)
{
    const int K = Cin * 9, Kp = kpad(K);
    const int Kt = Cout * 9, Ktp = kpad(Kt);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 32 * Kp) {
        const int co = i / Kp, k = i - co * Kp;
        wp[i] = (co < Cout && k < K) ? f2bf(w32[co * K + k]) : (uint16_t)0;
    }
    if (wt && i < 32 * Ktp) {
        // data gradient: conv with Cout inputs and Cin outputs, taps flipped
        const int ci = i / Ktp, k = i - ci * Ktp;
        uint16_t v = 0;
        if (ci < Cin && k < Kt) {
            const int co = k / 9, tp = k - co * 9;
            v = f2bf(w32[co * K + ci * 9 + (8 - tp)]);
        }
        wt[i] = v;
    }
}

__global__ void k_to_bf16(const float* __restrict__ x, uint16_t* __restrict__ y, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

__global__ void k_mse_grad(const float* __restrict__ y, const float* __restrict__ t, const float* __restrict__ mask,
                           float* __restrict__ dy, int nc, int64_t HW, int64_t n, double inv_norm)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t b = i / (nc * HW), p = i % HW;
    const float m = mask[b * HW + p];
    dy[i] = (float)(2.0 * inv_norm) * m * (y[i] - t[i]);
}

// The two reductions below are one block each; a thread's terms are added in
// the order i = tid, tid + 1024, ..., with kRedBatch loads in flight (one at a
// time took 82 us for the loss and 22 us for the mask on 32 images of 64 x 39, this
// takes 47 and 9).
constexpr int kRedBatch = 16;

__device__ __forceinline__ void block_sum_1024(double s, double scale, double* out)
{
    __shared__ double red[1024];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 512; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0] * scale;
}

// loss = sum mask (y - t)^2 * inv_norm, fixed order; INT: index type that holds n
template <class INT>
__global__ __launch_bounds__(1024) void k_mse_loss(const float* __restrict__ y, const float* __restrict__ t,
                                                  const float* __restrict__ mask, double* __restrict__ loss, int nc,
                                                  INT HW, INT n, double inv_norm)
{
    double s = 0.0;
    for (INT i0 = threadIdx.x; i0 < n; i0 += 1024 * kRedBatch) {
        float a[kRedBatch], c[kRedBatch], m[kRedBatch];
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u) {
            const INT i = i0 + 1024 * u < n ? i0 + 1024 * u : i0;
            const INT b = i / (nc * HW), p = i % HW;
            a[u] = y[i];
            c[u] = t[i];
            m[u] = mask[b * HW + p];
        }
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u)
            if (i0 + 1024 * u < n) {
                const double d = (double)a[u] - (double)c[u];
                s += (double)m[u] * d * d;
            }
    }
    block_sum_1024(s, inv_norm, loss);
}

__global__ __launch_bounds__(1024) void k_mask_sum(const float* __restrict__ mask, int64_t n, double* __restrict__ out)
{
    double s = 0.0;
    for (int64_t i0 = threadIdx.x; i0 < n; i0 += 1024 * kRedBatch) {
        float m[kRedBatch];
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u) m[u] = mask[i0 + 1024 * u < n ? i0 + 1024 * u : i0];
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u)
            if (i0 + 1024 * u < n) s += m[u];
    }
    block_sum_1024(s, 1.0, out);
}

__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

int status(hipError_t e) { return e == hipSuccess ? 0 : -3; }

// Lets a kernel use the whole LDS of the current device; `done` holds a bit per
// device on which that has been set (the attribute belongs to the device).
int allow_lds(const void* kernel, std::atomic<uint64_t>& done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return -3;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0;
    if (done.load(std::memory_order_relaxed) & bit) return 0;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return -3;
    done.fetch_or(bit, std::memory_order_relaxed);
    return 0;
}

}  // namespace

extern "C" {

int slbm_conv3x3_forward(const uint16_t* x, const uint16_t* w, const float* bias, float* y, uint16_t* y_bf16,
                         int32_t B, int32_t Cin, int32_t Cout, int32_t H, int32_t W, int32_t relu, int32_t dilation,
                         void* stream)
{
    if (!x || !w || !y || B < 1 || Cin < 1 || Cout < 1 || Cout > 32 || H < 1 || W < 1 || dilation < 1) return -1;
    const int Kp = kpad(Cin * 9);
    const size_t xbytes = region_bytes(Cin, dilation);
    size_t lds = (size_t)32 * (Kp + 8) * sizeof(uint16_t);
    if ((size_t)64 * Kp > 83 * 1024) return -3;   // over 147 input channels (LDS)
    const int ntx = (W + kTileX - 1) / kTileX, nty = (H + kTileY - 1) / kTileY;
    const size_t slds = lds + (size_t)Kp * sizeof(int) + (xbytes <= kStageMax ? xbytes : 0);
    const bool stage = xbytes <= kStageMax && fwd_staged(B, H, W, dilation, slds);
    if (stage) lds = slds;
    const int wide = ((uintptr_t)w & 15) == 0;   // 16-byte loads of the weights
    static std::atomic<uint64_t> fwd_mem{0}, fwd_staged_form{0};
    const int rc = stage ? allow_lds(reinterpret_cast<const void*>(&k_conv_fwd<true>), fwd_staged_form)
                         : allow_lds(reinterpret_cast<const void*>(&k_conv_fwd<false>), fwd_mem);
    if (rc) return rc;
    const dim3 grid(stage ? (unsigned)ntx * (unsigned)nty : blocks((int64_t)H * W, kTilePix), (unsigned)B);
    hipLaunchKernelGGL(stage ? k_conv_fwd<true> : k_conv_fwd<false>, grid, dim3(256), lds, (hipStream_t)stream, x, w,
                       bias, y, y_bf16, Cin, Cout, H, W, Kp, relu, dilation, ntx, wide);
    return status(hipGetLastError());
}

int64_t slbm_conv3x3_backward_weight_workspace(int32_t B, int32_t Cin, int32_t H, int32_t W, int32_t dilation)
{
    BwdSplit s;
    if (B < 1 || Cin < 1 || H < 1 || W < 1 || dilation < 1 || !bwd_split(B, Cin, H, W, dilation, &s)) return 0;
    return (int64_t)(s.words * sizeof(float));
}

int slbm_conv3x3_backward_weight_ws(const float* dz, const uint16_t* x, float* dw, float* db, int32_t B, int32_t Cin,
                                    int32_t Cout, int32_t H, int32_t W, int32_t dilation, void* ws, int64_t ws_bytes,
                                    void* stream)
{
    if (!dz || !x || !dw || B < 1 || Cin < 1 || Cout < 1 || Cout > 32 || H < 1 || W < 1 || dilation < 1) return -1;
    BwdSplit s;
    if (!ws || (int64_t)B * H * W <= bwd_few(Cin) || !bwd_split(B, Cin, H, W, dilation, &s) ||
        ws_bytes < (int64_t)(s.words * sizeof(float)))
        return slbm_conv3x3_backward_weight(dz, x, dw, db, B, Cin, Cout, H, W, dilation, stream);
    static std::atomic<uint64_t> split{0};
    const int rc = allow_lds(reinterpret_cast<const void*>(&k_conv_bwd_w_split), split);
    if (rc) return rc;
    hipLaunchKernelGGL(k_conv_bwd_w_split, dim3((unsigned)s.nsplit), dim3(64u * s.nb * s.parts), s.lds,
                       (hipStream_t)stream, dz, x, (float*)ws, B, Cin, Cout, H, W, dilation, s.nb, s.parts, s.ntx,
                       s.nty, s.run);
    hipLaunchKernelGGL(k_conv_bwd_w_sum, dim3((unsigned)(s.nb * 32 + 1)), dim3(256), 0, (hipStream_t)stream,
                       (const float*)ws, dw, db, s.nsplit * s.parts, s.nb, Cin, Cout);
    return status(hipGetLastError());
}

int slbm_conv3x3_backward_weight(const float* dz, const uint16_t* x, float* dw, float* db, int32_t B, int32_t Cin,
                                 int32_t Cout, int32_t H, int32_t W, int32_t dilation, void* stream)
{
    if (!dz || !x || !dw || B < 1 || Cin < 1 || Cout < 1 || H < 1 || W < 1 || dilation < 1) return -1;
    if (Cout > 32) return -1;
    hipLaunchKernelGGL(k_conv_bwd_w, dim3((unsigned)((Cin * 9 + 31) / 32)), dim3(1024), 0, (hipStream_t)stream, dz, x,
                       dw, db, B, Cin, Cout, H, W, dilation);
    return status(hipGetLastError());
}

int slbm_act_backward(const float* dy, const float* y, float* dz, uint16_t* dz_bf16, int64_t n, int32_t relu,
                      void* stream)
{
    if (!dy || (relu && !y) || n < 0) return -1;
    if (n == 0) return 0;
    hipLaunchKernelGGL(k_act_bwd, dim3(blocks(n, 256)), dim3(256), 0, (hipStream_t)stream, dy, y, dz, dz_bf16, n,
                       relu);
    return status(hipGetLastError());
}

int slbm_pack_weights(const float* w32, uint16_t* wp, uint16_t* wt, int32_t Cin, int32_t Cout, void* stream)
{
    if (!w32 || !wp || Cin < 1 || Cin > 32 || Cout < 1 || Cout > 32) return -1;
    int n = 32 * (kpad(Cin * 9) > kpad(Cout * 9) ? kpad(Cin * 9) : kpad(Cout * 9));
    hipLaunchKernelGGL(k_pack, dim3(blocks(n, 256)), dim3(256), 0, (hipStream_t)stream, w32, wp, wt, Cin, Cout);
    return status(hipGetLastError());
}

int slbm_to_bf16(const float* x, uint16_t* y, int64_t n, void* stream)
{
    if (!x || !y || n < 0) return -1;
    if (n == 0) return 0;
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks(n, 256)), dim3(256), 0, (hipStream_t)stream, x, y, n);
    return status(hipGetLastError());
}

int slbm_mse(const float* y, const float* t, const float* mask, float* dy, double* loss, int32_t B, int32_t nc,
             int64_t HW, void* stream)
{
    if (!y || !t || !mask || !dy || B < 1 || nc < 1 || HW < 1) return -1;
    hipStream_t s = (hipStream_t)stream;
    // normalisation: nc * sum(mask), computed on the device into loss[0] first
    double* tmp = loss;
    if (!tmp) return -1;
    hipLaunchKernelGGL(k_mask_sum, dim3(1), dim3(1024), 0, s, mask, (int64_t)B * HW, tmp);
    double msum = 0.0;
    hipError_t e = hipMemcpyAsync(&msum, tmp, sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return -3;
    if (!(msum > 0.0)) return -1;
    const double inv = 1.0 / (nc * msum);
    const int64_t n = (int64_t)B * nc * HW;
    hipLaunchKernelGGL(k_mse_grad, dim3(blocks(n, 256)), dim3(256), 0, s, y, t, mask, dy, nc, HW, n, inv);
    if (n < INT32_MAX - 1024 * kRedBatch)
        hipLaunchKernelGGL(k_mse_loss<int32_t>, dim3(1), dim3(1024), 0, s, y, t, mask, loss, nc, (int32_t)HW,
                           (int32_t)n, inv);
    else
        hipLaunchKernelGGL(k_mse_loss<int64_t>, dim3(1), dim3(1024), 0, s, y, t, mask, loss, nc, HW, n, inv);
    return status(hipGetLastError());
}

int slbm_adam(float* w, const float* g, float* m, float* v, int64_t n, float lr, float beta1, float beta2, float eps,
              int32_t t, void* stream)
{
    if (!w || !g || !m || !v || n < 0 || t < 1) return -1;
    if (n == 0) return 0;
    float c1 = 1.0f - powf(beta1, (float)t), c2 = 1.0f - powf(beta2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(blocks(n, 256)), dim3(256), 0, (hipStream_t)stream, w, g, m, v, n, lr, beta1,
                       beta2, eps, c1, c2);
    return status(hipGetLastError());
}

}  // extern "C"
