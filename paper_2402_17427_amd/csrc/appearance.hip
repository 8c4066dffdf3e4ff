// Kernels of the decoupled appearance model (gs_appearance_*).
//
// VastGaussian (arXiv 2402.17427), section 4.2 and supplement S1.1: the
// rendered image is downsampled 32 times, an appearance embedding is
// concatenated to every pixel, and a CNN (3x3 convolution to 256 channels;
// four blocks of pixel shuffle, 3x3 convolution halving the channels, ReLU;
// bilinear interpolation to the image size; 3x3 convolution, ReLU, 3x3
// convolution to 3 channels) produces the transformation map M; the
// adjusted image is I^r * M.
//
// Every layer works on planar FP32 maps [C][H][W].  Convolutions with more
// than four output channels are implicit GEMMs on the matrix cores
// (k_conv_mfma); the 3-channel map M takes the matrix cores' 4 x 4 outer
// products (k_conv_few).  Both stage rows of 64 columns with their one-pixel
// halo and the weights of a few input channels at a time in LDS, loading the
// next channels meanwhile; the same kernels run the transposed convolutions
// of the backward (weights read flipped and transposed) with the layer's
// ReLU mask applied to the input as it is staged, and write their output in
// the next layer's (or the layer before's) pixel-shuffled order.  The
// low-resolution layers split their input channels over several workgroups
// whose partial sums a second kernel adds in a fixed order.  Weight
// gradients are per-workgroup partial sums over pixel tiles on the matrix
// cores, reduced in a fixed order by a second kernel, so every result is
// deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace gs {

namespace {

constexpr int kT = 256;
constexpr int kCI = 8;             // input channels staged per round
constexpr int kFC = 4;             // the same for the few-output kernel
constexpr int kTile = 16;          // tile edge that the input-channel splits count workgroups by
constexpr int kFewWgs = 5;         // its workgroups a CU
constexpr int kCR = 4;             // rows of a convolution's pixel tile
constexpr int kWR = 4, kWC = 64;   // pixel tile of the weight gradient: a row a wave, a column a lane

constexpr int kXcds = 8;   // XCDs of an MI355X; workgroups are dealt to them round-robin

// Tile (x, y) of a workgroup of a 2D tile grid, in an XCD-aware order: the
// workgroups dealt to one XCD take a contiguous band of tiles (in row
// order), so horizontally adjacent tiles, which share halo columns and the
// cache lines of their output rows, go through the same L2.
__device__ __forceinline__ void xcd_tile(int* tx, int* ty) {
    const int nx = (int)gridDim.x, n = nx * (int)gridDim.y;
    const int b = (int)blockIdx.y * nx + (int)blockIdx.x;
    const int per = n / kXcds;
    const int t = b < per * kXcds ? (b % kXcds) * per + b / kXcds : b;
    *ty = t / nx;
    *tx = t - *ty * nx;
}

// A window of N channels of planar maps [C][H][W], rows y0 .. y0 + R - 1 and
// columns x0 .. x0 + kWave - 1, on its way to LDS: CH = N / 4 consecutive
// channels a wave, a lane a column.  load() issues the loads (of the next
// step, before the current one is computed), store() writes row r of channel
// c to dst + c pitch + r row_pitch + lane.  Elements outside the map, and
// channels from C on, are zero; MASK: also where the mask map is <= 0 (the
// ReLU mask of a backward pass).  A row's address is scalar work and a lane
// adds nothing but its column, where an element-by-element loop spends some
// thirty vector instructions an element on divisions and 64-bit products.
// plain (the window lies inside the map) leaves out the clamps and selects:
// a tenth of the scalar instructions.  The selects come with the LDS store
// because one right after a load waits for that load.
template <int CH, int R, bool MASK>
struct Rows {
    float v[CH * R], m[MASK ? CH * R : 1];
    __device__ __forceinline__ void load(const float* __restrict__ src, const float* __restrict__ mask, int c0, int C,
                                         int y0, int x0, int H, int W, bool plain) {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
        const int64_t HW = (int64_t)H * W;
        if (plain) {
            const int64_t q = (int64_t)(c0 + CH * wave) * HW + (int64_t)y0 * W + x0;
            const float *p = src + q, *pm = MASK ? mask + q : nullptr;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    v[c * R + r] = p[lane];
                    p += W;
                    if (MASK) {
                        m[c * R + r] = pm[lane];
                        pm += W;
                    }
                }
                p += HW - R * (int64_t)W;
                if (MASK) pm += HW - R * (int64_t)W;
            }
            return;
        }
        const int col = min(max(x0 + lane, 0), W - 1);
        int64_t ch = (int64_t)min(c0 + CH * wave, C - 1) * HW;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            int64_t q = ch + (int64_t)min(max(y0, 0), H - 1) * W;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int y = y0 + r;
                v[c * R + r] = (src + q)[col];
                if (MASK) m[c * R + r] = (mask + q)[col];
                q += y >= 0 && y + 1 < H ? W : 0;
            }
            ch += c0 + CH * wave + c + 1 < C ? HW : 0;
        }
    }
    __device__ __forceinline__ void store(float* dst, int pitch, int row_pitch, int c0, int C, int y0, int x0, int H,
                                          int W, bool plain) const {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
        const int x = x0 + lane;
        float* d = dst + CH * wave * pitch + lane;
        if (plain) {
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int k = c * R + r;
                    d[c * pitch + r * row_pitch] = !MASK || m[MASK ? k : 0] > 0.f ? v[k] : 0.f;
                }
            return;
        }
        const bool in = x >= 0 && x < W;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const bool ok = c0 + CH * wave + c < C;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = c * R + r, y = y0 + r;
                const bool on = ok && y >= 0 && y < H && in && (!MASK || m[MASK ? k : 0] > 0.f);
                d[c * pitch + r * row_pitch] = on ? v[k] : 0.f;
            }
        }
    }
};

// The two columns right of those, x and x + 1, of N channels of R rows, an
// element a thread; store() writes them from column `at` of the rows.
template <int N, int R, bool MASK>
struct Edge {
    static_assert(2 * N * R <= kT, "an element a thread");
    float v, m;
    bool on;
    __device__ __forceinline__ void load(const float* __restrict__ src, const float* __restrict__ mask, int c0, int C,
                                         int y0, int x, int H, int W, bool plain) {
        const int k = (int)threadIdx.x, j = k >> 1;
        const int dc = j / R, dy = j % R;
        if (plain) {
            const int64_t q = ((int64_t)c0 * H + y0) * W + x;                  // the same for all threads
            const int64_t at = j < N * R ? ((int64_t)dc * H + dy) * W + (k & 1) : 0;
            v = (src + q)[at];
            if (MASK) m = (mask + q)[at];
            on = true;
            return;
        }
        const int c = c0 + dc, y = y0 + dy, xx = x + (k & 1);
        const bool ok = j < N * R && c < C && y >= 0 && y < H && xx >= 0 && xx < W;
        const int64_t q = ok ? ((int64_t)c * H + y) * W + xx : 0;
        v = src[q];
        if (MASK) m = mask[q];
        on = ok;
    }
    __device__ __forceinline__ void store(float* dst, int pitch, int row_pitch, int at) const {
        const int k = (int)threadIdx.x, j = k >> 1;
        if (j < N * R) dst[j / R * pitch + j % R * row_pitch + at + (k & 1)] = on && (!MASK || m > 0.f) ? v : 0.f;
    }
};

// whether channels c0 .. c0 + n - 1, rows y0 .. y0 + r - 1 and columns x0 ..
// x0 + w - 1 all lie inside [C][H][W]
__device__ __forceinline__ bool inside(int c0, int n, int C, int y0, int r, int H, int x0, int w, int W) {
    return c0 + n <= C && y0 >= 0 && y0 + r <= H && x0 >= 0 && x0 + w <= W;
}

__global__ __launch_bounds__(kT) void k_down_concat(const float* __restrict__ img, int H, int W, int h, int w,
                                                    const float* __restrict__ embed, int m, float* __restrict__ D) {
    __shared__ float red[kT / kWave][2];
    const int by = blockIdx.x / w, bx = blockIdx.x - by * w;
    const int64_t HW = (int64_t)H * W, hw = (int64_t)h * w;
    const int ny = min(32, H - 32 * by), nx = min(32, W - 32 * bx);
    for (int c = 0; c < 3; ++c) {
        float s = 0.f;
        for (int k = threadIdx.x; k < 1024; k += kT) {
            const int yy = k >> 5, xx = k & 31;
            if (yy < ny && xx < nx) s += img[c * HW + (int64_t)(32 * by + yy) * W + 32 * bx + xx];
        }
        for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave][0] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.f;
            for (int k = 0; k < kT / kWave; ++k) t += red[k][0];
            D[c * hw + blockIdx.x] = t / (float)(ny * nx);
        }
        __syncthreads();
    }
    for (int k = threadIdx.x; k < m; k += kT) D[(3 + k) * hw + blockIdx.x] = embed[k];
}

// d_img[c][y][x] += g[c][y/32][x/32] / (pixels of that block)
__global__ __launch_bounds__(kT) void k_down_adjoint(const float* __restrict__ g, int H, int W, int h, int w,
                                                     float* __restrict__ d_img) {
    const int64_t HW = (int64_t)H * W;
    const int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (q >= 3 * HW) return;
    const int c = (int)(q / HW);
    const int64_t p = q - c * HW;
    const int y = (int)(p / W), x = (int)(p - (int64_t)y * W);
    const int by = y >> 5, bx = x >> 5;
    const int ny = min(32, H - 32 * by), nx = min(32, W - 32 * bx);
    d_img[q] += g[(int64_t)c * h * w + (int64_t)by * w + bx] / (float)(ny * nx);
}

// Which pixel tiles a workgroup of a persistent grid works on, t_beg,
// t_beg + t_step, ... < t_end: the workgroups dealt to one XCD (blockIdx.x %
// kXcds) walk a contiguous band of tiles, so neighbouring tiles' halos share
// an L2.
__device__ __forceinline__ void tile_run(int n_tiles, int* t_beg, int* t_end, int* t_step) {
    *t_beg = (int)blockIdx.x;
    *t_end = n_tiles;
    *t_step = (int)gridDim.x;
    if (gridDim.x % kXcds == 0) {
        const int xcd = (int)blockIdx.x % kXcds;
        *t_beg = (int)((int64_t)n_tiles * xcd / kXcds) + (int)blockIdx.x / kXcds;
        *t_end = (int)((int64_t)n_tiles * (xcd + 1) / kXcds);
        *t_step = (int)gridDim.x / kXcds;
    }
}

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

// Weight element (k = tap, channel ci) of output channel o: forward w[o][ci][t];
// transposed w[ci][o][8 - t] of the forward layer (its output channel ci,
// input channel o).
__device__ __forceinline__ int64_t weight_at(const ConvArgs& a, int o, int ci, int t) {
    return a.transposed ? ((int64_t)ci * a.CinF + o) * 9 + (8 - t) : ((int64_t)o * a.Cin + ci) * 9 + t;
}

// Layers of at most four output channels (the map M), on the matrix cores
// with v_mfma_f32_4x4x1_16b_f32 (sixteen 4 x 4 outer products, FP32): lane =
// pixel column, out[o][column] += w[o][k] x[k][column], the four weights of
// one (channel, tap) in the other operand, so no matrix row is padding but
// the absent fourth output.  A wave computes four rows of 64 columns, and
// the sum runs over channels, then taps, like the vector kernel's it
// replaced (the same bits).  The grid is persistent as in k_conv_mfma.  The
// epilogue also writes the adjusted image and the copy of M the caller
// wanted (each a pass over memory of its own before: 14 and 8 us).  16 to 3
// channels at 1600 x 1066: 62 us for 191 MB with the epilogue's; the vector
// kernel took 68 without.  Eight channels a round: 77.
template <bool MASK>
__global__ __launch_bounds__(kT, kFewWgs) void k_conv_few(ConvArgs a) {
    constexpr int R = 4, TR = 4 * R, SR = TR + 2, SC = kWave + 2;
    __shared__ float s_in[kFC * SR * SC];
    __shared__ float s_w[kFC * 9 * 4];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int64_t HW = (int64_t)a.H * a.W;
    const int tiles_x = (a.W + kWave - 1) / kWave, tiles_y = (a.H + TR - 1) / TR;
    int t, t_end, t_step;
    tile_run(tiles_x * tiles_y, &t, &t_end, &t_step);
    if (t >= t_end) return;
    mfma_f4 bias, acc[R];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        const float b = a.b ? a.b[o < a.Cout ? o : 0] : 0.f;
        bias[o] = o < a.Cout ? b : 0.f;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = bias;
    Rows<kFC / 4, SR, MASK> rx;
    constexpr int kEdge = kFC * SR * 2, kWts = kFC * 9 * 4;
    constexpr int JE = (kEdge + kT - 1) / kT, JW = (kWts + kT - 1) / kT;
    float ev[JE], em[JE], wv[JW];
    int y0 = t / tiles_x * TR, x0 = (t % tiles_x) * kWave, c0 = 0;
    bool plain = false;
    auto load = [&] {
        plain = inside(c0, kFC, a.Cin, y0 - 1, SR, a.H, x0 - 1, kWave, a.W);
        rx.load(a.in, a.mask, c0, a.Cin, y0 - 1, x0 - 1, a.H, a.W, plain);
#pragma unroll
        for (int e = 0; e < JE; ++e) {
            const int k = (int)threadIdx.x + e * kT, j = k >> 1;
            const int c = c0 + j / SR, y = y0 - 1 + j % SR, x = x0 + kWave - 1 + (k & 1);
            const bool ok = k < kEdge && c < a.Cin && y >= 0 && y < a.H && x < a.W;
            const int64_t q = ok ? ((int64_t)c * a.H + y) * a.W + x : 0;
            ev[e] = a.in[q];
            em[e] = MASK ? a.mask[q] : 1.f;
        }
#pragma unroll
        for (int e = 0; e < JW; ++e) {
            const int k = (int)threadIdx.x + e * kT, ci = c0 + k / 36, tap = k / 4 % 9, o = k % 4;
            wv[e] = a.w[k < kWts && ci < a.Cin && o < a.Cout ? weight_at(a, o, ci, tap) : 0];
        }
    };
    load();
    while (true) {
        __syncthreads();
        rx.store(s_in, SR * SC, SC, c0, a.Cin, y0 - 1, x0 - 1, a.H, a.W, plain);
#pragma unroll
        for (int e = 0; e < JE; ++e) {
            const int k = (int)threadIdx.x + e * kT, j = k >> 1;
            const int c = c0 + j / SR, y = y0 - 1 + j % SR, x = x0 + kWave - 1 + (k & 1);
            const bool ok = c < a.Cin && y >= 0 && y < a.H && x < a.W && em[e] > 0.f;
            if (k < kEdge) s_in[j * SC + kWave + (k & 1)] = ok ? ev[e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < JW; ++e) {
            const int k = (int)threadIdx.x + e * kT;
            if (k < kWts) s_w[k] = c0 + k / 36 < a.Cin && k % 4 < a.Cout ? wv[e] : 0.f;
        }
        __syncthreads();
        const int cy = y0, px = x0 + lane, cn = min(kFC, a.Cin - c0);   // this step; then the next
        c0 += kFC;
        const bool last = c0 >= a.Cin;
        if (last) {
            c0 = 0;
            t += t_step;
            y0 = t / tiles_x * TR;
            x0 = (t - t / tiles_x * tiles_x) * kWave;
        }
        if (t < t_end) load();
        for (int c = 0; c < cn; ++c) {
            float v[R + 2][3], w[9];
            const float* src = s_in + (c * SR + R * wave) * SC + lane;
#pragma unroll
            for (int r = 0; r < R + 2; ++r)
#pragma unroll
                for (int k = 0; k < 3; ++k) v[r][k] = src[r * SC + k];
#pragma unroll
            for (int k = 0; k < 9; ++k) w[k] = s_w[(c * 9 + k) * 4 + (lane & 3)];
#pragma unroll
            for (int k = 0; k < 9; ++k)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[k], v[r + k / 3][k % 3], acc[r], 0, 0, 0);
        }
        if (!last) continue;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int py = cy + R * wave + r;
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                if (o >= a.Cout || py >= a.H || px >= a.W) continue;
                const int64_t q = (int64_t)o * HW + (int64_t)py * a.W + px;
                const float v = a.relu ? fmaxf(acc[r][o], 0.f) : acc[r][o];
                a.out[q] = v;
                if (a.img) a.adj[q] = a.img[q] * v;
                if (a.copy) a.copy[q] = v;
            }
            acc[r] = bias;
        }
        if (t >= t_end) return;
    }
}

// Where a convolution's output (o, y, x) goes besides, or instead of, the
// plain map: SHUF: the pixel-shuffled map [Cout / 4][2 H][2 W] (the next
// layer's input), element (o / 4, 2 y + (o >> 1 & 1), 2 x + (o & 1));
// UNSHUF: that map read backwards, [4 Cout][H / 2][W / 2].
__device__ __forceinline__ int64_t shuffled_at(int o, int y, int x, int H, int W) {
    return ((int64_t)(o >> 2) * (2 * H) + 2 * y + (o >> 1 & 1)) * (2 * W) + 2 * x + (o & 1);
}
__device__ __forceinline__ int64_t unshuffled_at(int o, int y, int x, int H, int W) {
    return ((int64_t)(4 * o + 2 * (y & 1) + (x & 1)) * (H >> 1) + (y >> 1)) * (W >> 1) + (x >> 1);
}

// The convolution as an implicit GEMM on the matrix cores:
// out[o][p] = sum_k W[o][k] X[k][p] with k = 8 tap + input channel (within
// a chunk of 8 channels), sixteen output channels by sixteen pixels per
// v_mfma_f32_16x16x4f32 (FP32 in, FP32 accumulate).  A workgroup computes
// tiles of 64 columns by four rows for 16 output channels; wave w owns
// columns 16 w .. 16 w + 15, one accumulator a row.  Per chunk the input rows
// (with their halo) and the [k][o] weights are staged in LDS; each k-step
// gives every lane one weight (A: row o = lane % 16, k = lane / 16) and, per
// row, one input sample (B: k = lane / 16, pixel = lane % 16; the channel
// pitch, 16 mod 32, spreads two k over all 32 banks).  Split launches (splits
// > 1) sum input channels [s cps 8, (s + 1) cps 8) and write raw partial sums
// for k_conv_reduce.
//
// The grid is persistent: a workgroup walks a run of tiles, and the rows of
// the next step (the next chunk, or the next tile's first) are loaded while
// one is computed and stored to the other half of LDS behind it, one barrier
// a step.  KEPT: at most two chunks, whose weights stay in LDS for all tiles.
// Otherwise the weights are staged with their chunk, and a folded launch
// (fold) sums the splits itself in the order of k_conv_reduce: acc is the
// current split's sum, added to sum at its end (the same bits).
//
// What bounds it: the matrix cores take 50 us for 16 to 16 channels at 1600 x
// 1066 (7.9 GFLOP), the rest is the first and last steps of each run and a
// last round of tiles that is not full: 100 us (129 as a workgroup per 16 x
// 16 tile staged element by element); transposed with the mask, 327 MB: 119
// us (142).  Eight rows a tile: 110 and 144; five workgroups a CU: 103 and 139.
template <bool MASK, bool KEPT>
__global__ __launch_bounds__(kT, KEPT ? 4 : 3) void k_conv_mfma(ConvArgs a, int splits, int fold, int cps) {
    constexpr int KC = kCI * 9;                    // k values per chunk (72)
    constexpr int R = kCR, SR = R + 2, SC = kWave + 2;
    constexpr int P0 = SR * SC, P = P0 + (48 - P0 % 32) % 32;   // 16 mod 32
    static_assert(P % 32 == 16, "channel pitch");
    __shared__ float s_in[2][kCI * P];
    __shared__ float s_w[2][16 * KC];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    // blockIdx.y = split * (output-channel groups) + group; split s sums
    // input channels [s cps kCI, (s + 1) cps kCI), all of them if folded
    const int n_og = (a.Cout + 15) / 16;
    const int split = (int)blockIdx.y / n_og;
    const int og = ((int)blockIdx.y - split * n_og) * 16;
    const int cbeg = split * cps * kCI, cend = fold ? a.Cin : min(a.Cin, cbeg + cps * kCI);
    const int64_t HW = (int64_t)a.H * a.W;
    const int li = lane % 16, lk = lane / 16;
    const int tiles_x = (a.W + kWave - 1) / kWave, tiles_y = (a.H + R - 1) / R;
    int t, t_end, t_step;
    tile_run(tiles_x * tiles_y, &t, &t_end, &t_step);
    if (t >= t_end || cbeg >= cend) return;   // (uniform; a split without channels: launch_conv makes none)
    // D[o = 4 (lane / 16) + r][pixel = lane % 16] of row g: four output
    // channels, one 2 x 2 block of the shuffled map
    const int o4 = og + 4 * lk;
    float bias[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float bv = a.b ? a.b[o4 + r < a.Cout ? o4 + r : 0] : 0.f;
        bias[r] = o4 + r < a.Cout ? bv : 0.f;
    }
    Rows<kCI / 4, SR, MASK> rx;
    Edge<kCI, SR, MASK> ex;
    constexpr int JW = (16 * KC + kT - 1) / kT;
    float wv[JW];
    // weights as [k][o] with k = 8 tap + channel; chunk c0's lie wstep after
    // the chunk's before
    int wq[JW];
    const int wstep = a.transposed ? kCI * a.CinF * 9 : kCI * 9;
#pragma unroll
    for (int j = 0; j < JW; ++j) {
        const int e = (int)threadIdx.x + j * kT, k = e >> 4;
        wq[j] = (int)weight_at(a, min(og + (e & 15), a.Cout - 1), k & 7, min(k >> 3, 8));
    }
    auto load_w = [&](int c0) {
        const float* w = a.w + (int64_t)(c0 / kCI) * wstep;
#pragma unroll
        for (int j = 0; j < JW; ++j) {
            const int k = ((int)threadIdx.x + j * kT) >> 4;
            wv[j] = w[c0 + (k & 7) < cend ? wq[j] : wq[j] - (k & 7) * (wstep / kCI)];
        }
    };
    auto store_w = [&](int c0, float* dst) {
#pragma unroll
        for (int j = 0; j < JW; ++j) {
            const int e = (int)threadIdx.x + j * kT, k = e >> 4;
            if (e < 16 * KC) dst[e] = c0 + (k & 7) < cend && og + (e & 15) < a.Cout ? wv[j] : 0.f;
        }
    };
    int y0 = t / tiles_x * R, x0 = (t % tiles_x) * kWave, c0 = cbeg;
    bool plain = false;
    auto load = [&] {
        plain = inside(c0, kCI, cend, y0 - 1, SR, a.H, x0 - 1, SC, a.W);
        rx.load(a.in, a.mask, c0, cend, y0 - 1, x0 - 1, a.H, a.W, plain);
        ex.load(a.in, a.mask, c0, cend, y0 - 1, x0 + kWave - 1, a.H, a.W, plain);
        if (!KEPT) load_w(c0);
    };
    auto store = [&](int buf) {
        rx.store(s_in[buf], P, SC, c0, cend, y0 - 1, x0 - 1, a.H, a.W, plain);
        ex.store(s_in[buf], P, SC, kWave);
        if (!KEPT) store_w(c0, s_w[buf]);
    };
    load();
    if (KEPT) {
        load_w(cbeg);
        store_w(cbeg, s_w[0]);
        if (cbeg + kCI < cend) {
            load_w(cbeg + kCI);
            store_w(cbeg + kCI, s_w[1]);
        }
    }
    store(0);
    // acc: the current split's sum; sum: the splits before it
    mfma_f4 acc[R], sum[KEPT ? 1 : R];
#pragma unroll
    for (int g = 0; g < R; ++g) acc[g] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    if (!KEPT)
#pragma unroll
        for (int g = 0; g < R; ++g) sum[g] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    for (int buf = 0, step = 0;; buf ^= 1) {
        __syncthreads();   // this step is staged, and the one before computed
        const int cy = y0, cx = x0, cc = c0;   // this step; then the next
        c0 += kCI;
        const bool last = c0 >= cend;
        if (last) {
            c0 = cbeg;
            t += t_step;
            y0 = t / tiles_x * R;
            x0 = (t - t / tiles_x * tiles_x) * kWave;
        }
        const bool more = t < t_end;
        if (more) load();
        // k-step s = 2 tap + h takes k = 4 s + lane / 16: channels 4 h ..
        // 4 h + 3 of one tap, so every operand offset is a constant from
        // the lane's base; the upper channel half is skipped when the chunk
        // has at most four channels
        const float* aw = s_w[KEPT ? cc > cbeg : buf] + lane;
        const float* bb = s_in[buf] + lk * P + 16 * wave + li;
        auto taps = [&](auto halves) {
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
#pragma unroll
                for (int h = 0; h < decltype(halves)::value; ++h) {
                    const float av = aw[64 * (2 * tap + h)];
                    const float* src = bb + h * 4 * P + (tap / 3) * SC + tap % 3;
#pragma unroll
                    for (int g = 0; g < R; ++g)
                        acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, src[g * SC], acc[g], 0, 0, 0);
                }
            }
        };
        if (cend - cc > 4) taps(std::integral_constant<int, 2>());
        else taps(std::integral_constant<int, 1>());
        if (more) store(buf ^ 1);
        if (!KEPT && (++step == cps || last)) {
            step = 0;
#pragma unroll
            for (int g = 0; g < R; ++g)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sum[g][r] += acc[g][r];
                    acc[g][r] = 0.f;
                }
        }
        if (!last) continue;
        const int px = cx + 16 * wave + li;
        const bool parts = splits > 1 && !fold;
        float v[R][4];
#pragma unroll
        for (int g = 0; g < R; ++g) {
            mfma_f4& total = KEPT ? acc[g] : sum[KEPT ? 0 : g];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[g][r] = total[r];
                if (!parts) {
                    v[g][r] += bias[r];
                    v[g][r] = a.relu ? fmaxf(v[g][r], 0.f) : v[g][r];
                }
                total[r] = 0.f;
            }
        }
        float* dst = parts ? a.part + (int64_t)split * a.Cout * HW : a.unshuf ? nullptr : a.out;
        if (dst) {
            float* q = dst + (int64_t)o4 * HW + (int64_t)cy * a.W + px;
            if (og + 16 <= a.Cout && cy + R <= a.H && cx + kWave <= a.W) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
#pragma unroll
                    for (int g = 0; g < R; ++g) q[(int64_t)g * a.W] = v[g][r];
                    q += HW;
                }
            } else {
#pragma unroll
                for (int g = 0; g < R; ++g)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (o4 + r < a.Cout && cy + g < a.H && px < a.W) q[r * HW + (int64_t)g * a.W] = v[g][r];
            }
        }
        if (!parts && a.unshuf) {
#pragma unroll
            for (int g = 0; g < R; ++g)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (o4 + r < a.Cout && cy + g < a.H && px < a.W)
                        a.out[unshuffled_at(o4 + r, cy + g, px, a.H, a.W)] = v[g][r];
        }
        if (!parts && a.shuf && o4 < a.Cout && px < a.W) {   // Cout is a multiple of 4 there
#pragma unroll
            for (int g = 0; g < R; ++g)
                if (cy + g < a.H) {
                    float* q = a.shuf + shuffled_at(o4, cy + g, px, a.H, a.W);
                    *reinterpret_cast<float2*>(q) = make_float2(v[g][0], v[g][1]);
                    *reinterpret_cast<float2*>(q + 2 * a.W) = make_float2(v[g][2], v[g][3]);
                }
        }
        if (!more) return;
    }
}

// out[o][p] = (bias[o] + sum over the splits, in order, of part[s][o][p]),
// ReLU if asked: the end of a split convolution
__global__ __launch_bounds__(kT) void k_conv_reduce(ConvArgs a, int splits) {
    const int o = blockIdx.y;
    const int64_t p = (int64_t)blockIdx.x * kT + threadIdx.x, HW = (int64_t)a.H * a.W;
    if (p >= HW) return;
    float s = 0.f;
    for (int k = 0; k < splits; ++k) s += a.part[((int64_t)k * a.Cout + o) * HW + p];
    if (a.b) s += a.b[o];
    s = a.relu ? fmaxf(s, 0.f) : s;
    const int y = (int)(p / a.W), x = (int)(p - (int64_t)y * a.W);
    if (a.unshuf) a.out[unshuffled_at(o, y, x, a.H, a.W)] = s;
    else if (a.out) a.out[(int64_t)o * HW + p] = s;
    if (a.shuf) a.shuf[shuffled_at(o, y, x, a.H, a.W)] = s;
}

// Staged rows and channels.  A channel's pitch is 2 times an odd number mod
// 32, so that sixteen channels by two consecutive pixels (half a matrix
// operand) hit 32 different banks.
constexpr int kHR = kWR + 2, kHC = kWC + 2;   // with the one-pixel halo
constexpr int kGP = kWR * kWC + 2;            // 258 (2 mod 32)
constexpr int kXP = kHR * kHC + 2;            // 398 (14 mod 32)

// Per-workgroup partial sums of dW[o][i][tap] and db[o] over its pixel
// tiles, for a block of sixteen output by sixteen input channels, on the
// matrix cores: for each tap, dW[o][i] += sum over the pixels of g[o][p]
// x[i][p + tap], four pixels per v_mfma_f32_16x16x4f32 (FP32 operands and
// accumulation; A: o = lane % 16, B: i = lane % 16, pixel = lane / 16).  A
// wave takes a row of the tile and nine accumulators, one a tap; per four
// columns it reads one gradient and nine input operands for nine matrix
// instructions.  The waves' sums are added in order at the end.  The next
// tile's rows are loaded while a tile is computed (42 KB of LDS a tile, three
// workgroups a CU).  16 to 16 channels at 1600 x 1066: 109 us for 327 MB and
// 50 us of matrix-core time, 141 - 169 us as the vector form this replaced (a
// thread per (o, i) and a sliding 3 x 3 window in registers: 2.4 LDS reads
// for every nine multiply-adds, and chains of 1700 pixels).  Selecting zeros
// where the loads are issued instead of at the LDS store made every load wait
// for the one before: 134 us.
template <bool MASK>
__global__ __launch_bounds__(kT, 3) void k_wgrad(WgradArgs a) {
    __shared__ float s_g[16 * kGP];
    __shared__ float s_in[16 * kXP];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int li = lane % 16, lk = lane / 16;
    const int n_ig = (a.Cin + 15) / 16;
    const int o0 = ((int)blockIdx.y / n_ig) * 16, i0 = ((int)blockIdx.y % n_ig) * 16;
    const int tiles_x = (a.W + kWC - 1) / kWC, tiles_y = (a.H + kWR - 1) / kWR;
    mfma_f4 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = mfma_f4{0.f, 0.f, 0.f, 0.f};
    float bacc = 0.f;
    int t_beg, t_end, t_step;
    tile_run(tiles_x * tiles_y, &t_beg, &t_end, &t_step);
    Rows<4, kWR, MASK> rg;
    Rows<4, kHR, false> rx;
    Edge<16, kHR, false> ex;
    bool plain = false, plain_g = false;   // of the loaded tile
    auto load = [&](int tile) {
        const int y0 = (tile / tiles_x) * kWR, x0 = (tile % tiles_x) * kWC;
        plain = inside(i0, 16, a.Cin, y0 - 1, kHR, a.H, x0 - 1, kHC, a.W);
        plain_g = plain && o0 + 16 <= a.Cout;
        rg.load(a.g, a.mask, o0, a.Cout, y0, x0, a.H, a.W, plain_g);
        rx.load(a.in, nullptr, i0, a.Cin, y0 - 1, x0 - 1, a.H, a.W, plain);
        ex.load(a.in, nullptr, i0, a.Cin, y0 - 1, x0 + kWave - 1, a.H, a.W, plain);
    };
    if (t_beg < t_end) load(t_beg);
    for (int tile = t_beg; tile < t_end; tile += t_step) {
        const int y0 = (tile / tiles_x) * kWR, x0 = (tile % tiles_x) * kWC;
        __syncthreads();
        rg.store(s_g, kGP, kWC, o0, a.Cout, y0, x0, a.H, a.W, plain_g);
        rx.store(s_in, kXP, kHC, i0, a.Cin, y0 - 1, x0 - 1, a.H, a.W, plain);
        ex.store(s_in, kXP, kHC, kWave);
        __syncthreads();
        if (tile + t_step < t_end) load(tile + t_step);
        const float* pg = s_g + li * kGP + wave * kWC + lk;
        const float* px = s_in + li * kXP + wave * kHC + lk;
#pragma unroll 4
        for (int c = 0; c < kWC; c += 4) {
            const float g = pg[c];
            float x[3][3];
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int t = 0; t < 3; ++t) x[r][t] = px[r * kHC + c + t];
            bacc += g;
#pragma unroll
            for (int t = 0; t < 9; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(g, x[t / 3][t % 3], acc[t], 0, 0, 0);
        }
    }
    // D[o = 4 (lane / 16) + r][i = lane % 16]: the waves' sums in order,
    // through LDS a tap at a time
    bacc += __shfl_xor(bacc, 16, kWave);
    bacc += __shfl_xor(bacc, 32, kWave);
    float* red = s_in;   // [4 waves][256], then [4][16] for the bias
    float* part = a.partial + (int64_t)blockIdx.x * a.J;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave * 256 + (4 * lk + r) * 16 + li] = acc[t][r];
        if (t == 0 && lk == 0) red[4 * 256 + wave * 16 + li] = bacc;
        __syncthreads();
        const int o = (int)threadIdx.x / 16, i = (int)threadIdx.x % 16;
        float s = red[threadIdx.x];
        for (int w = 1; w < 4; ++w) s += red[w * 256 + threadIdx.x];
        if (o0 + o < a.Cout && i0 + i < a.Cin) part[((int64_t)(o0 + o) * a.Cin + i0 + i) * 9 + t] = s;
        if (t == 0 && i0 == 0 && threadIdx.x < 16 && o0 + (int)threadIdx.x < a.Cout) {
            float d = red[4 * 256 + threadIdx.x];
            for (int w = 1; w < 4; ++w) d += red[4 * 256 + w * 16 + threadIdx.x];
            part[(int64_t)a.Cout * a.Cin * 9 + o0 + threadIdx.x] = d;
        }
    }
}

// The same for layers of at most four output channels (27 or 36 rows (o,
// tap) by sixteen input channels): x is the A operand (input channel = lane %
// 16), and the sixteen columns of each of the three B operands are (o, tap)
// pairs, g[o][p - tap] read from a gradient tile with its own halo, so that
// the matrix tile is filled by taps instead of padded with absent output
// channels.  16 to 3 channels at 1600 x 1066: 47 us (the vector form: 71).
template <bool MASK>
__global__ __launch_bounds__(kT, 4) void k_wgrad_few(WgradArgs a) {
    constexpr int NB = 3;   // 48 columns >= 4 x 9
    __shared__ float s_g[4 * kXP];    // gradient tile with halo
    __shared__ float s_in[16 * kGP];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int li = lane % 16, lk = lane / 16;
    const int i0 = (int)blockIdx.y * 16;
    const int tiles_x = (a.W + kWC - 1) / kWC, tiles_y = (a.H + kWR - 1) / kWR;
    mfma_f4 acc[NB];
    int off[NB];
    bool used[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        acc[b] = mfma_f4{0.f, 0.f, 0.f, 0.f};
        const int n = 16 * b + li, o = n / 9, t = n % 9;
        used[b] = o < a.Cout;
        // x[p] meets the gradient of the pixels it reached: dW[o][i][t] =
        // sum over p of g[o][p] x[i][p + tap t], with q = p + tap: g[o][q - tap]
        off[b] = used[b] ? o * kXP + (2 - t / 3) * kHC + (2 - t % 3) : 0;
    }
    float bacc = 0.f;
    int t_beg, t_end, t_step;
    tile_run(tiles_x * tiles_y, &t_beg, &t_end, &t_step);
    Rows<1, kHR, MASK> rg;
    Edge<4, kHR, MASK> eg;
    Rows<4, kWR, false> rx;
    bool plain = false, plain_g = false;   // of the loaded tile
    auto load = [&](int tile) {
        const int y0 = (tile / tiles_x) * kWR, x0 = (tile % tiles_x) * kWC;
        plain = inside(i0, 16, a.Cin, y0 - 1, kHR, a.H, x0 - 1, kHC, a.W);
        plain_g = plain && a.Cout == 4;
        rg.load(a.g, a.mask, 0, a.Cout, y0 - 1, x0 - 1, a.H, a.W, plain_g);
        eg.load(a.g, a.mask, 0, a.Cout, y0 - 1, x0 + kWave - 1, a.H, a.W, plain_g);
        rx.load(a.in, nullptr, i0, a.Cin, y0, x0, a.H, a.W, plain);
    };
    if (t_beg < t_end) load(t_beg);
    for (int tile = t_beg; tile < t_end; tile += t_step) {
        const int y0 = (tile / tiles_x) * kWR, x0 = (tile % tiles_x) * kWC;
        __syncthreads();
        rg.store(s_g, kXP, kHC, 0, a.Cout, y0 - 1, x0 - 1, a.H, a.W, plain_g);
        eg.store(s_g, kXP, kHC, kWave);
        rx.store(s_in, kGP, kWC, i0, a.Cin, y0, x0, a.H, a.W, plain);
        __syncthreads();
        if (tile + t_step < t_end) load(tile + t_step);
        const float* px = s_in + li * kGP + wave * kWC + lk;
        const float* pg = s_g + wave * kHC + lk;
#pragma unroll 4
        for (int c = 0; c < kWC; c += 4) {
            const float x = px[c];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float g = used[b] ? pg[off[b] + c] : 0.f;
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, g, acc[b], 0, 0, 0);
            }
        }
        // the bias: output channel `wave`, a column a lane
#pragma unroll
        for (int r = 0; r < kWR; ++r) bacc += s_g[wave * kXP + (r + 1) * kHC + lane + 1];
    }
    // D[i = 4 (lane / 16) + r][(o, tap) = 16 b + lane % 16]
    for (int d = 32; d > 0; d >>= 1) bacc += __shfl_xor(bacc, d, kWave);
    float* red = s_in;
    float* part = a.partial + (int64_t)blockIdx.x * a.J;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(wave * NB + b) * 256 + (4 * lk + r) * 16 + li] = acc[b][r];
    __syncthreads();
    for (int e = threadIdx.x; e < NB * 256; e += kT) {
        const int b = e / 256, i = (e / 16) % 16, n = 16 * b + e % 16, o = n / 9, t = n % 9;
        float s = red[e];
        for (int w = 1; w < 4; ++w) s += red[w * NB * 256 + e];
        if (o < a.Cout && i0 + i < a.Cin) part[((int64_t)o * a.Cin + i0 + i) * 9 + t] = s;
    }
    if (i0 == 0 && lane == 0 && wave < a.Cout) part[(int64_t)a.Cout * a.Cin * 9 + wave] = bacc;
}

// out[j] = sum over the parts of partial[part][j]: 1024 / COLS threads a
// column add every (1024 / COLS)th part in order, then their sums are added
// as a fixed tree
template <int COLS>
__global__ __launch_bounds__(1024) void k_reduce_parts(const float* __restrict__ partial, int parts, int64_t J,
                                                       float* __restrict__ out) {
    constexpr int T = 1024 / COLS;
    __shared__ float red[T][COLS + 1];
    const int jj = threadIdx.x % COLS, pp = threadIdx.x / COLS;
    const int64_t j = (int64_t)blockIdx.x * COLS + jj;
    float s = 0.f;
    if (j < J)
#pragma unroll 4
        for (int p = pp; p < parts; p += T) s += partial[(int64_t)p * J + j];
    red[pp][jj] = s;
    __syncthreads();
    for (int n = T / 2; n > 0; n >>= 1) {
        if (pp < n) red[pp][jj] += red[pp + n][jj];
        __syncthreads();
    }
    if (pp == 0 && j < J) out[j] = red[0][jj];
}

// per-axis interpolation tables (half-pixel centres), FP64 coordinates
__global__ void k_bilin_table(int n_in, int n_out, int* __restrict__ i0, int* __restrict__ i1, float* __restrict__ f) {
    const int d = blockIdx.x * kT + threadIdx.x;
    if (d >= n_out) return;
    double s = ((double)d + 0.5) * (double)n_in / (double)n_out - 0.5;
    if (s < 0.0) s = 0.0;
    int a = (int)floor(s);
    if (a > n_in - 1) a = n_in - 1;
    i0[d] = a;
    i1[d] = min(a + 1, n_in - 1);
    f[d] = (float)(s - (double)a);
}

constexpr int kRows = 8;   // rows per workgroup of the interpolation kernels

// kRows output rows (channel c, row Y) per workgroup, one column per
// thread: the column's taps are read once, the rows' loads are independent
__global__ __launch_bounds__(kT) void k_bilinear(const float* __restrict__ in, int C, int h, int w, int H, int W,
                                                 const int* __restrict__ y0, const int* __restrict__ y1,
                                                 const float* __restrict__ fy, const int* __restrict__ x0,
                                                 const int* __restrict__ x1, const float* __restrict__ fx,
                                                 float* __restrict__ out) {
    int bx, by;
    xcd_tile(&bx, &by);
    const int X = bx * kT + (int)threadIdx.x;
    if (X >= W) return;
    const int ex0 = x0[X], ex1 = x1[X];
    const float e = fx[X];
    const int rows = C * H;
    for (int r0 = by * kRows; r0 < rows; r0 += (int)gridDim.y * kRows) {
        // all loads of the kRows rows first (rows past the end repeat the
        // last one and are not stored), then the blends
        float v[kRows][4], a[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int row = min(r0 + k, rows - 1);
            const int c = row / H, Y = row - c * H;
            const float* b = in + (int64_t)c * h * w;
            const float* p0 = b + (int64_t)y0[Y] * w;
            const float* p1 = b + (int64_t)y1[Y] * w;
            a[k] = fy[Y];
            v[k][0] = p0[ex0];
            v[k][1] = p0[ex1];
            v[k][2] = p1[ex0];
            v[k][3] = p1[ex1];
        }
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            if (r0 + k >= rows) break;
            const float top = (1.f - e) * v[k][0] + e * v[k][1];
            const float bot = (1.f - e) * v[k][2] + e * v[k][3];
            out[(int64_t)(r0 + k) * W + X] = (1.f - a[k]) * top + a[k] * bot;
        }
    }
}

// Row kernels of the interpolation for images up to kRowW = 2048 wide (the
// source rows then hold at most 1024 values): a workgroup handles a
// contiguous run of rows, staging each row's sources in LDS with coalesced
// loads (every load of the thread issued before its LDS writes), and each
// thread keeps the taps of its output columns in registers for all rows.
constexpr int kRowW = 2048;
constexpr int kRowCols = kRowW / kT;   // output columns per thread (forward)
constexpr int kRowSrc = kRowW / 2 / kT;   // source values per thread and row (forward)

__global__ __launch_bounds__(kT) void k_bilinear_rows(const float* __restrict__ in, int C, int h, int w, int H,
                                                      int W, const int* __restrict__ y0, const int* __restrict__ y1,
                                                      const float* __restrict__ fy, const int* __restrict__ x0,
                                                      const int* __restrict__ x1, const float* __restrict__ fx,
                                                      float* __restrict__ out) {
    extern __shared__ float s_src[];   // the two source rows, 2 w floats
    const int tid = (int)threadIdx.x;
    int ex0[kRowCols], ex1[kRowCols];
    float e[kRowCols];
#pragma unroll
    for (int m = 0; m < kRowCols; ++m) {
        const int X = tid + m * kT;
        const bool ok = X < W;
        ex0[m] = ok ? x0[X] : 0;
        ex1[m] = ok ? x1[X] : 0;
        e[m] = ok ? fx[X] : 0.f;
    }
    const int rows = C * H;
    const int chunk = (rows + (int)gridDim.x - 1) / (int)gridDim.x;
    const int r_beg = (int)blockIdx.x * chunk, r_end = min(rows, r_beg + chunk);
    // a row's source values are loaded while the previous row is blended
    float v0[kRowSrc], v1[kRowSrc], an = 0.f;
    auto load = [&](int row) {
        const int c = row / H, Y = row - c * H;
        const float* p0 = in + ((int64_t)c * h + y0[Y]) * w;
        const float* p1 = in + ((int64_t)c * h + y1[Y]) * w;
        an = fy[Y];
#pragma unroll
        for (int j = 0; j < kRowSrc; ++j) {
            const int k = tid + j * kT;
            v0[j] = p0[k < w ? k : 0];
            v1[j] = p1[k < w ? k : 0];
        }
    };
    if (r_beg < r_end) load(r_beg);
    for (int row = r_beg; row < r_end; ++row) {
        const float a = an;
        __syncthreads();   // the previous row's blends are done with s_src
#pragma unroll
        for (int j = 0; j < kRowSrc; ++j) {
            const int k = tid + j * kT;
            if (k < w) {
                s_src[k] = v0[j];
                s_src[w + k] = v1[j];
            }
        }
        __syncthreads();
        if (row + 1 < r_end) load(row + 1);
#pragma unroll
        for (int m = 0; m < kRowCols; ++m) {
            const int X = tid + m * kT;
            if (X < W) {
                const float top = (1.f - e[m]) * s_src[ex0[m]] + e[m] * s_src[ex1[m]];
                const float bot = (1.f - e[m]) * s_src[w + ex0[m]] + e[m] * s_src[w + ex1[m]];
                out[(int64_t)row * W + X] = (1.f - a) * top + a * bot;
            }
        }
    }
}

// Outputs d reading input i along one axis are those with i0[d] <= i <=
// i1[d] (i1 is i0 or i0 + 1, both nondecreasing in d): a contiguous range,
// found by a short scan from its estimate.
__device__ __forceinline__ void axis_range(int i, int n_in, int n_out, const int* i0, const int* i1, int* lo, int* hi) {
    const float sc = (float)n_out / (float)n_in;
    int d = (int)floorf(((float)i - 0.5f) * sc - 0.5f) - 2;
    d = max(0, min(d, n_out));
    while (d > 0 && i1[d - 1] >= i) --d;
    while (d < n_out && i1[d] < i) ++d;
    int e = d;
    while (e < n_out && i0[e] <= i) ++e;
    *lo = d;
    *hi = e;
}

// per input index, the [lo, hi) range of outputs that read it
__global__ void k_bilin_ranges(int n_in, int n_out, const int* __restrict__ i0, const int* __restrict__ i1,
                               int* __restrict__ lo, int* __restrict__ hi) {
    const int i = blockIdx.x * kT + threadIdx.x;
    if (i >= n_in) return;
    int a, b;
    axis_range(i, n_in, n_out, i0, i1, &a, &b);
    lo[i] = a;
    hi[i] = b;
}

// Adjoint of k_bilinear along x: tmp[c][Y][i] = sum over the outputs X
// that read input column i of their weight times g[c][Y][X] (one row per
// grid row, one input column per thread)
__device__ __forceinline__ float adj_weight(int d, int i, const int* i0, const int* i1, const float* f) {
    return (i0[d] == i ? 1.f - f[d] : 0.f) + (i1[d] == i ? f[d] : 0.f);
}

__global__ __launch_bounds__(kT) void k_bilin_adj_x(const float* __restrict__ g, int rows, int W, int w,
                                                    const int* __restrict__ i0, const int* __restrict__ i1,
                                                    const float* __restrict__ f, const int* __restrict__ rlo,
                                                    const int* __restrict__ rhi, float* __restrict__ out) {
    int bx, by;
    xcd_tile(&bx, &by);
    const int i = bx * kT + (int)threadIdx.x;
    if (i >= w) return;
    const int lo = rlo[i], hi = rhi[i];
    // upsampling by at most 2 (the only use): at most four outputs read an
    // input, five at the clamped last one; their taps are loaded once,
    // padded to six with weight-0 taps (which leave the sum unchanged);
    // longer ranges take the plain loop
    constexpr int K = 6;
    const bool fits = hi - lo <= K;
    int dk[K];
    float wk[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool on = lo + k < hi;
        dk[k] = on ? lo + k : 0;
        wk[k] = on ? adj_weight(lo + k, i, i0, i1, f) : 0.f;
    }
    for (int r0 = by * kRows; r0 < rows; r0 += (int)gridDim.y * kRows) {
        if (fits) {
            float v[kRows][K];
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const float* gl = g + (int64_t)min(r0 + k, rows - 1) * W;
#pragma unroll
                for (int t = 0; t < K; ++t) v[k][t] = gl[dk[t]];
            }
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                if (r0 + k >= rows) break;
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < K; ++t) s = fmaf(wk[t], v[k][t], s);
                out[(int64_t)(r0 + k) * w + i] = s;
            }
        } else {
            for (int k = 0; k < kRows && r0 + k < rows; ++k) {
                const float* gl = g + (int64_t)(r0 + k) * W;
                float s = 0.f;
                for (int d = lo; d < hi; ++d) s = fmaf(adj_weight(d, i, i0, i1, f), gl[d], s);
                out[(int64_t)(r0 + k) * w + i] = s;
            }
        }
    }
}

// Both passes of the adjoint as one, for images up to kRowW wide whose height
// is not below the map's: a workgroup marches down the image rows that reach
// its band of output rows of one channel, forms the x pass's sums of a row in
// registers and adds them, with the row's two y weights, to the sums of the
// two output rows it reaches (rows ascending, as the two passes add: the same
// bits).  The intermediate map, as large as the output in x and as the image
// in y, is never stored.  A row is loaded while the one before is summed and
// staged in the other half of LDS, one barrier a row.  Thread columns i = tid
// + m kT (i < w <= kRowW / 2) keep their x taps in registers (at most four
// when upsampling by at most 2, five at the clamped last input; padded to six
// with weight-0 taps; a longer range falls back to the plain loop over the
// staged row).  16 channels at 1600 x
// 1066 to 800 x 544: 51 us for 136 MB, 103 as two passes (61 and 42).
// Bands of 12 output rows there; 8, 16 and 32: 71, 62 and 97 us.
__global__ __launch_bounds__(kT) void k_bilin_adj_rows(const float* __restrict__ g, int H, int W, int h, int w,
                                                       BilinTab t, int band, float* __restrict__ out) {
    extern __shared__ float s_row[];   // 2 W floats
    constexpr int M = kRowW / 2 / kT, K = 6, J = kRowW / kT;
    const int tid = (int)threadIdx.x;
    int dk[M][K], lo[M], hi[M];
    float wk[M][K];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int i = tid + m * kT;
        lo[m] = i < w ? t.xlo[i] : 0;
        hi[m] = i < w ? t.xhi[i] : 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool on = lo[m] + k < hi[m];
            dk[m][k] = on ? lo[m] + k : 0;
            wk[m][k] = on ? adj_weight(lo[m] + k, i, t.x0, t.x1, t.fx) : 0.f;
        }
    }
    const int a = (int)blockIdx.x * band, b = min(h, a + band);
    const int d_end = t.yhi[b - 1];
    int d = t.ylo[a];
    const float* gc = g + (int64_t)blockIdx.y * H * W;
    float* oc = out + (int64_t)blockIdx.y * h * w;
    float v[J];
    auto load = [&](int row) {
        const float* gl = gc + (int64_t)row * W;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k = tid + j * kT;
            v[j] = gl[k < W ? k : 0];
        }
    };
    int cur = t.y0[d];   // the output row of acc0 (acc1: the next), up to one above the band at first
    float acc0[M], acc1[M];
#pragma unroll
    for (int m = 0; m < M; ++m) acc0[m] = acc1[m] = 0.f;
    auto write = [&] {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int i = tid + m * kT;
            if (i < w && cur >= a && cur < b) oc[(int64_t)cur * w + i] = acc0[m];
            acc0[m] = acc1[m];
            acc1[m] = 0.f;
        }
        ++cur;
    };
    load(d);
    for (int buf = 0; d < d_end; ++d, buf ^= 1) {
        float* row = s_row + buf * W;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k = tid + j * kT;
            if (k < W) row[k] = v[j];
        }
        __syncthreads();
        if (d + 1 < d_end) load(d + 1);
        const int y0 = t.y0[d], y1 = t.y1[d];
        const float w0 = adj_weight(d, y0, t.y0, t.y1, t.fy), w1 = y1 > y0 ? adj_weight(d, y1, t.y0, t.y1, t.fy) : 0.f;
        while (cur < y0) write();
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int i = tid + m * kT;
            if (i < w) {
                float s = 0.f;
                if (hi[m] - lo[m] <= K) {
#pragma unroll
                    for (int k = 0; k < K; ++k) s = fmaf(wk[m][k], row[dk[m][k]], s);
                } else {
                    for (int x = lo[m]; x < hi[m]; ++x) s = fmaf(adj_weight(x, i, t.x0, t.x1, t.fx), row[x], s);
                }
                acc0[m] = fmaf(w0, s, acc0[m]);
                if (y1 > y0) acc1[m] = fmaf(w1, s, acc1[m]);
            }
        }
    }
    while (cur < b) write();
}

// ... and along y: out[c][i][x] = sum over the output rows Y that read
// input row i of their weight times tmp[c][Y][x] (one (c, i) per grid row,
// one column per thread)
__global__ __launch_bounds__(kT) void k_bilin_adj_y(const float* __restrict__ tmp, int C, int H, int h, int w,
                                                    const int* __restrict__ i0, const int* __restrict__ i1,
                                                    const float* __restrict__ f, const int* __restrict__ rlo,
                                                    const int* __restrict__ rhi, float* __restrict__ out) {
    int bx, by;
    xcd_tile(&bx, &by);
    const int x = bx * kT + (int)threadIdx.x;
    if (x >= w) return;
    const int rows = C * h;
    constexpr int K = 6;   // as in the x pass: at most five taps when upsampling by at most 2
    for (int r0 = by * kRows; r0 < rows; r0 += (int)gridDim.y * kRows) {
        float v[kRows][K], wt[kRows][K];
        bool fits = true;
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int row = min(r0 + k, rows - 1);
            const int c = row / h, i = row - c * h;
            const int lo = rlo[i], hi = rhi[i];
            fits = fits && hi - lo <= K;
            const float* tc = tmp + (int64_t)c * H * w + x;
#pragma unroll
            for (int t = 0; t < K; ++t) {
                const bool on = lo + t < hi;
                const int d = on ? lo + t : 0;
                wt[k][t] = on ? adj_weight(d, i, i0, i1, f) : 0.f;
                v[k][t] = tc[(int64_t)d * w];
            }
        }
        if (fits) {
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                if (r0 + k >= rows) break;
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < K; ++t) s = fmaf(wt[k][t], v[k][t], s);
                out[(int64_t)(r0 + k) * w + x] = s;
            }
        } else {
            for (int k = 0; k < kRows && r0 + k < rows; ++k) {
                const int row = r0 + k;
                const int c = row / h, i = row - c * h;
                const int lo = rlo[i], hi = rhi[i];
                const float* tc = tmp + (int64_t)c * H * w + x;
                float s = 0.f;
                for (int d = lo; d < hi; ++d) s = fmaf(adj_weight(d, i, i0, i1, f), tc[(int64_t)d * w], s);
                out[(int64_t)row * w + x] = s;
            }
        }
    }
}

// dM = dIa * Ir; dIr += dIa * M
__global__ __launch_bounds__(kT) void k_mul_bwd(const float* __restrict__ d_adj, const float* __restrict__ img,
                                                const float* __restrict__ M, int64_t n, float* __restrict__ dM,
                                                float* __restrict__ d_img) {
    const int64_t q = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (q >= n) return;
    const float g = d_adj[q];
    dM[q] = g * img[q];
    d_img[q] += g * M[q];
}

// d_embed[k] = sum over the pixels of channel 3 + k of dD
__global__ __launch_bounds__(kT) void k_embed_grad(const float* __restrict__ dD, int64_t hw, float* __restrict__ d_embed) {
    __shared__ float red[kT / kWave];
    const float* src = dD + (int64_t)(3 + blockIdx.x) * hw;
    float s = 0.f;
    for (int64_t p = threadIdx.x; p < hw; p += kT) s += src[p];
    for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int k = 0; k < kT / kWave; ++k) t += red[k];
        d_embed[blockIdx.x] = t;
    }
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

}  // namespace

void launch_down_concat(const float* img, int H, int W, int h, int w, const float* embed, int m, float* D,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_down_concat, dim3(h * w), dim3(kT), 0, st, img, H, W, h, w, embed, m, D);
}

void launch_down_adjoint(const float* g, int H, int W, int h, int w, float* d_img, hipStream_t st) {
    hipLaunchKernelGGL(k_down_adjoint, dim3(blocks_for(3 * (int64_t)H * W)), dim3(kT), 0, st, g, H, W, h, w, d_img);
}

int conv_splits(int Cin, int Cout, int H, int W) {
    if (Cout <= 4) return 1;   // k_conv_few takes all channels
    // the low-resolution layers give too few workgroups to fill 256 CUs:
    // split their input channels until the grid has about 2048
    const int64_t wgs = (int64_t)((W + kTile - 1) / kTile) * ((H + kTile - 1) / kTile) * ((Cout + 15) / 16);
    const int chunks = (Cin + kCI - 1) / kCI;
    if (wgs >= 1024 || chunks < 2) return 1;
    const int want = (int)std::min<int64_t>(chunks, (2048 + wgs - 1) / wgs);
    const int cps = (chunks + want - 1) / want;
    return (chunks + cps - 1) / cps;
}

// workgroups that share n tiles in equal runs, as many as fit at once
// (per_cu a CU, over `groups` channel groups)
unsigned runs(int64_t n, int per_cu, int64_t groups) {
    const int64_t fit = 256 * per_cu;
    const int64_t each = (n * groups + fit - 1) / fit;
    const int64_t wgs = (n + each - 1) / each;
    return (unsigned)(wgs < 64 ? wgs : (wgs + kXcds - 1) / kXcds * kXcds);   // a multiple of the XCDs: tile_run's bands
}

void launch_conv(const ConvArgs& a, hipStream_t st) {
    const int64_t tx = (a.W + kWave - 1) / kWave;
    if (a.Cout > 4) {
        const int splits = a.part ? conv_splits(a.Cin, a.Cout, a.H, a.W) : 1;
        const int chunks = (a.Cin + kCI - 1) / kCI;
        const int cps = (chunks + splits - 1) / splits;
        const int64_t tiles = tx * ((a.H + kCR - 1) / kCR), groups = (a.Cout + 15) / 16;
        // Splits cost a pass over their partial sums (9 - 15 us), folding
        // them a chain of steps in too few workgroups.  Measured (64 x 4
        // tiles x groups of 16 channels, folded against split): 272: 36.7
        // against 33.5 us and 38.9 against 34.7; 476: 23.6 against 34.3; 544:
        // 28.2 against 34.0; 952: 23.8 against 38.0.  The line lies between.
        const int fold = splits > 1 && tiles * groups >= 400;
        const unsigned gy = (unsigned)(fold ? groups : groups * splits);
        const bool kept = !fold && cps <= 2;
        const dim3 grid(runs(tiles, kept ? 4 : 3, gy), gy);
        if (a.mask && kept) hipLaunchKernelGGL((k_conv_mfma<true, true>), grid, dim3(kT), 0, st, a, splits, fold, cps);
        else if (a.mask) hipLaunchKernelGGL((k_conv_mfma<true, false>), grid, dim3(kT), 0, st, a, splits, fold, cps);
        else if (kept) hipLaunchKernelGGL((k_conv_mfma<false, true>), grid, dim3(kT), 0, st, a, splits, fold, cps);
        else hipLaunchKernelGGL((k_conv_mfma<false, false>), grid, dim3(kT), 0, st, a, splits, fold, cps);
        if (splits > 1 && !fold)
            hipLaunchKernelGGL(k_conv_reduce, dim3(blocks_for((int64_t)a.H * a.W), a.Cout), dim3(kT), 0, st, a,
                               splits);
        return;
    }
    const dim3 grid(runs(tx * ((a.H + 15) / 16), kFewWgs, 1));
    if (a.mask) hipLaunchKernelGGL(k_conv_few<true>, grid, dim3(kT), 0, st, a);
    else hipLaunchKernelGGL(k_conv_few<false>, grid, dim3(kT), 0, st, a);
}

// workgroups a channel block: as many as fit on the device at once (three a
// CU), so that a full-resolution layer takes one round of equal runs of tiles
constexpr int kWgradParts = 768;

int wgrad_parts(int H, int W) {
    const int tiles = ((W + kWC - 1) / kWC) * ((H + kWR - 1) / kWR);
    return tiles < kWgradParts ? tiles : kWgradParts;
}

void launch_wgrad(const WgradArgs& a, float* dw, hipStream_t st) {
    const int parts = wgrad_parts(a.H, a.W);
    const bool m = a.mask != nullptr;
    if (a.Cout <= 4) {
        const dim3 grid(parts, (a.Cin + 15) / 16);
        if (m) hipLaunchKernelGGL(k_wgrad_few<true>, grid, dim3(kT), 0, st, a);
        else hipLaunchKernelGGL(k_wgrad_few<false>, grid, dim3(kT), 0, st, a);
    } else {
        const dim3 grid(parts, ((a.Cout + 15) / 16) * ((a.Cin + 15) / 16));
        if (m) hipLaunchKernelGGL(k_wgrad<true>, grid, dim3(kT), 0, st, a);
        else hipLaunchKernelGGL(k_wgrad<false>, grid, dim3(kT), 0, st, a);
    }
    // few columns of many parts (435 - 2320 by 768, the high-resolution
    // layers) leave 64-column workgroups few and their chains long (15 us
    // against 5); many columns of few parts (154368 by 9) leave 16-column
    // ones short of work (24 us against 6)
    if (parts > 128)
        hipLaunchKernelGGL(k_reduce_parts<16>, dim3((unsigned)((a.J + 15) / 16)), dim3(1024), 0, st, a.partial, parts,
                           a.J, dw);
    else
        hipLaunchKernelGGL(k_reduce_parts<64>, dim3((unsigned)((a.J + 63) / 64)), dim3(1024), 0, st, a.partial, parts,
                           a.J, dw);
}

void launch_bilin_table(int n_in, int n_out, int* i0, int* i1, float* f, hipStream_t st) {
    hipLaunchKernelGGL(k_bilin_table, dim3(blocks_for(n_out)), dim3(kT), 0, st, n_in, n_out, i0, i1, f);
}

// workgroup rows for kRows rows each (the kernels stride over the rest)
unsigned grid_rows(int64_t rows) { return (unsigned)std::min<int64_t>((rows + kRows - 1) / kRows, 65535); }

// workgroups of the row kernels: about eight per CU, each a run of rows
unsigned row_groups(int64_t rows) { return (unsigned)std::min<int64_t>(rows, 2048); }

void launch_bilinear(const float* in, int C, int h, int w, int H, int W, const BilinTab& t, float* out,
                     hipStream_t st) {
    if (W <= kRowW) {
        const int64_t rows = (int64_t)C * H;
        hipLaunchKernelGGL(k_bilinear_rows, dim3(row_groups(rows)), dim3(kT), 2 * w * sizeof(float), st, in, C, h, w,
                           H, W, t.y0, t.y1, t.fy, t.x0, t.x1, t.fx, out);
        return;
    }
    hipLaunchKernelGGL(k_bilinear, dim3(blocks_for(W), grid_rows((int64_t)C * H)), dim3(kT), 0, st, in, C, h, w, H,
                       W, t.y0, t.y1, t.fy, t.x0, t.x1, t.fx, out);
}

bool bilinear_adj_one_pass(int H, int W, int h) { return W <= kRowW && H >= h; }

void launch_bilinear_adj(const float* g, int C, int H, int W, int h, int w, const BilinTab& t, float* tmp,
                         float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_bilin_ranges, dim3(blocks_for(w)), dim3(kT), 0, st, w, W, t.x0, t.x1, t.xlo, t.xhi);
    hipLaunchKernelGGL(k_bilin_ranges, dim3(blocks_for(h)), dim3(kT), 0, st, h, H, t.y0, t.y1, t.ylo, t.yhi);
    if (bilinear_adj_one_pass(H, W, h)) {
        // bands that fill the chip's three workgroups a CU once, but of four
        // rows at least (each starts with the rows above its own)
        const int band = std::max(4, (int)(((int64_t)C * h + 767) / 768));
        hipLaunchKernelGGL(k_bilin_adj_rows, dim3((h + band - 1) / band, C), dim3(kT), 2 * W * sizeof(float), st, g, H,
                           W, h, w, t, band, out);
        return;
    }
    // x pass: [C][H][W] -> tmp [C][H][w]; lines = C H rows
    const int64_t rows = (int64_t)C * H;
    hipLaunchKernelGGL(k_bilin_adj_x, dim3(blocks_for(w), grid_rows(rows)), dim3(kT), 0, st, g, (int)rows, W, w,
                           t.x0, t.x1, t.fx, t.xlo, t.xhi, tmp);
    // y pass: tmp [C][H][w] -> out [C][h][w]
    hipLaunchKernelGGL(k_bilin_adj_y, dim3(blocks_for(w), grid_rows((int64_t)C * h)), dim3(kT), 0, st, tmp, C, H, h,
                       w, t.y0, t.y1, t.fy, t.ylo, t.yhi, out);
}

void launch_mul_bwd(const float* d_adj, const float* img, const float* M, int64_t n, float* dM, float* d_img,
                    hipStream_t st) {
    hipLaunchKernelGGL(k_mul_bwd, dim3(blocks_for(n)), dim3(kT), 0, st, d_adj, img, M, n, dM, d_img);
}

void launch_embed_grad(const float* dD, int64_t hw, int m, float* d_embed, hipStream_t st) {
    hipLaunchKernelGGL(k_embed_grad, dim3(m), dim3(kT), 0, st, dD, hw, d_embed);
}

}  // namespace gs
