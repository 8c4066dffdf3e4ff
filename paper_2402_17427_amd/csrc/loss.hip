// The training loss of one image and its gradient, fused in one pass.
//
// VastGaussian (arXiv 2402.17427) optimises each cell's Gaussians against
// its training images with the loss of Eq. 1 (section 3):
// (1 - lambda) L1(I^r, I) + lambda D-SSIM(I^r, I), and, with decoupled
// appearance modelling, Eq. 3 (section 4.2): the L1 term on the adjusted
// image I^a and the D-SSIM term on the rendered I^r.  D-SSIM comes from
// 3DGS: 1 - SSIM, SSIM averaged over every pixel and channel, with an
// 11 x 11 Gaussian window (sigma 1.5), C1 = 0.01^2, C2 = 0.03^2, and window
// sums that treat the outside of the image as zero.
//
// Per pixel p, with the window sums m = G*x, E = G*x^2, X = G*xy (x = I^r)
// and mu_y, E_y of the target, the SSIM map is S = a1 a2 / (b1 b2),
// a1 = 2 m mu_y + C1, a2 = 2 (X - m mu_y) + C2, b1 = m^2 + mu_y^2 + C1,
// b2 = (E - m^2) + (E_y - mu_y^2) + C2.  With g = dLoss/dS = -lambda / n,
//   dm = g 2 (mu_y (a2 - a1) - m S (b2 - b1)) / (b1 b2),
//   dE = -g S / b2,   dX = g 2 a1 / (b1 b2),
// and because the window is symmetric and zero padded, the gradient of the
// D-SSIM term at pixel q is (G*dm)(q) + 2 x(q) (G*dE)(q) + y(q) (G*dX)(q),
// the maps dm, dE, dX being zero outside the image.
//
// Two kernels compute the same gradient bits (the same sums in the same
// order); the loss value they add in their own order each, no lane more than
// a few pixels in FP32:
//
// k_loss_tile, for small images.  One workgroup computes one 32 x 32 output
// tile of one channel entirely in LDS: the input with a 10-pixel halo, the
// five forward window sums on the tile plus a 5-pixel halo (separable: a
// horizontal then a vertical 11-tap pass, three planes at a time so that
// three workgroups fit on a CU), the three SSIM partials there, their window
// sums on the tile (again two passes), and the L1 term.  Halo recompute
// replaces any intermediate HBM traffic.
//
// k_loss_strips, for the others, with the window sums on the matrix cores.
// v_mfma_f32_4x4x1_16b_f32 is sixteen 4 x 4 outer products (FP32 in and out,
// one fused multiply-add per result): with lane = image column, one
// instruction adds a row to four consecutive rows of vertical sums at 64
// columns, D[r][column] += g[t - r] v[t][column], the window weights in the
// other operand (zero outside the window), so four rows of 11-tap sums take
// 14 instructions of 8 cycles instead of 44 fused multiply-adds of 4.  With
// the operands exchanged it adds a column to four columns of horizontal
// sums, and its results come back one column per lane.  A workgroup owns a
// strip of 236 output columns (256 with the 10-column halo) and walks down a
// segment of its rows four at a time:
//   input rows -> LDS -> horizontal sums of x, y, xy, x^2, y^2 -> vertical
//   sums, pending in registers for the groups that are not complete yet ->
//   SSIM and its three partials -> LDS -> horizontal sums -> vertical sums,
//   pending likewise -> gradient.
// The image is read once (plus the halos, mostly from cache) and no
// intermediate touches HBM.  Halo recompute: 20 columns of 256, and 24 rows
// a segment.  A zero weight times an infinity or NaN would spread it beyond
// the window: a workgroup that meets a value whose square, or a partial
// that, reaches 1e37 starts its segment over with plain fused multiply-adds
// over the window's own taps.
//
// The loss value is reduced from per-workgroup partial sums by a last,
// one-workgroup kernel in double precision, in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>

#include "api_internal.h"
#include "kernels.h"

namespace gs {

namespace {

constexpr int kXcds = 8;          // XCDs of an MI355X (workgroups are dealt round-robin)
constexpr int kR = 5;             // window radius
constexpr int kTaps = 2 * kR + 1;

// ---- k_loss_tile
constexpr int kTileThreads = 256;
constexpr int kT = 32;            // output tile edge
constexpr int kAY = kT + 4 * kR;  // input rows (52)
constexpr int kAX = 56;           // input row stride; columns loaded: 54
constexpr int kALoad = 54;
constexpr int kBY = kT + 2 * kR;  // rows of the forward sums / partials (42)
constexpr int kBX = kT + 2 * kR;  // their columns (42)
constexpr int kHX = 44;           // row stride of the horizontal sums (4 groups of 11)
constexpr int kHGroup = 11;       // columns per thread in the forward horizontal pass
constexpr int kVGroup = 7;        // rows per thread in the forward vertical pass (42 = 6 x 7)
constexpr int kQGroup = 8;        // columns per thread in the backward horizontal pass
constexpr int kDGroup = 4;        // rows per thread in the backward vertical pass

constexpr int kSA = kAY * kAX;      // one input plane
constexpr int kSH = kAY * kHX;      // one horizontal-sum plane
constexpr int kSP = kBY * kHX;      // one partial plane
constexpr int kSQ = kBY * kT;       // one backward horizontal plane
constexpr int kRegX = 2 * kSA;      // inputs; later the backward horizontal sums
constexpr int kRegH = 3 * kSH;      // horizontal sums; later the partials
constexpr int kLdsFloats = kRegX + kRegH;  // 50.8 KB: three workgroups per CU
static_assert(3 * kSQ <= kRegX, "backward horizontal sums reuse the input planes");
static_assert(3 * kSP <= kRegH, "partials reuse the horizontal sums");

// ---- k_loss_strips
constexpr int kColWaves = 4;
constexpr int kCols = kColWaves * kWave;   // input columns of a strip
constexpr int kThreads = 2 * kCols;
constexpr int kOutW = kCols - 4 * kR;      // output columns of a strip (236)
constexpr int kG = 4;             // rows (and columns) of a group of sums
constexpr int kSteps = kTaps + kG - 1;        // inputs that reach a group (14)
constexpr int kPend = 3;          // groups of vertical sums pending at a time
// LDS row stride of the sums: 256 columns and the 13 beyond that the last
// lanes read; 8 mod 32 so that the 16-byte reads of four rows by two
// neighbouring blocks hit different banks
constexpr int kStride = 296;
constexpr float kBig = 1e37f;     // from it on a value takes the plain sums
constexpr int kResident = 512;    // workgroups that fit on the device at once (two per CU)

constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

struct Win {
    float g[kTaps];
};

struct LossArgs {
    int tiles_x, tiles_y;     // k_loss_tile
    const float* x;    // I^r  [C][H][W]
    const float* xa;   // I^a  [C][H][W] or NULL (then x)
    const float* y;    // I    [C][H][W]
    float* dx;         // [C][H][W]
    float* dxa;        // [C][H][W] or NULL
    float2* partial;   // per workgroup (sum S, sum |xa - y|)
    int W, H;
    int strips, segs, rows;   // k_loss_strips: strips of kOutW columns, segments of `rows` rows (a multiple of kG)
    float gs;          // dLoss/dS = -lambda / n
    float g1;          // (1 - lambda) / n
    Win win;
};

typedef float f4 __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Horizontal 11-tap sums of NM products of the input rows: thread
// (row r, group j) writes columns 11j .. 11j+10 of row r of each plane.
template <int NM, typename F>
__device__ __forceinline__ void hpass(const Win& win, const float* sx, const float* sy, float* sh, int tid, F prod) {
    if (tid >= kAY * 4) return;
    const int r = tid >> 2, c0 = (tid & 3) * kHGroup;
    float vx[kHGroup + 2 * kR], vy[kHGroup + 2 * kR];
#pragma unroll
    for (int t = 0; t < kHGroup + 2 * kR; ++t) {
        vx[t] = sx[r * kAX + c0 + t];
        vy[t] = sy[r * kAX + c0 + t];
    }
    float pr[NM][kHGroup + 2 * kR];
#pragma unroll
    for (int t = 0; t < kHGroup + 2 * kR; ++t) prod(vx[t], vy[t], pr, t);
#pragma unroll
    for (int o = 0; o < kHGroup; ++o) {
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            float s = 0.f;
#pragma unroll
            for (int t = 0; t < kTaps; ++t) s = fmaf(win.g[t], pr[m][o + t], s);
            sh[m * kSH + r * kHX + c0 + o] = s;
        }
    }
}

// Vertical 11-tap sums of NM horizontal-sum planes: thread (column vc,
// group) produces rows vr0 .. vr0+6 of the tile-plus-halo region.
template <int NM>
__device__ __forceinline__ void vpass(const Win& win, const float* sh, int vc, int vr0, float (&acc)[NM][kVGroup]) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        float col[kVGroup + 2 * kR];
#pragma unroll
        for (int t = 0; t < kVGroup + 2 * kR; ++t) col[t] = sh[m * kSH + (vr0 + t) * kHX + vc];
#pragma unroll
        for (int o = 0; o < kVGroup; ++o) {
            float s = 0.f;
#pragma unroll
            for (int t = 0; t < kTaps; ++t) s = fmaf(win.g[t], col[o + t], s);
            acc[m][o] = s;
        }
    }
}

__global__ __launch_bounds__(kTileThreads, 3) void k_loss_tile(LossArgs a) {
    __shared__ float lds[kLdsFloats];
    float* sx = lds;
    float* sy = lds + kSA;
    float* sq = lds;          // 3 planes [kBY][kT], after the inputs are consumed
    float* sh = lds + kRegX;  // 3 planes [kAY][kHX]
    float* sp = sh;           // 3 planes [kBY][kHX], after the sums are consumed
    __shared__ float red[2][kTileThreads / kWave];

    const int tid = threadIdx.x;
    // Workgroups are dealt round-robin to the XCDs: give each XCD a
    // contiguous band of tiles so that neighbouring tiles, which read each
    // other's halos, share an L2.
    const int nb = a.tiles_x * a.tiles_y * (int)gridDim.z;
    const int b = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const int per = nb / kXcds;
    const int lb = b < per * kXcds ? (b % kXcds) * per + b / kXcds : b;
    const int ch = lb / (a.tiles_x * a.tiles_y);
    const int rem = lb - ch * a.tiles_x * a.tiles_y;
    const int ty = rem / a.tiles_x, tx = rem - ty * a.tiles_x;
    const int x0 = tx * kT, y0 = ty * kT;
    const int W = a.W, H = a.H;
    const int64_t plane = (int64_t)ch * W * H;
    const float* __restrict__ gx = a.x + plane;
    const float* __restrict__ gy = a.y + plane;

    // ---- input with a 10-pixel halo, zero outside the image: a wave per
    // row (lanes 0..53 load), four rows per pass
    {
        const int c = tid % kWave, px = x0 - 2 * kR + c;
        const bool col_ok = c < kALoad && px >= 0 && px < W;
        for (int r = tid / kWave; r < kAY; r += kTileThreads / kWave) {
            const int py = y0 - 2 * kR + r;
            float vx = 0.f, vy = 0.f;
            if (col_ok && py >= 0 && py < H) {
                const int64_t q = (int64_t)py * W + px;
                vx = gx[q];
                vy = gy[q];
            }
            if (c < kALoad) {
                sx[r * kAX + c] = vx;
                sy[r * kAX + c] = vy;
            }
        }
    }
    __syncthreads();

    // the inputs at this thread's output pixels, for the last step
    const int oc = tid % kT, or0 = (tid / kT) * kDGroup;
    float xo[kDGroup], yo[kDGroup];
#pragma unroll
    for (int o = 0; o < kDGroup; ++o) {
        const int li = (or0 + o + 2 * kR) * kAX + oc + 2 * kR;
        xo[o] = sx[li];
        yo[o] = sy[li];
    }

    // ---- forward window sums on the tile plus a 5-pixel halo: x, y, xy
    // first, then x^2, y^2 (three horizontal planes at a time)
    const bool vact = tid < kBX * (kBY / kVGroup);
    const int vc = tid % kBX, vr0 = (tid / kBX) * kVGroup;
    hpass<3>(a.win, sx, sy, sh, tid, [](float u, float v, float (&pr)[3][kHGroup + 2 * kR], int t) {
        pr[0][t] = u;
        pr[1][t] = v;
        pr[2][t] = u * v;
    });
    __syncthreads();
    float m1[3][kVGroup];
    if (vact) vpass<3>(a.win, sh, vc, vr0, m1);
    __syncthreads();
    hpass<2>(a.win, sx, sy, sh, tid, [](float u, float v, float (&pr)[2][kHGroup + 2 * kR], int t) {
        pr[0][t] = u * u;
        pr[1][t] = v * v;
    });
    __syncthreads();

    // ---- SSIM and its partials w.r.t. the window sums of x
    float pm[kVGroup], pe[kVGroup], pxy[kVGroup];
    float ssum = 0.f;
    if (vact) {
        float m2[2][kVGroup];
        vpass<2>(a.win, sh, vc, vr0, m2);
        const int px = x0 - kR + vc;
        const bool col_in = px >= 0 && px < W;
        const bool col_tile = vc >= kR && vc < kR + kT;
#pragma unroll
        for (int o = 0; o < kVGroup; ++o) {
            const int py = y0 - kR + vr0 + o;
            const float mx = m1[0][o], my = m1[1][o];
            const float vx = m2[0][o] - mx * mx, vy = m2[1][o] - my * my, cxy = m1[2][o] - mx * my;
            const float a1 = 2.f * mx * my + kC1, a2 = 2.f * cxy + kC2;
            const float b1 = mx * mx + my * my + kC1, b2 = vx + vy + kC2;
            const float inv = __builtin_amdgcn_rcpf(b1 * b2);
            const float S = a1 * a2 * inv;
            const bool in = col_in && py >= 0 && py < H;
            const int rr = vr0 + o;
            if (in && col_tile && rr >= kR && rr < kR + kT) ssum += S;
            pm[o] = in ? a.gs * 2.f * inv * (my * (a2 - a1) - mx * S * (b2 - b1)) : 0.f;
            pe[o] = in ? -a.gs * S * b1 * inv : 0.f;
            pxy[o] = in ? a.gs * 2.f * a1 * inv : 0.f;
        }
    }
    __syncthreads();  // every read of the horizontal sums is done
    if (vact) {
#pragma unroll
        for (int o = 0; o < kVGroup; ++o) {
            const int q = (vr0 + o) * kHX + vc;
            sp[q] = pm[o];
            sp[kSP + q] = pe[o];
            sp[2 * kSP + q] = pxy[o];
        }
    }
    __syncthreads();

    // ---- backward horizontal pass: rows 0..41, output columns 0..31
    if (tid < kBY * (kT / kQGroup)) {
        const int r = tid / (kT / kQGroup), c0 = (tid % (kT / kQGroup)) * kQGroup;
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            float v[kQGroup + 2 * kR];
#pragma unroll
            for (int t = 0; t < kQGroup + 2 * kR; ++t) v[t] = sp[m * kSP + r * kHX + c0 + t];
#pragma unroll
            for (int o = 0; o < kQGroup; ++o) {
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < kTaps; ++t) s = fmaf(a.win.g[t], v[o + t], s);
                sq[m * kSQ + r * kT + c0 + o] = s;
            }
        }
    }
    __syncthreads();

    // ---- backward vertical pass, gradient and L1 term on the tile
    float l1sum = 0.f;
    {
        float d[3][kDGroup];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            float v[kDGroup + 2 * kR];
#pragma unroll
            for (int t = 0; t < kDGroup + 2 * kR; ++t) v[t] = sq[m * kSQ + (or0 + t) * kT + oc];
#pragma unroll
            for (int o = 0; o < kDGroup; ++o) {
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < kTaps; ++t) s = fmaf(a.win.g[t], v[o + t], s);
                d[m][o] = s;
            }
        }
        const int px = x0 + oc;
#pragma unroll
        for (int o = 0; o < kDGroup; ++o) {
            const int py = y0 + or0 + o;
            if (px < W && py < H) {
                const int64_t q = plane + (int64_t)py * W + px;
                const float xa = a.xa ? a.xa[q] : xo[o];
                const float df = xa - yo[o];
                l1sum += fabsf(df);
                const float d1 = df > 0.f ? a.g1 : (df < 0.f ? -a.g1 : 0.f);
                const float ds = d[0][o] + 2.f * xo[o] * d[1][o] + yo[o] * d[2][o];
                if (a.dxa) {
                    a.dx[q] = ds;
                    a.dxa[q] = d1;
                } else {
                    a.dx[q] = ds + d1;
                }
            }
        }
    }

    // ---- per-workgroup partial sums
    ssum = wave_sum(ssum);
    l1sum = wave_sum(l1sum);
    if ((tid & (kWave - 1)) == 0) {
        red[0][tid / kWave] = ssum;
        red[1][tid / kWave] = l1sum;
    }
    __syncthreads();
    if (tid == 0) {
        float s = 0.f, l = 0.f;
        for (int k = 0; k < kTileThreads / kWave; ++k) {
            s += red[0][k];
            l += red[1][k];
        }
        a.partial[lb] = make_float2(s, l);
    }
}

// Adds the four rows v[NQ] of row group n to the vertical sums of
// the four groups they reach, input step t = 4 k + i of the group k back:
// completes group n - 3 (returned in `done`), adds to the pending groups
// n - 2 and n - 1 (acc[q][0] and acc[q][1] afterwards) and starts group n
// (acc[q][2]).  kw[t] holds the lane's window weights g[t - lane % 4].
// PLAIN: by fused multiply-adds over the window's own taps.
template <bool PLAIN, int NQ>
__device__ __forceinline__ void add_rows(const f4 (&v)[NQ], const float (&kw)[kSteps], const Win& win,
                                         f4 (&acc)[NQ][kPend], f4 (&done)[NQ]) {
    f4 grp[kPend + 1][NQ];   // group n - k
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int k = 1; k <= kPend; ++k) grp[k][q] = acc[q][kPend - k];
        grp[0][q] = f4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int k = kPend; k >= 0; --k)
#pragma unroll
        for (int i = 0; i < kG; ++i) {
            const int t = kG * k + i;
            if (t >= kSteps) continue;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if (!PLAIN) {
                    grp[k][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(kw[t], v[q][i], grp[k][q], 0, 0, 0);
                } else {
#pragma unroll
                    for (int r = 0; r < kG; ++r)
                        if (t - r >= 0 && t - r < kTaps)
                            grp[k][q][r] = fmaf(win.g[t - r], v[q][i], grp[k][q][r]);
                }
            }
        }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        done[q] = grp[kPend][q];
#pragma unroll
        for (int k = 0; k < kPend; ++k) acc[q][kPend - 1 - k] = grp[k][q];
    }
}

// Horizontal sums of the four staged rows s[planes][kG][kStride]: out[q][r] =
// row r at the wave's column `lane`, over the staged columns lane .. lane +
// 10.  A lane reads the fourteen columns from 4 (lane / 4) of row lane % 4.
// MOMENTS: two planes x, y staged, sums of x, y, xy, x^2, y^2 (NQ = 5);
// else the NQ planes themselves.
template <bool PLAIN, bool MOMENTS, int NQ>
__device__ __forceinline__ void row_sums(const float* __restrict__ s, int lane, const float (&kw)[kSteps],
                                         const Win& win, f4 (&out)[NQ]) {
    constexpr int NP = MOMENTS ? 2 : NQ;
    auto values = [](const float (&c)[NP], float (&v)[NQ]) {
#pragma unroll
        for (int q = 0; q < NP; ++q) v[q] = c[q];
        if constexpr (MOMENTS) {
            v[2] = c[0] * c[1];
            v[3] = c[0] * c[0];
            v[4] = c[1] * c[1];
        }
    };
#pragma unroll
    for (int q = 0; q < NQ; ++q) out[q] = f4{0.f, 0.f, 0.f, 0.f};
    if (PLAIN) {
#pragma unroll
        for (int r = 0; r < kG; ++r)
            for (int t = 0; t < kTaps; ++t) {
                float c[NP], v[NQ];
#pragma unroll
                for (int q = 0; q < NP; ++q) c[q] = s[(q * kG + r) * kStride + lane + t];
                values(c, v);
#pragma unroll
                for (int q = 0; q < NQ; ++q) out[q][r] = fmaf(win.g[t], v[q], out[q][r]);
            }
        return;
    }
    const float* src = s + (lane & (kG - 1)) * kStride + (lane & ~(kG - 1));
#pragma unroll
    for (int j = 0; j < kSteps; j += 4) {
        float c[4][NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const float* p = src + q * kG * kStride + j;
            if (j + 4 <= kSteps) {
                const float4 w = *reinterpret_cast<const float4*>(p);
                c[0][q] = w.x;
                c[1][q] = w.y;
                c[2][q] = w.z;
                c[3][q] = w.w;
            } else {
                const float2 w = *reinterpret_cast<const float2*>(p);
                c[0][q] = w.x;
                c[1][q] = w.y;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (j + e >= kSteps) continue;
            float v[NQ];
            values(c[e], v);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                out[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(v[q], kw[j + e], out[q], 0, 0, 0);
        }
    }
}

struct LossLds {
    float in[2][2 * kG * kStride];   // input rows x, y of this step and the next
    float p[2][3 * kG * kStride];    // the SSIM partials of this step and the last
    float g[kTaps + 2 * (kG - 1)];   // the window between zeros
    // the step in which a value that a zero weight would not cancel was
    // staged; looked at one step later, so that every thread sees the same
    int big;
    double red[2][kColWaves];
};

// One workgroup's segment; false (for every thread alike) when a big value
// was met, which only the PLAIN form treats right.
template <bool PLAIN>
__device__ __forceinline__ bool segment(const LossArgs& a, LossLds& L, int lb, const float (&kw)[kSteps]) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const bool front = tid < kCols;                                // the SSIM half, else the gradient half
    const int cw = (tid / kWave) % kColWaves, col = tid % kCols;   // its 64 columns, its column
    const int ch = lb / (a.strips * a.segs);
    const int rem = lb - ch * a.strips * a.segs;
    const int strip = rem / a.segs, seg = rem - strip * a.segs;
    const int x0 = strip * kOutW, y0 = seg * a.rows;
    const int W = a.W, H = a.H;
    const int64_t plane = (int64_t)ch * W * H;
    const float* __restrict__ gx = a.x + plane;
    const float* __restrict__ gy = a.y + plane;
    const int out_w = min(kOutW, W - x0), y1 = min(H, y0 + a.rows);
    const int steps = (y1 - y0 + kG - 1) / kG + 6;
    // a wave whose columns no output of the strip needs only keeps the
    // barriers (its staged columns stay zero)
    const bool active = cw * kWave < out_w + 4 * kR;

    // Step n: the front takes input rows group n (staged in step n - 1) and,
    // from n = 3 on, stages the partials of SSIM rows group n - 3; the back
    // takes those in step n + 1 and completes output rows group n - 6.
    if (front) {
        // input column x0 - 10 + col, from row y0 - 10; SSIM column x0 - 5
        // + col, from row y0 - 5
        const int ix = x0 - 2 * kR + col, sxc = x0 - kR + col;
        const bool in_col = ix >= 0 && ix < W, ss_col = sxc >= 0 && sxc < W;
        const bool sum_col = col >= kR && col < kR + out_w;
        const int ixc = in_col ? ix : 0;
        f4 acc[5][kPend];
#pragma unroll
        for (int k = 0; k < kPend; ++k)
#pragma unroll
            for (int q = 0; q < 5; ++q) acc[q][k] = f4{0.f, 0.f, 0.f, 0.f};
        const float gs = a.gs;
        double ssum = 0.0;   // a lane's sum runs down the whole segment: FP64 above a group's four rows
        float nx[kG], ny[kG];   // the rows staged next
        auto load = [&](int n) {
#pragma unroll
            for (int i = 0; i < kG; ++i) {
                const int py = y0 - 2 * kR + kG * n + i;
                const bool ok = in_col && py >= 0 && py < H;
                const int64_t q = (int64_t)min(max(py, 0), H - 1) * W + ixc;
                const float u = gx[q], w = gy[q];
                nx[i] = ok ? u : 0.f;
                ny[i] = ok ? w : 0.f;
            }
        };
        auto put = [&](int n, int step) {
            float* dst = L.in[n & 1] + col;
            float worst = 0.f;
#pragma unroll
            for (int i = 0; i < kG; ++i) {
                dst[i * kStride] = nx[i];
                dst[(kG + i) * kStride] = ny[i];
                worst += nx[i] * nx[i] + ny[i] * ny[i];
            }
            if (!PLAIN && !(worst < kBig)) L.big = step;
        };
        if (active) {
            load(0);
            put(0, -1);
            load(1);
        }
        __syncthreads();
        for (int n = 0; n < steps; ++n) {
            if (!PLAIN && __builtin_amdgcn_readfirstlane(L.big) < n) return false;
            if (active) {
                put(n + 1, n);
                load(n + 2);
                f4 h[5], m[5];
                row_sums<PLAIN, true, 5>(L.in[n & 1] + cw * kWave, lane, kw, a.win, h);
                add_rows<PLAIN, 5>(h, kw, a.win, acc, m);
                if (n >= 3) {
                    float* dst = L.p[n & 1] + col;
                    float worst = 0.f, group = 0.f;
#pragma unroll
                    for (int i = 0; i < kG; ++i) {
                        const int py = y0 - kR + kG * (n - 3) + i;
                        const float mx = m[0][i], my = m[1][i];
                        const float vx = m[3][i] - mx * mx, vy = m[4][i] - my * my, cxy = m[2][i] - mx * my;
                        const float a1 = 2.f * mx * my + kC1, a2 = 2.f * cxy + kC2;
                        const float b1 = mx * mx + my * my + kC1, b2 = vx + vy + kC2;
                        const float inv = __builtin_amdgcn_rcpf(b1 * b2);
                        const float S = a1 * a2 * inv;
                        const bool in = ss_col && py >= 0 && py < H;
                        if (in && sum_col && py >= y0 && py < y1) group += S;
                        const float p0 = in ? gs * 2.f * inv * (my * (a2 - a1) - mx * S * (b2 - b1)) : 0.f;
                        const float p1 = in ? -gs * S * b1 * inv : 0.f;
                        const float p2 = in ? gs * 2.f * a1 * inv : 0.f;
                        worst += fabsf(p0) + fabsf(p1) + fabsf(p2);
                        dst[i * kStride] = p0;
                        dst[(kG + i) * kStride] = p1;
                        dst[(2 * kG + i) * kStride] = p2;
                    }
                    ssum += (double)group;
                    if (!PLAIN && !(worst < kBig)) L.big = n;
                }
            }
            __syncthreads();
        }
        if (!PLAIN && __builtin_amdgcn_readfirstlane(L.big) < steps) return false;
        ssum = wave_sum(ssum);
        if (lane == 0) L.red[0][cw] = ssum;
    } else {
        // output column x0 + col, from row y0
        const bool out_col = col < out_w;
        const int oxc = out_col ? x0 + col : 0;
        f4 acc[3][kPend];
#pragma unroll
        for (int k = 0; k < kPend; ++k)
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[q][k] = f4{0.f, 0.f, 0.f, 0.f};
        const bool eq3 = a.xa != nullptr;
        const float* __restrict__ ga = (eq3 ? a.xa : a.x) + plane;
        float* __restrict__ dx = a.dx + plane;
        float* __restrict__ dxa = eq3 ? a.dxa + plane : nullptr;
        const float g1 = a.g1;
        double l1sum = 0.0;
        // the partials staged in step n; output rows group n - 6
        auto take = [&](int n) {
            float xo[kG], yo[kG], ao[kG];   // the inputs at the output rows
            if (n >= 6) {
#pragma unroll
                for (int i = 0; i < kG; ++i) {
                    const int64_t q = (int64_t)min(y0 + kG * (n - 6) + i, H - 1) * W + oxc;
                    xo[i] = gx[q];
                    yo[i] = gy[q];
                    ao[i] = ga[q];
                }
            }
            f4 h[3], d[3];
            row_sums<PLAIN, false, 3>(L.p[n & 1] + cw * kWave, lane, kw, a.win, h);
            add_rows<PLAIN, 3>(h, kw, a.win, acc, d);
            if (n < 6) return;
            float group = 0.f;
#pragma unroll
            for (int i = 0; i < kG; ++i) {
                const int py = y0 + kG * (n - 6) + i;
                const float df = ao[i] - yo[i];
                const float d1 = df > 0.f ? g1 : (df < 0.f ? -g1 : 0.f);
                const float ds = d[0][i] + 2.f * xo[i] * d[1][i] + yo[i] * d[2][i];
                if (out_col && py < y1) {
                    const int64_t q = (int64_t)py * W + oxc;
                    group += fabsf(df);
                    dx[q] = eq3 ? ds : ds + d1;
                    if (eq3) dxa[q] = d1;
                }
            }
            l1sum += (double)group;
        };
        __syncthreads();
        for (int n = 0; n < steps; ++n) {
            if (!PLAIN && __builtin_amdgcn_readfirstlane(L.big) < n) return false;
            if (active && n >= 4) take(n - 1);
            __syncthreads();
        }
        if (!PLAIN && __builtin_amdgcn_readfirstlane(L.big) < steps) return false;
        if (active) take(steps - 1);
        l1sum = wave_sum(l1sum);
        if (lane == 0) L.red[1][cw] = l1sum;
    }

    // ---- per-workgroup partial sums
    __syncthreads();
    if (tid == 0) {
        double s = 0.0, l = 0.0;
        for (int k = 0; k < kColWaves; ++k) {
            s += L.red[0][k];
            l += L.red[1][k];
        }
        a.partial[lb] = make_float2((float)s, (float)l);
    }
    return true;
}

// Zeros in the staged columns that no active wave writes.
__device__ __forceinline__ void clear_staged(LossLds& L, int active_cols) {
    for (int c = active_cols + (int)(threadIdx.x % kWave); c < kStride; c += kWave)
        for (int r = threadIdx.x / kWave; r < 5 * kG; r += kThreads / kWave)
            for (int k = 0; k < 2; ++k)
                (r < 2 * kG ? L.in[k] + r * kStride : L.p[k] + (r - 2 * kG) * kStride)[c] = 0.f;
}

// What bounds it: the issue of the matrix and vector instructions (about 56
// matrix and 60 vector ones per row and 64 columns, halo included: 26 and 20
// of its 68 us at 1920 x 1080 x 3) and the waits at one barrier a step.  The
// front and the gradient half of a row are different waves, so that a
// step's latency chain is cut in two and four waves fit a SIMD.
__global__ __launch_bounds__(kThreads, 4) void k_loss_strips(LossArgs a) {
    __shared__ __align__(16) LossLds L;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    // Workgroups are dealt round-robin to the XCDs: give each XCD a
    // contiguous run of segments so that neighbours, which read each
    // other's halos, share an L2.
    const int nb = (int)gridDim.x, b = (int)blockIdx.x, per = nb / kXcds;
    const int lb = b < per * kXcds ? (b % kXcds) * per + b / kXcds : b;
    const int strip = lb / a.segs % a.strips;
    const int used = min(kOutW, a.W - strip * kOutW) + 4 * kR;   // input columns
    const int active_cols = min(kCols, (used + kWave - 1) / kWave * kWave);
    clear_staged(L, active_cols);
    if (tid < kTaps + 2 * (kG - 1)) {
        float w = 0.f;
#pragma unroll
        for (int t = 0; t < kTaps; ++t) w = tid == kG - 1 + t ? a.win.g[t] : w;
        L.g[tid] = w;
    }
    if (tid == 0) L.big = INT_MAX;
    __syncthreads();
    float kw[kSteps];
#pragma unroll
    for (int t = 0; t < kSteps; ++t) kw[t] = L.g[kG - 1 + t - (lane & (kG - 1))];
    if (!segment<false>(a, L, lb, kw)) {
        __syncthreads();
        segment<true>(a, L, lb, kw);
    }
}

// 512: the whole call 16.0 us at 333 x 251 and 35.1 at 760 x 560 (1296
// partials); 256: 16.2 and 35.6; 1024: 16.5 and 35.3
constexpr int kFinThreads = 512;

// loss[0] = (1 - lambda) L1 + lambda (1 - SSIM), loss[1] = L1, loss[2] = SSIM
__global__ __launch_bounds__(kFinThreads) void k_loss_finish(const float2* __restrict__ partial, int64_t count,
                                                             double n, double lam, float* __restrict__ loss,
                                                             int n_out) {
    constexpr int kW = kFinThreads / kWave;
    __shared__ double red[2][kW];
    double s = 0.0, l = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += kFinThreads) {
        const float2 p = partial[i];
        s += (double)p.x;
        l += (double)p.y;
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, kWave);
        l += __shfl_xor(l, o, kWave);
    }
    const int lane = threadIdx.x & (kWave - 1);
    if (lane == 0) {
        red[0][threadIdx.x / kWave] = s;
        red[1][threadIdx.x / kWave] = l;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    s = lane < kW ? red[0][lane] : 0.0;
    l = lane < kW ? red[1][lane] : 0.0;
    for (int o = kW / 2; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, kWave);
        l += __shfl_xor(l, o, kWave);
    }
    if (lane == 0) {
        const double ssim = s / n, l1 = l / n;
        loss[0] = (float)((1.0 - lam) * l1 + lam * (1.0 - ssim));
        if (n_out == 3) {
            loss[1] = (float)l1;
            loss[2] = (float)ssim;
        }
    }
}

Win make_window() {
    Win w;
    double g[kTaps], tot = 0.0;
    for (int t = 0; t < kTaps; ++t) {
        const double k = t - kR;
        g[t] = std::exp(-k * k / (2.0 * 1.5 * 1.5));
        tot += g[t];
    }
    for (int t = 0; t < kTaps; ++t) w.g[t] = (float)(g[t] / tot);
    return w;
}

}  // namespace

int64_t loss_blocks(int channels, int width, int height) {
    return (int64_t)channels * ((width + kT - 1) / kT) * ((height + kT - 1) / kT);
}

namespace {

// Strips and segments of an image, or tiles (strips = 0).  Up to two rounds
// of tiles (three workgroups a CU) the tiles are as fast or faster, the
// strips' chain of steps being too long for so little work: 333 x 251 x 3
// 16 against 21 us, 800 x 600 x 3 (1425 tiles) 36 us both, 1000 x 700 x 3
// (2112) 50 against 43, 1920 x 1080 x 3 118 against 72 (both kernels).  As
// many segments as fill the resident workgroups once (a longer segment
// recomputes fewer halo rows, but a second round of workgroups would run
// nearly empty), and never more workgroups than the workspace holds
// partials (one per 32 x 32 tile; segments of 32 rows always meet that).
struct LossPlan {
    int strips, segs, rows;
};
constexpr int64_t kTileRounds = 2 * 768;

LossPlan loss_plan(int channels, int width, int height) {
    LossPlan p = {0, 0, 0};
    const int64_t tiles = loss_blocks(channels, width, height);
    if (tiles <= kTileRounds) return p;
    p.strips = (width + kOutW - 1) / kOutW;
    const int64_t lines = (int64_t)channels * p.strips;
    const int64_t want = std::max<int64_t>(1, kResident / lines);
    int64_t rows = (height + want - 1) / want;
    rows = std::max<int64_t>(2 * kG, (rows + kG - 1) / kG * kG);
    while (rows < kT && lines * ((height + rows - 1) / rows) > tiles) rows += kG;
    p.rows = (int)rows;
    p.segs = (int)((height + rows - 1) / rows);
    return p;
}

int64_t plan_blocks(const LossPlan& p, int channels, int width, int height) {
    return p.strips ? (int64_t)channels * p.strips * p.segs : loss_blocks(channels, width, height);
}

}  // namespace

size_t loss_workspace_bytes(int channels, int width, int height) {
    return (size_t)loss_blocks(channels, width, height) * sizeof(float2);
}

void launch_loss(const float* image, const float* image_l1, const float* target, int channels, int width, int height,
                 float lambda, float* d_image, float* d_image_l1, void* ws, hipStream_t st) {
    static const Win win = make_window();
    const double n = (double)channels * width * height;
    const LossPlan p = loss_plan(channels, width, height);
    LossArgs a;
    a.x = image;
    a.xa = image_l1;
    a.y = target;
    a.dx = d_image;
    a.dxa = image_l1 ? d_image_l1 : nullptr;
    a.partial = static_cast<float2*>(ws);
    a.W = width;
    a.H = height;
    a.tiles_x = (width + kT - 1) / kT;
    a.tiles_y = (height + kT - 1) / kT;
    a.strips = p.strips;
    a.segs = p.segs;
    a.rows = p.rows;
    a.gs = (float)(-(double)lambda / n);
    a.g1 = (float)((1.0 - (double)lambda) / n);
    a.win = win;
    if (p.strips)
        hipLaunchKernelGGL(k_loss_strips, dim3((unsigned)plan_blocks(p, channels, width, height)), dim3(kThreads), 0,
                           st, a);
    else
        hipLaunchKernelGGL(k_loss_tile, dim3(a.tiles_x, a.tiles_y, channels), dim3(kTileThreads), 0, st, a);
}

void launch_loss_finish(int channels, int width, int height, float lambda, const void* ws, float* loss,
                        hipStream_t st, int n_out) {
    const double n = (double)channels * width * height;
    hipLaunchKernelGGL(k_loss_finish, dim3(1), dim3(kFinThreads), 0, st, static_cast<const float2*>(ws),
                       plan_blocks(loss_plan(channels, width, height), channels, width, height), n, (double)lambda,
                       loss, n_out);
}

}  // namespace gs

// ---- the loss without a caller workspace ---------------------------------
// For callers that cannot allocate (code under stream capture, serving
// loops): the per-tile partial sums go to a fixed device array instead of
// a workspace.  Every call on a device uses that device's copy of the
// array, so calls that overlap on one device race; each call rewrites
// every partial it reads, so nothing needs clearing between calls.
namespace gs {
namespace {

constexpr size_t kLossScratchBytes = (size_t)1 << 20;   // 131072 (tile, channel) partials: 8K RGB
static __device__ __align__(256) unsigned char scratch[kLossScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices];

// Device address of the current device's `scratch`, looked up once per
// device with that device current (each device holds its own copy).
gs_status scratch_of_current_device(void** out) {
    int dev = 0;
    const hipError_t ed = hipGetDevice(&dev);
    if (ed != hipSuccess) return fail(GS_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(ed));
    if (dev < 0 || dev >= kMaxDevices) return fail(GS_ERR_UNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(GS_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        g_scratch[dev] = p;
    }
    *out = g_scratch[dev];
    return GS_OK;
}

}  // namespace
}  // namespace gs

extern "C" gs_status gs_loss_noalloc(const float* image, const float* image_l1, const float* target,
                                     int32_t channels, int32_t width, int32_t height, float lambda, float* loss,
                                     float* d_image, float* d_image_l1, gs_stream stream) {
    using namespace gs;
    size_t need = 0;
    gs_status s;
    if ((s = gs_loss_workspace(channels, width, height, &need))) return s;
    if (!image || !target || !loss || !d_image) return fail(GS_ERR_INVALID, "buffer is NULL");
    if (image_l1 && !d_image_l1) return fail(GS_ERR_INVALID, "image_l1 given without d_image_l1");
    if (!std::isfinite(lambda)) return fail(GS_ERR_INVALID, "lambda not finite");
    if (need > kLossScratchBytes)
        return fail(GS_ERR_CAPACITY, "a %dx%dx%d image needs %zu bytes of partial sums, more than the %zu this call holds",
                    channels, height, width, need, kLossScratchBytes);
    void* ws = nullptr;
    if ((s = scratch_of_current_device(&ws))) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    launch_loss(image, image_l1, target, channels, width, height, lambda, d_image, image_l1 ? d_image_l1 : nullptr,
                ws, st);
    launch_loss_finish(channels, width, height, lambda, ws, loss, st);
    return check_hip("gs_loss_noalloc");
}
