// Image-quality metric on the device: mean SSIM of two CHW float images
// (the third metric of the quality table, Table 4; Wang et al. 2004).
//
// Per channel, local means, variances and covariance under an 11 x 11
// Gaussian window (sigma 1.5, normalised), constants C1 = 0.01^2 and
// C2 = 0.03^2 (dynamic range 1), the SSIM map over every window position
// inside the image, averaged over positions and channels.
//
//   k_ssim        a wave per strip of 64 window columns (of two or four planes
//                 whose maps are narrow) and some rows, no wave waiting for
//                 another.  Four image rows at a time: a
//                 lane makes the five horizontal window sums (mean a, mean b,
//                 a^2, b^2, a b) of four neighbouring positions of one row
//                 from 14 pixels of its own, and they change to a lane per
//                 column through LDS; there each row is added to the eleven
//                 windows that it lies in (55 running sums in registers), and
//                 the window that it completes gives a map value.  All in
//                 FP64 (the variances are differences of nearly equal sums,
//                 and FP64 vector FMA runs at the non-packed FP32 rate); the
//                 strip's sum to its own slot
//   k_ssim_total  one block adds the slots in a fixed order (deterministic)
//
// Bound by FP64 issue: about 200 operations a position, which three planes of
// 2048x1080 issue in 50 us (an FP64 instruction of one wave takes 6 cycles
// here, not 4).  Sums kept in registers down a strip of rows and products made
// once per pixel take the place of 26 x 26 patches per 16 x 16 positions with
// every product made eleven times and every horizontal sum 1.6 times: 123 ->
// 63 us, and the sum of one slot per strip in place of one per tile 28 -> 4 us.
#include <cmath>

#include "gsc_common.h"
#include "gsc_ctx.h"

namespace gsc {

namespace {

constexpr int kWin = 11;
constexpr int kWaves = 4;      // per block
constexpr int kCols = 64;      // window columns of a strip
constexpr int kRows = 4;       // image rows at a time
constexpr int kPix = kWin + 3; // pixels under four neighbouring windows

// The 14 pixels of both images from column x of a row on (clamped to the
// image: a pixel outside it is only read for positions outside the map; no
// column of the strip needs that when `inside`).
struct Pixels {
    float a[kPix], b[kPix];
};
struct __attribute__((packed, aligned(4))) Float4 {  // four floats at any float's address
    float v[4];
};
__device__ __forceinline__ void load_row(float (&v)[kPix], const float* __restrict__ p) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const Float4 f = *reinterpret_cast<const Float4*>(p + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * i + e] = f.v[e];
    }
    v[12] = p[12];
    v[13] = p[13];
}
__device__ __forceinline__ void load_pixels(Pixels& p, const float* __restrict__ A, const float* __restrict__ B, int y,
                                            int x, int H, int W, bool inside) {
    const int64_t row = (int64_t)min(y, H - 1) * W;
    if (inside) {
        load_row(p.a, A + row + x);
        load_row(p.b, B + row + x);
    } else {
#pragma unroll
        for (int i = 0; i < kPix; ++i) {
            const int64_t at = row + min(x + i, W - 1);
            p.a[i] = A[at];
            p.b[i] = B[at];
        }
    }
}

struct Strips {
    int cols, rows;  // strips across and down the map
    int height;      // window rows of a strip
    int planes;      // groups of planes that share their strips
};

// kWide: a strip's columns of one plane (64 / kWide planes side by side).
template <int kWide>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_ssim(
    const float* __restrict__ a, const float* __restrict__ b, int C, int H, int W, SsimWindow win, Strips sp,
    double* __restrict__ partial) {
    constexpr int kPlanes = kCols / kWide;
    __shared__ __align__(16) double s_h[kWaves][5][kRows][kCols];  // horizontal sums of the wave's rows
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int strip = blockIdx.x * kWaves + w, strips = sp.cols * sp.rows;
    if (strip >= strips) return;  // (waves share nothing)
    const int x0 = strip % sp.cols * kCols, y0 = strip / sp.cols * sp.height;
    const int y1 = min(y0 + sp.height, H - kWin + 1);  // the strip's window rows [y0, y1)
    const int tr = lane >> 4, tc = (lane & 15) * 4;    // horizontal sums: row, first column
    // this lane's window column is in the map of a plane
    const bool column = x0 + lane % kWide <= W - kWin && (int)blockIdx.y * kPlanes + lane / kWide < C;
    const int64_t plane = (int64_t)min((int)blockIdx.y * kPlanes + tc / kWide, C - 1) * H * W;
    const float *A = a + plane, *B = b + plane;
    const int xh = x0 + tc % kWide;
    double acc[kWin][5];  // acc[t]: rows 0 .. t of the window that has come to its row t
#pragma unroll
    for (int t = 0; t < kWin; ++t)
#pragma unroll
        for (int q = 0; q < 5; ++q) acc[t][q] = 0.0;
    const bool inside = kPlanes == 1 && x0 + kCols + kWin - 1 <= W;  // (wave-uniform)
    double sum = 0.0;
    Pixels px;
    load_pixels(px, A, B, y0 + tr, xh, H, W, inside);
    for (int yb = y0; yb < y1 + kWin - 1; yb += kRows) {
        {
            double h[4][5];
#pragma unroll
            for (int i = 0; i < kPix; ++i) {
                const double x = px.a[i], y = px.b[i], xx = x * x, yy = y * y, xy = x * y;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = i - j;
                    if (t < 0 || t >= kWin) continue;
                    const double wt = win.w[t];
                    h[j][0] = fma(wt, x, t ? h[j][0] : 0.0);
                    h[j][1] = fma(wt, y, t ? h[j][1] : 0.0);
                    h[j][2] = fma(wt, xx, t ? h[j][2] : 0.0);
                    h[j][3] = fma(wt, yy, t ? h[j][3] : 0.0);
                    h[j][4] = fma(wt, xy, t ? h[j][4] : 0.0);
                }
            }
#pragma unroll
            for (int q = 0; q < 5; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) s_h[w][q][tr][tc + j] = h[j][q];
        }
        // the next rows' pixels are on their way during the vertical sums
        load_pixels(px, A, B, yb + kRows + tr, xh, H, W, inside);
        __builtin_amdgcn_wave_barrier();  // a wave's LDS accesses complete in order
        // (every row gives a value: a strip's first ten complete no window of
        // its own and count for nothing)
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            double h[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) h[q] = s_h[w][q][r][lane];
#pragma unroll
            for (int t = kWin - 1; t >= 0; --t)
#pragma unroll
                for (int q = 0; q < 5; ++q) acc[t][q] = fma(win.w[t], h[q], t ? acc[t ? t - 1 : 0][q] : 0.0);
            const int oy = yb + r - (kWin - 1);  // the window that this row completes
            const double c1 = 1e-4, c2 = 9e-4;
            const double m1 = acc[kWin - 1][0], m2 = acc[kWin - 1][1];
            const double vx = acc[kWin - 1][2] - m1 * m1, vy = acc[kWin - 1][3] - m2 * m2,
                         cxy = acc[kWin - 1][4] - m1 * m2;
            const double v = ((2.0 * m1 * m2 + c1) * (2.0 * cxy + c2)) / ((m1 * m1 + m2 * m2 + c1) * (vx + vy + c2));
            sum += column && oy >= y0 && oy < y1 ? v : 0.0;
        }
        __builtin_amdgcn_wave_barrier();
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) partial[(int64_t)blockIdx.y * strips + strip] = sum;
}

// Strips of a map of C planes: one wave on every SIMD (its 55 chains of sums
// are enough to fill it, and each strip reads ten rows more than it has: twice
// as many strips took 67 us in place of 63), of at least two rows, a whole
// number of steps of kRows image rows each.  Many planes of at most 32 or 16
// window columns share their strips by two or four (4,000 of 12x12 54 -> 31 us
// a call, 65,535 of 11x11 554 -> 179, 1,000 of 40x40 51 -> 44); few of them
// are better off with a strip each (1 of 20,000x20 38 -> 34).
int planes_of(int C, int W) {
    return C < 512 || W - kWin + 1 > 32 ? 1 : (W - kWin + 1 > 16 ? 2 : 4);
}
Strips strips_of(int C, int H, int W) {
    const int64_t h = H - kWin + 1, waves = 1024, np = planes_of(C, W);
    Strips sp;
    sp.cols = (W - kWin + 1 + kCols - 1) / kCols;
    sp.planes = (int)((C + np - 1) / np);
    int64_t down = waves / ((int64_t)sp.planes * sp.cols);
    if (down < 1) down = 1;
    const int64_t rows = (h + down - 1) / down + kWin - 1;
    sp.height = (int)((rows + kRows - 1) / kRows * kRows - (kWin - 1));
    sp.rows = (int)((h + sp.height - 1) / sp.height);
    return sp;
}

__global__ __launch_bounds__(256) void k_ssim_total(const double* __restrict__ partial, int64_t n, double* out) {
    __shared__ double s[256];
    double t = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) t += partial[i];
    s[threadIdx.x] = t;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

}  // namespace

SsimWindow ssim_window() {
    SsimWindow win;
    double g[kWin], sum = 0.0;
    for (int i = 0; i < kWin; ++i) {
        const double x = i - 0.5 * (kWin - 1);
        g[i] = std::exp(-x * x / (2.0 * 1.5 * 1.5));
        sum += g[i];
    }
    for (int i = 0; i < kWin; ++i) win.w[i] = g[i] / sum;
    return win;
}

int64_t ssim_slots(int C, int H, int W) {
    const Strips sp = strips_of(C, H, W);
    return (int64_t)sp.cols * sp.rows * sp.planes;
}

hipError_t ssim_launch(const float* a, const float* b, int C, int H, int W, const SsimWindow& win, double* partial,
                       double* total, hipStream_t st) {
    const Strips sp = strips_of(C, H, W);
    const unsigned blocks = (unsigned)((sp.cols * sp.rows + kWaves - 1) / kWaves);
    const dim3 grid(blocks, (unsigned)sp.planes);
    switch (planes_of(C, W)) {
        case 4: hipLaunchKernelGGL(k_ssim<16>, grid, dim3(64 * kWaves), 0, st, a, b, C, H, W, win, sp, partial); break;
        case 2: hipLaunchKernelGGL(k_ssim<32>, grid, dim3(64 * kWaves), 0, st, a, b, C, H, W, win, sp, partial); break;
        default: hipLaunchKernelGGL(k_ssim<64>, grid, dim3(64 * kWaves), 0, st, a, b, C, H, W, win, sp, partial);
    }
    hipLaunchKernelGGL(k_ssim_total, dim3(1), dim3(256), 0, st, partial, ssim_slots(C, H, W), total);
    return hipGetLastError();
}

}  // namespace gsc
