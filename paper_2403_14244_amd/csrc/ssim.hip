// The loss of the paper (Section 3): the SSIM term and the L1 term.
//
// SSIM: mean structural similarity of a rendered
// image and its target under an 11 x 11 Gaussian window (sigma 1.5, zero outside the
// image), C1 = 0.01^2, C2 = 0.03^2, and its gradient with respect to the rendered image.
//
// Forward: one workgroup per 32 x 22 output tile and channel. The tile's 42 x 32 input region
// is staged in LDS, filtered along rows then columns (the window is separable) for the five
// local statistics (G*x, G*y, G*x^2, G*y^2, G*xy); each pixel forms S and the three partial
// derivatives the backward needs (dS/dm1, dS/de11, dS/de12, with m1 = G*x, e11 = G*x^2,
// e12 = G*xy), which are stored in the workspace. Block sums of S (and of |x - y|, for the
// combined loss) are added in FP64 in a fixed order by one workgroup, so the mean is
// reproducible.
// Backward: the same tiling filters the three derivative maps (the window is symmetric,
// so the transposed filter is the filter) and combines them per pixel:
// dSSIM/dx = (G*dS/dm1 + 2 x G*dS/de11 + y G*dS/de12) / N.
//
// The filters are bound by LDS reads and FMAs, so a thread holds a sliding window in
// registers: four neighbouring outputs of a row from four 16-byte reads per plane, three
// neighbouring outputs of a column from thirteen reads. 32 staged rows of eight 4-column
// groups are one row task per thread; 22 = 32 - 10 output rows are three per thread.
// 3 x 1080 x 1920 values: forward 103 -> 63 us, backward 97 -> 37 us against 16 x 16
// tiles with one output per thread and read (and the L1 term's own pass of 17 us folded in).
#include "common.h"
#include "kernels.h"

#include <algorithm>

namespace isogs {

namespace {

constexpr int kWin = 11, kHalo = 5;
constexpr int kTileW = 32, kTileH = 22;              // output tile
constexpr int kRows = kTileH + 2 * kHalo;            // staged rows: 32
constexpr int kCols = kTileW + 2 * kHalo;            // staged columns: 42
constexpr int kPitch = 44;                           // staged row pitch (16-byte multiples)
constexpr int kThreads = 256, kRowOut = 4, kColOut = 3;
constexpr float kC1 = 0.0001f, kC2 = 0.0009f;
static_assert(kRows * (kTileW / kRowOut) == kThreads, "one row task per thread");
static_assert(kTileW * ((kTileH + kColOut - 1) / kColOut) == kThreads, "one column task per thread");
static_assert(kPitch % 4 == 0 && kTileW + 12 <= kPitch, "row tasks read four aligned vectors");

struct Window {
    float g[kWin];
};

// Stages the region around the tile at (x0, y0) of N planes (zero outside the image). A wave
// takes whole rows, one column per lane, so that the row part of the addresses is scalar;
// every load is issued before the first LDS write (addresses clamped into the plane, values
// selected after), so that a workgroup waits for memory once. Columns kCols .. kPitch - 1 are
// read by the last row task of a row but enter no output.
constexpr int kWaves = kThreads / kWave, kStage = kRows / kWaves;
static_assert(kPitch <= kWave && kRows % kWaves == 0, "one staged column per lane, whole rows per wave");

template <int N>
__device__ __forceinline__ void stage_regions(float (*dst)[kRows][kPitch], const float* const (&src)[N], int x0,
                                              int y0, int width, int height) {
    const int c = (int)lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int x = x0 - kHalo + c, xc = min(max(x, 0), width - 1);
    const bool x_in = x >= 0 && x < width;
    float v[N][kStage];
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
        const int y = y0 - kHalo + w + i * kWaves;
        const size_t row = (size_t)min(max(y, 0), height - 1) * width;
#pragma unroll
        for (int q = 0; q < N; ++q) v[q][i] = src[q][row + xc];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (c < kPitch) {
#pragma unroll
        for (int i = 0; i < kStage; ++i) {
            const int r = w + i * kWaves, y = y0 - kHalo + r;
            const bool in = x_in && y >= 0 && y < height;
#pragma unroll
            for (int q = 0; q < N; ++q) dst[q][r][c] = in ? v[q][i] : 0.0f;
        }
    }
}

// The sixteen staged values from column c (a multiple of four) of a row.
__device__ __forceinline__ void load_row16(const float* __restrict__ row, int c, float v[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 f = *reinterpret_cast<const float4*>(row + c + 4 * q);
        v[4 * q] = f.x;
        v[4 * q + 1] = f.y;
        v[4 * q + 2] = f.z;
        v[4 * q + 3] = f.w;
    }
}

// Row-filtered statistics reuse the LDS of the staged planes (a barrier between). The last
// column task reads two rows past them, for outputs below the tile that nothing keeps.
constexpr int kHRows = (kTileH + kColOut - 1) / kColOut * kColOut + kWin - 1;
template <int IN, int OUT>
struct FilterShared {
    union {
        float in[IN][kRows][kPitch];
        float h[OUT][kHRows][kTileW];
    };
};

// Column task: three outputs from row r of the row-filtered plane h, column c.
__device__ __forceinline__ void filter_column(const float (*h)[kTileW], const Window& win, int r, int c,
                                              float out[kColOut]) {
    float v[kColOut + kWin - 1];
#pragma unroll
    for (int k = 0; k < kColOut + kWin - 1; ++k) v[k] = h[r + k][c];
#pragma unroll
    for (int j = 0; j < kColOut; ++j) {
        float a = 0.0f;
#pragma unroll
        for (int k = 0; k < kWin; ++k) a = fmaf(win.g[k], v[j + k], a);
        out[j] = a;
    }
}

// Sum of two FP64 values over the workgroup in a fixed order, valid in thread 0.
__device__ __forceinline__ void block_sum2(double& a, double& b, double (*part)[2]) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, kWave);
        b += __shfl_xor(b, o, kWave);
    }
    if ((threadIdx.x & 63u) == 0) {
        part[threadIdx.x >> 6][0] = a;
        part[threadIdx.x >> 6][1] = b;
    }
    __syncthreads();
    a = ((part[0][0] + part[1][0]) + part[2][0]) + part[3][0];
    b = ((part[0][1] + part[1][1]) + part[2][1]) + part[3][1];
}

// L1: also the block sums of |x - y| (the combined loss; its planes are read once for both).
template <bool L1>
__global__ void __launch_bounds__(kThreads) ssim_fwd_kernel(const float* __restrict__ image,
                                                            const float* __restrict__ target, int width,
                                                            int height, int tiles_x, const Window win,
                                                            float* __restrict__ d_m1, float* __restrict__ d_e11,
                                                            float* __restrict__ d_e12,
                                                            double* __restrict__ block_sum,
                                                            double* __restrict__ l1_sum) {
    __shared__ __align__(16) FilterShared<2, 5> sh;
    __shared__ double part[kThreads / kWave][2];
    const uint32_t t = threadIdx.x, tile = xcd_swizzle(blockIdx.x, gridDim.x), ch = blockIdx.y;
    const int x0 = (int)(tile % (uint32_t)tiles_x) * kTileW, y0 = (int)(tile / (uint32_t)tiles_x) * kTileH;
    const size_t plane = (size_t)width * height;
    const float* const planes[2] = {image + ch * plane, target + ch * plane};
    stage_regions(sh.in, planes, x0, y0, width, height);
    __syncthreads();
    // column task of this thread: column c, rows r0 .. r0 + 2 of the tile
    const int c = (int)(t % kTileW), r0 = (int)(t / kTileW) * kColOut;
    float l1 = 0.0f;
    if (L1) {
#pragma unroll
        for (int j = 0; j < kColOut; ++j) {
            const int r = r0 + j;
            if (r < kTileH && y0 + r < height && x0 + c < width)
                l1 += fabsf(sh.in[0][r + kHalo][c + kHalo] - sh.in[1][r + kHalo][c + kHalo]);
        }
    }
    {
        const int r = (int)(t / (kTileW / kRowOut)), cc = (int)(t % (kTileW / kRowOut)) * kRowOut;
        float xv[16], yv[16];
        load_row16(sh.in[0][r], cc, xv);
        load_row16(sh.in[1][r], cc, yv);
        float a[5][kRowOut];
#pragma unroll
        for (int j = 0; j < kRowOut; ++j)
#pragma unroll
            for (int q = 0; q < 5; ++q) a[q][j] = 0.0f;
#pragma unroll
        for (int k = 0; k < kWin + kRowOut - 1; ++k) {
            const float x = xv[k], y = yv[k], xx = x * x, yy = y * y, xy = x * y;
#pragma unroll
            for (int j = 0; j < kRowOut; ++j) {
                if (k - j < 0 || k - j >= kWin) continue;
                const float g = win.g[k - j];
                a[0][j] = fmaf(g, x, a[0][j]);
                a[1][j] = fmaf(g, y, a[1][j]);
                a[2][j] = fmaf(g, xx, a[2][j]);
                a[3][j] = fmaf(g, yy, a[3][j]);
                a[4][j] = fmaf(g, xy, a[4][j]);
            }
        }
        __syncthreads();   // every read of the staged planes is done
#pragma unroll
        for (int q = 0; q < 5; ++q)
            *reinterpret_cast<float4*>(&sh.h[q][r][cc]) = make_float4(a[q][0], a[q][1], a[q][2], a[q][3]);
    }
    __syncthreads();
    float m[5][kColOut];
#pragma unroll
    for (int q = 0; q < 5; ++q) filter_column(sh.h[q], win, r0, c, m[q]);
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kColOut; ++j) {
        const float m1 = m[0][j], m2 = m[1][j];
        const float A1 = 2.0f * m1 * m2 + kC1;
        const float A2 = 2.0f * (m[4][j] - m1 * m2) + kC2;
        const float B1 = m1 * m1 + m2 * m2 + kC1;
        const float B2 = (m[2][j] - m1 * m1) + (m[3][j] - m2 * m2) + kC2;
        const float rB1 = 1.0f / B1, rB2 = 1.0f / B2;
        const float S = A1 * A2 * rB1 * rB2;
        const int px = x0 + c, py = y0 + r0 + j;
        if (r0 + j < kTileH && px < width && py < height) {
            const size_t o = ch * plane + (size_t)py * width + px;
            d_e11[o] = -S * rB2;                      // -A1 A2 / (B1 B2^2)
            d_e12[o] = 2.0f * A1 * rB1 * rB2;         // 2 A1 / (B1 B2)
            d_m1[o] = 2.0f * m2 * (A2 - A1) * rB1 * rB2 - 2.0f * m1 * S * rB1 + 2.0f * m1 * S * rB2;
            s += (double)S;
        }
    }
    double d1 = (double)l1;
    block_sum2(s, d1, part);
    if (t == 0) {
        block_sum[(size_t)ch * gridDim.x + tile] = s;
        if (L1) l1_sum[(size_t)ch * gridDim.x + tile] = d1;
    }
}

// Sum of n FP64 values by one workgroup of 1024 threads in a fixed order (strided runs per
// thread, then halving); valid in thread 0. s_run: 1024 words.
constexpr int kMeanThreads = 1024;
__device__ __forceinline__ double ordered_sum(const double* __restrict__ v, uint32_t n, double* s_run) {
    const uint32_t t = threadIdx.x;
    double a = 0.0;
    for (uint32_t i = t; i < n; i += kMeanThreads) a += v[i];
    s_run[t] = a;
    for (uint32_t o = kMeanThreads / 2; o > 0; o >>= 1) {
        __syncthreads();
        if (t < o) s_run[t] += s_run[t + o];
    }
    __syncthreads();
    const double r = s_run[0];
    __syncthreads();
    return r;
}

// Mean of the block sums.
__global__ void __launch_bounds__(kMeanThreads) ssim_mean_kernel(const double* __restrict__ block_sum,
                                                                 uint32_t n_blocks, double inv_n,
                                                                 float* __restrict__ ssim) {
    __shared__ double s_run[kMeanThreads];
    const double tot = ordered_sum(block_sum, n_blocks, s_run);
    if (threadIdx.x == 0) *ssim = (float)(tot * inv_n);
}

__global__ void __launch_bounds__(kThreads) ssim_bwd_kernel(const float* __restrict__ image,
                                                            const float* __restrict__ target, int width,
                                                            int height, int tiles_x, const Window win,
                                                            const float* __restrict__ d_m1,
                                                            const float* __restrict__ d_e11,
                                                            const float* __restrict__ d_e12,
                                                            const float* __restrict__ dL_dssim, float inv_n,
                                                            float ssim_w, float l1_w,
                                                            float* __restrict__ dL_dimage) {
    __shared__ __align__(16) FilterShared<3, 3> sh;
    const uint32_t t = threadIdx.x, tile = xcd_swizzle(blockIdx.x, gridDim.x), ch = blockIdx.y;
    const int x0 = (int)(tile % (uint32_t)tiles_x) * kTileW, y0 = (int)(tile / (uint32_t)tiles_x) * kTileH;
    const size_t plane = (size_t)width * height;
    // this thread's pixels are read while the maps are filtered
    const int c = (int)(t % kTileW), r0 = (int)(t / kTileW) * kColOut;
    const int px = x0 + c;
    float xi[kColOut], yi[kColOut];
#pragma unroll
    for (int j = 0; j < kColOut; ++j) {
        const int py = y0 + r0 + j;
        const bool in = r0 + j < kTileH && px < width && py < height;
        const size_t o = ch * plane + (size_t)py * width + px;
        xi[j] = in ? image[o] : 0.0f;
        yi[j] = in ? target[o] : 0.0f;
    }
    const float* const planes[3] = {d_m1 + ch * plane, d_e11 + ch * plane, d_e12 + ch * plane};
    stage_regions(sh.in, planes, x0, y0, width, height);
    __syncthreads();
    {
        const int r = (int)(t / (kTileW / kRowOut)), cc = (int)(t % (kTileW / kRowOut)) * kRowOut;
        float a[3][kRowOut];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            float v[16];
            load_row16(sh.in[q][r], cc, v);
#pragma unroll
            for (int j = 0; j < kRowOut; ++j) {
                a[q][j] = 0.0f;
#pragma unroll
                for (int k = 0; k < kWin; ++k) a[q][j] = fmaf(win.g[k], v[j + k], a[q][j]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q)
            *reinterpret_cast<float4*>(&sh.h[q][r][cc]) = make_float4(a[q][0], a[q][1], a[q][2], a[q][3]);
    }
    __syncthreads();
    float b[3][kColOut];
#pragma unroll
    for (int q = 0; q < 3; ++q) filter_column(sh.h[q], win, r0, c, b[q]);
    // dL/dimage = ssim_w g dSSIM/dimage (+ l1_w g sign(image - target) / n for the paper's
    // combined loss), g = dL_dssim[0]
    const float g = *dL_dssim;
    const float scale = ssim_w * g * inv_n;
#pragma unroll
    for (int j = 0; j < kColOut; ++j) {
        const int py = y0 + r0 + j;
        if (r0 + j >= kTileH || px >= width || py >= height) continue;
        float out = scale * (b[0][j] + 2.0f * xi[j] * b[1][j] + yi[j] * b[2][j]);
        if (l1_w != 0.0f) {
            const float gl = l1_w * g * inv_n, d = xi[j] - yi[j];
            out += d > 0.0f ? gl : (d < 0.0f ? -gl : 0.0f);
        }
        dL_dimage[ch * plane + (size_t)py * width + px] = out;
    }
}

// The paper's loss (1 - lambda) L1 + lambda (1 - SSIM) from the block sums of both terms.
__global__ void __launch_bounds__(kMeanThreads) loss_combine_kernel(const double* __restrict__ ssim_blocks,
                                                                    const double* __restrict__ l1_blocks,
                                                                    uint32_t n_blocks, double inv_n, double lam,
                                                                    float* __restrict__ loss) {
    __shared__ double s_run[kMeanThreads];
    const double st = ordered_sum(ssim_blocks, n_blocks, s_run);
    const double lt = ordered_sum(l1_blocks, n_blocks, s_run);
    if (threadIdx.x == 0) {
        const float ssim = (float)(st * inv_n);
        loss[0] = (float)((1.0 - lam) * (lt * inv_n) + lam * (1.0 - (double)ssim));
        loss[1] = ssim;
    }
}

Window make_window() {
    Window w{};
    double g[kWin], s = 0.0;
    for (int k = 0; k < kWin; ++k) {
        const double r = (double)(k - kHalo);
        g[k] = exp(-r * r / (2.0 * 1.5 * 1.5));
        s += g[k];
    }
    for (int k = 0; k < kWin; ++k) w.g[k] = (float)(g[k] / s);
    return w;
}

struct SsimWs {
    size_t off_m1, off_e11, off_e12, off_blocks, bytes, off_l1, loss_bytes;
};

int tiles_of(int32_t n, int edge) { return (int)(((int64_t)n + edge - 1) / edge); }

SsimWs ssim_layout(int32_t channels, int32_t height, int32_t width) {
    const size_t n = (size_t)channels * height * width;
    const size_t blocks = (size_t)channels * tiles_of(width, kTileW) * tiles_of(height, kTileH);
    auto a256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
    SsimWs w{};
    w.off_m1 = 0;
    w.off_e11 = a256(n * 4);
    w.off_e12 = w.off_e11 + a256(n * 4);
    w.off_blocks = w.off_e12 + a256(n * 4);
    w.bytes = w.off_blocks + a256(blocks * 8);
    // the combined loss also keeps the L1 block sums
    w.off_l1 = w.bytes;
    w.loss_bytes = w.off_l1 + a256(blocks * 8);
    return w;
}

}  // namespace

size_t ssim_ws_bytes(int32_t channels, int32_t height, int32_t width) {
    return ssim_layout(channels, height, width).bytes;
}

// The per-block kernel of both terms; l1: the L1 block sums, or NULL. Returns the block count.
static uint32_t launch_ssim_blocks(const float* image, const float* target, int32_t channels, int32_t height,
                                   int32_t width, const SsimWs& L, char* base, double* l1, hipStream_t stream) {
    const int tx = tiles_of(width, kTileW), ty = tiles_of(height, kTileH);
    const uint32_t tiles = (uint32_t)(tx * ty);
    auto k = l1 ? ssim_fwd_kernel<true> : ssim_fwd_kernel<false>;
    hipLaunchKernelGGL(k, dim3(tiles, (unsigned)channels), dim3(kThreads), 0, stream, image, target, width, height, tx,
                       make_window(), reinterpret_cast<float*>(base + L.off_m1),
                       reinterpret_cast<float*>(base + L.off_e11), reinterpret_cast<float*>(base + L.off_e12),
                       reinterpret_cast<double*>(base + L.off_blocks), l1);
    return tiles * (uint32_t)channels;
}

int launch_ssim_fwd(const float* image, const float* target, int32_t channels, int32_t height, int32_t width,
                    float* ssim, void* ws, hipStream_t stream) {
    const SsimWs L = ssim_layout(channels, height, width);
    char* base = static_cast<char*>(ws);
    const uint32_t nb = launch_ssim_blocks(image, target, channels, height, width, L, base, nullptr, stream);
    const double n = (double)channels * height * width;
    hipLaunchKernelGGL(ssim_mean_kernel, dim3(1), dim3(kMeanThreads), 0, stream,
                       reinterpret_cast<const double*>(base + L.off_blocks), nb, 1.0 / n, ssim);
    return hipPeekAtLastError() == hipSuccess ? 0 : -1;
}

int launch_ssim_bwd(const float* image, const float* target, int32_t channels, int32_t height, int32_t width,
                    const float* dL_dssim, const void* ws, float* dL_dimage, hipStream_t stream) {
    return launch_ssim_bwd_weighted(image, target, channels, height, width, dL_dssim, ws, 1.0f, 0.0f, dL_dimage,
                                    stream);
}

size_t loss_ws_bytes(int32_t channels, int32_t height, int32_t width) {
    return ssim_layout(channels, height, width).loss_bytes;
}

int launch_loss_fwd(const float* image, const float* target, int32_t channels, int32_t height, int32_t width,
                    float lambda, float* loss, void* ws, hipStream_t stream) {
    const SsimWs L = ssim_layout(channels, height, width);
    char* base = static_cast<char*>(ws);
    double* l1b = reinterpret_cast<double*>(base + L.off_l1);
    const uint32_t nb = launch_ssim_blocks(image, target, channels, height, width, L, base, l1b, stream);
    const double n = (double)channels * height * width;
    hipLaunchKernelGGL(loss_combine_kernel, dim3(1), dim3(kMeanThreads), 0, stream,
                       reinterpret_cast<const double*>(base + L.off_blocks), l1b, nb, 1.0 / n, (double)lambda, loss);
    return hipPeekAtLastError() == hipSuccess ? 0 : -1;
}

int launch_loss_bwd(const float* image, const float* target, int32_t channels, int32_t height, int32_t width,
                    float lambda, const float* dL_dloss, const void* ws, float* dL_dimage, hipStream_t stream) {
    // d/dimage [(1 - lambda) L1 + lambda (1 - SSIM)] = (1 - lambda) dL1 - lambda dSSIM
    return launch_ssim_bwd_weighted(image, target, channels, height, width, dL_dloss, ws, -lambda, 1.0f - lambda,
                                    dL_dimage, stream);
}

int launch_ssim_bwd_weighted(const float* image, const float* target, int32_t channels, int32_t height,
                             int32_t width, const float* dL_dssim, const void* ws, float ssim_w, float l1_w,
                             float* dL_dimage, hipStream_t stream) {
    const SsimWs L = ssim_layout(channels, height, width);
    const char* base = static_cast<const char*>(ws);
    const int tx = tiles_of(width, kTileW), ty = tiles_of(height, kTileH);
    const float inv_n = (float)(1.0 / ((double)channels * height * width));
    hipLaunchKernelGGL(ssim_bwd_kernel, dim3((unsigned)(tx * ty), (unsigned)channels), dim3(kThreads), 0, stream,
                       image, target, width, height, tx, make_window(),
                       reinterpret_cast<const float*>(base + L.off_m1), reinterpret_cast<const float*>(base + L.off_e11),
                       reinterpret_cast<const float*>(base + L.off_e12), dL_dssim, inv_n, ssim_w, l1_w, dL_dimage);
    return hipPeekAtLastError() == hipSuccess ? 0 : -1;
}

}  // namespace isogs

// ---- L1 term of the loss -------------------------------------------------------------
// mean |image - target|: block b sums its contiguous chunk of kL1Chunk values (FP32 per
// lane, then FP64 across the block's lanes in a fixed order); one workgroup adds the block
// sums in FP64 in block order. The backward writes g sign(image - target) / n, sign(0) = 0.
namespace isogs {

namespace {

constexpr int kL1Threads = 256, kL1PerThread = 16;
constexpr uint32_t kL1Chunk = kL1Threads * kL1PerThread;

__global__ void __launch_bounds__(kL1Threads) l1_partial_kernel(const float* __restrict__ image,
                                                                const float* __restrict__ target, uint64_t n,
                                                                double* __restrict__ block_sum) {
    __shared__ double s_w[kL1Threads / kWave];
    const uint64_t base = (uint64_t)blockIdx.x * kL1Chunk;
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < kL1PerThread; ++i) {
        const uint64_t k = base + (uint64_t)i * kL1Threads + threadIdx.x;
        if (k < n) a += fabsf(image[k] - target[k]);
    }
    double d = (double)a;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o, kWave);
    if ((threadIdx.x & 63u) == 0) s_w[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) block_sum[blockIdx.x] = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
}

__global__ void __launch_bounds__(256) l1_final_kernel(const double* __restrict__ block_sum, uint32_t n_blocks,
                                                       double inv_n, float* __restrict__ loss) {
    __shared__ double s_run[256];
    const uint32_t t = threadIdx.x, per = (n_blocks + 255u) / 256u;
    double a = 0.0;
    for (uint32_t i = t * per; i < min(n_blocks, (t + 1u) * per); ++i) a += block_sum[i];
    s_run[t] = a;
    __syncthreads();
    if (t == 0) {
        double tot = 0.0;
        for (int i = 0; i < 256; ++i) tot += s_run[i];
        *loss = (float)(tot * inv_n);
    }
}

__global__ void __launch_bounds__(kL1Threads) l1_grad_kernel(const float* __restrict__ image,
                                                             const float* __restrict__ target, uint64_t n,
                                                             const float* __restrict__ dL_dloss, float inv_n,
                                                             float* __restrict__ dL_dimage) {
    const float g = *dL_dloss * inv_n;
    for (uint64_t k = (uint64_t)blockIdx.x * kL1Threads + threadIdx.x; k < n; k += (uint64_t)gridDim.x * kL1Threads) {
        const float d = image[k] - target[k];
        dL_dimage[k] = d > 0.0f ? g : (d < 0.0f ? -g : 0.0f);
    }
}

}  // namespace

size_t l1_ws_bytes(uint64_t n) { return ((n + kL1Chunk - 1) / kL1Chunk + 1) * sizeof(double); }

int launch_l1_fwd(const float* image, const float* target, uint64_t n, float* loss, void* ws, hipStream_t stream) {
    double* blocks = static_cast<double*>(ws);
    const uint32_t nb = (uint32_t)((n + kL1Chunk - 1) / kL1Chunk);
    if (nb)
        hipLaunchKernelGGL(l1_partial_kernel, dim3(nb), dim3(kL1Threads), 0, stream, image, target, n, blocks);
    hipLaunchKernelGGL(l1_final_kernel, dim3(1), dim3(256), 0, stream, blocks, nb, n ? 1.0 / (double)n : 0.0, loss);
    return hipPeekAtLastError() == hipSuccess ? 0 : -1;
}

int launch_l1_bwd(const float* image, const float* target, uint64_t n, const float* dL_dloss, float* dL_dimage,
                  hipStream_t stream) {
    if (!n) return 0;
    const uint64_t blocks = std::min<uint64_t>((n + kL1Threads - 1) / kL1Threads, 8192);
    hipLaunchKernelGGL(l1_grad_kernel, dim3((unsigned)blocks), dim3(kL1Threads), 0, stream, image, target, n, dL_dloss,
                       (float)(1.0 / (double)n), dL_dimage);
    return hipPeekAtLastError() == hipSuccess ? 0 : -1;
}

}  // namespace isogs
