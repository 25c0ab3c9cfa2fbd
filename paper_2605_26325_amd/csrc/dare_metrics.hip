// Image similarity of a reslice against the acquired frame at the same pose: the evaluation of
// Sec. 3 ("Quantitative image similarity": normalised cross-correlation and the structural
// similarity index between resliced images and their ground truth).
//
// The paper names the measures only; the readings are the standard ones.  NCC is zero-mean and
// taken over the pixels the reslice assigns (finite); SSIM is Wang et al.'s index with an 11 x 11
// Gaussian window (sigma 1.5, weights summing to 1), K1 = 0.01, K2 = 0.03, L = 255, averaged over
// the pixels whose whole window lies inside the image and is assigned in the reslice.
//
// The window is a product of two 11-tap Gaussians, so its five sums (a, b, aa, bb, ab) are taken
// along the rows and then down the columns: 22 taps a pixel instead of 121.  A workgroup takes
// tiles of 32 x 16 pixels in turn: the tile and its 5-pixel border go to LDS (pixels that are not
// finite or outside the image as NaN, which marks every window that holds one), the row sums to
// LDS in FP64, and each thread sums two pixels of a column and adds its tile's contributions to the
// eight totals in registers.  Workgroups write their totals to a workspace row each, and one
// workgroup adds the rows, in a fixed order, and finishes NCC from the sums (one pass: FP64 keeps
// the cancellation far below the comparison's tolerance at these sizes).
//
// Bound: latency, a few dependent phases of two tiles per CU.  512 x 512: 11.0 us and 3.8 us for
// the total, against 47.8 us and 11.4 us with 121 taps per pixel from global memory and a total of
// one sum after another.
#include <math.h>
#include <string.h>

#include <algorithm>

#include "dare_host.h"

#pragma clang fp contract(off)

using namespace dare;

namespace {

constexpr int kWin = 11;
constexpr int kHalf = kWin / 2;
constexpr int kSums = 8;                 // n, sum a, sum b, sum a^2, sum b^2, sum ab, sum ssim, n ssim
constexpr int kMaxGroups = 1024;

constexpr int kTileX = 32, kTileY = 16;
constexpr int kBoxX = kTileX + kWin - 1, kBoxY = kTileY + kWin - 1;

struct Window {
    double g[kWin];                      // one axis, summing to 1
};

// An assigned pixel's part of the sums for NCC.
__device__ __forceinline__ void add_pixel(double (&acc)[kSums], float a, float b) {
    const double da = (double)a, db = (double)b;
    acc[0] += 1.0;
    acc[1] += da;
    acc[2] += db;
    acc[3] += da * da;
    acc[4] += db * db;
    acc[5] += da * db;
}

// A workgroup's totals into its row of the workspace.
__device__ __forceinline__ void group_totals(const double (&acc)[kSums], double (&red)[4][kSums], double* partials) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
        double v = acc[k];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        if ((tid & 63) == 0) red[tid >> 6][k] = v;
    }
    __syncthreads();
    if (tid < kSums) partials[(size_t)blockIdx.x * kSums + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

__global__ void __launch_bounds__(256) k_compare(const float* __restrict__ img, const uint8_t* __restrict__ frm,
                                                 int w, int h, int tiles_x, int64_t tiles, Window win,
                                                 double* __restrict__ partials) {
    __shared__ float a[kBoxY][kBoxX], b[kBoxY][kBoxX];
    __shared__ double rows[5][kBoxY][kTileX];
    __shared__ double red[4][kSums];
    const int tid = threadIdx.x;
    double acc[kSums] = {0, 0, 0, 0, 0, 0, 0, 0};
    const double c1 = (0.01 * 255.0) * (0.01 * 255.0), c2 = (0.03 * 255.0) * (0.03 * 255.0);
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int ty = (int)(t / tiles_x), tx = (int)(t - (int64_t)ty * tiles_x);
        const int x0 = tx * kTileX - kHalf, y0 = ty * kTileY - kHalf;   // the box's first pixel
        for (int e = tid; e < kBoxY * kBoxX; e += 256) {
            const int r = e / kBoxX, c = e - r * kBoxX, x = x0 + c, y = y0 + r;
            float va = __builtin_nanf(""), vb = 0.0f;
            if (x >= 0 && x < w && y >= 0 && y < h) {
                const int64_t p = (int64_t)y * w + x;
                const float v = img[p];
                va = isfinite(v) ? v : va;
                vb = (float)frm[p];
            }
            a[r][c] = va;
            b[r][c] = vb;
        }
        __syncthreads();
        for (int e = tid; e < kBoxY * kTileX; e += 256) {
            const int r = e / kTileX, c = e % kTileX;
            double sa = 0.0, sb = 0.0, saa = 0.0, sbb = 0.0, sab = 0.0;
#pragma unroll
            for (int k = 0; k < kWin; ++k) {
                const double xa = (double)a[r][c + k], xb = (double)b[r][c + k];
                const double ga = win.g[k] * xa, gb = win.g[k] * xb;
                sa += ga;
                sb += gb;
                saa = __builtin_fma(ga, xa, saa);
                sbb = __builtin_fma(gb, xb, sbb);
                sab = __builtin_fma(ga, xb, sab);
            }
            rows[0][r][c] = sa;
            rows[1][r][c] = sb;
            rows[2][r][c] = saa;
            rows[3][r][c] = sbb;
            rows[4][r][c] = sab;
        }
        __syncthreads();
        const int c = tid % kTileX, r0 = 2 * (tid / kTileX);   // two pixels, (c, r0) and (c, r0 + 1)
        double s[2][5] = {{0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}};
#pragma unroll
        for (int k = 0; k <= kWin; ++k)
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const double v = rows[q][r0 + k][c];
                if (k < kWin) s[0][q] = __builtin_fma(win.g[k < kWin ? k : 0], v, s[0][q]);
                if (k > 0) s[1][q] = __builtin_fma(win.g[k > 0 ? k - 1 : 0], v, s[1][q]);
            }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float fa = a[r0 + u + kHalf][c + kHalf];
            if (fa == fa) add_pixel(acc, fa, b[r0 + u + kHalf][c + kHalf]);
            const double ma = s[u][0], mb = s[u][1];
            if (ma == ma) {   // every pixel of the window assigned and inside the image
                const double va = s[u][2] - ma * ma, vb = s[u][3] - mb * mb, cab = s[u][4] - ma * mb;
                acc[6] += ((2.0 * ma * mb + c1) * (2.0 * cab + c2)) / ((ma * ma + mb * mb + c1) * (va + vb + c2));
                acc[7] += 1.0;
            }
        }
        __syncthreads();
    }
    group_totals(acc, red, partials);
}

// An image too narrow or too flat for a window: the six sums of NCC alone, pixel by pixel (1 x 100000
// pixels: the call 24 us, 70 in tiles of 32 x 16, 40 with 121 taps per pixel that all stop early).
__global__ void __launch_bounds__(256) k_compare_pixels(const float* __restrict__ img, const uint8_t* __restrict__ frm,
                                                        int64_t n, double* __restrict__ partials) {
    __shared__ double red[4][kSums];
    double acc[kSums] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
        const float v = img[p];
        if (isfinite(v)) add_pixel(acc, v, (float)frm[p]);
    }
    group_totals(acc, red, partials);
}

// The groups' rows added up (thread (row, k) of 32 x 8 takes every 32nd row of total k) and the four
// results from them, to device memory or to the caller's pinned host memory.
__global__ void __launch_bounds__(256) k_compare_total(const double* __restrict__ partials, int groups,
                                                       double* __restrict__ out) {
    __shared__ double red[4][kSums];
    const int k = threadIdx.x % kSums;
    double v = 0.0;
#pragma unroll 8
    for (int b = threadIdx.x / kSums; b < groups; b += 256 / kSums) v += partials[(size_t)b * kSums + k];
#pragma unroll
    for (int off = 32; off >= kSums; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) < kSums) red[threadIdx.x >> 6][k] = v;
    __syncthreads();
    if (threadIdx.x != 0) return;
    double tot[kSums];
#pragma unroll
    for (int t = 0; t < kSums; ++t) tot[t] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
    const double n = tot[0];
    double ncc = __builtin_nan("");
    if (n >= 2.0) {
        const double saa = tot[3] - tot[1] * tot[1] / n, sbb = tot[4] - tot[2] * tot[2] / n;
        const double sab = tot[5] - tot[1] * tot[2] / n;
        if (saa > 0.0 && sbb > 0.0) ncc = sab / sqrt(saa * sbb);
    }
    out[0] = ncc;
    out[1] = tot[7] > 0.0 ? tot[6] / tot[7] : __builtin_nan("");
    out[2] = n;
    out[3] = tot[7];
}

// Pinned host memory that the GPU addresses as the host does: the total kernel writes it itself.
bool pinned_host(const void* p) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {   // pageable
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeHost && at.devicePointer == p && (uintptr_t)p % alignof(double) == 0;
}

}  // namespace

extern "C" {

uint64_t dare_compare_workspace_bytes(void) { return (uint64_t)(kMaxGroups + 1) * kSums * sizeof(double); }

dare_status dare_compare_to_frame(const float* image_dev, const uint8_t* frame_dev, int32_t w, int32_t h,
                                  void* workspace_dev, uint64_t workspace_bytes, double* out_host, void* stream_) {
    if (!image_dev || !frame_dev || !workspace_dev || !out_host || w <= 0 || h <= 0) return DARE_ERR_INVALID_ARG;
    if ((int64_t)w * h > (int64_t)1 << 30 || workspace_bytes < dare_compare_workspace_bytes())
        return DARE_ERR_INVALID_ARG;
    if (((uintptr_t)workspace_dev % alignof(double)) != 0) return DARE_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    Window win;
    double s = 0.0;
    for (int x = 0; x < kWin; ++x) {
        const double dx = x - kHalf;
        win.g[x] = exp(-(dx * dx) / (2.0 * 1.5 * 1.5));
        s += win.g[x];
    }
    for (double& g : win.g) g /= s;
    const int tiles_x = (w + kTileX - 1) / kTileX;
    const int64_t tiles = (int64_t)tiles_x * ((h + kTileY - 1) / kTileY);
    const bool windows = w >= kWin && h >= kWin;
    const int64_t pixels = (int64_t)w * h;
    const int groups = (int)std::min<int64_t>(windows ? tiles : (pixels + 255) / 256, kMaxGroups);
    double* partials = (double*)workspace_dev;
    if (windows) {
        hipLaunchKernelGGL(k_compare, dim3(groups), dim3(256), 0, stream, image_dev, frame_dev, w, h, tiles_x, tiles,
                           win, partials);
    } else {
        hipLaunchKernelGGL(k_compare_pixels, dim3(groups), dim3(256), 0, stream, image_dev, frame_dev, pixels, partials);
    }
    // results into pinned memory need no copy command behind the kernels, a fifth of the call
    // (512 x 512: 23 us into pinned memory, 32 into any other)
    const bool direct = pinned_host(out_host);
    double* const out = direct ? out_host : partials + (size_t)kMaxGroups * kSums;
    hipLaunchKernelGGL(k_compare_total, dim3(1), dim3(256), 0, stream, partials, groups, out);
    double res[4];
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !direct) e = hipMemcpyAsync(res, out, sizeof(res), hipMemcpyDeviceToHost, stream);
    const hipError_t done = hipStreamSynchronize(stream);   // whatever went before: nothing writes once this returns
    if (e != hipSuccess || done != hipSuccess) return DARE_ERR_HIP;
    if (!direct) memcpy(out_host, res, sizeof(res));
    return DARE_OK;
}

}  // extern "C"
