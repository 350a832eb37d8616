// Scatter-image post-processing of the paper's correction loop (section
// II-C-3 dual interpolation, II-C-4 smoothing): Savitzky-Golay smoothing
// (separable, rows then columns, mirrored edges) and Keys cubic up-sampling
// (a = -0.5, pixel centres aligned, clamped edges), plus the fixed-point
// tally to float conversion.  Small stencil kernels bound by memory traffic
// and launches, rows contiguous across a wave.
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mcx {

constexpr int kMaxSgWindow = 31;

struct SgCoeffs {
    float c[kMaxSgWindow];
};

__device__ __forceinline__ int mirror_index(int i, int n) {
    if (i >= 0 && i < n) return i;
    if (n == 1) return 0;
    const int period = 2 * (n - 1);
    i %= period;
    if (i < 0) i += period;
    return i < n ? i : period - i;
}

// Both passes in one launch, for images that are not smoothed in place.  Two
// launches and a modulo per tap took 17 us on 576 x 800; the bytes take under
// one, so launch and latency bound it (7.2 us now, window 9).  A block makes a kSgX x
// kSgY tile: the input with its halo and the row sums stay in LDS (edges are
// mirrored once per staged value), the sums in the order of savgol_kernel.  The
// window is a template argument, so that a sum's LDS reads are all in flight.
constexpr int kSgX = 64, kSgY = 8;

template <int HALF>
__global__ void __launch_bounds__(256) savgol_tile_kernel(const float *in, float *out, int nx,
                                                          int ny, SgCoeffs co) {
    constexpr int W = kSgX + 2 * HALF, H = kSgY + 2 * HALF;
    __shared__ float s_in[H][W];
    __shared__ float s_row[H][kSgX];
    const int x0 = blockIdx.x * kSgX, y0 = blockIdx.y * kSgY;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    // as much of the tile as the image fills
    const int cols = min(W, nx - x0 + 2 * HALF), rows = min(H, ny - y0 + 2 * HALF);
    for (int r = ty; r < rows; r += 4) {
        const float *src = in + (size_t)mirror_index(y0 + r - HALF, ny) * nx;
        for (int c = tx; c < cols; c += 64) s_in[r][c] = src[mirror_index(x0 + c - HALF, nx)];
    }
    __syncthreads();
    const bool live = x0 + tx < nx;
    if (live)
        for (int r = ty; r < rows; r += 4) {
            float s = 0.0f;
#pragma unroll
            for (int k = 0; k <= 2 * HALF; ++k) s += co.c[k] * s_in[r][tx + k];
            s_row[r][tx] = s;
        }
    __syncthreads();
    if (!live) return;
#pragma unroll
    for (int r = ty; r < kSgY; r += 4) {
        if (y0 + r >= ny) break;
        float s = 0.0f;
#pragma unroll
        for (int k = 0; k <= 2 * HALF; ++k) s += co.c[k] * s_row[r + k][tx];
        out[(size_t)(y0 + r) * nx + x0 + tx] = s;
    }
}

template <int HALF>
static void launch_savgol_tile(const float *in, float *out, int nx, int ny, int half,
                               const SgCoeffs &co, hipStream_t s) {
    if (half != HALF) {
        if constexpr (HALF < kMaxSgWindow / 2) launch_savgol_tile<HALF + 1>(in, out, nx, ny, half, co, s);
        return;
    }
    hipLaunchKernelGGL(savgol_tile_kernel<HALF>, dim3((nx + kSgX - 1) / kSgX, (ny + kSgY - 1) / kSgY),
                       dim3(256), 0, s, in, out, nx, ny, co);
}

// along x when `along_x`, else along y; fp32 sum in window order
__global__ void savgol_kernel(const float *in, float *out, int nx, int ny, int half,
                              SgCoeffs co, int along_x) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= nx || y >= ny) return;
    float s = 0.0f;
    if (along_x) {
        const float *row = in + (size_t)y * nx;
        for (int k = -half; k <= half; ++k) s += co.c[k + half] * row[mirror_index(x + k, nx)];
    } else {
        for (int k = -half; k <= half; ++k)
            s += co.c[k + half] * in[(size_t)mirror_index(y + k, ny) * nx + x];
    }
    out[(size_t)y * nx + x] = s;
}

__device__ __forceinline__ float keys_weight(float t) {
    t = fabsf(t);
    const float a = -0.5f;
    if (t <= 1.0f) return ((a + 2.0f) * t - (a + 3.0f)) * t * t + 1.0f;
    if (t < 2.0f) return ((a * t - 5.0f * a) * t + 8.0f * a) * t - 4.0f * a;
    return 0.0f;
}

// (nx*f) x (ny*f) image from the nx x ny input: separable 4 x 4 cubic
// convolution at input coordinate (i + 0.5)/f - 0.5.  A thread takes one output
// column down `strip` rows: its four column weights are found once, each input
// row is interpolated along x once and kept while output rows use it, and the
// rows' weights are made once per block.  Bound by the stores (a thread per
// output, with its own 20 weights, took 44 us for 2304 x 3200; 10.5 now, 2.8 TB/s).
constexpr int kUpStrip = 16;    // most rows of a strip

__global__ void __launch_bounds__(256) upsample_kernel(const float *in, float *out, int nx, int ny,
                                                       int f, int strip) {
    __shared__ float4 s_w[kUpStrip];
    __shared__ int s_y[kUpStrip];
    const int mx = nx * f, my = ny * f;
    const int oy0 = blockIdx.y * strip;
    const int rows = min(strip, my - oy0);
    auto coord = [f](int o) { return ((float)o + 0.5f) / (float)f - 0.5f; };
    if ((int)threadIdx.x < rows) {
        const float uy = coord(oy0 + threadIdx.x);
        const int y0 = (int)floorf(uy);
        s_y[threadIdx.x] = y0;
        s_w[threadIdx.x] = make_float4(
            keys_weight(uy - (float)(y0 - 1)), keys_weight(uy - (float)y0),
            keys_weight(uy - (float)(y0 + 1)), keys_weight(uy - (float)(y0 + 2)));
    }
    __syncthreads();
    const int ox = blockIdx.x * blockDim.x + threadIdx.x;
    if (ox >= mx) return;
    const float ux = coord(ox);
    const int x0 = (int)floorf(ux);
    float wx[4];
    int xs[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        wx[k] = keys_weight(ux - (float)(x0 - 1 + k));
        xs[k] = min(max(x0 - 1 + k, 0), nx - 1);
    }
    // input row m (clamped) at this column's four pixels, and along x
    auto load = [&](int m, float (&v)[4]) {
        const float *p = in + (size_t)min(max(m, 0), ny - 1) * nx;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = p[xs[k]];
    };
    auto along = [&](const float (&v)[4]) {
        float r = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) r += wx[k] * v[k];
        return r;
    };
    int top = __builtin_amdgcn_readfirstlane(s_y[0]) - 1;   // r0 .. r3 are rows top .. top + 3
    float v0[4], v1[4], v2[4], v3[4], next[4];
    load(top, v0);
    load(top + 1, v1);
    load(top + 2, v2);
    load(top + 3, v3);
    load(top + 4, next);                                    // in flight until it is needed
    float r0 = along(v0), r1 = along(v1), r2 = along(v2), r3 = along(v3);
    for (int t = 0; t < rows; ++t) {
        // the next output row is at most one input row on
        const int y = __builtin_amdgcn_readfirstlane(s_y[t]) - 1;
        if (y != top) {
            top = y;
            r0 = r1;
            r1 = r2;
            r2 = r3;
            r3 = along(next);
            load(top + 4, next);
        }
        const float4 w = s_w[t];
        float acc = 0.0f;
        acc += w.x * r0;
        acc += w.y * r1;
        acc += w.z * r2;
        acc += w.w * r3;
        out[(size_t)(oy0 + t) * mx + ox] = acc;
    }
}

__global__ void tally_to_float_kernel(const long long *in, float *out, uint64_t n, double scale) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = (float)((double)in[i] * scale);
}

hipError_t launch_savgol(const float *in, float *out, float *tmp, int nx, int ny, int window,
                         const float *coeffs, hipStream_t s) {
    SgCoeffs co{};
    for (int i = 0; i < window; ++i) co.c[i] = coeffs[i];
    const uintptr_t a = (uintptr_t)in, b = (uintptr_t)out;
    const size_t bytes = (size_t)nx * ny * sizeof(float);
    if (a + bytes <= b || b + bytes <= a) {
        launch_savgol_tile<0>(in, out, nx, ny, window / 2, co, s);
        return hipGetLastError();
    }
    // in place (or overlapping): rows into tmp, then columns
    const dim3 block(256), grid((nx + 255) / 256, ny);
    hipLaunchKernelGGL(savgol_kernel, grid, block, 0, s, in, tmp, nx, ny, window / 2, co, 1);
    hipLaunchKernelGGL(savgol_kernel, grid, block, 0, s, (const float *)tmp, out, nx, ny,
                       window / 2, co, 0);
    return hipGetLastError();
}

hipError_t launch_upsample(const float *in, float *out, int nx, int ny, int f, hipStream_t s) {
    const int bx = (nx * f + 255) / 256, my = ny * f;
    // strips as long as leave two blocks a compute unit (longer ones reuse more)
    int strip = kUpStrip;
    while (strip > 1 && (int64_t)bx * ((my + strip - 1) / strip) < 512) strip /= 2;
    hipLaunchKernelGGL(upsample_kernel, dim3(bx, (my + strip - 1) / strip), dim3(256), 0, s, in,
                       out, nx, ny, f, strip);
    return hipGetLastError();
}

// out[y][x] = alpha * in[flip_y ? ny-1-y : y][flip_x ? nx-1-x : x] + beta * out[y][x]
// (mirror images of a map, optionally accumulated; out is not read when beta
// is 0): training pairs are augmented with them and predictions averaged
__global__ void flip2d_kernel(const float *in, float *out, int nx, int ny, int fx, int fy,
                              float alpha, float beta) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= nx) return;
    const int sx = fx ? nx - 1 - x : x, sy = fy ? ny - 1 - y : y;
    const size_t o = (size_t)y * nx + x;
    const float v = alpha * in[(size_t)sy * nx + sx];
    out[o] = beta != 0.0f ? v + beta * out[o] : v;
}

hipError_t launch_flip2d(const float *in, float *out, int nx, int ny, int fx, int fy, float alpha,
                         float beta, hipStream_t s) {
    hipLaunchKernelGGL(flip2d_kernel, dim3((nx + 255) / 256, ny), dim3(256), 0, s, in, out, nx,
                       ny, fx, fy, alpha, beta);
    return hipGetLastError();
}

hipError_t launch_tally_to_float(const int64_t *in, float *out, uint64_t n, double scale,
                                 hipStream_t s) {
    uint64_t grid = (n + 255) / 256;
    if (grid > 8192) grid = 8192;
    if (grid == 0) grid = 1;
    hipLaunchKernelGGL(tally_to_float_kernel, dim3((unsigned)grid), dim3(256), 0, s,
                       (const long long *)in, out, n, scale);
    return hipGetLastError();
}

}  // namespace mcx
