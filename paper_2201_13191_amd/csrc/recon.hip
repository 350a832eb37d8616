// Reconstruction side of the iterative scatter correction (section II-E and its
// flowchart): line integrals of the measured intensities, the Feldkamp-Davis-
// Kress filtered backprojection of the projector's circular orbit, a histogram
// for Otsu's threshold, volume to density, and eq. (8),
// c = a - ln(Ip / (Ip + Is)).  All of it is bandwidth-light next to the
// Monte Carlo: the filter is a product with Toeplitz matrices on the fp64
// matrix cores, the backprojection a thread per column of voxels over the angles.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "fp64_math.hpp"

namespace mcx {

struct FdkGeom {
    double R, D;           // source to axis, source to panel
    double pu, pv;         // panel pitch
    int nu, nv, n_ang;
};

// a = -ln(I / I0), I0 per panel pixel (n0 of them, repeated for each projection)
__global__ void line_integrals_kernel(const float *I, uint64_t n, const float *I0, uint64_t n0,
                                      float *a) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        double v = (double)I[i];
        v = v > 1e-30 ? v : 1e-30;
        a[i] = (float)(-log(v / (double)I0[i % n0]));
    }
}

// eq. (8)
__global__ void scatter_correct_kernel(const float *a, const float *ip, const float *is,
                                       uint64_t n, float *c) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double p = (double)ip[i];
        c[i] = (float)((double)a[i] - log(p / (p + (double)is[i])));
    }
}

typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

// The cosine weight of panel column k on the virtual panel through the axis
// (coordinates scaled by s = R / D): R / sqrt(R^2 + a^2 + b^2).
__device__ __forceinline__ double cosine_weight(const FdkGeom &g, double s, int k, double b2) {
    const double a = (-(double)g.nu * g.pu / 2 + (k + 0.5) * g.pu) * s;
    return g.R * fast_rsqrt(g.R * g.R + a * a + b2);
}

__device__ __forceinline__ double row_height2(const FdkGeom &g, double s, int r) {
    const double b = (-(double)g.nv * g.pv / 2 + (r + 0.5) * g.pv) * s;
    return b * b;
}

// The discrete Ram-Lak filter of the virtual pitch t: h(0) = 1/(4 t^2),
// h(odd d) = -1/(d pi t)^2, h(even d) = 0, times t.  One block per panel row,
// the weighted row in LDS: for rows wider than one block of the matrix form
// below that are filtered in place (it reads a whole row before it writes any
// of it), and for few and short rows (launch_fdk).
__global__ void fdk_filter_row_kernel(const float *proj, FdkGeom g, float *q) {
    extern __shared__ double row[];
    const int r = blockIdx.x % g.nv, i = blockIdx.x / g.nv;
    const double s = g.R / g.D, t = g.pu * s;
    const double b2 = row_height2(g, s, r);
    const float *src = proj + ((size_t)i * g.nv + r) * g.nu;
    for (int k = threadIdx.x; k < g.nu; k += blockDim.x)
        row[k] = (double)src[k] * cosine_weight(g, s, k, b2);
    __syncthreads();
    const double pi = 3.141592653589793;
    for (int j = threadIdx.x; j < g.nu; j += blockDim.x) {
        double acc = row[j] * (1.0 / (4.0 * t * t));
        // odd offsets: j - k = +-1, +-3, ...
        for (int d = 1; d < g.nu; d += 2) {
            const double w = -1.0 / ((d * pi * t) * (d * pi * t));
            double x = 0.0;
            if (j - d >= 0) x += row[j - d];
            if (j + d < g.nu) x += row[j + d];
            acc += w * x;
        }
        q[((size_t)i * g.nv + r) * g.nu + j] = (float)(acc * t);
    }
}

// The same filter as matrix products.  Apart from its centre tap it couples
// even columns only to odd ones and odd only to even, so with columns in
// pairs (2 jj, 2 jj + 1) the two halves of the output are
//     Q_even[row][jj] = sum_kk W_odd [row][kk] T[jj - kk - 1]
//     Q_odd [row][jj] = sum_kk W_even[row][kk] T[jj - kk],  T[m] = h(2 m + 1):
// Toeplitz matrices of half the row's width, on v_mfma_f64_16x16x4_f64.  What
// bounds it is that instruction's rate (nu / 2 fp64 multiply-adds a pixel,
// 0.6 ms of them at 360 x 512^2 against 0.16 ms for the bytes); the row form
// spent its time on an fp64 division per pixel and tap.  A block takes
// 32 * WR rows and 16 * NT * WC column pairs, each of its 4 waves 32 rows by
// 16 * NT pairs of both halves, so every weighted value is made once for rows
// of up to 512 pixels and read from LDS 2 * NT times (17.2 -> 1.76 ms at
// 360 x 512^2, 188 -> 20 us at 180 x 128^2; 1.2 ms with the registers held to
// two blocks a compute unit); the reduction runs over
// chunks of 32 column pairs, whose weighted inputs and the NT * WC * 16 + 32
// taps that the chunk meets are staged in LDS.  Sums are fp64 throughout.
constexpr int kFltPairs = 32;      // column pairs per chunk

template <int WR, int WC, int NT>
__global__ void __launch_bounds__(256, 2) fdk_filter_kernel(const float *proj, FdkGeom g,
                                                         int rows, float *q) {
    static_assert(WR * WC == 4, "four waves");
    constexpr int TR = 32 * WR;              // rows of a block
    constexpr int RS = 32 * WR + 16;         // doubles between kk of a staged half: the two kk
                                             // that 32 lanes read fall on different banks
    constexpr int TP = 16 * NT * WC;         // column pairs of a block
    constexpr int kTaps = TP + kFltPairs;    // jj - kk - 1 of a chunk: -kFltPairs .. TP - 1
    __shared__ double s_in[2][kFltPairs][RS];   // [column parity][kk][row]
    __shared__ double s_tap[kTaps];
    __shared__ double s_b2[TR];                 // squared height of each row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave % WR, wc = wave / WR;
    const int row0 = (int)blockIdx.x * TR;
    const int jj0 = blockIdx.y * TP;
    const double s = g.R / g.D, t = g.pu * s;
    const double pi = 3.141592653589793;
    const int pairs = (g.nu + 1) / 2;
    const int lr = lane & 15, lk = lane >> 4;
    f64x4 acc[2][2][NT];                     // [output parity][row half][tile]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[h][i][n] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (threadIdx.x < TR)
        s_b2[threadIdx.x] = row_height2(g, s, (int)((uint32_t)(row0 + threadIdx.x) % (uint32_t)g.nv));
    __syncthreads();
    for (int kk0 = 0; kk0 < pairs; kk0 += kFltPairs) {
        // weighted inputs: 64 consecutive columns per row, one row per wave
        // and trip; columns past the row's end are zero
        const int k = 2 * kk0 + lane;
#pragma unroll 4
        for (int rr = wave; rr < TR; rr += 4) {
            const int row = row0 + rr;
            double v = 0.0;
            if (row < rows && k < g.nu)
                v = (double)proj[(size_t)row * g.nu + k] *
                    cosine_weight(g, s, k, s_b2[rr]);
            s_in[lane & 1][lane >> 1][rr] = v;
        }
        for (int m = threadIdx.x; m < kTaps; m += 256) {
            // T[jj - kk - 1] at m = jj - jj0 - (kk - kk0) + kFltPairs - 1
            const int d = 2 * (m + jj0 - kk0 - kFltPairs) + 1;
            s_tap[m] = -1.0 / ((d * pi * t) * (d * pi * t));
        }
        __syncthreads();
#pragma unroll 2
        for (int k4 = 0; k4 < kFltPairs; k4 += 4) {
            double a[2][2], b[2][NT];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i) a[h][i] = s_in[1 - h][k4 + lk][wr * 32 + i * 16 + lr];
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int m = (wc * NT + n) * 16 + lr - (k4 + lk) + kFltPairs - 1;
                b[0][n] = s_tap[m];
                b[1][n] = s_tap[m + 1];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[h][i][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[h][i], b[h][n],
                                                                             acc[h][i][n], 0, 0, 0);
        }
        __syncthreads();
    }
    // element e of a 16 x 16 tile is row 4 e + lane / 16, column lane % 16; the
    // centre tap is added here
    const double centre = 1.0 / (4.0 * t * t);
    const bool pair_ok = (g.nu & 1) == 0 && ((uintptr_t)q & 7) == 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int rr = wr * 32 + i * 16 + 4 * e + lk;
            const int row = row0 + rr;
            if (row >= rows) continue;
            const double b2 = s_b2[rr];
            const float *src = proj + (size_t)row * g.nu;
            float *dst = q + (size_t)row * g.nu;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int j = 2 * (jj0 + (wc * NT + n) * 16 + lr);
                float v[2] = {0.0f, 0.0f};
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (j + h < g.nu)
                        v[h] = (float)((acc[h][i][n][e] + (double)src[j + h] *
                                        cosine_weight(g, s, j + h, b2) * centre) * t);
                if (pair_ok) {
                    if (j < g.nu) *(float2 *)(dst + j) = make_float2(v[0], v[1]);
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (j + h < g.nu) dst[j + h] = v[h];
                }
            }
        }
}

// f = 1/2 (2 pi / n) sum_i R^2 / L^2 q_i(a, b), the filtered projections read
// by bilinear interpolation between pixel centres (zero outside the panel).
// fp64 instructions bound it, with the L1's gathers next: one thread per voxel
// and two divisions, a floor and the source-frame coordinates in fp64 for
// each of them took 30.3 ms at 256^3 x 360.  A thread now takes NZ voxels of
// one (x, y) column: the distance, its reciprocal, the column's u and weights
// are found once per angle, the panel row is linear in z, and each voxel costs
// two 8-byte gathers and some twenty fp64 operations (23 vector instructions a
// voxel and angle over all, the vector units 54 % busy): 6.5 ms at 256^3 x 360.
// All 2 NZ gathers of an angle are in flight before the first is used (used
// one voxel at a time they took 8.1 ms).  Lanes run along x, so that a wave's
// gathers fall on a few lines.  Small volumes, whose columns
// alone do not fill the chip, split the angles over the AS waves of a block
// (angles w, w + AS, ...; the sums added in LDS in a fixed order).  The columns'
// pieces are dealt to the lanes without gaps between planes: a block's share of every
// plane of its own left most lanes idle where planes are small (2^20 x 1 x 1, 60
// angles: 15.4 ms, 0.12 now; 65536 x 4 x 4 0.97 and 0.12).
template <int NZ, int AS>
__global__ void __launch_bounds__(256) fdk_backproject_kernel(const float *q, FdkGeom g, int nx,
                                                              int ny, int nz, double h,
                                                              float *vol) {
    extern __shared__ double cs[];   // [2 * n_ang]; then the partial sums of AS > 1
    for (int i = threadIdx.x; i < g.n_ang; i += blockDim.x) {
        double sb, cb;
        sincos(2.0 * 3.141592653589793 * i / g.n_ang, &sb, &cb);
        cs[2 * i] = cb;
        cs[2 * i + 1] = sb;
    }
    __syncthreads();
    constexpr int kCols = 256 / AS;
    const int col = AS > 1 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    const int part = AS > 1 ? (int)(threadIdx.x >> 6) : 0;
    static_assert(AS == 1 || AS == 4, "a wave per part");
    // pieces of NZ voxels of a column, (z, y, x) with x fastest, 2^31 at most; blocks go on
    // from one plane of pieces to the next, and surplus lanes go along with the last piece
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const uint32_t pieces = plane * (uint32_t)((nz + NZ - 1) / NZ);
    const uint32_t own = blockIdx.x * (uint32_t)kCols + (uint32_t)col;
    const bool live = own < pieces;
    const uint32_t piece = live ? own : pieces - 1;
    const uint32_t zi = piece / plane, xy = piece - zi * plane;
    const int z0 = (int)zi * NZ;
    const int ix = (int)(xy % (uint32_t)nx), iy = (int)(xy / (uint32_t)nx);
    const double X = (ix + 0.5) * h - nx * h / 2, Y = (iy + 0.5) * h - ny * h / 2;
    const double Z0 = (z0 + 0.5) * h - nz * h / 2;
    const double s = g.R / g.D;
    const double ku = g.R / (s * g.pu), kv = g.R / (s * g.pv);
    const double ou = 0.5 * g.nu - 0.5, ov = 0.5 * g.nv - 0.5;
    const uint32_t row_bytes = (uint32_t)g.nu * 4u;
    double f[NZ];
#pragma unroll
    for (int n = 0; n < NZ; ++n) f[n] = 0.0;
    for (int i = part; i < g.n_ang; i += AS) {
        const double cb = cs[2 * i], sb = cs[2 * i + 1];
        const double rl = fast_rcp(g.R - (X * cb + Y * sb));
        const double fu = __builtin_fma(ku * (Y * cb - X * sb), rl, ou);
        const double dv = kv * rl * h;                   // panel rows per voxel in z
        const double fv0 = __builtin_fma(kv * rl, Z0, ov);
        const double fv1 = __builtin_fma((double)(NZ - 1), dv, fv0);
        const double w2 = (g.R * rl) * (g.R * rl);
        // The 2 x 2 pixels of the NZ voxels, all in flight at once.  A lane off
        // the panel takes zeros for the pixels that are not there (its
        // coordinates clamped to just outside, which also keeps the integer
        // conversions in range).
        const char *qi = (const char *)(q + (size_t)i * g.nv * g.nu);
        const double fuc = fmin(fmax(fu, -2.0), g.nu + 1.0);
        const double u0 = floor(fuc);
        const double wu = fuc - u0, wu1 = 1.0 - wu;
        const int iu = (int)u0;
        double wv[NZ];
        float2 lo[NZ], hi[NZ];
        // every lane's pixels on the panel (fv grows with n; rounding cannot
        // take its last value past the margin)
        const bool in = fu >= 0.0 && fu < g.nu - 1.0 && fv0 >= 0.0 && fv1 < g.nv - 1.001;
        if (__all(in)) {
#pragma unroll
            for (int n = 0; n < NZ; ++n) {
                const double fv = __builtin_fma((double)n, dv, fv0);
                const double v0 = floor(fv);
                wv[n] = fv - v0;
                const uint32_t off = (__umul24((uint32_t)(int)v0, (uint32_t)g.nu) + (uint32_t)iu) << 2;
                __builtin_memcpy(&lo[n], qi + off, 8);              // 4-byte aligned pairs
                __builtin_memcpy(&hi[n], qi + row_bytes + off, 8);
            }
        } else {
            const bool ul = iu >= 0 && iu < g.nu, ur = iu + 1 >= 0 && iu + 1 < g.nu;
            const float *qf = (const float *)qi;
#pragma unroll
            for (int n = 0; n < NZ; ++n) {
                const double fv = fmin(fmax(__builtin_fma((double)n, dv, fv0), -2.0), g.nv + 1.0);
                const double v0 = floor(fv);
                wv[n] = fv - v0;
                const int iv = (int)v0;
                const bool vl = iv >= 0 && iv < g.nv, vr = iv + 1 >= 0 && iv + 1 < g.nv;
                const int at = iv * g.nu + iu;
                lo[n].x = vl && ul ? qf[at] : 0.0f;
                lo[n].y = vl && ur ? qf[at + 1] : 0.0f;
                hi[n].x = vr && ul ? qf[at + g.nu] : 0.0f;
                hi[n].y = vr && ur ? qf[at + g.nu + 1] : 0.0f;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NZ; ++n) {
            const double t0 = __builtin_fma((double)lo[n].y, wu, (double)lo[n].x * wu1);
            const double t1 = __builtin_fma((double)hi[n].y, wu, (double)hi[n].x * wu1);
            f[n] = __builtin_fma(w2, __builtin_fma(t1, wv[n], t0 * (1.0 - wv[n])), f[n]);
        }
    }
    if constexpr (AS > 1) {
        double *parts = cs;                              // [AS - 1][NZ][64], over the angles
        __syncthreads();
        if (part > 0) {
#pragma unroll
            for (int n = 0; n < NZ; ++n) parts[((part - 1) * NZ + n) * 64 + col] = f[n];
        }
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int p = 0; p < AS - 1; ++p)
#pragma unroll
            for (int n = 0; n < NZ; ++n) f[n] += parts[(p * NZ + n) * 64 + col];
    }
    if (!live) return;
    const double scale = 0.5 * (2.0 * 3.141592653589793 / g.n_ang);
#pragma unroll
    for (int n = 0; n < NZ; ++n)
        if (z0 + n < nz) vol[(size_t)(z0 + n) * plane + xy] = (float)(scale * f[n]);
}

// counts of x in [lo, hi) in `bins` equal bins, bin floor((x - lo) / (hi - lo) * bins)
__global__ void histogram_kernel(const float *x, uint64_t n, double lo, double hi, int bins,
                                 unsigned int *hist) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double k = floor(((double)x[i] - lo) / (hi - lo) * bins);
        if (k >= 0.0 && k < (double)bins) atomicAdd(hist + (int)k, 1u);
    }
}

__global__ void zero_u32_kernel(unsigned int *p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

// voxels with mu >= threshold: `material` with density mu / (0.1 mu/rho) rounded
// to multiples of step (half to even); the others air
__global__ void to_density_kernel(const float *mu, uint64_t n, double threshold, double mu_rho,
                                  int material, double air_rho, double step, uint8_t *ids,
                                  float *rho) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double m = (double)mu[i];
        const bool obj = m >= threshold;
        ids[i] = obj ? (uint8_t)material : (uint8_t)0;
        rho[i] = (float)(obj ? __builtin_rint(m / (0.1 * mu_rho) / step) * step : air_rho);
    }
}

static unsigned grid_for(uint64_t n) {
    uint64_t g = (n + 255) / 256;
    return (unsigned)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

hipError_t launch_line_integrals(const float *I, uint64_t n, const float *I0, uint64_t n0,
                                 float *a, hipStream_t s) {
    hipLaunchKernelGGL(line_integrals_kernel, dim3(grid_for(n)), dim3(256), 0, s, I, n, I0, n0, a);
    return hipGetLastError();
}

hipError_t launch_scatter_correct(const float *a, const float *ip, const float *is, uint64_t n,
                                  float *c, hipStream_t s) {
    hipLaunchKernelGGL(scatter_correct_kernel, dim3(grid_for(n)), dim3(256), 0, s, a, ip, is, n, c);
    return hipGetLastError();
}

hipError_t launch_fdk(const float *proj, double R, double D, double pu, double pv, int nu, int nv,
                      int n_ang, float *q, int nx, int ny, int nz, double h, float *vol,
                      hipStream_t s) {
    const FdkGeom g{R, D, pu, pv, nu, nv, n_ang};
    const int rows = n_ang * nv;      // below 2^26 (n_ang <= 4096, nv <= 16384)
    const int pairs = (nu + 1) / 2;
    auto filter = [&](auto kernel, int block_rows, int block_pairs) {
        const dim3 grid((unsigned)((rows + block_rows - 1) / block_rows),
                        (unsigned)((pairs + block_pairs - 1) / block_pairs));
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, proj, g, rows, q);
    };
    const bool in_place = (const float *)q == proj;
    // The block's width follows the row's (16-pair tiles past the row are
    // computed for nothing), with as few rows as four waves then need: short
    // panels have few blocks (180 x 128^2: 64-row blocks, 1.4 a compute unit,
    // took 28.8 us, 32-row ones 20 us).  Rows above 512 pixels take several
    // blocks, which read what others would overwrite in place.
    //   Few rows leave a block's own length to wait for: then its columns are shared out
    // over blocks of 32 x 64 while these run two to a compute unit (with the
    // backprojection of one voxel, 66 rows of 130 pixels 30.0 and 15.4 us, 3840 of 192
    // 40.8 and 25.2, 7680 of 256 45.1 and 44.0, 16384 of 192 71.5 and 70.3, 16384 of 512 143 and
    // 163), or, where that cannot be or rows are short, a block takes a row (164 rows of 80
    // pixels 10.9 and 12.6 us in 32 x 64, 306 of 100 14.2 and 13.4; in place, 924 rows of
    // 130 20.6 and 33.3 in 64 x 192, 387 of 256 25.2 and 25.5).
    const bool row_form = pairs > 48 && !in_place ? false
                          : pairs <= 48           ? rows <= 256
                          : pairs <= 64           ? false
                          : pairs <= 96           ? rows <= 1024
                          : pairs <= 128          ? rows <= 400
                                                  : pairs > 256;
    const int64_t narrow = (int64_t)((rows + 31) / 32) * ((pairs + 63) / 64);
    if (row_form)
        hipLaunchKernelGGL(fdk_filter_row_kernel, dim3((unsigned)rows), dim3(256),
                           (size_t)nu * sizeof(double), s, proj, g, q);
    else if (narrow < 512 && (pairs <= 64 || !in_place))
        filter(fdk_filter_kernel<1, 4, 1>, 32, 64);
    else if (pairs <= 32)
        filter(fdk_filter_kernel<2, 2, 1>, 64, 32);
    else if (pairs <= 64)
        filter(fdk_filter_kernel<1, 4, 1>, 32, 64);
    else if (pairs <= 96)
        filter(fdk_filter_kernel<2, 2, 3>, 64, 96);
    else if (pairs <= 128)
        filter(fdk_filter_kernel<1, 4, 2>, 32, 128);
    else if (pairs <= 192)
        filter(fdk_filter_kernel<1, 4, 3>, 32, 192);
    else
        filter(fdk_filter_kernel<1, 4, 4>, 32, 256);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t plane = (int64_t)nx * ny;
    const size_t lds = (size_t)2 * n_ang * sizeof(double);
    auto back = [&](auto kernel, int cols, int zs, size_t bytes) {
        const dim3 grid((unsigned)((plane * ((nz + zs - 1) / zs) + cols - 1) / cols));
        hipLaunchKernelGGL(kernel, grid, dim3(256), bytes, s, (const float *)q, g, nx, ny, nz, h,
                           vol);
    };
    // 8 voxels a thread once that leaves two waves a SIMD; below, 4 and the
    // angles split (64^3 x 180: 360 us with a thread a voxel, 68 us).  Fewer where the
    // volume has fewer (2048^2 x 1, 60 angles: 1.69 ms with 8, 0.39 with one)
    if (plane * nz >= (int64_t)8 * 64 * 2048) {
        if (nz > 4)
            back(fdk_backproject_kernel<8, 1>, 256, 8, lds);
        else if (nz > 2)
            back(fdk_backproject_kernel<4, 1>, 256, 4, lds);
        else if (nz > 1)
            back(fdk_backproject_kernel<2, 1>, 256, 2, lds);
        else
            back(fdk_backproject_kernel<1, 1>, 256, 1, lds);
    } else {
        back(fdk_backproject_kernel<4, 4>, 64, 4,
             lds > 3 * 4 * 64 * sizeof(double) ? lds : 3 * 4 * 64 * sizeof(double));
    }
    return hipGetLastError();
}

hipError_t launch_histogram(const float *x, uint64_t n, double lo, double hi, int bins,
                            unsigned int *hist, hipStream_t s) {
    hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((bins + 255) / 256)), dim3(256), 0, s,
                       hist, bins);
    hipLaunchKernelGGL(histogram_kernel, dim3(grid_for(n)), dim3(256), 0, s, x, n, lo, hi, bins,
                       hist);
    return hipGetLastError();
}

hipError_t launch_to_density(const float *mu, uint64_t n, double threshold, double mu_rho,
                             int material, double air_rho, double step, uint8_t *ids, float *rho,
                             hipStream_t s) {
    hipLaunchKernelGGL(to_density_kernel, dim3(grid_for(n)), dim3(256), 0, s, mu, n, threshold,
                       mu_rho, material, air_rho, step, ids, rho);
    return hipGetLastError();
}

}  // namespace mcx
