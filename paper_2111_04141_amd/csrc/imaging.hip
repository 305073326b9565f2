// Imaging chain: origin shift, inverse FFT and the Correction Step.
//
// The grids have their origin at the centre (cell n/2 is u = 0).  For even
// sizes the centred unnormalised inverse transform
//     I[y, x] = sum_k G[kv, ku] exp(+j2pi ((ku - nx/2)(x - nx/2)/nx + ...))
// is (-1)^(x + y + nx/2 + ny/2) times the plain inverse FFT of
// (-1)^(ku + kv) G.
//  * Power-of-two sides (own_fft): two kernels of this file.  fft_rows_kernel
//    transforms every row (its loads carry the signs), fft_columns_kernel
//    every column and applies the signs, the correctors and the crop as it
//    stores: the grid crosses HBM twice each way.  The platform library's 2-D
//    transform alone takes two row passes and two transpositions.  4 x 2048 x
//    2048: rows 51 us (near a device copy's rate), columns 63 us, 124 us in all;
//    with the library's transform between two kernels of its own 280 us.
//  * Other even sides: the platform library's batched C2C transform, in place in
//    the scratch, between a kernel that copies the grid with its signs and one
//    for the other signs, correctors and crop.  (The library may overwrite its
//    input even out of place, and the grid is read only.)
// The Correction Step (Section 2.4.5, corrector h_co;
// Section 2.4.4 for Hybrid Gridding, with the pruning kernel's corrector
// along v) multiplies by separable corrector vectors, computed on the device
// from the kernel tables (corrector_kernel):
//     h(l) = 1 / ( (1/P) sum_e T[e] cos(2pi ((e - E/2)/beta) l) sinc(l/beta) ),
// l = (i - n/2)/n, for a symmetric table T of E + 1 values whose entry e lies
// (e - E/2)/beta cells from the centre, averaged over its P sub-cell phases.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <cmath>
#include <new>
#include <string>
#include <type_traits>

#include "fft.h"
#include "internal.h"

struct mg_imager {
    hipfftHandle plan = 0;
    int32_t npol = 0, nx = 0, ny = 0;
};

struct mg_wstack_imager {
    hipfftHandle plan = 0;
    int32_t npol = 0, layers = 0, nx = 0, ny = 0;
};

namespace mg {
namespace {

__global__ __launch_bounds__(256) void corrector_kernel(int32_t n, int32_t beta, int32_t ntab,
                                                        int32_t phases, int32_t nn_sinc,
                                                        const float *__restrict__ table,
                                                        float *__restrict__ corr) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double l = (double)(i - n / 2) / (double)n;
    const double half = 0.5 * (double)(ntab - 1);
    const double two_pi = 6.283185307179586476925286766559;
    double s = 0.0;
    for (int e = 0; e < ntab; ++e)
        s += (double)table[e] * cos(two_pi * (((double)e - half) / (double)beta) * l);
    s /= (double)phases;
    if (nn_sinc) {
        const double a = 3.14159265358979323846264338328 * l / (double)beta;
        s *= (a == 0.0) ? 1.0 : sin(a) / a;
    }
    corr[i] = (float)(1.0 / s);
}

// Each row of `in` (nrows rows of N points, row r of index parity r) times
// (-1)^(x + r), transformed, to the same row of `out`.  256 threads or one row.
template <int LOGN>
__global__ __launch_bounds__(LOGN > 12 ? 512 : 256) void fft_rows_kernel(
    const float2 *in, float2 *out, int64_t nrows) {
    constexpr int N = 1 << LOGN, T = N / 16;
    constexpr int THREADS = LOGN > 12 ? 512 : 256, ROWS = THREADS / T;
    __shared__ float2 s[ROWS][fft_points(LOGN)];
    const int t = threadIdx.x % T, rr = threadIdx.x / T;
    const int64_t row = (int64_t)blockIdx.x * ROWS + rr;
    const bool on = row < nrows;
    float2 v[16];
    const float sign = ((t + (int)(row & 1)) & 1) ? -1.0f : 1.0f;   // (T is even)
    const float2 *src = in + row * N + t;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const float2 x = on ? src[k * T] : make_float2(0.0f, 0.0f);
        v[k] = make_float2(sign * x.x, sign * x.y);
    }
    fft_inverse<LOGN>(v, t, [&](auto put) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) s[rr][fft_pad(put(k))] = v[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = s[rr][fft_pad(t + k * T)];
    });
    if (!on) return;
    float2 *dst = out + row * N + t;
#pragma unroll
    for (int k = 0; k < 16; ++k) dst[k * T] = v[k];
}

// Columns of a workgroup of the column kernels: four 2048- or 4096-point
// columns (32-byte pieces of each row; the tiles that share a line run
// together, see first_column), eight shorter ones, more of the shortest (256
// threads at least).  4 x 2048 x 2048, the column kernel: eight columns of 2048
// points 77 us, four 60 us (two workgroups to a CU load and compute in turn);
// 4 x 4096 x 2048 cropped to half: four columns 160 us, two 182 us.
constexpr int fft_cols(int logn) { return logn > 10 ? 4 : logn < 9 ? 256 * 16 >> logn : 8; }
constexpr int fft_col_threads(int logn) { return fft_cols(logn) * (1 << logn) / 16; }
constexpr size_t fft_col_lds(int logn) {
    return sizeof(float) * (size_t)fft_cols(logn) * fft_points(logn);
}

// First column of workgroup b of n.  Workgroups go to the eight XCDs in turn,
// and each XCD has its own L2: neighbouring tiles, which share 128-byte lines of
// every row, go to workgroups eight apart, on the same XCD and at about the
// same time (4 x 4096 x 2048, four columns each: 311 us in plain order, 160 us
// so).
template <int C>
__device__ inline int first_column(int b, int n) {
    return C * (n % 8 == 0 ? (b % 8) * (n / 8) + b / 8 : b);
}

// The points of a workgroup's columns through LDS, real parts and then
// imaginary ones (half the LDS: two workgroups share a CU).
template <int LOGN, typename P>
__device__ inline void exchange_columns(float2 (&v)[16], float *s, int t, int c, P &&put) {
    constexpr int T = (1 << LOGN) / 16, C = fft_cols(LOGN);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) s[fft_pad(put(k)) * C + c] = v[k].x;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k].x = s[fft_pad(t + k * T) * C + c];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) s[fft_pad(put(k)) * C + c] = v[k].y;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k].y = s[fft_pad(t + k * T) * C + c];
}

// image[p][y][x] = (-1)^(x + y0 + y + nx/2 + ny/2) cx[x] cy[y] times the
// transform of column x of work[p] at row y0 + y, y < out_ny.  (A workgroup has
// read its columns before it stores them: work and image may be the same
// buffer where nothing is cropped.)  PLAIN: the transform alone, uncropped.
template <int LOGN, bool PLAIN>
__global__ __launch_bounds__(fft_col_threads(LOGN)) void fft_columns_kernel(
    const float2 *work, float2 *image, int32_t nx, int32_t y0,
    int32_t out_ny, const float *__restrict__ cx, const float *__restrict__ cy) {
    constexpr int N = 1 << LOGN, T = N / 16, C = fft_cols(LOGN);
    extern __shared__ float s_col[];
    const int c = threadIdx.x % C, t = threadIdx.x / C;
    const int x = first_column<C>(blockIdx.x, gridDim.x) + c, p = blockIdx.y;
    float2 v[16];
    const float2 *src = work + ((int64_t)p * N + t) * nx + x;
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = src[(int64_t)k * T * nx];
    fft_inverse<LOGN>(v, t, [&](auto put) { exchange_columns<LOGN>(v, s_col, t, c, put); });
    if constexpr (PLAIN) {
#pragma unroll
        for (int k = 0; k < 16; ++k) image[((int64_t)p * N + t + k * T) * nx + x] = v[k];
        return;
    }
    float f = cx[x];
    if ((x + t + nx / 2 + N / 2) & 1) f = -f;   // (T is even)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int y = t + k * T - y0;
        if (y < 0 || y >= out_ny) continue;
        const float g = f * cy[y];
        image[((int64_t)p * out_ny + y) * nx + x] = make_float2(v[k].x * g, v[k].y * g);
    }
}

// work[p][y][x] = (-1)^(x + y) grid[p][y][x]
__global__ __launch_bounds__(256) void shift_in_kernel(const float2 *__restrict__ grid,
                                                       float2 *__restrict__ work, int32_t nx,
                                                       int64_t total) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = k / nx;
        const int x = (int)(k - row * nx);
        float2 g = grid[k];
        if ((x + row) & 1) {
            g.x = -g.x;
            g.y = -g.y;
        }
        work[k] = g;
    }
}

// image[p][y][x] = (-1)^(x + y0 + y + nx/2 + ny/2) corr_x[x] corr_y[y]
//                  work[p][y0 + y][x], y < out_ny
// (work and image may be the same buffer where nothing is cropped)
__global__ __launch_bounds__(256) void correct_out_kernel(const float2 *work, float2 *image,
                                                          int32_t nx, int32_t ny, int32_t y0,
                                                          int32_t out_ny, int32_t npol,
                                                          const float *__restrict__ cx,
                                                          const float *__restrict__ cy) {
    const int64_t total = (int64_t)npol * out_ny * nx;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t prow = k / nx;
        const int x = (int)(k - prow * nx);
        const int p = (int)(prow / out_ny);
        const int y = (int)(prow - (int64_t)p * out_ny);
        float2 v = work[((int64_t)p * ny + y0 + y) * nx + x];
        float f = cx[x] * cy[y];
        if ((x + y0 + y + nx / 2 + ny / 2) & 1) f = -f;
        v.x *= f;
        v.y *= f;
        image[k] = v;
    }
}

// W-stacking: image[p][y][x] = (-1)^(x + y + nx/2 + ny/2) cx[x] cy[y]
//   sum_j I_j[p][y][x] gbar_{w_j}(l_x, m_y), I_j the transform of layer j,
// gbar_w = exp(+j2pi w (sqrt(1 - l^2 - m^2) - 1)), w_j = (j - (L-1)/2) dw,
// l_x = (x - nx/2)/nx fov_x, m_y = (y - ny/2)/ny fov_y.  n - 1 is formed as
// -r^2 / (1 + sqrt(1 - r^2)) (no cancellation) and each phase, in cycles, is
// reduced to (-1/2, 1/2] in FP64 before the FP32 sine and cosine.
__device__ inline double w_n_minus_1(int x, int y, int nx, int ny, double fov_x, double fov_y) {
    const double l = (double)(x - nx / 2) / (double)nx * fov_x;
    const double m = (double)(y - ny / 2) / (double)ny * fov_y;
    const double r2 = l * l + m * m;
    return r2 < 1.0 ? -r2 / (1.0 + sqrt(1.0 - r2)) : -1.0;
}

// sum += v gbar, at layer w and n - 1
__device__ inline void add_screened(float2 &sum, float2 v, double w, double nm1) {
    double cyc = w * nm1;
    cyc -= rint(cyc);
    float sn, cs;
    sincospif(2.0f * (float)cyc, &sn, &cs);
    sum.x += v.x * cs - v.y * sn;
    sum.y += v.x * sn + v.y * cs;
}

// Power-of-two sides: the columns of every layer transformed, screened and
// summed in registers, so the transformed layers never reach HBM.  Held to 128
// VGPRs (two workgroups of 512 threads to a CU): 64 transforms of 2048 x 2048
// take 1.07 ms (0.88, against 1.33 with the registers it would take, before the
// twiddles were formed in FP64); the layers' one read takes 0.42 ms at a device
// copy's rate.
template <int LOGN>
__global__ __launch_bounds__(fft_col_threads(LOGN)) __attribute__((amdgpu_waves_per_eu(4)))
void wstack_columns_kernel(
    const float2 *__restrict__ work, float2 *__restrict__ image, int32_t nx, int32_t layers,
    double dw, double fov_x, double fov_y, const float *__restrict__ cx,
    const float *__restrict__ cy) {
    constexpr int N = 1 << LOGN, T = N / 16, C = fft_cols(LOGN);
    extern __shared__ float s_col[];
    const int c = threadIdx.x % C, t = threadIdx.x / C;
    const int x = first_column<C>(blockIdx.x, gridDim.x) + c, p = blockIdx.y;
    double nm1[16];
    float2 sum[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        nm1[k] = w_n_minus_1(x, t + k * T, nx, N, fov_x, fov_y);
        sum[k] = make_float2(0.0f, 0.0f);
    }
    for (int j = 0; j < layers; ++j) {
        float2 v[16];
        const float2 *src = work + (((int64_t)p * layers + j) * N + t) * nx + x;
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = src[(int64_t)k * T * nx];
        // (the twiddles are formed again for each layer: kept, they would spill
        // the sums)
        int tj = t;
        asm volatile("" : "+v"(tj));
        fft_inverse<LOGN>(v, tj, [&](auto put) { exchange_columns<LOGN>(v, s_col, tj, c, put); });
        const double wj = ((double)j - 0.5 * (double)(layers - 1)) * dw;
#pragma unroll
        for (int k = 0; k < 16; ++k) add_screened(sum[k], v[k], wj, nm1[k]);
    }
    float f = cx[x];
    if ((x + t + nx / 2 + N / 2) & 1) f = -f;   // (T is even)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const float g = f * cy[t + k * T];
        image[((int64_t)p * N + t + k * T) * nx + x] = make_float2(sum[k].x * g, sum[k].y * g);
    }
}

// From the transforms of the layers: other sides, and power-of-two ones with too
// few columns (wstack_fused).
__global__ __launch_bounds__(256) void wstack_combine_kernel(
    const float2 *__restrict__ work, float2 *__restrict__ image, int32_t nx, int32_t ny,
    int32_t npol, int32_t layers, double dw, double fov_x, double fov_y,
    const float *__restrict__ cx, const float *__restrict__ cy) {
    const int64_t plane = (int64_t)ny * nx;
    const int64_t total = (int64_t)npol * plane;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int p = (int)(k / plane);
        const int64_t yx = k - (int64_t)p * plane;
        const int y = (int)(yx / nx);
        const int x = (int)(yx - (int64_t)y * nx);
        const double nm1 = w_n_minus_1(x, y, nx, ny, fov_x, fov_y);
        float2 sum = make_float2(0.0f, 0.0f);
        const float2 *src = work + (int64_t)p * layers * plane + yx;
        for (int j = 0; j < layers; ++j)
            add_screened(sum, src[(int64_t)j * plane],
                         ((double)j - 0.5 * (double)(layers - 1)) * dw, nm1);
        float f = cx[x] * cy[y];
        if ((x + y + nx / 2 + ny / 2) & 1) f = -f;
        image[k] = make_float2(sum.x * f, sum.y * f);
    }
}

// wstack_columns_kernel takes the layers of a column one after another, so its
// columns alone have to fill the chip: four waves a SIMD, 1024 threads a CU.
// Below that the layers' columns are transformed side by side, in place, and
// combined in another pass.  One polarisation, 128 layers of 256^2: 563 us one
// after another, 84 side by side; 16 of 2048^2 (which fill it): 503 and 595.
bool wstack_fused(int64_t groups, int threads, int layers) {
    return layers == 1 || groups * threads >= (int64_t)device_cus() * 1024;
}

int blocks_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (int)(b < 1 ? 1 : (b > 16384 ? 16384 : b));
}

// Sides the kernels of this file transform: powers of two, rows of 64 to 8192
// cells and columns of 64 to 4096 (a column's 16-point share of 1024 threads;
// four columns at least, for 32-byte pieces of each row).
int log2_side(int n, int most) {
    for (int l = 6; l <= most; ++l)
        if (n == 1 << l) return l;
    return 0;
}
bool own_fft(int nx, int ny) { return log2_side(nx, 13) && log2_side(ny, 12); }

template <int LOGN>
void launch_rows(const void *in, void *out, int64_t nrows, hipStream_t stream) {
    constexpr int THREADS = LOGN > 12 ? 512 : 256, ROWS = THREADS * 16 >> LOGN;
    hipLaunchKernelGGL(fft_rows_kernel<LOGN>, dim3((unsigned)((nrows + ROWS - 1) / ROWS)),
                       dim3(THREADS), 0, stream, (const float2 *)in, (float2 *)out, nrows);
}

void fft_rows(int logn, const void *in, void *out, int64_t nrows, hipStream_t stream) {
    switch (logn) {
    case 6: launch_rows<6>(in, out, nrows, stream); break;
    case 7: launch_rows<7>(in, out, nrows, stream); break;
    case 8: launch_rows<8>(in, out, nrows, stream); break;
    case 9: launch_rows<9>(in, out, nrows, stream); break;
    case 10: launch_rows<10>(in, out, nrows, stream); break;
    case 11: launch_rows<11>(in, out, nrows, stream); break;
    case 12: launch_rows<12>(in, out, nrows, stream); break;
    default: launch_rows<13>(in, out, nrows, stream); break;
    }
}

// f(integral_constant<logn>), logn in 6..12
template <typename F> void column_size(int logn, F &&f) {
    switch (logn) {
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 11: f(std::integral_constant<int, 11>{}); break;
    default: f(std::integral_constant<int, 12>{}); break;
    }
}

// The library's batched plan, for sides that are not own_fft's.
mg_status library_plan(hipfftHandle *plan, int nx, int ny, int batch) {
    if (own_fft(nx, ny)) return MG_OK;
    int dims[2] = {ny, nx};
    const int dist = ny * nx;
    const hipfftResult r = hipfftPlanMany(plan, 2, dims, nullptr, 1, dist, nullptr, 1, dist,
                                          HIPFFT_C2C, batch);
    if (r != HIPFFT_SUCCESS)
        return set_error(MG_EDEVICE, "FFT plan creation failed (" + std::to_string((int)r) + ")");
    return MG_OK;
}

// The centred transforms (but for the signs of the output) of the nx x ny planes
// of `grid`, `total` cells, in `work`.
mg_status library_fft(hipfftHandle plan, const void *grid, void *work, int nx, int64_t total,
                      hipStream_t stream) {
    hipLaunchKernelGGL(shift_in_kernel, dim3(blocks_for(total)), dim3(256), 0, stream,
                       (const float2 *)grid, (float2 *)work, nx, total);
    if (hipfftSetStream(plan, stream) != HIPFFT_SUCCESS) return set_error(MG_EDEVICE, "FFT stream");
    const hipfftResult r = hipfftExecC2C(plan, (hipfftComplex *)work, (hipfftComplex *)work,
                                         HIPFFT_BACKWARD);
    if (r != HIPFFT_SUCCESS)
        return set_error(MG_EDEVICE, "FFT execution failed (" + std::to_string((int)r) + ")");
    return MG_OK;
}

}  // namespace
}  // namespace mg

using namespace mg;

extern "C" {

mg_status mg_corrector(int32_t n, int32_t beta, int32_t table_len, int32_t phases,
                       int32_t nn_sinc, const float *table, float *corr, hipStream_t stream) {
    if (n < 1 || beta < 1 || table_len < 1 || phases < 1 || !table || !corr)
        return set_error(MG_EINVAL, "bad corrector arguments");
    hipLaunchKernelGGL(corrector_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       n, beta, table_len, phases, nn_sinc, table, corr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("corrector: ") + hipGetErrorString(e));
    return MG_OK;
}

mg_status mg_imager_create(mg_imager **im, int32_t npol, int32_t nx, int32_t ny) {
    if (!im) return set_error(MG_EINVAL, "null imager output");
    *im = nullptr;
    if (npol < 1 || npol > 4 || nx < 2 || ny < 2 || (nx & 1) || (ny & 1))
        return set_error(MG_EINVAL, "imager sizes must be even, npol 1..4");
    mg_imager *p = new (std::nothrow) mg_imager;
    if (!p) return set_error(MG_ENOMEM, "host allocation failed");
    p->npol = npol;
    p->nx = nx;
    p->ny = ny;
    const mg_status st = library_plan(&p->plan, nx, ny, npol);
    if (st != MG_OK) {
        delete p;
        return st;
    }
    *im = p;
    return MG_OK;
}

mg_status mg_imager_exec(mg_imager *im, const void *grid, void *work, void *image,
                         const float *corr_x, const float *corr_y, int32_t y0, int32_t out_ny,
                         hipStream_t stream) {
    if (!im || !grid || !work || !image || !corr_x || !corr_y)
        return set_error(MG_EINVAL, "null argument");
    if (y0 < 0 || out_ny < 1 || y0 + out_ny > im->ny)
        return set_error(MG_EINVAL, "rows out of range");
    if (work == image && !(y0 == 0 && out_ny == im->ny))
        return set_error(MG_EINVAL, "a cropped image needs its own buffer");
    if (own_fft(im->nx, im->ny)) {
        fft_rows(log2_side(im->nx, 13), grid, work, (int64_t)im->npol * im->ny, stream);
        column_size(log2_side(im->ny, 12), [&](auto l) {
            constexpr int L = decltype(l)::value;
            hipLaunchKernelGGL((fft_columns_kernel<L, false>),
                               dim3((unsigned)(im->nx / fft_cols(L)), (unsigned)im->npol),
                               dim3(fft_col_threads(L)), fft_col_lds(L), stream,
                               (const float2 *)work, (float2 *)image, im->nx, y0, out_ny, corr_x,
                               corr_y);
        });
    } else {
        const mg_status st = library_fft(im->plan, grid, work, im->nx,
                                         (int64_t)im->npol * im->ny * im->nx, stream);
        if (st != MG_OK) return st;
        hipLaunchKernelGGL(correct_out_kernel,
                           dim3(blocks_for((int64_t)im->npol * out_ny * im->nx)), dim3(256), 0,
                           stream, (const float2 *)work, (float2 *)image, im->nx, im->ny, y0,
                           out_ny, im->npol, corr_x, corr_y);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("imaging kernels: ") + hipGetErrorString(e));
    return MG_OK;
}

mg_status mg_imager_destroy(mg_imager *im) {
    if (!im) return MG_OK;
    if (im->plan) hipfftDestroy(im->plan);
    delete im;
    return MG_OK;
}

mg_status mg_wstack_imager_create(mg_wstack_imager **im, int32_t npol, int32_t layers,
                                  int32_t nx, int32_t ny) {
    if (!im) return set_error(MG_EINVAL, "null imager output");
    *im = nullptr;
    if (npol < 1 || npol > 4 || layers < 1 || layers > kMaxPlanes || nx < 2 || ny < 2 ||
        (nx & 1) || (ny & 1))
        return set_error(MG_EINVAL, "imager sizes must be even, npol 1..4, layers 1..128");
    mg_wstack_imager *p = new (std::nothrow) mg_wstack_imager;
    if (!p) return set_error(MG_ENOMEM, "host allocation failed");
    p->npol = npol;
    p->layers = layers;
    p->nx = nx;
    p->ny = ny;
    const mg_status st = library_plan(&p->plan, nx, ny, npol * layers);
    if (st != MG_OK) {
        delete p;
        return st;
    }
    *im = p;
    return MG_OK;
}

mg_status mg_wstack_imager_exec(mg_wstack_imager *im, const void *grids, void *work, void *image,
                                const float *corr_x, const float *corr_y, double fov_x,
                                double fov_y, double dw, hipStream_t stream) {
    if (!im || !grids || !work || !image || !corr_x || !corr_y)
        return set_error(MG_EINVAL, "null argument");
    if (!std::isfinite(fov_x) || !std::isfinite(fov_y) || !std::isfinite(dw))
        return set_error(MG_EINVAL, "fov and dw must be finite");
    if (work == image) return set_error(MG_EINVAL, "the image needs its own buffer");
    const bool own = own_fft(im->nx, im->ny);
    bool combine = !own;
    if (own) {
        fft_rows(log2_side(im->nx, 13), grids, work, (int64_t)im->npol * im->layers * im->ny,
                 stream);
        column_size(log2_side(im->ny, 12), [&](auto l) {
            constexpr int L = decltype(l)::value;
            const unsigned tiles = (unsigned)(im->nx / fft_cols(L));
            combine = !wstack_fused((int64_t)tiles * im->npol, fft_col_threads(L), im->layers);
            if (combine)
                hipLaunchKernelGGL((fft_columns_kernel<L, true>),
                                   dim3(tiles, (unsigned)(im->npol * im->layers)),
                                   dim3(fft_col_threads(L)), fft_col_lds(L), stream,
                                   (const float2 *)work, (float2 *)work, im->nx, 0, im->ny,
                                   nullptr, nullptr);
            else
                hipLaunchKernelGGL(wstack_columns_kernel<L>, dim3(tiles, (unsigned)im->npol),
                                   dim3(fft_col_threads(L)), fft_col_lds(L), stream,
                                   (const float2 *)work, (float2 *)image, im->nx, im->layers, dw,
                                   fov_x, fov_y, corr_x, corr_y);
        });
    } else {
        const mg_status st =
            library_fft(im->plan, grids, work, im->nx,
                        (int64_t)im->npol * im->layers * im->ny * im->nx, stream);
        if (st != MG_OK) return st;
    }
    if (combine)
        hipLaunchKernelGGL(wstack_combine_kernel,
                           dim3(blocks_for((int64_t)im->npol * im->ny * im->nx)), dim3(256), 0,
                           stream, (const float2 *)work, (float2 *)image, im->nx, im->ny,
                           im->npol, im->layers, dw, fov_x, fov_y, corr_x, corr_y);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("W-stacking kernels: ") + hipGetErrorString(e));
    return MG_OK;
}

mg_status mg_wstack_imager_destroy(mg_wstack_imager *im) {
    if (!im) return MG_OK;
    if (im->plan) hipfftDestroy(im->plan);
    delete im;
    return MG_OK;
}

}  // extern "C"
