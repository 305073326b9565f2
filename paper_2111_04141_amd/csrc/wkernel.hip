// W-projection kernel bank builder.
//
// Plane p of the bank tabulates, at 1/beta cells over its support S_p, the
// GCF convolved with the transform of the inverse W-term (Section 1.7.1,
// W-projection; Section 1.3 for the W-term g_w and gbar_w = 1 / g_w):
//     K_p = F[ c(l) c(m) gbar_{w_p}(l, m) ],
//     gbar_w(l, m) = exp(+j2pi w (sqrt(1 - l^2 - m^2) - 1)),
// with c the image-domain taper of the separable GCF C (c = F^-1 C) and F
// the transform with exp(-j2pi (ul + vm)).  Discretisation: an M x M image
// grid, M = 2 beta S_p, of spacing beta / M field units (so its transform
// has uv spacing 1/beta cells and spans 2 S_p cells), physical direction
// cosines = field units x fov; the central beta S_p + 1 samples per axis
// are kept.
//
// The image is even along both axes (the taper is real and even, the W-term
// depends on l^2 + m^2), so its transform is a cosine transform of one
// quadrant, and even again: with H = M/2 and e_i = 1 for i = 0 and i = H, else
// 2,
//     K[a][b] = sum_{i, j = 0..H} e_i e_j img[i][j] cos(2pi a i/M) cos(2pi b j/M)
// for a, b = 0 .. H/2, an eighth of the samples a full transform computes.
// The two sums are small FP64 matrix products on the matrix cores (any M, no
// transform sizes with large prime factors), and every step covers all planes
// in one launch: 32 planes of S 8 -> 64, oversampling 4, took 1.36 ms as 32
// library transforms and some 200 launches, bound by launch latency, and
// takes 0.058 ms here.
//   tables_kernel  cos(2pi k/M), and the taper
//                  c[i] = (1/M) sum_tau T[tau] cos(2pi tau i / M), i = 0..H
//   screen_kernel  X[i][j] = e_i e_j c[i] c[j] gbar(l_i, m_j)
//   cosine_kernel  B[i][b] = sum_j X[i][j] cos(2pi b j/M)  (X is symmetric),
//                  then K[a][b] = sum_i cos(2pi a i/M) B[i][b] and the largest
//                  |K|
//   store_kernel   bank = K / max, converted to the output tap format, row
//                  (v offset) major.
// The products grow with H^3 and a transform with H^2 log H: planes of H above
// kCosineMax take the platform library's transform of the full M x M image, in
// place, and quadrant_kernel keeps K and its maximum.
// All steps in FP64.  Plane parameters travel as kernel arguments, so the
// call copies nothing from the host and does not synchronise.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "internal.h"

namespace mg {
namespace {

// The planes of a bank (kernel argument).  The workspace of plane p, in
// doubles from ws[p]: cos table [M], taper [H + 1], padded to even, then
// complex K [h + 1][h + 1], X [H + 1][H + 1], B [H + 1][h + 1], H = M/2 = beta
// S, h = H/2; H above kCosineMax: K, X [M][M] (its transform takes its place).
struct BankPlanes {
    int64_t ws[kMaxPlanes];
    int64_t bank[kMaxPlanes];   // complex elements into the bank
    double w[kMaxPlanes];
    uint8_t S[kMaxPlanes];
};

struct PlaneWork {
    int M, H, h;
    double *ct, *taper;
    double2 *X, *B, *K;
};

constexpr int kMaxBank = 512;   // largest beta S whose cos table goes to LDS
// Largest beta S by cosine products: one plane of 1024 takes 151 us (190 by a
// transform of its full image), one of 2048 1122 us (678), of 4096 11.4 ms
// (3.2).
constexpr int kCosineMax = 1024;

constexpr int64_t table_doubles(int64_t H) { return (2 * H + H + 1 + 1) & ~int64_t(1); }
constexpr int64_t work_doubles(int64_t H) {
    if (H > kCosineMax) return table_doubles(H) + 2 * (4 * H * H + (H / 2 + 1) * (H / 2 + 1));
    return table_doubles(H) + 2 * ((H + 1) * (H + 1) + (H + 1) * (H / 2 + 1) + (H / 2 + 1) * (H / 2 + 1));
}

__device__ inline PlaneWork plane_work(const BankPlanes &P, int p, int beta, double *ws) {
    PlaneWork w;
    w.H = beta * (int)P.S[p];
    w.M = 2 * w.H;
    w.h = w.H / 2;
    w.ct = ws + P.ws[p];
    w.taper = w.ct + w.M;
    w.K = reinterpret_cast<double2 *>(w.ct + table_doubles(w.H));
    w.X = w.K + (int64_t)(w.h + 1) * (w.h + 1);
    w.B = w.X + (int64_t)(w.H + 1) * (w.H + 1);
    return w;
}

// One wave per taper value (lanes share the sum); also the cos table, and the
// cleared maximum.
__global__ __launch_bounds__(256) void tables_kernel(BankPlanes P, int32_t beta, int32_t base_len,
                                                     const double *__restrict__ T,
                                                     double *__restrict__ ws,
                                                     unsigned long long *mx) {
    const PlaneWork w = plane_work(P, blockIdx.y, beta, ws);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *mx = 0ull;
    const int first = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    for (int k = first; k < w.M; k += step) w.ct[k] = cospi(2.0 * (double)k / (double)w.M);
    const int lane = threadIdx.x & 63, half = (base_len - 1) / 2;
    for (int i = first >> 6; i <= w.H; i += step >> 6) {
        double s = 0.0;
        for (int t = lane; t < base_len; t += 64) {
            // tau i mod M keeps the cosine argument small and exact
            const int ph = (t - half) * i % w.M;   // (below 2^25)
            s += T[t] * cospi(2.0 * (double)ph / (double)w.M);
        }
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) w.taper[i] = s / (double)w.M;
    }
}

// The weighted quadrant of every plane up to kCosineMax; FULL: the whole image of
// plane `plane`, in transform order.
template <bool FULL>
__global__ __launch_bounds__(256) void screen_kernel(BankPlanes P, int32_t plane, int32_t beta,
                                                     double fov, double *__restrict__ ws) {
    const int p = FULL ? plane : (int)blockIdx.y;
    const PlaneWork w = plane_work(P, p, beta, ws);
    if (!FULL && w.H > kCosineMax) return;
    const int side = FULL ? w.M : w.H + 1;
    const double wp = P.w[p];
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < side * side;
         k += gridDim.x * blockDim.x) {
        int i = k / side, j = k - i * side;
        if constexpr (FULL) {   // (even along both axes)
            i = min(i, w.M - i);
            j = min(j, w.M - j);
        }
        const double l = (double)i * ((double)beta / (double)w.M) * fov;
        const double m = (double)j * ((double)beta / (double)w.M) * fov;
        const double r2 = l * l + m * m;
        const double nn = r2 < 1.0 ? sqrt(1.0 - r2) : 0.0;
        double sn, cs;
        sincospi(2.0 * (wp * (nn - 1.0)), &sn, &cs);
        double e = 1.0;
        if constexpr (!FULL) e = (i == 0 || i == w.H ? 1.0 : 2.0) * (j == 0 || j == w.H ? 1.0 : 2.0);
        const double a = e * w.taper[i] * w.taper[j];
        w.X[k] = make_double2(a * cs, a * sn);
    }
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// D = A B on 16 x 16 x 4 FP64 matrix instructions, one 16 x 16 tile (real and
// imaginary parts) per workgroup, whose four waves each take a quarter of the
// sum; lane l holds A[row l % 16][k l / 16], B[k l / 16][column l % 16] and
// D[row l / 16 + 4 r][column l % 16], r = 0..3.
// Pass 0: D[i][b] = sum_j X[i][j] cos(2pi b j/M) (X[j][i] is read for X[i][j],
// so lanes read consecutive words).  Pass 1: D[a][b] = sum_i cos(2pi a i/M)
// B[i][b], and the largest |D|.
// Bound by latency: a sum is a chain of H / 4 instructions (64 for S = 64,
// beta = 4).  One wave per tile and one operand load at a time took 36 us a
// pass for 32 planes of S 8 -> 64; eight loads together 24 us; the split sum
// with the cosines in LDS 20 us.
template <int PASS>
__global__ __launch_bounds__(256) void cosine_kernel(BankPlanes P, int32_t beta,
                                                     double *__restrict__ ws,
                                                     unsigned long long *mx) {
    const PlaneWork w = plane_work(P, blockIdx.y, beta, ws);
    const int rows = PASS == 0 ? w.H + 1 : w.h + 1, cols = w.h + 1;
    const int tc = (cols + 15) / 16, tiles = ((rows + 15) / 16) * tc;
    const int tile = blockIdx.x;
    if (tile >= tiles || w.H > kCosineMax) return;
    __shared__ double s_cos[2 * kMaxBank];
    __shared__ f64x4 s_part[2][3][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kk = lane >> 4;
    const int r0 = (tile / tc) * 16, c0 = (tile % tc) * 16;
    const bool in_lds = w.H <= kMaxBank;
    if (in_lds)
        for (int k = threadIdx.x; k < w.M; k += blockDim.x) s_cos[k] = w.ct[k];
    __syncthreads();
    // rows and columns past the end repeat the last one and are not stored
    const int row = min(r0 + l16, rows - 1), col = min(c0 + l16, cols - 1);
    // this wave's instructions: k = 4 n + kk, n in [n0, n1)
    const int steps = w.H / 4 + 1, n0 = steps * wave / 4, n1 = steps * (wave + 1) / 4;
    // cosine operand: index (PASS == 0 ? col : row) * k mod M
    const int f = PASS == 0 ? col : row;
    int ph = (int)((uint32_t)(f * (4 * n0 + kk)) % (uint32_t)w.M);   // (below 2^25)
    const int dph = (int)((uint32_t)(f * 4) % (uint32_t)w.M);
    f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
    constexpr int kAhead = 8;   // operands loaded together
    for (int nb = n0; nb < n1; nb += kAhead) {
        double c[kAhead];
        double2 x[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int k = 4 * (nb + a) + kk;
            c[a] = 0.0;
            x[a] = make_double2(0.0, 0.0);
            if (nb + a < n1 && k <= w.H) {
                c[a] = in_lds ? s_cos[ph] : w.ct[ph];
                x[a] = PASS == 0 ? w.X[(int64_t)k * (w.H + 1) + row] : w.B[(int64_t)k * cols + col];
            }
            ph += dph;
            if (ph >= w.M) ph -= w.M;
        }
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            if (PASS == 0) {
                re = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a].x, c[a], re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a].y, c[a], im, 0, 0, 0);
            } else {
                re = __builtin_amdgcn_mfma_f64_16x16x4f64(c[a], x[a].x, re, 0, 0, 0);
                im = __builtin_amdgcn_mfma_f64_16x16x4f64(c[a], x[a].y, im, 0, 0, 0);
            }
        }
    }
    if (wave > 0) {
        s_part[0][wave - 1][lane] = re;
        s_part[1][wave - 1][lane] = im;
    }
    __syncthreads();
    if (wave > 0) return;
    for (int v = 0; v < 3; ++v) {
        re += s_part[0][v][lane];
        im += s_part[1][v][lane];
    }
    double best = 0.0;
    double2 *out = PASS == 0 ? w.B : w.K;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = r0 + kk + 4 * r, j = c0 + l16;
        if (i < rows && j < cols) {
            out[(int64_t)i * cols + j] = make_double2(re[r], im[r]);
            best = fmax(best, sqrt(re[r] * re[r] + im[r] * im[r]));
        }
    }
    if constexpr (PASS == 1) {
        // magnitudes are non-negative, so their bit patterns order like the values
        for (int o = 32; o > 0; o >>= 1) best = fmax(best, __shfl_xor(best, o));
        if (lane == 0) atomicMax(mx, (unsigned long long)__double_as_longlong(best));
    }
}

// K of plane p from its transform, and the largest |K|.
__global__ __launch_bounds__(256) void quadrant_kernel(BankPlanes P, int32_t p, int32_t beta,
                                                       double *__restrict__ ws,
                                                       unsigned long long *mx) {
    const PlaneWork w = plane_work(P, p, beta, ws);
    const int side = w.h + 1;
    double best = 0.0;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < side * side;
         k += gridDim.x * blockDim.x) {
        const int a = k / side, b = k - a * side;
        const double2 v = w.X[(int64_t)a * w.M + b];
        w.K[k] = v;
        best = fmax(best, sqrt(v.x * v.x + v.y * v.y));
    }
    for (int o = 32; o > 0; o >>= 1) best = fmax(best, __shfl_xor(best, o));
    if ((threadIdx.x & 63) == 0) atomicMax(mx, (unsigned long long)__double_as_longlong(best));
}

template <typename OutT> __device__ inline void store_tap(OutT *bank, int64_t i, double re, double im);
template <> __device__ inline void store_tap<float>(float *bank, int64_t i, double re, double im) {
    bank[2 * i] = (float)re;
    bank[2 * i + 1] = (float)im;
}
// FP16 and BF16: rounded to FP32, then to the nearest value of the format
// (ties to even)
template <> __device__ inline void store_tap<__half>(__half *bank, int64_t i, double re, double im) {
    bank[2 * i] = __float2half((float)re);
    bank[2 * i + 1] = __float2half((float)im);
}
template <>
__device__ inline void store_tap<__hip_bfloat16>(__hip_bfloat16 *bank, int64_t i, double re,
                                                 double im) {
    bank[2 * i] = __float2bfloat16((float)re);
    bank[2 * i + 1] = __float2bfloat16((float)im);
}

template <typename OutT>
__global__ __launch_bounds__(256) void store_kernel(BankPlanes P, int32_t beta,
                                                    double *__restrict__ ws,
                                                    const unsigned long long *mx,
                                                    OutT *__restrict__ bank) {
    const PlaneWork w = plane_work(P, blockIdx.y, beta, ws);
    const int E = w.H + 1;   // beta S + 1 kept samples per axis, the centre at h
    OutT *dst = bank + 2 * P.bank[blockIdx.y];
    const double m = __longlong_as_double((long long)*mx);
    const double inv = m > 0.0 ? 1.0 / m : 0.0;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < E * E; t += gridDim.x * blockDim.x) {
        const int ta = t / E, tb = t - ta * E;
        const double2 v = w.K[(int64_t)abs(ta - w.h) * (w.h + 1) + abs(tb - w.h)];
        store_tap<OutT>(dst, t, v.x * inv, v.y * inv);
    }
}

struct Layout {
    BankPlanes planes;
    int64_t bank_elems = 0;
    int64_t H_max = 0;          // largest beta S
    int64_t H_cosine = 0;       // the same up to kCosineMax (0: none)
    size_t bytes = 0, off_max = 0;
};

mg_status make_layout(int32_t nplanes, const int32_t *sup, int32_t beta, Layout &L) {
    if (nplanes < 1 || nplanes > kMaxPlanes) return set_error(MG_EINVAL, "nplanes must be in 1..128");
    if (!sup) return set_error(MG_EINVAL, "null plane supports");
    if (beta < 1 || beta > kMaxBeta) return set_error(MG_EINVAL, "beta must be in 1..256");
    int64_t doubles = 0;
    for (int p = 0; p < nplanes; ++p) {
        const int S = sup[p];
        if (S < 1 || S > kMaxSupport) return set_error(MG_EINVAL, "plane support must be in 1..64");
        if (((int64_t)beta * S) % 2) return set_error(MG_EINVAL, "beta * support must be even");
        // the FP64 image of a large plane is (2 beta S)^2 x 16 bytes
        if ((int64_t)beta * S > 4096) return set_error(MG_EINVAL, "beta * support must be <= 4096");
        const int64_t H = (int64_t)beta * S;
        L.planes.S[p] = (uint8_t)S;
        L.planes.ws[p] = doubles;
        L.planes.bank[p] = L.bank_elems;
        L.bank_elems += (H + 1) * (H + 1);
        doubles += work_doubles(H);
        L.H_max = std::max(L.H_max, H);
        if (H <= kCosineMax) L.H_cosine = std::max(L.H_cosine, H);
    }
    L.off_max = arena_round(sizeof(double) * (size_t)doubles);
    L.bytes = L.off_max + arena_round(sizeof(unsigned long long));
    return MG_OK;
}

// FFT plans by (device, M), kept for the life of the process, with the bytes of
// work area one needs.  Builds bring a work area of their own each, so a plan's
// transforms may overlap on several streams.
struct BankFft {
    hipfftHandle h = nullptr;
    size_t work = 0;
};
std::mutex g_fft_mu;
std::map<std::pair<int, int>, BankFft> g_fft;

// (with g_fft_mu held)
hipfftResult bank_fft(int dev, int M, BankFft *out) {
    auto it = g_fft.find({dev, M});
    if (it == g_fft.end()) {
        BankFft f;
        hipfftResult r = hipfftCreate(&f.h);
        if (r != HIPFFT_SUCCESS) return r;
        r = hipfftSetAutoAllocation(f.h, 0);
        if (r == HIPFFT_SUCCESS) r = hipfftMakePlan2d(f.h, M, M, HIPFFT_Z2Z, &f.work);
        if (r == HIPFFT_SUCCESS) r = hipfftGetSize(f.h, &f.work);
        if (r != HIPFFT_SUCCESS) {
            hipfftDestroy(f.h);
            return r;
        }
        it = g_fft.emplace(std::make_pair(dev, M), f).first;
    }
    *out = it->second;
    return HIPFFT_SUCCESS;
}

// Images, transforms and quadrants of the planes above kCosineMax.
mg_status large_planes(const Layout &L, int32_t nplanes, int32_t beta, double fov, double *ws,
                       unsigned long long *mx, hipStream_t stream) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return set_error(MG_EDEVICE, "no device");
    auto fft_error = [](hipfftResult r) {
        return set_error(MG_EDEVICE, "FFT failed (" + std::to_string((int)r) + ")");
    };
    // one work area for them all, in the stream's order
    size_t bytes = 0;
    for (int p = 0; p < nplanes; ++p) {
        const int H = beta * (int)L.planes.S[p];
        if (H <= kCosineMax) continue;
        std::lock_guard<std::mutex> lk(g_fft_mu);
        BankFft f;
        const hipfftResult r = bank_fft(dev, 2 * H, &f);
        if (r != HIPFFT_SUCCESS) return fft_error(r);
        bytes = std::max(bytes, f.work);
    }
    void *area = nullptr;
    if (bytes) {
        const hipError_t e = scratch_alloc(&area, bytes, stream);
        if (e != hipSuccess)
            return set_error(MG_ENOMEM, std::string("FFT work area: ") + hipGetErrorString(e));
    }
    hipfftResult r = HIPFFT_SUCCESS;
    for (int p = 0; p < nplanes && r == HIPFFT_SUCCESS; ++p) {
        const int H = beta * (int)L.planes.S[p];
        if (H <= kCosineMax) continue;
        const int64_t n = (int64_t)(H / 2 + 1) * (H / 2 + 1), m = 4 * (int64_t)H * H;
        hipfftDoubleComplex *img = reinterpret_cast<hipfftDoubleComplex *>(
            ws + L.planes.ws[p] + table_doubles(H) + 2 * n);
        hipLaunchKernelGGL(screen_kernel<true>, dim3((unsigned)std::min<int64_t>((m + 255) / 256, 4096)),
                           dim3(256), 0, stream, L.planes, p, beta, fov, ws);
        {
            // the plan is shared: its stream and work area are set and the
            // transform queued under the lock
            std::lock_guard<std::mutex> lk(g_fft_mu);
            BankFft f;
            r = bank_fft(dev, 2 * H, &f);
            if (r == HIPFFT_SUCCESS) r = hipfftSetStream(f.h, stream);
            if (r == HIPFFT_SUCCESS && f.work) r = hipfftSetWorkArea(f.h, area);
            if (r == HIPFFT_SUCCESS) r = hipfftExecZ2Z(f.h, img, img, HIPFFT_FORWARD);
        }
        if (r == HIPFFT_SUCCESS)
            hipLaunchKernelGGL(quadrant_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)),
                               dim3(256), 0, stream, L.planes, p, beta, ws, mx);
    }
    if (area) scratch_free(area, stream);
    return r == HIPFFT_SUCCESS ? MG_OK : fft_error(r);
}

}  // namespace
}  // namespace mg

using namespace mg;

extern "C" {

mg_status mg_wkernel_bank_size(int32_t nplanes, const int32_t *plane_support, int32_t beta,
                               int64_t *bank_elems, size_t *workspace_bytes) {
    if (!bank_elems || !workspace_bytes) return set_error(MG_EINVAL, "null output");
    Layout L;
    const mg_status st = make_layout(nplanes, plane_support, beta, L);
    if (st != MG_OK) return st;
    *bank_elems = L.bank_elems;
    *workspace_bytes = L.bytes;
    return MG_OK;
}

mg_status mg_wkernel_bank(int32_t nplanes, const int32_t *plane_support, const double *plane_w,
                          int32_t beta, int32_t base_len, const double *base_taps, double fov,
                          mg_dtype out_dtype, void *bank, int64_t *plane_offset, void *workspace,
                          size_t workspace_bytes, hipStream_t stream) {
    Layout L;
    mg_status st = make_layout(nplanes, plane_support, beta, L);
    if (st != MG_OK) return st;
    if (!plane_w || !base_taps || !bank || !plane_offset || !workspace)
        return set_error(MG_EINVAL, "null argument");
    if (workspace_bytes < L.bytes) return set_error(MG_EINVAL, "workspace too small");
    if (base_len < 1 || (base_len % 2) == 0) return set_error(MG_EINVAL, "base table length must be odd");
    if (!(fov > 0.0) || !std::isfinite(fov)) return set_error(MG_EINVAL, "fov must be positive");
    if (out_dtype != MG_F32 && out_dtype != MG_F16 && out_dtype != MG_BF16)
        return set_error(MG_EINVAL, "bank dtype must be MG_F32, MG_F16 or MG_BF16");
    for (int p = 0; p < nplanes; ++p) {
        if (!std::isfinite(plane_w[p])) return set_error(MG_EINVAL, "plane w must be finite");
        if (base_len > beta * plane_support[p] + 1)
            return set_error(MG_EINVAL, "plane support narrower than the base kernel");
        L.planes.w[p] = plane_w[p];
    }
    double *ws = static_cast<double *>(workspace);
    unsigned long long *mx =
        reinterpret_cast<unsigned long long *>(static_cast<char *>(workspace) + L.off_max);
    // grids for the largest plane; the others' spare workgroups have nothing
    // to do
    const int64_t tile_rows = (L.H_cosine + 1 + 15) / 16,
                  tile_cols = (L.H_cosine / 2 + 1 + 15) / 16;
    auto over = [&](int64_t groups) {
        return dim3((unsigned)std::max<int64_t>(1, groups), (unsigned)nplanes);
    };
    auto elems = [&](int64_t side) {
        return over(std::min<int64_t>((side * side + 255) / 256, 4096));
    };
    const dim3 kept = elems(L.H_max + 1);
    hipLaunchKernelGGL(tables_kernel, over((L.H_max + 1 + 3) / 4), dim3(256), 0, stream, L.planes, beta,
                       base_len, base_taps, ws, mx);
    if (L.H_cosine) {
        hipLaunchKernelGGL(screen_kernel<false>, elems(L.H_cosine + 1), dim3(256), 0, stream,
                           L.planes, 0, beta, fov, ws);
        hipLaunchKernelGGL(cosine_kernel<0>, over(tile_rows * tile_cols), dim3(256), 0,
                           stream, L.planes, beta, ws, mx);
        hipLaunchKernelGGL(cosine_kernel<1>, over(tile_cols * tile_cols), dim3(256), 0,
                           stream, L.planes, beta, ws, mx);
    }
    if (L.H_max > kCosineMax) {
        st = large_planes(L, nplanes, beta, fov, ws, mx, stream);
        if (st != MG_OK) return st;
    }
    const unsigned long long *cmx = mx;
    if (out_dtype == MG_F16)
        hipLaunchKernelGGL(store_kernel<__half>, kept, dim3(256), 0, stream, L.planes, beta, ws,
                           cmx, (__half *)bank);
    else if (out_dtype == MG_BF16)
        hipLaunchKernelGGL(store_kernel<__hip_bfloat16>, kept, dim3(256), 0, stream, L.planes,
                           beta, ws, cmx, (__hip_bfloat16 *)bank);
    else
        hipLaunchKernelGGL(store_kernel<float>, kept, dim3(256), 0, stream, L.planes, beta, ws,
                           cmx, (float *)bank);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(MG_EDEVICE, std::string("kernel bank: ") + hipGetErrorString(e));
    for (int p = 0; p < nplanes; ++p) plane_offset[p] = L.planes.bank[p];
    return MG_OK;
}

}  // extern "C"
