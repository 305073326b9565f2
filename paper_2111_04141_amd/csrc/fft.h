// Inverse (exp(+j2pi)) complex FP32 transforms of power-of-two length for the
// imaging chain, in registers and LDS.
//
// Stockham form: a transform of N = 2^LOGN points belongs to N/16 threads of
// 16 points each; every pass is one radix-16 butterfly per thread (the first
// takes the radix 2, 4 or 8 that is left over, 16 / radix butterflies), and
// between passes the points are exchanged through LDS, so 2048 points take
// three passes and two exchanges and the data crosses HBM once each way.
// Twiddles: e^{ja} by its series in FP64 (which runs at the FP32 rate here), the
// powers as FP64 products, each rounded once to FP32: error of a 4 x 2048^2 image
// 1.7e-7 (2.0e-7 with FP32 products of sincospif values, as the platform
// library's), 124 us in place of 128; the layers' columns, whose registers
// are full, pay 1.07 ms in place of 0.88.
#pragma once

#include <hip/hip_runtime.h>

namespace mg {

__device__ inline float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ inline float2 cmul(float2 a, float2 b) {
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}
// a j
__device__ inline float2 cmulj(float2 a) { return make_float2(-a.y, a.x); }

__device__ inline void fft2(float2 &a, float2 &b) {
    const float2 t = csub(a, b);
    a = cadd(a, b);
    b = t;
}

// in place, natural order in and out
__device__ inline void fft4(float2 &a, float2 &b, float2 &c, float2 &d) {
    const float2 s = cadd(a, c), t = csub(a, c), u = cadd(b, d), v = cmulj(csub(b, d));
    a = cadd(s, u);
    b = cadd(t, v);
    c = csub(s, u);
    d = csub(t, v);
}

__device__ inline void fft8(float2 (&x)[8]) {
    constexpr float h = 0.70710678118654752440f;
    float2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    fft4(e[0], e[1], e[2], e[3]);
    fft4(o[0], o[1], o[2], o[3]);
    o[1] = make_float2(h * (o[1].x - o[1].y), h * (o[1].x + o[1].y));    // e^{j pi/4}
    o[2] = cmulj(o[2]);
    o[3] = make_float2(-h * (o[3].x + o[3].y), h * (o[3].x - o[3].y));   // e^{j 3pi/4}
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        x[k] = cadd(e[k], o[k]);
        x[k + 4] = csub(e[k], o[k]);
    }
}

// X[k1 + 4 k2] = sum_{n2} W16^{n2 k1} W4^{n2 k2} sum_{n1} x[4 n1 + n2] W4^{n1 k1}
__device__ inline void fft16(float2 (&x)[16]) {
    constexpr float c1 = 0.92387953251128675613f, s1 = 0.38268343236508977173f;
    constexpr float h = 0.70710678118654752440f;
#pragma unroll
    for (int n = 0; n < 4; ++n) fft4(x[n], x[n + 4], x[n + 8], x[n + 12]);
    // x[4 k1 + n2] times e^{j 2pi n2 k1 / 16}
    x[5] = cmul(x[5], make_float2(c1, s1));
    x[6] = cmul(x[6], make_float2(h, h));
    x[7] = cmul(x[7], make_float2(s1, c1));
    x[9] = cmul(x[9], make_float2(h, h));
    x[10] = cmulj(x[10]);
    x[11] = cmul(x[11], make_float2(-h, h));
    x[13] = cmul(x[13], make_float2(s1, c1));
    x[14] = cmul(x[14], make_float2(-h, h));
    x[15] = cmul(x[15], make_float2(-c1, -s1));
#pragma unroll
    for (int k = 0; k < 4; ++k) fft4(x[4 * k], x[4 * k + 1], x[4 * k + 2], x[4 * k + 3]);
    // x[4 k1 + k2] -> x[k1 + 4 k2]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = a + 1; b < 4; ++b) {
            const float2 t = x[4 * a + b];
            x[4 * a + b] = x[a + 4 * b];
            x[a + 4 * b] = t;
        }
}

struct Phase64 { double x, y; };
__device__ inline Phase64 pmul(Phase64 a, Phase64 b) {
    return {fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x)};
}

// v[r] *= e^{j pi r frac}, r = 1..15, 0 <= frac < 1/8
__device__ inline void twiddle16(float2 (&v)[16], float frac) {
    // Taylor series of an angle below pi / 8: the first terms left out are
    // below 1e-12 (sine) and 6e-14 (cosine)
    const double a = 3.14159265358979323846 * (double)frac, q = a * a;
    double s = fma(q, 1.0 / 362880.0, -1.0 / 5040.0);
    s = fma(q, s, 1.0 / 120.0);
    s = fma(q, s, -1.0 / 6.0);
    double c = fma(q, -1.0 / 3628800.0, 1.0 / 40320.0);
    c = fma(q, c, -1.0 / 720.0);
    c = fma(q, c, 1.0 / 24.0);
    c = fma(q, c, -0.5);
    const Phase64 w1 = {fma(q, c, 1.0), fma(a * q, s, a)};
    const Phase64 w2 = pmul(w1, w1), w3 = pmul(w2, w1), w4 = pmul(w2, w2);
    auto turn = [&](int r, Phase64 w) { v[r] = cmul(v[r], make_float2((float)w.x, (float)w.y)); };
    turn(1, w1);
    turn(2, w2);
    turn(3, w3);
    Phase64 b = w4;
#pragma unroll
    for (int r = 4; r < 16; r += 4) {
        turn(r, b);
        turn(r + 1, pmul(b, w1));
        turn(r + 2, pmul(b, w2));
        turn(r + 3, pmul(b, w3));
        if (r < 12) b = pmul(b, w4);
    }
}

// LDS index of point i: one word of padding per 16 keeps the strided writes of
// an exchange off each other's banks.
__device__ constexpr int fft_pad(int i) { return i + (i >> 4); }
constexpr int fft_points(int logn) { return (1 << logn) + (1 << logn) / 16; }

// The transform of the points v[k] = x[t + k N/16] of thread t (t < N/16); on
// return v[k] = X[t + k N/16].  exchange(put, get): moves the points through
// LDS; put(k) is the index point v[k] goes to, get(k) the one it takes.
template <int LOGN, typename F>
__device__ inline void fft_inverse(float2 (&v)[16], const int t, F &&exchange) {
    constexpr int N = 1 << LOGN, T = N / 16;
    constexpr int REST = LOGN % 4;
    constexpr int R1 = REST == 0 ? 16 : 1 << REST;
    constexpr int Q = 16 / R1;
    // first pass: Q butterflies, butterfly q of points v[q + r Q]
    if constexpr (R1 == 16) {
        fft16(v);
    } else if constexpr (R1 == 8) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float2 x[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) x[r] = v[q + r * Q];
            fft8(x);
#pragma unroll
            for (int r = 0; r < 8; ++r) v[q + r * Q] = x[r];
        }
    } else if constexpr (R1 == 4) {
#pragma unroll
        for (int q = 0; q < Q; ++q) fft4(v[q], v[q + Q], v[q + 2 * Q], v[q + 3 * Q]);
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) fft2(v[q], v[q + Q]);
    }
    // point v[q + r Q] is output r of butterfly j = t + q T: index j R1 + r
    exchange([&](int k) { return (t + (k % Q) * T) * R1 + k / Q; });
#pragma unroll
    for (int ns = R1; ns < N; ns *= 16) {
        const int jm = t & (ns - 1);
        twiddle16(v, (float)jm * (1.0f / (8.0f * (float)ns)));
        fft16(v);
        if (ns * 16 < N) exchange([&](int k) { return (t - jm) * 16 + jm + k * ns; });
    }
}

}  // namespace mg
