// fft1536.hpp -- one 1536-point complex FFT per wavefront, for gfx950 (wave64).
//
// The FP32 chip-rate correlations (length 1023, circular) take the samples in
// two segments of 512, so that a correlation at 1023 lags needs 512 + 1023 - 1
// <= 1536 points instead of 2048: with g = g_0 + g_1 (samples 0..511 and
// 512..1022) and cc_i[u] = C[(512 i + u) mod 1023] at u in [-1022, 511] (mod
// 1536),
//   R[q] = IDFT_1536(sum_i DFT_1536(g_i) conj(DFT_1536(cc_i)))[q] / 1536.
//
// 1536 = 512 x 3 with coprime factors, so the transform is 512-point DFTs and
// 3-point DFTs with no twiddles between them (Good-Thomas):
//   spectral index k = (3 kappa + 512 c) mod 1536, kappa < 512, c < 3
//   natural index  q: i = q mod 512, d = q mod 3
//   x[q] = sum_c W3^(c d) sum_kappa X[k(kappa, c)] W512^(kappa i),  W_L = e^(+2 pi i / L).
// A 512-point DFT is 8 x 8 x 8 on eight registers per lane:
//   kappa = 64 n1 + l, l = 8 m1 + m2;  i = k1 + 8 k2a + 64 k2b
//   radix-8 over n1 -> LDS exchange A -> W512^(l k1), radix-8 over m1 ->
//   LDS exchange B -> W64^(m2 k2a), radix-8 over m2.
// The twiddles are the same for the three values of c and are applied after
// the exchanges, within the next pass's first stage.
//
// Storage order: lane l, register 8 c + n1 holds kappa = 64 n1 + l; a stored
// spectrum is 768 float4, float4 64 (4 c + p) + l holding registers 8 c + 2 p
// and 8 c + 2 p + 1 of lane l.  Natural order: lane l, register k2b holds i =
// l + 64 k2b.  The forward transform is the exact adjoint of the inverse.
#pragma once

#include "fft2048.hpp"

namespace gnss {

constexpr int kSeg3 = 512;            // samples of a segment (the second one has 511)
constexpr int kLen3 = 1536;
constexpr int kSpec3 = 768;           // float4 per stored segment spectrum
constexpr int kVec3 = 2 * kSpec3;     // float4 per polyphase vector (two segments)
// code spectra (divided by 3): the c = 0 and c = 1 thirds only (the code is real, so
// X[2][kappa] = conj X[1][-kappa])
constexpr int kCode3 = 2 * 2 * kSeg3;  // float2 per PRN: [segment][c < 2][kappa]
// in LDS with a copy of kappa = 0 at kappa = 512 of c = 1 (mirrored reads)
constexpr int kCodeLds3 = 2 * (2 * kSeg3 + 1);

// LDS scratch of a wave, in float2.  Both exchanges hit 16 distinct 8-byte
// banks per 16 lanes: A writes rows k1 of 64 with stride 72 (= 8 mod 16: its
// reads take 2 rows x 8 columns), B is indexed k1 + 8 k2a + 66 m2 (66 = 2 mod
// 16: its writes take 2 k1 x 8 m2, its reads 16 consecutive).
constexpr int kStrideA3 = 72, kStrideB3 = 66;
constexpr int kXbuf3 = 8 * kStrideA3;

// The lane's twiddles and 3-point coefficients, 36 registers held for the
// whole kernel: with the twiddles in LDS the correlation kernel was bound by LDS
// bandwidth (97 KB per transform instead of 74; 2.88 against 2.56 ms for the
// weak-signal search).
struct Lane3 {
    float2 t1[8];  // after exchange A, lane l = 8 k1 + m2: W512^((8 m1 + m2) k1)
    float2 t2[7];  // after exchange B, lane l = k1 + 8 k2a: W64^(m2 k2a), m2 = 1..7
    float al[3], be[3];  // W3^d = al + i be of d = (l + t) mod 3, t < 3
    // twg: the table of e^(-2 pi i j / 32768)
    __device__ __forceinline__ Lane3(const float2 *twg, int l)
    {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const float2 a = twg[64 * ((8 * m + (l & 7)) * (l >> 3))];
            t1[m] = make_float2(a.x, -a.y);
        }
#pragma unroll
        for (int m = 0; m < 7; ++m) {
            const float2 a = twg[512 * (m + 1) * (l >> 3)];
            t2[m] = make_float2(a.x, -a.y);
        }
        const int r = l % 3;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int d = (r + t) % 3;
            al[t] = d == 0 ? 1.f : -0.5f;
            be[t] = d == 0 ? 0.f : d == 1 ? 0.86602540378443864676f : -0.86602540378443864676f;
        }
    }
};

// Inverse radix-8 pass of values a[n] with twiddles w(n): the first stage's
// second product is added onto the first, a[n] - a[n + 4] = 2 a[n] - (a[n] +
// a[n + 4]): two instructions less per butterfly than products and sums apart.
// ONE: w(0) = 1.
template <bool ONE, typename W>
__device__ __forceinline__ void dft8_twiddled(float2 (&a)[8], W w)
{
    float2 s[4], d[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const float2 z = ONE && n == 0 ? a[0] : c_mul(a[n], w(n));
        s[n] = c_mul_add(a[n + 4], w(n + 4), z);
        d[n] = make_float2(fmaf(2.f, z.x, -s[n].x), fmaf(2.f, z.y, -s[n].y));
    }
    dft8_rest<true>(s, d, a);
}

template <bool INV>
__device__ __forceinline__ void dft8_plain(float2 (&a)[8])
{
    float2 s[4], d[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        s[n] = c_add(a[n], a[n + 4]);
        d[n] = c_sub(a[n], a[n + 4]);
    }
    dft8_rest<INV>(s, d, a);
}

// Inverse 512-point transform after its first radix-8 pass: storage order in,
// natural order out.
__device__ __forceinline__ void ifft512_rest(float2 (&v)[8], float2 *xb, const Lane3 &w, int l)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) xb[k * kStrideA3 + l] = v[k];
    wave_lds_order();
    const float2 *src = xb + (l >> 3) * kStrideA3 + (l & 7);
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = src[8 * m];
    wave_lds_order();
    dft8_twiddled<false>(v, [&](int m) { return w.t1[m]; });
    float2 *dst = xb + (l >> 3) + kStrideB3 * (l & 7);
#pragma unroll
    for (int k = 0; k < 8; ++k) dst[8 * k] = v[k];
    wave_lds_order();
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = xb[l + kStrideB3 * m];
    wave_lds_order();
    dft8_twiddled<true>(v, [&](int m) { return w.t2[m - 1]; });
}

// Forward 512-point transform, the adjoint: natural order in, storage order out.
__device__ __forceinline__ void fft512(float2 (&v)[8], float2 *xb, const Lane3 &w, int l)
{
    dft8_plain<false>(v);
#pragma unroll
    for (int m = 0; m < 8; ++m) xb[l + kStrideB3 * m] = m ? c_mulc(v[m], w.t2[m - 1]) : v[0];
    wave_lds_order();
    const float2 *src = xb + (l >> 3) + kStrideB3 * (l & 7);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = src[8 * k];
    wave_lds_order();
    dft8_plain<false>(v);
    float2 *dst = xb + (l >> 3) * kStrideA3 + (l & 7);
#pragma unroll
    for (int m = 0; m < 8; ++m) dst[8 * m] = c_mulc(v[m], w.t1[m]);
    wave_lds_order();
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = xb[k * kStrideA3 + l];
    wave_lds_order();
    dft8_plain<false>(v);
}

// The 3-point DFTs of the inverse for natural indices q < 1024 (i < 512: q =
// i, d = i mod 3, and q = i + 512, d = (i + 2) mod 3; the third output, q = i +
// 1024, is not a lag): f(j, value) for q = l + 64 j, j < 16.
template <typename Sink>
__device__ __forceinline__ void lags3(const float2 (&v)[3][8], const Lane3 &w, Sink f)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float2 x = v[0][j], s = c_add(v[1][j], v[2][j]), e = c_sub(v[1][j], v[2][j]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float a = w.al[(j + 2 * h) % 3], b = w.be[(j + 2 * h) % 3];
            f(j + 8 * h, make_float2(fmaf(-b, e.y, fmaf(a, s.x, x.x)), fmaf(b, e.x, fmaf(a, s.y, x.y))));
        }
    }
}

// Third c of the forward transform of a segment, x[j] = sample l + 64 j (j < 8;
// zero above 511): v in storage order.
template <int C>
__device__ __forceinline__ void fft1536_seg(const float2 (&x)[8], float2 (&v)[8], float2 *xb, const Lane3 &w, int l)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if constexpr (C == 0) {
            v[j] = x[j];
        } else {  // times W3^(-c d), d = i mod 3
            const float a = w.al[j % 3], b = C == 1 ? w.be[j % 3] : -w.be[j % 3];
            v[j] = make_float2(fmaf(b, x[j].y, a * x[j].x), fmaf(-b, x[j].x, a * x[j].y));
        }
    }
    fft512(v, xb, w, l);
}

}  // namespace gnss
