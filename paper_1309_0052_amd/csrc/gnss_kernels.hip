// gnss_kernels.hip -- HIP kernels (gfx950) of the GPS L1 C/A acquisition search.
//
// The acquisition channel of the paper (Sec. 3, Fig. 2): code and carrier
// NCOs, first mixing stage, FFTs of mixed signal and code replica, second
// mixing (spectrum product), IFFT, detection; block processing (Sec. 4) and
// batching of the whole coherent integration on the device (Sec. 5).
//
// Correlation in polyphase form.  With spc = fs/1.023 MHz integer samples per
// chip the code replica is c[n] = C[floor(n/spc)] (C the +-1 chip code), so
// for the folded block f (length N = 1023 spc) the circular correlation
//   R[tau] = sum_n f[n] c[(n - tau) mod N]
// at tau = spc q + s equals the length-1023 circular correlation
//   R[spc q + s] = sum_m g_s[m] C[(m - q) mod 1023],
//   g_s[m] = F[spc m + s],  F[n] = sum_{t<spc} f[(n + t) mod N]
// (a boxcar over one chip, then a polyphase split).  Each g_s is correlated
// with the chip-rate code through zero-padded transforms (padding makes the
// circular length-1023 correlation a linear one), so one code spectrum per PRN
// serves every sample rate, and each transform lives in one wavefront's
// registers.  FP32 contexts take g_s in two segments on 1536-point transforms
// (fft1536.hpp), FP16 ones 2048-point transforms (fft2048.hpp).
//
// Kernel sequence of a batch (every kernel walks a device table of the batch's
// requests; a single request is a batch of one):
//   k_meta           the request table (small batches; larger ones by a copy);
//                    k_reset clears its work counters where a table is used again
//   k_box_fft        NCO wipe-off + coherent fold + boxcar + polyphase split
//                    (exact int32) + forward FFT of every g_s -> G (storage order)
//   k_corr           per (PRN tile, Doppler, phase): G * conj(code spectrum),
//                    IFFT, |.|^2, sum over blocks in registers -> grid
//   k_colmax/k_peak  column max over Doppler, argmax, second peak, mean, FP64
//                    parabolic refinement
// FP16 contexts use k_box (the polyphase values to memory, F[k][b][s][1024]),
// k_fft_poly_h and k_corr_h (packed half precision with per-vector
// power-of-two scaling).  k_track computes the tracking channel's
// early / prompt / late correlators (Fig. 3).
#include "fft1536.hpp"
#include "fft2048.hpp"
#include "gnss_internal.hpp"
#include "pfa1023.hpp"

#include <math.h>
#include <string.h>

#include <algorithm>

namespace gnss {

// Device pointers of a request live in the request table, so the compiler
// cannot tell that they address global memory; these casts let it use global
// (not flat) loads and stores for them.
#define GNSS_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GNSS_GLOBAL T *gmem(T *p)
{
    return (GNSS_GLOBAL T *)p;
}

typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// f(std::integral_constant<int, i>()) for i < N, in order
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        unrolled<N, I + 1>(f);
    }
}

// A workgroup-uniform 64-bit value in scalar registers.
__device__ __forceinline__ long long uniform64(long long v)
{
    const unsigned long long u = (unsigned long long)v;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}


// ===========================================================================
// C/A codes (IS-GPS-200 Table 3-Ia), G2-delay construction
// ===========================================================================
// G2 delay in chips for PRN 1..37: chip_n = G1_n xor G2_(n - delay).
__constant__ int16_t c_g2_delay[kMaxPrn] = {
    5,   6,   7,   8,   17,  18,  139, 140, 141, 251, 252, 254, 255, 256, 257, 258, 469, 470, 471,
    472, 473, 474, 509, 512, 513, 514, 515, 516, 859, 860, 861, 862, 863, 950, 947, 948, 950};

// 10-stage registers, stage i in bit i-1, output is stage 10 (bit 9).
__device__ __forceinline__ uint32_t g1_next(uint32_t r)
{
    uint32_t fb = ((r >> 2) ^ (r >> 9)) & 1u;  // stages 3, 10
    return ((r << 1) | fb) & 0x3FFu;
}
__device__ __forceinline__ uint32_t g2_next(uint32_t r)
{
    uint32_t fb = ((r >> 1) ^ (r >> 2) ^ (r >> 5) ^ (r >> 7) ^ (r >> 8) ^ (r >> 9)) & 1u;  // 2,3,6,8,9,10
    return ((r << 1) | fb) & 0x3FFu;
}

// One thread per PRN row (row 0 is all zeros).  codes is [38][1023].
__global__ void k_gold_codes(uint8_t *codes)
{
    int prn = threadIdx.x;
    if (prn > kMaxPrn) return;
    uint8_t *row = codes + prn * kCodeLen;
    if (prn == 0) {
        for (int n = 0; n < kCodeLen; ++n) row[n] = 0;
        return;
    }
    const int delay = c_g2_delay[prn - 1];
    uint32_t g1 = 0x3FFu, g2 = 0x3FFu;
    // bring G2 to sequence index (-delay mod 1023)
    for (int i = 0; i < (kCodeLen - delay) % kCodeLen; ++i) g2 = g2_next(g2);
    for (int n = 0; n < kCodeLen; ++n) {
        row[n] = (uint8_t)(((g1 ^ g2) >> 9) & 1u);
        g1 = g1_next(g1);
        g2 = g2_next(g2);
    }
}

hipError_t launch_gold_codes(uint8_t *d_codes, hipStream_t s)
{
    hipLaunchKernelGGL(k_gold_codes, dim3(1), dim3(64), 0, s, d_codes);
    return hipGetLastError();
}

// Code replica at sample rate fs: out[i*n + m] = 1 - 2 code[floor(m*1023000/fs) mod 1023].
__global__ void k_code_replica(const uint8_t *codes, PrnList prns, int n_prn, long long fs_hz,
                               long long n, int8_t *out)
{
    const long long total = (long long)n_prn * n;
    for (long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x; idx < total;
         idx += (long long)gridDim.x * blockDim.x) {
        long long i = idx / n, m = idx - i * n;
        long long chip = (m * 1023000LL) / fs_hz;
        int bit = codes[prns.v[i] * kCodeLen + (int)(chip % kCodeLen)];
        out[idx] = (int8_t)(1 - 2 * bit);
    }
}

hipError_t launch_code_replica(const uint8_t *d_codes, PrnList prns, int n_prn, int64_t fs_hz,
                               int64_t n, int8_t *d_out, hipStream_t s)
{
    long long total = (long long)n_prn * n;
    long long blocks = (total + 255) / 256;
    if (blocks > 65535) blocks = 65535;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_code_replica, dim3((unsigned)blocks), dim3(256), 0, s, d_codes, prns,
                       n_prn, (long long)fs_hz, (long long)n, d_out);
    return hipGetLastError();
}

// ===========================================================================
// carrier LUT and FFT twiddles
// ===========================================================================
// packed[i] = (uint16)cos16 | (uint16)sin16 << 16, values lround(4096 cos/sin(2 pi i/1024)).
__global__ void k_lut(uint32_t *packed, int16_t *cosL, int16_t *sinL)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 1024) return;
    double s, c;
    sincospi((double)i / 512.0, &s, &c);
    int ci = (int)llround(4096.0 * c);
    int si = (int)llround(4096.0 * s);
    if (packed) packed[i] = (uint32_t)(uint16_t)(int16_t)ci | ((uint32_t)(uint16_t)(int16_t)si << 16);
    if (cosL) cosL[i] = (int16_t)ci;
    if (sinL) sinL[i] = (int16_t)si;
}

hipError_t launch_lut(uint32_t *d_lut_packed, int16_t *d_cos, int16_t *d_sin, hipStream_t s)
{
    hipLaunchKernelGGL(k_lut, dim3(4), dim3(256), 0, s, d_lut_packed, d_cos, d_sin);
    return hipGetLastError();
}

__global__ void k_twiddles(float2 *tw)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    double s, c;
    if (i < kT1Elems) {
        int hk = i >> 6, l = i & 63;
        int h = hk >> 4, k1 = hk & 15;
        int e = ((l + 64 * h) * k1) & 2047;  // angle 2 pi e / 2048
        sincospi((double)e / 1024.0, &s, &c);
        tw[i] = make_float2((float)c, (float)s);
    } else if (i < kTwElems) {
        int j = i - kT1Elems;
        int k2a = j >> 3, m2 = j & 7;
        int e = (m2 * k2a) & 127;  // angle 2 pi e / 128
        sincospi((double)e / 64.0, &s, &c);
        tw[i] = make_float2((float)c, (float)s);
    }
}

hipError_t launch_twiddles(float2 *d_tw, hipStream_t s)
{
    hipLaunchKernelGGL(k_twiddles, dim3((kTwElems + 255) / 256), dim3(256), 0, s, d_tw);
    return hipGetLastError();
}

__device__ __forceinline__ void stage_twiddles(float2 *s_tw, const float2 *tw, int tid, int nthreads)
{
    for (int i = tid; i < kTwElems; i += nthreads) s_tw[i] = tw[i];
}

// ===========================================================================
// code spectra: CS[prn] = conj(FFT_2048(cc_prn)) in storage order, where
// cc[i] = C[i] (i < 1023), 0 (1023..1025), C[i - 1025] (1026..2047), so that
// IFFT_2048(FFT(g0) * CS)[q] = 2048 * sum_m g[m] C[(m - q) mod 1023] for q < 1023.
// ===========================================================================
__global__ __launch_bounds__(256) void k_code_spectra(const uint8_t *codes, const float2 *tw,
                                                      float4 *cs)
{
    __shared__ float2 s_tw[kTwElems];
    __shared__ float2 s_xb[4][kXbufElems];
    stage_twiddles(s_tw, tw, threadIdx.x, 256);
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int prn = blockIdx.x * 4 + w;
    if (prn > kMaxPrn) return;
    const uint8_t *code = codes + prn * kCodeLen;
    float2 v[32];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k2b = 0; k2b < 8; ++k2b) {
            int q = l + 64 * u + 256 * k2b;
            float val = 0.f;
            if (prn != 0) {
                if (q < kCodeLen)
                    val = 1.f - 2.f * (float)code[q];
                else if (q >= 1026)
                    val = 1.f - 2.f * (float)code[q - 1025];
            }
            v[8 * u + k2b] = make_float2(val, 0.f);
        }
    fft2048<false>(v, s_xb[w], s_tw, s_tw + kT1Elems, l);
    float4 *dst = cs + (long long)prn * kVec;
#pragma unroll
    for (int jj = 0; jj < 16; ++jj)
        dst[jj * 64 + l] = make_float4(v[2 * jj].x, -v[2 * jj].y, v[2 * jj + 1].x, -v[2 * jj + 1].y);
}

// FP32 contexts: conj(DFT_1536(cc_i)) / 3 of the two segments' replicas (see
// fft1536.hpp), the c < 2 thirds, [prn][segment][c][kappa], in FP64 and rounded
// once; row 0 is all zeros.  One thread per value.  (The third keeps the powers of
// integer correlations whole multiples of a power of two: with samples of few bits
// and a carrier at a quarter of the rate the sums over blocks are then exact, as on
// transforms of 2^k points.  With the factor 9 of an unscaled 1536-point transform in
// them they round, for equal blocks the same way every time: up to 5e-6 off after
// 256 blocks.)
__global__ __launch_bounds__(256) void k_code_spectra3(const uint8_t *codes, float2 *cs)
{
    __shared__ double2 s_w[kLen3];
    __shared__ int8_t s_c[kCodeLen];
    const int prn = blockIdx.y, idx = blockIdx.x * 256 + threadIdx.x;
    for (int i = threadIdx.x; i < kLen3; i += 256) {
        double sn, cn;
        sincospi((double)i / (kLen3 / 2), &sn, &cn);
        s_w[i] = make_double2(cn, sn);
    }
    for (int i = threadIdx.x; i < kCodeLen; i += 256) s_c[i] = prn ? (int8_t)(1 - 2 * (int)codes[prn * kCodeLen + i]) : 0;
    __syncthreads();
    const int seg = idx >> 10, c = (idx >> 9) & 1, k = (3 * (idx & 511) + 512 * c) % kLen3;
    double re = 0.0, im = 0.0;
    // u in [-1022, 511]: cc[u] = C[(512 seg + u) mod 1023], times e^(2 pi i k u / 1536)
    int j = (kSeg3 * seg + 1) % kCodeLen, e = (int)((long long)k * (kLen3 - (kCodeLen - 1)) % kLen3);
    for (int u = -(kCodeLen - 1); u < kSeg3; ++u) {
        re += s_c[j] * s_w[e].x;
        im += s_c[j] * s_w[e].y;
        if (++j == kCodeLen) j = 0;
        e += k;
        if (e >= kLen3) e -= kLen3;
    }
    cs[(long long)prn * kCode3 + idx] = make_float2((float)(re / 3.0), (float)(im / 3.0));
}

hipError_t launch_code_spectra3(const uint8_t *d_codes, float2 *d_cs, hipStream_t s)
{
    hipLaunchKernelGGL(k_code_spectra3, dim3(kCode3 / 256, kMaxPrn + 1), dim3(256), 0, s, d_codes, d_cs);
    return hipGetLastError();
}

hipError_t launch_code_spectra(const uint8_t *d_codes, const float2 *d_tw, float4 *d_cs,
                               hipStream_t s)
{
    hipLaunchKernelGGL(k_code_spectra, dim3((kMaxPrn + 1 + 3) / 4), dim3(256), 0, s, d_codes,
                       d_tw, d_cs);
    return hipGetLastError();
}

__device__ __forceinline__ void load_sample(const void *samples, int fmt, long long n, int &xr, int &xi)
{
    if (fmt == GNSS_CPLX_I8) {
        const uint32_t v = ((const GNSS_GLOBAL uint16_t *)samples)[n];  // I in the low byte
        xr = (int)(int8_t)(v & 0xFFu);
        xi = (int)(int8_t)(v >> 8);
    } else if (fmt == GNSS_REAL_I8) {
        xr = ((const GNSS_GLOBAL int8_t *)samples)[n];
        xi = 0;
    } else {
        uint32_t byte = ((const GNSS_GLOBAL uint8_t *)samples)[n >> 2];
        uint32_t code = (byte >> (2 * (uint32_t)(n & 3))) & 3u;
        // 00:+1 01:+3 10:-1 11:-3
        int mag = (code & 1u) ? 3 : 1;
        xr = (code & 2u) ? -mag : mag;
        xi = 0;
    }
}

// y[n] = x[n] * (cosL - j sinL)[phase(n) >> 22], summed over the Tc
// milliseconds of coherent block b at in-block offset m.
__device__ __forceinline__ int2 wipe_fold_one(const void *samples, int fmt, int N, int Tc,
                                              const uint32_t *lut, uint32_t D, int b, int m)
{
    int yr = 0, yi = 0;
    for (int c = 0; c < Tc; ++c) {
        long long ng = (long long)(b * Tc + c) * N + m;
        int xr, xi;
        load_sample(samples, fmt, ng, xr, xi);
        uint32_t ph = (uint32_t)(unsigned long long)ng * D;
        uint32_t e = lut[ph >> 22];
        int cs = (int)(int16_t)(e & 0xFFFFu), sn = (int)(int16_t)(e >> 16);
        yr += xr * cs + xi * sn;
        yi += xi * cs - xr * sn;
    }
    return make_int2(yr, yi);
}

// Standalone wipe + fold (stage entry) of request 0 of a staged batch:
// out[((k*Nnc + b)*N + m)*2 + {0,1}].
__global__ __launch_bounds__(256) void k_wipe_fold(const ReqDesc *__restrict__ R, const uint32_t *lut, int2 *out)
{
    __shared__ uint32_t s_lut[1024];
    for (int i = threadIdx.x; i < 1024; i += 256) s_lut[i] = lut[i];
    const ReqDesc &d = R[0];
    const int k = blockIdx.x / d.Nnc, b = blockIdx.x % d.Nnc;
    const uint32_t D = d.dk[k];
    __syncthreads();
    int2 *dst = out + (long long)blockIdx.x * d.N;
    for (int m = threadIdx.x; m < d.N; m += 256)
        dst[m] = wipe_fold_one(d.samples, d.fmt, d.N, d.Tc, s_lut, D, d.b0 + b, m);
}

hipError_t launch_wipe_fold(const Launch &L, const Plan &p, const uint32_t *d_lut, int32_t *d_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_wipe_fold, dim3(p.n_dopp * p.Nnc), dim3(256), 0, s, L.reqs, d_lut, (int2 *)d_out);
    return hipGetLastError();
}

// ===========================================================================
// batch plumbing
// ===========================================================================
// Request owning work item `it` of a stage: the last r with pre[r] <= it.
__device__ __forceinline__ int find_req(const long long *pre, int n_req, long long it)
{
    int lo = 0, hi = n_req - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= it) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// A request's first item.  A single request's is not loaded: that load would
// stand between the batch's header and the request's fields, a memory latency
// in each of a search's kernels.
__device__ __forceinline__ long long first_item(const long long *pre, int n_req, int r)
{
    return n_req == 1 ? 0 : pre[r];
}

// Metadata of small batches as a kernel argument (by value, so the host keeps
// no staging buffer and waits for nothing): one launch writes it, in place of
// a copy through the DMA engine and the counters' reset after it.  One
// strong-signal search spent 19 us between the previous one's last kernel and
// its first on that copy, its queue's wait and the reset, and spends 5 us
// (129 -> 97 us a call with 32 PRNs x 21 bins x 10 blocks, 108 before this).
template <int N>
struct MetaArg {
    uint4 v[N];
};
template <int N>
__global__ __launch_bounds__(256) void k_meta(const MetaArg<N> a, uint4 *dst, int n)
{
    const int i = threadIdx.x;
    if (i < n) dst[i] = a.v[i];
}

template <int N>
static hipError_t launch_meta_n(const void *src, size_t bytes, void *dst, hipStream_t s)
{
    MetaArg<N> a;
    const size_t n = (bytes + 15) / 16;
    memcpy(a.v, src, bytes);
    memset((char *)a.v + bytes, 0, n * 16 - bytes);
    hipLaunchKernelGGL(k_meta<N>, dim3(1), dim3(256), 0, s, a, (uint4 *)dst, (int)n);
    return hipGetLastError();
}

hipError_t launch_meta(const void *src, size_t bytes, void *dst, hipStream_t s)
{
    return bytes <= 64 * 16    ? launch_meta_n<64>(src, bytes, dst, s)
           : bytes <= 128 * 16 ? launch_meta_n<128>(src, bytes, dst, s)
                               : launch_meta_n<kMetaArgBytes / 16>(src, bytes, dst, s);
}

__global__ void k_reset(BatchHdr *h)
{
    int i = threadIdx.x;
    if (i < kNumStages * kXcds) h->counter[i] = 0u;
}

// Work distribution.  A stage launched with at least one workgroup per item
// runs one item per workgroup; the ids are dealt so that each XCD (workgroups
// go to the 8 XCDs round-robin) takes a contiguous range of items, which share
// data through that XCD's L2.  A persistent launch (fewer workgroups than
// items) instead splits the items into 8 contiguous ranges, one per XCD; each
// workgroup takes the next item of its own XCD's range from that XCD's
// counter and, once that range is exhausted, takes items from the others.
// Returns -1 when no item is left.  Called by every thread of the workgroup;
// `first` is true on the first call.
__device__ __forceinline__ long long xcd_remap(long long bid, long long nwg)
{
    const long long q = nwg / kXcds, r = nwg % kXcds;
    const long long xcd = bid % kXcds, local = bid / kXcds;
    return xcd < r ? xcd * (q + 1) + local : r * (q + 1) + (xcd - r) * q + local;
}

__device__ __forceinline__ long long next_item(BatchHdr *h, int stage, long long total, long long *s_item,
                                               bool &first)
{
    if ((long long)gridDim.x >= total) {
        if (!first) return -1;
        first = false;
        const long long id = xcd_remap(blockIdx.x, gridDim.x);
        return id < total ? id : -1;
    }
    first = false;
    const long long per = (total + kXcds - 1) / kXcds;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long found = -1;
        const int home = blockIdx.x % kXcds;
        for (int t = 0; t < kXcds; ++t) {
            const int x = (home + t) % kXcds;
            const long long lo = (long long)x * per;
            const long long hi = min(total, lo + per);
            if (lo >= hi) continue;
            const unsigned int got = atomicAdd(&h->counter[stage * kXcds + x], 1u);
            if (lo + (long long)got < hi) {
                found = lo + (long long)got;
                break;
            }
        }
        *s_item = found;
    }
    __syncthreads();
    return uniform64(*s_item);
}

// ===========================================================================
// stage A1: wipe + fold, then the one-chip boxcar
// F[n] = sum_{t<spc} f[(n+t) mod N], split by phase: F[spc m + s] (m < 1023) at
// element m of phase s, 0 at m = 1023.  All integer, exact.
// ===========================================================================
// Mixing by integer dot products.  A sample as two 16-bit halves (re, im) and
// a table entry {(cos, sin), (-sin, cos)} give y = x (cos - j sin), added to
// (yr, yi), in two v_dot2_i32_i16: exact (|x| <= 127, |LUT| <= 4096, 32-bit
// sums), 7 vector instructions per sample with decode and phase where
// separate bytes and products took about 20.
typedef short s2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void mix_add(s2v x, uint2 e, int &yr, int &yi)
{
    yr = __builtin_amdgcn_sdot2(x, __builtin_bit_cast(s2v, e.x), yr, false);
    yi = __builtin_amdgcn_sdot2(x, __builtin_bit_cast(s2v, e.y), yi, false);
}
// The table in LDS from the packed (cos, sin) one.
__device__ __forceinline__ void stage_mix_lut(uint2 *s_lut, const uint32_t *lut, int tid, int nthreads)
{
    for (int i = tid; i < 1024; i += nthreads) {
        const uint32_t v = lut[i];
        s_lut[i] = make_uint2(v, ((0u - (v >> 16)) & 0xFFFFu) | (v << 16));
    }
}
// Sample `off` (bytes; sample index if packed) of a record segment at p.
template <int FMT>
__device__ __forceinline__ s2v load_mix(const GNSS_GLOBAL uint8_t *p, uint32_t off)
{
    if constexpr (FMT == GNSS_CPLX_I8) {
        const uint32_t v = *(const GNSS_GLOBAL uint16_t *)(p + off);  // I in the low byte
        // (256 I, 256 Q), then the sign-extending shifts
        return __builtin_bit_cast(s2v, __builtin_amdgcn_perm(v, v, 0x010C000Cu)) >> 8;
    } else if constexpr (FMT == GNSS_REAL_I8) {
        return s2v{(short)(int8_t)p[off], 0};
    } else {
        const uint32_t code = (p[off >> 2] >> (2u * (off & 3u))) & 3u;
        // 00:+1 01:+3 10:-1 11:-3
        const int mag = (code & 1u) ? 3 : 1;
        return s2v{(short)((code & 2u) ? -mag : mag), 0};
    }
}

constexpr int kBfThreads = 512, kBfSlots = 16;
// The folded samples in LDS, one row of spc per m (the runs the boxcars read),
// rows an odd number of 8-byte slots apart: no bank conflicts between lanes that
// read different rows.  row_inv: i / spc as (i row_inv) >> 18, exact below 2^14.
__device__ __forceinline__ uint32_t row_inv(int spc) { return (spc & 1) ? 0u : (1u << 18) / (uint32_t)spc + 1u; }
__device__ __forceinline__ int row_pad(int i, uint32_t inv) { return i + (int)(__umul24((uint32_t)i, inv) >> 18); }
static_assert(2 * (kBfSlots * kXbuf3 + 1024) * 8 <= 160 * 1024, "two workgroups of k_box_fft per CU");
static_assert((kSeg3 + 1) * (kMaxSpc + 1) <= kBfSlots * kXbuf3 && (2 * kSeg3 - 1) * 9 + 8 <= kBfSlots * kXbuf3,
              "samples and transforms share the LDS");

// Wipe + fold of samples n0 + i, i = i0 + tid + 512 j < len (j < J), of block b
// into s_f, the J samples' loads of a millisecond in flight together; the phase
// of the folded milliseconds advances by N D (mod 2^32) from one to the next.
// Same values as wipe_fold_one.  Samples are addressed from the block's first byte
// (the same pointer in every thread) by 32-bit in-block offsets: a block holds
// Tc N <= 64 * 16368 samples.
template <int FMT, int J>
__device__ __forceinline__ void bf_wipe(const ReqDesc &d, const uint2 *s_lut, uint32_t D, int b, int n0, int i0,
                                        int len, uint32_t inv, int2 *s_f)
{
    const int N = d.N, Tc = d.Tc;
    const uint32_t dN = (uint32_t)N * D;
    const long long base = (long long)b * Tc * N;
    // 2-bit packed records: the block may start inside a byte
    const uint32_t sub = FMT == GNSS_REAL_2BIT_PACKED ? (uint32_t)(base & 3) : 0u;
    const long long blk_byte = FMT == GNSS_CPLX_I8 ? 2 * base : FMT == GNSS_REAL_I8 ? base : (base >> 2);
    const GNSS_GLOBAL uint8_t *blk = (const GNSS_GLOBAL uint8_t *)d.samples + blk_byte;
    const uint32_t step = FMT == GNSS_CPLX_I8 ? 2u * (uint32_t)N : (uint32_t)N;  // bytes (samples if packed)
    constexpr uint32_t kUnit = FMT == GNSS_CPLX_I8 ? 2u : 1u;
    uint32_t off[J], ph[J];
    int yr[J], yi[J];
    const int na = n0 + i0 + (int)threadIdx.x;
    const uint32_t ph0 = (uint32_t)(base + n0 + i0 + (int)threadIdx.x) * D;
    const bool whole = n0 + i0 >= 0 && n0 + i0 + kBfThreads * J <= N;  // no sample past either end
#pragma unroll
    for (int j = 0; j < J; ++j) {
        ph[j] = ph0 + (uint32_t)(kBfThreads * j) * D;
        off[j] = kUnit * (uint32_t)(na + kBfThreads * j) + sub;
        yr[j] = 0;
        yi[j] = 0;
    }
    if (!whole) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            int n = na + kBfThreads * j;  // in (-N, 2N): the block read circularly, N D (mod 2^32) of phase back or on
            if (n < 0) {
                n += N;
                ph[j] += dN;
            }
            if (n >= N) {
                n -= N;
                ph[j] -= dN;
            }
            if (i0 + (int)threadIdx.x + kBfThreads * j >= len) n = 0;  // not stored
            off[j] = kUnit * (uint32_t)n + sub;
        }
    }
#pragma unroll 1
    for (int c = 0; c < Tc; ++c) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            mix_add(load_mix<FMT>(blk, off[j]), s_lut[ph[j] >> 22], yr[j], yi[j]);
            if (FMT == GNSS_REAL_2BIT_PACKED) off[j] += step;
            ph[j] += dN;
        }
        if (FMT != GNSS_REAL_2BIT_PACKED) blk += step;
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = i0 + (int)threadIdx.x + kBfThreads * j;
        if (i < len) s_f[row_pad(i, inv)] = make_int2(yr[j], yi[j]);
    }
}

// In batches of 8, 4 and 1 samples per thread: 8 loads in flight while more than 4 x
// 512 samples are left.  At 4, 8 and 16 samples per chip the parts are whole batches;
// elsewhere a batch's rest is mixed and not stored (a quarter of it at 3 samples per
// chip and of the first part at 9 and 12, half at 1).
template <int FMT>
__device__ __forceinline__ void bf_wipe_all(const ReqDesc &d, const uint2 *s_lut, uint32_t D, int b, int n0, int len,
                                            uint32_t inv, int2 *s_f)
{
    int i0 = 0;
    for (; len - i0 > 4 * kBfThreads; i0 += 8 * kBfThreads) bf_wipe<FMT, 8>(d, s_lut, D, b, n0, i0, len, inv, s_f);
    for (; len - i0 > kBfThreads; i0 += 4 * kBfThreads) bf_wipe<FMT, 4>(d, s_lut, D, b, n0, i0, len, inv, s_f);
    // the rest of up to 512 (a part's halo), by the waves that have any of it
    if (i0 + (int)(threadIdx.x & ~63u) < len) bf_wipe<FMT, 1>(d, s_lut, D, b, n0, i0, len, inv, s_f);
}

// F[S m + s], s < S, of one m: the sum of the row's S samples, then from one output
// to the next a sample in (of the next row) and one out.
template <int S, typename P2>
__device__ __forceinline__ void bf_boxcar(const int2 *s_f, int m, P2 (&o)[16], int at)
{
    constexpr int kRow = S | 1;
    const int2 *run = s_f + m * kRow;
    int2 a[S];
#pragma unroll
    for (int t = 0; t < S; ++t) a[t] = run[t];
    int sx = 0, sy = 0;
#pragma unroll
    for (int t = 0; t < S; ++t) {
        sx += a[t].x;
        sy += a[t].y;
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
        o[at + s].x = sx;
        o[at + s].y = sy;
        if (s + 1 < S) {
            const int2 v = run[kRow + s];
            sx += v.x - a[s].x;
            sy += v.y - a[s].y;
        }
    }
}

template <int S, typename P2>
__device__ __forceinline__ void bf_split(int part, P2 *s_x)
{
    const int tid = threadIdx.x;
    const int2 *s_f = (const int2 *)s_x;
    constexpr int kRuns = S > 8 ? 1 : 2;  // rows m = tid (and 512 + tid, if a part is a whole block)
    P2 o[16];
    const bool last = tid == kSeg3 - 1;   // m = 1023 of the second segment is zero
#pragma unroll
    for (int q = 0; q < kRuns; ++q) {
        if (last && (q == 1 || part == 1)) {
#pragma unroll
            for (int s = 0; s < S; ++s) o[q * S + s] = P2{0, 0};
        } else {
            bf_boxcar<S>(s_f, q * kSeg3 + tid, o, q * S);
        }
    }
    __syncthreads();  // the samples are read
#pragma unroll
    for (int s = 0; s < kRuns * S; ++s) s_x[s * kXbuf3 + tid] = o[s];
}

// The wipe, fold, boxcar and polyphase split of part `part` of (Doppler, block) kb
// of request d: F[spc m + s] at element m mod 512 of slot s (of a part) or of
// slot (segment, s) (of a whole block), and 0 for m = 1023.  A part is 8192
// outputs at most: one segment (512 values of m) with more than 8 samples per
// chip, else both.  The 512 threads wipe and fold the samples into LDS; each then
// has the outputs of one or two m, its reads and writes at constant distances (one
// instance per number of samples per chip), and leaves them by slot.  Vector issue
// bounds it: with runs of 16 consecutive outputs, each one's slot and element found
// as it went, it took 0.30 ms on the weak-signal search (121 bins x 25 blocks x
// 4 ms at 16.368 MHz) where it takes 0.14, the polyphase values' write included.
// The caller synchronises before it reads the slots.
template <typename P2>
__device__ __forceinline__ void bf_front(const ReqDesc &d, int kb, int part, int parts, const uint2 *s_lut, P2 *s_x)
{
    const int N = d.N, spc = d.spc;
    int2 *s_f = (int2 *)s_x;
    const int k = kb / d.Nnc, b = kb - k * d.Nnc;
    const uint32_t D = d.dk[k], inv = row_inv(spc);
    // code-Doppler drift of this (bin, block) in samples, in [0, N): delaying
    // the folded block by it circularly shifts its correlation by as many lags
    const int shift = d.cshift ? d.cshift[kb] : 0;
    const int n0 = part * kSeg3 * spc;  // first output
    const int len = min(N - n0, parts == 2 ? kSeg3 * spc : N) + spc - 1;
    __syncthreads();  // the table is staged; the previous item's slots are read
    if (d.fmt == GNSS_CPLX_I8)
        bf_wipe_all<GNSS_CPLX_I8>(d, s_lut, D, d.b0 + b, n0 - shift, len, inv, s_f);
    else if (d.fmt == GNSS_REAL_I8)
        bf_wipe_all<GNSS_REAL_I8>(d, s_lut, D, d.b0 + b, n0 - shift, len, inv, s_f);
    else
        bf_wipe_all<GNSS_REAL_2BIT_PACKED>(d, s_lut, D, d.b0 + b, n0 - shift, len, inv, s_f);
    __syncthreads();
    switch (spc) {
    case 1: bf_split<1>(part, s_x); break;
    case 2: bf_split<2>(part, s_x); break;
    case 3: bf_split<3>(part, s_x); break;
    case 4: bf_split<4>(part, s_x); break;
    case 5: bf_split<5>(part, s_x); break;
    case 6: bf_split<6>(part, s_x); break;
    case 7: bf_split<7>(part, s_x); break;
    case 8: bf_split<8>(part, s_x); break;
    case 9: bf_split<9>(part, s_x); break;
    case 10: bf_split<10>(part, s_x); break;
    case 11: bf_split<11>(part, s_x); break;
    case 12: bf_split<12>(part, s_x); break;
    case 13: bf_split<13>(part, s_x); break;
    case 14: bf_split<14>(part, s_x); break;
    case 15: bf_split<15>(part, s_x); break;
    default: bf_split<16>(part, s_x); break;
    }
}

// ===========================================================================
// stage A, FP16 modes: wipe, fold, boxcar and polyphase split.  One workgroup
// per (Doppler, block), its parts in turn; the polyphase vectors go out in whole
// rows.  Bound: vector issue (the wipe's dot products, the boxcar's sliding sums) and
// the write of 8 bytes per output, which go on at the same time.
// Weak-signal search, 0.40 GB: 0.146 ms; with chunks of 2048 outputs, each thread's runs
// of 8 written as they came, 0.158.
// ===========================================================================
__global__ __launch_bounds__(kBfThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_box(
    const ReqDesc *__restrict__ R, const BatchHdr *H, const long long *pre, const uint32_t *lut, int2 *F)
{
    __shared__ int2 s_x[kBfSlots * kXbuf3];
    __shared__ uint2 s_lut[1024];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    stage_mix_lut(s_lut, lut, tid, kBfThreads);
    const int n_req = H->n_req;
    const long long total = H->total[kStBox];
    const long long *pst = pre + (long long)kStBox * (n_req + 1);
    for (long long it = xcd_remap(blockIdx.x, gridDim.x); it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        // (Doppler, block)-major items (dealing them block-major, so that the bins of
        // a block share its samples in L2, was measured 15% slower)
        const int kb = (int)(it - first_item(pst, n_req, r));  // < 2^31 by the plan checks
        const int spc = d.spc, parts = bf_parts(spc);
        for (int part = 0; part < parts; ++part) {
            bf_front(d, kb, part, parts, s_lut, s_x);
            __syncthreads();
            const int slots = parts == 2 ? spc : 2 * spc;
            for (int slot = w; slot < slots; slot += kBfThreads / 64) {
                const int sg = parts == 2 ? part : slot / spc, s = parts == 2 ? slot : slot - sg * spc;
                const int2 *src = s_x + slot * kXbuf3;
                int2 *dst = F + (d.vec_off + (long long)kb * spc + s) * kPolyLen + sg * kSeg3;
#pragma unroll
                for (int j = 0; j < kSeg3 / 64; ++j) dst[l + 64 * j] = src[l + 64 * j];
            }
        }
    }
}

// ===========================================================================
// stage A, FP32: wipe, fold, boxcar, polyphase split and forward transforms in
// one kernel.  A work item is a part of a (Doppler, block) (bf_front); each wave
// transforms the segments w and w + 8 where that left them in LDS.  What
// bounds it is the write of the spectra (24 KB per (Doppler, block, phase));
// the polyphase values, written and read again by two kernels before, stay in
// LDS.  80 KB of LDS, half of a CU's to the byte: two workgroups per CU, so that
// one's transforms overlap the other's sample loads.  Measured on the
// weak-signal search (121 bins x 25 blocks x 16 phases, 1.19 GB of spectra):
// 0.29 ms, 4.1 TB/s, against 0.17 + 0.27 ms for the two kernels it replaces.
// ===========================================================================
__global__ __launch_bounds__(kBfThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_box_fft(
    const ReqDesc *__restrict__ R, const BatchHdr *H, const long long *pre, const uint32_t *lut, const float2 *twg,
    float4 *G)
{
    __shared__ float2 s_x[kBfSlots * kXbuf3];
    __shared__ uint2 s_lut[1024];
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    stage_mix_lut(s_lut, lut, tid, kBfThreads);
    const int n_req = H->n_req;
    const long long total = H->total[kStBoxFft];
    const long long *pst = pre + (long long)kStBoxFft * (n_req + 1);
    const long long id = xcd_remap(blockIdx.x, gridDim.x);
    for (long long it = id; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const int spc = d.spc, parts = bf_parts(spc);
        const int local = (int)(it - first_item(pst, n_req, r));
        const int kb = local / parts, part = local - kb * parts;
        bf_front(d, kb, part, parts, s_lut, s_x);
        int l = tid & 63;
        asm volatile("" : "+v"(l));  // the twiddle addresses are formed here, not hoisted and held
        const Lane3 lw(twg, l);
        __syncthreads();
        const int slots = parts == 2 ? spc : 2 * spc;
        {
            for (int slot = w; slot < slots; slot += kBfThreads / 64) {
                const int sg = parts == 2 ? part : slot / spc, s = parts == 2 ? slot : slot - sg * spc;
                float2 *xb = s_x + slot * kXbuf3;  // the slot's own LDS carries its exchanges
                float2 x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = xb[l + 64 * j];
                wave_lds_order();
                float4 *dst = G + (d.vec_off + (long long)kb * spc + s) * kVec3 + sg * kSpec3;
                auto third = [&](auto cc) {
                    constexpr int c = decltype(cc)::value;
                    float2 v[8];
                    fft1536_seg<c>(x, v, xb, lw, l);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        dst[(4 * c + p) * 64 + l] = make_float4(v[2 * p].x, v[2 * p].y, v[2 * p + 1].x, v[2 * p + 1].y);
                    phase_barrier();
                };
                unrolled<3>(third);
            }
        }
    }
}

// ===========================================================================
// stage B: fused conj-multiply -> IFFT -> |.|^2 -> non-coherent sum
// ===========================================================================

// Grid write of a correlation work item.  Lag tau = spc*q + s interleaves the
// waves' phases, so the sums are staged in LDS ([1024 q][W + 1] floats per
// PRN: both the per-wave writes and the per-row reads are free of bank
// conflicts) and written as contiguous runs of consecutive tau.
// write_rows writes one PRN's staged sums (column w = wave w's (Doppler,
// phase) item; consecutive items of a bin are consecutive lags), or adds
// them to the grid (add): the element-to-thread map depends only on the
// request, chunk and thread, so each thread reads back its own earlier store.
//
// write_run writes ns consecutive phases of a bin, V at a time (columns wa to
// wa + ns - 1).  Vector issue is what it costs, as everywhere in these kernels:
// a thread's next element is found by adding, without a division, and runs of 4
// phases go out as one 16-byte store (4-byte aligned).  One element at a time, with its
// division, was 27 vector instructions: 430 per wave and item, where a block's
// transform is 250 to 940; in fours it is 22 per four.  One launch: strong-signal search
// (10 blocks) 93.6 -> 91.3 us, weak-signal (25 blocks) 2.99 -> 2.93 ms.
template <int W, int V>
__device__ __forceinline__ void write_run(const float *st, GNSS_GLOBAL float *row, int spc, int ns, int wa, int tid, bool add)
{
    typedef float fv __attribute__((ext_vector_type(V), aligned(4)));
    constexpr int kPad = W + 1, T = 64 * W;
    const int u = ns / V;  // vectors per lag row
    const int dq = T / u, dj = (T - dq * u) * V;
    int q = tid / u, j = (tid - q * u) * V;
    while (q < kCodeLen) {
        GNSS_GLOBAL fv *o = (GNSS_GLOBAL fv *)(row + (unsigned)(spc * q + j));
        const float *src = st + q * kPad + wa + j;
        fv v;
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = src[i];
        if (add) v += *o;
        *o = v;
        q += dq;
        j += dj;
        if (j >= ns) {
            j -= ns;
            ++q;
        }
    }
}

template <int W>
__device__ __forceinline__ void write_rows(const float *st, const ReqDesc &d, int pi, int chunk, int tid, bool add = false)
{
    const int spc = d.spc;
    const int first = chunk * W;
    const int n_items_here = min(W, d.n_items - first);
    int wa = 0;
    while (wa < n_items_here) {
        const int ka = (first + wa) / spc, sa = (first + wa) - ka * spc;
        const int ns = min(spc - sa, n_items_here - wa);  // consecutive phases of bin ka
        GNSS_GLOBAL float *row = gmem(d.grid) + ((long long)pi * d.n_dopp + ka) * d.N + sa;
        if ((ns & 3) == 0)
            write_run<W, 4>(st, row, spc, ns, wa, tid, add);
        else
            write_run<W, 1>(st, row, spc, ns, wa, tid, add);
        wa += ns;
    }
}

// Stages and writes a tile's sums, P = |IFFT|^2 * scale (2^-22 for the
// unnormalised 2048-point IFFT and 2^-24 for the LUT scale, times the FP16
// path's code-spectrum scaling); add: adds them to the grid's sums instead
// (every wave of the workgroup passes the same flag).
// Sum 4 u + k2b of lane l is lag q = l + 64 (4 u + k2b) with QL (1536-point
// transforms), else q = l + 64 u + 256 k2b (2048-point ones).
template <int PT, int W, bool QL>
__device__ __forceinline__ void store_tile(const float (&acc)[PT][16], float *s_stage, const ReqDesc &d,
                                           int ptile, int chunk, int w, int l, int tid, float scale,
                                           bool add = false)
{
    constexpr int kPad = W + 1;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k2b = 0; k2b < 4; ++k2b) {
                int q = QL ? l + 64 * (4 * u + k2b) : l + 64 * u + 256 * k2b;
                s_stage[(p * 1024 + q) * kPad + w] = acc[p][4 * u + k2b] * scale;
            }
    __syncthreads();
    for (int p = 0; p < PT; ++p) {
        const int pi = ptile * PT + p;
        if (pi >= d.n_prn) break;
        write_rows<W>(s_stage + p * 1024 * kPad, d, pi, chunk, tid, add);
    }
}

// Cascaded non-coherent sums: a wave adds its lanes' sums of the group of
// blocks just done to the grid (add) or stores them there (the first group),
// then clears them; each lane reads back only its own stores, and the final
// write (store_tile with add, another thread per element) comes after its
// workgroup barriers.  Lane l holds the lags q = l + 64 j of the
// item (bin k, phase s): grid column s + spc q.
template <int PT>
__device__ __forceinline__ void add_group(float (&acc)[PT][16], const ReqDesc &d, int ptile, int k, int s, int l,
                                          float scale, bool add)
{
#pragma unroll
    for (int p = 0; p < PT; ++p) {
        const int pi = ptile * PT + p;
        if (pi < d.n_prn) {
            GNSS_GLOBAL float *row = gmem(d.grid) + ((long long)pi * d.n_dopp + k) * d.N + s;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int q = l + 64 * j;
                if (q < kCodeLen) {
                    GNSS_GLOBAL float *o = row + (long long)d.spc * q;
                    const float v = acc[p][j] * scale;
                    *o = add ? *o + v : v;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[p][i] = 0.f;
    }
}

// Work item = (request, PRN tile, chunk of W (Doppler, phase) items); one wave
// per (Doppler, phase) item, looping over the blocks and the tile's PT PRNs
// with the sums in registers.  W waves per workgroup, WPE the waves per SIMD
// the registers are budgeted for (PRN tile 1 at three waves per SIMD: 165
// VGPRs; tiles 2 and 4 at two).
// Bound: vector issue (925 vector instructions per transform, one per 1.8 ns and
// SIMD; LDS carries 74 KB per transform, three quarters of its rate).  On the
// weak-signal search (32 PRNs x 121 bins x 25 blocks x 16 phases, 1.55 million
// transforms) 2.55-2.75 ms, against 3.15-3.3 for one 2048-point transform per
// block (1 257 instructions, 97 KB); before the twiddles went into registers
// 2.9, before the thirds' spectra were loaded ahead 3.1.
template <int PT, int W, int WPE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(WPE))) void k_corr(const ReqDesc *__restrict__ R, BatchHdr *H,
                                                          const long long *pre, const float4 *G,
                                                          const float2 *__restrict__ CS,
                                                          const float2 *__restrict__ twg)
{
    constexpr int kCcBytes = PT * kCodeLds3 * (int)sizeof(float2);
    constexpr int kXbBytes = W * kXbuf3 * (int)sizeof(float2);
    constexpr int kStageBytes = PT * 1024 * (W + 1) * (int)sizeof(float);
    constexpr int kSmem = kCcBytes + kXbBytes > kStageBytes ? kCcBytes + kXbBytes : kStageBytes;
    // 2^-24 (LUT scale) over the square of the unnormalised transform's length and of
    // the code spectra's third
    constexpr float kScale = (float)(0x1p-24 * 9.0 / ((double)kLen3 * kLen3));
    __shared__ __align__(16) unsigned char smem[kSmem];
    __shared__ long long s_item;
    float2 *s_cc = (float2 *)smem;
    float2 *s_xb = (float2 *)(smem + kCcBytes);
    float *s_stage = (float *)smem;  // reused after the transforms

    const int tid = threadIdx.x;
    // the wave index as a wave-uniform (scalar) value: the item's bin and
    // phase derived from it stay out of the vector registers
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const Lane3 lw(twg, l);
    const int n_req = H->n_req;
    const long long total = H->total[kStCorr];
    const long long *pst = pre + (long long)kStCorr * (n_req + 1);
    bool first = true;
    for (;;) {
        const long long it = next_item(H, kStCorr, total, &s_item, first);
        if (it < 0) break;
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const long long local = it - first_item(pst, n_req, r);
        const int ptile = (int)(local % d.n_ptiles), chunk = (int)(local / d.n_ptiles);
        const int item = chunk * W + w;
        const bool active = item < d.n_items;
        const int spc = d.spc;
        const int k = item / spc, s = item - k * spc;

        // code spectra of the tile's PRNs (in a persistent launch this overwrites
        // the staging area of the previous item's write: the barrier inside
        // next_item separates them)
        for (int i = tid; i < PT * kCode3; i += 64 * W) {
            const int p = i / kCode3, e = i - p * kCode3, sg = e >> 10, m = e & 1023;
            const int pi = ptile * PT + p;
            const int prn = pi < d.n_prn ? d.prns[pi] : 0;
            const float2 v = CS[(long long)prn * kCode3 + e];
            float2 *dst = s_cc + p * kCodeLds3 + sg * (2 * kSeg3 + 1);
            dst[m] = v;
            if (m == kSeg3) dst[2 * kSeg3] = v;
        }
        __syncthreads();

        float acc[PT][16];
#pragma unroll
        for (int p = 0; p < PT; ++p)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[p][i] = 0.f;

        if (active) {
            float2 *xb = s_xb + w * kXbuf3;
            const float4 *gk = G + (d.vec_off + (long long)k * d.Nnc * spc + s) * kVec3;
            // The thirds of the spectra go one after another through product and
            // 512-point transform; each third's spectra are loaded while the third
            // before it is transformed (the last one's while the next block's first
            // third is).  The block spectrum is re-read for every PRN of the tile
            // (L1/L2 hits after the first) rather than pinned in registers.
            f4v gl[2][4];
            auto load = [&](const float4 *gp, int zero, auto cc) {
                constexpr int c = decltype(cc)::value;
                // a scalar base (uniform over the wave) and the lane's 32-bit offset
                const GNSS_GLOBAL f4v *gq = (const GNSS_GLOBAL f4v *)uniform64((long long)(gp + zero));
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) gl[i][q] = (gq + (i * kSpec3 + (4 * c + q) * 64))[(unsigned)l];
            };
            load(gk, 0, std::integral_constant<int, 0>());
            // groups of kSumGroup blocks (one for most requests)
            for (int b0 = 0; b0 < d.Nnc; b0 += kSumGroup) {
                if (b0) add_group<PT>(acc, d, ptile, k, s, l, kScale, d.acc || b0 > kSumGroup);
                const int b1 = min(d.Nnc, b0 + kSumGroup);
                for (int b = b0; b < b1; ++b, gk += (long long)spc * kVec3) {
                    // PRN slots past n_prn hold the all-zero spectrum of row 0; they are
                    // computed (no branch in the loop) but never written.
#pragma unroll
                    for (int p = 0; p < PT; ++p) {
                        float2 v[3][8];
                        auto third = [&](auto c3) {
                            constexpr int c = decltype(c3)::value;
                            constexpr int S1 = 2 * kSeg3 + 1;
                            const float2 *cc = s_cc + p * kCodeLds3 + l;
                            const float2 *cm = s_cc + p * kCodeLds3 + 2 * kSeg3 - l;  // mirrored
                            // z[n] = G_0 conj(C_0) + G_1 conj(C_1) and the first stage of the
                            // radix-8 pass: z[n + 4]'s products are added onto z[n], and
                            // z[n] - z[n + 4] = 2 z[n] - (z[n] + z[n + 4])
                            float2 sm[4], df[4];
#pragma unroll
                            for (int n = 0; n < 4; ++n) {
                                const f4v a0 = gl[0][n / 2], a1 = gl[1][n / 2], b0 = gl[0][n / 2 + 2], b1 = gl[1][n / 2 + 2];
                                const int e = 2 * (n & 1);
                                const float2 g0 = make_float2(a0[e], a0[e + 1]), g1 = make_float2(a1[e], a1[e + 1]);
                                const float2 h0 = make_float2(b0[e], b0[e + 1]), h1 = make_float2(b1[e], b1[e + 1]);
                                float2 z;
                                if constexpr (c < 2) {
                                    z = c_mul_add(g1, cc[S1 + kSeg3 * c + 64 * n], c_mul(g0, cc[kSeg3 * c + 64 * n]));
                                    sm[n] = c_mul_add(h1, cc[S1 + kSeg3 * c + 64 * (n + 4)],
                                                      c_mul_add(h0, cc[kSeg3 * c + 64 * (n + 4)], z));
                                } else {
                                    z = c_mulc_add(g1, cm[S1 - 64 * n], c_mulc(g0, cm[-64 * n]));
                                    sm[n] = c_mulc_add(h1, cm[S1 - 64 * (n + 4)], c_mulc_add(h0, cm[-64 * (n + 4)], z));
                                }
                                df[n] = make_float2(fmaf(2.f, z.x, -sm[n].x), fmaf(2.f, z.y, -sm[n].y));
                                if (n & 1) phase_barrier();  // bounds the code values in flight
                            }
                            // the products before the loads that take over their registers
                            int zero = 0;
                            asm volatile("" : "+s"(zero), "+v"(sm[0].x), "+v"(sm[0].y), "+v"(sm[1].x), "+v"(sm[1].y),
                                         "+v"(sm[2].x), "+v"(sm[2].y), "+v"(sm[3].x), "+v"(sm[3].y), "+v"(df[0].x),
                                         "+v"(df[0].y), "+v"(df[1].x), "+v"(df[1].y), "+v"(df[2].x), "+v"(df[2].y),
                                         "+v"(df[3].x), "+v"(df[3].y));
                            if constexpr (c < 2)
                                load(gk, zero, std::integral_constant<int, c + 1>());
                            else if (p + 1 < PT)
                                load(gk, zero, std::integral_constant<int, 0>());
                            else  // (after the last block its own again: no branch around the loads)
                                load(gk + (b + 1 < d.Nnc ? (long long)spc * kVec3 : 0), zero,
                                     std::integral_constant<int, 0>());
                            phase_barrier();
                            dft8_rest<true>(sm, df, v[c]);
                            ifft512_rest(v[c], xb, lw, l);
                            if constexpr (c < 2) phase_barrier();
                        };
                        unrolled<3>(third);
                        lags3(v, lw, [&](int j, float2 o) { acc[p][j] = fmaf(o.x, o.x, fmaf(o.y, o.y, acc[p][j])); });
                        phase_barrier();
                    }
                }
            }
        }

        store_tile<PT, W, true>(acc, s_stage, d, ptile, chunk, w, l, tid, kScale, d.acc || d.Nnc > kSumGroup);
    }
}

bool corr_shape_valid(CorrShape c, int precision)
{
    if (!corr_ptile_valid(c.pt, precision)) return false;
    if (precision != GNSS_FP32 || c.pt != 1) return c.w == corr_waves(precision, c.pt);
    return c.w == 12 || c.w == 6 || c.w == 4;
}

int corr_ptile_valid(int pt, int precision)
{
    return precision == GNSS_FP32 ? (pt == 1 || pt == 2 || pt == 4)
           : precision == GNSS_FP16 ? (pt == 2 || pt == 4)
                                    : (pt == 1 || pt == 2 || pt == 4 || pt == 8);
}

// ===========================================================================
// FP16 path: packed half-precision transforms with block floating point
// ===========================================================================
// Scaling.  Each polyphase vector g is scaled by 2^-e (e per vector, from its
// l1 norm) so that ||g 2^-e||_1 <= 32, and every code spectrum by the common
// 2^-ecs with max|C 2^-ecs| <= 1.  Then every intermediate stays below 2^15:
// all forward-transform values are bounded by the l1 norm (<= 32); the
// spectrum product by 32; the inverse transform's radix-16 outputs by 16*32
// and 256*32, the radix-8 partial sums by 4*256*32 = 2^15; and its outputs
// (the correlation times 2048 * 2^-ecs) by 2^(16 - ecs).  The scale factors
// are exact powers of two; |.|^2 and the sum over blocks are FP32.
constexpr int kL1Exp = 5;  // ||g 2^-e||_1 <= 2^5

// Smallest e with s * 2^-e <= 2^kL1Exp for a float sum s of non-negative
// terms (the factor covers the rounding of that sum).
__device__ __forceinline__ int l1_exponent(float s)
{
    if (!(s > 0.f)) return 0;
    int x;
    (void)frexpf(s * (1.f + 0x1p-10f), &x);  // s' < 2^x
    return x - kL1Exp;
}

// Sum over the wave; every lane gets the same value (each butterfly level adds
// the same two operands on both partner lanes).
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ uint32_t h2_bits(__half2 h) { return __builtin_bit_cast(uint32_t, h); }
__device__ __forceinline__ __half2 bits_h2(uint32_t u) { return __builtin_bit_cast(__half2, u); }

// hc2 twiddles: the T1/T2 tables of the FP32 path rounded to FP16 from the
// exact angle, each value in both halves.
__global__ void k_twiddles_h(hc2 *tw)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    double s, c;
    int e;
    double den;
    if (i < kT1Elems) {
        int hk = i >> 6, l = i & 63;
        int h = hk >> 4, k1 = hk & 15;
        e = ((l + 64 * h) * k1) & 2047;
        den = 1024.0;
    } else if (i < kTwElems) {
        int j = i - kT1Elems;
        int k2a = j >> 3, m2 = j & 7;
        e = (m2 * k2a) & 127;
        den = 64.0;
    } else {
        return;
    }
    sincospi((double)e / den, &s, &c);
    // one rounding, double -> FP16 (round to nearest even)
    const __half hc = __builtin_bit_cast(__half, (_Float16)c), hs = __builtin_bit_cast(__half, (_Float16)s);
    tw[i] = make_hc2(__halves2half2(hc, hc), __halves2half2(hs, hs));
}

// FP16 code spectra: CSh[prn] = conj(C) * 2^-ecs as (re, im) half2 in the
// packed storage order (uint4 unit 64 jj + l holds registers 4 jj .. 4 jj + 3
// of lane l), from the FP32 spectra.
__global__ void k_code_spectra_h(const float4 *cs, uint4 *csh, int ecs)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;  // prn * 512 + 64 jj + l
    if (i >= (kMaxPrn + 1) * 512) return;
    const int prn = i >> 9, unit = i & 511, jj = unit >> 6, l = unit & 63;
    const float sc = ldexpf(1.f, -ecs);
    const float4 *src = cs + (long long)prn * kVec;
    const float4 a = src[(2 * jj) * 64 + l], b = src[(2 * jj + 1) * 64 + l];
    csh[i] = make_uint4(h2_bits(__floats2half2_rn(a.x * sc, a.y * sc)), h2_bits(__floats2half2_rn(a.z * sc, a.w * sc)),
                        h2_bits(__floats2half2_rn(b.x * sc, b.y * sc)), h2_bits(__floats2half2_rn(b.z * sc, b.w * sc)));
}

// dck[prn] = 2048 * 2^-ecs * sum(code) / 1023 (PRN 0: 0)
__global__ void k_code_dc_h(const uint8_t *codes, float *dck, int ecs)
{
    const int prn = blockIdx.x * blockDim.x + threadIdx.x;
    if (prn > kMaxPrn) return;
    int sum = 0;
    if (prn > 0)
        for (int m = 0; m < kCodeLen; ++m) sum += codes[prn * kCodeLen + m] ? -1 : 1;
    dck[prn] = ldexpf(2048.f, -ecs) * (float)sum / (float)kCodeLen;
}

hipError_t launch_tables_h(const float4 *d_cs, const uint8_t *d_codes, void *d_tw_h, void *d_cs_h, int cs_exp,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_code_dc_h, dim3(1), dim3(64), 0, s, d_codes, (float *)((char *)d_cs_h + kCsHSpecBytes),
                       cs_exp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_twiddles_h, dim3((kTwElems + 255) / 256), dim3(256), 0, s, (hc2 *)d_tw_h);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_code_spectra_h, dim3(((kMaxPrn + 1) * 512 + 255) / 256), dim3(256), 0, s, d_cs,
                       (uint4 *)d_cs_h, cs_exp);
    return hipGetLastError();
}

__device__ __forceinline__ void stage_twiddles_h(hc2 *s_tw, const hc2 *tw, int tid, int nthreads)
{
    for (int i = tid; i < kTwElems; i += nthreads) s_tw[i] = tw[i];
}

// Forward transforms, two polyphase vectors per wave (the low and high
// halves).  Each vector is transformed with its mean S/1023 removed (S its
// sum over the 1023 values), scaled by 2^-e with e from the l1 norm of the
// mean-removed vector plus |S|; the correlation adds the mean's part back as
// the constant S/1023 * sum(code) of every lag.  (A strong DC component would
// otherwise cancel in the inverse transform against values far larger than
// the result, and the FP16 roundings of those values would dominate it.)
// Output: Gh[vec] in the packed storage order, the vector's exponent E[vec]
// and its scaled sum Dc[vec] = S * 2^-e.
// three waves per SIMD (168 VGPRs with a 44-byte spill): faster than two
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_fft_poly_h(const int2 *F, const hc2 *tw, uint4 *Gh, int *E,
                                                    float2 *Dc, const BatchHdr *H)
{
    __shared__ hc2 s_tw[kTwElems];
    __shared__ hc2 s_xb[4][kXbufElemsQ];
    stage_twiddles_h(s_tw, tw, threadIdx.x, 256);
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const long long n_vec = H->total[kStVec];
    const long long n_pair = (n_vec + 1) / 2;
    for (long long pr = (long long)blockIdx.x * 4 + w; pr < n_pair; pr += (long long)gridDim.x * 4) {
        const long long va = 2 * pr, vb = va + 1;
        const bool has_b = vb < n_vec;
        const int2 *sa = F + va * kPolyLen, *sb = F + vb * kPolyLen;
        int2 a[16], b[16];
        float sar = 0.f, sai = 0.f, sbr = 0.f, sbi = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k2b = 0; k2b < 4; ++k2b) {
                const int idx = l + 64 * u + 256 * k2b;  // element 1023 is zero
                a[4 * u + k2b] = sa[idx];
                b[4 * u + k2b] = has_b ? sb[idx] : make_int2(0, 0);
                sar += (float)a[4 * u + k2b].x;
                sai += (float)a[4 * u + k2b].y;
                sbr += (float)b[4 * u + k2b].x;
                sbi += (float)b[4 * u + k2b].y;
            }
        const float Sar = wave_sum(sar), Sai = wave_sum(sai), Sbr = wave_sum(sbr), Sbi = wave_sum(sbi);
        // IEEE division: a constant vector's mean is its value exactly
        const float mar = Sar / (float)kCodeLen, mai = Sai / (float)kCodeLen;
        const float mbr = Sbr / (float)kCodeLen, mbi = Sbi / (float)kCodeLen;
        float na = 0.f, nb = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k2b = 0; k2b < 4; ++k2b)
                if (l + 64 * u + 256 * k2b < kCodeLen) {
                    na += fabsf((float)a[4 * u + k2b].x - mar) + fabsf((float)a[4 * u + k2b].y - mai);
                    nb += fabsf((float)b[4 * u + k2b].x - mbr) + fabsf((float)b[4 * u + k2b].y - mbi);
                }
        const int ea = l1_exponent(wave_sum(na) + fabsf(Sar) + fabsf(Sai));
        const int eb = l1_exponent(wave_sum(nb) + fabsf(Sbr) + fabsf(Sbi));
        const float fa = ldexpf(1.f, -ea), fb = ldexpf(1.f, -eb);
        hc2 v[32];
        const __half2 zero = __floats2half2_rn(0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k2b = 0; k2b < 8; ++k2b) {
                if (k2b < 4) {
                    const int2 x = a[4 * u + k2b], y = b[4 * u + k2b];
                    // the zero element 1023 stays zero
                    const bool in = l + 64 * u + 256 * k2b < kCodeLen;
                    const float xr = in ? ((float)x.x - mar) * fa : 0.f, xi = in ? ((float)x.y - mai) * fa : 0.f;
                    const float yr = in ? ((float)y.x - mbr) * fb : 0.f, yi = in ? ((float)y.y - mbi) * fb : 0.f;
                    v[8 * u + k2b] = make_hc2(__floats2half2_rn(xr, yr), __floats2half2_rn(xi, yi));
                } else {
                    v[8 * u + k2b] = make_hc2(zero, zero);
                }
            }
        fft2048<true, true>(v, s_xb[w], s_tw, s_tw + kT1Elems, l);
        uint4 *ga = Gh + va * 512, *gb = Gh + vb * 512;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const hc2 *q = v + 4 * jj;
            ga[jj * 64 + l] = make_uint4(h2_bits(__lows2half2(q[0].re, q[0].im)), h2_bits(__lows2half2(q[1].re, q[1].im)),
                                         h2_bits(__lows2half2(q[2].re, q[2].im)), h2_bits(__lows2half2(q[3].re, q[3].im)));
            if (has_b)
                gb[jj * 64 + l] = make_uint4(h2_bits(__highs2half2(q[0].re, q[0].im)), h2_bits(__highs2half2(q[1].re, q[1].im)),
                                             h2_bits(__highs2half2(q[2].re, q[2].im)), h2_bits(__highs2half2(q[3].re, q[3].im)));
        }
        if (l == 0) {
            E[va] = ea;
            Dc[va] = make_float2(Sar * fa, Sai * fa);
            if (has_b) {
                E[vb] = eb;
                Dc[vb] = make_float2(Sbr * fb, Sbi * fb);
            }
        }
    }
}

// (g.re + i g.im) * c for both transforms of c
__device__ __forceinline__ hc2 c_mul_bcast(__half2 g, hc2 c)
{
    const __half2 gr = __low2half2(g), gi = __high2half2(g);
    return make_hc2(__hfma2(gr, c.re, __hneg2(__hmul2(gi, c.im))), __hfma2(gr, c.im, __hmul2(gi, c.re)));
}

// FP16 correlation: as k_corr, with the tile's PRNs in pairs, one packed
// inverse transform per pair and block.  Work item = (request, PRN tile,
// chunk of kCorrWavesH (Doppler, phase) items).
template <int PT>
__global__ __launch_bounds__(64 * kCorrWavesH) __attribute__((amdgpu_waves_per_eu(PT == 2 ? 3 : 1))) void k_corr_h(const ReqDesc *__restrict__ R, BatchHdr *H,
                                                             const long long *pre, const uint4 *Gh,
                                                             const int *E, const float2 *Dc,
                                                             const uint4 *__restrict__ CSh,
                                                             const float *__restrict__ dck,
                                                             const hc2 *__restrict__ tw, float out_scale)
{
    static_assert(PT % 2 == 0, "PRNs go in pairs");
    constexpr int NP = PT / 2;
    constexpr int W = kCorrWavesH;
    constexpr int kCcBytes = NP * 1024 * (int)sizeof(uint4);
    constexpr int kTwBytes = kTwElems * (int)sizeof(hc2);
    constexpr int kXbBytes = W * kXbufElemsQ * (int)sizeof(hc2);
    constexpr int kStageBytes = PT * 1024 * (W + 1) * (int)sizeof(float);
    constexpr int kSmem = (kCcBytes + kTwBytes + kXbBytes) > kStageBytes ? (kCcBytes + kTwBytes + kXbBytes)
                                                                          : kStageBytes;
    __shared__ __align__(16) unsigned char smem[kSmem];
    __shared__ long long s_item;
    uint4 *s_cc = (uint4 *)smem;  // unit 64 jj2 + l: registers 2 jj2, 2 jj2 + 1 of lane l (hc2 each)
    hc2 *s_tw = (hc2 *)(smem + kCcBytes);
    hc2 *s_xb = (hc2 *)(smem + kCcBytes + kTwBytes);
    float *s_stage = (float *)smem;

    const int tid = threadIdx.x;
    const int w = tid >> 6, l = tid & 63;
    const int n_req = H->n_req;
    const long long total = H->total[kStCorr];
    const long long *pst = pre + (long long)kStCorr * (n_req + 1);
    bool first = true;
    for (;;) {
        const long long it = next_item(H, kStCorr, total, &s_item, first);
        if (it < 0) break;
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const long long local = it - first_item(pst, n_req, r);
        const int ptile = (int)(local % d.n_ptiles), chunk = (int)(local / d.n_ptiles);
        for (int i = tid; i < NP * 1024; i += 64 * W) {
            const int pp = i >> 10, unit = i & 1023, jj2 = unit >> 6, ll = unit & 63;
            const int pa = ptile * PT + 2 * pp, pb = pa + 1;
            const int prn_a = pa < d.n_prn ? d.prns[pa] : 0, prn_b = pb < d.n_prn ? d.prns[pb] : 0;
            const uint4 ca = CSh[(long long)prn_a * 512 + (jj2 >> 1) * 64 + ll];
            const uint4 cb = CSh[(long long)prn_b * 512 + (jj2 >> 1) * 64 + ll];
            const uint32_t a0 = (jj2 & 1) ? ca.z : ca.x, a1 = (jj2 & 1) ? ca.w : ca.y;
            const uint32_t b0 = (jj2 & 1) ? cb.z : cb.x, b1 = (jj2 & 1) ? cb.w : cb.y;
            s_cc[i] = make_uint4(h2_bits(__lows2half2(bits_h2(a0), bits_h2(b0))), h2_bits(__highs2half2(bits_h2(a0), bits_h2(b0))),
                                 h2_bits(__lows2half2(bits_h2(a1), bits_h2(b1))), h2_bits(__highs2half2(bits_h2(a1), bits_h2(b1))));
        }
        stage_twiddles_h(s_tw, tw, tid, 64 * W);
        __syncthreads();

        const int item = chunk * W + w;
        const bool active = item < d.n_items;
        const int spc = d.spc;
        const int k = item / spc, s = item - k * spc;

        float acc[PT][16];
#pragma unroll
        for (int p = 0; p < PT; ++p)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[p][i] = 0.f;
        // per PRN: the lag-independent part of the inverse output per unit of
        // the scaled block sum, 2048 * 2^-ecs * sum(code) / 1023
        float kdc[PT];
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int pi = ptile * PT + p;
            kdc[p] = dck[pi < d.n_prn ? d.prns[pi] : 0];
        }

        if (active) {
            const long long v0 = d.vec_off + (long long)k * d.Nnc * spc + s;
            hc2 *xb = s_xb + w * kXbufElemsQ;
            for (int b = 0; b < d.Nnc; ++b) {
                const long long vec = v0 + (long long)b * spc;
                const float sc = ldexpf(1.f, 2 * E[vec]);
                const float2 ds = Dc[vec];
#pragma unroll
                for (int pp = 0; pp < NP; ++pp) {
                    const __half2 dre = __floats2half2_rn(kdc[2 * pp] * ds.x, kdc[2 * pp + 1] * ds.x);
                    const __half2 dim = __floats2half2_rn(kdc[2 * pp] * ds.y, kdc[2 * pp + 1] * ds.y);
                    const uint4 *gv = Gh + vec * 512;
                    asm volatile("" : "+v"(gv));
                    const GNSS_GLOBAL u4v *gq = (const GNSS_GLOBAL u4v *)gv;  // global, not flat, loads
                    phase_barrier();
                    hc2 z[32];
#pragma unroll
                    for (int jj = 0; jj < 8; ++jj) {
                        const u4v g = gq[jj * 64 + l];
                        const uint4 c0 = s_cc[pp * 1024 + (2 * jj) * 64 + l];
                        const uint4 c1 = s_cc[pp * 1024 + (2 * jj + 1) * 64 + l];
                        z[4 * jj + 0] = c_mul_bcast(bits_h2(g.x), make_hc2(bits_h2(c0.x), bits_h2(c0.y)));
                        z[4 * jj + 1] = c_mul_bcast(bits_h2(g.y), make_hc2(bits_h2(c0.z), bits_h2(c0.w)));
                        z[4 * jj + 2] = c_mul_bcast(bits_h2(g.z), make_hc2(bits_h2(c1.x), bits_h2(c1.y)));
                        z[4 * jj + 3] = c_mul_bcast(bits_h2(g.w), make_hc2(bits_h2(c1.z), bits_h2(c1.w)));
                    }
                    phase_barrier();
                    ifft2048<true, true>(z, xb, s_tw, s_tw + kT1Elems, l);
                    phase_barrier();
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int k2b = 0; k2b < 4; ++k2b) {
                            const hc2 o = z[8 * u + k2b];
                            const float2 re = __half22float2(__hadd2(o.re, dre)), im = __half22float2(__hadd2(o.im, dim));
                            const float ta = fmaf(re.x, re.x, im.x * im.x);
                            const float tb = fmaf(re.y, re.y, im.y * im.y);
                            acc[2 * pp][4 * u + k2b] = fmaf(ta, sc, acc[2 * pp][4 * u + k2b]);
                            acc[2 * pp + 1][4 * u + k2b] = fmaf(tb, sc, acc[2 * pp + 1][4 * u + k2b]);
                        }
                }
            }
        }

        store_tile<PT, W, false>(acc, s_stage, d, ptile, chunk, w, l, tid, out_scale, d.acc != 0);
    }
}

// ===========================================================================
// Exact-length mode (GNSS_FP16_PFA): the length-1023 correlations of the
// polyphase form with 1023-point transforms (Good-Thomas 31 x 33, no zero
// padding, pfa1023.hpp) whose two passes are FP16 x FP16 -> FP32 products on
// the matrix cores.  Scaling as in the FP16 mode: each polyphase vector is
// scaled by 2^-e so that its l1 norm is <= 32, and the code spectra by
// 2^-ecs so that max |C| <= 1.  Every pass output is bounded by the l1 norm
// of its input: the forward transform's values by 32, the spectrum product's
// by 32, the inverse 31-pass by 31 * 32 (rounded to FP16 for the second
// pass) and the 33-pass output (FP32) by 33 * 31 * 32.  |.|^2 is formed in
// FP32, times 2^(2e), summed over blocks; the grid gets 2^(2 ecs - 24) / 1023^2.
// ===========================================================================

// Real-form weight of an L-point DFT (L = 31 or 33): input (i_in, part p_in)
// to output (i_out, part p_out), parts 0 = re, 1 = im; zero outside [0, L).
// The complex weight is e^(-+ 2 pi i i_in i_out / L) (forward: minus).
__device__ double pfa_weight(int L, bool inv, int i_in, int p_in, int i_out, int p_out)
{
    if (i_in < 0 || i_out < 0 || i_in >= L || i_out >= L) return 0.0;
    if (L == pfa::kN2) (inv ? i_in : i_out) = pfa::column_b(inv ? i_in : i_out);
    const int e = (i_in * i_out) % L;
    double sn, cs;
    sincospi(2.0 * (double)e / (double)L, &sn, &cs);
    const double sg = inv ? 1.0 : -1.0;  // weight = cs + i sg sn
    // (xr + i xi)(cs + i sg sn) = (xr cs - xi sg sn) + i (xr sg sn + xi cs)
    if (p_out == 0) return p_in == 0 ? cs : -sg * sn;
    return p_in == 0 ? sg * sn : cs;
}

// two doubles to FP16 (one rounding, to nearest even)
__device__ __forceinline__ uint32_t pack2d(double x, double y)
{
    pfa::h2v v = {(_Float16)x, (_Float16)y};
    return __builtin_bit_cast(uint32_t, v);
}

// Output column of an x32 weight fragment: (index, part); index -1 = unused.
__device__ __forceinline__ void pfa_column(int L, bool inv, int tile, int c, int &i_out, int &p_out)
{
    if (L == pfa::kN1) {
        i_out = 16 * (tile & 1) + c;
        p_out = tile >> 1;
    } else if (tile < 4 || !inv) {
        i_out = 16 * (tile >> 1) + c;
        p_out = tile & 1;
    } else {  // inverse tile 4: column 32, re in lane c = 0, im in lane c = 1
        i_out = c < 2 ? 32 : -1;
        p_out = c & 1;
    }
}

// B fragments of the four passes (forward / inverse, 31 / 33), FP16.  K
// slot 8 g + j of step `step` is input index 16 step + 4 g + (j & 3), part
// j >> 2.
__global__ void k_pfa_frags(pfa::u4 *fr)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pfa::kFrags * 64) return;
    const int f = i >> 6, l = i & 63, g = l >> 4, c = l & 15;
    int L, step, tile;
    bool inv;
    if (f < pfa::kFragInv33) {
        L = pfa::kN1, inv = true, step = f / 4, tile = f % 4;
    } else if (f < pfa::kFragFwd31) {
        L = pfa::kN2, inv = true, step = (f - pfa::kFragInv33) / 5, tile = (f - pfa::kFragInv33) % 5;
    } else if (f < pfa::kFragFwd33) {
        L = pfa::kN1, inv = false, step = (f - pfa::kFragFwd31) / 4, tile = (f - pfa::kFragFwd31) % 4;
    } else {
        L = pfa::kN2, inv = false, step = (f - pfa::kFragFwd33) / 6, tile = (f - pfa::kFragFwd33) % 6;
    }
    int i_out, p_out;
    pfa_column(L, inv, tile, c, i_out, p_out);
    double wv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) wv[j] = pfa_weight(L, inv, 16 * step + 4 * g + (j & 3), j >> 2, i_out, p_out);
    fr[i] = pfa::u4{pack2d(wv[0], wv[1]), pack2d(wv[2], wv[3]), pack2d(wv[4], wv[5]), pack2d(wv[6], wv[7])};
}

// Exact 1023-point spectra of the +-1 codes in FP64, [prn][a][b] at
// k = k(a, b) (PRN 0: zero).  Grid (31, 38), one thread per b.
__global__ __launch_bounds__(64) void k_code_spectra_x(const uint8_t *codes, double2 *out)
{
    __shared__ double2 s_w[kCodeLen];  // e^(-2 pi i j / 1023)
    for (int j = threadIdx.x; j < kCodeLen; j += 64) {
        double sn, cs;
        sincospi(2.0 * (double)j / (double)kCodeLen, &sn, &cs);
        s_w[j] = make_double2(cs, -sn);
    }
    __syncthreads();
    const int a = blockIdx.x, prn = blockIdx.y, b = threadIdx.x;
    if (b >= pfa::kN2) return;
    const int k = pfa::freq_index(a, b);
    double re = 0.0, im = 0.0;
    if (prn != 0) {
        const uint8_t *code = codes + prn * kCodeLen;
        int idx = 0;
        for (int m = 0; m < kCodeLen; ++m) {
            const double chip = code[m] ? -1.0 : 1.0;
            re += chip * s_w[idx].x;
            im += chip * s_w[idx].y;
            idx += k;
            if (idx >= kCodeLen) idx -= kCodeLen;
        }
    }
    out[((long long)prn * pfa::kN1 + a) * pfa::kN2 + b] = make_double2(re, im);
}

// Coordinates of stored unit `unit` of a spectrum (see pfa::kUnits).
__device__ __forceinline__ void pfa_unit(int unit, int &t, int &s, int &g, int &c)
{
    if (unit < pfa::kTailUnit) {
        const int ff = unit >> 6, l = unit & 63;
        t = ff >> 1, s = ff & 1, g = l >> 4, c = l & 15;
    } else {
        t = 2, s = (unit - pfa::kTailUnit) >> 2, g = (unit - pfa::kTailUnit) & 3, c = 0;
    }
}

// FP16 code spectra C * 2^-ecs in the stored fragment layout.
__global__ void k_code_spectra_x_pack(const double2 *cs, pfa::u4 *out, int ecs)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (kMaxPrn + 1) * pfa::kUnits) return;
    const int prn = i / pfa::kUnits, unit = i % pfa::kUnits;
    int t, s, g, c;
    pfa_unit(unit, t, s, g, c);
    double re[4], im[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int a = 16 * s + 4 * g + j, b = 16 * t + c;
        double2 v = make_double2(0.0, 0.0);
        if (a < pfa::kN1 && b < pfa::kN2) v = cs[((long long)prn * pfa::kN1 + a) * pfa::kN2 + b];
        re[j] = ldexp(v.x, -ecs);
        im[j] = ldexp(v.y, -ecs);
    }
    out[i] = pfa::u4{pack2d(re[0], re[1]), pack2d(re[2], re[3]), pack2d(im[0], im[1]), pack2d(im[2], im[3])};
}

hipError_t launch_tables_x_frags(void *d_frags, hipStream_t s)
{
    constexpr int n = pfa::kFrags * 64;
    hipLaunchKernelGGL(k_pfa_frags, dim3((n + 255) / 256), dim3(256), 0, s, (pfa::u4 *)d_frags);
    return hipGetLastError();
}

hipError_t launch_code_spectra_x(const uint8_t *d_codes, double2 *d_tmp, hipStream_t s)
{
    hipLaunchKernelGGL(k_code_spectra_x, dim3(pfa::kN1, kMaxPrn + 1), dim3(64), 0, s, d_codes, d_tmp);
    return hipGetLastError();
}

hipError_t launch_code_spectra_x_pack(const double2 *d_tmp, void *d_cs_x, int cs_exp, hipStream_t s)
{
    constexpr int n = (kMaxPrn + 1) * pfa::kUnits;
    hipLaunchKernelGGL(k_code_spectra_x_pack, dim3((n + 255) / 256), dim3(256), 0, s, d_tmp, (pfa::u4 *)d_cs_x,
                       cs_exp);
    return hipGetLastError();
}

// Forward transform of one polyphase vector held in LDS (xs, 1024 int2, the
// last zero) by one wave: its sum S and mean S/1023, the exponent from the l1
// norm of the mean-removed vector plus |S|, the Good-Thomas gather of the
// mean-removed vector into fragments, two passes, and the spectrum stored as
// fragments (dst) with its exponent (*e_out, lane 0).  The DC bin is stored as
// S itself.  Removing the mean keeps the FP16 weights from leaking a strong DC
// component into the other bins: the code spectra are +-1 at DC and about 32
// elsewhere, so a leak of a few 10^-6 of the DC amplitude into every bin would
// reach percents of the correlation of a DC-dominated block (a constant
// offset in the samples).
__device__ __forceinline__ void fft_x_vector(const int2 *xs, const pfa::FwdB &B, pfa::u4 *dst, int *e_out, int l)
{
    const int g = l >> 4, c = l & 15;
    int2 v[kPolyLen / 64];
    float sr = 0.f, si = 0.f;
#pragma unroll
    for (int i = 0; i < kPolyLen / 64; ++i) {
        v[i] = xs[l + 64 * i];  // element 1023 is zero
        sr += (float)v[i].x;
        si += (float)v[i].y;
    }
    const float Sr = wave_sum(sr), Si = wave_sum(si);
    // IEEE division: a constant vector's mean is its value exactly
    const float mr = Sr / (float)kCodeLen, mi = Si / (float)kCodeLen;
    float nrm = 0.f;
#pragma unroll
    for (int i = 0; i < kPolyLen / 64; ++i)
        if (l + 64 * i < kCodeLen) nrm += fabsf((float)v[i].x - mr) + fabsf((float)v[i].y - mi);
    const int e = l1_exponent(wave_sum(nrm) + fabsf(Sr) + fabsf(Si));
    const float f = ldexpf(1.f, -e);
    pfa::u4 a1[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float re[4], im[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n1 = 16 * s + 4 * g + j, n2 = 16 * t + c;
                re[j] = 0.f;
                im[j] = 0.f;
                if (n1 < pfa::kN1 && n2 < pfa::kN2) {
                    const int2 x = xs[pfa::time_index(n1, n2)];
                    re[j] = ((float)x.x - mr) * f;
                    im[j] = ((float)x.y - mi) * f;
                }
            }
            a1[t][s] = pfa::u4{pfa::pack2(re[0], re[1]), pfa::pack2(re[2], re[3]), pfa::pack2(im[0], im[1]),
                               pfa::pack2(im[2], im[3])};
        }
    pfa::f4 o[2][6];
    pfa::forward(a1, B, o);
    if (l == 0) {  // bin 0 (a = 0, b = 0, column 32): the vector's sum
        o[0][4].x = Sr * f;
        o[0][5].x = Si * f;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const pfa::f4 re = o[s][2 * t], im = o[s][2 * t + 1];
            dst[(2 * t + s) * 64 + l] = pfa::u4{pfa::pack2(re.x, re.y), pfa::pack2(re.z, re.w),
                                                pfa::pack2(im.x, im.y), pfa::pack2(im.z, im.w)};
        }
    if (c == 0) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const pfa::f4 re = o[s][4], im = o[s][5];
            dst[pfa::kTailUnit + 4 * s + g] = pfa::u4{pfa::pack2(re.x, re.y), pfa::pack2(re.z, re.w),
                                                      pfa::pack2(im.x, im.y), pfa::pack2(im.z, im.w)};
        }
    }
    if (l == 0) *e_out = e;
}

// Forward transforms of the polyphase vectors in F: one vector per wave,
// copied into LDS, then fft_x_vector.  (Fusing this with the wipe/fold stage,
// the spc vectors of a (Doppler, block) item built in LDS and transformed
// there, was measured slower: one 154 KB workgroup per CU left the wipe's
// memory latency exposed, 0.63 ms against 0.33 ms for the two kernels.)
__global__ __launch_bounds__(256) void k_fft_x(const int2 *F, const pfa::u4 *__restrict__ fr, pfa::u4 *Gx, int *E,
                                               const BatchHdr *H)
{
    __shared__ int2 s_x[4][kPolyLen];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    pfa::FwdB B;
    pfa::load_fwd(B, fr, l);
    const long long n_vec = H->total[kStVec];
    int2 *xs = s_x[w];
    for (long long vec = (long long)blockIdx.x * 4 + w; vec < n_vec; vec += (long long)gridDim.x * 4) {
        const int2 *src = F + vec * kPolyLen;
        lds_fence();  // the previous vector's gathers are complete
#pragma unroll
        for (int i = 0; i < kPolyLen / 64; ++i) xs[l + 64 * i] = src[l + 64 * i];
        lds_fence();
        fft_x_vector(xs, B, Gx + vec * pfa::kUnits, E + vec, l);
    }
}

// LDS copy of one stored spectrum: the four full fragments (1 KB each) and
// the 128-byte tail, staged as 32 dwords (lanes 32..63 repeat them).
constexpr int kXBuf = pfa::kTailUnit + 16;  // u4 units per LDS spectrum buffer
template <bool TAIL>
__device__ __forceinline__ void stage_spectrum(const pfa::u4 *src, pfa::u4 *dst, int l)
{
    typedef __attribute__((address_space(1))) const void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    // (the immediate offset moves both the global and the LDS address)
    __builtin_amdgcn_global_load_lds((gvoid *)(src + l), (lvoid *)dst, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((gvoid *)(src + l), (lvoid *)dst, 16, 1024, 0);
    __builtin_amdgcn_global_load_lds((gvoid *)(src + l), (lvoid *)dst, 16, 2048, 0);
    __builtin_amdgcn_global_load_lds((gvoid *)(src + l), (lvoid *)dst, 16, 3072, 0);
    if constexpr (TAIL) {
        const uint32_t *tail = (const uint32_t *)(src + pfa::kTailUnit);
        __builtin_amdgcn_global_load_lds((gvoid *)(tail + (l & 31)), (lvoid *)(dst + pfa::kTailUnit), 4, 0, 0);
    }
}

// Value of lane 4 q + 1 in lane 4 q (DPP quad permutation [1, 1, 3, 3]).
__device__ __forceinline__ float from_next_lane(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xF5, 0xF, 0xF, false));
}

// G * conj(C) for the four complex values of a fragment (packed FP16)
__device__ __forceinline__ pfa::u4 cmul_conj_frag(pfa::u4 g, pfa::u4 c)
{
    const __half2 gr0 = bits_h2(g.x), gr1 = bits_h2(g.y), gi0 = bits_h2(g.z), gi1 = bits_h2(g.w);
    const __half2 cr0 = bits_h2(c.x), cr1 = bits_h2(c.y), ci0 = bits_h2(c.z), ci1 = bits_h2(c.w);
    const __half2 yr0 = __hfma2(gr0, cr0, __hmul2(gi0, ci0)), yr1 = __hfma2(gr1, cr1, __hmul2(gi1, ci1));
    const __half2 yi0 = __hfma2(gi0, cr0, __hneg2(__hmul2(gr0, ci0)));
    const __half2 yi1 = __hfma2(gi1, cr1, __hneg2(__hmul2(gr1, ci1)));
    return pfa::u4{h2_bits(yr0), h2_bits(yr1), h2_bits(yi0), h2_bits(yi1)};
}

// The 33rd column's 31-point transforms of 16 (block, PRN) pairs in LDS: rows of
// [part][n1 < 32] floats, padded against bank conflicts of the lanes' writes.
constexpr int kCol0Row = 68;
static_assert(kCorrWavesX * 16 * kCol0Row <= 1024 * (kCorrWavesX + 1), "held in the grid's staging area");

// Sum over an item's blocks of |IDFT(G conj(C))|^2 for NP PRNs (one or two), by
// one wave.  Block b + 1's spectrum is copied into the wave's other LDS buffer
// (direct-to-LDS loads, no registers) while block b is transformed.  Matrix and
// vector instructions take turns on a SIMD, so their sum is what it costs; the
// 33rd column (b = 0) fits no tile and is kept from costing tiles of its own:
// * its 31-point transforms are made for 16 (block, PRN) pairs at once, as the
//   16 columns of one product with the weights as A operand, rounded to FP16 as
//   every other column is and kept in LDS for the blocks that follow;
// * its weight in the 33-pass is 1 for every output, so it enters that pass as
//   the accumulator's first value (the same for all columns of a row).
// 36.5 matrix instructions per transform instead of 54 (8 + 10 went to that column).
// With those gone the waves waited for their spectra, so a wave takes two PRNs per
// staged spectrum and nothing between one copy and the next waits for memory.  The
// weak-signal search's correlations (32 PRNs, 121 bins, 25 blocks, 16 phases):
// 1.11 -> 0.82 to 0.87 ms, the matrix units busy for 58% of the cycles and the vector
// instructions, at four clocks each, for 57%.
template <int NP>
__device__ __forceinline__ void blocks_x(float (&acc)[NP][2][3][4], const ReqDesc &d, const pfa::u4 *gx, const int *ex,
                                         const pfa::u4 *__restrict__ s_c, pfa::u4 *__restrict__ bufs,
                                         float *__restrict__ col0, const pfa::InvB &B, int l)
{
    constexpr int NB = 16 / NP;   // blocks per batch of the 33rd column
    constexpr int kRow = kCol0Row;
    const int g = l >> 4, c = l & 15;
    const long long step = (long long)d.spc * pfa::kUnits;
    const int Nnc = d.Nnc, spc = d.spc;
    const pfa::f4 z = {0.f, 0.f, 0.f, 0.f};
    stage_spectrum<false>(gx, bufs, l);
    int ev = 0, e_ref = ex[0], e_max = e_ref;
    for (int b = 0; b < Nnc; ++b) {
        const int beta = b & (NB - 1);
        if (beta == 0) {
            const int bc = min(b + (c & (NB - 1)), Nnc - 1);
            const pfa::u4 *tp = gx + (long long)bc * step + pfa::kTailUnit + g;
            const pfa::u4 *cp = s_c + (NP == 1 ? 0 : (c >> 3) * pfa::kUnits) + pfa::kTailUnit + g;
            const pfa::u4 t0 = tp[0], t1 = tp[4];
            ev = ex[(long long)bc * spc];
            const pfa::u4 y0 = cmul_conj_frag(t0, cp[0]), y1 = cmul_conj_frag(t1, cp[4]);
            wave_lds_order();  // the previous batch's reads come before these writes
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const pfa::f4 v = pfa::mma32(B.b31[1][n], y1, pfa::mma32(B.b31[0][n], y0, z));
                float4 r;
                r.x = (float)(_Float16)v.x;
                r.y = (float)(_Float16)v.y;
                r.z = (float)(_Float16)v.z;
                r.w = (float)(_Float16)v.w;
                *(float4 *)(col0 + c * kRow + 32 * (n >> 1) + 16 * (n & 1) + 4 * g) = r;
            }
            wave_lds_order();
            asm volatile("" : "+v"(ev));  // arrived here: no wait for it behind the next block's copy
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // block b is in LDS
        const pfa::u4 *cur = bufs + (b & 1) * kXBuf;
        pfa::u4 gf[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) gf[i] = cur[i * 64 + l];
        // The other buffer was last read for block b - 1.  (The copy is issued behind
        // this block's reads, and the other LDS arrays are declared disjoint from the
        // buffers: the compiler waits for a copy in flight before any LDS read that
        // might see it.)
        if (b + 1 < Nnc)
            stage_spectrum<false>((const pfa::u4 *)uniform64((long long)(gx + (b + 1) * step)),
                                  bufs + ((b + 1) & 1) * kXBuf, l);
        // The sums are kept in units of 2^(2 e_ref), e_ref the exponent of the last
        // block added: a block at e_ref adds its power unscaled.
        const int e_cur = __builtin_amdgcn_readlane(ev, beta);
        bool drop = false;
        if (e_cur != e_ref) {
            // Another block exponent: bring the sums to it (a power of two, exact).
            // A block's power is below 2^30 in its own units and Nnc < 2^17, so the
            // sums stay below 2^47 in the units of the largest exponent so far,
            // e_max; scaling to e_cur >= e_max - 30 multiplies them by at most 2^60
            // over that, which stays finite.  A block more than 2^30 below e_max
            // adds less than 2^-60 of that block's power and is dropped (an
            // all-zero block has exponent 0 and power 0).
            drop = e_cur < e_max - 30;
        }
        if (e_cur != e_ref && !drop) {
            const float f = ldexpf(1.f, 2 * (e_ref - e_cur));
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int h = 0; h < 3; ++h)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[p][u][h][q] *= f;
            e_ref = e_cur;
            e_max = max(e_max, e_cur);
        }
        if (drop) continue;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            pfa::u4 a1[2][2], a2[2][2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int ss = 0; ss < 2; ++ss)
                    a1[t][ss] = cmul_conj_frag(gf[2 * t + ss], s_c[p * pfa::kUnits + (2 * t + ss) * 64 + l]);
            const float *z0 = col0 + (beta + NB * p) * kRow + 4 * g;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                pfa::f4 d1[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) d1[n] = pfa::mma32(a1[t][1], B.b31[1][n], pfa::mma32(a1[t][0], B.b31[0][n], z));
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    a2[u][t] = pfa::u4{pfa::pack2(d1[u].x, d1[u].y), pfa::pack2(d1[u].z, d1[u].w),
                                       pfa::pack2(d1[u + 2].x, d1[u + 2].y), pfa::pack2(d1[u + 2].z, d1[u + 2].w)};
            }
            // |.|^2 into the sums.  Output column 32 has its real part in lane c = 0 and
            // its imaginary part in lane c = 1: each lane sums its own square and the
            // two are added at the end.
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const pfa::f4 c_re = *(const pfa::f4 *)(z0 + 16 * u), c_im = *(const pfa::f4 *)(z0 + 32 + 16 * u);
                const pfa::f4 c_32 = *(const pfa::f4 *)(z0 + 32 * (c & 1) + 16 * u);
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    const pfa::f4 o = pfa::mma32(a2[u][1], B.b33[1][v],
                                                 pfa::mma32(a2[u][0], B.b33[0][v], v == 4 ? c_32 : v & 1 ? c_im : c_re));
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[p][u][v >> 1][q] = fmaf(o[q], o[q], acc[p][u][v >> 1][q]);
                }
            }
        }
    }
    // column 32: lane c = 0 adds lane c = 1's imaginary part; then the sums in
    // absolute units
    const float f = ldexpf(1.f, 2 * e_ref);
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[p][u][2][q] += from_next_lane(acc[p][u][2][q]);
#pragma unroll
            for (int h = 0; h < 3; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[p][u][h][q] *= f;
        }
}

// Correlation, exact-length mode.  Work item = (request, PRN tile, chunk of
// kCorrWavesX (Doppler, phase) items); one wave per item; the tile's PRNs in
// turn, each over all blocks with its sums in registers, then written.
template <bool PAIRS>
__global__ __launch_bounds__(64 * kCorrWavesX) void k_corr_x(const ReqDesc *__restrict__ R, BatchHdr *H,
                                                             const long long *pre, const pfa::u4 *Gx,
                                                             const int *__restrict__ E, const pfa::u4 *__restrict__ CSx,
                                                             const pfa::u4 *__restrict__ fr, float out_scale)
{
    constexpr int W = kCorrWavesX;
    constexpr int kPad = W + 1;
    constexpr int NP = PAIRS ? 1 : 2;  // PRNs a wave works on at a time
    __shared__ pfa::u4 s_c[NP * pfa::kUnits];
    __shared__ __align__(16) float s_stage[1024 * kPad];  // blocks_x keeps its 33rd column there, 16 bytes at a time
    __shared__ pfa::u4 s_g[W * 2 * kXBuf];  // two block spectra per wave
    __shared__ long long s_item;
    const int tid = threadIdx.x;
    // the wave index is uniform: item indices, block addresses and exponents stay scalar
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, g = l >> 4, c = l & 15;
    pfa::InvB B;
    pfa::load_inv(B, fr, l);
    const int n_req = H->n_req;
    const int pt = H->corr_pt;
    const long long total = H->total[kStCorr];
    const long long *pst = pre + (long long)kStCorr * (n_req + 1);
    const pfa::u4 zero4 = {0u, 0u, 0u, 0u};
    bool first = true;
    for (;;) {
        const long long it = next_item(H, kStCorr, total, &s_item, first);
        if (it < 0) break;
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const long long local = it - first_item(pst, n_req, r);
        const int ptile = (int)(local % d.n_ptiles), chunk = (int)(local / d.n_ptiles);
        const int item = chunk * W + w;
        const bool active = item < d.n_items;
        const int spc = d.spc;
        const int k = item / spc, s = item - k * spc;
        const long long v0 = d.vec_off + (long long)k * d.Nnc * spc + s;
        for (int pp = 0; pp < pt; pp += NP) {
            const int pi = ptile * pt + pp;
            if (pi >= d.n_prn) break;
            const int np = min(NP, min(pt - pp, d.n_prn - pi));
            __syncthreads();  // the previous PRNs' reads of s_c and s_stage are done
            for (int p = 0; p < np; ++p)
                for (int i = tid; i < pfa::kUnits; i += 64 * W)
                    s_c[p * pfa::kUnits + i] = CSx[(long long)d.prns[pi + p] * pfa::kUnits + i];
            __syncthreads();
            float acc[NP][2][3][4];
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int h = 0; h < 3; ++h)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[p][u][h][q] = 0.f;
            if (active) {
                pfa::u4 *bufs = s_g + w * 2 * kXBuf;
                auto spectrum = [&](int b) { return Gx + (v0 + (long long)b * spc) * pfa::kUnits; };
                if constexpr (PAIRS) {
                    // Navigation-bit hypotheses: blocks 2i and 2i + 1 combined
                    // coherently with both relative signs, max over the two;
                    // R_a +- R_b is the inverse transform of (G_a +- G_b) conj(C).
                    // The + hypothesis's power waits in the wave's part of s_stage,
                    // which is free until the item's grid write.
                    float *pplus = s_stage + w * 1024;
                    for (int b = 0; b < d.Nnc; b += 2) {
                        stage_spectrum<true>(spectrum(b), bufs, l);
                        stage_spectrum<true>(spectrum(b + 1), bufs + kXBuf, l);
                        const int ea = E[v0 + (long long)b * spc], eb = E[v0 + (long long)(b + 1) * spc];
                        const int e = max(ea, eb);
                        // 2^(ea - e) and 2^(eb - e) in FP16 (exact; below 2^-24 they vanish,
                        // as that block's contribution does at FP16 precision)
                        const float fa32 = ldexpf(1.f, ea - e), fb32 = ldexpf(1.f, eb - e);
                        const __half2 fa = __floats2half2_rn(fa32, fa32), fb = __floats2half2_rn(fb32, fb32);
                        const float sc = ldexpf(1.f, 2 * e);
                        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // both blocks are in LDS
#pragma unroll
                        for (int hyp = 0; hyp < 2; ++hyp) {
                            pfa::u4 a1[3][2];
#pragma unroll
                            for (int t = 0; t < 3; ++t)
#pragma unroll
                                for (int ss = 0; ss < 2; ++ss) {
                                    const int unit = t < 2 ? (2 * t + ss) * 64 + l : pfa::kTailUnit + 4 * ss + g;
                                    if (t < 2 || c == 0) {
                                        const pfa::u4 ga = bufs[unit], gb = bufs[kXBuf + unit];
                                        pfa::u4 gs;
#pragma unroll
                                        for (int q = 0; q < 4; ++q) {
                                            const __half2 x = __hmul2(bits_h2(ga[q]), fa), y = __hmul2(bits_h2(gb[q]), fb);
                                            gs[q] = h2_bits(hyp == 0 ? __hadd2(x, y) : __hsub2(x, y));
                                        }
                                        a1[t][ss] = cmul_conj_frag(gs, s_c[unit]);
                                    } else {
                                        a1[t][ss] = zero4;
                                    }
                                }
                            pfa::f4 o[2][5];
                            pfa::inverse(a1, B, o);
#pragma unroll
                            for (int u = 0; u < 2; ++u)
#pragma unroll
                                for (int h = 0; h < 3; ++h)
#pragma unroll
                                    for (int q = 0; q < 4; ++q) {
                                        float pw;
                                        if (h < 2) {
                                            const float yr = o[u][2 * h][q], yi = o[u][2 * h + 1][q];
                                            pw = fmaf(yr, yr, yi * yi);
                                        } else {  // column 32: re in lane c = 0, im in lane c = 1
                                            const float t2 = o[u][4][q] * o[u][4][q];
                                            pw = t2 + from_next_lane(t2);
                                        }
                                        const int n1 = 16 * u + 4 * g + q, n2 = 16 * h + c;
                                        if (n1 < pfa::kN1 && n2 < pfa::kN2) {
                                            float *slot = pplus + pfa::time_index(n1, n2);
                                            if (hyp == 0)
                                                *slot = pw;
                                            else
                                                acc[0][u][h][q] = fmaf(fmaxf(*slot, pw), sc, acc[0][u][h][q]);
                                        }
                                    }
                            lds_fence();
                        }
                    }
                } else {
                    float *col0 = s_stage + w * 16 * kCol0Row;
                    if (np == NP) {
                        blocks_x<NP>(acc, d, Gx + v0 * pfa::kUnits, E + v0, s_c, bufs, col0, B, l);
                    } else {  // a tile's last PRN
                        float(&a1)[1][2][3][4] = *(float(*)[1][2][3][4]) & acc[0];
                        blocks_x<1>(a1, d, Gx + v0 * pfa::kUnits, E + v0, s_c, bufs, col0, B, l);
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if (p >= np) break;
                // every wave is done with s_stage (the 33rd column, the pair hypotheses
                // and the previous PRN's write use it)
                __syncthreads();
                if (active) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int h = 0; h < 3; ++h)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const int n1 = 16 * u + 4 * g + q, n2 = 16 * h + c;
                                if (n1 < pfa::kN1 && n2 < pfa::kN2)
                                    s_stage[pfa::time_index(n1, n2) * kPad + w] = acc[p][u][h][q] * out_scale;
                            }
                }
                __syncthreads();
                write_rows<W>(s_stage, d, pi + p, chunk, tid, d.acc != 0);
            }
        }
    }
}

// ===========================================================================
// Frequency-domain Doppler (exact-length contexts, option doppler_fd).  The
// carrier is removed once per block at the base frequency f_if + lo by an
// exact exponential (64-bit integer phase, FP32 sin/cos; phase zero at the block start,
// which leaves |R|^2 unchanged), and one zero-padded DFT of length
// M = P T_coh N = A * 1023 serves every Doppler bin: bin k's folded block has
// the N-point spectrum F^[q] = Y_M[P T_coh q + k kappa] (folding T_coh
// milliseconds keeps every (P T_coh)-th bin of the long spectrum, and the
// residual carrier k*step shifts it by k*kappa bins).  The one-chip boxcar
// multiplies by H[q] = sum_{t<spc} e^(2 pi i t q / N), and the polyphase
// spectra follow from
//   G_s[j] = (1/spc) e^(2 pi i s j / N) sum_{r<spc} B^[j + 1023 r] e^(2 pi i s r / spc).
// The long DFT is a prime-factor transform, A x 1023 (coprime): 1023-point
// DFTs on the matrix cores over the inner index, then A-point DFTs in FP32.
// Input map n = (1023 n1 + A m) mod M; the final spectrum is kept as
// X[k1][a * 33 + b'] with k1 = k mod A and (a, b') = (k mod 31, k mod 33).
// ===========================================================================

// Per (block, residue) maxima of max(|re|, |im|) of the final long spectrum
// (float bits; non-negative, so they order as unsigned integers), after the
// request's two spectra in the long-DFT buffer.
__device__ __forceinline__ uint32_t *fd_rowmax(const float2 *FD, const ReqDesc &d)
{
    return (uint32_t *)(FD + d.fd_off + 2LL * d.Nnc * d.fd_A * kCodeLen);
}

// First pass: one wave per (request, block, n1): the 1023-point DFT over m of
// the base-wiped samples y[(1023 n1 + A m) mod M] (zero past the block),
// scaled by its l1 exponent; written in FP32 times 2^e as Z[b][n1][a*33 + b'].
__global__ __launch_bounds__(256) void k_fd_pass1(const ReqDesc *__restrict__ R, const BatchHdr *H,
                                                  const long long *pre, const pfa::u4 *__restrict__ fr,
                                                  float2 *FD)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
    pfa::FwdB B;
    pfa::load_fwd(B, fr, l);
    const int n_req = H->n_req;
    const long long total = H->total[kStFdA];
    const long long *pst = pre + (long long)kStFdA * (n_req + 1);
    for (long long it = (long long)blockIdx.x * 4 + w; it < total; it += (long long)gridDim.x * 4) {
        const int r = find_req(pst, n_req, uniform64(it));
        const ReqDesc &d = R[r];
        const long long local = it - first_item(pst, n_req, r);
        const int A = d.fd_A, b = (int)(local / A), n1 = (int)(local % A);
        const long long M = (long long)A * kCodeLen, L = (long long)d.Tc * d.N;
        const long long base = (long long)(d.b0 + b) * L;
        if (n1 < d.fd_PTc && l == 0) fd_rowmax(FD, d)[b * d.fd_PTc + n1] = 0u;  // for the second pass
        float vr[3][2][4], vi[3][2][4];
        float nrm = 0.f;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i31 = 16 * s + 4 * g + j, i33 = 16 * t + c;
                    float yr = 0.f, yi = 0.f;
                    if (i31 < pfa::kN1 && i33 < pfa::kN2) {
                        const long long n = (1023LL * n1 + (long long)A * pfa::time_index(i31, i33)) % M;
                        if (n < L) {
                            int xr, xi;
                            load_sample(d.samples, d.fmt, base + n, xr, xi);
                            // carrier phase of in-block sample n: the top 24 bits of the
                            // 64-bit accumulator n * fd_dphase, exact as a float in [0, 1)
                            const unsigned long long ph = (unsigned long long)n * d.fd_dphase;
                            const float cyc = (float)(uint32_t)(ph >> 40) * 0x1p-24f;
                            float sn, cs;
                            sincospif(2.f * cyc, &sn, &cs);
                            yr = (float)xr * cs + (float)xi * sn;  // x e^(-i theta)
                            yi = (float)xi * cs - (float)xr * sn;
                        }
                    }
                    vr[t][s][j] = yr;
                    vi[t][s][j] = yi;
                    nrm += fabsf(yr) + fabsf(yi);
                }
        const int e = l1_exponent(wave_sum(nrm));
        const float f = ldexpf(1.f, -e), fo = ldexpf(1.f, e);
        pfa::u4 a1[3][2];
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                a1[t][s] = pfa::u4{pfa::pack2(vr[t][s][0] * f, vr[t][s][1] * f), pfa::pack2(vr[t][s][2] * f, vr[t][s][3] * f),
                                   pfa::pack2(vi[t][s][0] * f, vi[t][s][1] * f), pfa::pack2(vi[t][s][2] * f, vi[t][s][3] * f)};
        pfa::f4 o[2][6];
        pfa::forward(a1, B, o);
        float *dst = (float *)(FD + d.fd_off + (long long)(b * A + n1) * kCodeLen);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 6; ++v)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int a = 16 * u + 4 * g + q, bb = 16 * (v >> 1) + c;
                    if (a < pfa::kN1 && bb < pfa::kN2) dst[2 * (a * pfa::kN2 + bb) + (v & 1)] = o[u][v][q] * fo;
                }
    }
}

// Second pass: one workgroup per (request, block, 8 columns sigma): the
// columns' A x 8 values in LDS, the A-point DFTs over n1 in FP32,
//   Y_M[i] = sum_n1 Z[b][n1][sigma] e^(-2 pi i n1 k1 / A),
// i = (k1 crt1 + k2 crt2) mod M, k2 the frequency of sigma; stored by residue,
// Yt[b][i mod P T_coh][i div P T_coh] (i mod P T_coh = k1 mod P T_coh, since
// crt1 = 1 mod A and crt2 = 0 mod A), so that a Doppler bin's folded spectrum
// (every (P T_coh)-th bin from an offset) is a contiguous circular run of one
// row; and each row's max(|re|, |im|).  For A >= 4 a thread computes the four
// outputs k1 + m A/4 from each LDS value: their weights differ by (-i)^(n1 m).
__device__ __forceinline__ float2 quarter_turns(float2 t, int q)  // t (-i)^q, q in 0..3
{
    return q == 0 ? t : q == 1 ? make_float2(t.y, -t.x) : q == 2 ? make_float2(-t.x, -t.y) : make_float2(-t.y, t.x);
}

__global__ __launch_bounds__(256) void k_fd_pass2(const ReqDesc *__restrict__ R, const BatchHdr *H,
                                                  const long long *pre, float2 *FD)
{
    __shared__ float2 s_w[256];  // e^(-2 pi i m / 256); A divides 256
    __shared__ float2 s_z[256 * kFdCols];
    __shared__ uint32_t s_max[256];
    for (int m = threadIdx.x; m < 256; m += 256) {
        float sn, cs;
        sincospif((float)m / 128.f, &sn, &cs);
        s_w[m] = make_float2(cs, -sn);
    }
    const int n_req = H->n_req;
    const long long total = H->total[kStFdB];
    const long long *pst = pre + (long long)kStFdB * (n_req + 1);
    constexpr int kChunks = (kCodeLen + kFdCols - 1) / kFdCols;
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const long long local = it - first_item(pst, n_req, r);
        const int A = d.fd_A, PTc = d.fd_PTc;
        const int b = (int)(local / kChunks), sig0 = (int)(local % kChunks) * kFdCols;
        const int ncol = min(kFdCols, kCodeLen - sig0);
        const long long M = (long long)A * kCodeLen;
        const int N = (int)(M / PTc);
        const float2 *z = FD + d.fd_off + (long long)b * A * kCodeLen + sig0;
        __syncthreads();  // twiddles staged; the previous item's reads of s_z and s_max are done
        for (int i = threadIdx.x; i < A * kFdCols; i += 256) {
            const int n1 = i / kFdCols, cc = i % kFdCols;
            s_z[i] = cc < ncol ? z[(long long)n1 * kCodeLen + cc] : make_float2(0.f, 0.f);
        }
        if (threadIdx.x < PTc) s_max[threadIdx.x] = 0u;
        __syncthreads();
        const int step = 256 / A;
        float2 *yt = FD + d.fd_off + (long long)d.Nnc * M + (long long)b * M;
        auto emit = [&](int k1, int cc, float ar, float ai) {
            const int sigma = sig0 + cc;
            const int k2 = pfa::freq_index(sigma / pfa::kN2, sigma % pfa::kN2);
            const long long i = ((long long)k1 * d.fd_crt1 + (long long)k2 * d.fd_crt2) % M;
            yt[(i % PTc) * N + i / PTc] = make_float2(ar, ai);
            atomicMax(&s_max[k1 % PTc], __float_as_uint(fmaxf(fabsf(ar), fabsf(ai))));
        };
        if (A >= 4) {
            const int qa = A / 4;
            for (int o = threadIdx.x; o < qa * ncol; o += 256) {
                const int k1 = o / ncol, cc = o % ncol;
                float2 acc[4] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
                for (int p4 = 0; p4 < A; p4 += 4) {
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int n1 = p4 + rr;
                        const float2 v = s_z[n1 * kFdCols + cc];
                        const float2 wv = s_w[(n1 * k1 * step) & 255];
                        const float2 t = make_float2(v.x * wv.x - v.y * wv.y, v.x * wv.y + v.y * wv.x);
#pragma unroll
                        for (int m = 0; m < 4; ++m) {
                            const float2 u = quarter_turns(t, (rr * m) & 3);
                            acc[m].x += u.x;
                            acc[m].y += u.y;
                        }
                    }
                }
#pragma unroll
                for (int m = 0; m < 4; ++m) emit(k1 + m * qa, cc, acc[m].x, acc[m].y);
            }
        } else {
            for (int o = threadIdx.x; o < A * ncol; o += 256) {
                const int k1 = o / ncol, cc = o % ncol;
                float ar = 0.f, ai = 0.f;
                for (int n1 = 0; n1 < A; ++n1) {
                    const float2 v = s_z[n1 * kFdCols + cc];
                    const float2 wv = s_w[(n1 * k1 * step) & 255];
                    ar = fmaf(v.x, wv.x, fmaf(-v.y, wv.y, ar));
                    ai = fmaf(v.x, wv.y, fmaf(v.y, wv.x, ai));
                }
                emit(k1, cc, ar, ai);
            }
        }
        __syncthreads();
        if (threadIdx.x < PTc) atomicMax(fd_rowmax(FD, d) + b * PTc + threadIdx.x, s_max[threadIdx.x]);
    }
}

// In-register inverse DFT of S points, u_s = sum_r v_r e^(2 pi i s r / S):
// radix 2, decimation in frequency, then the bit-reversal permutation.  tw16[m]
// = e^(2 pi i m / 16).
template <int S>
__device__ __forceinline__ void idft_small(float2 (&v)[kMaxSpc], const float2 *tw16)
{
#pragma unroll
    for (int half = S / 2; half >= 1; half /= 2) {
#pragma unroll
        for (int i0 = 0; i0 < S; i0 += 2 * half)
#pragma unroll
            for (int j = 0; j < half; ++j) {
                const float2 a = v[i0 + j], b = v[i0 + j + half];
                const float2 w = tw16[j * (8 / half)];  // e^(2 pi i j / (2 half))
                const float2 d = make_float2(a.x - b.x, a.y - b.y);
                v[i0 + j] = make_float2(a.x + b.x, a.y + b.y);
                v[i0 + j + half] = make_float2(d.x * w.x - d.y * w.y, d.x * w.y + d.y * w.x);
            }
    }
    float2 t[kMaxSpc];
#pragma unroll
    for (int i = 0; i < S; ++i) {
        int rv = 0;
#pragma unroll
        for (int k = 1, m = S >> 1; k < S; k <<= 1, m >>= 1)
            if (i & k) rv |= m;
        t[rv] = v[i];
    }
#pragma unroll
    for (int i = 0; i < S; ++i) v[i] = t[i];
}

// Synthesis: one workgroup (512 threads) per (request, Doppler bin, block),
// the items of k_box.  For each frequency j < 1023 (one thread, reading the
// long spectrum contiguously) the spc values F^[j + 1023 r] give the
// polyphase spectra of the fold,
//   F_s'[j] = (1/spc) e^(2 pi i s' j / N) sum_r F^[j + 1023 r] e^(2 pi i s' r / spc),
// and the one-chip boxcar (g_s[m] = sum_{s'>=s} f_s'[m] + sum_{s'<s} f_s'[m+1])
// is G_s[j] = T + (e^(2 pi i j / 1023) - 1) P_s with T = sum_s' F_s' and
// P_s = sum_{s'<s} F_s'.  The spc spectra are staged in LDS in the stored
// fragment layout and written out whole.  |G_s| <= spc max |F^| sets the
// exponent e of the item's vectors (from the row maximum of the second pass).
constexpr int kSynthThreads = 512;
__global__ __launch_bounds__(kSynthThreads) void k_fd_synth(const ReqDesc *__restrict__ R, BatchHdr *H,
                                                            const long long *pre, const float2 *FD, pfa::u4 *Gx,
                                                            int *E)
{
    __shared__ pfa::u4 s_out[kMaxSpc * pfa::kUnits];
    __shared__ float2 s_tw16[16];
    __shared__ long long s_item;
    const int n_req = H->n_req;
    const long long total = H->total[kStBox];
    const long long *pst = pre + (long long)kStBox * (n_req + 1);
    const int tid = threadIdx.x;
    if (tid < 16) {
        float sn, cs;
        sincospif((float)tid / 8.f, &sn, &cs);
        s_tw16[tid] = make_float2(cs, sn);
    }
    bool first = true;
    for (;;) {
        const long long it = next_item(H, kStBox, total, &s_item, first);
        if (it < 0) break;
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const int kb = (int)(it - first_item(pst, n_req, r));
        const int k = kb / d.Nnc, b = kb - k * d.Nnc;
        const int N = d.N, spc = d.spc, A = d.fd_A, PTc = d.fd_PTc;
        const long long M = (long long)A * kCodeLen;
        const long long shift = ((long long)k * d.fd_kappa) % M;
        // F^[q] = Y_M[(q P T_coh + k kappa) mod M] = Yt[rho][(q + delta) mod N] with
        // k kappa = delta P T_coh + rho
        const int rho = (int)(shift % PTc), delta = (int)(shift / PTc);
        const float2 *row = FD + d.fd_off + (long long)d.Nnc * M + (long long)b * M + (long long)rho * N;
        const float mx = __uint_as_float(fd_rowmax(FD, d)[b * PTc + rho]) * 1.41421357f * (float)spc;
        int e = 0;
        if (mx > 0.f) {
            int x;
            (void)frexpf(mx * (1.f + 0x1p-10f), &x);  // mx' < 2^x
            e = x - kL1Exp;
        }
        const float scale = ldexpf(1.f, -e) / (float)spc;
        __syncthreads();  // tables staged; the previous item's copy out of s_out is done
        uint16_t *o16 = (uint16_t *)s_out;
        for (int j = tid; j < kCodeLen; j += kSynthThreads) {
            float2 v[kMaxSpc];
#pragma unroll
            for (int rr = 0; rr < kMaxSpc; ++rr) {
                int qq = j + kCodeLen * rr + delta;
                if (qq >= N) qq -= N;
                v[rr] = rr < spc ? row[qq] : make_float2(0.f, 0.f);
            }
            switch (spc) {
            case 2: idft_small<2>(v, s_tw16); break;
            case 4: idft_small<4>(v, s_tw16); break;
            case 8: idft_small<8>(v, s_tw16); break;
            case 16: idft_small<16>(v, s_tw16); break;
            default: break;  // spc 1: the value itself
            }
            float s1, c1, s2, c2;
            sincospif(2.f * (float)j / (float)N, &s1, &c1);         // e^(2 pi i j / N)
            sincospif(2.f * (float)j / (float)kCodeLen, &s2, &c2);  // e^(2 pi i j / 1023)
            float2 wv = make_float2(1.f, 0.f), tsum = make_float2(0.f, 0.f);
#pragma unroll
            for (int sp = 0; sp < kMaxSpc; ++sp) {
                if (sp < spc) {
                    const float2 f = make_float2((v[sp].x * wv.x - v[sp].y * wv.y) * scale,
                                                 (v[sp].x * wv.y + v[sp].y * wv.x) * scale);
                    v[sp] = f;
                    tsum.x += f.x;
                    tsum.y += f.y;
                    wv = make_float2(wv.x * c1 - wv.y * s1, wv.x * s1 + wv.y * c1);
                }
            }
            // fragment position of frequency j: row j mod 31, column (j - 1) mod 33
            const int a = j % pfa::kN1, bb = (j + pfa::kN2 - 1) % pfa::kN2;
            const int t = bb >> 4, cc = bb & 15, s31 = a >> 4, gg = (a >> 2) & 3, jj = a & 3;
            const int unit = t < 2 ? (2 * t + s31) * 64 + 16 * gg + cc : pfa::kTailUnit + 4 * s31 + gg;
            const float2 wm1 = make_float2(c2 - 1.f, s2);
            float2 pre_s = make_float2(0.f, 0.f);
#pragma unroll
            for (int ss = 0; ss < kMaxSpc; ++ss) {
                if (ss < spc) {
                    const float gr = tsum.x + wm1.x * pre_s.x - wm1.y * pre_s.y;
                    const float gi = tsum.y + wm1.x * pre_s.y + wm1.y * pre_s.x;
                    uint16_t *u16 = o16 + ((long long)ss * pfa::kUnits + unit) * 8;
                    u16[jj] = __builtin_bit_cast(uint16_t, (_Float16)gr);
                    u16[4 + jj] = __builtin_bit_cast(uint16_t, (_Float16)gi);
                    if (a == pfa::kN1 - 1) {  // the unit's padding slot a = 31 (every other slot is written)
                        u16[3] = 0;
                        u16[7] = 0;
                    }
                    pre_s.x += v[ss].x;
                    pre_s.y += v[ss].y;
                }
            }
        }
        __syncthreads();
        const long long vec0 = d.vec_off + (long long)kb * spc;
        for (int i = tid; i < spc * pfa::kUnits; i += kSynthThreads) Gx[vec0 * pfa::kUnits + i] = s_out[i];
        if (tid < spc) E[vec0 + tid] = e;
    }
}

// ===========================================================================
// General sample rates: fs a whole number of kHz that is not k * 1.023 MHz
// (k <= 16), so the replica has no whole number of samples per chip and the
// polyphase form does not apply.  The length-N circular correlation of each
// folded block is done on zero-padded transforms of length M = 2^ceil(log2
// 2N): the block f at [0, N), the replica over two code periods cc[j] =
// c[j mod N] at [0, 2N), and
//   R[tau] = sum_n f[n] c[(n - tau) mod N] = IDFT_M(DFT_M(f) conj(DFT_M(cc)))[M - N + tau] / M
// (no wrap-around because M >= 2N).  When N is a power of two, M = N: the
// same formula is then the N-point circular correlation itself (cc is one
// period on [0, M)).  FP32 throughout, in every context precision.
//
// Two segments.  Only N of the M outputs are lags, so a transform of half the
// length is enough when the block is taken as two segments of at most P - N
// samples (P = M/2): with f = f_0 + f_1, f_1 starting at sample n_1, and
// cc_i[u] = c[(n_i + u) mod N] at [0, L + N), L = ceil(N/2),
//   R[tau] = IDFT_P(sum_i DFT_P(f_i) conj(DFT_P(cc_i)))[P - N + tau] / P,
// no wrap-around because L + N <= P.  The products are summed before the one
// inverse, so a (PRN, bin, block) costs one P-point inverse instead of two or of
// one twice as long,
// and the two P-point spectra take the room of the M-point one.  Rule
// (gen_two_segments): N + ceil(N/2) <= M/2, i.e. N in (2^k, 4/3 2^k]; three or
// more segments would cover more lengths but need more room than the single
// M-point spectrum.
//
// Each transform of P points runs in one workgroup's LDS.  Without segments
// P = min(M, 16384); for M = 32768 the even and odd bins are two 16384-point
// transforms:
//   X[2k] = DFT_P(x[j] + x[j + P])[k],  X[2k + 1] = DFT_P((x[j] - x[j + P]) W_M^j)[k],
// and the inverse's upper half (the only outputs needed, as N <= M/2) is
//   out[P + k] = A[k] - W_M^-k B[k],  A = IDFT_P(Z even bins), B = IDFT_P(Z odd bins).
// In one piece (P <= 2048, and P = 4096 with few items: gen_in_rows): in-place
// radix-8 passes and one radix-2 or 4 pass in a 1024-thread workgroup, decimation in frequency forward (natural order in,
// digit-reversed out) and the exact adjoint inverse (digit-reversed in,
// natural out), so spectra are multiplied in the order they are stored.
// In rows (P = 4096 with many items, 8192 and 16384): four-step P/2048 x 2048
// transforms (below).
// ===========================================================================

// Radix of the LDS passes (a radix-16 butterfly with its twiddles needs about
// twice the registers, too many beside the correlation's per-lag sums at
// 1024 threads).
constexpr int kGenRad = 8;
// LDS layout of a transform: element i at i + i/32 (one unused slot per 32,
// P + P/32 slots), which spreads the strided accesses of the small-span
// passes over the banks
__device__ __forceinline__ int gx(int i) { return i + (i >> 5); }

// The first octant of the P-point twiddles, s_tw[i] = W_P^i for i < P/8,
// taken from the table of W_32768^i (forward sign).  A pass of span s needs
// W_{8s}^j = W_P^(j P / 8s) with j < s, always in this octant.
__device__ __forceinline__ void gen_load_tw(float2 *s_tw, int P, const float2 *tw)
{
    const int st = kGenTwLen / P;
    for (int i = threadIdx.x; i < P / kGenRad; i += kGenThreads) s_tw[i] = tw[i * st];
}

// w[r] = W^(j r) for r = 1..7 from w1 = W^j: products of at most three
// table values, a few ulp from the correctly rounded twiddles
__device__ __forceinline__ void gen_powers(float2 (&w)[kGenRad], float2 w1)
{
    w[1] = w1;
    w[2] = c_mul(w1, w1);
    w[3] = c_mul(w[2], w1);
    w[4] = c_mul(w[2], w[2]);
    w[5] = c_mul(w[4], w1);
    w[6] = c_mul(w[3], w[3]);
    w[7] = c_mul(w[4], w[3]);
}

// One radix-8 pass of span S over a P-point transform (both powers of two,
// compile time), one butterfly per thread-iteration on the 8 values at
// i0 + r S, i0 = 8 (t - j) + j, j = t mod S, in place.  Forward (decimation
// in frequency): 8-point DFT, then output r times W_{8S}^(j r).  Inverse:
// the adjoint, conjugate twiddles first.  In the padded layout
// gx(i0 + r S) = gx(i0) + r S + floor(r S / 32) for every such i0, so only
// gx(i0) is computed.
template <int P, int S, bool INV>
__device__ __forceinline__ void gen_pass(float2 *x, const float2 *s_tw)
{
    constexpr int ts = P / kGenRad / S;
#pragma unroll 1
    for (int t = threadIdx.x; t < P / kGenRad; t += kGenThreads) {
        const int j = t & (S - 1);
        float2 *base = x + gx((t - j) * kGenRad + j);
        float2 v[kGenRad], w[kGenRad];
#pragma unroll
        for (int r = 0; r < kGenRad; ++r) v[r] = base[r * S + ((r * S) >> 5)];
        if constexpr (S > 1) gen_powers(w, s_tw[j * ts]);
        if constexpr (INV) {
            if constexpr (S > 1) {
#pragma unroll
                for (int r = 1; r < kGenRad; ++r) v[r] = c_mulc(v[r], w[r]);
            }
            dft8<true, false, false, 0>(v);
        } else {
            dft8<false, false, false, 0>(v);
            if constexpr (S > 1) {
#pragma unroll
                for (int r = 1; r < kGenRad; ++r) v[r] = c_mul(v[r], w[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < kGenRad; ++r) base[r * S + ((r * S) >> 5)] = v[r];
    }
}

// The last pass of span 1 when P is not a power of 8: DFTs of R = 2 or 4
// consecutive values (no twiddles; gx(i0 + r) = gx(i0) + r, as R <= 4
// values never cross a 32-slot row).
template <int P, int R, bool INV>
__device__ __forceinline__ void gen_tail(float2 *x)
{
    for (int t = threadIdx.x; t < P / R; t += kGenThreads) {
        float2 *base = x + gx(t * R);
        if constexpr (R == 2) {
            const float2 a = base[0], b = base[1];
            base[0] = c_add(a, b);
            base[1] = c_sub(a, b);
        } else {
            float2 v0 = base[0], v1 = base[1], v2 = base[2], v3 = base[3];
            dft4<INV>(v0, v1, v2, v3);
            base[0] = v0;
            base[1] = v1;
            base[2] = v2;
            base[3] = v3;
        }
    }
}

// the factor of P left after its radix-8 passes (1, 2 or 4)
constexpr int gen_tail_radix(int P)
{
    int R = 1;
    while (R * kGenRad <= P) R *= kGenRad;
    return P / R;
}

// forward passes of spans S, S/8, ..., 1 (each followed by a barrier)
template <int P, int S>
__device__ __forceinline__ void gen_fwd_passes(float2 *x, const float2 *s_tw)
{
    if constexpr (S >= 1) {
        gen_pass<P, S, false>(x, s_tw);
        __syncthreads();
        gen_fwd_passes<P, S / kGenRad>(x, s_tw);
    }
}

// inverse passes of spans S, 8S, ..., P/8
template <int P, int S>
__device__ __forceinline__ void gen_inv_passes(float2 *x, const float2 *s_tw)
{
    if constexpr (S <= P / kGenRad) {
        gen_pass<P, S, true>(x, s_tw);
        __syncthreads();
        gen_inv_passes<P, S * kGenRad>(x, s_tw);
    }
}

// P-point forward transform in LDS (natural order in, digit-reversed out):
// radix-8 passes of spans P/8, P/64, ... and a last radix-2 or 4 pass when
// P is not a power of 8.  Callers synchronise before (the data and s_tw are
// written) and after.
template <int P>
__device__ __forceinline__ void gen_forward(float2 *x, const float2 *s_tw)
{
    gen_fwd_passes<P, P / kGenRad>(x, s_tw);
    constexpr int R = gen_tail_radix(P);
    if constexpr (R > 1) {
        gen_tail<P, R, false>(x);
        __syncthreads();
    }
}

// Exact adjoint of gen_forward: digit-reversed in, natural order out,
// unnormalised exp(+2 pi i nk / P).
template <int P>
__device__ __forceinline__ void gen_inverse(float2 *x, const float2 *s_tw)
{
    constexpr int R = gen_tail_radix(P);
    if constexpr (R > 1) {
        gen_tail<P, R, true>(x);
        __syncthreads();
    }
    gen_inv_passes<P, R>(x, s_tw);
}

// The thread index through an empty asm statement, so that the compiler
// does not hoist the per-lag addresses derived from it out of the loops
// (16 lags x 64-bit addresses, held across the transforms, spill).
__device__ __forceinline__ int opaque_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The one-piece kernels are instantiated per transform length P <= 4096 (LDS
// sized by P, so smaller transforms share a CU) and launched once for each
// length present in a batch; items of requests with another length, or in
// rows, are skipped.

// The chip floor(n 1023000 / fs) of sample n < N, fs = 1000 N: floor(1023 n / N),
// in 32 bits (below 2^24) and already below 1023.
__device__ __forceinline__ int gen_chip(int n, int N) { return (int)((unsigned)n * (unsigned)kCodeLen / (unsigned)N); }

// The spectra of a general-rate request, one launch for both kinds so that
// neither waits for the other: an item is one segment of a PRN's code
// (n_prn of them, first) or of a (Doppler bin, block).
// Code: CC[p][h P + i] = DFT_P(cc_h)[bin of storage position i], cc_h[j] =
// c[(n_h + j) mod N] for j below the segment's length + N, else 0 (one
// segment: c[j mod N] for j < 2N).
// Block: the carrier NCO, first mixing stage and fold (the integer
// arithmetic of the polyphase path), delayed circularly by the code-Doppler
// shift if any, then the zero-padded forward transform.
template <int P>
__global__ __launch_bounds__(kGenThreads) void k_gen_spec(const ReqDesc *__restrict__ R, const BatchHdr *H,
                                                          const long long *pre, const uint8_t *codes,
                                                          const uint32_t *lut, const float2 *tw, float2 *gen)
{
    __shared__ float2 x[P + P / 32];
    __shared__ float2 s_tw[P / kGenRad];
    __shared__ uint32_t s_lut[1024];
    for (int i = threadIdx.x; i < 1024; i += kGenThreads) s_lut[i] = lut[i];
    gen_load_tw(s_tw, P, tw);
    const int n_req = H->n_req;
    const long long total = H->total[kStGenX];
    const long long *pst = pre + (long long)kStGenX * (n_req + 1);
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        if (d.gen_P != P || d.gen_rows) continue;
        const int N = d.N, M = d.gen_M;
        const int S = d.gen_seg ? 2 : 1, seg = d.gen_seg ? gen_segment(N) : N;
        const long long local = it - first_item(pst, n_req, r);
        const long long idx = local / S;
        const int h = (int)(local - idx * S), n0 = h * seg, n1 = min(N, n0 + seg);
        float2 *dst;
        __syncthreads();  // the tables are staged; the previous item's outputs are read
        if (idx < d.n_prn) {
            const uint8_t *code = codes + (long long)d.prns[idx] * kCodeLen;
            dst = gen + d.gen_c_off + idx * M + h * P;
            for (int j = threadIdx.x; j < P; j += kGenThreads) {
                const int n = gen_code_sample(j, n0, n1, N);
                x[gx(j)] = make_float2(n < 0 ? 0.f : code[gen_chip(n, N)] ? -1.f : 1.f, 0.f);
            }
        } else {
            const int kb = (int)(idx - d.n_prn), k = kb / d.Nnc, b = kb - k * d.Nnc;
            const uint32_t D = d.dk[k];
            const int shift = d.cshift ? d.cshift[kb] : 0;
            dst = gen + d.gen_x_off + (long long)kb * M + h * P;
            // samples n0 .. n1 - 1 at [0, n1 - n0), zero above
#pragma unroll 2
            for (int j = threadIdx.x; j < P; j += kGenThreads) {
                float2 f = make_float2(0.f, 0.f);
                if (n0 + j < n1) {
                    int m = n0 + j - shift;
                    if (m < 0) m += N;
                    const int2 v = wipe_fold_one(d.samples, d.fmt, N, d.Tc, s_lut, D, d.b0 + b, m);
                    f = make_float2((float)v.x, (float)v.y);
                }
                x[gx(j)] = f;
            }
        }
        __syncthreads();
        gen_forward<P>(x, s_tw);
        for (int j = threadIdx.x; j < P; j += kGenThreads) dst[j] = x[gx(j)];
    }
}

// One correlation item in one piece, P <= 4096 (see k_gen_corr).
template <int P>
__device__ __forceinline__ void gen_corr_item(const ReqDesc &d, int k, int pi, const float2 *tw, const float2 *gen,
                                              float2 *x, float2 *s_tw)
{
    constexpr int kPer = kGenMaxN / kGenThreads;
    constexpr int kFill = (P + kGenThreads - 1) / kGenThreads;  // spectrum values per thread
    const int N = d.N, M = d.gen_M;  // M = P, or 2 P: two segments
    const float2 *C = gen + d.gen_c_off + (long long)pi * M;
    // 2^-24 (LUT scale) / P^2 (two unnormalised transforms), an exact power of two
    const float scale = ldexpf(1.f, -24 - 2 * (31 - __clz(P)));
    GNSS_GLOBAL float *row = gmem(d.grid) + ((long long)pi * d.n_dopp + k) * N;
    // fill x with the product of block b's spectrum and the code's; the first
    // loads are issued before the barrier that frees x
    auto product = [&](int b, bool first) {
        const float2 *X = gen + d.gen_x_off + ((long long)k * d.Nnc + b) * M;
        const int tid = opaque_tid();
        float2 xv[2][kFill], cv[2][kFill];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h && M == P) break;
#pragma unroll
            for (int u = 0; u < kFill; ++u) {
                const int j = u * kGenThreads + tid;
                if (j < P) {
                    xv[h][u] = X[h * P + j];
                    cv[h][u] = C[h * P + j];
                }
            }
        }
        __syncthreads();  // the previous inverse's outputs are read
        if (first) gen_load_tw(s_tw, P, tw);
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            const int j = u * kGenThreads + tid;
            if (j < P) {
                float2 z = c_mulc(xv[0][u], cv[0][u]);
                if (M > P) z = c_mulc_add(xv[1][u], cv[1][u], z);  // the second segment's product on top
                x[gx(j)] = z;
            }
        }
        __syncthreads();
    };
    // lag tau is output P - N + tau; the sums in groups of kSumGroup blocks,
    // each group's added to the row by the thread that holds it
    for (int b0 = 0; b0 < d.Nnc; b0 += kSumGroup) {
        float acc[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) acc[i] = 0.f;
        const int b1 = min(d.Nnc, b0 + kSumGroup);
        for (int b = b0; b < b1; ++b) {
            product(b, b == 0);
            gen_inverse<P>(x, s_tw);
            const int tid = opaque_tid();
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int tau = tid + kGenThreads * i;
                if (tau < N) {
                    const float2 o = x[gx(P - N + tau)];
                    acc[i] = fmaf(o.x, o.x, fmaf(o.y, o.y, acc[i]));
                }
            }
        }
        const int tid = opaque_tid();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int tau = tid + kGenThreads * i;
            if (tau < N) row[tau] = (b0 || d.acc) ? row[tau] + acc[i] * scale : acc[i] * scale;
        }
    }
}

// Correlation of a general-rate request in one piece, P <= 4096: item =
// (request, Doppler bin, PRN), Doppler-major so that the workgroups running
// together share the block spectra; over the blocks, Z = X conj(CC) (summed
// over the segments), the inverse transform and |.|^2 of the lags' outputs,
// summed in block order in registers; the grid gets sum |out|^2 2^-24 / P^2.
template <int P>
__global__ __launch_bounds__(kGenThreads) void k_gen_corr(const ReqDesc *__restrict__ R, const BatchHdr *H,
                                                          const long long *pre, const float2 *tw,
                                                          const float2 *gen)
{
    __shared__ float2 x[P + P / 32];
    __shared__ float2 s_tw[P / kGenRad];
    const int n_req = H->n_req;
    const long long total = H->total[kStGenCorr];
    const long long *pst = pre + (long long)kStGenCorr * (n_req + 1);
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        if (d.gen_P != P || d.gen_rows) continue;
        const long long local = it - first_item(pst, n_req, r);
        const int k = (int)(local / d.n_prn), pi = (int)(local % d.n_prn);
        gen_corr_item<P>(d, k, pi, tw, gen, x, s_tw);
    }
}

// v W_16^a (forward sign) or v W_16^-a (INV) for a < 8; a is a constant once
// the callers' loops are unrolled
__device__ __forceinline__ float2 twiddle16(float2 v, int a, bool inv)
{
    switch (a) {
    case 0: return v;
    case 1: return inv ? tw<16, 1, true>(v) : tw<16, 1, false>(v);
    case 2: return inv ? tw<16, 2, true>(v) : tw<16, 2, false>(v);
    case 3: return inv ? tw<16, 3, true>(v) : tw<16, 3, false>(v);
    case 4: return inv ? tw<16, 4, true>(v) : tw<16, 4, false>(v);
    case 5: return inv ? tw<16, 5, true>(v) : tw<16, 5, false>(v);
    case 6: return inv ? tw<16, 6, true>(v) : tw<16, 6, false>(v);
    default: return inv ? tw<16, 7, true>(v) : tw<16, 7, false>(v);
    }
}

// a copy the compiler cannot see through (keeps per-column products from
// being hoisted out of loops and held)
__device__ __forceinline__ float2 opaque(float2 v)
{
    asm volatile("" : "+v"(v.x), "+v"(v.y));
    return v;
}

// ---------------------------------------------------------------------------
// P = 4096, 8192, 16384: four-step transforms, R x 2048 with R = P / 2048.
// With n = 2048 a + b and k = k1 + R k2 (a, k1 < R; b, k2 < 2048)
//   X[k1 + R k2] = DFT_2048 over b of ( W_P^(b k1) DFT_R over a of x[2048 a + b] )[k2]:
// a radix-R stage across the R 2048-point rows (in LDS, one column b per
// thread-iteration), then one 2048-point transform per wave (the register
// FFT of the polyphase path, its transposes in the wave's own LDS row).  The
// forward transform's rows end in the 2048-point storage order, so a
// P-point spectrum is stored as [k1][1024 float4] exactly as that FFT leaves
// it; the inverse is the adjoint (2048-point inverse per row, then conjugate
// twiddles and the inverse radix-R stage).  Two workgroup barriers per
// transform instead of one per radix pass.
//
// What bounds the correlation is vector issue and, before that, the waits
// between its phases (spectrum loads, LDS transposes, barriers), which other
// waves have to fill.  So the rows meet the columns in two halves of 1024
// columns each: a transform then needs 64 KB (P = 16384) or 32 KB of LDS for
// its rows beside the 16 KB of twiddles, and two 8-wave workgroups (128
// VGPRs, 8 of them spilled) or three 4-wave ones share a CU.  Measured, 32
// PRNs x 121 bins x 25 blocks at 10 MHz: 3.7 ms, against 4.9 with whole rows
// (148 KB, one workgroup per CU) and 7.84 with the two 16384-point inverses
// per block that two segments replace (the whole search 8.42 -> 4.2 ms, the
// vector work of the correlation 2.6 ms); 32 x 41 x 10 at 5 MHz: 0.62 -> 0.30
// ms, where one 8192-point transform in radix-8 passes took 0.70.  A 4096-
// point workgroup does two PRNs (one twiddle table for both).
// ---------------------------------------------------------------------------
constexpr int kRowMin = 4096;  // shortest transform done in rows
template <int P>
struct RowFft {
    static constexpr int R = P / 2048;              // rows, one wave each
    static constexpr int C = 32 / R;                // columns b per thread
    static constexpr int T = 64 * R;                // threads of a transform
    static constexpr int kGroups = gen_group(P);    // transforms per correlation workgroup
    // rows a segment's samples reach: at most (P + 1) / 3 of them (N + ceil(N/2) <= P)
    static constexpr int kSegRows = ((P + 1) / 3 + 2047) / 2048;
    static_assert(P >= kRowMin && P <= kGenLds && R * C == 32, "four-step lengths");
};

// The 2048-point twiddles without their unit entries (k1 = 0, k2a = 0), so
// that two 80 KB workgroups share a CU's 160 KB.
constexpr int kTrimT1 = 30 * 64, kTrimTw = kTrimT1 + 15 * 8;
__device__ __forceinline__ void stage_twiddles_trim(float2 *s_tw, const float2 *tw, int tid, int nthreads)
{
    for (int i = tid; i < kTrimTw; i += nthreads) {
        int src = kT1Elems + 8 + (i - kTrimT1);
        if (i < kTrimT1) src = i + 64 * (i < 15 * 64 ? 1 : 2);
        s_tw[i] = tw[src];
    }
}

// one column's W_P^(b k1), k1 = 1 .. R - 1, from w1 = W_P^b
template <int R>
__device__ __forceinline__ void row_powers(float2 (&w)[8], float2 w1)
{
    if constexpr (R == 8) {
        gen_powers(w, w1);
    } else {
        w[1] = w1;
        if constexpr (R == 4) {
            w[2] = c_mul(w1, w1);
            w[3] = c_mul(w[2], w1);
        }
    }
}

template <int R, bool INV>
__device__ __forceinline__ void row_dft(float2 (&v)[R])
{
    if constexpr (R == 8) {
        dft8<INV, false, false, 0>(v);
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else {
        const float2 a = v[0], b = v[1];
        v[0] = c_add(a, b);
        v[1] = c_sub(a, b);
    }
}

// Forward radix-R stage: y[k1][b] = W_P^(b k1) sum_a x(2048 a + b) W_R^(a k1)
// for this thread's columns b = tid + T j; x(j, a, b) supplies the input;
// wb[j] = W_P^b (row_bases).
template <int P, typename Src>
__device__ __forceinline__ void row_fwd_stage(float2 *y, int t, const float2 (&wb)[RowFft<P>::C], Src x)
{
    constexpr int R = RowFft<P>::R;
#pragma unroll
    for (int j = 0; j < RowFft<P>::C; ++j) {
        const int b = t + RowFft<P>::T * j;
        float2 v[R], w[8];
#pragma unroll
        for (int a = 0; a < R; ++a) v[a] = x(j, a, b);
        row_dft<R, false>(v);
        row_powers<R>(w, opaque(wb[j]));  // formed here, not hoisted and held
#pragma unroll
        for (int r = 1; r < R; ++r) v[r] = c_mul(v[r], w[r]);
#pragma unroll
        for (int k1 = 0; k1 < R; ++k1) y[k1 * 2048 + b] = v[k1];
        phase_barrier();  // one column at a time (registers)
    }
}

// W_P^b of this thread's columns b, from the table of W_32768^i (loaded once
// per kernel: the stages' column loop would otherwise wait for each)
template <int P>
__device__ __forceinline__ void row_bases(float2 (&wb)[RowFft<P>::C], int t, const float2 *twg)
{
#pragma unroll
    for (int j = 0; j < RowFft<P>::C; ++j) wb[j] = twg[(kGenTwLen / P) * (t + RowFft<P>::T * j)];
}

// Wave k1 transforms row k1 of y (natural order) and stores the storage-order
// result at dst[k1][1024 float4].  The row is the wave's transpose buffer.
__device__ __forceinline__ void row_fwd_rows(float2 *y, int t, const float2 *s_tw, float4 *dst)
{
    const int w = t >> 6, l = t & 63;
    float2 *row = y + w * 2048;
    float2 v[32];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k2b = 0; k2b < 8; ++k2b) v[8 * u + k2b] = row[l + 64 * u + 256 * k2b];
    fft2048<false, true, true>(v, row, s_tw, s_tw + kTrimT1, l);
    float4 *d = dst + w * 1024;
#pragma unroll
    for (int jj = 0; jj < 16; ++jj)
        d[jj * 64 + l] = make_float4(v[2 * jj].x, v[2 * jj].y, v[2 * jj + 1].x, v[2 * jj + 1].y);
}

// Registers 2 jj, 2 jj + 1 of row k1 of X conj(C), J0 <= jj < J0 + NJ (spectra in
// the stored layout); with SEGS = 2 the sum of the two segments' products, the
// second segment P/2 float4 on.  X and C point at this lane of its row.
template <int P, int SEGS, int J0, int NJ>
__device__ __forceinline__ void row_product(float2 (&z)[32], const float4 *X, const float4 *C)
{
    float4 x[SEGS][NJ], c[SEGS][NJ];
#pragma unroll
    for (int i = 0; i < SEGS; ++i)
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            x[i][q] = X[i * (P / 2) + (J0 + q) * 64];
            c[i][q] = C[i * (P / 2) + (J0 + q) * 64];
        }
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
        float2 &z0 = z[2 * (J0 + q)], &z1 = z[2 * (J0 + q) + 1];
        z0 = c_mulc(make_float2(x[0][q].x, x[0][q].y), make_float2(c[0][q].x, c[0][q].y));
        z1 = c_mulc(make_float2(x[0][q].z, x[0][q].w), make_float2(c[0][q].z, c[0][q].w));
        if constexpr (SEGS == 2) {
            z0 = c_mulc_add(make_float2(x[1][q].x, x[1][q].y), make_float2(c[1][q].x, c[1][q].y), z0);
            z1 = c_mulc_add(make_float2(x[1][q].z, x[1][q].w), make_float2(c[1][q].z, c[1][q].w), z1);
        }
    }
}

// Wave k1 transforms its row z back and leaves the natural-order row in y.
__device__ __forceinline__ void row_inv_rows(float2 (&z)[32], float2 *y, int t, const float2 *s_tw)
{
    const int w = t >> 6, l = t & 63;
    float2 *row = y + w * 2048;
    ifft2048<false, true, true>(z, row, s_tw, s_tw + kTrimT1, l);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k2b = 0; k2b < 8; ++k2b) row[l + 64 * u + 256 * k2b] = z[8 * u + k2b];
}

// Column j of the inverse radix-R stage: v[a] = out(2048 a + b) =
// sum_k1 W_R^(-a k1) W_P^(-b k1) y[k1][b], b = t + T j.  LEN: columns of y held
// at a time (2048, or 1024: b mod 1024).
template <int P, int LEN>
__device__ __forceinline__ void row_inv_column(const float2 *y, int t, int j, float2 wb, float2 (&v)[RowFft<P>::R])
{
    constexpr int R = RowFft<P>::R;
    const int b = t + RowFft<P>::T * (j % (RowFft<P>::C * LEN / 2048));
    float2 w[8];
#pragma unroll
    for (int k1 = 0; k1 < R; ++k1) v[k1] = y[k1 * LEN + b];
    row_powers<R>(w, opaque(wb));  // formed here, not hoisted and held
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = c_mulc(v[r], w[r]);
    row_dft<R, true>(v);
}

// The wipe-off and fold of this thread's samples n = n0 + 2048 a + t + T j
// (a < NA, j < C) of block b (zero at n >= n1), delayed circularly by shift:
// the values of wipe_fold_one, mixed by dot products (mix_add) with the
// milliseconds outermost, so that the samples' loads of one millisecond are in
// flight together.  In-block offsets have 32 bits (Tc N <= 64 * 16384 samples), and the
// phase advances by N D (mod 2^32) from one millisecond to the next.  Vector issue is
// what it costs: at 10 MHz (121 bins x 25 blocks of 4 ms, P = 16384) the spectra took
// 0.50 ms with bytes, products and a 64-bit index per sample, and take 0.34.
template <int FMT, int P, int NA>
__device__ __forceinline__ void row_fold_fmt(const ReqDesc &d, int b, uint32_t D, int shift, const uint2 *s_lut,
                                             int t, int n0, int n1, float2 (&f)[RowFft<P>::C][NA])
{
    constexpr int C = RowFft<P>::C;
    constexpr uint32_t kUnit = FMT == GNSS_CPLX_I8 ? 2u : 1u;
    const int N = d.N, Tc = d.Tc;
    const uint32_t dN = (uint32_t)N * D;
    const long long base = (long long)(d.b0 + b) * Tc * N;
    // 2-bit packed records: the block may start inside a byte
    const uint32_t sub = FMT == GNSS_REAL_2BIT_PACKED ? (uint32_t)(base & 3) : 0u;
    const long long blk_byte = FMT == GNSS_CPLX_I8 ? 2 * base : FMT == GNSS_REAL_I8 ? base : (base >> 2);
    const GNSS_GLOBAL uint8_t *blk = (const GNSS_GLOBAL uint8_t *)d.samples + blk_byte;
    const uint32_t step = kUnit * (uint32_t)N;  // bytes (samples if packed)
    const uint32_t ph0 = (uint32_t)(base + n0 + t - shift) * D;
    int yr[C][NA], yi[C][NA];
    uint32_t off[C][NA], ph[C][NA];
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            const int n = n0 + 2048 * a + t + RowFft<P>::T * j;
            int m = n - shift;
            uint32_t p = ph0 + (uint32_t)(2048 * a + RowFft<P>::T * j) * D;
            if (m < 0) {
                m += N;
                p += dN;
            }
            off[j][a] = kUnit * (uint32_t)(n < n1 ? m : 0) + sub;  // (not used past n1)
            ph[j][a] = p;
            yr[j][a] = 0;
            yi[j][a] = 0;
        }
#pragma unroll 1
    for (int c = 0; c < Tc; ++c) {
#pragma unroll
        for (int j = 0; j < C; ++j)
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                mix_add(load_mix<FMT>(blk, off[j][a]), s_lut[ph[j][a] >> 22], yr[j][a], yi[j][a]);
                if (FMT == GNSS_REAL_2BIT_PACKED) off[j][a] += step;
                ph[j][a] += dN;
            }
        if (FMT != GNSS_REAL_2BIT_PACKED) blk += step;
    }
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            const bool in = n0 + 2048 * a + t + RowFft<P>::T * j < n1;
            f[j][a] = in ? make_float2((float)yr[j][a], (float)yi[j][a]) : make_float2(0.f, 0.f);
        }
}

template <int P, int NA>
__device__ __forceinline__ void row_fold(const ReqDesc &d, int b, uint32_t D, int shift, const uint2 *s_lut, int t,
                                         int n0, int n1, float2 (&f)[RowFft<P>::C][NA])
{
    if (d.fmt == GNSS_CPLX_I8)
        row_fold_fmt<GNSS_CPLX_I8, P, NA>(d, b, D, shift, s_lut, t, n0, n1, f);
    else if (d.fmt == GNSS_REAL_I8)
        row_fold_fmt<GNSS_REAL_I8, P, NA>(d, b, D, shift, s_lut, t, n0, n1, f);
    else
        row_fold_fmt<GNSS_REAL_2BIT_PACKED, P, NA>(d, b, D, shift, s_lut, t, n0, n1, f);
}

// Spectra in rows (see k_gen_spec).  The carrier table lies in the
// transform's LDS, which the fold does not need yet.  M = 2 P without
// segments (P = 16384): an item does the even and then the odd bins.
template <int P>
__global__ __launch_bounds__(RowFft<P>::T) void k_gen_spec_rows(const ReqDesc *__restrict__ R, const BatchHdr *H,
                                                                const long long *pre, const uint8_t *codes,
                                                                const uint32_t *lut, const float2 *tw,
                                                                const float2 *twg, float2 *gen)
{
    using F = RowFft<P>;
    constexpr int NS = F::kSegRows;
    __shared__ float2 y[P];
    __shared__ float2 s_tw[kTrimTw];
    uint2 *s_lut = (uint2 *)y;
    stage_twiddles_trim(s_tw, tw, threadIdx.x, F::T);
    const int n_req = H->n_req;
    const long long total = H->total[kStGenX];
    const long long *pst = pre + (long long)kStGenX * (n_req + 1);
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        if (d.gen_P != P || !d.gen_rows) continue;
        const int N = d.N, M = d.gen_M;
        const int S = d.gen_seg ? 2 : 1, seg = d.gen_seg ? gen_segment(N) : N;
        const long long local = it - first_item(pst, n_req, r);
        const long long idx = local / S;
        const int h = (int)(local - idx * S), n0 = h * seg, n1 = min(N, n0 + seg);
        const bool halves = P == kGenLds && !d.gen_seg && M > P;
        const int t = opaque_tid();
        float2 f[F::C][F::R], wb[F::C];
        float4 *dst;
        __syncthreads();  // the previous item's rows are read
        if (idx < d.n_prn) {
            const uint8_t *code = codes + (long long)d.prns[idx] * kCodeLen;
            auto cc = [&](int j) -> float {
                const int n = gen_code_sample(j, n0, n1, N);
                return n < 0 ? 0.f : code[gen_chip(n, N)] ? -1.f : 1.f;
            };
#pragma unroll
            for (int j = 0; j < F::C; ++j)
#pragma unroll
                for (int a = 0; a < F::R; ++a) {
                    // (x[n], x[n + P]) with two halves, else (x[n], 0): x is real
                    const int n = 2048 * a + t + F::T * j;
                    f[j][a] = make_float2(cc(n), halves ? cc(n + P) : 0.f);
                }
            dst = (float4 *)(gen + d.gen_c_off + idx * M) + h * (P / 2);
        } else {
            const int kb = (int)(idx - d.n_prn), k = kb / d.Nnc, b = kb - k * d.Nnc;
            const uint32_t D = d.dk[k];
            const int shift = d.cshift ? d.cshift[kb] : 0;
            stage_mix_lut(s_lut, lut, threadIdx.x, F::T);
            __syncthreads();
            // the first rows only, where the rest is zero
            auto fold = [&](auto na) {
                constexpr int NA = decltype(na)::value;
                float2 g[F::C][NA];
                row_fold<P, NA>(d, b, D, shift, s_lut, t, n0, n1, g);
#pragma unroll
                for (int j = 0; j < F::C; ++j)
#pragma unroll
                    for (int a = 0; a < F::R; ++a) f[j][a] = a < NA ? g[j][a < NA ? a : 0] : make_float2(0.f, 0.f);
            };
            if (d.gen_seg)  // rows a >= NS are zero
                fold(std::integral_constant<int, NS>());
            else if (2 * N <= P)  // M = P
                fold(std::integral_constant<int, F::R / 2>());
            else  // N = M, or N <= M/2 = P (zeros above, so none at n + P)
                fold(std::integral_constant<int, F::R>());
            dst = (float4 *)(gen + d.gen_x_off + (long long)kb * M) + h * (P / 2);
            __syncthreads();  // the carrier table is read
        }
        row_bases<P>(wb, t, twg);
        const bool two_reals = halves && idx < d.n_prn;
        row_fwd_stage<P>(y, t, wb, [&](int j, int a, int) -> float2 {
            return two_reals ? make_float2(f[j][a].x + f[j][a].y, 0.f) : f[j][a];
        });
        __syncthreads();
        row_fwd_rows(y, t, s_tw, dst);
        if (halves) {
            // the odd bins: (x[n] - x[n + P]) W_M^n, n = 2048 a + b: W_M^b W_16^a
            float2 wm[F::C];
#pragma unroll
            for (int j = 0; j < F::C; ++j) wm[j] = twg[t + F::T * j];
            __syncthreads();  // the even bins' rows are read
            row_fwd_stage<P>(y, t, wb, [&](int j, int a, int) -> float2 {
                const float2 v = two_reals ? make_float2(f[j][a].x - f[j][a].y, 0.f) : f[j][a];
                return twiddle16(c_mul(v, opaque(wm[j])), a, false);
            });
            __syncthreads();
            row_fwd_rows(y, t, s_tw, dst + P / 2);
        }
    }
}

// Correlation in rows (see k_gen_corr): item = (request, Doppler bin, group
// of gen_group(P) PRNs, one transform each), Doppler-major; this thread's
// lags are the outputs n = 2048 a + b_j at or above P - N, their sums in
// registers in groups of kSumGroup blocks.  MODE 1, 2: one and two segments;
// MODE 0 (P = 16384, M = 32768): two inverses, of the even and the odd bins,
// the first one's outputs A kept beside the sums.  Requests of another length
// or mode are skipped.
template <int P, int MODE>
__global__ __launch_bounds__(RowFft<P>::T *RowFft<P>::kGroups)
    __attribute__((amdgpu_waves_per_eu(MODE == 0 ? 2 : P == kGenLds ? 4 : 3))) void k_gen_corr_rows(
    const ReqDesc *__restrict__ R, const BatchHdr *H, const long long *pre, const float2 *tw, const float2 *twg,
    const float2 *gen)
{
    using F = RowFft<P>;
    // one and two segments: the rows and columns meet in halves of 1024
    // columns, so that more waves share a CU
    constexpr int LEN = MODE == 0 ? 2048 : 1024;
    __shared__ float2 ys[F::kGroups * F::R * LEN];
    __shared__ float2 s_tw[kTrimTw];
    stage_twiddles_trim(s_tw, tw, threadIdx.x, F::T * F::kGroups);
    const int n_req = H->n_req;
    const long long total = H->total[kStGenCorr];
    const long long *pst = pre + (long long)kStGenCorr * (n_req + 1);
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const int N = d.N, M = d.gen_M;
        if (d.gen_P != P || !d.gen_rows || MODE != (M == P ? 1 : d.gen_seg ? 2 : 0)) continue;
        const long long local = it - first_item(pst, n_req, r);
        const int n_grp = (d.n_prn + F::kGroups - 1) / F::kGroups;
        const int k = (int)(local / n_grp);
        // the transform's threads t and PRN; a PRN past the list's end repeats the last one, unwritten
        const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / F::T);
        const int pl = (int)(local % n_grp) * F::kGroups + grp;
        const bool written = pl < d.n_prn;
        const int pi = written ? pl : d.n_prn - 1;
        float2 *y = ys + grp * F::R * LEN;
        const float scale = ldexpf(1.f, -24 - 2 * (31 - __clz(MODE ? P : 2 * P)));
        GNSS_GLOBAL float *row = gmem(d.grid) + ((long long)pi * d.n_dopp + k) * N;
        const float4 *C0 = (const float4 *)(gen + d.gen_c_off + (long long)pi * M);
        const float4 *X0 = (const float4 *)(gen + d.gen_x_off + (long long)k * d.Nnc * M);
        // this lane of its row of block b's spectrum and of the code's (opaque,
        // so that no address is hoisted out of the loops and held)
        auto lane = [&](const float4 *base) {
            const int t = opaque_tid() - grp * F::T;
            return base + (t >> 6) * 1024 + (t & 63);
        };
        // the sums in groups of kSumGroup blocks, each group's added to the row
        // by the thread that holds it
        for (int b0 = 0; b0 < d.Nnc; b0 += kSumGroup) {
            float acc[F::C][F::R];
#pragma unroll
            for (int j = 0; j < F::C; ++j)
#pragma unroll
                for (int a = 0; a < F::R; ++a) acc[j][a] = 0.f;
            const int b1 = min(d.Nnc, b0 + kSumGroup);
            for (int b = b0; b < b1; ++b) {
                const float4 *X = X0 + (long long)b * (M / 2);
                float2 z[32];
                if constexpr (MODE == 0) {
                    row_product<P, 1, 0, 16>(z, lane(X), lane(C0));
                } else {
                    constexpr int NJ = P == kGenLds ? 2 : 4;
                    const float4 *xl = lane(X), *cl = lane(C0);
                    unrolled<16 / NJ>([&](auto jc) {
                        row_product<P, MODE, decltype(jc)::value * NJ, NJ>(z, xl, cl);
                        phase_barrier();
                    });
                }
                __syncthreads();  // the twiddles are staged, the previous stage's reads of y done
                int t = opaque_tid() - grp * F::T;
                if constexpr (MODE != 0) {
                    // the wave's transposes go through its own row of y, which its
                    // half row of results then fills
                    float2 *row_y = y + (t >> 6) * LEN;
                    ifft2048<false, true, true, true>(z, row_y, s_tw, s_tw + kTrimT1, t & 63);
                    auto half = [&](auto hc) {
                        constexpr int h = decltype(hc)::value;
                        // this half's W_P^b (needed after the barrier; held through the
                        // transform they would not fit the registers)
                        float2 wb[F::C / 2];
#pragma unroll
                        for (int jj = 0; jj < F::C / 2; ++jj)
                            wb[jj] = twg[(kGenTwLen / P) * (t + F::T * (h * (F::C / 2) + jj))];
                        if (h) __syncthreads();  // the first half's columns are read
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int k2b = 0; k2b < 4; ++k2b)
                                row_y[(t & 63) + 64 * u + 256 * k2b] = z[8 * u + 4 * h + k2b];
                        __syncthreads();
                        // lag tau = n - (P - N)
#pragma unroll
                        for (int jj = 0; jj < F::C / 2; ++jj) {
                            const int j = h * (F::C / 2) + jj;
                            float2 v[F::R];
                            row_inv_column<P, LEN>(y, t, j, wb[jj], v);
#pragma unroll
                            for (int a = 0; a < F::R; ++a) {
                                const int n = 2048 * a + t + F::T * j;
                                if (n >= P - N) acc[j][a] = fmaf(v[a].x, v[a].x, fmaf(v[a].y, v[a].y, acc[j][a]));
                            }
                            phase_barrier();  // one column at a time (registers)
                        }
                    };
                    half(std::integral_constant<int, 0>());
                    half(std::integral_constant<int, 1>());
                } else {
                    row_inv_rows(z, y, t, s_tw);
                    __syncthreads();
                    // lag tau is output P + kk, kk = n - (P - N): A - W_M^-kk B
                    float2 A[F::C][F::R], wb[F::C], wm[F::C];
                    row_bases<P>(wb, t, twg);
#pragma unroll
                    for (int j = 0; j < F::C; ++j) {
                        row_inv_column<P, LEN>(y, t, j, wb[j], A[j]);
                        phase_barrier();
                    }
                    row_product<P, 1, 0, 16>(z, lane(X + P / 2), lane(C0 + P / 2));
                    __syncthreads();
                    t = opaque_tid() - grp * F::T;
                    row_inv_rows(z, y, t, s_tw);
                    __syncthreads();
                    t = opaque_tid() - grp * F::T;
#pragma unroll
                    for (int j = 0; j < F::C; ++j) wm[j] = twg[t + F::T * j];
#pragma unroll
                    for (int j = 0; j < F::C; ++j) {
                        float2 v[F::R];
                        row_inv_column<P, LEN>(y, t, j, wb[j], v);
#pragma unroll
                        for (int a = 0; a < F::R; ++a) {
                            const int n = 2048 * a + t + F::T * j;
                            if (n >= P - N) {
                                // W_M^-n = conj(W_M^b) W_16^-a
                                const float2 o = c_sub(A[j][a], twiddle16(c_mulc(v[a], opaque(wm[j])), a, true));
                                acc[j][a] = fmaf(o.x, o.x, fmaf(o.y, o.y, acc[j][a]));
                            }
                        }
                        phase_barrier();
                    }
                }
            }
            const int t = opaque_tid() - grp * F::T;
            if (written) {
#pragma unroll
                for (int j = 0; j < F::C; ++j)
#pragma unroll
                    for (int a = 0; a < F::R; ++a) {
                        const int n = 2048 * a + t + F::T * j;
                        if (n >= P - N) {
                            GNSS_GLOBAL float *o = row + (n - (P - N));
                            *o = (b0 || d.acc) ? *o + acc[j][a] * scale : acc[j][a] * scale;
                        }
                    }
            }
        }
    }
}

// ===========================================================================
// detection: column max over Doppler, argmax, second peak, mean; refinement
// ===========================================================================
// Sum over the first wave's lanes in a fixed binary tree (32 + 32, 16 + 16, ...);
// lane 0 has it.
__device__ __forceinline__ float wave_tree_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    return v;
}

// Work item = (request, PRN, block of 256 lags).  Q[tau] = max_k P (lowest k
// on ties), K = that k; part = the block's FP32 sum of P: each column summed
// in row order, then the block's columns in a fixed binary tree, so the mean
// does not depend on scheduling.  The relative error of a sum of positive
// terms is at most (depth of its addition tree) * 2^-24.
__global__ __launch_bounds__(kPeakThreads) void k_colmax(const ReqDesc *__restrict__ R, BatchHdr *H,
                                                         const long long *pre, float *Q, int32_t *K,
                                                         float *part)
{
    __shared__ float red[kPeakThreads];
    const int n_req = H->n_req;
    const long long total = H->total[kStColmax];
    const long long *pst = pre + (long long)kStColmax * (n_req + 1);
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const long long local = it - first_item(pst, n_req, r);
        const int p = (int)(local / d.n_tau_blk), blk = (int)(local % d.n_tau_blk);
        const int N = d.N, tau = blk * kPeakThreads + threadIdx.x;
        float colsum = 0.f;
        if (tau < N) {
            const GNSS_GLOBAL float *col = gmem(d.grid) + (long long)p * d.n_dopp * N + tau;
            float best = col[0];
            int kb = 0;
            colsum = best;
            int k = 1;
            // eight rows' loads in flight at a time; max and sum in row order
            for (; k + 8 <= d.n_dopp; k += 8) {
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = col[(long long)(k + j) * N];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    colsum += v[j];
                    if (v[j] > best) {
                        best = v[j];
                        kb = k + j;
                    }
                }
            }
            for (; k < d.n_dopp; ++k) {
                float v = col[(long long)k * N];
                colsum += v;
                if (v > best) {
                    best = v;
                    kb = k;
                }
            }
            Q[d.qk_off + (long long)p * N + tau] = best;
            K[d.qk_off + (long long)p * N + tau] = kb;
        }
        __syncthreads();
        red[threadIdx.x] = colsum;
        __syncthreads();
        // the tree's upper levels in LDS, the last six in the first wave
        for (int st = kPeakThreads / 2; st >= 64; st >>= 1) {
            if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x < 64) {
            const float v = wave_tree_sum(red[threadIdx.x]);
            if (threadIdx.x == 0) part[d.part_off + (long long)p * d.n_tau_blk + blk] = v;
        }
    }
}

__device__ __forceinline__ double parabola(double ym, double y0, double yp)
{
    double den = ym - 2.0 * y0 + yp;
    if (den == 0.0) return 0.0;
    return 0.5 * (ym - yp) / den;
}

// Work item = (request, PRN): argmax (lowest tau on ties), second peak outside
// +-spc (circular), mean, ratio test, and the FP64 sub-bin refinement (the only
// FP64 arithmetic of a search on the device: the carrier and code-Doppler
// steps are computed on the host; FP64 elsewhere in this file builds the
// constant tables once per context: the carrier LUT, twiddles and exact-length
// code spectra).  Latency is what it costs: each thread keeps its column
// maxima in registers (up to kPeakLags lags, read once, all loads in flight;
// a longer grid of the caller's is read twice) and the reductions are wave
// shuffles and one exchange in LDS, three barriers in all; with LDS trees,
// forty barriers and the refinement as a launch of its own a strong-signal
// search (32 PRNs, 21 bins, 4092 lags) spent 11.1 us here and spends 7.0.
__global__ __launch_bounds__(kArgThreads) void k_peak(const ReqDesc *__restrict__ R, BatchHdr *H,
                                                       const long long *pre, const float *Q,
                                                       const int32_t *K, const float *part)
{
    constexpr int kWaves = kArgThreads / 64, kPer = kPeakLags / kArgThreads;
    __shared__ float sv[kWaves], sm[kWaves], su[kWaves];
    __shared__ int st[kWaves];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int n_req = H->n_req;
    const long long total = H->total[kStPeak];
    const long long *pst = pre + (long long)kStPeak * (n_req + 1);
    for (long long it = blockIdx.x; it < total; it += gridDim.x) {
        const int r = find_req(pst, n_req, it);
        const ReqDesc &d = R[r];
        const int p = (int)(it - first_item(pst, n_req, r));
        const int N = d.N;
        const float *q = Q + d.qk_off + (long long)p * N;
        // the blocks' partial sums in a fixed binary tree (FP32)
        float ps = 0.f;
        for (int i = tid; i < d.n_tau_blk; i += kArgThreads) ps += part[d.part_off + (long long)p * d.n_tau_blk + i];
        ps = wave_tree_sum(ps);
        float v[kPer];
        auto load = [&](unsigned t0) {
#pragma unroll
            for (int j = 0; j < kPer; ++j) v[j] = t0 + j * kArgThreads < (unsigned)N ? q[t0 + j * kArgThreads] : -INFINITY;
        };
        float bv = -INFINITY;
        int bt = 0x7fffffff;
        for (unsigned t0 = tid; t0 < (unsigned)N; t0 += kPeakLags) {
            load(t0);
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (v[j] > bv) {
                    bv = v[j];
                    bt = (int)t0 + j * kArgThreads;
                }
        }
        // the row of this thread's own maximum: used if it is the overall one
        const int own = bt;
        const int kown = K[d.qk_off + (long long)p * N + (own < N ? own : 0)];
        auto better = [&](float v2, int t2) {
            if (v2 > bv || (v2 == bv && t2 < bt)) {
                bv = v2;
                bt = t2;
            }
        };
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float v2 = __shfl_xor(bv, o);
            const int t2 = __shfl_xor(bt, o);
            better(v2, t2);
        }
        __syncthreads();  // the previous item's reads of the exchange are done
        if (l == 0) {
            sv[w] = bv;
            st[w] = bt;
        }
        __syncthreads();
        for (int i = 0; i < kWaves; ++i) better(sv[i], st[i]);
        // a grid with no ordered maximum (all NaN) leaves tau* unset: keep it in range
        const int tstar = (bt >= 0 && bt < N) ? bt : 0;
        // The refinement's samples are loaded by the thread that found the maximum,
        // behind the search for the second peak: parabolas along tau (circular) and
        // along Doppler (not at the ends).
        const bool owner = own == tstar || (bt != tstar && tid == 0);
        const int nd = d.n_dopp, k = kown;
        const bool inner = k > 0 && k < nd - 1;
        float y0 = 0.f, tm = 0.f, tp = 0.f, km = 0.f, kp = 0.f;
        if (owner) {
            const GNSS_GLOBAL float *row = gmem(d.grid) + ((long long)p * nd + k) * N;
            y0 = row[tstar];
            tm = row[tstar ? tstar - 1 : N - 1];
            tp = row[tstar + 1 < N ? tstar + 1 : 0];
            km = row[tstar - (inner ? (long long)N : 0)];
            kp = row[tstar + (inner ? (long long)N : 0)];
        }
        float m2 = -INFINITY;
        for (unsigned t0 = tid; t0 < (unsigned)N; t0 += kPeakLags) {
            if (N > kPeakLags) load(t0);
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                int dd = abs((int)t0 + j * kArgThreads - tstar);
                dd = min(dd, N - dd);
                if (dd > d.spc) m2 = fmaxf(m2, v[j]);  // past the last lag: -infinity
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m2 = fmaxf(m2, __shfl_xor(m2, o));
        if (l == 0) {
            sm[w] = m2;
            su[w] = ps;
        }
        __syncthreads();
        if (owner) {
#pragma unroll
            for (int i = 0; i < kWaves; ++i) m2 = fmaxf(m2, sm[i]);
            float us[kWaves];
#pragma unroll
            for (int i = 0; i < kWaves; ++i) us[i] = su[i];
#pragma unroll
            for (int o = kWaves / 2; o > 0; o >>= 1)
#pragma unroll
                for (int i = 0; i < o; ++i) us[i] += us[i + o];
            const float second = m2 == -INFINITY ? 0.f : m2;
            const double dc = parabola(tm, y0, tp), dd = inner ? parabola(km, y0, kp) : 0.0;
            const double fk = __dadd_rn(d.lo, __dmul_rn((double)k, d.step));
            gnss_peak rr;
            rr.prn = d.prns[p];
            rr.doppler_bin = k;
            rr.code_phase = tstar;
            rr.peak = bv;
            rr.second = second;
            rr.mean = us[0] / ((float)nd * (float)N);
            rr.ratio = second > 0.f ? bv / second : INFINITY;
            rr.detected = rr.ratio >= d.threshold ? 1 : 0;
            rr.doppler_hz = __dadd_rn(fk, __dmul_rn(dd, d.step));
            rr.code_phase_frac = __dadd_rn((double)tstar, dc);
            d.peaks[p] = rr;
        }
    }
}

// ===========================================================================
// launch of a whole batch (or of its detection stages only)
// ===========================================================================
template <typename K>
static int occupancy(K kernel, int threads, int n_cu)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return per_cu * n_cu;
}

// Grid of a stage with `work` items: one workgroup per item, or, for a
// persistent launch (or a stage too large for one grid), `cap` workgroups
// that take items from the work counters.  At least one workgroup per XCD.
static unsigned grid_for(long long work, long long cap, bool persistent)
{
    long long g = work;
    if ((persistent && g > cap) || g > 0x7fffffffLL) g = cap;
    if (g < kXcds) g = kXcds;
    return (unsigned)g;
}

// The wipe + fold + boxcar + polyphase stage of a staged batch alone, launched
// exactly as launch_batch launches it in the FP16 modes (stage entry point; an FP32
// search runs the same front end inside k_box_fft).
hipError_t launch_box(const Launch &L, const uint32_t *d_lut, int2 *d_F, int n_cu, hipStream_t s)
{
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, s, L.hdr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || L.total[kStBox] == 0) return e;
    static int cap = 0;
    if (!cap) cap = occupancy(k_box, kBfThreads, n_cu);
    hipLaunchKernelGGL(k_box, dim3(grid_for(L.total[kStBox], cap, false)), dim3(kBfThreads), 0, s, L.reqs, L.hdr, L.pre,
                       d_lut, d_F);
    return hipGetLastError();
}

// Frequency-domain Doppler: long DFT of every block (two passes), then the
// block spectra of every (Doppler, block) item; replaces k_box and k_fft_x.
static hipError_t launch_fd(const Launch &L, const Tables &T, void *d_fd, void *d_G, int *d_E, int n_cu,
                            hipStream_t s)
{
    hipError_t e;
    if (L.total[kStFdA] > 0) {
        static int cap = 0;
        if (!cap) cap = occupancy(k_fd_pass1, 256, n_cu);
        hipLaunchKernelGGL(k_fd_pass1, dim3(grid_for((L.total[kStFdA] + 3) / 4, cap, false)), dim3(256), 0, s,
                           L.reqs, L.hdr, L.pre, (const pfa::u4 *)T.frags_x, (float2 *)d_fd);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        static int cap2 = 0;
        if (!cap2) cap2 = occupancy(k_fd_pass2, 256, n_cu);
        hipLaunchKernelGGL(k_fd_pass2, dim3(grid_for(L.total[kStFdB], cap2, false)), dim3(256), 0, s,
                           L.reqs, L.hdr, L.pre, (float2 *)d_fd);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (L.total[kStBox] > 0) {
        static int cap = 0;
        if (!cap) cap = occupancy(k_fd_synth, kSynthThreads, n_cu);
        hipLaunchKernelGGL(k_fd_synth, dim3(grid_for(L.total[kStBox], cap, false)), dim3(kSynthThreads), 0, s,
                           L.reqs, L.hdr, L.pre, (const float2 *)d_fd, (pfa::u4 *)d_G, d_E);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// Calls f(std::integral_constant<int, Q>()) for each general-rate transform
// length Q >= P whose bit is set in mask (bit Q, a power of two), in
// increasing order; stops at the first error.
template <int P, typename F>
static hipError_t gen_lengths(unsigned mask, F &f)
{
    if constexpr (P > kGenLds) {
        return hipSuccess;
    } else {
        if (mask & (unsigned)P) {
            const hipError_t e = f(std::integral_constant<int, P>());
            if (e != hipSuccess) return e;
        }
        return gen_lengths<P * 2>(mask, f);
    }
}

hipError_t launch_batch(const Launch &L, const Tables &T, int2 *d_F, void *d_G, float *d_Q, int32_t *d_K,
                        float *d_part, int n_cu, hipStream_t s, hipEvent_t *marks)
{
    const uint32_t *d_lut = T.lut;
    const void *d_cs = T.cs;
    const bool h = L.precision == GNSS_FP16, x = L.precision == GNSS_FP16_PFA;
    // FP16 modes: packed spectra, then the per-vector exponents
    uint4 *d_Gh = (uint4 *)d_G;
    int *d_E = (int *)((char *)d_G + g_spectra_bytes(L.total[kStVec], L.precision));
    float2 *d_Dc = (float2 *)((char *)d_E + round256((size_t)L.total[kStVec] * 4));  // GNSS_FP16 only
    const float *d_dck = h ? (const float *)((const char *)T.cs_h + kCsHSpecBytes) : nullptr;
    hipError_t e;
    const bool pers = L.persistent != 0;
    auto mark = [&](int i) -> hipError_t { return marks ? hipEventRecord(marks[i], s) : hipSuccess; };
    if (!L.fresh) {
        hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, s, L.hdr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = mark(0)) != hipSuccess) return e;
    if (x && L.fd) {
        if ((e = launch_fd(L, T, d_F, d_G, d_E, n_cu, s)) != hipSuccess) return e;
    } else if (!x && !h) {
        if (L.total[kStBoxFft] > 0) {
            hipLaunchKernelGGL(k_box_fft, dim3((unsigned)std::min(L.total[kStBoxFft], 0x7fffffffLL)), dim3(kBfThreads),
                               0, s, L.reqs, L.hdr, L.pre, d_lut, T.tw_gen, (float4 *)d_G);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    } else if (L.total[kStBox] > 0) {
        static int cap = 0;
        if (!cap) cap = occupancy(k_box, kBfThreads, n_cu);
        hipLaunchKernelGGL(k_box, dim3(grid_for(L.total[kStBox], cap, false)), dim3(kBfThreads), 0, s, L.reqs,
                           L.hdr, L.pre, d_lut, d_F);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = mark(1)) != hipSuccess) return e;
    if (x && L.fd) {
        // the block spectra are already written
    } else if (L.total[kStVec] > 0 && x) {
        static int cap = 0;
        if (!cap) cap = occupancy(k_fft_x, 256, n_cu);
        hipLaunchKernelGGL(k_fft_x, dim3(grid_for((L.total[kStVec] + 3) / 4, cap, false)), dim3(256), 0, s, d_F,
                           (const pfa::u4 *)T.frags_x, (pfa::u4 *)d_G, d_E, L.hdr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (L.total[kStVec] > 0 && h) {
        static int cap = 0;
        if (!cap) cap = occupancy(k_fft_poly_h, 256, n_cu);
        hipLaunchKernelGGL(k_fft_poly_h, dim3(grid_for((L.total[kStVec] + 7) / 8, cap, false)), dim3(256), 0,
                           s, d_F, (const hc2 *)T.tw_h, d_Gh, d_E, d_Dc, L.hdr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (L.total[kStGenX] > 0) {  // general rates: code spectra and block spectra
        float2 *d_gen = (float2 *)((char *)d_G + L.gen_off);
        auto spectra = [&](auto pc) -> hipError_t {
            constexpr int P = decltype(pc)::value;
            const unsigned wgs = grid_for(L.total[kStGenX], 65535, false);
            if constexpr (P >= kRowMin) {
                if (L.gen_rmask & (unsigned)P) {
                    constexpr int kT = RowFft<P>::T;
                    hipLaunchKernelGGL(k_gen_spec_rows<P>, dim3(wgs), dim3(kT), 0, s, L.reqs, L.hdr, L.pre, T.codes,
                                       d_lut, T.tw, T.tw_gen, d_gen);
                    const hipError_t e2 = hipGetLastError();
                    if (e2 != hipSuccess) return e2;
                }
            }
            if constexpr (P <= kRowMin) {
                if (L.gen_pmask & (unsigned)P)
                    hipLaunchKernelGGL(k_gen_spec<P>, dim3(wgs), dim3(kGenThreads), 0, s, L.reqs, L.hdr, L.pre,
                                       T.codes, d_lut, T.tw_gen, d_gen);
            }
            return hipGetLastError();
        };
        if ((e = gen_lengths<64>(L.gen_pmask | L.gen_rmask, spectra)) != hipSuccess) return e;
    }
    if ((e = mark(2)) != hipSuccess) return e;
    if (L.total[kStGenCorr] > 0) {
        const float2 *d_gen = (const float2 *)((char *)d_G + L.gen_off);
        auto corr = [&](auto pc) -> hipError_t {
            constexpr int P = decltype(pc)::value;
            const unsigned wgs = grid_for(L.total[kStGenCorr], 65535, false);
            if constexpr (P >= kRowMin) {
                if (L.gen_rmask & (unsigned)P) {
                    // one instance per mode present (see k_gen_corr_rows)
                    auto rows = [&](auto kernel, int mode) -> hipError_t {
                        if (!(L.gen_modes >> mode & 1)) return hipSuccess;
                        hipLaunchKernelGGL(kernel, dim3(wgs), dim3(RowFft<P>::T * RowFft<P>::kGroups), 0, s, L.reqs,
                                           L.hdr, L.pre, T.tw, T.tw_gen, d_gen);
                        return hipGetLastError();
                    };
                    hipError_t e2 = rows(k_gen_corr_rows<P, 1>, 1);
                    if (e2 == hipSuccess) e2 = rows(k_gen_corr_rows<P, 2>, 2);
                    if constexpr (P == kGenLds) {
                        if (e2 == hipSuccess) e2 = rows(k_gen_corr_rows<P, 0>, 0);
                    }
                    if (e2 != hipSuccess) return e2;
                }
            }
            if constexpr (P <= kRowMin) {
                if (L.gen_pmask & (unsigned)P)
                    hipLaunchKernelGGL(k_gen_corr<P>, dim3(wgs), dim3(kGenThreads), 0, s, L.reqs, L.hdr, L.pre,
                                       T.tw_gen, d_gen);
            }
            return hipGetLastError();
        };
        if ((e = gen_lengths<64>(L.gen_pmask | L.gen_rmask, corr)) != hipSuccess) return e;
    }
    if (L.total[kStCorr] > 0 && x) {
        // the frequency-domain variant wipes with unit exponentials (no LUT scale 2^12)
        const float osc = ldexpf(1.f, 2 * T.cs_exp - (L.fd ? 0 : 24)) / (float)(kCodeLen * kCodeLen);
        // the pair variant is a separate instantiation: its registers would halve the
        // plain kernel's occupancy
        if (L.nav_pairs) {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr_x<true>, 64 * kCorrWavesX, n_cu);
            hipLaunchKernelGGL(k_corr_x<true>, dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * kCorrWavesX),
                               0, s, L.reqs, L.hdr, L.pre, (const pfa::u4 *)d_G, d_E, (const pfa::u4 *)T.cs_x,
                               (const pfa::u4 *)T.frags_x, osc);
        } else {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr_x<false>, 64 * kCorrWavesX, n_cu);
            hipLaunchKernelGGL(k_corr_x<false>, dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * kCorrWavesX),
                               0, s, L.reqs, L.hdr, L.pre, (const pfa::u4 *)d_G, d_E, (const pfa::u4 *)T.cs_x,
                               (const pfa::u4 *)T.frags_x, osc);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (L.total[kStCorr] > 0 && h) {
        const float osc = ldexpf(1.f, 2 * T.cs_exp - 46);
        if (L.corr_pt == 2) {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr_h<2>, 64 * kCorrWavesH, n_cu);
            hipLaunchKernelGGL(k_corr_h<2>, dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * kCorrWavesH),
                               0, s, L.reqs, L.hdr, L.pre, d_Gh, d_E, d_Dc, (const uint4 *)T.cs_h, d_dck, (const hc2 *)T.tw_h, osc);
        } else {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr_h<4>, 64 * kCorrWavesH, n_cu);
            hipLaunchKernelGGL(k_corr_h<4>, dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * kCorrWavesH),
                               0, s, L.reqs, L.hdr, L.pre, d_Gh, d_E, d_Dc, (const uint4 *)T.cs_h, d_dck, (const hc2 *)T.tw_h, osc);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if (L.total[kStCorr] > 0) {
        if (L.corr_pt == 1 && L.corr_w == 4) {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr<1, 4, 3>, 64 * 4, n_cu);
            hipLaunchKernelGGL((k_corr<1, 4, 3>), dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * 4), 0, s,
                               L.reqs, L.hdr, L.pre, (const float4 *)d_G, (const float2 *)d_cs, T.tw_gen);
        } else if (L.corr_pt == 1 && L.corr_w == 6) {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr<1, 6, 3>, 64 * 6, n_cu);
            hipLaunchKernelGGL((k_corr<1, 6, 3>), dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * 6), 0, s,
                               L.reqs, L.hdr, L.pre, (const float4 *)d_G, (const float2 *)d_cs, T.tw_gen);
        } else if (L.corr_pt == 1) {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr<1, 12, 3>, 64 * 12, n_cu);
            hipLaunchKernelGGL((k_corr<1, 12, 3>), dim3(grid_for(L.total[kStCorr], cap, pers)), dim3(64 * 12), 0, s,
                               L.reqs, L.hdr, L.pre, (const float4 *)d_G, (const float2 *)d_cs, T.tw_gen);
        } else if (L.corr_pt == 2) {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr<2, kCorrWaves, 2>, 64 * kCorrWaves, n_cu);
            hipLaunchKernelGGL((k_corr<2, kCorrWaves, 2>), dim3(grid_for(L.total[kStCorr], cap, pers)),
                               dim3(64 * kCorrWaves), 0, s, L.reqs, L.hdr, L.pre, (const float4 *)d_G, (const float2 *)d_cs, T.tw_gen);
        } else {
            static int cap = 0;
            if (!cap) cap = occupancy(k_corr<4, kCorrWaves, 2>, 64 * kCorrWaves, n_cu);
            hipLaunchKernelGGL((k_corr<4, kCorrWaves, 2>), dim3(grid_for(L.total[kStCorr], cap, pers)),
                               dim3(64 * kCorrWaves), 0, s, L.reqs, L.hdr, L.pre, (const float4 *)d_G, (const float2 *)d_cs, T.tw_gen);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = mark(3)) != hipSuccess) return e;
    {
        static int cap = 0;
        if (!cap) cap = occupancy(k_colmax, kPeakThreads, n_cu);
        hipLaunchKernelGGL(k_colmax, dim3(grid_for(L.total[kStColmax], cap, false)), dim3(kPeakThreads), 0, s,
                           L.reqs, L.hdr, L.pre, d_Q, d_K, d_part);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_peak, dim3(grid_for(L.total[kStPeak], 4LL * n_cu, false)), dim3(kArgThreads), 0,
                           s, L.reqs, L.hdr, L.pre, d_Q, d_K, d_part);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return mark(4);
}

// ===========================================================================
// tracking correlators (the tracking channel's carrier and code NCOs, first
// mixing stage and time-domain correlation, Fig. 3): early / prompt / late
// sums per (request, channel, epoch), exact in integers.
// ===========================================================================

// One round of the wave reduce-scatter below: value i pairs with value
// i + H; the lane whose bit O is set keeps the upper one, its partner the
// lower, and each adds the one the other sends.
template <int O, int H>
__device__ __forceinline__ void rs_round(long long (&v)[24], int l)
{
    const bool up = (l & O) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const long long send = up ? v[i] : v[i + H];
        const long long keep = up ? v[i + H] : v[i];
        v[i] = keep + __shfl_xor(send, O);
    }
}

// The workgroup's sums of kTrackCG x 6 per-thread sums, with one
// pair of barriers for all of them.  Within a wave a reduce-scatter halves
// the values per lane each round (24, 12, 6, 3, padded to 4, 2, 1) while
// the lanes paired across bits 5 .. 1 add them, and the last round over bit
// 0 completes the wave's sum; the lane's bits then name its value.  The
// waves' sums meet in LDS and thread i < 24 adds them.  Returns value i's
// total in thread i (0 in the others); the sums are exact (int64), so their
// order does not matter.
constexpr int kTrackVals = kTrackCG * 6;
static_assert(kTrackVals == 24, "the reduce-scatter rounds are laid out for 24 values");
__device__ __forceinline__ long long block_sums64(const int (&acc)[kTrackCG][6], long long *s_red)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    long long v[24];
#pragma unroll
    for (int cc = 0; cc < kTrackCG; ++cc)
#pragma unroll
        for (int k = 0; k < 6; ++k) v[cc * 6 + k] = acc[cc][k];
    rs_round<32, 12>(v, l);
    rs_round<16, 6>(v, l);
    rs_round<8, 3>(v, l);
    v[3] = 0;
    rs_round<4, 2>(v, l);
    rs_round<2, 1>(v, l);
    const long long sum = v[0] + __shfl_xor(v[0], 1);
    const int j = ((l & 4) ? 2 : 0) + ((l & 2) ? 1 : 0);  // 3: the padding
    const int idx = ((l & 32) ? 12 : 0) + ((l & 16) ? 6 : 0) + ((l & 8) ? 3 : 0) + j;
    __syncthreads();  // the previous pass's reads of s_red are done
    if ((l & 1) == 0 && j < 3) s_red[w * kTrackVals + idx] = sum;
    __syncthreads();
    long long t = 0;
    if (threadIdx.x < kTrackVals)
        for (int i = 0; i < kTrackThreads / 64; ++i) t += s_red[i * kTrackVals + threadIdx.x];
    return t;
}

// Code replicas of a pass as +-1 bytes with one chip of wrap-around on each
// side: s_sign[c][i] = 1 - 2 code[(i - 1) mod 1023], i in [0, 1024], so the
// early (chip in [0, 1023]) and late (chip in [-1, 1022]) lookups need no wrap.
constexpr int kSignRow = 1028;

// A code phase of less than two periods, brought below one period: the period
// has a zero low word, so only the chip number takes part, and of hi and hi -
// 1023 (mod 2^32) the smaller one is right.
__device__ __forceinline__ unsigned long long code_wrap(unsigned long long q)
{
    const uint32_t hi = (uint32_t)(q >> 32);
    return ((unsigned long long)min(hi, hi - (uint32_t)kCodeLen) << 32) | (uint32_t)q;
}

// Correlates the workgroup's epoch with kTrackCG channels, FMT-specialised so
// that the sample decode leaves the loop; returns value i's sum in thread i <
// kTrackVals.  p is the byte of the epoch's first sample (the same pointer in
// every thread), off the thread's offset from it.  qe, ql: early and late
// offsets, one chip more (the sign rows start at chip -1).  Mixing is two dot
// products per channel (mix_add); |y| < 2^20, so the 24-bit multiply-adds by
// the +-1 chips are exact and int32 holds the sums of 1024 samples; longer
// epochs are summed over the workgroup in parts.
template <int FMT>
__device__ __forceinline__ long long track_pass(const GNSS_GLOBAL uint8_t *p, uint32_t off, int epoch_len,
                                                const uint2 *s_lut, const int8_t (*s_sign)[kSignRow],
                                                long long *s_red, uint32_t (&ph)[kTrackCG],
                                                const uint32_t (&dph)[kTrackCG], unsigned long long (&q)[kTrackCG],
                                                const unsigned long long (&dq)[kTrackCG],
                                                const unsigned long long (&qe)[kTrackCG],
                                                const unsigned long long (&ql)[kTrackCG])
{
    constexpr int kStep = FMT == GNSS_CPLX_I8 ? 2 * kTrackThreads
                          : FMT == GNSS_REAL_I8 ? kTrackThreads
                                                : kTrackThreads / 4;  // bytes of 256 samples
    const int n_full = epoch_len / kTrackThreads;  // samples of every thread; one more below the remainder
    int acc[kTrackCG][6];
    auto sample = [&](s2v x) {
#pragma unroll
        for (int cc = 0; cc < kTrackCG; ++cc) {
            // mix_add onto 0.  |y| is far from saturating; with the clamp bit the
            // instruction is the three-operand one, which takes the 0 as a constant
            // (the other form adds in place and needs its accumulators cleared).  From
            // the builtin, so that the compiler sees a dot product: its result must not
            // be read by another kind of vector instruction within three wait states.
            const uint2 e = s_lut[ph[cc] >> 22];
            int yr = __builtin_amdgcn_sdot2(x, __builtin_bit_cast(s2v, e.x), 0, true);
            int yi = __builtin_amdgcn_sdot2(x, __builtin_bit_cast(s2v, e.y), 0, true);
            // keeps the compiler from distributing the +-1 factors below into the products
            asm("" : "+v"(yr), "+v"(yi));
            const int8_t *row = s_sign[cc];
            const int se = row[(uint32_t)((q[cc] + qe[cc]) >> 32)], sp = row[(uint32_t)(q[cc] >> 32) + 1];
            const int sl = row[(uint32_t)((q[cc] + ql[cc]) >> 32)];
            acc[cc][0] += __mul24(se, yr);
            acc[cc][1] += __mul24(se, yi);
            acc[cc][2] += __mul24(sp, yr);
            acc[cc][3] += __mul24(sp, yi);
            acc[cc][4] += __mul24(sl, yr);
            acc[cc][5] += __mul24(sl, yi);
            ph[cc] += dph[cc];
            q[cc] = code_wrap(q[cc] + dq[cc]);
        }
    };
    long long total = 0;
    int j = 0;
    do {
#pragma unroll
        for (int cc = 0; cc < kTrackCG; ++cc)
#pragma unroll
            for (int k = 0; k < 6; ++k) acc[cc][k] = 0;
        const int j1 = min(n_full, j + 1023);
        for (; j < j1; ++j) sample(load_mix<FMT>(p + (long long)j * kStep, off));  // packed: off counts samples
        if (j == n_full && (int)threadIdx.x < epoch_len - n_full * kTrackThreads)
            sample(load_mix<FMT>(p + (long long)j * kStep, off));
        total += block_sums64(acc, s_red);
    } while (j < n_full);
    return total;
}

// One workgroup per (request, epoch, group of kTrackCG channels); the groups of
// an epoch are neighbours on one XCD, whose L2 holds the epoch's samples.
// Thread t handles samples t, t + 256, ... of the epoch with the NCO words
// advanced by 256 steps between them; the code phase is kept in [0, 1023 *
// 2^32), which leaves every chip index mod 1023 unchanged.  Bound: integer
// vector issue, 67 instructions per sample and four channels (133 with byte
// extraction and products, 64-bit compares and borrows), at five waves per SIMD
// (96 VGPRs; 144 and three when int64 totals were held beside the int32 sums).
// 32 records x 12 channels x 100 epochs of 1 ms at 16.368 MHz: 0.60 -> 0.36 ms
// (1.05 -> 1.75 10^12 sample-channels/s); one record x 10 channels x 20 epochs
// at 4.092 MHz: 35 -> 12 us, its three groups side by side instead of one after
// another.
__global__ __launch_bounds__(kTrackThreads) void k_track(const TrackDesc *__restrict__ R, const long long *pre,
                                                         int n_req, long long total, const TrackCh *__restrict__ CH,
                                                         const uint8_t *codes, const uint32_t *lut)
{
    __shared__ uint2 s_lut[1024];
    __shared__ int8_t s_sign[kTrackCG][kSignRow];
    __shared__ long long s_red[kTrackThreads / 64 * kTrackVals];
    const int tid = threadIdx.x;
    stage_mix_lut(s_lut, lut, tid, kTrackThreads);
    for (long long it = xcd_remap(blockIdx.x, gridDim.x); it < total; it += gridDim.x) {
        const int r = find_req(pre, n_req, it);
        const TrackDesc &d = R[r];
        const int groups = (d.n_ch + kTrackCG - 1) / kTrackCG;
        const long long local = it - first_item(pre, n_req, r);
        const int e = (int)(local / groups), c0 = (int)(local - (long long)e * groups) * kTrackCG;
        const long long n_e = d.start + (long long)e * d.epoch_len;  // the epoch's first sample
        __syncthreads();  // table staged; previous item done with s_sign and s_red
#pragma unroll
        for (int cc = 0; cc < kTrackCG; ++cc) {
            const uint8_t *code = codes + CH[d.ch_off + min(c0 + cc, d.n_ch - 1)].prn * kCodeLen;
            for (int k = tid; k < kCodeLen + 2; k += kTrackThreads) {
                const int chip = k == 0 ? kCodeLen - 1 : (k == kCodeLen + 1 ? 0 : k - 1);
                s_sign[cc][k] = (int8_t)(1 - 2 * (int)(code[chip] & 1u));
            }
        }
        uint32_t ph[kTrackCG], dph[kTrackCG];
        unsigned long long q[kTrackCG], dq[kTrackCG], qe[kTrackCG], ql[kTrackCG];
#pragma unroll
        for (int cc = 0; cc < kTrackCG; ++cc) {
            const TrackCh c = CH[d.ch_off + min(c0 + cc, d.n_ch - 1)];
            ph[cc] = c.phi0 + (uint32_t)((unsigned long long)(n_e + tid) * c.D);
            dph[cc] = (uint32_t)kTrackThreads * c.D;
            // q0 + n R < 2^62; 256 R is at most one period, so a thread's offset t R is
            // below one and the step 256 R needs one wrap
            const unsigned long long q0 = (unsigned long long)(c.q0 + n_e * c.R);
            const unsigned long long q1 = ((unsigned long long)((uint32_t)(q0 >> 32) % (uint32_t)kCodeLen) << 32) | (uint32_t)q0;
            q[cc] = code_wrap(q1 + (unsigned long long)(tid * c.R));
            dq[cc] = code_wrap((unsigned long long)(kTrackThreads * c.R));
            qe[cc] = (1ull << 32) + (unsigned long long)c.dl;
            ql[cc] = (1ull << 32) - (unsigned long long)c.dl;
            // not seen as each other's negatives (two additions, not an addition and a
            // subtraction with its borrow)
            asm volatile("" : "+s"(ql[cc]));
        }
        __syncthreads();
        const GNSS_GLOBAL uint8_t *p = (const GNSS_GLOBAL uint8_t *)d.samples;
        long long v;
        if (d.fmt == GNSS_CPLX_I8)
            v = track_pass<GNSS_CPLX_I8>(p + 2 * n_e, 2u * (uint32_t)tid, d.epoch_len, s_lut, s_sign, s_red, ph, dph, q,
                                         dq, qe, ql);
        else if (d.fmt == GNSS_REAL_I8)
            v = track_pass<GNSS_REAL_I8>(p + n_e, (uint32_t)tid, d.epoch_len, s_lut, s_sign, s_red, ph, dph, q, dq, qe,
                                         ql);
        else
            v = track_pass<GNSS_REAL_2BIT_PACKED>(p + (n_e >> 2), (uint32_t)(n_e & 3) + (uint32_t)tid, d.epoch_len,
                                                  s_lut, s_sign, s_red, ph, dph, q, dq, qe, ql);
        if (tid < kTrackVals) {
            const int cc = tid / 6, k = tid - cc * 6;
            if (c0 + cc < d.n_ch) gmem(d.out)[((long long)(c0 + cc) * d.n_epochs + e) * 6 + k] = v;
        }
    }
}

hipError_t launch_track(const TrackDesc *d_reqs, const long long *d_pre, int n_req, long long total,
                        const TrackCh *d_ch, const uint8_t *d_codes, const uint32_t *d_lut, hipStream_t s)
{
    const long long g = total < 0x7fffffffLL ? total : 0x7fffffffLL;
    hipLaunchKernelGGL(k_track, dim3((unsigned)(g > 0 ? g : 1)), dim3(kTrackThreads), 0, s, d_reqs, d_pre, n_req,
                       total, d_ch, d_codes, d_lut);
    return hipGetLastError();
}

size_t peak_scratch_part_elems(const Plan &p)
{
    return (size_t)p.n_prn * ((p.N + kPeakThreads - 1) / kPeakThreads);
}

// ===========================================================================
// test entry: batched natural-order 2048-point FFT / IFFT
// ===========================================================================
__global__ __launch_bounds__(256) void k_fft_test(const float2 *in, float2 *out, int batch,
                                                  int inverse, const float2 *tw)
{
    __shared__ float2 s_tw[kTwElems];
    __shared__ float2 s_xb[4][kXbufElems];
    stage_twiddles(s_tw, tw, threadIdx.x, 256);
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const long long vec = (long long)blockIdx.x * 4 + w;
    if (vec >= batch) return;
    const float2 *src = in + vec * 2048;
    float2 *dst = out + vec * 2048;
    float2 v[32];
    if (!inverse) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k2b = 0; k2b < 8; ++k2b) v[8 * u + k2b] = src[l + 64 * u + 256 * k2b];
        fft2048<false>(v, s_xb[w], s_tw, s_tw + kT1Elems, l);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int n1 = 0; n1 < 16; ++n1) dst[128 * n1 + l + 64 * h] = v[16 * h + n1];
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int n1 = 0; n1 < 16; ++n1) v[16 * h + n1] = src[128 * n1 + l + 64 * h];
        ifft2048<false>(v, s_xb[w], s_tw, s_tw + kT1Elems, l);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k2b = 0; k2b < 8; ++k2b) dst[l + 64 * u + 256 * k2b] = v[8 * u + k2b];
    }
}

hipError_t launch_fft_test(const float2 *d_in, float2 *d_out, int batch, int inverse,
                           const float2 *d_tw, hipStream_t s)
{
    hipLaunchKernelGGL(k_fft_test, dim3((batch + 3) / 4), dim3(256), 0, s, d_in, d_out, batch,
                       inverse, d_tw);
    return hipGetLastError();
}


// ===========================================================================
// test entry: batched natural-order 1023-point DFT / unnormalised inverse in
// the exact-length mode's arithmetic (per-vector exponent from the l1 norm,
// FP16 operands, FP32 accumulation); one wave per vector
// ===========================================================================
__global__ __launch_bounds__(256) void k_dft1023_test(const float2 *in, float2 *out, int batch, int inverse,
                                                      const pfa::u4 *__restrict__ fr)
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
    const long long vec = (long long)blockIdx.x * 4 + w;
    if (vec >= batch) return;
    const float2 *src = in + vec * kCodeLen;
    float *dst = (float *)(out + vec * kCodeLen);
    float nrm = 0.f;
    for (int i = l; i < kCodeLen; i += 64) nrm += fabsf(src[i].x) + fabsf(src[i].y);
    const int e = l1_exponent(wave_sum(nrm));
    const float f = ldexpf(1.f, -e), fo = ldexpf(1.f, e);
    pfa::u4 a1[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float re[4], im[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i1 = 16 * s + 4 * g + j, i2 = 16 * t + c;
                float2 v = make_float2(0.f, 0.f);
                if (i1 < pfa::kN1 && i2 < pfa::kN2)
                    v = src[inverse ? pfa::freq_index(i1, i2) : pfa::time_index(i1, i2)];
                re[j] = v.x * f;
                im[j] = v.y * f;
            }
            a1[t][s] = pfa::u4{pfa::pack2(re[0], re[1]), pfa::pack2(re[2], re[3]), pfa::pack2(im[0], im[1]),
                               pfa::pack2(im[2], im[3])};
        }
    if (!inverse) {
        pfa::FwdB B;
        pfa::load_fwd(B, fr, l);
        pfa::f4 o[2][6];
        pfa::forward(a1, B, o);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 6; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int a = 16 * u + 4 * g + r, b = 16 * (v >> 1) + c;
                    if (a < pfa::kN1 && b < pfa::kN2) dst[2 * pfa::freq_index(a, b) + (v & 1)] = o[u][v][r] * fo;
                }
    } else {
        pfa::InvB B;
        pfa::load_inv(B, fr, l);
        pfa::f4 o[2][5];
        pfa::inverse(a1, B, o);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 5; ++v)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int n1 = 16 * u + 4 * g + r;
                    const int n2 = v < 4 ? 16 * (v >> 1) + c : (c < 2 ? 32 : pfa::kN2);
                    const int part = v < 4 ? (v & 1) : c;
                    if (n1 < pfa::kN1 && n2 < pfa::kN2) dst[2 * pfa::time_index(n1, n2) + part] = o[u][v][r] * fo;
                }
    }
}

hipError_t launch_dft1023_test(const float2 *d_in, float2 *d_out, int batch, int inverse, const void *d_frags,
                               hipStream_t s)
{
    hipLaunchKernelGGL(k_dft1023_test, dim3((batch + 3) / 4), dim3(256), 0, s, d_in, d_out, batch, inverse,
                       (const pfa::u4 *)d_frags);
    return hipGetLastError();
}

}  // namespace gnss
