// Device-facing part of libwpk: helper kernels (weight re-pack, direct reference kernel, fills,
// comparison), kernel-family dispatch, the one-shot entry points, the on-device tuner and plans.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "wpk_split.h"

namespace wpk {

#define WPK_HIP(call)                                  \
    do {                                               \
        hipError_t e_ = (call);                        \
        if (e_ != hipSuccess) {                        \
            set_last_hip_error((int)e_);               \
            return WPK_E_HIP;                          \
        }                                              \
    } while (0)

// ---- dispatch table, same order as kVariants ------------------------------------------------------
typedef hipError_t (*LaunchFn)(const IgemmArgs &, hipStream_t);
#define WPK_VARIANT(PART, BM, BN, BK, WM, WN, PD) \
    extern template hipError_t launch_igemm<BM, BN, BK, WM, WN, PD>(const IgemmArgs &, hipStream_t);
#include WPK_VARIANTS_FILE
#undef WPK_VARIANT
#define WPK_VARIANT(PART, BM, BN, BK, WM, WN, PD) &launch_igemm<BM, BN, BK, WM, WN, PD>,
static const LaunchFn kLaunch[] = {
#include WPK_VARIANTS_FILE
};
#undef WPK_VARIANT
hipError_t launch_strip(const IgemmArgs &, const StripShape &, hipStream_t);  // wpk_strip.h

// ---- helper kernels ---------------------------------------------------------------------------------
// w[K][CRS] -> wp[CRSpad/4][Kpad][4] (element (kk, k) at ((kk/4)*Kpad + k)*4 + kk%4), zero padded,
// through a 32x32 LDS tile so both sides coalesce.
// With RS > 0 the packed reduction index runs (r, s, c) instead of the source's (c, r, s): the
// order the channels-last gather walks.
__global__ void __launch_bounds__(256) pack_weights_kernel(const float *__restrict__ w,
                                                           float *__restrict__ wp, int K, int CRS,
                                                           int Kpad, int C, int RS)
{
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int kk0 = blockIdx.x * 32, k0 = blockIdx.y * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int k = k0 + ty + i * 8, kk = kk0 + tx;
        int src = RS > 0 ? (kk % C) * RS + kk / C : kk;
        tile[ty + i * 8][tx] = (k < K && kk < CRS) ? w[(size_t)k * CRS + src] : 0.0f;
    }
    __syncthreads();
    // a thread writes one quad: channel k0 + (t % 32), k quad kk0/4 + t/32
    const int kq = threadIdx.x >> 5, kc = threadIdx.x & 31;
    float4 v = make_float4(tile[kc][4 * kq], tile[kc][4 * kq + 1], tile[kc][4 * kq + 2], tile[kc][4 * kq + 3]);
    *reinterpret_cast<float4 *>(wp + ((size_t)(kk0 / 4 + kq) * Kpad + k0 + kc) * 4) = v;
}

// Where row kk of the split members' reduction comes from: its place among the C*R*S rows of the source, or
// -1 for a padding row.  Of layers that fit STRIPS the first `strips` rows run (c, r, s) with s padded to eight and the others in the source's
// order; of others all rows with RS > 0 (c / 32, r, s, c % 32), else in the source's order.
template <bool STRIPS>
__device__ inline int split_source_row(int kk, int C, int CRS, int RS, int strips, int S)
{
    if (STRIPS) {
        if (kk >= strips) return kk - strips < CRS ? kk - strips : -1;
        const int row = (kk >> 3) * S + (kk & 7);
        return (kk & 7) < S && row < CRS ? row : -1;
    }
    if (RS == 0) return kk < CRS ? kk : -1;
    const int c32 = kk / (32 * RS), t = kk - c32 * 32 * RS, c = c32 * 32 + (t & 31);
    // (sixteen rows at a time: the two halves of the 32 channels follow each other for every tap)
    return c < C ? c * RS + (t >> 5) : -1;
}

// w[K][CRS] -> [depths of 16 rows][Kpad/32][3 parts][64 lanes][8 bf16], zero padded: what lane l of a wave feeds the
// bf16 MFMA of one depth and 32-channel block is channel l % 32, rows (l / 32)*8 .. +7.  Parts: see split_weight.
// (STRIPS by template: looking for strips' rows in every layer cost one-shot calls 1 %, 352 to 32 channels, 1x3, 18x18, 31 images, 19.1 us, 19.3.)
template <bool STRIPS>
__global__ void __launch_bounds__(256) pack_split_kernel(const float *__restrict__ w, v4u *__restrict__ wp, int K,
                                                         int C, int CRS, int depths, int blocks, int RS, int strips, int S)
{
    const int lane = threadIdx.x & 63, t = blockIdx.x * 4 + (threadIdx.x >> 6), kb = blockIdx.y;
    if (t >= depths) return;
    const int k = kb * 32 + (lane & 31);
    unsigned part[3][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = split_source_row<STRIPS>(t * 16 + (lane >> 5) * 8 + j, C, CRS, RS, strips, S);
        const float v = k < K && row >= 0 ? w[(size_t)k * CRS + row] : 0.0f;
        unsigned v3[3];
        split_weight(v, v3);
#pragma unroll
        for (int q = 0; q < 3; ++q) part[q][j / 2] = j % 2 ? part[q][j / 2] | v3[q] << 16 : v3[q];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
        wp[(((size_t)t * blocks + kb) * 3 + q) * 64 + lane] = (v4u){part[q][0], part[q][1], part[q][2], part[q][3]};
}

// The same for large weights: a block takes eight c of 32 k (`octets` times), whose values lie together in w, and fetches them
// into LDS as they lie.  Above, a line of w is fetched again for every tap (512 x 512 x 3x3: 14.0 us, here 6.5; 1024 x 1024 x 3x3: 48.0 and
// 20.6; 1536 x 1024: 6.4 and 4.7; 256 x 256: 3.4 and 3.0).  With few blocks of many taps each the order turns (96 x 96 x 7x7, 48 blocks:
// 4.0 and 8.1).  Rows in the source's order are CRS c of one tap.
__global__ void __launch_bounds__(256) pack_split_staged_kernel(const float *__restrict__ w, v4u *__restrict__ wp, int K,
                                                                int C, int RS, int blocks, int octets, int all_octets)
{
    extern __shared__ float rows[];  // [32 k][8 * RS * octets + 1]
    const int o0 = blockIdx.x * octets, kb = blockIdx.y, CRS = C * RS;
    const int span = min(octets, all_octets - o0) * 8 * RS, pitch = octets * 8 * RS + 1;
    for (int i = threadIdx.x & 31; i < span; i += 32) {
        const int at = o0 * 8 * RS + i;
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = kb * 32 + j * 8 + (threadIdx.x >> 5);
            v[j] = k < K && at < CRS ? w[(size_t)k * CRS + at] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) rows[(j * 8 + (threadIdx.x >> 5)) * pitch + i] = v[j];
    }
    __syncthreads();
    const int k = threadIdx.x & 31;
    for (int u = threadIdx.x >> 5; u < span / 8; u += 8) {  // a tap of an octet
        const int o = u / RS, rs = u - o * RS;
        unsigned part[3][4];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            unsigned v3[3];
            split_weight(rows[k * pitch + (o * 8 + j) * RS + rs], v3);
#pragma unroll
            for (int q = 0; q < 3; ++q) part[q][j / 2] = j % 2 ? part[q][j / 2] | v3[q] << 16 : v3[q];
        }
        const int oc = o0 + o, t = (oc >> 2) * 2 * RS + rs * 2 + (oc >> 1 & 1);
#pragma unroll
        for (int q = 0; q < 3; ++q)
            wp[(((size_t)t * blocks + kb) * 3 + q) * 64 + (oc & 1) * 32 + k] =
                (v4u){part[q][0], part[q][1], part[q][2], part[q][3]};
    }
}

// The way back, from either packed form, exactly: w[K][CRS] (a plan whose configuration moves to the other form).
__global__ void __launch_bounds__(256) unpack_weights_kernel(const void *__restrict__ packed, float *__restrict__ w,
                                                             int K, int C, int CRS, int Kpad, int RS, int split)
{
    const long long total = (long long)K * CRS;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
        const int k = (int)(i / CRS), row = (int)(i - (long long)k * CRS);
        const int c = RS > 0 ? row / RS : 0, rs = RS > 0 ? row - c * RS : 0;
        if (split) {
            const int kk = RS > 0 ? (c / 32 * RS + rs) * 32 + c % 32 : row;
            const int lane = (kk >> 3 & 1) * 32 + (k & 31);
            const unsigned short *p = (const unsigned short *)packed +
                                      (((size_t)(kk >> 4) * (Kpad / 32) + k / 32) * 3 * 64 + lane) * 8 + (kk & 7);
            w[i] = join_weight(p[0], p[512], p[2 * 512]);
        } else {
            const int kk = RS > 0 ? rs * C + c : row;
            w[i] = ((const float *)packed)[((size_t)(kk / 4) * Kpad + k) * 4 + kk % 4];
        }
    }
}

// One output element per lane, the three reduction loops written out; 64-bit indexing.
__global__ void __launch_bounds__(256) direct_conv_kernel(const float *__restrict__ x,
                                                          const float *__restrict__ w,
                                                          float *__restrict__ y,
                                                          float *__restrict__ dnorm,
                                                          wpk_conv_desc d, int P, int Q, long long total)
{
    const bool xl = d.layout & 1, yl = d.layout & 2;  // channels-last x / y
    for (long long o = (long long)blockIdx.x * blockDim.x + threadIdx.x; o < total;
         o += (long long)gridDim.x * blockDim.x) {
        int q, p, k;
        long long n, t = o;
        if (yl) {
            k = (int)(t % d.k); t /= d.k;
            q = (int)(t % Q); t /= Q;
            p = (int)(t % P);
            n = t / P;
        } else {
            q = (int)(t % Q); t /= Q;
            p = (int)(t % P); t /= P;
            k = (int)(t % d.k);
            n = t / d.k;
        }
        float acc = 0.0f, mag = 0.0f;
        for (int c = 0; c < d.c; ++c)
            for (int r = 0; r < d.r; ++r) {
                int ih = p * d.stride_h - d.pad_h + r * d.dil_h;
                if (ih < 0 || ih >= d.h) continue;
                for (int s = 0; s < d.s; ++s) {
                    int iw = q * d.stride_w - d.pad_w + s * d.dil_w;
                    if (iw < 0 || iw >= d.w) continue;
                    float xv = xl ? x[((n * d.h + ih) * (long long)d.w + iw) * d.c + c]
                                  : x[((n * d.c + c) * d.h + ih) * (long long)d.w + iw];
                    float wv = w[(((long long)k * d.c + c) * d.r + r) * d.s + s];
                    acc = fmaf(xv, wv, acc);
                    mag += fabsf(xv * wv);
                }
            }
        y[o] = acc;
        if (dnorm) dnorm[o] = mag;
    }
}

__global__ void fill_zero_kernel(float4 *__restrict__ p4, float *__restrict__ tail, long long n4,
                                 int ntail)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (long long j = i; j < n4; j += stride) p4[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < ntail) tail[i] = 0.0f;
}

// Zero y for all pixels m >= m_begin (every channel): the tiles a persistent launch accumulates
// into with atomics.  One lane per (channel, pixel), pixels fastest.
__global__ void zero_pixels_kernel(float *__restrict__ y, int m_begin, int M, int K, int PQ, int yl)
{
    const long long span = M - m_begin;
    if (yl) {  // channels-last: those pixels are one contiguous range
        for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < span * K;
             i += (long long)gridDim.x * blockDim.x)
            y[(long long)m_begin * K + i] = 0.0f;
        return;
    }
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < span * K;
         i += (long long)gridDim.x * blockDim.x) {
        int m = m_begin + (int)(i % span), k = (int)(i / span);
        int n = m / PQ, pq = m - n * PQ;
        y[((long long)n * K + k) * PQ + pq] = 0.0f;
    }
}

// y = act(y + bias[k] + res): the fused epilogue as a pass of its own, for the launches that
// cannot apply it while storing (atomic accumulation, the direct kernel).
__global__ void epilogue_kernel(float *__restrict__ y, const float *__restrict__ bias,
                                const float *__restrict__ res, int relu, int K, int PQ, int yl,
                                long long total)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        float v = y[i];
        if (bias) v += bias[yl ? i % K : (i / PQ) % K];
        if (res) v += res[i];
        if (relu) v = fmaxf(v, 0.0f);
        y[i] = v;
    }
}

__global__ void fill_value_kernel(float *__restrict__ p, long long n, float v)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

// Synthetic operands for the tuner: value = lo + (hi-lo) * hash(index, seed) / 2^24.
__global__ void fill_hash_kernel(float *__restrict__ p, long long n, unsigned seed, float lo, float hi)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        unsigned h = (unsigned)i * 2654435761u ^ seed;
        h ^= h >> 16; h *= 0x7feb352du; h ^= h >> 15; h *= 0x846ca68bu; h ^= h >> 16;
        p[i] = lo + (hi - lo) * (float)(h >> 8) * (1.0f / 16777216.0f);
    }
}

// max over outputs of |y - ref| / max(dnorm, tiny); NaN counts as +inf.  Result as float bits.
__global__ void compare_kernel(const float *__restrict__ y, const float *__restrict__ ref,
                               const float *__restrict__ dnorm, long long n, unsigned *out_bits)
{
    float worst = 0.0f;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        float e = fabsf(y[i] - ref[i]) / fmaxf(dnorm[i], 1e-30f);
        if (!(e == e)) e = INFINITY;
        worst = fmaxf(worst, e);
    }
    atomicMax(out_bits, __float_as_uint(worst));
}

// Zero several tensors with one launch: entry e covers blocks [first[e], first[e+1]), each block
// 1024 sixteen-byte quads of the tensor's aligned body; block 0 of an entry also clears the few
// floats before and after the body.
static const int kZeroListMax = 48;
struct ZeroList {
    float *p[kZeroListMax];
    long long n[kZeroListMax];
    int first[kZeroListMax + 1];
    int count;
};
__global__ void __launch_bounds__(256) zero_many_kernel(const ZeroList z)
{
    int e = 0;
    while (e + 1 < z.count && (int)blockIdx.x >= z.first[e + 1]) ++e;
    const int b = blockIdx.x - z.first[e];
    float *p = z.p[e];
    const long long n = z.n[e];
    long long head = (long long)(((16 - ((unsigned long long)p & 15)) & 15) / 4);
    if (head > n) head = n;
    const long long n4 = (n - head) / 4, tail = n - head - n4 * 4;
    float4 *p4 = (float4 *)(p + head);
    for (int u = 0; u < 4; ++u) {
        long long j = (long long)b * 1024 + u * 256 + threadIdx.x;
        if (j < n4) p4[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (b == 0) {
        if ((long long)threadIdx.x < head) p[threadIdx.x] = 0.0f;
        if ((long long)threadIdx.x < tail) p[head + n4 * 4 + threadIdx.x] = 0.0f;
    }
}

// ---- calibration kernels (measured ceilings reported beside the published ones) ----------------------
// Nothing but fp32 MFMAs: four independent accumulators per wave, so an MFMA never waits for the one
// before it, and sixteen operand pairs of hashed values in [0,1) x [-0.5,0.5) (operands that never
// change make the figure unrepresentative: at four waves per SIMD they measure 20 % low here).
__device__ inline float unit_hash(unsigned x)
{
    x ^= x >> 16;
    x *= 0x7feb352dU;
    x ^= x >> 15;
    x *= 0x846ca68bU;
    x ^= x >> 16;
    return (float)(x >> 8) * (1.0f / 16777216.0f);
}

__global__ void __launch_bounds__(256) mfma_only_kernel(float *out, int iters)
{
    v16f acc[4];
    for (int i = 0; i < 4; ++i)
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    float a[16], b[16];
    for (int i = 0; i < 16; ++i) {
        a[i] = unit_hash(blockIdx.x * 4096u + threadIdx.x * 16u + i);
        b[i] = unit_hash(0x9e3779b9u + threadIdx.x * 16u + i) - 0.5f;
    }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int u = 0; u < 16; ++u)
            acc[u & 3] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], b[u], acc[u & 3], 0, 0, 0);
    }
    float s = 0.f;
    for (int i = 0; i < 4; ++i)
        for (int e = 0; e < 16; ++e) s += acc[i][e];
    out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

// Streaming copy, 16 bytes per lane per trip.
__global__ void __launch_bounds__(256) copy16_kernel(const float4 *__restrict__ src, float4 *__restrict__ dst,
                                                     long long n16)
{
    const long long stride = (long long)gridDim.x * 256;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

// ---- device state -----------------------------------------------------------------------------------
static std::mutex g_mu;
static bool g_dev_ready = false;
static int g_cus = 0;

static int ensure_device()
{
    if (g_dev_ready) return WPK_OK;
    int dev = 0;
    WPK_HIP(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    WPK_HIP(hipGetDeviceProperties(&prop, dev));
    g_cus = prop.multiProcessorCount;
    // architecture string and compute-unit count: the marketing name is not stable across tools
    std::string name = std::string(prop.gcnArchName) + ":cu" + std::to_string(g_cus);
    std::replace(name.begin(), name.end(), ' ', '_');
    set_device_name(name);
    g_dev_ready = true;
    return WPK_OK;
}

// Tap tables of a problem, two ints per row: {byte offset, mask bit of filter row r | mask bit of
// filter column s (16 + s) << 8}.
//  - Periodic table [R*S phases][32 rows]: row j of phase ph describes reduction row ph + j of a
//    step that starts at tap ph of some channel c0: tap (ph + j) % RS of channel c0 + (ph + j) / RS.
//    Offset = (channel advance*H*W + (r*dil_h - pad_h)*W + s*dil_w - pad_w)*4 + bias, where
//    bias = (pad_h*W + pad_w)*4 keeps it non-negative; the kernel adds c0*H*W*4.
//  - Three tail tables [32 rows], for K-steps of 8, 16 and 32: the rows from the start of the last
//    step of the reduction, with absolute offsets; rows past C*R*S point at the always-set bit 31.
// Layout: periodic | tail(8) | tail(16) | tail(32).
// Tap-major forms (quad != 0: channels-last in channel quads, or [N][C][H][W] with C a multiple of
// every K-step): one entry per filter tap instead, {byte offset of the tap (biased like the
// descriptor base), mask bits}, padded with zero entries to 32.
// The tables are written on the device (one lane per entry) so that preparing a descriptor is a
// launch on the caller's stream and nothing else: no host-to-device copy, no synchronisation.
struct TapGeom {
    int32_t R, S, W, C, CRS;
    int32_t pad_h, pad_w, dil_h, dil_w;
    int32_t cs, ps;   // element strides of x between channels / between pixels of a row
    int32_t quad;
    int32_t entries;
};
static TapGeom tap_geometry(const Problem &pr)
{
    const wpk_conv_desc &d = pr.d;
    TapGeom g;
    g.R = d.r; g.S = d.s; g.W = d.w; g.C = d.c; g.CRS = pr.CRS;
    g.pad_h = d.pad_h; g.pad_w = d.pad_w; g.dil_h = d.dil_h; g.dil_w = d.dil_w;
    g.cs = pr.xl ? 1 : d.h * d.w;
    g.ps = pr.xl ? d.c : 1;
    g.quad = pr.xquad || pr.tapmajor ? 1 : 0;
    const int RS = d.r * d.s;
    g.entries = g.quad ? std::max(RS, 32) : (RS + 3) * 32;
    return g;
}
static size_t tap_table_bytes(const Problem &pr) { return (size_t)tap_geometry(pr).entries * 2 * sizeof(int32_t); }

__global__ void __launch_bounds__(256) tap_table_kernel(int32_t *__restrict__ t, const TapGeom g)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= g.entries) return;
    const int RS = g.R * g.S;
    int off = 0, bits = 0;
    if (g.quad) {
        if (e < RS) {
            const int r = e / g.S, s = e - r * g.S;
            // ((r*dil_h - pad_h)*W + s*dil_w - pad_w)*ps*4 plus the bias (pad_h*W + pad_w)*ps*4
            off = (r * g.dil_h * g.W + s * g.dil_w) * g.ps * 4;
            bits = r | (16 + s) << 8;
        }
    } else {
        const int table = e >> 5, j = e & 31;
        int kk;          // reduction row relative to the step's channel base, or absolute (tails)
        bool pad = false;
        if (table < RS) {
            kk = table + j;
        } else {
            const int bk = 8 << (table - RS);
            kk = (g.CRS + bk - 1) / bk * bk - bk + j;
            pad = kk >= g.CRS;
        }
        if (pad) {
            bits = kPadTapBit | kPadTapBit << 8;
        } else {
            const int c = kk / RS, rs = kk - c * RS, r = rs / g.S, s = rs - r * g.S;
            // (c*cs + ((r*dil_h - pad_h)*W + s*dil_w - pad_w)*ps)*4 plus the bias (pad_h*W + pad_w)*ps*4
            off = (c * g.cs + (r * g.dil_h * g.W + s * g.dil_w) * g.ps) * 4;
            bits = r | (16 + s) << 8;
        }
    }
    t[2 * e] = off;
    t[2 * e + 1] = bits;
}

static int write_tap_table(const Problem &pr, int32_t *dptr, hipStream_t st)
{
    const TapGeom g = tap_geometry(pr);
    hipLaunchKernelGGL(tap_table_kernel, dim3((g.entries + 255) / 256), dim3(256), 0, st, dptr, g);
    WPK_HIP(hipGetLastError());
    return WPK_OK;
}

// A table in memory of its own, ready when `st` reaches this point.
static int upload_tap_table(const Problem &pr, int32_t **out, hipStream_t st)
{
    int32_t *dptr = nullptr;
    WPK_HIP(hipMalloc((void **)&dptr, tap_table_bytes(pr)));
    int rc = write_tap_table(pr, dptr, st);
    if (rc != WPK_OK) {
        (void)hipFree(dptr);
        return rc;
    }
    *out = dptr;
    return WPK_OK;
}

// Bytes of a problem's weights in the form the tiled and wave-split members (split = false) or the split members
// read them.
static size_t packed_bytes(const Problem &pr, bool split)
{
    return split ? (size_t)split_rows(pr) * pr.Kpad * kSplitWeightBytes : (size_t)pr.CRSpad * pr.Kpad * sizeof(float);
}

// Of these, the bytes in the strips' order that lie ahead of the others.
static size_t strip_bytes(const Problem &pr) { return (size_t)strip_depths(pr) * 16 * pr.Kpad * kSplitWeightBytes; }

// The order of the packed rows (but for strips), as split_source_row and pack_weights_kernel have it.
static int packed_order(const Problem &pr, bool split)
{
    return (split ? split_taps(pr) : pr.xquad || pr.tapmajor) ? pr.d.r * pr.d.s : 0;
}

static int pack_weights(const Problem &pr, bool split, const float *w, float *wp, hipStream_t st)
{
    const int RS = packed_order(pr, split);
    if (split) {
        const int blocks = pr.Kpad / 32, taps = RS > 0 ? RS : 1, strips = strip_depths(pr) * 16;
        const int all_octets = (int)(split_rows(pr) / taps / 8), octets = std::max(1, 8 / taps);
        const int chunks = (all_octets + octets - 1) / octets;
        // a block per compute unit, or a single tap (see there); at most 64 KB of LDS
        if (strips == 0 && (taps == 1 || (int64_t)chunks * blocks >= 256) && taps < 64) {
            hipLaunchKernelGGL(pack_split_staged_kernel, dim3(chunks, blocks), dim3(256),
                               32 * (octets * 8 * taps + 1) * sizeof(float), st, w, (v4u *)wp, pr.d.k,
                               RS > 0 ? pr.d.c : pr.CRS, taps, blocks, octets, all_octets);
        } else {
            const int depths = (int)(split_rows(pr) / 16);
            hipLaunchKernelGGL(strips ? pack_split_kernel<true> : pack_split_kernel<false>, dim3((depths + 3) / 4, blocks),
                               dim3(256), 0, st, w, (v4u *)wp, pr.d.k, pr.d.c, pr.CRS, depths, blocks, RS, strips, pr.d.s);
        }
    } else {
        dim3 grid(pr.CRSpad / 32, pr.Kpad / 32);
        hipLaunchKernelGGL(pack_weights_kernel, grid, dim3(256), 0, st, w, wp, pr.d.k, pr.CRS, pr.Kpad, pr.d.c, RS);
    }
    WPK_HIP(hipGetLastError());
    return WPK_OK;
}

static int zero_fill(float *p, int64_t n, hipStream_t st)
{
    // y comes from the caller with 4-byte alignment only: peel to a 16-byte boundary
    uintptr_t addr = (uintptr_t)p;
    int head = (int)(((16 - (addr & 15)) & 15) / 4);
    if (head > n) head = (int)n;
    int64_t n4 = (n - head) / 4;
    int tail = (int)(n - head - n4 * 4);
    if (head) {
        hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(64), 0, st, (float4 *)nullptr, p, 0LL, head);
        WPK_HIP(hipGetLastError());
    }
    int blocks = (int)std::min<int64_t>(2048, std::max<int64_t>(1, (n4 + 255) / 256));
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, st, (float4 *)(p + head),
                       p + head + n4 * 4, (long long)n4, tail);
    WPK_HIP(hipGetLastError());
    return WPK_OK;
}

static int run_ref(const Problem &pr, const float *x, const float *w, float *y, float *dnorm,
                   hipStream_t st)
{
    int blocks = (int)std::min<int64_t>(1 << 20, (pr.y_elems + 255) / 256);
    hipLaunchKernelGGL(direct_conv_kernel, dim3(blocks), dim3(256), 0, st, x, w, y, dnorm, pr.d, pr.P,
                       pr.Q, (long long)pr.y_elems);
    WPK_HIP(hipGetLastError());
    return WPK_OK;
}

static int run_epilogue(const Problem &pr, const Epilogue &epi, float *y, hipStream_t st)
{
    if (!epi.any()) return WPK_OK;
    int blocks = (int)std::min<int64_t>(4096, (pr.y_elems + 255) / 256);
    hipLaunchKernelGGL(epilogue_kernel, dim3(blocks), dim3(256), 0, st, y, epi.bias, epi.res, epi.relu,
                       pr.d.k, pr.P * pr.Q, pr.yl ? 1 : 0, (long long)pr.y_elems);
    WPK_HIP(hipGetLastError());
    return WPK_OK;
}

// Device buffer for the fix-up of persistent launches: counters (kept zero between launches) in
// the first kFixupCounterBytes, partial-tile slots after them.
struct FixupBuf {
    char *ptr = nullptr;
    size_t bytes = 0;
};
static int fixup_reserve(FixupBuf &b, size_t bytes)
{
    if (bytes <= b.bytes) return WPK_OK;
    if (b.ptr) WPK_HIP(hipFree(b.ptr));  // synchronises: earlier users are done
    b.ptr = nullptr;
    b.bytes = 0;
    WPK_HIP(hipMalloc((void **)&b.ptr, bytes));
    WPK_HIP(hipMemset(b.ptr, 0, kFixupCounterBytes));
    WPK_HIP(hipDeviceSynchronize());  // filled before a launch on any stream can follow
    b.bytes = bytes;
    return WPK_OK;
}
static void fixup_release(FixupBuf &b)
{
    if (b.ptr) (void)hipFree(b.ptr);
    b.ptr = nullptr;
    b.bytes = 0;
}

// Launch one member of the tiled family.  cfg must be legal for pr (checked by the callers).
// `fix` is the fix-up workspace of a persistent launch, large enough for fixup_need(); with a
// NULL workspace shared tiles are accumulated with atomics into zeroed outputs.
// Whether a launch of cfg accumulates into all of y with atomics, so that all of y has to be
// zeroed first (no workspace that covers it, and a split reduction or a persistent launch without
// a whole round).
static bool zeroes_all_of_y(const Problem &pr, const wpk_conv_config &cfg, const FixupBuf *fix)
{
    FixupNeed need = fixup_need(pr, cfg, g_cus);
    if (need.bytes > 0 && fix && fix->ptr && fix->bytes >= (size_t)need.bytes) return false;
    int nsteps = reduction_of(pr, cfg).steps;
    int per = (nsteps + cfg.split_k - 1) / cfg.split_k;
    if ((nsteps + per - 1) / per > 1) return true;
    if (const int persist = persistent_of(pr, cfg, g_cus)) {
        int64_t tiles = ((pr.M + cfg.bm - 1) / cfg.bm) * ((pr.d.k + cfg.bn - 1) / cfg.bn);
        int64_t G = (int64_t)persist * (g_cus > 0 ? g_cus : 256);
        return tiles < G;
    }
    return false;
}

// (y_zeroed: the caller has already zeroed all of y on this stream)
static int run_config(const Problem &pr, const wpk_conv_config &cfg, const int32_t *ktab,
                      const float *x, const float *wp, float *y, const FixupBuf *fix, hipStream_t st,
                      const Epilogue &epi = Epilogue(), bool y_zeroed = false)
{
    int vi = find_variant(cfg.bm, cfg.bn, cfg.bk, cfg.wm, cfg.wn, cfg.stages);
    if (vi < 0) return WPK_E_NO_CONFIG;
    const wpk_conv_desc &d = pr.d;
    IgemmArgs a;
    const bool strip = runs_strip(pr, cfg);
    const size_t ahead = split_member(cfg) && !strip ? strip_bytes(pr) : 0;  // (weights of the other order)
    a.x = x; a.wp = (const float *)((const char *)wp + ahead); a.y = y; a.ktab = ktab;
    a.RS = d.r * d.s;
    a.HW4 = pr.xl ? 4 : d.h * d.w * 4;  // byte stride between channels of x
    const Reduction red = reduction_of(pr, cfg);
    const int persist = persistent_of(pr, cfg, g_cus);
    a.bk_div_rs = red.rows / a.RS;
    a.bk_mod_rs = red.rows % a.RS;
    a.ttab = ktab + ((size_t)a.RS + (red.rows == 8 ? 0 : red.rows == 16 ? 1 : 2)) * 32 * 2;
    a.N = d.n; a.C = d.c; a.H = d.h; a.W = d.w; a.K = d.k; a.Q = pr.Q; a.R = d.r; a.S = d.s;
    a.stride_h = d.stride_h; a.stride_w = d.stride_w; a.pad_h = d.pad_h; a.pad_w = d.pad_w;
    a.dil_h = d.dil_h; a.dil_w = d.dil_w;
    a.M = (int32_t)pr.M; a.PQ = pr.P * pr.Q; a.HW = d.h * d.w; a.CRS = pr.CRS; a.Kpad = pr.Kpad;
    a.nsteps = red.steps;
    a.halo = !split_member(cfg) ? 0 : strip ? -2 : split_point(pr) ? -1 : halo_positions(pr, cfg);
    a.producers = (int16_t)split_producers(pr, cfg, g_cus);
    // slices of ceil(nsteps/split_k) steps; launch only as many as are not empty
    a.steps_per_split = (a.nsteps + cfg.split_k - 1) / cfg.split_k;
    a.split_k = (a.nsteps + a.steps_per_split - 1) / a.steps_per_split;
    a.tiles_m = (int32_t)((pr.M + cfg.bm - 1) / cfg.bm);
    a.tiles_n = (d.k + cfg.bn - 1) / cfg.bn;
    a.remap = cfg.xcd_remap;
    a.x_bytes = (uint32_t)(pr.x_elems * 4);
    a.x_bias = (uint32_t)((d.pad_h * d.w + d.pad_w) * 4 * (pr.xl ? d.c : 1));
    a.xl = pr.xquad ? 2 : pr.tapmajor ? 3 : split_member(cfg) && split_taps(pr) ? (pr.xl ? 2 : 3) : pr.xl ? 1 : 0;
    a.yl = pr.yl ? 1 : 0;
    // whole channel quads with 16-byte stores when the tensors allow it
    if (pr.yl && d.k % 4 == 0 && ((uintptr_t)y & 15) == 0 && ((uintptr_t)epi.res & 15) == 0 &&
        ((uintptr_t)epi.bias & 15) == 0)
        a.yl = 2;
    a.w_bytes = (uint32_t)(strip ? strip_bytes(pr) : packed_bytes(pr, split_member(cfg)) - ahead);
    a.y_bytes = (uint32_t)(pr.y_elems * 4);
    a.persist = persist;
    a.grid_persist = persist * (g_cus > 0 ? g_cus : 256);
    a.tiles = a.tiles_m * a.tiles_n;
    a.tiles_dp = persist > 0 ? a.tiles / a.grid_persist * a.grid_persist : 0;
    a.two_per_unit = persist > 0 ? persist <= 2 : (int64_t)a.tiles * a.split_k <= 2 * (int64_t)(g_cus > 0 ? g_cus : 256);
    {
        int64_t units = (int64_t)(a.tiles - a.tiles_dp) * a.nsteps;  // < 2^31: checked by legal_for
        int64_t groups = persist > 0 ? streamk_groups(units, a.grid_persist, red.rows) : 0;
        a.sk_groups = (int32_t)groups;
        a.sk_q = groups > 0 ? (int32_t)(units / groups) : 0;
        a.sk_rem = groups > 0 ? (int32_t)(units % groups) : 0;
        a.runners = 0;  // (the launcher decides: it knows how many workgroups of the variant a compute unit holds)
    }
    a.div_pq = make_fastdiv((uint32_t)a.PQ);
    a.div_q = make_fastdiv((uint32_t)a.Q);
    a.div_tiles_n = make_fastdiv((uint32_t)a.tiles_n);
    a.div_tiles_m = make_fastdiv((uint32_t)a.tiles_m);
    a.div_s = make_fastdiv((uint32_t)d.s);
    // weights the larger operand: tiles that share them are made neighbours (see IgemmArgs::mfast)
    a.mfast = pr.w_elems > pr.x_elems ? 1 : 0;
    a.div_tiles = make_fastdiv((uint32_t)a.tiles);
    a.div_nsteps = make_fastdiv((uint32_t)a.nsteps);
    a.div_q1 = make_fastdiv((uint32_t)a.sk_q + 1);
    a.div_q0 = make_fastdiv((uint32_t)std::max(a.sk_q, 1));
    a.div_tap = make_fastdiv((uint32_t)(a.halo > 0 ? d.h * d.w
                                               : (pr.xquad || pr.tapmajor) && !split_member(cfg) ? d.c : a.RS));
    a.ws = nullptr;
    a.ws_cnt = nullptr;
    a.ws_maxc = 0;
    FixupNeed need = fixup_need(pr, cfg, g_cus);
    if (need.bytes > 0 && fix && fix->ptr && fix->bytes >= (size_t)need.bytes) {
        a.ws_cnt = (int32_t *)fix->ptr;
        a.ws = (float *)(fix->ptr + need.slots_offset);
        a.ws_maxc = (int32_t)need.maxc;
    }
    // with atomics into y nobody holds a finished output: the epilogue follows as its own pass
    const bool shared_by_atomics =
        !a.ws && (a.split_k > 1 || (persist > 0 && (a.tiles_m * a.tiles_n) % a.grid_persist != 0));
    a.bias = shared_by_atomics ? nullptr : epi.bias;
    a.res = shared_by_atomics ? nullptr : epi.res;
    a.relu = shared_by_atomics ? 0 : epi.relu;
    if (a.split_k > 1 && !a.ws) {
        int rc = y_zeroed ? WPK_OK : zero_fill(y, pr.y_elems, st);
        if (rc != WPK_OK) return rc;
    } else if (a.split_k == 1 && persist > 0 && !a.ws) {
        // tiles beyond the last whole round are accumulated with atomics: zero their pixels
        int tiles = a.tiles_m * a.tiles_n;
        int tiles_dp = tiles / a.grid_persist * a.grid_persist;
        if (tiles_dp < tiles) {
            // (tiles ordered along the pixels first: the remainder is a range of channels, not of pixels)
            int m_begin = a.mfast ? 0 : tiles_dp / a.tiles_n * cfg.bm;
            if (m_begin == 0) {
                int rc = y_zeroed ? WPK_OK : zero_fill(y, pr.y_elems, st);
                if (rc != WPK_OK) return rc;
            } else {
                long long n = (long long)(a.M - m_begin) * a.K;
                int blocks = (int)std::min<long long>(4096, (n + 255) / 256);
                hipLaunchKernelGGL(zero_pixels_kernel, dim3(blocks), dim3(256), 0, st, y, m_begin, a.M,
                                   a.K, a.PQ, a.yl);
                WPK_HIP(hipGetLastError());
            }
        }
    }
    WPK_HIP(strip ? launch_strip(a, strip_shape(pr, g_cus), st) : kLaunch[vi](a, st));
    if (shared_by_atomics) return run_epilogue(pr, epi, y, st);
    return WPK_OK;
}

// ---- per-descriptor state of the one-shot entry points -------------------------------------------
struct Prepared {
    Problem pr;
    int32_t *ktab;
};
static std::map<std::string, Prepared> g_prepared;
static FixupBuf g_fixup;
static float *g_wscratch = nullptr;
static size_t g_wscratch_bytes = 0;

static int get_prepared(const Problem &pr, Prepared **out, hipStream_t st)
{
    std::string key = desc_key(&pr.d);
    auto it = g_prepared.find(key);
    if (it == g_prepared.end()) {
        Prepared p{pr, nullptr};
        int rc = upload_tap_table(pr, &p.ktab, st);
        if (rc != WPK_OK) return rc;
        prepare_strip(&p.pr, g_cus);
        it = g_prepared.emplace(key, p).first;
    }
    *out = &it->second;
    return WPK_OK;
}

static int get_wscratch(size_t bytes, float **out)
{
    if (bytes > g_wscratch_bytes) {
        if (g_wscratch) WPK_HIP(hipFree(g_wscratch));  // synchronises: earlier users are done
        g_wscratch = nullptr;
        g_wscratch_bytes = 0;
        WPK_HIP(hipMalloc((void **)&g_wscratch, bytes));
        g_wscratch_bytes = bytes;
    }
    *out = g_wscratch;
    return WPK_OK;
}

static int check_io(const wpk_conv_desc *d, const void *x, const void *w, const void *y, Problem *pr)
{
    if (!d) return WPK_E_NULL_PTR;
    int rc = make_problem(d, pr);
    if (rc != WPK_OK) return rc;
    if (!x || !w || !y) return WPK_E_NULL_PTR;
    return WPK_OK;
}

static int fwd_with(const Problem &pr, const wpk_conv_config &cfg, const float *x, const float *w,
                    float *y, hipStream_t st, const Epilogue &epi = Epilogue())
{
    std::lock_guard<std::mutex> g(g_mu);
    int rc = ensure_device();
    if (rc != WPK_OK) return rc;
    Prepared *prep;
    rc = get_prepared(pr, &prep, st);
    if (rc != WPK_OK) return rc;
    float *wp;
    rc = get_wscratch(packed_bytes(pr, split_member(cfg)), &wp);
    if (rc != WPK_OK) return rc;
    rc = pack_weights(pr, split_member(cfg), w, wp, st);
    if (rc != WPK_OK) return rc;
    FixupNeed need = fixup_need(pr, cfg, g_cus);
    if (need.bytes > 0) {
        rc = fixup_reserve(g_fixup, (size_t)need.bytes);
        if (rc != WPK_OK) return rc;
    }
    return run_config(prep->pr, cfg, prep->ktab, x, wp, y, &g_fixup, st, epi);
}

// ---- timing protocol of the tuner ------------------------------------------------------------------
struct TuneCtx {
    Problem pr;
    wpk_tune_options opt;
    hipStream_t st;
    hipEvent_t e0, e1;
    float *x, *w, *wp[2], *y, *yref, *dref;  // wp: packed for the split members ([1]) and for the others
    unsigned *err_bits;
    int32_t *ktab;
    FixupBuf fix;
    int rejected;
    int hip_failed;
    int phase;                       // which stage of the search is evaluating (WPK_STAGE_*)
    std::map<int, double> times_us;  // config id (of same_launch) -> median microseconds
    std::map<int, int> stage_of;     // config id -> stage that first timed it
};

static int measure_us(TuneCtx &t, const wpk_conv_config &cfg, double *us_out, double *err_out)
{
    // one verification launch, compared on the device with the direct kernel's output; y is filled
    // with NaN first, so an output the candidate fails to store cannot pass on the value an earlier
    // candidate left there
    WPK_HIP(hipMemsetAsync(t.err_bits, 0, sizeof(unsigned), t.st));
    hipLaunchKernelGGL(fill_value_kernel, dim3(1024), dim3(256), 0, t.st, t.y, (long long)t.pr.y_elems,
                       __builtin_nanf(""));
    WPK_HIP(hipGetLastError());
    FixupNeed need = fixup_need(t.pr, cfg, g_cus);
    if (need.bytes > 0) {
        WPK_HIP(hipStreamSynchronize(t.st));
        int rf = fixup_reserve(t.fix, (size_t)need.bytes);
        if (rf != WPK_OK) return rf;
    }
    int rc = run_config(t.pr, cfg, t.ktab, t.x, t.wp[split_member(cfg)], t.y, &t.fix, t.st);
    if (rc != WPK_OK) return rc;
    hipLaunchKernelGGL(compare_kernel, dim3(512), dim3(256), 0, t.st, t.y, t.yref, t.dref,
                       (long long)t.pr.y_elems, t.err_bits);
    WPK_HIP(hipGetLastError());
    unsigned bits = 0;
    WPK_HIP(hipMemcpyAsync(&bits, t.err_bits, sizeof(unsigned), hipMemcpyDeviceToHost, t.st));
    WPK_HIP(hipStreamSynchronize(t.st));
    float err;
    memcpy(&err, &bits, sizeof err);
    *err_out = err;
    if (!(err <= 1e-4f)) {
        *us_out = 0.0;
        return WPK_OK;
    }
    // estimate, then timed groups sized to last at least min_group_us
    auto timed = [&](int launches, double *ms) -> int {
        WPK_HIP(hipEventRecord(t.e0, t.st));
        for (int i = 0; i < launches; ++i) {
            // (zero_ahead: y keeps accumulating from launch to launch, which costs the same time)
            Epilogue epi;
            epi.relu = t.opt.epilogue != 0;
            int r = run_config(t.pr, cfg, t.ktab, t.x, t.wp[split_member(cfg)], t.y, &t.fix, t.st, epi,
                               t.opt.zero_ahead != 0);
            if (r != WPK_OK) return r;
        }
        WPK_HIP(hipEventRecord(t.e1, t.st));
        WPK_HIP(hipEventSynchronize(t.e1));
        float f = 0;
        WPK_HIP(hipEventElapsedTime(&f, t.e0, t.e1));
        *ms = f;
        return WPK_OK;
    };
    double ms = 0;
    rc = timed(2, &ms);
    if (rc != WPK_OK) return rc;
    double est_us = std::max(ms * 1000.0 / 2, 0.5);
    int group = (int)std::min(1000.0, std::max(1.0, ceil(t.opt.min_group_us / est_us)));
    std::vector<double> samples;
    for (int r = 0; r < std::max(1, t.opt.reps); ++r) {
        rc = timed(group, &ms);
        if (rc != WPK_OK) return rc;
        samples.push_back(ms * 1000.0 / group);
    }
    std::sort(samples.begin(), samples.end());
    *us_out = samples[samples.size() / 2];
    // zero_ahead leaves the zeroing of y out of the launches; its share of the one zeroing launch
    // per pass is charged at 3 TB/s
    if (t.opt.zero_ahead && zeroes_all_of_y(t.pr, cfg, &t.fix)) *us_out += (double)t.pr.y_elems * 4.0 / 3.0e6;
    return WPK_OK;
}

static int tune_constraint(const int32_t *genes, int32_t n, void *user)
{
    TuneCtx *t = (TuneCtx *)user;
    wpk_conv_config cfg;
    if (n != WPK_N_GENES || wpk_config_from_genes(genes, &cfg) != WPK_OK) return 0;
    return legal_for(t->pr, cfg) ? 1 : 0;
}

// Step2: fitness = 1 / measured runtime; a candidate that fails verification gets 0.
// Whether the launch that cfg makes has been timed (and passed).
static bool tune_known(const TuneCtx &t, const wpk_conv_config &cfg)
{
    const wpk_conv_config c = same_launch(t.pr, cfg, g_cus);
    return t.times_us.count(wpk_config_id(&c)) != 0;
}

static double tune_fitness(const int32_t *genes, int32_t n, void *user)
{
    TuneCtx *t = (TuneCtx *)user;
    wpk_conv_config cfg;
    if (n != WPK_N_GENES || wpk_config_from_genes(genes, &cfg) != WPK_OK) return 0.0;
    cfg = same_launch(t->pr, cfg, g_cus);
    const auto known = t->times_us.find(wpk_config_id(&cfg));
    if (known != t->times_us.end()) return 1.0 / known->second;
    double us = 0, err = 0;
    int rc = measure_us(*t, cfg, &us, &err);
    if (rc != WPK_OK) {
        t->hip_failed = rc;
        return 0.0;
    }
    if (us <= 0.0) {
        t->rejected++;
        if (t->opt.verbose)
            fprintf(stderr, "[wpk tune] rejected %s split %d: normalised error %.3g\n",
                    wpk_config_kernel_name(&cfg), cfg.split_k, err);
        return 0.0;
    }
    t->times_us[wpk_config_id(&cfg)] = us;
    t->stage_of.emplace(wpk_config_id(&cfg), t->phase);
    if (t->opt.verbose >= 2)
        fprintf(stderr, "[wpk tune] %-32s split %2d remap %d persist %d reduce %d: %9.2f us\n",
                wpk_config_kernel_name(&cfg), cfg.split_k, cfg.xcd_remap, cfg.persist, cfg.reduce, us);
    return 1.0 / us;
}

static void tune_free(TuneCtx &t)
{
    if (t.x) (void)hipFree(t.x);
    if (t.w) (void)hipFree(t.w);
    for (float *p : t.wp)
        if (p) (void)hipFree(p);
    if (t.y) (void)hipFree(t.y);
    if (t.yref) (void)hipFree(t.yref);
    if (t.dref) (void)hipFree(t.dref);
    if (t.err_bits) (void)hipFree(t.err_bits);
    if (t.ktab) (void)hipFree(t.ktab);
    fixup_release(t.fix);
    if (t.e0) (void)hipEventDestroy(t.e0);
    if (t.e1) (void)hipEventDestroy(t.e1);
    if (t.st) (void)hipStreamDestroy(t.st);
}

static int tune_setup(TuneCtx &t)
{
    const Problem &pr = t.pr;
    WPK_HIP(hipStreamCreate(&t.st));
    WPK_HIP(hipEventCreate(&t.e0));
    WPK_HIP(hipEventCreate(&t.e1));
    WPK_HIP(hipMalloc((void **)&t.x, pr.x_elems * 4));
    WPK_HIP(hipMalloc((void **)&t.w, pr.w_elems * 4));
    for (int split = 0; split < 2; ++split) WPK_HIP(hipMalloc((void **)&t.wp[split], packed_bytes(pr, split != 0)));
    WPK_HIP(hipMalloc((void **)&t.y, pr.y_elems * 4));
    WPK_HIP(hipMalloc((void **)&t.yref, pr.y_elems * 4));
    WPK_HIP(hipMalloc((void **)&t.dref, pr.y_elems * 4));
    WPK_HIP(hipMalloc((void **)&t.err_bits, sizeof(unsigned)));
    int rc = upload_tap_table(pr, &t.ktab, t.st);
    if (rc != WPK_OK) return rc;
    float wscale = sqrtf(6.0f / (float)pr.CRS);  // uniform with the variance of Kaiming-normal
    hipLaunchKernelGGL(fill_hash_kernel, dim3(1024), dim3(256), 0, t.st, t.x, (long long)pr.x_elems,
                       0x1234u, 0.0f, 1.0f);
    hipLaunchKernelGGL(fill_hash_kernel, dim3(1024), dim3(256), 0, t.st, t.w, (long long)pr.w_elems,
                       0x9876u, -wscale, wscale);
    WPK_HIP(hipGetLastError());
    for (int split = 0; split < 2; ++split) {
        rc = pack_weights(pr, split != 0, t.w, t.wp[split], t.st);
        if (rc != WPK_OK) return rc;
    }
    rc = run_ref(pr, t.x, t.w, t.yref, t.dref, t.st);
    if (rc != WPK_OK) return rc;
    WPK_HIP(hipStreamSynchronize(t.st));
    return WPK_OK;
}

}  // namespace wpk

using namespace wpk;

// ---- plans ------------------------------------------------------------------------------------------
struct wpk_plan {
    struct Layer {
        Problem pr;
        wpk_conv_config cfg;       // of a launch without an epilogue,
        wpk_conv_config cfg_fused; // and with one: two choices where the default rule made them, else the same
        int unique;
        // packed weights, in the form of the split members ([1]) and of the others ([0]): whichever the layer's
        // configurations need; the direct kernel's plain [K][C][R][S] weights are in [0]
        float *wp[2];
        bool has_w;
        float *bias;  // library-owned copy of the layer's bias, or NULL
        int relu;
        bool direct;  // outside the tiled family
        // two-way pipelining: the batch split into images [0, half[0].d.n) and the rest
        Problem half[2];
        wpk_conv_config half_cfg[2], half_cfg_fused[2];
        // what a launch of the layer, or of half its batch, runs with (epilogue: it has a bias, a residual or a rectifier)
        const wpk_conv_config &config(int which, bool epilogue) const
        {
            return which < 0 ? (epilogue ? cfg_fused : cfg) : (epilogue ? half_cfg_fused[which] : half_cfg[which]);
        }
        bool epilogue(const float *residual) const { return bias || relu || residual; }
    };
    FixupBuf fix;  // fix-up workspace shared by the layers (they run one after another)
    // two-way pipelining (wpk_plan_set_pipeline): the second half-batch chain runs on `side`
    // with a workspace of its own; fork/join order it against the caller's stream
    int ways = 1;
    hipStream_t side = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    FixupBuf fix_side;
    std::vector<Layer> layers;
    std::vector<int32_t *> ktabs;  // one per distinct descriptor
    // verdict of the last check whether a pass's two half-batch chains touch disjoint memory,
    // and the pointers it was made for
    std::vector<const float *> chk_ptrs;
    bool chk_independent = false;
    std::vector<int32_t> tensor_layout;  // wpk_conv_plan_graph: the layout chosen for every tensor
};

// Makes sure that the layer holds its weights in the form cfg reads.  A plan allocates when it is built; only a
// configuration of the other form set afterwards comes here with weights already in place: they are
// taken from the form at hand (exactly), with the device drained before and after.
static int plan_need_weights(wpk_plan::Layer &L, const wpk_conv_config &cfg)
{
    const int s = split_member(cfg);
    if (L.wp[s]) return WPK_OK;
    float *packed = nullptr, *plain = nullptr;
    WPK_HIP(hipMalloc((void **)&packed, packed_bytes(L.pr, s != 0)));
    if (!L.has_w) {
        L.wp[s] = packed;
        return WPK_OK;
    }
    const int RS = packed_order(L.pr, s == 0);  // (of the form at hand)
    const void *const from = (const char *)L.wp[1 - s] + (s == 0 ? strip_bytes(L.pr) : 0);
    int rc = WPK_OK;
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMalloc((void **)&plain, (size_t)L.pr.w_elems * sizeof(float));
    if (e == hipSuccess) {
        hipLaunchKernelGGL(unpack_weights_kernel, dim3((unsigned)std::min<int64_t>(4096, (L.pr.w_elems + 255) / 256)),
                           dim3(256), 0, nullptr, from, plain, L.pr.d.k, L.pr.d.c, L.pr.CRS,
                           L.pr.Kpad, RS, 1 - s);
        rc = pack_weights(L.pr, s != 0, plain, packed, nullptr);
        e = hipDeviceSynchronize();
    }
    if (plain) (void)hipFree(plain);
    if (e != hipSuccess) {
        set_last_hip_error((int)e);
        rc = WPK_E_HIP;
    }
    if (rc == WPK_OK) L.wp[s] = packed;
    else (void)hipFree(packed);
    return rc;
}

// A layer's configurations where nobody set one: the cached result of a search, or the defaults.
static void plan_choose(const Problem &pr, wpk_conv_config *cfg, wpk_conv_config *cfg_fused)
{
    if (wpk_cache_lookup(&pr.d, cfg) == 1 && legal_for(pr, *cfg)) {
        *cfg_fused = *cfg;
        return;
    }
    default_config(pr, g_cus, cfg, true);
    *cfg_fused = *cfg;  // (only the wave-split members have two; the others would be priced twice)
    if (cfg->bm == kWaveSplitBm) default_config(pr, g_cus, cfg_fused, false);
}

// Room for the shared tiles of either.
static int plan_reserve(FixupBuf &fix, const Problem &pr, const wpk_conv_config &cfg, const wpk_conv_config &cfg_fused)
{
    const int64_t bytes = std::max(fixup_need(pr, cfg, g_cus).bytes, fixup_need(pr, cfg_fused, g_cus).bytes);
    return bytes > 0 ? fixup_reserve(fix, (size_t)bytes) : WPK_OK;
}

extern "C" {

int wpk_device_info(char *name, int32_t cap, int32_t *cus)
{
    std::lock_guard<std::mutex> g(g_mu);
    int rc = ensure_device();
    if (rc != WPK_OK) return rc;
    if (name && cap > 0) {
        strncpy(name, device_name().c_str(), cap - 1);
        name[cap - 1] = 0;
    }
    if (cus) *cus = g_cus;
    return WPK_OK;
}

int wpk_measure_peaks(double sustain_ms, double *mfma_burst, double *mfma_sustained, double *copy_gbs, void *stream)
{
    std::lock_guard<std::mutex> g(g_mu);
    int rc = ensure_device();
    if (rc != WPK_OK) return rc;
    if (!(sustain_ms >= 0.0) || sustain_ms > 10000.0) return WPK_E_BAD_ARG;
    hipStream_t st = (hipStream_t)stream;
    const int blocks = 2 * g_cus, iters = 350;          // about 0.3 ms per launch at 2.4 GHz
    const double flop = (double)blocks * 4 * iters * 16 * 4096.0;
    const long long copy_bytes = 256ll << 20;
    float *out = nullptr, *src = nullptr, *dst = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t err = hipSuccess;
    auto ok = [&](hipError_t e) { if (err == hipSuccess) err = e; return err == hipSuccess; };
    float ms = 0.f;
    if (ok(hipMalloc((void **)&out, (size_t)blocks * 256 * 4)) && ok(hipEventCreate(&e0)) && ok(hipEventCreate(&e1))) {
        if (mfma_burst || mfma_sustained) {
            // clocks settle high while the device idles: one launch right after a pause
            hipLaunchKernelGGL(mfma_only_kernel, dim3(blocks), dim3(256), 0, st, out, 8);
            ok(hipStreamSynchronize(st));
            std::this_thread::sleep_for(std::chrono::milliseconds(20));
            ok(hipEventRecord(e0, st));
            hipLaunchKernelGGL(mfma_only_kernel, dim3(blocks), dim3(256), 0, st, out, iters);
            ok(hipEventRecord(e1, st));
            ok(hipEventSynchronize(e1));
            if (ok(hipEventElapsedTime(&ms, e0, e1)) && mfma_burst) *mfma_burst = flop / (ms * 1e-3) / 1e12;
            // then back-to-back launches for sustain_ms; the rate of the second half counts
            const int half = std::max(1, (int)(sustain_ms / 0.3 / 2));
            for (int i = 0; i < half; ++i) hipLaunchKernelGGL(mfma_only_kernel, dim3(blocks), dim3(256), 0, st, out, iters);
            ok(hipEventRecord(e0, st));
            for (int i = 0; i < half; ++i) hipLaunchKernelGGL(mfma_only_kernel, dim3(blocks), dim3(256), 0, st, out, iters);
            ok(hipEventRecord(e1, st));
            ok(hipEventSynchronize(e1));
            if (ok(hipEventElapsedTime(&ms, e0, e1)) && mfma_sustained)
                *mfma_sustained = flop * half / (ms * 1e-3) / 1e12;
        }
        if (copy_gbs && ok(hipMalloc((void **)&src, copy_bytes)) && ok(hipMalloc((void **)&dst, copy_bytes)) &&
            ok(hipMemsetAsync(src, 0, copy_bytes, st))) {
            const int reps = 5;
            hipLaunchKernelGGL(copy16_kernel, dim3(g_cus * 8), dim3(256), 0, st, (const float4 *)src, (float4 *)dst,
                               copy_bytes / 16);
            ok(hipEventRecord(e0, st));
            for (int i = 0; i < reps; ++i)
                hipLaunchKernelGGL(copy16_kernel, dim3(g_cus * 8), dim3(256), 0, st, (const float4 *)src,
                                   (float4 *)dst, copy_bytes / 16);
            ok(hipEventRecord(e1, st));
            ok(hipEventSynchronize(e1));
            if (ok(hipEventElapsedTime(&ms, e0, e1))) *copy_gbs = 2.0 * copy_bytes * reps / (ms * 1e-3) / 1e9;
        }
        ok(hipGetLastError());
    }
    (void)hipStreamSynchronize(st);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (out) (void)hipFree(out);
    if (src) (void)hipFree(src);
    if (dst) (void)hipFree(dst);
    if (err != hipSuccess) {
        set_last_hip_error((int)err);
        return WPK_E_HIP;
    }
    return WPK_OK;
}

int wpk_config_default(const wpk_conv_desc *d, wpk_conv_config *out)
{
    if (!out) return WPK_E_NULL_PTR;
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    if (!pr.tiled_ok) return WPK_E_UNSUPPORTED;
    default_config(pr, g_cus, out);
    return WPK_OK;
}

int wpk_conv2d_ref(const wpk_conv_desc *d, const float *x, const float *w, float *y, void *stream)
{
    Problem pr;
    int rc = check_io(d, x, w, y, &pr);
    if (rc != WPK_OK) return rc;
    return run_ref(pr, x, w, y, nullptr, (hipStream_t)stream);
}

int wpk_conv2d_fwd_config(const wpk_conv_desc *d, const wpk_conv_config *cfg, const float *x,
                          const float *w, float *y, void *stream)
{
    Problem pr;
    int rc = check_io(d, x, w, y, &pr);
    if (rc != WPK_OK) return rc;
    if (!cfg) return WPK_E_NULL_PTR;
    if (!legal_for(pr, *cfg)) return WPK_E_NO_CONFIG;
    return fwd_with(pr, *cfg, x, w, y, (hipStream_t)stream);
}

int wpk_conv2d_fwd(const wpk_conv_desc *d, const float *x, const float *w, float *y, void *stream)
{
    Problem pr;
    int rc = check_io(d, x, w, y, &pr);
    if (rc != WPK_OK) return rc;
    if (!pr.tiled_ok) return run_ref(pr, x, w, y, nullptr, (hipStream_t)stream);
    {
        std::lock_guard<std::mutex> g(g_mu);
        rc = ensure_device();
        if (rc != WPK_OK) return rc;
    }
    wpk_conv_config cfg;
    if (wpk_cache_lookup(d, &cfg) != 1 || !legal_for(pr, cfg)) default_config(pr, g_cus, &cfg);
    return fwd_with(pr, cfg, x, w, y, (hipStream_t)stream);
}

// ---- the entry point that allocates nothing ---------------------------------------------------------
// Everything wpk_conv2d_fwd_config keeps in library-owned device memory (lookup table, packed
// weights, arrival counters and partial-tile slots of shared tiles) lives in one static device
// array instead.  Layout: [lookup table, 64 KiB][arrival counters, 1 MiB][slots][packed weights];
// the counters stay where they are from call to call, so they are zero whenever a launch starts.
// In host code the array's name is only a handle: its device address is asked for once per
// device and kept.
static const size_t kScratchTapBytes = 64 << 10;
static const size_t kScratchRoom = (size_t)WPK_NOALLOC_SCRATCH_BYTES - kScratchTapBytes - (size_t)kFixupCounterBytes;
// (the limits are stated for weights of four bytes; the split members' take six, and so does the array's room)
static const size_t kScratchRoomSplit = kScratchRoom / sizeof(float) * kSplitWeightBytes;
static __device__ __align__(256) unsigned char scratch[kScratchTapBytes + kFixupCounterBytes + kScratchRoomSplit];
static const int kScratchMaxDevices = 64;
static char *g_scratch_ptr[kScratchMaxDevices];   // per device, filled on first use (under g_mu)

extern "C" int wpk_conv2d_fwd_noalloc(const wpk_conv_desc *d, const wpk_conv_config *cfg_in, const float *x,
                                      const float *w, float *y, void *stream)
{
    Problem pr;
    int rc = check_io(d, x, w, y, &pr);
    if (rc != WPK_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    if (!pr.tiled_ok) {
        if (cfg_in) return WPK_E_NO_CONFIG;
        return run_ref(pr, x, w, y, nullptr, st);  // the direct kernel needs no scratch
    }
    if (cfg_in && !legal_for(pr, *cfg_in)) return WPK_E_NO_CONFIG;
    std::lock_guard<std::mutex> g(g_mu);
    rc = ensure_device();
    if (rc != WPK_OK) return rc;
    int dev = 0;
    WPK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kScratchMaxDevices) return WPK_E_UNSUPPORTED;
    if (!g_scratch_ptr[dev]) {
        char *ptr = nullptr;
        WPK_HIP(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return WPK_E_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    char *const base = g_scratch_ptr[dev];
    wpk_conv_config cfg;
    if (cfg_in) cfg = *cfg_in;
    else if (wpk_cache_lookup(d, &cfg) != 1 || !legal_for(pr, cfg)) default_config(pr, g_cus, &cfg);
    auto round256 = [](size_t v) { return (v + 255) / 256 * 256; };
    // (split weights of padded channels may not fit where four bytes each of the plain ones do)
    if (split_member(cfg) && round256(packed_bytes(pr, true)) > kScratchRoomSplit)
        cfg = wpk_conv_config{64, 64, 32, 2, 2, 1, 1, 0, 2, 0};
    const bool split = split_member(cfg);
    const size_t wbytes = round256(packed_bytes(pr, split)), room = split ? kScratchRoomSplit : kScratchRoom;
    if (tap_table_bytes(pr) > kScratchTapBytes || round256(packed_bytes(pr, false)) > kScratchRoom) return WPK_E_TOO_LARGE;
    // shared tiles meet in the slots if they fit beside the weights, else through atomics into y
    const FixupNeed need = fixup_need(pr, cfg, g_cus);
    const size_t slot_bytes = need.bytes > 0 ? round256((size_t)(need.bytes - need.slots_offset)) : 0;
    FixupBuf fix;
    fix.ptr = base + kScratchTapBytes;
    fix.bytes = 0;
    if (need.bytes > 0 && wbytes + slot_bytes <= room) fix.bytes = (size_t)need.bytes;
    float *const wp = (float *)(base + kScratchTapBytes + kFixupCounterBytes + (fix.bytes ? slot_bytes : 0));
    int32_t *const ktab = (int32_t *)base;
    if (fix.bytes) {
        // the counters this launch uses start at zero whatever an earlier call left (a fill kernel:
        // memset nodes do not replay reliably from a captured graph)
        const long long n4 = (need.shared_tiles + 3) / 4;
        hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)std::min<long long>(256, (n4 + 255) / 256)), dim3(256), 0,
                           st, (float4 *)fix.ptr, (float *)nullptr, n4, 0);
        WPK_HIP(hipGetLastError());
    }
    rc = write_tap_table(pr, ktab, st);
    if (rc != WPK_OK) return rc;
    rc = pack_weights(pr, split, w, wp, st);
    if (rc != WPK_OK) return rc;
    return run_config(pr, cfg, ktab, x, wp, y, fix.bytes ? &fix : nullptr, st);
}

static int fwd_fused(const wpk_conv_desc *d, const wpk_conv_config *cfg_in, const float *x,
                     const float *w, const Epilogue &epi, float *y, hipStream_t st)
{
    Problem pr;
    int rc = check_io(d, x, w, y, &pr);
    if (rc != WPK_OK) return rc;
    if (cfg_in && !legal_for(pr, *cfg_in)) return WPK_E_NO_CONFIG;
    if (!pr.tiled_ok) {
        rc = run_ref(pr, x, w, y, nullptr, st);
        return rc != WPK_OK ? rc : run_epilogue(pr, epi, y, st);
    }
    {
        std::lock_guard<std::mutex> g(g_mu);
        rc = ensure_device();
        if (rc != WPK_OK) return rc;
    }
    wpk_conv_config cfg;
    if (cfg_in) cfg = *cfg_in;
    else if (wpk_cache_lookup(d, &cfg) != 1 || !legal_for(pr, cfg)) default_config(pr, g_cus, &cfg, !epi.any());
    return fwd_with(pr, cfg, x, w, y, st, epi);
}

int wpk_conv2d_fwd_fused(const wpk_conv_desc *d, const float *x, const float *w, const float *bias,
                         const float *residual, int32_t relu, float *y, void *stream)
{
    Epilogue epi;
    epi.bias = bias; epi.res = residual; epi.relu = relu != 0;
    return fwd_fused(d, nullptr, x, w, epi, y, (hipStream_t)stream);
}

int wpk_conv2d_fwd_fused_config(const wpk_conv_desc *d, const wpk_conv_config *cfg, const float *x,
                                const float *w, const float *bias, const float *residual,
                                int32_t relu, float *y, void *stream)
{
    if (!cfg) return WPK_E_NULL_PTR;
    Epilogue epi;
    epi.bias = bias; epi.res = residual; epi.relu = relu != 0;
    return fwd_fused(d, cfg, x, w, epi, y, (hipStream_t)stream);
}

int wpk_conv_tune_ex(const wpk_conv_desc *d, const wpk_tune_options *opt_in, int force,
                     wpk_tune_report *report)
{
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    if (!pr.tiled_ok) return WPK_E_UNSUPPORTED;
    {
        std::lock_guard<std::mutex> g(g_mu);
        rc = ensure_device();
        if (rc != WPK_OK) return rc;
    }
    wpk_conv_config cached;
    if (!force && wpk_cache_lookup(d, &cached) == 1 && legal_for(pr, cached)) {
        if (report) {
            memset(report, 0, sizeof *report);
            report->best = cached;
        }
        return wpk_config_id(&cached);
    }
    auto t_start = std::chrono::steady_clock::now();
    TuneCtx t;
    t.pr = pr;
    prepare_strip(&t.pr, g_cus);
    if (opt_in) t.opt = *opt_in; else wpk_tune_default_options(&t.opt);
    t.st = nullptr; t.e0 = t.e1 = nullptr;
    t.x = t.w = t.wp[0] = t.wp[1] = t.y = t.yref = t.dref = nullptr;
    t.err_bits = nullptr; t.ktab = nullptr;
    t.rejected = 0; t.hip_failed = 0;
    t.phase = WPK_STAGE_SEARCH;
    rc = tune_setup(t);
    if (rc != WPK_OK) {
        tune_free(t);
        return rc;
    }
    wpk_conv_config defcfg;
    default_config(pr, g_cus, &defcfg, t.opt.epilogue == 0);
    double def_us = 0, def_err = 0;
    rc = measure_us(t, defcfg, &def_us, &def_err);
    if (rc != WPK_OK) {
        tune_free(t);
        return rc;
    }
    int32_t lo[WPK_N_GENES], hi[WPK_N_GENES], best_genes[WPK_N_GENES];
    wpk_config_gene_ranges(lo, hi);
    double best_f = 0;
    int32_t evals = 0;
    int gens = 0;
    if (t.opt.mode == 2) {  // exhaustive: every legal chromosome once
        int32_t g[WPK_N_GENES] = {0};
        for (;;) {
            if (tune_constraint(g, WPK_N_GENES, &t)) {
                double f = tune_fitness(g, WPK_N_GENES, &t);
                ++evals;
                if (f > best_f) {
                    best_f = f;
                    memcpy(best_genes, g, sizeof g);
                }
            }
            int i = 0;
            while (i < WPK_N_GENES && ++g[i] > hi[i]) g[i++] = 0;
            if (i == WPK_N_GENES) break;
        }
        gens = 1;
    } else {
        gens = wpk_ga_search(WPK_N_GENES, lo, hi, tune_constraint, tune_fitness, &t, &t.opt,
                             best_genes, &best_f, &evals, nullptr, nullptr, nullptr, 0);
    }
    const double search_us = best_f > 0.0 ? 1.0 / best_f : 0.0;  // what the search alone found
    int best_stage = WPK_STAGE_SEARCH;
    if (t.opt.mode != 2 && t.opt.refine > 0 && best_f > 0.0 && !t.hip_failed && gens >= 0) {
        t.phase = WPK_STAGE_RULE;
        // rule-based candidates beside the search's winner: the tile shapes that exhaustive
        // searches over the workloads' layers put on top most often, each with the persistent
        // schedules and with reductions split to about 3.5 workgroups per compute unit
        {
            static const int32_t kShapes[][6] = {{64, 64, 16, 2, 2, 2},  {64, 64, 32, 2, 2, 2}, {64, 128, 16, 2, 2, 2},
                                                 {128, 64, 16, 2, 2, 2}, {64, 64, 32, 2, 2, 1}, {128, 64, 32, 4, 2, 2}};
            auto consider = [&](const wpk_conv_config &c) {
                int32_t g[WPK_N_GENES];
                if (wpk_config_to_genes(&c, g) != WPK_OK || !tune_constraint(g, WPK_N_GENES, &t) || tune_known(t, c))
                    return;
                double f = tune_fitness(g, WPK_N_GENES, &t);
                ++evals;
                if (f > best_f) {
                    best_f = f;
                    memcpy(best_genes, g, sizeof g);
                }
            };
            const int cus = g_cus > 0 ? g_cus : 256;
            for (const auto &sh : kShapes) {
                wpk_conv_config c = {sh[0], sh[1], sh[2], sh[3], sh[4], 1, 0, 0, sh[5], 0};
                for (int p = 1; p <= 4; ++p) {
                    c.persist = p;
                    c.xcd_remap = 1;
                    c.reduce = 0;
                    consider(c);
                    c.reduce = 1;
                    consider(c);
                }
                c.persist = 0;
                c.reduce = 0;
                c.xcd_remap = 1;
                int64_t tiles = ((pr.M + c.bm - 1) / c.bm) * ((pr.d.k + c.bn - 1) / c.bn);
                int want = (int)std::max<int64_t>(1, (7 * (int64_t)cus / 2 + tiles / 2) / tiles);
                for (int i = 0; i < kGeneCounts[5]; ++i) {
                    int sk = kSplitVals[i];
                    if (sk < want - 1 || sk > want + 2) continue;
                    c.split_k = sk;
                    c.reduce = 0;
                    consider(c);
                    if (sk > 1) {
                        c.reduce = 1;
                        consider(c);
                    }
                }
            }
            // small launches: the wave-split members, one to four waves per tile, the reduction cut
            // between workgroups to about one wave per SIMD (half and twice that as well)
            if (wave_split_candidate(pr, 65536)) {
                const int64_t blocks = ((pr.M + 31) / 32) * ((pr.d.k + 31) / 32), octets = pr.CRS / 8;
                for (int wk = 1; wk <= 4; wk *= 2)
                    for (int st = 1; st <= 2; ++st) {
                        if (blocks * wk > 8 * (int64_t)cus) continue;
                        wpk_conv_config c = {kWaveSplitBm, 32, 8, wk, 1, 1, 1, 0, st, 0};
                        const int64_t want = std::max<int64_t>(1, 4 * (int64_t)cus / (blocks * wk));
                        for (int i = 0; i < kGeneCounts[5]; ++i) {
                            const int sk = kSplitVals[i];
                            if (2 * sk < want || sk > 2 * want || (sk > 1 && octets / (wk * sk) < 4)) continue;
                            c.split_k = sk;
                            c.reduce = 0;
                            consider(c);
                            if (sk > 1) {
                                c.reduce = 1;
                                consider(c);
                            }
                        }
                    }
            }
            // few pixels, long reductions (late layers of a batch): the wave-split members with 64 channels
            // per tile came out level with the best tiled member in exhaustive searches there (3x3, 512
            // channels, 7x7 pixels, 16 images: 38.8 against 39.2 us), with the reduction cut to about two
            // waves per SIMD
            else if ((pr.tapmajor || pr.xquad) && pr.M <= 1024) {
                const int64_t blocks = ((pr.M + 31) / 32) * ((pr.d.k + 63) / 64), octets = pr.CRS / 8;
                for (int wk = 2; wk <= 4; wk *= 2) {
                    wpk_conv_config c = {kWaveSplitBm, 64, 8, wk, 1, 1, 0, 0, 1, 0};
                    const int64_t want = std::max<int64_t>(1, 8 * (int64_t)cus / (blocks * wk));
                    for (int i = 0; i < kGeneCounts[5]; ++i) {
                        const int sk = kSplitVals[i];
                        if (2 * sk < want || sk > 2 * want || (sk > 1 && octets / (wk * sk) < 4)) continue;
                        c.split_k = sk;
                        for (int rm = 0; rm <= 1; ++rm) {
                            c.xcd_remap = rm;
                            consider(c);
                        }
                    }
                }
            }
        }
        // one gene of the winner at a time, every other value of it
        t.phase = WPK_STAGE_REFINE;
        for (int round = 0; round < t.opt.refine; ++round) {
            bool moved = false;
            for (int gi = 0; gi < WPK_N_GENES; ++gi) {
                int32_t cand[WPK_N_GENES];
                memcpy(cand, best_genes, sizeof cand);
                for (int32_t v = lo[gi]; v <= hi[gi]; ++v) {
                    cand[gi] = v;
                    wpk_conv_config c;
                    if (v == best_genes[gi] || !tune_constraint(cand, WPK_N_GENES, &t) ||
                        wpk_config_from_genes(cand, &c) != WPK_OK || tune_known(t, c))
                        continue;
                    double f = tune_fitness(cand, WPK_N_GENES, &t);
                    ++evals;
                    if (f > best_f) {
                        best_f = f;
                        best_genes[gi] = v;
                        moved = true;
                    }
                }
            }
            if (!moved) break;
        }
        // the five fastest so far once more, in groups long enough for the clocks to settle
        // where they stay under continuous load: neither a lucky sample nor a short burst at
        // boost clocks must decide
        std::vector<std::pair<double, int>> order;
        for (auto &kv : t.times_us) order.push_back({kv.second, kv.first});
        std::sort(order.begin(), order.end());
        double again_best = 0;
        const double group_us = t.opt.min_group_us;
        const int reps = t.opt.reps;
        t.opt.min_group_us = std::max(group_us, 4000.0);
        t.opt.reps = 3;
        for (size_t i = 0; i < order.size() && i < 5 && !t.hip_failed; ++i) {
            wpk_conv_config c;
            int32_t g[WPK_N_GENES];
            if (wpk_config_from_id(order[i].second, &c) != WPK_OK || wpk_config_to_genes(&c, g) != WPK_OK)
                continue;
            double us = 0, err = 0;
            int r = measure_us(t, c, &us, &err);
            if (r != WPK_OK) { t.hip_failed = r; break; }
            if (us > 0.0 && (again_best == 0 || us < again_best)) {
                again_best = us;
                memcpy(best_genes, g, sizeof g);
                best_stage = t.stage_of.count(order[i].second) ? t.stage_of[order[i].second] : WPK_STAGE_SEARCH;
            }
        }
        // Launch order against XCD-contiguous ranges is a few percent of time either way, but a half to a
        // third of the bytes fetched from memory where every XCD would otherwise read all the weights: a
        // winner in launch order gives way to its XCD-contiguous twin when that is within 2 % of it.
        if (again_best > 0 && !t.hip_failed) {
            wpk_conv_config c;
            int32_t g[WPK_N_GENES];
            if (wpk_config_from_genes(best_genes, &c) == WPK_OK && c.xcd_remap == 0 && c.persist == 0) {
                c.xcd_remap = 1;
                if (wpk_config_to_genes(&c, g) == WPK_OK && tune_constraint(g, WPK_N_GENES, &t)) {
                    double us = 0, err = 0;
                    int r = measure_us(t, c, &us, &err);
                    if (r != WPK_OK) {
                        t.hip_failed = r;
                    } else if (us > 0.0 && us <= 1.02 * again_best) {
                        again_best = us;
                        memcpy(best_genes, g, sizeof g);
                    }
                }
            }
        }
        if (again_best > 0) best_f = 1.0 / again_best;
        // the default once more under the same protocol, so that the comparison below is between
        // two measurements taken the same way
        if (def_us > 0.0 && !t.hip_failed) {
            double us = 0, err = 0;
            int r = measure_us(t, defcfg, &us, &err);
            if (r != WPK_OK) t.hip_failed = r;
            else if (us > 0.0) def_us = us;
        }
        t.opt.min_group_us = group_us;
        t.opt.reps = reps;
    }
    int result;
    if (t.hip_failed) {
        result = t.hip_failed;
    } else if (gens < 0) {
        result = gens;
    } else if (!(best_f > 0.0)) {
        result = WPK_E_VERIFY;
    } else {
        wpk_conv_config best;
        wpk_config_from_genes(best_genes, &best);
        best = same_launch(pr, best, g_cus);
        double best_us = 1.0 / best_f;
        if (def_us > 0.0 && def_us < best_us) {  // never hand back something slower than the default
            best = defcfg;
            best_us = def_us;
            best_stage = WPK_STAGE_DEFAULT;
        }
        wpk_cache_store(d, &best, best_us);
        if (report) {
            report->best = best;
            report->best_us = best_us;
            report->default_us = def_us;
            report->evaluations = evals;
            report->generations = gens;
            report->rejected = t.rejected;
            report->stage = best_stage;
            report->search_us = search_us;
            report->seconds =
                std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
        }
        result = wpk_config_id(&best);
    }
    tune_free(t);
    return result;
}

int wpk_conv_tune(const wpk_conv_desc *d) { return wpk_conv_tune_ex(d, nullptr, 0, nullptr); }

// Runtime of one layer for the layout choice: the cached search result's, a fresh search's, or the
// default configuration timed under the tuner's protocol (synthetic operands of its own).
static int layer_runtime_us(const wpk_conv_desc *d, int32_t tune, double *us)
{
    wpk_conv_config cfg;
    if (wpk_cache_lookup_time(d, &cfg, us) == 1 && *us > 0.0) return WPK_OK;
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    if (!pr.tiled_ok) {  // direct kernel: no estimate worth taking; a large constant keeps it out of the choice
        *us = 1e9;
        return WPK_OK;
    }
    if (tune) {
        wpk_tune_report rep;
        int id = wpk_conv_tune_ex(d, nullptr, 0, &rep);
        if (id < 0) return id;
        *us = rep.best_us;
        return WPK_OK;
    }
    TuneCtx t;
    t.pr = pr;
    prepare_strip(&t.pr, g_cus);
    wpk_tune_default_options(&t.opt);
    t.opt.reps = 3;
    t.st = nullptr; t.e0 = t.e1 = nullptr;
    t.x = t.w = t.wp[0] = t.wp[1] = t.y = t.yref = t.dref = nullptr;
    t.err_bits = nullptr; t.ktab = nullptr;
    t.rejected = 0; t.hip_failed = 0;
    t.phase = WPK_STAGE_DEFAULT;
    rc = tune_setup(t);
    if (rc == WPK_OK) {
        default_config(pr, g_cus, &cfg);
        double err = 0;
        rc = measure_us(t, cfg, us, &err);
        if (rc == WPK_OK && !(*us > 0.0)) rc = WPK_E_VERIFY;
    }
    tune_free(t);
    return rc;
}

int wpk_conv_plan_graph(const wpk_conv_desc *layers, int32_t n_layers, const int32_t *x_tensor,
                        const int32_t *y_tensor, const int32_t *residual_tensor,
                        const int32_t *tensor_layout, int32_t n_tensors, int32_t tune, wpk_plan **out)
{
    if (!layers || !out || !x_tensor || !y_tensor || !tensor_layout) return WPK_E_NULL_PTR;
    if (n_layers <= 0 || n_tensors <= 0) return WPK_E_BAD_ARG;
    {
        std::lock_guard<std::mutex> g(g_mu);
        int rc = ensure_device();
        if (rc != WPK_OK) return rc;
    }
    // validate the graph before anything is timed (the optimiser checks ranges and ties)
    std::vector<double> cost((size_t)n_layers * 4, 0.0);
    std::vector<int32_t> chosen(n_tensors, 0);
    int rc = wpk_choose_layouts(n_layers, x_tensor, y_tensor, residual_tensor, tensor_layout, n_tensors,
                                cost.data(), chosen.data(), nullptr);
    if (rc != WPK_OK) return rc;
    // cost of every layer under every combination its tensors may take; identical layers share it
    std::map<std::string, double> timed;
    for (int i = 0; i < n_layers; ++i)
        for (int lx = 0; lx < 2; ++lx)
            for (int ly = 0; ly < 2; ++ly) {
                const int fx = tensor_layout[x_tensor[i]], fy = tensor_layout[y_tensor[i]];
                if ((fx >= 0 && fx != lx) || (fy >= 0 && fy != ly)) continue;
                wpk_conv_desc d = layers[i];
                d.layout = lx | (ly << 1);
                const std::string key = desc_key(&d);
                auto it = timed.find(key);
                if (it == timed.end()) {
                    double us = 0.0;
                    rc = layer_runtime_us(&d, tune, &us);
                    if (rc != WPK_OK) return rc;
                    it = timed.emplace(key, us).first;
                }
                cost[(size_t)i * 4 + lx * 2 + ly] = it->second;
            }
    rc = wpk_choose_layouts(n_layers, x_tensor, y_tensor, residual_tensor, tensor_layout, n_tensors, cost.data(),
                            chosen.data(), nullptr);
    if (rc != WPK_OK) return rc;
    std::vector<wpk_conv_desc> laid(layers, layers + n_layers);
    for (int i = 0; i < n_layers; ++i) laid[i].layout = chosen[x_tensor[i]] | (chosen[y_tensor[i]] << 1);
    rc = wpk_conv_plan(laid.data(), n_layers, tune, out);
    if (rc != WPK_OK) return rc;
    (*out)->tensor_layout = chosen;
    return WPK_OK;
}

int wpk_plan_tensor_layout(const wpk_plan *plan, int32_t tensor)
{
    if (!plan) return WPK_E_NULL_PTR;
    if (tensor < 0 || tensor >= (int)plan->tensor_layout.size()) return WPK_E_BAD_ARG;
    return plan->tensor_layout[tensor];
}

int wpk_plan_layer_layout(const wpk_plan *plan, int32_t layer)
{
    if (!plan) return WPK_E_NULL_PTR;
    if (layer < 0 || layer >= (int)plan->layers.size()) return WPK_E_BAD_ARG;
    return plan->layers[layer].pr.d.layout;
}

int wpk_conv_plan(const wpk_conv_desc *layers, int32_t n_layers, int32_t tune, wpk_plan **out)
{
    if (!layers || !out) return WPK_E_NULL_PTR;
    if (n_layers <= 0) return WPK_E_BAD_ARG;
    {
        std::lock_guard<std::mutex> g(g_mu);
        int rc = ensure_device();
        if (rc != WPK_OK) return rc;
    }
    wpk_plan *plan = new wpk_plan();
    std::map<std::string, int> seen;  // identical descriptors share one search and one tap table
    int rc = WPK_OK;
    for (int i = 0; i < n_layers && rc == WPK_OK; ++i) {
        wpk_plan::Layer L;
        rc = make_problem(&layers[i], &L.pr);
        if (rc != WPK_OK) break;
        L.wp[0] = L.wp[1] = nullptr;
        L.has_w = false;
        L.bias = nullptr;
        L.relu = 0;
        L.direct = !L.pr.tiled_ok;
        if (L.direct) {  // oversized filter, or a channels-last shape the tiled gather does not take
            memset(&L.cfg, 0, sizeof L.cfg);
            L.cfg_fused = L.cfg;
            L.unique = -1;
            hipError_t e = hipMalloc((void **)&L.wp[0], (size_t)L.pr.w_elems * sizeof(float));
            if (e != hipSuccess) { set_last_hip_error((int)e); rc = WPK_E_HIP; break; }
            plan->layers.push_back(L);
            continue;
        }
        std::string key = desc_key(&layers[i]);
        auto it = seen.find(key);
        if (it == seen.end()) {
            int32_t *ktab = nullptr;
            rc = upload_tap_table(L.pr, &ktab, nullptr);
            if (rc != WPK_OK) break;
            plan->ktabs.push_back(ktab);
            it = seen.emplace(key, (int)plan->ktabs.size() - 1).first;
            if (tune) {
                int id = wpk_conv_tune(&layers[i]);
                if (id < 0) { rc = id; break; }
            }
        }
        L.unique = it->second;
        prepare_strip(&L.pr, g_cus);
        plan_choose(L.pr, &L.cfg, &L.cfg_fused);
        rc = plan_need_weights(L, L.cfg);
        if (rc == WPK_OK) rc = plan_need_weights(L, L.cfg_fused);
        plan->layers.push_back(L);
        if (rc != WPK_OK) break;
        rc = plan_reserve(plan->fix, L.pr, L.cfg, L.cfg_fused);
    }
    if (rc == WPK_OK) {  // the tap tables were written on the null stream: complete before any stream reads them
        hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) { set_last_hip_error((int)e); rc = WPK_E_HIP; }
    }
    if (rc != WPK_OK) {
        wpk_plan_destroy(plan);
        return rc;
    }
    *out = plan;
    return WPK_OK;
}

int wpk_plan_set_weights(wpk_plan *plan, int32_t layer, const float *w, void *stream)
{
    if (!plan || !w) return WPK_E_NULL_PTR;
    if (layer < 0 || layer >= (int)plan->layers.size()) return WPK_E_BAD_ARG;
    wpk_plan::Layer &L = plan->layers[layer];
    if (L.direct) {
        WPK_HIP(hipMemcpyAsync(L.wp[0], w, (size_t)L.pr.w_elems * sizeof(float), hipMemcpyDeviceToDevice,
                               (hipStream_t)stream));
        L.has_w = true;
        return WPK_OK;
    }
    int rc = WPK_OK;
    for (int s = 0; s < 2 && rc == WPK_OK; ++s)
        if (L.wp[s]) rc = pack_weights(L.pr, s != 0, w, L.wp[s], (hipStream_t)stream);
    if (rc == WPK_OK) L.has_w = true;
    return rc;
}

int wpk_plan_set_epilogue(wpk_plan *plan, int32_t layer, const float *bias, int32_t relu, void *stream)
{
    if (!plan) return WPK_E_NULL_PTR;
    if (layer < 0 || layer >= (int)plan->layers.size()) return WPK_E_BAD_ARG;
    wpk_plan::Layer &L = plan->layers[layer];
    if (bias) {
        if (!L.bias) WPK_HIP(hipMalloc((void **)&L.bias, (size_t)L.pr.d.k * 4));
        WPK_HIP(hipMemcpyAsync(L.bias, bias, (size_t)L.pr.d.k * 4, hipMemcpyDeviceToDevice,
                               (hipStream_t)stream));
    } else if (L.bias) {
        WPK_HIP(hipFree(L.bias));  // synchronises: no launch still reads it
        L.bias = nullptr;
    }
    L.relu = relu != 0;
    return WPK_OK;
}

// One layer (or, with which = 0/1, one half-batch of it) on stream st.
static int plan_launch(wpk_plan *plan, wpk_plan::Layer &L, int which, const float *x,
                       const float *residual, float *y, hipStream_t st, bool y_zeroed = false)
{
    const Problem &pr = which < 0 ? L.pr : L.half[which];
    const wpk_conv_config &cfg = L.config(which, L.epilogue(residual));
    if (which == 1) {  // the second half starts after the images of the first
        x += L.half[0].x_elems;
        y += L.half[0].y_elems;
        if (residual) residual += L.half[0].y_elems;
    }
    Epilogue epi;
    epi.bias = L.bias; epi.res = residual; epi.relu = L.relu;
    if (L.direct) {
        int rc = run_ref(pr, x, L.wp[0], y, nullptr, st);
        return rc != WPK_OK ? rc : run_epilogue(pr, epi, y, st);
    }
    return run_config(pr, cfg, plan->ktabs[L.unique], x, L.wp[split_member(cfg)], y,
                      which == 1 ? &plan->fix_side : &plan->fix, st, epi, y_zeroed);
}

static int plan_fork(wpk_plan *plan, hipStream_t user)
{
    WPK_HIP(hipEventRecord(plan->fork, user));
    WPK_HIP(hipStreamWaitEvent(plan->side, plan->fork, 0));
    return WPK_OK;
}

static int plan_join(wpk_plan *plan, hipStream_t user)
{
    WPK_HIP(hipEventRecord(plan->join, plan->side));
    WPK_HIP(hipStreamWaitEvent(user, plan->join, 0));
    return WPK_OK;
}

int wpk_plan_run_layer_fused(wpk_plan *plan, int32_t layer, const float *x, const float *residual,
                             float *y, void *stream)
{
    if (!plan || !x || !y) return WPK_E_NULL_PTR;
    if (layer < 0 || layer >= (int)plan->layers.size()) return WPK_E_BAD_ARG;
    wpk_plan::Layer &L = plan->layers[layer];
    if (!L.has_w) return WPK_E_BAD_ARG;
    if (plan->ways == 1) return plan_launch(plan, L, -1, x, residual, y, (hipStream_t)stream);
    int rc = plan_fork(plan, (hipStream_t)stream);
    if (rc == WPK_OK) rc = plan_launch(plan, L, 0, x, residual, y, (hipStream_t)stream);
    if (rc == WPK_OK) rc = plan_launch(plan, L, 1, x, residual, y, plan->side);
    int rj = plan_join(plan, (hipStream_t)stream);  // joined even after a failed launch
    return rc != WPK_OK ? rc : rj;
}

int wpk_plan_set_pipeline(wpk_plan *plan, int32_t ways)
{
    if (!plan) return WPK_E_NULL_PTR;
    if (ways != 1 && ways != 2) return WPK_E_BAD_ARG;
    if (ways == 1) {
        plan->ways = 1;
        return WPK_OK;
    }
    for (auto &L : plan->layers)
        if (L.pr.d.n < 2) return WPK_E_UNSUPPORTED;
    if (!plan->side) {
        WPK_HIP(hipStreamCreateWithFlags(&plan->side, hipStreamNonBlocking));
        WPK_HIP(hipEventCreateWithFlags(&plan->fork, hipEventDisableTiming));
        WPK_HIP(hipEventCreateWithFlags(&plan->join, hipEventDisableTiming));
    }
    WPK_HIP(hipDeviceSynchronize());  // workspaces may grow below
    for (auto &L : plan->layers) {
        for (int h = 0; h < 2; ++h) {
            int rc = make_part(L.pr, h == 0 ? (L.pr.d.n + 1) / 2 : L.pr.d.n / 2, &L.half[h]);
            if (rc != WPK_OK) return rc;
            if (L.direct) continue;
            prepare_strip(&L.half[h], g_cus);
            plan_choose(L.half[h], &L.half_cfg[h], &L.half_cfg_fused[h]);
            rc = plan_need_weights(L, L.half_cfg[h]);
            if (rc == WPK_OK) rc = plan_need_weights(L, L.half_cfg_fused[h]);
            if (rc == WPK_OK) rc = plan_reserve(h == 0 ? plan->fix : plan->fix_side, L.half[h], L.half_cfg[h], L.half_cfg_fused[h]);
            if (rc != WPK_OK) return rc;
        }
    }
    plan->ways = 2;
    return WPK_OK;
}

int wpk_plan_run_layer(wpk_plan *plan, int32_t layer, const float *x, float *y, void *stream)
{
    return wpk_plan_run_layer_fused(plan, layer, x, nullptr, y, stream);
}

// The two half-batch chains of a pipelined pass run with no ordering between them, so the pass
// may be split only if nothing one chain writes is touched by the other chain at ANY layer.  With
// buffers reused in turns by layers of different channel counts that fails: the second half of a
// small tensor starts inside the first half of a large one.  The verdict is kept for the pointers
// it was made for (a caller replays the same arrays pass after pass).
static bool chains_independent(wpk_plan *plan, const float *const *x, const float *const *residual,
                               float *const *y)
{
    const size_t nl = plan->layers.size();
    std::vector<const float *> key(3 * nl);
    for (size_t i = 0; i < nl; ++i) {
        key[3 * i] = x[i];
        key[3 * i + 1] = y[i];
        key[3 * i + 2] = residual ? residual[i] : nullptr;
    }
    if (key == plan->chk_ptrs) return plan->chk_independent;
    struct Range { uintptr_t lo, hi; };
    auto half_of = [](const float *p, int64_t first, int64_t second, int h) {
        Range r = {0, 0};
        if (p) {
            r.lo = (uintptr_t)(p + (h ? first : 0));
            r.hi = r.lo + (uintptr_t)(h ? second : first) * sizeof(float);
        }
        return r;
    };
    auto hit = [](const Range &a, const Range &b) { return a.lo < b.hi && b.lo < a.hi; };
    // per layer and chain: what it writes, and everything it touches
    std::vector<Range> wr(2 * nl), rd_x(2 * nl), rd_r(2 * nl);
    for (size_t i = 0; i < nl; ++i)
        for (int h = 0; h < 2; ++h) {
            const wpk_plan::Layer &L = plan->layers[i];
            wr[2 * i + h] = half_of(y[i], L.half[0].y_elems, L.half[1].y_elems, h);
            rd_x[2 * i + h] = half_of(x[i], L.half[0].x_elems, L.half[1].x_elems, h);
            rd_r[2 * i + h] = half_of(residual ? residual[i] : nullptr, L.half[0].y_elems, L.half[1].y_elems, h);
        }
    bool ok = true;
    for (size_t i = 0; i < nl && ok; ++i)
        for (int h = 0; h < 2 && ok; ++h)
            for (size_t j = 0; j < nl && ok; ++j) {
                const int o = 1 - h;
                ok = !hit(wr[2 * i + h], wr[2 * j + o]) && !hit(wr[2 * i + h], rd_x[2 * j + o]) &&
                     !hit(wr[2 * i + h], rd_r[2 * j + o]);
            }
    plan->chk_ptrs.swap(key);
    plan->chk_independent = ok;
    return ok;
}

int wpk_plan_run_fused(wpk_plan *plan, const float *const *x, const float *const *residual,
                       float *const *y, void *stream)
{
    if (!plan || !x || !y) return WPK_E_NULL_PTR;
    for (size_t i = 0; i < plan->layers.size(); ++i)
        if (!x[i] || !y[i]) return WPK_E_NULL_PTR;
    if (plan->ways == 1 || !chains_independent(plan, x, residual, y)) {
        const size_t nl = plan->layers.size();
        for (size_t i = 0; i < nl; ++i)
            if (!x[i] || !y[i]) return WPK_E_NULL_PTR;
            else if (!plan->layers[i].has_w) return WPK_E_BAD_ARG;
        // Outputs that their layer accumulates into with atomics have to be zero beforehand.  All
        // pointers of the pass are known here, so those outputs are zeroed by one launch up front
        // instead of one launch each -- but only an output that overlaps nothing an earlier layer
        // of the pass reads or writes, nor its own layer's inputs; the others are zeroed right
        // before their layer as usual.
        auto overlaps = [](const float *p, int64_t n, const float *q, int64_t m) {
            return p && q && (uintptr_t)p < (uintptr_t)(q + m) && (uintptr_t)q < (uintptr_t)(p + n);
        };
        std::vector<char> ahead(nl, 0);
        ZeroList z;
        z.count = 0;
        z.first[0] = 0;
        hipStream_t st = (hipStream_t)stream;
        auto flush = [&]() -> int {
            if (z.count == 0) return WPK_OK;
            hipLaunchKernelGGL(zero_many_kernel, dim3(z.first[z.count]), dim3(256), 0, st, z);
            z.count = 0;
            WPK_HIP(hipGetLastError());
            return WPK_OK;
        };
        for (size_t j = 0; j < nl; ++j) {
            const wpk_plan::Layer &L = plan->layers[j];
            const wpk_conv_config &cfg = L.config(-1, L.epilogue(residual ? residual[j] : nullptr));
            if (L.direct || !zeroes_all_of_y(L.pr, cfg, &plan->fix)) continue;
            const int64_t ny = L.pr.y_elems;
            bool ok = !overlaps(y[j], ny, x[j], L.pr.x_elems) &&
                      !(residual && overlaps(y[j], ny, residual[j], ny));
            for (size_t i = 0; i < j && ok; ++i) {
                const Problem &pi = plan->layers[i].pr;
                ok = !overlaps(y[j], ny, x[i], pi.x_elems) && !overlaps(y[j], ny, y[i], pi.y_elems) &&
                     !(residual && overlaps(y[j], ny, residual[i], pi.y_elems));
            }
            if (!ok) continue;
            ahead[j] = 1;
            z.p[z.count] = y[j];
            z.n[z.count] = ny;
            z.first[z.count + 1] = z.first[z.count] + (int)std::max<int64_t>(1, (ny / 4 + 1023) / 1024);
            if (++z.count == kZeroListMax) {
                int rc = flush();
                if (rc != WPK_OK) return rc;
            }
        }
        int rc = flush();
        for (size_t i = 0; i < nl && rc == WPK_OK; ++i)
            rc = plan_launch(plan, plan->layers[i], -1, x[i], residual ? residual[i] : nullptr, y[i], st,
                             ahead[i] != 0);
        return rc;
    }
    // two chains of half-batches: one on the caller's stream, one on the plan's, forked and
    // joined once around the whole pass
    for (size_t i = 0; i < plan->layers.size(); ++i)
        if (!x[i] || !y[i]) return WPK_E_NULL_PTR;
        else if (!plan->layers[i].has_w) return WPK_E_BAD_ARG;
    int rc = plan_fork(plan, (hipStream_t)stream);
    for (size_t i = 0; i < plan->layers.size() && rc == WPK_OK; ++i) {
        const float *r = residual ? residual[i] : nullptr;
        rc = plan_launch(plan, plan->layers[i], 0, x[i], r, y[i], (hipStream_t)stream);
        if (rc == WPK_OK) rc = plan_launch(plan, plan->layers[i], 1, x[i], r, y[i], plan->side);
    }
    int rj = plan_join(plan, (hipStream_t)stream);  // joined even after a failed launch
    return rc != WPK_OK ? rc : rj;
}

int wpk_plan_run(wpk_plan *plan, const float *const *x, float *const *y, void *stream)
{
    return wpk_plan_run_fused(plan, x, nullptr, y, stream);
}

int wpk_plan_num_layers(const wpk_plan *plan) { return plan ? (int)plan->layers.size() : WPK_E_NULL_PTR; }
int wpk_plan_num_unique(const wpk_plan *plan) { return plan ? (int)plan->ktabs.size() : WPK_E_NULL_PTR; }

int wpk_plan_layer_config(const wpk_plan *plan, int32_t layer, wpk_conv_config *out)
{
    if (!plan || !out) return WPK_E_NULL_PTR;
    if (layer < 0 || layer >= (int)plan->layers.size()) return WPK_E_BAD_ARG;
    const wpk_plan::Layer &L = plan->layers[layer];
    *out = L.config(-1, L.epilogue(nullptr));
    return WPK_OK;
}

int wpk_plan_set_layer_config(wpk_plan *plan, int32_t layer, const wpk_conv_config *cfg)
{
    if (!plan || !cfg) return WPK_E_NULL_PTR;
    if (layer < 0 || layer >= (int)plan->layers.size()) return WPK_E_BAD_ARG;
    if (plan->layers[layer].direct || !legal_for(plan->layers[layer].pr, *cfg)) return WPK_E_NO_CONFIG;
    int rw = plan_need_weights(plan->layers[layer], *cfg);
    if (rw != WPK_OK) return rw;
    FixupNeed need = fixup_need(plan->layers[layer].pr, *cfg, g_cus);
    if (need.bytes > (int64_t)plan->fix.bytes) {
        WPK_HIP(hipDeviceSynchronize());  // the old workspace may still be in use
        int rc = fixup_reserve(plan->fix, (size_t)need.bytes);
        if (rc != WPK_OK) return rc;
    }
    plan->layers[layer].cfg = plan->layers[layer].cfg_fused = *cfg;
    // the half-batch launches of a pipelined plan follow, where the configuration is legal for them
    if (plan->side) {
        wpk_plan::Layer &L = plan->layers[layer];
        for (int h = 0; h < 2; ++h) {
            if (!legal_for(L.half[h], *cfg)) continue;
            FixupNeed nh = fixup_need(L.half[h], *cfg, g_cus);
            FixupBuf &fb = h == 0 ? plan->fix : plan->fix_side;
            if (nh.bytes > (int64_t)fb.bytes) {
                WPK_HIP(hipDeviceSynchronize());
                int rc = fixup_reserve(fb, (size_t)nh.bytes);
                if (rc != WPK_OK) return rc;
            }
            L.half_cfg[h] = L.half_cfg_fused[h] = *cfg;
        }
    }
    return WPK_OK;
}

void wpk_plan_destroy(wpk_plan *plan)
{
    if (!plan) return;
    for (auto &L : plan->layers) {
        for (float *p : L.wp)
            if (p) (void)hipFree(p);
        if (L.bias) (void)hipFree(L.bias);
    }
    for (int32_t *t : plan->ktabs)
        if (t) (void)hipFree(t);
    fixup_release(plan->fix);
    fixup_release(plan->fix_side);
    if (plan->fork) (void)hipEventDestroy(plan->fork);
    if (plan->join) (void)hipEventDestroy(plan->join);
    if (plan->side) (void)hipStreamDestroy(plan->side);
    delete plan;
}

}  // extern "C"
