// The strip form of the split members: layers of few input channels (the 3-channel stem of a network), whose reduction has
// too few channels to be cut into groups of 32, or even 16, of them.
//
// Rows of the reduction are ordered (c, r, s) with s padded to eight: an octet is the filter row r of channel c, and a lane's
// octet of a pixel is eight neighbouring columns of one row of x.  The rows of x under a strip of output rows are fetched, split
// into three bf16 parts and put into LDS once (the other forms split each of them R * S / (stride * stride) times over), two
// columns to a dword: [channel, row][part][columns / 2].  With an even stride every octet begins at a dword and is read as four of
// them; with an odd one every second begins in the middle of one and is shifted out of five.
//
// Workgroup.  Four waves, all of which fill the strip and then multiply, 32 channels each; the weights of those, the whole reduction
// of C * R octets at most 22, stay in registers (132 for 22 octets) while the wave goes through its pixels in blocks of 32, so that the loop
// asks memory for nothing.  Two workgroups per compute unit.  What bounds it: the six MFMAs of a depth take 192 cycles, the wave's other
// instructions (six LDS reads of two dwords for an even stride) 60; the strip's filling is not overlapped within a workgroup.
// 7x7, stride 2, 3 -> 64 channels, 224x224, 16 images: 28.4 to 30.5 us by the device's clock, the tiled members 44.2 to 44.9 (row by row on the
// split members 47.5).  Of 43300 cycles of a workgroup (median; up to 59100 beside another) 12800 are the start and the strip, 4000 to 4400 each of
// seven blocks (up to 8000 beside another; 2112 of MFMAs, 1350 the way out); the matrix pipes are busy 47 % of a compute unit's time, no bank conflicts.
#ifndef WPK_STRIP_H
#define WPK_STRIP_H

#include "wpk_split.h"

namespace wpk {

// The launch's own numbers, behind the common ones.
struct StripGeom {
    int32_t rows;        // output rows of a strip
    int32_t per_image;   // strips of an image
    int32_t strips;      // of all images
    int32_t P;
    int32_t groups;      // groups of 32 * waves_c channels, of which a workgroup does `per_group`
    int32_t per_group;
    int32_t waves_c;     // waves side by side along the channels: 1, 2 or 4
    int32_t in_rows;     // rows of x under a strip, of each channel
    int32_t inv_r;       // 65536 / R, rounded up: o * inv_r >> 16 is o / R for o < 32
    FastDiv div_strips, div_image, div_rows;
};

constexpr int kStripLds = 78 * 1024;  // two workgroups per compute unit

// DEPTHS: MFMA depths of two octets; PAIRS: columns / 2 of a row of the strip; ODD: the stride along the row is odd.
template <int DEPTHS, int PAIRS, bool ODD>
__global__ void __launch_bounds__(256, 2) strip_kernel(const IgemmArgs a, const StripGeom g)
{
    constexpr int KP = (PAIRS + 63) / 64;      // pairs of a row per lane
    constexpr int BATCH = KP == 1 ? 16 : 10;   // rows a wave fetches at a time
    constexpr int LINE = 3 * PAIRS * 4;        // bytes of a row of x
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ __attribute__((aligned(16))) float bias[4][32];
    const int lane = threadIdx.x & 63, lrow = lane >> 5, lcol = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int part = fdiv(id, g.div_strips), strip = id - part * g.strips;
    const int n = fdiv(strip, g.div_image), p0 = (strip - n * g.per_image) * g.rows;
    const int rows = min(g.rows, g.P - p0), count = rows * a.Q;  // output rows and pixels of this strip
    const int m0 = n * a.PQ + p0 * a.Q;
    const int in_rows = g.in_rows, lines = a.C * in_rows;  // rows of x (of a whole strip's, in the last one of an image too)

    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.wp, 0, (int)a.w_bytes, 0x00020000);

    // ---- a wave's weights and bias: asked for ahead of the strip, and again for every further group of channels -------------
    const int wc = wave & (g.waves_c - 1), first = wave / g.waves_c, step = 4 / g.waves_c;
    const int group_end = min(g.groups, (part + 1) * g.per_group);
    int grp = part * g.per_group, n0 = (grp * g.waves_c + wc) * 32;
    const unsigned depth_bytes = (unsigned)(a.Kpad / 32) * 3072u;
    v8bf w[DEPTHS * 3];
    float bval;
    auto fetch_weights = [&]() WPK_LAMBDA {
        const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(a.bias ? a.bias : a.x), 0, a.bias ? a.K * 4 : 0, 0x00020000);
        bval = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(brsrc, (n0 + lcol) * 4, 0, 0));
        static_for<DEPTHS * 3>([&](auto I) WPK_LAMBDA {
            constexpr int i = decltype(I)::value;
            w[i] = __builtin_bit_cast(v8bf, __builtin_amdgcn_raw_buffer_load_b128(
                                                wrsrc, lane * 16, n0 / 32 * 3072 + i / 3 * depth_bytes + i % 3 * 1024, 0));
        });
    };

    // where the lane's octet of every depth begins in the strip (past the last one: at the first, with weights of zero)
    int oct[DEPTHS];
    static_for<DEPTHS>([&](auto D) WPK_LAMBDA {
        const int o = 2 * decltype(D)::value + lrow, c = o * g.inv_r >> 16, r = o - c * a.R;
        oct[decltype(D)::value] = c < a.C ? (c * g.in_rows + r * a.dil_h) * LINE : 0;
    });

    // ---- the strip ------------------------------------------------------------------------------------------
    {
        const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, (int)a.x_bytes, 0x00020000);
        const int px4 = a.xl ? a.C * 4 : 4;    // bytes between neighbouring pixels of x
        int col[KP][2];                        // byte offset of the lane's columns, all ones outside the image
        static_for<KP * 2>([&](auto I) WPK_LAMBDA {
            constexpr int k = decltype(I)::value / 2, h = decltype(I)::value % 2;
            const int iw = 2 * (lane + 64 * k) + h - a.pad_w;
            col[k][h] = (unsigned)iw < (unsigned)a.W ? iw * px4 : -1;
        });
        int l0 = wave;
        do {
            float v[BATCH][KP][2];
            static_for<BATCH>([&](auto B) WPK_LAMBDA {
                constexpr int b = decltype(B)::value;
                const int line = l0 + 4 * b;
                const int c = fdiv(line, g.div_rows), ih = p0 * a.stride_h - a.pad_h + line - c * in_rows;
                const int out = line < lines && (unsigned)ih < (unsigned)a.H ? 0 : -1;
                // (a row outside the image has all its lanes past the tensor: its own offset must not matter)
                const int at = (n * a.C * a.HW + (a.xl ? ih * a.W * a.C + c : c * a.HW + ih * a.W)) * 4 & ~out;
                static_for<KP * 2>([&](auto I) WPK_LAMBDA {
                    constexpr int k = decltype(I)::value / 2, h = decltype(I)::value % 2;
                    v[b][k][h] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src, col[k][h] | out, at, 0));
                });
            });
            __builtin_amdgcn_sched_barrier(0);
            if (l0 == wave) fetch_weights();
            __builtin_amdgcn_sched_barrier(0);
            static_for<BATCH * KP>([&](auto I) WPK_LAMBDA {
                constexpr int b = decltype(I)::value / KP, k = decltype(I)::value % KP;
                const float v0 = v[b][k][0] * kOperandScale, v1 = v[b][k][1] * kOperandScale;
                const unsigned h = pack_bf16(v0, v1);
                const float r0 = v0 - bf16_low(h), r1 = v1 - bf16_high(h);
                const unsigned m = pack_bf16(r0, r1);
                const unsigned l = pack_bf16(r0 - bf16_low(m), r1 - bf16_high(m));
                const int line = l0 + 4 * b, pair = lane + 64 * k;
                if (line < lines && pair < PAIRS) {
                    unsigned *const p = reinterpret_cast<unsigned *>(lds + line * LINE) + pair;
                    p[0] = h;
                    p[PAIRS] = m;
                    p[2 * PAIRS] = l;
                }
            });
        } while ((l0 += 4 * BATCH) < lines);
    }
    __syncthreads();

    const int blocks = (count + 31) / 32;
    for (;;) {
        if (n0 >= a.K) break;
        if (lane < 32) bias[wave][lane] = bval;
        for (int b = first; b < blocks; b += step) {
            const int t = min(b * 32 + lcol, count - 1);
            const int pr = fdiv(t, a.div_q), q = (t - pr * a.Q) * a.stride_w;
            const int base = pr * a.stride_h * LINE + (q >> 1) * 4;
            const unsigned shift = ODD ? (q & 1) * 16 : 0;
            v4u x[3];  // the three parts of a depth, each read anew as soon as its last MFMA has been issued
            auto read = [&](auto D, auto PART) WPK_LAMBDA {
                constexpr int d = decltype(D)::value, part = decltype(PART)::value;
                if constexpr (d < DEPTHS) {
                    const unsigned *const p = reinterpret_cast<const unsigned *>(lds + (base + oct[d])) + part * PAIRS;
                    if constexpr (ODD) {
                        unsigned e[5];
                        static_for<5>([&](auto E) WPK_LAMBDA { e[decltype(E)::value] = p[decltype(E)::value]; });
                        static_for<4>([&](auto E) WPK_LAMBDA {
                            constexpr int i = decltype(E)::value;
                            x[part][i] = __builtin_amdgcn_alignbit(e[i + 1], e[i], shift);
                        });
                    } else {
                        static_for<4>([&](auto E) WPK_LAMBDA { x[part][decltype(E)::value] = p[decltype(E)::value]; });
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // (the small terms in two sums that take turns: an MFMA that adds to the one before it takes 48 cycles, not 32)
            v16f acc[1], sml[2];
            static_for<16>([&](auto E) WPK_LAMBDA {
                acc[0][decltype(E)::value] = 0.0f;
                sml[0][decltype(E)::value] = 0.0f;
                sml[1][decltype(E)::value] = 0.0f;
            });
            using H = std::integral_constant<int, 0>;
            using M = std::integral_constant<int, 1>;
            using L = std::integral_constant<int, 2>;
            static_for<3>([&](auto P) WPK_LAMBDA { read(std::integral_constant<int, 0>{}, std::integral_constant<int, 2 - decltype(P)::value>{}); });
            static_for<DEPTHS>([&](auto D) WPK_LAMBDA {
                constexpr int d = decltype(D)::value, e = d % 2, f = 1 - e;
                using NEXT = std::integral_constant<int, d + 1>;
                auto part = [&](auto P) WPK_LAMBDA { return __builtin_bit_cast(v8bf, x[decltype(P)::value]); };
                sml[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[d * 3], part(L{}), sml[e], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                read(NEXT{}, L{});
                sml[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[d * 3 + 1], part(M{}), sml[f], 0, 0, 0);
                sml[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[d * 3], part(M{}), sml[e], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                read(NEXT{}, M{});
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[d * 3], part(H{}), acc[0], 0, 0, 0);
                sml[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[d * 3 + 1], part(H{}), sml[f], 0, 0, 0);
                sml[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[d * 3 + 2], part(H{}), sml[e], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                read(NEXT{}, H{});
            });
            static_for<16>([&](auto E) WPK_LAMBDA { sml[0][decltype(E)::value] += sml[1][decltype(E)::value]; });
            v16f(&small)[1] = *reinterpret_cast<v16f(*)[1]>(&sml[0]);
            if (join_sums(acc, small)) {
                const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)((const char *)a.x - a.x_bias), 0, (int)(a.x_bytes + a.x_bias), 0x00020000);
                fp32_tile<kStrip, 1, 1>(acc, xrsrc, wrsrc, m0 + b * 32, n0 / 32 * 3072u, DEPTHS, [](int i) WPK_LAMBDA { return i; }, lane);
            }
            store_wave_tile<1, 1, 1>(&a, acc, m0 + b * 32, n0, lrow, lcol, false, bias[wave], m0 + count);
        }
        if (++grp >= group_end) break;
        n0 += 32 * g.waves_c;
        fetch_weights();
    }
}

template <int DEPTHS, int PAIRS, bool ODD>
hipError_t launch_strip_form(const IgemmArgs &a, const StripGeom &g, size_t bytes, hipStream_t stream)
{
    if (bytes > 64 * 1024) {  // (the runtime's default limit per launch)
        hipError_t e = hipFuncSetAttribute((const void *)strip_kernel<DEPTHS, PAIRS, ODD>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kStripLds);
        if (e != hipSuccess) return e;
    }
    const int parts = (g.groups + g.per_group - 1) / g.per_group;
    hipLaunchKernelGGL((strip_kernel<DEPTHS, PAIRS, ODD>), dim3((unsigned)(g.strips * parts)), dim3(256), bytes, stream, a, g);
    return hipGetLastError();
}

template <int DEPTHS, int PAIRS>
hipError_t launch_strip_odd(const IgemmArgs &a, const StripGeom &g, size_t bytes, hipStream_t stream)
{
    return a.stride_w % 2 ? launch_strip_form<DEPTHS, PAIRS, true>(a, g, bytes, stream)
                          : launch_strip_form<DEPTHS, PAIRS, false>(a, g, bytes, stream);
}

// s: the layer's, from strip_shape.
hipError_t launch_strip(const IgemmArgs &a, const StripShape &s, hipStream_t stream)
{
    StripGeom g;
    g.P = a.PQ / a.Q;
    g.rows = s.rows;
    g.per_image = (g.P + s.rows - 1) / s.rows;
    g.strips = a.N * g.per_image;
    g.waves_c = s.waves_c;
    g.groups = (a.K + 32 * s.waves_c - 1) / (32 * s.waves_c);
    g.per_group = s.per_group;
    g.in_rows = (s.rows - 1) * a.stride_h + (a.R - 1) * a.dil_h + 1;
    g.inv_r = 65536 / a.R + 1;
    g.div_rows = make_fastdiv((uint32_t)g.in_rows);
    g.div_strips = make_fastdiv((uint32_t)g.strips);
    g.div_image = make_fastdiv((uint32_t)g.per_image);
    const size_t bytes = (size_t)s.lds;
    if (s.pairs == 64) {
        if (s.depths == 3) return launch_strip_odd<3, 64>(a, g, bytes, stream);
        if (s.depths == 5) return launch_strip_odd<5, 64>(a, g, bytes, stream);
        if (s.depths == 8) return launch_strip_odd<8, 64>(a, g, bytes, stream);
        return launch_strip_odd<11, 64>(a, g, bytes, stream);
    }
    if (s.depths == 3) return launch_strip_odd<3, 120>(a, g, bytes, stream);
    if (s.depths == 5) return launch_strip_odd<5, 120>(a, g, bytes, stream);
    if (s.depths == 8) return launch_strip_odd<8, 120>(a, g, bytes, stream);
    return launch_strip_odd<11, 120>(a, g, bytes, stream);
}

}  // namespace wpk
#endif
