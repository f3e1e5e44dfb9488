// The split members of the convolution kernel family for gfx950: fp32 products formed on the bf16 matrix
// pipes, which multiply sixteen times as fast as the fp32 ones.
//
// Arithmetic.  An fp32 number is the exact sum of three bf16 numbers, v = h + m + l: h is v rounded to
// bf16 (8 significant bits), m what is left of v rounded to bf16, l the rest (24 = 8 + 8 + 8 bits).  A
// product of two such sums has nine terms; the six of them down to 2^-17 of the product,
//     hh,  hm + mh + mm + hl + lh,
// are formed by v_mfma_f32_32x32x16_bf16 (bf16 products are exact in fp32) and the other three, below
// 2^-25 each, are dropped.  hh accumulates in one set of registers and the five small terms in another,
// added once at the end: the running sum of hh is rounded once per sixteen terms of the reduction
// instead of once per term, and the small terms are rounded at a 256th of its size, so the result is
// closer to the exact sum than fp32 FMAs bring it (2-norm of the error over 2-norm of the result, normal operands:
// 3.5e-7 against 8.6e-7 at 4608 terms, 1.1e-7 against 3.1e-7 at 576, 4.2e-8 against 1.1e-7 at 64; with
// all six in one accumulator 1.0e-6, 3.5e-7, 1.1e-7).  Six MFMAs of 32 cycles per 32 x 32 block and
// sixteen rows of the reduction stand against eight fp32 ones of 64.
//
// Both operands are split 2^16 times as large as they are, which makes every one below 2^111 three bf16 numbers exactly, however
// small (one more vector instruction per activation).  Weights above that are packed whole beside a NaN (split_weight); an activation
// above that, or infinite, leaves NaN in m or l (inf - inf): both show in the accumulators, as do sums above 2^95, scaled, and
// infinities or NaN that fp32 sums would give too.  A wave that finds a sum not finite computes its tile again with fp32 MFMAs
// (fp32_tile below) from the same operands.
//
// Workgroup.  64 pixels x 32 WN channels.  WN waves multiply, each all 64 pixels by 32 channels of its own: every
// weight is wanted by one wave only and goes from memory straight into the registers the MFMAs read; it is
// packed for that (pack_split_kernel), already split, 16 bytes per lane.  Activations are shared by the waves: NP further
// waves fetch them as fp32, split them once and put them into LDS, from where a lane of a multiplying wave
// reads eight consecutive rows of its pixel per part with one 16-byte access.  Two buffers, one barrier per step.
// NP: a wave issues an instruction every five cycles, so splitting a step of 64 pixels and 32 rows, 250 of them, takes it 1570 cycles,
// in which two multiplying waves of a SIMD are done with theirs (1536), but one has waited half of the time.  So two waves fetch
// where a compute unit has few workgroups, each half of every step (in turns they gain nothing: with two buffers a step is split
// while the one before it is multiplied), and one where it has four (split_producers).
// Why waves of their own for it: (a) loads return in order, so in a wave that fetches both, a weight waits for
// every activation asked for before it, however far ahead that was -- with both in one wave a 1x1 layer of 256
// channels at 56x56 (N = 16, K = 128) ran at 2.2 TB/s whatever the depth of its prefetch; (b) the splitting (6.5 vector
// instructions per element) and the address arithmetic leave the waves that multiply with 2.5 instructions per MFMA,
// and one such wave per SIMD keeps the matrix pipes busy within the loop (28-31 % of a whole launch's cycles on the batched 3x3
// layers, counters).  What bounds the loop then is power: with random operands
// back-to-back bf16 MFMAs hold the clock at 1.75-1.85 GHz (2.3 with zeros), 17.7 ns each instead of 13.3.
// Registers are held to 168, three waves per SIMD: the accumulators are 64 of them.
#ifndef WPK_SPLIT_H
#define WPK_SPLIT_H

#include "wpk_igemm.h"

namespace wpk {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// two floats rounded to nearest even, packed: a in the low half
__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    const v2f v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, v2bf));
}
__device__ __forceinline__ float bf16_low(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_high(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// Operands are split 2^16 times as large as they are, so that the smallest fp32 number, 2^-149, is the smallest bf16
// one, 2^-133, and every operand below 2^111 is exactly three bf16 numbers; the sums are scaled back by join_sums.
constexpr float kOperandScale = 0x1p16f, kSumScale = 0x1p-32f;
// The parts of a weight as bf16 bits: the scaled weight rounded to bf16, the remainder rounded to bf16, the rest.  A weight that
// would round to infinity so, an infinity or NaN has NaN as its first part, which shows in every sum it enters, and its own
// bits in the other two.
__device__ __forceinline__ void split_weight(const float w, unsigned (&part)[3])
{
    const float v = w * kOperandScale;
    const unsigned h = pack_bf16(v, 0.0f) & 0xffffu;
    const float r = v - bf16_low(h);
    const unsigned m = pack_bf16(r, 0.0f) & 0xffffu, l = pack_bf16(r - bf16_low(m), 0.0f) & 0xffffu;
    const unsigned bits = __builtin_bit_cast(unsigned, w);
    const bool whole = (h & 0x7f80u) == 0x7f80u;
    part[0] = whole ? 0x7fffu : h;
    part[1] = whole ? bits >> 16 : m;
    part[2] = whole ? bits & 0xffffu : l;
}
// The weight again, exactly.
__device__ __forceinline__ float join_weight(const unsigned h, const unsigned m, const unsigned l)
{
    // (all ones where the exponent is; masks, since a select becomes a branch in the kernel)
    const unsigned whole = (unsigned)__builtin_amdgcn_sbfe((int)((h & 0x7f80u) + 0x80u), 15, 1);
    const float sum = ((bf16_low(l) + bf16_low(m)) + bf16_low(h)) * (1.0f / kOperandScale);
    return __builtin_bit_cast(float, (whole & (m << 16 | l)) | (~whole & __builtin_bit_cast(unsigned, sum)));
}

// eight activations as their three bf16 parts, sixteen bytes each
__device__ __forceinline__ void split_octet(const float (&v)[8], v4u &h, v4u &m, v4u &l)
{
    static_for<4>([&](auto P) WPK_LAMBDA {
        constexpr int p = decltype(P)::value;
        const float v0 = v[2 * p] * kOperandScale, v1 = v[2 * p + 1] * kOperandScale;
        const unsigned ph = pack_bf16(v0, v1);
        const float r0 = v0 - bf16_low(ph), r1 = v1 - bf16_high(ph);
        const unsigned pm = pack_bf16(r0, r1);
        h[p] = ph;
        m[p] = pm;
        l[p] = pack_bf16(r0 - bf16_low(pm), r1 - bf16_high(pm));
    });
}

// The two sums of every output become one; true if the split was not able to hold this wave's tile.
template <int NB>
__device__ __forceinline__ bool join_sums(v16f (&acc)[NB], const v16f (&sml)[NB])
{
    unsigned top = 0;
    static_for<NB>([&](auto I) WPK_LAMBDA {
        static_for<16>([&](auto E) WPK_LAMBDA {
            constexpr int i = decltype(I)::value, e = decltype(E)::value;
            const float v = acc[i][e] + sml[i][e];
            top = max(top, __builtin_bit_cast(unsigned, v) & 0x7fffffffu);
            acc[i][e] = v * kSumScale;
        });
    });
    return __builtin_amdgcn_ballot_w64(top >= 0x7f800000u) != 0;  // inf or NaN
}

// How activations are found (the XL of the tiled members, and the patch):
//   kRows   row by row through the tap table, any C; rows in the source's order (c, r, s)
//   kQuads  channels-last, C padded to 32: a lane fetches an octet of one pixel with two 16-byte loads
//   kTaps   [N][C][H][W], C padded to 32: one filter tap per step, eight one-dword loads per octet
//   kPoint  [N][C][H][W], C padded to 32, 1x1 filters, stride 1, no padding, H * W a multiple of 4: four neighbouring pixels of a
//           channel are sixteen contiguous bytes, so a wave fetches a whole step with eight loads instead of 32
//   kPatch, kPatchQuads: 3x3 filters (C padded to 16): the nine taps of sixteen channels read one patch of x.  The pixels of a
//           tile are consecutive, and so are the positions of x that their windows cover (numbered through the
//           images): `halo` of them at most, any stride and dilation for which that fits.  A position is fetched and
//           split once per sixteen channels instead of nine times.  A multiplying wave knows the LDS address of every
//           tap of its pixels from the start; a tap outside the image has the address of a row of zeros.
// Rows of the reduction are ordered (c / 32, r, s, c % 32) but for kRows, so that the taps of 32 channels follow each
// other and find their pixels in the L1; a step is 32 rows, for patches the nine taps of sixteen channels.
enum SplitForm { kStrip, kRows, kQuads, kTaps, kPoint, kPatch, kPatchQuads };  // (kStrip: wpk_strip.h)
// The wave's blocks again, in fp32, over the MFMA depths depth(0 .. count - 1), with the operands where a lane's eight rows of a
// depth are: MFMA number q of eight contracts rows q and 8 + q.  Bound by the 16 MFMAs of 64 cycles and some 240 other instructions
// of a depth, without branches (masks instead of selects) and with the next two depths' operands on their way.  A launch with
// one infinity in x takes 86 us on the 256-channel 3x3 layer at 14x14 (N = 16; 24 without one) and 51 on the 64-channel
// one at 56x56 (24); with branches and one depth after the other 232 and 125.  The tiled members take 40 and 42 on any data.
template <SplitForm FORM, int NMT, int DEPTH = 2, class D>
__device__ __forceinline__ void fp32_tile(v16f (&acc)[NMT], const __amdgpu_buffer_rsrc_t xrsrc,
                                          const __amdgpu_buffer_rsrc_t wrsrc, const int m0, const unsigned wbase,
                                          const int count, D &&depth, const int lane)
{
    constexpr bool PATCH = FORM == kPatch || FORM == kPatchQuads;
    const cold_ptr c = cold_args();
    const int lrow = lane >> 5, lcol = lane & 31;
    const unsigned wblk_bytes = (unsigned)(c->Kpad / 32) * 3072u;
    const int px4 = c->xl == 1 || c->xl == 2 ? c->C * 4 : 4;
    int voff[NMT];
    unsigned inv[NMT];
    static_for<NMT>([&](auto J) WPK_LAMBDA {
        constexpr int j = decltype(J)::value;
        pixel_window(c, m0 + j * 32 + lcol, voff[j], inv[j]);
        static_for<16>([&](auto E) WPK_LAMBDA { acc[j][decltype(E)::value] = 0.0f; });
    });
    float xv[DEPTH][NMT][8];  // (DEPTH: depths in flight)
    v4u wv[DEPTH][3];
    auto fetch = [&](auto SET, const int it) WPK_LAMBDA {
        constexpr int set = decltype(SET)::value;
        const int t = depth(min(it, count - 1));
        static_for<3>([&](auto Q) WPK_LAMBDA {
            wv[set][decltype(Q)::value] = __builtin_amdgcn_raw_buffer_load_b128(
                wrsrc, lane * 16, wbase + (unsigned)t * wblk_bytes + decltype(Q)::value * 1024, 0);
        });
        static_for<8>([&](auto Q) WPK_LAMBDA {
            constexpr int q = decltype(Q)::value;
            int ch, rs, past;  // past: all ones beyond the last row
            if constexpr (FORM == kRows) {  // rows in the source's order (c, r, s)
                const int kk = t * 16 + lrow * 8 + q;
                ch = fdiv(kk, WPK_COLD_DIV(c, div_tap));
                rs = kk - ch * c->RS;
                past = (c->CRS - 1 - kk) >> 31;
            } else if constexpr (FORM == kStrip) {  // (c, r, s), s padded to eight
                const int o = t * 2 + lrow;
                past = (c->C * c->R - 1 - o) >> 31 | (c->S - 1 - q) >> 31;
                ch = o / c->R;
                rs = ((o - ch * c->R) * c->S + q) & ~past;
                ch &= ~past;
            } else {                        // (c / 32, r, s, c % 32)
                const int c32 = PATCH ? t / 18 : fdiv(t >> 1, WPK_COLD_DIV(c, div_tap));
                rs = (t >> 1) - c32 * c->RS;
                ch = c32 * 32 + (t & 1) * 16 + lrow * 8 + q;
                past = (c->C - 1 - ch) >> 31;
            }
            const int fr = fdiv(rs, WPK_COLD_DIV(c, div_s)), fs = rs - fr * c->S;
            const int at = (fr * c->dil_h * c->W + fs * c->dil_w) * px4 + ch * c->HW4;
            static_for<NMT>([&](auto J) WPK_LAMBDA {
                constexpr int j = decltype(J)::value;
                const int out = past | __builtin_amdgcn_sbfe((int)inv[j], fr, 1) |
                                __builtin_amdgcn_sbfe((int)inv[j], 16 + fs, 1);
                xv[set][j][q] =
                    __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, (voff[j] + at) | out, 0, 0));
            });
        });
    };
    auto multiply = [&](auto SET) WPK_LAMBDA {
        constexpr int set = decltype(SET)::value;
        static_for<8>([&](auto Q) WPK_LAMBDA {
            constexpr int q = decltype(Q)::value, sh = q % 2 * 16;
            const float w = join_weight(wv[set][0][q / 2] >> sh & 0xffffu, wv[set][1][q / 2] >> sh & 0xffffu,
                                        wv[set][2][q / 2] >> sh & 0xffffu);
            static_for<NMT>([&](auto J) WPK_LAMBDA {
                constexpr int j = decltype(J)::value;
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, xv[set][j][q], acc[j], 0, 0, 0);
            });
        });
    };
    static_for<DEPTH>([&](auto S) WPK_LAMBDA { fetch(S, decltype(S)::value); });
    constexpr int LAPS = DEPTH == 1 ? 1 : 4;
    int it = 0;
    auto one = [&](auto P) WPK_LAMBDA {
        constexpr int p = decltype(P)::value;
        using SET = std::integral_constant<int, p % DEPTH>;
        if (it + p >= count) return false;
        multiply(SET{});
        fetch(SET{}, it + p + DEPTH);
        __builtin_amdgcn_sched_barrier(0);
        return true;
    };
    while (static_all<LAPS>(one)) it += LAPS;
}

constexpr int kHaloPitch = 112;    // LDS bytes per position of a patch: one depth of 3 parts x 32 bytes, 16 of padding, and
constexpr int kStepPitch = 240;    // per pixel of a step: two depths, 48 of padding, of which a pixel's rows
                                   // are moved on by 16 for every 16 pixels.  Both put the 16 lanes served at a time
                                   // on 16 different groups of four banks, whether they hold neighbouring pixels or
                                   // every fourth.  Where a tile's pixels run over rows of the image they do not: cycles
                                   // lost to bank conflicts over cycles of LDS instructions 0.10 at 56x56, 0.28 at 28x28,
                                   // 0.39 at 14x14, 0.44 at 7x7 (waves wait for LDS 2 % of their time).
__host__ __device__ constexpr int step_place(int px) { return px * kStepPitch + (px >> 4) * 16; }
// What a wave of a workgroup does: 0 .. WN - 1 multiply, the others fetch.
// A compute unit deals the waves of a workgroup to its four SIMDs in turn and begins the next workgroup one SIMD further on (read
// from HW_ID, workgroups of three, four and six waves).  So of two workgroups with two multiplying waves each, the first ones, one
// SIMD would have two of them and another none, and the loop takes twice as long as it could; the second workgroup of a
// compute unit has waves 1 and 2 multiply instead.  (Workgroups of two waves set by hand, which no default chose before: 3x3, 128 channels, 28x28,
// 16 images, 392 workgroups, 22.7 us, 29.7 without; 256 channels, 14x14 in two slices 24.8, 32.0; 1x1, 512 to 128 channels at 28x28 16.1, 19.0.
// The defaults of these three then took 21.4, 24.1 and 16.3.)  With three or four workgroups on a
// compute unit the SIMDs have as much to do either way, and asking costs 0.4 us (64 channels, 56x56: 22.5, 22.9 with): not done there.
// Nor where a single wave fetches, but for patches: 1x1 layers took 17.4 either way, channels-last ones 4 to 9 % longer with
// it (55 layers of one or two workgroups per compute unit; 5x5, 640 to 64 channels, 17x45, 8 images, 90.1 us, 83.5 without).
template <int WN, int NP, bool CHANGE, class F>
__device__ __forceinline__ int role_of_wave(const int wave, F &&two_per_unit)
{
    if constexpr (!CHANGE) return wave;
    if (!two_per_unit()) return wave;
    // (the second workgroup's LDS begins where the first one's ends; LDS_ALLOC: base in bits 0 .. 8, size in bits 12 .. 20)
    const unsigned alloc = __builtin_amdgcn_s_getreg(6 | 31 << 11);
    if ((alloc & 0x1ff) != (alloc >> 12 & 0x1ff)) return wave;
    return wave == 0 ? WN + NP - 1 : wave - 1;
}

// ANY: C may be no multiple of 32 (of 16 for kPatchQuads).  What is fetched for the channels that fill the last group up has weights of
// zero: kTaps and kPatch fetch the last channel again, the others what lies behind it, the next pixel or image, or zeros
// past the tensor, whose end the range check knows only where the whole offset is the lane's.
template <int WN, SplitForm FORM, int NP, bool ANY>
__global__ void __launch_bounds__(64 * (WN + NP), 3) split_kernel(const IgemmArgs a)
{
    constexpr bool PATCH = FORM == kPatch || FORM == kPatchQuads, QUAD = FORM == kQuads || FORM == kPatchQuads;
    constexpr int BM = 64, BN = 32 * WN, NMT = 2, T = 64 * WN;
    constexpr int NT = PATCH ? 9 : 2;          // MFMA depths (of 16 rows) per step
    extern __shared__ __attribute__((aligned(16))) char lds[];  // two steps of activations
    __shared__ __attribute__((aligned(16))) float bias[2][BN];  // of this segment's channels and of the one before
    __shared__ int arrival;

    touch_kernarg_lines();
    const int wave = role_of_wave<WN, NP, WN == 2 && (PATCH || NP == 2)>(
        __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), [&] { return a.two_per_unit != 0; });
    const int tid = wave * 64 + (threadIdx.x & 63);
    const int buf_bytes = PATCH ? (a.halo + 1) * kHaloPitch : BM * kStepPitch;
    int parity = 0;                            // of the segment

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const char *)a.x - a.x_bias), 0, (int)(a.x_bytes + a.x_bias), 0x00020000);
    const __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.wp, 0, (int)a.w_bytes, 0x00020000);

    if (PATCH && tid < 14)  // the rows of zeros
        *reinterpret_cast<v4u *>(lds + (tid < 7 ? 0 : buf_bytes) + a.halo * kHaloPitch + tid % 7 * 16) = (v4u){0, 0, 0, 0};

    // ---- a wave that fetches: its part of a segment ---------------------------------------------------------
    // Step 0 goes to LDS, then while the others multiply step r, step r + 1 does, from registers into which it was
    // fetched DEPTH steps (patches: one) before.  Past the end of the segment the same instructions are issued with lane
    // offsets of all ones: nothing is fetched, zeros are stored and nobody reads them.
    auto fetch_segment = [&](const int m0, const int n0, const int kbeg, const int kend, const int lane) WPK_LAMBDA {
        const int nr = kend - kbeg;
        const int prod = NP == 1 ? 0 : wave - WN;
        // the channels' bias: asked for now, stored once the first fetches are on their way
        constexpr int BI = (BN + NP * 64 - 1) / (NP * 64);
        float bval[BI];
        {
            const cold_ptr c = cold_args();
            const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(c->bias ? c->bias : c->y), 0, c->bias ? c->K * 4 : 0, 0x00020000);
            static_for<BI>([&](auto I) WPK_LAMBDA {
                bval[decltype(I)::value] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(
                               brsrc, (n0 + prod * 64 + lane + decltype(I)::value * NP * 64) * 4, 0, 0));
            });
        }
        auto store_bias = [&]() WPK_LAMBDA {
            static_for<BI>([&](auto I) WPK_LAMBDA {
                const int i = prod * 64 + lane + decltype(I)::value * NP * 64;
                if (BN % (NP * 64) == 0 || i < BN) bias[parity][i] = bval[decltype(I)::value];
            });
        };
        if constexpr (PATCH) {
            // Blocks of 64 positions, of which each of the NP waves takes every NP-th.
            constexpr int NPB = kHaloMax / 64 / NP;
            static_assert(kHaloMax % (64 * NP) == 0, "as many blocks for each");
            int j0, npos;
            {
                const cold_ptr c = cold_args();
                const int mb = min(c->M, m0 + BM) - 1;
                const int na = fdiv(m0, WPK_COLD_DIV(c, div_pq)), pqa = m0 - na * c->PQ;
                const int pa = fdiv(pqa, WPK_COLD_DIV(c, div_q)), qa = pqa - pa * c->Q;
                const int nb = fdiv(mb, WPK_COLD_DIV(c, div_pq)), pqb = mb - nb * c->PQ;
                const int pb = fdiv(pqb, WPK_COLD_DIV(c, div_q)), qb = pqb - pb * c->Q;
                j0 = patch_first(na, pa, qa, c->stride_h, c->stride_w, c->pad_h, c->pad_w, c->H, c->W);
                npos = min(patch_last(nb, pb, qb, c->stride_h, c->stride_w, c->pad_h, c->pad_w, c->dil_h, c->dil_w, c->H,
                                      c->W) - j0 + 1, c->halo);
            }
            // a lane holds sixteen channels of position `lane` of a block; QUAD: an octet each of positions
            // lane / 2 and 32 + lane / 2
            float v[NPB][16];
            int off[NPB][2];
            auto block = [&](auto PB) WPK_LAMBDA { return decltype(PB)::value * NP + prod; };
            auto fetch = [&](auto PB, const int chunk) WPK_LAMBDA {
                constexpr int pb = decltype(PB)::value;
                static_for<2>([&](auto O) WPK_LAMBDA {
                    constexpr int o = decltype(O)::value;
                    if constexpr (QUAD) {
                        static_for<2>([&](auto H) WPK_LAMBDA {
                            constexpr int b = o * 8 + decltype(H)::value * 4;
                            const int at = chunk * 64 + decltype(H)::value * 16;
                            const v4f q = __builtin_bit_cast(
                                v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                         xrsrc, ANY ? (off[pb][o] + at) | off[pb][o] >> 31 : off[pb][o], ANY ? 0 : at, 0));
                            static_for<4>([&](auto E) WPK_LAMBDA { v[pb][b + decltype(E)::value] = q[decltype(E)::value]; });
                        });
                    } else {
                        static_for<8>([&](auto J) WPK_LAMBDA {
                            constexpr int b = o * 8 + decltype(J)::value;
                            v[pb][b] = __builtin_bit_cast(
                                float, __builtin_amdgcn_raw_buffer_load_b32(
                                           xrsrc, off[pb][0], patch_channel_at(chunk * 16 + b, a.C, a.HW4), 0));
                        });
                    }
                });
            };
            auto put = [&](auto PB, const int buf) WPK_LAMBDA {
                constexpr int pb = decltype(PB)::value;
                static_for<2>([&](auto O) WPK_LAMBDA {
                    constexpr int o = decltype(O)::value;
                    const int pos = QUAD ? block(PB) * 64 + o * 32 + (lane >> 1) : block(PB) * 64 + lane;
                    float e[8];
                    static_for<8>([&](auto J) WPK_LAMBDA { e[decltype(J)::value] = v[pb][o * 8 + decltype(J)::value]; });
                    v4u h, m, l;
                    split_octet(e, h, m, l);
                    if (pos < npos) {
                        char *const p = lds + buf * buf_bytes + pos * kHaloPitch + (QUAD ? lane & 1 : o) * 16;
                        *reinterpret_cast<v4u *>(p) = h;
                        *reinterpret_cast<v4u *>(p + 32) = m;
                        *reinterpret_cast<v4u *>(p + 64) = l;
                    }
                });
            };
            auto each_block = [&](auto &&f) WPK_LAMBDA {
                static_for<NPB>([&](auto PB) WPK_LAMBDA {
                    if (block(PB) * 64 < npos) f(PB);
                });
            };
            each_block([&](auto PB) WPK_LAMBDA {
                constexpr int pb = decltype(PB)::value;
                static_for<2>([&](auto O) WPK_LAMBDA {  // byte offset of a position in x, or all ones
                    constexpr int o = decltype(O)::value;
                    if constexpr (o == 0 || QUAD) {
                        const int pos = QUAD ? block(PB) * 64 + o * 32 + (lane >> 1) : block(PB) * 64 + lane, j = j0 + pos;
                        const int n = fdiv(j, a.div_tap);
                        const int at = (QUAD ? j * a.C * 4 + (lane & 1) * 32 : (n * a.C * a.HW + j - n * a.HW) * 4) +
                                       (int)a.x_bias;
                        off[pb][o] = pos < npos && n < a.N ? at : -1;
                    }
                });
                fetch(PB, kbeg);
            });
            store_bias();
            each_block([&](auto PB) WPK_LAMBDA {
                put(PB, 0);
                if (nr > 1) fetch(PB, kbeg + 1);
            });
            __syncthreads();
            for (int r = 0; r < nr; ++r) {
                if (r + 1 < nr)
                    each_block([&](auto PB) WPK_LAMBDA {
                        put(PB, (r + 1) & 1);
                        if (r + 2 < nr) fetch(PB, kbeg + r + 2);
                    });
                __syncthreads();
            }
        } else if constexpr (FORM == kPoint) {
            // A lane holds PX pixels of an octet.  One wave fetches and splits whole steps (four pixels a lane), two half of each step,
            // an MFMA depth each.
            constexpr int PX = 4 / NP, LANES = 64 / PX;  // (lanes per octet)
            constexpr int DEPTH = 3 * NP;                // steps in flight: 24 KB per wave
            const int px0 = lane % LANES * PX, oct = prod * (4 / NP) + lane / LANES;
            const int m = m0 + px0;
            int voff;
            {
                const cold_ptr c = cold_args();
                const int n = fdiv(m, WPK_COLD_DIV(c, div_pq));
                voff = m < c->M ? (n * c->C * c->HW + m - n * c->HW + oct * 8 * c->HW) * 4 : -1;
            }
            const int place = step_place(px0) + (oct >> 1) * 96 + (oct & 1) * 16;
            float v[DEPTH][8 * PX];  // channel of the octet, pixel
            int step = kbeg;
            auto fetch = [&](auto SLOT) WPK_LAMBDA {
                constexpr int sl = decltype(SLOT)::value;
                const int live = voff | (step < kend ? 0 : -1), first = step * 32 * a.HW4;
                static_for<8>([&](auto J) WPK_LAMBDA {
                    constexpr int j = decltype(J)::value;
                    const int ch = first + j * a.HW4, at = ANY ? (live + ch) | live >> 31 : live, past = ANY ? 0 : ch;
                    if constexpr (PX == 4) {
                        const v4f q = __builtin_bit_cast(
                            v4f, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, at, past, 0));
                        static_for<4>([&](auto E) WPK_LAMBDA { v[sl][j * 4 + decltype(E)::value] = q[decltype(E)::value]; });
                    } else {
                        const v2f q = __builtin_bit_cast(
                            v2f, __builtin_amdgcn_raw_buffer_load_b64(xrsrc, at, past, 0));
                        v[sl][j * 2] = q[0];
                        v[sl][j * 2 + 1] = q[1];
                    }
                });
                step += 1;
            };
            auto put = [&](auto SLOT, const int buf) WPK_LAMBDA {
                constexpr int sl = decltype(SLOT)::value;
                static_for<PX>([&](auto P) WPK_LAMBDA {
                    constexpr int px = decltype(P)::value;
                    float e[8];
                    static_for<8>([&](auto J) WPK_LAMBDA { e[decltype(J)::value] = v[sl][decltype(J)::value * PX + px]; });
                    v4u h, m, l;
                    split_octet(e, h, m, l);
                    char *const p = lds + place + buf * buf_bytes + px * kStepPitch;
                    *reinterpret_cast<v4u *>(p) = h;
                    *reinterpret_cast<v4u *>(p + 32) = m;
                    *reinterpret_cast<v4u *>(p + 64) = l;
                });
            };
            static_for<DEPTH>([&](auto D) WPK_LAMBDA {
                fetch(D);
                __builtin_amdgcn_sched_barrier(0);
            });
            store_bias();
            // nr + 1 meetings in all: number r has step r in place and the buffer of step r - 1 free.  Step r is stored
            // between meetings r - 1 and r.
            int left = nr + 1, turn = 0;  // (of the two buffers)
            auto one = [&](auto P) WPK_LAMBDA {
                constexpr int p = decltype(P)::value;
                using SLOT = std::integral_constant<int, p % DEPTH>;
                if (left <= 0) return false;
                put(SLOT{}, turn);
                turn ^= 1;
                __builtin_amdgcn_sched_barrier(0);
                fetch(SLOT{});
                __builtin_amdgcn_sched_barrier(0);
                __syncthreads();
                --left;
                __builtin_amdgcn_sched_barrier(0);
                return true;
            };
            while (static_all<DEPTH>(one)) {}
        } else {
            constexpr int UN = 4 / NP;                  // octets of 64 pixels per wave and step
            // steps in flight: 24 KB of x per wave, or as much as the counter of loads in flight (63) allows
            constexpr int DEPTH = QUAD ? 3 * NP : 3;
            static_assert(QUAD || NP == 2, "three steps of 16 loads");
            constexpr int XP = QUAD ? UN : 1;           // pixels per lane
            // QUAD: four lanes hold the four octets of a pixel (128 contiguous bytes of x), else a lane its pixel's
            int xvoff[XP], xvb[XP];
            unsigned xinv[XP];
            {
                const cold_ptr c = cold_args();
                static_for<XP>([&](auto I) WPK_LAMBDA {
                    constexpr int i = decltype(I)::value;
                    pixel_window(c, m0 + (QUAD ? (prod * UN + i) * 16 + (lane >> 2) : lane), xvoff[i], xinv[i]);
                    if constexpr (QUAD) xvoff[i] += (lane & 3) * 32;
                });
            }
            // the place in the reduction of the step fetched next: kRows: channel and phase of its first row (see the
            // tap table of the tiled members); else filter tap (r, s), its byte offset and the first channel
            const tap_ptr taps = (tap_ptr)(unsigned long long)a.ktab;
            const int px4 = QUAD ? a.C * 4 : 4;  // bytes between neighbouring pixels of x
            const int tap_step_s = a.dil_w * px4;
            const int tap_step_r = (a.dil_h * a.W - (a.S - 1) * a.dil_w) * px4;
            int step = kbeg, tap_r = 0, tap_s = 0, tap_off = 0, ch = 0;
            {
                const cold_ptr c = cold_args();
                if constexpr (FORM == kRows) {
                    ch = fdiv(kbeg * 32, WPK_COLD_DIV(c, div_tap));
                    tap_s = kbeg * 32 - ch * a.RS;
                } else {
                    const int c32 = fdiv(kbeg, WPK_COLD_DIV(c, div_tap)), tap = kbeg - c32 * a.RS;
                    ch = c32 * 32;
                    tap_r = fdiv(tap, WPK_COLD_DIV(c, div_s));
                    tap_s = tap - tap_r * a.S;
                    tap_off = (tap_r * a.dil_h * a.W + tap_s * a.dil_w) * px4;
                }
            }
            float v[DEPTH][UN * 8];
            auto fetch = [&](auto SLOT) WPK_LAMBDA {
                constexpr int sl = decltype(SLOT)::value;
                const int dead = step < kend ? 0 : -1;
                if constexpr (FORM == kRows) {
                    const bool last = step == a.nsteps - 1;
                    const tap_ptr tp = (last ? (tap_ptr)(unsigned long long)a.ttab : taps + 2 * tap_s * 32) + prod * UN * 16;
                    const int base = last ? 0 : ch * a.HW4;
                    static_for<UN * 8>([&](auto E) WPK_LAMBDA {
                        constexpr int e = decltype(E)::value;
                        const int off = tp[2 * e], rs = tp[2 * e + 1];
                        const int bad = __builtin_amdgcn_sbfe((int)xinv[0], rs & 0xff, 1) |
                                        __builtin_amdgcn_sbfe((int)xinv[0], rs >> 8, 1) | dead;
                        v[sl][e] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, xvoff[0] | bad, off + base, 0));
                    });
                    const int over = ~((tap_s + a.bk_mod_rs - a.RS) >> 31);  // all ones: past the last tap
                    ch += a.bk_div_rs + (over & 1);
                    tap_s += a.bk_mod_rs - (over & a.RS);
                } else {
                    static_for<XP>([&](auto I) WPK_LAMBDA {
                        constexpr int i = decltype(I)::value;
                        xvb[i] = xvoff[i] | __builtin_amdgcn_sbfe((int)xinv[i], tap_r, 1) |
                                 __builtin_amdgcn_sbfe((int)xinv[i], 16 + tap_s, 1) | dead;
                    });
                    static_for<UN>([&](auto U) WPK_LAMBDA {
                        constexpr int u = decltype(U)::value;
                        if constexpr (QUAD) {
                            static_for<2>([&](auto H) WPK_LAMBDA {
                                constexpr int hf = decltype(H)::value;
                                const int at = tap_off + ch * 4 + hf * 16;
                                const v4f q = __builtin_bit_cast(
                                    v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                             xrsrc, ANY ? (xvb[u] + at) | xvb[u] >> 31 : xvb[u], ANY ? 0 : at, 0));
                                static_for<4>([&](auto E) WPK_LAMBDA {
                                    v[sl][u * 8 + hf * 4 + decltype(E)::value] = q[decltype(E)::value];
                                });
                            });
                        } else {
                            const int first = (ch + (prod * UN + u) * 8) * a.HW4, last = (a.C - 1) * a.HW4;
                            static_for<8>([&](auto J) WPK_LAMBDA {
                                constexpr int j = decltype(J)::value;
                                const int at = ANY ? min(first + j * a.HW4, last) : first + j * a.HW4;
                                v[sl][u * 8 + j] = __builtin_bit_cast(
                                    float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, xvb[0], tap_off + at, 0));
                            });
                        }
                    });
                    // one step on, by masks (selects become branches here, and at every join of two paths the compiler
                    // has all loads in flight waited for): along the filter row, to the next one, to the next 32 channels
                    const int row = (tap_s + 1 - a.S) >> 31, chn = (((tap_r + 1 - a.R) >> 31) | row);  // 0: moves on
                    ch += ~chn & 32;
                    tap_off = chn & (tap_off + (row & tap_step_s) + (~row & tap_step_r));
                    tap_r = chn & (tap_r + (~row & 1));
                    tap_s = row & (tap_s + 1);
                }
                step += 1;
            };
            auto put = [&](auto SLOT, const int buf) WPK_LAMBDA {
                constexpr int sl = decltype(SLOT)::value;
                static_for<UN>([&](auto U) WPK_LAMBDA {
                    constexpr int u = decltype(U)::value;
                    float e[8];
                    static_for<8>([&](auto J) WPK_LAMBDA { e[decltype(J)::value] = v[sl][u * 8 + decltype(J)::value]; });
                    v4u h, m, l;
                    split_octet(e, h, m, l);
                    const int px = QUAD ? (prod * UN + u) * 16 + (lane >> 2) : lane;
                    const int oct = QUAD ? lane & 3 : prod * UN + u;
                    char *const p = lds + buf * buf_bytes + step_place(px) + (oct >> 1) * 96 + (oct & 1) * 16;
                    *reinterpret_cast<v4u *>(p) = h;
                    *reinterpret_cast<v4u *>(p + 32) = m;
                    *reinterpret_cast<v4u *>(p + 64) = l;
                });
            };
            static_for<DEPTH>([&](auto D) WPK_LAMBDA {
                fetch(D);
                __builtin_amdgcn_sched_barrier(0);
            });
            store_bias();
            put(std::integral_constant<int, 0>{}, 0);
            fetch(std::integral_constant<int, 0>{});
            __syncthreads();
            int r = 0;
            auto one = [&](auto P) WPK_LAMBDA {
                constexpr int p = decltype(P)::value;
                if (r + p >= nr) return false;
                using SLOT = std::integral_constant<int, (p + 1) % DEPTH>;
                put(SLOT{}, (r + p + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
                fetch(SLOT{});
                __builtin_amdgcn_sched_barrier(0);
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
                return true;
            };
            // (the compiler has every load in flight waited for at the top of the body: twelve steps long)
            constexpr int LAPS = 12;
            while (static_all<LAPS>(one)) r += LAPS;
        }
    };

    auto run_segment = [&](const int tile, const int kbeg, const int kend, const int mode,
                           const int fix_j, const int fix_slot, const int fix_n) WPK_LAMBDA {
    if (kbeg >= kend) return;
    // (the lane's numbers formed anew for every segment and for the way out: what is derived from those of the kernel's entry is
    // held all through otherwise, and the patch forms spill three to twelve registers)
    int seg_tid = tid;
    asm volatile("" : "+v"(seg_tid));
    const int lane = seg_tid & 63, lrow = lane >> 5, lcol = lane & 31;
    int tile_m, tile_n;
    {
        const cold_ptr c = cold_args();
        if (c->mfast) {
            tile_n = fdiv(tile, WPK_COLD_DIV(c, div_tiles_m));
            tile_m = tile - tile_n * c->tiles_m;
        } else {
            tile_m = fdiv(tile, WPK_COLD_DIV(c, div_tiles_n));
            tile_n = tile - tile_m * c->tiles_n;
        }
    }
    const int m0 = tile_m * BM;
    parity ^= 1;
    if (wave >= WN) {
        fetch_segment(m0, tile_n * BN, kbeg, kend, lane);
        if (mode == kFixup) {  // (the three barriers of the meeting)
            __syncthreads();
            __syncthreads();
            __syncthreads();
        }
        return;
    }

    // ---- a wave that multiplies ---------------------------------------------------------------------------
    const int nr = kend - kbeg, n0 = tile_n * BN + wave * 32;
    const unsigned depth_bytes = (unsigned)(a.Kpad / 32) * 3072u;  // weights: one depth further
    const unsigned wbase = (unsigned)(n0 / 32) * 3072u;
    v8bf aw[3 * 3];  // weights: three depths, two of them ahead
    constexpr unsigned kTapStride = split_depth(PATCH, 0, 1);
    auto step_base = [&](const int r) WPK_LAMBDA {
        return split_weights_at(PATCH, wbase, kbeg + r, a.nsteps, depth_bytes);
    };
    auto load_a = [&](auto SET, const unsigned base, auto E) WPK_LAMBDA {
        constexpr int set = decltype(SET)::value, e = decltype(E)::value;
        aw[set * 3 + e] = __builtin_bit_cast(
            v8bf, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16, base + e * 1024, 0));
    };
    unsigned wcur = step_base(0);
    static_for<2>([&](auto S) WPK_LAMBDA {
        static_for<3>([&](auto E) WPK_LAMBDA { load_a(S, wcur + decltype(S)::value * kTapStride * depth_bytes, E); });
    });
    unsigned addr[PATCH ? NMT * 5 : 1];  // of every tap, in units of 16 bytes, two per register
    if constexpr (PATCH) {
        // (the tile's first position, as the wave that fetches has it)
        const cold_ptr c = cold_args();
        const int na = fdiv(m0, WPK_COLD_DIV(c, div_pq)), pqa = m0 - na * c->PQ;
        const int pa = fdiv(pqa, WPK_COLD_DIV(c, div_q)), qa = pqa - pa * c->Q;
        const int j0 = patch_first(na, pa, qa, c->stride_h, c->stride_w, c->pad_h, c->pad_w, c->H, c->W);
        static_for<NMT>([&](auto J) WPK_LAMBDA {
            constexpr int j = decltype(J)::value;
            const int m = m0 + j * 32 + lcol;
            const int n = fdiv(m, WPK_COLD_DIV(c, div_pq)), pq = m - n * c->PQ;
            const int p = fdiv(pq, WPK_COLD_DIV(c, div_q)), q = pq - p * c->Q;
            const int ih = p * c->stride_h - c->pad_h, iw = q * c->stride_w - c->pad_w;
            const int first = n * c->HW + ih * c->W + iw - j0;
            static_for<9>([&](auto TAP) WPK_LAMBDA {
                constexpr int t = decltype(TAP)::value, r = t / 3, s = t % 3;
                const bool in = m < c->M && (unsigned)(ih + r * c->dil_h) < (unsigned)c->H &&
                                (unsigned)(iw + s * c->dil_w) < (unsigned)c->W;
                const int pos = first + r * c->dil_h * c->W + s * c->dil_w;
                // (never out of range by construction; the unsigned minimum keeps it so whatever happens)
                const unsigned at = min(in ? (unsigned)pos : (unsigned)c->halo, (unsigned)c->halo) * (kHaloPitch / 16) + lrow;
                addr[j * 5 + t / 2] = t % 2 ? addr[j * 5 + t / 2] | at << 16 : at;
            });
        });
    }
    v16f acc[NMT], sml[NMT];
    static_for<NMT>([&](auto I) WPK_LAMBDA {
        static_for<16>([&](auto E) WPK_LAMBDA {
            acc[decltype(I)::value][decltype(E)::value] = 0.0f;
            sml[decltype(I)::value][decltype(E)::value] = 0.0f;
        });
    });
    // The operands of a depth: three parts for each of the wave's two pixel blocks.  The products are issued in an
    // order that is done with l after two MFMAs, with m after six and with h after twelve, and each part of the
    // NEXT depth is read into the registers the moment they are free: six MFMAs or more ahead of its use.
    v8bf bx[NMT * 3];
    int bofs = 0;  // the step's buffer
    auto read_part = [&](auto PART, auto TAP) WPK_LAMBDA {
        constexpr int part = decltype(PART)::value, t = decltype(TAP)::value;
        static_for<NMT>([&](auto J) WPK_LAMBDA {
            constexpr int j = decltype(J)::value;
            if constexpr (PATCH) {
                const unsigned at = t % 2 ? addr[j * 5 + t / 2] >> 16 : addr[j * 5 + t / 2] & 0xffffu;
                bx[j * 3 + part] = *reinterpret_cast<const v8bf *>(lds + (at * 16 + bofs) + part * 32);
            } else {
                bx[j * 3 + part] = *reinterpret_cast<const v8bf *>(lds + (bofs + step_place(lcol) + lrow * 16) +
                                                                   step_place(j * 32) + t * 96 + part * 32);
            }
        });
    };
    // step number r of the segment; P: its number within the loop's body
    auto step_body = [&](const int r, auto P) WPK_LAMBDA {
        const unsigned wnext = step_base(r + 1);
        static_for<NT>([&](auto TAP) WPK_LAMBDA {
            constexpr int t = decltype(TAP)::value, g = decltype(P)::value * NT + t;
            using NEXT = std::integral_constant<int, (t + 1) % NT>;
            using SET = std::integral_constant<int, (g + 2) % 3>;  // the set that the depth before this one has left
            const unsigned ahead = t + 2 < NT ? wcur + (t + 2) * kTapStride * depth_bytes
                                              : wnext + (t + 2 - NT) * kTapStride * depth_bytes;
            static_for<6>([&](auto PQ) WPK_LAMBDA {
                constexpr int q = decltype(PQ)::value;
                // (A part, B part), 0 h, 1 m, 2 l: hl | mm, hm | hh, mh, lh
                constexpr int pa = q == 1 || q == 4 ? 1 : q == 5 ? 2 : 0, pb = q == 0 ? 2 : q == 1 || q == 2 ? 1 : 0;
                static_for<NMT>([&](auto J) WPK_LAMBDA {
                    constexpr int j = decltype(J)::value;
                    const v8bf av = aw[g % 3 * 3 + pa];
                    if constexpr (q == 3)
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bx[j * 3 + pb], acc[j], 0, 0, 0);
                    else
                        sml[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bx[j * 3 + pb], sml[j], 0, 0, 0);
                    // weights two depths ahead
                    if constexpr (q * NMT + j < 3) load_a(SET{}, ahead, std::integral_constant<int, q * NMT + j>{});
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (t + 1 == NT) {
                    if constexpr (q == 1) {
                        // every wave holds its last operands of this step, and the next one is in place (the MFMAs
                        // just issued run on while the waves meet)
                        __syncthreads();
                        bofs = buf_bytes - bofs;
                        read_part(std::integral_constant<int, 2>{}, NEXT{});
                    }
                } else {
                    if constexpr (q == 0) read_part(std::integral_constant<int, 2>{}, NEXT{});
                }
                if constexpr (q == 2) read_part(std::integral_constant<int, 1>{}, NEXT{});
                if constexpr (q == 5) read_part(std::integral_constant<int, 0>{}, NEXT{});
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        wcur = wnext;
    };
    __syncthreads();
    static_for<3>([&](auto PART) WPK_LAMBDA { read_part(PART, std::integral_constant<int, 0>{}); });
    constexpr int BODY = PATCH ? 1 : 3;  // steps after which the weights' sets come round
    int r = 0;
    auto step = [&](auto P) WPK_LAMBDA {
        if (r + decltype(P)::value >= nr) return false;
        step_body(r + decltype(P)::value, P);
        return true;
    };
    while (static_all<BODY>(step)) r += BODY;

    if (join_sums(acc, sml))
        fp32_tile<FORM, NMT>(acc, xrsrc, wrsrc, m0, wbase, nr * NT, [&](int i) WPK_LAMBDA {
            return split_depth(PATCH, kbeg + i / NT, i % NT);
        }, lane);
    const cold_ptr ce = cold_args();
    asm volatile("" : "+v"(seg_tid));
    if (mode == kFixup &&
        !meet_shared_tile<NMT, T>(ce, acc, BM * BN, seg_tid, fix_j, fix_slot, fix_n, &arrival))
        return;  // not the last: done with this tile
    store_wave_tile<1, NMT, 2>(ce, acc, m0, n0, seg_tid >> 5 & 1, seg_tid & 31, mode == kAtomic, &bias[parity][wave * 32]);
    };  // run_segment

    for_each_segment(a, run_segment);
}

template <int WN, SplitForm FORM, int NP, bool ANY>
hipError_t launch_split_form(const IgemmArgs &a, hipStream_t stream)
{
    const size_t lds = 2 * (size_t)(FORM >= kPatch ? (a.halo + 1) * kHaloPitch : 64 * kStepPitch);
    return launch_kernel<split_kernel<WN, FORM, NP, ANY>, 64 * (WN + NP), 2 * (kHaloMax + 1) * kHaloPitch>(
        a, stream, lds, 2 * 32 * WN * sizeof(float) + sizeof(int));  // (bias, arrival)
}

// How activations are found, with or without padded channels, by NP fetching waves; ONE: there is a form with one for these WN.
template <int WN, SplitForm FORM, bool ANY, bool ONE>
hipError_t launch_split_waves(const IgemmArgs &a, hipStream_t stream)
{
    if constexpr (ONE)
        if (a.producers == 1) return launch_split_form<WN, FORM, 1, ANY>(a, stream);
    if constexpr (!ONE || WN >= 2 || FORM >= kPatch)
        return launch_split_form<WN, FORM, 2, ANY>(a, stream);
    return hipErrorInvalidValue;
}

// (the K-step gene says whether patches may be used, which the host has looked at; `stages` has no meaning here)
template <int WN>
hipError_t launch_split(const IgemmArgs &a, hipStream_t stream)
{
    const bool any = a.C % 32 != 0;
    if (a.halo > 0) {
        if (a.xl != 2) return launch_split_waves<WN, kPatch, false, (WN < 4)>(a, stream);
        return any ? launch_split_waves<WN, kPatchQuads, true, (WN < 4)>(a, stream)
                   : launch_split_waves<WN, kPatchQuads, false, (WN < 4)>(a, stream);
    }
    if (a.xl == 2)
        return any ? launch_split_form<WN, kQuads, WN == 4 ? 2 : 1, true>(a, stream)
                   : launch_split_form<WN, kQuads, WN == 4 ? 2 : 1, false>(a, stream);
    if (a.halo == -1)
        return any ? launch_split_waves<WN, kPoint, true, (WN < 4)>(a, stream)
                   : launch_split_waves<WN, kPoint, false, (WN < 4)>(a, stream);
    if (a.xl == 3)
        return any ? launch_split_form<WN, kTaps, 2, true>(a, stream) : launch_split_form<WN, kTaps, 2, false>(a, stream);
    return launch_split_form<WN, kRows, 2, false>(a, stream);
}

}  // namespace wpk
#endif
