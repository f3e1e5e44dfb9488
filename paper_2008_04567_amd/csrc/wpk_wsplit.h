// The wave-split members of the convolution kernel family for gfx950: for launches whose
// arithmetic is a few microseconds at most (single images, late layers of few pixels).
//
// Same GEMM view and same packed weights as the tiled members (wpk_igemm.h);
// the filter taps are followed by arithmetic instead of being read from the tap table, and every wave carries out
// a part of the tile.  What differs is who shares what.  A tiled workgroup stages its operands through
// LDS so that every wave reuses them, and it needs a long reduction per workgroup to repay the
// staging, the barriers and -- when the reduction has to be cut between workgroups to fill the
// device -- the meeting of the partial tiles in memory, several dependent memory round trips at
// the end of a launch that has little else to do.  Here a workgroup owns one tile of 32 pixels by
// BN channels and its WK waves cut the REDUCTION between them: every wave multiplies the whole tile
// over its own run of reduction rows, fetching both operands from global memory straight into
// the registers the MFMAs read (nothing in them is shared with another wave, so LDS would only add
// a store, a barrier and a load), and the waves' partial tiles meet in LDS: one barrier.  Where
// the tiled members need a reduction cut five ways across workgroups, these need none, or a
// shorter one.
//
// Operands.  Reduction rows are ordered (r, s, c) (the tap-major forms of the family: C a multiple
// of 32, see Problem::tapmajor and Problem::xquad), and the unit of work is an octet of eight
// rows: eight consecutive channels of one filter tap.  In the
// octet's four MFMAs (v_mfma_f32_32x32x2_f32) the low half-wave supplies rows 0..3 and the high
// half-wave rows 4..7, as in the tiled members.  So per octet a lane loads
//   weights: one 16-byte quad per 32-channel block -- packed [row/4][channel][4] is exactly that;
//   x [N][C][H][W]: four dwords, a channel stride apart (the stride rides in the scalar offset);
//   x [N][H][W][C]: one 16-byte quad (four consecutive channels of its pixel and tap).
// Out-of-image taps and pixels past the last one get a lane offset of all ones, which the buffer
// range check turns into a zero, as everywhere in the family.  PD octets are in flight per wave.
#ifndef WPK_WSPLIT_H
#define WPK_WSPLIT_H

#include "wpk_igemm.h"

namespace wpk {

// What a wave carries out of a tile: accumulator quads first .. first + QW - 1, quad q being channels
// 8 (q % 4) + 4 (lane / 32) .. + 3 of block q / 4 for pixel lane % 32.  fetch_bias() and fetch_residual() ask for what its
// outputs add, store() adds that and stores, or adds to y by atomics.  Behind the loop nothing is asked for where there is
// nothing to add (a wave per tile, 1x1, 64 -> 256 channels at 56x56, N = 2, no epilogue: 5.6 us, with loads out of range 6.1).
template <int QW>
struct OutQuads {
    float b[QW * 4], r[QW * 4];
    int k;           // the lane's first channel
    unsigned place;  // byte offset in y of that channel of the lane's pixel; kNowhere past the last pixel

    // channel of register e behind the first
    static constexpr int channel(const int e) { return e / 16 * 32 + e % 16 / 4 * 8 + e % 4; }

    __device__ __forceinline__ void first_channel(const int n0, const int first, const int lrow)
    {
        k = n0 + 4 * lrow + (first >> 2) * 32 + (first & 3) * 8;
    }

    __device__ __forceinline__ void fetch_bias(const IgemmArgs *const c)
    {
        static_for<QW * 4>([&](auto E) WPK_LAMBDA { b[decltype(E)::value] = 0.0f; });
        if (!c->bias) return;
        const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc((void *)c->bias, 0, c->K * 4, 0x00020000);
        static_for<QW * 4>([&](auto E) WPK_LAMBDA {
            constexpr int e = decltype(E)::value;
            b[e] = __builtin_bit_cast(float,
                                      __builtin_amdgcn_raw_buffer_load_b32(brsrc, (k + channel(e)) * 4, 0, 0));
        });
    }

    __device__ __forceinline__ void find_place(const IgemmArgs *const c, const int m)
    {
        const int n = fdiv(m, WPK_COLD_DIV(c, div_pq)), pq = m - n * c->PQ;
        place = output_place(m, c->M, n, pq, k, c->K, c->PQ, c->yl != 0);
    }

    // The whole offset is the lane's, which the range check covers: a pixel or a channel past the last one loads zero.
    // ISSUE: the loads are issued whether there is a residual or not, out of range where not (ahead of the loop, which counts the
    // loads in flight); live: this wave has outputs.
    template <class ISSUE>
    __device__ __forceinline__ void fetch_residual(const IgemmArgs *const c, const bool live, ISSUE)
    {
        static_for<QW * 4>([&](auto E) WPK_LAMBDA { r[decltype(E)::value] = 0.0f; });
        if (!ISSUE::value && !(c->res && live)) return;
        const __amdgpu_buffer_rsrc_t rrsrc = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(c->res ? c->res : c->y), 0, c->res && live ? (int)c->y_bytes : 0, 0x00020000);
        const unsigned ch4 = c->yl ? 4 : c->PQ * 4;
        static_for<QW * 4>([&](auto E) WPK_LAMBDA {
            constexpr int e = decltype(E)::value;
            r[e] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rrsrc, output_at(place, k, channel(e), c->K, ch4), 0, 0));
        });
    }

    __device__ __forceinline__ void store(const IgemmArgs *const c, const v4f (&sum)[QW], const bool whole, const bool atomic)
    {
        if (place == kNowhere) return;
        const __amdgpu_buffer_rsrc_t yrsrc =
            __builtin_amdgcn_make_buffer_rsrc((void *)c->y, 0, (int)c->y_bytes, 0x00020000);
        const int ch4 = c->yl ? 4 : c->PQ * 4;
        if (atomic) {
            static_for<QW * 4>([&](auto E) WPK_LAMBDA {
                constexpr int e = decltype(E)::value;
                const float v = sum[e / 4][e % 4];
                if (whole || k + channel(e) < c->K)
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(v, yrsrc, place, channel(e) * ch4, 0);
            });
            return;
        }
        float v[QW * 4];
        static_for<QW * 4>([&](auto E) WPK_LAMBDA {
            constexpr int e = decltype(E)::value;
            const float t = sum[e / 4][e % 4] + (b[e] + r[e]);
            v[e] = c->relu ? fmaxf(t, 0.0f) : t;
        });
        // WHOLE: every channel exists (the usual case), no check per register
        auto emit = [&](auto WHOLE, auto POLICY) WPK_LAMBDA {
            static_for<QW * 4>([&](auto E) WPK_LAMBDA {
                constexpr int e = decltype(E)::value;
                if (decltype(WHOLE)::value || k + channel(e) < c->K)
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v[e]), yrsrc, place, channel(e) * ch4,
                                                          decltype(POLICY)::value);
            });
        };
        // whole 128-byte runs are written through, channels-last pieces are not (kYStorePolicy)
        using Through = std::integral_constant<int, kYStorePolicy>;
        using Back = std::integral_constant<int, 0>;
        if (c->yl == 2) {  // (K a multiple of four, everything 16-byte aligned)
            static_for<QW>([&](auto Q) WPK_LAMBDA {
                constexpr int q = decltype(Q)::value;
                if (whole || k + channel(q * 4) < c->K)
                    store_quad(__builtin_bit_cast(v4u, (v4f){v[q * 4], v[q * 4 + 1], v[q * 4 + 2], v[q * 4 + 3]}), yrsrc,
                               place + channel(q * 4) * 4, Back{});
            });
        } else if (c->yl == 1) {
            emit(std::false_type{}, Back{});
        } else if (whole) {
            emit(std::true_type{}, Through{});
        } else {
            emit(std::false_type{}, Through{});
        }
    }
};

// QUAD: x is channels-last and moves as channel quads (a.xl == 2); else [N][C][H][W] (a.xl == 3).
template <int BN, int WK, int PD, bool QUAD>
__global__ void __launch_bounds__(64 * WK) wsplit_kernel(const IgemmArgs a)
{
    constexpr int NNT = BN / 32;
    static_assert(BN % 32 == 0 && NNT >= 1 && NNT <= 2, "one or two 32-channel blocks per wave");
    static_assert(WK >= 1 && WK <= 8 && (WK & (WK - 1)) == 0, "1, 2, 4 or 8 waves");
    static_assert(PD >= 2 && PD <= 12, "octets in flight");
    // the waves' partial tiles: accumulator quad q (= 4 * block + quad of the block) of wave w and lane l at float
    // (w * NQ + q) * 256 + 4 * l -- 16-byte accesses, consecutive lanes, no conflicts
    constexpr int NQ = NNT * 4;                      // accumulator quads of a tile
    constexpr int OUT = WK < NQ ? WK : NQ;           // waves that carry the tile out,
    constexpr int QW = NQ / OUT;                     // so many quads each
    __shared__ __attribute__((aligned(16))) float red[wave_split_floats(BN, WK)];
    int *const arrival = reinterpret_cast<int *>(red);  // (64 KB are taken by eight waves of 64 channels: no room beside them)

    touch_kernarg_lines();
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wk = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane >> 5, lcol = lane & 31;

    // ---- which tile, which slice of the reduction -------------------------------------------------
    // (the arguments are used straight from the by-value kernel argument: this kernel has scalar
    // registers to spare, and every argument read at its place of use would be one more wait on the
    // scalar cache in a set-up that is a sixth of a short launch)
    const IgemmArgs *const c = &a;
    const int g = blockIdx.x;
    const int gr = a.remap ? xcd_remap(g, (int)gridDim.x) : g;
    const int slice = fdiv(gr, WPK_COLD_DIV(c, div_tiles));
    const int tile = gr - slice * c->tiles;
    int tile_m, tile_n;
    if (c->mfast) {
        tile_n = fdiv(tile, WPK_COLD_DIV(c, div_tiles_m));
        tile_m = tile - tile_n * c->tiles_m;
    } else {
        tile_m = fdiv(tile, WPK_COLD_DIV(c, div_tiles_n));
        tile_n = tile - tile_m * c->tiles_n;
    }
    const int m0 = tile_m * 32, n0 = tile_n * BN;
    // the slice's octets [s0, s1), cut evenly between the waves: this wave's are [obeg, oend)
    // (a wave with none contributes a tile of zeros)
    const int s0 = slice * c->steps_per_split, s1 = min(a.nsteps, s0 + c->steps_per_split);
    const int obeg = s0 + (s1 - s0) * wk / WK, oend = s0 + (s1 - s0) * (wk + 1) / WK;
    const int nr = oend - obeg;

    __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const char *)a.x - a.x_bias), 0, (int)(a.x_bytes + a.x_bias), 0x00020000);
    __amdgpu_buffer_rsrc_t wrsrc =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.wp, 0, (int)a.w_bytes, 0x00020000);
    // (kept whole: the compiler puts descriptors together from their words at every load otherwise, four scalar
    // instructions an octet, 0.3-0.6 us per launch)
    asm volatile("" : "+s"(xrsrc), "+s"(wrsrc));

    // ---- the loader's place in the reduction: its filter tap (r, s) and the offsets of the next octet to fetch.  Kept by
    //      arithmetic on the scalar unit, not read from the tap table: a table entry costs a memory round trip before the first
    //      fetch can go out, which a launch of a few microseconds notices.  Between two events -- a change of tap, the end of
    //      the run -- an octet moves the offsets on by constants and counts down to the next event, nine scalar
    //      instructions; what an event changes is behind a branch.  (A wave issues one instruction every four or
    //      five cycles whatever it is, and four MFMAs give it time for 50: with selects instead of the branch, 35 scalar
    //      instructions an octet, 3x3 with 64 channels at 56x56, N = 1, takes 6.4 us instead of 5.6, 1x1 512 -> 128 at 28x28
    //      5.8 instead of 5.1.)
    const int px4 = QUAD ? a.C * 4 : 4;  // bytes between neighbouring pixels of x
    const int tap_step_s = c->dil_w * px4;
    const int tap_step_r = (c->dil_h * a.W - (a.S - 1) * c->dil_w) * px4;
    const int tap0 = fdiv(obeg * 8, WPK_COLD_DIV(c, div_tap));  // by C
    const int ch0 = obeg * 8 - tap0 * a.C;
    int tap_r = fdiv(tap0, WPK_COLD_DIV(c, div_s));
    int tap_s = tap0 - tap_r * a.S;
    int tap_off = (tap_r * c->dil_h * a.W + tap_s * c->dil_w) * px4;
    const int ch4 = a.HW4;               // bytes between channels of x
    int xo[QUAD ? 1 : 4];                // offsets of the octet's channels behind the lane's
    auto at_channel = [&](const int ch) WPK_LAMBDA {
        static_for<QUAD ? 1 : 4>([&](auto Q) WPK_LAMBDA { xo[decltype(Q)::value] = tap_off + (ch + decltype(Q)::value) * ch4; });
    };
    at_channel(ch0);
    int seg = min(nr, (a.C - ch0) >> 3);  // octets up to the next event
    int left = nr - seg;                  // and behind it
    // weights: the lane's quad of the octet's first block row, its channel
    const int wvoff = (lrow * a.Kpad + n0 + lcol) * 16;
    const int woct_bytes = 2 * a.Kpad * 16;  // one octet further
    int wv = nr > 0 ? wvoff : -1, wo = obeg * woct_bytes;
    // activations: the pixel's window, the half-wave's four channels
    int xvoff;
    unsigned xinv;
    pixel_window(c, m0 + lcol, xvoff, xinv);
    xvoff += lrow * 4 * (QUAD ? 4 : a.HW4);
    auto masked = [&]() WPK_LAMBDA {  // the lane's offset under the present tap, or all ones
        return xvoff | __builtin_amdgcn_sbfe((int)xinv, tap_r, 1) | __builtin_amdgcn_sbfe((int)xinv, 16 + tap_s, 1);
    };
    int xvb = nr > 0 ? masked() : -1;

    float xr[PD * 4];
    v4f wr[PD * NNT];
    // Loads of the loader's octet into register set SET; then the loader moves one octet on.
    // Every call issues the same loads whether the octet is inside the run or past its end,
    // so that the count of loads in flight behind any register is the same on every path and the
    // waits the compiler places stay exact; an octet past the end gets lane offsets of all ones
    // (nothing is fetched, nobody reads the registers).
    auto issue = [&](auto SET) WPK_LAMBDA {
        constexpr int set = decltype(SET)::value;
        if constexpr (QUAD) {
            v4f v = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xvb, xo[0], 0));
            xr[set * 4] = v[0];
            xr[set * 4 + 1] = v[1];
            xr[set * 4 + 2] = v[2];
            xr[set * 4 + 3] = v[3];
            xo[0] += 8 * 4;
        } else {
            static_for<4>([&](auto Q) WPK_LAMBDA {
                constexpr int q = decltype(Q)::value;
                xr[set * 4 + q] =
                    __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrsrc, xvb, xo[q], 0));
                xo[q] += 8 * ch4;
            });
        }
        static_for<NNT>([&](auto I) WPK_LAMBDA {
            constexpr int i = decltype(I)::value;
            wr[set * NNT + i] =
                __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wv, wo + i * 32 * 16, 0));
        });
        wo += woct_bytes;
        if (--seg == 0) {
            asm volatile("");  // (keeps this a branch)
            const bool row = tap_s + 1 == a.S;
            tap_off += row ? tap_step_r : tap_step_s;
            tap_r += row ? 1 : 0;
            tap_s = row ? 0 : tap_s + 1;
            at_channel(0);
            seg = left > 0 ? min(left, a.C >> 3) : 0x7fffffff;
            xvb = left > 0 ? masked() : -1;
            wv = left > 0 ? wv : -1;
            left -= seg;
        }
    };

    // Two sums per block that take turns and meet at the end: half as many roundings at the size of the whole sum.  Error
    // against 64 bits (2-norm) of ResNet-50, N = 1, 4.3e-7 -> 3.4e-7, of 3x3, 512 channels, 7x7 1.7e-7 -> 1.3e-7, for 0.2-0.3 us a launch
    // (372 -> 386 and 8.3 -> 8.6).  (For one block of channels; two have no registers to spare.)
    constexpr int SUMS = NNT == 1 ? 2 : 1;
    v16f acc[NNT * SUMS];
    static_for<NNT * SUMS>([&](auto I) WPK_LAMBDA {
        static_for<16>([&](auto E) WPK_LAMBDA { acc[decltype(I)::value][decltype(E)::value] = 0.0f; });
    });
    auto multiply = [&](auto SET) WPK_LAMBDA {
        constexpr int set = decltype(SET)::value;
        static_for<4>([&](auto Q) WPK_LAMBDA {
            constexpr int q = decltype(Q)::value;
            static_for<NNT>([&](auto I) WPK_LAMBDA {
                constexpr int i = decltype(I)::value;
                constexpr int t = i + q % SUMS;
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[set * NNT + i][q], xr[set * 4 + q], acc[t], 0, 0, 0);
            });
        });
    };
    // Octet number r of the wave's run travels in register set r % PD.  The loop is left at the
    // first octet past the end of the run: no join inside it, so the accumulators stay where they
    // are and the fetched registers are not live after it.  Its body is kGroups groups of PD octets:
    // the compiler waits for every load in flight at the top of a loop body (not only for the set
    // the first step needs), which empties the pipeline once per pass through the body.
    constexpr int kGroups = 4;
    static_for<PD>([&](auto P) WPK_LAMBDA {
        issue(P);
        __builtin_amdgcn_sched_barrier(0);
    });
    // The residual of this wave's outputs is asked for behind the first octets: it arrives while they are multiplied instead
    // of after the last one, a round trip to memory less.  Not where slices meet, of which only one stores, and not by one or two
    // waves, which have four times or twice as many outputs each.
    constexpr bool AHEAD = QW == 1;
    OutQuads<QW> out;
    if constexpr (AHEAD) {
        out.first_channel(n0, wk * QW, lrow);
        out.find_place(c, m0 + lcol);
        out.fetch_residual(c, wk < OUT && c->split_k == 1, std::true_type{});
    }
    __builtin_amdgcn_sched_barrier(0);
    int r = 0;
    auto step = [&](auto P) WPK_LAMBDA {
        constexpr int p = decltype(P)::value;
        if (r + p >= nr) return false;
        multiply(std::integral_constant<int, p % PD>{});
        issue(std::integral_constant<int, p % PD>{});
        __builtin_amdgcn_sched_barrier(0);
        return true;
    };
    while (static_all<kGroups * PD>(step)) r += kGroups * PD;
    if constexpr (SUMS == 2)
        static_for<16>([&](auto E) WPK_LAMBDA { acc[0][decltype(E)::value] += acc[1][decltype(E)::value]; });

    if constexpr (!AHEAD) {
        out.first_channel(n0, wk * QW, lrow);
        out.find_place(c, m0 + lcol);
    }
    if constexpr (QW < 8) out.fetch_bias(c);
    // ---- the waves' partial tiles meet in LDS: wave w adds up quads w QW .. of all of them and carries these on ------
    v4f sum[QW];
    if constexpr (WK == 1) {
        static_for<QW>([&](auto Q) WPK_LAMBDA {
            constexpr int q = decltype(Q)::value, i = q / 4, e = q % 4 * 4;
            sum[q] = (v4f){acc[i][e], acc[i][e + 1], acc[i][e + 2], acc[i][e + 3]};
        });
    } else {
        static_for<NQ>([&](auto Q) WPK_LAMBDA {
            constexpr int q = decltype(Q)::value, i = q / 4, e = q % 4 * 4;
            *reinterpret_cast<v4f *>(red + (wk * NQ + q) * 256 + 4 * lane) =
                (v4f){acc[i][e], acc[i][e + 1], acc[i][e + 2], acc[i][e + 3]};
        });
        __syncthreads();
        if (wk >= OUT && c->split_k == 1) return;
        const float *const mine = red + (wk < OUT ? wk : 0) * QW * 256 + 4 * lane;
        static_for<WK>([&](auto U) WPK_LAMBDA {
            static_for<QW>([&](auto Q) WPK_LAMBDA {
                constexpr int u = decltype(U)::value, q = decltype(Q)::value;
                const v4f v = *reinterpret_cast<const v4f *>(mine + (u * NQ + q) * 256);
                if constexpr (u == 0) sum[q] = v;
                else sum[q] += v;
            });
        });
    }

    // ---- a reduction cut between workgroups: the slices of a tile meet through the workspace (each
    //      stores its partial tile to its slot and counts itself in; whoever comes last adds up the
    //      others and stores y), or, without one, through atomics into y, which the host zeroed ------
    bool atomic = false;
    if (c->split_k > 1) {
        if (!c->ws) {
            atomic = true;
            if (wk >= OUT) return;
        } else {
            constexpr int kCoherent = 17;  // sc0 | sc1: past the L2s, which do not snoop each other
            constexpr int SLOT = 32 * BN;  // floats; quad q of lane l at q * 256 + 4 * l
            const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(c->ws + (size_t)tile * c->ws_maxc * SLOT), 0, c->ws_maxc * SLOT * 4, 0x00020000);
            const int at = (wk * QW * 256 + 4 * lane) * 4;
            if (wk < OUT)
                static_for<QW>([&](auto Q) WPK_LAMBDA {
                    store_quad(__builtin_bit_cast(v4u, sum[decltype(Q)::value]), srsrc,
                               slice * SLOT * 4 + at + decltype(Q)::value * 1024,
                               std::integral_constant<int, kCoherent>{});
                });
            // every store of this wave acknowledged, then every wave's, before the arrival is counted
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0) *arrival = atomicAdd(c->ws_cnt + tile, 1);
            __syncthreads();
            if (*arrival != c->split_k - 1 || wk >= OUT) return;  // not the last: done with this tile
            if (tid == 0) c->ws_cnt[tile] = 0;                   // leave the counter clean for the next launch
            // seven slots at a time (one quad per lane; fewer where a wave carries more), all requested before the
            // first is added (a slot number past the last becomes an out-of-range offset, which loads 0)
            constexpr int kGang = QW == 1 ? 7 : 4;
            for (int t0 = 0; t0 < c->split_k - 1; t0 += kGang) {
                v4f part[kGang][QW];
                static_for<kGang>([&](auto U) WPK_LAMBDA {
                    constexpr int u = decltype(U)::value;
                    const int t = t0 + u, sl = t + (t >= slice ? 1 : 0);  // t-th slot not mine
                    const unsigned off = t < c->split_k - 1 ? (unsigned)(sl * SLOT * 4 + at) : 0xffffffffu;
                    static_for<QW>([&](auto Q) WPK_LAMBDA {
                        part[u][decltype(Q)::value] = __builtin_bit_cast(
                            v4f, __builtin_amdgcn_raw_buffer_load_b128(srsrc, off, decltype(Q)::value * 1024, kCoherent));
                    });
                });
                static_for<kGang * QW>([&](auto UQ) WPK_LAMBDA {
                    constexpr int u = decltype(UQ)::value / QW, q = decltype(UQ)::value % QW;
                    sum[q] += part[u][q];
                });
            }
        }
    }
    if constexpr (QW == 8) out.fetch_bias(c);
    if (!AHEAD || c->split_k > 1) out.fetch_residual(c, !atomic, std::false_type{});
    out.store(c, sum, n0 + BN <= c->K, atomic);
}

template <int BN, int WK, int PD>
hipError_t launch_wsplit(const IgemmArgs &a, hipStream_t stream)
{
    dim3 grid((unsigned)(a.tiles_m * a.tiles_n * a.split_k));
    if (a.xl == 2)
        hipLaunchKernelGGL((wsplit_kernel<BN, WK, PD, true>), grid, dim3(64 * WK), 0, stream, a);
    else
        hipLaunchKernelGGL((wsplit_kernel<BN, WK, PD, false>), grid, dim3(64 * WK), 0, stream, a);
    return hipGetLastError();
}

}  // namespace wpk
#endif
