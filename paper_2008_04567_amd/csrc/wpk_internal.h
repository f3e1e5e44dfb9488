// Internal declarations shared by the translation units of libwpk.  Not part of the ABI.
#ifndef WPK_INTERNAL_H
#define WPK_INTERNAL_H

#include <stdint.h>

#include <atomic>
#include <string>
#include <vector>

#include "wpk.h"

// The list of compiled tile combinations; a build may name a shorter list of its own (the gene
// space shrinks with it: the constraint check only admits combinations on the list).
#ifndef WPK_VARIANTS_FILE
#define WPK_VARIANTS_FILE "wpk_variants.def"
#endif

namespace wpk {

// ---- gene value lists (the search sees index ranges into them) -------------------------------
extern const int32_t kBmVals[4];     // 32 (the wave-split members), 64, 128, 256
extern const int32_t kBnVals[3];     // 32, 64, 128
extern const int32_t kBkVals[3];     // 8, 16, 32
extern const int32_t kWmVals[3];     // 1, 2, 4
extern const int32_t kWnVals[3];     // 1, 2, 4
extern const int32_t kSplitVals[18]; // 1 .. 16, 20, 24
extern const int32_t kRemapVals[2];  // 0, 1
extern const int32_t kStageVals[3];   // 1, 2, 3 tiles in flight in registers
extern const int32_t kReduceVals[2];  // 0 workspace, 1 atomics
extern const int32_t kPersistVals[5]; // 0 (off), 1, 2, 3, 4 workgroups per compute unit
extern const int kGeneCounts[WPK_N_GENES];
const int32_t *gene_values(int g);

// Reduction entries are padded up to a multiple of kRedAlign rows (the largest K-step) and
// packed output channels to a multiple of kKoutAlign (the largest channel tile), so tile loads
// of packed weights and of the tap table never need a bounds check.
static const int kRedAlign = 32;
static const int kKoutAlign = 128;
// Per pixel, filter rows and columns outside the image are tracked in one 32-bit mask: bits
// 0..15 for rows, bits 16..30 for columns, bit 31 reserved as "always outside" for the padded
// reduction rows.  So the tiled family takes filters up to 16 rows by 15 columns.
static const int kMaxFilterRows = 16;
static const int kMaxFilterCols = 15;
static const int kPadTapBit = 31;
static const int kNumXcd = 8;
// Members with this pixel tile are the wave-split form (wpk_wsplit.h): their wm x wn waves cut the
// reduction between them, bk is the octet they work in, and `stages` counts four octets in flight each.
static const int kWaveSplitBm = 32;
// Floats of LDS that their waves meet in: every wave's partial tile of 32 pixels and bn channels (none for one wave, whose
// slices leave a word there).
constexpr int wave_split_floats(int bn, int waves) { return waves > 1 ? waves * bn * 32 : 4; }
// Tiled members whose waves all lie along the channels (wm = 1) are the split form (wpk_split.h): fp32
// products formed on the bf16 matrix pipes, weights packed as three bf16 parts (kSplitWeightBytes each).
inline bool split_member(const wpk_conv_config &c) { return c.bm != kWaveSplitBm && c.wm == 1; }
static const int kSplitWeightBytes = 6;
static const int64_t kMaxSplitBytes = 0xffff0000;  // (their offsets are unsigned: every layer whose plain weights fit does)
// Positions of x that the split members' patch form holds at most (two patches of 112 bytes each in LDS: 84 KB).
static const int kHaloMax = 384;
// LDS per workgroup: two stages of (BM + BN) columns of BK + 4 floats; two workgroups of the
// largest tile still fit the 160 KB of a compute unit.
static const int kMaxLdsBytes = 80 * 1024;
// Tensors are addressed with 32-bit byte offsets through buffer descriptors.
static const int64_t kMaxTiledBytes = 0x7fffffff;

// ---- one compiled tile combination -------------------------------------------------------------
struct Variant {
    int32_t bm, bn, bk, wm, wn, stages;
    const char *name;
};
extern const Variant kVariants[];
extern const int kNumVariants;
int find_variant(int bm, int bn, int bk, int wm, int wn, int stages);  // index or -1

// Layers of few channels on the split members (wpk_strip.h): strips of whole output rows, the rows of x under them in LDS.
struct StripShape {
    int32_t depths;     // MFMA depths of two filter rows each; 0: not so
    int32_t pairs;      // columns / 2 that a row of the strip has room for
    int32_t rows;       // output rows of a strip
    int32_t lds;        // bytes
    int32_t waves_c;    // waves side by side along the channels
    int32_t per_group;  // groups of 32 * waves_c channels that a workgroup does
    double us;          // what a launch is estimated to take
};

// ---- everything derived from one descriptor ------------------------------------------------------
struct Problem {
    wpk_conv_desc d;
    int32_t P, Q;
    int64_t M;       // N*P*Q output pixels (GEMM columns)
    int32_t CRS;     // reduction length
    int32_t CRSpad;  // rounded up to kRedAlign
    int32_t Kpad;    // K rounded up to kKoutAlign
    int64_t x_elems, w_elems, y_elems;
    bool tiled_ok;   // the tiled family can run it (else only the direct kernel)
    bool xl, yl;     // x / y channels-last (bits 0 and 1 of the descriptor's layout)
    bool xquad;      // channels-last x gathered as 16-byte channel quads (C a multiple of every K-step)
    bool tapmajor;   // x [N][C][H][W] with C a multiple of every K-step: reduction ordered (r, s, c) as well
    bool padtaps;    // neither, but the split members pad C and order the reduction by taps (split_taps)
    StripShape strip;  // of a prepared layer (prepare_strip), depths 0 before
};
int make_problem(const wpk_conv_desc *d, Problem *out);  // WPK_OK or a WPK_E_* code
// The first or last `images` images of a problem, to be run on weights that were packed for the whole of it: whether channels are padded
// depends on the number of images too (offsets), and the packed order is that of the whole.
int make_part(const Problem &whole, int images, Problem *out);
std::string desc_key(const wpk_conv_desc *d);

// Division of a 31-bit number by a launch constant as a multiply, an add and a shift (the
// divisor's multiplier is computed on the host): with L = ceil(log2 d) and
// mul = floor(2^32 * (2^L - d) / d) + 1, q = (mulhi(n, mul) + n) >> L is exact for every
// n < 2^31 and every d >= 1 (d = 1 and powers of two give mul = 1, which adds nothing), and the
// sum cannot overflow 32 bits because mulhi(n, mul) <= n.
struct FastDiv {
    uint32_t mul, sh;
};
inline FastDiv make_fastdiv(uint32_t d)
{
    uint32_t L = 0;
    while ((1ull << L) < d) ++L;
    FastDiv f = {(uint32_t)((((uint64_t)1 << 32) * ((1ull << L) - d)) / d + 1), L};
    return f;
}

// Persistent launches: the reduction steps of the tiles beyond the last whole round (`units` of
// them) are dealt to the first `streamk_groups` of the G workgroups in runs of equal length (+-1).
// A run over fewer than kMinRunRows reduction rows does not repay its prologue and its part in
// the fix-up (measured on the 56x56 layer of 64 channels: 45 us per launch with runs of 64-96
// rows against 49-59 us with runs of one or two K-steps of 16), so fewer workgroups take part
// when there is little to deal out.
static const int kMinRunRows = 64;
inline int64_t streamk_groups(int64_t units, int64_t G, int rows)
{
    if (units <= 0) return 0;
    int64_t min_steps = kMinRunRows / rows > 1 ? kMinRunRows / rows : 1;
    int64_t want = units / min_steps;
    return want < 1 ? 1 : want < G ? want : G;
}

// Kernel argument block of the tiled implicit-GEMM family (passed by value).
struct IgemmArgs {
    const float *x;
    const float *wp;      // packed weights [CRSpad/4][Kpad][4]; split members: [CRSpad/16][Kpad/32][3 parts][64 lanes][8 bf16]
    float *y;
    const int32_t *ktab;  // periodic tap table [R*S phases][32 rows][2]: byte offset relative to the
                          // step's channel base (biased); mask bit of r | mask bit of s << 8
    const int32_t *ttab;  // the same for the 32 rows from the start of the last reduction step, exact
    int32_t N, C, H, W, K, Q, R, S;
    int32_t stride_h, stride_w, pad_h, pad_w, dil_h, dil_w;
    int32_t M, PQ, HW, CRS, Kpad;
    int32_t RS, HW4;               // R*S, H*W*4
    int32_t bk_div_rs, bk_mod_rs;  // BK / RS, BK % RS
    int32_t nsteps, steps_per_split, split_k;
    int32_t tiles_m, tiles_n, remap;
    int32_t persist;       // 0, or persistent workgroups per compute unit
    int32_t grid_persist;  // persist * compute units
    int32_t runners;       // persistent: workgroups appended to the grid that do a dealt-out run and nothing else
                           // (set by the launcher: sk_groups, or 0 when the first sk_groups workgroups do their run
                           // themselves)
    uint32_t x_bytes;   // size of x
    uint32_t x_bias;    // (pad_h*W + pad_w)*4: added to every tap offset, subtracted from the base
    uint32_t w_bytes;   // size of the packed weights
    uint32_t y_bytes;   // size of y (and of a residual)
    // fix-up workspace of shared tiles (NULL = accumulate with atomics into zeroed y instead)
    float *ws;          // [shared tiles][ws_maxc slots][BM*BN] partial tiles
    int32_t *ws_cnt;    // [shared tiles] arrival counters, zero between launches
    int32_t ws_maxc;    // slots per shared tile
    // fused epilogue, applied where y is stored plainly: y = act(acc + bias[k] + res[n][k][p][q])
    const float *bias;  // [K] or NULL
    const float *res;   // laid out like y, or NULL
    int32_t relu;       // act = max(., 0) when nonzero
    // launch constants of the work iterator and their fast divisors
    int32_t tiles;      // tiles_m * tiles_n
    int32_t tiles_dp;   // persistent: tiles done whole, floor(tiles / G) * G
    int32_t sk_groups;     // persistent: how many workgroups (the first ones) share out the other tiles' steps,
    int32_t sk_q, sk_rem;  // in runs of sk_q steps (+1 for the first sk_rem)
    FastDiv div_pq, div_q, div_tiles_n, div_tiles, div_nsteps, div_q1, div_q0;  // by PQ, Q, tiles_n,
                        // tiles, nsteps, sk_q + 1, max(sk_q, 1)
    FastDiv div_tap;    // by what a reduction row index is divided to find its first table entry: C where a
                        // K-step lies inside one filter tap, else R*S (split members: R*S, or H*W if halo)
    int32_t mfast;      // order of the tiles: 0: tile = tile_m * tiles_n + tile_n (neighbours in the order share rows
                        // of x); 1: tile = tile_n * tiles_m + tile_m (neighbours share weights) -- whichever operand is
                        // the larger, since with XCD-contiguous ranges the other one is what every XCD fetches whole
    FastDiv div_tiles_m;  // by tiles_m
    FastDiv div_s;        // by S (the wave-split members find their first filter tap with it)
    int32_t xl;         // 0: x is [N][C][H][W]; 1: channels-last, gathered row by row; 2: channels-last,
                        // gathered as 16-byte channel quads (reduction rows ordered (r, s, c)); 3: [N][C][H][W]
                        // with the reduction ordered (r, s, c), one filter tap per step
    int32_t yl;         // 1: y (and the residual) are channels-last; 2: also K % 4 == 0 and y, residual and
                        // bias 16-byte aligned, so a pixel's channel quads move as 16-byte accesses
    int32_t halo;       // split members: positions of x the patch of a 3x3 tile holds, 0: each tap fetched by itself, -1: a
                        // 1x1 layer fetched four pixels at a time (split_point), -2: strips (wpk_strip.h)
    int16_t producers;     // split members: waves of a workgroup that fetch,
    int16_t two_per_unit;  // and whether no compute unit gets more than two workgroups
};

// What follows the convolution inside the same launch (Section 2.1, operator fusion).
struct Epilogue {
    const float *bias = nullptr;
    const float *res = nullptr;
    int relu = 0;
    bool any() const { return bias || res || relu; }
};

static const int64_t kFixupCounterBytes = 1 << 20;   // room for 262144 shared tiles
static const int64_t kFixupMaxBytes = (int64_t)1 << 30;  // default cap; beyond it, atomics
extern std::atomic<int64_t> g_workspace_limit;  // wpk_set_workspace_limit()
// Fix-up workspace a launch of `cfg` needs (split reduction or persistent): shared tiles, slots per tile, bytes
// (a fixed-size counter region first, then the slots).  All zero when nothing is shared or the
// workspace would be too large (the launch then accumulates with atomics).
struct FixupNeed {
    int64_t shared_tiles, maxc, bytes, slots_offset;
};
FixupNeed fixup_need(const Problem &pr, const wpk_conv_config &cfg, int compute_units);

// host-side state shared between wpk_host.cpp and wpk_api.hip
void set_last_hip_error(int e);
void set_device_name(const std::string &name);
std::string device_name();
bool legal_for(const Problem &pr, const wpk_conv_config &cfg);
// Bound on the positions of x that the windows of bm consecutive output pixels cover, where a split member with a
// K-step of 16 (any K-step where C is no multiple of 32) works from such a patch (3x3 filters, ordinary padding, at most
// kHaloMax positions); else 0.
int halo_positions(const Problem &pr, const wpk_conv_config &cfg);
#ifdef __HIP__
#define WPK_HOST_DEVICE __host__ __device__
#else
#define WPK_HOST_DEVICE
#endif
// First position of x (numbered through the images) that a tap of a 3x3 tile's pixels can touch: that of the first pixel's
// window, (n, p, q), clipped to the image -- unless the row below is clipped to the same row, where a later pixel's
// window begins further left.
WPK_HOST_DEVICE inline int patch_first(int n, int p, int q, int stride_h, int stride_w, int pad_h, int pad_w, int H, int W)
{
    const int r = p * stride_h - pad_h, c = q * stride_w - pad_w;
    return (n * H + (r > 0 ? r : 0)) * W + (r + stride_h > 0 && c > 0 ? c : 0);
}
// The last one alike, from the last pixel.
WPK_HOST_DEVICE inline int patch_last(int n, int p, int q, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h,
                                      int dil_w, int H, int W)
{
    const int r = p * stride_h - pad_h + 2 * dil_h, c = q * stride_w - pad_w + 2 * dil_w;
    return (n * H + (r < H - 1 ? r : H - 1)) * W + (r - stride_h < H - 1 && c < W - 1 ? c : W - 1);
}
// Whether the split members order pr's reduction by filter taps, (c / 32, r, s, c % 32): where the tiled members do, and where padding
// C to whole groups of 32, of 16 where they work from patches, lengthens it by half at most and the layer does not fit strips.  The weights of the padding are
// zero, and what is fetched for it lies in x (wpk_split.h): what is finite adds nothing, and what is not has the tile
// computed again.
inline bool split_taps(const Problem &pr) { return pr.tapmajor || pr.xquad || pr.padtaps; }
// MFMA depths of pr on the strip form of the split members, 0 where it does not fit that.
int strip_depths(const Problem &pr);
static const int64_t kMaxStripGroups = 0xffffff;  // workgroups of a launch
// Whether cfg runs pr in strips.  Where pr fits them, the split members' configurations of K-step 16 without slices or persistent
// workgroups do (a strip has the whole reduction, and a workgroup its own strips); the others go row by row, as the caller asked for.
// So do more output rows than a launch has workgroups of 256 threads for, 2^32 threads in all (strips of one row each, one group of channels).
inline bool runs_strip(const Problem &pr, const wpk_conv_config &cfg)
{
    return split_member(cfg) && cfg.bk == 16 && cfg.split_k == 1 && cfg.persist == 0 && strip_depths(pr) > 0 &&
           (int64_t)pr.d.n * pr.P <= kMaxStripGroups;
}
// Rows of the reduction as the split members pack it: where pr fits strips, those in the strips' order and then those in the source's.
inline int64_t split_rows(const Problem &pr)
{
    if (const int depths = strip_depths(pr)) return depths * 16 + pr.CRSpad;
    return split_taps(pr) ? (int64_t)((pr.d.c + 31) / 32 * 32) * pr.d.r * pr.d.s : pr.CRSpad;
}
// Whether a split member fetches pr's x four neighbouring pixels at a time: 1x1 filters on [N][C][H][W] in the order of taps,
// stride 1, no padding, images of a multiple of four pixels.
inline bool split_point(const Problem &pr)
{
    const wpk_conv_desc &d = pr.d;
    return !pr.xl && split_taps(pr) && d.r == 1 && d.s == 1 && d.stride_h == 1 && d.stride_w == 1 && d.pad_h == 0 && d.pad_w == 0 &&
           (int64_t)d.h * d.w % 4 == 0;
}
// Byte offset of channel ch in an image of [N][C][H][W], HW4 bytes per channel.  Chunks of 16 channels may run past the
// last one: what is fetched there is the last channel (its weights are zero).  (Unsigned: split_taps keeps ch below 3/2 C, so
// with C * HW4 below 2^31 the product is below 2^32, but not always below 2^31.)
WPK_HOST_DEVICE inline uint32_t patch_channel_at(int ch, int C, int HW4)
{
    const uint32_t at = (uint32_t)ch * (uint32_t)HW4, last = (uint32_t)(C - 1) * (uint32_t)HW4;
    return at < last ? at : last;
}
// The split members' weights lie depth by depth (16 rows of the reduction); step `step` of the reduction multiplies depths
// split_depth(patch, step, 0), (.., 1), ...  A step is two depths that follow each other, or with a patch the nine taps of
// sixteen channels: the two halves of 32 channels alternate (pack_split_kernel).
WPK_HOST_DEVICE constexpr int split_depth(bool patch, int step, int t)
{
    return patch ? (step >> 1) * 18 + (step & 1) + 2 * t : step * 2 + t;
}
// Byte offset of a step's first depth for the 32 channels that start at `block` in the first depth of all.  A wave asks for
// weights two depths ahead of those it multiplies, past the last step as well (nobody reads these): there the last step's are
// fetched again, since the whole offset is a scalar one and a buffer's range check does not cover that.
WPK_HOST_DEVICE inline uint32_t split_weights_at(bool patch, uint32_t block, int step, int nsteps, uint32_t depth_bytes)
{
    return block + (uint32_t)split_depth(patch, step < nsteps ? step : nsteps - 1, 0) * depth_bytes;
}
// The shape that pr's strips have: the prepared one, or priced for this many compute units.  Pricing takes 1 us (one group of
// channels) to 5 (K = 4096), so what is run again and again is prepared once.
StripShape strip_shape(const Problem &pr, int compute_units);
void prepare_strip(Problem *pr, int compute_units);
// Waves of a split member's workgroup that fetch and split activations.
int split_producers(const Problem &pr, const wpk_conv_config &cfg, int compute_units);
// LDS that such a workgroup takes, in the units of 1280 bytes (128 per compute unit) it is given out in.
int split_lds_units(int halo, int wn);
// Where outputs lie in y (and in a residual laid out alike), as the offsets of buffer accesses.  A lane of no output gets
// kNowhere: past every tensor (they are smaller than 2 GiB), a multiple of four, and still past all of them with any
// existing channel's offset added.
static const uint32_t kNowhere = 0x80000000u;
// Byte offset of channel k of pixel m, number pq of image n; M pixels, K channels; channels-last where yl.  (Of a channel past the
// last one it says nothing: see output_at.)
WPK_HOST_DEVICE inline uint32_t output_place(int m, int M, int n, int pq, int k, int K, int PQ, bool yl)
{
    const uint32_t at = yl ? (uint32_t)m * (uint32_t)K + (uint32_t)k : ((uint32_t)n * (uint32_t)K + (uint32_t)k) * (uint32_t)PQ + (uint32_t)pq;
    return m < M ? at * 4u : kNowhere;
}
// The same for channel k + dk, from channel k's; ch4: bytes between channels.
WPK_HOST_DEVICE inline uint32_t output_at(uint32_t place, int k, int dk, int K, uint32_t ch4)
{
    return k + dk < K ? place + (uint32_t)dk * ch4 : kNowhere;
}
// The same as the lane's and the wave-uniform part of an access.  WHOLE: every channel of the block exists; then the channel's offset
// may be the uniform part, below 2^31 as it lies inside y.  That of a channel past the last one may be anything (31 channels
// of 4200 x 4200 pixels are 2.2e9 bytes), and a buffer's range check does not cover the uniform part.
struct OutputAccess {
    uint32_t lane, uniform;
};
template <bool WHOLE>
WPK_HOST_DEVICE inline OutputAccess output_access(uint32_t place, int k, int dk, int K, uint32_t ch4)
{
    return WHOLE ? OutputAccess{place, (uint32_t)dk * ch4} : OutputAccess{output_at(place, k, dk, K, ch4), 0};
}
// What a configuration counts the reduction in: K-steps, or chunks of 16 channels where it works from patches.
struct Reduction {
    int32_t steps, rows;  // how many, and how many rows of the reduction each holds
};
Reduction reduction_of(const Problem &pr, const wpk_conv_config &cfg);
// Persistent workgroups per compute unit a launch of cfg has, 0 where it runs one workgroup per tile and slice.
int persistent_of(const Problem &pr, const wpk_conv_config &cfg, int compute_units);
// The configuration that stands for all those that make the same launch as cfg: split members have no prefetch depths, K-steps
// only where they decide about patches, and slices and persistent schedules that come out as another's.
wpk_conv_config same_launch(const Problem &pr, const wpk_conv_config &cfg, int compute_units);
// (plain: of a launch without an epilogue.  The two differ in the wave-split members' slices and how they meet.)
void default_config(const Problem &pr, int compute_units, wpk_conv_config *out, bool plain = true);
// Whether the wave-split members can run pr at all and its 32 x 32 output blocks times its octets of
// reduction rows stay within the bound (the work is then small enough for them to be worth timing).
bool wave_split_candidate(const Problem &pr, int64_t max_block_octets);

}  // namespace wpk
#endif
