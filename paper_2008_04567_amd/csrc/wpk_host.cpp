// Host-only part of libwpk: descriptor validation, the configuration (chromosome) encoding and
// its constraint check, the search-result cache and the genetic search engine.  No HIP calls.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <charconv>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "wpk_internal.h"

namespace wpk {

const int32_t kBmVals[4] = {32, 64, 128, 256};
const int32_t kBnVals[3] = {32, 64, 128};
const int32_t kBkVals[3] = {8, 16, 32};
const int32_t kWmVals[3] = {1, 2, 4};
const int32_t kWnVals[3] = {1, 2, 4};
const int32_t kSplitVals[18] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 20, 24};
const int32_t kRemapVals[2] = {0, 1};
const int32_t kPersistVals[5] = {0, 1, 2, 3, 4};
const int32_t kStageVals[3] = {1, 2, 3};
const int32_t kReduceVals[2] = {0, 1};
const int kGeneCounts[WPK_N_GENES] = {4, 3, 3, 3, 3, 18, 2, 5, 3, 2};

const int32_t *gene_values(int g)
{
    switch (g) {
    case 0: return kBmVals;
    case 1: return kBnVals;
    case 2: return kBkVals;
    case 3: return kWmVals;
    case 4: return kWnVals;
    case 5: return kSplitVals;
    case 6: return kRemapVals;
    case 7: return kPersistVals;
    case 8: return kStageVals;
    case 9: return kReduceVals;
    }
    return nullptr;
}

#define WPK_STR2(x) #x
#define WPK_STR(x) WPK_STR2(x)
#define WPK_VARIANT(PART, BM, BN, BK, WM, WN, PD)                                                  \
    {BM, BN, BK, WM, WN, PD,                                                                       \
     "wpk_igemm_" WPK_STR(BM) "x" WPK_STR(BN) "x" WPK_STR(BK) "_" WPK_STR(WM) "x" WPK_STR(WN) "_p" WPK_STR(PD)},
const Variant kVariants[] = {
#include WPK_VARIANTS_FILE
};
#undef WPK_VARIANT
const int kNumVariants = (int)(sizeof(kVariants) / sizeof(kVariants[0]));

static int value_index(int g, int32_t v)
{
    const int32_t *vals = gene_values(g);
    for (int i = 0; i < kGeneCounts[g]; ++i)
        if (vals[i] == v) return i;
    return -1;
}

// (A table over the genes' values: every default of a layer that the model has to price asks 2400 times, and each time a
// search through all variants made that 40 to 120 us of host time per one-shot call.)
int find_variant(int bm, int bn, int bk, int wm, int wn, int stages)
{
    auto place = [](const int32_t (&v)[6]) {
        static const int genes[6] = {0, 1, 2, 3, 4, 8};
        int at = 0;
        for (int j = 0; j < 6; ++j) {
            const int i = value_index(genes[j], v[j]);
            if (i < 0) return -1;
            at = at * kGeneCounts[genes[j]] + i;
        }
        return at;
    };
    static const std::vector<int16_t> table = [&] {
        std::vector<int16_t> t(kGeneCounts[0] * kGeneCounts[1] * kGeneCounts[2] * kGeneCounts[3] * kGeneCounts[4] * kGeneCounts[8], -1);
        for (int i = 0; i < kNumVariants; ++i) {
            const Variant &v = kVariants[i];
            const int at = place({v.bm, v.bn, v.bk, v.wm, v.wn, v.stages});
            if (at >= 0 && t[at] < 0) t[at] = (int16_t)i;
        }
        return t;
    }();
    const int at = place({bm, bn, bk, wm, wn, stages});
    return at < 0 ? -1 : table[at];
}

static thread_local int g_last_hip_error = 0;
void set_last_hip_error(int e) { g_last_hip_error = e; }

// Written once by the first call that looks at the device, read by every cache access.
static std::mutex g_device_name_mu;
static std::string g_device_name = "unknown";
void set_device_name(const std::string &name)
{
    std::lock_guard<std::mutex> g(g_device_name_mu);
    g_device_name = name;
}
std::string device_name()
{
    std::lock_guard<std::mutex> g(g_device_name_mu);
    return g_device_name;
}

// Output extent along one axis by the floor rule; <= 0 if the dilated window does not fit.
static int64_t out_extent(int64_t in, int64_t pad, int64_t dil, int64_t win, int64_t stride)
{
    int64_t span = in + 2 * pad - dil * (win - 1) - 1;
    return span < 0 ? 0 : span / stride + 1;
}

static bool pads_to_taps(const Problem &pr);
int make_problem(const wpk_conv_desc *d, Problem *out)
{
    if (!d || !out) return WPK_E_NULL_PTR;
    if (d->n <= 0 || d->c <= 0 || d->h <= 0 || d->w <= 0 || d->k <= 0 || d->r <= 0 || d->s <= 0 ||
        d->stride_h <= 0 || d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0 || d->dil_h <= 0 ||
        d->dil_w <= 0)
        return WPK_E_BAD_DESC;
    if (d->dtype != WPK_F32 || d->layout < 0 || d->layout > WPK_NHWC) return WPK_E_UNSUPPORTED;
    int64_t P = out_extent(d->h, d->pad_h, d->dil_h, d->r, d->stride_h);
    int64_t Q = out_extent(d->w, d->pad_w, d->dil_w, d->s, d->stride_w);
    if (P <= 0 || Q <= 0) return WPK_E_BAD_DESC;
    Problem pr;
    pr.d = *d;
    pr.P = (int32_t)P;
    pr.Q = (int32_t)Q;
    pr.M = (int64_t)d->n * P * Q;
    int64_t crs = (int64_t)d->c * d->r * d->s;
    pr.x_elems = (int64_t)d->n * d->c * d->h * d->w;
    pr.w_elems = (int64_t)d->k * crs;
    pr.y_elems = pr.M * d->k;
    const int64_t lim = (int64_t)1 << 40;  // beyond this even the direct kernel is not offered
    if (pr.x_elems > lim || pr.w_elems > lim || pr.y_elems > lim || crs > (1 << 30))
        return WPK_E_UNSUPPORTED;
    pr.CRS = (int32_t)crs;
    pr.CRSpad = (int32_t)((crs + kRedAlign - 1) / kRedAlign * kRedAlign);
    pr.Kpad = (d->k + kKoutAlign - 1) / kKoutAlign * kKoutAlign;
    pr.xl = (d->layout & 1) != 0;
    pr.xquad = pr.xl && d->c % kRedAlign == 0;
    pr.tapmajor = !pr.xl && d->c % kRedAlign == 0;
    pr.yl = (d->layout & 2) != 0;
    int64_t bias = ((int64_t)d->pad_h * d->w + d->pad_w) * 4 * (pr.xl ? d->c : 1);
    pr.tiled_ok = d->r <= kMaxFilterRows && d->s <= kMaxFilterCols &&
                  pr.x_elems * 4 + bias <= kMaxTiledBytes &&
                  pr.y_elems * 4 <= kMaxTiledBytes && (int64_t)pr.CRSpad * pr.Kpad * 4 <= kMaxTiledBytes;
    pr.strip = StripShape();
    pr.padtaps = pads_to_taps(pr);
    *out = pr;
    return WPK_OK;
}

int make_part(const Problem &whole, int images, Problem *out)
{
    wpk_conv_desc d = whole.d;
    d.n = images;
    const int rc = make_problem(&d, out);
    if (rc == WPK_OK) out->padtaps = whole.padtaps;
    return rc;
}

// (every one-shot call makes one or two of these; snprintf took a microsecond for each)
std::string desc_key(const wpk_conv_desc *d)
{
    const int32_t fields[] = {d->n, d->c, d->h, d->w, d->k, d->r, d->s, d->stride_h, d->stride_w, d->pad_h, d->pad_w,
                              d->dil_h, d->dil_w, d->dtype, d->layout};
    char buf[15 * 12], *at = buf;  // eleven characters at most and a comma
    for (const int32_t f : fields) {
        if (at != buf) *at++ = ',';
        at = std::to_chars(at, buf + sizeof buf, f).ptr;
    }
    return std::string(buf, at);
}

static const int32_t *cfg_fields(const wpk_conv_config *c, int32_t f[WPK_N_GENES])
{
    f[0] = c->bm; f[1] = c->bn; f[2] = c->bk; f[3] = c->wm; f[4] = c->wn; f[5] = c->split_k;
    f[6] = c->xcd_remap;
    f[7] = c->persist;
    f[8] = c->stages;
    f[9] = c->reduce;
    return f;
}

// The constraint check of Step1 for the convolution kernel family.
bool legal_for(const Problem &pr, const wpk_conv_config &cfg)
{
    int32_t f[WPK_N_GENES];
    cfg_fields(&cfg, f);
    for (int g = 0; g < WPK_N_GENES; ++g)
        if (value_index(g, f[g]) < 0) return false;
    if (!pr.tiled_ok) return false;
    if (find_variant(cfg.bm, cfg.bn, cfg.bk, cfg.wm, cfg.wn, cfg.stages) < 0) return false;
    int threads = 64 * cfg.wm * cfg.wn;
    if (threads > 1024) return false;                                             // workgroup size
    if (cfg.bm == kWaveSplitBm) {
        // the wave-split members: tap-major reduction order only, one workgroup per tile and slice
        if (!(pr.tapmajor || pr.xquad) || cfg.persist != 0) return false;
        if (wave_split_floats(cfg.bn, cfg.wm * cfg.wn) * 4 > kMaxLdsBytes) return false;
    } else {
        if (2 * (cfg.bk + 4) * (cfg.bm + cfg.bn) * 4 > kMaxLdsBytes) return false;    // two LDS stages
        if (threads > cfg.bm && (cfg.bk * cfg.bm / threads) % 4 != 0) return false;   // whole k quads per thread
        if (split_member(cfg) && split_rows(pr) * pr.Kpad * kSplitWeightBytes > kMaxSplitBytes) return false;
    }
    int32_t nsteps = (pr.CRS + cfg.bk - 1) / cfg.bk;
    if (cfg.split_k > nsteps) return false;
    // the persistent schedule balances the reduction itself: no fixed slices; and it always maps
    // tiles and runs XCD-contiguously (the same speed as launch order within noise, a half to a
    // fifth of the L2 fill traffic: 43 -> 17 MB, 103 -> 20 MB, 94 -> 34 MB on the 64-, 128- and
    // 256-channel layers of the batched 3x3 workload), so the gene has one legal value there
    if (cfg.persist > 0 && (cfg.split_k != 1 || cfg.xcd_remap != 1)) return false;
    // how partial tiles meet is a choice only where tiles can be shared
    if (cfg.reduce != 0 && cfg.split_k == 1 && cfg.persist == 0) return false;
    int64_t tiles = ((pr.M + cfg.bm - 1) / cfg.bm) * ((pr.d.k + cfg.bn - 1) / cfg.bn);
    if (tiles * cfg.split_k > 0x7fffffff) return false;
    // the persistent schedule counts reduction steps of up to 4*CUs tiles in 32 bits
    if (cfg.persist > 0 && (int64_t)nsteps * 4096 > 0x7fffffff) return false;
    return true;
}

static int patch_bound(const Problem &pr)
{
    const wpk_conv_desc &d = pr.d;
    if (d.r != 3 || d.s != 3 || d.pad_h > 2 * (int64_t)d.dil_h || d.pad_w > 2 * (int64_t)d.dil_w) return 0;
    // From the first pixel's window to the last one's: 63 steps along the row, for every change of row
    // what the next row's start is further away than a step, for every change of image alike; then the window itself.
    const int64_t W = d.w, HW = (int64_t)d.h * W, PQ = (int64_t)pr.P * pr.Q, n = 64 - 1;
    const int64_t rows = (n + pr.Q - 1) / pr.Q, images = (n + PQ - 1) / PQ;
    const int64_t span = n * d.stride_w + rows * std::max<int64_t>(0, d.stride_h * W - (int64_t)pr.Q * d.stride_w) +
                         images * std::max<int64_t>(0, HW - pr.P * d.stride_h * W) +
                         2 * ((int64_t)d.dil_h * W + d.dil_w) + 1;
    return span <= kHaloMax ? (int)span : 0;
}

static bool pads_to_taps(const Problem &pr)
{
    if (pr.tapmajor || pr.xquad) return false;
    if (strip_depths(pr)) return false;  // (an order of their own: 22 channels of one filter row would be both)
    const int64_t C = pr.d.c, c16 = (C + 15) / 16 * 16, c32 = (C + 31) / 32 * 32;
    if (c32 * pr.d.r * pr.d.s * pr.Kpad * kSplitWeightBytes > kMaxSplitBytes) return false;
    const bool patch = patch_bound(pr) > 0;
    if (2 * (patch ? c16 : c32) > 3 * C) return false;
    // (offsets of the channels that fill the last group up)
    return (patch && !pr.xl) || (pr.d.n * c32 + 32) * pr.d.h * pr.d.w * 4 <= kMaxTiledBytes;
}

int halo_positions(const Problem &pr, const wpk_conv_config &cfg)
{
    if (!split_member(cfg) || !split_taps(pr) || ((pr.tapmajor || pr.xquad) && cfg.bk != 16)) return 0;
    return patch_bound(pr);
}

// MFMA depths of a strip and the columns / 2 its rows have room for, 0 depths where a layer does not fit.  (240 columns: what the kernel is
// instantiated for, one or two columns / 2 a lane, the second 56 lanes of them; wider rows were neither built nor measured.)
static int strip_fits(int C, int Q, int R, int S, int stride_w, int dil_h, int dil_w, int *pairs)
{
    const int64_t octets = (int64_t)C * R, columns = (int64_t)(Q - 1) * stride_w + 8 + (stride_w % 2 ? 2 : 0);
    if (octets > 22 || S < 2 || S > 8 || dil_w != 1 || columns > 240) return 0;
    *pairs = columns <= 128 ? 64 : 120;
    if (C * ((int64_t)(R - 1) * dil_h + 1) * *pairs * 12 > 78 * 1024) return 0;  // (a strip of one row)
    return octets <= 6 ? 3 : octets <= 10 ? 5 : octets <= 16 ? 8 : 11;
}

// A strip's rows: as few as keep all compute units busy with as little filling as possible.  The cost of a choice, in cycles, from
// what the kernel was measured to take: a workgroup's start and end, a row of x (per 64 columns / 2), a block of 32 pixels by 32
// channels; two workgroups share a compute unit and its matrix pipes.
static StripShape price_strip(const Problem &pr, int compute_units)
{
    const wpk_conv_desc &d = pr.d;
    const int N = d.n, C = d.c, P = pr.P, Q = pr.Q, K = d.k, R = d.r, stride_h = d.stride_h, dil_h = d.dil_h;
    StripShape best = {0, 0, 0, 0, 0, 0, 0.0};
    int pairs;
    const int depths = strip_fits(C, Q, R, d.s, d.stride_w, dil_h, d.dil_w, &pairs);
    if (depths == 0) return best;
    const int waves_c = K > 64 ? 4 : K > 32 ? 2 : 1, groups = (K + 32 * waves_c - 1) / (32 * waves_c);
    double least = 1e300;
    for (int rows = 1; rows <= P && rows <= 64; ++rows) {
        const int64_t lines = C * ((int64_t)(rows - 1) * stride_h + (int64_t)(R - 1) * dil_h + 1), lds = lines * pairs * 12;
        if (lds > 78 * 1024) break;
        const int64_t strips = (int64_t)N * ((P + rows - 1) / rows), blocks = ((int64_t)rows * Q + 31) / 32;
        const int64_t wave_blocks = (blocks + 4 / waves_c - 1) / (4 / waves_c);
        for (int per = groups; per >= 1; per = per == 1 ? 0 : (per + 1) / 2) {
            const int64_t work = strips * ((groups + per - 1) / per);
            if (work > kMaxStripGroups) continue;
            const double fill = 8000.0 + lines * ((pairs + 63) / 64) * 60.0;
            const double multiply = per * (1500.0 + wave_blocks * (depths * 225.0 + 1900.0));
            const double units = compute_units > 0 ? compute_units : 256;
            const double cost = ceil(work / (2 * units)) * fill + std::max(0.62 * ceil(work / units), 1.0) * multiply;
            if (cost < least) {
                least = cost;
                best = StripShape{depths, pairs, rows, (int32_t)lds, waves_c, per, 3.5 + cost / 2000.0};
            }
        }
    }
    return best;
}

StripShape strip_shape(const Problem &pr, int compute_units)
{
    return pr.strip.depths ? pr.strip : price_strip(pr, compute_units);
}

void prepare_strip(Problem *pr, int compute_units)
{
    if (strip_depths(*pr)) pr->strip = strip_shape(*pr, compute_units);
}

int strip_depths(const Problem &pr)
{
    const wpk_conv_desc &d = pr.d;
    int pairs;
    if (pr.tapmajor || pr.xquad || !pr.tiled_ok) return 0;
    const int depths = strip_fits(d.c, pr.Q, d.r, d.s, d.stride_w, d.dil_h, d.dil_w, &pairs);
    // (the weights' offsets, of both orders)
    return ((int64_t)depths * 16 + pr.CRSpad) * pr.Kpad * kSplitWeightBytes <= kMaxSplitBytes ? depths : 0;
}

int split_lds_units(int halo, int wn)
{
    return ((halo > 0 ? (halo + 1) * 224 : 30720) + 256 * wn + 4 + 1279) / 1280;
}

int split_producers(const Problem &pr, const wpk_conv_config &cfg, int compute_units)
{
    if (!split_member(cfg)) return 0;
    const int halo = halo_positions(pr, cfg);
    if (halo > 0) {
        // A second one wherever as many workgroups as with one fit a compute unit (twelve waves): 0.6 to 0.95 of the time with four or more
        // blocks of 64 positions, 0.9 to 1 with three.  Not where four workgroups fit: of three blocks one wave takes two
        // either way, and the four second waves are in the way (one multiplying wave each, 75 layers, median 1.02, up to 1.41); where no compute
        // unit gets more than two, they are not (0.95 to 1, one layer of 144 1.05; with more 0.88 to 1.14 on either side, 196 layers).
        const int fit = std::min(12 / (cfg.wn + 1), 128 / split_lds_units(halo, cfg.wn));
        const int64_t tiles = ((pr.M + cfg.bm - 1) / cfg.bm) * ((pr.d.k + cfg.bn - 1) / cfg.bn);
        const int persist = persistent_of(pr, cfg, compute_units), units = compute_units > 0 ? compute_units : 256;
        const bool few = persist > 0 ? persist <= 2 : tiles * cfg.split_k <= 2 * (int64_t)units;
        return (fit < 4 || few) && 12 / (cfg.wn + 2) >= fit ? 2 : 1;
    }
    if (pr.xl && split_taps(pr)) return cfg.wn == 4 ? 2 : 1;
    if (split_point(pr)) return cfg.wn == 4 || (cfg.wn == 2 && cfg.bk == 32) ? 2 : 1;
    return 2;
}

Reduction reduction_of(const Problem &pr, const wpk_conv_config &cfg)
{
    if (halo_positions(pr, cfg) > 0) return Reduction{(pr.d.c + 15) / 16, 9 * 16};
    if (runs_strip(pr, cfg)) return Reduction{1, strip_depths(pr) * 16};  // (strips have the whole of it)
    const int rows = split_member(cfg) ? 32 : cfg.bk;
    if (split_member(cfg) && split_taps(pr)) return Reduction{(int32_t)(split_rows(pr) / 32), 32};
    return Reduction{(pr.CRS + rows - 1) / rows, rows};
}

// A split member whose tiles make up one round that fills more than half of the persistent workgroups
// runs them whole, a workgroup each: dealing the steps of every tile out would have all of them meet in memory
// (3x3, 128 channels, 28x28, 16 images, 196 tiles on 256 compute units: 22.4 us whole, 28.7 dealt out).
int persistent_of(const Problem &pr, const wpk_conv_config &cfg, int compute_units)
{
    if (cfg.persist == 0 || !split_member(cfg)) return cfg.persist;
    const int64_t tiles = ((pr.M + cfg.bm - 1) / cfg.bm) * ((pr.d.k + cfg.bn - 1) / cfg.bn);
    const int64_t G = (int64_t)cfg.persist * (compute_units > 0 ? compute_units : 256);
    return tiles <= G && 2 * tiles > G ? 0 : cfg.persist;
}

wpk_conv_config same_launch(const Problem &pr, const wpk_conv_config &cfg, int compute_units)
{
    wpk_conv_config c = cfg;
    if (!split_member(cfg)) return c;
    c.stages = 1;
    if (runs_strip(pr, cfg)) return wpk_conv_config{64, 64, 16, 1, 2, 1, 1, 0, 1, 0};
    wpk_conv_config other = c;
    other.bk = 16;
    if (strip_depths(pr)) c.bk = 32;  // (row by row; what is a round of whole tiles has neither slices nor persistent workgroups below)
    else if (halo_positions(pr, other) == halo_positions(pr, c) && split_producers(pr, other, compute_units) == split_producers(pr, c, compute_units)) c.bk = 16;
    if (c.persist > 0 && persistent_of(pr, c, compute_units) == 0) {
        c.persist = 0;
        c.reduce = 0;
    }
    if (c.split_k > 1) {
        const int steps = reduction_of(pr, c).steps, per = (steps + c.split_k - 1) / c.split_k;
        c.split_k = (steps + per - 1) / per;
        if (value_index(5, c.split_k) < 0) c.split_k = cfg.split_k;  // (no such gene)
        if (c.split_k == 1) c.reduce = 0;
    }
    return c;
}

// Workspace of the persistent schedule's fix-up: the tiles beyond the last whole round are shared;
// a tile of nsteps consecutive units cut into runs of at least q units meets at most
// ceil((nsteps-1)/q) + 1 runs (every run holds one unit when there are fewer units than runs).
std::atomic<int64_t> g_workspace_limit{kFixupMaxBytes};

FixupNeed fixup_need(const Problem &pr, const wpk_conv_config &cfg, int compute_units)
{
    FixupNeed n = {0, 0, 0, 0};
    if (cfg.reduce != 0) return n;  // atomics asked for
    if (compute_units <= 0) compute_units = 256;
    int64_t tiles = ((pr.M + cfg.bm - 1) / cfg.bm) * ((pr.d.k + cfg.bn - 1) / cfg.bn);
    const Reduction red = reduction_of(pr, cfg);
    const int64_t nsteps = red.steps;
    if (const int persist = persistent_of(pr, cfg, compute_units)) {
        // tiles of the last partial round, their steps dealt in runs of q or q+1 to at most G
        // workgroups: a tile's nsteps steps meet at most ceil((nsteps-1)/q)+1 runs, and never
        // more than nsteps
        int64_t G = (int64_t)persist * compute_units;
        int64_t shared = tiles - tiles / G * G;
        if (shared == 0 || nsteps <= 1) return n;
        int64_t q = shared * nsteps / streamk_groups(shared * nsteps, G, red.rows);
        n.shared_tiles = shared;
        n.maxc = q > 0 ? std::min<int64_t>(nsteps, (nsteps - 1 + q - 1) / q + 1) : nsteps;
    } else {
        // every tile is shared by its non-empty reduction slices
        int64_t per = (nsteps + cfg.split_k - 1) / cfg.split_k;
        int64_t slices = (nsteps + per - 1) / per;
        if (slices <= 1) return n;
        n.shared_tiles = tiles;
        n.maxc = slices;
    }
    // the counters sit in a region of fixed size at the front, so that buffers reused between
    // configurations never find slot data where counters are expected
    n.slots_offset = kFixupCounterBytes;
    n.bytes = n.slots_offset + n.shared_tiles * n.maxc * cfg.bm * cfg.bn * 4;
    if (n.shared_tiles * 4 > kFixupCounterBytes || n.bytes > g_workspace_limit.load(std::memory_order_relaxed))
        n = FixupNeed{0, 0, 0, 0};  // use atomics
    return n;
}

// Untuned default, distilled from exhaustive searches over the layer shapes of the workloads:
// 32x32 wave tiles in 64-pixel workgroup tiles with the largest K-step win or come within a few
// percent nearly everywhere, provided the launch has 3-4 workgroups per compute unit; where the
// tiles alone do not give that many, the reduction is split, and many small slices add up with
// atomics rather than through the workspace.  Falls back to a crude cost model over all
// variants if that choice is illegal for the shape.
static void model_config(const Problem &pr, int compute_units, wpk_conv_config *out);
bool wave_split_candidate(const Problem &pr, int64_t max_block_octets)
{
    if (!(pr.tapmajor || pr.xquad)) return false;
    const int64_t blocks = ((pr.M + 31) / 32) * ((pr.d.k + 31) / 32), octets = pr.CRS / 8;
    return blocks * octets <= max_block_octets;
}
static bool wave_split_default(const Problem &pr, int compute_units, bool plain, wpk_conv_config *out)
{
    if (!wave_split_candidate(pr, 20000)) return false;
    const int64_t blocks = ((pr.M + 31) / 32) * ((pr.d.k + 31) / 32), octets = pr.CRS / 8;
    // As many waves per tile (four at most) as leave every wave two octets and keep the launch within two waves per SIMD
    // (1x1, 256 -> 128 channels, 56x56, N = 1, 392 tiles: 5.4 us with four, 7.1 with two), or within one where they would get
    // fewer than four (3x3, 32 channels); many tiles of one short run take a wave each (64 -> 256, 56x56: 4.3, with two 4.8).
    int wk = 4;
    while (wk > 1 && (octets / wk < 2 || blocks * wk > (octets / wk >= 4 ? 8 : 4) * (int64_t)compute_units)) wk /= 2;
    if (octets <= 8 && blocks > 2 * (int64_t)compute_units) wk = 1;
    // The reduction is cut until there is one wave per SIMD, but not into runs of fewer than ten octets (five for eight tiles
    // or fewer, whose slices meet sooner): the meeting through the workspace takes as long as eight or so (1x1, 512 -> 2048
    // channels, 7x7, N = 1: 5.1 us in one, 6.1 in two; 512 -> 128 at 28x28: 5.1, 5.9; 3x3, 512 channels, 7x7: 8.4 in eight).
    // With an epilogue, atomics take two more launches, y zeroed and the epilogue: 13.9 us for that layer, 9.5 without them.
    // (233 layers, ResNet-50 at N = 1 and 2 and drawn ones, bias and rectifier fused: 1.4 % above the best of all
    // waves, slices and channels on average, 8 by more than a tenth; by the rule below: 3.2 %, 28.)
    const int64_t most = std::max<int64_t>(1, 4 * (int64_t)compute_units / (blocks * wk));
    auto slices = [&](int64_t cap, int64_t run) {
        int64_t n = std::min(cap, most);
        while (n > 1 && octets / (wk * n) < run) --n;
        return n;
    };
    int64_t want = slices(24, blocks <= 8 ? 5 : 10);
    // Beyond eight slices what they cost decides: the last to arrive reads the others seven at a time, a round trip to memory each that
    // takes as long as six octets, and all of them store first.  (31 such layers of 180 to 3000 octets and 1 to 24 tiles in 2
    // to 24 slices, rectifier fused: 0.5 % above the best number on average, 8 % at worst; 3.3 and 10 for as many slices as
    // above, at most 16 or, for eight tiles or fewer, 24: 3x3, 17 tiles, 468 octets 8.1 us in eight, 8.6 in eleven; 5x5, five tiles, 1700
    // octets 10.4 in 16, 10.0 in 20, 9.9 in 24, and 9.0 or, with y zeroed for it alone, 10.3 by atomics.)
    if (want > 8) {
        double least = 1e300;
        for (int i = 0; i < kGeneCounts[5]; ++i) {
            const int64_t n = kSplitVals[i];
            if (n > std::min<int64_t>(24, most)) continue;
            const double cost = (double)octets / (wk * n) + 6.0 * ((n - 1 + 6) / 7) + blocks * n / 32.0;
            if (cost < least) {
                least = cost;
                want = n;
            }
        }
    }
    // Without one, atomics take the zeroing alone, and in a pass not even that (one launch for all layers): four slices or more add up
    // with them, and need eight octets only (layers in a pass, then by themselves, workspace and atomics: 3x3, 256 channels, 14x14, N = 1,
    // 8.2 and 7.2 us, 8.3 and 8.5; 5x5, 544 -> 32 channels, 12x12, N = 1, five tiles in 24 slices, 9.8 and 6.8, 9.7 and 8.1; 40
    // such layers, 1.18 and 1.02 times the atomics' time).  Three slices of eight octets meet in the workspace (3x3, 96
    // channels: 6.4, 6.8 in two); two are not worth it (six layers of 64 to 72 octets: 6.3 in two, 5.9 in one).
    // Not into channels-last outputs: 18 such layers, workspace 0.79 and 0.70 times the atomics' time, 1.2 at worst (289 pixels
    // of nine channels).
    bool atomics = false;
    if (plain && !pr.yl) {
        const int64_t n = slices(24, 8);
        if (n != 2) want = n;
        atomics = n >= 4;
    }
    wpk_conv_config c = {kWaveSplitBm, 32, 8, wk, 1, 1, 1, 0, 1, 0};
    for (int i = 0; i < kGeneCounts[5]; ++i)
        if (kSplitVals[i] <= want) c.split_k = kSplitVals[i];
    c.reduce = atomics ? 1 : 0;
    if (!legal_for(pr, c)) return false;
    *out = c;
    return true;
}
// What a launch of a split or a tiled member is estimated to take, in microseconds: the workgroups' chain of latencies, the
// matrix pipes, the memory and the way into a compute unit, their squares added up.  The constants are fitted to the
// measured times of 747 layers (ResNet-50 at N = 1 to 32 and layers drawn over the same ranges as those that the library's speed is
// measured on, bias and rectifier fused): 8600 launches of split members within 1.5 times the layer's best, off by 14 %
// (standard deviation), and one tiled default each, off by 11 %.  They are good for choosing between the two, no more.
static double split_time(const Problem &pr, const wpk_conv_config &c, int compute_units)
{
    const wpk_conv_desc &d = pr.d;
    const int halo = halo_positions(pr, c), wn = c.wn;
    const bool patch = halo > 0, point = !patch && split_point(pr), taps = !patch && !point && !pr.xl;
    const int producers = split_producers(pr, c, compute_units);
    const Reduction red = reduction_of(pr, c);
    const int per = (red.steps + c.split_k - 1) / c.split_k, slices = (red.steps + per - 1) / per;
    const int64_t tiles = ((pr.M + c.bm - 1) / c.bm) * ((d.k + c.bn - 1) / c.bn);
    const int64_t lds = split_lds_units(halo, wn);  // (of 128)
    const double resident = (double)std::min<int64_t>(128 / lds, 12 / (wn + producers));
    const double depths = per * (patch ? 9 : 2);
    const double fetched = patch ? (halo + 63) / 64 * 64 * 16 / 9.0 : 1024.0;  // elements split per depth
    const double start = patch ? 0.07 + 0.0063 * halo : point ? 0.15 : taps ? 1.2 : 0.99;
    const double depth = std::max(0.12, fetched / producers * 17e-5 + (taps ? 0.092 : 0.0));
    const double end = 4.5 + (slices > 1 ? 0.57 + 0.42 * slices : 0.0);
    const double n = (double)((tiles * slices + compute_units - 1) / compute_units);  // workgroups of the busiest compute unit
    const double chain = (start + depths * depth + end) * std::max(1.0, n / resident);
    const double pipes = n * depths * (wn * 0.25 + fetched * 20e-5) / 4 + start + end;
    const double memory = 4.0 * (pr.x_elems + pr.y_elems * (slices > 1 ? 1.0 + 2 * slices : 1.0)) / 4.0e6;
    const double way_in = n * depths * (wn * 3072 + (patch ? halo * 64 / 9.0 : 4096.0)) / 230e3 + start;
    return 0.08 + sqrt(chain * chain + pipes * pipes + memory * memory + way_in * way_in);
}
static double tiled_time(const Problem &pr, const wpk_conv_config &c, int compute_units)
{
    const wpk_conv_desc &d = pr.d;
    const int steps = (pr.CRS + c.bk - 1) / c.bk, per = (steps + c.split_k - 1) / c.split_k;
    const int slices = (steps + per - 1) / per;
    const int64_t tiles_m = (pr.M + c.bm - 1) / c.bm, tiles_n = (d.k + c.bn - 1) / c.bn;
    const bool atomics = c.reduce != 0 && slices > 1, dealt = c.persist == 1;
    const double all = (double)(tiles_m * tiles_n * slices) / compute_units;
    const double n = c.persist > 0 ? std::max(1.0, all) : ceil(all);
    // (steps of 32 rows; one persistent workgroup per compute unit shares them out evenly)
    const double depth = dealt ? (double)(tiles_m * tiles_n) * steps * c.bk / 32.0 / compute_units : per * c.bk / 32.0;
    const double ends = 1.8 + (slices > 1 && !atomics ? 1.2 + 0.029 * slices : 0.0) + (dealt ? 1.2 : 0.0);
    const double chain = (depth * (d.c % kRedAlign ? 0.457 : 0.38) + ends) * (dealt ? 1.0 : std::max(1.0, n / 1.4));
    const double pipes = depth * (dealt ? 1.0 : n) * 0.38 * c.wm * c.wn / 4 + ends;
    const double memory =
        4.0 * (pr.x_elems * (1 + 0.2 * (tiles_n - 1)) + pr.y_elems * (slices > 1 ? 1.0 + 2 * slices : 1.0)) / 7.7e6;
    // atomics: y zeroed ahead and the epilogue behind; into channels-last outputs they are slow
    const double y_mb = 4e-6 * pr.y_elems;
    return 2.9 + sqrt(chain * chain + pipes * pipes + memory * memory) +
           (atomics ? 5.7 + 3 * y_mb / 7.7 + (pr.yl ? 5.5 * y_mb * slices : 0.0) : 0.0);
}
// Whether tiles beyond whole rounds of two persistent workgroups per compute unit (taps: of one with four waves) are dealt out.  pairs: tiles of
// 64 pixels and channels; whole: what would be taken else, estimated to take us.  Times are of that.
static bool deals_out(const Problem &pr, int halo, bool taps, bool narrow, const wpk_conv_config &whole, double us, int64_t pairs, int steps,
                      int compute_units)
{
    const int64_t round = 2 * (int64_t)compute_units, beyond = pairs % round;
    // Two to two and a half tiles per compute unit.  (narrow: where whole tiles of 32 channels are priced a sixth faster, as with 96 or 160
    // channels, they stay: 0.78 to 1.18, 14 layers, half of them more.)
    if (pairs > round && 4 * pairs <= 5 * round && steps >= 4 && !narrow) {
        // patches: 0.85 on average, 138 layers, six slower by more than 3 %, two of them, against four and six slices of two waves, 1.11 and 1.26
        if (halo > 0) return true;
        // Taps against four waves: 0.87, 0.97 at worst, 77 layers.  Against two, of whose 128-wide tiles some channels are padding, with a stride, 0.89,
        // 11 layers; not without (1.03, up to 1.18, 22 layers; 32 to 320 channels, 5x5, 31x31, nine images, 28.8 us, 34.0 dealt out).  Not with up to 64
        // channels, where two of the waves have none (1.27 to 1.6, 42 layers; 3x3, stride 2, 32 to 64, 56x56, 48 images, 20.1 us, 30.7), nor 1x1
        // (1.03 to 1.14, 72 layers), nor below 16 steps (3x3, 32 to 100, 19.8, 22.6).
        if (taps)
            return pr.d.k > 64 && pr.d.r * pr.d.s > 1 && steps >= 16 && (whole.wn == 4 || pr.d.stride_h > 1 || pr.d.stride_w > 1);
        // Channels-last against four waves: 0.84 to 0.98, 105 layers, unless those in slices are estimated to be a quarter faster (1.04, 12
        // layers); against two, 0.95 from twelve steps on, 48 layers; below that 1.08, up to 1.34, 17 layers (160 to 160 channels, 1x1, 49x49, five images,
        // 11.3 us, 15.2 dealt out).
        const wpk_conv_config dealt = {64, 64, 32, 1, 2, 1, 1, 2, 1, 0};
        return whole.wn == 4 ? split_time(pr, dealt, compute_units) <= 1.35 * us : steps >= 12;
    }
    // Patches, more than four tiles per compute unit.  Against four waves (two tiles of 64 channels in one) 0.93 with less than half of a round left
    // over, 176 layers; with more, 0.95 with two steps, 43 layers, and 1.02 from three steps on, half of 99 layers slower by more than 3 %.  Against fewer waves 0.87
    // from five steps on, 101 layers, 0.96 with four, 59 layers; with two or three 0.95 where less than a quarter of a round is left over and the rounds are few, 1.01
    // elsewhere, 0.85 to 1.34, 73 layers (37 to 138 channels, 43x43, 61 images, 99.6 us, 117.8 dealt out).
    if (halo > 0 && pairs > 2 * round && steps >= 2)
        return whole.wn == 4 ? steps == 2 || 2 * beyond < round : steps >= 4 || (4 * beyond < round && pairs < 8 * round);
    return false;
}

// The split members' default, where they order the reduction by taps or take the layer in strips (row by row they gain nothing over
// the tiled members).  Waves of 64 pixels by 32 channels; patches where a 3x3 layer allows them.
//  - As many waves per workgroup as the channels call for, four at most: a wider workgroup fetches and splits its pixels
//    for more channels at once; what that is worth against padded channels is the weight of 20 / bn, from the measured
//    times of 64- and 128-channel tiles.  1x1 layers fetched four pixels at a time take two: fetching is cheap there, the
//    launch is bound by memory, and four small workgroups on a compute unit are out of step with each other where two
//    large ones fetch, multiply and store at the same time (256 to 128 channels, 56x56, 16 images: 29.5 us against 42;
//    256 to 1024 at 14x14: 15.3 against 21.4).
//    With up to two tiles of 64 channels per compute unit they take four waves and two that fetch, like the others (512 to 128 at 28x28, hot:
//    12.6 us, with two and one that fetches 16.3, two and two 15.2; 110 layers, 0.6 to 0.99 of the time), in slices only as far as each
//    compute unit gets one workgroup (1440 to 768 at 16x16, 7 images, in 3 slices of 168 workgroups 33.1, in two waves 29.5).  Not up to 32
//    channels (1.0 to 1.3, 7 layers), up to a quarter of a tile, where that makes eight slices and more (1.1 to 1.2, 5 layers), or where 65 to 96 channels
//    fit three 32-wide workgroups and there are fewer than 5 / 8 of a tile (0.99 to 1.09, 5 layers).
//  - The reduction is cut until there is about one wave per SIMD, no further: a second wave hides what a second
//    slice's prologue and meeting cost, no more (3x3, 256 channels, 14x14, 16 images, 98 tiles: 25.5 us in 2 slices,
//    27-30 in 1 or 3-5; 512 channels at 7x7, 52 tiles: 28.0 in 4, 28.7 in 3, 32.6 in 8).
//  - Any other number of waves or slices that is estimated to be faster by more than a fifth goes before that (3x3 layers of 260 to
//    340 tiles of two waves, one per compute unit and a few over: 175 -> 87 us in 3 slices, 832 to 448 channels at 10x10, N = 24).
//  - The tiled default stays where it is estimated to be faster by more than a tenth (the split members are the more exact), and
//    below 0.45 GFLOP, where it was faster for 78 of 84 measured layers -- but where it would sum with atomics into
//    channels-last outputs (up to four times as slow).
// (The two margins are where estimates that err cost least: with 5 and 10 % 23 of the 747 layers are slower than the tiled default by
// more than 10 % and 25 than by waves per SIMD alone, with these 27 and 12.)
// The tiled default was the faster one by more than 10 % for 139 of the 747 layers before the last two rules and is for 27 with
// them; of 730 others, drawn afterwards, for 122 and 30.  On average the split members, where chosen, and the tiled default elsewhere
// are 1.22 (1.27) times as fast as the tiled default alone, 1.14 (1.21) before.
static bool split_default(const Problem &pr, int compute_units, const wpk_conv_config &tiled, wpk_conv_config *out)
{
    const double flops = 2.0 * pr.M * pr.d.k * pr.CRS;
    if (strip_depths(pr)) {
        const wpk_conv_desc &d = pr.d;
        // Only where half of what is multiplied is no padding, S to eight and C * R to the depths: filters of five columns and more (two to four: 1.04
        // and 0.96 of the time of the tiled members, up to 1.41, 38 layers; five to eight 0.69 to 0.80, 188 layers).  Nor with short reductions and a
        // large y, which both forms wait for (up to ten octets, 100 MB and more: 0.57 to 1.30, 18 layers), nor where y leaves a lane four bytes
        // at a time (2 to 130 channels, channels-last, 403 us against 273).
        const int depths = strip_depths(pr);
        if (flops < 0.45e9 || (pr.yl && d.k % 4) || d.s < 5 || pr.CRS < 8 * depths || (depths <= 5 && pr.y_elems >= 25000000)) return false;
        *out = wpk_conv_config{64, 64, 16, 1, 2, 1, 1, 0, 1, 0};
        return runs_strip(pr, *out) && 1.1 * strip_shape(pr, compute_units).us < tiled_time(pr, tiled, compute_units) && legal_for(pr, *out);
    }
    if (!split_taps(pr)) return false;
    // (padded channels, but for patches of [N][C][H][W]: 46 to 128 channels, 5x5, 12x8, one image, 0.03 GFLOP, 17.8 us against 14.9 one shot; 300
    // to 224, 3x3, 12x16, 0.17 GFLOP, 14.8 against 26.7)
    const bool whole = pr.tapmajor || pr.xquad || (!pr.xl && patch_bound(pr) > 0);
    if (flops < 0.45e9 && !(pr.yl && tiled.reduce && (whole || flops >= 0.1e9))) return false;
    const int64_t pairs = (pr.M + 63) / 64 * ((pr.d.k + 63) / 64);
    // (and those of 1x1 filters fetched pixel by pixel, where there are many tiles of few steps: 1.0 to 1.45 of the time of the tiled members up to seven
    // steps of [N][C][H][W], 26 layers, 0.86 to 1.0 beyond, 20; channels-last up to two, 0.97 to 1.07; and of 17 to 23 channels and 5x5, 1.06 to 1.17, 3)
    if (!whole && !split_point(pr) && pairs > 2 * (int64_t)compute_units) {
        const int64_t steps = split_rows(pr) / 32, RS = (int64_t)pr.d.r * pr.d.s;
        if (RS == 1 ? steps < (pr.xl ? 3 : 8) : !pr.xl && pr.d.c < 24 && RS <= 25) return false;
    }
    const bool small_point = split_point(pr) && pr.d.k > 32 && pairs <= 2 * (int64_t)compute_units && 4 * pairs > compute_units &&
                             (pr.d.k <= 64 || pr.d.k > 96 || 8 * pairs >= 5 * (int64_t)compute_units);
    const bool point = split_point(pr) && !small_point;
    int wn = 4;
    double best = 1e300;
    for (int w = point ? 2 : 4; w >= 1; w /= 2) {
        const int bn = 32 * w;
        const double cost = (double)((pr.d.k + bn - 1) / bn * bn) * (1.0 + 20.0 / bn);
        if (cost < best) {
            best = cost;
            wn = w;
        }
    }
    wpk_conv_config c = {64, 32 * wn, 16, 1, wn, 1, 1, 0, 1, 0};
    const int halo = halo_positions(pr, c);
    if (halo == 0 && !point) c.bk = 32;
    const Reduction red = reduction_of(pr, c);
    const int64_t tiles = ((pr.M + c.bm - 1) / c.bm) * ((pr.d.k + c.bn - 1) / c.bn);
    const int64_t want = point ? 5 * (int64_t)compute_units / 2 : 4 / wn * (int64_t)compute_units;
    const int64_t G = 3 * (int64_t)compute_units;
    const bool taps = halo == 0 && !pr.xl;
    if (2 * tiles <= want) {
        // (slices of 64 rows at least, see kMinRunRows)
        const int64_t most = std::min<int64_t>(want / tiles, red.steps / std::max(1, kMinRunRows / red.rows));
        for (int i = 0; i < kGeneCounts[5]; ++i)
            if (kSplitVals[i] <= most) c.split_k = kSplitVals[i];
    } else if (tiles <= std::min(4 / wn, 2) * (int64_t)compute_units) {
        c.persist = std::min(4 / wn, 2);  // one round: whole tiles (persistent_of)
    }
    double time = split_time(pr, c, compute_units);
    wpk_conv_config other = c;  // the best by the model
    double least = 1e300;
    for (int w = point ? 2 : 4; w >= 1; w /= 2)
        for (const int slices : {1, 2, 3, 4, 5, 6, 8, 12}) {
            if (slices > red.steps) break;
            wpk_conv_config o = {64, 32 * w, c.bk, 1, w, slices, 1, 0, 1, 0};
            if (small_point && w == 4 && slices > 1 && (pr.M + 63) / 64 * ((pr.d.k + 127) / 128) * slices > compute_units) break;
            const double t = split_time(pr, o, compute_units);
            if (t < least) {
                least = t;
                other = o;
            }
        }
    const bool better = 1.2 * least < time, narrow = better && other.wn == 1 && other.split_k == 1;
    const wpk_conv_config whole_tiles = better ? other : c;  // what is taken where nothing is dealt out
    if (wn <= 2 && tiles > G && tiles < (point && wn == 2 ? 5 : 3) * G && tiles % G * 12 <= G &&
        (point ? red.steps >= 2 : halo > 0 && halo <= 240 && tiles % G * 20 <= G)) {
        // Just over one or two whole rounds of three workgroups per compute unit (1x1 layers of two waves: four): the tiles
        // left over are dealt out (3x3, 64 channels, 56x56, 16 images, 784 tiles: 25.0 us against 25.4 with a workgroup
        // per tile; 1x1, 256 to 128 channels, 1568 tiles: 29.5 against 31.4; -5 to +24 % over 35 such layers).  Beyond that,
        // with more tiles left over, patches of which three do not fit, taps or single steps it loses up to half.
        c.persist = 3;
        time *= 0.95;
    } else if (!point && pr.d.k > 32 && split_lds_units(halo, 2) <= 64 &&
               deals_out(pr, halo, taps, narrow, whole_tiles, better ? least : time, pairs, red.steps, compute_units)) {
        // Two persistent workgroups of two waves per compute unit, whose SIMDs then have one multiplying wave each, and the tiles beyond
        // whole rounds dealt out (deals_out).
        // Taps take one workgroup of four waves.
        c = wpk_conv_config{64, taps ? 128 : 64, c.bk, 1, taps ? 4 : 2, 1, 1, taps ? 1 : 2, 1, 0};
        time = 0.9 * std::min(time, split_time(pr, c, compute_units));
    } else if (better) {
        c = other;
        time = least;
    }
    // (channels-last with padded channels the tiled members fetch four bytes at a time and take 1.5 times their estimate, 483 layers: up to where the
    // split ones were estimated a fifth slower they took 0.47 of the time, 1.03 at worst)
    const double margin = pr.xl && pr.padtaps ? 1.2 : 1.1, tiled_us = tiled_time(pr, tiled, compute_units);
    if (time > margin * tiled_us || !legal_for(pr, c)) return false;
    if (taps && pr.padtaps && !split_point(pr)) {
        // Padded channels fetched pixel by pixel.  Up to 32 channels, where the fetched pixels serve a single wave: against tiled members that deal
        // tiles out, or add slices up by atomics into channels-last outputs, 0.60, 0.91 at worst, 30 layers; against others 0.99, up to 1.40, 74 layers (168
        // to 32, 5x5, stride 2, 43x22, 43 images, 51.4 us against 36.8), but 0.87, 1.10 at worst, without a stride where the estimate is by 13 % less.
        const bool strides = pr.d.stride_h > 1 || pr.d.stride_w > 1;
        if (pr.d.k <= 32 && tiled.persist != 1 && !(tiled.reduce && pr.yl) && (strides || time > 0.87 * tiled_us)) return false;
        // Above, up to three steps 1.08 to 1.24, 6 layers; with more than one and a half waves per SIMD only where the estimate is less: 1.05 where it
        // is not, up to 1.24, 34 layers.
        const int64_t waves = ((pr.M + 63) / 64) * ((pr.d.k + c.bn - 1) / c.bn) * c.wn * c.split_k;
        if (pr.d.k > 32 && (red.steps <= 3 || (c.persist == 0 && waves > 6 * (int64_t)compute_units && time > tiled_us))) return false;
    }
    *out = c;
    return true;
}
static void tiled_default(const Problem &pr, int compute_units, wpk_conv_config *out);
void default_config(const Problem &pr, int compute_units, wpk_conv_config *out, bool plain)
{
    if (compute_units <= 0) compute_units = 256;
    // A launch with a few microseconds of arithmetic at most (single images, late layers): the
    // wave-split members.  (Measured on the single-image ResNet-50 layers: 3.4-9.1 us where the tiled members' best
    // is 4.9-10.6.)
    if (wave_split_default(pr, compute_units, plain, out)) return;
    wpk_conv_config tiled;
    tiled_default(pr, compute_units, &tiled);
    if (!split_default(pr, compute_units, tiled, out)) *out = tiled;
}

static void tiled_default(const Problem &pr, int compute_units, wpk_conv_config *out)
{
    wpk_conv_config c = {64, pr.d.k <= 32 ? 32 : 64, pr.CRS >= 64 ? 32 : pr.CRS >= 32 ? 16 : 8, 2,
                         pr.d.k <= 32 ? 1 : 2, 1, 1, 0, 2, 0};
    int64_t tiles = ((pr.M + c.bm - 1) / c.bm) * ((pr.d.k + c.bn - 1) / c.bn);
    int64_t nsteps = (pr.CRS + c.bk - 1) / c.bk;
    // slices of at least four steps, enough of them for 3.5 workgroups per compute unit
    int64_t want = std::min<int64_t>((7 * (int64_t)compute_units / 2 + tiles / 2) / tiles, nsteps / 4);
    for (int i = 0; i < kGeneCounts[5]; ++i)
        if (kSplitVals[i] <= want) c.split_k = kSplitVals[i];
    // Just over a whole number of rounds of three workgroups per compute unit: persistent
    // workgroups run the rounds as whole tiles and deal out only the few tiles left over,
    // instead of a last round that leaves most of the device idle.
    int64_t G = 3 * (int64_t)compute_units;
    if (tiles > G && tiles % G != 0 && (tiles % G) * 8 <= G) {
        wpk_conv_config h = c;
        h.bk = pr.CRS >= 32 ? 16 : 8;
        h.split_k = 1;
        h.xcd_remap = 1;
        h.persist = 3;
        h.reduce = 0;
        if (legal_for(pr, h)) {
            *out = h;
            return;
        }
    }
    // Between one and two tiles per compute unit: one persistent workgroup per compute unit takes a
    // whole tile, the steps of the other tiles are dealt out in runs that proceed beside them (a
    // split reduction would share every tile instead of the remainder only).
    if (tiles > compute_units && tiles < 2 * (int64_t)compute_units && nsteps >= 8) {
        wpk_conv_config h = c;
        h.split_k = 1;
        h.xcd_remap = 1;
        h.persist = 1;
        h.reduce = 0;
        if (legal_for(pr, h)) {
            *out = h;
            return;
        }
    }
    // atomics where many slices meet in a small output (zeroing it is cheap and the last
    // workgroup need not read every slot); the workspace otherwise
    int64_t per = (nsteps + c.split_k - 1) / c.split_k, slices = (nsteps + per - 1) / per;
    c.reduce = (slices >= 5 && pr.y_elems * 4 <= (1 << 20)) || slices > 12 ? 1 : 0;
    if (legal_for(pr, c)) {
        *out = c;
        return;
    }
    model_config(pr, compute_units, out);
}

// Smallest estimated time under a crude model -- workgroups are dealt to the compute units in
// rounds, a workgroup costs its multiply-accumulate count plus a fixed per-step and
// per-workgroup overhead, small wave tiles pay for their operand re-reads and a split reduction
// pays for its extra passes over y.
static void model_config(const Problem &pr, int compute_units, wpk_conv_config *out)
{
    double best = 1e300;
    wpk_conv_config bc = {128, 64, 16, 2, 2, 1, 1, 0, 2, 0};
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        if (v.bm == kWaveSplitBm || v.wm == 1) continue;  // (the model prices fp32 LDS-staged tiles)
        for (int si = 0; si < kGeneCounts[5]; ++si) {
            wpk_conv_config c = {v.bm, v.bn, v.bk, v.wm, v.wn, kSplitVals[si], 1, 0, v.stages, 0};
            if (!legal_for(pr, c)) continue;
            double nsteps = ceil((double)pr.CRS / v.bk);
            double steps = ceil(nsteps / c.split_k);
            double tiles = ceil((double)pr.M / v.bm) * ceil((double)pr.d.k / v.bn);
            double blocks = tiles * c.split_k;
            double waves = v.wm * v.wn;
            double tm = v.bm / v.wm, tn = v.bn / v.wn;
            // MFMA cycles per step per SIMD (waves share the 4 SIMDs of a compute unit)
            double mfma = (double)v.bm * v.bn * v.bk / 2048.0 * 64.0 / std::min(4.0, waves);
            double operand = 1.0 + 16.0 * (1.0 / tm + 1.0 / tn);  // LDS operand traffic per MFMA
            double step_cost = mfma * operand + 220.0;
            double block_cost = steps * step_cost + 2500.0;
            double rounds = ceil(blocks / compute_units);
            double cost = rounds * block_cost;
            if (c.split_k > 1) cost += (double)pr.y_elems * c.split_k / compute_units * 0.5;
            if (cost < best) { best = cost; bc = c; }
        }
    }
    int64_t nsteps = (pr.CRS + bc.bk - 1) / bc.bk, per = (nsteps + bc.split_k - 1) / bc.split_k;
    bc.reduce = (nsteps + per - 1) / per > 8 ? 1 : 0;
    *out = bc;
}

// ---- search-result cache ----------------------------------------------------------------------
struct CacheEntry {
    wpk_conv_config cfg;
    double us;
};
static std::mutex g_cache_mu;
static std::map<std::string, CacheEntry> g_cache;
static std::string cache_key(const wpk_conv_desc *d) { return desc_key(d) + "|" + device_name(); }

// ---- splitmix64 (Steele, Lea, Flood 2014): state += gamma; output = mix(state) -------------------
struct SplitMix64 {
    uint64_t s;
    explicit SplitMix64(uint64_t seed) : s(seed) {}
    uint64_t next()
    {
        s += 0x9E3779B97F4A7C15ull;
        uint64_t z = s;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }
    double uniform() { return (double)(next() >> 11) * (1.0 / 9007199254740992.0); }
    int32_t randint(int32_t lo, int32_t hi)
    {
        return lo + (int32_t)(next() % (uint64_t)((int64_t)hi - lo + 1));
    }
};

// ---- genetic search engine (Section 2.3 "Genetic search") -----------------------------------------
typedef std::vector<int32_t> Chrom;

struct Ga {
    int32_t n;
    const int32_t *lo, *hi;
    wpk_ga_constraint_fn constraint;
    wpk_ga_fitness_fn fitness;
    void *user;
    SplitMix64 rng;
    std::map<Chrom, double> memo;

    bool ok(const Chrom &c) { return !constraint || constraint(c.data(), n, user) != 0; }

    double eval(const Chrom &c)
    {
        auto it = memo.find(c);
        if (it != memo.end()) return it->second;
        double f = fitness(c.data(), n, user);
        if (!(f > 0.0)) f = 0.0;
        memo[c] = f;
        return f;
    }

    // Step1: uniform draws per gene, re-drawn until the constraint check passes.
    bool random_legal(Chrom &c)
    {
        c.resize(n);
        for (int t = 0; t < 100000; ++t) {
            for (int g = 0; g < n; ++g) c[g] = rng.randint(lo[g], hi[g]);
            if (ok(c)) return true;
        }
        return false;
    }
};

// Indices by decreasing fitness; equal fitness keeps population order.
static std::vector<int> sort_by_fitness(const std::vector<double> &fit)
{
    std::vector<int> idx(fit.size());
    std::iota(idx.begin(), idx.end(), 0);
    std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return fit[a] > fit[b]; });
    return idx;
}

// Roulette wheel by inverse sampling: first i with v <= P(a_i); P(a_0) = 0, so v = 0 picks i = 1.
static int roulette_pick(const std::vector<double> &P, double v)
{
    for (size_t i = 0; i < P.size(); ++i)
        if (v <= P[i]) return (int)i;
    return (int)P.size() - 1;
}

static bool runtimes_close(const std::vector<double> &fit, double eps)
{
    double tmin = 1e300, tmax = 0;
    for (double f : fit) {
        if (f <= 0.0) return false;
        double t = 1.0 / f;
        tmin = std::min(tmin, t);
        tmax = std::max(tmax, t);
    }
    return (tmax - tmin) / tmin < eps;
}

}  // namespace wpk

using namespace wpk;

extern "C" {

int wpk_conv_out_shape(const wpk_conv_desc *d, int32_t *p, int32_t *q)
{
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    if (p) *p = pr.P;
    if (q) *q = pr.Q;
    return WPK_OK;
}

double wpk_conv_flops(const wpk_conv_desc *d)
{
    Problem pr;
    if (make_problem(d, &pr) != WPK_OK) return 0.0;
    return 2.0 * (double)pr.M * d->k * pr.CRS;
}

const char *wpk_status_string(int status)
{
    switch (status) {
    case WPK_OK: return "ok";
    case WPK_E_BAD_DESC: return "bad convolution descriptor";
    case WPK_E_NULL_PTR: return "null pointer argument";
    case WPK_E_UNSUPPORTED: return "unsupported dtype, layout or size";
    case WPK_E_HIP: return "HIP runtime error";
    case WPK_E_NO_CONFIG: return "configuration not legal for this descriptor";
    case WPK_E_BAD_ARG: return "bad argument";
    case WPK_E_IO: return "cache file i/o error";
    case WPK_E_VERIFY: return "no candidate passed verification";
    case WPK_E_TOO_LARGE: return "packed weights exceed the static scratch of the entry point that does not allocate";
    }
    return status > 0 ? "ok (id)" : "unknown status";
}

int wpk_last_hip_error(void) { return g_last_hip_error; }

int wpk_config_gene_ranges(int32_t lo[WPK_N_GENES], int32_t hi[WPK_N_GENES])
{
    if (!lo || !hi) return WPK_E_NULL_PTR;
    for (int g = 0; g < WPK_N_GENES; ++g) {
        lo[g] = 0;
        hi[g] = kGeneCounts[g] - 1;
    }
    return WPK_OK;
}

int wpk_config_from_genes(const int32_t genes[WPK_N_GENES], wpk_conv_config *out)
{
    if (!genes || !out) return WPK_E_NULL_PTR;
    for (int g = 0; g < WPK_N_GENES; ++g)
        if (genes[g] < 0 || genes[g] >= kGeneCounts[g]) return WPK_E_BAD_ARG;
    out->bm = kBmVals[genes[0]];
    out->bn = kBnVals[genes[1]];
    out->bk = kBkVals[genes[2]];
    out->wm = kWmVals[genes[3]];
    out->wn = kWnVals[genes[4]];
    out->split_k = kSplitVals[genes[5]];
    out->xcd_remap = kRemapVals[genes[6]];
    out->persist = kPersistVals[genes[7]];
    out->stages = kStageVals[genes[8]];
    out->reduce = kReduceVals[genes[9]];
    return WPK_OK;
}

int wpk_config_to_genes(const wpk_conv_config *cfg, int32_t genes[WPK_N_GENES])
{
    if (!cfg || !genes) return WPK_E_NULL_PTR;
    int32_t f[WPK_N_GENES];
    cfg_fields(cfg, f);
    for (int g = 0; g < WPK_N_GENES; ++g) {
        int i = value_index(g, f[g]);
        if (i < 0) return WPK_E_BAD_ARG;
        genes[g] = i;
    }
    return WPK_OK;
}

int wpk_config_legal(const wpk_conv_desc *d, const wpk_conv_config *cfg)
{
    if (!cfg) return WPK_E_NULL_PTR;
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    return legal_for(pr, *cfg) ? 1 : 0;
}

int wpk_config_id(const wpk_conv_config *cfg)
{
    int32_t genes[WPK_N_GENES];
    int rc = wpk_config_to_genes(cfg, genes);
    if (rc != WPK_OK) return rc;
    int id = 0;
    for (int g = WPK_N_GENES - 1; g >= 0; --g) id = id * kGeneCounts[g] + genes[g];
    return id;
}

int wpk_config_from_id(int id, wpk_conv_config *out)
{
    if (!out) return WPK_E_NULL_PTR;
    if (id < 0) return WPK_E_NO_CONFIG;
    int32_t genes[WPK_N_GENES];
    for (int g = 0; g < WPK_N_GENES; ++g) {
        genes[g] = id % kGeneCounts[g];
        id /= kGeneCounts[g];
    }
    if (id != 0) return WPK_E_NO_CONFIG;
    return wpk_config_from_genes(genes, out);
}

const char *wpk_config_kernel_name(const wpk_conv_config *cfg)
{
    if (!cfg) return "";
    int i = find_variant(cfg->bm, cfg->bn, cfg->bk, cfg->wm, cfg->wn, cfg->stages);
    return i < 0 ? "" : kVariants[i].name;
}

const char *wpk_version(void) { return "wpk-conv 0.1 (gfx950)"; }

// ---- cache -----------------------------------------------------------------------------------
int wpk_cache_lookup(const wpk_conv_desc *d, wpk_conv_config *out)
{
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    std::lock_guard<std::mutex> g(g_cache_mu);
    if (g_cache.empty()) return 0;
    auto it = g_cache.find(cache_key(d));
    if (it == g_cache.end()) return 0;
    if (out) *out = it->second.cfg;
    return 1;
}

int wpk_cache_lookup_time(const wpk_conv_desc *d, wpk_conv_config *out, double *us)
{
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    std::lock_guard<std::mutex> g(g_cache_mu);
    auto it = g_cache.find(cache_key(d));
    if (it == g_cache.end()) return 0;
    if (out) *out = it->second.cfg;
    if (us) *us = it->second.us;
    return 1;
}

int wpk_cache_store(const wpk_conv_desc *d, const wpk_conv_config *cfg, double us)
{
    if (!cfg) return WPK_E_NULL_PTR;
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    if (!legal_for(pr, *cfg)) return WPK_E_NO_CONFIG;
    std::lock_guard<std::mutex> g(g_cache_mu);
    g_cache[cache_key(d)] = CacheEntry{*cfg, us};
    return WPK_OK;
}

int wpk_cache_clear(void)
{
    std::lock_guard<std::mutex> g(g_cache_mu);
    g_cache.clear();
    return WPK_OK;
}

int wpk_cache_size(void)
{
    std::lock_guard<std::mutex> g(g_cache_mu);
    return (int)g_cache.size();
}

int wpk_cache_save(const char *path)
{
    if (!path) return WPK_E_NULL_PTR;
    FILE *f = fopen(path, "w");
    if (!f) return WPK_E_IO;
    std::lock_guard<std::mutex> g(g_cache_mu);
    fprintf(f, "# wpk search-result cache v3: key bm bn bk wm wn split_k xcd_remap persist stages reduce microseconds\n");
    for (auto &kv : g_cache) {
        std::string key = kv.first;
        std::replace(key.begin(), key.end(), ' ', '_');
        const wpk_conv_config &c = kv.second.cfg;
        fprintf(f, "%s %d %d %d %d %d %d %d %d %d %d %.6f\n", key.c_str(), c.bm, c.bn, c.bk, c.wm, c.wn,
                c.split_k, c.xcd_remap, c.persist, c.stages, c.reduce, kv.second.us);
    }
    return fclose(f) == 0 ? WPK_OK : WPK_E_IO;
}

int wpk_cache_load(const char *path)
{
    if (!path) return WPK_E_NULL_PTR;
    FILE *f = fopen(path, "r");
    if (!f) return WPK_E_IO;
    char line[1024];
    int count = 0;
    std::lock_guard<std::mutex> g(g_cache_mu);
    while (fgets(line, sizeof line, f)) {
        if (line[0] == '#' || line[0] == '\n') continue;
        char key[512];
        wpk_conv_config c;
        double us;
        if (sscanf(line, "%511s %d %d %d %d %d %d %d %d %d %d %lf", key, &c.bm, &c.bn, &c.bk, &c.wm,
                   &c.wn, &c.split_k, &c.xcd_remap, &c.persist, &c.stages, &c.reduce, &us) != 12)
            continue;  // also skips lines of older formats: those layers are searched again
        int32_t genes[WPK_N_GENES];
        if (wpk_config_to_genes(&c, genes) != WPK_OK) continue;
        g_cache[key] = CacheEntry{c, us};
        ++count;
    }
    fclose(f);
    return count;
}

// ---- layouts of the tensors between layers (Section 2.1, data layout transformation) ----------------
// Every tensor is stored [N][C][H][W] (0) or channels-last (1); a layer's cost depends on the layouts
// of the tensor it reads and of the tensor it writes; a residual is read in the layout its layer
// writes, so the two tensors are tied into one group.  Minimise the sum of the layers' costs over
// the free groups.  Exact, by elimination along the layer order: a table over the assignments of
// the groups that layers already seen AND layers still to come refer to (a network's frontier: two
// to four groups for chains with shortcut branches); a group is minimised out after its last layer,
// with the minimising value kept per remaining assignment for the way back.
int wpk_choose_layouts(int32_t n_layers, const int32_t *x_tensor, const int32_t *y_tensor,
                       const int32_t *residual_tensor, const int32_t *tensor_layout, int32_t n_tensors,
                       const double *cost, int32_t *chosen, double *total)
{
    if (!x_tensor || !y_tensor || !tensor_layout || !cost || !chosen) return WPK_E_NULL_PTR;
    if (n_layers <= 0 || n_tensors <= 0) return WPK_E_BAD_ARG;
    for (int i = 0; i < n_layers; ++i)
        if (x_tensor[i] < 0 || x_tensor[i] >= n_tensors || y_tensor[i] < 0 || y_tensor[i] >= n_tensors ||
            (residual_tensor && residual_tensor[i] >= n_tensors))
            return WPK_E_BAD_ARG;
    for (int t = 0; t < n_tensors; ++t)
        if (tensor_layout[t] < -1 || tensor_layout[t] > 1) return WPK_E_BAD_ARG;
    // groups of tied tensors (union-find); a group is fixed if any member is
    std::vector<int> parent(n_tensors);
    std::iota(parent.begin(), parent.end(), 0);
    auto find = [&](int t) { while (parent[t] != t) t = parent[t] = parent[parent[t]]; return t; };
    if (residual_tensor)
        for (int i = 0; i < n_layers; ++i)
            if (residual_tensor[i] >= 0) parent[find(residual_tensor[i])] = find(y_tensor[i]);
    std::vector<int> fixed(n_tensors, -1), last_use(n_tensors, -1), value(n_tensors, 0);
    for (int t = 0; t < n_tensors; ++t)
        if (tensor_layout[t] >= 0) {
            int r = find(t);
            if (fixed[r] >= 0 && fixed[r] != tensor_layout[t]) return WPK_E_BAD_ARG;  // tied tensors fixed differently
            fixed[r] = tensor_layout[t];
        }
    for (int i = 0; i < n_layers; ++i) last_use[find(x_tensor[i])] = last_use[find(y_tensor[i])] = i;
    for (int t = 0; t < n_tensors; ++t)
        if (find(t) == t && fixed[t] >= 0) value[t] = fixed[t];  // also for groups no layer refers to

    const double kNever = 1e300;
    const size_t kMaxOpen = 20;
    struct Closed {
        int group;
        std::vector<int> open_after;   // the groups still open once this one is gone, in table order
        int pos;                       // where it sat among the open groups
        std::vector<char> best;        // per assignment of open_after: the value that minimised
    };
    std::vector<Closed> history;
    std::vector<int> open;
    std::vector<double> tab(1, 0.0);
    auto pos_of = [&](int g) { return (int)(std::find(open.begin(), open.end(), g) - open.begin()); };
    for (int i = 0; i < n_layers; ++i) {
        const int gs[2] = {find(x_tensor[i]), find(y_tensor[i])};
        for (int k = 0; k < 2; ++k) {
            if (pos_of(gs[k]) < (int)open.size()) continue;
            if (open.size() >= kMaxOpen) return WPK_E_UNSUPPORTED;  // a frontier no network here comes near
            const size_t n = tab.size();
            tab.resize(2 * n);
            for (size_t st = 0; st < n; ++st) {
                const double base = tab[st];
                tab[st] = fixed[gs[k]] == 1 ? kNever : base;
                tab[st + n] = fixed[gs[k]] == 0 ? kNever : base;
            }
            open.push_back(gs[k]);
        }
        const int px = pos_of(gs[0]), py = pos_of(gs[1]);
        for (size_t st = 0; st < tab.size(); ++st)
            if (tab[st] < kNever) tab[st] += cost[(size_t)i * 4 + ((st >> px) & 1) * 2 + ((st >> py) & 1)];
        for (int k = 0; k < 2; ++k) {
            const int g = gs[k];
            const int p = pos_of(g);
            if (p == (int)open.size() || last_use[g] != i) continue;  // closed already (x == y group), or used later
            Closed c;
            c.group = g;
            c.pos = p;
            const size_t n = tab.size() / 2;
            std::vector<double> next(n);
            c.best.resize(n);
            const size_t low = ((size_t)1 << p) - 1;
            for (size_t r = 0; r < n; ++r) {
                const size_t s0 = (r & low) | ((r & ~low) << 1), s1 = s0 | ((size_t)1 << p);
                c.best[r] = tab[s1] < tab[s0] ? 1 : 0;
                next[r] = std::min(tab[s0], tab[s1]);
            }
            open.erase(open.begin() + p);
            c.open_after = open;
            tab.swap(next);
            history.push_back(std::move(c));
        }
    }
    if (tab.size() != 1 || !(tab[0] < kNever)) return WPK_E_BAD_ARG;
    for (size_t h = history.size(); h-- > 0;) {
        const Closed &c = history[h];
        size_t r = 0;
        for (size_t k = 0; k < c.open_after.size(); ++k) r |= (size_t)value[c.open_after[k]] << k;
        value[c.group] = c.best[r];
    }
    for (int t = 0; t < n_tensors; ++t) chosen[t] = value[find(t)];
    if (total) *total = tab[0];
    return WPK_OK;
}

// ---- tuning options and the engine ---------------------------------------------------------------
int64_t wpk_config_workspace_bytes(const wpk_conv_desc *d, const wpk_conv_config *cfg,
                                   int32_t compute_units, int64_t *shared_tiles, int64_t *slots)
{
    if (!cfg) return WPK_E_NULL_PTR;
    Problem pr;
    int rc = make_problem(d, &pr);
    if (rc != WPK_OK) return rc;
    if (!legal_for(pr, *cfg)) return WPK_E_NO_CONFIG;
    FixupNeed n = fixup_need(pr, *cfg, compute_units);
    if (shared_tiles) *shared_tiles = n.shared_tiles;
    if (slots) *slots = n.maxc;
    return n.bytes;
}

int wpk_set_workspace_limit(int64_t bytes)
{
    if (bytes < 0) return WPK_E_BAD_ARG;
    g_workspace_limit.store(bytes, std::memory_order_relaxed);
    return WPK_OK;
}

void wpk_tune_default_options(wpk_tune_options *o)
{
    if (!o) return;
    memset(o, 0, sizeof *o);
    o->population = 64;
    o->elites = 8;
    o->next_population = 64;
    o->participants = 64;
    o->max_generations = 16;
    o->patience = 5;
    o->mutation = 0.15;
    o->eps = 0.03;
    o->seed = 2008;
    o->reps = 5;
    o->min_group_us = 200.0;
    o->mode = 0;
    o->verbose = 0;
    o->refine = 2;
    o->zero_ahead = 0;
    o->epilogue = 0;
}

int wpk_ga_search(int32_t n_genes, const int32_t *lo, const int32_t *hi,
                  wpk_ga_constraint_fn constraint, wpk_ga_fitness_fn fitness, void *user,
                  const wpk_tune_options *opt_in, int32_t *best_genes, double *best_fitness,
                  int32_t *evaluations, int32_t *history_pop, double *history_fit,
                  int32_t *history_sizes, int32_t history_capacity)
{
    if (!lo || !hi || !fitness) return WPK_E_NULL_PTR;
    wpk_tune_options opt;
    if (opt_in) opt = *opt_in; else wpk_tune_default_options(&opt);
    if (n_genes <= 0 || opt.population <= 0 || opt.max_generations <= 0) return WPK_E_BAD_ARG;
    for (int g = 0; g < n_genes; ++g)
        if (hi[g] < lo[g]) return WPK_E_BAD_ARG;
    int32_t next_pop = opt.next_population > 0 ? opt.next_population : opt.population;
    int32_t width = std::max(opt.population, next_pop);
    const int retries = 8;

    Ga ga{n_genes, lo, hi, constraint, fitness, user, SplitMix64(opt.seed), {}};
    std::vector<Chrom> pop(opt.population);
    for (auto &c : pop)                                                        // Step1
        if (!ga.random_legal(c)) return WPK_E_NO_CONFIG;

    Chrom best;
    double best_f = -1.0;
    int stall = 0, gen = 0;
    for (;; ++gen) {
        std::vector<double> fit(pop.size());
        for (size_t i = 0; i < pop.size(); ++i) fit[i] = ga.eval(pop[i]);      // Step2
        if (gen < history_capacity) {
            if (history_sizes) history_sizes[gen] = (int32_t)pop.size();
            for (int i = 0; i < width; ++i) {
                if (history_fit) history_fit[(size_t)gen * width + i] = i < (int)pop.size() ? fit[i] : -1.0;
                if (history_pop)
                    for (int g = 0; g < n_genes; ++g)
                        history_pop[((size_t)gen * width + i) * n_genes + g] =
                            i < (int)pop.size() ? pop[i][g] : -1;
            }
        }
        std::vector<int> order = sort_by_fitness(fit);
        if (fit[order[0]] > best_f) {
            best = pop[order[0]];
            best_f = fit[order[0]];
            stall = 0;
        } else {
            ++stall;
        }
        if (opt.verbose)
            fprintf(stderr, "[wpk search] generation %d: size %zu, best fitness %.6g, evaluated %zu\n",
                    gen, pop.size(), best_f, ga.memo.size());
        if (runtimes_close(fit, opt.eps) || (opt.patience > 0 && stall >= opt.patience) ||
            gen == opt.max_generations - 1)                                    // Step4
            break;

        std::vector<Chrom> nxt;
        if (opt.mode == 1) {  // random search: a fresh random generation, nothing inherited
            nxt.resize(next_pop);
            for (auto &c : nxt)
                if (!ga.random_legal(c)) return WPK_E_NO_CONFIG;
        } else {              // Step3
            int k = std::min<int>(std::max(opt.elites, 0), (int)pop.size());
            k = std::min(k, (int)next_pop);
            int m = opt.participants > 0 ? std::min<int>(opt.participants, (int)pop.size())
                                         : (int)pop.size();
            for (int i = 0; i < k; ++i) nxt.push_back(pop[order[i]]);
            // eq. (1) over the m participants, then eq. (2)
            double total = 0.0;
            for (int i = 0; i < m; ++i) total += fit[order[i]];
            std::vector<double> P(m);
            double run = 0.0;
            for (int i = 0; i < m; ++i) {
                double p = total > 0.0 ? fit[order[i]] / total : 1.0 / m;
                run += p;
                P[i] = run;
            }
            P[m - 1] = 1.0;
            while ((int)nxt.size() < next_pop) {
                Chrom child(n_genes);
                bool done = false;
                for (int t = 0; t < retries && !done; ++t) {
                    const Chrom &a = pop[order[roulette_pick(P, ga.rng.uniform())]];
                    const Chrom &b = pop[order[roulette_pick(P, ga.rng.uniform())]];
                    for (int g = 0; g < n_genes; ++g) child[g] = ga.rng.uniform() < 0.5 ? a[g] : b[g];
                    for (int g = 0; g < n_genes; ++g)
                        if (ga.rng.uniform() < opt.mutation) child[g] = ga.rng.randint(lo[g], hi[g]);
                    done = ga.ok(child);
                }
                if (!done && !ga.random_legal(child)) return WPK_E_NO_CONFIG;
                nxt.push_back(child);
            }
        }
        pop.swap(nxt);
    }
    if (best_genes)
        for (int g = 0; g < n_genes; ++g) best_genes[g] = best[g];
    if (best_fitness) *best_fitness = best_f;
    if (evaluations) *evaluations = (int32_t)ga.memo.size();
    return gen + 1;
}

}  // extern "C"
