// Host-only validation and workspace planning (see plan.hpp).
#include <algorithm>

#include "plan.hpp"

namespace cbw {

namespace {

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

Region take(size_t* cursor, size_t bytes)
{
    Region r;
    r.off = *cursor;
    r.bytes = bytes;
    *cursor = align256(*cursor + bytes);
    return r;
}

constexpr int64_t kMaxElems = (int64_t)1 << 31;

}  // namespace

int validate_desc(const cbw_conv_desc* d)
{
    if (!d) return CBW_ERR_INVALID_ARG;
    if (d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0)
        return CBW_ERR_INVALID_ARG;
    if (d->stride_h <= 0 || d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0) return CBW_ERR_INVALID_ARG;
    const int64_t ph = (int64_t)d->H + 2 * (int64_t)d->pad_h - d->R;
    const int64_t pw = (int64_t)d->W + 2 * (int64_t)d->pad_w - d->S;
    if (ph < 0 || pw < 0) return CBW_ERR_INVALID_ARG;
    if (d->P != ph / d->stride_h + 1 || d->Q != pw / d->stride_w + 1) return CBW_ERR_INVALID_ARG;
    if (d->dtype != CBW_F32 && d->dtype != CBW_BF16) return CBW_ERR_INVALID_ARG;
    if (d->act_layout != CBW_NHWC && d->act_layout != CBW_NCHW) return CBW_ERR_INVALID_ARG;
    if (d->w_layout != CBW_KRSC && d->w_layout != CBW_KCRS) return CBW_ERR_INVALID_ARG;
    const int E = d->dtype == CBW_BF16 ? 8 : 4;
    if (d->C % E != 0 || d->K % E != 0) return CBW_ERR_UNSUPPORTED;
    const int64_t npix = (int64_t)d->N * d->H * d->W, npq = (int64_t)d->N * d->P * d->Q;
    if (npix * d->C >= kMaxElems || npq * d->K >= kMaxElems) return CBW_ERR_UNSUPPORTED;
    // every tensor the kernels read through a buffer descriptor stays below 2^31 bytes
    const int64_t esz = d->dtype == CBW_BF16 ? 2 : 4;
    if (npix * d->C * esz >= kMaxElems || npq * d->K * esz >= kMaxElems) return CBW_ERR_UNSUPPORTED;
    // the fp32 weight gradient (and each split partial of it) stays below 2^31 bytes
    if ((int64_t)d->K * d->C * d->R * d->S * 4 >= kMaxElems) return CBW_ERR_UNSUPPORTED;
    if (d->K > 1024 * kWeightTileK) return CBW_ERR_UNSUPPORTED;  // occupancy flags per chunk
    return CBW_OK;
}

int require_nhwc(const cbw_conv_desc* d)
{
    const int st = validate_desc(d);
    if (st != CBW_OK) return st;
    return d->act_layout == CBW_NHWC ? CBW_OK : CBW_ERR_UNSUPPORTED;
}

// The pixel classes of a strided data gradient, most taps first (ties keep
// the residue order); empty classes (no such row or column) are left out.
static int data_classes(const cbw_conv_desc* d, DataPlan::Class* out)
{
    if ((d->stride_h == 1 && d->stride_w == 1) || (int64_t)d->stride_h * d->stride_w > kDataMaxClasses) return 0;
    auto axis = [](int size, int pad, int st, int filt, int a, int* first, int* n, int* taps) {
        // positions h = st * i + a - pad in [0, size)
        *first = pad > a ? (pad - a + st - 1) / st : 0;
        const int last = size - 1 + pad - a;   // st * i <= last
        *n = last >= 0 ? std::max(0, last / st - *first + 1) : 0;
        *taps = a < filt ? (filt - 1 - a) / st + 1 : 0;
    };
    int n = 0;
    for (int a = 0; a < d->stride_h; ++a)
        for (int b = 0; b < d->stride_w; ++b) {
            DataPlan::Class c;
            c.a = a;
            c.b = b;
            axis(d->H, d->pad_h, d->stride_h, d->R, a, &c.i0, &c.nh, &c.nr);
            axis(d->W, d->pad_w, d->stride_w, d->S, b, &c.j0, &c.nw, &c.ns);
            if (c.nh == 0 || c.nw == 0) continue;
            c.npix = (int64_t)d->N * c.nh * c.nw;
            out[n++] = c;
        }
    std::stable_sort(out, out + n, [](const DataPlan::Class& x, const DataPlan::Class& y) {
        return x.nr * x.ns > y.nr * y.ns;
    });
    return n;
}

// Split of the bf16 class tiling, `most` ways at most: `tiles` tiles, `steps`
// steps in the longest one.  The classes have few steps and, a tile row of
// theirs being a part of an image's, many tiles, so the finest split (the rule
// without classes) writes more partials than its shorter chains save, and
// leaves no CU to the weight gradient's reduction in the same launch.  Fitted
// in us: 1.1 a step, 6 for a reduction at all, the partials written and read at
// 10 TB/s together.  Both gradients, N = 16, by the number of splits (16, 8, 4,
// 2, 1): 512 -> 512, 3x3, 8 x 8 48.9, 48.2, 50.6, 58.0, 68.0 us; 128 -> 256,
// 28 x 28 58.3 (9), 55.7, 52.4, 55.2, 55.2; 256 -> 512, 1x1, 28 x 28 -, 45.9,
// 44.6, 45.0, 42.6.  fp32 steps are six times as long: as fine as it goes.
static int class_split(int most, int tiles, int steps, double tile_mb)
{
    int best = 1;
    double best_cost = 1.1 * steps;
    for (int sp = 2; sp <= most; ++sp) {
        const double cost = 6.0 + 1.1 * ((steps + sp - 1) / sp) + tile_mb * tiles * sp / 10.0;
        if (cost < best_cost) {
            best = sp;
            best_cost = cost;
        }
    }
    return best;
}

int data_tile_index(int C)
{
    int best = 0, best_waste = -1;
    for (int t = 0; t < kDataTileCount; ++t) {
        const int bm = kDataTiles[t].bm;
        const int waste = (C + bm - 1) / bm * bm - C;
        if (8 * waste <= C) return t;
        if (best_waste < 0 || waste < best_waste) {
            best = t;
            best_waste = waste;
        }
    }
    return best;
}

bool data_rows_eligible(const cbw_conv_desc* d)
{
    return d->dtype == CBW_BF16 && d->R == 3 && d->S == 3 && d->stride_h == 1 && d->stride_w == 1 && d->C == 64 &&
           d->K == 64;
}

bool data_pw_eligible(const cbw_conv_desc* d)
{
    auto ok = [](int c) { return c == 64 || c == 128 || c == 256; };
    return d->dtype == CBW_BF16 && d->R == 1 && d->S == 1 && d->stride_h == 1 && d->stride_w == 1 &&
           d->pad_h == 0 && d->pad_w == 0 && ok(d->C) && ok(d->K) && d->C * d->K <= 16384;
}

int plan_data(const cbw_conv_desc* d, bool masked, DataPlan* out, bool no_split, bool allow_rows)
{
    int st = validate_desc(d);
    if (st != CBW_OK) return st;
    DataPlan p;
    if (allow_rows && data_pw_eligible(d)) {
        // as many resident waves as give every wave the same whole number of
        // 16-pixel blocks (the last wave takes the rest)
        p.tile = data_tile_index(d->C);
        p.bm = kDataTiles[p.tile].bm;
        p.bn = kDataTiles[p.tile].bn;
        p.npix = (int64_t)d->N * d->H * d->W;
        p.groups = (d->C + p.bm - 1) / p.bm;
        p.pw = true;
        const int64_t nblk = (p.npix + 15) / 16;
        p.pw_bpw = (int)((nblk + kDataPwMaxWaves - 1) / kDataPwMaxWaves);
        const int64_t waves = (nblk + p.pw_bpw - 1) / p.pw_bpw;
        p.pw_grid = (int)((waves + kDataPwWaves - 1) / kDataPwWaves);
        size_t cur = 0;
        p.header = take(&cur, 256);
        p.wt = take(&cur, (size_t)d->K * d->C * elem_bytes(d->dtype));
        p.row_counts = take(&cur, (size_t)p.pw_grid * 4);
        if (d->act_layout == CBW_NCHW) {
            p.t_dy = take(&cur, (size_t)d->N * d->P * d->Q * d->K * elem_bytes(d->dtype));
            p.t_dx = take(&cur, (size_t)p.npix * d->C * elem_bytes(d->dtype));
            if (masked) p.t_mask = take(&cur, ((size_t)p.npix * d->C + 31) / 32 * 4);
        }
        p.total = cur;
        *out = p;
        return CBW_OK;
    }
    if (allow_rows && data_rows_eligible(d)) {
        // one workgroup per CU: strips of consecutive output rows, as many
        // as make the segments times the strips fill the CUs once
        p.tile = data_tile_index(d->C);
        p.bm = kDataTiles[p.tile].bm;
        p.bn = kDataTiles[p.tile].bn;
        p.npix = (int64_t)d->N * d->H * d->W;
        p.groups = (d->C + p.bm - 1) / p.bm;
        p.rows = true;
        p.rows_nseg = (d->W + kDataRowsSegment - 1) / kDataRowsSegment;
        const int nrows = d->N * d->H;
        int strips = CBW_NUM_CUS / p.rows_nseg;
        if (strips < 1) strips = 1;
        p.rows_per_strip = (nrows + strips - 1) / strips;
        p.rows_grid = (nrows + p.rows_per_strip - 1) / p.rows_per_strip * p.rows_nseg;
        const int wseg = d->W < kDataRowsSegment ? d->W : kDataRowsSegment;
        p.rows_nbw = ((wseg + 15) / 16 + 3) / 4;
        // the deepest prefetch (at most 8 steps) whose rings fit the LDS:
        // depth + 3 dY rows and depth + 2 footprint rows
        // a slot holds the 16-column blocks' rows and the two halo columns
        p.rows_slot = ((wseg + 15) / 16 * 16 + 2 + 7) / 8 * 1024;
        p.rows_mslot = (wseg * 8 + 1023) / 1024 * 1024;   // whole 1 KB copies of 16-byte pieces
        p.rows_depth = 8;
        while (p.rows_depth > 1 &&
               (p.rows_depth + 3) * p.rows_slot + (p.rows_depth + 2) * p.rows_mslot > kDataRowsLds)
            --p.rows_depth;
        size_t cur = 0;
        p.header = take(&cur, 256);
        p.wt = take(&cur, (size_t)d->K * d->C * d->R * d->S * elem_bytes(d->dtype));
        p.row_counts = take(&cur, (size_t)p.rows_grid * 4);
        if (d->act_layout == CBW_NCHW) {
            p.t_dy = take(&cur, (size_t)d->N * d->P * d->Q * d->K * elem_bytes(d->dtype));
            p.t_dx = take(&cur, (size_t)p.npix * d->C * elem_bytes(d->dtype));
            if (masked) p.t_mask = take(&cur, ((size_t)p.npix * d->C + 31) / 32 * 4);
        }
        p.total = cur;
        *out = p;
        return CBW_OK;
    }
    p.tile = data_tile_index(d->C);
    p.bm = kDataTiles[p.tile].bm;
    p.bn = kDataTiles[p.tile].bn;
    p.npix = (int64_t)d->N * d->H * d->W;
    p.groups = (d->C + p.bm - 1) / p.bm;
    p.nblk = (int)((p.npix + kCompactBlock - 1) / kCompactBlock);
    size_t cur = 0;
    int cand[kDataRowChoices];
    for (int c = 0; c < kDataRowChoices; ++c) {
        const int rows = p.bn - 16 * c;
        cand[c] = p.groups * (int)((p.npix + rows - 1) / rows);
    }
    p.brows = data_rows_pick(cand, p.bn, kDataSlots);
    p.ptiles = p.ptaps = (int)((p.npix + p.brows - 1) / p.brows);
    const int bk = 8 * (d->dtype == CBW_BF16 ? 8 : 4);
    p.nsteps = d->R * d->S * ((d->K + bk - 1) / bk);
    p.ncls = data_classes(d, p.cls);
    // One step a tile in one round of tiles: the classes shorten no chain, and
    // their tiles store every other pixel's row (both gradients of 1x1 stride 2,
    // 53 x 53, N = 8, K = 32, C = 208, 240, 256, 328 with classes and without:
    // 28.3, 29.0, 24.3, 31.8 and 26.3, 26.9, 24.1, 29.0 us).  Not with tiles of
    // 64 channels, whose rows are a line or less (C = 64, 56 x 56, N = 32: 24.3
    // and 25.1; C = 144: 28.2 and 34.7).
    if (p.nsteps == 1 && p.bm > 64 && p.ptiles * p.groups <= kDataSlots) p.ncls = 0;
    if (p.ncls > 0) {
        const int all = p.groups * (int)((p.npix + p.bn - 1) / p.bn);
        p.list_tiles = host_data_split(all, p.nsteps) > 1 ? all : 0;
        // full tiles: a tile's time hardly depends on its rows, and with
        // classes of different taps rounds of tiles say little (128 -> 256
        // channels, 56 x 56, N = 32: 35 us with 448 rows, 37 with 416, 39
        // with 224; 256 -> 512: 71, 79, 93)
        p.brows = p.bn;
        p.ptiles = p.ptaps = 0;
        for (int c = 0; c < p.ncls; ++c) {
            p.cls[c].tile0 = p.ptiles;
            p.ptiles += (int)((p.cls[c].npix + p.brows - 1) / p.brows);
            if (p.cls[c].nr * p.cls[c].ns > 0) p.ptaps = p.ptiles;
        }
    }
    // (classes: no finer than the longest one's steps, the rest would write
    // partials for nothing)
    const int split_steps = p.ncls > 0 ? std::max(1, p.cls[0].nr * p.cls[0].ns * (p.nsteps / (d->R * d->S))) : p.nsteps;
    // Tiles that no tap reaches only write zeros: they are not split, and the
    // split of the others fills the CUs they leave.  Split like the others they
    // wrote partials of zeros, 8.3 of 11 MB for 256 -> 256 channels, 1x1 stride
    // 2, 27 x 27, N = 3 (both gradients 42.3 -> 39.8 us, 41.9 without classes;
    // 69 x 72: 54.6 -> 47.3, 53.4).
    p.split = no_split ? 1 : host_data_split(p.ptaps * p.groups, split_steps, (p.ptiles - p.ptaps) * p.groups);
    if (p.ncls > 0 && d->dtype == CBW_BF16)
        p.split = class_split(p.split, p.ptaps * p.groups, split_steps, p.bn * p.bm * 4e-6);
    p.header = take(&cur, 256);
    p.wt = take(&cur, (size_t)d->K * d->C * d->R * d->S * elem_bytes(d->dtype));
    if (masked) {
        p.blk_counts = take(&cur, (size_t)p.groups * p.nblk * 4);
        p.counts = take(&cur, (size_t)p.groups * 4);
        p.dead_flags = take(&cur, (size_t)p.groups * 4);
        p.lists = take(&cur, (size_t)p.groups * p.npix * 4);
        if (p.ncls > 0) p.live_bits = take(&cur, (size_t)p.groups * p.nblk * (kCompactBlock / 8));
    }
    // Split partial tiles.  Without skipping the host knows the split; with
    // compaction it is decided on the device, bounded by one partial tile
    // per resident workgroup.
    const size_t tile_bytes = (size_t)p.bn * p.bm * 4;
    if (masked && !no_split) p.partial = take(&cur, (size_t)kDataSlots * tile_bytes);
    else if (p.split > 1) p.partial = take(&cur, (size_t)p.ptaps * p.groups * p.split * tile_bytes);
    if (d->act_layout == CBW_NCHW) {
        p.t_dy = take(&cur, (size_t)d->N * d->P * d->Q * d->K * elem_bytes(d->dtype));
        p.t_dx = take(&cur, (size_t)p.npix * d->C * elem_bytes(d->dtype));
        if (masked) p.t_mask = take(&cur, ((size_t)p.npix * d->C + 31) / 32 * 4);
    }
    p.total = cur;
    *out = p;
    return CBW_OK;
}

int fwd_as_data_desc(const cbw_conv_desc* d, cbw_conv_desc* out)
{
    int st = require_nhwc(d);
    if (st != CBW_OK) return st;
    if (d->stride_h != 1 || d->stride_w != 1) return CBW_ERR_UNSUPPORTED;
    if (d->pad_h > d->R - 1 || d->pad_w > d->S - 1) return CBW_ERR_UNSUPPORTED;
    cbw_conv_desc v = *d;
    v.C = d->K; v.K = d->C;
    v.H = d->P; v.W = d->Q;
    v.P = d->H; v.Q = d->W;
    v.pad_h = d->R - 1 - d->pad_h;
    v.pad_w = d->S - 1 - d->pad_w;
    if ((st = validate_desc(&v)) != CBW_OK) return st;
    *out = v;
    return CBW_OK;
}

int weight_tile_k_for(const cbw_conv_desc* d)
{
    if (d->dtype != CBW_BF16) return kWeightTileK;   // fp32: 256 x 256 tiles in 64 x 64 parts
    if (d->K <= 64) return 64;
    if (d->K <= 128) return 128;
    return kWeightTileK;
}

int weight_taps_per_group(const cbw_conv_desc* d)
{
    const int rs = d->R * d->S;
    if (d->dtype != CBW_BF16 || rs == 1 || 2 * d->C > kWeightTileC) return 1;
    // as few groups as the tile allows, the taps spread evenly over them
    // (9 taps of 64 channels: 3 + 3 + 3 rather than 4 + 4 + 1)
    const int t = kWeightTileC / d->C;
    const int groups = (rs + t - 1) / t;
    return (rs + groups - 1) / groups;
}

bool weight_rows_eligible(const cbw_conv_desc* d)
{
    return d->dtype == CBW_BF16 && d->stride_h == 1 && d->stride_w == 1 && d->R <= 3 && d->S <= 3 &&
           d->C % 64 == 0 && d->K % 64 == 0 && d->C <= 128 && d->K <= 128;
}

// Splits of the fp32 weight gradient: `wgs` workgroups of four waves per
// split.  A CU runs its share one wave per SIMD each, 1.9 us of matrix work
// per chunk and wave, up to three workgroups at a time; starting and
// finishing takes about 3 us per three; every split writes and reads back
// the whole gradient at about 4 TB/s.  The cheapest count by that model:
// as many splits as fill the CUs once left them idle where the quotient is
// small (256 -> 256 channels, 28 x 28, N = 8: 144 workgroups a split, five
// splits).  Only the counts at
// which a CU's share (w) or a wave's chunks (g) change are tried, and none
// past the point where the partials and starts alone cost more than the
// difference to perfectly shared work: the same choice as by trying all of
// them (8 -> 32 channels, 1x1, 63 x 63, N = 100: the plans of a call 10.4 -> 3.7
// us of host time; 128 -> 128, 3x3, 28 x 28, N = 16: 1.4 -> 0.4).
int f32_weight_splits(const cbw_conv_desc* d, int64_t wgs, int nchunks, int max_split)
{
    const double part = (double)d->K * d->R * d->S * d->C * 8 / 4e6;
    const double shared = 1.9 * (double)wgs * nchunks / (4 * CBW_NUM_CUS);
    const int most = std::min(max_split, 3 * CBW_NUM_CUS);
    int best = 1;
    double best_cost = 0;
    for (int ns = 1; ns <= most;) {
        const int per = (nchunks + ns - 1) / ns, g = (per + 3) / 4;
        const int64_t w = (wgs * ns + CBW_NUM_CUS - 1) / CBW_NUM_CUS;
        if (ns > 1 && shared + (part + (double)wgs / CBW_NUM_CUS) * ns > best_cost) break;
        // (not the same ranges as fewer splits)
        if ((nchunks + per - 1) / per == ns) {
            const double cost = 1.9 * w * g + 3.0 * ((w + 2) / 3) + part * ns;
            if (ns == 1 || cost < best_cost) {
                best = ns;
                best_cost = cost;
            }
        }
        int64_t next = w * CBW_NUM_CUS / wgs + 1;   // the first with a larger w
        if (g > 1) next = std::min<int64_t>(next, (nchunks + 4 * (g - 1) - 1) / (4 * (g - 1)));   // with a smaller g
        ns = (int)std::min<int64_t>(next, most + 1);
    }
    return best;
}

int plan_weight(const cbw_conv_desc* d, WeightPlan* out, bool allow_rows)
{
    int st = validate_desc(d);
    if (st != CBW_OK) return st;
    WeightPlan p;
    p.npq = (int64_t)d->N * d->P * d->Q;
    p.rows = allow_rows && weight_rows_eligible(d);
    if (p.rows) {
        // row-window kernel: 64 x 64 (k, c) tiles, output rows in segments
        // of up to 128 columns; the skip chunks are whole output rows
        p.chunk = d->Q;
        p.nchunks = d->N * d->P;
        p.bk = 64;
        p.tpg = 1;
        p.cg = 64;
        p.tgroups = (d->Q + kRowSegment - 1) / kRowSegment;
        p.ctiles = d->C / 64;
    } else {
        p.chunk = weight_chunk_px(d->dtype);
        p.nchunks = (int)((p.npq + p.chunk - 1) / p.chunk);
        p.bk = weight_tile_k_for(d);
        p.tpg = weight_taps_per_group(d);
        p.cg = p.tpg > 1 ? d->C : kWeightTileC;
        p.tgroups = (d->R * d->S + p.tpg - 1) / p.tpg;
        p.ctiles = p.tpg > 1 ? 1 : (d->C + kWeightTileC - 1) / kWeightTileC;
    }
    p.ktiles = (d->K + p.bk - 1) / p.bk;
    const int tiles = p.tgroups * p.ctiles * p.ktiles;
    if (d->dtype != CBW_BF16) {
        // the parts of a 256 x 256 tile that hold channels
        p.subc = (std::min(d->C, kWeightTileC) + 63) / 64;
        p.subk = (std::min(d->K, kWeightTileK) + 63) / 64;
    }
    const int max_split = std::max(1, p.nchunks / 4);   // at least four chunks per workgroup
    // bf16: as many splits as fit in one round of resident workgroups
    const int nsplit = d->dtype == CBW_BF16
                           ? std::max(1, std::min(kWeightSlots / tiles, max_split))
                           : f32_weight_splits(d, (int64_t)tiles * p.subc * p.subk, p.nchunks, max_split);
    p.chunks_per_split = (p.nchunks + nsplit - 1) / nsplit;
    p.nsplit = (p.nchunks + p.chunks_per_split - 1) / p.chunks_per_split;
    p.grid = tiles * p.nsplit;
    // partial weight gradients to sum: one per split (and per column segment
    // for the row-window kernel)
    p.nparts = p.rows ? p.nsplit * p.tgroups : p.nsplit;
    p.direct = (p.nparts == 1 && d->w_layout == CBW_KRSC);
    size_t cur = 0;
    p.header = take(&cur, 256);
    p.occ = take(&cur, (size_t)p.nchunks * p.ktiles);
    // live pixels are recorded for the compaction where a split is long enough
    // to gain from it (see compact_range: a split of few chunks saves less
    // than the listing takes; 8 -> 32 channels, 3x3, 147 x 151, N = 1, four
    // chunks a split, 39% of the pixels live: 14.8 us without, 18.0 with)
    if (!p.rows && d->dtype == CBW_BF16 && p.chunks_per_split >= kCompactMinChunks) p.pmask = take(&cur, (size_t)p.nchunks * p.ktiles * 8);
    p.xlive = take(&cur, (size_t)p.nchunks * p.tgroups * p.ctiles);
    p.xbits = take(&cur, ((size_t)d->N * d->H * d->W * d->C + 31) / 32 * 4);
    p.skip_slots = take(&cur, (size_t)p.grid * 4);
    p.work_slots = take(&cur, (size_t)p.grid * 4);
    if (!p.direct) p.partials = take(&cur, (size_t)p.nparts * d->K * d->R * d->S * d->C * 4);
    if (d->act_layout == CBW_NCHW) {
        p.t_x = take(&cur, (size_t)d->N * d->H * d->W * d->C * elem_bytes(d->dtype));
        p.t_dy = take(&cur, (size_t)p.npq * d->K * elem_bytes(d->dtype));
        p.t_dymask = take(&cur, ((size_t)p.npq * d->K + 31) / 32 * 4);
    }
    p.total = cur;
    *out = p;
    return CBW_OK;
}

}  // namespace cbw

namespace cbw {

int weight_ws_bytes(const cbw_conv_desc* d, size_t* bytes)
{
    WeightPlan a, b;
    int st = plan_weight(d, &a, true);
    if (st != CBW_OK) return st;
    if (!a.rows) b = a;   // (the one plan there is)
    else if ((st = plan_weight(d, &b, false)) != CBW_OK) return st;
    *bytes = a.total > b.total ? a.total : b.total;
    return CBW_OK;
}

}  // namespace cbw
