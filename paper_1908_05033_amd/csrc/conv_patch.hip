// dsq_conv2d, LDS-patch kernel: tile planning and dispatch (host side).  The
// kernel itself is in conv_patch_kernel.h.
#include <stdio.h>

#include "conv_patch_kernel.h"

// Patch rows of the worst tile: the padded-row span of its output rows plus the filter.
// A tile covers the strip pixels [t, t + BP), t a multiple of BP, i.e. d + 1 strip rows,
// and passes from one image to the next k times:
//   span = d*stride + k*e,  e = Hp - Ho*stride  (the rows an image boundary adds).
// Exact (but for some 1x1 layers with stride 2 on odd heights, where e = -1 and the result can
// be one row too large), without a walk over all tiles (50 000 per strip width on a 224x224
// layer at batch 32: 3.4 ms a call, 10 to 80 times the kernel):
//   - images smaller than a tile: t modulo the strip pixels of an image repeats after fewer
//     than BP tiles;
//   - otherwise a tile inside an image passes (BP - 1) / TW rows, and one more if it begins in
//     one of the last columns: some tile does if they go through all the columns they can
//     (multiples of the gcd of TW and BP), else their first columns tell; and only one tile
//     crosses each image boundary: those tiles are looked at, until one spans the most that it
//     can or the boundaries' places inside a tile repeat.
// (A bound in place of the exact number, a row or two too large on some layers, had some of
// the largest patches refused and others staged in more units per thread.)
int dsq_patch_rows(const DsqConvArgs &a, int BP, int TW, int row_tiles)
{
    const int Ho = a.Ho, NHo = a.N * Ho, e = a.H + 2 * a.pad - Ho * a.stride;
    const int image = TW * Ho;
    const int G = (image & -image) < BP ? (image & -image) : BP;         // gcds with a power of two
    const int gw = (TW & -TW) < BP ? (TW & -TW) : BP;
    int span = 0;
    auto look_at = [&](int t) {
        const int g0 = t / TW, end = (t + BP - 1) / TW, g1 = end < NHo ? end : NHo - 1;
        const int s = (g1 - g0) * a.stride + (g1 / Ho - g0 / Ho) * e;
        if (s > span) span = s;
    };
    const int repeat = image / G, columns = TW / gw;
    if (image < BP || (e < 0 && a.N > 1 && row_tiles <= columns)) {
        for (int i = 0; i < row_tiles && i < repeat; ++i) look_at(i * BP);
    } else {
        const int passed = (BP - 1) / TW, rest = (BP - 1) % TW;           // a tile passes one row more from column TW - rest on
        int d = passed;
        if (row_tiles > columns) {
            if (gw <= rest) ++d;
        } else {
            look_at((row_tiles - 1) * BP);                                // (cut off by the end of the strip)
            if (row_tiles == 1) return span + a.R;
            if (TW >= BP) {                                               // (the last whole tile step of the first row)
                if (row_tiles - 1 > TW / BP) ++d;
            } else for (int i = 1, c = 0, step = BP % TW; i < row_tiles - 1; ++i) {
                c += step;
                if (c >= TW) c -= TW;
                if (c >= TW - rest) { ++d; break; }
            }
        }
        if (d * a.stride > span) span = d * a.stride;
        if (e < 0 && a.N > 1) {
            // (a tile spans most rows inside an image: one that does has to begin in a row from which
            // that many follow, at a column that reaches the last of them)
            const int col = d * TW - BP + 1 > 0 ? d * TW - BP + 1 : 0;
            bool inside = false;
            for (int row = 0; row + d < Ho && row < G / gw && !inside; ++row)
                inside = ((row * TW + col + G - 1) & -G) < (row + 1) * TW;
            if (!inside) span -= a.stride;
        }
        // the tile across the boundary after image n begins `back` pixels before it
        int across = -1;                                                  // rows that one passes
        for (int n = 1, back = 0; n < a.N && n <= BP / G && across <= passed; ++n) {
            back = (back + image) & (BP - 1);
            if (back == 0) continue;                                      // (the boundary is one between tiles)
            const int m = back < TW ? back : back % TW;
            across = m > 0 && m <= rest ? passed + 1 : across < passed ? passed : across;
        }
        if (across >= 0 && across * a.stride + e > span) span = across * a.stride + e;
    }
    return span + a.R;
}

namespace {

bool plan_patch(const DsqConvArgs &a, int BP, int BC, int PF, int CT, int UPT, int lds_limit, int KS, PatchPlan &best)
{
    // epilogue staging of the four waves; behind it the partial sums of a second wave group, then the table of
    // border terms for two rows of padding
    const int partial = KS == 2 ? 8 * PF * (CT / 2) * 4096 : 0, wide = has_wide_border(a) ? wide_table_bytes(BC) : 0;
    const int epi_bytes = 4 * KS * (32 * (128 + 16) + PF * 128) + (partial > wide ? partial : wide);
    const int cont = a.cont;
    const int UPP = cont == 2 ? 1 : 2;
    const int PIX_STRIDE = pix_stride(cont);
    const int Hp = a.H + 2 * a.pad;
    const int tiles_c = (a.C_out + BC - 1) / BC;
    // keep the operands of the index arithmetic small
    if ((long long)a.N * a.Ho >= (1 << 22) || (long long)a.N * Hp >= (1 << 22)) return false;
    const int NHo = a.N * a.Ho;
    // a layer whose wave groups each see a single stage never touches the second
    // buffer of a group: leave it out, so that more workgroups fit a CU
    const int nbuf = a.Cp / 64 > KS ? 2 : 1;
    const int e = Hp - a.Ho * a.stride, advance = a.stride + (e < 0 ? e : 0);
    bool found = false;
    long long best_cost = 0;
    // Strip widths that split the row evenly, the full row, or wide strips with a ragged
    // last one, from the widest down.  A plan's cost is led by its number of tiles, which the
    // full row has least of, so nearly all other widths are dismissed by that number alone.
    // Rows that are wider than any patch begin at the widest strip whose R rows fit, and a
    // width is dismissed by the rows that its first tile needs before they are counted exactly
    // (flat wide inputs, 3x4096: 1.7 ms a call without).
    const int widest = (256 * UPT / (UPP * a.R) - a.R) / a.stride + 1;
    for (int TW = a.Wo < widest ? a.Wo : widest; TW >= 1; --TW) {
        const long long strip_pixels = (long long)NHo * TW;
        if (strip_pixels + BP >= (1 << 22)) continue;          // keeps every index well inside 32 bits
        const int tiles_w = (int)((unsigned)(a.Wo + TW - 1) / (unsigned)TW);
        if (TW < 16 && TW != a.Wo && tiles_w * TW != a.Wo) continue;
        const int row_tiles = (int)(((unsigned)strip_pixels + BP - 1) / (unsigned)BP);
        const long long tiles = (long long)tiles_w * row_tiles;
        if ((found && tiles * 100000 > best_cost) || tiles * tiles_c >= (1 << 22)) continue;
        PatchPlan p;
        p.TW = TW; p.BP = BP; p.Hp = Hp; p.tiles_w = tiles_w; p.row_tiles = row_tiles;
        p.PC = (TW - 1) * a.stride + a.R;
        const int least = (row_tiles > 1 ? (BP - 1) / TW * advance : 0) + a.R;
        if (least * p.PC * UPP > 256 * UPT || (found && tiles * 100000 + least * p.PC > best_cost)) continue;
        p.PR = dsq_patch_rows(a, BP, TW, row_tiles);
        // row skew: consecutive tile pixels keep advancing by one pixel stride
        // (mod 256 bytes) when a fragment wraps from one strip row to the next
        int skew = ((TW * a.stride - p.PC) * PIX_STRIDE) % 256;
        if (skew < 0) skew += 256;
        p.RP = p.PC * PIX_STRIDE + (a.stride == 1 ? skew : 0);
        p.buf_bytes = (p.PR * p.RP + 64 + 255) & ~255;   // + dump slot for idle fetch units
        p.units = p.PR * p.PC * UPP;
        if (p.units > 256 * UPT) continue;
        p.aux_off = nbuf * KS * p.buf_bytes > epi_bytes ? nbuf * KS * p.buf_bytes : epi_bytes;
        const int lds_bytes = plan_lds_bytes(p, BC, a);
        if (plan_limit_bytes(p, BC, a) > lds_limit) continue;
        // equal work: prefer a footprint that lets three (else two) workgroups share a CU,
        // then the smaller patch, then the narrower strip
        const long long cost = tiles * 100000 + (lds_bytes <= 52 * 1024 ? 0 : lds_bytes <= 78 * 1024 ? 20000 : 40000) +
                               (long long)p.PR * p.PC;
        if (!found || cost <= best_cost) { best = p; best_cost = cost; found = true; }
    }
    if (!found) return false;
    best.mg_TW = dsq_division_constant(best.TW); best.mg_Hp = dsq_division_constant(Hp); best.mg_Ho = dsq_division_constant(a.Ho);
    best.mg_PC = dsq_division_constant(best.PC); best.mg_tiles_w = dsq_division_constant(best.tiles_w);
    best.step_q = (256 / UPP) / best.PC;
    best.step_r = (256 / UPP) % best.PC;
    return true;
}

struct TileCfg { int WP, WC, PF, CT; };
constexpr TileCfg kSmall  = {4, 1, 1, 2};
constexpr TileCfg kMedium = {2, 2, 2, 2};
constexpr TileCfg kLarge  = {2, 2, 4, 2};
constexpr TileCfg kTall   = {4, 1, 2, 2};
constexpr int kMaxUPT = 12;      // most 16-byte patch units a thread fetches per stage


const TileCfg &tile_cfg(int which)
{
    return which == TILE_LARGE ? kLarge : which == TILE_MEDIUM ? kMedium : which == TILE_TALL ? kTall : kSmall;
}

int pick_tile(const DsqConvArgs &a)
{
    const long long M = (long long)a.N * a.Ho * a.Wo;
    auto blocks = [&](const TileCfg &t) {
        const long long bp = 32 * t.PF * t.WP, bc = 32 * t.CT * t.WC;
        return ((M + bp - 1) / bp) * ((a.C_out + bc - 1) / bc);
    };
    // measured on the five benchmark configs: the 128x128 tile wins whenever it
    // yields enough workgroups (more for 1x1 layers, whose few channel blocks leave
    // nothing for two wave groups to split) and does not waste more than a quarter
    // of its channels; the 256x64 tile when it still runs in two rounds or more;
    // otherwise the 128x64 tile
    const int c_pad = ((a.C_out + 127) / 128) * 128;
    // (a 1x1 layer with at most 64 input channels is one matrix instruction deep:
    // wasted channels cost nothing there, fewer and wider output tiles still pay)
    // Chained layers gain more from fewer tiles: each adds to every pixel's sum, and one that holds all channels
    // stores it, without a clearing launch.  us, 256x64 or 128x64 tile / 128x128, 4 bits: 24 -> 80 1x1 at 56x56 x 64 30.3 / 17.9,
    // 256 -> 80 at 28x28 x 32 9.9 / 7.5, 64 -> 80 3x3 at 56x56 x 64 27.2 / 24.7, 64 -> 144 1x1 at 56x56 x 64 39.5 / 32.3,
    // 100 -> 260 60.8 / 49.0; but 256 -> 144 1x1 at 28x28 x 32 11.5 / 11.7, and 3x3 layers of more than 128 channels
    // pay for every wasted one: 64 -> 144 at 56x56 x 64 35.5 / 42.8.
    const bool wide = a.rq ? a.C_out <= 128 || (a.R == 1 && a.Cp <= 128) : a.R == 1 && a.Cp <= 64;
    const int waste_limit = wide ? 2 : 4;
    if (a.C_out > 64 && waste_limit * (c_pad - a.C_out) <= c_pad && blocks(kMedium) >= (a.R == 1 ? 320 : 192)) {
        // 2-bit layers (FP4 path: the 256x128 tile fits its registers): take that
        // tile when the 128x128 one leaves a nearly empty last round of workgroups
        // (3 per CU, 768 at a time) and the large one (2 per CU, 512) does not
        if (a.cont == 2) {
            const double bm = (double)blocks(kMedium), bl = (double)blocks(kLarge);
            const double waste_m = (double)((blocks(kMedium) + 767) / 768 * 768) / bm;
            const double waste_l = (double)((blocks(kLarge) + 511) / 512 * 512) / bl;
            if (bl >= 256 && waste_m > 1.35 * waste_l) return TILE_LARGE;
            // deep 3x3 layers with about one workgroup per CU (256 -> 256 at 14x14 x 64,
            // 512 -> 512 at 14x14 x 32): the 256x64 tile with one wave group measured 6-10 %
            // ahead of the 128x128 tile with two (plain call; the chained call measures the other way)
            if (!a.rq && a.R == 3 && a.stride == 1 && a.Cp >= 256 && !a.many_in_flight && blocks(kMedium) <= 320 &&
                blocks(kTall) >= 192)
                return TILE_TALL;
        }
        return TILE_MEDIUM;
    }
    if (blocks(kTall) >= 1536) return TILE_TALL;      // at least two rounds of workgroups; else finer tiles
    return TILE_SMALL;
}

constexpr int kLdsLimit = 150 * 1024;
static_assert(kLdsLimit + border_table_bytes(3, 128) <= 160 * 1024, "the tables for l_a != 0 fit beside the largest patch");

}  // namespace

namespace {

// Tile, wave-group count and plan for a layer.  Two wave groups (K split inside
// the workgroup) only pay when the layer yields about one workgroup per CU.
bool choose_plan(const DsqConvArgs &a, int force_tile, int &which, int &ks, PatchPlan &pl)
{
    if ((long long)a.N * a.H * a.W * (a.Cp * a.cont / 8) > 0x7FFFFFFFLL) return false;
    which = force_tile >= 0 ? force_tile : pick_tile(a);
    // chained mode: the 256x128 tile has a variant for 2-bit containers only (at 3 and
    // 4 bits it does not fit the registers), and layers with l_a != 0 (border-dependent
    // terms) go to the split-K kernel for few output tiles or the simple kernel
    if (a.rq && ((which == TILE_LARGE && a.cont != 2) || a.l_a != 0.0f)) return false;
    const TileCfg &tc = tile_cfg(which);
    const int BP = 32 * tc.PF * tc.WP, BC = 32 * tc.CT * tc.WC;
    const long long M = (long long)a.N * a.Ho * a.Wo;
    const long long blocks = ((M + BP - 1) / BP) * ((a.C_out + BC - 1) / BC);
    // (with several calls in flight the CUs are shared by workgroups of different calls
    // anyway, and one wave group per workgroup -- half the LDS, no exchange of partial
    // sums -- gives the higher throughput: measured +9 % on config 2 with four in flight)
    ks = (!a.many_in_flight && (which == TILE_SMALL || which == TILE_MEDIUM) && a.Cp >= 128 && blocks <= 320) ? 2 : 1;
    if (ks == 2 && plan_patch(a, BP, BC, tc.PF, tc.CT, kMaxUPT, kLdsLimit, 2, pl)) return true;
    ks = 1;
    return plan_patch(a, BP, BC, tc.PF, tc.CT, kMaxUPT, kLdsLimit, 1, pl);
}

}  // namespace

int dsq_conv_patch_describe(const DsqConvArgs &a, int force_tile, char *text, size_t n)
{
    int which, ks;
    PatchPlan pl;
    if (!choose_plan(a, force_tile, which, ks, pl)) return 0;
    const TileCfg &tc = tile_cfg(which);
    const int BC = 32 * tc.CT * tc.WC;
    const int need = (pl.units + 255) / 256;
    const int upt = need <= 2 ? 2 : need <= 4 ? 4 : need <= 8 ? 8 : 12;
    const int blocks = pl.tiles_w * pl.row_tiles * ((a.C_out + BC - 1) / BC);
    snprintf(text, n, "patch kernel: container %d, %dx%d filter, tile %dx%d (pixels x channels), %d wave group%s, "
             "%d fetch units per thread%s; strip width %d, patch %dx%d, %d workgroups, %d LDS bytes",
             a.cont, a.R, a.R, 32 * tc.PF * tc.WP, BC, ks, ks == 1 ? "" : "s", upt,
             a.rq ? ", chained epilogue" : "", pl.TW, pl.PR, pl.PC, blocks, plan_lds_bytes(pl, BC, a));
    return 1;
}

bool dsq_launch_conv_patch(const DsqConvArgs &args, int force_tile, hipStream_t stream, hipError_t &status)
{
    int which, ks;
    PatchPlan pl;
    if (!choose_plan(args, force_tile, which, ks, pl)) return false;
    DsqConvArgs a = args;
    if (a.rq) {
        // Next layer's pixel sums: a layer no wider than the tile has each pixel's
        // sum complete in one workgroup, which stores it; otherwise the workgroups
        // add to sums that a fill kernel clears first.
        const TileCfg &tc = tile_cfg(which);
        a.rq_store = a.C_out <= 32 * tc.CT * tc.WC;
        a.rq_share = a.rq_store || a.R == 1;
    }
    const int need = (pl.units + 255) / 256;      // fetch units per thread: instantiated 2, 4, 8, 12
    switch (2 * a.cont + (a.R == 3 ? 0 : 1)) {
    case 8: status = dsq_conv_patch_c4r3(a, pl, which, ks, need, stream); break;
    case 9: status = dsq_conv_patch_c4r1(a, pl, which, ks, need, stream); break;
    case 6: status = dsq_conv_patch_c3r3(a, pl, which, ks, need, stream); break;
    case 7: status = dsq_conv_patch_c3r1(a, pl, which, ks, need, stream); break;
    case 4: status = dsq_conv_patch_c2r3(a, pl, which, ks, need, stream); break;
    default: status = dsq_conv_patch_c2r1(a, pl, which, ks, need, stream); break;
    }
    return true;
}
