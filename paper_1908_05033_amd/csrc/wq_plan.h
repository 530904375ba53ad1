// Plan of a dsq_conv2d_wq launch: LDS layout, tiles and strip width (host arithmetic only; the
// kernel shares the layout's constants).
#pragma once
#include "patch_plan.h"

#if defined(__HIPCC__)
#define DSQ_BOTH __host__ __device__
#else
#define DSQ_BOTH
#endif

namespace {

struct WqPlan {
    int TW, PC, npx;           // strip width; patch columns, patch pixels (1x1: the tile's pixels)
    int Hp, tiles_w, tiles_c, total_blocks, xcd_chunk;
    uint32_t mg_TW, mg_PC, mg_Hp, mg_Ho, mg_tiles_w, mg_tiles_c;
};

DSQ_BOTH constexpr int kc_of(int R) { return R == 3 ? 32 : 64; }              // channels per stage
DSQ_BOTH constexpr int pixel_bytes(int R) { return kc_of(R) * 6 + 16; }       // odd multiple of 16: 8 pixels in distinct banks
constexpr int ROWB = 128 + 16;                                       // staged bytes per output pixel

// LDS: [patch, then the epilogue's staging][channel-group sums of x][patch addresses]
//      [zq, Dw * 2^-54, lr of BC channels][whether the tile cannot be split, whether any lr is not 0]
DSQ_BOTH constexpr int tables_at(int R, int KW, int tiles, int npx)
{
    const int staging = KW > 1 ? KW * tiles * 4096 : 4 * 32 * ROWB;      // (tiles: 32x32 tiles of a wave)
    return npx * pixel_bytes(R) > staging ? npx * pixel_bytes(R) : staging;
}
constexpr int lds_bytes(int R, int KW, int tiles, int BC, int npx)
{
    return tables_at(R, KW, tiles, npx) + npx * (kc_of(R) / 8 * 4 + 4) + 3 * BC * 4 + 16;
}

struct WqTile { int BP, BC, KW, tiles; };
constexpr WqTile kSquare = {64, 64, 1, 1}, kRow = {64, 128, 1, 2}, kLarge = {128, 128, 1, 4}, kNarrow = {128, 32, 1, 1},
                 kSplit = {32, 32, 4, 1};

// Strip width: the patch costs about 8/54 of a tile pixel's matrix work per patch
// pixel, and its LDS bytes decide how many workgroups share a CU.  Rows wider than any
// patch begin at the widest strip that fits, and a width is dismissed by the patch that
// its first tile needs before its patch is counted exactly: at most 6 us a call at 224x224
// and 9 at 3x4096 (5 and 96 to 242 with every width counted).
inline bool plan_wq(const DsqConvArgs &a, const WqTile &t, WqPlan &best, int &lds)
{
    const int NHo = a.N * a.Ho, Hp = a.H + 2 * a.pad;
    constexpr int kMostPixels = 1024, kMostBytes = 150 * 1024;
    const int widest = (kMostPixels / 3 - 3) / a.stride + 1;            // (R = 3: a patch has 3 rows at least)
    double best_cost = 0.0;
    bool found = false;
    for (int TW = a.R == 1 || a.Wo < widest ? a.Wo : widest; TW >= 1; --TW) {
        if (a.R == 1 && TW != a.Wo) break;
        const int tiles_w = (a.Wo + TW - 1) / TW;
        const long long strip = (long long)NHo * TW;
        const int row_tiles = (int)((strip + t.BP - 1) / t.BP);
        const double tiles = (double)tiles_w * row_tiles;
        if (found && tiles * t.BP * 54 > best_cost) continue;
        WqPlan p;
        p.TW = TW; p.Hp = Hp; p.tiles_w = tiles_w;
        p.PC = a.R == 1 ? 1 : (TW - 1) * a.stride + a.R;
        if (a.R != 1) {
            const int least = ((row_tiles > 1 ? (t.BP - 1) / TW * a.stride : 0) + a.R) * p.PC;
            if (least > kMostPixels || (found && tiles * ((double)t.BP * 54 + (double)least * 8) >= best_cost)) continue;
        }
        const long long npx = a.R == 1 ? t.BP : (long long)dsq_patch_rows(a, t.BP, TW, row_tiles) * p.PC;
        if (npx > kMostPixels) continue;
        p.npx = (int)npx;
        const int bytes = lds_bytes(a.R, t.KW, t.tiles, t.BC, p.npx);
        if (bytes > kMostBytes) continue;
        const double cost = tiles * ((double)t.BP * 54 + (double)p.npx * 8) *
                            (bytes <= 53 * 1024 ? 1.0 : bytes <= 80 * 1024 ? 1.15 : 1.6);
        if (!found || cost < best_cost) {
            found = true; best_cost = cost; best = p; lds = bytes;
            best.total_blocks = (int)(tiles_w * (long long)row_tiles);
        }
    }
    if (!found) return false;
    best.tiles_c = (a.C_out + t.BC - 1) / t.BC;
    const long long total = (long long)best.total_blocks * best.tiles_c;
    if (total > 0x7FFFFF00LL / 8) return false;
    best.total_blocks = (int)total;
    best.xcd_chunk = (best.total_blocks + 7) / 8;
    best.mg_TW = dsq_division_constant(best.TW); best.mg_PC = dsq_division_constant(best.PC);
    best.mg_Hp = dsq_division_constant(best.Hp); best.mg_Ho = dsq_division_constant(a.Ho);
    best.mg_tiles_w = dsq_division_constant(best.tiles_w); best.mg_tiles_c = dsq_division_constant(best.tiles_c);
    return true;
}

}  // namespace
